// Discrete Fourier transforms of a line held in LDS, for the spectral form of
// the band operator (psoam_spectral.hip).
//
// A line of n points, n = r_1 r_2 ... r_s, is transformed for 16 neighbouring
// columns at once: a workgroup's threads are 16 lanes (columns, adjacent in
// memory) x 16 rows (butterflies), so every access to HBM is 16 lanes x 8
// bytes = one 128-byte line and every LDS row is 128 bytes.  (24 rows, which
// divide the butterflies of 360 points evenly, ran the residual's transforms
// in 7.9 instead of 7.2 ms at 320 x 320 x 128 and in 0.86 instead of 0.51 ms at
// 128 x 128 x 64: fewer workgroups overlap their barriers and loads.  Radices
// stop at 10 for the same reason: with 12 and 16 the kernels hold a third
// more registers, 0.61 ms for the latter.)  Decimation in
// frequency, in place: stage i runs r_i-point butterflies over the leading
// digit of the index left and multiplies by the twiddles, so the array ends
// in digit-reversed order and each butterfly reads and writes its own
// locations (one barrier between stages).  The first stage takes its points
// from a functor (HBM) and the last one hands its results to one, so a
// transform touches LDS s - 1 times.  The transposed order (decimation in
// time: digit-reversed in, natural out) starts where the other ended, which
// lets a line be transformed back, changed and transformed again with the
// middle two butterflies in registers.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

// Every multiply-add of a transform is written out: left to the compiler, two
// kernels with the same transform could round differently (the residual with
// and without the objective's recurrence gives the same iterates, bit for bit).
#pragma clang fp contract(off)

namespace psoam {

constexpr int kFftLanes = 16;   // columns of a workgroup
constexpr int kFftRows = 16;    // butterflies in flight
constexpr int kFftThreads = kFftLanes * kFftRows;
constexpr int kFftMaxStages = 4;

struct FftDim {
  int n = 0, ns = 0;
  int rad[kFftMaxStages] = {1, 1, 1, 1};
  const float2* tw = nullptr;   // [n] exp(-2 pi i j / n)
  int m[kFftMaxStages] = {1, 1, 1, 1};  // n / (r_0 ... r_i): between a butterfly's points
  void derive() {
    for (int i = 0, p = 1; i < ns; ++i) m[i] = n / (p *= rad[i]);
  }
  // largest byte offset of a butterfly's first point on a line of this pitch
  size_t reach(size_t pitch) const {
    return (size_t)std::max(m[0], n / rad[ns - 1]) * pitch + 128;
  }
};

namespace fft {

constexpr double kPi = 3.14159265358979323846;
constexpr double csin_(double x) {  // |x| <= pi
  double t = x, s = x;
  for (int k = 1; k < 24; ++k) {
    t *= -x * x / ((2 * k) * (2 * k + 1));
    s += t;
  }
  return s;
}
constexpr double ccos_(double x) {
  double t = 1.0, s = 1.0;
  for (int k = 1; k < 24; ++k) {
    t *= -x * x / ((2 * k - 1) * (2 * k));
    s += t;
  }
  return s;
}
// exp(SIGN 2 pi i j / R), 0 <= j < R
constexpr double ang_(int j, int r) {
  return 2.0 * kPi * (2 * j > r ? j - r : j) / r;
}
template <int R, int J>
struct Tw {
  static constexpr float c = (float)ccos_(ang_(J % R, R));
  static constexpr float s = (float)csin_(ang_(J % R, R));
};

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return {a.x - b.x, a.y - b.y}; }
// a (wr + i wi)
// a + f b
__device__ __forceinline__ float2 cfma(float f, float2 b, float2 a) {
  return {__builtin_fmaf(f, b.x, a.x), __builtin_fmaf(f, b.y, a.y)};
}
__device__ __forceinline__ float2 cmul(float2 a, float wr, float wi) {
  return {__builtin_fmaf(a.x, wr, -(a.y * wi)), __builtin_fmaf(a.x, wi, a.y * wr)};
}
// SIGN i a
template <int SIGN>
__device__ __forceinline__ float2 muli(float2 a) {
  return SIGN > 0 ? float2{-a.y, a.x} : float2{a.y, -a.x};
}

template <int R, int SIGN>
struct Dft;

template <int SIGN>
struct Dft<2, SIGN> {
  static __device__ __forceinline__ void run(float2* v) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};
template <int SIGN>
struct Dft<3, SIGN> {
  static __device__ __forceinline__ void run(float2* v) {
    const float2 s = cadd(v[1], v[2]), d = muli<SIGN>(csub(v[1], v[2]));
    constexpr float h = Tw<3, 1>::s;
    const float2 m = cfma(-0.5f, s, v[0]);
    v[0] = cadd(v[0], s);
    v[1] = cfma(h, d, m);
    v[2] = cfma(-h, d, m);
  }
};
template <int SIGN>
struct Dft<4, SIGN> {
  static __device__ __forceinline__ void run(float2* v) {
    const float2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
    const float2 c = cadd(v[1], v[3]), d = muli<SIGN>(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
  }
};
template <int SIGN>
struct Dft<5, SIGN> {
  static __device__ __forceinline__ void run(float2* v) {
    constexpr float c1 = Tw<5, 1>::c, c2 = Tw<5, 2>::c, s1 = Tw<5, 1>::s, s2 = Tw<5, 2>::s;
    const float2 a = cadd(v[1], v[4]), b = cadd(v[2], v[3]);
    const float2 d = muli<SIGN>(csub(v[1], v[4])), e = muli<SIGN>(csub(v[2], v[3]));
    const float2 m1 = cfma(c2, b, cfma(c1, a, v[0]));
    const float2 m2 = cfma(c1, b, cfma(c2, a, v[0]));
    const float2 n1 = cfma(s2, e, {s1 * d.x, s1 * d.y});
    const float2 n2 = cfma(-s1, e, {s2 * d.x, s2 * d.y});
    v[0] = cadd(v[0], cadd(a, b));
    v[1] = cadd(m1, n1);
    v[2] = cadd(m2, n2);
    v[3] = csub(m2, n2);
    v[4] = csub(m1, n1);
  }
};
// n = n1 R2 + n2, k = k1 + R1 k2: R2 transforms of R1 points, the twiddles
// exp(SIGN 2 pi i k1 n2 / R), R1 transforms of R2 points
template <int R1, int R2, int SIGN, int K1 = 0, int N2 = 0>
__device__ __forceinline__ void inner_twiddle(float2* a) {
  if constexpr (K1 < R1) {
    if constexpr (K1 * N2 != 0) {
      using T = Tw<R1 * R2, K1 * N2>;
      a[K1 * R2 + N2] = cmul(a[K1 * R2 + N2], T::c, SIGN > 0 ? T::s : -T::s);
    }
    if constexpr (N2 + 1 < R2) inner_twiddle<R1, R2, SIGN, K1, N2 + 1>(a);
    else inner_twiddle<R1, R2, SIGN, K1 + 1, 0>(a);
  }
}
template <int R1, int R2, int SIGN>
__device__ __forceinline__ void dft2d(float2* v) {
  float2 a[R1 * R2];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
    float2 t[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) t[n1] = v[n1 * R2 + n2];
    Dft<R1, SIGN>::run(t);
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) a[k1 * R2 + n2] = t[k1];
  }
  inner_twiddle<R1, R2, SIGN>(a);
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) {
    Dft<R2, SIGN>::run(a + k1 * R2);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) v[k1 + R1 * k2] = a[k1 * R2 + k2];
  }
}
#define PSOAM_DFT2D(R, R1, R2)                                                    \
  template <int SIGN>                                                             \
  struct Dft<R, SIGN> {                                                           \
    static __device__ __forceinline__ void run(float2* v) { dft2d<R1, R2, SIGN>(v); } \
  };
PSOAM_DFT2D(6, 2, 3)
PSOAM_DFT2D(8, 2, 4)
PSOAM_DFT2D(9, 3, 3)
PSOAM_DFT2D(10, 2, 5)
#undef PSOAM_DFT2D

// twiddle j of the forward table, conjugated for SIGN > 0
template <int SIGN>
__device__ __forceinline__ float2 twmul(float2 a, float2 w) {
  return cmul(a, w.x, SIGN > 0 ? -w.y : w.y);
}

// runs f with the stage's radix as a compile-time constant
template <class F>
__device__ __forceinline__ void with_radix(int r, F&& f) {
  switch (r) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    default: f(std::integral_constant<int, 10>{}); break;
  }
}

// a line's place in LDS: [n][16] points, then the twiddles [n]
struct Lds {
  float2* a;
  float2* tw;
};
__device__ __forceinline__ Lds carve(unsigned char* raw, const FftDim& D) {
  Lds L{(float2*)raw, (float2*)raw + (size_t)D.n * kFftLanes};
  for (int i = (int)threadIdx.x; i < D.n; i += kFftThreads) L.tw[i] = D.tw[i];
  return L;
}

// Integer arithmetic costs as much as the transform where it is left to 64-bit
// and 32-bit multiplies (a quarter of the rate) and divisions: indices below
// fit 24 bits, a division is a float multiply (exact for b < 2^20, the reciprocal
// being good to an ulp: (b + 1/2) / m is 1/2m away from the next integer), and a point in memory is a scalar base
// plus a 32-bit offset that a butterfly computes once.  That and the cheaper
// marks took a third of the vector instructions out, and tiles that share lines
// on one XCD a third of the reads; us before and after at 320 x 320 x 128 (256
// samples, 40 pulses; two pulses an image then): residual 3660 -> 3150, y ->
// spectrum 2440 -> 2115, spectrum -> y 2500 -> 1990, S c 1500 -> 1205; at 128 x
// 128 x 64 (160 samples, 32 pulses) 330 -> 340, 196 -> 178, 214 -> 194 and 104 ->
// 73.  With a pulse's own pairs: residual 3350 and S c 1325 at the larger size,
// 298, 150, 196 and 82 at the smaller, at 4.1 and 4.1, 5.6, 3.8 and 2.2 TB/s
// (a copy's 4.9; what the cache behind L2 holds comes faster).
__device__ __forceinline__ int mul24(int a, int b) { return (int)__umul24((unsigned)a, (unsigned)b); }
__device__ __forceinline__ float inv_of(int m) { return __builtin_amdgcn_rcpf((float)m); }
__device__ __forceinline__ int div_by(int b, float inv) { return (int)(((float)b + 0.5f) * inv); }
template <class T>
__device__ __forceinline__ T& lds_at(T* base, unsigned byte) {
  return *(T*)((char*)base + byte);
}

// natural index of the first output (q = 0) of butterfly b of the last stage
__device__ __forceinline__ int rev_index(const FftDim& D, int nb, int b) {
  int k = 0, w = nb;  // r1 ... r_{s-1}
  // b = ((k1 r2 + k2) r3 + k3): peel the last digit first
  for (int i = D.ns - 2; i >= 0; --i) {
    const int r = D.rad[i];
    const float inv = inv_of(r);
    const int q = div_by(b, inv);
    w = div_by(w, inv);
    k += mul24(w, b - mul24(q, r));
    b = q;
  }
  return k;
}

// Byte offsets of points i0 + q step (q < R) on a line of n points `pitch`
// bytes apart; those past the end are its last point's.  lane: this lane's
// offset at a point.
template <int R>
__device__ __forceinline__ void offsets(unsigned pitch, unsigned lane, int i0, int step, int n,
                                        unsigned (&off)[R]) {
  const unsigned o = (unsigned)i0 * pitch;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int c = q * step < n ? q * step : n - 1;
    const unsigned last = (unsigned)(n - 1 - c) * pitch;
    off[q] = (o < last ? o : last) + (unsigned)c * pitch + lane;
  }
}
template <class T>
__device__ __forceinline__ T& at(T* base, unsigned byte) {
  return *(T*)((char*)base + byte);
}
template <class T>
__device__ __forceinline__ const T& at(const T* base, unsigned byte) {
  return *(const T*)((const char*)base + byte);
}

// stage 0 of the natural-order side: load(radix, first index, step, points)
// fills a butterfly's points, so that it can issue all their loads before it
// looks at any (a branch between two loads makes each wait for the one
// before); barriers: one before (the twiddles are in LDS) and one after, which
// late() precedes
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <int SIGN, class Load, class Late = Nothing>
__device__ __forceinline__ void first_stage(const FftDim& D, const Lds& L, Load&& load,
                                            Late&& late = Nothing{}) {
  const int lane = threadIdx.x & 15, row = threadIdx.x >> 4;
  __syncthreads();
  with_radix(D.rad[0], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int m = D.m[0];
    const unsigned mb = (unsigned)m * (kFftLanes * sizeof(float2));
    for (int b = row; b < m; b += kFftRows) {
      float2 v[R];
      load(rc, b, m, v);
      Dft<R, SIGN>::run(v);
      float2* a = L.a + b * kFftLanes + lane;
      unsigned t = 0;
#pragma unroll
      for (int q = 0; q < R; ++q, t += 8u * b)
        lds_at(a, q * mb) = q ? twmul<SIGN>(v[q], lds_at(L.tw, t)) : v[q];
    }
  });
  late();
  __syncthreads();
}

// points of a strided line in HBM (base: its first column, lane: this lane's
// byte offset; those from index n on are zero); FULL: n is the line's length
template <bool FULL>
__device__ __forceinline__ auto strided(const float2* base, unsigned pitch, int n, unsigned lane) {
  return [=](auto rc, int i0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    const unsigned o = (unsigned)i0 * pitch;
    if constexpr (FULL) {
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = at(base + (size_t)(q * step) * (pitch / 8), o + lane);
    } else {
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int c = q * step < n ? q * step : n - 1;
        // (a plane may pass 4 GiB, a butterfly's first point does not)
        const size_t end = (size_t)(n - 1 - c) * pitch;
        const unsigned last = end < 0xffffff00u ? (unsigned)end : 0xffffff00u;
        v[q] = at(base + (size_t)c * (pitch / 8), (o < last ? o : last) + lane);
      }
#pragma unroll
      for (int q = 0; q < R; ++q)
        if (i0 >= n - q * step) v[q] = {0.0f, 0.0f};
    }
  };
}

// stages 1 .. ns - 2, in place; DIT applies the twiddles before the butterfly
template <int SIGN, bool DIT>
__device__ __forceinline__ void middle_stage(const FftDim& D, const Lds& L, int s, int p) {
  // p = r_0 ... r_{s-1}
  const int lane = threadIdx.x & 15, row = threadIdx.x >> 4;
  with_radix(D.rad[s], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int m = D.m[s], nb = p * m, p8 = 8 * p;
    const float inv = inv_of(m);
    const unsigned mb = (unsigned)m * (kFftLanes * sizeof(float2));
    for (int b = row; b < nb; b += kFftRows) {
      // block b / m of R m points, point j of it
      const int blk = div_by(b, inv), skip = mul24(blk, m), j = b - skip;
      float2* a = L.a + (b + skip * (R - 1)) * kFftLanes + lane;
      const unsigned tj = (unsigned)mul24(p8, j);
      float2 v[R];
      unsigned t = 0;
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = lds_at(a, q * mb);
      if constexpr (DIT) {
#pragma unroll
        for (int q = 1; q < R; ++q) v[q] = twmul<SIGN>(v[q], lds_at(L.tw, t += tj));
      }
      Dft<R, SIGN>::run(v);
#pragma unroll
      for (int q = 0; q < R; ++q)
        lds_at(a, q * mb) = (!DIT && q) ? twmul<SIGN>(v[q], lds_at(L.tw, t += tj)) : v[q];
    }
  });
  __syncthreads();
}

template <int SIGN>
__device__ __forceinline__ void middle_stages(const FftDim& D, const Lds& L) {
  int p = D.rad[0];
  for (int s = 1; s < D.ns - 1; ++s) {
    middle_stage<SIGN, false>(D, L, s, p);
    p *= D.rad[s];
  }
}

// last stage: store(radix, natural index of the first result, step, results)
template <int SIGN, class Store>
__device__ __forceinline__ void last_stage(const FftDim& D, const Lds& L, Store&& store) {
  const int lane = threadIdx.x & 15, row = threadIdx.x >> 4;
  with_radix(D.rad[D.ns - 1], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int nb = D.n / R;
    for (int b = row; b < nb; b += kFftRows) {
      const float2* a = L.a + b * R * kFftLanes + lane;
      float2 v[R];
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = a[q * kFftLanes];
      Dft<R, SIGN>::run(v);
      store(rc, rev_index(D, nb, b), nb, v);
    }
  });
}

// results of a strided line in HBM, those before index n; ok: the lane has a
// column
template <bool FULL>
__device__ __forceinline__ auto strided_out(float2* base, unsigned pitch, int n, bool ok) {
  const unsigned lane = (threadIdx.x & 15) * 8;
  return [=](auto rc, int i0, int step, const float2* v) {
    constexpr int R = decltype(rc)::value;
    const unsigned o = (unsigned)i0 * pitch + lane;
    if (!ok) return;
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (FULL || i0 < n - q * step) at(base + (size_t)(q * step) * (pitch / 8), o) = v[q];
  };
}

// the last stage of an inverse transform, change(natural index, values of the
// butterfly) and the first stage of the forward transform that follows
template <class Change>
__device__ __forceinline__ void turn_stage(const FftDim& D, const Lds& L, Change&& change) {
  const int lane = threadIdx.x & 15, row = threadIdx.x >> 4;
  with_radix(D.rad[D.ns - 1], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int nb = D.n / R;
    for (int b = row; b < nb; b += kFftRows) {
      float2* a = L.a + b * R * kFftLanes + lane;
      float2 v[R];
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = a[q * kFftLanes];
      Dft<R, 1>::run(v);
      change(rc, rev_index(D, nb, b), nb, v);
      Dft<R, -1>::run(v);
#pragma unroll
      for (int q = 0; q < R; ++q) a[q * kFftLanes] = v[q];
    }
  });
  __syncthreads();
}

// forward stages from the digit-reversed side: ns - 2 .. 1 in LDS, stage 0
// to store (as last_stage's)
template <class Store>
__device__ __forceinline__ void dit_stages(const FftDim& D, const Lds& L, Store&& store) {
  for (int s = D.ns - 2; s >= 1; --s)
    middle_stage<-1, true>(D, L, s, (int)((unsigned)D.n / (unsigned)(D.m[s] * D.rad[s])));
  const int lane = threadIdx.x & 15, row = threadIdx.x >> 4;
  with_radix(D.rad[0], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int m = D.m[0];
    const unsigned mb = (unsigned)m * (kFftLanes * sizeof(float2));
    for (int b = row; b < m; b += kFftRows) {
      float2* a = L.a + b * kFftLanes + lane;
      float2 v[R];
      unsigned t = 0;
#pragma unroll
      for (int q = 0; q < R; ++q, t += 8u * b) {
        v[q] = lds_at(a, q * mb);
        if (q) v[q] = twmul<-1>(v[q], lds_at(L.tw, t));
      }
      Dft<R, -1>::run(v);
      store(rc, b, m, v);
    }
  });
}

}  // namespace fft
}  // namespace psoam
