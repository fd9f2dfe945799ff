// Spectral form of the band operator.
//
// H is a correlation over the lateral offsets (dy, dx) for every (sample,
// depth) pair (eqs. q-above-1d, q-below-1d: the impulse response is the same
// at every scan position), so on a lateral grid padded to NY >= Ny + R, NX >=
// Nx + R points it is diagonal in the lateral frequency kappa:
//     Y(kappa)[t][k] = sum_z T(kappa)[t][z] B(kappa)[z][k],
//     T(kappa)[t][z] = sum_{dy,dx} h[z][dy][dx][t] e^{+2 pi i (kappa_y dy / NY + kappa_x dx / NX)},
// and H^T multiplies by conj(T)^T.  (Offsets reach at most R past the grid
// and outputs past Ny, Nx are dropped, so a period of Ny + R, not Ny + 2 R,
// keeps the wrapped images apart.)  The direct form spends 2 nnz K Nx Ny
// operations on a band that fills a quarter of its matrix-core tiles; this
// one spends the transforms (~40 operations a point and axis) and one product
// per frequency with the 16 x 16 blocks of (t, z) that the band meets at any
// offset (15% of them at 320 x 320 x 128).
//
// All arithmetic is float32 (transforms on the vector units, products on
// v_mfma_f32_16x16x4_f32); the table is summed in FP64.  A 16-bit plan's
// operands and table are rounded exactly as the direct form rounds them and
// then carried in float32, so every precision keeps its meaning.
//
// Two pulses share one complex image (real and imaginary part): H is real, so
// the pair goes through the transforms unseparated; the product takes kappa
// and -kappa together and separates them in registers.
//
//   spec_x_switch   S c (or phi c), rounded, pairs packed, transform along x
//   spec_y          transform along y (forward, or inverse onto the grid)
//   spec_gemm_fwd   T B per frequency
//   spec_x_out      inverse along x, y written
//   spec_x_resid    inverse along x, r = y - p, rounded, transform along x
//   spec_x_pack     y -> rounded, transform along x (the external adjoint)
//   spec_gemm_adj   conj(T)^T R per frequency, and S^T for a per-depth fluence
//   spec_x_vox      inverse along x, c (or the pulse volumes) written
//   spec_st         S^T for a per-voxel fluence
//   spec_reach      which outputs nonzero and non-finite operand values reach
//
// The transforms and the products are bound by HBM: at 320 x 320 x 128 (40
// pulses, 512 samples of which band entries meet 256, 360 x 360 frequencies) a
// spectrum of y is 5.3 GB and the table 5 GB.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "psoam_internal.h"
#include "psoam_fft.h"

namespace psoam {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

// rounding of an operand value: the 16-bit value the direct form would store
enum Rnd { kRndNone = 0, kRndBf16 = 1, kRndF16 = 2 };
template <int RND>
__device__ __forceinline__ float rnd(float v, float sc, float inv) {
  if constexpr (RND == kRndBf16) return (float)(__bf16)v;
  else if constexpr (RND == kRndF16) return (float)(_Float16)(v * sc) * inv;
  else return v;
}
__device__ __forceinline__ bool finite_(float v) { return fabsf(v) <= 3.402823466e38f; }

__device__ __forceinline__ float spec_coef(const SwitchParams& sw, float phi, int k, int s) {
  if (sw.diag) return k == s ? phi : 0.0f;
  const float pg = (sw.gamma == 0.0f) ? 1.0f : powf(phi, sw.gamma);
  return phi * __builtin_fmaf(sw.b[s], expf(-(float)k * pg * sw.inv_tau[s]), sw.a[s]);
}

// Where the operand is not zero, and where it is not finite.  A transform
// spreads its rounding over the whole image, and a value that is not finite
// over all of it; the direct form reaches a footprint.  So every pass that
// makes an operand marks its positions, spec_reach widens the marks by the
// footprint, and the pass that writes the result writes zero where no nonzero
// value reaches and NaN where a non-finite one does (such a value enters the
// transforms as zero).  A mark is the number of the call that set it, so that
// no call sees an older one's; and since a captured call repeats its number,
// the pass that reads the reach last clears the marks it came from (and the
// product before the residual's pass those of r, which an objective leaves
// behind).
struct Marks {
  unsigned* at;         // [planes][Ny][Nx]: a nonzero value
  unsigned* bad;        // the same: a non-finite one
  unsigned char* near;  // the same: bit 0 a nonzero value in reach, bit 1 a non-finite one
  unsigned now;
  int planes;           // 1, or one per pulse (pulse volumes of their own)
};
enum Near { kNearSome = 1, kNearBad = 2 };
// The marks of a workgroup's row collect in LDS (a byte per column x and plane,
// after the line and its twiddles) and go out once, and the reach of a row's
// columns comes in once: a mark or a look at one never waits for HBM.
struct RowMarks {
  unsigned char* hit;  // [2][n]
  signed char* near;   // [2][n]
};
__device__ __forceinline__ RowMarks row_marks(unsigned char* raw, int n) {
  unsigned char* a = raw + (size_t)n * (kFftLanes + 1) * sizeof(float2);
  return RowMarks{a, (signed char*)a + 2 * n};
}
__host__ __device__ constexpr size_t row_lds(int n) {
  return (size_t)n * ((kFftLanes + 1) * sizeof(float2) + 4);
}
// One butterfly's operand values v (R positions x0, x0 + step, ..): the 16
// lanes of a position (a DPP row) join their nonzero bits and lane q writes
// position q's byte (every position belongs to one butterfly); non-finite
// values, which are rare, are marked in HBM and become zero.  two: the planes
// differ.
__device__ __forceinline__ unsigned row_or(unsigned h) {
  h |= (unsigned)__builtin_amdgcn_mov_dpp((int)h, 0x128, 0xf, 0xf, true);  // row_ror:8
  h |= (unsigned)__builtin_amdgcn_mov_dpp((int)h, 0x124, 0xf, 0xf, true);
  h |= (unsigned)__builtin_amdgcn_mov_dpp((int)h, 0x122, 0xf, 0xf, true);
  h |= (unsigned)__builtin_amdgcn_mov_dpp((int)h, 0x121, 0xf, 0xf, true);
  return h;
}
template <int R>
__device__ __forceinline__ void mark_points(const RowMarks& W, int n, const Marks& M, size_t row0,
                                            size_t row1, bool two, int x0, int step, float2* v) {
  const int lane = threadIdx.x & 15;
  const int at = x0 + fft::mul24(lane, step);
  bool bad = false;
  unsigned h0 = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    // zero where both are, not finite where either is not (or the sum overflows)
    const float s = fabsf(v[q].x) + fabsf(v[q].y);
    bad |= !finite_(s);
    h0 |= s != 0.0f ? 1u << q : 0u;
  }
  if (two) {
    unsigned h1 = 0;
    h0 = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      h0 |= v[q].x != 0.0f ? 1u << q : 0u;
      h1 |= v[q].y != 0.0f ? 1u << q : 0u;
    }
    h1 = row_or(h1);
    if (lane < R) W.hit[n + at] = (unsigned char)(h1 >> lane & 1u);
  }
  h0 = row_or(h0);
  if (lane < R) W.hit[at] = (unsigned char)(h0 >> lane & 1u);
  if (bad) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (!finite_(v[q].x)) {
        M.bad[row0 + x0 + q * step] = M.now;
        v[q].x = 0.0f;
      }
      if (!finite_(v[q].y)) {
        M.bad[row1 + x0 + q * step] = M.now;
        v[q].y = 0.0f;
      }
    }
  }
}
// The reach of the row's columns as bytes to and a value with: all ones where a
// nonzero value reaches, 0 where none does (and past the grid), kReachBad where
// a non-finite one does.
constexpr signed char kReachBad = 127;
__device__ __forceinline__ signed char reach_of(unsigned char near) {
  return near & kNearBad ? kReachBad : near & kNearSome ? (signed char)-1 : (signed char)0;
}
__device__ __forceinline__ void load_near(const RowMarks& W, int n, const Marks& M, size_t row,
                                          size_t p0, size_t p1, int nx) {
  for (int x = (int)threadIdx.x; x < n; x += kFftThreads) {
    W.near[x] = x < nx ? reach_of(M.near[p0 + row + x]) : (signed char)0;
    if (p1 != p0) W.near[n + x] = x < nx ? reach_of(M.near[p1 + row + x]) : (signed char)0;
  }
}
// a butterfly's results, zero or NaN where the reach says so
template <int R>
__device__ __forceinline__ void reach_points(const RowMarks& W, int n, bool two, int x0, int step,
                                             float2* v) {
  int r0[R], r1[R], most = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) r0[q] = r1[q] = W.near[x0 + q * step];
  if (two) {
#pragma unroll
    for (int q = 0; q < R; ++q) r1[q] = W.near[n + x0 + q * step];
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    most = max(most, max(r0[q], r1[q]));
    v[q].x = __builtin_bit_cast(float, __builtin_bit_cast(int, v[q].x) & r0[q]);
    v[q].y = __builtin_bit_cast(float, __builtin_bit_cast(int, v[q].y) & r1[q]);
  }
  if (most > 0) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (r0[q] > 0) v[q].x = __builtin_nanf("");
      if (r1[q] > 0) v[q].y = __builtin_nanf("");
    }
  }
}
// (after a barrier) marks of the row into planes p0 and, where it differs, p1
__device__ __forceinline__ void store_hits(const RowMarks& W, int n, const Marks& M, size_t row,
                                           size_t p0, size_t p1, int nx) {
  for (int x = (int)threadIdx.x; x < nx; x += kFftThreads) {
    if (W.hit[x] && M.at[p0 + row + x] != M.now) M.at[p0 + row + x] = M.now;
    if (p1 != p0 && W.hit[n + x] && M.at[p1 + row + x] != M.now) M.at[p1 + row + x] = M.now;
  }
}
// a workgroup's row of marks, once per row and plane
__device__ __forceinline__ void clear_row(const Marks& M, size_t row, size_t p0, size_t p1, int nx) {
  for (int x = (int)threadIdx.x; x < nx; x += kFftThreads) {
    M.at[p0 + row + x] = M.bad[p0 + row + x] = 0u;
    if (p1 != p0) M.at[p1 + row + x] = M.bad[p1 + row + x] = 0u;
  }
}

struct Geo {
  int ny, nx, nyp, nxp;  // grid and transform lengths
  int nz, nt, lz, lt;    // depths, samples; transformed depths and samples (multiples of 16)
  int tlo;               // first transformed sample
  int nk, np;            // pulses, pairs
  int r, f;
};

// ------------------------------------------------------------ x transforms
// Block: 16 columns (depths or samples l0 .. l0 + 15) of row iy of pair p.  On
// the grid's side 16 columns are half of a 128-byte line, so neighbouring tiles
// go to one XCD at about the same time: blocks are dealt to the 8 XCDs
// round-robin, so of 8 kNear successive ones kNear neighbours are 8 apart.
struct RowAt {
  int p, iy, l0;
  int b;  // its number in that order
};
constexpr int kTilesNear = 4;
__device__ __forceinline__ RowAt row_at(int ny, int l) {
  int b = (int)blockIdx.x;
  const int g = 8 * kTilesNear, first = b / g * g;
  if (first + g <= (int)gridDim.x) b = first + (b & 7) * kTilesNear + ((b - first) >> 3);
  RowAt a;
  a.b = b;
  const int tiles = l >> 4;
  a.l0 = (b % tiles) * 16;
  b /= tiles;
  a.iy = b % ny;
  a.p = b / ny;
  return a;
}

// where S comes from: the per-depth table, the fluence of each voxel, or
// diagonal switching (pulse volumes)
enum Src { kSrcDepth = 0, kSrcVoxel = 1, kSrcDiag = 2 };
template <int RND, int SRC>
__global__ __launch_bounds__(kFftThreads) void spec_x_switch(
    const float* __restrict__ c, const float* __restrict__ phi, const float* __restrict__ stab_t,
    const float* __restrict__ f16, SwitchParams sw, float2* __restrict__ out, Geo G, FftDim D,
    Marks M, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.lz);
  const RowMarks W = row_marks(raw, D.n);
  const int z = at.l0 + (threadIdx.x & 15);
  const bool zok = z < G.nz;
  const int k0 = 2 * at.p, k1 = k0 + 1;
  // the pulses' mark planes
  const size_t grid = (size_t)G.ny * G.nx, mrow = (size_t)at.iy * G.nx;
  const size_t p0 = M.planes == 1 ? 0 : k0 * grid, p1 = M.planes > k1 ? k1 * grid : p0;
  const size_t vol = (size_t)G.ny * G.nx * G.nz;
  const size_t row = (size_t)at.iy * G.nx * G.nz + at.l0;
  const unsigned pitch = 4u * (unsigned)G.nz, lane = zok ? (threadIdx.x & 15) * 4 : 0,
                 top = 4u * (unsigned)min(15, G.nz - 1 - at.l0);
  const float sc = RND == kRndF16 ? f16[0] : 1.0f, inv = RND == kRndF16 ? f16[1] : 1.0f;
  float w[2][kMaxSpecies];
  if constexpr (SRC == kSrcDepth) {
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      w[0][s] = (zok && s < sw.ns) ? stab_t[((size_t)k0 * sw.ns + s) * G.nz + z] : 0.0f;
      w[1][s] = (zok && s < sw.ns && k1 < G.nk) ? stab_t[((size_t)k1 * sw.ns + s) * G.nz + z] : 0.0f;
    }
  }
  auto load = [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    // points of a volume's row; past the grid they are its last column (their
    // values are dropped)
    unsigned off[R];
    fft::offsets(pitch, lane, top, x0, step, G.nx, off);
    auto get = [&](const float* volume, float (&to)[R]) {
#pragma unroll
      for (int q = 0; q < R; ++q) to[q] = fft::at(volume + row, off[q]);
    };
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = {0.0f, 0.0f};
    if constexpr (SRC == kSrcDiag) {
      const size_t o0 = k0 < sw.ns ? (size_t)k0 * vol : 0, o1 = k1 < sw.ns ? (size_t)k1 * vol : 0;
      float c0[R], c1[R], ph[R];
      get(c + o0, c0);
      get(c + o1, c1);
      if (sw.per_voxel) {
        get(phi, ph);
      } else {
        const float pz = phi[zok ? z : 0];
#pragma unroll
        for (int q = 0; q < R; ++q) ph[q] = pz;
      }
#pragma unroll
      for (int q = 0; q < R; ++q)
        v[q] = {k0 < sw.ns ? ph[q] * c0[q] : 0.0f, k1 < sw.ns ? ph[q] * c1[q] : 0.0f};
    } else if constexpr (SRC == kSrcDepth) {
#pragma unroll
      for (int s = 0; s < kMaxSpecies; ++s)
        if (s < sw.ns) {
          float cv[R];
          get(c + (size_t)s * vol, cv);
#pragma unroll
          for (int q = 0; q < R; ++q) {
            v[q].x = __builtin_fmaf(w[0][s], cv[q], v[q].x);
            v[q].y = __builtin_fmaf(w[1][s], cv[q], v[q].y);
          }
        }
    } else {
      float ph[R];
      get(phi, ph);
      for (int s = 0; s < sw.ns; ++s) {
        float cv[R];
        get(c + (size_t)s * vol, cv);
#pragma unroll
        for (int q = 0; q < R; ++q) {
          v[q].x = __builtin_fmaf(spec_coef(sw, ph[q], k0, s), cv[q], v[q].x);
          v[q].y = __builtin_fmaf(spec_coef(sw, ph[q], k1, s), cv[q], v[q].y);
        }
      }
    }
    // (no pulse k1: its zero weights may have met an infinity)
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool ok = zok && x0 + q * step < G.nx;
      v[q].x = ok ? rnd<RND>(v[q].x, sc, inv) : 0.0f;
      v[q].y = ok && k1 < G.nk ? rnd<RND>(v[q].y, sc, inv) : 0.0f;
    }
    mark_points<R>(W, D.n, M, p0 + mrow, p1 + mrow, p1 != p0, x0, step, v);
  };
  fft::first_stage<-1>(D, L, load);
  store_hits(W, D.n, M, mrow, p0, p1, G.nx);
  fft::middle_stages<-1>(D, L);
  float2* o = out + ((size_t)at.p * G.nyp + at.iy) * G.nxp * G.lz + at.l0;
  fft::last_stage<-1>(D, L, fft::strided_out<true>(o, 8u * G.lz, G.nxp));
}

template <int RND>
__global__ __launch_bounds__(kFftThreads) void spec_x_pack(const float* __restrict__ y,
                                                           const float* __restrict__ f16,
                                                           float2* __restrict__ out, Geo G,
                                                           FftDim D, Marks M,
                                                           const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.lt);
  const RowMarks W = row_marks(raw, D.n);
  const int tl = at.l0 + (threadIdx.x & 15), t = G.tlo + tl;
  const bool tok = t < G.nt;
  const int k0 = 2 * at.p, k1 = k0 + 1;
  const size_t grid = (size_t)G.ny * G.nx, mrow = (size_t)at.iy * G.nx;
  const size_t p0 = M.planes == 1 ? 0 : k0 * grid, p1 = M.planes > k1 ? k1 * grid : p0;
  const float sc = RND == kRndF16 ? f16[2] : 1.0f, inv = RND == kRndF16 ? f16[3] : 1.0f;
  const size_t plane = (size_t)G.ny * G.nx * G.nt;
  const int t0 = G.tlo + at.l0;  // (inside the row: the tiles end with its last sample's)
  const float* y0 = y + (size_t)k0 * plane + (size_t)at.iy * G.nx * G.nt + t0;
  const float* y1 = k1 < G.nk ? y0 + plane : y0;
  const unsigned pitch = 4u * (unsigned)G.nt, lane = tok ? (threadIdx.x & 15) * 4 : 0,
                 top = 4u * (unsigned)min(15, G.nt - 1 - t0);
  // loads past the grid read its last position (their values are dropped)
  auto load = [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    unsigned off[R];
    fft::offsets(pitch, lane, top, x0, step, G.nx, off);
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = {fft::at(y0, off[q]), fft::at(y1, off[q])};
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool ok = tok && x0 + q * step < G.nx;
      v[q].x = ok ? rnd<RND>(v[q].x, sc, inv) : 0.0f;
      v[q].y = ok && k1 < G.nk ? rnd<RND>(v[q].y, sc, inv) : 0.0f;
    }
    mark_points<R>(W, D.n, M, p0 + mrow, p1 + mrow, p1 != p0, x0, step, v);
  };
  fft::first_stage<-1>(D, L, load);
  store_hits(W, D.n, M, mrow, p0, p1, G.nx);
  fft::middle_stages<-1>(D, L);
  float2* o = out + ((size_t)at.p * G.ny + at.iy) * G.nxp * G.lt + at.l0;
  fft::last_stage<-1>(D, L, fft::strided_out<true>(o, 8u * G.lt, G.nxp));
}

// y = H b of the pair's two pulses
__global__ __launch_bounds__(kFftThreads) void spec_x_out(const float2* __restrict__ in,
                                                          float* __restrict__ y, Geo G, FftDim D,
                                                          Marks M, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.lt);
  const int tl = at.l0 + (threadIdx.x & 15), t = G.tlo + tl;
  const int k0 = 2 * at.p, k1 = k0 + 1;
  const RowMarks W = row_marks(raw, D.n);
  const size_t grid = (size_t)G.ny * G.nx, mrow = (size_t)at.iy * G.nx;
  const size_t p0 = M.planes == 1 ? 0 : k0 * grid, p1 = M.planes > k1 ? k1 * grid : p0;
  load_near(W, D.n, M, mrow, p0, p1, G.nx);
  if (at.l0 == 0 && (M.planes > 1 || at.p == 0)) clear_row(M, mrow, p0, p1, G.nx);
  const float2* i = in + ((size_t)at.p * G.nyp + at.iy) * G.nxp * G.lt + at.l0;
  fft::first_stage<1>(D, L, fft::strided<true>(i, 8u * G.lt, G.nxp));
  fft::middle_stages<1>(D, L);
  float* y0 = y + ((size_t)k0 * grid + (size_t)at.iy * G.nx) * G.nt + G.tlo + at.l0;
  float* y1 = y0 + grid * G.nt;
  const unsigned pitch = 4u * (unsigned)G.nt, lane = (threadIdx.x & 15) * 4;
  const bool two = k1 < G.nk;
  fft::last_stage<1>(D, L, [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    reach_points<R>(W, D.n, p1 != p0, x0, step, v);
    const unsigned o = (unsigned)x0 * pitch + lane;
    if (t >= G.nt) return;
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (x0 < G.nx - q * step) {
        const unsigned oq = o + (unsigned)(q * step) * pitch;
        fft::at(y0, oq) = v[q].x;
        if (two) fft::at(y1, oq) = v[q].y;
      }
  });
}

// The residual of the solver: y back on the grid, r = y - p, its FP64 square
// sum per block, and r (rounded as the direct form's H^T operand) transformed
// along x again, the two butterflies on either side of r in registers.  REC:
// also A c of the iterate by the momentum recurrence, whose (A c - p)^2 the
// sums are then (see BandArgs::yc).
// (four workgroups a CU: 128 registers)
template <int RND, bool REC>
__global__ __launch_bounds__(kFftThreads, 4) void spec_x_resid(
    const float2* __restrict__ in, const float* __restrict__ pm, const float* __restrict__ f16,
    float2* __restrict__ out, float* __restrict__ yc, float yc_beta, float yc_inv, int yc_first,
    double* __restrict__ partial, Geo G, FftDim D, Marks M, Marks MR,
    const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  __shared__ double sh[kFftThreads / 64];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.lt);
  const int tl = at.l0 + (threadIdx.x & 15), t = G.tlo + tl;
  const int k0 = 2 * at.p, k1 = k0 + 1;
  const bool two = k1 < G.nk;
  const RowMarks W = row_marks(raw, D.n);
  const size_t grid = (size_t)G.ny * G.nx, mrow = (size_t)at.iy * G.nx;
  const size_t p0 = M.planes == 1 ? 0 : k0 * grid, p1 = M.planes > k1 ? k1 * grid : p0;
  const size_t r0 = MR.planes == 1 ? 0 : k0 * grid, r1 = MR.planes > k1 ? k1 * grid : r0;
  load_near(W, D.n, M, mrow, p0, p1, G.nx);
  if (at.l0 == 0 && (M.planes > 1 || at.p == 0)) clear_row(M, mrow, p0, p1, G.nx);
  const float sc = RND == kRndF16 ? f16[2] : 1.0f, inv = RND == kRndF16 ? f16[3] : 1.0f;
  const float2* i = in + ((size_t)at.p * G.nyp + at.iy) * G.nxp * G.lt + at.l0;
  fft::first_stage<1>(D, L, fft::strided<true>(i, 8u * G.lt, G.nxp));
  fft::middle_stages<1>(D, L);
  const size_t plane = grid * G.nt;
  // the row's samples t0 .. of both pulses (of k0 alone: its own again); loads
  // past the grid read inside it (values dropped)
  const int t0 = G.tlo + at.l0;
  const size_t row0 = ((size_t)k0 * grid + (size_t)at.iy * G.nx) * G.nt + t0,
               row1 = row0 + (two ? plane : 0);
  const bool tok = t < G.nt;
  const unsigned pitch = 4u * (unsigned)G.nt, lane = tok ? (threadIdx.x & 15) * 4 : 0,
                 top = 4u * (unsigned)min(15, G.nt - 1 - t0);
  double ss = 0.0;
  fft::turn_stage(D, L, [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    unsigned off[R];
    fft::offsets(pitch, lane, top, x0, step, G.nx, off);
    float2 pv[R];
    float2 yo[REC ? R : 1];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      auto get = [&](const float* a) {
        return float2{fft::at(a + row0, off[q]), fft::at(a + row1, off[q])};
      };
      pv[q] = {0.0f, 0.0f};
      if (pm) pv[q] = get(pm);
      if constexpr (REC) {
        yo[q] = {0.0f, 0.0f};
        if (!yc_first) yo[q] = get(yc);
      }
    }
    reach_points<R>(W, D.n, p1 != p0, x0, step, v);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool in = tok && x0 < G.nx - q * step;
      const float2 w = {v[q].x, two ? v[q].y : 0.0f};
      if (!two) pv[q].y = 0.0f;
      float2 d = {w.x - pv[q].x, w.y - pv[q].y};
      if constexpr (REC) {
        if (in) {
          float2 n = w;
          if (!yc_first)
            n = {__builtin_fmaf(yc_beta, yo[q].x, w.x) * yc_inv,
                 __builtin_fmaf(yc_beta, yo[q].y, w.y) * yc_inv};
          fft::at(yc + row0, off[q]) = n.x;
          if (two) fft::at(yc + row1, off[q]) = n.y;
          const double e0 = (double)n.x - (double)pv[q].x,
                       e1 = two ? (double)n.y - (double)pv[q].y : 0.0;
          ss += e0 * e0 + e1 * e1;
        }
      } else {
        // (a product of floats is exact in FP64, so its sum rounds once)
        const double e0 = in ? (double)d.x : 0.0, e1 = in ? (double)d.y : 0.0;
        ss += __builtin_fma(e0, e0, e1 * e1);
      }
      d.x = in ? rnd<RND>(d.x, sc, inv) : 0.0f;
      d.y = in ? rnd<RND>(d.y, sc, inv) : 0.0f;
      v[q] = d;
    }
    mark_points<R>(W, D.n, MR, r0 + mrow, r1 + mrow, r1 != r0, x0, step, v);
  });
  store_hits(W, D.n, MR, mrow, r0, r1, G.nx);
  float2* ov = out + ((size_t)at.p * G.ny + at.iy) * G.nxp * G.lt + at.l0;
  fft::dit_stages(D, L, fft::strided_out<true>(ov, 8u * G.lt, G.nxp));
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kFftThreads / 64; ++w) s += sh[w];
    partial[at.b] = s;
  }
}

// The samples no band entry meets (half of them at 320 x 320 x 128 with 512
// samples and at 128 x 128 x 64 with 256) are not transformed: y is zero there,
// H^T does not read them, and the objective takes their p^2.  Bound by memory
// (the zeros are written at 5.5 TB/s: 0.77 ms of 4.2 GB at the larger size).
// With every sample transformed spec_x_resid took 7.2 ms at that size, without
// them 3.6 ms; at the smaller one an A took 1.01 and 0.80 ms, an A^T 0.87 and
// 0.61.
__global__ __launch_bounds__(256) void spec_idle_zero(float* __restrict__ y, size_t rows, int nt,
                                                      int lo, int hi,
                                                      const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  const int idle = nt - (hi - lo);
  const size_t n = rows * idle;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const size_t r = i / idle;
    const int j = (int)(i - r * idle);
    y[r * nt + (j < lo ? j : j + hi - lo)] = 0.0f;
  }
}
// the same where rows and bounds are multiples of four samples
__global__ __launch_bounds__(256) void spec_idle_zero4(f32x4* __restrict__ y, size_t rows, int nt4,
                                                       int lo4, int hi4,
                                                       const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  const unsigned idle = (unsigned)(nt4 - (hi4 - lo4));
  for (size_t r = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += (size_t)gridDim.x * 4)
    for (unsigned j = threadIdx.x & 63; j < idle; j += 64)
      y[r * nt4 + (j < (unsigned)lo4 ? j : j + hi4 - lo4)] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}
constexpr int kIdleSums = 1024;
__global__ __launch_bounds__(256) void spec_idle_sums(const float* __restrict__ pm, size_t rows,
                                                      int nt, int lo, int hi,
                                                      double* __restrict__ partial,
                                                      const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  __shared__ double sh[4];
  double ss = 0.0;
  const int idle = nt - (hi - lo);
  if (pm)
    for (size_t r = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += (size_t)kIdleSums * 4)
      for (int j = threadIdx.x & 63; j < idle; j += 64) {
        const double v = (double)pm[r * nt + (j < lo ? j : j + hi - lo)];
        ss += v * v;
      }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// c-side output of H^T: the pair's two volumes (species after S^T, or pulses)
// times the fluence (diagonal switching) or one
__global__ __launch_bounds__(kFftThreads) void spec_x_vox(const float2* __restrict__ in,
                                                          float* __restrict__ c,
                                                          const float* __restrict__ phi,
                                                          int phi_mode, int nvol, Geo G, FftDim D,
                                                          Marks M, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.lz);
  const int z = at.l0 + (threadIdx.x & 15);
  const int v0 = 2 * at.p, v1 = v0 + 1;
  const RowMarks W = row_marks(raw, D.n);
  // (planes of their own: volumes are pulses)
  const size_t grid = (size_t)G.ny * G.nx, mrow = (size_t)at.iy * G.nx;
  const size_t p0 = M.planes == 1 ? 0 : v0 * grid, p1 = M.planes > v1 ? v1 * grid : p0;
  load_near(W, D.n, M, mrow, p0, p1, G.nx);
  if (at.l0 == 0 && (M.planes > 1 || at.p == 0)) clear_row(M, mrow, p0, p1, G.nx);
  const float2* i = in + ((size_t)at.p * G.nyp + at.iy) * G.nxp * G.lz + at.l0;
  fft::first_stage<1>(D, L, fft::strided<true>(i, 8u * G.lz, G.nxp));
  fft::middle_stages<1>(D, L);
  const size_t vol = (size_t)G.ny * G.nx * G.nz;
  const size_t row = (size_t)at.iy * G.nx * G.nz + at.l0;
  const unsigned pitch = 4u * (unsigned)G.nz, lane = (threadIdx.x & 15) * 4;
  fft::last_stage<1>(D, L, [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    if (z >= G.nz) return;
    const unsigned o = (unsigned)x0 * pitch + lane;
    const float pz = phi_mode == 1 ? phi[z] : 1.0f;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool in = x0 < G.nx - q * step;
      const float ph = phi_mode == 2 && in ? fft::at(phi + row, o + (unsigned)(q * step) * pitch) : pz;
      v[q] = {ph * v[q].x, ph * v[q].y};
    }
    reach_points<R>(W, D.n, p1 != p0, x0, step, v);
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (x0 < G.nx - q * step) {
        const unsigned oq = o + (unsigned)(q * step) * pitch;
        fft::at(c + (size_t)v0 * vol + row, oq) = v[q].x;
        if (v1 < nvol) fft::at(c + (size_t)v1 * vol + row, oq) = v[q].y;
      }
  });
}

// c[s][v] = sum_k S_v[k][s] b[k][v], per-voxel fluence
__global__ __launch_bounds__(256) void spec_st(const float* __restrict__ b, float* __restrict__ c,
                                               const float* __restrict__ phi, SwitchParams sw,
                                               size_t vol, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  const size_t v = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= vol) return;
  const float ph = phi[v];
  const float pg = sw.gamma == 0.0f ? 1.0f : powf(ph, sw.gamma);
  float acc[kMaxSpecies];
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s) acc[s] = 0.0f;
  for (int k = 0; k < sw.nk; ++k) {
    const float bv = b[(size_t)k * vol + v];
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s)
      if (s < sw.ns)
        acc[s] = __builtin_fmaf(
            ph * __builtin_fmaf(sw.b[s], expf(-(float)k * pg * sw.inv_tau[s]), sw.a[s]), bv, acc[s]);
  }
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s)
    if (s < sw.ns) c[(size_t)s * vol + v] = acc[s];
}

// ------------------------------------------------------------- y transform
// Block: 16 columns of kappa_x of pair p; points of rows 0 .. n_in - 1 (the
// others are zero), outputs of rows 0 .. n_out - 1.  in and out may be one
// buffer: every point is read before the first barrier.
template <int SIGN>
__global__ __launch_bounds__(kFftThreads) void spec_y(const float2* in, float2* out, int nxp,
                                                      int l, int rows_in, int rows_out, int n_in,
                                                      int n_out, FftDim D,
                                                      const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  int b = (int)blockIdx.x;
  const int tiles = l >> 4;
  const int l0 = (b % tiles) * 16;
  b /= tiles;
  const int kx = b % nxp, p = b / nxp;
  const size_t step = (size_t)nxp * l;
  const unsigned pitch = 8u * (unsigned)step;
  const size_t col = (size_t)kx * l + l0;
  const float2* i = in + (size_t)p * rows_in * step + col;
  // (the grid's side is the shorter one)
  fft::first_stage<SIGN>(D, L, fft::strided<(SIGN > 0)>(i, pitch, n_in));
  fft::middle_stages<SIGN>(D, L);
  float2* o = out + (size_t)p * rows_out * step + col;
  fft::last_stage<SIGN>(D, L, fft::strided_out<(SIGN < 0)>(o, pitch, n_out));
}

// ------------------------------------------------- products per frequency
// Frequency f of the half plane: kx in 1 .. (NX - 1) / 2 with every ky, then
// kx = 0 (and NX / 2) with ky <= NY / 2.
struct Freq {
  size_t at, neg;  // element offsets (ky NX + kx) of kappa and -kappa
  bool self;       // kappa == -kappa
};
__device__ __forceinline__ Freq freq_at(int f, int nyp, int nxp) {
  const int ni = (nxp - 1) / 2;
  int kx, ky;
  if (f < ni * nyp) {
    ky = f / ni;
    kx = 1 + f - ky * ni;
  } else {
    const int h = nyp / 2 + 1, g = f - ni * nyp;
    kx = g >= h ? nxp / 2 : 0;
    ky = g >= h ? g - h : g;
  }
  const int my = ky ? nyp - ky : 0, mx = kx ? nxp - kx : 0;
  return Freq{(size_t)ky * nxp + kx, (size_t)my * nxp + mx, ky == my && kx == mx};
}

// Values of one column at four consecutive contracted indices, separated from
// the pair's image: pulse 2p is (Z(kappa) + conj Z(-kappa)) / 2 and pulse 2p +
// 1 is (Z(kappa) - conj Z(-kappa)) / 2i; the halves are in the table's scale.
// self: the lane's own part (real for even columns, imaginary for odd ones);
// the part that meets the imaginary table is the neighbouring lane's.
__device__ __forceinline__ void unpair(const float4* zp, const float4* zm, int h, int c,
                                       float (&self)[4]) {
  const float4 a0 = zp[0], a1 = zp[1], b0 = zm[0], b1 = zm[1];
  const float zr[4] = {a0.x, a0.z, a1.x, a1.z}, zi[4] = {a0.y, a0.w, a1.y, a1.w};
  const float wr[4] = {b0.x, b0.z, b1.x, b1.z}, wi[4] = {b0.y, b0.w, b1.y, b1.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float re = h ? zi[i] + wi[i] : zr[i] + wr[i];
    const float im = h ? wr[i] - zr[i] : zi[i] - wi[i];
    self[i] = c ? im : re;
  }
}

__device__ __forceinline__ float quad_mirror(float v) {  // lane 4i + j <- 4i + 3 - j
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x1B, 0xf, 0xf, true));
}
__device__ __forceinline__ float quad_swap(float v) {    // lane j <- j ^ 1
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));
}

// Packs the products of a quad of lanes (pulse 2p: re, im, pulse 2p + 1: re,
// im; four consecutive rows each) into the pair's image and stores it at
// kappa (lanes 0, 1) and -kappa (lanes 2, 3): Z(kappa) = Y0 + i Y1, Z(-kappa)
// = conj Y0 + i conj Y1.  Each lane stores two rows, 16 bytes.
__device__ __forceinline__ void pair_store(f32x4 v, float2* zp, float2* zm, int c, int h, bool ok,
                                           bool self) {
  // lane 0: re - other.im (re of kappa); 1: im + other.re (im of kappa);
  // lane 2: re1 - im0 (im of -kappa); 3: im1 + re0 (re of -kappa)
  float own[4], oth[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float m = quad_mirror(v[i]);
    own[i] = c ? v[i] + m : v[i] - m;
    oth[i] = quad_swap(own[i]);
  }
  // kappa: lane 0 has re, lane 1 im; -kappa: lane 3 has re, lane 2 im
  const bool re = (c ^ h) == 0;
  float4 o;
  if (re) o = {own[0], oth[0], own[1], oth[1]};
  else o = {oth[2], own[2], oth[3], own[3]};
  float2* z = h ? zm : zp;
  if (ok && !(h && self)) *(float4*)(z + (re ? 0 : 2)) = o;
}

struct GemmArgs {
  const float* tab;       // [nf][nblk][real, imaginary][64][4]
  const unsigned* mask;   // [t tiles] the tile's 16-depth blocks
  int nblk, ntt;          // blocks of a frequency, t tiles
  int nyp, nxp, lz, lt, np, nk;
  const float2* in;
  float2* out;
  // H before a residual: r's marks (at, bad), cleared
  unsigned* clear;
  size_t n_clear;
  // H^T with S^T: the species' coefficients [K][S][Nz]
  const float* stab_t;
  int ns, nz;
  const int* gate;
};

// Y = T B.  A wave holds eight pulses (16 real columns); its operand for all
// depths sits in registers, the table's 16 x 16 blocks stream past it (the
// block's waves share them through the caches).
template <int ZC>
__global__ __launch_bounds__(512) void spec_gemm_fwd(GemmArgs A) {
  if (A.gate && *A.gate) return;  // a device stop test has ended the solve
  const int f = (int)blockIdx.x;
  // (frequencies x threads, NX NY / 2 x at least 8 a pulse, outnumber the positions of all planes)
  if (A.clear) {
    const size_t i = (size_t)f * blockDim.x + threadIdx.x;
    if (i < A.n_clear) A.clear[i] = 0u;
  }
  const Freq F = freq_at(f, A.nyp, A.nxp);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 4, n = lane & 15, c = n & 1, h = (n >> 1) & 1;
  const int p = wave * 4 + (n >> 2);
  const bool ok = p < A.np;
  const size_t img = (size_t)A.nyp * A.nxp;
  const float2* zp = A.in + ((size_t)(ok ? p : 0) * img + F.at) * A.lz;
  const float2* zm = A.in + ((size_t)(ok ? p : 0) * img + F.neg) * A.lz;
  float bs[ZC][4];
  const float sg = c ? 1.0f : -1.0f;
#pragma unroll
  for (int zc = 0; zc < ZC; ++zc) {
    if (zc * 16 < A.lz) {
      const int z = zc * 16 + 4 * g;
      unpair((const float4*)(zp + z), (const float4*)(zm + z), h, c, bs[zc]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) bs[zc][i] = 0.0f;
    }
  }
  float2* op = A.out + ((size_t)(ok ? p : 0) * img + F.at) * A.lt + 4 * g;
  float2* om = A.out + ((size_t)(ok ? p : 0) * img + F.neg) * A.lt + 4 * g;
  const float4* tab = (const float4*)A.tab + (size_t)f * A.nblk * 128 + lane;
  float4 ar = tab[0], ai = tab[64];  // (the table ends with a spare block)
  for (int tt = 0; tt < A.ntt; ++tt) {
    const unsigned m = A.mask[tt];
    f32x4 a0 = {0.0f, 0.0f, 0.0f, 0.0f}, a1 = a0;
#pragma unroll
    for (int zc = 0; zc < ZC; ++zc)
      if (m >> zc & 1u) {
        const float r[4] = {ar.x, ar.y, ar.z, ar.w}, q[4] = {ai.x, ai.y, ai.z, ai.w};
        tab += 128;
        ar = tab[0];
        ai = tab[64];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(r[i], bs[zc][i], a0, 0, 0, 0);
          a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(q[i], sg * quad_swap(bs[zc][i]), a1, 0, 0, 0);
        }
      }
    a0 += a1;
    pair_store(a0, op + tt * 16, om + tt * 16, c, h, ok, F.self);
  }
}

// G = conj(T)^T R, the accumulators of all depths in registers; ST: S^T over
// the pulses in LDS, pairs of species written instead of pairs of pulses.
template <int ZC, bool ST>
__global__ __launch_bounds__(512) void spec_gemm_adj(GemmArgs A) {
  if (A.gate && *A.gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const int f = (int)blockIdx.x;
  const Freq F = freq_at(f, A.nyp, A.nxp);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 4, n = lane & 15, c = n & 1, h = (n >> 1) & 1;
  const int p = wave * 4 + (n >> 2);
  const bool ok = p < A.np;
  const size_t img = (size_t)A.nyp * A.nxp;
  const float2* zp = A.in + ((size_t)(ok ? p : 0) * img + F.at) * A.lt + 4 * g;
  const float2* zm = A.in + ((size_t)(ok ? p : 0) * img + F.neg) * A.lt + 4 * g;
  const float sg = c ? -1.0f : 1.0f;
  f32x4 acc[ZC];
#pragma unroll
  for (int zc = 0; zc < ZC; ++zc) acc[zc] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const float4* tab = (const float4*)A.tab + (size_t)f * A.nblk * 128 + lane;
  float4 ar = tab[0], ai = tab[64];
  for (int tt = 0; tt < A.ntt; ++tt) {
    const unsigned m = A.mask[tt];
    if (m == 0) continue;
    float rs[4], ro[4];
    unpair((const float4*)(zp + tt * 16), (const float4*)(zm + tt * 16), h, c, rs);
    // conj(T): real columns meet +imaginary parts, imaginary ones -real parts
#pragma unroll
    for (int i = 0; i < 4; ++i) ro[i] = sg * quad_swap(rs[i]);
#pragma unroll
    for (int zc = 0; zc < ZC; ++zc)
      if (m >> zc & 1u) {
        const float r[4] = {ar.x, ar.y, ar.z, ar.w}, q[4] = {ai.x, ai.y, ai.z, ai.w};
        tab += 128;
        ar = tab[0];
        ai = tab[64];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[zc] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[i], rs[i], acc[zc], 0, 0, 0);
          acc[zc] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[i], ro[i], acc[zc], 0, 0, 0);
        }
      }
  }
  if constexpr (!ST) {
    float2* op = A.out + ((size_t)(ok ? p : 0) * img + F.at) * A.lz + 4 * g;
    float2* om = A.out + ((size_t)(ok ? p : 0) * img + F.neg) * A.lz + 4 * g;
#pragma unroll
    for (int zc = 0; zc < ZC; ++zc)
      if (zc * 16 < A.lz) pair_store(acc[zc], op + zc * 16, om + zc * 16, c, h, ok, F.self);
  } else {
    float* gb = (float*)raw;  // [2 pairs][lz][2]
    const int q = 2 * p + h;
    if (ok) {
#pragma unroll
      for (int zc = 0; zc < ZC; ++zc)
        if (zc * 16 < A.lz) {
#pragma unroll
          for (int j = 0; j < 4; ++j) gb[((size_t)q * A.lz + zc * 16 + 4 * g + j) * 2 + c] = acc[zc][j];
        }
    }
    __syncthreads();
    const float2* gv = (const float2*)raw;
    const int nps = (A.ns + 1) / 2;
    for (int i = (int)threadIdx.x; i < nps * A.lz; i += (int)blockDim.x) {
      const int ps = i / A.lz, z = i - ps * A.lz;
      float2 s0 = {0.0f, 0.0f}, s1 = {0.0f, 0.0f};
      if (z < A.nz) {
        const bool two = 2 * ps + 1 < A.ns;
        const float* w = A.stab_t + (size_t)(2 * ps) * A.nz + z;
        for (int k = 0; k < A.nk; ++k, w += (size_t)A.ns * A.nz) {
          const float2 v = gv[(size_t)k * A.lz + z];
          const float w0 = w[0], w1 = two ? w[A.nz] : 0.0f;
          s0 = fft::cfma(w0, v, s0);
          s1 = fft::cfma(w1, v, s1);
        }
      }
      float2* o = A.out + (size_t)ps * img * A.lz + z;
      o[F.at * A.lz] = float2{s0.x - s1.y, s0.y + s1.x};
      if (!F.self) o[F.neg * A.lz] = float2{s0.x + s1.y, s1.x - s0.y};
    }
  }
}

// ------------------------------------------------------- the table (FP64)
// Partial sums over dx of one 16 x 16 block of (t, z): P[kx][dy][256]
__global__ __launch_bounds__(256) void spec_table_x(const int* __restrict__ t0,
                                                    const float* __restrict__ taps, int f, int w,
                                                    int nz, int nt, int tb, int zb, int nxp,
                                                    double2* __restrict__ P) {
  const int kx = blockIdx.x, jy = blockIdx.y;
  const int tl = threadIdx.x & 15, zl = threadIdx.x >> 4;
  const int t = tb * 16 + tl, z = zb * 16 + zl, r = (f - 1) / 2;
  double2 a = {0.0, 0.0};
  if (t < nt && z < nz) {
    const size_t col = ((size_t)z * f + jy) * f;
    for (int jx = 0; jx < f; ++jx) {
      const int j = t - t0[col + jx];
      if (j < 0 || j >= w) continue;
      const double h = (double)taps[(col + jx) * w + j];
      // the phase's integer part dropped before it is scaled
      const int ph = (int)((((long long)kx * (jx - r)) % nxp + nxp) % nxp);
      double sn, cs;
      sincospi(2.0 * (double)ph / (double)nxp, &sn, &cs);
      a.x += h * cs;
      a.y += h * sn;
    }
  }
  P[((size_t)kx * f + jy) * 256 + threadIdx.x] = a;
}

// T at the frequencies f0 + 0 .. of the block: sums over dy, scaled, in the
// lane order of both directions
constexpr int kTabY = 8;  // ky of a workgroup
__global__ __launch_bounds__(256) void spec_table_y(const double2* __restrict__ P, int f, int nyp,
                                                    int nxp, int blk, int nblk, double scale,
                                                    float* __restrict__ tf,
                                                    float* __restrict__ ta) {
  const int kx = blockIdx.x, r = (f - 1) / 2;
  const int ni = (nxp - 1) / 2;
  const bool edge = kx == 0 || (nxp % 2 == 0 && kx == nxp / 2);
  const int nky = edge ? nyp / 2 + 1 : nyp;
  const int ky0 = blockIdx.y * kTabY;
  if (ky0 >= nky) return;
  double2 a[kTabY];
#pragma unroll
  for (int i = 0; i < kTabY; ++i) a[i] = double2{0.0, 0.0};
  __shared__ double2 ph[kTabY];
  for (int jy = 0; jy < f; ++jy) {
    __syncthreads();
    if (threadIdx.x < kTabY) {
      const int ky = ky0 + threadIdx.x;
      const int q = (int)((((long long)ky * (jy - r)) % nyp + nyp) % nyp);
      double sn, cs;
      sincospi(2.0 * (double)q / (double)nyp, &sn, &cs);
      ph[threadIdx.x] = double2{cs, sn};
    }
    __syncthreads();
    const double2 v = P[((size_t)kx * f + jy) * 256 + threadIdx.x];
#pragma unroll
    for (int i = 0; i < kTabY; ++i) {
      a[i].x += v.x * ph[i].x - v.y * ph[i].y;
      a[i].y += v.x * ph[i].y + v.y * ph[i].x;
    }
  }
  const int tl = threadIdx.x & 15, zl = threadIdx.x >> 4;
  for (int i = 0; i < kTabY; ++i) {
    const int ky = ky0 + i;
    if (ky >= nky) break;
    const size_t fr = edge ? (size_t)ni * nyp + (kx ? nyp / 2 + 1 : 0) + ky
                           : (size_t)ky * ni + (kx - 1);
    const size_t b = (fr * nblk + blk) * 512;
    const float re = (float)(a[i].x * scale), im = (float)(a[i].y * scale);
    // forward: row t, contracted z = 4 g + slot; adjoint: row z, contracted t
    const size_t wf = b + ((size_t)(zl >> 2) * 16 + tl) * 4 + (zl & 3);
    const size_t wa = b + ((size_t)(tl >> 2) * 16 + zl) * 4 + (tl & 3);
    if (tf) {
      tf[wf] = re;
      tf[wf + 256] = im;
    }
    if (ta) {
      ta[wa] = re;
      ta[wa + 256] = im;
    }
  }
}

// ------------------------------------------------------ reach of the marks
// Block: one row of one plane.  The marks of the 2 R + 1 rows around it are
// joined per column, then the columns over 2 R + 1 neighbours.
__global__ __launch_bounds__(256) void spec_reach(Marks M, int ny, int nx, int r,
                                                  const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const int iy = (int)blockIdx.x % ny;
  const size_t plane = (size_t)((int)blockIdx.x / ny) * ny * nx;
  const int y0 = max(0, iy - r), y1 = min(ny - 1, iy + r);
  for (int x = (int)threadIdx.x; x < nx; x += 256) {
    unsigned f = 0;
    for (int y = y0; y <= y1; ++y) {
      const size_t i = plane + (size_t)y * nx + x;
      f |= (M.at[i] == M.now ? kNearSome : 0) | (M.bad[i] == M.now ? kNearBad : 0);
    }
    raw[x] = (unsigned char)f;
  }
  __syncthreads();
  for (int x = (int)threadIdx.x; x < nx; x += 256) {
    unsigned f = 0;
    for (int i = max(0, x - r); i <= min(nx - 1, x + r); ++i) f |= raw[i];
    M.near[plane + (size_t)iy * nx + x] = (unsigned char)f;
  }
}

// ------------------------------------------------------------------- host
// radices of n in at most kFftMaxStages stages, as few and as even as found
bool factor(int n, FftDim& D) {
  static const int rs[] = {10, 9, 8, 6, 5, 4, 3, 2};
  int best_ns = kFftMaxStages + 1, best_max = 99;
  int cur[kFftMaxStages];
  auto rec = [&](auto&& self, int left, int depth, int cap) -> void {
    if (left == 1) {
      if (depth < 2) return;
      const int mx = cur[0];
      if (depth < best_ns || (depth == best_ns && mx < best_max)) {
        best_ns = depth;
        best_max = mx;
        D.ns = depth;
        for (int i = 0; i < depth; ++i) D.rad[i] = cur[i];
      }
      return;
    }
    if (depth == kFftMaxStages) return;
    for (int r : rs) {
      if (r > cap || left % r) continue;
      cur[depth] = r;
      self(self, left / r, depth + 1, r);
    }
  };
  rec(rec, n, 0, 99);
  if (best_ns > kFftMaxStages) return false;
  D.n = n;
  return true;
}

size_t fft_lds(int n) { return (size_t)n * (kFftLanes + 1) * sizeof(float2); }

// the cheapest transform length of at least `need` points: a stage costs a
// pass over LDS, a point a pass over HBM
bool choose_length(int need, FftDim& D) {
  double best = 0.0;
  bool found = false;
  for (int n = std::max(need, 4); n <= need + need / 2 + 16; ++n) {
    if (row_lds(n) > (size_t)kLdsMaxBytes - 1024) break;
    FftDim t;
    if (!factor(n, t)) continue;
    const double cost = n * (1.0 + 0.15 * t.ns);
    if (!found || cost < best) {
      best = cost;
      D = t;
      found = true;
    }
  }
  return found;
}

Geo geo_of(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  Geo G;
  G.ny = P->g.ny;
  G.nx = P->g.nx;
  G.nyp = Q.ny;
  G.nxp = Q.nx;
  G.nz = P->g.nz;
  G.nt = P->g.nt;
  G.lz = Q.lz;
  G.lt = Q.lt;
  G.tlo = Q.tlo;
  G.nk = P->g.n_pulses;
  G.np = Q.np;
  G.r = P->R;
  G.f = P->F;
  return G;
}

// marks of H's operand (b) and of H^T's (r): pulse volumes of their own have a
// plane each, species that every pulse mixes share one
int mark_planes(const psoam_plan* P) { return P->sw.diag ? P->g.n_pulses : 1; }
Marks marks_b(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  return Marks{Q.d_at_b, Q.d_bad_b, Q.d_near_b, Q.call_b, mark_planes(P)};
}
Marks marks_r(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  return Marks{Q.d_at_r, Q.d_bad_r, Q.d_near_r, Q.call_r, mark_planes(P)};
}

FftDim dim_of(const SpecPlan& Q, int axis) {
  FftDim D;
  D.n = axis ? Q.nx : Q.ny;
  D.ns = axis ? Q.nsx : Q.nsy;
  for (int i = 0; i < kFftMaxStages; ++i) D.rad[i] = axis ? Q.radx[i] : Q.rady[i];
  D.tw = (const float2*)(axis ? Q.d_twx : Q.d_twy);
  D.derive();
  return D;
}

int rnd_of(const psoam_plan* P) {
  switch (P->prec) {
    case PSOAM_BF16:
    case PSOAM_BF16_REFINED: return kRndBf16;
    case PSOAM_FP16: return kRndF16;
    default: return kRndNone;
  }
}

template <class K, class... Args>
hipError_t go(K kern, size_t blocks, int threads, size_t lds, hipStream_t s, Args... args) {
  if (blocks == 0) return hipSuccess;
  if (lds > 64 * 1024)
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), lds, s, args...);
  return hipGetLastError();
}

GemmArgs gemm_args(const psoam_plan* P, bool adj) {
  const SpecPlan& Q = *P->spec;
  GemmArgs A;
  A.tab = adj ? Q.d_ta : Q.d_tf;
  A.mask = Q.d_mask;
  A.nblk = Q.nblk;
  A.ntt = Q.lt / 16;
  A.nyp = Q.ny;
  A.nxp = Q.nx;
  A.lz = Q.lz;
  A.lt = Q.lt;
  A.np = Q.np;
  A.nk = P->g.n_pulses;
  A.in = (const float2*)(adj ? Q.d_y : Q.d_x);
  A.out = (float2*)(adj ? Q.d_g : Q.d_y);
  A.stab_t = P->d_stab_t;
  A.ns = P->sw.ns;
  A.nz = P->g.nz;
  A.gate = gate_now();
  A.clear = nullptr;
  A.n_clear = 0;
  return A;
}

// S^T inside the product: per-depth fluence, species mixed
bool st_in_gemm(const psoam_plan* P) { return P->d_stab_t && !P->sw.diag; }

// c-side planes (pairs) of H^T
int adj_pairs(const psoam_plan* P) {
  return st_in_gemm(P) ? (P->sw.ns + 1) / 2 : (P->g.n_pulses + 1) / 2;
}

#define SPEC_HIP(call)                 \
  do {                                 \
    hipError_t _e = (call);            \
    if (_e != hipSuccess) return _e;   \
  } while (0)

}  // namespace

size_t spec_partials(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  return (size_t)Q.np * P->g.ny * (Q.lt / 16) + kIdleSums;
}

hipError_t spec_switch(const psoam_plan* P, const float* c, hipStream_t s) {
  SpecPlan& Q = *P->spec;
  const Geo G = geo_of(P);
  const FftDim X = dim_of(Q, 1), Y = dim_of(Q, 0);
  ++Q.call_b;
  const Marks M = marks_b(P);
  const size_t nb = (size_t)Q.np * G.ny * (G.lz / 16);
  auto x = [&](auto kern) {
    return go(kern, nb, kFftThreads, row_lds(G.nxp), s, c, P->d_phi, P->d_stab_t, P->d_f16, P->sw,
              (float2*)Q.d_x, G, X, M, gate_now());
  };
  const int src = P->sw.diag ? kSrcDiag : P->d_stab_t ? kSrcDepth : kSrcVoxel;
#define SPEC_SW(R)                                                            \
  SPEC_HIP(src == kSrcDiag    ? x(spec_x_switch<R, kSrcDiag>)                 \
           : src == kSrcDepth ? x(spec_x_switch<R, kSrcDepth>)                \
                              : x(spec_x_switch<R, kSrcVoxel>))
  switch (rnd_of(P)) {
    case kRndBf16: SPEC_SW(kRndBf16); break;
    case kRndF16: SPEC_SW(kRndF16); break;
    default: SPEC_SW(kRndNone); break;
  }
#undef SPEC_SW
  SPEC_HIP(go(spec_reach, (size_t)M.planes * G.ny, 256, (size_t)G.nx, s, M, G.ny, G.nx, G.r, gate_now()));
  return go(spec_y<-1>, (size_t)Q.np * G.nxp * (G.lz / 16), kFftThreads, fft_lds(G.nyp), s,
            (const float2*)Q.d_x, (float2*)Q.d_x, G.nxp, G.lz, G.nyp, G.nyp, G.ny, G.nyp, Y, gate_now());
}

// The reach of r's marks, beside the pass that made r: what follows only reads
// it, so that H^T may run again on the same r.
static hipError_t reach_r(const psoam_plan* P, hipStream_t s) {
  const Geo G = geo_of(P);
  const Marks M = marks_r(P);
  return go(spec_reach, (size_t)M.planes * G.ny, 256, (size_t)G.nx, s, M, G.ny, G.nx, G.r, gate_now());
}

hipError_t spec_pack(const psoam_plan* P, const float* y, hipStream_t s) {
  SpecPlan& Q = *P->spec;
  const Geo G = geo_of(P);
  const FftDim X = dim_of(Q, 1);
  ++Q.call_r;
  const Marks M = marks_r(P);
  const size_t nb = (size_t)Q.np * G.ny * (G.lt / 16);
  auto x = [&](auto kern) {
    return go(kern, nb, kFftThreads, row_lds(G.nxp), s, y, P->d_f16, (float2*)Q.d_r, G, X, M,
              gate_now());
  };
  switch (rnd_of(P)) {
    case kRndBf16: SPEC_HIP(x(spec_x_pack<kRndBf16>)); break;
    case kRndF16: SPEC_HIP(x(spec_x_pack<kRndF16>)); break;
    default: SPEC_HIP(x(spec_x_pack<kRndNone>)); break;
  }
  return reach_r(P, s);
}

hipError_t spec_band(const psoam_plan* P, int mode, float* out, const float* pmeas,
                     double* partial, hipStream_t s, float* yc, double yc_beta, int yc_first,
                     bool sums) {
  SpecPlan& Q = *P->spec;
  const Geo G = geo_of(P);
  const FftDim X = dim_of(Q, 1), Y = dim_of(Q, 0);
  const int waves = (Q.np + 3) / 4;
  const Marks MB = marks_b(P);
  if (mode != 2) {
    GemmArgs A = gemm_args(P, false);
    if (mode != 0) {
      A.clear = Q.d_at_r;  // d_bad_r follows it
      A.n_clear = 2 * (size_t)MB.planes * G.ny * G.nx;
    }
    const int zc = Q.lz / 16;
    if (zc <= 4) SPEC_HIP(go(spec_gemm_fwd<4>, (size_t)Q.nf, waves * 64, 0, s, A));
    else if (zc <= 8) SPEC_HIP(go(spec_gemm_fwd<8>, (size_t)Q.nf, waves * 64, 0, s, A));
    else SPEC_HIP(go(spec_gemm_fwd<16>, (size_t)Q.nf, waves * 64, 0, s, A));
    SPEC_HIP(go(spec_y<1>, (size_t)Q.np * G.nxp * (G.lt / 16), kFftThreads, fft_lds(G.nyp), s,
                (const float2*)Q.d_y, (float2*)Q.d_y, G.nxp, G.lt, G.nyp, G.nyp, G.nyp, G.ny, Y,
                gate_now()));
    const size_t nb = (size_t)Q.np * G.ny * (G.lt / 16);
    // samples [tlo, thi) are transformed
    const int thi = std::min(G.nt, G.tlo + G.lt);
    const size_t rows = (size_t)G.nk * G.ny * G.nx;
    if (mode == 0 && thi - G.tlo < G.nt) {
      if (G.nt % 4 == 0 && thi % 4 == 0)  // (y is 16-byte aligned)
        SPEC_HIP(go(spec_idle_zero4, std::min<size_t>((rows + 3) / 4, 16384), 256, 0, s, (f32x4*)out,
                    rows, G.nt / 4, G.tlo / 4, thi / 4, gate_now()));
      else
        SPEC_HIP(go(spec_idle_zero, std::min<size_t>((rows * 64 + 255) / 256, 16384), 256, 0, s, out,
                    rows, G.nt, G.tlo, thi, gate_now()));
    }
    if (mode != 0 && sums)
      SPEC_HIP(go(spec_idle_sums, (size_t)kIdleSums, 256, 0, s, pmeas, rows, G.nt, G.tlo, thi,
                  partial + nb, gate_now()));
    if (mode == 0)
      return go(spec_x_out, nb, kFftThreads, row_lds(G.nxp), s, (const float2*)Q.d_y, out, G, X, MB,
                gate_now());
    ++Q.call_r;
    const Marks MR = marks_r(P);
    const float beta = (float)yc_beta, inv = (float)(1.0 / (1.0 + yc_beta));
    auto r = [&](auto kern) {
      return go(kern, nb, kFftThreads, row_lds(G.nxp), s, (const float2*)Q.d_y, pmeas, P->d_f16,
                (float2*)Q.d_r, yc, beta, inv, yc_first, partial, G, X, MB, MR, gate_now());
    };
    const bool rec = yc != nullptr;
    switch (rnd_of(P)) {
      case kRndBf16: SPEC_HIP(rec ? r(spec_x_resid<kRndBf16, true>) : r(spec_x_resid<kRndBf16, false>)); break;
      case kRndF16: SPEC_HIP(rec ? r(spec_x_resid<kRndF16, true>) : r(spec_x_resid<kRndF16, false>)); break;
      default: SPEC_HIP(rec ? r(spec_x_resid<kRndNone, true>) : r(spec_x_resid<kRndNone, false>)); break;
    }
    return reach_r(P, s);
  }
  const Marks MR = marks_r(P);
  SPEC_HIP(go(spec_y<-1>, (size_t)Q.np * G.nxp * (G.lt / 16), kFftThreads, fft_lds(G.nyp), s,
              (const float2*)Q.d_r, (float2*)Q.d_y, G.nxp, G.lt, G.ny, G.nyp, G.ny, G.nyp, Y,
              gate_now()));
  const GemmArgs A = gemm_args(P, true);
  const int zc = Q.lz / 16;
  const bool st = st_in_gemm(P);
  const size_t lds = st ? (size_t)2 * Q.np * Q.lz * sizeof(float2) : 0;
  if (st) {
    if (zc <= 4) SPEC_HIP(go(spec_gemm_adj<4, true>, (size_t)Q.nf, waves * 64, lds, s, A));
    else if (zc <= 8) SPEC_HIP(go(spec_gemm_adj<8, true>, (size_t)Q.nf, waves * 64, lds, s, A));
    else SPEC_HIP(go(spec_gemm_adj<16, true>, (size_t)Q.nf, waves * 64, lds, s, A));
  } else {
    if (zc <= 4) SPEC_HIP(go(spec_gemm_adj<4, false>, (size_t)Q.nf, waves * 64, lds, s, A));
    else if (zc <= 8) SPEC_HIP(go(spec_gemm_adj<8, false>, (size_t)Q.nf, waves * 64, lds, s, A));
    else SPEC_HIP(go(spec_gemm_adj<16, false>, (size_t)Q.nf, waves * 64, lds, s, A));
  }
  const int na = adj_pairs(P);
  SPEC_HIP(go(spec_y<1>, (size_t)na * G.nxp * (G.lz / 16), kFftThreads, fft_lds(G.nyp), s,
              (const float2*)Q.d_g, (float2*)Q.d_g, G.nxp, G.lz, G.nyp, G.nyp, G.nyp, G.ny, Y,
              gate_now()));
  const size_t nb = (size_t)na * G.ny * (G.lz / 16);
  const bool mix = !st && !P->sw.diag;  // per-voxel fluence: S^T after the pulses are back
  float* dst = mix ? (float*)Q.d_y : out;
  const int nvol = st ? P->sw.ns : G.nk;
  const int phi_mode = P->sw.diag ? (P->sw.per_voxel ? 2 : 1) : 0;
  SPEC_HIP(go(spec_x_vox, nb, kFftThreads, row_lds(G.nxp), s, (const float2*)Q.d_g, dst, P->d_phi,
              phi_mode, nvol, G, X, MR, gate_now()));
  if (mix) {
    const size_t vol = P->v_elems();
    SPEC_HIP(go(spec_st, (vol + 255) / 256, 256, 0, s, (const float*)Q.d_y, out, P->d_phi, P->sw, vol,
                gate_now()));
  }
  return hipSuccess;
}

void spec_free(psoam_plan* P) {
  if (!P->spec) return;
  SpecPlan& Q = *P->spec;
  for (void* b : {Q.d_x, Q.d_y, Q.d_r, Q.d_g, (void*)Q.d_tf, (void*)Q.d_ta, (void*)Q.d_mask, Q.d_twx,
                  Q.d_twy, (void*)Q.d_marks})
    if (b) (void)hipFree(b);
  delete P->spec;
  P->spec = nullptr;
}

bool spec_build(psoam_plan* P, const int32_t* t0, const float* taps_f, const float* taps_a,
                bool force, double direct_us, bool fact, hipStream_t stream) {
  const auto& g = P->g;
  FftDim X, Y;
  if (!choose_length(g.nx + P->R, X) || !choose_length(g.ny + P->R, Y)) return false;
  const int lz = (g.nz + 15) / 16 * 16;
  if (lz > 256) return false;  // the product holds every depth in registers
  const int F = P->F, W = P->W;
  // the 16 x 16 blocks of (t, z) with a nonzero entry at any offset
  std::vector<unsigned> mask((g.nt + 15) / 16, 0);
  for (int z = 0; z < g.nz; ++z)
    for (size_t o = 0; o < (size_t)F * F; ++o) {
      const size_t col = (size_t)z * F * F + o;
      for (int j = 0; j < W; ++j) {
        const int t = t0[col] + j;
        if (t >= 0 && t < g.nt && (taps_f[col * W + j] != 0.0f || taps_a[col * W + j] != 0.0f))
          mask[t >> 4] |= 1u << (z >> 4);
      }
    }
  // the range of tiles that any block meets
  while (mask.size() > 1 && mask.back() == 0) mask.pop_back();
  int tb0 = 0;
  while (tb0 + 1 < (int)mask.size() && mask[tb0] == 0) ++tb0;
  mask.erase(mask.begin(), mask.begin() + tb0);
  const int ntt = (int)mask.size(), lt = 16 * ntt;
  int nblk = 0;
  for (unsigned m : mask) nblk += __builtin_popcount(m);
  const int np = (g.n_pulses + 1) / 2;
  const int ni = (X.n - 1) / 2, edges = X.n % 2 ? 1 : 2;
  const size_t nf = (size_t)ni * Y.n + (size_t)edges * (Y.n / 2 + 1);
  const bool st = !g.phi_per_voxel && !P->sw.diag;
  const size_t img = (size_t)Y.n * X.n;
  const size_t xb = (size_t)np * img * lz * 8;
  // per-voxel fluence: y's spectrum also holds the pulse volumes S^T reads,
  // which are the larger where the depths outnumber the samples
  const size_t yb = std::max((size_t)np * img * lt * 8, (size_t)g.n_pulses * P->v_elems() * sizeof(float));
  const size_t rb = (size_t)np * g.ny * X.n * lt * 8;
  const size_t gb = (size_t)(st ? (P->sw.ns + 1) / 2 : np) * img * lz * 8;
  const size_t tb = (nf * nblk + 2) * 512 * sizeof(float);
  const size_t pb = (size_t)(X.n / 2 + 1) * F * 256 * sizeof(double2);
  const size_t grid = (size_t)g.ny * g.nx;
  // the transforms' offsets within a line are 32 bits, its positions 20
  X.derive();
  Y.derive();
  const size_t most = (size_t)std::max(lz, lt) * 8;
  if (std::max({X.n * std::max<size_t>(most, 4 * (size_t)std::max(g.nt, g.nz)),
                Y.reach(most * X.n)}) >= (1ull << 32) ||
      std::max(X.n, Y.n) >= (1 << 20))
    return false;
  // launch grids are 32-bit counts of blocks
  if (nf >= (1u << 31) || (size_t)np * X.n * (lt / 16) >= (1u << 31)) return false;
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return false;
  const size_t need = xb + yb + rb + gb + 2 * tb + pb;
  // the direct form needs about the operands alone; this one stays where a
  // user's own arrays still have most of the card
  if (need > free_b / 3) return false;
  if (!force) {
    // Predicted time of one A and one A^T: the launches, and the bytes of all
    // passes at 4.0 TB/s (a fit to 400 random geometries: half of the
    // predictions within 13%, 90% within 28%).  At 128 x 128 x 64 with 32
    // pulses and a footprint of 31 the pair takes 1.4 ms against the direct
    // form's 41 ms in FP32 and 3.2 ms in BF16; at 97 x 95 x 16 with a
    // footprint of 7 and 64 samples it takes 0.8 ms against 0.28 ms in BF16.
    const double a = 2.0 * np * g.ny * X.n * lz * 8 + 2.0 * xb + tb + 2.0 * yb + 2.0 * rb;
    const double at = 2.0 * rb + 2.0 * yb + tb + 4.0 * gb;
    const double y = 4.0 * g.n_pulses * grid;  // a sample of every A-scan
    const double us = 62.0 + 0.248e-6 * (a + at + y * (g.nt + lt) + (fact ? 2.0 : 0.0) * y * g.nt);
    // 16-bit operands are rounded from sums that differ in their last FP32
    // bits between the forms: the change has to be worth it
    const bool rounds = rnd_of(P) != kRndNone;
    if (us > (rounds ? 0.9 : 1.0) * direct_us) return false;
    // FP32 against FP64: from a footprint of 7 on the direct form's longer
    // sums err as much as the transforms or more (medians of the error over
    // the direct form's 0.96 and 0.65 for A and A^T at 7, 0.40 and 0.30 at
    // 17), below it less (1.67 and 1.46 at 3)
    if (P->prec == PSOAM_FP32 && P->F < kSpecMinFp32F) return false;
  }
  SpecPlan* Qp = new (std::nothrow) SpecPlan();
  if (!Qp) return false;
  P->spec = Qp;
  SpecPlan& Q = *Qp;
  Q.nx = X.n;
  Q.ny = Y.n;
  Q.nsx = X.ns;
  Q.nsy = Y.ns;
  for (int i = 0; i < kFftMaxStages; ++i) {
    Q.radx[i] = X.rad[i];
    Q.rady[i] = Y.rad[i];
  }
  Q.lz = lz;
  Q.lt = lt;
  Q.tlo = 16 * tb0;
  Q.np = np;
  Q.nf = nf;
  Q.nblk = nblk;
  double2* d_p = nullptr;
  int* d_t0 = nullptr;
  float* d_taps = nullptr;
  const bool twice = taps_a != taps_f;  // a table of its own for H^T
  const size_t ntab = (size_t)g.nz * F * F;
  bool ok = true;
  auto alloc = [&](auto** p, size_t bytes) {
    if (ok && hipMalloc((void**)p, std::max<size_t>(bytes, 16)) != hipSuccess) {
      (void)hipGetLastError();
      *p = nullptr;
      ok = false;
    }
  };
  auto check = [&](hipError_t e) {
    if (e != hipSuccess) ok = false;
  };
  alloc(&Q.d_x, xb);
  alloc(&Q.d_y, yb);
  alloc(&Q.d_r, rb);
  alloc(&Q.d_g, gb);
  alloc(&Q.d_tf, tb);
  alloc(&Q.d_ta, tb);
  alloc(&Q.d_mask, sizeof(unsigned) * ntt);
  alloc(&Q.d_twx, sizeof(float2) * X.n);
  alloc(&Q.d_twy, sizeof(float2) * Y.n);
  // marks of b and of r: two words and a byte per position and plane
  const size_t planes = mark_planes(P);
  const size_t mb = 2 * planes * grid * (2 * sizeof(unsigned) + 1);
  alloc(&Q.d_marks, mb);
  if (ok) {
    Q.d_at_b = (unsigned*)Q.d_marks;
    Q.d_bad_b = Q.d_at_b + planes * grid;
    Q.d_at_r = Q.d_bad_b + planes * grid;
    Q.d_bad_r = Q.d_at_r + planes * grid;
    Q.d_near_b = (unsigned char*)(Q.d_bad_r + planes * grid);
    Q.d_near_r = Q.d_near_b + planes * grid;
  }
  alloc(&d_p, pb);
  alloc(&d_t0, sizeof(int) * ntab);
  alloc(&d_taps, sizeof(float) * ntab * W);
  if (ok) {
    auto upload = [&](void* dst, int n) {
      std::vector<float2> tw(n);
      for (int j = 0; j < n; ++j) {
        const double a = 2.0 * M_PI * (double)j / (double)n;
        tw[j] = float2{(float)std::cos(a), (float)-std::sin(a)};
      }
      check(hipMemcpy(dst, tw.data(), sizeof(float2) * n, hipMemcpyHostToDevice));
    };
    upload(Q.d_twx, X.n);
    upload(Q.d_twy, Y.n);
    check(hipMemcpy(Q.d_mask, mask.data(), sizeof(unsigned) * ntt, hipMemcpyHostToDevice));
    check(hipMemcpy(d_t0, t0, sizeof(int) * ntab, hipMemcpyHostToDevice));
    // the marks start below every call's number; the table's spare blocks are
    // read and not used
    check(hipMemsetAsync(Q.d_marks, 0, mb, stream));
    check(hipMemsetAsync(Q.d_tf + (nf * nblk) * 512, 0, 1024 * sizeof(float), stream));
    check(hipMemsetAsync(Q.d_ta + (nf * nblk) * 512, 0, 1024 * sizeof(float), stream));
    // 1/2 from the pairs' separation, 1 / (NX NY) from the inverse transform
    const double scale = 0.5 / ((double)X.n * (double)Y.n);
    const int kxn = X.n / 2 + 1;
    for (int pass = 0; pass < (twice ? 2 : 1) && ok; ++pass) {
      check(hipMemcpyAsync(d_taps, pass ? taps_a : taps_f, sizeof(float) * ntab * W,
                           hipMemcpyHostToDevice, stream));
      float* tf = pass ? nullptr : Q.d_tf;
      float* ta = pass || !twice ? Q.d_ta : nullptr;
      int blk = 0;
      for (int tt = 0; tt < ntt && ok; ++tt)
        for (int zb = 0; zb < lz / 16 && ok; ++zb) {
          if (!(mask[tt] >> zb & 1u)) continue;
          hipLaunchKernelGGL(spec_table_x, dim3(kxn, F), dim3(256), 0, stream, d_t0, d_taps, F, W,
                             g.nz, g.nt, tb0 + tt, zb, X.n, d_p);
          hipLaunchKernelGGL(spec_table_y, dim3(kxn, (Y.n + kTabY - 1) / kTabY), dim3(256), 0, stream,
                             d_p, F, Y.n, X.n, blk, nblk, scale, tf, ta);
          check(hipGetLastError());
          ++blk;
        }
    }
    check(hipStreamSynchronize(stream));
  }
  for (void* b : {(void*)d_p, (void*)d_t0, (void*)d_taps})
    if (b) (void)hipFree(b);
  if (!ok) spec_free(P);
  return ok;
}

}  // namespace psoam
