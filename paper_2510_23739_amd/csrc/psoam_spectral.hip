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
// Two neighbouring depths (samples) of a pulse share one complex image (real
// and imaginary part): H is real, so the pair goes through the transforms
// unseparated; the product takes kappa and -kappa together and separates them
// in registers.  A transform rounds in proportion to the largest values of its
// image, so what shares one has to be of one scale: neighbouring depths and
// samples meet the same band entries, where pulses (paired once) may differ by
// any factor.
//
//   spec_x_switch   S c (or phi c), rounded, transform along x
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
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));  // two floats of a line

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

// Per-voxel switching: phi^gamma is 1 (gamma 0, phig null), phi (gamma 1, phig
// the fluence itself) or an array that the plan holds: powf beside the
// exponentials, though it ran for other gammas alone, took their kernel from 27
// to 69 us at 77 x 61 x 50 with 19 pulses.
__device__ __forceinline__ float switch_coef(const SwitchParams& sw, float phi, float pg, int k, int s) {
  return phi * __builtin_fmaf(sw.b[s], expf(-(float)k * pg * sw.inv_tau[s]), sw.a[s]);
}
__global__ __launch_bounds__(256) void spec_rate(const float* __restrict__ phi, float* __restrict__ out,
                                                 float gamma, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) out[i] = powf(phi[i], gamma);
}

// Where the operand is not zero, and where it is not finite.  A transform
// spreads its rounding over the whole image, and a value that is not finite
// over all of it; the direct form reaches the footprint, and of it the tiles of
// depths or samples that band entries meet.  So every pass that makes an operand
// marks its positions, spec_reach widens the marks by the footprint, and the
// pass that writes the result writes zero where no nonzero value reaches and NaN
// where a non-finite one does (such a value enters the transforms as zero).  A
// mark is a bit per 16 depths: those of an operand of H, those that the sample
// tile meets (the product's mask) of one of H^T, looked at the other way round
// by the results.  spec_reach leaves the marks cleared: the next operand finds
// them so, whatever ran before it, eagerly or replayed.
struct Marks {
  unsigned* at;    // [planes][Ny][Nx]: bits 0 .. 15 nonzero, 16 .. 31 not finite
  unsigned* near;  // the same, of all positions in reach
  int* seen;       // [planes][Ny]: how many rows have looked at this one
  int planes;      // 1, or one per pulse (pulse volumes of their own)
};
constexpr int kBadBit = 16;
// The marks of a workgroup's row collect in LDS (a byte per column x, after
// the line and its twiddles) and go out once, and the reach of a row's
// columns comes in once: a mark or a look at one never waits for HBM.  The
// workgroup's two tiles have a bit each, lanes 0 .. 7 the first, 8 .. 15 the
// second.
struct RowMarks {
  unsigned char* hit;   // [n]: bits 0, 1 a nonzero value of the tile
  unsigned char* near;  // [n]: bits 0, 1 one in the tile's reach, bits 2, 3 a non-finite one
  unsigned tile[2];     // the tiles' bits of a mark
};
// mask: the depths that each sample tile meets (null: the tiles are depths)
__device__ __forceinline__ RowMarks row_marks(unsigned char* raw, int n, const unsigned* __restrict__ mask,
                                              int c0, int h) {
  unsigned char* a = raw + (size_t)n * (kFftLanes + 1) * sizeof(float2);
  const int t = c0 >> 3;
  const bool two = c0 + 8 < h;
  return RowMarks{a, a + n, {mask ? mask[t] : 1u << t, two ? mask ? mask[t + 1] : 1u << (t + 1) : 0u}};
}
__host__ __device__ constexpr size_t row_lds(int n) {
  return (size_t)n * ((kFftLanes + 1) * sizeof(float2) + 2);
}
__device__ __forceinline__ void set_mark(const Marks& M, size_t i, unsigned bits) {
  if ((M.at[i] & bits) != bits) atomicOr(&M.at[i], bits);
}
// One butterfly's operand values v (R positions x0, x0 + step, ..): the eight
// lanes of a tile join their nonzero bits and lane q writes position q's byte
// (every position belongs to one butterfly); non-finite values, which are rare,
// are marked in HBM (row: the plane's row) and become zero.
template <int CTRL>
__device__ __forceinline__ unsigned or_dpp(unsigned h) {
  return h | (unsigned)__builtin_amdgcn_mov_dpp((int)h, CTRL, 0xf, 0xf, true);
}
template <int R>
__device__ __forceinline__ void mark_points(const RowMarks& W, const Marks& M, size_t row, int x0,
                                            int step, float2* v) {
  const int lane = threadIdx.x & 15;
  bool bad = false;
  unsigned h = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    // zero where both are, not finite where either is not (or the sum overflows)
    const float s = fabsf(v[q].x) + fabsf(v[q].y);
    bad |= !finite_(s);
    h |= s != 0.0f ? 1u << q : 0u;
  }
  h = or_dpp<0x141>(or_dpp<0x4E>(or_dpp<0xB1>(h)));  // lanes j ^ 1, j ^ 2, 7 - j of eight
  const unsigned other = (unsigned)__builtin_amdgcn_mov_dpp((int)h, 0x128, 0xf, 0xf, true);  // row_ror:8
  const unsigned a = lane < 8 ? h : other, b = lane < 8 ? other : h;
  if (lane < R)
    W.hit[x0 + fft::mul24(lane, step)] = (unsigned char)((a >> lane & 1u) | (b >> lane & 1u) << 1);
  if (bad) {
    const unsigned bits = (lane < 8 ? W.tile[0] : W.tile[1]) << kBadBit;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if (!(finite_(v[q].x) && finite_(v[q].y))) set_mark(M, row + x0 + q * step, bits);
      if (!finite_(v[q].x)) v[q].x = 0.0f;
      if (!finite_(v[q].y)) v[q].y = 0.0f;
    }
  }
}
// The reach of the row's columns (past the grid: none): on its way while the
// first stage loads and computes, then into LDS.
constexpr int kNearWords = 5;  // of 256 columns: more than a line in LDS has
struct NearWords {
  unsigned w[kNearWords];
};
__device__ __forceinline__ NearWords load_near(const Marks& M, size_t row, int nx) {
  NearWords N;
#pragma unroll
  for (int i = 0; i < kNearWords; ++i) {
    const int x = (int)threadIdx.x + i * kFftThreads;
    N.w[i] = x < nx ? M.near[row + x] : 0u;
  }
  return N;
}
__device__ __forceinline__ void keep_near(const RowMarks& W, int n, const NearWords& N) {
#pragma unroll
  for (int i = 0; i < kNearWords; ++i) {
    const int x = (int)threadIdx.x + i * kFftThreads;
    const unsigned w = N.w[i], b = w >> kBadBit;
    if (x < n)
      W.near[x] = (unsigned char)((w & W.tile[0] ? 1 : 0) | (w & W.tile[1] ? 2 : 0) |
                                  (b & W.tile[0] ? 4 : 0) | (b & W.tile[1] ? 8 : 0));
  }
}
// a butterfly's results, zero or NaN where the reach says so
template <int R>
__device__ __forceinline__ void reach_points(const RowMarks& W, int x0, int step, float2* v) {
  const int tile = threadIdx.x >> 3 & 1;
  int r[R], any = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) r[q] = W.near[x0 + q * step];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    any |= r[q];
    const int keep = __builtin_amdgcn_sbfe(r[q], tile, 1);  // all ones or zero
    v[q].x = __builtin_bit_cast(float, __builtin_bit_cast(int, v[q].x) & keep);
    v[q].y = __builtin_bit_cast(float, __builtin_bit_cast(int, v[q].y) & keep);
  }
  if (any >> 2) {
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (r[q] >> (2 + tile) & 1) v[q].x = v[q].y = __builtin_nanf("");
  }
}
// (after a barrier) marks into their plane's row
__device__ __forceinline__ void store_hits(const RowMarks& W, const Marks& M, size_t row, int nx) {
  for (int x = (int)threadIdx.x; x < nx; x += kFftThreads) {
    const unsigned char h = W.hit[x];
    if (h) set_mark(M, row + x, (h & 1 ? W.tile[0] : 0u) | (h & 2 ? W.tile[1] : 0u));
  }
}

// Operand values enter the transforms times 1 / 2^e >= 1 / (NX NY) (exact; the
// table has the rest of the inverse transform's 1 / (NX NY)): every value on the
// way is then at most about as large as the largest operand or result, where
// sums over a plane would overflow for operands beyond 3e38 / (NX NY).
template <int R>
__device__ __forceinline__ void scale_points(float in_scale, float2* v) {
#pragma unroll
  for (int q = 0; q < R; ++q) v[q] = {v[q].x * in_scale, v[q].y * in_scale};
}

struct Geo {
  int ny, nx, nyp, nxp;  // grid and transform lengths
  int nz, nt, hz, ht;    // depths, samples; columns (pairs of them) of the transformed ones
  int tlo;               // first transformed sample
  int nk;                // pulses
  float in_scale;        // 1 / 2^e (see scale_points)
};

// ------------------------------------------------------------ x transforms
// Block: 16 columns (pairs of depths or samples 2 c0 .. 2 c0 + 31) of row iy of
// pulse (or volume) k.  Where rows of the grid are not whole lines, neighbouring
// tiles share some, so they go to one XCD at about the same time: blocks are
// dealt to the 8 XCDs round-robin, so of 8 kTilesNear successive ones kTilesNear
// neighbours are 8 apart.
struct RowAt {
  int k, iy, c0;
  int b;  // its number in that order
};
__host__ __device__ constexpr int col_tiles(int h) { return (h + kFftLanes - 1) / kFftLanes; }
constexpr int kTilesNear = 4;
__device__ __forceinline__ int near_order(int near) {
  const int b = (int)blockIdx.x, g = 8 * near, first = b / g * g;
  return first + g <= (int)gridDim.x ? first + (b & 7) * near + ((b - first) >> 3) : b;
}
__device__ __forceinline__ RowAt row_at(int ny, int h) {
  int b = near_order(kTilesNear);
  RowAt a;
  a.b = b;
  const int tiles = col_tiles(h);
  a.c0 = (b % tiles) * kFftLanes;
  b /= tiles;
  a.iy = b % ny;
  a.k = b / ny;
  return a;
}
// The same with kPulsesNear pulses of a tile next to each other, which read the
// same c (blocks: of a multiple of so many pulses).  us of spec_x_switch for 1,
// 2, 4 and 8 of them: 539, 367, 366 and 497 at 256 x 256 x 96 with 32 pulses,
// 1237, 1319, 1470 and 1433 at 320 x 320 x 128 with 40, 87, 83, 90 and 90 at 128
// x 128 x 64 with 32.
constexpr int kPulsesNear = 2;
__host__ __device__ constexpr int pulses_near(int nk) {
  return (nk + kPulsesNear - 1) / kPulsesNear * kPulsesNear;
}
__device__ __forceinline__ RowAt row_at_pulses(int ny, int h) {
  int b = near_order(kPulsesNear);
  RowAt a;
  a.b = b;
  a.k = b % kPulsesNear;
  b /= kPulsesNear;
  const int tiles = col_tiles(h);
  a.c0 = (b % tiles) * kFftLanes;
  b /= tiles;
  a.iy = b % ny;
  a.k += b / ny * kPulsesNear;
  return a;
}
// A lane's column: its pair of depths (samples) l and l + 1 of n >= 2, the first
// one `lo`, of which it holds two, one or (past the last column) none.  On a line
// of the grid two floats at byte offset `lane` from the tile's `base` hold them:
// a lane of one reads the value before it too (where the tile has just that one,
// base is the value before), a lane of none the tile's first two (dropped).
struct Pair {
  bool first, both;
  unsigned lane;
  int base;
  // the two floats, and the pair they hold: apart, so that a branch around loads
  // holds nothing that waits for one
  __device__ __forceinline__ float2 load(const float* base, unsigned byte) const {
    const float2u v = *(const float2u*)((const char*)base + byte);
    return {v.x, v.y};
  }
  __device__ __forceinline__ float2 pick(float2 v) const { return {first && !both ? v.y : v.x, v.y}; }
  __device__ __forceinline__ float2 get(const float* base, unsigned byte) const {
    return pick(load(base, byte));
  }
  __device__ __forceinline__ void put(float* base, unsigned byte, float2 v) const {
    if (both) *(float2u*)((char*)base + byte) = float2u{v.x, v.y};
    else if (first) *(float*)((char*)base + byte + 4) = v.x;
  }
};
__device__ __forceinline__ Pair pair_at(int c0, int h, int lo, int n) {
  const int c = threadIdx.x & 15, l = lo + 2 * (c0 + c);
  Pair p;
  p.first = c0 + c < h && l < n;
  p.both = c0 + c < h && l + 1 < n;
  const int start = lo + 2 * c0, one = start + 1 == n ? 1 : 0;
  p.base = start - one;
  p.lane = p.both ? 8u * (unsigned)c : p.first ? 8u * (unsigned)c - (one ? 0u : 4u) : 0u;
  return p;
}
// the lane's column of a spectrum's line (past the last column: the last)
struct Column {
  unsigned lane;
  bool ok;
};
__device__ __forceinline__ Column column_at(size_t c0, size_t h) {
  const unsigned c = threadIdx.x & 15, last = (unsigned)min((size_t)15, h - 1 - c0);
  return Column{8u * min(c, last), c <= last};
}

// where S comes from: the per-depth table, the fluence of each voxel, or
// diagonal switching (pulse volumes)
enum Src { kSrcDepth = 0, kSrcVoxel = 1, kSrcDiag = 2 };
template <int RND, int SRC>
__global__ __launch_bounds__(kFftThreads, 4) void spec_x_switch(
    const float* __restrict__ c, const float* __restrict__ phi, const float* phig,
    const float* __restrict__ stab_t, const float* __restrict__ f16, SwitchParams sw,
    float2* __restrict__ out, Geo G, FftDim D, Marks M, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at_pulses(G.ny, G.hz);
  if (at.k >= G.nk) return;
  const RowMarks W = row_marks(raw, D.n, nullptr, at.c0, G.hz);
  const Pair pr = pair_at(at.c0, G.hz, 0, G.nz);
  const int k = at.k, z = pr.first ? 2 * (at.c0 + (int)(threadIdx.x & 15)) : 0, z1 = pr.both ? z + 1 : z;
  // the pulses' mark planes
  const size_t grid = (size_t)G.ny * G.nx;
  const size_t mrow = (M.planes == 1 ? 0 : k * grid) + (size_t)at.iy * G.nx;
  const size_t vol = grid * G.nz;
  const size_t row = (size_t)at.iy * G.nx * G.nz + pr.base;
  const unsigned pitch = 4u * (unsigned)G.nz;
  const float sc = RND == kRndF16 ? f16[0] : 1.0f, inv = RND == kRndF16 ? f16[1] : 1.0f;
  float w[2][kMaxSpecies];
  if constexpr (SRC == kSrcDepth) {
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s) {
      const float* st = stab_t + ((size_t)k * sw.ns + s) * G.nz;
      w[0][s] = s < sw.ns ? st[z] : 0.0f;
      w[1][s] = s < sw.ns ? st[z1] : 0.0f;
    }
  }
  auto load = [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    // points of a volume's row; past the grid they are its last column (their
    // values are dropped)
    unsigned off[R];
    fft::offsets(pitch, pr.lane, x0, step, G.nx, off);
    auto get = [&](const float* volume, float2 (&to)[R]) {
#pragma unroll
      for (int q = 0; q < R; ++q)
        to[q] = pr.get(volume + row, off[q]);
    };
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = {0.0f, 0.0f};
    if constexpr (SRC == kSrcDiag) {
      float2 cv[R], ph[R];
      get(c + (size_t)k * vol, cv);
      if (sw.per_voxel) {
        get(phi, ph);
      } else {
        const float2 pz = {phi[z], phi[z1]};
#pragma unroll
        for (int q = 0; q < R; ++q) ph[q] = pz;
      }
#pragma unroll
      for (int q = 0; q < R; ++q) v[q] = {ph[q].x * cv[q].x, ph[q].y * cv[q].y};
    } else if constexpr (SRC == kSrcDepth) {
#pragma unroll
      for (int s = 0; s < kMaxSpecies; ++s)
        if (s < sw.ns) {
          float2 cv[R];
          get(c + (size_t)s * vol, cv);
#pragma unroll
          for (int q = 0; q < R; ++q) {
            v[q].x = __builtin_fmaf(w[0][s], cv[q].x, v[q].x);
            v[q].y = __builtin_fmaf(w[1][s], cv[q].y, v[q].y);
          }
        }
    } else {
      float2 ph[R], pg[R];
      get(phi, ph);
#pragma unroll
      for (int q = 0; q < R; ++q) pg[q] = phig ? ph[q] : float2{1.0f, 1.0f};
      if (phig && phig != phi) get(phig, pg);
      for (int s = 0; s < sw.ns; ++s) {
        float2 cv[R];
        get(c + (size_t)s * vol, cv);
#pragma unroll
        for (int q = 0; q < R; ++q) {
          v[q].x = __builtin_fmaf(switch_coef(sw, ph[q].x, pg[q].x, k, s), cv[q].x, v[q].x);
          v[q].y = __builtin_fmaf(switch_coef(sw, ph[q].y, pg[q].y, k, s), cv[q].y, v[q].y);
          if (q & 1) __builtin_amdgcn_sched_barrier(0);  // (few exponentials at a time: registers)
        }
      }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool in = x0 + q * step < G.nx;
      v[q].x = in && pr.first ? rnd<RND>(v[q].x, sc, inv) : 0.0f;
      v[q].y = in && pr.both ? rnd<RND>(v[q].y, sc, inv) : 0.0f;
    }
    mark_points<R>(W, M, mrow, x0, step, v);
    scale_points<R>(G.in_scale, v);
  };
  fft::first_stage<-1>(D, L, load);
  store_hits(W, M, mrow, G.nx);
  fft::middle_stages<-1>(D, L);
  float2* o = out + ((size_t)k * G.nyp + at.iy) * G.nxp * G.hz + at.c0;
  fft::last_stage<-1>(D, L, fft::strided_out<true>(o, 8u * G.hz, G.nxp, column_at(at.c0, G.hz).ok));
}

template <int RND>
__global__ __launch_bounds__(kFftThreads) void spec_x_pack(const float* __restrict__ y,
                                                           const float* __restrict__ f16,
                                                           float2* __restrict__ out, Geo G,
                                                           FftDim D, Marks M,
                                                           const unsigned* __restrict__ mask,
                                                           const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.ht);
  const RowMarks W = row_marks(raw, D.n, mask, at.c0, G.ht);
  const Pair pr = pair_at(at.c0, G.ht, G.tlo, G.nt);
  const size_t grid = (size_t)G.ny * G.nx, yrow = (size_t)at.iy * G.nx;
  const size_t mrow = (M.planes == 1 ? 0 : at.k * grid) + yrow;
  const float sc = RND == kRndF16 ? f16[2] : 1.0f, inv = RND == kRndF16 ? f16[3] : 1.0f;
  // (inside the row: the tiles end with its last sample's)
  const float* yk = y + (at.k * grid + yrow) * G.nt + pr.base;
  const unsigned pitch = 4u * (unsigned)G.nt;
  // loads past the grid read its last position (their values are dropped)
  auto load = [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    unsigned off[R];
    fft::offsets(pitch, pr.lane, x0, step, G.nx, off);
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = pr.get(yk, off[q]);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool in = x0 + q * step < G.nx;
      v[q].x = in && pr.first ? rnd<RND>(v[q].x, sc, inv) : 0.0f;
      v[q].y = in && pr.both ? rnd<RND>(v[q].y, sc, inv) : 0.0f;
    }
    mark_points<R>(W, M, mrow, x0, step, v);
    scale_points<R>(G.in_scale, v);
  };
  fft::first_stage<-1>(D, L, load);
  store_hits(W, M, mrow, G.nx);
  fft::middle_stages<-1>(D, L);
  float2* o = out + ((size_t)at.k * G.ny + at.iy) * G.nxp * G.ht + at.c0;
  fft::last_stage<-1>(D, L, fft::strided_out<true>(o, 8u * G.ht, G.nxp, column_at(at.c0, G.ht).ok));
}

// y = H b of a pulse
__global__ __launch_bounds__(kFftThreads) void spec_x_out(const float2* __restrict__ in,
                                                          float* __restrict__ y, Geo G, FftDim D,
                                                          Marks M, const unsigned* __restrict__ mask,
                                                          const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.ht);
  const Pair pr = pair_at(at.c0, G.ht, G.tlo, G.nt);
  const RowMarks W = row_marks(raw, D.n, mask, at.c0, G.ht);
  const size_t grid = (size_t)G.ny * G.nx, yrow = (size_t)at.iy * G.nx;
  const size_t mrow = (M.planes == 1 ? 0 : at.k * grid) + yrow;
  const NearWords nw = load_near(M, mrow, G.nx);
  const float2* i = in + ((size_t)at.k * G.nyp + at.iy) * G.nxp * G.ht + at.c0;
  fft::first_stage<1>(D, L, fft::strided<true>(i, 8u * G.ht, G.nxp, column_at(at.c0, G.ht).lane),
                      [&] { keep_near(W, D.n, nw); });
  fft::middle_stages<1>(D, L);
  float* yk = y + (at.k * grid + yrow) * G.nt + pr.base;
  const unsigned pitch = 4u * (unsigned)G.nt;
  fft::last_stage<1>(D, L, [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    reach_points<R>(W, x0, step, v);
    const unsigned o = (unsigned)x0 * pitch + pr.lane;
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (x0 < G.nx - q * step) pr.put(yk, o + (unsigned)(q * step) * pitch, v[q]);
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
    const unsigned* __restrict__ mask, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  __shared__ double sh[kFftThreads / 64];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.ht);
  const Pair pr = pair_at(at.c0, G.ht, G.tlo, G.nt);
  const RowMarks W = row_marks(raw, D.n, mask, at.c0, G.ht);
  const size_t grid = (size_t)G.ny * G.nx, yrow = (size_t)at.iy * G.nx;
  const size_t mrow = (M.planes == 1 ? 0 : at.k * grid) + yrow;
  const size_t rrow = (MR.planes == 1 ? 0 : at.k * grid) + yrow;
  const NearWords nw = load_near(M, mrow, G.nx);
  const float sc = RND == kRndF16 ? f16[2] : 1.0f, inv = RND == kRndF16 ? f16[3] : 1.0f;
  const Column col = column_at(at.c0, G.ht);
  const float2* i = in + ((size_t)at.k * G.nyp + at.iy) * G.nxp * G.ht + at.c0;
  fft::first_stage<1>(D, L, fft::strided<true>(i, 8u * G.ht, G.nxp, col.lane),
                      [&] { keep_near(W, D.n, nw); });
  fft::middle_stages<1>(D, L);
  // the row's samples of the tile; loads past the grid read inside it (values
  // dropped)
  const size_t row = (at.k * grid + yrow) * G.nt + pr.base;
  const unsigned pitch = 4u * (unsigned)G.nt;
  double ss = 0.0;
  fft::turn_stage(D, L, [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    unsigned off[R];
    fft::offsets(pitch, pr.lane, x0, step, G.nx, off);
    float2 pv[R];
    float2 yo[REC ? R : 1];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      pv[q] = {0.0f, 0.0f};
      if (pm) pv[q] = pr.load(pm + row, off[q]);
      if constexpr (REC) {
        yo[q] = {0.0f, 0.0f};
        if (!yc_first) yo[q] = pr.load(yc + row, off[q]);
      }
    }
    reach_points<R>(W, x0, step, v);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      pv[q] = pr.pick(pv[q]);
      if constexpr (REC) yo[q] = pr.pick(yo[q]);
      const bool in = x0 < G.nx - q * step, in0 = in && pr.first, in1 = in && pr.both;
      const float2 w = v[q];
      float2 d = {w.x - pv[q].x, w.y - pv[q].y};
      if constexpr (REC) {
        if (in0) {
          float2 n = w;
          if (!yc_first)
            n = {__builtin_fmaf(yc_beta, yo[q].x, w.x) * yc_inv,
                 __builtin_fmaf(yc_beta, yo[q].y, w.y) * yc_inv};
          pr.put(yc + row, off[q], n);
          const double e0 = (double)n.x - (double)pv[q].x,
                       e1 = in1 ? (double)n.y - (double)pv[q].y : 0.0;
          ss += e0 * e0 + e1 * e1;
        }
      } else {
        // (a product of floats is exact in FP64, so its sum rounds once)
        const double e0 = in0 ? (double)d.x : 0.0, e1 = in1 ? (double)d.y : 0.0;
        ss += __builtin_fma(e0, e0, e1 * e1);
      }
      d.x = in0 ? rnd<RND>(d.x, sc, inv) : 0.0f;
      d.y = in1 ? rnd<RND>(d.y, sc, inv) : 0.0f;
      v[q] = d;
    }
    mark_points<R>(W, MR, rrow, x0, step, v);
    scale_points<R>(G.in_scale, v);
  });
  store_hits(W, MR, rrow, G.nx);
  float2* ov = out + ((size_t)at.k * G.ny + at.iy) * G.nxp * G.ht + at.c0;
  fft::dit_stages(D, L, fft::strided_out<true>(ov, 8u * G.ht, G.nxp, col.ok));
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

// c-side output of H^T: a volume (species after S^T, or pulse) times the fluence
// (diagonal switching) or one
__global__ __launch_bounds__(kFftThreads) void spec_x_vox(const float2* __restrict__ in,
                                                          float* __restrict__ c,
                                                          const float* __restrict__ phi,
                                                          int phi_mode, Geo G, FftDim D, Marks M,
                                                          const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const RowAt at = row_at(G.ny, G.hz);
  const Pair pr = pair_at(at.c0, G.hz, 0, G.nz);
  const RowMarks W = row_marks(raw, D.n, nullptr, at.c0, G.hz);
  // (planes of their own: volumes are pulses)
  const size_t grid = (size_t)G.ny * G.nx, yrow = (size_t)at.iy * G.nx;
  const size_t mrow = (M.planes == 1 ? 0 : at.k * grid) + yrow;
  const NearWords nw = load_near(M, mrow, G.nx);
  const float2* i = in + ((size_t)at.k * G.nyp + at.iy) * G.nxp * G.hz + at.c0;
  fft::first_stage<1>(D, L, fft::strided<true>(i, 8u * G.hz, G.nxp, column_at(at.c0, G.hz).lane),
                      [&] { keep_near(W, D.n, nw); });
  fft::middle_stages<1>(D, L);
  const size_t row = yrow * G.nz + pr.base;
  float* ck = c + at.k * grid * G.nz + row;
  const unsigned pitch = 4u * (unsigned)G.nz;
  fft::last_stage<1>(D, L, [&](auto rc, int x0, int step, float2* v) {
    constexpr int R = decltype(rc)::value;
    if (!pr.first) return;
    const unsigned o = (unsigned)x0 * pitch + pr.lane;
    float2 pz = {1.0f, 1.0f};
    if (phi_mode == 1) pz = pr.get(phi + pr.base, pr.lane);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const unsigned oq = o + (unsigned)(q * step) * pitch;
      float2 ph = pz;
      if (phi_mode == 2 && x0 < G.nx - q * step) ph = pr.get(phi + row, oq);
      v[q] = {ph.x * v[q].x, ph.y * v[q].y};
    }
    reach_points<R>(W, x0, step, v);
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (x0 < G.nx - q * step) pr.put(ck, o + (unsigned)(q * step) * pitch, v[q]);
  });
}

// c[s][v] = sum_k S_v[k][s] b[k][v], per-voxel fluence
__global__ __launch_bounds__(256) void spec_st(const float* __restrict__ b, float* __restrict__ c,
                                               const float* __restrict__ phi, const float* phig,
                                               SwitchParams sw, size_t vol, const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  const size_t v = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= vol) return;
  const float ph = phi[v];
  const float pg = !phig ? 1.0f : phig == phi ? ph : phig[v];
  float acc[kMaxSpecies];
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s) acc[s] = 0.0f;
  for (int k = 0; k < sw.nk; ++k) {
    const float bv = b[(size_t)k * vol + v];
#pragma unroll
    for (int s = 0; s < kMaxSpecies; ++s)
      if (s < sw.ns) acc[s] = __builtin_fmaf(switch_coef(sw, ph, pg, k, s), bv, acc[s]);
  }
#pragma unroll
  for (int s = 0; s < kMaxSpecies; ++s)
    if (s < sw.ns) c[(size_t)s * vol + v] = acc[s];
}

// ------------------------------------------------------------- y transform
// Block: 16 columns of image k (of all kappa_x: a row's columns lie in one line);
// points of rows 0 .. n_in - 1 (the others are zero), outputs of rows 0 ..
// n_out - 1.  in and out may be one buffer: every point is read before the first
// barrier.
template <int SIGN>
__global__ __launch_bounds__(kFftThreads) void spec_y(const float2* in, float2* out, unsigned cols,
                                                      int rows_in, int rows_out, int n_in,
                                                      int n_out, FftDim D,
                                                      const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const fft::Lds L = fft::carve(raw, D);
  const unsigned tiles = (cols + kFftLanes - 1) / kFftLanes;
  const unsigned k = blockIdx.x / tiles, c0 = (blockIdx.x - k * tiles) * kFftLanes;
  const unsigned pitch = 8u * cols;
  const Column col = column_at(c0, cols);
  const float2* i = in + (size_t)k * rows_in * cols + c0;
  // (the grid's side is the shorter one)
  fft::first_stage<SIGN>(D, L, fft::strided<(SIGN > 0)>(i, pitch, n_in, col.lane));
  fft::middle_stages<SIGN>(D, L);
  float2* o = out + (size_t)k * rows_out * cols + c0;
  fft::last_stage<SIGN>(D, L, fft::strided_out<(SIGN < 0)>(o, pitch, n_out, col.ok));
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

__device__ __forceinline__ float quad_swap(float v) {    // lane j <- j ^ 1
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));
}

// Values of one pulse at four consecutive contracted indices of two 16-wide
// tiles A and B, separated from the images of their pairs: index 2j is
// (Z(kappa) + conj Z(-kappa)) / 2 and index 2j + 1 is (Z(kappa) - conj
// Z(-kappa)) / 2i; the halves are in the table's scale.  A lane's result is its
// own part (real for even lanes, imaginary for odd ones); the part that meets
// the imaginary table is the neighbouring lane's.  The even lane reads tile A,
// the odd one tile B (zp, zm: its own), and each hands the other its part: a
// load covers a whole line of both tiles, and no value is read twice.
__device__ __forceinline__ void unpair(const float2* zp, const float2* zm, int c, float (&A)[4],
                                       float (&B)[4]) {
  const float4 a = *(const float4*)zp, b = *(const float4*)zm;
  const float re[4] = {a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w};
  const float im[4] = {a.y - b.y, b.x - a.x, a.w - b.w, b.z - a.z};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float other = quad_swap(c ? re[i] : im[i]);
    A[i] = c ? other : re[i];
    B[i] = c ? im[i] : other;
  }
}

// The first of the pairs of sample tiles that a product takes: pairs are lines,
// and a position of an odd number of tiles starts inside one every other time
// (256 x 256 x 96 with 13 tiles: H's product 1390 us without this, 1220 with it).
__device__ __forceinline__ int first_tile(int ht, size_t at) { return (ht & 8) && (at & 1) ? -1 : 0; }

// Packs a pulse's products (an even lane's real, an odd one's imaginary parts;
// four consecutive rows Y0 .. Y3) into its pairs' images: Z(kappa) = Y0 + i Y1 on
// even lanes, Z(-kappa) = conj Y0 + i conj Y1 on odd ones.
__device__ __forceinline__ f32x4 pair_pack(f32x4 v, int c) {
  float m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) m[i] = quad_swap(v[i]);
  const float s0 = v[1] + m[0], s1 = v[3] + m[2];
  const float d0 = v[0] - m[1], d1 = v[2] - m[3];
  return f32x4{c ? s0 : d0, c ? -d0 : s0, c ? s1 : d1, c ? -d1 : s1};
}
// and stores tiles A and B: the even lane tile A's and the odd one tile B's
// values at kappa and -kappa (op: its own tile's at kappa, neg further at
// ok: the lane has a pulse and its tile is there
__device__ __forceinline__ void pair_store(f32x4 va, f32x4 vb, float2* op, ptrdiff_t neg, int c, bool ok,
                                           bool self) {
  const f32x4 a = pair_pack(va, c), b = pair_pack(vb, c);
  f32x4 p, m;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float r = quad_swap(c ? a[i] : b[i]);
    p[i] = c ? r : a[i];
    m[i] = c ? b[i] : r;
  }
  if (ok) {
    *(f32x4*)op = p;
    if (!self) *(f32x4*)(op + neg) = m;
  }
}

// (mask, [t tiles], the tile's 16-depth blocks, is an argument of its own: known
// not to alias, it comes by scalar loads, which wait for no store)
struct GemmArgs {
  const float* tab;       // [nf][nblk][real, imaginary][64][4]
  int nblk, ntt;          // blocks of a frequency, t tiles
  int nyp, nxp, lz, lt, nk;
  const float2* in;
  float2* out;
  // H^T with S^T: the species' coefficients [K][S][Nz]
  const float* stab_t;
  int ns, nz;
  const int* gate;
};

// Y = T B.  A wave holds eight pulses (16 real columns); its operand for all
// depths sits in registers, the table's 16 x 16 blocks stream past it (the
// block's waves share them through the caches).
template <int ZC>
__global__ __launch_bounds__(512, ZC <= 4 ? 8 : ZC <= 8 ? 7 : 4) void spec_gemm_fwd(
    GemmArgs A, const unsigned* __restrict__ mask) {
  if (A.gate && *A.gate) return;  // a device stop test has ended the solve
  const int f = (int)blockIdx.x;
  const Freq F = freq_at(f, A.nyp, A.nxp);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 4, n = lane & 15, c = n & 1;
  const int k = wave * 8 + (n >> 1);
  const bool ok = k < A.nk;
  const size_t img = (size_t)(ok ? k : 0) * A.nyp * A.nxp;
  const int hz = A.lz / 2, ht = A.lt / 2;
  const float2* zp = A.in + (img + F.at) * hz + 2 * g;
  const float2* zm = A.in + (img + F.neg) * hz + 2 * g;
  float bs[ZC][4];
  const float sg = c ? 1.0f : -1.0f;
#pragma unroll
  for (int zc = 0; zc < ZC; zc += 2) {
    if (zc * 16 < A.lz) {
      // (no second tile: the first one's again, which no block meets)
      const int own = zc * 8 + ((zc + 1) * 16 < A.lz ? 8 * c : 0);
      unpair(zp + own, zm + own, c, bs[zc], bs[zc + 1]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) bs[zc][i] = bs[zc + 1][i] = 0.0f;
    }
  }
  // (a uniform base and a lane's offset, and the way from kappa to -kappa: registers)
  float2* op = A.out + (img + F.at) * ht + 2 * g + 8 * c;
  const ptrdiff_t neg = ((ptrdiff_t)F.neg - (ptrdiff_t)F.at) * ht;
  const float4* tab = (const float4*)A.tab + (size_t)f * A.nblk * 128;
  float4 ar = tab[lane], ai = tab[64 + lane];  // (the table ends with a spare block)
  for (int tt = first_tile(ht, F.at); tt < A.ntt; tt += 2) {
    f32x4 y[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const unsigned m = tt + u >= 0 && tt + u < A.ntt ? mask[tt + u] : 0u;
      f32x4 a0 = {0.0f, 0.0f, 0.0f, 0.0f}, a1 = a0;
#pragma unroll
      for (int zc = 0; zc < ZC; ++zc)
        if (m >> zc & 1u) {
          const float r[4] = {ar.x, ar.y, ar.z, ar.w}, q[4] = {ai.x, ai.y, ai.z, ai.w};
          tab += 128;
          ar = tab[lane];
          ai = tab[64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            a0 = __builtin_amdgcn_mfma_f32_16x16x4f32(r[i], bs[zc][i], a0, 0, 0, 0);
            a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(q[i], sg * quad_swap(bs[zc][i]), a1, 0, 0, 0);
          }
        }
      y[u] = a0 + a1;
    }
    pair_store(y[0], y[1], op + tt * 8, neg, c, ok && tt + c >= 0 && tt + c < A.ntt, F.self);
  }
}

// G = conj(T)^T R, the accumulators of all depths in registers; ST: S^T over
// the pulses in LDS, species written instead of pulses.
template <int ZC, bool ST>
__global__ __launch_bounds__(512, ZC <= 4 ? 8 : ZC <= 8 ? 7 : 4) void spec_gemm_adj(
    GemmArgs A, const unsigned* __restrict__ mask) {
  if (A.gate && *A.gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  const int f = (int)blockIdx.x;
  const Freq F = freq_at(f, A.nyp, A.nxp);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 4, n = lane & 15, c = n & 1;
  const int k = wave * 8 + (n >> 1);
  const bool ok = k < A.nk;
  const size_t img = (size_t)(ok ? k : 0) * A.nyp * A.nxp;
  const int hz = A.lz / 2, ht = A.lt / 2;
  const float2* zp = A.in + (img + F.at) * ht + 2 * g;
  const ptrdiff_t away = ((ptrdiff_t)F.neg - (ptrdiff_t)F.at) * ht;
  const float sg = c ? -1.0f : 1.0f;
  f32x4 acc[ZC];
#pragma unroll
  for (int zc = 0; zc < ZC; ++zc) acc[zc] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const float4* tab = (const float4*)A.tab + (size_t)f * A.nblk * 128;
  float4 ar = tab[lane], ai = tab[64 + lane];
  for (int tt = first_tile(ht, F.at); tt < A.ntt; tt += 2) {
    const unsigned ms[2] = {tt >= 0 ? mask[tt] : 0u, tt + 1 < A.ntt ? mask[tt + 1] : 0u};
    if ((ms[0] | ms[1]) == 0) continue;
    float rs[2][4];
    // (one tile alone is read twice)
    const int own = 8 * min(max(tt + c, 0), A.ntt - 1);
    unpair(zp + own, zp + own + away, c, rs[0], rs[1]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      // conj(T): real columns meet +imaginary parts, imaginary ones -real parts
      float ro[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) ro[i] = sg * quad_swap(rs[u][i]);
#pragma unroll
      for (int zc = 0; zc < ZC; ++zc)
        if (ms[u] >> zc & 1u) {
          const float r[4] = {ar.x, ar.y, ar.z, ar.w}, q[4] = {ai.x, ai.y, ai.z, ai.w};
          tab += 128;
          ar = tab[lane];
          ai = tab[64 + lane];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc[zc] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[i], rs[u][i], acc[zc], 0, 0, 0);
            acc[zc] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[i], ro[i], acc[zc], 0, 0, 0);
          }
        }
    }
  }
  if constexpr (!ST) {
    float2* op = A.out + (img + F.at) * hz + 2 * g + 8 * c;
    const ptrdiff_t neg = ((ptrdiff_t)F.neg - (ptrdiff_t)F.at) * hz;
#pragma unroll
    for (int zc = 0; zc < ZC; zc += 2)
      if (zc * 16 < A.lz)
        pair_store(acc[zc], acc[zc + 1], op + zc * 8, neg, c, ok && (zc + c) * 16 < A.lz, F.self);
  } else {
    float* gb = (float*)raw;  // [nk][lz][2]
    if (ok) {
#pragma unroll
      for (int zc = 0; zc < ZC; ++zc)
        if (zc * 16 < A.lz) {
#pragma unroll
          for (int j = 0; j < 4; ++j) gb[((size_t)k * A.lz + zc * 16 + 4 * g + j) * 2 + c] = acc[zc][j];
        }
    }
    __syncthreads();
    const float4* gv = (const float4*)raw;
    for (int i = (int)threadIdx.x; i < A.ns * hz; i += (int)blockDim.x) {
      const int s = i / hz, j = i - s * hz;
      float2 s0 = {0.0f, 0.0f}, s1 = {0.0f, 0.0f};
      if (2 * j < A.nz) {
        const int next = 2 * j + 1 < A.nz ? 1 : 0;
        const float* w = A.stab_t + (size_t)s * A.nz + 2 * j;
        for (int q = 0; q < A.nk; ++q, w += (size_t)A.ns * A.nz) {
          const float4 v = gv[(size_t)q * hz + j];
          s0 = fft::cfma(w[0], float2{v.x, v.y}, s0);
          s1 = fft::cfma(w[next], float2{v.z, v.w}, s1);
        }
        if (!next) s1 = {0.0f, 0.0f};
      }
      float2* o = A.out + (size_t)s * A.nyp * A.nxp * hz + j;
      o[F.at * hz] = float2{s0.x - s1.y, s0.y + s1.x};
      if (!F.self) o[F.neg * hz] = float2{s0.x + s1.y, s1.x - s0.y};
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
// joined per column, then the columns over 2 R + 1 neighbours.  The last block to
// have read a row clears its marks.
__global__ __launch_bounds__(256) void spec_reach(Marks M, int ny, int nx, int r,
                                                  const int* __restrict__ gate) {
  if (gate && *gate) return;  // a device stop test has ended the solve
  extern __shared__ __attribute__((aligned(16))) unsigned char raw[];
  unsigned* row = (unsigned*)raw;           // [nx]
  int* done = (int*)raw + nx;               // [1 + 2 R + 1]: how many rows to clear, and which
  const int iy = (int)blockIdx.x % ny, p = (int)blockIdx.x / ny;
  const size_t plane = (size_t)p * ny * nx;
  const int y0 = max(0, iy - r), y1 = min(ny - 1, iy + r);
  if (threadIdx.x == 0) done[0] = 0;
  for (int x = (int)threadIdx.x; x < nx; x += 256) {
    unsigned f = 0;
    for (int y = y0; y <= y1; ++y) f |= M.at[plane + (size_t)y * nx + x];
    row[x] = f;
  }
  __syncthreads();
  for (int y = y0 + (int)threadIdx.x; y <= y1; y += 256) {
    const int readers = min(ny - 1, y + r) - max(0, y - r) + 1;
    if (atomicAdd(&M.seen[p * ny + y], 1) == readers - 1) done[1 + atomicAdd(&done[0], 1)] = y;
  }
  for (int x = (int)threadIdx.x; x < nx; x += 256) {
    unsigned f = 0;
    for (int i = max(0, x - r); i <= min(nx - 1, x + r); ++i) f |= row[i];
    M.near[plane + (size_t)iy * nx + x] = f;
  }
  __syncthreads();
  for (int i = 0; i < done[0]; ++i) {
    const int y = done[1 + i];
    for (int x = (int)threadIdx.x; x < nx; x += 256) M.at[plane + (size_t)y * nx + x] = 0u;
    if (threadIdx.x == 0) M.seen[p * ny + y] = 0;
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

// the power of two at or above NX NY
double plane_scale(int nx, int ny) { return std::exp2(std::ceil(std::log2((double)nx * (double)ny))); }

Geo geo_of(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  Geo G;
  G.ny = P->g.ny;
  G.nx = P->g.nx;
  G.nyp = Q.ny;
  G.nxp = Q.nx;
  G.nz = P->g.nz;
  G.nt = P->g.nt;
  G.hz = Q.lz / 2;
  G.ht = Q.lt / 2;
  G.tlo = Q.tlo;
  G.nk = P->g.n_pulses;
  G.in_scale = (float)(1.0 / plane_scale(Q.nx, Q.ny));
  return G;
}

// marks of H's operand (b) and of H^T's (r): pulse volumes of their own have a
// plane each, species that every pulse mixes share one
int mark_planes(const psoam_plan* P) { return P->sw.diag ? P->g.n_pulses : 1; }
Marks marks_b(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  return Marks{Q.d_at_b, Q.d_near_b, Q.d_seen, mark_planes(P)};
}
Marks marks_r(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  return Marks{Q.d_at_r, Q.d_near_r, Q.d_seen, mark_planes(P)};
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

// widens the marks of the operand just made
hipError_t reach(const psoam_plan* P, const Marks& M, hipStream_t s) {
  const int ny = P->g.ny, nx = P->g.nx;
  return go(spec_reach, (size_t)M.planes * ny, 256, sizeof(unsigned) * ((size_t)nx + 2 * P->R + 2), s, M,
            ny, nx, P->R, gate_now());
}

GemmArgs gemm_args(const psoam_plan* P, bool adj) {
  const SpecPlan& Q = *P->spec;
  GemmArgs A;
  A.tab = adj ? Q.d_ta : Q.d_tf;
  A.nblk = Q.nblk;
  A.ntt = Q.lt / 16;
  A.nyp = Q.ny;
  A.nxp = Q.nx;
  A.lz = Q.lz;
  A.lt = Q.lt;
  A.nk = P->g.n_pulses;
  A.in = (const float2*)(adj ? Q.d_y : Q.d_x);
  A.out = (float2*)(adj ? Q.d_g : Q.d_y);
  A.stab_t = P->d_stab_t;
  A.ns = P->sw.ns;
  A.nz = P->g.nz;
  A.gate = gate_now();
  return A;
}

// S^T inside the product: per-depth fluence, species mixed
bool st_in_gemm(const psoam_plan* P) { return P->d_stab_t && !P->sw.diag; }

// phi^gamma of each voxel (see switch_coef)
const float* rates(const psoam_plan* P) {
  return P->sw.gamma == 0.0f ? nullptr : P->sw.gamma == 1.0f ? P->d_phi : P->spec->d_rate;
}

// c-side images of H^T
int adj_images(const psoam_plan* P) { return st_in_gemm(P) ? P->sw.ns : P->g.n_pulses; }

#define SPEC_HIP(call)                 \
  do {                                 \
    hipError_t _e = (call);            \
    if (_e != hipSuccess) return _e;   \
  } while (0)

// a transform along y of `images` images of h columns a position
template <class K>
hipError_t y_pass(K kern, int images, int h, const void* in, void* out, const Geo& G, int rows_in,
                  int rows_out, int n_in, int n_out, const FftDim& Y, hipStream_t s) {
  const unsigned cols = (unsigned)G.nxp * (unsigned)h;
  return go(kern, (size_t)images * ((cols + kFftLanes - 1) / kFftLanes), kFftThreads, fft_lds(G.nyp), s,
            (const float2*)in, (float2*)out, cols, rows_in, rows_out, n_in, n_out, Y, gate_now());
}

}  // namespace

size_t spec_partials(const psoam_plan* P) {
  const SpecPlan& Q = *P->spec;
  return (size_t)P->g.n_pulses * P->g.ny * col_tiles(Q.lt / 2) + kIdleSums;
}

hipError_t spec_switch(const psoam_plan* P, const float* c, hipStream_t s) {
  SpecPlan& Q = *P->spec;
  const Geo G = geo_of(P);
  const FftDim X = dim_of(Q, 1), Y = dim_of(Q, 0);
  const Marks M = marks_b(P);
  const size_t nb = (size_t)pulses_near(G.nk) * G.ny * col_tiles(G.hz);
  auto x = [&](auto kern) {
    return go(kern, nb, kFftThreads, row_lds(G.nxp), s, c, P->d_phi, rates(P), P->d_stab_t, P->d_f16, P->sw,
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
  SPEC_HIP(reach(P, M, s));
  return y_pass(spec_y<-1>, G.nk, G.hz, Q.d_x, Q.d_x, G, G.nyp, G.nyp, G.ny, G.nyp, Y, s);
}

// (r's reach is found beside the pass that makes r: what follows only reads it,
// so that H^T may run again on the same r)
hipError_t spec_pack(const psoam_plan* P, const float* y, hipStream_t s) {
  SpecPlan& Q = *P->spec;
  const Geo G = geo_of(P);
  const FftDim X = dim_of(Q, 1);
  const Marks M = marks_r(P);
  const size_t nb = (size_t)G.nk * G.ny * col_tiles(G.ht);
  auto x = [&](auto kern) {
    return go(kern, nb, kFftThreads, row_lds(G.nxp), s, y, P->d_f16, (float2*)Q.d_r, G, X, M,
              Q.d_mask, gate_now());
  };
  switch (rnd_of(P)) {
    case kRndBf16: SPEC_HIP(x(spec_x_pack<kRndBf16>)); break;
    case kRndF16: SPEC_HIP(x(spec_x_pack<kRndF16>)); break;
    default: SPEC_HIP(x(spec_x_pack<kRndNone>)); break;
  }
  return reach(P, M, s);
}

hipError_t spec_band(const psoam_plan* P, int mode, float* out, const float* pmeas,
                     double* partial, hipStream_t s, float* yc, double yc_beta, int yc_first,
                     bool sums) {
  SpecPlan& Q = *P->spec;
  const Geo G = geo_of(P);
  const FftDim X = dim_of(Q, 1), Y = dim_of(Q, 0);
  const int waves = (G.nk + 7) / 8;  // eight pulses a wave
  const Marks MB = marks_b(P);
  if (mode != 2) {
    const GemmArgs A = gemm_args(P, false);
    const int zc = Q.lz / 16;
    if (zc <= 4) SPEC_HIP(go(spec_gemm_fwd<4>, (size_t)Q.nf, waves * 64, 0, s, A, Q.d_mask));
    else if (zc <= 8) SPEC_HIP(go(spec_gemm_fwd<8>, (size_t)Q.nf, waves * 64, 0, s, A, Q.d_mask));
    else SPEC_HIP(go(spec_gemm_fwd<16>, (size_t)Q.nf, waves * 64, 0, s, A, Q.d_mask));
    SPEC_HIP(y_pass(spec_y<1>, G.nk, G.ht, Q.d_y, Q.d_y, G, G.nyp, G.nyp, G.nyp, G.ny, Y, s));
    const size_t nb = (size_t)G.nk * G.ny * col_tiles(G.ht);
    // samples [tlo, thi) are transformed
    const int thi = std::min(G.nt, G.tlo + Q.lt);
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
                Q.d_mask, gate_now());
      const Marks MR = marks_r(P);
    const float beta = (float)yc_beta, inv = (float)(1.0 / (1.0 + yc_beta));
    auto r = [&](auto kern) {
      return go(kern, nb, kFftThreads, row_lds(G.nxp), s, (const float2*)Q.d_y, pmeas, P->d_f16,
                (float2*)Q.d_r, yc, beta, inv, yc_first, partial, G, X, MB, MR, Q.d_mask, gate_now());
    };
    const bool rec = yc != nullptr;
    switch (rnd_of(P)) {
      case kRndBf16: SPEC_HIP(rec ? r(spec_x_resid<kRndBf16, true>) : r(spec_x_resid<kRndBf16, false>)); break;
      case kRndF16: SPEC_HIP(rec ? r(spec_x_resid<kRndF16, true>) : r(spec_x_resid<kRndF16, false>)); break;
      default: SPEC_HIP(rec ? r(spec_x_resid<kRndNone, true>) : r(spec_x_resid<kRndNone, false>)); break;
    }
    return reach(P, MR, s);
  }
  const Marks MR = marks_r(P);
  SPEC_HIP(y_pass(spec_y<-1>, G.nk, G.ht, Q.d_r, Q.d_y, G, G.ny, G.nyp, G.ny, G.nyp, Y, s));
  const GemmArgs A = gemm_args(P, true);
  const int zc = Q.lz / 16;
  const bool st = st_in_gemm(P);
  const size_t lds = st ? (size_t)G.nk * Q.lz * sizeof(float2) : 0;
  if (st) {
    if (zc <= 4) SPEC_HIP(go(spec_gemm_adj<4, true>, (size_t)Q.nf, waves * 64, lds, s, A, Q.d_mask));
    else if (zc <= 8) SPEC_HIP(go(spec_gemm_adj<8, true>, (size_t)Q.nf, waves * 64, lds, s, A, Q.d_mask));
    else SPEC_HIP(go(spec_gemm_adj<16, true>, (size_t)Q.nf, waves * 64, lds, s, A, Q.d_mask));
  } else {
    if (zc <= 4) SPEC_HIP(go(spec_gemm_adj<4, false>, (size_t)Q.nf, waves * 64, lds, s, A, Q.d_mask));
    else if (zc <= 8) SPEC_HIP(go(spec_gemm_adj<8, false>, (size_t)Q.nf, waves * 64, lds, s, A, Q.d_mask));
    else SPEC_HIP(go(spec_gemm_adj<16, false>, (size_t)Q.nf, waves * 64, lds, s, A, Q.d_mask));
  }
  const int na = adj_images(P);
  SPEC_HIP(y_pass(spec_y<1>, na, G.hz, Q.d_g, Q.d_g, G, G.nyp, G.nyp, G.nyp, G.ny, Y, s));
  const size_t nb = (size_t)na * G.ny * col_tiles(G.hz);
  const bool mix = !st && !P->sw.diag;  // per-voxel fluence: S^T after the pulses are back
  float* dst = mix ? (float*)Q.d_y : out;
  const int phi_mode = P->sw.diag ? (P->sw.per_voxel ? 2 : 1) : 0;
  SPEC_HIP(go(spec_x_vox, nb, kFftThreads, row_lds(G.nxp), s, (const float2*)Q.d_g, dst, P->d_phi,
              phi_mode, G, X, MR, gate_now()));
  if (mix) {
    const size_t vol = P->v_elems();
    SPEC_HIP(go(spec_st, (vol + 255) / 256, 256, 0, s, (const float*)Q.d_y, out, P->d_phi,
                rates(P), P->sw, vol, gate_now()));
  }
  return hipSuccess;
}

void spec_free(psoam_plan* P) {
  if (!P->spec) return;
  SpecPlan& Q = *P->spec;
  for (void* b : {Q.d_x, Q.d_y, Q.d_r, Q.d_g, (void*)Q.d_tf, (void*)Q.d_ta, (void*)Q.d_mask,
                  (void*)Q.d_rate, Q.d_twx, Q.d_twy, (void*)Q.d_marks})
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
  if (g.nz < 2 || g.nt < 2) return false;  // columns are pairs
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
  const int ni = (X.n - 1) / 2, edges = X.n % 2 ? 1 : 2;
  const size_t nf = (size_t)ni * Y.n + (size_t)edges * (Y.n / 2 + 1);
  const bool st = !g.phi_per_voxel && !P->sw.diag;
  const size_t img = (size_t)Y.n * X.n;
  // a complex value holds two depths or samples
  const size_t xb = (size_t)g.n_pulses * img * lz * 4;
  // per-voxel fluence: y's spectrum also holds the pulse volumes S^T reads,
  // which are the larger where the depths outnumber the samples
  const size_t yb =
      std::max((size_t)g.n_pulses * img * lt * 4, (size_t)g.n_pulses * P->v_elems() * sizeof(float));
  const size_t rb = (size_t)g.n_pulses * g.ny * X.n * lt * 4;
  const size_t gb = (size_t)(st ? P->sw.ns : g.n_pulses) * img * lz * 4;
  const size_t tb = (nf * nblk + 2) * 512 * sizeof(float);
  const size_t pb = (size_t)(X.n / 2 + 1) * F * 256 * sizeof(double2);
  const size_t grid = (size_t)g.ny * g.nx;
  // the transforms' offsets within a line are 32 bits, its positions 20
  X.derive();
  Y.derive();
  const size_t most = (size_t)std::max(lz, lt) * 4;
  if (std::max({X.n * std::max<size_t>(most, 4 * (size_t)std::max(g.nt, g.nz)),
                Y.reach(most * X.n)}) >= (1ull << 32) ||
      std::max(X.n, Y.n) >= (1 << 20))
    return false;
  // launch grids are 32-bit counts of blocks
  const size_t tiles_y = (size_t)X.n * (std::max(lz, lt) / 2) / 16 + 1;
  if (nf >= (1u << 31) || g.n_pulses * tiles_y >= (1u << 31)) return false;
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return false;
  const size_t need = xb + yb + rb + gb + 2 * tb + pb;
  // the direct form needs about the operands alone; this one stays where a
  // user's own arrays still have most of the card
  if (need > free_b / 3) {
    P->spec_short = true;
    return false;
  }
  if (!force) {
    // Predicted time of one A and one A^T: the launches, and the bytes of all
    // passes at 4.0 TB/s (a fit to 400 random geometries: half of the
    // predictions within 13%, 90% within 28%).  At 128 x 128 x 64 with 32
    // pulses and a footprint of 31 the pair takes 1.4 ms against the direct
    // form's 41 ms in FP32 and 3.2 ms in BF16; at 97 x 95 x 16 with a
    // footprint of 7 and 64 samples it takes 0.8 ms against 0.28 ms in BF16.
    const double a = 2.0 * g.n_pulses * g.ny * X.n * lz * 4 + 2.0 * xb + tb + 2.0 * yb + 2.0 * rb;
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
  Q.nf = nf;
  Q.nblk = nblk;
  Q.xb = xb;
  Q.rb = rb;
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
      P->spec_short = true;
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
  const bool rate = P->sw.per_voxel && !P->sw.diag && P->sw.gamma != 0.0f && P->sw.gamma != 1.0f;
  if (rate) alloc(&Q.d_rate, sizeof(float) * P->v_elems());
  alloc(&Q.d_twx, sizeof(float2) * X.n);
  alloc(&Q.d_twy, sizeof(float2) * Y.n);
  // marks and reach of b and of r, a word each per position and plane
  const size_t planes = mark_planes(P);
  const size_t mb = sizeof(unsigned) * planes * (4 * grid + (size_t)g.ny);
  alloc(&Q.d_marks, mb);
  Q.bytes = xb + yb + rb + gb + 2 * tb + mb + sizeof(float2) * ((size_t)X.n + Y.n) +
            sizeof(unsigned) * ntt + (rate ? sizeof(float) * P->v_elems() : 0);
  if (ok) {
    Q.d_at_b = (unsigned*)Q.d_marks;
    Q.d_at_r = Q.d_at_b + planes * grid;
    Q.d_near_b = Q.d_at_r + planes * grid;
    Q.d_near_r = Q.d_near_b + planes * grid;
    Q.d_seen = (int*)(Q.d_near_r + planes * grid);
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
    // nothing marked, nothing in reach; the table's spare blocks are read and
    // not used
    check(hipMemsetAsync(Q.d_marks, 0, mb, stream));
    check(hipMemsetAsync(Q.d_tf + (nf * nblk) * 512, 0, 1024 * sizeof(float), stream));
    check(hipMemsetAsync(Q.d_ta + (nf * nblk) * 512, 0, 1024 * sizeof(float), stream));
    if (rate)
      check(go(spec_rate, (P->v_elems() + 255) / 256, 256, 0, stream, P->d_phi, Q.d_rate, P->sw.gamma,
               P->v_elems()));
    // 1/2 from the pairs' separation, 1 / (NX NY) from the inverse transform
    // with the operands' scale taken out
    const double scale = 0.5 * plane_scale(X.n, Y.n) / ((double)X.n * (double)Y.n);
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
