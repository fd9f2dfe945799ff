// TV prox on the device, several dual steps a launch (Alg. alg:prox-inner).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "psoam_internal.h"

namespace psoam {

namespace {

// K dual steps of the TV prox in one pass over the volume (K = 2 to 4).
//
// tv_step_kernel moves ten floats per voxel and step at the rate of a copy (small
// volumes: 9 us a launch of latencies); this one reads seven and writes six per
// voxel and K steps.  us a step, tv_step_kernel -> this one: 400 -> 139 (320 x
// 320 x 128, 3 species), 198 -> 69 (256 x 256 x 96), 107 -> 33 (200 x 190 x 70),
// 28.5 -> 13.1 (128 x 128 x 64), 27 -> 10.8 (97 x 97 x 56), 9.2 -> 3.1 (32 x 32 x
// 16): large volumes move 3.5 TB/s beside a plane's arithmetic (half of the
// time) and LDS, small ones wait for a plane's barriers.  (With two barriers a
// step, the divergence's tests and the x and z parts in registers: 171, 87, 40,
// 18.6, 13 and 3.5 us; with strips split along z as well, less overlap but
// unaligned rows: 174 us at the largest.)  A workgroup owns a strip of x columns, all depths, and
// marches along y: plane y enters step 0, whose new duals enter step 1 one
// plane behind, and so on.  A thread keeps its columns' duals of the last plane
// of every step in registers (the y neighbours).  The x and z parts of eta wait
// for their step in LDS, where the neighbours read them; w is exchanged through
// two planes of LDS in turn, so that a step takes one barrier.  The strip
// overlaps its neighbours by K columns on either side and its y range by K
// planes, which it computes and does not write (the values there are wrong by
// one more plane a step and never reach an output).  All depths in one strip:
// no overlap along z.  A thread holds P positions (P = 5 at K = 4 takes 256
// registers; 6 would spill), the next plane's values among them, loaded a plane
// ahead.
// Every value is the same expression in the same order as in tv_step_kernel, so
// results equal its bit for bit.  The duals of the last column, row and depth
// are zero (they start so, and the differences there are taken as zero), and so
// is eta_x of the column before the first: the divergence needs no test at the
// borders.
constexpr int kTvMarchThreads = 512;
struct TvMarch {
  const float *z, *uc, *up;   // u_j and u_{j-1} (null: zero, equal to u_j)
  float *ua, *ub;             // u_{j+K-1}, u_{j+K}
  float beta[kTvMaxSteps];    // of the K steps
  float inv_mu, theta;
  int tx, ty;                 // columns and rows a workgroup writes
  int txb, tyb;               // strips along x, ranges along y
  int ny, nx, nz;
  size_t sv;                  // species-voxels
  const int* gate;
};

__device__ __forceinline__ float ld_at(const float* base, unsigned byte) {
  return *(const float*)((const char*)base + byte);
}
__device__ __forceinline__ void st_at(float* base, unsigned byte, float v) {
  *(float*)((char*)base + byte) = v;
}

template <int K, int P>
__global__ __launch_bounds__(kTvMarchThreads) void tv_march_kernel(TvMarch M) {
  if (M.gate && *M.gate) return;  // a device stop test has ended the solve
  constexpr int NT = kTvMarchThreads, PL = NT * P;
  extern __shared__ float tv_lds[];
  const int nz = M.nz, ny = M.ny, nx = M.nx;
  // planes: eta_x and eta_z of every step, two of w; a column of slack on
  // either side (reads beyond a plane meet its neighbour's values, in columns
  // that are never written)
  float* lx = tv_lds + nz;
  float* lz = lx + K * PL;
  float* lw = lz + K * PL;
  // neighbouring strips from the same L2 (blocks are dealt to the 8 XCDs
  // round-robin)
  const int n = (int)gridDim.x;
  int b = (n & 7) == 0 ? ((int)blockIdx.x & 7) * (n >> 3) + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
  const int xb = b % M.txb;
  b /= M.txb;
  const int yb = b % M.tyb, sp = b / M.tyb;
  const int tid = (int)threadIdx.x;
  const int ya = yb * M.ty, ye = min(ny, ya + M.ty);
  const int xa = xb * M.tx - K;  // the strip's first column, overlap included
  const size_t sbase = (size_t)sp * ny * nx * nz;
  const int ps = nx * nz;
  // per position: byte offset in a plane (clamped into it), and what it may do
  unsigned off[P];
  bool grid_x[P], fwd_x[P], fwd_z[P], out[P];
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int pos = tid + i * NT;
    const int c = pos / nz, z = pos - c * nz;
    const int x = xa + c;
    off[i] = 4u * (unsigned)(min(max(x, 0), nx - 1) * nz + z);
    grid_x[i] = x >= 0;
    fwd_x[i] = x >= 0 && x < nx - 1;
    fwd_z[i] = z < nz - 1;
    out[i] = c >= K && c < K + M.tx && x < nx;
  }
  // absent duals: z is read in their place and dropped
  const bool has_c = M.uc != nullptr, has_p = M.up != nullptr;
  const float *zs = M.z + sbase, *uc = has_c ? M.uc + sbase : zs, *up = has_p ? M.up + sbase : zs;
  float *ua = M.ua + sbase, *ub = M.ub + sbase;
  const size_t sv = M.sv, sc = has_c ? sv : 0, spv = has_p ? sv : 0;
  // the next plane's values, loaded an iteration ahead
  float nu[3][P], np[3][P], nzv[P];
  auto fetch = [&](int y) {
    const size_t o = (size_t)min(max(y, 0), ny - 1) * ps;
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int i = 0; i < P; ++i) {
        nu[d][i] = ld_at(uc + d * sc + o, off[i]);
        np[d][i] = ld_at(up + d * spv + o, off[i]);
      }
#pragma unroll
    for (int i = 0; i < P; ++i) nzv[i] = ld_at(zs + o, off[i]);
  };
  // state of step s between planes: eta_y, u_y and w of its last plane; u_x and
  // u_z of the plane it takes next, whose eta_x and eta_z are in LDS
  float ey[K][P], uy[K][P], wl[K][P], ux[K][P], uz[K][P];
  float zr[K][P];        // z of the plane each step takes next
  float cy0[P], vy0[P];  // eta_y and u_y of step 0's next plane
#pragma unroll
  for (int s = 0; s < K; ++s)
#pragma unroll
    for (int i = 0; i < P; ++i)
      ey[s][i] = uy[s][i] = wl[s][i] = ux[s][i] = uz[s][i] = zr[s][i] = 0.0f;
  const int y0 = max(0, ya - K), y1 = ye - 1 + K;
  const float im = M.inv_mu, th = M.theta;
  // the fetched plane becomes step 0's next
  auto enter = [&](float (&u0)[P], float (&u2)[P], float (&z0)[P]) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      float u[3], h[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const bool in = d != 1 || grid_x[i];
        u[d] = has_c && in ? nu[d][i] : 0.0f;
        h[d] = has_p && in ? __builtin_fmaf(M.beta[0], u[d] - np[d][i], u[d]) : u[d];
      }
      lx[tid + i * NT] = h[1];
      lz[tid + i * NT] = h[2];
      u0[i] = u[1];
      u2[i] = u[2];
      cy0[i] = h[0];
      vy0[i] = u[0];
      z0[i] = nzv[i];
    }
  };
  // eta_x and eta_z of step s's next plane and of the neighbours before
  float own_x[P], own_z[P], back_x[P], back_z[P];
  auto ask = [&](int s) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int p = tid + i * NT;
      own_x[i] = lx[s * PL + p];
      own_z[i] = lz[s * PL + p];
      back_x[i] = lx[s * PL + p - nz];
      back_z[i] = lz[s * PL + p - 1];
    }
  };
  // plane y into step 0, plane y - 1 into step 1, ..; w0: the plane of w that
  // step 0 uses
  auto plane = [&](int y, int w0) {
    // (opaque, so that the offsets stay 32 bits beside a scalar base)
#pragma unroll
    for (int i = 0; i < P; ++i) asm volatile("" : "+v"(off[i]));
    float cy[P], vy[P];                      // eta_y and u_y of the step's plane
    float hx[P], hz[P], htx[P], htz[P];      // for this step from the one before
    float e0[P], e1[P], z0[P];               // step 0's next
#pragma unroll
    for (int i = 0; i < P; ++i) {
      cy[i] = cy0[i];
      vy[i] = vy0[i];
    }
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const int q = y - s;  // this step's plane
      float* const lws = lw + ((w0 + s) & 1) * PL;
      float* const lxs = lx + s * PL;
      float* const lzs = lz + s * PL;
      float w[P], ex[P], ez[P];
#pragma unroll
      for (int i = 0; i < P; ++i) {
        ex[i] = own_x[i];
        ez[i] = own_z[i];
        float acc = 0.0f + ey[s][i];
        acc -= cy[i];
        acc += back_x[i];
        acc -= ex[i];
        acc += back_z[i];
        acc -= ez[i];
        w[i] = zr[s][i] - acc;
        lws[tid + i * NT] = w[i];
      }
      if (s == K - 1) enter(e0, e1, z0);  // (step 0 has read its plane)
      __syncthreads();
      if (s == K - 1 && y < y1) fetch(y + 2);
      // y differences inside the grid
      const bool fwd_y = q >= 1 && q < ny;
      const bool wx = q >= ya && q < ye, wy = q - 1 >= ya && q - 1 < ye;
      float* o = s == K - 1 ? ub : ua;
      const size_t oq = (size_t)max(q, 0) * ps, oy = (size_t)max(q - 1, 0) * ps;
      float *ox = o + sv + oq, *oz = o + 2 * sv + oq, *oyp = o + oy;
      float fx[P], fz[P];
#pragma unroll
      for (int i = 0; i < P; ++i) {
        fx[i] = lws[tid + i * NT + nz];
        fz[i] = lws[tid + i * NT + 1];
      }
      ask((s + 1) % K);
      // (all reads in flight before the first wait)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int p = tid + i * NT;
        asm volatile("" : "+v"(fx[i]), "+v"(fz[i]));
        const float gx = fwd_x[i] ? fx[i] - w[i] : 0.0f;
        const float gz = fwd_z[i] ? fz[i] - w[i] : 0.0f;
        const float gy = fwd_y ? w[i] - wl[s][i] : 0.0f;
        // (a NaN gives -th, as fmin of fmax does)
        const float tx = __builtin_amdgcn_fmed3f(__builtin_fmaf(im, gx, ex[i]), -th, th);
        const float tz = __builtin_amdgcn_fmed3f(__builtin_fmaf(im, gz, ez[i]), -th, th);
        const float ty = __builtin_amdgcn_fmed3f(__builtin_fmaf(im, gy, ey[s][i]), -th, th);
        if (s >= K - 2 && out[i]) {
          if (wx) {
            st_at(ox, off[i], tx);
            st_at(oz, off[i], tz);
          }
          if (wy) st_at(oyp, off[i], ty);
        }
        if (s > 0) {
          // this step's next plane, from the step before
          lxs[p] = hx[i];
          lzs[p] = hz[i];
        }
        const float be = M.beta[s + 1 < K ? s + 1 : 0];
        const float nex = __builtin_fmaf(be, tx - ux[s][i], tx);
        const float nez = __builtin_fmaf(be, tz - uz[s][i], tz);
        const float ney = __builtin_fmaf(be, ty - uy[s][i], ty);
        if (s > 0) {
          ux[s][i] = htx[i];
          uz[s][i] = htz[i];
        }
        ey[s][i] = cy[i];
        uy[s][i] = vy[i];
        wl[s][i] = w[i];
        if (s + 1 < K) {
          hx[i] = nex;
          hz[i] = nez;
          htx[i] = tx;
          htz[i] = tz;
          cy[i] = ney;
          vy[i] = ty;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
      for (int s = K - 1; s > 0; --s) zr[s][i] = zr[s - 1][i];
      zr[0][i] = z0[i];
      ux[0][i] = e0[i];
      uz[0][i] = e1[i];
    }
  };
  fetch(y0);
  enter(ux[0], uz[0], zr[0]);
  __syncthreads();
  fetch(y0 + 1);
  ask(0);
  for (int y = y0; y <= y1; ++y) plane(y, K & (y - y0) & 1);
}

size_t march_lds(int k, int p, int nz) {
  return sizeof(float) * ((size_t)(2 * k + 2) * kTvMarchThreads * p + 2 * nz);
}

// Registers of tv_march_kernel<K, P>, which bound the workgroups a CU holds.
constexpr int kMarchRegs[kTvMaxSteps + 1][6] = {
    {}, {}, {0, 39, 76, 106, 144, 177}, {0, 48, 91, 128, 175, 215}, {0, 54, 109, 144, 199, 256}};

// Launch shapes for k steps a launch, chosen with the plan: positions per
// thread, strip and range by a predicted time.  A step of a plane takes a
// workgroup alone 0.15 us for its barrier and 0.1 us per position of a thread,
// and a CU 0.16 us per position whoever's, with 0.15 us a plane to load and
// store it; the bytes are seven floats read and six written, the strips'
// overlap counted six tenths (the rest comes from the caches), at 6 TB/s; the
// shorter of the two adds two tenths.  Over nine volumes from 32 x 32 x 16 to
// 320 x 320 x 128 and every K and P the choice is within 8% of the fastest
// measured, in seven of them the fastest.
double march_shape(const psoam_geom& g, int k, TvMarchShape& S) {
  double best = 0.0;
  S.p = 0;
  for (int p = 1; p <= 5; ++p) {
    const int cols = kTvMarchThreads * p / g.nz;
    int tx = cols - 2 * k;
    if (tx < 2 * k) continue;  // more overlap than strip
    tx = std::min(tx, g.nx);
    const int txb = (g.nx + tx - 1) / tx;
    tx = (g.nx + txb - 1) / txb;
    const int waves = 512 / ((kMarchRegs[k][p] + 7) / 8 * 8);  // per SIMD
    const int held = std::max(1, std::min({4, waves / 2, (int)(160 * 1024 / march_lds(k, p, g.nz))}));
    for (int n = 1; n <= g.ny; ++n) {
      const int ty = (g.ny + n - 1) / n;
      const int tyb = (g.ny + ty - 1) / ty;
      const double per_cu = std::ceil((double)txb * tyb * g.n_species / 256.0);
      const double planes = ty + 2 * k;
      const double busy = std::max(planes * k * (0.15 + 0.1 * p) * std::ceil(per_cu / held),
                                   per_cu * planes * p * (0.15 + 0.16 * k));
      const double over = (double)std::min(g.nx, tx + 2 * k) / tx * std::min((double)g.ny, planes) / ty;
      const double voxels = (double)g.nx * g.ny * g.nz * g.n_species;
      const double bytes = voxels * (24.0 + 28.0 * (0.4 + 0.6 * over)) / 6e6;
      const double us = (3.0 + std::max(busy, bytes) + 0.2 * std::min(busy, bytes)) / k;
      if (S.p == 0 || us < best) {
        best = us;
        S = TvMarchShape{p, tx, ty, txb, tyb};
      }
    }
  }
  return best;
}

}  // namespace

void tv_march_plan(psoam_plan* P) {
  const psoam_geom& g = P->g;
  // a single step: 40 bytes a voxel at the rate of a copy, 9 us at the least
  double best = std::max(9.0, 40e-6 * (double)P->c_elems() / 4.2);
  P->tv_march = 0;
  for (int k = 2; k <= kTvMaxSteps; ++k) {
    TvMarchShape& S = P->tv_shape[k];
    const double us = march_shape(g, k, S);
    if (S.p && us < best) {
      best = us;
      P->tv_march = k;
    }
  }
}

int tv_march_steps(const psoam_plan* P, int left) {
  const int most = P->tv_march;
  if (most < 2 || left < 2) return 1;
  int k = std::min(most, left);
  // no single step at the end where two or three a launch avoid it
  if (left - k == 1) k = k > 2 ? k - 1 : P->tv_shape[3].p ? 3 : 2;
  return P->tv_shape[k].p ? k : 1;
}

hipError_t launch_tv_march(const psoam_plan* P, int k, float* ua, float* ub, const float* z,
                           const float* u_cur, const float* u_prev, const float* beta, float inv_mu,
                           float theta, hipStream_t s) {
  if (k < 2 || k > kTvMaxSteps || P->tv_shape[k].p == 0) return hipErrorInvalidValue;
  const TvMarchShape& S = P->tv_shape[k];
  TvMarch M;
  M.z = z;
  M.uc = u_cur;
  M.up = u_prev;
  M.ua = ua;
  M.ub = ub;
  for (int i = 0; i < kTvMaxSteps; ++i) M.beta[i] = i < k ? beta[i] : 0.0f;
  M.inv_mu = inv_mu;
  M.theta = theta;
  M.tx = S.tx;
  M.ty = S.ty;
  M.txb = S.txb;
  M.tyb = S.tyb;
  M.ny = P->g.ny;
  M.nx = P->g.nx;
  M.nz = P->g.nz;
  M.sv = P->c_elems();
  M.gate = gate_now();
  const unsigned nb = (unsigned)(S.txb * S.tyb * P->g.n_species);
  auto go = [&](auto kern, int p) {
    const size_t lds = march_lds(k, p, P->g.nz);
    if (lds > 64 * 1024)
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(nb), dim3(kTvMarchThreads), lds, s, M);
  };
#define PSOAM_MARCH(PP)                                                        \
  case PP:                                                                     \
    if (k == 2) go(tv_march_kernel<2, PP>, PP);                                \
    else if (k == 3) go(tv_march_kernel<3, PP>, PP);                           \
    else go(tv_march_kernel<4, PP>, PP);                                       \
    break;
  switch (S.p) {
    PSOAM_MARCH(1)
    PSOAM_MARCH(2)
    PSOAM_MARCH(3)
    PSOAM_MARCH(4)
    PSOAM_MARCH(5)
    default: return hipErrorInvalidValue;
  }
#undef PSOAM_MARCH
  return hipGetLastError();
}

}  // namespace psoam
