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
// voxel and K steps.  us a step, tv_step_kernel -> this one: 400 -> 171 (320 x
// 320 x 128, 3 species), 198 -> 87 (256 x 256 x 96), 107 -> 40 (200 x 190 x 70),
// 28.5 -> 18.6 (128 x 128 x 64), 11.9 -> 7.7 (77 x 61 x 50, 2 species), 9.2 -> 3.5
// (32 x 32 x 16): large volumes are bound by HBM (5.3 TB/s with the overlap),
// small ones by a plane's barriers.  A workgroup owns a strip of x columns, all depths, and marches along
// y: plane y enters step 1, whose new duals enter step 2 one plane behind, and
// so on.  A thread keeps its columns' duals of the last plane of every step in
// registers (the y neighbours); the x and z neighbours go through LDS, three
// planes of it, two barriers a step.  The strip overlaps its neighbours by K
// columns on either side and its y range by K planes, which it computes and
// does not write (the values there are wrong by one more plane a step and
// never reach an output).  All depths in one strip: no overlap along z.
// Every value is the same expression in the same order as in tv_step_kernel,
// so results equal its bit for bit.
// A thread holds P positions (P = 5 at K = 4 takes 241 registers; 6 spill), the
// next plane's values among them, loaded a plane ahead.
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

template <int K, int P>
__global__ __launch_bounds__(kTvMarchThreads) void tv_march_kernel(TvMarch M) {
  if (M.gate && *M.gate) return;  // a device stop test has ended the solve
  constexpr int NT = kTvMarchThreads;
  extern __shared__ float tv_lds[];
  const int nz = M.nz, ny = M.ny, nx = M.nx;
  // one plane each of eta_x, eta_z and w, a column of slack on either side
  const int plane_lds = NT * P + 2 * nz;
  float* lx = tv_lds + nz;
  float* lz = lx + plane_lds;
  float* lw = lz + plane_lds;
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
  const int cols = M.tx + 2 * K;
  const size_t sbase = (size_t)sp * ny * nx * nz;
  const int ps = nx * nz;
  // per position: offset in a plane (clamped into it), and what it may do
  enum { kBackX = 1, kFwdX = 2, kBackZ = 4, kFwdZ = 8, kOut = 16 };
  int off[P];
  unsigned can[P];
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const int pos = tid + i * NT;
    const int c = pos / nz, z = pos - c * nz;
    const int x = xa + c;
    const bool in = c < cols && x >= 0 && x < nx;
    off[i] = min(max(x, 0), nx - 1) * nz + z;
    can[i] = (in && x > 0 ? kBackX : 0) | (in && x < nx - 1 ? kFwdX : 0) | (z > 0 ? kBackZ : 0) |
             (z < nz - 1 ? kFwdZ : 0) | (in && c >= K && c < K + M.tx ? kOut : 0);
  }
  const float *zs = M.z + sbase, *uc = M.uc ? M.uc + sbase : nullptr,
              *up = M.up ? M.up + sbase : nullptr;
  float *ua = M.ua + sbase, *ub = M.ub + sbase;
  const size_t sv = M.sv;
  // the next plane's values, loaded an iteration ahead
  float nu[3][P], np[3][P], nzv[P];
  auto fetch = [&](int y) {
    const size_t o = (size_t)min(max(y, 0), ny - 1) * ps;
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        nu[d][i] = uc ? uc[d * sv + o + off[i]] : 0.0f;
        np[d][i] = up ? up[d * sv + o + off[i]] : 0.0f;
      }
      nzv[i] = zs[o + off[i]];
    }
  };
  // state of step s (0-based) between planes: eta_y, u_y and w of its last
  // plane; for s > 0 the x and z parts of the plane it takes next
  float ey[K][P], uy[K][P], wl[K][P];
  float ex[K][P], ez[K][P], ux[K][P], uz[K][P];  // [0] unused between planes
  float zr[K][P];                                // z of planes y, y - 1, ..
#pragma unroll
  for (int s = 0; s < K; ++s)
#pragma unroll
    for (int i = 0; i < P; ++i) {
      ey[s][i] = uy[s][i] = wl[s][i] = ex[s][i] = ez[s][i] = ux[s][i] = uz[s][i] = zr[s][i] = 0.0f;
    }
  float lxs[K > 1 ? K - 1 : 1][P], lzs[K > 1 ? K - 1 : 1][P];  // a step's new x and z parts
  float lux[K > 1 ? K - 1 : 1][P], luz[K > 1 ? K - 1 : 1][P];
  const int y0 = max(0, ya - K), y1 = ye - 1 + K;
  const float im = M.inv_mu, th = M.theta;
  fetch(y0);
  for (int y = y0; y <= y1; ++y) {
    // plane y into step 0
    float cy[P], vy[P];  // eta_y and u_y of the current step's plane
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
      for (int s = K - 1; s > 0; --s) zr[s][i] = zr[s - 1][i];
      zr[0][i] = nzv[i];
      ux[0][i] = nu[1][i];
      uz[0][i] = nu[2][i];
      vy[i] = nu[0][i];
      ex[0][i] = up ? __builtin_fmaf(M.beta[0], nu[1][i] - np[1][i], nu[1][i]) : nu[1][i];
      ez[0][i] = up ? __builtin_fmaf(M.beta[0], nu[2][i] - np[2][i], nu[2][i]) : nu[2][i];
      cy[i] = up ? __builtin_fmaf(M.beta[0], nu[0][i] - np[0][i], nu[0][i]) : nu[0][i];
    }
    if (y < y1) fetch(y + 1);
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const int q = y - s;  // this step's plane
#pragma unroll
      for (int i = 0; i < P; ++i) {
        lx[tid + i * NT] = ex[s][i];
        lz[tid + i * NT] = ez[s][i];
      }
      __syncthreads();
      float w[P];
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int p = tid + i * NT;
        float acc = 0.0f;
        if (q > 0) acc += ey[s][i];
        if (q < ny - 1) acc -= cy[i];
        const float bx = lx[p - nz], bz = lz[p - 1];
        if (can[i] & kBackX) acc += bx;
        if (can[i] & kFwdX) acc -= ex[s][i];
        if (can[i] & kBackZ) acc += bz;
        if (can[i] & kFwdZ) acc -= ez[s][i];
        w[i] = zr[s][i] - acc;
        lw[p] = w[i];
      }
      __syncthreads();
      const bool wx = q >= ya && q < ye, wy = q - 1 >= ya && q - 1 < ye;
      float* o = s == K - 1 ? ub : ua;
      const size_t oq = (size_t)max(q, 0) * ps, oy = (size_t)max(q - 1, 0) * ps;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        const int p = tid + i * NT;
        const float fx = lw[p + nz], fz = lw[p + 1];
        const float gx = can[i] & kFwdX ? fx - w[i] : 0.0f;
        const float gz = can[i] & kFwdZ ? fz - w[i] : 0.0f;
        const float gy = q - 1 < ny - 1 ? w[i] - wl[s][i] : 0.0f;
        const float tx = fminf(fmaxf(__builtin_fmaf(im, gx, ex[s][i]), -th), th);
        const float tz = fminf(fmaxf(__builtin_fmaf(im, gz, ez[s][i]), -th), th);
        const float ty = fminf(fmaxf(__builtin_fmaf(im, gy, ey[s][i]), -th), th);
        if (s >= K - 2 && (can[i] & kOut)) {
          if (wx) {
            o[sv + oq + off[i]] = tx;
            o[2 * sv + oq + off[i]] = tz;
          }
          if (wy) o[oy + off[i]] = ty;
        }
        if (s + 1 < K) {
          // the next step takes plane q - 1: its x and z parts were left here
          // by the plane before, its y part is this one's
          const float be = M.beta[s + 1 < K ? s + 1 : 0];
          const float nex = __builtin_fmaf(be, tx - ux[s][i], tx);
          const float nez = __builtin_fmaf(be, tz - uz[s][i], tz);
          const float ney = __builtin_fmaf(be, ty - uy[s][i], ty);
          // (swap in after the next step has used the old ones)
          ey[s][i] = cy[i];
          uy[s][i] = vy[i];
          cy[i] = ney;
          vy[i] = ty;
          lxs[s][i] = nex;
          lzs[s][i] = nez;
          lux[s][i] = tx;
          luz[s][i] = tz;
        } else {
          ey[s][i] = cy[i];
          uy[s][i] = vy[i];
        }
        wl[s][i] = w[i];
      }
    }
    // each step's new x and z parts wait for its successor's next plane
#pragma unroll
    for (int s = 0; s + 1 < K; ++s)
#pragma unroll
      for (int i = 0; i < P; ++i) {
        ex[s + 1][i] = lxs[s][i];
        ez[s + 1][i] = lzs[s][i];
        ux[s + 1][i] = lux[s][i];
        uz[s + 1][i] = luz[s][i];
      }
  }
}

// Registers of tv_march_kernel<K, P>, which bound the workgroups a CU holds.
constexpr int kMarchRegs[kTvMaxSteps + 1][6] = {
    {}, {}, {0, 50, 74, 110, 144, 176}, {0, 62, 86, 120, 156, 195}, {0, 74, 106, 150, 196, 241}};

// Launch shapes for k steps a launch, chosen with the plan: positions per
// thread, strip and range by a predicted time.  A step of a plane takes a
// workgroup alone 0.2 us for its barriers and 0.15 us per position of a
// thread, and a CU 0.2 us per position whoever's; the bytes are seven floats
// read and six written, the strips' overlap counted six tenths (the rest comes
// from the caches), at 6 TB/s; the shorter of the two adds four tenths.  Over
// seven volumes from 32 x 32 x 16 to 320 x 320 x 128 and every K and P the
// choice is within 2% of the fastest measured.
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
    const int held = std::max(1, std::min(4, waves / 2));
    for (int n = 1; n <= g.ny; ++n) {
      const int ty = (g.ny + n - 1) / n;
      const int tyb = (g.ny + ty - 1) / ty;
      const double per_cu = std::ceil((double)txb * tyb * g.n_species / 256.0);
      const double planes = ty + 2 * k;
      const double busy = std::max(planes * k * (0.2 + 0.15 * p) * std::ceil(per_cu / held),
                                   per_cu * planes * k * 0.2 * p);
      const double over = (double)std::min(g.nx, tx + 2 * k) / tx * std::min((double)g.ny, planes) / ty;
      const double voxels = (double)g.nx * g.ny * g.nz * g.n_species;
      const double bytes = voxels * (24.0 + 28.0 * (0.4 + 0.6 * over)) / 6e6;
      const double us = (3.0 + std::max(busy, bytes) + 0.4 * std::min(busy, bytes)) / k;
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
    const size_t lds = sizeof(float) * 3 * ((size_t)kTvMarchThreads * p + 2 * P->g.nz);
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
