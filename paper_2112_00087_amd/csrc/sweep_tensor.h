// Multi-vector product of the frequency sweep in the tensor form (tensor.h):
// Y[:, c] = A(k_c) X[:, c] for the columns of an [n][s] block on a box whose
// nodes lie on a tensor-product grid.
//
// A wave's lanes are s columns by 64 / s groups of kTwI nodes along x; it
// takes kTwJ lines along y and marches a run of planes along z.  Each plane
// step loads the (kTwI + 2)(kTwJ + 2) rows of the patch and its rim, each a
// contiguous run of s columns, at 64 columns one step ahead of their use
// (fewer columns hold the x entries per lane, and those registers are gone),
// forms per plane
//     a = Mx x, b = Kx x;  p = My a, q = My b + Ky a - m_c p
// and adds p and q, weighted with the plane's entries of Kz and Mz, to the
// sums of its rows in the planes below, at and above, kept in registers.
// There is no matrix to read or to broadcast over the columns: the 1-D
// entries are wave-uniform (y, z: scalar loads) or held in registers (x), and
// the frequency enters through m_c and, on the wall nodes, i k_c beta.  In
// complex128 Kx x is formed from differences (its rows sum to zero but for the
// walls), so it rounds relative to the result; FP64 sums of complex64 vectors
// need no such care.  The product is bound by the block's read and write
// (67 us of copy at 80x48x40 and 64 columns, where it takes 92 repeated alone and
// 109 between a solve's vector passes, which leave less of x in the caches; the
// stencil form took 163 us, streaming 27 pairs a row through the broadcast unit); the
// patch is 2 x 2 because its 4 rows in 16 loads (4 from L1 / L2 per row,
// against 9 in the stencil form) still leave two waves per SIMD with the next
// plane's loads in flight.  With an absorption field 118 : 200 us there; fewer
// columns then leave one wave per SIMD: at two, 54 registers went to scratch memory
// (32 columns at 80x48x40 124 -> 76 us, 16 at 20x12x10 12.1 -> 8.0 us).
// On small blocks the march is a chain of load latencies: 13 : 126 us at
// 80x48x40 and 4 columns, 10.8 : 13.4 us at 37x25x19 and 13, laid out as 16
// (a later run on another card: 9.3).  One plane a wave with all its loads at
// once took 11.2 : 9.3 us there, and 6.9 : 7.3 us at 4.
// Arithmetic is FP64 for both vector types.
#pragma once

#include "tensor.h"

constexpr int kTwI = 2, kTwJ = 2;
constexpr int kTwWaves = 4;          // waves per block, adjacent along x

struct TwOp {
  const TzAxis* tab = nullptr;       // axis tables x, y, z without frequency (NULL: no tensor form)
  const double* eta = nullptr;       // absorption field per element
  int nx = 0, ny = 0, nz = 0;
  z_t beta[6] = {};                  // wall admittances (0 where the wall has no faces)
};

// acc += i k beta v
__device__ __forceinline__ void tw_wall(z_t& acc, double k, z_t beta, z_t v) {
  cfma(acc, z_t{-k * beta.im, k * beta.re}, v);
}

// The rows of the padding beyond the box's nodes stay zero.
template <typename T>
__device__ __forceinline__ void tw_zero_tail(int64_t n, int64_t tail, cx<T>* __restrict__ Y) {
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < tail; e += int64_t(gridDim.x) * blockDim.x)
    Y[n + e] = cx<T>{T(0), T(0)};
}

template <typename T, int LS, bool ETA>
__global__ void __launch_bounds__(kTwWaves * kWave)
    __attribute__((amdgpu_waves_per_eu(ETA && LS < 6 ? 1 : 2, ETA && LS < 6 ? 1 : 2))) k_spmm_tz(TwOp A, int npx, int npy, int zc, int64_t tail, const double* __restrict__ kc,
              const cx<T>* __restrict__ X, cx<T>* __restrict__ Y) {
  constexpr int S = 1 << LS, G = kWave >> LS;
  tw_zero_tail((int64_t(A.nx) * A.ny * A.nz) << LS, tail, Y);
  constexpr bool AHEAD = LS == 6 && !ETA;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  int L = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = L % npx;
  L /= npx;
  const int by = L % npy, bz = L / npy;
  const int NX = A.nx, NY = A.ny, NZ = A.nz;
  const int c = lane & (S - 1);
  const int i0 = ((bx * kTwWaves + w) * G + (lane >> LS)) * kTwI;   // the lane's first node along x
  const int j0 = by * kTwJ;
  const int z0 = bz * zc, z1 = z0 + zc < NZ ? z0 + zc : NZ;
  const int zs = z0 > 0 ? z0 - 1 : 0, ze = z1 < NZ ? z1 : NZ - 1;
  if ((bx * kTwWaves + w) * G * kTwI >= NX) return;
  const double k = kc[2 * c], m = kc[2 * c + 1];
  const int64_t plane = int64_t(NX) * NY;

  TzAxis ax[kTwI];
#pragma unroll
  for (int u = 0; u < kTwI; ++u) ax[u] = A.tab[i0 + u < NX ? i0 + u : NX - 1];
  const bool x_lo = i0 == 0, x_hi = i0 <= NX - 1 && i0 + kTwI >= NX;   // the patch holds a wall node
  TzAxis ay[kTwJ];
#pragma unroll
  for (int t = 0; t < kTwJ; ++t) ay[t] = tz_uniform(A.tab, NX + (j0 + t < NY ? j0 + t : NY - 1));

  // the rim beyond a wall reads the wall's own nodes: its weights are 0
  auto clampi = [](int v, int n) { return v < 0 ? 0 : (v < n ? v : n - 1); };
  unsigned off[kTwI + 2];
#pragma unroll
  for (int u = 0; u < kTwI + 2; ++u) off[u] = (unsigned(clampi(i0 - 1 + u, NX)) << LS) + unsigned(c);
  auto load = [&](int zz, z_t (&v)[kTwJ + 2][kTwI + 2]) {
#pragma unroll
    for (int t = 0; t < kTwJ + 2; ++t) {
      const cx<T>* line = X + ((zz * plane + int64_t(clampi(j0 - 1 + t, NY)) * NX) << LS);
#pragma unroll
      for (int u = 0; u < kTwI + 2; ++u) v[t][u] = tz_ld(line + off[u]);
    }
  };
  // absorption field of the element columns i0 - 1 .. i0 + kTwI - 1 and lines j0 - 1 .. j0 + kTwJ - 1
  auto load_eta = [&](int ez, double (&e)[kTwJ + 1][kTwI + 1]) {
#pragma unroll
    for (int t = 0; t < kTwJ + 1; ++t) {
      const double* line =
          A.eta + (int64_t(clampi(ez, NZ - 1)) * (NY - 1) + clampi(j0 - 1 + t, NY - 1)) * (NX - 1);
#pragma unroll
      for (int u = 0; u < kTwI + 1; ++u) e[t][u] = line[unsigned(clampi(i0 - 1 + u, NX - 1))];
    }
  };

  z_t s0[kTwJ][kTwI], s1[kTwJ][kTwI];   // sums of the rows in this plane and the next
#pragma unroll
  for (int t = 0; t < kTwJ; ++t)
#pragma unroll
    for (int u = 0; u < kTwI; ++u) s0[t][u] = s1[t][u] = z_t{0.0, 0.0};
  z_t nv[kTwJ + 2][kTwI + 2];
  double elo[ETA ? kTwJ + 1 : 1][ETA ? kTwI + 1 : 1], ehi[ETA ? kTwJ + 1 : 1][ETA ? kTwI + 1 : 1];
  if constexpr (AHEAD) load(zs, nv);
  if constexpr (ETA) load_eta(zs - 1, ehi);
  for (int zz = zs; zz <= ze; ++zz) {
    z_t v[kTwJ + 2][kTwI + 2];
    if constexpr (AHEAD) {
#pragma unroll
      for (int t = 0; t < kTwJ + 2; ++t)
#pragma unroll
        for (int u = 0; u < kTwI + 2; ++u) v[t][u] = nv[t][u];
      if (zz < ze) load(zz + 1, nv);
    } else {
      load(zz, v);
    }
    if constexpr (ETA) {
#pragma unroll
      for (int t = 0; t < kTwJ + 1; ++t)
#pragma unroll
        for (int u = 0; u < kTwI + 1; ++u) elo[t][u] = ehi[t][u];
      load_eta(zz, ehi);
    }
    const TzAxis Z = tz_uniform(A.tab, NX + NY + zz);
    const bool z_wall = zz == 0 || zz == NZ - 1;
#pragma unroll
    for (int u = 0; u < kTwI; ++u) {
      const TzAxis& C = ax[u];
      // x stage on the patch's lines
      z_t a[kTwJ + 2], b[kTwJ + 2];
#pragma unroll
      for (int t = 0; t < kTwJ + 2; ++t) {
        a[t] = tz_mul(C.md, v[t][u + 1]);
        tz_add(a[t], C.ml, v[t][u]);
        tz_add(a[t], C.mh, v[t][u + 2]);
        if constexpr (sizeof(T) == 8) {
          b[t] = tz_mul(C.kl, v[t][u] - v[t][u + 1]);
          tz_add(b[t], C.kh, v[t][u + 2] - v[t][u + 1]);
        } else {
          b[t] = tz_mul(C.kd, v[t][u + 1]);
          tz_add(b[t], C.kl, v[t][u]);
          tz_add(b[t], C.kh, v[t][u + 2]);
        }
      }
      if (x_lo && u == 0) {
#pragma unroll
        for (int t = 0; t < kTwJ + 2; ++t) tw_wall(b[t], k, A.beta[0], v[t][1]);
      }
      if (x_hi && i0 + u == NX - 1) {
#pragma unroll
        for (int t = 0; t < kTwJ + 2; ++t) tw_wall(b[t], k, A.beta[1], v[t][u + 1]);
      }
#pragma unroll
      for (int t = 0; t < kTwJ; ++t) {
        const TzAxis& B = ay[t];
        const int j = j0 + t;
        z_t p = tz_mul(B.md, a[t + 1]), q = tz_mul(B.md, b[t + 1]);
        tz_add(p, B.ml, a[t]);
        tz_add(p, B.mh, a[t + 2]);
        tz_add(q, B.ml, b[t]);
        tz_add(q, B.mh, b[t + 2]);
        tz_add(q, B.kd, a[t + 1]);
        tz_add(q, B.kl, a[t]);
        tz_add(q, B.kh, a[t + 2]);
        tz_add(q, -m, p);
        if (j == 0) tw_wall(q, k, A.beta[2], a[t + 1]);
        if (j == NY - 1) tw_wall(q, k, A.beta[3], a[t + 1]);
        z_t below = tz_mul(Z.ml, q), here = tz_mul(Z.md, q), above = tz_mul(Z.mh, q);
        tz_add(below, Z.kl, p);
        tz_add(here, Z.kd, p);
        tz_add(above, Z.kh, p);
        if (z_wall) {
          if (zz == 0) tw_wall(here, k, A.beta[4], p);
          if (zz == NZ - 1) tw_wall(here, k, A.beta[5], p);
        }
        if constexpr (ETA) {
          // element sums of the plane: columns u (left) and u + 1 (right), lines t and t + 1
          z_t lo = {0.0, 0.0}, hi = {0.0, 0.0};
#pragma unroll
          for (int ex = 0; ex < 2; ++ex) {
            const double wx = ex ? C.mh : C.ml;
            z_t h[3];
#pragma unroll
            for (int l = 0; l < 3; ++l) {
              const z_t far = ex ? v[t + l][u + 2] : v[t + l][u];
              h[l] = tz_mul(wx, z_t{fma(2.0, v[t + l][u + 1].re, far.re), fma(2.0, v[t + l][u + 1].im, far.im)});
            }
#pragma unroll
            for (int ey = 0; ey < 2; ++ey) {
              const z_t far = ey ? h[2] : h[0];
              const z_t e = tz_mul(ey ? B.mh : B.ml, z_t{fma(2.0, h[1].re, far.re), fma(2.0, h[1].im, far.im)});
              tz_add(lo, elo[t + ey][u + ex], e);
              tz_add(hi, ehi[t + ey][u + ex], e);
            }
          }
          const double wl = m * Z.ml, wh = m * Z.mh;   // i k^2 (m = k^2 with an absorption field)
          tz_addi(below, wl, lo);
          tz_addi(here, 2.0 * wl, lo);
          tz_addi(here, 2.0 * wh, hi);
          tz_addi(above, wh, hi);
        }
        const int i = i0 + u, zo = zz - 1;
        if (zo >= z0 && i < NX && j < NY)
          Y[((zo * plane + int64_t(j) * NX + i) << LS) + c] = ccast<T>(s0[t][u] + below);
        s0[t][u] = s1[t][u] + here;
        s1[t][u] = above;
      }
    }
  }
  if (z1 == NZ) {
#pragma unroll
    for (int t = 0; t < kTwJ; ++t)
#pragma unroll
      for (int u = 0; u < kTwI; ++u)
        if (i0 + u < NX && j0 + t < NY)
          Y[(((NZ - 1) * plane + int64_t(j0 + t) * NX + i0 + u) << LS) + c] = ccast<T>(s0[t][u]);
  }
}
