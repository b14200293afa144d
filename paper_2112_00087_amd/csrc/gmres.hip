// Restarted GMRES(m) on the right-Jacobi operator, for every segment of a
// segmented system (added beside the paper's Sec. 4 solvers).
//
// Arnoldi uses classical Gram-Schmidt with one re-orthogonalisation (CGS2),
// h1 = V^H w, w1 = w - V h1, h2 = V^H w1, w2 = w1 - V h2, in three passes
// over the basis per step instead of four:
//   1. the product w = A v_j, and h1's partial sums from the same rows;
//   2. w1 formed in registers from the row's basis entries, which stay in
//      registers for h2's partial sums (no write of w1);
//   3. w2 = w - V (h1 + h2) written as the next basis vector, with the
//      partial sums of ||w2||^2.
// The basis is stored unnormalised: v_i = s_i V_i with s_i = 1 / ||w2|| of
// the step that made it (1 / beta for V_0), applied wherever V is read, so
// no pass rescales it.  Each pass is followed by one small finalize kernel
// (coefficients; then the Hessenberg column, the complex Givens rotations
// and the residual estimate, in FP64 on the device), so a whole restart
// cycle is queued without a host round trip; the host reads the
// per-segment state once per cycle.  With storage type float the basis and
// the operator are complex64 while the Gram-Schmidt coefficients, H and
// the rotations remain FP64.
#include "ops.h"

namespace {

constexpr int kGmMaxM = 128;   // largest restart length

constexpr int NV = 8;    // basis vectors per multi-dot chunk

struct GmSt {
  double beta, thr2, est, inv_next;
  int k, done, cyc, nan;
  int iters, off;      // off: cyc as of the step before (k_few_prod)
};

struct GmArr {         // per-segment small arrays (FP64)
  z_t* H;              // [(m+1) x m] column-major, per segment
  double* cs;          // [m]
  z_t* sn;             // [m]
  z_t* g;              // [m+1]
  z_t* y;              // [m]
  z_t* h1;             // [m+1] first-pass coefficients
  z_t* h2;             // [m+1] second-pass coefficients
  double* vs;          // [m+1] scale of each stored basis vector (v_i = vs_i V_i)
  int m;
};

template <typename T> __device__ __forceinline__ z_t zd(cx<T> a) { return ccast<double>(a); }

// V0 = f - A u; partial ||V0||^2
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_resid(Seg L, SellOp<T> A, const cx<T>* __restrict__ f,
                                                  const cx<T>* __restrict__ u, cx<T>* __restrict__ V0,
                                                  double* part) {
  SumTile t = prod_tile_sums<F>(L);
  double q[1] = {0.0};
  for_rows<F, true>(A, t, u, [=](int64_t row) { return f[row]; },
              [&](int64_t row, cx<T> y, cx<T> fv) {
                const cx<T> rs = ccast<T>(zd(fv) - zd(y));
                V0[row] = rs;
                q[0] += norm2(zd(rs));
              });
  store_partials<1>(q, part, t);
}

__global__ void k_beta_fin(Seg L, GmSt* st, GmArr G, const double* part) {
  int s = blockIdx.x;
  double o[1];
  seg_sums<1>(L, part, s, o);
  if (threadIdx.x == 0) {
    const double rr = o[0];
    GmSt& S = st[s];
    double b = sqrt(rr);
    S.beta = b;
    S.est = b;
    S.k = 0;
    S.nan = !isfinite(rr);
    S.done = (rr <= S.thr2) || S.nan;
    S.cyc = S.off = S.done;
    S.inv_next = b > 0.0 ? 1.0 / b : 0.0;
    G.vs[int64_t(s) * (G.m + 1)] = S.inv_next;
    z_t* g = G.g + int64_t(s) * (G.m + 1);
    g[0] = z_t{b, 0.0};
    for (int i = 1; i <= G.m; ++i) g[i] = z_t{0.0, 0.0};
  }
}

// Partial sums of 2 (j + 1) quantities, 16 per chunk of 8 basis vectors:
// chunk_to_lds reduces one chunk's 16 values within each wave and puts the
// waves' sums in LDS; after all chunks, lds_to_partials (one barrier) adds
// the waves in order and stores quantity u of chunk c at
// part[(16 c + u) nblk + tile]: each quantity's block partials contiguous,
// the layout k_mdot_fin reads.  Fixed summation order.
constexpr int kMaxChunks = (128 + 1 + NV - 1) / NV;
typedef double ChunkLds[kMaxChunks][2 * NV][kBlock / kWave];

// Wave sums of 16 quantities by recursive halving: at each of the first
// four exchanges (lane distance 32, 16, 8, 4) a lane keeps half of its
// quantities, adds its partner's copies of them and hands over the other
// half, so 8 + 4 + 2 + 1 values cross lanes instead of 16 x 6; then lane
// distances 2 and 1 finish the one quantity each lane holds.  Afterwards
// lane l holds the wave sum of quantity 8 b5 + 4 b4 + 2 b3 + b2 (b = the
// bits of l).  A fixed order: the result does not depend on timing.
__device__ __forceinline__ double wave_sum16(const double (&q)[2 * NV], int lane, int* which) {
  double a[8], b[4], c[2], d;
  const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8, h2 = lane & 4;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double keep = h5 ? q[8 + k] : q[k], give = h5 ? q[k] : q[8 + k];
    a[k] = keep + __shfl_xor(give, 32, kWave);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double keep = h4 ? a[4 + k] : a[k], give = h4 ? a[k] : a[4 + k];
    b[k] = keep + __shfl_xor(give, 16, kWave);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double keep = h3 ? b[2 + k] : b[k], give = h3 ? b[k] : b[2 + k];
    c[k] = keep + __shfl_xor(give, 8, kWave);
  }
  {
    const double keep = h2 ? c[1] : c[0], give = h2 ? c[0] : c[1];
    d = keep + __shfl_xor(give, 4, kWave);
  }
  d += __shfl_xor(d, 2, kWave);
  d += __shfl_xor(d, 1, kWave);
  *which = 8 * h5 + 4 * h4 + 2 * h3 + h2;
  return d;
}

__device__ __forceinline__ void chunk_to_lds(const double (&q)[2 * NV], int c, ChunkLds& lds) {
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  int u = 0;
  const double v = wave_sum16(q, lane, &u);
  if ((lane & 3) == 0) lds[c][u][w] = v;
}

__device__ __forceinline__ void lds_to_partials(const ChunkLds& lds, int nchunk, double* part, int nblk, int tile) {
  __syncthreads();
  for (int e = threadIdx.x; e < nchunk * 2 * NV; e += kBlock) {
    const int c = e / (2 * NV), u = e % (2 * NV);
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) t += lds[c][u][i];
    part[(int64_t(c) * 2 * NV + u) * nblk + tile] = t;
  }
}

// conj(a) b accumulated into q[0] (re), q[1] (im)
__device__ __forceinline__ void dot_acc(double* q, z_t a, z_t b) {
  q[0] = fma(a.re, b.re, fma(a.im, b.im, q[0]));
  q[1] = fma(a.re, b.im, fma(-a.im, b.re, q[1]));
}

// Pass 1: w = A v_j = s_j (A V_j), and the partial sums of h1_i = v_i^H w
// (i <= j) from the same rows.
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_gs_prod(Seg L, SellOp<T> A, const GmSt* st, GmArr G,
                                                    const cx<T>* __restrict__ V, int64_t ld, int j,
                                                    cx<T>* __restrict__ w, double* __restrict__ part) {
  __shared__ ChunkLds lds;
  Tile t = tile_of(L);
  if (st[t.seg].cyc) return;
  const double* vs = G.vs + int64_t(t.seg) * (G.m + 1);
  const z_t y = vs[j] * zd(sell_row_form<F>(A, t.row, V + int64_t(j) * ld));
  const cx<T> ys = ccast<T>(y);
  w[t.row] = ys;
  const z_t wv = zd(ys);
  const int nchunk = (j + NV) / NV;
  for (int c = 0; c < nchunk; ++c) {
    double q[2 * NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int i = c * NV + u;
      q[2 * u] = q[2 * u + 1] = 0.0;
      if (i <= j) dot_acc(&q[2 * u], vs[i] * zd(V[int64_t(i) * ld + t.row]), wv);
    }
    chunk_to_lds(q, c, lds);
  }
  lds_to_partials(lds, nchunk, part, L.nblk, t.tile);
}

// Pass 1 in the tensor form, whose blocks are not rows of the basis: the
// product alone; k_mdot takes the dots.
// Its input is the D^-1-scaled copy that pass 3 leaves beside the vector.
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_gs_only(Seg L, SellOp<T> A, const GmSt* st, GmArr G,
                                                    const cx<T>* __restrict__ in, int j, cx<T>* __restrict__ w) {
  Tile t = prod_tile<F>(L);
  if (st[t.seg].cyc) return;
  const double s = G.vs[int64_t(t.seg) * (G.m + 1) + j];
  for_rows<F>(A, t, in, [](int64_t) { return 0; },
              [=](int64_t row, cx<T> y, int) { w[row] = ccast<T>(s * zd(y)); });
}

// in = D^-1 V_0 (tensor form)
template <typename T>
__global__ void __launch_bounds__(kBlock) k_gs_start(Seg L, TzOp Z, const cx<T>* __restrict__ V, cx<T>* __restrict__ in) {
  const Tile t = tile_of(L);
  in[t.row] = ccast<T>(tz_pre<kFormTensor>(Z, tz_seg(Z, t.seg), t.row, zd(V[t.row])));
}

// Pass 2 with R threads per row (R = 4 or 8), for j + 1 <= R Q: a block of
// 256 threads walks its 256-row tile 256 / R rows at a time; thread (row r,
// part p) holds basis vectors p Qa .. p Qa + Qa - 1 (Qa = ceil((j + 1) / R))
// of its row in registers; the R parts' sums of h1_i v_i meet by lane
// exchanges (the same value in all R lanes), giving w1; each thread
// accumulates its part's dots v_i^H w1 over its rows, and only then are
// they summed over the wave's rows of that part and over the block's waves
// in order (a fixed order), and stored in the chunk layout of k_mdot_fin.
template <typename T, int R, int Q>
__global__ void __launch_bounds__(kBlock) k_gs_second(Seg L, const GmSt* st, GmArr G, const cx<T>* __restrict__ V,
                                                      int64_t ld, int j, const cx<T>* __restrict__ w,
                                                      double* __restrict__ part) {
  constexpr int kW = kBlock / kWave;
  constexpr int kRowsPerWave = kWave / R;
  __shared__ double lds[R * Q][2][kW];
  const int tile = xcd_chunk_tile(blockIdx.x, gridDim.x);
  const int seg = L.blk_seg[tile];
  if (st[seg].cyc) return;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int p = lane / kRowsPerWave, rl = lane % kRowsPerWave;
  const int n = j + 1, qa = (n + R - 1) / R, i0 = p * qa;
  const double* vs = G.vs + int64_t(seg) * (G.m + 1);
  const z_t* h1 = G.h1 + int64_t(seg) * (G.m + 1);
  double d[Q][2];
#pragma unroll
  for (int u = 0; u < Q; ++u) d[u][0] = d[u][1] = 0.0;
#pragma unroll(Q <= 4 ? 2 : 1)
  for (int r0 = 0; r0 < kBlock; r0 += kW * kRowsPerWave) {
    const int64_t row = int64_t(tile) * kBlock + r0 + wave * kRowsPerWave + rl;
    cx<T> v[Q];
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      const int i = i0 + u;
      v[u] = (u < qa && i < n) ? V[int64_t(i) * ld + row] : cx<T>{T(0), T(0)};
    }
    z_t acc = p == 0 ? zd(w[row]) : z_t{0.0, 0.0};
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      const int i = i0 + u;
      if (u < qa && i < n) {
        const z_t h = vs[i] * h1[i], x = zd(v[u]);
        acc.re -= h.re * x.re - h.im * x.im;
        acc.im -= h.re * x.im + h.im * x.re;
      }
    }
#pragma unroll
    for (int o = kRowsPerWave; o < kWave; o <<= 1) {
      acc.re += __shfl_xor(acc.re, o, kWave);
      acc.im += __shfl_xor(acc.im, o, kWave);
    }
    const z_t w1 = zd(ccast<T>(acc));   // the storage precision's w1, as if stored
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      const int i = i0 + u;
      if (u < qa && i < n) dot_acc(d[u], vs[i] * zd(v[u]), w1);
    }
  }
#pragma unroll
  for (int u = 0; u < Q; ++u) {
#pragma unroll
    for (int o = kRowsPerWave / 2; o > 0; o >>= 1) {
      d[u][0] += __shfl_xor(d[u][0], o, kWave);
      d[u][1] += __shfl_xor(d[u][1], o, kWave);
    }
    const int i = i0 + u;
    if (rl == 0 && u < qa && i < n) {
      lds[i][0][wave] = d[u][0];
      lds[i][1][wave] = d[u][1];
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * n; e += kBlock) {
    const int i = e >> 1, ri = e & 1;
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kW; ++k) t += lds[i][ri][k];
    part[(int64_t(i / NV) * 2 * NV + 2 * (i % NV) + ri) * L.nblk + tile] = t;
  }
}

// Pass 3: w2 = w1 - sum_i h2_i v_i with w1 = w - sum_i h1_i v_i, written in
// place of w (the next stored basis vector), in the tensor form also scaled
// into in; partial ||w2||^2.
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_gs_third(Seg L, TzOp Z, const GmSt* st, GmArr G,
                                                     const cx<T>* __restrict__ V, int64_t ld, int j,
                                                     cx<T>* __restrict__ w, cx<T>* __restrict__ in, double* part) {
  SumTile t = tile_of_sums(L);
  if (st[t.seg].cyc) return;
  const double* vs = G.vs + int64_t(t.seg) * (G.m + 1);
  const z_t* h1 = G.h1 + int64_t(t.seg) * (G.m + 1);
  const z_t* h2 = G.h2 + int64_t(t.seg) * (G.m + 1);
  z_t a1 = zd(w[t.row]), a2 = {0.0, 0.0};
  for (int i = 0; i <= j; ++i) {
    const z_t v = vs[i] * zd(V[int64_t(i) * ld + t.row]);
    const z_t p = h1[i], r = h2[i];
    a1.re -= p.re * v.re - p.im * v.im;
    a1.im -= p.re * v.im + p.im * v.re;
    a2.re -= r.re * v.re - r.im * v.im;
    a2.im -= r.re * v.im + r.im * v.re;
  }
  const z_t w1 = zd(ccast<T>(a1));
  const cx<T> ws = ccast<T>(w1 + a2);
  w[t.row] = ws;
  if (F == kFormTensor) in[t.row] = ccast<T>(tz_pre<F>(Z, form_seg<F>(Z, t), t.row, zd(ws)));
  double q[1] = {norm2(zd(ws))};
  store_partials<1>(q, part, t);
}

// partial h_i = V_i^H w for i in chunk blockIdx.y (i <= j)
template <typename T>
__global__ void __launch_bounds__(kBlock) k_mdot(Seg L, const GmSt* st, GmArr G, const cx<T>* __restrict__ V,
                                                 int64_t ld, int j, const cx<T>* __restrict__ w,
                                                 double* part) {
  SumTile t = tile_of_sums(L);
  if (st[t.seg].cyc) return;
  int i0 = blockIdx.y * NV;
  z_t wv = zd(w[t.row]);
  double q[2 * NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    int i = i0 + c;
    z_t a = {0.0, 0.0};
    if (i <= j) a = G.vs[int64_t(t.seg) * (G.m + 1) + i] * zd(V[int64_t(i) * ld + t.row]);
    q[2 * c] = a.re * wv.re + a.im * wv.im;
    q[2 * c + 1] = a.re * wv.im - a.im * wv.re;
  }
  store_partials_qmajor<2 * NV>(q, part + int64_t(blockIdx.y) * L.nblk * 2 * NV, L.nblk, t);
}

// block (s, i): coefficient i of segment s.  pass 1 -> h1; pass 2 -> h2 and H[:, j] = h1 + h2.
// The real and imaginary block partials of a coefficient are two
// contiguous runs: coalesced loads, several in flight per thread, then the
// block's sum in a fixed order.
__global__ void __launch_bounds__(kFinBlock) k_mdot_fin(Seg L, const GmSt* st, GmArr G, const double* part, int j,
                                                        int pass) {
  int s = blockIdx.x, i = blockIdx.y;
  const int cyc = st[s].cyc;
  int c = i / NV, q = i % NV;
  const double* pre = part + (int64_t(c) * 2 * NV + 2 * q) * L.nblk;
  const double* pim = pre + L.nblk;
  const int b0 = L.nseg == 1 ? 0 : L.seg_blk[s], b1 = L.nseg == 1 ? L.nblk : L.seg_blk[s + 1];
  double ar = 0.0, ai = 0.0;
#pragma unroll 4
  for (int b = b0 + int(threadIdx.x); b < b1; b += kFinBlock) {
    ar += pre[b];
    ai += pim[b];
  }
  __shared__ double lds[2][kFinBlock / kWave];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  ar = wave_sum(ar);
  ai = wave_sum(ai);
  if (lane == 0) {
    lds[0][w] = ar;
    lds[1][w] = ai;
  }
  __syncthreads();
  if (cyc) return;
  if (threadIdx.x == 0) {
    double re = 0.0, im = 0.0;
    for (int k = 0; k < kFinBlock / kWave; ++k) {
      re += lds[0][k];
      im += lds[1][k];
    }
    z_t h = {re, im};
    if (pass == 1) {
      G.h1[int64_t(s) * (G.m + 1) + i] = h;
    } else {
      G.h2[int64_t(s) * (G.m + 1) + i] = h;
      z_t* H = G.H + int64_t(s) * (G.m + 1) * G.m;
      H[int64_t(j) * (G.m + 1) + i] = G.h1[int64_t(s) * (G.m + 1) + i] + h;
    }
  }
}

// w -= sum_{i<=j} h_i V_i (h = h1 or h2); optionally partial ||w||^2
template <typename T, bool NORM, int F>
__global__ void __launch_bounds__(kBlock) k_axpy(Seg L, TzOp Z, const GmSt* st, GmArr G, const cx<T>* __restrict__ V,
                                                 int64_t ld, int j, int pass, cx<T>* __restrict__ w,
                                                 cx<T>* __restrict__ in, double* part) {
  SumTile t = tile_of_sums(L);
  if (st[t.seg].cyc) return;
  const z_t* h = (pass == 1 ? G.h1 : G.h2) + int64_t(t.seg) * (G.m + 1);
  const double* vs = G.vs + int64_t(t.seg) * (G.m + 1);
  z_t acc = zd(w[t.row]);
  for (int i = 0; i <= j; ++i) {
    z_t v = vs[i] * zd(V[int64_t(i) * ld + t.row]);
    z_t hi = h[i];
    acc.re -= hi.re * v.re - hi.im * v.im;
    acc.im -= hi.re * v.im + hi.im * v.re;
  }
  cx<T> ws = ccast<T>(acc);
  w[t.row] = ws;
  if (NORM) {
    if (F == kFormTensor) in[t.row] = ccast<T>(tz_pre<F>(Z, form_seg<F>(Z, t), t.row, zd(ws)));
    double q[1] = {norm2(zd(ws))};
    store_partials<1>(q, part, t);
  }
}

// New Hessenberg column j: subdiagonal, previous rotations, new rotation,
// residual estimate |g_{j+1}|.
// The column and the previous rotations are staged in LDS by the whole
// block, so the sequential rotation loop of thread 0 reads no global memory.
struct GivensLds {
  z_t h[kGmMaxM + 1], sn[kGmMaxM];
  double cs[kGmMaxM];
};
__device__ __forceinline__ void givens_stage(const GmArr& G, int s, int j, GivensLds& W) {
  const z_t* H = G.H + int64_t(s) * (G.m + 1) * G.m + int64_t(j) * (G.m + 1);
  for (int i = threadIdx.x; i <= j; i += int(blockDim.x)) {
    W.h[i] = H[i];
    if (i < j) {
      W.cs[i] = G.cs[int64_t(s) * G.m + i];
      W.sn[i] = G.sn[int64_t(s) * G.m + i];
    }
  }
}
// by one thread, after a barrier; ww = ||w||^2 of the new vector
__device__ __forceinline__ void givens_step(GmSt& S, const GmArr& G, int s, int j, double ww, GivensLds& W) {
  const int m = G.m;
  z_t* H = G.H + int64_t(s) * (m + 1) * m + int64_t(j) * (m + 1);
  z_t* g = G.g + int64_t(s) * (m + 1);
  double hn = sqrt(ww);
  W.h[j + 1] = z_t{hn, 0.0};
  for (int i = 0; i < j; ++i) {
    z_t a = W.h[i], b = W.h[i + 1];
    W.h[i] = W.cs[i] * a + W.sn[i] * b;
    W.h[i + 1] = (-1.0 * (conj(W.sn[i]) * a)) + W.cs[i] * b;
  }
  for (int i = 0; i < j; ++i) H[i] = W.h[i];
  z_t a = W.h[j], b = W.h[j + 1];
  double rho = sqrt(norm2(a) + norm2(b));
  double c;
  z_t sv;
  if (rho == 0.0) {
    c = 1.0;
    sv = z_t{0.0, 0.0};
  } else if (norm2(a) == 0.0) {
    c = 0.0;
    sv = z_t{1.0, 0.0};
  } else {
    double aa = sqrt(norm2(a));
    c = aa / rho;
    sv = (1.0 / (aa * rho)) * (a * conj(b));
  }
  G.cs[int64_t(s) * m + j] = c;
  G.sn[int64_t(s) * m + j] = sv;
  H[j] = c * a + sv * b;
  H[j + 1] = z_t{0.0, 0.0};
  z_t gj = g[j];
  g[j + 1] = -1.0 * (conj(sv) * gj);
  g[j] = c * gj;
  S.k = j + 1;
  S.iters += 1;
  S.est = sqrt(norm2(g[j + 1]));
  bool bad = !isfinite(hn) || !isfinite(S.est);
  if (bad) S.nan = 1;
  if (bad || hn == 0.0 || S.est * S.est <= S.thr2) S.cyc = 1;
  S.inv_next = hn > 0.0 ? 1.0 / hn : 0.0;
  G.vs[int64_t(s) * (m + 1) + j + 1] = S.inv_next;
}
__global__ void __launch_bounds__(kFinBlock) k_givens_fin(Seg L, GmSt* st, GmArr G, const double* part, int j) {
  __shared__ GivensLds W;
  const int s = blockIdx.x;
  const int cyc = st[s].cyc;
  if (!cyc) givens_stage(G, s, j, W);
  double o[1];
  seg_sums<1>(L, part, s, o);   // its barriers also order the staging above
  if (cyc || threadIdx.x != 0) return;
  givens_step(st[s], G, s, j, o[0], W);
}

// y = H(0:k,0:k)^-1 g(0:k), one wave per segment: H's triangle staged in LDS
// (up to 56 columns; beyond, read as it is used), the terms H_il y_l of a row
// in parallel over l, then added in order by lane 0.  One thread forming and
// adding them took 47 us at k = 30, a chain of dependent global loads.
constexpr int kSolveStaged = 56;
struct SolveLds {
  z_t h[kSolveStaged * (kSolveStaged + 1) / 2], t[kGmMaxM], y[kGmMaxM], g[kGmMaxM];
};
__device__ __forceinline__ void solve_y(const GmSt& S, const GmArr& G, int s, SolveLds& W) {
  const int m = G.m, k = S.k, lane = threadIdx.x;
  const z_t* H = G.H + int64_t(s) * (m + 1) * m;
  const bool staged = k <= kSolveStaged;
  for (int i = lane; i < k; i += kWave) W.g[i] = G.g[int64_t(s) * (m + 1) + i];
  if (staged) {
    for (int l = 0; l < k; ++l)      // column l: rows 0..l
      if (lane <= l) W.h[l * (l + 1) / 2 + lane] = H[int64_t(l) * (m + 1) + lane];
  }
  auto at = [&](int i, int l) { return staged ? W.h[l * (l + 1) / 2 + i] : H[int64_t(l) * (m + 1) + i]; };
  __syncthreads();
  for (int i = k - 1; i >= 0; --i) {
    for (int l = i + 1 + lane; l < k; l += kWave) {
      const z_t h = at(i, l), v = W.y[l];
      W.t[l] = z_t{fma(h.re, v.re, -(h.im * v.im)), fma(h.im, v.re, h.re * v.im)};
    }
    __syncthreads();
    if (lane == 0) {
      z_t acc = W.g[i];
#pragma unroll 4
      for (int l = i + 1; l < k; ++l) acc = acc - W.t[l];
      W.y[i] = cdiv(acc, at(i, i));
    }
    __syncthreads();
  }
  for (int i = lane; i < k; i += kWave) G.y[int64_t(s) * m + i] = W.y[i];
}
__global__ void __launch_bounds__(kWave) k_solve_fin(const GmSt* st, GmArr G) {
  __shared__ SolveLds W;
  const GmSt& S = st[blockIdx.x];
  if (S.done || S.nan) return;
  solve_y(S, G, blockIdx.x, W);
}

// u += sum_{i<k} y_i V_i (D^-1 times the sum in the tensor form)
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_update(Seg L, TzOp Z, const GmSt* st, GmArr G, const cx<T>* __restrict__ V,
                                                   int64_t ld, cx<T>* __restrict__ u) {
  Tile t = tile_of(L);
  const GmSt& S = st[t.seg];
  if (S.done || S.nan || S.k == 0) return;
  const z_t* y = G.y + int64_t(t.seg) * G.m;
  const double* vs = G.vs + int64_t(t.seg) * (G.m + 1);
  const z_t u0 = zd(u[t.row]);
  z_t acc = F == kFormTensor ? z_t{0.0, 0.0} : u0;
  for (int i = 0; i < S.k; ++i) {
    z_t v = vs[i] * zd(V[int64_t(i) * ld + t.row]);
    z_t yi = y[i];
    acc.re += yi.re * v.re - yi.im * v.im;
    acc.im += yi.re * v.im + yi.im * v.re;
  }
  if (F == kFormTensor) acc = u0 + tz_pre<F>(Z, form_seg<F>(Z, t), t.row, acc);
  u[t.row] = ccast<T>(acc);
}

// ---- one small system in the tensor form (few_cycle)
// A step of the path above is seven launches there, each a few us of latency.
// Here it is four: the sums are added by the kernel that needs them, and the
// Givens step of a column runs in a block of its own beside the next column's
// product.  A block takes 64 rows with four threads each (a quarter of the
// basis per thread, 16 rows a wave), so 3,003 rows are 47 blocks whose loads
// are all in flight at once.  Measured at 21x13x11 nodes, m = 30: 33 -> 24 us of
// kernels a step; a solve of 857 steps 46 ms with the seven launches, 29 ms with
// these replayed as a graph.
constexpr int kFewRows = 64, kFewParts = kBlock / kFewRows;
//
// Every block adds every block's partials, which ends the gain at 160 blocks, with
// short cycles, whose vector work is small against it, at 96: 600 products, ms, the
// general path : this one, at 48, 96, 140, 244 and 336 blocks (3,003 to 21,450
// rows): restart 5 15.4:13.3 15.4:15.1 15.4:16.2 15.8:21.2 15.7:24.2, restart 16
// 16.9:13.1 17.0:14.9 16.9:16.3 17.0:22.0 17.2:25.8, restart 30 19.1:13.9 19.2:15.7
// 19.2:17.2 19.5:23.1 19.5:27.3, restart 56 23.0:16.5 23.2:19.0 23.4:21.8 24.7:29.6
// 24.5:36.8.
constexpr int few_blocks(int m) { return m < 16 ? 96 : 160; }
constexpr int kFewMaxM = 56;         // basis vectors per thread: 14

// Sum of nb partials, by one wave; the same value in every lane.
__device__ __forceinline__ double few_sum(const double* __restrict__ p, int nb) {
  double v = 0.0;
  for (int b = threadIdx.x & (kWave - 1); b < nb; b += kWave) v += p[b];
  return wave_sum(v);
}
// The n complex coefficients of partials [nb][2 n], by the whole block: a
// thread adds one of E sums over every (kBlock / E)-th block, with its loads
// in flight together (one sum a wave after the other took 6 us at n = 30).
template <int E>
__device__ __forceinline__ void few_coefs(const double* __restrict__ p, int n, int nb, z_t* h) {
  constexpr int kGroups = kBlock / E;
  __shared__ double lds[kGroups][E];
  const int e = threadIdx.x % E, g = threadIdx.x / E;
  double v = 0.0;
  if (e < 2 * n) {
#pragma unroll 16
    for (int b = g; b < nb; b += kGroups) v += p[int64_t(b) * 2 * n + e];
  }
  lds[g][e] = v;
  __syncthreads();
  if (int(threadIdx.x) < 2 * n) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) t += lds[k][e];
    reinterpret_cast<double*>(h)[e] = t;
  }
  __syncthreads();
}

// w = A v_j = s_j (A V_j) from the D^-1-scaled copy in; the last block adds
// the norm's partials of column j - 1 and runs its Givens step.  The product's
// blocks read neither what that step writes nor its flag: they stop one column
// later (off).
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_few_prod(Seg L, SellOp<T> A, GmSt* st, GmArr G, const cx<T>* __restrict__ in,
                                                     int j, cx<T>* __restrict__ w, const double* __restrict__ pn, int nb) {
  __shared__ GivensLds W;
  if (int(blockIdx.x) == L.nblk) {
    if (st->cyc) return;
    givens_stage(G, 0, j - 1, W);
    const double ww = few_sum(pn, nb);
    __syncthreads();
    if (threadIdx.x == 0) givens_step(*st, G, 0, j - 1, ww, W);
    return;
  }
  if (st->off) return;
  double s;
  if (j == 0) {
    s = G.vs[0];
  } else {
    const double hn = sqrt(few_sum(pn, nb));
    s = hn > 0.0 ? 1.0 / hn : 0.0;
  }
  Tile t;
  t.tile = xcd_tile(blockIdx.x, L.nblk);
  t.seg = 0;
  t.row = 0;
  for_rows<F>(A, t, in, [](int64_t) { return 0; },
              [=](int64_t row, cx<T> y, int) { w[row] = ccast<T>(s * zd(y)); });
}

// A thread's row and its share of the basis: vectors i0 .. i0 + q - 1 < n.
struct FewRow {
  int64_t row;
  int part, i0, q;
};
__device__ __forceinline__ FewRow few_row(int n) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  FewRow r;
  r.part = lane / 16;
  r.row = int64_t(blockIdx.x) * kFewRows + wave * 16 + lane % 16;
  const int qa = (n + kFewParts - 1) / kFewParts;
  r.i0 = r.part * qa;
  r.q = n - r.i0 < qa ? n - r.i0 : qa;
  return r;
}
// Partials [nb][2 n] of the dots d[u] of a block's rows with vector i0 + u.
template <int Q>
__device__ __forceinline__ void few_partials(double (&d)[Q][2], const FewRow& r, int n, double* part) {
  __shared__ double lds[2 * kFewMaxM][kBlock / kWave];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
  for (int u = 0; u < Q; ++u)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double v = d[u][c];          // over the wave's 16 rows
      v += row_rotate<8>(v);
      v += row_rotate<4>(v);
      v += row_rotate<2>(v);
      v += row_rotate<1>(v);
      if (lane % 16 == 0 && u < r.q) lds[2 * (r.i0 + u) + c][wave] = v;
    }
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * n; e += kBlock) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kBlock / kWave; ++k) t += lds[e][k];
    part[int64_t(blockIdx.x) * 2 * n + e] = t;
  }
}

// Partials of h1_i = v_i^H w, i <= j.
template <typename T, int Q>
__global__ void __launch_bounds__(kBlock) k_few_dots(GmSt* st, GmArr G, const cx<T>* __restrict__ V, int64_t ld, int j,
                                                     const cx<T>* __restrict__ w, double* __restrict__ p1) {
  if (st->cyc) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->off = 1;
    return;
  }
  const int n = j + 1;
  const FewRow r = few_row(n);
  cx<T> v[Q];
#pragma unroll
  for (int u = 0; u < Q; ++u) v[u] = u < r.q ? V[int64_t(r.i0 + u) * ld + r.row] : cx<T>{T(0), T(0)};
  const z_t x = zd(w[r.row]);
  double d[Q][2];
#pragma unroll
  for (int u = 0; u < Q; ++u) {
    d[u][0] = d[u][1] = 0.0;
    if (u < r.q) dot_acc(d[u], G.vs[r.i0 + u] * zd(v[u]), x);
  }
  few_partials<Q>(d, r, n, p1);
}

// FIRST: w1 = w - sum_i h1_i v_i in place of w and the partials of h2_i =
// v_i^H w1.  Else: w2 = w1 - sum_i h2_i v_i in place of w, its D^-1-scaled copy
// in, the partials of ||w2||^2, and H[:, j] = h1 + h2.
template <typename T, int Q, bool FIRST>
__global__ void __launch_bounds__(kBlock) k_few_axpy(TzOp Z, const GmSt* st, GmArr G, const cx<T>* __restrict__ V,
                                                     int64_t ld, int j, cx<T>* __restrict__ w, cx<T>* __restrict__ in,
                                                     const double* __restrict__ p, double* __restrict__ out, int nb) {
  __shared__ z_t h[kFewMaxM];
  __shared__ double nrm[kBlock / kWave];
  if (st->cyc) return;
  const int n = j + 1;
  const FewRow r = few_row(n);
  cx<T> v[Q];
#pragma unroll
  for (int u = 0; u < Q; ++u) v[u] = u < r.q ? V[int64_t(r.i0 + u) * ld + r.row] : cx<T>{T(0), T(0)};
  const z_t x = zd(w[r.row]);
  few_coefs<(2 * Q * kFewParts <= kWave ? kWave : 2 * kWave)>(p, n, nb, h);
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < n; i += kBlock) {
      if (FIRST) G.h1[i] = h[i];
      else G.H[int64_t(j) * (G.m + 1) + i] = G.h1[i] + h[i];
    }
  z_t acc = r.part == 0 ? x : z_t{0.0, 0.0};
#pragma unroll
  for (int u = 0; u < Q; ++u)
    if (u < r.q) {
      const z_t c = G.vs[r.i0 + u] * h[r.i0 + u], b = zd(v[u]);
      acc = acc - c * b;
    }
  // over the four parts of the row: lane distances 16 and 32
#pragma unroll
  for (int o = 16; o < kWave; o <<= 1) {
    acc.re += __shfl_xor(acc.re, o, kWave);
    acc.im += __shfl_xor(acc.im, o, kWave);
  }
  const cx<T> ws = ccast<T>(acc);
  if (r.part == 0) w[r.row] = ws;
  const z_t y = zd(ws);
  if constexpr (FIRST) {
    double d[Q][2];
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      d[u][0] = d[u][1] = 0.0;
      if (u < r.q) dot_acc(d[u], G.vs[r.i0 + u] * zd(v[u]), y);
    }
    few_partials<Q>(d, r, n, out);
  } else {
    if (r.part == 0) in[r.row] = ccast<T>(tz_pre<kFormTensor>(Z, tz_seg(Z, 0), r.row, y));
    const double q = wave_sum(r.part == 0 ? norm2(y) : 0.0);
    if ((threadIdx.x & (kWave - 1)) == 0) nrm[threadIdx.x / kWave] = q;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < kBlock / kWave; ++k) t += nrm[k];
      out[blockIdx.x] = t;
    }
  }
}

// The last column's Givens step and y, by one wave.
__global__ void __launch_bounds__(kWave) k_few_end(GmSt* st, GmArr G, int j, const double* __restrict__ pn, int nb) {
  __shared__ GivensLds W;
  __shared__ SolveLds Y;
  if (!st->cyc) {
    givens_stage(G, 0, j, W);
    const double ww = few_sum(pn, nb);
    __syncthreads();
    if (threadIdx.x == 0) {
      givens_step(*st, G, 0, j, ww, W);
      __threadfence_block();
    }
  }
  __syncthreads();
  if (st->done || st->nan) return;
  solve_y(*st, G, 0, Y);
}

template <typename T>
int few_cycle(hipStream_t s, const SellOp<T>& A, GmSt* st, const GmArr& G, cx<T>* V, int64_t ld, int mc, cx<T>* in,
              double* pt) {
  const int nb = int(ld / kFewRows);
  double *p1 = pt, *p2 = p1 + 2 * int64_t(kFewMaxM) * nb, *pn = p2 + 2 * int64_t(kFewMaxM) * nb;
  const Seg& P = A.tz.lp;
  for (int j = 0; j < mc; ++j) {
    cx<T>* w = V + int64_t(j + 1) * ld;
    const int grid = P.nblk + (j > 0);
    if (A.tz.on == 1) k_few_prod<T, kFormTensor><<<grid, kBlock, 0, s>>>(P, A, st, G, in, j, w, pn, nb);
    else k_few_prod<T, kFormTensorExt><<<grid, kBlock, 0, s>>>(P, A, st, G, in, j, w, pn, nb);
    auto rest = [&](auto Qc) {
      constexpr int Q = decltype(Qc)::value;
      k_few_dots<T, Q><<<nb, kBlock, 0, s>>>(st, G, V, ld, j, w, p1);
      k_few_axpy<T, Q, true><<<nb, kBlock, 0, s>>>(A.tz, st, G, V, ld, j, w, in, p1, p2, nb);
      k_few_axpy<T, Q, false><<<nb, kBlock, 0, s>>>(A.tz, st, G, V, ld, j, w, in, p2, pn, nb);
    };
    if (j < 4 * kFewParts) rest(std::integral_constant<int, 4>{});
    else if (j < 8 * kFewParts) rest(std::integral_constant<int, 8>{});
    else rest(std::integral_constant<int, kFewMaxM / kFewParts>{});
    HZ_HIP(hipGetLastError());
  }
  k_few_end<<<1, kWave, 0, s>>>(st, G, mc - 1, pn, nb);
  HZ_HIP(hipGetLastError());
  return HZ_OK;
}

__global__ void k_init_st(int nseg, GmSt* st, const double* fn2, double tol) {
  int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= nseg) return;
  GmSt z = {};
  z.thr2 = tol * tol * fn2[s];
  st[s] = z;
}

// pass 1 in the operator's storage form
template <typename T>
int gs_pass1(hipStream_t s, const Seg& L, const SellOp<T>& A, const GmSt* st, const GmArr& G, const cx<T>* V,
             int64_t ld, int j, cx<T>* w, const cx<T>* in, double* pt, int grid) {
  if (A.tz.on) {
    const Seg& P = A.tz.lp;
    if (A.tz.on == 1) k_gs_only<T, kFormTensor><<<P.nblk, kBlock, 0, s>>>(P, A, st, G, in, j, w);
    else k_gs_only<T, kFormTensorExt><<<P.nblk, kBlock, 0, s>>>(P, A, st, G, in, j, w);
    k_mdot<T><<<dim3(grid, ceil_div(j + 1, NV)), kBlock, 0, s>>>(L, st, G, V, ld, j, w, pt);
  } else if (A.val) {
    k_gs_prod<T, kFormComplex><<<grid, kBlock, 0, s>>>(L, A, st, G, V, ld, j, w, pt);
  } else if (A.st) {
    k_gs_prod<T, kFormStencil><<<grid, kBlock, 0, s>>>(L, A, st, G, V, ld, j, w, pt);
  } else {
    k_gs_prod<T, kFormSplit><<<grid, kBlock, 0, s>>>(L, A, st, G, V, ld, j, w, pt);
  }
  HZ_HIP(hipGetLastError());
  return HZ_OK;
}

}  // namespace

template <typename T>
int gmres_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
              const KrylovCtl& ctl, KrylovOut* out, const std::string& tag) {
  int rc = 0;
  const int m = ctl.restart;
  if (m < 1 || m > kGmMaxM) return hz_fail(HZ_ERR_INVALID, "GMRES restart %d not in 1..%d", m, kGmMaxM);
  const int64_t ld = S.nrows;
  const std::string p = "gm." + tag + (sizeof(T) == 8 ? ".z." : ".c.");
  DevBuf* Vb = ctx->buf(p + "V", sizeof(cx<T>) * ld * (m + 1), &rc);
  if (rc) return rc;
  const int nchunk = ceil_div(m + 1, NV);
  // One small system in the tensor form takes its own kernels: up to few_blocks
  // blocks of 64 rows, beyond which adding the partials in every block costs more than
  // the launches it saves, and 56 basis vectors (14 a thread, in registers).
  const bool few = A.tz.on && S.nseg == 1 && m <= kFewMaxM && ld <= int64_t(few_blocks(m)) * kFewRows;
  int64_t np = std::max(int64_t(nchunk) * S.nblk * 2 * NV, int64_t(prod_seg(A, S.dev).nblk));
  if (few) np = std::max(np, (4 * kFewMaxM + 1) * (ld / kFewRows));
  DevBuf* part = ctx->buf(p + "part", sizeof(double) * np, &rc);
  if (rc) return rc;
  DevBuf* stb = ctx->buf(p + "st", sizeof(GmSt) * S.nseg, &rc);
  if (rc) return rc;
  const int64_t ns = S.nseg;
  DevBuf* small = ctx->buf(p + "small",
                           sizeof(z_t) * ns * ((m + 1) * m + m + (m + 1) + m + 2 * (m + 1)) +
                               sizeof(double) * ns * (m + (m + 1)), &rc);
  if (rc) return rc;
  DevBuf* fnb = ctx->buf(p + "fn2", sizeof(double) * S.nseg, &rc);
  if (rc) return rc;
  GmArr G;
  G.m = m;
  z_t* zp = small->as<z_t>();
  G.H = zp; zp += ns * (m + 1) * m;
  G.sn = zp; zp += ns * m;
  G.g = zp; zp += ns * (m + 1);
  G.y = zp; zp += ns * m;
  G.h1 = zp; zp += ns * (m + 1);
  G.h2 = zp; zp += ns * (m + 1);
  G.cs = reinterpret_cast<double*>(zp);
  G.vs = G.cs + ns * m;
  cx<T>* in = nullptr;             // tensor form: D^-1 times the next product's vector
  if (A.tz.on) {
    DevBuf* ib = ctx->buf(p + "in", sizeof(cx<T>) * ld, &rc);
    if (rc) return rc;
    in = ib->as<cx<T>>();
  }
  GmSt* st = stb->as<GmSt>();
  cx<T>* V = Vb->as<cx<T>>();
  double* pt = part->as<double>();
  hipStream_t s = ctx->stream;
  const Seg& L = S.dev;
  const Seg& P = prod_seg(A, L);   // the residual product's layout

  std::vector<double> fn2;
  HZ_TRY(seg_norm2_t<T>(ctx, S, f, &fn2));
  out->fnorm.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) out->fnorm[i] = std::sqrt(fn2[i]);
  HZ_HIP(hipMemcpyAsync(fnb->p, fn2.data(), sizeof(double) * S.nseg, hipMemcpyHostToDevice, s));
  k_init_st<<<ceil_div(S.nseg, kBlock), kBlock, 0, s>>>(S.nseg, st, fnb->as<double>(), ctl.tol);
  HZ_HIP(hipGetLastError());

  void* hp = nullptr;
  HZ_TRY(ctx_pinned(ctx, sizeof(GmSt) * S.nseg, &hp));
  GmSt* hst = static_cast<GmSt*>(hp);
  std::vector<int64_t> mv(S.nseg, 0), chk_mv(S.nseg, 0);
  std::vector<double> chk(S.nseg, -1.0);   // residual norm at the last stall checkpoint
  std::vector<int> stalled(S.nseg, 0), met(S.nseg, 0), missed(S.nseg, 0);
  constexpr int kMissed = 4;
  int64_t mv_max = 0;
  const int grid = S.nblk;
  // one restart cycle of mc steps (0: the residual alone)
  auto enqueue_cycle = [&](int mc) -> int {
    // residual of the current iterate; converged segments stop here
    HZ_BY_FORM(A, k_resid<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, f, u, V, pt));
    k_beta_fin<<<S.nseg, kFinBlock, 0, s>>>(P, st, G, pt);
    if (A.tz.on) k_gs_start<T><<<grid, kBlock, 0, s>>>(L, A.tz, V, in);
    HZ_HIP(hipGetLastError());
    if (mc >= 1) {
      if (few) HZ_TRY(few_cycle<T>(s, A, st, G, V, ld, mc, in, pt));
      for (int j = 0; j < mc && !few; ++j) {
        cx<T>* w = V + int64_t(j + 1) * ld;
        dim3 gd(grid, ceil_div(j + 1, NV));
        dim3 gf(S.nseg, j + 1);
        HZ_TRY(gs_pass1<T>(s, L, A, st, G, V, ld, j, w, in, pt, grid));
        k_mdot_fin<<<gf, kFinBlock, 0, s>>>(L, st, G, pt, j, 1);
        if (j + 1 <= 16) k_gs_second<T, 4, 4><<<grid, kBlock, 0, s>>>(L, st, G, V, ld, j, w, pt);
        else if (j + 1 <= 32) k_gs_second<T, 8, 4><<<grid, kBlock, 0, s>>>(L, st, G, V, ld, j, w, pt);
        else if (j + 1 <= 56) k_gs_second<T, 8, 7><<<grid, kBlock, 0, s>>>(L, st, G, V, ld, j, w, pt);
        else {
          // beyond 56 basis vectors: w1 stored, then a multi-dot pass
          k_axpy<T, false, kFormComplex><<<grid, kBlock, 0, s>>>(L, A.tz, st, G, V, ld, j, 1, w, in, pt);
          k_mdot<T><<<gd, kBlock, 0, s>>>(L, st, G, V, ld, j, w, pt);
        }
        k_mdot_fin<<<gf, kFinBlock, 0, s>>>(L, st, G, pt, j, 2);
        if (j + 1 <= 56) {
          HZ_BY_SCALING(A, k_gs_third<T, F><<<grid, kBlock, 0, s>>>(L, A.tz, st, G, V, ld, j, w, in, pt));
        } else {
          HZ_BY_SCALING(A, k_axpy<T, true, F><<<grid, kBlock, 0, s>>>(L, A.tz, st, G, V, ld, j, 2, w, in, pt));
        }
        k_givens_fin<<<S.nseg, kFinBlock, 0, s>>>(L, st, G, pt, j);
        HZ_HIP(hipGetLastError());
      }
      if (!few) k_solve_fin<<<S.nseg, kWave, 0, s>>>(st, G);
      HZ_BY_SCALING(A, k_update<T, F><<<grid, kBlock, 0, s>>>(L, A.tz, st, G, V, ld, u));
      HZ_HIP(hipGetLastError());
    }
    return HZ_OK;
  };
  auto run_cycle = [&](hipStream_t on) -> int {
    s = on;
    const int crc = enqueue_cycle(m);
    s = ctx->stream;
    return crc;
  };
  ReplayKey key;
  key.op(A).add(f).add(u).add(L).add(P).add(st).add(G.H).add(G.cs).add(G.sn).add(G.g).add(G.y).add(G.h1).add(G.h2).add(G.vs).add(G.m).add(V).add(ld).add(in).add(pt).add(S.nseg);
  for (;;) {
    const int mc = int(std::min<int64_t>(m, ctl.max_matvec - mv_max - 1));
    bool ran = false;
    if (mc == m && ld <= kReplayRowsGmres) HZ_TRY(replay(ctx, p, key, run_cycle, &ran, kReplayAfterGmres));
    if (!ran) HZ_TRY(enqueue_cycle(mc));
    HZ_HIP(hipMemcpyAsync(hst, st, sizeof(GmSt) * S.nseg, hipMemcpyDeviceToHost, s));
    HZ_HIP(hipStreamSynchronize(s));
    bool all_done = true, all_ended = true;   // ended: done, or stalled
    for (int i = 0; i < S.nseg; ++i) {
      mv[i] += 1;
      if (!hst[i].done) mv[i] += hst[i].k;
      mv_max = std::max(mv_max, mv[i]);
      all_done = all_done && (hst[i].done || hst[i].nan);
      if (ctl.stall_halfsteps > 0) {
        // beta: the residual this cycle began with; a residual at its rounding level shows as
        // cycles whose estimate meets the target and whose residual then does not
        missed[i] += met[i];
        if (chk[i] < 0.0) chk[i] = hst[i].beta;
        if (mv[i] - chk_mv[i] >= ctl.stall_halfsteps || missed[i] >= kMissed) {
          stalled[i] = hst[i].beta > 0.5 * chk[i];
          chk[i] = hst[i].beta;
          chk_mv[i] = mv[i];
          missed[i] = 0;
        }
        met[i] = hst[i].est * hst[i].est <= hst[i].thr2;
      }
      all_ended = all_ended && (hst[i].done || hst[i].nan || stalled[i]);
    }
    if (all_done || all_ended || mc < 1 || mv_max >= ctl.max_matvec) break;
  }
  out->iters.resize(S.nseg);
  out->matvecs.resize(S.nseg);
  out->status.resize(S.nseg);
  out->relres_est.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) {
    out->iters[i] = hst[i].iters;
    out->matvecs[i] = int(mv[i]);
    double fnv = out->fnorm[i];
    out->relres_est[i] = fnv > 0 ? hst[i].est / fnv : 0.0;
    out->status[i] = hst[i].nan ? HZ_BREAKDOWN : (hst[i].done ? HZ_OK : HZ_NOT_CONVERGED);
  }
  return HZ_OK;
}

template int gmres_run<double>(hz_ctx, const SegHost&, const SellOp<double>&, const z_t*, z_t*,
                               const KrylovCtl&, KrylovOut*, const std::string&);
template int gmres_run<float>(hz_ctx, const SegHost&, const SellOp<float>&, const c_t*, c_t*,
                              const KrylovCtl&, KrylovOut*, const std::string&);
