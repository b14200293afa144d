// BiCGStab(l) of Sleijpen and Fokkema (ETNA 1, 1993), the family of the
// paper's P-BiCGSTAB(8) (Sec. 4, solver comparison table), on the
// right-Jacobi operator B = A D^-1, for every segment of a segmented system.
//
// A cycle is l bi-conjugate gradient steps followed by one minimal-residual
// step.  Step j extends the chains u_0..u_{j+1} and r_0..r_{j+1} with
// u_{j+1} = B u_j and r_{j+1} = B r_j; the minimal-residual step picks gamma
// minimising ||r_0 - sum_j gamma_j r_j|| and updates
//     x += sum_j gamma_j r_{j-1},  r_0 -= sum_j gamma_j r_j,  u_0 -= sum_j gamma_j u_j.
// The least-squares problem is solved through the Gram matrix G = R^H R of
// r_1..r_l and c = R^H r_0, all of them formed in one fused pass over the
// l + 1 vectors, followed by a Cholesky solve on the device (the original
// paper orthogonalises r_1..r_l by modified Gram-Schmidt, which costs l
// passes; both give the same gamma in exact arithmetic).  Should G lose
// positive definiteness in the working precision, the solve keeps the
// leading well-conditioned directions and the segment restarts from its
// true residual after the cycle.
//
// Per cycle: 4 l + 3 launches, 2 l products, and a launch for the report once a
// chunk.  The scalar steps run at the start of the kernel that needs them
// (advance) or, on large systems, 2 l in kernels of their own (k_step), on a state
// that moves through three slots.  Krylov scalars stay on the device; the host
// reads the per-segment state after each chunk of cycles (Pace).
//
// In the tensor form the products take D^-1-scaled inputs: the kernels that
// make u_j and r_j also write the scaled copy that their product reads, and x
// is the solution: the corrections, which are sums of unscaled vectors,
// collect in e and enter x as D^-1 e at a restart and at the end.
#include <chrono>

#include "ops.h"

namespace {

constexpr int kMaxL = 8;

enum { kBlNone = 0, kBlAlpha, kBlBeta, kBlCycle };
struct BlSt {
  z_t rho0, alpha, omega, beta;
  z_t gam[kMaxL + 1];   // gamma_1..gamma_l
  double rr, thr2, rhat2;
  int iter, done, brk, nan, restart, trunc;
  int due, pad;         // due: the step that the sums formed next (or last) are for
};

template <typename T>
struct BlV {
  const cx<T>* f;
  cx<T>* x;                 // iterate
  cx<T>* e;                 // where its corrections go: x itself, or e (tensor form)
  cx<T>* in;                // tensor form: D^-1 times the next product's vector
  cx<T>* rt;                // shadow residual
  cx<T>* r[kMaxL + 1];
  cx<T>* u[kMaxL + 1];
};

template <typename T> __device__ __forceinline__ z_t zd(cx<T> a) { return ccast<double>(a); }
template <typename T> __device__ __forceinline__ cx<T> zt(z_t a) { return ccast<T>(a); }

__device__ __forceinline__ bool bl_off(const BlSt& S) { return S.done || S.brk || S.nan; }

// a^H b accumulated into q[0], q[1]
__device__ __forceinline__ void acc_dot(double* q, z_t a, z_t b) {
  q[0] = fma(a.re, b.re, fma(a.im, b.im, q[0]));
  q[1] = fma(a.re, b.im, fma(-a.im, b.re, q[1]));
}

// ---------------------------------------------------------------- scalar steps
// Run by one thread once a segment's sums are complete.
__device__ __forceinline__ void bl_resid(BlSt& S, const double* tot) {
  const double rr = tot[0];
  S.rr = rr;
  S.rhat2 = rr;
  S.rho0 = z_t{rr, 0.0};     // first step: beta = 0, rho0 = rt^H r_0
  S.alpha = S.beta = z_t{0.0, 0.0};
  S.omega = z_t{1.0, 0.0};
  S.nan = !isfinite(rr);
  S.done = (rr <= S.thr2) || S.nan;
  S.brk = 0;
  S.trunc = 0;
  S.restart = 0;
  S.due = kBlAlpha;
}
// alpha = rho0 / rt^H u_{j+1}
__device__ __forceinline__ void bl_alpha(BlSt& S, const double* tot) {
  S.due = kBlBeta;
  const z_t sg = {tot[0], tot[1]};
  if (norm2(sg) == 0.0 || !isfinite(sg.re) || !isfinite(sg.im)) S.brk = 1;
  else S.alpha = cdiv(S.rho0, sg);
}
// rho1 = rt^H r_{j+1}; beta = alpha rho1 / rho0; rho0 = rho1
__device__ __forceinline__ void bl_beta(BlSt& S, const double* tot) {
  S.due = kBlAlpha;
  const z_t rho1 = {tot[0], tot[1]};
  if (norm2(S.rho0) == 0.0 || !isfinite(rho1.re) || !isfinite(rho1.im)) {
    S.brk = 1;
  } else {
    S.beta = S.alpha * cdiv(rho1, S.rho0);
    S.rho0 = rho1;
  }
}
// gamma of the minimal-residual step
template <int LL>
__device__ __forceinline__ void bl_mr(BlSt& S, const double* tot, double piv) {
  z_t g[LL];
  const int m = gram_solve<LL>(tot, piv, g);
  if (m == 0) S.brk = 1;
  bool bad = false;
#pragma unroll
  for (int i = 0; i < LL; ++i) bad = bad || !isfinite(g[i].re) || !isfinite(g[i].im);
  if (bad) {
    S.brk = 1;
    return;
  }
#pragma unroll
  for (int i = 0; i < LL; ++i) S.gam[i + 1] = g[i];
  S.omega = g[LL - 1];
  S.trunc = (m < LL) ? 1 : 0;
  S.due = S.brk ? kBlNone : kBlCycle;   // k_bl_update forms the sums of the cycle's end
}
__device__ __forceinline__ void bl_cycle(BlSt& S, const double* tot) {
  S.due = kBlAlpha;
  const z_t rho1 = {tot[0], tot[1]};
  const double rr = tot[2];
  S.iter += 1;
  S.rr = rr;
  if (!isfinite(rr) || !isfinite(rho1.re) || !isfinite(rho1.im)) {
    S.nan = 1;
    S.done = 1;
    return;
  }
  if (rr <= S.thr2) {
    S.done = 1;
    return;
  }
  const z_t rho0 = -1.0 * (S.omega * S.rho0);
  if (S.trunc || norm2(rho0) == 0.0 || sqrt(norm2(rho1)) < 1e-300 * sqrt(S.rhat2 * rr)) {
    S.brk = 1;                 // restart from the true residual
    return;
  }
  S.beta = S.alpha * cdiv(rho1, rho0);
  S.rho0 = rho1;
}

struct BlResid {
  __device__ bool on(const BlSt& S) const { return S.restart != 0; }
  __device__ void operator()(BlSt& S, const double* o) const { bl_resid(S, o); }
};
struct BlAlpha {
  __device__ bool on(const BlSt& S) const { return !bl_off(S) && S.due == kBlAlpha; }
  __device__ void operator()(BlSt& S, const double* o) const { bl_alpha(S, o); }
};
struct BlBeta {
  __device__ bool on(const BlSt& S) const { return !bl_off(S) && S.due == kBlBeta; }
  __device__ void operator()(BlSt& S, const double* o) const { bl_beta(S, o); }
};
template <int LL>
struct BlMr {
  double piv;
  __device__ bool on(const BlSt& S) const { return !bl_off(S); }
  __device__ void operator()(BlSt& S, const double* o) const { bl_mr<LL>(S, o, piv); }
};
struct BlCycle {
  __device__ bool on(const BlSt& S) const { return S.due == kBlCycle; }
  __device__ void operator()(BlSt& S, const double* o) const { bl_cycle(S, o); }
};

// ---------------------------------------------------------------- restart
// x += D^-1 e, e = 0 (tensor form): the segments that restart, or all.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_bl_fold(Seg L, TzOp Z, const BlSt* st, BlV<T> V, int all) {
  const Tile t = vec_tile(L);
  if (!all && !st[t.seg].restart) return;
  const TzSeg B = tz_seg(Z, t.seg);
  vec_rows(L, t, [&](int64_t row) {
    V.x[row] = zt<T>(zd(V.x[row]) + tz_pre<kFormTensor>(Z, B, row, zd(V.e[row])));
    V.e[row] = cx<T>{T(0), T(0)};
  });
}

// r_0 = f - B x, rt = r_0, u_0 = 0; partial ||r_0||^2.
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_bl_resid(Seg L, SellOp<T> A, const BlSt* st, BlV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  if (!st[t.seg].restart) return;
  double q[1] = {0.0};
  for_rows<F, true>(A, t, V.x, [=](int64_t row) { return V.f[row]; },
              [&](int64_t row, cx<T> y, cx<T> f) {
                const cx<T> rs = zt<T>(zd(f) - zd(y));
                V.r[0][row] = rs;
                V.rt[row] = rs;
                V.u[0][row] = cx<T>{T(0), T(0)};
                q[0] += norm2(zd(rs));
              });
  store_partials<1>(q, part, t);
}

// ---------------------------------------------------------------- bi-conjugate gradient step j
// Steps 0..3 are unrolled (J = j + 1): all vectors of a row are loaded before the
// first is stored.  A store between two loads, which may alias, costs a load
// latency each (4.8 us a kernel on average at 41x25x21, 4.4 us unrolled).  Later
// steps (J = 0) load as they go.
#define HZ_BY_STEP(j, ...)                                   \
  do {                                                       \
    if ((j) == 0) { constexpr int J = 1; __VA_ARGS__; }      \
    else if ((j) == 1) { constexpr int J = 2; __VA_ARGS__; } \
    else if ((j) == 2) { constexpr int J = 3; __VA_ARGS__; } \
    else if ((j) == 3) { constexpr int J = 4; __VA_ARGS__; } \
    else { constexpr int J = 0; __VA_ARGS__; }               \
  } while (0)

// beta (at j = 0 of the cycle before); u_i = r_i - beta u_i, i = 0..j
template <typename T, int F, int J>
__global__ void __launch_bounds__(kBlock) k_bl_u(Seg L, TzOp Z, Part P, Part Pc, const BlSt* in, BlSt* out, BlV<T> V,
                                                 int j) {
  const Tile t = vec_tile(L);
  const BlSt& S = j == 0 ? advance<3, (F < kFormTensor)>(Pc, in, out, t, first_block(L, t), BlCycle{})
                         : advance<2, (F < kFormTensor)>(P, in, out, t, first_block(L, t), BlBeta{});
  if (bl_off(S)) return;
  const TzSeg B = form_seg<F>(Z, t);
  const z_t b = S.beta;
  vec_rows(L, t, [&](int64_t row) {
    cx<T> u = {};
    if constexpr (J > 0) {
      cx<T> ri[J], ui[J];
#pragma unroll
      for (int i = 0; i < J; ++i) {
        ri[i] = V.r[i][row];
        ui[i] = V.u[i][row];
      }
#pragma unroll
      for (int i = 0; i < J; ++i) V.u[i][row] = u = zt<T>(zd(ri[i]) - b * zd(ui[i]));
    } else {
      for (int i = 0; i <= j; ++i) V.u[i][row] = u = zt<T>(zd(V.r[i][row]) - b * zd(V.u[i][row]));
    }
    if (F == kFormTensor) V.in[row] = zt<T>(tz_pre<F>(Z, B, row, zd(u)));
  });
}

// y_{j+1} = B y_j for the chain y (u or r), from yj = y_j (scaled in the
// tensor form); partial rt^H y_{j+1} (SUMS).
template <typename T, int F, bool SUMS>
__global__ void HZ_PRODUCT_BOUNDS k_bl_prod(Seg L, SellOp<T> A, const BlSt* st, const cx<T>* __restrict__ yj,
                                            cx<T>* __restrict__ yj1, const cx<T>* __restrict__ rt, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  if (bl_off(st[t.seg])) return;
  if constexpr (!SUMS) {
    for_rows<F>(A, t, yj, [](int64_t) { return 0; }, [=](int64_t row, cx<T> y, int) { yj1[row] = y; });
  } else {
    double q[2] = {0.0, 0.0};
    for_rows<F>(A, t, yj, [=](int64_t row) { return rt[row]; },
                [&](int64_t row, cx<T> y, cx<T> r) {
                  yj1[row] = y;
                  acc_dot(q, zd(r), zd(y));
                });
    store_partials<2>(q, part, t);
  }
}

// alpha; r_i -= alpha u_{i+1}, i = 0..j; x += alpha u_0
template <typename T, int F, int J>
__global__ void __launch_bounds__(kBlock) k_bl_r(Seg L, TzOp Z, Part P, const BlSt* in, BlSt* out, BlV<T> V, int j) {
  const Tile t = vec_tile(L);
  const BlSt& S = advance<2, (F < kFormTensor)>(P, in, out, t, first_block(L, t), BlAlpha{});
  if (bl_off(S)) return;
  const TzSeg B = form_seg<F>(Z, t);
  const z_t a = S.alpha;
  vec_rows(L, t, [&](int64_t row) {
    cx<T> r = {};
    if constexpr (J > 0) {
      cx<T> ri[J], ui[J];
#pragma unroll
      for (int i = 0; i < J; ++i) {
        ri[i] = V.r[i][row];
        ui[i] = V.u[i + 1][row];
      }
      const cx<T> e = V.e[row], u0 = V.u[0][row];
#pragma unroll
      for (int i = 0; i < J; ++i) V.r[i][row] = r = zt<T>(zd(ri[i]) - a * zd(ui[i]));
      V.e[row] = zt<T>(zd(e) + a * zd(u0));
    } else {
      for (int i = 0; i <= j; ++i) V.r[i][row] = r = zt<T>(zd(V.r[i][row]) - a * zd(V.u[i + 1][row]));
      V.e[row] = zt<T>(zd(V.e[row]) + a * zd(V.u[0][row]));
    }
    if (F == kFormTensor) V.in[row] = zt<T>(tz_pre<F>(Z, B, row, zd(r)));
  });
}

// ---------------------------------------------------------------- minimal-residual step
// Partials of c_i = r_i^H r_0 (i = 1..LL) and G_ij = r_i^H r_j (1 <= i <= j <= LL).
template <int LL> constexpr int gram_nq() { return 2 * (LL + LL * (LL + 1) / 2); }

template <typename T, int LL>
__global__ void __launch_bounds__(kBlock) k_bl_gram(Seg L, const BlSt* st, BlV<T> V, double* part) {
  const SumTile t = vec_tile_sums(L);
  if (bl_off(st[t.seg])) return;
  constexpr int NQ = gram_nq<LL>();
  double q[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) q[i] = 0.0;
  vec_rows(L, t, [&](int64_t row) {
    z_t r[LL + 1];
#pragma unroll
    for (int i = 0; i <= LL; ++i) r[i] = zd(V.r[i][row]);
    int k = 0;
#pragma unroll
    for (int i = 1; i <= LL; ++i) {
      acc_dot(q + k, r[i], r[0]);
      k += 2;
    }
#pragma unroll
    for (int i = 1; i <= LL; ++i) {
#pragma unroll
      for (int jj = i; jj <= LL; ++jj) {
        acc_dot(q + k, r[i], r[jj]);
        k += 2;
      }
    }
  });
  store_partials<NQ>(q, part, t);
}

// gamma by one block per segment: its 2 LL + LL (LL + 1) sums are too many to
// add in every block, and its registers would limit k_bl_update.
template <int LL>
__global__ void __launch_bounds__(kBlock) k_bl_mr(Part P, const BlSt* in, BlSt* out, double piv) {
  Tile t;
  t.tile = t.seg = blockIdx.x;
  t.row = 0;
  advance<gram_nq<LL>(), false>(P, in, out, t, true, BlMr<LL>{piv});
}

// x += sum gamma_j r_{j-1}; r_0 -= sum gamma_j r_j; u_0 -= sum gamma_j u_j;
// partials rt^H r_0, ||r_0||^2
template <typename T, int LL>
__global__ void __launch_bounds__(kBlock) k_bl_update(Seg L, const BlSt* st, BlV<T> V, double* part) {
  const SumTile t = vec_tile_sums(L);
  const BlSt& S = st[t.seg];
  if (bl_off(S)) return;
  double q[3] = {0.0, 0.0, 0.0};
  vec_rows(L, t, [&](int64_t row) {
    z_t x = zd(V.e[row]), r0 = zd(V.r[0][row]), u0 = zd(V.u[0][row]);
    z_t rprev = r0;
#pragma unroll
    for (int jj = 1; jj <= LL; ++jj) {
      const z_t g = S.gam[jj];
      const z_t rj = zd(V.r[jj][row]);
      x = x + g * rprev;
      r0 = r0 - g * rj;
      u0 = u0 - g * zd(V.u[jj][row]);
      rprev = rj;
    }
    cx<T> rs = zt<T>(r0);
    V.e[row] = zt<T>(x);
    V.r[0][row] = rs;
    V.u[0][row] = zt<T>(u0);
    const z_t rv = zd(rs);
    acc_dot(q, zd(V.rt[row]), rv);
    q[2] += norm2(rv);
  });
  store_partials<3>(q, part, t);
}

__global__ void k_bl_set_thr(int nseg, BlSt* st, const double* fn2, double tol) {
  int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= nseg) return;
  st[s].thr2 = tol * tol * fn2[s];
  st[s].iter = 0;
  st[s].restart = 1;
}

template <typename T, int LL>
int enqueue_mr(hipStream_t q, const Seg& W, const BlSt* in, BlSt* out, BlSt* next, const BlV<T>& V, const PartBuf& pg,
               const PartBuf& pc) {
  k_bl_gram<T, LL><<<W.nblk, kBlock, 0, q>>>(W, in, V, pg.raw);
  k_bl_mr<LL><<<W.nseg, kBlock, 0, q>>>(pg.part, in, out, 1e-13);
  k_bl_update<T, LL><<<W.nblk, kBlock, 0, q>>>(W, out, V, pc.raw);
  HZ_HIP(hipGetLastError());
  return pc.step<3>(q, out, next, BlCycle{});
}

}  // namespace

template <typename T>
int bicgstabl_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* x,
                  const KrylovCtl& ctl, KrylovOut* out, const std::string& tag) {
  const int l = ctl.ell;
  if (l < 1 || l > kMaxL) return hz_fail(HZ_ERR_INVALID, "BiCGStab(l): l = %d not in 1..%d", l, kMaxL);
  int rc = 0;
  const int64_t nr = S.nrows;
  const size_t vb = sizeof(cx<T>) * nr;
  const std::string p = "bicgl." + tag + (sizeof(T) == 8 ? ".z." : ".c.");
  BlV<T> V = {};
  V.f = f;
  V.x = x;
  auto vec = [&](const std::string& nm) -> cx<T>* {
    DevBuf* b = ctx->buf(p + nm, vb, &rc);
    return rc ? nullptr : b->as<cx<T>>();
  };
  V.rt = vec("rt");
  for (int i = 0; i <= l; ++i) {
    V.r[i] = vec("r" + std::to_string(i));
    V.u[i] = vec("u" + std::to_string(i));
  }
  V.e = A.tz.on ? vec("e") : x;
  V.in = A.tz.on ? vec("in") : nullptr;
  if (rc) return rc;
  // state slots: start of a cycle, after beta, after alpha; one nobody reads
  DevBuf* stb = ctx->buf(p + "st", sizeof(BlSt) * 4 * S.nseg, &rc);
  if (rc) return rc;
  DevBuf* fnb = ctx->buf(p + "fn2", sizeof(double) * S.nseg, &rc);
  if (rc) return rc;
  BlSt *st = stb->as<BlSt>(), *st_b = st + S.nseg, *st_a = st_b + S.nseg, *st_u = st_a + S.nseg;   // st: what a cycle starts from
  hipStream_t s = ctx->stream;
  const Seg& L = S.dev;
  const Seg& P = prod_seg(A, L);   // the products' layout

  std::vector<double> fn2;
  HZ_TRY(seg_norm2_t<T>(ctx, S, f, &fn2));
  out->fnorm.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) out->fnorm[i] = std::sqrt(fn2[i]);
  HZ_HIP(hipMemcpyAsync(fnb->p, fn2.data(), sizeof(double) * S.nseg, hipMemcpyHostToDevice, s));
  HZ_HIP(hipMemsetAsync(stb->p, 0, sizeof(BlSt) * 4 * S.nseg, s));
  k_bl_set_thr<<<ceil_div(S.nseg, kBlock), kBlock, 0, s>>>(S.nseg, st, fnb->as<double>(), ctl.tol);
  HZ_HIP(hipGetLastError());

  StatePoll poll;
  HZ_TRY(poll.init(ctx, sizeof(BlSt) * S.nseg));
  const Seg& W = A.tz.on ? S.vec_runs : S.vec;   // vector layout
  PartBuf pr, pa, pb, pg, pc;        // sums of the residual, alpha, beta, minimal-residual and cycle steps
  HZ_TRY(pr.init(ctx, S, P, 1, W.nblk, p + "part.r"));
  HZ_TRY(pa.init(ctx, S, P, 2, W.nblk, p + "part.a"));
  HZ_TRY(pb.init(ctx, S, P, 2, W.nblk, p + "part.b"));
  HZ_TRY(pg.init(ctx, S, W, 2 * l + l * (l + 1), 0, p + "part.g"));   // (k_bl_mr adds them)
  HZ_TRY(pc.init(ctx, S, W, 3, W.nblk, p + "part.c"));
  int64_t resid_calls = 0;
  if (A.tz.on) HZ_HIP(hipMemsetAsync(V.e, 0, vb, s));

  auto report = [&]() -> int {
    HZ_TRY(pc.step_now<3>(s, st, poll.slot<BlSt>(), BlCycle{}));
    return poll.posted_one();
  };
  auto enqueue_resid = [&](int all) -> int {
    if (resid_calls > 0) HZ_TRY(pc.step_now<3>(s, st, st, Settle<BlCycle>{{}, all}));
    if (A.tz.on && resid_calls > 0) k_bl_fold<T><<<W.nblk, kBlock, 0, s>>>(W, A.tz, st, V, 0);
    HZ_BY_FORM(A, k_bl_resid<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, st, V, pr.raw));
    HZ_HIP(hipGetLastError());
    // (no step is due: st_b is what the next cycle's first step would make of st)
    HZ_TRY(pr.step_now<1>(s, st, st, BlResid{}, poll.slot<BlSt>(), st_b));
    ++resid_calls;
    HZ_TRY(poll.posted_one());
    return poll.wait(poll.posted - 1);
  };
  auto enqueue_cycle = [&]() -> int {
    for (int j = 0; j < l; ++j) {
      const BlSt* in = j == 0 ? st : st_a;
      const PartBuf& pu = j == 0 ? pc : pb;   // whose sums k_bl_u's step takes
      HZ_BY_STEP(j, HZ_BY_SCALING(A, k_bl_u<T, F, J><<<W.nblk, kBlock, 0, s>>>(W, A.tz, pb.part, pc.part, pu.from(in, st_b), pu.to(st_b, st_u), V, j)));
      const cx<T>* uj = A.tz.on ? V.in : V.u[j];
      HZ_BY_FORM(A, k_bl_prod<T, F, true><<<P.nblk, kBlock, 0, s>>>(P, A, st_b, uj, V.u[j + 1], V.rt, pa.raw));
      HZ_TRY(pa.step<2>(s, st_b, st_a, BlAlpha{}));
      HZ_BY_STEP(j, HZ_BY_SCALING(A, k_bl_r<T, F, J><<<W.nblk, kBlock, 0, s>>>(W, A.tz, pa.part, pa.from(st_b, st_a), pa.to(st_a, st_u), V, j)));
      const cx<T>* rj = A.tz.on ? V.in : V.r[j];
      if (j + 1 < l) {
        HZ_BY_FORM(A, k_bl_prod<T, F, true><<<P.nblk, kBlock, 0, s>>>(P, A, st_a, rj, V.r[j + 1], V.rt, pb.raw));
        HZ_TRY(pb.step<2>(s, st_a, st_b, BlBeta{}));
      } else {
        HZ_BY_FORM(A, k_bl_prod<T, F, false><<<P.nblk, kBlock, 0, s>>>(P, A, st_a, rj, V.r[j + 1], V.rt, nullptr));
      }
    }
    switch (l) {
      case 1: return enqueue_mr<T, 1>(s, W, st_a, st, st_b, V, pg, pc);
      case 2: return enqueue_mr<T, 2>(s, W, st_a, st, st_b, V, pg, pc);
      case 3: return enqueue_mr<T, 3>(s, W, st_a, st, st_b, V, pg, pc);
      case 4: return enqueue_mr<T, 4>(s, W, st_a, st, st_b, V, pg, pc);
      case 5: return enqueue_mr<T, 5>(s, W, st_a, st, st_b, V, pg, pc);
      case 6: return enqueue_mr<T, 6>(s, W, st_a, st, st_b, V, pg, pc);
      case 7: return enqueue_mr<T, 7>(s, W, st_a, st, st_b, V, pg, pc);
      default: return enqueue_mr<T, 8>(s, W, st_a, st, st_b, V, pg, pc);
    }
  };

  const bool replays = nr <= (A.tz.on ? kReplayRowsTensor : kReplayRowsStored);
  const int kChunk = l >= 4 && !replays ? 1 : 2;   // cycles between reports
  const Pace pace = {1, 1, kChunk, l >= 4 ? 4 : replays ? 3 : 1, replays};
  ReplayKey key;
  key.op(A).add(V).add(P).add(W).add(st).add(S.nseg).add(l);
  for (const PartBuf* b : {&pa, &pb, &pg, &pc}) b->key(&key);
  auto run_chunk = [&](hipStream_t on) -> int {
    s = on;
    int crc = HZ_OK;
    for (int c = 0; c < kChunk && crc == HZ_OK; ++c) crc = enqueue_cycle();
    s = ctx->stream;
    return crc;
  };
  HZ_TRY(enqueue_resid(1));
  const BlSt* hst = poll.state<BlSt>(poll.posted - 1);
  int64_t queued = 0;                // cycles so far
  for (;;) {
    // everything queued has run: hst is the state
    bool all_done = true, any_brk = false;
    int max_iter = 0;
    for (int i = 0; i < S.nseg; ++i) {
      all_done = all_done && hst[i].done;
      any_brk = any_brk || (hst[i].brk && !hst[i].done);
      max_iter = std::max(max_iter, hst[i].iter);
    }
    int64_t mv = 2 * int64_t(l) * max_iter + resid_calls;
    if (all_done) {
      // the recursive residuals say converged: confirm with the true residual
      // (a segment whose recursion drifted restarts from it)
      HZ_TRY(enqueue_resid(1));
      hst = poll.state<BlSt>(poll.posted - 1);
      bool ok = true;
      for (int i = 0; i < S.nseg; ++i) ok = ok && hst[i].done;
      if (ok || mv + 1 >= ctl.max_matvec) break;
      continue;
    }
    if (mv + 2 * l > ctl.max_matvec) break;
    if (any_brk) {
      HZ_TRY(enqueue_resid(0));
      hst = poll.state<BlSt>(poll.posted - 1);
      continue;
    }
    int64_t left = (ctl.max_matvec - mv) / (2 * l);   // cycles that may still be queued
    const int first = poll.posted;
    for (bool stop = false; !stop && left > 0;) {
      const int n_cyc = int(std::min<int64_t>(pace.next(queued), left));
      bool ran = false;
      if (n_cyc == kChunk && replays) HZ_TRY(replay(ctx, p, key, run_chunk, &ran, kReplayAfter * 2 / kChunk));
      for (int c = 0; c < n_cyc && !ran; ++c) HZ_TRY(enqueue_cycle());
      left -= n_cyc;
      queued += n_cyc;
      HZ_TRY(report());
      const int k = poll.posted - (pace.at_once(queued) ? 1 : 2);
      if (k >= first) {
        HZ_TRY(poll.wait(k));
        const BlSt* h = poll.state<BlSt>(k);
        bool off = true, brk = false;
        for (int i = 0; i < S.nseg; ++i) {
          off = off && h[i].done;
          brk = brk || (h[i].brk && !h[i].done);
        }
        stop = off || brk;
      }
    }
    HZ_TRY(poll.wait(poll.posted - 1));
    hst = poll.state<BlSt>(poll.posted - 1);
  }
  if (A.tz.on) {
    k_bl_fold<T><<<W.nblk, kBlock, 0, s>>>(W, A.tz, st, V, 1);
    HZ_HIP(hipGetLastError());
  }
  out->iters.resize(S.nseg);
  out->matvecs.resize(S.nseg);
  out->status.resize(S.nseg);
  out->relres_est.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) {
    out->iters[i] = hst[i].iter;
    out->matvecs[i] = 2 * l * hst[i].iter + int(resid_calls);
    double fnv = out->fnorm[i];
    out->relres_est[i] = fnv > 0 ? std::sqrt(hst[i].rr) / fnv : 0.0;
    out->status[i] = hst[i].nan ? HZ_BREAKDOWN : (hst[i].done ? HZ_OK : HZ_NOT_CONVERGED);
  }
  return HZ_OK;
}

template int bicgstabl_run<double>(hz_ctx, const SegHost&, const SellOp<double>&, const z_t*, z_t*,
                                   const KrylovCtl&, KrylovOut*, const std::string&);
template int bicgstabl_run<float>(hz_ctx, const SegHost&, const SellOp<float>&, const c_t*, c_t*,
                                  const KrylovCtl&, KrylovOut*, const std::string&);
