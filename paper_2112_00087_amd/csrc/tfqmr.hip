// Transpose-free QMR of Freund (SIAM J. Sci. Comput. 14, 1993), the
// paper's P-tfQMR (Sec. 4, solver comparison table), on the right-Jacobi
// operator B = A D^-1, for every segment of a segmented system.
//
// Half-steps come in pairs (m even, m + 1 odd), one product each:
//   even:  alpha known;  u' = u - alpha v;  w -= alpha uhat;  d = u + (theta^2/alpha) eta d
//          theta = ||w|| / tau, c = 1/sqrt(1 + theta^2), tau *= theta c, eta = c^2 alpha
//          x += eta d;  uhat = B u'
//   odd:   w -= alpha uhat;  d = u' + (theta^2/alpha) eta d;  theta, c, tau, eta as above
//          x += eta d;  rho' = r*^H w, beta = rho'/rho;  u = w + beta u'
//          v = beta uhat + beta^2 v + B u;  uhat = B u;  alpha = rho' / r*^H v
// Kernels: 3 vector and 2 product (with fused dot) per pair; in the tensor form
// the odd update rides on the even product, 2 vector and 2 product kernels.
// The scalar steps run at the start of the kernel that needs them (advance) or,
// on large systems, in two or three kernels of their own (k_step), on a state
// that moves through three slots.  In the tensor form u, u', d and
// x are kept scaled by D^-1 (x is the solution itself), so only w and v are
// scaled where they enter u and u' and the product's inputs need no pass of
// their own.  u' lives in its own buffer for the odd half-step (it is never
// copied back into u), and the odd product reads B u' from uhat and writes B u
// over it row by row, so v needs no staging buffer: 32 vector passes per pair
// with the products' own, 29 in the tensor form.  A segment whose
// quasi-residual bound tau sqrt(m+1) meets the target makes its last x update
// in the kernel that finds it and stops; the host confirms with the true
// residual (restarting a segment that has not converged), and restarts
// segments that broke down (r*^H v or rho zero).
#include <chrono>

#include "ops.h"

namespace {

enum { kTqNone = 0, kTqAlpha, kTqEven, kTqOdd };
struct TqSt {
  z_t alpha, rho, beta, eta;
  double theta, tau, thr, thr2, rr;
  double chk;           // quasi-residual bound at the last stall checkpoint
  int m, iter, done, brk, nan, restart;
  int due, pad;         // due: the step that the sums formed next (or last) are for
  int mchk, stall_win;  // half-step of that checkpoint; its spacing (0: off)
  int stalled, pad2;    // the bound stalled: the solve ends unconfirmed
};

template <typename T>
struct TqV {
  const cx<T>* f;
  cx<T>* x;       // iterate of B x = f
  cx<T>* rs;      // shadow vector r*
  cx<T>* w;
  cx<T>* u;
  cx<T>* un;      // u' of the even half-step
  cx<T>* v;
  cx<T>* uh;      // B u, then B u'
  cx<T>* d;
};

template <typename T> __device__ __forceinline__ z_t zd(cx<T> a) { return ccast<double>(a); }
template <typename T> __device__ __forceinline__ cx<T> zt(z_t a) { return ccast<T>(a); }

template <typename T, int N>
struct TqRow {                     // a row of N vectors
  cx<T> v[N];
};
template <typename T>
struct TqPair {
  cx<T> a, b;
};

__device__ __forceinline__ bool tq_off(const TqSt& S) { return S.done || S.brk || S.nan; }

__device__ __forceinline__ void acc_dot(double* q, z_t a, z_t b) {
  q[0] = fma(a.re, b.re, fma(a.im, b.im, q[0]));
  q[1] = fma(a.re, b.im, fma(-a.im, b.re, q[1]));
}

// theta, c, tau, eta after w was updated; the stopping bound
__device__ __forceinline__ void tq_qmr(TqSt& S, double ww) {
  S.theta = sqrt(ww) / S.tau;
  const double c2 = 1.0 / (1.0 + S.theta * S.theta);
  S.tau = S.tau * S.theta * sqrt(c2);
  S.eta = c2 * S.alpha;
  S.iter += 1;
  if (!isfinite(ww)) {
    S.nan = 1;
    return;
  }
  const double bound = S.tau * sqrt(double(S.m + 1));
  if (bound <= S.thr) {
    S.done = 1;       // quasi-residual bound met: the last x update follows
  } else if (S.stall_win > 0 && S.m - S.mchk >= S.stall_win) {
    if (bound > 0.5 * S.chk) {
      S.done = 1;     // stalled: stop with the iterate reached (last x update follows)
      S.stalled = 1;
    }
    S.chk = bound;
    S.mchk = S.m;
  }
  S.m += 1;
}

// The scalar steps, run by one thread once a segment's sums are complete.
__device__ __forceinline__ void tq_resid(TqSt& S, const double* o) {
  const double rr = o[0];
  S.rr = rr;
  S.nan = !isfinite(rr);
  S.done = (rr <= S.thr2) || S.nan;
  S.brk = 0;
  S.restart = S.done ? 0 : 2;   // 2: the first product, v = uhat = B u, is due
  S.due = S.done ? kTqNone : kTqAlpha;
  S.tau = sqrt(rr);
  S.theta = 0.0;
  S.eta = z_t{0.0, 0.0};
  S.rho = z_t{rr, 0.0};
  S.m = 0;
  S.chk = S.tau;
  S.mchk = 0;
}
// alpha = rho / r*^H v
__device__ __forceinline__ void tq_alpha(TqSt& S, const double* o) {
  S.due = kTqEven;
  S.restart = 0;
  const z_t sg = {o[0], o[1]};
  if (norm2(sg) == 0.0 || !isfinite(o[0]) || !isfinite(o[1])) S.brk = 1;
  else S.alpha = cdiv(S.rho, sg);
}
__device__ __forceinline__ void tq_odd(TqSt& S, const double* o) {
  tq_qmr(S, o[0]);
  const z_t rho1 = {o[1], o[2]};
  if (norm2(S.rho) == 0.0 || !isfinite(o[1]) || !isfinite(o[2])) {
    if (!S.done) S.brk = 1;
  } else {
    S.beta = cdiv(rho1, S.rho);
    S.rho = rho1;
  }
  S.due = tq_off(S) ? kTqNone : kTqAlpha;   // k_tq_odd3 forms the sums of the alpha step
}
__device__ __forceinline__ void tq_even(TqSt& S, const double* o) {
  S.due = kTqOdd;
  tq_qmr(S, o[0]);
}
struct TqResid {
  __device__ bool on(const TqSt& S) const { return S.restart == 1; }
  __device__ void operator()(TqSt& S, const double* o) const { tq_resid(S, o); }
};
struct TqAlpha {
  __device__ bool on(const TqSt& S) const { return S.due == kTqAlpha; }
  __device__ void operator()(TqSt& S, const double* o) const { tq_alpha(S, o); }
};
struct TqEven {
  __device__ bool on(const TqSt& S) const { return !tq_off(S) && S.due == kTqEven; }
  __device__ void operator()(TqSt& S, const double* o) const { tq_even(S, o); }
};
struct TqOdd {
  __device__ bool on(const TqSt& S) const { return !tq_off(S) && S.due == kTqOdd; }
  __device__ void operator()(TqSt& S, const double* o) const { tq_odd(S, o); }
};

// ---------------------------------------------------------------- restart
// r0 = f - B x; r* = w = u = r0; d = 0; partial ||r0||^2
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_tq_resid(Seg L, SellOp<T> A, const TqSt* st, TqV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  if (st[t.seg].restart != 1) return;
  double q[1] = {0.0};
  for_rows<F, true>(A, t, V.x, [=](int64_t row) { return V.f[row]; },
              [&](int64_t row, cx<T> y, cx<T> f) {
                const cx<T> r = zt<T>(zd(f) - zd(y));
                V.rs[row] = r;
                V.w[row] = r;
                V.u[row] = r;
                V.d[row] = cx<T>{T(0), T(0)};
                q[0] += norm2(zd(r));
              });
  store_partials<1>(q, part, t);
}

// Tensor form: u is kept scaled by D^-1
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_tq_start(Seg L, TzOp Z, const TqSt* st, TqV<T> V) {
  const Tile t = vec_tile(L);
  if (st[t.seg].restart != 2) return;
  const TzSeg B = form_seg<F>(Z, t);
  vec_rows(L, t, [&](int64_t row) { V.u[row] = zt<T>(tz_pre<F>(Z, B, row, zd(V.u[row]))); });
}

// v = uhat = B u for restarting segments; partial r*^H v
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_tq_resid_prod(Seg L, SellOp<T> A, const TqSt* st, TqV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  if (st[t.seg].restart != 2) return;
  double q[2] = {0.0, 0.0};
  for_rows<F>(A, t, V.u, [=](int64_t row) { return V.rs[row]; },
              [&](int64_t row, cx<T> y, cx<T> rs) {
                V.v[row] = y;
                V.uh[row] = y;
                acc_dot(q, zd(rs), zd(y));
              });
  store_partials<2>(q, part, t);
}

// ---------------------------------------------------------------- even half-step
// alpha; u' = u - alpha v; w -= alpha uhat; d = u + (theta^2/alpha) eta d; partial ||w||^2
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_tq_even1(Seg L, TzOp Z, Part P, const TqSt* in, TqSt* out, TqV<T> V, double* part) {
  const SumTile t = vec_tile_sums(L);
  const TqSt& S = advance<2, (F < kFormTensor)>(P, in, out, t, first_block(L, t), TqAlpha{});
  if (tq_off(S)) return;
  const TzSeg B = form_seg<F>(Z, t);
  const z_t a = S.alpha;
  const z_t g = (S.theta * S.theta) * cdiv(S.eta, a);
  double q[1] = {0.0};
  vec_rows(L, t, [&](int64_t row) {
    const z_t u = zd(V.u[row]);
    const z_t av = a * zd(V.v[row]);
    const z_t w0 = zd(V.w[row]), uh = zd(V.uh[row]), d = zd(V.d[row]);
    const cx<T> w = zt<T>(tz_axmy<F>(a, uh, w0));
    V.un[row] = zt<T>(u - tz_pre<F>(Z, B, row, av));
    V.w[row] = w;
    V.d[row] = zt<T>(tz_axpy<F>(g, d, u));
    q[0] += norm2(zd(w));
  });
  store_partials<1>(q, part, t);
}

// theta, tau, eta; x += eta d; then (unless stopping) uhat = B u' (stored forms).
// prev: the state before the step, whoever made it.
// x is updated ahead of the product: with eta and the stop flag held across it
// the kernel took 98 VGPRs instead of 92 and lost a wave per SIMD (38.5 -> 42.3
// us at 289,937 rows in split form).
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_tq_even2(Seg L, SellOp<T> A, Part P, const TqSt* prev, const TqSt* in, TqSt* out,
                                             TqV<T> V) {
  const Tile t = tile_of(L);
  const bool was_done = prev[t.seg].done;
  const TqSt& S = advance<1, (F < kFormTensor)>(P, in, out, t, first_block(L, t), TqEven{});
  if (S.brk || S.nan || was_done) return;
  V.x[t.row] = zt<T>(zd(V.x[t.row]) + S.eta * zd(V.d[t.row]));
  if (S.done) return;
  V.uh[t.row] = sell_row_form<F>(A, t.row, V.un);
}

// ---------------------------------------------------------------- odd half-step
// w -= alpha uhat; d = u' + (theta^2/alpha) eta d; partials ||w||^2, r*^H w
template <typename T>
__global__ void __launch_bounds__(kBlock) k_tq_odd1(Seg L, const TqSt* st, TqV<T> V, double* part) {
  const SumTile t = vec_tile_sums(L);
  const TqSt& S = st[t.seg];
  if (tq_off(S)) return;
  const z_t a = S.alpha;
  const z_t g = (S.theta * S.theta) * cdiv(S.eta, a);
  double q[3] = {0.0, 0.0, 0.0};
  vec_rows(L, t, [&](int64_t row) {
    const cx<T> w = zt<T>(zd(V.w[row]) - a * zd(V.uh[row]));
    const z_t d = zd(V.un[row]) + g * zd(V.d[row]), rs = zd(V.rs[row]);
    V.w[row] = w;
    V.d[row] = zt<T>(d);
    const z_t wv = zd(w);
    q[0] += norm2(wv);
    acc_dot(q + 1, rs, wv);
  });
  store_partials<3>(q, part, t);
}

// Both at once in the tensor form, whose product kernel has registers to
// spare: the odd update of a row only needs that row's B u', so w and d are
// read and written beside it instead of by a pass that also reads u', uhat
// and d again (12 -> 9 vector passes; at 161x97x81 nodes 45.8 -> 38.1 us,
// and one launch less where launches count).
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_tq_even2_odd1(Seg L, SellOp<T> A, Part P, const TqSt* prev, const TqSt* in,
                                                  TqSt* out, TqV<T> V, double* part) {
  const SumTile t = prod_tile_sums<F>(L);
  const bool was_done = prev[t.seg].done;
  const TqSt& S = advance<1, (F < kFormTensor)>(P, in, out, t, first_block(L, t), TqEven{});
  if (S.brk || S.nan || was_done) return;
  const z_t eta = S.eta, a = S.alpha;
  const z_t g = (S.theta * S.theta) * cdiv(eta, a);
  const bool done = S.done;
  double q[3] = {0.0, 0.0, 0.0};
  for_rows<F>(A, t, V.un,
              [=](int64_t row) { return TqRow<T, 5>{V.x[row], V.d[row], V.w[row], V.rs[row], V.un[row]}; },
              [&](int64_t row, cx<T> y, const TqRow<T, 5>& r) {
                const z_t d0 = zd(r.v[1]);
                V.x[row] = zt<T>(tz_axpy<F>(eta, d0, zd(r.v[0])));
                if (done) return;
                const cx<T> w = zt<T>(tz_axmy<F>(a, zd(y), zd(r.v[2])));
                V.uh[row] = y;
                V.w[row] = w;
                V.d[row] = zt<T>(tz_axpy<F>(g, d0, zd(r.v[4])));
                const z_t wv = zd(w);
                q[0] += norm2(wv);
                acc_dot(q + 1, zd(r.v[3]), wv);
              });
  store_partials<3>(q, part, t);
}

// theta, tau, eta, beta; x += eta d; then (unless stopping) u = w + beta u'
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_tq_odd2(Seg L, TzOp Z, Part P, const TqSt* prev, const TqSt* in, TqSt* out,
                                                    TqV<T> V) {
  const Tile t = vec_tile(L);
  const bool was_done = prev[t.seg].done;
  const TqSt& S = advance<3, (F < kFormTensor)>(P, in, out, t, first_block(L, t), TqOdd{});
  if (S.nan || (S.brk && !S.done) || was_done) return;
  const TzSeg B = form_seg<F>(Z, t);
  if (S.done) {
    vec_rows(L, t, [&](int64_t row) { V.x[row] = zt<T>(zd(V.x[row]) + S.eta * zd(V.d[row])); });
    return;
  }
  const z_t eta = S.eta, beta = S.beta;
  vec_rows(L, t, [&](int64_t row) {
    const z_t x = zd(V.x[row]), d = zd(V.d[row]), w = zd(V.w[row]), un = zd(V.un[row]);
    V.x[row] = zt<T>(tz_axpy<F>(eta, d, x));
    V.u[row] = zt<T>(tz_axpy<F>(beta, un, tz_pre<F>(Z, B, row, w)));
  });
}

// uhat = B u over B u' (each row reads its old value first); v = beta B u'
// + beta^2 v + B u, the first two terms rounded to the storage type before
// the product is added; partial r*^H v
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_tq_odd3(Seg L, SellOp<T> A, const TqSt* st, TqV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  const TqSt& S = st[t.seg];
  if (tq_off(S)) return;
  const z_t b = S.beta;
  const z_t b2 = b * b;
  double q[2] = {0.0, 0.0};
  if constexpr (F == kFormTensor || F == kFormTensorExt) {
    for_rows<F>(A, t, V.u,
                [=](int64_t row) { return TqPair<T>{zt<T>(b * zd(V.uh[row]) + b2 * zd(V.v[row])), V.rs[row]}; },
                [&](int64_t row, cx<T> y, TqPair<T> a) {
                  V.uh[row] = y;
                  const cx<T> v = zt<T>(zd(a.a) + zd(y));
                  V.v[row] = v;
                  acc_dot(q, zd(a.b), zd(v));
                });
  } else {
    const cx<T> vt = zt<T>(b * zd(V.uh[t.row]) + b2 * zd(V.v[t.row]));
    const cx<T> y = sell_row_form<F>(A, t.row, V.u);
    V.uh[t.row] = y;
    const cx<T> v = zt<T>(zd(vt) + zd(y));
    V.v[t.row] = v;
    acc_dot(q, zd(V.rs[t.row]), zd(v));
  }
  store_partials<2>(q, part, t);
}

__global__ void k_tq_set_thr(int nseg, TqSt* st, const double* fn2, double tol, int stall_win) {
  int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= nseg) return;
  st[s].thr2 = tol * tol * fn2[s];
  st[s].thr = tol * sqrt(fn2[s]);
  st[s].iter = 0;
  st[s].restart = 1;
  st[s].stall_win = stall_win;
  st[s].stalled = 0;
}

}  // namespace

template <typename T>
int tfqmr_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* x, const KrylovCtl& ctl,
              KrylovOut* out, const std::string& tag) {
  int rc = 0;
  const int64_t nr = S.nrows;
  const size_t vb = sizeof(cx<T>) * nr;
  const std::string p = "tfqmr." + tag + (sizeof(T) == 8 ? ".z." : ".c.");
  TqV<T> V = {};
  V.f = f;
  V.x = x;
  cx<T>** vecs[7] = {&V.rs, &V.w, &V.u, &V.un, &V.v, &V.uh, &V.d};
  const char* names[7] = {"rs", "w", "u", "un", "v", "uh", "d"};
  for (int i = 0; i < 7; ++i) {
    DevBuf* b = ctx->buf(p + names[i], vb, &rc);
    if (rc) return rc;
    *vecs[i] = b->as<cx<T>>();
  }
  // state slots: start of a pair, after alpha, after the even half-step; one nobody reads
  DevBuf* stb = ctx->buf(p + "st", sizeof(TqSt) * 4 * S.nseg, &rc);
  if (rc) return rc;
  DevBuf* fnb = ctx->buf(p + "fn2", sizeof(double) * S.nseg, &rc);
  if (rc) return rc;
  TqSt *st = stb->as<TqSt>(), *st_a = st + S.nseg, *st_e = st_a + S.nseg, *st_u = st_e + S.nseg;   // st: what a pair starts from
  hipStream_t s = ctx->stream;
  const Seg& L = S.dev;
  const Seg& P = prod_seg(A, L);   // the products' layout

  std::vector<double> fn2;
  HZ_TRY(seg_norm2_t<T>(ctx, S, f, &fn2));
  out->fnorm.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) out->fnorm[i] = std::sqrt(fn2[i]);
  HZ_HIP(hipMemcpyAsync(fnb->p, fn2.data(), sizeof(double) * S.nseg, hipMemcpyHostToDevice, s));
  HZ_HIP(hipMemsetAsync(stb->p, 0, sizeof(TqSt) * 4 * S.nseg, s));
  k_tq_set_thr<<<ceil_div(S.nseg, kBlock), kBlock, 0, s>>>(S.nseg, st, fnb->as<double>(), ctl.tol,
                                                            ctl.stall_halfsteps);
  HZ_HIP(hipGetLastError());

  StatePoll poll;
  HZ_TRY(poll.init(ctx, sizeof(TqSt) * S.nseg));
  const Seg& W = A.tz.on ? S.vec_runs : S.vec;   // vector layout
  PartBuf pr, pa, pe, po;            // sums of the residual, alpha, even and odd steps
  HZ_TRY(pr.init(ctx, S, P, 1, W.nblk, p + "part.r"));
  HZ_TRY(pa.init(ctx, S, P, 2, W.nblk, p + "part.a"));
  HZ_TRY(pe.init(ctx, S, W, 1, W.nblk, p + "part.e"));
  HZ_TRY(po.init(ctx, S, A.tz.on ? P : W, 3, W.nblk, p + "part.o"));
  int64_t restarts = 0, pairs = 0;

  auto report = [&]() -> int {
    HZ_TRY(pa.step_now<2>(s, st, poll.slot<TqSt>(), TqAlpha{}));
    return poll.posted_one();
  };
  auto enqueue_restart = [&](int all) -> int {
    if (restarts > 0) HZ_TRY(pa.step_now<2>(s, st, st, Settle<TqAlpha>{{}, all}));
    HZ_BY_FORM(A, k_tq_resid<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, st, V, pr.raw));
    HZ_TRY(pr.step_now<1>(s, st, st, TqResid{}));
    // u = r_0 is the first product's input
    if (A.tz.on) HZ_BY_SCALING(A, k_tq_start<T, F><<<W.nblk, kBlock, 0, s>>>(W, A.tz, st, V));
    HZ_BY_FORM(A, k_tq_resid_prod<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, st, V, pa.raw));
    HZ_TRY(pa.step<2>(s, st, st_a, TqAlpha{}));
    HZ_HIP(hipGetLastError());
    ++restarts;
    HZ_TRY(report());
    return poll.wait(poll.posted - 1);
  };
  auto enqueue_pair = [&]() -> int {
    HZ_BY_SCALING(A, k_tq_even1<T, F><<<W.nblk, kBlock, 0, s>>>(W, A.tz, pa.part, pa.from(st, st_a), pa.to(st_a, st_u), V, pe.raw));
    HZ_TRY(pe.step<1>(s, st_a, st_e, TqEven{}));
    if (A.tz.on == 1) {
      k_tq_even2_odd1<T, kFormTensor><<<P.nblk, kBlock, 0, s>>>(P, A, pe.part, st_a, pe.from(st_a, st_e), pe.to(st_e, st_u), V, po.raw);
    } else if (A.tz.on) {
      k_tq_even2_odd1<T, kFormTensorExt><<<P.nblk, kBlock, 0, s>>>(P, A, pe.part, st_a, pe.from(st_a, st_e), pe.to(st_e, st_u), V, po.raw);
    } else {
      HZ_BY_STORED(A, k_tq_even2<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, pe.part, st_a, pe.from(st_a, st_e), pe.to(st_e, st_u), V));
      k_tq_odd1<T><<<W.nblk, kBlock, 0, s>>>(W, st_e, V, po.raw);
    }
    HZ_TRY(po.step<3>(s, st_e, st, TqOdd{}));
    HZ_BY_SCALING(A, k_tq_odd2<T, F><<<W.nblk, kBlock, 0, s>>>(W, A.tz, po.part, st_e, po.from(st_e, st), po.to(st, st_u), V));
    HZ_BY_FORM(A, k_tq_odd3<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, st, V, pa.raw));
    HZ_TRY(pa.step<2>(s, st, st_a, TqAlpha{}));
    HZ_HIP(hipGetLastError());
    return HZ_OK;
  };

  constexpr int kChunk = 8;          // pairs between reports
  const bool replays = nr <= (A.tz.on ? kReplayRowsTensor : kReplayRowsStored);
  const Pace pace = {4, 2, kChunk, replays ? 12 : 4, replays};
  ReplayKey key;
  key.op(A).add(V).add(P).add(W).add(st).add(S.nseg);
  for (const PartBuf* b : {&pa, &pe, &po}) b->key(&key);
  auto run_chunk = [&](hipStream_t on) -> int {
    s = on;
    int crc = HZ_OK;
    for (int c = 0; c < kChunk && crc == HZ_OK; ++c) crc = enqueue_pair();
    s = ctx->stream;
    return crc;
  };
  HZ_TRY(enqueue_restart(1));
  const TqSt* hst = poll.state<TqSt>(poll.posted - 1);
  for (;;) {
    // everything queued has run: hst is the state
    bool all_done = true, any_brk = false, any_stalled = false;
    for (int i = 0; i < S.nseg; ++i) {
      all_done = all_done && hst[i].done;
      any_brk = any_brk || (hst[i].brk && !hst[i].done);
      any_stalled = any_stalled || hst[i].stalled;
    }
    // products so far: two per restart, two per queued pair (stopped segments idle)
    const int64_t mv = 2 * restarts + 2 * pairs;
    if (all_done && any_stalled) break;   // hand the iterate reached back to the refinement
    if (all_done) {
      HZ_TRY(enqueue_restart(1));   // confirm with the true residual
      hst = poll.state<TqSt>(poll.posted - 1);
      bool ok = true;
      for (int i = 0; i < S.nseg; ++i) ok = ok && hst[i].done;
      if (ok || mv + 2 >= ctl.max_matvec) break;
      continue;
    }
    if (mv + 2 > ctl.max_matvec) break;
    if (any_brk) {
      HZ_TRY(enqueue_restart(0));
      hst = poll.state<TqSt>(poll.posted - 1);
      continue;
    }
    int64_t left = (ctl.max_matvec - mv) / 2;   // pairs that may still be queued
    const int first = poll.posted;
    for (bool stop = false; !stop && left > 0;) {
      const int n_pair = int(std::min<int64_t>(pace.next(pairs), left));
      bool ran = false;
      if (n_pair == kChunk && replays) HZ_TRY(replay(ctx, p, key, run_chunk, &ran, kReplayAfter));
      for (int c = 0; c < n_pair && !ran; ++c) HZ_TRY(enqueue_pair());
      pairs += n_pair;
      left -= n_pair;
      HZ_TRY(report());
      const int k = poll.posted - (pace.at_once(pairs) ? 1 : 2);
      if (k >= first) {
        HZ_TRY(poll.wait(k));
        const TqSt* h = poll.state<TqSt>(k);
        bool off = true, brk = false;
        for (int i = 0; i < S.nseg; ++i) {
          off = off && h[i].done;
          brk = brk || (h[i].brk && !h[i].done);
        }
        stop = off || brk;
      }
    }
    HZ_TRY(poll.wait(poll.posted - 1));
    hst = poll.state<TqSt>(poll.posted - 1);
  }
  out->iters.resize(S.nseg);
  out->matvecs.resize(S.nseg);
  out->status.resize(S.nseg);
  out->relres_est.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) {
    out->iters[i] = hst[i].iter;
    out->matvecs[i] = hst[i].iter + 2 * int(restarts);
    const double fnv = out->fnorm[i];
    out->relres_est[i] = fnv > 0 ? std::sqrt(hst[i].rr) / fnv : 0.0;
    out->status[i] = hst[i].nan ? HZ_BREAKDOWN : (hst[i].done && !hst[i].stalled ? HZ_OK : HZ_NOT_CONVERGED);
  }
  return HZ_OK;
}

template int tfqmr_run<double>(hz_ctx, const SegHost&, const SellOp<double>&, const z_t*, z_t*, const KrylovCtl&,
                               KrylovOut*, const std::string&);
template int tfqmr_run<float>(hz_ctx, const SegHost&, const SellOp<float>&, const c_t*, c_t*, const KrylovCtl&,
                              KrylovOut*, const std::string&);
