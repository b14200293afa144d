// Stabilised bi-conjugate gradient method (the paper's P-BiCGSTAB, Sec. 4)
// on the right-Jacobi operator, for every segment of a segmented system.
//
// One iteration of van der Vorst's method is five kernels, two of them
// products.  The scalar steps (alpha, omega, rho and beta) run at the start
// of the kernel that needs them (advance), on large systems in three kernels of
// their own (k_step), on a state that moves through three slots.  The
// early-exit test on ||s|| rides on the omega step.  The scalars never leave
// the device; the host reads the per-segment state after each chunk of
// iterations, once the next chunk is queued (Pace).
// Every kernel first reads its segment's flags and returns if that segment
// has converged, so extra queued iterations cost only empty launches.
#include <chrono>

#include "ops.h"

namespace {

enum { kBiNone = 0, kBiAlpha, kBiOmega, kBiRho };
struct BiSt {
  z_t rho, rho_old, alpha, omega;
  z_t beta;                       // (rho / rho_old) (alpha / omega) for the next p update
  double rr, ss, thr2, rhat2;
  int iter, done, early, reset;
  int nan, due;                   // due: the step that the sums formed next (or last) are for
};

template <typename T>
struct BiV {
  const cx<T>* f;
  cx<T>* u;
  cx<T>* r;
  cx<T>* rhat;
  cx<T>* p;
  cx<T>* v;
  cx<T>* s;
  cx<T>* t;
};

template <typename T> __device__ __forceinline__ z_t zd(cx<T> a) { return ccast<double>(a); }
template <typename T> __device__ __forceinline__ cx<T> zt(z_t a) { return ccast<T>(a); }

// ---- the scalar steps, run by one thread once a segment's sums are complete
__device__ __forceinline__ void bi_resid(BiSt& S, const double* o) {
  const double rr = o[0];
  S.rr = rr;
  S.rho = z_t{rr, 0.0};
  S.rho_old = S.alpha = S.omega = z_t{1.0, 0.0};
  S.beta = z_t{rr, 0.0};
  S.rhat2 = rr;
  S.early = 0;
  S.reset = 0;
  S.due = kBiAlpha;
  S.nan = !isfinite(rr);
  S.done = (rr <= S.thr2) || S.nan;
}
__device__ __forceinline__ void bi_alpha(BiSt& S, const double* o) {
  S.reset = 0;
  S.due = kBiOmega;
  const z_t rv = {o[0], o[1]};
  if (norm2(rv) == 0.0 || !isfinite(o[0]) || !isfinite(o[1])) {
    S.alpha = z_t{0.0, 0.0};   // minimal-residual step this iteration, restart after it
    S.reset = 1;
  } else {
    S.alpha = cdiv(S.rho, rv);
  }
}
// omega = t^H s / t^H t, or the early exit when ||s|| already meets the target
// (then x += alpha p completes the iteration).
__device__ __forceinline__ void bi_omega(BiSt& S, const double* o) {
  const double re = o[0], im = o[1], tt = o[2], ss = o[3];
  S.ss = ss;
  S.early = (ss <= S.thr2) ? 1 : 0;
  S.omega = (tt > 0.0 && !S.early) ? z_t{re / tt, im / tt} : z_t{0.0, 0.0};
  S.due = kBiRho;            // k_xr forms the sums of the rho step
}
__device__ __forceinline__ void bi_rho(BiSt& S, const double* o) {
  S.due = kBiAlpha;
  if (S.early) {
    S.iter += 1;
    S.rr = S.ss;
    S.done = 1;
    S.early = 0;
    return;
  }
  const double re = o[0], im = o[1], rr = o[2];
  S.iter += 1;
  S.rho_old = S.rho;
  S.rho = z_t{re, im};
  S.rr = rr;
  if (!isfinite(rr) || !isfinite(re) || !isfinite(im)) {
    S.nan = 1;
    S.done = 1;
  } else if (rr <= S.thr2) {
    S.done = 1;
  } else if (sqrt(norm2(S.rho)) < 1e-300 * sqrt(S.rhat2 * rr) || norm2(S.omega) == 0.0) {
    // breakdown: restart the shadow residual from the current residual
    S.reset = 1;
    S.rho = z_t{rr, 0.0};
    S.rho_old = S.alpha = S.omega = z_t{1.0, 0.0};
    S.rhat2 = rr;
  }
  S.beta = cdiv(S.rho, S.rho_old) * cdiv(S.alpha, S.omega);
}

struct BiResid {
  __device__ bool on(const BiSt&) const { return true; }
  __device__ void operator()(BiSt& S, const double* o) const { bi_resid(S, o); }
};
struct BiAlpha {
  __device__ bool on(const BiSt& S) const { return !S.done && S.due == kBiAlpha; }
  __device__ void operator()(BiSt& S, const double* o) const { bi_alpha(S, o); }
};
struct BiOmega {
  __device__ bool on(const BiSt& S) const { return !S.done && S.due == kBiOmega; }
  __device__ void operator()(BiSt& S, const double* o) const { bi_omega(S, o); }
};
struct BiRho {
  __device__ bool on(const BiSt& S) const { return S.due == kBiRho; }
  __device__ void operator()(BiSt& S, const double* o) const { bi_rho(S, o); }
};

// r = f - A u; restart: rhat = r, p = v = 0.  Partial ||r||^2.
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_resid(Seg L, SellOp<T> A, BiV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  double q[1] = {0.0};
  for_rows<F>(A, t, V.u, [=](int64_t row) { return V.f[row]; },
              [&](int64_t row, cx<T> y, cx<T> f) {
                const cx<T> rs = zt<T>(zd(f) - zd(y));
                V.r[row] = rs;
                V.rhat[row] = rs;
                V.p[row] = cx<T>{T(0), T(0)};
                V.v[row] = cx<T>{T(0), T(0)};
                q[0] += norm2(zd(rs));
              });
  store_partials<1>(q, part, t);
}

// rho and beta; p = r + beta (p - omega v), beta = (rho / rho_old) (alpha / omega); on reset
// rhat = p = r.  In the tensor form p is kept scaled by D^-1.
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_p(Seg L, TzOp Z, Part P, const BiSt* in, BiSt* out, BiV<T> V) {
  const Tile t = vec_tile(L);
  const BiSt& S = advance<3, (F < kFormTensor)>(P, in, out, t, first_block(L, t), BiRho{});
  if (S.done) return;
  const TzSeg B = form_seg<F>(Z, t);
  if (S.reset) {
    vec_rows(L, t, [&](int64_t row) {
      const cx<T> r = V.r[row];
      V.rhat[row] = r;
      V.p[row] = zt<T>(tz_pre<F>(Z, B, row, zd(r)));
    });
    return;
  }
  const z_t beta = S.beta, omega = S.omega, bo = beta * omega;
  vec_rows(L, t, [&](int64_t row) {
    const z_t r = zd(V.r[row]), p = zd(V.p[row]), v = zd(V.v[row]);
    if (F == kFormComplex) V.p[row] = zt<T>(r + beta * (p - omega * v));
    else V.p[row] = zt<T>(tz_pre<F>(Z, B, row, r - bo * v) + beta * p);
  });
}

// v = A p; partial rhat^H v.  Instantiated per storage form F of A (one form
// per kernel keeps the register count, hence the occupancy, of that form).
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_v(Seg L, SellOp<T> A, const BiSt* st, BiV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  if (st[t.seg].done) return;
  double q[2] = {0.0, 0.0};
  for_rows<F>(A, t, V.p, [=](int64_t row) { return V.rhat[row]; },
              [&](int64_t row, cx<T> y, cx<T> rh) {
                V.v[row] = y;
                const z_t a = zd(rh), b = zd(y);
                q[0] += a.re * b.re + a.im * b.im;
                q[1] += a.re * b.im - a.im * b.re;
              });
  store_partials<2>(q, part, t);
}

// alpha; s = r - alpha v (scaled by D^-1 in the tensor form).
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_s(Seg L, TzOp Z, Part P, const BiSt* in, BiSt* out, BiV<T> V) {
  const Tile t = vec_tile(L);
  const BiSt& S = advance<2, (F < kFormTensor)>(P, in, out, t, first_block(L, t), BiAlpha{});
  if (S.done) return;
  const TzSeg B = form_seg<F>(Z, t);
  const z_t alpha = S.alpha;
  vec_rows(L, t, [&](int64_t row) {
    V.s[row] = zt<T>(tz_pre<F>(Z, B, row, zd(V.r[row]) - alpha * zd(V.v[row])));
  });
}

// t = A s; partials t^H s, t^H t, s^H s (s unscaled; per storage form F, as k_v).
template <typename T, int F>
__global__ void HZ_PRODUCT_BOUNDS k_t(Seg L, SellOp<T> A, const BiSt* st, BiV<T> V, double* part) {
  SumTile t = prod_tile_sums<F>(L);
  if (st[t.seg].done) return;
  const TzSeg B = form_seg<F>(A.tz, t);
  double q[4] = {0.0, 0.0, 0.0, 0.0};
  for_rows<F>(A, t, V.s, [&](int64_t row) { return tz_unpre<F>(A.tz, B, row, zd(V.s[row])); },
              [&](int64_t row, cx<T> y, z_t b) {
                V.t[row] = y;
                const z_t a = zd(y);
                q[0] += a.re * b.re + a.im * b.im;
                q[1] += a.re * b.im - a.im * b.re;
                q[2] += norm2(a);
                q[3] += norm2(b);
              });
  store_partials<4>(q, part, t);
}

// omega; u += alpha p + omega s; r = s - omega t (s unscaled); partials rhat^H r, ||r||^2.
template <typename T, int F>
__global__ void __launch_bounds__(kBlock) k_xr(Seg L, TzOp Z, Part P, const BiSt* in, BiSt* out, BiV<T> V, double* part) {
  const SumTile t = vec_tile_sums(L);
  const BiSt& S = advance<4, (F < kFormTensor)>(P, in, out, t, first_block(L, t), BiOmega{});
  if (S.done) return;
  const TzSeg B = form_seg<F>(Z, t);
  double q[3] = {0.0, 0.0, 0.0};
  if (S.early) {
    vec_rows(L, t, [&](int64_t row) { V.u[row] = zt<T>(zd(V.u[row]) + S.alpha * zd(V.p[row])); });
  } else {
    vec_rows(L, t, [&](int64_t row) {
      const z_t u = zd(V.u[row]) + S.alpha * zd(V.p[row]);
      const z_t s = zd(V.s[row]);
      V.u[row] = zt<T>(u + S.omega * s);
      const cx<T> r = zt<T>(tz_unpre<F>(Z, B, row, s) - S.omega * zd(V.t[row]));
      V.r[row] = r;
      const z_t a = zd(V.rhat[row]), b = zd(r);
      q[0] += a.re * b.re + a.im * b.im;
      q[1] += a.re * b.im - a.im * b.re;
      q[2] += norm2(b);
    });
  }
  store_partials<3>(q, part, t);
}

__global__ void k_set_thr(int nseg, BiSt* st, const double* fn2, double tol, int reset_iter) {
  int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= nseg) return;
  st[s].thr2 = tol * tol * fn2[s];
  if (reset_iter) st[s].iter = 0;
}

}  // namespace

template <typename T>
int bicgstab_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
                 const KrylovCtl& ctl, KrylovOut* out, const std::string& tag) {
  int rc = 0;
  const int64_t nr = S.nrows;
  const size_t vb = sizeof(cx<T>) * nr;
  const std::string p = "bicg." + tag + (sizeof(T) == 8 ? ".z." : ".c.");
  BiV<T> V;
  V.f = f;
  V.u = u;
  cx<T>** vecs[6] = {&V.r, &V.rhat, &V.p, &V.v, &V.s, &V.t};
  const char* names[6] = {"r", "rhat", "p", "v", "s", "t"};
  for (int i = 0; i < 6; ++i) {
    DevBuf* b = ctx->buf(p + names[i], vb, &rc);
    if (rc) return rc;
    *vecs[i] = b->as<cx<T>>();
  }
  // state slots: after rho (start of an iteration), alpha, omega; one nobody reads
  DevBuf* stb = ctx->buf(p + "st", sizeof(BiSt) * 4 * S.nseg, &rc);
  if (rc) return rc;
  DevBuf* fnb = ctx->buf(p + "fn2", sizeof(double) * S.nseg, &rc);
  if (rc) return rc;
  BiSt *st = stb->as<BiSt>(), *st_a = st + S.nseg, *st_b = st_a + S.nseg, *st_u = st_b + S.nseg;   // st: what an iteration starts from
  hipStream_t s = ctx->stream;
  const Seg& L = S.dev;
  const Seg& P = prod_seg(A, L);   // the products' layout

  // ||f||^2 per segment -> thresholds
  std::vector<double> fn2;
  HZ_TRY(seg_norm2_t<T>(ctx, S, f, &fn2));
  out->fnorm.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) out->fnorm[i] = std::sqrt(fn2[i]);
  HZ_HIP(hipMemcpyAsync(fnb->p, fn2.data(), sizeof(double) * S.nseg, hipMemcpyHostToDevice, s));
  HZ_HIP(hipMemsetAsync(stb->p, 0, sizeof(BiSt) * 4 * S.nseg, s));
  k_set_thr<<<ceil_div(S.nseg, kBlock), kBlock, 0, s>>>(S.nseg, st, fnb->as<double>(), ctl.tol, 1);
  HZ_HIP(hipGetLastError());

  StatePoll poll;
  HZ_TRY(poll.init(ctx, sizeof(BiSt) * S.nseg));
  const Seg& W = A.tz.on ? S.vec_runs : S.vec;   // vector layout
  PartBuf pr, pa, po, pn;            // sums of the residual, alpha, omega and rho steps
  HZ_TRY(pr.init(ctx, S, P, 1, W.nblk, p + "part.r"));
  HZ_TRY(pa.init(ctx, S, P, 2, W.nblk, p + "part.a"));
  HZ_TRY(po.init(ctx, S, P, 4, W.nblk, p + "part.o"));
  HZ_TRY(pn.init(ctx, S, W, 3, W.nblk, p + "part.n"));
  int64_t resid_calls = 0;

  auto report = [&]() -> int {
    HZ_TRY(pn.step_now<3>(s, st, poll.slot<BiSt>(), BiRho{}));
    return poll.posted_one();
  };
  auto enqueue_resid = [&]() -> int {
    // the slot an iteration starts from takes up the sums of its rho step
    if (resid_calls > 0) HZ_TRY(pn.step_now<3>(s, st, st, BiRho{}));
    HZ_BY_FORM(A, k_resid<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, V, pr.raw));
    HZ_HIP(hipGetLastError());
    // (no rho step is due: st_a is what the next iteration's first step would make of st)
    HZ_TRY(pr.step_now<1>(s, st, st, BiResid{}, poll.slot<BiSt>(), st_a));
    ++resid_calls;
    return poll.posted_one();
  };
  auto enqueue_iter = [&]() -> int {
    HZ_BY_SCALING(A, k_p<T, F><<<W.nblk, kBlock, 0, s>>>(W, A.tz, pn.part, pn.from(st, st_a), pn.to(st_a, st_u), V));
    HZ_BY_FORM(A, k_v<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, st_a, V, pa.raw));
    HZ_TRY(pa.step<2>(s, st_a, st_b, BiAlpha{}));
    HZ_BY_SCALING(A, k_s<T, F><<<W.nblk, kBlock, 0, s>>>(W, A.tz, pa.part, pa.from(st_a, st_b), pa.to(st_b, st_u), V));
    HZ_BY_FORM(A, k_t<T, F><<<P.nblk, kBlock, 0, s>>>(P, A, st_b, V, po.raw));
    HZ_TRY(po.step<4>(s, st_b, st, BiOmega{}));
    HZ_BY_SCALING(A, k_xr<T, F><<<W.nblk, kBlock, 0, s>>>(W, A.tz, po.part, po.from(st_b, st), po.to(st, st_u), V, pn.raw));
    HZ_TRY(pn.step<3>(s, st, st_a, BiRho{}));
    HZ_HIP(hipGetLastError());
    return HZ_OK;
  };

  constexpr int kChunk = 8;          // iterations between reports
  const bool replays = nr <= (A.tz.on ? kReplayRowsTensor : kReplayRowsStored);
  const Pace pace = {4, 2, kChunk, replays ? 12 : 4, replays};
  ReplayKey key;
  key.op(A).add(V).add(P).add(W).add(st).add(S.nseg);
  for (const PartBuf* b : {&pa, &po, &pn}) b->key(&key);
  auto run_chunk = [&](hipStream_t on) -> int {
    s = on;
    int crc = HZ_OK;
    for (int it = 0; it < kChunk && crc == HZ_OK; ++it) crc = enqueue_iter();
    s = ctx->stream;
    return crc;
  };
  HZ_TRY(enqueue_resid());
  HZ_TRY(poll.wait(0));
  const BiSt* hst = poll.state<BiSt>(0);
  int64_t queued = 0;                // iterations so far
  for (;;) {
    // everything queued has run: hst is the state
    bool all_done = true;
    int max_iter = 0;
    for (int i = 0; i < S.nseg; ++i) {
      all_done = all_done && hst[i].done;
      max_iter = std::max(max_iter, hst[i].iter);
    }
    const int64_t mv = 2 * int64_t(max_iter) + resid_calls;
    if (all_done) {
      // the recursive residuals say converged: confirm with the true residual
      // (a fresh residual also restarts any segment that drifted)
      HZ_TRY(enqueue_resid());
      HZ_TRY(poll.wait(poll.posted - 1));
      hst = poll.state<BiSt>(poll.posted - 1);
      bool ok = true;
      for (int i = 0; i < S.nseg; ++i) ok = ok && hst[i].done;
      if (ok || mv + 1 >= ctl.max_matvec) break;
      continue;
    }
    int64_t left = (ctl.max_matvec - mv) / 2;   // iterations that may still be queued
    if (left < 1) break;
    const int first = poll.posted;
    for (bool stop = false; !stop && left > 0;) {
      const int n_it = int(std::min<int64_t>(pace.next(queued), left));
      bool ran = false;
      if (n_it == kChunk && replays) HZ_TRY(replay(ctx, p, key, run_chunk, &ran, kReplayAfter));
      for (int it = 0; it < n_it && !ran; ++it) HZ_TRY(enqueue_iter());
      left -= n_it;
      queued += n_it;
      HZ_TRY(report());
      const int k = poll.posted - (pace.at_once(queued) ? 1 : 2);
      if (k >= first) {
        HZ_TRY(poll.wait(k));
        const BiSt* h = poll.state<BiSt>(k);
        stop = true;
        for (int i = 0; i < S.nseg; ++i) stop = stop && h[i].done;
      }
    }
    HZ_TRY(poll.wait(poll.posted - 1));
    hst = poll.state<BiSt>(poll.posted - 1);
  }
  out->iters.resize(S.nseg);
  out->matvecs.resize(S.nseg);
  out->status.resize(S.nseg);
  out->relres_est.resize(S.nseg);
  for (int i = 0; i < S.nseg; ++i) {
    out->iters[i] = hst[i].iter;
    out->matvecs[i] = 2 * hst[i].iter + int(resid_calls);
    double fnv = out->fnorm[i];
    out->relres_est[i] = fnv > 0 ? std::sqrt(hst[i].rr) / fnv : 0.0;
    out->status[i] = hst[i].nan ? HZ_BREAKDOWN : (hst[i].done ? HZ_OK : HZ_NOT_CONVERGED);
  }
  return HZ_OK;
}

template int bicgstab_run<double>(hz_ctx, const SegHost&, const SellOp<double>&, const z_t*, z_t*,
                                  const KrylovCtl&, KrylovOut*, const std::string&);
template int bicgstab_run<float>(hz_ctx, const SegHost&, const SellOp<float>&, const c_t*, c_t*,
                                 const KrylovCtl&, KrylovOut*, const std::string&);
