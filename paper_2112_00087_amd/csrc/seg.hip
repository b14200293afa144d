// Segment layouts and segmented reductions shared by the solvers.
#include "ops.h"

namespace {

template <typename T>
__global__ void __launch_bounds__(kBlock) k_norm_part(Seg L, const cx<T>* __restrict__ x, double* part) {
  SumTile t = tile_of_sums(L);
  double q[1] = {norm2(ccast<double>(x[t.row]))};
  store_partials<1>(q, part, t);
}

__global__ void k_seg_fin1(Seg L, const double* part, double* out) {
  int s = blockIdx.x;
  double o[1];
  seg_sums<1>(L, part, s, o);
  if (threadIdx.x == 0) out[s] = o[0];
}

// r = f - A u (FP64), partial ||r||^2; per storage form F of A.
template <int F>
__global__ void __launch_bounds__(kBlock) k_true_resid(Seg L, SellOp<double> A, const z_t* __restrict__ f,
                                                       const z_t* __restrict__ u, z_t* __restrict__ r,
                                                       double* part) {
  SumTile t = prod_tile_sums<F>(L);
  double q[1] = {0.0};
  for_rows<F, true>(A, t, u, [=](int64_t row) { return f[row]; },
              [&](int64_t row, z_t y, z_t fv) {
                const z_t v = fv - y;
                if (r) r[row] = v;
                q[0] += norm2(v);
              });
  store_partials<1>(q, part, t);
}

int fetch_seg(hz_ctx ctx, const SegHost& S, const double* dev, std::vector<double>* out) {
  void* hp = nullptr;
  HZ_TRY(ctx_pinned(ctx, sizeof(double) * S.nseg, &hp));
  HZ_HIP(hipMemcpyAsync(hp, dev, sizeof(double) * S.nseg, hipMemcpyDeviceToHost, ctx->stream));
  HZ_HIP(hipStreamSynchronize(ctx->stream));
  out->assign(static_cast<double*>(hp), static_cast<double*>(hp) + S.nseg);
  return HZ_OK;
}

}  // namespace

template <typename T>
int seg_norm2_t(hz_ctx ctx, const SegHost& S, const cx<T>* x, std::vector<double>* out) {
  int rc = 0;
  DevBuf* part = ctx->buf("segn.part", sizeof(double) * S.nblk, &rc);
  if (rc) return rc;
  DevBuf* res = ctx->buf("segn.out", sizeof(double) * S.nseg, &rc);
  if (rc) return rc;
  k_norm_part<T><<<S.nblk, kBlock, 0, ctx->stream>>>(S.dev, x, part->as<double>());
  k_seg_fin1<<<S.nseg, kFinBlock, 0, ctx->stream>>>(S.dev, part->as<double>(), res->as<double>());
  HZ_HIP(hipGetLastError());
  return fetch_seg(ctx, S, res->as<double>(), out);
}
template int seg_norm2_t<double>(hz_ctx, const SegHost&, const z_t*, std::vector<double>*);
template int seg_norm2_t<float>(hz_ctx, const SegHost&, const c_t*, std::vector<double>*);

int true_residual(hz_ctx ctx, const SegHost& S, const SellOp<double>& A, const z_t* f, const z_t* u,
                  z_t* r, std::vector<double>* rr) {
  int rc = 0;
  const Seg& P = prod_seg(A, S.dev);
  DevBuf* part = ctx->buf("tres.part", sizeof(double) * P.nblk, &rc);
  if (rc) return rc;
  DevBuf* res = ctx->buf("tres.out", sizeof(double) * S.nseg, &rc);
  if (rc) return rc;
  HZ_BY_FORM(A, k_true_resid<F><<<P.nblk, kBlock, 0, ctx->stream>>>(P, A, f, u, r, part->as<double>()));
  k_seg_fin1<<<S.nseg, kFinBlock, 0, ctx->stream>>>(P, part->as<double>(), res->as<double>());
  HZ_HIP(hipGetLastError());
  return fetch_seg(ctx, S, res->as<double>(), rr);
}

int StatePoll::init(hz_ctx c, size_t nbytes) {
  ctx = c;
  bytes = nbytes;
  posted = 0;
  void* hp = nullptr;
  HZ_TRY(ctx_pinned(c, 2 * nbytes, &hp));
  host = static_cast<char*>(hp);
  for (hipEvent_t& e : c->poll_ev)
    if (!e) HZ_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  return HZ_OK;
}
int StatePoll::posted_one() {
  HZ_HIP(hipEventRecord(ctx->poll_ev[posted & 1], ctx->stream));
  ++posted;
  return HZ_OK;
}
int StatePoll::wait(int k) {
  HZ_HIP(hipEventSynchronize(ctx->poll_ev[k & 1]));
  return HZ_OK;
}

int PartBuf::init(hz_ctx ctx, const SegHost& S, const Seg& L, int nq, int consumers, const std::string& name) {
  int rc = 0;
  stepped = int64_t(L.nblk) * consumers > kMaxConsumed * S.nseg;
  DevBuf* b = ctx->buf(name, sizeof(double) * nq * size_t(L.nblk), &rc);
  if (rc) return rc;
  raw = b->as<double>();
  lay = L;
  part.nseg = S.nseg;
  part.p = raw;
  part.seg_blk = stepped ? S.zeros : L.seg_blk;
  part.nblk = stepped ? 0 : L.nblk;
  return HZ_OK;
}

int seg_upload(hz_ctx ctx, SegHost* S, const std::string& tag) {
  int rc = 0;
  // the segments tile the blocks (the finalize kernels rely on it)
  if (int(S->seg_blk.size()) != S->nseg + 1 || S->seg_blk.front() != 0 || S->seg_blk.back() != S->nblk)
    return hz_fail(HZ_ERR_INVALID, "segment table does not tile the %d blocks", S->nblk);
  std::vector<int> blk_seg(S->nblk);
  for (int s = 0; s < S->nseg; ++s)
    for (int b = S->seg_blk[s]; b < S->seg_blk[s + 1]; ++b) blk_seg[b] = s;
  DevBuf* a = ctx->buf(tag + ".blk_seg", sizeof(int) * S->nblk, &rc);
  if (rc) return rc;
  DevBuf* b = ctx->buf(tag + ".seg_blk", sizeof(int) * (S->nseg + 1), &rc);
  if (rc) return rc;
  HZ_HIP(hipMemcpy(a->p, blk_seg.data(), sizeof(int) * S->nblk, hipMemcpyHostToDevice));
  HZ_HIP(hipMemcpy(b->p, S->seg_blk.data(), sizeof(int) * (S->nseg + 1), hipMemcpyHostToDevice));
  // vector layouts: one tile per block, and runs of tiles of one segment
  auto layout = [&](int per, const std::string& name, Seg* V) -> int {
    std::vector<int> vseg, vrow, vblk(1, 0);
    for (int s = 0; s < S->nseg; ++s) {
      for (int b = S->seg_blk[s]; b < S->seg_blk[s + 1]; b += per) {
        vseg.push_back(s);
        vrow.push_back(b * kBlock);
      }
      vblk.push_back(int(vseg.size()));
    }
    vrow.push_back(S->nblk * kBlock);
    const size_t nv = vseg.size();
    DevBuf* vb = ctx->buf(tag + name, sizeof(int) * (nv + (nv + 1) + (S->nseg + 1)), &rc);
    if (rc) return rc;
    int* vp = vb->as<int>();
    HZ_HIP(hipMemcpy(vp, vseg.data(), sizeof(int) * nv, hipMemcpyHostToDevice));
    HZ_HIP(hipMemcpy(vp + nv, vrow.data(), sizeof(int) * (nv + 1), hipMemcpyHostToDevice));
    HZ_HIP(hipMemcpy(vp + 2 * nv + 1, vblk.data(), sizeof(int) * (S->nseg + 1), hipMemcpyHostToDevice));
    V->nseg = S->nseg;
    V->nblk = int(nv);
    V->nrows = S->nrows;
    V->blk_seg = vp;
    V->blk_row = vp + nv;
    V->seg_blk = vp + 2 * nv + 1;
    return HZ_OK;
  };
  const int per = std::max(1, ceil_div(S->nblk, 1024));
  HZ_TRY(layout(1, ".vec", &S->vec));
  S->vec.xcd_runs = 1;
  if (per > 1) HZ_TRY(layout(per, ".vecr", &S->vec_runs));
  else S->vec_runs = S->vec;
  S->vec_runs.xcd_runs = 0;
  DevBuf* zb = ctx->buf(tag + ".zeros", sizeof(int) * (S->nseg + 1), &rc);
  if (rc) return rc;
  const std::vector<int> zeros(S->nseg + 1, 0);
  HZ_HIP(hipMemcpy(zb->p, zeros.data(), sizeof(int) * (S->nseg + 1), hipMemcpyHostToDevice));
  S->zeros = zb->as<int>();
  S->dev.nseg = S->nseg;
  S->dev.nblk = S->nblk;
  S->dev.nrows = S->nrows;
  S->dev.blk_seg = a->as<int>();
  S->dev.seg_blk = b->as<int>();
  return HZ_OK;
}
