// Tensor form of the operator: which meshes have it, its tables, and the
// wave layout of its product (tensor.h).
#include <algorithm>
#include <cstdlib>

#include "ops.h"

namespace {

// 1-D rows of node i on the grid c[0..n): linear elements, exact integrals
__device__ __forceinline__ TzAxis axis_row(const double* c, int n, int i, z_t corner_lo, z_t corner_hi) {
  const double hl = i > 0 ? c[i] - c[i - 1] : 0.0, hr = i + 1 < n ? c[i + 1] - c[i] : 0.0;
  TzAxis a;
  a.ml = hl / 6.0;
  a.mh = hr / 6.0;
  a.md = (hl + hr) / 3.0;
  a.kl = i > 0 ? -1.0 / hl : 0.0;
  a.kh = i + 1 < n ? -1.0 / hr : 0.0;
  a.kd = -(a.kl + a.kh);
  a.ki = 0.0;
  a.pad = 0.0;
  if (i == 0) {
    a.kd += corner_lo.re;
    a.ki += corner_lo.im;
  }
  if (i == n - 1) {
    a.kd += corner_hi.re;
    a.ki += corner_hi.im;
  }
  return a;
}
__device__ __forceinline__ TzAxis minus_mass(TzAxis a, double m) {
  a.kl = fma(-m, a.ml, a.kl);
  a.kd = fma(-m, a.md, a.kd);
  a.kh = fma(-m, a.mh, a.kh);
  return a;
}

// Axis tables (x, y with K - m M, z) and the line table of one box, and k^2; c
// holds the axes' coordinates one after the other.
__global__ void k_tz_tables(TzSeg S, const double* __restrict__ c, TzCorner w, double m, double k2,
                            TzAxis* __restrict__ tab, TzLine* __restrict__ dx, TzLine* __restrict__ lt,
                            double* __restrict__ k2_out) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  if (t == 0) *k2_out = k2;
  const double *cx = c, *cy = c + S.nx, *cz = c + S.nx + S.ny;
  const int na = S.nx + S.ny + S.nz;
  if (t < S.nx) {
    const TzAxis a = axis_row(cx, S.nx, t, w.v[0], w.v[1]);
    tab[S.xt + t] = a;
    dx[S.xt + t] = TzLine{a.kd, a.md, a.ki, 0.0};
  } else if (t < S.nx + S.ny) {
    const int j = t - S.nx;
    tab[S.yt + j] = minus_mass(axis_row(cy, S.ny, j, w.v[2], w.v[3]), m);
  } else if (t < na) {
    const int k = t - S.nx - S.ny;
    tab[S.zt + k] = axis_row(cz, S.nz, k, w.v[4], w.v[5]);
  } else if (t < na + S.ny * S.nz) {
    const int l = t - na, j = l % S.ny, k = l / S.ny;
    const TzAxis y = minus_mass(axis_row(cy, S.ny, j, w.v[2], w.v[3]), m);
    const TzAxis z = axis_row(cz, S.nz, k, w.v[4], w.v[5]);
    lt[S.lt + l] = TzLine{y.md * z.md, fma(y.kd, z.md, y.md * z.kd), fma(y.ki, z.md, y.md * z.ki), 0.0};
  }
}

// Axis rows without frequency and walls (the sweep adds them per column).
__global__ void k_tz_axes(TzSeg S, const double* __restrict__ c, TzAxis* __restrict__ tab) {
  const int t = blockIdx.x * kBlock + threadIdx.x;
  const z_t z = {0.0, 0.0};
  if (t < S.nx) tab[t] = axis_row(c, S.nx, t, z, z);
  else if (t < S.nx + S.ny) tab[t] = axis_row(c + S.nx, S.ny, t - S.nx, z, z);
  else if (t < S.nx + S.ny + S.nz) tab[t] = axis_row(c + S.nx + S.ny, S.nz, t - S.nx - S.ny, z, z);
}

// diag(A) and its reciprocal of one box's rows (1 on padding rows)
__global__ void k_tz_diag(TzSeg S, const TzAxis* __restrict__ tab, const TzLine* __restrict__ lt,
                          const double* __restrict__ ed, double k2, z_t* __restrict__ d, z_t* __restrict__ dinv) {
  const int64_t r = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (r >= S.nrows) return;
  const int64_t row = S.row0 + r;
  z_t v = {1.0, 0.0}, vi = {1.0, 0.0};
  if (r < S.n) {
    const int i = int(r % S.nx);
    const TzAxis a = tab[S.xt + i];
    const TzLine l = lt[S.lt + r / S.nx];
    v = z_t{fma(a.kd, l.a, a.md * l.b), fma(a.ki, l.a, a.md * l.c)};
    if (ed) v.im = fma(k2, ed[row], v.im);
    vi = crecip(v);
  }
  d[row] = v;
  dinv[row] = vi;
}

// Diagonal of sum_e eta_e M_e on one box: each of a node's elements adds
// eta_e hx hy hz / 27.
__global__ void k_tz_eta_diag(TzSeg S, const double* __restrict__ c, const double* __restrict__ eta,
                              double* __restrict__ ed) {
  const int64_t r = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (r >= S.nrows) return;
  double v = 0.0;
  if (r < S.n) {
    const int i = int(r % S.nx), j = int(r / S.nx % S.ny), k = int(r / (int64_t(S.nx) * S.ny));
    const double *cx = c, *cy = c + S.nx, *cz = c + S.nx + S.ny;
    for (int ek = k - 1; ek <= k; ++ek)
      for (int ej = j - 1; ej <= j; ++ej)
        for (int ei = i - 1; ei <= i; ++ei)
          if (ei >= 0 && ei < S.nx - 1 && ej >= 0 && ej < S.ny - 1 && ek >= 0 && ek < S.nz - 1)
            v += eta[S.e0 + (int64_t(ek) * (S.ny - 1) + ej) * (S.nx - 1) + ei] * (cx[ei + 1] - cx[ei]) *
                 (cy[ej + 1] - cy[ej]) * (cz[ek + 1] - cz[ek]);
  }
  ed[S.row0 + r] = v / 27.0;
}

template <typename V>
int put(hz_ctx ctx, DevBuf& b, const V* src, size_t count) {
  const size_t before = b.bytes;
  HZ_TRY(b.ensure(sizeof(V) * std::max<size_t>(count, 1)));
  ctx->dev_bytes += int64_t(b.bytes) - int64_t(before);
  if (count && src) HZ_HIP(hipMemcpy(b.p, src, sizeof(V) * count, hipMemcpyHostToDevice));
  return HZ_OK;
}

}  // namespace

// The mesh has no Dirichlet source, the box is a tensor-product grid in its
// own numbering, its elements are the grid's cells in order, and each of its six walls is either covered
// once by faces of one tag or not at all.
bool tensor_detect(const HostAsm& a, const int32_t elems[3], TensorGrid* g) {
  const int64_t nx = elems[0], ny = elems[1], nz = elems[2];
  if (a.npe != 8 || !a.dir.empty() || nx < 1 || ny < 1 || nz < 1) return false;
  const int64_t NX = nx + 1, NY = ny + 1, NZ = nz + 1;
  if (int64_t(a.n) != NX * NY * NZ || int64_t(a.ne) != nx * ny * nz) return false;
  const int64_t cnt[3] = {NX, NY, NZ}, step[3] = {1, NX, NX * NY};
  for (int d = 0; d < 3; ++d) {
    g->c[d].resize(cnt[d]);
    for (int64_t i = 0; i < cnt[d]; ++i) g->c[d][i] = a.xyz[i * step[d] * 3 + d];
    for (int64_t i = 0; i + 1 < cnt[d]; ++i)
      if (!(g->c[d][i + 1] > g->c[d][i])) return false;
  }
  int64_t r = 0;
  for (int64_t k = 0; k < NZ; ++k)
    for (int64_t j = 0; j < NY; ++j)
      for (int64_t i = 0; i < NX; ++i, ++r)
        if (a.xyz[r * 3] != g->c[0][i] || a.xyz[r * 3 + 1] != g->c[1][j] || a.xyz[r * 3 + 2] != g->c[2][k])
          return false;
  int64_t e = 0;
  for (int64_t k = 0; k < nz; ++k)
    for (int64_t j = 0; j < ny; ++j)
      for (int64_t i = 0; i < nx; ++i, ++e)
        for (int l = 0; l < 8; ++l)
          if (a.hex[e * 8 + l] != (i + (l & 1)) + NX * ((j + ((l >> 1) & 1)) + NY * (k + ((l >> 2) & 1)))) return false;
  // walls: each face's four nodes are one cell of one wall, in tensor order
  // (the pairs 0-3 and 1-2 are its diagonals); counted once per cell
  const int64_t el[3] = {nx, ny, nz};
  std::vector<std::vector<uint8_t>> seen(6);
  int64_t left[6];
  for (int w = 0; w < 6; ++w) {
    const int d = w / 2, u = d == 0 ? 1 : 0, v = d == 2 ? 1 : 2;
    seen[w].assign(el[u] * el[v], 0);
    left[w] = el[u] * el[v];
    g->tag[w] = -1;
  }
  for (int64_t f = 0; f < a.nb; ++f) {
    int64_t lo[3] = {INT64_MAX, INT64_MAX, INT64_MAX}, hi[3] = {-1, -1, -1}, s03 = 0, s12 = 0;
    for (int l = 0; l < 4; ++l) {
      const int64_t v = a.bface[f * 4 + l];
      const int64_t p[3] = {v % NX, v / NX % NY, v / (NX * NY)};
      for (int d = 0; d < 3; ++d) {
        lo[d] = std::min(lo[d], p[d]);
        hi[d] = std::max(hi[d], p[d]);
      }
      (l == 0 || l == 3 ? s03 : s12) += v;
    }
    if (s03 != s12) return false;
    for (int l = 0; l < 4; ++l)
      for (int o = 0; o < l; ++o)
        if (a.bface[f * 4 + l] == a.bface[f * 4 + o]) return false;
    int d = -1;
    for (int t = 0; t < 3; ++t) {
      if (hi[t] == lo[t]) {
        if (d >= 0) return false;
        d = t;
      } else if (hi[t] != lo[t] + 1) {
        return false;
      }
    }
    if (d < 0 || (lo[d] != 0 && lo[d] != el[d])) return false;
    const int w = 2 * d + (lo[d] != 0), u = d == 0 ? 1 : 0, v = d == 2 ? 1 : 2;
    uint8_t& cell = seen[w][lo[u] + el[u] * lo[v]];
    if (cell++) return false;
    if (g->tag[w] >= 0 && g->tag[w] != a.btag[f]) return false;
    g->tag[w] = a.btag[f];
    --left[w];
  }
  for (int w = 0; w < 6; ++w)
    if (g->tag[w] >= 0 && left[w] != 0) return false;
  return true;
}

// Wave grid of one box.
void tensor_layout(const int nodes[3], TzSeg* S) {
  S->nx = nodes[0];
  S->ny = nodes[1];
  S->nz = nodes[2];
  S->njb = ceil_div(S->ny, kTzJ);
  S->nxc = ceil_div(S->nx, kTzOut);
  S->nzc = ceil_div(S->nz, kTzZ);
  S->nblk = ceil_div(int64_t(S->njb) * S->nxc * S->nzc, kBlock / kWave);
}

int tensor_build(hz_ctx ctx, const std::vector<TensorGrid>& grids, const std::vector<int64_t>& row0,
                 const std::vector<int64_t>& nrows, const std::string& name, TensorDev* D) {
  const int ns = int(grids.size());
  D->segs.assign(ns, TzSeg{});
  D->cat.assign(ns, 0);
  std::vector<double> c;
  int tab = 0, lines = 0, blk = 0;
  int64_t rows = 0, e0 = 0;
  for (int s = 0; s < ns; ++s) {
    TzSeg& S = D->segs[s];
    const int nodes[3] = {int(grids[s].c[0].size()), int(grids[s].c[1].size()), int(grids[s].c[2].size())};
    tensor_layout(nodes, &S);
    S.n = nodes[0] * nodes[1] * nodes[2];
    S.inv_nx = 1.0 / nodes[0];
    S.row0 = int(row0[s]);
    S.nrows = int(nrows[s]);
    S.blk0 = blk;
    blk += S.nblk;
    S.xt = tab;
    S.yt = tab + nodes[0];
    S.zt = tab + nodes[0] + nodes[1];
    tab += nodes[0] + nodes[1] + nodes[2];
    S.lt = lines;
    lines += nodes[1] * nodes[2];
    S.e0 = int(e0);
    e0 += int64_t(nodes[0] - 1) * (nodes[1] - 1) * (nodes[2] - 1);
    D->cat[s] = int64_t(c.size());
    for (int d = 0; d < 3; ++d) c.insert(c.end(), grids[s].c[d].begin(), grids[s].c[d].end());
    rows = std::max(rows, row0[s] + nrows[s]);
  }
  HZ_TRY(put(ctx, D->coord, c.data(), c.size()));
  HZ_TRY(put<TzAxis>(ctx, D->tab, nullptr, tab));
  HZ_TRY(put<TzLine>(ctx, D->dx, nullptr, tab));
  HZ_TRY(put<TzLine>(ctx, D->lt, nullptr, lines));
  HZ_TRY(put(ctx, D->dsegs, D->segs.data(), D->segs.size()));
  HZ_TRY(put<double>(ctx, D->k2, nullptr, 1));
  D->lay.nseg = ns;
  D->lay.nblk = blk;
  D->lay.nrows = rows;
  D->lay.seg_blk.assign(1, 0);
  for (const TzSeg& S : D->segs) D->lay.seg_blk.push_back(S.blk0 + S.nblk);
  return seg_upload(ctx, &D->lay, name);
}

int tensor_tables(hz_ctx ctx, TensorDev* D, const std::vector<TzCorner>& corners, double m, double k2) {
  for (size_t s = 0; s < D->segs.size(); ++s) {
    const TzSeg& S = D->segs[s];
    const int count = S.nx + S.ny + S.nz + S.ny * S.nz;
    k_tz_tables<<<ceil_div(count, kBlock), kBlock, 0, ctx->stream>>>(
        S, D->coord.as<double>() + D->cat[s], corners[s], m, k2, D->tab.as<TzAxis>(), D->dx.as<TzLine>(),
        D->lt.as<TzLine>(), D->k2.as<double>());
  }
  HZ_HIP(hipGetLastError());
  return HZ_OK;
}

int tensor_axes(hz_ctx ctx, const TensorDev& D, DevBuf* tab) {
  const TzSeg& S = D.segs[0];
  const int count = S.nx + S.ny + S.nz;
  HZ_TRY(tab->ensure(sizeof(TzAxis) * count));
  k_tz_axes<<<ceil_div(count, kBlock), kBlock, 0, ctx->stream>>>(S, D.coord.as<double>(), tab->as<TzAxis>());
  HZ_HIP(hipGetLastError());
  return HZ_OK;
}

int tensor_diag(hz_ctx ctx, const TensorDev& D, double k2, z_t* d, z_t* dinv) {
  for (const TzSeg& S : D.segs)
    k_tz_diag<<<ceil_div(S.nrows, kBlock), kBlock, 0, ctx->stream>>>(S, D.tab.as<TzAxis>(), D.lt.as<TzLine>(),
                                                                    D.have_eta ? D.ed.as<double>() : nullptr, k2, d, dinv);
  HZ_HIP(hipGetLastError());
  return HZ_OK;
}

int tensor_eta(hz_ctx ctx, TensorDev* D, const double* eta_host, int64_t count) {
  D->have_eta = false;
  if (!eta_host) return HZ_OK;
  HZ_TRY(put(ctx, D->eta, eta_host, size_t(count)));
  HZ_TRY(put<double>(ctx, D->ed, nullptr, size_t(D->lay.nrows)));
  for (size_t s = 0; s < D->segs.size(); ++s)
    k_tz_eta_diag<<<ceil_div(D->segs[s].nrows, kBlock), kBlock, 0, ctx->stream>>>(
        D->segs[s], D->coord.as<double>() + D->cat[s], D->eta.as<double>(), D->ed.as<double>());
  HZ_HIP(hipGetLastError());
  D->have_eta = true;
  return HZ_OK;
}

TzOp tensor_op(const TensorDev& D, bool scale) {
  TzOp o;
  o.on = D.have_eta ? 2 : 1;
  o.scale = scale;
  o.nseg = int(D.segs.size());
  o.s0 = D.segs[0];
  o.segs = D.dsegs.as<TzSeg>();
  o.tab = D.tab.as<TzAxis>();
  o.dx = D.dx.as<TzLine>();
  o.lt = D.lt.as<TzLine>();
  o.eta = D.have_eta ? D.eta.as<double>() : nullptr;
  o.ed = D.have_eta ? D.ed.as<double>() : nullptr;
  o.k2 = D.k2.as<double>();
  o.lp = D.lay.dev;
  return o;
}
