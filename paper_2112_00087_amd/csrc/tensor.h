// Separable ("tensor") form of the operator on a box whose nodes lie on a
// tensor-product grid (x_i, y_j, z_k, any spacings).
//
// There trilinear elements give K, M and the wall masses as sums of
// Kronecker products of the axes' tridiagonal 1-D matrices, and a wall's
// Robin term i k beta B0_w adds to one corner entry of its axis' 1-D
// stiffness (the same for a Schwarz interface term alpha M_G), so
//     A = Kx (x) My (x) Mz + Mx (x) (Ky - m My) (x) Mz + Mx (x) My (x) Kz
// with complex first and last diagonal entries in Kx, Ky, Kz.  The product
//     a = Mx x, b = Kx x;  p = My a, q = My b + (Ky - m My) a;  y = Mz q + Kz p
// streams no matrix: it reads x and writes y, and its coefficients are three
// short tables.  An absorption field adds i k^2 sum_e eta_e M_e with the
// element masses in the same factored form (8 bytes per element).  (A box
// with a Dirichlet source keeps the stored forms, whose eliminated rows and
// columns are zeros of the matrix.)
//
// One wave takes 62 consecutive nodes along x (its two outer lanes only load
// the neighbours), kTzJ lines along y and kTzZ planes along z, and issues
// all its (kTzJ + 2)(kTzZ + 2) line loads before the first use: at these
// sizes a product is bound by latency and by the vectors' bandwidth, not by
// its FP64 instructions.  The stages run z, y, x: the z and y sums are
// lane-local with wave-uniform coefficients (scalar loads), and the x stage,
// which needs the neighbour lanes, then runs once per output row instead of
// once per loaded line (two shifted values per row).  Measured, us a complex128
// product, stencil form -> tensor form: 21x13x11 nodes 8.4 -> 3.8 (latency),
// 81x49x41 17 -> 4.8, 161x97x81 68 -> 10.9 (40 MB of vectors in the Infinity
// Cache, 3.7 TB/s), 201x121x101 128 -> 18.5; with an absorption field (complex
// form before) 81x49x41 7.1, 161x97x81 15.7.  Against it: 2,048 waves marching
// along z, with D^-1 applied inside, 23 us at 161x97x81 (a serial chain of
// plane loads).
//
// All arithmetic is FP64 whatever the vectors' type.  The right-Jacobi
// scaling is not part of the product: the solvers hand in D^-1-scaled
// vectors (tz_pre), so their iterates are the solution itself.
#pragma once

#include "krylov.h"

constexpr int kTzOut = kWave - 2;    // nodes along x that a wave writes
constexpr int kTzJ = 2;              // lines along y per wave
constexpr int kTzZ = 2;              // planes along z per wave

// Axis table entry of a node: mass and stiffness rows (below, diagonal,
// above) and the imaginary part of the stiffness diagonal (wall nodes only).
// y tables hold K - m M in place of K.
struct TzAxis {
  double ml, md, mh, kl, kd, kh, ki, pad;
};
// diag(A)_row = kd c1 + md c2 + i (ki c1 + md ci) from an entry (kd, md, ki)
// per x node and an entry (c1, c2, ci) per line (j, k).
struct TzLine {
  double a, b, c, pad;
};
// x loaded as FP64
template <typename T> __device__ __forceinline__ z_t tz_ld(const cx<T>* p) { return ccast<double>(*p); }

// Wave-uniform table entries by scalar loads (the tables do not change while
// a kernel that reads them runs).
template <typename V>
using TzConst = const __attribute__((address_space(4))) V*;
template <typename V> __device__ __forceinline__ TzConst<V> tz_const(const V* p) {
  return (TzConst<V>)(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ TzAxis tz_uniform(const TzAxis* p, int at) {
  TzConst<double> q = tz_const(reinterpret_cast<const double*>(p + at));
  return TzAxis{q[0], q[1], q[2], q[3], q[4], q[5], q[6], 0.0};
}

// The value of the lane to the left (right); 0 in the wave's first (last)
// lane.  Data-parallel-primitive moves (wave_shr:1, wave_shl:1) run on the
// vector pipe of the wave's own SIMD; a shuffle would queue on the LDS pipe
// that the whole CU shares.
template <int CTRL>
__device__ __forceinline__ double tz_shift(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double tz_left(double v) { return tz_shift<0x138>(v); }
__device__ __forceinline__ double tz_right(double v) { return tz_shift<0x130>(v); }

// acc += c v (c real)
__device__ __forceinline__ void tz_add(z_t& acc, double c, z_t v) {
  acc.re = fma(c, v.re, acc.re);
  acc.im = fma(c, v.im, acc.im);
}
// acc += i c v (c real)
__device__ __forceinline__ void tz_addi(z_t& acc, double c, z_t v) {
  acc.re = fma(-c, v.im, acc.re);
  acc.im = fma(c, v.re, acc.im);
}
__device__ __forceinline__ z_t tz_mul(double c, z_t v) { return z_t{c * v.re, c * v.im}; }

// The rows of one wave.  EXT: with an absorption field.  aux(row) loads what
// the epilogue needs besides the product; epi(row, y, aux) takes the finished
// row.
template <bool EXT, typename T, class Aux, class Epi>
__device__ __forceinline__ void tz_wave(const TzOp& A, const TzSeg& S, int wave, const cx<T>* __restrict__ x, Aux aux,
                                        Epi epi) {
  const int lane = threadIdx.x & (kWave - 1);
  const int jb = wave % S.njb, rem = wave / S.njb;
  const int xc = rem % S.nxc, zc = rem / S.nxc;
  const int NX = S.nx, NY = S.ny, NZ = S.nz;
  const int i = xc * kTzOut + lane - 1;
  const bool inx = i >= 0 && i < NX;
  const bool outx = inx && lane >= 1 && lane <= kTzOut;
  const int j0 = jb * kTzJ, z0 = zc * kTzZ;
  const int64_t plane = int64_t(NX) * NY;
  const int64_t at0 = S.row0 + (z0 - 1) * plane + int64_t(j0 - 1) * NX + i;   // first line read
  // line t of plane c is inside the box (wave-uniform)
  auto in_j = [&](int t) { return j0 - 1 + t >= 0 && j0 - 1 + t < NY; };
  auto in_z = [&](int c) { return z0 - 1 + c >= 0 && z0 - 1 + c < NZ; };
  auto row_of = [&](int c, int t) { return at0 + c * plane + int64_t(t) * NX; };

  z_t v[kTzZ + 2][kTzJ + 2];
#pragma unroll
  for (int c = 0; c < kTzZ + 2; ++c)
#pragma unroll
    for (int t = 0; t < kTzJ + 2; ++t) {
      v[c][t] = z_t{0.0, 0.0};
      if (in_z(c) && in_j(t) && inx) v[c][t] = tz_ld(x + row_of(c, t));
    }
  TzAxis cx_ = {};
  if (inx) cx_ = A.tab[S.xt + i];
  double eta[EXT ? kTzZ + 1 : 1][EXT ? kTzJ + 1 : 1];   // element layer z0 - 1 + c, element line j0 - 1 + t
  if constexpr (EXT) {
#pragma unroll
    for (int c = 0; c < kTzZ + 1; ++c)
#pragma unroll
      for (int t = 0; t < kTzJ + 1; ++t) {
        const int ez = z0 - 1 + c, ey = j0 - 1 + t;
        eta[c][t] = 0.0;
        if (ez >= 0 && ez < NZ - 1 && ey >= 0 && ey < NY - 1 && i >= 0 && i < NX - 1)
          eta[c][t] = A.eta[S.e0 + (int64_t(ez) * (NY - 1) + ey) * (NX - 1) + i];
      }
  }
  decltype(aux(int64_t(0))) ax[kTzZ][kTzJ];
#pragma unroll
  for (int c = 0; c < kTzZ; ++c)
#pragma unroll
    for (int t = 0; t < kTzJ; ++t)
      if (in_z(c + 1) && in_j(t + 1) && outx) ax[c][t] = aux(row_of(c + 1, t + 1));
  double k2 = 0.0;
  if constexpr (EXT) k2 = *tz_const(A.k2);
  TzAxis cy[kTzJ], cz[kTzZ];
#pragma unroll
  for (int t = 0; t < kTzJ; ++t) cy[t] = tz_uniform(A.tab, S.yt + (j0 + t < NY ? j0 + t : NY - 1));
#pragma unroll
  for (int c = 0; c < kTzZ; ++c) cz[c] = tz_uniform(A.tab, S.zt + (z0 + c < NZ ? z0 + c : NZ - 1));

#pragma unroll
  for (int c = 0; c < kTzZ; ++c) {
    if (!in_z(c + 1)) break;
    const TzAxis& Z = cz[c];
    z_t a[kTzJ + 2], b[kTzJ + 2];   // Mz x, Kz x on the lines
#pragma unroll
    for (int t = 0; t < kTzJ + 2; ++t) {
      a[t] = tz_mul(Z.md, v[c + 1][t]);
      tz_add(a[t], Z.ml, v[c][t]);
      tz_add(a[t], Z.mh, v[c + 2][t]);
      b[t] = tz_mul(Z.kd, v[c + 1][t]);
      tz_add(b[t], Z.kl, v[c][t]);
      tz_add(b[t], Z.kh, v[c + 2][t]);
      tz_addi(b[t], Z.ki, v[c + 1][t]);
    }
#pragma unroll
    for (int t = 0; t < kTzJ; ++t) {
      const TzAxis& Y = cy[t];
      z_t p = tz_mul(Y.md, a[t + 1]), q = tz_mul(Y.md, b[t + 1]);   // (My Mz) x; (My Kz + (Ky - m My) Mz) x
      tz_add(p, Y.ml, a[t]);
      tz_add(p, Y.mh, a[t + 2]);
      tz_add(q, Y.ml, b[t]);
      tz_add(q, Y.mh, b[t + 2]);
      tz_add(q, Y.kd, a[t + 1]);
      tz_add(q, Y.kl, a[t]);
      tz_add(q, Y.kh, a[t + 2]);
      tz_addi(q, Y.ki, a[t + 1]);
      // x stage: each node forms its share in its neighbours' rows (the 1-D matrices are symmetric)
      z_t own = tz_mul(cx_.md, q), to_r = tz_mul(cx_.mh, q), to_l = tz_mul(cx_.ml, q);
      tz_add(own, cx_.kd, p);
      tz_addi(own, cx_.ki, p);
      tz_add(to_r, cx_.kh, p);
      tz_add(to_l, cx_.kl, p);
      if constexpr (EXT) {
        // s(ez, ey): the node's share of the four elements around its line,
        // summed along z and y; al = sum eta s over the elements to the
        // right of the node, ar over those to its left
        z_t al = {0.0, 0.0}, ar = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 2; ++e) {        // element layer below, above
          z_t h[3];
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            const z_t far = e ? v[c + 2][t + u] : v[c][t + u];
            const double wz = e ? Z.mh : Z.ml;
            h[u] = tz_mul(wz, z_t{fma(2.0, v[c + 1][t + u].re, far.re), fma(2.0, v[c + 1][t + u].im, far.im)});
          }
#pragma unroll
          for (int g = 0; g < 2; ++g) {      // element line below, above
            const z_t far = g ? h[2] : h[0];
            const double wy = g ? Y.mh : Y.ml;
            const z_t sv = tz_mul(wy, z_t{fma(2.0, h[1].re, far.re), fma(2.0, h[1].im, far.im)});
            const double er = eta[c + e][t + g], el = tz_left(er);
            tz_add(al, er, sv);
            tz_add(ar, el, sv);
          }
        }
        const double wr = k2 * cx_.mh, wl = k2 * cx_.ml;
        tz_addi(own, 2.0 * wr, al);
        tz_addi(own, 2.0 * wl, ar);
        tz_addi(to_r, wr, al);
        tz_addi(to_l, wl, ar);
      }
      z_t y = {own.re + (tz_left(to_r.re) + tz_right(to_l.re)), own.im + (tz_left(to_r.im) + tz_right(to_l.im))};
      if (in_j(t + 1) && outx) epi(row_of(c + 1, t + 1), y, ax[c][t]);
    }
  }
}

__device__ __forceinline__ TzSeg tz_seg(const TzOp& Z, int seg) {
  TzSeg S = Z.s0;
  if (Z.nseg > 1) {
    TzConst<int> q = tz_const(reinterpret_cast<const int*>(Z.segs + seg));
    int* d = reinterpret_cast<int*>(&S);
#pragma unroll
    for (int u = 0; u < int(sizeof(TzSeg) / sizeof(int)); ++u) d[u] = q[u];
  }
  return S;
}

// diag(A) at a row of box S (1 on padding rows), from the tables: two 32-byte
// entries, the x nodes' consecutive over the lanes and the line's mostly
// shared by the wave, instead of 16 bytes of a stored diagonal per row and
// pass.
__device__ __forceinline__ z_t tz_diag_at(const TzOp& A, const TzSeg& S, int64_t row) {
  const int r = int(row - S.row0);
  if (r >= S.n) return z_t{1.0, 0.0};
  int l = int(double(r) * S.inv_nx);   // r / nx, then put right
  int i = r - l * S.nx;
  if (i < 0) {
    --l;
    i += S.nx;
  } else if (i >= S.nx) {
    ++l;
    i -= S.nx;
  }
  const TzLine d = A.dx[S.xt + i], c = A.lt[S.lt + l];
  z_t v = {fma(d.a, c.a, d.b * c.b), fma(d.c, c.a, d.b * c.c)};
  if (A.ed) v.im = fma(*tz_const(A.k2), A.ed[row], v.im);
  return v;
}
// 1 / v: the hardware estimate and two Newton steps (full FP64 precision)
__device__ __forceinline__ double tz_rcp(double v) {
  double r = __builtin_amdgcn_rcp(v);
  r = fma(r, fma(-v, r, 1.0), r);
  return fma(r, fma(-v, r, 1.0), r);
}
// y + a x and y - a x: in the tensor form with one rounding per term, in the
// stored forms as these expressions always were compiled there.
template <int F>
__device__ __forceinline__ z_t tz_axpy(z_t a, z_t x, z_t y) {
  if constexpr (F == kFormTensor || F == kFormTensorExt)
    return z_t{fma(a.re, x.re, fma(-a.im, x.im, y.re)), fma(a.re, x.im, fma(a.im, x.re, y.im))};
  else
    return y + a * x;
}
template <int F>
__device__ __forceinline__ z_t tz_axmy(z_t a, z_t x, z_t y) {
  if constexpr (F == kFormTensor || F == kFormTensorExt)
    return z_t{fma(-a.re, x.re, fma(a.im, x.im, y.re)), fma(-a.re, x.im, fma(-a.im, x.re, y.im))};
  else
    return y - a * x;
}

// D^-1 v and D v of the right-Jacobi operator A D^-1 in the tensor form; in
// the stored forms D is folded into the values and both are v itself.
template <int F>
__device__ __forceinline__ z_t tz_pre(const TzOp& A, const TzSeg& S, int64_t row, z_t v) {
  if constexpr (F == kFormTensor || F == kFormTensorExt) {
    if (!A.scale) return v;
    const z_t d = tz_diag_at(A, S, row);
    const double r = tz_rcp(fma(d.re, d.re, d.im * d.im));
    return z_t{r * fma(v.re, d.re, v.im * d.im), r * fma(v.im, d.re, -v.re * d.im)};
  } else {
    return v;
  }
}
template <int F>
__device__ __forceinline__ z_t tz_unpre(const TzOp& A, const TzSeg& S, int64_t row, z_t v) {
  if constexpr (F == kFormTensor || F == kFormTensorExt) {
    if (!A.scale) return v;
    return tz_diag_at(A, S, row) * v;
  } else {
    return v;
  }
}

// All rows of a product kernel's block, in any storage form: aux(row) and
// epi(row, y, aux(row)) with y = (A x)[row] rounded to the vectors' type.
// aux is what the epilogue reads besides y: the tensor form loads it ahead of
// the product's stages, the stored forms behind the row sum (AUX_FIRST: ahead
// of it), whose registers the product loop needs.
template <int F, bool AUX_FIRST = false, typename T, class Aux, class Epi>
__device__ __forceinline__ void for_rows(const SellOp<T>& A, const Tile& t, const cx<T>* __restrict__ x, Aux aux,
                                         Epi epi) {
  if constexpr (F == kFormTensor || F == kFormTensorExt) {
    const TzOp& Z = A.tz;
    const TzSeg S = tz_seg(Z, t.seg);
    const int w = __builtin_amdgcn_readfirstlane(int((t.tile - S.blk0) * (kBlock / kWave) + threadIdx.x / kWave));
    if (w < S.njb * S.nxc * S.nzc)
      tz_wave<F == kFormTensorExt>(Z, S, w, x, aux, [&](int64_t row, z_t y, auto a) { epi(row, ccast<T>(y), a); });
    if (t.tile == S.blk0 + S.nblk - 1) {   // padding rows of the segment stay zero
      const int64_t r = int64_t(S.row0) + S.n + threadIdx.x;
      if (r < int64_t(S.row0) + S.nrows) epi(r, cx<T>{T(0), T(0)}, aux(r));
    }
  } else {
    if constexpr (AUX_FIRST) {
      const auto a = aux(t.row);
      epi(t.row, sell_row_form<F>(A, t.row, x), a);
    } else {
      const cx<T> y = sell_row_form<F>(A, t.row, x);
      epi(t.row, y, aux(t.row));
    }
  }
}

// Tile of a product kernel: 256 rows in the stored forms; in the tensor form
// a block of four waves of tz_wave (t.row is not used), each XCD taking one
// contiguous range of blocks.
template <int F>
__device__ __forceinline__ Tile prod_tile(const Seg& L) {
  if constexpr (F == kFormTensor || F == kFormTensorExt) {
    Tile t;
    t.tile = xcd_tile(blockIdx.x, gridDim.x);
    t.seg = L.nseg == 1 ? 0 : L.blk_seg[t.tile];
    t.row = 0;
    return t;
  } else {
    return tile_of(L);
  }
}
template <int F>
__device__ __forceinline__ SumTile prod_tile_sums(const Seg& L) {
  SumTile t;
  static_cast<Tile&>(t) = prod_tile<F>(L);
  if (threadIdx.x == 0) *block_wave_count() = 0;
  __syncthreads();
  return t;
}

// Box of a tile's segment (unused in the stored forms).
template <int F>
__device__ __forceinline__ TzSeg form_seg(const TzOp& A, const Tile& t) {
  if constexpr (F == kFormTensor || F == kFormTensorExt) return tz_seg(A, t.seg);
  return TzSeg{};
}

// Layout that a product with A runs in: the tensor form's own blocks, or the rows'.
template <typename T>
inline const Seg& prod_seg(const SellOp<T>& A, const Seg& L) { return A.tz.on ? A.tz.lp : L; }

// Run the statement with F set for a vector kernel, which only distinguishes
// whether the product's inputs are scaled by D^-1 (tensor form) or not.
#define HZ_BY_SCALING(A, ...)                                                \
  do {                                                                       \
    if ((A).tz.on) { constexpr int F = kFormTensor; __VA_ARGS__; }           \
    else { constexpr int F = kFormComplex; __VA_ARGS__; }                    \
  } while (0)

// Run the statement with F set to the operator's stored form.
#define HZ_BY_STORED(A, ...)                                                 \
  do {                                                                       \
    if ((A).val) { constexpr int F = kFormComplex; __VA_ARGS__; }            \
    else if ((A).st) { constexpr int F = kFormStencil; __VA_ARGS__; }        \
    else { constexpr int F = kFormSplit; __VA_ARGS__; }                      \
  } while (0)

// Run the statement with F set to the operator's storage form.
#define HZ_BY_FORM(A, ...)                                                   \
  do {                                                                       \
    if ((A).tz.on == 1) { constexpr int F = kFormTensor; __VA_ARGS__; }             \
    else if ((A).tz.on == 2) { constexpr int F = kFormTensorExt; __VA_ARGS__; }     \
    else if ((A).val) { constexpr int F = kFormComplex; __VA_ARGS__; }              \
    else if ((A).st) { constexpr int F = kFormStencil; __VA_ARGS__; }               \
    else { constexpr int F = kFormSplit; __VA_ARGS__; }                             \
  } while (0)
