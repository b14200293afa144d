// Device building blocks shared by the Krylov solvers.
//
// Row layout.  A solve works on one system, or on a batch of independent
// systems ("segments") stacked one after the other, each padded to a whole
// number of 256-row blocks.  Every vector kernel runs one block per 256 rows,
// so each block belongs to exactly one segment (in the tensor form a vector
// kernel's block takes a run of 256-row tiles); reductions write one partial
// per block, and the kernel that needs the sum (advance), or one block per
// segment, adds that segment's partials in block order.  Sums are therefore reproducible bit for bit, and
// every segment carries its own Krylov scalars and convergence flag: a batch
// of subdomain solves advances in lock-step but each one is its own Krylov
// iteration.  Padding rows hold zero matrix rows and zero vector entries.
#pragma once

#include <vector>

#include "common.h"

struct Seg {
  int nseg = 0;
  int nblk = 0;
  int64_t nrows = 0;              // nblk * kBlock
  const int* blk_seg = nullptr;   // [nblk]
  const int* seg_blk = nullptr;   // [nseg + 1]
  const int* blk_row = nullptr;   // [nblk + 1] first rows (vector layout; NULL: 256 rows a block)
  int64_t xcd_runs = 0;           // vector layout: 1 if blocks go to the XCDs in tile_of's runs
};

// A sliced-ELL operator in one of two storage forms.
//  complex form (val != NULL): one complex value per stored entry.
//  split form (val == NULL): the real part of every stored entry (re) plus,
//    per row, a short list of the entries whose imaginary part can be
//    nonzero (imeta/icol/iim, interleaved per slice).  Without an absorption
//    field only the entries that touch the absorbing walls are complex (the
//    wall term and the Jacobi scaling of wall columns), so this form streams
//    8 (FP64) or 4 (FP32) bytes per entry instead of 16 or 8.
//  Column indices are int32 (col) or, when every |col - row| fits, int16
//  offsets from the row (dcol).
//  stencil form (st != NULL, structured boxes): the split form's real parts
//    stored with implied columns: slot k of every row is the neighbour at
//    offset soff[k] (the 27 neighbours of a node of the box, ascending), a
//    missing neighbour holds 0; 64-row slices of 27 slots, slot k of lane l
//    at 27 * 64 * slice + 64 k + l.  No index is streamed; the imaginary
//    entries are the split form's row lists.
constexpr int kStencil = 27;
struct StencilOffsets {
  int o[kStencil];
};
// Imaginary entries of one 64-row slice (split and stencil forms).  The
// lanes whose row has any (bit l of mask) keep their lists interleaved:
// entry k of the j-th such lane at base + k nl + j, every list padded with
// zero values (column: the row itself) to the slice's longest, w.  Each step
// of the lists' loop then loads consecutive values and columns across the
// lanes, instead of one scattered list per lane.
struct ImSlice {
  int base, nl, w, pad;
  unsigned long long mask;
};

// Tensor form (tensor.h): the operator of a box on a tensor-product grid,
// applied from the 1-D matrices of its axes; no stored entries.
struct TzAxis;
struct TzLine;
struct TzSeg {                    // one box: a segment's rows
  int nx, ny, nz;                 // nodes along the axes
  int njb, nxc, nzc;              // wave grid: line groups, x pieces, plane groups
  int blk0, nblk;                 // its blocks in the product layout
  int row0, n, nrows;             // first row, nodes, rows with padding
  int xt, yt, zt, lt;             // axis tables and line table offsets
  int e0;                         // first element (absorption field)
  double inv_nx;                  // 1 / nx
};
struct TzOp {
  int on = 0;                     // 1: plain, 2: with an absorption field
  int scale = 0;                  // the operator is A D^-1: vector kernels scale the product's inputs (tz_pre)
  int nseg = 0;
  TzSeg s0 = {};                  // the only segment (nseg 1)
  const TzSeg* segs = nullptr;    // [nseg] on the device
  const TzAxis* tab = nullptr;
  const TzLine* dx = nullptr;     // diag(A) tables: per x node and per line
  const TzLine* lt = nullptr;
  const double* eta = nullptr;    // absorption field per element (NULL: none)
  const double* ed = nullptr;     // its mass diagonal per row
  const double* k2 = nullptr;     // [1], beside the tables (read with an absorption field only)
  Seg lp;                         // layout of the product kernels
};
struct TzCorner {                 // what each wall adds to its corner of the 1-D stiffness
  z_t v[6];
};
template <typename T>
struct SellOp {
  const int* ptr = nullptr;       // [nrows / 64 + 1] slice offsets
  const int* col = nullptr;
  const cx<T>* val = nullptr;
  const T* re = nullptr;          // split form
  const int16_t* dcol = nullptr;  // split form: column - row (NULL: use col)
  const ImSlice* imeta = nullptr; // [nrows / 64] imaginary entries of each slice
  const int* icol = nullptr;      // their columns and values, interleaved per slice
  const T* iim = nullptr;
  const T* st = nullptr;          // stencil form
  int64_t nrows = 0;              // stencil form: rows of the vectors (gathers are clamped to them)
  StencilOffsets soff = {};
  TzOp tz;                        // tensor form
};

// Non-temporal loads for the streamed matrix data (read once per product):
// keeps L2 / Infinity Cache for the gathered vector.
typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ z_t ld_stream(const z_t* p) {
  d2v v = __builtin_nontemporal_load(reinterpret_cast<const d2v*>(p));
  return z_t{v.x, v.y};
}
__device__ __forceinline__ c_t ld_stream(const c_t* p) {
  f2v v = __builtin_nontemporal_load(reinterpret_cast<const f2v*>(p));
  return c_t{v.x, v.y};
}
__device__ __forceinline__ int ld_stream(const int* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ int ld_stream(const int16_t* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ double ld_stream(const double* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ float ld_stream(const float* p) { return __builtin_nontemporal_load(p); }

// Real-part sweep of the split form: acc += re_k * x[col_k] over the row.
template <typename T, typename I>
__device__ __forceinline__ void split_real(const I* __restrict__ c, const T* __restrict__ v, int w, int64_t row,
                                           const cx<T>* __restrict__ x, T& ar, T& ai) {
#pragma unroll 9
  for (int k = 0; k < w; ++k) {
    int j = ld_stream(c + (k << 6));
    if (sizeof(I) == 2) j += int(row);
    T a = ld_stream(v + (k << 6));
    cx<T> xv = x[j];
    ar = fma(a, xv.re, ar);
    ai = fma(a, xv.im, ai);
  }
}

// Storage forms of a SellOp (compile-time selector of sell_row_form).
enum { kFormComplex = 0, kFormSplit = 1, kFormStencil = 2, kFormTensor = 3, kFormTensorExt = 4 };

// Launch bounds of the solver kernels that carry a sparse product (T: the
// vector type).  Capping the FP64 kernels at 6 waves per SIMD lets the
// compiler give the product loop more registers (measured: 88 VGPRs, 5 waves,
// 250.5 us per BiCGStab iteration on the 160x96x80 cavity, against 76 VGPRs,
// 6 waves, 258.5 us uncapped); the complex64 kernels ran slower capped.
#define HZ_PRODUCT_BOUNDS __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, sizeof(T) == 8 ? 6 : 8)))

// y_row = sum_k A[row, col_k] x[col_k] over the row's sliced-ELL entries,
// for an operator known to be in form F.
template <int F, typename T>
__device__ __forceinline__ cx<T> sell_row_form(const SellOp<T>& A, int64_t row, const cx<T>* __restrict__ x) {
  const int slice = int(row >> 6), lane = int(row & 63);
  if constexpr (F == kFormComplex) {
    const int beg = A.ptr[slice];
    const int w = (A.ptr[slice + 1] - beg) >> 6;
    const int* __restrict__ c = A.col + beg + lane;
    const cx<T>* __restrict__ v = A.val + beg + lane;
    cx<T> acc = {T(0), T(0)};
#pragma unroll 6
    for (int k = 0; k < w; ++k) {
      int j = ld_stream(c + (k << 6));
      cx<T> a = ld_stream(v + (k << 6));
      cx<T> xv = x[j];
      cfma(acc, a, xv);
    }
    return acc;
  }
  T ar = T(0), ai = T(0);
  // the slice's imaginary-list descriptor, loaded ahead of the real-part sweep
  const ImSlice im = A.imeta[slice];
  const bool listed = (im.mask >> lane) & 1ull;
  const int jl = __builtin_popcountll(im.mask & ((1ull << lane) - 1ull));
  if constexpr (F == kFormStencil) {
    // Slots 3 t, 3 t + 1, 3 t + 2 are one line of the box (offsets o - 1,
    // o, o + 1).  The wave's 64 consecutive rows load the centre x[row + o]
    // once; the left and right neighbours come from the adjacent lanes,
    // and only the wave's two end lanes load their outer value (one load
    // with two lanes active).  Terms are added in slot order, as before.
    // Every caller runs this with all 64 lanes of the wave active.
    const T* __restrict__ v = A.st + int64_t(slice) * (kStencil * 64) + lane;
    const int64_t last = A.nrows - 1;
    auto clampi = [last](int64_t j) { return j < 0 ? int64_t(0) : (j > last ? last : j); };
#pragma unroll 3
    for (int t = 0; t < kStencil / 3; ++t) {
      const int o = A.soff.o[3 * t + 1];
      const cx<T> xc = x[clampi(row + o)];
      cx<T> xe = {T(0), T(0)};
      if (lane == 0 || lane == kWave - 1) xe = x[clampi(lane == 0 ? row + o - 1 : row + o + 1)];
      cx<T> xl, xr;
      xl.re = __shfl_up(xc.re, 1, kWave);
      xl.im = __shfl_up(xc.im, 1, kWave);
      xr.re = __shfl_down(xc.re, 1, kWave);
      xr.im = __shfl_down(xc.im, 1, kWave);
      if (lane == 0) xl = xe;
      if (lane == kWave - 1) xr = xe;
      const T a0 = ld_stream(v + ((3 * t) << 6));
      const T a1 = ld_stream(v + ((3 * t + 1) << 6));
      const T a2 = ld_stream(v + ((3 * t + 2) << 6));
      ar = fma(a0, xl.re, ar);
      ai = fma(a0, xl.im, ai);
      ar = fma(a1, xc.re, ar);
      ai = fma(a1, xc.im, ai);
      ar = fma(a2, xr.re, ar);
      ai = fma(a2, xr.im, ai);
    }
  } else {
    const int beg = A.ptr[slice];
    const int w = (A.ptr[slice + 1] - beg) >> 6;
    if (A.dcol) split_real(A.dcol + beg + lane, A.re + beg + lane, w, row, x, ar, ai);
    else split_real(A.col + beg + lane, A.re + beg + lane, w, row, x, ar, ai);
  }
  // imaginary entries, four steps at a time: the four value/column loads,
  // then the four gathers, issue back to back (a step past the slice's
  // longest list gathers x[0] and adds nothing; a padded entry adds zero);
  // the terms are added in list order
  if (listed) {
    const T* __restrict__ pb = A.iim + im.base + jl;
    const int* __restrict__ pc = A.icol + im.base + jl;
    for (int k = 0; k < im.w; k += 4) {
      T b[4];
      int c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool on = k + u < im.w;
        b[u] = on ? pb[(k + u) * im.nl] : T(0);
        c[u] = on ? pc[(k + u) * im.nl] : 0;
      }
      cx<T> xv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) xv[u] = x[c[u]];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k + u < im.w) {         // i b x = -b x.im + i b x.re
          ar = fma(-b[u], xv[u].im, ar);
          ai = fma(b[u], xv[u].re, ai);
        }
    }
  }
  return cx<T>{ar, ai};
}


// Block geometry of a segmented kernel: tile, row, segment.  Tile t holds
// rows [256 t, 256 t + 256); workgroups take tiles in runs of 8 per XCD
// (xcd_chunk_tile), so rows whose neighbourhoods overlap mostly share one
// XCD's L2.  Measured on the 27-point products this beats both plain
// dispatch order and one contiguous row range per XCD.
struct Tile {
  int tile;
  int seg;
  int64_t row;
};
__device__ __forceinline__ Tile tile_of(const Seg& L) {
  Tile t;
  t.tile = xcd_chunk_tile(blockIdx.x, gridDim.x);
  t.seg = L.blk_seg[t.tile];
  t.row = int64_t(t.tile) * kBlock + threadIdx.x;
  return t;
}
// Count of this block's waves that have stored their sums in store_partials.
__device__ __forceinline__ int* block_wave_count() {
  __shared__ int n;
  return &n;
}
// The tile of a kernel that stores block partials (store_partials takes
// only this type): all its threads call it first, before any return, and
// the block's wave count is zeroed behind a barrier.
struct SumTile : Tile {};
__device__ __forceinline__ SumTile tile_of_sums(const Seg& L) {
  SumTile t;
  static_cast<Tile&>(t) = tile_of(L);
  if (threadIdx.x == 0) *block_wave_count() = 0;
  __syncthreads();
  return t;
}

// Block-sum NQ doubles and store them as partial[tile * NQ + q]: every
// quantity is reduced within each wave, each wave puts its sums in LDS and
// counts itself in, and the wave that counts last adds the waves' sums in
// wave order (so the result does not depend on which wave that is) and
// stores them.  No barrier closes the kernel: a wave that is not last
// leaves at once instead of holding its slot until the block's slowest wave
// finishes (measured 79 -> 75 us for the 27-point product with four sums).
// Called once per kernel, by every wave of the block or by none (the
// callers return early only for a whole segment, hence a whole block), with
// the tile from tile_of_sums, which zeroed the count.
template <int NQ>
__device__ __forceinline__ void store_partials(double (&v)[NQ], double* partial, const SumTile& t) {
  const int tile = t.tile;
  constexpr int kWaves = kBlock / kWave;
  __shared__ double lds[NQ][kWaves];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  double s[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) s[q] = wave_sum(v[q]);
  int last = 0;
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) lds[q][w] = s[q];
    // release: the sums are in LDS before the count; acquire for the last
    last = __hip_atomic_fetch_add(block_wave_count(), 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) ==
           kWaves - 1;
  }
  last = __shfl(last, 0, kWave);
  if (!last) return;
  // every lane of the last wave reads the other waves' sums after the count
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (int q = lane; q < NQ; q += kWave) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i)
      t += __hip_atomic_load(&lds[q][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    partial[int64_t(tile) * NQ + q] = t;
  }
}

// The same, storing quantity q at partial[q * qstride + tile] (each
// quantity's block partials contiguous, for finalize kernels that reduce one
// quantity per block).
template <int NQ>
__device__ __forceinline__ void store_partials_qmajor(double (&v)[NQ], double* partial, int64_t qstride,
                                                      const SumTile& t) {
  const int tile = t.tile;
  constexpr int kWaves = kBlock / kWave;
  __shared__ double lds[NQ][kWaves];
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  double s[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) s[q] = wave_sum(v[q]);
  int last = 0;
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) lds[q][w] = s[q];
    last = __hip_atomic_fetch_add(block_wave_count(), 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) ==
           kWaves - 1;
  }
  last = __shfl(last, 0, kWave);
  if (!last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (int q = lane; q < NQ; q += kWave) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i)
      t += __hip_atomic_load(&lds[q][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    partial[int64_t(q) * qstride + tile] = t;
  }
}

// Finalize kernels run with kFinBlock threads, one block per segment.
constexpr int kFinBlock = 1024;

// Partial sums of a segmented reduction, NQ per block: blocks
// [seg_blk[s], seg_blk[s + 1]) belong to segment s; none, if a kernel of its own
// (k_step) has made the scalar step: the state then says that it is not due.
struct Part {
  double* p = nullptr;
  const int* seg_blk = nullptr;
  int nseg = 0, nblk = 0;
};

// Scalar steps without kernels of their own.  A kernel that forms sums leaves
// block partials; the kernel that needs the scalars adds all partials of its
// segment at its start, in block order, in every block alike (a fixed order:
// every block gets the same bits), and one thread runs the scalar step.  The
// state it starts from is read from one slot and the state it reaches is
// written to another by the segment's first block, so no block reads what
// another one writes in the same kernel.  Against a finalize kernel between
// the two (4 to 6 us: a launch and one block's chain of loads) this costs the
// kernel 2.5 to 3 us; against finishing in the producing kernel's last block,
// which pays a store, two atomic arrivals and a reload one after the other
// across the XCDs, it saved 3 us per reduction at 20 to 160 thousand rows.
//
// A step f of a state St: f.on(state) says whether it is due, f(state, sums) makes it.
//
// All threads of the block call it; the state is in LDS afterwards.
// EARLY: leave at once where the step has been made.  The stored forms beyond
// 260,000 rows, where it is (kMaxConsumed), gain 1 to 2% by it; in the tensor form
// it gains nothing at 1.26 million and the test costs small systems 1%.
template <int NQ, bool EARLY, class St, class Step>
__device__ __forceinline__ const St& advance(const Part& P, const St* in, St* out, const Tile& t, bool first, Step f) {
  constexpr int kPasses = kFinBlock / kBlock, kWaves = kFinBlock / kWave;
  __shared__ double lds[NQ][kWaves];
  __shared__ double tot[NQ];
  __shared__ St st;
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  // the state goes through LDS word by word: a private copy of the struct would
  // live in scratch memory, which alone costs a kernel 10 us
  static_assert(sizeof(St) % sizeof(int) == 0, "state is copied by words");
  constexpr int kWords = sizeof(St) / sizeof(int);
  int* sw = reinterpret_cast<int*>(&st);
  const int b0 = P.nseg == 1 ? 0 : P.seg_blk[t.seg], b1 = P.nseg == 1 ? P.nblk : P.seg_blk[t.seg + 1];
  // the order of a kFinBlock-thread finalize kernel (seg_sums): thread u takes
  // blocks u, u + kFinBlock, ..., here threads u of pass m stand for u + 256 m
  // (passes without blocks would add zeros)
  const int passes = min(kPasses, (b1 - b0 + kBlock - 1) / kBlock);
  double acc[kPasses][NQ];
#pragma unroll
  for (int m = 0; m < kPasses; ++m) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[m][q] = 0.0;
    if (m < passes)
      for (int b = b0 + m * kBlock + int(threadIdx.x); b < b1; b += kFinBlock) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[m][q] += P.p[int64_t(b) * NQ + q];
      }
  }
  for (int u = threadIdx.x; u < kWords; u += kBlock) sw[u] = reinterpret_cast<const int*>(in + t.seg)[u];
  if (EARLY && P.nblk == 0) {      // the step has been made
    __syncthreads();
    return st;
  }
#pragma unroll
  for (int m = 0; m < kPasses; ++m) {
    if (m < passes) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const double s = wave_sum(acc[m][q]);
        if (lane == 0) lds[q][m * (kBlock / kWave) + w] = s;
      }
    }
  }
  __syncthreads();
  // (unrolled: the LDS reads issue together; one after the other they were
  // 2 us of a 9.7 us kernel at 16 waves and 4 sums)
  auto total = [&](int q) {
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < kPasses; ++m)
      if (m < passes) {
#pragma unroll
        for (int i = 0; i < kBlock / kWave; ++i) s += lds[q][m * (kBlock / kWave) + i];
      }
    return s;
  };
  if (NQ > 4) {
    for (int q = threadIdx.x; q < NQ; q += kBlock) tot[q] = total(q);
    __syncthreads();
  }
  if (threadIdx.x == 0 && f.on(st)) {
    if (NQ <= 4) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) tot[q] = total(q);
    }
    f(st, static_cast<const double*>(tot));
  }
  __syncthreads();
  if (first)
    for (int u = threadIdx.x; u < kWords; u += kBlock) reinterpret_cast<int*>(out + t.seg)[u] = sw[u];
  return st;
}
// First block of its segment in layout L.
__device__ __forceinline__ bool first_block(const Seg& L, const Tile& t) {
  return t.tile == (L.nseg == 1 ? 0 : L.seg_blk[t.seg]);
}

// Vector layout: block b works on rows [blk_row[b], blk_row[b + 1]) of one
// segment, a whole number of 256-row tiles.  With one tile a block (stored forms)
// the blocks take the tiles in the products' order, so a vector that a product
// just wrote is read on the XCD whose L2 holds it (TFQMR, us a product, in
// dispatch order : so: 289,937 rows of hexahedra 57.3:56.4, 146,657 of tetrahedra
// 28.4:27.2, 230,230 of a box 35.7:34.9).
__device__ __forceinline__ Tile vec_tile(const Seg& L) {
  Tile t;
  t.tile = L.xcd_runs ? xcd_chunk_tile(blockIdx.x, gridDim.x) : int(blockIdx.x);
  t.seg = L.nseg == 1 ? 0 : L.blk_seg[t.tile];
  t.row = L.blk_row[t.tile] + int(threadIdx.x);
  return t;
}
__device__ __forceinline__ SumTile vec_tile_sums(const Seg& L) {
  SumTile t;
  static_cast<Tile&>(t) = vec_tile(L);
  if (threadIdx.x == 0) *block_wave_count() = 0;
  __syncthreads();
  return t;
}
template <class Body>
__device__ __forceinline__ void vec_rows(const Seg& L, const Tile& t, Body body) {
  const int64_t end = L.blk_row[t.tile + 1];
#pragma unroll 2
  for (int64_t row = t.row; row < end; row += kBlock) body(row);
}

// Sum every quantity of this segment's partials in one pass (thread t takes
// tiles t, t + blockDim, ...; then wave sums and the waves in order); the
// totals are valid in thread 0.  Finalize kernels call it before they branch
// on the segment's state (read into registers first), so the partials'
// loads do not wait for the state's; the sums of a segment that is off are
// simply not used.
template <int NQ>
__device__ __forceinline__ void seg_sums(const Seg& L, const double* partial, int seg, double (&out)[NQ]) {
  __shared__ double lds[NQ][kFinBlock / kWave];
  // one segment spans every block: no dependent load of its block range
  const int b0 = L.nseg == 1 ? 0 : L.seg_blk[seg], b1 = L.nseg == 1 ? L.nblk : L.seg_blk[seg + 1];
  double acc[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
#pragma unroll 4
  for (int i = b0 + int(threadIdx.x); i < b1; i += int(blockDim.x)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] += partial[int64_t(i) * NQ + q];
  }
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave, nw = blockDim.x / kWave;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double s = wave_sum(acc[q]);
    if (lane == 0) lds[q][w] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      double s = 0.0;
      for (int i = 0; i < nw; ++i) s += lds[q][i];
      out[q] = s;
    }
  }
  __syncthreads();
}

// A scalar step by a kernel of its own, one block per segment, in place
// (restarts), into the slot of the kernels that need it (PartBuf::step) or for
// the host; copy and next (or NULL) take the state too.  The sums' order and the
// step are advance's, so the state has the same bits either way.
template <int NQ, class St, class Step>
__global__ void __launch_bounds__(kFinBlock) k_step(Seg L, const double* part, const St* in, St* out, St* copy, St* next,
                                                    Step f) {
  __shared__ St st;
  const int s = blockIdx.x;
  constexpr int kWords = sizeof(St) / sizeof(int);
  int* sw = reinterpret_cast<int*>(&st);
  if (threadIdx.x < kWords) sw[threadIdx.x] = reinterpret_cast<const int*>(in + s)[threadIdx.x];
  static_assert(kWords <= kFinBlock, "one word a thread");
  double o[NQ];
  seg_sums<NQ>(L, part, s, o);   // (its barriers also order the state's words)
  if (threadIdx.x == 0 && f.on(st)) f(st, static_cast<const double*>(o));
  __syncthreads();
  if (threadIdx.x < kWords) reinterpret_cast<int*>(out + s)[threadIdx.x] = sw[threadIdx.x];
  if (copy && threadIdx.x < kWords) reinterpret_cast<int*>(copy + s)[threadIdx.x] = sw[threadIdx.x];
  if (next && threadIdx.x < kWords) reinterpret_cast<int*>(next + s)[threadIdx.x] = sw[threadIdx.x];
}
// Makes a segment's due step and sets which segments restart: all of
// them, or those that broke down.  One step on the state in LDS: the words of
// the stored state are written by different threads, so none may be read or
// written again behind it.
template <class Step>
struct Settle {
  Step f;
  int all;
  template <class St> __device__ bool on(const St&) const { return true; }
  template <class St> __device__ void operator()(St& S, const double* tot) const {
    if (f.on(S)) f(S, tot);
    S.restart = all ? 1 : S.brk;
  }
};

// In a finalize kernel (one block per segment): sum quantity q of this
// segment's partials; valid in thread 0.
template <int NQ>
__device__ __forceinline__ double seg_sum(const Seg& L, const double* partial, int seg, int q) {
  __shared__ double lds[kFinBlock / kWave];
  const int b0 = L.nseg == 1 ? 0 : L.seg_blk[seg], b1 = L.nseg == 1 ? L.nblk : L.seg_blk[seg + 1];
  return block_sum_strided(partial + int64_t(b0) * NQ + q, b1 - b0, NQ, lds);
}

// conj(a) b, each part with one rounding of its second product
__device__ __forceinline__ z_t conj_mul(z_t a, z_t b) {
  return {fma(a.re, b.re, a.im * b.im), fma(a.re, b.im, -(a.im * b.re))};
}
// Minimal-residual step of BiCGStab(l): Cholesky solve of G gamma = c (G
// Hermitian, LL x LL) from the sums tot (c, then the rows of G's upper
// triangle), truncated at the first pivot below piv times its diagonal entry
// (G is exact for the stored vectors, so piv guards the FP64 Cholesky only).
// Returns the number of pivots used; gamma beyond it is 0.  Every loop is unrolled,
// so the matrix sits in registers (as a scratch array this step took 23 us
// at LL = 4, five times the kernel around it).
template <int LL>
__device__ __forceinline__ int gram_solve(const double* tot, double piv, z_t (&g)[LL]) {
  z_t c[LL], G[LL][LL];      // G: lower triangle
  int k = 0;
#pragma unroll
  for (int i = 0; i < LL; ++i, k += 2) c[i] = z_t{tot[k], tot[k + 1]};
#pragma unroll
  for (int i = 0; i < LL; ++i)
#pragma unroll
    for (int jj = i; jj < LL; ++jj, k += 2) G[jj][i] = z_t{tot[k], -tot[k + 1]};
  // G = C C^H, C lower triangular (diagonal real)
  int m = LL;
#pragma unroll
  for (int jj = 0; jj < LL; ++jj) {
    double d = G[jj][jj].re;
#pragma unroll
    for (int p = 0; p < jj; ++p) d -= fma(G[jj][p].re, G[jj][p].re, G[jj][p].im * G[jj][p].im);
    if (m == LL && (!(d > piv * G[jj][jj].re) || !isfinite(d))) m = jj;
    const double cd = m == LL ? sqrt(d) : 1.0, ci = 1.0 / cd;
    G[jj][jj] = z_t{cd, 0.0};
#pragma unroll
    for (int i = jj + 1; i < LL; ++i) {
      z_t v = G[i][jj];
#pragma unroll
      for (int p = 0; p < jj; ++p) v = v - conj_mul(G[jj][p], G[i][p]);
      G[i][jj] = ci * v;
    }
  }
  z_t y[LL];
#pragma unroll
  for (int i = 0; i < LL; ++i) {           // C y = c
    z_t v = c[i];
#pragma unroll
    for (int p = 0; p < i; ++p) {
      const z_t a = G[i][p];
      v = v - z_t{fma(a.re, y[p].re, -(a.im * y[p].im)), fma(a.im, y[p].re, a.re * y[p].im)};
    }
    y[i] = i < m ? (1.0 / G[i][i].re) * v : z_t{0.0, 0.0};
  }
#pragma unroll
  for (int i = LL - 1; i >= 0; --i) {      // C^H g = y
    z_t v = y[i];
#pragma unroll
    for (int p = i + 1; p < LL; ++p)
      if (p < m) v = v - conj_mul(G[p][i], g[p]);
    g[i] = i < m ? (1.0 / G[i][i].re) * v : z_t{0.0, 0.0};
  }
  return m;
}

// Host-side description of a segmented system on the device.
struct SegHost {
  int nseg = 0, nblk = 0;
  int64_t nrows = 0;
  std::vector<int> seg_blk;       // host copy [nseg + 1]
  std::vector<int64_t> seg_n;     // true (unpadded) rows per segment
  Seg dev;                        // device view
  const int* zeros = nullptr;     // [nseg + 1] (device)
  // vector layouts of the same segments: one 256-row tile per block (stored
  // forms), and runs of tiles, about 1,000 blocks (four per CU) at most, so
  // that advance has few partials to add (tensor form)
  Seg vec, vec_runs;
};
