// Host-side interface of the operator kernels and solvers.
#pragma once

#include <string>
#include <type_traits>

#include "ctx.h"
#include "krylov.h"
#include "tensor.h"

// Device pointers of the real operator parts (SELL layout).
struct OpParts {
  const double* K = nullptr;
  const double* M = nullptr;
  const double* Meta = nullptr;   // NULL: no absorption field
  const int* bidx = nullptr;      // per stored entry: boundary slot or -1
  const z_t* Bb = nullptr;        // per boundary slot: sum_w beta_w B0_w
  const int* diag = nullptr;      // per row: stored position of the diagonal
  const uint8_t* emask = nullptr; // Dirichlet elimination per entry (NULL: none)
  double gls_h = 0.0;             // GLS element size (0: Galerkin mass coefficient)
};

// Mass coefficient m(k) of A = K - m(k) M + ...: k^2, or with the Galerkin
// least-squares stabilisation of Harari and Hughes (1992) for linear
// elements k^2 (1 - tau k^2), tau k^2 = 1 - 6 (1 - cos kh) / ((kh)^2 (2 +
// cos kh)), the value that makes the 1-D discrete dispersion exact.
inline double mass_coefficient(double k, double gls_h) {
  const double k2 = k * k;
  if (!(gls_h > 0.0) || k == 0.0) return k2;
  const double t = k * gls_h, c = std::cos(t);
  const double tau_k2 = 1.0 - 6.0 * (1.0 - c) / (t * t * (2.0 + c));
  return k2 * (1.0 - tau_k2);
}

inline OpParts op_parts(hz_ctx ctx) {
  OpParts P;
  P.K = ctx->d_K.as<double>();
  P.M = ctx->d_M.as<double>();
  P.Meta = ctx->have_eta ? ctx->d_Meta.as<double>() : nullptr;
  P.bidx = ctx->d_bidx.as<int>();
  P.Bb = ctx->d_Bb.as<z_t>();
  P.diag = ctx->d_diag.as<int>();
  P.emask = ctx->dirichlet ? ctx->d_emask.as<uint8_t>() : nullptr;
  P.gls_h = ctx->h.gls_h;
  return P;
}

// The current operator in complex form.
inline SellOp<double> op_A_complex(hz_ctx ctx) {
  SellOp<double> A;
  A.ptr = ctx->d_sptr.as<int>();
  A.col = ctx->d_scol.as<int>();
  A.val = ctx->d_A.as<z_t>();
  return A;
}
inline SellOp<float> op_A32_complex(hz_ctx ctx) {
  SellOp<float> A;
  A.ptr = ctx->d_sptr.as<int>();
  A.col = ctx->d_scol.as<int>();
  A.val = ctx->d_A32.as<c_t>();
  return A;
}
// The same operator in split form (valid when ctx->have_split / have_split32).
template <typename T>
inline SellOp<T> op_split(hz_ctx ctx) {
  SellOp<T> A;
  A.ptr = ctx->d_sptr.as<int>();
  A.col = ctx->d_scol.as<int>();
  A.dcol = ctx->split_dcol ? ctx->d_dcol.as<int16_t>() : nullptr;
  A.imeta = ctx->d_imeta.as<ImSlice>();
  A.icol = ctx->d_icol.as<int>();
  A.re = sizeof(T) == 8 ? static_cast<T*>(ctx->d_R.p) : static_cast<T*>(ctx->d_R32.p);
  A.iim = sizeof(T) == 8 ? static_cast<T*>(ctx->d_I.p) : static_cast<T*>(ctx->d_I32.p);
  return A;
}
// The same in stencil form (valid when ctx->have_stencil / have_stencil32).
template <typename T>
inline SellOp<T> op_stencil(hz_ctx ctx) {
  SellOp<T> A = op_split<T>(ctx);   // imaginary lists
  A.st = sizeof(T) == 8 ? static_cast<T*>(ctx->d_S.p) : static_cast<T*>(ctx->d_S32.p);
  A.nrows = ctx->sell.n_rows;
  A.soff = ctx->soff;
  return A;
}
// ---------------------------------------------------------------- tensor form
bool tensor_detect(const HostAsm& a, const int32_t elems[3], TensorGrid* g);
// Layout, tables and buffers of stacked boxes; rows of box s: [row0[s], row0[s] + nrows[s]).
int tensor_build(hz_ctx ctx, const std::vector<TensorGrid>& grids, const std::vector<int64_t>& row0,
                 const std::vector<int64_t>& nrows, const std::string& name, TensorDev* D);
// The tables for mass coefficient m, k^2 and the walls' corner terms (stream-ordered).
int tensor_tables(hz_ctx ctx, TensorDev* D, const std::vector<TzCorner>& corners, double m, double k2);
int tensor_axes(hz_ctx ctx, const TensorDev& D, DevBuf* tab);   // without frequency and walls
int tensor_diag(hz_ctx ctx, const TensorDev& D, double k2, z_t* d, z_t* dinv);
int tensor_eta(hz_ctx ctx, TensorDev* D, const double* eta_host, int64_t count);
TzOp tensor_op(const TensorDev& D, bool scale);

// The operator the solvers use: the tensor form, else the stencil form, else
// the split form, when formed.
inline TzOp op_tensor(hz_ctx ctx) {
  return tensor_op(*ctx->tz, ctx->scaled == HZ_JACOBI);
}
inline SellOp<double> op_A(hz_ctx ctx) {
  if (ctx->tz) {
    SellOp<double> A;
    A.tz = op_tensor(ctx);
    return A;
  }
  return ctx->have_stencil ? op_stencil<double>(ctx) : ctx->have_split ? op_split<double>(ctx) : op_A_complex(ctx);
}
inline SellOp<float> op_A32(hz_ctx ctx) {
  if (ctx->tz) {
    SellOp<float> A;
    A.tz = op_tensor(ctx);
    return A;
  }
  return ctx->have_stencil32 ? op_stencil<float>(ctx)
                             : ctx->have_split32 ? op_split<float>(ctx) : op_A32_complex(ctx);
}

// The solvers' operator at wavenumber k: the tensor form's tables, or the stored forms.
int op_set_frequency(hz_ctx ctx, double k, int scale, bool want32);
// The stored forms (complex, split, stencil) whatever form the solvers use.
int op_form_stored(hz_ctx ctx, const OpParts& P, double k, int scale, bool want32);
// Forms A(k) (optionally column-scaled by 1/diag) on an explicit sliced-ELL
// system; rows i >= n or with diag[i] < 0 are padding (d = 1).
int op_form(hipStream_t s, int64_t n, int64_t nrows, int64_t npad, const int* col, const OpParts& P, double k,
            int scale, z_t* A, c_t* A32, z_t* d, z_t* dinv, double* R = nullptr, float* R32 = nullptr);
// I[q] = Im A[ipos[q]] (0 where ipos[q] < 0), and its FP32 copy when I32 is
// given: the imaginary lists of a split-form operator.
int op_split_im(hipStream_t s, int64_t ni, const int* ipos, const z_t* A, double* I, float* I32);
template <typename T>
int op_spmv(hipStream_t s, int64_t nrows, int64_t nout, const SellOp<T>& A, const cx<T>* x, cx<T>* y);
int op_mul(hipStream_t s, int64_t n, const z_t* a, const z_t* b, z_t* c);
int op_fill(hipStream_t s, int64_t n, z_t* y, z_t v);
int op_copy(hipStream_t s, int64_t n, const z_t* x, z_t* y);
int op_load(hz_ctx ctx, const z_t* g, z_t* f);
int op_dotc(hz_ctx ctx, int64_t n, const z_t* a, const z_t* b, double* out_dev);
// Dirichlet load in the internal numbering (padded vectors of nrows):
// f_i = g_i on D rows, f_i = -sum_{j in D} A_ij g_j on the others, with the
// entries of A before the elimination (paper Sec. 3.2 Dirichlet source).
int op_lift(hz_ctx ctx, const z_t* g, z_t* f);
// The same two kernels with the caller's partial-sum buffer (2 reduce_grid(n)
// doubles) on the given stream.
int op_dotc_into(hipStream_t stream, int64_t n, const z_t* a, const z_t* b, double* part, double* out_dev);

// ---------------------------------------------------------------- solvers
// Per-segment controls and results of one Krylov run.
struct KrylovCtl {
  double tol = 1e-8;              // relative to ||f_seg||
  int max_matvec = 20000;
  int restart = 30;               // GMRES
  int ell = 4;                    // BiCGStab(l)
  // TFQMR: a quasi-residual bound that has not halved over this many
  // half-steps ends the solve (0: never); GMRES: a residual over as many
  // products, or over four cycles that met the target by their estimate alone, on
  // every segment that is not done.  Set for complex64 inner solves
  // of the refinement, which can stall above the inner tolerance (a GMRES solve
  // restarted from its iterate loses nothing by it).
  int stall_halfsteps = 0;
};
struct KrylovOut {
  std::vector<int> iters, matvecs, status;
  std::vector<double> relres_est, fnorm;
};

// The solvers' view of their device state.  Chunks of iterations are queued
// one ahead: while a chunk runs, the state that the chunk before it left is
// already in one of two pinned slots, so the device never waits for the
// host's decision.  Kernels of a chunk queued after a segment has
// stopped return at once, but each still takes 2 to 4 us, so short solves must
// not queue much past their end (Pace).  Chunks of 2, 4, 8, 8, ...
// iterations, all queued ahead, against this: 8 BiCGStab products at 289,937
// rows 0.89 -> 0.61 ms, 18 of BiCGStab(8) at 162,729 1.27 -> 0.83 ms, 9 of TFQMR
// there 0.57 -> 0.38 ms, long solves the same within 2%.
struct StatePoll {
  hz_ctx ctx;
  size_t bytes = 0;
  char* host = nullptr;
  int posted = 0;                    // copies queued so far
  int init(hz_ctx c, size_t nbytes);
  // Where the kernel that reports the state next writes it (pinned host
  // memory that the device can write); posted_one() after its launch.
  template <typename S> S* slot() const { return reinterpret_cast<S*>(host + (posted & 1) * bytes); }
  int posted_one();
  int wait(int k);                   // report k (0-based, one of the last two) has arrived
  template <typename S> const S* state(int k) const { return reinterpret_cast<const S*>(host + (k & 1) * bytes); }
};

// How many iterations (BiCGStab(l): cycles) to queue next, and whether to wait
// for the chunk just queued instead of the one before it (until `sync` are
// queued).  Small systems (replays), whose iterations take hardly longer than idle
// ones or than the report of a chunk, go on to whole chunks at once; on large
// ones the chunks grow with an eighth of what has been queued.
struct Pace {
  int first, least, most, sync;
  bool replays;
  int next(int64_t queued) const {
    if (queued == 0) return first;
    if (replays) return std::min(most, queued == first ? 2 * first : most);
    return int(std::min<int64_t>(most, std::max<int64_t>(least, queued / 8)));
  }
  bool at_once(int64_t queued) const { return queued <= sync; }   // queued: with this chunk
};

// Runs of iterations as HIP graphs.  A solver's chunk of iterations is the
// same list of kernels with the same arguments every time, and on small
// systems the host cannot issue them as fast as the device runs them (4 to 10
// us of host time a launch against 2 to 5 us kernels): it is captured once and
// replayed on the context's stream.  Measured at 20x12x10, GMRES(30): 46.6 ->
// 30.1 ms.
//
// The capture is kept in the context under the solver's tag together with
// every argument its kernels take (ReplayKey), so a later solve replays it
// only if it would launch exactly that; there is one per tag, the next
// differing solve replaces it.  What a frequency or new parameters change is
// in device memory at the same addresses, so a loop over frequencies captures
// once.  Only kernels are captured, and a capture that fails leaves the solver
// launching them one by one.
//
// A capture takes 40 us (BiCGStab, 40 kernels) to 100 us (GMRES(30), 123
// kernels) of host time, the first of a context 0.2 to 0.9 ms, and saves 10 us a
// chunk of 8 BiCGStab iterations and 140 us a GMRES(30) cycle, so runs are captured
// once the same one has been launched kReplayAfter (Gmres) times, in one solve or
// over several: about where a capture pays for itself.  GMRES(30) to 100 products
// in a new context took 4.2 ms at 40x24x20 before there were replays, 4.4 ms
// captured at its second cycle, 4.1 ms so, and 3.35 ms once captured.  A loop over
// 16 frequencies at 20x12x10: BiCGStab(2) to 20 products 7.2 ms capturing at each
// solve's first full chunk and 6.4 ms so (6.5 without graphs), to 60 products 15.1
// and 14.3 ms (15.0 without), GMRES(30) to 200 products 87.3 and 75.6 ms (86.4
// without).
//
// On larger systems the device is the slower of the two and the gap between a
// graph's kernels a little longer than between launches.  600 products,
// launched : replayed, ms, BiCGStab / BiCGStab(2) / BiCGStab(8) / TFQMR / mixed
// TFQMR: tensor form at 102,900 rows 9.11:8.78 9.23:8.96 12.4:12.4 9.86:9.69
// 11.4:11.2, at 162,729 11.2:10.9 11.4:11.5 16.6:16.7 11.8:11.9 13.7:13.0, at
// 308,050 13.0:13.2 13.6:13.9 21.4:21.2 13.3:13.6 14.2:14.4; stored forms at
// 29,725 9.90:9.40 10.3:9.48 10.3:9.88 10.2:10.0 10.6:9.87, at 64,800 10.8:10.8
// 11.3:11.4 13.5:13.6 11.5:11.6 10.9:10.6, at 162,729 17.0:17.0 17.3:17.6
// 23.0:23.1 17.9:18.0 15.4:15.3.  GMRES(30), which has six launches a step:
// 35.7:33.0 at 162,729 (tensor), 44.9:44.2 at 308,050, 35.8:35.8 at 162,729 (stored).
struct ReplayKey {
  std::string s;
  template <typename V>
  ReplayKey& add(const V& v) {       // types without padding
    static_assert(std::is_trivially_copyable<V>::value, "keys are compared byte by byte");
    s.append(reinterpret_cast<const char*>(&v), sizeof(V));
    return *this;
  }
  template <typename T>
  ReplayKey& op(const SellOp<T>& A) {
    add(A.ptr).add(A.col).add(A.val).add(A.re).add(A.dcol).add(A.imeta).add(A.icol).add(A.iim).add(A.st).add(A.nrows);
    const TzOp& Z = A.tz;
    add(A.soff).add(Z.on).add(Z.scale).add(Z.nseg).add(Z.s0).add(Z.segs).add(Z.tab).add(Z.dx).add(Z.lt).add(Z.eta);
    return add(Z.ed).add(Z.k2).add(Z.lp);
  }
};
constexpr int kReplayAfter = 8, kReplayAfterGmres = 6;
constexpr int64_t kReplayRowsTensor = 196608, kReplayRowsStored = 49152, kReplayRowsGmres = 262144;
// Replays the run of body on the context's stream, capturing it first if the
// same run has come up more than `after` times; *ran = false if it has to be
// launched directly.  body(stream) launches only kernels.
template <class Body>
int replay(hz_ctx ctx, const std::string& tag, const ReplayKey& key, Body body, bool* ran, int after) {
  *ran = false;
  if (!ctx->graphs_on) return HZ_OK;
  Replay& R = ctx->replays[tag];
  if (R.failed > 2) return HZ_OK;
  if (!R.exec || R.key != key.s) {
    if (R.seen_key != key.s) {
      R.seen_key = key.s;
      R.seen = 0;
    }
    if (R.seen++ < after) return HZ_OK;
    R.drop();
    if (!ctx->cap && hipStreamCreateWithFlags(&ctx->cap, hipStreamNonBlocking) != hipSuccess) {
      (void)hipGetLastError();
      ++R.failed;
      return HZ_OK;
    }
    int rc = HZ_OK;
    bool ok = hipStreamBeginCapture(ctx->cap, hipStreamCaptureModeThreadLocal) == hipSuccess;
    if (ok) {
      rc = body(ctx->cap);
      ok = hipStreamEndCapture(ctx->cap, &R.graph) == hipSuccess && rc == HZ_OK &&
           hipGraphInstantiate(&R.exec, R.graph, nullptr, nullptr, 0) == hipSuccess;
    }
    if (!ok) {
      (void)hipGetLastError();
      R.drop();
      ++R.failed;
      return HZ_OK;
    }
    R.key = key.s;
    ++ctx->n_captures;
  }
  HZ_HIP(hipGraphLaunch(R.exec, ctx->stream));
  ++ctx->n_replays;
  *ran = true;
  return HZ_OK;
}

// Block partials of one reduction.  The kernels that need the sums add the
// partials themselves (advance) as long as their blocks together read no more
// than kMaxConsumed of them; beyond, every block would read more partials than
// rows, and step() makes the scalar step once with a kernel of its own (4.6 us),
// whose state the others only copy.  It is called after every kernel that forms
// the sums.  Measured, us a product, consumed : stepped, BiCGStab / TFQMR: stored
// forms (as many consuming as producing blocks, 256 rows each) at 162,729 rows
// 28.9:29.5 30.4:31.0, at 308,050 40.1:38.8 42.4:41.8, at 608,076 68.8:61.0
// 75.4:67.2, at 1,264,977 130:105 144:117; tensor form (912, 1,506 and 2,520
// product blocks, 800 to 1,000 vector blocks) at 608,076 32.9:32.8 37.2:36.7, at
// 1,264,977 47.0:46.8 58.1:56.6, at 2,456,421 85.9:83.8 129:125.
constexpr int64_t kMaxConsumed = int64_t(1024) * 1024;
struct PartBuf {
  double* raw = nullptr;             // where the producing kernel stores
  Part part;                         // what the consuming kernels add (nothing, if step makes the step)
  bool stepped = false;
  Seg lay;
  // consumers: blocks of the kernels that would add the partials (0: one block
  // per segment does, by advance)
  int init(hz_ctx ctx, const SegHost& S, const Seg& L, int nq, int consumers, const std::string& name);
  // The scalar step from state in to out, if the consumers do not make it
  // themselves; always, at a restart or for the host.
  template <int NQ, class St, class Step>
  int step(hipStream_t s, const St* in, St* out, Step f) const { return stepped ? step_now<NQ>(s, in, out, f) : HZ_OK; }
  // The slots of a consuming kernel whose step goes from in to out: it starts from
  // out if the step has been made, and then leaves its copy in a slot nobody reads.
  template <class St>
  const St* from(const St* in, const St* out) const { return stepped ? out : in; }
  template <class St>
  St* to(St* out, St* unread) const { return stepped ? unread : out; }
  template <int NQ, class St, class Step>
  int step_now(hipStream_t s, const St* in, St* out, Step f, St* copy = nullptr, St* next = nullptr) const {
    k_step<NQ, St, Step><<<lay.nseg, kFinBlock, 0, s>>>(lay, raw, in, out, copy, next, f);
    HZ_HIP(hipGetLastError());
    return HZ_OK;
  }
  void key(ReplayKey* k) const { k->add(raw).add(part).add(lay); }
};

// Solve A u = f on every segment (u: in x0 / out), vectors of the storage
// type T, reductions and Krylov scalars in FP64.  In the stored forms A is
// A D^-1 and u = D x; in the tensor form A is unscaled and u is x.
template <typename T>
int bicgstab_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
                 const KrylovCtl& ctl, KrylovOut* out, const std::string& tag);
template <typename T>
int gmres_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
              const KrylovCtl& ctl, KrylovOut* out, const std::string& tag);
template <typename T>
int bicgstabl_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
                  const KrylovCtl& ctl, KrylovOut* out, const std::string& tag);
template <typename T>
int tfqmr_run(hz_ctx ctx, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
              const KrylovCtl& ctl, KrylovOut* out, const std::string& tag);
// Dispatch on opts->method (HZ_GMRES, HZ_BICGSTAB, HZ_BICGSTABL or HZ_TFQMR).
template <typename T>
int krylov_run(hz_ctx ctx, int method, const SegHost& S, const SellOp<T>& A, const cx<T>* f, cx<T>* u,
               const KrylovCtl& ctl, KrylovOut* out, const std::string& tag) {
  if (method == HZ_BICGSTAB) return bicgstab_run<T>(ctx, S, A, f, u, ctl, out, tag);
  if (method == HZ_BICGSTABL) return bicgstabl_run<T>(ctx, S, A, f, u, ctl, out, tag);
  if (method == HZ_TFQMR) return tfqmr_run<T>(ctx, S, A, f, u, ctl, out, tag);
  return gmres_run<T>(ctx, S, A, f, u, ctl, out, tag);
}

// ||f_seg - A u_seg||^2 per segment (FP64), written to host vector rr.
int true_residual(hz_ctx ctx, const SegHost& S, const SellOp<double>& A, const z_t* f, const z_t* u,
                  z_t* r, std::vector<double>* rr);
template <typename T>
int seg_norm2_t(hz_ctx ctx, const SegHost& S, const cx<T>* x, std::vector<double>* out);

// Segment layout of the context's single system (one segment, padded rows).
int ctx_single_seg(hz_ctx ctx, SegHost** out);
int seg_upload(hz_ctx ctx, SegHost* S, const std::string& tag);
