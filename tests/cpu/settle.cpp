// The settle step of the BiCGStab(l) and TFQMR recursions, block by block
// with the threads in either order: the state left must be the same, and a
// segment restarts if it broke down or if all do.  DEVICE_PART is the device
// part of the solver's source.
#include DEVICE_PART

#include <cstdio>

#if defined(BICGSTABL)
using St = BlSt;
constexpr int kSums = 3;
static void start(St& S) { S.rho0 = S.omega = z_t{1.0, 0.5}; }
using Pending = BlCycle;
constexpr int kDue = kBlCycle;
static void breaks(St& S, double* sums) { S.trunc = 1; sums[0] = sums[2] = 2.0; }   // a truncated Gram matrix
#else
using St = TqSt;
constexpr int kSums = 2;
static void start(St& S) { S.rho = z_t{1.0, 0.5}; }
using Pending = TqAlpha;
constexpr int kDue = kTqAlpha;
static void breaks(St& S, double* sums) { sums[0] = sums[1] = 0.0; }                // r*^H v = 0
#endif

int main() {
  int bad = 0;
  for (int all : {0, 1})
    for (int pend : {0, 1})
      for (int brk : {0, 1}) {
        St out[2][2];
        for (int down : {0, 1}) {
          St st[2] = {};
          double part[2][kSums];
          const int seg_blk[3] = {0, 1, 2};
          for (int s = 0; s < 2; ++s) {
            for (double& v : part[s]) v = 1.5;
            start(st[s]);
            st[s].alpha = z_t{0.5, 0.25};
            st[s].due = pend ? kDue : 0;
            st[s].restart = 1 - brk;   // left by an earlier restart
            if (brk && pend) breaks(st[s], part[s]);
            if (brk && !pend) st[s].brk = 1;
          }
          Seg L;
          L.seg_blk = seg_blk;
          L.nseg = 2;
          L.nblk = 2;
          for (int b = 0; b < 2; ++b)
            fiber::run_block(b, kFinBlock, down,
                             [&] { k_step<kSums, St>(L, &part[0][0], st, st, nullptr, nullptr, Settle<Pending>{{}, all}); });
          for (int s = 0; s < 2; ++s) {
            out[down][s] = st[s];
            if (st[s].restart != (all || brk) || st[s].brk != brk || st[s].due == kDue) {
              std::printf("all %d pending %d breaks %d, threads %s: segment %d restart %d brk %d due %d\n", all, pend, brk,
                          down ? "downwards" : "upwards", s, st[s].restart, st[s].brk, st[s].due);
              ++bad;
            }
          }
        }
        if (std::memcmp(out[0], out[1], sizeof(out[0]))) {
          std::printf("all %d pending %d breaks %d: the state depends on the order of the threads\n", all, pend, brk);
          ++bad;
        }
      }
  std::printf("%d faults\n", bad);
  return bad != 0;
}
