// Pool-bypass dispatch for BR-0 (Appendix "Pool-bypass deployment path for BR-0"): arrivals are
// placed one at a time, in order, on argmax_g F_g(s) over the workers that can take them, against
// the virtual load (every placement counts at once).  One wavefront per cluster, lane g = worker g.
// The score does not fall with the margin, and every worker whose margin the request does not exceed gives it the same
// score, its length: the best worker is the lowest index among the eligible ones with L_g <= M - s (a compare and a
// ballot), and only if there is none the lightest eligible one (a reduction).  A dependent chain bound by its
// instructions: lengths come from a register by readlane, decisions are kept in one, 64 arrivals at a time, and the chosen
// worker's words are changed by writelane, so that the arithmetic is scalar.  4096 clusters, G = 16, 60 arrivals each: 27 us
// with a score and a reduction per arrival and a second pass to commit, 21.7 with vector updates (whole pass 52.9), 17.5 so (48.9).
#include "br_device.h"
#include "br_launch.h"

// lane `lane` of old replaced by value (both uniform).  The compiler's builtin where it has one; else the intrinsic by its
// base name, without a type suffix: the compiler completes that for the type at hand, so it does not depend on how a version
// spells the overloads, and a compiler that does not know the name leaves a symbol that the device link refuses.
#if __has_builtin(__builtin_amdgcn_writelane)
__device__ __forceinline__ int br_writelane(int value, int lane, int old) { return __builtin_amdgcn_writelane(value, lane, old); }
#else
extern "C" __device__ int br_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane");
#endif

#define BR_STATB(o, inst, k) (o).stats[(int64_t)(inst) * 16 + (k)]

__global__ __launch_bounds__(256) void br_k_bypass(BrParams p, BrArr a, BrOut o) {
  const int inst = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
  if (inst >= p.N) return;
  const int lane = br_lane();
  const int G = p.G;
  int cnt = a.count[inst], q = p.qlen[inst];
  const int64_t arow = (int64_t)inst * a.arr_cap, qrow = (int64_t)inst * p.Q;

  const bool act = lane < G;
  const int64_t wrow = (int64_t)inst * G + lane;
  int nn = act ? min(max(p.n[wrow], 0), p.B) : p.B;
  int cap = p.B - nn;
  int L = act ? p.L[wrow] : BR_LOW;
  int M = br_wave_max(L);
  auto sum_loads = [&]() -> long long {
    const int L0 = act ? L : 0;
    return ((long long)br_wave_sum(L0 >> 16) << 16) + br_wave_sum(L0 & 0xffff);
  };
  cnt = br_uniform(min(max(cnt, 0), a.arr_cap));
  q = br_uniform(min(max(q, 0), p.Q));
  const long long I_before = o.stats ? (long long)G * M - sum_loads() : 0;

  int admitted = 0;
  const int top = p.W > 0 ? p.W : INT32_MAX;  // (loads stay below 2^25)
  int dropped = 0;
  // loads as the choice sees them: a worker without a free slot is beyond every bound
  int Lk = cap > 0 ? L : INT32_MAX;
  int s_next = 1, o_next = 1, id_next = 0;  // the next 64 arrivals, requested while the ones in hand are placed
  auto fetch = [&](int c) {
    const int i = c + lane;
    if (i < cnt) {
      s_next = a.s[arow + i];
      o_next = a.o[arow + i];
      id_next = a.id ? a.id[arow + i] : i;
    }
  };
  fetch(0);
  for (int c = 0; c < cnt; c += BR_WAVE) {
    const int s64 = min(max(s_next, 1), BR_MAX_S_DEV), o64 = max(o_next, 1), id64 = id_next;
    fetch(c + BR_WAVE);
    const int nc = br_uniform(min(BR_WAVE, cnt - c));
    int d64 = -1;
    for (int i = 0; i < nc; ++i) {
      const int s = __builtin_amdgcn_readlane(s64, i);
      unsigned long long pickm = br_ballot(Lk <= min(M, top) - s);
      if (__builtin_expect(pickm == 0ull, 0)) {  // no worker takes it within its margin: the lightest eligible one
        const int Le = Lk <= top - s ? Lk : INT32_MAX;  // (top - s stays below what marks a full worker)
        const int Lmin = br_wave_min(Le);
        pickm = Lmin == INT32_MAX ? 0ull : br_ballot(Le == Lmin);
      }
      if (__builtin_expect(pickm != 0ull, 1)) {
        const int g = (int)__builtin_ctzll(pickm);
        const int Lg = __builtin_amdgcn_readlane(Lk, g) + s, slot = __builtin_amdgcn_readlane(nn, g);
        M = max(M, Lg);
        d64 = br_writelane((g << 16) | slot, i, d64);
        L = br_writelane(Lg, g, L);
        Lk = br_writelane(slot + 1 < p.B ? Lg : INT32_MAX, g, Lk);
        nn = br_writelane(slot + 1, g, nn);
      }
    }
    admitted += __builtin_popcountll(br_ballot(d64 >= 0));
    // commit: placed arrivals go to their workers' lists; the rest join the waiting queue in order
    const int i = c + lane;
    const bool in = lane < nc, left = in && d64 < 0;
    const unsigned long long bal = br_ballot(left);
    const int qpos = q + br_rank_below(bal);
    int res = -2;
    if (in && d64 >= 0) {
      const int g = d64 >> 16, slot = d64 & 0xffff;
      if (g < G && slot < p.B) {
        const int64_t row = ((int64_t)inst * G + g) * p.Bs + slot;
        p.kv[row] = s64;
        p.rem[row] = o64;
      }
      res = g;
    } else if (left && qpos < p.Q) {
      p.qs[qrow + qpos] = s64;
      p.qo[qrow + qpos] = o64;
      p.qid[qrow + qpos] = id64;
      res = -1;
    }
    if (in && o.assign) o.assign[arow + i] = res;
    const int nleft = __builtin_popcountll(bal);
    const int fit = min(nleft, p.Q - q);
    dropped += nleft - fit;
    q += fit;
  }

  if (act) {
    p.L[wrow] = L;
    p.n[wrow] = nn;
  }
  const int Lmax = br_wave_max(L);
  const int Lmin = br_wave_min(act ? L : INT32_MAX);
  const int over = __builtin_popcountll(br_ballot(act && p.C > 0 && L > p.C));
  const int wide = __builtin_popcountll(br_ballot(act && L >= (1 << 25)));
  const long long sumL = o.stats ? sum_loads() : 0;
  if (lane == 0) {
    p.qlen[inst] = q;
    if (o.stats) {
      for (int k = 0; k < 16; ++k) BR_STATB(o, inst, k) = 0;
      BR_STATB(o, inst, 0) = admitted;
      BR_STATB(o, inst, 1) = q;
      BR_STATB(o, inst, 2) = dropped;
      BR_STATB(o, inst, 6) = over;
      BR_STATB(o, inst, 7) = I_before;
      BR_STATB(o, inst, 8) = (long long)G * Lmax - sumL;
      BR_STATB(o, inst, 9) = (long long)Lmax - Lmin;
      BR_STATB(o, inst, 10) = cnt;
      BR_STATB(o, inst, 12) = wide;
    }
  }
}

void br_launch_bypass(const BrParams &p, const BrArr &a, const BrOut &o, hipStream_t st) {
  const int wpb = br_waves_per_block(p.N);
  hipLaunchKernelGGL(br_k_bypass, dim3((unsigned)((p.N + wpb - 1) / wpb)), dim3(BR_WAVE * wpb), 0, st, p, a, o);
}
