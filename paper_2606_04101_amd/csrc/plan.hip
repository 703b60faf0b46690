// Step 2 — Algorithm 1 of the paper on the device: SolveReplication (the
// threshold bisection with greedy feasibility probes of Sec. 5.1) and
// SolveReroute (locality-first proportional split of Sec. 5.2).
//
// Feasibility is not monotone in tau (the u_min floor), so the probes must be
// exactly those of the printed sequential bisection.  They are evaluated
// speculatively across the whole chip:
//   k_plan_prep   one workgroup: lambda_e, ell_r, the rank visiting order
//                 (descending excess at any threshold is descending ell), each
//                 rank's experts by descending load, tau_lo0 and tau_hi0.
//   k_plan_round  x2 launches of 1023 one-wave workgroups.  Each workgroup
//                 replays the walk of the earlier round from its stored
//                 outcome bits, then runs the probe of its node of the next
//                 depth-10 subtree of the bisection (one probe per wave on its
//                 own SIMD, so the 1023 probes of a round run at single-probe
//                 latency).  Two rounds cover threshold ranges below 2^20,
//                 which holds for every workload here; a longer bisection
//                 ends with its remaining probes run one after another in
//                 k_plan_emit.  A probe keeps the admissible targets as a
//                 sorted list across the lanes and takes the targets an
//                 expert drains whole with one ballot over the prefix sums of
//                 their slacks; a feasible probe stores its transfers.
//   k_plan_emit   one wave per expert: walks the last round to tau* and the
//                 last feasible probe, and materialises that probe's record
//                 into its expert's row of U, its CSR host list and its rank's
//                 row of X (SolveReplication ends here).
//   k_plan_reroute one wave per expert: SolveReroute, locality first, then the
//                 sources in ascending rank order split their residual demand
//                 over the residual quotas by largest remainder.  It is a
//                 separate entry point so that callers can run it alongside
//                 the weight distribution, as the paper's forward pipeline
//                 does (Eq. 1).
#include "common.hpp"
#include "kernels.hpp"
#include "pack_core.hpp"

namespace uep {

constexpr int kMaxE = 1024;
constexpr int kMaxR = 64;
constexpr int kEntRegs = 4;                // entries per lane of the first 256 experts
constexpr int kMaxRec = 256;               // R * n_slot: one transfer per slot at most
constexpr int kDepth = 10;                 // bisection levels per round
constexpr int kNodes = (1 << kDepth) - 1;  // probes per round
constexpr int kRounds = 2;                 // 20 levels, the rest in k_plan_emit
constexpr int64_t kMaxLoad = int64_t(1) << 30;
constexpr int kNotReached = INT32_MIN;
constexpr int kPrepThreads = 1024;
constexpr int kHdr = 4 + 4 * kRounds;  // int64 header words
constexpr int kHdrSpan = 16;           // the header's share of the workspace: one 128-byte line
constexpr int kBitWords = (kNodes + 63) / 64;  // outcome bits per round
// Copies of each round's outcome words, one 128-byte line each: probe b sets
// its bit in copy b % kCopies, which spreads the round's atomics over
// kCopies lines instead of one.
constexpr int kCopies = 8;
static_assert(kHdr <= kHdrSpan && kBitWords * 8 == 128, "outcome copies are whole lines");

// The workspace is 8-byte aligned (its 64-bit words and atomics need that), so
// its 16-byte entries are declared with that alignment: still one load each.
typedef v4i v4i_ws __attribute__((aligned(8)));

struct PlanWs {
  int64_t *hdr;    // [4] tau_lo0, tau_hi0, L, status, then per round j the
                   // bisection state after rounds 0..j: lo, hi, best, probes
  uint64_t *bits;  // [kRounds][kCopies][kBitWords] feasible probes, one bit per node
  v4i_ws *rank;    // [kMaxR] i-th rank of the visiting order (descending load):
                   // its load and its largest expert load; i-th rank of the
                   // target order (ascending load): rank and load; 0 past R
  uint2 *ent;      // [E] (load, expert) in visiting order: rank by rank, each
                   // rank's main experts by descending load
  int32_t *ell;    // [R]
  int32_t *lam;    // [E] lambda_e
  int32_t *res;    // [kRounds][kNodes] probe outcome
  uint32_t *rec;   // [kRounds][kNodes][2 * RS] (e | t << 16, delta) pairs
};

static_assert(alignof(v4i_ws) == 8 && alignof(uint2) <= 8 && alignof(uint64_t) <= 8,
              "no part of the workspace asks for more than 8 bytes");

constexpr int64_t even(int64_t n) { return (n + 1) / 2 * 2; }

size_t plan_ws_bytes(int32_t R, int32_t E, int32_t NS) {
  const int64_t RS = static_cast<int64_t>(R) * NS;
  const int64_t ints = 4 * kMaxR + 2 * E + even(R) + even(E) + even(kRounds * kNodes) +
                       int64_t(kRounds) * kNodes * 2 * RS;
  return static_cast<size_t>(kHdrSpan * 8 + kRounds * kCopies * kBitWords * 8 +
                             (ints * 4 + 255) / 256 * 256);
}

static PlanWs carve(void *ws, int32_t R, int32_t E, int32_t NS) {
  (void)NS;
  PlanWs w;
  w.hdr = static_cast<int64_t *>(ws);
  w.bits = reinterpret_cast<uint64_t *>(w.hdr + kHdrSpan);
  w.rank = reinterpret_cast<v4i_ws *>(w.bits + kRounds * kCopies * kBitWords);
  w.ent = reinterpret_cast<uint2 *>(w.rank + kMaxR);
  int32_t *p = reinterpret_cast<int32_t *>(w.ent + E);
  w.ell = p;
  p += even(R);
  w.lam = p;
  p += even(E);
  w.res = p;
  p += even(kRounds * kNodes);
  w.rec = reinterpret_cast<uint32_t *>(p);
  return w;
}

struct PlanArgs {
  const int32_t *load;
  int32_t R, E, NS, nm, ncol;
  int32_t u_min;  // clamped to int32 range
  int64_t beta_num, beta_den;
  int32_t *X, *U, *hp, *hr, *hs, *q;
  int64_t *stats;
  PlanWs ws;
};

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ double readlane_d(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = readlane(static_cast<int>(b), l), hi = readlane(static_cast<int>(b >> 32), l);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<uint32_t>(lo));
}

// ---------------------------------------------------------------- prep

__global__ void __launch_bounds__(kPrepThreads) k_plan_prep(PlanArgs a) {
  __shared__ int32_t s_lam[kMaxE];
  __shared__ int32_t s_ell[kMaxR];
  __shared__ int32_t s_top[kMaxR];  // largest expert load of each rank
  __shared__ int32_t s_pos[kMaxR];  // place of each rank in the visiting order
  __shared__ int64_t s_part[kPrepThreads];
  __shared__ unsigned long long s_L;
  __shared__ int32_t s_bad;
  const int tid = threadIdx.x, lane = lane_id();
  const int R = a.R, E = a.E, nm = a.nm;
  if (tid == 0) {
    s_L = 0;
    s_bad = 0;
  }
  if (tid < kRounds * kCopies * kBitWords) a.ws.bits[tid] = 0;
  __syncthreads();
  // lambda_e: thread (part, e) sums rows part, part + parts, ... with up to
  // 16 loads in flight, the parts are then combined in LDS
  const int parts = max(1, kPrepThreads / E);
  const int pe = tid % E, part = tid / E;
  int64_t psum = 0;
  bool neg = false;
  if (part < parts) {
    for (int r0 = part; r0 < R; r0 += 16 * parts) {
      int v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int r = r0 + u * parts;
        v[u] = r < R ? a.load[static_cast<int64_t>(r) * E + pe] : 0;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        neg |= v[u] < 0;
        psum += v[u];
      }
    }
  }
  if (neg) atomicOr(&s_bad, 1);
  s_part[tid] = psum;
  {
    const int64_t w = wave_sum64(psum);
    if (lane == 0) atomicAdd(&s_L, static_cast<unsigned long long>(w));
  }
  __syncthreads();
  if (tid < E) {
    int64_t lam = 0;
    for (int p = 0; p < parts; ++p) lam += s_part[p * E + tid];
    if (lam > kMaxLoad) atomicOr(&s_bad, 1);
    s_lam[tid] = static_cast<int32_t>(min(lam, kMaxLoad));
    a.ws.lam[tid] = static_cast<int32_t>(min(lam, kMaxLoad));
  }
  __syncthreads();
  const int64_t L = static_cast<int64_t>(s_L);
  if (s_bad || L > kMaxLoad) {
    if (tid == 0) {
      a.ws.hdr[2] = L;
      a.ws.hdr[3] = ULTRAEP_EDATA;
    }
    return;
  }
  if (tid < R) {
    int s = 0;
    for (int j = 0; j < nm; ++j) s += s_lam[tid * nm + j];
    s_ell[tid] = s;
    a.ws.ell[tid] = s;
  }
  // each rank's main experts by descending load (ties: lower id)
  int pos = 0, le = 0;
  if (tid < E) {
    const int r = tid / nm;
    le = s_lam[tid];
    for (int j = r * nm; j < r * nm + nm; ++j) {
      const int lj = s_lam[j];
      pos += (lj > le) || (lj == le && j < tid);
    }
    if (pos == 0) s_top[r] = le;
  }
  __syncthreads();
  {  // ranks by descending and by ascending load (ties: lower rank): 16
     // threads per rank each compare it with 4 others, then a DPP row sum
    const int i = tid >> 4, part = tid & 15;
    int cnt = 0;  // ranks ahead in descending order << 16 | ahead in ascending
    int li = 0;
    if (i < R) {
      li = s_ell[i];
#pragma unroll
      for (int k = 0; k < kMaxR / 16; ++k) {
        const int r = part * (kMaxR / 16) + k;
        if (r < R) {
          const int lr = s_ell[r];
          const bool tie = lr == li && r < i;
          cnt += ((lr > li || tie) ? (1 << 16) : 0) + ((lr < li || tie) ? 1 : 0);
        }
      }
    }
    cnt = row_sum(cnt);
    if (part == 0) {
      const int dn = i < R ? cnt >> 16 : i, up = i < R ? cnt & 0xFFFF : i;
      if (i < R) s_pos[i] = dn;
      int2 *rk = reinterpret_cast<int2 *>(a.ws.rank);
      rk[2 * dn] = i < R ? make_int2(li, s_top[i]) : make_int2(0, 0);
      rk[2 * up + 1] = i < R ? make_int2(i, li) : make_int2(0, 0);
    }
  }
  __syncthreads();
  if (tid < E)
    a.ws.ent[s_pos[tid / nm] * nm + pos] = make_uint2(static_cast<uint32_t>(le), static_cast<uint32_t>(tid));
  if (tid < kWave) {
    const int hi = wave_max(tid < R ? s_ell[tid] : -1);
    if (tid == 0) {
      const int64_t m = (L + R - 1) / R;
      const int64_t lo = (a.beta_num * m + a.beta_den - 1) / a.beta_den;
      a.ws.hdr[0] = lo;
      a.ws.hdr[1] = hi;
      a.ws.hdr[2] = L;
      a.ws.hdr[3] = 0;
    }
  }
}

// ---------------------------------------------------------------- rounds

// DPP wave_shl:1 - lane i receives lane i+1 (lane 63 keeps its value)
__device__ __forceinline__ int wave_shl1(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x130, 0xF, 0xF, false);
}

// Greedy feasibility probes of SolveReplication at threshold tau (Sec. 5.1),
// one wave each.  Lane i holds the excess over tau of the i-th rank of the
// visiting order (descending load, ties to the lower rank) and the i-th rank of
// ascending load with that load.  A probe returns the number of accepted
// transfers, recorded as (e | t << 16, delta) in acceptance order, or -1 if the
// threshold is infeasible.
//
// The admissible targets (slack > 0, a free slot) form a list sorted by
// slack descending, rank ascending, one per lane from the head h on.  It
// starts as the ranks of load below tau in ascending load order.  With the
// slacks m in lanes and their inclusive prefix P (B = P before the head),
// an expert that has to shed need = min(excess, its load) takes whole every
// target from the head whose running slack stays below need (one ballot),
// then the rest d from the next target.  A whole transfer is bound by the
// target's slack, so one below u_min makes the probe infeasible, and the
// target leaves the list, exactly as transfer-by-transfer evaluation finds.
// The experts are visited in one flat loop (rank by rank, experts by
// descending load) with scalar loop state.

// A probe is one dependent chain on one wave, and on this chip an instruction
// of such a chain costs 8 cycles, a readlane with a computed lane or a
// ballot with its population count about 35, and a branch about 25, so the
// loops below keep a visit to one ballot, a few readlanes and three branches:
// the excess x and the first expert's need of every overloaded rank sit in
// lanes, the failure tests are one sign test, and an expert is recorded by its
// place in the visiting order.  A visit takes about 200-240 ns (420 ns with a
// branch per test and an LDS fetch of the experts per rank).  Code that runs
// once costs about 85 ns per 64 bytes to fetch, so it is kept short.
struct Probe {
  int tau, lane;
  int nover;         // overloaded ranks: the first nover of the visiting order
  int xv, nv;        // lane i: excess of the i-th, and min(excess, largest load)
  int as_r, as_l;    // lane i: i-th target rank and its load
  const uint2 *ent;  // (load, expert) in visiting order
};

// After a visit that left x of the excess: the rank's next expert, or the
// next rank, whose excess and need are xn and nn.  ok counts up to 0 ranks
// left and is 1 when a rank's experts ran out.
__device__ __forceinline__ void next_visit(const Probe &s, int nm, int &x, int &need, int &p,
                                           int &end, int &oi, int &ok, int xn, int nn) {
  if (x > 0) {
    ++p;
    need = min(x, uni(static_cast<int>(s.ent[min(p, end - 1)].x)));
    ok = p == end ? 1 : ok;
  } else {
    x = xn;
    need = nn;
    p = end;
    end += nm;
    ++oi;
    ++ok;
  }
}

// One redundant slot per rank: every transfer uses up its target, so
// transfer k goes to the k-th listed target and its record stays in lane k.
// The slacks never change, so P is the fixed inclusive prefix of the list
// (m and Q = P - m its slacks and exclusive prefix) and the lanes with
// P < B + need are the prefix [0, hh) (lanes before the head have P <= B, and
// the lanes past the list have P = the total, which is below B + need only
// if every target is whole): the whole targets are [h, hh).  The list is
// sorted, so a whole target below u_min shows as hh past the nbig targets of
// at least u_min.
template <int kSite>
__device__ __forceinline__ int probe_one_slot(const PlanArgs &a, const Probe &s, uint2 *rec) {
  const int nm = a.nm, u_min = a.u_min, lane = s.lane;
  const bool tv = lane < a.R && s.as_l < s.tau;
  const int m = tv ? s.tau - s.as_l : 0;
  // inclusive prefix of the slacks: each is below 2^25, the sum below 2^31
  const int P = wave_scan_incl(m), Q = P - m;
  const int last = __popcll(ballot(tv)) - 1, nbig = __popcll(ballot(tv && m >= u_min));
  int rec_p = 0, rec_d = 0;
  int h = 0, B = 0;  // head, slack before it
  int oi = 0, p = 0, end = nm, x = readlane(s.xv, 0), need = readlane(s.nv, 0), ok = -s.nover;
  while (ok < 0) {
    const int xn = readlane(s.xv, (oi + 1) & (kWave - 1)), nn = readlane(s.nv, (oi + 1) & (kWave - 1));
    const int hh = __popcll(ballot(static_cast<uint32_t>(P) < static_cast<uint32_t>(B + need)));
    const int Qh = readlane(Q, hh & (kWave - 1)), mh = readlane(m, hh & (kWave - 1));
    const int d = need - (Qh - B);  // the rest after the whole targets, at most mh
    x -= Qh - B;
    // an expert with no load left, no target for the rest (every target
    // whole), a whole target below u_min, or a rest below u_min that is not
    // only this expert's shortfall (max(d, min(x, mh)) < u_min)
    const int bad = (need - 1) | (min(max(h, nbig), last) - hh) | (max(d, min(x, mh)) - u_min);
    // the whole targets and, when the rest is taken, target hh
    const int take = 1 + ((d - u_min) >> 31);  // d >= u_min, in scalar integers
    const bool mine = static_cast<uint32_t>(lane - h) < static_cast<uint32_t>(hh - h + take);
    rec_p = mine ? p : rec_p;
    rec_d = mine ? (lane == hh ? d : m) : rec_d;
    x -= d & -take;
    B = Qh + (mh & -take);
    h = hh + take;
    next_visit(s, nm, x, need, p, end, oi, ok, xn, nn);
    ok = bad < 0 ? 1 : ok;
  }
  if (ok > 0) return -1;
  if (lane < h)
    rec[lane] = make_uint2(s.ent[rec_p].y | (static_cast<uint32_t>(s.as_r) << 16),
                           static_cast<uint32_t>(rec_d));
  return h;
}

// Several redundant slots per rank: a target that keeps slack and a free
// slot after an expert's last (partial) transfer moves back to its place in
// the list; the lanes it passes shift down by one (DPP) and the prefixes are
// patched.  The list entries are packed keys (slack << 6) | (63 - rank), in
// descending order over all lanes (the consumed ones before the head keep
// theirs), so one ballot and a population count find places in it.  In the
// loop a record is (place of the expert, key of the transfer: amount << 6 |
// 63 - rank), written to s_rec by the lanes of the targets themselves; the
// records are put into the common form once the probe has succeeded.
template <int kSite>
__device__ __forceinline__ int probe_multi(const PlanArgs &a, const Probe &s, uint2 *s_rec,
                                           uint2 *rec) {
  const int NS = a.NS, nm = a.nm, u_min = a.u_min, lane = s.lane;
  const bool tv = lane < a.R && s.as_l < s.tau && NS > 0;
  int m = tv ? s.tau - s.as_l : 0;
  int key = tv ? (m << 6) | (kWave - 1 - s.as_r) : 0;
  int used = 0;
  int P = wave_scan_incl(m), Q = P - m;
  const int last = __popcll(ballot(tv)) - 1;  // the list's length never changes
  int nbig = __popcll(ballot(tv && m >= u_min));
  int h = 0, B = 0, n = 0;
  int oi = 0, p = 0, end = nm, x = readlane(s.xv, 0), need = readlane(s.nv, 0), ok = -s.nover;
  while (ok < 0) {
    const int xn = readlane(s.xv, (oi + 1) & (kWave - 1)), nn = readlane(s.nv, (oi + 1) & (kWave - 1));
    const int hh = __popcll(ballot(static_cast<uint32_t>(P) < static_cast<uint32_t>(B + need)));
    const int Qh = readlane(Q, hh & (kWave - 1)), kh = readlane(key, hh & (kWave - 1));
    const int uh = readlane(used, hh & (kWave - 1)) + 1;
    const int mh = kh >> 6;
    const int d = need - (Qh - B);
    x -= Qh - B;
    // as in probe_one_slot
    const int bad = (need - 1) | (min(max(h, nbig), last) - hh) | (max(d, min(x, mh)) - u_min);
    const int take = 1 + ((d - u_min) >> 31);  // d >= u_min, in scalar integers
    {  // the other lanes write a spare area past the records (n <= kMaxRec)
      const int o = lane - h;
      const int at = static_cast<uint32_t>(o) < static_cast<uint32_t>(hh - h + take)
                         ? n + o
                         : kMaxRec + lane;
      s_rec[at] = make_uint2(
          static_cast<uint32_t>(p),
          static_cast<uint32_t>(lane == hh ? (d << 6) | (key & (kWave - 1)) : key));
    }
    n += hh - h + take;
    x -= d & -take;
    // out of slack or slots: target hh leaves the list, else a used one goes
    // back to its place, after every key still larger
    const int out = take & (((mh - d - 1) >> 31) | ((NS - 1 - uh) >> 31));
    B = Qh + (mh & -out);
    h = hh + out;
    if (take > out) {
      const int nk = ((mh - d) << 6) | (kh & (kWave - 1));
      const int to = __popcll(ballot(key > nk)) - 1;
      const bool mv = static_cast<uint32_t>(lane - hh) < static_cast<uint32_t>(to - hh);
      const int ks = wave_shl1(key), us = wave_shl1(used), ps = wave_shl1(P);
      key = mv ? ks : (lane == to ? nk : key);
      used = mv ? us : (lane == to ? uh : used);
      P = mv ? ps - mh : (lane >= to ? P - d : P);
      m = key >> 6;
      Q = P - m;
      nbig = __popcll(ballot(m >= u_min));
    }
    next_visit(s, nm, x, need, p, end, oi, ok, xn, nn);
    ok = bad < 0 ? 1 : ok;
  }
  if (ok > 0) return -1;
  __syncthreads();
  for (int i = lane; i < n; i += kWave) {
    const uint2 v = s_rec[i];
    rec[i] = make_uint2(s.ent[v.x].y | ((kWave - 1 - (v.y & (kWave - 1))) << 16), v.y >> 6);
  }
  return n;
}

// The same probe for slacks of 25 bits or more: lane t holds rank t's slack
// and slot count, and the target is a wave max plus a ballot for the lowest
// rank among ties.
template <int kSite>
__device__ __forceinline__ int probe_wide(const PlanArgs &a, const Probe &s, uint2 *rec) {
  const int lane = s.lane;
  int slk = lane < a.R ? max(s.tau - a.ws.ell[lane], 0) : 0;
  int used = 0;
  int n = 0;
  for (int oi = 0; oi < s.nover; ++oi) {
    int exc = readlane(s.xv, oi);
    for (int j = 0; j < a.nm && exc > 0; ++j) {
      const uint2 v = s.ent[oi * a.nm + j];
      const int e = uni(static_cast<int>(v.y));
      int cap = uni(static_cast<int>(v.x));
      while (exc > 0 && cap > 0) {
        const bool ok = slk > 0 && used < a.NS;
        const int sv = ok ? slk : 0;
        const int m = wave_max(sv);
        if (m == 0) return -1;
        const int ts = uni(__ffsll(static_cast<unsigned long long>(ballot(sv == m && ok))) - 1);
        const int d = min(min(exc, m), cap);
        if (d < a.u_min) {
          if (min(exc, m) < a.u_min) return -1;
          break;
        }
        if (lane == ts) {
          slk -= d;
          ++used;
        }
        if (lane == 0)
          rec[n] = make_uint2(static_cast<uint32_t>(e) | (static_cast<uint32_t>(ts) << 16),
                              static_cast<uint32_t>(d));
        ++n;
        exc -= d;
        cap -= d;
      }
    }
    if (exc > 0) return -1;
  }
  return n;
}

// One probe at tau with the variant the thresholds and slots allow; a
// feasible one leaves its transfers in rec as (e | rank << 16, amount).  rk =
// this lane's entry of PlanWs::rank.  At least one rank is not overloaded
// (tau is no less than the mean), so nover < R.  kSite gives every call site
// its own copy: shared by two kernels, the compiler loses sight of the
// probes' scalar loop state.
template <int kSite>
__device__ __forceinline__ int run_probe(const PlanArgs &a, bool packed, int tau, int lane, v4i rk,
                                         const uint2 *ent, uint2 *s_rec, uint2 *rec) {
  Probe s;
  s.tau = tau;
  s.lane = lane;
  s.xv = rk.x - tau;
  s.nv = min(s.xv, rk.y);
  s.nover = __popcll(ballot(lane < a.R && s.xv > 0));
  s.as_r = rk.z;
  s.as_l = rk.w;
  s.ent = ent;
  if (!packed) return probe_wide<kSite>(a, s, rec);
  if (a.NS == 1) return probe_one_slot<kSite>(a, s, rec);
  return probe_multi<kSite>(a, s, s_rec, rec);
}

// Bisection state before round rd: the initial interval, or the state
// after round rd - 1 that round rd's first workgroup published.
struct BisState {
  int64_t lo, hi;
  int best;   // last feasible probe: round * kNodes + node, or -1
  int probes; // probes of the sequential bisection so far
};

// One pointer and four loads whatever rd is (no branch that would make the
// loads wait for each other).
__device__ __forceinline__ BisState state_before(const PlanArgs &a, int rd) {
  const int64_t *h = a.ws.hdr + (rd == 0 ? 0 : 4 + 4 * (rd - 1));
  const int64_t lo = h[0], hi = h[1], best = h[2], probes = h[3];
  return {lo, hi, rd == 0 ? -1 : static_cast<int>(best), rd == 0 ? 0 : static_cast<int>(probes)};
}

// Round rd's outcome words: the kCopies copies of 32-bit word w into lane w
// (the lanes past the last word read it too).  No branch between the loads,
// so that they stay in flight together with the kernel's other inputs.
__device__ __forceinline__ void outcome_load(const PlanArgs &a, int rd, uint32_t (&v)[kCopies]) {
  const uint32_t *w = reinterpret_cast<const uint32_t *>(a.ws.bits + rd * kCopies * kBitWords) +
                      min(lane_id(), 2 * kBitWords - 1);
#pragma unroll
  for (int c = 0; c < kCopies; ++c) v[c] = w[c * 2 * kBitWords];
}

// The OR of the copies: word w in lane w.
__device__ __forceinline__ int outcome_or(const uint32_t (&v)[kCopies]) {
  uint32_t bw = 0;
#pragma unroll
  for (int c = 0; c < kCopies; ++c) bw |= v[c];
  return static_cast<int>(bw);
}

// The sequential bisection through round rd's depth-kDepth subtree, from
// state st, over the round's outcome bits (32-bit word w in lane w).  An
// interval that is not empty lies within [0, 2^30], so it is walked in 32
// bits, without branches on the outcomes: 10 levels take 0.8 us.
__device__ __forceinline__ void walk_bits(int bw, int rd, BisState &st) {
  if (st.lo >= st.hi) return;
  int lo = static_cast<int>(st.lo), hi = static_cast<int>(st.hi);
  int node = 0, best = -1, d = 0;
#pragma unroll 1
  for (; d < kDepth && lo < hi; ++d) {
    const int mid = (lo + hi) >> 1;
    const int bit = static_cast<int>(static_cast<uint32_t>(readlane(bw, node >> 5)) >> (node & 31)) & 1;
    best = bit ? node : best;
    hi = bit ? mid : hi;
    lo = bit ? lo : mid + 1;
    node = 2 * node + 2 - bit;
  }
  st.lo = lo;
  st.hi = hi;
  st.best = best >= 0 ? rd * kNodes + best : st.best;
  st.probes += d;
}

__global__ void __launch_bounds__(kWave) k_plan_round(PlanArgs a, int round) {
  __shared__ uint2 s_ent[kMaxE];
  __shared__ uint2 s_rec[kMaxRec + kWave];
  const int lane = threadIdx.x, b = blockIdx.x;
  const int E = a.E, RS = a.R * a.NS;
  // every input is requested up front, with no branch between the loads
  // (indices clamped into range, values masked afterwards), so the round
  // waits for memory once: the state before the previous round and that
  // round's outcome bits (round 0 reads the last round's words, which
  // nothing writes before that round), the rank orders and the visiting order
  const int64_t status = a.ws.hdr[3];
  const bool packed = a.ws.hdr[1] < (int64_t(1) << 25);
  BisState st = state_before(a, round > 0 ? round - 1 : 0);
  uint32_t bv[kCopies];
  outcome_load(a, round > 0 ? round - 1 : kRounds - 1, bv);
  const v4i rk = a.ws.rank[lane];
  uint2 ent[kEntRegs], more[kMaxE / kWave - kEntRegs];
#pragma unroll
  for (int u = 0; u < kEntRegs; ++u) ent[u] = a.ws.ent[min(u * kWave + lane, E - 1)];
  if (E > kEntRegs * kWave) {
#pragma unroll
    for (int u = kEntRegs; u < kMaxE / kWave; ++u)
      more[u - kEntRegs] = a.ws.ent[min(u * kWave + lane, E - 1)];
  }
  // the loads above are issued before the status test (which the compiler
  // would otherwise move ahead of them, waiting for the header first)
  asm volatile("" ::: "memory");
  if (status != 0) return;
#pragma unroll
  for (int u = 0; u < kEntRegs; ++u) s_ent[u * kWave + lane] = ent[u];
  if (E > kEntRegs * kWave) {
#pragma unroll
    for (int u = kEntRegs; u < kMaxE / kWave; ++u) s_ent[u * kWave + lane] = more[u - kEntRegs];
  }
  if (round > 0) {  // every workgroup walks the previous round; the first publishes it
    walk_bits(outcome_or(bv), round - 1, st);
    if (b == 0 && lane == 0) {
      int64_t *h = a.ws.hdr + 4 + 4 * (round - 1);
      h[0] = st.lo;
      h[1] = st.hi;
      h[2] = st.best;
      h[3] = st.probes;
    }
  }
  if (st.lo >= st.hi) return;  // the bisection has ended
  // this workgroup's node of the round's subtree
  int lo = static_cast<int>(st.lo), hi = static_cast<int>(st.hi);
  const int id = b + 1, depth = 31 - __clz(id);
  // (an interval that has become empty stays empty)
#pragma unroll 1
  for (int bit = depth - 1; bit >= 0; --bit) {
    const int mid = (lo + hi) >> 1;
    const bool right = (id >> bit) & 1;  // that probe failed
    lo = right ? mid + 1 : lo;
    hi = right ? hi : mid;
  }
  int n = kNotReached;
  if (lo < hi) {
    __syncthreads();
    uint2 *rec = reinterpret_cast<uint2 *>(a.ws.rec) + (static_cast<int64_t>(round) * kNodes + b) * RS;
    n = run_probe<0>(a, packed, (lo + hi) >> 1, lane, rk, s_ent, s_rec, rec);
  }
  if (lane == 0) {
    a.ws.res[round * kNodes + b] = n;
    if (n >= 0)
      atomicOr(a.ws.bits + (round * kCopies + (b % kCopies)) * kBitWords + (b >> 6),
               uint64_t(1) << (b & 63));
  }
}

// ---------------------------------------------------------------- reroute

// DPP wave_shr:1 - lane i receives lane i-1 (lane 0 keeps its value)
__device__ __forceinline__ int wave_shr1(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138, 0xF, 0xF, false);
}

// Two hosts (home first, one replica): with residual quotas (u0, u1) and
// residual demand D = u0 + u1, a source with demand lh gives host 0
// b0 = floor(lh * u0 / D) plus the one leftover unit when its remainder is
// at least the other host's (ties go to the earlier host), i.e.
// q0 = floor((lh * u0 + D / 2) / D).  The sources run in ascending order with
// the state u0 carried from lane r to lane r + 1 by a DPP shift, so the chain
// has no scalar round trip and no branch.  Lane r returns q0 of source r.
//   kExact: lh * u0 + D / 2 < 2^52 (total load below 2^26), so the fp64
//   numerator is exact and one correction of the reciprocal estimate
//   gives the floor; otherwise the same in int64.
template <bool kExact>
__device__ __forceinline__ int split_two(int lamhat, int Dr, int u0_init, int R) {
  const bool act = lamhat > 0;
  const double lhd = static_cast<double>(lamhat);
  const double Dd = act ? static_cast<double>(Dr) : 1.0;
  const double rD = 1.0 / Dd;
  const double half = 0.5 * Dd;
  int u0 = u0_init, qout = 0;
  const int lane = lane_id();
  for (int r = 0; r < R; ++r) {
    int q;
    if (kExact) {
      const double N = __builtin_fma(lhd, static_cast<double>(u0), half);
      const double t = __builtin_trunc(N * rD);
      const double rr = __builtin_fma(-t, Dd, N);
      q = static_cast<int>(t) + (rr >= Dd ? 1 : 0) - (rr < 0.0 ? 1 : 0);
    } else {
      const int64_t D = act ? Dr : 1;
      const int64_t N = 2 * static_cast<int64_t>(lamhat) * u0 + D;
      int64_t t = static_cast<int64_t>(static_cast<double>(N) * (0.5 * rD));
      const int64_t rr = N - t * 2 * D;
      t += (rr >= 2 * D ? 1 : 0) - (rr < 0 ? 1 : 0);
      q = static_cast<int>(t);
    }
    qout = lane == r ? q : qout;
    u0 = wave_shr1(u0 - q);
  }
  return qout;
}

// LDS of one expert's SolveReroute: its hosts' ranks (kWave), then the
// shares of the lane-mirrored split (8 hosts x kMaxR sources, and a spare
// area for the lanes that are not host slots)
constexpr int kRrLds = kWave + 8 * kMaxR + kWave;

// DPP row_ror:k - within each row of 16 lanes, a rotation by k lanes (every
// lane has a source, so no old value is needed and the move folds into the
// instruction that consumes it)
template <int K>
__device__ __forceinline__ int row_ror(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x120 + K, 0xF, 0xF, true);
}

// 1 when the host k rotations away has the larger key (its key minus ours
// is positive; keys are below 2^29, so the difference cannot wrap)
template <int K>
__device__ __forceinline__ int ahead(int key) {
  return static_cast<int>(static_cast<uint32_t>(key - row_ror<K>(key)) >> 31);
}

// Sum over the kH host slots of a row that repeats them with period kH.
template <int kH>
__device__ __forceinline__ int host_sum(int b) {
  int sb = kH == 8 ? b + row_ror<4>(b) : b;
  sb += row_ror<2>(sb);
  return sb + row_ror<1>(sb);
}

// Number of the kH - 1 other host slots whose key is larger.
template <int kH>
__device__ __forceinline__ int rank_of(int key) {
  if (kH == 4) return (ahead<1>(key) + ahead<2>(key)) + ahead<3>(key);
  return (ahead<1>(key) + ahead<2>(key)) + (ahead<3>(key) + ahead<4>(key)) +
         ((ahead<5>(key) + ahead<6>(key)) + ahead<7>(key));
}

// Lowest set bit of m (63 when there is none).
__device__ __forceinline__ int first_bit(uint64_t m) {
  return __builtin_ctzll(m | (uint64_t(1) << 63));
}

// Three to eight hosts, total load below 2^26: host i sits in lane i and in
// its mirror lane i + 8, so that rotations by 1 .. 7 within the 16 lanes of
// row 0 bring every other host's value to every host lane with no scalar
// round trip.  Lanes of host slots i >= nh, and every lane past 15, hold a
// zero residual quota (so a zero share and a zero remainder).  Per source
// with residual demand, in ascending order:
//   b_i = floor(lh * u_i / D) and rem_i exactly: the estimate
//         trunc((lh / D) * u_i) in fp64 is within one of the floor (the
//         quotient is below 2^26), and the remainder for the estimate lies
//         in (-D, 2D), so wrapping 32-bit arithmetic gives it exactly and
//         one correction gives both,
//   left = lh - sum_i b_i, the sum taken by three rotations (4, 2, 1),
//   host i gets one of the left units iff fewer than `left` hosts are ahead
//   of it in (remainder descending, host ascending): the keys rem * 8 +
//   (7 - i) order exactly so, and a zero-quota slot i >= nh is never ahead
//   of a host (its key 7 - i is below every host's),
// then u_i -= q_i.  The shares go to s_q[r * 8 + i] (lanes past 7 write a
// spare area); afterwards lane r writes source r's row of Q, adding the
// locality share of the host that is r itself.  s_hosts lists the hosts'
// ranks, s_q holds kRrLds - kWave ints.  kSmall (the expert's residual
// demand below 2^19): the same with an fp32 estimate and 24-bit products.
// kH = 4 (at most four hosts): the slots repeat with period 4 in row 0
// (lanes i, i + 4, i + 8, i + 12), so three rotations rank the keys
// rem * 4 + (3 - i) and two sum the floors.
template <int kH, bool kSmall>
__device__ __forceinline__ void split_lanes(int lane, int nh, int lamhat_r, int Dr, int loc_r,
                                            int R, int64_t ncol, int32_t *qbase,
                                            const int32_t *s_hosts, int32_t *s_q,
                                            int ures_r) {
  static_assert(kH == 4 || kH == 8, "host slots mirror with period 4 or 8 in a row");
  const int hidx = lane & (kH - 1);
  const bool slot = lane < 16 && hidx < nh;
  int ures = __shfl(ures_r, slot ? s_hosts[hidx] : 0);
  ures = slot ? ures : 0;
  const int qstep = lane < kH ? 8 : 0;
  const int qoff = lane < kH ? lane : 8 * kMaxR + lane;
  uint64_t act = ballot(lane < R && lamhat_r > 0);
  const int key_lo = kH - 1 - hidx;
  if (kSmall) {
    // Residual demand below 2^19: c = (lh / D)(1 - 2^-20) rounded to fp32
    // makes y = fl(c * u) fall strictly below x = lh * u / D and above
    // x - 1 (relative errors below 2^-20 + 2^-23 on x < 2^19), so trunc(y)
    // is floor(x) or floor(x) - 1, and the remainder lh * u - trunc(y) * D
    // lies in [0, 2D): 24-bit products wrapped to 32 bits give it exactly,
    // and one subtraction with a min gives the floor's remainder
    const float c_r = lamhat_r > 0 ? static_cast<float>(static_cast<double>(lamhat_r) *
                                                        (1.0 - 0x1p-20) / static_cast<double>(Dr))
                                   : 0.0f;
    const int nD_r = -Dr;
    // a source's scalars are read one step ahead: the lane reads then run
    // beside the vector chain of the source before it
    int r = first_bit(act), lh = readlane(lamhat_r, r), nD = readlane(nD_r, r);
    int cb = readlane(__float_as_int(c_r), r);
    while (act) {
      act &= act - 1;
      const int rn = first_bit(act);
      const int lhn = readlane(lamhat_r, rn), nDn = readlane(nD_r, rn);
      const int cbn = readlane(__float_as_int(c_r), rn);
      const int be = static_cast<int>(__int_as_float(cb) * static_cast<float>(ures));
      const int re = static_cast<int>(static_cast<uint32_t>(__mul24(be, nD)) +
                                      __umul24(lh, static_cast<uint32_t>(ures)));
      const int t = re + nD;  // re - D, in [-D, D)
      const int rem = static_cast<int>(min(static_cast<uint32_t>(re), static_cast<uint32_t>(t)));
      const int b = be + 1 + (t >> 31);
      const int left = lh - host_sum<kH>(b);
      const int rk = rank_of<kH>((rem << (kH == 8 ? 3 : 2)) | key_lo);
      const int qi = b + ((slot && rk < left) ? 1 : 0);
      ures -= qi;
      s_q[r * qstep + qoff] = qi;
      r = rn;
      lh = lhn;
      nD = nDn;
      cb = cbn;
    }
  } else {
    // lh / D of source `lane`
    const double c_r = lamhat_r > 0 ? static_cast<double>(lamhat_r) / static_cast<double>(Dr) : 0.0;
    while (act) {
      const int r = __ffsll(static_cast<unsigned long long>(act)) - 1;
      act &= act - 1;
      const int lh = readlane(lamhat_r, r);
      const int D = readlane(Dr, r);
      const double c = readlane_d(c_r, r);
      const int be = static_cast<int>(c * static_cast<double>(ures));
      const int re = static_cast<int>(static_cast<uint32_t>(lh) * static_cast<uint32_t>(ures) -
                                      static_cast<uint32_t>(be) * static_cast<uint32_t>(D));
      const bool lo = re < 0, hi = re >= D;
      const int b = lo ? be - 1 : (hi ? be + 1 : be);
      const int rem = lo ? re + D : (hi ? re - D : re);
      const int left = lh - host_sum<kH>(b);
      const int rk = rank_of<kH>((rem << (kH == 8 ? 3 : 2)) | key_lo);
      const int qi = b + ((slot && rk < left) ? 1 : 0);
      ures -= qi;
      s_q[r * qstep + qoff] = qi;
    }
  }
  if (lane < R) {
    const bool dem = lamhat_r > 0;
    int32_t *qrow = qbase + static_cast<int64_t>(lane) * ncol;
    for (int i = 0; i < nh; ++i)
      qrow[i] = (dem ? s_q[lane * 8 + i] : 0) + (s_hosts[i] == lane ? loc_r : 0);
  }
}

// Any number of hosts: lane i is host i (home first, then replicas by
// ascending rank) with residual quota ures; the sources run in ascending
// order, each splitting its residual demand by largest remainder.  Writes
// q of source r, host `lane` to qcol[r * ncol].  Used above eight hosts or
// when the total load reaches 2^26.
template <bool kExact, bool kOneRow>
__device__ __forceinline__ void split_many(int lane, int nh, int lamhat_r, int Dr, int ures, int R,
                           int64_t ncol, int32_t *qcol, int t_i, int qloc_i) {
  const double rDr = lamhat_r > 0 ? 1.0 / static_cast<double>(Dr) : 0.0;
  const bool host = lane < nh;
  for (int r = 0; r < R; ++r) {
    const int lh = readlane(lamhat_r, r);
    int qi = 0;
    if (lh > 0) {
      const int D = readlane(Dr, r);
      const double rD = readlane_d(rDr, r);
      // floor(lh * ures / D) and its remainder, exact after one correction
      int b, rem;
      if (kExact) {  // lh * ures < 2^52
        const double Dd = static_cast<double>(D);
        const double pr = static_cast<double>(lh) * static_cast<double>(ures);
        const double bq = __builtin_trunc(pr * rD);
        const double rd = __builtin_fma(-bq, Dd, pr);
        const int lo = rd < 0.0 ? 1 : 0, hi = rd >= Dd ? 1 : 0;
        b = static_cast<int>(bq) + hi - lo;
        rem = static_cast<int>(rd) + (lo ? D : 0) - (hi ? D : 0);
      } else {
        b = static_cast<int>(static_cast<double>(lh) * static_cast<double>(ures) * rD);
        int64_t rm = static_cast<int64_t>(lh) * ures - static_cast<int64_t>(b) * D;
        const bool lo = rm < 0, hi = rm >= D;
        b += lo ? -1 : (hi ? 1 : 0);
        rm += lo ? D : (hi ? -D : 0);
        rem = static_cast<int>(rm);
      }
      const int left = lh - (kOneRow ? readlane(row_sum(b), 0) : wave_sum(b));
      // the `left` hosts with the largest remainders (ties: earlier host)
      int rk = 0;
      for (int j = 0; j < nh; ++j) {
        const int rj = readlane(rem, j);
        rk += (rj > rem) || (rj == rem && j < lane);
      }
      qi = b + ((host && rk < left) ? 1 : 0);
      ures -= qi;
    }
    if (host) qcol[r * ncol] = qi + (t_i == r ? qloc_i : 0);
  }
}

// SolveReroute for expert e, run by one wave.  The hosts of e are its home
// and every other rank with a positive quota (a replica's quota is at least
// u_min), so the expert's row of U (u_r: its quota on rank `lane`), its load
// column (lam_r), its first CSR column j0 and the number of CSR entries are
// all the inputs.  Locality first: a host consumes its own tokens up to its
// quota; the residual demands are then split over the residual quotas.
__device__ __forceinline__ void reroute_expert(const PlanArgs &a, int e, int j0, int total, int lam_r,
                               int u_r, int64_t L, int32_t *s_t) {
  const int lane = lane_id();
  const int R = a.R, E = a.E;
  const int64_t ncol = a.ncol;
  const int h = e / a.nm;
  const uint64_t rep = ballot(lane < R && lane != h && u_r > 0);
  const int nh = 1 + __popcll(rep);
  if (j0 < e || j0 + nh > total || total > ncol) {  // not a plan of this group
    if (lane == 0) a.stats[6] = ULTRAEP_EDATA;
    return;
  }
  const int loc_r = min(lam_r, u_r);  // 0 on ranks that do not host e
  const int lamhat_r = lam_r - loc_r;
  const int ures_r = u_r - loc_r;
  // residual demand still to place when source r comes: D0 minus the
  // demand of the sources before it
  const int incl = wave_scan_incl(lamhat_r);
  const int D0 = readlane(incl, kWave - 1);
  const int Dr = D0 - (incl - lamhat_r);
  const bool exact = L < (int64_t(1) << 26);
  int32_t *qrow = a.q + static_cast<int64_t>(lane) * ncol;
  if (nh == 1) {
    if (lane < R) qrow[j0] = lam_r;
  } else if (nh == 2) {
    const int t = __ffsll(static_cast<unsigned long long>(rep)) - 1;
    const int u0 = readlane(ures_r, h);
    const int q0 = exact ? split_two<true>(lamhat_r, Dr, u0, R)
                         : split_two<false>(lamhat_r, Dr, u0, R);
    if (lane < R) {
      qrow[j0] = q0 + (lane == h ? loc_r : 0);
      qrow[j0 + 1] = lamhat_r - q0 + (lane == t ? loc_r : 0);
    }
  } else {
    if (lane == h) s_t[0] = h;
    if ((rep >> lane) & 1) s_t[1 + popc_below(rep)] = lane;
    __syncthreads();
    if (exact && nh <= 8) {
      int32_t *qb = a.q + j0, *s_q = s_t + kWave;
      if (D0 < (1 << 19)) {
        if (nh <= 4)
          split_lanes<4, true>(lane, nh, lamhat_r, Dr, loc_r, R, ncol, qb, s_t, s_q, ures_r);
        else
          split_lanes<8, true>(lane, nh, lamhat_r, Dr, loc_r, R, ncol, qb, s_t, s_q, ures_r);
      } else {
        split_lanes<8, false>(lane, nh, lamhat_r, Dr, loc_r, R, ncol, qb, s_t, s_q, ures_r);
      }
      for (int j = total + e; j < ncol; j += E)
        if (lane < R) qrow[j] = 0;
      return;
    }
    const int t_i = lane < nh ? s_t[lane] : 0;
    // every lane takes part in the shuffles: a lane reads only from lanes
    // that execute the same shuffle
    const int ures_t = __shfl(ures_r, t_i);
    const int qloc_i = __shfl(loc_r, t_i);
    const int ures_i = lane < nh ? ures_t : 0;
    int32_t *qcol = a.q + j0 + lane;
    if (exact && nh <= 16)
      split_many<true, true>(lane, nh, lamhat_r, Dr, ures_i, R, ncol, qcol, t_i, qloc_i);
    else if (exact)
      split_many<true, false>(lane, nh, lamhat_r, Dr, ures_i, R, ncol, qcol, t_i, qloc_i);
    else if (nh <= 16)
      split_many<false, true>(lane, nh, lamhat_r, Dr, ures_i, R, ncol, qcol, t_i, qloc_i);
    else
      split_many<false, false>(lane, nh, lamhat_r, Dr, ures_i, R, ncol, qcol, t_i, qloc_i);
  }
  // CSR padding columns of Q
  for (int j = total + e; j < ncol; j += E)
    if (lane < R) qrow[j] = 0;
}

// ---------------------------------------------------------------- emit

// kReroute: the same workgroup then runs SolveReroute for its expert from
// the values it has just produced (ultraep_plan's single-launch ending).
template <bool kReroute>
__global__ void __launch_bounds__(kWave) k_plan_emit(PlanArgs a) {
  __shared__ int32_t s_t[kRrLds];
  __shared__ uint32_t s_et[kMaxRec];
  __shared__ int32_t s_d[kMaxRec];
  __shared__ int32_t s_ht[kMaxR];  // hosts of this expert: rank
  __shared__ int32_t s_hu[kMaxR];  //                       quota
  __shared__ int32_t s_fan[kMaxE];
  const int e = blockIdx.x, lane = threadIdx.x;
  const int R = a.R, E = a.E, NS = a.NS, nm = a.nm, ncol = a.ncol, RS = R * NS;
  const int64_t status = a.ws.hdr[3], L = a.ws.hdr[2];
  const int64_t lo0 = a.ws.hdr[0], hi0 = a.ws.hdr[1];
  BisState fin = state_before(a, kRounds - 1);
  uint32_t bv[kCopies];
  outcome_load(a, kRounds - 1, bv);
  const int lam_e = a.ws.lam[e];
  const int lam_v = kReroute ? a.load[static_cast<int64_t>(min(lane, R - 1)) * E + e] : 0;
  asm volatile("" ::: "memory");  // the loads above go out before the status test
  const int lam_r = lane < R ? lam_v : 0;
  if (status != 0) {
    if (e == 0 && lane < 8) a.stats[lane] = lane == 6 ? ULTRAEP_EDATA : (lane == 7 ? L : 0);
    return;
  }
  walk_bits(outcome_or(bv), kRounds - 1, fin);
  int nb = 0;  // transfers of the last feasible probe, read into s_et / s_d
  if (fin.lo < fin.hi) {
    // a bisection longer than the rounds: the remaining probes run here, one
    // after another, the same ones in every workgroup
    __shared__ uint2 s_ent[kMaxE];
    __shared__ uint2 s_rec[kMaxRec + kWave];
    __shared__ uint2 s_out[kMaxRec];
    for (int i = lane; i < E; i += kWave) s_ent[i] = a.ws.ent[i];
    const v4i rk = a.ws.rank[lane];
    const bool packed = hi0 < (int64_t(1) << 25);
    bool local = false;
    __syncthreads();
    while (fin.lo < fin.hi) {
      const int64_t mid = (fin.lo + fin.hi) / 2;
      ++fin.probes;
      const int n = run_probe<1>(a, packed, static_cast<int>(mid), lane, rk, s_ent, s_rec, s_out);
      __syncthreads();
      if (n >= 0) {
        fin.hi = mid;
        local = true;
        nb = n;
        for (int i = lane; i < n; i += kWave) {
          s_et[i] = s_out[i].x;
          s_d[i] = static_cast<int32_t>(s_out[i].y);
        }
      } else {
        fin.lo = mid + 1;
      }
      __syncthreads();
    }
    if (local) fin.best = -2;  // records already in s_et / s_d
  }
  const int64_t hi = fin.hi;
  const int n_probe = fin.probes;
  const int best = fin.best;
  if (best >= 0) {
    // the count and the node's records are requested together: every slot's
    // record is read (at most RS), the ones past the count are dropped
    const uint32_t *rec = a.ws.rec + static_cast<int64_t>(best) * 2 * RS;
    uint32_t rv_e[kMaxRec / kWave], rv_d[kMaxRec / kWave];
#pragma unroll
    for (int u = 0; u < kMaxRec / kWave; ++u) {
      if (u * kWave < RS) {
        const int i = min(u * kWave + lane, RS - 1);
        rv_e[u] = rec[2 * i];
        rv_d[u] = rec[2 * i + 1];
      }
    }
    nb = a.ws.res[best];
#pragma unroll
    for (int u = 0; u < kMaxRec / kWave; ++u) {
      const int i = u * kWave + lane;
      if (u * kWave < RS && i < nb) {
        s_et[i] = rv_e[u];
        s_d[i] = static_cast<int32_t>(rv_d[u]);
      }
    }
  }
  __syncthreads();
  const int h = e / nm;

  // CSR row pointer: every expert has 1 + (its replicas) entries
  int before = 0, shed = 0;
  for (int i = lane; i < nb; i += kWave) {
    const int ei = static_cast<int>(s_et[i] & 0xFFFFu);
    before += ei < e;
    if (ei == e) shed += s_d[i];
  }
  before = wave_sum(before);
  shed = wave_sum(shed);
  const int hp_e = e + before;
  // this expert's replicas: position among them = replicas on lower ranks
  // (an expert's transfers go to distinct ranks, so a mask of them gives
  // it); slot on the host = earlier accepted transfers to the same rank,
  // from a match of equal ranks within 64 records and per-rank counts of
  // the records before them
  uint64_t tmask = 0;
  for (int i0 = 0; i0 < nb; i0 += kWave) {
    const int i = i0 + lane;
    const uint32_t x = i < nb ? s_et[i] : 0xFFFFFFFFu;  // expert field 0xFFFF: no expert
    uint64_t mb = ballot(static_cast<int>(x & 0xFFFFu) == e);
    while (mb) {
      const int l = __ffsll(static_cast<unsigned long long>(mb)) - 1;
      mb &= mb - 1;
      tmask |= uint64_t(1) << readlane(static_cast<int>(x >> 16), l);
    }
  }
  const int fan = __popcll(tmask);
  if (fan > 0) {
    const int tb = bits_for(R);
    for (int i = lane; i < kMaxR; i += kWave) s_fan[i] = 0;  // records per rank so far
    __syncthreads();
    for (int i0 = 0; i0 < nb; i0 += kWave) {
      const int i = i0 + lane;
      const bool valid = i < nb;
      const uint32_t x = valid ? s_et[i] : 0;
      const int t = static_cast<int>(x >> 16);
      const uint64_t same = match_any(static_cast<uint32_t>(t), tb, ballot(valid));
      const int before_t = valid ? s_fan[t] : 0;
      if (valid && static_cast<int>(x & 0xFFFFu) == e) {
        const int pos = __popcll(tmask & ((uint64_t(1) << t) - 1));
        const int slot = before_t + popc_below(same);
        s_ht[1 + pos] = t;
        s_hu[1 + pos] = s_d[i];
        a.hr[hp_e + 1 + pos] = t;
        a.hs[hp_e + 1 + pos] = nm + slot;
      }
      __syncthreads();
      if (valid && popc_below(same) == 0) s_fan[t] = before_t + __popcll(same);
      __syncthreads();
    }
  }
  const int nh = 1 + fan;
  if (lane == 0) {
    s_ht[0] = h;
    s_hu[0] = lam_e - shed;
    a.hp[e] = hp_e;
    a.hr[hp_e] = h;
    a.hs[hp_e] = e - h * nm;
    if (e == E - 1) a.hp[E] = E + nb;
  }
  for (int j = E + nb + e; j < ncol; j += E) {  // CSR padding
    if (lane == 0) {
      a.hr[j] = -1;
      a.hs[j] = -1;
    }
  }
  // row e of U
  __syncthreads();
  int u_r = 0;  // quota of this expert on rank `lane`
  for (int i = 0; i < nh; ++i)
    if (s_ht[i] == lane) u_r = s_hu[i];
  if (lane < R) a.U[static_cast<int64_t>(e) * R + lane] = u_r;
  (void)ncol;
  // row t = e of X (one workgroup per rank): slots in acceptance order
  if (e < R && NS > 0) {
    int cnt = 0;
    for (int i0 = 0; i0 < nb; i0 += kWave) {
      const int i = i0 + lane;
      const bool to_me = i < nb && static_cast<int>(s_et[i] >> 16) == e;
      const uint64_t mb = ballot(to_me);
      if (to_me) a.X[e * NS + cnt + popc_below(mb)] = static_cast<int>(s_et[i] & 0xFFFFu);
      cnt += __popcll(mb);
    }
    for (int s = cnt + lane; s < NS; s += kWave) a.X[e * NS + s] = -1;
  }
  if (e == 0) {  // stats
    for (int i = lane; i < E; i += kWave) s_fan[i] = 0;
    __syncthreads();
    for (int i = lane; i < nb; i += kWave) atomicAdd(&s_fan[s_et[i] & 0xFFFFu], 1);
    __syncthreads();
    int mf = 0;
    for (int i = lane; i < E; i += kWave) mf = max(mf, s_fan[i]);
    mf = wave_max(mf);
    if (lane == 0) {
      a.stats[0] = hi;
      a.stats[1] = lo0;
      a.stats[2] = hi0;
      a.stats[3] = n_probe;
      a.stats[4] = nb;
      a.stats[5] = 1 + mf;
      a.stats[6] = 0;
      a.stats[7] = L;
    }
  }
  if (kReroute) reroute_expert(a, e, hp_e, E + nb, lam_r, u_r, L, s_t);
}

__global__ void __launch_bounds__(kWave) k_plan_reroute(PlanArgs a) {
  __shared__ int32_t s_t[kRrLds];
  const int e = blockIdx.x, lane = threadIdx.x;
  const int R = a.R, E = a.E;
  const int64_t status = a.stats[6], L = a.stats[7];
  const int j0 = a.hp[e], total = a.hp[E];
  const int lam_r = lane < R ? a.load[static_cast<int64_t>(lane) * E + e] : 0;
  const int u_r = lane < R ? a.U[static_cast<int64_t>(e) * R + lane] : 0;
  if (status != 0) return;
  reroute_expert(a, e, j0, total, lam_r, u_r, L, s_t);
}

// SolveReroute and the local weight packing in one launch, as the forward
// pipeline overlaps them (Eq. 1): workgroup e < E runs expert e's split on
// its first wave, the others pack tiles.  Packing needs only the replica
// placement, which SolveReplication has already written.  The reroute
// workgroups come first so they are placed before the packing fills the
// chip.
__global__ void __launch_bounds__(kPkThreads) k_reroute_pack(PlanArgs a, PkArgs p) {
  __shared__ int32_t s_t[kRrLds];
  const int b = blockIdx.x;
  if (b < a.E) {
    if (threadIdx.x >= kWave) return;
    const int e = b, lane = threadIdx.x;
    const int R = a.R, E = a.E;
    const int64_t status = a.stats[6], L = a.stats[7];
    const int j0 = a.hp[e], total = a.hp[E];
    const int lam_r = lane < R ? a.load[static_cast<int64_t>(lane) * E + e] : 0;
    const int u_r = lane < R ? a.U[static_cast<int64_t>(e) * R + lane] : 0;
    if (status != 0) return;
    reroute_expert(a, e, j0, total, lam_r, u_r, L, s_t);
    return;
  }
  pack_block(p, b - a.E, static_cast<int64_t>(gridDim.x) - a.E, b == a.E);
}

static PlanArgs plan_args(const int32_t *load, const ultraep_group &g,
                          const ultraep_plan_buf &out, void *ws) {
  PlanArgs a{};
  a.load = load;
  a.R = g.R;
  a.E = g.E;
  a.NS = g.n_slot;
  a.nm = g.E / g.R;
  a.ncol = g.E + g.R * g.n_slot;
  a.u_min = static_cast<int32_t>(g.u_min > INT32_MAX ? INT32_MAX : g.u_min);
  a.beta_num = g.beta_num;
  a.beta_den = g.beta_den;
  a.X = out.slot_expert;
  a.U = out.quota;
  a.hp = out.host_ptr;
  a.hr = out.host_rank;
  a.hs = out.host_pslot;
  a.q = out.reroute;
  a.stats = out.stats;
  if (ws) a.ws = carve(ws, g.R, g.E, g.n_slot);
  return a;
}

hipError_t launch_plan_replicate(const int32_t *load, const ultraep_group &g,
                                 const ultraep_plan_buf &out, void *ws, hipStream_t stream) {
  const PlanArgs a = plan_args(load, g, out, ws);
  hipLaunchKernelGGL(k_plan_prep, dim3(1), dim3(kPrepThreads), 0, stream, a);
  hipError_t err = hipGetLastError();
  for (int round = 0; round < kRounds && err == hipSuccess; ++round) {
    hipLaunchKernelGGL(k_plan_round, dim3(kNodes), dim3(kWave), 0, stream, a, round);
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_plan_emit<false>, dim3(g.E), dim3(kWave), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_plan(const int32_t *load, const ultraep_group &g,
                       const ultraep_plan_buf &out, void *ws, hipStream_t stream) {
  const PlanArgs a = plan_args(load, g, out, ws);
  hipLaunchKernelGGL(k_plan_prep, dim3(1), dim3(kPrepThreads), 0, stream, a);
  hipError_t err = hipGetLastError();
  for (int round = 0; round < kRounds && err == hipSuccess; ++round) {
    hipLaunchKernelGGL(k_plan_round, dim3(kNodes), dim3(kWave), 0, stream, a, round);
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_plan_emit<true>, dim3(g.E), dim3(kWave), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_reroute_pack(const int32_t *load, const ultraep_group &g,
                               const ultraep_plan_buf &out, const uint16_t *w_main, int64_t W,
                               int32_t rank, uint16_t *staging, int64_t cap, int64_t *dest_off,
                               int32_t *status, hipStream_t stream) {
  const PlanArgs a = plan_args(load, g, out, nullptr);
  const PkArgs p = pack_args(w_main, W, rank, g, out, staging, cap, dest_off, status);
  hipLaunchKernelGGL(k_reroute_pack, dim3(g.E + kPkGrid), dim3(kPkThreads), 0, stream, a, p);
  return hipGetLastError();
}

hipError_t launch_plan_reroute(const int32_t *load, const ultraep_group &g,
                               const ultraep_plan_buf &out, hipStream_t stream) {
  const PlanArgs a = plan_args(load, g, out, nullptr);
  hipLaunchKernelGGL(k_plan_reroute, dim3(g.E), dim3(kWave), 0, stream, a);
  return hipGetLastError();
}

}  // namespace uep
