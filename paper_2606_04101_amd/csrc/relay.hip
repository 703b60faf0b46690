// Relay trees for hot-expert fan-out (Sec. 6.2, load-aware relay
// scheduling): which rank sends each redundant slot its expert's blob.
//
// The paper tracks each rank's sending volume under the replication plan
// and then, one hot expert at a time, picks first-stage relays among the
// expert's replica ranks with the smallest volume and attaches every other
// replica to the relay whose volume stays smallest after taking it; the
// source's and relays' volumes are updated before the next expert.  The
// points the text leaves open are fixed as follows, for this library and
// for its tests alike:
//   - eligible: replica count f = |H(e)| - 1 exceeds the threshold (4 in the
//     paper);
//   - relay count: the integer nearest sqrt(f) (no ties for integer f);
//   - volume unit: one expert blob; a rank starts with one blob per replica
//     of each of its main experts;
//   - hot experts by f descending, then id ascending;
//   - relays: the replica ranks of smallest volume, ties to the smaller rank;
//   - leaves: the other replicas by ascending rank, each to the relay of
//     smallest volume (ties to the smaller rank), counted at once;
//   - after the expert, the source's volume drops by f minus the relays.
//
// One workgroup; what bounds it is the chain of dependent latencies, not
// work.  Every input is requested at once and staged in LDS, so memory is
// waited for once.  The host lists are validated a column per thread: a home
// column must be its expert's first one, a replica column must lie behind it in
// the list of the expert that its slot holds, at ascending ranks (walking each
// list in one thread waited for memory once per replica).  The hot experts are
// compacted and ranked by counting.  They depend on each other only through
// the volumes, so one wave walks them in order, a host per lane (f + 1 <= R <=
// 64).  The n relays are n wave minima over (volume, rank).  The leaves need no
// order of their own: dealing them one by one to the smallest (volume, rank)
// hands out the merged keys (V_i + q, rank) of the relays in ascending order, so
// with the relays sorted and C_i the number of keys below volume V_i, leaf m
// falls among relays 0..i for the last i with C_i <= m, at place (m - C_i)
// mod (i + 1) by rank.
// Each expert's columns are read while the expert before it is dealt.
// Graph of 20 calls: 3.3 us without a hot expert at R = 64, E = 128 (3.9 with a
// list per thread and leaves one by one), 5.4 with two hot experts at R = 32,
// E = 256 (7.5), 12.9 with five of fan-outs up to 63 (54.3), 19.7 with twelve
// at E = 256 (47.8), 32.7 with thirty at R = 16, E = 1024 (48.9).
#include "common.hpp"
#include "kernels.hpp"

namespace uep {

constexpr int kRlThreads = 1024;
constexpr int kRlMaxE = 1024;
constexpr int kRlMaxSlots = 256;                   // R * n_slot
constexpr int kRlMaxCol = kRlMaxE + kRlMaxSlots;   // host-list columns
constexpr int kRlColIters = 2;                     // columns per thread
static_assert(kRlThreads >= kRlMaxE && kRlColIters * kRlThreads >= kRlMaxCol,
              "an expert and its columns fit the threads");

struct RlArgs {
  int32_t R, E, NS, nm, ncol, threshold;
  const int32_t *X, *hp, *hr, *hs;
  const int64_t *plan_stats;
  int32_t *slot_src, *send_vol;
  int64_t *stats;
  int32_t *status;
};

// The minimum of the 64 lanes, uniform: rows of 16 by DPP mirrors, then across
// the rows by DPP broadcasts into lane 63.  Every lane must be active.
__device__ __forceinline__ int wave_min(int v) {
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xF, 0xF, false));  // row_mirror
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return readlane(v, 63);
}

__global__ void __launch_bounds__(kRlThreads) k_relay(RlArgs a) {
  __shared__ int32_t s_hp[kRlMaxE + 1];
  __shared__ int32_t s_hr[kRlMaxCol];
  __shared__ int32_t s_hs[kRlMaxCol];
  __shared__ int32_t s_x[kRlMaxSlots];
  __shared__ int32_t s_src[kRlMaxSlots];
  __shared__ int32_t s_vol[kWave];
  __shared__ int32_t s_hot[kRlMaxSlots];   // hot experts, unsorted
  __shared__ int32_t s_ord[kRlMaxSlots];   // sorted
  __shared__ int32_t s_wcnt[kRlThreads / kWave];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int R = a.R, E = a.E, NS = a.NS, nm = a.nm, RS = R * NS, ncol = a.ncol;
  // inputs, indices clamped into range
  int vr[kRlColIters], vs[kRlColIters];
#pragma unroll
  for (int u = 0; u < kRlColIters; ++u) {
    if (u * kRlThreads < ncol) {
      const int j = min(u * kRlThreads + tid, ncol - 1);
      vr[u] = a.hr[j];
      vs[u] = a.hs[j];
    }
  }
  const int vp = a.hp[min(tid, E)], total = a.hp[E];
  const int vx = tid < RS ? a.X[tid] : -1;
  bool bad = a.plan_stats[6] != 0;
  if (tid < kWave) s_vol[tid] = 0;
#pragma unroll
  for (int u = 0; u < kRlColIters; ++u) {
    const int j = u * kRlThreads + tid;
    if (j < ncol) {
      s_hr[j] = vr[u];
      s_hs[j] = vs[u];
    }
  }
  if (tid < E) s_hp[tid] = vp;
  if (tid == 0) s_hp[E] = total;
  if (tid < RS) s_x[tid] = vx;
  __syncthreads();
  // The pointers start at 0, ascend and end within the columns, a list has at
  // most R entries; then every column below `total` is in one expert's list
  // and the checks of the columns are those of the lists.
  bad |= total > ncol;
  int f = -1;
  if (tid < E) {
    f = static_cast<int>(static_cast<uint32_t>(s_hp[tid + 1]) - static_cast<uint32_t>(vp) - 1u);
    bad |= f < 0 || f >= R || (tid == 0 && vp != 0);
  }
#pragma unroll
  for (int u = 0; u < kRlColIters; ++u) {
    const int j = u * kRlThreads + tid;
    if (j < min(total, ncol)) {
      const int t = vr[u], s = vs[u];
      bool ok = t >= 0 && t < R && s >= 0 && s < nm + NS;
      if (ok && s < nm) {
        ok = s_hp[t * nm + s] == j;  // the home column: the first of its expert
      } else if (ok) {
        const int e = s_x[t * NS + s - nm];
        ok = e >= 0 && e < E && e / nm != t;
        if (ok) {
          // (the pointers are not known to be sound here: j0 >= 0 keeps j - 1
          // inside the columns)
          const int j0 = s_hp[e];
          ok = j0 >= 0 && j > j0 && j < s_hp[e + 1] && (j == j0 + 1 || t > s_hr[j - 1]);
        }
      }
      bad |= !ok;
    }
  }
  // senders start at the home ranks; volumes count one blob per replica
  if (tid < RS) {
    const bool ok = vx >= -1 && vx < E;
    bad |= !ok;
    const int h = ok && vx >= 0 ? vx / nm : -1;
    s_src[tid] = h;
    if (h >= 0) atomicAdd(&s_vol[h], 1);
  }
  const bool hot = f > a.threshold;
  const uint64_t hb = ballot(hot);
  if (lane == 0) s_wcnt[wave] = __popcll(hb);
  if (__syncthreads_or(bad)) {
    if (tid == 0) report(a.status, ULTRAEP_EDATA);
    return;
  }
  // compact the hot experts
  int pos = popc_below(hb), nhot = 0;
  for (int w = 0; w < kRlThreads / kWave; ++w) {
    const int n = s_wcnt[w];
    pos += w < wave ? n : 0;
    nhot += n;
  }
  int vmax0 = 0, n_relays = 0;
  if (wave == 0) vmax0 = wave_max(lane < R ? s_vol[lane] : 0);
  if (nhot > 0) {  // uniform
    if (hot) s_hot[pos] = tid;
    __syncthreads();
    // order: replica count descending, then id ascending (rank by counting)
    if (tid < nhot) {
      const int e = s_hot[tid], fe = s_hp[e + 1] - s_hp[e];
      int r = 0;
      for (int i = 0; i < nhot; ++i) {
        const int o = s_hot[i], fo = s_hp[o + 1] - s_hp[o];
        r += fo > fe || (fo == fe && o < e);
      }
      s_ord[r] = e;
    }
    __syncthreads();
    if (wave == 0) {
      const int recip = 65536 / (lane + 1) + 1;  // x / (lane + 1) for x < 64, lane < 8
      // an expert's home, its replica count and the replicas' ranks and slots,
      // read while the expert before it is dealt
      int n_home, n_fe, n_t, n_s;
      const auto fetch = [&](int hi) {
        const int e = s_ord[hi], j0 = s_hp[e];
        n_fe = s_hp[e + 1] - j0 - 1;
        n_home = s_hr[j0];
        const int j = j0 + 1 + min(lane, n_fe - 1);
        n_t = s_hr[j];
        n_s = s_hs[j] - nm;
      };
      fetch(0);
      for (int hi = 0; hi < nhot; ++hi) {
        const int fe = __builtin_amdgcn_readfirstlane(n_fe);
        const int home = n_home, t = n_t, s = n_s;
        // the integer nearest sqrt(fe): the i >= 0 with i * i + i < fe
        const int n = __popcll(ballot(lane * lane + lane < fe));
        const bool act = lane < fe;
        // relays: the n smallest (volume, rank); lane i keeps C_i and the
        // set of the ranks of relays 0..i
        int key = act ? (s_vol[t] << 6) | t : INT32_MAX;
        fetch(min(hi + 1, nhot - 1));
        n_relays += n;
        if (n == fe) continue;  // one replica, the relay: no volume changes
        uint64_t set = 0;
        int C = 0, vprev = 0, l_c = 0, l_lo = 0, l_hi = 0;
        bool leaf = act;
        for (int i = 0; i < n; ++i) {
          const int m = wave_min(key);
          if (key == m) {
            key = INT32_MAX;
            leaf = false;
          }
          C += ((m >> 6) - vprev) * i;
          vprev = m >> 6;
          set |= uint64_t(1) << (m & 63);
          if (lane == i) {
            l_c = C;
            l_lo = static_cast<int>(set);
            l_hi = static_cast<int>(set >> 32);
          }
        }
        // leaves, ascending rank
        const int m = popc_below(ballot(leaf));
        int off = 0, cnt = 1, rc = 0, lo = 0, hi32 = 0;
        for (int i = 0; i < n; ++i) {
          const int Ci = readlane(l_c, i);
          if (m >= Ci) {
            off = m - Ci;
            cnt = i + 1;
            rc = readlane(recip, i);
            lo = readlane(l_lo, i);
            hi32 = readlane(l_hi, i);
          }
        }
        if (leaf) {
          const int place = off - ((off * rc) >> 16) * cnt;
          uint64_t rest = (static_cast<uint64_t>(static_cast<uint32_t>(hi32)) << 32) |
                          static_cast<uint32_t>(lo);
          for (int u = 0; u < place; ++u) rest &= rest - 1;
          const int win = __builtin_ctzll(rest);
          s_src[t * NS + s] = win;
          atomicAdd(&s_vol[win], 1);
        }
        if (lane == 0) s_vol[home] -= fe - n;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the volumes, to the next expert
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < RS; i += kRlThreads) a.slot_src[i] = s_src[i];
  if (tid < R) a.send_vol[tid] = s_vol[tid];
  if (wave == 0) {
    const int vmax1 = wave_max(lane < R ? s_vol[lane] : 0);
    if (lane == 0) {
      a.stats[0] = nhot;
      a.stats[1] = n_relays;
      a.stats[2] = vmax0;
      a.stats[3] = vmax1;
    }
  }
}

hipError_t launch_relay(const ultraep_group &g, const ultraep_plan_buf &plan, int32_t threshold,
                        int32_t *slot_src, int32_t *send_vol, int64_t *stats, int32_t *status,
                        hipStream_t stream) {
  RlArgs a;
  a.R = g.R;
  a.E = g.E;
  a.NS = g.n_slot;
  a.nm = g.E / g.R;
  a.ncol = g.E + g.R * g.n_slot;
  a.threshold = threshold;
  a.X = plan.slot_expert;
  a.hp = plan.host_ptr;
  a.hr = plan.host_rank;
  a.hs = plan.host_pslot;
  a.plan_stats = plan.stats;
  a.slot_src = slot_src;
  a.send_vol = send_vol;
  a.stats = stats;
  a.status = status;
  hipLaunchKernelGGL(k_relay, dim3(1), dim3(kRlThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace uep
