// Step 3 — token-to-replica assignment and dispatch permutation of one
// source rank (Sec. 5.2 Token Assignment), then the bf16 row scatter.
//
// Layout (integer only; two launches, or k_dl_one for few chunks):
//   k_dl_hist  : workgroup c < n_chunks counts the expert ids of slots
//                [c*2048, (c+1)*2048); the last workgroup turns row `rank` of
//                the reroute split into block sizes (t, p), their exclusive
//                prefix block_off, and per CSR entry the running share over
//                all columns and the first row minus the entry's start in it.
//   k_dl_rows  : workgroup c sums the histograms of chunks < c (its base
//                ordinal per expert; up to 16 threads share the chunks, and the
//                loads past the first four and past the first eight per
//                thread are skipped when there are no such chunks: code
//                that runs once costs its fetch), then each wave ranks its 128 slots
//                stably with ballot matches (wave-private running counts in
//                LDS, scanned across waves), bisects for the first
//                instance whose running share exceeds the ordinal and writes
//                the row.
//   Both kernels (graph of 20 calls, one rank of R = 64): 9.2 us for 32768 slots
//   of E = 256 and 10.2 us for 131072; 10.1 and 11.2 us with the shares of an
//   expert summed by one thread and its instances searched one by one, and 13.0
//   for the latter with the sums over chunks in one thread per expert too.
// Scatter (bandwidth bound): persistent waves walk the tokens; a wave holds
//   one token's row in registers (16-byte non-temporal loads) while the next
//   token's row is being loaded, and stores each 1 KiB chunk to all k
//   destination rows before the next chunk, with sc1 buffer stores.  The
//   rows are a permutation of the send buffer, and writing such a
//   permutation of 14 KiB rows measures about 5.2 TB/s on its own, against
//   6.5 TB/s for a sequential stream; rows past the routed count are
//   zero-filled.
#include "common.hpp"
#include "kernels.hpp"

namespace uep {

constexpr int kDlThreads = 1024;
constexpr int kDlWaves = kDlThreads / kWave;
constexpr int kSlotsPerWave = kDispatchChunk / kDlWaves;  // 128

static_assert(kSlotsPerWave % kWave == 0, "chunk must split into wave steps");
// CSR columns (E + R * n_slot <= 1024 + 256) and start pointers (E + 1) per
// thread when a 1024-thread workgroup stages them
constexpr int kLutIters = 2;
constexpr int kSumFirst = 4;   // chunk histograms per thread in the first loads,
constexpr int kSumSecond = 4;  // in the second ones
constexpr int kSumBatch = 12;  // and in a batch (the second ones and more)
constexpr int kSumParts = 16;  // threads that share an expert's chunks at most
static_assert(kLutIters * kDlThreads >= 1024 + 256 && kLutIters * kDlThreads >= 1024 + 1,
              "the lookup tables fit the staging loops");
constexpr int kOneChunks = 10;  // chunks up to which one launch makes the layout
constexpr int kOneBatch = 8;    // ids of earlier chunks in flight per thread
constexpr int kOneCopies = 8;   // counts of them at most, dealt over the lanes,
constexpr int kOneFew = 2;      // for two chunks
constexpr int kSteps = kSlotsPerWave / kWave;  // 64-slot steps per wave

size_t dispatch_ws_bytes(int64_t V, int32_t E, int32_t ncol) {
  const int64_t n_chunks = (V + kDispatchChunk - 1) / kDispatchChunk;
  const int64_t ints = n_chunks * E + 2 * static_cast<int64_t>(ncol) + E;
  return static_cast<size_t>((ints * 4 + 255) / 256 * 256);
}

DispatchWs dispatch_ws(void *ws, int64_t V, int32_t E, int32_t ncol) {
  DispatchWs w;
  w.n_chunks = (V + kDispatchChunk - 1) / kDispatchChunk;
  int32_t *p = static_cast<int32_t *>(ws);
  w.hist = p;
  p += w.n_chunks * E;
  w.ent_cum = p;
  p += ncol;
  w.ent_base = p;
  p += ncol;
  w.exp_tot = p;
  return w;
}

struct DlArgs {
  const int32_t *topk;
  int64_t V;
  int32_t rank, R, E, NS, nm, S, ncol, nbits;
  int32_t parts, div_E;  // threads per expert in the sums over chunks, 2^20 / E rounded up
  int32_t stage_lut;  // copy host_ptr / entry tables into LDS
  int32_t copies;     // k_dl_one: counts of the earlier ids, a power of two
  const int32_t *hp, *hr, *hs, *q;  // q = reroute row of `rank`
  int32_t *row_of_slot;
  int64_t *block_off;
  DispatchWs ws;
  int32_t *status;
};

// Sum of the first row's 16 lanes, in every lane.
__device__ __forceinline__ int row_first_sum(int v) { return readlane(row_sum(v), 0); }
static_assert(kDlWaves == 16, "the waves' totals fill one row of lanes");

// This rank's layout tables in LDS.
struct DlTables {
  int32_t *cnt;  // [ncol = R * S] rows per (rank, slot) block, then its first row
  int32_t *tmp;  // [2 * kDlWaves]
  int32_t *hp;   // [E + 1]
  int32_t *hr;   // [ncol] host rank, then the entry's first row minus P
  int32_t *hs;   // [ncol] its slot
  int32_t *q;    // [ncol] this rank's share, then P + share
};

__host__ __device__ __forceinline__ int lut_ints(int E, int ncol) {
  return 2 * kDlWaves + E + 1 + 4 * ncol;
}

// Clears n 32-bit words of LDS (n a multiple of 4, p 16-byte aligned).
__device__ __forceinline__ void clear_lds(int32_t *p, int n) {
  v4i *v = reinterpret_cast<v4i *>(p);
  for (int i = threadIdx.x; i < n / 4; i += kDlThreads) v[i] = v4i{0, 0, 0, 0};
}

__device__ __forceinline__ DlTables carve_tables(int32_t *p, int E, int ncol) {
  DlTables t;
  t.cnt = p;
  t.tmp = t.cnt + ncol;
  t.hp = t.tmp + 2 * kDlWaves;
  t.hr = t.hp + E + 1;
  t.hs = t.hr + ncol;
  t.q = t.hs + ncol;
  return t;
}

// The inputs of the tables: requested at once (indices clamped into range, no
// branch between the loads), then staged in LDS.
struct DlInputs {
  int hp[kLutIters], hr[kLutIters], hs[kLutIters], q[kLutIters];
  __device__ __forceinline__ void load(const DlArgs &a) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < kLutIters; ++u) {
      if (u * kDlThreads <= a.E) hp[u] = a.hp[min(u * kDlThreads + tid, a.E)];
      if (u * kDlThreads < a.ncol) {
        const int j = min(u * kDlThreads + tid, a.ncol - 1);
        hr[u] = a.hr[j];
        hs[u] = a.hs[j];
        q[u] = a.q[j];
      }
    }
  }
  __device__ __forceinline__ void stage(const DlArgs &a, const DlTables &t) const {
#pragma unroll
    for (int u = 0; u < kLutIters; ++u) {
      const int i = u * kDlThreads + threadIdx.x;
      if (i <= a.E) t.hp[i] = hp[u];
      if (i < a.ncol) {
        t.hr[i] = hr[u];
        t.hs[i] = hs[u];
        t.q[i] = q[u];
      }
    }
  }
};

// Block sizes and offsets, and per CSR column the running share over ALL
// columns: with P the shares of the columns before it, a slot of expert e with
// ordinal o belongs to the first column of e whose P + share exceeds
// P(first column of e) + o, and its row is that sum plus the block's first row
// minus the column's P.  One block scan gives every P (a loop over an
// expert's columns in one thread took a chain of LDS reads per replica).  The
// inputs are staged and cnt is cleared, before a barrier; the tables are
// complete at the return.  False: not a plan of this group.
__device__ __forceinline__ bool build_tables(const DlArgs &a, const DlTables &t, bool writes) {
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int E = a.E, ncol = a.ncol, nblk = a.R * a.S;
  // the CSR must start at 0, never decrease and end within the columns,
  // so every entry index below is inside the tables
  const int total = t.hp[E];
  bool bad = t.hp[0] != 0 || total < E || total > ncol;
  for (int e = tid; e < E; e += kDlThreads) bad |= t.hp[e] > t.hp[e + 1];
  if (__syncthreads_or(bad)) return false;
  static_assert(2 * kDlThreads >= 1024 + 256, "two blocks and two columns per thread");
  const int j0 = 2 * tid, j1 = 2 * tid + 1;
  int blk[2], q[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int j = 2 * tid + u;
    blk[u] = -1;
    q[u] = 0;
    if (j < total) {
      const int r = t.hr[j], p = t.hs[j];
      q[u] = t.q[j];
      if (r >= 0 && r < a.R && p >= 0 && p < a.S) {
        blk[u] = r * a.S + p;
        t.cnt[blk[u]] = q[u];
      } else if (writes) {
        report(a.status, ULTRAEP_EDATA);
      }
    }
  }
  __syncthreads();
  // exclusive scans, two elements per thread
  const int v0 = j0 < nblk ? t.cnt[j0] : 0, v1 = j1 < nblk ? t.cnt[j1] : 0;
  const int incl = wave_scan_incl(v0 + v1), inclq = wave_scan_incl(q[0] + q[1]);
  if (lane == kWave - 1) {
    t.tmp[wave] = incl;
    t.tmp[kDlWaves + wave] = inclq;
  }
  __syncthreads();
  const int before = lane & (kDlWaves - 1);  // totals of the waves before
  const int ex0 = row_first_sum(lane < wave ? t.tmp[before] : 0) + incl - v0 - v1;
  const int P0 = row_first_sum(lane < wave ? t.tmp[kDlWaves + before] : 0) + inclq - q[0] - q[1];
  if (j0 < nblk) t.cnt[j0] = ex0;
  if (j1 < nblk) t.cnt[j1] = ex0 + v0;
  if (writes) {
    if (j0 < nblk) a.block_off[j0] = ex0;
    if (j1 < nblk) a.block_off[j1] = ex0 + v0;
    if (j1 == nblk || j0 == nblk) a.block_off[nblk] = ex0 + (j0 == nblk ? 0 : v0);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int j = 2 * tid + u;
    if (j < total) {
      const int P = u ? P0 + q[0] : P0;
      t.hr[j] = (blk[u] >= 0 ? t.cnt[blk[u]] : 0) - P;
      t.q[j] = P + q[u];
    }
  }
  __syncthreads();
  return true;
}

// P of an expert's first column j0 (clamped: a CSR that is not a plan of this
// group cannot send the read outside the tables).
__device__ __forceinline__ int share_before(const int32_t *cum, int j0, int ncol) {
  j0 = min(max(j0, 0), ncol);
  return j0 > 0 ? cum[j0 - 1] : 0;
}

// Stable ordinals of a wave's slots, their instance and rows.  wh: per expert,
// P of its first column plus the ordinal that the wave starts at.
__device__ __forceinline__ void write_rows(const DlArgs &a, const int32_t (&ev)[kSteps], int64_t s0,
                                           int32_t *wh, const int32_t *hp, const int32_t *cum,
                                           const int32_t *base) {
  const int lane = lane_id();
  for (int s = 0; s < kSteps; ++s) {
    const int64_t i = s0 + s * kWave + lane;
    const int32_t e = ev[s];
    const bool valid = e >= 0 && e < a.E;
    const uint64_t act = ballot(valid);
    if (act == 0) {
      if (i < a.V) a.row_of_slot[i] = -1;
      continue;
    }
    const uint64_t m = match_any(static_cast<uint32_t>(valid ? e : 0), a.nbits, act);
    int row = -1;
    if (valid) {
      const int below = popc_below(m);
      const int at = wh[e] + below;
      if (below == 0) wh[e] += __popcll(m);
      // entry range of e, clamped to the tables (a CSR that is not a plan
      // of this group cannot send the search outside them); bisected, since
      // a hot expert has up to R entries
      const int j1 = min(max(hp[e + 1], 0), a.ncol);
      int j = min(max(hp[e], 0), j1), n = j1 - j;
      while (n > 0) {
        const int half = n >> 1;
        const bool up = cum[j + half] <= at;
        j = up ? j + half + 1 : j;
        n = up ? n - half - 1 : half;
      }
      if (j < j1) row = base[j] + at;
      // a plan row that does not match these ids can point past the buffer
      if (row < 0 || row >= a.V) {
        row = -1;
        report(a.status, ULTRAEP_EDATA);
      }
    }
    if (i < a.V) a.row_of_slot[i] = row;
  }
}

__global__ void __launch_bounds__(kDlThreads) k_dl_hist(DlArgs a) {
  extern __shared__ int32_t lds[];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int E = a.E;
  if (blockIdx.x < a.ws.n_chunks) {
    int32_t *hist = lds;  // [kDlWaves][E]
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kDispatchChunk;
    int32_t *wh = hist + wave * E;
    bool bad = false;
    int32_t ev[kSteps];  // on their way while the bins are cleared
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int64_t i = c0 + wave * kSlotsPerWave + s * kWave + lane;
      ev[s] = i < a.V ? a.topk[i] : -1;
    }
    for (int i = tid; i < kDlWaves * E; i += kDlThreads) hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int32_t e = ev[s];
      if (e >= 0 && e < E) atomicAdd(wh + e, 1);
      bad |= e < -1 || e >= E;
    }
    if (bad) report(a.status, ULTRAEP_EDATA);
    __syncthreads();
    int32_t *dst = a.ws.hist + blockIdx.x * static_cast<int64_t>(E);
    for (int e = tid; e < E; e += kDlThreads) {
      int s = 0;
#pragma unroll
      for (int w = 0; w < kDlWaves; ++w) s += hist[w * E + e];
      dst[e] = s;
    }
    return;
  }
  // ---- layout workgroup: block sizes, offsets, entry lookup tables ----
  DlInputs in;
  in.load(a);
  const DlTables t = carve_tables(lds, E, a.ncol);
  for (int b = tid; b < a.R * a.S; b += kDlThreads) t.cnt[b] = 0;
  in.stage(a, t);
  __syncthreads();
  if (!build_tables(a, t, true)) {  // not a plan of this group
    if (tid == 0) report(a.status, ULTRAEP_EDATA);
    return;
  }
  for (int j = tid; j < t.hp[E]; j += kDlThreads) {
    a.ws.ent_base[j] = t.hr[j];
    a.ws.ent_cum[j] = t.q[j];
  }
  for (int e = tid; e < E; e += kDlThreads)
    a.ws.exp_tot[e] = share_before(t.q, t.hp[e + 1], a.ncol) - share_before(t.q, t.hp[e], a.ncol);
}

__global__ void __launch_bounds__(kDlThreads) k_dl_rows(DlArgs a) {
  extern __shared__ int32_t lds[];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int E = a.E, ncol = a.ncol;
  const int c = blockIdx.x;
  int32_t *whist = lds;                  // [kDlWaves][E]
  int32_t *psum = lds + kDlWaves * E;    // [kDlThreads] partial sums over chunks
  // Every input is requested at once (indices clamped into range, no branch
  // between the loads), so the workgroup waits for memory once: its slots'
  // expert ids, the histograms of the chunks before it (of every chunk in
  // workgroup 0, which checks them against the expected totals; thread
  // (part, e) takes chunks part, part + parts, ... of expert e) and the
  // instance lookup tables.
  const int64_t s0 = static_cast<int64_t>(c) * kDispatchChunk + wave * kSlotsPerWave;
  int32_t ev[kSteps];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) ev[s] = a.topk[min(s0 + s * kWave + lane, a.V - 1)];
  const int parts = a.parts;
  const int part = (tid * a.div_E) >> 20, e_t = tid - part * E;  // tid / E, tid % E
  const int nsum = c == 0 ? static_cast<int>(a.ws.n_chunks) : c;
  const int32_t *h = a.ws.hist + e_t;
  const bool many = nsum > kSumFirst * parts;  // else the other loads are skipped
  const bool more = nsum > (kSumFirst + kSumSecond) * parts;
  int hv[kSumFirst], hw[kSumBatch];
#pragma unroll
  for (int u = 0; u < kSumFirst; ++u) hv[u] = h[min(part + u * parts, nsum - 1) * E];
  if (many && part < parts) {
#pragma unroll
    for (int u = 0; u < kSumSecond; ++u)
      hw[u] = h[min(part + (kSumFirst + u) * parts, nsum - 1) * static_cast<int64_t>(E)];
    if (more) {
#pragma unroll
      for (int u = kSumSecond; u < kSumBatch; ++u)
        hw[u] = h[min(part + (kSumFirst + u) * parts, nsum - 1) * static_cast<int64_t>(E)];
    }
  }
  const int exp_tot = c == 0 ? a.ws.exp_tot[e_t] : 0;
  int vhp[kLutIters], vcum[kLutIters], vbase[kLutIters];
  if (a.stage_lut) {
#pragma unroll
    for (int u = 0; u < kLutIters; ++u) {
      if (u * kDlThreads <= E) vhp[u] = a.hp[min(u * kDlThreads + tid, E)];
      if (u * kDlThreads < ncol) {
        const int jj = min(u * kDlThreads + tid, ncol - 1);
        vcum[u] = a.ws.ent_cum[jj];
        vbase[u] = a.ws.ent_base[jj];
      }
    }
  }
  for (int i = tid; i < kDlWaves * E; i += kDlThreads) whist[i] = 0;
  __syncthreads();
  int32_t *wh = whist + wave * E;
  // pass 1: per-wave counts
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    if (s0 + s * kWave + lane >= a.V) ev[s] = -1;
    const int32_t e = ev[s];
    if (e >= 0 && e < E) atomicAdd(wh + e, 1);
  }
  // instance lookup tables, staged in LDS when they fit
  const int32_t *l_hp = a.hp, *l_cum = a.ws.ent_cum, *l_base = a.ws.ent_base;
  if (a.stage_lut) {
    int32_t *p = psum + kDlThreads;
#pragma unroll
    for (int u = 0; u < kLutIters; ++u) {
      const int ii = u * kDlThreads + tid;
      if (ii <= E) p[ii] = vhp[u];
      if (ii < ncol) {
        p[E + 1 + ii] = vcum[u];
        p[E + 1 + ncol + ii] = vbase[u];
      }
    }
    l_hp = p;
    l_cum = p + E + 1;
    l_base = p + E + 1 + ncol;
  }
  // sums over the chunks (further batches of loads when there are more than
  // kSumFirst + kSumBatch chunks per thread)
  {
    int s = 0;
#pragma unroll
    for (int u = 0; u < kSumFirst; ++u) s += part + u * parts < nsum ? hv[u] : 0;
    if (many && part < parts) {
      int c0 = part + kSumFirst * parts;
#pragma unroll
      for (int u = 0; u < kSumSecond; ++u) s += c0 + u * parts < nsum ? hw[u] : 0;
      if (more) {
        int u0 = kSumSecond;
        for (;;) {
#pragma unroll
          for (int u = 0; u < kSumBatch; ++u) s += u >= u0 && c0 + u * parts < nsum ? hw[u] : 0;
          u0 = 0;
          c0 += kSumBatch * parts;
          if (c0 - part >= nsum) break;
#pragma unroll
          for (int u = 0; u < kSumBatch; ++u)
            hw[u] = h[min(c0 + u * parts, nsum - 1) * static_cast<int64_t>(E)];
        }
      }
    }
    psum[tid] = s;
  }
  __syncthreads();
  // base ordinals, then every wave's start in the chunk
  if (tid < E) {
    int run = 0, w[kDlWaves];
    for (int p = 0; p < parts; ++p) run += psum[p * E + tid];
    if (c == 0) {
      if (run != exp_tot) report(a.status, ULTRAEP_EDATA);
      run = 0;
    }
    run += share_before(l_cum, l_hp[tid], ncol);
#pragma unroll
    for (int i = 0; i < kDlWaves; ++i) w[i] = whist[i * E + tid];
#pragma unroll
    for (int i = 0; i < kDlWaves; ++i) {
      whist[i * E + tid] = run;
      run += w[i];
    }
  }
  __syncthreads();
  // pass 2: stable ordinals, instance lookup, rows
  write_rows(a, ev, s0, wh, l_hp, l_cum, l_base);
}

// LDS words of k_dl_one's copies of the earlier ids' counts.
__host__ __device__ __forceinline__ int prev_ints(int copies, int E) {
  return (copies * (E | 1) + 3) / 4 * 4;
}

// The whole layout in one launch, for few chunks: every workgroup builds the
// tables for itself and counts the ids of the chunks before it, which costs
// less than a second launch and the tables' way through memory.  Equal ids of a
// wave add to one LDS address one after another, so the counts of the earlier
// ids are kept in several copies, lane by lane, in different banks: with every
// id the same expert, 10 chunks of E = 64 take 10.4 us (23.5 with one count).
__global__ void __launch_bounds__(kDlThreads) k_dl_one(DlArgs a) {
  extern __shared__ __attribute__((aligned(16))) int32_t lds[];
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int E = a.E, c = blockIdx.x;
  const int stride = E | 1;            // the copies of an expert's count in different banks
  int32_t *whist = lds;                // [kDlWaves][E]
  int32_t *prev = lds + kDlWaves * E;  // [copies][stride] ids of the chunks before
  const int n_cnt = prev_ints(a.copies, E);
  const DlTables t = carve_tables(prev + n_cnt, E, a.ncol);
  DlInputs in;
  in.load(a);
  const int64_t s0 = static_cast<int64_t>(c) * kDispatchChunk + wave * kSlotsPerWave;
  int32_t ev[kSteps], pv[kOneBatch];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) ev[s] = a.topk[min(s0 + s * kWave + lane, a.V - 1)];
  const int n_prev = c * kDispatchChunk;  // all below V
  if (n_prev > 0) {
#pragma unroll
    for (int u = 0; u < kOneBatch; ++u) pv[u] = a.topk[min(u * kDlThreads + tid, n_prev - 1)];
  }
  clear_lds(whist, kDlWaves * E + (n_prev > 0 ? n_cnt : 0));
  for (int b = tid; b < a.R * a.S; b += kDlThreads) t.cnt[b] = 0;
  in.stage(a, t);
  __syncthreads();
  int32_t *wh = whist + wave * E;
  bool bad = false;
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    if (s0 + s * kWave + lane >= a.V) ev[s] = -1;
    const int32_t e = ev[s];
    if (e >= 0 && e < E) atomicAdd(wh + e, 1);
    bad |= e < -1 || e >= E;
  }
  if (bad) report(a.status, ULTRAEP_EDATA);
  int32_t *mine = prev + (lane & (a.copies - 1)) * stride;
  for (int i0 = 0; i0 < n_prev;) {
#pragma unroll
    for (int u = 0; u < kOneBatch; ++u)
      if (i0 + u * kDlThreads + tid < n_prev && pv[u] >= 0 && pv[u] < E) atomicAdd(mine + pv[u], 1);
    i0 += kOneBatch * kDlThreads;
    if (i0 < n_prev) {
#pragma unroll
      for (int u = 0; u < kOneBatch; ++u) pv[u] = a.topk[min(i0 + u * kDlThreads + tid, n_prev - 1)];
    }
  }
  if (!build_tables(a, t, c == 0)) {  // not a plan of this group
    if (tid == 0) report(a.status, ULTRAEP_EDATA);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int64_t i = s0 + s * kWave + lane;
      if (i < a.V) a.row_of_slot[i] = -1;
    }
    return;
  }
  if (tid < E) {
    int run = 0, w[kDlWaves];
    if (n_prev > 0) {
#pragma unroll
      for (int p = 0; p < kOneFew; ++p) {
        const int v = prev[min(p, a.copies - 1) * stride + tid];
        run += p < a.copies ? v : 0;
      }
      if (a.copies > kOneFew) {
#pragma unroll
        for (int p = kOneFew; p < kOneCopies; ++p) {
          const int v = prev[min(p, a.copies - 1) * stride + tid];
          run += p < a.copies ? v : 0;
        }
      }
    }
    const int before = share_before(t.q, t.hp[tid], a.ncol);
#pragma unroll
    for (int i = 0; i < kDlWaves; ++i) w[i] = whist[i * E + tid];
#pragma unroll
    for (int i = 0; i < kDlWaves; ++i) {
      whist[i * E + tid] = before + run;
      run += w[i];
    }
    // the last workgroup has counted every id: the shares have to add up to them
    if (c + 1 == static_cast<int>(gridDim.x) &&
        run != share_before(t.q, t.hp[tid + 1], a.ncol) - before)
      report(a.status, ULTRAEP_EDATA);
  }
  __syncthreads();
  write_rows(a, ev, s0, wh, t.hp, t.q, t.hr);
}

hipError_t launch_dispatch_layout(const int32_t *topk, int64_t V, int32_t rank,
                                  const ultraep_group &g,
                                  const ultraep_plan_buf &plan,
                                  int32_t *row_of_slot, int64_t *block_off,
                                  const DispatchWs &ws, int32_t *status,
                                  hipStream_t stream) {
  DlArgs a;
  a.topk = topk;
  a.V = V;
  a.rank = rank;
  a.R = g.R;
  a.E = g.E;
  a.NS = g.n_slot;
  a.nm = g.E / g.R;
  a.S = a.nm + g.n_slot;
  a.ncol = g.E + g.R * g.n_slot;
  a.nbits = bits_for(g.E);
  // tid * div_E >> 20 is tid / E for tid < 1024: the excess of the product
  // over tid * 2^20 / E is below tid, so below 2^20 / E
  // few enough that adding up an expert's partial sums stays short (E = 1, 16
  // chunks: 19.4 us for the layout with 1024 parts, 8.6 with 16)
  a.parts = kDlThreads / g.E < kSumParts ? kDlThreads / g.E : kSumParts;
  a.div_E = ((1 << 20) + g.E - 1) / g.E;
  a.hp = plan.host_ptr;
  a.hr = plan.host_rank;
  a.hs = plan.host_pslot;
  a.q = plan.reroute + static_cast<int64_t>(rank) * a.ncol;
  a.row_of_slot = row_of_slot;
  a.block_off = block_off;
  a.ws = ws;
  a.status = status;
  a.stage_lut = 0;
  // One launch for up to 10 chunks.  Two launches / one, graph of 20 calls, ids
  // spread over E = 128 (R = 64): 1 chunk 8.7 / 6.0 us, 4 chunks 8.8 / 6.9, 10
  // chunks 9.0 / 8.2, 16 chunks 9.0 / 9.0; two experts alone: 4 chunks 10.0 /
  // 8.5, 10 chunks 10.1 / 10.3, 12 chunks 10.2 / 10.7; one expert alone: 8 chunks
  // 10.9 / 10.3, 10 chunks 10.8 / 11.0, 12 chunks 10.8 / 11.4.  The same line at
  // E = 8, 256 and 512.  Two chunks do with two copies (spread ids 6.7 us against
  // 6.8 with eight, one expert alone 9.7 against 9.2).  Where LDS holds fewer
  // copies the line lies where one expert alone loses about half of what spread
  // ids win, two launches / one: four copies (R = 8, E = 600), 8 chunks 9.7 / 8.3
  // spread and 11.3 / 12.1 alone, 10 chunks 10.1 / 9.0 and 11.7 / 13.2; two (R = 64,
  // E = 640, n_slot = 4), 5 chunks 9.9 / 7.7 and 11.8 / 12.8, 6 chunks 9.8 / 8.3 and
  // 11.8 / 13.9; one (E = 704), 3 chunks 9.7 / 7.7 and 11.7 / 12.8.
  a.copies = ws.n_chunks <= 2 ? kOneFew : kOneCopies;
  const auto lds_for = [&](int copies) {
    return sizeof(int32_t) * static_cast<size_t>(kDlWaves * g.E + prev_ints(copies, g.E) +
                                                 lut_ints(g.E, a.ncol));
  };
  while (a.copies > 1 && lds_for(a.copies) > 64 * 1024) a.copies /= 2;
  const size_t lds_one = lds_for(a.copies);
  // Rows written over the ids (row_of_slot == topk) take two launches unless
  // one workgroup does it all: k_dl_one reads the ids of earlier chunks, which
  // their workgroups may have overwritten by then; k_dl_hist has read them all
  // before k_dl_rows, whose workgroups read their own chunk's and then write it.
  const uintptr_t ids = reinterpret_cast<uintptr_t>(topk), out = reinterpret_cast<uintptr_t>(row_of_slot);
  const uintptr_t span = static_cast<uintptr_t>(V) * sizeof(int32_t);
  const bool apart = ids + span <= out || out + span <= ids;
  const int64_t most = a.copies == kOneCopies ? kOneChunks : a.copies == 4 ? 8 : a.copies == 2 ? 5 : 3;
  if (ws.n_chunks > 0 && ws.n_chunks <= most &&
      (apart || ws.n_chunks == 1) && lds_one <= 64 * 1024) {
    hipLaunchKernelGGL(k_dl_one, dim3(ws.n_chunks), dim3(kDlThreads), lds_one, stream, a);
    return hipGetLastError();
  }
  const size_t lds_hist = sizeof(int32_t) * kDlWaves * g.E;
  const size_t lds_lay = sizeof(int32_t) * static_cast<size_t>(lut_ints(g.E, a.ncol));
  hipLaunchKernelGGL(k_dl_hist, dim3(ws.n_chunks + 1), dim3(kDlThreads),
                     lds_hist > lds_lay ? lds_hist : lds_lay, stream, a);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess || ws.n_chunks == 0) return err;
  size_t lds_rows = sizeof(int32_t) * (kDlWaves * static_cast<size_t>(g.E) + kDlThreads);
  const size_t lut = sizeof(int32_t) * (g.E + 1 + 2 * static_cast<size_t>(a.ncol));
  if (lds_rows + lut <= 64 * 1024) {
    lds_rows += lut;
    a.stage_lut = 1;
  }
  hipLaunchKernelGGL(k_dl_rows, dim3(ws.n_chunks), dim3(kDlThreads), lds_rows, stream, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------- scatter

constexpr int kScThreads = 256;
constexpr int kScWaves = kScThreads / kWave;
// Resident workgroups of the streaming scatter (two per CU); each wave then
// walks tokens t, t + 2048, ...  Whole rows, 256 / 512 / 1024 workgroups over
// rotating buffers, k = 8, us: H = 7168, 4096 tokens 102.3 / 97.5 / 102.3; H = 4096,
// 4096 59.0 / 58.1 / 61.3; H = 2880, 2999 30.6 / 29.8 / 30.1; but narrow rows and
// many tokens do better with more (H = 4096, 8192 123.2 / 119.9 / 116.4; H = 2880,
// 8192 86.8 / 85.7 / 80.6; H = 256, 16384 28.3 / 21.2 / 16.0).
constexpr int kScGrid = 512;
constexpr int64_t kScFill = 2048;  // units that fill the resident waves
constexpr int kScWide = 16;        // 64-chunk steps of a unit of a wide row at most
// dword 3 of a raw buffer resource (32-bit data format) and the store cache
// policy: sc1 streams the rows out at the device scope.  Buffer stores with
// sc1 measured 3-4 % faster than plain or non-temporal global stores.
constexpr uint32_t kRawBufferWord3 = 0x00020000u;
constexpr int kStoreSc1 = 16;

// Stores chunk-lane values of one token (chunks c0 .. c_end - 1, at most 64 U)
// to its k destination rows, one 1 KiB chunk (64 lanes x 16 B) to every row
// before the next chunk.  Each row gets its own buffer resource (base = the
// row, size = the row), so offsets stay 32-bit and anything past the row is
// dropped by the hardware.  kPlain: ordinary stores, see launch_dispatch_scatter.
template <int U, bool kPlain>
__device__ __forceinline__ void store_rows(const v4u (&v)[U], int rows, int k, int64_t V,
                                           int32_t nch, int c0, int c_end, int lane, v4u *send) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int cc = c0 + u * kWave + lane;
    if (cc < c_end) {
      for (int kk = 0; kk < k; ++kk) {
        const int row = readlane(rows, kk);
        if (row >= 0 && row < V) {
          if constexpr (kPlain) {
            send[static_cast<int64_t>(row) * nch + cc] = v[u];
            continue;
          }
          const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
              send + static_cast<int64_t>(row) * nch, 0, static_cast<uint32_t>(nch) * 16u,
              kRawBufferWord3);
          __builtin_amdgcn_raw_buffer_store_b128(v[u], r, static_cast<uint32_t>(cc) * 16u, 0,
                                                 kStoreSc1);
        }
      }
    }
  }
}

// Rows of up to 64 * U chunks (H <= 8192), one unit each, or (kSplit) rows cut
// into `pieces` units of `per` <= 64 * U chunks: persistent waves, each holding
// one unit in registers while the next one is being loaded.  A wave takes `run`
// units in a row (1, or all of a token's) before it goes on by the grid.
template <int U, bool kSplit>
__global__ void __launch_bounds__(kScThreads)
k_scatter(const v4u *__restrict__ x, int64_t T, int32_t k, int32_t nch, int32_t pieces,
          int32_t per, int32_t run, const int32_t *__restrict__ row_of_slot,
          const int64_t *n_routed, v4u *__restrict__ send) {
  constexpr bool kPlain = kSplit && U == kScWide;
  const int lane = lane_id();
  const int64_t V = T * k, n = kSplit ? T * pieces : T;
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kScWaves;
  const int64_t gw = static_cast<int64_t>(blockIdx.x) * kScWaves + threadIdx.x / kWave;
  const auto end_of = [&](int c0) { return kSplit ? min(nch, c0 + per) : nch; };
  const auto fetch = [&](int64_t unit, v4u(&v)[U], int &rows, int &c0) {
    const int64_t t = kSplit ? unit / pieces : unit;
    c0 = kSplit ? static_cast<int>(unit - t * pieces) * per : 0;
    const int c_end = end_of(c0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = c0 + u * kWave + lane;
      if (cc < c_end) v[u] = __builtin_nontemporal_load(x + t * nch + cc);
    }
    rows = lane < k ? row_of_slot[t * k + lane] : -1;
  };
  int64_t unit = kPlain ? gw * run : gw;
  int left = run;
  if (unit < n) {
    v4u v[U];
    int rows, c0;
    fetch(unit, v, rows, c0);
    for (;;) {
      int64_t un = unit + nw;
      if constexpr (kPlain) {
        left = left > 1 ? left - 1 : run;
        un = unit + 1 + (left == run ? (nw - 1) * run : 0);
      }
      v4u w[U];
      int rn = -1, cn = 0;
      if (un < n) fetch(un, w, rn, cn);
      store_rows<U, kPlain>(v, rows, k, V, nch, c0, end_of(c0), lane, send);
      if (un >= n) break;
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = w[u];
      rows = rn;
      c0 = cn;
      unit = un;
    }
  }
  // rows after the routed ones (masked slots) are zero-filled
  // a routed count outside [0, V] (not a layout of these slots) fills no row
  const int64_t nr = *n_routed;
  if (nr >= 0 && nr < V) {
    const v4u z = v4u{0u, 0u, 0u, 0u};
    for (int64_t row = nr + gw; row < V; row += nw)
      for (int cc = lane; cc < nch; cc += kWave) send[row * nch + cc] = z;
  }
}

template <int U, bool kSplit>
static void start_scatter(const v4u *x, int64_t T, int32_t k, int32_t nch, const int32_t *row_of_slot,
                          const int64_t *n_routed, v4u *send, hipStream_t stream, bool together) {
  const int32_t pieces = kSplit ? (nch + U * kWave - 1) / (U * kWave) : 1;
  // the pieces of a wide row are equal, in whole 128-byte lines of an aligned row
  const int32_t per = U == kScWide ? ((nch + pieces - 1) / pieces + 7) / 8 * 8 : U * kWave;
  const int32_t run = together ? pieces : 1;
  const int64_t need = (T * (pieces / run) + kScWaves - 1) / kScWaves;
  hipLaunchKernelGGL((k_scatter<U, kSplit>), dim3(static_cast<unsigned>(need < kScGrid ? need : kScGrid)),
                     dim3(kScThreads), 0, stream, x, T, k, nch, pieces, per, run,
                     row_of_slot, n_routed, send);
}

hipError_t launch_dispatch_scatter(const uint16_t *x, int64_t T, int32_t k,
                                   int32_t H, const int32_t *row_of_slot,
                                   const int64_t *n_routed, uint16_t *send,
                                   hipStream_t stream) {
  const int32_t nch = H / 8;
  const int per_lane = nch / kWave + (nch % kWave != 0);
  const v4u *xs = reinterpret_cast<const v4u *>(x);
  v4u *sd = reinterpret_cast<v4u *>(send);
  const auto start = [&](auto f, bool together = false) {
    f(xs, T, k, nch, row_of_slot, n_routed, sd, stream, together);
  };
  // Whole rows per wave keep the stores of a row together; they are cut where
  // that leaves waves idle or where a row does not fit the registers.  Measured
  // over rotating buffers (past the last-level cache), us.
  // Rows of up to 16 steps of 64 chunks are cut below `whole` tokens (below 768 where
  // they are no whole lines: k = 12, H = 7240, 633 tokens 35.2 / 33.9), whole / cut,
  // k = 8: H = 4096, 511 tokens 10.4 / 8.2, 700 11.4 / 10.9; H = 5120, 600 12.4 /
  // 11.4, 700 12.8 / 15.6; H = 7168, 511 15.7 / 13.2, 640 16.5 / 17.4, 767 18.3 /
  // 19.6; k = 16: H = 4096, 511 15.1 / 14.1, 700 17.6 / 18.9; H = 5120, 600 19.4 /
  // 20.7; H = 1024, 640 6.2 / 5.6; k = 12: H = 3712, 597 in a whole step 53.4 / 51.5;
  // k = 1: H = 7168, 767 9.0 / 7.9.  More rows a token keep the memory busy with
  // fewer waves.
  // The units are the widest that are enough: of 4 steps and more, a third over
  // the resident waves, as a few units over them leave the second turn nearly
  // empty (4 / 2 steps: H = 6144, k = 8, 683 tokens, 2049 / 4098 units 18.9 / 15.1;
  // H = 5120, k = 2, 767, 2301 / 3835 8.3 / 6.5; H = 8192, k = 8, 600, 2400 / 4800
  // 19.3 / 17.8).
  // Wide rows that are no whole lines take equal pieces of up to 16 steps and
  // ordinary stores from 800 units on: sc1 stores pass the L2 by, which otherwise
  // joins the lines that two rows or two pieces share.  One wave per token walking
  // the row in passes / units of 8 steps, sc1 / these: H = 8200, 4096 tokens, k = 1
  // 31.5 / 37.4 / 31.1, k = 8 154 / 176 / 155; H = 12296, 519, k = 4 19.1 / 22.8 / 15.6.
  // Below, and where all buffers stay in the last-level cache, units of up to 8
  // steps are ahead (three states of 56 MB in turn, 355 tokens of H = 8744, k = 8,
  // with the plan and the combine 60.6 us, these 63.3; three of 106 MB, 612 of H =
  // 9592 27.2 and 28.6).  With many rows one wave writes a token's pieces one after
  // another; pieces dealt to all waves / to the token's: H = 10008, 519 tokens, k =
  // 16 51.8 / 41.8, k = 8 23.2 / 21.8, k = 6 17.6 / 18.3; H = 12296, 1500, k = 12 134.5 /
  // 121.1, k = 2 21.7 / 21.8, 400, k = 16 43.8 / 37.4, k = 10 24.7 / 27.2.
  // Rows of whole lines, or halves, do so for one row a token only (H = 12288, 1500
  // tokens 17.9 / 21.1 / 15.9): with more, ordinary stores leave their write-back to
  // the next kernel (a whole step, H = 9216, 9834 tokens, k = 2 159 with sc1, 164
  // without; H = 10720, 3340, k = 8 197 and 204, but H = 10952, 1557, k = 8, no whole
  // halves, 136 and 120).
  const auto units = [&](int u) { return T * ((per_lane + u - 1) / u); };
  const bool wide = per_lane > kScWide;
  const bool lines = nch % 4 == 0;  // rows of whole 64-byte halves of a line
  const int64_t whole = nch % 8 || per_lane <= 2 ? 768
                        : per_lane <= 8 ? (k >= 16 ? 512 : 768)
                                        : (k >= 12 ? 512 : k >= 8 ? 640 : 768);
  if (wide && units(kScWide) >= (lines ? (k == 1 ? 2 * kScFill / 3 : INT64_MAX) : 800)) {
    start(start_scatter<kScWide, true>, !lines && T * k >= (T >= 500 ? 4000 : 6400));
  } else if (wide || (per_lane > 1 && T < whole)) {
    if (per_lane > 8 && units(8) >= kScFill * 4 / 3) start(start_scatter<8, true>);
    else if (per_lane > 4 && units(4) >= kScFill * 4 / 3) start(start_scatter<4, true>);
    else if (per_lane > 2 && units(2) >= kScFill) start(start_scatter<2, true>);
    else start(start_scatter<1, true>);
  } else if (per_lane <= 1) {
    start(start_scatter<1, false>);
  } else if (per_lane <= 2) {
    start(start_scatter<2, false>);
  } else if (per_lane <= 4) {
    start(start_scatter<4, false>);
  } else if (per_lane <= 8) {
    start(start_scatter<8, false>);
  } else if (per_lane <= 14) {
    start(start_scatter<14, false>);
  } else {
    start(start_scatter<16, false>);
  }
  return hipGetLastError();
}

}  // namespace uep
