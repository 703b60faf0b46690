// Reverse reroute: the combine gather.  After the experts have run, each
// source rank gets its rows back in the dispatch layout; token t's output
// is the gate-weighted sum of the rows its k slots were sent to (the
// scatter-to-gather inversion of the forward token assignment, Sec. 4.2).
//
// Arithmetic (the paper fixes bf16 activations only; this library and its
// tests read it so): every product gate * row and every partial sum is an
// fp32 value (no fused multiply-add), the sum runs over k ascending from
// +0, masked slots (row -1) add nothing, and the fp32 result is rounded to
// bf16 to nearest-even, every NaN to 0x7FC0.
//
// Bandwidth bound: each routed row is read once, each output row written
// once.  A wave takes a work unit of two 16-byte chunks (8 bf16 each) per
// lane of one token's row, issues the k rows' loads of both chunks together
// (16 loads in flight for k = 8), accumulates and stores.  Many short waves
// keep the most row reads in flight: on the DeepSeek-V3-shaped layer this
// measured 90 us against 99-121 us for persistent waves that walk whole
// rows, and against 92-105 us for units of 1, 3 or 4 chunks per lane.
// More than 8 rows per token run in groups of 8, the sums carried in
// registers from group to group: 3001 tokens of k = 12, H = 4104 (300 MB)
// take 52.7 us (5.7 TB/s), against 82.8 us (3.6 TB/s) with one row's load in
// flight at a time.  Groups of 4 or 6 rows, groups of equal size, and 12 or 16
// rows together measured the same or up to 15 % slower.  Where a call has few
// units or a row is short, latency and instructions bound it instead: there the
// loads take no branch (bounds-checked buffer loads, so a masked row reads
// nothing and counts as +0 times +0).  With a branch around each load the
// one-chunk kernel waits for a load before it issues the next one: 300 tokens of
// k = 16, H = 512 took 10.0 us, now 5.7 (8.7 with one row in flight).
#include "common.hpp"
#include "kernels.hpp"

#pragma clang fp contract(off)

namespace uep {

constexpr int kCbThreads = 256;
constexpr int kCbWaves = kCbThreads / kWave;
constexpr int kCbGrid = 65535;
constexpr int kCbRows = 8;  // rows loaded together per chunk
constexpr int kCbChunks = 2;       // k <= kCbRows: 16-byte chunks per lane per step
constexpr int kCbLaneChunks = 2;   //               and per lane per work unit
// dword 3 of a raw buffer resource (32-bit data format), non-temporal loads
constexpr uint32_t kRawBufferWord3 = 0x00020000u;
constexpr int kLoadNt = 2;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// fp32 -> bf16, round to nearest-even by adding 0x7FFF plus the kept
// part's lowest bit before dropping 16 bits; NaN -> 0x7FC0
__device__ __forceinline__ uint32_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ void acc_chunk(float (&acc)[8], float g, v4u v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[2 * i] = __fadd_rn(acc[2 * i], __fmul_rn(g, bf16_lo(w[i])));
    acc[2 * i + 1] = __fadd_rn(acc[2 * i + 1], __fmul_rn(g, bf16_hi(w[i])));
  }
}

__device__ __forceinline__ v4u pack_chunk(const float (&acc)[8]) {
  v4u o;
  o.x = to_bf16(acc[0]) | (to_bf16(acc[1]) << 16);
  o.y = to_bf16(acc[2]) | (to_bf16(acc[3]) << 16);
  o.z = to_bf16(acc[4]) | (to_bf16(acc[5]) << 16);
  o.w = to_bf16(acc[6]) | (to_bf16(acc[7]) << 16);
  return o;
}

// rows of token t for this lane (lane < k); -1 = masked; out-of-range rows
// are reported and treated as masked
__device__ __forceinline__ void token_rows(const int32_t *row_of_slot, const float *gate,
                                           int64_t t, int k, int lane, int64_t n_rows,
                                           int32_t *status, int &row, float &g) {
  row = -1;
  g = 0.f;
  if (lane < k) {
    row = row_of_slot[t * k + lane];
    g = gate[t * k + lane];
    if (row < -1 || row >= n_rows) {
      report(status, ULTRAEP_EDATA);
      row = -1;
    }
  }
}

// k <= kCbRows.  Work unit: kCbLaneChunks 16-byte chunks per lane of one
// token's row; the k rows' loads of kCbChunks chunks are in flight together.
__global__ void __launch_bounds__(kCbThreads)
k_combine(const v4u *__restrict__ y, int64_t n_rows, const float *__restrict__ gate,
          const int32_t *__restrict__ row_of_slot, int64_t T, int32_t k, int32_t nch,
          v4u *__restrict__ out, int32_t *status) {
  const int lane = lane_id();
  const int nblk = (nch + kCbLaneChunks * kWave - 1) / (kCbLaneChunks * kWave);
  const int64_t n_units = T * nblk;
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kCbWaves;
  for (int64_t unit = static_cast<int64_t>(blockIdx.x) * kCbWaves + threadIdx.x / kWave;
       unit < n_units; unit += nw) {
    const int64_t t = unit / nblk;
    const int b = static_cast<int>(unit - t * nblk);
    int row;
    float g;
    token_rows(row_of_slot, gate, t, k, lane, n_rows, status, row, g);
    const int c_end = min(nch, (b + 1) * kCbLaneChunks * kWave);
    for (int c0 = b * kCbLaneChunks * kWave + lane; c0 < c_end; c0 += kCbChunks * kWave) {
      v4u v[kCbChunks][kCbRows];
#pragma unroll
      for (int kk = 0; kk < kCbRows; ++kk) {
        const int r = kk < k ? readlane(row, kk) : -1;
#pragma unroll
        for (int u = 0; u < kCbChunks; ++u) {
          const int cc = c0 + u * kWave;
          if (r >= 0 && cc < c_end)
            v[u][kk] = __builtin_nontemporal_load(y + static_cast<int64_t>(r) * nch + cc);
        }
      }
#pragma unroll
      for (int u = 0; u < kCbChunks; ++u) {
        const int cc = c0 + u * kWave;
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < kCbRows; ++kk) {
          const int r = kk < k ? readlane(row, kk) : -1;
          if (r >= 0 && cc < c_end)
            acc_chunk(acc, __int_as_float(readlane(__float_as_int(g), kk)), v[u][kk]);
        }
        if (cc < c_end) __builtin_nontemporal_store(pack_chunk(acc), out + t * nch + cc);
      }
    }
  }
}

// k > kCbRows: up to kCh 16-byte chunks per lane of one token's row, `per`
// chunks in all (nblk equal units per row); the loads of kCbRows rows are in
// flight together, then those of the next group.  kFew: loads without a branch
// (a resource per row; chunks from c_end on, and all of a masked row's, are out
// of its bounds and load as 0), and only the rows past k are left out of the
// sums: a masked row adds gate 0 times 0, which changes no sum (none is -0).
template <int kCh, bool kFew>
__global__ void __launch_bounds__(kCbThreads)
k_combine_many(const v4u *__restrict__ y, int64_t n_rows, const float *__restrict__ gate,
               const int32_t *__restrict__ row_of_slot, int64_t T, int32_t k, int32_t nch,
               int32_t nblk, int32_t per, v4u *__restrict__ out, int32_t *status) {
  const int lane = lane_id();
  const int64_t n_units = T * nblk;
  const int64_t nw = static_cast<int64_t>(gridDim.x) * kCbWaves;
  for (int64_t unit = static_cast<int64_t>(blockIdx.x) * kCbWaves + threadIdx.x / kWave;
       unit < n_units; unit += nw) {
    const int64_t t = unit / nblk;
    const int b = static_cast<int>(unit - t * nblk);
    int row;
    float g;
    token_rows(row_of_slot, gate, t, k, lane, n_rows, status, row, g);
    if (kFew && row < 0) g = 0.f;
    const int c0 = b * per + lane, c_end = min(nch, (b + 1) * per);
    // (uniform, and known to be: a resource in scalar registers)
    const uint32_t bytes = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(c_end)) * 16u;
    float acc[kCh][8] = {};
    for (int k0 = 0; k0 < k; k0 += kCbRows) {
      v4u v[kCh][kCbRows];
#pragma unroll
      for (int kk = 0; kk < kCbRows; ++kk) {
        // k <= 64, so the lane read is in the wave; lanes past k hold -1
        const int r = kFew || k0 + kk < k ? readlane(row, k0 + kk) : -1;
        if constexpr (kFew) {
          const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
              const_cast<v4u *>(y) + static_cast<int64_t>(max(r, 0)) * nch, 0,
              r < 0 ? 0u : bytes, kRawBufferWord3);
#pragma unroll
          for (int u = 0; u < kCh; ++u)
            v[u][kk] = __builtin_amdgcn_raw_buffer_load_b128(
                rs, static_cast<uint32_t>(c0 + u * kWave) * 16u, 0, kLoadNt);
        } else {
#pragma unroll
          for (int u = 0; u < kCh; ++u) {
            const int cc = c0 + u * kWave;
            if (r >= 0 && cc < c_end)
              v[u][kk] = __builtin_nontemporal_load(y + static_cast<int64_t>(r) * nch + cc);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kCh; ++u) {
#pragma unroll
        for (int kk = 0; kk < kCbRows; ++kk) {
          const int r = k0 + kk < k ? (kFew ? 0 : readlane(row, k0 + kk)) : -1;
          if (r >= 0 && (kFew || c0 + u * kWave < c_end))
            acc_chunk(acc[u], __int_as_float(readlane(__float_as_int(g), k0 + kk)), v[u][kk]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kCh; ++u) {
      const int cc = c0 + u * kWave;
      if (cc < c_end) __builtin_nontemporal_store(pack_chunk(acc[u]), out + t * nch + cc);
    }
  }
}

static dim3 combine_grid(int64_t units) {
  const int64_t need = (units + kCbWaves - 1) / kCbWaves;
  return dim3(static_cast<unsigned>(need < kCbGrid ? need : kCbGrid));
}

template <int kCh, bool kFew>
static void start_many(const v4u *y, int64_t n_rows, const float *gate, const int32_t *row_of_slot,
                       int64_t T, int32_t k, int32_t nch, v4u *out, int32_t *status,
                       hipStream_t stream) {
  // equal units per row, so that a row a little over a multiple of the
  // unit's width leaves no nearly empty wave; in whole 128-byte lines
  const int32_t nblk = (nch + kCh * kWave - 1) / (kCh * kWave);
  const int32_t per = ((nch + nblk - 1) / nblk + 7) / 8 * 8;
  hipLaunchKernelGGL((k_combine_many<kCh, kFew>), combine_grid(T * nblk), dim3(kCbThreads), 0, stream, y,
                     n_rows, gate, row_of_slot, T, k, nch, nblk, per, out, status);
}

hipError_t launch_combine(const uint16_t *y, int64_t n_rows, const float *gate,
                          const int32_t *row_of_slot, int64_t T, int32_t k, int32_t H,
                          uint16_t *out, int32_t *status, hipStream_t stream) {
  const int32_t nch = H / 8;
  const v4u *ys = reinterpret_cast<const v4u *>(y);
  v4u *os = reinterpret_cast<v4u *>(out);
  // k > kCbRows takes the rows in groups of kCbRows.  One chunk per lane where
  // one-chunk units fill at least 95 % of their lanes, two where they do not
  // (fewer partly filled waves).  Measured, one / two chunks, T = 3001 rows of
  // k = 12: H = 7168 85.8 / 89.1 us, 4096 50.0 / 51.2, 5608 70.1 / 71.8; but
  // 4104 (89 % filled) 55.3 / 52.7, 2880 (94 %) 39.4 / 37.0, and 520 (51 %,
  // T = 16000) 46.4 / 40.5.  Rows of one chunk per lane, and calls of few
  // units, load without branches.  Measured over rotating buffers, with one row
  // in flight / one or two chunks as above / without branches: H = 256, k = 10,
  // T = 1 3.7 / 4.5 / 3.4 us, T = 300 6.3 / 5.3 / 4.6, T = 16000 24.5 / 25.9 /
  // 21.6; T = 33, H = 1024, k = 12 7.9 / 8.2 / 5.3; T = 300, H = 4096, k = 12
  // (2400 units) 55.9 / 10.7 / 8.6; with full rows of one chunk (H = 512, k = 12)
  // T = 300 7.2 / 8.0 / 5.4 and T = 3001 13.8 / 11.2 / 9.4.  Above the lines the
  // rest is ahead by up to 4 % (H = 4096, k = 12, T = 3001 53.5 / 55.7; H = 7168,
  // k = 9, T = 300 10.8 / 11.2).  One row in flight stays ahead where a row is a
  // few lanes and tokens are many (H = 8, k = 9, T = 16000 12.5 / 23.1 / 15.4).
  const int64_t ones = (nch + kWave - 1) / kWave;
  const bool full = 20 * static_cast<int64_t>(nch) >= 19 * kWave * ones;
  if (k <= kCbRows)
    hipLaunchKernelGGL(k_combine,
                       combine_grid(T * ((nch + kCbLaneChunks * kWave - 1) / (kCbLaneChunks * kWave))),
                       dim3(kCbThreads), 0, stream, ys, n_rows, gate, row_of_slot, T, k, nch, os,
                       status);
  else if (T * ones <= (ones == 1 ? 6000 : 2400) || (ones == 1 && !full))
    start_many<1, true>(ys, n_rows, gate, row_of_slot, T, k, nch, os, status, stream);
  else if (full)
    start_many<1, false>(ys, n_rows, gate, row_of_slot, T, k, nch, os, status, stream);
  else
    start_many<2, false>(ys, n_rows, gate, row_of_slot, T, k, nch, os, status, stream);
  return hipGetLastError();
}

}  // namespace uep
