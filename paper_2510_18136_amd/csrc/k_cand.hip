// Candidate extraction (threshold + top-K by S/N).
//
// Paper section 2.2: a 6-sigma S/N threshold turns the maximum-S/N maps into
// candidates; section 2.3: post-processing keeps the ten highest-S/N ones.
// Here one candidate is a pixel whose best (DM, width) trial has S/N >= theta.
// Candidates are ordered by S/N descending, then pixel index ascending; the
// first K are returned together with the total count.
//
// Each candidate is encoded as a 64-bit key whose unsigned order is that
// ranking: high word = order-preserving bits of the FP32 S/N, low word =
// ~pixel.
//
// k_cand_top (short lists): every workgroup keeps the top K of its pixels, and
// the last one to finish merges them, so one launch does it for a cube or for
// every cube of a batch. What bounds it is latency, a chain of barriers: the
// K-th largest S/N is found bit by bit (one compare per key in registers, one
// barrier per bit) and only the K keys left are ranked, each by counting the
// larger ones. The compaction, 8-bit radix selection by one workgroup and
// bitonic sort it replaces took 65 us for 4,096 pixels, 92 us for 20,000 and
// 195 us for 65,536 with three launches and two copies; they stay for lists too
// long for the merge (top_blocks).
//
// Records and counts are written straight to pinned host memory (a few hundred
// bytes; no copies follow). The run's flag counter is handed over with them and
// left at zero for the next run.
#include "device_common.h"
#include "nsfrb_internal.h"
#include "../../include/nsfrb.h"

namespace nsfrb {

constexpr int kSortCap = 4096;     // keys sorted directly in LDS
constexpr int kSelThreads = 1024;

__device__ __forceinline__ uint32_t ordered_bits(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float unordered_bits(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

constexpr int kTopThreads = 256;
constexpr int kTopMerge = 4096;    // keys the last workgroup merges (kTopMerge / kTopThreads per thread, in registers)
constexpr int kTopMaxK = 256;      // the K kept are ranked against each other: quadratic
constexpr int kTopMaxPer = 32;     // pixels per thread

__device__ __forceinline__ int block_sum(int v, int* sh) {    // v uniform per wave; sh: one slot per wave
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) sh[w] = v;
  __syncthreads();
  int s = 0;
#pragma unroll
  for (int k = 0; k < kTopThreads / kWave; ++k) s += sh[k];
  return s;
}

// Largest T such that at least K of the block's keys are >= T (0 if there are
// fewer than K nonzero keys): the K-th largest key, or less once exactly K keys
// are >= T. sh: 2 * (waves) slots.
template <int N>
__device__ __forceinline__ uint32_t kth_largest(const uint32_t (&key)[N], int K, int* sh) {
  constexpr int W = kTopThreads / kWave;
  uint32_t T = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t t = T | (1u << bit);
    int c = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) c += popc64(ballot(key[i] >= t));
    c = block_sum(c, sh + W * (bit & 1));
    if (c >= K) T = t;
    if (c == K) break;                                        // uniform: every thread has the same count
  }
  __syncthreads();
  return T;
}

// A workgroup's LDS, declared by the kernels: the batch kernel holds every PER's
// code, and an array of each's own would be four times this.
struct TopShared {
  unsigned long long s[kTopMaxK];        // keys to rank
  int sh[2 * kTopThreads / kWave], fill, last;
};

// Pixels PER * kTopThreads of one cube by one workgroup.
template <int PER>
__device__ __forceinline__ void cand_top(const CandDesc& d, int blk, TopShared& lds) {
  unsigned long long* s = lds.s;
  int *sh = lds.sh, &fill = lds.fill, &last = lds.last;
  if (blk >= d.blocks) return;
  const int tid = threadIdx.x, K = d.k_max;
  const int p0 = blk * PER * kTopThreads;
  if (tid == 0) fill = 0;
  uint32_t key[PER];
  int hits = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int p = p0 + i * kTopThreads + tid;
    const float v = p < d.n_pix ? d.best_snr[p] : -__builtin_inff();
    const bool hit = __builtin_isfinite(v) && v >= d.theta;
    key[i] = hit ? ordered_bits(v) : 0u;                      // (a hit's bits are never 0)
    hits += popc64(ballot(hit));
  }
  hits = block_sum(hits, sh);
  __syncthreads();
  // keys above T, then, if the K-th is tied, the tied ones of the smallest pixels
  const uint32_t T = hits > K ? kth_largest<PER>(key, K, sh) : 1u;
  int above = 0, equal = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    above += popc64(ballot(key[i] > T));
    equal += popc64(ballot(key[i] == T));
  }
  above = block_sum(above, sh);
  __syncthreads();
  equal = block_sum(equal, sh);
  int ties = above + equal > K ? K - above : equal;           // ties kept (all of them unless the list would overflow)
  const bool all_ties = ties == equal;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    bool keep = key[i] > T || (all_ties && key[i] == T);
    if (!all_ties) {                                          // uniform: pixels in order, i outermost
      const bool tie = key[i] == T;
      const uint64_t m = ballot(tie);
      __syncthreads();
      const int before_me = lanes_below(m);
      if (lane_id() == 0) sh[tid / kWave] = popc64(m);
      __syncthreads();
      int before = 0, total = 0;
      for (int k = 0; k < kTopThreads / kWave; ++k) {
        before += k < tid / kWave ? sh[k] : 0;
        total += sh[k];
      }
      keep = keep || (tie && before + before_me < ties);
      ties = max(0, ties - total);
    }
    if (keep)
      s[atomicAdd(&fill, 1)] = ((unsigned long long)key[i] << 32) |
                               (unsigned long long)(0xffffffffu - (uint32_t)(p0 + i * kTopThreads + tid));
  }
  __syncthreads();
  int n = fill, total = hits;                                 // keys to rank, pixels at or above the threshold
  if (d.blocks > 1) {
    for (int i = tid; i < n; i += kTopThreads) d.keys[(size_t)blk * K + i] = s[i];
    if (tid == 0) {
      d.count[2 + blk] = n;
      atomicAdd(&d.count[0], hits);
    }
    // keys and counts before the ticket: every wave writes back and waits for its
    // own stores (a barrier alone does not wait for stores, and the workgroup that
    // merges may sit on another XCD, behind another L2)
    __threadfence();
    __syncthreads();
    // (the last ticket wraps the counter to 0 by itself: should the runs of one
    // handle ever overlap, no reset loses the other's tickets, and the next run
    // starts from 0 again)
    if (tid == 0) last = atomicInc((unsigned*)&d.count[1], (unsigned)d.blocks - 1) == (unsigned)d.blocks - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();                                          // the others' keys after it
    // merge: at most kTopMerge keys, thread t holding every kTopThreads-th
    constexpr int PM = kTopMerge / kTopThreads;
    if (tid == 0) total = atomicExch(&d.count[0], 0);         // (only this thread reports it)
    unsigned long long k64[PM];
    uint32_t k32[PM];
    n = 0;
#pragma unroll
    for (int i = 0; i < PM; ++i) {
      const int q = i * kTopThreads + tid, b = q / K, j = q - b * K;
      const bool ok = b < d.blocks && j < __hip_atomic_load(&d.count[2 + (b < d.blocks ? b : 0)], __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
      k64[i] = ok ? __hip_atomic_load(&d.keys[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
      k32[i] = (uint32_t)(k64[i] >> 32);
      n += popc64(ballot(ok));
    }
    n = block_sum(n, sh);
    __syncthreads();
    const uint32_t Tm = n > K ? kth_largest<PM>(k32, K, sh) : 1u;
    if (tid == 0) fill = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PM; ++i)
      if (k32[i] >= Tm) {
        const int at = atomicAdd(&fill, 1);
        if (at < kTopMaxK) s[at] = k64[i];
      }
    __syncthreads();
    n = fill;                                                 // K, or more if the K-th is tied
    if (__builtin_expect(n > kTopMaxK, 0)) {
      // too many ties to rank: only those of the smallest pixels, whose low words
      // are the largest (4,096 equal keys ranked took 0.89 ms, so 0.04)
      int above = 0;
      uint32_t low[PM];
#pragma unroll
      for (int i = 0; i < PM; ++i) {
        above += popc64(ballot(k32[i] > Tm));
        low[i] = k32[i] == Tm ? (uint32_t)k64[i] : 0u;
      }
      above = block_sum(above, sh);
      __syncthreads();
      const uint32_t Tp = max(1u, kth_largest<PM>(low, K - above, sh));
      if (tid == 0) fill = 0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < PM; ++i)
        if (k32[i] > Tm || low[i] >= Tp) {
          const int at = atomicAdd(&fill, 1);
          if (at < kTopMaxK) s[at] = k64[i];
        }
      __syncthreads();
      n = fill;
    }
    n = min(n, kTopMaxK);                                     // (more only if runs overlap)
  }
  const int kept = n < K ? n : K;
  for (int r = tid; r < n; r += kTopThreads) {
    const unsigned long long k = s[r];
    int rank = 0;
    for (int q = 0; q < n; ++q) rank += s[q] > k;
    const int p = (int)(0xffffffffu - (uint32_t)(k & 0xffffffffull));
    if (rank >= K || (uint32_t)p >= (uint32_t)d.n_pix) continue;   // (every key names a pixel, unless runs overlap)
    nsfrb_candidate c;
    c.x = p % d.nx;
    c.y = p / d.nx;
    c.dm_index = d.best_d[p];
    c.width_index = d.best_w[p];
    c.toa = d.best_t[p];
    c.snr = unordered_bits((uint32_t)(k >> 32));
    ((nsfrb_candidate*)d.out)[rank] = c;
  }
  if (tid == 0) {
    d.n_out[0] = kept;
    d.n_out[1] = total;
    *(unsigned long long*)(d.n_out + 2) = atomicExch(d.flags, 0ull);
  }
}

template <int PER>
__global__ __launch_bounds__(kTopThreads) void k_cand_top(CandDesc d) {
  __shared__ TopShared lds;
  cand_top<PER>(d, blockIdx.x, lds);
}
// Cube blockIdx.y of a batch.
__global__ __launch_bounds__(kTopThreads) void k_cand_top_batch(const CandDesc* __restrict__ descs) {
  __shared__ TopShared lds;
  const CandDesc d = descs[blockIdx.y];
  switch (d.per) {
    case 4: cand_top<4>(d, blockIdx.x, lds); break;
    case 8: cand_top<8>(d, blockIdx.x, lds); break;
    case 16: cand_top<16>(d, blockIdx.x, lds); break;
    default: cand_top<kTopMaxPer>(d, blockIdx.x, lds);
  }
}

__global__ void k_cand_zero(int* count) { if (threadIdx.x == 0) { count[0] = 0; } }

__global__ __launch_bounds__(256) void k_cand_compact(const float* __restrict__ best, int n_pix, float theta,
                                                      unsigned long long* __restrict__ keys, int* __restrict__ count) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  bool hit = false;
  float v = 0.f;
  if (p < n_pix) {
    v = best[p];
    hit = __builtin_isfinite(v) && v >= theta;
  }
  const uint64_t m = ballot(hit);
  if (m == 0) return;
  const int leader = __ffsll((long long)m) - 1;
  int base = 0;
  if (lane_id() == leader) base = atomicAdd(count, popc64(m));
  base = __shfl(base, leader);
  if (hit) {
    const int pos = base + lanes_below(m);
    keys[pos] = ((unsigned long long)ordered_bits(v) << 32) | (unsigned long long)(0xffffffffu - (uint32_t)p);
  }
}

// Bitonic sort, descending, of n2 (power of two) keys in LDS.
__device__ void block_sort_desc(unsigned long long* s, int n2) {
  for (int k = 2; k <= n2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < n2; i += blockDim.x) {
        const int ixj = i ^ j;
        if (ixj > i) {
          const unsigned long long a = s[i], b = s[ixj];
          const bool desc = (i & k) == 0;
          if (desc ? (a < b) : (a > b)) { s[i] = b; s[ixj] = a; }
        }
      }
      __syncthreads();
    }
  }
}

__global__ __launch_bounds__(kSelThreads) void k_cand_select(
    const unsigned long long* __restrict__ keys, const int* __restrict__ count, int k_max, int nx,
    const int* __restrict__ best_d, const int* __restrict__ best_w, const int* __restrict__ best_t,
    nsfrb_candidate* __restrict__ out, int* __restrict__ n_out, unsigned long long* __restrict__ flags) {
  __shared__ unsigned long long s[kSortCap];
  __shared__ uint32_t hist[256];
  __shared__ unsigned long long prefix_sh, mask_sh;
  __shared__ int need_sh, fill_sh;
  const int n = count[0];
  const int K = n < k_max ? n : k_max;
  int m = n;                                  // keys that go into the LDS sort
  if (n > kSortCap) {
    // radix-select the K-th largest key: fix the key 8 bits at a time from the top
    if (threadIdx.x == 0) { prefix_sh = 0; mask_sh = 0; need_sh = K; }
    __syncthreads();
    for (int shift = 56; shift >= 0; shift -= 8) {
      for (int i = threadIdx.x; i < 256; i += blockDim.x) hist[i] = 0;
      __syncthreads();
      const unsigned long long pre = prefix_sh, msk = mask_sh;
      for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const unsigned long long k = keys[i];
        if ((k & msk) == pre) atomicAdd(&hist[(k >> shift) & 0xff], 1u);
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        int need = need_sh;
        int dsel = 0;
        for (int dg = 255; dg >= 0; --dg) {
          if ((int)hist[dg] >= need) { dsel = dg; break; }
          need -= (int)hist[dg];
        }
        need_sh = need;
        prefix_sh = pre | ((unsigned long long)dsel << shift);
        mask_sh = msk | (0xffull << shift);
      }
      __syncthreads();
    }
    // prefix_sh is now the K-th largest key; gather every key >= it (exactly K)
    const unsigned long long thr = prefix_sh;
    if (threadIdx.x == 0) fill_sh = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const unsigned long long k = keys[i];
      if (k >= thr) { const int pos = atomicAdd(&fill_sh, 1); if (pos < kSortCap) s[pos] = k; }
    }
    __syncthreads();
    m = K;
  } else {
    for (int i = threadIdx.x; i < n; i += blockDim.x) s[i] = keys[i];
  }
  int n2 = 1;
  while (n2 < m) n2 <<= 1;
  for (int i = m + threadIdx.x; i < n2; i += blockDim.x) s[i] = 0ull;
  __syncthreads();
  if (n2 > 1) block_sort_desc(s, n2);
  for (int i = threadIdx.x; i < K; i += blockDim.x) {
    const unsigned long long k = s[i];
    const int p = (int)(0xffffffffu - (uint32_t)(k & 0xffffffffull));
    nsfrb_candidate c;
    c.x = p % nx;
    c.y = p / nx;
    c.dm_index = best_d[p];
    c.width_index = best_w[p];
    c.toa = best_t[p];
    c.snr = unordered_bits((uint32_t)(k >> 32));
    out[i] = c;
  }
  if (threadIdx.x == 0) {
    n_out[0] = K;
    n_out[1] = n;
    *(unsigned long long*)(n_out + 2) = atomicExch(flags, 0ull);
  }
}

// Pixels per thread of the short-list kernel: as few as leave the last
// workgroup at most kTopMerge keys to merge (the workgroups run at once, so
// fewer pixels each is faster); 0 if the list is too long for it.
static int top_pixels_per_thread(int n_pix, int k_max) {
  if (k_max > kTopMaxK) return 0;
  for (int per = 4; per <= kTopMaxPer; per *= 2) {
    const long long blocks = ((long long)n_pix + per * kTopThreads - 1) / (per * kTopThreads);
    if (blocks * k_max <= kTopMerge) return per;
  }
  return 0;
}
void plan_candidates_list(CandDesc& d) {
  d.per = top_pixels_per_thread(d.n_pix, d.k_max);
  d.blocks = d.per ? (d.n_pix + d.per * kTopThreads - 1) / (d.per * kTopThreads) : 0;
}
int cand_counters() { return kTopMerge + 2; }

hipError_t launch_candidates(const CandDesc& a, hipStream_t st) {
  switch (a.per) {
    case 4: hipLaunchKernelGGL(k_cand_top<4>, dim3(a.blocks), dim3(kTopThreads), 0, st, a); break;
    case 8: hipLaunchKernelGGL(k_cand_top<8>, dim3(a.blocks), dim3(kTopThreads), 0, st, a); break;
    case 16: hipLaunchKernelGGL(k_cand_top<16>, dim3(a.blocks), dim3(kTopThreads), 0, st, a); break;
    case kTopMaxPer: hipLaunchKernelGGL(k_cand_top<kTopMaxPer>, dim3(a.blocks), dim3(kTopThreads), 0, st, a); break;
    default:
      hipLaunchKernelGGL(k_cand_zero, dim3(1), dim3(64), 0, st, a.count);
      hipLaunchKernelGGL(k_cand_compact, dim3((a.n_pix + 255) / 256), dim3(256), 0, st, a.best_snr, a.n_pix,
                         a.theta, a.keys, a.count);
      hipLaunchKernelGGL(k_cand_select, dim3(1), dim3(kSelThreads), 0, st, a.keys, a.count, a.k_max, a.nx,
                         a.best_d, a.best_w, a.best_t, (nsfrb_candidate*)a.out, a.n_out, a.flags);
  }
  return hipGetLastError();
}

hipError_t launch_candidates_batch(const CandDesc* descs, int n, int max_blocks, hipStream_t st) {
  hipLaunchKernelGGL(k_cand_top_batch, dim3(max_blocks, n), dim3(kTopThreads), 0, st, descs);
  return hipGetLastError();
}

}  // namespace nsfrb
