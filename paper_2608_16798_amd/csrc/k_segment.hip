// Policy-token compaction, rollout segmentation and group-relative advantages.
//
// Compaction keeps the positions t with M_t = 1 (Sec. 2.3.1: only valid policy-generated
// tokens are optimised) inside rollouts that are not excluded (Sec. 3.4: sandbox
// failures leave advantage estimation and policy optimisation), in ascending order.  Every
// later GEMM operand is gathered through this list, so masked tokens cost no MFMA work.
// Optionally (zero_grad: the caller's loss has no term but the advantage-weighted surrogate) the
// tokens of rollouts whose advantage is exactly 0 (an all-equal group, Sec. 2.3.2) go after all
// others, in their own ascending run: their surrogate gradient is exactly 0, so the backward
// covers only the first n_grad rows of the list while the forward covers all n_eff.
// The per-rollout count of kept tokens is the normaliser of the per-rollout token mean
// (masked GRPO objective, Sec. 2.3.2; shared-prefix tokens counted once, Sec. 3.2.3).
//
// Advantages follow the GRPO equation of Sec. 2.3.2 / Sec. 3.2.3: mean and population
// std over the non-excluded rollouts of a group (a task-harness pair, Sec. 3.3), with
// group keys treated as opaque and unordered.  All reductions run in a fixed order, in
// fp64, so results are bitwise reproducible.
#include "rlk_internal.h"

namespace rlk {

namespace {

constexpr int kThreads = 256;
constexpr int kPerThread = kScanTile / kThreads;  // 4 tokens per thread

__device__ inline int rollout_of(const int32_t* cu, int R, int64_t t) {
  // first r with cu[r+1] > t, clamped to [0, R-1]; tolerant of malformed cu
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if ((int64_t)cu[mid + 1] > t) hi = mid; else lo = mid + 1;
  }
  return lo;
}

__device__ inline int wave_inclusive_scan(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int n = __shfl_up(v, o, 64);
    if (lane >= o) v += n;
  }
  return v;
}

template <typename X>
__device__ inline X wave_sum(X v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Error bits of cu_seqlens, found by the whole workgroup (every thread gets them).
__device__ inline int check_cu(const int32_t* cu, int R, int64_t N) {
  __shared__ int err;
  if (threadIdx.x == 0) err = 0;
  __syncthreads();
  int e = 0;
  if (cu && R > 0) {
    for (int r = threadIdx.x; r < R; r += blockDim.x)
      if (cu[r] > cu[r + 1]) e |= RLK_DERR_CU_SEQLENS;
    if (threadIdx.x == 0 && (cu[0] != 0 || (int64_t)cu[R] != N)) e |= RLK_DERR_CU_SEQLENS;
  }
  if (e) atomicOr(&err, e);
  __syncthreads();
  return err;
}

__device__ inline void reset_header(WsHeader* hdr, int err, int n_groups, int n_valid) {
  hdr->status = err;
  hdr->n_eff = 0;
  hdr->n_grad = 0;
  hdr->n_groups = n_groups;
  hdr->n_valid = n_valid;
  hdr->ref_fallback = 0;
  hdr->n_dz_chunks = 0;
}

__global__ void __launch_bounds__(kThreads) k_begin(WsHeader* hdr, const int32_t* cu, int R, int64_t N) {
  const int err = check_cu(cu, R, N);
  if (threadIdx.x == 0) reset_header(hdr, err, 0, 0);
}

__device__ inline bool keep_token(const uint8_t* mask, const int32_t* gid, int r, int64_t t) {
  bool k = mask ? (mask[t] != 0) : true;
  if (gid) k = k && (gid[r] >= 0);
  return k;
}

// keep[t]: 0 = not trained, 1 = trained, 2 = trained with an exactly zero surrogate gradient (its
// rollout's advantage is 0 and zero_adv is given).  blkcnt[b] counts the 1s of block b and
// blkcnt[nblk + b] its 2s, so one exclusive scan over both halves places every 2 after every 1.
// begin: block 0 also resets the header and checks cu.
__global__ void __launch_bounds__(kThreads)
k_count(const uint8_t* mask, const int32_t* cu, const int32_t* gid, const float* zero_adv, int R, int64_t N,
        uint8_t* keep, int32_t* blkcnt, int nblk, WsHeader* hdr, int begin) {
  __shared__ int partial[2][kThreads / 64];
  if (begin && blockIdx.x == 0) {
    const int err = check_cu(cu, R, N);
    if (threadIdx.x == 0) reset_header(hdr, err, 0, 0);
  }
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPerThread;
  int cnt1 = 0, cnt2 = 0;
  if (t0 < N) {
    int r = rollout_of(cu, R, t0);
    uint32_t kp = 0;
    for (int i = 0; i < kPerThread; ++i) {
      int64_t t = t0 + i;
      if (t >= N) break;
      while (r < R - 1 && (int64_t)cu[r + 1] <= t) ++r;
      const bool k = keep_token(mask, gid, r, t);
      const bool zg = k && zero_adv && zero_adv[r] == 0.0f;
      kp |= (uint32_t)(!k ? 0 : (zg ? 2 : 1)) << (8 * i);
      cnt1 += (k && !zg) ? 1 : 0;
      cnt2 += zg ? 1 : 0;
    }
    reinterpret_cast<uint32_t*>(keep)[t0 / kPerThread] = kp;  // the workspace segment is padded to 256 bytes
  }
  cnt1 = wave_sum(cnt1);
  cnt2 = wave_sum(cnt2);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    partial[0][w] = cnt1;
    partial[1][w] = cnt2;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    int s = 0;
    for (int i = 0; i < kThreads / 64; ++i) s += partial[threadIdx.x][i];
    blkcnt[threadIdx.x * nblk + blockIdx.x] = s;
  }
}

// Exclusive scan of the per-block counts (both halves: nblk2 = 2 nblk); n_eff = the total, n_grad =
// the offset of the second half (the tokens with a gradient).  With a caller bound on the trained
// tokens (max_policy > 0) a larger total is flagged and both counts clamped to the bound, so every
// later kernel stays within the chunk loop the host sized for it.
__global__ void __launch_bounds__(1024) k_scan(const int32_t* blkcnt, int32_t* blkoff, int nblk2, int nblk,
                                               int32_t max_policy, WsHeader* hdr) {
  __shared__ int wsum[16];
  __shared__ int carry_s, ngrad_s;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int base = 0; base < nblk2; base += 1024) {
    int i = base + threadIdx.x;
    int v = i < nblk2 ? blkcnt[i] : 0;
    int inc = wave_inclusive_scan(v, lane);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int woff = 0;
    for (int j = 0; j < w; ++j) woff += wsum[j];
    int carry = carry_s;
    if (i < nblk2) blkoff[i] = carry + woff + inc - v;
    if (i == nblk) ngrad_s = carry + woff + inc - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry_s = carry + woff + inc;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    int n = carry_s, g = ngrad_s;
    if (max_policy > 0 && n > max_policy) {
      atomicOr(&hdr->status, RLK_DERR_POLICY_BOUND);
      n = max_policy;
      g = g < n ? g : n;
    }
    hdr->n_eff = n;
    hdr->n_grad = g;
  }
}

// Sum of a[0 .. n) by the calling wavefront.
__device__ inline int wave_sum_of(const int32_t* a, int n, int lane) {
  int s = 0;
  for (int i = lane; i < n; i += 64) s += a[i];
  return wave_sum(s);
}

// Blocks [0, nblk): the gather lists of the block's tokens.  The blocks after them: the rollouts' runs,
// one wavefront each (the rollout's tokens form one ascending run inside its part of the list, [0, n_grad)
// or, for a rollout of zero advantage, [n_grad, n_eff); its start is the number of earlier tokens of
// that part, from the block counts and the keep flags of one block).
//   blkoff: the scanned counts; NULL when the blocks add the counts up themselves (nblk at most
// kOwnScanBlocks, so sixteen loads per lane and part), which saves the launch of k_scan.  Launch bound: at
// 2,048 tokens count, scan, write and offsets (16 tokens per thread) took 9.8 + 4.4 + 14.4 + 5.1 us, the
// two launches now 4.6 + 6.0 us.
constexpr int kOwnScanBlocks = 1024;
__global__ void __launch_bounds__(kThreads)
k_write_idx(const uint8_t* keep, const int32_t* cu, int R, int64_t N, const int32_t* blkcnt, const int32_t* blkoff,
            int nblk, int32_t max_policy, const float* zero_adv, const int32_t* targets, int V, int32_t* idx,
            int32_t* tokr, int32_t* ytgt, float* zy, int32_t* rstart, int32_t* rnpol, WsHeader* hdr) {
  __shared__ int wsum[2][kThreads / 64];
  __shared__ int sum_s[kThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const bool lists = (int)blockIdx.x < nblk;
  // tokens of the first part, and of both (clamped to the caller's bound)
  int total1, total;
  if (blkoff) {
    total1 = hdr->n_grad;
    total = hdr->n_eff;
  } else {
    // wavefronts 0, 1: the parts' totals; 2, 3: what lies before this block
    const int n = w < 2 ? nblk : (lists ? (int)blockIdx.x : 0);
    const int v = wave_sum_of(blkcnt + (w & 1) * nblk, n, lane);
    if (lane == 0) sum_s[w] = v;
    __syncthreads();
    total1 = sum_s[0];
    total = sum_s[0] + sum_s[1];
    const bool over = max_policy > 0 && total > max_policy;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (over) atomicOr(&hdr->status, RLK_DERR_POLICY_BOUND);
      hdr->n_eff = over ? max_policy : total;
      hdr->n_grad = over && total1 > max_policy ? max_policy : total1;
    }
  }
  if (!lists) {
    const int r = ((int)blockIdx.x - nblk) * (kThreads / 64) + w;
    if (r >= R) return;
    const bool second = zero_adv && zero_adv[r] == 0.0f;
    const int want = second ? 2 : 1;
    int at[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      int64_t t = cu[r + e];
      t = t < 0 ? 0 : (t > N ? N : t);
      const int b = (int)(t / kScanTile);
      int c;
      if (blkoff) c = b < nblk ? blkoff[(second ? nblk : 0) + b] - (second ? total1 : 0) : 0;
      else c = wave_sum_of(blkcnt + (second ? nblk : 0), b, lane);
      if (blkoff && b >= nblk) c = (second ? total - total1 : total1);
      int in = 0;
      for (int64_t u = (int64_t)b * kScanTile + lane; u < t; u += 64) in += keep[u] == want;
      at[e] = c + wave_sum(in);
    }
    if (lane == 0) {
      int n1 = total1, n = total;
      if (max_policy > 0 && n > max_policy) {
        n = max_policy;
        n1 = min(n1, n);
      }
      const int lo = second ? n1 : 0, most = second ? n - n1 : n1;
      const int s = min(at[0], most), e = max(min(at[1], most), s);
      rstart[r] = lo + s;
      rnpol[r] = e - s;
    }
    return;
  }
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPerThread;
  const uint32_t kp = t0 < N ? reinterpret_cast<const uint32_t*>(keep)[t0 / kPerThread] : 0u;
  const int cnt1 = __popc(kp & 0x01010101u), cnt2 = __popc(kp & 0x02020202u);
  const int inc1 = wave_inclusive_scan(cnt1, lane), inc2 = wave_inclusive_scan(cnt2, lane);
  if (lane == 63) {
    wsum[0][w] = inc1;
    wsum[1][w] = inc2;
  }
  __syncthreads();
  int off1 = blkoff ? blkoff[blockIdx.x] : sum_s[2], off2 = blkoff ? blkoff[nblk + blockIdx.x] : total1 + sum_s[3];
  for (int j = 0; j < w; ++j) {
    off1 += wsum[0][j];
    off2 += wsum[1][j];
  }
  off1 += inc1 - cnt1;
  off2 += inc2 - cnt2;
  if (kp == 0) return;
  int r = rollout_of(cu, R, t0);
  int bad = 0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int64_t t = t0 + i;
    const uint32_t k = (kp >> (8 * i)) & 0xffu;
    if (k) {
      while (r < R - 1 && (int64_t)cu[r + 1] <= t) ++r;
      const int y = targets ? targets[t] : 0;
      if (y < 0 || y >= V) bad = 1;
      const int off = k == 1 ? off1++ : off2++;
      idx[off] = (int32_t)t;
      tokr[off] = r;
      ytgt[off] = y;
      zy[off] = 0.0f;
    }
  }
  if (bad) atomicOr(&hdr->status, RLK_DERR_TARGET);
}

// ---- group-relative advantages ----
//
// Segmentation by sorting: the (key, rollout) pairs of the non-excluded rollouts are sorted, so each
// group becomes a run of consecutive entries with its members in ascending rollout order; a scan over the
// run starts gives the dense group index (the rank of the key among the sorted distinct keys).  The
// statistics are a segmented reduction, one wavefront per run.
//   Up to kSortRun rollouts everything is one workgroup and one launch, which also resets the header: an
// entry per thread, sorted by shuffles (strides below 64) and LDS.  Beyond, one workgroup per run of
// kSortRun entries sorts it, every entry finds its rank in the other runs by binary search, one workgroup
// per run counts the group starts before it, and the groups' wavefronts spread over the GPU.  16,384 rollouts:
// 268 us with one workgroup sorting them all by a bitonic network in LDS, 32 us now (10 + 8 + 9 + 4).

constexpr int kSortRun = 1024;
static_assert(kMaxRollouts % kSortRun == 0, "whole runs");
constexpr int kMaxRuns = kMaxRollouts / kSortRun;

// entry = (key' << 32) | rollout with key' = key for a kept rollout and 0xFFFFFFFF for an excluded one
// (and for the padding), so kept rollouts sort first, by key, then by rollout.
__device__ inline uint64_t sort_entry(const int32_t* gid, int R, int i) {
  if (i >= R) return ~0ull;
  const int32_t key = gid[i];
  const uint32_t hi = key >= 0 ? (uint32_t)key : 0xFFFFFFFFu;
  return ((uint64_t)hi << 32) | (uint32_t)i;
}
__device__ inline bool kept_entry(uint64_t v) { return (v >> 32) != 0xFFFFFFFFull; }

// Bitonic sort of the first P (a power of two) threads' entries, ascending by thread.
__device__ inline uint64_t sort_run(uint64_t v, int P, uint64_t (&e)[kSortRun]) {
  const int i = threadIdx.x;
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      uint64_t o;
      if (j >= 64) {
        e[i] = v;
        __syncthreads();
        o = e[i ^ j];
        __syncthreads();
      } else {
        o = __shfl_xor((unsigned long long)v, j, 64);
      }
      const bool low = ((i & j) == 0) == ((i & k) == 0);
      v = (v < o) == low ? v : o;
    }
  }
  return v;
}

// Statistics and advantages of one group by L lanes (a power of two; sub = the lane among them), members
// (ascending rollout order) from member(i): lanes stride the run, partial sums combined by a fixed shuffle
// tree: mean and population std in fp64; exactly 0 where every reward of the group is bitwise equal.  Every
// lane of the wavefront calls it (n = 0: no group).
template <typename F>
__device__ inline void group_advantage(int n, int sub, int L, F member, const float* rewards, float adv_eps,
                                       int32_t* gsize, float* adv) {
  double sum = 0.0;
  float mn = INFINITY, mx = -INFINITY;
  for (int i = sub; i < n; i += L) {
    const float v = rewards[member(i)];
    sum += (double)v;
    mn = fminf(mn, v);
    mx = fmaxf(mx, v);
  }
  for (int o = L >> 1; o > 0; o >>= 1) {
    sum += __shfl_xor(sum, o, 64);
    mn = fminf(mn, __shfl_xor(mn, o, 64));
    mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  }
  const double mu = n > 0 ? sum / (double)n : 0.0;
  double ss = 0.0;
  for (int i = sub; i < n; i += L) {
    const double dv = (double)rewards[member(i)] - mu;
    ss += dv * dv;
  }
  for (int o = L >> 1; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  const double sig = n > 0 ? sqrt(ss / (double)n) : 0.0;
  if (sub == 0 && n > 0) *gsize = n;
  for (int i = sub; i < n; i += L) {
    const int r = member(i);
    adv[r] = mn == mx ? 0.0f : (float)(((double)rewards[r] - mu) / (sig + (double)adv_eps));
  }
}

// Exclusive scan over the workgroup's threads of a count; total = the sum.
__device__ inline int block_exclusive(int v, int& total) {
  __shared__ int wsum[kSortRun / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int inc = wave_inclusive_scan(v, lane);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int off = 0;
  total = 0;
#pragma unroll
  for (int j = 0; j < kSortRun / 64; ++j) {
    if (j < w) off += wsum[j];
    total += wsum[j];
  }
  __syncthreads();
  return off + inc - v;
}

__global__ void __launch_bounds__(kSortRun)
k_advantage_one(const float* rewards, const int32_t* gid, int R, float adv_eps, int32_t* members, int32_t* gstart,
                int32_t* gidx, int32_t* gsize, float* adv, int32_t* n_groups_out, WsHeader* hdr, const int32_t* cu,
                int64_t N) {
  __shared__ uint64_t e[kSortRun];
  __shared__ float rw[kSortRun];
  __shared__ int start_s[kSortRun + 1];
  __shared__ int large[kSortRun / 65 + 1], n_large;
  const int i = threadIdx.x;
  if (i == 0) n_large = 0;  // barriers lie before its use
  const int err = check_cu(cu, R, N);
  int P = 64;
  while (P < R) P <<= 1;
  if (i < R) rw[i] = rewards[i];
  const uint64_t v = sort_run(sort_entry(gid, R, i), P, e);
  e[i] = v;
  __syncthreads();
  const bool kept = kept_entry(v);
  const bool first = kept && (i == 0 || (e[i - 1] >> 32) != (v >> 32));
  int Q, nv;
  const int q = block_exclusive(first ? 1 : 0, Q) + (first ? 1 : 0) - 1;  // dense index of the entry's group
  block_exclusive(kept ? 1 : 0, nv);
  const int r = (int)(uint32_t)v;
  if (kept) {
    members[i] = r;
    gidx[r] = q;
    if (first) {
      gstart[q] = i;
      start_s[q] = i;
    }
  } else if (i < R) {  // the excluded rollouts follow the kept ones, before the padding
    gidx[r] = -1;
    adv[r] = 0.0f;
  }
  if (i == 0) {
    gstart[Q] = nv;
    start_s[Q] = nv;
    reset_header(hdr, err, Q, nv);
    if (n_groups_out) *n_groups_out = Q;
  }
  __syncthreads();
  // A wavefront takes 1.6 us per group, so groups of up to 64 rollouts share them, the workgroup's threads dealt
  // over the groups, and each larger one (at most 15) has a wavefront of its own.  1,024 rollouts in as many
  // groups: 126 us with a wavefront for every group, 17 us now; 128 groups of 8: 27 and 14 us.
  if (i < Q && start_s[i + 1] - start_s[i] > 64) large[atomicAdd(&n_large, 1)] = i;
  __syncthreads();
  auto group = [&](int g, int sub, int L) {
    const int b = g >= 0 ? start_s[g] : 0;
    group_advantage(g >= 0 ? start_s[g + 1] - b : 0, sub, L, [&](int k) { return (int)(uint32_t)e[b + k]; }, rw, adv_eps,
                    gsize + max(g, 0), adv);
  };
  if ((i >> 6) < n_large) group(large[i >> 6], i & 63, 64);
  int L = 64;
  while (L > 4 && Q * L > kSortRun) L >>= 1;
  for (int g0 = 0; g0 < Q; g0 += kSortRun / L) {
    const int g = g0 + i / L;
    group(g < Q && start_s[g + 1] - start_s[g] <= 64 ? g : -1, i % L, L);
  }
}

// runs of kSortRun entries, sorted (excluded rollouts get their index and advantage here); block 0
// resets the header
__global__ void __launch_bounds__(kSortRun)
k_sort_runs(const int32_t* gid, int R, uint64_t* runs, int32_t* gidx, float* adv, WsHeader* hdr, const int32_t* cu,
            int64_t N) {
  __shared__ uint64_t e[kSortRun];
  if (blockIdx.x == 0) {
    const int err = check_cu(cu, R, N);
    if (threadIdx.x == 0) reset_header(hdr, err, 0, 0);
  }
  const int i = blockIdx.x * kSortRun + threadIdx.x;
  const uint64_t own = sort_entry(gid, R, i);
  if (i < R && !kept_entry(own)) {
    gidx[i] = -1;
    adv[i] = 0.0f;
  }
  const uint64_t v = sort_run(own, kSortRun, e);
  if (i < R) runs[i] = v;
}

// rank of every entry among all runs (entries are distinct): the number of smaller entries of each run, by
// binary searches side by side
__global__ void __launch_bounds__(64) k_merge_runs(const uint64_t* runs, int R, uint64_t* sorted) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= R) return;
  const uint64_t v = runs[i];
  int pos[kMaxRuns];
#pragma unroll
  for (int b = 0; b < kMaxRuns; ++b) pos[b] = 0;
  for (int step = kSortRun; step > 0; step >>= 1) {
    uint64_t x[kMaxRuns];
#pragma unroll
    for (int b = 0; b < kMaxRuns; ++b)  // clamped, so that all loads go out together
      x[b] = runs[min(b * kSortRun + min(pos[b] + step, kSortRun) - 1, R - 1)];
#pragma unroll
    for (int b = 0; b < kMaxRuns; ++b)
      if (pos[b] + step <= min(kSortRun, R - b * kSortRun) && x[b] < v) pos[b] += step;
  }
  int rank = 0;
#pragma unroll
  for (int b = 0; b < kMaxRuns; ++b) rank += pos[b];
  sorted[rank] = v;
}

// whether sorted entry i starts a group
__device__ inline bool starts_group(const uint64_t* sorted, int i, int R, uint64_t& v) {
  v = i < R ? sorted[i] : ~0ull;
  const uint64_t before = i > 0 && i < R ? sorted[i - 1] : ~0ull;
  return kept_entry(v) && (i == 0 || (before >> 32) != (v >> 32));
}

// group starts and dense indices of the sorted entries, one per thread; a workgroup counts the starts
// before its entries itself (at most fifteen more loads per thread)
__global__ void __launch_bounds__(kSortRun)
k_group_index(const uint64_t* sorted, int R, int32_t* members, int32_t* gstart, int32_t* gidx, int32_t* n_groups_out,
              WsHeader* hdr) {
  const int i = blockIdx.x * kSortRun + threadIdx.x;
  int before = 0;
  uint64_t v;
#pragma unroll 4
  for (int b = 0; b < (int)blockIdx.x; ++b) before += starts_group(sorted, b * kSortRun + threadIdx.x, R, v);
  const bool first = starts_group(sorted, i, R, v);
  int base, Q, nv;
  block_exclusive(before, base);
  const int q = base + block_exclusive(first ? 1 : 0, Q) + (first ? 1 : 0) - 1;
  block_exclusive(kept_entry(v) ? 1 : 0, nv);
  if (kept_entry(v)) {
    const int r = (int)(uint32_t)v;
    members[i] = r;
    gidx[r] = q;
    if (first) gstart[q] = i;
  }
  // kept entries come first: the workgroup that holds the last of them (or, without any, the first) ends
  // the runs
  const int next = (blockIdx.x + 1) * kSortRun;
  const bool none_after = nv < kSortRun || next >= R || !kept_entry(sorted[next]);
  if (threadIdx.x == 0 && none_after && (nv > 0 || blockIdx.x == 0)) {
    gstart[base + Q] = i + nv;
    hdr->n_groups = base + Q;
    hdr->n_valid = i + nv;
    if (n_groups_out) *n_groups_out = base + Q;
  }
}

__global__ void __launch_bounds__(kThreads)
k_group_advantage(const float* rewards, const int32_t* members, const int32_t* gstart, float adv_eps,
                  const WsHeader* hdr, int32_t* gsize, float* adv) {
  const int lane = threadIdx.x & 63;
  const int q = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (q >= hdr->n_groups) return;
  const int b = gstart[q];
  group_advantage(gstart[q + 1] - b, lane, 64, [&](int k) { return members[b + k]; }, rewards, adv_eps, gsize + q,
                  adv);
}

inline dim3 blocks_for(int64_t n, int per) { return dim3((unsigned)((n + per - 1) / per)); }

}  // namespace

hipError_t launch_begin(int32_t* status_hdr, const int32_t* cu, int R, int64_t N, hipStream_t s) {
  prof_mark(KK_BEGIN, true, s);
  k_begin<<<1, kThreads, 0, s>>>(reinterpret_cast<WsHeader*>(status_hdr), cu, R, N);
  prof_mark(KK_BEGIN, false, s);
  return hipGetLastError();
}

hipError_t launch_compact(const uint8_t* mask, const int32_t* cu, const int32_t* gid, int R, int64_t N,
                          const int32_t* targets, int V, int32_t max_policy, const float* zero_adv, bool begin, char* ws,
                          const WsLayout& L, hipStream_t s) {
  WsHeader* hdr = reinterpret_cast<WsHeader*>(ws + L.hdr);
  uint8_t* keep = reinterpret_cast<uint8_t*>(ws + L.keep);
  int32_t* blkcnt = reinterpret_cast<int32_t*>(ws + L.blkcnt);
  int32_t* blkoff = reinterpret_cast<int32_t*>(ws + L.blkoff);
  if (N == 0 && begin) {
    hipError_t e = launch_begin(reinterpret_cast<int32_t*>(hdr), cu, R, N, s);
    if (e != hipSuccess) return e;
  }
  const int nblk = N > 0 ? L.nblk : 0;
  if (nblk > 0) {
    prof_mark(KK_COUNT, true, s);
    k_count<<<nblk, kThreads, 0, s>>>(mask, cu, gid, zero_adv, R, N, keep, blkcnt, nblk, hdr, begin ? 1 : 0);
    prof_mark(KK_COUNT, false, s);
  }
  const bool own_scan = nblk <= kOwnScanBlocks;
  if (!own_scan) {
    prof_mark(KK_SCAN, true, s);
    k_scan<<<1, 1024, 0, s>>>(blkcnt, blkoff, 2 * nblk, nblk, max_policy, hdr);
    prof_mark(KK_SCAN, false, s);
  }
  const int grid = nblk + (R + kThreads / 64 - 1) / (kThreads / 64);
  if (grid > 0) {
    prof_mark(KK_WRITE_IDX, true, s);
    k_write_idx<<<grid, kThreads, 0, s>>>(
        keep, cu, R, N, blkcnt, own_scan ? nullptr : blkoff, nblk, max_policy, zero_adv, targets, V,
        reinterpret_cast<int32_t*>(ws + L.idx), reinterpret_cast<int32_t*>(ws + L.tokr),
        reinterpret_cast<int32_t*>(ws + L.ytgt), reinterpret_cast<float*>(ws + L.zy),
        reinterpret_cast<int32_t*>(ws + L.rstart), reinterpret_cast<int32_t*>(ws + L.rnpol), hdr);
    prof_mark(KK_WRITE_IDX, false, s);
  }
  return hipGetLastError();
}

hipError_t launch_begin_advantage(int R, const float* rewards, const int32_t* gid, float adv_eps, int32_t* members,
                                  int32_t* gstart, int32_t* gidx, int32_t* gsize, uint64_t* sort_a, uint64_t* sort_b,
                                  float* adv, int32_t* n_groups_out, WsHeader* hdr, const int32_t* cu, int64_t N,
                                  hipStream_t s) {
  if (R > kMaxRollouts) return hipErrorInvalidValue;
  prof_mark(KK_GROUP_RANK, true, s);
  uint64_t *runs = sort_a, *sorted = sort_b;
  if (R <= kSortRun) {
    k_advantage_one<<<1, kSortRun, 0, s>>>(rewards, gid, R, adv_eps, members, gstart, gidx, gsize, adv, n_groups_out,
                                           hdr, cu, N);
  } else {
    k_sort_runs<<<(R + kSortRun - 1) / kSortRun, kSortRun, 0, s>>>(gid, R, runs, gidx, adv, hdr, cu, N);
    k_merge_runs<<<(R + 63) / 64, 64, 0, s>>>(runs, R, sorted);
    k_group_index<<<(R + kSortRun - 1) / kSortRun, kSortRun, 0, s>>>(sorted, R, members, gstart, gidx, n_groups_out, hdr);
  }
  prof_mark(KK_GROUP_RANK, false, s);
  if (R > kSortRun) {
    prof_mark(KK_ADVANTAGE, true, s);
    k_group_advantage<<<blocks_for(R, kThreads / 64), kThreads, 0, s>>>(rewards, members, gstart, adv_eps, hdr, gsize,
                                                                        adv);
    prof_mark(KK_ADVANTAGE, false, s);
  }
  return hipGetLastError();
}

}  // namespace rlk
