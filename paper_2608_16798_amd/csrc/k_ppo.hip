// PPO path kernels (ClawGym II, Sec. 2.3.1 GAE and value loss; Sec. 3.2.3 simplified variant):
// masked generalised advantage estimation as a per-rollout reverse scan, and the masked
// mean-squared value loss with its gradient.
//
// GAE over a rollout's policy rows t_1 < ... < t_n (tool rows are stepped over):
//   delta_j = gamma V[t_{j+1}] - V[t_j]  (j < n),   delta_n = R - V[t_n],
//   A_j = delta_j + c A_{j+1}, c = gamma lambda,  returns = A + V.
// One workgroup per rollout walks the rollout backwards, kGaeRows consecutive rows per thread and
// pass.  Thread i holds the i-th group of rows from the end, so increasing thread order is decreasing
// row order and both quantities are exclusive scans over threads, carried from pass to pass:
//   - the value of the nearest later policy row (a "latest seen" scan), which gives delta;
//   - A as the composition of the affine maps x -> (policy ? c x + delta : x).
// Inside a wavefront the first is one ballot and one lane read, the second a shuffle scan; the
// wavefronts meet in LDS.
#include "rlk_internal.h"

#include <algorithm>

namespace rlk {

namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

constexpr int kGaeRows = 8;    // consecutive rows per thread

__device__ __forceinline__ int64_t clamp64(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Rows [g, g + 8), g a multiple of 8, of the rollout's [s0, s1): bit k of the result is set where row
// g + k belongs to it and its mask is set; v gets the values of those rows.  VEC: the array bases are
// 16-byte aligned, so a group inside the arrays is read in three loads.
template <bool VEC>
__device__ __forceinline__ uint32_t load_rows(int64_t g, int64_t s0, int64_t s1, int64_t N, const uint8_t* mask,
                                              const float* values, float (&v)[kGaeRows]) {
  uint32_t pol = 0;
  if (g + kGaeRows <= s0 || g >= s1) return 0;
  if (VEC && g + kGaeRows <= N) {
    const u32x2 m = *reinterpret_cast<const u32x2*>(mask + g);
    const f32x4 a = *reinterpret_cast<const f32x4*>(values + g), b = *reinterpret_cast<const f32x4*>(values + g + 4);
#pragma unroll
    for (int k = 0; k < kGaeRows; ++k) {
      v[k] = k < 4 ? a[k & 3] : b[k & 3];
      if (((m[k >> 2] >> (8 * (k & 3))) & 0xffu) != 0 && g + k >= s0 && g + k < s1) pol |= 1u << k;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kGaeRows; ++k) {
      v[k] = 0.0f;
      if (g + k >= s0 && g + k < s1 && mask[g + k] != 0) {
        v[k] = values[g + k];
        pol |= 1u << k;
      }
    }
  }
  return pol;
}

// the group's rows of [s0, s1) of an output
template <bool VEC>
__device__ __forceinline__ void store_rows(int64_t g, int64_t s0, int64_t s1, float* out, const float (&o)[kGaeRows]) {
  if (VEC && g >= s0 && g + kGaeRows <= s1) {
    *reinterpret_cast<f32x4*>(out + g) = f32x4{o[0], o[1], o[2], o[3]};
    *reinterpret_cast<f32x4*>(out + g + 4) = f32x4{o[4], o[5], o[6], o[7]};
  } else {
#pragma unroll
    for (int k = 0; k < kGaeRows; ++k)
      if (g + k >= s0 && g + k < s1) out[g + k] = o[k];
  }
}

// Latency bound: 26 bytes per row move, and a rollout is one workgroup.  A pass takes 8 rows per
// thread and two barriers; rollouts of up to 8 x THREADS rows take one pass.  128 rollouts of 1,024 to
// 7,168 rows: 69 us with one row per thread, 256 rows a pass and LDS scans -> 10.4 us.
template <bool VEC, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_gae(int64_t N, const int32_t* cu, const uint8_t* mask, const float* values, const float* rewards,
      const int32_t* gid, float gamma, float lam, float* adv, float* ret) {
  constexpr int NW = THREADS / 64;
  __shared__ int s_has[2][NW];
  __shared__ double s_val[2][NW], s_a[2][NW], s_b[2][NW];
  const int r = blockIdx.x;
  const int i = threadIdx.x, lane = i & 63, w = i >> 6;
  const int64_t s0 = clamp64(cu[r], 0, N), s1 = clamp64(cu[r + 1], s0, N);
  const bool excluded = gid && gid[r] < 0;
  const double c = (double)gamma * (double)lam, gam = (double)gamma;
  const double R = (double)rewards[r];
  bool carry_has = false;   // a policy row exists after the current pass
  double carry_val = 0.0;   // its value
  double carry_A = 0.0;     // advantage of the nearest policy row at or after the pass's end
  int par = 0;
  for (int64_t e = (s1 + kGaeRows - 1) / kGaeRows * kGaeRows; e > s0; e -= (int64_t)kGaeRows * THREADS, par ^= 1) {
    const int64_t g = e - (int64_t)(i + 1) * kGaeRows;
    float v[kGaeRows];
#pragma unroll
    for (int k = 0; k < kGaeRows; ++k) v[k] = 0.0f;
    uint32_t pol = g >= 0 ? load_rows<VEC>(g, s0, s1, N, mask, values, v) : 0u;
    if (excluded) pol = 0;
    // (1) nearest later policy row: the earliest one of the nearest lower thread that has any
    double first = 0.0;
#pragma unroll
    for (int k = kGaeRows - 1; k >= 0; --k)
      if (pol >> k & 1) first = (double)v[k];
    const uint64_t have = __ballot(pol != 0);
    const uint64_t below = have & ((1ull << lane) - 1);
    const double near = __shfl(first, below ? 63 - __clzll((long long)below) : 0, 64);
    const double last = __shfl(first, have ? 63 - __clzll((long long)have) : 0, 64);
    if (lane == 0) {
      s_has[par][w] = have != 0;
      s_val[par][w] = last;
    }
    __syncthreads();
    bool nh = below != 0;
    double nv = near;
    if (!nh) {
      nh = carry_has;
      nv = carry_val;
      for (int x = 0; x < w; ++x)
        if (s_has[par][x]) {
          nh = true;
          nv = s_val[par][x];
        }
    }
    for (int x = 0; x < NW; ++x)
      if (s_has[par][x]) {
        carry_has = true;
        carry_val = s_val[par][x];
      }
    // (2) A: the thread's map x -> a x + b over its rows, latest row first, then the scan over threads
    const double next0 = nh ? gam * nv : R;  // gamma V of the next policy row, or the reward
    double next = next0, a = 1.0, b = 0.0;
#pragma unroll
    for (int k = kGaeRows - 1; k >= 0; --k) {
      if (pol >> k & 1) {
        b = c * b + (next - (double)v[k]);
        a = c * a;
        next = gam * (double)v[k];
      }
    }
    for (int off = 1; off < 64; off <<= 1) {
      const double pa = __shfl_up(a, off, 64), pb = __shfl_up(b, off, 64);
      if (lane >= off) {
        b = a * pb + b;  // this map after the earlier one: x -> a (pa x + pb) + b
        a = a * pa;
      }
    }
    if (lane == 63) {
      s_a[par][w] = a;
      s_b[par][w] = b;
    }
    __syncthreads();
    double A = carry_A;  // advantage entering the wavefront, then the thread
    for (int x = 0; x < w; ++x) A = s_a[par][x] * A + s_b[par][x];
    for (int x = 0; x < NW; ++x) carry_A = s_a[par][x] * carry_A + s_b[par][x];
    const double ea = __shfl_up(a, 1, 64), eb = __shfl_up(b, 1, 64);
    if (lane > 0) A = ea * A + eb;
    if (g < 0 || g + kGaeRows <= s0) continue;  // no rows of this rollout (the barriers are behind)
    float oa[kGaeRows], orr[kGaeRows];
    next = next0;
#pragma unroll
    for (int k = kGaeRows - 1; k >= 0; --k) {
      const bool p = pol >> k & 1;
      if (p) {
        A = c * A + (next - (double)v[k]);
        next = gam * (double)v[k];
      }
      oa[k] = p ? (float)A : 0.0f;
      orr[k] = p ? (float)(A + (double)v[k]) : 0.0f;
    }
    store_rows<VEC>(g, s0, s1, adv, oa);
    if (ret) store_rows<VEC>(g, s0, s1, ret, orr);
  }
}

// ---- value loss: fp64 partial sums of (rollout, slice of its rows), their total, then the gradient.
// A rollout's rows are cut into groups of 8 x THREADS rows, dealt to kValueSplit slices, so that a batch of
// few long rollouts still fills the GPU.  128 rollouts of 1,024 to 7,168 rows: three launches of one
// row per thread 22.7 us -> two launches 9.8 us.
template <bool VEC, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_value_partial(int64_t N, const int32_t* cu, const uint8_t* mask, const float* values, const float* ret,
                const int32_t* gid, double* part) {
  __shared__ double sh[THREADS / 64][2];
  const int r = blockIdx.x;
  const int64_t s0 = clamp64(cu[r], 0, N), s1 = clamp64(cu[r + 1], s0, N);
  double ss = 0.0, cnt = 0.0;
  if (!(gid && gid[r] < 0)) {
    for (int64_t g = s0 / kGaeRows * kGaeRows + ((int64_t)blockIdx.y * THREADS + threadIdx.x) * kGaeRows;
         g < s1; g += (int64_t)gridDim.y * THREADS * kGaeRows) {
      float v[kGaeRows], t[kGaeRows];
      const uint32_t pol = load_rows<VEC>(g, s0, s1, N, mask, values, v);
      load_rows<VEC>(g, s0, s1, N, mask, ret, t);
#pragma unroll
      for (int k = 0; k < kGaeRows; ++k)
        if (pol >> k & 1) {
          const double d = (double)v[k] - (double)t[k];
          ss += d * d;
          cnt += 1.0;
        }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    ss += __shfl_xor(ss, o, 64);
    cnt += __shfl_xor(cnt, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[threadIdx.x >> 6][0] = ss;
    sh[threadIdx.x >> 6][1] = cnt;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
    for (int k = 0; k < THREADS / 64; ++k) t += sh[k][threadIdx.x];
    part[((int64_t)r * gridDim.y + blockIdx.y) * 2 + threadIdx.x] = t;
  }
}

// total of n partials in a fixed order (the same in every block that forms it)
template <int THREADS>
__device__ __forceinline__ void value_total(int n, const double* part, double& sum, double& count) {
  __shared__ double sh[THREADS / 64][2];
  double ss = 0.0, cnt = 0.0;
  for (int r = threadIdx.x; r < n; r += THREADS) {
    ss += part[(int64_t)r * 2];
    cnt += part[(int64_t)r * 2 + 1];
  }
  for (int o = 32; o > 0; o >>= 1) {
    ss += __shfl_xor(ss, o, 64);
    cnt += __shfl_xor(cnt, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[threadIdx.x >> 6][0] = ss;
    sh[threadIdx.x >> 6][1] = cnt;
  }
  __syncthreads();
  sum = 0.0;
  count = 0.0;
  for (int k = 0; k < THREADS / 64; ++k) {
    sum += sh[k][0];
    count += sh[k][1];
  }
}

__global__ void __launch_bounds__(1024) k_value_final(int n, const double* part, double* total, float* loss) {
  double a, cnt;
  value_total<1024>(n, part, a, cnt);
  if (threadIdx.x == 0) {
    total[0] = cnt;
    loss[0] = cnt > 0 ? (float)(a / cnt) : 0.0f;
  }
}

// With npart > 0 every block adds up the partials itself (and block 0 writes the loss), which saves the
// launch of k_value_final; otherwise the count is in total.
template <bool VEC, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_value_grad(int64_t N, const int32_t* cu, const uint8_t* mask, const float* values, const float* ret,
             const int32_t* gid, int npart, const double* part, const double* total, float* loss, float* dv) {
  const int r = blockIdx.x;
  double n;
  if (npart > 0) {
    double sum;
    value_total<THREADS>(npart, part, sum, n);
    if (r == 0 && blockIdx.y == 0 && threadIdx.x == 0) loss[0] = n > 0 ? (float)(sum / n) : 0.0f;
  } else {
    n = total[0];
  }
  const int64_t s0 = clamp64(cu[r], 0, N), s1 = clamp64(cu[r + 1], s0, N);
  const bool on = !(gid && gid[r] < 0) && n > 0;
  for (int64_t g = s0 / kGaeRows * kGaeRows + ((int64_t)blockIdx.y * THREADS + threadIdx.x) * kGaeRows;
       g < s1; g += (int64_t)gridDim.y * THREADS * kGaeRows) {
    float v[kGaeRows], t[kGaeRows], o[kGaeRows];
    const uint32_t pol = load_rows<VEC>(g, s0, s1, N, mask, values, v);
    load_rows<VEC>(g, s0, s1, N, mask, ret, t);
#pragma unroll
    for (int k = 0; k < kGaeRows; ++k)
      o[k] = on && (pol >> k & 1) ? (float)(2.0 * ((double)v[k] - (double)t[k]) / n) : 0.0f;
    store_rows<VEC>(g, s0, s1, dv, o);
  }
}

// ---- linear value head V_t = w . h_t + b on the kept rows (mask = 1, rollout not excluded) and
// its backward.  Reductions run in a fixed order (wavefront trees, block partials in row order),
// so results are bitwise reproducible.
__device__ __forceinline__ int rollout_of_row(const int32_t* cu, int R, int64_t t) {
  int lo = 0, hi = R - 1;  // first r with cu[r+1] > t, clamped to [0, R-1]
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)cu[mid + 1] > t) hi = mid; else lo = mid + 1;
  }
  return lo;
}

__device__ __forceinline__ bool kept_row(const uint8_t* mask, const int32_t* cu, const int32_t* gid, int R,
                                         int64_t t) {
  if (mask && !mask[t]) return false;
  return !gid || gid[rollout_of_row(cu, R, t)] >= 0;
}

template <typename T>
__device__ __forceinline__ void unpack8(const u32x4 v, float (&f)[16 / sizeof(T)]);
template <>
__device__ __forceinline__ void unpack8<bf16_t>(const u32x4 v, float (&f)[8]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
template <>
__device__ __forceinline__ void unpack8<float>(const u32x4 v, float (&f)[4]) {
  f[0] = __uint_as_float(v.x);
  f[1] = __uint_as_float(v.y);
  f[2] = __uint_as_float(v.z);
  f[3] = __uint_as_float(v.w);
}
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)hi) << 16);
}

constexpr int kHeadRows = 128;    // rows per workgroup of the backward

// The kept ones of the ROWS rows from t0 on, in row order, listed in LDS by the first ROWS threads (every
// thread of the workgroup calls it); returns their number, and in keep whether the thread's own row is one.
template <int ROWS>
__device__ __forceinline__ int list_kept(int64_t t0, int64_t N, const uint8_t* mask, const int32_t* cu,
                                         const int32_t* gid, int R, int16_t (&list)[ROWS], bool& keep) {
  static_assert(ROWS % 64 == 0, "whole ballots");
  __shared__ int count[ROWS / 64];
  const int i = threadIdx.x;
  keep = i < ROWS && t0 + i < N && kept_row(mask, cu, gid, R, t0 + i);
  const uint64_t b = __ballot(keep);
  if (i < ROWS && (i & 63) == 0) count[i >> 6] = __popcll(b);
  __syncthreads();
  int off = 0, n = 0;
#pragma unroll
  for (int w = 0; w < ROWS / 64; ++w) {
    if (w < (i >> 6)) off += count[w];
    n += count[w];
  }
  if (keep) list[off + __popcll(b & ((1ull << (i & 63)) - 1))] = (int16_t)i;
  __syncthreads();
  return n;
}

// Forward: HBM bound (one read of the kept rows), one wavefront per row, BATCH 16-byte loads in flight per lane (8,
// or for rows of one load per lane 1: 300,000 rows of 64 bf16, all kept, 79 us with
// the batch, 75 us without):
// 131,072 rows of 4,096 bf16, 40 % kept, after a pass that writes 1 GB: 132 us without the batch, 122 us
// with it (3.5 TB/s).  Listing the kept rows of 32 first, so that no wavefront starts for the others, took 158 us.
template <typename T, int BATCH>
__global__ void __launch_bounds__(256)
k_value_head_fwd(int64_t N, int d, const T* h, const T* w, float b, const uint8_t* mask, const int32_t* cu,
                 const int32_t* gid, int R, float* values) {
  constexpr int EPC = 16 / sizeof(T);
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= N) return;
  if (!kept_row(mask, cu, gid, R, t)) {
    if (lane == 0) values[t] = 0.0f;
    return;
  }
  const T* row = h + t * d;
  const int nch = d / EPC;
  float acc = 0.0f;
  for (int cb = lane; cb < nch; cb += 64 * BATCH) {
    u32x4 x[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      x[u] = cb + 64 * u < nch ? *reinterpret_cast<const u32x4*>(row + (cb + 64 * u) * EPC) : u32x4{0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      if (cb + 64 * u >= nch) break;
      float f[EPC], y[EPC];
      unpack8<T>(x[u], f);
      unpack8<T>(*reinterpret_cast<const u32x4*>(w + (cb + 64 * u) * EPC), y);
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc = fmaf(f[e], y[e], acc);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) values[t] = acc + b;
}

// Backward, HBM bound (one read of the kept rows, one write of every dhidden row): both in one launch, so
// that the reads and the writes overlap.  The first 256 threads form the workgroup's partial sum
// part[blk][j] = sum_t dV_t h_t[j] over its rows (fp32, row order; the thread owns a 16-byte column
// chunk, and for a row of fewer than 256 chunks the threads deal the rows among themselves and add up
// in LDS); part_db[blk] = sum_t dV_t (fp64).  131,072 rows of 4,096 bf16, 40 % kept: three passes
// (dhidden, partial sums of 256 rows four at a time, totals) 615 us -> 320 us with the totals, 4.7 TB/s.
//   The other 256 (with dh) write the dhidden rows: kept rows get (dh +) dV_t w, the others are zeroed unless
// accumulating.  Apart, a read's wait does not include the writes issued before it.
//   A workgroup takes `window` 16-byte chunks of every row (blockIdx.y: which ones).
template <typename T>
__global__ void __launch_bounds__(512)
k_value_head_bwd(int64_t N, int d, const T* h, const T* w, const float* dv, const uint8_t* mask, const int32_t* cu,
                 const int32_t* gid, int R, T* dh, int accumulate, int window, float* part, double* part_db) {
  constexpr int EPC = 16 / sizeof(T);
  constexpr int BATCH = 8;  // rows in flight per thread
  __shared__ int16_t list[kHeadRows];
  __shared__ float g_s[kHeadRows], grow_s[kHeadRows];  // gradients by list position, by row
  __shared__ int keep_s[kHeadRows];
  __shared__ double db_s[kHeadRows / 64];
  __shared__ float sum_s[256 * EPC];
  const int64_t t0 = (int64_t)blockIdx.x * kHeadRows;
  const int rows = (int)min((int64_t)kHeadRows, N - t0);
  bool keep;
  const int n = list_kept<kHeadRows>(t0, N, mask, cu, gid, R, list, keep);
  const int i = threadIdx.x;
  if (i < kHeadRows) {
    const float g = keep ? dv[t0 + i] : 0.0f;
    grow_s[i] = g;
    keep_s[i] = keep;
    g_s[i] = i < n ? dv[t0 + list[i]] : 0.0f;
    double s = (double)g;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((i & 63) == 0) db_s[i >> 6] = s;
  }
  __syncthreads();
  const int w0 = blockIdx.y * window, nch = min(window, d / EPC - w0);  // the workgroup's 16-byte chunks of a row
  const int deal = nch >= 256 ? 1 : 256 / nch;  // rows side by side
  const int ti = i & 255;
  const int c0 = deal == 1 ? ti : ti % nch, sub = deal == 1 ? 0 : ti / nch;
  // from here on columns are counted from the window's first
  h += w0 * EPC;
  w += w0 * EPC;
  if (dh) dh += w0 * EPC;
  part += (int64_t)blockIdx.x * d + w0 * EPC;
  if (i < 256) {
    if (i == 0 && w0 == 0) {
      double s = 0.0;
      for (int k = 0; k < kHeadRows / 64; ++k) s += db_s[k];
      part_db[blockIdx.x] = s;
    }
    for (int cb = 0; cb < nch; cb += 256) {
      const int c = cb + c0;
      const bool on = c < nch && sub < deal;
      float acc[EPC];
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] = 0.0f;
      for (int k = sub; on && k < n; k += BATCH * deal) {
        u32x4 x[BATCH];
        float g[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const int p = k + u * deal;
          g[u] = p < n ? g_s[p] : 0.0f;
          x[u] = u32x4{0, 0, 0, 0};
          if (p < n) x[u] = *reinterpret_cast<const u32x4*>(h + (t0 + list[p]) * d + c * EPC);
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          if (g[u] == 0.0f) continue;  // a row without gradient adds nothing, whatever it holds
          float f[EPC];
          unpack8<T>(x[u], f);
#pragma unroll
          for (int e = 0; e < EPC; ++e) acc[e] = fmaf(g[u], f[e], acc[e]);
        }
      }
      if (deal == 1) {
        if (on) {
#pragma unroll
          for (int e = 0; e < EPC; e += 4)
            *reinterpret_cast<f32x4*>(part + c * EPC + e) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
        }
      } else {
#pragma unroll
        for (int e = 0; e < EPC; ++e) sum_s[ti * EPC + e] = acc[e];
      }
    }
  } else {
    for (int cb = 0; cb < nch; cb += 256) {
      const int c = cb + c0;
      if (c >= nch || sub >= deal) continue;
      float y[EPC];
      unpack8<T>(*reinterpret_cast<const u32x4*>(w + c * EPC), y);
#pragma unroll 4
      for (int rl = sub; rl < rows; rl += deal) {
        const bool kept = keep_s[rl] != 0;
        if (!kept && accumulate) continue;
        T* row = dh + (t0 + rl) * d + c * EPC;
        float o[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) o[e] = 0.0f;
        if (kept) {
          if (accumulate) unpack8<T>(*reinterpret_cast<const u32x4*>(row), o);
          const float g = grow_s[rl];
#pragma unroll
          for (int e = 0; e < EPC; ++e) o[e] = fmaf(g, y[e], o[e]);
        }
        u32x4 v;
        if constexpr (sizeof(T) == 2) {
          v = u32x4{bf16_pair(o[0], o[1]), bf16_pair(o[2], o[3]), bf16_pair(o[4], o[5]), bf16_pair(o[6], o[7])};
        } else {
          v = u32x4{__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
        }
        *reinterpret_cast<u32x4*>(row) = v;
      }
    }
  }
  if (deal > 1) {
    __syncthreads();
    for (int j = i; j < nch * EPC; j += blockDim.x) {
      float s = 0.0f;
      for (int k = 0; k < deal; ++k) s += sum_s[k * nch * EPC + j];
      part[j] = s;
    }
  }
}

// final sums over the workgroup partials in a fixed order (fp64): a block owns 32 columns; thread
// (column, part) adds the partials of its 32nd of the workgroups in workgroup order, then the part
// sums of a column are added in part order.
__global__ void __launch_bounds__(1024)
k_value_head_dw_final(int nblk, int d, const float* part, const double* part_db, float* dw, float* dbias) {
  __shared__ double sh[32][33];
  const int col = threadIdx.x & 31, pt = threadIdx.x >> 5;
  const int j = blockIdx.x * 32 + col;
  const int b0 = (int)((int64_t)nblk * pt / 32), b1 = (int)((int64_t)nblk * (pt + 1) / 32);
  double s = 0.0;
  if (j < d) {
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += (double)part[(int64_t)b * d + j];
  }
  sh[pt][col] = s;
  __syncthreads();
  if (pt == 0 && j < d) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 32; ++q) t += sh[q][col];
    dw[j] = (float)t;
  }
  if (blockIdx.x > 0) return;
  __syncthreads();
  double t = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 1024) t += part_db[b];
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if ((threadIdx.x & 63) == 0) sh[0][threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    t = 0.0;
    for (int k = 0; k < 16; ++k) t += sh[0][k];
    dbias[0] = (float)t;
  }
}

}  // namespace

size_t value_head_workspace(int64_t N, int d) {
  const int64_t nblk = (N + kHeadRows - 1) / kHeadRows;
  return (size_t)(((nblk * d * 4 + 255) / 256) * 256 + ((nblk * 8 + 255) / 256) * 256);
}

hipError_t launch_value_head_fwd(int dtype, int64_t N, int d, int R, const void* h, const void* w, float b,
                                 const uint8_t* mask, const int32_t* cu, const int32_t* gid, float* values,
                                 hipStream_t s) {
  if (N == 0) return hipSuccess;
  prof_mark(KK_VALUE_HEAD, true, s);
  const unsigned grid = (unsigned)((N + 3) / 4);
  if (dtype == RLK_DTYPE_BF16)
    (d <= 64 * 8 ? k_value_head_fwd<bf16_t, 1> : k_value_head_fwd<bf16_t, 8>)<<<grid, 256, 0, s>>>(
        N, d, (const bf16_t*)h, (const bf16_t*)w, b, mask, cu, gid, R, values);
  else
    (d <= 64 * 4 ? k_value_head_fwd<float, 1> : k_value_head_fwd<float, 8>)<<<grid, 256, 0, s>>>(
        N, d, (const float*)h, (const float*)w, b, mask, cu, gid, R, values);
  prof_mark(KK_VALUE_HEAD, false, s);
  return hipGetLastError();
}

hipError_t launch_value_head_bwd(int dtype, int64_t N, int d, int R, const void* h, const void* w,
                                 const uint8_t* mask, const int32_t* cu, const int32_t* gid, const float* dv,
                                 void* dh, int accumulate, float* dw, float* dbias, char* ws, hipStream_t s) {
  prof_mark(KK_VALUE_HEAD, true, s);
  const int64_t nblk64 = (N + kHeadRows - 1) / kHeadRows;
  const int nblk = (int)nblk64;
  float* part = reinterpret_cast<float*>(ws);
  double* part_db = reinterpret_cast<double*>(ws + ((nblk64 * d * 4 + 255) / 256) * 256);
  const unsigned threads = dh ? 512 : 256;
  // Whole rows per workgroup where those fill the GPU by half; below that, windows of 32 chunks (four lines of a
  // row), so that a call of few rows is not one workgroup (accumulating, 127 rows of 4,096 bf16: 91 -> 23 us).
  const int nch = d / (dtype == RLK_DTYPE_BF16 ? 8 : 4), window = nblk < 128 ? 32 : nch;
  const dim3 grid(nblk, (nch + window - 1) / window);
  if (nblk > 0) {
    if (dtype == RLK_DTYPE_BF16)
      k_value_head_bwd<bf16_t><<<grid, threads, 0, s>>>(N, d, (const bf16_t*)h, (const bf16_t*)w, dv, mask, cu, gid, R,
                                                        (bf16_t*)dh, accumulate, window, part, part_db);
    else
      k_value_head_bwd<float><<<grid, threads, 0, s>>>(N, d, (const float*)h, (const float*)w, dv, mask, cu, gid, R,
                                                       (float*)dh, accumulate, window, part, part_db);
  }
  k_value_head_dw_final<<<(unsigned)((d + 31) / 32), 1024, 0, s>>>(nblk, d, part, part_db, dw, dbias);
  prof_mark(KK_VALUE_HEAD, false, s);
  return hipGetLastError();
}

// Rollouts enough to fill the GPU with single wavefronts, and for the most part one pass of a wavefront (512 rows)
// or less: below 1,024 of them a wavefront is no quicker (15 us of launch and latency either way).
inline bool many_short_rollouts(int64_t N, int R) { return R > 1024 && N / R <= 256; }

hipError_t launch_gae(int64_t N, int R, const int32_t* cu, const uint8_t* mask, const float* values,
                      const float* rewards, const int32_t* gid, float gamma, float lam, float* adv, float* ret,
                      hipStream_t s) {
  // Up to two workgroups of 1,024 threads per compute unit, long rollouts get one each, which covers 8,192 rows in
  // one pass; more of them fill the GPU with smaller ones, and the large ones would wait for each other
  // (16,384 rollouts of 2,000 rows: 437 us, with 256 threads 131 us; 2,048: 22 us with 256, 1,024 30 us with
  // 1,024 threads).  Many short ones get a wavefront (16,384 of 61 rows: 62 us with 256 threads, 19 us with 64).
  // The mean length decides; each is right for any length.
  prof_mark(KK_GAE, true, s);
  const bool vec = aligned16(mask) && aligned16(values) && aligned16(adv) && aligned16(ret);
  const int threads = many_short_rollouts(N, R) ? 64 : (R <= 512 && N / R > 1024 ? 1024 : 256);
  auto* k = threads == 1024 ? (vec ? k_gae<true, 1024> : k_gae<false, 1024>)
            : threads == 256 ? (vec ? k_gae<true, 256> : k_gae<false, 256>)
                             : (vec ? k_gae<true, 64> : k_gae<false, 64>);
  k<<<R, threads, 0, s>>>(N, cu, mask, values, rewards, gid, gamma, lam, adv, ret);
  prof_mark(KK_GAE, false, s);
  return hipGetLastError();
}

hipError_t launch_value_loss(int64_t N, int R, const int32_t* cu, const uint8_t* mask, const float* values,
                             const float* ret, const int32_t* gid, double* part, double* total, float* loss,
                             float* dv, hipStream_t s) {
  prof_mark(KK_VALUE_LOSS, true, s);
  const bool vec = aligned16(mask) && aligned16(values) && aligned16(ret) && aligned16(dv);
  // slices per rollout: one per 2,048 rows of the mean length, as many as the workspace holds
  const int ny = (int)std::min<int64_t>(std::max<int64_t>(R > 0 ? N / R / 2048 : 1, 1), kValueSplit);
  const dim3 grid(R, ny);
  const int np = R * ny;
  const bool small = many_short_rollouts(N, R);  // a wavefront each (16,384 of 61 rows: 44 -> 29 us)
  const unsigned threads = small ? 64 : 256;
  (small ? (vec ? k_value_partial<true, 64> : k_value_partial<false, 64>)
         : (vec ? k_value_partial<true, 256> : k_value_partial<false, 256>))<<<grid, threads, 0, s>>>(N, cu, mask, values,
                                                                                                  ret, gid, part);
  // up to 1,024 partials the gradient's blocks add them up themselves (four loads per thread)
  const bool own_total = dv && np <= 1024;
  if (!own_total) k_value_final<<<1, 1024, 0, s>>>(np, part, total, loss);
  if (dv)
    (small ? (vec ? k_value_grad<true, 64> : k_value_grad<false, 64>)
           : (vec ? k_value_grad<true, 256> : k_value_grad<false, 256>))<<<grid, threads, 0, s>>>(
        N, cu, mask, values, ret, gid, own_total ? np : 0, part, total, loss, dv);
  prof_mark(KK_VALUE_LOSS, false, s);
  return hipGetLastError();
}

}  // namespace rlk
