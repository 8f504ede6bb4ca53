// MFMA GEMMs of the LM-head projection and its two gradient contractions, with fused
// epilogues.  One core computes C[m][n] = sum_k A[m][k] * B[n][k] with both operands
// K-contiguous ("NT"); the three uses are
//   forward : A = W [V, d],          B = gathered hidden [tokens, d]   -> online log-softmax
//   dhidden : A = dz [tokens, Vp],   B = W^T [d, Vp] (or W [V, d])     -> scatter to dh[idx]
//   dW      : A = dz^T [Vp, tokens], B = hidden^T [d, tokens]          -> fp32 dW (+)=
// In the token-reference layout (dz = diag(s) q) the gradient GEMMs read the forward's q and q^T
// as A, the dhidden epilogue scales its rows by s and the dW GEMM's B is (diag(s) hidden)^T.
//
// For few tokens the bf16 dhidden GEMM reads W as it lies ("K-major": K rows of features) by transposing
// fragment reads, which saves the W^T copy.
//
// Tile geometry (gfx950): a 256 x 256 output tile per workgroup of 2 x 4 wavefronts, two per SIMD.
// The tile is four 128 x 128 quadrants; in each, wavefront (wm, wn) owns the 64 x 32 block at
// (64 wm, 32 wn), as 4 x 2 blocks of 16 x 16 (v_mfma_f32_16x16x32_bf16; fp32 operands use
// v_mfma_f32_16x16x4_f32), so its 128 fp32 accumulators cover every half of either operand.  Operands
// stream through LDS in K slices of 128 bytes per row, copied straight from global memory by
// buffer_load ... lds (no staging registers) into two buffers of half tiles (128 rows); rows are
// XOR-swizzled at 16-byte granularity so the fragment reads are bank-conflict free.  Each lane's MFMA
// fragment carries 16 consecutive bytes of one row; A and B use the same K assignment, so the lane
// split of K inside the MFMA is irrelevant to the sum.
//
// The gradient GEMMs of shapes with few output tiles split K over several workgroups per tile
// (fp32 partials in the workspace, summed in split order by k_splitk_reduce).
//
// Output layout of a 16x16 MFMA block D = X Y^T: lane l holds column l % 16 (a row of Y), register r
// row 4 (l / 16) + r (a row of X).  The forward takes X = vocabulary and Y = tokens, so every lane's
// accumulators belong to one token per column block and the vocabulary reduction of the online
// log-softmax is in-register, then over the four lane groups, then one LDS exchange between the two
// wavefronts of a column.  The gradient GEMMs take X = features, so a lane's four registers are
// consecutive in the row-major output and leave in one store.
#include "rlk_internal.h"

#include <algorithm>
#include <type_traits>

namespace rlk {

namespace {

constexpr int WAVES_M = 2, WAVES_N = 4;
constexpr int NWAVE = WAVES_M * WAVES_N;
constexpr int NT = 64 * NWAVE;
constexpr int HALF = kTile / 2;         // rows of a half tile
constexpr int WTM = HALF / WAVES_M;     // rows of a wavefront's block in a quadrant
constexpr int WTN = HALF / WAVES_N;     // columns of it
constexpr int MB = WTM / 16, NB = WTN / 16;  // 16x16 MFMA blocks of it
constexpr int KS = kGemmSliceBytes;     // bytes of K per pipeline slice per row
constexpr int KSE = KS / 2;             // K elements of it (bf16)
constexpr int CPR = KS / 16;            // 16-byte chunks per row of a slice
constexpr int RPI = 64 / CPR;           // rows per LDS-DMA instruction
constexpr int IPH = HALF / RPI / NWAVE; // LDS-DMA instructions per wavefront per half tile
constexpr int HALF_B = HALF * KS;       // a half tile in LDS
constexpr int OPND_B = 4 * HALF_B;      // one operand: two buffers of two half tiles
constexpr int PIPE_B = 2 * OPND_B;      // A then B
static_assert(KS == 128 && IPH == 2 && WTM == 64 && WTN == 32, "pipeline geometry");
constexpr int QROW = kTile * 2 + 16;    // LDS row stride of the bf16 probability tile (bytes)
constexpr int RED_OFF = kTile * QROW;   // 135168: reduction scratch after the staged tile
// The staged tile holds token t's 16-byte vocabulary chunk c at chunk c ^ qswz(t) of row t, so that
// the transposing reads of 8 tokens 8 apart (same chunk) fall in distinct bank groups.
__device__ __forceinline__ int qswz(int t) { return (t >> 3) & 7; }
constexpr int LDS_B = RED_OFF + 3 * WAVES_M * kTile * 4;
static_assert(LDS_B >= PIPE_B && LDS_B <= 163840, "LDS of a compute unit");
constexpr int GROUP_M = 16;
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
constexpr int kBufferFlags = 0x00020000;  // raw buffer: 32-bit data format, offset range-checked

#define LDSP(p) ((__attribute__((address_space(3))) void*)(p))

// 16-byte-chunk XOR swizzle of an LDS row of 8 chunks.  A 16-byte fragment read serves 16 lanes =
// 16 consecutive rows per cycle; with 128-byte rows two rows share one 256-byte bank window, and
// (row parity, chunk ^ swz(row)) is distinct over the 16 rows, so the reads are conflict free.
// swz depends on r mod 16 only: the fragment addresses of a wavefront's 16-row blocks then differ by
// immediate offsets, and a copy's lane offset depends on its instruction only through the
// instruction's parity.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }
// The same for a K-major half tile, rows of 256 bytes: in a transposing read the 16 lanes of a group take
// 32 bytes of each of four K rows 8 lg .. + 3, and the 32-byte unit's XOR with kswz(row) spreads the
// 16 rows of a wavefront's read over the 8 units of the 256-byte bank window, two to each.
__device__ __forceinline__ int kswz(int r) { return (r & 3) | ((r >> 3) & 1) << 2; }

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt[3:0] in
// bits 3:0, vmcnt[5:4] in bits 15:14, expcnt 7 and lgkmcnt 15 = no wait).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}
// LDS/scalar counter to zero, vector memory unconstrained.
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Workgroup barrier without a memory fence: the copies still in flight must stay in flight, so
// the waits are explicit (above); nothing is scheduled across it.
__device__ __forceinline__ void block_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

enum { EPI_FWD = 0, EPI_DH = 1, EPI_DW = 2 };

template <typename T>
struct Op;

template <>
struct Op<bf16_t> {
  static __device__ __forceinline__ void mma(f32x4& c, u32x4 x, u32x4 y) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c,
                                                0, 0, 0);
  }
};

template <>
struct Op<float> {
  static __device__ __forceinline__ void mma(f32x4& c, u32x4 x, u32x4 y) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.x), __uint_as_float(y.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.y), __uint_as_float(y.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.z), __uint_as_float(y.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.w), __uint_as_float(y.w), c, 0, 0, 0);
  }
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2 v;
  v.x = (__bf16)lo;
  v.y = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// four consecutive output elements (16-byte aligned fp32, 8-byte aligned bf16)
__device__ __forceinline__ void store4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void store4(bf16_t* p, f32x4 v) {
  *reinterpret_cast<u32x2*>(p) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

// XCD-aware tile mapping.  Workgroup ids are dispatched round-robin over the 8 XCDs, so the 256
// workgroups resident at a time are 256 consecutive ids.  Tiles are rastered in column groups of
// GROUP_M = 16 M-tiles, so 256 consecutive raster positions cover a 16 x 16 block of tiles; within
// each aligned run of 256 ids the ids are permuted so that XCD x computes the 4 x 8 sub-block
// (M-tiles 4 (x % 4) .. + 4, N-tiles 8 (x / 4) .. + 8) of that block: its 32 CUs then share 4 A
// and 8 B panels in the XCD's L2, and each panel is shared by 2 (A) or 4 (B) XCDs through the
// memory-side cache.  Returns false for workgroups beyond the tile grid.
__device__ __forceinline__ bool map_tile(int tm, int tn, int& tile_m, int& tile_n) {
  const int total = tm * tn;
  const int pid = blockIdx.x;
  if (pid >= total) return false;
  int idx = pid;
  if ((pid | 255) < total) {  // a complete run of 256 ids: XCD-blocked permutation
    const int xcd = pid & 7, slot = (pid >> 3) & 31;
    const int m = 4 * (xcd & 3) + (slot & 3), n = 8 * (xcd >> 2) + (slot >> 2);
    idx = (pid & ~255) + n * 16 + m;
  }
  const int group_sz = GROUP_M * tn;
  const int g = idx / group_sz;
  const int first_m = g * GROUP_M;
  const int gm = min(tm - first_m, GROUP_M);
  const int in = idx - g * group_sz;
  tile_m = first_m + in % gm;
  tile_n = in / gm;
  return true;
}

// The memory step of a K-major operand: fragments f[i][kk] of its 16-row blocks by transposing reads
// (block i's two K steps at LDS address u[i] + AT), the two copies of one of its half tiles (range rs,
// vector offsets o, LDS destinations dst), and the step's waits.  One statement: the
// compiler would wait for every copy in flight before each transposing read of its own (it takes the
// read to alias the copies' LDS writes).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // m0 is set before each copy, here and by the compiler
template <int AT, int VM>
__device__ __forceinline__ void kmajor_step(const int (&u)[NB], u32x4 (&f)[NB][2], u32x4 rs, const uint32_t (&o)[2],
                                            int dst0, int dst1) {
  static_assert(AT + 36 * 256 < 65536, "offset field");
  static_assert(NB == 2, "operand list");
  u32x2 l[NB][2], h[NB][2];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8 offset:%10\n\tds_read_b64_tr_b16 %1, %8 offset:%11\n\t"
      "ds_read_b64_tr_b16 %2, %9 offset:%10\n\tds_read_b64_tr_b16 %3, %9 offset:%11\n\t"
      "ds_read_b64_tr_b16 %4, %8 offset:%12\n\tds_read_b64_tr_b16 %5, %8 offset:%13\n\t"
      "ds_read_b64_tr_b16 %6, %9 offset:%12\n\tds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
      "s_mov_b32 m0, %17\n\ts_nop 0\n\tbuffer_load_dwordx4 %15, %14, 0 offen lds\n\t"
      "s_mov_b32 m0, %18\n\ts_nop 0\n\tbuffer_load_dwordx4 %16, %14, 0 offen lds\n\t"
      "s_waitcnt vmcnt(%19) lgkmcnt(0)"
      : "=&v"(l[0][0]), "=&v"(h[0][0]), "=&v"(l[1][0]), "=&v"(h[1][0]), "=&v"(l[0][1]), "=&v"(h[0][1]),
        "=&v"(l[1][1]), "=&v"(h[1][1])
      : "v"(u[0]), "v"(u[1]), "i"(AT), "i"(AT + 4 * 256), "i"(AT + 32 * 256), "i"(AT + 36 * 256), "s"(rs), "v"(o[0]),
        "v"(o[1]), "s"(dst0), "s"(dst1), "i"(VM)
      : "memory", "m0");
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) f[i][kk] = u32x4{l[i][kk].x, l[i][kk].y, h[i][kk].x, h[i][kk].y};
}
#pragma clang diagnostic pop

// Reference of the stored probabilities of chunk column n in a forward tile with maximum m: m itself,
// or with a.zr (token-reference layout) the column's reference logit r, clamped to m - kRefSpan where
// it lies further below (then, with mark, the chunk is flagged: its dz needs the explicit pass).
// Columns n >= N (padding) keep m.
__device__ __forceinline__ float tile_ref(const GemmArgs& a, float m, int n, int N, bool mark) {
  if (!a.zr || n >= N) return m;
  const float r = a.zr[n];
  if (r >= m - kRefSpan) return r;
  if (mark) *a.fb = 1;
  return m - kRefSpan;
}

// KM_B (dhidden): B is [K][N], K-major.
template <typename T, int EPI, bool STORE_Q, bool KTAIL, bool KM_B = false>
__global__ void __launch_bounds__(NT) k_gemm(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[EPI == EPI_FWD ? LDS_B : PIPE_B];

  int M = a.M, N = a.N, K = a.K;
  // rows of the chunk: every trained token for the forward, those with a surrogate gradient for the
  // gradient GEMMs
  int64_t rc = (int64_t)(EPI == EPI_FWD ? a.hdr->n_eff : a.hdr->n_grad) - a.c0;
  rc = rc < 0 ? 0 : (rc > a.Mc ? a.Mc : rc);
  if (EPI == EPI_FWD) N = (int)rc;
  if (EPI == EPI_DH) M = (int)rc;
  if (EPI == EPI_DW) {
    if (rc == 0 && a.c0 > 0) return;  // nothing to add from an empty chunk
    K = (int)((rc + kKAlign - 1) / kKAlign * kKAlign);
  }
  if (M <= 0 || N <= 0) return;
  const int tm = (M + kTile - 1) / kTile, tn = (N + kTile - 1) / kTile;
  int tile_m, tile_n;
  if (!map_tile(tm, tn, tile_m, tile_n)) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wid / WAVES_N, wn = wid % WAVES_N;
  const int lr = lane & 15, lg = lane >> 4;

  // ---- operand panels as buffer resources: rows beyond M/N (and, with KTAIL, K chunks beyond K)
  // read as zero through the hardware range check; 32-bit offsets address one 256-row panel.
  const uint32_t lda_b = (uint32_t)(a.lda * (int64_t)sizeof(T)), ldb_b = (uint32_t)(a.ldb * (int64_t)sizeof(T));
  const int rows_a = min(kTile, M - tile_m * kTile), rows_b = min(kTile, N - tile_n * kTile);
  char* const pa = const_cast<char*>(reinterpret_cast<const char*>(a.A) + (int64_t)tile_m * kTile * lda_b);
  char* const pb = const_cast<char*>(reinterpret_cast<const char*>(a.B) +
                                     (int64_t)tile_n * kTile * (KM_B ? (int64_t)sizeof(T) : (int64_t)ldb_b));
  // bytes of the whole panel, or (K-major) of one of its K rows
  const uint32_t size_a = (uint32_t)rows_a * lda_b;
  const uint32_t size_b = KM_B ? (uint32_t)rows_b * (uint32_t)sizeof(T) : (uint32_t)rows_b * ldb_b;
  const int64_t Kb = (int64_t)K * sizeof(T);
  int nk = (int)((Kb + KS - 1) / KS);
  // split K: this workgroup covers slices [ks0, ks0 + nk) of the tile's K range
  int ks0 = 0;
  if (EPI != EPI_FWD && a.ksplit > 1) {
    ks0 = (int)blockIdx.y * a.kslices;
    nk = max(0, min(nk, ks0 + a.kslices) - ks0);
  }

  // Direct global->LDS copies (LDS DMA): one instruction moves 64 lanes x 16 bytes into 1 KiB of
  // LDS at consecutive addresses, i.e. RPI rows of one K slice.  Wave w fills rows
  // [w * IPH * RPI, (w + 1) * IPH * RPI) of each half tile; lane l of instruction j carries row
  // (w * IPH + j) * RPI + l / CPR into LDS slot l % CPR, which holds the logical 16-byte K chunk
  // (l % CPR) ^ swz(row).  The row part of the address is uniform and goes into the scalar offset.
  // Rows past the panel (ragged last tiles) read as zero because their vector offset alone is out of
  // range: 0x80000000 >= num_records (every 256-row panel is at most 2 GiB, checked by the host), so
  // the read stays inside the panel whether or not the hardware adds the scalar offset to the check.
  //   A K-major half tile is KSE K rows of 128 elements (256 bytes): an instruction moves four rows, lane
  // l the 16-byte chunk (l % 16) ^ 2 kswz(row) of row l / 16.  Chunks past the operand's last column are
  // put out of range in the same way.  Every wavefront's range starts at the first of the slice's K rows that
  // it copies and ends with the last K row, and the vector offset is the whole offset, so K rows past the last
  // one are out of range too.
  uint32_t vo_a[2][IPH], vo_b[2][IPH];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < IPH; ++j) {
      const int row = (wid * IPH + j) * RPI + lane / CPR;
      const int chunk = (lane % CPR) ^ swz(row);
      vo_a[h][j] = h * HALF + row < rows_a ? (uint32_t)(lane / CPR) * lda_b + chunk * 16 : 0x80000000u;
      if constexpr (KM_B) {
        const uint32_t col = h * 2 * HALF + ((lane & 15) ^ (2 * kswz((wid * IPH + j) * 4 + lane / 16))) * 16;
        vo_b[h][j] = col < size_b ? (uint32_t)(j * 4 + lane / 16) * ldb_b + col : 0x80000000u;
      } else {
        vo_b[h][j] = h * HALF + row < rows_b ? (uint32_t)(lane / CPR) * ldb_b + chunk * 16 : 0x80000000u;
      }
    }
  // Range of this wavefront's copies of slice kt of a K-major B: its K rows of [0, a.V) in this split
  constexpr int KROWS = IPH * 4;  // K rows of them
  auto kmajor_range = [&](int kt) {
    const int row = (kt + ks0) * KSE + wid * KROWS, left = min(a.V, (ks0 + nk) * KSE) - row;
    const uint64_t base = reinterpret_cast<uint64_t>(pb) + (uint64_t)row * (uint64_t)ldb_b;
    return u32x4{(uint32_t)base, (uint32_t)(base >> 32) & 0xffffu,
                 left > 0 ? (uint32_t)(min(left, KROWS) - 1) * ldb_b + size_b : 0u, (uint32_t)kBufferFlags};
  };
  // this wavefront's copies of half h of one operand of slice kt into buffer kt % 2.  Slices past the
  // last one are copied from an empty panel (zeros, no memory access: every vector offset is out of range),
  // which keeps the number of copies in flight the same to the end of the loop.
  auto copy_half = [&](bool op_b, int h, int kt, int buf) {
    const uint32_t kb = (uint32_t)(kt + ks0) * KS;
    const bool km = KM_B && op_b;
    char* base = op_b ? pb : pa;
    uint32_t size = kt < nk ? (op_b ? size_b : size_a) : 0u;
    if (km) {
      const u32x4 r = kmajor_range(kt);
      base = reinterpret_cast<char*>((uint64_t)r.x | (uint64_t)r.y << 32);
      size = r.z;
    }
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)size, kBufferFlags);
#pragma unroll
    for (int j = 0; j < IPH; ++j) {
      uint32_t o = op_b ? vo_b[h][j] : vo_a[h][j];
      if constexpr (KTAIL) {
        // chunks past the end of K would read the next row: push them out of range (zero fill)
        const int row = (wid * IPH + j) * RPI + lane / CPR;
        const uint32_t ck = kb + (((lane % CPR) ^ swz(row)) * 16);
        if ((int64_t)ck >= Kb) o = 0x80000000u;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, LDSP(smem + (op_b ? OPND_B : 0) + (buf * 2 + h) * HALF_B + (wid * IPH + j) * 1024), 16, o,
          km ? 0u : kb + (uint32_t)(h * HALF + (wid * IPH + j) * RPI) * (op_b ? ldb_b : lda_b), 0, 0);
    }
  };
  // Fragment reads: lane (lr, lg) takes logical K chunk 4 kk + lg of row lr of each 16-row block.
  // K-major: the same eight K elements of the same row by two transposing reads; in one, the 16 lanes of
  // group lg address K rows 32 kk + 8 lg + 4 hf + lr / 4, 8 bytes each of the block's 32, and lane lr
  // receives column lr of those four rows.
  const int rd_a = (wm * WTM + lr) * KS, rd_b = OPND_B + (wn * WTN + lr) * KS;
  const int ch0 = (lg ^ swz(lr)) * 16, ch1 = ((4 + lg) ^ swz(lr)) * 16;
  int ku_b[NB];
  {
    const int krow = 8 * lg + (lr >> 2);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      ku_b[nb] = (int)(uintptr_t)LDSP(smem) + OPND_B + krow * 256 + (lr & 3) * 8 + ((wn * NB + nb) ^ kswz(krow)) * 32;
  }
  u32x4 fa[MB][2], fb[2][NB][2];
  auto read_a = [&](int buf, int h) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        fa[mb][kk] = *reinterpret_cast<const u32x4*>(smem + rd_a + (kk ? ch1 : ch0) + (buf * 2 + h) * HALF_B +
                                                     mb * 16 * KS);
  };
  auto read_b = [&](int buf, int h) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        fb[h][nb][kk] = *reinterpret_cast<const u32x4*>(smem + rd_b + (kk ? ch1 : ch0) + (buf * 2 + h) * HALF_B +
                                                        nb * 16 * KS);
  };

  f32x4 acc[2][2][MB][NB];
#pragma unroll
  for (int i = 0; i < 4 * MB * NB; ++i) acc[i / (2 * MB * NB)][i / (MB * NB) % 2][i / NB % MB][i % NB] = f32x4{0, 0, 0, 0};
  // one quadrant of one slice: 16 MFMAs
  auto mma = [&](int ha, int hb) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          if constexpr (EPI == EPI_FWD) Op<T>::mma(acc[ha][hb][mb][nb], fa[mb][kk], fb[hb][nb][kk]);
          else Op<T>::mma(acc[ha][hb][mb][nb], fb[hb][nb][kk], fa[mb][kk]);
        }
    __builtin_amdgcn_s_setprio(0);
  };

  // Main loop.  A slice takes four phases, one quadrant each: (A0, B0), (A0, B1), (A1, B0), (A1, B1).  A
  // phase of a wavefront is a memory step (fragment reads of the operand half that the phase needs
  // first, the copies of one half tile, a wait for the half tile that the next phase reads), a barrier,
  // the 16 MFMAs, and a barrier.  The wavefronts of wm = 1 run one barrier behind those of wm = 0, and
  // the two of a SIMD are of different wm: while one runs its MFMAs the other does its memory step.
  //   A half tile read in phase p is safe to overwrite from the memory step of phase p + 2 on: by then
  // the wavefronts of both groups have waited for their reads (after phase p's barrier) and passed
  // another barrier.  (The first read, of B0 of slice 0, is waited for at once: the copy of slice 2 into
  // that half tile follows the group of wm = 1's second barrier, its first wait of the loop comes after it.)
  // Half tiles are therefore copied in the order B0 A0 B1 A1, two slices ahead, one
  // per phase, and every copy has five phases (1.25 slices) to land: with two copies per half tile, the
  // wait leaves 10 in flight.  B0 of the next slice is read in the last phase of a slice, so the phases
  // read 8, 4, 8 and 4 fragments.
  //   Bound by the matrix cores' power: at 16,384-row chunks and up dhidden and dW keep them busy 86-88 %
  // of the cycles at 1.6 GHz.  Against one barrier and one burst of copies per slice (32 x 32 MFMAs, every
  // copy one slice ahead), d = 4096, V = 151,936, 211,143 tokens: forward 218 -> 193 ms, dhidden 177 ->
  // 155 ms, dW 177 -> 153 ms.  Issuing the copies before the fragment reads costs 5-10 %; raising the
  // copies' lead to six phases, or leaving out s_setprio, changes nothing.
  constexpr int IN_FLIGHT = 5 * IPH;
  // memory step of a phase that reads half RH of B from buffer RB and copies half CH of slice kt of B into
  // buffer CB
  auto step_b = [&](auto RB, auto RH, auto CB, auto CH, int kt) {
    constexpr int rb = decltype(RB)::value, h = decltype(RH)::value, cb = decltype(CB)::value, ch = decltype(CH)::value;
    if constexpr (KM_B) {
      const int dst = (int)(uintptr_t)LDSP(smem) + OPND_B + (cb * 2 + ch) * HALF_B + wid * IPH * 1024;
      kmajor_step<(rb * 2 + h) * HALF_B, IN_FLIGHT>(ku_b, fb[h], kmajor_range(kt), vo_b[ch], dst, dst + 1024);
    } else {
      read_b(rb, h);
      copy_half(true, ch, kt, cb);
      wait_vmcnt<IN_FLIGHT>();
    }
  };
  const std::integral_constant<int, 0> c0{};
  const std::integral_constant<int, 1> c1{};
  copy_half(true, 0, 0, 0);
  copy_half(false, 0, 0, 0);
  copy_half(true, 1, 0, 0);
  copy_half(false, 1, 0, 0);
  copy_half(true, 0, 1, 1);
  copy_half(false, 0, 1, 1);
  wait_vmcnt<IN_FLIGHT>();
  block_barrier();
  step_b(c0, c0, c1, c1, 1);
  wait_lgkm0();
  block_barrier();
  if (wm == 1) block_barrier();
  auto slice = [&](int kt, auto BUF) {
    constexpr int buf = decltype(BUF)::value;
    const std::integral_constant<int, buf> cur{};
    const std::integral_constant<int, buf ^ 1> nxt{};
    read_a(buf, 0);
    copy_half(false, 1, kt + 1, buf ^ 1);
    wait_vmcnt<IN_FLIGHT>();
    block_barrier();
    wait_lgkm0();
    mma(0, 0);
    block_barrier();
    step_b(cur, c1, cur, c0, kt + 2);
    block_barrier();
    wait_lgkm0();
    mma(0, 1);
    block_barrier();
    read_a(buf, 1);
    copy_half(false, 0, kt + 2, buf);
    wait_vmcnt<IN_FLIGHT>();
    block_barrier();
    wait_lgkm0();
    mma(1, 0);
    block_barrier();
    step_b(nxt, c0, cur, c1, kt + 2);
    block_barrier();
    wait_lgkm0();
    mma(1, 1);
    block_barrier();
  };
  for (int kt = 0; kt < nk; kt += 2) {
    slice(kt, c0);
    if (kt + 1 < nk) slice(kt + 1, c1);
  }
  if (wm == 0) block_barrier();
  // the epilogues reuse the LDS of the pipeline
  wait_vmcnt<0>();
  wait_lgkm0();
  block_barrier();

  // ------------------------------------------------------------------ epilogues
  if constexpr (EPI != EPI_FWD) {
    // rows (tokens of the chunk, or vocabulary) of this lane's accumulators: tile row
    // ha*HALF + wm*WTM + mb*16 + lr; columns (features): hb*HALF + wn*WTN + nb*16 + 4*lg + 0..3.
    // N is a multiple of 8, so a group of four columns is inside or outside as a whole.
    const int row0 = tile_m * kTile + wm * WTM + lr, col0 = tile_n * kTile + wn * WTN + 4 * lg;
    auto half_rows = [&](auto FULL, int ha, auto&& f) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int rl = row0 + ha * HALF + mb * 16;
        if (decltype(FULL)::value || rl < M) f(ha, mb, rl);
      }
    };
    auto rows = [&](auto FULL, auto&& f) {
      half_rows(FULL, 0, f);
      half_rows(FULL, 1, f);
    };
    auto cols = [&](auto FULL, auto&& f) {
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int cl = col0 + hb * HALF + nb * 16;
          if (decltype(FULL)::value || cl < N) f(hb, nb, cl);
        }
    };
    auto emit = [&](auto FULL) {
      if (a.ksplit > 1) {
        // split K: fp32 partial of this K range; the reduction kernel applies the epilogue
        float* part = a.part + (int64_t)blockIdx.y * a.mp * a.ldp;
        rows(FULL, [&](int ha, int mb, int rl) {
          cols(FULL, [&](int hb, int nb, int cl) { store4(part + (int64_t)rl * a.ldp + cl, acc[ha][hb][mb][nb]); });
        });
      } else if constexpr (EPI == EPI_DH) {
        // scatter to dh[idx[c0 + row]]; with row scales (token-reference layout), dh = diag(s) (q W^T)
        T* out = reinterpret_cast<T*>(a.out);
        const bool scaled = a.rs != nullptr && *a.rs_off == 0;
        int64_t row[2][MB];
        float sc[2][MB];
        rows(FULL, [&](int ha, int mb, int rl) {
          row[ha][mb] = a.idx[a.c0 + rl];
          sc[ha][mb] = scaled ? a.rs[rl] : 1.0f;
        });
        rows(FULL, [&](int ha, int mb, int rl) {
          cols(FULL, [&](int hb, int nb, int cl) {
            store4(out + row[ha][mb] * a.ldo + cl, acc[ha][hb][mb][nb] * sc[ha][mb]);
          });
        });
      } else {
        // dW is overwritten by the first chunk unless the caller accumulates; dW may be aligned to its
        // elements only
        const bool wide = (reinterpret_cast<uintptr_t>(a.dw) & 15) == 0;
        const bool add = a.accumulate || a.c0 > 0;
#pragma unroll
        for (int ha = 0; ha < 2; ++ha) {
          // the 16 loads of a half are in flight together; those of both halves would not fit the
          // registers
          if (wide && add)
            half_rows(FULL, ha, [&](int, int mb, int rl) {
              cols(FULL, [&](int hb, int nb, int cl) {
                acc[ha][hb][mb][nb] += *reinterpret_cast<const f32x4*>(a.dw + (int64_t)rl * a.ldo + cl);
              });
            });
          half_rows(FULL, ha, [&](int, int mb, int rl) {
            cols(FULL, [&](int hb, int nb, int cl) {
              float* p = a.dw + (int64_t)rl * a.ldo + cl;
              if (wide) {
                store4(p, acc[ha][hb][mb][nb]);
              } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) p[r] = add ? p[r] + acc[ha][hb][mb][nb][r] : acc[ha][hb][mb][nb][r];
              }
            });
          });
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if (rows_a == kTile && rows_b == kTile) emit(std::true_type{});
    else emit(std::false_type{});
  } else {
    // rows = vocabulary v = v0 + rl with rl = ha*HALF + wm*WTM + mb*16 + 4*lg + r, columns =
    // chunk-local token n, tile column hb*HALF + wn*WTN + nb*16 + lr.  Logits z = (W h) / tau.
    if (a.inv_tau != 1.0f) {
#pragma unroll
      for (int i = 0; i < 4 * MB * NB; ++i) acc[i / (2 * MB * NB)][i / (MB * NB) % 2][i / NB % MB][i % NB] *= a.inv_tau;
    }
    const int v0 = tile_m * kTile;
    const int V = a.V;
    // q and q^T are read only for the tokens with a surrogate gradient (the first n_grad of the
    // list): the stores stop there (q^T writes zero columns up to the K pad)
    int ng = N;
    if constexpr (STORE_Q) {
      const int64_t g = (int64_t)a.hdr->n_grad - a.c0;
      ng = g < 0 ? 0 : (g < N ? (int)g : N);
    }
    float* red_m = reinterpret_cast<float*>(smem + RED_OFF);  // [WAVES_M][256]
    float* red_s = red_m + WAVES_M * kTile;                    // [WAVES_M][256]
    float* red_u = red_s + WAVES_M * kTile;                    // [WAVES_M][256]

    char* sQ = smem;
    // Phases 1 and 2, bound by the vector ALU (128 elements per lane): a tile of 256 vocabulary rows (all but
    // the last) takes them without the row checks and u reuses e's exponent.  The forward of 38,900 tokens, d =
    // 2048, V = 32,768: 4.44 -> 4.30 ms; log-probs of 49,000 tokens, d = 5120, V = 151,936: 54.2 -> 53.1 ms.
    auto stats = [&](auto FULL) {
      // phase 1: per-token max over this tile's 256 vocabulary rows; gather the target logit.
#pragma unroll
      for (int cb = 0; cb < 2 * NB; ++cb) {
        const int hb = cb / NB, nb = cb % NB;
        const int cl = hb * HALF + wn * WTN + nb * 16 + lr;
        const int n = tile_n * kTile + cl;
        float mx = -INFINITY;
#pragma unroll
        for (int rb = 0; rb < 2 * MB; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int rl = (rb / MB) * HALF + wm * WTM + (rb % MB) * 16 + 4 * lg + r;
            const float z = (decltype(FULL)::value || v0 + rl < V) ? acc[rb / MB][hb][rb % MB][nb][r] : -INFINITY;
            mx = fmaxf(mx, z);
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (lg == 0) red_m[wm * kTile + cl] = mx;
        if (n < N) {
          const int y = a.ytgt[a.c0 + n];
          const int yl = y - v0;
          if (y >= 0 && y < V && yl >= 0 && yl < kTile && ((yl / WTM) & 1) == wm && ((yl >> 2) & 3) == lg) {
            const int trb = (yl / HALF) * MB + (yl % WTM) / 16, tr = yl & 3;
            float z = 0.0f;
#pragma unroll
            for (int rb = 0; rb < 2 * MB; ++rb)
#pragma unroll
              for (int r = 0; r < 4; ++r) z = (rb == trb && r == tr) ? acc[rb / MB][hb][rb % MB][nb][r] : z;
            a.zy[a.c0 + n] = z;
          }
        }
      }
      __syncthreads();

      // phase 2: e = exp(z - c), s = sum e, u = sum e (z - c) against the token's reference c (the
      // tile maximum m, or with a.zr the reference logit r clamped to m - kRefSpan); e optionally
      // staged for storage.  u sums the exponents of 2 that e is formed from, so the rounding of c log2(e)
      // shifts ln s and u / s alike and leaves the entropy.
#pragma unroll
      for (int cb = 0; cb < 2 * NB; ++cb) {
        const int hb = cb / NB, nb = cb % NB;
        const int cl = hb * HALF + wn * WTN + nb * 16 + lr;
        float mt = red_m[cl];
#pragma unroll
        for (int w = 1; w < WAVES_M; ++w) mt = fmaxf(mt, red_m[w * kTile + cl]);
        const float ref = tile_ref(a, mt, tile_n * kTile + cl, N, true);
        const float mt2 = ref * kLog2e;
        float s = 0.0f, u = 0.0f;
#pragma unroll
        for (int rb = 0; rb < 2 * MB; ++rb) {
          const int rl0 = (rb / MB) * HALF + wm * WTM + (rb % MB) * 16 + 4 * lg;
          float ev[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float z = acc[rb / MB][hb][rb % MB][nb][i];
            const bool valid = decltype(FULL)::value || v0 + rl0 + i < V;
            const float t = fmaf(z, kLog2e, -mt2);
            const float e = valid ? __builtin_amdgcn_exp2f(t) : 0.0f;
            s += e;
            u = fmaf(e, t, u);
            ev[i] = e;
          }
          if constexpr (STORE_Q) {
            if constexpr (sizeof(T) == 2) {
              u32x2 pk;
              pk.x = pack_bf16x2(ev[0], ev[1]);
              pk.y = pack_bf16x2(ev[2], ev[3]);
              *reinterpret_cast<u32x2*>(sQ + cl * QROW + (((rl0 >> 3) ^ qswz(cl)) << 4) + (rl0 & 7) * 2) = pk;
            } else {
              const int n = tile_n * kTile + cl;
              if (n < ng) {
                float* qp = reinterpret_cast<float*>(a.q) + (int64_t)n * a.ldq + v0 + rl0;
                store4(qp, f32x4{ev[0], ev[1], ev[2], ev[3]});
              }
            }
          }
        }
        s += __shfl_xor(s, 16, 64);
        u += __shfl_xor(u, 16, 64);
        s += __shfl_xor(s, 32, 64);
        u += __shfl_xor(u, 32, 64);
        if (lg == 0) {
          red_s[wm * kTile + cl] = s;
          red_u[wm * kTile + cl] = u * kLn2;
        }
      }
    };
    if (v0 + kTile <= V) stats(std::true_type{});
    else stats(std::false_type{});
    __syncthreads();
    if (wm == 0 && lg == 0) {
#pragma unroll
      for (int cb = 0; cb < 2 * NB; ++cb) {
        const int cl = (cb / NB) * HALF + wn * WTN + (cb % NB) * 16 + lr;
        const int n = tile_n * kTile + cl;
        if (n < N) {
          float m = red_m[cl], s = red_s[cl], u = red_u[cl];
#pragma unroll
          for (int w = 1; w < WAVES_M; ++w) {
            m = fmaxf(m, red_m[w * kTile + cl]);
            s += red_s[w * kTile + cl];
            u += red_u[w * kTile + cl];
          }
          const int64_t o = (int64_t)tile_m * a.Mc + n;
          a.pm[o] = tile_ref(a, m, n, N, false);
          a.ps[o] = s;
          a.pu[o] = u;
        }
      }
    }
    if constexpr (STORE_Q && sizeof(T) == 2) {
      // phase 3: coalesced copy of the staged bf16 tile to q[n][v0 .. v0 + 255].  q is read once,
      // by the dz kernel or the dhidden GEMM after this launch: non-temporal stores keep it from
      // displacing the operand panels that later tiles of this launch re-read from the caches.
      const int chunk = tid & 31;
#pragma unroll 4
      for (int it = 0; it < kTile * 32 / NT; ++it) {
        const int cl = (tid >> 5) + (NT / 32) * it;
        const int n = tile_n * kTile + cl;
        if (n < ng) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(sQ + cl * QROW + ((chunk ^ qswz(cl)) << 4));
          char* dst = reinterpret_cast<char*>(a.q) + ((int64_t)n * a.ldq + v0) * 2 + chunk * 16;
          __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
        }
      }
      if (a.qt) {
        // phase 4: the same tile transposed into q^T[v0 .. v0 + 255][tokens of the tile], the dW
        // GEMM's operand (columns of tokens >= n_grad as zero, up to the K pad).  Each lane transposes
        // an 8 x 8 square in registers: wavefront w covers the 16 x 256 blocks (vocabulary rows x
        // tokens) w and w + 8, lane (a8, b8) = (lane / 32, lane % 32) the vocabulary rows 8 a8 .. + 7
        // and tokens 8 b8 .. + 7 of a block, so each store writes two rows of 512 contiguous bytes
        // (8 rows of 128 bytes per store measured 1.5 ms per step slower).  With the chunk swizzle the
        // reads of 8 consecutive lanes fall in distinct bank groups.
        const int a8 = lane >> 5, b8 = lane & 31;
        const int ngpad = (ng + kKAlign - 1) / kKAlign * kKAlign;
#pragma unroll
        for (int it = 0; it < kTile * kTile / 4096 / NWAVE; ++it) {
          const int blk = wid + NWAVE * it;
          const int rl0 = blk * 16 + a8 * 8, cl0 = b8 * 8;
          const int n0 = tile_n * kTile + cl0;
          if (n0 >= ngpad) continue;
          u32x4 in[8];
#pragma unroll
          for (int j = 0; j < 8; ++j)
            in[j] = n0 + j < ng
                        ? *reinterpret_cast<const u32x4*>(sQ + (cl0 + j) * QROW + (((rl0 >> 3) ^ qswz(cl0 + j)) << 4))
                        : u32x4{0, 0, 0, 0};
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            u32x4 o;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              const uint32_t lo = in[2 * m][k >> 1], hi = in[2 * m + 1][k >> 1];
              o[m] = (k & 1) ? ((lo >> 16) | (hi & 0xffff0000u)) : ((lo & 0xffffu) | (hi << 16));
            }
            char* dst = reinterpret_cast<char*>(a.qt) + ((int64_t)(v0 + rl0 + k) * a.ldqt + n0) * 2;
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(dst));
          }
        }
      }
    }
  }
}

// ---- fp32 operands, few output tiles: a 256 x 64 tile per workgroup of four wavefronts, wavefront w the
// 64 x 64 block of its rows 64 w .. + 63 in 32 x 32 MFMA blocks.  A small fp32 call is bound by the fp32 matrix
// rate (1/16 of bf16) and by the compute units without a tile; a slice's MFMAs take 4,096 cycles of a SIMD, so
// one barrier per slice and copies one slice ahead hide the memory.  1,024 tokens, d = 256, V = 4,096, against
// 256 x 256 tiles: forward 75 -> 29 us (64 -> 256 tiles), dhidden 43 -> 27 us, dW 43 -> 26 us.
constexpr int F_MB = kTile / 4 / 32, F_NB = 2;  // 32x32 MFMA blocks of a wavefront

template <int EPI, bool STORE_Q>
__global__ void __launch_bounds__(256, 2) k_gemm_f32(GemmArgs a) {
  constexpr int TN = kTileN32;
  constexpr int F_NW = 4;                     // wavefronts, 64 rows each
  constexpr int F_ROWS = kTile + TN;          // rows of a slice in LDS: A, then B
  constexpr int F_BUF = F_ROWS * KS;
  constexpr int F_IPW = F_ROWS / RPI / F_NW;  // copies of a slice per wavefront
  static_assert(F_ROWS % (RPI * F_NW) == 0 && kTile % (RPI * F_NW) == 0, "a copy is of one operand");
  __shared__ __attribute__((aligned(16))) char smem[2 * F_BUF];
  int M = a.M, N = a.N, K = a.K;
  int64_t rc = (int64_t)(EPI == EPI_FWD ? a.hdr->n_eff : a.hdr->n_grad) - a.c0;
  rc = rc < 0 ? 0 : (rc > a.Mc ? a.Mc : rc);
  if (EPI == EPI_FWD) N = (int)rc;
  if (EPI == EPI_DH) M = (int)rc;
  if (EPI == EPI_DW) {
    if (rc == 0 && a.c0 > 0) return;  // nothing to add from an empty chunk
    K = (int)((rc + kKAlign - 1) / kKAlign * kKAlign);
  }
  if (M <= 0 || N <= 0) return;
  const int tm = (M + kTile - 1) / kTile, tn = (N + TN - 1) / TN;
  int tile_m, tile_n;
  if (!map_tile(tm, tn, tile_m, tile_n)) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const int row0 = tile_m * kTile, col0 = tile_n * TN;

  // operand panels as in k_gemm: rows beyond M / N and K chunks beyond K read as zero
  const uint32_t lda_b = (uint32_t)(a.lda * 4), ldb_b = (uint32_t)(a.ldb * 4);
  const int rows_a = min(kTile, M - row0), rows_b = min(TN, N - col0);
  char* const pa = const_cast<char*>(reinterpret_cast<const char*>(a.A) + (int64_t)row0 * lda_b);
  char* const pb = const_cast<char*>(reinterpret_cast<const char*>(a.B) + (int64_t)col0 * ldb_b);
  const int64_t Kb = (int64_t)K * 4;
  int nk = (int)((Kb + KS - 1) / KS);
  int ks0 = 0;
  if (EPI != EPI_FWD && a.ksplit > 1) {
    ks0 = (int)blockIdx.y * a.kslices;
    nk = max(0, min(nk, ks0 + a.kslices) - ks0);
  }
  const __amdgpu_buffer_rsrc_t ra =
      __builtin_amdgcn_make_buffer_rsrc(pa, (short)0, (int)((uint32_t)rows_a * lda_b), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc(pb, (short)0, (int)((uint32_t)rows_b * ldb_b), kBufferFlags);
  // copy j of this wavefront: rows 8 (wid + F_NW j) .. + 7 of the slice's F_ROWS (A's rows, then B's); lane l
  // carries row l / 8 of them into LDS slot l % 8, which holds the K chunk (l % 8) ^ swz(row)
  auto copy_slice = [&](int kt, int buf) {
    const uint32_t kb = (uint32_t)(kt + ks0) * KS;
#pragma unroll
    for (int j = 0; j < F_IPW; ++j) {
      const int r8 = (wid + F_NW * j) * RPI;
      const bool is_b = j >= kTile / (RPI * F_NW);
      const int r = (is_b ? r8 - kTile : r8), row = r + lane / CPR;
      const int chunk = (lane % CPR) ^ swz(row);
      uint32_t o = (uint32_t)(lane / CPR) * (is_b ? ldb_b : lda_b) + chunk * 16;
      if (row >= (is_b ? rows_b : rows_a) || (int64_t)kb + chunk * 16 >= Kb) o = 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(is_b ? rb : ra, LDSP(smem + buf * F_BUF + r8 * KS), 16, o,
                                               kb + (uint32_t)r * (is_b ? ldb_b : lda_b), 0, 0);
    }
  };

  // two sums per output, of the even and the odd halves of the slices (shorter fp32 chains)
  f32x16 acc[F_MB][F_NB] = {}, acc1[F_MB][F_NB] = {};
  // half hs of a slice: lane (lr, lh) holds chunks 4 hs + lh and 4 hs + 2 + lh of row lr of each 32-row block
  u32x4 fa[F_MB][2][2], fb[F_NB][2][2];
  auto read = [&](int buf, int hs) {
    const char* base = smem + buf * F_BUF;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int ch = ((4 * hs + 2 * c + lh) ^ swz(lr)) * 16;
#pragma unroll
      for (int mb = 0; mb < F_MB; ++mb)
        fa[mb][hs][c] = *reinterpret_cast<const u32x4*>(base + (wid * 64 + mb * 32 + lr) * KS + ch);
#pragma unroll
      for (int nb = 0; nb < F_NB; ++nb)
        fb[nb][hs][c] = *reinterpret_cast<const u32x4*>(base + (kTile + nb * 32 + lr) * KS + ch);
    }
  };
  auto mma = [&](f32x16 (&d)[F_MB][F_NB], int hs) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int mb = 0; mb < F_MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < F_NB; ++nb) {
          const float x = __uint_as_float(fa[mb][hs][e / 4][e % 4]), y = __uint_as_float(fb[nb][hs][e / 4][e % 4]);
          d[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(EPI == EPI_FWD ? x : y, EPI == EPI_FWD ? y : x, d[mb][nb],
                                                           0, 0, 0);
        }
  };
  // Each half of a slice is read under the MFMAs of the half before it.  At the barrier in the middle of slice
  // kt, slice kt + 1 has landed and every wavefront holds the second half of slice kt, whose buffer the copies
  // of slice kt + 2 take.
  if (nk > 0) {
    copy_slice(0, 0);
    wait_vmcnt<0>();
    block_barrier();
    read(0, 0);
    if (nk > 1) copy_slice(1, 1);
  }
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    read(buf, 1);
    mma(acc, 0);
    wait_vmcnt<0>();
    wait_lgkm0();
    block_barrier();
    if (kt + 1 < nk) read(buf ^ 1, 0);
    if (kt + 2 < nk) copy_slice(kt + 2, buf);
    mma(acc1, 1);
  }
#pragma unroll
  for (int i = 0; i < F_MB * F_NB; ++i) acc[i / F_NB][i % F_NB] += acc1[i / F_NB][i % F_NB];
  // Block D = X Y^T: lane (lr, lh) holds column lr (a row of Y), register 4 g + r row 8 g + 4 lh + r (of X)
  auto four = [&](int mb, int nb, int g) {
    const f32x16& d = acc[mb][nb];
    return f32x4{d[4 * g], d[4 * g + 1], d[4 * g + 2], d[4 * g + 3]};
  };

  if constexpr (EPI != EPI_FWD) {
    // rows row0 + 64 wid + 32 mb + lr, columns (features) col0 + 32 nb + 8 g + 4 lh + 0..3
    const bool add = EPI == EPI_DW && (a.accumulate || a.c0 > 0);
    const bool wide = EPI == EPI_DH || (reinterpret_cast<uintptr_t>(a.dw) & 15) == 0;
#pragma unroll
    for (int mb = 0; mb < F_MB; ++mb) {
      const int m = row0 + wid * 64 + mb * 32 + lr;
      if (m >= M) continue;
      float* out;
      if (a.ksplit > 1) out = a.part + ((int64_t)blockIdx.y * a.mp + m) * a.ldp;
      else if constexpr (EPI == EPI_DH) out = reinterpret_cast<float*>(a.out) + (int64_t)a.idx[a.c0 + m] * a.ldo;
      else out = a.dw + (int64_t)m * a.ldo;
#pragma unroll
      for (int i = 0; i < 4 * F_NB; ++i) {
        const int n = col0 + i * 8 + 4 * lh;
        if (n >= N) continue;
        const f32x4 v = four(mb, i / 4, i % 4);
        if (a.ksplit > 1 || (wide && !add)) {
          store4(out + n, v);
        } else if (wide) {
          store4(out + n, *reinterpret_cast<const f32x4*>(out + n) + v);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) out[n + r] = add ? out[n + r] + v[r] : v[r];
        }
      }
    }
  } else {
    // vocabulary rows v = row0 + rl, rl = 64 wid + 8 i + 4 lh + r, i = 4 mb + g; token columns n = col0 + 32 nb + lr
    const int V = a.V;
    int ng = N;
    if constexpr (STORE_Q) {
      const int64_t g = (int64_t)a.hdr->n_grad - a.c0;
      ng = g < 0 ? 0 : (g < N ? (int)g : N);
    }
    block_barrier();  // the reduction reuses the LDS of the pipeline
    float* red_m = reinterpret_cast<float*>(smem);  // [4][TN]
    float* red_s = red_m + 4 * TN;
    float* red_u = red_s + 4 * TN;
#pragma unroll
    for (int nb = 0; nb < F_NB; ++nb) {
      const int cl = nb * 32 + lr, n = col0 + cl;
      float mx = -INFINITY;
#pragma unroll
      for (int mb = 0; mb < F_MB; ++mb) {
        acc[mb][nb] *= a.inv_tau;
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (row0 + wid * 64 + mb * 32 + 8 * (e / 4) + 4 * lh + e % 4 < V) mx = fmaxf(mx, acc[mb][nb][e]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      if (lh == 0) red_m[wid * TN + cl] = mx;
      if (n < N) {
        // the target's logit, if it is one of this lane's
        const int y = a.ytgt[a.c0 + n], yl = y - row0;
        if (y >= 0 && y < V && yl >= 0 && yl < kTile && (yl >> 6) == wid && ((yl >> 2) & 1) == lh) {
          float z = 0.0f;
#pragma unroll
          for (int mb = 0; mb < F_MB; ++mb)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              z = (mb == ((yl >> 5) & 1) && e / 4 == ((yl >> 3) & 3) && e % 4 == (yl & 3)) ? acc[mb][nb][e] : z;
          a.zy[a.c0 + n] = z;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < F_NB; ++nb) {
      const int cl = nb * 32 + lr, n = col0 + cl;
      float m = red_m[cl];
#pragma unroll
      for (int w = 1; w < 4; ++w) m = fmaxf(m, red_m[w * TN + cl]);
      const float m2 = m * kLog2e;
      float s = 0.0f, u = 0.0f;
#pragma unroll
      for (int i = 0; i < 4 * F_MB; ++i) {
        const int rl = wid * 64 + i * 8 + 4 * lh;
        const f32x4 z = four(i / 4, nb, i % 4);
        f32x4 e4;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float t = fmaf(z[r], kLog2e, -m2);
          const float e = row0 + rl + r < V ? __builtin_amdgcn_exp2f(t) : 0.0f;
          s += e;
          u = fmaf(e, t, u);
          e4[r] = e;
        }
        if constexpr (STORE_Q)
          if (n < ng) store4(reinterpret_cast<float*>(a.q) + (int64_t)n * a.ldq + row0 + rl, e4);
      }
      s += __shfl_xor(s, 32, 64);
      u += __shfl_xor(u, 32, 64);
      if (lh == 0) {
        red_s[wid * TN + cl] = s;
        red_u[wid * TN + cl] = u * kLn2;
      }
    }
    __syncthreads();
    const int n = col0 + tid;
    if (tid < TN && n < N) {
      float m = red_m[tid], s = red_s[tid], u = red_u[tid];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        m = fmaxf(m, red_m[w * TN + tid]);
        s += red_s[w * TN + tid];
        u += red_u[w * TN + tid];
      }
      const int64_t o = (int64_t)tile_m * a.Mc + n;
      a.pm[o] = m;
      a.ps[o] = s;
      a.pu[o] = u;
    }
  }
}

// Split-K reduction: out = sum of the partials in split order (deterministic), then the dhidden
// scatter or the dW overwrite / accumulate.  Rows and the empty-chunk rule follow the GEMM.  HBM bound:
// four outputs per thread (N is a multiple of 8), four splits' loads in flight.  A split launch has fewer
// than 256 tiles and the rest of a tile row, so 32 bits count its groups of four.
template <typename T, int EPI>
__global__ void __launch_bounds__(256) k_splitk_reduce(GemmArgs a) {
  int64_t rc = (int64_t)a.hdr->n_grad - a.c0;
  rc = rc < 0 ? 0 : (rc > a.Mc ? a.Mc : rc);
  int M = a.M;
  if (EPI == EPI_DH) M = (int)rc;
  if (EPI == EPI_DW && rc == 0 && a.c0 > 0) return;
  const uint32_t N4 = (uint32_t)a.N / 4, total = (uint32_t)M * N4;
  const bool add = EPI == EPI_DW && (a.accumulate || a.c0 > 0);
  const int64_t step = a.mp * a.ldp;
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
    const uint32_t m = e / N4, n = (e - m * N4) * 4;
    const float* part = a.part + (int64_t)m * a.ldp + n;
    f32x4 acc = {0, 0, 0, 0};
#pragma unroll 4
    for (int y = 0; y < a.ksplit; ++y) acc += *reinterpret_cast<const f32x4*>(part + y * step);
    if constexpr (EPI == EPI_DH) {
      const int64_t row = a.idx[a.c0 + m];
      if (a.rs && *a.rs_off == 0) acc *= a.rs[m];
      store4(reinterpret_cast<T*>(a.out) + row * a.ldo + n, acc);
    } else {
      float* p = a.dw + (int64_t)m * a.ldo + n;  // aligned to its elements only
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = add ? p[r] + acc[r] : acc[r];
    }
  }
}

inline unsigned tiles(int64_t n) { return (unsigned)((n + kTile - 1) / kTile); }

// fp32: of many outputs 256 x 256 tiles are the quicker ones (16,384 rows, d = 2048, V = 32,768, the three GEMMs:
// 14.2-14.7 ms against 16.1-16.6 ms of 64 columns, which read the operands 2.5 times as often); of fewer, compute
// units idle (4,096 rows, d = 512, V = 6,000, forward and dhidden: 137 and 147 us against 115 and 143 us).  The
// two form their sums in different orders, so for a forward and an unsplit dhidden, whose results do not depend
// on the chunk rows, the line is drawn by the rows of the whole batch, from four waves of 256 tiles on: about two
// of the half that is trained.  dW has its outputs fixed: two waves.
inline bool wide_f32(const GemmArgs& a, int epi) {
  if (epi == EPI_DW) return tiles(a.M) * tiles(a.N) >= 512;
  return a.ksplit <= 1 && tiles(epi == EPI_FWD ? a.M : a.N) * tiles(a.rows) >= 1024;
}

// a.M x a.N outputs (dhidden: of at most rows a.Mc)
template <typename T, int EPI>
hipError_t grad_impl(const GemmArgs& a, hipStream_t s) {
  const unsigned tm = tiles(EPI == EPI_DH ? a.Mc : a.M), ny = a.ksplit > 1 ? (unsigned)a.ksplit : 1u;
  const dim3 grid(tm * tiles(a.N), ny);
  if constexpr (sizeof(T) == 4) {
    if (wide_f32(a, EPI)) k_gemm<T, EPI, false, false><<<grid, NT, 0, s>>>(a);
    else k_gemm_f32<EPI, false><<<dim3(tm * (unsigned)((a.N + kTileN32 - 1) / kTileN32), ny), 256, 0, s>>>(a);
  } else if constexpr (EPI == EPI_DH) {
    if (a.b_kmajor) k_gemm<T, EPI, false, false, true><<<grid, NT, 0, s>>>(a);
    else k_gemm<T, EPI, false, false><<<grid, NT, 0, s>>>(a);
  } else {
    k_gemm<T, EPI, false, false><<<grid, NT, 0, s>>>(a);
  }
  if (a.ksplit > 1) {
    const int64_t total = (int64_t)a.M * a.N / 4;
    const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 8192);
    k_splitk_reduce<T, EPI><<<blocks, 256, 0, s>>>(a);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t fwd_impl(const GemmArgs& a, bool store_q, hipStream_t s) {
  const dim3 grid(tiles(a.M) * tiles(a.Mc));
  const bool ktail = ((int64_t)a.K * (int64_t)sizeof(T)) % KS != 0;
  if constexpr (sizeof(T) == 4)
    if (!wide_f32(a, EPI_FWD)) {
      const dim3 small(tiles(a.M) * (unsigned)((a.Mc + kTileN32 - 1) / kTileN32));
      if (store_q) k_gemm_f32<EPI_FWD, true><<<small, 256, 0, s>>>(a);
      else k_gemm_f32<EPI_FWD, false><<<small, 256, 0, s>>>(a);
      return hipGetLastError();
    }
  if (store_q) {
    if (ktail) k_gemm<T, EPI_FWD, true, true><<<grid, NT, 0, s>>>(a);
    else k_gemm<T, EPI_FWD, true, false><<<grid, NT, 0, s>>>(a);
  } else {
    if (ktail) k_gemm<T, EPI_FWD, false, true><<<grid, NT, 0, s>>>(a);
    else k_gemm<T, EPI_FWD, false, false><<<grid, NT, 0, s>>>(a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_gemm(int dtype, const GemmArgs& a, bool store_q, hipStream_t s) {
  prof_mark(KK_FWD_GEMM, true, s);
  const hipError_t e = dtype == RLK_DTYPE_BF16 ? fwd_impl<bf16_t>(a, store_q, s) : fwd_impl<float>(a, store_q, s);
  prof_mark(KK_FWD_GEMM, false, s);
  return e;
}

hipError_t launch_dh_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  prof_mark(KK_DH_GEMM, true, s);
  const hipError_t e = dtype == RLK_DTYPE_BF16 ? grad_impl<bf16_t, EPI_DH>(a, s) : grad_impl<float, EPI_DH>(a, s);
  prof_mark(KK_DH_GEMM, false, s);
  return e;
}

hipError_t launch_dw_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  prof_mark(KK_DW_GEMM, true, s);
  const hipError_t e = dtype == RLK_DTYPE_BF16 ? grad_impl<bf16_t, EPI_DW>(a, s) : grad_impl<float, EPI_DW>(a, s);
  prof_mark(KK_DW_GEMM, false, s);
  return e;
}

}  // namespace rlk
