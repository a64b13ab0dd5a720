// Dense GEMMs of the decoder: C[M,N] (op)= A[M,K] * W[N,K]^T.
// bf16 operands on gfx950 MFMA (v_mfma_f32_16x16x32_bf16), fp32 accumulate.
// Epilogues: store fp32, store bf16, add into an fp32 residual, SwiGLU
// (W rows interleaved in groups of 16: 16 gate rows then the 16 matching up
// rows; output silu(gate) * up as bf16).
//
// Three kernel families, chosen per launch from (M, N, K):
//  * tiled: BM x BN block tile whose A and W slices are copied global -> LDS
//    by direct loads (no register staging) through a ring of 2-4 LDS stages;
//    4 or 8 wavefronts each own a WM x WN register tile.  Blocks are
//    renumbered so that the blocks an XCD runs are neighbours in (m, n) and
//    share operand tiles in that XCD's L2.  Configs: 128x128 with 2 stages
//    (64 KB, two blocks per CU: one block's barrier wait is covered by the
//    other), 128x128 with 4 stages (one block per CU, deepest prefetch: for
//    weight streaming over very wide N), 256x128 with 3 stages, 256x192 and
//    256x256 with 2, all with 8 wavefronts (the large plans that the next family
//    does not run, see plan_alternates), and 64- or 128-row tiles 64 or 96 wide
//    with 4 stages for small batches, where they give exactly one block per CU.
//  * alternating groups (large M): 256x128, 256x192 and 256x256 tiles on
//    persistent blocks of 8 wavefronts in two groups, one fetching fragments
//    while the other issues MFMAs.
//  * skinny (M <= 32 with small W): no LDS for operands; each wavefront loads
//    W and A fragments straight into MFMA operand registers, 8 wavefronts of a
//    block split K and are reduced through LDS.
// Any of them may split K across blocks; partial sums then go to a
// workspace and a reduce kernel adds them in a fixed order (bitwise
// deterministic).  The plan is a pure function of (M, N, K), so results do
// not depend on the device or on earlier calls.
//
// Grouped GEMMs (mixture of experts) run over a device-built list of expert row
// tiles: the tiled kernel, for the gate/up projection in decode batches a
// kernel that streams strip-packed weights straight into MFMA registers (see
// the strip layout below), and in large batches the alternating groups; a plan
// per launch (grouped_plan) picks the row tile and the kernel from the routed
// pairs per expert.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace darts {


__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }

template <int EPI>
__device__ __forceinline__ void epi_store(void* C, int ldc, int M, int m, int n, float v) {
  if (m >= M) return;
  if (EPI == EPI_F32) ((float*)C)[(int64_t)m * ldc + n] = v;
  else if (EPI == EPI_BF16) ((bf16_t*)C)[(int64_t)m * ldc + n] = f32_to_bf16(v);
  else if (EPI == EPI_ADD_F32) ((float*)C)[(int64_t)m * ldc + n] += v;
}

// Write a 16x16 MFMA output tile pair / single tile.  acc layout: lane holds
// rows r0 + 4*(lane/16) + i, column c0 + lane%16.
template <int EPI>
__device__ __forceinline__ void store_tile(void* C, int ldc, int M, int r0, int c0, int lane,
                                           const f32x4_t& v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) epi_store<EPI>(C, ldc, M, r0 + 4 * (lane >> 4) + i, c0 + (lane & 15), v[i]);
}
// gate tile (physical cols 32g..32g+15) and up tile (32g+16..32g+31) -> H cols 16g..16g+15
__device__ __forceinline__ void store_swiglu(bf16_t* H, int ldc, int M, int r0, int pc0, int lane,
                                             const f32x4_t& g, const f32x4_t& u) {
  const int col = (pc0 >> 5) * 16 + (lane & 15);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = r0 + 4 * (lane >> 4) + i;
    if (m < M) H[(int64_t)m * ldc + col] = f32_to_bf16(silu_f(g[i]) * u[i]);
  }
}
__device__ __forceinline__ void store_partial(float* P, int M, int N, int r0, int c0, int lane,
                                              const f32x4_t& v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = r0 + 4 * (lane >> 4) + i;
    if (m < M) P[(int64_t)m * N + c0 + (lane & 15)] = v[i];
  }
}

// ------------------------------------------------------------ strip layout
// Strip-packed weights: a [N][K] matrix (N % 16 == 0, K % 32 == 0) is stored
// as N/16 strips of 16 consecutive rows; strip g holds K/32 blocks of 64 x 8
// bf16, and lane l of block s holds W[16g + l%16][32s + 8(l/16), +8), the B
// operand of v_mfma_f32_16x16x32_bf16 for that strip and K step.  A strip
// occupies the same 16*K elements as in the row-major layout, only reordered.
// Element offset of the 8-element chunk W[n][k, k+8), k % 8 == 0:
__device__ __forceinline__ int64_t strip_off(int n, int k, int K) {
  return (((int64_t)(n >> 4) * (K >> 5) + (k >> 5)) * 64 + (n & 15) + 16 * ((k >> 3) & 3)) * 8;
}

// In-place repack of a row-major [16 * gridDim.x][K] bf16 matrix into the
// strip layout: one block per strip, staged through 16*K*2 bytes of LDS.
__global__ void __launch_bounds__(256) pack_strips_kernel(bf16_t* __restrict__ W, int K) {
  extern __shared__ __attribute__((aligned(16))) bf16_t strip[];
  bf16_t* base = W + (int64_t)blockIdx.x * 16 * K;
  const int nch = 2 * K;                     // 16-byte chunks per strip
  for (int c = threadIdx.x; c < nch; c += blockDim.x)
    *(u32x4_t*)(strip + c * 8) = *(const u32x4_t*)(base + (int64_t)c * 8);
  __syncthreads();
  for (int c = threadIdx.x; c < nch; c += blockDim.x) {
    const int s = c >> 6, l = c & 63;        // block s, lane l: row l%16, K 32s + 8(l/16)
    *(u32x4_t*)(base + (int64_t)c * 8) = *(const u32x4_t*)(strip + (l & 15) * K + 32 * s + 8 * (l >> 4));
  }
}

// ------------------------------------------------------------------ tiled
// Operand tiles travel global -> LDS with direct 16-byte LDS loads (no
// staging registers) through a STAGES-deep ring of LDS buffers.  A KB-wide K
// slice of a row is KB/8 chunks of 16 bytes, stored in a swizzled chunk order
// (dma_swz) so that the 16-byte fragment reads of consecutive rows hit
// distinct banks.  Rows of A past M load row M-1 (their results are never
// stored).  Each wavefront owns a (BM/WGM) x (BN/WGN) register tile of
// 16x16 MFMA accumulators.
// s_waitcnt vmcnt(N) (gfx9 encoding: vmcnt bits 3:0 and 15:14; expcnt and
// lgkmcnt left at their "don't wait" maxima)
template <int N>
__device__ __forceinline__ void vm_wait() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

typedef __attribute__((address_space(3))) void lds_void_t;

// Cache-policy operand of the direct LDS loads that marks them non-temporal
// (the nt bit of gfx950's global loads).  A streaming read of 8 GiB measured
// 7.0 TB/s with non-temporal 16-byte loads against 6.3 TB/s with plain ones;
// the weight streams of the MoE expert GEMMs gain 4-13% from it wherever each
// weight tile is read once per launch.
constexpr int kNtLoad = 2;

// LDS chunk swizzle for a tile row of KB bf16 (KB/8 chunks of 16 bytes): the
// chunk order of row r is permuted so that the 8 rows a 16-byte fragment read
// touches in one LDS pass land in distinct banks.
template <int KB>
__device__ __forceinline__ int dma_swz(int r) {
  if constexpr (KB == 64) return r & 7;
  else return (r >> 1) & 3;
}

// One BM x BN output tile (rows m0.., cols n0.., K range [z*k_chunk, +k_chunk)).
// arow != NULL: row r of the tile's A operand is row arow[r] of A (a gather).
// PW: W is strip-packed (pack_strips_kernel; ldw = K): the same LDS tile is
// filled from the packed addresses, so results are bitwise those of the
// row-major layout.  WAUX: cache policy of the W loads (kNtLoad: non-temporal,
// for weights a launch reads once).
template <int BM, int BN, int KB, int WGM, int WGN, int STAGES, int EPI, bool SPLIT, bool PW = false,
          int WAUX = 0>
__device__ __forceinline__ void dma_gemm_tile(const bf16_t* __restrict__ A, int lda,
                                              const bf16_t* __restrict__ W, int ldw,
                                              void* __restrict__ C, int ldc, int M, int N,
                                              int k_chunk, int mi, int ni, int z,
                                              float* __restrict__ ws,
                                              const int32_t* __restrict__ arow = nullptr) {
  static_assert(KB == 32 || KB == 64, "K tile");
  constexpr int NW = WGM * WGN;                    // wavefronts per block
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  constexpr int CH = KB / 8, RPI = 64 / CH;        // chunks per row, rows per 1 KB load instruction
  constexpr int AI = BM / (RPI * NW), WI = BN / (RPI * NW);   // load instructions per wave per stage
  static_assert(AI * RPI * NW == BM && WI * RPI * NW == BN, "tile rows must split over the waves");
  constexpr int KH = KB / 32;                      // 32-wide MFMA K steps per tile
  constexpr int STAGE_ELEMS = (BM + BN) * KB;      // bf16 elements per stage
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int m0 = mi * BM, n0 = ni * BN;
  const int kbeg = z * k_chunk;
  const int nk = k_chunk / KB;

  // per-lane global source rows for this wave's load instructions: lane i fills
  // LDS bytes [16i, 16i+16) of the instruction's RPI rows, which hold source
  // chunk (i % CH) ^ swizzle(row)
  const int lrow = lane / CH;
  const int gchunk = (lane % CH) ^ dma_swz<KB>(lrow);
  const bf16_t* asrc[AI];
  const bf16_t* wsrc[WI];
#pragma unroll
  for (int j = 0; j < AI; ++j) {
    int r = m0 + wave * (BM / NW) + RPI * j + lrow;
    r = r < M ? r : M - 1;
    if (arow) r = arow[r];
    asrc[j] = A + (int64_t)r * lda + kbeg + gchunk * 8;
  }
#pragma unroll
  for (int j = 0; j < WI; ++j) {
    const int n = n0 + wave * (BN / NW) + RPI * j + lrow;
    if constexpr (PW) wsrc[j] = W + strip_off(n, kbeg + gchunk * 8, ldw);
    else wsrc[j] = W + (int64_t)n * ldw + kbeg + gchunk * 8;
  }
  // one KB-wide K step moves a row-major source KB elements on, a packed one
  // KB/32 blocks of 512 elements
  constexpr int WSTEP = PW ? KB * 16 : KB;

  auto issue = [&](int kt, int buf) {
    bf16_t* sa = smem + buf * STAGE_ELEMS;
    bf16_t* sw = sa + BM * KB;
#pragma unroll
    for (int j = 0; j < AI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(asrc[j] + kt * KB),
                                       (lds_void_t*)(sa + (wave * (BM / NW) + RPI * j) * KB), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < WI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(wsrc[j] + kt * WSTEP),
                                       (lds_void_t*)(sw + (wave * (BN / NW) + RPI * j) * KB), 16, 0, WAUX);
  };

  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue(s, s);

  const int fr = lane & 15, fq = lane >> 4;
  for (int kt = 0; kt < nk; ++kt) {
    // this wave's loads of stage kt are done once at most the (STAGES-2) later
    // stages' loads are outstanding (all outstanding in the last stages); the
    // raw barrier then publishes every wave's stage kt (no memory fence: it
    // would drain the prefetches still in flight)
    if (kt + STAGES - 2 < nk) vm_wait<(STAGES - 2) * (AI + WI)>();
    else vm_wait<0>();
    __builtin_amdgcn_s_barrier();
    if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1, (kt + STAGES - 1) % STAGES);
    const bf16_t* sa = smem + (kt % STAGES) * STAGE_ELEMS;
    const bf16_t* sw = sa + BM * KB;
    // fragments of every 32-wide K step are read before the first MFMA, so
    // LDS latency overlaps matrix work
    bf16x8_t a[KH][TM], bb[KH][TN];
#pragma unroll
    for (int ks = 0; ks < KH; ++ks) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int r = wm * WM + 16 * i + fr;
        a[ks][i] = *(const bf16x8_t*)(sa + r * KB + (((ks * 4 + fq) ^ dma_swz<KB>(r)) * 8));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int r = wn * WN + 16 * j + fr;
        bb[ks][j] = *(const bf16x8_t*)(sw + r * KB + (((ks * 4 + fq) ^ dma_swz<KB>(r)) * 8));
      }
    }
#pragma unroll
    for (int ks = 0; ks < KH; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], bb[ks][j], acc[i][j], 0, 0, 0);
  }

  const int rb = m0 + wm * WM, cb = n0 + wn * WN;
  if constexpr (SPLIT) {
    float* P = ws + (int64_t)z * M * N;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) store_partial(P, M, N, rb + 16 * i, cb + 16 * j, lane, acc[i][j]);
  } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; j += 2)
        store_swiglu((bf16_t*)C, ldc, M, rb + 16 * i, cb + 16 * j, lane, acc[i][j], acc[i][j + 1]);
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) store_tile<EPI>(C, ldc, M, rb + 16 * i, cb + 16 * j, lane, acc[i][j]);
  }
}

// ------------------------------------------------------- alternating groups
// BM x BN output tile for compute-bound launches: 8 wavefronts in two groups
// of four (one wavefront of each group per SIMD) that alternate between
// fetching operands from LDS and issuing MFMAs, so the matrix cores of a SIMD
// run one wavefront's products while the other wavefront reads its next
// fragments.  The second group runs one barrier behind the first.
//
// A 64-wide K tile is four half tiles in LDS (A0, A1 of BM/2 rows, B0, B1 of
// BN/2 rows of W), double-buffered.  A wavefront owns TM x TN 16x16
// accumulators of each of the four A half x B half quadrants and takes two
// quadrants per phase: (A0,B0) (A0,B1), then (A1,B0) (A1,B1).  The first phase
// reads A0 and B1 (B0's fragments are there already), the second A1 and the
// next K tile's B0, so both read equally much and the reads of one group last
// about as long as the MFMAs of the other.  Each phase also issues the direct
// LDS loads of two half tiles one or two K tiles ahead, into the half tiles
// read one phase earlier, and waits until at most the four youngest half tiles
// are in flight; the barrier that ends the fetch section then publishes the
// half tiles the next phase reads.
//
// MFMAs take W as the first operand, so a lane's four accumulators are four
// consecutive columns of one output row and the epilogue stores them together.
// For SwiGLU B0 holds the gate rows and B1 the up rows of the tile's columns,
// so a lane has both of a feature.  The sums run over K in the same order as
// in dma_gemm_tile, so results are bitwise those of the tiled kernel.
//
// Bound by the matrix cores, at the clock that the card's power allows: a
// library GEMM of the same sizes reaches 1530 TFLOP/s.  Measured on the
// Qwen3-8B gate/up projection against the tiled kernel, where every wavefront
// reads its fragments and then issues its MFMAs behind one barrier per K tile:
// 16384 rows 2080 us (1590 TFLOP/s) against 2880 us, 4096 rows 535 against 747
// us, 389 rows (256x192 tiles, weights cold) 76 against 96 us; QKV at 4096 rows
// 154 against 187 us.  Four phases of one quadrant each (8 barriers per K tile)
// took 561 us at 4096 rows.
template <int N>
__device__ __forceinline__ void vm_lgkm_wait() {   // vmcnt(N) and lgkmcnt(0)
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4));
}
// Neither memory accesses nor MFMAs are moved across.
__device__ __forceinline__ void order_fence() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// The same with a raw barrier.
__device__ __forceinline__ void fenced_barrier() {
  order_fence();
  __builtin_amdgcn_s_barrier();
  order_fence();
}

// One output tile of alt_gemm_items.
struct AltItem {
  const bf16_t* a;       // its first row of A (arow set: A itself), at the first column of its K range
  const bf16_t* w;       // its first row of W, at the first column of its K range
  char* c;               // its first output element
  int rows;              // rows of the output from the tile's first one on (> 0)
  const int32_t* arow;   // NULL, or the A row of each of them
};

// A block's items, one after the other; next(item) yields the first, then each
// following one, or false.  nk: 64-wide K tiles of every item, even.  PW: W is
// strip-packed (ldw = K).  An item's row list is read during the last K tiles of
// the item before it, and its first loads are issued before that item's results
// are stored, so neither latency is waited for (EPI_ADD_F32 reads the results'
// old values behind those loads, and waits for them).
template <int BM, int BN, int WGM, int WGN, int EPI, bool SPLIT, bool PW, typename Next>
__device__ __forceinline__ void alt_gemm_items(int lda, int ldw, int ldc, int nk, Next next) {
#ifdef __HIP_DEVICE_COMPILE__   // the host pass knows no buffer resources
  constexpr int KB = 64, NW = 8;
  static_assert(WGM * WGN == NW, "8 wavefronts");
  constexpr int HM = BM / 2, HN = BN / 2;             // half tile rows
  constexpr int TM = HM / WGM / 16, TN = HN / WGN / 16;
  static_assert(TM * WGM * 16 == HM && TN * WGN * 16 == HN, "half tiles split evenly over the wavefronts");
  // 1 KB (8-row) loads per half tile, load i by wavefront i % 8; per wavefront
  // of the first and of the second group
  constexpr int IA = HM / 8, IB = HN / 8;
  constexpr int LA = IA / NW, LB = (IB + NW - 1) / NW;
  static_assert(IA % NW == 0 && IB % 4 == 0 && IB >= NW, "a group's wavefronts issue equally many loads");
  constexpr int LB1 = IB / NW;                        // second group
  // LDS: the two stages of A0, of A1, of B0, of B1, so that either operand's
  // fragment reads differ by constants that fit the instruction's offset
  constexpr int HA = HM * KB, HB = HN * KB;
  constexpr bool kSwiglu = !SPLIT && EPI == EPI_SWIGLU;
  constexpr int kEsz = !SPLIT && (EPI == EPI_BF16 || EPI == EPI_SWIGLU) ? 2 : 4;   // output element
  // stores of a whole tile per lane (16 bytes, or 8 at addresses that are not
  // adjacent, so that none are merged)
  constexpr int kStores = 2 * TM * TN * (kSwiglu ? 1 : 2) / (kEsz == 2 && TN % 2 == 0 ? 2 : 1);
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool first = wave < 4;                        // group
  const int wm = wave / WGN, wn = wave % WGN;

  // Source addresses are a buffer resource, a 32-bit lane offset in bytes that
  // stays the same over K, and a uniform offset that moves on (no vector
  // registers or instructions per load).  Gathered A rows are offsets from A
  // itself (the launcher checks that they fit), others from the tile's first row.
  const int lrow = lane >> 3;
  const int gchunk = (lane & 7) ^ lrow;               // source chunk of this lane's LDS slot
  // Order of W's rows in a half tile.  With 16-bit results and an even number
  // of column tiles per wavefront, two tiles t = 0, 1 share 32 columns, column
  // c of tile t being column 8*(c/4) + 4*t + c%4 of them: a lane's four
  // accumulators of either tile are then 8 consecutive columns, one 16-byte
  // store, and a row's four lanes write 64 bytes in one piece.  (8-byte stores
  // in 32-byte pieces cost the MoE down projection of 32768 rows, 1.07 GB of
  // results, 0.43 ms of its 1.03 ms.)  Otherwise rows are in order.
  constexpr bool kPair = kEsz == 2 && TN % 2 == 0;
  const int wlane = kPair ? 8 * (lrow >> 2) + (lrow & 3) : lrow;   // row in a strip of 16, but for a uniform part
  const int woff = PW ? ((gchunk & 3) * 16 + wlane) * 16 + (gchunk >> 2) * 1024 : (wlane * ldw + gchunk * 8) * 2;
  auto row_ids = [&](const AltItem& t, int (&row)[2][LA]) {
    int row0 = lrow;
    asm volatile("" : "+v"(row0));                    // recomputed here, not kept over the K loop
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < LA; ++j) {
        int r = min(h * HM + (wave + NW * j) * 8 + row0, t.rows - 1);
        row[h][j] = t.arow ? t.arow[r] : r;
      }
  };
  AltItem cur;
  int arow[2][LA], aoff[2][LA];
  if (!next(cur)) return;
  row_ids(cur, arow);
  auto ares = __builtin_amdgcn_make_buffer_rsrc((void*)cur.a, 0, -1, 0x00020000);
  auto wres = __builtin_amdgcn_make_buffer_rsrc((void*)cur.w, 0, -1, 0x00020000);
  // K tile kt belongs in stage kt & 1, which the callers know as a constant
  auto issue_a = [&](int kt, int stage, int h) {
    bf16_t* s = smem + (2 * h + stage) * HA + wave * 8 * KB;
#pragma unroll
    for (int j = 0; j < LA; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ares, (lds_void_t*)(s + NW * j * 8 * KB), 16, aoff[h][j],
                                               kt * (KB * 2), 0, 0);
  };
  auto issue_b = [&](int kt, int stage, int h) {
    bf16_t* s = smem + 4 * HA + (2 * h + stage) * HB + wave * 8 * KB;
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      if (j == LB1 && !first) break;
      const int q = wave + NW * j;                    // 8 rows of the half tile: of which strip, from which row
      const int strip = kPair ? (q >> 2) * 2 + (q & 1) : q >> 1, sub = kPair ? ((q >> 1) & 1) * 4 : (q & 1) * 8;
      // a wavefront's TN column tiles of B0 and then its TN of B1 are neighbours
      const int row = (kSwiglu ? strip * 2 + h : strip / TN * 2 * TN + h * TN + strip % TN) * 16;
      const int off = PW ? row * 2 * ldw + sub * 16 + kt * (KB * 32) : (row + sub) * 2 * ldw + kt * (KB * 2);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(wres, (lds_void_t*)(s + NW * j * 8 * KB), 16, woff, off, 0, 0);
    }
  };

  const int fr = lane & 15, fq = lane >> 4;
  const int cvoff = (fr * ldc + fq * (kPair ? 8 : 4)) * kEsz;
  // fragments [K step][tile]: of an A half, of B1, and of B0 for this K tile
  // and the next (by parity of the K tile)
  bf16x8_t a[2][TM], b1[2][TN], b0[2][2][TN];
  f32x4_t acc[2][2][TM][TN];
  // rows are multiples of 16 apart, so the swizzle of a lane's row is fr & 7
  const bf16_t* pa = smem + (wm * TM * 16 + fr) * KB;
  const bf16_t* pb = smem + 4 * HA + (wn * TN * 16 + fr) * KB;
  const int c0 = (fq ^ (fr & 7)) * 8, c1 = ((4 + fq) ^ (fr & 7)) * 8;
  auto read_a = [&](int stage, int h) {
    const bf16_t* s = pa + (2 * h + stage) * HA;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      a[0][i] = *(const bf16x8_t*)(s + i * 16 * KB + c0);
      a[1][i] = *(const bf16x8_t*)(s + i * 16 * KB + c1);
    }
  };
  auto read_b = [&](int stage, int h, bf16x8_t (&f)[2][TN]) {
    const bf16_t* s = pb + (2 * h + stage) * HB;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      f[0][j] = *(const bf16x8_t*)(s + j * 16 * KB + c0);
      f[1][j] = *(const bf16x8_t*)(s + j * 16 * KB + c1);
    }
  };
  auto mma = [&](int h, const bf16x8_t (&f0)[2][TN]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[h][0][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f0[ks][j], a[ks][i], acc[h][0][i][j], 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[h][1][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b1[ks][j], a[ks][i], acc[h][1][i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // The fetch section ends: this wavefront's fragments are in registers, and
  // all but the NA youngest A and NB youngest B half tiles have landed (vector
  // memory operations retire in order).  MAYBE, stored: the kStores stores of
  // the item before may be younger than those half tiles, too.
  auto landed = [&](auto NA, auto NB, auto MAYBE, bool stored) {
    constexpr int na = decltype(NA)::value, nb = decltype(NB)::value, st = decltype(MAYBE)::value ? kStores : 0;
    static_assert(na * LA + nb * LB + st < 64, "vmcnt range");
    if (st && stored) {
      if (LB1 == LB || first) vm_lgkm_wait<na * LA + nb * LB + st>();
      else vm_lgkm_wait<na * LA + nb * LB1 + st>();
    } else {
      if (LB1 == LB || first) vm_lgkm_wait<na * LA + nb * LB>();
      else vm_lgkm_wait<na * LA + nb * LB1>();
    }
    fenced_barrier();
  };
  constexpr std::integral_constant<int, 0> n0{};
  constexpr std::integral_constant<int, 1> n1{};
  constexpr std::integral_constant<int, 2> n2{};
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  // LEFT: 0 in the steady loop, 1 for the last tile but one, 2 for the last
  auto tile = [&](int kt, auto P, auto LEFT, auto MAYBE, bool stored) {
    constexpr int p = decltype(P)::value, left = decltype(LEFT)::value;
    if constexpr (left < 2) issue_a(kt + 1, 1 - p, 1);
    if constexpr (left < 1) issue_b(kt + 2, p, 0);
    read_a(p, 0);
    read_b(p, 1, b1);
    if constexpr (left == 0) landed(n2, n2, MAYBE, stored);
    else if constexpr (left == 1) landed(n2, n1, MAYBE, stored);
    else landed(n0, n0, MAYBE, false);
    mma(0, b0[p]);
    fenced_barrier();
    if constexpr (left < 1) { issue_a(kt + 2, p, 0); issue_b(kt + 2, p, 1); }
    read_a(p, 1);
    if constexpr (left < 2) read_b(1 - p, 0, b0[1 - p]);
    if constexpr (left == 0) landed(n2, n2, MAYBE, stored);
    else if constexpr (left == 1) landed(n1, n0, MAYBE, stored);
    else landed(n0, n0, MAYBE, false);
    mma(1, b0[p]);
    fenced_barrier();
  };
  // the first loads of cur, whose rows are in arow
  auto start = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < LA; ++j)
        aoff[h][j] = (int)(((uint32_t)arow[h][j] * (uint32_t)lda + gchunk * 8) * 2u);
    ares = __builtin_amdgcn_make_buffer_rsrc((void*)cur.a, 0, -1, 0x00020000);
    wres = __builtin_amdgcn_make_buffer_rsrc((void*)cur.w, 0, -1, 0x00020000);
    issue_b(0, 0, 0); issue_a(0, 0, 0); issue_b(0, 0, 1);
    issue_a(0, 0, 1); issue_b(1, 1, 0); issue_a(1, 1, 0); issue_b(1, 1, 1);
  };

  start();
  bool stored = false;
  while (true) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[h][g][i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    landed(n2, n2, yes, stored);
    read_b(0, 0, b0[0]);
    landed(n2, n2, yes, stored);
    if (!first) fenced_barrier();                     // the second group runs one barrier behind
    if (nk > 2) {
      tile(0, n0, n0, yes, stored);
      tile(1, n1, n0, no, false);
      for (int kt = 2; kt < nk - 2; kt += 2) {
        tile(kt, n0, n0, no, false);
        tile(kt + 1, n1, n0, no, false);
      }
    }
    AltItem nxt;
    const bool more = next(nxt);
    if (more) row_ids(nxt, arow);                     // read while the last two K tiles are computed
    tile(nk - 2, n0, n1, no, false);
    tile(nk - 1, n1, n2, no, false);
    if (first) fenced_barrier();

    const auto cres = __builtin_amdgcn_make_buffer_rsrc((void*)cur.c, 0, -1, 0x00020000);
    const int rows = cur.rows;
    if (more) {
      cur = nxt;
      start();
    }
    order_fence();   // landed() counts the stores below as younger than start()'s loads
    // accumulators: row 16*i + lane%16, columns 16*j + 4*(lane/16) .. +3, or with
    // kPair those of tiles j, j + 1 columns 16*j + 8*(lane/16) .. +7
    auto store = [&](int h, int i) {
      const int m = h * HM + (wm * TM + i) * 16;      // this wavefront's 16 rows
      if constexpr (kEsz == 2) {
#pragma unroll
        for (int g = 0; g < (kSwiglu ? 1 : 2); ++g) {
          uint2 v[TN];
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            f32x4_t u = acc[h][g][i][j];
            if constexpr (kSwiglu) {
#pragma unroll
              for (int e = 0; e < 4; ++e) u[e] = silu_f(u[e]) * acc[h][1][i][j][e];
            }
            v[j] = make_uint2(f32_to_bf16x2(u[0], u[1]), f32_to_bf16x2(u[2], u[3]));
          }
#pragma unroll
          for (int j = 0; j < TN; j += kPair ? 2 : 1) {
            const int o = (m * ldc + ((kSwiglu ? wn : 2 * wn + g) * TN + j) * 16) * kEsz;
            if constexpr (kPair)
              __builtin_amdgcn_raw_buffer_store_b128((u32x4_t){v[j].x, v[j].y, v[j + 1].x, v[j + 1].y}, cres, cvoff, o, 0);
            else
              __builtin_amdgcn_raw_buffer_store_b64((u32x2_t){v[j].x, v[j].y}, cres, cvoff, o, 0);
          }
        }
      } else {
        f32x4_t r[2][TN];
        if constexpr (!SPLIT && EPI == EPI_ADD_F32) {
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              r[g][j] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                        cres, cvoff, (m * ldc + ((kSwiglu ? wn : 2 * wn + g) * TN + j) * 16) * kEsz, 0));
        }
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            f32x4_t v = acc[h][g][i][j];
            if constexpr (!SPLIT && EPI == EPI_ADD_F32) v += r[g][j];
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), cres, cvoff,
                                                   (m * ldc + ((kSwiglu ? wn : 2 * wn + g) * TN + j) * 16) * kEsz, 0);
          }
      }
    };
    stored = rows >= BM;
    if (stored) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i) store(h, i);
    } else {
      int row0 = fr;
      asm volatile("" : "+v"(row0));
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
          if (row0 < rows - (h * HM + (wm * TM + i) * 16)) store(h, i);
    }
    if (!more) break;
  }
#endif
}

// Blocks are renumbered so that the blocks one XCD runs (dispatch is round
// robin over the 8 XCDs) are consecutive tiles and share operands in its L2.
__device__ __forceinline__ int xcd_block() {
  const int nb = gridDim.x;
  int b = blockIdx.x;
  const int full = (nb / 8) * 8;
  if (b < full) b = (b % 8) * (full / 8) + b / 8;
  return b;
}

template <int BM, int BN, int KB, int WGM, int WGN, int STAGES, int EPI, bool SPLIT, int WAUX>
__global__ void __launch_bounds__(64 * WGM * WGN) gemm_dma_kernel(const bf16_t* __restrict__ A, int lda,
                                                       const bf16_t* __restrict__ W, int ldw,
                                                       void* __restrict__ C, int ldc, int M,
                                                       int N, int /*K*/, int k_chunk, int mt, int nt,
                                                       float* __restrict__ ws) {
  const int b = xcd_block();
  const int mi = b % mt, ni = (b / mt) % nt, z = b / (mt * nt);
  dma_gemm_tile<BM, BN, KB, WGM, WGN, STAGES, EPI, SPLIT, false, WAUX>(A, lda, W, ldw, C, ldc, M, N, k_chunk, mi,
                                                                       ni, z, ws);
}

// Tile order of one XCD's run of consecutive tiles: panels of kPanel row tiles,
// column tiles fastest after the panel's rows, so that the 32 tiles the XCD has
// in flight are about 8 x 4 and read 12 operand tiles, not 33.
constexpr int kPanel = 8;
__device__ __forceinline__ void panel_order(int b, int mt, int nt, int& mi, int& ni) {
  const int p = b / (kPanel * nt), rows = min(kPanel, mt - p * kPanel);
  const int r = b - p * kPanel * nt;
  mi = p * kPanel + r % rows;
  ni = r / rows;
}

// One persistent block per CU.  Each XCD takes a contiguous eighth of the tiles
// (blocks are dealt to the 8 XCDs round robin), its blocks in turn.
template <int BM, int BN, int WGM, int WGN, int EPI, bool SPLIT>
__global__ void __launch_bounds__(512, 2) gemm_alt_kernel(const bf16_t* __restrict__ A, int lda,
                                                          const bf16_t* __restrict__ W, int ldw,
                                                          void* __restrict__ C, int ldc, int M, int N,
                                                          int k_chunk, int mt, int nt, int n_split,
                                                          float* __restrict__ ws) {
  constexpr int esz = (SPLIT || EPI == EPI_F32 || EPI == EPI_ADD_F32) ? 4 : 2;
  const int total = mt * nt * n_split, chunk = (total + 7) >> 3;
  const int hi = min(total, ((int)(blockIdx.x & 7) + 1) * chunk);
  int it = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
  auto next = [&](AltItem& t) {
    if (it >= hi) return false;
    const int z = it / (mt * nt);
    int mi, ni;
    panel_order(it - z * mt * nt, mt, nt, mi, ni);
    it += (int)(gridDim.x >> 3);
    t.a = A + (int64_t)mi * BM * lda + z * k_chunk;
    t.w = W + (int64_t)ni * BN * ldw + z * k_chunk;
    const int64_t out = (int64_t)mi * BM * ldc + (EPI == EPI_SWIGLU && !SPLIT ? ni * BN / 2 : ni * BN);
    t.c = SPLIT ? (char*)(ws + (int64_t)z * M * N + out) : (char*)C + out * esz;
    t.rows = M - mi * BM;
    t.arow = nullptr;
    return true;
  };
  alt_gemm_items<BM, BN, WGM, WGN, EPI, SPLIT, false>(lda, ldw, ldc, k_chunk / 64, next);
}

// Grouped GEMM (mixture-of-experts): group e owns rows [off[e], off[e] +
// cnt[e]) of C (and of A, or of the gather list arow into A) and the weight
// matrix W + e * w_stride ([N][K]).  The
// non-empty row tiles are listed on the device (mtiles[i] = e << 16 | m tile,
// *n_mtiles of them); persistent blocks take items (row tile, n tile), n tile
// fastest, in a grid-stride loop.  PW: W strip-packed; WAUX: W cache policy.
template <int BM, int BN, int KB, int WGM, int WGN, int STAGES, int EPI, bool PW, int WAUX>
__global__ void __launch_bounds__(64 * WGM * WGN) gemm_dma_grouped_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int64_t w_stride, int ldw,
    void* __restrict__ C, int ldc, int N, int K, const int32_t* __restrict__ g_off,
    const int32_t* __restrict__ g_cnt, const int32_t* __restrict__ mtiles,
    const int32_t* __restrict__ n_mtiles, int nt, const int32_t* __restrict__ arow) {
  const int total = n_mtiles[0] * nt;
  constexpr int esz = (EPI == EPI_F32 || EPI == EPI_ADD_F32) ? 4 : 2;
  // Items are (row tile, column tile) in row-tile order.  With gathered A
  // rows, each XCD takes one contiguous eighth of the items (blocks are dealt
  // to the 8 XCDs round robin, block b on XCD b % 8), so the column tiles of
  // one expert row tile run on one XCD and find its gathered input rows in
  // that XCD's L2; the grid is a multiple of 8 blocks and the eighths
  // partition [0, total).  Otherwise items go to blocks round robin (the
  // down projection measured no gain from the XCD split).
  const bool by_xcd = arow != nullptr;
  const int chunk = (total + 7) >> 3;
  const int lo = by_xcd ? (int)(blockIdx.x & 7) * chunk : 0;
  const int hi = by_xcd ? min(total, lo + chunk) : total;
  const int step = by_xcd ? (int)(gridDim.x >> 3) : (int)gridDim.x;
  for (int it = by_xcd ? lo + (int)(blockIdx.x >> 3) : (int)blockIdx.x; it < hi; it += step) {
    const int mt = mtiles[it / nt], ni = it % nt;
    const int e = mt >> 16, mi = mt & 0xffff;
    const int cnt = g_cnt[e];
    const int64_t off = g_off[e];
    // other waves may still read the previous item's last LDS stage: a raw
    // barrier (their LDS reads have retired once their MFMAs issued); no
    // memory fence, which would also wait for the previous item's stores
    __builtin_amdgcn_s_barrier();
    void* Ce = (char*)C + off * ldc * esz;
    // with arow, A rows are gathered: segment row r is A row arow[off + r]
    dma_gemm_tile<BM, BN, KB, WGM, WGN, STAGES, EPI, false, PW, WAUX>(arow ? A : A + off * lda, lda,
                                                            W + (int64_t)e * w_stride, ldw, Ce, ldc,
                                                            cnt, N, K, mi, ni, 0, nullptr,
                                                            arow ? arow + off : nullptr);
  }
}

// Grouped GEMM of large batches (the prefill): 256 x 256 tiles of the
// alternating-group kernel, one persistent block per CU.  Items (row tile,
// column tile), column tile fastest, in eighths by XCD as above: the column
// tiles of an expert's row tile run on one XCD and share its rows in that
// XCD's L2.  The last barrier of an item also frees its LDS stages.
template <int EPI, bool PW>
__global__ void __launch_bounds__(512, 2) gemm_alt_grouped_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int64_t w_stride, int ldw,
    void* __restrict__ C, int ldc, int N, int K, const int32_t* __restrict__ g_off,
    const int32_t* __restrict__ g_cnt, const int32_t* __restrict__ mtiles,
    const int32_t* __restrict__ n_mtiles, int nt, const int32_t* __restrict__ arow) {
  constexpr int esz = (EPI == EPI_F32 || EPI == EPI_ADD_F32) ? 4 : 2;
  constexpr int BM = 256, BN = 256;
  const int total = n_mtiles[0] * nt, chunk = (total + 7) >> 3;
  const int hi = min(total, ((int)(blockIdx.x & 7) + 1) * chunk);
  int it = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
  auto next = [&](AltItem& t) {
    if (it >= hi) return false;
    const int mt = mtiles[it / nt], ni = it % nt;
    it += (int)(gridDim.x >> 3);
    const int e = mt >> 16, m0 = (mt & 0xffff) * BM;
    const int64_t row = (int64_t)g_off[e] + m0;
    t.a = arow ? A : A + row * lda;
    t.w = W + (int64_t)e * w_stride + (int64_t)ni * BN * ldw;
    t.c = (char*)C + (row * ldc + (EPI == EPI_SWIGLU ? ni * BN / 2 : ni * BN)) * esz;
    t.rows = g_cnt[e] - m0;
    t.arow = arow ? arow + row : nullptr;
    return true;
  };
  alt_gemm_items<BM, BN, 2, 4, EPI, false, PW>(lda, ldw, ldc, K / 64, next);
}

// ------------------------------------------- grouped, weights into registers
// Grouped GEMM for decode batches with strip-packed W (the MoE gate/up
// projection).  Block = 4 wavefronts over an item (expert row tile of BM
// rows, slab of 4 x CPW columns); wavefront w owns CPW columns and loads
// their W blocks (one 1 KB block per 16-column strip and 32-wide K step)
// straight from memory into MFMA B-operand registers, P K steps of 64
// ahead (non-temporal loads: each block is read once), so W never passes
// through LDS.  The BM x 64 A tiles of the
// expert's rows (gathered through arow when given; rows past the expert's
// count repeat its last row) go through a P-stage LDS ring shared by the
// four wavefronts, filled by direct 16-byte LDS loads in the swizzled layout
// of the tiled kernel.  Per output tile the MFMAs run over K in order, as in
// the tiled kernel, so results are bitwise those of the tiled kernel.
// Items are dealt XCD by XCD as in the tiled grouped kernel.
template <int BM, int CPW, int P, int EPI>
__global__ void __launch_bounds__(256, 2) gemm_wd_grouped_kernel(
    const bf16_t* __restrict__ A, int lda, const bf16_t* Wp, int64_t w_stride,
    void* __restrict__ C, int ldc, int N, int K, const int32_t* __restrict__ g_off,
    const int32_t* __restrict__ g_cnt, const int32_t* __restrict__ mtiles,
    const int32_t* __restrict__ n_mtiles, const int32_t* __restrict__ arow) {
  constexpr int NW = 4, KB = 64, CH = KB / 8, RPI = 64 / CH;
  constexpr int AI = BM / (RPI * NW);                 // A load instructions per wave per stage
  static_assert(AI * RPI * NW == BM, "A tile rows must split over the waves");
  static_assert(CPW % 32 == 0 || EPI != EPI_SWIGLU, "SwiGLU pairs gate and up strips");
  constexpr int TM = BM / 16, TN = CPW / 16;
  constexpr int WL = 2 * TN;                          // W loads per wave per 64-wide K step
  constexpr int STAGE = BM * KB;
  constexpr int SLAB = NW * CPW;
  constexpr int esz = (EPI == EPI_F32 || EPI == EPI_ADD_F32) ? 4 : 2;
  __shared__ __attribute__((aligned(16))) bf16_t sA[P * STAGE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nt = N / SLAB;
  const int total = n_mtiles[0] * nt;
  const int nk = K / KB;                              // a multiple of P
  const int k32 = K >> 5;
  const int chunk = (total + 7) >> 3;
  const int lo = (int)(blockIdx.x & 7) * chunk;
  const int hi = min(total, lo + chunk);
  const int step = (int)(gridDim.x >> 3);
  const int lrow = lane / CH;
  const int gchunk = (lane % CH) ^ dma_swz<KB>(lrow);
  const int fr = lane & 15, fq = lane >> 4;
  for (int it = lo + (int)(blockIdx.x >> 3); it < hi; it += step) {
    const int mt = mtiles[it / nt], ni = it % nt;
    const int e = mt >> 16, mi = mt & 0xffff;
    const int cnt = g_cnt[e];
    const int64_t off = g_off[e];
    // the previous item's last LDS stage may still be read by other waves
    __builtin_amdgcn_s_barrier();
    const bf16_t* asrc[AI];
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      int r = mi * BM + wave * (BM / NW) + RPI * j + lrow;
      r = r < cnt ? r : cnt - 1;
      const int64_t row = arow ? (int64_t)arow[off + r] : off + r;
      asrc[j] = A + row * lda + gchunk * 8;
    }
    // this wave's first strip; block (strip g0 + j, K step q) at (j*k32 + q)*512
    const int g0 = (ni * SLAB + wave * CPW) >> 4;
    const bf16_t* wsrc = Wp + (int64_t)e * w_stride + (int64_t)g0 * k32 * 512 + lane * 8;
    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    bf16x8_t wr[P][2][TN];   // register ring: slot u holds K step k0 + u
#define DARTS_WD_ISSUE(KT, SLOT)                                                                  \
    {                                                                                            \
      bf16_t* sa_ = sA + (SLOT) * STAGE;                                                         \
      _Pragma("unroll") for (int j = 0; j < AI; ++j)                                             \
        __builtin_amdgcn_global_load_lds((const void*)(asrc[j] + (KT) * KB),                    \
                                         (lds_void_t*)(sa_ + (wave * (BM / NW) + RPI * j) * KB), \
                                         16, 0, 0);                                              \
      _Pragma("unroll") for (int h = 0; h < 2; ++h)                                              \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                           \
          wr[SLOT][h][j] = __builtin_bit_cast(                                                  \
              bf16x8_t, __builtin_nontemporal_load(                                              \
                            (const u32x4_t*)(wsrc + ((int64_t)j * k32 + 2 * (KT) + h) * 512)));  \
    }
#pragma unroll
    for (int u = 0; u < P - 1; ++u)
      if (u < nk) DARTS_WD_ISSUE(u, u)
    for (int k0 = 0; k0 < nk; k0 += P) {
#pragma unroll
      for (int u = 0; u < P; ++u) {
        const int kt = k0 + u;
        // K step kt's A and W loads are done once at most the loads of the
        // (P - 2) later steps are outstanding (whatever the order of the A
        // and W loads inside a step); the raw barrier then publishes every
        // wave's A stage kt, and the scheduling barrier keeps the next
        // step's loads from moving above it
        if (kt + P - 2 < nk) vm_wait<(P - 2) * (AI + WL)>();
        else vm_wait<0>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int kn = kt + P - 1;
        if (kn < nk) DARTS_WD_ISSUE(kn, (u + P - 1) % P)
        const bf16_t* sa = sA + u * STAGE;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          bf16x8_t a[TM];
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            const int r = 16 * i + fr;
            a[i] = *(const bf16x8_t*)(sa + r * KB + (((h * 4 + fq) ^ dma_swz<KB>(r)) * 8));
          }
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], wr[u][h][j], acc[i][j], 0, 0, 0);
        }
      }
    }
#undef DARTS_WD_ISSUE
    void* Ce = (char*)C + off * ldc * esz;
    const int r0 = mi * BM, c0 = ni * SLAB + wave * CPW;
    if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; j += 2)
          store_swiglu((bf16_t*)Ce, ldc, cnt, r0 + 16 * i, c0 + 16 * j, lane, acc[i][j], acc[i][j + 1]);
    } else {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) store_tile<EPI>(Ce, ldc, cnt, r0 + 16 * i, c0 + 16 * j, lane, acc[i][j]);
    }
  }
}

// ----------------------------------------------------------------- skinny
// Block: 8 wavefronts, NS*16 output columns, all M <= 16*MT rows.  Wavefront
// w handles K range [kbeg + w*kw, kbeg + (w+1)*kw).
template <int MT, int NS, int EPI, bool SPLIT>
__global__ void __launch_bounds__(512) gemm_skinny_kernel(const bf16_t* __restrict__ A, int lda,
                                                          const bf16_t* __restrict__ W, int ldw,
                                                          void* __restrict__ C, int ldc, int M,
                                                          int N, int /*K*/, int k_chunk, int nt,
                                                          float* __restrict__ ws) {
  __shared__ f32x4_t red[8][MT * NS][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ni = blockIdx.x % nt, z = blockIdx.x / nt;
  const int n0 = ni * NS * 16;
  const int kw = k_chunk / 8;
  const int kbeg = z * k_chunk + wave * kw;
  const int kq = (lane >> 4) * 8, r = lane & 15;
  f32x4_t acc[MT][NS];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NS; ++j) acc[i][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  const bf16_t* wp[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) wp[j] = W + (int64_t)(n0 + 16 * j + r) * ldw + kbeg + kq;
  const bf16_t* ap[MT];
  bool av[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    av[i] = (16 * i + r) < M;
    ap[i] = A + (int64_t)(av[i] ? 16 * i + r : 0) * lda + kbeg + kq;
  }
  for (int k = 0; k < kw; k += 32) {
    bf16x8_t a[MT], b[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) b[j] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(wp[j] + k));
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      u32x4_t v = *(const u32x4_t*)(ap[i] + k);
      if (!av[i]) v = (u32x4_t){0u, 0u, 0u, 0u};
      a[i] = __builtin_bit_cast(bf16x8_t, v);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NS; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NS; ++j) red[wave][i * NS + j][lane] = acc[i][j];
  __syncthreads();
  // wave t sums tile t (in wave order 0..7) and stores it
  for (int t = wave; t < MT * NS; t += 8) {
    f32x4_t s = red[0][t][lane];
#pragma unroll
    for (int w = 1; w < 8; ++w) s += red[w][t][lane];
    red[0][t][lane] = s;
  }
  __syncthreads();
  if constexpr (SPLIT) {
    float* P = ws + (int64_t)z * M * N;
    for (int t = wave; t < MT * NS; t += 8)
      store_partial(P, M, N, 16 * (t / NS), n0 + 16 * (t % NS), lane, red[0][t][lane]);
  } else if constexpr (EPI == EPI_SWIGLU) {
    for (int t = wave; t < MT * NS / 2; t += 8) {
      const int i = t / (NS / 2), jp = t % (NS / 2);
      store_swiglu((bf16_t*)C, ldc, M, 16 * i, n0 + 32 * jp, lane, red[0][i * NS + 2 * jp][lane],
                   red[0][i * NS + 2 * jp + 1][lane]);
    }
  } else {
    for (int t = wave; t < MT * NS; t += 8)
      store_tile<EPI>(C, ldc, M, 16 * (t / NS), n0 + 16 * (t % NS), lane, red[0][t][lane]);
  }
}

// Sum split-K partials in order z = 0..S-1 and apply the epilogue.
template <int EPI>
__global__ void splitk_reduce_kernel(const float* __restrict__ ws, int S, int M, int N, void* C,
                                     int ldc) {
  // four consecutive output columns per thread (N % 128 == 0 and, for SwiGLU,
  // four consecutive hidden columns stay inside one 16-column gate/up group)
  const int64_t ncol = (EPI == EPI_SWIGLU) ? N / 2 : N;
  const int64_t nout4 = (int64_t)M * ncol / 4;
  const int64_t zs = (int64_t)M * N;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nout4;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int m = (int)(t / (ncol / 4));
    const int c = (int)(t % (ncol / 4)) * 4;
    if constexpr (EPI == EPI_SWIGLU) {
      const int pg = (c >> 4) * 32 + (c & 15), pu = pg + 16;
      float4 g = make_float4(0.f, 0.f, 0.f, 0.f), u = g;
      for (int z = 0; z < S; ++z) {
        const float4 a = *(const float4*)(ws + z * zs + (int64_t)m * N + pg);
        const float4 b = *(const float4*)(ws + z * zs + (int64_t)m * N + pu);
        g.x += a.x; g.y += a.y; g.z += a.z; g.w += a.w;
        u.x += b.x; u.y += b.y; u.z += b.z; u.w += b.w;
      }
      uint2 p;
      p.x = (uint32_t)f32_to_bf16(silu_f(g.x) * u.x) | ((uint32_t)f32_to_bf16(silu_f(g.y) * u.y) << 16);
      p.y = (uint32_t)f32_to_bf16(silu_f(g.z) * u.z) | ((uint32_t)f32_to_bf16(silu_f(g.w) * u.w) << 16);
      *(uint2*)((bf16_t*)C + (int64_t)m * ldc + c) = p;
    } else {
      float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int z = 0; z < S; ++z) {
        const float4 a = *(const float4*)(ws + z * zs + (int64_t)m * N + c);
        s4.x += a.x; s4.y += a.y; s4.z += a.z; s4.w += a.w;
      }
      if constexpr (EPI == EPI_F32) {
        *(float4*)((float*)C + (int64_t)m * ldc + c) = s4;
      } else if constexpr (EPI == EPI_ADD_F32) {
        float4* o = (float4*)((float*)C + (int64_t)m * ldc + c);
        const float4 x = *o;
        *o = make_float4(x.x + s4.x, x.y + s4.y, x.z + s4.z, x.w + s4.w);
      } else {
        uint2 p;
        p.x = (uint32_t)f32_to_bf16(s4.x) | ((uint32_t)f32_to_bf16(s4.y) << 16);
        p.y = (uint32_t)f32_to_bf16(s4.z) | ((uint32_t)f32_to_bf16(s4.w) << 16);
        *(uint2*)((bf16_t*)C + (int64_t)m * ldc + c) = p;
      }
    }
  }
}

// Split-K reduce fused with the residual add and the next RMSNorm: one block
// of 1024 threads per row, one float4 of the row per thread (N % 4 == 0,
// N <= 4096); x[m] += sum_z ws[z][m] in z order (all S partial loads issued
// together), then xn[m] = bf16(x[m] / sqrt(mean(x[m]^2) + eps)).
constexpr int kAddNormMaxN = 4096;
constexpr int kMaxSplits = 8;
__global__ void __launch_bounds__(1024) splitk_add_norm_kernel(const float* __restrict__ ws, int S,
                                                               int M, int N, float* __restrict__ x,
                                                               int ldx, float eps,
                                                               bf16_t* __restrict__ xn) {
  __shared__ float red[16];
  const int m = blockIdx.x, tid = threadIdx.x;
  const int64_t zs = (int64_t)M * N;
  const int c = tid * 4;
  const bool act = c < N;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  if (act) {
    float4 p[kMaxSplits];
#pragma unroll
    for (int z = 0; z < kMaxSplits; ++z)
      p[z] = z < S ? *(const float4*)(ws + z * zs + (int64_t)m * N + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    a = *(const float4*)(x + (int64_t)m * ldx + c);
#pragma unroll
    for (int z = 0; z < kMaxSplits; ++z) {
      a.x += p[z].x; a.y += p[z].y; a.z += p[z].z; a.w += p[z].w;
    }
    *(float4*)(x + (int64_t)m * ldx + c) = a;
  }
  float ss = a.x * a.x;
  ss = fmaf(a.y, a.y, ss);
  ss = fmaf(a.z, a.z, ss);
  ss = fmaf(a.w, a.w, ss);
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / (float)N + eps);
  if (act) {
    uint2 q;
    q.x = (uint32_t)f32_to_bf16(a.x * inv) | ((uint32_t)f32_to_bf16(a.y * inv) << 16);
    q.y = (uint32_t)f32_to_bf16(a.z * inv) | ((uint32_t)f32_to_bf16(a.w * inv) << 16);
    *(uint2*)(xn + (int64_t)m * N + c) = q;
  }
}

// fp32 GEMM (fp32 models) on v_mfma_f32_16x16x4_f32, whose products and sums
// are fp32: a 16x16 output tile per block of 8 wavefronts (for SwiGLU the gate
// tile and the up tile of 16 features), which split K and are added in
// wavefront order.  Lane (r, q) loads four consecutive K of its row at once;
// MFMA i of the four takes element i of both operands, so K runs 4q + i.  Any M,
// N, K; VEC: K, lda and ldw are multiples of 4 and A and W 16-byte aligned.
//
// These launches are latency: the tiny model's down projection (32 x 128, K 512)
// took 11.8 us with an LDS tile and a barrier pair per 16 of K and takes 4.8, its
// SwiGLU projection (32 x 1024, K 128) 34 us with a thread per output and 3.7.
constexpr int kF32Waves = 8;
template <bool VEC>
__device__ __forceinline__ float4 load_k4(const float* row, int k, int K) {
  if constexpr (VEC) return k < K ? *(const float4*)(row + k) : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 v;
  v.x = k < K ? row[k] : 0.f;
  v.y = k + 1 < K ? row[k + 1] : 0.f;
  v.z = k + 2 < K ? row[k + 2] : 0.f;
  v.w = k + 3 < K ? row[k + 3] : 0.f;
  return v;
}
template <int EPI, bool VEC>
__global__ void __launch_bounds__(64 * kF32Waves) gemm_f32_kernel(const float* __restrict__ A, int lda,
                                                                  const float* __restrict__ W, int ldw, float* C,
                                                                  int ldc, int M, int N, int K) {
  constexpr int NT = EPI == EPI_SWIGLU ? 2 : 1;
  __shared__ f32x4_t red[kF32Waves][NT][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;     // first row and output column
  const float* a = A + (int64_t)min(m0 + r, M - 1) * lda;
  const float* b[NT];
  // SwiGLU: features n0 .. n0+15 are W rows 2*n0 .. (gate) and the 16 after them (up)
#pragma unroll
  for (int t = 0; t < NT; ++t) b[t] = W + (int64_t)min((EPI == EPI_SWIGLU ? 2 * n0 + 16 * t : n0) + r, N - 1) * ldw;
  f32x4_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  const int kw = (K + 16 * kF32Waves - 1) / (16 * kF32Waves) * 16, kend = min(K, (w + 1) * kw);
#pragma unroll 4
  for (int k = w * kw; k < kend; k += 16) {
    const float4 x = load_k4<VEC>(a, k + 4 * q, K);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const float4 y = load_k4<VEC>(b[t], k + 4 * q, K);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.y, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, y.z, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, y.w, acc[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) red[w][t][lane] = acc[t];
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    acc[t] = red[0][t][lane];
#pragma unroll
    for (int i = 1; i < kF32Waves; ++i) acc[t] += red[i][t][lane];
  }
  // lane holds rows 4q + i of column r
  const int n = n0 + r, ncol = EPI == EPI_SWIGLU ? N / 2 : N;
  if (n >= ncol) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + 4 * q + i;
    if (m >= M) break;
    float* c = C + (int64_t)m * ldc + n;
    if (EPI == EPI_SWIGLU) *c = silu_f(acc[0][i]) * acc[NT - 1][i];
    else if (EPI == EPI_ADD_F32) *c += acc[0][i];
    else *c = acc[0][i];
  }
}

// ------------------------------------------------------------ dispatch
struct Plan {
  int kind;        // 0 skinny; tiled: 1 = 128x128 4 stages, 2 = 128x128 2 stages,
                   // 3 = 256x128, 4 = 256x256, 5 = 256x192, alternating groups
                   // (plan_alternates says when not),
                   // exact-fill tiles with 4 stages and 4 waves: 6 = 128x96 (4x1),
                   // 7 = 128x64 (4x1), 8 = 64x64 (2x2), 9 = 64x96 (4x1)
  int mt, nt, S;   // tiles and K splits
  int MT, NS;      // skinny shape
  bool nt_w;       // weights loaded non-temporal (tiled kernels; set per call, see stream_weights)
};

// Planning assumes MI355X's 256 CUs whatever device runs the call, so a
// shape always gets the same plan (and the same summation order).
static constexpr int kCus = 256;

static void set_tiled(Plan& p, int kind, int bm, int bn, int M, int N, int S) {
  p.kind = kind; p.mt = (M + bm - 1) / bm; p.nt = N / bn; p.S = S;
}

// Tiled configs with the throughput model fitted to MI355X timings of every
// projection of the supported models (M = 1..512, weights streamed from HBM,
// not cache-resident): per-CU MFMA rate of one block (TFLOP/s), the weight
// streaming rate (GB/s) and blocks resident per CU.
struct TileCfg {
  int kind, bm, bn, occ;
  double rate, bw;
};
// The 256x192 tile (4 x 2 wavefronts of 64 x 96) fills all 256 CUs at
// M in (256, 512] for the gate/up projection of the 8B shape (N = 128 * 192).
// The rates of the 256-row tiles were fitted to the tiled kernel; with the
// alternating groups the plans they give are still within 2.2% of the fastest
// forced plan on average (150 cases of the projections from 140 to 8192 rows),
// and rates fitted again within 1.4%.
static const TileCfg kTileCfgs[5] = {
    {1, 128, 128, 1, 3.38, 6425.0},
    {2, 128, 128, 2, 2.26, 6423.0},
    {3, 256, 128, 1, 4.89, 6325.0},
    {4, 256, 256, 1, 6.68, 6298.0},
    {5, 256, 192, 1, 5.84, 6298.0},
};
static constexpr double kOcc2Gain = 1.76;   // CU throughput with two co-resident blocks / one block
static constexpr double kLaunchUs = 0.16;
static constexpr double kSplitGBs = 4106.0;  // partial sums: written once, read once by the reduce
static constexpr double kReduceUs = 3.19;

// Estimated time (us): rounds of resident blocks at the config's rate, at
// least the weight bytes at its streaming rate, plus the K-split partial-sum
// round trip and reduce launch.
static double tile_estimate(const TileCfg& c, int S, int M, int N, int K) {
  const int mt = (M + c.bm - 1) / c.bm, nt = N / c.bn;
  const double blocks = (double)mt * nt * S;
  const double mflop = 2.0 * c.bm * c.bn * ((double)K / S) * 1e-6;
  double t;
  if (blocks <= kCus) t = mflop / c.rate;
  else {
    const double rounds = std::ceil(blocks / (c.occ * kCus));
    t = rounds * c.occ * mflop / (c.occ == 2 ? c.rate * kOcc2Gain : c.rate);
  }
  t = std::max(t, 2.0 * N * (double)K / (c.bw * 1e3)) + kLaunchUs;
  if (S > 1) t += 2.0 * S * (double)M * N * 4.0 / (kSplitGBs * 1e3) + kReduceUs;
  return t;
}

// Small batches stream the weights once: what matters is that every CU
// streams an equal share.  Up to 128 rows, a tile of the batch's height
// (64 or 128 rows) and a K split whose block count is exactly one per CU is
// used when one exists (fewest splits, then the wider tile; a 64-column tile
// with 128 rows only for blocks of at most 1024 of K, where the 128x128
// tile's better reuse does not pay).  Measured on the Qwen3-8B projections
// (cache-cold weights), 8-20% faster than the best of the other configs up
// to 64 rows and up to 12% up to 128.
static bool exact_fill_plan(int M, int N, int K, Plan& p) {
  if (M > 128) return false;
  struct T { int kind, bm, bn; };
  static const T small[2] = {{9, 64, 96}, {8, 64, 64}};
  static const T mid[2] = {{6, 128, 96}, {7, 128, 64}};
  const T* cand = M <= 64 ? small : mid;
  for (int S = 1; S <= 8; S *= 2) {
    if (K % (S * 256) != 0 || K / S < 256) break;
    for (int i = 0; i < 2; ++i) {
      const T& t = cand[i];
      if (N % t.bn != 0 || (N / t.bn) * S != kCus) continue;
      if (M > 64 && t.bn == 64 && K / S > 1024) continue;
      set_tiled(p, t.kind, t.bm, t.bn, M, N, S);
      return true;
    }
  }
  return false;
}

//  * up to 128 rows: the exact-fill tile when one exists;
//  * M <= 32 with W up to 40 MB (and K <= 2048 beyond 16 rows): skinny;
//  * otherwise the tiled config and K split with the least estimated time
//    (256-row tiles only above 128 rows).
static Plan plan_gemm(int M, int N, int K) {
  Plan p{};
  if (exact_fill_plan(M, N, K, p)) return p;
  const double wbytes = 2.0 * N * K;
  if (M <= 32 && wbytes <= 40e6 && (M <= 16 || K <= 2048) && N % 32 == 0) {
    p.kind = 0;
    p.MT = (M + 15) / 16;
    p.NS = (M <= 16) ? 2 : 4;
    if (N % (p.NS * 16) != 0) p.NS = 2;
    p.nt = N / (p.NS * 16);
    p.mt = 1;
    // split K across blocks until there are ~2 blocks per CU (each wave keeps >= 256 of K)
    p.S = 1;
    while (p.nt * p.S < 2 * kCus && K % (p.S * 2 * 8 * 32) == 0 && K / (p.S * 2) >= 8 * 256) p.S *= 2;
    return p;
  }
  double best = 1e30;
  for (const TileCfg& c : kTileCfgs) {
    if (N % c.bn != 0 || (c.bm > 128 && M <= 128)) continue;
    for (int S = 1; S <= 8; S *= 2) {
      if (K % (S * 256) != 0 || K / S < 256) break;
      const double t = tile_estimate(c, S, M, N, K);
      if (t < best) { best = t; set_tiled(p, c.kind, c.bm, c.bn, M, N, S); }
    }
  }
  return p;
}

// Non-temporal weight loads: for weights that one row tile reads once and that
// no cache holds when they come round again.  pass_bytes are what the caller
// reads between two uses of W (0: unknown, W itself may come next), and the
// Infinity Cache is 256 MiB.  Measured, default policy against non-temporal:
// read again at once, 8B gate/up (201 MB) at 45 rows 31.4 against 39.4 us, down
// (101 MB) 20.0 against 22.4, 268 MB 43.3 against 57; from 302 MB on, non-temporal
// is ahead either way (302 MB 76.3 / 75.2, 403 MB 91.4 / 78.8).  Behind other
// weights (a decoder's pass) it gains 2-10% from 64 MB on up to 48 rows (down at
// 45 rows 24.7 / 23.4), and up to 128 rows between 128 and 450 MB (gate/up at 128
// rows 2%, 134 MB 5%, 403 MB 8%); below and above that more rows lose (67 MB at 100
// rows 20.9 / 23.8, LM head of the 8B shape at 100 rows 258 / 268).
constexpr double kNtWeightBytes = 64e6, kNtPassBytes = 300e6, kNtMidFrom = 128e6, kNtMidTo = 450e6;
constexpr int kNtRows = 48, kNtMidRows = 128;
static bool stream_weights(int M, int N, int K, double pass_bytes) {
  const double w = 2.0 * N * K;
  return M <= (w >= kNtMidFrom && w <= kNtMidTo ? kNtMidRows : kNtRows) && w >= kNtWeightBytes &&
         std::max(w, pass_bytes) >= kNtPassBytes;
}

size_t gemm_workspace_bytes(int M, int N, int K) {
  const Plan p = plan_gemm(M, N, K);
  return p.S > 1 ? (size_t)p.S * M * N * sizeof(float) : 0;
}

template <int EPI>
static hipError_t reduce_launch(const void* ws, int S, int M, int N, void* C, int ldc,
                                hipStream_t st) {
  const int64_t nout = ((EPI == EPI_SWIGLU) ? (int64_t)M * (N / 2) : (int64_t)M * N) / 4;
  int64_t blocks = (nout + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(splitk_reduce_kernel<EPI>, dim3((unsigned)blocks), dim3(256), 0, st,
                     (const float*)ws, S, M, N, C, ldc);
  return hipGetLastError();
}

template <int EPI, int MT, int NS>
static void skinny_go(const Plan& p, const void* A, int lda, const void* W, int ldw, void* C,
                      int ldc, int M, int N, int K, void* ws, hipStream_t st) {
  const dim3 grid(p.nt * p.S), blk(512);
  if (p.S == 1)
    hipLaunchKernelGGL((gemm_skinny_kernel<MT, NS, EPI, false>), grid, blk, 0, st, (const bf16_t*)A,
                       lda, (const bf16_t*)W, ldw, C, ldc, M, N, K, K, p.nt, (float*)nullptr);
  else
    hipLaunchKernelGGL((gemm_skinny_kernel<MT, NS, EPI, true>), grid, blk, 0, st, (const bf16_t*)A,
                       lda, (const bf16_t*)W, ldw, C, ldc, M, N, K, K / p.S, p.nt, (float*)ws);
}

template <int EPI, int BM_, int BN_, int KB, int WGM, int WGN, int ST, bool SPLIT, int WAUX>
static void dma_go_as(const Plan& p, const void* A, int lda, const void* W, int ldw, void* C, int ldc,
                      int M, int N, int K, void* ws, hipStream_t st) {
  const dim3 grid(p.mt * p.nt * p.S), blk(64 * WGM * WGN);
  const size_t lds = (size_t)ST * (BM_ + BN_) * KB * sizeof(bf16_t);
  static bool attr_done = false;
  auto kern = gemm_dma_kernel<BM_, BN_, KB, WGM, WGN, ST, EPI, SPLIT, WAUX>;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_done = true;
  }
  hipLaunchKernelGGL(kern, grid, blk, lds, st, (const bf16_t*)A, lda, (const bf16_t*)W, ldw, C, ldc, M, N, K,
                     K / p.S, p.mt, p.nt, (float*)ws);
}
template <int EPI, int BM_, int BN_, int KB, int WGM, int WGN, int ST>
static void dma_go(const Plan& p, const void* A, int lda, const void* W, int ldw, void* C, int ldc,
                   int M, int N, int K, void* ws, hipStream_t st) {
  if (p.S == 1) {
    if (p.nt_w) dma_go_as<EPI, BM_, BN_, KB, WGM, WGN, ST, false, kNtLoad>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
    else dma_go_as<EPI, BM_, BN_, KB, WGM, WGN, ST, false, 0>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
  } else {
    if (p.nt_w) dma_go_as<EPI, BM_, BN_, KB, WGM, WGN, ST, true, kNtLoad>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
    else dma_go_as<EPI, BM_, BN_, KB, WGM, WGN, ST, true, 0>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
  }
}

// The ring kernel with a large tile of the alternating groups, where those don't
// run (plan_alternates).
template <int EPI, int BM_, int BN_, int WGM, int WGN>
static void dma_far(const Plan& p, const void* A, int lda, const void* W, int ldw, void* C, int ldc, int M, int N,
                    int K, void* ws, hipStream_t st) {
  if (p.S == 1) dma_go_as<EPI, BM_, BN_, 64, WGM, WGN, 2, false, 0>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
  else dma_go_as<EPI, BM_, BN_, 64, WGM, WGN, 2, true, 0>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
}

// The alternating groups address a tile's rows of A, W and C by 32-bit byte
// offsets from its first row, so 256 rows of each have to lie within 2 GiB.
// Longer rows (fp32 results of 2^21 columns and more, K of 2^22 and more) take
// the ring kernel with the same tile: its addresses are 64-bit, the plan and
// its workspace stay valid.
static bool alt_reaches(int64_t lda, int64_t ldw, int64_t ldc, int esz) {
  return 256 * std::max(2 * std::max(lda, ldw), esz * ldc) < ((int64_t)1 << 31);
}
// Whether plan p runs on the alternating groups.  Whole K mostly does; a split keeps the
// ring kernel where it streams weights more than it computes (weights cold, ring
// against alternating):
//  * K ranges below 2048, but for 256x256 tiles of several row tiles: 12288 x 5120
//    in 4 splits at 129-200 rows 42-49 / 48-55 us; QKV of the 8B shape
//    in 4 splits at 256 rows 27.9 / 29.3, at 280 rows 34.4 / 38.4, at 340-400 rows
//    38-40 / 38-40; 5120 x 12288 in 8 at 129-200 rows 49.5-54 / 51-57.  (256x256
//    over two row tiles: down of the 8B shape in 8 splits at 300 rows 61 / 57.)
//  * one row tile of weights on every CU: gate/up of the 8B shape in 2 splits at
//    129-156 rows 63-66 / 69.  (On 192 CUs, 18432 x 4096, 55-61 / 51-57.)
// Longer ranges alternate: 4096 x 12288 in 4 splits at 347-512 rows 62-65 / 56-65,
// at 600-1000 rows 92-116 / 82-98; 8192 x 8192 in 2 at 640 rows 121 / 97.
// Plain fp32 results of a short K are bound by their stores, which the blocks of
// the ring kernel overlap better: K below 1024 (20480 x 512 at 129-256 rows 11.7-13.6
// / 11.9-15.5, at 3000 rows 89 / 100; 16384 x 256 at 600 rows 14.5 / 17.2), below
// 2048 up to 11 row tiles (151936 x 1024 at 256 rows 108 / 117; 1536 x 1024 at 3000
// rows, 12 row tiles, 19.6 / 19.1), and 256x128 tiles of one row tile below K 3072
// (151936 x 2048 at 183-256 rows 188-198 / 189-206; K 4096 349-355 / 320-342).
static bool plan_alternates(const Plan& p, int lda, int ldw, int ldc, int N, int K, int epi) {
  if (p.kind < 3 || p.kind > 5) return false;
  if (p.S == 1) {
    if (epi == EPI_F32 && (K < 2048 ? K < 1024 || p.mt < 12 : K < 3072 && p.mt == 1 && p.kind == 3))
      return false;
    return alt_reaches(lda, ldw, ldc, epi == EPI_BF16 || epi == EPI_SWIGLU ? 2 : 4);
  }
  if (K / p.S < 2048 && (p.kind != 4 || p.mt == 1)) return false;
  if (K / p.S < 4096 && p.mt == 1 && p.nt * p.S >= kCus) return false;
  return alt_reaches(lda, ldw, N, 4);
}

void gemm_plan_info(int M, int N, int K, int epi, int32_t* out) {
  const Plan p = plan_gemm(M, N, K);
  const int32_t v[6] = {p.kind, p.mt, p.nt, p.S, plan_alternates(p, K, K, epi == EPI_SWIGLU ? N / 2 : N, N, K, epi),
                        p.kind > 0 && stream_weights(M, N, K, 0.0)};
  std::copy(v, v + 6, out);
}

template <int EPI, int BM, int BN, int WGM, int WGN>
static void alt_go(const Plan& p, const void* A, int lda, const void* W, int ldw, void* C, int ldc, int M,
                   int N, int K, void* ws, hipStream_t st) {
  // a multiple of 8 blocks, at most one per CU
  const dim3 grid(std::min((p.mt * p.nt * p.S + 7) / 8 * 8, kCus)), blk(512);
  constexpr int lds = 2 * (BM + BN) * 64 * (int)sizeof(bf16_t);
  static bool attr_done[2] = {false, false};
  auto whole = gemm_alt_kernel<BM, BN, WGM, WGN, EPI, false>;
  auto split = gemm_alt_kernel<BM, BN, WGM, WGN, EPI, true>;
  auto kern = p.S == 1 ? whole : split;
  if (!attr_done[p.S > 1]) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    attr_done[p.S > 1] = true;
  }
  hipLaunchKernelGGL(kern, grid, blk, lds, st, (const bf16_t*)A, lda, (const bf16_t*)W, ldw, C,
                     p.S == 1 ? ldc : N, M, N, K / p.S, p.mt, p.nt, p.S, (float*)ws);
}

GroupedPlan grouped_plan(int64_t n_pairs, int E, bool gate_up, int64_t gathered_bytes) {
  if (n_pairs > (int64_t)96 * E)
    return {gathered_bytes < ((int64_t)1 << 32) ? kGroupedTileRows : kGroupedTileRowsFar, false, false};
  if (!gate_up) return {kGroupedTileRowsMin, false, n_pairs <= (int64_t)48 * E};
  if (n_pairs > (int64_t)48 * E) return {kGroupedTileRowsGU, true, true};
  return {kGroupedTileRowsMin, n_pairs >= (int64_t)2 * E, true};
}

hipError_t launch_pack_strips(void* W, int64_t rows, int K, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (rows % 16 || K % 32 || K < 32 || (size_t)16 * K * 2 > 160 * 1024 || rows / 16 > INT32_MAX)
    return hipErrorInvalidValue;
  const size_t lds = (size_t)16 * K * sizeof(bf16_t);
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)pack_strips_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024);
    attr_done = true;
  }
  hipLaunchKernelGGL(pack_strips_kernel, dim3((unsigned)(rows / 16)), dim3(256), lds, st, (bf16_t*)W, K);
  return hipGetLastError();
}

// Persistent blocks over (row tile, n tile) items.  Large batches (above 96 rows
// per expert: the prefill): 256x256 tiles of the alternating groups; gathered
// rows beyond 32-bit offsets: 128x128 with a 4-stage ring, one block per CU.
// Measured at 32768 rows of the Qwen3-30B-A3B experts, 256-row against 128-row
// tiles: gate/up 1395 against 2450 us, down 904 against 1605 us; from 97 rows per
// expert: see GroupedPlan.  64-row tiles
// (decode batches, where the expert weights are streamed): two blocks per
// CU, so one block's loads stream while the other waits at its barrier or
// refills its ring at an item boundary; 64x64 tiles with a 4-stage ring for
// the gate/up projection (K = d), 64x128 tiles with a 3-stage ring for the
// down projection (K = expert FFN).  Measured on the Qwen3-30B-A3B expert
// shapes from 1 to 1024 rows against one block per CU with 64x128 tiles and
// a 6-stage ring: 6-18% faster for gate/up, 10-18% for down.  96-row tiles:
// 96x128 with a 3-stage ring, one block per CU.  At 64 rows per expert about
// half the experts exceed 64 rows, and a 64-row tile list streams their
// weights twice; the 96-row tile streams them once (171-180 us per launch at
// 1024 rows against 222 us).  The gate/up plan now runs its 96-row (and most
// of its 64-row) tiles on the weights-into-registers kernel below, which is
// faster still; the down projection gains nothing from 96-row tiles (its
// second pass mostly hits in cache) and keeps 64-row tiles up to 96 rows per
// expert.
template <int BM_, int ST, int EPI, int BN_, int BPC, bool PW, int WAUX>
static hipError_t grouped_launch(const void* A, int lda, const void* W, int64_t w_stride, int ldw,
                                 void* C, int ldc, int N, int K, const int32_t* g_off,
                                 const int32_t* g_cnt, const int32_t* mtiles,
                                 const int32_t* n_mtiles, const int32_t* arow, hipStream_t st) {
  constexpr int KB = 64;
  if (N % BN_ != 0) return hipErrorInvalidValue;
  if (PW && (ldw != K || K % 32 != 0)) return hipErrorInvalidValue;
  const int nt = N / BN_;
  const size_t lds = (size_t)ST * (BM_ + BN_) * KB * sizeof(bf16_t);
  auto kern = gemm_dma_grouped_kernel<BM_, BN_, KB, 2, 2, ST, EPI, PW, WAUX>;
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_done = true;
  }
  static_assert((kCus * BPC) % 8 == 0, "the grouped kernel deals items to 8 XCDs");
  hipLaunchKernelGGL(kern, dim3(kCus * BPC), dim3(256), lds, st, (const bf16_t*)A, lda, (const bf16_t*)W,
                     w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, nt, arow);
  return hipGetLastError();
}

template <int EPI, bool PW>
static hipError_t alt_grouped_launch(const void* A, int lda, const void* W, int64_t w_stride, int ldw, void* C,
                                     int ldc, int N, int K, const int32_t* g_off, const int32_t* g_cnt,
                                     const int32_t* mtiles, const int32_t* n_mtiles, const int32_t* arow,
                                     hipStream_t st) {
  if (N % 256 != 0 || K % 128 != 0 || (PW && ldw != K)) return hipErrorInvalidValue;
  constexpr int lds = 2 * 512 * 64 * (int)sizeof(bf16_t);
  auto kern = gemm_alt_grouped_kernel<EPI, PW>;
  static bool attr_done = false;
  if (!attr_done) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    attr_done = true;
  }
  static_assert(kCus % 8 == 0, "the grouped kernel deals items to 8 XCDs");
  hipLaunchKernelGGL(kern, dim3(kCus), dim3(512), lds, st, (const bf16_t*)A, lda, (const bf16_t*)W, w_stride, ldw,
                     C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, N / 256, arow);
  return hipGetLastError();
}

template <int EPI, bool PW, int WAUX>
static hipError_t grouped_by_rows_aux(int tile_rows, const void* A, int lda, const void* W, int64_t w_stride,
                                      int ldw, void* C, int ldc, int N, int K, const int32_t* g_off,
                                      const int32_t* g_cnt, const int32_t* mtiles, const int32_t* n_mtiles,
                                      const int32_t* arow, hipStream_t st) {
  if (tile_rows == kGroupedTileRowsMin) {
    if constexpr (EPI == EPI_SWIGLU)
      return grouped_launch<kGroupedTileRowsMin, 4, EPI, 64, 2, PW, WAUX>(A, lda, W, w_stride, ldw, C, ldc, N, K,
                                                                          g_off, g_cnt, mtiles, n_mtiles, arow, st);
    else
      return grouped_launch<kGroupedTileRowsMin, 3, EPI, 128, 2, PW, WAUX>(A, lda, W, w_stride, ldw, C, ldc, N, K,
                                                                           g_off, g_cnt, mtiles, n_mtiles, arow, st);
  }
  if (tile_rows == kGroupedTileRowsGU)
    return grouped_launch<kGroupedTileRowsGU, 3, EPI, 128, 1, PW, WAUX>(A, lda, W, w_stride, ldw, C, ldc, N, K,
                                                                        g_off, g_cnt, mtiles, n_mtiles, arow, st);
  if (tile_rows == kGroupedTileRows)
    return alt_grouped_launch<EPI, PW>(A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, arow,
                                       st);
  if (tile_rows == kGroupedTileRowsFar)
    return grouped_launch<kGroupedTileRowsFar, 4, EPI, 128, 1, PW, WAUX>(A, lda, W, w_stride, ldw, C, ldc, N, K,
                                                                      g_off, g_cnt, mtiles, n_mtiles, arow, st);
  return hipErrorInvalidValue;
}

template <int EPI, bool PW>
static hipError_t grouped_by_rows(int tile_rows, bool nt_w, const void* A, int lda, const void* W,
                                  int64_t w_stride, int ldw, void* C, int ldc, int N, int K,
                                  const int32_t* g_off, const int32_t* g_cnt, const int32_t* mtiles,
                                  const int32_t* n_mtiles, const int32_t* arow, hipStream_t st) {
  return nt_w ? grouped_by_rows_aux<EPI, PW, kNtLoad>(tile_rows, A, lda, W, w_stride, ldw, C, ldc, N, K, g_off,
                                                      g_cnt, mtiles, n_mtiles, arow, st)
              : grouped_by_rows_aux<EPI, PW, 0>(tile_rows, A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt,
                                                mtiles, n_mtiles, arow, st);
}

// Weights into registers: 32 columns per wavefront (a 128-column slab per
// block), a 2-step register ring and 2-stage A ring, two blocks per CU.
// Measured against the tiled kernel on the Qwen3-30B-A3B gate/up shape
// (random routings, weights cache-cold, outputs bitwise equal), per launch:
// 96-row tiles 154 against 178 us at 1024 rows and 147 against 170 us at
// 768; 64-row tiles 139 against 150 us at 512, 132 against 138 at 256,
// 128 against 132 at 64 and 86 against 88 at 16; below 2 rows per expert
// (8 live rows) the tiled kernel is faster (67 against 73 us).
template <int BM>
static hipError_t wd_launch(const void* A, int lda, const void* W, int64_t w_stride, int ldw, void* C, int ldc,
                            int N, int K, const int32_t* g_off, const int32_t* g_cnt, const int32_t* mtiles,
                            const int32_t* n_mtiles, const int32_t* arow, hipStream_t st) {
  constexpr int CPW = 32, P = 2, BPC = 2;
  if (N % (4 * CPW) != 0 || ldw != K || (K / 64) % P != 0) return hipErrorInvalidValue;
  static_assert((kCus * BPC) % 8 == 0, "the grouped kernel deals items to 8 XCDs");
  hipLaunchKernelGGL((gemm_wd_grouped_kernel<BM, CPW, P, EPI_SWIGLU>), dim3(kCus * BPC), dim3(256), 0, st,
                     (const bf16_t*)A, lda, (const bf16_t*)W, w_stride, C, ldc, N, K, g_off, g_cnt, mtiles,
                     n_mtiles, arow);
  return hipGetLastError();
}

hipError_t launch_gemm_grouped(const void* A, int lda, const void* W, int64_t w_stride, int ldw,
                               void* C, int ldc, int N, int K, int epi, const int32_t* g_off,
                               const int32_t* g_cnt, const int32_t* mtiles, const int32_t* n_mtiles,
                               const int32_t* arow, GroupedPlan plan, bool packed_w, hipStream_t st) {
  if (N % 128 != 0 || K % 64 != 0 || K < 64) return hipErrorInvalidValue;
  const int tile_rows = plan.tile_rows;
  if (packed_w) {
    // strip-packed weights: the gate/up projection
    if (epi != EPI_SWIGLU) return hipErrorInvalidValue;
    if (plan.wdirect) {
      if (tile_rows == kGroupedTileRowsMin)
        return wd_launch<kGroupedTileRowsMin>(A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles,
                                              n_mtiles, arow, st);
      if (tile_rows == kGroupedTileRowsGU)
        return wd_launch<kGroupedTileRowsGU>(A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles,
                                             n_mtiles, arow, st);
      return hipErrorInvalidValue;
    }
    return grouped_by_rows<EPI_SWIGLU, true>(tile_rows, plan.nt_w, A, lda, W, w_stride, ldw, C, ldc, N, K,
                                             g_off, g_cnt, mtiles, n_mtiles, arow, st);
  }
  if (plan.wdirect) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_F32: return grouped_by_rows<EPI_F32, false>(tile_rows, plan.nt_w, A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, arow, st);
    case EPI_BF16: return grouped_by_rows<EPI_BF16, false>(tile_rows, plan.nt_w, A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, arow, st);
    case EPI_ADD_F32: return grouped_by_rows<EPI_ADD_F32, false>(tile_rows, plan.nt_w, A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, arow, st);
    case EPI_SWIGLU: return grouped_by_rows<EPI_SWIGLU, false>(tile_rows, plan.nt_w, A, lda, W, w_stride, ldw, C, ldc, N, K, g_off, g_cnt, mtiles, n_mtiles, arow, st);
    default: return hipErrorInvalidValue;
  }
}

// Launch the GEMM kernel of plan p (partial sums into ws when p.S > 1).
template <int EPI>
static hipError_t launch_plan(const Plan& p, const void* A, int lda, const void* W, int ldw, void* C,
                              int ldc, int M, int N, int K, void* ws, hipStream_t st) {
  if (p.kind == 0) {
    if (p.NS == 2) {
      switch (p.MT) {
        case 1: skinny_go<EPI, 1, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
        case 2: skinny_go<EPI, 2, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
        case 3: skinny_go<EPI, 3, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
        default: skinny_go<EPI, 4, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      }
    } else {
      switch (p.MT) {
        case 1: skinny_go<EPI, 1, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
        case 2: skinny_go<EPI, 2, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
        case 3: skinny_go<EPI, 3, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
        default: skinny_go<EPI, 4, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      }
    }
  } else {
    const bool alt = plan_alternates(p, lda, ldw, ldc, N, K, EPI);
    switch (p.kind) {
      case 1: dma_go<EPI, 128, 128, 64, 2, 2, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      case 2: dma_go<EPI, 128, 128, 64, 2, 2, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      case 3:
        if (alt) alt_go<EPI, 256, 128, 4, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
        else dma_go<EPI, 256, 128, 64, 4, 2, 3>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
        break;
      case 4:
        if (alt) alt_go<EPI, 256, 256, 2, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
        else dma_far<EPI, 256, 256, 2, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
        break;
      case 5:
        if (alt) alt_go<EPI, 256, 192, 4, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
        else dma_far<EPI, 256, 192, 4, 2>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
        break;
      case 6: dma_go<EPI, 128, 96, 64, 4, 1, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      case 7: dma_go<EPI, 128, 64, 64, 4, 1, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      case 8: dma_go<EPI, 64, 64, 64, 2, 2, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
      default: dma_go<EPI, 64, 96, 64, 4, 1, 4>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st); break;
    }
  }
  return hipGetLastError();
}

template <int EPI>
static hipError_t gemm_bf16_launch(const void* A, int lda, const void* W, int ldw, void* C, int ldc,
                                   int M, int N, int K, void* ws, size_t ws_bytes, hipStream_t st,
                                   double pass_bytes) {
  Plan p = plan_gemm(M, N, K);
  p.nt_w = stream_weights(M, N, K, pass_bytes);
  if (p.S > 1 && (ws == nullptr || ws_bytes < (size_t)p.S * M * N * sizeof(float)))
    return hipErrorInvalidValue;
  hipError_t e = launch_plan<EPI>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
  if (e != hipSuccess || p.S == 1) return e;
  return reduce_launch<EPI>(ws, p.S, M, N, C, ldc, st);
}

template <int EPI>
static hipError_t gemm_f32_launch(const void* A, int lda, const void* W, int ldw, void* C, int ldc,
                                  int M, int N, int K, hipStream_t st) {
  const int ncol = EPI == EPI_SWIGLU ? N / 2 : N;
  const bool vec = K % 4 == 0 && lda % 4 == 0 && ldw % 4 == 0 && ((uintptr_t)A | (uintptr_t)W) % 16 == 0;
  // rows of more than 65535 tiles go in several launches (the grid's y limit)
  for (int64_t m = 0; m < M; m += 65535 * 16) {
    const int rows = (int)std::min<int64_t>(M - m, 65535 * 16);
    const dim3 grid((ncol + 15) / 16, (rows + 15) / 16);
    const float* a = (const float*)A + m * lda;
    float* c = (float*)C + m * ldc;
    if (vec)
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, true>), grid, dim3(64 * kF32Waves), 0, st, a, lda, (const float*)W, ldw,
                         c, ldc, rows, N, K);
    else
      hipLaunchKernelGGL((gemm_f32_kernel<EPI, false>), grid, dim3(64 * kF32Waves), 0, st, a, lda, (const float*)W,
                         ldw, c, ldc, rows, N, K);
  }
  return hipGetLastError();
}

hipError_t launch_gemm(bool bf16, const void* A, int lda, const void* W, int ldw, void* C, int ldc,
                       int M, int N, int K, int epi, void* ws, size_t ws_bytes, hipStream_t st,
                       double pass_bytes) {
  if (M <= 0) return hipSuccess;
  if (!bf16) {
    switch (epi) {
      case EPI_F32: return gemm_f32_launch<EPI_F32>(A, lda, W, ldw, C, ldc, M, N, K, st);
      case EPI_BF16: return gemm_f32_launch<EPI_F32>(A, lda, W, ldw, C, ldc, M, N, K, st);
      case EPI_ADD_F32: return gemm_f32_launch<EPI_ADD_F32>(A, lda, W, ldw, C, ldc, M, N, K, st);
      case EPI_SWIGLU: return gemm_f32_launch<EPI_SWIGLU>(A, lda, W, ldw, C, ldc, M, N, K, st);
    }
    return hipErrorInvalidValue;
  }
  if (N % 128 != 0 || K % 256 != 0) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_F32: return gemm_bf16_launch<EPI_F32>(A, lda, W, ldw, C, ldc, M, N, K, ws, ws_bytes, st, pass_bytes);
    case EPI_BF16: return gemm_bf16_launch<EPI_BF16>(A, lda, W, ldw, C, ldc, M, N, K, ws, ws_bytes, st, pass_bytes);
    case EPI_ADD_F32:
      return gemm_bf16_launch<EPI_ADD_F32>(A, lda, W, ldw, C, ldc, M, N, K, ws, ws_bytes, st, pass_bytes);
    case EPI_SWIGLU:
      return gemm_bf16_launch<EPI_SWIGLU>(A, lda, W, ldw, C, ldc, M, N, K, ws, ws_bytes, st, pass_bytes);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_f32_or_partials(const void* A, int lda, const void* W, int ldw, float* C,
                                       int ldc, int M, int N, int K, void* ws, size_t ws_bytes,
                                       hipStream_t st, int* n_split, double pass_bytes) {
  *n_split = 1;
  if (M <= 0) return hipSuccess;
  if (N % 128 != 0 || K % 256 != 0) return hipErrorInvalidValue;
  Plan p = plan_gemm(M, N, K);
  p.nt_w = stream_weights(M, N, K, pass_bytes);
  if (p.S == 1) return launch_plan<EPI_F32>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
  if (ws == nullptr || ws_bytes < (size_t)p.S * M * N * sizeof(float)) return hipErrorInvalidValue;
  *n_split = p.S;
  return launch_plan<EPI_F32>(p, A, lda, W, ldw, C, ldc, M, N, K, ws, st);
}

// x[M, N] += A . W^T followed by xn = bf16(RMSNorm(x)).  When the plan splits
// K the add and the norm are fused into the reduce (returns *fused = true);
// otherwise the GEMM adds in its epilogue and the caller normalises.
hipError_t launch_gemm_add_norm(const void* A, int lda, const void* W, int ldw, float* x, int ldx,
                                int M, int N, int K, void* ws, size_t ws_bytes, float eps,
                                void* xn, hipStream_t st, bool* fused, double pass_bytes) {
  *fused = false;
  if (M <= 0) return hipSuccess;
  if (N % 128 != 0 || K % 256 != 0) return hipErrorInvalidValue;
  Plan p = plan_gemm(M, N, K);
  p.nt_w = stream_weights(M, N, K, pass_bytes);
  if (p.S == 1 || p.S > kMaxSplits || N > kAddNormMaxN)
    return gemm_bf16_launch<EPI_ADD_F32>(A, lda, W, ldw, x, ldx, M, N, K, ws, ws_bytes, st, pass_bytes);
  if (ws == nullptr || ws_bytes < (size_t)p.S * M * N * sizeof(float)) return hipErrorInvalidValue;
  // the partial-sum GEMM of the plan, then the fused reduce
  hipError_t e = launch_plan<EPI_ADD_F32>(p, A, lda, W, ldw, x, ldx, M, N, K, ws, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(splitk_add_norm_kernel, dim3(M), dim3(1024), 0, st, (const float*)ws, p.S, M, N,
                     x, ldx, eps, (bf16_t*)xn);
  *fused = true;
  return hipGetLastError();
}

}  // namespace darts
