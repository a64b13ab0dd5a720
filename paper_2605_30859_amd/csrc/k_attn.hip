// Paged GQA decode attention on gfx950.
//
// out[r][h] = sum_j softmax_j(q[r][h] . k_j / sqrt(hd)) v_j over the row's ctx
// keys; key j sits in page page_table[pt_row][j/16], slot j%16, kv head
// h / G (G = Hq/Hkv).
//
// Work unit = (row, kv head, chunk of C pages), one wavefront each, with a
// grid-stride loop; the wavefront attends 16 query vectors (MFMA rows) to a
// run of pages with an online softmax (attn_page_loop).  Rows of equal context
// (every decode step) map units arithmetically; ragged contexts use a work
// list built on the device (no host round trip, no idle blocks).  Contexts
// are split into chunks only when there are too few (row, kv head) units to
// fill the GPU; chunk partials (o, max, sum) are merged by a combine kernel.
//
// Shared prompt prefix (the rollout): the m trajectories of a prompt share
// its prompt pages.  A prefix kernel stacks the query vectors of a group's
// members 16 to a wavefront and reads each prefix page once per 16 query
// vectors (the per-row kernel fills only G of its 16 MFMA rows); the per-row
// kernel then covers the keys after the prefix, starting from the prefix
// partials.
//
// The prefill of bf16 models has a kernel of its own (attn_prefill_kernel).
#include <math.h>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace darts {

struct CtxSpec {
  const int32_t* ctx_len;  // per-row context, or NULL
  int mod, base;           // ctx(r) = ctx_len ? ctx_len[r] : (mod ? r % mod : 0) + base
  const int32_t* row_pt;   // page-table row of row r, or NULL (identity)
  int max_ctx;             // contexts are clamped to max_ctx (memory safety)
  int64_t n_pages;         // page ids are clamped into [0, n_pages)
  int skip;                // keys [0, skip) are attended by the shared-prefix kernel (a
                           // multiple of 16; 0 when prefixes are not shared)
  int pt_rows;             // row_pt values are clamped into [0, pt_rows) when > 0
  int nt_from;             // pages from this index of a row's list on are the row's alone: their
                           // loads are non-temporal; -1: the kernel looks
};
// KV bytes of a call from which unshared pages are loaded non-temporal when the
// caller may come back with the same pools: the size of the Infinity Cache
constexpr double kNtKvBytes = 256e6;
__device__ __forceinline__ int pt_row(const CtxSpec& c, int r) {
  if (!c.row_pt) return r;
  const int v = c.row_pt[r];
  return c.pt_rows > 0 ? min(max(v, 0), c.pt_rows - 1) : v;
}
__device__ __forceinline__ int ctx_of(const CtxSpec& c, int r) {
  const int v = c.ctx_len ? c.ctx_len[r] : (c.mod ? r % c.mod : 0) + c.base;
  return min(v, c.max_ctx);
}
// keys the per-row kernel covers: those after the shared prefix
__device__ __forceinline__ int span_of(const CtxSpec& c, int r) { return max(ctx_of(c, r) - c.skip, 0); }
__device__ __forceinline__ int clamp_page(const CtxSpec& c, int p) {
  return (int)min((int64_t)max(p, 0), c.n_pages - 1);
}

// Single block: per-row chunk counts -> exclusive offsets and the work list
// (*info items), and info[1] = whether the rows' keys come to nt_keys or more.
__global__ void attn_plan_kernel(CtxSpec cs, int n_rows, int chunk_tokens, int32_t* chunk_off,
                                 int2* work, int32_t* info, int64_t nt_keys) {
  __shared__ int32_t sh[32];
  __shared__ unsigned long long keys;
  const int tid = threadIdx.x;
  if (tid == 0) keys = 0;      // (the scans' barriers publish it)
  unsigned long long mine = 0;
  int running = 0;
  for (int base = 0; base < n_rows; base += 1024) {
    const int r = base + tid;
    const int span = r < n_rows ? span_of(cs, r) : 0;
    const int c = (span + chunk_tokens - 1) / chunk_tokens;
    mine += span;
    int total;
    const int excl = running + block_excl_scan1024(c, sh, &total);
    if (r < n_rows) {
      chunk_off[r] = excl;
      for (int j = 0; j < c; ++j) work[excl + j] = make_int2(r, j);
    }
    running += total;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
  if ((tid & 63) == 0 && mine > 0) atomicAdd(&keys, mine);
  __syncthreads();
  if (tid == 0) {
    info[0] = running;
    info[1] = (int64_t)keys >= nt_keys ? 1 : 0;
  }
}

// Single block: row ranges of the prompt groups in a row list sorted by
// group (group of row r = traj[r] / m): grp_row0[i], grp_n[i], *n_groups.
__global__ void attn_groups_kernel(const int32_t* __restrict__ traj, int n_rows, int m,
                                   int32_t* __restrict__ grp_row0, int32_t* __restrict__ grp_n,
                                   int32_t* __restrict__ n_groups, int32_t* __restrict__ n_groups_out) {
  __shared__ int32_t sums[1024];
  __shared__ int32_t running;
  const int tid = threadIdx.x;
  if (tid == 0) running = 0;
  __syncthreads();
  for (int base = 0; base < n_rows; base += 1024) {
    const int r = base + tid;
    const int st = (r < n_rows && (r == 0 || traj[r] / m != traj[r - 1] / m)) ? 1 : 0;
    sums[tid] = st;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int v = tid >= o ? sums[tid - o] : 0;
      __syncthreads();
      sums[tid] += v;
      __syncthreads();
    }
    if (st) grp_row0[running + sums[tid] - 1] = r;
    __syncthreads();
    if (tid == 1023) running += sums[1023];
    __syncthreads();
  }
  const int ng = running;
  for (int i = tid; i < ng; i += 1024) grp_n[i] = (i + 1 < ng ? grp_row0[i + 1] : n_rows) - grp_row0[i];
  if (tid == 0) {
    *n_groups = ng;
    if (n_groups_out) *n_groups_out = ng;
  }
}

struct AttnBf16Args {
  const bf16_t* q; const bf16_t* kpool; const bf16_t* vpool;
  const int32_t* page_table; int pt_stride; CtxSpec cs; int hq, hkv, chunk_pages;
  int n_rows;
  int uniform_nch;            // > 0: every row has this many chunks, no work list
  const int2* work; const int32_t* chunk_off; const int32_t* info;
  float* ws_o; float2* ws_ml; bf16_t* out;
  // shared-prefix partials of each (row, q head): pre_nch (o, max, sum) sets
  // that chunk 0 of the row starts from; pre_nch == 0 when there are none
  const float* pre_o; const float2* pre_ml; int pre_nch;
};

struct AttnPrefixArgs {
  const bf16_t* q; const bf16_t* kpool; const bf16_t* vpool;
  const int32_t* page_table; int pt_stride; CtxSpec cs; int hq, hkv;
  int prefix_pages;           // shared pages at the front of every member's page list
  int chunk_pages;            // prefix pages per wavefront
  int pre_nch;                // ceil(prefix_pages / chunk_pages)
  int qblocks;                // 16-query blocks per (group, kv head)
  const int32_t* grp_row0; const int32_t* grp_n; const int32_t* n_groups;
  float* pre_o; float2* pre_ml;
};

// K and V of one pair of pages (32 keys) for one kv head, in MFMA operand layout
template <int HD>
struct PagePair {
  bf16x8_t ka[HD / 32], kb[HD / 32], vv[HD / 16];
  bool hasb;
};

// Online-softmax state of one wavefront's 16 query vectors (the MFMA rows):
// lane (quad, col) holds, for query vector 4*quad+i, the running max m[i],
// its share l[i] of the denominator (summed over the 16 lanes at the end) and
// output dims nb*16+col in O[nb][i].
template <int HD>
struct AttnAcc {
  float m[4], l[4];
  f32x4_t O[HD / 16];
};

constexpr int kPst = 40;   // P row stride in LDS (bf16): 80 bytes

// Attend the wavefront's 16 query vectors (A operand qa) to the keys of pages
// [pbeg, pend) of page list pt (kv head kvh); keys at or after ctx are masked.
//   S[16 x 32]  = Q[16 x hd] . K^T      MFMA 16x16x32 bf16 per pair of pages
//   online softmax per query row (16-lane shuffles)
//   O[16 x hd] += P[16 x 32] . V[32 x hd]   MFMA 16x16x32 bf16, P via LDS
// K is read token-major straight into the MFMA B operand (16 B per lane, one
// contiguous 1 KB block of the page per 32-wide K step);
// V pages store 8 consecutive tokens of one dim contiguously, so the P.V
// B operand is also one 16 B load per lane.  The page-id -> key/value load chain is
// not serial: a wavefront holds the ids of 64 pages, one per lane, and those of
// the next 64.  One pair is in flight per wavefront; two (245 registers) were no
// faster once a wavefront's page ids and addresses are scalar and its own
// pages' loads non-temporal.
// NT: non-temporal loads.
template <bool NT>
__device__ __forceinline__ bf16x8_t load_frag(const bf16_t* p) {
  if constexpr (NT) return __builtin_bit_cast(bf16x8_t, __builtin_nontemporal_load((const u32x4_t*)p));
  else return __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)p);
}
template <int HD, bool NT>
__device__ __forceinline__ void attn_page_run(const bf16x8_t (&qa)[HD / 32], const bf16_t* kpool,
                                               const bf16_t* vpool, const CtxSpec& cs,
                                               const int32_t* pt, int pbeg, int pend, int ctx,
                                               int kvh, int hkv, bf16_t* P, AttnAcc<HD>& acc) {
  constexpr int NKK = HD / 32, NNB = HD / 16;
  const int lane = threadIdx.x & 63;
  const int quad = lane >> 4, col = lane & 15;
  const float scale = 1.0f / sqrtf((float)HD);
  auto load = [&](int p, PagePair<HD>& F, int ida, int idb) {
    const int pa = clamp_page(cs, ida);
    F.hasb = (p + 1) < pend;
    const int pb = F.hasb ? clamp_page(cs, idb) : pa;
    const bf16_t* kpa = kpool + k_off(pa, kvh, col, quad * 8, hkv, HD);
    const bf16_t* kpb = kpool + k_off(pb, kvh, col, quad * 8, hkv, HD);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      F.ka[kk] = load_frag<NT>(kpa + kk * kPage * 32);
      F.kb[kk] = load_frag<NT>(kpb + kk * kPage * 32);
    }
    const int vpage = quad < 2 ? pa : pb;
    const bf16_t* vb = vpool + v_off(vpage, kvh, (quad & 1) * 8, col, hkv, HD);
#pragma unroll
    for (int nb = 0; nb < NNB; ++nb)
      F.vv[nb] = load_frag<NT>(vb + nb * 16 * 8);
  };
  auto compute = [&](int p, const PagePair<HD>& F) {
    f32x4_t sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[kk], F.ka[kk], sa, 0, 0, 0);
      sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[kk], F.kb[kk], sb, 0, 0, 0);
    }
    // lane holds S[query 4*quad+i][key p*16+col] (sa) and [(p+1)*16+col] (sb)
    const bool va = p * kPage + col < ctx;
    const bool vb2 = F.hasb && ((p + 1) * kPage + col < ctx);
    float pva[4], pvb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float s1 = va ? sa[i] * scale : -INFINITY;
      const float s2 = vb2 ? sb[i] * scale : -INFINITY;
      float mx = fmaxf(s1, s2);
      mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 4, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 8, 64));
      const float mnew = fmaxf(acc.m[i], mx);
      const float alpha = __expf(acc.m[i] - mnew);
      // the denominator sums the same bf16-rounded weights that multiply V
      pva[i] = bf16_to_f32(f32_to_bf16(__expf(s1 - mnew)));
      pvb[i] = bf16_to_f32(f32_to_bf16(__expf(s2 - mnew)));
      acc.l[i] = acc.l[i] * alpha + pva[i] + pvb[i];
      acc.m[i] = mnew;
#pragma unroll
      for (int nb = 0; nb < NNB; ++nb) acc.O[nb][i] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      P[(4 * quad + i) * kPst + col] = f32_to_bf16(pva[i]);
      P[(4 * quad + i) * kPst + 16 + col] = f32_to_bf16(pvb[i]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bf16x8_t pa8 = *(const bf16x8_t*)(&P[col * kPst + quad * 8]);
#pragma unroll
    for (int nb = 0; nb < NNB; ++nb)
      acc.O[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa8, F.vv[nb], acc.O[nb], 0, 0, 0);
    __builtin_amdgcn_wave_barrier();   // P is rewritten by the next pair
  };
  PagePair<HD> F;
  // lane i: the id of page i of this run of 64 pages, and of the next run
  int ids = pt[min(pbeg + lane, pend - 1)], next_ids = ids;
  for (int p = pbeg; p < pend; p += 2) {
    const int i = (p - pbeg) & 63;
    if (i == 0) {
      if (p > pbeg) ids = next_ids;
      if (p + 64 < pend) next_ids = pt[min(p + 64 + lane, pend - 1)];
    }
    load(p, F, __builtin_amdgcn_readlane(ids, i), __builtin_amdgcn_readlane(ids, i + 1));
    compute(p, F);
  }
}

// The pages other rows share, whose re-reads hit the caches, then the row's own.
template <int HD>
__device__ __forceinline__ void attn_page_loop(const bf16x8_t (&qa)[HD / 32], const bf16_t* kpool,
                                               const bf16_t* vpool, const CtxSpec& cs, int nt_from,
                                               const int32_t* pt, int pbeg, int pend, int ctx,
                                               int kvh, int hkv, bf16_t* P, AttnAcc<HD>& acc) {
  const int mid = min(max(nt_from, pbeg), pend);
  if (pbeg < mid) attn_page_run<HD, false>(qa, kpool, vpool, cs, pt, pbeg, mid, ctx, kvh, hkv, P, acc);
  if (mid < pend) attn_page_run<HD, true>(qa, kpool, vpool, cs, pt, mid, pend, ctx, kvh, hkv, P, acc);
}

// sum of a lane-partial over the 16 lanes of a query row
__device__ __forceinline__ float row16_sum(float l) {
  l += __shfl_xor(l, 1, 64);
  l += __shfl_xor(l, 2, 64);
  l += __shfl_xor(l, 4, 64);
  l += __shfl_xor(l, 8, 64);
  return l;
}

// Per-row decode attention.  Work unit = (row, kv head, chunk of C pages),
// one wavefront each, grid-stride loop; the G query heads sharing the kv head
// fill MFMA rows 0..G-1.  Rows of equal context (every decode step) map units
// arithmetically; ragged contexts use a work list built on the device.  A row
// whose keys span several chunks writes unnormalised partials (o, max, sum)
// and the combine kernel merges them.  With a shared prefix the row's keys
// start at cs.skip and chunk 0 starts from the prefix partials.
//
// Bound by HBM.  Two wavefronts per SIMD (head dim 128: 149 vector and 32
// accumulation registers; 160 and 32 when page ids and addresses were not scalar).
// With scalar ids and non-temporal loads of unshared pages: 777 rows x 1123 keys, 32/4 heads x
// 128: 300 us (6.0 TB/s), before 378; 1024 ragged rows, 32/8 heads: 1700 us,
// before 1800; 512 rows of which 16 at a time share 32 of 57 pages: 196 us,
// before 211.  Equal contiguous shares of all page pairs per wavefront, whatever
// the rows, were no faster: cut rows cost more to merge than an uneven last
// round loses.
template <int HD>
__global__ void __launch_bounds__(256) attn_bf16_kernel(AttnBf16Args A) {
  constexpr int NKK = HD / 32, NNB = HD / 16;
  __shared__ __attribute__((aligned(16))) bf16_t plds[4][16 * kPst];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hq = A.hq, hkv = A.hkv;
  const int G = hq / hkv;
  const int quad = lane >> 4, col = lane & 15;
  const int total = (A.uniform_nch > 0 ? A.n_rows * A.uniform_nch : A.info[0]) * hkv;
  const int skip_pages = A.cs.skip / kPage;
  // ragged rows: the host knows their largest context only, the plan their sum
  const int nt_all = A.uniform_nch > 0 || A.cs.nt_from >= 0 || A.info[1] ? A.cs.nt_from : INT32_MAX;
  bf16_t* P = plds[w];
  for (int item = blockIdx.x * 4 + w; item < total; item += gridDim.x * 4) {
    const int wi = item / hkv, kvh = item - wi * hkv;
    int row, chunk, cid;
    if (A.uniform_nch > 0) {
      row = wi / A.uniform_nch; chunk = wi - row * A.uniform_nch; cid = wi;
    } else {
      const int2 rc = A.work[wi];
      row = rc.x; chunk = rc.y; cid = A.chunk_off[row] + chunk;
    }
    const int ctx = ctx_of(A.cs, row);
    const int32_t* pt = A.page_table + (int64_t)pt_row(A.cs, row) * A.pt_stride;
    const int npg = (ctx + kPage - 1) / kPage;
    const int nch = (npg - skip_pages + A.chunk_pages - 1) / A.chunk_pages;
    const int pbeg = skip_pages + chunk * A.chunk_pages;
    const int pend = min(pbeg + A.chunk_pages, npg);
    int nt_from = nt_all;
    if (nt_from < 0 && pbeg < pend) {
      // not told: a chunk whose first page a neighbouring row lists at the same
      // place is taken to be shared (only the loads' cache policy depends on it)
      const int id = pt[pbeg];
      const int up = row > 0 ? pt[pbeg - A.pt_stride] : -1, down = row + 1 < A.n_rows ? pt[pbeg + A.pt_stride] : -1;
      nt_from = __builtin_amdgcn_readfirstlane(id == up || id == down) ? pend : pbeg;
    }

    bf16x8_t qa[NKK];
    {
      const bool valid = col < G;
      const bf16_t* qrow = A.q + ((int64_t)row * hq + kvh * G + (valid ? col : 0)) * HD + quad * 8;
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        u32x4_t v = valid ? *(const u32x4_t*)(qrow + 32 * kk) : (u32x4_t){0u, 0u, 0u, 0u};
        qa[kk] = __builtin_bit_cast(bf16x8_t, v);
      }
    }
    AttnAcc<HD> acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) { acc.m[i] = -INFINITY; acc.l[i] = 0.f; }
#pragma unroll
    for (int nb = 0; nb < NNB; ++nb) acc.O[nb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    if (A.pre_nch > 0 && chunk == 0) {
      // start from the merged prefix partials of this row's heads
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int h = 4 * quad + i;
        if (h >= G) continue;
        const int64_t base = ((int64_t)row * hq + kvh * G + h) * A.pre_nch;
        float M = -INFINITY;
        for (int c = 0; c < A.pre_nch; ++c) M = fmaxf(M, A.pre_ml[base + c].x);
        float L = 0.f;
        for (int c = 0; c < A.pre_nch; ++c) {
          const float2 ml = A.pre_ml[base + c];
          const float f = __expf(ml.x - M);
          L += ml.y * f;
#pragma unroll
          for (int nb = 0; nb < NNB; ++nb) acc.O[nb][i] += A.pre_o[(base + c) * HD + nb * 16 + col] * f;
        }
        acc.m[i] = M;
        acc.l[i] = col == 0 ? L : 0.f;
      }
    }
    attn_page_loop<HD>(qa, A.kpool, A.vpool, A.cs, nt_from, pt, pbeg, pend, ctx, kvh, hkv, P, acc);

    float lrow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) lrow[i] = row16_sum(acc.l[i]);
    if (nch == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int h = 4 * quad + i;
        if (h >= G) continue;
        const float inv = 1.0f / lrow[i];
        bf16_t* orow = A.out + ((int64_t)row * hq + kvh * G + h) * HD + col;
#pragma unroll
        for (int nb = 0; nb < NNB; ++nb) orow[nb * 16] = f32_to_bf16(acc.O[nb][i] * inv);
      }
      continue;
    }
    // several chunks: write this chunk's unnormalised partial; the combine
    // kernel merges the chunks of a row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = 4 * quad + i;
      if (h >= G) continue;
      const int qh = kvh * G + h;
      float* po = A.ws_o + ((int64_t)cid * hq + qh) * HD + col;
#pragma unroll
      for (int nb = 0; nb < NNB; ++nb) po[nb * 16] = acc.O[nb][i];
      if (col == 0) A.ws_ml[(int64_t)cid * hq + qh] = make_float2(acc.m[i], lrow[i]);
    }
  }
}

// Shared-prefix attention.  The members of a prompt group (consecutive rows
// of one group) share their first prefix_pages pages, so their query vectors
// (rows x G heads) are stacked 16 to a wavefront as the MFMA rows and attend
// to the prefix keys together: each prefix key and value is read once per
// 16 query vectors instead of once per G.  Work unit = (group, kv head,
// 16-query block, chunk of chunk_pages prefix pages); it writes the
// unnormalised partial (o, max, sum) of each of its query vectors.
template <int HD>
__global__ void __launch_bounds__(256) attn_prefix_kernel(AttnPrefixArgs A) {
  constexpr int NKK = HD / 32, NNB = HD / 16;
  __shared__ __attribute__((aligned(16))) bf16_t plds[4][16 * kPst];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int hq = A.hq, hkv = A.hkv;
  const int G = hq / hkv;
  const int quad = lane >> 4, col = lane & 15;
  const int total = A.n_groups[0] * hkv * A.qblocks * A.pre_nch;
  const int ctx = A.prefix_pages * kPage;
  bf16_t* P = plds[w];
  for (int item = blockIdx.x * 4 + w; item < total; item += gridDim.x * 4) {
    int t = item;
    const int pc = t % A.pre_nch; t /= A.pre_nch;
    const int qb = t % A.qblocks; t /= A.qblocks;
    const int kvh = t % hkv;
    const int gi = t / hkv;
    const int r0 = A.grp_row0[gi], ng = A.grp_n[gi];
    bf16x8_t qa[NKK];
    {
      const int qv = qb * 16 + col, rl = qv / G, h = qv - rl * G;
      const bool valid = rl < ng;
      const bf16_t* qrow = A.q + ((int64_t)(r0 + (valid ? rl : 0)) * hq + kvh * G + h) * HD + quad * 8;
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        u32x4_t v = valid ? *(const u32x4_t*)(qrow + 32 * kk) : (u32x4_t){0u, 0u, 0u, 0u};
        qa[kk] = __builtin_bit_cast(bf16x8_t, v);
      }
    }
    const int32_t* pt = A.page_table + (int64_t)pt_row(A.cs, r0) * A.pt_stride;
    const int pbeg = pc * A.chunk_pages;
    const int pend = min(pbeg + A.chunk_pages, A.prefix_pages);
    AttnAcc<HD> acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) { acc.m[i] = -INFINITY; acc.l[i] = 0.f; }
#pragma unroll
    for (int nb = 0; nb < NNB; ++nb) acc.O[nb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    attn_page_run<HD, false>(qa, A.kpool, A.vpool, A.cs, pt, pbeg, pend, ctx, kvh, hkv, P, acc);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float l = row16_sum(acc.l[i]);
      const int qv = qb * 16 + 4 * quad + i, rl = qv / G, h = qv - rl * G;
      if (rl >= ng) continue;
      const int64_t idx = ((int64_t)(r0 + rl) * hq + kvh * G + h) * A.pre_nch + pc;
      float* po = A.pre_o + idx * HD + col;
#pragma unroll
      for (int nb = 0; nb < NNB; ++nb) po[nb * 16] = acc.O[nb][i];
      if (col == 0) A.pre_ml[idx] = make_float2(acc.m[i], l);
    }
  }
}

// ------------------------------------------------------------------ prefill
// Causal attention of whole prompts (bf16): query position t of a prompt
// attends to its keys 0..t, which lie in the prompt's pages.
//
// Block = 4 wavefronts over (prompt, kv head, run of query vectors).  The
// query vectors of a (prompt, kv head) are its positions times the G heads that
// share the kv head, position-major, whatever G is; a wavefront takes NT tiles
// of 16.  Keys and values pass through LDS in stages of 64 keys (4 pages,
// one copied by each wavefront with direct 16-byte LDS loads, the next stage
// while this one is computed), so each is read once per block and not once per
// query.  Products are transposed, so that a lane's scores belong to one query:
//   S^T[keys x 16] = K . Q^T     two tiles of 16 keys per 32 keys; row 4q+i of
//                                tile u is key 8q + 4u + i
//   P^T            = 2^(c S^T - m), in fp32, rounded to bf16: the lane's eight
//                                weights are the eight keys of its quad, which
//                                is the next product's operand as it stands
//   O^T[dims x 16] += V^T . P^T  two tiles of 16 dims per 32 dims; row 4q+i of
//                                tile u is dim 8q + 4u + i, so that a lane ends
//                                with 8 consecutive dims
//   l              += 1 . P^T    the denominator: the sum of the rounded weights
// The running maximum m follows every score (O and l are rescaled), so that the
// largest weight is 1, which bf16 holds exactly.  Letting m lag by up to 8 in the
// exponent saves 7% of the time, but rounds that weight too: the weights'
// share of the error grew from 7e-4 to 1.1e-3 of the result (head dim 128, 2048
// keys, scores of a few units).
//
// Bound by VALU and matrix issue (the exponentials of a 16 x 32 tile take about
// as long as its products), hence two blocks per CU.  64 prompts x 512 tokens,
// 32/4 heads x 128: 278 us per layer (137 GFLOP, 490 TFLOP/s), against 1600 us
// for the decode kernel with one row per query position, which reads every key
// once per query.  With 2 or 4 tiles per wavefront instead of 3: 7% and 50% more
// (4 spill past 256 registers; head dims 64 and 32 take 1 or 2).
struct PrefillArgs {
  const bf16_t* q; const bf16_t* kpool; const bf16_t* vpool;
  const int32_t* page_table; int64_t pt_step;   // page list of prompt i: page_table + i * pt_step
  int64_t n_pages;
  int n_prompts, len, hq, hkv;                  // len: positions per prompt, a multiple of 16
  bf16_t* out;
};
constexpr int kPreWaves = 4, kPreKeys = 64;     // wavefronts per block (one copies one page), keys per stage

template <int HD, int NT>
__global__ void __launch_bounds__(64 * kPreWaves, 2) attn_prefill_kernel(PrefillArgs A) {
  constexpr int NKK = HD / 32;                  // 32-dim blocks: K steps of S, dim pairs of tiles of O
  constexpr int PB = kPage * HD;                // elements of a page of one kv head (K or V)
  __shared__ __attribute__((aligned(16))) bf16_t smem[2][2][kPreWaves * PB];   // [stage][K | V][page]
  static_assert(kPreWaves * kPage == kPreKeys, "a wavefront copies a page");
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int quad = lane >> 4, col = lane & 15;
  const int G = A.hq / A.hkv;
  const int pairs = A.n_prompts * A.hkv;
  const int nvec = A.len * G, ntile = (int)(gridDim.x / pairs);
  // longest runs (last positions) first
  const int run = ntile - 1 - (int)(blockIdx.x / pairs), pair = (int)(blockIdx.x % pairs);
  const int prompt = pair / A.hkv, kvh = pair % A.hkv;
  const int v0 = (run * kPreWaves + w) * NT * 16;           // this wavefront's query vectors
  const int vend = min((run + 1) * kPreWaves * NT * 16, nvec);
  const int n_stage = ((vend - 1) / G) / kPreKeys + 1;      // stages the block needs
  const int tlast = v0 < nvec ? min(v0 + NT * 16 - 1, nvec - 1) / G : -1;   // the wavefront's last position

  bf16x8_t qb[NT][NKK];
  int t[NT];                                                // position of the lane's query
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int v = min(v0 + n * 16 + col, nvec - 1);
    t[n] = v / G;
    const bf16_t* src = A.q + (((int64_t)prompt * A.len + t[n]) * A.hq + kvh * G + (v - t[n] * G)) * HD + quad * 8;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) qb[n][kk] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(src + 32 * kk));
  }
  // Copy of page w of a stage.  LDS holds K's 16-byte chunk (slot, dims 8c..)
  // of a 32-dim block at chunk slot*4 + (c ^ (slot/4) ^ (page parity)), and V's
  // (dim) at chunk dim ^ 4*(dim/16 odd): the 16 lanes of a quad then read 256
  // bytes that lie in different banks.
  const int kslot = lane >> 2, kch = (lane & 3) ^ (kslot >> 2) ^ (w & 1);
  const int ksrc = kslot * 32 + kch * 8, vsrc = (lane ^ (((lane >> 4) & 1) << 2)) * 8;
  const int32_t* pt = A.page_table + prompt * A.pt_step;
  const int last_page = A.len / kPage - 1;
  int ids = 0;                                              // lane i: this wavefront's page of stage i (mod 64)
  auto copy = [&](int stage, int buf) {
    if ((stage & 63) == 0) ids = pt[min((stage + lane) * kPreWaves + w, last_page)];
    const int id = __builtin_amdgcn_readlane(ids, stage & 63);
    const int64_t page = min((int64_t)max(id, 0), A.n_pages - 1);
    const bf16_t* k = A.kpool + (page * A.hkv + kvh) * PB;
    const bf16_t* v = A.vpool + (page * A.hkv + kvh) * PB;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      __builtin_amdgcn_global_load_lds((const void*)(k + kk * 512 + ksrc),
                                       (__attribute__((address_space(3))) void*)(&smem[buf][0][w * PB + kk * 512]), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)(v + kk * 512 + vsrc),
                                       (__attribute__((address_space(3))) void*)(&smem[buf][1][w * PB + kk * 512]), 16, 0, 0);
    }
  };
  // fragment offsets in a 32-key half of a stage (pages 2*half, 2*half + 1):
  // key 8*(col/4) + 4u + col%4 and dim 8*(col/4) + 4u + col%4 of a block of 32
  int koff[2], voff[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int x = 8 * (col >> 2) + 4 * u + (col & 3), slot = x & 15, pg = x >> 4;
    koff[u] = pg * PB + slot * 32 + ((quad ^ (slot >> 2) ^ pg) * 8);
    voff[u] = (quad >> 1) * PB + ((quad & 1) * HD + (x ^ (((x >> 4) & 1) << 2))) * 8;
  }

  f32x4_t O[NT][NKK][2], l[NT];
  float m[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    m[n] = -INFINITY;
    l[n] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NKK; ++b) O[n][b][0] = O[n][b][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  }
  const u32x4_t ones_bits = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, ones_bits);
  const float c = 1.4426950408889634f / sqrtf((float)HD);   // scores to exponents of 2

  copy(0, 0);
  for (int st = 0; st < n_stage; ++st) {
    // this stage's copies (this wavefront's) have landed, then everybody's; all
    // reads of the other buffer were done before this barrier
    __builtin_amdgcn_s_waitcnt(0xf70);                      // vmcnt(0)
    __syncthreads();
    if (st + 1 < n_stage) copy(st + 1, (st + 1) & 1);
    const bf16_t* sk = smem[st & 1][0];
    const bf16_t* sv = smem[st & 1][1];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int k0 = st * kPreKeys + half * 32;
      if (k0 > tlast) break;
      f32x4_t S[NT][2];
#pragma unroll
      for (int n = 0; n < NT; ++n) S[n][0] = S[n][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bf16x8_t kf = *(const bf16x8_t*)(sk + half * 2 * PB + kk * 512 + koff[u]);
#pragma unroll
          for (int n = 0; n < NT; ++n) S[n][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qb[n][kk], S[n][u], 0, 0, 0);
        }
      bf16x8_t pf[NT];
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        if (k0 + 31 > v0 / G) {                             // some query of the wavefront ends in these keys
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (k0 + 8 * quad + 4 * u + i > t[n]) S[n][u][i] = -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(S[n][0][0], S[n][0][1]), fmaxf(S[n][0][2], S[n][0][3])),
                         fmaxf(fmaxf(S[n][1][0], S[n][1][1]), fmaxf(S[n][1][2], S[n][1][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c;
        if (__any(mx > m[n])) {
          const float mnew = fmaxf(m[n], mx);
          const float alpha = exp2f(m[n] - mnew);
          m[n] = mnew;
          l[n] *= alpha;
#pragma unroll
          for (int b = 0; b < NKK; ++b) { O[n][b][0] *= alpha; O[n][b][1] *= alpha; }
        }
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(S[n][e >> 2][e & 3], c, -m[n]));
        const u32x4_t pk = {f32_to_bf16x2(p[0], p[1]), f32_to_bf16x2(p[2], p[3]), f32_to_bf16x2(p[4], p[5]),
                            f32_to_bf16x2(p[6], p[7])};
        pf[n] = __builtin_bit_cast(bf16x8_t, pk);
      }
#pragma unroll
      for (int n = 0; n < NT; ++n) l[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[n], l[n], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < NKK; ++b)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bf16x8_t vf = *(const bf16x8_t*)(sv + half * 2 * PB + b * 256 + voff[u]);
#pragma unroll
          for (int n = 0; n < NT; ++n) O[n][b][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[n], O[n][b][u], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int v = v0 + n * 16 + col;
    if (v >= nvec) continue;
    const float inv = 1.0f / l[n][0];
    bf16_t* dst = A.out + (((int64_t)prompt * A.len + t[n]) * A.hq + kvh * G + (v - t[n] * G)) * HD + quad * 8;
#pragma unroll
    for (int b = 0; b < NKK; ++b) {
      const f32x4_t x = O[n][b][0] * inv, y = O[n][b][1] * inv;
      *(u32x4_t*)(dst + 32 * b) = (u32x4_t){f32_to_bf16x2(x[0], x[1]), f32_to_bf16x2(x[2], x[3]),
                                            f32_to_bf16x2(y[0], y[1]), f32_to_bf16x2(y[2], y[3])};
    }
  }
}

static int64_t prefill_blocks(const PrefillArgs& a, int nt) {
  const int vecs = kPreWaves * nt * 16;
  return ((int64_t)a.len * (a.hq / a.hkv) + vecs - 1) / vecs * a.n_prompts * a.hkv;
}
template <int HD, int NT>
static void attn_prefill_go(const PrefillArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((attn_prefill_kernel<HD, NT>), dim3((unsigned)prefill_blocks(a, NT)), dim3(64 * kPreWaves), 0, st,
                     a);
}
// Head dims 64 and 32: two tiles per wavefront from so many blocks on, else one.
// Prefill of six layers in 1 / 2 / 4 tiles: 16/4 heads x 64, 4 x 512 tokens 480 /
// 512 / 561 us (512, 256 and 128 blocks), 8 x 512 624 / 640 / 688, 16 x 512 819 /
// 808 / 859, 48 x 512 1606 / 1555 / 1630, 1 x 4096 974 / 1125 / 1504; 32/8 heads x
// 32, 4 x 512 468 / 495 / 547, 8 x 512 629 / 628 / 672, 4 x 4096 2498 / 2382 / 2556.
constexpr int64_t kPreBlocks2 = 1024;

hipError_t launch_attention_prefill(const void* q, const void* k_pool, const void* v_pool, int64_t n_pages,
                                    const int32_t* page_table, int64_t pt_step, int n_prompts, int len, int hq,
                                    int hkv, int hd, void* out, hipStream_t st) {
  if (n_prompts <= 0) return hipSuccess;
  if (len < kPage || len % kPage || hkv < 1 || hq % hkv || n_pages < 1) return hipErrorInvalidValue;
  PrefillArgs a;
  a.q = (const bf16_t*)q; a.kpool = (const bf16_t*)k_pool; a.vpool = (const bf16_t*)v_pool;
  a.page_table = page_table; a.pt_step = pt_step; a.n_pages = n_pages;
  a.n_prompts = n_prompts; a.len = len; a.hq = hq; a.hkv = hkv; a.out = (bf16_t*)out;
  if (hd == 128) attn_prefill_go<128, 3>(a, st);
  else if (hd == 64 && prefill_blocks(a, 2) >= kPreBlocks2) attn_prefill_go<64, 2>(a, st);
  else if (hd == 64) attn_prefill_go<64, 1>(a, st);
  else if (hd == 32 && prefill_blocks(a, 2) >= kPreBlocks2) attn_prefill_go<32, 2>(a, st);
  else if (hd == 32) attn_prefill_go<32, 1>(a, st);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// One exchange of a sum over lanes in which every lane holds 2H dims of o: the
// lanes of a pair x apart keep H of them each, summed.  H = 0: both keep the one.
template <int H, int x>
__device__ __forceinline__ void halve_dims(float* o, int lane, int& keep) {
  if constexpr (H == 0) {
    o[0] += __shfl_xor(o[0], x, 64);
  } else {
    const bool up = (lane & x) != 0;
#pragma unroll
    for (int d = 0; d < H; ++d) {
      const float mine = up ? o[d + H] : o[d], other = up ? o[d] : o[d + H];
      o[d] = mine + __shfl_xor(other, x, 64);
    }
    keep += up ? H : 0;
  }
}

// fp32 attention (fp32 models): one wavefront per (row, q head, chunk), a key per
// lane.  (Tiny model, 32 rows x 4 heads x 32: 6.2 us per launch, 16.6 with a
// 64-lane sum per dim.)
template <int HD>
__global__ void __launch_bounds__(256) attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ kpool, const float* __restrict__ vpool,
    const int32_t* __restrict__ page_table, int pt_stride, CtxSpec cs, int hq, int hkv,
    int chunk_pages, const int2* __restrict__ work, const int32_t* __restrict__ chunk_off,
    const int32_t* __restrict__ info, float* __restrict__ ws_o, float2* __restrict__ ws_ml,
    float* __restrict__ out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int G = hq / hkv;
  const float scale = 1.0f / sqrtf((float)HD);
  const int total = info[0] * hq;
  for (int item = blockIdx.x * 4 + w; item < total; item += gridDim.x * 4) {
    const int wi = item / hq, qh = item - wi * hq, kvh = qh / G;
    const int2 rc = work[wi];
    const int row = rc.x, chunk = rc.y;
    const int ctx = ctx_of(cs, row);
    const int32_t* pt = page_table + (int64_t)pt_row(cs, row) * pt_stride;
    const int tbeg = chunk * chunk_pages * kPage;
    const int tend = min(tbeg + chunk_pages * kPage, ctx);
    const float* qv = q + ((int64_t)row * hq + qh) * HD;
    float qreg[HD];
#pragma unroll
    for (int d = 0; d < HD; ++d) qreg[d] = qv[d];
    float m = -INFINITY, l = 0.f, o[HD];
#pragma unroll
    for (int d = 0; d < HD; ++d) o[d] = 0.f;
#pragma unroll 1
    for (int j = tbeg + lane; j < tend; j += 64) {
      const int page = clamp_page(cs, pt[j / kPage]), slot = j % kPage;
      // four dims of a key are one load; a value's dims are 8 floats apart
      const float4* kp = (const float4*)(kpool + k_off(page, kvh, slot, 0, hkv, HD));
      const float* vp = vpool + v_off(page, kvh, slot, 0, hkv, HD);
      float s = 0.f;
#pragma unroll
      for (int d = 0; d < HD; d += 4) {
        const float4 k4 = kp[((d >> 5) * kPage * 32 + (d & 31)) / 4];
        s = fmaf(qreg[d], k4.x, s);
        s = fmaf(qreg[d + 1], k4.y, s);
        s = fmaf(qreg[d + 2], k4.z, s);
        s = fmaf(qreg[d + 3], k4.w, s);
      }
      s *= scale;
      const float mn = fmaxf(m, s);
      const float a = __expf(m - mn), pj = __expf(s - mn);
      l = l * a + pj;
#pragma unroll
      for (int d = 0; d < HD; ++d) o[d] = o[d] * a + pj * vp[d * 8];
      m = mn;
    }
    const float mw = wave_max(m);
    const float a = (m == -INFINITY) ? 0.f : __expf(m - mw);
    const float lw = wave_sum(l * a);
    const int nch = ((ctx + kPage - 1) / kPage + chunk_pages - 1) / chunk_pages;
    const int cid = chunk_off[row] + chunk;
    // sum the lanes' HD-dim partials, halving the dims a lane keeps at each
    // exchange (HD exchanges in all, not 6 HD): afterwards lane x holds dims
    // whose bit h was decided by bit h of x
#pragma unroll
    for (int d = 0; d < HD; ++d) o[d] *= a;
    int keep = 0;                         // the first of the dims this lane has kept
    halve_dims<HD / 2, 32>(o, lane, keep);
    halve_dims<HD / 4, 16>(o, lane, keep);
    halve_dims<HD / 8, 8>(o, lane, keep);
    halve_dims<HD / 16, 4>(o, lane, keep);
    halve_dims<HD / 32, 2>(o, lane, keep);
    halve_dims<HD / 64, 1>(o, lane, keep);
    constexpr int KEPT = HD > 64 ? HD / 64 : 1;             // dims per lane
    if (HD >= 64 || (lane & (64 / HD - 1)) == 0) {
#pragma unroll
      for (int d = 0; d < KEPT; ++d) {
        if (nch == 1) out[((int64_t)row * hq + qh) * HD + keep + d] = o[d] / lw;
        else ws_o[((int64_t)cid * hq + qh) * HD + keep + d] = o[d];
      }
    }
    if (nch > 1 && lane == 0) ws_ml[(int64_t)cid * hq + qh] = make_float2(mw, lw);
  }
}

// Merge chunk partials: one wavefront per (row, q head); rows with a single
// chunk were written directly by the attention kernel.  The chunk maxima and
// denominators are reduced across lanes (lane = chunk), then each lane
// accumulates its output dims over the chunks, taking each chunk's weight
// exp(m_c - M) from the lane that computed it.  The first batch of partial
// outputs and the lane's own chunk statistics are loaded together, before
// any reduction, so a row of up to kCB chunks costs one round trip to memory.
template <typename OUT>
__global__ void attn_combine_kernel(CtxSpec cs, int n_rows, int hq, int hd, int chunk_tokens,
                                    int uniform_nch, const int32_t* __restrict__ chunk_off,
                                    const float* __restrict__ ws_o, const float2* __restrict__ ws_ml,
                                    OUT* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= n_rows * hq) return;
  const int row = item / hq, qh = item % hq;
  const int nch = (span_of(cs, row) + chunk_tokens - 1) / chunk_tokens;
  if (nch <= 1) return;
  // equal contexts (no work list): row r's chunks are partial sets r*nch ..
  const int c0 = uniform_nch > 0 ? row * uniform_nch : chunk_off[row];
  const float2* ml = ws_ml + (int64_t)c0 * hq + qh;          // chunk c at ml[c * hq]
  const int nd = (hd + 63) / 64;                             // output dims per lane: lane + 64 t
  const float* ob = ws_o + ((int64_t)c0 * hq + qh) * hd + lane;   // chunk c at ob[c * hq * hd]
  const int64_t cstride = (int64_t)hq * hd;
  // batches of up to kCB chunks: every partial of the batch is loaded before
  // any is accumulated, so a lane keeps 2 * kCB loads in flight
  constexpr int kCB = 16;
  float o0[kCB], o1[kCB];
  auto load_batch = [&](int c) {
#pragma unroll
    for (int j = 0; j < kCB; ++j) {
      const float* o = ob + (int64_t)(c + j) * cstride;
      const bool ok = c + j < nch;
      o0[j] = (ok && lane < hd) ? o[0] : 0.f;
      o1[j] = (ok && nd > 1) ? o[64] : 0.f;
    }
  };
  load_batch(0);
  const float2 v0 = lane < nch ? ml[(int64_t)lane * hq] : make_float2(-INFINITY, 0.f);
  float M = v0.x;
  for (int c = lane + 64; c < nch; c += 64) M = fmaxf(M, ml[(int64_t)c * hq].x);
  M = wave_max(M);
  float L = lane < nch ? v0.y * __expf(v0.x - M) : 0.f;
  for (int c = lane + 64; c < nch; c += 64) {
    const float2 v = ml[(int64_t)c * hq];
    L += v.y * __expf(v.x - M);
  }
  L = wave_sum(L);
  const float invL = 1.0f / L;
  float acc[2] = {0.f, 0.f};
  for (int base = 0; base < nch; base += 64) {
    const int nb = min(64, nch - base);
    const float w = lane < nb ? __expf((base == 0 ? v0.x : ml[(int64_t)(base + lane) * hq].x) - M) : 0.f;
    for (int j0 = 0; j0 < nb; j0 += kCB) {
      if (base + j0 > 0) load_batch(base + j0);
#pragma unroll
      for (int j = 0; j < kCB; ++j) {
        const float wj = __shfl(w, (j0 + j) & 63, 64);
        acc[0] += wj * o0[j];
        acc[1] += wj * o1[j];
      }
    }
  }
  for (int t = 0; t < nd; ++t) {
    const int d = lane + 64 * t;
    if (d >= hd) break;
    const float v = acc[t] * invL;
    if constexpr (sizeof(OUT) == 2) out[((int64_t)row * hq + qh) * hd + d] = f32_to_bf16(v);
    else out[((int64_t)row * hq + qh) * hd + d] = v;
  }
}

// Resident wavefronts of the per-row bf16 kernel on MI355X: 256 CUs times its
// occupancy (a property of the compiled kernel).  Fixed CU count: the chunking,
// and with it the summation order, depends on the shapes only.
constexpr int kAttnMaxSlots = 256 * 16;
static int attn_slots(int hd) {
  static int cached[3] = {0, 0, 0};
  const int i = hd == 128 ? 0 : (hd == 64 ? 1 : 2);
  if (cached[i] == 0) {
    int nb = 0;
    hipError_t e = hd == 128 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, attn_bf16_kernel<128>, 256, 0)
                 : hd == 64  ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, attn_bf16_kernel<64>, 256, 0)
                             : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, attn_bf16_kernel<32>, 256, 0);
    if (e != hipSuccess || nb < 1) nb = 2;
    cached[i] = std::min(256 * 4 * nb, kAttnMaxSlots);
  }
  return cached[i];
}

// Estimated time (us, less what every split has) of an equal-context launch in n
// chunks of c pages per row.  A wavefront spends kTau per page when few run; the
// pages of w wavefronts take w * c * page bytes / kBw when many do (a tenth of
// them counted by whole blocks per CU); in between the two add up in cubes.  A last round after full ones costs at least
// kLastRound of a full one.  Split rows pay for the combine launch, its
// wavefronts (one per row and query head) and the partial sums.
static double chunk_estimate(int n_rows, int hq, int hkv, int hd, int slots, int64_t n, int c) {
  constexpr double kBw = 6.7e6, kStart = 0.9, kLastRound = 0.4;           // bytes/us, us
  constexpr double kCombine = 3.1, kCombineRow = 4e-4, kPartBw = 3.5e6;   // us, us, bytes/us
  const double tau = 0.33 + 0.0038 * hd, page = 4.0 * kPage * hd;         // us, bytes
  const double lat = (c + (c & 1)) * tau + kStart;
  auto round = [&](double w) {
    const double full_cus = std::ceil(w / (4 * 256)) * (4 * 256);
    const double bw = (w > 4 * 256 ? w + 0.1 * (full_cus - w) : w) * c * page / kBw;
    return std::cbrt(lat * lat * lat + bw * bw * bw);
  };
  const int64_t items = (int64_t)n_rows * hkv * n, full = items / slots, rest = items - full * slots;
  double t = full > 0 ? (double)full * round(slots) : 0.0;
  if (rest > 0) t += full > 0 ? std::max(round((double)rest), kLastRound * round(slots)) : round((double)rest);
  if (n > 1) t += kCombine + kCombineRow * n_rows * hq + 8.0 * (double)n * n_rows * hq * hd / kPartBw;
  return t;
}

// Pages per chunk.  Ragged contexts: 128 pages (2048 keys), so that the
// longest rows are spread over many wavefronts instead of one while short rows
// stay whole (on the sweep's lognormal contexts, 32 / 64 / 128 / 256 pages
// took 1.85 / 1.76 / 1.72 / 1.82 ms: fewer chunks mean fewer partial sums and
// less per-item work, more mean better balance).  Equal contexts: the chunk
// count with the least estimated time, at most ~4 rounds of items and chunks of
// at least 4 pages.  The estimate's figures were fitted to 2200 forced splits of
// 580 sizes (1 to 1024 rows, 40 to 12000 keys; 32/8, 32/4 heads x 128, 16/4 x
// 64, 32/8 x 32).  Its choices take 0.5-0.9% more than the fastest split on
// average; counting whole or partial rounds alone took 5% more, and up to 1.5
// times as long (450 rows x 120 keys, 16/4 x 64: whole rows 13.1 us, halves 22.2).
constexpr int kRaggedChunkPages = 128;
static int choose_chunk_pages(int n_rows, int hq, int hkv, int max_ctx, bool uniform, int hd) {
  const int64_t units = (int64_t)n_rows * hkv;
  const int npg = (max_ctx + kPage - 1) / kPage;
  if (!uniform) return npg <= kRaggedChunkPages ? npg + (npg & 1) : kRaggedChunkPages;
  const int slots = attn_slots(hd);
  const int64_t nmax = std::max<int64_t>(1, (4 * (int64_t)slots + units - 1) / units);
  double best = 1e30;
  int best_c = npg;
  for (int64_t n = 1; n <= std::min<int64_t>(nmax, npg); ++n) {
    const int c = (int)((npg + n - 1) / n);
    const int64_t nch = (npg + c - 1) / c;
    if (nch != n) continue;                 // same split as a smaller n
    if (n > 1 && c < 4) break;              // chunks of at least 4 pages (64 keys)
    const double t = chunk_estimate(n_rows, hq, hkv, hd, slots, n, c);
    if (t < best) { best = t; best_c = c; }
  }
  return best_c;
}

constexpr int kPrefixChunkPages = 8;   // shared-prefix pages per wavefront (128 keys)

struct AttnWs {
  int32_t* chunk_off; int2* work; int32_t* info; float* ws_o; float2* ws_ml;
  int64_t max_chunks;          // partial sets the workspace holds
  float* pre_o; float2* pre_ml; int32_t* grp_row0; int32_t* grp_n; int32_t* n_groups;
};
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
// Workspace: [chunk_off | work list | info | partial o | partial (m, l)], then
// with a shared prefix [prefix partial o | prefix (m, l) | group row0 | group n | n_groups].
static size_t ws_layout(int n_rows, int hq, int hkv, int hd, int max_ctx, int prefix_pages, char* base,
                        AttnWs* w) {
  // partial sets for either chunking: ragged rows split into kRaggedChunkPages chunks;
  // equal contexts into at most max(1, ceil(4 * slots / units)) chunks per row
  // (choose_chunk_pages), i.e. at most n_rows + 4 * kAttnMaxSlots / hkv sets
  const int npg = (max_ctx + kPage - 1) / kPage;
  const int64_t ragged = (int64_t)n_rows * ((npg + kRaggedChunkPages - 1) / kRaggedChunkPages);
  const int64_t equal = (int64_t)n_rows + (4 * (int64_t)kAttnMaxSlots + hkv - 1) / hkv;
  const int64_t maxch = std::max(ragged, std::min<int64_t>(equal, (int64_t)n_rows * npg));
  (void)prefix_pages;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return base ? base + o : nullptr; };
  char* a = take((size_t)n_rows * 4);
  char* b = take((size_t)maxch * sizeof(int2));
  char* c = take(64);
  char* d = take((size_t)maxch * hq * hd * sizeof(float));
  char* e = take((size_t)maxch * hq * sizeof(float2));
  char *f = nullptr, *g = nullptr, *h = nullptr, *i = nullptr, *j = nullptr;
  if (prefix_pages > 0) {
    const int64_t pn = (prefix_pages + kPrefixChunkPages - 1) / kPrefixChunkPages;
    f = take((size_t)n_rows * hq * pn * hd * sizeof(float));
    g = take((size_t)n_rows * hq * pn * sizeof(float2));
    h = take((size_t)n_rows * 4);
    i = take((size_t)n_rows * 4);
    j = take(64);
  }
  if (w) {
    w->chunk_off = (int32_t*)a; w->work = (int2*)b; w->info = (int32_t*)c;
    w->ws_o = (float*)d; w->ws_ml = (float2*)e; w->max_chunks = maxch;
    w->pre_o = (float*)f; w->pre_ml = (float2*)g; w->grp_row0 = (int32_t*)h; w->grp_n = (int32_t*)i;
    w->n_groups = (int32_t*)j;
  }
  return off;
}

size_t attn_workspace_bytes(int n_rows, int hq, int hkv, int hd, int max_ctx) {
  return ws_layout(n_rows, hq, hkv, hd, max_ctx, 0, nullptr, nullptr);
}
size_t attn_shared_workspace_bytes(int n_rows, int hq, int hkv, int hd, int ctx, int prefix_pages) {
  return ws_layout(n_rows, hq, hkv, hd, ctx, prefix_pages, nullptr, nullptr);
}

template <int HD>
static void attn_f32_go(dim3 grid, hipStream_t st, const void* q, const void* k, const void* v,
                        const int32_t* pt, int pts, CtxSpec cs, int hq, int hkv, int cp, AttnWs w,
                        void* out) {
  hipLaunchKernelGGL(attn_f32_kernel<HD>, grid, dim3(256), 0, st, (const float*)q,
                     (const float*)k, (const float*)v, pt, pts, cs, hq, hkv, cp, w.work,
                     w.chunk_off, w.info, w.ws_o, w.ws_ml, (float*)out);
}

// uniform: every row has the same context (cs.ctx_len == NULL, cs.mod == 0)
hipError_t launch_attention_spec(const void* q, const void* k_pool, const void* v_pool,
                                 const int32_t* page_table, int pt_stride, CtxSpec cs, int n_rows,
                                 int hq, int hkv, int hd, int max_ctx, bool bf16, void* out,
                                 void* ws, size_t ws_bytes, hipStream_t st, hipEvent_t ev0,
                                 hipEvent_t ev1) {
  if (n_rows <= 0) return hipSuccess;
  cs.max_ctx = max_ctx;
  cs.skip = 0;
  AttnWs w;
  const size_t need = ws_layout(n_rows, hq, hkv, hd, max_ctx, 0, (char*)ws, &w);
  if (ws == nullptr || ws_bytes < need) return hipErrorInvalidValue;
  const bool uniform = bf16 && cs.ctx_len == nullptr && cs.mod == 0;
  const int cp = choose_chunk_pages(n_rows, hq, hkv, max_ctx, uniform, hd);
  const int uni_nch = uniform ? ((min(cs.base, max_ctx) + cp * kPage - 1) / (cp * kPage)) : 0;
  if (!uniform)
    hipLaunchKernelGGL(attn_plan_kernel, dim3(1), dim3(1024), 0, st, cs, n_rows, cp * kPage,
                       w.chunk_off, w.work, w.info, (int64_t)(kNtKvBytes / (4.0 * hkv * hd)));
  const int64_t maxch = uniform ? (int64_t)n_rows * uni_nch
                                : (int64_t)n_rows * ((max_ctx + cp * kPage - 1) / (cp * kPage));
  const int64_t items = maxch * (bf16 ? hkv : hq);
  int64_t blocks = (items + 3) / 4;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  const dim3 grid((unsigned)blocks);
  if (bf16) {
    AttnBf16Args a;
    a.q = (const bf16_t*)q; a.kpool = (const bf16_t*)k_pool; a.vpool = (const bf16_t*)v_pool;
    a.page_table = page_table; a.pt_stride = pt_stride; a.cs = cs; a.hq = hq; a.hkv = hkv;
    a.chunk_pages = cp; a.n_rows = n_rows; a.uniform_nch = uni_nch;
    a.work = w.work; a.chunk_off = w.chunk_off; a.info = w.info;
    a.ws_o = w.ws_o; a.ws_ml = w.ws_ml; a.out = (bf16_t*)out;
    a.pre_o = nullptr; a.pre_ml = nullptr; a.pre_nch = 0;
    if (ev0) (void)hipEventRecord(ev0, st);
    if (hd == 128) hipLaunchKernelGGL(attn_bf16_kernel<128>, grid, dim3(256), 0, st, a);
    else if (hd == 64) hipLaunchKernelGGL(attn_bf16_kernel<64>, grid, dim3(256), 0, st, a);
    else if (hd == 32) hipLaunchKernelGGL(attn_bf16_kernel<32>, grid, dim3(256), 0, st, a);
    else return hipErrorInvalidValue;
    if (ev1) (void)hipEventRecord(ev1, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((uniform ? uni_nch : (max_ctx + cp * kPage - 1) / (cp * kPage)) > 1) {
      const int64_t nb = ((int64_t)n_rows * hq + 3) / 4;
      hipLaunchKernelGGL(attn_combine_kernel<bf16_t>, dim3((unsigned)nb), dim3(256), 0, st, cs,
                         n_rows, hq, hd, cp * kPage, uni_nch, w.chunk_off, w.ws_o, w.ws_ml,
                         (bf16_t*)out);
      e = hipGetLastError();
    }
    return e;
  }
  if (hd == 128) attn_f32_go<128>(grid, st, q, k_pool, v_pool, page_table, pt_stride, cs, hq, hkv, cp, w, out);
  else if (hd == 64) attn_f32_go<64>(grid, st, q, k_pool, v_pool, page_table, pt_stride, cs, hq, hkv, cp, w, out);
  else if (hd == 32) attn_f32_go<32>(grid, st, q, k_pool, v_pool, page_table, pt_stride, cs, hq, hkv, cp, w, out);
  else return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((max_ctx + cp * kPage - 1) / (cp * kPage) > 1) {
    const int64_t nb = ((int64_t)n_rows * hq + 3) / 4;
    hipLaunchKernelGGL(attn_combine_kernel<float>, dim3((unsigned)nb), dim3(256), 0, st, cs,
                       n_rows, hq, hd, cp * kPage, 0, w.chunk_off, w.ws_o, w.ws_ml, (float*)out);
    e = hipGetLastError();
  }
  return e;
}

template <int HD>
static void attn_shared_go(dim3 gpre, dim3 grow, hipStream_t st, const AttnPrefixArgs& p,
                           const AttnBf16Args& a) {
  hipLaunchKernelGGL(attn_prefix_kernel<HD>, gpre, dim3(256), 0, st, p);
  hipLaunchKernelGGL(attn_bf16_kernel<HD>, grow, dim3(256), 0, st, a);
}

hipError_t launch_attention_shared(const void* q, const void* k_pool, const void* v_pool,
                                   int64_t n_pages, const int32_t* page_table, int pt_stride,
                                   const int32_t* row_traj, int pt_rows, int m, int prefix_pages,
                                   bool build_groups, int ctx, int n_rows, int hq, int hkv, int hd,
                                   void* out, void* ws, size_t ws_bytes, hipStream_t st,
                                   hipEvent_t ev0, hipEvent_t ev1, int32_t* n_groups_out) {
  if (n_rows <= 0) return hipSuccess;
  const int G = hq / hkv;
  if (prefix_pages < 1 || ctx <= prefix_pages * kPage || m < 1 || G < 1 || G > 16 || hq % hkv)
    return hipErrorInvalidValue;
  if (!(hd == 32 || hd == 64 || hd == 128)) return hipErrorInvalidValue;
  AttnWs w;
  const size_t need = ws_layout(n_rows, hq, hkv, hd, ctx, prefix_pages, (char*)ws, &w);
  if (ws == nullptr || ws_bytes < need) return hipErrorInvalidValue;
  CtxSpec cs;
  cs.ctx_len = nullptr; cs.mod = 0; cs.base = ctx; cs.row_pt = row_traj; cs.max_ctx = ctx;
  cs.n_pages = n_pages; cs.skip = prefix_pages * kPage; cs.pt_rows = pt_rows;
  cs.nt_from = prefix_pages;
  if (build_groups)
    hipLaunchKernelGGL(attn_groups_kernel, dim3(1), dim3(1024), 0, st, row_traj, n_rows, m, w.grp_row0,
                       w.grp_n, w.n_groups, n_groups_out);
  AttnPrefixArgs p;
  p.q = (const bf16_t*)q; p.kpool = (const bf16_t*)k_pool; p.vpool = (const bf16_t*)v_pool;
  p.page_table = page_table; p.pt_stride = pt_stride; p.cs = cs; p.hq = hq; p.hkv = hkv;
  p.prefix_pages = prefix_pages; p.chunk_pages = kPrefixChunkPages;
  p.pre_nch = (prefix_pages + kPrefixChunkPages - 1) / kPrefixChunkPages;
  p.qblocks = (m * G + 15) / 16;
  p.grp_row0 = w.grp_row0; p.grp_n = w.grp_n; p.n_groups = w.n_groups;
  p.pre_o = w.pre_o; p.pre_ml = w.pre_ml;
  // at most n_rows groups
  int64_t pre_items = (int64_t)std::min(n_rows, (n_rows + m - 1) / m + n_rows) * hkv * p.qblocks * p.pre_nch;
  int64_t gpre = std::min<int64_t>(std::max<int64_t>((pre_items + 3) / 4, 1), 2048);
  // per-row kernel over the keys after the prefix
  const int span = ctx - cs.skip;
  const int cp = choose_chunk_pages(n_rows, hq, hkv, span, true, hd);
  const int nch = (span + cp * kPage - 1) / (cp * kPage);
  if ((int64_t)n_rows * nch > w.max_chunks) return hipErrorInvalidValue;
  AttnBf16Args a;
  a.q = (const bf16_t*)q; a.kpool = (const bf16_t*)k_pool; a.vpool = (const bf16_t*)v_pool;
  a.page_table = page_table; a.pt_stride = pt_stride; a.cs = cs; a.hq = hq; a.hkv = hkv;
  a.chunk_pages = cp; a.n_rows = n_rows; a.uniform_nch = nch;
  a.work = w.work; a.chunk_off = w.chunk_off; a.info = w.info;
  a.ws_o = w.ws_o; a.ws_ml = w.ws_ml; a.out = (bf16_t*)out;
  a.pre_o = w.pre_o; a.pre_ml = w.pre_ml; a.pre_nch = p.pre_nch;
  const int64_t items = (int64_t)n_rows * nch * hkv;
  const int64_t grow = std::min<int64_t>(std::max<int64_t>((items + 3) / 4, 1), 2048);
  if (ev0) (void)hipEventRecord(ev0, st);
  if (hd == 128) attn_shared_go<128>(dim3((unsigned)gpre), dim3((unsigned)grow), st, p, a);
  else if (hd == 64) attn_shared_go<64>(dim3((unsigned)gpre), dim3((unsigned)grow), st, p, a);
  else attn_shared_go<32>(dim3((unsigned)gpre), dim3((unsigned)grow), st, p, a);
  if (ev1) (void)hipEventRecord(ev1, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nch > 1) {
    const int64_t nb = ((int64_t)n_rows * hq + 3) / 4;
    hipLaunchKernelGGL(attn_combine_kernel<bf16_t>, dim3((unsigned)nb), dim3(256), 0, st, cs,
                       n_rows, hq, hd, cp * kPage, nch, w.chunk_off, w.ws_o, w.ws_ml, (bf16_t*)out);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_attention(const void* q, const void* k_pool, const void* v_pool,
                            int64_t n_pages, const int32_t* page_table, int pt_stride,
                            const int32_t* row_pt, const int32_t* ctx_len, int ctx_mod,
                            int ctx_base, int n_rows, int hq, int hkv, int hd, int max_ctx,
                            bool bf16, void* out, void* ws, size_t ws_bytes, hipStream_t st,
                            hipEvent_t ev0, hipEvent_t ev1, int shared_pages) {
  CtxSpec cs;
  // Non-temporal loads of what no other row reads (streams run at 7.0 TB/s with
  // them, at 6.3 without): in a rollout the pages after the prompt's, since the
  // other layers pass through the caches before a layer is read again.  A
  // stateless call's rows may share pages, which the kernel looks at, and below
  // the size of the Infinity Cache a caller that comes back with the same pools
  // finds them there (6 rows of 6000 keys: 25.9 us, non-temporal 28.0).
  // (Ragged rows: by the sum of their contexts, on the device; 1024 rows of
  // median 60 keys, 32/4 heads x 128, 173 MB under a bound of 3 GB, read again:
  // 101 us, non-temporal 114.)
  const double kv_bytes = 4.0 * n_rows * hkv * hd * max_ctx;
  cs.nt_from = row_pt ? shared_pages : kv_bytes >= kNtKvBytes ? -1 : INT32_MAX;
  cs.ctx_len = ctx_len; cs.mod = ctx_mod; cs.base = ctx_base; cs.row_pt = row_pt;
  cs.max_ctx = max_ctx; cs.n_pages = n_pages; cs.skip = 0; cs.pt_rows = 0;
  return launch_attention_spec(q, k_pool, v_pool, page_table, pt_stride, cs, n_rows, hq, hkv, hd,
                               max_ctx, bf16, out, ws, ws_bytes, st, ev0, ev1);
}

}  // namespace darts
