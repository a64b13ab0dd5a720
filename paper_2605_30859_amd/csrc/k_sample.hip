// Fused sampler: one pass over a logits row computes
//   * the Gumbel-max token  argmax_i fl32(z_i + g_i),  z = logits / T,
//     g_i = -ln(-ln u_i), u_i from Philox(counter=(i>>2, traj, step, TAG_SAMPLE),
//     key=seed), ties to the smallest index;
//   * log-sum-exp and entropy with an online (max, sum e^(z-m), sum e^(z-m)(z-m))
//     state merged across lanes and wavefronts;
// then the log-prob of the taken token.  In the stateful form the same block
// applies the exogenous termination rule (forced end-of-sequence length,
// truncation at cap) and accumulates the trajectory's score.  When few rows
// are live (given room for partials), a row's vocabulary is split into
// slices, one block each, and a finalize kernel merges the slices' states
// and winners before finishing the row.
//
// Filtered argmax.  g_i is defined by the library's exact float32 logarithm
// (two per element, each with a correctly rounded division), which would
// dominate the kernel's arithmetic.  The scan instead drops every element that
// a threshold shows to be no winner (sample_kernel) and takes the exact score
// of the few that are left, so the token is the exact-map argmax, bit for bit.
// The first threshold comes from a fast map (two hardware log2 evaluations)
// whose distance from the exact map is at most kGumbelFastBound over all 2^23
// possible u (checked exhaustively on the device by the test suite).
//
// Bound by VALU issue: Philox (17 64-bit products per 4 logits), one
// exponential per logit, the softmax sums.  1024 x 151936 bf16 logits take
// 135 us (about 95 vector instructions per 4 logits and lane, 17 of them 64-bit
// products and 4 exponentials), against 325 us when every element's fast score was evaluated,
// each thread's best two compared and the division by T computed for T = 1 too.
#include <math.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace darts {

struct SoftState {
  float m, s, t;   // max, sum e^(z-m), sum e^(z-m)(z-m)
};
__device__ __forceinline__ SoftState soft_merge(SoftState a, SoftState b) {
  if (a.m == -INFINITY) return b;
  if (b.m == -INFINITY) return a;
  const float m = fmaxf(a.m, b.m);
  const float ea = __expf(a.m - m), eb = __expf(b.m - m);
  SoftState r;
  r.m = m;
  r.s = a.s * ea + b.s * eb;
  r.t = ea * (a.t + a.s * (a.m - m)) + eb * (b.t + b.s * (b.m - m));
  return r;
}
struct Best {
  float v;
  int i;
};
__device__ __forceinline__ Best best_merge(Best a, Best b) {
  if (b.v > a.v || (b.v == a.v && b.i < a.i)) return b;
  return a;
}

// Four consecutive logits as they are in memory, and as floats.
template <bool BF16>
struct Raw4 {
  uint2 v;
  __device__ __forceinline__ void load(const void* row, int j) { v = ((const uint2*)row)[j]; }
  __device__ __forceinline__ void get(float z[4]) const {
    z[0] = __uint_as_float(v.x << 16);
    z[1] = __uint_as_float(v.x & 0xffff0000u);
    z[2] = __uint_as_float(v.y << 16);
    z[3] = __uint_as_float(v.y & 0xffff0000u);
  }
};
template <>
struct Raw4<false> {
  float4 v;
  __device__ __forceinline__ void load(const void* row, int j) { v = ((const float4*)row)[j]; }
  __device__ __forceinline__ void get(float z[4]) const { z[0] = v.x; z[1] = v.y; z[2] = v.z; z[3] = v.w; }
};

// Fast Gumbel map: -ln(-ln u) from two hardware log2 evaluations (the only
// approximation; products by ln 2 in float32).  u in [2^-24, 1 - 2^-24]
// keeps both log2 arguments normal.
__device__ __forceinline__ float gumbel_fast(float u) {
  constexpr float kLn2 = 0.693147180559945309f;
  const float a = -kLn2 * __builtin_amdgcn_logf(u);
  return -kLn2 * __builtin_amdgcn_logf(a);
}
// |gumbel_fast(u) - gumbel_of(u)| <= kGumbelFastBound for every u the sampler
// draws (measured maximum 1.9e-6; the bound is 2^-17)
constexpr float kGumbelFastBound = 7.62939453125e-06f;

template <bool BF16>
__device__ __forceinline__ float logit_at(const void* row, int i, bool tscale, float temperature) {
  float z = BF16 ? bf16_to_f32(((const bf16_t*)row)[i]) : ((const float*)row)[i];
  return tscale ? __fdiv_rn(z, temperature) : z;
}

// Per-row values every part of a row shares.
struct RowCtx {
  int g, step;
  const void* row;
};
template <bool BF16, bool STATEFUL>
__device__ __forceinline__ RowCtx row_ctx(const SampleArgs& a, int r) {
  RowCtx c;
  c.g = a.traj[r];
  const int lrow = a.row_logit ? a.row_logit[r] : (a.logit_div > 0 ? c.g / a.logit_div : r);
  c.row = BF16 ? (const void*)((const bf16_t*)a.logits + (int64_t)lrow * a.vocab)
               : (const void*)((const float*)a.logits + (int64_t)lrow * a.vocab);
  c.step = STATEFUL ? a.gen[c.g] : a.step[r];
  return c;
}

// Row r's result from its merged softmax state and Gumbel-max winner: the
// taken token (forced end of sequence, teacher forcing), its log-prob, the
// entropy and, in the stateful form, termination and score accumulation.
template <bool BF16, bool STATEFUL>
__device__ __forceinline__ void finish_row(const SampleArgs& a, int r, const RowCtx& c, SoftState st,
                                           Best best) {
  const int g = c.g, step = c.step;
  // A row with no finite perturbed score (every logit -inf or NaN) has no
  // Gumbel-max winner: token 0 stands in (the lowest index, as for equal
  // scores), and its log-prob and entropy are NaN.
  const bool has_winner = best.i >= 0 && best.i < a.vocab;
  const float lse = st.m + logf(st.s);
  const float ent = has_winner ? logf(st.s) - st.t / st.s : NAN;
  const int sampled = has_winner ? best.i : 0;
  int taken = sampled;
  uint8_t fin = 0;
  if (STATEFUL) {
    const int s_new = step + 1;
    const int d = a.forced_len[g];
    if (d <= a.cap && s_new == d) { taken = a.eos; fin = 1; }
    else {
      if (a.force && a.force[g] >= 0) taken = a.force[g];
      if (s_new >= a.cap) fin = 2;
    }
  } else if (a.force && a.force[r] >= 0) {
    taken = a.force[r];
  }
  if (taken < 0 || taken >= a.vocab) taken = sampled;   // sampled is in [0, vocab)
  const float zt = logit_at<BF16>(c.row, taken, a.temperature != 1.0f, a.temperature);
  const float lp = has_winner ? zt - lse : NAN;
  if (a.token_out) a.token_out[r] = taken;
  if (a.sampled_out) a.sampled_out[r] = sampled;
  if (a.logprob_out) a.logprob_out[r] = lp;
  if (a.entropy_out) a.entropy_out[r] = ent;
  if (STATEFUL) {
    if (a.hist_tok && step < a.cap) {
      a.hist_tok[(int64_t)g * a.cap + step] = taken;
      a.hist_lp[(int64_t)g * a.cap + step] = lp;
    }
    a.gen[g] = step + 1;
    a.sum_lp[g] = a.sum_lp[g] + lp;
    a.last_tok[g] = taken;
    if (fin) a.status[g] = fin;
    if (a.finished_out) a.finished_out[r] = fin;
    if (a.traj_out) a.traj_out[r] = g;
  }
}

// Block (r, part): part `part` of the a.parts contiguous slices of row r's
// vocabulary.  With one part the block finishes the row; with several it
// writes its partial (softmax state, winner) and the finalize kernel merges
// the parts.
//
// The scan filters the elements by a threshold T, the largest exact score (or
// a bound just below a fast one) that the block has seen so far: an element can
// only be the winner if z + g >= T.  Since -ln u >= 1 - u, that needs
//   1 - u <= exp(z - T) = e^(z-m) * e^(m-T),
// and e^(z-m) is at hand from the softmax sums, so the test is a conversion, a
// fused multiply-add and a comparison per element instead of two logarithms.
// Whatever passes (about one element in a few thousand once T has settled) gets
// its exact score.  kSlackAbs + kSlackRel |T| on the exponent covers the
// float32 errors: the noise map's 2e-6, the rounding of z + g (2^-24 |T|), of
// both exponentials' arguments (at most 20 in magnitude where the outcome
// matters: g <= 16.7 and T >= m - 2.9) and of the words' conversion (kWordSlack).
constexpr float kSlackAbs = 1.953125e-03f;       // 2^-9
constexpr float kSlackRel = 4.76837158203125e-07f;   // 2^-21
constexpr float kWordSlack = 1024.0f;            // in units of the 32-bit word, which rounds to 256

// float <-> int keys of the same order (NaN never gets here)
__device__ __forceinline__ int order_key(float f) {
  const int b = __float_as_int(f);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_order(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }

// Division by the temperature: none (1), by a correctly rounded reciprocal with
// one fused correction, or the full division.  q = z y with y = RN(1/T), then
// RN(q + (z - q T) y) is the correctly rounded quotient while nothing
// over- or underflows and T's significand is not all ones (Markstein's
// theorem); other temperatures, and groups with a logit outside
// [2^-100, 2^100], take the full division, which costs as much as Philox.
enum { T_ONE, T_RECIP, T_FULL };
template <bool BF16, bool STATEFUL, int THREADS, int TMODE>
__global__ void __launch_bounds__(THREADS) sample_kernel(SampleArgs a) {
  constexpr int NW = THREADS / 64;
  __shared__ SoftState ss[NW];
  __shared__ Best sb[NW];
  __shared__ int s_thr;                          // the block's T, as an order key
  const int parts = a.parts > 1 ? a.parts : 1;
  const int r = blockIdx.x / parts, part = blockIdx.x - r * parts;
  const int tid = threadIdx.x;
  if (tid == 0) s_thr = (int)0x807fffff;          // -INFINITY
  const RowCtx c = row_ctx<BF16, STATEFUL>(a, r);
  const int g = c.g, step = c.step;
  const uint32_t gc = (uint32_t)g + (uint32_t)a.traj_base;   // the counter's (global) trajectory id
  const void* row = c.row;
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  SoftState st = {-INFINITY, 0.f, 0.f};
  Best best = {-INFINITY, 0x7fffffff};           // this thread's best exact score
  const int n4 = a.vocab >> 2;
  const int span = (n4 + parts - 1) / parts;
  const int jb = part * span, je = min(n4, jb + span);
  constexpr int kNone = (int)0x807fffff;         // order_key(-INFINITY)
  int thr = kNone;                               // T as this thread knows it
  float lim = 0.f;                               // 2^32 e^(m - T + slack), finite; 0 while m is -inf
  auto set_lim = [&]() {
    const float T = key_order(thr);
    const float x = 4294967296.0f * __expf(st.m - T + (kSlackAbs + kSlackRel * fabsf(T)));
    lim = st.m == -INFINITY ? 0.f : fminf(x, 3.0e38f);      // also when x is NaN (an infinite logit)
  };
  auto block_thr = [&]() { return __hip_atomic_load(&s_thr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  Raw4<BF16> next;
  if (jb + tid < je) next.load(row, jb + tid);
  __syncthreads();                               // s_thr, while the first loads are under way
  for (int j = jb + tid; j < je; j += THREADS) {
    float z[4];
    next.get(z);
    int known = block_thr();                     // read early; any earlier T is as sound
    if (j + THREADS < je) next.load(row, j + THREADS);
    if constexpr (TMODE != T_ONE) {
      constexpr float kBig = 1.2676506e+30f, kSmall = 7.8886091e-31f;   // 2^100, 2^-100
      const float hi = fmaxf(fmaxf(fabsf(z[0]), fabsf(z[1])), fmaxf(fabsf(z[2]), fabsf(z[3])));
      const float lo = fminf(fminf(fabsf(z[0]), fabsf(z[1])), fminf(fabsf(z[2]), fabsf(z[3])));
      if (TMODE == T_RECIP && hi <= kBig && lo >= kSmall) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float q = z[e] * a.inv_temperature;
          z[e] = fmaf(fmaf(-q, a.temperature, z[e]), a.inv_temperature, q);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = __fdiv_rn(z[e], a.temperature);
      }
    }
    const Philox4 p = philox4x32_10((uint32_t)j, gc, (uint32_t)step, kTagSample, k0, k1);
    float word[4];       // the elements' word + lim e^(z-m)
    float top = 0.f;     // the largest of them
    const float lm = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
    bool moved = false;
    if (lm > st.m) {
      if (st.s > 0.f) {   // rescale the running sums to the new maximum
        const float sc = __expf(st.m - lm);
        st.t = sc * (st.t + st.s * (st.m - lm));
        st.s = st.s * sc;
      }
      st.m = lm;
      moved = true;
      if (lm == INFINITY) top = 4294967296.0f;   // only the first infinite logit can win
    }
    if (known == kNone) {
      // nothing seen yet: T from the fast scores of this group, less their error
      float f = -INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) f = fmaxf(f, z[e] + gumbel_fast(open_unit(p.x[e])));
      f -= 2.0f * (kGumbelFastBound + 2.384185791015625e-07f * fabsf(f));
      if (f > -INFINITY) atomicMax(&s_thr, order_key(f));
      known = block_thr();
    }
    if (known > thr || moved) {
      thr = max(thr, known);
      set_lim();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // masked (-inf) logits add nothing: d clamps to -FLT_MAX (also when the
      // running max is still -inf), so e^d = 0 and the entropy term 0 * d = 0
      const float d = fmaxf(z[e] - st.m, -3.40282347e+38f);
      const float ez = __expf(d);
      st.s += ez;
      st.t = fmaf(ez, d, st.t);
      word[e] = fmaf(ez, lim, (float)p.x[e]);
    }
    const float forced = top;
    top = fmaxf(fmaxf(fmaxf(word[0], word[1]), fmaxf(word[2], word[3])), forced);
    if (top >= 4294967296.0f - kWordSlack) {
      const float before = best.v;
      // the elements that pass, one at a time: early in a row every wavefront gets
      // here, but mostly for one of a lane's four (a row of 4096 fp32 logits, four
      // groups per lane: 7.1 us, with all four every time 8.0; evaluating the fast
      // map for every element and the exact one once at the end: 6.4, which 200
      // rows pay for with 16.2 against 9.2)
      uint32_t pass = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) pass |= (fmaxf(word[e], forced) >= 4294967296.0f - kWordSlack ? 1u : 0u) << e;
#pragma unroll 1
      for (; pass; pass &= pass - 1) {
        const int e = __ffs(pass) - 1;
        const uint32_t x = e == 0 ? p.x[0] : e == 1 ? p.x[1] : e == 2 ? p.x[2] : p.x[3];
        const float sc = (e == 0 ? z[0] : e == 1 ? z[1] : e == 2 ? z[2] : z[3]) + gumbel_of(open_unit(x));
        if (sc > best.v) { best.v = sc; best.i = 4 * j + e; }
      }
      if (best.v > before) atomicMax(&s_thr, order_key(best.v));
    }
  }
  // wavefront merge
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    SoftState other = {__shfl_xor(st.m, o, 64), __shfl_xor(st.s, o, 64), __shfl_xor(st.t, o, 64)};
    st = soft_merge(st, other);
    Best ob = {__shfl_xor(best.v, o, 64), __shfl_xor(best.i, o, 64)};
    best = best_merge(best, ob);
  }
  if ((tid & 63) == 0) { ss[tid >> 6] = st; sb[tid >> 6] = best; }
  __syncthreads();
  if (tid != 0) return;
  // pairs of wavefronts, then pairs of pairs
#pragma unroll
  for (int o = 1; o < NW; o <<= 1)
#pragma unroll
    for (int i = 0; i + o < NW; i += 2 * o) {
      ss[i] = soft_merge(ss[i], ss[i + o]);
      sb[i] = best_merge(sb[i], sb[i + o]);
    }
  st = ss[0];
  best = sb[0];
  if (parts > 1) {
    SamplePart o;
    o.m = st.m; o.s = st.s; o.t = st.t; o.v = best.v; o.i = best.i;
    a.part_out[blockIdx.x] = o;
    return;
  }
  finish_row<BF16, STATEFUL>(a, r, c, st, best);
}

// One wavefront per row: lane l merges parts l, l + 64 (in that order), the
// lanes are then merged by a fixed butterfly (a fixed order, so the result
// is reproducible), and lane 0 finishes the row.
template <bool BF16, bool STATEFUL>
__global__ void __launch_bounds__(256) sample_finalize_kernel(SampleArgs a) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= a.n_rows) return;
  SoftState st = {-INFINITY, 0.f, 0.f};
  Best best = {-INFINITY, 0x7fffffff};
  for (int p = lane; p < a.parts; p += 64) {
    const SamplePart o = a.part_out[(int64_t)r * a.parts + p];
    st = soft_merge(st, SoftState{o.m, o.s, o.t});
    best = best_merge(best, Best{o.v, o.i});
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    SoftState other = {__shfl_xor(st.m, o, 64), __shfl_xor(st.s, o, 64), __shfl_xor(st.t, o, 64)};
    st = soft_merge(st, other);
    Best ob = {__shfl_xor(best.v, o, 64), __shfl_xor(best.i, o, 64)};
    best = best_merge(best, ob);
  }
  if (lane == 0) finish_row<BF16, STATEFUL>(a, r, row_ctx<BF16, STATEFUL>(a, r), st, best);
}

int sample_parts(int n_rows, int vocab) {
  // about kSampleBlocks blocks in all, each part at least kSampleMinGroups
  // groups of 4 logits (two per thread), at most kSampleMaxParts per row
  const int n4 = vocab >> 2;
  int parts = (kSampleBlocks + n_rows - 1) / n_rows;
  parts = std::min(parts, std::max(1, n4 / kSampleMinGroups));
  return std::max(1, std::min(parts, kSampleMaxParts));
}

hipError_t launch_sample(const SampleArgs& a0, hipStream_t st) {
  if (a0.n_rows <= 0) return hipSuccess;
  SampleArgs a = a0;
  a.parts = a.part_out ? sample_parts(a.n_rows, a.vocab) : 1;
  if (a.parts > 1 && (int64_t)a.n_rows * a.parts > a.part_cap) a.parts = 1;
  const bool stateful = a.gen != nullptr;
  const dim3 grid((unsigned)(a.n_rows * a.parts));
  const dim3 gfin((unsigned)((a.n_rows + 3) / 4));
  // Without room for partials a row is one block: of 16 wavefronts instead of 4
  // while two such blocks per CU hold every row and each thread still gets a
  // few groups (21 rows of 151936, T = 0.7: 45 against 104 us; from 513 rows on the blocks of 4
  // wavefronts fill the card and their ends overlap).
  const bool wide = a.parts == 1 && a.n_rows <= kSampleWideRows && (a.vocab >> 2) >= kSampleWideGroups;
  uint32_t tbits;
  std::memcpy(&tbits, &a.temperature, 4);
  const bool recip = a.temperature >= 9.5367432e-07f && a.temperature <= 1048576.0f &&   // 2^-20 .. 2^20
                     (tbits & 0x7fffffu) != 0x7fffffu;
  a.inv_temperature = 1.0f / a.temperature;
  auto go_t = [&](auto BF, auto ST, auto TS) {
    constexpr bool bf = decltype(BF)::value, sf = decltype(ST)::value;
    constexpr int ts = decltype(TS)::value;
    if (wide) hipLaunchKernelGGL((sample_kernel<bf, sf, 1024, ts>), grid, dim3(1024), 0, st, a);
    else hipLaunchKernelGGL((sample_kernel<bf, sf, 256, ts>), grid, dim3(256), 0, st, a);
  };
  auto go = [&](auto BF, auto ST) {
    constexpr bool bf = decltype(BF)::value, sf = decltype(ST)::value;
    if (a.temperature == 1.0f) go_t(BF, ST, std::integral_constant<int, T_ONE>{});
    else if (recip) go_t(BF, ST, std::integral_constant<int, T_RECIP>{});
    else go_t(BF, ST, std::integral_constant<int, T_FULL>{});
    if (a.parts > 1) hipLaunchKernelGGL((sample_finalize_kernel<bf, sf>), gfin, dim3(256), 0, st, a);
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  if (a.bf16) {
    if (stateful) go(yes, yes);
    else go(yes, no);
  } else {
    if (stateful) go(no, yes);
    else go(no, no);
  }
  return hipGetLastError();
}

}  // namespace darts

namespace darts {
__global__ void gumbel_map_kernel(const float* __restrict__ u, float* __restrict__ g, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    g[i] = gumbel_of(u[i]);
}
__global__ void gumbel_fast_map_kernel(const float* __restrict__ u, float* __restrict__ g, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    g[i] = gumbel_fast(u[i]);
}
hipError_t launch_gumbel_map(const float* u, float* g, int64_t n, bool fast, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (fast) hipLaunchKernelGGL(gumbel_fast_map_kernel, dim3((unsigned)blocks), dim3(256), 0, st, u, g, n);
  else hipLaunchKernelGGL(gumbel_map_kernel, dim3((unsigned)blocks), dim3(256), 0, st, u, g, n);
  return hipGetLastError();
}
float gumbel_fast_bound() { return kGumbelFastBound; }
}  // namespace darts
