// Selection kernels: top-F bonus-token candidates per accept length (Sec. 4.1.1), the branch sampler
// (argmax / Gumbel-max), and lossless verification (Sec. 2.1).  All orderings are (score descending,
// token id ascending); NaN ranks below every number.
#include <mutex>

#include "common.h"
#include "lanes.h"
#include "rng.h"

namespace ssd {

namespace {

constexpr int kSelBlock = 1024;
constexpr int kSelWaves = kSelBlock / 64;

// 64-bit sort key of (fp32 logit, token id): larger key = better candidate.
__device__ __forceinline__ uint64_t make_key(float f, int id) {
  uint32_t hi;
  if (f != f) hi = 0u;                              // NaN: below -inf
  else {
    if (f == 0.f) f = 0.f;                          // -0 and +0 tie
    uint32_t u = __float_as_uint(f);
    hi = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  }
  return ((uint64_t)hi << 32) | (uint32_t)(~(uint32_t)id);
}
__device__ __forceinline__ int key_id(uint64_t k) { return (int)(~(uint32_t)k); }

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  return lanes_reduce(v, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
}

// One block per row.  Every thread keeps the best FMAX keys of its strided share in sorted registers; then F
// rounds of a block-wide maximum over the threads' current heads pick the row's top F in order.
// groups == 0: every row takes F ids, stored at ids[row][F].  groups == K+1 (the fan-out of a round, Sec. 4.1.1 with
// the cache shape of Sec. 4.1.2): row (b, k) takes F_k ids, stored at ids[b][off[k] ..].
// gridDim.y > 1: the vocabulary is cut into gridDim.y parts, block (row, part) leaves the sorted keys of its part's
// top F in part_keys[row][part][FMAX] and top_f_merge_kernel picks the row's top F among them (keys are unique, so
// the result is the same as that of one block).
constexpr int kTopFMaxParts = 32;
template <int FMAX>
__global__ __launch_bounds__(kSelBlock) void top_f_kernel(const float* __restrict__ logits, int64_t ld,
                                                          const int32_t* __restrict__ exclude, int V, int F, int groups,
                                                          FanTable fan, int32_t* __restrict__ ids,
                                                          uint64_t* __restrict__ part_keys) {
  __shared__ uint64_t wave_best[kSelWaves];
  __shared__ uint64_t round_best;
  const int row = blockIdx.x;
  const int parts = gridDim.y, part = blockIdx.y;
  int32_t* out = ids + (int64_t)row * F;
  if (groups > 0) {
    const int b = row / groups, k = row - b * groups;
    F = fan.off[k + 1] - fan.off[k];
    out = ids + (int64_t)b * fan.off[groups] + fan.off[k];
  }
  const int chunk = (V + parts - 1) / parts;
  const int lo = part * chunk, hi = lo + chunk < V ? lo + chunk : V;
  const float* z = logits + (int64_t)row * ld;
  const int ex = exclude ? exclude[row] : -1;
  uint64_t best[FMAX];
#pragma unroll
  for (int i = 0; i < FMAX; ++i) best[i] = 0ull;    // 0 is below every real key (ids < 2^32-1)
  auto offer = [&](float v, int t) {
    if (t == ex) return;
    uint64_t k = make_key(v, t);
    if (k > best[FMAX - 1]) {
      best[FMAX - 1] = k;
#pragma unroll
      for (int i = FMAX - 1; i > 0; --i) {
        if (best[i] > best[i - 1]) { uint64_t tmp = best[i]; best[i] = best[i - 1]; best[i - 1] = tmp; }
      }
    }
  };
  // eight loads in flight per thread: one dependent load per iteration would cost a memory latency each
  constexpr int U = 8;
  for (int t0 = lo + threadIdx.x; t0 < hi; t0 += kSelBlock * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * kSelBlock;
      v[u] = z[t < hi ? t : t0];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * kSelBlock;
      if (t < hi) offer(v[u], t);
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int f = 0; f < F; ++f) {
    uint64_t w = wave_max_u64(best[0]);
    if (lane == 0) wave_best[wave] = w;
    __syncthreads();
    if (wave == 0) {
      uint64_t v = lane < kSelWaves ? wave_best[lane] : 0ull;
      v = wave_max_u64(v);
      if (lane == 0) {
        round_best = v;
        if (parts == 1) out[f] = key_id(v);
        else part_keys[((int64_t)row * parts + part) * FMAX + f] = v;     // 0 when the part ran out of tokens
      }
    }
    __syncthreads();
    if (best[0] == round_best) {                    // keys are unique: exactly one thread pops
#pragma unroll
      for (int i = 0; i < FMAX - 1; ++i) best[i] = best[i + 1];
      best[FMAX - 1] = 0ull;
    }
  }
}

// One wavefront per row: the top F of the parts' candidates.  Keys are unique and positive, 0 marks "none".
template <int FMAX>
__global__ __launch_bounds__(64) void top_f_merge_kernel(const uint64_t* __restrict__ part_keys, int parts, int F, int groups,
                                                          FanTable fan, int32_t* __restrict__ ids) {
  const int row = blockIdx.x, lane = threadIdx.x;
  int32_t* out = ids + (int64_t)row * F;
  if (groups > 0) {
    const int b = row / groups, k = row - b * groups;
    F = fan.off[k + 1] - fan.off[k];
    out = ids + (int64_t)b * fan.off[groups] + fan.off[k];
  }
  constexpr int PER = kTopFMaxParts * FMAX / 64;      // candidates per lane
  uint64_t mine[PER];
  const int n = parts * F;                            // part p holds its F best at [p][0..F-1]
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int c = lane + 64 * i;
    mine[i] = c < n ? part_keys[((int64_t)row * parts + c / F) * FMAX + c % F] : 0ull;
  }
  uint64_t prev = ~0ull;
  for (int f = 0; f < F; ++f) {
    uint64_t best = 0ull;
#pragma unroll
    for (int i = 0; i < PER; ++i) best = mine[i] < prev && mine[i] > best ? mine[i] : best;
    best = wave_max_u64(best);
    if (lane == 0) out[f] = key_id(best);
    prev = best;
  }
}

struct ScoreId {
  double s;
  int id;
};
// The sampler's rows are shared among small blocks: a block of 1024 threads waits with all 16 wavefronts for the slowest of them, and
// only two fit a compute unit.  About 2048 blocks, of 1024 and 256 threads, us with the merge: 24 rows of 128256 at temperature
// 0.7 15.9 and 15.0, 48 rows 25.8 and 17.8 (greedy 16.9 and 10.2), 96 rows 41.0 and 25.4 (23.9 and 13.5), 384 rows 74 and 63 (greedy,
// logits not in the caches, 46.5 and 47.7); 512 threads lie between, 1024 or 4096 blocks of 256 measure 0 to 4 us more from 48 rows on.  A row of one block takes 1024.
constexpr int kSampleBlock = 256;
constexpr int kSampleMaxParts = 128;  // blocks that share one row of the sampler
__device__ __forceinline__ bool better(const ScoreId& a, const ScoreId& b) {
  return a.s > b.s || (a.s == b.s && a.id < b.id);
}
__device__ __forceinline__ ScoreId lanes_best(ScoreId v) {
  struct Packed { double s; int id, pad; };          // (whole registers)
  const Packed r = lanes_reduce(Packed{v.s, v.id, 0}, [](Packed a, Packed b) { return a.s > b.s || (a.s == b.s && a.id < b.id) ? a : b; });
  return {r.s, r.id};
}
template <int WAVES>
__device__ __forceinline__ ScoreId block_argmax(ScoreId v, ScoreId* smem) {
  v = lanes_best(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) smem[wave] = v;
  __syncthreads();
  ScoreId r = smem[0];
  for (int i = 1; i < WAVES; ++i)
    if (better(smem[i], r)) r = smem[i];
  __syncthreads();
  return r;
}
__device__ __forceinline__ double score_of(float z) { return z != z ? -INFINITY : (double)z; }

// Branch sampler: greedy argmax or Gumbel-max sample of softmax(z / T).  grid = (rows, parts): a block scans one
// part of its row's vocabulary; with one part it writes the token, otherwise its best (score, id) goes to `scratch`
// [row][part] and sample_merge_kernel picks the row's winner (the order `better` defines is total, so any grouping
// gives the same token).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void sample_kernel(const float* __restrict__ logits, int64_t ld,
                                                       const float* __restrict__ temperature, int rows_per_seq,
                                                       int V, uint64_t seed, int row_base, int step,
                                                       int32_t* __restrict__ out, int64_t out_stride,
                                                       ScoreId* __restrict__ scratch, int exact_scan) {
  __shared__ ScoreId smem[BLOCK / 64];
  const int row = blockIdx.x, part = blockIdx.y, parts = gridDim.y;
  const float* z = logits + (int64_t)row * ld;
  const double T = (double)temperature[row / rows_per_seq];
  const uint64_t prefix = draw_prefix(seed, STREAM_DRAFT, (uint64_t)(row_base + row), (uint64_t)step);
  // this block's share of the vocabulary, in groups of 4 tokens
  const int n4_all = (V + 3) >> 2;
  const int per = (n4_all + parts - 1) / parts;
  const int q_begin = part * per, q_end = min(n4_all, q_begin + per);
  ScoreId best = {-INFINITY, 0x7fffffff};
  if (T <= 0.0 && (V & 3) == 0 && (ld & 3) == 0 && ((uintptr_t)logits & 15) == 0) {
    // greedy rows: 16-byte loads, eight of them in flight per thread (one dependent 4-byte load per iteration
    // would cost a memory latency each)
    typedef __attribute__((ext_vector_type(4))) float f4;
    const f4* z4 = (const f4*)z;
    for (int t0 = q_begin + threadIdx.x; t0 < q_end; t0 += BLOCK * 8) {
      f4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        int t = t0 + u * BLOCK;
        v[u] = z4[t < q_end ? t : t0];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        int t = t0 + u * BLOCK;
        if (t < q_end) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ScoreId c = {score_of(v[u][e]), t * 4 + e};
            if (better(c, best)) best = c;
          }
        }
      }
    }
  } else if (T <= 0.0 || exact_scan) {
    const int t_end = min(V, q_end * 4);
    for (int t = q_begin * 4 + threadIdx.x; t < t_end; t += BLOCK) {
      ScoreId c;
      c.id = t;
      c.s = score_of(z[t]);
      if (T > 0.0) c.s = c.s / T + gumbel_from_u(draw_u(prefix, (uint64_t)t));
      if (better(c, best)) best = c;
    }
  } else {
    // Sampled rows.  The decision is the fp64 one (score = z / T + g in double, as specified), but two fp64 logarithms
    // per token of a 128256-token row cost more than the rest of the sampler together, so the scan runs in fp32 and
    // only the tokens that can still win are scored in fp64: with |s32 - s64| <= delta for every token near the top,
    // the fp64 winner t* has s32(t*) >= s64(t*) - delta >= s64(t32) - delta >= max32 - 2 delta.  delta: z / T in
    // fp32 is within 2^-22 |z / T|; u is exact in fp32 (a 24-bit odd integer times 2^-24); the hardware's base-2 logarithm
    // times ln 2 is good to 3 ulp, so g = -log(-log u) (at most 16.7 in magnitude) to 1e-5; near the top
    // |z / T| <= |s| + 17.  The bound used is more than four times that.
    const int t_begin = q_begin * 4, t_end = min(V, q_end * 4);
    const float inv_t = 1.0f / (float)T;
    auto s32 = [&](int t, float zt) {
      if (zt != zt) return -INFINITY;
      const uint32_t m = (uint32_t)(mix64(prefix + (uint64_t)t) >> 41);   // (32 bits: a 64-bit conversion is a dozen instructions)
      const float u = ((float)m + 0.5f) * (1.0f / 8388608.0f);
      constexpr float kLn2 = 0.69314718f;
      return zt * inv_t - __builtin_amdgcn_logf(__builtin_amdgcn_logf(u) * -kLn2) * kLn2;
    };
    // Hashes and logarithms set the pace (two 64-bit products and two quarter-rate logarithms a token), so the next four logits
    // are on their way while four are scored.  Each thread remembers its best token and the second best score: only where
    // both can win does it go over its tokens again, a chain of a memory round trip per token that somebody in every block
    // used to walk (96 rows of 128256: 48 -> 41 us).
    constexpr int kAhead = 4;
    float mine = -INFINITY, second = -INFINITY;
    int at = t_begin + (int)threadIdx.x;
    float ahead[kAhead];
    auto load = [&](int t0) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) ahead[u] = z[min(t0 + u * BLOCK, t_end - 1)];
    };
    if (at < t_end) load(at);
    for (int t0 = at; t0 < t_end; t0 += BLOCK * kAhead) {
      float zv[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) zv[u] = ahead[u];
      if (t0 + BLOCK * kAhead < t_end) load(t0 + BLOCK * kAhead);
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int t = t0 + u * BLOCK;
        const float sc = t < t_end ? s32(t, zv[u]) : -INFINITY;
        second = fmaxf(second, fminf(mine, sc));     // (an equal score, or one that is not a number, counts as a second one)
        at = sc > mine ? t : at;
        mine = fmaxf(mine, sc);
      }
    }
    float mx = mine;
    mx = lanes_max(mx);
    __shared__ float fmx[BLOCK / 64];
    if ((threadIdx.x & 63) == 0) fmx[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmx[0];
    for (int i = 1; i < BLOCK / 64; ++i) mx = fmaxf(mx, fmx[i]);
    // an infinite or empty maximum: score everything in fp64
    const float thr = mx > -INFINITY && mx < INFINITY ? mx - 2.0f * (2e-6f * (fabsf(mx) + 40.0f) + 2e-5f) : -INFINITY;
    auto score = [&](int t) {
      ScoreId c;
      c.id = t;
      c.s = score_of(z[t]) / T + gumbel_from_u(draw_u(prefix, (uint64_t)t));
      if (better(c, best)) best = c;
    };
    if (mine >= thr) {
      const bool one = second < thr;
      for (int t = one ? at : t_begin + (int)threadIdx.x; t < t_end; t += one ? V : BLOCK)
        if (one || s32(t, z[t]) >= thr) score(t);
    }
  }
  best = block_argmax<BLOCK / 64>(best, smem);
  if (threadIdx.x == 0) {
    if (parts == 1) out[(int64_t)row * out_stride] = best.id;
    else scratch[(int64_t)row * parts + part] = best;
  }
}

__global__ __launch_bounds__(64) void sample_merge_kernel(const ScoreId* __restrict__ scratch, int parts,
                                                          int32_t* __restrict__ out, int64_t out_stride) {
  const int row = blockIdx.x;
  ScoreId best = {-INFINITY, 0x7fffffff};
  for (int i = threadIdx.x; i < parts; i += 64) {
    const ScoreId c = scratch[(int64_t)row * parts + i];
    if (better(c, best)) best = c;
  }
  best = lanes_best(best);
  if (threadIdx.x == 0) out[(int64_t)row * out_stride] = best.id;
}

// ---- lossless verification (Sec. 2.1) in two launches.  What bounds a verification is not its bytes (11 rows of 128256 logits
// are 5.6 MB) but the chain of dependent passes: maximum of a row -> softmax denominator -> accept decisions -> residual mass
// -> bonus token, five kernels of 4 to 20 us each when every pass is a launch that re-reads and re-merges the one before.
// Here a row is read once for maximum and denominator together (a running maximum per thread, the partial sums rescaled when
// they meet), and the second kernel does everything behind them: every block merges the rows' partial results for itself,
// decides, and scores its share of the bonus row for the residual; the block of a sequence that finishes last merges the
// shares.  A row and the bonus row are shared among `parts` blocks, so that the few rows of one verification occupy the chip;
// partial results are merged in a fixed order (the result does not depend on timing).  Measured (V = 128256, K = 5,
// temperature 1): B = 1 16.5 us a call (rows 6.5, decisions 9.5: five dependent memory round trips and three reductions; 18.1 with the
// reductions through the LDS crossbar), B = 16 half of it greedy 39.4 us (23 + 16; 40.9; rows without their exponentials 18, of which
// 70 MB at the rate of a copy are 10).
constexpr int kVerifyBlock = 256, kVerifyWaves = kVerifyBlock / 64;
constexpr int kVerifyMaxParts = 32;     // blocks that share a row (one lane of a wavefront merges one of them)
constexpr int kVerifyMaxBonusParts = 64;
struct VerifyPart {       // one part of a row: best logit and its token, sum exp((z - max) / T) relative to that logit
  float max;
  int32_t id;
  double sum;
};
struct VerifyCand {       // one part of the bonus row: best candidate of the exponential race, residual mass
  uint64_t score, id, mass;
};
struct VerifyWs {
  VerifyPart* part;       // [B rows_per_seq][parts]: target rows 0..K, then draft rows 0..K-1 of each sequence
  VerifyCand* cand;       // [B][kVerifyMaxBonusParts]
  uint32_t* done;         // [B] blocks of the second kernel that have stored their candidate
};
__host__ inline VerifyWs verify_ws_carve(void* base, int B, int K) {
  const size_t rows = (size_t)B * (2 * K + 1);
  char* p = (char*)base;
  VerifyWs w;
  w.part = (VerifyPart*)p;   p += rows * kVerifyMaxParts * sizeof(VerifyPart);
  w.cand = (VerifyCand*)p;   p += (size_t)B * kVerifyMaxBonusParts * sizeof(VerifyCand);
  w.done = (uint32_t*)p;
  return w;
}

// this block's share [lo, hi) of a vocabulary of V tokens
__device__ __forceinline__ void verify_share(int V, int& lo, int& hi) {
  const int chunk = (V + (int)gridDim.y - 1) / (int)gridDim.y;
  lo = (int)blockIdx.y * chunk;
  hi = lo + chunk < V ? lo + chunk : V;
}
__device__ __forceinline__ bool better_logit(float v, int t, float m, int id) { return v > m || (v == m && t < id); }
// exp((x - m) / T) of scores where -infinity is "no probability" (also against a maximum of -infinity), in fp64.
// A verification evaluates one exponential per logit and two per token of the bonus row.  Table-driven after P. T. P. Tang, "Table-driven implementation of the
// exponential function in IEEE floating-point arithmetic" (1989): with n = round(32 a / ln 2), a = n ln 2 / 32 + r, |r| <=
// ln 2 / 64, exp(a) = 2^(n >> 5) 2^((n & 31) / 32) (1 + r + .. + r^6 / 720) (next term 4e-18): 19 instructions, none of them a
// conversion or ldexp (a batch of 16 50.7 -> 48.6 us against the library's exp).  No branch, so that several run side by side.
// What it is off by comes from the rounding of the argument, as with a division and a correctly rounded exp: over arguments
// down to -40 at most 3.9e-15 relative (3.7e-15 there), 1.08e-15 on average (1.08e-15), against 80-bit arithmetic.
__device__ __forceinline__ void exp_table_init(double* table) {
  if (threadIdx.x < 32) table[threadIdx.x] = exp2((double)threadIdx.x * (1.0 / 32.0));
}
__device__ __forceinline__ double exp_core(double a, const double* table) {
  constexpr double kMagic = 6755399441055744.0;            // 1.5 2^52: adding it leaves round(a 32 / ln 2) in the low bits
  constexpr double kLn2 = 0.693147180559945309417232121458, kLn2Tail = 2.3190468138462996e-17;   // ln 2 = their sum
  constexpr double kStepHi = (float)(kLn2 / 32.0);         // 24 bits: n kStepHi is exact
  constexpr double kStepLo = (kLn2 / 32.0 - kStepHi) + kLn2Tail / 32.0;
  const double biased = fma(a, 32.0 / kLn2, kMagic);
  const int n = (int)(uint32_t)__double_as_longlong(biased);
  const double nd = biased - kMagic;
  const double r = fma(nd, -kStepLo, fma(nd, -kStepHi, a));
  double q = fma(r, 1.0 / 720.0, 1.0 / 120.0);
  q = fma(r, q, 1.0 / 24.0);
  q = fma(r, q, 1.0 / 6.0);
  q = fma(r, q, 0.5);
  q = fma(r, q, 1.0);
  const double t = table[n & 31];
  const double y = fma(t * r, q, t);                       // in [1, 2] (1 + 2^-6)
  return __hiloint2double(__double2hiint(y) + ((n >> 5) << 20), __double2loint(y));
}
__device__ __forceinline__ double exp_rel(float x, float m, double inv_t, const double* table) {
  const double a = ((double)x - (double)m) * inv_t;
  const double scaled = exp_core(a, table);
  // below e^-700 (and for "no probability"): 0; NaN (an infinite maximum) stays NaN
  return x == -INFINITY || a < -700.0 ? 0.0 : (a == a ? scaled : a);
}
__device__ __forceinline__ float logit_score(float z) { return z != z ? -INFINITY : z; }

// max(ep / sum_p - eq / sum_q, 0) without contraction: where p and q are equal the two products must round alike and cancel
// exactly (a fused multiply-add would leave a residue of 1e-17 of the mass and draw the token from rounding noise)
__device__ __forceinline__ double residual_of(double ep, double pinv, double eq, double qinv) {
#pragma clang fp contract(off)
  const double p = ep * pinv, q = eq * qinv;
  return fmax(p - q, 0.0);
}

// Bounds in fp32 of a token's score in the race, r / -log(u).  The race in fp64 costs two exponentials, a logarithm and a
// division per token, and only the tokens whose upper bound reaches the highest lower bound found so far can win it: the
// others are left out (V = 128256: decisions of B = 1 12.5 -> 10.5 us, of B = 16 half of it greedy 24 -> 17, with the loads of the
// next tokens ahead of the scores and without U copies of the fp64 code, which the first wavefronts have to fetch).
// Relative error of p = exp2(e) pinv: the argument e is a difference, a product and two rounded factors, 4 2^-24 |e|, times ln 2;
// the hardware exponential and the two products add 2^-22.  Terms below 2^-126 may have been flushed: 1e-37 absolute, also after
// the subtraction (pinv <= 1).  -logf(u) and the reciprocal: below 2^-21 together.
struct Fp32Race {
  float pmax, qmax, scale, pinv, qinv;
  __device__ __forceinline__ void bounds(float zp, float zq, bool residual, uint64_t prefix, uint64_t t, float& lo, float& hi) const {
    const float ep = (zp - pmax) * scale, eq = (zq - qmax) * scale;
    const float p = __builtin_amdgcn_exp2f(ep) * pinv, q = residual ? __builtin_amdgcn_exp2f(eq) * qinv : 0.f;
    // (an exponent of -infinity: the probability is 0 and so is its share of the error)
    float err = p * (fabsf(fmaxf(ep, -150.f)) * 2.5e-7f + 1e-6f) + 2e-37f;
    if (residual) err += q * (fabsf(fmaxf(eq, -150.f)) * 2.5e-7f + 1e-6f);
    const float m = (float)(uint32_t)(mix64(prefix + t) >> 41) + 0.5f;              // 24 significant bits: exact
    const float inv_e = __builtin_amdgcn_rcpf(-logf(m * (1.0f / 8388608.0f)));
    lo = (p - q - err) * inv_e * (1.0f - 2e-6f);
    hi = (p - q + err) * inv_e * (1.0f + 2e-6f);
  }
};

// (best logit, its token, sum relative to it) over groups of W lanes; every lane returns its group's result
template <int W>
__device__ __forceinline__ VerifyPart lanes_merge(VerifyPart v, double inv_t, bool sampled, const double* table) {
  struct Top { float max; int32_t id; };
  const Top top = lanes_reduce<W / 2>(Top{v.max, v.id}, [](Top a, Top b) { return better_logit(a.max, a.id, b.max, b.id) ? a : b; });
  if (sampled) v.sum = lanes_sum<W / 2>(v.sum * exp_rel(v.max, top.max, inv_t, table));
  v.max = top.max;
  v.id = top.id;
  return v;
}

// Kernel 1: per logit row and part, the best (logit, token) and the partial softmax denominator.  grid (B rows_per_seq, parts);
// rows_per_seq = 2K+1, or K+1 without draft logits (then every sequence is greedy).
__global__ __launch_bounds__(kVerifyBlock) void verify_rows_kernel(const float* __restrict__ zt, const float* __restrict__ zd,
                                                                   const float* __restrict__ temperature, int K, int V,
                                                                   int rows_per_seq, VerifyWs ws) {
  constexpr int U = 8;    // tokens of a thread scored side by side (as many again are on their way)
  __shared__ VerifyPart wave_part[kVerifyWaves];
  __shared__ double table[32];
  const int b = blockIdx.x / rows_per_seq, r = blockIdx.x % rows_per_seq;
  if (r == 0 && blockIdx.y == 0 && threadIdx.x == 0) ws.done[b] = 0;    // for the next kernel
  const float* z = r <= K ? zt + ((int64_t)b * (K + 1) + r) * V : zd + ((int64_t)b * K + (r - K - 1)) * V;
  int lo, hi;
  verify_share(V, lo, hi);
  const int last = (hi > lo ? hi : V) - 1;
  float ahead[U];
  auto load = [&](int t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) ahead[u] = z[(uint32_t)min(t0 + u * kVerifyBlock, last)];
  };
  // (a target row is on its way while the temperature is read; a draft row waits for it: that of a greedy sequence is not read.
  // 16 greedy sequences of K = 5 with draft logits 17.3 -> 15.4 us, half of them sampled 42.4 -> 41.9)
  if (r <= K) load(lo + threadIdx.x);
  const double T = zd ? (double)temperature[b] : 0.0;
  const bool sampled = T > 0.0;
  if (r > K) {
    if (!sampled) return;                                               // a draft row of a greedy sequence
    load(lo + threadIdx.x);
  }
  const double inv_t = sampled ? 1.0 / T : 0.0;
  if (sampled) {
    exp_table_init(table);
    __syncthreads();
  }
  VerifyPart best = {-INFINITY, 0x7fffffff, 0.0};
  for (int t0 = lo + threadIdx.x; t0 < hi; t0 += kVerifyBlock * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = ahead[u];
    if (t0 + kVerifyBlock * U < hi) load(t0 + kVerifyBlock * U);
    // (a thread's tokens come in rising order, past the end its last one again: an equal logit does not replace one found
    // before it)
    const float before = best.max;
    float top = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] = logit_score(v[u]);
      top = fmaxf(top, v[u]);
    }
    if (top > before || best.id == 0x7fffffff) {
      best.max = top;
#pragma unroll
      for (int u = U - 1; u >= 0; --u) best.id = v[u] == top ? min(t0 + u * kVerifyBlock, last) : best.id;
      if (sampled) best.sum *= exp_rel(before, top, inv_t, table);
    }
    if (sampled) {
      // Every term is at most 1 and the thread's largest is 1: terms below e^-708, "no probability" (-infinity) among them, are
      // held at e^-708, which leaves the sum as it is and saves the tests (32 -> 25 instructions a term)
      const double m = best.max;
      double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float x = t0 + u * kVerifyBlock < hi ? v[u] : -INFINITY;
        part[u & 3] += exp_core(fmax(((double)x - m) * inv_t, -708.0), table);
      }
      best.sum += (part[0] + part[1]) + (part[2] + part[3]);
    }
  }
  // a row without any probability, and one whose maximum is infinite (no distribution)
  if (best.max == -INFINITY) best.sum = 0.0;
  if (best.max == INFINITY) best.sum = __longlong_as_double(0x7ff8000000000000ll);
  best = lanes_merge<64>(best, inv_t, sampled, table);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) wave_part[wave] = best;
  __syncthreads();
  if (wave == 0) {
    best = lane < kVerifyWaves ? wave_part[lane] : VerifyPart{-INFINITY, 0x7fffffff, 0.0};
    best = lanes_merge<kVerifyWaves>(best, inv_t, sampled, table);
    if (lane == 0) ws.part[(int64_t)blockIdx.x * gridDim.y + blockIdx.y] = best;
  }
}

// Kernel 2.  grid (B, parts): every block of a sequence merges the partial results of its rows, takes the sequential accept
// decisions (one lane per position, the first rejection by ballot) and, for sampled sequences, finds this part's candidate for
// the bonus token at position k: from the residual max(p - q, 0), or from p at k = K and where the residual has no mass.
// The candidate is the winner of an exponential race, r / -log(u): log(r) + (-log(-log u)), the Gumbel-max score, is its
// logarithm, so the order is the same at one logarithm per token instead of three.
__global__ __launch_bounds__(kVerifyBlock) void verify_decide_kernel(const float* __restrict__ zt, const float* __restrict__ zd,
                                                                     const int32_t* __restrict__ spec,
                                                                     const float* __restrict__ temperature, int K, int V,
                                                                     uint64_t seed, int rows_per_seq, int row_parts, VerifyWs ws,
                                                                     int32_t* __restrict__ accept_len, int32_t* __restrict__ bonus) {
  constexpr int U = 4;    // tokens of a thread scored side by side (as many again are on their way)
  constexpr int H = 2;    // rows of a half wavefront whose partial results are requested at once
  __shared__ double table[32];
  __shared__ VerifyPart row_s[2 * SSD_MAX_K + 1];
  __shared__ int k_s, last_s;
  __shared__ double mass_s[kVerifyWaves];
  __shared__ ScoreId best_s[kVerifyWaves];
  const int b = blockIdx.x, parts = gridDim.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // ---- requested together: the temperature, the drafted tokens, the first rows' partial results (rows of draft logits of a
  // greedy sequence hold nothing and are not used)
  int tok = -1;
  if ((int)threadIdx.x < K) tok = spec[(int64_t)b * K + threadIdx.x];
  static_assert(kVerifyMaxParts <= 32, "half a wavefront merges a row");
  VerifyPart v[H];
  auto load_parts = [&](int r0) {
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int r = r0 + 2 * kVerifyWaves * i;
      v[i] = {-INFINITY, 0x7fffffff, 0.0};
      if (r < rows_per_seq && (lane & 31) < row_parts) v[i] = ws.part[((int64_t)b * rows_per_seq + r) * row_parts + (lane & 31)];
    }
  };
  load_parts(2 * wave + (lane >> 5));
  const double T = zd ? (double)temperature[b] : 0.0;
  const bool sampled = T > 0.0;
  if (!sampled && blockIdx.y > 0) return;
  const double inv_t = sampled ? 1.0 / T : 0.0;
  // ---- the drafted tokens' logits, requested ahead of the merge
  float zt_s = 0.f, zd_s = 0.f;
  if (sampled && tok >= 0 && tok < V) {
    zt_s = zt[((int64_t)b * (K + 1) + threadIdx.x) * V + tok];
    zd_s = zd[((int64_t)b * K + threadIdx.x) * V + tok];
  }
  if (sampled) exp_table_init(table);
  // ---- the rows' maxima and denominators: half a wavefront per row, a lane per part, two rows' chains side by side
  const int n_rows = sampled ? 2 * K + 1 : K + 1;
  __syncthreads();
  for (int r0 = 2 * wave + (lane >> 5); r0 < n_rows; r0 += 2 * H * kVerifyWaves) {
    if (r0 >= 2 * H * kVerifyWaves) load_parts(r0);
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int r = r0 + 2 * kVerifyWaves * i;
      v[i] = lanes_merge<32>(v[i], inv_t, sampled, table);
      if (r < n_rows && (lane & 31) == 0) row_s[r] = v[i];
    }
  }
  __syncthreads();
  // ---- accept s_{i+1} while u q(s) < p(s) (greedy: while it is the target's argmax)
  if (wave == 0) {
    bool ok = true;
    if (lane < K) {
      if (!sampled) ok = row_s[lane].id == tok;
      else if (tok < 0 || tok >= V) ok = false;
      else {
        const double p = exp_rel(logit_score(zt_s), row_s[lane].max, inv_t, table) / row_s[lane].sum;
        const double q = exp_rel(logit_score(zd_s), row_s[K + 1 + lane].max, inv_t, table) / row_s[K + 1 + lane].sum;
        ok = draw_u(draw_prefix(seed, STREAM_ACCEPT, (uint64_t)b, (uint64_t)lane), 0ull) * q < p;
      }
    }
    const unsigned long long rejected = __ballot(!ok);
    if (lane == 0) k_s = rejected ? __ffsll((long long)rejected) - 1 : K;
  }
  __syncthreads();
  const int k = k_s;
  if (blockIdx.y == 0 && threadIdx.x == 0) {
    accept_len[b] = k;
    if (!sampled) bonus[b] = row_s[k].id;
  }
  if (!sampled) return;

  // ---- this part's share of the bonus row
  const float* zp = zt + ((int64_t)b * (K + 1) + k) * V;
  const float* zq = zd + ((int64_t)b * K + (k < K ? k : 0)) * V;
  const float pmax = row_s[k].max, qmax = k < K ? row_s[K + 1 + k].max : 0.f;
  const double pinv = 1.0 / row_s[k].sum, qinv = k < K ? 1.0 / row_s[K + 1 + k].sum : 0.0;
  const uint64_t prefix = draw_prefix(seed, STREAM_BONUS, (uint64_t)b, (uint64_t)k);
  int lo, hi;
  verify_share(V, lo, hi);
  const Fp32Race race{pmax, qmax, (float)inv_t * 1.44269504f, (float)pinv, (float)qinv};
  ScoreId best;
  double mass;     // only its sign is used: above 0 where some token of this part has residual mass
  // once for the residual and, where this part of it has no mass (its candidate counts only if no part has any, and is then
  // p's), once more for p (without qinv, which is no number where the draft's row has no distribution)
  for (bool residual = k < K;; residual = false) {
    best = {-1.0, 0x7fffffff};
    mass = 0.0;
    float floor_s = -INFINITY;             // a score that some token of this wavefront is known to reach
    float ahead_p[U], ahead_q[U];
    auto load = [&](int t0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t t = max(min(t0 + u * kVerifyBlock, hi - 1), 0);
        ahead_p[u] = zp[t];
        ahead_q[u] = zq[t];
      }
    };
    load(lo + threadIdx.x);
    for (int t0 = lo + threadIdx.x; __any(t0 < hi); t0 += kVerifyBlock * U) {
      float vp[U], vq[U], most[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        vp[u] = ahead_p[u];
        vq[u] = ahead_q[u];
      }
      load(t0 + kVerifyBlock * U);
      float least = -INFINITY;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float lo_s;
        race.bounds(logit_score(vp[u]), logit_score(vq[u]), residual, prefix, (uint64_t)(t0 + u * kVerifyBlock), lo_s, most[u]);
        const bool in = t0 + u * kVerifyBlock < hi;
        least = fmaxf(least, in ? lo_s : -INFINITY);
        most[u] = in ? most[u] : -INFINITY;
      }
      least = lanes_max(least);
      floor_s = fmaxf(floor_s, least);
      // in fp64, the tokens that may win (all of them where none is known to have mass; a bound that is no number excludes
      // nothing).  A loop over a lane's tokens rather than U copies of its body: most wavefronts take it once, and every
      // copy would be fetched
      uint32_t open = 0;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (t0 + u * kVerifyBlock < hi && !(floor_s > 0.f && most[u] < floor_s)) open |= 1u << u;
      while (__any(open != 0)) {
        const int u1 = open ? __ffs((int)open) - 1 : 0;
        float xp = vp[0], xq = vq[0];
#pragma unroll
        for (int u = 1; u < U; ++u) {
          xp = u1 == u ? vp[u] : xp;
          xq = u1 == u ? vq[u] : xq;
        }
        if (open) {
          const int t = t0 + u1 * kVerifyBlock;
          double r = residual_of(exp_rel(logit_score(xp), pmax, inv_t, table), pinv,
                                 residual ? exp_rel(logit_score(xq), qmax, inv_t, table) : 0.0, residual ? qinv : 0.0);
          r = r > 0.0 ? r : 0.0;
          mass += r;
          const ScoreId c = {r / -log(draw_u(prefix, (uint64_t)t)), t};
          if (better(c, best)) best = c;
        }
        open &= open - 1;
      }
    }
    mass = lanes_sum(mass);
    best = lanes_best(best);
    __syncthreads();
    if (lane == 0) { mass_s[wave] = mass; best_s[wave] = best; }
    __syncthreads();
    mass = 0.0;
    best = best_s[0];
    for (int w = 0; w < kVerifyWaves; ++w) {
      mass += mass_s[w];
      if (better(best_s[w], best)) best = best_s[w];
    }
    if (!residual) {
      if (k < K) mass = 0.0;
      break;
    }
    if (mass > 0.0) break;
  }
  // ---- the part's candidate goes out with agent-scope stores (visible to every compute unit once vmcnt is zero); the block
  // that counts last of the sequence's parts reads them all back and picks the token
  if (threadIdx.x == 0) {
    VerifyCand* c = ws.cand + (int64_t)b * kVerifyMaxBonusParts + blockIdx.y;
    __hip_atomic_store(&c->score, (uint64_t)__double_as_longlong(best.s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&c->id, (uint64_t)(uint32_t)best.id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&c->mass, (uint64_t)__double_as_longlong(mass), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    last_s = __hip_atomic_fetch_add(ws.done + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == (uint32_t)parts;
  }
  __syncthreads();
  if (!last_s || wave != 0) return;
  ScoreId mine = {-1.0, 0x7fffffff};
  double m = 0.0;
  if (lane < parts) {
    const VerifyCand* c = ws.cand + (int64_t)b * kVerifyMaxBonusParts + lane;
    mine.s = __longlong_as_double((long long)__hip_atomic_load(&c->score, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    mine.id = (int)__hip_atomic_load(&c->id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    m = __longlong_as_double((long long)__hip_atomic_load(&c->mass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  }
  if (k < K && __any(m > 0.0) && !(m > 0.0)) mine = {-1.0, 0x7fffffff};
  mine = lanes_best(mine);
  if (lane == 0) bonus[b] = mine.id;
}

}  // namespace

namespace {

// Parts per row: enough blocks to occupy the chip when there are few rows, at least 4096 tokens per part.
int top_f_parts(int rows, int V, const void* scratch) {
  if (!scratch) return 1;
  int parts = 512 / rows;
  parts = parts > kTopFMaxParts ? kTopFMaxParts : parts;
  while (parts > 1 && V / parts < 4096) --parts;
  return parts < 1 ? 1 : parts;
}

template <int FMAX>
int run_top_f(const float* logits, int64_t ld, const int32_t* exclude, int rows, int V, int F, int groups, const FanTable& fan,
              int32_t* ids, void* scratch, hipStream_t s) {
  const int parts = top_f_parts(rows, V, scratch);
  top_f_kernel<FMAX><<<dim3(rows, parts), kSelBlock, 0, s>>>(logits, ld, exclude, V, F, groups, fan, ids, (uint64_t*)scratch);
  if (parts > 1) top_f_merge_kernel<FMAX><<<rows, 64, 0, s>>>((const uint64_t*)scratch, parts, F, groups, fan, ids);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

}  // namespace

size_t top_f_scratch_bytes(int rows) { return (size_t)rows * kTopFMaxParts * SSD_MAX_F * sizeof(uint64_t); }

int launch_top_f(const float* logits, int64_t ld, const int32_t* exclude, int rows, int V, int F, int32_t* ids,
                 void* scratch, hipStream_t s) {
  if (rows <= 0) return SSD_OK;
  const FanTable none = {};
  if (F <= 4) return run_top_f<4>(logits, ld, exclude, rows, V, F, 0, none, ids, scratch, s);
  if (F <= 8) return run_top_f<8>(logits, ld, exclude, rows, V, F, 0, none, ids, scratch, s);
  return run_top_f<16>(logits, ld, exclude, rows, V, F, 0, none, ids, scratch, s);
}

// Random-token backup speculator (Sec. 4.3): token i of sequence b is the 64-bit hash of (seed, backup stream, b, i, 0)
// modulo the vocabulary size.
__global__ void backup_random_kernel(int32_t* __restrict__ tokens, int B, int K, int V, uint64_t seed) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= B * K) return;
  const int b = idx / K, i = idx - b * K;
  tokens[idx] = (int32_t)(mix64(draw_prefix(seed, STREAM_BACKUP, (uint64_t)b, (uint64_t)i)) % (uint64_t)V);
}

int launch_backup_random(int32_t* tokens, int B, int K, int V, uint64_t seed, hipStream_t s) {
  if (B * K <= 0) return SSD_OK;
  backup_random_kernel<<<(B * K + 255) / 256, 256, 0, s>>>(tokens, B, K, V, seed);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

int launch_top_f_fan(const float* logits, int64_t ld, const int32_t* exclude, int B, int K, const FanTable& fan, int V,
                     int32_t* ids, void* scratch, hipStream_t s) {
  const int rows = B * (K + 1);
  if (rows <= 0) return SSD_OK;
  int f_max = 0;
  for (int k = 0; k <= K; ++k) f_max = fan.off[k + 1] - fan.off[k] > f_max ? fan.off[k + 1] - fan.off[k] : f_max;
  if (f_max <= 4) return run_top_f<4>(logits, ld, exclude, rows, V, 0, K + 1, fan, ids, scratch, s);
  if (f_max <= 8) return run_top_f<8>(logits, ld, exclude, rows, V, 0, K + 1, fan, ids, scratch, s);
  return run_top_f<16>(logits, ld, exclude, rows, V, 0, K + 1, fan, ids, scratch, s);
}

// Saguaro sampling scheme sigma_{F,C} (Sec. 4.2.1) on rows of logits, in place: the F tokens in ids[row] (the row's own
// top-F) get T log C added, which multiplies their weight exp(z/T) by C.  Greedy rows (T == 0) are left alone.
__global__ void sigma_shift_kernel(float* __restrict__ logits, int64_t ld, const float* __restrict__ temperature,
                                   int rows_per_seq, int rows, int F, const int32_t* __restrict__ ids, float log_c) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * F) return;
  const int row = i / F;
  const float T = temperature[row / rows_per_seq];
  if (T > 0.f) logits[(int64_t)row * ld + ids[i]] += T * log_c;
}

int launch_sigma_shift(float* logits, int64_t ld, const float* temperature, int rows_per_seq, int rows, int F,
                       const int32_t* ids, float log_c, hipStream_t s) {
  if (rows <= 0) return SSD_OK;
  sigma_shift_kernel<<<(rows * F + 255) / 256, 256, 0, s>>>(logits, ld, temperature, rows_per_seq, rows, F, ids, log_c);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

size_t sample_scratch_bytes(int rows) { return (size_t)rows * kSampleMaxParts * sizeof(ScoreId); }

// scratch: sample_scratch_bytes(rows) of device memory, or null (then every row is one block)
int launch_sample(const float* logits, int64_t ld, const float* temperature, int rows_per_seq, int rows, int V,
                  uint64_t seed, int row_base, int step, int32_t* out, int64_t out_stride, void* scratch, int exact_scan,
                  hipStream_t s) {
  if (rows <= 0) return SSD_OK;
  int parts = 1;
  if (scratch && V > 4096) {                                            // (fewer tokens: a block has them in 4 loads a thread)
    parts = (2048 + rows - 1) / rows;                                   // about 2048 blocks
    const int by_len = (V + kSampleBlock * 4 - 1) / (kSampleBlock * 4); // at least 4 tokens per thread
    parts = parts < by_len ? parts : by_len;
    parts = parts < kSampleMaxParts ? parts : kSampleMaxParts;
    parts = parts < 1 ? 1 : parts;
  }
  // exact_scan: score every token of a sampled row in fp64 instead of pre-selecting in fp32 (a test aid: both give the
  // same token)
  const dim3 grid(rows, parts);
  if (parts > 1)
    sample_kernel<kSampleBlock><<<grid, kSampleBlock, 0, s>>>(logits, ld, temperature, rows_per_seq, V, seed, row_base, step, out,
                                                              out_stride, (ScoreId*)scratch, exact_scan);
  else
    sample_kernel<kSelBlock><<<grid, kSelBlock, 0, s>>>(logits, ld, temperature, rows_per_seq, V, seed, row_base, step, out, out_stride,
                                                        (ScoreId*)scratch, exact_scan);
  SSD_HIP(hipGetLastError());
  if (parts > 1) {
    sample_merge_kernel<<<rows, 64, 0, s>>>((const ScoreId*)scratch, parts, out, out_stride);
    SSD_HIP(hipGetLastError());
  }
  return SSD_OK;
}


int launch_verify(const float* zt, const float* zd, const int32_t* spec, const float* temperature, int B, int K, int V,
                  uint64_t seed, int32_t* accept_len, int32_t* bonus, void* workspace, hipStream_t s) {
  const VerifyWs ws = verify_ws_carve(workspace, B, K);
  const int rows_per_seq = zd ? 2 * K + 1 : K + 1;    // without draft logits every sequence is greedy
  const int rows = B * rows_per_seq;
  // enough blocks to occupy the chip, at least 1024 tokens (4 per thread) to each
  auto cut = [&](int blocks, int n, int most) {
    int parts = blocks / n;
    parts = parts > most ? most : parts;
    parts = parts > V / 1024 ? V / 1024 : parts;
    return parts < 1 ? 1 : parts;
  };
  const int parts = cut(2048, rows, kVerifyMaxParts);
  const int parts_b = zd ? cut(1024, B, kVerifyMaxBonusParts) : 1;
  verify_rows_kernel<<<dim3(rows, parts), kVerifyBlock, 0, s>>>(zt, zd, temperature, K, V, rows_per_seq, ws);
  verify_decide_kernel<<<dim3(B, parts_b), kVerifyBlock, 0, s>>>(zt, zd, spec, temperature, K, V, seed, rows_per_seq, parts, ws,
                                                                 accept_len, bonus);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

// ---- verification for callers that cannot allocate: the workspace is a file-scope device array.  Host code never
// passes the array's name to a kernel (there it is only a host-side stand-in): the device address is looked up once
// per device with hipGetSymbolAddress and kept.
constexpr size_t kStaticScratchBytes = (size_t)1 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t verify_static_capacity() { return kStaticScratchBytes; }

int launch_verify_static(const float* zt, const float* zd, const int32_t* spec, const float* temperature, int B, int K, int V,
                         uint64_t seed, int32_t* accept_len, int32_t* bonus, hipStream_t s) {
  const size_t need = verify_workspace_bytes(B, K);
  SSD_CHECK_ARG(need <= kStaticScratchBytes,
                "ssd_verify_static: B = %d, K = %d needs %zu bytes of scratch, the static buffer holds %zu (512 (2K+1) + 1540 bytes per sequence)",
                B, K, need, kStaticScratchBytes);
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr_of_device[kMaxDevices] = {};
  int dev = 0;
  SSD_HIP(hipGetDevice(&dev));
  SSD_CHECK_ARG(dev >= 0 && dev < kMaxDevices, "ssd_verify_static: device ordinal %d out of range", dev);
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of_device[dev]) {
      void* p = nullptr;
      SSD_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));   // this device's copy of the array (the current device)
      ptr_of_device[dev] = p;
    }
    ptr = ptr_of_device[dev];
  }
  // nothing in the workspace has to start at zero: every word a pass reads was written by an earlier pass of the same call
  return launch_verify(zt, zd, spec, temperature, B, K, V, seed, accept_len, bonus, ptr, s);
}

size_t verify_workspace_bytes(int B, int K) {
  const size_t rows = (size_t)B * (2 * K + 1);
  return rows * kVerifyMaxParts * sizeof(VerifyPart) + (size_t)B * kVerifyMaxBonusParts * sizeof(VerifyCand) +
         (((size_t)B * sizeof(uint32_t) + 15) & ~(size_t)15);
}

}  // namespace ssd
