// Decode attention over "shared trunk + private suffix" (App. B: every branch row attends the verified trunk
// up to its fork point and only its own path).  No mask is materialised: a row is described by the number of
// trunk positions it sees and the number of private suffix positions it sees.
#include "common.h"
#include "lanes.h"

namespace ssd {

namespace {

template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void load(const float* p, float* o) {
    float4 v = *(const float4*)p;
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void load(const bf16_t* p, float* o) {
    uint4 v = *(const uint4*)p;
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

// One block per (row, KV head); wavefront w takes query heads w, w+4, .. of the group.  Each lane owns the keys
// lane, lane+64, .. and keeps its own running softmax (max, sum, weighted V); lanes are merged at the end.  The
// kernel for passes with many rows (every row is a block of its own, the chip is full without splitting keys).
template <typename T, int D>
__global__ __launch_bounds__(256) void attention_rowwise_kernel(const float* __restrict__ q, const T* __restrict__ trunk_k,
                                                                 const T* __restrict__ trunk_v,
                                                                 const T* __restrict__ suffix_k,
                                                                 const T* __restrict__ suffix_v, void* __restrict__ out,
                                                                 int64_t out_plane,
                                                                 const RowDesc* __restrict__ rows, int n_q_heads,
                                                                 int n_kv_heads, int max_trunk, int suffix_cap) {
  __shared__ float q_s[4][D];
  const int m = blockIdx.x, hk = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int group = n_q_heads / n_kv_heads;
  const RowDesc r = rows[m];
  const int n_keys = r.vis + r.suffix_len;
  const float scale = rsqrtf((float)D);
  const int64_t kv_stride = (int64_t)n_kv_heads * D;
  const T* tk = trunk_k + ((int64_t)r.seq * max_trunk) * kv_stride + hk * D;
  const T* tv = trunk_v + ((int64_t)r.seq * max_trunk) * kv_stride + hk * D;
  const T* sk = suffix_k + ((int64_t)m * suffix_cap) * kv_stride + hk * D;
  const T* sv = suffix_v + ((int64_t)m * suffix_cap) * kv_stride + hk * D;

  for (int g = wave; g < group; g += 4) {
    const int hq = hk * group + g;
    const float* qp = q + ((int64_t)m * n_q_heads + hq) * D;
    for (int d = lane; d < D; d += 64) q_s[wave][d] = qp[d];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");

    float m_run = -INFINITY, l_run = 0.f;
    float acc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) acc[d] = 0.f;

    for (int j = lane; j < n_keys; j += 64) {
      const T* kp = j < r.vis ? tk + (int64_t)j * kv_stride : sk + (int64_t)(j - r.vis) * kv_stride;
      const T* vp = j < r.vis ? tv + (int64_t)j * kv_stride : sv + (int64_t)(j - r.vis) * kv_stride;
      float s = 0.f;
#pragma unroll
      for (int d0 = 0; d0 < D; d0 += Vec16<T>::N) {
        float kk[Vec16<T>::N];
        Vec16<T>::load(kp + d0, kk);
#pragma unroll
        for (int e = 0; e < Vec16<T>::N; ++e) s = fmaf(q_s[wave][d0 + e], kk[e], s);
      }
      s *= scale;
      float m_new = fmaxf(m_run, s);
      float corr = expf(m_run - m_new);      // exp(-inf) = 0 on the first key
      float p = expf(s - m_new);
      l_run = l_run * corr + p;
#pragma unroll
      for (int d0 = 0; d0 < D; d0 += Vec16<T>::N) {
        float vv[Vec16<T>::N];
        Vec16<T>::load(vp + d0, vv);
#pragma unroll
        for (int e = 0; e < Vec16<T>::N; ++e) acc[d0 + e] = fmaf(p, vv[e], acc[d0 + e] * corr);
      }
      m_run = m_new;
    }
    // merge the 64 lanes
    float m_all = m_run;
    m_all = lanes_max(m_all);
    float w = m_run == -INFINITY ? 0.f : expf(m_run - m_all);
    float l_all = l_run * w;
    l_all = lanes_sum(l_all);
    float inv = 1.0f / l_all;
    const int64_t obase = ((int64_t)m * n_q_heads + hq) * D;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      float v = acc[d] * w;
      v = lanes_sum(v);
      if (lane == (d & 63)) Act<T>::store(out, out_plane, obase + d, v * inv);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

constexpr int kMaxSplits = 64;          // key splits of a row
constexpr int kSplitKeys = 256;         // most keys of a split: one per thread
constexpr int kSplitMaxRows = 64;       // rows up to which the scratch allows the most splits
constexpr int kSplitMaxGroup = 8;       // query heads per KV head the split kernel holds

// VEC consecutive elements: 16 bytes, or (bf16) 4, (either type) one
template <typename T, int VEC>
__device__ __forceinline__ void load_elems(const T* p, float* o) {
  if constexpr (VEC == Vec16<T>::N) Vec16<T>::load(p, o);
  else if constexpr (VEC == 2 && sizeof(T) == 2) {
    const uint32_t w = *(const uint32_t*)p;
    o[0] = __uint_as_float(w << 16);
    o[1] = __uint_as_float(w & 0xffff0000u);
  } else {
#pragma unroll
    for (int e = 0; e < VEC; ++e) o[e] = Elem<T>::load(p + e);
  }
}

// the same from a register
template <typename T, int VEC>
__device__ __forceinline__ void unpack_elems(uint4 v, float* o) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    if constexpr (sizeof(T) == 4) o[e] = __uint_as_float(w[e & 3]);
    else o[e] = __uint_as_float(e & 1 ? w[e / 2 & 3] & 0xffff0000u : w[e / 2 & 3] << 16);
  }
}

// Passes with few rows (an extend, a verification forward, a small decode batch): one block per (row, KV head, split
// of at most 256 keys), all query heads of the group (at most G) at once.  Scores: one key per thread against the group's
// queries (in LDS); softmax over the block; weighted values: every wavefront takes a quarter of the keys the split really
// has, 16 bytes per lane and kPvBatch loads together (a load covers KPI keys), so
// a split of 64 keys is one memory round trip there, where 64 fixed keys per wavefront and one row per load made it eight.
// Writes the split's partial softmax (max, sum, unnormalised output) to `partial` [row][query head][split][D + 2];
// attention_merge_kernel adds the splits up in split order.  A single split is the result (partial == nullptr).
// 10 rows x 4 heads x 138 keys, fp32: 6.4 us (18.5 us and 4.7 us of merge before; 6.6 with the values requested behind the scores).
// Values ahead: as many loads as cost no wavefront in flight (one query head, bf16: 8 leave five per SIMD, 12 four; rounds of 24 rows over 700
// keys of 8 heads of 128 dimensions 1243 us with 8, 1321 with 12, 1246 with none, 1337 before there were any), 12 for one fp32 head, which
// keeps more than four with them (96 rows over 8000 keys 10.72 ms with 12, 11.15 with 8).  MANY: a launch of many more blocks than the chip
// holds is bound by the keys and values its L2s miss: values behind the scores and four wavefronts per SIMD spread over fewer of them
// (384 rows over 8000 keys, 16 heads of 64 dimensions: 36.4 ms, 36.8 with 8 values ahead, 37.2 with 12; 36.0 before the sums over lanes left
// the LDS crossbar, the one size that stayed slower by 1 %).
template <typename T, int D, int G, bool MANY = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MANY ? 4 : 1, MANY ? 4 : 8))) void attention_split_kernel(const float* __restrict__ q, const T* __restrict__ trunk_k,
                                                               const T* __restrict__ trunk_v, const T* __restrict__ suffix_k,
                                                               const T* __restrict__ suffix_v, const RowDesc* __restrict__ rows,
                                                               int n_q_heads, int n_kv_heads, int max_trunk, int suffix_cap,
                                                               float* __restrict__ partial, int keys_per_split,
                                                               void* __restrict__ out, int64_t out_plane) {
  // head dimensions per lane: 16 bytes, or with a large group one consecutive share of a whole-wavefront row per key (8
  // heads x 8 dimensions of accumulators and their exchange across lanes cost a 70B-shaped row more than they saved:
  // 55 -> 70 us for 6 rows x 8 heads x 4096 keys)
  constexpr int KV = Vec16<T>::N, VEC = G * KV <= 32 ? KV : D / 64, LPR = D / VEC, KPI = 64 / LPR;
  constexpr int kPvBatch = 8, kPvAhead = MANY ? 0 : G == 1 && sizeof(T) == 4 ? 12 : 8;
  __shared__ float q_s[G][D];
  __shared__ float p_s[G][kSplitKeys];
  __shared__ float red_s[4][G][D];
  __shared__ float mx_s[G][4], sum_s[G][4];
  const int m = blockIdx.x, hk = blockIdx.y, split = blockIdx.z, n_splits = gridDim.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int group = n_q_heads / n_kv_heads;
  const RowDesc r = rows[m];
  const int n_keys = r.vis + r.suffix_len;
  const int j_begin = split * keys_per_split;
  const int j_end = min(n_keys, j_begin + keys_per_split);
  const float scale = rsqrtf((float)D);
  const int64_t kv_stride = (int64_t)n_kv_heads * D;
  const T* tk = trunk_k + ((int64_t)r.seq * max_trunk) * kv_stride + hk * D;
  const T* tv = trunk_v + ((int64_t)r.seq * max_trunk) * kv_stride + hk * D;
  const T* sk = suffix_k + ((int64_t)m * suffix_cap) * kv_stride + hk * D;
  const T* sv = suffix_v + ((int64_t)m * suffix_cap) * kv_stride + hk * D;

  // ---- the first values of this wavefront's quarter of the keys (addresses only: they are on their way while the scores are taken)
  const int n_here = max(j_end - j_begin, 0), quarter = (n_here + 3) >> 2;
  const int jq0 = wave * quarter, jq1 = min(jq0 + quarter, n_here);
  const int sub = lane / LPR, d0 = (lane & (LPR - 1)) * VEC;
  auto value_row = [&](int jk) { return (jk < r.vis ? tv + (int64_t)jk * kv_stride : sv + (int64_t)(jk - r.vis) * kv_stride) + d0; };
  constexpr int kAhead = VEC * sizeof(T) == 16 ? kPvAhead : 0;
  uint4 ahead[kAhead > 0 ? kAhead : 1];
  if (kAhead > 0 && jq0 < jq1) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) ahead[u] = *(const uint4*)value_row(j_begin + min(jq0 + u * KPI + sub, jq1 - 1));
  }
  for (int i = tid; i < group * D; i += 256) {
    const int g = i / D, d = i - g * D;
    q_s[g][d] = q[((int64_t)m * n_q_heads + hk * group + g) * D + d] * scale;
  }
  __syncthreads();

  // ---- scores of key j_begin + tid against the group's queries
  const int j = j_begin + tid;
  const bool have = j < j_end;
  float sc[G];
#pragma unroll
  for (int g = 0; g < G; ++g) sc[g] = 0.f;
  if (have) {
    const T* kp = j < r.vis ? tk + (int64_t)j * kv_stride : sk + (int64_t)(j - r.vis) * kv_stride;
    // (fully unrolled: the key row's loads all go out before the first product; in groups of 4 a row of 128 bf16
    // cost four memory round trips)
#pragma unroll
    for (int d0 = 0; d0 < D; d0 += KV) {
      float kk[KV];
      Vec16<T>::load(kp + d0, kk);
#pragma unroll
      for (int g = 0; g < G; ++g)
        if (g < group) {
#pragma unroll
          for (int e = 0; e < KV; ++e) sc[g] = fmaf(q_s[g][d0 + e], kk[e], sc[g]);
        }
    }
  }
  // ---- softmax over the split: maximum and sum per query head
#pragma unroll
  for (int g = 0; g < G; ++g) {
    float v = have ? sc[g] : -INFINITY;
    v = lanes_max(v);
    if (lane == 0) mx_s[g][wave] = v;
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float mg = fmaxf(fmaxf(mx_s[g][0], mx_s[g][1]), fmaxf(mx_s[g][2], mx_s[g][3]));
    const float m_use = mg == -INFINITY ? 0.f : mg;
    const float pe = have ? expf(sc[g] - m_use) : 0.f;
    p_s[g][tid] = pe;
    float v = pe;
    v = lanes_sum(v);
    if (lane == 0) sum_s[g][wave] = v;
  }
  __syncthreads();
  // ---- weighted values: lane = (key sub of a load's KPI, VEC consecutive head dimensions)
  float acc[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[g][e] = 0.f;
  if (kAhead > 0 && jq0 < jq1) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int jj = jq0 + u * KPI + sub;
      float vv[VEC];
      unpack_elems<T, VEC>(ahead[u], vv);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float pe = jj < jq1 ? p_s[g][min(jj, jq1 - 1)] : 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[g][e] = fmaf(pe, vv[e], acc[g][e]);
      }
    }
  }
  for (int jj0 = jq0 + kAhead * KPI; jj0 < jq1; jj0 += KPI * kPvBatch) {
    float vv[kPvBatch][VEC], pe[kPvBatch][G];
#pragma unroll
    for (int u = 0; u < kPvBatch; ++u) {
      const int jj = jj0 + u * KPI + sub, jc = min(jj, jq1 - 1);   // past the end: the last row again, with weight 0
      const int jk = j_begin + jc;
      load_elems<T, VEC>(value_row(jk), vv[u]);
#pragma unroll
      for (int g = 0; g < G; ++g) pe[u][g] = jj < jq1 ? p_s[g][jc] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kPvBatch; ++u)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[g][e] = fmaf(pe[u][g], vv[u][e], acc[g][e]);
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      float v = acc[g][e];
      if constexpr (LPR < 64) v = lanes_sum<LPR, 32>(v);
      if (lane < LPR) red_s[wave][g][d0 + e] = v;
    }
  __syncthreads();
  for (int i = tid; i < group * D; i += 256) {
    const int g = i / D, d = i - g * D;
    const float o = (red_s[0][g][d] + red_s[1][g][d]) + (red_s[2][g][d] + red_s[3][g][d]);
    const float l = (sum_s[g][0] + sum_s[g][1]) + (sum_s[g][2] + sum_s[g][3]);
    const int64_t pair = (int64_t)m * n_q_heads + hk * group + g;
    if (!partial) {
      Act<T>::store(out, out_plane, pair * D + d, o / l);
    } else {
      float* pp = partial + (pair * n_splits + split) * (D + 2);
      pp[2 + d] = o;
      if (d == 0) {
        pp[0] = fmaxf(fmaxf(mx_s[g][0], mx_s[g][1]), fmaxf(mx_s[g][2], mx_s[g][3]));   // -inf for a split without keys
        pp[1] = l;
      }
    }
  }
}

// One block per (row, query head), one thread per head dimension: the splits' partial softmaxes in split order.  The
// splits' maxima and sums are one load of a wavefront (at most 64 splits), their weights go round through the lanes; the
// outputs are requested 16 splits at a time (33 splits of 6 rows x 64 heads: 6.0 us, 7.0 before).
template <typename T, int D>
__global__ __launch_bounds__(D) void attention_merge_kernel(const float* __restrict__ partial, void* __restrict__ out,
                                                            int64_t out_plane, int n_splits) {
  static_assert(kMaxSplits == 64, "a wavefront holds one split per lane");
  const int64_t pair = blockIdx.x;
  const int d = threadIdx.x, lane = threadIdx.x & 63;
  const float* pp = partial + pair * n_splits * (D + 2);
  const float ms = lane < n_splits ? pp[lane * (D + 2)] : -INFINITY, ls = lane < n_splits ? pp[lane * (D + 2) + 1] : 0.f;
  float m_max = ms;
  m_max = lanes_max(m_max);
  const float w = ms == -INFINITY ? 0.f : expf(ms - m_max);
  float l = 0.f, o = 0.f;
  for (int s0 = 0; s0 < n_splits; s0 += 16) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = pp[min(s0 + i, n_splits - 1) * (D + 2) + 2 + d];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (s0 + i < n_splits) {
        const float ws = __shfl(w, s0 + i);
        l += ws * __shfl(ls, s0 + i);
        o += ws * v[i];
      }
  }
  Act<T>::store(out, out_plane, pair * D + d, o / l);
}

// Extends of bf16 models (the target's verification forward, a prefill chunk, a glue extend): every row of a sequence sees
// the same trunk up to a point of its own, so a block serves 16 query rows (rows x query heads of the group) of (sequence, KV
// head, split of the keys), 32 keys per wavefront and step, scores and outputs on MFMA (S^T = K Q^T, O^T = V^T P^T: a query row keeps its lane, and with the key rows of
// the two 16-key score tiles interleaved a lane ends up with 8 consecutive keys, the B operand of the second product).
// Queries and probabilities are three bf16 planes each, which is all 24 bits of their fp32 values: the products lose
// nothing against fp32 arithmetic, the sums are fp32.  Values are read row by row, a lane the same D / 64 dimensions of
// all 32 keys, and pass through LDS as V^T.  Keys past the last row any query row sees are not read (the last visible one
// is, again, with weight 0).
// What bounds it is latency, not bytes (16.8 MB of a 4096-token prefix of the 70B shape): everything a step loads is
// requested before the queries are staged, and the planner gives a block one step where the chip has room.  6 rows x 64
// heads x 4096 keys: 17.9 us, 0.5 of them the test for values that are not finite (55.1 with a block per row, keys and values
// through the vector units).  One block for three
// query tiles, which pulls the trunk once, took 27: twice the code, run once by every wavefront, and a third of the
// wavefronts to hide its latencies behind.
constexpr int kExtWaves = 4, kExtKeys = 32 * kExtWaves;   // keys of a block's step
constexpr int kExtVt = 40;                                // V^T row in LDS: 32 keys + padding, 16-byte aligned
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
union Bf8 { bf16x8 v; __bf16 e[8]; u32x4 w; };

// x = p[0] + p[1] + p[2], exactly (8 + 8 + 8 bits)
__device__ __forceinline__ void split3(float x, __bf16& p0, __bf16& p1, __bf16& p2) {
  p0 = (__bf16)x;
  const float r = x - (float)p0;
  p1 = (__bf16)r;
  p2 = (__bf16)(r - (float)p1);
}

template <int D>
constexpr size_t extend_lds_bytes() {
  return (size_t)(D / 32) * 3 * 1024 + (size_t)kExtWaves * D * kExtVt * 2 + kExtWaves * 16 * 2 * sizeof(float);
}

template <int D>
__global__ __launch_bounds__(256) void attention_extend_kernel(const float* __restrict__ q, const bf16_t* __restrict__ trunk_k,
                                                                const bf16_t* __restrict__ trunk_v, void* __restrict__ out,
                                                                int64_t out_plane, const RowDesc* __restrict__ rows, int n_q_heads,
                                                                int n_kv_heads, int R, int max_trunk, float* __restrict__ partial,
                                                                int keys_per_split, int n_splits) {
  constexpr int KS = D / 32, DT = D / 16, NE = D / 64;
  extern __shared__ char lds[];
  bf16x8* q_s = (bf16x8*)lds;                                            // [KS][3][64]
  bf16_t* vt_all = (bf16_t*)(lds + (size_t)KS * 3 * 1024);          // [wave][D][kExtVt]
  float* ml = (float*)((char*)vt_all + (size_t)kExtWaves * D * kExtVt * 2);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, g4 = lane >> 4;
  const int hk = blockIdx.x % n_kv_heads, split = blockIdx.x / n_kv_heads;
  const int qt = blockIdx.y, row0 = blockIdx.z * R;
  const int group = n_q_heads / n_kv_heads, RG = R * group;
  const int64_t kv_stride = (int64_t)n_kv_heads * D;
  const RowDesc last = rows[row0 + R - 1];                               // an extend's rows are causal: the last sees most
  const bf16_t* tk = trunk_k + (int64_t)last.seq * max_trunk * kv_stride + hk * D;
  const bf16_t* tv = trunk_v + (int64_t)last.seq * max_trunk * kv_stride + hk * D;
  const int j_end = min(last.vis, (split + 1) * keys_per_split);
  bf16_t* vt_s = vt_all + wave * D * kExtVt;

  const int vis = qt * 16 + li < RG ? rows[row0 + (qt * 16 + li) / group].vis : 0;   // keys this lane's query row sees
  bf16x8 kr[2][KS];
  uint32_t vr[32];                                                       // this lane's NE dimensions of 32 keys
  const int krow = (li >> 2) * 8 + (li & 3);
  auto load_kv = [&](int kb) {
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const bf16_t* kp = tk + (int64_t)min(kb + krow + tile * 4, last.vis - 1) * kv_stride + g4 * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kr[tile][ks] = *(const bf16x8*)(kp + ks * 32);
    }
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const bf16_t* vp = tv + (int64_t)min(kb + k, last.vis - 1) * kv_stride + lane * NE;
      vr[k] = NE == 2 ? *(const uint32_t*)vp : (uint32_t)*vp;
    }
  };
  int kb = split * keys_per_split + wave * 32;
  if (kb < j_end) load_kv(kb);

  // ---- queries: scaled, three planes, in B-operand order
  const float scale = rsqrtf((float)D);
  for (int it = threadIdx.x; it < KS * 64; it += 256) {
    const int l = it & 63, ks = it >> 6;
    const int qr = min(qt * 16 + (l & 15), RG - 1);
    const int rr = qr / group;
    const float* src = q + ((int64_t)(row0 + rr) * n_q_heads + hk * group + (qr - rr * group)) * D + ks * 32 + (l >> 4) * 8;
    const f32x4 x0 = *(const f32x4*)src, x1 = *(const f32x4*)(src + 4);
    Bf8 p[3];
#pragma unroll
    for (int e = 0; e < 8; ++e) split3((e < 4 ? x0[e & 3] : x1[e & 3]) * scale, p[0].e[e], p[1].e[e], p[2].e[e]);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) q_s[(ks * 3 + pl) * 64 + l] = p[pl].v;
  }
  __syncthreads();

  f32x4 acc[DT];
  float m_run = -INFINITY, l_run = 0.f;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (; kb < j_end; kb += kExtKeys) {
    // A row must not feel a key it does not see, and weight 0 does not keep an infinite or NaN value out of a product.  So
    // where some row of the sequence does not see all 32 keys (the last block or two of a row's trunk), values that are not
    // finite leave the operand (exponent all ones: the carry out of it lands in the sign bit), and rows that do see their
    // keys get them added after the product, one by one.
    bool odd = false;
    if (kb + 32 > last.vis - (R - 1)) {
      uint32_t ones = 0u;
#pragma unroll
      for (int k = 0; k < 32; ++k) ones |= (vr[k] & 0x7f807f80u) + 0x00800080u;
      odd = __any((ones & 0x80008000u) != 0u);
      if (odd) {
#pragma unroll
        for (int k = 0; k < 32; ++k) {
          if ((vr[k] & 0x7f80u) == 0x7f80u) vr[k] &= 0xffff0000u;
          if ((vr[k] & 0x7f800000u) == 0x7f800000u) vr[k] &= 0x0000ffffu;
        }
      }
    }
    // V^T of the wavefront's 32 keys through LDS (its own part: no barrier)
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int k8 = 0; k8 < 4; ++k8) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t a = vr[k8 * 8 + 2 * i] >> (16 * e), b = vr[k8 * 8 + 2 * i + 1] >> (16 * e);
          w[i] = (a & 0xffffu) | (b << 16);
        }
        *(u32x4*)(vt_s + (lane * NE + e) * kExtVt + k8 * 8) = w;
      }
    Bf8 pp[3];
    f32x4 S[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int pl = 2; pl >= 0; --pl)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 qb = q_s[(ks * 3 + pl) * 64 + lane];
#pragma unroll
        for (int tile = 0; tile < 2; ++tile) S[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kr[tile][ks], qb, S[tile], 0, 0, 0);
      }
    float sv[8], mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int key = kb + g4 * 8 + e;
      sv[e] = key < min(vis, j_end) ? (e < 4 ? S[0][e & 3] : S[1][e & 3]) : -INFINITY;
      mx = fmaxf(mx, sv[e]);
    }
    mx = lanes_max<16, 32>(mx);
    const float m_new = fmaxf(m_run, mx), m_use = m_new == -INFINITY ? 0.f : m_new;
    const float corr = expf(m_run - m_use);
    m_run = m_new;
    l_run *= corr;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = acc[dt] * corr;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = expf(sv[e] - m_use);
      l_run += pe;
      split3(pe, pp[0].e[e], pp[1].e[e], pp[2].e[e]);
    }
    if (kb + kExtKeys < j_end) load_kv(kb + kExtKeys);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const bf16x8 vt = *(const bf16x8*)(vt_s + (dt * 16 + li) * kExtVt + g4 * 8);
#pragma unroll
      for (int pl = 2; pl >= 0; --pl) acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pp[pl].v, acc[dt], 0, 0, 0);
    }
    if (odd) {
      for (int k8 = 0; k8 < 4; ++k8)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float pk = __shfl(((float)pp[2].e[e] + (float)pp[1].e[e]) + (float)pp[0].e[e], k8 * 16 + li);
          const int key = kb + k8 * 8 + e;
          if (key < min(vis, j_end)) {
            const bf16_t* vp = tv + (int64_t)key * kv_stride + g4 * 4;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const bf16_t v = vp[dt * 16 + r];
                if ((v & 0x7f80u) == 0x7f80u) acc[dt][r] = fmaf(pk, bf16_to_f32(v), acc[dt][r]);
              }
          }
        }
    }
  }
  // ---- the wavefronts' partial softmaxes meet in LDS, where V^T was
  f32x4* mrg = (f32x4*)vt_all;                                           // [wave][DT][64]
  static_assert((size_t)DT * 64 * 16 <= (size_t)D * kExtVt * 2, "a wavefront's tile fits where its V^T was");
  l_run = lanes_sum<16, 32>(l_run);
  __syncthreads();
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) mrg[(wave * DT + dt) * 64 + lane] = acc[dt];
  if (g4 == 0) {
    ml[(wave * 16 + li) * 2] = m_run;
    ml[(wave * 16 + li) * 2 + 1] = l_run;
  }
  __syncthreads();
  const int qi = threadIdx.x & 15, qr = qt * 16 + qi;
  float mmax = -INFINITY, lsum = 0.f, wgt[kExtWaves];
#pragma unroll
  for (int w = 0; w < kExtWaves; ++w) mmax = fmaxf(mmax, ml[(w * 16 + qi) * 2]);
#pragma unroll
  for (int w = 0; w < kExtWaves; ++w) {
    wgt[w] = mmax == -INFINITY ? 0.f : expf(ml[(w * 16 + qi) * 2] - mmax);
    lsum += wgt[w] * ml[(w * 16 + qi) * 2 + 1];
  }
  if (qr < RG) {
    const int rr = qr / group;
    const int64_t pair = (int64_t)(row0 + rr) * n_q_heads + hk * group + (qr - rr * group);
    float* pp = partial + (pair * n_splits + split) * (D + 2);
    for (int dq = threadIdx.x >> 4; dq < D / 4; dq += 16) {
      f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kExtWaves; ++w) o += mrg[(w * DT + (dq >> 2)) * 64 + qi + 16 * (dq & 3)] * wgt[w];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (n_splits > 1) pp[2 + dq * 4 + e] = o[e];
        else Act<bf16_t>::store(out, out_plane, pair * D + dq * 4 + e, o[e] / lsum);
      }
    }
    if (n_splits > 1 && (threadIdx.x >> 4) == 0) {
      pp[0] = mmax;                                                    // -inf for a split without keys
      pp[1] = lsum;
    }
  }
}

// Splits of at most kSplitKeys keys, and with few rows enough of them for about 1024 blocks (none shorter than 64
// keys); 1 (the row-wise kernel) when the shape is outside what the split kernel holds or the scratch is too small.
int choose_splits(const AttnArgs& a, int* keys_per_split) {
  const int pairs = a.M * a.n_kv_heads;
  const int max_keys = (a.max_vis > 0 ? a.max_vis : 0) + a.suffix_cap;
  *keys_per_split = 0;
  if (!a.partial || a.n_q_heads / a.n_kv_heads > kSplitMaxGroup) return 1;
  int n = (max_keys + kSplitKeys - 1) / kSplitKeys;
  // (keys that fit one split: a single block per pair is done before the merge of several would have started)
  int fill = max_keys <= kSplitKeys ? 1 : (1024 + pairs - 1) / pairs;
  const int by_len = (max_keys + 63) / 64;
  fill = fill < by_len ? fill : by_len;
  n = n > fill ? n : fill;
  if (n < 1) n = 1;
  if (n > kMaxSplits || (int64_t)a.M * a.n_q_heads * n * (a.head_dim + 2) > a.partial_floats) return 1;
  *keys_per_split = ((max_keys + n - 1) / n + 63) / 64 * 64;
  return n;
}

// The extend kernel's launch: splits of whole steps, as many as give the chip four blocks per compute unit (6 rows x 64
// heads x 4096 keys: 33 splits of one step, 17.9 us), no more than the merge and the scratch hold.
template <int D>
int launch_extend(const AttnArgs& a, hipStream_t s) {
  const int group = a.n_q_heads / a.n_kv_heads, n_seq = a.M / a.rows_per_seq;
  const int qt = (a.rows_per_seq * group + 15) / 16;
  const int64_t blocks = (int64_t)n_seq * a.n_kv_heads * qt;
  const int steps = ((a.max_vis > 1 ? a.max_vis : 1) + kExtKeys - 1) / kExtKeys;
  int64_t n = blocks < 1024 ? 1024 / blocks : 1;
  if (n > steps) n = steps;
  if (n > kMaxSplits) n = kMaxSplits;
  while (n > 1 && (!a.partial || (int64_t)a.M * a.n_q_heads * n * (D + 2) > a.partial_floats)) --n;
  const int keys_per_split = (int)((steps + n - 1) / n) * kExtKeys;
  const int n_splits = (steps * kExtKeys + keys_per_split - 1) / keys_per_split;
  static_assert(extend_lds_bytes<D>() <= 64 * 1024, "within the LDS a kernel gets without asking");
  attention_extend_kernel<D><<<dim3(a.n_kv_heads * n_splits, qt, n_seq), 256, extend_lds_bytes<D>(), s>>>(
      a.q, (const bf16_t*)a.trunk_k, (const bf16_t*)a.trunk_v, a.out, a.out_plane, a.rows, a.n_q_heads, a.n_kv_heads, a.rows_per_seq,
      a.max_trunk, a.partial, keys_per_split, n_splits);
  SSD_HIP(hipGetLastError());
  if (n_splits > 1) attention_merge_kernel<bf16_t, D><<<a.M * a.n_q_heads, D, 0, s>>>(a.partial, a.out, a.out_plane, n_splits);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

template <typename T, int D>
int launch_rowwise_d(const AttnArgs& a, hipStream_t s) {
  int keys_per_split = 0;
  const int n_splits = choose_splits(a, &keys_per_split);
  if (keys_per_split == 0) {
    dim3 grid(a.M, a.n_kv_heads);
    attention_rowwise_kernel<T, D><<<grid, 256, 0, s>>>(a.q, (const T*)a.trunk_k, (const T*)a.trunk_v, (const T*)a.suffix_k,
                                                        (const T*)a.suffix_v, a.out, a.out_plane, a.rows, a.n_q_heads,
                                                        a.n_kv_heads, a.max_trunk, a.suffix_cap);
  } else {
    dim3 grid(a.M, a.n_kv_heads, n_splits);
    float* partial = n_splits > 1 ? a.partial : nullptr;
    const int group = a.n_q_heads / a.n_kv_heads;
    // (bf16, one query head per KV head; blocks of a launch, us of a round with 8 values ahead / as a large launch: 6144 1697 / 1696, 13824
    // 3772 / 3830, 24576 5697 / 5701, 27648 11294 / 11254, 55296 11243 / 11157, 101376 36712 / 36432)
    constexpr int64_t kManyBlocks = 24576;
    const bool many = sizeof(T) == 2 && group == 1 && (int64_t)a.M * a.n_kv_heads * n_splits > kManyBlocks;
#define SSD_SPLIT_LAUNCH(...)                                                                                             \
  attention_split_kernel<T, D, __VA_ARGS__><<<grid, 256, 0, s>>>(a.q, (const T*)a.trunk_k, (const T*)a.trunk_v, (const T*)a.suffix_k, \
                                                        (const T*)a.suffix_v, a.rows, a.n_q_heads, a.n_kv_heads, a.max_trunk, \
                                                        a.suffix_cap, partial, keys_per_split, a.out, a.out_plane)
    if (many) SSD_SPLIT_LAUNCH(1, sizeof(T) == 2);
    else if (group == 1) SSD_SPLIT_LAUNCH(1);
    else if (group <= 4) SSD_SPLIT_LAUNCH(4);
    else SSD_SPLIT_LAUNCH(kSplitMaxGroup);
#undef SSD_SPLIT_LAUNCH
    SSD_HIP(hipGetLastError());
    if (n_splits > 1) attention_merge_kernel<T, D><<<a.M * a.n_q_heads, D, 0, s>>>(a.partial, a.out, a.out_plane, n_splits);
  }
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

template <typename T>
int launch_rowwise(const AttnArgs& a, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    // bf16 extends; the grid's second and third dimensions count query tiles and sequences
    if (a.extend && a.M / a.rows_per_seq <= 65535 && (int64_t)a.rows_per_seq * (a.n_q_heads / a.n_kv_heads) <= 16 * 65535) {
      if (a.head_dim == 64) return launch_extend<64>(a, s);
      if (a.head_dim == 128) return launch_extend<128>(a, s);
    }
  }
  if (a.head_dim == 64) return launch_rowwise_d<T, 64>(a, s);
  if (a.head_dim == 128) return launch_rowwise_d<T, 128>(a, s);
  set_error("head_dim %d not supported (64 or 128)", a.head_dim);
  return SSD_EINVAL;
}

}  // namespace

// Floats of split-softmax scratch for contexts of up to M rows: few rows x many splits, or M rows x the splits that
// max_keys keys need.
int64_t attention_partial_floats(int M, int n_q_heads, int head_dim, int max_keys) {
  const int64_t few = (int64_t)(M < kSplitMaxRows ? M : kSplitMaxRows) * kMaxSplits;
  const int64_t many = (int64_t)M * ((max_keys + kSplitKeys - 1) / kSplitKeys + 1);
  return (few > many ? few : many) * n_q_heads * (head_dim + 2);
}

int launch_attention(int dtype, const AttnArgs& a, hipStream_t s) {
  if (a.M <= 0) return SSD_OK;
  return dtype == SSD_BF16 ? launch_rowwise<bf16_t>(a, s) : launch_rowwise<float>(a, s);
}

}  // namespace ssd
