// Branch-batched linear layers: y[m][n] = sum_k x[m][k] w[n][k] for a handful of rows m (the branch rows of a
// decode step, or the tokens of an extend) against a large weight matrix that is streamed from HBM once.
//
// bf16 models: MFMA 16x16x32.  The weight matrix is the MFMA A operand (16 output features x 32 inputs per
// instruction), the activations are the B operand (32 inputs x 16 rows).  Weights are kept in HBM in "tile
// order": tile (nt, kt) = 16 features x 32 inputs is 1 KiB, laid out exactly as the 64 lanes hold it (lane l:
// feature nt*16 + l%16, inputs kt*32 + (l/16)*8 .. +7), tiles of one nt consecutive over kt.  A wavefront
// therefore streams its share of a feature tile with fully coalesced 16-byte-per-lane loads.
// Activations arrive as two bf16 planes, head and remainder (x = hi + lo, written by the producing kernel), and
// take two MFMAs per weight tile, so the only bf16 rounding left in a layer is that of the weights themselves
// and of the KV cache.  With a handful of rows the extra MFMAs are free: the kernel is bound by the weight stream.
// fp32 models (the small correctness configuration): plain FMA dot products.
#include "common.h"
#include "lanes.h"

namespace ssd {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kWaves = 4;        // wavefronts per block; they split the reduction dimension
constexpr int kMaxMT = 4;        // 16-row activation tiles per block pass (64 rows)

__global__ void tile_weights_kernel(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst, int N, int Kd) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // one thread per 8-element lane chunk
  int KT = Kd / 32;
  int64_t n_chunks = (int64_t)(N / 16) * KT * 64;
  if (idx >= n_chunks) return;
  int l = (int)(idx & 63);
  int64_t tile = idx >> 6;
  int kt = (int)(tile % KT);
  int64_t nt = tile / KT;
  const bf16_t* s = src + (nt * 16 + (l & 15)) * (int64_t)Kd + kt * 32 + (l >> 4) * 8;
  *(u32x4*)(dst + idx * 8) = *(const u32x4*)s;
}

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// grid.x = N/16 feature tiles, grid.y = passes of 64 rows.  Each of the 4 wavefronts reduces a quarter of Kd;
// partial tiles meet in LDS; wavefront w finishes activation tile w.
// U = weight tiles a wavefront keeps in flight per stream (gate/up has two streams): 4 KiB did not cover the memory
// latency for the single-stream layers of large models, so they take 8 when the reduction dimension allows.
// PACK (at most 8 rows): the two planes of the activations share one B operand, the head of row r in column r, its
// remainder in column r + 8, and the columns are added at the end: one activation load and one MFMA per weight tile instead
// of two.  The loads go through the same vector memory path as the weight stream and its rows are 16 strided segments, so
// they, not HBM, set the pace: 6 rows of the 70B shape take 34 us for qkv (168 MB), 25 for o, 76 for down and 151 for
// gate/up (38, 28, 85 and 162 while the activations of a group were requested behind the next group's weights).
template <int EPI, int MT, int U, bool PACK>
__global__ __launch_bounds__(kWaves * 64) void gemm_bf16_kernel(const bf16_t* __restrict__ x, int64_t x_plane,
                                                                 const bf16_t* __restrict__ w,
                                                                 const bf16_t* __restrict__ w2, void* __restrict__ out,
                                                                 int64_t ld, int64_t out_plane, int M, int N, int Kd) {
  __shared__ f32x4 red[(EPI == EPI_SWIGLU ? 2 : 1) * kWaves * MT * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nt = blockIdx.x;
  const int m0 = blockIdx.y * (kMaxMT * 16);
  const int KT = Kd / 32;
  const int kt_per_wave = KT / kWaves;
  const int kt0 = wave * kt_per_wave;

  f32x4 acc[MT];
  f32x4 acc2[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) { acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f}; acc2[t] = (f32x4){0.f, 0.f, 0.f, 0.f}; }

  const bf16x8* wp = (const bf16x8*)(w + ((int64_t)nt * KT + kt0) * 512) + lane;
  const bf16x8* wp2 = EPI == EPI_SWIGLU ? (const bf16x8*)(w2 + ((int64_t)nt * KT + kt0) * 512) + lane : nullptr;
  // activation operand: row (clamped to M-1; those columns are never stored), 8 inputs at (lane/16)*8
  const bf16_t* xrow[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    int m = m0 + t * 16 + (lane & (PACK ? 7 : 15));
    m = m < M ? m : M - 1;
    xrow[t] = x + (int64_t)m * Kd + (int64_t)kt0 * 32 + (lane >> 4) * 8;
    if (PACK && (lane & 8)) xrow[t] += x_plane;
  }

  // Two register sets of U tiles per stream: the next group's weight loads go out before the current group is
  // multiplied, so a wavefront always has a group in flight (with one set the wavefront idled for a memory round trip per
  // group, and the layers with few feature tiles per compute unit had nobody else to fill it).
  auto load_group = [&](bf16x8* wr, bf16x8* wr2, int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      wr[u] = __builtin_nontemporal_load(wp + (int64_t)(kt + u) * 64);
      if (EPI == EPI_SWIGLU) wr2[u] = __builtin_nontemporal_load(wp2 + (int64_t)(kt + u) * 64);
    }
  };
  auto mfma_group = [&](const bf16x8* wr, const bf16x8* wr2, int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        bf16x8 hi = *(const bf16x8*)(xrow[t] + (kt + u) * 32);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[u], hi, acc[t], 0, 0, 0);
        if (EPI == EPI_SWIGLU) acc2[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr2[u], hi, acc2[t], 0, 0, 0);
        if (!PACK) {
          bf16x8 lo = *(const bf16x8*)(xrow[t] + x_plane + (kt + u) * 32);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[u], lo, acc[t], 0, 0, 0);
          if (EPI == EPI_SWIGLU) acc2[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr2[u], lo, acc2[t], 0, 0, 0);
        }
      }
    }
  };
  if constexpr (MT <= 2) {
    // Up to 32 rows: the activations of a group travel with its weights.  Requested where they are used, behind the next group's
    // weights, they made every group wait for those (loads return in order).  4 layers of the 70B shape with a head of 16384: 6 rows
    // 1476 -> 1360 us, 10 rows 1771 -> 1566, 16 rows 2127 -> 1877, 24 rows 2826 -> 2424 (groups of 4 tiles; at 6 rows they
    // measured 1393).  More row tiles do not fit the registers.
    constexpr int NX = PACK ? 1 : 2;
    bf16x8 wr[2][U], wr2[2][EPI == EPI_SWIGLU ? U : 1], xr[2][U][MT][NX];
    auto load = [&](int set, int kt) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        wr[set][u] = __builtin_nontemporal_load(wp + (int64_t)(kt + u) * 64);
        if (EPI == EPI_SWIGLU) wr2[set][u] = __builtin_nontemporal_load(wp2 + (int64_t)(kt + u) * 64);
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int i = 0; i < NX; ++i) xr[set][u][t][i] = *(const bf16x8*)(xrow[t] + i * x_plane + (kt + u) * 32);
      }
    };
    auto mul = [&](int set) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int i = 0; i < NX; ++i) {
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[set][u], xr[set][u][t][i], acc[t], 0, 0, 0);
            if (EPI == EPI_SWIGLU) acc2[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr2[set][u], xr[set][u][t][i], acc2[t], 0, 0, 0);
          }
    };
    const int n_groups = kt_per_wave / U;            // kt_per_wave is a multiple of U (host check)
    if (n_groups > 0) load(0, 0);
    int g = 0;
    for (; g + 2 <= n_groups; g += 2) {
      load(1, (g + 1) * U);
      mul(0);
      if (g + 2 < n_groups) load(0, (g + 2) * U);
      mul(1);
    }
    if (g < n_groups) mul(0);                        // odd number of groups
  } else {
  bf16x8 wa[U], wa2[U], wb[U], wb2[U];
  const int n_groups = kt_per_wave / U;            // kt_per_wave is a multiple of U (host check)
  if (n_groups > 0) load_group(wa, wa2, 0);
  int g = 0;
  for (; g + 2 <= n_groups; g += 2) {
    load_group(wb, wb2, (g + 1) * U);
    mfma_group(wa, wa2, g * U);
    if (g + 2 < n_groups) load_group(wa, wa2, (g + 2) * U);
    mfma_group(wb, wb2, (g + 1) * U);
  }
  if (g < n_groups) mfma_group(wa, wa2, g * U);    // odd number of groups: the last one is already in wa
  }

#pragma unroll
  for (int t = 0; t < MT; ++t) {
    red[(wave * MT + t) * 64 + lane] = acc[t];
    if (EPI == EPI_SWIGLU) red[kWaves * MT * 64 + (wave * MT + t) * 64 + lane] = acc2[t];
  }
  __syncthreads();
  for (int t = wave; t < MT; t += kWaves) {
    f32x4 sum = red[t * 64 + lane];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) sum += red[(v * MT + t) * 64 + lane];
    if (PACK) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] = lanes_sum<8, 8>(sum[r]);
    }
    int m = m0 + t * 16 + (lane & 15);
    int n = nt * 16 + (lane >> 4) * 4;
    f32x4 up;
    if (EPI == EPI_SWIGLU) {
      up = red[kWaves * MT * 64 + t * 64 + lane];
#pragma unroll
      for (int v = 1; v < kWaves; ++v) up += red[kWaves * MT * 64 + (v * MT + t) * 64 + lane];
      if (PACK) {
#pragma unroll
        for (int r = 0; r < 4; ++r) up[r] = lanes_sum<8, 8>(up[r]);
      }
    }
    if (m >= M) continue;
    if (EPI == EPI_STORE_F32) {
      *(f32x4*)((float*)out + (int64_t)m * ld + n) = sum;
    } else if (EPI == EPI_RESIDUAL_ADD) {
      f32x4* p = (f32x4*)((float*)out + (int64_t)m * ld + n);
      *p = *p + sum;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) Act<bf16_t>::store(out, out_plane, (int64_t)m * ld + n + r, silu(sum[r]) * up[r]);
    }
  }
}

// fp32 models.  A pass is a handful of rows over matrices of a few hundred KiB that sit in L2, so a layer costs its memory
// round trips, not its bytes: a wavefront takes one output feature (or, PAIR, two: gate and up of SwiGLU, or the two
// members of a rotary pair; TWO: two neighbours) over 1 / WPF of the reduction dimension and up to kRowsF32 rows, requests 16 bytes per lane of
// the weights and of every row at a time, kStepsF32 such steps together, and adds the lanes up with a butterfly that
// halves the number of rows it carries at each step (10 exchanges for 8 rows instead of 48).  WPF = 4 (few features, long
// reduction dimension): the four wavefronts of a block share a feature.  NORM: the input is the residual stream, the RMSNorm
// runs along in the same loads (y = 1/rms(x) * sum x gain w): no kernel of its own.  A round of the 2-layer, 256-wide
// configuration (10 rows, prefix 128): 3.4 (o), 3.5 (down), 4.5 (qkv) and 5.3 us (gate/up); 12.3, 12.3, 7.1 and 9.4 with one 4-byte element
// per lane and step, behind separate norm (4.2 us) and rotary (3.3 us) kernels.
constexpr int kRowsF32 = 8;
constexpr int kStepsF32 = 4;
enum F32Epilogue { F32_STORE = 0, F32_RESIDUAL = 1, F32_SWIGLU = 2, F32_ROPE = 3 };

// v[r] summed over the 64 lanes; lane l ends up with the sum of row l >> 3.
__device__ __forceinline__ float rows_sum(float v[kRowsF32]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = lanes_split_sum<32>(v[i], v[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) v[i] = lanes_split_sum<16>(v[i], v[i + 2]);
  return lanes_sum<4>(lanes_split_sum<8>(v[0], v[1]));
}
static_assert(kRowsF32 == 8, "rows_sum leaves row lane >> 3 in a lane");

struct GemmF32 {
  const float* x;       // [M][Kd]
  const float* gain;    // NORM: [Kd]
  const float* w;       // [N][Kd]
  const float* w2;      // SWIGLU: the up matrix
  float* out;           // STORE, RESIDUAL, SWIGLU: [M][ld]
  int64_t ld;
  int M, N, Kd;
  int m_base, rows;     // first row of this launch, rows per block (<= kRowsF32)
  float eps;
  // ROPE: out = the rotated queries [M][qd]; rotated keys and values go to the row's KV slot
  const RowDesc* desc;
  const float* cos_sin;
  float* hidden;      // STORE behind a norm: the normalised rows [M][hidden_ld], or null
  int64_t hidden_ld;
  float *trunk_k, *trunk_v, *suffix_k, *suffix_v;
  int qd, kvd, half, max_trunk, suffix_cap;
};

template <int EPI, bool NORM, int WPF, bool TWO>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32 a) {
  constexpr bool PAIR = EPI == F32_SWIGLU || EPI == F32_ROPE || TWO;
  __shared__ float part[3][4][kRowsF32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int u = WPF == 4 ? (int)blockIdx.x : (int)blockIdx.x * 4 + wave;   // feature, or feature pair (ROPE)
  const int n_units = EPI == F32_ROPE ? a.N >> 1 : (TWO ? (a.N + 1) >> 1 : a.N);
  if (WPF == 1 && u >= n_units) return;
  int n = TWO ? 2 * u : u, n2 = TWO ? min(2 * u + 1, a.N - 1) : u;
  if (EPI == F32_ROPE) {
    const int head = u / a.half;
    n = head * 2 * a.half + (u - head * a.half);
    n2 = n + a.half;
  }
  const int m0 = a.m_base + (int)blockIdx.y * a.rows, rows = min(a.rows, a.M - m0);
  const float* w1 = a.w + (int64_t)n * a.Kd;
  const float* w2 = EPI == F32_SWIGLU ? a.w2 + (int64_t)n * a.Kd : a.w + (int64_t)n2 * a.Kd;
  const int kq = (a.Kd / 4 + WPF - 1) / WPF * 4;                    // inputs per wavefront
  const int k_begin = WPF == 4 ? wave * kq : 0, k_end = min(a.Kd, k_begin + kq);
  // what the lane that ends a row's sum will want beside it, requested first: behind the sum it would cost a memory round trip
  const int r = lane >> 3, m = m0 + r, i_rope = EPI == F32_ROPE ? u % a.half : 0;
  float old[2] = {0.f, 0.f}, cos_v = 1.f, sin_v = 0.f;
  RowDesc d = {};
  if ((lane & 7) == 0 && r < rows && (WPF == 1 || wave == 0)) {
    if (EPI == F32_RESIDUAL) {
      old[0] = a.out[(int64_t)m * a.ld + n];
      if (TWO) old[1] = a.out[(int64_t)m * a.ld + n2];
    }
    if (EPI == F32_ROPE) {
      cos_v = a.cos_sin[((int64_t)m * a.half + i_rope) * 2];
      sin_v = a.cos_sin[((int64_t)m * a.half + i_rope) * 2 + 1];
      if (n >= a.qd) d = a.desc[m];
    }
  }
  float acc[kRowsF32], acc2[kRowsF32], ssq[kRowsF32];
#pragma unroll
  for (int r = 0; r < kRowsF32; ++r) { acc[r] = 0.f; acc2[r] = 0.f; ssq[r] = 0.f; }
  for (int k0 = k_begin; k0 < k_end; k0 += 256 * kStepsF32) {
#pragma unroll
    for (int st = 0; st < kStepsF32; ++st) {
      const int k = k0 + st * 256 + lane * 4;
      const bool in = k < k_end;                                     // (Kd is a multiple of 4)
      if (k0 + st * 256 >= k_end) break;
      const int kc = in ? k : k_begin;
      const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
      float4 wv = *(const float4*)(w1 + kc), wv2 = zero, g = zero;
      if (PAIR) wv2 = *(const float4*)(w2 + kc);
      if (NORM) g = *(const float4*)(a.gain + kc);
      if (!in) { wv = zero; wv2 = zero; }
#pragma unroll
      for (int r = 0; r < kRowsF32; ++r) {
        const float4 x = *(const float4*)(a.x + (int64_t)(m0 + (r < rows ? r : 0)) * a.Kd + kc);
        float v[4] = {in ? x.x : 0.f, in ? x.y : 0.f, in ? x.z : 0.f, in ? x.w : 0.f};
        if (NORM) {
#pragma unroll
          for (int e = 0; e < 4; ++e) ssq[r] = fmaf(v[e], v[e], ssq[r]);
          v[0] *= g.x; v[1] *= g.y; v[2] *= g.z; v[3] *= g.w;
        }
        acc[r] = fmaf(v[0], wv.x, fmaf(v[1], wv.y, fmaf(v[2], wv.z, fmaf(v[3], wv.w, acc[r]))));
        if (PAIR) acc2[r] = fmaf(v[0], wv2.x, fmaf(v[1], wv2.y, fmaf(v[2], wv2.z, fmaf(v[3], wv2.w, acc2[r]))));
      }
    }
  }
  float y = rows_sum(acc), y2 = 0.f, ss = 0.f;
  if (PAIR) y2 = rows_sum(acc2);
  if (NORM) ss = rows_sum(ssq);
  if (WPF == 4) {
    if ((lane & 7) == 0) {
      part[0][wave][r] = y;
      if (PAIR) part[1][wave][r] = y2;
      if (NORM) part[2][wave][r] = ss;
    }
    __syncthreads();
    if (wave != 0) return;
    auto total = [&](int i) { return (part[i][0][r] + part[i][1][r]) + (part[i][2][r] + part[i][3][r]); };
    y = total(0);
    if (PAIR) y2 = total(1);
    if (NORM) ss = total(2);
  }
  if (EPI == F32_STORE && NORM && a.hidden && u < rows) {               // (the grid has a unit for each of a group's 8 rows: host check)
    const float rs = 1.0f / sqrtf(__shfl(ss, u * 8) / (float)a.Kd + a.eps);
    for (int k = lane * 4; k < a.Kd; k += 256) {
      const float4 x = *(const float4*)(a.x + (int64_t)(m0 + u) * a.Kd + k), g = *(const float4*)(a.gain + k);
      *(float4*)(a.hidden + (int64_t)(m0 + u) * a.hidden_ld + k) = make_float4(x.x * rs * g.x, x.y * rs * g.y, x.z * rs * g.z, x.w * rs * g.w);
    }
  }
  if ((lane & 7) != 0 || r >= rows) return;
  if (NORM) {
    const float rs = 1.0f / sqrtf(ss / (float)a.Kd + a.eps);
    y *= rs;
    if (PAIR) y2 *= rs;
  }
  if (EPI == F32_STORE || EPI == F32_RESIDUAL) {
    float* dst = a.out + (int64_t)m * a.ld + n;
    dst[0] = EPI == F32_STORE ? y : old[0] + y;
    if (TWO && n2 > n) dst[1] = EPI == F32_STORE ? y2 : old[1] + y2;
  } else if (EPI == F32_SWIGLU) a.out[(int64_t)m * a.ld + n] = (y / (1.0f + expf(-y))) * y2;
  else {
    if (n < a.qd + a.kvd) {
      const float ra = y * cos_v - y2 * sin_v, rb = y2 * cos_v + y * sin_v;
      y = ra;
      y2 = rb;
    }
    float* dst = a.out + (int64_t)m * a.qd + n;
    if (n >= a.qd) {
      const int64_t row = (d.is_branch ? ((int64_t)m * a.suffix_cap + d.kv_slot) : ((int64_t)d.seq * a.max_trunk + d.kv_slot)) * a.kvd;
      if (n < a.qd + a.kvd) dst = (d.is_branch ? a.suffix_k : a.trunk_k) + row + (n - a.qd);
      else dst = (d.is_branch ? a.suffix_v : a.trunk_v) + row + (n - a.qd - a.kvd);
    }
    dst[0] = y;
    dst[a.half] = y2;
  }
}

template <int EPI>
int launch_bf16(const void* x, int64_t x_plane, const void* w, const void* w2, void* out, int64_t ld, int64_t out_plane,
                int M, int N, int Kd, hipStream_t s) {
  dim3 grid(N / 16, (M + kMaxMT * 16 - 1) / (kMaxMT * 16));
  int rows_in_pass = M < kMaxMT * 16 ? M : kMaxMT * 16;
  int mt = (rows_in_pass + 15) / 16;
  const bf16_t *xb = (const bf16_t*)x, *wb = (const bf16_t*)w, *w2b = (const bf16_t*)w2;
  const bool deep = EPI != EPI_SWIGLU && (Kd / 32 / kWaves) % 8 == 0;
#define SSD_GEMM_LAUNCH(MTV, PACK)                                                                                        \
  do {                                                                                                                   \
    if (deep && (MTV) != 2) gemm_bf16_kernel<EPI, MTV, (MTV) == 2 ? 4 : 8, PACK><<<grid, kWaves * 64, 0, s>>>(xb, x_plane, wb, w2b, out, ld, out_plane, M, N, Kd); \
    else gemm_bf16_kernel<EPI, MTV, 4, PACK><<<grid, kWaves * 64, 0, s>>>(xb, x_plane, wb, w2b, out, ld, out_plane, M, N, Kd);      \
  } while (0)
  if (M <= 8) {
    SSD_GEMM_LAUNCH(1, true);
  } else {
    switch (mt) {
      case 1: SSD_GEMM_LAUNCH(1, false); break;
      case 2: SSD_GEMM_LAUNCH(2, false); break;
      case 3: SSD_GEMM_LAUNCH(3, false); break;
      default: SSD_GEMM_LAUNCH(4, false); break;
    }
  }
#undef SSD_GEMM_LAUNCH
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

// Four wavefronts per feature where that still leaves at most four blocks per compute unit and a wavefront has at least
// one full step of 256 inputs: down of the 256-wide configuration (K = 1024) takes 4.6 us in 256 blocks, hardly more than
// o (K = 256, 64 blocks of one wavefront per feature, 4.2 us), where its reduction would be four steps in a row.
// Two features per wavefront (o, down, LM head) where the rows make several groups and the halved number of blocks is still
// three per compute unit: with many rows the loads of the rows, once per feature, are what a layer pays for.  4 layers of
// width 2048 and a head of 32000: 384 rows 15.5 -> 12.5 ms (14.3 with 16 rows of 4-byte elements per wavefront), 18 rows
// (768 blocks) 1.20 -> 1.17, 16 rows (512 blocks) 0.94 -> 1.03; width 1024: 48 rows (768) 0.81 -> 0.78, 30 rows (512)
// 0.59 -> 0.63.
template <int EPI, bool NORM>
int launch_f32(GemmF32 a, hipStream_t s) {
  const int n_units = EPI == F32_ROPE ? a.N / 2 : a.N;
  const int gy = (a.M + kRowsF32 - 1) / kRowsF32;
  a.rows = (a.M + gy - 1) / gy;
  constexpr int kMaxGridY = 65535;
  constexpr bool kPlain = EPI == F32_STORE || EPI == F32_RESIDUAL;
  const int blocks2 = ((n_units + 1) / 2 + 3) / 4;
  const bool two = kPlain && gy > 1 && (int64_t)blocks2 * gy >= 768;
  for (int y0 = 0; y0 < gy; y0 += kMaxGridY) {
    const int ny = gy - y0 < kMaxGridY ? gy - y0 : kMaxGridY;
    if ((a.m_base = y0 * a.rows) >= a.M) break;
    if (two) gemm_f32_kernel<EPI, NORM, 1, kPlain><<<dim3(blocks2, ny), 256, 0, s>>>(a);
    else if (n_units <= 1024 && a.Kd >= 1024) gemm_f32_kernel<EPI, NORM, 4, false><<<dim3(n_units, ny), 256, 0, s>>>(a);
    else gemm_f32_kernel<EPI, NORM, 1, false><<<dim3((n_units + 3) / 4, ny), 256, 0, s>>>(a);
    SSD_HIP(hipGetLastError());
  }
  return SSD_OK;
}

}  // namespace

int launch_tile_weights_bf16(const bf16_t* src, bf16_t* dst, int N, int Kd, hipStream_t s) {
  SSD_CHECK_ARG(N % 16 == 0 && Kd % (32 * kWaves * 4) == 0,
                "bf16 weight %d x %d: features must be a multiple of 16 and inputs of %d", N, Kd, 32 * kWaves * 4);
  int64_t n_chunks = (int64_t)(N / 16) * (Kd / 32) * 64;
  tile_weights_kernel<<<(int)((n_chunks + 255) / 256), 256, 0, s>>>(src, dst, N, Kd);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

int launch_gemm(int dtype, int epi, const void* x, int64_t x_plane, const void* w, const void* w2, void* out, int64_t ld,
                int64_t out_plane, int M, int N, int Kd, hipStream_t s) {
  if (M <= 0) return SSD_OK;
  if (dtype == SSD_BF16) {
    switch (epi) {
      case EPI_STORE_F32: return launch_bf16<EPI_STORE_F32>(x, x_plane, w, w2, out, ld, out_plane, M, N, Kd, s);
      case EPI_RESIDUAL_ADD: return launch_bf16<EPI_RESIDUAL_ADD>(x, x_plane, w, w2, out, ld, out_plane, M, N, Kd, s);
      default: return launch_bf16<EPI_SWIGLU>(x, x_plane, w, w2, out, ld, out_plane, M, N, Kd, s);
    }
  }
  GemmF32 a{};
  a.x = (const float*)x; a.w = (const float*)w; a.w2 = (const float*)w2; a.out = (float*)out; a.ld = ld; a.M = M; a.N = N; a.Kd = Kd;
  switch (epi) {
    case EPI_STORE_F32: return launch_f32<F32_STORE, false>(a, s);
    case EPI_RESIDUAL_ADD: return launch_f32<F32_RESIDUAL, false>(a, s);
    default: set_error("fp32 gate/up layers run with their norm (launch_norm_swiglu_f32)"); return SSD_EINVAL;
  }
}

int launch_norm_head_f32(const float* h, const float* gain, const float* w, float* logits, int64_t ld, float* hidden, int64_t hidden_ld,
                         int M, int V, int d_model, float eps, hipStream_t s) {
  if (M <= 0) return SSD_OK;
  SSD_CHECK_ARG(V >= 2 * kRowsF32 && hidden_ld % 4 == 0 && (uintptr_t)hidden % 16 == 0, "fp32 head of %d features", V);
  GemmF32 a{};
  a.x = h; a.gain = gain; a.w = w; a.out = logits; a.ld = ld; a.M = M; a.N = V; a.Kd = d_model; a.eps = eps; a.hidden = hidden; a.hidden_ld = hidden_ld;
  return launch_f32<F32_STORE, true>(a, s);
}

int launch_norm_swiglu_f32(const float* h, const float* gain, const float* w_gate, const float* w_up, float* act, int M, int d_ffn,
                           int d_model, float eps, hipStream_t s) {
  if (M <= 0) return SSD_OK;
  GemmF32 a{};
  a.x = h; a.gain = gain; a.w = w_gate; a.w2 = w_up; a.out = act; a.ld = d_ffn; a.M = M; a.N = d_ffn; a.Kd = d_model; a.eps = eps;
  return launch_f32<F32_SWIGLU, true>(a, s);
}

int launch_norm_qkv_rope_f32(const float* h, const float* gain, const float* wqkv, float* q, float* trunk_k, float* trunk_v,
                             float* suffix_k, float* suffix_v, const RowDesc* rows, const float* cos_sin, int M, const Dims& d,
                             int max_trunk, int suffix_cap, hipStream_t s) {
  if (M <= 0) return SSD_OK;
  GemmF32 a{};
  a.x = h; a.gain = gain; a.w = wqkv; a.out = q; a.M = M; a.N = d.qkv_dim(); a.Kd = d.d_model; a.eps = d.rms_eps;
  a.desc = rows; a.cos_sin = cos_sin; a.trunk_k = trunk_k; a.trunk_v = trunk_v; a.suffix_k = suffix_k; a.suffix_v = suffix_v;
  a.qd = d.q_dim(); a.kvd = d.kv_dim(); a.half = d.head_dim / 2; a.max_trunk = max_trunk; a.suffix_cap = suffix_cap;
  return launch_f32<F32_ROPE, true>(a, s);
}

}  // namespace ssd
