// The fused decode pass (see fused.h): every phase of the decoder runs on all compute units at once inside one
// persistent kernel.
//
// Linear layers.  A workgroup owns whole output-feature tiles ("owner computes"): over the full reduction dimension
// for the qkv, gate/up and LM-head projections, over one of 2 or 4 k-slices of it for the o and down projections,
// whose slices hand their partial tiles to slice 0 through memory; slice 0 adds them in slice order, so the result
// does not depend on timing.  The 8 wavefronts of a workgroup split its reduction range; each streams its own
// contiguous run of 1 KiB weight tiles (MFMA 16x16x32 A operands, fp16) and reads the matching activation tiles (B
// operands: 16 rows x 32 inputs, written by the producing phase as fp16 head/remainder planes in exactly the lane
// order the MFMA wants).  Two loop shapes: where a workgroup has at most one unit (qkv, o, down, and with one activation
// plane gate/up) ALL its weight tiles are requested before it waits at the grid barrier in front of the phase; the LM head,
// and gate/up with two planes, stream weights and activations together through a ring of register chunks whose first
// chunks go out before the barrier.
// Weights depend on nothing, so HBM keeps streaming while the barrier and the activation exchange take their latency.
// One exchange needs less than the grid: an attention unit reads the projections of its KV head's group only, so the
// qkv units of a group announce themselves in a line of flags that the group's attention units poll (group_wait), and
// no grid barrier stands between a layer's qkv phase and its attention phase.
//
// RMSNorm is split around the linear layer: the producer of the residual stream writes (h * gain) and the
// per-feature-tile sums of h^2; the consumer multiplies its accumulators by the row's 1/rms.
//
// Attention (App. B: every branch row sees the verified trunk up to its fork point plus its own path).  The trunk
// keys of one (sequence, KV head) are shared by all rows and all query heads of the group, so they are scored with
// MFMAs: a unit = (sequence, KV head, one 16-row query tile of rows x group heads, key split); S^T = K Q^T and
// O^T = V^T P^T keep every query row in a fixed lane, so the probabilities feed the second MFMA without leaving their
// registers (the two 16-key score tiles take interleaved key rows so that each lane ends up with 8 consecutive
// keys).  Values are stored transposed in the trunk.  The keys computed in this very pass (a branch row's own token
// and its earlier branch tokens, the other tokens of an extend) are rotated and staged in LDS by the unit and go
// through the same MFMAs under a per-row visibility test; the unit appends them to the KV store afterwards.  With
// one key split the unit writes the final output; with several, every unit stores its partial softmax and counts its
// arrival, and the unit that arrives last of a tile's splits merges them in split order (wide passes: a merge phase).
// No mask is ever materialised: a row is (visible trunk length, private suffix length).
#include <type_traits>
#include <vector>

#include "fused.h"
#include "lanes.h"
#include "wide_blocks.h"
#include "wide_rows.h"

namespace ssd {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
// pointers into global memory: loads and stores through these are global_*, never flat_* instructions
typedef __attribute__((address_space(1))) bf16x8 gbf16x8;
typedef __attribute__((address_space(1))) f32x4 gf32x4;
typedef __attribute__((address_space(1))) u32x2 gu32x2;
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) bf16_t gbf16;

// 16-bit planes per activation tensor: 2 = head + remainder, 1 = the head alone.  xn: (h * gain) feeding qkv, gate/up
// and the LM head; att: attention output feeding the o-projection; act: SwiGLU output feeding the down-projection:
// these three meet the weights and are fp16 (head alone: 11 significant bits; with the remainder about 22).  q, p: the
// rotated queries and the softmax probabilities inside the attention unit, which meet the bf16 keys and values and are
// bf16 (8 bits, or about 16 with the remainder).
template <int X, int T, int C, int Q, int P>
struct Planes {
  static constexpr int xn = X, att = T, act = C, q = Q, p = P;
};
constexpr float kLog2e = 1.4426950408889634f;

// Workgroup barrier that waits for LDS traffic only: global loads issued before it stay in flight.
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Write-through stores: visible to every other compute unit once the issuing wavefront's vmcnt reaches zero.
__device__ __forceinline__ void st_u64(void* p, uint64_t v) {
  __hip_atomic_store((uint64_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_f32(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t pack_f32x2(float a, float b) {
  return (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32);
}
__device__ __forceinline__ void st_f32x4(float* p, f32x4 v) {
  st_u64(p, pack_f32x2(v[0], v[1]));
  st_u64(p + 2, pack_f32x2(v[2], v[3]));
}
// Partial tiles of a K-split are their own "ready" flag: a word that holds kFixEmpty (a NaN pattern no sum of
// products produces) has not been written in this launch.  The reader takes the tile with agent-scope loads (coherent
// across the XCDs) and writes kFixEmpty back.
constexpr unsigned kFixEmpty = 0xffffffffu;
__device__ __forceinline__ f32x4 ld_f32x4_coherent(const float* p) {
  const uint64_t a = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t b = __hip_atomic_load((const uint64_t*)p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (f32x4){__uint_as_float((unsigned)a), __uint_as_float((unsigned)(a >> 32)), __uint_as_float((unsigned)b),
                 __uint_as_float((unsigned)(b >> 32))};
}
__device__ __forceinline__ bool fix_ready(f32x4 v) {
  return __float_as_uint(v[0]) != kFixEmpty && __float_as_uint(v[1]) != kFixEmpty && __float_as_uint(v[2]) != kFixEmpty &&
         __float_as_uint(v[3]) != kFixEmpty;
}
__device__ __forceinline__ f32x4 fix_empty() {
  const float e = __uint_as_float(kFixEmpty);
  return (f32x4){e, e, e, e};
}
// A plain 16-byte store the compiler does not see as a memory operation.  With a store pending, the compiler's waits
// for loads degrade to "wait for everything", which would empty the weight pipeline at every unit of the LM head.
// Hidden, the store only makes a later counted wait err on the safe side: loads complete in order among themselves,
// so "at most N operations outstanding" still implies that every load older than the N youngest has arrived.
// (the s_nop: a VALU write of its data registers has to stay two instructions behind a store of more than 8 bytes, a hazard the
// compiler covers for its own stores and cannot see inside this one; and v must come from a VALU instruction, not straight from an
// MFMA, whose latency it would not wait out either)
__device__ __forceinline__ void st_f32x4_uncounted(float* p, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" : : "v"(p), "v"(v));
}
// Thread coordinates read afresh where they are called: everything derived from them (row and tile indices, LDS and
// global addresses) is then local to the phase that computes it.  Derived from the kernel-wide threadIdx they would be
// hoisted out of the phase loop, stay live through every phase and be spilled where registers are short.  (With the linear
// layers and the row scales on fresh indices the instances use at most 28 bytes of scratch, up to 120 before: a
// 24-row round over 1024 keys of the 1B shape 5162 -> 5057 us, 8 rows over 211 keys 3098 -> 3044.  With the attention unit
// on fresh indices as well, beside the gate/up loop that holds all its weights: 4968 -> 4941, 2965 -> 2939, and 48 rows
// over 8192 keys 7429 -> 7310, but single-token drafting 3950 -> 3985.)
struct ThreadIds { int tid, lane, wave; };
__device__ __forceinline__ ThreadIds fresh_thread_ids() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return ThreadIds{t, t & 63, __builtin_amdgcn_readfirstlane(t >> 6)};
}
// The lane index, recomputed where it is called (the compiler can neither hoist nor remember the result).
__device__ __forceinline__ int fresh_lane_id() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}
__device__ __forceinline__ uint64_t pack_bf16x4(bf16_t a, bf16_t b, bf16_t c, bf16_t d) {
  return (uint64_t)a | ((uint64_t)b << 16) | ((uint64_t)c << 32) | ((uint64_t)d << 48);
}
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
// fp32 -> bf16, round to nearest even, on the conversion unit gfx950 has for it (v_cvt_pk_bf16_f32): the softmax and the
// head/remainder splits convert thousands of values per phase, and the integer sequence costs ~8 VALU instructions each
__device__ __forceinline__ bf16_t to_bf16(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
// The linear layers multiply in fp16 x fp16 -> fp32.  An activation that travels as ONE 16-bit plane keeps 11 significant
// bits in fp16 where bf16 keeps 8: through 16 layers that is 2.5e-3 instead of 2e-2 between the hidden states and a
// float64 reference (measured on 384-row passes), for the same bytes and the same MFMA rate.  The weights are converted
// once, when the stream-order layout is built (exact for |w| >= 2^-14; smaller ones round to fp16 subnormals, absolute
// error <= 2^-25); activations saturate at the fp16 range.  Keys, values, queries and probabilities stay bf16.
__device__ __forceinline__ uint16_t to_f16(float x) {
  const _Float16 h = (_Float16)fminf(fmaxf(x, -65504.0f), 65504.0f);
  return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float f16_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
__device__ __forceinline__ f32x4 mfma16_f16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32_f16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Optional phase clocks (a measurement aid): [phase][slot][workgroup] ticks of the 100 MHz real-time counter; slot 0
// phase entry, 1 after the grid barrier, 2 end of the phase's work, 3.. probes inside a phase (wide passes: 6 and 7 of the
// o- and down-projections are entry and end of the residual launch behind them).
__device__ __forceinline__ void stamp(const FusedParams& p, int ph, int which, int column) {
  // (launches of more workgroups than the grid of the persistent kernel - the attention, merge and hidden-state launches
  // of a wide pass - record their first p.nwg workgroups: the table has p.nwg columns)
  if (p.prof && threadIdx.x == 0 && column < p.nwg)
    p.prof[((int64_t)ph * kFusedClockSlots + which) * p.nwg + column] = __builtin_amdgcn_s_memrealtime();
}
__device__ __forceinline__ void stamp(const FusedParams& p, int ph, int which) { stamp(p, ph, which, (int)blockIdx.x); }

// Offset of element (row m, input k) in a B-operand-ordered activation plane with MT row tiles:
// [k / 32][m / 16][lane = m % 16 + 16 ((k % 32) / 8)][k % 8].
__device__ __forceinline__ int64_t b_off_of(int mt, int k, int m) {
  return ((int64_t)((k >> 5) * mt + (m >> 4)) * 64 + (m & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}
template <int MT>
__device__ __forceinline__ int64_t b_off(int k, int m) {
  return b_off_of(MT, k, m);
}

union Bf8 {
  bf16x8 v;
  uint16_t u[8];
  u32x4 w;
};

// ---------------------------------------------------------------------------------------------- grid barrier
// Two levels: kBarGroups group counters (workgroup g arrives at counter g % kBarGroups), the last arrival of a group
// publishes the epoch in that group's flag, every workgroup polls all the flags.  Relaxed agent-scope atomics only: data written
// before the arrival went out with write-through stores and s_waitcnt 0.  Every wait is bounded; on expiry the
// error word is set and the workgroup leaves the kernel.
constexpr int kBarGroups = 2;        // a power of two that divides the grid; measured per layer of the 1B shape:
                                     // 1 group 51.7 us, 2 50.5, 4 50.9, 8 51.3, 16 52.2, 32 53.8 (more flags to poll
                                     // against fewer arrivals queueing at one counter)
constexpr int kBarFlags = 1024;      // barrier words: group counters at 32 g (a cache line each), flags at 1024 + g,
constexpr int kBarEpochWord = 1100;  // the epoch here
struct Grid {
  unsigned* bar;
  unsigned* err;
  unsigned epoch;
  int persistent;
  int nwg;
  int* dead;   // LDS
  unsigned spin_limit;   // polls a bounded wait may take before it gives up
};

__device__ __forceinline__ void grid_arrive(Grid& g) {
  if (!g.persistent) return;
  __builtin_amdgcn_s_waitcnt(0);
  wg_barrier();
  ++g.epoch;
  if (threadIdx.x == 0) {
    unsigned grp = blockIdx.x & (unsigned)(kBarGroups - 1), per = (unsigned)g.nwg / kBarGroups;
    unsigned old = __hip_atomic_fetch_add(g.bar + 32 * grp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 == g.epoch * per)
      __hip_atomic_store(g.bar + kBarFlags + grp, g.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ bool grid_wait(Grid& g) {
  if (!g.persistent) return true;
  if (threadIdx.x < kBarGroups) {
    unsigned spins = 0;
    // (compared as a signed difference: the epoch counts on across launches and may wrap)
    while ((int)(__hip_atomic_load(g.bar + kBarFlags + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - g.epoch) < 0) {
      if (++spins > g.spin_limit) {
        __hip_atomic_store(g.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        *g.dead = 1;
        break;
      }
      // no pause between polls: each one already takes a memory round trip, and only kBarGroups lanes of a
      // workgroup poll (measured: 0.3 us per layer faster than with a 64-cycle sleep; several polls in flight: no gain)
    }
  }
  wg_barrier();
  return *g.dead == 0;
}

// Attention needs less than the whole grid behind it: an attention unit of KV head g reads the projections of that
// head's group only (its query heads, its key head, its value head), which `n` workgroups own in the qkv phase.  Each of
// them, once its stores have left, writes the current barrier number into its word of the group's line of flags
// (one 64-byte line per layer and group); the unit polls that one line.  The grid barrier between the qkv and the
// attention phase is gone with it; workgroups without a unit pass straight on.  The barrier number is the same on
// both sides (nobody arrives at a grid barrier in between) and differs from launch to launch.
__device__ __forceinline__ bool group_wait(Grid& g, const unsigned* line, int n) {
  if (!g.persistent) return true;
  if ((int)threadIdx.x < n) {
    unsigned spins = 0;
    while (__hip_atomic_load(line + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != g.epoch) {
      if (++spins > g.spin_limit) {
        __hip_atomic_store(g.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        *g.dead = 1;
        break;
      }
    }
  }
  wg_barrier();
  return *g.dead == 0;
}

// 1/rms of every row from the per-feature-tile partial sums of squares: r_s[m] (LDS).  MP: row capacity of the workspace.
template <int MP>
__device__ __forceinline__ void compute_row_scales(const FusedParams& p, const float* ssq, float* r_s) {
  const int n_tiles = p.d >> 4;
  const int tid = fresh_thread_ids().tid;
  const int m = tid >> 3, part = tid & 7;
  const gfloat* src = (const gfloat*)ssq + (m < p.M ? m : 0);
  float s = 0.f;
  // 16 independent loads at a time: a chain of dependent loads would cost a memory latency each
  for (int j0 = part; j0 < n_tiles; j0 += 128) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int j = j0 + 8 * i;
      v[i] = src[(j < n_tiles ? j : j0) * MP];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s += j0 + 8 * i < n_tiles ? v[i] : 0.f;
  }
  s = lanes_sum<1, 4>(s);
  if (m < p.M && part == 0) r_s[m] = 1.0f / sqrtf(s / (float)p.d + p.eps);
  wg_barrier();
}

// The same in two halves around other work, for gate/up with its weights ahead (see gemm_phase): the sums are requested, and met
// later.  N: feature tiles of the model width for each of a row's 8 threads.  The caller's next workgroup barrier publishes r_s.
// tid: the thread index, read afresh by the caller.
template <int MP, int N>
__device__ __forceinline__ void row_scales_issue(const FusedParams& p, const float* ssq, float (&v)[N], int tid) {
  const unsigned off = ((tid >> 3) < p.M ? tid >> 3 : 0) + (tid & 7) * MP;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = ((const gfloat*)ssq + 8 * i * MP)[off];
}
template <int N>
__device__ __forceinline__ void row_scales_finish(const FusedParams& p, const float (&v)[N], float* r_s, int tid) {
  const int m = tid >> 3;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) s += v[i];
  s = lanes_sum<1, 4>(s);
  if (m < p.M && (tid & 7) == 0) r_s[m] = 1.0f / sqrtf(s / (float)p.d + p.eps);
}

// Residual-stream epilogue shared by the embedding, the o-projection and the down-projection: store the new h
// (4 consecutive features n..n+3 of row m per lane), (h * gain) as fp16 head/remainder planes for the next linear
// layer, and this feature tile's sum of squares per row.
template <int MT, int MP, int NPX>
__device__ __forceinline__ void resid_store(const FusedParams& p, f32x4 hn, int m, int n, int lane, u32x2 gb,
                                            float* h_out, bf16_t* xn_out, float* ssq_out, int tile) {
  const bool ok = m < p.M;
  float s = 0.f;
  if (ok) {
    st_f32x4(h_out + (int64_t)m * p.d + n, hn);
    float g[4] = {__uint_as_float(gb.x << 16), __uint_as_float(gb.x & 0xffff0000u), __uint_as_float(gb.y << 16),
                  __uint_as_float(gb.y & 0xffff0000u)};
    bf16_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float x = hn[i] * g[i];
      hi[i] = to_f16(x);
      lo[i] = to_f16(x - f16_to_f32(hi[i]));
      s += hn[i] * hn[i];
    }
    int64_t off = b_off<MT>(n, m);
    st_u64(xn_out + off, pack_bf16x4(hi[0], hi[1], hi[2], hi[3]));
    if (NPX == 2) st_u64(xn_out + (int64_t)MP * p.d + off, pack_bf16x4(lo[0], lo[1], lo[2], lo[3]));
  }
  s = lanes_sum<16, 32>(s);
  if (ok && lane < 16) st_f32(ssq_out + tile * MP + m, s);
}

// ---------------------------------------------------------------------------------------------- linear layers
enum { FE_QKV = 0, FE_RESID = 1, FE_SWIGLU = 2, FE_LOGITS = 3, FE_PART = 4 };   // FE_PART: wide passes only

struct EpiArgs {
  float* out;          // QKV: [M][ld] raw projections; LOGITS: [M][ld] logits
  int64_t ld;
  const float* h_in;   // RESID
  float* h_out;
  const bf16_t* gain;
  bf16_t* xn_out;
  float* ssq_out;
  bf16_t* act_out;     // SWIGLU
  float* fix_buf;      // K-split: [tile group][slice][tile][64 lanes][4] partial tiles of this phase instance
};

template <int AT, int MT, int NP>
struct Chunk {
  bf16x8 a[AT];
  bf16x8 b[MT * NP];
};

// One linear layer over the workgroup's units.  bsrc: activation planes in B-operand order, `bplane` elements apart.
// ssq_in: if not null, row scales are computed into r_s after the barrier (SWIGLU and LOGITS need them).
// AT = 2 serves the qkv, o and down projections (epilogue FE_QKV / FE_RESID), AT = 4 the gate/up projection and the
// LM head (FE_SWIGLU / FE_LOGITS).  The epilogue kind is a run-time argument so that the loop of qkv, o and down, and the ring,
// exist once each in the kernel, beside gate/up's: the code has to stay resident in the instruction cache across the layers.
// MP: row capacity of the workspace; NPX / NPC: planes of the (h * gain) / SwiGLU outputs the epilogues write.
// KT: k-tiles per wavefront and unit of gate/up with its weights ahead.
template <int AT, int MT, int NP, int D, bool PRE, int MP, int NPX, int NPC, int KT = 0>
__device__ __forceinline__ bool gemm_phase(const FusedParams& p, const FusedGemm g, const bf16_t* bsrc, int64_t bplane,
                                           const int EPI, const EpiArgs& e, Grid& grid, bool do_wait, f32x4* red, float* r_s,
                                           const float* ssq_in, int ph, int my_unit) {
  // my_unit: the unit of this workgroup in a phase of at most one unit per workgroup (PRE), or -1
  const ThreadIds ids = fresh_thread_ids();
  const int lane = ids.lane, wave = ids.wave;
  const int KTW = g.KTW;
  // K-split (g.KS > 1, at most one unit per workgroup): unit u = (feature-tile group u / KS, k-slice u % KS)
  const int KS = g.KS, ks = KS > 1 ? (my_unit < 0 ? 0 : my_unit % KS) : 0;
  const gbf16x8* b_first = (const gbf16x8*)(bsrc + ((int64_t)((ks * kFusedWaves + wave) * KTW) * MT * 64 + lane) * 8);
  const int64_t bplane_v = bplane / 8;

  f32x4 acc[AT][MT];
#pragma unroll
  for (int j = 0; j < AT; ++j)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[j][t] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // End of a unit: sum the 8 wavefronts' partial tiles in LDS and run the epilogue.
  auto finish_unit = [&](int unit) {
    // The lane index of the epilogue is read afresh here: addresses derived from the function-wide `lane` would be
    // kept across the streaming loop, where registers are short, spilled, and their reloads (memory loads like any
    // other) would make the compiler wait for the whole weight pipeline at every unit.
    const int lane = fresh_lane_id();
    // the residual-stream tile and the gains this wavefront's epilogue will want: requested now, so that they arrive
    // under the LDS reduction and the K-split fix-up instead of costing a memory latency at the very end
    f32x4 h_pre = (f32x4){0.f, 0.f, 0.f, 0.f};
    u32x2 gain_pre = (u32x2){0u, 0u};
    if (AT <= 2 && EPI == FE_RESID && wave < AT * MT && ks == 0) {
      const int j = wave / MT, t = wave - j * MT;
      const int tile = (KS > 1 ? unit / KS : unit) * AT + j;
      const int m = t * 16 + (lane & 15), n = tile * 16 + (lane >> 4) * 4;
      if (m < p.M) h_pre = *(const gf32x4*)(e.h_in + (int64_t)m * p.d + n);
      gain_pre = *(const gu32x2*)(e.gain + n);
    }
#pragma unroll
    for (int j = 0; j < AT; ++j)
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        red[(wave * (AT * MT) + j * MT + t) * 64 + lane] = acc[j][t];
        acc[j][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
    wg_barrier();
    const int NOUT = EPI == FE_SWIGLU ? 2 * MT : AT * MT;
    const int tg = KS > 1 ? unit / KS : unit;     // feature-tile group of the unit
    if (KS > 1 && ks > 0) {
      // K-split, slices 1..: publish the reduced tiles.  The partial-tile buffer holds kFixEmpty words between
      // launches, so the data are their own "ready" flag and no counter or extra round trip is needed.
      float* fix = e.fix_buf + ((int64_t)tg * KS) * (AT * MT) * 256;
      for (int idx = wave; idx < AT * MT; idx += kFusedWaves) {
        f32x4 v = red[idx * 64 + lane];
#pragma unroll
        for (int w = 1; w < kFusedWaves; ++w) v += red[(w * (AT * MT) + idx) * 64 + lane];
        st_f32x4(fix + ((int64_t)ks * (AT * MT) + idx) * 256 + lane * 4, v);
      }
      __builtin_amdgcn_s_waitcnt(0);
      wg_barrier();
      return;
    }
    for (int idx = wave; idx < NOUT; idx += kFusedWaves) {
      const int j = idx / MT, t = idx - j * MT;
      f32x4 v = red[(j * MT + t) * 64 + lane];
#pragma unroll
      for (int w = 1; w < kFusedWaves; ++w) v += red[(w * (AT * MT) + j * MT + t) * 64 + lane];
      if (KS > 1) {
        // Ordered fix-up: slice 0 polls the other slices' tiles until no word is kFixEmpty, adds them in slice order
        // (the result does not depend on timing) and puts kFixEmpty back for the next launch.
        float* fix = e.fix_buf + ((int64_t)tg * KS) * (AT * MT) * 256 + (int64_t)idx * 256 + lane * 4;
        f32x4 pv[kFusedMaxSlices - 1];
        unsigned pending = (1u << (KS - 1)) - 1u, spins = 0;
        while (pending) {
#pragma unroll
          for (int q = 0; q < kFusedMaxSlices - 1; ++q)
            if (pending >> q & 1u) pv[q] = ld_f32x4_coherent(fix + (int64_t)(q + 1) * (AT * MT) * 256);
#pragma unroll
          for (int q = 0; q < kFusedMaxSlices - 1; ++q)
            if ((pending >> q & 1u) && fix_ready(pv[q])) pending &= ~(1u << q);
          if (pending && ++spins > grid.spin_limit) {
            __hip_atomic_store(grid.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            *grid.dead = 1;
            break;
          }
        }
#pragma unroll
        for (int q = 0; q < kFusedMaxSlices - 1; ++q)
          if (q + 1 < KS) {
            v += pv[q];
            st_f32x4(fix + (int64_t)(q + 1) * (AT * MT) * 256, fix_empty());
          }
      }
      const int m = t * 16 + (lane & 15);
      const int f4 = (lane >> 4) * 4;
      if (AT <= 2 && EPI == FE_QKV) {
        const int n = (tg * AT + j) * 16 + f4;
        if (m < p.M) st_f32x4(e.out + (int64_t)m * e.ld + n, v);
      } else if (AT <= 2 && EPI == FE_RESID) {
        const int tile = tg * AT + j;
        const int n = tile * 16 + f4;
        resid_store<MT, MP, NPX>(p, h_pre + v, m, n, lane, gain_pre, e.h_out, e.xn_out, e.ssq_out, tile);   // idx == wave here
      } else if (AT == 4 && EPI == FE_SWIGLU) {
        // tiles 0,1 of the unit are gate, 2,3 the matching up tiles; idx = (gate tile j, row tile t)
        f32x4 u = red[((j + 2) * MT + t) * 64 + lane];
#pragma unroll
        for (int w = 1; w < kFusedWaves; ++w) u += red[(w * (AT * MT) + (j + 2) * MT + t) * 64 + lane];
        if (m < p.M) {
          const float rs = r_s[m];
          bf16_t hi[4], lo[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float gg = v[i] * rs, uu = u[i] * rs;
            float a = gg / (1.0f + __expf(-gg)) * uu;
            hi[i] = to_f16(a);
            lo[i] = to_f16(a - f16_to_f32(hi[i]));
          }
          const int k = unit * 32 + j * 16 + f4;    // input index of the down-projection
          int64_t off = b_off<MT>(k, m);
          st_u64(e.act_out + off, pack_bf16x4(hi[0], hi[1], hi[2], hi[3]));
          if (NPC == 2) st_u64(e.act_out + (int64_t)MP * p.ffn + off, pack_bf16x4(lo[0], lo[1], lo[2], lo[3]));
        }
      } else if (AT == 4) {
        const int tile = unit * AT + j;
        const int n = tile * 16 + f4;
        if (m < p.M && tile < g.NT) {
          const float rs = r_s[m];
          st_f32x4_uncounted(e.out + (int64_t)m * e.ld + n, v * rs);
        }
      }
    }
    // Loads and stores share one counter and may complete out of order with respect to each other: drain it here,
    // once per unit, so that the chunk waits in the streaming loop stay exact.  The LM head, the one phase with several
    // units per workgroup, must not drain (the next unit's weights are already in flight): its stores are not counted
    // (see st_f32x4_uncounted) and complete under the next unit; the drain before the grid barrier covers them.
    if (EPI != FE_LOGITS) __builtin_amdgcn_s_waitcnt(0);
    wg_barrier();
  };


  if constexpr (PRE && AT == 4) {
    // ---- gate/up with at most one unit per workgroup: ALL of a wavefront's weight tiles are requested before the workgroup
    // waits at the barrier (the ring below: 3 of 8 k-tiles), activation tiles through a ring behind it, and the row scales, which
    // only the epilogue wants, are requested with the first activation tiles and met after the MFMAs.  Bound by the 67 MB of
    // weights of a layer of the 1B shape, 9.3 of the 13 us the phase now takes with its barrier (16 before), and by the exchange before
    // it: the flood slows the o-projection's last workgroups, so more of it, earlier, loses (requested under the o-projection: 24-row
    // rounds over 1024 keys 4.97 -> 5.8 ms; a part held back until the barrier: 5.0 to 5.2).  Against the ring, 24 rows over 1024
    // keys 5057 -> 4968 us per round, 8 rows over 211 keys 3044 -> 2971, single-token drafting 4000 -> 3945, 48 rows over 8192 keys
    // 7429 -> 7415.  (The scales behind the MFMAs alone: 4988 -> 4960, 2990 -> 2957, single-token drafting 3980 -> 4007, 48 rows over 8192
    // keys 7139 -> 7131.)  16 layers of width 1024 (d_ffn 4096) and
    // 512 (2048), rounds: 8 rows over 211 keys 2215 -> 2083 and 2078 -> 1975, 24 rows over 1024 keys 3666 -> 3472 and 3443 -> 3263, 48 rows
    // over 8192 keys 4771 -> 4563 and 4131 -> 3941; five single tokens over 1024 keys 2794 -> 2639 and 2633 -> 2463.
    if (my_unit >= g.n_units) {
      if (do_wait && !grid_wait(grid)) return false;
      stamp(p, ph, 1);
      return true;
    }
    // chunks of activation tiles in flight, as the registers allow: 1 row tile 8 (single-token drafting 3999 -> 3973 us with 8
    // instead of 4), 2 row tiles 4 (6 use scratch and gain nothing), 3 row tiles 3 (48 rows over 8192 keys 7222 -> 7140 us with 3
    // instead of 2, of 28 bytes of scratch; 4 use more: 7205)
    constexpr int DA = KT, DB_MAX = MT * NP > 2 ? 3 : MT * NP > 1 ? 4 : 8, DB = DB_MAX < DA ? DB_MAX : DA;
    const gbf16x8* a_next = (const gbf16x8*)(g.w + (((int64_t)my_unit * kFusedWaves + wave) * DA * AT) * 512);
    bf16x8 a[DA][AT], b[DB][MT * NP];
    auto load_a = [&](bf16x8 (&dst)[AT]) {
#pragma unroll
      for (int j = 0; j < AT; ++j) dst[j] = __builtin_nontemporal_load(a_next + j * 64 + (unsigned)lane);
      a_next += AT * 64;
    };
#pragma unroll
    for (int c = 0; c < DA; ++c) load_a(a[c]);
    if (do_wait && !grid_wait(grid)) return false;
    stamp(p, ph, 1);
    unsigned b_lane[MT];   // rows beyond M (padding of the last row tile) are not fetched: their lanes re-read row 0
#pragma unroll
    for (int t = 0; t < MT; ++t) b_lane[t] = lane - (t * 16 + (lane & 15) < p.M ? 0 : (lane & 15));
    const gbf16x8* b_next = (const gbf16x8*)(bsrc + (int64_t)(wave * DA) * MT * 512);
    auto load_b = [&](bf16x8 (&dst)[MT * NP]) {
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) dst[t * NP + pl] = (b_next + pl * bplane_v + t * 64)[b_lane[t]];
      b_next += MT * 64;
    };
    auto mfma_chunk = [&](const bf16x8 (&ca)[AT], const bf16x8 (&cb)[MT * NP]) {
#pragma unroll
      for (int j = 0; j < AT; ++j)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int pl = 0; pl < NP; ++pl) acc[j][t] = mfma16_f16(ca[j], cb[t * NP + pl], acc[j][t]);
    };
#pragma unroll
    for (int c = 0; c < DB - 1; ++c) load_b(b[c]);
    float ssq_v[2 * KT];   // KT k-tiles of 32 inputs in each of 8 wavefronts: 16 KT feature tiles, 2 KT for each of a row's 8 threads
    row_scales_issue<MP>(p, ssq_in, ssq_v, ids.tid);
    stamp(p, ph, 3);
#pragma unroll
    for (int c = 0; c < DA; ++c) {
      if (c + DB - 1 < DA) load_b(b[(c + DB - 1) % DB]);
      mfma_chunk(a[c], b[c % DB]);
    }
    stamp(p, ph, 4);
    row_scales_finish(p, ssq_v, r_s, ids.tid);
    stamp(p, ph, 5);
    finish_unit(my_unit);
    return true;
  } else if constexpr (PRE) {
    // ---- at most one unit per workgroup (the host checks n_units <= grid): ALL of the wavefront's weight tiles are
    // requested before the workgroup waits at the barrier, so the weight stream of the phase runs under the barrier
    // latency, the activation fetch and the row scales; after the barrier only the activation tiles (L2) are loaded,
    // through a short ring.  KTW is a run-time value: one fully unrolled instance per supported value, so that every
    // register index is static and the compiler counts outstanding loads exactly.
    if (my_unit < 0 || my_unit >= g.n_units) {
      if (do_wait && !grid_wait(grid)) return false;
      stamp(p, ph, 1);
      if (ssq_in) compute_row_scales<MP>(p, ssq_in, r_s);
      return true;
    }
    constexpr int KMAX = 16 / AT;   // most k-tiles per wavefront and unit (the host checks)
    const gbf16x8* a_base = (const gbf16x8*)(g.w + (((int64_t)my_unit * kFusedWaves + wave) * KTW * AT) * 512 + lane * 8);
    bf16x8 a[KMAX][AT];
#pragma unroll
    for (int i = 0; i < KMAX; ++i)
      if (i < KTW) {
#pragma unroll
        for (int j = 0; j < AT; ++j) a[i][j] = __builtin_nontemporal_load(a_base + (i * AT + j) * 64);
      }
    if (do_wait && !grid_wait(grid)) return false;
    stamp(p, ph, 1);
    // Activation tiles.  Every workgroup reads the whole activation matrix of its k-range, and all of them the same
    // lines at the same time: this L2-to-CU traffic, not the weight stream, is what limits these phases, so rows
    // beyond M (the padding of the last 16-row tile) are not fetched at all.
    // (their lanes re-read row 0 of their k-group, a line that is fetched anyway; an unconditional load keeps the
    // compiler's count of outstanding loads exact, and those rows' results are never stored)
    int row_fix[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) row_fix[t] = t * 16 + (lane & 15) < p.M ? 0 : -(lane & 15);
    auto load_b = [&](bf16x8* dst, int c) {
      const gbf16x8* bp = b_first + (int64_t)c * MT * 64;
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) dst[t * NP + pl] = bp[pl * bplane_v + t * 64 + row_fix[t]];
    };
    // the activation tiles of KC chunks through a ring of DB (DB = KC: all requested at once), straight-line code with static
    // register indices
    auto run = [&](auto kc_tag) {
      constexpr int KC = decltype(kc_tag)::value;
      // (three row tiles of one plane: all at once, 48 rows over 8192 keys 7306 -> 7222 us per round; fewer rows gain nothing,
      // 24 rows over 1024 keys 4930 -> 4950, 8 rows over 211 keys 2940 -> 2939)
      constexpr int DB = KC < 4 || (MT == 3 && NP == 1) ? KC : 4;
      bf16x8 b[DB][MT * NP];
#pragma unroll
      for (int c = 0; c < (DB == KC ? DB : DB - 1); ++c) load_b(b[c], c);
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        if (DB < KC && c + DB - 1 < KC) load_b(b[(c + DB - 1) % DB], c + DB - 1);
#pragma unroll
        for (int j = 0; j < AT; ++j)
#pragma unroll
          for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int pl = 0; pl < NP; ++pl)
              acc[j][t] = mfma16_f16(a[c][j], b[c % DB][t * NP + pl], acc[j][t]);
      }
    };
    if (KTW == 2) run(std::integral_constant<int, 2>());
    else if (KTW == 4) run(std::integral_constant<int, 4>());
    else run(std::integral_constant<int, 8>());
    stamp(p, ph, 3);
    if (ssq_in) compute_row_scales<MP>(p, ssq_in, r_s);   // for the next phase (qkv -> attention)
    stamp(p, ph, 4);
    finish_unit(my_unit);
    stamp(p, ph, 5);
    return true;
  } else {
    // ---- any number of units per workgroup (the LM head): weights and activations travel together through a ring
    // of D register chunks
    const int n_my = (int)blockIdx.x < g.n_units ? (g.n_units - 1 - (int)blockIdx.x) / p.nwg + 1 : 0;
    const int n_chunks = n_my * KTW;
    Chunk<AT, MT, NP> ring[D];
    // chunk c = (unit blockIdx.x + n * grid, k-tile i of this wavefront); the load cursors advance one chunk at a time
    const gbf16x8* a_next = (const gbf16x8*)(g.w + (((int64_t)blockIdx.x * kFusedWaves + wave) * KTW * AT) * 512 + lane * 8);
    const int64_t a_unit_jump = ((int64_t)p.nwg * kFusedWaves - 1) * KTW * AT * 64;   // in 16-byte vectors, at a unit's end
    int a_i = 0;
    auto load_a = [&](Chunk<AT, MT, NP>& ck) {
#pragma unroll
      for (int j = 0; j < AT; ++j) ck.a[j] = __builtin_nontemporal_load(a_next + j * 64);
      a_next += AT * 64;
      if (++a_i == KTW) { a_i = 0; a_next += a_unit_jump; }
    };
    int b_i = 0;
    int row_fix[MT];   // rows beyond M (padding of the last row tile) are not fetched: their lanes re-read row 0
#pragma unroll
    for (int t = 0; t < MT; ++t) row_fix[t] = t * 16 + (lane & 15) < p.M ? 0 : -(lane & 15);
    auto load_b = [&](Chunk<AT, MT, NP>& ck) {
      const gbf16x8* bp = b_first + (int64_t)b_i * MT * 64;
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int pl = 0; pl < NP; ++pl) ck.b[t * NP + pl] = bp[pl * bplane_v + t * 64 + row_fix[t]];
      if (++b_i == KTW) b_i = 0;
    };
    auto mfma_chunk = [&](const Chunk<AT, MT, NP>& ck) {
#pragma unroll
      for (int j = 0; j < AT; ++j)
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int pl = 0; pl < NP; ++pl)
            acc[j][t] = mfma16_f16(ck.a[j], ck.b[t * NP + pl], acc[j][t]);
    };
    // weights of the first chunks go out before the barrier: they depend on nothing
    if (n_chunks > 0) {
#pragma unroll
      for (int s = 0; s < D - 1; ++s) load_a(ring[s]);
    }
    if (do_wait && !grid_wait(grid)) return false;
    stamp(p, ph, 1);
    if (n_chunks > 0) {
#pragma unroll
      for (int s = 0; s < D - 1; ++s) load_b(ring[s]);
    }
    if (ssq_in) compute_row_scales<MP>(p, ssq_in, r_s);
    stamp(p, ph, 3);
    // The host guarantees KTW % D == 0: a unit ends only at the end of a group of D chunks, and every load inside
    // the steady loop is unconditional (the compiler then counts outstanding loads exactly).
    const int n_outer = n_chunks / D;
    int c_i = 0, c_unit = blockIdx.x;
    for (int q = 0; q + 1 < n_outer; ++q) {
#pragma unroll
      for (int s = 0; s < D; ++s) {
        load_a(ring[(s + D - 1) % D]);
        load_b(ring[(s + D - 1) % D]);
        mfma_chunk(ring[s]);
      }
      c_i += D;
      if (c_i == KTW) {
        c_i = 0;
        finish_unit(c_unit);
        c_unit += p.nwg;
      }
    }
    if (n_outer > 0) {
      stamp(p, ph, 4);
      load_a(ring[D - 1]);
      load_b(ring[D - 1]);
#pragma unroll
      for (int s = 0; s < D; ++s) mfma_chunk(ring[s]);
      stamp(p, ph, 5);
      finish_unit(c_unit);
    }
    return true;
  }
}

// ---------------------------------------------------------------------------------------------- attention
// Reductions over the four 16-lane rows of a wavefront (lanes l, l^16, l^32, l^48 hold values of one query row)
__device__ __forceinline__ float max_over_rows(float x) { return lanes_max<16, 32>(x); }
__device__ __forceinline__ float sum_over_rows(float x) { return lanes_sum<16, 32>(x); }
struct OnlineSoftmax {
  float m_run, l_run;   // running maximum (base-2 exponent) and this lane's share of the running sum
  f32x4 acc[4];         // O^T: dims dt*16 + (lane>>4)*4 + r of query row lane & 15
};

// Online-softmax update with the block's masked scores sv (this lane's 8 keys) and their maximum mx.  The running
// accumulators are rescaled only when some row's maximum moved (a wavefront-uniform test): after the first blocks it
// rarely does.
template <int NPP>
__device__ __forceinline__ void softmax_update(OnlineSoftmax& st, const float sv[8], float mx, const bf16x8 vt[4]) {
  mx = max_over_rows(mx);
  const float m_new = fmaxf(st.m_run, mx);
  const float m_use = m_new == -INFINITY ? 0.f : m_new;
  if (__any(m_new != st.m_run)) {
    const float corr = exp2_fast(st.m_run - m_use);
    st.l_run *= corr;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) st.acc[dt] = st.acc[dt] * corr;
    st.m_run = m_new;
  }
  Bf8 ph, pl;
  float psum = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float pe = exp2_fast(sv[i] - m_use);
    psum += pe;
    ph.u[i] = to_bf16(pe);
    pl.u[i] = to_bf16(pe - bf16_to_f32(ph.u[i]));
  }
  st.l_run += psum;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) {
    st.acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[dt], ph.v, st.acc[dt], 0, 0, 0);
    if (NPP == 2) st.acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[dt], pl.v, st.acc[dt], 0, 0, 0);
  }
}


// One 32-key block: scores S[tile][r] of this lane's query row against keys (lane>>4)*8 + tile*4 + r of the block,
// `vis` = visibility of those 8 keys, vt[dt] = V^T operands of the block.
template <int NPP>
__device__ __forceinline__ void softmax_block(OnlineSoftmax& st, const f32x4 S[2], const bool vis[8], const bf16x8 vt[4]) {
  float sv[8];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float x = i < 4 ? S[0][i] : S[1][i - 4];
    sv[i] = vis[i] ? x : -INFINITY;
    mx = fmaxf(mx, sv[i]);
  }
  softmax_update<NPP>(st, sv, mx, vt);
}

template <int NPQ>
__device__ __forceinline__ f32x4 score_tile(bf16x8 k0, bf16x8 k1, const Bf8 qh[2], const Bf8 ql[2]) {
  f32x4 s = (f32x4){0.f, 0.f, 0.f, 0.f};
  s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qh[0].v, s, 0, 0, 0);
  s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qh[1].v, s, 0, 0, 0);
  if (NPQ == 2) {
    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, ql[0].v, s, 0, 0, 0);
    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, ql[1].v, s, 0, 0, 0);
  }
  return s;
}

// Attention unit = (sequence b, KV head hk, 16-row query tile qt, key split s).  A query tile holds 16 / G whole
// rows with all G query heads of the group.  The 8 wavefronts take the 32-key blocks of the unit round-robin:
// first the stored trunk keys of the split, then (split 0 only) the blocks of "fresh" keys: keys that exist only in
// this pass or only for one row.  Branch rows: fresh key f = (row of the tile f / SL, slot f % SL), the row's
// stored private suffix followed by its own token, visible to that row alone.  Extend rows: fresh key f = token f
// of this pass, visible to rows f and later.  All 512 threads stage the fresh K rows and V^T columns in LDS (and
// append the new K/V to the suffix or the trunk).  A dependent global load costs more than a microsecond here, so
// every load whose address is pure index arithmetic (row descriptors, the query tile, the first trunk blocks, the
// fresh-key sources) is issued up front; loop counts come from the host's bound on the visible trunk, the true
// visibility only masks.  The 8 partial softmaxes meet in LDS; with one split the result goes straight to the
// o-projection's operand planes, otherwise to the partial buffers that the last unit of the tile to arrive merges.
// SM: the unit that arrives last of a tile's key splits merges them (a kernel of its own for passes with several splits:
// compiled into the one-split kernel, the merge costs its linear layers 1 % through their register allocation).
template <int MT, int MP, int NPQ, int NPP, int NPT, bool PG, bool SM>
__device__ __forceinline__ bool attn_unit(const FusedParams& p, const FusedLayer& L, const float* qkv, int unit,
                                          const float* r_s, f32x4* lds, bf16_t* att_out, float* part_o, float* part_ml,
                                          unsigned* arrivals, int ph, Grid* wait_on, const unsigned* group_flags) {
  const ThreadIds ids = fresh_thread_ids();
  const int lane = ids.lane, wave = ids.wave;
  const int li = lane & 15, g4 = lane >> 4;
  const int hk = unit % p.Hkv;
  int rem = unit / p.Hkv;
  const int qt = rem % p.QT;
  rem /= p.QT;
  const int s = rem % p.NS, b = rem / p.NS;
  const int g_log = 31 - __builtin_clz(p.G), sl_log = p.SL == 8 ? 3 : 4;   // G and SL are powers of two
  const int RG = p.R << g_log;
  const int qr = qt * 16 + li;
  const bool vq = qr < RG;
  const int qrc = vq ? qr : RG - 1;
  const int rloc = qrc >> g_log;           // row of the sequence
  const int m = b * p.R + rloc;
  const int hq = hk * p.G + (qrc & (p.G - 1));
  const bool is_branch = p.is_branch != 0;
  const gfloat* gq = (const gfloat*)qkv;
  const gfloat* gcs = (const gfloat*)p.cos_sin;

  // ---- issue: the first trunk blocks of this wavefront (block counts from the host's bound)
  const int kb0 = s * p.KPU;
  const int kend_ub = min(kb0 + p.KPU, p.tv_ub);
  const int n_tb = kend_ub > kb0 ? (kend_ub - kb0 + 31) >> 5 : 0;
  const int n_mine = n_tb > wave ? (n_tb - wave + kFusedWaves - 1) / kFusedWaves : 0;
  const int rpt = 16 >> g_log;                                // rows per query tile
  const int n_fresh_keys = is_branch ? rpt << sl_log : p.R;
  const int n_fb = s == 0 ? (n_fresh_keys + 31) >> 5 : 0;
  const int krow = (li >> 2) * 8 + (li & 3);                  // key of this lane's A-operand row in a block (tile 0)
  // trunk K [B][Hkv][vt_stride][64]; trunk V^T [B][Hkv][vt_stride / 32][64 dims][32 keys]: a 32-key block of one head is
  // 4 KiB of contiguous memory in both, so every operand load covers whole cache lines
  // PG (paged trunk, App. B "PagedAttention"): block j of sequence b is page p.pages[b][j] of a pool shared by all
  // sequences, a page = the same 4 KiB per head and operand as a block of the contiguous layouts.  Lane i of a wavefront
  // fetches the page of the wavefront's i-th block up front (one load), so the block loop itself stays free of
  // dependent loads; entries behind a sequence's allocation name page 0, which exists and holds zeros.
  const int64_t head0 = PG ? 0 : ((int64_t)(b * p.Hkv + hk) * p.vt_stride) * 64;
  const gbf16* kbase = (const gbf16*)L.trunk_k + head0 + g4 * 8;
  const gbf16* vbase = (const gbf16*)L.trunk_vt + head0 + li * 32 + g4 * 8;
  int pgs = 0;
  if constexpr (PG) pgs = p.pages[(int64_t)b * p.page_stride + min((kb0 >> 5) + wave + kFusedWaves * lane, p.page_stride - 1)];
  struct TrunkBlock {
    bf16x8 k[2][2];
    bf16x8 vt[4];
  };
  // (3 or 4 blocks fit the registers but lose: 24 rows over 1024 keys 4941 -> 5183 or 5193 us per round, 48 rows over 8192 keys
  // 7310 -> 7559 or 7434: what a wavefront polls for returns behind its K/V loads, and a compute unit ingests no more of them)
  constexpr int RING = 2;
  TrunkBlock ring[RING];
  auto load_trunk = [&](TrunkBlock& tb, int i) {   // i-th block of this wavefront, clamped to its last one
    const int ic = max(min(i, n_mine - 1), 0);
    const int blk = wave + kFusedWaves * ic;
    const int kb = min(kb0 + blk * 32, p.vt_stride - 32);
    const int64_t bo = PG ? ((int64_t)__builtin_amdgcn_readlane(pgs, ic) * p.Hkv + hk) * 2048 : (int64_t)kb * 64;
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const gbf16* kp = kbase + bo + (krow + tile * 4) * 64;
      tb.k[tile][0] = *(const gbf16x8*)kp;
      tb.k[tile][1] = *(const gbf16x8*)(kp + 32);
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) tb.vt[dt] = *(const gbf16x8*)(vbase + bo + dt * 16 * 32);
  };
#pragma unroll
  for (int i = 0; i < RING; ++i) load_trunk(ring[i], i);   // unconditional (a wavefront without blocks re-reads block 0)
  // The stored keys do not depend on the phase before: the first unit of a workgroup requests its ring ahead of the
  // grid barrier.
  if (wait_on) {
    // the projections of this KV head's group (group_flags: one line of flags per group), or the whole grid
    if (!(group_flags ? group_wait(*wait_on, group_flags + hk * 16, p.qkv_ug) : grid_wait(*wait_on))) return false;
    stamp(p, ph, 1);
  }
  stamp(p, ph, 3);

  // ---- issue: row descriptor, raw query tile
  const RowDesc rd = p.rows[m];
  const gfloat* qp = gq + (int64_t)m * p.qkvd + hq * 64 + g4 * 8;
  const f32x4 qa0 = *(const gf32x4*)qp, qa1 = *(const gf32x4*)(qp + 4);
  const f32x4 qb0 = *(const gf32x4*)(qp + 32), qb1 = *(const gf32x4*)(qp + 36);
  const gfloat* qcs = gcs + ((int64_t)m * 32 + g4 * 8) * 2;
  const f32x4 qc0 = *(const gf32x4*)qcs, qc1 = *(const gf32x4*)(qcs + 4), qc2 = *(const gf32x4*)(qcs + 8), qc3 = *(const gf32x4*)(qcs + 12);

  // ---- issue: sources of the fresh key this thread stages (item = key f, rotary quad / 8-dim group q8)
  struct Fresh {
    int f, q8, m_o;
    bool valid, stored;
    u32x2 k_lo, k_hi;      // stored: 4 + 4 key elements
    bf16x8 v;              // stored: 8 value elements
    f32x4 a, bb, c0, c1, v0, v1;   // computed: raw projections and rotary table
  };
  int fresh_slot = 0;    // extend rows: trunk position the fresh key is appended at
  Fresh fr[1];
  const int nf8 = n_fb * 32 * 8;   // at most 512: one item per thread
#pragma unroll
  for (int t = 0; t < 1; ++t) {
    Fresh& x = fr[t];
    const int it = ids.tid + t * kFusedThreads;
    x.f = it >> 3;
    x.q8 = it & 7;
    x.valid = false;
    x.stored = false;
    x.m_o = b * p.R;
    if (it < nf8) {
      if (is_branch) {
        const int rt = qt * rpt + (x.f >> sl_log), j = x.f & (p.SL - 1);
        x.m_o = b * p.R + min(rt, p.R - 1);
        x.valid = rt < p.R && j < p.suffix_len;
        x.stored = j < p.suffix_len - 1;
      } else {
        x.m_o = b * p.R + min(x.f, p.R - 1);
        x.valid = x.f < p.R;
        fresh_slot = p.rows[x.m_o].kv_slot;
      }
      if (x.valid) {
        // both sources in one stretch of loads: a branch on `stored` makes the second wait for the first (the slots of a
        // row up to its own are inside its suffix)
        const gfloat* kp = gq + (int64_t)x.m_o * p.qkvd + p.qd + hk * 64 + x.q8 * 4;
        x.a = *(const gf32x4*)kp;
        x.bb = *(const gf32x4*)(kp + 32);
        const gfloat* cs = gcs + ((int64_t)x.m_o * 32 + x.q8 * 4) * 2;
        x.c0 = *(const gf32x4*)cs;
        x.c1 = *(const gf32x4*)(cs + 4);
        const gfloat* vp = gq + (int64_t)x.m_o * p.qkvd + p.qd + p.kvd + hk * 64 + x.q8 * 8;
        x.v0 = *(const gf32x4*)vp;
        x.v1 = *(const gf32x4*)(vp + 4);
        if (is_branch) {
          const int64_t row = (((int64_t)x.m_o * p.suffix_cap + (x.f & (p.SL - 1))) * p.Hkv + hk) * 64;
          x.k_lo = *(const gu32x2*)(L.suffix_k + row + x.q8 * 4);
          x.k_hi = *(const gu32x2*)(L.suffix_k + row + 32 + x.q8 * 4);
          x.v = *(const gbf16x8*)(L.suffix_v + row + x.q8 * 8);
        }
      }
    }
  }

  // ---- Q operand: dims g4*8..+7 (k-step 0) and 32+g4*8..+7 (k-step 1) of this lane's query row, rotated, scaled
  // stored trunk keys the row sees (an extend's descriptor counts the pass's own tokens, here fresh keys, up to itself; the
  // kind of the pass comes from the launch: a test of the descriptor would wait for it)
  const int tv = vq ? rd.vis - (is_branch ? 0 : 1 + rloc) : 0;
  Bf8 qh[2], ql[2];
  {
    float a[8] = {qa0[0], qa0[1], qa0[2], qa0[3], qa1[0], qa1[1], qa1[2], qa1[3]};
    float bb[8] = {qb0[0], qb0[1], qb0[2], qb0[3], qb1[0], qb1[1], qb1[2], qb1[3]};
    float cc[16] = {qc0[0], qc0[1], qc0[2], qc0[3], qc1[0], qc1[1], qc1[2], qc1[3],
                    qc2[0], qc2[1], qc2[2], qc2[3], qc3[0], qc3[1], qc3[2], qc3[3]};
    const float scale = r_s[m] * 0.125f * kLog2e;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float c = cc[2 * i], sn = cc[2 * i + 1];
      float x0 = (a[i] * c - bb[i] * sn) * scale, x1 = (bb[i] * c + a[i] * sn) * scale;
      qh[0].u[i] = to_bf16(x0);
      qh[1].u[i] = to_bf16(x1);
      ql[0].u[i] = to_bf16(x0 - bf16_to_f32(qh[0].u[i]));
      ql[1].u[i] = to_bf16(x1 - bf16_to_f32(qh[1].u[i]));
    }
  }
  stamp(p, ph, 4);

  // ---- stage the fresh keys in LDS: K rows [64][72] (row padding against bank conflicts), V^T columns [64][72]
  bf16_t* kf_s = (bf16_t*)(lds + kFusedWaves * 4 * 64 + 64);
  bf16_t* vf_s = kf_s + 64 * 72;
  if (n_fb > 0) {
#pragma unroll
    for (int t = 0; t < 1; ++t) {
      Fresh& x = fr[t];
      if (ids.tid + t * kFusedThreads < nf8) {
        u32x2 k_lo = (u32x2){0u, 0u}, k_hi = (u32x2){0u, 0u};
        Bf8 vv;
        vv.w = (u32x4){0u, 0u, 0u, 0u};
        if (x.valid && x.stored) {
          k_lo = x.k_lo;
          k_hi = x.k_hi;
          vv.v = x.v;
        } else if (x.valid) {
          const float rs = r_s[x.m_o];
          float cc[8] = {x.c0[0], x.c0[1], x.c0[2], x.c0[3], x.c1[0], x.c1[1], x.c1[2], x.c1[3]};
          bf16_t x0[4], x1[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float c = cc[2 * e], sn = cc[2 * e + 1];
            x0[e] = to_bf16((x.a[e] * c - x.bb[e] * sn) * rs);
            x1[e] = to_bf16((x.bb[e] * c + x.a[e] * sn) * rs);
          }
          uint64_t p0 = pack_bf16x4(x0[0], x0[1], x0[2], x0[3]), p1 = pack_bf16x4(x1[0], x1[1], x1[2], x1[3]);
          k_lo = (u32x2){(uint32_t)p0, (uint32_t)(p0 >> 32)};
          k_hi = (u32x2){(uint32_t)p1, (uint32_t)(p1 >> 32)};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vv.u[e] = to_bf16(x.v0[e] * rs);
            vv.u[4 + e] = to_bf16(x.v1[e] * rs);
          }
        }
        *(u32x2*)(kf_s + x.f * 72 + x.q8 * 4) = k_lo;
        *(u32x2*)(kf_s + x.f * 72 + 32 + x.q8 * 4) = k_hi;
#pragma unroll
        for (int e = 0; e < 8; ++e) vf_s[(x.q8 * 8 + e) * 72 + x.f] = vv.u[e];
      }
    }
    wg_barrier();
  }
  stamp(p, ph, 5);

  OnlineSoftmax st;
  st.m_run = -INFINITY;
  st.l_run = 0.f;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) st.acc[dt] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // ---- stored trunk keys: RING blocks in flight.  Steady groups compute and reload unconditionally, the last group
  // only computes (blocks past the wavefront's last one are clamped duplicates with every key masked), so the load
  // counting stays exact and nothing is fetched twice.
  auto trunk_block = [&](const TrunkBlock& tb, int i) {
    const int kb = kb0 + (wave + kFusedWaves * i) * 32;
    f32x4 S[2];
    bool vis[8];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) S[tile] = score_tile<NPQ>(tb.k[tile][0], tb.k[tile][1], qh, ql);
#pragma unroll
    for (int e = 0; e < 8; ++e) vis[e] = i < n_mine && kb + g4 * 8 + e < tv;
    softmax_block<NPP>(st, S, vis, tb.vt);
  };
  int i0 = 0;
  for (; i0 + RING < n_mine; i0 += RING) {
#pragma unroll
    for (int r = 0; r < RING; ++r) {
      trunk_block(ring[r], i0 + r);
      load_trunk(ring[r], i0 + r + RING);
    }
  }
  if (n_mine > 0) {
#pragma unroll
    for (int r = 0; r < RING; ++r) trunk_block(ring[r], i0 + r);
  }
  stamp(p, ph, 6);
  // ---- fresh blocks continue the round-robin after the trunk blocks
  for (int blk = n_tb + ((wave - n_tb) & (kFusedWaves - 1)); blk < n_tb + n_fb; blk += kFusedWaves) {
    const int f0 = (blk - n_tb) * 32;
    f32x4 S[2];
    bool vis[8];
    bf16x8 vt[4];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const bf16_t* kp = kf_s + (f0 + krow + tile * 4) * 72 + g4 * 8;
      S[tile] = score_tile<NPQ>(*(const bf16x8*)kp, *(const bf16x8*)(kp + 32), qh, ql);
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) vt[dt] = *(const bf16x8*)(vf_s + (dt * 16 + li) * 72 + f0 + g4 * 8);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int f = f0 + g4 * 8 + e;
      vis[e] = vq && (is_branch ? ((f >> sl_log) == (li >> g_log) && (f & (p.SL - 1)) < p.suffix_len) : f <= rloc);
    }
    softmax_block<NPP>(st, S, vis, vt);
  }
  st.l_run = sum_over_rows(st.l_run);
  stamp(p, ph, 7);

  // the o-projection's operand planes: dims 4 dq .. 4 dq + 3 of query row qrow of this unit's tile
  auto write_att = [&](int qrow, int dq, f32x4 x4) {
    const int mm = b * p.R + qrow / p.G;
    const int k = (hk * p.G + qrow % p.G) * 64 + dq * 4;
    bf16_t hi[4], lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      hi[i] = to_f16(x4[i]);
      lo[i] = to_f16(x4[i] - f16_to_f32(hi[i]));
    }
    const int64_t off = b_off<MT>(k, mm);
    st_u64(att_out + off, pack_bf16x4(hi[0], hi[1], hi[2], hi[3]));
    if (NPT == 2) st_u64(att_out + (int64_t)MP * p.qd + off, pack_bf16x4(lo[0], lo[1], lo[2], lo[3]));
  };
  const int tid = fresh_thread_ids().tid;
  // ---- the 8 wavefronts' partial softmaxes meet in LDS: acc [wave][dt][lane], (m, l) [wave][16]
  float* ml = (float*)(lds + kFusedWaves * 4 * 64);
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) lds[(wave * 4 + dt) * 64 + lane] = st.acc[dt];
  if (g4 == 0) {
    ml[(wave * 16 + li) * 2] = st.m_run;
    ml[(wave * 16 + li) * 2 + 1] = st.l_run;
  }
  wg_barrier();
  if (tid < 256) {
    const int q = tid & 15, dq = tid >> 4;       // query row of the tile, dims 4 dq .. 4 dq + 3
    float mmax = -INFINITY;
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) mmax = fmaxf(mmax, ml[(w * 16 + q) * 2]);
    const float m_use = mmax == -INFINITY ? 0.f : mmax;
    float lsum = 0.f;
    f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) {
      const float wgt = exp2_fast(ml[(w * 16 + q) * 2] - m_use);
      lsum += wgt * ml[(w * 16 + q) * 2 + 1];
      o += lds[(w * 4 + (dq >> 2)) * 64 + q + 16 * (dq & 3)] * wgt;
    }
    const int qrow = qt * 16 + q;
    if (qrow < RG) {
      if (p.NS == 1) {
        const float inv = 1.0f / lsum;
        write_att(qrow, dq, o * inv);
      } else {
        const int64_t pb = ((int64_t)(b * p.Hkv + hk) * p.NS + s) * (p.QT * 16) + qrow;
        if (dq == 0) st_u64(part_ml + pb * 2, pack_f32x2(mmax, lsum));
        st_f32x4(part_o + pb * 64 + dq * 4, o);
      }
    }
  }
  // ---- several key splits: this unit's arrival is counted once its partial softmax has left (write-through stores,
  // vmcnt 0); the count comes back while the fresh keys are appended below
  int* last_s = (int*)(vf_s + 64 * 72);
  if (SM && p.NS > 1) {
    __builtin_amdgcn_s_waitcnt(0);
    wg_barrier();
    if (tid == 0) {
      unsigned* cnt = arrivals + (b * p.Hkv + hk) * p.QT + qt;
      const unsigned old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int is_last = old + 1 == (unsigned)p.NS;
      if (is_last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next pass
      *last_s = is_last;
    }
  }
  // ---- append the keys and values computed in this pass for later passes, from their LDS copies: the row's private
  // suffix slot (branch) or its trunk position (extend).  Last, so that the stores are not in the way of any load.
  {
    const Fresh& x = fr[0];
    if (n_fb > 0 && tid < nf8 && x.valid && !x.stored) {
      const u32x2 k_lo = *(const u32x2*)(kf_s + x.f * 72 + x.q8 * 4), k_hi = *(const u32x2*)(kf_s + x.f * 72 + 32 + x.q8 * 4);
      Bf8 vv;
#pragma unroll
      for (int e = 0; e < 8; ++e) vv.u[e] = vf_s[(x.q8 * 8 + e) * 72 + x.f];
      if (is_branch) {
        const int64_t row = (((int64_t)x.m_o * p.suffix_cap + (p.suffix_len - 1)) * p.Hkv + hk) * 64;
        *(gu32x2*)(L.suffix_k + row + x.q8 * 4) = k_lo;
        *(gu32x2*)(L.suffix_k + row + 32 + x.q8 * 4) = k_hi;
        *(gbf16x8*)(L.suffix_v + row + x.q8 * 8) = vv.v;
      } else {
        const int64_t bb = PG ? ((int64_t)p.pages[(int64_t)b * p.page_stride + (fresh_slot >> 5)] * p.Hkv + hk) * 2048
                              : (int64_t)(b * p.Hkv + hk) * p.vt_stride * 64 + (int64_t)(fresh_slot >> 5) * 2048;
        const int64_t row = bb + (int64_t)(fresh_slot & 31) * 64;
        *(gu32x2*)(L.trunk_k + row + x.q8 * 4) = k_lo;
        *(gu32x2*)(L.trunk_k + row + 32 + x.q8 * 4) = k_hi;
        gbf16* vcol = (gbf16*)L.trunk_vt + bb + (x.q8 * 8) * 32 + (fresh_slot & 31);
#pragma unroll
        for (int e = 0; e < 8; ++e) vcol[e * 32] = vv.u[e];
      }
    }
  }
  // ---- the unit that arrived last of a tile's NS splits merges them, in split order whoever it is: no unit ever waits
  // for another, and the merge phase with its grid barrier is gone.  Its loads are agent-scope (coherent across the
  // XCDs); the other splits' stores were complete before their arrivals were counted.
  if (SM && p.NS > 1) {
    wg_barrier();
    if (*last_s != 0 && tid < 256) {
      const int q = tid & 15, dq = tid >> 4;
      const int qrow = qt * 16 + q;
      if (qrow < RG) {
        constexpr int kMaxSplits = kFusedMaxSplits;
        const int64_t pb0 = ((int64_t)(b * p.Hkv + hk) * p.NS) * (p.QT * 16) + qrow, pstep = p.QT * 16;
        uint64_t mlv[kMaxSplits];
#pragma unroll
        for (int t = 0; t < kMaxSplits; ++t)
          mlv[t] = __hip_atomic_load((const uint64_t*)(part_ml + (pb0 + (t < p.NS ? t : 0) * pstep) * 2), __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        float mmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < kMaxSplits; ++t) mmax = t < p.NS ? fmaxf(mmax, __uint_as_float((unsigned)mlv[t])) : mmax;
        const float m_use = mmax == -INFINITY ? 0.f : mmax;
        float lsum = 0.f;
        f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t0 = 0; t0 < kMaxSplits; t0 += 4) {
          if (t0 < p.NS) {
            f32x4 ov[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) ov[t] = ld_f32x4_coherent(part_o + (pb0 + (t0 + t < p.NS ? t0 + t : 0) * pstep) * 64 + dq * 4);
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (t0 + t < p.NS) {
                const float wgt = exp2_fast(__uint_as_float((unsigned)mlv[t0 + t]) - m_use);
                lsum += wgt * __uint_as_float((unsigned)(mlv[t0 + t] >> 32));
                o += ov[t] * wgt;
              }
          }
        }
        write_att(qrow, dq, o * (1.0f / lsum));
      }
    }
  }
  wg_barrier();
  return true;
}

// Merge unit (only when the trunk is split over several units): one wavefront per (row, query head), lane = head
// dimension, merges the NS partial softmaxes and writes the attention output planes.
template <int MP, int NPT>
__device__ __forceinline__ void attn_merge_unit(const FusedParams& p, int mt, int unit, const float* part_o, const float* part_ml,
                                                bf16_t* att_out) {
  const int d = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int pair = unit * kFusedWaves + wave;
  if (pair >= p.M * p.Hq) return;
  const int m = pair / p.Hq, hq = pair - m * p.Hq;
  const int hk = hq / p.G, gq = hq - hk * p.G;
  const int b = m / p.R;
  const int qrow = (m - b * p.R) * p.G + gq;
  const int64_t pb0 = ((int64_t)(b * p.Hkv + hk) * p.NS) * (p.QT * 16) + qrow;
  const gfloat* gml = (const gfloat*)part_ml;
  const gfloat* go = (const gfloat*)part_o;
  float mmax = -INFINITY;
  for (int s = 0; s < p.NS; ++s) mmax = fmaxf(mmax, gml[(pb0 + (int64_t)s * (p.QT * 16)) * 2]);
  const float m_use = mmax == -INFINITY ? 0.f : mmax;
  float lsum = 0.f, o = 0.f;
  for (int s = 0; s < p.NS; ++s) {
    const int64_t pb = pb0 + (int64_t)s * (p.QT * 16);
    const float wgt = exp2_fast(gml[pb * 2] - m_use);
    lsum += wgt * gml[pb * 2 + 1];
    o += wgt * go[pb * 64 + d];
  }
  const float x = o / lsum;
  const bf16_t hi = to_f16(x);
  const bf16_t lo = to_f16(x - f16_to_f32(hi));
  // lanes d, d+1, d+2, d+3 -> one 8-byte store per plane from lane d (d % 4 == 0)
  uint32_t w = (uint32_t)hi | ((uint32_t)lo << 16);
  uint32_t w1 = __shfl_down(w, 1), w2 = __shfl_down(w, 2), w3 = __shfl_down(w, 3);
  if ((d & 3) == 0) {
    const int k = hq * 64 + d;
    const int64_t off = b_off_of(mt, k, m);
    st_u64(att_out + off, pack_bf16x4((bf16_t)w, (bf16_t)w1, (bf16_t)w2, (bf16_t)w3));
    if (NPT == 2)
      st_u64(att_out + (int64_t)MP * p.qd + off,
             pack_bf16x4((bf16_t)(w >> 16), (bf16_t)(w1 >> 16), (bf16_t)(w2 >> 16), (bf16_t)(w3 >> 16)));
  }
}

// ---------------------------------------------------------------------------------------------- wide passes
// Passes of more than kFusedMaxRows rows (up to kFusedWideRows: the branch rows of a batch of sequences, App. C:
// B (K+1) F rows per step).  With hundreds of rows a linear layer is no longer a pure weight stream: every weight tile
// meets 24 row tiles, and what limits a compute unit is the rate at which it pulls operands from L2 (about 64 bytes
// per clock) and the latency of each pull, so the work of a layer is cut in two dimensions and every phase is a kernel
// of its own, shaped for its work (a wide step takes milliseconds: the dozens of launches cost little beside it).
//
// What bounds them, measured with 256 workgroups that only load: data in an XCD's L2 reach a compute unit at 110-125 GB/s,
// a stream from memory shared by 8 workgroups of one XCD at 86-104, but everything that misses the L2s together, from HBM
// and the memory-side cache alike, at 6-7.4 TB/s (24-29 GB/s per compute unit).  So a layer's cost is what crosses into the
// L2s: the weights once, and the activations once per XCD that needs them.
//
// Linear layers: wide_block_kernel, below, and wide_few_kernel for up to 48 rows.  The o- and down-projections have few features under a long reduction dimension: they are
// cut into up to 8 k-slices, XCD x working on slice x mod S, so that an XCD's L2 takes in only that slice of the activations and, among
// the XCDs of a slice, only its own features' weights.  Their fp32 partial sums go to memory, and wide_resid_kernel, a workgroup per
// row, adds them to the residual stream in slice order and leaves the row's 1/rms: the linear layers that follow load one number per
// row where they had to add up partial sums of squares.
constexpr int kWideThreads = 256, kWideWaves = 4;

// k-tiles of a layer's reduction dimension
__host__ __device__ __forceinline__ int wide_k_tiles(const FusedGemm& g) { return g.KS * kFusedWaves * g.KTW; }

struct WideEpi {
  float* out;          // QKV: [M][ld] projections, row scale applied; LOGITS: [M][ld] logits; PART: [slice][M][ld] partial sums
  int64_t ld;
  bf16_t* act_out;     // SWIGLU
  int S;               // k-slices (PART; 1 otherwise)
  int ph;              // phase id (for the optional clocks)
};

// Memory to LDS without a register in between: 64 lanes x 16 (4) bytes, lane i at the wavefront's LDS address + 16 i (4 i).
__device__ __forceinline__ void dma16(const bf16_t* src, uint32_t lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)(uintptr_t)lds, 16, 0, 0);
}
__device__ __forceinline__ void dma4(const float* src, uint32_t lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)(uintptr_t)lds, 4, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// The linear layers of a wide pass.  A workgroup computes a block of FT feature tiles x RT row tiles (16 each) over the whole reduction
// dimension (PART: over one of S slices of it); WN x WM wavefronts hold FT / WN x RT / WM tiles of it each.  Both operands go from memory
// to LDS without passing registers, a k-tile (FT + RT KiB) to a buffer (G of them, one for each of G groups of wavefronts, where steps are
// short), NB buffers in flight; in memory a tile already has the lane order of
// the MFMA, so a tile is one load, its LDS image the same 1 KiB, and reading it back free of bank conflicts.  A step is one k-tile: wait
// until the next one has landed, barrier, then the MFMAs of this one with the LDS reads of the next and the loads for the buffer that
// has just become free between them (sched_barrier: a burst of memory operations would hold up the MFMAs behind it).
// What bounds it, by count and counters (1B shape): with many rows the LDS beside the MFMAs.  A step of gate/up takes about 910 clocks at 384
// rows, in which the LDS moves 84 KiB in 672 and the matrix pipes work 384, and 1950 at 1020 rows (128 KiB in 1024, 1024; the clock falls to 2.15
// GHz), so operands are moved as few times as possible: large blocks, and 16x16x32 MFMAs, which draw a tenth less power for the same work.
// With few rows the weight stream and the steps' latency (0.2 us each).  us of a launch at 2048 inputs, 16384 gate/up features, one machine,
// against the kernels it replaces (64 features with the reduction dimension over the wavefronts, as wide_few_kernel still does, and 256
// features x 96 or 128 rows with the weights in registers): 96 rows 18.0 and 21.8 + 2.4 (gap), 192 rows 22.9 and 27 + 2.4, 384 rows 31.3 and
// 35.1, 1020 rows 61 and 77.  2048 features, 8192 inputs in slices: 96 rows 11.9 and 13.1, 384 rows 22.5 and 28.0.
// Past its last block a workgroup goes on loading the last k-tile (the waits count loads), and it leaves when everything has landed.
template <int ATW, int EPI, int FT, int RT, int WN, int G, int NB, int TH>
__global__ __launch_bounds__(TH) void wide_block_kernel(FusedParams p, FusedGemm g, const bf16_t* bsrc, WideEpi e) {
  constexpr int W = TH / 64, WG = W / G, WM = WG / WN, FTW = FT / WN, RTW = RT / WM;
  constexpr int NTILE = G * (FT + RT), STAGE = NTILE * 64;   // tiles and 16-byte vectors of a buffer
  constexpr int LPW = (NTILE + W - 1) / W;                   // loads of a wavefront per step (the last tile again where they do not divide)
  constexpr int NM = FTW * RTW, NF = FTW + RTW, NO = NF + LPW;
  static_assert(W % G == 0 && WG % WN == 0 && FT % WN == 0 && RT % WM == 0 && FT % ATW == 0 && NB >= 3 && (NB - 1) * LPW < 64, "block shape");
  static_assert(EPI != FE_SWIGLU || FTW == 2 || FTW % 4 == 0, "a wavefront holds gate tiles together with their up tiles");
  extern __shared__ f32x4 lds[];                             // [NB][NTILE][64], the rows' 1/rms, then (G > 1) partial tiles
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave / WG, wn = wave % WG % WN, wm = wave % WG / WN;
  const int NKT = wide_k_tiles(g);
  const int S = EPI == FE_PART ? e.S : 1, steps = NKT / (S * G);   // (even: host check)
  const int n_groups = g.n_units / g.KS;                     // units of ATW feature tiles
  const int n_sets = (n_groups * ATW + FT - 1) / FT;
  const int n_rg = (((p.M + 15) >> 4) + RT - 1) / RT;
  // XCD x = blockIdx.x % 8 works on slice x % S and, among the XCDs of that slice, on the sets q = y, y + ys, ..; its workgroups take
  // (set, row group) pairs t = wx, wx + per_xcd, .. with the row group running fastest
  const int x = (int)blockIdx.x & 7, wx = (int)blockIdx.x >> 3, per_xcd = (int)gridDim.x >> 3;
  const int slice = x % S, y = x / S, ys = 8 / S;            // S is 1, 2, 4 or 8
  const int nqy = y < n_sets ? (n_sets - y + ys - 1) / ys : 0;
  const int ty = nqy * n_rg;
  const int n_my = wx < ty ? (ty - wx + per_xcd - 1) / per_xcd : 0;
  stamp(p, e.ph, 0);
  if (n_my == 0) return;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  float* r_s = (float*)(lds + NB * STAGE);
  if (EPI != FE_PART) {
    for (int r = wave * 64; r < p.M; r += TH) dma4(p.ssq + min(r + lane, p.M - 1), lds0 + NB * STAGE * 16 + r * 4);
  }
  // feature tile of the block that is this wavefront's f-th: whole units, or (two tiles a wavefront) a gate tile and its up tile
  auto tile_of = [&](int f) { return EPI == FE_SWIGLU && FTW == 2 ? (wn >> 1) * 4 + (wn & 1) + 2 * f : wn * FTW + f; };
  auto pair_of = [&](int n, int& set, int& rg) {
    const int t = wx + min(n, n_my - 1) * per_xcd, qh = t / n_rg;
    set = qh * ys + y;
    rg = t - qh * n_rg;
  };
  // the loads: step ld_k of pair ld_n to buffer ld_buf
  int ld_n = 0, ld_k = 0, ld_buf = 0;
  const bf16_t* src[LPW];
  int step_a = G * ATW * 512, step_b = G * p.row_tiles * 512;
  auto place = [&]() {
    int set, rg;
    pair_of(ld_n, set, rg);
    const bool past = ld_n >= n_my;
    const int kt0 = (slice * steps + (past ? steps - 1 : 0)) * G;
    if (past) step_a = step_b = 0;
#pragma unroll
    for (int n = 0; n < LPW; ++n) {
      // (units behind the last and row tiles behind the last row: the last one again, computed and not stored)
      const int i = min(wave * LPW + n, NTILE - 1), kt = kt0 + i / (FT + RT), t = i % (FT + RT);
      src[n] = t < FT ? g.w + (((int64_t)min(set * (FT / ATW) + t / ATW, n_groups - 1) * NKT + kt) * ATW + t % ATW) * 512
                      : bsrc + ((int64_t)kt * p.row_tiles + min(rg * RT + t - FT, (p.M - 1) >> 4)) * 512;
    }
  };
  auto load = [&](int n) {
    const int i = min(wave * LPW + n, NTILE - 1);
    dma16(src[n] + lane * 8, lds0 + (ld_buf * STAGE + i * 64) * 16);
    src[n] += i % (FT + RT) < FT ? step_a : step_b;
  };
  auto next_load = [&]() {
    ld_buf = ld_buf + 1 == NB ? 0 : ld_buf + 1;
    if (++ld_k == steps) {
      ld_k = 0;
      ++ld_n;
      place();
    }
  };
  place();
  for (int s = 0; s < NB; ++s) {
#pragma unroll
    for (int n = 0; n < LPW; ++n) load(n);
    next_load();
  }
  stamp(p, e.ph, 3);
  bf16x8 a[2][FTW], b[2][RTW];
  f32x4 acc[FTW][RTW];
#pragma unroll
  for (int f = 0; f < FTW; ++f)
#pragma unroll
    for (int t = 0; t < RTW; ++t) acc[f][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  auto fragment = [&](int i, int to, const bf16x8* buf) {
    if (i < RTW) b[to][i] = buf[(FT + wm * RTW + i) * 64];
    else a[to][i - RTW] = buf[tile_of(i - RTW) * 64];
  };
  // loads return in order: the first buffer has landed when only those of the others are outstanding
  wait_loads<(NB - 1) * LPW>();
  wg_barrier();
#pragma unroll
  for (int i = 0; i < NF; ++i) fragment(i, 0, (const bf16x8*)lds + grp * (FT + RT) * 64 + lane);
  int rd = 0;
  for (int n = 0; n < n_my; ++n) {
    for (int k = 0; k < steps; k += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        // the next k-tile has landed here, behind the barrier everywhere; and everyone has read this one's buffer
        wait_loads<(NB - 2) * LPW>();
        wg_barrier();
        rd = rd + 1 == NB ? 0 : rd + 1;
        const bf16x8* buf = (const bf16x8*)lds + rd * STAGE + grp * (FT + RT) * 64 + lane;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const int f = i / RTW, t = i % RTW;
          acc[f][t] = mfma16_f16(a[u][f], b[u][t], acc[f][t]);
#pragma unroll
          for (int o = i * NO / NM; o < (i + 1) * NO / NM; ++o) {
            if (o < NF) fragment(o, u ^ 1, buf);
            else load(o - NF);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        next_load();
      }
    }
    if (n == 0) stamp(p, e.ph, 4);
    if constexpr (G > 1) {                                   // the groups' partial tiles meet in LDS: group 0 adds them in order
      f32x4* red = lds + NB * STAGE + kFusedPromptRows / 4;
      if (grp > 0) {
#pragma unroll
        for (int i = 0; i < NM; ++i) red[((wave - WG) * NM + i) * 64 + lane] = acc[i / RTW][i % RTW];
      }
      wg_barrier();
      if (grp == 0) {
#pragma unroll
        for (int o = 1; o < G; ++o)
#pragma unroll
          for (int i = 0; i < NM; ++i) acc[i / RTW][i % RTW] += red[(((o - 1) * WG + wave) * NM + i) * 64 + lane];
      }
      if (n + 1 < n_my) wg_barrier();
    }
    // ---- epilogue from the accumulators: tile (f, t) holds features 4 (lane >> 4) .. + 3 of row lane & 15
    int set, rg;
    pair_of(n, set, rg);
    const int f4 = (lane >> 4) * 4;
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
      const int m = (rg * RT + wm * RTW + t) * 16 + (lane & 15);
      if (m < p.M && grp == 0) {
        const float rs = EPI == FE_PART ? 1.0f : r_s[m];
        if constexpr (EPI == FE_SWIGLU) {
#pragma unroll
          for (int i = 0; i < FTW / 2; ++i) {
            const int f = FTW == 2 ? 0 : (i >> 1) * 4 + (i & 1), tile = set * FT + tile_of(f);   // gate; its up tile is two further in the unit
            if (tile / 4 >= n_groups) continue;
            bf16_t hi[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float gg = acc[f][t][c] * rs, uu = acc[FTW == 2 ? 1 : f + 2][t][c] * rs;
              hi[c] = to_f16(gg / (1.0f + __expf(-gg)) * uu);
            }
            // input index of the down-projection
            *(uint64_t*)(e.act_out + b_off_of(p.row_tiles, (tile / 4) * 32 + (tile & 1) * 16 + f4, m)) = pack_bf16x4(hi[0], hi[1], hi[2], hi[3]);
          }
        } else {
          float* out = e.out + ((int64_t)slice * p.M + m) * e.ld;
#pragma unroll
          for (int f = 0; f < FTW; ++f) {
            const int tile = set * FT + tile_of(f);
            if (tile < g.NT) *(gf32x4*)((gfloat*)out + tile * 16 + f4) = EPI == FE_PART ? acc[f][t] : acc[f][t] * rs;
          }
        }
      }
#pragma unroll
      for (int f = 0; f < FTW; ++f) acc[f][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    if (n == 0) stamp(p, e.ph, 5);
  }
  wait_loads<0>();
  stamp(p, e.ph, 2);
}

// The linear layers of the narrowest wide passes: few rows over a short reduction dimension, where the k-tiles of wide_block_kernel's
// steps (0.2 us each) and its two trips to memory outlast the work.  A workgroup takes 4 feature tiles x a group of MTG row tiles over one of
// S slices; its four wavefronts, one per SIMD, split the slice, stream their weight tiles and the matching activation tiles into a ring of D
// register chunks, D - 1 of them in flight, and meet once, in LDS, where the partial tiles are added in wavefront order.  MTG = 2: 32x32x16
// MFMAs on operands kept in 16x16x32 tile order, see wide_tile_kernel.
// Graphs of 16 layers of width 512, us, against the blocks alone and the kernels before them: 20 rows 509, 576, 508; 48 rows 560, 592, 564.
template <int ATW, int EPI, int D, int MTG>
__global__ __launch_bounds__(kWideThreads) void wide_few_kernel(FusedParams p, FusedGemm g, const bf16_t* bsrc, WideEpi e) {
  constexpr int MTOT = kFusedWideRows / 16, NT = 4 * MTG;  // 1 KiB blocks of a wavefront's partial tiles
  constexpr bool BIG = MTG == 2;
  extern __shared__ f32x4 red[];
  __shared__ float r_s[kFewRows];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NKT = wide_k_tiles(g);
  const int S = EPI == FE_PART ? e.S : 1;
  const int NCH = NKT / (kWideWaves * S);           // k-tiles of this wavefront per pair (a multiple of D: host check)
  const int n_groups = g.n_units / g.KS;
  const int nq = ATW == 4 ? n_groups : n_groups >> 1;
  const int n_rg = (((p.M + 15) >> 4) + MTG - 1) / MTG;
  // the pairs of this workgroup: as in wide_block_kernel
  const int x = (int)blockIdx.x & 7, wx = (int)blockIdx.x >> 3, per_xcd = (int)gridDim.x >> 3;
  const int slice = x % S, y = x / S, ys = 8 / S;
  const int nqy = y < nq ? (nq - y + ys - 1) / ys : 0;
  const int ty = nqy * n_rg;
  const int n_my = wx < ty ? (ty - wx + per_xcd - 1) / per_xcd : 0;
  stamp(p, e.ph, 0);
  if (n_my == 0) return;

  // operand vector of this lane in a tile (BIG: in two neighbouring tiles, k-half 0; k-half 1 is 32 vectors further)
  const int lsrc = BIG ? ((lane >> 4) & 1) * 64 + (lane & 15) + ((lane >> 5) << 4) : lane;
  const int64_t a_group2 = (int64_t)NKT * 2 * 512;  // ATW == 2: from the set's first tile group to its second
  const int kt0 = (slice * kWideWaves + wave) * NCH;
  // the load cursor walks the chunks of this wavefront, pair after pair (behind the last: the last one again)
  const bf16_t *src_a = nullptr, *src_b = nullptr;
  int ld_i = 0, ld_n = 0;
  auto place = [&]() {
    const int t = wx + min(ld_n, n_my - 1) * per_xcd, qh = t / n_rg;
    const int q = qh * ys + y, rg = t - qh * n_rg;
    src_a = g.w + ((int64_t)(ATW == 4 ? q : 2 * q) * NKT + kt0) * ATW * 512;
    src_b = bsrc + ((int64_t)kt0 * MTOT + rg * MTG) * 512;
  };
  struct Chunk { bf16x8 a[4], b[MTG]; };
  auto load = [&](Chunk& ck, int l) {
    const gbf16x8* ap = (const gbf16x8*)(ATW == 4 || l < 2 ? src_a : src_a + a_group2) + lsrc;
    const gbf16x8* bp = (const gbf16x8*)src_b + lsrc;
    // BIG: a[2 f + h] features 32 f .. 32 f + 31 of the set, k-half h; b[h] k-half h
    if (l < 4) ck.a[l] = ap[(ATW == 4 ? (l >> 1) * 128 : 0) + (l & 1) * (BIG ? 32 : 64)];
    else ck.b[l - 4] = bp[(l - 4) * (BIG ? 32 : 64)];
  };
  auto advance = [&]() {
    src_a += ATW * 512;
    src_b += MTOT * 512;
    if (++ld_i == NCH) {
      ld_i = 0;
      ++ld_n;
      place();
    }
  };
  f32x16 accb[2];
  f32x4 acc[4][MTG];
  auto zero_acc = [&]() {
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int i = 0; i < 16; ++i) accb[f][i] = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < MTG; ++t) acc[j][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
  };
  zero_acc();
  // the rows' 1/rms: requested first, in LDS under the ring's loads, read behind the barrier
  float rs = 0.f;
  if (EPI != FE_PART) rs = ((const gfloat*)p.ssq)[min((int)threadIdx.x, p.M - 1)];
  Chunk ring[D];
  place();
#pragma unroll
  for (int s = 0; s < D - 1; ++s) {
#pragma unroll
    for (int l = 0; l < 4 + MTG; ++l) load(ring[s], l);
    advance();
  }
  if (EPI != FE_PART && threadIdx.x < kFewRows) r_s[threadIdx.x] = rs;
  stamp(p, e.ph, 3);
  // a chunk's loads between the MFMAs of the one before (a burst of them would hold the wavefront up)
  constexpr int NM = BIG ? 4 : 4 * MTG, NL = 4 + MTG;
  auto turn = [&](const Chunk& ck, Chunk& to) {
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      if constexpr (BIG) accb[i & 1] = mfma32_f16(ck.a[2 * (i & 1) + (i >> 1)], ck.b[i >> 1], accb[i & 1]);
      else acc[i / MTG][i % MTG] = mfma16_f16(ck.a[i / MTG], ck.b[i % MTG], acc[i / MTG][i % MTG]);
#pragma unroll
      for (int l = i * NL / NM; l < (i + 1) * NL / NM; ++l) load(to, l);
      __builtin_amdgcn_sched_barrier(0);
    }
    advance();
  };
  for (int n = 0; n < n_my; ++n) {
    const int t = wx + n * per_xcd;
    const int q = (t / n_rg) * ys + y, rg = t - (t / n_rg) * n_rg;
    for (int c = 0; c < NCH; c += D) {
#pragma unroll
      for (int s = 0; s < D; ++s) turn(ring[s], ring[(s + D - 1) % D]);
    }
    if (n == 0) stamp(p, e.ph, 4);
    // ---- the four wavefronts' partial tiles meet; every wavefront sums its share of the blocks and runs their epilogue.  Block idx: BIG
    // (f, c) = registers 4 c .. 4 c + 3 of accb[f]: features 32 f + 8 c + 4 (lane >> 5) .. + 3, row lane & 31; else (j, t): features 16 j + 4
    // (lane >> 4) .. + 3, row 16 t + (lane & 15)
    if constexpr (BIG) {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const f32x16& v = accb[i >> 2];
        const int c = (i & 3) * 4;
        red[(wave * NT + i) * 64 + lane] = (f32x4){v[c], v[c + 1], v[c + 2], v[c + 3]};
      }
    } else {
#pragma unroll
      for (int i = 0; i < NT; ++i) red[(wave * NT + i) * 64 + lane] = acc[i / MTG][i % MTG];
    }
    wg_barrier();
    auto total = [&](int idx) {
      f32x4 v = red[idx * 64 + lane];
#pragma unroll
      for (int w = 1; w < kWideWaves; ++w) v += red[(w * NT + idx) * 64 + lane];
      return v;
    };
    auto feature_of = [&](int idx) { return BIG ? (idx >> 2) * 32 + (idx & 3) * 8 + (lane >> 5) * 4 : (idx / MTG) * 16 + (lane >> 4) * 4; };
    auto row_of = [&](int idx) { return rg * MTG * 16 + (BIG ? lane & 31 : (idx % MTG) * 16 + (lane & 15)); };
    if constexpr (EPI == FE_SWIGLU) {
      // features 0..31 of the set are gate, 32..63 the matching up features: blocks idx and idx + NT / 2
      for (int idx = wave; idx < NT / 2; idx += kWideWaves) {
        const f32x4 gv = total(idx), uv = total(idx + NT / 2);
        const int m = row_of(idx);
        if (m < p.M) {
          const float rs = r_s[m];
          bf16_t hi[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float gg = gv[i] * rs, uu = uv[i] * rs;
            hi[i] = to_f16(gg / (1.0f + __expf(-gg)) * uu);
          }
          // input index of the down-projection
          *(uint64_t*)(e.act_out + b_off<MTOT>(q * 32 + feature_of(idx), m)) = pack_bf16x4(hi[0], hi[1], hi[2], hi[3]);
        }
      }
    } else {
      float* out = e.out + (int64_t)slice * p.M * e.ld;
      for (int idx = wave; idx < NT; idx += kWideWaves) {
        const f32x4 v = total(idx);
        const int m = row_of(idx), n0 = q * 64 + feature_of(idx);
        if ((n0 >> 4) < g.NT && m < p.M) *(gf32x4*)((gfloat*)out + (int64_t)m * e.ld + n0) = EPI == FE_PART ? v : v * r_s[m];
      }
    }
    wg_barrier();
    zero_acc();
    if (n == 0) stamp(p, e.ph, 5);
  }
  stamp(p, e.ph, 2);
}

// The residual stream of a wide pass: a workgroup per row.  EMBED: h = the token's embedding; otherwise h += the row's partial sums of
// the linear layer before, slice after slice.  Then (h * gain) as the fp16 B operand of the next linear layer (8 consecutive
// features per thread are one lane's 16 bytes of it), the row's 1/rms, which that layer's epilogue multiplies in, and, where
// asked for, the normalised row as fp32 hidden states.  Reads S + 1 rows of d floats: at 96 rows of the 1B shape (S = 4 and 8)
// 4.9 us, at 384 (S = 2) 5.3, at 1020 10.3, of which launch and two memory round trips are about 4.
// PIECES: rows go to the XCDs in pieces of 8 (wide_rows.h) instead of singly; see launch_wide_resid.
// CLOCKS: with phase clocks (an instance of its own: the test of p.prof alone cost a wide round 1 %).
template <bool EMBED, bool PIECES, bool CLOCKS>
__global__ __launch_bounds__(kWideThreads) void wide_resid_kernel(FusedParams p, const float* part, int S, const bf16_t* gain,
                                                                  float* hidden, int ph) {
  constexpr int kHeld = 2;                       // 8-feature chunks per thread kept in registers (d <= 4096); others are re-read
  __shared__ float sum_s[kWideWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m = PIECES ? (int)wide_resid_row(blockIdx.x) : (int)blockIdx.x;
  if (PIECES) {
    // What the row's first loads need comes in one batch of scalar loads with the number of rows; left to itself the compiler loads
    // that alone, waits, and asks for the rest behind the branch.
    if (EMBED) asm volatile("" ::"s"(p.M), "s"(p.d), "s"(p.V), "s"(p.tokens), "s"(p.embed), "s"(gain));
    else asm volatile("" ::"s"(p.M), "s"(p.d), "s"(p.h), "s"(part), "s"(S), "s"(gain));
    if (m >= p.M) return;
  }
  if (CLOCKS) stamp(p, ph, EMBED ? 0 : 6, m);       // (the phase's other slots are the linear layer's)
  gfloat* h = (gfloat*)p.h + (int64_t)m * p.d;
  int tok = 0;
  if (EMBED) {
    tok = p.tokens[m];
    tok = tok < 0 ? 0 : (tok >= p.V ? p.V - 1 : tok);
  }
  f32x4 held[kHeld][2];
  u32x4 gheld[kHeld];
  float ss = 0.f;
  auto chunk = [&](int c, f32x4 v[2]) {
    if (EMBED) {
      Bf8 eb;
      eb.v = *(const gbf16x8*)((const gbf16*)p.embed + (int64_t)tok * p.d + c);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i >> 2][i & 3] = bf16_to_f32(eb.u[i]);
    } else {
      const gfloat* pp = (const gfloat*)part + (int64_t)m * p.d + c;
      v[0] = *(const gf32x4*)(h + c);
      v[1] = *(const gf32x4*)(h + c + 4);
      for (int s0 = 0; s0 < S; s0 += 4) {
        f32x4 pv[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const gfloat* q = pp + (int64_t)min(s0 + i, S - 1) * p.M * p.d;
          pv[i][0] = *(const gf32x4*)q;
          pv[i][1] = *(const gf32x4*)(q + 4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (s0 + i < S) { v[0] += pv[i][0]; v[1] += pv[i][1]; }
      }
    }
    *(gf32x4*)(h + c) = v[0];
    *(gf32x4*)(h + c + 4) = v[1];
#pragma unroll
    for (int i = 0; i < 8; ++i) ss += v[i >> 2][i & 3] * v[i >> 2][i & 3];
  };
  const int step = kWideThreads * 8;
#pragma unroll
  for (int i = 0; i < kHeld; ++i) {
    const int c = (int)threadIdx.x * 8 + i * step;
    if (c < p.d) {
      gheld[i] = *(const u32x4*)(gain + c);
      chunk(c, held[i]);
    }
  }
  for (int c = (int)threadIdx.x * 8 + kHeld * step; c < p.d; c += step) {
    f32x4 v[2];
    chunk(c, v);
  }
  ss = lanes_sum(ss);
  if (lane == 0) sum_s[wave] = ss;
  __syncthreads();
  const float rs = 1.0f / sqrtf(((sum_s[0] + sum_s[1]) + (sum_s[2] + sum_s[3])) / (float)p.d + p.eps);
  if (threadIdx.x == 0) ((gfloat*)p.ssq)[m] = rs;
  auto put = [&](int c, const f32x4 v[2], u32x4 gw) {
    Bf8 gb, x;
    gb.w = gw;
    f32x4 n[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float xg = v[i >> 2][i & 3] * bf16_to_f32(gb.u[i]);
      x.u[i] = to_f16(xg);
      n[i >> 2][i & 3] = xg * rs;
    }
    *(gbf16x8*)((gbf16*)p.xn + b_off_of(p.row_tiles, c, m)) = x.v;
    if (hidden) {
      *(gf32x4*)((gfloat*)hidden + (int64_t)m * p.hidden_ld + c) = n[0];
      *(gf32x4*)((gfloat*)hidden + (int64_t)m * p.hidden_ld + c + 4) = n[1];
    }
  };
#pragma unroll
  for (int i = 0; i < kHeld; ++i) {
    const int c = (int)threadIdx.x * 8 + i * step;
    if (c < p.d) put(c, held[i], gheld[i]);
  }
  for (int c = (int)threadIdx.x * 8 + kHeld * step; c < p.d; c += step) {
    f32x4 v[2] = {*(const gf32x4*)(h + c), *(const gf32x4*)(h + c + 4)};   // this thread's own stores
    put(c, v, *(const u32x4*)(gain + c));
  }
  if (CLOCKS) stamp(p, ph, EMBED ? 2 : 7, m);
}

// The LM head of up to 96 rows: a stream of weights, each read once.  A workgroup = 4 wavefronts x 64 features x 96 rows over the whole
// reduction dimension.  The weights of a wavefront's own features go straight into registers (a ring of 8 k-tiles, non-temporal); the
// activations, which all four need, through LDS (stages of 4 k-tiles, double buffered, requested two stages ahead); nothing has to be
// reduced across wavefronts.  Every LDS read, load and LDS write sits between two MFMAs (sched_barrier): a burst of them blocks the one
// wavefront of a SIMD until the memory pipeline has taken it in, and left to itself the scheduler sinks the loads to just before their
// use.  The MFMAs are 32x32x16.  Both operands stay in their 16x16x32 tile order in memory and LDS: a 32x32x16 operand is the k-half h of
// two neighbouring tiles, and lane l takes its 16 bytes from lane (l & 15) + 16 (l >> 5) + 32 h of tile (l >> 4) & 1, a fixed offset per
// lane.  96 rows of the 1B shape 107 to 110 us, 525 MB of weights and 49 MB of logits (stages of 8 k-tiles with the memory operations in
// bursts 109; wide_block_kernel 117).
constexpr int kTileRows = 96;
constexpr int kTileStage = 4, kTileRing = 8;         // k-tiles of an LDS stage, of the weight ring
__global__ __launch_bounds__(kWideThreads) void wide_tile_kernel(FusedParams p, FusedGemm g, const bf16_t* bsrc, WideEpi e) {
  constexpr int KC = kTileStage, RT = kTileRows / 16, R32 = RT / 2, NF = 2, ATW = 4;   // (64 features of a wavefront: one unit)
  constexpr int STAGE = KC * RT * 64, BL = STAGE / kWideThreads, NM = NF * R32;
  static_assert(kTileRing == 2 * KC && 2 * ((BL + KC - 1) / KC) <= NM && NF + 1 < NM, "a turn of the ring is two stages; memory operations between MFMAs");
  extern __shared__ f32x4 lds[];                     // [2][KC][RT][64] B-operand vectors
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int NKT = wide_k_tiles(g);
  const int NST = NKT / KC;                          // stages per set (even: host check)
  const int n_groups = g.n_units;                    // units of ATW feature tiles
  const int n_sets = (n_groups + 3) / 4;
  const int n_my = (int)blockIdx.x < n_sets ? (n_sets - 1 - (int)blockIdx.x) / (int)gridDim.x + 1 : 0;
  stamp(p, e.ph, 0);
  if (n_my == 0) return;

  const int lpos = (lane & 15) + ((lane >> 5) << 4), ltile = (lane >> 4) & 1;
  const int lsrc = ltile * 64 + lpos;                // operand vector of this lane in two neighbouring tiles, k-half 0
  constexpr int fstep = 128;                         // vectors from a wavefront's first 32 features to its second
  f32x16 acc[NF][R32];
  auto zero_acc = [&]() {
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int t = 0; t < R32; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[f][t][i] = 0.f;
  };
  zero_acc();
  // this wavefront's unit of the workgroup's n-th set (past the last: the last unit again, computed and never stored)
  auto unit_of = [&](int n) { return min(((int)blockIdx.x + min(n, n_my - 1) * (int)gridDim.x) * 4 + wave, n_groups - 1); };
  int b_rel[BL];
#pragma unroll
  for (int i = 0; i < BL; ++i) {
    const int v = (int)threadIdx.x + kWideThreads * i;
    const int kt = v / (RT * 64);
    b_rel[i] = (kt * p.row_tiles * 64 + v - kt * (RT * 64)) * 8;
  }
  struct Cursor { int n, s; const bf16_t* q; };      // set ordinal, stage; operand address of that stage
  auto place_a = [&](Cursor& c) { c.q = g.w + ((int64_t)unit_of(c.n) * NKT + c.s * KC) * (ATW * 512); };
  auto place_b = [&](Cursor& c) { c.q = bsrc + (int64_t)(c.s * KC) * p.row_tiles * 512; };
  auto step = [&](Cursor& c) { if (++c.s == NST) { c.s = 0; ++c.n; } };
  auto weight = [](const gbf16x8* q) { return __builtin_nontemporal_load(q); };
  bf16x8 ring[kTileRing][2 * NF], breg[2][BL], bt[2][R32];
  Cursor ca{0, 0, nullptr}, cb{0, 0, nullptr};
  place_b(cb);
#pragma unroll
  for (int u = 0; u < 2; ++u) {                      // stages 0 and 1
#pragma unroll
    for (int i = 0; i < BL; ++i) breg[u][i] = *(const gbf16x8*)(cb.q + b_rel[i]);
    step(cb);
    place_b(cb);
  }
  place_a(ca);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      __builtin_amdgcn_sched_barrier(0);             // (requested in the order in which the loop refills them)
      const gbf16x8* ap = (const gbf16x8*)(ca.q + j * (ATW * 512)) + lsrc;
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h) ring[u * KC + j][2 * f + h] = weight(ap + f * fstep + h * 32);
    }
    step(ca);
    place_a(ca);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < BL; ++i) *(bf16x8*)&lds[(int)threadIdx.x + kWideThreads * i] = breg[0][i];
  wg_barrier();
  stamp(p, e.ph, 3);

  for (int n = 0; n < n_my; ++n) {
    float rs[R32];                                   // the rows' 1/rms
#pragma unroll
    for (int t = 0; t < R32; ++t)
      rs[t] = ((const gfloat*)p.ssq)[min(t * 32 + (lane & 31), p.M - 1)];
    for (int st = 0; st < NST; st += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        // stage st + u is in LDS (buffer u), the one after it in breg[u ^ 1]; the loads of this turn are for two stages on
        const bf16x8* bs = (const bf16x8*)&lds[u * STAGE] + lsrc;
#pragma unroll
        for (int t = 0; t < R32; ++t) bt[0][t] = bs[t * 128];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < KC; ++j) {
          const gbf16x8* ap = (const gbf16x8*)(ca.q + j * (ATW * 512)) + lsrc;
          const int b0 = j * BL / KC, b1 = (j + 1) * BL / KC;         // the k-tile's share of a thread's staging
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int nx = 2 * j + h + 1;            // the k-half to come
#pragma unroll
            for (int i = 0; i < NM; ++i) {
              const int f = i / R32, t = i % R32;
              acc[f][t] = mfma32_f16(ring[u * KC + j][2 * f + h], bt[h][t], acc[f][t]);
              // between two MFMAs: an LDS read of the coming half and one of the k-tile's other memory operations
              if (nx < 2 * KC && i < R32) bt[nx & 1][i] = bs[(nx >> 1) * (RT * 64) + i * 128 + (nx & 1) * 32];
              if (h == 0 && (i & 1) == 0 && b0 + i / 2 < b1) breg[u][b0 + i / 2] = *(const gbf16x8*)(cb.q + b_rel[b0 + i / 2]);
              if (h == 0 && (i & 1) == 1 && b0 + i / 2 < b1)
                *(bf16x8*)&lds[(u ^ 1) * STAGE + (int)threadIdx.x + kWideThreads * (b0 + i / 2)] = breg[u ^ 1][b0 + i / 2];
              if (h == 1 && i >= 1 && i - 1 < NF) ring[u * KC + j][2 * (i - 1)] = weight(ap + (i - 1) * fstep);
              if (h == 1 && i + 1 == NM) {
#pragma unroll
                for (int ff = 0; ff < NF; ++ff) ring[u * KC + j][2 * ff + 1] = weight(ap + ff * fstep + 32);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
        step(ca);
        place_a(ca);
        step(cb);
        place_b(cb);
        wg_barrier();
      }
    }
    if (n == 0) stamp(p, e.ph, 4);
    // ---- epilogue from the accumulators.  Registers 4 q .. 4 q + 3 of a 32x32 tile: features 8 q + 4 (lane >> 5) .. + 3, row lane & 31
    const int f4 = (lane >> 5) * 4;
    const int unit = ((int)blockIdx.x + n * (int)gridDim.x) * 4 + wave;
    if (unit < n_groups) {
#pragma unroll
      for (int t = 0; t < R32; ++t) {
        const int m = t * 32 + (lane & 31);
        if (m < p.M) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int f = 0; f < NF; ++f) {
              const int n0 = unit * (ATW * 16) + f * 32 + 8 * q + f4;
              const f32x4 v = (f32x4){acc[f][t][4 * q], acc[f][t][4 * q + 1], acc[f][t][4 * q + 2], acc[f][t][4 * q + 3]};
              if ((n0 >> 4) < g.NT) st_f32x4_uncounted(e.out + (int64_t)m * e.ld + n0, v * rs[t]);
            }
        }
      }
    }
    zero_acc();
    if (n == 0) stamp(p, e.ph, 5);
  }
  stamp(p, e.ph, 2);
}

// The attention unit of the wide passes, a workgroup: NQ query tiles of one (sequence, KV head, key split) share every
// stored key and value block the unit pulls (a wide pass has 6 and more query tiles per sequence and head: units of one
// tile would pull the same trunk once per tile).  Same method and same layouts as attn_unit; the qkv projections
// arrive with the norm's row scale applied.  What shapes it, measured on 384 rows over 2048 keys of the 1B shape:
// - order of the loads: they return in order, and the first ring of stored keys is a burst of 32 MB over the chip, so the
//   queries and the fresh keys are requested before it and staged under it;
// - every query tile is rotated once, by one wavefront, and reaches the others through LDS;
// - vector instructions per score (they, not the MFMAs, fill the SIMDs): a row's reference maximum enters the score MFMAs as
//   their C operand, so scores come out ready for the exponential; the reference moves only when a score exceeds it by
//   2^8 (probabilities up to 256 are as exact as those up to 1), which one comparison per lane tests, instead of a maximum
//   across lanes per block; visibility is tested only in blocks that reach past a tile's shortest row;
// - the eight wavefronts' partial softmaxes of all NQ tiles meet in LDS at once, after the new keys have been appended.
// 26.0 us (36.1 with a unit that did none of this), 15.1 for 170 prompt tokens (22), 14.4 for 96 rows over 4 sequences of up
// to 1500 keys (26.8).
constexpr int kMultiFreshKeys = kFusedWideFreshKeys;   // LDS room: NQ x (rows per tile x slots per row) for NQ = 3, or the tokens of an extend
constexpr int kMultiVs = kMultiFreshKeys + 8;          // V^T row of the fresh keys
constexpr int kMultiQ = kFusedWideQueryTiles;          // most query tiles of a unit
constexpr float kMultiSlack = 8.0f;                    // log2 of how far scores may exceed the reference
// LDS: fresh keys [f][72], fresh values^T [64][kMultiVs]; then the query operands, later (same place) the partial outputs
// [NQ][wave][4][64] f32x4; then the partial (reference, sum) [NQ][wave][16][2]
constexpr size_t kMultiFreshBytes = (size_t)(kMultiFreshKeys * 72 + 64 * kMultiVs) * 2;
constexpr size_t kMultiRedBytes = (size_t)kMultiQ * kFusedWaves * 4 * 64 * 16;
constexpr size_t kMultiLdsBytes = kMultiFreshBytes + kMultiRedBytes + (size_t)kMultiQ * kFusedWaves * 16 * 2 * 4;
static_assert(kMultiFreshBytes % 16 == 0 && kMultiLdsBytes <= 160 * 1024, "LDS of the wide attention unit");

template <int NPQ, int NPP, int NQ, bool PG>
__global__ __launch_bounds__(kFusedThreads) void wide_attn_kernel(FusedParams p, bf16_t* trunk_k, bf16_t* trunk_vt, bf16_t* suffix_k,
                                                                  bf16_t* suffix_v, int ph) {
  extern __shared__ f32x4 lds[];
  bf16_t* kf_s = (bf16_t*)lds;
  bf16_t* vf_s = kf_s + kMultiFreshKeys * 72;
  f32x4* red = (f32x4*)((char*)lds + kMultiFreshBytes);
  bf16x8* q_s = (bf16x8*)red;                                  // [NQ][2 k-steps][NPQ planes][64]
  float* ml = (float*)((char*)red + kMultiRedBytes);
  stamp(p, ph, 0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g4 = lane >> 4;
  const int QG = (p.QT + NQ - 1) / NQ;        // groups of query tiles per (sequence, KV head)
  const int unit = blockIdx.x;
  const int hk = unit % p.Hkv;
  int rem = unit / p.Hkv;
  // (a prompt's later rows see more keys: their units go first, so that the last ones to start are the short ones.  Prefill of 700
  // tokens 2880 -> 2851 us, 1000 3325 -> 3306, 3000 10803 -> 10737, four runs a side in turn that do not overlap)
  const int qg = p.appended ? QG - 1 - rem % QG : rem % QG;
  rem /= QG;
  const int s = rem % p.NS, b = rem / p.NS;
  const int g_log = 31 - __builtin_clz(p.G), sl_log = p.SL == 8 ? 3 : 4;   // G and SL are powers of two
  const int RG = p.R << g_log;
  const bool is_branch = p.is_branch != 0;
  const gfloat* gq = (const gfloat*)p.qkv;
  const gfloat* gcs = (const gfloat*)p.cos_sin;
  const int rpt = 16 >> g_log;                                // rows per query tile
  // query row of a lane in tile t (clamped: rows past the last are computed like it and never stored)
  auto row_of = [&](int t) { return min((qg * NQ + t) * 16 + li, RG - 1); };

  const int kb0 = s * p.KPU;
  int pgs = 0;
  if constexpr (PG) pgs = p.pages[(int64_t)b * p.page_stride + min((kb0 >> 5) + wave + kFusedWaves * lane, p.page_stride - 1)];
  // ---- issue: row descriptors, the raw queries (wavefront t: tile t), the first fresh keys
  int tv[NQ];                                                 // stored keys this lane's query rows see
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    // (an extend's descriptor counts the pass's own tokens, here fresh keys, up to the row itself.  The pass's kind comes
    // from the launch: tested per row it would put a round trip to memory between these loads and the next)
    const int rloc = row_of(t) >> g_log;
    tv[t] = p.rows[b * p.R + rloc].vis - (is_branch || p.appended ? 0 : 1 + rloc);
  }
  f32x4 qraw[4], qcs[4];
  if (wave < NQ) {
    const int qr = row_of(wave), m = b * p.R + (qr >> g_log);
    const gfloat* qp = gq + (int64_t)m * p.qkvd + (hk * p.G + (qr & (p.G - 1))) * 64 + g4 * 8;
    qraw[0] = *(const gf32x4*)qp;
    qraw[1] = *(const gf32x4*)(qp + 4);
    qraw[2] = *(const gf32x4*)(qp + 32);
    qraw[3] = *(const gf32x4*)(qp + 36);
    const gfloat* cp = gcs + ((int64_t)m * 32 + g4 * 8) * 2;
#pragma unroll
    for (int i = 0; i < 4; ++i) qcs[i] = *(const gf32x4*)(cp + 4 * i);
  }
  // fresh keys: item = (key f, rotary quad / 8-dim group q8)
  const int n_fresh_keys = is_branch ? (NQ * rpt) << sl_log : p.R;
  const int n_fb = s == 0 && !p.appended ? (n_fresh_keys + 31) >> 5 : 0;
  const int nf8 = n_fb * 32 * 8;
  auto fresh_row = [&](int f, int& m_o, bool& valid, bool& stored) {
    if (is_branch) {
      const int rt = qg * NQ * rpt + (f >> sl_log), j = f & (p.SL - 1);
      m_o = b * p.R + min(rt, p.R - 1);
      valid = rt < p.R && j < p.suffix_len;
      stored = j < p.suffix_len - 1;
    } else {
      m_o = b * p.R + min(f, p.R - 1);
      valid = f < p.R;
      stored = false;
    }
  };
  struct Fresh {
    bool valid, stored;
    u32x2 k_lo, k_hi;              // stored: 4 + 4 key elements
    bf16x8 v;                      // stored: 8 value elements
    f32x4 a, bb, c0, c1, v0, v1;   // computed: raw projections and rotary table
  };
  auto load_fresh = [&](Fresh& x, int it) {
    const int f = it >> 3, q8 = it & 7;
    int m_o;
    fresh_row(f, m_o, x.valid, x.stored);
    x.valid = x.valid && it < nf8;
    if (!x.valid) return;
    // both sources in one stretch of loads (a branch on `stored` made the second wait for the first); the slots of a row
    // up to its own are inside its suffix
    const gfloat* kp = gq + (int64_t)m_o * p.qkvd + p.qd + hk * 64 + q8 * 4;
    x.a = *(const gf32x4*)kp;
    x.bb = *(const gf32x4*)(kp + 32);
    const gfloat* cs = gcs + ((int64_t)m_o * 32 + q8 * 4) * 2;
    x.c0 = *(const gf32x4*)cs;
    x.c1 = *(const gf32x4*)(cs + 4);
    const gfloat* vp = gq + (int64_t)m_o * p.qkvd + p.qd + p.kvd + hk * 64 + q8 * 8;
    x.v0 = *(const gf32x4*)vp;
    x.v1 = *(const gf32x4*)(vp + 4);
    if (is_branch) {
      const int64_t row = (((int64_t)m_o * p.suffix_cap + (f & (p.SL - 1))) * p.Hkv + hk) * 64;
      x.k_lo = *(const gu32x2*)(suffix_k + row + q8 * 4);
      x.k_hi = *(const gu32x2*)(suffix_k + row + 32 + q8 * 4);
      x.v = *(const gbf16x8*)(suffix_v + row + q8 * 8);
    }
  };
  auto stage_fresh = [&](const Fresh& x, int it) {   // rotated, to LDS (zeros where there is no key)
    if (it >= nf8) return;
    const int f = it >> 3, q8 = it & 7;
    u32x2 k_lo = (u32x2){0u, 0u}, k_hi = (u32x2){0u, 0u};
    Bf8 vv;
    vv.w = (u32x4){0u, 0u, 0u, 0u};
    if (x.valid && x.stored) {
      k_lo = x.k_lo;
      k_hi = x.k_hi;
      vv.v = x.v;
    } else if (x.valid) {
      const float cc[8] = {x.c0[0], x.c0[1], x.c0[2], x.c0[3], x.c1[0], x.c1[1], x.c1[2], x.c1[3]};
      bf16_t x0[4], x1[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float c = cc[2 * e], sn = cc[2 * e + 1];
        x0[e] = to_bf16(x.a[e] * c - x.bb[e] * sn);
        x1[e] = to_bf16(x.bb[e] * c + x.a[e] * sn);
        vv.u[e] = to_bf16(x.v0[e]);
        vv.u[4 + e] = to_bf16(x.v1[e]);
      }
      const uint64_t p0 = pack_bf16x4(x0[0], x0[1], x0[2], x0[3]), p1 = pack_bf16x4(x1[0], x1[1], x1[2], x1[3]);
      k_lo = (u32x2){(uint32_t)p0, (uint32_t)(p0 >> 32)};
      k_hi = (u32x2){(uint32_t)p1, (uint32_t)(p1 >> 32)};
    }
    *(u32x2*)(kf_s + f * 72 + q8 * 4) = k_lo;
    *(u32x2*)(kf_s + f * 72 + 32 + q8 * 4) = k_hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) vf_s[(q8 * 8 + e) * kMultiVs + f] = vv.u[e];
  };
  Fresh fr[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) load_fresh(fr[i], (int)threadIdx.x + i * kFusedThreads);
  __builtin_amdgcn_sched_barrier(0);

  // ---- issue: the first trunk blocks of this wavefront (block counts from the host's bound)
  // (appended: the rows of the pass before the unit's last one are stored keys too)
  const int kend_ub = min(kb0 + p.KPU, p.tv_ub + (p.appended ? min(((qg + 1) * NQ * 16 - 1) >> g_log, p.R - 1) + 1 : 0));
  const int n_tb = kend_ub > kb0 ? (kend_ub - kb0 + 31) >> 5 : 0;
  const int n_mine = n_tb > wave ? (n_tb - wave + kFusedWaves - 1) / kFusedWaves : 0;
  const int krow = (li >> 2) * 8 + (li & 3);                  // key of this lane's A-operand row in a block (tile 0)
  // PG (paged trunk, App. B "PagedAttention"): block j of sequence b is page p.pages[b][j] of a pool shared by all
  // sequences, a page = the same 4 KiB per head and operand as a block of the contiguous layouts.  Lane i of a wavefront
  // fetched the page of the wavefront's i-th block first of all (one load), so the block loop itself stays free of
  // dependent loads; entries behind a sequence's allocation name page 0, which exists and holds zeros.
  const int64_t head0 = PG ? 0 : ((int64_t)(b * p.Hkv + hk) * p.vt_stride) * 64;
  const gbf16* kbase = (const gbf16*)trunk_k + head0 + g4 * 8;
  const gbf16* vbase = (const gbf16*)trunk_vt + head0 + li * 32 + g4 * 8;
  struct KvBlock {
    bf16x8 k[2][2];
    bf16x8 vt[4];
  };
  constexpr int RING = 2;
  KvBlock ring[RING];
  auto load_trunk = [&](KvBlock& tb, int i) {   // i-th block of this wavefront, clamped to its last one
    const int ic = max(min(i, n_mine - 1), 0);
    const int blk = wave + kFusedWaves * ic;
    const int kb = min(kb0 + blk * 32, p.vt_stride - 32);
    const int64_t bo = PG ? ((int64_t)__builtin_amdgcn_readlane(pgs, ic) * p.Hkv + hk) * 2048 : (int64_t)kb * 64;
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const gbf16* kp = kbase + bo + (krow + tile * 4) * 64;
      tb.k[tile][0] = *(const gbf16x8*)kp;
      tb.k[tile][1] = *(const gbf16x8*)(kp + 32);
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) tb.vt[dt] = *(const gbf16x8*)(vbase + bo + dt * 16 * 32);
  };
#pragma unroll
  for (int i = 0; i < RING; ++i) load_trunk(ring[i], i);   // unconditional (a wavefront without blocks re-reads block 0)
  __builtin_amdgcn_sched_barrier(0);
  stamp(p, ph, 3);

  // ---- query operands: dims g4*8..+7 (k-step 0) and 32+g4*8..+7 (k-step 1) of the rows, rotated and scaled
  if (wave < NQ) {
    const float scale = 0.125f * kLog2e;
    Bf8 qh[2], ql[2];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float a = qraw[e >> 2][e & 3], bb = qraw[2 + (e >> 2)][e & 3];
      const float c = qcs[e >> 1][2 * (e & 1)], sn = qcs[e >> 1][2 * (e & 1) + 1];
      const float x0 = (a * c - bb * sn) * scale, x1 = (bb * c + a * sn) * scale;
      qh[0].u[e] = to_bf16(x0);
      qh[1].u[e] = to_bf16(x1);
      ql[0].u[e] = to_bf16(x0 - bf16_to_f32(qh[0].u[e]));
      ql[1].u[e] = to_bf16(x1 - bf16_to_f32(qh[1].u[e]));
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      q_s[((wave * 2 + ks) * NPQ) * 64 + lane] = qh[ks].v;
      if (NPQ == 2) q_s[((wave * 2 + ks) * NPQ + 1) * 64 + lane] = ql[ks].v;
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) stage_fresh(fr[i], (int)threadIdx.x + i * kFusedThreads);
  for (int it = threadIdx.x + 2 * kFusedThreads; it < nf8; it += kFusedThreads) {
    load_fresh(fr[0], it);
    stage_fresh(fr[0], it);
  }
  wg_barrier();
  bf16x8 q[NQ][2][NPQ];
#pragma unroll
  for (int t = 0; t < NQ; ++t)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int pl = 0; pl < NPQ; ++pl) q[t][ks][pl] = q_s[((t * 2 + ks) * NPQ + pl) * 64 + lane];
  stamp(p, ph, 5);

  // running softmax per tile: negref = minus the reference (all four elements), thr = how far above the reference a score
  // moves it (-inf before the row's first visible key), sum of this lane's share, outputs
  f32x4 negref[NQ], acc[NQ][4];
  float thr[NQ], l_run[NQ];
  int vmin[NQ];                                               // stored keys every row of the tile sees
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    negref[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    thr[t] = -INFINITY;
    l_run[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) acc[t][dt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    int v = tv[t];
    v = lanes_reduce<8>(v, [](int a, int b) { return min(a, b); });
    vmin[t] = __builtin_amdgcn_readfirstlane(v);
  }
  // one 32-key block against tile t: scores of this lane's row for keys g4*8..+7 of the block
  auto tile_step = [&](int t, const bf16x8 (&k)[2][2], const bf16x8 (&vt)[4], bool masked, auto visible) {
    f32x4 S[2];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      S[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[tile][0], q[t][0][0], negref[t], 0, 0, 0);
      S[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[tile][1], q[t][1][0], S[tile], 0, 0, 0);
      if (NPQ == 2) {
        S[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[tile][0], q[t][0][NPQ - 1], S[tile], 0, 0, 0);
        S[tile] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[tile][1], q[t][1][NPQ - 1], S[tile], 0, 0, 0);
      }
    }
    float sv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sv[e] = S[e >> 2][e & 3];
    if (masked) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] = visible(e) ? sv[e] : -INFINITY;
    }
    const float mx = fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
    if (__any(mx > thr[t])) {
      const float mr = max_over_rows(mx);
      const bool move = mr > thr[t];                          // (the same for the four lanes of a row)
      const float shift = move ? mr : 0.f;
      const float corr = thr[t] == -INFINITY ? 1.0f : exp2_fast(-shift);
      l_run[t] *= corr;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) acc[t][dt] = acc[t][dt] * corr;
      const float nr = negref[t][0] - shift;
      negref[t] = (f32x4){nr, nr, nr, nr};
      if (move) thr[t] = kMultiSlack;
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] -= shift;
    }
    Bf8 phi, plo;
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = exp2_fast(sv[e]);
      psum += pe;
      phi.u[e] = to_bf16(pe);
      if (NPP == 2) plo.u[e] = to_bf16(pe - bf16_to_f32(phi.u[e]));
    }
    l_run[t] += psum;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      acc[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[dt], phi.v, acc[t][dt], 0, 0, 0);
      if (NPP == 2) acc[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[dt], plo.v, acc[t][dt], 0, 0, 0);
    }
  };

  // ---- stored trunk keys: RING blocks in flight, every block scored against all NQ query tiles.  The last turn of the
  // ring loads nothing new that is used (clamped duplicates of the last block)
  for (int i0 = 0; i0 < n_mine; i0 += RING) {
#pragma unroll
    for (int r = 0; r < RING; ++r) {
      if (i0 + r < n_mine) {
        const int kb = kb0 + (wave + kFusedWaves * (i0 + r)) * 32;
#pragma unroll
        for (int t = 0; t < NQ; ++t)
          tile_step(t, ring[r].k, ring[r].vt, kb + 32 > vmin[t], [&](int e) { return kb + g4 * 8 + e < tv[t]; });
      }
      load_trunk(ring[r], i0 + r + RING);
    }
  }
  stamp(p, ph, 6);
  // ---- fresh blocks continue the round-robin after the trunk blocks; a tile skips blocks none of its rows can see
  for (int blk = n_tb + ((wave - n_tb) & (kFusedWaves - 1)); blk < n_tb + n_fb; blk += kFusedWaves) {
    const int f0 = (blk - n_tb) * 32;
    bf16x8 kk[2][2], vt[4];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      const bf16_t* kp = kf_s + (f0 + krow + tile * 4) * 72 + g4 * 8;
      kk[tile][0] = *(const bf16x8*)kp;
      kk[tile][1] = *(const bf16x8*)(kp + 32);
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) vt[dt] = *(const bf16x8*)(vf_s + (dt * 16 + li) * kMultiVs + f0 + g4 * 8);
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      const bool any = is_branch ? f0 < ((t + 1) * rpt) << sl_log && f0 + 32 > (t * rpt) << sl_log
                                 : f0 <= ((qg * NQ + t) * 16 + 15) >> g_log;
      if (!any) continue;
      const int rloc = row_of(t) >> g_log;                    // row of the sequence; its keys as (row in the unit, slot)
      const int own = rloc - qg * NQ * rpt;
      tile_step(t, kk, vt, true, [&](int e) {
        const int f = f0 + g4 * 8 + e;
        return is_branch ? (f >> sl_log) == own && (f & (p.SL - 1)) < p.suffix_len : f <= rloc;
      });
    }
  }
  stamp(p, ph, 7);
  // ---- append the keys and values computed in this pass for later passes, from their LDS copies: the row's private
  // suffix slot (branch) or its trunk position (extend)
  for (int it = threadIdx.x; it < nf8; it += kFusedThreads) {
    const int f = it >> 3, q8 = it & 7;
    int m_o;
    bool valid, stored;
    fresh_row(f, m_o, valid, stored);
    if (!valid || stored) continue;
    const u32x2 k_lo = *(const u32x2*)(kf_s + f * 72 + q8 * 4), k_hi = *(const u32x2*)(kf_s + f * 72 + 32 + q8 * 4);
    Bf8 vv;
#pragma unroll
    for (int e = 0; e < 8; ++e) vv.u[e] = vf_s[(q8 * 8 + e) * kMultiVs + f];
    if (is_branch) {
      const int64_t row = (((int64_t)m_o * p.suffix_cap + (p.suffix_len - 1)) * p.Hkv + hk) * 64;
      *(gu32x2*)(suffix_k + row + q8 * 4) = k_lo;
      *(gu32x2*)(suffix_k + row + 32 + q8 * 4) = k_hi;
      *(gbf16x8*)(suffix_v + row + q8 * 8) = vv.v;
    } else {
      const int slot = p.rows[m_o].kv_slot;
      if (slot < 0) continue;                                 // a row that only pads
      const int64_t bb = PG ? ((int64_t)p.pages[(int64_t)b * p.page_stride + (slot >> 5)] * p.Hkv + hk) * 2048
                            : (int64_t)(b * p.Hkv + hk) * p.vt_stride * 64 + (int64_t)(slot >> 5) * 2048;
      const int64_t row = bb + (int64_t)(slot & 31) * 64;
      *(gu32x2*)(trunk_k + row + q8 * 4) = k_lo;
      *(gu32x2*)(trunk_k + row + 32 + q8 * 4) = k_hi;
      gbf16* vcol = (gbf16*)trunk_vt + bb + (q8 * 8) * 32 + (slot & 31);
#pragma unroll
      for (int e = 0; e < 8; ++e) vcol[e * 32] = vv.u[e];
    }
  }
  // ---- the 8 wavefronts' partial softmaxes meet in LDS (every wavefront read its queries before the barrier above and has
  // passed it, but another may still be on its way there: a barrier before their place is written)
  wg_barrier();
#pragma unroll
  for (int t = 0; t < NQ; ++t) {
    l_run[t] = sum_over_rows(l_run[t]);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) red[((t * kFusedWaves + wave) * 4 + dt) * 64 + lane] = acc[t][dt];
    if (g4 == 0) {
      ml[((t * kFusedWaves + wave) * 16 + li) * 2] = thr[t] == -INFINITY ? -INFINITY : -negref[t][0];
      ml[((t * kFusedWaves + wave) * 16 + li) * 2 + 1] = l_run[t];
    }
  }
  wg_barrier();
  for (int idx = threadIdx.x; idx < NQ * 256; idx += kFusedThreads) {
    const int t = idx >> 8, qi = idx & 15, dq = (idx >> 4) & 15;       // query row of tile t, dims 4 dq .. 4 dq + 3
    const float* mlt = ml + (t * kFusedWaves * 16 + qi) * 2;
    float mmax = -INFINITY;
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) mmax = fmaxf(mmax, mlt[w * 32]);
    const float m_use = mmax == -INFINITY ? 0.f : mmax;
    float lsum = 0.f;
    f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kFusedWaves; ++w) {
      const float wgt = exp2_fast(mlt[w * 32] - m_use);
      lsum += wgt * mlt[w * 32 + 1];
      o += red[((t * kFusedWaves + w) * 4 + (dq >> 2)) * 64 + qi + 16 * (dq & 3)] * wgt;
    }
    const int qrow = (qg * NQ + t) * 16 + qi;
    if (qrow >= RG) continue;
    if (p.NS == 1) {
      const int mm = b * p.R + (qrow >> g_log);
      const int k = (hk * p.G + (qrow & (p.G - 1))) * 64 + dq * 4;
      const float inv = 1.0f / lsum;
      bf16_t hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) hi[e] = to_f16(o[e] * inv);
      *(uint64_t*)(p.att + b_off_of(p.row_tiles, k, mm)) = pack_bf16x4(hi[0], hi[1], hi[2], hi[3]);
    } else {
      const int64_t pb = ((int64_t)(b * p.Hkv + hk) * p.NS + s) * (p.QT * 16) + qrow;
      if (dq == 0) *(uint64_t*)(p.part_ml + pb * 2) = pack_f32x2(mmax, lsum);
      *(gf32x4*)((gfloat*)p.part_o + pb * 64 + dq * 4) = o;
    }
  }
  stamp(p, ph, 2);
}

// The keys (rotated) and values of an extend of many tokens, into the trunk ahead of its attention, which then finds every
// key in one place: units of a prompt chunk would each rotate and stage all of its keys (170 tokens: 1360 items per unit)
// and have LDS room for kFusedWideFreshKeys of them.  Thread = (row, KV head, rotary quad / 8-dim group).  5.0 us at 340 rows.
template <bool PG>
__global__ __launch_bounds__(256) void wide_append_kernel(FusedParams p, bf16_t* trunk_k, bf16_t* trunk_vt) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int q8 = idx & 7, hk = (idx >> 3) % p.Hkv, m = (idx >> 3) / p.Hkv;
  if (m >= p.M) return;
  const int stored_at = p.rows[m].kv_slot, slot = max(stored_at, 0), b = m / p.R;
  const gfloat* src = (const gfloat*)p.qkv + (int64_t)m * p.qkvd + p.qd + hk * 64;
  const f32x4 a = *(const gf32x4*)(src + q8 * 4), bb = *(const gf32x4*)(src + 32 + q8 * 4);
  const gfloat* cs = (const gfloat*)p.cos_sin + ((int64_t)m * 32 + q8 * 4) * 2;
  const f32x4 c0 = *(const gf32x4*)cs, c1 = *(const gf32x4*)(cs + 4);
  const f32x4 v0 = *(const gf32x4*)(src + p.kvd + q8 * 8), v1 = *(const gf32x4*)(src + p.kvd + q8 * 8 + 4);
  const int64_t base = PG ? ((int64_t)p.pages[(int64_t)b * p.page_stride + (slot >> 5)] * p.Hkv + hk) * 2048
                          : (int64_t)(b * p.Hkv + hk) * p.vt_stride * 64 + (int64_t)(slot >> 5) * 2048;
  bf16_t x0[4], x1[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float c = e < 2 ? c0[2 * e] : c1[2 * e - 4], sn = e < 2 ? c0[2 * e + 1] : c1[2 * e - 3];
    x0[e] = to_bf16(a[e] * c - bb[e] * sn);
    x1[e] = to_bf16(bb[e] * c + a[e] * sn);
  }
  if (stored_at < 0) return;                                  // a row that only pads (tested behind the loads)
  const int64_t row = base + (int64_t)(slot & 31) * 64 + q8 * 4;
  *(uint64_t*)(trunk_k + row) = pack_bf16x4(x0[0], x0[1], x0[2], x0[3]);
  *(uint64_t*)(trunk_k + row + 32) = pack_bf16x4(x1[0], x1[1], x1[2], x1[3]);
  gbf16* vcol = (gbf16*)trunk_vt + base + (q8 * 8) * 32 + (slot & 31);
#pragma unroll
  for (int e = 0; e < 8; ++e) vcol[e * 32] = to_bf16(e < 4 ? v0[e & 3] : v1[e & 3]);
}

// Merge of a wide pass's key splits.
__global__ __launch_bounds__(kFusedThreads) void wide_merge_kernel(FusedParams p, int ph) {
  stamp(p, ph, 0);
  attn_merge_unit<kFusedWideRows, 1>(p, p.row_tiles, blockIdx.x, p.part_o, p.part_ml, p.att);
  stamp(p, ph, 2);
}

// ---------------------------------------------------------------------------------------------- the kernel
// Register chunks in flight per wavefront in the ring: a divisor of the KT k-tiles a wavefront takes of a unit.
template <int MT, int KT, int NP> struct Depth {
  static constexpr int a4 = KT == 2 ? 2 : (MT * NP > 4 ? 2 : 4);   // four feature tiles per unit
};

// KT: k-tiles per wavefront of a unit over the model width (d / 256: 8, 4 or 2, what the host admits).  An instance for each: the loop of
// gate/up holds that many in registers, and two such loops in one kernel spill.
template <int MT, int KT, class PL, bool PG, bool SM>
__global__ __launch_bounds__(kFusedThreads) void fused_kernel(FusedParams p, int first, int last, int persistent) {
  constexpr int MP = kFusedMaxRows;
  extern __shared__ f32x4 red[];
  __shared__ float r_s[64];
  __shared__ int dead;
  if (threadIdx.x == 0) dead = 0;
  wg_barrier();
  // The barrier counts on from where the previous launch stopped (its last epoch is kept in a word of its own), so
  // the barrier words never have to be cleared between launches.
  Grid grid{p.bar, p.err, persistent ? p.bar[kBarEpochWord] : 0u, persistent, p.nwg, &dead, p.spin_limit};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t h_stride = (int64_t)MP * p.d;
  const int64_t ssq_stride = (int64_t)(p.d >> 4) * MP;
  const int lm_phase = fused_last_phase(p.L);

  for (int ph = first; ph <= last; ++ph) {
    // the merge phase: none with one key split, and none where the attention units merge their splits themselves
    if ((SM || p.NS == 1) && ph > 0 && ph < lm_phase && (ph - 1) % 6 == 2) continue;
    const int l = ph == 0 ? 0 : (ph == lm_phase ? p.L - 1 : (ph - 1) / 6);
    const int sub = ph == 0 ? -1 : (ph == lm_phase ? 6 : (ph - 1) % 6);
    // group sync (see group_wait): no grid barrier between a layer's qkv phase and its attention phase
    const bool gs = persistent && p.qkv_ug > 0;
    const bool do_wait = persistent && ph > first && !(gs && sub == 1);
    stamp(p, ph, 0);
    if (ph == 0 && p.prof && threadIdx.x == 0) {
      unsigned xcc;
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
      p.prof[(int64_t)7 * p.nwg + blockIdx.x] = xcc;   // phase 0, slot 7: the XCD this workgroup runs on
    }
    const FusedLayer L = p.layers[l];
    float* qkv = p.qkv + (int64_t)l * MP * p.qkvd;
    bf16_t* att = p.att + (int64_t)l * 2 * MP * p.qd;
    bf16_t* act = p.act + (int64_t)l * 2 * MP * p.ffn;

    // ---- what a linear-layer phase streams, reads and writes
    FusedGemm g{};
    const bf16_t* bsrc = nullptr;
    int64_t bplane = 0;
    int epi = 0;
    EpiArgs e{};
    const float* ssq_in = nullptr;
    // the unit of this workgroup in the phases of at most one unit per workgroup: the workgroup's index, or, with group
    // sync, the qkv units of KV head gq's group (2 G for its query heads, 2 for its keys, 2 for its values, 32
    // features each) on workgroups 7 - gq, 15 - gq, ..: the XCD on which that head's attention units run
    int my_unit = (int)blockIdx.x;
    int qkv_flag = -1;    // word of the flags this workgroup sets after its qkv unit
    if (gs && sub == 0) {
      const int gq = 7 - ((int)blockIdx.x & 7), jj = (int)blockIdx.x >> 3;
      my_unit = -1;
      if (gq < p.Hkv && jj < p.qkv_ug) {
        const int nq = 2 * p.G;
        my_unit = jj < nq ? gq * nq + jj : (jj < nq + 2 ? 2 * p.Hq + 2 * gq + (jj - nq) : 2 * p.Hq + 2 * p.Hkv + 2 * gq + (jj - nq - 2));
        qkv_flag = (l * 8 + gq) * 16 + jj;
      }
    }
    // K-split scratch of this phase instance (sub 0, 3, 5 -> slot 0, 1, 2)
    const int fix_slot = l * 3 + (sub == 0 ? 0 : (sub == 3 ? 1 : 2));
    e.fix_buf = p.fix_buf + (int64_t)fix_slot * p.fix_stride;
    if (sub == 0) {
      g = L.qkv; bsrc = p.xn + (int64_t)(2 * l) * 2 * h_stride; bplane = h_stride; epi = FE_QKV;
      e.out = qkv; e.ld = p.qkvd;
      // the attention phase finds this layer's row scales in LDS; attention units are dealt out from the far end of
      // the grid, so (few rows) the workgroups that compute them here are not the ones that hold a qkv unit
      if (p.nwg - 1 - (int)blockIdx.x < p.n_attn_units) ssq_in = p.ssq + (int64_t)(2 * l) * ssq_stride;
    } else if (sub == 3 || sub == 5) {
      const int v = sub == 3 ? 2 * l + 1 : 2 * l + 2;
      g = sub == 3 ? L.o : L.down;
      bsrc = sub == 3 ? att : act;
      bplane = sub == 3 ? (int64_t)MP * p.qd : (int64_t)MP * p.ffn;
      epi = FE_RESID;
      e.h_in = p.h + (int64_t)(v - 1) * h_stride;
      e.h_out = p.h + (int64_t)v * h_stride;
      e.gain = sub == 3 ? L.mlp_norm : (l + 1 < p.L ? p.layers[l + 1].attn_norm : p.final_norm);
      e.xn_out = p.xn + (int64_t)v * 2 * h_stride;
      e.ssq_out = p.ssq + (int64_t)v * ssq_stride;
    } else if (sub == 4) {
      const int v = 2 * l + 1;
      g = L.gu; bsrc = p.xn + (int64_t)v * 2 * h_stride; bplane = h_stride; epi = FE_SWIGLU;
      e.act_out = act;
      ssq_in = p.ssq + (int64_t)v * ssq_stride;
    } else if (sub == 6) {
      const int v = 2 * p.L;
      g = p.lm; bsrc = p.xn + (int64_t)v * 2 * h_stride; bplane = h_stride; epi = FE_LOGITS;
      e.out = p.logits; e.ld = p.logits_ld;
      ssq_in = p.ssq + (int64_t)v * ssq_stride;
      if (!p.logits) g.n_units = 0;   // hidden states only
    }

    if (sub == -1) {
      // ---- embedding gather: residual stream version 0
      for (int u = blockIdx.x; u < (p.d >> 4); u += p.nwg) {
        if (wave < MT) {
          const int m = wave * 16 + (lane & 15);
          const int n = u * 16 + (lane >> 4) * 4;
          int tok = p.tokens[min(m, p.M - 1)];
          tok = tok < 0 ? 0 : (tok >= p.V ? p.V - 1 : tok);
          u32x2 eb = *(const gu32x2*)(p.embed + (int64_t)tok * p.d + n);
          f32x4 hn = (f32x4){__uint_as_float(eb.x << 16), __uint_as_float(eb.x & 0xffff0000u),
                             __uint_as_float(eb.y << 16), __uint_as_float(eb.y & 0xffff0000u)};
          resid_store<MT, MP, PL::xn>(p, hn, m, n, lane, *(const gu32x2*)(L.attn_norm + n), p.h, p.xn, p.ssq, u);
        }
      }
    } else if (sub == 0 || sub == 3 || sub == 5) {
      // one instance of the loop for the three phases where their operands have the same number of planes (the code
      // has to stay resident in the instruction cache across the layers)
      bool ok;
      if constexpr (PL::xn == PL::att && PL::xn == PL::act) {
        ok = gemm_phase<kAtQkv, MT, PL::xn, 2, true, MP, PL::xn, PL::act>(p, g, bsrc, bplane, epi, e, grid, do_wait, red, r_s, ssq_in, ph, my_unit);
      } else {
        if (sub == 0) ok = gemm_phase<kAtQkv, MT, PL::xn, 2, true, MP, PL::xn, PL::act>(p, g, bsrc, bplane, epi, e, grid, do_wait, red, r_s, ssq_in, ph, my_unit);
        else if (sub == 3) ok = gemm_phase<kAtQkv, MT, PL::att, 2, true, MP, PL::xn, PL::act>(p, g, bsrc, bplane, epi, e, grid, do_wait, red, r_s, ssq_in, ph, my_unit);
        else ok = gemm_phase<kAtQkv, MT, PL::act, 2, true, MP, PL::xn, PL::act>(p, g, bsrc, bplane, epi, e, grid, do_wait, red, r_s, ssq_in, ph, my_unit);
      }
      if (!ok) return;
      // (the unit's stores have left: it ended with a drain and a workgroup barrier)
      if (qkv_flag >= 0 && threadIdx.x == 0)
        __hip_atomic_store(p.qkv_flags + qkv_flag, grid.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (PL::xn == 1 && sub == 4 && g.n_units <= p.nwg) {
      // (more units than workgroups exist only on a device of fewer than 256 compute units: the down-projection admits a d_ffn of
      // at most 8192; they stream through the ring)
      if (!gemm_phase<4, MT, PL::xn, 2, true, MP, PL::xn, PL::act, KT>(p, g, bsrc, bplane, FE_SWIGLU, e, grid, do_wait, red, r_s, ssq_in, ph,
                                                                       (int)blockIdx.x)) return;
    } else if (sub == 4 || sub == 6) {
      const bool ok = gemm_phase<4, MT, PL::xn, Depth<MT, KT, PL::xn>::a4, false, MP, PL::xn, PL::act>(p, g, bsrc, bplane, epi, e, grid, do_wait, red, r_s, ssq_in, ph, my_unit);
      if (!ok) return;
      if (sub == 6 && p.hidden) {
        // final-norm hidden states (the row scales are in LDS)
        const gfloat* hv = (const gfloat*)(p.h + (int64_t)(2 * p.L) * h_stride);
        for (int m = blockIdx.x; m < p.M; m += p.nwg)
          for (int c = threadIdx.x; c < p.d; c += kFusedThreads)
            p.hidden[(int64_t)m * p.hidden_ld + c] = hv[(int64_t)m * p.d + c] * bf16_to_f32(p.final_norm[c]) * r_s[m];
      }
    } else if (sub == 1) {
      float* part_o = p.part_o + (int64_t)l * p.part_layer_stride * 64;
      float* part_ml = p.part_ml + (int64_t)l * p.part_layer_stride * 2;
      // the qkv phase left this layer's row scales in LDS; a launch that starts here computes them itself
      if (ph == first) compute_row_scales<MP>(p, p.ssq + (int64_t)(2 * l) * ssq_stride, r_s);
      // a workgroup with a unit waits for the grid inside its first unit, after requesting that unit's stored keys
      const bool group = gs && ph > first;           // wait for the unit's group instead of the grid
      bool waited = !(do_wait || group);
      for (int u = p.nwg - 1 - (int)blockIdx.x; u < p.n_attn_units; u += p.nwg) {
        if (!attn_unit<MT, MP, PL::q, PL::p, PL::att, PG, SM>(p, L, qkv, u, r_s, red, att, part_o, part_ml,
                                                           p.arrivals + (int64_t)l * p.arrivals_stride, ph, waited ? nullptr : &grid,
                                                           group ? p.qkv_flags + l * 128 : nullptr)) return;
        waited = true;
      }
      if (!waited && !group) {
        if (!grid_wait(grid)) return;
        stamp(p, ph, 1);
      }
    } else {
      // merge of the key splits; with a single split the attention units wrote the final output and this phase
      // (and its barrier) does not exist
      float* part_o = p.part_o + (int64_t)l * p.part_layer_stride * 64;
      float* part_ml = p.part_ml + (int64_t)l * p.part_layer_stride * 2;
      if (do_wait && !grid_wait(grid)) return;
      stamp(p, ph, 1);
      for (int u = blockIdx.x; u < p.n_pair_units; u += p.nwg) attn_merge_unit<MP, PL::att>(p, MT, u, part_o, part_ml, att);
    }
    stamp(p, ph, 2);
    if (ph < last && !(gs && sub == 0)) grid_arrive(grid);
  }
  // every workgroup read the word before the first barrier of this launch, which workgroup 0 has passed by now
  if (persistent && blockIdx.x == 0 && threadIdx.x == 0) p.bar[kBarEpochWord] = grid.epoch;
}

// ---------------------------------------------------------------------------------------------- set-up kernels
__global__ void retile_stream_kernel(const bf16_t* __restrict__ src0, int rows0, const bf16_t* __restrict__ src1, int rows1,
                                     const bf16_t* __restrict__ src2, int rows2, int mode, int AT, int KS, int Kd, int n_units,
                                     bf16_t* __restrict__ dst) {
  const int KTW = Kd / 32 / kFusedWaves / KS;
  const int64_t total = (int64_t)n_units * kFusedWaves * KTW * AT * 64;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int lane = (int)(idx & 63);
  int64_t tile = idx >> 6;
  const int j = (int)(tile % AT);
  tile /= AT;
  const int i = (int)(tile % KTW);
  tile /= KTW;
  const int w = (int)(tile % kFusedWaves);
  const int64_t unit = tile / kFusedWaves;
  const int64_t u = unit / KS;            // feature-tile group
  const int ks = (int)(unit % KS);        // k-slice
  const int kt = (ks * kFusedWaves + w) * KTW + i;
  const bf16_t* src = nullptr;
  int64_t row = 0;
  if (mode == 0) {
    int64_t n = (u * AT + j) * 16 + (lane & 15);
    if (n < rows0) { src = src0; row = n; }
    else if (n < (int64_t)rows0 + rows1) { src = src1; row = n - rows0; }
    else if (n < (int64_t)rows0 + rows1 + rows2) { src = src2; row = n - rows0 - rows1; }
  } else {
    int64_t n = (2 * u + (j & 1)) * 16 + (lane & 15);
    if (n < rows0) { src = j < 2 ? src0 : src1; row = n; }
  }
  u32x4 v = (u32x4){0u, 0u, 0u, 0u};
  if (src) v = *(const u32x4*)(src + row * Kd + kt * 32 + (lane >> 4) * 8);
  *(u32x4*)(dst + idx * 8) = v;
}

// [B][len][Hkv][64] keys and values -> the head-major trunk layouts of the fused pass
// pages != null: paged trunk, block j of sequence b in page pages[b * page_stride + j] of the pool
__global__ void copy_kv_fused_kernel(bf16_t* trunk_k, bf16_t* trunk_vt, const bf16_t* src_k, const bf16_t* src_v, int len,
                                     int Hkv, int vt_stride, int64_t total, const int32_t* pages, int page_stride) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // over [B][len][Hkv][64]
  if (idx >= total) return;
  int d = (int)(idx & 63);
  int64_t r = idx >> 6;
  int hk = (int)(r % Hkv);
  r /= Hkv;
  int pos = (int)(r % len);
  int64_t b = r / len;
  const int64_t bb = pages ? ((int64_t)pages[b * page_stride + (pos >> 5)] * Hkv + hk) * 2048
                           : (b * Hkv + hk) * (int64_t)vt_stride * 64 + (int64_t)(pos >> 5) * 2048;
  trunk_k[bb + (int64_t)(pos & 31) * 64 + d] = src_k[idx];
  trunk_vt[bb + d * 32 + (pos & 31)] = src_v[idx];
}

constexpr size_t kFusedLdsBytes = 96 * 1024;   // reduction tiles (<= 8 wavefronts x 12 tiles x 1 KiB); also keeps one workgroup per CU

template <int MT, int KT, class PL, bool PG, bool SM>
int check_residency_sm(int nwg, int cus) {
  SSD_HIP(hipFuncSetAttribute((const void*)fused_kernel<MT, KT, PL, PG, SM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFusedLdsBytes));
  int per_cu = 0;
  SSD_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fused_kernel<MT, KT, PL, PG, SM>, kFusedThreads, kFusedLdsBytes));
  SSD_CHECK_ARG((int64_t)per_cu * cus >= nwg,
                "fused pass: %d workgroups cannot be resident at once (%d per compute unit x %d compute units): the grid barrier "
                "would never complete", nwg, per_cu, cus);
  return SSD_OK;
}

template <int MT, int KT, class PL, bool PG>
int check_residency_mt(int nwg, int cus) {
  SSD_TRY((check_residency_sm<MT, KT, PL, PG, false>(nwg, cus)));
  return check_residency_sm<MT, KT, PL, PG, true>(nwg, cus);
}

template <int MT, int KT, class PL, bool PG, bool SM>
int launch_sm(const FusedParams& p, int first, int last, int persistent, hipStream_t s) {
  const size_t lds = kFusedLdsBytes;
  static bool configured = false;
  if (!configured) {
    SSD_HIP(hipFuncSetAttribute((const void*)fused_kernel<MT, KT, PL, PG, SM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    configured = true;
  }
  if (persistent) {
    fused_kernel<MT, KT, PL, PG, SM><<<p.nwg, kFusedThreads, lds, s>>>(p, first, last, 1);
    SSD_HIP(hipGetLastError());
  } else {
    const int lm_phase = fused_last_phase(p.L);
    for (int ph = first; ph <= last; ++ph) {
      if ((SM || p.NS == 1) && ph > 0 && ph < lm_phase && (ph - 1) % 6 == 2) continue;   // no merge phase
      fused_kernel<MT, KT, PL, PG, SM><<<p.nwg, kFusedThreads, lds, s>>>(p, ph, ph, 0);
      SSD_HIP(hipGetLastError());
    }
  }
  return SSD_OK;
}

// Passes with several key splits take the kernel whose attention units merge them.
template <int MT, int KT, class PL, bool PG>
int launch_mt(const FusedParams& p, int first, int last, int persistent, hipStream_t s) {
  if (p.NS > 1) return launch_sm<MT, KT, PL, PG, true>(p, first, last, persistent, s);
  return launch_sm<MT, KT, PL, PG, false>(p, first, last, persistent, s);
}

}  // namespace

int64_t stream_order_elems(int N, int Kd, int AT) {
  int64_t nt = (N + 15) / 16;
  int64_t units = (nt + AT - 1) / AT;
  return units * AT * 16 * (int64_t)Kd;
}

int launch_retile_stream(const bf16_t* src0, int rows0, const bf16_t* src1, int rows1, const bf16_t* src2, int rows2,
                         int mode, int AT, int KS, int Kd, bf16_t* dst, hipStream_t s) {
  SSD_CHECK_ARG(KS >= 1 && Kd % (256 * KS) == 0, "fused path: reduction dimension %d must be a multiple of %d", Kd, 256 * KS);
  SSD_CHECK_ARG(mode == 0 || (AT == 4 && rows0 == rows1 && rows0 % 32 == 0), "gate/up interleave needs AT = 4 and equal heights");
  int64_t nt = mode == 0 ? ((int64_t)rows0 + rows1 + rows2 + 15) / 16 : (int64_t)2 * (rows0 / 16);
  int n_units = (int)((nt + AT - 1) / AT) * KS;
  int64_t total = (int64_t)(n_units / KS) * AT * (Kd / 32) * 64;
  retile_stream_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(src0, rows0, src1, rows1, src2, rows2, mode, AT, KS, Kd,
                                                                       n_units, dst);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

// A stream-order weight buffer from bf16 to fp16: same layout, every element converted (8 per thread)
__global__ void bf16_to_f16_kernel(const bf16_t* src, bf16_t* dst, int64_t n8) {   // dst may be src
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n8) return;
  Bf8 v, o;
  v.w = *(const u32x4*)(src + i * 8);
#pragma unroll
  for (int e = 0; e < 8; ++e) o.u[e] = to_f16(bf16_to_f32(v.u[e]));
  *(u32x4*)(dst + i * 8) = o.w;
}

int launch_bf16_to_f16(const bf16_t* src, bf16_t* dst, int64_t n, hipStream_t s) {
  SSD_CHECK_ARG(n % 8 == 0, "bf16_to_f16: element count %lld is not a multiple of 8", (long long)n);
  if (n == 0) return SSD_OK;
  bf16_to_f16_kernel<<<(unsigned)((n / 8 + 255) / 256), 256, 0, s>>>(src, dst, n / 8);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

int launch_copy_kv_fused(bf16_t* trunk_k, bf16_t* trunk_vt, const bf16_t* src_k, const bf16_t* src_v, int B, int len, int Hkv,
                         int vt_stride, const int32_t* pages, int page_stride, hipStream_t s) {
  int64_t total = (int64_t)B * len * Hkv * 64;
  if (total == 0) return SSD_OK;
  copy_kv_fused_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(trunk_k, trunk_vt, src_k, src_v, len, Hkv, vt_stride, total, pages, page_stride);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

bool fused_supported(const Dims& d, int max_rows) {
  return d.dtype == SSD_BF16 && d.head_dim == 64 && max_rows <= kFusedMaxRows && d.d_model % 512 == 0 &&
         d.q_dim() % 512 == 0 && d.d_ffn % 512 == 0 && d.kv_dim() % 16 == 0 && d.vocab % 16 == 0 &&
         d.n_q_heads % d.n_kv_heads == 0 && 16 % (d.n_q_heads / d.n_kv_heads) == 0;
}

int fused_init_barrier(unsigned* bar, unsigned epoch0, int nwg) {
  static_assert(kBarEpochWord < kFusedSyncWords && kBarFlags + kBarGroups <= kFusedSyncWords, "barrier words");
  std::vector<unsigned> w(kFusedSyncWords + 64, 0u);
  for (int g = 0; g < kBarGroups; ++g) {
    w[32 * g] = epoch0 * (unsigned)(nwg / kBarGroups);   // arrivals so far, modulo 2^32 like the counter itself
    w[kBarFlags + g] = epoch0;
  }
  w[kBarEpochWord] = epoch0;
  SSD_HIP(hipMemcpy(bar, w.data(), w.size() * sizeof(unsigned), hipMemcpyHostToDevice));
  return SSD_OK;
}

int fused_init_group_flags(unsigned* flags, int n_layers, unsigned epoch0) {
  std::vector<unsigned> w((size_t)n_layers * 128, epoch0);
  SSD_HIP(hipMemcpy(flags, w.data(), w.size() * sizeof(unsigned), hipMemcpyHostToDevice));
  return SSD_OK;
}

int fused_grid_size(int* out) {
  int dev = 0;
  SSD_HIP(hipGetDevice(&dev));
  int cus = 0;
  SSD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  cus -= cus % 8;
  if (cus < 8) {
    set_error("fused path needs at least 8 compute units");
    return SSD_EINVAL;
  }
  *out = cus;
  return SSD_OK;
}

// The plane configurations that are compiled in: bit i of the mask set = that tensor travels as ONE plane
// (bit 0 xn, 1 att, 2 act, 3 q, 4 p).  The default, and the only one with a paged trunk: xn, att, act one fp16 plane,
// q and p two bf16 planes (what the second plane of the former costs a 24-row step of the 1B shape: 4 %; 11 % at 48 rows
// and 8192 keys; the error against a float64 reference goes from 1.1e-3 to 2.6e-3).
constexpr int kFusedDefaultPlanes = 7;
#ifndef SSD_FUSED_PLANE_MASKS
#define SSD_FUSED_PLANE_MASKS X(0) X(7)
#endif
template <int MASK>
using PlanesOf = Planes<(MASK & 1) ? 1 : 2, (MASK & 2) ? 1 : 2, (MASK & 4) ? 1 : 2, (MASK & 8) ? 1 : 2, (MASK & 16) ? 1 : 2>;

// The instance of a model width: with two planes gate/up streams through the ring, which takes 4 k-tiles as it takes 8.
template <class PL> constexpr int kt_of(int kt) { return PL::xn == 2 && kt == 4 ? 8 : kt; }

template <int KT, class PL, bool PG>
int check_residency_kt(int nwg, int cus) {
  SSD_TRY((check_residency_mt<1, KT, PL, PG>(nwg, cus)));
  SSD_TRY((check_residency_mt<2, KT, PL, PG>(nwg, cus)));
  return check_residency_mt<3, KT, PL, PG>(nwg, cus);
}
template <class PL, bool PG>
int check_residency_pl(int nwg, int cus, int kt) {
  if (kt == 2) return check_residency_kt<2, PL, PG>(nwg, cus);
  if (kt == 4) return check_residency_kt<kt_of<PL>(4), PL, PG>(nwg, cus);
  return check_residency_kt<8, PL, PG>(nwg, cus);
}

template <int ATW, int EPI, int FT, int RT, int WN, int G, int NB, int TH>
int launch_wide_block_of(const FusedParams& p, const FusedGemm& g, const bf16_t* bsrc, const WideEpi& e, hipStream_t s) {
  constexpr int kLds = (NB * G * (FT + RT) + (G - 1) * FT * RT) * 1024 + kFusedPromptRows * 4;
  static_assert(kLds <= 160 * 1024, "LDS of a block");
  static const hipError_t configured = hipFuncSetAttribute((const void*)wide_block_kernel<ATW, EPI, FT, RT, WN, G, NB, TH>,
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  SSD_HIP(configured);
  SSD_CHECK_ARG(wide_k_tiles(g) % (2 * e.S * G) == 0 && (ATW == 2 || ATW == 4) && p.M <= kFusedPromptRows && p.row_tiles * 16 >= p.M,
                "wide pass: layer does not cut into blocks");
  wide_block_kernel<ATW, EPI, FT, RT, WN, G, NB, TH><<<p.nwg, TH, kLds, s>>>(p, g, bsrc, e);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

template <int EPI> constexpr int kBlocksOf = EPI == FE_LOGITS ? kNumWideBlocks : EPI == FE_SWIGLU ? kGateUpBlocks : kLayerBlocks;
// The blocks a linear layer of the pass is cut into
template <int ATW, int EPI>
WideChoice wide_choice(const FusedParams& p, const FusedGemm& g) {
  return choose_wide_block(g.n_units / g.KS * ATW, wide_k_tiles(g), p.M, p.nwg, kBlocksOf<EPI>, kFusedWideSlices,
                           EPI == FE_PART ? p.fix_stride : 0, p.d);
}

// One linear layer of a wide pass in the blocks chosen for it; e.S = the k-slices (PART).  Four wavefronts where their share of a block
// fits their registers, eight for more (and for 8 x 8 and 8 x 12: 25.2 against 26.1 and 22.5 against 22.6 us); buffers: five or six are as
// good as more (96 rows of gate/up 18.0 us with six, 18.3 with eight, 20 with sixteen).  Two groups of wavefronts where a block is small and
// its steps many: qkv of 96 rows 10.3 us in blocks of 4 x 2, 11.3 with one; gate/up of 96 rows (4 x 6) 19.6, 18.4 with one.
template <int ATW, int EPI>
int launch_wide_block(const WideChoice& c, const FusedParams& p, const FusedGemm& g, const bf16_t* bsrc, WideEpi& e, hipStream_t s) {
  constexpr int kBlocks = kBlocksOf<EPI>;
  constexpr bool kSlices = EPI == FE_PART;
  e.S = c.S;
  switch (c.block) {
    case 0: return launch_wide_block_of<ATW, EPI, 4, 2, 2, kSlices ? 1 : 2, 6, 256>(p, g, bsrc, e, s);
    case 1: return launch_wide_block_of<ATW, EPI, 4, 4, 2, 1, 6, 256>(p, g, bsrc, e, s);
    case 2: return launch_wide_block_of<ATW, EPI, 4, 6, 2, 1, 6, 256>(p, g, bsrc, e, s);
    case 3: return launch_wide_block_of<ATW, EPI, 4, 8, 2, 1, 6, 256>(p, g, bsrc, e, s);
    case 4: return launch_wide_block_of<ATW, EPI, 8, 6, 2, 1, 6, 256>(p, g, bsrc, e, s);
    case 5: return launch_wide_block_of<ATW, EPI, 8, 8, 4, 1, 5, 512>(p, g, bsrc, e, s);
    case 6: return launch_wide_block_of<ATW, EPI, 8, 12, 4, 1, 5, 512>(p, g, bsrc, e, s);
    case 7: return launch_wide_block_of<ATW, EPI, 16, 8, 2, 1, 5, 512>(p, g, bsrc, e, s);
    default: break;
  }
  if constexpr (kBlocks > 8) {
    if (c.block == 8) return launch_wide_block_of<ATW, EPI, 16, 12, 2, 1, 5, 256>(p, g, bsrc, e, s);
    if (c.block == 9) return launch_wide_block_of<ATW, EPI, 16, 16, 2, 1, 4, 512>(p, g, bsrc, e, s);
  }
  if constexpr (kBlocks > 10) return launch_wide_block_of<ATW, EPI, 16, 6, 4, 1, 5, 256>(p, g, bsrc, e, s);
  return SSD_EINVAL;
}

template <int ATW, int EPI, int D, int MTG>
int launch_wide_few_of(const FusedParams& p, const FusedGemm& g, const bf16_t* bsrc, const WideEpi& e, hipStream_t s) {
  SSD_CHECK_ARG(p.M <= kFewRows && p.row_tiles == kFusedWideRows / 16 && wide_k_tiles(g) % (kWideWaves * e.S * D) == 0 &&
                    (ATW == 4 || g.n_units / g.KS % 2 == 0), "wide pass: layer does not cut into sets");
  wide_few_kernel<ATW, EPI, D, MTG><<<p.nwg, kWideThreads, kWideWaves * 4 * MTG * 1024, s>>>(p, g, bsrc, e);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}
template <int EPI, int MTG>
int launch_wide_few(const FewChoice& c, const FusedParams& p, const FusedGemm& g, const bf16_t* bsrc, const WideEpi& e, hipStream_t s) {
  constexpr int ATW = EPI == FE_SWIGLU ? 4 : 2;
  return c.depth == 8 ? launch_wide_few_of<ATW, EPI, 8, MTG>(p, g, bsrc, e, s) : launch_wide_few_of<ATW, EPI, 4, MTG>(p, g, bsrc, e, s);
}

// How the layers of a pass are cut (the layers of a model have one shape: once per pass; 0.2 us of the host per layer, and passes of narrow
// models wait for the host), and one of them launched; e.S = the k-slices (o and down).
struct WideCut { WideChoice block; FewChoice few; };
template <int EPI>
WideCut wide_cut(const FusedParams& p, const FusedGemm& g) {
  constexpr int ATW = EPI == FE_SWIGLU ? 4 : 2;
  constexpr FewLayer kLayer = EPI == FE_SWIGLU ? FEW_GATE_UP : EPI == FE_PART ? FEW_PART : FEW_QKV;
  return {wide_choice<ATW, EPI>(p, g), choose_wide_few(kLayer, g.n_units / g.KS * ATW, wide_k_tiles(g), p.M, p.nwg, kFusedWideSlices, p.fix_stride)};
}
template <int EPI>
int launch_wide_layer(const WideCut& c, const FusedParams& p, const FusedGemm& g, const bf16_t* bsrc, WideEpi& e, hipStream_t s) {
  if (c.few.depth == 0) return launch_wide_block<EPI == FE_SWIGLU ? 4 : 2, EPI>(c.block, p, g, bsrc, e, s);
  e.S = c.few.S;
  if constexpr (EPI != FE_SWIGLU)
    if (c.few.mtg == 1) return launch_wide_few<EPI, 1>(c.few, p, g, bsrc, e, s);
  if constexpr (EPI != FE_QKV) return c.few.mtg == 2 ? launch_wide_few<EPI, 2>(c.few, p, g, bsrc, e, s) : launch_wide_few<EPI, 3>(c.few, p, g, bsrc, e, s);
  return SSD_EINVAL;
}

// The attention units of a pass, p.NQ query tiles each (the host chooses them together with the key splits)
template <class PL, bool PG, int NQ>
int launch_wide_attn_nq(const FusedParams& p, const FusedLayer& L, int ph, hipStream_t s) {
  static const hipError_t configured = hipFuncSetAttribute((const void*)wide_attn_kernel<PL::q, PL::p, NQ, PG>,
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMultiLdsBytes);
  SSD_HIP(configured);
  wide_attn_kernel<PL::q, PL::p, NQ, PG><<<p.n_attn_units, kFusedThreads, kMultiLdsBytes, s>>>(p, L.trunk_k, L.trunk_vt, L.suffix_k, L.suffix_v, ph);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}
template <class PL, bool PG>
int launch_wide_attn(const FusedParams& p, const FusedLayer& L, int ph, hipStream_t s) {
  static_assert(kMultiQ == 3, "an instance per number of query tiles");
  if (p.NQ == 1) return launch_wide_attn_nq<PL, PG, 1>(p, L, ph, s);
  if (p.NQ == 2) return launch_wide_attn_nq<PL, PG, 2>(p, L, ph, s);
  return launch_wide_attn_nq<PL, PG, 3>(p, L, ph, s);
}

// LM head.  Up to 96 rows it is a stream of weights, each read once, which goes faster straight into registers and past the caches
// (96 rows 109 us, 117 in blocks of 256 features x 96 rows).
int launch_wide_logits(const FusedParams& p, WideEpi& e, hipStream_t s) {
  if (p.M > kTileRows) return launch_wide_block<4, FE_LOGITS>(wide_choice<4, FE_LOGITS>(p, p.lm), p, p.lm, p.xn, e, s);
  SSD_CHECK_ARG(p.lm.KS == 1 && wide_k_tiles(p.lm) % kTileRing == 0, "wide pass: the LM head does not cut into tiles");
  constexpr int kLds = 2 * kTileStage * kTileRows / 16 * 1024;
  wide_tile_kernel<<<p.nwg, kWideThreads, kLds, s>>>(p, p.lm, p.xn, e);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

template <bool EMBED>
int launch_wide_resid_e(const FusedParams& p, const float* part, int S, const bf16_t* gain, float* hidden, int ph, bool pieces, hipStream_t s) {
  const unsigned grid = pieces ? wide_resid_grid((unsigned)p.M) : (unsigned)p.M;
  if (pieces && p.prof) wide_resid_kernel<EMBED, true, true><<<grid, kWideThreads, 0, s>>>(p, part, S, gain, hidden, ph);
  else if (pieces) wide_resid_kernel<EMBED, true, false><<<grid, kWideThreads, 0, s>>>(p, part, S, gain, hidden, ph);
  else if (p.prof) wide_resid_kernel<EMBED, false, true><<<grid, kWideThreads, 0, s>>>(p, part, S, gain, hidden, ph);
  else wide_resid_kernel<EMBED, false, false><<<grid, kWideThreads, 0, s>>>(p, part, S, gain, hidden, ph);
  SSD_HIP(hipGetLastError());
  return SSD_OK;
}

// Single rows send every 128-byte line of the operand to memory in eight parts, one from each die; pieces of 8 rows send it whole, but
// leave the few rows of a small launch on few dies, whose L2s then take longer to write back than eight would.  Whole passes, us, single
// rows / pieces: 8 layers of the 1B shape 32 rows 498 / 497, 96 rows 589 / 586, 128 rows 600 / 596, 192 rows 744 / 737, 384 rows 989 / 977, prompts of
// 450 tokens 932 / 921, 1020 tokens 1445 / 1435; of width 1024 32 rows 337 / 336, 96 rows 374 / 374, 160 rows 405 / 398, 384 rows 547 / 538; of
// width 512 32 rows 255 / 257, 96 rows 303 / 305, 128 rows 304 / 297, 256 rows 326 / 316, 384 rows 350 / 343.
int launch_wide_resid(const FusedParams& p, bool embed, const float* part, int S, const bf16_t* gain, float* hidden, int ph, hipStream_t s) {
  const bool pieces = p.M >= 128;
  return embed ? launch_wide_resid_e<true>(p, part, S, gain, hidden, ph, pieces, s)
               : launch_wide_resid_e<false>(p, part, S, gain, hidden, ph, pieces, s);
}

// One wide pass: phases [first, last] as one launch each (two for o and down).  layers_host: the pass's layer table in host
// memory.
template <class PL, bool PG>
int launch_wide_pl(const FusedParams& p, const FusedLayer* layers_host, int first, int last, hipStream_t s) {
  const int lm_phase = fused_last_phase(p.L);
  const FusedLayer& any = layers_host[0];
  const WideCut cut_qkv = wide_cut<FE_QKV>(p, any.qkv), cut_o = wide_cut<FE_PART>(p, any.o), cut_gu = wide_cut<FE_SWIGLU>(p, any.gu),
                cut_down = wide_cut<FE_PART>(p, any.down);
  for (int ph = first; ph <= last; ++ph) {
    if (ph == 0) {
      SSD_TRY(launch_wide_resid(p, true, nullptr, 0, layers_host[0].attn_norm, nullptr, ph, s));
      continue;
    }
    WideEpi e{};
    e.ph = ph;
    e.S = 1;
    if (ph == lm_phase) {
      if (p.logits) {
        e.out = p.logits; e.ld = p.logits_ld;
        SSD_TRY(launch_wide_logits(p, e, s));
      }
      continue;
    }
    const int l = (ph - 1) / 6, sub = (ph - 1) % 6;
    const FusedLayer& L = layers_host[l];
    if (sub == 0) {
      e.out = p.qkv; e.ld = p.qkvd;
      SSD_TRY(launch_wide_layer<FE_QKV>(cut_qkv, p, L.qkv, p.xn, e, s));
    } else if (sub == 3 || sub == 5) {
      e.out = p.fix_buf; e.ld = p.d;
      SSD_TRY(launch_wide_layer<FE_PART>(sub == 3 ? cut_o : cut_down, p, sub == 3 ? L.o : L.down, sub == 3 ? p.att : p.act, e, s));
      const bool fin = sub == 5 && l + 1 == p.L;
      const bf16_t* gain = sub == 3 ? L.mlp_norm : (fin ? p.final_norm : layers_host[l + 1].attn_norm);
      SSD_TRY(launch_wide_resid(p, false, p.fix_buf, e.S, gain, fin ? p.hidden : nullptr, ph, s));
    } else if (sub == 4) {
      e.act_out = p.act;
      SSD_TRY(launch_wide_layer<FE_SWIGLU>(cut_gu, p, L.gu, p.xn, e, s));
    } else if (sub == 1) {
      // (a pass without outputs ends where the last layer's keys and values are stored: no attention there, also where the units would stage
      // the keys.  Three prompts of 100 tokens, 2 layers of the 1B shape: 139 us, 155 with the last attention, 147 with all keys appended first)
      if (p.appended || ph == last) {
        wide_append_kernel<PG><<<(p.M * p.Hkv * 8 + 255) / 256, 256, 0, s>>>(p, L.trunk_k, L.trunk_vt);
        SSD_HIP(hipGetLastError());
        if (ph == last) continue;
      }
      SSD_TRY((launch_wide_attn<PL, PG>(p, L, ph, s)));
    } else if (p.NS > 1) {                           // (no merge phase with one key split)
      wide_merge_kernel<<<p.n_pair_units, kFusedThreads, 0, s>>>(p, ph);
      SSD_HIP(hipGetLastError());
    }
  }
  return SSD_OK;
}

template <int KT, class PL, bool PG>
int launch_kt(const FusedParams& p, int first, int last, int persistent, hipStream_t s) {
  const int mt = (p.M + 15) / 16;
  if (mt == 1) return launch_mt<1, KT, PL, PG>(p, first, last, persistent, s);
  if (mt == 2) return launch_mt<2, KT, PL, PG>(p, first, last, persistent, s);
  return launch_mt<3, KT, PL, PG>(p, first, last, persistent, s);
}
template <class PL, bool PG>
int launch_pl(const FusedParams& p, int first, int last, int persistent, hipStream_t s) {
  if (p.kt == 2) return launch_kt<2, PL, PG>(p, first, last, persistent, s);
  if (p.kt == 4) return launch_kt<kt_of<PL>(4), PL, PG>(p, first, last, persistent, s);
  return launch_kt<8, PL, PG>(p, first, last, persistent, s);
}

bool fused_planes_supported(int mask) {
#define X(m) if (mask == (m)) return true;
  SSD_FUSED_PLANE_MASKS
#undef X
  return false;
}

int fused_check_residency(int nwg, int kt, int planes, int paged) {
  int dev = 0, cus = 0;
  SSD_HIP(hipGetDevice(&dev));
  SSD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  if (paged) {
    SSD_CHECK_ARG(planes == kFusedDefaultPlanes, "a paged trunk takes the default activation planes only");
    return check_residency_pl<PlanesOf<kFusedDefaultPlanes>, true>(nwg, cus, kt);
  }
#define X(m) if (planes == (m)) return check_residency_pl<PlanesOf<(m)>, false>(nwg, cus, kt);
  SSD_FUSED_PLANE_MASKS
#undef X
  set_error("fused pass: plane configuration %d is not compiled in", planes);
  return SSD_EINVAL;
}

// Wide passes carry xn, att and act as ONE fp16 plane each (2.5e-3 between hidden states and a float64 reference through
// 16 layers, measured); the attention unit's queries and probabilities keep two bf16 planes unless both of their bits
// are set in p.planes.
int launch_fused_wide(const FusedParams& p, const FusedLayer* layers_host, int first, int last, hipStream_t s) {
  const int max_rows = p.is_branch || p.logits || p.hidden ? kFusedWideRows : kFusedPromptRows;
  SSD_CHECK_ARG(p.M >= 1 && p.M <= max_rows, "wide fused pass of %d rows (1..%d supported)", p.M, max_rows);
  SSD_CHECK_ARG(p.row_tiles == (p.M > kFusedWideRows ? kFusedPromptRows : kFusedWideRows) / 16, "row tiles %d of an operand plane", p.row_tiles);
  SSD_CHECK_ARG(p.nwg >= 8 && p.nwg % 8 == 0, "fused grid of %d workgroups must be a multiple of 8", p.nwg);
  SSD_CHECK_ARG(p.KPU >= 32 && p.KPU % 32 == 0 && p.NS >= 1 && p.QT >= 1 && (p.SL == 8 || p.SL == 16) && 16 % p.G == 0 &&
                    (16 / p.G) * p.SL <= 64,
                "bad attention split");
  SSD_CHECK_ARG(p.NQ >= 1 && p.NQ <= kMultiQ && p.n_attn_units == p.B * p.Hkv * ((p.QT + p.NQ - 1) / p.NQ) * p.NS, "bad attention units");
  SSD_CHECK_ARG(p.M <= p.fix_stride, "no room for the partial sums of %d rows", p.M);
  SSD_CHECK_ARG(!p.is_branch || !p.appended, "branch rows keep their own keys");
  SSD_CHECK_ARG(p.is_branch || p.appended || p.R <= kFusedWideFreshKeys, "an extend of %d tokens must append its keys first", p.R);
  // What the attention and append kernels index with: trunk slots (a row's own included), the lane that holds a wavefront's
  // n-th page, private slots.  The units' LDS extents follow from NQ, G, SL and R above.
  static_assert(kMultiQ * 64 <= kMultiFreshKeys, "fresh keys of a unit of branch rows");
  SSD_CHECK_ARG(p.tv_ub >= 0 && p.tv_ub + (p.is_branch ? 0 : p.R) <= p.vt_stride, "trunk positions up to %d + %d, room for %d", p.tv_ub, p.R, p.vt_stride);
  SSD_CHECK_ARG(!p.pages || (p.page_stride * 32 == p.vt_stride && p.KPU <= 64 * kFusedWaves * 32), "%d keys per unit in a paged trunk", p.KPU);
  SSD_CHECK_ARG(!p.is_branch || (p.suffix_len >= 1 && p.suffix_len <= p.suffix_cap && p.suffix_cap <= p.SL), "private slot %d of %d", p.suffix_len, p.suffix_cap);
  SSD_CHECK_ARG(first >= 0 && last <= fused_last_phase(p.L) && first <= last && layers_host, "bad phase range");
  if (p.pages) {
    SSD_CHECK_ARG((p.planes & 24) != 24, "a paged trunk takes the default planes of the attention unit only");
    return launch_wide_pl<Planes<1, 1, 1, 2, 2>, true>(p, layers_host, first, last, s);
  }
  if ((p.planes & 24) == 24) return launch_wide_pl<Planes<1, 1, 1, 1, 1>, false>(p, layers_host, first, last, s);
  return launch_wide_pl<Planes<1, 1, 1, 2, 2>, false>(p, layers_host, first, last, s);
}

// Shapes the wide pass takes: every layer's stream-order layout must cut into sets of 4 feature tiles, and its reduction dimension into
// eight slices of an even number of k-tiles (a step of a block is one k-tile and its loop takes two).
bool fused_wide_gemm_ok(const FusedGemm& g, int at) {
  if (g.KS * g.KTW % 2) return false;                        // (8 KS KTW k-tiles)
  if (at == 4) return g.KS == 1;
  return at == 2 && (g.n_units / g.KS) % 2 == 0;
}

int launch_fused(const FusedParams& p, int first, int last, int persistent, hipStream_t s) {
  SSD_CHECK_ARG(p.M >= 1 && p.M <= kFusedMaxRows, "fused pass of %d rows (1..%d supported)", p.M, kFusedMaxRows);
  SSD_CHECK_ARG(p.nwg >= 8 && p.nwg % 8 == 0, "fused grid of %d workgroups must be a multiple of 8", p.nwg);
  SSD_CHECK_ARG(p.KPU >= 32 && p.KPU % 32 == 0 && p.NS >= 1 && p.QT >= 1 && (p.SL == 8 || p.SL == 16) && 16 % p.G == 0 &&
                    (16 / p.G) * p.SL <= 64,
                "bad attention split");
  SSD_CHECK_ARG(first >= 0 && last <= fused_last_phase(p.L) && first <= last, "bad phase range");
  SSD_CHECK_ARG((p.kt == 2 || p.kt == 4 || p.kt == 8) && p.kt * 256 == p.d && p.lm.KTW == p.kt, "fused pass: no kernel for a width of %d", p.d);
  SSD_CHECK_ARG(p.NS <= 16 && (p.NS == 1 || p.arrivals), "fused pass: %d key splits (at most 16, with arrival counters)", p.NS);
  SSD_CHECK_ARG(p.qkv_ug == 0 || (p.qkv_flags && p.qkv_ug <= 16 && p.qkv_ug == 2 * p.G + 4 && p.Hkv <= 8 && 8 % p.Hkv == 0 &&
                                  8 * p.qkv_ug <= p.nwg && (!persistent || first == 0)),
                "fused pass: group sync does not fit this shape or phase range");
  if (p.pages) {
    SSD_CHECK_ARG(p.planes == kFusedDefaultPlanes, "a paged trunk takes the default activation planes only");
    return launch_pl<PlanesOf<kFusedDefaultPlanes>, true>(p, first, last, persistent, s);
  }
#define X(m) if (p.planes == (m)) return launch_pl<PlanesOf<(m)>, false>(p, first, last, persistent, s);
  SSD_FUSED_PLANE_MASKS
#undef X
  set_error("fused pass: plane configuration %d is not compiled in", p.planes);
  return SSD_EINVAL;
}

}  // namespace ssd
