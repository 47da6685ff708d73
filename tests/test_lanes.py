"""The exchanges between lanes (csrc/lanes.h) on the CPU: 64 threads stand for a wavefront, and the few instructions the header uses are
spelled out over what they hold.  Every butterfly takes the partners of __shfl_xor in the order its name says, down to the bits of a sum."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_03251_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <array>
#include <barrier>
#include <cmath>
#include <cstdint>
#include <cstring>
#define __device__
#define __forceinline__ inline
inline uint32_t __float_as_uint(float f) { uint32_t u; std::memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(uint32_t u) { float f; std::memcpy(&f, &u, 4); return f; }
inline thread_local struct { unsigned x; } threadIdx;
inline std::barrier<> wave(64);
inline uint32_t reg[2][64];
inline void put(uint32_t a, uint32_t b) { reg[0][threadIdx.x] = a; reg[1][threadIdx.x] = b; wave.arrive_and_wait(); }
template <typename T> inline T done(T v) { wave.arrive_and_wait(); return v; }
// rows of W lanes: the odd rows of the first operand change places with the even rows of the second
template <unsigned W> inline std::array<uint32_t, 2> rows_swap(uint32_t a, uint32_t b) {
  put(a, b);
  const unsigned l = threadIdx.x;
  return done(l & W ? std::array<uint32_t, 2>{reg[1][l - W], b} : std::array<uint32_t, 2>{a, reg[0][l + W]});
}
#define __builtin_amdgcn_permlane32_swap(a, b, fi, bc) rows_swap<32>(a, b)
#define __builtin_amdgcn_permlane16_swap(a, b, fi, bc) rows_swap<16>(a, b)
inline uint32_t __builtin_amdgcn_update_dpp(uint32_t, uint32_t v, int ctrl, int, int, bool) {
  put(v, 0);
  const unsigned l = threadIdx.x, row = l & ~15u, quad = l & ~3u;
  unsigned from = quad + (ctrl >> 2 * (l & 3) & 3);             // a permutation within four lanes
  if (ctrl == 0x128) from = row + ((l + 8) & 15);               // rows of 16 rotated by 8
  if (ctrl == 0x141) from = l ^ 7;                              // halves of a row mirrored
  return done(reg[0][from]);
}
"""

MAIN = r"""
#include "lanes.h"
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>
using namespace ssd;
static float in[8][64], out[64];
static double pairs_in[64], pairs_out[64];
static int bad = 0;
template <typename F> void run(F f) {
  std::vector<std::thread> t;
  for (unsigned l = 0; l < 64; ++l) t.emplace_back([=] { threadIdx.x = l; f(l); });
  for (auto& x : t) x.join();
}
static void check(const char* what, int from, int last, const void* got, const void* want, size_t n) {
  if (std::memcmp(got, want, n)) { ++bad; std::printf("%s<%d, %d> differs\n", what, from, last); }
}
template <typename T, typename Op> static void reference(T* v, int from, int last, Op op) {
  for (int o = from;; o = from > last ? o / 2 : o * 2) {
    T r[64];
    for (int l = 0; l < 64; ++l) r[l] = op(v[l], v[l ^ o]);
    std::memcpy(v, r, sizeof(r));
    if (o == last) break;
  }
}
template <int FROM, int LAST> static void sums(int tells) {
  bool told = !tells;
  for (const float* row : in) {
    float want[64], other[64];
    std::memcpy(want, row, sizeof(want));
    std::memcpy(other, row, sizeof(other));
    reference(want, FROM, LAST, [](float a, float b) { return a + b; });
    reference(other, LAST, FROM, [](float a, float b) { return a + b; });
    told = told || std::memcmp(want, other, sizeof(want));
    run([=](unsigned l) { out[l] = lanes_sum<FROM, LAST>(row[l]); });
    check("lanes_sum", FROM, LAST, out, want, sizeof(out));
    std::memcpy(want, row, sizeof(want));
    reference(want, FROM, LAST, [](float a, float b) { return fmaxf(a, b); });
    run([=](unsigned l) { out[l] = lanes_max<FROM, LAST>(row[l]); });
    check("lanes_max", FROM, LAST, out, want, sizeof(out));
  }
  if (!told) { ++bad; std::printf("sums<%d, %d>: the values tell no order\n", FROM, LAST); }
}
int main() {
  uint64_t x = 88172645463325252ull;
  auto next = [&] { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return (float)(int64_t)x / 9.3e18f * (float)(1 << (x % 19)); };
  for (auto& row : in) for (float& v : row) v = next();
  for (double& v : pairs_in) v = (double)next() * 1e-30 + (double)next();
  sums<32, 1>(1); sums<16, 1>(1); sums<4, 1>(1); sums<1, 4>(1); sums<1, 32>(1); sums<2, 32>(1); sums<4, 32>(1); sums<8, 32>(1); sums<16, 32>(1);
  sums<32, 16>(1); sums<8, 8>(0); sums<32, 32>(0);
  double want[64];
  std::memcpy(want, pairs_in, sizeof(want));
  reference(want, 32, 1, [](double a, double b) { return a + b; });
  run([](unsigned l) { pairs_out[l] = lanes_sum(pairs_in[l]); });
  check("lanes_sum of two registers", 32, 1, pairs_out, want, sizeof(want));
  // lanes_split_sum: those with the bit set keep the second value
  auto split = [&](int o, auto f) {
    float w[64];
    for (int l = 0; l < 64; ++l) { const float* v = in[l & o ? 1 : 0]; w[l] = v[l] + v[l ^ o]; }
    run(f);
    check("lanes_split_sum", o, o, out, w, sizeof(w));
  };
  split(32, [](unsigned l) { out[l] = lanes_split_sum<32>(in[0][l], in[1][l]); });
  split(16, [](unsigned l) { out[l] = lanes_split_sum<16>(in[0][l], in[1][l]); });
  split(8, [](unsigned l) { out[l] = lanes_split_sum<8>(in[0][l], in[1][l]); });
  if (!bad) std::puts("ok");
  return bad != 0;
}
"""


def test_the_lanes_meet_in_the_order_that_is_asked_for(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "lanes.cpp").write_text(MAIN)
    exe = tmp_path / "lanes"
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-ffp-contract=off", "-I", str(tmp_path), "-I", CSRC, "-o", str(exe), str(tmp_path / "lanes.cpp")],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
