// Shared host/device helpers of libss (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include "ss.h"

namespace ss {

// ---------------------------------------------------------------- errors (host)
void set_error(const char* fmt, ...);
void clear_error();

#define SS_FAIL(code, ...)        \
  do {                            \
    ::ss::set_error(__VA_ARGS__); \
    return (code);                \
  } while (0)

#define SS_REQUIRE(cond, code, ...)        \
  do {                                     \
    if (!(cond)) SS_FAIL(code, __VA_ARGS__); \
  } while (0)

// Checks the launch that was just issued.
inline int check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) SS_FAIL(SS_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
  return SS_OK;
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---------------------------------------------------------------- vector types
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t uintx4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t uintx2;

// ---------------------------------------------------------------- device helpers
#define SS_DEV __device__ __forceinline__
#define SS_HD __host__ __device__ __forceinline__

// fp32 -> bf16 bits, round to nearest even (inputs are finite here).
SS_DEV uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
SS_DEV uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}
SS_DEV float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// One step of merging per-split attention results (both the merge kernel and the in-kernel merge use it, so
// that they agree bit for bit): acc <- acc*keep + v*w with the roundings fixed.
SS_DEV floatx4 merge_step(floatx4 acc, float keep, floatx4 v, float w) {
  floatx4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = __builtin_fmaf(v[i], w, acc[i] * keep);
  return r;
}

// Node 0 is the root; for i > 0 a parent outside [0,i) counts as 0 (documented clamp).
SS_DEV int clamp_parent(int p, int i) { return (i == 0) ? -1 : ((p < 0 || p >= i) ? 0 : p); }

// Tree row r of a sequence with T nodes and gamma streams -> (node, stream); stream 0 = main row.
SS_DEV void row_split(int r, int T, int gamma, int& node, int& strm) {
  if (r < T) {
    node = r;
    strm = 0;
  } else {
    node = (r - T) / gamma;
    strm = (r - T) % gamma + 1;
  }
}

// What one query row needs to decide which of the step's own keys it may attend
// (Eq. 1 / Eq. 2 with the tree mask): main key c < T is visible iff bit c of anc;
// stream key c >= T is visible iff lo <= c < hi.
struct RowVis {
  uint64_t anc;
  int lo, hi;
};
// Both alternatives are evaluated and then selected (no control flow per score).
SS_DEV bool row_sees(const RowVis& v, int c, int T) {
  const bool as_main = ((v.anc >> (c & 63)) & 1ull) != 0;
  const bool as_stream = (c >= v.lo) & (c < v.hi);
  return (c < T) ? as_main : as_stream;
}
// anc: ancestors-or-self of the row's node.
SS_DEV RowVis make_row_vis(int node, int strm, uint64_t anc, int T, int gamma, bool exclude_self) {
  RowVis v;
  v.anc = anc;
  v.lo = T + node * gamma;
  v.hi = v.lo + (strm == 0 ? 0 : (exclude_self ? strm - 1 : strm));
  return v;
}

// Ancestors-or-self of node i (bit set) in a tree of T nodes, lane i of a wavefront holding node i's clamped parent p; all
// lanes take part.  The set doubles its reach with every step: complete for nodes of at most `reach` ancestors, of the others
// it holds more than `reach`.
SS_DEV uint64_t ancestors(int i, int p, int T, int reach) {
  uint64_t bits = i < T ? 1ull << i : 1ull;
  int up = i < T && i > 0 ? p : 0;
  for (int r = 1; r <= reach; r <<= 1) {
    const uint32_t lo = __shfl((uint32_t)bits, up, 64), hi = __shfl((uint32_t)(bits >> 32), up, 64);
    bits |= ((uint64_t)hi << 32) | lo;
    up = __shfl(up, up, 64);
  }
  return bits;
}
// The same for one node per lane, any of them: walks up from it, a lane shuffle per level.
SS_DEV uint64_t ancestors_of(int node, int p) {
  uint64_t bits = 0;
  int n = node;
  for (int step = 0; step < 64 && __any(n >= 0); ++step) {
    const int up = __shfl(p, max(n, 0), 64);
    bits |= n >= 0 ? 1ull << n : 0ull;
    n = n >= 0 ? up : -1;
  }
  return bits;
}
// Maxima over a wavefront by register moves: rotations within rows of 16 lanes, then the row swaps.  A lane shuffle is a trip
// through LDS, and a maximum of 64-bit keys is twelve of them one after the other.
template <int ROR>
SS_DEV uint32_t row_ror(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x120 + ROR, 0xf, 0xf, false);
}
template <typename Max>
SS_DEV uint32_t wave_max(uint32_t v, Max max_of) {
  v = max_of(v, row_ror<8>(v));
  v = max_of(v, row_ror<4>(v));
  v = max_of(v, row_ror<2>(v));
  v = max_of(v, row_ror<1>(v));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max_of(a[0], a[1]);
  const auto c = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max_of(c[0], c[1]);
}
SS_DEV uint32_t wave_max_u32(uint32_t v) {  // known to be uniform
  return __builtin_amdgcn_readfirstlane(wave_max(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; }));
}
SS_DEV float wave_max_f32(float v) {
  return __uint_as_float(wave_max(__float_as_uint(v), [](uint32_t a, uint32_t b) { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); }));
}
// x / d for 0 <= x < 2^23, 0 < d: the rounded quotient is off by one at most.  Fewer than half the instructions of an
// integer division, in kernels that last little longer than their start.
SS_DEV int fast_div(int x, int d) {
  const int q = (int)((float)x * __builtin_amdgcn_rcpf((float)d)), r = x - q * d;
  return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}

}  // namespace ss
