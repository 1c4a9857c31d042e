// What the two bf16 attention kernels share: vector types, lane-group reductions, softmax constants, the output store.
#pragma once

#include <type_traits>

#include "usv_internal.h"

namespace usv {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short short4v;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short short8v;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// Accumulators are kept four 16x16 tiles to a 16-register tuple and the MFMAs work on quarter q of it:
// with one allocation unit per tuple the compiler updates the accumulators in place (given 64 separate
// 4-register values it rotated them through fresh registers and copied all of them back on every tile).
__device__ __forceinline__ f32x4 quarter(const f32x16& v, int q) {
  switch (q) {
    case 0: return __builtin_shufflevector(v, v, 0, 1, 2, 3);
    case 1: return __builtin_shufflevector(v, v, 4, 5, 6, 7);
    case 2: return __builtin_shufflevector(v, v, 8, 9, 10, 11);
    default: return __builtin_shufflevector(v, v, 12, 13, 14, 15);
  }
}
__device__ __forceinline__ void set_quarter(f32x16& v, int q, const f32x4& c) {
  const f32x16 w = __builtin_shufflevector(c, c, 0, 1, 2, 3, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1);
  switch (q) {
    case 0: v = __builtin_shufflevector(v, w, 16, 17, 18, 19, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15); break;
    case 1: v = __builtin_shufflevector(v, w, 0, 1, 2, 3, 16, 17, 18, 19, 8, 9, 10, 11, 12, 13, 14, 15); break;
    case 2: v = __builtin_shufflevector(v, w, 0, 1, 2, 3, 4, 5, 6, 7, 16, 17, 18, 19, 12, 13, 14, 15); break;
    default: v = __builtin_shufflevector(v, w, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 16, 17, 18, 19); break;
  }
}

constexpr float kRescaleSlack = 8.0f;  // log2 units
// The probabilities are computed as 2^(logit - m - p_shift): the common factor 2^-p_shift cancels in
// sum(p v) / sum(p), and it pushes every p below tau = 2^-(126 - p_shift) of the row's reference under
// the fp32 normal range, where v_exp_f32 returns an exact 0.  Zero operands keep the matrix cores'
// multipliers quiet, which matters because the chip is power-limited under this kernel (measured:
// +3 % at tau = 2^-24, +10 % on dense lists at tau = 2^-16).  The dropped mass of a row is below
// keys * tau of its largest term; the launcher picks tau so that this is at most 2^-12 (2.4e-4
// relative, against an error budget of ~2.5e-3), i.e. tau = 2^-12 / (keys of the longest list).
constexpr int kDropLog2 = 12;

// p_shift for lists of at most kmax blocks: 126 + log2(tau), kept within [64, 110]
inline float probability_shift(int kmax) {
  int bits = 0;
  while ((1LL << bits) < (long long)kmax * kBlock) ++bits;
  const int shift = 126 - kDropLog2 - bits;
  return (float)(shift < 64 ? 64 : shift > 110 ? 110 : shift);
}

__device__ __forceinline__ float4 bf16_pair(unsigned x, unsigned y) {  // four bf16, two per register
  return make_float4(__uint_as_float(x << 16), __uint_as_float(x & 0xffff0000u), __uint_as_float(y << 16),
                     __uint_as_float(y & 0xffff0000u));
}
__device__ __forceinline__ float4 load_bf16x4(const uint16_t* p) {
  // (the gates of the fused second branch: read once, so a streaming read)
  typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2;
  const u32x2 ww = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
  return bf16_pair(ww[0], ww[1]);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// v_permlane32_swap on two copies of x leaves (x of lane l % 32, x of lane l % 32 + 32) in both lanes:
// one VALU op, no LDS round trip.
__device__ __forceinline__ void both_halves(float x, float& lo, float& hi) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  lo = __uint_as_float(r[0]);
  hi = __uint_as_float(r[1]);
}

// Max of the 8 accumulator values a lane holds for one query, in 4 instructions.  One assembly block:
// v_max3 without the NaN-quieting moves the compiler adds around fmaxf (the inputs are never NaN).
__device__ __forceinline__ float max8(float a0, float a1, float a2, float a3, float b0, float b1, float b2, float b3) {
  float x, y;
  asm("v_max3_f32 %0, %2, %3, %4\n\t"
      "v_max3_f32 %1, %5, %6, %7\n\t"
      "v_max3_f32 %0, %0, %8, %9\n\t"
      "v_max_f32 %0, %0, %1"
      : "=&v"(x), "=&v"(y)
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(b0), "v"(b1), "v"(b2), "v"(b3));
  return x;
}

// The four lanes c, c + 16, c + 32, c + 48 hold the keys of one query.  v_permlane16_swap on two copies
// of x leaves (x of the even 16-lane row, x of the odd row) of each row pair in both rows, and
// v_permlane32_swap does the same for the two wave halves: two VALU ops per step, no LDS round trip.
__device__ __forceinline__ void row_pair(float x, float& even, float& odd) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  even = __uint_as_float(r[0]);
  odd = __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_over_groups(float x) {
  float a, b;
  row_pair(x, a, b);
  x = fmaxf(a, b);
  both_halves(x, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum_over_groups(float x) {
  float a, b;
  row_pair(x, a, b);
  x = a + b;
  both_halves(x, a, b);
  return a + b;
}

__device__ __forceinline__ unsigned lds_address(const void* p) {  // LDS byte address of a __shared__ pointer
  return (unsigned)(uintptr_t)p;
}

// Four channels of one output row.  stream (the launcher's choice, the same for every workgroup): streaming stores.  The
// output is not read again by the launch, and written the ordinary way its lines push K/V tiles out of the L2.
template <bool OUT_F32>
__device__ __forceinline__ void store4(void* dst, const float4& val, int stream) {
  if constexpr (OUT_F32) {
    const f32x4 vv = {val.x, val.y, val.z, val.w};
    if (stream) __builtin_nontemporal_store(vv, reinterpret_cast<f32x4*>(dst));
    else *reinterpret_cast<f32x4*>(dst) = vv;
  } else {
    bf16x4 pk;
    pk[0] = (__bf16)val.x; pk[1] = (__bf16)val.y; pk[2] = (__bf16)val.z; pk[3] = (__bf16)val.w;
    if (stream) __builtin_nontemporal_store(pk, reinterpret_cast<bf16x4*>(dst));
    else *reinterpret_cast<bf16x4*>(dst) = pk;
  }
}
// Eight channels of one output row.
template <bool OUT_F32>
__device__ __forceinline__ void store8(void* dst, const float4 (&val)[2], int stream) {
  if constexpr (OUT_F32) {
    store4<true>(dst, val[0], stream);
    store4<true>(static_cast<float*>(dst) + 4, val[1], stream);
  } else {
    bf16x8 pk;
    pk[0] = (__bf16)val[0].x; pk[1] = (__bf16)val[0].y; pk[2] = (__bf16)val[0].z; pk[3] = (__bf16)val[0].w;
    pk[4] = (__bf16)val[1].x; pk[5] = (__bf16)val[1].y; pk[6] = (__bf16)val[1].z; pk[7] = (__bf16)val[1].w;
    if (stream) __builtin_nontemporal_store(pk, reinterpret_cast<bf16x8*>(dst));
    else *reinterpret_cast<bf16x8*>(dst) = pk;
  }
}
// Streaming output stores where the L2 has something to lose: measured -1 % at the 480p shape (a head's K and V:
// 16.8 MB), -2.7 % with ragged budgets at 16384 tokens, nothing on dense lists, but +4.4 % at the 720p shape
// (38.7 MB per head: the L2 serves a quarter of the tile requests there whatever the output does, and the launch
// runs at the limit of the fabric, which ordinary stores load more evenly).
inline int stream_output(const Dims& s) { return 4LL * s.nb * kBlock * s.d <= (32LL << 20); }

// Workgroups that the chip runs together in the wide kernel; and whether a launch of long heads makes two to four such rounds, give or take a
// twenty-fourth of one.  Sweeps that are kept together end together, and what is left behind a round then runs by itself.
inline long long wide_round(const Dims& s) { return s.d == 128 ? 1024 : 1536; }
inline bool full_rounds(const Dims& s) {
  const long long round = wide_round(s), past = s.bh() * s.nb + round / 24;
  return s.nb > 640 && past >= 2 * round && past < 5 * round && 12 * (past % round) < round;
}

// Second branch folded into the store: gate_fine * attention + gate_coarse * cube-level row.
__device__ __forceinline__ void fuse4(float4& val, const float4& gf, const float4& gc, const float4& cz) {
  val.x = fmaf(gf.x, val.x, gc.x * cz.x);
  val.y = fmaf(gf.y, val.y, gc.y * cz.y);
  val.z = fmaf(gf.z, val.z, gc.z * cz.z);
  val.w = fmaf(gf.w, val.w, gc.w * cz.w);
}
// gate_off in elements.  The cube-level row is requested first: behind the gates, whose loads are awaited where they branch, it
// is one more round trip per pass (768 query blocks, 6 listed, both gates 38.7 -> 41.5 us).
__device__ __forceinline__ void fuse4(float4& val, const FuseArgs& fuse, long long coarse_off, long long gate_off) {
  const float4 cz = *reinterpret_cast<const float4*>(fuse.coarse + coarse_off);
  float4 gf = make_float4(1.f, 1.f, 1.f, 1.f), gc = gf;
  if (fuse.gate_fine) gf = load_bf16x4(fuse.gate_fine + gate_off);
  if (fuse.gate_coarse) gc = load_bf16x4(fuse.gate_coarse + gate_off);
  fuse4(val, gf, gc, cz);
}

}  // namespace
}  // namespace usv
