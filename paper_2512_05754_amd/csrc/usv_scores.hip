// Stage 1: pooled block scores (coarse stage of the coarse-to-fine sparse attention,
// paper Sections 2.2 and 3.2).  Two kernels:
//   pool_means   HBM-bound: reads Q and K once with 16-byte coalesced loads, reduces each
//                64-token cube to its fp32 mean over the valid tokens.
//   score_gemm   S = Qm Km^T / sqrt(d) per head to fp32 accuracy: operands in three bf16 parts each, on the
//                bf16 matrix cores (usv_attn_f32.hip says how; where a split does not carry the operands, fp32 ones).
#include "usv_split.h"

namespace usv {
namespace {

constexpr int kPoolThreads = 256;

template <typename T>
struct Vec16;  // 16 bytes of T
template <>
struct Vec16<float> {
  static constexpr int kElems = 4;
  __device__ static void load(const float* p, float (&out)[4]) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
  }
};
template <>
struct Vec16<uint16_t> {  // bf16 bit patterns
  static constexpr int kElems = 8;
  __device__ static void load(const uint16_t* p, float (&out)[8]) {
    // streaming read: nothing in this kernel touches a row twice (2.5 us of 50 at the 480p shape)
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u4;
    const u4 vv = __builtin_nontemporal_load(reinterpret_cast<const u4*>(p));
    const uint4 v = make_uint4(vv[0], vv[1], vv[2], vv[3]);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

// grid = (B*Hh*nb, 2); blockIdx.y selects Q (0) or K (1).  One workgroup per cube.
// RASTER: the tensors are in raster token order; row r of cube i is token ras.order[64 i + r].
template <typename T, int D, bool RASTER = false>
__global__ __launch_bounds__(kPoolThreads) void pool_means(const T* __restrict__ q, const T* __restrict__ k,
                                                           float* __restrict__ ws, int nb, int Nv,
                                                           long long mean_elems_per_tensor, RasterArgs ras = RasterArgs{}) {
  constexpr int VEC = Vec16<T>::kElems;
  constexpr int LPR = D / VEC;              // lanes per token row
  constexpr int RPI = kPoolThreads / LPR;   // rows per iteration
  constexpr int ITERS = kBlock / RPI;
  __shared__ float part[RPI][D + 4];

  const long long blk = blockIdx.x;         // (b*Hh + h) * nb + i
  const int i = (int)(blk % nb);
  const T* src = (blockIdx.y == 0 ? q : k) + blk * (long long)kBlock * D;
  const unsigned char* rbase = nullptr;
  if constexpr (RASTER) {
    const long long bh = blk / nb, b = bh / ras.Hh, h = bh - b * ras.Hh;
    rbase = reinterpret_cast<const unsigned char*>(blockIdx.y == 0 ? q : k) + b * ras.batch + h * ras.head;
  }
  float* dst = ws + (long long)blockIdx.y * mean_elems_per_tensor + blk * D;
  int nvalid = min(kBlock, max(0, Nv - i * kBlock));
  if constexpr (RASTER)
    if (ras.block_valid) nvalid = min(kBlock, max(0, ras.block_valid[i]));

  const int tid = threadIdx.x;
  const int r0 = tid / LPR, c0 = (tid % LPR) * VEC;
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int r = r0 + it * RPI;
    if (r < nvalid) {
      float x[VEC];
      if constexpr (RASTER)
        Vec16<T>::load(reinterpret_cast<const T*>(rbase + (long long)ras.order[i * kBlock + r] * ras.tok) + c0, x);
      else
        Vec16<T>::load(src + (long long)r * D + c0, x);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += x[e];
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) part[r0][c0 + e] = acc[e];
  __syncthreads();
  if (tid < D) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < RPI; ++r) s += part[r][tid];
    // a cube with no valid token has no mean; its scores are overwritten with -inf later
    dst[tid] = nvalid > 0 ? s / (float)nvalid : 0.f;
  }
}

// S[bh, i, j] = sum_c Qm[bh,i,c] Km[bh,j,c] * rsqrt_d.  64x64 output tile per workgroup, one 32x32 quadrant per wave.
//
// A tile with fp32 operands on the fp32 matrix cores (v_mfma_f32_32x32x2_f32): the pooled means are staged in LDS
// 64 channels at a time.  An MFMA step contracts 2 channels, one per 32-lane half; which channels a
// step takes is free as long as both operands agree, so half g takes channels 32 g + t at step t
// and every lane reads its operands as contiguous 16-byte pieces.
// For heads below 512 blocks (the launcher says why), and for operands that three bf16 parts do not carry: infinities, and values of which a lower
// part or a part's product runs out of exponent.
constexpr int kTileLd = 64 + 4;  // row stride in floats: 16-byte reads of 32 consecutive rows spread over the banks
template <int D, typename Put, typename Ahead>  // put(p): stages pass p; ahead(p): what may be asked for while it is multiplied
__device__ __forceinline__ void fp32_tile(float* As, float* Bs, Put put, Ahead ahead, float* __restrict__ out, int i0, int j0, int nb, int nb_valid,
                                          float rsqrt_d) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;  // this wave's quadrant
  const int r = lane & 31, g = lane >> 5;
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
  for (int p = 0; p < D / 64; ++p) {
    if (p) __syncthreads();
    put(p);
    __syncthreads();
    ahead(p);
    const float* ap = As + (wi + r) * kTileLd + 32 * g;
    const float* bp = Bs + (wj + r) * kTileLd + 32 * g;
#pragma unroll
    for (int t = 0; t < 32; t += 4) {
      const float4 a = *reinterpret_cast<const float4*>(ap + t);
      const float4 b = *reinterpret_cast<const float4*>(bp + t);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
    }
  }
  // accumulator register e of lane (r, g): row wi + 8 (e/4) + 4 g + (e%4), column wj + r
  const int j = j0 + wj + r;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = i0 + wi + 8 * (e >> 2) + 4 * g + (e & 3);
    if (i < nb && j < nb) out[(long long)i * nb + j] = (i < nb_valid && j < nb_valid) ? acc[e] * rsqrt_d : -INFINITY;
  }
}

// The products of three bf16 parts on v_mfma_f32_16x16x32_bf16 (lane = (c, G): rows / columns c of the operands, channels 8 G .. + 8), the
// leading one and the five small ones in sums of their own; parts staged in LDS as planes, 64 channels at a time.
// Six products at sixteen times the rate of the fp32 matrix pipe, which the fp32 form was bound by (5.8 of its 14 us at
// 12 x 512 x 512, 110 of 200 us at 40 x 1182 x 1182).  What is left is the chain of load, split, barrier and product, and the store.
// Operands below 2^59 that are 0 or not below 2^-50 (2^-100 beside larger ones).  Below 2^59 no sum of 128 products overflows
// (beyond, the leading and the small sums could do so with opposite signs, and a leading part rounded up could where the value does not).  A value
// from 2^-100 on is its three parts exactly, each of which is 0 or at least the value's last bit; what is lost of a product is what falls below
// 2^-126.  From 2^-50 on only the product of two second parts can, which is 2^-26 of the leading one.  A smaller value (of a channel that is nearly
// dead) may stand beside larger ones, as long as every group of eight channels has one from 2^-40 on: all that a score's products lose there is
// below 2^-116, which is less than its fp32 rounding if its terms add up to 2^-92.
// The look at the operands comes ahead of the products, with the means of all passes requested at once for it.  (Behind them, a tile that fp32
// operands were taken for was multiplied twice.)  Stage 1, look behind / ahead: 40 x 1182 x 1182 391 / 382 us, 12 x 512 x 512 44.7 / 44.8, d = 64 201.6 /
// 203.8, 27.3 / 27.2; one channel nearly dead 525 / 391, 52.5 / 45.2, 265 / 206, 30.9 / 27.3; eight adjacent ones, which takes fp32 operands (from the registers they
// were fetched into; fetched again 469, 50.4), 526 / 449, 53.4 / 48.5; fp32 operands alone 421, 46.9.
constexpr float kScoreMost = 0x1p59f;
constexpr unsigned below(int e) { return 2u * ((unsigned)(127 + e) << 23) - 1u; }  // twice the bits of 2^e less 1
template <int D>
__global__ __launch_bounds__(256, 3) void score_gemm(const float* __restrict__ qm, const float* __restrict__ km,
                                                  float* __restrict__ scores, int nb, int nb_valid,
                                                  float rsqrt_d, int fp32) {
  constexpr int KC = 64, P = D / KC, kPlane = 64 * KC * 2;  // channels per pass, passes; bytes of one part of 64 rows
  static_assert(2 * 64 * kTileLd * 4 <= 6 * kPlane, "the fp32 tile's operands overlay the planes");
  __shared__ __attribute__((aligned(16))) unsigned char smem[6 * kPlane];  // three planes of Q, three of K
  __shared__ int refused[4];  // per wave: operands that parts do not carry
  const int bh = blockIdx.z;
  const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  const float* qbase = qm + (long long)bh * nb * D;
  const float* kbase = km + (long long)bh * nb * D;
  float* out = scores + (long long)bh * nb * nb;
  float* const As = reinterpret_cast<float*>(smem);
  float* const Bs = As + 64 * kTileLd;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (fp32) {  // (the launcher's choice, the same for every workgroup)
    // each thread stages 4 + 4 float4 per pass; the next pass's loads are issued before this pass's MFMAs
    float4 ra[4], rb[4];
    auto fetch = [&](int p) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = tid + u * 256, row = e / 16, c = 64 * p + (e % 16) * 4;
        ra[u] = rb[u] = make_float4(0.f, 0.f, 0.f, 0.f);  // zero rows beyond nb
        if (i0 + row < nb) ra[u] = *reinterpret_cast<const float4*>(qbase + (long long)(i0 + row) * D + c);
        if (j0 + row < nb) rb[u] = *reinterpret_cast<const float4*>(kbase + (long long)(j0 + row) * D + c);
      }
    };
    fetch(0);
    auto put = [&](int) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = tid + u * 256, row = e / 16, c = (e % 16) * 4;
        *reinterpret_cast<float4*>(As + row * kTileLd + c) = ra[u];
        *reinterpret_cast<float4*>(Bs + row * kTileLd + c) = rb[u];
      }
    };
    return fp32_tile<D>(As, Bs, put, [&](int p) { if (p + 1 < P) fetch(p + 1); }, out, i0, j0, nb, nb_valid, rsqrt_d);
  }
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;  // this wave's quadrant
  const int c16 = lane & 15, G = lane >> 4;
  // a row's eight 16-byte chunks are stored at chunk ^ (row % 8): sixteen rows of a fragment spread over the banks
  auto at = [](int row, int chunk) { return row * (KC * 2) + ((chunk ^ (row & 7)) << 4); };
  // thread: two pieces of eight channels of either operand per pass, those of all passes requested at once
  float4 raw[P][2][2][2];  // [pass][operand][piece][half]
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = tid + 256 * u, row = e >> 3, c = p * KC + (e & 7) * 8;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        raw[p][0][u][half] = raw[p][1][u][half] = make_float4(0.f, 0.f, 0.f, 0.f);  // zero rows beyond nb
        if (i0 + row < nb) raw[p][0][u][half] = *reinterpret_cast<const float4*>(qbase + (long long)(i0 + row) * D + c + 4 * half);
        if (j0 + row < nb) raw[p][1][u][half] = *reinterpret_cast<const float4*>(kbase + (long long)(j0 + row) * D + c + 4 * half);
      }
    }
  f32x4 big[2][2], small[2][2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) big[mt][nt] = small[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  // do parts carry the operands of all passes?
  float top = 0.f, least_top = INFINITY;  // largest magnitude; the smallest that is the largest of its piece
  unsigned least = ~0u;                   // the smallest that is not 0: twice its bits less 1, of which 0 makes the largest number
  auto look = [&](const float(&x)[8]) {
    float t = 0.f;
    largest8(t, x);
    top = fmaxf(top, t), least_top = fminf(least_top, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) least = min(least, 2u * __float_as_uint(x[i]) - 1u);
  };
  auto bad = [&] {  // (a NaN stays a NaN either way)
    return top >= kScoreMost || (least < below(-50) && (least_top < 0x1p-40f || least < below(-100)));
  };
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (p) __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = tid + 256 * u;
        float x[8];
        *reinterpret_cast<float4*>(x) = raw[p][o][u][0];
        *reinterpret_cast<float4*>(x + 4) = raw[p][o][u][1];
        if (p == 0) look(x);
        const Split s = split8(x);
#pragma unroll
        for (int part = 0; part < 3; ++part)
          *reinterpret_cast<bf16x8*>(smem + (3 * o + part) * kPlane + at(e >> 3, e & 7)) = s.p[part];
      }
    if (p == 0) {
#pragma unroll
      for (int f = 4; f < 4 * P; ++f) {
        float x[8];
        *reinterpret_cast<float4*>(x) = raw[f >> 2][(f >> 1) & 1][f & 1][0];
        *reinterpret_cast<float4*>(x + 4) = raw[f >> 2][(f >> 1) & 1][f & 1][1];
        look(x);
      }
      const int any = __any(bad());
      if (lane == 0) refused[wave] = any;
    }
    __syncthreads();
    if (p == 0 && (refused[0] | refused[1] | refused[2] | refused[3])) {
      auto put = [&](int of) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const int e = tid + 256 * u, at = (e >> 3) * kTileLd + (e & 7) * 8 + 4 * half;
            *reinterpret_cast<float4*>(As + at) = raw[of][0][u][half];
            *reinterpret_cast<float4*>(Bs + at) = raw[of][1][u][half];
          }
      };
      return fp32_tile<D>(As, Bs, put, [](int) {}, out, i0, j0, nb, nb_valid, rsqrt_d);
    }
#pragma unroll
    for (int t = 0; t < KC / 32; ++t) {
      bf16x8 a[2][3], b[2][3];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int part = 0; part < 3; ++part) {
          a[x][part] = *reinterpret_cast<const bf16x8*>(smem + part * kPlane + at(wi + 16 * x + c16, 4 * t + G));
          b[x][part] = *reinterpret_cast<const bf16x8*>(smem + (3 + part) * kPlane + at(wj + 16 * x + c16, 4 * t + G));
        }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          f32x4& s = small[mt][nt];
          s = mfma(a[mt][2], b[nt][0], s);
          s = mfma(a[mt][0], b[nt][2], s);
          s = mfma(a[mt][1], b[nt][1], s);
          s = mfma(a[mt][1], b[nt][0], s);
          s = mfma(a[mt][0], b[nt][1], s);
          big[mt][nt] = mfma(a[mt][0], b[nt][0], big[mt][nt]);
        }
    }
  }
  // element r of tile (mt, nt): row wi + 16 mt + 4 G + r, column wj + 16 nt + c16
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int j = j0 + wj + 16 * nt + c16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + wi + 16 * mt + 4 * G + r;
        if (i < nb && j < nb)
          out[(long long)i * nb + j] = (i < nb_valid && j < nb_valid) ? (big[mt][nt][r] + small[mt][nt][r]) * rsqrt_d : -INFINITY;
      }
    }
}

template <typename T, int D>
hipError_t run(const void* q, const void* k, const Dims& s, float* scores, float* ws, hipStream_t st,
               const RasterArgs* ras = nullptr) {
  const long long cubes = s.bh() * s.nb;
  const long long mean_elems = cubes * D;
  if (ras)
    pool_means<T, D, true><<<dim3((unsigned)cubes, 2), kPoolThreads, 0, st>>>(
        static_cast<const T*>(q), static_cast<const T*>(k), ws, s.nb, s.Nv, mean_elems, *ras);
  else
    pool_means<T, D><<<dim3((unsigned)cubes, 2), kPoolThreads, 0, st>>>(
        static_cast<const T*>(q), static_cast<const T*>(k), ws, s.nb, s.Nv, mean_elems);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int tiles = (s.nb + 63) / 64;
  // Parts from 512 blocks on; from there a head's tiles fill the chip with a few heads.  Batch and heads have no part in this: a head has the same
  // scores, to the bit, in any launch.  Stage 1 with fp32 operands / in parts, d = 128: 1 head x 512 blocks 8.9 / 9.9 us, 2 11.4 / 12.4, 6 27.4 / 27.5, 12
  // 45.7 / 44.8, 40 146 / 137; 1 x 1182 18.0 / 18.0, 40 x 1182 421 / 382; d = 64 7.1 / 7.5 (1 x 512), 27.6 / 27.2 (12 x 512), 222 / 204 (40 x 1182).  Below:
  // 12 x 55 9.9 / 11.0, 12 x 256 24.3 / 25.4, 12 x 448 43.0 / 42.8, 24 x 448 80.8 / 76.  (Error against 64 bits, 2-norm: 2.06e-7 / 0.72e-7 at d = 128,
  // 1.46e-7 / 0.5e-7 at d = 64.)
  const int fp32 = s.nb < 512;
  score_gemm<D><<<dim3(tiles, tiles, (unsigned)s.bh()), 256, 0, st>>>(ws, ws + mean_elems, scores, s.nb,
                                                                         s.nb_valid, 1.0f / sqrtf((float)D), fp32);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t run_pool(const void* x, const Dims& s, float* means, hipStream_t st, const RasterArgs* ras) {
  const long long cubes = s.bh() * s.nb;
  if (ras)
    pool_means<T, D, true><<<dim3((unsigned)cubes, 1), kPoolThreads, 0, st>>>(
        static_cast<const T*>(x), static_cast<const T*>(x), means, s.nb, s.Nv, cubes * D, *ras);
  else
    pool_means<T, D><<<dim3((unsigned)cubes, 1), kPoolThreads, 0, st>>>(static_cast<const T*>(x), static_cast<const T*>(x),
                                                                        means, s.nb, s.Nv, cubes * D);
  return hipGetLastError();
}

}  // namespace

// Pooled fp32 means of ONE tensor [B, Hh, N, d] -> means [B, Hh, nb, d].
hipError_t launch_pool_means(const void* x, const Dims& s, float* means, hipStream_t st, const RasterArgs* ras) {
  if (s.bf16)
    return s.d == 128 ? run_pool<uint16_t, 128>(x, s, means, st, ras) : run_pool<uint16_t, 64>(x, s, means, st, ras);
  return s.d == 128 ? run_pool<float, 128>(x, s, means, st, ras) : run_pool<float, 64>(x, s, means, st, ras);
}

hipError_t launch_block_scores(const void* q, const void* k, const Dims& s, float* scores, float* ws,
                               hipStream_t st, const RasterArgs* ras) {
  if (s.bf16)
    return s.d == 128 ? run<uint16_t, 128>(q, k, s, scores, ws, st, ras) : run<uint16_t, 64>(q, k, s, scores, ws, st, ras);
  return s.d == 128 ? run<float, 128>(q, k, s, scores, ws, st, ras) : run<float, 64>(q, k, s, scores, ws, st, ras);
}

}  // namespace usv
