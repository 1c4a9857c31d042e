// Stage 3, fp32 variant: block-sparse attention for fp32 Q/K/V to fp32 accuracy
// (masked-attention equation, paper Section 3.2).  This is the accuracy path (inputs that must
// match an fp64 evaluation to 1e-5); the throughput path is the bf16 kernel.
//
// The fp32 matrix pipe bounds a kernel that feeds it fp32 operands (157 TFLOP/s; 2 heads, 32768 tokens, 51 of 512 blocks:
// 944 us at 117 TFLOP/s).  So every operand is split into three bf16 parts instead: x = x0 + x1 + x2 with x0 the nearest bf16
// to x, x1 the nearest to x - x0 and x2 the rest, which fits 8 bits: the split is exact (24 bits of fp32 = 3 x 8) as long as x2
// has a place in bf16, that is for |x| >= 2^-110 and 0; and the products of parts are exact in the bf16 matrix core's fp32
// accumulation.  (Splitting fp32 operands so is a published method: Henry, Tang, Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", 2019.)  Of the nine products six are formed:
//   x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0);
// the three left out are below 2^-24 |x y| together (typically 2^-27, of either sign), under one rounding of the fp32
// sum.  Six products at sixteen times the rate leave 3/8 of the matrix time.
// Measured there: 944 -> 610 us (0.66 PFLOP of bf16 products at 1.08 PFLOP/s, the rate the bf16 attention kernels reach under
// the chip's power limit: matrix pipes busy 48 % of the clocks at 1.93 GHz).  Error against a 64-bit evaluation (2-norm,
// relative), fp32 operands / split: 4 of 16 blocks 1.95e-7 / 1.51e-7, 51 of 512 1.22e-6 / 1.10e-6, flat weights 7.8e-7 /
// 4.5e-7, 300 of 512 6.9e-6 / 6.3e-6; lower in all of 16 settings (both head dimensions).
// Splitting the V rows between the MFMAs of the first product and the next K rows between those of the second took as many
// clocks and more power (645 us): the second workgroup already fills those gaps.
//
// attn_f32_few: 16 query rows to a workgroup, for launches of few query blocks; the same products and the same bounds on what a split can carry.
// attn_f32: one workgroup = 4 KH wavefronts = one 64-row query block; wave w owns query rows 16 (w % 4) .. + 15.  KH = 1: 32 keys
// (half a listed block) per step, every wave sees them all and nothing is merged at the end.  KH = 2 (small grids, see the
// launcher): a whole block per step, waves 0..3 take its first half and waves 4..7 its second, merged once through LDS.  K and V rows are fetched into
// registers one step ahead, split there by the whole workgroup and staged in LDS as three bf16 planes each; a
// second workgroup on the CU computes meanwhile.  Products on the transposes as in usv_attn_wide.hip
// (v_mfma_f32_16x16x32_bf16; lane = (c, G)): lane (c, G) holds query c, keys 16 mt + 4 G + r, and those eight values are, as
// they stand, the contraction slots of the P^T operand.
//
// fp32_block: the same block with fp32 operands on the fp32 matrix cores, for what a split cannot carry: infinities and NaN
// (inf - inf), values the rounding to bf16 takes past its largest, and lower parts that run out of exponent where that matters.
// The first two show in the row sum or in the result; for the third the workgroup keeps the largest magnitudes it has split
// (four instructions per eight values: 632 -> 642 us there) and looks at the size of its results: the bounds stand at kTiny.  Such a workgroup computes its
// block again this way.
#include <type_traits>

#include "usv_split.h"

namespace usv {
namespace {

// ---- fp32 operands ------------------------------------------------------------------------------
// wave (qh, kh) = 32 queries x 32 keys of every listed 64-key tile, an online softmax per key half, the two halves merged
// once at the end through LDS.  Both products run on v_mfma_f32_32x32x2_f32, on the transposes:
//   S^T (32 keys x 32 queries) = K (A operand) x Q^T (B operand)
//   O^T (32 d    x 32 queries) = V^T (A operand) x P^T (B operand)
// so that one query sits in one lane column and max / sum / rescale are per-lane values.  An MFMA
// step contracts two indices, one per 32-lane half g.  Which two is free as long as both operands
// agree: in the first product half g takes channels g*D/2 + t at step t (every lane reads its
// operands as contiguous 16-byte pieces), in the second the step r takes, in half g, exactly the
// key that accumulator register r of that half holds, so P^T needs no data movement at all.
// K and V tiles are staged in LDS as fp32 (rows padded by 4 floats), single-buffered.
template <int D>
constexpr int kF32Lds = 2 * kBlock * (D + 4) * (int)sizeof(float);

template <int D>  // (inlined: a call would need scratch memory)
__device__ __forceinline__ void fp32_block(unsigned char* smem, const float* __restrict__ q, const float* __restrict__ k,
                           const float* __restrict__ v, const int32_t* __restrict__ idx, int n_list,
                           float* __restrict__ out, float* __restrict__ lse, long long blk, int nb, int Nv, int kmax,
                           float scale_log2e, int row_lo = 0, int row_hi = kBlock) {  // writes rows row_lo .. row_hi - 1
  constexpr int LD = D + 4;      // LDS row stride in floats: 16-byte reads of consecutive rows spread over the banks
  constexpr int DSUB = D / 32;   // 32-wide d sub-tiles of the output
  constexpr int HALF = D / 2;    // channels per lane half in the first product
  constexpr int XROWS = DSUB * 16 + 2;  // exchange rows per wave: O registers, m, l
  static_assert(2 * XROWS * 64 == kBlock * LD, "the exchange area of the two query halves fills the K tile exactly");
  float* const Ks = reinterpret_cast<float*>(smem);  // K tile; at the end the exchange area
  float* const Vs = Ks + kBlock * LD;                // V tile; at the end the output staging rows

  const int i = (int)(blk % nb);
  const long long head = blk / nb;
  const long long head_off = head * (long long)nb * kBlock * D;
  const int tid = threadIdx.x & 255, lane = tid & 63;  // (a second set of four waves does the same work, to the same places)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qh = wave & 1, kh = wave >> 1;
  const int col = lane & 31, g = lane >> 5;

  // Q fragments: lane (col, g) holds channels g*HALF .. +HALF of query row 32 qh + col
  float qf[HALF];
  {
    const float* qp = q + head_off + (long long)(i * kBlock + qh * 32 + col) * D + g * HALF;
#pragma unroll
    for (int e = 0; e < HALF; e += 4) {
      const float4 t = *reinterpret_cast<const float4*>(qp + e);
      qf[e] = t.x; qf[e + 1] = t.y; qf[e + 2] = t.z; qf[e + 3] = t.w;
    }
  }
  f32x16 o[DSUB];
#pragma unroll
  for (int ds = 0; ds < DSUB; ++ds)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ds][r] = 0.f;
  float m = -INFINITY;  // running max of this wave's keys (log2 domain), identical in both lane halves
  float l = 0.f;        // this lane's partial row sum

  for (int n = 0; n < n_list; ++n) {
    const int j = min(max(idx[blk * kmax + n], 0), nb - 1);
    __syncthreads();  // the previous tile is fully consumed
    {
      const float* kp = k + head_off + (long long)j * kBlock * D;
      const float* vp = v + head_off + (long long)j * kBlock * D;
#pragma unroll
      for (int e = tid; e < kBlock * (D / 4); e += 256) {
        const int row = e / (D / 4), c = (e % (D / 4)) * 4;
        *reinterpret_cast<float4*>(Ks + row * LD + c) = *reinterpret_cast<const float4*>(kp + row * D + c);
        *reinterpret_cast<float4*>(Vs + row * LD + c) = *reinterpret_cast<const float4*>(vp + row * D + c);
      }
    }
    __syncthreads();

    // ---- S^T = K Q^T over this wave's 32 keys -------------------------------------------------
    // Four partial sums, a quarter of the channel steps each, added pairwise: the logits reach several
    // hundred before scaling, and a single 64-step fp32 chain rounds them too coarsely for the 1e-5 bound.
    f32x16 s;
    {
      const float* kr = Ks + (kh * 32 + col) * LD + g * HALF;
      auto quarter = [&](auto a_c) {  // channel steps a * HALF / 4 .. of the product
        constexpr int A = decltype(a_c)::value;
        f32x16 p;
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = 0.f;
#pragma unroll
        for (int t = A * (HALF / 4); t < (A + 1) * (HALF / 4); t += 4) {
          const float4 kv = *reinterpret_cast<const float4*>(kr + t);
          p = __builtin_amdgcn_mfma_f32_32x32x2f32(kv.x, qf[t], p, 0, 0, 0);
          p = __builtin_amdgcn_mfma_f32_32x32x2f32(kv.y, qf[t + 1], p, 0, 0, 0);
          p = __builtin_amdgcn_mfma_f32_32x32x2f32(kv.z, qf[t + 2], p, 0, 0, 0);
          p = __builtin_amdgcn_mfma_f32_32x32x2f32(kv.w, qf[t + 3], p, 0, 0, 0);
        }
        return p;
      };
      auto add = [](const f32x16& x, const f32x16& y) {
        f32x16 z;
#pragma unroll
        for (int r = 0; r < 16; ++r) z[r] = x[r] + y[r];
        return z;
      };
      using Q0 = std::integral_constant<int, 0>;
      using Q1 = std::integral_constant<int, 1>;
      using Q2 = std::integral_constant<int, 2>;
      using Q3 = std::integral_constant<int, 3>;
      f32x16 lo = quarter(Q0{});
      lo = add(lo, quarter(Q1{}));
      __builtin_amdgcn_sched_barrier(0);
      f32x16 hi = quarter(Q2{});
      s = add(lo, add(hi, quarter(Q3{})));
    }
    // register r of lane (col, g) is key 32 kh + 8 (r/4) + 4 g + (r%4) of the tile, query col
    const int nkeys = Nv - j * kBlock;  // valid keys of the tile (>= 64 except in the last, partial block)
    if (nkeys < kBlock) {
      const int lim = nkeys - (kh * 32 + 4 * g);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = (8 * (r >> 2) + (r & 3)) < lim ? s[r] : -INFINITY;
    }

    // ---- online softmax (log2 domain) ---------------------------------------------------------
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    {
      float lo, hi;
      both_halves(mx, lo, hi);
      mx = fmaxf(lo, hi) * scale_log2e;
    }
    const float m_new = fmaxf(m, mx);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // every key so far masked: all p are exp2(-inf) = 0
    if (__any(m_new > m)) {  // wave-uniform; rows whose max did not move get alpha = 1
      const float alpha = __builtin_amdgcn_exp2f(m - m_ref);  // m = -inf -> 0
      l *= alpha;
#pragma unroll
      for (int ds = 0; ds < DSUB; ++ds)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[ds][r] *= alpha;
    }
    m = m_new;
    float p[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2e, -m_ref));
      l += p[r];
    }

    // ---- O^T += V^T P^T: step r contracts, in half g, the key that register r of that half holds ----
    {
      const float* vr = Vs + (kh * 32 + 4 * g) * LD + col;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float* vk = vr + (8 * (r >> 2) + (r & 3)) * LD;
#pragma unroll
        for (int ds = 0; ds < DSUB; ++ds) o[ds] = __builtin_amdgcn_mfma_f32_32x32x2f32(vk[32 * ds], p[r], o[ds], 0, 0, 0);
      }
    }
  }

  // ---- merge the two key halves, stage the block row-major, store coalesced -------------------
  __syncthreads();  // every wave is done with the last tile: Ks and Vs are free
  float l_lo, l_hi;
  both_halves(l, l_lo, l_hi);
  const float l_row = l_lo + l_hi;
  float* xch = Ks + qh * XROWS * 64;  // [XROWS][64 lanes] of this query half
  if (kh == 1) {
    float* dst = xch + lane;
#pragma unroll
    for (int ds = 0; ds < DSUB; ++ds)
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[(ds * 16 + r) * 64] = o[ds][r];
    dst[(DSUB * 16) * 64] = m;
    dst[(DSUB * 16 + 1) * 64] = l_row;
  }
  __syncthreads();
  if (kh == 0) {
    const float* src = xch + lane;
    const float m1 = src[(DSUB * 16) * 64], l1 = src[(DSUB * 16 + 1) * 64];
    const float mm = fmaxf(m, m1);
    const float m_ref = mm == -INFINITY ? 0.f : mm;
    const float a0 = __builtin_amdgcn_exp2f(m - m_ref), a1 = __builtin_amdgcn_exp2f(m1 - m_ref);
    const float lt = l_row * a0 + l1 * a1;
    const int token = i * kBlock + qh * 32 + col;
    const bool live = token < Nv && n_list > 0 && lt > 0.f;
    const float inv = live ? 1.f / lt : 0.f;
    const float w0 = live ? a0 * inv : 0.f, w1 = live ? a1 * inv : 0.f;
    float* stage = Vs + (qh * 32 + col) * LD;  // row (32 qh + col) of the block
#pragma unroll
    for (int ds = 0; ds < DSUB; ++ds)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {  // register r = 4 rq + e is channel 32 ds + 8 rq + 4 g + e
        float4 val;
        val.x = live ? o[ds][rq * 4] * w0 + src[(ds * 16 + rq * 4) * 64] * w1 : 0.f;
        val.y = live ? o[ds][rq * 4 + 1] * w0 + src[(ds * 16 + rq * 4 + 1) * 64] * w1 : 0.f;
        val.z = live ? o[ds][rq * 4 + 2] * w0 + src[(ds * 16 + rq * 4 + 2) * 64] * w1 : 0.f;
        val.w = live ? o[ds][rq * 4 + 3] * w0 + src[(ds * 16 + rq * 4 + 3) * 64] * w1 : 0.f;
        *reinterpret_cast<float4*>(stage + 32 * ds + 8 * rq + 4 * g) = val;
      }
    const int row = qh * 32 + col;
    if (lse && g == 0 && row >= row_lo && row < row_hi)
      lse[head * (long long)nb * kBlock + token] = live ? (mm + __log2f(lt)) * kLn2 : -INFINITY;
  }
  __syncthreads();
  {
    // 64 rows x D channels, 4 channels per thread per pass, consecutive threads -> consecutive addresses
    float* ob = out + head_off + (long long)i * kBlock * D;
#pragma unroll
    for (int e = tid; e < kBlock * (D / 4); e += 256) {
      const int row = e / (D / 4), c = (e % (D / 4)) * 4;
      if (row < row_lo || row >= row_hi) continue;
      *reinterpret_cast<float4*>(ob + row * D + c) = *reinterpret_cast<const float4*>(Vs + row * LD + c);
    }
  }
}

// ---- operands in three bf16 parts ---------------------------------------------------------------
// What three parts cannot carry.  A part below 2^-133 has no place in bf16 (and below 2^-126 it need not keep its last bits), so
// an operand is good to 2^-24 of itself or to 2^-125, whichever is more, and so is a product.  That is too little where
//  - a Q or K beside it is larger than 2^80 / scale: up to there the logits move by less than 2^-36;
//  - a result is below 2^-80, or below 2^-80 of the largest |V| of its channels (a small p against a large V): down to there
//    2^18 keys' errors of 2^-125 stay under 2^-26 of it.  A result of exactly 0 is below both, but V may well be 0 there: it
//    counts if those channels hold nothing but values below 2^-80, or if a look through the listed rows of V (only then) finds a
//    subnormal value.
// Overflows, infinities and NaN make the row sum or the result infinite or NaN.
constexpr float kTiny = 0x1p-80f;
constexpr float kQkLimit = 0x1p80f;

template <int D, int KH>
__global__ __launch_bounds__(256 * KH, 2) void attn_f32(const float* __restrict__ q, const float* __restrict__ k,
                                                   const float* __restrict__ v, const int32_t* __restrict__ idx,
                                                   const int32_t* __restrict__ cnt, float* __restrict__ out,
                                                   float* __restrict__ lse, int nb, int Nv, int kmax, float scale_log2e,
                                                   float qk_limit, int total, int per_xcd) {
  constexpr int KS = D / 32, DT = D / 16;      // channel steps of the first product, 16-channel tiles of the second
  constexpr int kThreads = 256 * KH;
  constexpr int kKeys = 32 * KH;               // keys per step
  constexpr int kRow = D * 2;                  // bytes of a key's row in a plane
  constexpr int kPlane = kKeys * kRow;         // one part of K or V
  constexpr int CH = D / 8;                    // 16-byte chunks per row
  constexpr int PIECES = kKeys * CH / kThreads;     // chunks (eight channels) of K, and of V, that a thread fetches and splits
  constexpr int LD = D + 4;                    // row stride of the output staging rows
  constexpr int kLds = kF32Lds<D> > 6 * kPlane ? kF32Lds<D> : 6 * kPlane;
  constexpr int XROWS = DT * 4 + 2;            // exchange rows of 64 floats per wave: O, reference and sum
  constexpr int kExchange = KH == 2 ? 4 * XROWS * 64 : 0;  // floats
  static_assert((kExchange + kBlock * LD) * (int)sizeof(float) <= kLds, "exchange area and output rows overlay the planes");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kLds];
  __shared__ int redo[4 * KH];
  __shared__ unsigned v_top[CH];  // largest |V| that was staged, per 8 channels (bits of the float)
  __shared__ unsigned zero_at;    // groups of eight channels with a result of 0 beside other values
  __shared__ int subnormal_v;     // ... and V is not 0 there

  const int work = xcd_contiguous_id(blockIdx.x, per_xcd);  // neighbouring query blocks share K and V in an XCD's L2
  if (work >= total) return;  // whole workgroup leaves before any barrier
  const long long blk = work;  // (b*Hh + h) * nb + i
  const int i = work % nb;
  const long long head = work / nb;
  const long long head_off = head * (long long)nb * kBlock * D;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave & 3, kh = wave >> 2;  // query rows 16 qw .., keys 32 kh .. of a step
  const int c16 = lane & 15, G = lane >> 4;
  const int n_list = min(max(cnt[blk], 0), kmax);  // device contents are not trusted with addresses
  const int32_t* list = idx + blk * kmax;

  // Position of chunk c of row r inside a plane.  The 16 rows of a K fragment read, and the 8 rows of half of a transposing V
  // read (32 bytes each), fall on different banks.
  auto k_at = [](int r, int c) { return D == 128 ? r * kRow + ((c ^ (r & 15)) << 4) : r * kRow + ((c ^ ((r >> 1) & 7)) << 4); };
  auto v_at = [](int r, int c) {
    return D == 128 ? r * kRow + ((c ^ ((r & 7) << 1)) << 4) : r * kRow + ((c ^ (((r >> 1) & 3) << 1)) << 4);
  };

  // The rows of a step on their way from memory: this thread's pieces, piece u = row (kThreads u + tid) / CH, chunk (tid % CH)
  float4 kraw[PIECES][2], vraw[PIECES][2];
  auto fetch = [&](int j, int half) {
    const long long at = head_off + ((long long)j * kBlock + half * 32) * D;
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
      const long long off = at + (long long)(kThreads * u + tid) * 8;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        kraw[u][e] = reinterpret_cast<const float4*>(k + off)[e];
        vraw[u][e] = reinterpret_cast<const float4*>(v + off)[e];
      }
    }
  };
  auto block_at = [&](int n) { return min(max(list[n], 0), nb - 1); };

  int j = n_list > 0 ? block_at(0) : 0;
  if (n_list > 0) fetch(j, 0);

  // Q^T fragments: query row 16 qw + c16, channels 32 t + 8 G .. + 8
  Split qf[KS];
  float q_top = 0.f, k_top = 0.f, v_max = 0.f;  // largest magnitudes this lane splits (a thread's pieces share their channels)
  {
    const float* qp = q + head_off + (long long)(i * kBlock + qw * 16 + c16) * D + G * 8;
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      float x[8];
      *reinterpret_cast<float4*>(x) = reinterpret_cast<const float4*>(qp + 32 * t)[0];
      *reinterpret_cast<float4*>(x + 4) = reinterpret_cast<const float4*>(qp + 32 * t)[1];
      largest8(q_top, x);
      qf[t] = split8(x);
    }
  }
  // channel 16 dt + 4 G + r of query c16: the leading products and the small ones in sums of their own (in one sum every small
  // product would round the whole of it)
  f32x4 o[DT], o5[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = o5[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, m_ref = 0.f;  // reference maximum (log2 domain), identical in the four lanes of a query; 0 in its place before the first live key
  float l = 0.f;        // this lane's partial row sum

  const unsigned char* const ks = smem;
  const unsigned char* const vs = smem + 3 * kPlane;
  if (tid < CH) v_top[tid] = 0;  // (the barriers of the loop stand between this and the first maximum)
  if (tid == 0) zero_at = 0, subnormal_v = 0;

  constexpr int kSteps = 2 / KH;  // steps per listed block
  for (int st = 0; st < kSteps * n_list; ++st) {
    const int half = st % kSteps;
    const int nkeys = Nv - j * kBlock - half * 32;  // valid keys of this step (below kKeys only at the end of the sequence)
    __syncthreads();  // the previous step's planes are fully consumed
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
      const int e = kThreads * u + tid, row = e / CH, c = e % CH;
      float x[8];
      *reinterpret_cast<float4*>(x) = kraw[u][0];
      *reinterpret_cast<float4*>(x + 4) = kraw[u][1];
      largest8(k_top, x);
      const Split a = split8(x);
#pragma unroll
      for (int part = 0; part < 3; ++part) *reinterpret_cast<bf16x8*>(smem + part * kPlane + k_at(row, c)) = a.p[part];
      *reinterpret_cast<float4*>(x) = vraw[u][0];
      *reinterpret_cast<float4*>(x + 4) = vraw[u][1];
      if (nkeys < kKeys) {  // padded rows may hold any finite value, also one that rounds to infinity: their p is 0
#pragma unroll
        for (int y = 0; y < 8; ++y) x[y] = row < nkeys ? x[y] : 0.f;
      }
      largest8(v_max, x);
      const Split b = split8(x);
#pragma unroll
      for (int part = 0; part < 3; ++part)
        *reinterpret_cast<bf16x8*>(smem + (3 + part) * kPlane + v_at(row, c)) = b.p[part];
    }
    if (half == kSteps - 1) j = block_at(min(st / kSteps + 1, n_list - 1));
    if (st + 1 < kSteps * n_list) fetch(j, (st + 1) % kSteps);
    __syncthreads();

    // ---- S^T = K Q^T: the leading product and the five small ones in sums of their own ----
    f32x4 s[2], t5[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) s[mt] = t5[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[2][3];  // the fragments of this product and, on their way from LDS, of the next
    auto read_k = [&](int f) {  // fragment f = 2 t + mt
#pragma unroll
      for (int part = 0; part < 3; ++part)
        a[f & 1][part] = *reinterpret_cast<const bf16x8*>(ks + part * kPlane + k_at(32 * kh + 16 * (f & 1) + c16, 4 * (f >> 1) + G));
    };
    read_k(0);
#pragma unroll
    for (int f = 0; f < 2 * KS; ++f) {
      if (f + 1 < 2 * KS) read_k(f + 1);
      __builtin_amdgcn_sched_barrier(0);
      const bf16x8(&x)[3] = a[f & 1];
      const bf16x8(&y)[3] = qf[f >> 1].p;
      f32x4& big = s[f & 1];
      f32x4& small = t5[f & 1];
      small = mfma(x[2], y[0], small);
      small = mfma(x[0], y[2], small);
      small = mfma(x[1], y[1], small);
      small = mfma(x[1], y[0], small);
      small = mfma(x[0], y[1], small);
      big = mfma(x[0], y[0], big);
      __builtin_amdgcn_sched_barrier(0);
    }
    float x[8];  // key 16 (e / 4) + 4 G + e % 4 of the step, query c16
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = s[e >> 2][e & 3] + t5[e >> 2][e & 3];
    if (nkeys < kKeys) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 32 * kh + 16 * (e >> 2) + 4 * G + (e & 3) < nkeys ? x[e] : -INFINITY;
    }

    // ---- online softmax (log2 domain, lazily raised reference maximum: p stays below 2^slack, which fp32 does not feel) ----
    float mx = x[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mx = fmaxf(mx, x[e]);
    if (__any(mx * scale_log2e - m > kRescaleSlack)) {  // wave-uniform; always taken on the first step with a live key
      const float m_new = fmaxf(m, max_over_groups(mx) * scale_log2e);
      m_ref = m_new == -INFINITY ? 0.f : m_new;  // every key so far masked: all p are exp2(-inf) = 0
      const float alpha = fast_exp2(m - m_ref);  // m = -inf -> 0
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[dt][r] *= alpha, o5[dt][r] *= alpha;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      x[e] = fast_exp2(fmaf(x[e], scale_log2e, -m_ref));
      l += x[e];
    }
    const Split pf = split8(x);

    // ---- O^T += V^T P^T ----
    auto read_v = [&](int dt) {
#pragma unroll
      for (int part = 0; part < 3; ++part) {
        // rows 4 G + (0..3) and 16 + 4 G + (0..3); the 16 lanes of a group address 4 rows x 16 channels
        const int row = 32 * kh + 4 * G + (c16 >> 2);
        const unsigned char* at = vs + part * kPlane + v_at(row, 2 * dt + ((c16 >> 1) & 1)) + (c16 & 1) * 8;
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)at);
        const short4v hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(at + 16 * kRow));
        a[dt & 1][part] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    };
    read_v(0);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      if (dt + 1 < DT) read_v(dt + 1);
      __builtin_amdgcn_sched_barrier(0);
      const bf16x8(&y)[3] = a[dt & 1];
      o5[dt] = mfma(y[2], pf.p[0], o5[dt]);
      o5[dt] = mfma(y[0], pf.p[2], o5[dt]);
      o5[dt] = mfma(y[1], pf.p[1], o5[dt]);
      o5[dt] = mfma(y[1], pf.p[0], o5[dt]);
      o5[dt] = mfma(y[0], pf.p[1], o5[dt]);
      o[dt] = mfma(y[0], pf.p[0], o[dt]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- merge the key halves, stage the rows row-major, store coalesced ----
  v_max = max_over_groups(v_max);
  if (CH == 8) v_max = fmaxf(v_max, __shfl_xor(v_max, 8));
  if (n_list > 0 && lane < CH) atomicMax(&v_top[lane], __float_as_uint(v_max));  // (not negative: the bits order as the floats do)
  __syncthreads();  // every wave is done with the last planes; v_top is complete
  float lt = sum_over_groups(l);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 4; ++r) o[dt][r] += o5[dt][r];
  if constexpr (KH == 2) {
    float* xch = reinterpret_cast<float*>(smem) + qw * XROWS * 64 + lane;
    if (kh == 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) xch[(dt * 4 + r) * 64] = o[dt][r];
      xch[(DT * 4) * 64] = m;
      xch[(DT * 4 + 1) * 64] = lt;
    }
    __syncthreads();
    if (kh == 0) {
      const float m1 = xch[(DT * 4) * 64], l1 = xch[(DT * 4 + 1) * 64];
      const float mm = fmaxf(m, m1);
      const float ref = mm == -INFINITY ? 0.f : mm;
      const float a0 = fast_exp2(m - ref), a1 = fast_exp2(m1 - ref);
      lt = lt * a0 + l1 * a1;
      m = mm;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[dt][r] = o[dt][r] * a0 + xch[(dt * 4 + r) * 64] * a1;
    }
  }
  float* const rows = reinterpret_cast<float*>(smem) + kExchange;
  const int token = i * kBlock + qw * 16 + c16;
  const bool mine = token < Nv && n_list > 0 && kh == 0;
  const bool live = mine && lt > 0.f;  // lt == 0: every listed key is padding
  const float inv = live ? 1.f / lt : 0.f;
  bool bad = (mine && (!(lt < INFINITY) || q_top >= qk_limit)) || k_top >= qk_limit;
  bool small = false;
  float finite = 0.f;  // NaN as soon as a result is not finite
  float* stage = rows + (qw * 16 + c16) * LD;
  auto least = [&](float top) { return fmaxf(kTiny, top * kTiny); };
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      y[r] = live ? o[dt][r] * inv : 0.f;
      finite = fmaf(y[r], 0.f, finite);
    }
    small |= fminf(fminf(fabsf(y[0]), fabsf(y[1])), fminf(fabsf(y[2]), fabsf(y[3]))) < least(__uint_as_float(v_top[2 * dt + (G >> 1)]));
    if (kh == 0) *reinterpret_cast<float4*>(stage + 16 * dt + 4 * G) = make_float4(y[0], y[1], y[2], y[3]);
  }
  bad |= finite != 0.f;
  if (__any(live && small)) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int ch = 2 * dt + (G >> 1);
      const float top = __uint_as_float(v_top[ch]);
      bool zero = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float a = fabsf(o[dt][r] * inv);
        bad |= live && a < least(top) && (a > 0.f || (top > 0.f && top < kTiny));
        zero |= live && a == 0.f && top > 0.f;
      }
      if (zero) atomicOr(&zero_at, 1u << ch);
    }
  }
  const int any_bad = __any(bad);
  if (lane == 0) redo[wave] = any_bad;
  __syncthreads();
  int again = 0;
#pragma unroll
  for (int w = 0; w < 4 * KH; ++w) again |= redo[w];
  if (!again && zero_at) {  // results of 0 beside other values: is V 0 there, or too small to be split?
    bool sub = false;
    auto is_sub = [](unsigned x) { return (x & 0x7fffffffu) - 1u < 0x007fffffu; };
    for (unsigned left = zero_at; left; left &= left - 1) {
      const int ch = __ffs(left) - 1;
#pragma unroll 4
      for (int e = tid; e < n_list * kBlock; e += kThreads) {  // a row of these eight channels each
        const int jn = block_at(e / kBlock), row = jn * kBlock + e % kBlock;
        const uint4* at = reinterpret_cast<const uint4*>(v + head_off + (long long)min(row, Nv - 1) * D + ch * 8);
        const uint4 x = at[0], y = at[1];
        const bool any = is_sub(x.x) | is_sub(x.y) | is_sub(x.z) | is_sub(x.w) | is_sub(y.x) | is_sub(y.y) | is_sub(y.z) | is_sub(y.w);
        sub |= any && row < Nv;
      }
    }
    if (__any(sub) && lane == 0) subnormal_v = 1;
    __syncthreads();
    again = subnormal_v;
  }
  if (again) {
    fp32_block<D>(smem, q, k, v, idx, n_list, out, lse, blk, nb, Nv, kmax, scale_log2e);
    return;
  }
  if (lse && G == 0 && kh == 0) lse[head * (long long)nb * kBlock + token] = live ? (m + __log2f(lt)) * kLn2 : -INFINITY;
  float* ob = out + head_off + (long long)i * kBlock * D;
#pragma unroll
  for (int e = tid; e < kBlock * (D / 4); e += kThreads) {
    const int row = e / (D / 4), c = (e % (D / 4)) * 4;
    *reinterpret_cast<float4*>(ob + row * D + c) = *reinterpret_cast<const float4*>(rows + row * LD + c);
  }
}

// Few query blocks: one workgroup of eight waves = 16 query rows, so that four times as many CUs have work, and the waves share out
// the 32-key halves of the listed blocks instead of staging them together: a wave fetches its half straight into the lanes that
// need it (V by single channels, which is the transpose the second product wants), splits it there, and meets the others once, at
// the end, through LDS.  The loop has no barrier and no LDS.  What is paid for it: every half is split by four workgroups
// instead of one.  Bound by latency: launch, list, one round trip for the operands, the splits, the store (times at the
// launcher's rule).
template <int D>
__global__ __launch_bounds__(512, 2) void attn_f32_few(const float* __restrict__ q, const float* __restrict__ k,
                                                       const float* __restrict__ v, const int32_t* __restrict__ idx,
                                                       const int32_t* __restrict__ cnt, float* __restrict__ out,
                                                       float* __restrict__ lse, int nb, int Nv, int kmax, float scale_log2e,
                                                       float qk_limit, int total, int per_xcd) {
  constexpr int KS = D / 32, DT = D / 16, CH = D / 8, W = 8, ROWS = 16;
  constexpr bool kEarlyV = D == 64;   // registers for K and V of a half at once
  constexpr int LD = D + 4;           // row stride of a wave's part of O
  constexpr int VE = ROWS * D / 512;  // channels of a row that a thread finishes
  constexpr int kParts = W * (ROWS * LD + 2 * ROWS) * (int)sizeof(float);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kF32Lds<D> > kParts ? kF32Lds<D> : kParts];
  __shared__ float v_tops[W][CH];  // largest |V| that a wave has split, per 8 channels
  __shared__ int redo[W];
  __shared__ int redo_any, subnormal_v;
  __shared__ unsigned zero_at;

  const int work = xcd_contiguous_id(blockIdx.x, per_xcd);
  if (work >= total) return;  // whole workgroup leaves before any barrier
  const long long blk = work >> 2;
  const int rg = work & 3, i = (int)(blk % nb);
  const long long head_off = (blk / nb) * (long long)nb * kBlock * D;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, G = lane >> 4;
  const int32_t* list = idx + blk * kmax;
  auto block_at = [&](int n) { return min(max(list[n], 0), nb - 1); };  // device contents are not trusted with addresses

  // half h of block j: K fragment (mt, t): key 16 mt + c16, channels 32 t + 8 G .. + 8; V^T fragment dt: channel 16 dt + c16, keys 16 (e / 4) + 4 G + e % 4
  float4 kraw[2 * KS][2];
  float vraw[DT][8];
  auto fetch_k = [&](int j, int half) {
    const float* p = k + head_off + ((long long)j * kBlock + half * 32 + c16) * D + 8 * G;
#pragma unroll
    for (int f = 0; f < 2 * KS; ++f)
#pragma unroll
      for (int e = 0; e < 2; ++e) kraw[f][e] = reinterpret_cast<const float4*>(p + 16 * (f & 1) * D + 32 * (f >> 1))[e];
  };
  auto fetch_v = [&](int j, int half) {
    const float* p = v + head_off + ((long long)j * kBlock + half * 32 + 4 * G) * D + c16;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int e = 0; e < 8; ++e) vraw[dt][e] = p[(16 * (e >> 2) + (e & 3)) * D + 16 * dt];
  };
  // the wave's first half: asked for before the list's length is known (the entry is there to be read, whatever it says)
  int j = block_at(min(wave >> 1, kmax - 1));
  fetch_k(j, wave & 1);
  Split qf[KS];
  float q_top = 0.f, k_top = 0.f, v_max[DT];
  {
    const float* qp = q + head_off + ((long long)i * kBlock + rg * ROWS + c16) * D + G * 8;
    float4 raw[KS][2];
#pragma unroll
    for (int t = 0; t < KS; ++t) raw[t][0] = reinterpret_cast<const float4*>(qp + 32 * t)[0], raw[t][1] = reinterpret_cast<const float4*>(qp + 32 * t)[1];
    if (kEarlyV) fetch_v(j, wave & 1);
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      float x[8];
      *reinterpret_cast<float4*>(x) = raw[t][0];
      *reinterpret_cast<float4*>(x + 4) = raw[t][1];
      largest8(q_top, x);
      qf[t] = split8(x);
    }
  }
  const int n_list = min(max(cnt[blk], 0), kmax);
  f32x4 o[DT], o5[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = o5[dt] = f32x4{0.f, 0.f, 0.f, 0.f}, v_max[dt] = 0.f;
  float m = -INFINITY, m_ref = 0.f, l = 0.f;

  for (int c = wave; c < 2 * n_list; c += W) {
    const int nkeys = Nv - j * kBlock - (c & 1) * 32;  // valid keys of this half (below 32 only at the end of the sequence)
    const int jn = block_at(min((c + W) >> 1, n_list - 1));
    f32x4 s[2], t5[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) s[mt] = t5[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int f = 0; f < 2 * KS; ++f) {
      float x[8];
      *reinterpret_cast<float4*>(x) = kraw[f][0];
      *reinterpret_cast<float4*>(x + 4) = kraw[f][1];
      largest8(k_top, x);
      const Split a = split8(x);
      const bf16x8(&y)[3] = qf[f >> 1].p;
      f32x4& big = s[f & 1];
      f32x4& small = t5[f & 1];
      small = mfma(a.p[2], y[0], small);
      small = mfma(a.p[0], y[2], small);
      small = mfma(a.p[1], y[1], small);
      small = mfma(a.p[1], y[0], small);
      small = mfma(a.p[0], y[1], small);
      big = mfma(a.p[0], y[0], big);
    }
    if (!kEarlyV) fetch_v(j, c & 1);
    else if (c + W < 2 * n_list) fetch_k(jn, c & 1);
    float x[8];  // key 16 (e / 4) + 4 G + e % 4 of the half, query c16
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = s[e >> 2][e & 3] + t5[e >> 2][e & 3];
    if (nkeys < 32) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 16 * (e >> 2) + 4 * G + (e & 3) < nkeys ? x[e] : -INFINITY;
    }
    // online softmax, as in attn_f32
    float mx = x[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mx = fmaxf(mx, x[e]);
    if (__any(mx * scale_log2e - m > kRescaleSlack)) {
      const float m_new = fmaxf(m, max_over_groups(mx) * scale_log2e);
      m_ref = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = fast_exp2(m - m_ref);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[dt][r] *= alpha, o5[dt][r] *= alpha;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      x[e] = fast_exp2(fmaf(x[e], scale_log2e, -m_ref));
      l += x[e];
    }
    const Split pf = split8(x);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      if (nkeys < 32) {  // padded rows may hold any finite value, also one that rounds to infinity: their p is 0
#pragma unroll
        for (int e = 0; e < 8; ++e) vraw[dt][e] = 16 * (e >> 2) + 4 * G + (e & 3) < nkeys ? vraw[dt][e] : 0.f;
      }
      largest8(v_max[dt], vraw[dt]);
      const Split y = split8(vraw[dt]);
      o5[dt] = mfma(y.p[2], pf.p[0], o5[dt]);
      o5[dt] = mfma(y.p[0], pf.p[2], o5[dt]);
      o5[dt] = mfma(y.p[1], pf.p[1], o5[dt]);
      o5[dt] = mfma(y.p[1], pf.p[0], o5[dt]);
      o5[dt] = mfma(y.p[0], pf.p[1], o5[dt]);
      o[dt] = mfma(y.p[0], pf.p[0], o[dt]);
    }
    if (c + W < 2 * n_list) {
      if (kEarlyV) fetch_v(jn, c & 1);
      else fetch_k(jn, c & 1);
    }
    j = jn;
  }

  // ---- the waves' parts meet: row c16's O, reference and sum of each ----
  float* const part = reinterpret_cast<float*>(smem) + wave * ROWS * LD;
  float* const stats = reinterpret_cast<float*>(smem) + W * ROWS * LD;  // [W][2][ROWS]
  {
    const float lt = sum_over_groups(l);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4 both = o[dt] + o5[dt];
      *reinterpret_cast<f32x4*>(part + c16 * LD + 16 * dt + 4 * G) = both;
      float top = max_over_groups(v_max[dt]);
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) top = fmaxf(top, __shfl_xor(top, d));
      if (G == 0 && (c16 & 7) == 0) v_tops[wave][2 * dt + (c16 >> 3)] = top;
    }
    if (G == 0) stats[2 * ROWS * wave + c16] = m, stats[2 * ROWS * wave + ROWS + c16] = lt;
    const bool bad = (q_top >= qk_limit && i * kBlock + rg * ROWS + c16 < Nv && n_list > 0) || k_top >= qk_limit;
    const int any_bad = __any(bad);
    if (lane == 0) redo[wave] = any_bad;
    if (tid == 0) redo_any = 0, zero_at = 0, subnormal_v = 0;
  }
  __syncthreads();
  const int row = tid >> 5, ch = (tid & 31) * VE;  // 32 threads to a row
  float mm = -INFINITY, lt = 0.f, top = 0.f, y[VE];
  int again = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) mm = fmaxf(mm, stats[2 * ROWS * w + row]), top = fmaxf(top, v_tops[w][ch >> 3]), again |= redo[w];
  const float ref = mm == -INFINITY ? 0.f : mm;
#pragma unroll
  for (int e = 0; e < VE; ++e) y[e] = 0.f;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const float a = fast_exp2(stats[2 * ROWS * w + row] - ref);  // (a wave without keys: -inf, sum and O 0)
    lt += stats[2 * ROWS * w + ROWS + row] * a;
    const float* src = reinterpret_cast<const float*>(smem) + (w * ROWS + row) * LD + ch;
#pragma unroll
    for (int e = 0; e < VE; ++e) y[e] += src[e] * a;
  }
  const int token = i * kBlock + rg * ROWS + row;
  const bool mine = token < Nv && n_list > 0, live = mine && lt > 0.f;  // lt == 0: every listed key is padding
  const float inv = live ? 1.f / lt : 0.f, least = fmaxf(kTiny, top * kTiny);
  bool bad = mine && !(lt < INFINITY), zero = false;
#pragma unroll
  for (int e = 0; e < VE; ++e) {
    y[e] = live ? y[e] * inv : 0.f;
    const float a = fabsf(y[e]);
    bad |= !(a < INFINITY) || (live && a < least && (a > 0.f || (top > 0.f && top < kTiny)));
    zero |= live && a == 0.f && top > 0.f;
  }
  if (zero) atomicOr(&zero_at, 1u << (ch >> 3));
  if (bad) redo_any = 1;
  __syncthreads();
  again |= redo_any;
  if (!again && zero_at) {  // results of 0 beside other values: is V 0 there, or too small to be split?
    bool sub = false;
    auto is_sub = [](unsigned x) { return (x & 0x7fffffffu) - 1u < 0x007fffffu; };
    for (unsigned left = zero_at; left; left &= left - 1) {
      const int c8 = __ffs(left) - 1;
#pragma unroll 4
      for (int e = tid; e < n_list * kBlock; e += 512) {  // a row of these eight channels each
        const int r = block_at(e / kBlock) * kBlock + e % kBlock;
        const uint4* at = reinterpret_cast<const uint4*>(v + head_off + (long long)min(r, Nv - 1) * D + c8 * 8);
        const uint4 a = at[0], b = at[1];
        const bool any = is_sub(a.x) | is_sub(a.y) | is_sub(a.z) | is_sub(a.w) | is_sub(b.x) | is_sub(b.y) | is_sub(b.z) | is_sub(b.w);
        sub |= any && r < Nv;
      }
    }
    if (__any(sub) && lane == 0) subnormal_v = 1;
    __syncthreads();
    again = subnormal_v;
  }
  if (again) {  // (these 16 rows only: the block's other rows are other workgroups')
    fp32_block<D>(smem, q, k, v, idx, n_list, out, lse, blk, nb, Nv, kmax, scale_log2e, rg * ROWS, (rg + 1) * ROWS);
    return;
  }
  if (lse && ch == 0) lse[(blk / nb) * (long long)nb * kBlock + token] = live ? (mm + __log2f(lt)) * kLn2 : -INFINITY;
  float* dst = out + head_off + (long long)token * D + ch;
  if constexpr (VE == 2) *reinterpret_cast<float2*>(dst) = make_float2(y[0], y[1]);
  else *reinterpret_cast<float4*>(dst) = make_float4(y[0], y[1], y[2], y[3]);
}

}  // namespace

hipError_t launch_attn_f32(const float* q, const float* k, const float* v, const Dims& s, const int32_t* idx,
                           const int32_t* cnt, int kmax, float scale, float* out, float* lse, hipStream_t st) {
  const int total = (int)(s.bh() * s.nb), per_xcd = (total + kNumXcd - 1) / kNumXcd;
  const unsigned grid = (unsigned)per_xcd * kNumXcd;
  const float sl2 = scale * kLog2e;
  auto launch = [&](auto d_c, auto kh_c) {
    constexpr int KH = decltype(kh_c)::value;
    attn_f32<decltype(d_c)::value, KH><<<grid, 256 * KH, 0, st>>>(q, k, v, idx, cnt, out, lse, s.nb, s.Nv, kmax, sl2,
                                                                kQkLimit / fmaxf(scale, 1.f), total, per_xcd);
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  // Up to one workgroup per CU, eight waves that take both halves of a block at once; beyond, four waves, so that a CU holds a
  // second workgroup to compute while one stages.  KH = 1 / 2, 20 listed: d = 64, 128 blocks 50.2 / 37.1 us, 256: 50.6 / 38.7, 320:
  // 68.6 / 70.6, 512: 72.8 / 73.7; d = 128, 128 blocks 87 / 64 us, 256: 88 / 69, 320: 117 / 126, 512: 127 / 135.
  const bool few = total <= 256;
  // Up to 64 query blocks, four workgroups of 16 rows to a block still have a CU each.  attn_f32<D, 2> / attn_f32_few, lists of 1, 3, 6, 12, 16: d = 64,
  // 64 blocks 8.7 / 8.4, 9.8 / 8.2, 14.8 / 9.7, 24.0 / 13.9, 30.2 / 16.8 us (8 us are the host's), 128 blocks 9.9 / 14.5 (3), 30.4 / 31.0 (16);
  // d = 128, 64 blocks 9.6 / 10.3, 15.7 / 12.8, 24.2 / 16.2, 41.4 / 25.4, 52.8 / 31.9, 128 blocks 16.1 / 24.3, 53.4 / 60.2.
  if (total <= 64 && (s.d == 64 || kmax > 1)) {
    const int groups = 4 * total, per = (groups + kNumXcd - 1) / kNumXcd;
    auto go = [&](auto d_c) {
      attn_f32_few<decltype(d_c)::value><<<(unsigned)per * kNumXcd, 512, 0, st>>>(q, k, v, idx, cnt, out, lse, s.nb, s.Nv, kmax, sl2,
                                                                              kQkLimit / fmaxf(scale, 1.f), groups, per);
    };
    if (s.d == 128) go(std::integral_constant<int, 128>{});
    else go(std::integral_constant<int, 64>{});
    return hipGetLastError();
  }
  if (s.d == 128) few ? launch(std::integral_constant<int, 128>{}, I2{}) : launch(std::integral_constant<int, 128>{}, I1{});
  else few ? launch(std::integral_constant<int, 64>{}, I2{}) : launch(std::integral_constant<int, 64>{}, I1{});
  return hipGetLastError();
}

}  // namespace usv
