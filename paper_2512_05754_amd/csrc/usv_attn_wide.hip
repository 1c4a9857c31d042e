// Stage 3, bf16 path: block-sparse flash attention on the gfx950 matrix cores
// (masked-attention equation, paper Section 3.2; only listed K/V cubes are touched).
//
// This file: the kernel for grids that fill the chip (the one for small grids, and the rule, are in usv_attn_bf16.hip).
//
// Work decomposition: one workgroup = 2 wavefronts = one 64-row query block.  Wave w owns ALL 64 queries and half w (32
// keys) of every listed 64-key tile, with an online softmax of its own, and the two partial results are merged once, at
// the end, through LDS.  A wave therefore fetches, waits for and reads its own K and V only: the main loop has no
// barrier, and every fragment read from LDS feeds four MFMAs.
//
// Matrix-core mapping (v_mfma_f32_16x16x32_bf16, fp32 accumulate; lane = (c, G) with c = lane % 16, G = lane / 16; the A
// operand holds row c, contraction slots 8 G .. 8 G + 7, the B operand column c and the same slots, the result column c,
// rows 4 G .. 4 G + 3):
//   S^T (16 keys x 16 queries) = K_tile (A, rows = keys) x Q^T (B, cols = queries), D / 32 steps over the channels
//   O^T (16 d    x 16 queries) = V^T    (A, rows = d)    x P^T (B, cols = queries), ONE step over the wave's 32 keys
// i.e. 2 x 4 tiles of S^T and D/16 x 4 tiles of O^T per wave and step.  Working on the transposes keeps a query in a lane
// column: lane (c, G) holds queries c, 16 + c, 32 + c, 48 + c, eight keys of each (16 mt + 4 G + r), and those eight S^T
// accumulator values are, as they stand, the eight contraction slots of the P^T operand for that query (the contraction
// index of an MFMA can be enumerated in any order as long as both operands agree).  Row statistics stay in the lane; only a
// raise of the reference maximum (rare) looks across the four lanes of a query.  V^T fragments come from the row-major V
// rows with the LDS transpose read ds_read_b64_tr_b16.
//
// LDS ring: an item is 32 keys x 64 channels of K or V (one 128-byte line of every row, 4 KiB), fetched by four
// global_load_lds_dwordx4 (16 bytes per lane, no register staging).  A wave holds one half tile (D/64 items of K, D/64 of
// V); as soon as the last fragment of an item is in registers its slot is refilled with the same item of the next half tile.
// Inside an item the stored row order is the one in which DMA instruction r, whose offset is added to the global AND the
// LDS address, takes the rows 4 r + {0..3} and 16 + 4 r + {0..3} (D = 128): one M0 write per item, and stored row 8 r + x
// is key slot 8 r + x of the fragments (which key that is matters to the mask only).  Within a 128-byte line the 16-byte
// chunks are XOR-permuted (on the global side) so that both the 16-byte K reads and the transposing V reads are
// bank-conflict free (measured: 0), and every other fragment address is an immediate.
//
// What bounds the kernel, measured on MI355X: the chip's power limit (it clocks this kernel at ~1.65 GHz of 2.4), and on
// lists that neighbouring query blocks do not share the L2-miss path, which delivers 7.0 TB/s whatever the number of loads in
// flight.  Against 4 waves of 32 queries x 32 keys of a shared tile, with two barriers per tile (usv_attn_bf16.hip), the
// split halves the LDS fragment reads and drops the barriers: lists of one head that are all alike 0.712 -> 0.676 ms (12
// heads, 32768 tokens, 51 of 512 blocks), all blocks listed 6.07 -> 5.74 ms, 8..64 of 256 blocks with a work order 0.526 ->
// 0.483 ms.  Two waves per workgroup (four workgroups per CU) and not four: the prologue and the epilogue of one
// workgroup overlap with three others, and 128 instead of 64 query blocks of an XCD can share a fetched tile (a four-wave
// form: 51 of 512 blocks 0.755 ms, 59 of 1182 8.3 ms).  That sharing needs their sweeps over the keys to stay together: see
// "where the list starts" below.
#include "usv_attn_bf16.h"

namespace usv {
namespace {

constexpr int NW = 2;        // waves per workgroup
constexpr int kItem = 4096;  // one item of the ring: 32 keys x 64 channels
constexpr float kNoKey = 3.4028234e38f;  // reference of a row that has seen no key yet

// One item, global -> LDS: instruction r lands at lds + 1024 r + 16 * lane.  Inline assembly so that the compiler does not
// pair the DMA with a conservative "wait for all memory" before the next LDS read of ANOTHER item; completion is
// awaited explicitly (vmcnt).  M0 carries the LDS address; nothing else in this kernel uses M0 (no LDS-direct reads, no
// relative register indexing), and the compiler refuses M0 on a clobber list (reserved register), so every block
// writes M0 itself right before the instructions that read it.
__device__ __forceinline__ void dma_item(unsigned lds, const void* base, int even, int odd) {  // rows a fixed pitch apart
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "global_load_lds_dwordx4 %1, %3\n\t"
      "global_load_lds_dwordx4 %2, %3 offset:1024\n\t"
      "global_load_lds_dwordx4 %1, %3 offset:2048\n\t"
      "global_load_lds_dwordx4 %2, %3 offset:3072"
      :
      : "s"(lds), "v"(even), "v"(odd), "s"(base)
      : "memory");
}
// Half an item, rows anywhere: instructions 2 HALF and 2 HALF + 1.  Offset of instruction r from base: its rows' plus kBack - 1024 r
// (the instruction's own offset goes to both addresses).  Halves, so that two address registers do.
constexpr int kBack = 3072;
template <int HALF>
__device__ __forceinline__ void dma_half(unsigned lds, const void* base, unsigned v0, unsigned v1) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "global_load_lds_dwordx4 %1, %3 offset:%4\n\t"
      "global_load_lds_dwordx4 %2, %3 offset:%5"
      :
      : "s"(lds), "v"(v0), "v"(v1), "s"(static_cast<const unsigned char*>(base) - kBack), "n"(2048 * HALF), "n"(2048 * HALF + 1024)
      : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vm() {  // at most N vector-memory operations of this wave are still in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}

// The lane number, formed anew where it is asked for: a value that is kept ahead of the loop is a register raster mode has not got.
__device__ __forceinline__ int lane_again() {
  unsigned all = ~0u;
  asm volatile("" : "+s"(all));
  return __builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

// WPS: waves per SIMD the register budget is sized for.  DEEP: one more ring slot (requests half a tile further ahead), for
// heads whose K and V are far beyond the L2.  TURNS: the waves of a SIMD
// take turns ("taking turns" below).
// RASTER: Q, K, V and the output are in raster token order (any strides); `ras.order[p]` gives the raster index of
// cube-major position p.  Every wave fetches the 32 order entries of a half tile one step ahead of its K/V requests (one
// more 4-byte-per-lane DMA per step, into a small LDS ring that only this wave reads), turns them into byte offsets where they
// lie, once per step, and adds them to the per-lane offsets of its DMA instructions; the epilogue stores each row at its raster position.
// (The entries read and multiplied anew for each of a step's sixteen DMA instructions, in front of the MFMAs, took 24 % more clocks than
// the kernel for cube-major tensors; and the order entries of Q and of the output rows were loaded one after the other, 2.5 + 4.4 us a
// workgroup.  12 heads, 51 of 512 blocks 764 -> 734 us, cubes 62 of 624 1056 -> 1014; cube-major 667.)
template <int D, bool OUT_F32, int WPS, bool RASTER, bool DEEP, bool TURNS>
__global__ __launch_bounds__(64 * NW, WPS) void attn_wide(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                                                          const uint16_t* __restrict__ v, const int32_t* __restrict__ idx,
                                                          const int32_t* __restrict__ cnt, void* __restrict__ out,
                                                          float* __restrict__ lse, int nb, int Nv, int kmax,
                                                          float scale_log2e, float p_shift, int total, int per_xcd,
                                                          FuseArgs fuse, RasterArgs ras,
                                                          const int32_t* __restrict__ work_order, int stream_out,
                                                          int sweep_wgs, int rotate_short) {
  constexpr int KS = D / 32, DT = D / 16, OT = (DT + 3) / 4;  // channel steps, 16-channel tiles of O, their 16-register tuples
  constexpr int LINES = D / 64, IPS = 2 * LINES;              // 128-byte lines per row; items per step
  constexpr int SLOTS = IPS + (DEEP ? 1 : 0);                 // ring slots
  constexpr int KF = 3, VF = 2;                               // fragments of K, V in flight
  constexpr int kRowBytes = D * 2;
  constexpr int XROWS = DT * 8 + 4;  // exchange rows of 64 floats per wave: O of two query tiles, reference and sum of both
  constexpr int OSTRIDE = D + 4;     // fp32 staging row stride (floats), bank-spread
  constexpr int kWaveBytes = SLOTS * kItem > XROWS * 256 ? SLOTS * kItem : XROWS * 256;  // ring, later the exchange area
  static_assert(XROWS * 64 >= 32 * OSTRIDE, "the staging rows of 32 queries overlay an exchange area");
  static_assert(kWaveBytes % 1024 == 0, "fragment addresses are formed with XOR below bit 10");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * kWaveBytes];
  // raster mode at d = 128 has no registers left for the whole of Q: the fragments of the last QL query tiles' last channel
  // step are read back from LDS
  constexpr int QL = RASTER && D == 128 ? 4 : 0;
  __shared__ __attribute__((aligned(16))) unsigned char q_tail[QL > 0 ? QL * 1024 : 16];
  __shared__ __attribute__((aligned(256))) int ord_ring[RASTER ? NW * 64 : 1];  // per wave: two half tiles' order entries

  const int work = xcd_contiguous_id(blockIdx.x, per_xcd);
  if (work >= total) return;  // whole workgroup leaves before any barrier
  const long long head = work / nb;
  // which query block of the head this workgroup takes: its slot number, or what the caller's work order puts there
  int i = work % nb;
  if (work_order) i = min(max(work_order[work], 0), nb - 1);
  const long long row_id = head * nb + i;
  const long long head_off = head * (long long)nb * kBlock * D;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform by construction; keep it scalar
  const int c16 = lane & 15, G = lane >> 4;
  const int n_list = min(max(cnt[row_id], 0), kmax);  // device contents are not trusted with addresses:
  const int32_t* list = idx + row_id * kmax;
  // valid query rows of this block: the first nq of its 64 positions hold tokens
  int nq = min(kBlock, max(0, Nv - i * kBlock));
  if constexpr (RASTER)
    if (ras.block_valid) nq = min(kBlock, max(0, ras.block_valid[i]));
  long long ras_off = 0, ras_out = 0;  // raster mode: byte bases of this (batch, head)
  if constexpr (RASTER) {
    const long long b = head / ras.Hh, h = head - b * ras.Hh;
    ras_off = b * ras.batch + h * ras.head;
    ras_out = b * ras.o_batch + h * ras.o_head;
  }
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(k) + (RASTER ? ras_off : head_off * 2 + wave * 32 * kRowBytes);
  const unsigned char* vbase = reinterpret_cast<const unsigned char*>(v) + (RASTER ? ras_off : head_off * 2 + wave * 32 * kRowBytes);

  // DMA lane -> stored row lane / 8 of an instruction's 8 rows, stored 16-byte chunk lane % 8 of the line
  const int drow = D == 128 ? ((lane >> 3) & 3) + 16 * (lane >> 5) : lane >> 3;  // row of instruction r: drow + (D == 128 ? 4 : 8) r
  int kofs = (RASTER ? 0 : drow * kRowBytes) + (((lane & 7) ^ (lane >> 4)) << 4);
  const int vofs = (RASTER ? 0 : drow * kRowBytes) + (((lane & 7) ^ (((lane >> 4) & 3) << 1)) << 4);
  const unsigned wave_lds = lds_address(smem) + wave * kWaveBytes;
  int* const my_ord = ord_ring + (RASTER ? wave * 64 : 0);
  // raster mode: byte offsets of the rows this lane fetches in its DMA instructions for step n (the same rows of K and of V)
  unsigned row_at[RASTER ? 4 : 1];
  auto read_order = [&](int n) {
    if constexpr (RASTER) {
      const int* p = my_ord + (n & 1) * 32 + drow;
#pragma unroll
      for (int r = 0; r < 4; ++r) row_at[r] = p[r * (D == 128 ? 4 : 8)];
    }
  };
  auto scale_order = [&]() {
    if constexpr (RASTER) {
#pragma unroll
      for (int r = 0; r < 4; ++r) row_at[r] *= (unsigned)ras.tok;
    }
  };
  // item x of tile j (step n): x < LINES: line x of K, else line x - LINES of V
  auto dma = [&](auto x_c, int j, int n, unsigned at) {
    constexpr int x = decltype(x_c)::value;
    const unsigned lds = wave_lds + at;
    const unsigned char* base = (x < LINES ? kbase : vbase) + (x % LINES) * 128;
    if constexpr (x < LINES) asm volatile("" : "+v"(kofs));  // (the odd half is one XOR here, not a register)
    if constexpr (RASTER) {
      const unsigned even = x < LINES ? kofs : vofs, odd = x < LINES ? kofs ^ 64 : vofs;
      dma_half<0>(lds, base, row_at[0] + even + kBack, row_at[1] + odd + (kBack - 1024));
      dma_half<1>(lds, base, row_at[2] + even + (kBack - 2048), row_at[3] + odd + (kBack - 3072));
    } else {
      base += (long long)j * (kBlock * kRowBytes);
      if constexpr (x < LINES) dma_item(lds, base, kofs, kofs ^ 64);
      else dma_item(lds, base, vofs, vofs);
    }
  };
  // raster mode: the 32 order entries of this wave's half of tile j, step n -> slot n % 2 of its ring
  auto request_order = [&](int j, int n) {
    if constexpr (RASTER) {
      const int ln = lane_again();
      if (ln < 32) {
        const unsigned dst = lds_address(my_ord) + (n & 1) * 128;
        const int32_t* src = ras.order + (long long)j * kBlock + wave * 32;
        const int voff = ln * 4;
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" : : "s"(dst), "v"(voff), "s"(src) : "memory");
      }
    }
  };

  // raster mode: where this lane's four query rows lie
  int q_order[RASTER ? 4 : 1];
  if constexpr (RASTER) {
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) q_order[nt] = ras.order[i * kBlock + 16 * nt + c16];
  }

  // ---- where the list starts -------------------------------------------------------------------
  // The workgroups of an XCD that run together share fetched tiles through its L2 as long as their sweeps over the
  // head's keys stay together.  Starting every list at its first entry keeps them together in the first round only: later
  // workgroups start whenever a slot frees, and those times spread from round to round (measured with TURNS at 12 heads, 512 blocks, 51
  // listed, as a share of one sweep: 0.18 at m = 1 (m as below), 0.28, 0.37, 0.47, 0.54 at m = 5; 40 heads of 1182 blocks 0.19 to 0.8
  // at m = 6, where it stays).  So a workgroup starts its sweep where the others can be expected to be at its time.  The
  // k-th of the sweep_wgs of round m = rank / sweep_wgs starts before or after the round's middle by its share of that
  // spread, and the middles of all rounds meet the same place of the sweep: the list is walked from the first block at or past
  // nb * width(m) * (k / sweep_wgs - 1/2), modulo nb, around the end, back to it.  Without turns the oldest wave of a SIMD runs ahead, the first
  // quarter of a round starts far ahead of the rest, and a place counted from the round's first start is the better guess.
  // A pure function of the launch: same bits every time; but the first tile sets the reference that a row's weights are
  // rounded to bf16 against, so in another slot of a launch (or with another kmax) the same list may give a result that
  // differs by that rounding.
  // Measured (start at 0 -> without turns -> with): 512 blocks x 12, 51 listed 800 -> 699 -> 661 us, 25 listed 487 -> 400 -> 385, 624 x 12,
  // 62 listed 1078 -> 1006, 800 x 12, 64 listed 1635 -> 1396, 1182 x 40, 59 listed 10.8 -> 7.70 -> 6.99 ms.  A width of 0.25 / 0.3 / 0.35 sqrt(m):
  // 673 / 673 / 678 us, 398 / 385 / 383, 993 / 1006 / 1024, 1374 / 1396 / 1449, 7.25 / 7.00 / 6.92 ms; without turns spread 0.3 / 0.4 / 0.5 / 0.6
  // / 0.8 sqrt(m) from the first start: 722 / 713 / 712 / 717 / 727 us.
  int first = 0;  // entry the sweep starts with
  int list_v;     // lane t: block of step 64 (n / 64) + t
  {
    const int raw = lane < kmax ? list[lane] : 0;  // (whatever the count says: this load does not wait for the count's)
    int pos = 0;
    if (sweep_wgs > 0 && (rotate_short || n_list == kmax)) {
      const int rank = blockIdx.x / kNumXcd, m = rank / sweep_wgs;
      const float width = fminf(1.0f, (TURNS ? 0.3f : 0.5f) * __builtin_amdgcn_sqrtf((float)m));
      float at = width * ((float)(rank - m * sweep_wgs) / (float)sweep_wgs - (TURNS ? 0.5f : 0.f));
      if (at < 0.f) at += 1.0f;
      pos = (int)(at * (float)nb);
    }
    pos = __builtin_amdgcn_readfirstlane(pos);
    if (pos > 0 && n_list > 0) {  // entries below pos, of an ascending list (of any other list: some entry)
      if (n_list <= 64) {
        first = __popcll(__builtin_amdgcn_ballot_w64(lane < n_list && raw < pos));
      } else {  // 64 samples, then the stretch between two of them
        const int at = (int)((long long)lane * n_list / 64);
        const int below = __popcll(__builtin_amdgcn_ballot_w64(list[at] < pos));
        if (below > 0) {
          const int lo = (int)((long long)(below - 1) * n_list / 64), hi = (int)((long long)below * n_list / 64);
          const bool in = lo + lane < hi;
          first = lo + __popcll(__builtin_amdgcn_ballot_w64(in && list[in ? lo + lane : lo] < pos));
        }
      }
      if (first >= n_list) first = 0;
    }
    first = __builtin_amdgcn_readfirstlane(first);
    int e = lane + first;
    if (e >= n_list) e -= n_list;
    int j;
    if (n_list <= 64) j = __shfl(raw, e & 63);
    else j = list[e];
    list_v = lane < n_list ? min(max(j, 0), nb - 1) : 0;  // ids are clamped into [0, nb)
  }
  // raster mode: the valid keys of every listed block travel in the upper half beside its id
  auto load_valid = [&]() {
    if constexpr (RASTER)
      list_v |= (ras.block_valid ? min(kBlock, max(0, ras.block_valid[list_v])) : min(kBlock, max(0, Nv - list_v * kBlock))) << 16;
  };
  load_valid();
  auto list_at = [&](int n) { return __builtin_amdgcn_readlane(list_v, n & 63); };
  auto id_of = [&](int e) { return RASTER ? e & 0xffff : e; };

  // tile ids of steps n, n + 1, n + 2 (steps past the end read as some block, unused)
  int j0 = list_at(0), j1 = list_at(1), j2 = list_at(2);
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  if (n_list > 0) {
    if constexpr (RASTER) {
      request_order(id_of(j0), 0);
      if (n_list > 1) request_order(id_of(j1), 1);
      wait_vm<0>();
      read_order(0);
      scale_order();
    }
    dma(I0{}, j0, 0, 0 * kItem);
    dma(I1{}, j0, 0, 1 * kItem);
    if constexpr (IPS == 4) {
      dma(I2{}, j0, 0, 2 * kItem);
      dma(I3{}, j0, 0, 3 * kItem);
    }
    if constexpr (DEEP)
      if (n_list > 1) dma(I0{}, j1, 1, IPS * kItem);
  }

  // Q fragments: for query tile nt the lane holds query row 16 nt + c16, channels 32 t + 8 G .. + 8 for every step t
  bf16x8 qf[4][KS];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    const int qrow = i * kBlock + 16 * nt + c16;
    const uint16_t* qp = q + head_off + (long long)qrow * D + G * 8;
    if constexpr (RASTER)
      qp = reinterpret_cast<const uint16_t*>(reinterpret_cast<const unsigned char*>(q) + ras_off +
                                             (long long)q_order[nt] * ras.tok) + G * 8;
#pragma unroll
    for (int t = 0; t < KS; ++t) qf[nt][t] = *reinterpret_cast<const bf16x8*>(qp + t * 32);
  }
  if constexpr (RASTER) {
    // padding positions have no token: their query rows are zero, as in a gathered copy (their lanes
    // take part in the wave-wide rescale decisions, so what they hold is not quite without effect)
    if (nq < kBlock) {  // (after all the loads: a branch between them would wait for each)
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const unsigned keep = 16 * nt + c16 < nq ? ~0u : 0u;
#pragma unroll
        for (int t = 0; t < KS; ++t) {
          typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
          qf[nt][t] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[nt][t]) & u32x4{keep, keep, keep, keep});
        }
      }
    }
  }
  if constexpr (QL > 0) {  // (both key halves write the same values, and a wave reads back what it wrote itself)
#pragma unroll
    for (int e = 0; e < QL; ++e) *reinterpret_cast<bf16x8*>(q_tail + e * 1024 + lane * 16) = qf[4 - QL + e][KS - 1];
  }
  // O^T accumulators: quarter dt % 4 of o[nt][dt / 4], element r = channel 16 dt + 4 G + r of query 16 nt + c16
  f32x16 o[4][OT];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int x = 0; x < OT; ++x)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[nt][x][r] = 0.f;
  // Per query tile (this lane's four queries).  nm = -(reference maximum) - p_shift in the log2 domain, identical in the four
  // lanes of its query, kNoKey while no key has been seen (the first live key raises it, whatever its logit: with the largest
  // float here no finite logit is beyond it, and a masked one still gives 2^-inf = 0); l = this lane's partial row sum (its 8
  // keys per step).
  float nm[4], l[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) nm[nt] = kNoKey, l[nt] = 0.f;
  const float raise_at = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(kRescaleSlack - p_shift)));

  // Lane bases of the fragment reads; what else an address needs is an immediate or one XOR.
  // K fragment (mt, t): stored row 16 mt + c16, chunks 4 t + G; a line's chunks are stored at chunk ^ (row / 2 % 8)
  unsigned kl = wave * kWaveBytes + (c16 >> 3) * 1024 + (c16 & 7) * 128 + ((G ^ (c16 >> 1)) << 4);
  // V^T fragment of d tile dt: contraction slots 0..3 are stored rows 4 G + (0..3), slots 4..7 rows 16 + 4 G + (0..3) (the
  // order in which the S^T accumulators hold the keys); the 16 lanes of a group address the 4 rows x 16 channels that the
  // transposing read hands out column by column; chunks are stored at chunk ^ 2 (row / 2 % 4)
  unsigned vl = wave * kWaveBytes + (G >> 1) * 1024 + (4 * (G & 1) + (c16 >> 2)) * 128 +
                ((((c16 >> 1) & 1) ^ (((2 * (G & 1) + (c16 >> 3)) & 3) << 1)) << 4) + (c16 & 1) * 8;

  wait_vm<0>();  // the first half tile and Q have landed
  // pin the Q fragments here: otherwise the compiler sinks their loads into the loop and then waits
  // for "all outstanding loads" there, which would also wait for the requests it cannot see
#pragma unroll
  for (int nt = 0; nt < 4; ++nt)
#pragma unroll
    for (int t = 0; t < KS; ++t)
      if (t < KS - 1 || nt < 4 - QL) asm volatile("" : "+v"(qf[nt][t]));

  // blocks from this one on hold padded keys: the partial block (if Nv is not a multiple of 64) and, when the
  // tensors are padded by whole blocks, every block behind it.  A caller's list may name those too: all of
  // their keys are masked, as the masked-attention equation has it (they then add nothing to the row).
  // (raster mode carries the valid key count of every listed block beside its id instead)
  const int first_padded_j = Nv / kBlock;

  // One half tile.  LAST: there is no next one to request.
  int ring[SLOTS];  // byte offset of the slot of item x of the current step; DEEP: [IPS] that of item 0 of the next
#pragma unroll
  for (int x = 0; x < SLOTS; ++x) ring[x] = x * kItem;
  auto step = [&](auto last_c, int n) {
    constexpr bool LAST = decltype(last_c)::value;
    if constexpr (RASTER && !LAST)
      if (n + 2 < n_list) request_order(id_of(j2), n + 2);
    // Item x of this step is in LDS.  Younger requests: the items behind it of this step and those of the next step that
    // have been asked for by then (the second line of K, or of V, is awaited just before its first line's refill).
    // (Raster mode: and one request for order entries; leaving it out of the count only makes the wait stricter.)
    auto await = [&](auto x_c) {
      constexpr int x = decltype(x_c)::value;
      wait_vm<(LAST ? IPS - 1 - x : LINES == 2 && (x & 1) ? SLOTS - 2 : SLOTS - 1) * 4>();
    };
    // every fragment of item x is in registers: its slot takes item x of the next half tile
    auto refill = [&](auto x_c) {
      constexpr int x = decltype(x_c)::value;
      if constexpr (!LAST && x < IPS) {
        if constexpr (!DEEP) dma(x_c, j1, n + 1, ring[x]);
        else if constexpr (x + 1 < IPS) dma(std::integral_constant<int, x + 1>{}, j1, n + 1, ring[x]);
        else if (n + 2 < n_list) dma(I0{}, j2, n + 2, ring[x]);
      }
    };

    // ---- S^T = K Q^T: s[mt], quarter nt = tile (mt, nt) ----
    f32x16 s[2];
    asm volatile("" : "+v"(kl), "+v"(vl));  // keeps the XORs in the loop (hoisted, they are registers this kernel has not got)
    bf16x8 kf[KF], ql[QL > 0 ? QL : 1];
    auto read_k = [&](int f) {  // fragment f = 2 t + mt
      kf[f % KF] = *reinterpret_cast<const bf16x8*>(smem + ((kl + ring[f >> 2]) ^ (((f >> 1) & 1) << 6)) + (f & 1) * 2048);
    };
    await(I0{});
    if constexpr (!LAST) read_order(n + 1);  // (asked for before this step's first item was: they are there)
#pragma unroll
    for (int f = 0; f < KF - 1; ++f) read_k(f);
#pragma unroll
    for (int f = 0; f < 2 * KS; ++f) {
      if (LINES == 2 && f + KF - 1 == 4) await(I1{});
      if (f + KF - 1 < 2 * KS) read_k(f + KF - 1);
      if (f == 1 && !LAST) scale_order();
      if (f == 3) {
        wait_lds<(LINES == 2 ? KF - 1 : 0)>();  // (LDS reads return in order)
        refill(I0{});
      }
      if (LINES == 2 && f == 2 * KS - 2) {
        wait_lds<0>();
        refill(I1{});
      }
      if (QL > 0 && f == 2 * KS - 2) {  // (for the last two fragments)
        const unsigned ql_at = lane_again() * 16;
#pragma unroll
        for (int e = 0; e < QL; ++e) ql[e] = *reinterpret_cast<const bf16x8*>(q_tail + ql_at + e * 1024);
      }
      // the fences keep the order written here: a read two fragments ahead, then the MFMAs of this one
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        set_quarter(s[f & 1], nt,
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[f % KF], QL > 0 && f >= 2 * KS - 2 && nt >= 4 - QL ? ql[nt >= 4 - QL ? nt - (4 - QL) : 0] : qf[nt][f >> 1], f < 2 ? zero : quarter(s[f & 1], nt), 0, 0, 0));
      }
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" : "+v"(s[f & 1]));  // in place (see quarter())
    }

    // s[mt][4 nt + r] of lane (c16, G) is stored row 16 mt + 4 G + r, query 16 nt + c16
    if (RASTER ? (j0 >> 16) < kBlock : j0 >= first_padded_j) {
      int ln = RASTER ? lane_again() : __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
      float ninf = -INFINITY;
      asm volatile("" : "+v"(ln), "+v"(ninf));  // formed here, on the rare path, instead of kept in registers
      const int g = ln >> 4;
      // valid keys of the tile ahead of this lane's first; stored row -> key as the DMA lays them out
      const int lim = (RASTER ? j0 >> 16 : Nv - j0 * kBlock) - (wave * 32 + (D == 128 ? 16 * (g & 1) + 4 * (g >> 1) : 4 * g));
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            s[mt][4 * nt + r] = ((D == 128 ? 8 : 16) * mt + r) < lim ? s[mt][4 * nt + r] : ninf;
    }

    // ---- online softmax (log2 domain, lazily raised reference max) ----
    // The raise test needs no cross-lane step: if no lane holds a value above its query's threshold,
    // no query has one.  Only a raise itself (rare) takes the maximum over the four lanes of a query.
    float mx[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
      mx[nt] = max8(s[0][4 * nt], s[0][4 * nt + 1], s[0][4 * nt + 2], s[0][4 * nt + 3], s[1][4 * nt], s[1][4 * nt + 1],
                    s[1][4 * nt + 2], s[1][4 * nt + 3]);
    float over = fmaf(mx[0], scale_log2e, nm[0]);
#pragma unroll
    for (int nt = 1; nt < 4; ++nt) over = fmaxf(over, fmaf(mx[nt], scale_log2e, nm[nt]));
    if (__any(over > raise_at)) {  // wave-uniform; always taken on the first live step
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const float nm_new = fminf(nm[nt], -max_over_groups(mx[nt]) * scale_log2e - p_shift);
        const float alpha = fast_exp2(nm_new - nm[nt]);  // nm = kNoKey -> 0
        nm[nt] = nm_new;
        l[nt] *= alpha;
#pragma unroll
        for (int x = 0; x < OT; ++x)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[nt][x][r] *= alpha;
      }
    }
    // P^T, rounded to bf16 and packed two per register: per query the same four registers feed the row sum (v_dot2 with
    // ones) and, as they stand, the B operand of the second product
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned uint4v;
    bf16x8 pf[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      bf16x2 pk[4];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          pk[2 * mt + (r >> 1)][0] = (__bf16)fast_exp2(fmaf(s[mt][4 * nt + r], scale_log2e, nm[nt]));
          pk[2 * mt + (r >> 1)][1] = (__bf16)fast_exp2(fmaf(s[mt][4 * nt + r + 1], scale_log2e, nm[nt]));
        }
      // the row sum is taken over the ROUNDED probabilities, the ones P V actually uses, so that
      // the final division cancels the rounding of a dominant key instead of keeping it
      bf16x2 ones;
      ones[0] = (__bf16)1.0f;
      ones[1] = (__bf16)1.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) l[nt] = __builtin_amdgcn_fdot2_f32_bf16(pk[r], ones, l[nt], false);
      const uint4v w = {__builtin_bit_cast(unsigned, pk[0]), __builtin_bit_cast(unsigned, pk[1]),
                        __builtin_bit_cast(unsigned, pk[2]), __builtin_bit_cast(unsigned, pk[3])};
      pf[nt] = __builtin_bit_cast(bf16x8, w);
    }

    // ---- O^T += V^T P^T: one MFMA per (d tile, query tile), its 32 contraction slots = this step's keys ----
    bf16x8 vf[VF];
    auto read_v = [&](int dt) {
      const unsigned char* p = smem + ((vl + ring[LINES + (dt >> 2)]) ^ ((dt & 3) << 5));
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)p);
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(p + 2048));
      const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      __builtin_memcpy(&vf[dt % VF], &both, sizeof(bf16x8));
    };
    await(std::integral_constant<int, LINES>{});
#pragma unroll
    for (int dt = 0; dt < VF - 1; ++dt) read_v(dt);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      if (LINES == 2 && dt + VF - 1 == 4) await(I3{});
      if (dt + VF - 1 < DT) read_v(dt + VF - 1);
      if (dt == 3) {
        wait_lds<(LINES == 2 ? 2 * (VF - 1) : 0)>();
        refill(std::integral_constant<int, LINES>{});
      }
      if (LINES == 2 && dt == DT - 1) {
        wait_lds<0>();
        refill(I3{});
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
        set_quarter(o[nt][dt >> 2], dt & 3,
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt % VF], pf[nt], quarter(o[nt][dt >> 2], dt & 3), 0, 0, 0));
      __builtin_amdgcn_sched_barrier(0);
    }
    // pin each accumulator tuple to one 16-register unit once per step (see quarter())
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int x = 0; x < OT; ++x) asm volatile("" : "+v"(o[nt][x]));

    if constexpr (!LAST) {
      j0 = j1;
      j1 = j2;
      if (((n + 3) & 63) == 0) {  // the next 64 entries; awaited right here (once in 64 steps) so that the hot path
        int t = RASTER ? lane_again() : __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));  // carries no vector-memory wait
        asm volatile("" : "+v"(t));
        t += n + 3;
        int e = t + first;
        if (e >= n_list) e -= n_list;
        list_v = t < n_list ? min(max(list[e], 0), nb - 1) : 0;
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(list_v)::"memory");
        if constexpr (RASTER) {
          load_valid();
          asm volatile("s_waitcnt vmcnt(0)" : "+v"(list_v)::"memory");
        }
      }
      j2 = list_at(n + 3);
    }
  };
  {
    // Taking turns: between equals the SIMD issues from its oldest wave first, so of the WPS waves that share one the oldest runs
    // ahead (measured at d = 128: 85 us a list against 110) and the sweeps of an XCD part already in the first round.  Where
    // their staying together counts, a wave's priority goes round with its steps, counted from its slot: whoever is ahead is
    // overtaken.  (Durations in the first round 120 +- 13 -> 113 +- 6 us.  Where the L2 serves the tiles anyway the old order
    // is the better one, as it keeps prologues and epilogues apart: all 512 blocks listed 5.73 / 5.93 ms.)
    unsigned turn = TURNS ? __builtin_amdgcn_s_getreg(4 | (3 << 11)) : 0;  // HW_ID, bits 0..3: the wave's slot of its SIMD
    if (WPS == 3) turn %= 3;
    int n = 0;
    for (; n + 1 < n_list; ++n) {
      if constexpr (TURNS) {
        if (WPS == 2 ? turn & 1 : turn == 1) __builtin_amdgcn_s_setprio(1);
        else if (WPS == 3 && turn == 2) __builtin_amdgcn_s_setprio(2);
        else __builtin_amdgcn_s_setprio(0);
        ++turn;
        if (WPS == 3 && turn == 3) turn = 0;
      }
      step(std::false_type{}, n);
      if constexpr (DEEP) {  // item x + 1 of the next step went where item x of this one was
        const int spare = ring[SLOTS - 1];
#pragma unroll
        for (int x = SLOTS - 1; x > 0; --x) ring[x] = ring[x - 1];
        ring[0] = spare;
      }
    }
    if (n < n_list) step(std::true_type{}, n);
  }

  // ---- merge the two waves' partial results, stage the rows row-major in LDS, store coalesced ------
  // Wave w finishes query tiles 2 w and 2 w + 1.  It gives the other two away through its own ring (dead by now:
  // everything requested has landed and been read), adds what the other wave gave, and stages its rows where it has just read.
  float l_row[4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) l_row[nt] = sum_over_groups(l[nt]);
  int my_order = 0;  // raster mode: lane r holds where the wave's row r % 32 lies; asked for here, used behind the exchange
  if constexpr (RASTER) my_order = ras.order[i * kBlock + 32 * wave + (lane & 31)];
  auto give = [&](auto first_c) {
    constexpr int F = decltype(first_c)::value;
    float* dst = reinterpret_cast<float*>(smem + wave * kWaveBytes) + lane;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[((e * DT + dt) * 4 + r) * 64] = o[F + e][dt >> 2][4 * (dt & 3) + r];
      dst[(DT * 8 + e) * 64] = nm[F + e];
      dst[(DT * 8 + 2 + e) * 64] = l_row[F + e];
    }
  };
  auto take = [&](auto first_c) {
    constexpr int F = decltype(first_c)::value;
    float* area = reinterpret_cast<float*>(smem + (wave ^ 1) * kWaveBytes);
    const float* src = area + lane;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float n1 = src[(DT * 8 + e) * 64], l1 = src[(DT * 8 + 2 + e) * 64];
      const float ref = fminf(nm[F + e], n1);
      const float a0 = fast_exp2(ref - nm[F + e]), a1 = fast_exp2(ref - n1);  // (a side without keys: l = 0, O = 0)
      const float lt = l_row[F + e] * a0 + l1 * a1;
      const int row = 16 * (F + e) + c16;
      const bool live = row < nq && lt > 0.f;  // lt == 0: empty list, or every listed key is padding
      const float inv = live ? 1.f / lt : 0.f;
      const float w0 = live ? a0 * inv : 0.f, w1 = live ? a1 * inv : 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float val = o[F + e][dt >> 2][4 * (dt & 3) + r] * w0 + src[((e * DT + dt) * 4 + r) * 64] * w1;
          o[F + e][dt >> 2][4 * (dt & 3) + r] = live ? val : 0.f;
        }
      if (lse && G == 0) {
        const float val = live ? (__log2f(lt) - ref) * kLn2 : -INFINITY;  // (ref carries p_shift, as lt does)
        if constexpr (RASTER) {  // [B, Hh, Nv] in raster order; padded rows have no place there
          if (row < nq) lse[head * (long long)Nv + ras.order[i * kBlock + row]] = val;
        } else {
          lse[head * (long long)nb * kBlock + i * kBlock + row] = val;
        }
      }
    }
    wait_lds<0>();  // every exchange value of this wave is in registers before its area is overwritten
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float* stage = area + (16 * e + c16) * OSTRIDE;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const f32x16& t = o[F + e][dt >> 2];
        const int x = 4 * (dt & 3);
        *reinterpret_cast<float4*>(stage + 16 * dt + 4 * G) = make_float4(t[x], t[x + 1], t[x + 2], t[x + 3]);
      }
    }
  };
  float* other = reinterpret_cast<float*>(smem + (wave ^ 1) * kWaveBytes);
  if (wave == 0) give(I2{});
  else give(I0{});
  __syncthreads();
  if (wave == 0) take(I0{});
  else take(I2{});
  const long long blk_off = head_off + (long long)i * kBlock * D;
  // 32 rows x D channels, 4 (second branch: 8) channels per lane per pass, consecutive lanes -> consecutive addresses (the
  // rows this wave staged itself: no barrier)
  auto out_row = [&](int row) -> unsigned char* {
    if constexpr (RASTER)
      return static_cast<unsigned char*>(out) + ras_out + (long long)__shfl(my_order, row & 31) * ras.o_tok;
    else
      return static_cast<unsigned char*>(out) + (blk_off + row * D) * (OUT_F32 ? 4 : 2);
  };
  if (fuse.coarse) {
    // Second branch.  Piece p = 64 it + lane: row p / (D / 8) of the wave's 32, channels c8 .. c8 + 7, the same channels in
    // every pass.  All of the wave's gate rows are requested before the first store: left to the passes, each of them waited
    // for its own two loads (12 heads, 32768 tokens, 51 of 512 blocks, both gates, the whole two-branch layer: 878 -> 822 us).
    constexpr int PIECES8 = 32 * D / 8 / 64;
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned gate8;
    const int c8 = (lane % (D / 8)) * 8;
    gate8 gf[PIECES8], gc[PIECES8];
    float4 cz[2];
#pragma unroll
    for (int it = 0; it < PIECES8; ++it) {
      const int row = 32 * wave + (it * 64 + lane) / (D / 8);
      long long at = blk_off + row * D + c8;  // (padded rows are there to be read; a padding position's order entry is a valid token)
      if constexpr (RASTER)  // the gates are raster tensors laid out like q
        at = (ras_off + (long long)__shfl(my_order, row & 31) * ras.tok) / 2 + c8;
      constexpr unsigned kOnes = 0x3f803f80u;  // an absent gate is 1
      gf[it] = gc[it] = gate8{kOnes, kOnes, kOnes, kOnes};
      if (fuse.gate_fine) gf[it] = __builtin_nontemporal_load(reinterpret_cast<const gate8*>(fuse.gate_fine + at));
      if (fuse.gate_coarse) gc[it] = __builtin_nontemporal_load(reinterpret_cast<const gate8*>(fuse.gate_coarse + at));
    }
    {
      const float* row = fuse.coarse + (head * nb + i) * (long long)D + c8;
      cz[0] = reinterpret_cast<const float4*>(row)[0];
      cz[1] = reinterpret_cast<const float4*>(row)[1];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < PIECES8; ++it) {
      const int rr = (it * 64 + lane) / (D / 8), row = 32 * wave + rr;
      unsigned char* const dst = out_row(row) + c8 * (OUT_F32 ? 4 : 2);  // (ahead of the branch: it reads other lanes)
      if (RASTER && row >= nq) continue;  // the raster tensor has no padded rows
      float4 val[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        val[e] = *reinterpret_cast<const float4*>(other + rr * OSTRIDE + c8 + 4 * e);
        if (row < nq) fuse4(val[e], bf16_pair(gf[it][2 * e], gf[it][2 * e + 1]), bf16_pair(gc[it][2 * e], gc[it][2 * e + 1]), cz[e]);
      }
      store8<OUT_F32>(dst, val, stream_out);
    }
  } else {
    constexpr int PIECES = 32 * D / 4;
#pragma unroll
    for (int it = 0; it < PIECES / 64; ++it) {
      const int id = it * 64 + lane;
      const int rr = id / (D / 4), row = 32 * wave + rr, c4 = (id % (D / 4)) * 4;
      unsigned char* const dst = out_row(row) + c4 * (OUT_F32 ? 4 : 2);
      if (RASTER && row >= nq) continue;
      const float4 val = *reinterpret_cast<const float4*>(other + rr * OSTRIDE + c4);
      store4<OUT_F32>(dst, val, stream_out);
    }
  }
}

template <int D, bool OUT_F32, bool RASTER>
hipError_t run(const AttnBf16Args& a, hipStream_t st) {
  const Dims& s = a.s;
  const long long total = s.bh() * s.nb;
  const int per_xcd = (int)((total + kNumXcd - 1) / kNumXcd);
  constexpr int WPS = D == 128 ? 2 : 3;                          // waves per SIMD the registers allow
  constexpr int kSweepWgs = 256 / kNumXcd * (WPS * 4 / NW);      // workgroups of an XCD (32 CUs) that run together
  const long long kv_head = 4LL * s.nb * kBlock * D;             // bytes of one head's K and V
  // Lists that keep more than a fifth of the blocks stay together by themselves (whoever is ahead misses the L2 and is held
  // up): start at the expected place / start at the first entry: 43 of 256 blocks 553 / 568 us, 51 of 256 639 / 650, 64 of 256
  // 789 / 783, 85 of 512 1037 / 1140, 102 of 512 1245 / 1260, 128 of 512 1558 / 1535, 170 of 512 2051 / 1980.  In index order, heads
  // beyond the L2 need more to stay together: 12 heads of 700 blocks, 175 listed 0.78 of the time, 800, 168 0.75, 900, 225
  // 0.71, 1182, 248 0.73, 900 x 3, 297 0.93; 40 % listed: 800 x 12 1.04, 900 x 3 0.97, 1182 x 3 1.08.
  // Time with starts and turns (below), as a multiple of that from the first entry, where a small rest follows two rounds, index order, 35 % listed:
  // 600 x 4 1.05, 720 x 3 1.05, 800 x 3 1.02, 1024 x 2 1.07, but 1060 to 1230 x 2 0.83 to 0.98; in a work order, 19 %: lists of equal lengths 1024 x 2 1.15, x 3 1.10, x
  // 4 1.04, ragged ones 0.84, 0.80; 900 x 3 0.93.
  const long long k = a.kmax, nb = s.nb, round = wide_round(s);
  const bool sweep = a.work_order ? (full_rounds(s) ? 6 : 5) * k <= nb
                                  : 5 * k <= nb || (D == 128 && nb > 512 && nb <= 1280 && 5 * k < 2 * nb &&
                                                    !(nb <= 1024 && total >= 2 * round && 5 * total < 12 * round));
  // Taking turns keeps sweeps together, and it lets all workgroups of a round end at once: a part of a round behind them runs
  // alone.  So it pays on long heads, and on many rounds.  Time with turns, as a multiple of the time without; d = 128, 4 % / 8 / 14 / 19.5 of the
  // blocks listed: 160 blocks x 28 1.05 / 1.03 / 1.02 / 1.03, x 45 1.02 / 1.02 / 1.00 / 1.00; 230 x 10 0.98 / 1.02 / 1.05 / 1.07; 300 x 8 1.01 / 1.04 / 1.06 / 1.10, x 24 1.00 / 1.00 / 1.01 / 1.01; 512 x 4 0.95 / 1.06 / 1.09 / 1.09, x 9 0.94 / 0.93 / 0.99 / 1.00, x 14 0.97 /
  // 0.98 / 0.98 / 0.98; 620 x 3 0.93 / 0.88 / 0.93 / 0.92, x 12 0.97 / 0.91 / 0.93 / 0.90.  d = 64: 512 x 21 1.02 / 1.02 / 1.04 / 1.03, 620 x 17
  // 1.02 / 1.04 / 1.02 / 1.02, 1182 x 8, 100 listed 0.98.
  // Up to 640 blocks it does not where half a round or less follows two full ones, on lists of more than an eighth (600 x 4, 13 % / 19 % listed 1.04 / 1.05, 630 x
  // 4, 80 listed in a work order 1.06), nor up to 1024 where hardly anything follows, on lists of more than a sixth (712 x 3, 120 listed 1.03, 1024 x 2, 194 1.06; but 802 x
  // 3, 145 0.975), nor on short lists in index order in a single round of up to 860 (800 x 1, 64 listed 1.02; 1024 x 1, 81 0.91).  (d = 64 from 800 blocks on: 820 x 6, 4 % to 19 %
  // listed 1.01 to 1.03, but in a work order with ragged lists 831 x 6, 58 0.97, 847 x 51, 45 0.93.)
  const long long behind_two = total - 2 * round;
  const bool alone = behind_two >= 0 && ((nb <= 640 && 8 * k > nb && 2 * behind_two < round) || (nb <= 1024 && 6 * k > nb && 5 * behind_two < round));
  const bool one_short = total <= round && nb <= 860 && 8 * k <= nb && !a.work_order;
  const bool turns = sweep && !alone && !one_short && (D == 64 ? nb > 800 : nb > 560 || (nb > 256 && total > 4096));
  // Lists of different lengths sweep at different speeds.  In index order they gain as the others do (40 of 512 at most:
  // 492 / 521 us); a work order brings equal lengths together, which keeps them together as long as a head is not much
  // beyond the L2: 16.8 MB 2480 / 2078 us, but 38.7 MB 7270 / 8050 us and (d = 64) 19.4 MB 2809 / 3235 us.
  const int rotate_short = !a.work_order || kv_head > (18LL << 20);
  auto launch = [&](auto deep_c, auto turns_c) {
    attn_wide<D, OUT_F32, WPS, RASTER, decltype(deep_c)::value, decltype(turns_c)::value><<<(unsigned)per_xcd * kNumXcd, 64 * NW, 0, st>>>(
        static_cast<const uint16_t*>(a.q), static_cast<const uint16_t*>(a.k), static_cast<const uint16_t*>(a.v), a.idx,
        a.cnt, a.out, a.lse, s.nb, s.Nv, a.kmax, a.scale * kLog2e, probability_shift(a.kmax), (int)total, per_xcd, a.fuse,
        a.ras, a.work_order, stream_output(s), sweep ? kSweepWgs : 0, rotate_short);
  };
  // The extra slot costs a rotation of the ring offsets, 1.3 % where the L2 serves the requests (480p 709 -> 718 us), and
  // pays where it does not: 49152 tokens (25 MB) 1870 -> 1815 us, 75600 (38.7 MB) 8.09 -> 7.83 ms, 7.26 -> 7.21 with a work
  // order.  (At d = 64 it changes nothing; raster mode has no LDS left for it.)
  constexpr bool kCanDeep = D == 128 && !RASTER;
  using Deep = std::integral_constant<bool, kCanDeep>;
  const bool deep = kCanDeep && kv_head > (24LL << 20);
  if (turns) deep ? launch(Deep{}, std::true_type{}) : launch(std::false_type{}, std::true_type{});
  else deep ? launch(Deep{}, std::false_type{}) : launch(std::false_type{}, std::false_type{});
  return hipGetLastError();
}

template <bool RASTER>
hipError_t dispatch(const AttnBf16Args& a, bool d128, bool out_f32, hipStream_t st) {
  if (d128) return out_f32 ? run<128, true, RASTER>(a, st) : run<128, false, RASTER>(a, st);
  return out_f32 ? run<64, true, RASTER>(a, st) : run<64, false, RASTER>(a, st);
}

}  // namespace

hipError_t launch_attn_wide(const AttnBf16Args& a, bool out_f32, hipStream_t st) {
  return a.ras.order ? dispatch<true>(a, a.s.d == 128, out_f32, st) : dispatch<false>(a, a.s.d == 128, out_f32, st);
}

}  // namespace usv
