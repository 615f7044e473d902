// fp32 attention over [prefix cache | block | gathered suffix] (paper Eq. 8 and the paragraph
// after it).  Full fp32 arithmetic on the matrix cores (v_mfma_f32_16x16x4_f32: products and sums in fp32)
// with an accurate exp: the correctness-grade path (max-abs error <= 1e-5 against the fp64 definition).
//
// Work decomposition
//   group = (batch, KV head): the g * Nq query rows that share its K/V are one list of "virtual rows", cut into
//   16-row blocks.  A workgroup has NR x NK waves: wave (r, k) owns row block r of the workgroup and every NK-th
//   16-key block of the sequence; the NK partial (O, m, l) of a row block merge through LDS in a fixed order.
//   No wave shares an operand with another: V goes from global memory straight into registers in operand layout, K too or
//   through a region of LDS of the wave's own; there is no barrier in the loop.  Waves of a workgroup that own different rows
//   read the same key blocks at about the same time and meet in the L1.
// Operand layout (lane: l16 = lane % 16, G = lane / 16; a 16x16x4 operand is ONE float per lane, row / column l16,
// contraction index G)
//   S^T = K Q^T   the contraction runs over d in any order, so the four instructions of 16-element slice s take the
//                 components of one 16-byte load: d = 16 s + 4 G + j in instruction j.
//   O^T = V^T P^T lane (q = l16, G) of the S^T accumulators holds keys 4 G + i, which is the B operand of instruction
//                 i as it is; the A operand of output block (dg, j) is V[4 G + i][64 dg + 4 l16 + j], so one 16-byte
//                 load of a V row serves the four blocks j.
// What bounds it: the matrix pipe in principle (256 flop / cycle / CU in fp32, 157 TFLOP/s; two waves per SIMD cover each
// other's softmax and load latency), at layer sizes the fixed parts of a short launch.  Measured, B2, 32 query / 8 KV heads
// x 128, 64 query rows x 672 keys: 21.6 us (65 TFLOP/s) against 276 us for one query row per wave
// with fp32 FMAs out of LDS; B1, 4 heads x 64, 48 x 112: 7.2 against 17.5 us.
#include "common.h"
#include <algorithm>
#include <cfloat>
#include <type_traits>

namespace sdllm {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct AttnF32Args {
  const float* q_block; const float* q_suffix;
  const float* k_cache; const float* v_cache;
  const float* k_block; const float* v_block;
  const float* k_suffix; const float* v_suffix;
  const int32_t* keep_idx;
  float* out;
  int Hq, Hkv, g, D, P, cap, K, S, n_keep, Nq, Nkv, Rtot;
  int n_groups, q_tiles, key_blocks;
  int nr, nk;                     // waves of a workgroup: row blocks x key shares
  int xcd_map;                    // workgroups of a group on one XCD (group count a good fit for 8)
  float scale;
};

constexpr int kF32Rows = 16;      // query rows per wave
constexpr int kF32Keys = 16;      // keys per block
// Workgroups in a row of the grid: a launch takes fewer than 2^32 work-items in each dimension, which 2^23 workgroups of
// 512 would reach.  A multiple of the chip's parts, so that the workgroup number mod 8 is the part in every row.
constexpr unsigned kF32GridX = 1u << 22;

// most waves of a workgroup: 8 (two per SIMD); 4 for 256-wide heads, whose operands and accumulators need the registers
template <int NS> constexpr int f32_max_waves() { return NS <= 8 ? 8 : 4; }

typedef const __attribute__((address_space(4))) int32_t* f32_const_i32_ptr;   // scalar loads

// keep_idx of the first and last key of a block that lies wholly in the kept suffix, asked for one block ahead
struct F32Ahead { int first, last; };

__device__ __forceinline__ F32Ahead f32_ahead(const AttnF32Args& a, int blk) {
  F32Ahead ka{0, 0};
  const int s0 = blk * kF32Keys - a.P - a.K;
  if (s0 >= 0 && s0 + kF32Keys <= a.n_keep) {
    const f32_const_i32_ptr keep = (f32_const_i32_ptr)(uintptr_t)a.keep_idx;
    ka.first = keep[s0]; ka.last = keep[s0 + kF32Keys - 1];
  }
  return ka;
}

// Pointers into a tensor's three places.  Global address space by type: through a select or a null test the compiler
// loses it, and generic loads are counted (and waited for) as LDS accesses too.  Three separate values wherever a row is
// selected (in a struct the select becomes a table lookup in scratch memory).
typedef const __attribute__((address_space(1))) float* f32_gptr;
__device__ __forceinline__ f32x4 f32_load4(f32_gptr p) { return *reinterpret_cast<const __attribute__((address_space(1))) f32x4*>(p); }

// Start of the 16 rows of key block `blk` where they are consecutive rows of one place (in the suffix: where keep_idx
// maps them to consecutive rows), else nullptr.  Uniform.
__device__ __forceinline__ f32_gptr f32_run(const AttnF32Args& a, f32_gptr tc, f32_gptr tb, f32_gptr ts, int blk, const F32Ahead& ka) {
  const int r0 = blk * kF32Keys;
  if (r0 + kF32Keys <= a.P) return tc + (long long)r0 * a.D;
  if (r0 >= a.P && r0 + kF32Keys <= a.P + a.K) return tb + (long long)(r0 - a.P) * a.D;
  if (ka.last - ka.first == kF32Keys - 1) return ts + (long long)ka.first * a.D;
  return nullptr;
}

// Any N rows (past the end: the last one, whose score is masked), by selects.  keep_idx is readable at entry 0 also
// when nothing is kept (the launcher sees to it), so that the loads need no branch and travel together.
template <int N>
__device__ __forceinline__ void f32_rows(const AttnF32Args& a, f32_gptr tc, f32_gptr tb, f32_gptr ts, int row0, f32_gptr (&p)[N]) {
  int row[N], kidx[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    row[i] = min(row0 + i, a.Nkv - 1);
    kidx[i] = a.keep_idx[max(row[i] - a.P - a.K, 0)];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool in_c = row[i] < a.P, in_b = row[i] < a.P + a.K;
    p[i] = (in_c ? tc : (in_b ? tb : ts)) + (long long)(in_c ? row[i] : (in_b ? row[i] - a.P : kidx[i])) * a.D;
  }
}

// The loads below run over all NS slices whatever D is (no branches: the loads of a block travel together and the
// wait counts stay exact); past D they re-read the row's last elements, which no product takes and no store writes.
// K operands: lane (l16, G) takes d = 16 s + 4 G .. + 3 of key l16
template <int NS>
__device__ __forceinline__ void f32_load_k(const AttnF32Args& a, int l16, int G, f32_gptr tc, f32_gptr tb, f32_gptr ts, int blk,
                                           const F32Ahead& ka, f32x4 (&k)[NS]) {
  const f32_gptr run = f32_run(a, tc, tb, ts, blk, ka);
  f32_gptr kp[1];
  if (run != nullptr) kp[0] = run + l16 * a.D;
  else f32_rows<1>(a, tc, tb, ts, blk * kF32Keys + l16, kp);
#pragma unroll
  for (int s = 0; s < NS; ++s) k[s] = f32_load4(kp[0] + min(16 * s + 4 * G, a.D - 4));
}

// Heads of 65 to 128 elements, short launches (the rule is at the launch): K goes through LDS, into a region of the wave's own (no
// barrier).  The operand layout takes 64
// bytes of each of 16 rows a load, half lines; a 128-wide block's eight such loads keep the load path busy for 512 cycles a
// wave, half as long as the matrix pipe of a SIMD needs for the scores, and the CU's eight waves share one load path.  A
// transfer brings one kilobyte of whole lines.  B2, 32 / 8 heads x 128, 64 rows x 672 keys: 23.5 -> 21.6 us; B1, 32 / 32, 64 rows
// x 1088 keys: 32.0 -> 29.0.  (64-wide heads have half the scores' time to cover the round trip, 2112 keys 30.2 -> 30.8; wider ones have one
// wave per SIMD, 8 heads x 252, 1532 keys 77 -> 85: both keep their loads.)  A row is CPR 16-byte chunks (its head
// padded to the slices by re-reading the last one); place p of row r holds chunk p ^ r in the low four bits, so that an operand
// read (one chunk of 16 rows; the hardware serves rows 0-3 and 12-15 of it with rows 4-11 of the next) is free of conflicts.
template <int NS> struct F32K {
  static constexpr int CPR = 4 * NS;             // chunks per row
  static constexpr int RPT = 64 / CPR;           // rows per transfer; NS transfers per block
  static constexpr int BUF = NS * 1024;          // bytes of a block
  unsigned voff[NS];                             // this lane's byte offset of transfer j from the block's first row
  unsigned lds;                                  // the wave's region: two blocks
};

template <int NS>
__device__ __forceinline__ void f32_dma_k(const AttnF32Args& a, const F32K<NS>& kk, int lane, f32_gptr tc, f32_gptr tb, f32_gptr ts,
                                          int blk, int buf, const F32Ahead& ka) {
  using S = F32K<NS>;
  const unsigned dst = __builtin_amdgcn_readfirstlane(kk.lds + buf * S::BUF);
  const f32_gptr run = f32_run(a, tc, tb, ts, blk, ka);
  if (run != nullptr) {
    const unsigned long long p = (unsigned long long)run;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
    const unsigned long long base = ((unsigned long long)hi << 32) | lo;
#pragma unroll
    for (int j = 0; j < NS; ++j)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :: "s"(dst + j * 1024), "v"(kk.voff[j]), "s"(base) : "memory", "m0");
  } else {
    f32_gptr own[1];                             // row lane % 16 of the block
    f32_rows<1>(a, tc, tb, ts, blk * kF32Keys + (lane & 15), own);
    const unsigned lo = (unsigned)(unsigned long long)own[0], hi = (unsigned)((unsigned long long)own[0] >> 32);
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int row = j * S::RPT + lane / S::CPR;
      const unsigned long long rp = ((unsigned long long)(unsigned)__shfl((int)hi, row) << 32) | (unsigned)__shfl((int)lo, row);
      const unsigned long long va = rp + (kk.voff[j] - (unsigned)(row * a.D * 4));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   :: "s"(dst + j * 1024), "v"(va) : "memory", "m0");
    }
  }
}

// K operands out of the wave's region: lane (l16, G) takes d = 16 s + 4 G .. + 3 of key l16
template <int NS>
__device__ __forceinline__ void f32_read_k(const unsigned char* buf, int l16, int G, f32x4 (&k)[NS]) {
#pragma unroll
  for (int s = 0; s < NS; ++s)
    k[s] = *reinterpret_cast<const f32x4*>(buf + l16 * (NS * 64) + (((4 * s + G) ^ l16) << 4));
}

// V operands: lane (l16, G) takes d = 64 dg + 4 l16 .. + 3 of keys 4 G + i
template <int NS>
__device__ __forceinline__ void f32_load_v(const AttnF32Args& a, int l16, int G, f32_gptr tc, f32_gptr tb, f32_gptr ts, int blk,
                                           const F32Ahead& ka, f32x4 (&v)[NS / 4][4]) {
  const f32_gptr run = f32_run(a, tc, tb, ts, blk, ka);
  f32_gptr vp[4];
  if (run != nullptr) {
#pragma unroll
    for (int i = 0; i < 4; ++i) vp[i] = run + (4 * G + i) * a.D;
  } else {
    f32_rows<4>(a, tc, tb, ts, blk * kF32Keys + 4 * G, vp);
  }
#pragma unroll
  for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
    for (int i = 0; i < 4; ++i) v[dg][i] = f32_load4(vp[i] + min(64 * dg + 4 * l16, a.D - 4));
}

// S^T of one key block, times the scale.  RAGGED: the head is narrower than its NS slices; slices past D are left out,
// and in the one that D ends in K becomes zero like Q (the re-read elements may be infinite, and zero times those is NaN).
// PARTIAL: the sequence's last keys, fewer than a block; those past the end get -inf.
template <int NS, bool RAGGED, bool PARTIAL>
__device__ __forceinline__ f32x4 f32_scores(const AttnF32Args& a, int G, int blk, const f32x4 (&k)[NS], const f32x4 (&q)[NS]) {
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    constexpr int kWhole = NS == 4 ? 0 : NS / 2;   // slices that every width served by this NS fills
    if (RAGGED && s >= kWhole && 16 * s >= a.D) break;       // uniform
    f32x4 ks = k[s];
    if (RAGGED && s >= kWhole && 16 * s + 16 > a.D) {        // uniform
      // (holds the branch: turned into selects in every slice, a 252-wide layer, 64 rows x 736 keys, took 43.8 us, not 41.2)
      asm volatile("");
      if (16 * s + 4 * G >= a.D) ks = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(ks[j], q[s][j], acc[j & 1], 0, 0, 0);
  }
  f32x4 sc = (acc[0] + acc[1]) * a.scale;
  if constexpr (PARTIAL) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (blk * kF32Keys + 4 * G + i >= a.Nkv) sc[i] = -INFINITY;
  }
  return sc;
}

// Online softmax step and O^T += V^T P^T
template <int NS, bool PARTIAL>
__device__ __forceinline__ void f32_accumulate(const AttnF32Args& a, int G, int blk, const f32x4& sc, f32x4 (&v)[NS / 4][4],
                                               f32x4 (&o)[NS / 4][4], float& m, float& l) {
  float mx = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
  const auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
  mx = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
  const auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
  mx = fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
  const float m_new = fmaxf(m, mx);                // not -inf, also where every score so far is: those weigh exp(-inf) = 0
  if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {      // uniform: some row's reference moves
    const float corr = expf(m - m_new);            // first block: 0 (or 1, and nothing to scale)
    l *= corr;
#pragma unroll
    for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[dg][j] *= corr;
    m = m_new;
  }
  if constexpr (PARTIAL) {                         // zeros past the end: the re-read last row may be infinite, p is 0
#pragma unroll
    for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (blk * kF32Keys + 4 * G + i >= a.Nkv) v[dg][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // key by key: the matrix instructions of one key cover the next one's exponential
  float p[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = expf(sc[i] - m_new);
#pragma unroll
    for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[dg][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[dg][i][j], p[i], o[dg][j], 0, 0, 0);
  }
  l += (p[0] + p[1]) + (p[2] + p[3]);              // this lane's keys; summed across the row's lanes at the end
}

// KLDS: K goes through LDS
template <int NS, bool RAGGED, bool KLDS>
__global__ __launch_bounds__(64 * f32_max_waves<NS>(), f32_max_waves<NS>() / 4) void attention_f32_kernel(AttnF32Args a) {
  extern __shared__ __attribute__((aligned(16))) float f32_lds[];
  const int lane = threadIdx.x & 63, l16 = lane & 15, G = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave % a.nr, wk = wave / a.nr;
  // ---- which piece of work: with xcd_map the row tiles of a group sit on one XCD (its L2 holds the group's K/V)
  const unsigned wg = blockIdx.y * kF32GridX + blockIdx.x, q_tiles = a.q_tiles;
  unsigned ugrp;
  int qt;
  if (a.xcd_map) {
    const unsigned xcd = wg % kNumXCDs, slot = wg / kNumXCDs;
    ugrp = (slot / q_tiles) * kNumXCDs + xcd; qt = slot % q_tiles;
  } else {
    ugrp = wg / q_tiles; qt = wg % q_tiles;
  }
  if (ugrp >= (unsigned)a.n_groups) return;
  const int grp = ugrp;
  const int b = grp / a.Hkv, kvh = grp - b * a.Hkv, D = a.D;
  const long long bh = grp;
  const f32_gptr kc = (f32_gptr)a.k_cache + bh * a.cap * D, vc = (f32_gptr)a.v_cache + bh * a.cap * D;
  const f32_gptr kb = (f32_gptr)a.k_block + bh * a.K * D, vb = (f32_gptr)a.v_block + bh * a.K * D;
  const f32_gptr ks = (f32_gptr)a.k_suffix + bh * a.S * D, vs = (f32_gptr)a.v_suffix + bh * a.S * D;

  // ---- this wave's query rows; the first key block's K goes in flight while a kept row's keep_idx entry travels
  const int R = (qt * a.nr + wr) * kF32Rows + l16;
  const int Rc = min(R, a.Rtot - 1);
  const int hl = Rc / a.Nq, qi = Rc - hl * a.Nq;
  const long long qbh = (long long)b * a.Hq + (long long)kvh * a.g + hl;
  const int q_keep = a.keep_idx[max(qi - a.K, 0)];
  using KS = F32K<NS>;
  KS kk;
  unsigned char* const kbuf = reinterpret_cast<unsigned char*>(f32_lds) + wave * 2 * KS::BUF;
  kk.lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)reinterpret_cast<unsigned char*>(f32_lds) +
           wave * 2 * KS::BUF;
  f32x4 k[NS], v[NS / 4][4];
  F32Ahead ka = f32_ahead(a, wk);
  if constexpr (KLDS) {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int row = j * KS::RPT + lane / KS::CPR;
      kk.voff[j] = 4u * (unsigned)(row * D + min(4 * ((lane % KS::CPR) ^ (row & 15)), D - 4));
    }
    if (wk < a.key_blocks) f32_dma_k<NS>(a, kk, lane, kc, kb, ks, wk, 0, ka);
  } else {
    f32_load_k<NS>(a, l16, G, kc, kb, ks, min(wk, a.key_blocks - 1), ka, k);
  }
  __builtin_amdgcn_sched_barrier(0);
  const f32_gptr qp = qi < a.K ? (f32_gptr)a.q_block + (qbh * a.K + qi) * D : (f32_gptr)a.q_suffix + (qbh * a.S + q_keep) * D;
  f32x4 q[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) q[s] = f32_load4(qp + min(16 * s + 4 * G, D - 4));
  if constexpr (RAGGED) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (16 * s + 4 * G >= D) q[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 o[NS / 4][4];
#pragma unroll
  for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
    for (int j = 0; j < 4; ++j) o[dg][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the lowest finite reference, not -inf: scores may be -inf themselves (overflow, infinite operands), also all of a block
  float m = -FLT_MAX, l = 0.f;

  // ---- key blocks wk, wk + nk, ...: a block's V travels during its scores; the next block's K too where it goes through LDS,
  // otherwise during the P V.  (The transfers into LDS are invisible to the compiler's wait counts; asked for before V, they
  // are complete whenever V is, since loads return in order.  The wait in front of the reads of K therefore costs nothing
  // after the first block.)
  int buf = 0;
  auto block = [&](int blk, auto partial) {
    if constexpr (KLDS) {
      // K of this block has landed, and the other region, which the next transfers fill, has been read
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      const F32Ahead kn = f32_ahead(a, blk + a.nk);
      if (blk + a.nk < a.key_blocks) f32_dma_k<NS>(a, kk, lane, kc, kb, ks, blk + a.nk, buf ^ 1, kn);
      f32_load_v<NS>(a, l16, G, vc, vb, vs, blk, ka, v);
      ka = kn;
      f32_read_k<NS>(kbuf + buf * KS::BUF, l16, G, k);
      buf ^= 1;
    } else {
      f32_load_v<NS>(a, l16, G, vc, vb, vs, blk, ka, v);
      ka = f32_ahead(a, blk + a.nk);
    }
    const f32x4 sc = f32_scores<NS, RAGGED, partial.value>(a, G, blk, k, q);
    if constexpr (!KLDS) f32_load_k<NS>(a, l16, G, kc, kb, ks, min(blk + a.nk, a.key_blocks - 1), ka, k);   // (past the end:
    f32_accumulate<NS, partial.value>(a, G, blk, sc, v, o, m, l);                                           // never used)
  };
  const int full = a.Nkv / kF32Keys;
  int blk = wk;
  for (; blk < full; blk += a.nk) block(blk, std::false_type{});
  if (blk < a.key_blocks) block(blk, std::true_type{});      // the sequence's last keys, not a whole block
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // ---- lane (q = l16, G) holds O[q][64 dg + 4 (4 G + i) + j]: for fixed i four consecutive elements
  float* orow = a.out + (((long long)b * a.Hq + (long long)kvh * a.g) * a.Nq + R) * D;
  if (a.nk == 1) {
    const float inv = 1.0f / l;
    if (R < a.Rtot) {
#pragma unroll
      for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = 64 * dg + 16 * G + 4 * i;
          if (d < D) *reinterpret_cast<f32x4*>(orow + d) = f32x4{o[dg][0][i], o[dg][1][i], o[dg][2][i], o[dg][3][i]} * inv;
        }
    }
    return;
  }
  const int nw = a.nr * a.nk;
  if constexpr (KLDS) __syncthreads();                                   // the exchange area lies over the regions of K
  f32x4* xo = reinterpret_cast<f32x4*>(f32_lds);                         // [wave][NS pieces][64 lanes]
  float2* xml = reinterpret_cast<float2*>(f32_lds + nw * NS * 256);      // [wave][16 rows]
#pragma unroll
  for (int dg = 0; dg < NS / 4; ++dg)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      xo[(wave * NS + 4 * dg + i) * 64 + lane] = f32x4{o[dg][0][i], o[dg][1][i], o[dg][2][i], o[dg][3][i]};
  if (G == 0) xml[wave * 16 + l16] = make_float2(m, l);
  __syncthreads();
  // the nk waves of a row block share its NS pieces; shares are merged in index order
  float M = -INFINITY;
  for (int k = 0; k < a.nk; ++k) M = fmaxf(M, xml[(k * a.nr + wr) * 16 + l16].x);
  float L = 0.f;
  for (int k = 0; k < a.nk; ++k) {
    const float2 ml = xml[(k * a.nr + wr) * 16 + l16];
    L += expf(ml.x - M) * ml.y;
  }
  const float inv = 1.0f / L;
  for (int u = wk; u < NS; u += a.nk) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < a.nk; ++k) {
      const int w = k * a.nr + wr;
      acc += xo[(w * NS + u) * 64 + lane] * expf(xml[w * 16 + l16].x - M);
    }
    const int d = 64 * (u >> 2) + 16 * G + 4 * (u & 3);
    if (R < a.Rtot && d < D) *reinterpret_cast<f32x4*>(orow + d) = acc * inv;
  }
}

// Waves of a workgroup: NR row blocks x NK key shares.  The aim is 8 waves per CU (two per SIMD).
//   NR  1 unless the call has 16-row blocks for two (four, eight) per CU; then a workgroup holds as many, which share K/V in
//       the L1, as long as the last tile of a group is not mostly empty.
//   NK  what NR leaves of the workgroup's waves, but no more than there are key blocks.  Where the call has 8 waves per CU
//       with half as many shares, a share holds at least 4 key blocks: the merge through LDS costs as much as several of
//       them.  Measured with / without that: 32768 groups of one row, 4 wide, 65 keys 95 / 320 us (one query row per
//       wave with FMAs: 174), 2048 groups of one row, 16 wide, 65 keys 9.4 / 23.0 (18.4), 8192 groups of one row, 128
//       wide, 65 keys 99 / 244 (304).  With 8 blocks as the limit, 3200 groups of 10 rows, 64 wide, 710 keys took 205
//       us, not 202; without one, 2048 groups of one row, 64 wide, 1025 keys 184, not 177.
struct F32Plan { int nr, nk, q_tiles, xcd_map; long long workgroups; };
static F32Plan plan_attention_f32(const sdllm_attn_params& p) {
  const int max_waves = p.D <= 128 ? f32_max_waves<8>() : f32_max_waves<16>();
  const long long Rtot = (long long)(p.Hq / p.Hkv) * (p.K + p.n_keep);
  const long long groups = (long long)p.B * p.Hkv;
  const long long tiles = (Rtot + kF32Rows - 1) / kF32Rows;
  const long long blocks = ((long long)p.prefix_len + p.K + p.n_keep + kF32Keys - 1) / kF32Keys;
  F32Plan pl;
  pl.nr = max_waves;
  while (pl.nr > 1 && (pl.nr * (long long)kNumCUs > tiles * groups || (tiles + pl.nr - 1) / pl.nr * pl.nr * 8 > tiles * 9)) pl.nr >>= 1;
  pl.nk = max_waves / pl.nr;
  while (pl.nk > 1 && pl.nk / 2 >= blocks) pl.nk >>= 1;
  pl.q_tiles = (int)((tiles + pl.nr - 1) / pl.nr);
  while (pl.nk > 1 && blocks < 4 * pl.nk && groups * pl.q_tiles * pl.nr * (pl.nk / 2) >= 8LL * kNumCUs) pl.nk >>= 1;
  const long long padded = (groups + kNumXCDs - 1) / kNumXCDs * kNumXCDs;
  pl.xcd_map = padded * 4 <= groups * 5;
  pl.workgroups = (pl.xcd_map ? padded : groups) * pl.q_tiles;
  return pl;
}

void attention_f32_plan(const sdllm_attn_params& p, sdllm_attn_plan* plan) {
  const F32Plan pl = plan_attention_f32(p);
  plan->kv_splits = 1; plan->rows_per_workgroup = kF32Rows * pl.nr; plan->workgroups = (int32_t)std::min(pl.workgroups, 0x7fffffffLL);
  plan->key_tiles_per_split = (p.prefix_len + p.K + p.n_keep + kF32Keys - 1) / kF32Keys;
  plan->workgroup_shape = 0; plan->ring_stages = 2;
}

// the exchange area of the merge, or the regions of K that it lies over
template <int NS, bool KLDS> constexpr size_t f32_lds_bytes(int waves) {
  constexpr int exchange = NS * 1024 + 16 * (int)sizeof(float2);
  static_assert(2 * F32K<NS>::BUF >= exchange, "the exchange area fits the regions of K");
  return (size_t)waves * (KLDS ? 2 * F32K<NS>::BUF : exchange);
}

template <int NS, bool RAGGED, bool KLDS>
static hipError_t f32_opt_in() {
  static LdsOptIn st;
  return ensure_lds_opt_in(reinterpret_cast<const void*>(&attention_f32_kernel<NS, RAGGED, KLDS>),
                           f32_lds_bytes<NS, KLDS>(f32_max_waves<NS>()), st);
}

hipError_t prepare_attention_f32() {
  hipError_t e = f32_opt_in<4, false, false>();
  if (e == hipSuccess) e = f32_opt_in<4, true, false>();
  if (e == hipSuccess) e = f32_opt_in<8, false, false>();
  if (e == hipSuccess) e = f32_opt_in<8, true, false>();
  if (e == hipSuccess) e = f32_opt_in<8, false, true>();
  if (e == hipSuccess) e = f32_opt_in<8, true, true>();
  if (e == hipSuccess) e = f32_opt_in<16, false, false>();
  if (e == hipSuccess) e = f32_opt_in<16, true, false>();
  return e;
}

template <int NS, bool RAGGED, bool KLDS = false>
static hipError_t f32_launch(const AttnF32Args& a, const F32Plan& pl, hipStream_t stream) {
  const hipError_t e = f32_opt_in<NS, RAGGED, KLDS>();
  if (e != hipSuccess) return e;
  const int waves = pl.nr * pl.nk;
  const dim3 grid((unsigned)std::min(pl.workgroups, (long long)kF32GridX), (unsigned)((pl.workgroups + kF32GridX - 1) / kF32GridX));
  const size_t lds = KLDS || pl.nk > 1 ? f32_lds_bytes<NS, KLDS>(waves) : 0;
  hipLaunchKernelGGL((attention_f32_kernel<NS, RAGGED, KLDS>), grid, dim3(64 * waves), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_attention_f32(const sdllm_attn_params& p,
                                const void* q_block, const void* q_suffix,
                                const void* k_cache, const void* v_cache,
                                const void* k_block, const void* v_block,
                                const void* k_suffix, const void* v_suffix,
                                const int32_t* keep_idx, void* out, hipStream_t stream) {
  const F32Plan pl = plan_attention_f32(p);
  AttnF32Args a;
  a.q_block = (const float*)q_block; a.q_suffix = (const float*)q_suffix;
  a.k_cache = (const float*)k_cache; a.v_cache = (const float*)v_cache;
  a.k_block = (const float*)k_block; a.v_block = (const float*)v_block;
  a.k_suffix = (const float*)k_suffix; a.v_suffix = (const float*)v_suffix;
  // (f32_rows reads entry 0 without a branch when nothing is kept: any readable address will do)
  a.keep_idx = p.n_keep > 0 ? keep_idx : (const int32_t*)q_block; a.out = (float*)out;
  a.Hq = p.Hq; a.Hkv = p.Hkv; a.g = p.Hq / p.Hkv; a.D = p.D; a.P = p.prefix_len; a.cap = p.prefix_cap;
  a.K = p.K; a.S = p.S; a.n_keep = p.n_keep;
  a.Nq = p.K + p.n_keep; a.Nkv = p.prefix_len + p.K + p.n_keep; a.Rtot = a.g * a.Nq;
  a.n_groups = p.B * p.Hkv; a.q_tiles = pl.q_tiles; a.key_blocks = (a.Nkv + kF32Keys - 1) / kF32Keys;
  a.nr = pl.nr; a.nk = pl.nk; a.xcd_map = pl.xcd_map;
  a.scale = p.scale > 0.f ? p.scale : 1.0f / sqrtf((float)p.D);
  // K through LDS (heads of 65 to 128 elements) pays where the launch is a chain of latencies: a round and a half of workgroups
  // at most, and four whole key blocks or more.  In longer launches a workgroup's 128 KB of LDS keep the next one from starting
  // beside it, and a shorter sequence only adds the wait for K in front of V.  Measured over 90 geometries x 5 widths x up to 10 lengths, registers / LDS in us:
  //   within the rule 0.86 to 1.02 of the registers' time; 16 groups x 256 rows x 672 keys, 128 wide, 23.5 / 21.6
  //   512 to 2048 workgroups of one 16-row block, 128 wide, 129 to 600 keys: 1.00 to 1.17 of it; 512 groups x 272 keys 26.3 / 27.1
  //   fewer keys: 8192 groups of one row x 1 key 20.7 / 22.4; 8 groups x 128 rows x 32 keys 6.06 / 6.41
  const bool k_lds = pl.workgroups <= kNumCUs * 3 / 2 && a.Nkv >= 4 * kF32Keys;
  switch (p.D) {
    case 64: return f32_launch<4, false>(a, pl, stream);
    case 128: return k_lds ? f32_launch<8, false, true>(a, pl, stream) : f32_launch<8, false>(a, pl, stream);
    case 256: return f32_launch<16, false>(a, pl, stream);
  }
  if (p.D < 64) return f32_launch<4, true>(a, pl, stream);
  if (p.D < 128) return k_lds ? f32_launch<8, true, true>(a, pl, stream) : f32_launch<8, true>(a, pl, stream);
  return f32_launch<16, true>(a, pl, stream);
}

}  // namespace sdllm
