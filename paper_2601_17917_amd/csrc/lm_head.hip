// Vocabulary projection fused into the confidence-aware unmask (paper Eq. 3 -> Eq. 4): the logits
// z_i = W h_i of the masked positions are formed tile by tile on the matrix cores and reduced to
// (max, sum of exp, lowest argmax id) triples in registers; they are never written to memory.
// The triples go to the same commit kernel as those of the streaming reduction over stored logits.
//
//   * Masked rows are compacted inside the kernels (every workgroup scans the mask bytes), so the matrix cores only see rows
//     that Eq. 4 asks for.
//   * logits^T tile = W_tile h^T (v_mfma_f32_16x16x32_bf16, fp32 accumulate): a lane ends up with vocabulary ids
//     4 (lane / 16) + r of row lane % 16, so the row reduction is in-lane first, then two lane exchanges.
//   * Shapes: more than 128 masked positions go to lm_head_rows_kernel in chunks of 160 to 256 rows, a tiled product with both
//     operands in LDS.  Calls with at most 128 masked positions are a read of W and take the stream kernels further down,
//     which turn the roles around: the hidden operands stay in registers and W goes through LDS (1 KB row pieces through
//     registers up to 64 positions, global -> LDS transfers up to 128), or, when W is the packed image, comes straight from it.
//   * The masked count is device data: the host launches every shape that B x K admits and each launch
//     exits unless the count is in its range.
#include "common.h"
#include "unmask_common.h"
#include <climits>
#include <type_traits>

namespace sdllm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kLmThreads = 256;
constexpr int kLmWaves = kLmThreads / 64;

struct LmHeadArgs {
  const uint16_t* hidden;     // [rows_total][ld_h]
  const uint16_t* weight;     // [V][ld_w], or the packed image [ceil(V/16)][Hd/32][64 lanes][8] (packed != 0)
  const uint8_t* masked;      // [rows_total]
  Partial* partials;          // [rows_total][ntile]
  long long ld_h, ld_w;       // elements
  int rows_total, V, Hd;
  int ntile;                  // vocabulary tiles
  int nchunk;                 // row chunks in the grid (upper bound of ceil(masked rows / kRwBM))
  // The masked count is device data, the shape that suits it is not known to the host: a call launches every
  // shape its B x K admits and each launch exits at once unless min_masked <= masked count <= max_masked.
  int min_masked, max_masked;
  // a position's triples are [ntile_out] (the largest tile count among the call's launches); the launch that
  // runs writes its ntile of them and neutral triples into the rest (slot tile + j ntile from workgroup tile)
  int ntile_out;
  int packed;                 // weight is the packed image: the A operand of 16-row block nb and k-step ks is
                              // the kilobyte at ((nb * Hd/32 + ks) * 64 + lane) * 8 elements
};

__device__ __forceinline__ void store_partial(const LmHeadArgs& a, int row, int tile, const Partial& p) {
  Partial* out = a.partials + (long long)row * a.ntile_out;
  out[tile] = p;
  for (int j = tile + a.ntile; j < a.ntile_out; j += a.ntile) out[j] = Partial{kNegBig, 0.f, 0x7fffffff};
}

// Number of masked positions of the call (uniform over the workgroup): one pass over the mask bytes without
// barriers, then one reduction.  wsum: kLmWaves ints of LDS, free for other use on return.
template <int THREADS = kLmThreads>
__device__ __forceinline__ int lm_masked_count(const LmHeadArgs& a, int* wsum) {
  const int tid = threadIdx.x;
  int mine = 0;
  for (int i = tid; i < a.rows_total; i += THREADS) mine += a.masked[i] != 0;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) mine += __shfl_xor(mine, off);
  if ((tid & 63) == 0) wsum[tid >> 6] = mine;
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) total += wsum[w];
  __syncthreads();
  return total;
}

template <int N> __device__ __forceinline__ void lm_wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt is a six-bit field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));    // expcnt / lgkmcnt: no wait
}
// one transfer: lane i's 16 bytes at vaddr land at lds_addr + 16 i (lds_addr uniform)
template <bool NT>
__device__ __forceinline__ void lm_dma16(unsigned lds_addr, const void* vaddr) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(vaddr) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(vaddr) : "memory", "m0");
}

// lm_head_rows_kernel: 512 threads, two waves per SIMD.  A workgroup owns 256 vocabulary rows x JB 16-row blocks of
// positions; wave (wv, wp) owns four 16-row blocks of W x half of the position blocks.  Both operands go from global memory
// straight into LDS, 64 elements of Hd (two k-steps) per ring stage: three stages of W, two of the hidden rows.
constexpr int kRwThreads = 512;
constexpr int kRwWaves = kRwThreads / 64;
constexpr int kRwBM = 256;                       // most positions of a workgroup
constexpr int kRwBN = 256;                       // vocabulary rows of a workgroup
constexpr int kRwStage = 256 * 128;              // 32 KB: one stage of either operand
constexpr int kRwWNST = 3, kRwHNST = 2;
constexpr int kRwHid = kRwWNST * kRwStage;       // byte offset of the hidden stages
constexpr int kRwLds = (kRwWNST + kRwHNST) * kRwStage;
static_assert(kRwLds <= 160 * 1024, "LDS of a CU");

// acc += A B with the accumulator pinned to the accumulation registers.  The compiler does not see a matrix instruction
// inside the asm statement and puts no wait states behind it.  Between matrix instructions none are needed; the LAST one
// before other instructions read the accumulators brings its own, the 8 that the compiler itself puts between this
// instruction and a read of its result.  They are part of the statement because a wait by itself behind the loop holds
// nothing back: the register copies that the compiler makes between the loop and the first read pass it, with or without
// a memory clobber, and also when the accumulators are its operands.
template <bool WAIT>
__device__ __forceinline__ void mfma_acc(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  if constexpr (WAIT) asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 7" : "+a"(acc) : "v"(a), "v"(b));
  else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// The vocabulary tiles tile0, tile0 + tile_step, ... for one row chunk of JB 16-row blocks of positions.
// Between its roofs: 256 positions x 126464 x 4096 take 421k to 460k cycles by card, of which the matrix pipe is busy 253k, at a
// clock that falls to 2.1 GHz and below under matrix work on a full stream of W; without the transfers 389k cycles, without the
// matrix instructions 180 us at 2.4 GHz (on the card with 421k).  What this split gains over one wave per SIMD with W straight into registers: whole
// 128-byte lines of both operands (16 rows x 64 bytes a transfer took 1.5 times as long), two waves per SIMD that fill each
// other's gaps, one prologue per workgroup instead of one per tile.  Per call over 126464 x 4096, before / after in turn on one
// card: row-major W 160 positions 263 / 213 us, 256: 282 / 249, 282: 412 / 313, 384: 443 / 357, 512: 503 / 454 (1.17 PFLOP/s);
// packed 200 / 192, 264 / 250, 344 / 308, 381 / 348, 478 / 445.
template <bool PACKED, int JB>
__device__ __forceinline__ void lm_head_rows_tiles(const LmHeadArgs& a, unsigned char* lds, const int* row_of,
                                                   int tile0, int tile_step) {
  static_assert(JB % 2 == 0 && JB * 16 <= kRwBM, "two halves");
  constexpr int JH = JB / 2;                     // position blocks per wave
  constexpr int NH = (2 * JB + kRwWaves - 1) / kRwWaves;       // hidden transfers per wave and stage, at most
  static_assert(NH <= 4 && JH >= 4, "one transfer per group of matrix instructions");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = wave & 3, wp = wave >> 2;
  const int q = lane >> 4, l16 = lane & 15;
  const unsigned lds_wave = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds + wave * 1024;
  const int NK = a.Hd / 32, NP = (NK + 1) / 2;   // k-steps, pairs of them

  // ---- transfers.  Row-major operands: a transfer is 8 rows x 128 bytes (whole lines); transfer 2 b + h brings rows
  // 8 h .. 8 h + 7 of 16-row block b.  Lane i lands at 16 i, that is place i / 8 of the kilobyte's 8 row places, slot i % 8.
  // Place g holds row 8 h + g / 2 + 4 (g % 2), slot s piece s ^ (row % 4 + 4 h) of the pair's eight 16-byte pieces.  The 16
  // lanes that an operand read serves at a time are 0-3, 12-15, 20-27 (and 4-11, 16-19, 28-31; the same 32 higher), rows
  // 0-3, 12-15 of one piece and 4-11 of the next: with this order they fall into 16 different 16-byte groups of banks, as
  // 16 rows of one piece do.  (Place g = row % 8, xor 1 in the second half, slot = piece ^ (row % 8), free of conflicts
  // only for 16 consecutive lanes, cost 4 cycles a read.)
  // Packed W: a transfer is one operand tile, block b and k-step h of the pair.
  // This wave brings transfers wave, wave + 8, wave + 16, wave + 24 of either operand.
  const unsigned klast = (unsigned)(a.Hd - 8);
  const int g = lane >> 3, h = wave & 1;         // kRwWaves is even: h is the same for all of a wave's transfers
  const int r8 = (g >> 1) + 4 * (g & 1);
  const unsigned piece = (unsigned)(8 * ((lane & 7) ^ ((g >> 1) + 4 * h)));    // elements
  const uint16_t* wsrc[4];
  auto w_tile = [&](int tile) {                  // W's transfers bring this tile from here on
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int blk = (wave + kRwWaves * i) >> 1;
      if constexpr (PACKED) {
        const int nb = min(tile * (kRwBN / 16) + blk, (a.V + 15) / 16 - 1);                // blocks past V: the last one
        wsrc[i] = a.weight + ((long long)nb * NK * 64 + lane) * 8;
      } else {
        const int n = min(tile * kRwBN + blk * 16 + 8 * h + r8, a.V - 1);                  // rows past V: any valid row
        wsrc[i] = a.weight + (long long)n * a.ld_w;
      }
    }
  };
  const uint16_t* hsrc[NH];
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    const int r = min(((wave + kRwWaves * i) >> 1) * 16 + 8 * h + r8, JB * 16 - 1);
    hsrc[i] = a.hidden + (long long)max(row_of[r], 0) * a.ld_h;
  }
  const int my_row = tid < JB * 16 ? row_of[tid] : -1;
  __syncthreads();                               // the list's place in LDS belongs to the ring from here on

  // Every workgroup walks a tile's pairs in a rotation of the tile's, so that the workgroups resident at one time do not all
  // ask for the same columns of W at once.  Pairs form one sequence over all of the workgroup's tiles: the transfers run ahead
  // into the next tile; behind the last one they bring its last pair again (into stages that nobody reads any more).
  struct Walk { int tile, left, pair; };         // pairs left in the tile, this one included
  const int turn = tile_step % NP;               // from one tile's rotation to the next one's
  const int last_tile = a.ntile - tile_step;     // tiles below it have a successor
  auto next = [&](Walk& w) -> bool {             // true: a new tile.  By selects: branches here split the trip's halves
    const bool end = w.left == 1, more = end && w.tile < last_tile;
    const int p = w.pair + 1 + (more ? turn : 0);              // a tile's walk ends one pair before its first
    w.pair = end && !more ? w.pair : p - (p >= NP ? NP : 0);
    w.left = end ? (more ? NP : 1) : w.left - 1;
    w.tile += more ? tile_step : 0;
    return more;
  };
  auto issue_w = [&](int i, int pr, int stage_ofs) {           // transfer i (0..3) of pair pr
    const unsigned dst = lds_wave + (unsigned)stage_ofs + kRwWaves * i * 1024;
    if constexpr (PACKED) lm_dma16<true>(dst, wsrc[i] + (long long)min(2 * pr + h, NK - 1) * 512);
    else lm_dma16<true>(dst, wsrc[i] + min(64u * pr + piece, klast));
  };
  auto issue_h = [&](int i, int pr, int stage_ofs) {           // transfer i (0..NH - 1), if this wave has it
    const unsigned dst = lds_wave + kRwHid + (unsigned)stage_ofs + kRwWaves * i * 1024;
    if ((i + 1) * kRwWaves <= 2 * JB || wave + kRwWaves * i < 2 * JB) lm_dma16<false>(dst, hsrc[i] + min(64u * pr + piece, klast));
  };
  // Where Hd ends in mid-pair (an odd number of k-steps), the hidden pieces past it, which the transfers filled with the row's
  // last one, become zeros: this wave's own transfers, landed, before the barrier that hands them out.
  auto zero_past_end = [&](int pr, int stage_ofs) {
    if (2 * pr + 1 < NK) return;                 // uniform
    if (64u * pr + piece <= klast) return;
#pragma unroll
    for (int i = 0; i < NH; ++i)
      if ((i + 1) * kRwWaves <= 2 * JB || wave + kRwWaves * i < 2 * JB)
        *reinterpret_cast<u32x4*>(lds + kRwHid + stage_ofs + (wave + kRwWaves * i) * 1024 + lane * 16) = u32x4{0u, 0u, 0u, 0u};
  };

  // ---- operand reads (two kilobytes per 16-row block and stage)
  const unsigned rm = (unsigned)((l16 >> 3) * 1024 + (2 * (l16 & 3) + ((l16 >> 2) & 1)) * 128 +
                                 ((q ^ ((l16 & 3) + 4 * (l16 >> 3))) << 4));
  const unsigned char* abase[2];
  const unsigned char* bbase[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    abase[ks] = lds + wv * 8192 + (PACKED ? ks * 1024 + lane * 16 : rm ^ (ks << 6));
    bbase[ks] = lds + kRwHid + wp * JH * 2048 + (rm ^ (ks << 6));
  }
  // The operands of the next k-step go in flight during this one.  The B operands are replaced in place, each behind the
  // matrix instructions that read it; those of the last two groups and the A operands, which all groups read, have a second
  // set, so that no read is asked for right before the barrier that waits for it.
  constexpr int ND = 2, NPL = JH - ND;
  f32x4 acc[4][JH];
  bf16x8 av[2][4], bv[NPL], bd[2][ND];
  auto step = [&](auto par_c, const unsigned char* an, const unsigned char* bn, auto transfer) {
    constexpr int P = decltype(par_c)::value;
#pragma unroll
    for (int jb = 0; jb < JH; ++jb) {
      if (jb < 4) av[P ^ 1][jb] = *reinterpret_cast<const bf16x8*>(an + jb * 2048);
      if (jb < ND) bd[P ^ 1][jb] = *reinterpret_cast<const bf16x8*>(bn + (NPL + jb) * 2048);
      const bf16x8 b = jb < NPL ? bv[jb < NPL ? jb : 0] : bd[P][jb < NPL ? 0 : jb - NPL];
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) {
        if (P == 1 && jb == JH - 1 && ib == 3) mfma_acc<true>(acc[ib][jb], av[P][ib], b);        // the trip's last
        else mfma_acc<false>(acc[ib][jb], av[P][ib], b);
      }
      if (jb < NPL) bv[jb < NPL ? jb : 0] = *reinterpret_cast<const bf16x8*>(bn + jb * 2048);
      if (jb < 4) transfer(jb);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- prologue: two pairs in flight
  Walk ww{tile0, NP, tile0 % NP}, wh = ww;
  w_tile(tile0);
#pragma unroll
  for (int m = 0; m < 2; ++m) {
#pragma unroll
    for (int i = 0; i < 4; ++i) issue_w(i, ww.pair, m * kRwStage);
#pragma unroll
    for (int i = 0; i < NH; ++i) issue_h(i, wh.pair, m * kRwStage);
    if (m == 0) next(wh);
    if (next(ww)) w_tile(ww.tile);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  zero_past_end(tile0 % NP, 0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

  // ---- one pair per trip.  A k-step's operands are read during the one before it, so pair m's stage is read in the second
  // half of trip m - 1 and the first half of trip m.  The barrier between a trip's halves therefore says two things: pair m + 1
  // has landed (every wave waited for its own transfers), and pair m's stages are free (every wave's reads are complete).
  // W's pair m + 2 is asked for in the first half of trip m (its stage was pair m - 1's), the hidden rows of pair m + 2 in the
  // second half (pair m's stage).  Younger than pair m + 1 are then, at the wait, W's four transfers of pair m + 2.
  int ws = 0, wn = kRwStage, wf = 2 * kRwStage;  // W stages: pair m, m + 1, m + 2
  int hs = 0;                                    // hidden stage: pair m (m + 1 is the other)
  for (int tile = tile0; tile < a.ntile; tile += tile_step) {
#pragma unroll
    for (int ib = 0; ib < 4; ++ib)
#pragma unroll
      for (int jb = 0; jb < JH; ++jb) acc[ib][jb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) av[0][ib] = *reinterpret_cast<const bf16x8*>(abase[0] + ws + ib * 2048);
#pragma unroll
    for (int jb = 0; jb < JH; ++jb)
      (jb < NPL ? bv[jb < NPL ? jb : 0] : bd[0][jb < NPL ? 0 : jb - NPL]) =
          *reinterpret_cast<const bf16x8*>(bbase[0] + hs + jb * 2048);
    int m = 0;
    do {
      step(std::integral_constant<int, 0>{}, abase[1] + ws, bbase[1] + hs, [&](int i) { issue_w(i, ww.pair, wf); });
      const int hn = kRwStage - hs;
      asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      zero_past_end(wh.pair, hn);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      next(wh);
      if (__builtin_expect(next(ww), 0)) w_tile(ww.tile);
      // (a tile's last trip reads the next tile's first operands in vain: they are read again behind the reduction, where
      // their registers are needed)
      step(std::integral_constant<int, 1>{}, abase[0] + wn, bbase[0] + hn, [&](int i) { if (i < NH) issue_h(i, wh.pair, hs); });
      const int tmp = ws; ws = wn; wn = wf; wf = tmp; hs = hn;
    } while (__builtin_expect(++m < NP, 1));

    // ---- row reduction of the tile, in the stage that W's last pair has left (free since the last barrier, asked for again only
    // in the next tile's first trip)
    Partial* red = reinterpret_cast<Partial*>(lds + wf);           // [4 waves of a half][kRwBM]
    // ---- row reduction of the tile: the maximum over this lane's vocabulary ids and the four lane groups first, so that
    // every exponential is taken relative to it and the rest are plain sums; then over the four waves of a position half.
    const int n0 = tile * kRwBN + wv * 64 + 4 * q;               // this lane's ids: n0 + 16 ib + r
    auto reduce = [&](auto ragged_c) {
#pragma unroll
    for (int jb = 0; jb < JH; ++jb) {
      // this row block's accumulators leave the accumulation registers here, not earlier (a register spilled without it)
#pragma unroll
      for (int ib = 0; ib < 4; ++ib) asm volatile("" : "+a"(acc[ib][jb]));
      int left = a.V - n0;
      if constexpr (decltype(ragged_c)::value) asm volatile("" : "+v"(left));    // (sixteen masks kept for all row blocks spill)
      float v[16];
#pragma unroll
      for (int ib = 0; ib < 4; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[ib * 4 + r] = !decltype(ragged_c)::value || 16 * ib + r < left ? acc[ib][jb][r] : -INFINITY;
      float m = kNegBig;
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, v[i]);
      m = row_allreduce(m, [](float x, float y) { return fmaxf(x, y); });
      int idx = 0x7fffffff;
#pragma unroll
      for (int i = 15; i >= 0; --i) idx = (v[i] == m) ? n0 + 16 * (i / 4) + i % 4 : idx;     // lowest id of a tie
      idx = row_allreduce(idx, [](int x, int y) { return min(x, y); });
      const float ml = m * kLog2e;
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) s += fast_exp2(fmaf(v[i], kLog2e, -ml));
      s = row_allreduce(s, [](float x, float y) { return x + y; });
      if (q == 0) red[wv * kRwBM + (wp * JH + jb) * 16 + l16] = Partial{m, s, idx};
    }
    };
    if ((tile + 1) * kRwBN <= a.V) reduce(std::false_type{});
    else reduce(std::true_type{});                 // the last tile runs past V
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (my_row >= 0) {
      Partial p = red[tid];
#pragma unroll
      for (int w = 1; w < 4; ++w) {
        const Partial p2 = red[w * kRwBM + tid];
        merge_partial(p.m, p.s, p.idx, p2.m, p2.s, p2.idx);
      }
      store_partial(a, my_row, tile, p);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // the stage is free again
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing of this workgroup's is in flight when it ends
}

// Into how many parts the vocabulary tiles of an XCD are cut, for nact row chunks each (parts x nact workgroups per XCD, one of
// them on a CU at a time).  Where the chunks divide the CUs every CU has one workgroup.  Otherwise the workgroups come in rounds,
// and what counts is the rounds times a workgroup's length: its tiles, each as long as its pairs of k-steps and one more for the
// reduction, and its start, which is two scans of all mask bytes and the first transfers.  Each lane prices a length of 1 to 64
// tiles; the longest of the cheapest is taken.  (The grid has room for one workgroup per tile and chunk.)
// One workgroup per CU for any number of chunks left CUs without work.  Row-major W, in us, one per CU / now (and with one per
// tile and chunk, of one wave per SIMD): 32000 x 2048, 1500 positions (6 chunks) 235 / 209 (208), 4352 (17) 775 / 585 (587),
// 8448 (33) 1646 / 1120 (1174); 126464 x 4096, 2600 positions (11) 2954 / 2638 (2601).
__device__ __forceinline__ int lm_rows_parts(const LmHeadArgs& a, int nact) {
  constexpr int kSlots = kNumCUs / kNumXCDs;
  if (kSlots % nact == 0) return kSlots / nact;
  const int nt = (a.ntile + kNumXCDs - 1) / kNumXCDs;
  const int t = (threadIdx.x & 63) + 1, rounds = (((nt + t - 1) / t) * nact + kSlots - 1) / kSlots;
  const float cost = (float)rounds * ((float)t * (float)(a.Hd / 64 + 1) + (float)(2 + a.rows_total / 1024));
  float best = cost;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) best = fminf(best, __shfl_xor(best, off));
  const int len = 64 - __builtin_clzll(__ballot(cost == best));
  return __builtin_amdgcn_readfirstlane((nt + len - 1) / len);
}

template <bool PACKED>
__global__ __launch_bounds__(kRwThreads, 2) void lm_head_rows_kernel(LmHeadArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  // the ring takes all of the LDS; before it starts, its place holds the list of masked rows
  int* row_of = reinterpret_cast<int*>(lds_raw);                           // kRwBM compacted row ids (-1 = none)
  int* wsum = row_of + kRwBM;                                              // kRwWaves

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // ---- the masked count decides how many row chunks there are
  const int total = lm_masked_count<kRwThreads>(a, wsum);
  if (total < max(a.min_masked, 1)) return;        // another shape's launch has this call, or nothing is masked
  // The rows go to as few chunks as their number allows, spread evenly and rounded up to 32: a chunk's matrix
  // instructions follow from the 16-row blocks it is built for, so 282 rows as 160 + 122 cost 320 rows' worth and not
  // the 512 of two full chunks (with the count above 128, an even share always exceeds 128 rows).
  const int share = (total + kRwBM - 1) / kRwBM;
  const int bm = (((total + share - 1) / share) + 31) & ~31;         // 160, 192, 224 or 256 rows
  const int nact = (total + bm - 1) / bm;          // <= share <= a.nchunk, since total <= rows_total
  // ---- workgroup -> (row chunk, every parts-th vocabulary tile of an XCD), the grid's first parts x nact of each XCD.  Chunks of a
  // tile share the id mod 8 (the XCD) and are adjacent in dispatch order: W comes from HBM once.
  const int slot = blockIdx.x >> 3, chunk = slot % nact, part = slot / nact, parts = lm_rows_parts(a, nact);
  const int tile0 = part * kNumXCDs + (blockIdx.x & 7);
  if (part >= parts || tile0 >= a.ntile) return;

  // ---- compact the masked rows; this workgroup takes compacted rows [lo, lo + bm)
  const int lo = chunk * bm;
  int running = 0;
  for (int base = 0; base < a.rows_total; base += kRwThreads) {
    const int i = base + tid;
    const bool f = i < a.rows_total && a.masked[i] != 0;
    const unsigned long long bal = __ballot(f);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kRwWaves; ++w) { const int c = wsum[w]; pre += (w < wave) ? c : 0; tot += c; }
    const int ci = running + pre + rank - lo;
    if (f && ci >= 0 && ci < bm) row_of[ci] = i;
    running += tot;
    __syncthreads();
    if (running >= lo + bm) break;                 // uniform: the chunk is full
  }
  const int n_valid = min(running - lo, bm);       // uniform, >= 1 because chunk < nact
  if (tid < bm && tid >= n_valid) row_of[tid] = -1;
  __syncthreads();

  switch (bm / 32) {                               // uniform
    case 8: lm_head_rows_tiles<PACKED, 16>(a, lds_raw, row_of, tile0, parts * kNumXCDs); break;
    case 7: lm_head_rows_tiles<PACKED, 14>(a, lds_raw, row_of, tile0, parts * kNumXCDs); break;
    case 6: lm_head_rows_tiles<PACKED, 12>(a, lds_raw, row_of, tile0, parts * kNumXCDs); break;
    default: lm_head_rows_tiles<PACKED, 10>(a, lds_raw, row_of, tile0, parts * kNumXCDs); break;
  }
}


// ---------------------------------------------------------------------------------------------------
// Stream shape (at most 32 positions in the block): the call is a read of W, so the kernel is built around
// that stream.  A workgroup owns 32 TT consecutive vocabulary rows (TT = 16: 512) and walks Hd in chunks of 512
// elements; within a chunk it visits its 16 sub-tiles of 32 rows one after the other, so that every
// wave-wide load is ONE KILOBYTE OF ONE ROW of W (registers -> LDS, swizzled, two stages, one barrier per
// sub-tile), and the matrix instructions read W back from LDS in operand layout.  The hidden rows never
// touch LDS: wave (ib, jb) computes vocabulary block ib x row block jb of every sub-tile, its B operands of
// a chunk (16 k-steps) sit in registers for all 16 sub-tiles and the next chunk's are asked for two
// sub-tiles ahead.  All 16 x (16 x 16) accumulators of a wave stay in registers until the end: one triple
// per (position, 512 vocabulary rows), a quarter of what the 128-row tiles of the other shapes write.
constexpr int kStSub = 32;                 // vocabulary rows per sub-tile
constexpr int kStTTMax = 20;               // most sub-tiles per workgroup: the accumulators a wave can hold
constexpr int kSt2TTMax = 16;              // the same with two row blocks per wave (33..64 positions)
constexpr int kStKC = 512;                 // elements of Hd per chunk (1 KB per row)
constexpr int kStKS = kStKC / 32;          // k-steps per chunk
constexpr int kStStage = kStSub * kStKC * 2;   // 32 KB

template <int TT>   // sub-tiles per workgroup (even: the two W stages alternate across chunk boundaries)
__global__ __launch_bounds__(kLmThreads) void lm_head_stream_kernel(LmHeadArgs a) {
  static_assert(TT % 2 == 0 && TT >= 2 && TT <= kStTTMax, "sub-tiles per workgroup");
  constexpr int kStTT = TT, kStRows = TT * kStSub;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  unsigned char* stage = lds_raw;                                            // 2 x kStStage
  int* row_of = reinterpret_cast<int*>(lds_raw + 2 * kStStage);              // 32 compacted row ids (-1 = none)
  Partial* red = reinterpret_cast<Partial*>(row_of + 32);                    // [waves][16]
  __shared__ int wsum[kLmWaves];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = blockIdx.x;                                               // < a.ntile by the grid size

  // ---- this launch works only if the masked count is in its range (another shape's launch has the call
  // otherwise); then the masked rows are compacted
  {
    const int total = lm_masked_count(a, wsum);
    if (total < a.min_masked || total > a.max_masked) return;
  }
  int running = 0;
  for (int base = 0; base < a.rows_total; base += kLmThreads) {
    const int i = base + tid;
    const bool f = i < a.rows_total && a.masked[i] != 0;
    const unsigned long long bal = __ballot(f);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kLmWaves; ++w) { const int c = wsum[w]; pre += (w < wave) ? c : 0; tot += c; }
    const int ci = running + pre + rank;
    if (f && ci < 32) row_of[ci] = i;
    running += tot;
    __syncthreads();
  }
  const int n_valid = min(running, 32);            // uniform
  if (n_valid <= 0) return;
  if (tid < 32 && tid >= n_valid) row_of[tid] = -1;
  __syncthreads();

  const int NCH = (a.Hd + kStKC - 1) / kStKC;      // chunks of Hd
  const int NU = NCH * kStTT;                      // (chunk, sub-tile) steps of the walk
  const int c0 = tile % NCH;                       // this workgroup's rotation of the chunk order
  const int q = lane >> 4, l16 = lane & 15;
  const int ib = wave & 1, jb = wave >> 1;
  const unsigned klast = (unsigned)(a.Hd - 8);     // last whole 16-byte piece of a row

  // W staging: this wave moves rows 8 wave + i (i = 0..7) of a sub-tile, lane l the l-th 16 bytes of the chunk
  const long long vrow0 = (long long)tile * kStRows + 8 * wave;
  unsigned sdst[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = 8 * wave + i;
    sdst[i] = (unsigned)(r * (kStKC * 2) + ((lane ^ (r & 15)) << 4));
  }
  auto load_w_sub = [&](int u, u32x4 (&dst)[8]) {          // step u of the walk (clamped to the last one)
    const int uc = min(u, NU - 1);
    const int kc = uc / kStTT, t = uc - kc * kStTT;
    int kcw = kc + c0; kcw -= (kcw >= NCH) ? NCH : 0;
    const unsigned k = min((unsigned)(kcw * kStKC + 8 * lane), klast);     // pieces past Hd: any valid piece
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const long long n = min(vrow0 + t * kStSub + i, (long long)a.V - 1);   // rows past V: any valid row
      // every byte of W is read once and whole lines at a time here: streaming loads (cfg2: 182 -> 172 us)
      dst[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(a.weight + n * a.ld_w + k));
    }
  };
  // B operands of a chunk for this wave's row block: row jb * 16 + l16, k-step ks, elements 8 q .. 8 q + 7
  const long long hrow = (long long)max(row_of[jb * 16 + l16], 0) * a.ld_h;
  auto load_b_chunk = [&](int kc, bf16x8 (&dst)[kStKS]) {  // chunk at walk position kc (clamped); zeros past Hd
    int kcw = min(kc, NCH - 1) + c0; kcw -= (kcw >= NCH) ? NCH : 0;
#pragma unroll
    for (int ks = 0; ks < kStKS; ++ks) {
      const unsigned k = (unsigned)(kcw * kStKC + 32 * ks + 8 * q);
      const unsigned keep = (k < (unsigned)a.Hd) ? 0xffffffffu : 0u;
      const u32x4 v = *reinterpret_cast<const u32x4*>(a.hidden + hrow + min(k, klast));
      dst[ks] = __builtin_bit_cast(bf16x8, v & u32x4{keep, keep, keep, keep});
    }
  };
  // A operand of k-step ks: row ib * 16 + l16 of the sub-tile, piece 4 ks + q, swizzled by the row
  const unsigned aoff = (unsigned)((ib * 16 + l16) * (kStKC * 2));

  f32x4 acc[kStTT];
#pragma unroll
  for (int t = 0; t < kStTT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- prologue: step 0 into stage 0, step 1 into registers, the first chunk's B operands
  u32x4 wreg[2][8];
  load_w_sub(0, wreg[0]);
  load_w_sub(1, wreg[1]);
  bf16x8 bcur[kStKS], bnext[kStKS];
  load_b_chunk(0, bcur);
#pragma unroll
  for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(stage + sdst[i]) = wreg[0][i];
  __syncthreads();

  // ---- main loop: chunks of Hd (rotated), 16 sub-tiles each; step u = kc * 16 + t reads stage u & 1
  for (int kc = 0; kc < NCH; ++kc) {
#pragma unroll
    for (int t = 0; t < kStTT; ++t) {
      const int u = kc * kStTT + t;
      // two steps ahead into the register set that was written to LDS one step ago
      load_w_sub(u + 2, wreg[t & 1]);
      if (t == kStTT - 2) load_b_chunk(kc + 1, bnext);
      __builtin_amdgcn_sched_barrier(0);
      const unsigned char* cur = stage + (t & 1) * kStStage;
#pragma unroll
      for (int ks = 0; ks < kStKS; ++ks) {
        const bf16x8 aop = *reinterpret_cast<const bf16x8*>(cur + aoff + (unsigned)(((4 * ks + q) ^ l16) << 4));
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bcur[ks], acc[t], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      // step u + 1 (asked for one step ago) into the other stage, which step u - 1 has finished reading
      unsigned char* nxt = stage + ((t + 1) & 1) * kStStage;
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(nxt + sdst[i]) = wreg[(t + 1) & 1][i];
      __syncthreads();
    }
#pragma unroll
    for (int ks = 0; ks < kStKS; ++ks) bcur[ks] = bnext[ks];
  }

  // ---- row reduction: this lane holds, for row jb * 16 + l16, the ids t * 32 + ib * 16 + 4 q + r of the tile
  float m = kNegBig; int idx = 0x7fffffff;
#pragma unroll
  for (int t = 0; t < kStTT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = tile * kStRows + t * kStSub + ib * 16 + 4 * q + r;
      float v = acc[t][r];
      if (n >= a.V) v = -INFINITY;
      acc[t][r] = v;
      if (v > m) { m = v; idx = n; }                 // ascending ids, strict: the lowest id keeps a tie
    }
  const float ml = m * kLog2e;
  float s = 0.f;
#pragma unroll
  for (int t = 0; t < kStTT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) s += fast_exp2(fmaf(acc[t][r], kLog2e, -ml));
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float m2 = __shfl_xor(m, off); const float s2 = __shfl_xor(s, off); const int i2 = __shfl_xor(idx, off);
    merge_partial(m, s, idx, m2, s2, i2);
  }
  if (q == 0) red[wave * 16 + l16] = Partial{m, s, idx};
  __syncthreads();
  if (tid < 32 && row_of[tid] >= 0) {
    const int rb = tid >> 4, l = tid & 15;           // row block, row inside it; its two waves are 2 rb and 2 rb + 1
    Partial p0 = red[(2 * rb) * 16 + l];
    const Partial p1 = red[(2 * rb + 1) * 16 + l];
    merge_partial(p0.m, p0.s, p0.idx, p1.m, p1.s, p1.idx);
    store_partial(a, row_of[tid], tile, p0);
  }
}

// Stream shape for 33..64 positions: same walk and the same W route as lm_head_stream_kernel, but a wave owns two
// 16-row blocks of positions, and the B operands of two chunks for two blocks (256 registers) do not fit beside
// its 128 accumulator registers.  The hidden chunk (64 rows x 1 KB) therefore lives in LDS, one stage: the next
// chunk is asked for at the start of a chunk, waits in registers, and is written between two barriers at the
// chunk's end; B operands are read from LDS per matrix instruction (a stream-bound kernel has the LDS cycles).
constexpr int kSt2Rows = 64;                               // positions per workgroup
constexpr int kSt2Hid = kSt2Rows * kStKC * 2;              // 64 KB: one hidden chunk

template <int TT>
__global__ __launch_bounds__(kLmThreads) void lm_head_stream64_kernel(LmHeadArgs a) {
  static_assert(TT % 2 == 0 && TT >= 2 && TT <= kSt2TTMax, "sub-tiles per workgroup");
  constexpr int kStTT = TT, kStRows = TT * kStSub;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  unsigned char* stage = lds_raw;                                            // 2 x kStStage (W ring)
  unsigned char* hid = lds_raw + 2 * kStStage;                               // kSt2Hid (hidden chunk)
  int* row_of = reinterpret_cast<int*>(hid + kSt2Hid);                       // 64 compacted row ids (-1 = none)
  Partial* red = reinterpret_cast<Partial*>(row_of + kSt2Rows);              // [waves][32]
  __shared__ int wsum[kLmWaves];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = blockIdx.x;                                               // < a.ntile by the grid size

  // ---- this launch works only if the masked count is in its range (another shape's launch has the call
  // otherwise); then the masked rows are compacted
  {
    const int total = lm_masked_count(a, wsum);
    if (total < a.min_masked || total > a.max_masked) return;
  }
  int running = 0;
  for (int base = 0; base < a.rows_total; base += kLmThreads) {
    const int i = base + tid;
    const bool f = i < a.rows_total && a.masked[i] != 0;
    const unsigned long long bal = __ballot(f);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kLmWaves; ++w) { const int c = wsum[w]; pre += (w < wave) ? c : 0; tot += c; }
    const int ci = running + pre + rank;
    if (f && ci < kSt2Rows) row_of[ci] = i;
    running += tot;
    __syncthreads();
  }
  const int n_valid = min(running, kSt2Rows);      // uniform
  if (n_valid <= 0) return;
  if (tid < kSt2Rows && tid >= n_valid) row_of[tid] = -1;
  __syncthreads();

  const int NCH = (a.Hd + kStKC - 1) / kStKC;      // chunks of Hd
  const int NU = NCH * kStTT;                      // (chunk, sub-tile) steps of the walk
  const int c0 = tile % NCH;                       // this workgroup's rotation of the chunk order
  const int q = lane >> 4, l16 = lane & 15;
  const int ib = wave & 1, jw = wave >> 1;         // vocabulary block of a sub-tile; row blocks 2 jw, 2 jw + 1
  const unsigned klast = (unsigned)(a.Hd - 8);     // last whole 16-byte piece of a row

  // W staging: this wave moves rows 8 wave + i (i = 0..7) of a sub-tile, lane l the l-th 16 bytes of the chunk
  const long long vrow0 = (long long)tile * kStRows + 8 * wave;
  unsigned sdst[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = 8 * wave + i;
    sdst[i] = (unsigned)(r * (kStKC * 2) + ((lane ^ (r & 15)) << 4));
  }
  auto load_w_sub = [&](int u, u32x4 (&dst)[8]) {          // step u of the walk (clamped to the last one)
    const int uc = min(u, NU - 1);
    const int kc = uc / kStTT, t = uc - kc * kStTT;
    int kcw = kc + c0; kcw -= (kcw >= NCH) ? NCH : 0;
    const unsigned k = min((unsigned)(kcw * kStKC + 8 * lane), klast);     // pieces past Hd: any valid piece
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const long long n = min(vrow0 + t * kStSub + i, (long long)a.V - 1);   // rows past V: any valid row
      dst[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(a.weight + n * a.ld_w + k));
    }
  };
  // hidden staging: this wave moves rows 16 wave + i (i = 0..15) of the chunk, lane l the l-th 16 bytes
  unsigned hsrc[16], hdst[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = 16 * wave + i;
    hsrc[i] = (unsigned)((long long)max(row_of[r], 0) * a.ld_h);           // B*K*ld_h < 2^31 is validated
    hdst[i] = (unsigned)(r * (kStKC * 2) + ((lane ^ (r & 15)) << 4));
  }
  auto load_hidden = [&](int kc, u32x4 (&dst)[16]) {       // chunk at walk position kc (clamped); zeros past Hd
    int kcw = min(kc, NCH - 1) + c0; kcw -= (kcw >= NCH) ? NCH : 0;
    const unsigned k = (unsigned)(kcw * kStKC + 8 * lane);
    const unsigned keep = (k < (unsigned)a.Hd) ? 0xffffffffu : 0u;
    const unsigned kk = min(k, klast);
#pragma unroll
    for (int i = 0; i < 16; ++i)
      dst[i] = *reinterpret_cast<const u32x4*>(a.hidden + hsrc[i] + kk) & u32x4{keep, keep, keep, keep};
  };
  // operands of k-step ks: A = row ib * 16 + l16 of the sub-tile, B = row (2 jw + rb) * 16 + l16 of the hidden
  // chunk; both piece 4 ks + q, swizzled by the row (row & 15 = l16 for both)
  const unsigned aoff = (unsigned)((ib * 16 + l16) * (kStKC * 2));
  const unsigned boff0 = (unsigned)(((2 * jw) * 16 + l16) * (kStKC * 2));
  const unsigned boff1 = boff0 + 16 * (kStKC * 2);

  f32x4 acc[kStTT][2];
#pragma unroll
  for (int t = 0; t < kStTT; ++t) { acc[t][0] = f32x4{0.f, 0.f, 0.f, 0.f}; acc[t][1] = f32x4{0.f, 0.f, 0.f, 0.f}; }

  // ---- prologue: W step 0 into stage 0, step 1 into registers, the first hidden chunk into LDS
  u32x4 wreg[2][8];
  u32x4 hreg[16];
  load_w_sub(0, wreg[0]);
  load_w_sub(1, wreg[1]);
  load_hidden(0, hreg);
#pragma unroll
  for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(stage + sdst[i]) = wreg[0][i];
#pragma unroll
  for (int i = 0; i < 16; ++i) *reinterpret_cast<u32x4*>(hid + hdst[i]) = hreg[i];
  __syncthreads();

  for (int kc = 0; kc < NCH; ++kc) {
    load_hidden(kc + 1, hreg);                     // waits in registers until the end of this chunk
#pragma unroll
    for (int t = 0; t < kStTT; ++t) {
      const int u = kc * kStTT + t;
      load_w_sub(u + 2, wreg[t & 1]);
      __builtin_amdgcn_sched_barrier(0);
      const unsigned char* cur = stage + (t & 1) * kStStage;
#pragma unroll
      for (int ks = 0; ks < kStKS; ++ks) {
        const unsigned po = (unsigned)(((4 * ks + q) ^ l16) << 4);
        const bf16x8 aop = *reinterpret_cast<const bf16x8*>(cur + aoff + po);
        const bf16x8 b0 = *reinterpret_cast<const bf16x8*>(hid + boff0 + po);
        const bf16x8 b1 = *reinterpret_cast<const bf16x8*>(hid + boff1 + po);
        acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, b0, acc[t][0], 0, 0, 0);
        acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, b1, acc[t][1], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      unsigned char* nxt = stage + ((t + 1) & 1) * kStStage;
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(nxt + sdst[i]) = wreg[(t + 1) & 1][i];
      __syncthreads();
    }
    // every wave has passed the barrier of the last sub-tile: nobody reads the hidden chunk any more
#pragma unroll
    for (int i = 0; i < 16; ++i) *reinterpret_cast<u32x4*>(hid + hdst[i]) = hreg[i];
    __syncthreads();
  }

  // ---- row reduction: this lane holds, for row (2 jw + rb) * 16 + l16, the ids t * 32 + ib * 16 + 4 q + r
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    float m = kNegBig; int idx = 0x7fffffff;
#pragma unroll
    for (int t = 0; t < kStTT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = tile * kStRows + t * kStSub + ib * 16 + 4 * q + r;
        float v = acc[t][rb][r];
        if (n >= a.V) v = -INFINITY;
        acc[t][rb][r] = v;
        if (v > m) { m = v; idx = n; }               // ascending ids, strict: the lowest id keeps a tie
      }
    const float ml = m * kLog2e;
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < kStTT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) s += fast_exp2(fmaf(acc[t][rb][r], kLog2e, -ml));
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float m2 = __shfl_xor(m, off); const float s2 = __shfl_xor(s, off); const int i2 = __shfl_xor(idx, off);
      merge_partial(m, s, idx, m2, s2, i2);
    }
    if (q == 0) red[wave * 32 + rb * 16 + l16] = Partial{m, s, idx};
  }
  __syncthreads();
  if (tid < kSt2Rows && row_of[tid] >= 0) {
    // position tid sits in row block tid / 16 = 2 jw + rb; its two waves are 2 jw (ib = 0) and 2 jw + 1 (ib = 1)
    const int blk = tid >> 4, l = tid & 15;
    const int w0 = 2 * (blk >> 1), rb = blk & 1;
    Partial p0 = red[w0 * 32 + rb * 16 + l];
    const Partial p1 = red[(w0 + 1) * 32 + rb * 16 + l];
    merge_partial(p0.m, p0.s, p0.idx, p1.m, p1.s, p1.idx);
    store_partial(a, row_of[tid], tile, p0);
  }
}

// Stream shape for 64 RB positions (RB = 2: 128).  The walk is the same, the route is not: W and the hidden rows
// go from global memory straight into LDS (global_load_lds_dwordx4, no staging registers, no LDS store
// instructions), so the registers hold accumulators and B operands only and the number of sub-tiles per
// workgroup needs no parity.  A chunk is 256 elements of Hd (8 k-steps), a sub-tile 32 vocabulary rows x 512
// bytes (16 KB; a transfer of one wave = two rows), the W ring has five stages and is filled four steps
// ahead.  A wave owns RB 16-row blocks of positions and both vocabulary blocks of a sub-tile; its hidden rows of
// the next chunk are transferred into a region of LDS that only this wave touches, as soon as it has read the
// current chunk's B operands from there into registers (8 RB reads per chunk).  No wave shares a position
// with another, so the row reduction ends in the wave.
// The transfers are inline assembly, invisible to the compiler's wait-count insertion: every wait for them
// is written out below, counted in transfers issued by the same wave after the one waited for (they complete
// in issue order), and the kernel has no other global load after its prologue.
constexpr int kDmSub = 32;                     // vocabulary rows per sub-tile
constexpr int kDmKC = 256;                     // elements of Hd per chunk (512 bytes per row)
constexpr int kDmKS = kDmKC / 32;              // k-steps per chunk
constexpr int kDmStage = kDmSub * kDmKC * 2;   // 16 KB
constexpr int kDmNST = 5;                      // W ring stages: filled kDmNST - 1 steps ahead (64 KB per CU in flight)
constexpr int kDmWT = kDmStage / 1024 / kLmWaves;   // W transfers per wave and step (4)
constexpr int kDmTTMax = 16;

// PACKED: W is the packed image; a transfer is then one operand tile (16 rows x one k-step, a contiguous
// kilobyte), the ring holds the tiles as they are and an A operand is read lane by lane, without a swizzle.
template <int TT, int RB, bool PACKED>
__global__ __launch_bounds__(kLmThreads) void lm_head_dma_kernel(LmHeadArgs a) {
  static_assert(TT >= 1 && TT <= kDmTTMax && (RB == 1 || RB == 2), "shape");
  constexpr int ROWS = kLmWaves * RB * 16;                                   // positions per workgroup
  constexpr int BT = RB * 8;                                                 // hidden transfers per wave and chunk
  constexpr int kHidWave = RB * 16 * kDmKC * 2;                              // bytes of a wave's hidden region
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  int* row_of = reinterpret_cast<int*>(lds_raw + kDmNST * kDmStage + kLmWaves * kHidWave);   // ROWS ids (-1 = none)
  __shared__ int wsum[kLmWaves];
  // LDS byte addresses (what m0 and the read instructions take)
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds_raw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned hid0 = lds0 + kDmNST * kDmStage + wave * kHidWave;          // this wave's hidden region
  const int tile = blockIdx.x;                                               // < a.ntile by the grid size

  // ---- this launch works only if the masked count is in its range (another shape's launch has the call
  // otherwise); then the masked rows are compacted
  {
    const int total = lm_masked_count(a, wsum);
    if (total < a.min_masked || total > a.max_masked) return;
  }
  int running = 0;
  for (int base = 0; base < a.rows_total; base += kLmThreads) {
    const int i = base + tid;
    const bool f = i < a.rows_total && a.masked[i] != 0;
    const unsigned long long bal = __ballot(f);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kLmWaves; ++w) { const int c = wsum[w]; pre += (w < wave) ? c : 0; tot += c; }
    const int ci = running + pre + rank;
    if (f && ci < ROWS) row_of[ci] = i;
    running += tot;
    __syncthreads();
  }
  const int n_valid = min(running, ROWS);          // uniform
  if (n_valid <= 0) return;
  if (tid < ROWS && tid >= n_valid) row_of[tid] = -1;
  __syncthreads();

  const int NCH = (a.Hd + kDmKC - 1) / kDmKC;      // chunks of Hd
  const int NU = NCH * TT;                         // (chunk, sub-tile) steps of the walk
  const int c0 = tile % NCH;                       // this workgroup's rotation of the chunk order
  const int q = lane >> 4, l16 = lane & 15;
  const unsigned klast = (unsigned)(a.Hd - 8);     // last whole 16-byte piece of a row
  const int half = lane >> 5, slot = lane & 31;    // a transfer covers two LDS rows of 32 slots
  auto chunk_at = [&](int kc) { int c = min(kc, NCH - 1) + c0; return c - ((c >= NCH) ? NCH : 0); };

  // W transfer j (0..3) of this wave fills rows 8 wave + 2 j + half of a sub-tile; LDS slot s of row r
  // holds piece s ^ (r & 15)
  unsigned wpiece[kDmWT];
#pragma unroll
  for (int j = 0; j < kDmWT; ++j) {
    const int r = 8 * wave + 2 * j + half;
    wpiece[j] = (unsigned)(slot ^ (r & 15));
  }
  const long long vrow0 = (long long)tile * (TT * kDmSub) + 8 * wave + half;
  const int NKS = a.Hd / 32, NB = (a.V + 15) / 16;             // k-steps, 16-row blocks (packed image)
  auto issue_w = [&](int u) {                      // step u of the walk (clamped to the last one) into stage u % 5
    const int uc = min(u, NU - 1);
    const int kc = uc / TT, t = uc - kc * TT;
    const unsigned st = lds0 + (unsigned)(u % kDmNST) * kDmStage + wave * (kDmWT * 1024);
    if constexpr (PACKED) {
      // transfer j of this wave is tile x = 4 wave + j of the 16 in a step: vocabulary block x / 8, k-step x % 8
      const int ks0 = chunk_at(kc) * kDmKS;
#pragma unroll
      for (int j = 0; j < kDmWT; ++j) {
        const int x = kDmWT * wave + j;
        const int nb = min((tile * TT + t) * 2 + x / kDmKS, NB - 1);           // blocks past V: the last one
        const int ks = min(ks0 + x % kDmKS, NKS - 1);                           // k-steps past Hd: the last one
        lm_dma16<true>(st + j * 1024, a.weight + (((long long)nb * NKS + ks) * 64 + lane) * 8);
      }
    } else {
      const unsigned kb = (unsigned)(chunk_at(kc) * kDmKC);
#pragma unroll
      for (int j = 0; j < kDmWT; ++j) {
        const long long n = min(vrow0 + t * kDmSub + 2 * j, (long long)a.V - 1);   // rows past V: any valid row
        const unsigned k = min(kb + 8 * wpiece[j], klast);                          // pieces past Hd: any valid piece
        lm_dma16<true>(st + j * 1024, a.weight + n * a.ld_w + k);
      }
    }
  };
  // hidden transfer j (0..BT-1) fills rows 2 j + half of this wave's region (row = rb * 16 + position in block)
  unsigned hoff[BT], hpiece[BT];
#pragma unroll
  for (int j = 0; j < BT; ++j) {
    const int r = 2 * j + half;                    // 0 .. RB * 16 - 1
    hoff[j] = (unsigned)((long long)max(row_of[wave * RB * 16 + r], 0) * a.ld_h);   // B*K*ld_h < 2^31 is validated
    hpiece[j] = (unsigned)(slot ^ (r & 15));
  }
  auto issue_b = [&](int kc) {                     // chunk at walk position kc (clamped to the last one)
    const unsigned kb = (unsigned)(chunk_at(kc) * kDmKC);
#pragma unroll
    for (int j = 0; j < BT; ++j)
      lm_dma16<false>(hid0 + j * 1024, a.hidden + hoff[j] + min(kb + 8 * hpiece[j], klast));
  };
  // operand reads: row (block * 16 + l16), piece 4 ks + q, swizzled by the row (row & 15 = l16)
  bf16x8 bcur[kDmKS][RB];
  auto read_b = [&](int kc) {                      // this wave's region -> registers; zeros past Hd
    const unsigned kb = (unsigned)(chunk_at(kc) * kDmKC);
#pragma unroll
    for (int ks = 0; ks < kDmKS; ++ks) {
      const unsigned keep = (kb + 32 * ks + 8 * q < (unsigned)a.Hd) ? 0xffffffffu : 0u;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const unsigned off = (unsigned)((rb * 16 + l16) * (kDmKC * 2) + (((4 * ks + q) ^ l16) << 4));
        const u32x4 v = *reinterpret_cast<const u32x4*>(lds_raw + kDmNST * kDmStage + wave * kHidWave + off);
        bcur[ks][rb] = __builtin_bit_cast(bf16x8, v & u32x4{keep, keep, keep, keep});
      }
    }
  };

  f32x4 acc[TT][2][RB];
#pragma unroll
  for (int t = 0; t < TT; ++t)
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[t][ib][rb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- prologue: the first chunk's hidden rows, steps 0..2 of W
  issue_b(0);
#pragma unroll
  for (int u = 0; u < kDmNST - 1; ++u) issue_w(u);
  lm_wait_vmcnt<0>();
  __syncthreads();

  for (int kc = 0; kc < NCH; ++kc) {
    // the hidden rows of this chunk were asked for at the start of the chunk before (or in the prologue);
    // issued after them by this wave: that chunk's TT steps of W
    lm_wait_vmcnt<(TT * kDmWT < 63 ? TT * kDmWT : 63)>();
    read_b(kc);
    // the next chunk's rows may only start to arrive in the region once these reads have returned
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue_b(kc + 1);
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int u = kc * TT + t;
      issue_w(u + kDmNST - 1);                     // into the stage that step u - 1 has finished reading
      __builtin_amdgcn_sched_barrier(0);
      const unsigned char* cur = lds_raw + (unsigned)(u % kDmNST) * kDmStage;
      // all A operands of the step are asked for at once: the matrix instructions then run back to back,
      // each waiting only for its own operand
      bf16x8 aop[kDmKS][2];
#pragma unroll
      for (int ks = 0; ks < kDmKS; ++ks) {
        if constexpr (PACKED) {
          aop[ks][0] = *reinterpret_cast<const bf16x8*>(cur + ks * 1024 + lane * 16);
          aop[ks][1] = *reinterpret_cast<const bf16x8*>(cur + (kDmKS + ks) * 1024 + lane * 16);
        } else {
          const unsigned po = (unsigned)(l16 * (kDmKC * 2) + (((4 * ks + q) ^ l16) << 4));
          aop[ks][0] = *reinterpret_cast<const bf16x8*>(cur + po);
          aop[ks][1] = *reinterpret_cast<const bf16x8*>(cur + 16 * (kDmKC * 2) + po);
        }
      }
      __builtin_amdgcn_sched_barrier(0);           // (the scheduler would sink the reads back between the MFMAs)
#pragma unroll
      for (int ks = 0; ks < kDmKS; ++ks)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          acc[t][0][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop[ks][0], bcur[ks][rb], acc[t][0][rb], 0, 0, 0);
          acc[t][1][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop[ks][1], bcur[ks][rb], acc[t][1][rb], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      // step u + 1 must have landed before the barrier: issued after it by this wave are the D = kDmNST - 2
      // steps u + 2 .. u + kDmNST - 1 (one in each of the steps u - D + 1 .. u), and the next chunk's hidden
      // rows wherever one of those steps began a chunk (t < D; with TT < D more than one of them may have)
      constexpr int D = kDmNST - 2;
      const int chunk_starts = TT >= D ? (t < D ? 1 : 0) : (D - 1 - t) / TT + 1;
      static_assert(D * kDmWT + D * BT <= 63, "vmcnt");
      if (chunk_starts == 0) lm_wait_vmcnt<D * kDmWT>();
      else if (chunk_starts == 1) lm_wait_vmcnt<D * kDmWT + BT>();
      else if (chunk_starts == 2) lm_wait_vmcnt<D * kDmWT + 2 * BT>();
      else lm_wait_vmcnt<D * kDmWT + 3 * BT>();
      __syncthreads();
    }
  }
  lm_wait_vmcnt<0>();                              // nothing of this workgroup's is in flight when it ends

  // ---- row reduction: this lane holds, for row (wave RB + rb) * 16 + l16, the ids t * 32 + ib * 16 + 4 q + r
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    float m = kNegBig; int idx = 0x7fffffff;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int n = tile * (TT * kDmSub) + t * kDmSub + ib * 16 + 4 * q + r;
          float v = acc[t][ib][rb][r];
          if (n >= a.V) v = -INFINITY;
          acc[t][ib][rb][r] = v;
          if (v > m) { m = v; idx = n; }             // ascending ids, strict: the lowest id keeps a tie
        }
    const float ml = m * kLog2e;
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) s += fast_exp2(fmaf(acc[t][ib][rb][r], kLog2e, -ml));
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float m2 = __shfl_xor(m, off); const float s2 = __shfl_xor(s, off); const int i2 = __shfl_xor(idx, off);
      merge_partial(m, s, idx, m2, s2, i2);
    }
    const int row = row_of[(wave * RB + rb) * 16 + l16];
    if (q == 0 && row >= 0) store_partial(a, row, tile, Partial{m, s, idx});
  }
}

// ---------------------------------------------------------------------------------------------------
// The packed image of W: one wave per operand tile (16 vocabulary rows x one k-step = one kilobyte).
__global__ __launch_bounds__(kLmThreads) void lm_head_pack_kernel(const uint16_t* __restrict__ W, long long ld_w,
                                                                  int V, int NK, long long ntiles, u32x4* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const long long g = (long long)blockIdx.x * kLmWaves + (threadIdx.x >> 6);     // tile: block g / NK, k-step g % NK
  if (g >= ntiles) return;
  const long long nb = g / NK;
  const int ks = (int)(g - nb * NK);
  const long long row = min(nb * 16 + (lane & 15), (long long)V - 1);             // rows past V repeat the last row
  out[g * 64 + lane] = *reinterpret_cast<const u32x4*>(W + row * ld_w + ks * 32 + 8 * (lane >> 4));
}

// Stream shape for at most 32 positions over a packed W.  Nothing is shared between the waves but the list of
// masked rows: a wave owns TT 16-row vocabulary blocks and both row blocks of positions, loads its A operands
// straight from the image (every load of a wave is one contiguous kilobyte, nontemporal) and keeps the B operands of
// a chunk of 8 k-steps in registers, the next chunk's beside them.  No LDS and no barrier in the loop.
// Bound by the stream of W.  A chunk is walked block by block, a block's 8 k-steps in a row: eight contiguous kilobytes at
// a time, two such runs in flight per wave.  Walked k-step by k-step (one kilobyte of each block in turn, as many bytes in
// flight) the blocks' starts, Hd x 32 bytes apart, met in the same memory channels where Hd is a power of two: 126464 x 4096
// 175.6 -> 163.5 us per call with 16 masked positions, 181 -> 165 with 32 (the kernel alone 153 us, 6.8 TB/s; a plain read 7.0), 32000 x 4096 59.7 ->
// 53.7, 8000 x 768 21.1 -> 19.4; 152064 x 3584 170.4 and 171.1, 50257 x 1600 41.8 both.
constexpr int kPkKS = 8;                       // k-steps per chunk of B operands
constexpr int kPkPF = 2;                       // vocabulary blocks (chunks of 8 KB) of A operands in flight per wave
constexpr int kPkTTMax = 10;

template <int TT>
__global__ __launch_bounds__(kLmThreads) void lm_head_packed_kernel(LmHeadArgs a) {
  static_assert(TT >= 1 && TT <= kPkTTMax, "shape");
  __shared__ int row_of[32];                     // compacted row ids (-1 = none)
  __shared__ Partial red[kLmWaves][32];
  __shared__ int wsum[kLmWaves];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = blockIdx.x;                   // < a.ntile by the grid size

  {
    const int total = lm_masked_count(a, wsum);
    if (total < a.min_masked || total > a.max_masked) return;
  }
  int running = 0;
  for (int base = 0; base < a.rows_total; base += kLmThreads) {
    const int i = base + tid;
    const bool f = i < a.rows_total && a.masked[i] != 0;
    const unsigned long long bal = __ballot(f);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(bal);
    __syncthreads();
    int pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kLmWaves; ++w) { const int c = wsum[w]; pre += (w < wave) ? c : 0; tot += c; }
    const int ci = running + pre + rank;
    if (f && ci < 32) row_of[ci] = i;
    running += tot;
    __syncthreads();
  }
  const int n_valid = min(running, 32);            // uniform
  if (n_valid <= 0) return;
  if (tid < 32 && tid >= n_valid) row_of[tid] = -1;
  __syncthreads();

  const int NK = a.Hd / 32;                        // k-steps
  const int NCH = (NK + kPkKS - 1) / kPkKS;        // chunks
  const int NB = (a.V + 15) / 16;                  // 16-row blocks of the image
  const int q = lane >> 4, l16 = lane & 15;
  // This workgroup's rotation of the chunk order.  With exactly eight chunks, blocks 64 KB apart, tile % NCH would be the number of
  // the chip part and all of its workgroups would read the same columns at a time: 126464 x 2048 112 -> 91 us per call, 100000 x 2048
  // 106 -> 76, 152064 and 32000 rows level (walked k-step by k-step, 100 and 98).  Other widths of eight chunks, whose blocks do
  // not start on the same address bits, are level or up to 7 % slower that way, and so is 1024 with its four chunks.
  const int c0 = (NK == kNumXCDs * kPkKS ? tile >> 3 : tile) % NCH;
  auto chunk_at = [&](int c) { int ch = min(c, NCH - 1) + c0; return ch - ((ch >= NCH) ? NCH : 0); };
  // A operands: block nb0 + t of the image, this lane's 16 bytes of every k-step 512 elements apart
  const int nb0 = (tile * kLmWaves + wave) * TT;
  const uint16_t* wblk[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) wblk[t] = a.weight + ((long long)min(nb0 + t, NB - 1) * NK * 64 + lane) * 8;
  auto load_a = [&](int c, int t, bf16x8 (&dst)[kPkKS]) {        // block t's k-steps of the chunk at walk position c
    const int k0 = chunk_at(c) * kPkKS;
#pragma unroll
    for (int ks = 0; ks < kPkKS; ++ks) {           // k-steps past Hd: the last one (its B operands are zeros)
      const long long off = (long long)min(k0 + ks, NK - 1) * 512;
      dst[ks] = __builtin_bit_cast(bf16x8, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wblk[t] + off)));
    }
  };
  // B operands: hidden row of position rb * 16 + l16, elements 8 q .. 8 q + 7 of every k-step of a chunk
  const uint16_t* hrow[2];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) hrow[rb] = a.hidden + (long long)max(row_of[rb * 16 + l16], 0) * a.ld_h + 8 * q;
  // (loaded as they are; k-steps past Hd are zeroed when the chunk becomes the current one: a mask applied at
  // the load would make the compiler wait for it there, behind every A load in flight)
  auto load_b = [&](int c, u32x4 (&dst)[kPkKS][2]) {             // chunk at walk position c
    const int k0 = chunk_at(c) * kPkKS;
#pragma unroll
    for (int ks = 0; ks < kPkKS; ++ks) {
      const int kk = min(k0 + ks, NK - 1);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) dst[ks][rb] = *reinterpret_cast<const u32x4*>(hrow[rb] + 32 * kk);
    }
  };
  auto take_b = [&](int c, const u32x4 (&src)[kPkKS][2], bf16x8 (&dst)[kPkKS][2]) {   // zeros past Hd
    const int k0 = chunk_at(c) * kPkKS;
#pragma unroll
    for (int ks = 0; ks < kPkKS; ++ks) {
      const unsigned keep = (k0 + ks < NK) ? 0xffffffffu : 0u;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) dst[ks][rb] = __builtin_bit_cast(bf16x8, src[ks][rb] & u32x4{keep, keep, keep, keep});
    }
  };

  f32x4 acc[TT][2];
#pragma unroll
  for (int t = 0; t < TT; ++t) { acc[t][0] = f32x4{0.f, 0.f, 0.f, 0.f}; acc[t][1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  bf16x8 abuf[kPkPF][kPkKS];                     // items (chunk, block) i and i + 1 of the walk; item i = c TT + t
  bf16x8 bcur[kPkKS][2];
  u32x4 bnext[kPkKS][2];
  load_b(0, bnext);
#pragma unroll
  for (int i = 0; i < kPkPF; ++i) load_a(i / TT, i % TT, abuf[i]);
  take_b(0, bnext, bcur);

  constexpr int U = TT % kPkPF == 0 ? 1 : kPkPF; // chunks per unrolled body, so that an item's buffer is known
  static_assert(U * TT % kPkPF == 0, "buffers");
  for (int kc0 = 0; kc0 < NCH; kc0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kc = kc0 + u;
      if (U > 1 && kc >= NCH) break;               // uniform
      load_b(kc + 1, bnext);                       // older than every A load below: it is back before they are
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        constexpr int PF = kPkPF;
        bf16x8 (&cur)[kPkKS] = abuf[(u * TT + t) % PF];
#pragma unroll
        for (int ks = 0; ks < kPkKS; ++ks) {
          acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur[ks], bcur[ks][0], acc[t][0], 0, 0, 0);
          acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur[ks], bcur[ks][1], acc[t][1], 0, 0, 0);
        }
        load_a(kc + (t + PF) / TT, (t + PF) % TT, cur);
        __builtin_amdgcn_sched_barrier(0);
      }
      take_b(kc + 1, bnext, bcur);
    }
  }

  // ---- row reduction: this lane holds, for position rb * 16 + l16, the ids (nb0 + t) * 16 + 4 q + r
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    float m = kNegBig; int idx = 0x7fffffff;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int n = (nb0 + t) * 16 + 4 * q + r;
        float v = acc[t][rb][r];
        if (n >= a.V) v = -INFINITY;
        acc[t][rb][r] = v;
        if (v > m) { m = v; idx = n; }               // ascending ids, strict: the lowest id keeps a tie
      }
    const float ml = m * kLog2e;
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) s += fast_exp2(fmaf(acc[t][rb][r], kLog2e, -ml));
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float m2 = __shfl_xor(m, off); const float s2 = __shfl_xor(s, off); const int i2 = __shfl_xor(idx, off);
      merge_partial(m, s, idx, m2, s2, i2);
    }
    if (q == 0) red[wave][rb * 16 + l16] = Partial{m, s, idx};
  }
  __syncthreads();
  if (tid < 32 && row_of[tid] >= 0) {
    Partial p = red[0][tid];                         // waves hold ascending vocabulary ranges
#pragma unroll
    for (int w = 1; w < kLmWaves; ++w) merge_partial(p.m, p.s, p.idx, red[w][tid].m, red[w][tid].s, red[w][tid].idx);
    store_partial(a, row_of[tid], tile, p);
  }
}

// ---- host side ----
// The kernel shapes, by the masked counts they serve.  Row-major W: up to 32 (stream, B operands in
// registers), up to 64 (stream, hidden chunk in LDS), up to 128 (stream, global -> LDS transfers), any (256-row
// chunks).  Packed W: up to 32 (operands straight from the image), up to 64 and up to 128 (global -> LDS
// transfers of operand tiles), any (256-row chunks).
enum { kShape32 = 0, kShape64, kShape128, kShapeRows, kNumShapes };
constexpr int kShapeMax[kNumShapes] = {32, kSt2Rows, 128, INT_MAX};

// Sub-tiles per workgroup of a stream kernel, out of the counts it is compiled for.  One workgroup per CU is
// resident, so a launch runs in rounds of kNumCUs workgroups and costs about rounds x (sub-tiles + a half for
// the prologue): 126464 vocabulary rows take 16 sub-tiles (247 workgroups), 152064 take 20 (238 workgroups; 16
// would leave 41 of 297 for a second round) or, where the accumulators allow no more, 10 (476, two rounds).
constexpr int kStTTs[] = {2, 4, 8, 12, 16, 20};
constexpr int kSt2TTs[] = {2, 4, 8, 10, 12, 16};
constexpr int kDmTTs[] = {1, 2, 3, 4, 6, 8, 10, 16};
constexpr int kPkTTs[] = {1, 2, 4, 6, 8, 10};      // 16-row blocks per wave: 64 rows per workgroup each
constexpr int kPkSub = kLmWaves * 16;
static_assert(kStSub == kDmSub, "one sub-tile size for the tile-size choice");

template <size_t N>
static int stream_tt(int V, const int (&tts)[N], int sub = kStSub) {
  const int nsub = (V + sub - 1) / sub;
  int best = tts[0];
  long long best_cost = LLONG_MAX;
  for (int tt : tts) {
    const int ntile = (nsub + tt - 1) / tt;
    const long long cost = (long long)((ntile + kNumCUs - 1) / kNumCUs) * (2 * tt + 1);
    if (cost <= best_cost) { best_cost = cost; best = tt; }     // ties: fewer, larger tiles
  }
  return best;
}

// top: the shape for B x K positions all masked; the shapes below it are launched too and serve the smaller
// masked counts; ntile_out is the largest tile count among the launched shapes.
// first: the smallest shape launched.  Over a packed W, where both would be launched, the 64-position kernel serves 1..64 masked
// positions and the call has one idle launch less.  Call with up to 32 masked of 40 to 256 positions, us, with it / with the
// 32-position kernel launched too: 8000 x 768 16 / 16-26, 32000 x 4096 56-61 / 55-70, 50257 x 1600 39-43 / 39-50, 126464 x 2048
// 108-116 / 112-124, 100000 x 5120 163-168 / 161-180, 152064 x 3584 173-185 / 172-182; only 126464 x 4096, where the 64-position
// kernel's blocks start in the same memory channels, prefers the other: 175-184 / 162-172.  With 33 to 64 masked the idle launch
// costs 1-2 % (8000 x 768: 11 %).
struct LmPlan { int first, top, nchunk, packed, tt[kNumShapes], bn[kNumShapes], ntile[kNumShapes], ntile_out; };

static LmPlan lm_plan(const sdllm_lm_head_params& p) {
  const long long rows = (long long)p.B * p.K;
  LmPlan pl;
  pl.packed = p.weight_packed;
  int sub[kNumShapes] = {kStSub, kStSub, kStSub, 256};
  if (pl.packed) {
    pl.tt[kShape32] = stream_tt(p.V, kPkTTs, kPkSub); sub[kShape32] = kPkSub;
    pl.tt[kShape64] = stream_tt(p.V, kDmTTs);
  } else {
    pl.tt[kShape32] = stream_tt(p.V, kStTTs);
    pl.tt[kShape64] = stream_tt(p.V, kSt2TTs);
  }
  pl.tt[kShape128] = stream_tt(p.V, kDmTTs);
  pl.tt[kShapeRows] = 1;                  // 256-row tiles (also for a half-empty chunk: it beat 128-row tiles)
  pl.top = 0;
  while (rows > kShapeMax[pl.top]) ++pl.top;
  pl.first = (pl.packed && pl.top > kShape32) ? kShape64 : kShape32;
  pl.ntile_out = 0;
  for (int i = 0; i < kNumShapes; ++i) {
    pl.bn[i] = pl.tt[i] * sub[i];
    pl.ntile[i] = (p.V + pl.bn[i] - 1) / pl.bn[i];
    if (i >= pl.first && i <= pl.top) pl.ntile_out = std::max(pl.ntile_out, pl.ntile[i]);
  }
  pl.nchunk = pl.top == kShapeRows ? (int)((rows + 255) / 256) : 1;
  return pl;
}

constexpr size_t dma_lds_bytes(int rb) {
  return (size_t)kDmNST * kDmStage + (size_t)kLmWaves * (rb * 16 * kDmKC * 2) + (size_t)kLmWaves * rb * 16 * sizeof(int);
}

static size_t lm_lds_bytes(int shape, int packed) {
  switch (shape) {
    case kShape32: return packed ? 0 : 2 * (size_t)kStStage + 32 * sizeof(int) + (size_t)kLmWaves * 16 * sizeof(Partial);
    case kShape64: return packed ? dma_lds_bytes(1)
                                 : 2 * (size_t)kStStage + kSt2Hid + kSt2Rows * sizeof(int) + (size_t)kLmWaves * 32 * sizeof(Partial);
    case kShape128: return dma_lds_bytes(2);
    default: return kRwLds;
  }
}

void lm_head_plan(const sdllm_lm_head_params& p, sdllm_lm_head_plan* plan) {
  const LmPlan pl = lm_plan(p);
  const int t = pl.top;
  plan->rows_per_chunk = t == kShapeRows ? 256 : kShapeMax[t];
  plan->vocab_rows_per_tile = pl.bn[t]; plan->vocab_tiles = pl.ntile[t];
  plan->row_chunks = pl.nchunk;
  plan->workgroups = t != kShapeRows ? pl.ntile[t] : ((pl.ntile[t] + kNumXCDs - 1) / kNumXCDs) * pl.nchunk * kNumXCDs;
  plan->lds_bytes = (int32_t)lm_lds_bytes(t, pl.packed);
  plan->triples_per_position = pl.ntile_out;
}

size_t lm_head_workspace_bytes(const sdllm_lm_head_params& p) {
  return (size_t)p.B * p.K * lm_plan(p).ntile_out * sizeof(Partial);
}

size_t lm_head_packed_weight_bytes(int V, int Hd) {
  return (size_t)((V + 15) / 16) * (size_t)(Hd / 32) * 1024;
}

hipError_t launch_lm_head_pack_weight(int V, int Hd, long long ld_w, const void* weight, void* packed, hipStream_t stream) {
  const int NK = Hd / 32;
  const long long ntiles = (long long)((V + 15) / 16) * NK;
  const long long grid = (ntiles + kLmWaves - 1) / kLmWaves;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(lm_head_pack_kernel, dim3((unsigned)grid), dim3(kLmThreads), 0, stream,
                     (const uint16_t*)weight, ld_w, V, NK, ntiles, (u32x4*)packed);
  return hipGetLastError();
}

// One launch, or (r.hidden == nullptr: the preparation pass of sdllm_init) only the kernel's opt-in to its
// dynamic LDS size on the current device.
static hipError_t launch_kernel(void (*kernel)(LmHeadArgs), LdsOptIn& st, size_t lds, unsigned grid,
                                const LmHeadArgs& r, hipStream_t stream, int threads = kLmThreads) {
  hipError_t e = ensure_lds_opt_in(reinterpret_cast<const void*>(kernel), lds, st);
  if (e != hipSuccess || r.hidden == nullptr) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, stream, r);
  return hipGetLastError();
}

template <int TT>
static hipError_t launch_stream32(const LmHeadArgs& r, hipStream_t stream) {
  static LdsOptIn st;
  return launch_kernel(lm_head_stream_kernel<TT>, st, lm_lds_bytes(kShape32, 0), (unsigned)r.ntile, r, stream);
}
template <int TT>
static hipError_t launch_stream64(const LmHeadArgs& r, hipStream_t stream) {
  static LdsOptIn st;
  return launch_kernel(lm_head_stream64_kernel<TT>, st, lm_lds_bytes(kShape64, 0), (unsigned)r.ntile, r, stream);
}
template <int TT>
static hipError_t launch_packed32(const LmHeadArgs& r, hipStream_t stream) {
  static LdsOptIn st;
  return launch_kernel(lm_head_packed_kernel<TT>, st, 0, (unsigned)r.ntile, r, stream);
}
template <int TT, int RB, bool PACKED>
static hipError_t launch_dma(const LmHeadArgs& r, hipStream_t stream) {
  static LdsOptIn st;
  return launch_kernel(lm_head_dma_kernel<TT, RB, PACKED>, st, dma_lds_bytes(RB), (unsigned)r.ntile, r, stream);
}
template <int RB, bool PACKED>
static hipError_t launch_dma_tt(int tt, const LmHeadArgs& r, hipStream_t stream) {
  switch (tt) {                        // kDmTTs
    case 1: return launch_dma<1, RB, PACKED>(r, stream);
    case 2: return launch_dma<2, RB, PACKED>(r, stream);
    case 3: return launch_dma<3, RB, PACKED>(r, stream);
    case 4: return launch_dma<4, RB, PACKED>(r, stream);
    case 6: return launch_dma<6, RB, PACKED>(r, stream);
    case 8: return launch_dma<8, RB, PACKED>(r, stream);
    case 10: return launch_dma<10, RB, PACKED>(r, stream);
    case 16: return launch_dma<16, RB, PACKED>(r, stream);
  }
  return hipErrorInvalidValue;
}
static hipError_t launch_rows(const LmHeadArgs& r, hipStream_t stream) {
  static LdsOptIn st[2];
  const unsigned grid = (unsigned)(((r.ntile + kNumXCDs - 1) / kNumXCDs) * r.nchunk * kNumXCDs);
  if (r.packed) return launch_kernel(lm_head_rows_kernel<true>, st[1], lm_lds_bytes(kShapeRows, 1), grid, r, stream, kRwThreads);
  return launch_kernel(lm_head_rows_kernel<false>, st[0], lm_lds_bytes(kShapeRows, 0), grid, r, stream, kRwThreads);
}

static hipError_t launch_shape(int shape, int tt, const LmHeadArgs& r, hipStream_t stream) {
  switch (shape) {
    case kShape32:
      if (r.packed) switch (tt) {      // kPkTTs
        case 1: return launch_packed32<1>(r, stream);
        case 2: return launch_packed32<2>(r, stream);
        case 4: return launch_packed32<4>(r, stream);
        case 6: return launch_packed32<6>(r, stream);
        case 8: return launch_packed32<8>(r, stream);
        case 10: return launch_packed32<10>(r, stream);
      } else switch (tt) {             // kStTTs
        case 2: return launch_stream32<2>(r, stream);
        case 4: return launch_stream32<4>(r, stream);
        case 8: return launch_stream32<8>(r, stream);
        case 12: return launch_stream32<12>(r, stream);
        case 16: return launch_stream32<16>(r, stream);
        case 20: return launch_stream32<20>(r, stream);
      }
      break;
    case kShape64:
      if (r.packed) return launch_dma_tt<1, true>(tt, r, stream);
      switch (tt) {                    // kSt2TTs
        case 2: return launch_stream64<2>(r, stream);
        case 4: return launch_stream64<4>(r, stream);
        case 8: return launch_stream64<8>(r, stream);
        case 10: return launch_stream64<10>(r, stream);
        case 12: return launch_stream64<12>(r, stream);
        case 16: return launch_stream64<16>(r, stream);
      }
      break;
    case kShape128:
      return r.packed ? launch_dma_tt<2, true>(tt, r, stream) : launch_dma_tt<2, false>(tt, r, stream);
    case kShapeRows: return launch_rows(r, stream);
  }
  return hipErrorInvalidValue;      // not reached: lm_plan picks from the same lists
}

// Every kernel shape and tile size the plan can pick, for both weight layouts: opt-ins only, nothing is launched.
hipError_t prepare_lm_head() {
  LmHeadArgs r{};
  r.hidden = nullptr; r.ntile = 1; r.nchunk = 1;
  hipError_t e = hipSuccess;
  for (int packed = 0; packed <= 1 && e == hipSuccess; ++packed) {
    r.packed = packed;
    if (packed) { for (int tt : kPkTTs) if (e == hipSuccess) e = launch_shape(kShape32, tt, r, nullptr); }
    else        { for (int tt : kStTTs) if (e == hipSuccess) e = launch_shape(kShape32, tt, r, nullptr); }
    if (packed) { for (int tt : kDmTTs) if (e == hipSuccess) e = launch_shape(kShape64, tt, r, nullptr); }
    else        { for (int tt : kSt2TTs) if (e == hipSuccess) e = launch_shape(kShape64, tt, r, nullptr); }
    for (int tt : kDmTTs) if (e == hipSuccess) e = launch_shape(kShape128, tt, r, nullptr);
    if (e == hipSuccess) e = launch_shape(kShapeRows, 1, r, nullptr);
  }
  return e;
}

hipError_t launch_lm_head_unmask(const sdllm_lm_head_params& p, const void* hidden, const void* weight,
                                 int32_t* tokens, uint8_t* masked, float* confidence, int32_t* n_committed,
                                 uint8_t* block_done, uint8_t* eos_seen, void* workspace, hipStream_t stream) {
  const LmPlan pl = lm_plan(p);
  LmHeadArgs r;
  r.hidden = (const uint16_t*)hidden; r.weight = (const uint16_t*)weight; r.masked = masked;
  r.partials = (Partial*)workspace;
  r.ld_h = p.ld_h; r.ld_w = p.ld_w;
  r.rows_total = p.B * p.K; r.V = p.V; r.Hd = p.Hd;
  r.nchunk = pl.nchunk; r.ntile_out = pl.ntile_out; r.packed = pl.packed;
  hipError_t e = hipSuccess;
  // every shape up to the one that B x K needs: the smaller ones take the call when few enough positions are
  // still masked (the later steps of a block); each launch exits unless the masked count is in its range
  for (int i = pl.first; i <= pl.top && e == hipSuccess; ++i) {
    r.ntile = pl.ntile[i];
    r.min_masked = i == pl.first ? 1 : kShapeMax[i - 1] + 1;
    r.max_masked = i == pl.top ? INT_MAX : kShapeMax[i];
    e = launch_shape(i, pl.tt[i], r, stream);
  }
  if (e != hipSuccess) return e;

  UnmaskArgs u;
  u.logits = nullptr; u.partials = (Partial*)workspace;
  u.tokens = tokens; u.masked = masked; u.confidence = confidence;
  u.n_committed = n_committed; u.block_done = block_done; u.eos_seen = eos_seen;
  u.ld = 0; u.V = p.V; u.nvec = 0; u.vec_per_split = 0;
  u.nsplit = pl.ntile_out; u.nsplit_p2 = 1; u.K = p.K;
  u.tau0 = p.tau0; u.alpha = p.alpha; u.r_extra_masked = p.r_extra_masked; u.r_extra_total = p.r_extra_total;
  u.eos_id = p.eos_id; u.tau_eos = p.tau_eos;
  return launch_unmask_commit(u, p.B, stream);
}

}  // namespace sdllm
