// Prefix (and pool) expansion on the matrix cores (paper Section 3.1 "Prefill": the shared part of
// the latent caches is expanded through the up-projection into per-head K and V):
//     K[h, t, 0:128] = W_UK[h] c_t,   K[h, t, 128:192] = r_t,   V[h, t, :] = W_UV[h] c_t
// i.e. one GEMM [tokens x 512] x [512 x 256 H] whose epilogue writes the matrix-core operand
// order the decode kernels read (see typhoon_mla.h).
//
// MFMA-bound in principle (256 * 512 MAC against 640 + 1024 / H bytes per token and head), in
// practice by the package power limit: MFMA and a stream of stores at once.
//
// A workgroup keeps ONE head's weights -- 256 output rows x 512, 256 KiB -- in registers (each of
// the four wavefronts 64 rows, 256 registers per lane: half of its register file) and walks a
// range of tokens, 32 at a time: only the latent rows travel, 1 KiB per token for 64 clocks of
// matrix work, and every block of 32 tokens leaves as soon as it is done, its conversion and
// stores between the MFMAs of the next one.  Every fragment read from LDS feeds two MFMAs (half of
// the LDS rate).  Both operands are k-contiguous in memory (rows of c_KV, rows of W), so either
// can be the MFMA row operand: the K wavefronts (0, 1) compute W c^T (lanes own tokens), the V
// wavefronts (2, 3) c W^T (lanes own d, 8 consecutive accumulators are one 16-byte V chunk).
// Latent rows stream global -> LDS (global_load_lds) through a ring of four 32-token tiles.
// Measured on MI355X against a tile of 256 tokens x 256 outputs per workgroup with the whole
// contraction streamed through LDS and an epilogue of its own: 32768 tokens x 128 heads 1573 ->
// 930 to 975 us (1.13 to 1.18 PFLOP/s with 2.8 TB/s of stores; 800 us without the stores, 690 us
// without any transfer), 4096 x 128 194 -> 122 us, 1003 x 16 20.0 -> 8.4 us.  Stores without the
// non-temporal hint: 1240 us.
#include <algorithm>
#include <type_traits>

#include "tmla_common.hpp"
#include "tmla_lds_asm.hpp"
#include "tmla_mfma.hpp"

namespace tmla {

constexpr int EX_ROW_BYTES = D_L * 2;                      // 1 KiB: one transfer
constexpr int EX_ROPE_OFF = TOK_BLK * EX_ROW_BYTES;        // 32 KiB of latent rows
constexpr int EX_TILE_BYTES = EX_ROPE_OFF + 4 * 1024;      // and the four rope fragments
constexpr int EX_RING = 4;
constexpr int EX_LDS_BYTES = EX_RING * EX_TILE_BYTES;      // 144 KiB
constexpr int EX_W_PIECE = 32 * 256;   // of the weights on their way to the registers
static_assert(4 * 3 * EX_W_PIECE <= 3 * EX_TILE_BYTES, "three pieces per wavefront beside the first tile");
constexpr int EX_DMA = 9;        // transfers of a wavefront per tile: 8 rows, 1 rope fragment
constexpr int EX_NKS = D_L / 16;                           // 32 k-steps of an MFMA
constexpr int EX_SYNC_KS = 22;   // k-step of a block behind which the next tile must have landed

struct ExpandArgs {
  const __bf16* c; int64_t c_stride;      // latent rows [ntok, 512] (element stride between rows)
  const __bf16* r; int64_t r_stride;      // rope rows   [ntok, 64]
  const __bf16* w_uk; const __bf16* w_uv; // [H, 128, 512]
  __bf16* k_out; __bf16* v_out;
  int64_t ntok, ntb;                      // tokens; blocks of 32 tokens
  int H, splits, units;                   // units = H * splits workgroups (twice that in halves)
};

// The weights sit in accumulation registers and the sums in vector registers, which only assembly
// pins down (left to the allocator, weights are copied from file to file in front of their use).
// The assembler does not see these MFMAs: their sums are read 4 MFMAs later at the earliest, or
// behind expand_drain(), and no vector-ALU instruction writes their operands.  WAIT: the fragment
// arrived (six younger requests may be in flight).
template <bool IS_V, bool FIRST, bool WAIT>
__device__ __forceinline__ void expand_mfma(f32x16& d, const bf16x8& c, const bf16x8& w) {
#define TMLA_EX_MFMA(PRE, SRC_C, D)                                                          \
  if constexpr (IS_V)                                                                        \
    asm volatile(PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, " SRC_C : D(d) : "v"(c), "a"(w)); \
  else                                                                                       \
    asm volatile(PRE "v_mfma_f32_32x32x16_bf16 %0, %2, %1, " SRC_C : D(d) : "v"(c), "a"(w));
  if constexpr (WAIT && FIRST) { TMLA_EX_MFMA("s_waitcnt lgkmcnt(6)\n\t", "0", "=&v") }
  else if constexpr (WAIT) { TMLA_EX_MFMA("s_waitcnt lgkmcnt(6)\n\t", "%0", "+v") }
  else if constexpr (FIRST) { TMLA_EX_MFMA("", "0", "=&v") }
  else { TMLA_EX_MFMA("", "%0", "+v") }
#undef TMLA_EX_MFMA
}
// enough idle issue slots for the last MFMA to have written its result
__device__ inline void expand_drain() {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
}

// One wavefront's part of the walk over blocks [b0, b1) of head h.  LDS tile: row r (token) at
// r * 1024, its 16-byte chunk c in slot c ^ (r & 15): the 16 rows a 16-byte read serves at a time
// fall on distinct banks.  Behind the rows, the rope part in fragment order, one fragment per
// wavefront.
// NI: 32-row blocks of the weights per wavefront -- two, or one where the workgroup has half of the
// head's rows (K or V) to itself.  ROPE: the workgroup writes the rope part as well.
template <bool IS_V, int NI, bool ROPE>
__device__ __forceinline__ void expand_walk(const ExpandArgs& a, char* smem, int h, int64_t b0,
                                            int64_t b1, int wave, int lane) {
  const int n = lane & 31, g = lane >> 5;
  const int rb0 = NI == 2 ? 2 * (wave & 1) : wave;   // first of the 32-row blocks of the 128 K or V rows
  constexpr int STORES = 2 * NI + ROPE;              // vector stores of a wavefront per finished block
  const int nblk = (int)(b1 - b0);

  // ---- transfers: wavefront w moves rows 8 w .. 8 w + 7 of a tile and rope fragment w; rows past
  // the last token repeat it (their results are replaced by zeros).  Row numbers inside the range
  // are 32-bit.
  const int last = (int)min((int64_t)0x7fffffff, a.ntok - 1 - b0 * TOK_BLK);
  const char* c_src = (const char*)(a.c + b0 * TOK_BLK * a.c_stride);
  const char* r_src = (const char*)(a.r + b0 * TOK_BLK * a.r_stride + 16 * wave + 8 * g);
  const int64_t c_bytes = a.c_stride * 2, r_bytes = a.r_stride * 2;
  auto issue = [&](int blk, int slot, auto part_) __attribute__((always_inline)) {
    constexpr int part = decltype(part_)::value;
    if constexpr (part < 8) {
      const int row = 8 * wave + part;
      dma16(c_src + min(blk * TOK_BLK + row, last) * c_bytes + ((lane ^ (row & 15)) << 4),
            smem + slot + row * EX_ROW_BYTES);
    } else {
      dma16(r_src + min(blk * TOK_BLK + n, last) * r_bytes, smem + slot + EX_ROPE_OFF + wave * 1024);
    }
  };

  // The first tile is requested in front of the weights.
  static_for<EX_DMA>([&](auto p_) { issue(0, 0, p_); });

  // ---- weights: fragment (i, ks) = rows 32 (rb0 + i) + n, k = 16 ks + 8 g .. + 7.  They come
  // through LDS in pieces of 32 rows x 128 columns, three of a wavefront's eight under way at a time
  // in the ring's other slots: row r of a piece at r * 256, its 16-byte chunk c in place c ^ (r & 15).
  // (32 whole rows at a time, each half waited for by itself and the first tiles behind them, they
  // held up 1003 tokens x 16 heads, K and V in one workgroup, by 1.3 us; read straight into the registers, 32
  // bytes of 32 rows per load, by another 4 us.)
  bf16x8 w[NI][EX_NKS];
  {
    constexpr int PIECES = 4 * NI, AHEAD = 3, DMAS = EX_W_PIECE / 1024;
    const char* wp = (const char*)((IS_V ? a.w_uv : a.w_uk) + ((size_t)h * 128 + 32 * rb0) * D_L);
    char* mine = smem + EX_TILE_BYTES + wave * (AHEAD * EX_W_PIECE);
    const uint32_t rd = lds_addr(mine) + n * 256, swz = (uint32_t)(g ^ (n & 15)) << 4;
    uint32_t off[4];   // rows 4 t .. 4 t + 3, 16 lanes each
#pragma unroll
    for (int t = 0; t < 4; t++)
      off[t] = (lane >> 4) * EX_ROW_BYTES + (((lane & 15) ^ (4 * t + (lane >> 4))) << 4);
    auto request = [&](auto p_) __attribute__((always_inline)) {
      constexpr int p = decltype(p_)::value, i = p >> 2, kq = p & 3;
#pragma unroll
      for (int t = 0; t < DMAS; t++)
        dma16(wp + (32 * i + 4 * t) * EX_ROW_BYTES + 256 * kq + off[t & 3],
              mine + (p % AHEAD) * EX_W_PIECE + t * 1024);
    };
    static_for<AHEAD>([&](auto p_) { request(p_); });
    static_for<PIECES>([&](auto p_) {
      constexpr int p = decltype(p_)::value, i = p >> 2, kq = p & 3;
      constexpr int behind = PIECES - 1 - p < AHEAD - 1 ? PIECES - 1 - p : AHEAD - 1;
      vm_wait<behind * DMAS>();
      static_for<8>([&](auto ks_) {
        constexpr int ks = decltype(ks_)::value;
        w[i][8 * kq + ks] = lds_read_b128<(p % AHEAD) * EX_W_PIECE>(rd + (swz ^ (ks << 5)));
      });
      static_for<2>([&](auto k_) {
        constexpr int k = 8 * kq + 4 * decltype(k_)::value;
        lgkm_wait<0>(w[i][k], w[i][k + 1], w[i][k + 2], w[i][k + 3]);
        asm volatile("" : "+a"(w[i][k]), "+a"(w[i][k + 1]), "+a"(w[i][k + 2]), "+a"(w[i][k + 3]));
      });
      if constexpr (p + AHEAD < PIECES) request(std::integral_constant<int, p + AHEAD>{});
    });
    raw_barrier();   // slots 1 to 3 are free, and the first tile is there
  }
  static_for<EX_RING - 2>([&](auto b_) {
    constexpr int b = decltype(b_)::value + 1;
    static_for<EX_DMA>([&](auto p_) { issue(b, b * EX_TILE_BYTES, p_); });
  });

  const uint32_t row_addr = lds_addr(smem) + n * EX_ROW_BYTES;
  const uint32_t rope_addr = lds_addr(smem) + wave * 1024 + lane * 16;
  const uint32_t sw = (uint32_t)(g ^ (n & 15)) << 4;   // chunk 2 ks + g: slot (2 ks) ^ (g ^ n)

  const int64_t blk_base = (int64_t)h * a.ntb + b0;
  __bf16* k_dst = a.k_out + blk_base * K_BLK_ELEMS + lane * 8;
  __bf16* v_dst = a.v_out + blk_base * V_BLK_ELEMS + lane * 8;

  f32x16 acc[2][NI];     // [parity of the block][32-row block of the weights]
  bf16x8 rope;           // this wavefront's rope fragment of the block at work
  bf16x8 fr[8];          // fragments on their way from LDS, six ahead

  // slots of the ring as byte offsets: that of the block at work, and k slots behind it
  int cur = 0;
  auto behind = [&](int k) __attribute__((always_inline)) {
    const int s = cur - k * EX_TILE_BYTES;
    return s < 0 ? s + EX_LDS_BYTES : s;
  };
  auto read_frag = [&](int slot, auto ks_) __attribute__((always_inline)) {
    constexpr int ks = decltype(ks_)::value;
    const uint32_t base = row_addr + slot;
    // chunk 2 ks + g: its low four bits are swizzled, the high two select 256 bytes
    fr[ks & 7] = lds_read_b128<256 * (ks >> 3)>(base + (sw ^ ((2 * ks & 15) << 4)));
  };
  // stores one of 2 NI pieces of this wavefront's part of the finished block blk
  auto store_piece = [&](int blk, auto par_, auto piece_, auto tail_) __attribute__((always_inline)) {
    constexpr int P = decltype(par_)::value, piece = decltype(piece_)::value;
    constexpr bool TAIL = decltype(tail_)::value;
    constexpr int i = piece >> 1, hp = piece & 1;
    f32x16& d = acc[P][i];
    asm volatile("" : "+v"(d));   // (no conversion is moved up to the MFMAs that form the sums)
    bf16x8 o;
    if constexpr (IS_V) {
      // rows = tokens 16 hp + 4 g + 8 (e / 4) + e % 4, column d = 32 (rb0 + i) + n
#pragma unroll
      for (int e = 0; e < 8; e++) o[e] = (__bf16)d[8 * hp + e];
      if constexpr (TAIL) {
        const int left = (int)(a.ntok - (b0 + blk) * TOK_BLK);
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (acc_row(8 * hp + e, g) >= left) o[e] = (__bf16)0.f;
      }
      __builtin_nontemporal_store(o, (bf16x8*)(v_dst + (int64_t)blk * V_BLK_ELEMS +
                                               ((hp * 4 + rb0 + i) * 64) * 8));
    } else {
      // column = token n, rows d = 32 (rb0 + i) + 16 hp + 8 x + 4 g + (0..3), x = 0, 1: the two
      // halves of the wavefront trade so that a lane holds eight consecutive d of its token
      typedef int int2v __attribute__((ext_vector_type(2)));
      typedef int int4v __attribute__((ext_vector_type(4)));
      bf16x4 lo, hi;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        lo[e] = (__bf16)d[8 * hp + e];
        hi[e] = (__bf16)d[8 * hp + 4 + e];
      }
      const int2v l2 = __builtin_bit_cast(int2v, lo), h2 = __builtin_bit_cast(int2v, hi);
      auto r0 = __builtin_amdgcn_permlane32_swap(l2[0], h2[0], false, false);
      auto r1 = __builtin_amdgcn_permlane32_swap(l2[1], h2[1], false, false);
      int4v w4 = {(int)r0[0], (int)r1[0], (int)r0[1], (int)r1[1]};
      if constexpr (TAIL)
        if ((b0 + blk) * TOK_BLK + n >= a.ntok) w4 = int4v{0, 0, 0, 0};
      o = __builtin_bit_cast(bf16x8, w4);
      __builtin_nontemporal_store(o, (bf16x8*)(k_dst + (int64_t)blk * K_BLK_ELEMS +
                                               ((2 * (rb0 + i) + hp) * 64) * 8));
    }
  };
  auto store_rope = [&](int blk) __attribute__((always_inline)) {
    const bf16x8 o = blk * TOK_BLK + n <= last ? rope : bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    __builtin_nontemporal_store(o, (bf16x8*)(k_dst + (int64_t)blk * K_BLK_ELEMS +
                                             (8 + wave) * 64 * 8));
  };

  // One block: 32 k-steps of two MFMAs; the block before it (FIRST: there is none) is converted
  // and stored in between.  No branches: past the last block of the range the requests for
  // fragments and tiles go on, over whatever the ring holds and the last token again.
  // Behind k-step EX_SYNC_KS: the next tile has landed for everyone, and everyone is done with
  // the tile of the block before this one, whose slot takes the transfers of block blk + 3.
  auto block = [&](int blk, auto par_, auto first_) __attribute__((always_inline)) {
    constexpr int P = decltype(par_)::value;
    constexpr bool FIRST = decltype(first_)::value;
    constexpr std::integral_constant<int, P ^ 1> Q{};
    const int next = behind(EX_RING - 1), slot2 = behind(2), slot3 = behind(1);
    static_for<EX_NKS>([&](auto ks_) {
      constexpr int ks = decltype(ks_)::value;
      // fragment ks + 6, of this block or the next one
      if constexpr (ks + 6 < EX_NKS) read_frag(cur, std::integral_constant<int, ks + 6>{});
      else read_frag(next, std::integral_constant<int, ks + 6 - EX_NKS>{});
      expand_mfma<IS_V, ks == 0, true>(acc[P][0], fr[ks & 7], w[0][ks]);
      if constexpr (NI == 2) expand_mfma<IS_V, ks == 0, false>(acc[P][1], fr[ks & 7], w[1][ks]);
      if constexpr (!FIRST && NI == 2 && ks >= 2 && ks < 18 && (ks - 2) % 4 == 0)
        store_piece(blk - 1, Q, std::integral_constant<int, (ks - 2) / 4>{}, std::false_type{});
      if constexpr (!FIRST && NI == 1 && (ks == 6 || ks == 12))
        store_piece(blk - 1, Q, std::integral_constant<int, ks / 6 - 1>{}, std::false_type{});
      // the rope fragment: requested behind k-step 4, there behind k-step 16 (the eleven younger
      // requests of then are six)
      if constexpr (ROPE && ks == 4) rope = lds_read_b128<EX_ROPE_OFF>(rope_addr + cur);
      if constexpr (ROPE && ks == 16) {
        lgkm_wait<6>(rope);
        store_rope(blk);
      }
      if constexpr (ks == EX_SYNC_KS) {
        // The transfers of block blk + 1 have landed.  Younger and possibly in flight: the nine of
        // block blk + 2 and this block's stores (of the first block: the rope fragment's).
        vm_wait<EX_DMA + (FIRST ? (int)ROPE : STORES)>();
        raw_barrier();
      }
      // transfers: two of block blk + 3 behind the barrier, the other seven in the next block
      if constexpr (ks >= 24 && ks % 4 == 0)
        issue(blk + 3, slot3, std::integral_constant<int, (ks - 24) / 4>{});
      if constexpr (!FIRST && ks < EX_SYNC_KS - 1 && ks % 3 == 0)
        issue(blk + 2, slot2, std::integral_constant<int, 2 + ks / 3>{});
    });
    cur = next;
  };

  constexpr std::integral_constant<int, 0> P0{};
  constexpr std::integral_constant<int, 1> P1{};
  static_for<6>([&](auto ks_) { read_frag(0, ks_); });
  block(0, P0, std::true_type{});
  int blk = 1;
  for (; blk + 1 < nblk; blk += 2) {
    block(blk, P1, std::false_type{});
    block(blk + 1, P0, std::false_type{});
  }
  // (the fragment requests that ran past the last block: their registers stay taken until the
  // data is there)
  auto settle = [&]() __attribute__((always_inline)) {
    lgkm_wait<0>(fr[0], fr[1], fr[2], fr[3]);
    lgkm_wait<0>(fr[4], fr[5]);
    expand_drain();
  };
  auto finish = [&](auto par_, auto tail_) __attribute__((always_inline)) {
    static_for<2 * NI>([&](auto p_) { store_piece(nblk - 1, par_, p_, tail_); });
  };
  const bool tail = b1 * TOK_BLK > a.ntok;
  if (blk < nblk) {
    block(blk, P1, std::false_type{});
    settle();
    if (tail) finish(P1, std::true_type{});
    else finish(P1, std::false_type{});
  } else {
    settle();
    if (tail) finish(P0, std::true_type{});
    else finish(P0, std::false_type{});
  }
  vm_wait<0>();   // no transfer may land in LDS that another workgroup owns by then
}

template <bool HALVES>
__global__ void __launch_bounds__(256, 1) expand_gemm_kernel(ExpandArgs a) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // consecutive workgroup ids go round-robin over the 8 XCDs: an XCD gets consecutive units, i.e.
  // the token ranges of few heads, whose weights then come into one L2 only
  const int per = (a.units + 7) / 8;
  const int unit = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (unit >= a.units) return;
  const int item = HALVES ? unit >> 1 : unit;
  const int split = item % a.splits, h = item / a.splits;
  const int64_t b0 = a.ntb * split / a.splits, b1 = a.ntb * (split + 1) / a.splits;
  if (b0 >= b1) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if constexpr (HALVES) {
    if (unit & 1) expand_walk<true, 1, false>(a, smem, h, b0, b1, wave, lane);
    else expand_walk<false, 1, true>(a, smem, h, b0, b1, wave, lane);
  } else {
    if (wave < 2) expand_walk<false, 2, true>(a, smem, h, b0, b1, wave, lane);
    else expand_walk<true, 2, true>(a, smem, h, b0, b1, wave, lane);
  }
}

// Token ranges per head.  One workgroup fits per compute unit, so H * splits workgroups take
// ceil(H splits / 256) turns of a start-up (launch and weights: 6 us; EX_START blocks of
// 1.85 us) and ceil(blocks / splits) blocks each.  For every number of turns the most ranges that
// fit are taken; the cheapest number wins.
constexpr int EX_START = 4, EX_MAX_TURNS = 8;
static int expand_splits(int H, int64_t ntb) {
  int64_t best = -1;
  int best_s = 1;
  for (int turns = 1; turns <= EX_MAX_TURNS; turns++) {
    const int s = (int)std::max<int64_t>(1, std::min<int64_t>(ntb, turns * NUM_CU / H));
    const int64_t taken = ((int64_t)H * s + NUM_CU - 1) / NUM_CU;
    const int64_t cost = taken * ((ntb + s - 1) / s + EX_START);
    if (best < 0 || cost < best) { best = cost; best_s = s; }
  }
  return best_s;
}
// K and V of a head by workgroups of their own: half of the weights to fetch, twice the blocks, and each
// of them bound by LDS (a fragment feeds one MFMA) rather than by the matrix cores.  Where all ranges run at
// once, a workgroup takes 6.0 us + 1.75 per block with both and 5.2 + 1.0 with one of them (16 to
// 64 heads, one to eight blocks, within 4 %, launch included): back to back, 200 tokens x 16 heads 6.7 /
// 5.5 us, 600 x 32 10.3 / 9.2, 1003 x 16 8.4 / 8.0, 1003 x 32 11.4 / 11.4, 434 x 64 10.5 / 10.0, 700 x 64 14.0 /
// 15.0, 434 x 128 18.0 / 20.0.
static bool expand_in_halves(int H, int64_t ntb, int splits) {
  if (2 * H > NUM_CU || H * splits > NUM_CU) return false;
  const int64_t s = std::min<int64_t>(ntb, NUM_CU / (2 * H));
  return 5.2 + 1.0 * ((ntb + s - 1) / s) < 6.0 + 1.75 * ((ntb + splits - 1) / splits);
}

int mfma_expand(int H, int64_t ntok, const void* c, int64_t c_stride, const void* r,
                int64_t r_stride, const void* w_uk, const void* w_uv, void* k_out, void* v_out,
                hipStream_t stream) {
  if (ntok <= 0) return TMLA_OK;
  ExpandArgs a;
  a.c = (const __bf16*)c; a.c_stride = c_stride; a.r = (const __bf16*)r; a.r_stride = r_stride;
  a.w_uk = (const __bf16*)w_uk; a.w_uv = (const __bf16*)w_uv;
  a.k_out = (__bf16*)k_out; a.v_out = (__bf16*)v_out;
  a.ntok = ntok; a.ntb = (ntok + TOK_BLK - 1) / TOK_BLK; a.H = H;
  a.splits = expand_splits(H, a.ntb);
  const bool halves = expand_in_halves(H, a.ntb, a.splits);
  if (halves) a.splits = (int)std::min<int64_t>(a.ntb, NUM_CU / (2 * H));
  if ((int64_t)a.splits * H > 0x7ffffff0) return TMLA_ERR_UNSUPPORTED;
  a.units = a.splits * H * (halves ? 2 : 1);
  static LdsOptIn lds[2];
  auto kernel = halves ? expand_gemm_kernel<true> : expand_gemm_kernel<false>;
  if (lds[halves].ensure((const void*)kernel, EX_LDS_BYTES) != hipSuccess) return TMLA_ERR_HIP;
  hipLaunchKernelGGL(kernel, dim3((unsigned)((a.units + 7) / 8 * 8)), dim3(256), EX_LDS_BYTES, stream, a);
  return TMLA_OK;
}

}  // namespace tmla
