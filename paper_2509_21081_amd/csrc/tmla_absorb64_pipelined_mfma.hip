// Absorb-formulation flash-decode over latent cache rows (paper Algorithm 1 step 6), 64 query rows
// per workgroup, 32 tokens per period: the suffixes of requests with more than 32 query rows
// (S_q * H > 32), the latent prefix for groups of 64 rows cut from all requests, and on small
// grids both in one launch, whatever the rows per request.  (What the 64-token-step kernel of
// tmla_absorb64_mfma.hip keeps: keeps_steps() below.)
//
// The two matrix products of a tile of 32 tokens want different work splits, so the four wavefronts hand
// the probabilities over through LDS:
//   scores   S^T = C Q_abs^T : wavefront (qb, th) takes query block qb (32 rows) and 16 of the tokens, as two
//            16 x 16 x 32 products a k-step of 32 columns, so that every fragment read from LDS feeds two MFMAs:
//            36 of them, every score computed exactly once;
//   outputs  O^T += C_N^T P^T: wavefront w takes latent columns [128 w, 128 w + 128) for all 64
//            queries, so each transposed cache fragment feeds two MFMAs (one per query block): 16 of them.
// One barrier a period: period t runs the scores of tile t + 1 and the outputs of tile t, with the exponentials
// of tile t + 1 among the latter's MFMAs, while tiles t + 2 and t + 3 are on their way (four tiles fill the
// LDS).  A lone wavefront issues one instruction in about five cycles whatever its kind, so LDS reads and
// transfers are dealt out between the MFMAs, and so are the exponentials as far as the compiler follows: in the
// period that requests a tile, the branches around that tile's address end a basic block behind the third pair of
// output MFMAs, and the first four exponentials with their arithmetic, some twenty vector instructions, run behind
// them without an MFMA; in the last periods of a walk they are dealt out as written.  The probes behind this order
// (cycles a period without / with barrier): reads of a pair in front of its MFMAs 1473 / 1646, between them
// 1353 / 1494.  In the kernel a period takes about 1850 cycles for 1088 of matrix time (0.81 us); the kernel that
// walked 64 tokens a step, products and exponentials one behind the other with three barriers, took 1.04 us
// per 32 tokens.  Neither the transfers' arrival nor the barrier is waited for (8 and 40 cycles): issue
// bounds it.  Pass alone, before -> after: 37 requests x 3 x 64 heads, 1 to 1500 ragged tokens 34.1 -> 29.4 us, 128
// heads x 16384 + 512 tokens 15.2 -> 14.3 us; steps of 11 x 64 heads absorb form over 24326 + 184 tokens 62.5 -> 54.3,
// 259 x 3 x 48 heads mixed over 416 + 1197 259 -> 225 us.
//
// Exponent references are fixed for a whole walk over the chunk (the result does not depend on the
// reference, only the float range does: scores about 2^7 log2-units above it overflow): the first walk takes
// the maxima of tile 0; if a denominator ends up outside a moderate finite range, the exact maxima are formed
// in a scores-only pass and the chunk is walked again with those.
#include "tmla_absorb_tile.hpp"

namespace tmla {

constexpr int A64P_P_OFF = AB_NSLOT * AB_TILE_BYTES;       // probabilities of two tiles, 4 KiB each
constexpr int A64P_LDS_BYTES = A64P_P_OFF + 2 * 4096;       // 163840 = all of LDS
static_assert(AB_NSLOT == 4 && A64P_LDS_BYTES <= 163840, "LDS layout");

struct Absorb64PipelinedArgs {
  AbsorbArgs a;
  AbsorbGrid grid;
  int exact_only;    // debug: skip the walk with the first tile's references
};

// The MFMAs of the walk are written in assembly so that they and the LDS reads stay in the order in
// which they are laid out, and to fix where their operands live (outputs and most of the resident
// query fragments in accumulation registers).  The assembler does not see that these statements are
// MFMAs: a vector-ALU read of a result is two output MFMAs away or behind a64p_drain().
// N: behind a wait until at most N LDS reads are in flight (one statement, so that nothing is put between).
// ACC: the query fragment is in an accumulation register, else in a vector register.
template <int N, bool ACC>
__device__ inline void a64p_mfma_s_first(f32x4& d, const bf16x8& a, const bf16x8& b) {
  static_assert(ACC, "k-step 0");
  asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b), "n"(N));
}
template <int N, bool ACC>
__device__ inline void a64p_mfma_s_w(f32x4& d, const bf16x8& a, const bf16x8& b) {
  if constexpr (ACC)
    asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b), "n"(N));
  else
    asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b), "n"(N));
}
template <bool ACC>
__device__ inline void a64p_mfma_s(f32x4& d, const bf16x8& a, const bf16x8& b) {
  if constexpr (ACC) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
template <int N>
__device__ inline void a64p_mfma_o_w(f32x16& d, const bf16x8& a, const bf16x8& b) {
  asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b), "n"(N));
}
__device__ inline void a64p_mfma_o(f32x16& d, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
// The same with one global -> LDS transfer behind it (M0 is set in front of the MFMA, which fills the
// wait state that the hardware wants between a write of M0 and its use).  `lds` + IMM: wave-uniform
// LDS address, `base`: wave-uniform, `off`: per lane.
template <bool ACC, bool STREAM, int IMM>
__device__ inline void a64p_mfma_s_dma(f32x4& d, const bf16x8& a, const bf16x8& b, uint32_t off,
                                      const char* base, uint32_t lds) {
  uint32_t m0;
#define A64P_S_DMA(B, POLICY)                                                                      \
  asm volatile("s_add_u32 %1, %6, %7\n\tv_mfma_f32_16x16x32_bf16 %0, %2, %3, %0\n\t"              \
               "global_load_lds_dwordx4 %4, %5" POLICY                                            \
               : "+v"(d), "=&{m0}"(m0)                                                            \
               : "v"(a), B(b), "v"(off), "s"(base), "s"(lds), "n"(IMM) : "memory", "scc")
  if constexpr (ACC && STREAM) A64P_S_DMA("a", TMLA_STREAM_POLICY);
  else if constexpr (ACC) A64P_S_DMA("a", "");
  else if constexpr (STREAM) A64P_S_DMA("v", TMLA_STREAM_POLICY);
  else A64P_S_DMA("v", "");
#undef A64P_S_DMA
}
// enough idle issue slots for the last MFMA to have written its result
__device__ inline void a64p_drain() {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
}
template <int OFF>
__device__ inline bf16x8 a64p_read_acc(uint32_t addr) {   // into accumulation registers
  bf16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=a"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
// (values that MFMAs in assembly have left: nothing that reads them is moved in front of this)
__device__ inline void a64p_tie(f32x4& x, f32x4& y) { asm volatile("" : "+v"(x), "+v"(y)); }
__device__ inline void a64p_write_b64(uint32_t addr, bf16x4 v) {
  asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
// max / sum over the four lanes n, n + 16, n + 32, n + 48
__device__ inline float a64p_max_quads(float x) {
  const int xi = __float_as_int(x);
  auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  return max_halves(fmaxf(__int_as_float(r[0]), __int_as_float(r[1])));
}
__device__ inline float a64p_sum_quads(float x) {
  const int xi = __float_as_int(x);
  auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  return sum_halves(__int_as_float(r[0]) + __int_as_float(r[1]));
}
#define A64P_SB() __builtin_amdgcn_sched_barrier(0)

// HAS_PREFIX: the launch has work items over the shared latent prefix (absorb_only mode).  Those
// rows are read by every request and must stay cached, and a per-transfer choice of the cache
// policy is a branch in the hot loop (-13 % at 64 heads), so such a launch uses ordinary
// transfers throughout; a launch over suffix rows alone streams them with the non-temporal hint.
template <bool HAS_PREFIX>
__global__ void __launch_bounds__(256, 1) absorb64_pipelined_kernel(Absorb64PipelinedArgs args) {
  constexpr bool STREAM = !HAS_PREFIX;
  const AbsorbArgs& a = args.a;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const AbsorbUnit unit = absorb_unit<HAS_PREFIX>(a, args.grid, blockIdx.x);
  if (unit.none) return;
  const int item = unit.item, qg = unit.qg, b = unit.b, R = unit.R;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, g = lane >> 5;
  const int n16 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb = wave & 1, th = wave >> 1;

  // ---- which tokens
  int t0, t1;
  const bool is_prefix = HAS_PREFIX && unit.is_prefix;
  int len = 0, first_blk = 0, bt_cache = 0;
  const int32_t* bt = a.block_table + (size_t)b * a.max_blocks;
  if (is_prefix) {
    t0 = item * a.ap_chunk;
    t1 = min(a.Ls, t0 + a.ap_chunk);
  } else {
    t0 = (item - a.ap_chunks) * a.as_chunk;
    // (the chunk's block-table entries are requested beside the request's length)
    first_blk = t0 >> a.bs_shift;
    bt_cache = (lane < a.as_chunk >> a.bs_shift && first_blk + lane < a.max_blocks) ? bt[first_blk + lane] : 0;
    len = scalar_load_i32(a.lens + b);
    t1 = min(len, t0 + a.as_chunk);
  }
  // lane (n16, q4) of wavefront (qb, th) scores query rows r_own[0], r_own[1]
  const int r_own[2] = {(qg * 2 + qb) * 32 + n16, (qg * 2 + qb) * 32 + 16 + n16};
  if (t1 <= t0) {   // empty chunk (workgroup-uniform): only the LSEs are defined
#pragma unroll
    for (int s = 0; s < 2; s++)
      if (th == 0 && q4 == 0 && r_own[s] < R)
        a.lat_lse[(size_t)item * a.rows + (int64_t)b * R + r_own[s]] = -INFINITY;
    return;
  }
  const int ntile = (t1 - t0 + 31) / 32;
  // tokens of the chunk that this lane's queries see, and those that every query sees
  int vis[2] = {t1 - t0, t1 - t0}, vis_all = t1 - t0;
  if (!is_prefix) {
#pragma unroll
    for (int s = 0; s < 2; s++)
      vis[s] = min(t1, max(0, min(len, len - a.Sq + query_position(r_own[s], a.H, R) + 1))) - t0;
    vis_all = min(t1, len - a.Sq + 1) - t0;
  }

  // ---- tile streaming: global -> LDS (see tmla_absorb_tile.hpp)
  // Rows in slots c ^ f((row >> 2) & 3) with f = 0, 3, 2, 1: a 16-byte read is served sixteen lanes at a time, 0 .. 3, 12 ..
  // 15, 20 .. 27 first, i.e. rows 0 .. 3 and 12 .. 15 of one chunk and 4 .. 11 of the next (8.2 cycles a read with f = 0, 1,
  // 2, 3, 4.4 with this one).
  DmaLane dl = dma_lane(wave, lane);
  dl.off[1] = (lane ^ 3) << 4;
  dl.off[3] = (lane ^ 1) << 4;
  // The absorbed queries, staged like cache tiles in slots 2 and 3; the block-table entries are on
  // their way meanwhile.
  {
    const int64_t req_row0 = (int64_t)b * R;
#pragma unroll
    for (int j = 0; j < 2; j++) {
      const int blk_row0 = (qg * 2 + j) * 32;
      RowSrc qs;
      qs.stream = false;
      qs.last = min(31, R - 1 - blk_row0);
      int64_t first = req_row0 + blk_row0;
      if (qs.last < 0) {   // block entirely past the request's rows: any valid row will do
        qs.last = 0;
        first = req_row0 + R - 1;
      }
      qs.lat = (const char*)(a.qabs + first * D_ROW);
      qs.rope = qs.lat + D_L * 2;
      qs.lat_stride = qs.rope_stride = D_ROW * 2;
      issue_all(qs, smem + (2 + j) * AB_TILE_BYTES, dl);
    }
  }
  asm volatile("" : "+v"(bt_cache));   // (the compiler waits for the entries alone)
  const int bs_shift = a.bs_shift;
  const int lat_stride = is_prefix ? D_L * 2 : D_ROW * 2, rope_stride = is_prefix ? D_R * 2 : D_ROW * 2;
  // Where tile `tile` (32 tokens) of the chunk comes from; a cache block holds a multiple of 32 tokens.
  auto tile_src = [&](int tile, const char*& lat, const char*& rope) __attribute__((always_inline)) {
    const int tok0 = t0 + tile * 32;
    if (is_prefix) {
      lat = (const char*)a.pc + (size_t)tok0 * (D_L * 2);
      rope = (const char*)a.pr + (size_t)tok0 * (D_R * 2);
    } else {
      const int bi = __builtin_amdgcn_readfirstlane((tok0 >> bs_shift) - first_blk);
      const int blk = bi < 64 ? __builtin_amdgcn_readlane(bt_cache, bi)
                              : scalar_load_i32(bt + first_blk + bi);
      lat = (const char*)(a.pool + (((size_t)blk << bs_shift) + (tok0 & ((1 << bs_shift) - 1))) * D_ROW);
      rope = lat + D_L * 2;
    }
  };
  // This lane's offsets of the nine transfers of its wavefront; rows behind the chunk's last one repeat it
  // (only the last tile has any).
  uint32_t doff[AB_DMA_PER_WAVE];
  auto set_doff = [&](int last) __attribute__((always_inline)) {
#pragma unroll
    for (int K = 0; K < 8; K++) doff[K] = min(wave + 4 * K, last) * lat_stride + dl.off[K & 3];
    doff[8] = min(dl.rope_row, last) * rope_stride + dl.rope_ch;
  };
  const int last_row = t1 - t0 - 1 - (ntile - 1) * 32;   // of the last tile
  const uint32_t smem_base = lds_addr(smem);
  auto slot_of = [&](int tile) __attribute__((always_inline)) { return smem_base + (tile & 3) * AB_TILE_BYTES; };
  auto issue_tile = [&](int tile, uint32_t dst) __attribute__((always_inline)) {
    const char *lat, *rope;
    tile_src(tile, lat, rope);
    if (tile == ntile - 1) set_doff(last_row);
    static_for<8>([&](auto k) {
      constexpr int K = decltype(k)::value;
      dma16_scalar_base<STREAM>(doff[K], lat, dst, (wave + 4 * K) * AB_ROW_BYTES);
    });
    dma16_scalar_base<STREAM>(doff[8], rope, dst, AB_MAIN_BYTES + wave * 1024);
  };

  // ---- per-lane LDS byte offsets inside a tile (layout in tmla_absorb_tile.hpp)
  //   score product, k-step ks < 16 of 32 latent columns: row 16 th + n16, chunk 4 ks + q4 -> k_off + 64 ks
  //                  rope k-step k: chunk 4 k + q4 -> r_off ^ (k << 6)
  const int swz = -(n16 >> 2) & 3;
  const uint32_t k_off = (16 * th + n16) * AB_ROW_BYTES + ((q4 ^ swz) << 4);
  const uint32_t r_off = AB_MAIN_BYTES + (16 * th + n16) * 128 + ((q4 ^ ((n16 >> 1) & 7)) << 4);
  //   output product (transposing 8-byte reads; 16-lane group j = lane / 16, r = lane % 16): tokens
  //   16 ks + 8 g + r / 4 (v_lo) and four rows down (v_hi), latent columns 128 wave + 32 mb + 16 (j % 2) +
  //   4 (r % 4) .. + 3 -> + 16 ks rows + 64 mb
  const int vchunk = 2 * (q4 & 1) + ((n16 & 3) >> 1);
  const uint32_t v_lo = (8 * g + (n16 >> 2)) * AB_ROW_BYTES + 8 * (n16 & 1) + ((vchunk ^ (2 * g)) << 4) + 256 * wave;
  const uint32_t v_hi = (8 * g + 4 + (n16 >> 2)) * AB_ROW_BYTES + 8 * (n16 & 1) + ((vchunk ^ (3 - 2 * g)) << 4) + 256 * wave;
  //   probabilities [tile & 1][query block][16-token half][lane of the reader]: 16 B = 8 tokens of a query
  const uint32_t p_wr = smem_base + A64P_P_OFF + (qb * 2 + th) * 1024 + (q4 >> 1) * 512 + n16 * 16 + (q4 & 1) * 8;
  const uint32_t p_rd = smem_base + A64P_P_OFF + lane * 16;
  // maxima, later denominators: [token half][query], in the probabilities' second buffer
  const uint32_t x_wr = smem_base + A64P_P_OFF + 4096 + (th * 64 + qb * 32 + n16) * 4;

  set_doff(31);
  issue_tile(0, slot_of(0));
  if (ntile > 1) issue_tile(1, slot_of(1));
  f32x16 o[4][2];      // [latent block of the own quarter][query block]
  auto clear_o = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < 4; mb++)
#pragma unroll
      for (int q = 0; q < 2; q++)
#pragma unroll
        for (int v = 0; v < 16; v++) o[mb][q][v] = 0.f;
#pragma unroll
    for (int mb = 0; mb < 4; mb++) asm volatile("" : "+a"(o[mb][0]), "+a"(o[mb][1]));
  };
  clear_o();           // (while the queries are on their way)
  if (ntile > 1) vm_wait<18>();
  else vm_wait<9>();
  raw_barrier();
  // ---- query fragments of the own query block (B operand of the score product): k-step ks of 32, rows n16
  // and 16 + n16 of the block
  constexpr int QA = 14;          // k-steps whose fragments are in accumulation registers
  bf16x8 qa[QA][2], qv[18 - QA][2];
  {
    const uint32_t base = smem_base + (2 + qb) * AB_TILE_BYTES;
    static_for<18>([&](auto ks_) {
      constexpr int ks = decltype(ks_)::value;
      static_for<2>([&](auto s_) {
        constexpr int s = decltype(s_)::value;
        const uint32_t row = 16 * s + n16;
        const uint32_t lat = base + row * AB_ROW_BYTES + ((q4 ^ swz) << 4);
        const uint32_t rope = base + AB_MAIN_BYTES + row * 128 + ((q4 ^ ((n16 >> 1) & 7)) << 4);
        if constexpr (ks < QA) qa[ks < QA ? ks : 0][s] = a64p_read_acc<64 * (ks & 15)>(lat);
        else if constexpr (ks < 16) qv[ks >= QA ? ks - QA : 0][s] = lds_read_b128<64 * (ks & 15)>(lat);
        else qv[ks >= QA ? ks - QA : 0][s] = lds_read_b128<0>(rope ^ ((ks - 16) << 6));
      });
    });
#pragma unroll
    for (int ks = 0; ks < QA; ks += 2)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+a"(qa[ks][0]), "+a"(qa[ks][1]), "+a"(qa[ks + 1][0]), "+a"(qa[ks + 1][1])::"memory");
#pragma unroll
    for (int ks = 0; ks < 18 - QA; ks += 2) lgkm_wait<0>(qv[ks][0], qv[ks][1], qv[ks + 1][0], qv[ks + 1][1]);
  }

  f32x4 sacc[2];              // scores of 16 tokens: [query half of the block]
  bf16x8 fr[8];               // ring of score fragments
  // requests fragment i of the tile whose lane addresses are ka, ra
  auto rd_k = [&](auto i_, uint32_t ka, uint32_t ra) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value;
    if constexpr (i < 16) fr[i % 8] = lds_read_b128<64 * (i & 15)>(ka);
    else fr[i % 8] = lds_read_b128<0>(ra ^ ((i - 16) << 6));
  };
  // the MFMA of k-step i for the first query half, behind a wait for its fragment, and that for the second
  auto mfma_k0 = [&](auto i_, auto later_) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value, N = decltype(later_)::value;
    if constexpr (i == 0) a64p_mfma_s_first<N, true>(sacc[0], fr[0], qa[0][0]);
    else if constexpr (i < QA) a64p_mfma_s_w<N, true>(sacc[0], fr[i % 8], qa[i < QA ? i : 0][0]);
    else a64p_mfma_s_w<N, false>(sacc[0], fr[i % 8], qv[i >= QA ? i - QA : 0][0]);
  };
  auto mfma_k1 = [&](auto i_) __attribute__((always_inline)) {
    constexpr int i = decltype(i_)::value;
    if constexpr (i == 0) a64p_mfma_s_first<15, true>(sacc[1], fr[0], qa[0][1]);
    else if constexpr (i < QA) a64p_mfma_s<true>(sacc[1], fr[i % 8], qa[i < QA ? i : 0][1]);
    else a64p_mfma_s<false>(sacc[1], fr[i % 8], qv[i >= QA ? i - QA : 0][1]);
  };
  constexpr int AHEAD = 6;    // score fragments requested ahead of their use
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  // The scores of the tile behind ka, ra, its first AHEAD fragments requested already.  OUT: the first twelve
  // reads of the output product behind it, `rd_out(j)`, are requested in the last k-steps.  PF: this
  // wavefront's nine transfers of a tile from lat, rope to LDS address `dst`, one behind every second k-step.
  // (A 16 x 16 MFMA leaves room for two or three other instructions, so they are dealt out between all of
  // them: with the reads in front of each pair of MFMAs 691 cycles, one between the two 648.)
  auto score_steps = [&](uint32_t ka, uint32_t ra, auto out_tag, auto prefetch_tag, const char* lat, const char* rope,
                         uint32_t dst, auto&& rd_out) __attribute__((always_inline)) {
    constexpr bool OUT = decltype(out_tag)::value, PF = decltype(prefetch_tag)::value;
    static_for<18>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      // requests behind that of fragment i
      constexpr int behind = (i + AHEAD - 1 < 17 ? AHEAD - 1 : 17 - i) + (OUT && i > 18 - AHEAD ? 2 * (i - 18 + AHEAD) : 0);
      mfma_k0(i_, std::integral_constant<int, behind>{});
      if constexpr (i + AHEAD < 18) rd_k(std::integral_constant<int, i + AHEAD>{}, ka, ra);
      else if constexpr (OUT) rd_out(std::integral_constant<int, 2 * (i + AHEAD - 18)>{});
      if constexpr (PF && i % 2 == 1) {
        constexpr int K = i / 2;
        const bf16x8& qf = i < QA ? qa[i < QA ? i : 0][1] : qv[i >= QA ? i - QA : 0][1];
        if constexpr (K < 8)
          a64p_mfma_s_dma<(i < QA), STREAM, 4 * K * AB_ROW_BYTES>(sacc[1], fr[i % 8], qf, doff[K], lat, dst + wave * AB_ROW_BYTES);
        else
          a64p_mfma_s_dma<(i < QA), STREAM, AB_MAIN_BYTES>(sacc[1], fr[i % 8], qf, doff[8], rope, dst + wave * 1024);
      } else {
        mfma_k1(i_);
      }
      if constexpr (OUT && i + AHEAD >= 18) rd_out(std::integral_constant<int, 2 * (i + AHEAD - 18) + 1>{});
    });
  };
  // the scores of a tile by themselves (first tile of a walk, maxima); PF: with the transfers of tile `next`
  auto scores = [&](uint32_t tb, auto prefetch_tag, int next) __attribute__((always_inline)) {
    const uint32_t ka = tb + k_off, ra = tb + r_off;
    const char *lat = nullptr, *rope = nullptr;
    if constexpr (decltype(prefetch_tag)::value) {
      tile_src(next, lat, rope);
      if (next == ntile - 1 && last_row < 31) set_doff(last_row);
    }
    static_for<AHEAD>([&](auto i) { rd_k(i, ka, ra); });
    score_steps(ka, ra, std::false_type{}, prefetch_tag, lat, rope, slot_of(next), [](auto) {});
    a64p_drain();
    a64p_tie(sacc[0], sacc[1]);
  };
  // scores of tokens this lane's queries must not see -> -inf (element v: token 16 th + 4 q4 + v)
  auto mask = [&](int tile) __attribute__((always_inline)) {
    if ((tile + 1) * 32 > vis_all) {
#pragma unroll
      for (int s = 0; s < 2; s++) {
        const int lim = vis[s] - (tile * 32 + 16 * th + 4 * q4);
#pragma unroll
        for (int v = 0; v < 4; v++)
          if (v >= lim) sacc[s][v] = -INFINITY;
      }
    }
  };
  float m[2], mu[2];   // exponent references of the two queries (log2 units); 0 in place of -inf
  float l[2];          // denominators: own 16-token halves, own 4 tokens of each
  auto prob = [&](int s, int v) __attribute__((always_inline)) {
    return fast_exp2(__builtin_fmaf(sacc[s][v], a.c, -mu[s]));
  };
  // maxima of the two queries over both token halves
  auto exchange_max = [&](float (&mx)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; s++) {
      mx[s] = a64p_max_quads(mx[s]);
      if (q4 == 0) lds_write_b32(x_wr + 64 * s, mx[s]);
    }
    lgkm_wait<0>();
    raw_barrier();
    float other[2] = {lds_read_f32(x_wr ^ 256), lds_read_f32((x_wr ^ 256) + 64)};
    lgkm_wait<0>(other[0], other[1]);
    mx[0] = fmaxf(mx[0], other[0]);
    mx[1] = fmaxf(mx[1], other[1]);
  };

  // A walk over the chunk.  References: in the first attempt the maxima of tile 0, in the second the exact
  // maxima of the chunk.  One copy of the code for both and one epilogue behind the loop.
  float den[2];        // denominators of column n in either query block
  float own[2];        // and of the two queries whose references this lane holds
  const bool exact_first = args.exact_only != 0;
  for (int attempt = exact_first ? 1 : 0;; attempt++) {
    const bool exact = attempt == 1;
    if (exact) {
      // (every transfer has landed and nobody reads the tiles any more)
      float mx[2] = {-INFINITY, -INFINITY};
      vm_wait<0>();
      for (int tile = 0; tile < ntile; tile++) {
        raw_barrier();
        set_doff(31);
        issue_tile(tile, smem_base);
        vm_wait<0>();
        raw_barrier();
        scores(smem_base, std::false_type{}, 0);
        mask(tile);
#pragma unroll
        for (int s = 0; s < 2; s++)
#pragma unroll
          for (int v = 0; v < 4; v++) mx[s] = fmaxf(mx[s], sacc[s][v]);
      }
      raw_barrier();
      exchange_max(mx);
      m[0] = mx[0] * a.c;
      m[1] = mx[1] * a.c;
      raw_barrier();
      set_doff(31);
      issue_tile(0, slot_of(0));
      if (ntile > 1) issue_tile(1, slot_of(1));
      clear_o();
    }
    if (ntile > 1) vm_wait<9>();
    else vm_wait<0>();
    raw_barrier();   // tile 0 has landed for everybody; everybody has its query fragments
    if (ntile > 2) scores(slot_of(0), std::true_type{}, 2);
    else scores(slot_of(0), std::false_type{}, 0);
    mask(0);
    if (!exact) {
      float mx[2];
#pragma unroll
      for (int s = 0; s < 2; s++) mx[s] = fmaxf(fmaxf(sacc[s][0], sacc[s][1]), fmaxf(sacc[s][2], sacc[s][3]));
      exchange_max(mx);
      m[0] = mx[0] * a.c;
      m[1] = mx[1] * a.c;
    }
#pragma unroll
    for (int s = 0; s < 2; s++) {
      mu[s] = m[s] == -INFINITY ? 0.f : m[s];
      bf16x4 p;
      l[s] = 0.f;
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const float x = prob(s, v);
        l[s] += x;
        p[v] = (__bf16)x;
      }
      a64p_write_b64(p_wr + 256 * s, p);
    }
    lgkm_wait<0>();
    if (ntile > 2) vm_wait<9>();
    else vm_wait<0>();
    raw_barrier();   // tile 1 and the probabilities of tile 0

    // Period t: the scores of tile t + 1, then the outputs of tile t with the exponentials of t + 1 between
    // their MFMAs.  The last two of the eight pairs of output MFMAs run behind the barrier at the end, on
    // registers alone, while the first fragments of the next scores are on their way.
    short4v vl[8], vh[8];     // transposed cache fragments of pair p = 2 mb + ks, lower and upper half
    bf16x8 pf[2][2];          // probability fragments [ks][query block]
#pragma unroll
    for (int p = 6; p < 8; p++) vl[p] = vh[p] = short4v{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 2; ks++) pf[ks][0] = pf[ks][1] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
      asm volatile("" : "+v"(pf[ks][0]), "+v"(pf[ks][1]), "+v"(vl[6 + ks]), "+v"(vh[6 + ks]));
    auto mfma_v = [&](auto p_, auto q_) __attribute__((always_inline)) {
      constexpr int p = decltype(p_)::value, q = decltype(q_)::value;
      a64p_mfma_o(o[p >> 1][q], join_tr(vl[p], vh[p]), pf[p & 1][q]);
    };
    auto mfma_v0 = [&](auto p_, auto later_) __attribute__((always_inline)) {   // behind a wait for its reads
      constexpr int p = decltype(p_)::value, N = decltype(later_)::value;
      a64p_mfma_o_w<N>(o[p >> 1][0], join_tr(vl[p], vh[p]), pf[p & 1][0]);
    };
    auto carry = [&]() __attribute__((always_inline)) {
      static_for<2>([&](auto k) {
        constexpr int p = 6 + decltype(k)::value;
        mfma_v(std::integral_constant<int, p>{}, C0{});
        mfma_v(std::integral_constant<int, p>{}, C1{});
      });
    };
    // the twenty reads of the output product, in the order of their use
    auto rd_o = [&](auto r_, uint32_t va, uint32_t vb, uint32_t pa) __attribute__((always_inline)) {
      constexpr int r = decltype(r_)::value;
      if constexpr (r == 0) pf[0][0] = lds_read_b128<0>(pa);
      else if constexpr (r == 1) pf[0][1] = lds_read_b128<2048>(pa);
      else if constexpr (r == 4) pf[1][0] = lds_read_b128<1024>(pa);
      else if constexpr (r == 5) pf[1][1] = lds_read_b128<3072>(pa);
      else {
        constexpr int j = r < 4 ? r - 2 : r - 4;   // 0 .. 15
        constexpr int p = j >> 1, off = (p & 1) * 16 * AB_ROW_BYTES + 64 * (p >> 1);
        if constexpr (j & 1) vh[p] = lds_read_tr16_b64<off>(vb);
        else vl[p] = lds_read_tr16_b64<off>(va);
      }
    };
    constexpr auto need = [](int p) { return p == 0 ? 3 : 5 + 2 * p; };   // the last read that pair p waits for
    const char *pf_lat = nullptr, *pf_rope = nullptr;   // the tile whose transfers are next
    auto prefetch_src = [&](int tile) __attribute__((always_inline)) {
      if (tile >= ntile) return;
      if (tile > 3 && (is_prefix || (tile & 1))) {   // (chunks begin on a 64-token boundary, cache blocks too)
        pf_lat += 32 * lat_stride;
        pf_rope += 32 * rope_stride;
      } else {
        tile_src(tile, pf_lat, pf_rope);
      }
      if (tile == ntile - 1 && last_row < 31) set_doff(last_row);
    };
    uint32_t ring[4] = {slot_of(0), slot_of(1), slot_of(2), slot_of(3)};   // of tiles t .. t + 3
    auto period = [&](int t, auto prefetch_tag) __attribute__((always_inline)) {
      constexpr bool PF = decltype(prefetch_tag)::value;
      const uint32_t cur = ring[0], nxt = ring[1], dst = ring[3];
      const uint32_t ka = nxt + k_off, ra = nxt + r_off, va = cur + v_lo, vb = cur + v_hi;
      const uint32_t pa = p_rd + (t & 1) * 4096, pw = p_wr + ((t + 1) & 1) * 4096;
      static_for<AHEAD>([&](auto i) { rd_k(i, ka, ra); });
      carry();
      score_steps(ka, ra, std::true_type{}, prefetch_tag, pf_lat, pf_rope, dst, [&](auto j_) __attribute__((always_inline)) { rd_o(j_, va, vb, pa); });
      // outputs; twelve of their reads are requested, two more with every pair
      bf16x4 pr[2];
      auto prob_at = [&](auto e_) __attribute__((always_inline)) {
        constexpr int s = decltype(e_)::value >> 2, v = decltype(e_)::value & 3;
        const float x = prob(s, v);
        l[s] += x;
        pr[s][v] = (__bf16)x;
      };
      static_for<6>([&](auto p_) {
        constexpr int p = decltype(p_)::value;
        constexpr int requested = 12 + 2 * p < 20 ? 12 + 2 * p : 20;
        mfma_v0(p_, std::integral_constant<int, requested - 1 - need(p)>{});
        if constexpr (p < 4) rd_o(std::integral_constant<int, 12 + 2 * p>{}, va, vb, pa);
        // one exponential behind each MFMA from the second pair on (where prefetch_src() follows, the compiler
        // moves the first four of them behind its branches)
        if constexpr (p > 0) {
          if constexpr (p < 5) prob_at(std::integral_constant<int, 2 * (p - 1)>{});
          A64P_SB();
        }
        mfma_v(p_, C1{});
        if constexpr (p < 4) rd_o(std::integral_constant<int, 13 + 2 * p>{}, va, vb, pa);
        if constexpr (p == 0) {
          a64p_tie(sacc[0], sacc[1]);
          mask(t + 1);
        } else if constexpr (p < 5) {
          prob_at(std::integral_constant<int, 2 * (p - 1) + 1>{});
          if constexpr (PF && p == 2) prefetch_src(t + 4);
        } else {
          a64p_write_b64(pw, pr[0]);
          a64p_write_b64(pw + 256, pr[1]);
        }
        A64P_SB();
      });
      ring[0] = nxt;
      ring[1] = ring[2];
      ring[2] = dst;
      ring[3] = cur;
      lgkm_wait<0>(vl[6], vh[6], vl[7], vh[7]);
      vm_wait<(PF ? 9 : 0)>();   // tile t + 2
      raw_barrier();
    };
    prefetch_src(3);
    int t = 0;
    for (; t + 3 < ntile; t++) period(t, std::true_type{});
    for (; t + 1 < ntile; t++) period(t, std::false_type{});
    {
      const uint32_t cur = ring[0];
      const uint32_t va = cur + v_lo, vb = cur + v_hi, pa = p_rd + (t & 1) * 4096;
      carry();
      // (the fragments of the pairs carried over are free only now)
      static_for<20>([&](auto r) { rd_o(r, va, vb, pa); });
      static_for<8>([&](auto p_) {
        constexpr int p = decltype(p_)::value;
        constexpr int later = 19 - need(p);
        mfma_v0(p_, std::integral_constant<int, (later < 15 ? later : 15)>{});
        mfma_v(p_, C1{});
      });
      a64p_drain();
    }

    // ---- denominators: the token halves of every query meet in LDS
    raw_barrier();   // everyone is past its last read of the probabilities
#pragma unroll
    for (int s = 0; s < 2; s++) {
      // (where every score of tile 0 was -inf there was no reference for the tokens behind it)
      const bool none = !exact && m[s] == -INFINITY && vis[s] > 32;
      const float lh = none ? INFINITY : a64p_sum_quads(l[s]);
      if (q4 == 0) lds_write_b32(x_wr + 64 * s, lh);
    }
    lgkm_wait<0>();
    raw_barrier();
    {
      const uint32_t at = smem_base + A64P_P_OFF + 4096 + n * 4;
      float x[4] = {lds_read_f32(at), lds_read_f32(at + 128), lds_read_f32(at + 256), lds_read_f32(at + 384)};
      float y[4] = {lds_read_f32(x_wr), lds_read_f32(x_wr + 64), lds_read_f32(x_wr ^ 256), lds_read_f32((x_wr ^ 256) + 64)};
      lgkm_wait<0>(x[0], x[1], x[2], x[3]);
      lgkm_wait<0>(y[0], y[1], y[2], y[3]);
      den[0] = x[0] + x[2];
      den[1] = x[1] + x[3];
      own[0] = y[0] + y[2];
      own[1] = y[1] + y[3];
    }
    if (exact) break;
    // a denominator that is not a moderate finite number: the references did not hold.  Every wavefront
    // reads the same numbers, so the verdict is the same in all of them.
    const bool bad = !(den[0] < 0x1p100f) || !(den[1] < 0x1p100f);
    if (__builtin_amdgcn_ballot_w64(bad) == 0) break;
    raw_barrier();   // everyone has read the denominators
  }
  // ---- outputs, turned around in LDS (slots 2 and 3, which nobody reads any more) and stored as whole rows of
  // 1 KiB, as in the kernel of 64-token steps, whose comment has the times of both ways.
  constexpr int ST_ROW = D_L * 2 + 16;   // conflict-free for the 8-byte writes of 16 rows x 2 halves
  char* st = smem + 2 * AB_TILE_BYTES;
  static_assert(2 * AB_TILE_BYTES + 64 * ST_ROW <= A64P_LDS_BYTES, "the outputs fit the idle slots");
#pragma unroll
  for (int q = 0; q < 2; q++) {
    const float lt = den[q];
    // (0: the causal mask hid every token of this chunk from this query; the row is not read)
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    char* dst = st + (32 * q + n) * ST_ROW + (128 * wave + 4 * g) * 2;
#pragma unroll
    for (int mb = 0; mb < 4; mb++)
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; e++) w[e] = (__bf16)(o[mb][q][4 * v4 + e] * inv);
        *(bf16x4*)(dst + (32 * mb + 8 * v4) * 2) = w;
      }
  }
#pragma unroll
  for (int s = 0; s < 2; s++) {
    const float lt = own[s];
    if (th == 0 && q4 == 0 && r_own[s] < R)
      a.lat_lse[(size_t)item * a.rows + (int64_t)b * R + r_own[s]] =
          lt > 0.f ? (m[s] + fast_log2(lt)) * LN2 : -INFINITY;
  }
  lgkm_wait<0>();
  raw_barrier();
  __bf16* o_dst =
      a.lat_o + ((size_t)item * a.rows + (int64_t)b * R + qg * 64) * D_L + lane * 8;
  const int nrow = min(64, R - qg * 64);
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const int r = 4 * i + wave;
    if (r < nrow) *(bf16x8*)(o_dst + (size_t)r * D_L) = *(const bf16x8*)(st + r * ST_ROW + lane * 16);
  }
}

// Launches that keep the kernel that walks 64 tokens a step.  Chunks of up to 128 tokens: this kernel's code is
// the longer one, and inside a step, where other kernels run in between, its first pass over it costs what
// one or two steps' worth of tiles gain (pass by itself / step, that kernel and this one: 2 x 64 heads over 2048 +
// 603 tokens in chunks of 64 9.75, 9.66 / 19.5, 20.0 us; 8 x 16 over 4096 + 1200 in chunks of 128 10.4, 10.4 / 20.1, 20.7; of
// 192 11.9, 11.1 / 21.7, 21.2).  And launches that cover the chip:
//   * suffixes of up to 64 rows a request, whose workgroups stream rows that no other reads, beside another
//     pass of the call.  Behind a latent prefix the chip's power sets the pace of the step, and the faster pass
//     draws more of it: 256 requests x 64 heads absorb_only, 4096 + 512 tokens, the pass 34.5 us with that kernel and
//     32.0 with this one, the step 189.6 us at 2.15 GHz and 195.0 at 2.04 (on another box 182.5 and 183.3); 339 random
//     absorb_only steps of 33 to 64 rows take 0.98 of their time with this one on average and 1.04 at most.  Behind a
//     naive prefix the line is too wide: 1250 random mixed steps would take 0.96 with this one, 1.00 at most.
//     Without a prefix 256 x 64 heads take 52.6 and 51.7.  Rows in more groups share their tiles: 259 requests x 3 x
//     48 heads over 416 + 1197 tokens 259 and 225 us; fewer workgroups: 28 x 48 heads x 2 over 608 + 537 49.5 and 48.4;
//   * suffixes and latent prefix in one launch, above 32 rows a request.  This kernel would be the faster one (128 x 64
//     heads over 1024 + 512 tokens 61.2 and 52.1 us), but auto mode says mixed from there on (61.7 us): its
//     cross-over for 64 heads and 1024 tokens, which callers know as 128 requests, was measured with that kernel.
//     Up to 32 rows nothing hangs on that kernel: 1736 random steps of 16 and 32 rows that it ran take 0.906 of their
//     time with this one, 1.02 at most, and the cross-overs fit better (16 heads x 4096 + 512, that one / this one / mixed: 128
//     requests 58.6, 50.6, 55.1 us; 192 73.1, 63.3, 70.5; 224 84.3, 76.0, 74.3, cross-over 198).
static bool keeps_steps(const Plan& p, int what, long long wgs) {
  const int longest = std::max((what & WITH_PREFIX) ? p.ap_chunk : 0, (what & WITH_SUFFIX) ? p.as_chunk : 0);
  if (longest <= 128) return true;
  if (wgs < NUM_CU) return false;
  if (what == WITH_SUFFIX) return p.Sq * p.H <= 64 && p.n_naive + p.ap_chunks > 0;
  return what == (WITH_PREFIX | WITH_SUFFIX) && p.Sq * p.H > 32;
}

int mfma_absorb64_attention(const Plan& p, const DecodeArgs& d, const AbsorbArgs& a, int what) {
  Absorb64PipelinedArgs args;
  args.a = a;
  args.exact_only = (debug_flags() & 0x800) != 0;
  long long ids, wgs;
  if (!absorb_grid(p, what, 64, &args.grid, &ids, &wgs)) return TMLA_ERR_UNSUPPORTED;
  if (wgs == 0) return TMLA_OK;
  if (keeps_steps(p, what, wgs)) return mfma_absorb64_steps_attention(p, d, a, what);
  static LdsOptIn lds[2];
  const bool prefix = what & WITH_PREFIX;
  auto kernel = prefix ? absorb64_pipelined_kernel<true> : absorb64_pipelined_kernel<false>;
  if (lds[prefix].ensure((const void*)kernel, A64P_LDS_BYTES) != hipSuccess) return TMLA_ERR_HIP;
  args.a.order = (what & WITH_SUFFIX) ? suffix_request_order(p, d, wgs) : nullptr;
  hipLaunchKernelGGL(kernel, dim3((unsigned)ids), dim3(256), A64P_LDS_BYTES, d.stream, args);
  return TMLA_OK;
}

}  // namespace tmla
