// Absorb-formulation flash-decode over latent cache rows on the matrix cores
// (paper Algorithm 1 step 6; the absorbed queries of step 5 arrive precomputed, the W_UV
// up-projection of step 7 is applied after the split partials are merged because it is linear).
//
// The kernel here takes the suffixes of requests with 17 to 32 query rows (H = 16 with S_q = 2, or
// H = 32): one workgroup = one request x one token chunk.  Each 576-wide cache row is read from HBM
// once per workgroup (fully coalesced 1152-byte rows) into an LDS tile of 32 tokens, and serves both
// products:
//   S^T  = C   Q_abs^T   (tokens x queries, k = 576): A operand = token-major rows (ds_read_b128)
//   O^T += C_N^T P^T     (latent x queries, k = tokens): A operand = the same tile read through
//                         the transposing LDS load (ds_read_b64_tr_b16), no second copy.
// Queries sit on the MFMA column axis, so softmax statistics are per-lane and P^T feeds the second
// product straight from the accumulator registers.  The four wavefronts own 128 latent columns
// each; the scores are recomputed per wavefront, which this HBM-bound case affords.
// Behind it, the dispatch over the absorb kernels.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "tmla_absorb_tile.hpp"

namespace tmla {

__global__ void __launch_bounds__(256, 1) absorb_attn_kernel(AbsorbArgs a) {
  constexpr int MBW = 4;  // 32-latent blocks owned by a wavefront
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int item = a.ap_chunks + blockIdx.x;
  const int b = a.order ? scalar_load_i32(a.order + blockIdx.y) : (int)blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: transfer bookkeeping is SALU
  const bool q_valid = n < a.R;                    // n: this lane's query row within the request
  const int64_t row = (int64_t)b * a.R + n;        // global output row (b, s, h)

  // ---- which tokens
  const int len = scalar_load_i32(a.lens + b);
  const int t0 = (item - a.ap_chunks) * a.as_chunk;
  const int t1 = min(len, t0 + a.as_chunk);
  const int vis_q = max(0, min(len, len - a.Sq + query_position(n, a.H, a.R) + 1));
  float* l_dst = a.lat_lse + (size_t)item * a.rows + row;
  if (t1 <= t0) {   // empty chunk (workgroup-uniform)
    if (q_valid && wave == 0 && g == 0) *l_dst = -INFINITY;
    return;
  }
  const int ntile = (t1 - t0 + 31) / 32;

  // ---- tile streaming: global -> LDS.
  // The physical blocks of this chunk are fetched once, one entry per lane (a chunk spans at most
  // 64 blocks here, longer ones fall back to a scalar load per tile), and picked with v_readlane:
  // no memory latency on the tile-issue path.
  const int32_t* bt = a.block_table + (size_t)b * a.max_blocks;
  const int first_blk = t0 >> a.bs_shift;
  const int nblk_chunk = ((t1 - 1) >> a.bs_shift) - first_blk + 1;
  int bt_cache = (lane < nblk_chunk) ? bt[first_blk + lane] : 0;
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(bt_cache)::"memory");
  const DmaLane dl = dma_lane(wave, lane);
  auto tile_src = [&](int tile) __attribute__((always_inline)) {
    RowSrc s;
    const int tok0 = t0 + tile * 32;
    s.last = t1 - 1 - tok0;              // last valid row of this tile (>= 0)
    s.stream = true;
    const int bi = __builtin_amdgcn_readfirstlane((tok0 >> a.bs_shift) - first_blk);
    const int blk = bi < 64 ? __builtin_amdgcn_readlane(bt_cache, bi)
                            : scalar_load_i32(bt + first_blk + bi);
    s.lat = (const char*)(a.pool + ((size_t)blk << a.bs_shift) * D_ROW + (tok0 & ((1 << a.bs_shift) - 1)) * D_ROW);
    s.rope = s.lat + D_L * 2;
    s.lat_stride = s.rope_stride = D_ROW * 2;
    return s;
  };
  auto slot_ptr = [&](int tile) __attribute__((always_inline)) {
    return smem + (tile % AB_NSLOT) * AB_TILE_BYTES;
  };

  // per-lane LDS byte offsets inside a tile (tmla_absorb_tile.hpp)
  const uint32_t smem_base = lds_addr(smem);
  const TileLane tl = tile_lane(lane);
  const uint32_t v_lo = tl.v_lo + 64 * (wave * MBW), v_hi = tl.v_hi + 64 * (wave * MBW);

  // ---- absorbed query fragments (B operand): 36 k-steps of 16.
  // The absorbed-query rows are staged like a cache tile (same transfers, same layout) in the last
  // ring slot, and every wavefront picks the fragments with the score-product read pattern: the
  // rows are fetched once per workgroup with full 1 KiB transfers instead of once per wavefront
  // with 32-byte pieces.  The first tiles of the chunk stream into the other slots meanwhile.
  constexpr int NPRE = AB_NSLOT - 1;   // tiles issued next to the query block
  {
    RowSrc qs;
    qs.stream = false;
    qs.last = a.R - 1;                 // (17 to 32 rows a request)
    qs.lat = (const char*)(a.qabs + (int64_t)b * a.R * D_ROW);
    qs.rope = qs.lat + D_L * 2;
    qs.lat_stride = qs.rope_stride = D_ROW * 2;
    issue_all(qs, smem + NPRE * AB_TILE_BYTES, dl);
  }
#pragma unroll
  for (int t = 0; t < NPRE; t++)
    if (t < ntile) issue_all(tile_src(t), slot_ptr(t), dl);
  {
    const int pre = min(ntile, NPRE);    // tiles in flight behind the query block
    if (pre >= 3) vm_wait<3 * AB_DMA_PER_WAVE>();
    else if (pre == 2) vm_wait<2 * AB_DMA_PER_WAVE>();
    else vm_wait<AB_DMA_PER_WAVE>();
  }
  raw_barrier();
  bf16x8 qf[36];
  {
    const uint32_t qa = smem_base + NPRE * AB_TILE_BYTES;
    static_for<32>([&](auto ks) { qf[decltype(ks)::value] = tile_score_frag<decltype(ks)::value>(qa, tl); });
    static_for<4>([&](auto k) { qf[32 + decltype(k)::value] = lds_read_b128<0>(qa + tl.r_off[decltype(k)::value]); });
#pragma unroll
    for (int ks = 0; ks < 36; ks += 4)
      lgkm_wait<0>(qf[ks], qf[ks + 1], qf[ks + 2], qf[ks + 3]);
  }
  raw_barrier();   // the query slot may now be overwritten by a tile

  f32x16 o[MBW];
#pragma unroll
  for (int mb = 0; mb < MBW; mb++)
#pragma unroll
    for (int v = 0; v < 16; v++) o[mb][v] = 0.f;
  float m = -INFINITY, l = 0.f;

  for (int tile = 0; tile < ntile; tile++) {
    // this wavefront's transfers of `tile` are complete once at most the transfers of the
    // following (up to two) tiles remain in flight
    const int ahead = ntile - 1 - tile;
    if (ahead >= 2) vm_wait<2 * AB_DMA_PER_WAVE>();
    else if (ahead == 1) vm_wait<AB_DMA_PER_WAVE>();
    else vm_wait<0>();
    raw_barrier();   // everyone's part of `tile` has landed; everyone is done with tile - 1
    // The four wavefronts run the same instruction stream; leaving the barrier together they
    // would present their transfers and LDS reads at the same cycle and queue behind each
    // other.  A skew of 32 cycles per wavefront (one MFMA) keeps them apart.
    if (wave & 1) asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    if (wave & 2) asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    // the tile three ahead goes into the slot freed by the barrier; its transfers are spread
    // over the score product (one per group of four MFMAs) so that the wavefront never sits
    // behind a full memory-instruction queue
    const int pf = tile + AB_NSLOT - 1;
    const bool do_pf = pf < ntile;
    RowSrc pf_src;
    if (do_pf) pf_src = tile_src(pf);
    char* pf_dst = slot_ptr(pf);

    const uint32_t tbase = smem_base + (tile % AB_NSLOT) * AB_TILE_BYTES;
    f32x16 sacc;
#pragma unroll
    for (int v = 0; v < 16; v++) sacc[v] = 0.f;
    {
      // 9 groups of 4 k-steps (the last one is the rope part); three fragment buffers in
      // rotation keep two groups of LDS reads in flight behind the one feeding the MFMAs
      bf16x8 f[3][4];
      auto rd = [&](auto gsel, auto dsel) __attribute__((always_inline)) {
        constexpr int G = decltype(gsel)::value;
        constexpr int D = decltype(dsel)::value;
        if constexpr (G < 8) {
          static_for<4>([&](auto j) {
            f[D][j] = tile_score_frag<4 * G + decltype(j)::value>(tbase, tl);
          });
        } else {
          static_for<4>([&](auto j) {
            f[D][j] = lds_read_b128<0>(tbase + tl.r_off[decltype(j)::value]);
          });
        }
      };
      rd(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
      rd(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
      static_for<9>([&](auto grp) {
        constexpr int G = decltype(grp)::value;
        constexpr int cur = G % 3;
        if constexpr (G + 2 < 9) {
          rd(std::integral_constant<int, G + 2>{}, std::integral_constant<int, (G + 2) % 3>{});
          lgkm_wait<8>(f[cur][0], f[cur][1], f[cur][2], f[cur][3]);
        } else if constexpr (G + 1 < 9) {
          lgkm_wait<4>(f[cur][0], f[cur][1], f[cur][2], f[cur][3]);
        } else {
          lgkm_wait<0>(f[cur][0], f[cur][1], f[cur][2], f[cur][3]);
        }
        static_for<4>([&](auto j) {
          sacc = mfma32(f[cur][j], qf[4 * G + decltype(j)::value], sacc);
        });
        if (do_pf) issue_part<G>(pf_src, pf_dst, dl);
      });
    }
    const int limit = min(32, vis_q - (t0 + tile * 32));
    bf16x8 p[2];
    bool rescale;
    const float alpha = softmax_block(sacc, m, l, a.c, limit, g, p[0], p[1], rescale);
    if (rescale) {
      // (the asm statements keep the accumulator <-> vector register copies inside this branch)
#pragma unroll
      for (int mb = 0; mb < MBW; mb++) {
        asm volatile("" : "+a"(o[mb]));
#pragma unroll
        for (int v = 0; v < 16; v++) o[mb][v] *= alpha;
        asm volatile("" : "+a"(o[mb]));
      }
    }
    {
      // step st = 2*mb + kk; groups of 4 steps (8 transposing reads), double buffered
      const uint32_t va = tbase + v_lo, vh = tbase + v_hi;
      constexpr int NSTEP = 2 * MBW, NGRP = NSTEP / 4;
      short4v lo[2][4], hi[2][4];
      static_for<4>([&](auto j) {
        constexpr int st = decltype(j)::value;
        constexpr int off = (16 * (st & 1)) * AB_ROW_BYTES + 64 * (st >> 1);
        lo[0][st] = lds_read_tr16_b64<off>(va);
        hi[0][st] = lds_read_tr16_b64<off>(vh);
      });
      static_for<NGRP>([&](auto grp) {
        constexpr int G = decltype(grp)::value;
        constexpr int cur = G & 1, nxt = cur ^ 1;
        if constexpr (G + 1 < NGRP) {
          static_for<4>([&](auto j) {
            constexpr int st = 4 * (G + 1) + decltype(j)::value;
            constexpr int off = (16 * (st & 1)) * AB_ROW_BYTES + 64 * (st >> 1);
            lo[nxt][decltype(j)::value] = lds_read_tr16_b64<off>(va);
            hi[nxt][decltype(j)::value] = lds_read_tr16_b64<off>(vh);
          });
          lgkm_wait<8>(lo[cur][0], lo[cur][1], lo[cur][2], lo[cur][3]);
          lgkm_wait<8>(hi[cur][0], hi[cur][1], hi[cur][2], hi[cur][3]);
        } else {
          lgkm_wait<0>(lo[cur][0], lo[cur][1], lo[cur][2], lo[cur][3]);
          lgkm_wait<0>(hi[cur][0], hi[cur][1], hi[cur][2], hi[cur][3]);
        }
        static_for<4>([&](auto j) {
          constexpr int st = 4 * G + decltype(j)::value;
          o[st >> 1] = mfma32(join_tr(lo[cur][decltype(j)::value], hi[cur][decltype(j)::value]),
                              p[st & 1], o[st >> 1]);
        });
      });
    }
  }

  // ---- outputs, turned around in the slot that the last barrier left idle: whole rows of 1 KiB
  // instead of 8-byte pieces of 32 rows per instruction (steps of 1 to 40 requests x 32 heads, 64 to
  // 2500 tokens, 0.8 to 1.2 us shorter: 12 x 64 16.4 -> 15.4)
  constexpr int ST_ROW = D_L * 2 + 16;
  static_assert(32 * ST_ROW <= AB_TILE_BYTES, "the outputs fit a slot");
  const float lt = sum_halves(l);
  // (0: the causal mask hid every token of this chunk from this query; the row is not read)
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  char* st = slot_ptr(ntile);
#pragma unroll
  for (int mb = 0; mb < MBW; mb++)
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; e++) w[e] = (__bf16)(o[mb][4 * v4 + e] * inv);
      *(bf16x4*)(st + n * ST_ROW + (32 * (wave * MBW + mb) + 8 * v4 + 4 * g) * 2) = w;
    }
  if (wave == 0 && g == 0 && q_valid) *l_dst = lt > 0.f ? (m + fast_log2(lt)) * LN2 : -INFINITY;
  lgkm_wait<0>();
  raw_barrier();
  __bf16* o_dst = a.lat_o + ((size_t)item * a.rows + (int64_t)b * a.R) * D_L + lane * 8;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int r = 4 * i + wave;
    if (r < a.R) *(bf16x8*)(o_dst + (size_t)r * D_L) = *(const bf16x8*)(st + r * ST_ROW + lane * 16);
  }
}

__global__ void __launch_bounds__(256) suffix_order_kernel(const int32_t* lens, int B, int32_t* order) {
  rank_suffix(lens, B, order, blockIdx.x * 4 + (threadIdx.x >> 6));
}

// Workgroups are handed to the compute units in index order, each unit taking the next one when
// it is free.  When there are more workgroups than units and the suffix lengths differ, the
// pass ends with a few units working on late long requests while the rest idle; starting the
// longest requests first evens that out.  Debug flags:
// bit 14 orders whatever the grid size, bit 15 never orders.
constexpr int ORDER_MAX_BATCH = 4096;   // the ranking is quadratic in the batch size
static bool order_wanted(const Plan& p, long long wgs) {
  if (p.as_chunks <= 0 || p.B < 2 || p.B > ORDER_MAX_BATCH || (debug_flags() & 0x8000)) return false;
  return wgs > NUM_CU || (debug_flags() & 0x4000);
}
const int32_t* suffix_request_order(const Plan& p, const DecodeArgs& d, long long wgs) {
  if (!order_wanted(p, wgs)) return nullptr;
  int32_t* order = (int32_t*)(d.ws + p.off_order);
  if (!d.ranked)
    hipLaunchKernelGGL(suffix_order_kernel, dim3((p.B + 3) / 4), dim3(256), 0, d.stream, d.suffix_lens,
                       p.B, order);
  return order;
}

bool absorb_grid(const Plan& p, int what, int rows_per_wg, AbsorbGrid* g, long long* ids,
                 long long* wgs) {
  constexpr int XCDS = 8;
  const int R = p.Sq * p.H;
  const long long groups = (p.rows + rows_per_wg - 1) / rows_per_wg;
  const long long pre = (what & WITH_PREFIX) ? p.ap_chunks * groups : 0;
  const int suf_chunks = (what & WITH_SUFFIX) ? p.as_chunks : 0;
  const int suf_groups = (R + rows_per_wg - 1) / rows_per_wg;
  const long long units = (long long)suf_chunks * p.B;
  *wgs = pre + units * suf_groups;
  // rounds of workgroups on the fullest XCD with whole units, and with the work dealt out evenly.
  // (4 requests x 3 x 128 heads absorb_only over 1000 + 2485 tokens, 72 + 28 x 6 = 240 workgroups:
  // 33 on four XCDs of 32 units, 64 us a step; 30 on each, 45 us.)
  long long fullest = 0;
  for (int x = 0; x < XCDS; x++) {
    const int r = (int)((x + XCDS - pre % XCDS) % XCDS);   // its residue among the suffix ids
    fullest = std::max(fullest, pre / XCDS + (x < pre % XCDS) +
                                    suf_groups * (units / XCDS + (r < units % XCDS)));
  }
  auto rounds = [](long long n) { return (n + NUM_CU / XCDS - 1) / (NUM_CU / XCDS); };
  const bool spread = rounds(fullest) > rounds((*wgs + XCDS - 1) / XCDS);
  const long long whole = spread ? units / XCDS * XCDS : (units + XCDS - 1) / XCDS * XCDS;
  *ids = spread ? *wgs : pre + whole * suf_groups;
  if (*ids > 0x7fffffffLL) return false;
  g->pre_wgs = (int)pre;
  g->pre_each = (int)(pre / XCDS);
  g->pre_more = (int)(pre % XCDS);
  g->rotate = p.B % XCDS == 0 ? XCDS - 1 : 0;
  g->suf_units = (int)units;
  g->spread_id = (int)(whole * suf_groups);
  g->spread_unit = (int)whole;
  g->pre_groups.set((uint32_t)groups);
  g->suf_groups.set((uint32_t)suf_groups);
  g->batch.set((uint32_t)p.B);
  return true;
}

// The kernels of a call's absorb passes.  Debug flags: bit 12 keeps the 64-row kernel, bit 13 takes the
// 128-row kernel whatever the grid size.
struct AbsorbKernels {
  bool joint;              // prefix and suffixes in one launch of pre_rows rows a workgroup
  int pre_rows, own_rows;  // 64 or 128; the suffixes' kernel: 16, 32, 64 or 128
};
static AbsorbKernels absorb_kernels(const Plan& p) {
  const bool keep64 = debug_flags() & 0x1000, force128 = debug_flags() & 0x2000;
  const int R = p.Sq * p.H;
  AbsorbKernels k;
  k.joint = p.abs_joint && !force128;
  k.pre_rows = (p.ap_rows == 128 && !keep64) || force128 ? 128 : 64;
  // 128 rows per workgroup when the request has whole blocks of them and the grid still covers
  // the chip.  Pass of 256 requests x 128 heads with 128 / 64 rows a workgroup: 256 tokens 31.0 / 37.6 us, 512 45.1 /
  // 52.1, 1024 74.7 / 85.7, 2048 137 / 167, 4096 272 / 307 (beside 32768 prefix tokens 153 / 166 and the step 743 /
  // 760); 128 x 2 x 128 heads over 1024 72.3 / 83.6; latent prefix and suffix, 256 x 128 over 4096 + 512 280 / 295.
  const bool rows128 = R % 128 == 0 && !keep64 &&
                       (force128 || (long long)p.as_chunks * p.B * (R / 128) >= NUM_CU);
  k.own_rows = R <= 16 ? 16 : rows128 ? 128 : R > 32 ? 64 : 32;
  return k;
}

bool suffix_order_wanted(const Plan& p) {
  if (p.n_lat <= 0 || p.rows == 0 || p.as_chunks <= 0) return false;
  const AbsorbKernels k = absorb_kernels(p);
  const int rows = k.joint ? k.pre_rows : k.own_rows;
  if (rows <= 32) return order_wanted(p, (long long)p.as_chunks * p.B);
  AbsorbGrid grid;
  long long ids, wgs;
  return absorb_grid(p, k.joint ? WITH_PREFIX | WITH_SUFFIX : WITH_SUFFIX, rows, &grid, &ids, &wgs) &&
         order_wanted(p, wgs);
}

int mfma_absorb_attention(const Plan& p, const DecodeArgs& d) {
  if (p.n_lat <= 0 || p.rows == 0) return TMLA_OK;
  AbsorbArgs a;
  a.qabs = (const __bf16*)(d.ws + p.off_qabs);
  a.pc = (const __bf16*)d.prefix_ckv;
  a.pr = (const __bf16*)d.prefix_krope;
  a.pool = (const __bf16*)d.suffix_pool;
  a.block_table = d.block_table;
  a.lens = d.suffix_lens;
  a.order = nullptr;
  a.lat_o = (__bf16*)(d.ws + p.off_lat_o);
  a.lat_lse = (float*)(d.ws + p.off_lat_lse);
  a.Sq = p.Sq; a.H = p.H; a.R = p.Sq * p.H; a.Ls = p.Ls;
  a.ap_chunks = p.ap_chunks; a.ap_chunk = p.ap_chunk;
  a.as_chunks = p.as_chunks; a.as_chunk = p.as_chunk;
  a.max_blocks = d.max_blocks; a.bs_shift = __builtin_ctz((unsigned)d.block_size);
  a.rows = p.rows;
  a.c = d.sm_scale * LOG2E;
  const AbsorbKernels k = absorb_kernels(p);
  if (k.joint)
    return k.pre_rows == 128 ? mfma_absorb128_attention(p, d, a, WITH_PREFIX | WITH_SUFFIX)
                             : mfma_absorb64_attention(p, d, a, WITH_PREFIX | WITH_SUFFIX);
  if (p.ap_chunks > 0) {
    const int rc = k.pre_rows == 128 ? mfma_absorb128_attention(p, d, a, WITH_PREFIX)
                                     : mfma_absorb64_attention(p, d, a, WITH_PREFIX);
    if (rc != TMLA_OK || p.as_chunks == 0) return rc;
  }
  if (k.own_rows == 16) return mfma_absorb16_attention(p, d, a);
  if (k.own_rows == 128) return mfma_absorb128_attention(p, d, a, WITH_SUFFIX);
  if (k.own_rows == 64) return mfma_absorb64_attention(p, d, a, WITH_SUFFIX);
  static LdsOptIn lds;
  auto kernel = absorb_attn_kernel;
  if (lds.ensure((const void*)kernel, AB_LDS_BYTES) != hipSuccess) return TMLA_ERR_HIP;
  dim3 grid(p.as_chunks, p.B);
  a.order = suffix_request_order(p, d, (long long)p.as_chunks * p.B);
  hipLaunchKernelGGL(kernel, grid, dim3(256), AB_LDS_BYTES, d.stream, a);
  return TMLA_OK;
}

}  // namespace tmla
