// Absorb-formulation flash-decode for requests with at most 16 query rows (S_q * H <= 16: one
// tensor-parallel rank's head share), paper Algorithm 1 step 6.  This is the HBM-bound case
// (about 30 FLOP per cache byte), so the design minimises everything except the cache stream:
//
//   * v_mfma_f32_16x16x32_bf16 with the 16 queries on the column axis: no padding to 32 columns;
//   * every wavefront walks a contiguous quarter of the workgroup's chunk with a private 32-token
//     LDS tile: it streams its own tokens (global -> LDS), reads the tile once for the scores and
//     once (transposed) for P V, and does not synchronise with the other wavefronts meanwhile.
//     Each cache row is therefore read from LDS exactly twice per workgroup, and the latency of
//     a wavefront's tile load is hidden by the other three wavefronts of the compute unit.  The
//     chunk is divided at run time, so that a request shorter than the planned chunk still uses
//     all four;
//   * the four partial softmaxes are merged in fp32 through LDS at the end: one latent partial per
//     chunk, whole rows of 1 KiB.  Written out one by one, in 8-byte pieces, they were four bf16
//     partials a row that the projection had to fetch and to merge: 512 requests x 16 heads mixed,
//     16384 + 512 to 4096 tokens, 67 -> 42 MB for it to read, step 348 -> 327 us.
//
// MFMA 16x16x32 operand layout (lane = n + 16*q, n in [0,16), q in [0,4)):
//   A (16 x 32): row n, k = 8*q + e;   B (32 x 16): column n, k = 8*q + e;
//   D (16 x 16): column n, rows 4*q + v, v in [0,4).
#include <type_traits>

#include "tmla_absorb_tile.hpp"

namespace tmla {

// private tile layout: latent rows at r * 1056 with the 16-byte chunk c in slot
// c ^ ((r >> 3) & 1), then 32 x 128 B of rope with chunk c of row r in slot c ^ ((r >> 1) & 7).
// The LDS has 64 four-byte banks; a 16-byte read is served 16 lanes at a time (of each half 0 .. 3, 12 .. 15 and
// 20 .. 27, then the others), an 8-byte transposing read 32 lanes at a time.  The row stride is 8 banks mod
// 64: the transposing reads of the output product (8 rows x 32 B per 32 lanes) cover the banks exactly.
// The score product's reads take two turns a group: rows r and r + 8 sit in different halves of a 32-byte
// pair, but a group has rows 0 .. 3 and 12 .. 15 of one chunk with 4 .. 11 of the next, which fall
// on the same banks (8.2 cycles a read, 4.3 without conflicts).  Rope rows of equal parity share 32 banks; the swizzle separates the eight
// of them that a 16-lane group reads.
constexpr int A16_ROW_BYTES = 1056;
constexpr int A16_MAIN_BYTES = 32 * A16_ROW_BYTES;
constexpr int A16_TILE_BYTES = A16_MAIN_BYTES + 32 * 128;   // 37888
constexpr int A16_ML_OFF = 4 * A16_TILE_BYTES;              // [wavefront][reference, denominator][row]
// A chunk of up to this many tokens is one wavefront's, which writes its rows itself: the shares of two meet
// in LDS (32 KiB a wavefront, there and back) later than one has walked two tiles.  Steps in one chunk
// of 20 / 64 tokens, shared out and alone: 8 requests 16.5 / 16.8 and 14.4 / 15.9 us, 300 requests 32.5 / 34.5
// and 28.3 / 33.0.
constexpr int A16_ALONE = 64;
constexpr int A16_LDS_BYTES = A16_ML_OFF + 4 * 2 * 16 * 4;
// a wavefront's outputs in its tile at the end: 512 floats a row, conflict-free for 16 rows x 16 B
constexpr int A16_OUT_ROW = D_L * 4 + 16;
static_assert(16 * A16_OUT_ROW <= A16_TILE_BYTES && A16_LDS_BYTES <= 163840, "LDS layout");

__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// max / sum over the four lanes n, n+16, n+32, n+48 (all four end up with the result)
__device__ inline float max_quads(float x) {
  int xi = __float_as_int(x);
  auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  x = fmaxf(__int_as_float(r[0]), __int_as_float(r[1]));
  return max_halves(x);
}
__device__ inline float sum_quads(float x) {
  int xi = __float_as_int(x);
  auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
  x = __int_as_float(r[0]) + __int_as_float(r[1]);
  return sum_halves(x);
}

__global__ void __launch_bounds__(256, 1) absorb16_kernel(AbsorbArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int chunk = blockIdx.x, b = a.order ? scalar_load_i32(a.order + blockIdx.y) : (int)blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool q_valid = n < a.R;
  const int64_t row = (int64_t)b * a.R + n;

  // ---- the chunk of this workgroup and this wavefront's share of it
  const int len = scalar_load_i32(a.lens + b);
  const int span0 = chunk * a.as_chunk;
  const int span1 = min(len, span0 + a.as_chunk);
  const int item = a.ap_chunks + chunk;
  float* l_dst = a.lat_lse + (size_t)item * a.rows + row;
  if (span1 <= span0) {   // empty chunk (workgroup-uniform): only the LSEs are defined
    if (wave == 0 && q_valid && q4 == 0) *l_dst = -INFINITY;
    return;
  }
  const bool alone = span1 - span0 <= A16_ALONE;
  if (alone && wave > 0) return;
  // tokens per wavefront, tile aligned
  const int part = alone ? A16_ALONE : ((span1 - span0 + 3) / 4 + 31) & ~31;
  const int t0 = __builtin_amdgcn_readfirstlane(span0 + wave * part);
  const int t1 = __builtin_amdgcn_readfirstlane(min(span1, t0 + part));
  const int vis_q = max(0, min(len, len - a.Sq + query_position(n, a.H, a.R) + 1));
  const int ntile = t1 > t0 ? (t1 - t0 + 31) / 32 : 0;

  // ---- tile streaming into this wavefront's private slot: 32 latent rows + 4 rope groups
  char* slot = smem + wave * A16_TILE_BYTES;
  // physical blocks of this wavefront's token range: one entry per lane, picked with v_readlane
  // (ranges longer than 64 blocks fall back to a scalar load per tile)
  const int32_t* bt = a.block_table + (size_t)b * a.max_blocks;
  const int first_blk = t0 >> a.bs_shift;
  const int nblk_mine = ((t1 - 1) >> a.bs_shift) - first_blk + 1;
  int bt_cache = (lane < nblk_mine) ? bt[first_blk + lane] : 0;
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(bt_cache)::"memory");
  const uint32_t tbase = lds_addr(slot);
  const int lane_off0 = lane << 4, lane_off1 = (lane ^ 1) << 4;
  const int rope_ch = ((lane & 7) ^ (lane >> 4)) << 4;   // rope group 0; odd groups: ^ 64
  auto issue = [&](int tile) __attribute__((always_inline)) {
    const int tok0 = t0 + tile * 32;
    const int last = t1 - 1 - tok0;      // last valid row of this tile (>= 0)
    const int bi = __builtin_amdgcn_readfirstlane((tok0 >> a.bs_shift) - first_blk);
    const int blk = bi < 64 ? __builtin_amdgcn_readlane(bt_cache, bi)
                            : scalar_load_i32(bt + first_blk + bi);
    const char* base =
        (const char*)(a.pool + ((size_t)blk << a.bs_shift) * D_ROW + (tok0 & ((1 << a.bs_shift) - 1)) * D_ROW);
    constexpr int row_bytes = D_ROW * 2;
    // (scalar base + lane offset: with a 64-bit vector address per transfer the 64 x 3000-token
    // pass takes 39 us instead of 34.5)
#pragma unroll
    for (int r = 0; r < 32; r++) {
      const int rr = min(r, last);
      const int loff = ((r >> 3) & 1) ? lane_off1 : lane_off0;
      dma16_scalar_base<true>(loff, base + (size_t)rr * row_bytes, tbase, r * A16_ROW_BYTES);
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int rr = min(8 * j + (lane >> 3), last);
      dma16_scalar_base<true>(rr * row_bytes + (rope_ch ^ ((j & 1) << 6)), base + D_L * 2, tbase, A16_MAIN_BYTES + j * 1024);
    }
  };
  if (ntile > 0) issue(0);

  // ---- absorbed query fragments (B operand): 18 k-steps of 32
  bf16x8 qf[18];
  {
    const __bf16* qp = a.qabs + row * D_ROW + 8 * q4;
#pragma unroll
    for (int ks = 0; ks < 18; ks++) {
      bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
      qf[ks] = q_valid ? *(const bf16x8*)(qp + 32 * ks) : z;
    }
  }
#pragma unroll
  for (int ks = 0; ks < 18; ks += 3)
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(qf[ks]), "+v"(qf[ks + 1]), "+v"(qf[ks + 2])::"memory");

  // ---- per-lane LDS addresses
  //   scores, latent k-step ks < 16, token block mb: row 16*mb + n, chunk 4*ks + q4
  //       -> (16*mb + n)*1056 + ((q4 ^ sw) * 16) + 64*ks,  sw = (n >> 3) & 1 (16*mb does not change it)
  //   rope k-step k < 2: chunk c = 4*k + q4 in slot c ^ ((row >> 1) & 7), the same for row n
  //       and row 16 + n
  const uint32_t s_addr = tbase + n * A16_ROW_BYTES + ((q4 ^ ((n >> 3) & 1)) << 4);
  uint32_t r_addr[2];
#pragma unroll
  for (int k = 0; k < 2; k++)
    r_addr[k] = tbase + A16_MAIN_BYTES + n * 128 + (((4 * k + q4) ^ ((n >> 1) & 7)) << 4);
  //   P V (transposing read inside the 16-lane group q4, r = lane % 16):
  //     token row 16*half + 4*q4 + r/4, latent 16*mb + 4*(r%4); row swizzle bit = q4 >> 1
  const uint32_t v_addr = tbase + (4 * q4 + (n >> 2)) * A16_ROW_BYTES +
                          ((((n & 3) >> 1) ^ (q4 >> 1)) << 4) + 8 * (n & 1);

  f32x4 o[32];
#pragma unroll
  for (int mb = 0; mb < 32; mb++)
#pragma unroll
    for (int v = 0; v < 4; v++) o[mb][v] = 0.f;
  float m = -INFINITY, l = 0.f;

  for (int tile = 0; tile < ntile; tile++) {
    vm_wait<0>();   // this wavefront's own transfers of the tile (nothing else is in flight)
    // ---- scores: two 16-token blocks x 18 k-steps
    f32x4 sacc[2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int v = 0; v < 4; v++) sacc[i][v] = 0.f;
    {
      // groups of 2 k-steps = 4 fragments (2 token blocks each), double buffered; 9 groups,
      // the last one is the rope part
      bf16x8 f[2][4];
      auto rd = [&](auto gsel, auto dsts) {
        constexpr int G = decltype(gsel)::value;
        constexpr int D = decltype(dsts)::value;
        if constexpr (G < 8) {
          f[D][0] = lds_read_b128<64 * (2 * G)>(s_addr);
          f[D][1] = lds_read_b128<64 * (2 * G) + 16 * A16_ROW_BYTES>(s_addr);
          f[D][2] = lds_read_b128<64 * (2 * G + 1)>(s_addr);
          f[D][3] = lds_read_b128<64 * (2 * G + 1) + 16 * A16_ROW_BYTES>(s_addr);
        } else {
          f[D][0] = lds_read_b128<0>(r_addr[0]);
          f[D][1] = lds_read_b128<16 * 128>(r_addr[0]);
          f[D][2] = lds_read_b128<0>(r_addr[1]);
          f[D][3] = lds_read_b128<16 * 128>(r_addr[1]);
        }
      };
      rd(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
      static_for<9>([&](auto grp_c) {
        constexpr int G = decltype(grp_c)::value;
        constexpr int cur = G & 1, nxt = cur ^ 1;
        if constexpr (G + 1 < 9) {
          rd(std::integral_constant<int, G + 1>{}, std::integral_constant<int, nxt>{});
          lgkm_wait<4>(f[cur][0], f[cur][1], f[cur][2], f[cur][3]);
        } else {
          lgkm_wait<0>(f[cur][0], f[cur][1], f[cur][2], f[cur][3]);
        }
        sacc[0] = mfma16(f[cur][0], qf[2 * G], sacc[0]);
        sacc[1] = mfma16(f[cur][1], qf[2 * G], sacc[1]);
        sacc[0] = mfma16(f[cur][2], qf[2 * G + 1], sacc[0]);
        sacc[1] = mfma16(f[cur][3], qf[2 * G + 1], sacc[1]);
      });
    }
    // ---- online softmax over the 8 scores this lane holds (tokens 16*i + 4*q4 + v)
    const int limit = vis_q - (t0 + tile * 32);
    float s8[8];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const float x = sacc[i][v];
        s8[4 * i + v] = (limit < 32 && 16 * i + 4 * q4 + v >= limit) ? -INFINITY : x;
      }
    float mx = s8[0];
#pragma unroll
    for (int e = 1; e < 8; e++) mx = fmaxf(mx, s8[e]);
    mx = max_quads(mx) * a.c;
    const float m_new = (mx > m + RESCALE_TAU) ? mx : m;   // lazy reference, see softmax_block
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
      const float alpha = fast_exp2(m - m_use);
      l *= alpha;
      // the accumulators live in accumulation registers, which the vector ALU cannot address;
      // routing them through these statements keeps their copies inside the rare branch
      // (otherwise the copies are hoisted and run for every tile)
#pragma unroll
      for (int mb = 0; mb < 32; mb++) {
        asm volatile("" : "+a"(o[mb]));
#pragma unroll
        for (int v = 0; v < 4; v++) o[mb][v] *= alpha;
        asm volatile("" : "+a"(o[mb]));
      }
    }
    m = m_new;
    bf16x8 p;
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float pe = fast_exp2(__builtin_fmaf(s8[e], a.c, -m_use));
      sum += pe;
      p[e] = (__bf16)pe;
    }
    l += sum;
    // ---- P V: 32 latent blocks of 16, one k-step of 32 tokens; groups of 4 blocks
    {
      short4v lo[2][4], hi[2][4];
      auto rdv = [&](auto gsel, auto dsts) {
        constexpr int G = decltype(gsel)::value;
        constexpr int D = decltype(dsts)::value;
        static_for<4>([&](auto j) {
          constexpr int mb = 4 * G + decltype(j)::value;
          lo[D][decltype(j)::value] = lds_read_tr16_b64<32 * mb>(v_addr);
          hi[D][decltype(j)::value] = lds_read_tr16_b64<32 * mb + 16 * A16_ROW_BYTES>(v_addr);
        });
      };
      rdv(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
      static_for<8>([&](auto grp_c) {
        constexpr int G = decltype(grp_c)::value;
        constexpr int cur = G & 1, nxt = cur ^ 1;
        if constexpr (G + 1 < 8) {
          rdv(std::integral_constant<int, G + 1>{}, std::integral_constant<int, nxt>{});
          lgkm_wait<8>(lo[cur][0], lo[cur][1], lo[cur][2], lo[cur][3]);
          lgkm_wait<8>(hi[cur][0], hi[cur][1], hi[cur][2], hi[cur][3]);
        } else {
          lgkm_wait<0>(lo[cur][0], lo[cur][1], lo[cur][2], lo[cur][3]);
          lgkm_wait<0>(hi[cur][0], hi[cur][1], hi[cur][2], hi[cur][3]);
        }
        static_for<4>([&](auto j) {
          constexpr int mb = 4 * G + decltype(j)::value;
          o[mb] = mfma16(join_tr(lo[cur][decltype(j)::value], hi[cur][decltype(j)::value]), p,
                         o[mb]);
        });
      });
    }
    // every LDS read of the tile has been consumed: the slot can be refilled
    if (tile + 1 < ntile) issue(tile + 1);
  }

  if (alone) {
    const float lt = sum_quads(l), inv = lt > 0.f ? 1.f / lt : 0.f;
    if (!q_valid) return;
    __bf16* o_dst = a.lat_o + ((size_t)item * a.rows + row) * D_L + 4 * q4;
#pragma unroll
    for (int mb = 0; mb < 32; mb++) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; e++) w[e] = (__bf16)(o[mb][e] * inv);
      *(bf16x4*)(o_dst + 16 * mb) = w;
    }
    if (q4 == 0) *l_dst = lt > 0.f ? (m + fast_log2(lt)) * LN2 : -INFINITY;
    return;
  }

  // ---- merge of the four wavefronts: weights from their references and denominators, weighted
  // outputs into the own tile (free by now), whole rows out
  float* ml = (float*)(smem + A16_ML_OFF);
  const float lt = sum_quads(l);
  if (q4 == 0) {
    ml[(wave * 2 + 0) * 16 + n] = m;
    ml[(wave * 2 + 1) * 16 + n] = lt;
  }
  lgkm_wait<0>();
  raw_barrier();
  float mw[4], lw[4], ms = -INFINITY, ls = 0.f;
#pragma unroll
  for (int w = 0; w < 4; w++) {
    mw[w] = ml[(w * 2 + 0) * 16 + n];
    lw[w] = ml[(w * 2 + 1) * 16 + n];
    if (lw[w] != 0.f) ms = fmaxf(ms, mw[w]);   // (0: no token of that share is visible)
  }
#pragma unroll
  for (int w = 0; w < 4; w++) ls += lw[w] != 0.f ? lw[w] * fast_exp2(mw[w] - ms) : 0.f;
  const bool use = lt != 0.f;   // (a share that scored NaN takes the whole chunk with it: ls > 0 fails)
  const float f = use ? fast_exp2(m - ms) / ls : 0.f;
  {
    char* dst = slot + n * A16_OUT_ROW + 16 * q4;
#pragma unroll
    for (int mb = 0; mb < 32; mb++) {
      f32x4 w;
#pragma unroll
      for (int e = 0; e < 4; e++) w[e] = use ? o[mb][e] * f : 0.f;
      *(f32x4*)(dst + 64 * mb) = w;
    }
  }
  if (wave == 0 && q4 == 0 && q_valid) *l_dst = ls > 0.f ? (ms + fast_log2(ls)) * LN2 : -INFINITY;
  lgkm_wait<0>();
  raw_barrier();
  __bf16* o_dst = a.lat_o + ((size_t)item * a.rows + (int64_t)b * a.R) * D_L + lane * 8;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = 4 * i + wave;
    if (r >= a.R) continue;
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; w++) {
      const f32x4* src = (const f32x4*)(smem + w * A16_TILE_BYTES + r * A16_OUT_ROW + lane * 32);
#pragma unroll
      for (int e = 0; e < 8; e++) x[e] += src[e >> 2][e & 3];
    }
    bf16x8 w8;
#pragma unroll
    for (int e = 0; e < 8; e++) w8[e] = (__bf16)x[e];
    *(bf16x8*)(o_dst + (size_t)r * D_L) = w8;
  }
}

int mfma_absorb16_attention(const Plan& p, const DecodeArgs& d, AbsorbArgs a) {
  static LdsOptIn lds;
  if (lds.ensure((const void*)absorb16_kernel, A16_LDS_BYTES) != hipSuccess) return TMLA_ERR_HIP;
  dim3 grid(p.as_chunks, p.B);
  a.order = suffix_request_order(p, d, (long long)grid.x * grid.y);
  hipLaunchKernelGGL(absorb16_kernel, grid, dim3(256), A16_LDS_BYTES, d.stream, a);
  return TMLA_OK;
}

}  // namespace tmla
