// Pieces shared by the absorb-formulation attention kernels for 32 or more query rows per
// request (paper Algorithm 1 step 6): kernel arguments, the LDS tile of 32 latent cache rows and
// the global -> LDS transfers that fill it.
#pragma once
#include <type_traits>
#include <utility>

#include "tmla_common.hpp"
#include "tmla_lds_asm.hpp"
#include "tmla_mfma.hpp"

namespace tmla {

struct AbsorbArgs {
  const __bf16* qabs;        // [rows, 576]
  const __bf16* pc;          // prefix latent [Ls, 512]  (absorb_only)
  const __bf16* pr;          // prefix rope   [Ls, 64]
  const __bf16* pool;        // [num_blocks, block_size, 576]
  const int32_t* block_table;
  const int32_t* lens;
  const int32_t* order;      // workgroup's request slot -> request, or nullptr (identity)
  __bf16* lat_o;             // [n_lat, rows, 512]
  float* lat_lse;            // [n_lat, rows]
  int Sq, H, R, Ls, ap_chunks, ap_chunk, as_chunks, as_chunk, max_blocks;
  int bs_shift;              // log2 of the tokens per cache block
  int64_t rows;
  float c;                   // sm_scale * log2(e)
};

// Division of wave-uniform numbers by one the host knows: scalar multiplications instead of the
// ~30 dependent vector instructions of an integer division (three of them in front of a
// workgroup's first transfer cost 0.4 us).  recip = min(2^32 - 1, floor(2^32 / d)): the product's
// high word is the quotient or one less, for every 32-bit numerator.
struct UniformDiv {
  uint32_t d, recip;
  void set(uint32_t div) {
    d = div > 0 ? div : 1;
    recip = d == 1 ? 0xffffffffu : (uint32_t)(0x100000000ull / d);
  }
  __device__ __forceinline__ void divide(uint32_t x, int& q, int& r) const {
    uint32_t qq = __umulhi(x, recip), rr = x - qq * d;
    if (rr >= d) { rr -= d; qq++; }
    q = (int)qq; r = (int)rr;
  }
};

// query position s of a request's query row r = s * H + h (R = S_q * H rows, S_q <= 8)
__device__ inline int query_position(int r, int H, int R) {
  int s = 0;
  for (int t = H; t < R; t += H) s += r >= t;
  return s;
}

// Work of a launch of the 64- or 128-row kernel: `pre_chunks` chunks of the latent prefix for
// `pre_groups` groups of query rows, then `suf_chunks` suffix chunks of B requests for `suf_groups`
// groups of a request's rows.  Every request attends to the whole prefix, so its groups are cut
// from the rows of all requests together (16 or 32 rows a request fill a group as well as 128),
// while a suffix belongs to one request.
struct AbsorbGrid {
  int pre_wgs;                 // pre_chunks * pre_groups
  int pre_each, pre_more;      // per XCD, and how many XCDs take one more
  int suf_units;               // suffix chunks * B
  int spread_id, spread_unit;  // suffix ids and units from which on the row groups are dealt out singly
  int rotate;                  // 7 for a batch of whole eights: an XCD takes another request of an
                               // eight with every chunk; else 0 (they go round by themselves)
  UniformDiv pre_groups, suf_groups, batch;
};
struct AbsorbUnit {
  int item, qg, b, R;   // partial slot, row group, first row / R, rows that the groups are cut from
  bool is_prefix, none;
};
// Hardware deals consecutive workgroup ids round-robin over the 8 XCDs of NUM_CU / 8 compute units,
// whatever they have left to do.  A prefix launch gives each XCD consecutive units, i.e. few chunks
// and many row groups: the chunk stays in its L2.  The row groups of one suffix chunk get ids 8
// apart: same XCD, at the same time, so the second reader of a tile finds it there.  The units of a
// suffix launch are the first chunks of all requests, then the second ones, ...: chunk by chunk
// within a request, two, four or eight of them would send every last chunk, which ragged requests
// leave short or empty, to the same XCDs (199 requests x 64 heads absorb_only over 559 + 1469 ragged
// tokens, two chunks: 129 us a step).  Of a number of
// chunks that is no multiple of 8, the last few would go to the first XCDs with all their groups;
// where that gives an XCD more rounds of workgroups than the launch needs (absorb_grid), they
// are dealt out group by group.
template <bool HAS_PREFIX>
__device__ inline AbsorbUnit absorb_unit(const AbsorbArgs& a, const AbsorbGrid& gr, int id) {
  // every argument that the way to the first transfer needs, fetched at once: left alone, the
  // compiler fetches them in four dependent rounds behind the branches (+0.4 us a launch)
  asm volatile("" ::"s"(a.lens), "s"(a.order), "s"(a.block_table), "s"(a.pool), "s"(a.qabs),
               "s"(a.ap_chunks), "s"(a.as_chunk), "s"(a.max_blocks), "s"(a.bs_shift), "s"(a.R),
               "s"(a.rows));
  AbsorbUnit u;
  if (HAS_PREFIX && id < gr.pre_wgs) {
    const int x = id & 7;
    gr.pre_groups.divide(x * gr.pre_each + min(x, gr.pre_more) + (id >> 3), u.item, u.qg);
    u.none = false;
    u.b = 0;
    u.R = (int)a.rows;
    u.is_prefix = true;
    return u;
  }
  if (HAS_PREFIX) id -= gr.pre_wgs;
  const bool single = id >= gr.spread_id;
  int sl, chunk;
  gr.suf_groups.divide(single ? id - gr.spread_id : id >> 3, sl, u.qg);
  const int j = single ? gr.spread_unit + sl : sl * 8 + (id & 7);
  u.none = j >= gr.suf_units;
  gr.batch.divide(j, chunk, u.b);
  u.b = (u.b & ~gr.rotate) | ((u.b + chunk) & gr.rotate);
  u.item = a.ap_chunks + chunk;
  if (a.order && !u.none) u.b = scalar_load_i32(a.order + u.b);
  u.R = a.R;
  u.is_prefix = false;
  return u;
}

// LDS tile of 32 tokens (38912 B).  The LDS has 64 four-byte banks; a 16-byte read is served 16
// lanes at a time -- of each half 0 .. 3, 12 .. 15 and 20 .. 27, then the others --, an 8-byte (transposing) read 32
// lanes at a time, and a group is conflict-free when its lanes cover all 64 banks once.
//   latent part: row r (token) at r * 1088, holding the 64 sixteen-byte chunks of its 512 latent
//     columns; chunk c sits in slot c ^ ((r >> 2) & 3).  The row stride is 16 banks mod 64, so
//     the transposing reads (4 rows x 64 B per 32 lanes) cover the banks exactly; the slot
//     swizzle separates rows r, r + 4, r + 8, r + 12 for the 16-byte reads of the score product
//     (16 rows, one chunk each: lane = row + 32 * chunk; the pipelined 64-row kernel, whose lanes are
//     row + 16 * chunk, permutes the swizzle).  The 64 bytes behind a row's chunks are never written by a
//     transfer (the 64-row kernel keeps its row maxima there).
//   rope part: 32 rows x 128 B behind it, chunk c of row r in slot c ^ ((r >> 1) & 7): rows of
//     equal parity share 32 banks and are separated by the swizzle.
// A tile is filled by 36 wavefront-wide 1 KiB transfers: one per latent row (the swizzle is
// uniform per row) and four for the rope parts of eight rows each.  Rows past the end of the
// chunk are filled from the last valid row: their scores are masked, so they only have to be
// finite.
constexpr int AB_ROW_BYTES = 1088;
constexpr int AB_MAIN_BYTES = 32 * AB_ROW_BYTES;   // 34816
constexpr int AB_TILE_BYTES = AB_MAIN_BYTES + 32 * 128;   // 38912
constexpr int AB_DMA_PER_WAVE = 9;                 // 8 latent rows + 1 rope group per wavefront
constexpr int AB_NSLOT = 4;                        // tiles resident in LDS (3 in flight + 1 in use)
constexpr int AB_LDS_BYTES = AB_NSLOT * AB_TILE_BYTES;   // 155648

// Per-lane byte offsets into a tile for the three read patterns (lane = n + 32 g):
//   score product, latent k-step ks < 32: row n, chunk 2 ks + g -> s_off[ks & 1] + 64 (ks >> 1)
//   score product, rope k-step 32 + k   : row n, chunk 2 k + g  -> r_off[k]
//   output product (transposing 8-byte reads; 16-lane group j = lane / 16, r = lane % 16):
//     token row 4 g + r / 4 (v_lo) or that + 8 (v_hi), latent columns 16 (j % 2) + 4 (r % 4) ..+3
//     of a 32-column block; the caller adds 16 rows per further k-step and 64 B per block.
struct TileLane {
  uint32_t s_off[2], r_off[4], v_lo, v_hi;
};
__device__ inline TileLane tile_lane(int lane) {
  const int n = lane & 31, g = lane >> 5, sw = (n >> 2) & 3;
  TileLane t;
#pragma unroll
  for (int par = 0; par < 2; par++) t.s_off[par] = n * AB_ROW_BYTES + (((2 * par + g) ^ sw) << 4);
#pragma unroll
  for (int k = 0; k < 4; k++)
    t.r_off[k] = AB_MAIN_BYTES + n * 128 + (((2 * k + g) ^ ((n >> 1) & 7)) << 4);
  const int j16 = lane >> 4, r16 = lane & 15;
  const int chunk = 2 * (j16 & 1) + ((r16 & 3) >> 1);
  const uint32_t row = (4 * g + (r16 >> 2)) * AB_ROW_BYTES + 8 * (r16 & 1);
  // rows 16 kk + 4 g + 0..3 have swizzle g, rows 8 further down g ^ 2
  t.v_lo = row + ((chunk ^ g) << 4);
  t.v_hi = row + 8 * AB_ROW_BYTES + ((chunk ^ g ^ 2) << 4);
  return t;
}
// fragment of latent k-step KS (rows = the tile's 32 tokens) for the score product
template <int KS>
__device__ inline bf16x8 tile_score_frag(uint32_t tile, const TileLane& t) {
  return lds_read_b128<64 * (KS >> 1)>(tile + t.s_off[KS & 1]);
}

// Where the 32 rows of one LDS tile come from: latent part and rope part of row i start at
// lat + i * lat_stride and rope + i * rope_stride; rows past `last` repeat row `last`.
struct RowSrc {
  const char* lat;
  const char* rope;
  int lat_stride, rope_stride, last;
  bool stream;   // rows nobody else reads (a request's own suffix): non-temporal transfers
};

// Per-lane constants of the tile transfers (see the tile layout above).
struct DmaLane {
  int wave, off[4], rope_row, rope_ch;
};
__device__ inline DmaLane dma_lane(int wave, int lane) {
  DmaLane d;
  d.wave = wave;
#pragma unroll
  for (int sw = 0; sw < 4; sw++) d.off[sw] = (lane ^ sw) << 4;
  d.rope_row = 8 * wave + (lane >> 3);
  d.rope_ch = ((lane & 7) ^ ((d.rope_row >> 1) & 7)) << 4;
  return d;
}

// K-th of the nine transfers with which one wavefront contributes to a tile: latent rows
// wave, wave + 4, ..., wave + 28 (K < 8), then the rope parts of rows 8*wave .. 8*wave+7 (K = 8).
// All row arithmetic is wave-uniform; the only per-lane terms are the swizzled lane offsets.
template <int K>
__device__ __attribute__((always_inline)) inline void issue_part(const RowSrc& s, char* dst,
                                                                 const DmaLane& d) {
  if constexpr (K < 8) {
    const int r = d.wave + 4 * K;          // (r >> 2) & 3 == K & 3
    const int rr = min(r, s.last);
    if (s.stream) dma16_stream(s.lat + (size_t)rr * s.lat_stride + d.off[K & 3], dst + r * AB_ROW_BYTES);
    else dma16(s.lat + (size_t)rr * s.lat_stride + d.off[K & 3], dst + r * AB_ROW_BYTES);
  } else {
    const int rr = min(d.rope_row, s.last);
    if (s.stream) dma16_stream(s.rope + (size_t)rr * s.rope_stride + d.rope_ch, dst + AB_MAIN_BYTES + d.wave * 1024);
    else dma16(s.rope + (size_t)rr * s.rope_stride + d.rope_ch, dst + AB_MAIN_BYTES + d.wave * 1024);
  }
}
__device__ __attribute__((always_inline)) inline void issue_all(const RowSrc& s, char* dst,
                                                                const DmaLane& d) {
  static_for<AB_DMA_PER_WAVE>([&](auto k) { issue_part<decltype(k)::value>(s, dst, d); });
}

// One launch over the latent prefix (WITH_PREFIX), the suffixes (WITH_SUFFIX) or both.
enum { WITH_PREFIX = 1, WITH_SUFFIX = 2 };
// its grid for `rows_per_wg` (64 or 128) rows a workgroup: ids to launch and workgroups among them
// that have work; false: too many
bool absorb_grid(const Plan& p, int what, int rows_per_wg, AbsorbGrid* grid, long long* ids,
                 long long* wgs);
int mfma_absorb64_attention(const Plan& p, const DecodeArgs& d, const AbsorbArgs& a, int what);
int mfma_absorb64_steps_attention(const Plan& p, const DecodeArgs& d, const AbsorbArgs& a, int what);
int mfma_absorb128_attention(const Plan& p, const DecodeArgs& d, const AbsorbArgs& a, int what);
int mfma_absorb16_attention(const Plan& p, const DecodeArgs& d, AbsorbArgs a);   // S_q * H <= 16, suffixes

}  // namespace tmla
