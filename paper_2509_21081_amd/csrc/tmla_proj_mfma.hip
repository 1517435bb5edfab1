// The two absorb projections on the matrix cores, each fused with its neighbour step:
//   * query absorption  Q_abs = Q_nope W_UK  (paper Algorithm 1 step 5), plus the copy of the
//     RoPE part, producing the 576-wide absorbed query rows the latent attention consumes;
//   * up-projection O_A = O_lat W_UV^T (step 7) fused with the LSE combine (step 8): the latent
//     split partials are projected and merged in fp32 with the 128-wide naive partials, and stored.
// Both are per-head GEMMs with the queries on the MFMA column axis (transposed products, see
// tmla_mfma.hpp), so all per-query softmax weights are per-lane scalars.
#include "tmla_common.hpp"
#include "tmla_lds_asm.hpp"
#include "tmla_mfma.hpp"

namespace tmla {

typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;

// ------------------------------------------------------------------ step 5
// grid (H, 4 latent quarters, ceil(M/128)); 4 wavefronts x 32 queries.  W_UK[h] is [128, 512]
// with the contraction index (noPE dim) as the row, i.e. k-major: a [128 x 128] slice is staged
// in LDS and read through the transposing LDS load to form the A operand (rows = latent columns).
constexpr int QA_ROW_BYTES = 320;  // 256 + 64: 16 banks on per row, so the 4 rows x 64 B of a transposing read (32 lanes) cover the 64 banks once

// Queries arrive as whole rows of 256 bytes and become fragments through LDS: fetched as fragments,
// 32 bytes from each of 32 rows an instruction, they took four times the cycles.  The RoPE parts
// are dealt out to the four quarters and requested with everything else.  Before and after: 111
// queries x 64 heads 7.7 -> 6.7 us, 256 x 64 10.8 -> 9.8, 512 x 16 7.8 -> 6.6, 256 x 128 16.8 -> 15.9.
// SMALL: up to 32 queries, which the wavefronts share, each with a quarter of the slice's columns (one
// wavefront with all of them is a longer chain): 1 x 128 6.8 -> 5.7 us, 8 x 16 4.8 -> 4.05.
// QBK: blocks of 128 queries a workgroup takes in turn with its weight slice staged once (large
// batches: the slice would otherwise be fetched again for every 128 queries).  The rows of
// the next block are requested right behind the MFMAs of the current one and arrive while its
// rows are turned around and stored.
// Rank: where the absorb pass behind it wants the requests by suffix length, the first `layers` of
// the grid's z rank them, a wavefront each, beside the others (a launch of its own takes 4.8 us).
struct RankArgs {
  const int32_t* lens;
  int32_t* order;
  int B, layers;
};
template <int QBK, bool SMALL>
__global__ void __launch_bounds__(256, QBK > 1 ? 2 : 4) qabs_kernel(const __bf16* __restrict__ q,
                                                   const __bf16* __restrict__ w_uk,
                                                   __bf16* __restrict__ qabs, int M, int H,
                                                   RankArgs rank) {
  constexpr int ST_ROW = 272;   // row of the query and store staging: 256 + 16 B, rows stay 16-byte aligned
  constexpr int MB = SMALL ? 1 : 4;
  static_assert(!SMALL || QBK == 1, "32 queries are one block");
  // 40 KiB weight slice (four workgroups a compute unit, to the byte); query and store staging: behind it
  // when the slice must survive for the next block, else the slice itself
  constexpr int WT_BYTES = 128 * QA_ROW_BYTES;
  __shared__ __attribute__((aligned(16))) char wt[WT_BYTES + (QBK > 1 ? 4 * 32 * ST_ROW : 0)];
  if ((int)blockIdx.z < rank.layers) {
    const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    rank_suffix(rank.lens, rank.B, rank.order, wg * 4 + (threadIdx.x >> 6));
    return;
  }
  const int h = blockIdx.x, lq = blockIdx.y, qs0 = (blockIdx.z - rank.layers) * QBK;
  const int nqs = (M + 127) / 128;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 31, g = lane >> 5;
  const int rr = lane >> 4, ch = lane & 15;
  const int wq = SMALL ? 0 : wave;   // this wavefront's 32 of the 128 queries
  // 32 queries as whole rows of 256 bytes (rows past the last one repeat it), and this workgroup's
  // quarter of the block's RoPE parts
  bf16x8 qr[8], rope;
  auto load_q = [&](int qsb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const int qq = min(qsb * 128 + wq * 32 + 4 * i + rr, M - 1);
      qr[i] = *(const bf16x8*)(q + ((size_t)qq * H + h) * D_QK + ch * 8);
    }
    const int qq = min(qsb * 128 + lq * 32 + (tid >> 3), M - 1);
    rope = *(const bf16x8*)(q + ((size_t)qq * H + h) * D_QK + D_N + (tid & 7) * 8);
  };
  char* mine = wt + (QBK > 1 ? WT_BYTES : 0) + wave * (32 * ST_ROW);
  bf16x8 qf[8];
  auto turn_q = [&]() __attribute__((always_inline)) {   // (each wavefront reads back what it wrote itself)
#pragma unroll
    for (int i = 0; i < 8; i++) *(bf16x8*)(mine + (4 * i + rr) * ST_ROW + ch * 16) = qr[i];
#pragma unroll
    for (int ks = 0; ks < 8; ks++) qf[ks] = *(const bf16x8*)(mine + n * ST_ROW + (16 * ks + 8 * g) * 2);
  };
  load_q(qs0);
  // stage W_UK[h][0:128][lq*128 : lq*128+128]: 128 rows x 16 chunks of 16 B
  bf16x8 wr[8];
  {
    const __bf16* src = w_uk + ((size_t)h * D_N) * D_L + lq * 128;
#pragma unroll
    for (int i = 0; i < 8; i++) wr[i] = *(const bf16x8*)(src + (size_t)(16 * i + (tid >> 4)) * D_L + (tid & 15) * 8);
  }
  // everything is requested before anything is waited for
#pragma unroll
  for (int i = 0; i < 8; i++) asm volatile("" : "+v"(qr[i]), "+v"(wr[i]));
  turn_q();
  if (QBK == 1) __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; i++) *(bf16x8*)(wt + (16 * i + (tid >> 4)) * QA_ROW_BYTES + (tid & 15) * 16) = wr[i];
  __syncthreads();
  const int j16 = lane >> 4, r16 = lane & 15;
  // transposing read: contraction row 16*ks + 8*g + 4*half + r/4, latent 32*mb + 16*(j%2) + 4*(r%4)
  const int a_off = (8 * g + (r16 >> 2)) * QA_ROW_BYTES + (16 * (j16 & 1) + 4 * (r16 & 3)) * 2 + (SMALL ? 64 * wave : 0);
  for (int it = 0; it < QBK; it++) {
    const int qsb = qs0 + it;
    if (qsb >= nqs) break;                    // workgroup-uniform
    f32x16 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; mb++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[mb][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ks++) {
#pragma unroll
      for (int mb = 0; mb < MB; mb++) {
        const char* src = wt + a_off + (16 * ks) * QA_ROW_BYTES + 64 * mb;
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src));
        const short4v hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src + 4 * QA_ROW_BYTES));
        const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        acc[mb] = mfma32(__builtin_bit_cast(bf16x8, both), qf[ks], acc[mb]);
      }
    }
    {
      const int qq = qsb * 128 + lq * 32 + (tid >> 3);   // RoPE part: verbatim copy
      if (qq < M) *(bf16x8*)(qabs + ((size_t)qq * H + h) * D_ROW + D_L + (tid & 7) * 8) = rope;
    }
    const bool more = QBK > 1 && it + 1 < QBK && qsb + 1 < nqs;
    if (more) load_q(qsb + 1);
    // Store through LDS: a lane holds 8-byte pieces of its query's row, 16 bytes apart from its
    // neighbour's; turned around in LDS, sixteen lanes write one query's 256 bytes of this latent
    // quarter in one piece.  With a single block the weight slice is free once everybody has
    // its fragments and serves as the staging buffer.
    if (QBK == 1) __syncthreads();
    char* st = SMALL ? wt : mine;
#pragma unroll
    for (int mb = 0; mb < MB; mb++)
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; e++) w[e] = (__bf16)acc[mb][4 * v4 + e];
        *(bf16x4*)(st + n * ST_ROW + (32 * (SMALL ? wave : mb) + 8 * v4 + 4 * g) * 2) = w;
      }
    // (each wavefront reads back only what it wrote itself: no barrier, but for the shared 32 rows)
    if (SMALL) __syncthreads();
#pragma unroll
    for (int i = 0; i < (SMALL ? 2 : 8); i++) {
      const int r = 4 * (SMALL ? 4 * i + wave : i) + rr;
      const bf16x8 w = *(const bf16x8*)(st + r * ST_ROW + ch * 16);
      const int qq = qsb * 128 + wq * 32 + r;
      if (qq < M) *(bf16x8*)(qabs + ((size_t)qq * H + h) * D_ROW + lq * 128 + ch * 8) = w;
    }
    if (more) turn_q();
  }
}

int mfma_query_absorb(const Plan& p, const DecodeArgs& d, bool* ranked) {
  *ranked = false;
  if (p.n_lat <= 0 || p.rows == 0) return TMLA_OK;
  const int M = p.B * p.Sq;
  const int nqs = (M + 127) / 128;
  // Four blocks of 128 queries per workgroup for large batches (measured: -13 % at 1024 queries
  // per head, nothing to gain at 256 and below), as long as the grid still covers the chip twice
  const int qbk = (nqs >= 8 && p.H * 4 * ((nqs + 3) / 4) >= 2 * NUM_CU) ? 4 : 1;
  RankArgs rank = {d.suffix_lens, (int32_t*)(d.ws + p.off_order), p.B, 0};
  *ranked = suffix_order_wanted(p);
  if (*ranked) rank.layers = (p.B + 16 * p.H - 1) / (16 * p.H);
  dim3 grid(p.H, 4, (nqs + qbk - 1) / qbk + rank.layers);
  const __bf16* q = (const __bf16*)d.q;
  const __bf16* w = (const __bf16*)d.w_uk;
  __bf16* out = (__bf16*)(d.ws + p.off_qabs);
  auto kernel = M <= 32 ? qabs_kernel<1, true> : qbk == 4 ? qabs_kernel<4, false> : qabs_kernel<1, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, d.stream, q, w, out, M, p.H, rank);
  return TMLA_OK;
}

// ------------------------------------------------------------------ steps 7 + 8
// grid (H, ceil(M/32)); the four wavefronts of a workgroup share 32 queries of one head and split
// the 512-wide contraction of the up-projection in four; their partial products are summed
// through LDS, after which wavefront w finishes value columns [32w, 32w+32): merge with the naive
// partials, normalise, store.
constexpr int FIN_MAX_LAT = 64;  // latent partials per row supported by the weight table in LDS
constexpr int MERGE_MAX_LAT = 128;   // ... by the separate merge pass (two per lane)
static_assert(2 * MAX_CHUNKS <= MERGE_MAX_LAT, "latent prefix + suffix chunks per request");

struct FinalizeArgs {
  const float* naive_o; const float* naive_lse; const __bf16* lat_o; const float* lat_lse;
  const __bf16* w_uv; __bf16* out; float* lse_out;
  int M, H, n_naive, n_lat;
  int64_t rows;
};

// The naive partials of a row for this lane (value columns 32 wave + 8 v4 + 4 g .. + 3), loaded
// ahead of the projection so that the epilogue does not pay a memory round trip of its own.
template <int NN>
struct NaivePrefetch {
  float lse[NN];
  f32x4 o[NN][4];
};
template <int NN>
__device__ inline void prefetch_naive(const FinalizeArgs& a, size_t row, int wave, int g,
                                      NaivePrefetch<NN>& pre) {
#pragma unroll
  for (int i = 0; i < NN; i++) {
    pre.lse[i] = a.naive_lse[(size_t)i * a.rows + row];
    const float* src = a.naive_o + ((size_t)i * a.rows + row) * D_V + 32 * wave + 4 * g;
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) pre.o[i][v4] = *(const f32x4*)(src + 8 * v4);
  }
}
// merge O_A (LSE l_a) with NN prefetched naive partials, normalise, store
template <int NN>
__device__ inline void finalize_tail_prefetched(const FinalizeArgs& a, size_t row, int wave, int g,
                                                float l_a, float (&oa)[16],
                                                const NaivePrefetch<NN>& pre) {
  float m2 = l_a;
#pragma unroll
  for (int i = 0; i < NN; i++) m2 = fmaxf(m2, pre.lse[i]);
  __bf16* dst = a.out + row * D_V + 32 * wave + 4 * g;
  if (m2 == -INFINITY) {
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      bf16x4 w = {0, 0, 0, 0};
      *(bf16x4*)(dst + 8 * v4) = w;
    }
    if (a.lse_out && wave == 0 && g == 0) a.lse_out[row] = -INFINITY;
    return;
  }
  const float w_a = (l_a > -INFINITY) ? __expf(l_a - m2) : 0.f;
  float z2 = w_a;
#pragma unroll
  for (int v = 0; v < 16; v++) oa[v] *= w_a;
#pragma unroll
  for (int i = 0; i < NN; i++) {
    // (a partial with LSE = -inf was never written: it is skipped, not multiplied by zero)
    if (pre.lse[i] == -INFINITY) continue;
    const float w = __expf(pre.lse[i] - m2);
    z2 += w;
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      const f32x4 x = pre.o[i][v4];
      oa[4 * v4] += w * x[0]; oa[4 * v4 + 1] += w * x[1];
      oa[4 * v4 + 2] += w * x[2]; oa[4 * v4 + 3] += w * x[3];
    }
  }
  const float inv2 = 1.f / z2;
#pragma unroll
  for (int v4 = 0; v4 < 4; v4++) {
    bf16x4 w;
#pragma unroll
    for (int e = 0; e < 4; e++) w[e] = (__bf16)(oa[4 * v4 + e] * inv2);
    *(bf16x4*)(dst + 8 * v4) = w;
  }
  if (a.lse_out && wave == 0 && g == 0) a.lse_out[row] = m2 + __logf(z2);
}

// Workgroup id -> (head, block of 32 queries).  The query blocks of a head read the same W_UV[h]:
// they get ids 8 apart and consecutive in that stride, so they run at the same time on one XCD
// (hardware deals consecutive ids round-robin over the 8 XCDs) and the weights come from HBM
// once.
template <bool SPLIT>
__device__ inline bool finalize_item(const FinalizeArgs& a, int& h, int& qb, int& vb) {
  const int nqb = (a.M + 31) / 32 * (SPLIT ? 4 : 1);
  const int id = blockIdx.x, x = id & 7, sl = id >> 3;
  qb = sl % nqb;
  h = (sl / nqb) * 8 + x;
  if constexpr (SPLIT) {
    vb = qb & 3;
    qb >>= 2;
  }
  return h < a.H;
}

constexpr int TAIL_UNROLL = 4;
// Steps shared by both finalize kernels: merge O_A (LSE l_a, this wavefront's 32 value columns
// in oa) with the naive partials, normalise, store.
__device__ inline void finalize_tail(const FinalizeArgs& a, size_t row, int wave, int g, float l_a,
                                     float (&oa)[16]) {
  // merge O_A (LSE l_a) with the naive partials; this wavefront owns value block `wave`
  // (unrolled, and without a branch around the loads, so that several are in flight)
  float m2 = l_a;
#pragma unroll 8
  for (int i = 0; i < a.n_naive; i++) m2 = fmaxf(m2, a.naive_lse[(size_t)i * a.rows + row]);
  __bf16* dst = a.out + row * D_V + 32 * wave + 4 * g;
  if (m2 == -INFINITY) {
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      bf16x4 w = {0, 0, 0, 0};
      *(bf16x4*)(dst + 8 * v4) = w;
    }
    if (a.lse_out && wave == 0 && g == 0) a.lse_out[row] = -INFINITY;
    return;
  }
  const float w_a = (l_a > -INFINITY) ? __expf(l_a - m2) : 0.f;
  float z2 = w_a;
#pragma unroll
  for (int v = 0; v < 16; v++) oa[v] *= w_a;
#pragma unroll TAIL_UNROLL
  for (int i = 0; i < a.n_naive; i++) {
    const float li = a.naive_lse[(size_t)i * a.rows + row];
    const bool use = li != -INFINITY;   // (else the partial was never written)
    const float w = use ? __expf(li - m2) : 0.f;
    z2 += w;
    const float* src = a.naive_o + ((size_t)i * a.rows + row) * D_V + 32 * wave + 4 * g;
#pragma unroll
    for (int v4 = 0; v4 < 4; v4++) {
      const f32x4 x = *(const f32x4*)(src + 8 * v4);
#pragma unroll
      for (int e = 0; e < 4; e++) oa[4 * v4 + e] += use ? w * x[e] : 0.f;
    }
  }
  const float inv2 = 1.f / z2;
#pragma unroll
  for (int v4 = 0; v4 < 4; v4++) {
    bf16x4 w;
#pragma unroll
    for (int e = 0; e < 4; e++) w[e] = (__bf16)(oa[4 * v4 + e] * inv2);
    *(bf16x4*)(dst + 8 * v4) = w;
  }
  if (a.lse_out && wave == 0 && g == 0) a.lse_out[row] = m2 + __logf(z2);
}

__global__ void __launch_bounds__(256) finalize_kernel(FinalizeArgs a) {
  __shared__ float wtab[FIN_MAX_LAT][32];    // normalised merge weight of each latent partial
  __shared__ float red[4][4][16][64];        // [wavefront][value block][acc register][lane]
  int h, qb, vb;
  if (!finalize_item<false>(a, h, qb, vb)) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 31, g = lane >> 5;
  const int qi = qb * 32 + n;
  const bool valid = qi < a.M;
  const size_t row = valid ? (size_t)qi * a.H + h : 0;

  float l_a = -INFINITY;
  float oa[16];   // this wavefront's 32 value columns of O_A after the cross-wavefront sum
#pragma unroll
  for (int v = 0; v < 16; v++) oa[v] = 0.f;
  if (a.n_lat > 0) {
    float mx = -INFINITY;
    for (int i = 0; i < a.n_lat; i++) mx = fmaxf(mx, a.lat_lse[(size_t)i * a.rows + row]);
    float z = 0.f;
    if (mx > -INFINITY)
      for (int i = 0; i < a.n_lat; i++) z += __expf(a.lat_lse[(size_t)i * a.rows + row] - mx);
    const float inv = (z > 0.f && valid) ? 1.f / z : 0.f;
    // every wavefront computes the same weights; wavefront 0 publishes them
    if (wave == 0 && g == 0)
      for (int i = 0; i < a.n_lat; i++)
        wtab[i][n] = (inv > 0.f) ? __expf(a.lat_lse[(size_t)i * a.rows + row] - mx) * inv : 0.f;
    if (z > 0.f && valid) l_a = mx + __logf(z);
    __syncthreads();

    f32x16 acc[4];
#pragma unroll
    for (int mb = 0; mb < 4; mb++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[mb][v] = 0.f;
    const __bf16* wp = a.w_uv + ((size_t)h * D_V + n) * D_L + 8 * g + 128 * wave;
    const __bf16* lp = a.lat_o + row * D_L + 8 * g + 128 * wave;
    for (int ks = 0; ks < 8; ks++) {
      float m8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      for (int i = 0; i < a.n_lat; i++) {
        const float w = wtab[i][n];
        if (w > 0.f) {
          const bf16x8 x = *(const bf16x8*)(lp + (size_t)i * a.rows * D_L + 16 * ks);
#pragma unroll
          for (int e = 0; e < 8; e++) m8[e] += w * (float)x[e];
        }
      }
      bf16x8 bfrag;
#pragma unroll
      for (int e = 0; e < 8; e++) bfrag[e] = (__bf16)m8[e];
#pragma unroll
      for (int mb = 0; mb < 4; mb++) {
        const bf16x8 afrag = *(const bf16x8*)(wp + (size_t)(32 * mb) * D_L + 16 * ks);
        acc[mb] = mfma32(afrag, bfrag, acc[mb]);
      }
    }
#pragma unroll
    for (int mb = 0; mb < 4; mb++)
#pragma unroll
      for (int v = 0; v < 16; v++) red[wave][mb][v][lane] = acc[mb][v];
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; v++)
      oa[v] = red[0][wave][v][lane] + red[1][wave][v][lane] + red[2][wave][v][lane] +
              red[3][wave][v][lane];
  }
  if (!valid) return;
  finalize_tail(a, row, wave, g, l_a, oa);
}

// Same computation for a compile-time number NL <= 4 of latent partials and so few rows that a
// workgroup takes one of the four value blocks: one per head and query block would leave compute
// units idle while each of the others fetches 128 KiB of weights.  Nothing depends on anything but
// the loads, so all of them -- partial LSEs, weight fragments, latent partials -- are issued back to
// back and the kernel pays one memory round trip instead of one per k-step; the merge weights live
// in registers.  NN > 0: the number of naive partials is NN and they are loaded up front with
// everything else (0: any number, loaded in the epilogue).
// The partials are projected one by one and merged in fp32.  Merged first, the latent row is
// rounded to bf16 once more on top of its partials, which would make a suffix that is cut only to
// fill the chip less precise than one left whole: 8 requests x 256 tokens x 16 heads, error of the
// output against fp64 2.95e-3 in one chunk, 3.33e-3 in four merged first, 2.87e-3 in four apart.
template <int NL, int NN>
__global__ void __launch_bounds__(256) finalize_few_kernel(FinalizeArgs a) {
  __shared__ float red[4][16][64];           // [wavefront][acc register][lane]
  int h, qb, vb = 0;
  if (!finalize_item<true>(a, h, qb, vb)) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n = lane & 31, g = lane >> 5;
  const int qi = qb * 32 + n;
  const bool valid = qi < a.M;
  const size_t row = valid ? (size_t)qi * a.H + h : 0;

  float ll[NL];
#pragma unroll
  for (int i = 0; i < NL; i++) ll[i] = a.lat_lse[(size_t)i * a.rows + row];
  const __bf16* wp = a.w_uv + ((size_t)h * D_V + 32 * vb + n) * D_L + 8 * g + 128 * wave;
  const __bf16* lp = a.lat_o + row * D_L + 8 * g + 128 * wave;
  bf16x8 wf[8];
#pragma unroll
  for (int ks = 0; ks < 8; ks++) wf[ks] = *(const bf16x8*)(wp + 16 * ks);
  bf16x8 x[NL][8];
#pragma unroll
  for (int i = 0; i < NL; i++)
#pragma unroll
    for (int ks = 0; ks < 8; ks++)
      x[i][ks] = *(const bf16x8*)(lp + (size_t)i * a.rows * D_L + 16 * ks);
  NaivePrefetch<(NN > 0 ? NN : 1)> pre;
  if constexpr (NN > 0) {
    prefetch_naive(a, row, vb, g, pre);
#pragma unroll
    for (int i = 0; i < NN; i++)
      asm volatile("" : "+v"(pre.lse[i]), "+v"(pre.o[i][0]), "+v"(pre.o[i][1]), "+v"(pre.o[i][2]),
                        "+v"(pre.o[i][3]));
  }

  // pin every load above this point: without it the scheduler sinks the loads next to their
  // uses to save registers, and each k-step waits for its own round trip
#pragma unroll
  for (int ks = 0; ks < 8; ks++) {
    asm volatile("" : "+v"(wf[ks]));
#pragma unroll
    for (int i = 0; i < NL; i++) asm volatile("" : "+v"(x[i][ks]));
  }

  // merge weights of the latent partials (a partial with LSE = -inf was never written)
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < NL; i++) mx = fmaxf(mx, ll[i]);
  float w[NL], z = 0.f;
#pragma unroll
  for (int i = 0; i < NL; i++) {
    w[i] = (ll[i] > -INFINITY) ? __expf(ll[i] - mx) : 0.f;
    z += w[i];
  }
  const bool any = z > 0.f && valid;
  const float inv = any ? 1.f / z : 0.f;
  const float l_a = any ? mx + __logf(z) : -INFINITY;
#pragma unroll
  for (int i = 0; i < NL; i++) w[i] *= inv;

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.f;
  if constexpr (NL > 1) {
    // every partial projected as it is and weighted afterwards: a query is one column of the MFMA,
    // so its weight is one number per lane, and a partial that was never written spoils its own
    // column only
#pragma unroll
    for (int i = 0; i < NL; i++) {
      f32x16 part;
#pragma unroll
      for (int v = 0; v < 16; v++) part[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ks++) part = mfma32(wf[ks], x[i][ks], part);
      const bool use = w[i] > 0.f;
#pragma unroll
      for (int v = 0; v < 16; v++) acc[v] += use ? w[i] * part[v] : 0.f;
    }
  } else {
    // a single partial is already the merged latent output (weight 1, or 0 if it saw nothing)
    const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 8; ks++) acc = mfma32(wf[ks], w[0] > 0.f ? x[0][ks] : zero, acc);
  }
#pragma unroll
  for (int v = 0; v < 16; v++) red[wave][v][lane] = acc[v];
  __syncthreads();
  if (wave > 0 || !valid) return;
  float oa[16];
#pragma unroll
  for (int v = 0; v < 16; v++) oa[v] = red[0][v][lane] + red[1][v][lane] + red[2][v][lane] + red[3][v][lane];
  if constexpr (NN > 0) finalize_tail_prefetched(a, row, vb, g, l_a, oa, pre);
  else finalize_tail(a, row, vb, g, l_a, oa);
}

// One to four latent partials and, as a rule, more blocks of 32 queries than half the compute units: a workgroup
// takes a run of consecutive blocks of its head, and everything comes through an LDS ring of 16 KiB
// units, up to eight under way: first W_UV[h] (eight units, whose fragments then stay in registers),
// then the partials of block after block, 32 rows x 512 B each -- half of a latent partial's columns
// or all of a naive one's.  Wavefront w owns value columns [32 w, 32 w + 32) over the whole
// contraction, so nothing is summed across wavefronts; the rows in LDS are shared by all four.
// What bounds it is the data that a compute unit takes in, and a load that fetches 32 bytes from each
// of 32 rows (MFMA fragments straight from memory) takes four times the cycles of one that fetches
// two runs of 512: the kernel that loaded fragments took 24.0 us for 256 x 64 rows of three latent
// partials (now 17.7 us), 13.0 for 111 x 64 rows of two latent and two naive ones (10.8), 13.7 for 64 x
// 128 of them (12.4), 15.6 for 512 x 16 of one and eight (14.2).  With the weights as fragments: 20.2,
// 12.8, 13.6, 18.2.  One latent partial, where the partials were streamed before, then and now: 256 x 128
// rows and two naive ones (92 MB) 20.8 and 21.4, 192 x 128 16.7 and 16.9, 400 x 64 24.8 and 16.8; one naive one,
// 320 x 128 20.4 and 20.3, 512 x 128 28.7 and 27.6, 700 x 128 52.0 and 44.1.
// Every latent partial is projected as it is and weighted afterwards: a query is one column of the
// MFMA, so its weight is one number per lane, and a partial that was never written spoils its own
// column only.  (Merged first, the row would be rounded to bf16 once more.)
//   LDS slot: row r at r * 512, its 16-byte chunk c (of 32) in place c ^ (r & 15) (a read takes
//   one chunk from each of 16 rows: the swizzle spreads them over the banks).
//   Behind the ring: the final weight of every partial, [partial][query of the run].
// vmcnt bookkeeping: a unit's four transfers are the youngest memory operations but for those of
// the units behind it, so "at most 4 x (units behind it) in flight" means it landed (stores in
// between only make the wait stricter).
constexpr int FR_UNIT = 32 * 512;
constexpr int FR_NSLOT = 9;
constexpr int FR_MAX_QBK = 8;        // a thread per query of the run computes the weights
constexpr int FR_MAX_WEIGHTS = 128;  // partials x blocks of a run
constexpr int FR_BYTES = FR_NSLOT * FR_UNIT + FR_MAX_WEIGHTS * 32 * 4;
static_assert(FR_BYTES <= 163840, "LDS of a compute unit");
constexpr int FR_MAX_HEADS = 32768;  // rows of a block within 32-bit offsets
constexpr int FR_LSE_AHEAD = 8;      // LSEs of a query held in registers (any others are read again)

__global__ void __launch_bounds__(256, 1) finalize_ring_kernel(FinalizeArgs a, int qbk) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int nqb = (a.M + 31) / 32, ngrp = (nqb + qbk - 1) / qbk;
  const int id = blockIdx.x, sl = id >> 3;
  const int qg = sl % ngrp, h = (sl / ngrp) * 8 + (id & 7);   // groups of a head: same XCD
  if (h >= a.H) return;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qb0 = qg * qbk, nblk = min(qbk, nqb - qb0);
  const int nlat2 = 2 * a.n_lat, units = nlat2 + a.n_naive, total = 8 + nblk * units;

  const uint32_t smem_base = lds_addr(smem), tab = smem_base + FR_NSLOT * FR_UNIT;

  // ---- the LSEs of this thread's query, into the table of the weights
  const int parts = a.n_lat + a.n_naive;
  const bool mine = tid < nblk * 32 && qb0 * 32 + tid < a.M;
  const size_t own_row = (size_t)(qb0 * 32 + tid) * a.H + h;
  if (mine) {
#pragma unroll 1
    for (int i = 0; i < parts; i++) {
      const float* src = i < a.n_lat ? a.lat_lse + i * (size_t)a.rows : a.naive_lse + (i - a.n_lat) * (size_t)a.rows;
      __builtin_amdgcn_global_load_lds((glb_void_ptr)(src + own_row),
                                       (lds_void_ptr)(lds_char_ptr)(smem + FR_NSLOT * FR_UNIT + (i * qbk * 32 + 64 * wave) * 4),
                                       4, 0, 0);
    }
  }

  // W_UV[h] is the ring's first eight units: all 128 rows x 128 B of each, rows 8 t ... 8 t + 7 for
  // t = wave, wave + 4, ...; row r at r * 128, chunk c (of 8) in place c ^ ((r >> 1) & 7)
#pragma unroll
  for (int j = 0; j < 8; j++)
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int r = 8 * (wave + 4 * k) + (lane >> 3);
      dma16((const char*)(a.w_uv + ((size_t)h * D_V + r) * D_L) + j * 128 + (((lane & 7) ^ ((r >> 1) & 7)) << 4),
            smem + j * FR_UNIT + (wave + 4 * k) * 1024);
    }

  // the next unit into the next ring slot: rows 2 t, 2 t + 1 for t = wave, wave + 4, ...; the rows of
  // the last block that are no query's are its last query's once more
  int iss_qb = qb0, iss_j = 0;
  uint32_t iss_at = 8 * FR_UNIT + wave * 1024, iss_row[4];
  auto block_rows = [&]() __attribute__((always_inline)) {
    const int last = a.M - 1 - iss_qb * 32;
#pragma unroll
    for (int k = 0; k < 4; k++) iss_row[k] = (uint32_t)min(2 * wave + g + 8 * k, last) * (uint32_t)a.H;
  };
  block_rows();
  const uint32_t chunk[2] = {(uint32_t)((n ^ (2 * wave + g)) << 4), (uint32_t)((n ^ (2 * wave + g + 8)) << 4)};
  auto issue = [&]() __attribute__((always_inline)) {
    const size_t row = (size_t)iss_qb * 32 * a.H + h;
    const bool lat = iss_j < nlat2;
    const char* src = lat ? (const char*)(a.lat_o + ((iss_j >> 1) * (size_t)a.rows + row) * D_L) + (iss_j & 1) * D_L
                          : (const char*)(a.naive_o + ((iss_j - nlat2) * (size_t)a.rows + row) * D_V);
    const int row_shift = lat ? 10 : 9;
#pragma unroll
    for (int k = 0; k < 4; k++)
      dma16_scalar_base<false>((iss_row[k] << row_shift) + chunk[k & 1], src, smem_base, iss_at + k * 4096);
    iss_at += FR_UNIT;
    if (iss_at >= FR_NSLOT * FR_UNIT) iss_at -= FR_NSLOT * FR_UNIT;
    if (++iss_j == units) {
      iss_j = 0;
      iss_qb++;
      block_rows();
    }
  };

  // waits for the next unit, requests the one eight behind it, returns where it is
  int slot = 0, behind = total - 1;
  auto next_unit = [&]() __attribute__((always_inline)) {
    static_assert(FR_NSLOT == 9, "cases below");
    if (behind >= 7) vm_wait<28>();
    else switch (behind) {
      case 0: vm_wait<0>(); break;
      case 1: vm_wait<4>(); break;
      case 2: vm_wait<8>(); break;
      case 3: vm_wait<12>(); break;
      case 4: vm_wait<16>(); break;
      case 5: vm_wait<20>(); break;
      default: vm_wait<24>();
    }
    raw_barrier();   // everybody's part of the unit is there; everybody is done with the one in front
    if (behind >= 8) issue();
    const uint32_t at = smem_base + slot * FR_UNIT;
    if (++slot == FR_NSLOT) slot = 0;
    behind--;
    return at;
  };
  // the A fragments of all 32 k-steps: row 32 wave + n, k = 16 ks + 8 g ..
  bf16x8 wf[32];
  static_for<8>([&](auto j_) {
    constexpr int j = decltype(j_)::value;
    const uint32_t at = next_unit() + (32 * wave + n) * 128;
#pragma unroll
    for (int q = 0; q < 4; q++) wf[4 * j + q] = lds_read_b128<0>(at + (((2 * q + g) ^ ((n >> 1) & 7)) << 4));
    lgkm_wait<0>(wf[4 * j], wf[4 * j + 1], wf[4 * j + 2], wf[4 * j + 3]);
  });
  // the weights of this thread's query in place of its LSEs: of a latent partial that was never written
  // (LSE = -inf) 0, of a naive one -1
  if (mine) {
    const uint32_t own = tab + tid * 4, step = qbk * 128;
    float l[FR_LSE_AHEAD], mx = -INFINITY, z = 0.f;
#pragma unroll
    for (int i = 0; i < FR_LSE_AHEAD; i++) l[i] = lds_read_f32(own + (i < parts ? i : 0) * step);
    lgkm_wait<0>(l[0], l[1], l[2], l[3]);
    lgkm_wait<0>(l[4], l[5], l[6], l[7]);
#pragma unroll
    for (int i = 0; i < 4; i++) mx = fmaxf(mx, i < a.n_lat ? l[i] : -INFINITY);
#pragma unroll
    for (int i = 0; i < 4; i++) z += i < a.n_lat && l[i] > -INFINITY ? __expf(l[i] - mx) : 0.f;
    const float l_a = z > 0.f ? mx + __logf(z) : -INFINITY;
    float m2 = l_a;
#pragma unroll
    for (int i = 1; i < FR_LSE_AHEAD; i++) m2 = fmaxf(m2, i >= a.n_lat && i < parts ? l[i] : -INFINITY);
    for (int i = FR_LSE_AHEAD; i < parts; i++) m2 = fmaxf(m2, lds_read_f32_now(own + i * step));
    const bool any = m2 > -INFINITY;
    const float w_a = l_a > -INFINITY ? __expf(l_a - m2) : 0.f;
    auto of = [&](float x) { return any && x != -INFINITY ? __expf(x - m2) : 0.f; };   // (NaN stays)
    float z2 = w_a;
#pragma unroll
    for (int i = 1; i < FR_LSE_AHEAD; i++) z2 += i >= a.n_lat && i < parts ? of(l[i]) : 0.f;
    for (int i = FR_LSE_AHEAD; i < parts; i++) z2 += of(lds_read_f32_now(own + i * step));
    const float inv2 = any ? 1.f / z2 : 0.f, inv = z > 0.f ? w_a / z * inv2 : 0.f;
    auto put_naive = [&](int i, float x) {
      lds_write_b32(own + i * step, any && x != -INFINITY ? of(x) * inv2 : -1.f);
    };
#pragma unroll
    for (int i = 0; i < FR_LSE_AHEAD; i++) {
      if (i < a.n_lat) lds_write_b32(own + i * step, z > 0.f && l[i] > -INFINITY ? __expf(l[i] - mx) * inv : 0.f);
      else if (i < parts) put_naive(i, l[i]);
    }
    for (int i = FR_LSE_AHEAD; i < parts; i++) put_naive(i, lds_read_f32_now(own + i * step));
    lgkm_wait<0>();
    if (a.lse_out) a.lse_out[own_row] = any ? m2 + __logf(z2) : -INFINITY;
  }

  const uint32_t x_lane = n * 512 + ((g ^ (n & 15)) << 4);
#pragma unroll 1
  for (int it = 0; it < nblk; it++) {
    const uint32_t w_lane = tab + (it * 32 + n) * 4;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; v++) acc[v] = 0.f;
#pragma unroll 1
    for (int i = 0; i < a.n_lat; i++) {
      f32x16 part;
#pragma unroll
      for (int v = 0; v < 16; v++) part[v] = 0.f;
      static_for<2>([&](auto half_) {
        constexpr int half = decltype(half_)::value;
        const uint32_t sb = next_unit();
        // fragments through a ring of eight registers, eight reads ahead
        uint32_t xa[8];
#pragma unroll
        for (int j = 0; j < 8; j++) xa[j] = (sb + x_lane) ^ (j << 5);
        bf16x8 fr[8];
        static_for<8>([&](auto j_) {
          constexpr int j = decltype(j_)::value;
          fr[j] = lds_read_b128<0>(xa[j]);
        });
        static_for<16>([&](auto ks_) {
          constexpr int ks = decltype(ks_)::value;
          constexpr int later = 15 - ks < 7 ? 15 - ks : 7;
          lgkm_wait<later>(fr[ks % 8]);
          part = mfma32(wf[16 * half + ks], fr[ks % 8], part);
          if constexpr (ks + 8 < 16) fr[ks % 8] = lds_read_b128<256>(xa[ks % 8]);
        });
      });
      const float w = lds_read_f32_now(w_lane + i * qbk * 128);
      const bool use = w > 0.f;
#pragma unroll
      for (int v = 0; v < 16; v++) acc[v] += use ? w * part[v] : 0.f;
    }
#pragma unroll 1
    for (int i = 0; i < a.n_naive; i++) {
      const uint32_t sb = next_unit() + n * 512;
      f32x4 x[4];
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) x[v4] = lds_read_f32x4(sb + (((8 * wave + 2 * v4 + g) ^ (n & 15)) << 4));
      const float w = lds_read_f32_now(w_lane + (a.n_lat + i) * qbk * 128);
      lgkm_wait<0>(x[0], x[1], x[2], x[3]);
      const bool use = !(w < 0.f);
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++)
#pragma unroll
        for (int e = 0; e < 4; e++) acc[4 * v4 + e] += use ? w * x[v4][e] : 0.f;
    }
    const int qi = (qb0 + it) * 32 + n;
    if (qi < a.M) {
      __bf16* dst = a.out + ((size_t)qi * a.H + h) * D_V + 32 * wave + 4 * g;
#pragma unroll
      for (int v4 = 0; v4 < 4; v4++) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = (__bf16)acc[4 * v4 + e];
        *(bf16x4*)(dst + 8 * v4) = o;
      }
    }
  }
}

template <int NL>
static void launch_finalize_few(const FinalizeArgs& a, dim3 grid, hipStream_t stream) {
  switch (a.n_naive) {
    case 1: hipLaunchKernelGGL((finalize_few_kernel<NL, 1>), grid, dim3(256), 0, stream, a); break;
    case 2: hipLaunchKernelGGL((finalize_few_kernel<NL, 2>), grid, dim3(256), 0, stream, a); break;
    default: hipLaunchKernelGGL((finalize_few_kernel<NL, 0>), grid, dim3(256), 0, stream, a);
  }
}

// Value of a lane whose number is wave-uniform, as a scalar.  (Fetched with __shfl, i.e. through LDS,
// the weights of one request's 66 partials took 3 us of the merge pass.)
__device__ inline float lane_value(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// More than four latent partials per row -- a small batch whose long prefix (absorb_only) or
// suffix is cut into many chunks so that the pass fills the chip -- are merged by a pass of its
// own into partial 0, after which the up-projection sees a single partial.  Merging inside the
// projection kernel walks the partials one dependent load after the other, for 32 query
// columns of which a small batch fills one or two: 53-110 us at batch 1-8 against 4-8 us here.
// One workgroup per row: the partials are dealt out to the four wavefronts (i = w, w + 4, ...),
// a wavefront reads a partial row as one contiguous KiB (lane = 16-byte chunk) eight at a time,
// the four sums meet in LDS.  Lane i holds the LSEs and the weights of partials i and i + 64 (at
// most MERGE_MAX_LAT = 128 partials).  A partial with LSE = -inf was never written and is skipped.
template <int N>
__global__ void __launch_bounds__(256) merge_latent_kernel(__bf16* lat_o, float* lat_lse,
                                                           int n_lat, int64_t rows) {
  __shared__ float part[4][64][8];
  const int64_t row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const __bf16* src = lat_o + (size_t)row * D_L + lane * 8;
  // everything that this wavefront may need is requested at once, before its weights are known
  // (N loads: 4 N partials at most), so the pass pays one memory round trip
  bf16x8 x[N];
#pragma unroll
  for (int j = 0; j < N; j++)
    if (wave + 4 * j < n_lat) x[j] = *(const bf16x8*)(src + (size_t)(wave + 4 * j) * rows * D_L);
  float li[2], e[2], wgt[2];
#pragma unroll
  for (int k = 0; k < 2; k++)
    li[k] = lane + 64 * k < n_lat ? lat_lse[(size_t)(lane + 64 * k) * rows + row] : -INFINITY;
#pragma unroll
  for (int j = 0; j < N; j++) asm volatile("" : "+v"(x[j]));
  float mx = fmaxf(li[0], li[1]);
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s));
#pragma unroll
  for (int k = 0; k < 2; k++) e[k] = mx > -INFINITY && li[k] > -INFINITY ? __expf(li[k] - mx) : 0.f;
  float z = e[0] + e[1];
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) z += __shfl_xor(z, s);
#pragma unroll
  for (int k = 0; k < 2; k++) wgt[k] = z > 0.f ? e[k] / z : 0.f;   // normalised weights
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < N; j++) {
    const int i = wave + 4 * j;
    const float w = i < n_lat ? lane_value(i < 64 ? wgt[0] : wgt[1], i & 63) : 0.f;
    if (w > 0.f) {
#pragma unroll
      for (int k = 0; k < 8; k++) acc[k] += w * (float)x[j][k];
    }
  }
#pragma unroll
  for (int k = 0; k < 8; k++) part[wave][lane][k] = acc[k];
  __syncthreads();   // every wavefront has read what it needs of partial 0 as well
  if (wave == 0) {
    bf16x8 o;
#pragma unroll
    for (int k = 0; k < 8; k++)
      o[k] = (__bf16)(part[0][lane][k] + part[1][lane][k] + part[2][lane][k] + part[3][lane][k]);
    *(bf16x8*)(lat_o + (size_t)row * D_L + lane * 8) = o;
    if (lane == 0) lat_lse[row] = z > 0.f ? mx + __logf(z) : -INFINITY;
  }
}

// The same merge and the projection in one launch, for so few rows that every one can have two
// workgroups, each for half of its value columns: a workgroup merges the row (both halves do) and
// multiplies it with 64 rows of W_UV[h], which it requests together with the partials.  Latency is
// all there is to it, so the row stays in fp32 and the products are vector arithmetic: thread 4 c + k
// takes column c and the k-th 8 of every 32 latent columns.  A head's workgroups have ids of one
// residue mod 8: same XCD.
template <int N>
__global__ void __launch_bounds__(256) merge_project_kernel(FinalizeArgs a) {
  __shared__ __attribute__((aligned(16))) float part[4][D_L];
  __shared__ __attribute__((aligned(16))) float merged[D_L];
  const int id = blockIdx.x, sl = id >> 3, groups = a.H >> 3;
  const int h = (sl % groups) * 8 + (id & 7), half = (sl / groups) & 1, qi = sl / groups >> 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = 64 * half + (tid >> 2), k4 = tid & 3;
  const size_t row = (size_t)qi * a.H + h;

  bf16x8 x[N];
  const __bf16* src = a.lat_o + row * D_L + lane * 8;
#pragma unroll
  for (int j = 0; j < N; j++)
    if (wave + 4 * j < a.n_lat) x[j] = *(const bf16x8*)(src + (size_t)(wave + 4 * j) * a.rows * D_L);
  float li[2], e[2], wgt[2];
#pragma unroll
  for (int k = 0; k < 2; k++)
    li[k] = lane + 64 * k < a.n_lat ? a.lat_lse[(size_t)(lane + 64 * k) * a.rows + row] : -INFINITY;
  bf16x8 wf[16];
  const __bf16* wp = a.w_uv + ((size_t)h * D_V + c) * D_L + 8 * k4;
#pragma unroll
  for (int j = 0; j < 16; j++) wf[j] = *(const bf16x8*)(wp + 32 * j);
  // naive partials k4, k4 + 4, ... of this thread's column (the first sixteen of a row; any others below)
  float nl[4], no[4];
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const int i = k4 + 4 * j;
    nl[j] = -INFINITY;
    no[j] = 0.f;
    if (i < a.n_naive) {
      nl[j] = a.naive_lse[(size_t)i * a.rows + row];
      no[j] = a.naive_o[((size_t)i * a.rows + row) * D_V + c];
    }
  }
#pragma unroll
  for (int j = 0; j < N; j++) asm volatile("" : "+v"(x[j]));
  float mx = fmaxf(li[0], li[1]);
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s));
#pragma unroll
  for (int k = 0; k < 2; k++) e[k] = mx > -INFINITY && li[k] > -INFINITY ? __expf(li[k] - mx) : 0.f;
  float z = e[0] + e[1];
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) z += __shfl_xor(z, s);
#pragma unroll
  for (int k = 0; k < 2; k++) wgt[k] = z > 0.f ? e[k] / z : 0.f;   // normalised weights
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int j = 0; j < N; j++) {
    const int i = wave + 4 * j;
    const float w = i < a.n_lat ? lane_value(i < 64 ? wgt[0] : wgt[1], i & 63) : 0.f;
    if (w > 0.f) {   // (a partial with LSE = -inf was never written)
#pragma unroll
      for (int k = 0; k < 8; k++) acc[k >> 2][k & 3] += w * (float)x[j][k];
    }
  }
  *(f32x4*)&part[wave][lane * 8] = acc[0];
  *(f32x4*)&part[wave][lane * 8 + 4] = acc[1];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; k++) {
    const int col = tid + 256 * k;
    merged[col] = part[0][col] + part[1][col] + part[2][col] + part[3][col];
  }
  __syncthreads();
  float oa = 0.f;
#pragma unroll
  for (int j = 0; j < 16; j++) {
    const f32x4 m0 = *(const f32x4*)&merged[32 * j + 8 * k4], m1 = *(const f32x4*)&merged[32 * j + 8 * k4 + 4];
#pragma unroll
    for (int k = 0; k < 4; k++) oa += (float)wf[j][k] * m0[k] + (float)wf[j][4 + k] * m1[k];
  }
  auto sum4 = [](float v) {
    v += __shfl_xor(v, 1);
    return v + __shfl_xor(v, 2);
  };
  oa = sum4(oa);

  // ---- combine with the naive partials (a NaN among their LSEs stays one)
  const float l_a = z > 0.f ? mx + __logf(z) : -INFINITY;
  float m2 = l_a;
#pragma unroll
  for (int j = 0; j < 4; j++) m2 = fmaxf(m2, nl[j]);
  for (int i = 16 + k4; i < a.n_naive; i += 4) m2 = fmaxf(m2, a.naive_lse[(size_t)i * a.rows + row]);
  m2 = fmaxf(m2, __shfl_xor(m2, 1));
  m2 = fmaxf(m2, __shfl_xor(m2, 2));
  float o2 = 0.f, z2 = 0.f;
  auto add = [&](float l, float v) {
    if (l == -INFINITY) return;
    const float w = __expf(l - m2);
    z2 += w;
    o2 += w * v;
  };
#pragma unroll
  for (int j = 0; j < 4; j++) add(nl[j], no[j]);
  for (int i = 16 + k4; i < a.n_naive; i += 4)
    add(a.naive_lse[(size_t)i * a.rows + row], a.naive_o[((size_t)i * a.rows + row) * D_V + c]);
  const float w_a = l_a > -INFINITY ? __expf(l_a - m2) : 0.f;
  z2 = sum4(z2) + w_a;
  o2 = sum4(o2) + w_a * oa;
  if (k4 == 0) {
    const bool any = m2 > -INFINITY;
    a.out[row * D_V + c] = (__bf16)(any ? o2 / z2 : 0.f);
    if (a.lse_out && half == 0 && tid == 0) a.lse_out[row] = any ? m2 + __logf(z2) : -INFINITY;
  }
}
// Where it pays: its time goes up with the rows, that of the others with the latent partials, with a third
// naive one (no longer requested up front there) and with a second round of workgroups (blocks > 64).
// Steps with this kernel less those without, 16 to 64 heads / 128, none to two naive partials:
//   one latent partial, 128 rows 0.0 ... +0.6 / -1.4 ... -0.5 us, 256 +0.5 ... +1.3 / -0.7 ... +0.3
//   two, 128 rows -0.5 ... 0.0 / -1.8 ... -1.5, 256 -0.2 ... +0.8 / -1.2 ... -0.6, 384 +0.3 ... +1.0 / -0.4 ... +0.2
//   three, 256 rows -1.1 ... +0.4 / -1.9 ... -1.2, 384 -0.8 ... +0.1 / -1.4 ... -0.5, 512 -0.7 ... +1.8 / -0.4 ... +0.2
//   four, 384 rows -1.7 ... -0.8 / -2.2 ... -1.5, 512 -1.8 ... +1.1 / -1.2 ... -0.7
// and with four to sixteen naive ones: one, 256 rows -2.1 ... -0.3, 384 -1.4 ... +0.2; two, 384 -2.1 ... -0.6.
// More than four need the merge pass without it: 16 rows 20.6 / 18.8 us a step, 128 rows 27.4 / 24.8, 384 30.0
// / 28.8, 512 30.6 / 30.3, 768 36.4 / 36.7.
static bool merge_project_pays(const FinalizeArgs& a, long long blocks) {
  const int ahead = 2 * a.n_lat + (a.n_naive > 2 ? 4 : 0) +
                    (blocks > NUM_CU / 4 ? 3 + (a.n_naive == 2 ? 1 : 0) : 0);
  return a.n_lat >= 1 && a.rows <= 64 * std::min(ahead - 2, 8);
}

int mfma_finalize(const Plan& p, const DecodeArgs& d) {
  if (p.rows == 0) return TMLA_OK;
  const bool merge_inside = (debug_flags() & 0x10000) != 0;   // debug: no separate merge pass
  if (p.n_lat > (merge_inside ? FIN_MAX_LAT : MERGE_MAX_LAT)) return TMLA_ERR_UNSUPPORTED;
  FinalizeArgs a;
  a.naive_o = (const float*)(d.ws + p.off_naive_o);
  a.naive_lse = (const float*)(d.ws + p.off_naive_lse);
  a.lat_o = (const __bf16*)(d.ws + p.off_lat_o);
  a.lat_lse = (const float*)(d.ws + p.off_lat_lse);
  a.w_uv = (const __bf16*)d.w_uv;
  a.out = (__bf16*)d.out;
  a.lse_out = d.lse_out;
  a.M = p.B * p.Sq; a.H = p.H; a.n_naive = p.n_naive; a.n_lat = p.n_lat; a.rows = p.rows;
  const int heads8 = (p.H + 7) / 8 * 8, nqb = (a.M + 31) / 32;
  const long long blocks = (long long)heads8 * nqb;   // of 32 queries
  if (!merge_inside && merge_project_pays(a, blocks)) {
    auto merge = a.n_lat <= 4 ? merge_project_kernel<1> : a.n_lat <= 16 ? merge_project_kernel<4> : a.n_lat <= 32 ? merge_project_kernel<8>
                 : a.n_lat <= 64 ? merge_project_kernel<16> : merge_project_kernel<32>;
    hipLaunchKernelGGL(merge, dim3((unsigned)(2 * p.rows)), dim3(256), 0, d.stream, a);
    return TMLA_OK;
  }
  if (a.n_lat > 4 && !merge_inside) {
    auto merge = a.n_lat <= 16 ? merge_latent_kernel<4> : a.n_lat <= 32 ? merge_latent_kernel<8>
                 : a.n_lat <= 64 ? merge_latent_kernel<16> : merge_latent_kernel<32>;
    hipLaunchKernelGGL(merge, dim3((unsigned)p.rows), dim3(256), 0, d.stream,
                       (__bf16*)(d.ws + p.off_lat_o), (float*)(d.ws + p.off_lat_lse), a.n_lat,
                       (int64_t)p.rows);
    a.n_lat = 1;
  }
  const int parts = a.n_lat + a.n_naive;
  // Up to half a workgroup per compute unit the value blocks are dealt out, unless their rows make it more
  // work to read all latent partials four times than the ring has with half of the units.  Steps with the
  // ring less those without, 10 to 256 queries x 16 to 128 heads, two / three / four latent partials and up
  // to six naive ones: 4096 rows -2.2 ... +0.1, -3.6 ... -0.9, -4.6 ... -2.9 us, 3200 rows -2.0 ... +0.6, -3.4
  // ... -0.2, -4.7 ... -1.4; 2048 rows (128 heads x 16) +0.3 ... +1.2, 0.0 ... +1.0, -0.5 ... +0.2; one: -1.2 ... +1.6
  // anywhere.  Eight to twelve naive ones and 3200 rows or more: -0.8 ... +1.7, -1.8 ... +1.0, -2.9 ... -0.7.
  const bool many_rows = p.rows > 3072 && a.n_lat >= 2 && (a.n_naive <= 6 || a.n_lat == 4);
  const bool split = blocks <= NUM_CU / 2 && !many_rows;
  if (a.n_lat >= 1 && a.n_lat <= 4 && !split && parts <= FR_MAX_WEIGHTS && p.H <= FR_MAX_HEADS) {
    // runs as short as one round of workgroups allows (every one takes in 128 KiB of weights); more
    // rounds than one as even as can be (2100 queries x 64 heads, runs of eight and of six: 76.6, 69.6 us)
    auto ceil_div = [](int x, int y) { return (x + y - 1) / y; };
    const int per_head = std::max(1, NUM_CU / heads8), one_round = ceil_div(nqb, per_head);
    const int rounds = ceil_div(one_round, std::min(FR_MAX_QBK, FR_MAX_WEIGHTS / parts)), qbk = ceil_div(one_round, rounds);
    static LdsOptIn lds;
    if (lds.ensure((const void*)finalize_ring_kernel, FR_BYTES) != hipSuccess) return TMLA_ERR_HIP;
    hipLaunchKernelGGL(finalize_ring_kernel, dim3(heads8 * ((nqb + qbk - 1) / qbk)), dim3(256), FR_BYTES, d.stream, a,
                       qbk);
    return TMLA_OK;
  }
  const dim3 grid((unsigned)blocks), grid4((unsigned)blocks * 4);
  switch (split ? a.n_lat : 0) {
    case 1: launch_finalize_few<1>(a, grid4, d.stream); break;
    case 2: launch_finalize_few<2>(a, grid4, d.stream); break;
    case 3: launch_finalize_few<3>(a, grid4, d.stream); break;
    case 4: launch_finalize_few<4>(a, grid4, d.stream); break;
    default: hipLaunchKernelGGL(finalize_kernel, grid, dim3(256), 0, d.stream, a);
  }
  return TMLA_OK;
}

}  // namespace tmla
