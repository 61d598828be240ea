// Block pooling (Section 5.1) and aggregated query-key block scores (Eq. 2).
//
// pool:  qbar_i = b^-1 sum_r q~_{i,r}, kbar_j likewise; the final partial block
//        is zero-padded and still divided by the nominal b.  One work-group per
//        block streams its b x D bf16 tile once with 16-byte loads (HBM-bound;
//        algorithmic bytes = 2*D per token read + 4*D + 4 per block written).
//        The mean is written split for the fp16 matrix cores (launch.h):
//        2^e (hi + lo) with e the row's power-of-two scale.
// score: S_ij = tau * qbar_i . kbar_j for selectable j, on fp16 MFMA with
//        fp32 accumulation as hi.hi + hi.lo + lo.hi: the dropped lo.lo term
//        and the split leave a relative error near 2^-21 of sum |q k|, the
//        level of an fp32 dot product; forced key blocks are neither pooled
//        nor scored (Section 5.2), their S columns are left untouched.
#include "device_common.h"

namespace sparstar {

// ---------------------------------------------------------------------------
// pool: grid = BH*n_q + BH*n_k work-groups (query blocks first), 256 threads.
// Thread t owns the 16-byte column chunk (t % CH) of rows g, g + RG, ... with
// g = t / CH, CH = D/8 chunks per row and RG = 256/CH row groups.
// ---------------------------------------------------------------------------
template <int D, int BLK>
__global__ __launch_bounds__(256) void pool_kernel(PoolArgs a) {
  constexpr int CH = D / 8;
  constexpr int RG = 256 / CH;
  constexpr int RPT = BLK / RG;
  __shared__ float red[RG][D + 1];
  __shared__ float wmax[4];

  const int64_t wg = blockIdx.x;
  const int64_t nqb = (int64_t)a.bh * a.n_q;
  const bool is_q = wg < nqb;
  const int64_t w = is_q ? wg : wg - nqb;
  const int nb = is_q ? a.n_q : a.n_k;
  const int64_t bh = w / nb;
  const int blk = (int)(w % nb);
  if (!is_q && keep_block(a.keep, blk)) return;  // uniform over the work-group

  const int64_t len = is_q ? a.lq : a.lk;
  const uint16_t* src = (is_q ? a.q : a.k) + (bh * len + (int64_t)blk * BLK) * D;
  const int t = threadIdx.x, c = t % CH, g = t / CH;
  const int64_t rows_left = len - (int64_t)blk * BLK;

  // all loads in flight at once (rows past the end re-read the last row, then
  // count as zeros); Q and K are read once here, so the loads are non-temporal
  // and do not displace what the caches hold
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  uint4 v[RPT];
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int row = g + r * RG;
    const int64_t rr = row < rows_left ? row : rows_left - 1;
    const u32x4 t4 = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + rr * D + c * 8));
    v[r] = make_uint4(t4[0], t4[1], t4[2], t4[3]);
  }
#pragma unroll
  for (int r = 0; r < RPT; ++r)
    if (g + r * RG >= rows_left) v[r] = make_uint4(0, 0, 0, 0);
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const uint32_t w4[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += bf16_lo(w4[e]);
      acc[2 * e + 1] += bf16_hi(w4[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[g][c * 8 + e] = acc[e];
  __syncthreads();
  float x = 0.f;  // element t of the block mean
  if (t < D) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < RG; ++r) s += red[r][t];
    x = s * (1.0f / BLK);
  }
  // the row's largest magnitude (a wave maximum, then over the four waves)
  // fixes its scale 2^e: |x| 2^-e < 2^14, inside fp16's range
  float m = fabsf(x);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  if (t % 64 == 0) wmax[t / 64] = m;
  __syncthreads();
  m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  const int ex = (m > 0.f && m <= 3.402823466e38f) ? __builtin_amdgcn_frexp_expf(m) - 14 : 0;
  const int64_t row = bh * nb + blk;
  if (t < D) {
    const float xs = __builtin_amdgcn_ldexpf(x, -ex);
    const _Float16 hi = (_Float16)xs;
    const _Float16 lo = (_Float16)(xs - (float)hi);  // the difference is exact in fp32
    uint16_t* dst = (is_q ? a.q_bar : a.k_bar) + row * (2 * D);
    dst[t] = __builtin_bit_cast(uint16_t, hi);
    dst[D + t] = __builtin_bit_cast(uint16_t, lo);
  }
  if (t == 0) (is_q ? a.q_exp : a.k_exp)[row] = ex;
}

// ---------------------------------------------------------------------------
// score: one work-group per (bh, 64 query blocks, `run` consecutive tiles of 64
// key blocks), four waves, each a 32 x 32 sub-tile of every tile on
// v_mfma_f32_32x32x16_f16.  A wave keeps its 32 query rows' operands (all of D,
// hi and lo) in registers, loaded from memory once; a key tile is staged whole
// in LDS while the next one's loads are in flight.
//
// LDS rows hold a pooled row's D hi then D lo values, padded by 16 bytes: 16
// consecutive rows read at one 16-byte offset then fall on 16 disjoint groups
// of four banks.
//
// MFMA operands (lane l, h = l / 32): A[m][k] = qbar[m = l % 32][d],
// B[k][n] = kbar[n = l % 32][d], k = 8 h + i over the lane's 8 fp16 values at
// d = 16 s + 8 h + i of k-step s.  C[m][n] sits at accumulator a with
// n = l % 32, m = 8 (a / 4) + 4 h + (a % 4).  Rows past the end of either
// operand repeat its last one: they reach only elements that are not stored.
//
// 24 heads, 1,125 x 2,259 blocks: 81 us, with S written at 3.0 TB/s (50 us at the
// copy rate; the matrix instructions alone are 22).  One tile per work-group with
// both operands read from LDS took 93: twice the LDS reads per product and no
// load in flight under them.  Operands read straight from memory in MFMA order
// (32-byte pieces of 32 rows) instead of through LDS: 91.
// ---------------------------------------------------------------------------
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int ST = 64;  // tile edge (query blocks and key blocks)

template <int D>
__global__ __launch_bounds__(256) void score_kernel(ScoreArgs a, int run) {
  constexpr int RB = 4 * D + 16;     // padded LDS row (bytes)
  constexpr int NP = D / 32;         // 16-byte pieces of a row per loading thread
  constexpr int NS = D / 16;         // k-steps
  __shared__ __attribute__((aligned(16))) unsigned char ts[ST * RB];
  __shared__ __attribute__((aligned(16))) int qe[ST];
  const int tiles_i = (a.n_q + ST - 1) / ST;
  const int tiles_j = (a.n_k + ST - 1) / ST;
  const int runs = (tiles_j + run - 1) / run;
  // consecutive tiles (one head's, key tiles fastest) on the same XCD, whose
  // L2 then holds that head's pooled blocks
  int64_t wg = xcd_linear(blockIdx.x, (int64_t)gridDim.x);
  const int tj0 = (int)(wg % runs) * run;
  const int tj1 = tj0 + run < tiles_j ? tj0 + run : tiles_j;
  wg /= runs;
  const int ti = (int)(wg % tiles_i);
  const int64_t bh = wg / tiles_i;
  const int i0 = ti * ST;

  const int t = threadIdx.x;
  const int wave = t / 64, lane = t % 64, l32 = lane % 32, h = lane / 32;
  const int wq = wave / 2, wk = wave % 2;  // the wave's 32 x 32 sub-tile

  // loader: eight threads read 128 contiguous bytes of a row; thread t has
  // pieces t % 8 + 8 p of rows t / 8 and t / 8 + 32, p turned by one in odd rows
  // so that a pair of rows is written to different banks
  const int lr = t / 8, odd = lr % 2;
  u32x4 v[2][NP];
  auto load = [&](const uint16_t* base, int r0, int n) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int i = r0 + lr + 32 * r < n ? r0 + lr + 32 * r : n - 1;
      const uint16_t* row = base + (int64_t)i * (2 * D) + 8 * (t % 8);
#pragma unroll
      for (int p = 0; p < NP; ++p) v[r][p] = *reinterpret_cast<const u32x4*>(row + 64 * (p ^ odd));
    }
  };
  auto stage = [&] {
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int p = 0; p < NP; ++p)
        *reinterpret_cast<u32x4*>(ts + (lr + 32 * r) * RB + 16 * (t % 8) + 128 * (p ^ odd)) = v[r][p];
  };
  const uint16_t* const kb = a.k_bar + bh * a.n_k * (2 * D);
  const int32_t* const kx = a.k_exp + bh * a.n_k;
  auto key_exp = [&](int tj) {
    const int j = tj * ST + wk * 32 + l32;
    return kx[j < a.n_k ? j : a.n_k - 1];
  };

  load(a.q_bar + bh * a.n_q * (2 * D), i0, a.n_q);
  if (t < ST) qe[t] = a.q_exp[bh * a.n_q + (i0 + t < a.n_q ? i0 + t : a.n_q - 1)];
  stage();
  load(kb, tj0 * ST, a.n_k);
  int ek = key_exp(tj0);
  __syncthreads();
  const unsigned char* const qr = ts + (wq * 32 + l32) * RB + 16 * h;
  f16x8 ah[NS], al[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    ah[s] = *reinterpret_cast<const f16x8*>(qr + 32 * s);
    al[s] = *reinterpret_cast<const f16x8*>(qr + 2 * D + 32 * s);
  }

  const unsigned char* const kr = ts + (wk * 32 + l32) * RB + 16 * h;
  const int irow = i0 + wq * 32 + 4 * h;  // the lane's first row of S
  float* const sbase = a.s + (bh * a.n_q + irow) * a.s_stride;
  for (int tj = tj0; tj < tj1; ++tj) {
    __syncthreads();  // the previous tile's reads are done
    stage();
    const int ej = ek;
    __syncthreads();
    if (tj + 1 < tj1) {
      load(kb, (tj + 1) * ST, a.n_k);
      ek = key_exp(tj + 1);
    }

    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const f16x8 bh_ = *reinterpret_cast<const f16x8*>(kr + 32 * s);
      const f16x8 bl = *reinterpret_cast<const f16x8*>(kr + 2 * D + 32 * s);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[s], bh_, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[s], bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[s], bh_, acc, 0, 0, 0);
    }

    const int j = tj * ST + wk * 32 + l32;
    if (j < a.n_k && !keep_block(a.keep, j)) {
      float* const scol = sbase + j;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const u32x4 eq = *reinterpret_cast<const u32x4*>(qe + wq * 32 + 8 * g + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (irow + 8 * g + e < a.n_q)
            scol[(int64_t)(8 * g + e) * a.s_stride] = a.tau * __builtin_amdgcn_ldexpf(acc[4 * g + e], (int)eq[e] + ej);
      }
    }
  }
}

hipError_t launch_pool(const PoolArgs& a, int d, int block, hipStream_t stream) {
  const int64_t grid = (int64_t)a.bh * (a.n_q + a.n_k);
  if (grid == 0) return hipSuccess;
  if (d == 128 && block == 64) pool_kernel<128, 64><<<grid, 256, 0, stream>>>(a);
  else if (d == 128 && block == 128) pool_kernel<128, 128><<<grid, 256, 0, stream>>>(a);
  else if (d == 64 && block == 64) pool_kernel<64, 64><<<grid, 256, 0, stream>>>(a);
  else if (d == 64 && block == 128) pool_kernel<64, 128><<<grid, 256, 0, stream>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// Key tiles per work-group.  A run shares one load of the query operands: 97 us at
// run 1, 85 at 2, 82 at 3, 80 at 4, 82 at 6 (24 heads, 1,125 x 2,259 blocks).  It is
// cut so that at least kScoreGroups work-groups remain (three fit a CU).
constexpr int kScoreRun = 4;
constexpr int64_t kScoreGroups = 2048;

hipError_t launch_score(const ScoreArgs& a, int d, hipStream_t stream) {
  const int64_t rows = (int64_t)a.bh * ((a.n_q + ST - 1) / ST);
  const int64_t tiles_j = (a.n_k + ST - 1) / ST;
  if (rows == 0 || tiles_j == 0) return hipSuccess;
  const int64_t fill = rows * tiles_j / kScoreGroups;
  const int run = (int)(fill < 1 ? 1 : fill > kScoreRun ? kScoreRun : fill);
  const int64_t grid = rows * ((tiles_j + run - 1) / run);
  if (d == 128) score_kernel<128><<<grid, 256, 0, stream>>>(a, run);
  else if (d == 64) score_kernel<64><<<grid, 256, 0, stream>>>(a, run);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace sparstar
