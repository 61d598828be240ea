// Retained attention mass (Section 4, Analysis): the share of each query's
// dense softmax mass that a block selection keeps, and the token-wise upper
// bound -- the largest share any equally many single keys can hold.
//
//   mass_kernel          mass_t = exp(lse_sel_t - lse_all_t), elementwise.
//   topk_scores_kernel   logits s_t,u = scale * q_t . k_u in fp32 for a few
//                        sampled query rows of a head against every key, on
//                        v_mfma_f32_16x16x32_bf16 (exact products, fp32
//                        accumulation): one work-group per (head, 256-key
//                        chunk), K streamed once.
//   topk_mass_kernel     per (head, sampled row): the n-th largest logit on
//                        order-preserving keys, and the sum over the top n of
//                        exp(s - lse_all), in one pass over the row (below).
#include "device_common.h"

namespace sparstar {

__global__ __launch_bounds__(256) void mass_kernel(const float* lse_sel, const float* lse_all, int64_t n,
                                                   float* mass) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float a = lse_sel[i];
    mass[i] = a == -INFINITY ? 0.f : expf(a - lse_all[i]);
  }
}

// Bound by the stream of K (2 D bytes per key; the logits written are 4 bytes per
// key and sampled row).  Each wave takes 16 keys at a time: A = K (lane l: key
// l % 16, d = 32 s + 8 (l / 16) + i), B = the sampled rows of Q (lane l: row
// l % 16, zeros past n_rows), and C leaves lane l four consecutive keys
// 4 (l / 16) + r of row l % 16.  Four such tiles' loads are in flight at once.
// 8 rows of 24 heads against 144,512 keys, D = 128 (888 MB of K read, 111 MB
// written): 168 us, 5.9 TB/s; with the products on the VALU, each lane reading a
// whole key row, 217 us.  Chunks of 512 and 1,024 keys 171 and 199 us;
// non-temporal loads 215 (a load takes half a 128-byte line, and the next load
// needs the other half).
template <int D>
__global__ __launch_bounds__(256) void topk_scores_kernel(TopkArgs a) {
  constexpr int CHUNK = 256;  // keys per work-group
  constexpr int KS = D / 32;   // k-steps
  constexpr int TU = 4;        // 16-key tiles in flight
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const int64_t bh = blockIdx.y;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int n16 = lane % 16, g = lane / 16;
  const int64_t key0 = (int64_t)blockIdx.x * CHUNK + wave * (CHUNK / 4);
  bf16x8 qf[KS];
  {
    const bool ok = n16 < a.n_rows;
    int64_t row = a.rows[0];
#pragma unroll
    for (int r = 1; r < kTopkMaxRows; ++r) row = ok && r == n16 ? a.rows[r] : row;
    const uint16_t* qp = a.q + (bh * a.lq + row) * D + 8 * g;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const uint4 u = *reinterpret_cast<const uint4*>(qp + 32 * s);
      qf[s] = __builtin_bit_cast(bf16x8, make_uint4(ok ? u.x : 0u, ok ? u.y : 0u, ok ? u.z : 0u, ok ? u.w : 0u));
    }
  }
  const uint16_t* const kb = a.k + bh * a.lk * D + 8 * g;
  float* const out = a.scores + (bh * a.n_rows + n16) * a.lk;
  const bool wide = a.lk % 4 == 0 && (reinterpret_cast<uintptr_t>(a.scores) & 15u) == 0;  // 16-byte stores
  for (int m = 0; m < CHUNK / 4; m += 16 * TU) {
    if (key0 + m >= a.lk) break;  // wave-uniform
    u32x4 kf[TU][KS];
#pragma unroll
    for (int t = 0; t < TU; ++t) {
      const int64_t u = key0 + m + 16 * t + n16;
      const uint16_t* kp = kb + (u < a.lk ? u : a.lk - 1) * D;
#pragma unroll
      for (int s = 0; s < KS; ++s)
        kf[t][s] = *reinterpret_cast<const u32x4*>(kp + 32 * s);
    }
#pragma unroll
    for (int t = 0; t < TU; ++t) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t][s]), qf[s], acc, 0, 0, 0);
      const int64_t u = key0 + m + 16 * t + 4 * g;
      if (n16 < a.n_rows) {
        if (wide && u < a.lk) {
          *reinterpret_cast<float4*>(out + u) =
              make_float4(acc[0] * a.scale, acc[1] * a.scale, acc[2] * a.scale, acc[3] * a.scale);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (u + r < a.lk) out[u + r] = acc[r] * a.scale;
        }
      }
    }
  }
}

// fp32 -> uint32 with the same order (-0 folded onto +0)
__device__ __forceinline__ uint32_t order_key(float x) {
  uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kTopkSamples = 512;
constexpr int kTopkCand = 32768;  // candidate keys held in LDS (128 KB)

// The digit of the want-th largest key in a 256-bin histogram, found by one
// wave: lane L owns bins 4 L .. 4 L + 3.  above: keys already known to be larger
// than every binned one.  Writes (digit, keys above the digit's bin) to sel.
__device__ __forceinline__ void find_digit(const uint32_t* hist, uint32_t above, uint32_t want, int lane,
                                           uint32_t* sel) {
  uint32_t c[4], own = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    c[e] = hist[4 * lane + e];
    own += c[e];
  }
  uint32_t suffix = own;  // sum over lanes >= lane
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_down(suffix, off, 64);
    if (lane + off < 64) suffix += o;
  }
  uint32_t up = above + suffix - own;  // keys above this lane's bins
#pragma unroll
  for (int e = 3; e >= 0; --e) {
    if (up < want && up + c[e] >= want) {
      sel[0] = (uint32_t)(4 * lane + e);
      sel[1] = up;
    }
    up += c[e];
  }
}

// One work-group per row.  512 evenly spaced keys of the row are ranked against
// each other, and two of them, about 4 standard deviations of the binomial
// count either side of the expected rank of the n-th largest key, bracket it.
// One pass over the row then counts the keys above the bracket and collects those
// inside it (a sixth of the row or so) in LDS, where a radix select finds the
// n-th largest; a second pass, in the row's order, sums exp(s - lse) over the
// keys above it.  A row of up to 32,768 keys goes to LDS as it is.  If the
// bracket missed or overflows, the radix select runs from memory: with many equal
// logits, and in long rows, since the bracket holds about 16% of the row where a
// quarter of it is wanted and 18% where half is, which pass 32,768 keys at some
// 205,000 and 178,000 keys (24 heads, 8 rows, a quarter wanted: 292 us in all
// at 144,512 keys, 735 at 205,000; histograms over the whole row 1,705).
// Bound by one CU's work per row (192 rows for 256 CUs, 144,512 keys each): two
// passes of key forming, compaction and expf, and the LDS steps between them:
// 110 us (loads in flight do not matter, 8 or 24 per lane); radix select in four passes of LDS
// histograms over the row, 256 threads a row, 965 us.
//
// Short rows take instances with room for just the row, so that a CU holds eight
// (2,048 keys) or four (8,192): the large instance fills a CU's LDS.  All of them
// add a whole row up in the same order.
template <int CAND, int NT>
__global__ __launch_bounds__(NT) void topk_mass_kernel(TopkArgs a) {
  constexpr bool WHOLE = CAND < kTopkCand;  // for rows of up to CAND keys only
  constexpr int SAMP = WHOLE ? 1 : kTopkSamples;
  __shared__ uint32_t cand[CAND];
  __shared__ uint32_t samp[SAMP], rank[SAMP], hist[256];
  __shared__ uint32_t sel[2];        // chosen digit, count of keys above it
  __shared__ uint32_t bracket[2];    // the lower and the upper key
  __shared__ uint32_t n_above, n_cand;
  __shared__ float part[NT];
  const int64_t row = blockIdx.x;  // bh * n_rows + r
  const int64_t bh = row / a.n_rows;
  const int r = (int)(row % a.n_rows);
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const float* s = a.scores + row * a.lk;
  int64_t want64 = a.n_tokens[row];
  want64 = want64 < 0 ? 0 : (want64 > a.lk ? a.lk : want64);
  const uint32_t want = (uint32_t)want64, lk = (uint32_t)a.lk;
  const float lse = a.lse_all[bh * a.lq + a.rows[r]];
  if (want == 0) {  // uniform
    if (tid == 0) a.mass[row] = 0.f;
    return;
  }
  // ---- the bracket [lo, hi) of keys (hi = 0: no upper end)
  uint32_t lo = 0, hi = 0;
  const bool whole = WHOLE || lk <= (uint32_t)CAND;  // the row as it is
  if (!whole) {
    if (tid < kTopkSamples) {
      samp[tid] = order_key(s[((2 * (uint64_t)tid + 1) * lk) / (2 * kTopkSamples)]);
      rank[tid] = 0;
    }
    if (tid < 2) bracket[tid] = 0;
    __syncthreads();
    {
      // samples larger than sample i (equal ones in index order), half of the
      // samples per thread
      constexpr int kShare = kTopkSamples * kTopkSamples / NT;  // samples per thread
      const int i = tid % kTopkSamples, q0 = tid / kTopkSamples * kShare;
      const uint32_t own = samp[i];
      uint32_t n = 0;
      for (int j = q0; j < q0 + kShare; ++j) {
        const uint32_t o = samp[j];
        n += (o > own || (o == own && j < i)) ? 1u : 0u;
      }
      atomicAdd(&rank[i], n);
    }
    __syncthreads();
    const float p = (float)want / (float)lk, mid = p * kTopkSamples;
    const int margin = (int)(4.f * sqrtf(mid * (1.f - p))) + 2;
    const int r_hi = (int)mid - margin, r_lo = (int)mid + margin;  // ranks of the bracket's ends
    if (tid < kTopkSamples) {
      if ((int)rank[tid] == r_lo) bracket[0] = samp[tid];
      if ((int)rank[tid] == r_hi) bracket[1] = samp[tid];
    }
    __syncthreads();
    lo = bracket[0];  // 0 past the last sample
    hi = bracket[1];  // 0 before the first one
  }
  if (tid == 0) {
    n_above = 0;
    n_cand = 0;
  }
  __syncthreads();

  // ---- one pass over the row
  constexpr int U = 16;
  uint32_t above_t = 0;
  for (uint32_t base = 0; base < lk; base += U * NT) {
    uint32_t key[U], n_in = 0;
    uint64_t mask[U];
    float x[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const uint32_t u = base + k * NT + tid;
      x[k] = s[u < lk ? u : lk - 1];
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const uint32_t u = base + k * NT + tid;
      key[k] = order_key(x[k]);
      if (whole && u < lk) cand[u] = key[k];
      const bool up = u < lk && hi != 0 && key[k] >= hi;
      above_t += up ? 1u : 0u;
      mask[k] = __ballot(u < lk && !up && key[k] >= lo);
      n_in += (uint32_t)__popcll(mask[k]);
    }
    if (whole || n_in == 0) continue;  // wave-uniform
    // one place reservation per wave and U keys
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&n_cand, n_in);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const uint32_t pos = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[k] >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask[k], 0u));
      if (((mask[k] >> lane) & 1ull) && pos < (uint32_t)CAND) cand[pos] = key[k];
      at += (uint32_t)__popcll(mask[k]);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) above_t += __shfl_xor(above_t, off, 64);
  if (lane == 0) atomicAdd(&n_above, above_t);
  __syncthreads();
  const uint32_t g_hi = n_above, m = whole ? lk : n_cand;
  const bool in_lds = g_hi < want && want <= g_hi + m && m <= (uint32_t)CAND;  // uniform

  // ---- radix select of the want-th largest key, most significant digit first,
  // among the candidates or, where the bracket failed, over the whole row
  uint32_t prefix = 0, pmask = 0;
  uint32_t above = in_lds ? g_hi : 0;  // keys known to be larger than the selected prefix
  const uint32_t n_keys = in_lds ? m : lk;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (uint32_t u = tid; u < n_keys; u += NT) {
      const uint32_t key = in_lds ? cand[u] : order_key(s[u]);
      const bool in = (key & pmask) == prefix;
      const uint32_t d = (key >> shift) & 255u;
      // (the lanes that share the first one's digit, often all of them in the
      // top digits, are counted with one add)
      const uint64_t act = __ballot(in);
      if (act != 0) {
        const int first = __builtin_ctzll(act);
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, first);
        const uint64_t same = __ballot(in && d == d0);
        if (lane == first) atomicAdd(&hist[d0], (uint32_t)__popcll(same));
        if (in && d != d0) atomicAdd(&hist[d], 1u);
      }
    }
    __syncthreads();
    if (wave == 0) find_digit(hist, above, want, lane, sel);
    __syncthreads();
    prefix |= sel[0] << shift;
    pmask |= 255u << shift;
    above = sel[1];
    __syncthreads();
  }
  // prefix is the want-th largest key; `above` keys are strictly larger.  The sum
  // runs in the row's order whatever the candidates' order in LDS: the call is
  // deterministic.
  auto value = [](uint32_t k) { return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k); };
  const int n_acc = whole ? 256 : NT;
  float sum = 0.f;
  if (whole) {
    if (tid < n_acc)
      for (uint32_t u = tid; u < lk; u += n_acc)
        if (cand[u] > prefix) sum += expf(value(cand[u]) - lse);
  } else {
    for (uint32_t base = 0; base < lk; base += U * NT) {
      float x[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint32_t u = base + k * NT + tid;
        x[k] = s[u < lk ? u : lk - 1];
      }
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (base + k * NT + tid < lk && order_key(x[k]) > prefix) sum += expf(x[k] - lse);
    }
  }
  part[tid] = sum;
  __syncthreads();
  for (int w = n_acc / 2; w > 0; w >>= 1) {
    if (tid < w) part[tid] += part[tid + w];
    __syncthreads();
  }
  // the ties at the threshold fill the remaining places
  if (tid == 0) a.mass[row] = part[0] + (float)(want - above) * expf(value(prefix) - lse);
}

hipError_t launch_retained_mass(const float* lse_sel, const float* lse_all, int64_t n, float* mass,
                                hipStream_t stream) {
  if (n == 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  mass_kernel<<<blocks, 256, 0, stream>>>(lse_sel, lse_all, n, mass);
  return hipGetLastError();
}

hipError_t launch_topk_mass(const TopkArgs& a, int d, hipStream_t stream) {
  if (a.bh == 0 || a.n_rows == 0) return hipSuccess;
  const dim3 grid((unsigned)((a.lk + 255) / 256), (unsigned)a.bh);
  if (d == 128) topk_scores_kernel<128><<<grid, 256, 0, stream>>>(a);
  else if (d == 64) topk_scores_kernel<64><<<grid, 256, 0, stream>>>(a);
  else return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // 6,144 rows of 1,152 keys: 52 us for the call, 250 with the large instance
  // alone; 3,072 of 8,192 keys: 134 and 274.  With fewer rows than CUs the number
  // held by one does not matter, and more threads a row do (192 rows of 8,192).
  const unsigned rows = (unsigned)(a.bh * a.n_rows);
  if (a.lk <= 2048) topk_mass_kernel<2048, 256><<<rows, 256, 0, stream>>>(a);
  else if (a.lk <= 8192 && rows > 256) topk_mass_kernel<8192, 512><<<rows, 512, 0, stream>>>(a);
  else topk_mass_kernel<kTopkCand, 1024><<<rows, 1024, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace sparstar
