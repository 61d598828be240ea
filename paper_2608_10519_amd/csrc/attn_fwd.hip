// Block-sparse attention forward (Eq. 7, Section 5.3) and its dense variant.
//
// Work decomposition.  One work-group per (batch*head, key range, query group).
// A query group of the sparse call is one query block of BLK rows; the dense
// call, whose rows all see the same keys, takes 128 rows whatever the block
// size, so that each K/V byte loaded feeds twice (b = 64) the queries.  A
// work-group has one wavefront per 32-row query slice, and every wave takes the
// whole of each tile (32 keys at D = 128, 64 at D = 64: 8 KB of K and of V), so
// no key is ever split between waves and a row's result does not depend on how
// many waves share its tiles.  Two waves per SIMD (under 256 VGPRs).
//
// Order of the work (XCDs and L2).  Work-groups go round-robin over the eight
// XCDs.  The id decodes so that each XCD runs the query groups of one (head, key
// range) pair after the other.  The work-groups in flight on an XCD (8,192 rows)
// then read the same range of K/V, but those that started earlier
// are further along their lists, so between them they touch all of the range.
// With several ranges, the i-th work-group of a pair therefore starts its list
// at the fraction (i mod C) / C of the range and wraps around, C being the
// number of work-groups in flight: when it starts, the one k before it has done
// about k / C of its list and has just reached the same place, and those in
// flight share a narrow moving window of K/V.  Ranges need not fit the 4 MB L2
// any more, and fewer of them write fewer partial results: at 24 heads, 72,000
// queries, 144,512 keys and 25% density the call took 33.2 ms rotated and 52.8
// plain with 4 ranges (8 ranges: 32.8 and 38.1; 16: 34.5 and 36.0; 2: 36.6 and
// 64.4).  Work-groups that run in step by themselves keep the plain order: the
// dense call and lists that name every block (27.8 ms plain, 29.9 rotated,
// at 25,920 queries and 98,432 keys), the first rounds of a call, and one
// range over the whole sequence, which the window loses (mid scale 5.3 rotated
// and 4.7 plain).  Each list decides by its own length, so that short lists in
// rows of full width are rotated too.
//
// Per tile of the query block's key-block list, a three-stage pipeline: step t
// runs the scores of tile t + 1, the softmax of tile t and P V of tile t - 1.
//   * K and V tiles (8 KB) go from global memory straight into LDS
//     (buffer_load ... lds, 1 KB per wave instruction, coalesced), with no
//     VGPR staging.  LDS holds two K tiles and two V tiles; each tile has one
//     and a half steps to land;
//   * S^T = K Q^T on v_mfma_f32_32x32x16_bf16 (fp32 accumulate).  The
//     transpose leaves each lane holding 16 keys of ONE query column -- exactly
//     the B-operand layout P^T needs -- so the softmax state is lane-local up to
//     one cross-half (lane l <-> l+32) max per refresh (v_permlane32_swap);
//   * online softmax in the log2 domain: the scale is folded into one FMA, the
//     exponential is the bare v_exp_f32, and the running maximum is not taken
//     per tile: P is formed against the current one, and only when some lane's
//     sum of a tile's P exceeds 2^8 (so that some p might) is the tile's
//     max taken, O and the sums rescaled by a power of two, and P formed
//     again -- nearly never after the first tiles;
//   * O^T += V^T P^T on the same MFMA (P rounded to bf16 once).  The V^T
//     operand comes straight from the row-major V tile through the LDS
//     transpose read ds_read_b64_tr_b16 (in each 16-lane group, source lane s
//     points at V[r0 + s/4][4 (c0 + s%4)], and lane j receives
//     V[r0 .. r0+3][4 c0 + j]: 4 keys of one d column).
// None of a step's MFMAs waits for the step's softmax or for an LDS read of the
// same half: the operands of each half are read during the half before.  Every
// MFMA is followed by its share of the softmax (one exponential, one FMA, one add
// and half a pack at D = 128, twice that at D = 64), which issues under it: a
// 32x32x16 MFMA takes 32 cycles, an FMA 2.7 and an exponential 8.
// The row sum of the bf16 P is taken by v_mfma_f32_4x4x4_16b_bf16 against ones
// (each lane's four values summed in 8 cycles).  v_dot2_f32_bf16, which sums
// two, runs on the matrix pipe as well but holds it for about 20 cycles: eight
// of them per tile cost 10% of the kernel (26.3 ms without them against 29.1 at
// 25,920 queries, dense).
// O = O^T / l in bf16 with l the row sum of the bf16-rounded P, and
// lse = ln2*(m + log2 le) with le the row sum of the unrounded fp32 p.
//
// What bounds it (24 heads, D = 128): the dense call runs at 1.10 to 1.16
// PFLOP/s against 1.28 for a large library GEMM on the same card; the matrix
// cores are busy 63% of the cycles at 1.65 GHz, the clock the chip holds under
// this load, and power sets that clock.  The sparse call at b = 64 moves 32 KB of
// K/V per 64 x 64 tile from L2 to LDS, as many texture-path clocks as MFMA
// clocks; without those loads it would take 25.6 instead of 33.4 ms.
//
// MFMA layouts (v_mfma_f32_32x32x16_bf16, lane l, h = l / 32):
//   A[m][k]: m = l % 32, k = 8h + i (i = 0..7 of the lane's bf16x8)
//   B[k][n]: n = l % 32, k = 8h + i
//   C[m][n]: n = l % 32, m = 8 (a / 4) + 4h + (a % 4), accumulator a = 0..15
// A and B only need to agree on k, so keys may be permuted consistently: the
// P^T operand reuses the S^T C layout directly, and the V^T operand reads the
// same key permutation.
#include <type_traits>

#include "device_common.h"

namespace sparstar {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// A step is sixteen MFMAs (and two barriers) at either head dim:
// 32-key tiles at D = 128 (64-key tiles need more than 256 VGPRs in this
// pipeline), 64-key tiles at D = 64, where 32 keys with three waves per SIMD spend
// as long on barriers, waits and addresses per 8 MFMAs.  Over 300 shapes at D = 64
// the best cut takes 4.7% less with 64 keys: 20% less where a CU holds one
// work-group (dense, 209 queries of 2 heads, 134,070 keys: 0.77 of the time), and
// up to 10% more on lists of a few blocks that fill the chip many times over.
template <int D, int BLK, int NWAVES>
struct AttnCfg {
  static constexpr int KB = attn_tile_keys(D);  // keys per K/V tile
  static constexpr int SUB = BLK / KB;        // tiles per key block (list entry)
  static constexpr int NW = NWAVES;           // waves: one per 32-row query slice
  static constexpr int NT = 64 * NW;          // threads
  static constexpr int KT = KB / 32;          // 32-key sub-tiles per step
  static constexpr int DS = D / 16;           // MFMA k-steps over D
  static constexpr int DT = D / 32;           // 32-row d tiles of O^T
  static constexpr int RB = D * 2;            // bytes per K/V row
  static constexpr int CPR = D / 8;           // 16-byte chunks per row
  static constexpr int RPB = 256 / RB;        // rows per 256 bytes (one pass over the 64 LDS banks)
  static constexpr int TILE = KB * D;         // elements per K or V tile
  static constexpr int TILE_BYTES = TILE * 2;
  static constexpr int RPD = 1024 / RB;       // rows per direct-to-LDS wave load (64 lanes x 16 B)
  static constexpr int DPW = TILE_BYTES / 1024 / NW;  // direct loads per wave and tile
  static_assert(DPW * NW * 1024 == TILE_BYTES, "tile split over the waves");
  static constexpr int NK = 2, NV = 2;        // LDS ring: K and V tiles held
  static_assert(KT * 32 == KB, "32-key sub-tiles");
  static_assert(SUB * KB == BLK, "whole tiles per key block");
};

// LDS tiles are stored unpadded (a direct-to-LDS load writes 1 KB contiguous
// per wave), with the 16-byte chunks of each row XOR-permuted so that both
// operand reads are free of bank conflicts:
//   K (ds_read_b128, 16 lanes per pass: 16 consecutive rows, one chunk):
//     physical chunk = c ^ (r / RPB mod CPR)
//   V (ds_read_b64_tr_b16, 32 lanes per pass: 4 consecutive rows x 4 chunks):
//     physical chunk = c ^ ((r / RPB mod 4) * 4 mod CPR)
template <class C>
__device__ __forceinline__ int k_swz(int r) {
  return (r / C::RPB) % C::CPR;
}
template <class C>
__device__ __forceinline__ int v_swz(int r) {
  return (((r / C::RPB) & 3) << 2) & (C::CPR - 1);
}

__device__ __forceinline__ float half_swap_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float half_swap_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}

__device__ __forceinline__ s16x4 lds_read_tr(const uint16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(const_cast<uint16_t*>(p)));
}

// Buffer descriptor as four dwords (raw buffer, stride 0, `bytes` records):
// the form the inline-asm direct-to-LDS load takes.
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 raw_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p);
}

// Direct-to-LDS loads: lane l of a wave-wide load copies 16 bytes from
// buffer offset voff (+ the instruction offset) to LDS byte m0 (+ the same
// instruction offset) + 16 l.  Written as inline assembly so that the compiler
// does not order every later LDS read behind them; each caller waits for these
// loads explicitly (vmcnt) before a barrier makes the tile visible.
//
// A wave's share of one tile: N wave-wide loads after a single M0 write.  The
// instruction offset moves the LDS destination and the memory address alike,
// so load i goes to LDS m0 + 1024 i + 16 l and reads voff[i] + 1024 i (the
// callers pass voff[i] already reduced by 1024 i).
template <int N>
__device__ __forceinline__ void dma_tile(uint32_t m0, const uint32_t* voff, i32x4 rsrc) {
  static_assert(N == 1 || N == 2 || N == 4, "loads per wave and tile");
  if constexpr (N == 1) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen lds"
        :
        : "s"(m0), "v"(voff[0]), "s"(rsrc)
        : "memory", "m0");
  } else if constexpr (N == 2) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
        "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds"
        :
        : "s"(m0), "v"(voff[0]), "v"(voff[1]), "s"(rsrc)
        : "memory", "m0");
  } else {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
        "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
        "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
        "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
        :
        : "s"(m0), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]), "s"(rsrc)
        : "memory", "m0");
  }
}

// s_waitcnt with only the vector-memory counter constrained (<= n outstanding)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <int D, int BLK, int NW, bool DENSE, bool SPLIT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(kAttnWavesPerSimd, kAttnWavesPerSimd)))
void attn_fwd_kernel(AttnArgs a) {
  using C = AttnCfg<D, BLK, NW>;
  static_assert(DENSE || 32 * NW == BLK, "a sparse work-group is one query block");
  __shared__ __attribute__((aligned(1024))) uint16_t ks[C::NK][C::TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t vs[C::NV][C::TILE];

  // Work item: query group qg of the (head, range) pair bh * n_splits + split.
  // A pair's groups are dealt out to 2^spread_bits XCDs (a unit: the pair's groups
  // on one of them).  Units go to the XCDs eight at a time, turned by one XCD
  // each time, so that every XCD gets every range in turn: forced blocks make
  // some ranges several times as long as others (reference and text forced at
  // 720p: 79 ms turned, 122 unturned).  An XCD runs a unit's groups one after the
  // other.  With all eight XCDs on a pair the items simply go in order, which
  // leaves no empty work-groups.  (All of it fits 32 bits, as the grid does.)
  const uint32_t n_g = DENSE ? (uint32_t)((a.lq + 32 * NW - 1) / (32 * NW)) : (uint32_t)a.n_q;  // groups per head
  const uint32_t range_bits = SPLIT ? __builtin_ctz(a.n_splits) : 0;  // n_splits is a power of two
  uint32_t gi, pair;  // gi: the place of the group among the pair's on this XCD
  int qg;
  if (a.spread_bits == 3) {
    pair = blockIdx.x / n_g;
    qg = (int)(blockIdx.x - pair * n_g);
    gi = (uint32_t)qg >> 3;
  } else {
    const uint32_t n_u = (n_g + (1u << a.spread_bits) - 1) >> a.spread_bits;
    const uint32_t id = blockIdx.x / 8, ui = id / n_u;
    gi = id - ui * n_u;
    const uint32_t unit = ui * 8 + (blockIdx.x + ui) % 8;
    pair = unit >> a.spread_bits;
    qg = (int)((gi << a.spread_bits) + (unit & ((1u << a.spread_bits) - 1)));
  }
  if (pair >= ((uint32_t)a.bh << range_bits) || qg >= (int)n_g) return;  // uniform: past the last unit or group
  const int64_t bh = pair >> range_bits;
  const int split = (int)(pair & ((1u << range_bits) - 1));
  const int blk_lo = (int)(((int64_t)split * a.n_k) >> range_bits);
  const int blk_hi = (int)(((int64_t)(split + 1) * a.n_k) >> range_bits);

  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int l32 = lane % 32, hh = lane / 32;

  // ---- Q fragment (B operand of S^T = K Q^T): Q[q][16 s + 8 hh .. +7]
  const int64_t q_row = (int64_t)qg * (32 * NW) + wave * 32 + l32;
  const bool q_ok = q_row < a.lq;
  const uint16_t* qp = a.q + (bh * a.lq + (q_ok ? q_row : 0)) * D;
  bf16x8 qf[C::DS];
#pragma unroll
  for (int s = 0; s < C::DS; ++s) {
    const uint4 u = q_ok ? *reinterpret_cast<const uint4*>(qp + 16 * s + 8 * hh) : make_uint4(0, 0, 0, 0);
    qf[s] = __builtin_bit_cast(bf16x8, u);
  }

  // ---- the list positions [pos_lo, pos_lo + cnt) that hold the blocks of
  // [blk_lo, blk_hi): an ascending list has them after the entries < blk_lo and
  // before the entries >= blk_hi (every wave counts them itself).  The walk
  // starts at position pos_lo + rot, the first entry >= blk_st, and wraps.
  int pos_lo, cnt, rot = 0;
  const int32_t* list = nullptr;
  if constexpr (DENSE) {
    pos_lo = blk_lo;
    cnt = blk_hi - blk_lo;
  } else {
    const int64_t r = bh * a.n_q + qg;
    int nblk = a.kv_num_blocks[r];
    nblk = nblk < 0 ? 0 : (nblk > a.stride ? a.stride : nblk);
    list = a.kv_indices + r * a.stride;
    if constexpr (!SPLIT) {
      // the whole list from its head: nothing to look for
      pos_lo = 0;
      cnt = __builtin_amdgcn_readfirstlane(nblk);
    } else {
      int blk_st = blk_lo;
      if (a.rotation > 0) {
        const uint32_t phase = gi % (uint32_t)a.rotation;
        blk_st += (int)((int64_t)phase * (blk_hi - blk_lo) / a.rotation);
      }
      // 64 x U entries per pass, all loads independent (one memory latency per
      // pass); the counts come from ballots, so they are wave-uniform at once
      constexpr int U = 12;
      int c_lo = 0, c_hi = 0, c_st = 0;
      // (the first pass does not wait for the count: it reads up to the stride)
      for (int base = 0; base == 0 || base < nblk; base += 64 * U) {
        int v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = base + 64 * u + lane;
          v[u] = i < a.stride ? list[i] : 0x7fffffff;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = base + 64 * u + lane < nblk;
          c_lo += __builtin_popcountll(__builtin_amdgcn_ballot_w64(in && v[u] < blk_lo));
          c_hi += __builtin_popcountll(__builtin_amdgcn_ballot_w64(in && v[u] < blk_hi));
          c_st += __builtin_popcountll(__builtin_amdgcn_ballot_w64(in && v[u] < blk_st));
        }
      }
      pos_lo = __builtin_amdgcn_readfirstlane(c_lo);
      cnt = __builtin_amdgcn_readfirstlane(c_hi) - pos_lo;
      rot = __builtin_amdgcn_readfirstlane(c_st) - pos_lo;
      // A list that names every block is walked from its head (rot is out of
      // [0, cnt) only past the range's last entry, or in a list that is not
      // ascending).
      if (nblk >= a.n_k || rot < 0 || rot >= cnt) rot = 0;
    }
  }

  // ---- the key tiles of the item.  Tile j (KB keys) is tile j % SUB of the key
  // block at the walk's entry j / SUB.  The entries are held 64 at a time
  // in a VGPR (lane i: entry lbase + i, as its first tile) and picked out with
  // v_readlane, so the loop issues no memory load of its own except one batch
  // load per 64 entries.  j >= cnt * SUB, and an entry outside [blk_lo, blk_hi)
  // -- only possible in a list that is not ascending --, give a negative tile:
  // one that is loaded as zeros and fully masked.
  int lreg = -1, lbase = 0;
  auto load_batch = [&](int base) {
    lbase = base;
    if constexpr (!DENSE) {
      const int e = base + lane + rot;
      const int b = base + lane < cnt ? list[pos_lo + (e >= cnt ? e - cnt : e)] : -1;
      lreg = (b >= blk_lo && b < blk_hi) ? b * C::SUB : -C::SUB;
      // consume the load here, so that its wait stays on this rare path and is
      // not merged into the common path of the loop
      asm volatile("; list batch %0" ::"v"(lreg));
    }
  };
  const int ntiles = cnt * C::SUB;
  auto fetch = [&](int j) -> int {
    if constexpr (DENSE) {
      // (opaque to the compiler, which would otherwise keep addresses of several
      // steps and spill registers to scratch)
      return __builtin_amdgcn_readfirstlane(j < ntiles ? blk_lo * C::SUB + j : -1);
    } else {
      const int e = j / C::SUB, sub = j % C::SUB;
      if (e >= lbase + 64) load_batch(lbase + 64);
      return __builtin_amdgcn_readlane(lreg, e - lbase) + sub;
    }
  };

  f32x16 acc_o[C::DT];
#pragma unroll
  for (int t = 0; t < C::DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc_o[t][e] = 0.f;
  float m_run = -INFINITY;  // running max (log2 domain), shared by both lane halves
  // Two row sums per lane (each over the lane's half of the keys):
  //   l_run:  of the bf16-rounded P that multiplies V, so that O = (P V) / l_run
  //           is an exact convex combination of the rounded weights (V = 1 gives
  //           O = 1 exactly);
  //   le_run: of the unrounded fp32 p, for the log-sum-exp.
  float l_run = 0.f;
  float le_run = 0.f;

  // ---- direct-to-LDS tile loads: load i of wave w fills LDS bytes
  // [(DPW w + i) KB, +1 KB); lane l writes 16 bytes at +16 l, i.e. physical
  // chunk l % CPR of row RPD (DPW w + i) + l / CPR, and so reads the logical
  // chunk that the XOR permutation puts there.  Each tile gets its own
  // descriptor (records = bytes of the tile that exist), so rows past Lk and
  // the tiles past the end of the list arrive as zeros.  Load i adds 1024 i
  // bytes (RPD rows) to both sides, which moves the K permutation by 4 chunks
  // (of 16 at D = 128, of 8 at D = 64, where two loads come full circle)
  // and leaves the V permutation unchanged; with the instruction offset taking
  // the 1024 i, the per-lane offset of load i is kdma ^ (64 i mod 16 CPR) for K
  // and vdma for V (the identity holds for every configuration built).
  uint32_t kdma, vdma;
  {
    const int row = C::RPD * C::DPW * wave + lane / C::CPR, pos = lane % C::CPR;
    kdma = (uint32_t)(row * C::RB + 16 * (pos ^ k_swz<C>(row)));
    vdma = (uint32_t)(row * C::RB + 16 * (pos ^ v_swz<C>(row)));
  }
  const uint16_t* const kbase = a.k + bh * a.lk * D;
  const uint16_t* const vbase = a.v + bh * a.lk * D;
  // Tiles [0, n_whole) lie wholly below Lk; tile n_whole holds the remaining
  // keys (none if Lk is a whole number of tiles); later tiles and -1 (as
  // unsigned) hold none.
  const uint32_t n_whole = (uint32_t)(a.lk / C::KB);
  const uint32_t last_bytes = (uint32_t)(a.lk % C::KB) * (uint32_t)C::RB;
  auto tile_bytes = [&](int kt) -> uint32_t {
    return (uint32_t)kt < n_whole ? (uint32_t)C::TILE_BYTES : ((uint32_t)kt == n_whole ? last_bytes : 0u);
  };
  auto dma = [&](const uint16_t* base, int blk, uint16_t* slot, uint32_t off0, uint32_t step) {
    const i32x4 rs = raw_rsrc(base + (int64_t)(blk < 0 ? 0 : blk) * C::TILE, tile_bytes(blk));
    uint32_t off[C::DPW];
#pragma unroll
    for (int i = 0; i < C::DPW; ++i) off[i] = off0 ^ (step * i % (16 * C::CPR));
    dma_tile<C::DPW>(lds_addr(slot) + (uint32_t)(C::DPW * wave) * 1024u, off, rs);
  };

  // ---- per-lane LDS read offsets (bytes within a tile)
  // K operand of S^T: row 32 kt + l32, logical chunk 2 s + hh
  uint32_t koff[C::DS];
  {
    const int r = l32;
#pragma unroll
    for (int s = 0; s < C::DS; ++s) koff[s] = (uint32_t)(r * C::RB + 16 * ((2 * s + hh) ^ k_swz<C>(r)));
  }
  // V^T operand through the transpose read: in each 16-lane group g, source lane
  // sl points at row R = 4 hh + sl / 4 (+ 32 kt + 16 half + 8 for the
  // second read), bytes 64 t + 32 (g % 2) + 8 (sl % 4), i.e. logical chunk
  // 4 t + 2 (g % 2) + (sl % 4) / 2, half (sl % 2); lane j then receives
  // V[R0 .. R0+3][4 c0 + j], four keys of one d column
  uint32_t voff[C::DT];
  {
    const int grp = lane >> 4, sl = lane & 15;
    const int r = 4 * hh + (sl >> 2);
#pragma unroll
    for (int t = 0; t < C::DT; ++t) {
      const int c = 4 * t + 2 * (grp & 1) + ((sl & 3) >> 1);
      voff[t] = (uint32_t)(r * C::RB + 16 * (c ^ v_swz<C>(r)) + 8 * (sl & 1));
    }
  }
  auto lds_u4 = [](const uint16_t* slot, uint32_t byte_off) -> uint4 {
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(slot) + byte_off);
  };

  const float sl2 = a.scale_log2;
  const s16x4 one4 = {0x3f80, 0x3f80, 0x3f80, 0x3f80};  // bf16 1.0

  // keys >= Lk of a partial last tile, and every key of a tile past it or of a
  // negative one, get -inf (element e of the lane is key 8 (e / 4) + 4 hh + e % 4
  // of its sub-tile, compared against one per-lane count of visible keys)
  auto mask_tile = [&](f32x16* acc, int kt_id) {
    const int64_t left = kt_id < 0 ? 0 : a.lk - (int64_t)kt_id * C::KB;
    const int vis = (int)(left < 0 ? 0 : (left > C::KB ? C::KB : left)) - 4 * hh;
#pragma unroll
    for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (kt * 32 + 8 * (e / 4) + (e % 4) >= vis) acc[kt][e] = -INFINITY;
  };
  f32x16 acc_s[C::KT];                     // S^T of tile t
  uint32_t pp[C::KT][8];                   // bf16 pairs of P^T of tile t-1
  uint4 kf[C::KT][C::DS];                  // K operands of tile t+1

  auto read_k = [&](const uint16_t* kt_lds) {
#pragma unroll
    for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
      for (int s = 0; s < C::DS; ++s) kf[kt][s] = lds_u4(kt_lds, koff[s] + kt * 32 * C::RB);
  };
  // S^T of the tile whose K operands are in kf
  auto scores = [&](f32x16* acc) {
#pragma unroll
    for (int kt = 0; kt < C::KT; ++kt) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[kt][e] = 0.f;
#pragma unroll
      for (int s = 0; s < C::DS; ++s)
        acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[kt][s]), qf[s], acc[kt], 0, 0, 0);
    }
  };
  // the tile's max logit (log2 domain) of the lane's query over both lane halves
  auto tile_max = [&](const f32x16* acc) -> float {
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, acc[kt][e]);
    return mx;
  };
  auto needs_mask = [&](int blk) { return (uint32_t)blk >= n_whole; };

  // V^T operands of one tile: step m = (2 kt + half) DT + dt.
  // accumulators a = 8 half + i of sub-tile kt hold keys
  //   base + 4 hh + i (i = 0..3) and base + 8 + 4 hh + (i - 4) (i = 4..7),
  // base = 32 kt + 16 half; the two transpose reads fetch the
  // same keys of V for d = 32 t + l % 32.
  constexpr int VM = 2 * C::KT * C::DT;
  auto read_v = [&](const uint16_t* vt, int m) -> s16x8 {
    const uint16_t* vp = reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(vt) + voff[m % C::DT] +
                                                           16 * (m / C::DT) * C::RB);
    const s16x4 v0 = lds_read_tr(vp);
    const s16x4 v1 = lds_read_tr(vp + 8 * D);
    return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // O^T += V^T P^T of one tile, MFMA m over a 16-key k-step
  auto pv = [&](int m, s16x8 v, const uint32_t (&pk)[C::KT][8]) {
    const int kt = m / C::DT / 2, half = m / C::DT % 2, dt = m % C::DT;
    uint4 pu;
    pu.x = pk[kt][4 * half + 0];
    pu.y = pk[kt][4 * half + 1];
    pu.z = pk[kt][4 * half + 2];
    pu.w = pk[kt][4 * half + 3];
    acc_o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pu),
                                                        acc_o[dt], 0, 0, 0);
  };

  if (cnt > 0) {
    // ---- prologue: S of tile 0, the K operands of tile 1 in registers, and the
    // loads of K(2), V(0), K(3) in the order in which the steps wait for them.
    load_batch(0);
    const int b0 = fetch(0);
    int b1 = fetch(1), b2 = fetch(2), b3 = fetch(3);  // tiles t+1 .. t+3
    dma(vbase, -1, vs[1], vdma, 0u);  // zeros: "tile -1" of the first step's P V
#pragma unroll
    for (int kt = 0; kt < C::KT; ++kt)
#pragma unroll
      for (int i = 0; i < 8; ++i) pp[kt][i] = 0u;
    dma(kbase, b0, ks[0], kdma, 64u);
    dma(kbase, b1, ks[1], kdma, 64u);
    wait_vmcnt<0>();
    __syncthreads();
    read_k(ks[0]);
    scores(acc_s);
    if (needs_mask(b0)) mask_tile(acc_s, b0);
    m_run = half_swap_max(tile_max(acc_s)) * sl2;  // O and the sums are still zero
    read_k(ks[1]);
    __syncthreads();  // both K slots are free
    dma(kbase, b2, ks[0], kdma, 64u);
    dma(vbase, b0, vs[0], vdma, 0u);
    dma(kbase, b3, ks[1], kdma, 64u);

    // One step (T = t mod 2 fixes the slots; tile j's K and V are in slot j % 2)
    // in two phases:
    //   A: S of tile t+1 (K operands in registers) while V(t-1) is read; then
    //      K(t+2) is waited for, a barrier frees V(t-1)'s slot for V(t+1);
    //   B: O += P V of tile t-1 while K(t+2) is read; then V(t) is waited for, a
    //      barrier frees K(t+2)'s slot for K(t+4).
    // The softmax of tile t is spread evenly over the MFMAs of both.  A tile's
    // loads have one and a half steps to land, and each wait leaves the two
    // tiles issued after it outstanding.
    int t = 0;
    auto step = [&](auto tc) {
      constexpr int T = decltype(tc)::value;
      uint16_t* const kr = ks[T % 2];        // K(t+2)
      uint16_t* const vr = vs[(T + 1) % 2];  // V(t-1)
      constexpr int MA = C::DS * C::KT;      // MFMAs of phase A
      constexpr int NE = 16 * C::KT;         // elements of S per lane
      constexpr int EPM = NE / (MA + VM);    // elements per MFMA
      static_assert(MA == VM && EPM * (MA + VM) == NE, "softmax spread over the MFMAs");

      f32x16 acc_n[C::KT];
      s16x8 vf[VM];
      uint32_t pk[C::KT][8];  // bf16 pairs of P^T of tile t
      float se = 0.f;         // row sum of the tile's fp32 p (the lane's keys)
      // exp2 offset -m; +inf for a query that has seen no key yet, which makes
      // the sum non-finite and takes the exact path
      const float neg_m = m_run == -INFINITY ? INFINITY : -m_run;
      float x[NE], p[NE];
      f32x4 st4 = {0.f, 0.f, 0.f, 0.f};  // row sum of the tile's bf16 P, in all four
      auto row_sum = [&](int i) {        // adds pairs i - 1 and i (i odd) of P
        const uint2 u = make_uint2(pk[i / 8][i % 8 - 1], pk[i / 8][i % 8]);
        st4 = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(one4, __builtin_bit_cast(s16x4, u), st4, 0, 0, 0);
      };
      auto logit = [&](int e) { x[e] = fmaf(acc_s[e / 16][e % 16], sl2, neg_m); };
      auto prob = [&](int e) { p[e] = __builtin_amdgcn_exp2f(x[e]); };
      // The softmax work that follows MFMA number e / EPM: each stage works one
      // element behind the stage before, so that no instruction waits for the
      // one ahead of it.
      auto element = [&](int e) {
        if (e + 2 < NE) logit(e + 2);
        if (e + 1 < NE) prob(e + 1);
        se = e == 0 ? p[0] : se + p[e];
        if (e % 2 == 1)
          pk[e / 16][e % 16 / 2] = pack2_bf16(p[e - 1], p[e]);
        else if (e >= 4 && e % 4 == 0)
          row_sum(e / 2 - 1);
        // holds the work here (it would otherwise sink to its uses)
        if (e + 2 < NE) asm volatile("" : "+v"(x[e + 2]));
        if (e + 1 < NE) asm volatile("" : "+v"(p[e + 1]));
        asm volatile("" : "+v"(se));
        if (e % 2 == 1) asm volatile("" : "+v"(pk[e / 16][e % 16 / 2]));
      };
      logit(0);
      logit(1);
      prob(0);
      __builtin_amdgcn_sched_barrier(0);

      // ---- phase A
#pragma unroll
      for (int i = 0; i < MA; ++i) {
        const int kt = i / C::DS, s = i % C::DS;
        if (s == 0)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc_n[kt][e] = 0.f;
        acc_n[kt] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[kt][s]), qf[s], acc_n[kt], 0, 0, 0);
        vf[i] = read_v(vr, i);
#pragma unroll
        for (int e = 0; e < EPM; ++e) element(EPM * i + e);
        __builtin_amdgcn_sched_barrier(0);
      }
      wait_vmcnt<2 * C::DPW>();  // K(t+2)
      __syncthreads();
      dma(vbase, b1, vr, vdma, 0u);  // V(t+1)

      // ---- phase B
#pragma unroll
      for (int i = 0; i < VM; ++i) {
        pv(i, vf[i], pp);
        kf[i / C::DS][i % C::DS] = lds_u4(kr, koff[i % C::DS] + i / C::DS * 32 * C::RB);
#pragma unroll
        for (int e = 0; e < EPM; ++e) element(EPM * (MA + i) + e);
        __builtin_amdgcn_sched_barrier(0);
      }
      row_sum(NE / 2 - 1);
      float st = st4[0];
      const int b4 = fetch(t + 4);
      wait_vmcnt<2 * C::DPW>();  // V(t)
      __syncthreads();
      dma(kbase, b4, kr, kdma, 64u);  // K(t+4)

      // The running max is only refreshed when the tile could break the bound
      // p <= 2^8: a lane's sum of its P stays <= 2^8 whenever every p does, so a
      // larger (or non-finite) sum in any lane sends the wave to the exact
      // path -- the tile's max, a rescale of O (which holds the tiles up to
      // t-1) and both sums to it, and the tile's P again (then p <= 1).
      if (__builtin_amdgcn_ballot_w64(!(st <= 256.f))) {
        const float mx = half_swap_max(tile_max(acc_s)) * sl2;
        if (mx > m_run) {
          // the max moves up by a whole number of binades (to >= mx), so the
          // rescale of O and both sums is exact.  A jump past 2^128 (or the
          // first key) drops the old terms, which are then below 2^-120 of
          // the new ones.
          float alpha = 0.f;
          const float dm = mx - m_run;
          if (dm > 128.f) {
            m_run = mx;
          } else {
            const float k = ceilf(dm);
            alpha = __builtin_amdgcn_ldexpf(1.f, -(int)k);
            m_run += k;
          }
          l_run *= alpha;
          le_run *= alpha;
#pragma unroll
          for (int d = 0; d < C::DT; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc_o[d][e] *= alpha;
        }
        st = 0.f;
        se = 0.f;
        const float off = m_run == -INFINITY ? 0.f : -m_run;
#pragma unroll
        for (int e = 0; e < NE; e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(acc_s[e / 16][e % 16], sl2, off));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(acc_s[e / 16][e % 16 + 1], sl2, off));
          se += p0;
          se += p1;
          const uint32_t u = pack2_bf16(p0, p1);
          st += __uint_as_float(u << 16) + __uint_as_float(u & 0xffff0000u);
          pk[e / 16][e % 16 / 2] = u;
        }
      }
      l_run += st;
      le_run += se;
      if (needs_mask(b1)) mask_tile(acc_n, b1);

#pragma unroll
      for (int kt = 0; kt < C::KT; ++kt) {
        acc_s[kt] = acc_n[kt];
#pragma unroll
        for (int i = 0; i < 8; ++i) pp[kt][i] = pk[kt][i];
      }
      b1 = b2;
      b2 = b3;
      b3 = b4;
    };
    // The loop fills many instruction-cache lines; where it begins in one depends
    // on the code before it, and moved by a few instructions it took 28.05 ms
    // instead of 26.90 (24 heads, 25,920 queries, dense).  Aligned here: 26.85.
    asm volatile(".p2align 6");
    while (true) {
      step(std::integral_constant<int, 0>{});
      if (++t >= ntiles) break;
      step(std::integral_constant<int, 1>{});
      if (++t >= ntiles) break;
    }
    // P V of the last tile, whose V the last step waited for
#pragma unroll
    for (int m = 0; m < VM; ++m) pv(m, read_v(vs[(ntiles - 1) % 2], m), pp);
    wait_vmcnt<0>();  // loads past the end of the list still write LDS
  }

  // ---- write O and lse.  The lane's row index is derived again from the lane
  // id (v_mbcnt) rather than kept live over the loop, where every VGPR counts.
  l_run = half_swap_sum(l_run);  // both lane halves now hold the query's row sums
  le_run = half_swap_sum(le_run);
  const int lane_o = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int l32o = lane_o % 32, hho = lane_o / 32;
  const int64_t row_o = (int64_t)qg * (32 * NW) + wave * 32 + l32o;
  const bool row_ok = row_o < a.lq;
  if constexpr (SPLIT) {
    // Partial result of this key range: the unnormalised P V, scaled by a
    // power of two 2^-ex per query row so that its largest magnitude lies in
    // [0.5, 1) and every value keeps fp16's relative precision whatever the
    // range of V; the merge undoes the scale exactly.
    float amax = 0.f;
#pragma unroll
    for (int t = 0; t < C::DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(acc_o[t][e]));
    amax = half_swap_max(amax);
    int ex = 0;
    if (amax > 0.f && amax <= 3.402823466e38f) ex = __builtin_amdgcn_frexp_expf(amax);
    ex = ex < -126 ? -126 : ex;
    const float sc = __builtin_amdgcn_ldexpf(1.0f, -ex);
    if (row_ok) {
      const int64_t prow = ((bh * a.n_q + row_o / BLK) * a.n_splits + split) * BLK + row_o % BLK;
      _Float16* po = reinterpret_cast<_Float16*>(a.part_o) + prow * D;
#pragma unroll
      for (int t = 0; t < C::DT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int d = 32 * t + 8 * g + 4 * hho;
          f16x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = (_Float16)(acc_o[t][4 * g + e] * sc);
          *reinterpret_cast<f16x4*>(po + d) = w;
        }
      if (hho == 0)
        reinterpret_cast<float4*>(a.part_meta)[prow] = make_float4(m_run, l_run, le_run, (float)ex);
    }
  } else if (row_ok) {
    const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
    uint16_t* op = a.o + (bh * a.lq + row_o) * D;
#pragma unroll
    for (int t = 0; t < C::DT; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int d = 32 * t + 8 * g + 4 * hho;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = acc_o[t][4 * g + e] * inv;
        uint2 w;
        w.x = pack2_bf16(o[0], o[1]);
        w.y = pack2_bf16(o[2], o[3]);
        *reinterpret_cast<uint2*>(op + d) = w;
      }
    if (a.lse != nullptr && hho == 0)
      a.lse[bh * a.lq + row_o] = le_run > 0.f ? (m_run + log2f(le_run)) * 0.69314718055994530942f : -INFINITY;
  }
}

// Combines the NS partial results of one query block.  Range r left, per
// query row, A_r = sum of bf16(p) v over its keys scaled by 2^-e_r (fp16), its
// running max m_r (log2 units), the row sums lb_r (of the bf16 p that multiply
// V) and le_r (of the fp32 p), and e_r.  With M = max_r m_r and
// w_r = 2^(m_r - M) over the ranges that saw a key (lb_r > 0):
//   O   = sum_r w_r 2^e_r A_r / sum_r w_r lb_r,
//   lse = ln2 (M + log2 sum_r w_r le_r).
// Ranges with no visible key have weight 0 and add nothing.
// One thread per 8-column chunk of the query block's rows (two chunks per
// thread at BLK = 128, D = 128).
template <int D, int BLK>
struct MergeCfg {
  static constexpr int CPR = D / 8;                     // 8-column chunks per row
  static constexpr int CHUNKS = BLK * CPR;
  static constexpr int NT = CHUNKS < 1024 ? CHUNKS : 1024;
  static constexpr int CPT = CHUNKS / NT;               // chunks per thread
  static_assert(CPT * NT == CHUNKS && NT >= BLK, "chunk split");
};

template <int D, int BLK, int NS>
__global__ __launch_bounds__((MergeCfg<D, BLK>::NT)) void attn_merge_kernel(AttnArgs a) {
  using M = MergeCfg<D, BLK>;
  __shared__ float wts[NS][BLK];
  const int64_t work = blockIdx.x;
  const int64_t bh = work / a.n_q;
  const int qb = (int)(work % a.n_q);
  const int tid = threadIdx.x;
  const int64_t rows = a.lq - (int64_t)qb * BLK;
  // every range's partial is written for every real row of the block (zeros
  // when it saw no key); rows past Lq are never read
  auto load_chunk = [&](int c, f16x8* v) {
    const int row = c / M::CPR, d0 = (c % M::CPR) * 8;
    const int rr = row < rows ? row : 0;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int64_t prow = (work * NS + r) * BLK + rr;
      v[r] = *reinterpret_cast<const f16x8*>(reinterpret_cast<const _Float16*>(a.part_o) + prow * D + d0);
    }
  };
  auto combine = [&](int c, const f16x8* v) {
    const int row = c / M::CPR, d0 = (c % M::CPR) * 8;
    if (row >= rows) return;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const float w = wts[r][row];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = w != 0.f ? fmaf(w, (float)v[r][e], acc[e]) : acc[e];
    }
    uint4 o;
    o.x = pack2_bf16(acc[0], acc[1]);
    o.y = pack2_bf16(acc[2], acc[3]);
    o.z = pack2_bf16(acc[4], acc[5]);
    o.w = pack2_bf16(acc[6], acc[7]);
    *reinterpret_cast<uint4*>(a.o + (bh * a.lq + (int64_t)qb * BLK + row) * D + d0) = o;
  };

  // The threads of the first BLK rows turn the per-row records into weights
  // first and then issue their partial loads; every other thread issues its
  // partial loads at once, so that their latency overlaps the records'.
  f16x8 v[NS];
  if (tid >= BLK) load_chunk(tid, v);
  if (tid < BLK && tid < rows) {
    const int row = tid;
    const float2* rec = reinterpret_cast<const float2*>(a.part_meta);  // record i = float2 pairs 2i, 2i + 1
    float m[NS], lb[NS], mm = -INFINITY;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const float2 x = rec[2 * ((work * NS + r) * BLK + row)];
      m[r] = x.x;
      lb[r] = x.y;
      if (lb[r] > 0.f) mm = fmaxf(mm, m[r]);
    }
    float den = 0.f, sum_e = 0.f;
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const float2 y = rec[2 * ((work * NS + r) * BLK + row) + 1];  // (le, e)
      const float w = lb[r] > 0.f ? exp2f(m[r] - mm) : 0.f;
      den = fmaf(w, lb[r], den);
      sum_e = fmaf(w, y.x, sum_e);
      wts[r][row] = __builtin_amdgcn_ldexpf(w, (int)y.y);
    }
    const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
    for (int r = 0; r < NS; ++r) wts[r][row] *= inv;
    if (a.lse != nullptr)
      a.lse[bh * a.lq + (int64_t)qb * BLK + row] =
          sum_e > 0.f ? (mm + log2f(sum_e)) * 0.69314718055994530942f : -INFINITY;
  }
  if (tid < BLK) load_chunk(tid, v);
  __syncthreads();
  combine(tid, v);
#pragma unroll
  for (int k = 1; k < M::CPT; ++k) {
    load_chunk(tid + k * M::NT, v);
    combine(tid + k * M::NT, v);
  }
}

template <int D, int BLK>
static hipError_t launch_merge(const AttnArgs& a, hipStream_t stream) {
  const int64_t items = (int64_t)a.bh * a.n_q;
  constexpr int NT = MergeCfg<D, BLK>::NT;
  if (a.n_splits == 2) attn_merge_kernel<D, BLK, 2><<<items, NT, 0, stream>>>(a);
  else if (a.n_splits == 4) attn_merge_kernel<D, BLK, 4><<<items, NT, 0, stream>>>(a);
  else if (a.n_splits == 8) attn_merge_kernel<D, BLK, 8><<<items, NT, 0, stream>>>(a);
  else if (a.n_splits == 16) attn_merge_kernel<D, BLK, 16><<<items, NT, 0, stream>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int D, int BLK, int NW, bool DENSE>
static hipError_t launch_cfg(const AttnArgs& a, hipStream_t stream) {
  if (a.grid == 0) return hipSuccess;
  if (a.part_o == nullptr) {
    attn_fwd_kernel<D, BLK, NW, DENSE, false><<<a.grid, 64 * NW, 0, stream>>>(a);
    return hipGetLastError();
  }
  attn_fwd_kernel<D, BLK, NW, DENSE, true><<<a.grid, 64 * NW, 0, stream>>>(a);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_merge<D, BLK>(a, stream);
}

template <int D, int BLK>
static hipError_t launch_mode(const AttnArgs& a, bool dense, hipStream_t stream) {
  if (!dense) return launch_cfg<D, BLK, BLK / 32, false>(a, stream);
  return a.group_rows == 64 ? launch_cfg<D, BLK, 2, true>(a, stream) : launch_cfg<D, BLK, 4, true>(a, stream);
}

hipError_t launch_attn(const AttnArgs& a, int d, int block, bool dense, hipStream_t stream) {
  if (d == 128 && block == 64) return launch_mode<128, 64>(a, dense, stream);
  if (d == 128 && block == 128) return launch_mode<128, 128>(a, dense, stream);
  if (d == 64 && block == 64) return launch_mode<64, 64>(a, dense, stream);
  if (d == 64 && block == 128) return launch_mode<64, 128>(a, dense, stream);
  return hipErrorInvalidValue;
}

}  // namespace sparstar
