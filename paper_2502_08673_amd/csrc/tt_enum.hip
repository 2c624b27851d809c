// tt_enum.hip -- truth-table enumeration kernels for gfx950.
//
// Factored enumeration.  Row r of a neuron splits into a word index h = r/64
// and a lane l = r%64.  Because the digits of r are bit fields, digit j of
// r = 64h + l is the sum of digit j of 64h and digit j of l, so the weighted
// sum splits exactly:
//
//     a(64h + l) = bias + P_hi[h] + P_lo[l],
//     P_hi[h] = sum_j w_j * x_j(64h),   P_lo[l] = sum_j w_j * x_j(l).
//
// P_hi over all words is the dense integer GEMM (digits of the rows 64h) x
// (weights).  From 256 words per plane on it is computed with
// v_mfma_i32_16x16x32_i8, 256 words of one neuron a product, the digits
// generated from h in registers (the row matrix is never stored), exact
// int32 accumulation; shorter tables sum it per lane.  P_lo takes only 64
// values per neuron, which are turned into a table of 64-bit row masks
// M[e] = { l : P_lo[l] - vmin >= e }.  Row l of word h reaches threshold t
// iff P_lo[l] >= t - bias - P_hi[h], so the whole 64-row word of a threshold
// is M[clamp(t - bias - vmin - P_hi[h])]: one LDS lookup per threshold
// replaces 64 compares.  ReLU only matters for thresholds t <= 0, which every
// row reaches; the folded thresholds say so.  The masks of the 2^o - 1
// thresholds are nested, so bit p of the code q is the XOR of the masks whose
// threshold index is a multiple of 2^p.
//
// Two kernels: enum_small_kernel (fewer than 2^12 words per plane) builds
// each neuron's mask table where it uses it; enum_wide_kernel (larger tables,
// many blocks per neuron) reads tables that prep_kernel wrote once.
//
// Histogram, fused: the mask of threshold k holds the rows whose code is at
// least k, so c_k = sum over words of popcount(mask_k) counts them, and
// hist[v] = c_v - c_{v+1} (c_0 = all rows, c_{2^o} = 0).  Each lane keeps its
// c_k in registers (two 16-bit counts per register).  The small kernel sums
// them over the neuron's wave or block and stores the histogram; a block of
// the wide kernel adds its share, c_v - c_{v+1} with c_0 = its rows, into
// hist in global memory: modulo-2^32 adds whose sum over the blocks is the
// histogram itself (the prep kernel zeroes it first), so no conversion pass
// follows.
#include <algorithm>

#include "tt_internal.h"

namespace tt {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// v_writelane_b32 of a 64-bit ballot: its low and high halves (wave-uniform
// SGPRs) into lane L of lo and hi.  Not a memory access.  The halves were
// just written by the compare (a VALU instruction), and a v_writelane that
// reads such an SGPR as data in the very next instruction gets the value
// before the write (measured on this hardware: the first of the two writes
// took the previous compare's half, the second, one instruction later, the
// right one).  The compiler does not see inside the asm, so the asm waits
// two cycles itself; the lane index is an inline constant.
template <int L>
__device__ __forceinline__ void write_lanes(int& lo, int& hi, uint64_t m) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
      : "+v"(lo), "+v"(hi)
      : "s"((int)(uint32_t)m), "s"((int)(uint32_t)(m >> 32)), "i"(L));
}

// Mask-table entries E .. E + 7 of a 64-entry chunk into lanes E .. E + 7 of
// (lo, hi): entry e holds the rows whose pe (P - vmin - chunk start; negative
// for rows past the table) is at least e.  Straight-line, lane indices as
// constants: one compare and two lane writes per entry, no scalar work.
template <int E>
__device__ __forceinline__ void mask_entries8(int& lo, int& hi, int pe) {
  write_lanes<E>(lo, hi, __ballot(pe >= E));
  if constexpr ((E & 7) != 7) mask_entries8<E + 1>(lo, hi, pe);
}

// entries 0 .. lim - 1 of a chunk in blocks of eight (the entries past lim
// of the last block land in lanes that are not stored)
template <int E>
__device__ __forceinline__ void mask_entries(int& lo, int& hi, int pe, int lim) {
  mask_entries8<E>(lo, hi, pe);
  if constexpr (E + 8 < 64) {
    if (E + 8 < lim) mask_entries<E + 8>(lo, hi, pe, lim);
  }
}

// P of row `lane` less its minimum over the rows (INT_MIN in lanes that hold
// no row), and the range of P: digit j contributes w_j times any value of its
// bits below bit min(6, F b), independently of the others, so the extremes
// are sums (wave-uniform, scalar work).
struct LowSums {
  int pv, vmin, range;
};
__device__ __forceinline__ LowSums low_sums(const NeuronRegs& d) {
  const int lane = threadIdx.x & 63;
  const int F = d.F, b = d.b, Fb = F * b;
  const int dmask = (1 << b) - 1;
  const int lowb = Fb < 6 ? Fb : 6;
  int P = 0, vmin = 0, vmax = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j < F && j * b < 6) {
      const int w = weight_at(d.wv, j);
      P += w * ((lane >> (j * b)) & dmask);
      const int nb = min(lowb - j * b, b);
      const int top = w * ((1 << nb) - 1);
      vmin += min(top, 0);
      vmax += max(top, 0);
    }
  }
  return LowSums{lane < (1 << lowb) ? P - vmin : INT_MIN, vmin, vmax - vmin};
}

// Entries e0 .. min(e0 + 63, r1) of a neuron's mask table (entry e: the rows
// with P - vmin >= e; one compare per entry, writelane puts the mask into
// lane e).
__device__ __forceinline__ void mask_chunk(uint64_t* lut, int pv, int e0, int r1) {
  const int lane = threadIdx.x & 63;
  const int lim = __builtin_amdgcn_readfirstlane(min(64, r1 + 1 - e0));
  int lo = 0, hi = 0;
  mask_entries<0>(lo, hi, pv >= 0 ? pv - e0 : -1, lim);
  if (lane < lim) lut[e0 + lane] = ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// Threshold k with bias, ReLU and the minimum of P_lo folded in: row l of
// word h reaches it iff pv[l] >= te - P_hi[h].  Thresholds far outside every
// sum are cut to +-2^30, which no sum reaches either.
__device__ __forceinline__ int folded_threshold(int32_t t, const NeuronRegs& d, int vmin) {
  if (d.act == TT_ACT_RELU && t <= 0) return kNegBig;
  return min(max(t, kNegBig), kPosBig) - d.bias - vmin;
}

// Neurons of the wide kernel, prep_waves waves each (role r = 0 ..
// prep_waves - 1): P_lo, its range, the mask table (64-entry chunks c, taken
// by role c mod prep_waves), the folded thresholds and the zeroed histogram
// (role 0), and, when asked, the support of a small-range neuron (the last
// role).  Several waves per neuron shorten the chain each wave runs when the
// plan has few neurons.
__global__ __launch_bounds__(256) void prep_kernel(EnumArgs a) {
  const int lane = threadIdx.x & 63;
  // wave-uniform by construction; said so, later branches on it are scalar
  const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
  const int W = a.prep_waves;
  const int i = gw / W, role = gw - (gw / W) * W;
  if (i >= a.prep_count) return;
  const int n = __builtin_amdgcn_readfirstlane(a.prep_list[i]);
  // every per-neuron input in one load instruction: lanes 0..15 the
  // descriptor, lanes 16..18 the plan's entries
  const uint32_t* src = neuron_dword(a.desc + n, lane);
  if (lane == 16) src = reinterpret_cast<const uint32_t*>(a.lut_cap + n);
  if (lane == 17) src = reinterpret_cast<const uint32_t*>(a.lut_off + n);
  if (lane == 18) src = reinterpret_cast<const uint32_t*>(a.lut_off + n) + 1;
  const uint32_t x = lane < 19 ? *src : 0u;
  const NeuronRegs d = neuron_from_lanes(x);
  const int cap = __builtin_amdgcn_readlane((int)x, 16);
  const uint64_t loff = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)x, 18) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)x, 17);
  uint64_t* lut = a.lut + loff;
  const LowSums ls = low_sums(d);
  const int r1 = min(ls.range + 1, cap - 1);
  for (int e0 = 64 * role; e0 <= r1; e0 += 64 * W) mask_chunk(lut, ls.pv, e0, r1);
  if (role == 0) {
    const int32_t thr_mine = thr_lane(d, lane >= 1 && lane <= 7 ? lane - 1 : 0);  // lane k + 1: thr[k]
    if (lane < 8) {
      int32_t val = kPosBig;
      if (lane == 0)
        val = r1;
      else if (lane - 1 < (1 << d.o) - 1)
        val = folded_threshold(thr_mine, d, ls.vmin);
      reinterpret_cast<int32_t*>(&a.params[n])[lane] = val;
      if (a.hist) a.hist[(size_t)n * 8 + lane] = 0u;  // histogram accumulators
    }
  }
  // the support of a small-range neuron, decided from its parameters by this
  // wave (the step's support of the plan's own tables)
  const int range = neuron_sum_range(d);
  if (role == W - 1 && a.support && range < 512) {
    const uint32_t sup = small_support_wave(d, range);
    if (lane == 0) a.support[n] = (uint8_t)sup;
  }
}

template <int O>
__device__ __forceinline__ void planes_from_masks(const uint64_t* mk, uint64_t* pl) {
  if constexpr (O == 1) {
    pl[0] = mk[0];
  } else if constexpr (O == 2) {
    pl[0] = mk[0] ^ mk[1] ^ mk[2];
    pl[1] = mk[1];
  } else {
    pl[0] = mk[0] ^ mk[1] ^ mk[2] ^ mk[3] ^ mk[4] ^ mk[5] ^ mk[6];
    pl[1] = mk[1] ^ mk[3] ^ mk[5];
    pl[2] = mk[3];
  }
}

// The four accumulator words of a lane of one 256-word unit (words 2 l + v
// and 128 + 2 l + v - 2 of the unit, see enum_wide_kernel): masks looked up,
// planes stored at dst (the lane's first word), threshold counts added.
// aligned: dst and its planes lie on 16-byte boundaries (wave-uniform).
template <int O, bool NT>
__device__ __forceinline__ void unit_words(const v4i& acc, const int* te, int r1, const uint64_t* lut, uint64_t* dst,
                                           uint64_t W, bool aligned, uint32_t* cnt) {
  constexpr int K = (1 << O) - 1;
  uint64_t pl[4][O];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int P = acc[v];
    uint64_t mk[K];
#pragma unroll
    for (int q = 0; q < K; ++q) mk[q] = lut[min(max(te[q] - P, 0), r1)];
    planes_from_masks<O>(mk, pl[v]);
#pragma unroll
    for (int q = 0; q < K; ++q) cnt[q >> 1] += (uint32_t)__popcll(mk[q]) << (16 * (q & 1));
  }
  if (aligned) {  // 16-byte runs
#pragma unroll
    for (int p = 0; p < O; ++p) {
      u64x2* q = reinterpret_cast<u64x2*>(dst + (uint64_t)p * W);
      if constexpr (NT) {
        __builtin_nontemporal_store(u64x2{pl[0][p], pl[1][p]}, q);
        __builtin_nontemporal_store(u64x2{pl[2][p], pl[3][p]}, q + 64);
      } else {
        q[0] = u64x2{pl[0][p], pl[1][p]};
        q[64] = u64x2{pl[2][p], pl[3][p]};
      }
    }
  } else {
#pragma unroll
    for (int p = 0; p < O; ++p)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        uint64_t* d = dst + (uint64_t)p * W + (v >> 1) * 128 + (v & 1);
        if constexpr (NT)
          __builtin_nontemporal_store(pl[v][p], d);
        else
          *d = pl[v][p];
      }
  }
}

// P_hi of the 256 words from h0 on (the product described at
// enum_wide_kernel); wv: weights with the entries past F cleared.
__device__ __forceinline__ v4i unit_sums(uint64_t wv, int F, int b, uint32_t h0) {
  const int lane = threadIdx.x & 63;
  const uint32_t dmask = (1u << b) - 1u;
  // lanes 0-15: the digits of the unit's row part; lanes 16-31: those of
  // the column part (word 2 j, row 64 * 2 j)
  const uint32_t r = lane < 16 ? (h0 + (uint32_t)(lane & 1) + ((uint32_t)(lane >> 2) << 5) +
                                  ((uint32_t)((lane >> 1) & 1) << 7)) << 6
                               : (uint32_t)(lane & 15) << 7;
  uint64_t dg = 0;
  for (int j = 0; j < F; ++j) dg |= (uint64_t)((r >> (j * b)) & dmask) << (8 * j);
  const long A = lane < 16 ? (long)dg : (lane < 32 ? (long)wv : 0L);
  const long B = lane < 16 ? (long)wv : (lane < 32 ? (long)dg : 0L);
  v4i acc = {0, 0, 0, 0};
  return __builtin_amdgcn_mfma_i32_16x16x32_i8(A, B, acc, 0, 0, 0);
}

// Sum of v over the wave, in lane 63 (DPP row shifts and broadcasts).
__device__ __forceinline__ uint32_t wave_sum_last(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return (uint32_t)x;
}

// One neuron's tables by the `nw` waves of a block (wave `wave`; nw = 1: one
// wave by itself), O = its output width.  lut: LDS entries the waves share.
// Histogram in LDS rows s_cnt[wave * 8 ..] for nw > 1, else written here.
template <int O, bool NT>
__device__ __forceinline__ void small_tables(const SmallArgs& a, const NeuronRegs& d, int n, uint64_t* lut,
                                             uint32_t* s_cnt, int wave, int nw) {
  constexpr int K = (1 << O) - 1;
  constexpr int NC = (K + 1) / 2;
  const int lane = threadIdx.x & 63;
  const int F = d.F, b = d.b, Fb = F * b;
  const uint32_t dmask = (1u << b) - 1u;
  const uint32_t W = Fb >= 6 ? 1u << (Fb - 6) : 1u;
  const LowSums ls = low_sums(d);
  int te[7];
#pragma unroll
  for (int k = 0; k < K; ++k) te[k] = folded_threshold(thr_uniform(d, k), d, ls.vmin);
  uint64_t* tab = a.tables + d.word_off;
  uint32_t c[K + 2];  // rows whose code is at least k (wave-uniform)
  c[0] = Fb >= 6 ? W << 6 : 1u << Fb;
  c[K + 1] = 0u;
  // P_hi of word `h`, one word per lane
  auto sum_of_word = [&](uint32_t h) {
    int P = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < F && (j + 1) * b > 6) P += weight_at(d.wv, j) * (int)(((h << 6) >> (j * b)) & dmask);
    return P;
  };
  if (W <= kDirectWords) {
    // a compare per threshold and word, at most 8 K: fewer instructions than
    // a mask table's entries (3 each, typically 25 to 35) plus the lookups
    const int ph = sum_of_word((uint32_t)lane);
    uint64_t out[O];
#pragma unroll
    for (int p = 0; p < O; ++p) out[p] = 0ull;
#pragma unroll
    for (int k = 1; k <= K; ++k) c[k] = 0u;
    for (int h = 0; h < (int)W; ++h) {
      const int P = __builtin_amdgcn_readlane(ph, h);
      uint64_t mk[K], pl[O];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        mk[k] = __ballot(ls.pv >= te[k] - P);  // lanes without a row hold INT_MIN
        c[k + 1] += (uint32_t)__popcll(mk[k]);
      }
      planes_from_masks<O>(mk, pl);
#pragma unroll
      for (int p = 0; p < O; ++p) out[p] = lane == h ? pl[p] : out[p];
    }
    if (lane < (int)W)
#pragma unroll
      for (int p = 0; p < O; ++p) tab[(uint32_t)p * W + (uint32_t)lane] = out[p];
  } else {
    const int r1 = ls.range + 1;
    for (int e0 = 64 * wave; e0 <= r1; e0 += 64 * nw) mask_chunk(lut, ls.pv, e0, r1);
    if (nw > 1)
      __syncthreads();
    else
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t cnt[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) cnt[q] = 0u;
    if (W >= 256) {
      const uint64_t wm = F < 8 ? d.wv & ((1ull << (8 * F)) - 1ull) : d.wv;
      for (uint32_t h0 = 256u * (uint32_t)wave; h0 < W; h0 += 256u * (uint32_t)nw)
        unit_words<O, NT>(unit_sums(wm, F, b, h0), te, r1, lut, tab + h0 + 2u * (uint32_t)lane, W,
                          (d.word_off & 1ull) == 0, cnt);
    } else {
      for (uint32_t h = 64u * (uint32_t)wave + (uint32_t)lane; h < W; h += 64u * (uint32_t)nw) {
        const int P = sum_of_word(h);
        uint64_t mk[K], pl[O];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          mk[k] = lut[min(max(te[k] - P, 0), r1)];
          cnt[k >> 1] += (uint32_t)__popcll(mk[k]) << (16 * (k & 1));
        }
        planes_from_masks<O>(mk, pl);
#pragma unroll
        for (int p = 0; p < O; ++p) {
          uint64_t* q = tab + (uint32_t)p * W + h;
          if constexpr (NT)
            __builtin_nontemporal_store(pl[p], q);
          else
            *q = pl[p];
        }
      }
    }
    if (!a.hist) return;
    // a wave takes at most 256 words, 2^14 rows: the packed halves hold the sums
    static_assert((1024 / kSmallWaves) * 64 < (1 << 16), "tables of up to 2^10 words, 512 and more by a block's waves");
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const uint32_t t = (uint32_t)__builtin_amdgcn_readlane((int)wave_sum_last(cnt[q]), 63);
      c[2 * q + 1] = t & 0xFFFFu;
      if (2 * q + 2 <= K) c[2 * q + 2] = t >> 16;
    }
    if (nw > 1) {
#pragma unroll
      for (int k = 1; k <= K; ++k)
        if (lane == k) s_cnt[wave * 8 + k] = c[k];
      return;  // the block adds them up
    }
  }
  if (a.hist && lane < 8) {
    uint32_t v = 0u;
#pragma unroll
    for (int k = 0; k <= K; ++k)
      if (lane == k) v = c[k] - c[k + 1];
    a.hist[(size_t)n * 8 + lane] = v;
  }
}

template <bool NT>
__device__ __forceinline__ void small_neuron(const SmallArgs& a, const NeuronRegs& d, int n, uint64_t* lut,
                                             uint32_t* s_cnt, int wave, int nw) {
  switch (d.o) {
    case 1: small_tables<1, NT>(a, d, n, lut, s_cnt, wave, nw); break;
    case 2: small_tables<2, NT>(a, d, n, lut, s_cnt, wave, nw); break;
    default: small_tables<3, NT>(a, d, n, lut, s_cnt, wave, nw); break;
  }
}

// Support of eight neurons whose sums span fewer than 64 values, lane 8 s + j
// deciding digit j of the s-th (the rule of tiny_support_wave, which spends
// a whole wave on one neuron: here the eight lanes of a neuron build their
// sets side by side and walk its thresholds in turn).
__device__ __forceinline__ void tiny_support_lanes(const tt_neuron* dp, bool live, uint8_t* support) {
  const int lane = threadIdx.x & 63, j = lane & 7;
  const uint64_t* q = reinterpret_cast<const uint64_t*>(dp);
  const uint64_t wv = live ? q[0] : 0ull;
  int32_t thr[7];
#pragma unroll
  for (int k = 0; k < 7; ++k) thr[k] = live ? dp->thr[k] : 0;
  const int bias = live ? dp->bias : 0, F = live ? dp->F : 0, b = live ? dp->b : 1;
  const int K = live ? (1 << dp->o) - 1 : 0, relu = live && dp->act == TT_ACT_RELU;
  const int n = live ? (int)dp->reserved : 0;
  const int dmax = (1 << b) - 1;
  uint64_t S = 1ull;
  int base = bias, wj = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int wi = i < F ? weight_at(wv, i) : 0;
    const int aw = wi < 0 ? -wi : wi;
    if (i == j) wj = wi;
    const bool other = i != j && wi != 0;
    if (other && wi < 0) base += wi * dmax;
    // every shift stays below 64: |w_i| 2^m is at most the range
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (other && m < b) S |= S << ((aw << m) & 63);
  }
  const int D = (wj < 0 ? -wj : wj) * dmax;
  bool hit = false;
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    // sums lie within 2^16 of zero: a threshold beyond 2^20 is out of reach
    const int t = min(max(thr[k], -(1 << 20)), 1 << 20);
    if (k < K && wj != 0 && !(relu && t < 1)) {
      const int lo = max((wj > 0 ? t - D : t) - base, 0), hi = min((wj > 0 ? t - 1 : t + D - 1) - base, 63);
      if (lo <= hi) hit = hit || ((S >> lo) << (63 - hi + lo)) != 0ull;
    }
  }
  const uint64_t bal = __ballot(hit);
  if (live && j == 0) support[n] = (uint8_t)(bal >> (lane & 56));
}

// Tables of fewer than 2^kWideMinLog2 words per plane (in fact at most 2^10:
// F b <= 16), histogram and, when asked, support of the neurons whose sums
// span fewer than 512 values, all in one launch and with no workspace: a
// neuron belongs to one wave, or to one block when its tables have 512 words
// or more (or a mask table beyond a wave's share of LDS), so its mask table
// is built where it is used, its histogram is stored and not added up across
// blocks, and nothing has to be cleared first.  Bound by VALU issue and, for
// few neurons, by the launch and one wave's chain: 8192 uneven neurons (17 MB
// of tables) take 11.5 us, 64 neurons of 4096 rows 4.4 us.  (A prep pass that
// wrote the mask tables to memory and a second kernel of tiles of up to 32
// neurons took 12 + 49 us and 5.7 + 12.7 us, most of it latency of their
// chains of loads and, in the tiles, lanes without a word.)  Blocks, in order: neurons of
// a block each, the support of neurons whose sums span 64 to 511 values (a
// wave each), neurons of a wave each, the support of the others (eight to a
// wave); the host lists the longest work first in each class.
template <bool NT>
__global__ __launch_bounds__(64 * kSmallWaves) void enum_small_kernel(SmallArgs a) {
  extern __shared__ uint64_t s_lut[];
  __shared__ uint32_t s_cnt[kSmallWaves * 8];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int blk = (int)blockIdx.x;
  if (blk < a.n_block) {
    const NeuronRegs d = load_neuron(a.desc + blk);
    const int n = __builtin_amdgcn_readlane((int)d.raw, 14);
    small_neuron<NT>(a, d, n, s_lut, s_cnt, wave, kSmallWaves);
    if (!a.hist) return;
    __syncthreads();
    const int k = threadIdx.x, K = (1 << d.o) - 1;
    if (k < 8) {
      const int Fb = d.F * d.b;
      uint32_t ck = k == 0 ? 1u << Fb : 0u, cn = 0u;
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        if (k >= 1 && k <= K) ck += s_cnt[w * 8 + k];
        if (k < K) cn += s_cnt[w * 8 + k + 1];
      }
      a.hist[(size_t)n * 8 + k] = ck - cn;
    }
    return;
  }
  blk -= a.n_block;
  if (a.support) {
    const int mid_blocks = (a.n_mid + kSmallWaves - 1) / kSmallWaves;
    if (blk < mid_blocks) {
      const int i = blk * kSmallWaves + wave;
      if (i >= a.n_mid) return;
      const NeuronRegs d = load_neuron(a.desc + __builtin_amdgcn_readfirstlane(a.mid[i]));
      const uint32_t sup = small_support_wave(d, neuron_sum_range(d));
      if (lane == 0) a.support[__builtin_amdgcn_readlane((int)d.raw, 14)] = (uint8_t)sup;
      return;
    }
    blk -= mid_blocks;
  }
  const int wave_blocks = (a.n_wave + kSmallWaves - 1) / kSmallWaves;
  if (blk < wave_blocks) {
    const int i = blk * kSmallWaves + wave;
    if (i >= a.n_wave) return;
    const NeuronRegs d = load_neuron(a.desc + a.n_block + i);
    small_neuron<NT>(a, d, __builtin_amdgcn_readlane((int)d.raw, 14), s_lut + wave * a.wave_lds, s_cnt, 0, 1);
    return;
  }
  blk -= wave_blocks;
  const int i = (blk * kSmallWaves + wave) * 8 + (lane >> 3);
  const bool live = i < a.n_tiny;
  tiny_support_lanes(a.desc + (live ? a.tiny[i] : 0), live, a.support);
}

// Wide tables (at least 2^kWideMinLog2 words per plane), one (F, b, o) group
// per launch.  A block of NW waves takes NW * upw consecutive 256-word
// units of one neuron (unit NW k + w for wave w in step k, so the block's
// stores at any time are adjacent), copies the neuron's mask table into LDS
// once, and then computes its units with no further global load: on this
// hardware a load issued after stores waits for those stores, so no load
// follows a store.  One v_mfma_i32_16x16x32_i8 gives P_hi of a unit's 256
// words.  Product row i = 4 q + v stands for word bits 0 (v % 2), 5-6 (q)
// and 7 (v / 2), column j for word bits 1-4; a digit of a row index is
// linear in the index's bits, so with
//     A[i][k] = x_k(row part of i),  B[k][j] = w_k            (k < 8),
//     A[i][8 + k] = w_k,             B[8 + k][j] = x_k(column part of j)
// the product is P_hi.  Lane l receives rows 4 (l / 16) + v (v = 0..3) of
// column l % 16: words 2 l + v (v < 2) and 128 + 2 l + v - 2 (v >= 2) of
// the unit, so each store instruction writes one contiguous 1 KiB run
// (16 bytes per lane) and a wave two per plane.  Threshold counts: packed per lane over the
// wave's units, summed over the wave, one atomic per threshold and wave.
template <int O, int NW, bool NT>
__global__ __launch_bounds__(NW * 64) void enum_wide_kernel(EnumArgs a) {
  constexpr int K = (1 << O) - 1;
  constexpr int NC = (K + 1) / 2;
  extern __shared__ uint64_t s_lut[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int upw = a.wide_upw;
  const int per_log2 = a.wide_wb - 8;  // units per neuron: W / 256, a multiple of NW * upw
  // XCD-aware order: blocks go round-robin to the eight XCDs, so block b
  // takes slot (b mod 8) * G/8 + b / 8 and each XCD writes one contiguous
  // eighth of the group's tables (a plain 2 GiB store stream measured 6.7
  // TB/s this way against 6.2 TB/s in launch order).  A tail of fewer than
  // eight blocks keeps its own slots.
  const uint32_t G8 = gridDim.x & ~7u;
  const uint32_t slot = blockIdx.x < G8 ? (blockIdx.x & 7u) * (G8 >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  const long u0 = (long)slot * NW * upw;
  const int n = a.wide_list[u0 >> per_log2];
  const uint32_t hb = (uint32_t)(u0 & ((1L << per_log2) - 1)) << 8;  // the block's first word
  const tt_neuron* dp = a.desc + n;
  // bias, F and b share one aligned dword: a single scalar load
  static_assert(offsetof(tt_neuron, bias) % 4 == 0 && offsetof(tt_neuron, F) == offsetof(tt_neuron, bias) + 2 &&
                    offsetof(tt_neuron, b) == offsetof(tt_neuron, bias) + 3,
                "descriptor layout");
  const uint32_t fbw = *reinterpret_cast<const uint32_t*>(&dp->bias);
  const int F = (int)((fbw >> 16) & 0xFFu), b = (int)(fbw >> 24);
  const uint32_t dmask = (1u << b) - 1u;
  uint64_t wv = *reinterpret_cast<const uint64_t*>(dp->w);
  if (F < 8) wv &= (1ull << (8 * F)) - 1ull;
  const NeuronParams pr = a.params[n];
  const uint64_t* lut = a.lut + a.lut_off[n];
  for (int e = threadIdx.x; e <= pr.r1; e += blockDim.x) s_lut[e] = lut[e];
  __shared__ uint32_t s_cnt[8];
  if (threadIdx.x < 8) s_cnt[threadIdx.x] = 0u;
  const uint64_t W = 1ull << a.wide_wb;
  const uint64_t woff = dp->word_off;
  // digits of the column part (lanes 16-31), the same for every unit
  uint64_t dgc = 0;
  {
    const uint32_t r = (uint32_t)(lane & 15) << 7;  // word 2 j, row 64 * 2 j
    for (int j = 0; j < F; ++j) dgc |= (uint64_t)((r >> (j * b)) & dmask) << (8 * j);
  }
  __syncthreads();
  uint32_t cnt[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) cnt[c] = 0u;
  for (int k = 0; k < upw; ++k) {
    const uint32_t h0 = hb + ((uint32_t)(NW * k + wave) << 8);
    long A = 0, B = 0;
    if (lane < 16) {
      const uint32_t r = (h0 + (uint32_t)(lane & 1) + ((uint32_t)(lane >> 2) << 5) + ((uint32_t)((lane >> 1) & 1) << 7))
                         << 6;
      uint64_t dg = 0;
      for (int j = 0; j < F; ++j) dg |= (uint64_t)((r >> (j * b)) & dmask) << (8 * j);
      A = (long)dg;
      B = (long)wv;
    } else if (lane < 32) {
      A = (long)wv;
      B = (long)dgc;
    }
    v4i acc = {0, 0, 0, 0};
    acc = __builtin_amdgcn_mfma_i32_16x16x32_i8(A, B, acc, 0, 0, 0);
    unit_words<O, NT>(acc, pr.te, pr.r1, s_lut, a.tables + woff + h0 + 2u * (uint32_t)lane, W, (woff & 1ull) == 0, cnt);
  }
  if (a.hist) {  // uniform
    // a lane counts at most 4 * 64 * upw <= 2^13 rows per threshold, so the
    // packed halves do not overflow; the wave sums run in 32 bits.  Lane q
    // of each wave adds the sum of threshold q + 1 into LDS; the block then
    // adds its share of the neuron's histogram, c_v - c_{v+1} with c_0 = its
    // rows, in at most 2^O global adds (modulo 2^32; the sum over the
    // neuron's blocks is the histogram).  About a hundred blocks share a
    // neuron's eight counters over the whole launch, so the adds do not
    // contend.  (The barrier does not wait for the block's table stores.)
    uint32_t mine = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      uint32_t lo = cnt[c] & 0xFFFFu, hi = cnt[c] >> 16;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        lo += (uint32_t)__shfl_xor((int)lo, off, 64);
        hi += (uint32_t)__shfl_xor((int)hi, off, 64);
      }
      if (lane == 2 * c) mine = lo;
      if (lane == 2 * c + 1) mine = hi;
    }
    if (lane < K) atomicAdd(&s_cnt[lane], mine);
    __syncthreads();
    if ((int)threadIdx.x <= K) {
      const int v = threadIdx.x;
      const uint32_t cv = v == 0 ? (uint32_t)(NW * upw) << 14 : s_cnt[v - 1];
      const uint32_t cn = v < K ? s_cnt[v] : 0u;
      if (cv != cn) atomicAdd(&a.hist[(size_t)n * 8 + v], cv - cn);
    }
  }
}

// prep_waves waves per neuron of the list, four waves per block.
hipError_t launch_prep(const EnumArgs& a, hipStream_t s) {
  if (a.prep_count <= 0) return hipSuccess;
  if (a.prep_waves < 1 || a.prep_waves > 64) return hipErrorInvalidValue;
  const int waves_per_block = 4;
  const long waves = (long)a.prep_count * a.prep_waves;
  const int grid = (int)((waves + waves_per_block - 1) / waves_per_block);
  hipLaunchKernelGGL(prep_kernel, dim3(grid), dim3(64 * waves_per_block), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_enum_small(const SmallArgs& a, int nontemporal, hipStream_t s) {
  const long per = kSmallWaves;
  long grid = (long)a.n_block + (a.n_wave + per - 1) / per;
  if (a.support) grid += (a.n_mid + per - 1) / per + (a.n_tiny + 8 * per - 1) / (8 * per);
  if (grid <= 0) return hipSuccess;
  if (a.wave_lds < 0 || a.wave_lds > kSmallWaveLut || a.block_lds < 0 || a.block_lds > kMaxLutCap)
    return hipErrorInvalidValue;
  const size_t lds = sizeof(uint64_t) * (size_t)std::max(kSmallWaves * a.wave_lds, a.block_lds);
  if (nontemporal)
    hipLaunchKernelGGL(enum_small_kernel<true>, dim3((unsigned)grid), dim3(64 * kSmallWaves), lds, s, a);
  else
    hipLaunchKernelGGL(enum_small_kernel<false>, dim3((unsigned)grid), dim3(64 * kSmallWaves), lds, s, a);
  return hipGetLastError();
}

template <int NW, bool NT>
static hipError_t launch_enum_wide_t(const EnumArgs& a, int o, hipStream_t s) {
  if (a.wide_count <= 0) return hipSuccess;
  if (a.wide_wb < kWideMinLog2 || a.wide_wb > 24) return hipErrorInvalidValue;
  const long units = (long)a.wide_count << (a.wide_wb - 8);
  const long per_block = (long)NW * a.wide_upw;
  if (a.wide_upw < 1 || a.wide_upw > kWideMaxUpw || (a.wide_upw & (a.wide_upw - 1)) ||
      per_block > (1L << (a.wide_wb - 8)) || a.wide_lds < 1 || a.wide_lds > kMaxLutCap)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)(units / per_block));
  const size_t lds = sizeof(uint64_t) * (size_t)a.wide_lds;
  switch (o) {
    case 1: hipLaunchKernelGGL((enum_wide_kernel<1, NW, NT>), grid, dim3(NW * 64), lds, s, a); break;
    case 2: hipLaunchKernelGGL((enum_wide_kernel<2, NW, NT>), grid, dim3(NW * 64), lds, s, a); break;
    default: hipLaunchKernelGGL((enum_wide_kernel<3, NW, NT>), grid, dim3(NW * 64), lds, s, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_enum_wide(const EnumArgs& a, int o, int waves, int nontemporal, hipStream_t s) {
  if (nontemporal)
    return waves == 8 ? launch_enum_wide_t<8, true>(a, o, s) : launch_enum_wide_t<4, true>(a, o, s);
  return waves == 8 ? launch_enum_wide_t<8, false>(a, o, s) : launch_enum_wide_t<4, false>(a, o, s);
}

}  // namespace tt
