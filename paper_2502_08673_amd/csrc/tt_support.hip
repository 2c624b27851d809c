// tt_support.hip -- input support and code histogram of packed tables, and
// packing of per-row codes into planes (gfx950).
//
// Support.  Input j is in the support iff two rows that differ only in digit
// j carry different codes.  Walking from one digit value to another one bit
// at a time shows that this holds iff flipping some single row bit inside
// digit j changes the code of some row, so the kernels test single-bit flips:
//  - row bits 0..5 (inside a 64-row word): XOR of a plane word with itself
//    shifted by 2^i, restricted to positions whose bit i is 0;
//  - row bits 6+k: word h against word h ^ 2^k.
// A row bit is recorded in found[n] (bit = row bit); a digit is in the
// support iff any of its b row bits is, and a digit is no longer tested once
// one of its bits is found.  Only the tables are read.  (For tables that are
// the enumeration of their descriptors, support_params_kernel below decides
// the support from the parameters instead.)
#include <algorithm>

#include "tt_internal.h"

namespace tt {

__device__ __forceinline__ uint64_t words_per_plane(int Fb) {
  return Fb >= 6 ? (1ull << (Fb - 6)) : 1ull;
}

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}


// Sum of x over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum_all(uint32_t x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += (uint32_t)__shfl_xor((int)x, off, 64);
  return x;
}

// Tables of 32 words or more go through items of up to 512 words in a wave's
// registers: register k of a lane holds word base + lane + (the bits of k at
// three chosen word bits), so an item's pairs cover the row bits inside a
// word (0-5), the lane bits (6-11) and the three chosen ones.  With word bits
// 6-8 an item is 512 contiguous words; with higher ones (a digit whose row
// bits reach 15 and up) every load still reads 512 contiguous bytes.  Either
// way the items partition the table, so one pass serves the histogram and
// the digits its bits decide.
//
// Three launches.  The first settles the tables of up to 16 words (a lane
// each) and of up to 512 (a wave each, one item), and probes the larger ones,
// a block each: four items spread over the table for every choice of bits
// that some digit needs.  The second scans the larger ones: one pass over
// each choice of bits that a digit still needs after the probes, and the
// histogram with the first of them, so a table is read once (more often only
// when several of its digits of row bits 12 or above never matter).  The third
// turns found bits into supports (a count of ended units in the second would
// need a device-wide fence per unit, which empties the XCD's L2: 480 us).
// Bound by HBM: 100 tables of 2^24 rows
// (419 MB, read 1.05 times), support and histogram: 131-138 us, 3.1 TB/s (a
// histogram pass beside probe, list, work and finish passes: 240 us).
constexpr int kProbes = 4;
constexpr int kRegs = 8;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// x of lane l xor x of lane l ^ 2^T
template <int T>
__device__ __forceinline__ uint32_t lane_flip_diff(uint32_t x) {
  if constexpr (T == 0) return x ^ dpp_mov<0xB1>(x);                  // quad permute 1 0 3 2
  if constexpr (T == 1) return x ^ dpp_mov<0x4E>(x);                  // 2 3 0 1
  if constexpr (T == 2) return x ^ dpp_mov<0x141>(dpp_mov<0x1B>(x));  // 3 2 1 0, then the half row mirrored
  if constexpr (T == 3) return x ^ dpp_mov<0x128>(x);                 // rows of 16 rotated by 8
  // rows of 16 (halves) swapped between two copies: each lane gets both sides
  if constexpr (T == 4) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return r[0] ^ r[1];
  }
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return r[0] ^ r[1];
}

template <int O>
struct Item {
  uint64_t p[O][kRegs];
};

// Word bits of register bits 0..2 (ascending).
struct RegBits {
  int b0, b1, b2;
};
__device__ __forceinline__ uint32_t reg_offset(const RegBits& B, int k) {
  return ((uint32_t)(k & 1) << B.b0) | ((uint32_t)((k >> 1) & 1) << B.b1) | ((uint32_t)(k >> 2) << B.b2);
}
// First word of item `it`: its bits around the lane bits and B.
__device__ __forceinline__ uint32_t item_base(uint32_t it, const RegBits& B) {
  uint32_t x = it << 6;
  x = ((x >> B.b0) << (B.b0 + 1)) | (x & ((1u << B.b0) - 1u));
  x = ((x >> B.b1) << (B.b1 + 1)) | (x & ((1u << B.b1) - 1u));
  x = ((x >> B.b2) << (B.b2 + 1)) | (x & ((1u << B.b2) - 1u));
  return x;
}

// nw: words of the table when it has fewer than 512 (else 512; the others
// read as zero)
template <int O>
__device__ __forceinline__ void load_item(Item<O>& v, const uint64_t* t0, uint64_t W, uint32_t base, const RegBits& B,
                                          int nw) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < kRegs; ++k)
#pragma unroll
    for (int p = 0; p < O; ++p) {
      v.p[p][k] = 0ull;
      const uint64_t* q = t0 + (uint64_t)p * W + base + reg_offset(B, k);
      if (64 * k + lane < nw) v.p[p][k] = q[lane];
    }
}

// Rows whose bit pattern holds a set of planes: c[s - 1] counts the rows with
// every plane of the set s.
template <int O>
__device__ __forceinline__ void count_sets(const Item<O>& v, uint32_t (&c)[(1 << O) - 1]) {
#pragma unroll
  for (int k = 0; k < kRegs; ++k) {
    uint64_t x[1 << O];
#pragma unroll
    for (int s = 1; s < (1 << O); ++s) {
      const int low = s & -s, p = low == 1 ? 0 : (low == 2 ? 1 : 2);
      x[s] = s == low ? v.p[p][k] : x[s ^ low] & v.p[p][k];
      c[s - 1] += (uint32_t)__popcll(x[s]);
    }
  }
}
// Rows of code v from the set counts c (c[-1] = all rows): inclusion and
// exclusion over the planes that v lacks.
template <int O>
__device__ __forceinline__ uint32_t rows_of_code(const uint32_t (&c)[(1 << O) - 1], uint32_t rows, int v) {
  uint32_t n = 0;
#pragma unroll
  for (int s = 0; s < (1 << O); ++s)
    if ((s & v) == v) {
      const uint32_t t = s == 0 ? rows : c[s > 0 ? s - 1 : 0];
      n += (__popc(s ^ v) & 1) ? 0u - t : t;
    }
  return n;
}

template <int O>
__device__ __forceinline__ uint32_t inword_diff(const Item<O>& v, int q) {
  uint32_t x = 0;
#pragma unroll
  for (int k = 0; k < kRegs; ++k)
#pragma unroll
    for (int p = 0; p < O; ++p) {
      const uint32_t lo = (uint32_t)v.p[p][k], hi = (uint32_t)(v.p[p][k] >> 32);
      // rows l and l + 2^q: for q < 5 both lie in one half, for q = 5 the
      // halves are the pairs
      x |= q == 5 ? lo ^ hi : (lo ^ (lo >> (1 << q))) | (hi ^ (hi >> (1 << q)));
    }
  return q == 5 ? x : x & (uint32_t)low_flip_select(q);
}
template <int O, int T>
__device__ __forceinline__ uint32_t lane_diff(const Item<O>& v) {
  uint32_t x = 0;
#pragma unroll
  for (int k = 0; k < kRegs; ++k)
#pragma unroll
    for (int p = 0; p < O; ++p) {
      const uint32_t lo = (uint32_t)v.p[p][k], hi = (uint32_t)(v.p[p][k] >> 32);
      x |= lane_flip_diff<T>(lo) | lane_flip_diff<T>(hi);
    }
  return x;
}
template <int O>
__device__ __forceinline__ uint32_t reg_diff(const Item<O>& v, int i) {
  uint64_t x = 0;
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (u == i) {  // uniform
#pragma unroll
      for (int k = 0; k < kRegs; ++k)
        if (!(k & (1 << u)))
#pragma unroll
          for (int p = 0; p < O; ++p) x |= v.p[p][k] ^ v.p[p][k | (1 << u)];
    }
  return (uint32_t)x | (uint32_t)(x >> 32);
}

// The row bits of `todo` (testable in this item) whose flip changes some
// code; of a digit only the first that does.
template <int O>
__device__ __forceinline__ uint32_t item_finds(const Item<O>& v, const RegBits& B, int b, uint32_t todo) {
  uint32_t fl = 0;
  while (todo) {  // uniform
    const int bit = __ffs(todo) - 1;
    todo &= todo - 1u;
    uint32_t x;
    if (bit < 6) {
      x = inword_diff<O>(v, bit);
    } else if (bit < 12) {
      switch (bit - 6) {
        case 0: x = lane_diff<O, 0>(v); break;
        case 1: x = lane_diff<O, 1>(v); break;
        case 2: x = lane_diff<O, 2>(v); break;
        case 3: x = lane_diff<O, 3>(v); break;
        case 4: x = lane_diff<O, 4>(v); break;
        default: x = lane_diff<O, 5>(v); break;
      }
    } else {
      x = reg_diff<O>(v, bit - 6 == B.b0 ? 0 : (bit - 6 == B.b1 ? 1 : 2));
    }
    if (__any(x != 0u)) {
      fl |= 1u << bit;
      todo &= ~(((1u << b) - 1u) << ((bit / b) * b));
    }
  }
  return fl;
}

__device__ __forceinline__ uint32_t testable(const RegBits& B) {
  return 0xFFFu | (64u << B.b0) | (64u << B.b1) | (64u << B.b2);
}
constexpr RegBits kNear = {6, 7, 8};

// Far group g (g = 0, 1, ...) of a neuron: up to three row bits from 15 up of
// one digit as register bits, the lowest word bits beside them; false when
// there is no such group.
__device__ __forceinline__ bool far_group(int F, int b, int g, int* digit, RegBits* B) {
  for (int j = 0; j < F; ++j) {
    const int lo = j * b > 15 ? j * b : 15, hi = (j + 1) * b;
    for (int s = lo; s < hi; s += 3)
      if (g-- == 0) {
        const int c = hi - s < 3 ? hi - s : 3, w = s - 6;
        *digit = j;
        *B = c == 3 ? RegBits{w, w + 1, w + 2} : (c == 2 ? RegBits{6, w, w + 1} : RegBits{6, 7, w});
        return true;
      }
  }
  return false;
}

__device__ __forceinline__ uint8_t support_of_bits(uint32_t found, int F, int b) {
  uint32_t s = 0;
  for (int j = 0; j < F; ++j)
    if (found & (((1u << b) - 1u) << (j * b))) s |= 1u << j;
  return (uint8_t)s;
}

// Support and/or histogram of the small tables (at most kSmallTableWords
// words per plane), one lane per neuron holding its whole table: in-word row
// bits by shifted XOR, word bits by comparing word pairs, codes by popcounts.
__device__ __forceinline__ void small_table(const SupportArgs& a, int n) {
  if (n >= a.n) return;
  const tt_neuron* dp = a.desc + n;
  const int F = dp->F, b = dp->b, o = dp->o;
  const int Fb = F * b, Wb = Fb > 6 ? Fb - 6 : 0;
  const int W = 1 << Wb;
  if (W > kSmallTableWords) return;
  const uint64_t* t0 = a.tables + dp->word_off;
  uint64_t P0[kSmallTableWords], P1[kSmallTableWords], P2[kSmallTableWords];
#pragma unroll
  for (int h = 0; h < kSmallTableWords; ++h) {
    P0[h] = P1[h] = P2[h] = 0ull;
    if (h < W) {
      P0[h] = t0[h];
      if (o > 1) P1[h] = t0[W + h];
      if (o > 2) P2[h] = t0[2 * W + h];
    }
  }
  if (a.hist) {
    const uint64_t validw = Fb >= 6 ? ~0ull : ((1ull << (1 << Fb)) - 1ull);
    uint32_t hv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < kSmallTableWords; ++h) {
      const uint64_t m0 = h < W ? validw : 0ull;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        uint64_t x = m0 & ((v & 1) ? P0[h] : ~P0[h]);
        x &= (v & 2) ? P1[h] : ~P1[h];
        x &= (v & 4) ? P2[h] : ~P2[h];
        hv[v] += (uint32_t)__popcll(x);
      }
    }
    uint4* hd = reinterpret_cast<uint4*>(a.hist + (size_t)n * 8);
    hd[0] = make_uint4(hv[0], hv[1], hv[2], hv[3]);
    hd[1] = make_uint4(hv[4], hv[5], hv[6], hv[7]);
  }
  if (a.support) {
    uint32_t fl = 0;
    const int lowbits = Fb < 6 ? Fb : 6;
    for (int q = 0; q < lowbits; ++q) {
      const int sh = 1 << q;
      uint64_t x = 0;
#pragma unroll
      for (int h = 0; h < kSmallTableWords; ++h)
        x |= (P0[h] ^ (P0[h] >> sh)) | (P1[h] ^ (P1[h] >> sh)) | (P2[h] ^ (P2[h] >> sh));
      if (x & low_flip_select(q)) fl |= 1u << q;
    }
    for (int t = 0; t < Wb; ++t) {
      bool df = false;
#pragma unroll
      for (int h = 0; h < kSmallTableWords; ++h) {
#pragma unroll
        for (int u = 0; u < 4; ++u)  // h ^ 2^t for the t of this iteration
          if (u == t && !(h & (1 << u)) && (h | (1 << u)) < kSmallTableWords)
            df |= P0[h] != P0[h | (1 << u)] || P1[h] != P1[h | (1 << u)] || P2[h] != P2[h | (1 << u)];
      }
      if (df) fl |= 1u << (6 + t);
    }
    uint32_t sres = 0;
    for (int j = 0; j < F; ++j)
      if (fl & (((1u << b) - 1u) << (j * b))) sres |= 1u << j;
    a.support[n] = (uint8_t)sres;
  }
}

// A table of 32 to 512 words per plane: one item, one wave.
template <int O>
__device__ __forceinline__ void medium_table(const SupportArgs& a, const NeuronRegs& d, int n) {
  const int lane = threadIdx.x & 63, Fb = d.F * d.b, nw = 1 << (Fb - 6);
  Item<O> v;
  load_item<O>(v, a.tables + d.word_off, (uint64_t)nw, 0u, kNear, nw);
  if (a.hist) {
    uint32_t c[(1 << O) - 1];
#pragma unroll
    for (int s = 0; s < (1 << O) - 1; ++s) c[s] = 0u;
    count_sets<O>(v, c);
#pragma unroll
    for (int s = 0; s < (1 << O) - 1; ++s) c[s] = wave_sum_all(c[s]);
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < (1 << O); ++q)
      if (lane == q) mine = rows_of_code<O>(c, 1u << Fb, q);
    if (lane < 8) a.hist[(size_t)n * 8 + lane] = mine;
  }
  if (a.support) {
    const uint32_t fl = item_finds<O>(v, kNear, d.b, unknown_row_bits(0u, d.F, d.b));
    if (lane == 0) a.support[n] = support_of_bits(fl, d.F, d.b);
  }
}

// The probes of a table of 2^10 words or more, by the block's waves.
template <int O>
__device__ __forceinline__ void probe_table(const SupportArgs& a, const NeuronRegs& d, uint32_t* s_found, int wave,
                                            int waves) {
  const int lane = threadIdx.x & 63, F = d.F, b = d.b, Wb = F * b - 6;
  const uint64_t W = 1ull << Wb;
  const uint64_t* t0 = a.tables + d.word_off;
  const uint32_t items = (uint32_t)(W >> 9);
  for (int u = wave;; u += waves) {
    const int g = u / kProbes, k = u % kProbes;
    int digit = 0;
    RegBits B = kNear;
    if (g > 0 && !far_group(F, b, g - 1, &digit, &B)) break;
    const uint32_t it = (uint32_t)((uint64_t)k * items / kProbes);
    if (k > 0 && it == (uint32_t)((uint64_t)(k - 1) * items / kProbes)) continue;
    const uint32_t seen = (uint32_t)__builtin_amdgcn_readfirstlane((int)*(volatile uint32_t*)s_found);
    uint32_t need = unknown_row_bits(seen, F, b) & testable(B);
    if (g > 0 && !(need & (((1u << b) - 1u) << (digit * b)))) continue;
    if (!need) continue;
    Item<O> v;
    load_item<O>(v, t0, W, item_base(it, B), B, 512);
    const uint32_t fl = item_finds<O>(v, B, b, need);
    if (fl && lane == 0) atomicOr(s_found, fl);
  }
}

// Blocks: larger tables (probes, a block each), tables of 32 to 512 words (a
// wave each), then all neurons a lane each for the smallest tables.
__global__ __launch_bounds__(512) void support_first_kernel(SupportArgs a) {
  __shared__ uint32_t s_found;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int blk = (int)blockIdx.x;
  if (blk < a.n_large) {
    const int n = a.large[blk];
    if (threadIdx.x == 0) s_found = 0u;
    __syncthreads();
    if (a.support) {
      const NeuronRegs d = load_neuron(a.desc + n);
      switch (d.o) {
        case 1: probe_table<1>(a, d, &s_found, wave, 8); break;
        case 2: probe_table<2>(a, d, &s_found, wave, 8); break;
        default: probe_table<3>(a, d, &s_found, wave, 8); break;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      a.probed[blk] = s_found;
      a.found[blk] = s_found;
    }
    if (a.hist && threadIdx.x < 8) a.hist[(size_t)n * 8 + threadIdx.x] = 0u;
    return;
  }
  blk -= a.n_large;
  const int medium_blocks = (a.n_medium + 7) / 8;
  if (blk < medium_blocks) {
    const int i = blk * 8 + wave;
    if (i >= a.n_medium) return;
    const int n = __builtin_amdgcn_readfirstlane(a.medium[i]);
    const NeuronRegs d = load_neuron(a.desc + n);
    switch (d.o) {
      case 1: medium_table<1>(a, d, n); break;
      case 2: medium_table<2>(a, d, n); break;
      default: medium_table<3>(a, d, n); break;
    }
    return;
  }
  blk -= medium_blocks;
  small_table(a, blk * 512 + (int)threadIdx.x);
}

// The smallest tables where there are no others, in blocks of four waves: the
// first kernel's blocks of eight put twice the waves on a CU while others idle.
// Same instructions and registers, 2 / 4 / 8 waves a block, support and
// histogram: 500 tables of 16 words, two planes, 9.3 / 10.6 / 15.6 us; 20000,
// three planes, 12.1 / 14.1 / 19.4; 50000, two planes, 16.9 / 14.6 / 18.0.
__global__ __launch_bounds__(256) void support_small_kernel(SupportArgs a) {
  small_table(a, (int)(blockIdx.x * 256 + threadIdx.x));
}

// One unit of a larger table: items part, part + units, ... of each pass.
template <int O>
__device__ __forceinline__ void scan_table(const SupportArgs& a, const NeuronRegs& d, int k, int n, uint32_t part,
                                           uint32_t units) {
  const int lane = threadIdx.x & 63, F = d.F, b = d.b, Wb = F * b - 6;
  const uint64_t W = 1ull << Wb;
  const uint64_t* t0 = a.tables + d.word_off;
  const uint32_t items = (uint32_t)(W >> 9);
  // what the probes left open chooses the passes (the same for every unit of
  // the neuron: the items of a pass are shared out between them)
  const uint32_t open = a.support ? unknown_row_bits(a.probed[k], F, b) : 0u;
  uint32_t fnd = a.support ? (uint32_t)__builtin_amdgcn_readfirstlane((int)a.found[k]) : ~0u;
  uint32_t c[(1 << O) - 1];
#pragma unroll
  for (int s = 0; s < (1 << O) - 1; ++s) c[s] = 0u;
  bool count = a.hist != nullptr;
  auto pass = [&](const RegBits& B, uint32_t wanted) {
    for (uint32_t it = part; it < items; it += units) {
      uint32_t need = a.support ? unknown_row_bits(fnd, F, b) & testable(B) & wanted : 0u;
      if (!count && !need) return;
      Item<O> v;
      load_item<O>(v, t0, W, item_base(it, B), B, 512);
      if (need) {
        // what other units have found since, now and then (a round trip)
        if (((it / units) & 3u) == 3u) fnd |= (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)__hip_atomic_load(&a.found[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        need = unknown_row_bits(fnd, F, b) & testable(B) & wanted;
        const uint32_t fl = item_finds<O>(v, B, b, need);
        if (fl && lane == 0) atomicOr(&a.found[k], fl);
        fnd |= fl;
      }
      if (count) count_sets<O>(v, c);
    }
    count = false;
  };
  bool any = false;
  if (open & 0x7000u) {  // a digit with row bits 12 - 14
    pass(kNear, ~0u);
    any = true;
  }
  int digit;
  RegBits B;
  for (int g = 0; far_group(F, b, g, &digit, &B); ++g) {
    const uint32_t D = ((1u << b) - 1u) << (digit * b);
    if (!(open & D)) continue;
    pass(B, any ? D : ~0u);  // the first pass also settles the low digits
    any = true;
  }
  if (!any && (open || count)) pass(kNear, ~0u);
  if (a.hist) {
#pragma unroll
    for (int s = 0; s < (1 << O) - 1; ++s) c[s] = wave_sum_all(c[s]);
    const uint32_t mine_items = part < items ? (items - 1u - part) / units + 1u : 0u;
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < (1 << O); ++q)
      if (lane == q) mine = rows_of_code<O>(c, mine_items << 15, q);
    if (lane < (1 << O) && mine) atomicAdd(&a.hist[(size_t)n * 8 + lane], mine);
  }
}

__global__ __launch_bounds__(256) void support_scan_kernel(SupportArgs a, uint32_t U) {
  const uint32_t gw = (uint32_t)__builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
  const uint32_t k = gw / U, part = gw - k * U;
  if (k >= (uint32_t)a.n_large) return;
  const int n = __builtin_amdgcn_readfirstlane(a.large[k]);
  const NeuronRegs d = load_neuron(a.desc + n);
  const uint32_t items = 1u << (d.F * d.b - 15), units = min(U, items);
  if (part >= units) return;
  switch (d.o) {
    case 1: scan_table<1>(a, d, (int)k, n, part, units); break;
    case 2: scan_table<2>(a, d, (int)k, n, part, units); break;
    default: scan_table<3>(a, d, (int)k, n, part, units); break;
  }
}

__global__ __launch_bounds__(256) void support_finish_kernel(SupportArgs a) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= a.n_large) return;
  const int n = a.large[k];
  a.support[n] = support_of_bits(a.found[k], a.desc[n].F, a.desc[n].b);
}

hipError_t launch_support_tables(const SupportArgs& a, int cus, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (a.n_large == 0 && a.n_medium == 0) {
    hipLaunchKernelGGL(support_small_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  const long first = (long)a.n_large + (a.n_medium + 7) / 8 + (a.n_small > 0 ? (a.n + 511) / 512 : 0);
  hipLaunchKernelGGL(support_first_kernel, dim3((unsigned)first), dim3(512), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_large <= 0) return e;
  // up to 64 waves a compute unit (four rounds of those resident), at most one
  // unit per item; a power of two, as the items are, so that every unit of a
  // neuron gets as many (100 tables of 2^24 rows: 16 units a compute unit at
  // most 189 us, 32: 143, 64: 138)
  long U = 1;
  while (2 * U <= a.max_items && 2 * U * a.n_large <= 64L * cus) U *= 2;
  const long waves = (long)a.n_large * U;
  hipLaunchKernelGGL(support_scan_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, a, (uint32_t)U);
  if ((e = hipGetLastError()) != hipSuccess || !a.support) return e;
  hipLaunchKernelGGL(support_finish_kernel, dim3((unsigned)((a.n_large + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Support of a neuron from its parameters, for tables that are its own
// enumeration.  q is a non-decreasing function of the pre-activation a
// (ReLU and the threshold count are both monotone), with jumps exactly at
// the thresholds (identity) or at the thresholds >= 1 (ReLU: q is constant
// for a <= 0).  Fix the other digits: their sum s (bias included) runs over
// the set S_j = bias + { sum_{i != j} w_i x_i }, and as x_j runs over
// 0 .. 2^b - 1 the pre-activation takes every value of s + w_j x_j, whose
// two ends are s and s + w_j (2^b - 1).  So digit j changes some code iff
// some jump point t has lo < t <= hi for the ends lo < hi of that range,
// for some s in S_j: exactly the definition of the support.  Offsets of S_j
// from its minimum form the set of sums of |w_i| x_i, a subset-sum bitset
// built by shift-ORs: x_i = sum of its bits 2^m, so b shifts by 2^m |w_i|
// per digit.  One wave per digit; the bitset (at most 8 * 128 * 15 + 1
// values) lives in registers, word k = lane + 64 m in register m of the
// lane; a shift is at most 8 * 128 bits (16 words), so each word takes
// its parts from registers m and m - 1 of another lane (shuffles).
constexpr int kSumRegs = 4;  // 4 x 64 words: 16384 values

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src) {
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, 64);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64);
  return ((uint64_t)hi << 32) | lo;
}

// Word k - d of the bitset, for the word k = lane + 64 m of this lane (0 < d < 64).
__device__ __forceinline__ uint64_t word_back(const uint64_t (&S)[kSumRegs], int m, int d, int lane) {
  const int src = (lane - d) & 63;
  const uint64_t same = shfl64(S[m], src);
  const uint64_t prev = m > 0 ? shfl64(S[m > 0 ? m - 1 : 0], src) : 0ull;
  return lane >= d ? same : prev;
}

// S |= S << a (a <= 1024) over the first nr registers.
__device__ __forceinline__ void shift_or(uint64_t (&S)[kSumRegs], int a, int nr, int lane) {
  const int q = a >> 6, r = a & 63;
  uint64_t out[kSumRegs];
#pragma unroll
  for (int m = 0; m < kSumRegs; ++m) {
    out[m] = S[m];
    if (m < nr) {  // uniform
      const uint64_t v1 = q == 0 ? S[m] : word_back(S, m, q, lane);
      const uint64_t v2 = word_back(S, m, q + 1, lane);
      out[m] |= (v1 << r) | (r ? (v2 >> (64 - r)) : 0ull);
    }
  }
#pragma unroll
  for (int m = 0; m < kSumRegs; ++m) S[m] = out[m];
}

// Whether any bit of S in [lo, hi] is set (wave-uniform).
__device__ __forceinline__ bool any_in_range(const uint64_t (&S)[kSumRegs], int64_t lo, int64_t hi, int lane) {
  bool hit = false;
#pragma unroll
  for (int m = 0; m < kSumRegs; ++m) {
    const int64_t k0 = (int64_t)(lane + 64 * m) * 64;
    const int64_t a = lo > k0 ? lo : k0, e = hi < k0 + 63 ? hi : k0 + 63;
    if (a <= e) {
      const int sa = (int)(a - k0), se = (int)(e - k0);
      const uint64_t mask = (se == 63 ? ~0ull : ((1ull << (se + 1)) - 1ull)) & ~((1ull << sa) - 1ull);
      hit |= (S[m] & mask) != 0ull;
    }
  }
  return __any(hit);
}

// One block of eight waves per neuron (grid-strided), wave j deciding digit j.
__global__ __launch_bounds__(512) void support_params_kernel(const tt_neuron* desc, const int32_t* list, int n,
                                                             uint8_t* support) {
  __shared__ uint32_t s_bits[8];
  const int lane = threadIdx.x & 63;
  const int j = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int c = blockIdx.x; c < n; c += gridDim.x) {
    const int i = list ? list[c] : c;
    const tt_neuron* dp = desc + i;
    const int F = dp->F, b = dp->b, o = dp->o, act = dp->act;
    const int K = (1 << o) - 1, dmax = (1 << b) - 1;
    int w[8];
    int Rall = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      w[k] = k < F ? (int)dp->w[k] : 0;
      Rall += (w[k] < 0 ? -w[k] : w[k]) * dmax;
    }
    const int nr = Rall / 4096 + 1;  // registers in use (64 words each)
    bool found = false;
    if (j < F && w[j] != 0) {  // uniform per wave
      // S_j as offsets from its minimum base
      int64_t base = dp->bias;
      int R = 0;
      uint64_t S[kSumRegs];
#pragma unroll
      for (int m = 0; m < kSumRegs; ++m) S[m] = (lane == 0 && m == 0) ? 1ull : 0ull;
      for (int i2 = 0; i2 < F; ++i2) {
        if (i2 == j || w[i2] == 0) continue;
        const int aw = w[i2] < 0 ? -w[i2] : w[i2];
        base += (int64_t)(w[i2] < 0 ? w[i2] : 0) * dmax;
        R += aw * dmax;
        for (int m = 0; m < b; ++m) shift_or(S, aw << m, nr, lane);
      }
      const int64_t D = (int64_t)(w[j] < 0 ? -w[j] : w[j]) * dmax;
      for (int k = 0; k < K && !found; ++k) {
        const int64_t t = dp->thr[k];
        if (act == TT_ACT_RELU && t < 1) continue;
        // s with s < t <= s + D (w_j > 0) or s - D < t <= s (w_j < 0)
        int64_t lo = w[j] > 0 ? t - D : t, hi = w[j] > 0 ? t - 1 : t + D - 1;
        lo -= base;
        hi -= base;
        if (lo < 0) lo = 0;
        if (hi > R) hi = R;
        if (lo <= hi) found = any_in_range(S, lo, hi, lane);
      }
    }
    if (lane == 0) s_bits[j] = found ? 1u << j : 0u;
    __syncthreads();
    if (threadIdx.x == 0)
      support[i] = (uint8_t)(s_bits[0] | s_bits[1] | s_bits[2] | s_bits[3] | s_bits[4] | s_bits[5] | s_bits[6] |
                             s_bits[7]);
    __syncthreads();  // s_bits is reused by the next neuron
  }
}

// Neurons whose sums span at most 512 values (sum_j |w_j| (2^b - 1) < 512,
// e.g. |w| <= 7 and b <= 3): one wave per neuron, lane group g (8 lanes,
// 8 words = 512 bits) deciding digit g; every shift is below 8 words and
// stays inside the group.
__global__ __launch_bounds__(256) void support_params_small_kernel(const tt_neuron* desc, const int32_t* list,
                                                                  int count, uint8_t* support) {
  const int gw = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
  const int nw = (int)((gridDim.x * blockDim.x) >> 6);
  for (int c = gw; c < count; c += nw) {
    const int i = __builtin_amdgcn_readfirstlane(list[c]);
    const NeuronRegs d = load_neuron(desc + i);
    const uint32_t sup = small_support_wave(d, neuron_sum_range(d));
    if ((threadIdx.x & 63) == 0) support[i] = (uint8_t)sup;
  }
}

hipError_t launch_support_params_small(const tt_neuron* desc, const int32_t* list, int count, uint8_t* support,
                                       hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const int blocks = (count + 3) / 4 < 4096 ? (count + 3) / 4 : 4096;
  hipLaunchKernelGGL(support_params_small_kernel, dim3(blocks), dim3(256), 0, s, desc, list, count, support);
  return hipGetLastError();
}

hipError_t launch_support_params(const tt_neuron* desc, const int32_t* list, int n, uint8_t* support,
                                 hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int blocks = n < 8192 ? n : 8192;
  hipLaunchKernelGGL(support_params_kernel, dim3(blocks), dim3(512), 0, s, desc, list, n, support);
  return hipGetLastError();
}

// Sixteen code bytes (any alignment) and the bits of one plane in them: a
// byte's bit weighted by its place, summed by four-byte dot products.
__device__ __forceinline__ uint4 load_codes16(const uint8_t* p) {
  uint4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}
template <int P>
__device__ __forceinline__ uint32_t plane_bits16(const uint4& c) {
  constexpr uint32_t m = 0x01010101u << P;
  auto byte = [](uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_udot4(lo & m, 0x08040201u, __builtin_amdgcn_udot4(hi & m, 0x80402010u, 0u, false), false) >> P;
  };
  return byte(c.x, c.y) | (byte(c.z, c.w) << 8);
}

// Pack: a wave takes up to 4096 rows of one neuron, 16 codes a lane and load
// (1 KiB runs), and turns them into 16 bits per plane, stored as a run of
// 128 bytes.  The tables' one-word planes are filled up with zeros.  Bound by
// HBM: 8191 uneven neurons, 69 MB of codes and 17 MB of planes, in 19 us
// (a byte per lane and a ballot per plane and word took 78 us, the wave's
// 64-byte loads one after the other).
__global__ __launch_bounds__(256) void pack_kernel(PackArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t it = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int k = 0;
  while (k < a.n_classes && it >= a.item_end[k]) ++k;
  if (k == a.n_classes) return;
  const int Fb = a.fb[k], sh = Fb > kPackRowsLog2 ? Fb - kPackRowsLog2 : 0;
  const int64_t first = it - (k > 0 ? a.item_end[k - 1] : 0);
  const PackRec r = a.rec[a.rec_begin[k] + (first >> sh)];
  const int o = (int)(r.code >> 62);
  const uint32_t R = 1u << Fb;
  const uint32_t r0 = (uint32_t)(first & ((1 << sh) - 1)) << kPackRowsLog2;
  const uint64_t W = words_per_plane(Fb);
  const uint8_t* codes = a.codes + (r.code & ~(3ull << 62));
  uint16_t* out = reinterpret_cast<uint16_t*>(a.tables + r.word_off);
  uint4 c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t row = r0 + 1024u * (uint32_t)i + 16u * (uint32_t)lane;
    c[i] = make_uint4(0u, 0u, 0u, 0u);
    if (row < R) {
      if (R >= 16u) {
        c[i] = load_codes16(codes + row);
      } else {  // (lane 0 of the first load)
        uint32_t w[2] = {0u, 0u};
        for (uint32_t t = 0; t < R; ++t) w[t >> 2] |= (uint32_t)codes[t] << (8 * (t & 3));
        c[i].x = w[0];
        c[i].y = w[1];
      }
    }
  }
  const uint32_t fill = max(R, 64u);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t row = r0 + 1024u * (uint32_t)i + 16u * (uint32_t)lane;
    if (row < fill) {
      uint16_t* q = out + (row >> 4);
      q[0] = (uint16_t)plane_bits16<0>(c[i]);
      if (o > 1) q[4 * W] = (uint16_t)plane_bits16<1>(c[i]);
      if (o > 2) q[8 * W] = (uint16_t)plane_bits16<2>(c[i]);
    }
  }
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_pack(const PackArgs& a, hipStream_t s) {
  if (a.n_classes <= 0) return hipSuccess;
  const int64_t items = a.item_end[a.n_classes - 1];
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace tt
