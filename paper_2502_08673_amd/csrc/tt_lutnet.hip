// tt_lutnet.hip -- a layered network of enumerated neurons evaluated through
// its packed truth tables (gfx950): lookups only, no arithmetic.
//
// Signals 0 .. n_inputs - 1 are primary input codes (uint8 per sample), and
// signal n_inputs + i is the output code of neuron i.  A neuron gathers its
// F input codes, forms the row r from their low b bits, and reads bit
// r % 64 of word r / 64 of each of its o planes.  Three forms: the whole
// network per block with the samples' signals in LDS (when a few dozen
// samples' signals fit), bytes for 64 samples or packed for 256 or 512, else
// one launch per level (a level reads only the primary inputs and earlier
// levels) with the signals in global memory.
#include <algorithm>
#include <utility>

#include "tt_internal.h"

namespace tt {

__global__ __launch_bounds__(256) void lutnet_level_kernel(LutnetArgs a) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)a.batch * a.count) return;
  const int s = (int)(t / a.count);
  const int i = a.level[t % a.count];
  const tt_neuron* dp = a.desc + i;
  const int F = dp->F, b = dp->b, o = dp->o;
  const uint32_t mask = (1u << b) - 1u;
  const int32_t* fi = a.fanin + 8 * (long)i;
  const uint8_t* in = a.inputs + (long)s * a.n_inputs;
  const uint8_t* prev = a.out + (long)s * a.n - a.n_inputs;  // prev[sig] for sig >= n_inputs
  uint32_t r = 0;
  for (int j = 0; j < F; ++j) {
    const int sig = fi[j];
    const uint32_t code = sig < a.n_inputs ? in[sig] : prev[sig];
    r |= (code & mask) << (j * b);
  }
  const int Fb = F * b;
  const uint64_t W = Fb >= 6 ? (1ull << (Fb - 6)) : 1ull;
  const uint64_t* t0 = a.tables + dp->word_off + (r >> 6);
  uint32_t q = 0;
  for (int p = 0; p < o; ++p) q |= (uint32_t)((t0[(uint64_t)p * W] >> (r & 63u)) & 1ull) << p;
  a.out[(long)s * a.n + i] = (uint8_t)q;
}

// Whole network per block: a block takes up to 64 samples, one per lane, and
// keeps their signal rows (n_inputs + n codes and one zero byte, the stride
// an odd number of dwords so that the 64 rows fall in distinct LDS banks) in
// LDS through all levels, with a barrier between levels.  A wave takes
// kNetStep neurons at a time: their records are wave-uniform (scalar loads,
// no chain of dependent loads), each lane reads the fan-in codes from its
// own row (FMAX reads, unused slots pointing at the zero byte, so no branch
// on F), and one load per lane returns the dword that holds the row's code,
// inside the neuron's table, which stays in cache.  The block writes its
// output rows at the end.
constexpr int kNetSamples = 64;
constexpr int kNetStep = 8;
constexpr int kNetThreads = 512;
constexpr long kNetMaxLds = 64 * 1024;
constexpr int kCopyRows = 8;  // rows per wave with their loads in flight together while staging

// Rows [0, rows) of `per_row` elements, contiguous at src, into LDS rows of
// `stride` bytes at dst, each element ANDed with its column's entry of
// colmask (when given).  Wave w takes rows w, w + waves, ... and lane l the
// columns l, l + 64, ...; a wave issues kCopyRows rows' loads before its
// first LDS store.  Rows up to `pad` are filled with zeros.
template <typename T>
__device__ __forceinline__ void rows_to_lds(const T* src, int rows, int pad, int per_row, uint8_t* dst, int stride,
                                            const T* colmask) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nw = blockDim.x >> 6;
  for (int c0 = 0; c0 < per_row; c0 += 64) {
    const int c = c0 + lane;
    const bool cok = c < per_row;
    const T m = colmask && cok ? colmask[c] : (T)~T(0);
    for (int r0 = wave; r0 < pad; r0 += nw * kCopyRows) {
      T v[kCopyRows];
#pragma unroll
      for (int u = 0; u < kCopyRows; ++u) {
        const int r = r0 + u * nw;
        v[u] = cok && r < rows ? src[(long)r * per_row + c] : T(0);
      }
#pragma unroll
      for (int u = 0; u < kCopyRows; ++u) {
        const int r = r0 + u * nw;
        if (cok && r < pad) reinterpret_cast<T*>(dst + r * stride)[c] = (T)(v[u] & m);
      }
    }
  }
}

// the reverse: LDS rows of `stride` bytes at src to contiguous rows at dst
template <typename T>
__device__ __forceinline__ void lds_to_rows(const uint8_t* src, int stride, int rows, int per_row, T* dst) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nw = blockDim.x >> 6;
  for (int c0 = 0; c0 < per_row; c0 += 64) {
    const int c = c0 + lane;
    const bool cok = c < per_row;
    for (int r0 = wave; r0 < rows; r0 += nw * kCopyRows) {
      T v[kCopyRows];
#pragma unroll
      for (int u = 0; u < kCopyRows; ++u) {
        const int r = r0 + u * nw;
        v[u] = cok && r < rows ? reinterpret_cast<const T*>(src + r * stride)[c] : T(0);
      }
#pragma unroll
      for (int u = 0; u < kCopyRows; ++u) {
        const int r = r0 + u * nw;
        if (cok && r < rows) dst[(long)r * per_row + c] = v[u];
      }
    }
  }
}

// SplitMix64 (Steele, Lea and Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014): output number k >= 1 of the stream seeded with
// seed, i.e. the finaliser applied to seed + k * golden gamma.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t k) {
  uint64_t z = seed + k * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <int FMAX, int OMAX, bool MASK>
__global__ __launch_bounds__(kNetThreads) void lutnet_fused_kernel(NetArgs a, const NetSample smp) {
  extern __shared__ uint8_t sig[];  // [kNetSamples][stride]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nwaves = blockDim.x >> 6;
  const long s0 = (long)blockIdx.x * kNetSamples;
  const int ns = (int)min((long)kNetSamples, (long)a.batch - s0);
  // the samples' input rows into LDS, each code reduced to the digits its
  // readers take when they all take the same number (then no reader masks).
  // Every lane looks tables up, so the rows past the batch are zeros: what
  // LDS held before would index past the tables.
  if (a.sample) {
    // drawn: bytes 8m .. 8m + 7 of row r are the bytes of output
    // (first + s0 + r) Q + m + 1 of the stream, masked per column.  With
    // Q < 64 draws per row a wave takes 64 / Q rows per pass (lane = sub Q +
    // m) and each lane's column mask is one 8-byte load, taken once; a whole
    // draw goes to LDS as two dword stores (rows are dword aligned)
    const int Q = (a.n_inputs + 7) >> 3;
    const bool wide = Q >= 64 || Q == 0;  // (no inputs: nothing to draw)
    const int RP = wide ? 1 : 64 / Q;  // rows per wave and pass
    const int sub = wide ? 0 : lane / Q;
    const int m0 = lane - sub * Q;
    if (sub < RP) {
      uint64_t mk0 = 0;
      if (m0 < Q && 8 * m0 + 8 <= a.n_inputs) mk0 = *reinterpret_cast<const uint64_t*>(a.in_mask + 8 * m0);
      for (int r = wave * RP + sub; r < kNetSamples; r += nwaves * RP)
        for (int m = m0; m < Q; m += 64) {
          // (rows past the batch take the draws that would follow: masked
          // as the others are, and not kept)
          const uint64_t z = splitmix64_at(smp.seed, (smp.first + (uint64_t)(s0 + r)) * (uint64_t)Q + m + 1);
          uint8_t* dst = sig + r * a.stride + 8 * m;
          if (8 * m + 8 <= a.n_inputs) {
            const uint64_t v = z & (m == m0 ? mk0 : *reinterpret_cast<const uint64_t*>(a.in_mask + 8 * m));
            reinterpret_cast<uint32_t*>(dst)[0] = (uint32_t)v;
            reinterpret_cast<uint32_t*>(dst)[1] = (uint32_t)(v >> 32);
          } else {
            for (int t = 0; 8 * m + t < a.n_inputs; ++t) dst[t] = (uint8_t)(z >> (8 * t)) & a.in_mask[8 * m + t];
          }
        }
    }
  } else if ((a.n_inputs & 3) == 0 && ((uintptr_t)a.inputs & 3) == 0) {
    rows_to_lds<uint32_t>(reinterpret_cast<const uint32_t*>(a.inputs + s0 * a.n_inputs), ns, kNetSamples,
                          a.n_inputs / 4, sig, a.stride, reinterpret_cast<const uint32_t*>(a.in_mask));
  } else {
    rows_to_lds<uint8_t>(a.inputs + s0 * a.n_inputs, ns, kNetSamples, a.n_inputs, sig, a.stride, a.in_mask);
  }
  if (threadIdx.x < kNetSamples) sig[threadIdx.x * a.stride + a.n_inputs + a.n] = 0;
  __syncthreads();
  const uint32_t rowb = (uint32_t)(lane * a.stride);
  for (int lv = 0; lv < a.depth; ++lv) {
    const int kb = a.level_begin[lv], count = a.level_begin[lv + 1] - kb;
    for (int k0 = wave * kNetStep; k0 < count; k0 += nwaves * kNetStep) {
      const NetRec* R[kNetStep];
#pragma unroll
      for (int u = 0; u < kNetStep; ++u) R[u] = a.rec + kb + min(k0 + u, count - 1);  // a repeat is not written
      uint32_t c[kNetStep][FMAX];
#pragma unroll
      for (int u = 0; u < kNetStep; ++u)
#pragma unroll
        for (int j = 0; j < FMAX; ++j) c[u][j] = sig[rowb + R[u]->sig[j]];
      constexpr int LW = OMAX <= 1 ? 0 : OMAX == 2 ? 1 : 2;
      uint32_t r[kNetStep], d[kNetStep];
#pragma unroll
      for (int u = 0; u < kNetStep; ++u) {
        const uint32_t mask = R[u]->mask, b = R[u]->b;
        uint32_t x = 0;
#pragma unroll
        for (int j = 0; j < FMAX; ++j) x |= (MASK ? c[u][j] & mask : c[u][j]) << (j * b);
        r[u] = x << LW;
        d[u] = a.tables[R[u]->tab + (x >> (5 - LW))];
      }
#pragma unroll
      for (int u = 0; u < kNetStep; ++u) {
        const uint32_t q = __builtin_amdgcn_ubfe(d[u], r[u], 1u << LW);
        // unconditional: a repeated neuron writes the value its first copy
        // writes, and lanes past the batch write rows that are never read out
        sig[rowb + R[u]->out] = (uint8_t)q;
      }
    }
    __syncthreads();
  }
  if (a.sample) {
    // wave 0 checks the targets of its lanes' draws, reserves places for the
    // kept ones with one atomic, and copies their input rows out together
    if (wave != 0) return;
    bool ok = lane < ns;
    for (int t = 0; t < smp.n_targets; ++t) ok = ok && sig[rowb + smp.tsig[t]] == smp.tval[t];
    const uint64_t kept = __ballot(ok);
    if (kept == 0) return;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(smp.count, (uint32_t)__popcll(kept));
    base = __shfl(base, 0);
    uint64_t rest = kept;
    for (uint64_t pos = base; rest != 0 && pos < (uint64_t)smp.max_found; ++pos) {
      const int l = __ffsll((unsigned long long)rest) - 1;
      rest &= rest - 1;
      for (int j = lane; j < a.n_inputs; j += 64) smp.found_inputs[pos * a.n_inputs + j] = sig[l * a.stride + j];
      if (lane == 0) smp.found_draw[pos] = smp.first + (uint64_t)(s0 + l);
    }
    return;
  }
  // output rows back: the block's rows are one contiguous run of the output
  if ((a.n & 3) == 0 && (a.n_inputs & 3) == 0 && ((uintptr_t)a.out & 3) == 0)
    lds_to_rows<uint32_t>(sig + a.n_inputs, a.stride, ns, a.n / 4, reinterpret_cast<uint32_t*>(a.out + s0 * a.n));
  else
    lds_to_rows<uint8_t>(sig + a.n_inputs, a.stride, ns, a.n, a.out + s0 * a.n);
}

// The packed form, for large batches: signals of BITS (2 or 4) bits, a signal
// row of 128 bytes in LDS for 1024 / BITS samples (33 dwords and one more
// every 64 rows: the 64 rows that a wave's lanes touch at one place while
// staging lie in 64 banks).  A wave takes a neuron for all of the block's
// samples, a lane 16 bits of each fan-in row: the rows of the table of its 8
// or 4 samples come from a few operations on all of them at once, and the
// neuron's table (at most 1 KiB, loaded two rounds ahead) is looked up in
// LDS.  The form above loads each code by itself and gathers from the cache,
// one address at a time per compute unit, which bounds it.  Here the bound is
// the LDS (eight gathers of 64 lanes in 64 banks, 54 of a neuron's 95 cycles)
// and the vector unit beside it (75 instructions a neuron and 512 samples);
// while all blocks load or write at once, HBM.  256 inputs, 448 neurons, F = 6,
// b = 2, 250001 samples: 73 us (that form: 133); 480 neurons of F = 4, b = 1,
// 262144 samples: 66.5 (98; 73 reading eight signals a neuron, as for F = 8);
// 60 of them: 12.6 (38.5).  Four waves that only write and load
// beside twelve that look up, with the next samples' inputs on the way: 73.
constexpr int kPackThreads = 64 * kPackWaves;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// LDS by its address: a pointer into the dynamic array costs an addition of
// its base (0) at every access
template <typename T>
__device__ __forceinline__ T lds_load(uint32_t byte) {
  return *(T __attribute__((address_space(3)))*)(uintptr_t)byte;
}
template <typename T>
__device__ __forceinline__ void lds_store(uint32_t byte, T v) {
  *(T __attribute__((address_space(3)))*)(uintptr_t)byte = v;
}

// bytes of four dwords transposed: out[t] = byte t of w[0], .. w[3]
__device__ __forceinline__ void transpose_bytes(const uint32_t (&w)[4], uint32_t (&out)[4]) {
  const uint32_t l01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), l23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
  const uint32_t h01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u), h23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
  out[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
}

// m ? x : y, bit by bit (as the instruction: from the expression the compiler
// makes three where it knows some of the bits)
__device__ __forceinline__ uint32_t select_bits(uint32_t m, uint32_t x, uint32_t y) {
  uint32_t r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(m), "v"(x), "v"(y));
  return r;
}

// The block's `left` rows of n codes into the signal rows 0, 1, ...; samples
// past the batch read its last row.  A thread takes a dword of samples of
// four signals (one signal, when a row is not made of aligned dwords): one
// dword per row.  A signal's dword holds row J k + j, J = 8 / BITS, in bits
// 8 k + BITS j.
template <int BITS>
__device__ __forceinline__ void pack_load(int n, const uint8_t* rows, uint32_t left) {
  constexpr int J = 8 / BITS, R = 4 * J;
  constexpr uint32_t kCode = (1u << BITS) - 1u, kCodes = 0x01010101u * kCode;
  const bool quads = (n & 3) == 0 && ((uintptr_t)rows & 3) == 0;
  const uint32_t cols = quads ? n / 4 : n;
  if (cols == 0) return;
  uint32_t g = threadIdx.x / cols, c = threadIdx.x - g * cols;
  const uint32_t dg = kPackThreads / cols, dc = kPackThreads - dg * cols;
  while (g < 32) {
    if (quads) {
      uint32_t d[R], v[4], t[4];
      if (left == 1024u / BITS) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          d[r] = *reinterpret_cast<const uint32_t*>(rows + (long)r * n + (__umul24(R * g, (uint32_t)n) + 4 * c));
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r)
          d[r] = *reinterpret_cast<const uint32_t*>(rows + (__umul24(min(R * g + r, left - 1), (uint32_t)n) + 4 * c));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[k] = d[J * k + J - 1];
#pragma unroll
        for (int j = J - 2; j >= 0; --j) v[k] = select_bits(kCodes, d[J * k + j], v[k] << BITS);
      }
      transpose_bytes(v, t);
#pragma unroll
      for (int q = 0; q < 4; ++q) lds_store<uint32_t>(net_row(4 * c + q) + 4 * g, t[q]);
    } else {
      uint32_t v = 0;
#pragma unroll
      for (int r = 0; r < R; ++r)
        v |= ((uint32_t)rows[__umul24(min(R * g + r, left - 1), (uint32_t)n) + c] & kCode) << (BITS * r);
      lds_store<uint32_t>(net_row(c) + 4 * g, v);
    }
    g += dg;
    c += dc;
    if (c >= cols) {
      c -= cols;
      ++g;
    }
  }
}

// The reverse: the n signal rows from sig0 on into the block's `left` rows
// (FULL: all of them) of codes.
template <int BITS, bool FULL>
__device__ __forceinline__ void pack_store(int sig0, int n, uint8_t* rows, uint32_t left) {
  constexpr int J = 8 / BITS, R = 4 * J;
  constexpr uint32_t kCode = (1u << BITS) - 1u, kCodes = 0x01010101u * kCode;
  const bool quads = (n & 3) == 0 && ((uintptr_t)rows & 3) == 0;
  const uint32_t cols = quads ? n / 4 : n;
  uint32_t g = threadIdx.x / cols, c = threadIdx.x - g * cols;
  const uint32_t dg = kPackThreads / cols, dc = kPackThreads - dg * cols;
  while (g < 32) {
    const uint32_t r0 = R * g;
    if (quads) {
      uint32_t v[4], t[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = lds_load<uint32_t>(net_row(sig0 + 4 * c + q) + 4 * g);
      transpose_bytes(v, t);
      const uint32_t at = __umul24(r0, (uint32_t)n) + 4 * c;
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (FULL || r0 + r < left)
          *reinterpret_cast<uint32_t*>(rows + (long)r * n + at) = (t[r / J] >> (BITS * (r % J))) & kCodes;
    } else {
      const uint32_t v = lds_load<uint32_t>(net_row(sig0 + c) + 4 * g), at = __umul24(r0, (uint32_t)n) + c;
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (FULL || r0 + r < left) rows[(long)r * n + at] = (uint8_t)((v >> (BITS * r)) & kCode);
    }
    g += dg;
    c += dc;
    if (c >= cols) {
      c -= cols;
      ++g;
    }
  }
}

// dword i of a NetSlot held one dword a lane in each row of 16 lanes
__device__ __forceinline__ uint32_t slot_word(uint32_t rec, int i) {
  return (uint32_t)__builtin_amdgcn_readlane((int)rec, i);
}
template <int I>
__device__ __forceinline__ uint32_t slot_bcast(uint32_t rec) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)rec, 0x150 + I, 0xF, 0xF, true);  // row_newbcast
}

// Rows x[4] of the table from four samples' nibbles: a holds index words 0
// and 2 (16 bits each), c words 1 and 3; a sample's nibbles side by side.
__device__ __forceinline__ void join_nibbles(uint32_t a, uint32_t c, bool wide, uint32_t& x0, uint32_t& x1,
                                             uint32_t& x2, uint32_t& x3) {
  const uint32_t e = select_bits(0x0F0F0F0Fu, a, c << 4), o = select_bits(0xF0F0F0F0u, c, a >> 4);
  if (wide) {
    x0 = __builtin_amdgcn_perm(0u, e, 0x0C0C0200u);
    x1 = __builtin_amdgcn_perm(0u, o, 0x0C0C0200u);
    x2 = __builtin_amdgcn_perm(0u, e, 0x0C0C0301u);
    x3 = __builtin_amdgcn_perm(0u, o, 0x0C0C0301u);
  } else {
    x0 = e & 255u;
    x1 = o & 255u;
    x2 = e >> 8;
    x3 = o >> 8;
  }
}

// the lane's 16 bits of each fan-in row
template <int N, int... I>
__device__ __forceinline__ void load_fanin(uint32_t rec, uint32_t lane2, uint32_t (&u)[N],
                                           std::integer_sequence<int, I...>) {
  ((u[I] = lds_load<uint16_t>(slot_bcast<8 + I>(rec) + lane2)), ...);
}

// Rows of the table of the lane's 16 / BITS samples (its 16 bits of each
// fan-in row): the digits, 4 / B a nibble, joined within the M index words
// of all samples first, then the nibbles of each sample.
template <int BITS, int B, int M>
__device__ __forceinline__ void pack_index(uint32_t rec, uint32_t lane2, uint32_t (&x)[16 / BITS]) {
  constexpr int K = B == 1 ? 4 : B == 2 ? 2 : 1;
  uint32_t u[K * M];
  load_fanin(rec, lane2, u, std::make_integer_sequence<int, K * M>{});
  if constexpr (BITS == 4) {
    constexpr uint32_t kDigit = 0x1111u * ((1u << B) - 1u);
    uint32_t P[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
      for (int k = 0; k < K; ++k) P[i] |= (u[i * K + k] & kDigit) << (k * B);
    if constexpr (B == 3) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        x[s] = 0;
#pragma unroll
        for (int i = 0; i < M; ++i) x[s] |= ((P[i] >> (4 * s)) & 7u) << (3 * i);
      }
    } else {
      join_nibbles(P[0] | P[2] << 16, P[1] | P[3] << 16, M > 2, x[0], x[1], x[2], x[3]);
    }
  } else {
    // two-bit digits first: even and odd samples' nibbles from pairs of them
    uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 2 * M; ++i) w[i] = B == 2 ? u[i] : select_bits(0x5555u, u[2 * i], u[2 * i + 1] << 1) & 0xFFFFu;
    const uint32_t a = w[0] | w[4] << 16, b = w[1] | w[5] << 16, c = w[2] | w[6] << 16, d = w[3] | w[7] << 16;
    join_nibbles(select_bits(0x33333333u, a, b << 2), select_bits(0x33333333u, c, d << 2), M > 2, x[0], x[2], x[4],
                 x[6]);
    join_nibbles(select_bits(0xCCCCCCCCu, b, a >> 2), select_bits(0xCCCCCCCCu, d, c >> 2), M > 2, x[1], x[3], x[5],
                 x[7]);
  }
}

template <int BITS, int B, int M, int LW>
__global__ __launch_bounds__(kPackThreads, 8) void lutnet_packed_kernel(NetArgs a, uint32_t tables_at) {
  // dynamic LDS, from byte 0 on: signal rows, then a table per wave
  constexpr int kAhead = kPackRounds / 2;  // tables on the way; records on the way: twice as many
  constexpr int S = 16 / BITS;
  constexpr uint32_t kRows = 1024 / BITS;
  const int lane = threadIdx.x & 63;
  const uint32_t lane2 = 2 * lane, lane16 = 16 * lane;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const long s0 = (long)blockIdx.x * kRows;
  const uint32_t left = (uint32_t)min((long)kRows, (long)a.batch - s0);
  const uint32_t tab = tables_at + wave * kPackTable;
  const uint32_t* slots = reinterpret_cast<const uint32_t*>(a.slots + wave) + (lane & 15);
  const uint8_t* tables = reinterpret_cast<const uint8_t*>(a.tables);
  uint32_t recs[kPackRounds];
  u32x4 ahead[kAhead];
  auto fetch = [&](uint32_t rec) {
    return *reinterpret_cast<const u32x4*>(tables + (slot_bcast<0>(rec) + min(lane16, slot_bcast<1>(rec))));
  };
#pragma unroll
  for (int u = 0; u < kPackRounds; ++u) recs[u] = slots[u * (kPackWaves * 16)];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) ahead[u] = fetch(recs[u]);
  pack_load<BITS>(a.n_inputs, a.inputs + s0 * a.n_inputs, left);
  if (threadIdx.x < 32) lds_store<uint32_t>(net_row(a.n_inputs + a.n) + 4 * threadIdx.x, 0u);
  __syncthreads();
  for (int t = 0; t < a.rounds; t += kPackRounds) {
    slots += kPackRounds * kPackWaves * 16;
#pragma unroll
    for (int u = 0; u < kPackRounds; ++u) {
      const uint32_t rec = recs[u], flags = slot_word(rec, 3);
      const u32x4 table = ahead[u % kAhead];
      ahead[u % kAhead] = fetch(recs[(u + kAhead) % kPackRounds]);
      if (flags & 1u) {
        lds_store<u32x4>(tab + lane16, table);
        __builtin_amdgcn_wave_barrier();
        uint32_t x[S], d[S], q = 0;
        pack_index<BITS, B, M>(rec, lane2, x);
#pragma unroll
        for (int s = 0; s < S; ++s) d[s] = lds_load<uint32_t>(select_bits(kPackTable - 4u, x[s] >> (3 - LW), tab));
#pragma unroll
        for (int s = 0; s < S; ++s) q |= __builtin_amdgcn_ubfe(d[s], x[s] << LW, 1u << LW) << (BITS * s);
        lds_store<uint16_t>(slot_bcast<2>(rec) + lane2, (uint16_t)q);
        __builtin_amdgcn_wave_barrier();
      }
      recs[u] = slots[u * (kPackWaves * 16)];
      if (flags & 2u) __syncthreads();
    }
  }
  if (left == kRows)
    pack_store<BITS, true>(a.n_inputs, a.n, a.out + s0 * a.n, left);
  else
    pack_store<BITS, false>(a.n_inputs, a.n, a.out + s0 * a.n, left);
}

// Dword g of the copy: the codes of rows (32 >> lw) g and on, bit p of a code
// from plane p (bits of a plane spread 2^lw apart).
__device__ __forceinline__ uint32_t code_dword(const uint32_t* src, uint64_t plane, uint32_t g, int o, int lw) {
  if (lw == 0) return src[g];
  uint32_t v = 0;
  for (int p = 0; p < o; ++p) {
    const uint32_t w = src[p * plane + (g >> lw)];
    uint32_t x = lw == 1 ? (w >> (16 * (g & 1u))) & 0xFFFFu : (w >> (8 * (g & 3u))) & 0xFFu;
    if (lw == 1) {
      x = (x | x << 8) & 0x00FF00FFu;
      x = (x | x << 4) & 0x0F0F0F0Fu;
      x = (x | x << 2) & 0x33333333u;
      x = (x | x << 1) & 0x55555555u;
    } else {
      x = (x | x << 12) & 0x000F000Fu;
      x = (x | x << 6) & 0x03030303u;
      x = (x | x << 3) & 0x11111111u;
    }
    v |= x << p;
  }
  return v;
}

__global__ __launch_bounds__(256) void lutnet_repack_kernel(const RepackItem* items, int n, int lw,
                                                            const uint64_t* tables, uint32_t* il) {
  for (int k = blockIdx.x; k < n; k += gridDim.x) {
    const RepackItem it = items[k];
    const uint32_t* src = reinterpret_cast<const uint32_t*>(tables + it.src_word);
    for (uint32_t g = threadIdx.x; g < it.dwords; g += blockDim.x)
      il[it.dst_dword + g] = code_dword(src, 2ull * it.W, g, (int)it.o, lw);
  }
}

hipError_t launch_lutnet_repack(const RepackItem* items, int n, int lw, const uint64_t* tables, uint32_t* il,
                                hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(lutnet_repack_kernel, dim3((unsigned)std::min(n, 4096)), dim3(256), 0, s, items, n, lw, tables,
                     il);
  return hipGetLastError();
}

template <int BITS, int B, int M, int LW>
hipError_t launch_packed(const NetArgs& a, hipStream_t s) {
  const int samples = 1024 / BITS;
  const unsigned blocks = (unsigned)(((long)a.batch + samples - 1) / samples);
  const uint32_t tables_at = (uint32_t)net_pack_tables_at(a.n_inputs + a.n);
  const size_t lds = (size_t)net_pack_lds(a.n_inputs + a.n);
  const auto kernel = lutnet_packed_kernel<BITS, B, M, LW>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kPackThreads), lds, s, a, tables_at);
  return hipGetLastError();
}

hipError_t launch_lutnet_packed(const NetArgs& a, hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  if (net_pack_samples(a.omax, a.digit) == 512) {
    const bool one = a.lw == 0;
    if (a.digit == 1 && a.fmax <= 4) return one ? launch_packed<2, 1, 1, 0>(a, s) : launch_packed<2, 1, 1, 1>(a, s);
    if (a.digit == 1) return one ? launch_packed<2, 1, 2, 0>(a, s) : launch_packed<2, 1, 2, 1>(a, s);
    if (a.fmax <= 4) return one ? launch_packed<2, 2, 2, 0>(a, s) : launch_packed<2, 2, 2, 1>(a, s);
    return one ? launch_packed<2, 2, 3, 0>(a, s) : launch_packed<2, 2, 3, 1>(a, s);
  }
  switch (a.digit * 4 + a.lw) {
    case 6: return a.fmax <= 4 ? launch_packed<4, 1, 1, 2>(a, s) : launch_packed<4, 1, 2, 2>(a, s);
    case 10: return launch_packed<4, 2, 3, 2>(a, s);
    case 12: return launch_packed<4, 3, 4, 0>(a, s);
    case 13: return launch_packed<4, 3, 4, 1>(a, s);
    case 14: return launch_packed<4, 3, 4, 2>(a, s);
    case 16: return launch_packed<4, 4, 3, 0>(a, s);
    case 17: return launch_packed<4, 4, 3, 1>(a, s);
    default: return launch_packed<4, 4, 3, 2>(a, s);
  }
}

long lutnet_fused_stride(int n_inputs, int n) {
  // the signals and the zero byte, rounded to an odd number of dwords
  long stride = ((long)n_inputs + n + 1 + 3) / 4 * 4;
  if ((stride / 4) % 2 == 0) stride += 4;
  return kNetSamples * stride <= kNetMaxLds ? stride : 0;
}

hipError_t launch_lutnet_fused(const NetArgs& a, const NetSample& smp, hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  const long blocks = ((long)a.batch + kNetSamples - 1) / kNetSamples;
  const size_t lds = (size_t)kNetSamples * a.stride;
  const int fk = (a.fmax + 1) / 2;  // FMAX rounded up to even: 2, 4, 6, 8
#define TT_NET_LAUNCH(FM, OM)                                                                          \
  if (a.mask)                                                                                          \
    hipLaunchKernelGGL((lutnet_fused_kernel<FM, OM, true>), dim3((unsigned)blocks), dim3(kNetThreads), \
                       lds, s, a, smp);                                                                     \
  else                                                                                                 \
    hipLaunchKernelGGL((lutnet_fused_kernel<FM, OM, false>), dim3((unsigned)blocks), dim3(kNetThreads), \
                       lds, s, a, smp);                                                                     \
  break
#define TT_NET_O(FM)                \
  switch (a.omax) {                 \
    case 1: TT_NET_LAUNCH(FM, 1);   \
    case 2: TT_NET_LAUNCH(FM, 2);   \
    default: TT_NET_LAUNCH(FM, 3);  \
  }                                 \
  break
  switch (fk) {
    case 1: TT_NET_O(2);
    case 2: TT_NET_O(4);
    case 3: TT_NET_O(6);
    default: TT_NET_O(8);
  }
#undef TT_NET_O
#undef TT_NET_LAUNCH
  return hipGetLastError();
}

hipError_t launch_lutnet_level(const LutnetArgs& a, hipStream_t s) {
  const long threads = (long)a.batch * a.count;
  if (threads <= 0) return hipSuccess;
  hipLaunchKernelGGL(lutnet_level_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace tt
