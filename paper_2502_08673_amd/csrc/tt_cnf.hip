// tt_cnf.hip -- the CNF-to-circuit transformation (Section "Transformation
// Algorithm", Algorithm 1) on packed truth tables (gfx950): eight instances a
// wave while SC stays within five variables (cnf_fast_kernel), else one wave
// per instance (cnf_transform_kernel), as follows.
//
// A wave walks its instance's clauses in order, growing the sub-clause list
// SC (a contiguous clause range, since SC is emptied whenever an expression
// is found).  After each clause it tries the variables of SC that are
// neither primary inputs nor intermediate, in decreasing index: lane w
// builds word w (rows 64w .. 64w + 63) of f (the conjunction of the clauses
// holding -v, that literal removed) and of g (the same for +v) over the
// other variables of SC, ascending index = ascending row digit, straight
// from literal bit patterns; the complement test is an XOR per word and one
// ballot.  A found expression is written with its table and its support
// (digit j is in the support when some pair of rows differing in digit j
// differs: a shifted XOR inside a word for j < 6, a lane exchange for
// j >= 6).  An SC with no output whose variables occur in no later clause
// becomes an auxiliary output constrained to 1 (the conjunction of SC).
#include <stddef.h>

#include <algorithm>

#include "tt_internal.h"

namespace tt {

namespace {

constexpr uint8_t kClsPI = 1, kClsIV = 2, kClsPO = 4;

// rows whose digit j is 1, for j < 6 (inside one 64-row word)
__device__ __forceinline__ uint64_t digit_pattern(int j) {
  switch (j) {
    case 0: return 0xAAAAAAAAAAAAAAAAull;
    case 1: return 0xCCCCCCCCCCCCCCCCull;
    case 2: return 0xF0F0F0F0F0F0F0F0ull;
    case 3: return 0xFF00FF00FF00FF00ull;
    case 4: return 0xFFFF0000FFFF0000ull;
    default: return 0xFFFFFFFF00000000ull;
  }
}

// word w of the literal on digit j (negated when neg)
__device__ __forceinline__ uint64_t literal_word(int j, int w, bool neg) {
  const uint64_t p = j < 6 ? digit_pattern(j) : (((w >> (j - 6)) & 1) ? ~0ull : 0ull);
  return neg ? ~p : p;
}

__device__ __forceinline__ uint64_t shfl_xor64(uint64_t x, int m) {
  const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, m);
  const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}

// Support over k digits of a table held as words (lane w < W holds word w,
// valid = the rows that exist in a one-word table).
__device__ uint32_t table_support(uint64_t t, int k, int W, uint64_t valid) {
  const int lane = threadIdx.x;
  uint32_t sup = 0;
  for (int j = 0; j < k; ++j) {
    bool d;
    if (j < 6) {
      const int s = 1 << j;
      d = lane < W && (((t ^ (t >> s)) & ~digit_pattern(j) & valid) != 0);
    } else {
      const uint64_t o = shfl_xor64(t, 1 << (j - 6));
      d = lane < W && t != o;
    }
    if (__ballot(d) != 0) sup |= 1u << j;
  }
  return sup;
}

}  // namespace

namespace {

// ---------------------------------------------------- eight instances a wave
// SC of at most kCnfFastVars variables (the gate encodings of circuits put a
// gate and its inputs in one SC: four or so): every table fits one 32-bit
// word, so a wave per instance would leave 63 lanes without a table word.
// Here eight lanes take an instance.  They read a clause's literals side by
// side, find each one's digit (the order of first use in SC) in a byte per
// variable in LDS and combine their patterns into the clause's word; a word
// over fewer variables is independent of the other digits, so appending a
// variable changes no word.  Lane q also is SC's q-th variable: with A the
// conjunction of SC's clauses and N and P those of the clauses holding the
// variable negated and plain, every lane tests its own variable as the
// output after each clause: f = N at v = 1 and g = P at v = 0 drop v's own
// literals, and v is the output when they differ in every row.  What is
// found goes to a list in LDS in this form.  When the list is full the
// block's second wave takes it, while the first goes on with another one:
// one lane per entry sorts the digits by variable (a sorting network, each
// exchange a swap of two digits of the word) and the wave writes the records
// in whole lines.
constexpr int kCnfFastVars = 5;
// Literals that a clause's record holds: a clause of more than kCnfFastVars
// is never walked by eight lanes, and shows it by a variable too many.
constexpr int kCnfRecLits = kCnfFastVars + 1;
constexpr int kCnfList = 64;      // entries of the two-wave kernel's lists
constexpr int kCnfWaveList = 16;  // and of the wave kernel's
constexpr int kCnfSweep = 8192;  // blocks that look for instances left over (more for more than twice as many)
constexpr uint32_t kNoVar = 0x8000u;
// A variable's byte in LDS: its class bits, and its digit in SC plus one
// (zero: not in SC) from bit 3 up.
constexpr int kDigitShift = 3;
constexpr uint32_t kClassBits = (1u << kDigitShift) - 1u;

template <int N>
struct alignas(16) CnfList {
  uint32_t tab[N];        // f (v's digit dropped) or SC's conjunction
  uint16_t var[N][8];     // variable of digit q; kNoVar: none, or v
  int32_t rec[N], first[N], last[N], out[N];
  int32_t count, more;    // entries; whether another list follows
};
static_assert(sizeof(CnfList<kCnfList>) % 16 == 0 && offsetof(CnfList<kCnfList>, var) % 16 == 0 &&
                  offsetof(CnfList<kCnfWaveList>, var) % 16 == 0,
              "var's rows are read as uint4");

// The lane, as a value that the compiler does not know: what is made from it
// in one phase of a loop is not kept in registers through the others.
__device__ __forceinline__ int lane_here() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// over the eight lanes of a group: quad permutes by 1 and 2, then the mirror
// of half a row
__device__ __forceinline__ uint32_t or8(uint32_t x) {
  x |= dpp<0xB1>(x);
  x |= dpp<0x4E>(x);
  x |= dpp<0x141>(x);
  return x;
}
__device__ __forceinline__ uint32_t max8(uint32_t x) {
  x = max(x, dpp<0xB1>(x));
  x = max(x, dpp<0x4E>(x));
  x = max(x, dpp<0x141>(x));
  return x;
}

__device__ __forceinline__ uint32_t digit_pattern32(int j) { return (uint32_t)digit_pattern(j); }

// digits A < B of the table and their variables exchanged when out of order
template <int A, int B>
__device__ __forceinline__ void order_digits(uint32_t (&v)[kCnfFastVars], uint32_t& t) {
  const uint32_t m = digit_pattern32(A) & ~digit_pattern32(B);
  uint32_t x = (t ^ (t >> ((1 << B) - (1 << A)))) & m;
  x = v[A] > v[B] ? x : 0u;
  t ^= x | (x << ((1 << B) - (1 << A)));
  const uint32_t lo = min(v[A], v[B]), hi = max(v[A], v[B]);
  v[A] = lo;
  v[B] = hi;
}

// The list's records to memory, by one wave; heads: 80 bytes of LDS a record.
template <int N>
__device__ __forceinline__ void cnf_flush(CnfList<N>& L, uint4 (*heads)[5], tt_cnf_expr* expr) {
  const int lane = lane_here();
  const int count = __builtin_amdgcn_readfirstlane(L.count);
  if (lane < count) {
    const uint4 vv = *reinterpret_cast<const uint4*>(&L.var[lane][0]);
    uint32_t v[kCnfFastVars] = {vv.x & 0xFFFFu, vv.x >> 16, vv.y & 0xFFFFu, vv.y >> 16, vv.z & 0xFFFFu};
    uint32_t t = L.tab[lane];
    order_digits<0, 3>(v, t);
    order_digits<1, 4>(v, t);
    order_digits<0, 2>(v, t);
    order_digits<1, 3>(v, t);
    order_digits<0, 1>(v, t);
    order_digits<2, 4>(v, t);
    order_digits<1, 2>(v, t);
    order_digits<3, 4>(v, t);
    order_digits<2, 3>(v, t);
    uint32_t k = 0, sup = 0;
#pragma unroll
    for (int j = 0; j < kCnfFastVars; ++j) {
      const bool used = v[j] != kNoVar;
      k += used ? 1u : 0u;
      // t does not depend on the digits past its variables
      if (((t ^ (t >> (1 << j))) & ~digit_pattern32(j)) != 0u) sup |= 1u << j;
      v[j] = used ? v[j] : 0u;
    }
    const uint32_t out = (uint32_t)L.out[lane];
    const uint32_t kind = out == 0u ? TT_CNF_AUX : (t == 0u || t == ~0u) ? TT_CNF_PO : TT_CNF_IV;
    L.tab[lane] = k >= 5u ? t : t & ((1u << (1u << k)) - 1u);
    heads[lane][0] = make_uint4(out, kind, (uint32_t)L.first[lane], (uint32_t)L.last[lane]);
    heads[lane][1] = make_uint4(k, sup, v[0], v[1]);
    heads[lane][2] = make_uint4(v[2], v[3], v[4], 0u);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // heads: eight lanes a record, 16 bytes each (the unused bytes as zeros, so
  // that whole lines are written)
#pragma unroll 2
  for (int e0 = 0; e0 < count; e0 += 8) {
    const int e = e0 + (lane >> 3), p = lane & 7;
    if (e < count)
      reinterpret_cast<uint4*>(expr + L.rec[e])[p] = p < 3 ? heads[e][p] : make_uint4(0u, 0u, 0u, 0u);
  }
  // tables: half a wave a record; word 0 holds the rows, the others are zero
#pragma unroll 4
  for (int e0 = 0; e0 < count; e0 += 2) {
    const int e = e0 + (lane >> 5), p = lane & 31;
    if (e < count)
      reinterpret_cast<uint4*>(expr[L.rec[e]].table)[p] = make_uint4(p == 0 ? L.tab[e] : 0u, 0u, 0u, 0u);
  }
}

}  // namespace

// A clause as eight 16-bit values: its first kCnfRecLits literals (zero past
// the last) and in 6 the last clause of its instance that uses any of its
// variables.
__global__ __launch_bounds__(256) void cnf_clause_kernel(const int32_t* lits, const int32_t* clause_off,
                                                         const int32_t* reach, int n_clauses, uint4* rec) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= n_clauses) return;
  const int p = clause_off[c], len = clause_off[c + 1] - p;
  uint32_t v[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = t < kCnfRecLits && t < len ? (uint32_t)lits[p + t] & 0xFFFFu : 0u;
  v[6] = (uint32_t)reach[c] & 0xFFFFu;
  rec[c] = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
}

// The walk of a group of eight lanes over its instance's clauses from i0 on
// (the same for every live group of the wave), until the instance ends or SC
// outgrows kCnfFastVars variables (pending: start is the clause that SC began
// with, and its variables' digits are cleared).  cls, sc and recs are the
// group's: a byte per variable, SC's variables by digit and eight clauses.
// Entries go to *list, `listed` so far; full() takes a list that has no room
// for a round of eight more and returns the next one.  ONE: only the wave's
// first group walks (the others come with nc = 0 and its LDS), and it returns
// when the list has no room (start: the next clause).
template <bool ONE, int N, typename Full>
__device__ __forceinline__ void cnf_narrow_walk(const uint4* rec, int c0, int nc, int i0, uint8_t* cls,
                                                uint16_t* sc, uint4* recs, CnfList<N>*& list, int& listed, int& start,
                                                int& nexpr, bool& pending, Full full) {
  const int lane = lane_here(), q = lane & 7;
  const uint32_t pat = digit_pattern32(q < kCnfFastVars ? q : kCnfFastVars - 1);
  // eight clauses at a time, one a lane, in LDS; the next eight in registers
  // (loaded eight clauses ahead)
  const int i8 = (i0 & ~7) + q;
  uint4 ahead = i8 < nc ? rec[i8] : make_uint4(0u, 0u, 0u, 0u);
  uint32_t A = ~0u, Nv = ~0u, P = ~0u;
  uint32_t blocked = 0;  // not zero: SC's q-th variable is a primary input or intermediate
  int nsc = 0, reach = -1;
  start = i0;
  pending = false;
  bool run = i0 < nc;
  int word = 0, creach = 0;  // lane q's 16 bits of the clause (literal q), and its reach
  if (!ONE || lane < 8) sc[q] = 0;
  auto fetch = [&](int i, bool first) {
    if ((i & 7) == 0 || first) {
      if (!ONE || lane < 8) recs[q] = ahead;
      const int next = (i & ~7) + 8 + q;
      if (next < nc) ahead = rec[next];
    }
    const uint16_t* cl = reinterpret_cast<const uint16_t*>(&recs[i & 7]);
    word = (int)(int16_t)cl[q];
    creach = (int)cl[6];
  };
  fetch(i0, true);
  for (int i = i0; __any(run); ++i) {
    const int lit = run && q < kCnfRecLits ? word : 0;
    const int here = creach;
    // the literals' digits; variables new to SC take the next ones
    const int x = lit < 0 ? -lit : lit;
    const uint32_t byte = cls[x];
    fetch(i + 1, false);  // in flight with the byte
    const uint32_t have = byte >> kDigitShift;
    const bool add = lit != 0 && have == 0u;
    const uint32_t adds = (uint32_t)(__ballot(add) >> (lane & 56)) & 0xFFu;
    const int digit = add ? nsc + __popc(adds & ((1u << q) - 1u)) : (int)have - 1;
    nsc += __popc(adds);
    if (run && nsc > kCnfFastVars) {
      pending = true;
      run = false;
    }
    const bool use = run && lit != 0;
    if (use && add) {
      cls[x] = (uint8_t)(byte | (uint32_t)(digit + 1) << kDigitShift);
      sc[digit] = (uint16_t)x;
    }
    // lane q's variable and its byte, wanted if something is found: read
    // here, so that they arrive while the words are combined
    const bool mine = run && q < nsc;
    const uint32_t my = mine ? sc[q] : 0u;
    const uint32_t my_cls = cls[my] & kClassBits;
    const uint32_t lp = digit & 4 ? 0xFFFF0000u
                                  : (digit & 2 ? (digit & 1 ? 0xFF00FF00u : 0xF0F0F0F0u)
                                               : (digit & 1 ? 0xCCCCCCCCu : 0xAAAAAAAAu));
    const uint32_t C = or8(use ? lp ^ (uint32_t)(lit >> 31) : 0u);
    // bits of the clause's variables: plain, negated, and (new ones) blocked
    uint32_t bits = use ? (lit > 0 ? 1u : 0x100u) : 0u;
    bits |= use && add && (byte & (kClsPI | kClsIV)) ? 0x10000u : 0u;
    bits = or8(bits << (digit & 7)) >> q;
    if (run) {
      A &= C;
      Nv &= C | (((bits >> 8) & 1u) - 1u);
      P &= C | ((bits & 1u) - 1u);
      blocked |= bits & 0x10000u;
      reach = max(reach, here);
    }
    // the candidates, each its own variable; the largest that passes
    const bool ok = mine && blocked == 0u && (((Nv >> (1 << q)) ^ P) | pat) == ~0u;
    const bool any_ok = ((uint32_t)(__ballot(ok) >> (lane & 56)) & 0xFFu) != 0u;
    const bool found = any_ok || (run && reach <= i);
    // one entry a group that found something
    const uint64_t who = __ballot(found && q == 0);
    run = run && i + 1 < nc;
    if (who == 0ull) continue;
    CnfList<N>& L = *list;
    const int at = listed + __popcll(who & ((1ull << (lane & 56)) - 1ull));
    const uint32_t v = max8(ok ? my : 0u);
    if (found) {
      const bool win = mine && my == v;
      const uint32_t n1 = Nv & pat;
      const uint32_t f = any_ok ? n1 | (n1 >> (1 << q)) : A;
      if (any_ok ? win : q == 0) {
        L.tab[at] = f;
        L.rec[at] = c0 + nexpr;
        L.first[at] = start;
        L.last[at] = i;
        L.out[at] = (int32_t)v;
      }
      L.var[at][q] = (uint16_t)(mine && !win ? my : kNoVar);
      if (mine) {
        const uint32_t mark = win ? (f == 0u || f == ~0u ? kClsPO : kClsIV) : (my_cls & kClsIV ? 0u : kClsPI);
        cls[my] = (uint8_t)(my_cls | mark);
      }
      ++nexpr;
      start = i + 1;
      reach = -1;
      nsc = 0;
      blocked = 0;
      A = Nv = P = ~0u;
    }
    listed += __popcll(who);
    if (listed > N - 8) {
      if constexpr (ONE) return;
      list = full(list, listed);
      listed = 0;
    }
  }
  // (every place of sc: those past SC's hold variables without a digit)
  if (pending) cls[sc[q]] &= (uint8_t)kClassBits;
}

// The first n_fast instances of the order (fewer than 2^16 clauses, few
// variables): eight to a block of two waves, the first walking, the second
// writing.  An instance whose SC outgrows kCnfFastVars variables stops there:
// cnf_transform_kernel goes on from the clause that this SC began with, with
// the classes and expressions so far.  Bound by the chain of the longest
// instances' clauses, about 200 instructions and 0.55 us each: 20000 circuits
// of 8 to 64 gates take 0.158 ms, 16 of them 0.14 ms (a wave each: 1.38 and
// 0.47 ms); without its stores, 0.5 GB, it takes 0.150 ms.
__global__ __launch_bounds__(128) void cnf_fast_kernel(CnfArgs a) {
  __shared__ CnfList<kCnfList> lists[2];
  __shared__ uint4 heads[kCnfList][5];
  __shared__ uint16_t s_sc[8][8];     // per instance: SC's variables by digit
  __shared__ uint4 s_rec[8][8];       // per instance: the clauses i .. i + 7
  extern __shared__ uint8_t s_cls[];  // a byte per variable, [8][cls_stride]
  const int lane = threadIdx.x & 63, q = lane & 7, g = lane >> 3;
  if (__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) == 1) {
    // the writer: list k when the walker has filled it (barrier k); the
    // walker fills the other one meanwhile
    for (int k = 0;; ++k) {
      __syncthreads();
      CnfList<kCnfList>& L = lists[k & 1];
      const bool more = __builtin_amdgcn_readfirstlane(L.more) != 0;
      cnf_flush(L, heads, a.expr);
      if (!more) return;
    }
  }
  const int slot = blockIdx.x * 8 + g;
  const bool live = slot < a.n_fast;
  const int inst = live ? a.order[slot] : 0;
  const int nvar = live ? a.n_vars[inst] : -1;
  const int c0 = live ? a.inst_off[inst] : 0;
  const int nc = live ? a.inst_off[inst + 1] - c0 : 0;
  uint8_t* cls = s_cls + g * a.cls_stride;
  for (int x = q; x <= nvar; x += 8) cls[x] = 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  CnfList<kCnfList>* list = &lists[0];
  int listed = 0, start = 0, nexpr = 0;
  bool pending = false;
  cnf_narrow_walk<false>(a.clause_rec + c0, c0, nc, 0, cls, s_sc[g], s_rec[g], list, listed, start, nexpr, pending,
                         [&](CnfList<kCnfList>* L, int count) {
                           if (lane == 0) {
                             L->count = count;
                             L->more = 1;
                           }
                           __syncthreads();  // the writer has this list now and is done with the other
                           return L == &lists[0] ? &lists[1] : &lists[0];
                         });
  if (lane == 0) {
    list->count = listed;
    list->more = 0;
  }
  __syncthreads();
  if (!live) return;
  for (int x = q; x <= nvar; x += 8) a.var_class[a.var_off[inst] + x] = cls[x];
  if (q == 0) {
    a.n_expr[inst] = nexpr;
    a.status[inst] = 0;
    a.left[slot] = pending ? start + 1 : 0;
  }
}

// What the wave kernel's eight-lane walk keeps in LDS.
struct CnfWaveLds {
  CnfList<kCnfWaveList> list;
  uint4 heads[kCnfWaveList][5];
  uint4 rec[8];
  uint16_t sc[8];
};

// One instance by one wave from clause `first` on (first > 0: with the classes
// and the number of expressions that the outputs hold).  The form
// described at the head of this file, a word of every table a lane; where the
// instance allows it (narrow), eight lanes walk on after each expression that
// this form found, until an SC outgrows them again.
// STAGED: the instance's clause offsets, literals and clause reaches are
// copied into LDS first (every later read is an LDS read), when the largest
// instance of the batch fits; else they are read from global memory.
template <bool STAGED>
__device__ __forceinline__ void cnf_transform_wave(const CnfArgs& a, int inst, int32_t* smem, CnfWaveLds& lds,
                                                   bool narrow, int first) {
  const int lane = threadIdx.x;
  const int nvar = a.n_vars[inst];
  const int c0 = a.inst_off[inst], nc = a.inst_off[inst + 1] - c0;
  const int32_t* coff;   // clause c of the instance: literals lits[coff[c] .. coff[c + 1] - 1]
  const int32_t* lits;
  const int32_t* creach;
  uint8_t* cls;          // variable classes of this instance, [n_vars + 1]
  if constexpr (STAGED) {
    int32_t* so = smem;
    int32_t* sr = so + a.stage_clauses + 1;
    int32_t* sl = sr + a.stage_clauses;
    const int l0 = a.clause_off[c0], nl = a.clause_off[c0 + nc] - l0;
    for (int c = lane; c <= nc; c += 64) so[c] = a.clause_off[c0 + c] - l0;
    for (int c = lane; c < nc; c += 64) sr[c] = a.clause_reach[c0 + c];
    for (int q = lane; q < nl; q += 64) sl[q] = a.lits[l0 + q];
    coff = so;
    creach = sr;
    lits = sl;
    cls = reinterpret_cast<uint8_t*>(sl + a.stage_lits);
  } else {
    coff = a.clause_off + c0;
    creach = a.clause_reach + c0;
    lits = a.lits;
    cls = reinterpret_cast<uint8_t*>(smem);
  }
  for (int x = lane; x <= nvar; x += 64) cls[x] = first > 0 ? a.var_class[a.var_off[inst] + x] : (uint8_t)0;
  __syncthreads();
  CnfList<kCnfWaveList>* list = &lds.list;
  int listed = 0, status = 0, in_vain = 0;
  int nexpr = first > 0 ? a.n_expr[inst] : 0;
  bool wide = true;
  int i = first;
  while (i < nc && status == 0) {
    if (wide) {
      const int lane = lane_here();
      // SC's variables, ascending, one per lane: lane q holds the q-th (lanes at
      // or past nsc hold INT_MAX), so finding a variable's place is one ballot
      int my = INT_MAX, nsc = 0;
      // with each variable, what SC says of it: bit 0 it occurs as +v, bit 1 as
      // -v, bit 2 in a clause of its own, bit 3 in two clauses or more (bit 4:
      // in an earlier clause, bit 5: in the current one).  A variable that
      // occurs with one sign only, in a single clause with other literals, is
      // never SC's output: f (or g) is then true and the other is that clause
      // without v, which some row satisfies.  Such variables are skipped
      // without a walk.
      int occ = 0;
      int start = i, reach = -1;
      for (; i < nc; ++i) {
        reach = max(reach, creach[i]);
        const bool unit = coff[i + 1] - coff[i] == 1;
        for (int p = coff[i]; p < coff[i + 1]; ++p) {  // merge the clause's variables
          const int L = lits[p], x = abs(L);
          if (__ballot(my == x) == 0) {
            const int pos = __popcll(__ballot(my < x));
            const int up = __shfl_up(my, 1), occ_up = __shfl_up(occ, 1);
            my = lane < pos ? my : (lane == pos ? x : up);
            occ = lane < pos ? occ : (lane == pos ? 0 : occ_up);
            ++nsc;
          }
          if (my == x) occ |= (L > 0 ? 1 : 2) | (unit ? 4 : 0) | 32;
        }
        if (occ & 32) occ = ((occ & 16) ? occ | 8 : occ | 16) & ~32;
        if (nsc > kCnfMaxVars) {
          status = 1;
          break;
        }
        bool found = false;
        for (int ci = nsc - 1; ci >= 0 && !found; --ci) {
          const int v = __shfl(my, ci);
          if (cls[v] & (kClsPI | kClsIV)) continue;
          const int ov = __shfl(occ, ci);
          if ((ov & 3) != 3 && !(ov & 12)) continue;
          const int k = nsc - 1;
          const int W = k > 6 ? 1 << (k - 6) : 1;
          const uint64_t valid = k >= 6 ? ~0ull : ((1ull << (1u << k)) - 1ull);
          // every lane runs the clause walk (the slot lookups are ballots); lanes
          // at or past W build words that are never used
          uint64_t f = ~0ull, g = ~0ull;
          for (int c = start; c <= i; ++c) {
            bool negv = false, posv = false;
            uint64_t word = 0;
            for (int p = coff[c]; p < coff[c + 1]; ++p) {
              const int L = lits[p], x = abs(L);
              if (x == v) {
                negv = negv || L < 0;
                posv = posv || L > 0;
                continue;
              }
              const int q = __ffsll((unsigned long long)__ballot(my == x)) - 1;
              word |= literal_word(q > ci ? q - 1 : q, lane, L < 0);
            }
            if (negv) f &= word;
            if (posv) g &= word;
          }
          const bool ok = lane >= W || ((f ^ g) & valid) == valid;
          if (__ballot(!ok) != 0) continue;
          found = true;
          f &= valid;
          const bool all1 = __ballot(lane < W && f != valid) == 0;
          const bool all0 = __ballot(lane < W && f != 0) == 0;
          const uint32_t sup = table_support(f, k, W, valid);
          tt_cnf_expr* e = a.expr + c0 + nexpr;
          e->table[lane] = lane < W ? f : 0ull;
          const int next = __shfl_down(my, 1);
          if (lane < kCnfMaxVars) e->vars[lane] = lane < ci ? my : (lane < k ? next : 0);
          if (lane == 0) {
            e->out = v;
            e->kind = (all1 || all0) ? TT_CNF_PO : TT_CNF_IV;
            e->first = start;
            e->last = i;
            e->n_vars = k;
            e->support = sup;
          }
          // classes: lane ci marks v, the other lanes of SC their own variable
          if (lane == ci) cls[v] |= (all1 || all0) ? kClsPO : kClsIV;
          if (lane < nsc && lane != ci && !(cls[my] & kClsIV)) cls[my] |= kClsPI;
          ++nexpr;
          start = i + 1;
          reach = -1;
          my = INT_MAX;
          occ = 0;
          nsc = 0;
        }
        if (!found && reach <= i) {
          // under-specified: the conjunction of SC over all its variables,
          // an auxiliary output constrained to 1
          const int W = nsc > 6 ? 1 << (nsc - 6) : 1;
          const uint64_t valid = nsc >= 6 ? ~0ull : ((1ull << (1u << nsc)) - 1ull);
          uint64_t t = ~0ull;
          for (int c = start; c <= i; ++c) {
            uint64_t word = 0;
            for (int p = coff[c]; p < coff[c + 1]; ++p) {
              const int L = lits[p];
              const int q = __ffsll((unsigned long long)__ballot(my == abs(L))) - 1;
              word |= literal_word(q, lane, L < 0);
            }
            t &= word;
          }
          t &= valid;
          const uint32_t sup = table_support(t, nsc, W, valid);
          tt_cnf_expr* e = a.expr + c0 + nexpr;
          e->table[lane] = lane < W ? t : 0ull;
          if (lane < kCnfMaxVars) e->vars[lane] = lane < nsc ? my : 0;
          if (lane == 0) {
            e->out = 0;
            e->kind = TT_CNF_AUX;
            e->first = start;
            e->last = i;
            e->n_vars = nsc;
            e->support = sup;
          }
          if (lane < nsc && !(cls[my] & kClsIV)) cls[my] |= kClsPI;
          ++nexpr;
          start = i + 1;
          reach = -1;
          my = INT_MAX;
          occ = 0;
          nsc = 0;
        }
        __syncthreads();
        if (narrow && start == i + 1) {  // SC is empty
          ++i;
          wide = false;
          break;
        }
      }
    } else {
      int start = i, end = nexpr;
      cnf_narrow_walk<true>(a.clause_rec + c0, c0, threadIdx.x < 8 ? nc : 0, i, cls, lds.sc, lds.rec, list, listed,
                            start, end, wide, [](CnfList<kCnfWaveList>* L, int) { return L; });
      // (the first group's)
      i = __builtin_amdgcn_readfirstlane(start);
      end = __builtin_amdgcn_readfirstlane(end);
      wide = __builtin_amdgcn_readfirstlane((int)wide) != 0;
      // an instance that twice gave eight lanes nothing is left to this form
      in_vain = end > nexpr ? 0 : in_vain + 1;
      narrow = in_vain < 2;
      nexpr = end;
      __syncthreads();
    }
    if (listed > kCnfWaveList - 8 || (listed > 0 && (i >= nc || status != 0))) {
      if (threadIdx.x == 0) list->count = listed;
      __syncthreads();
      cnf_flush(*list, lds.heads, a.expr);
      __syncthreads();
      listed = 0;
    }
  }
  __syncthreads();
  for (int x = lane; x <= nvar; x += 64) a.var_class[a.var_off[inst] + x] = cls[x];
  if (lane == 0) {
    a.n_expr[inst] = nexpr;
    a.status[inst] = status;
  }
  __syncthreads();  // the next instance overwrites smem
}

// One wave per instance.  The instances past n_fast in the order, one block
// each, longest first; then blocks that look through the first n_fast for
// those cnf_fast_kernel left over, the b-th at b, b + G, ... of G.  20000
// instances: 8192 blocks, some with three of them and some with two, spread
// many that are left over worst (all: 1.30 ms, wide SCs alone 5.2 ms); one
// each best (1.14 and 4.4 ms), but 4 us slower where none is left; 10000 take
// 1.27 and 4.85 ms, and 2 us.
template <bool STAGED>
__global__ __launch_bounds__(64) void cnf_transform_kernel(CnfArgs a) {
  extern __shared__ int32_t smem[];  // [staged clause offsets, reaches, literals] then the class bytes
  __shared__ CnfWaveLds lds;
  const int n_slow = a.n_inst - a.n_fast, blk = (int)blockIdx.x;
  const bool own = blk < n_slow;
  const int G = own ? 1 : (int)gridDim.x - n_slow;
  for (int slot = own ? 0 : blk - n_slow; slot < (own ? 1 : a.n_fast); slot += G) {
    const int left = own ? 1 : a.left[slot];
    if (left > 0) cnf_transform_wave<STAGED>(a, a.order[own ? a.n_fast + blk : slot], smem, lds, !own, left - 1);
  }
}

hipError_t launch_cnf_clauses(const CnfArgs& a, int n_clauses, uint4* rec, hipStream_t s) {
  if (n_clauses <= 0) return hipSuccess;
  hipLaunchKernelGGL(cnf_clause_kernel, dim3((unsigned)((n_clauses + 255) / 256)), dim3(256), 0, s, a.lits,
                     a.clause_off, a.clause_reach, n_clauses, rec);
  return hipGetLastError();
}

hipError_t launch_cnf_transform(const CnfArgs& args, int max_vars, hipStream_t s) {
  if (args.n_inst <= 0) return hipSuccess;
  CnfArgs a = args;
  if ((uintptr_t)a.expr % 16) a.n_fast = 0;  // its records go out in 16-byte pieces
  if (a.n_fast > 0) {
    hipLaunchKernelGGL(cnf_fast_kernel, dim3((unsigned)((a.n_fast + 7) / 8)), dim3(128), (size_t)8 * a.cls_stride, s,
                       a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const size_t cls_bytes = ((size_t)max_vars + 1 + 3) / 4 * 4;
  const size_t staged = 4 * (2 * (size_t)a.stage_clauses + 1 + (size_t)a.stage_lits) + cls_bytes;
  const unsigned grid =
      (unsigned)(a.n_inst - a.n_fast + std::min(a.n_fast, std::max(kCnfSweep, (a.n_fast + 1) / 2)));
  if (staged <= 64 * 1024) {
    if (staged + sizeof(CnfWaveLds) > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&cnf_transform_kernel<true>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)staged);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(cnf_transform_kernel<true>, dim3(grid), dim3(64), staged, s, a);
  } else
    hipLaunchKernelGGL(cnf_transform_kernel<false>, dim3(grid), dim3(64), cls_bytes, s, a);
  return hipGetLastError();
}

}  // namespace tt
