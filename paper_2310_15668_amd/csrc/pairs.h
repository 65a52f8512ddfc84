// Classification of pairs of neighbour groups, shared by the two pair kernels
// (exact.hip, pairs.hip): a lane holds one group k of a centre's row and walks
// groups j of the same row.
#pragma once

#include "classify.h"
#include "common.h"

constexpr int kGStride = kHistSlots + 1;   // odd stride spreads the histogram copies over banks

// Counts of a group: N members, A of them above the centre.  Where every row
// is shorter than 2^16 neighbours (kNarrow) they are the 16-bit halves
// A | N << 16 of one word, otherwise the two words (N, A).
template <bool kNarrow> struct GroupCount { using T = uint2; };
template <> struct GroupCount<true> { using T = uint32_t; };
__device__ __forceinline__ uint32_t cnt_all(const uint2& c) { return c.x; }
__device__ __forceinline__ uint32_t cnt_all(uint32_t c) { return c >> 16; }
__device__ __forceinline__ uint32_t cnt_above(const uint2& c) { return c.y; }
__device__ __forceinline__ uint32_t cnt_above(uint32_t c) { return c & 0xffffu; }

// max(a - b, 0) in one saturating subtract.
__device__ __forceinline__ uint32_t usat(uint32_t a, uint32_t b) { return a > b ? a - b : 0u; }

// max(a - b, 0) on both 16-bit halves at once (a packed saturating subtract).
using u16x2 = uint16_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_usat(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(
      uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// lo(a) * lo(b) + hi(a) * hi(b) + c, 16-bit halves: two multiply-adds of a
// Horner chain in one instruction.  The builtin, not asm: another instruction may
// read a dot product's result only three wait states later, which the compiler
// adds where it sees one.
__device__ __forceinline__ uint32_t dot2(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b), c, false);
}

// Twice the reversed ternary code 2186 - code of a pair (code as
// pair_code gives it, same digit order): the byte offset of its entry in
// the pair kernel's class table (stored reversed, 2-byte entries).  Digit r
// enters as 2 - min(R_r, 2) = max(2 - R_r, 0).  With tr holding t + 2 =
// |e_i ∩ e_j ∩ e_k| + 2 and r5 + 2 = |e_j ∩ e_k - e_i| + 2 (its heavy part)
// as 16-bit halves, three packed saturating subtracts give two digits each:
// (4, 4) - tr is (R7, R5), tr - (|e_i ∩ e_k|, k's outside count) is
// (R6, R3), tr - (pj, oj) is (R4, R2).  R1 = aks - pj + t (aks = |e_i| -
// |e_i ∩ e_k|) enters doubled, from 2 (t + 2) + aks2 with aks2 = 2 aks - 4,
// as the start of three two-term dot products that add 2 (3^6 R7 + ...)
// pair by pair.
// jy is j's record word: pj in bits 0-7, 2 pj + 4 in bits 8-15, oj in bits
// 16-23; kso = k.s | k.o << 16.
__device__ __forceinline__ uint32_t pair_rcode2(uint32_t t2, uint32_t tr, uint32_t aks2, uint32_t jy,
                                                uint32_t kso) {
  const uint32_t pjo = jy & 0x00ff00ffu, pj24 = (jy >> 8) & 0xffu;
  const uint32_t v2 = 2u * t2 + aks2;  // 2 (aks + t), one shift-add
  const uint32_t d75 = pk_usat(0x00040004u, tr);     // (R7, R5)
  const uint32_t d63 = pk_usat(tr, kso);             // (R6, R3)
  const uint32_t d42 = pk_usat(tr, pjo);             // (R4, R2)
  uint32_t c = usat(pj24, v2);                          // 2 R1
  c = dot2(d42, 54u | (6u << 16), c);
  c = dot2(d63, 486u | (18u << 16), c);
  return dot2(d75, 1458u | (162u << 16), c);
}

// t + 2 and r5 + 2 of a pair from its mask intersections: tr = (t + 2) |
// (r5 + 2) << 16, both constants added with the population count of xm, so t2 =
// t + 2 + kT2Bias, which pair_aks2 takes off again.
constexpr uint32_t kT2Bias = 2u << 16;
__device__ __forceinline__ void pair_counts(uint32_t xm, uint32_t xl, uint32_t xh, uint32_t& t2, uint32_t& tr) {
  t2 = uint32_t(__popc(xm)) + (kT2Bias | 2u);
  tr = ((uint32_t(__popc(xl)) + uint32_t(__popc(xh))) << 16) + t2;
}
// pair_rcode2's aks2 beside it: aks = |e_i| - |e_i ∩ e_k|.
__device__ __forceinline__ uint32_t pair_aks2(uint32_t aks) { return 2u * aks - 4u - 2u * kT2Bias; }

// The histogram word at a byte offset the class table gives.
__device__ __forceinline__ unsigned long long* hist_at(unsigned long long* hist, uint32_t off) {
  return reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(hist) + off);
}

// The class table entry at a byte offset.
__device__ __forceinline__ uint32_t lut_at(const uint16_t* __restrict__ lut, uint32_t off2) {
  return *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(lut) + off2);
}

// Every row is shorter than 2^24 (a graph has at most 200000 hyperedges), so
// a weight is a product of two 24-bit counts (two full-rate multiplies
// instead of a 64-bit one).  A disjoint pair (open at the centre) weighs nall_j * nall_k, an
// overlapping one nabove_j * nabove_k.  gwalk walks only groups j with
// members above the centre (they come first in a row), so the selected lane
// count is zero exactly when the pair weighs nothing (every group holds at
// least one neighbour, and kn = 0 on lanes past the row).
// kAllA: every lane's group and j have members above the centre, so every
// pair weighs at least 1 (N_j N_k or A_j A_k): no test and no branch (a lane
// past the row's end has N = A = 0 and adds 0 at a valid class).
// kNarrow: every row is shorter than 2^16 neighbours, so the group counts
// fit 16 bits and the weight of a pair of distinct groups, at most (row
// length / 2)^2, fits 32 bits: one 24-bit multiply (its high half is zero),
// or, in the full-class loop, a two-term dot product of the packed counts.
template <bool kNarrow>
__device__ __forceinline__ uint64_t pair_weight(uint32_t x, uint32_t y) {
  return kNarrow ? uint64_t(x * y) : uint64_t(x) * y;
}

template <bool kDiag, bool kAllA, bool kNarrow>
__device__ __forceinline__ void gpair_step(const uint4& rj, const typename GroupCount<kNarrow>::T& cj, int j, uint32_t aks2,
                                           const Side& k, uint32_t khl, uint32_t khh, uint32_t kso,
                                           uint32_t kn, uint32_t ka, int kp, const uint16_t* __restrict__ lut,
                                           unsigned long long* hist) {
  const uint32_t mj = rj.x;
  const uint32_t xm = mj & k.m, xl = rj.z & khl, xh = rj.w & khh;
  uint32_t t2, tr;
  pair_counts(xm, xl, xh, t2, tr);
  const bool disjoint = tr == 0x00020002u;  // t = r5 = 0
  // j's counts arrive in vector registers (gwalk loads them per lane), so
  // the selects below need no copies of scalar values
  const uint32_t y = disjoint ? kn : ka;
  if (kAllA && !kDiag) {
    const uint32_t x = (disjoint ? cnt_all(cj) : cnt_above(cj)) & 0xffffffu;
    const uint32_t rc2 = pair_rcode2(t2, tr, aks2, rj.y, kso);
    atomicAdd(hist_at(hist, lut_at(lut, rc2)), pair_weight<kNarrow>(x, y));
    return;
  }
  bool act = y != 0u;
  if (kDiag) act = act && (j < kp);
  if (act) {
    const uint32_t x = (disjoint ? cnt_all(cj) : cnt_above(cj)) & 0xffffffu;
    const uint64_t w = pair_weight<kNarrow>(x, y);
    const uint32_t rc2 = pair_rcode2(t2, tr, aks2, rj.y, kso);
    atomicAdd(hist_at(hist, lut_at(lut, rc2)), w);
  }
}

// A full-class pair's class table offset and weight (every lane's group and
// j with members above the centre).
// kNarrow: j's count word holds (nabove_j, nall_j) as 16-bit halves,
// so the weight is one dot product with the lane's (0, N_k) or (A_k, 0).
template <bool kNarrow>
__device__ __forceinline__ void pair_full(const uint4& rj, const typename GroupCount<kNarrow>::T& cj, uint32_t aks2, const Side& k,
                                          uint32_t khl, uint32_t khh, uint32_t kso, uint32_t kn,
                                          uint32_t ka, uint32_t kn16, uint32_t& rc2, uint64_t& w) {
  const uint32_t xm = rj.x & k.m, xl = rj.z & khl, xh = rj.w & khh;
  uint32_t t2, tr;
  pair_counts(xm, xl, xh, t2, tr);
  const bool disjoint = tr == 0x00020002u;  // t = r5 = 0
  rc2 = pair_rcode2(t2, tr, aks2, rj.y, kso);
  if constexpr (kNarrow) {
    w = dot2(cj, disjoint ? kn16 : ka, 0u);
  } else {
    const uint32_t y = disjoint ? kn : ka;
    const uint32_t x = (disjoint ? cj.x : cj.y) & 0xffffffu;
    w = pair_weight<kNarrow>(x, y);
  }
}

template <bool kDiag, bool kAllA, bool kNarrow>
__device__ __forceinline__ void gwalk(const uint4* __restrict__ grow, const typename GroupCount<kNarrow>::T* __restrict__ gc0,
                                      int j0, int j1, uint32_t aks, const Side& k, uint32_t kn,
                                      uint32_t ka, int kp, const uint16_t* __restrict__ lut,
                                      unsigned long long* hist) {
  const uint32_t khl = uint32_t(k.h), khh = uint32_t(k.h >> 32);
  // a lane-held zero makes the count loads vector loads (one 8-byte word
  // broadcast to every lane) instead of scalar loads
  int z = 0;
  asm volatile("" : "+v"(z));
  using C = typename GroupCount<kNarrow>::T;
  const C* gc = gc0 + z;
  const uint32_t aks2 = pair_aks2(aks);
  const uint32_t kso = k.s | (k.o << 16);
  const uint32_t kn16 = kn << 16;
  int j = j0;
  if (kAllA && !kDiag) {
    // four pairs at a time: the four class table reads are issued together
    // and waited for once, then the four histogram adds
    for (; j + 4 <= j1; j += 4) {
      const uint4 r0 = grow[j], r1 = grow[j + 1], r2 = grow[j + 2], r3 = grow[j + 3];
      const C c0 = gc[j], c1 = gc[j + 1], c2 = gc[j + 2], c3 = gc[j + 3];
      uint32_t o0, o1, o2, o3;
      uint64_t w0, w1, w2, w3;
      pair_full<kNarrow>(r0, c0, aks2, k, khl, khh, kso, kn, ka, kn16, o0, w0);
      pair_full<kNarrow>(r1, c1, aks2, k, khl, khh, kso, kn, ka, kn16, o1, w1);
      pair_full<kNarrow>(r2, c2, aks2, k, khl, khh, kso, kn, ka, kn16, o2, w2);
      pair_full<kNarrow>(r3, c3, aks2, k, khl, khh, kso, kn, ka, kn16, o3, w3);
      o0 = lut_at(lut, o0);
      o1 = lut_at(lut, o1);
      o2 = lut_at(lut, o2);
      o3 = lut_at(lut, o3);
      atomicAdd(hist_at(hist, o0), w0);
      atomicAdd(hist_at(hist, o1), w1);
      atomicAdd(hist_at(hist, o2), w2);
      atomicAdd(hist_at(hist, o3), w3);
    }
  } else {
    for (; j + 4 <= j1; j += 4) {
      const uint4 r0 = grow[j], r1 = grow[j + 1], r2 = grow[j + 2], r3 = grow[j + 3];
      const C c0 = gc[j], c1 = gc[j + 1], c2 = gc[j + 2], c3 = gc[j + 3];
      gpair_step<kDiag, kAllA, kNarrow>(r0, c0, j, aks2, k, khl, khh, kso, kn, ka, kp, lut, hist);
      gpair_step<kDiag, kAllA, kNarrow>(r1, c1, j + 1, aks2, k, khl, khh, kso, kn, ka, kp, lut, hist);
      gpair_step<kDiag, kAllA, kNarrow>(r2, c2, j + 2, aks2, k, khl, khh, kso, kn, ka, kp, lut, hist);
      gpair_step<kDiag, kAllA, kNarrow>(r3, c3, j + 3, aks2, k, khl, khh, kso, kn, ka, kp, lut, hist);
    }
  }
  for (; j < j1; ++j)
    gpair_step<kDiag, kAllA, kNarrow>(grow[j], gc[j], j, aks2, k, khl, khh, kso, kn, ka, kp, lut, hist);
}

// A pair in which one group has no member above the centre counts only when
// open at the centre (disjoint), with weight nall_j * nall_k and t = r5 = 0:
// its code is k0 (the lane's digits R6, R3) + j's digits R4, R2 + st3(|e_i|
// - k.s - pj) (R1), so j enters only through its open class (pj, st3(oj)).
// The groups are ordered by open class within each hash part, so each lane
// sums nall_j over a run of one class and adds sum * nall_k to the
// histogram when the class changes.
__device__ __forceinline__ void open_flush(uint32_t cls, uint32_t acc, uint32_t aks, uint32_t k0,
                                           uint32_t kn, const uint16_t* __restrict__ lut,
                                           unsigned long long* hist) {
  if (acc != 0u && kn != 0u) {
    const uint32_t pj = cls / 3u, oc = cls - 3u * pj;
    const uint32_t code = k0 + 27u * st3(pj) + 3u * oc + st3(aks - pj);
    atomicAdd(hist_at(hist, lut[kNumCodes - 1 - code]), uint64_t(acc) * kn);
  }
}

// (a & b) | c in one instruction, a taken from a scalar register.
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "s"(a), "v"(b), "v"(c));
  return r;
}

// acc += n if x = 0 (n < 2^24, from a scalar register): max(1 - x, 0), a
// saturating subtract (a full-rate instruction, unlike a minimum), and a
// 24-bit multiply-add, written as instructions so that they are not turned
// into a compare and a select.
__device__ __forceinline__ void acc_disjoint(uint32_t& acc, uint32_t x, uint32_t n) {
  uint32_t z;
  asm("v_sub_u32_e64 %1, 1, %2 clamp\n\tv_mad_u32_u24 %0, %1, %3, %0" : "+v"(acc), "=&v"(z) : "v"(x), "s"(n));
}

// Lanes past the diagonal block sum nall_j over the j of a run that are
// disjoint from the lane's group, as max(1 - overlap bits, 0) * nall_j (a
// saturating subtract and a multiply-add).  The diagonal block (j < k
// only) adds per lane.
template <bool kDiag, class C>
__device__ __forceinline__ void open_step(const uint4& rj, const C& cj, int j, const Side& k,
                                          uint32_t khl, uint32_t khh, uint32_t kn, int kp,
                                          uint32_t aks, uint32_t k0, uint32_t& cur, uint32_t& acc,
                                          const uint16_t* __restrict__ lut,
                                          unsigned long long* hist) {
  const uint32_t cls = rj.y >> 24;  // uniform: the open class the grouping stored
  if (cls != cur) {
    open_flush(cur, acc, aks, k0, kn, lut, hist);
    cur = cls;
    acc = 0u;
  }
  if (kDiag) {
    bool act = ((rj.x & k.m) | (rj.z & khl) | (rj.w & khh)) == 0u && kn != 0u;
    act = act && (j < kp);
    if (act) acc += cnt_all(cj);
  } else {
    const uint32_t x = and_or(rj.w, khh, and_or(rj.z, khl, rj.x & k.m));
    acc_disjoint(acc, x, cnt_all(cj));
  }
}

template <bool kDiag, class C>
__device__ __forceinline__ void owalk(const uint4* __restrict__ grow, const C* __restrict__ gc,
                                      int j0, int j1, uint32_t aks, uint32_t k0, const Side& k,
                                      uint32_t kn, int kp, const uint16_t* __restrict__ lut,
                                      unsigned long long* hist) {
  const uint32_t khl = uint32_t(k.h), khh = uint32_t(k.h >> 32);
  uint32_t cur = 0u, acc = 0u;
  int j = j0;
  for (; j + 4 <= j1; j += 4) {
    const uint4 r0 = grow[j], r1 = grow[j + 1], r2 = grow[j + 2], r3 = grow[j + 3];
    const C c0 = gc[j], c1 = gc[j + 1], c2 = gc[j + 2], c3 = gc[j + 3];
    open_step<kDiag>(r0, c0, j, k, khl, khh, kn, kp, aks, k0, cur, acc, lut, hist);
    open_step<kDiag>(r1, c1, j + 1, k, khl, khh, kn, kp, aks, k0, cur, acc, lut, hist);
    open_step<kDiag>(r2, c2, j + 2, k, khl, khh, kn, kp, aks, k0, cur, acc, lut, hist);
    open_step<kDiag>(r3, c3, j + 3, k, khl, khh, kn, kp, aks, k0, cur, acc, lut, hist);
  }
  for (; j < j1; ++j)
    open_step<kDiag>(grow[j], gc[j], j, k, khl, khh, kn, kp, aks, k0, cur, acc, lut, hist);
  open_flush(cur, acc, aks, k0, kn, lut, hist);
}

// ---------------------------------------------------------------------------
// Order of a row's groups.  Groups above the centre: those of a type that has
// at least kMinType groups in the row by type, then the rest by open class.
// A type is (popcount(m), outside count), for at most 3 nodes of e_i and 7
// heavy nodes, where the clamped outside count is at most 9.  The others: by
// open class.
constexpr int kTypes = 30;
constexpr int kMinType = 16;
constexpr int kOpenClasses = 128;
constexpr int kAboveKeys = kTypes + kOpenClasses;

// Type of a group from its record words m, z, w and clamped outside count o,
// or -1.
__device__ __forceinline__ int group_type(uint32_t m, uint32_t o, uint32_t z, uint32_t w) {
  const int p = __popc(m), hc = __popc(z) + __popc(w);
  return p <= 3 && hc <= 7 ? (p - 1) * 10 + int(o) : -1;
}
// Open class of a type.
__device__ __forceinline__ int type_open_class(int t) { return (t / 10 + 1) * 3 + min(t % 10, 2); }

// Bins -> first positions, by one wave: bins [0, n), from `start`.
__device__ __forceinline__ void wave_prefix(uint32_t* bins, int n, uint32_t start, int lane) {
  for (int b = 0; b < n; b += kWave) {
    const uint32_t v = b + lane < n ? bins[b + lane] : 0u;
    uint32_t inc = v;
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t up = __shfl_up(inc, off, kWave);
      if (lane >= off) inc += up;
    }
    if (b + lane < n) bins[b + lane] = start + inc - v;
    start += __shfl(inc, kWave - 1, kWave);
  }
}

// pairs.hip: rows of many groups on the matrix cores.  A work item is
// kMfmaCols columns of a row; rows of fewer than kMfmaRowGroups groups, and
// rows whose centre holds more than kMfmaMaxEdge nodes (two mask bits carry a
// window slot), stay with the lane-per-pair kernel.
// The line at 128 groups, one work item's columns: 9 graphs of 3,001 hyperedges
// (rows of 300 groups on average) 1.80 ms for their pairs, 2.46 with the line at
// 512, 1.93 at 256, 1.79 at 64.  A graph without a row of kMfmaMinDegree
// neighbours stays with the lane-per-pair kernel altogether: the two launches
// and the sorting cost more than they give (500 hyperedges: 0.06 ms, 0.12 with).
constexpr int kMfmaCols = 128;
constexpr int kMfmaRowGroups = 128;
constexpr int kMfmaMinDegree = 512;
constexpr int kMfmaMaxEdge = 30;
constexpr int kGroupSlack = 128;  // groups readable past the end of the group arrays

// Groups of the rows of a graph set (exact.hip builds them).
struct RowGroups {
  const int64_t* edge_ptr;
  const int64_t* goff;   // prefix of the rows' group counts
  const int64_t* gbase;  // row i's region: [gbase[i] - cap0, gbase[i + 1] - cap0)
  int64_t cap0;
  const uint4* rec;
  const uint32_t* cnt;
  const int32_t* gna;    // groups above the centre
  const int32_t* elig;   // of those, how many lead by type
};

// ---------------------------------------------------------------------------
// Work items (exact.hip builds the schedule).  Items are (row, block of
// columns).  Graph g's rows are at order[lo ...): first those of the
// lane-per-pair (or every-pair) kernel, then those of the matrix-core
// kernels, each by size, largest first; a row's items are consecutive, its
// last (largest) block first.  List l's item starts within graph g are
// start[l][lo + g + k] for its k-th row of that kind, k = 0 .. rows.
enum ItemList { kItemsLane = 0, kItemsFull, kItemsOpen, kItemLists };
struct GraphItems {
  int32_t lo;                 // first slot (relative to the schedule's first row)
  int32_t rows[2];            // rows of the lane-per-pair and the matrix-core kernels
  uint32_t total[kItemLists]; // items
};
struct WorkItems {
  const GraphItems* graphs;
  const int32_t* order;
  const uint32_t* start;  // of one list
  uint32_t* queue;        // next item of each graph
  int list;
  int g0, g1;             // graphs to count
};

// One graph's items of the launch's list, all values uniform over the wave
// (kept out of memory that lanes could address apart, so that the compiler
// sees them as uniform and the loops over rows branch on scalars).
struct ItemRange {
  const int32_t* order;
  const uint32_t* start;
  uint32_t* queue;
  int rows;
  uint32_t total;
};
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ ItemRange item_range(const WorkItems& I, int g) {
  const GraphItems* gi = I.graphs + g;
  const int lo = uniform(gi->lo), r0 = uniform(gi->rows[0]), r1 = uniform(gi->rows[1]);
  ItemRange r;
  r.order = I.order + lo + (I.list == kItemsLane ? 0 : r0);
  r.start = I.start + lo + g;
  r.queue = I.queue + g;
  r.rows = I.list == kItemsLane ? r0 : r1;
  r.total = uint32_t(uniform(int(gi->total[I.list])));
  return r;
}

// The next (row, block), or false once they are taken; uniform over the wave.
__device__ __forceinline__ bool next_item(const ItemRange& r, int lane, int32_t& row, int& block) {
  int v = 0;
  if (lane == 0) v = int(atomicAdd(r.queue, 1u));
  const uint32_t q = uint32_t(uniform(v));
  if (q >= r.total) return false;
  int lo = 0, hi = r.rows;  // start[lo] <= q < start[lo + 1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (uint32_t(uniform(int(r.start[mid]))) <= q) lo = mid; else hi = mid;
  }
  row = uniform(r.order[lo]);
  block = uniform(int(r.start[lo + 1])) - int(q) - 1;
  return true;
}

// Visits the graphs of a launch, each block starting at a share of its own:
// work(g, items) runs in every wave of the block until the graph's items are
// taken, then done(g) between barriers (it flushes what the block counted).
template <class Work, class Done>
__device__ __forceinline__ void visit_graphs(const WorkItems& I, Work&& work, Done&& done) {
  __shared__ uint32_t taken[2];
  const int n = I.g1 - I.g0;
  const int first = int(int64_t(blockIdx.x) * n / gridDim.x);
  for (int v = 0; v < n; ++v) {
    const int g = I.g0 + (first + v < n ? first + v : first + v - n);
    const ItemRange r = item_range(I, g);
    if (threadIdx.x == 0) taken[v & 1] = __hip_atomic_load(r.queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (uint32_t(uniform(int(taken[v & 1]))) >= r.total) continue;
    work(g, r);
    __syncthreads();
    done(g);
    __syncthreads();
  }
}

// The same for kernels of many small items (a lane per pair), whose launch may
// have thousands of graphs: kLook of them looked at for one barrier, and a block
// joins a graph past its share (own work first) only while that has kHelpItems
// items left, since a visit ends in adding up the block's counters: by the time
// fewer are left the blocks already there are done with them.  4,000 graphs of 40
// hyperedges 0.34 ms (2.5 a barrier to each graph, every graph joined), 1,000 of
// 1,000 2.6 (3.5; joined for any item 9.8, for 256 5.9, for 4,096 2.5).  The
// matrix-core kernels have fewer, longer items: 65 graphs of 6,100 hyperedges
// took 6 % longer this way.
constexpr int kLook = 8;
constexpr uint32_t kHelpItems = 1024;
template <class Work, class Done>
__device__ __forceinline__ void visit_many_graphs(const WorkItems& I, Work&& work, Done&& done) {
  __shared__ uint32_t s_left[2], s_now[2];
  const int n = I.g1 - I.g0;
  const int first = int(int64_t(blockIdx.x) * n / gridDim.x);
  const int own = max(1, int((int64_t(blockIdx.x) + 1) * n / gridDim.x) - first);
  auto graph = [&](int x) { return I.g0 + (first + x < n ? first + x : first + x - n); };
  auto worth = [&](int x, uint32_t now, uint32_t total) { return now < total && (x < own || total - now >= kHelpItems); };
  int flip = 0;
  for (int v = 0; v < n; v += kLook) {
    const int turn = (v / kLook) & 1;
    if (threadIdx.x < unsigned(kWave)) {
      const int x = v + int(threadIdx.x);
      bool some = false;
      if (int(threadIdx.x) < kLook && x < n)
        some = worth(x, __hip_atomic_load(I.queue + graph(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                     I.graphs[graph(x)].total[I.list]);
      const unsigned long long m = __ballot(some);
      if (threadIdx.x == 0) s_left[turn] = uint32_t(m);
    }
    __syncthreads();
    for (uint32_t m = uint32_t(uniform(int(s_left[turn]))); m; m &= m - 1u) {
      const int x = v + __ffs(int(m)) - 1, g = graph(x);
      const ItemRange r = item_range(I, g);
      uint32_t& now = s_now[flip++ & 1];  // as it stands by now
      if (threadIdx.x == 0) now = __hip_atomic_load(r.queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      if (!worth(x, uint32_t(uniform(int(now))), r.total)) continue;
      work(g, r);
      __syncthreads();
      done(g);
      __syncthreads();
    }
  }
}

// Adds a block's histogram copies into graph g's counts and clears them.
template <int kCopies>
__device__ __forceinline__ void hist_flush(unsigned long long* hist, int g, unsigned long long* out) {
  for (int t = threadIdx.x; t < kHistSlots; t += blockDim.x) {
    unsigned long long v = 0;
    for (int c = 0; c < kCopies; ++c) {
      v += hist[c * kGStride + t];
      hist[c * kGStride + t] = 0ull;
    }
    if (v) atomicAdd(&out[int64_t(g) * kHistSlots + t], v);
  }
}

void launch_sort_groups(int cus, const int32_t* rows, const unsigned long long* nrows, unsigned long long* queue,
                        const RowGroups& G, uint4* rec, uint32_t* cnt, int32_t* elig, hipStream_t s);
void launch_pairs_full(unsigned grid, const RowGroups& G, const WorkItems& I, const uint16_t* code_to_id3,
                       unsigned long long* hist, hipStream_t s);
void launch_pairs_open(unsigned grid, const RowGroups& G, const WorkItems& I, const uint16_t* code_to_id3,
                       unsigned long long* hist, hipStream_t s);
