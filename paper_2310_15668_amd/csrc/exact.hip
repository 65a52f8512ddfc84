// Exact h-motif / 3h-motif counts on the device (MoCHy-E, Algorithm 2).
//
// Algorithm 2 takes every centre e_i and every unordered pair {e_j, e_k} of
// its line-graph neighbours and counts the triple iff e_j and e_k are
// disjoint or i < min(j, k); the class comes from the seven region sizes of
// Lemma 2.  Here the neighbours of e_i are the row's positions 0..d-1 in
// ascending id order, and u = number of neighbours with id < i, so
//   * a pair with a position < u (a neighbour below i) is counted iff the two
//     neighbours are disjoint (an open instance whose middle is e_i);
//   * a pair with both positions >= u is always counted.
//
// Region sizes of a pair from the per-neighbour records of the centre:
//   t  = |e_i ∩ e_j ∩ e_k|     = popcount(m_j & m_k)
//   R4 = p_j - t, R6 = s_k - t, R1 = |e_i| - p_j - s_k + t, R7 = t
//   R5 = |e_j ∩ e_k - e_i|,  R2 = o_j - R5,  R3 = o_k - R5
// R5 is the only quantity that needs nodes outside e_i.  The records carry
// an exact bit for each of the 64 highest-degree nodes, so the main kernel
// uses R5 = popcount(h_j & h_k).  That is exact unless e_j and e_k also share
// a lower-degree ("light") node outside e_i; the correction kernel finds every
// such pair (from the node->hyperedge lists of the light nodes), undoes what
// the main kernel recorded for it and records the exact class.
//
// Main kernel work decomposition: an item is (row, block of 64 positions);
// lane l of a wave holds the record of position 64*block + l ("k") and the
// wave walks j over the positions below it; the j record is uniform and read
// through the scalar cache.  Items are ordered by block index descending, so
// the largest items start first, and pulled from a counter per graph by
// persistent waves.  Counts go to LDS histograms (several copies, picked by
// lane, to thin same-bin conflicts), flushed with 64-bit global atomics when a
// block leaves a graph.
//
// Grouped path (the default: k_group_*, then k_pairs_full and k_pairs_open of
// pairs.hip for rows of many groups, k_exact_grouped for the others):
// neighbours of e_i
// with equal records (m, outside count clamped to popcount(h) + 2, h) form a
// group with N members and A members above the centre; a pair of groups
// stands for N_j N_k candidates if they look disjoint, A_j A_k otherwise,
// and a group with itself for C(A, 2).  Each row's region holds the groups
// with A > 0 first.  A pair involving a group with A = 0 counts only if open,
// and an open class depends on j only through (popcount(m_j), min(o_j, 2)):
// such pairs are summed per lane over runs of one such class (the groups are
// class-ordered within each hash part) and added once per run.
#include <vector>

#include "classify.h"
#include "common.h"
#include "pairs.h"

namespace {

// The every-pair kernel's counters, shared by a block's waves: kCopies of each
// motif's in neighbouring banks, picked by lane, so that no more than 4 lanes
// of a wave add at one address and take turns (2 copies to a wave: 3.2 ms on
// 6,029 hyperedges, 4: 2.7, 16 to a block: 2.2).
constexpr int kCopies = 16;
constexpr int kMainThreads = 512, kMainWaves = kMainThreads / kWave;
// visits after which a wave empties the counters: they hold at most as many of
// each wave, 4 lanes' adds a visit (few for tests of the emptying)
constexpr int64_t kFlushVisits = int64_t(1) << 26, kFlushVisitsTest = 100;
static_assert(kFlushVisits * kMainWaves * (kWave / kCopies) < (int64_t(1) << 32), "32-bit counters");

// ---------------------------------------------------------------------------
// Scheduling (the lists pairs.h describes): one block per graph sorts its rows
// by kind and size (a counting sort over 8 sizes per octave, largest first)
// and forms their item starts.  One kernel: a small graph's count is launches
// and read-backs, and a graph of 85k rows takes the block 0.2 ms.
struct RowKinds {
  const int64_t* lg_ptr;   // every pair of neighbours: rows of 2 or more
  const int64_t* goff;     // otherwise groups: rows of 1 or more
  const int32_t* gna;
  const int64_t* edge_ptr;
  bool grouped, mfma;      // mfma: rows of many groups are the matrix-core kernels'
};

// Row i's kind (0, 1; -1: no pairs), size and items per list.
__device__ __forceinline__ int row_kind(const RowKinds& R, int64_t i, int& len) {
  const int64_t* p = R.grouped ? R.goff : R.lg_ptr;
  len = int(p[i + 1] - p[i]);
  if (len < (R.grouped ? 1 : 2)) return -1;
  return R.mfma && len >= kMfmaRowGroups && R.edge_ptr[i + 1] - R.edge_ptr[i] <= kMfmaMaxEdge ? 1 : 0;
}
// Size class, 8 per octave, ascending (below 256).
__device__ __forceinline__ int size_class(int len) {
  const int e = 31 - __clz(len);
  return e < 3 ? len : e * 8 + ((len >> (e - 3)) & 7);
}

__global__ __launch_bounds__(1024) void k_schedule(int64_t c0, int64_t c1, const int64_t* __restrict__ geoff,
                                                   RowKinds R, GraphItems* graphs, int32_t* order,
                                                   uint32_t* start_lane, uint32_t* start_full,
                                                   uint32_t* start_open, uint32_t* queues) {
  constexpr int kBins = 512;  // (kind, size class descending)
  __shared__ uint32_t bins[kBins];
  __shared__ unsigned long long wsum[1024 / kWave];
  const int g = blockIdx.x, ng = gridDim.x, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int64_t lo = min(max(geoff[g], c0), c1), hi = min(max(geoff[g + 1], c0), c1);
  const int slot0 = int(lo - c0);
  for (int t = tid; t < kBins; t += 1024) bins[t] = 0u;
  __syncthreads();
  for (int64_t i = lo + tid; i < hi; i += 1024) {
    int len;
    const int kind = row_kind(R, i, len);
    if (kind >= 0) atomicAdd(&bins[kind * 256 + 255 - size_class(len)], 1u);
  }
  __syncthreads();
  __shared__ int rows[2];
  if (wave == 0) {
    uint32_t s = 0;  // rows of kind 0
    for (int t = lane; t < 256; t += kWave) s += bins[t];
    uint32_t l = 0;
    for (int t = 256 + lane; t < kBins; t += kWave) l += bins[t];
    for (int off = kWave / 2; off > 0; off >>= 1) {
      s += __shfl_xor(s, off, kWave);
      l += __shfl_xor(l, off, kWave);
    }
    if (lane == 0) {
      rows[0] = int(s);
      rows[1] = int(l);
    }
    wave_prefix(bins, kBins, 0u, lane);
  }
  __syncthreads();
  const int n0 = rows[0], n = rows[0] + rows[1];
  for (int64_t i = lo + tid; i < hi; i += 1024) {
    int len;
    const int kind = row_kind(R, i, len);
    if (kind >= 0) order[slot0 + int(atomicAdd(&bins[kind * 256 + 255 - size_class(len)], 1u))] = int32_t(i);
  }
  __syncthreads();
  // item starts: an exclusive scan over the slots of (lane-per-pair or full
  // tiles, open tiles) as the halves of one word, four slots per thread
  unsigned long long run = 0;  // items before this sweep
  uint32_t* s0 = start_lane + slot0 + g;
  uint32_t* s1 = start_full ? start_full + slot0 + g : nullptr;
  uint32_t* s2 = start_open ? start_open + slot0 + g : nullptr;
  __shared__ uint32_t lane_total;
  if (tid == 0) lane_total = 0u;
  __syncthreads();
  for (int k0 = 0; k0 < n; k0 += 4096) {
    unsigned long long v[4], sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + tid * 4 + u;
      v[u] = 0;
      if (k < n) {
        const int64_t i = order[slot0 + k];
        int len;
        row_kind(R, i, len);
        if (k < n0) {
          v[u] = (unsigned long long)((len + kWave - 1) / kWave);
        } else {
          const int na = R.gna[i];
          v[u] = (unsigned long long)((na + kMfmaCols - 1) / kMfmaCols) |
                 ((unsigned long long)((len - na + kMfmaCols - 1) / kMfmaCols) << 32);
        }
      }
      sum += v[u];
    }
    unsigned long long inc = sum;
    for (int off = 1; off < kWave; off <<= 1) {
      const unsigned long long up = __shfl_up(inc, off, kWave);
      if (lane >= off) inc += up;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    unsigned long long at = run + inc - sum;
    unsigned long long all = 0;
    for (int w = 0; w < 1024 / kWave; ++w) {
      if (w < wave) at += wsum[w];
      all += wsum[w];
    }
    run += all;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + tid * 4 + u;
      if (k < n0) s0[k] = uint32_t(at);
      else if (k < n) {
        if (k == n0) lane_total = uint32_t(at);
        s1[k - n0] = uint32_t(at);  // the lane-per-pair items are taken off below
        s2[k - n0] = uint32_t(at >> 32);
      }
      at += v[u];
    }
    __syncthreads();
  }
  const uint32_t base = n > n0 ? lane_total : uint32_t(run);
  if (s1) {
    for (int k = tid; k < n - n0; k += 1024) s1[k] -= base;
  }
  if (tid == 0) {
    GraphItems gi;
    gi.lo = slot0;
    gi.rows[0] = n0;
    gi.rows[1] = n - n0;
    gi.total[kItemsLane] = base;
    gi.total[kItemsFull] = uint32_t(run) - base;
    gi.total[kItemsOpen] = uint32_t(run >> 32);
    graphs[g] = gi;
    s0[n0] = base;
    if (s1) s1[n - n0] = gi.total[kItemsFull];
    if (s2) s2[n - n0] = gi.total[kItemsOpen];
    for (int l = 0; l < kItemLists; ++l) queues[l * ng + g] = 0u;
  }
}

// The lane's k as the walks take it.
struct LaneSide {
  uint32_t m, hl, hh, kso;  // masks; |e_i ∩ e_k| | outside count << 16
  uint32_t aks2;            // pair_aks2 of |e_i| - |e_i ∩ e_k|
  uint32_t aksd;            // 2 (|e_i| - |e_i ∩ e_k|)
  uint32_t open;            // its digits R6 and R3 of a disjoint pair, and those of t = R5 = 0
  uint32_t one;             // 1, 0 past the row's end
  int kp;
};

// Pairs of the lane's k and kN records from j on (uniform); the class table
// reads are issued together.  kCountAll: both j and k are above the centre (every pair counts);
// otherwise only disjoint pairs count, whose codes are k's digits, j's (scalar
// work) and R1.  kDiag: the j range overlaps the lane block, so require j < kp.
template <int kN, bool kCountAll, bool kDiag>
__device__ __forceinline__ void pair_steps(const uint4* __restrict__ row, int j, const LaneSide& k,
                                           const uint16_t* __restrict__ lut, char* hist) {
  uint32_t code[kN], w[kN];
#pragma unroll
  for (int u = 0; u < kN; ++u) {
    const uint4 rj = row[j + u];
    const uint32_t pj = uint32_t(__popc(rj.x)), oj = rj.y & 0xffu;
    w[u] = kDiag && j + u >= k.kp ? 0u : k.one;
    if (kCountAll) {
      uint32_t t2, tr;
      pair_counts(rj.x & k.m, rj.z & k.hl, rj.w & k.hh, t2, tr);
      code[u] = pair_rcode2(t2, tr, k.aks2, pj | (2u * pj + 4u) << 8 | oj << 16, k.kso);
    } else {
      const uint32_t x = and_or(rj.w, k.hh, and_or(rj.z, k.hl, rj.x & k.m));
      // R1 held in range for a pair that overlaps
      code[u] = min(usat(2u * pj + 4u, k.aksd), 4u) + k.open + (54u * usat(2u, pj) + 6u * usat(2u, oj));
      w[u] = x ? 0u : w[u];
    }
  }
#pragma unroll
  for (int u = 0; u < kN; ++u) code[u] = lut_at(lut, code[u]);
#pragma unroll
  for (int u = 0; u < kN; ++u)
    if (w[u]) atomicAdd(reinterpret_cast<uint32_t*>(hist + code[u]), 1u);
}

template <bool kCountAll, bool kDiag>
__device__ __forceinline__ void walk(const uint4* __restrict__ row, int j0, int j1, const LaneSide& k,
                                     const uint16_t* __restrict__ lut, char* hist) {
  int j = j0;
  for (; j + 8 <= j1; j += 8) pair_steps<8, kCountAll, kDiag>(row, j, k, lut, hist);
  for (; j < j1; ++j) pair_steps<1, kCountAll, kDiag>(row, j, k, lut, hist);
}

// Adds the counters at x = first, first + step, .. to graph g's counts and
// empties them, while other waves may add.
__device__ __forceinline__ void flush_main(uint32_t (*hist)[kCopies], int first, int step, int64_t g,
                                           unsigned long long* hist_out) {
  for (int t = first; t < kHistSlots; t += step) {
    unsigned long long n = 0;
    for (int c = 0; c < kCopies; ++c) n += atomicExch(&hist[t][(c + t) % kCopies], 0u);
    if (n) atomicAdd(&hist_out[g * kHistSlots + t], n);
  }
}

__global__ __launch_bounds__(kMainThreads) void k_exact_main(
    const int64_t* __restrict__ edge_ptr, const int64_t* __restrict__ lg_ptr,
    const int32_t* __restrict__ up_first, const uint4* __restrict__ rec, WorkItems I,
    const uint16_t* __restrict__ code_to_id3, unsigned long long* hist_out, int64_t flush_visits) {
  __shared__ uint16_t lut[kNumCodes];
  __shared__ uint32_t hist[kHistSlots][kCopies];
  // by reversed code: byte offsets of the ids' counters
  for (int t = threadIdx.x; t < kNumCodes; t += blockDim.x) lut[t] = uint16_t(code_to_id3[kNumCodes - 1 - t] * (kCopies * 4u));
  for (int t = threadIdx.x; t < kHistSlots * kCopies; t += blockDim.x) hist[0][t] = 0u;
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  char* myhist = reinterpret_cast<char*>(&hist[0][lane % kCopies]);
  visit_graphs(I, [&](int g, const ItemRange& items) {
    int64_t visits = 0;
    int32_t i;
    int b;
    while (next_item(items, lane, i, b)) {
      if (visits > flush_visits) {
        flush_main(hist, lane, kWave, g, hist_out);
        visits = 0;
      }
      const int64_t base = lg_ptr[i];
      const int d = int(lg_ptr[i + 1] - base);
      const int u = up_first[i];
      const uint32_t a = uint32_t(edge_ptr[i + 1] - edge_ptr[i]);
      const uint4* __restrict__ row = rec + base;
      const int kp = b * kWave + lane;
      const bool valid = kp < d;
      LaneSide k;
      {
        const uint4 rk = valid ? row[kp] : make_uint4(0, 0, 0, 0);
        const uint32_t ks = uint32_t(__popc(rk.x)), ko = rk.y & 0xffu;
        k.m = rk.x;
        k.hl = rk.z;
        k.hh = rk.w;
        k.kso = ks | ko << 16;
        k.aksd = 2u * (a - ks);
        k.aks2 = pair_aks2(a - ks);
        k.open = 2u * 1458u + 2u * 162u + 486u * usat(2u, ks) + 18u * usat(2u, ko);
        k.one = valid ? 1u : 0u;
        k.kp = kp;
      }
      const int blo = b * kWave;
      const int kmax = min(blo + kWave, d);
      visits += int64_t(kmax);
      // j below the centre: count disjoint pairs only
      const int ua = min(u, blo);
      walk<false, false>(row, 0, ua, k, lut, myhist);
      walk<false, true>(row, max(ua, blo), min(u, kmax), k, lut, myhist);
      // j (and so k) above the centre: count every pair
      walk<true, false>(row, u, blo, k, lut, myhist);
      walk<true, true>(row, max(u, blo), kmax, k, lut, myhist);
    }
  }, [&](int g) { flush_main(hist, threadIdx.x, kMainThreads, g, hist_out); });
}

// ---------------------------------------------------------------------------
// Neighbour groups.  The main kernel's class of a pair (j, k) of a centre,
// and whether Algorithm 2 counts it, depend only on the two records: the
// masks m (nodes of e_i held) and h (heavy nodes outside e_i) and the outside
// counts o, where only min(o - R5, 2) is ever used and R5 <= popcount(h), so o
// may be clamped to popcount(h) + 2.  Neighbours with equal (m, clamped o, h)
// form a group; a group keeps N (members) and A (members above the centre).
// Between two groups x != y the main kernel's count is N_x N_y if they are
// disjoint (every pair counts) and A_x A_y otherwise (only pairs above the
// centre count); inside a group it is C(A, 2) (members share their nodes of
// e_i, so never disjoint).  Pairs sharing a light node are corrected from the
// ungrouped records afterwards, as before.
//
// One block per row groups the row's records in an LDS hash table
// keyed by a 64-bit hash of the signature.  A row longer than the table is
// cut into parts by the hash (records of one part per pass); a pass whose
// table fills is redone with twice the parts.  After each pass every record
// checks its signature against its slot's first member: two signatures with
// one hash restart the row with another hash seed, so groups are exact.
// Two table sizes.  Rows of at most kShortRow records: 512-thread blocks,
// 2048 slots (41 KB of LDS, three blocks per CU), one block per row over all
// rows (a longer row's block returns at once).  Longer rows: 1024-thread
// blocks with 8000 slots (160 KB, one block per CU) over a list of those
// rows: a larger table means fewer hash parts, and every part re-reads the
// row twice.  On medium the long-row table took the grouping from 62 ms (all
// rows at 2048 slots: up to 18 parts, 12,805 rows regrouped) to 37 ms (up to
// 4 parts); 4032 slots in 512-thread blocks took 48 ms.  Small graphs keep
// the short-row table, whose blocks clear only 2048 slots and share the CU.
constexpr int kShortThreads = 512, kShortSlots = 2048;
constexpr int kLongThreads = 1024, kLongSlots = 8000;
constexpr int64_t kShortRow = 2 * kShortSlots;

// Home slot of a 64-bit signature hash (multiply-shift range reduction of
// its low 32 bits, any table size) and the next slot of a linear probe.
template <int kSlots>
__device__ __forceinline__ uint32_t home_slot(uint64_t kk) {
  return uint32_t((uint64_t(uint32_t(kk)) * uint32_t(kSlots)) >> 32);
}
template <int kSlots>
__device__ __forceinline__ uint32_t next_slot(uint32_t s) { return s + 1u == uint32_t(kSlots) ? 0u : s + 1u; }

__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  // SplitMix64 finalizer (Steele, Lea, Flood, OOPSLA'14)
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  x ^= x >> 31;
  return x;
}

__device__ __forceinline__ uint32_t clamp_outside(const uint4& r) {
  const uint32_t o = r.y & 0xffu;
  const uint32_t cap = uint32_t(__popc(r.z) + __popc(r.w)) + 2u;
  return o < cap ? o : cap;
}

__device__ __forceinline__ uint64_t sig_hash(const uint4& r, uint32_t o, uint64_t seed) {
  uint64_t x = mix64(seed ^ (uint64_t(r.x) | (uint64_t(o) << 32)));
  x = mix64(x ^ (uint64_t(r.z) | (uint64_t(r.w) << 32)));
  return x | 1ull;  // 0 marks a free slot
}

constexpr int kGroupTries = 40;  // restarts before a row gives up (flags bit 0)

// Open class of a group: (|its overlap with e_i|, min(outside, 2)); the code
// of an open pair depends on j only through it.  Below kOpenClasses.
__device__ __forceinline__ uint32_t open_class(uint32_t m, uint32_t o) {
  return uint32_t(__popc(m)) * 3u + st3(o);
}

template <int kSlots>
struct GroupTable {
  unsigned long long key[kSlots];
  uint32_t nall[kSlots], nabove[kSlots], first[kSlots];
  uint32_t s_out, s_outb, s_bad, s_cnt;
  uint32_t cfill[kAboveKeys + kOpenClasses];  // per order key (above, others): count, then next slot
  uint32_t moved[kTypes];                     // types with too few groups, ordered by open class
  uint32_t s_elig;                            // groups of the other types
};

// Groups of row i with the block's table.  kWrite: row i's groups go to its
// region [base[i] - cap0, base[i + 1] - cap0) of grec / gcnt: base = lg_ptr
// with the row-capacity layout (a row has at most as many groups as
// records), or the prefix of the counts with cap0 = 0 (compact layout,
// counted by a first pass).  Groups with members above the centre fill the
// region from its start (their count goes to gna[i]), the others from its
// end, so that the pair kernels can take the pairs that can only be open
// apart; within each hash part of the row, both kinds are in the order that
// pairs.h states.  A row of one part is then in that order as a whole (elig[i]
// groups by type); one of several parts is listed in srows, to be sorted.
// The count goes to gcount[i].  Hash parts: a first guess of
// 2 * kSlots records per part, doubled whenever a part has more than
// 3/4 * kSlots groups (rows have 0.38 groups per record on medium).
template <bool kWrite, int kThreads, int kSlots>
__device__ __forceinline__ int64_t group_row(
    GroupTable<kSlots>& T, int64_t i, const int64_t* __restrict__ lg_ptr,
    const int32_t* __restrict__ up_first, const uint4* __restrict__ rec, int64_t* gcount,
    const int64_t* __restrict__ obase_of, int64_t cap0, uint4* grec, void* gcnt, int32_t* gna,
    int32_t* elig, int32_t* srows, unsigned long long* nsrows, int32_t* flags, bool pack16) {
  constexpr int64_t kPartRecords = 2 * kSlots;
  constexpr uint32_t kPartGroups = kSlots * 3 / 4;
  const int tid = threadIdx.x;
  const int64_t base = lg_ptr[i];
  const int64_t d = lg_ptr[i + 1] - base;
  const int64_t u = up_first[i];
  const uint4* row = rec + base;
  int64_t parts = (d + kPartRecords - 1) / kPartRecords;
  if (parts < 1) parts = 1;
  const int64_t parts0 = parts;
  uint64_t seed = 0;
  const int64_t obase = kWrite ? obase_of[i] - cap0 : 0;
  const int64_t oend = kWrite ? obase_of[i + 1] - cap0 : 0;  // one past the row's region
  for (int tries = 0;; ++tries) {  // until a grouping without overflow or hash collision
    if (tries == kGroupTries) {  // cannot happen with a sound hash; the host pairs records
      if (tid == 0) {
        atomicOr(flags, 1);
        if (gcount) gcount[i] = 0;
      }
      __syncthreads();
      return 0;
    }
    __syncthreads();
    if (tid == 0) {
      T.s_out = 0u;
      T.s_outb = 0u;
    }
    bool redo = false;
    for (int64_t part = 0; part < parts && !redo; ++part) {
      for (int t = tid; t < kSlots; t += kThreads) {
        T.key[t] = 0ull;
        T.nall[t] = 0u;
        T.nabove[t] = 0u;
      }
      if (tid == 0) {
        T.s_bad = 0u;
        T.s_cnt = 0u;
      }
      __syncthreads();
      for (int64_t r = tid; r < d; r += kThreads) {
        if (*(volatile uint32_t*)&T.s_bad) break;  // this part overflowed: the row is redone
        const uint4 rr = row[r];
        const uint64_t kk = sig_hash(rr, clamp_outside(rr), seed);
        if (int64_t((kk >> 40) % uint64_t(parts)) != part) continue;
        uint32_t slot = home_slot<kSlots>(kk);
        int n = 0;
        for (; n < kSlots; ++n) {
          const unsigned long long old = atomicCAS(&T.key[slot], 0ull, kk);
          if (old == 0ull) {
            T.first[slot] = uint32_t(r);
            if (atomicAdd(&T.s_cnt, 1u) >= kPartGroups) atomicOr(&T.s_bad, 4u);
            break;
          }
          if (old == kk) break;
          slot = next_slot<kSlots>(slot);
        }
        if (n == kSlots) { atomicOr(&T.s_bad, 1u); continue; }
        atomicAdd(&T.nall[slot], 1u);
        if (r >= u) atomicAdd(&T.nabove[slot], 1u);
      }
      __syncthreads();
      const uint32_t full = T.s_bad;
      __syncthreads();  // every thread has read the flag before it is written again
      if (full) {  // too many groups in the part: twice the parts
        parts *= 2;
        redo = true;
        break;
      }
      // every record against its slot's first member
      for (int64_t r = tid; r < d; r += kThreads) {
        const uint4 rr = row[r];
        const uint32_t o = clamp_outside(rr);
        const uint64_t kk = sig_hash(rr, o, seed);
        if (int64_t((kk >> 40) % uint64_t(parts)) != part) continue;
        uint32_t slot = home_slot<kSlots>(kk);
        while (T.key[slot] != kk) slot = next_slot<kSlots>(slot);
        const uint4 f = row[T.first[slot]];
        if (f.x != rr.x || f.z != rr.z || f.w != rr.w || clamp_outside(f) != o) atomicOr(&T.s_bad, 2u);
      }
      __syncthreads();
      const uint32_t clash = T.s_bad;
      __syncthreads();
      if (clash) {  // two signatures with one hash: another seed
        seed += 0x9E3779B97F4A7C15ull;
        redo = true;
        break;
      }
      if (!kWrite) {
        for (int t = tid; t < kSlots; t += kThreads)
          if (T.key[t] != 0ull) atomicAdd(&T.s_out, 1u);
        __syncthreads();
        continue;
      }
      // counting sort of the part's groups by order key
      for (int t = tid; t < kAboveKeys + kOpenClasses; t += kThreads) T.cfill[t] = 0u;
      if (tid == 0) T.s_elig = 0u;
      __syncthreads();
      auto key_of = [&](bool above, const uint4& f, uint32_t oc) -> int {
        const int ty = above ? group_type(f.x, oc, f.z, f.w) : -1;
        return ty >= 0 ? ty : (above ? kTypes : kAboveKeys) + int(open_class(f.x, oc));
      };
      for (int t = tid; t < kSlots; t += kThreads) {
        if (T.key[t] == 0ull) continue;
        const uint4 f = row[T.first[t]];
        atomicAdd(&T.cfill[key_of(T.nabove[t] != 0u, f, clamp_outside(f))], 1u);
      }
      __syncthreads();
      if (tid < kTypes) {  // one lane per type: few groups join the rest
        const uint32_t n = T.cfill[tid];
        T.moved[tid] = n < uint32_t(kMinType) ? 1u : 0u;
        if (n >= uint32_t(kMinType)) {
          atomicAdd(&T.s_elig, n);
        } else if (n) {
          T.cfill[tid] = 0u;
          atomicAdd(&T.cfill[kTypes + type_open_class(tid)], n);
        }
      }
      __syncthreads();
      // first positions of each kind (one wave each), from where its output stands
      if (tid < kWave) wave_prefix(T.cfill, kAboveKeys, T.s_out, tid);
      else if (tid < 2 * kWave) wave_prefix(T.cfill + kAboveKeys, kOpenClasses, T.s_outb, tid - kWave);
      __syncthreads();
      for (int t = tid; t < kSlots; t += kThreads) {
        if (T.key[t] == 0ull) continue;
        const bool above = T.nabove[t] != 0u;
        const uint4 f = row[T.first[t]];
        const uint32_t oc = clamp_outside(f);
        int key = key_of(above, f, oc);
        if (key < kTypes && T.moved[key]) key = kTypes + type_open_class(key);
        const uint32_t pos = atomicAdd(&T.cfill[key], 1u);
        const int64_t o = above ? obase + pos : oend - 1 - pos;
        // y: |m| (bits 0-7), 2 |m| + 4 (8-15), the clamped outside count
        // (16-23) and the open class (24-30), which the pair kernel then
        // reads instead of recomputing them per pair: (|m|, outside) is y
        // with bits 8-15 and 24-31 cleared, one scalar AND
        const uint32_t pm = uint32_t(__popc(f.x));
        grec[o] = make_uint4(f.x, pm | ((2u * pm + 4u) << 8) | (oc << 16) | (open_class(f.x, oc) << 24), f.z, f.w);
        // pack16 (every row shorter than 2^16 neighbours): one word holds
        // nabove and nall as 16-bit halves, for the pair kernels' weights
        if (pack16) static_cast<uint32_t*>(gcnt)[o] = T.nabove[t] | (T.nall[t] << 16);
        else static_cast<uint2*>(gcnt)[o] = make_uint2(T.nall[t], T.nabove[t]);
      }
      __syncthreads();
      if (tid == 0) {  // both kinds' ends: the last class's next slot
        T.s_out = T.cfill[kAboveKeys - 1];
        T.s_outb = T.cfill[kAboveKeys + kOpenClasses - 1];
      }
      __syncthreads();
    }
    if (!redo) break;
  }
  if (tid == 0) {
    if (gcount) gcount[i] = int64_t(T.s_out) + T.s_outb;
    if (kWrite) {
      gna[i] = int32_t(T.s_out);
      elig[i] = parts == 1 ? int32_t(T.s_elig) : 0;
      if (parts > 1) srows[atomicAdd(nsrows, 1ull)] = int32_t(i);
    }
  }
  __syncthreads();  // the table is free for the block's next row
  return parts > parts0 ? -parts : parts;  // the parts used, negative if the row was regrouped
}

// Short rows: one block per row of [c0, c0 + gridDim.x); longer rows are
// the long-row kernel's.
template <bool kWrite>
__global__ __launch_bounds__(kShortThreads) void k_group_short(
    int64_t c0, const int64_t* __restrict__ lg_ptr, const int32_t* __restrict__ up_first,
    const uint4* __restrict__ rec, int64_t* gcount, const int64_t* __restrict__ obase_of,
    int64_t cap0, uint4* grec, void* gcnt, int32_t* gna, int32_t* elig, int32_t* srows, unsigned long long* nsrows,
    int32_t* flags, unsigned long long* stats, bool pack16) {
  __shared__ GroupTable<kShortSlots> T;
  const int64_t i = c0 + blockIdx.x;
  if (lg_ptr[i + 1] - lg_ptr[i] > kShortRow) return;  // uniform
  const int64_t p = group_row<kWrite, kShortThreads, kShortSlots>(T, i, lg_ptr, up_first, rec, gcount, obase_of,
                                                                  cap0, grec, gcnt, gna, elig, srows, nsrows, flags, pack16);
  // one pass of the grouping reports the parts; a row of one part is the
  // common case and needs no report (the host's maximum starts at 1)
  if (stats && threadIdx.x == 0 && (p < 0 || p > 1)) {
    if (p < 0) atomicAdd(&stats[kStRegrouped], 1ull);
    atomicMax(&stats[kStMaxParts], (unsigned long long)(p < 0 ? -p : p));
  }
}

// Long rows: rows[0 .. *nrows), each block pulling the next from `queue`.
template <bool kWrite>
__global__ __launch_bounds__(kLongThreads) void k_group_long(
    const int32_t* __restrict__ rows, const unsigned long long* __restrict__ nrows,
    unsigned long long* queue,
    const int64_t* __restrict__ lg_ptr, const int32_t* __restrict__ up_first,
    const uint4* __restrict__ rec, int64_t* gcount, const int64_t* __restrict__ obase_of,
    int64_t cap0, uint4* grec, void* gcnt, int32_t* gna, int32_t* elig, int32_t* srows, unsigned long long* nsrows,
    int32_t* flags, unsigned long long* stats, bool pack16) {
  __shared__ GroupTable<kLongSlots> T;
  __shared__ int64_t s_q;
  const int64_t n = int64_t(*nrows);
  unsigned long long regrouped = 0, most = 0;  // this block's rows (thread 0's copy is used)
  for (;;) {  // rows pulled from a counter; every block leaves once the list is taken
    if (threadIdx.x == 0) s_q = int64_t(atomicAdd(queue, 1ull));
    __syncthreads();
    const int64_t q = s_q;
    __syncthreads();
    if (q >= n) break;
    const int64_t p = group_row<kWrite, kLongThreads, kLongSlots>(T, rows[q], lg_ptr, up_first, rec, gcount,
                                                                  obase_of, cap0, grec, gcnt, gna, elig, srows, nsrows, flags, pack16);
    regrouped += p < 0 ? 1ull : 0ull;
    most = max(most, (unsigned long long)(p < 0 ? -p : p));
  }
  if (stats && threadIdx.x == 0 && most > 0) {
    if (regrouped) atomicAdd(&stats[kStRegrouped], regrouped);
    atomicMax(&stats[kStMaxParts], most);
  }
}

// The rows of [c0, c1) longer than kShortRow, appended to rows[] (any order).
__global__ void k_long_rows(int64_t c0, int64_t c1, const int64_t* __restrict__ lg_ptr,
                            int32_t* rows, unsigned long long* nrows) {
  const int64_t i = c0 + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < c1 && lg_ptr[i + 1] - lg_ptr[i] > kShortRow) rows[atomicAdd(nrows, 1ull)] = int32_t(i);
}

// Per-row group statistics of rows [c0, c1): groups, groups with members
// above the centre, pairs of such groups (classified in full by the pair
// kernel) and the other pairs of groups (counted only when open).
__global__ __launch_bounds__(256) void k_group_stats(int64_t c0, int64_t c1, const int64_t* __restrict__ goff,
                                                     const int32_t* __restrict__ gna,
                                                     unsigned long long* stats) {
  const int64_t i = c0 + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  unsigned long long ng = 0, na = 0;
  if (i < c1) {
    ng = (unsigned long long)(goff[i + 1] - goff[i]);
    na = (unsigned long long)gna[i];
  }
  unsigned long long v[4] = {ng, na, na * (na - (na ? 1 : 0)) / 2,
                             ng * (ng - (ng ? 1 : 0)) / 2 - na * (na - (na ? 1 : 0)) / 2};
  __shared__ unsigned long long red[4][256 / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (int x = 0; x < 4; ++x) {
    for (int off = kWave / 2; off > 0; off >>= 1) v[x] += __shfl_xor(v[x], off, kWave);
    if (lane == 0) red[x][wave] = v[x];
  }
  __syncthreads();
  if (threadIdx.x < 4) {  // one atomic per block and counter
    unsigned long long t = 0;
    for (int w = 0; w < 256 / kWave; ++w) t += red[threadIdx.x][w];
    const int slot = kStGroups + int(threadIdx.x);  // groups, above, full pairs, open pairs
    if (t) atomicAdd(&stats[slot], t);
  }
}

// Pairs of groups (x < y) and each group with itself, weighted as above, a
// lane per pair: rows of few groups, and every row where one reaches 2^16
// neighbours.  512-thread blocks whose 8 histogram copies are shared by their
// waves, lane l adding to copy l % 8, flushed when the block leaves a graph:
// 32 KB of LDS per block, so 4 blocks (32 waves, as many as the registers
// allow) fit on a CU.  Lanes of one add that hit the same word are
// serialized, so the copies count: with every row of the medium workload
// counted here, 556 ms with 2 copies and 448 ms with 4 (256-thread blocks), 434
// ms with 8 (512-thread blocks), 538 ms with 16 (1024-thread blocks, 2 per
// CU), and 853 ms with a single histogram over the 2187 codes (no class table
// read).
constexpr int kGCopies = 8;
constexpr int kGThreads = 512;
// At most 100 scalar registers, so that a SIMD holds 8 of its waves (4 blocks
// of 512 threads per compute unit, the default launch); its loops left to
// themselves take 106 registers, which allow 7 waves per SIMD and so only 3
// blocks per compute unit (every row of medium: 403 ms at 3 blocks, 360 ms at 4).
template <bool kNarrow>
__global__ __launch_bounds__(kGThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_exact_grouped(
    const int64_t* __restrict__ edge_ptr, const int64_t* __restrict__ goff,
    const int64_t* __restrict__ gbase, int64_t cap0,
    const uint4* __restrict__ grec, const void* __restrict__ gcnt, const int32_t* __restrict__ gna,
    WorkItems I, const uint16_t* __restrict__ code_to_id3, unsigned long long* hist_out) {
  __shared__ uint16_t lut[kNumCodes];
  __shared__ unsigned long long hist[kGCopies * kGStride];
  // indexed by the reversed code; entries are byte offsets of the ids
  for (int t = threadIdx.x; t < kNumCodes; t += blockDim.x) lut[t] = uint16_t(code_to_id3[kNumCodes - 1 - t] * 8u);
  for (int t = threadIdx.x; t < kGCopies * kGStride; t += blockDim.x) hist[t] = 0ull;
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  unsigned long long* myhist = hist + (lane & (kGCopies - 1)) * kGStride;
  visit_many_graphs(I, [&](int g, const ItemRange& items) {
    int32_t i;
    int b;
    while (next_item(items, lane, i, b)) {
      const int64_t gb = gbase[i] - cap0;
      const int ng = int(goff[i + 1] - goff[i]);
      // groups with members above the centre at [0, na), the others at
      // [na, ng) + gap (gap = the row region's unused middle)
      const int na = gna[i];
      const int64_t gap = (gbase[i + 1] - gbase[i]) - ng;
      const uint32_t a = uint32_t(edge_ptr[i + 1] - edge_ptr[i]);
      const uint4* __restrict__ grow = grec + gb;
      using C = typename GroupCount<kNarrow>::T;
      const C* __restrict__ gc = static_cast<const C*>(gcnt) + gb;
      const uint4* __restrict__ growb = grow + gap;
      const C* __restrict__ gcb = gc + gap;
      const int kp = b * kWave + lane;
      const bool valid = kp < ng;
      Side k;
      uint32_t kn = 0, ka = 0;
      {
        const int64_t kpos = kp < na ? int64_t(kp) : kp + gap;
        const uint4 rk = valid ? grow[kpos] : make_uint4(0, 0, 0, 0);
        C ck = {};
        if (valid) ck = gc[kpos];
        k.m = rk.x;
        k.o = (rk.y >> 16) & 0xffu;
        k.s = __popc(rk.x);
        k.h = (unsigned long long)rk.z | ((unsigned long long)rk.w << 32);
        kn = cnt_all(ck);
        ka = cnt_above(ck);
      }
      kn &= 0xffffffu;
      ka &= 0xffffffu;
      const int blo = b * kWave;
      const int kmax = min(blo + kWave, ng);
      const uint32_t aks = a - k.s;
      const uint32_t k0 = 243u * st3(k.s) + 9u * st3(k.o);
      if (blo >= na) {  // no lane has members above the centre: open pairs only
        owalk<false>(grow, gc, 0, na, aks, k0, k, kn, kp, lut, myhist);
        owalk<false>(growb, gcb, na, blo, aks, k0, k, kn, kp, lut, myhist);
        owalk<true>(growb, gcb, blo, kmax, aks, k0, k, kn, kp, lut, myhist);
      } else if (blo + kWave <= na) {  // every lane has members above the centre
        gwalk<false, true, kNarrow>(grow, gc, 0, blo, aks, k, kn, ka, kp, lut, myhist);
        gwalk<true, false, kNarrow>(grow, gc, blo, kmax, aks, k, kn, ka, kp, lut, myhist);
      } else {  // j with members above the centre: every pair; the others: open only
        const int ka1 = min(kmax, na);
        gwalk<false, false, kNarrow>(grow, gc, 0, blo, aks, k, kn, ka, kp, lut, myhist);
        gwalk<true, false, kNarrow>(grow, gc, blo, ka1, aks, k, kn, ka, kp, lut, myhist);
        owalk<true>(growb, gcb, ka1, kmax, aks, k0, k, kn, kp, lut, myhist);
      }
      if (valid && ka >= 2u) {  // pairs inside the group: above the centre only
        const uint32_t r5 = uint32_t(__popcll(k.h));
        const uint32_t code = pair_code(a, k.s, k.o, k, k.s, r5);
        atomicAdd(hist_at(myhist, lut[kNumCodes - 1 - code]), uint64_t(ka) * (ka - 1u) / 2u);
      }
    }
  }, [&](int g) { hist_flush<kGCopies>(hist, g, hist_out); });
}

inline unsigned blocks(int64_t n, int t) { return unsigned((n + t - 1) / t); }

}  // namespace

namespace {

// The work items of rows [c0, c1) (pairs.h), built by one kernel.
struct Schedule {
  char* scratch = nullptr;
  GraphItems* graphs = nullptr;
  int32_t* order = nullptr;
  uint32_t* start[kItemLists] = {};
  uint32_t* queues = nullptr;  // [kItemLists][ng]
  int ng = 0;
  WorkItems items(int list, int g0, int g1) const {
    return WorkItems{graphs, order, start[list], queues + size_t(list) * ng, list, g0, g1};
  }
};

mochy_status build_schedule(mochy_ctx* ctx, const mochy_graph* g, int64_t c0, int64_t c1, const RowKinds& R,
                            Schedule& S) {
  const size_t ng = size_t(g->ng), rows = size_t(c1 - c0);
  const int lists = R.mfma ? kItemLists : 1;
  const mochy_status rc =
      device_alloc(ctx, (void**)&S.scratch,
                   ng * sizeof(GraphItems) + (rows + kItemLists * ng + size_t(lists) * (rows + ng)) * 4);
  if (rc != MOCHY_OK) return rc;
  S.ng = g->ng;
  S.graphs = (GraphItems*)S.scratch;
  S.queues = (uint32_t*)(S.graphs + ng);
  S.order = (int32_t*)(S.queues + kItemLists * ng);
  uint32_t* at = (uint32_t*)(S.order + rows);
  for (int l = 0; l < lists; ++l, at += rows + ng) S.start[l] = at;
  k_schedule<<<unsigned(ng), 1024, 0, ctx->stream>>>(c0, c1, g->geoff, R, S.graphs, S.order, S.start[kItemsLane],
                                                     S.start[kItemsFull], S.start[kItemsOpen], S.queues);
  return MOCHY_OK;
}

// Groups of rows [c0, c1) (see build_groups).
struct Groups {
  int64_t* goff = nullptr;
  uint4* rec = nullptr;
  void* cnt = nullptr;         // uint32_t (packed) or uint2
  int32_t* gna = nullptr;
  int32_t* elig = nullptr;
  int32_t* srows = nullptr;    // rows of several hash parts; *nsrows of them
  unsigned long long* nsrows = nullptr;  // and, next to it, a queue counter
  const int64_t* gbase = nullptr;
  int64_t cap0 = 0;
  void release(mochy_ctx* ctx) {
    device_free(ctx, goff);
    device_free(ctx, rec);
    device_free(ctx, cnt);
    device_free(ctx, gna);
    *this = Groups();
  }
};

// Groups of rows [c0, c1): goff[E+1] the prefix of the rows' group counts,
// row i's groups in grec / gcnt [gbase[i] - cap0, gbase[i + 1] - cap0): the
// gna[i] with members above the centre first, the others at the region's
// end (the region holds exactly the groups in the compact layout).  With up
// to ctx->group_cap_bytes of row capacity (a graph or a whole batch), one
// pass writes each row's groups at its line-graph offset (gbase = lg_ptr);
// otherwise, or if that capacity cannot be allocated, the groups are counted
// first and allocated exactly (gbase = goff, cap0 = 0).  Returns MOCHY_ENOMEM (nothing held) if
// the group arrays do not fit or a row could not be grouped; the caller then
// pairs every record.
mochy_status build_groups(mochy_ctx* ctx, const mochy_graph* g, int64_t c0, int64_t c1, Groups& G,
                          unsigned long long* stats, bool pack16) {
  hipStream_t st = ctx->stream;
  const int64_t E = g->E;
  int64_t* cntarr = nullptr;
  int64_t* tmp = nullptr;
  int32_t* longrows = nullptr;
  auto fail = [&](mochy_status rc) {
    device_free(ctx, cntarr);
    device_free(ctx, tmp);
    device_free(ctx, longrows);
    G.release(ctx);
    return rc;
  };
  MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small, g->lg_ptr + c0, 8, hipMemcpyDeviceToHost, st), fail);
  MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 1, g->lg_ptr + c1, 8, hipMemcpyDeviceToHost, st), fail);
  MOCHY_HIP_OR(hipStreamSynchronize(st), fail);
  const int64_t row0 = ctx->h_small[0];
  const int64_t cap = ctx->h_small[1] - row0;
  const size_t cbytes = pack16 ? 4 : 8;  // a group's counts
  // one pass into row capacity (a graph or a batch) when that fits the limit
  bool by_rows = cap * 24 <= ctx->group_cap_bytes;
  mochy_status rc;
  if ((rc = device_alloc(ctx, (void**)&cntarr, size_t(E + 1) * 8)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&tmp, scan_tmp_elems(E + 1) * 8)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&G.goff, size_t(E + 1) * 8)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&G.gna, size_t(std::max<int64_t>(E, 1)) * 12 + 24)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&longrows, size_t(std::max<int64_t>(c1 - c0, 1)) * 4)) != MOCHY_OK)
    return fail(rc);
  // one block: nsrows and its queue (8-byte aligned, first), gna, elig, srows
  G.nsrows = (unsigned long long*)G.gna;
  int32_t* const gna = (int32_t*)(G.nsrows + 2);
  G.elig = gna + E;
  G.srows = G.elig + E;
  launch_fill_u32(G.nsrows, 0u, 16, st);
  launch_fill_u32(cntarr, 0u, size_t(E + 1) * 8, st);
  launch_fill_u32(ctx->d_flags + 3, 0u, 4, st);
  // the rows too long for the short-row table, listed once; two queue
  // counters (one per grouping pass), all in the context's small scratch
  unsigned long long* nlong = (unsigned long long*)(ctx->d_small + 508);
  unsigned long long* lqueue = nlong + 1;  // [2]
  launch_fill_u32(nlong, 0u, 3 * 8, st);
  if (c1 > c0) k_long_rows<<<blocks(c1 - c0, 256), 256, 0, st>>>(c0, c1, g->lg_ptr, longrows, nlong);
  const unsigned lgrid = unsigned(ctx->num_cus);  // one 160 KB block per CU
  if (by_rows && ((ctx->test_faults & 1) ||
                  device_alloc(ctx, (void**)&G.rec, size_t(cap + kGroupSlack) * 16) != MOCHY_OK ||
                  device_alloc(ctx, &G.cnt, size_t(cap + kGroupSlack) * cbytes) != MOCHY_OK)) {
    // no room for the row capacity: count the groups first and allocate them exactly
    device_free(ctx, G.rec);
    device_free(ctx, G.cnt);
    G.rec = nullptr;
    G.cnt = nullptr;
    ctx->err.clear();
    by_rows = false;
  }
  if (by_rows) {
    G.gbase = g->lg_ptr;
    G.cap0 = row0;
    if (c1 > c0) {
      k_group_short<true><<<unsigned(c1 - c0), kShortThreads, 0, st>>>(
          c0, g->lg_ptr, g->up_first, g->rec, cntarr, g->lg_ptr, row0, G.rec, G.cnt, gna, G.elig, G.srows, G.nsrows,
          ctx->d_flags + 3, stats, pack16);
      k_group_long<true><<<lgrid, kLongThreads, 0, st>>>(
          longrows, nlong, lqueue, g->lg_ptr, g->up_first, g->rec, cntarr, g->lg_ptr, row0,
          G.rec, G.cnt, gna, G.elig, G.srows, G.nsrows, ctx->d_flags + 3, stats, pack16);
    }
    launch_exclusive_scan_i64(cntarr, G.goff, E + 1, tmp, st);
  } else {
    G.gbase = G.goff;
    G.cap0 = 0;
    if (c1 > c0) {
      k_group_short<false><<<unsigned(c1 - c0), kShortThreads, 0, st>>>(
          c0, g->lg_ptr, g->up_first, g->rec, cntarr, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
          ctx->d_flags + 3, stats, pack16);
      k_group_long<false><<<lgrid, kLongThreads, 0, st>>>(
          longrows, nlong, lqueue, g->lg_ptr, g->up_first, g->rec, cntarr, nullptr, 0,
          nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, ctx->d_flags + 3, stats, pack16);
    }
    launch_exclusive_scan_i64(cntarr, G.goff, E + 1, tmp, st);
    MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small, G.goff + E, 8, hipMemcpyDeviceToHost, st), fail);
    MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 1, ctx->d_flags + 3, 4, hipMemcpyDeviceToHost, st), fail);
    MOCHY_HIP_OR(hipStreamSynchronize(st), fail);
    if (*reinterpret_cast<int32_t*>(ctx->h_small + 1) != 0) return fail(MOCHY_ENOMEM);
    const int64_t ngroups = ctx->h_small[0];
    if ((rc = device_alloc(ctx, (void**)&G.rec, size_t(ngroups + kGroupSlack) * 16)) != MOCHY_OK ||
        (rc = device_alloc(ctx, &G.cnt, size_t(ngroups + kGroupSlack) * cbytes)) != MOCHY_OK)
      return fail(rc);
    // the same grouping again, written this time (its parts were reported above)
    if (c1 > c0) {
      k_group_short<true><<<unsigned(c1 - c0), kShortThreads, 0, st>>>(
          c0, g->lg_ptr, g->up_first, g->rec, nullptr, G.goff, 0, G.rec, G.cnt, gna, G.elig, G.srows, G.nsrows,
          ctx->d_flags + 3, nullptr, pack16);
      k_group_long<true><<<lgrid, kLongThreads, 0, st>>>(
          longrows, nlong, lqueue + 1, g->lg_ptr, g->up_first, g->rec, nullptr, G.goff, 0,
          G.rec, G.cnt, gna, G.elig, G.srows, G.nsrows, ctx->d_flags + 3, nullptr, pack16);
    }
  }
  if (c1 > c0)
    k_group_stats<<<blocks(c1 - c0, 256), 256, 0, st>>>(c0, c1, G.goff, gna, stats);
  MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 1, ctx->d_flags + 3, 4, hipMemcpyDeviceToHost, st), fail);
  MOCHY_HIP_OR(hipStreamSynchronize(st), fail);
  if (*reinterpret_cast<int32_t*>(ctx->h_small + 1) != 0) return fail(MOCHY_ENOMEM);
  device_free(ctx, cntarr);
  device_free(ctx, tmp);
  device_free(ctx, longrows);
  cntarr = nullptr;
  tmp = nullptr;
  longrows = nullptr;
  MOCHY_HIP_OR(hipGetLastError(), fail);
  return MOCHY_OK;
}

}  // namespace

mochy_status exact_device(mochy_ctx* ctx, const mochy_graph* g, int64_t c0, int64_t c1,
                          int64_t* d_hist) {
  hipStream_t st = ctx->stream;
  const int ng = g->ng;
  unsigned long long* stats = (unsigned long long*)(ctx->d_small + kExactStatsSlot);
  launch_fill_u32(d_hist, 0u, size_t(ng) * kHistSlots * 8, st);
  launch_fill_u32(stats, 0u, kStBatches * 8, st);
  ctx->table_bytes = 0;
  if (c1 <= c0 || g->max_deg < 2) return MOCHY_OK;
  if (g->max_deg >= (1 << 24)) {  // group sizes are multiplied as 24-bit numbers
    ctx->err = "a line-graph row of 2^24 or more neighbours";
    return MOCHY_EUNSUPPORTED;
  }
  Groups G;
  mochy_status rc;
  phase_begin(ctx, kPhSched);
  // rows shorter than 2^16 neighbours: the group counts fit 16 bits and a
  // pair's weight (below 2^32) is a two-term dot product of packed counts
  // (test bit 4 takes the 48-bit form regardless)
  const bool narrow = g->max_deg < (1 << 16) && !(ctx->test_faults & 16);
  bool grouped = ctx->group_neighbours;
  if (grouped) {
    rc = (ctx->test_faults & 4) && ng > 2
             ? MOCHY_ENOMEM  // forced for tests of the batch split
             : build_groups(ctx, g, c0, c1, G, stats, narrow);
    if (rc == MOCHY_ENOMEM && ng > 1) {
      return rc;  // a batch: the caller splits it and counts the parts with groups
    } else if (rc == MOCHY_ENOMEM) {  // not enough memory for one graph's groups: pair every record
      grouped = false;
      ctx->err.clear();
      launch_fill_u32(stats, 0u, kStBatches * 8, st);
    } else if (rc != MOCHY_OK) {
      return rc;
    }
  }
  Schedule S;
  auto release = [&](mochy_status s) {
    device_free(ctx, S.scratch);
    G.release(ctx);
    S = Schedule();
    return s;
  };
  // rows of many groups go to the matrix-core kernels
  const bool mfma = grouped && narrow && g->max_deg >= kMfmaMinDegree;
  ctx->routes |= (grouped ? MOCHY_ROUTE_GROUPS : MOCHY_ROUTE_EVERY_PAIR) | (mfma ? MOCHY_ROUTE_MATRIX : 0u);
  const int32_t* const gna = G.gna ? (const int32_t*)(G.nsrows + 2) : nullptr;
  const RowGroups RG = {g->edge_ptr, G.goff, G.gbase, G.cap0, G.rec, (const uint32_t*)G.cnt, gna, G.elig};
  rc = build_schedule(ctx, g, c0, c1, RowKinds{g->lg_ptr, G.goff, gna, g->edge_ptr, grouped, mfma}, S);
  if (rc != MOCHY_OK) return release(rc);
  if (mfma)
    launch_sort_groups(ctx->num_cus, G.srows, G.nsrows, G.nsrows + 1, RG, G.rec, (uint32_t*)G.cnt, G.elig, st);
  phase_end(ctx, kPhSched);
  phase_begin(ctx, kPhPairs);
  // one launch over all graphs, or one per graph (MOCHY_OPT_BATCH_LAUNCH);
  // no more waves than work items there can be
  const int step = ctx->batch_launch == 2 ? 1 : ng;
  const int64_t entries = 2 * g->W;
  const auto at_most = [](unsigned grid, int64_t items, int waves) {
    return unsigned(std::max<int64_t>(1, std::min<int64_t>(grid, (items + waves - 1) / waves)));
  };
  const unsigned lane_grid = unsigned(ctx->num_cus) * unsigned(ctx->pair_blocks);  // blocks of 4 waves
  unsigned long long* const h = (unsigned long long*)d_hist;
  for (int a = 0; a < ng; a += step) {
    const int b = std::min(ng, a + step);
    if (!grouped) {
      k_exact_main<<<at_most(std::max(1u, lane_grid * 256u / unsigned(kMainThreads)), entries / kWave + g->E, kMainWaves),
                     kMainThreads, 0, st>>>(
          g->edge_ptr, g->lg_ptr, g->up_first, g->rec, S.items(kItemsLane, a, b), ctx->d_code_to_id3, h,
          (ctx->test_faults & 16) ? kFlushVisitsTest : kFlushVisits);
      continue;
    }
    if (mfma) {
      const int64_t tiles = entries / kMfmaCols + g->E;
      // 75 KB of LDS (k_pairs_full) or the registers (k_pairs_open): two blocks reside per CU
      launch_pairs_open(at_most(unsigned(ctx->num_cus) * 2u, tiles, 4), RG, S.items(kItemsOpen, a, b),
                        ctx->d_code_to_id3, h, st);
      launch_pairs_full(at_most(unsigned(ctx->num_cus) * 2u, tiles, 4), RG, S.items(kItemsFull, a, b),
                        ctx->d_code_to_id3, h, st);
    }
    (narrow ? k_exact_grouped<true> : k_exact_grouped<false>)<<<
        at_most(std::max(1u, lane_grid * 256u / unsigned(kGThreads)), entries / kWave + g->E, kGThreads / kWave),
        kGThreads, 0, st>>>(g->edge_ptr, G.goff, G.gbase, G.cap0, G.rec, G.cnt, gna, S.items(kItemsLane, a, b),
                            ctx->d_code_to_id3, h);
  }
  phase_end(ctx, kPhPairs);
  MOCHY_HIP_OR(hipGetLastError(), release);
  release(MOCHY_OK);  // stream-ordered; the correction reads rows and records only
  phase_begin(ctx, kPhCorrect);
  rc = correct_device(ctx, g, c0, c1, d_hist, stats);
  if (rc != MOCHY_OK) return rc;
  phase_end(ctx, kPhCorrect);
  MOCHY_HIP(hipGetLastError());
  MOCHY_HIP(hipMemcpyAsync(ctx->h_small + kExactStatsSlot, stats, kStBatches * 8,
                           hipMemcpyDeviceToHost, st));
  MOCHY_HIP(hipStreamSynchronize(st));
  phases_collect(ctx);
  const int64_t* hs = ctx->h_small + kExactStatsSlot;
  for (int x = 0; x < kStBatches; ++x)  // the device counters (the batch count is the host's)
    ctx->exact_stats[x] = x == kStMaxParts ? std::max(ctx->exact_stats[x], hs[x]) : ctx->exact_stats[x] + hs[x];
  if (grouped) {
    ctx->exact_stats[kStRows] += c1 - c0;
    // rows of one hash part are not reported by the kernels
    ctx->exact_stats[kStMaxParts] = std::max<int64_t>(ctx->exact_stats[kStMaxParts], 1);
  }
  return MOCHY_OK;
}
