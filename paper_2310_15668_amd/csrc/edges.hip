// MoCHy-A (Algorithm 4, hyperedge sampling) and per-hyperedge profiles.
// Sample n draws Philox4x32-10 with counter (lo32 n, hi32 n, 1, 0) and key
// (lo32 seed, hi32 seed); u = (x1 << 32) | x0 picks hyperedge
// floor(u * |E| / 2^64).  Every instance containing the sampled e_i gets one
// hit: the pairs of N_i and the paths e_i - e_j - e_k (e_k in N_j outside N_i
// and e_i).  A profile is the same count for each hyperedge of a range.
//
// Scanning the row of every neighbour of e_i costs the square of the degree,
// 3.6e8 entries a sample on 85,353 hyperedges drawn over 20,000 nodes (mean
// degree 13,500).  Here N_i is grouped instead by what its records say (mask
// of e_i's nodes, outside count, heavy outside nodes): 5,800 groups there, and
// 3e7 pairs of groups.  With q = |e_j ∩ e_k| as the records give it (the
// shared nodes of e_i and the shared heavy nodes) the counts of e_i are
//
//     sum over pairs {j, k} of N_i of           class(j, k, q)
//   + sum over j in N_i, k in N_j, k != i of    path(j, k, |e_j ∩ e_k|)
//   - sum over ordered pairs (j, k) with q > 0  path(j, k, q)
//
// where path(j, k, q) is the class of the three as if e_k did not meet e_i; a
// path whose e_k does is in the second sum and taken back in the third.  Pairs
// of N_i sharing a light node outside e_i have a larger overlap than their
// records give: they are listed from the lists of those nodes, and both sums
// are moved from q to the true overlap.  The second sum needs of row j only
// its histogram by (|e_j ∩ e_k|, |e_k|), made once for all samples.  All sums
// are of whole numbers modulo 2^64, so the counts are the same as a scan's.
//
// Where no row is longer than kScanDegree the rows are scanned all the same
// (sampled.hip), and where the scratch for one sample's groups cannot be had.
#include "classify.h"
#include "common.h"
#include "pairs.h"
#include "rng.h"
#include "walk.h"

#include <algorithm>

namespace {

constexpr int kHsThreads = 256;
constexpr int kHsWaves = kHsThreads / kWave;
constexpr int kLightThreads = 512, kLightWaves = kLightThreads / kWave;
constexpr int kRankWords = 4;      // words of a row's bitmap to a rank
constexpr int64_t kNoEntries = -2;
constexpr int kGroupChunk = 1024;  // row entries a block groups
// A work item is 512 groups k against up to 512 << z groups j, or the
// histograms of 256 << z neighbours; z is the largest up to kMaxItemShift that
// leaves kMinItems items, as an item of a profile ends with adding its counters
// to the profile.
constexpr int kPairCols = 512, kSumChunk = 256, kMaxItemShift = 4;
constexpr int64_t kMinItems = 2048;
constexpr int kPairThreads = 512;
static_assert((int64_t(kSumChunk) << kMaxItemShift) * 200000 < (int64_t(1) << 32), "counters of a sum item");
constexpr int kNodePull = 4;       // light nodes (or neighbours) a wave takes from its block's share at a time
constexpr int kShortRow = 4;       // rows of fewer than 1 / kShortRow neighbours for each light node
constexpr int kNodeBlock = 1024;   // nodes a block sorts out light ones from
constexpr unsigned kLightBlocksPerCu = 6;  // blocks of the light pairs' kernel launched per CU, at least one a sample
constexpr int kMembers = kWave;    // members of a node's list held at a time
constexpr int kHistW = MOCHY_MAX_EDGE;  // row histogram: |e_k| fastest, then |e_j ∩ e_k| = 1 .. |e_j|
// Rows of up to this many neighbours are scanned: a scan is one kernel over
// them, groups are six and their scratch.  Samples of flat hypergraphs, groups
// and scan in ms, by the longest row: of 17 (30,000 hyperedges) 0.076 and 0.053
// (5 samples), 0.585 and 0.206 (10,000); of 40 0.072 and 0.065, 0.66 and 0.34;
// of 65 0.074 and 0.079, 0.85 and 0.57; of 141 0.086 and 0.134, 1.40 and 1.44;
// of 358 0.141 and 0.383, 4.4 and 5.3.
constexpr int32_t kScanDegree = 64;
// scratch of one batch of samples (tables of their rows' groups)
constexpr size_t kBatchBytes = size_t(512) << 20;
constexpr int64_t kMaxBatch = 32768;    // grid rows

// What the pair kernel reads of a group besides its record: members, and the
// parts of its path codes that do not depend on the other group.
struct GroupInfo {
  uint32_t n;     // members
  uint32_t base;  // path code digits fixed by |e_i ∩ e_j| (doubled, reversed)
  uint32_t far;   // outside count + 2 | (size + 2) << 16
  uint32_t kso;   // |e_i ∩ e_j| | outside count << 16
};

// Scratch of a batch: sample q's table of slots (representative's position in
// the row + 1, members), its groups' slots, records and infos.
struct HsScratch {
  int64_t* sample_i;   // [s] hyperedge
  int64_t* item_off;   // [s + 2] prefix of the pair kernel's work items, and their shift z
  uint32_t* ngroups;   // [s]
  uint2* table;        // [s][slots]
  uint32_t* gslot;     // [s][rows]
  uint4* grec;         // [s][rows]
  GroupInfo* ginfo;    // [s][rows]
  int64_t slots, rows;
  // of the whole call
  uint8_t* need;       // [E] 1: a sample needs the row's histogram, 2: it is made
  uint32_t* rowh;      // [nnz][kHistW] row histograms, row j's at edge_ptr[j]
  int32_t* lnodes;     // [nnz] light nodes in two hyperedges or more, graph g's at gnoff[g]
  uint32_t* nlight;    // [graphs] how many
  ulonglong2* lbits;   // [E] the light nodes of each hyperedge as bits (light_bits)
};

// A light node's bit under each of two hashes; kDistinct in a set's word if no
// two of its nodes share a bit there.
constexpr unsigned long long kDistinct = 1ull << 63;
__device__ __forceinline__ ulonglong2 light_bits(int32_t v) {
  return make_ulonglong2(1ull << __umulhi(uint32_t(v) * 0x9e3779b1u, 63u),
                         1ull << __umulhi((uint32_t(v) ^ 0x5bd1e995u) * 0xc2b2ae35u, 63u));
}

__host__ __device__ __forceinline__ uint32_t table_slots(int64_t d) {  // at most 3/4 full
  uint32_t n = 16;
  while (int64_t(n) * 3 < d * 4) n <<= 1;
  return n;
}

// Twice the reversed path code of (e_i, e_j, e_k), |e_i ∩ e_k| = 0, as
// pair_rcode2 gives it: digits enter as max(2 - R, 0).  The digits of R1 =
// a - p and R4 = p (and of R6 = R7 = 0) depend on e_j only: path_base.  Those
// of R2 = b - p - q and R3 = c - q are held to 2 where the difference is
// negative, as it can be for an e_k that meets e_i, whose path is taken back.
constexpr uint32_t kPathFixed = 2u * (243u + 729u);  // digits of R6 = R7 = 0
__device__ __forceinline__ uint32_t path_base(uint32_t a, uint32_t p) {
  return 2u * (usat(2u, a - p) + 27u * usat(2u, p) + kPathFixed);
}
__device__ __forceinline__ uint32_t path_code2(uint32_t base, uint32_t o, uint32_t c, uint32_t q) {
  const uint32_t d2 = min(usat(q + 2u, o), 2u), d3 = min(usat(q + 2u, c), 2u);
  return base + 2u * (3u * d2 + 9u * d3 + 81u * usat(2u, q));
}

// Batch start: the hyperedge of each sample (kProfile: hyperedges n0 .. in
// order), an empty table for its row, and on the first batch no row marked, no
// light node listed and each hyperedge's light nodes as bits.
template <bool kProfile>
__global__ __launch_bounds__(kHsThreads) void k_hs_begin(int64_t n0, int64_t s, uint64_t seed, int64_t E,
                                                         const int64_t* __restrict__ lg_ptr, HsScratch t,
                                                         bool first, int ng, const int64_t* __restrict__ edge_ptr,
                                                         const int32_t* __restrict__ edge_nodes,
                                                         const int8_t* __restrict__ heavy_bit) {
  if (first) {
    const int64_t at = int64_t(blockIdx.x) * kHsThreads + threadIdx.x, step = int64_t(gridDim.x) * kHsThreads;
    for (int64_t x = at; x < (E + 15) / 16; x += step) reinterpret_cast<uint4*>(t.need)[x] = make_uint4(0, 0, 0, 0);
    for (int64_t x = at; x < ng; x += step) t.nlight[x] = 0u;
    for (int64_t x = at; x < E; x += step) {
      ulonglong2 bits = make_ulonglong2(0ull, 0ull);
      int n = 0;
      for (int64_t r = edge_ptr[x]; r < edge_ptr[x + 1]; ++r) {
        const int32_t v = edge_nodes[r];
        if (heavy_bit[v] >= 0) continue;
        const ulonglong2 b = light_bits(v);
        bits.x |= b.x;
        bits.y |= b.y;
        ++n;
      }
      if (__popcll(bits.x) == n) bits.x |= kDistinct;
      if (__popcll(bits.y) == n) bits.y |= kDistinct;
      t.lbits[x] = bits;
    }
  }
  for (int64_t q = blockIdx.x; q < s; q += gridDim.x) {
    const uint64_t n = uint64_t(n0) + uint64_t(q);
    int64_t i = int64_t(n);
    if (!kProfile) {
      const uint4 x = philox_4x32_10(make_uint4(uint32_t(n), uint32_t(n >> 32), 1u, 0u), uint32_t(seed),
                                     uint32_t(seed >> 32));
      i = int64_t(__umul64hi((uint64_t(x.y) << 32) | x.x, uint64_t(E)));
    }
    if (threadIdx.x == 0) {
      t.sample_i[q] = i;
      t.ngroups[q] = 0u;
    }
    uint4* tab = reinterpret_cast<uint4*>(t.table + q * t.slots);
    const uint32_t n16 = table_slots(lg_ptr[i + 1] - lg_ptr[i]) / 2;
    for (uint32_t x = threadIdx.x; x < n16; x += kHsThreads) tab[x] = make_uint4(0, 0, 0, 0);
  }
}

__device__ __forceinline__ uint32_t group_hash(const uint4& r) {
  uint32_t h = r.x * 0x9e3779b1u ^ (r.y & 0xffu) * 0x85ebca77u;
  h = (h ^ (h >> 15)) + r.z * 0xc2b2ae3du;
  h = (h ^ (h >> 13)) * 0x27d4eb2fu + r.w * 0x165667b1u;
  h = (h ^ (h >> 16)) * 0x9e3779b1u;
  return h ^ (h >> 15);
}

// Groups of a sample's row, kGroupChunk entries a block: an entry takes a free
// slot of the table or joins the slot whose representative has an equal record
// (records are read-only, so a slot is whole as soon as it is taken).  Marks
// the rows whose histograms the sample needs.
__global__ __launch_bounds__(kHsThreads) void k_hs_group(const int64_t* __restrict__ lg_ptr,
                                                         const int32_t* __restrict__ lg_col,
                                                         const uint4* __restrict__ rec, HsScratch t) {
  const int64_t q = blockIdx.y;
  const int64_t i = t.sample_i[q];
  const int64_t base = lg_ptr[i];
  const int64_t d = lg_ptr[i + 1] - base;
  const uint32_t mask = table_slots(d) - 1u;
  uint2* tab = t.table + q * t.slots;
  const int64_t p1 = min(d, int64_t(blockIdx.x + 1) * kGroupChunk);
  for (int64_t p = int64_t(blockIdx.x) * kGroupChunk + threadIdx.x; p < p1; p += kHsThreads) {
    const uint4 r = rec[base + p];
    const int32_t j = lg_col[base + p];
    if (t.need[j] == 0) t.need[j] = 1;
    for (uint32_t s = group_hash(r) & mask;; s = (s + 1u) & mask) {
      uint32_t held = __hip_atomic_load(&tab[s].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (held == 0u) held = atomicCAS(&tab[s].x, 0u, uint32_t(p) + 1u);
      if (held == 0u) {
        const uint32_t g = atomicAdd(&t.ngroups[q], 1u);
        t.gslot[q * t.rows + g] = s;
        t.grec[q * t.rows + g] =
            make_uint4(r.x, uint32_t(__popc(r.x)) | (2u * uint32_t(__popc(r.x)) + 4u) << 8 | (r.y & 0xffu) << 16,
                       r.z, r.w);
      } else {
        const uint4 o = rec[base + held - 1u];
        if (o.x != r.x || (o.y & 0xffu) != (r.y & 0xffu) || o.z != r.z || o.w != r.w) continue;
      }
      atomicAdd(&tab[s].y, 1u);
      break;
    }
  }
}

__host__ __device__ __forceinline__ int64_t pair_items(uint32_t groups, int z) {  // chunk x of k meets j < kPairThreads (x + 1)
  const int64_t nx = (groups + kPairThreads - 1) / kPairThreads;
  const int64_t r = int64_t(kPairCols / kPairThreads) << z;
  const int64_t full = nx / r, rest = nx % r;
  return r * full * (full + 1) / 2 + rest * (full + 1);
}

// Block 0: the prefix of the samples' work items, and the queue.  The next,
// kInfoParts to a sample: the groups' infos, their tables being complete.  The
// others, on the first batch: the light nodes.
constexpr int kInfoParts = 8;
constexpr int kItemThreads = 256;
__global__ __launch_bounds__(kItemThreads) void k_hs_items(int64_t s, const int64_t* __restrict__ lg_ptr,
                                                           const int64_t* __restrict__ edge_ptr, HsScratch t,
                                                           int64_t V, int ng, const int64_t* __restrict__ gvoff,
                                                           const int64_t* __restrict__ gnoff,
                                                           const int64_t* __restrict__ node_ptr,
                                                           const int8_t* __restrict__ heavy_bit,
                                                           unsigned long long* queue) {
  if (int64_t(blockIdx.x) > s * kInfoParts) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t b0 = (int64_t(blockIdx.x) - 1 - s * kInfoParts) * kNodeBlock;
    for (int64_t v0 = b0 + threadIdx.x - lane; v0 < min(V, b0 + kNodeBlock); v0 += kItemThreads) {
      const int64_t v = v0 + lane;
      unsigned long long todo = __ballot(v < V && node_ptr[v + 1] - node_ptr[v] >= 2 && heavy_bit[v] < 0);
      while (todo) {  // the nodes of one graph at a time
        const int64_t u = v0 + __ffsll((long long)todo) - 1;
        int lo = 0, hi = ng;
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (gvoff[mid] <= u) lo = mid; else hi = mid;
        }
        const unsigned long long mine = __ballot(((todo >> lane) & 1ull) && v < gvoff[lo + 1]);
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&t.nlight[lo], uint32_t(__popcll(mine)));
        at = uint32_t(uniform(int(at)));
        if ((mine >> lane) & 1ull)
          t.lnodes[gnoff[lo] + at + __popcll(mine & ((1ull << lane) - 1ull))] = int32_t(v);
        todo &= ~mine;
      }
    }
    return;
  }
  if (blockIdx.x > 0) {
    const int64_t q = int64_t(blockIdx.x - 1) / kInfoParts;
    const int64_t i = t.sample_i[q];
    const uint32_t a = uint32_t(edge_ptr[i + 1] - edge_ptr[i]);
    const uint32_t n = t.ngroups[q];
    for (uint32_t g = (blockIdx.x - 1) % kInfoParts * kItemThreads + threadIdx.x; g < n; g += kInfoParts * kItemThreads) {
      const uint32_t y = t.grec[q * t.rows + g].y;
      const uint32_t p = y & 0xffu, o = y >> 16;
      GroupInfo f;
      f.n = t.table[q * t.slots + t.gslot[q * t.rows + g]].y;
      f.base = path_base(a, p);
      f.far = (o + 2u) | (p + o + 2u) << 16;
      f.kso = p | o << 16;
      t.ginfo[q * t.rows + g] = f;
    }
    return;
  }
  __shared__ int64_t wsum[kItemThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  auto items = [&](int64_t q, int z) {
    const int64_t i = t.sample_i[q];
    return pair_items(t.ngroups[q], z) + (lg_ptr[i + 1] - lg_ptr[i] + (int64_t(kSumChunk) << z) - 1) / (int64_t(kSumChunk) << z);
  };
  int64_t all[kMaxItemShift + 1] = {};
  for (int64_t q = threadIdx.x; q < s; q += kItemThreads)
#pragma unroll
    for (int z = 1; z <= kMaxItemShift; ++z) all[z] += items(q, z);
  int z = 0;
#pragma unroll
  for (int y = 1; y <= kMaxItemShift; ++y) {
    const int64_t n = wave_sum_i64(all[y]);
    if (lane == 0) wsum[wave] = n;
    __syncthreads();
    int64_t sum = 0;
    for (int w = 0; w < kItemThreads / kWave; ++w) sum += wsum[w];
    __syncthreads();
    if (sum >= kMinItems) z = y;
  }
  int64_t run = 0;
  for (int64_t q0 = 0; q0 < s; q0 += kItemThreads) {
    const int64_t q = q0 + threadIdx.x;
    const int64_t n = q < s ? items(q, z) : 0;
    const int64_t incl = wave_incl_scan_i64(n, lane);
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    int64_t before = run;
    for (int w = 0; w < kItemThreads / kWave; ++w) {
      if (w < wave) before += wsum[w];
      run += wsum[w];
    }
    if (q < s) t.item_off[q] = before + incl - n;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    t.item_off[s] = run;
    t.item_off[s + 1] = z;
    *queue = 0ull;
  }
}

// One wave per marked row j: entries by (|e_j ∩ e_k|, |e_k|), 32 |e_j|
// counters.  Bound by the read of the rows' size
// words, 2 bytes an entry: 0.77 ms for the 1.15e9 entries of 85,353 rows.  A
// row once made (mark 2) serves later batches.
__global__ __launch_bounds__(kHsThreads) void k_hs_rows(int64_t E, const int64_t* __restrict__ edge_ptr,
                                                        const int64_t* __restrict__ lg_ptr,
                                                        const uint16_t* __restrict__ rsz, HsScratch t) {
  __shared__ uint32_t s_h[kHsWaves][MOCHY_MAX_EDGE * kHistW];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t j = int64_t(blockIdx.x) * kHsWaves + wave;
  if (j >= E || t.need[j] != 1) return;  // whole wave; no block-wide barrier below
  uint32_t* h = s_h[wave];
  const int64_t es = edge_ptr[j];
  const int bins = int(edge_ptr[j + 1] - es) * kHistW;
  for (int x = lane; x < bins; x += kWave) h[x] = 0u;
  wave_sync();
  const int64_t p0 = lg_ptr[j], p1 = lg_ptr[j + 1];
  auto add = [&](uint32_t sz) { atomicAdd(&h[((sz & 0xffu) - 1u) * kHistW + (sz >> 8) - 1u], 1u); };
  // 8 entries to a load from the first 16-byte boundary on
  const int64_t a0 = min(p1, (p0 + 7) & ~int64_t(7)), a1 = max(a0, p1 & ~int64_t(7));
  if (p0 + lane < a0) add(rsz[p0 + lane]);
  for (int64_t p = a0 + lane * 8; p < a1; p += kWave * 8) {
    const uint4 v = *reinterpret_cast<const uint4*>(rsz + p);
    add(v.x & 0xffffu); add(v.x >> 16);
    add(v.y & 0xffffu); add(v.y >> 16);
    add(v.z & 0xffffu); add(v.z >> 16);
    add(v.w & 0xffffu); add(v.w >> 16);
  }
  if (a1 + lane < p1) add(rsz[a1 + lane]);
  wave_sync();
  for (int x = lane; x < bins; x += kWave) t.rowh[es * kHistW + x] = h[x];
  if (lane == 0) t.need[j] = 2;
}

// Class table by reversed code (2 bytes an entry): byte offsets of the ids'
// counters, `bytes` apart.
__device__ __forceinline__ void load_classes(const uint16_t* __restrict__ code_to_id3, uint16_t* lut, uint32_t bytes,
                                             int threads) {
  for (int t = threadIdx.x; t < kNumCodes; t += threads) lut[t] = uint16_t(code_to_id3[kNumCodes - 1 - t] * bytes);
}

// Empties the counters: what they gained less what was taken back.
__device__ __forceinline__ void flush(unsigned long long* plus, unsigned long long* minus, unsigned long long* out,
                                      int threads) {
  for (int t = threadIdx.x; t < kHistSlots; t += threads) {
    const unsigned long long v = plus[t] - minus[t];
    if (v) atomicAdd(&out[t], v);
    plus[t] = 0ull;
    minus[t] = 0ull;
  }
}

// Both halves held to 2
__device__ __forceinline__ uint32_t held2(uint32_t x) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, x), u16x2{2, 2}));
}

// A block's pairs by motif and the paths to be taken back by path code, in
// 4-byte counters, kCopies of each in neighbouring banks for the lanes to share
// out: lanes adding at one address take turns, and most pairs are of a few
// classes (with one counter each the adds took 66 cycles, with 16 copies no
// more than 4 lanes ever meet).
constexpr int kCopies = 16;
constexpr uint32_t kPathCodes = 243;
struct PairCounts {
  uint32_t motif[kHistSlots][kCopies];
  uint32_t path[kPathCodes][kCopies];
};

// The lane's group k against kN groups from j on (uniform): n_j n_k pairs of
// their class, and if they overlap as many paths each way to be taken back.  No
// branch: disjoint pairs add 0.  kBelow: only groups below k.
template <int kN, bool kBelow>
__device__ __forceinline__ void group_pairs(const uint4* __restrict__ grec, const GroupInfo* __restrict__ ginfo, int j,
                                            const uint4& rk, const GroupInfo& fk, int k, uint32_t aks2, uint32_t far_k,
                                            const uint16_t* lut, char* motif, char* path) {
  uint32_t code[kN], cj[kN], ck[kN], w[kN], wq[kN];
#pragma unroll
  for (int u = 0; u < kN; ++u) {
    const uint4 rj = grec[j + u];
    const GroupInfo fj = ginfo[j + u];
    uint32_t t2, tr;
    pair_counts(rj.x & rk.x, rj.z & rk.z, rj.w & rk.w, t2, tr);
    code[u] = pair_rcode2(t2, tr, aks2, rj.y, fk.kso);
    // q + 4 twice over; 2 + q less each side's outside count and the other's size
    const uint32_t q4 = dot2(tr, 0x00010001u, 0u);
    const uint32_t qq = q4 | q4 << 16;
    const uint32_t dj = held2(pk_usat(qq, fj.far));  // (R2 of the path through j, R3 of the path through k)
    const uint32_t dk = held2(pk_usat(qq, far_k));   // (R3 through j, R2 through k)
    const uint32_t r5 = q4 == 5u ? 162u : 0u;
    cj[u] = dot2(dk, 18u, dot2(dj, 6u, r5 + fj.base));
    ck[u] = dot2(dk, 6u << 16, dot2(dj, 18u << 16, r5 + fk.base));
    w[u] = (fj.n & 0xffffffu) * (kBelow && j + u >= k ? 0u : fk.n & 0xffffffu);
    wq[u] = q4 == 4u ? 0u : w[u];  // disjoint as far as the records tell
  }
#pragma unroll
  for (int u = 0; u < kN; ++u) code[u] = lut_at(lut, code[u]);
#pragma unroll
  for (int u = 0; u < kN; ++u) {
    atomicAdd(reinterpret_cast<uint32_t*>(path + cj[u] * (kCopies * 2)), wq[u]);
    atomicAdd(reinterpret_cast<uint32_t*>(path + ck[u] * (kCopies * 2)), wq[u]);
  }
#pragma unroll
  for (int u = 0; u < kN; ++u) atomicAdd(reinterpret_cast<uint32_t*>(motif + code[u]), w[u]);
}

// The motif of a doubled reversed code, from byte offsets of the counters.
__device__ __forceinline__ uint32_t motif_of(const uint16_t* lut, uint32_t code2) {
  return lut_at(lut, code2) / (kCopies * 4u);
}

// The same for one group j of many members, with 8-byte counters.
__device__ __forceinline__ void big_pair(const uint4& rj, const GroupInfo& fj, bool any, uint32_t a, const uint4& rk,
                                         const GroupInfo& fk, const uint16_t* lut, unsigned long long* plus,
                                         unsigned long long* minus) {
  if (!any || !fk.n) return;
  const uint32_t pj = fj.kso & 0xffffu, oj = fj.kso >> 16, pk = fk.kso & 0xffffu, ok = fk.kso >> 16;
  const uint32_t tt = uint32_t(__popc(rj.x & rk.x));
  const uint32_t r5 = uint32_t(__popc(rj.z & rk.z)) + uint32_t(__popc(rj.w & rk.w));
  const Side side = {rk.x, ok, pk, 0ull};
  const uint64_t w = uint64_t(fj.n) * fk.n;
  atomicAdd(&plus[motif_of(lut, 2u * (kNumCodes - 1 - pair_code(a, pj, oj, side, tt, r5)))], w);
  if (tt + r5 == 0u) return;
  atomicAdd(&minus[motif_of(lut, path_code2(fj.base, oj, pk + ok, tt + r5))], w);
  atomicAdd(&minus[motif_of(lut, path_code2(fk.base, ok, pj + oj, tt + r5))], w);
}

// Adds the block's 4-byte counters to its 8-byte ones by motif and empties
// them; the paths to `paths`.
__device__ __forceinline__ void flush_pairs(PairCounts& counts, const uint16_t* lut, unsigned long long* plus,
                                            unsigned long long* paths) {
  __syncthreads();
  for (uint32_t x = threadIdx.x; x < kHistSlots + kPathCodes; x += kPairThreads) {
    uint4* c = reinterpret_cast<uint4*>(x < kHistSlots ? counts.motif[x] : counts.path[x - kHistSlots]);
    unsigned long long n = 0;
#pragma unroll
    for (int y = 0; y < kCopies / 4; ++y) {
      const int z = (y + int(x)) & (kCopies / 4 - 1);  // in another order for each: fewer lanes in a bank
      n += (unsigned long long)c[z].x + c[z].y + c[z].z + c[z].w;
      c[z] = make_uint4(0, 0, 0, 0);
    }
    if (!n) continue;
    if (x < kHistSlots) atomicAdd(&plus[x], n);
    else atomicAdd(&paths[motif_of(lut, 2u * (x - kHistSlots + kPathFixed))], n);
  }
  __syncthreads();
}

// Work items from a queue.  Pairs: kPairThreads groups k, one to a lane, against
// up to kPairCols << z groups j <= k, read by scalar loads.  Sums: the histograms of
// kSumChunk << z neighbours' rows as paths, less the one that ends in e_i itself.
// Bound by vector issue, 37 instructions for 64 pairs and 3 LDS adds.  100
// samples on 85,353 hyperedges (5,800 groups to a sample): 2.3 ms.  With one
// 4-byte counter of each code and no table read it took 9.0 (66 cycles to an
// add, the lanes at one address taking turns), with 8-byte counters by motif
// 10.7.
template <bool kProfile>
__global__ __launch_bounds__(kPairThreads) void k_hs_pairs(
    int64_t n0, int64_t s, HsScratch t, const uint4* __restrict__ grecs, const GroupInfo* __restrict__ ginfos,
    const int64_t* __restrict__ edge_ptr, const int64_t* __restrict__ lg_ptr,
    const int32_t* __restrict__ lg_col, const uint16_t* __restrict__ rsz,
    const uint16_t* __restrict__ code_to_id3, unsigned long long* queue, unsigned long long* hist_out) {
  __shared__ uint16_t lut[kNumCodes];
  __shared__ unsigned long long plus[kHistSlots], minus[kHistSlots];
  __shared__ __align__(16) PairCounts counts;
  __shared__ int64_t s_item;
  __shared__ uint32_t s_nk[kPairThreads / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = uniform(threadIdx.x / kWave);
  load_classes(code_to_id3, lut, kCopies * 4u, kPairThreads);
  for (int x = threadIdx.x; x < kHistSlots; x += kPairThreads) plus[x] = minus[x] = 0ull;
  for (uint32_t x = threadIdx.x; x < sizeof(counts) / 4; x += kPairThreads) counts.motif[0][x] = 0u;
  char* motif = reinterpret_cast<char*>(&counts.motif[0][lane % kCopies]);
  char* path = reinterpret_cast<char*>(&counts.path[0][lane % kCopies]) - kPathFixed * kCopies * 4;
  uint64_t held = 0;  // no counter holds more, of the block's pairs since the last flush
  const int64_t total = t.item_off[s];
  const int z = int(t.item_off[s + 1]), cols = kPairCols << z, sums = kSumChunk << z;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = int64_t(atomicAdd(queue, 1ull));
    __syncthreads();
    const int64_t item = int64_t(uniform64(uint64_t(s_item)));
    if (item >= total) break;
    int64_t lo = 0, hi = s;  // the sample: last q with item_off[q] <= item
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (t.item_off[mid] <= item) lo = mid; else hi = mid;
    }
    const int64_t q = lo, i = t.sample_i[q];
    int64_t at = item - t.item_off[q];
    const uint32_t a = uint32_t(edge_ptr[i + 1] - edge_ptr[i]);
    const uint32_t ng = t.ngroups[q];
    const int64_t npair = pair_items(ng, z);
    if (at < npair) {
      int x = 0;  // chunk of kPairThreads k; its items cover j up to its last k
      for (;; ++x) {
        const int64_t n = (int64_t(x + 1) * kPairThreads + cols - 1) / cols;
        if (at < n) break;
        at -= n;
      }
      const uint4* __restrict__ grec = grecs + q * t.rows;
      const GroupInfo* __restrict__ ginfo = ginfos + q * t.rows;
      const int k0 = x * kPairThreads + wave * kWave, k = k0 + lane;
      const int j0 = int(at) * cols, j1 = min(min(j0 + cols, (x + 1) * kPairThreads), int(ng));
      uint4 rk = make_uint4(0, 0, 0, 0);
      GroupInfo fk = {0u, 2u * kPathFixed, 0u, 0u};  // past the row's end: 0 added at valid codes
      if (k < int(ng)) {
        rk = grec[k];
        fk = ginfo[k];
      }
      const uint32_t aks2 = pair_aks2(a - (fk.kso & 0xffffu));
      const uint32_t far_k = fk.far >> 16 | fk.far << 16;
      const uint32_t wave_nk = uint32_t(wave_sum_i64(int64_t(fk.n)));
      if (lane == 0) s_nk[wave] = wave_nk;
      __syncthreads();
      uint64_t nk = 0;  // members of the block's groups k
      for (int w = 0; w < kPairThreads / kWave; ++w) nk += s_nk[w];
      nk = uniform64(nk);
      for (int jb = j0; jb < j1; jb += kWave) {
        // kWave groups j, the same for every wave.  They add to a counter at most
        // their members times the block's, twice where both paths are of a code:
        // the counters are emptied before that could pass 2^32, and where these
        // could do so by themselves they go to the 8-byte ones.
        const int je = min(jb + kWave, j1);
        const uint64_t add =
            2u * nk * uniform64(uint64_t(wave_sum_i64(jb + lane < je ? int64_t(ginfo[jb + lane].n) : 0)));
        const bool big = (add >> 32) != 0;
        if (!big) {
          if ((held + add) >> 32) {
            flush_pairs(counts, lut, plus, minus);
            held = 0;
          }
          held += add;
        }
        const int stop = min(je, k0 + kWave);
        int j = jb;
        if (big) {
          for (; j < stop; ++j) big_pair(grec[j], ginfo[j], j < k, a, rk, fk, lut, plus, minus);
        } else if (k0 < int(ng)) {
          for (const int below = min(stop, k0); j + 4 <= below; j += 4)
            group_pairs<4, false>(grec, ginfo, j, rk, fk, k, aks2, far_k, lut, motif, path);
          for (; j < stop; ++j) group_pairs<1, true>(grec, ginfo, j, rk, fk, k, aks2, far_k, lut, motif, path);
        }
      }
      if (k0 >= j0 && k0 < j0 + cols && fk.n > 1u) {  // pairs within the lane's group
        const uint64_t w = uint64_t(fk.n) * (fk.n - 1u) / 2u;
        const uint32_t p = fk.kso & 0xffffu, o = fk.kso >> 16;
        const uint32_t r5 = uint32_t(__popc(rk.z)) + uint32_t(__popc(rk.w));
        const Side side = {rk.x, o, p, 0ull};
        atomicAdd(&plus[motif_of(lut, 2u * (kNumCodes - 1 - pair_code(a, p, o, side, p, r5)))], w);
        atomicAdd(&minus[motif_of(lut, path_code2(fk.base, o, p + o, p + r5))], 2u * w);
      }
    } else {
      const int64_t base = lg_ptr[i];
      const int64_t x0 = (at - npair) * sums;
      const int nj = int(min(int64_t(sums), lg_ptr[i + 1] - base - x0));
      if (held) flush_pairs(counts, lut, plus, minus);
      for (int x = wave; x < nj; x += kPairThreads / kWave) {  // less than 2^12 rows of less than 2^18
        const int32_t j = lg_col[base + x0 + x];
        const uint32_t sz = rsz[base + x0 + x];
        const uint32_t p = sz & 0xffu, b = sz >> 8;
        const uint32_t pb = path_base(a, p);
        const uint32_t* h = t.rowh + edge_ptr[j] * kHistW;
        for (uint32_t y = lane; y < b * kHistW; y += kWave) {
          const uint32_t n = h[y];
          if (n)
            atomicAdd(reinterpret_cast<uint32_t*>(path + path_code2(pb, b - p, y % kHistW + 1u, y / kHistW + 1u) * (kCopies * 2)), n);
        }
        if (lane == 0) atomicAdd(&minus[motif_of(lut, path_code2(pb, b - p, a, p))], 1ull);
      }
      flush_pairs(counts, lut, plus, plus);
      held = 0;
    }
    if (kProfile) {
      if (held) flush_pairs(counts, lut, plus, minus);
      held = 0;
      __syncthreads();
      flush(plus, minus, hist_out + (i - n0) * kHistSlots, kPairThreads);
    }
  }
  if (!kProfile) {
    flush_pairs(counts, lut, plus, minus);
    flush(plus, minus, hist_out, kPairThreads);
  }
}

// Members of N_i in a light node's list.
struct Members {
  uint4 rec[kMembers];      // y: position in row i | outside count << kPosBits
  ulonglong2 bits[kMembers];  // light nodes, less those of e_i where distinct
};
constexpr int kPosBits = 24;  // a graph has at most 200,000 hyperedges

// Pairs put off for a full wave: positions in row i and the node.
struct Pending {
  uint32_t x[2 * kWave], y[2 * kWave];
  int32_t v[2 * kWave];
};

// Block (x, q): the lists of a share of the light nodes of the graph of sample
// q's e_i.  A wave takes a node at a time, if it is outside e_i, and collects
// the members of N_i in its list (a bitmap of N_i with ranks gives the
// position in row i), kMembers at a time; the pairs of the members are spread
// over the lanes.  A pair sharing several light nodes outside e_i is taken at
// the smallest; if either of the two has only one, or their bits under one of
// two hashes show no other in common, that is it.  The others, whose nodes have to be compared, are put
// off until there is one for every lane: that costs thousands of cycles of
// dependent gathers, and among 64 pairs there nearly always is one.
//
// A row much shorter than the list of light nodes (kShortRow) is done from its
// neighbours instead, block x from a share of them: the lists of each e_j's
// light nodes outside e_i, each list as often as it has members then.
// A list of 10 with one member is the usual case there, and 70,000 rows of 30
// neighbours would each search 70,000 lists.
//
// Bound by the gathers.  100 samples on 85,353 hyperedges, 7e7 pairs: 4.6 ms;
// with one hash and e_i's own nodes among the bits, so that three pairs of four
// put off shared nothing more, 6.9; with the nodes compared on the spot 11.4.
template <bool kProfile>
__global__ __launch_bounds__(kLightThreads) void k_hs_light(
    int64_t n0, HsScratch t, const int32_t* __restrict__ row_graph, const int64_t* __restrict__ geoff,
    const int64_t* __restrict__ gnoff, const int64_t* __restrict__ edge_ptr, const int32_t* __restrict__ edge_nodes,
    const int64_t* __restrict__ node_ptr, const int32_t* __restrict__ node_edges,
    const int8_t* __restrict__ heavy_bit, const int64_t* __restrict__ lg_ptr, const int32_t* __restrict__ lg_col,
    const uint4* __restrict__ rec, const uint16_t* __restrict__ code_to_id3, unsigned long long* hist_out) {
  extern __shared__ uint32_t sm[];
  __shared__ uint16_t lut[kNumCodes];
  __shared__ unsigned long long plus[kHistSlots], minus[kHistSlots];
  __shared__ Members members[kLightWaves];
  __shared__ Pending pending[kLightWaves];
  __shared__ int32_t part[kLightThreads];
  __shared__ int32_t ei[MOCHY_MAX_EDGE];
  __shared__ ulonglong2 ei_bits[MOCHY_MAX_EDGE];  // 0 for heavy nodes
  __shared__ uint32_t s_node;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t i = t.sample_i[blockIdx.y];
  const int gi = row_graph[i];
  const int64_t e0 = geoff[gi];
  const int nw = int((geoff[gi + 1] - e0 + 31) / 32);
  const int32_t* nodes = t.lnodes + gnoff[gi];
  const int64_t nlight = t.nlight[gi];
  const int64_t ib = lg_ptr[i];
  const int di = int(lg_ptr[i + 1] - ib);
  const bool by_node = int64_t(di) * kShortRow >= nlight;
  const int64_t share = by_node ? nlight : int64_t(di);
  // the block's share, every gridDim.x-th: the longest lists are often next to each other
  const int step = int(gridDim.x), mine = int((share - blockIdx.x + step - 1) / step);
  if (mine <= 0 || di < 2) return;  // whole block
  const int64_t es = edge_ptr[i];
  const uint32_t a = uint32_t(edge_ptr[i + 1] - es);
  uint32_t* bm = sm;
  uint32_t* rank = sm + nw;
  load_classes(code_to_id3, lut, 8u, kLightThreads);
  for (int x = tid; x < kHistSlots; x += kLightThreads) plus[x] = minus[x] = 0ull;
  for (int w = tid; w < nw; w += kLightThreads) bm[w] = 0u;
  if (tid < int(a)) {
    ei[tid] = edge_nodes[es + tid];
    ei_bits[tid] = heavy_bit[ei[tid]] < 0 ? light_bits(ei[tid]) : make_ulonglong2(0ull, 0ull);
  }
  if (tid == 0) s_node = 0u;
  __syncthreads();
  for (int p = tid; p < di; p += kLightThreads) {
    const int64_t x = lg_col[ib + p] - e0;
    atomicOr(&bm[x >> 5], 1u << (x & 31));
  }
  __syncthreads();
  {  // ranks: set bits before each kRankWords words
    const int nr = (nw + kRankWords - 1) / kRankWords;
    const int per = (nr + kLightThreads - 1) / kLightThreads;
    const int r0 = min(nr, tid * per), r1 = min(nr, r0 + per);
    int32_t c = 0;
    for (int w = r0 * kRankWords; w < min(nw, r1 * kRankWords); ++w) c += __popc(bm[w]);
    part[tid] = c;
    __syncthreads();
    for (int off = 1; off < kLightThreads; off <<= 1) {
      const int32_t add = tid >= off ? part[tid - off] : 0;
      __syncthreads();
      part[tid] += add;
      __syncthreads();
    }
    int32_t run = part[tid] - c;
    for (int r = r0; r < r1; ++r) {
      rank[r] = uint32_t(run);
      for (int w = r * kRankWords; w < min(nw, (r + 1) * kRankWords); ++w) run += __popc(bm[w]);
    }
  }
  __syncthreads();
  // position in row i of neighbour x, the bit `bit` of its word
  auto position = [&](int64_t x, uint32_t word, uint32_t bit) {
    const int w = int(x >> 5), r = w / kRankWords;
    uint32_t n = rank[r] + uint32_t(__popc(word & (bit - 1u)));
#pragma unroll
    for (int y = 0; y < kRankWords - 1; ++y)
      if (r * kRankWords + y < w) n += uint32_t(__popc(bm[r * kRankWords + y]));
    return n;
  };
  const int32_t own = lane < int(a) ? ei[lane] : -1;
  // row i's record at pos as a member's; its light nodes outside e_i
  auto member = [&](uint32_t pos) {
    const uint4 r = rec[ib + pos];
    return make_uint4(r.x, pos | (r.y & 0xffu) << kPosBits, r.z, r.w);
  };
  // hyperedge x's light nodes as bits, those of e_i (mask m) taken out of a word
  // without shared bits
  auto outside_bits = [&](int64_t x, uint32_t m) {
    ulonglong2 b = t.lbits[x], out = make_ulonglong2(0ull, 0ull);
    for (; m; m &= m - 1u) {
      const ulonglong2 e = ei_bits[__ffs(m) - 1];
      out.x |= e.x;
      out.y |= e.y;
    }
    if (b.x & kDistinct) b.x &= ~out.x;
    if (b.y & kDistinct) b.y &= ~out.y;
    return b;
  };
  auto nlights = [](const uint4& r) { return (r.y >> kPosBits) - uint32_t(__popc(r.z)) - uint32_t(__popc(r.w)); };
  auto entry = [&](int64_t p, int64_t p1) { return p + lane < p1 ? int64_t(node_edges[p + lane]) - e0 : int64_t(-1); };
  // fills m from list position p on (first: the entries there); p is moved past
  // what was looked at
  auto fill = [&](Members& m, int64_t& p, int64_t p1, int64_t first) {
    int n = 0;
    while (p < p1 && n < kMembers) {
      const int64_t x = first != kNoEntries ? first : entry(p, p1);
      first = kNoEntries;
      const uint32_t word = x >= 0 ? bm[x >> 5] : 0u, bit = 1u << (x & 31);
      const bool in = (word & bit) != 0u;
      const unsigned long long all = __ballot(in);
      const int before = int(__popcll(all & ((1ull << lane) - 1ull)));
      const bool fits = in && n + before < kMembers;
      if (fits) {
        const uint32_t pos = position(x, word, bit);
        const uint4 r = member(pos);
        m.rec[n + before] = r;
        m.bits[n + before] = outside_bits(e0 + x, r.x);
      }
      const int found = int(__popcll(all));
      if (n + found > kMembers) {  // stop before the first that does not fit
        const unsigned long long over = __ballot(in && !fits);
        p += __ffsll((long long)over) - 1;
        n = kMembers;
      } else {
        p += kWave;
        n += found;
      }
    }
    p = min(p, p1);
    wave_sync();
    return n;
  };
  // moves a pair that shares `shared` light nodes outside e_i to its true overlap
  auto move = [&](const uint4& x, const uint4& y, uint32_t shared) {
    const uint32_t p = uint32_t(__popc(x.x)), ox = x.y >> kPosBits, ks = uint32_t(__popc(y.x)), oy = y.y >> kPosBits;
    const uint32_t tt = uint32_t(__popc(x.x & y.x));
    const uint32_t r5 = uint32_t(__popc(x.z & y.z)) + uint32_t(__popc(x.w & y.w));
    const Side side = {y.x, oy, ks, 0ull};
    const uint32_t bx = path_base(a, p), by = path_base(a, ks), q = tt + r5;
    atomicAdd(hist_at(minus, lut[kNumCodes - 1 - pair_code(a, p, ox, side, tt, r5)]), 1ull);
    atomicAdd(hist_at(plus, lut[kNumCodes - 1 - pair_code(a, p, ox, side, tt, r5 + shared)]), 1ull);
    if (q) {
      atomicAdd(hist_at(plus, lut_at(lut, path_code2(bx, ox, ks + oy, q))), 1ull);
      atomicAdd(hist_at(plus, lut_at(lut, path_code2(by, oy, p + ox, q))), 1ull);
    }
    atomicAdd(hist_at(minus, lut_at(lut, path_code2(bx, ox, ks + oy, q + shared))), 1ull);
    atomicAdd(hist_at(minus, lut_at(lut, path_code2(by, oy, p + ox, q + shared))), 1ull);
  };
  Pending& pend = pending[wave];
  int npend = 0;  // uniform
  auto settle = [&](int z) {  // the z-th pair put off
    const uint32_t px = pend.x[z], py = pend.y[z];
    const int32_t v = pend.v[z];
    int64_t x = lg_col[ib + px], y = lg_col[ib + py];
    int64_t xs = edge_ptr[x], ys = edge_ptr[y];
    int nx = int(edge_ptr[x + 1] - xs), ny = int(edge_ptr[y + 1] - ys);
    if (nx > ny) {  // the smaller one's nodes in the larger
      const int64_t z0 = x, z1 = xs;
      const int z2 = nx;
      x = y; xs = ys; nx = ny;
      y = z0; ys = z1; ny = z2;
    }
    const ulonglong2 by = t.lbits[y];
    uint32_t shared = 1;
    for (int r = 0; r < nx; r += 4) {
      int32_t u[4];
#pragma unroll
      for (int z = 0; z < 4; ++z) u[z] = edge_nodes[xs + min(r + z, nx - 1)];
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        const ulonglong2 b = light_bits(u[z]);
        if (r + z >= nx || u[z] == v || !(by.x & b.x) || !(by.y & b.y)) continue;
        if (in_sorted(ei, int(a), u[z]) || !in_sorted(edge_nodes + ys, ny, u[z]) || heavy_bit[u[z]] >= 0) continue;
        if (u[z] < v) return;  // the pair is u's
        ++shared;
      }
    }
    move(member(px), member(py), shared);
  };
  auto settle_all = [&]() {
    wave_sync();
    if (lane < npend) settle(lane);
    wave_sync();
    npend = 0;
  };
  // a pair of the lane (if any) sharing v; called by the whole wave
  auto pair = [&](bool any, const uint4& x, const ulonglong2& bx, const uint4& y, const ulonglong2& by, int32_t v,
                  const ulonglong2& bv) {
    const bool alone = nlights(x) <= 1u || nlights(y) <= 1u ||
                       (((bx.x | by.x) & kDistinct) && !(bx.x & by.x & ~(bv.x | kDistinct))) ||
                       (((bx.y | by.y) & kDistinct) && !(bx.y & by.y & ~(bv.y | kDistinct)));
    const bool later = any && !alone;
    const unsigned long long put = __ballot(later);
    if (put) {
      const int at = npend + int(__popcll(put & ((1ull << lane) - 1ull)));
      if (later) {
        pend.x[at] = x.y & ((1u << kPosBits) - 1u);
        pend.y[at] = y.y & ((1u << kPosBits) - 1u);
        pend.v[at] = v;
      }
      npend += int(__popcll(put));
    }
    if (any && alone) move(x, y, 1u);
    if (npend >= kWave) {  // the first 64, and the rest to their place
      wave_sync();
      settle(lane);
      wave_sync();
      const int rest = npend - kWave;
      if (lane < rest) {
        pend.x[lane] = pend.x[kWave + lane];
        pend.y[lane] = pend.y[kWave + lane];
        pend.v[lane] = pend.v[kWave + lane];
      }
      wave_sync();
      npend = rest;
    }
  };
  Members& ma = members[wave];
  // the pairs of N_i in v's list
  auto by_list = [&](int32_t v, int64_t p, int64_t p1, int64_t first) {
    const ulonglong2 bv = light_bits(v);
    while (p < p1) {
      const int n = fill(ma, p, p1, first);
      first = kNoEntries;
      if (n == 0) break;
      // each pair of the n members once: x and the d-th after it, d <= n / 2
      const int npairs = n * (n - 1) / 2;
      const float inv = 1.0f / float(n);
      for (int z0 = 0; z0 < npairs; z0 += kWave) {
        const int z = min(z0 + lane, npairs - 1);
        const int d = int((float(z) + 0.5f) * inv);
        const int x = z - d * n;
        int y = x + d + 1;
        if (y >= n) y -= n;
        pair(z0 + lane < npairs, ma.rec[x], ma.bits[x], ma.rec[y], ma.bits[y], v, bv);
      }
      if (p < p1) {  // and with each member further on, one at a time against the lanes' own
        const uint4 x = ma.rec[min(lane, n - 1)];
        const ulonglong2 bx = ma.bits[min(lane, n - 1)];
        for (int64_t r = p; r < p1; r += kWave) {
          const int64_t e = entry(r, p1);
          const uint32_t word = e >= 0 ? bm[e >> 5] : 0u, bit = 1u << (e & 31);
          const bool in = (word & bit) != 0u;
          uint4 m = make_uint4(0, 0, 0, 0);
          ulonglong2 b = make_ulonglong2(0ull, 0ull);
          if (in) {
            m = member(position(e, word, bit));
            b = outside_bits(e0 + e, m.x);
          }
          auto word_of = [](unsigned long long x, int src) {
            return (unsigned long long)(uint32_t(__builtin_amdgcn_readlane(uint32_t(x), src))) |
                   (unsigned long long)(uint32_t(__builtin_amdgcn_readlane(uint32_t(x >> 32), src))) << 32;
          };
          for (unsigned long long todo = __ballot(in); todo; todo &= todo - 1) {
            const int src = __ffsll((long long)todo) - 1;
            const uint4 y = make_uint4(__builtin_amdgcn_readlane(m.x, src), __builtin_amdgcn_readlane(m.y, src),
                                       __builtin_amdgcn_readlane(m.z, src), __builtin_amdgcn_readlane(m.w, src));
            const ulonglong2 by = make_ulonglong2(word_of(b.x, src), word_of(b.y, src));
            pair(lane < n, x, bx, y, by, v, bv);
          }
        }
      }
      wave_sync();
    }
  };
  for (;;) {
    uint32_t got = 0;
    if (lane == 0) got = atomicAdd(&s_node, uint32_t(kNodePull));
    const int vb = uniform(int(got));
    if (vb >= mine) break;
    const int nv = min(kNodePull, mine - vb);
    if (!by_node) {
      for (int y = int(blockIdx.x) + vb * step, z = 0; z < nv; ++z, y += step) {
        const uint4 rj = member(uint32_t(y));
        if (nlights(rj) == 0u) continue;
        const int64_t j = lg_col[ib + y], js = edge_ptr[j];
        const ulonglong2 bj = outside_bits(j, rj.x);
        int32_t u = -1;
        int64_t l0 = 0, l1 = 0;
        if (lane < int(edge_ptr[j + 1] - js)) {
          u = edge_nodes[js + lane];
          l0 = node_ptr[u];
          l1 = node_ptr[u + 1];
          if (l1 - l0 < 2 || heavy_bit[u] >= 0 || in_sorted(ei, int(a), u)) u = -1;
        }
        for (unsigned long long todo = __ballot(u >= 0); todo; todo &= todo - 1) {
          const int src = __ffsll((long long)todo) - 1;
          const int32_t v = __shfl(u, src);
          const ulonglong2 bv = light_bits(v);
          const int64_t p1 = __shfl(l1, src);
          for (int64_t p0 = __shfl(l0, src); p0 < p1; p0 += kWave) {
            const int64_t x = p0 + lane < p1 ? int64_t(node_edges[p0 + lane]) - e0 : -1;
            const uint32_t word = x >= 0 ? bm[x >> 5] : 0u, bit = 1u << (x & 31);
            const bool any = (word & bit) && x > j - e0;
            if (!__ballot(any)) continue;
            uint4 rk = make_uint4(0, 0, 0, 0);
            ulonglong2 bk = make_ulonglong2(0ull, 0ull);
            if (any) {
              rk = member(position(x, word, bit));
              bk = outside_bits(e0 + x, rk.x);
            }
            pair(any, rj, bj, rk, bk, v, bv);
          }
        }
      }
      continue;
    }
    int32_t node = -1;
    int64_t l0 = 0, l1 = 0;
    if (lane < nv) {
      node = nodes[int64_t(blockIdx.x) + int64_t(vb + lane) * step];
      l0 = node_ptr[node];
      l1 = node_ptr[node + 1];
    }
    int64_t first[kNodePull];  // the lists' first entries, loaded together
#pragma unroll
    for (int src = 0; src < kNodePull; ++src) first[src] = entry(__shfl(l0, src), __shfl(l1, src));
#pragma unroll
    for (int src = 0; src < kNodePull; ++src) {
      const int32_t v = __builtin_amdgcn_readlane(node, src);
      if (v < 0 || __ballot(own == v)) continue;  // a node of e_i
      int64_t p = int64_t(uniform64(uint64_t(__shfl(l0, src))));
      const int64_t p1 = int64_t(uniform64(uint64_t(__shfl(l1, src))));
      by_list(v, p, p1, first[src]);
    }
  }
  settle_all();
  __syncthreads();
  flush(plus, minus, hist_out + (kProfile ? (i - n0) * kHistSlots : 0), kLightThreads);
}

// 26 h-motif counts of each profile row from its 431 3h-motif counts.
__global__ void k_fold_rows(int64_t n, const int64_t* __restrict__ prof, const int32_t* __restrict__ parent,
                            int64_t* out26) {
  const int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (x >= n * MOCHY_NUM_H) return;
  const int64_t row = x / MOCHY_NUM_H;
  const int h = int(x % MOCHY_NUM_H);
  int64_t sum = 0;
  for (int id3 = 1; id3 < kHistSlots; ++id3)
    if (parent[id3] == h + 1) sum += prof[row * kHistSlots + id3];
  out26[x] = sum;
}

// Counts of s samples from n0 on (kProfile: of the hyperedges n0 .. n0 + s - 1,
// a row of out each), added to out.
template <bool kProfile>
mochy_status edges_device(mochy_ctx* ctx, const mochy_graph* g, int64_t n0, int64_t s, uint64_t seed,
                          unsigned long long* out) {
  if (g->max_deg == 0) return MOCHY_OK;  // no neighbours, no instances
  hipStream_t st = ctx->stream;
  char* blob = nullptr;
  auto done = [&](mochy_status rc) {
    device_free(ctx, blob);
    return rc;
  };
  // samples to a batch: as many as kBatchBytes holds, fewer where that much
  // memory is not to be had
  HsScratch t{};
  t.rows = (std::max<int64_t>(g->max_deg, 1) + 3) / 4 * 4;
  t.slots = table_slots(g->max_deg);
  const int64_t nnz = std::max<int64_t>(g->nnz, 1);
  const size_t fixed = size_t(g->E) * 17 + size_t(nnz) * (kHistW + 1) * 4 + size_t(g->ng) * 4 + 256;
  const size_t per = size_t(t.slots) * sizeof(uint2) + size_t(t.rows) * (4 + sizeof(uint4) + sizeof(GroupInfo)) + 32;
  int64_t batch = std::min(std::min(s, kMaxBatch), std::max<int64_t>(int64_t(kBatchBytes / per), 1));
  if (g->max_deg <= kScanDegree || (ctx->test_faults & 1)) batch = 0;
  while (batch && device_alloc(ctx, (void**)&blob, fixed + size_t(batch) * per) != MOCHY_OK) {
    ctx->err.clear();
    batch /= 2;
  }
  ctx->routes |= batch ? MOCHY_ROUTE_EDGE_GROUPS : MOCHY_ROUTE_EDGE_SCAN;
  if (batch == 0) return scan_edges_device(ctx, g, n0, s, seed, kProfile, out);
  char* at = blob;
  auto take = [&](auto*& p, size_t bytes) {
    p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(at);
    at += (bytes + 15) / 16 * 16;
  };
  take(t.table, size_t(batch) * t.slots * sizeof(uint2));
  take(t.grec, size_t(batch) * t.rows * sizeof(uint4));
  take(t.ginfo, size_t(batch) * t.rows * sizeof(GroupInfo));
  take(t.gslot, size_t(batch) * t.rows * 4);
  take(t.sample_i, size_t(batch) * 8);
  take(t.item_off, size_t(batch + 2) * 8);
  take(t.ngroups, size_t(batch) * 4);
  take(t.need, size_t(g->E));
  take(t.rowh, size_t(nnz) * kHistW * 4);
  take(t.lnodes, size_t(nnz) * 4);
  take(t.nlight, size_t(g->ng) * 4);
  take(t.lbits, size_t(g->E) * sizeof(ulonglong2));
  unsigned long long* queue = (unsigned long long*)(ctx->d_small + 496);
  const int64_t words = std::max<int64_t>((g->max_graph_edges + 31) / 32, 1);
  const size_t dyn = size_t(words + (words + kRankWords - 1) / kRankWords) * 4;
  const mochy_status rc = allow_lds(ctx, (const void*)k_hs_light<kProfile>, dyn);
  if (rc != MOCHY_OK) return done(rc);
  for (int64_t q0 = 0; q0 < s; q0 += batch) {
    const int64_t n = std::min(batch, s - q0);
    const bool first = q0 == 0;
    k_hs_begin<kProfile><<<unsigned(first ? std::max<int64_t>(n, std::min<int64_t>(blocks(g->E, kHsThreads), ctx->num_cus * 4)) : n),
                           kHsThreads, 0, st>>>(n0 + q0, n, seed, g->E, g->lg_ptr, t, first, g->ng,
                                                           g->edge_ptr, g->edge_nodes, g->heavy_bit);
    k_hs_group<<<dim3(blocks(g->max_deg, kGroupChunk), unsigned(n)), kHsThreads, 0, st>>>(g->lg_ptr, g->lg_col, g->rec, t);
    k_hs_items<<<unsigned(1 + n * kInfoParts) + (first ? blocks(g->V, kNodeBlock) : 0u), kItemThreads, 0, st>>>(
        n, g->lg_ptr, g->edge_ptr, t, g->V, g->ng, g->gvoff, g->gnoff, g->node_ptr, g->heavy_bit, queue);
    k_hs_rows<<<blocks(g->E, kHsWaves), kHsThreads, 0, st>>>(g->E, g->edge_ptr, g->lg_ptr, g->rsz, t);
    // two blocks to a CU (their counters fill its LDS), or one for each work item there can be
    const int64_t items = n * (pair_items(uint32_t(g->max_deg), 0) + (g->max_deg + kSumChunk - 1) / kSumChunk);
    k_hs_pairs<kProfile><<<unsigned(std::min<int64_t>(ctx->num_cus * 2, items)), kPairThreads, 0, st>>>(
        n0, n, t, t.grec, t.ginfo, g->edge_ptr, g->lg_ptr, g->lg_col, g->rsz, ctx->d_code_to_id3, queue, out);
    const unsigned parts = unsigned((int64_t(ctx->num_cus) * kLightBlocksPerCu + n - 1) / n);
    k_hs_light<kProfile><<<dim3(parts, unsigned(n)), kLightThreads, dyn, st>>>(
        n0, t, g->row_graph, g->geoff, g->gnoff, g->edge_ptr, g->edge_nodes, g->node_ptr, g->node_edges, g->heavy_bit,
        g->lg_ptr, g->lg_col, g->rec, ctx->d_code_to_id3, out);
  }
  MOCHY_HIP_OR(hipGetLastError(), done);
  return done(MOCHY_OK);
}

}  // namespace

mochy_status sampled_edges_device(mochy_ctx* ctx, const mochy_graph* g, int64_t s, uint64_t seed,
                                  int64_t n0, int64_t* d_hist) {
  MOCHY_HIP(hipMemsetAsync(d_hist, 0, kHistSlots * 8, ctx->stream));
  if (g->E == 0 || s == 0) return MOCHY_OK;
  phase_begin(ctx, kPhSample);
  const mochy_status rc = edges_device<false>(ctx, g, n0, s, seed, (unsigned long long*)d_hist);
  phase_end(ctx, kPhSample);
  return rc;
}

mochy_status profiles_device(mochy_ctx* ctx, const mochy_graph* g, int64_t c0, int64_t c1,
                             int64_t* d_prof, int64_t* d_prof26) {
  hipStream_t st = ctx->stream;
  const int64_t n = c1 - c0;
  if (n <= 0) return MOCHY_OK;
  MOCHY_HIP(hipMemsetAsync(d_prof, 0, size_t(n) * kHistSlots * 8, st));
  phase_begin(ctx, kPhSample);
  const mochy_status rc = edges_device<true>(ctx, g, c0, n, 0ull, (unsigned long long*)d_prof);
  if (rc != MOCHY_OK) return rc;
  k_fold_rows<<<unsigned((n * MOCHY_NUM_H + 255) / 256), 256, 0, st>>>(n, d_prof, ctx->d_id3_to_id26, d_prof26);
  phase_end(ctx, kPhSample);
  MOCHY_HIP(hipGetLastError());
  return MOCHY_OK;
}
