// Exact fix-up of the pairs the pair kernel classified with an incomplete R5.
//
// The pair kernel takes R5 = |e_j ∩ e_k - e_i| from exact bits for the 64
// highest-degree ("heavy") nodes only.  It is exact for every pair of
// neighbours of e_i unless e_j and e_k also share a lower-degree ("light")
// node outside e_i.  Whether two hyperedges share a light node does not
// depend on the centre, and few pairs do (sum over light nodes w of
// C(|E_w|, 2)), so the fix-up works pair by pair:
//
//  1. light pairs: for every light node w, every pair {e_j, e_k} of E_w whose
//     smallest shared light node is w (each pair once).  The pair is owned by
//     the endpoint with the longer line-graph row.
//  2. for every light pair, the centres are N_j ∩ N_k: one workgroup per
//     owner j holds row j as an LDS bitmap (with per-word ranks, so a hit gives
//     the position of e_i in row j) and scans the partner's row.  With masks
//     over the nodes of e_k (m_kj: e_k ∩ e_j, and its heavy and light parts
//     H, L, formed once per pair from the two node lists) and, for a centre
//     e_i, m_ki (e_k ∩ e_i) from the record of row k at the scanned position:
//        t   = popcount(m_ki & m_kj)                 = |e_i ∩ e_j ∩ e_k|
//        r5h = popcount(H & ~m_ki)                   heavy part of R5
//        ls  = popcount(L & ~m_ki)                   light part of R5
//     and |e_j ∩ e_i|, |e_i| from the size word of row j at e_i's position
//     (the only read outside the scanned row).  Where memory allows, a byte
//     table of the overlaps |e_j ∩ e_i| takes the place of the bitmap
//     (k_light_dense, the usual path).
//     If ls = 0 the pair kernel was exact at this centre.  Otherwise the pair
//     kernel recorded the class with R5 = r5h, counted iff both neighbours
//     are above e_i or the two looked disjoint; the exact class has
//     R5 = r5h + ls and, since e_j and e_k meet, is counted iff both are
//     above e_i (Algorithm 2's condition).  The first is removed, the second
//     added.
#include <algorithm>

#include "classify.h"
#include "common.h"
#include "pairs.h"

namespace {

// Is w the smallest light node shared by e_x and e_y?  (Both contain w.)
__device__ __forceinline__ bool smallest_shared_light(int32_t x, int32_t y, int32_t w,
                                                      const int64_t* __restrict__ edge_ptr,
                                                      const int32_t* __restrict__ edge_nodes,
                                                      const int8_t* __restrict__ heavy_bit) {
  int64_t p = edge_ptr[x], q = edge_ptr[y];
  const int64_t pe = edge_ptr[x + 1], qe = edge_ptr[y + 1];
  while (p < pe && q < qe) {
    const int32_t u = edge_nodes[p], v = edge_nodes[q];
    if (u >= w || v >= w) {
      if (u < v) ++p;
      else if (u > v) ++q;
      else return true;  // reached w (u == v >= w means u == w: first shared light is w)
      continue;
    }
    if (u < v) ++p;
    else if (u > v) ++q;
    else {
      if (heavy_bit[u] < 0) return false;
      ++p; ++q;
    }
  }
  return true;
}

// One wave per light node w: every pair of E_w whose smallest shared light
// node is w.  kCount counts pairs per owner; kFill also writes the partners
// (a second pass, after the owners' offsets are known).  Where the flat list
// of candidate slots fits, k_light_slots runs the merges once instead.
enum LightMode { kCount = 0, kFill = 1 };
template <int kMode>
__global__ __launch_bounds__(256) void k_light_pairs(
    int64_t V, const int64_t* __restrict__ node_ptr, const int32_t* __restrict__ node_edges,
    const int8_t* __restrict__ heavy_bit, const int64_t* __restrict__ edge_ptr,
    const int32_t* __restrict__ edge_nodes, const int64_t* __restrict__ lg_ptr,
    unsigned long long* pcount, const int64_t* __restrict__ poff, int32_t* partners) {
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
  if (w >= V || heavy_bit[w] >= 0) return;  // uniform per wave
  const int64_t lo = node_ptr[w];
  const int D = int(node_ptr[w + 1] - lo);
  for (int kc = 0; kc < D; kc += 64) {
    const int b = kc + lane;
    const int32_t yb = b < D ? node_edges[lo + b] : 0;
    const int64_t db = b < D ? lg_ptr[yb + 1] - lg_ptr[yb] : 0;
    const int aend = min(kc + 64, D) - 1;
    for (int a = 0; a < aend; ++a) {
      const int32_t ya = node_edges[lo + a];
      if (!(b < D && a < b)) continue;
      if (!smallest_shared_light(ya, yb, int32_t(w), edge_ptr, edge_nodes, heavy_bit)) continue;
      const int64_t da = lg_ptr[ya + 1] - lg_ptr[ya];
      const bool a_owns = da > db || (da == db && ya < yb);
      const int32_t owner = a_owns ? ya : yb, partner = a_owns ? yb : ya;
      const unsigned long long slot = atomicAdd(&pcount[owner], 1ull);
      if (kMode == kFill) partners[poff[owner] + int64_t(slot)] = partner;
    }
  }
}

// The hyperedges of every light node, longest line-graph row first (ties: the
// smaller id): of two of them the earlier owns the pair.  One thread per
// incidence, which takes the place that its rank among the node's gives.
// work: what the pairs would have scanned, row entries in [0] and in [1] their
// share of a row of the overlap table, in kShareUnit-ths.
constexpr unsigned long long kShareUnit = 32768;
__global__ __launch_bounds__(256) void k_sort_members(int64_t nnz, int64_t V, const int64_t* __restrict__ node_ptr,
                                                      const int32_t* __restrict__ node_edges,
                                                      const int8_t* __restrict__ heavy_bit,
                                                      const int64_t* __restrict__ lg_ptr,
                                                      const int32_t* __restrict__ row_graph,
                                                      const int64_t* __restrict__ geoff, int32_t* sorted,
                                                      unsigned long long* work) {
  __shared__ unsigned long long s_work[2];
  if (threadIdx.x < 2) s_work[threadIdx.x] = 0ull;
  __syncthreads();
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  unsigned long long entries = 0, share = 0;
  if (t < nnz) {
    int64_t lo = 0, hi = V;  // node_ptr[lo] <= t < node_ptr[lo + 1]
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (node_ptr[mid] <= t) lo = mid; else hi = mid;
    }
    if (heavy_bit[lo] < 0) {
      const int32_t y = node_edges[t];
      const int64_t d = lg_ptr[y + 1] - lg_ptr[y], q0 = node_ptr[lo], q1 = node_ptr[lo + 1];
      int rank = 0;
      for (int64_t q = q0; q < q1; ++q) {
        const int32_t x = node_edges[q];
        const int64_t dx = lg_ptr[x + 1] - lg_ptr[x];
        rank += dx > d || (dx == d && x < y) ? 1 : 0;
      }
      sorted[q0 + rank] = y;
      const int g = row_graph[y];
      entries = (unsigned long long)rank * (unsigned long long)d;
      share = entries * kShareUnit / (unsigned long long)(geoff[g + 1] - geoff[g]);
    }
  }
  for (int off = kWave / 2; off > 0; off >>= 1) {
    entries += __shfl_xor(entries, off, kWave);
    share += __shfl_xor(share, off, kWave);
  }
  if (threadIdx.x % kWave == 0) {
    atomicAdd(&s_work[0], entries);
    atomicAdd(&s_work[1], share);
  }
  __syncthreads();
  if (threadIdx.x < 2 && s_work[threadIdx.x]) atomicAdd(&work[threadIdx.x], s_work[threadIdx.x]);
}

// The flat list of candidate pairs, in units of kOwners slots: a light node w's
// hyperedges y_0, y_1, ... (as sorted above), owners a in [kOwners c, kOwners
// (c + 1)) and partner b > kOwners c, partners of one chunk c of owners in
// turn.  A slot holds (owner, partner), or (-1, -1) where a >= b or w is not
// the pair's smallest shared light node.
constexpr int kOwners = 4;
// Units before chunk c of a node of D hyperedges; the node's units.
__host__ __device__ __forceinline__ int64_t unit_offset(int64_t c, int64_t D) {
  return c * (D - 1) - kOwners * (c * (c - 1) / 2);
}
__host__ __device__ __forceinline__ int64_t node_units(int64_t D) {
  return D < 2 ? 0 : unit_offset((D - 1 + kOwners - 1) / kOwners, D);
}

// One thread per slot t: the light node w with noff[w] <= t < noff[w + 1] (a
// binary search), then the chunk and partner of its unit, merged as in
// k_light_pairs.  A node's merges are spread over as many threads, where the
// one-wave-per-node kernel leaves the largest light node's wave running long
// after the others.
__global__ __launch_bounds__(256) void k_light_slots(
    int64_t V, int64_t ncand, const int64_t* __restrict__ node_ptr, const int32_t* __restrict__ sorted,
    const int8_t* __restrict__ heavy_bit, const int64_t* __restrict__ edge_ptr,
    const int32_t* __restrict__ edge_nodes, unsigned long long* pcount, const int64_t* __restrict__ noff,
    int2* flat) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= ncand) return;
  int64_t lo = 0, hi = V;  // largest w with noff[w] <= t (noff is nondecreasing, noff[V] = ncand > t)
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (noff[mid] <= t) lo = mid; else hi = mid;
  }
  const int64_t w = lo, base = node_ptr[w], D = node_ptr[w + 1] - base;
  const int64_t u = (t - noff[w]) / kOwners;
  int64_t c0 = 0, c1 = (D - 1 + kOwners - 1) / kOwners;  // unit_offset(c0) <= u < unit_offset(c1)
  while (c1 - c0 > 1) {
    const int64_t mid = (c0 + c1) >> 1;
    if (unit_offset(mid, D) <= u) c0 = mid; else c1 = mid;
  }
  const int64_t b = u - unit_offset(c0, D) + kOwners * c0 + 1;
  const int64_t a = kOwners * c0 + (t - noff[w]) % kOwners;
  int2 v = make_int2(-1, -1);
  if (a < b) {
    const int32_t ya = sorted[base + a], yb = sorted[base + b];
    if (smallest_shared_light(ya, yb, int32_t(w), edge_ptr, edge_nodes, heavy_bit)) {
      v = make_int2(ya, yb);
      if (pcount) atomicAdd(&pcount[ya], 1ull);
    }
  }
  flat[t] = v;
}

// Slots of every light node's units (0 for heavy ones), the input of the flat
// list's offsets; cnt[V] = 0.  Clears k_sort_members' work.
__global__ void k_pair_slots(int64_t V, const int64_t* __restrict__ node_ptr,
                             const int8_t* __restrict__ heavy_bit, int64_t* cnt, unsigned long long* work) {
  const int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (w < 2) work[w] = 0ull;
  if (w > V) return;
  cnt[w] = w < V && heavy_bit[w] < 0 ? kOwners * node_units(node_ptr[w + 1] - node_ptr[w]) : 0;
}

// The flat list's pairs into each owner's partner range (cursor[] from zero).
__global__ void k_scatter_pairs(int64_t n, const int2* __restrict__ flat, const int64_t* __restrict__ eoff,
                                unsigned long long* cursor, int32_t* partners) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) {
    const int2 v = flat[t];
    if (v.x < 0) continue;
    const unsigned long long s = atomicAdd(&cursor[v.x], 1ull);
    partners[eoff[v.x] + int64_t(s)] = v.y;
  }
}

// First position of an ascending row whose id is v or more, by the whole wave:
// 64 probes a step, so three dependent loads where a row has up to 2^18 ids.
__device__ __forceinline__ int row_lower(const int32_t* __restrict__ row, int n, int64_t v, int lane) {
  int lo = 0;
  while (n > 0) {  // the answer is in [lo, lo + n]
    const int step = (n + kWave - 1) / kWave;
    const int at = lane * step;
    const int below = __popcll(__ballot(at < n && row[lo + at] < v));  // probes are ascending
    if (below == 0) break;
    lo += (below - 1) * step + 1;
    n = min(step - 1, n - ((below - 1) * step + 1));
  }
  return lo;
}

// The part [r_lo, r_hi) of row k that can need a fix: centres of [c0, c1) and,
// where e_j and e_k share a heavy node, those below both.  A centre not below
// both has its pair counted only if the two looked disjoint, and with a heavy
// node v shared they never do (v is in the triple overlap, or outside e_i with
// a bit of its own).  Rows are ascending, so both cut the row's ends; two
// thirds of the entries of medium's partner rows belong to such pairs.
// [e0, e1): the graph's hyperedges.
__device__ __forceinline__ void fix_range(const int32_t* __restrict__ row, int d, const int32_t* __restrict__ up_first,
                                          int32_t j, int32_t k, uint32_t Hk, int64_t c0, int64_t c1, int64_t e0,
                                          int64_t e1, int lane, int& r_lo, int& r_hi) {
  r_lo = c0 > e0 ? row_lower(row, d, c0, lane) : 0;
  r_hi = d;
  if (Hk != 0u) {
    const int32_t m = min(j, k);
    if (m >= c1) r_hi = row_lower(row, d, c1, lane);
    else r_hi = m == k ? up_first[k] : row_lower(row, d, m, lane);
  } else if (c1 < e1) {
    r_hi = row_lower(row, d, c1, lane);
  }
}

// Workgroups are dealt to the 8 XCDs in turn; block b takes the owner that
// gives each XCD a contiguous range of the owner list (a bijection onto
// [0, nb)), so that owners listed together share one XCD's L2.
constexpr unsigned kXcds = 8;
__device__ __forceinline__ int64_t xcd_block(unsigned b, unsigned nb) {
  const unsigned x = b % kXcds, k = b / kXcds, per = nb / kXcds, extra = nb % kXcds;
  return int64_t(x) * per + (x < extra ? x : extra) + k;
}

// One block per work item, an item being up to kFixChunk partners of one
// owner (an owner's items are consecutive, so they run at the same time on
// one XCD and share the owner's row in its L2); 512 threads, so that the LDS
// the row bitmap takes still leaves room for 24 resident waves per CU (the
// scan waits on loads).  128 partners per item build an owner's bitmap half
// as often as 64 (on medium 121 ms against 125; 256 no better).
constexpr int kFixThreads = 512;
constexpr size_t kFlatBytes = size_t(4) << 30;  // largest flat list of candidate light pairs
constexpr int kFixCopies = 2;
constexpr int kFixChunk = 128;

// At most 64 registers (8 waves per SIMD, room for 4 blocks, 32 waves per CU,
// when the LDS allows; the scan waits on loads, so resident waves count more
// than entries per lane).
__global__ __launch_bounds__(kFixThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_light_fix(
    int64_t c0, int64_t c1, const int32_t* __restrict__ row_graph, const int64_t* __restrict__ geoff,
    const int32_t* __restrict__ owners, const int32_t* __restrict__ item_owner,
    const int64_t* __restrict__ ioff, const int64_t* __restrict__ poff,
    const int32_t* __restrict__ partners,
    const int64_t* __restrict__ edge_ptr, const int32_t* __restrict__ edge_nodes,
    const int8_t* __restrict__ heavy_bit, const int64_t* __restrict__ lg_ptr,
    const int32_t* __restrict__ lg_col, const int32_t* __restrict__ up_first, const uint32_t* __restrict__ recm,
    const uint16_t* __restrict__ rsz, const uint16_t* __restrict__ code_to_id3,
    unsigned long long* hist_out, unsigned long long* tally) {
  extern __shared__ uint32_t sm[];
  __shared__ uint16_t lut[kNumCodes];
  // kFixCopies histogram copies, lane l adding to copy l % kFixCopies (fewer
  // same-word adds in one instruction); 2 keep a block within 40 KB of LDS on
  // graphs of up to 85k hyperedges, so that 4 blocks reside per CU
  __shared__ unsigned long long hist[kFixCopies * kHistSlots];
  __shared__ int32_t part[kFixThreads];
  __shared__ int32_t ej[MOCHY_MAX_EDGE];  // e_j's nodes (ascending)
  __shared__ unsigned long long s_tally[3];  // entries scanned, centres examined, centres reclassified
  const int64_t it = xcd_block(blockIdx.x, gridDim.x);
  const int64_t ob = item_owner[it];
  const int32_t j = owners[ob];
  const int64_t p0 = poff[ob] + (it - ioff[ob]) * kFixChunk;  // this item's partners
  const int64_t p1 = min(poff[ob + 1], p0 + kFixChunk);
  const int gj = row_graph[j];
  const int64_t e0 = geoff[gj];  // row j's graph owns hyperedges [e0, geoff[gj + 1])
  const int64_t e1 = geoff[gj + 1];
  const int nwE = int((e1 - e0 + 31) / 32);
  uint32_t* bm = sm;          // row j over the graph's hyperedge ids
  uint32_t* rank = sm + nwE;  // set bits before each word
  const int64_t jb = lg_ptr[j];
  const int dj = int(lg_ptr[j + 1] - jb);
  for (int t = threadIdx.x; t < kNumCodes; t += blockDim.x) lut[t] = code_to_id3[t];
  for (int t = threadIdx.x; t < kFixCopies * kHistSlots; t += blockDim.x) hist[t] = 0;
  for (int w = threadIdx.x; w < nwE; w += blockDim.x) bm[w] = 0;
  const uint32_t sizej = uint32_t(edge_ptr[j + 1] - edge_ptr[j]);
  if (threadIdx.x < sizej) ej[threadIdx.x] = edge_nodes[edge_ptr[j] + threadIdx.x];
  if (threadIdx.x < 3) s_tally[threadIdx.x] = 0ull;
  __syncthreads();
  for (int p = threadIdx.x; p < dj; p += blockDim.x) {
    const int64_t x = lg_col[jb + p] - e0;
    atomicOr(&bm[x >> 5], 1u << (x & 31));
  }
  __syncthreads();
  {
    const int chunk = (nwE + kFixThreads - 1) / kFixThreads;
    const int w0 = min(nwE, int(threadIdx.x) * chunk), w1 = min(nwE, w0 + chunk);
    int32_t c = 0;
    for (int w = w0; w < w1; ++w) c += __popc(bm[w]);
    part[threadIdx.x] = c;
    __syncthreads();
    for (int off = 1; off < kFixThreads; off <<= 1) {
      const int32_t add = threadIdx.x >= unsigned(off) ? part[threadIdx.x - off] : 0;
      __syncthreads();
      part[threadIdx.x] += add;
      __syncthreads();
    }
    int32_t run = part[threadIdx.x] - c;
    for (int w = w0; w < w1; ++w) {
      rank[w] = uint32_t(run);
      run += __popc(bm[w]);
    }
  }
  __syncthreads();
  // one partner per wave at a time (rows shorter than a block's sweep leave
  // no lanes idle)
  const int lane = int(threadIdx.x) & (kWave - 1), wave = int(threadIdx.x) / kWave;
  unsigned long long* myhist = hist + (lane & (kFixCopies - 1)) * kHistSlots;
  uint32_t n_scanned = 0, n_centres = 0, n_changed = 0;  // this wave's, for mochy_exact_stats
  for (int64_t pp = p0 + wave; pp < p1; pp += kFixThreads / kWave) {
    const int32_t k = partners[pp];
    // masks over e_k's nodes: e_j ∩ e_k (mkj), its heavy and light nodes
    const int64_t kn0 = edge_ptr[k];
    const uint32_t sizek = uint32_t(edge_ptr[k + 1] - kn0);
    bool in_j = false, heavy = false;
    if (uint32_t(lane) < sizek) {
      const int32_t v = edge_nodes[kn0 + lane];
      in_j = in_sorted(ej, int(sizej), v);
      heavy = heavy_bit[v] >= 0;
    }
    const uint32_t mkj = uint32_t(__ballot(in_j));
    const uint32_t Hk = mkj & uint32_t(__ballot(heavy)), Lk = mkj & ~Hk;
    const int64_t kb = lg_ptr[k];
    int r_lo, dk;
    fix_range(lg_col + kb, int(lg_ptr[k + 1] - kb), up_first, j, k, Hk, c0, c1, e0, e1, lane, r_lo, dk);
    n_scanned += uint32_t(max(dk - r_lo, 0));
    // row k scanned kUnroll entries per thread at a time; the loads of one
    // stage are issued together, with no branch between them (an entry that
    // is not a centre reads a valid dummy slot), since the work is bound by
    // load latency: 3 of 4 scanned entries are centres on hub-heavy graphs
    // (7 entries per lane fit the 64 registers; 8 spill and were slower)
    constexpr int kUnroll = 7;
    constexpr int step = kWave;
    for (int r0 = r_lo + lane; r0 < dk; r0 += kUnroll * step) {
      int32_t iv[kUnroll];
      uint32_t mki[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int r = r0 + u * step;
        iv[u] = r < dk ? lg_col[kb + r] : -1;
        mki[u] = recm[kb + min(r, dk - 1)];  // e_k ∩ e_i over e_k's nodes
      }
      int qj[kUnroll];
      bool hit[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int32_t i = iv[u];
        const bool in = i >= 0;  // not past the scanned part's end
        const int64_t il = in ? i - e0 : 0;
        const uint32_t iw = bm[il >> 5];
        const uint32_t ibit = 1u << (il & 31);
        hit[u] = in && (iw & ibit) != 0u;  // a neighbour of e_j (i == j never is)
        qj[u] = hit[u] ? int(rank[il >> 5] + __popc(iw & (ibit - 1u))) : 0;
      }
      uint32_t szj[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) szj[u] = rsz[jb + qj[u]];  // |e_j ∩ e_i| | |e_i| << 8
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        // wave-uniform tallies (a ballot counts the lanes still scanning)
        n_centres += uint32_t(__popcll(__ballot(hit[u])));
        const uint32_t ls = __popc(Lk & ~mki[u]);
        const bool fix = hit[u] && ls != 0u;  // otherwise the pair kernel was exact at this centre
        n_changed += uint32_t(__popcll(__ballot(fix)));
        if (!fix) continue;
        const int32_t i = iv[u];
        const uint32_t wik = __popc(mki[u]);
        const uint32_t t = __popc(mki[u] & mkj);
        const uint32_t r5h = __popc(Hk & ~mki[u]);
        const uint32_t pj = szj[u] & 0xffu;
        const uint32_t a = szj[u] >> 8;
        Side K;
        K.m = 0u; K.s = wik; K.o = sizek - wik; K.h = 0ull;
        const uint32_t oj = sizej - pj;
        const bool above = (j > i) && (k > i);
        if (above || (t | r5h) == 0u) atomicAdd(&myhist[lut[pair_code(a, pj, oj, K, t, r5h)]], ~0ull);
        if (above) atomicAdd(&myhist[lut[pair_code(a, pj, oj, K, t, r5h + ls)]], 1ull);
      }
    }
  }
  if (lane == 0 && n_scanned != 0u) {
    atomicAdd(&s_tally[0], (unsigned long long)n_scanned);
    atomicAdd(&s_tally[1], (unsigned long long)n_centres);
    atomicAdd(&s_tally[2], (unsigned long long)n_changed);
  }
  __syncthreads();
  if (threadIdx.x < 3) tally[it * 3 + threadIdx.x] = s_tally[threadIdx.x];  // summed by k_fix_tally
  for (int t = threadIdx.x; t < kHistSlots; t += blockDim.x) {
    unsigned long long v = 0;
    for (int c = 0; c < kFixCopies; ++c) v += hist[c * kHistSlots + t];
    if (v) atomicAdd(&hist_out[int64_t(gj) * kHistSlots + t], v);
  }
}

// ---------------------------------------------------------------------------
// The same from a table of overlaps, W[j][i] = |e_j ∩ e_i| as a byte (0: not
// neighbours): it answers at once whether a scanned entry is a centre and what
// the owner's overlap with it is, with no bitmap of the owner's row to build.
// So the pairs need no grouping by owner: the flat list is taken as it stands.
// A wave takes a unit of it (up to kOwners owners with one partner) and
// scans the partner's row once for all of them.  Columns of W are the centres
// of the range.
constexpr int kDenseThreads = 512;
// Where the rows of W are long (kLongStride bytes), the waves of an XCD pull
// kDensePull units at a time from a queue of its own, so that they are at few
// owners together and those rows stay in its L2 (with 128 units per block the
// blocks of an XCD are at 200 owners, 78 % of the reads miss and medium takes
// 77 ms instead of 53).  Where they are short, a block takes kBlockUnits of a
// queue and deals them out in LDS: a unit is then little work, and a global
// atomic for each would cost as much (65 graphs of 6k hyperedges: 4 ms, 10 with
// an atomic per unit).
constexpr int kLongStride = 32768;
constexpr int kDensePull = 2;
constexpr uint32_t kBlockUnits = 64;
constexpr int64_t kXcdUnits = 65536;  // by waves, a graph of as many units has a queue per XCD
constexpr int kDenseCopies = 4;
// entries of a wave between flushes (8 waves share a counter); few of them for
// tests of the flush
constexpr uint32_t kDenseFlush = 1u << 24, kDenseFlushTest = 256;
constexpr int kOverlapChunk = 32768;  // bytes of a row formed in LDS at a time

// The table takes a write of all its bytes and, for each entry scanned, a read
// in a row that other pairs may have left in the caches; owner by owner the same
// answer is a bit in LDS, after a sort of the pairs by owner and with a row of
// bits to build for each.  Tables of up to kSmallTable a graph, and kSmallTables
// in all, always pay.  Larger ones do where the scanned rows fill a kDenseRow-th of the table's or more and hold
// as many entries as the table bytes.  Correction in ms, table and owner by owner
// (the scanned rows' share; the table):
//   10,000 hyperedges, flat   (0.004, 0.1 GB)  0.20  0.34
//   20,000, exponent 0.8      (0.014, 0.4 GB)  0.86  1.01
//   9 of 20,000, exponent 0.3 (0.002, 3.6 GB)  2.6   3.1
//   33 of 6,000, exponent 0.8 (0.02, 1.2 GB)   2.4   3.8
//   17,636, exponent 1        (0.09, 0.3 GB)   1.22  1.70
//   30,000, exponent 0.9      (0.09, 0.7 GB)   8.3   12.1
//   50,000, exponent 0.9      (0.04, 2.2 GB)   14.3  17.0
//   85,311, exponent 1        (0.08, 7.3 GB)   56.6  84.7
//   30,000, exponent 0.5      (0.006, 0.9 GB)  3.7   2.2
//   50,000, exponent 0.8      (0.013, 2.4 GB)  8.9   6.1
//   100,000, exponent 0.7     (0.002, 10 GB)   12.3  4.7
//   100,000, flat             (0.003, 10 GB)   37.7  11.9
// Sets of more than kFewGraphs graphs of fewer than kGraphSlots candidate slots
// each (the kernel on the tables goes from graph to graph) have none:
//   9 of 300 hyperedges (1,100 slots)     0.09  0.15
//   33 of 500 (2,480)                     0.25  0.22
//   1,000 of 200 (530)                    2.3   0.92
//   3,000 of 100 (78)                     5.9   0.78
//   100 of 1,000 (6,110)                  0.66  0.85
//   1,000 of 1,000 (6,100)                6.2   7.8
// A range of up to half the centres always has its table where the rows are short
// ones (below kLongStride): owner by owner every pair is still to be listed and
// every owner's row to be built, whatever the range (table, owner by owner):
//   100,000 of 200,000 nodes, a 10th      (1 GB)    0.57  0.76
//   the same, a quarter                   (2.5 GB)  0.79  0.79
//   100,000 of 5,000 nodes, a quarter     (2.5 GB)  10.6  14.2
//   190,000 of 100,000 nodes, a 10th      (3.6 GB)  2.1   6.0
//   the same, a quarter: long rows        (9 GB)    8.4   6.0
constexpr size_t kSmallTable = size_t(512) << 20, kSmallTables = size_t(8) << 30;
constexpr int kFewGraphs = 16;
constexpr int64_t kGraphSlots = 4096;
constexpr unsigned long long kDenseRow = 32;

// Per graph: where its rows of W start, their stride (a multiple of 16) and the
// first centre; one block, a run of graphs to each thread.
struct OverlapTable {
  int64_t off;
  int32_t first, width, stride;
};
__device__ __forceinline__ OverlapTable overlap_of(int64_t e0, int64_t e1, int64_t c0, int64_t c1) {
  OverlapTable t;
  t.off = 0;
  const int64_t lo = min(max(e0, c0), e1), hi = max(min(e1, c1), lo);
  t.first = int32_t(lo);
  t.width = int32_t(hi - lo);
  t.stride = (t.width + 15) & ~15;
  return t;
}
constexpr int kOffsetThreads = 256;
__global__ __launch_bounds__(kOffsetThreads) void k_overlap_offsets(int ng, const int64_t* __restrict__ geoff,
                                                                    int64_t c0, int64_t c1, OverlapTable* tab) {
  __shared__ int64_t part[kOffsetThreads];
  const int tid = int(threadIdx.x), per = (ng + kOffsetThreads - 1) / kOffsetThreads;
  const int g0 = min(ng, tid * per), g1 = min(ng, g0 + per);
  int64_t sum = 0;
  for (int g = g0; g < g1; ++g)
    sum += (geoff[g + 1] - geoff[g]) * overlap_of(geoff[g], geoff[g + 1], c0, c1).stride;
  part[tid] = sum;
  __syncthreads();
  if (g0 >= g1) return;
  int64_t at = 0;  // of the threads before
  for (int x = 0; x < tid; ++x) at += part[x];
  for (int g = g0; g < g1; ++g) {
    OverlapTable t = overlap_of(geoff[g], geoff[g + 1], c0, c1);
    t.off = at;
    at += (geoff[g + 1] - geoff[g]) * t.stride;
    tab[g] = t;
  }
}

// One block per row: the row's bytes, kOverlapChunk at a time, from LDS.
__global__ __launch_bounds__(256) void k_overlap_rows(const int32_t* __restrict__ row_graph,
                                                      const int64_t* __restrict__ geoff,
                                                      const OverlapTable* __restrict__ tab,
                                                      const int64_t* __restrict__ lg_ptr,
                                                      const int32_t* __restrict__ lg_col,
                                                      const uint16_t* __restrict__ rsz, uint8_t* W) {
  __shared__ uint4 buf[kOverlapChunk / 16];
  uint8_t* bytes = reinterpret_cast<uint8_t*>(buf);
  const int64_t i = blockIdx.x;
  const int g = row_graph[i];
  const OverlapTable t = tab[g];
  uint8_t* out = W + t.off + (i - geoff[g]) * t.stride;
  const int64_t base = lg_ptr[i];
  const int d = int(lg_ptr[i + 1] - base);
  const int lane = int(threadIdx.x) & (kWave - 1);
  for (int x0 = 0; x0 < t.stride; x0 += kOverlapChunk) {
    const int n16 = min(t.stride - x0, kOverlapChunk) / 16;
    for (int x = threadIdx.x; x < n16; x += blockDim.x) buf[x] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const int p0 = row_lower(lg_col + base, d, int64_t(t.first) + x0, lane);
    const int p1 = row_lower(lg_col + base, d, int64_t(t.first) + min(x0 + kOverlapChunk, t.width), lane);
    for (int p = p0 + int(threadIdx.x); p < p1; p += blockDim.x)
      bytes[lg_col[base + p] - t.first - x0] = uint8_t(rsz[base + p] & 0xffu);
    __syncthreads();
    for (int x = threadIdx.x; x < n16; x += blockDim.x) reinterpret_cast<uint4*>(out + x0)[x] = buf[x];
    __syncthreads();
  }
}

// 6 waves per SIMD: 80 registers hold the owners' masks (at 8 waves some spill,
// 57 ms on medium against 53), and two entries per lane in flight for each of
// four owners.  What bounds it then is vector issue: 50 instructions per 64
// entries and owner, 1.3e9 such (3.4e10 entries of 4.4e6 units on medium).
__global__ __launch_bounds__(kDenseThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_light_dense(
    int64_t c0, int64_t c1, int ng, uint32_t* queues, const int64_t* __restrict__ noff, const int2* __restrict__ flat,
    const int64_t* __restrict__ geoff, const int64_t* __restrict__ gvoff, const OverlapTable* __restrict__ tab,
    const uint8_t* __restrict__ W, const int64_t* __restrict__ edge_ptr, const int32_t* __restrict__ edge_nodes,
    const int8_t* __restrict__ heavy_bit, const int64_t* __restrict__ lg_ptr, const int32_t* __restrict__ lg_col,
    const int32_t* __restrict__ up_first, const uint32_t* __restrict__ recm, const uint16_t* __restrict__ rsz,
    const uint16_t* __restrict__ code_to_id3, unsigned long long* hist_out, unsigned long long* tally,
    uint32_t flush) {
  __shared__ uint16_t lut[kNumCodes];              // by reversed code: word of the id in a histogram copy
  __shared__ int32_t hist[kDenseCopies * kGStride];
  __shared__ unsigned long long s_tally[3];        // entries scanned, centres examined, centres reclassified
  __shared__ uint32_t s_taken[2], s_base, s_next;
  for (int t = threadIdx.x; t < kNumCodes; t += blockDim.x) lut[t] = uint16_t(code_to_id3[kNumCodes - 1 - t] * 4u);
  for (int t = threadIdx.x; t < kDenseCopies * kGStride; t += blockDim.x) hist[t] = 0;
  if (threadIdx.x < 3) s_tally[threadIdx.x] = 0ull;
  const int lane = int(threadIdx.x) & (kWave - 1);
  char* myhist = reinterpret_cast<char*>(hist + (lane & (kDenseCopies - 1)) * kGStride);
  unsigned long long n_scanned = 0, n_centres = 0, n_changed = 0;  // this wave's, for mochy_exact_stats
  uint32_t unflushed = 0;  // entries this wave scanned since it last emptied the histogram
  const int first = int(int64_t(blockIdx.x) * ng / gridDim.x);
  for (int v = 0; v < ng; ++v) {  // every graph, each block from a share of its own
    const int g = first + v < ng ? first + v : first + v - ng;
    const int64_t slot0 = noff[gvoff[g]];
    const uint32_t units = uint32_t((noff[gvoff[g + 1]] - slot0) / kOwners);
    const OverlapTable t = tab[g];
    const bool by_wave = t.stride >= kLongStride;
    const uint32_t nq = by_wave && units >= kXcdUnits ? kXcds : 1u, per = (units + nq - 1u) / nq;
    const uint32_t bunits =
        uint32_t(min(max(int64_t(units) * ng / (gridDim.x * 2), int64_t(kDenseThreads / kWave)), int64_t(kBlockUnits)));
    uint32_t* queue = queues + size_t(g) * kXcds;
    if (threadIdx.x == 0)
      s_taken[v & 1] = nq > 1u ? 0u : __hip_atomic_load(queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (uint32_t(uniform(int(s_taken[v & 1]))) >= units) continue;
    const int64_t e0 = geoff[g], e1 = geoff[g + 1];
    uint32_t turn = 0, at = 0, stop = 0;  // by wave: queues tried; units in hand
    uint32_t base = 0, end = 0;           // by block: units in hand
    for (;;) {
      if (by_wave) {
        if (at == stop) {
          const uint32_t x = (blockIdx.x + turn) % nq;
          int got = 0;
          if (lane == 0) got = int(atomicAdd(&queue[x], uint32_t(kDensePull)));
          at = uint32_t(uniform(got));
          const uint32_t last = min(per, units - min(units, x * per));  // units of this queue
          if (at >= last) {
            stop = at;
            if (++turn == nq) break;
            continue;
          }
          stop = min(at + uint32_t(kDensePull), last) + x * per;
          at += x * per;
        }
      } else {
        int got = 0;
        if (base < end && lane == 0) got = int(atomicAdd(&s_next, 1u));
        at = base + uint32_t(uniform(got));
        if (at >= end) {  // every wave of the block comes here once per share
          __syncthreads();
          if (threadIdx.x == 0) {
            s_base = atomicAdd(queue, bunits);
            s_next = 0u;
          }
          __syncthreads();
          base = uint32_t(uniform(int(s_base)));
          end = min(base + bunits, units);
          if (base >= units) break;
          continue;
        }
      }
      if (unflushed >= flush) {  // keeps the 32-bit counters of the block far from their ends
        for (int q = lane; q < kDenseCopies * kGStride; q += kWave) {
          const int32_t n = atomicExch(&hist[q], 0);
          if (n) atomicAdd(&hist_out[int64_t(g) * kHistSlots + q % kGStride], (unsigned long long)int64_t(n));
        }
        n_scanned += unflushed;
        unflushed = 0;
      }
      const int64_t slot = slot0 + int64_t(at++) * kOwners;
      // The unit's owners side by side, 16 lanes each (the work before the scan
      // is a chain of dependent loads, so it is done once for all of them).
      const int part = lane & 48, sub = lane & 15;
      const int2 pr = flat[slot + (lane >> 4)];
      const unsigned long long valid = __ballot(pr.x >= 0);
      if (valid == 0ull) continue;
      const int32_t k = __builtin_amdgcn_readlane(pr.y, __builtin_ctzll(valid));
      const int32_t j = pr.x >= 0 ? pr.x : k;
      const int64_t kn0 = edge_ptr[k], kb = lg_ptr[k], jn0 = edge_ptr[j];
      const uint32_t sizek = uint32_t(edge_ptr[k + 1] - kn0), sizej = uint32_t(edge_ptr[j + 1] - jn0);
      const int d = int(lg_ptr[k + 1] - kb);
      const int32_t vk = uint32_t(lane) < sizek ? edge_nodes[kn0 + lane] : -1;
      const int32_t vj0 = uint32_t(sub) < sizej ? edge_nodes[jn0 + sub] : -2;
      const int32_t vj1 = uint32_t(sub) + 16u < sizej ? edge_nodes[jn0 + sub + 16] : -2;
      const uint32_t heavy = uint32_t(__ballot(vk >= 0 && heavy_bit[max(vk, 0)] >= 0));
      // masks over e_k's nodes: e_j ∩ e_k (mkj), its heavy and light nodes
      uint32_t mkj = 0;
      for (uint32_t q = 0; q < sizek; ++q) {
        const int32_t node = __builtin_amdgcn_readlane(vk, int(q));
        const unsigned long long eq = __ballot(vj0 == node || vj1 == node);
        mkj |= ((eq >> part) & 0xffffull) != 0ull ? 1u << q : 0u;
      }
      if (pr.x < 0) mkj = 0u;
      const uint32_t Hk = mkj & heavy, Lk = mkj & ~heavy;
      // The part of row k to scan: centres of [c0, c1) and, where e_j and e_k
      // share a heavy node, those below both (see fix_range); 16 probes a step
      const int32_t* row = lg_col + kb;
      const int64_t i1 = Hk != 0u ? min(c1, int64_t(min(j, k))) : c1;
      const int r_lo = c0 > e0 ? row_lower(row, d, c0, lane) : 0;
      int hi = r_lo;
      for (int n = i1 < e1 && pr.x >= 0 ? d - r_lo : 0; __ballot(n > 0) != 0ull;) {
        const int step = (n + 15) / 16;
        const int x = sub * step;
        const unsigned long long less = __ballot(x < n && row[hi + x] < i1);
        const int below = __popcll((less >> part) & 0xffffull);
        n = below == 0 ? 0 : min(step - 1, n - ((below - 1) * step + 1));
        if (below) hi += (below - 1) * step + 1;
      }
      if (i1 >= e1) hi = d;
      if (pr.x < 0) hi = 0;
      // per owner: the masks in vector registers (as scalars they are spilled)
      const uint32_t wofs = uint32_t((j - e0) * (t.stride / 16));  // the owner's row of W, in 16 bytes
      uint32_t mkj_o[kOwners], Hk_o[kOwners], Lk_o[kOwners];
      uint32_t sizej_o[kOwners], wj[kOwners];
      int32_t below_o[kOwners];
      int hi_o[kOwners], r_hi = 0;
#pragma unroll
      for (int o = 0; o < kOwners; ++o) {
        mkj_o[o] = uint32_t(__builtin_amdgcn_readlane(int(mkj), 16 * o));
        Hk_o[o] = uint32_t(__builtin_amdgcn_readlane(int(Hk), 16 * o));
        Lk_o[o] = uint32_t(__builtin_amdgcn_readlane(int(Lk), 16 * o));
        asm volatile("" : "+v"(mkj_o[o]), "+v"(Hk_o[o]), "+v"(Lk_o[o]));
        sizej_o[o] = uint32_t(__builtin_amdgcn_readlane(int(sizej), 16 * o));
        wj[o] = uint32_t(__builtin_amdgcn_readlane(int(wofs), 16 * o));
        below_o[o] = __builtin_amdgcn_readlane(min(j, k), 16 * o);
        hi_o[o] = __builtin_amdgcn_readlane(hi, 16 * o);
        r_hi = max(r_hi, hi_o[o]);
        unflushed += uint32_t(max(hi_o[o] - r_lo, 0));
      }
      const uint8_t* wg = W + t.off - t.first;
      // kUnroll entries of row k per lane at a time, the loads of one stage
      // issued together, with no branch between them
      constexpr int kUnroll = 2;
      for (int r0 = r_lo + lane; r0 < r_hi; r0 += kUnroll * kWave) {
        int32_t iv[kUnroll];
        uint32_t mki[kUnroll], sz[kUnroll], pj[kOwners][kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          const int r = min(r0 + u * kWave, r_hi - 1);
          iv[u] = lg_col[kb + r];
          mki[u] = recm[kb + r];  // e_k ∩ e_i over e_k's nodes
          sz[u] = rsz[kb + r];    // |e_k ∩ e_i| | |e_i| << 8
        }
#pragma unroll
        for (int o = 0; o < kOwners; ++o)
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) pj[o][u] = wg[int64_t(wj[o]) * 16 + iv[u]];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          const int r = r0 + u * kWave;
          const uint32_t wik = sz[u] & 0xffu, a = sz[u] >> 8;
          const uint32_t aks2 = 2u * (a - wik) - 4u;
          const uint32_t kso = wik | ((sizek - wik) << 16);
#pragma unroll
          for (int o = 0; o < kOwners; ++o) {
            const uint32_t p = pj[o][u];
            const bool hit = p != 0u && r < hi_o[o];  // a neighbour of e_j (i == j never is)
            n_centres += uint32_t(__popcll(__ballot(hit)));
            const uint32_t ls = uint32_t(__popc(Lk_o[o] & ~mki[u]));
            const bool fix = hit && ls != 0u;  // otherwise the pair kernel was exact at this centre
            n_changed += uint32_t(__popcll(__ballot(fix)));
            if (!fix) continue;
            const uint32_t t2 = uint32_t(__popc(mki[u] & mkj_o[o])) + 2u;
            const uint32_t r5h2 = uint32_t(__popc(Hk_o[o] & ~mki[u])) + 2u;
            const uint32_t jy = p | ((2u * p + 4u) << 8) | ((sizej_o[o] - p) << 16);
            const uint32_t tr = t2 | (r5h2 << 16);
            const bool above = iv[u] < below_o[o];
            if (above || tr == 0x00020002u)
              atomicAdd(reinterpret_cast<int32_t*>(myhist + lut_at(lut, pair_rcode2(t2, tr, aks2, jy, kso))), -1);
            if (above)
              atomicAdd(
                  reinterpret_cast<int32_t*>(myhist + lut_at(lut, pair_rcode2(t2, tr + (ls << 16), aks2, jy, kso))), 1);
          }
        }
      }
    }
    n_scanned += unflushed;
    unflushed = 0;
    __syncthreads();
    for (int q = threadIdx.x; q < kHistSlots; q += blockDim.x) {
      int64_t v = 0;
      for (int c = 0; c < kDenseCopies; ++c) {
        v += hist[c * kGStride + q];
        hist[c * kGStride + q] = 0;
      }
      if (v) atomicAdd(&hist_out[int64_t(g) * kHistSlots + q], (unsigned long long)v);
    }
    __syncthreads();
  }
  if (lane == 0 && n_scanned != 0u) {
    atomicAdd(&s_tally[0], (unsigned long long)n_scanned);
    atomicAdd(&s_tally[1], (unsigned long long)n_centres);
    atomicAdd(&s_tally[2], (unsigned long long)n_changed);
  }
  __syncthreads();
  if (threadIdx.x < 3) tally[blockIdx.x * 3 + threadIdx.x] = s_tally[threadIdx.x];  // summed by k_fix_tally
}

// Valid slots of the flat list (light pairs), for mochy_exact_stats.
__global__ __launch_bounds__(256) void k_count_pairs(int64_t n, const int2* __restrict__ flat,
                                                     unsigned long long* stats) {
  __shared__ unsigned long long red[256 / kWave];
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  unsigned long long v = 0;
  for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < n; t += stride) v += flat[t].x >= 0 ? 1u : 0u;
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    v = red[0] + red[1] + red[2] + red[3];
    if (v) atomicAdd(&stats[kStLightPairs], v);
  }
}

// The correction's work counters for mochy_exact_stats: the per-item tallies
// of the fix kernel, summed over a fixed grid with one atomic per block and
// counter (atomics on one address from every wave or item would serialize).
constexpr int kTallyBlocks = 64;
__global__ __launch_bounds__(256) void k_fix_tally(int64_t nitems, const unsigned long long* __restrict__ tally,
                                                   unsigned long long* stats) {
  __shared__ unsigned long long red[3][256 / kWave];
  unsigned long long v[3] = {0, 0, 0};
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; q < nitems; q += stride)
    for (int x = 0; x < 3; ++x) v[x] += tally[q * 3 + x];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (int x = 0; x < 3; ++x) {
    for (int off = kWave / 2; off > 0; off >>= 1) v[x] += __shfl_xor(v[x], off, kWave);
    if (lane == 0) red[x][wave] = v[x];
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    unsigned long long t = 0;
    for (int w = 0; w < 256 / kWave; ++w) t += red[threadIdx.x][w];
    const int slot = threadIdx.x == 0 ? kStFixScanned : threadIdx.x == 1 ? kStFixCentres : kStFixChanged;
    if (t) atomicAdd(&stats[slot], t);
  }
}

// owners: hyperedges with at least one light partner, compacted.
__global__ void k_owner_list(int64_t E, const unsigned long long* __restrict__ pcount,
                             unsigned long long* nown, int32_t* owners, int64_t* ocount) {
  const int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (x >= E || pcount[x] == 0) return;
  const unsigned long long s = atomicAdd(nown, 1ull);
  owners[s] = int32_t(x);
  ocount[s] = int64_t(pcount[x]);
}

__global__ void k_owner_offsets(int64_t n, const int32_t* __restrict__ owners,
                                const int64_t* __restrict__ poff, int64_t* eoff, int64_t* icount) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s < n) {
    eoff[owners[s]] = poff[s];
    icount[s] = (poff[s + 1] - poff[s] + kFixChunk - 1) / kFixChunk;
  }
  if (s == n) icount[n] = 0;
}

// item_owner[q] = the owner of work item q (items of owner s: [ioff[s], ioff[s + 1])).
__global__ void k_item_owners(int64_t n, const int64_t* __restrict__ ioff, int32_t* item_owner) {
  const int64_t s = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= n) return;
  for (int64_t q = ioff[s]; q < ioff[s + 1]; ++q) item_owner[q] = int32_t(s);
}

inline unsigned blocks(int64_t n, int t) { return unsigned((n + t - 1) / t); }

}  // namespace

mochy_status correct_device(mochy_ctx* ctx, const mochy_graph* g, int64_t c0, int64_t c1,
                            int64_t* d_hist, unsigned long long* stats) {
  hipStream_t st = ctx->stream;
  const int64_t E = g->E, V = g->V;
  if (c1 <= c0 || E == 0 || V == 0) return MOCHY_OK;
  const int nwE = int((g->max_graph_edges + 31) / 32);
  const size_t dyn = size_t(nwE) * 8;
  mochy_status rc = allow_lds(ctx, (const void*)k_light_fix, dyn);
  if (rc != MOCHY_OK) return rc;
  // pcount[E] | nown | owners[E] | ocount[E+1] | poff[E+1] | tmp
  const size_t tmpn = scan_tmp_elems(std::max(E, V) + 1);  // scans of E + 1 and V + 1 entries
  const size_t n64 = size_t(E) + 1 + size_t(E + 1) * 2 + tmpn;
  char* buf = nullptr;
  int64_t* eoff = nullptr;
  int32_t* partners = nullptr;
  int64_t* ioff = nullptr;
  int32_t* item_owner = nullptr;
  unsigned long long* tally = nullptr;
  int64_t* noff = nullptr;
  int32_t* sorted = nullptr;
  int2* flat = nullptr;
  auto done = [&](mochy_status s) {
    device_free(ctx, noff);
    device_free(ctx, sorted);
    device_free(ctx, flat);
    device_free(ctx, buf);
    device_free(ctx, eoff);
    device_free(ctx, partners);
    device_free(ctx, ioff);
    device_free(ctx, item_owner);
    device_free(ctx, tally);
    return s;
  };
  if ((rc = device_alloc(ctx, (void**)&buf, n64 * 8 + size_t(E) * 4)) != MOCHY_OK) return rc;
  unsigned long long* pcount = (unsigned long long*)buf;
  unsigned long long* nown = pcount + E;
  int64_t* ocount = (int64_t*)(nown + 1);
  int64_t* poff = ocount + (E + 1);
  int64_t* tmp = poff + (E + 1);
  int32_t* owners = (int32_t*)(buf + n64 * 8);
  launch_fill_u32(buf, 0u, (size_t(E) + 1 + size_t(E + 1)) * 8, st);
  const unsigned wblocks = blocks(V * 64, 256);
  // one pass over the candidate pairs into a flat list when it is small
  // (8 bytes per pair of a light node's hyperedges, at most kFlatBytes, not
  // carved from a caller's arena); otherwise a counting pass now and a
  // filling pass once the owners' offsets are known
  int64_t ncand = 0;
  unsigned long long* const work = (unsigned long long*)(ctx->d_small + 504);  // [2]
  if (!ctx->arena && !(ctx->test_faults & 8)) {
    if ((rc = device_alloc(ctx, (void**)&noff, size_t(V + 1) * 8)) != MOCHY_OK) return done(rc);
    k_pair_slots<<<blocks(V + 1, 256), 256, 0, st>>>(V, g->node_ptr, g->heavy_bit, noff, work);
    launch_exclusive_scan_i64(noff, noff, V + 1, tmp, st);
    MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 503, noff + V, 8, hipMemcpyDeviceToHost, st), done);
    MOCHY_HIP_OR(hipStreamSynchronize(st), done);
    ncand = ctx->h_small[503];
    if (ncand > 0 && size_t(ncand) * 8 <= kFlatBytes &&
        (device_alloc(ctx, (void**)&sorted, size_t(g->nnz) * 4) != MOCHY_OK ||
         device_alloc(ctx, (void**)&flat, size_t(ncand) * 8) != MOCHY_OK)) {
      flat = nullptr;  // no room for the list: the two passes instead
      ctx->err.clear();
    }
    if (flat)
      k_sort_members<<<blocks(g->nnz, 256), 256, 0, st>>>(g->nnz, V, g->node_ptr, g->node_edges, g->heavy_bit, g->lg_ptr,
                                                          g->row_graph, g->geoff, sorted, work);
  }
  // the overlap table: where it takes at most a sixth of the device memory (40 GB
  // for the largest graph), pays for itself and can be allocated
  uint8_t* W = nullptr;
  OverlapTable* tab = nullptr;
  const int64_t nblocks = std::min<int64_t>(int64_t(ctx->num_cus) * 4, (ncand + 4 * kOwners - 1) / (4 * kOwners));
  const size_t qbytes = size_t(g->ng) * kXcds * 4;
  if (flat) {
    size_t wbytes = 0, most = 0;
    for (int x = 0; x < g->ng; ++x) {
      const int64_t e0 = g->h_geoff[x], e1 = g->h_geoff[x + 1];
      const int64_t width = std::max<int64_t>(std::min(e1, c1) - std::max(e0, c0), 0);
      const size_t b = size_t(e1 - e0) * size_t((width + 15) & ~int64_t(15));
      wbytes += b;
      most = std::max(most, b);
    }
    bool pays = wbytes > 0 && wbytes <= size_t(ctx->total_mem / 6) && !(ctx->test_faults & 1) &&
                (g->ng <= kFewGraphs || ncand >= g->ng * kGraphSlots);
    const bool narrow = c1 - c0 < kLongStride && 2 * (c1 - c0) <= E;
    if (pays && !narrow && (most > kSmallTable || wbytes > kSmallTables)) {
      MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 504, work, 16, hipMemcpyDeviceToHost, st), done);
      MOCHY_HIP_OR(hipStreamSynchronize(st), done);
      // a range's columns of the rows are as many of their entries
      const double entries = double(ctx->h_small[504]) * double(c1 - c0) / double(E);
      pays = double(ctx->h_small[505]) * double(kDenseRow) >= double(ncand) * double(kShareUnit) &&
             entries >= double(wbytes);
    }
    if (pays && (device_alloc(ctx, (void**)&tally, size_t(nblocks) * 24 + qbytes) != MOCHY_OK ||
                 device_alloc(ctx, (void**)&tab, size_t(g->ng) * sizeof(OverlapTable)) != MOCHY_OK ||
                 device_alloc(ctx, (void**)&W, wbytes) != MOCHY_OK)) {
      device_free(ctx, tally);  // no room: owner by owner instead
      device_free(ctx, tab);
      tally = nullptr;
      tab = nullptr;
      W = nullptr;
      ctx->err.clear();
    }
    if (W) ctx->table_bytes = int64_t(wbytes);
  }
  ctx->routes |= (W ? MOCHY_ROUTE_TABLE : 0u) | (flat ? MOCHY_ROUTE_LISTED : 0u);
  if (W) {
    auto dense_done = [&](mochy_status s) {
      device_free(ctx, W);
      device_free(ctx, tab);
      return done(s);
    };
    uint32_t* const queues = (uint32_t*)(tally + nblocks * 3);
    launch_fill_u32(queues, 0u, qbytes, st);
    k_light_slots<<<blocks(ncand, 256), 256, 0, st>>>(V, ncand, g->node_ptr, sorted, g->heavy_bit, g->edge_ptr,
                                                      g->edge_nodes, nullptr, noff, flat);
    k_overlap_offsets<<<1, kOffsetThreads, 0, st>>>(g->ng, g->geoff, c0, c1, tab);
    k_overlap_rows<<<unsigned(E), 256, 0, st>>>(g->row_graph, g->geoff, tab, g->lg_ptr, g->lg_col, g->rsz, W);
    phase_begin(ctx, kPhFix);
    k_light_dense<<<unsigned(nblocks), kDenseThreads, 0, st>>>(
        c0, c1, g->ng, queues, noff, flat, g->geoff, g->gvoff, tab, W, g->edge_ptr, g->edge_nodes, g->heavy_bit,
        g->lg_ptr, g->lg_col, g->up_first, g->recm, g->rsz, ctx->d_code_to_id3, (unsigned long long*)d_hist, tally,
        (ctx->test_faults & 16) ? kDenseFlushTest : kDenseFlush);
    phase_end(ctx, kPhFix);
    k_fix_tally<<<kTallyBlocks, 256, 0, st>>>(nblocks, tally, stats);
    k_count_pairs<<<unsigned(std::min<int64_t>(blocks(ncand, 256), 256)), 256, 0, st>>>(ncand, flat, stats);
    MOCHY_HIP_OR(hipGetLastError(), dense_done);
    return dense_done(MOCHY_OK);
  }
  if (flat)
    k_light_slots<<<blocks(ncand, 256), 256, 0, st>>>(V, ncand, g->node_ptr, sorted, g->heavy_bit, g->edge_ptr,
                                                      g->edge_nodes, pcount, noff, flat);
  else
    k_light_pairs<kCount><<<wblocks, 256, 0, st>>>(V, g->node_ptr, g->node_edges, g->heavy_bit,
                                                   g->edge_ptr, g->edge_nodes, g->lg_ptr, pcount,
                                                   nullptr, nullptr);
  k_owner_list<<<blocks(E, 256), 256, 0, st>>>(E, pcount, nown, owners, ocount);
  MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 504, nown, 8, hipMemcpyDeviceToHost, st), done);
  MOCHY_HIP_OR(hipStreamSynchronize(st), done);
  const int64_t nowners = ctx->h_small[504];
  if (nowners == 0) return done(MOCHY_OK);
  ctx->routes |= MOCHY_ROUTE_OWNERS;
  launch_exclusive_scan_i64(ocount, poff, nowners + 1, tmp, st);  // ocount[nowners] is 0
  MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 505, poff + nowners, 8, hipMemcpyDeviceToHost, st), done);
  MOCHY_HIP_OR(hipStreamSynchronize(st), done);
  const int64_t npairs = ctx->h_small[505];
  ctx->exact_stats[kStLightPairs] += npairs;
  // per-owner offsets indexed by hyperedge id for the fill pass
  if ((rc = device_alloc(ctx, (void**)&eoff, size_t(E) * 8)) != MOCHY_OK) return done(rc);
  if ((rc = device_alloc(ctx, (void**)&partners, size_t(npairs) * 4)) != MOCHY_OK) return done(rc);
  if ((rc = device_alloc(ctx, (void**)&ioff, size_t(nowners + 1) * 8)) != MOCHY_OK) return done(rc);
  // scatter owner offsets to hyperedge ids and count each owner's work items
  // (ioff holds the counts, then their prefix, in place), reset counters, fill
  k_owner_offsets<<<blocks(nowners + 1, 256), 256, 0, st>>>(nowners, owners, poff, eoff, ioff);
  launch_exclusive_scan_i64(ioff, ioff, nowners + 1, tmp, st);
  MOCHY_HIP_OR(hipMemcpyAsync(ctx->h_small + 506, ioff + nowners, 8, hipMemcpyDeviceToHost, st), done);
  launch_fill_u32(pcount, 0u, size_t(E) * 8, st);
  if (flat)
    k_scatter_pairs<<<unsigned(std::min<int64_t>(blocks(ncand, 256), int64_t(ctx->num_cus) * 16)), 256, 0, st>>>(
        ncand, flat, eoff, pcount, partners);
  else
    k_light_pairs<kFill><<<wblocks, 256, 0, st>>>(V, g->node_ptr, g->node_edges, g->heavy_bit,
                                                  g->edge_ptr, g->edge_nodes, g->lg_ptr, pcount, eoff,
                                                  partners);
  MOCHY_HIP_OR(hipStreamSynchronize(st), done);
  const int64_t nitems = ctx->h_small[506];
  if ((rc = device_alloc(ctx, (void**)&item_owner, size_t(nitems) * 4)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&tally, size_t(nitems) * 24)) != MOCHY_OK)
    return done(rc);
  k_item_owners<<<blocks(nowners, 256), 256, 0, st>>>(nowners, ioff, item_owner);
  phase_begin(ctx, kPhFix);
  k_light_fix<<<unsigned(nitems), kFixThreads, dyn, st>>>(c0, c1, g->row_graph, g->geoff, owners, item_owner,
                                                          ioff, poff, partners,
                                                           g->edge_ptr, g->edge_nodes, g->heavy_bit, g->lg_ptr,
                                                           g->lg_col, g->up_first, g->recm, g->rsz, ctx->d_code_to_id3,
                                                           (unsigned long long*)d_hist, tally);
  phase_end(ctx, kPhFix);
  k_fix_tally<<<kTallyBlocks, 256, 0, st>>>(nitems, tally, stats);
  MOCHY_HIP_OR(hipGetLastError(), done);
  MOCHY_HIP_OR(hipStreamSynchronize(st), done);
  return done(MOCHY_OK);
}
