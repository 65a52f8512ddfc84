// Line-graph construction on the device (Algorithm 1, section 4.1).
//
// project_incidence (steps 1-3) is shared with the line-graph-free mode.
// Steps, all on the context stream:
//   1. validate the CSR (sorted, in range, non-empty, size <= MOCHY_MAX_EDGE);
//   2. transpose it into E_v (node -> hyperedges): count, scan, scatter;
//   3. pick the 64 highest-degree nodes ("heavy"; ties to the smaller id);
//   4. line-graph degree of every hyperedge: the row of e_i is the union of
//      E_v over v in e_i minus e_i itself, formed as a bitmap over hyperedge
//      ids in LDS (so the row comes out sorted and de-duplicated), from bitmaps
//      of the heavy nodes' lists and the other lists' hyperedges;
//   5. scan the degrees into row pointers; |wedges| = sum / 2;
//   6. fill the rows (ascending neighbour ids) from the same bitmap, with one
//      16-byte record per (centre, neighbour): which nodes of e_i the
//      neighbour holds (a 32-bit mask; omega = its popcount), how many of its
//      nodes lie outside e_i, which heavy nodes lie outside e_i, and whether a
//      non-heavy node does.  Identical hyperedges show up here (no outside
//      node, every node of e_i) and are reported.
#include "common.h"

namespace {

// Each hyperedge is checked against its own graph: incidences inside the
// graph's slice, node ids inside the graph's node range, strictly ascending.
__global__ void k_validate(int64_t E, int32_t ng, const int64_t* __restrict__ geoff,
                           const int64_t* __restrict__ gvoff, const int64_t* __restrict__ gnoff,
                           const int64_t* __restrict__ ptr, const int32_t* __restrict__ nodes,
                           int32_t* flags) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= E) return;
  int lo = 0, hi = ng;  // last graph with geoff[g] <= e
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (geoff[mid] <= e) lo = mid; else hi = mid;
  }
  const int64_t s = ptr[e], t = ptr[e + 1];
  if (s < gnoff[lo] || t > gnoff[lo + 1] || t <= s) { atomicOr(flags, kFlagInval); return; }
  if (t - s > MOCHY_MAX_EDGE) { atomicOr(flags, kFlagRange); return; }
  const int64_t v0 = gvoff[lo], v1 = gvoff[lo + 1];
  int64_t prev = v0 - 1;
  for (int64_t q = s; q < t; ++q) {
    const int64_t v = nodes[q];
    if (v < v0 || v >= v1 || v <= prev) { atomicOr(flags, kFlagInval); return; }
    prev = v;
  }
}

// Transpose: the nodes' degrees (kFill false), then E_v (kFill true), a thread
// to a hyperedge.  A node in many hyperedges is one address for as many atomics,
// some 18 ns each, so a block first adds its own up in an LDS table (a node
// whose place is another's goes to memory by itself) and takes a node's slots of
// E_v in one piece.  1.24e6 incidences, one node in 40,589 hyperedges: 0.16
// and 0.26 ms; with an atomic for each incidence 0.75 and 0.82.
constexpr int kNodeThreads = 512, kNodeTable = 2048;

template <bool kFill>
__global__ __launch_bounds__(kNodeThreads) void k_transpose(int64_t E, const int64_t* __restrict__ ptr,
                                                            const int32_t* __restrict__ nodes,
                                                            const int64_t* __restrict__ node_ptr,
                                                            unsigned long long* count, unsigned* fill,
                                                            int32_t* node_edges) {
  __shared__ int32_t tag[kNodeTable];  // node + 1, 0 = free
  __shared__ uint32_t n[kNodeTable], first[kFill ? kNodeTable : 1];
  for (int t = threadIdx.x; t < kNodeTable; t += kNodeThreads) {
    tag[t] = 0;
    n[t] = 0u;
  }
  __syncthreads();
  auto place = [](int32_t v) { return int((uint32_t(v) * 2654435761u) >> 21); };  // 11 bits
  static_assert(kNodeTable == 2048, "11-bit places");
  const int64_t e = int64_t(blockIdx.x) * kNodeThreads + threadIdx.x;
  const int64_t q0 = e < E ? ptr[e] : 0, q1 = e < E ? ptr[e + 1] : 0;
  for (int64_t q = q0; q < q1; ++q) {
    const int32_t v = nodes[q];
    const int t = place(v);
    const int32_t held = atomicCAS(&tag[t], 0, v + 1);
    if (held == 0 || held == v + 1) atomicAdd(&n[t], 1u);
    else if (!kFill) atomicAdd(&count[v], 1ull);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kNodeTable; t += kNodeThreads) {
    if (!n[t]) continue;
    if (kFill) {
      first[t] = atomicAdd(&fill[tag[t] - 1], n[t]);
      n[t] = 0u;
    } else {
      atomicAdd(&count[tag[t] - 1], (unsigned long long)n[t]);
    }
  }
  if (!kFill) return;
  __syncthreads();
  for (int64_t q = q0; q < q1; ++q) {
    const int32_t v = nodes[q];
    const int t = place(v);
    const unsigned slot = tag[t] == v + 1 ? first[t] + atomicAdd(&n[t], 1u) : atomicAdd(&fill[v], 1u);
    node_edges[node_ptr[v] + slot] = int32_t(e);
  }
}

// The 64 heavy nodes of a graph: those of largest degree, ties to the smaller
// id, degree 2 at least.  A block takes kHeavyChunk nodes of a graph, 8 to
// a thread, finds the degree T of the 64th by halving the range of degrees
// (each step a count over the block), and takes the nodes above T and the first
// of those at T.  Where a graph has more nodes than a block takes, the blocks
// put their 64 out as keys in order and the next launch takes those, until one
// block is left.
//
// Bound by the latency of the steps, some 0.4 us each.  300 nodes 8.8 us
// (64 rounds of a maximum over the block: 78), 200,003 nodes in two launches
// 25 us (3445).
constexpr int kHeavyThreads = 1024, kHeavyPer = 8;
constexpr int kHeavyChunk = kHeavyThreads * kHeavyPer;
constexpr int kHeavyWaves = kHeavyThreads / kWave;
constexpr int kHeavyGroups = kHeavyPer * kHeavyWaves;  // nodes in order of id: kHeavyPer turns of a block's waves

// node v as a key: larger keys first
__device__ __forceinline__ unsigned long long heavy_key(uint32_t deg, int64_t v) {
  return (unsigned long long)deg << 32 | (0xffffffffull - (unsigned long long)v);
}

__global__ __launch_bounds__(kHeavyThreads) void k_heavy(const int64_t* __restrict__ gvoff,
                                                         const int64_t* __restrict__ node_ptr,
                                                         const unsigned long long* __restrict__ in, int64_t nin,
                                                         unsigned parts,
                                                         unsigned long long* out, int8_t* heavy_bit) {
  __shared__ uint32_t cnt[2][kHeavyWaves];
  __shared__ uint32_t eq[kHeavyGroups];
  __shared__ unsigned long long top[kHeavyBits];
  __shared__ uint32_t s_n;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t g = blockIdx.x / parts, x0 = int64_t(blockIdx.x % parts) * kHeavyChunk;
  const int64_t v0 = gvoff[g], n = in ? nin : gvoff[g + 1] - v0;
  unsigned long long key[kHeavyPer];
  uint32_t most = 0;
#pragma unroll
  for (int r = 0; r < kHeavyPer; ++r) {
    const int64_t x = x0 + r * kHeavyThreads + tid;
    key[r] = 0ull;
    if (x >= n) continue;
    if (in) {
      key[r] = in[g * nin + x];
    } else {
      key[r] = heavy_key(uint32_t(node_ptr[v0 + x + 1] - node_ptr[v0 + x]), v0 + x);
      heavy_bit[v0 + x] = -1;
    }
    most = max(most, uint32_t(key[r] >> 32));
  }
  if (tid == 0) s_n = 0u;
  if (tid < kHeavyBits) top[tid] = 0ull;
  for (int off = 32; off > 0; off >>= 1) most = max(most, uint32_t(__shfl_xor(int(most), off)));
  if (lane == 0) cnt[0][wave] = most;
  __syncthreads();
  for (int w = 0; w < kHeavyWaves; ++w) most = max(most, cnt[0][w]);
  // T: the largest degree that 64 nodes reach, 2 if there is none
  uint32_t T = 2u, hi = most + 1u;  // 64 reach T (or T = 2), fewer reach hi
  for (int turn = 1; T + 1u < hi; turn ^= 1) {
    const uint32_t mid = T + (hi - T) / 2u;
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < kHeavyPer; ++r) c += uint32_t(__popcll(__ballot(uint32_t(key[r] >> 32) >= mid)));
    if (lane == 0) cnt[turn][wave] = c;
    __syncthreads();
    c = 0;
    for (int w = 0; w < kHeavyWaves; ++w) c += cnt[turn][w];
    if (c >= uint32_t(kHeavyBits)) T = mid; else hi = mid;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kHeavyPer; ++r) {
    const uint32_t d = uint32_t(key[r] >> 32);
    if (d > T) top[atomicAdd(&s_n, 1u)] = key[r];
    const unsigned long long at = __ballot(d == T);
    if (lane == 0) eq[r * kHeavyWaves + wave] = uint32_t(__popcll(at));
  }
  __syncthreads();
  const uint32_t above = s_n;
  uint32_t before = 0;  // of those at T, the ones before this wave's r-th group
  for (int y = 0; y < wave; ++y) before += eq[y];
#pragma unroll
  for (int r = 0; r < kHeavyPer; ++r) {
    const unsigned long long at = __ballot(uint32_t(key[r] >> 32) == T);
    const uint32_t slot = above + before + uint32_t(__popcll(at & ((1ull << lane) - 1ull)));
    if (((at >> lane) & 1ull) && slot < uint32_t(kHeavyBits)) top[slot] = key[r];
    if (r + 1 < kHeavyPer)
      for (int y = 0; y < kHeavyWaves; ++y) before += eq[r * kHeavyWaves + wave + y];
  }
  __syncthreads();
  if (tid < kHeavyBits) {  // their order
    const unsigned long long k = top[tid];
    int rank = 0;
    for (int y = 0; y < kHeavyBits; ++y) rank += top[y] > k || (top[y] == k && y < tid) ? 1 : 0;
    if (out) out[int64_t(blockIdx.x) * kHeavyBits + rank] = k;
    else if (k) heavy_bit[0xffffffffull - (k & 0xffffffffull)] = int8_t(rank);
  }
}

// What a row's records need of each hyperedge: its heavy nodes as a mask (bit
// heavy_bit[v]) and its size; and the heavy nodes' lists as bitmaps over all
// hyperedges (heavy index b of its own graph: row b), one wave turning 64 masks
// over at a time.
struct EdgeInfo {
  unsigned long long heavy;
  uint32_t size, pad;
};

__host__ __device__ constexpr int64_t heavy_words(int64_t E) { return (E + 63) / 64 + 1; }  // 64-bit, one to spare

__global__ __launch_bounds__(256) void k_edge_heavy(int64_t E, const int64_t* __restrict__ ptr,
                                                    const int32_t* __restrict__ nodes,
                                                    const int8_t* __restrict__ heavy_bit, EdgeInfo* info,
                                                    unsigned long long* rows) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t nw = heavy_words(E), w = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
  if (w >= nw) return;  // whole wave
  const int64_t x = w * 64 + lane;
  unsigned long long h = 0;
  if (x < E) {
    const int64_t s = ptr[x], e = ptr[x + 1];
    for (int64_t q = s; q < e; ++q) {
      const int b = heavy_bit[nodes[q]];
      if (b >= 0) h |= 1ull << b;
    }
    info[x] = EdgeInfo{h, uint32_t(e - s), 0u};
  }
  unsigned long long mine = 0;
  for (int b = 0; b < kHeavyBits; ++b) {
    const unsigned long long row = __ballot((h >> b) & 1ull);
    if (lane == b) mine = row;
  }
  rows[lane * nw + w] = mine;
}

// The nodes of e_i by how their lists enter the row's bitmap: as the heavy
// node's bitmap, or hyperedge by hyperedge.
struct RowNodes {
  int32_t ei[MOCHY_MAX_EDGE];
  int8_t hbit[MOCHY_MAX_EDGE], hpos[MOCHY_MAX_EDGE];  // heavy nodes: heavy index, position in e_i
  int8_t dense[MOCHY_MAX_EDGE];                       // heavy index of each list taken as a bitmap
  int64_t lo[MOCHY_MAX_EDGE], hi[MOCHY_MAX_EDGE];     // the other lists
  bool light[MOCHY_MAX_EDGE];
  int a, nh, nd, nl;
};

// A heavy list is taken as a bitmap if that is no more than kWalkWords words
// for each of its hyperedges: a word costs a load of 4 bytes in order (two
// where the graph's first hyperedge is not the first bit of one), a hyperedge
// its load and one or two LDS atomics at random.
constexpr int kWalkWords = 8;

// Builds the neighbour bitmap of row i in LDS: bit x - e0 for neighbour x,
// where the row's graph owns hyperedges [e0, e1), nwords words.  kLight: also
// the bitmap of those sharing a light node with e_i.  (i's own bit is 0.)
template <bool kLight>
__device__ void build_row_bitmap(int64_t i, int64_t e0, int64_t e1, int64_t E, const int64_t* __restrict__ ptr,
                                 const int32_t* __restrict__ nodes, const int64_t* __restrict__ node_ptr,
                                 const int32_t* __restrict__ node_edges, const int8_t* __restrict__ heavy_bit,
                                 const unsigned long long* __restrict__ hrows, RowNodes& rn, uint32_t* bm,
                                 uint32_t* light, int nwords) {
  const int64_t s = ptr[i];
  const int a = int(ptr[i + 1] - s);
  if (threadIdx.x < unsigned(kWave)) {  // the first wave sorts the nodes out
    const int lane = threadIdx.x;
    int32_t v = -1;
    int hb = -1;
    int64_t lo = 0, hi = 0;
    if (lane < a) {
      v = nodes[s + lane];
      hb = heavy_bit[v];
      lo = node_ptr[v];
      hi = node_ptr[v + 1];
      rn.ei[lane] = v;
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    const unsigned long long heavy = __ballot(hb >= 0);
    const unsigned long long dense = __ballot(hb >= 0 && (hi - lo) * kWalkWords >= nwords);
    const unsigned long long walk = __ballot(lane < a && hi - lo > 1) & ~dense;
    if ((heavy >> lane) & 1ull) {
      const int at = __popcll(heavy & below);
      rn.hbit[at] = int8_t(hb);
      rn.hpos[at] = int8_t(lane);
    }
    if ((dense >> lane) & 1ull) rn.dense[__popcll(dense & below)] = int8_t(hb);
    if ((walk >> lane) & 1ull) {
      const int at = __popcll(walk & below);
      rn.lo[at] = lo;
      rn.hi[at] = hi;
      rn.light[at] = hb < 0;
    }
    if (lane == 0) {
      rn.a = a;
      rn.nh = __popcll(heavy);
      rn.nd = __popcll(dense);
      rn.nl = __popcll(walk);
    }
  }
  __syncthreads();
  const int nd = rn.nd, nl = rn.nl;
  const int64_t stride = heavy_words(E) * 2;
  const uint32_t* hw = reinterpret_cast<const uint32_t*>(hrows) + (e0 >> 5);
  const int shift = int(e0 & 31);
  const int last = nwords - 1;
  const uint32_t tail = (e1 - e0) & 31 ? (1u << ((e1 - e0) & 31)) - 1u : ~0u;  // the last word's bits
  for (int w = threadIdx.x; w < nwords; w += blockDim.x) {
    uint32_t bits = 0;
    for (int d = 0; d < nd; ++d) {
      const uint32_t* row = hw + rn.dense[d] * stride + w;
      uint32_t x = row[0] >> shift;
      if (shift) x |= row[1] << (32 - shift);
      bits |= x;
    }
    bm[w] = w == last ? bits & tail : bits;
    if (kLight) light[w] = 0u;
  }
  __syncthreads();
  for (int l = 0; l < nl; ++l) {
    const int64_t hi = rn.hi[l];
    const bool is_light = rn.light[l];
    for (int64_t r = rn.lo[l] + threadIdx.x; r < hi; r += blockDim.x) {
      const int64_t x = int64_t(node_edges[r]) - e0;
      atomicOr(&bm[x >> 5], 1u << (x & 31));
      if (kLight && is_light) atomicOr(&light[x >> 5], 1u << (x & 31));
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) bm[(i - e0) >> 5] &= ~(1u << ((i - e0) & 31));
  __syncthreads();
}

// Largest value to *most: few rows exceed what is there, and as many atomics on
// one address as rows took four times as long as the rows (22,700 rows of 9
// graphs: 266 us).
__device__ __forceinline__ void note_max(int32_t* most, int32_t n) {
  if (n > __hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(most, n);
}

__global__ __launch_bounds__(256) void k_proj_degree(int64_t E, const int64_t* __restrict__ ptr,
                                                     const int32_t* __restrict__ nodes,
                                                     const int64_t* __restrict__ node_ptr,
                                                     const int32_t* __restrict__ node_edges,
                                                     const int8_t* __restrict__ heavy_bit,
                                                     const unsigned long long* __restrict__ hrows,
                                                     const int32_t* __restrict__ row_graph,
                                                     const int64_t* __restrict__ geoff,
                                                     int64_t* deg, int32_t* max_deg) {
  extern __shared__ uint32_t bm[];
  __shared__ RowNodes rn;
  __shared__ int32_t red[256 / kWave];
  const int64_t i = blockIdx.x;
  const int gi = row_graph[i];
  const int64_t e0 = geoff[gi], e1 = geoff[gi + 1];
  const int nwords = int((e1 - e0 + 31) / 32);
  build_row_bitmap<false>(i, e0, e1, E, ptr, nodes, node_ptr, node_edges, heavy_bit, hrows, rn, bm, nullptr, nwords);
  int32_t c = 0;
  for (int w = threadIdx.x; w < nwords; w += blockDim.x) c += __popc(bm[w]);
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    c = red[0] + red[1] + red[2] + red[3];
    deg[i] = c;
    note_max(max_deg, c);
  }
}

// Row i of the line graph and its records, a block to a row.  The row's bitmap
// is turned into sorted neighbours a tile of 256 words at a time, staged in LDS
// so that the records are written in order; a neighbour's mask of e_i's heavy
// nodes and its heavy outside nodes follow from its own heavy mask.  Those that
// share a light node as well (1 to 3 of a hundred) need their nodes compared
// with e_i's; they are put off until there is one for most threads.
//
// Bound by the latency of the tiles' steps and the 26 bytes written per entry
// (2.4 TB/s).  8.7e8 entries of 85,357 rows: 9.4 ms, where a kernel for the rows
// (4.1 ms, every list walked) was followed by one that compared every
// neighbour's nodes (19.0 ms, 470 instructions for 64 entries); the same with 2
// or 8 entries of a thread in flight, 512 threads to a block, or stores past the
// caches.
constexpr int kRowThreads = 256, kRowQueue = 512;
constexpr int kRowUnroll = 4;
// Rows of up to kSweepRow neighbours are staged in one sweep over the bitmap, a
// run of words to each thread, instead of tile by tile.  Those of up to
// kShortRow, where the hypergraph has many hyperedges, are a kernel of their own
// (kShort) that compares every neighbour's nodes and so needs no second bitmap:
// a block of the other takes 48 KB of bitmaps for 190,000 hyperedges, to hold
// a row of a few entries.  Flat hypergraphs, rows and records in ms, and where
// every row went tile by tile: 190,000 hyperedges (rows of 30) 1.39, 9.95;
// 100,000 (of 80) 0.47, 2.48; 20,000 (of 64) 0.075, 0.13.  With the line at 64
// neighbours 1.39, 1.29 and 0.11, at 1,024 1.61, 0.47 and 0.076; 17,600 hub-heavy
// ones 0.45 (0.43, 0.49; 0.41 tile by tile), 85,357 9.1 (9.2, 8.9; 9.4).
constexpr int kSweepRow = 4096, kShortRow = 256;
constexpr int64_t kShortFrom = 8192;  // hyperedges of the largest graph (above: more than one tile)

template <bool kShort>
__global__ __launch_bounds__(kRowThreads) void k_proj_rows(
    int64_t E, int skip, const int64_t* __restrict__ ptr, const int32_t* __restrict__ nodes,
    const int64_t* __restrict__ node_ptr, const int32_t* __restrict__ node_edges,
    const int8_t* __restrict__ heavy_bit, const EdgeInfo* __restrict__ info,
    const unsigned long long* __restrict__ hrows, const int32_t* __restrict__ row_graph,
    const int64_t* __restrict__ geoff, const int64_t* __restrict__ lg_ptr, int32_t* lg_col, int32_t* up_first,
    uint4* rec, uint32_t* recm, uint16_t* rsz, int32_t* flags) {
  extern __shared__ uint32_t bm[];
  __shared__ RowNodes rn;
  // bits of the tile that are set, or a short enough row's entries
  __shared__ uint32_t stage[kShort ? kShortRow : kSweepRow];
  __shared__ uint2 queue[kShort ? 1 : kRowQueue];  // neighbour, position: put off
  __shared__ uint32_t filt[32];  // membership filter of e_i's nodes by their low 10 bits
  __shared__ uint32_t s_wave[kRowThreads / kWave], s_put;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t i = blockIdx.x;
  const int64_t base = lg_ptr[i];
  const int d = int(lg_ptr[i + 1] - base);
  if (kShort ? d > kShortRow : d <= skip) return;  // the other launch's (whole block)
  const int gi = row_graph[i];
  const int64_t e0 = geoff[gi], e1 = geoff[gi + 1], il = i - e0;
  const int nwords = int((e1 - e0 + 31) / 32);
  uint32_t* light = bm + nwords;
  if (tid < 32) filt[tid] = 0u;
  if (tid == 0) s_put = 0u;
  build_row_bitmap<!kShort>(i, e0, e1, E, ptr, nodes, node_ptr, node_edges, heavy_bit, hrows, rn, bm, light, nwords);
  const int a = rn.a, nh = rn.nh;
  if (tid < a) atomicOr(&filt[(rn.ei[tid] >> 5) & 31], 1u << (rn.ei[tid] & 31));
  const unsigned long long hi = info[i].heavy;
  bool dup = false;
  auto write = [&](int64_t pos, const EdgeInfo& ix, uint32_t m) {
    const unsigned long long hv = ix.heavy & ~hi;  // heavy nodes of e_x outside e_i
    const uint32_t p = uint32_t(__popc(m)), o = ix.size - p;
    if (o == 0 && p == uint32_t(a)) dup = true;
    rec[pos] = make_uint4(m, o | (o > uint32_t(__popcll(hv)) ? kRecLight : 0u), uint32_t(hv), uint32_t(hv >> 32));
    recm[pos] = m;
    rsz[pos] = uint16_t(p | ix.size << 8);
  };
  // e_x's nodes against e_i's, four at a time, their loads issued together
  // before any is used; -1 pads past the list's end
  auto compare = [&](int64_t x, int64_t pos) {
    const EdgeInfo ix = info[x];
    const int64_t q0 = ptr[x], q1 = q0 + ix.size;
    uint32_t m = 0;
    for (int64_t q = q0; q < q1; q += 4) {
      int32_t v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = q + u < q1 ? nodes[q + u] : -1;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        int lo = 0, hb = a;  // binary search of v in e_i, past the filter
        if (v[u] < 0 || !((filt[(v[u] >> 5) & 31] >> (v[u] & 31)) & 1u)) hb = 0;
        while (lo < hb) {
          const int mid = (lo + hb) >> 1;
          if (rn.ei[mid] < v[u]) lo = mid + 1; else hb = mid;
        }
        if (lo < a && rn.ei[lo] == v[u]) m |= 1u << lo;
      }
    }
    write(pos, ix, m);
  };
  // staged entries before the thread's own `n`; the block's total
  auto before = [&](uint32_t n, uint32_t& total) {
    uint32_t incl = n;
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t o = uint32_t(__shfl_up(int(incl), off));
      if (lane >= off) incl += o;
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    __syncthreads();
    uint32_t at = incl - n;
    total = 0;
    for (int y = 0; y < kRowThreads / kWave; ++y) {
      if (y < wave) at += s_wave[y];
      total += s_wave[y];
    }
    return at;
  };
  // the entries staged as bits from x0 on, written from `found` on
  auto emit = [&](const auto* staged, int64_t x0, uint32_t found, uint32_t total) {
    for (uint32_t r0 = tid; r0 < total; r0 += kRowThreads * kRowUnroll) {
      int64_t x[kRowUnroll];
      EdgeInfo ix[kRowUnroll];
#pragma unroll
      for (int u = 0; u < kRowUnroll; ++u) {
        const uint32_t r = min(r0 + u * kRowThreads, total - 1u);
        x[u] = x0 + staged[r];
        ix[u] = info[e0 + x[u]];
      }
#pragma unroll
      for (int u = 0; u < kRowUnroll; ++u) {
        const uint32_t r = r0 + u * kRowThreads;
        if (r >= total) continue;
        const int64_t pos = base + found + r;
        lg_col[pos] = int32_t(e0 + x[u]);
        if ((light[x[u] >> 5] >> (x[u] & 31)) & 1u) {
          const uint32_t put = atomicAdd(&s_put, 1u);
          if (put < uint32_t(kRowQueue)) queue[put] = make_uint2(uint32_t(e0 + x[u]), found + r);
          else compare(e0 + x[u], pos);
          continue;
        }
        uint32_t m = 0;
        for (int h = 0; h < nh; ++h) m |= uint32_t((ix[u].heavy >> rn.hbit[h]) & 1ull) << rn.hpos[h];
        write(pos, ix[u], m);
      }
    }
  };
  auto settle = [&](uint32_t put) {
    for (uint32_t y = tid; y < put; y += kRowThreads) compare(queue[y].x, base + queue[y].y);
  };
  if (kShort || d <= kSweepRow) {
    const int per = (nwords + kRowThreads - 1) / kRowThreads | 1;  // odd: runs start in different banks
    const int w0 = min(nwords, tid * per), w1 = min(nwords, w0 + per);
    uint32_t n = 0, total;
    for (int w = w0; w < w1; ++w) n += uint32_t(__popc(bm[w]));
    uint32_t at = before(n, total);
    for (int w = w0; w < w1; ++w) {
      uint32_t bits = bm[w];
      if (w == int(il >> 5)) up_first[i] = int32_t(at + uint32_t(__popc(bits & ((1u << (il & 31)) - 1u))));
      for (; bits; bits &= bits - 1u) stage[at++] = uint32_t(w * 32 + __ffs(bits) - 1);
    }
    __syncthreads();
    if (kShort) {
      for (uint32_t r = tid; r < total; r += kRowThreads) {
        const int64_t x = e0 + stage[r];
        lg_col[base + r] = int32_t(x);
        compare(x, base + r);
      }
    } else {
      emit(stage, 0, 0u, total);
      __syncthreads();
      settle(min(s_put, uint32_t(kRowQueue)));
    }
    if (dup) atomicOr(flags, kFlagDup);
    return;
  }
  uint16_t* const tile = reinterpret_cast<uint16_t*>(stage);  // kRowThreads words' bits
  static_assert(kRowThreads * 32 * sizeof(uint16_t) <= kSweepRow * sizeof(uint32_t), "the tile's stage");
  uint32_t found = 0;  // entries before the tile
  for (int t0 = 0; t0 < nwords; t0 += kRowThreads) {
    const int w = t0 + tid;
    uint32_t bits = w < nwords ? bm[w] : 0u, total;
    uint32_t at = before(uint32_t(__popc(bits)), total);
    if (w == int(il >> 5)) up_first[i] = int32_t(found + at + uint32_t(__popc(bits & ((1u << (il & 31)) - 1u))));
    for (; bits; bits &= bits - 1u) tile[at++] = uint16_t(tid * 32 + __ffs(bits) - 1);
    __syncthreads();
    emit(tile, int64_t(t0) * 32, found, total);
    found += total;
    __syncthreads();
    const uint32_t put = min(s_put, uint32_t(kRowQueue));
    if (put >= uint32_t(kRowThreads) || (put && t0 + kRowThreads >= nwords)) {
      settle(put);
      __syncthreads();
      if (tid == 0) s_put = 0u;
      __syncthreads();
    }
  }
  if (dup) atomicOr(flags, kFlagDup);
}

__global__ void k_upper_len(int64_t E, const int64_t* __restrict__ lg_ptr,
                            const int32_t* __restrict__ up_first, int64_t* up_len) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < E) up_len[i] = (lg_ptr[i + 1] - lg_ptr[i]) - up_first[i];
  if (i == E) up_len[E] = 0;
}

__global__ void k_row_graph(int64_t E, int32_t ng, const int64_t* __restrict__ geoff,
                            int32_t* row_graph) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= E) return;
  int lo = 0, hi = ng;  // last g with geoff[g] <= i
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (geoff[mid] <= i) lo = mid; else hi = mid;
  }
  row_graph[i] = lo;
}

inline unsigned blocks(int64_t n, int t) { return unsigned((n + t - 1) / t); }

}  // namespace

// Heavy nodes of every graph of the set.
static mochy_status heavy_nodes(mochy_ctx* ctx, mochy_graph* g) {
  int64_t most = 0;
  for (size_t x = 0; x + 1 < g->h_gvoff.size(); ++x) most = std::max(most, g->h_gvoff[x + 1] - g->h_gvoff[x]);
  const unsigned long long* in = nullptr;
  unsigned long long* bufs[2] = {nullptr, nullptr};
  mochy_status rc = MOCHY_OK;
  for (int level = 0; most > 0; ++level) {
    const int64_t parts = (most + kHeavyChunk - 1) / kHeavyChunk;
    unsigned long long* out = nullptr;
    if (parts > 1) {
      device_free(ctx, bufs[level & 1]);
      bufs[level & 1] = nullptr;
      if ((rc = device_alloc(ctx, (void**)&bufs[level & 1], size_t(g->ng) * parts * kHeavyBits * 8)) != MOCHY_OK) break;
      out = bufs[level & 1];
    }
    k_heavy<<<unsigned(parts * g->ng), kHeavyThreads, 0, ctx->stream>>>(g->gvoff, g->node_ptr, in, most, unsigned(parts),
                                                                        out, g->heavy_bit);
    if (!out) break;
    in = out;
    most = parts * kHeavyBits;
  }
  device_free(ctx, bufs[0]);
  device_free(ctx, bufs[1]);
  return rc;
}

mochy_status project_incidence(mochy_ctx* ctx, mochy_graph* g) {
  hipStream_t st = ctx->stream;
  const int64_t E = g->E, V = g->V, nnz = g->nnz;
  MOCHY_HIP(hipMemsetAsync(ctx->d_flags, 0, 4 * sizeof(int32_t), st));
  if (E > 0)
    k_validate<<<blocks(E, 256), 256, 0, st>>>(E, g->ng, g->geoff, g->gvoff, g->gnoff, g->edge_ptr,
                                               g->edge_nodes, ctx->d_flags);
  phase_end(ctx, kPhUpload);
  MOCHY_HIP(hipMemcpyAsync(ctx->h_small, ctx->d_flags, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  MOCHY_HIP(hipStreamSynchronize(st));
  phases_collect(ctx);
  const int32_t f0 = *reinterpret_cast<int32_t*>(ctx->h_small);
  if (f0 & kFlagInval) { ctx->err = "malformed CSR (unsorted, out-of-range or empty hyperedge)"; return MOCHY_EINVAL; }
  if (f0 & kFlagRange) { ctx->err = "a hyperedge exceeds MOCHY_MAX_EDGE nodes"; return MOCHY_ERANGE; }

  // 2. transpose
  const size_t tmpn = scan_tmp_elems(std::max<int64_t>(V, E) + 1);
  int64_t* tmp = nullptr;
  int64_t* cnt = nullptr;
  unsigned int* fill = nullptr;
  mochy_status rc;
  auto cleanup = [&]() { device_free(ctx, tmp); device_free(ctx, cnt); device_free(ctx, fill); };
  if ((rc = device_alloc(ctx, (void**)&tmp, tmpn * 8)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&cnt, size_t(std::max(V, E) + 1) * 8)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&fill, size_t(V + 1) * 4)) != MOCHY_OK) {
    cleanup();
    return rc;
  }
  if ((rc = device_alloc(ctx, (void**)&g->node_ptr, size_t(V + 1) * 8)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->node_edges, size_t(std::max<int64_t>(nnz, 1)) * 4)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->heavy_bit, size_t(std::max<int64_t>(V, 1)))) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->up_ptr, size_t(E + 1) * 8)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->row_graph, size_t(std::max<int64_t>(E, 1)) * 4)) != MOCHY_OK) { cleanup(); return rc; }
  if (E > 0) k_row_graph<<<blocks(E, 256), 256, 0, st>>>(E, g->ng, g->geoff, g->row_graph);
  g->bytes += size_t(V + 1) * 8 + size_t(nnz) * 4 + size_t(V) + size_t(E + 1) * 8 + size_t(E) * 4;

  phase_begin(ctx, kPhTranspose);
  MOCHY_HIP(hipMemsetAsync(cnt, 0, size_t(V + 1) * 8, st));
  MOCHY_HIP(hipMemsetAsync(fill, 0, size_t(V + 1) * 4, st));
  if (E > 0)
    k_transpose<false><<<blocks(E, kNodeThreads), kNodeThreads, 0, st>>>(E, g->edge_ptr, g->edge_nodes, nullptr,
                                                                         (unsigned long long*)cnt, nullptr, nullptr);
  launch_exclusive_scan_i64(cnt, g->node_ptr, V + 1, tmp, st);
  if (E > 0)
    k_transpose<true><<<blocks(E, kNodeThreads), kNodeThreads, 0, st>>>(E, g->edge_ptr, g->edge_nodes, g->node_ptr,
                                                                        nullptr, fill, g->node_edges);
  // 3. heavy nodes
  if ((rc = heavy_nodes(ctx, g)) != MOCHY_OK) { cleanup(); return rc; }
  phase_end(ctx, kPhTranspose);
  MOCHY_HIP(hipStreamSynchronize(st));
  cleanup();
  return MOCHY_OK;
}

mochy_status project_device(mochy_ctx* ctx, mochy_graph* g) {
  hipStream_t st = ctx->stream;
  const int64_t E = g->E;
  if (g->max_graph_edges > kMaxGraphEdges) {
    ctx->err = "a graph of a batch exceeds 200000 hyperedges (the line-graph-free mode takes single graphs)";
    return MOCHY_EUNSUPPORTED;
  }
  mochy_status rc = project_incidence(ctx, g);
  if (rc != MOCHY_OK) return rc;
  const size_t tmpn = scan_tmp_elems(E + 1);
  int64_t* tmp = nullptr;
  int64_t* cnt = nullptr;
  EdgeInfo* info = nullptr;  // and the heavy nodes' bitmaps after it
  auto cleanup = [&]() { device_free(ctx, tmp); device_free(ctx, cnt); device_free(ctx, info); };
  auto fail = [&](mochy_status e) { cleanup(); return e; };
  if ((rc = device_alloc(ctx, (void**)&tmp, tmpn * 8)) != MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&info, size_t(E) * sizeof(EdgeInfo) + size_t(kHeavyBits) * heavy_words(E) * 8)) !=
          MOCHY_OK ||
      (rc = device_alloc(ctx, (void**)&cnt, size_t(E + 1) * 8)) != MOCHY_OK) {
    cleanup();
    return rc;
  }
  if ((rc = device_alloc(ctx, (void**)&g->lg_ptr, size_t(E + 1) * 8)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->up_first, size_t(std::max<int64_t>(E, 1)) * 4)) != MOCHY_OK) { cleanup(); return rc; }
  g->bytes += size_t(E + 1) * 8 + size_t(E) * 4;

  // 4-5. degrees and row pointers
  const int nwords = int((g->max_graph_edges + 31) / 32);
  const size_t bm_bytes = size_t(std::max(nwords, 1)) * 4;
  phase_begin(ctx, kPhDegree);
  MOCHY_HIP(hipMemsetAsync(cnt, 0, size_t(E + 1) * 8, st));
  MOCHY_HIP(hipMemsetAsync(ctx->d_flags + 1, 0, sizeof(int32_t), st));
  unsigned long long* hrows = reinterpret_cast<unsigned long long*>(info + E);
  if (E > 0) {
    k_edge_heavy<<<blocks(heavy_words(E) * kWave, 256), 256, 0, st>>>(E, g->edge_ptr, g->edge_nodes, g->heavy_bit, info,
                                                                      hrows);
    k_proj_degree<<<unsigned(E), 256, bm_bytes, st>>>(E, g->edge_ptr, g->edge_nodes, g->node_ptr, g->node_edges,
                                                      g->heavy_bit, hrows, g->row_graph, g->geoff, cnt,
                                                      ctx->d_flags + 1);
  }
  launch_exclusive_scan_i64(cnt, g->lg_ptr, E + 1, tmp, st);
  phase_end(ctx, kPhDegree);
  MOCHY_HIP(hipMemcpyAsync(ctx->h_small, g->lg_ptr + E, 8, hipMemcpyDeviceToHost, st));
  MOCHY_HIP(hipMemcpyAsync(ctx->h_small + 1, ctx->d_flags + 1, 4, hipMemcpyDeviceToHost, st));
  MOCHY_HIP(hipStreamSynchronize(st));
  phases_collect(ctx);
  const int64_t twoW = ctx->h_small[0];
  g->W = twoW / 2;
  g->max_deg = *reinterpret_cast<int32_t*>(ctx->h_small + 1);

  // 6. rows
  if ((rc = device_alloc(ctx, (void**)&g->lg_col, size_t(std::max<int64_t>(twoW, 1)) * 4)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->rec, size_t(std::max<int64_t>(twoW, 1)) * 16)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->recm, size_t(std::max<int64_t>(twoW, 1)) * 4)) != MOCHY_OK) { cleanup(); return rc; }
  if ((rc = device_alloc(ctx, (void**)&g->rsz, size_t(std::max<int64_t>(twoW, 1)) * 2)) != MOCHY_OK) { cleanup(); return rc; }
  g->bytes += size_t(twoW) * 26;
  phase_begin(ctx, kPhRows);
  const bool split = g->max_graph_edges > kShortFrom;
  if (split) {
    if ((rc = allow_lds(ctx, (const void*)k_proj_rows<true>, bm_bytes)) != MOCHY_OK) return fail(rc);
    k_proj_rows<true><<<unsigned(E), kRowThreads, bm_bytes, st>>>(
        E, 0, g->edge_ptr, g->edge_nodes, g->node_ptr, g->node_edges, g->heavy_bit, info, hrows, g->row_graph, g->geoff,
        g->lg_ptr, g->lg_col, g->up_first, g->rec, g->recm, g->rsz, ctx->d_flags);
  }
  if (E > 0 && (!split || g->max_deg > kShortRow)) {
    if ((rc = allow_lds(ctx, (const void*)k_proj_rows<false>, 2 * bm_bytes)) != MOCHY_OK) return fail(rc);
    k_proj_rows<false><<<unsigned(E), kRowThreads, 2 * bm_bytes, st>>>(
        E, split ? kShortRow : -1, g->edge_ptr, g->edge_nodes, g->node_ptr, g->node_edges, g->heavy_bit, info, hrows,
        g->row_graph, g->geoff, g->lg_ptr, g->lg_col, g->up_first, g->rec, g->recm, g->rsz, ctx->d_flags);
  }
  phase_end(ctx, kPhRows);
  phase_begin(ctx, kPhRecords);
  // upper-row prefix (hyperwedge order for sampling)
  k_upper_len<<<blocks(E + 1, 256), 256, 0, st>>>(E, g->lg_ptr, g->up_first, cnt);
  launch_exclusive_scan_i64(cnt, g->up_ptr, E + 1, tmp, st);
  phase_end(ctx, kPhRecords);
  MOCHY_HIP(hipMemcpyAsync(ctx->h_small, ctx->d_flags, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  MOCHY_HIP(hipStreamSynchronize(st));
  phases_collect(ctx);
  cleanup();
  const int32_t f1 = *reinterpret_cast<int32_t*>(ctx->h_small);
  if (f1 & kFlagDup) { ctx->err = "duplicate hyperedges (pass MOCHY_DEDUP for host input)"; return MOCHY_EDUP; }
  // what the on-the-fly sampler walks is built on a single graph's first
  // sampling call (mochy_count_sampled)
  return MOCHY_OK;
}
