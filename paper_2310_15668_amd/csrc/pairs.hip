// Pairs of neighbour groups of long rows on the matrix cores.
//
// A pair of groups (j, k) of a centre e_i enters the counts through t =
// popcount(m_j & m_k) and r5 = popcount(h_j & h_k) only, two dot products of
// bit vectors: an MFMA over the 32 mask bits and the 64 heavy bits forms them
// for 32 x 32 pairs at a time.  What is left per pair is a weighted count by
// (t, r5), done without classifying the pair:
//
//  * both groups above the centre: the MFMA's integer scales make its result
//    the LDS byte address of a counter of (j's type, t, r5) private to the
//    column k, and one ds_add_u32 adds j's counts (A | N << 16) there.  A
//    type is (|m|, outside count); the counters of a window of types are read
//    once the window's rows are done, classified once each, and weighted with
//    k's counts (N N where disjoint, A A otherwise);
//  * otherwise only disjoint pairs count: an FP4 MFMA with block scales forms
//    2^23 + (t + r5 of j) + 2^16 (t + r5 of j + 32) in one accumulator, and a
//    packed saturating subtract and a two-term dot product add the N of the
//    two rows where the overlap is zero (all exact: integers below 2^24).
//
// A wave takes 128 columns of one row (the same work item queue as the other
// pair kernel) and walks the rows j in blocks of 32 or 64.
//
// Measured on the medium workload (85,476 hyperedges; 4.4e11 pairs of groups
// above the centre, 7.7e11 others): 77 ms and 71 ms, where classifying pair by
// pair (19 and 5 vector instructions) took 345 ms for both.  k_pairs_full is
// bound by LDS atomics: a ds_add_u32 of 64 lanes at words of their own takes 4.1
// cycles of a CU, 46 ms of the 77 in all, the rest being counters read
// back, rows without a full block and latency at two waves per SIMD.
// k_pairs_open spends two half-rate vector instructions on two rows x 64
// columns, beside 0.75 cycles of MFMA per 64 pairs: a bound of 35 ms.
#include <algorithm>

#include "pairs.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------------------
// Rows and their order.

// Sorts the groups of one kind at rec[0 .. n), cnt[0 .. n) in place: by type
// and then open class (kAbove), or by open class.  Returns the number sorted
// by type.  Every thread of the block calls it; a thread holds kSortPer
// groups in registers, and groups past kSortMax keep their places.
constexpr int kSortThreads = 1024, kSortPer = 12;
constexpr int kSortMax = kSortThreads * kSortPer;

template <bool kAbove>
__device__ __forceinline__ int sort_groups(uint4* rec, uint32_t* cnt, int n, uint32_t* bins, uint32_t* s_el) {
  constexpr int kKeys = kAbove ? kTypes : 0;
  constexpr int kBins = kKeys + kOpenClasses;
  const int tid = threadIdx.x;
  n = min(n, kSortMax);
  for (int t = tid; t < kBins; t += kSortThreads) bins[t] = 0u;
  if (tid == 0) *s_el = 0u;
  __syncthreads();
  uint4 r[kSortPer];
  uint32_t c[kSortPer];
  auto key_of = [](const uint4& x) -> int {
    const int t = kAbove ? group_type(x.x, (x.y >> 16) & 0xffu, x.z, x.w) : -1;
    return t >= 0 ? t : kKeys + int(x.y >> 24);
  };
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const int x = tid + u * kSortThreads;
    if (x < n) {
      r[u] = rec[x];
      c[u] = cnt[x];
      atomicAdd(&bins[key_of(r[u])], 1u);
    }
  }
  __syncthreads();
  uint32_t* moved = bins + kBins;  // types with too few groups join the rest
  uint32_t mine = 0;
  if (tid < kKeys) {
    mine = bins[tid];
    moved[tid] = mine < uint32_t(kMinType) ? 1u : 0u;
    if (!moved[tid]) atomicAdd(s_el, mine);
  }
  __syncthreads();
  if (tid < kKeys && moved[tid]) {
    bins[tid] = 0u;
    if (mine) atomicAdd(&bins[kKeys + type_open_class(tid)], mine);
  }
  __syncthreads();
  if (tid < kWave) wave_prefix(bins, kBins, 0u, tid);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSortPer; ++u) {
    const int x = tid + u * kSortThreads;
    if (x < n) {
      int k = key_of(r[u]);
      if (k < kKeys && moved[k]) k = kKeys + int(r[u].y >> 24);
      const uint32_t pos = atomicAdd(&bins[k], 1u);
      rec[pos] = r[u];
      cnt[pos] = c[u];
    }
  }
  __syncthreads();
  const int el = int(*s_el);
  __syncthreads();
  return el;
}

// Rows grouped in several hash parts (listed by the grouping), whose groups
// come part by part: one block per row at a time, from a queue.
__global__ __launch_bounds__(kSortThreads) void k_sort_groups(
    const int32_t* __restrict__ rows, const unsigned long long* __restrict__ nrows, unsigned long long* queue,
    RowGroups G, uint4* rec, uint32_t* cnt, int32_t* elig) {
  __shared__ uint32_t bins[kAboveKeys + kTypes];
  __shared__ uint32_t s_el;
  __shared__ int64_t s_q;
  const int64_t n = int64_t(*nrows);
  for (;;) {  // every block leaves once the list is taken
    if (threadIdx.x == 0) s_q = int64_t(atomicAdd(queue, 1ull));
    __syncthreads();
    const int64_t q = s_q;
    __syncthreads();
    if (q >= n) break;
    const int32_t i = rows[q];
    const int ng = int(G.goff[i + 1] - G.goff[i]), na = G.gna[i];
    const int64_t gb = G.gbase[i] - G.cap0, end = G.gbase[i + 1] - G.cap0;
    const int e = sort_groups<true>(rec + gb, cnt + gb, na, bins, &s_el);
    sort_groups<false>(rec + end - (ng - na), cnt + end - (ng - na), ng - na, bins, &s_el);
    if (threadIdx.x == 0) elig[i] = e;
  }
}

// ---------------------------------------------------------------------------
// The pair kernel.

constexpr int kPairWaves = 4;               // waves per block
constexpr int kCells = 32;                  // counters per column
constexpr int kCellWords = kCells * kMfmaCols;
constexpr int kFullCopies = 2, kOpenCopies = 4;  // histogram copies per block

// Four bits as four bytes of value 1 << s.
template <int s>
__device__ __forceinline__ int bytes4(uint32_t nib) {
  constexpr int m = s < 2 ? s : 2;  // a 24-bit multiplier: bits 0, 7, 14, 21, moved up by m
  return int(__umul24(nib << (s - m), 0x204081u << m) & (0x01010101u << s));
}
template <int s>
__device__ __forceinline__ v4i bytes16(uint32_t b) {
  v4i r;
  r.x = bytes4<s>(b & 15u);
  r.y = bytes4<s>((b >> 4) & 15u);
  r.z = bytes4<s>((b >> 8) & 15u);
  r.w = bytes4<s>((b >> 12) & 15u);
  return r;
}
// The heavy bits of a row j, 16 of the 32 per wave half: bits 3..6 of every
// byte as they stand, values 8..64, and (the other half) the rest, brought
// there by swapping the nibbles.  The columns hold the same bits with values
// 64..8, so that every product is 512.
__device__ __forceinline__ uint32_t half_word(uint32_t x, int h) {
  return h ? ((x & 0x0f0f0f0fu) << 4) | ((x >> 4) & 0x0f0f0f0fu) : x;
}
__device__ __forceinline__ v4i row_bytes(uint32_t x, int h) {
  const uint32_t w = half_word(x, h);
  v4i r;
  r.x = int(w & 0x08080808u);
  r.y = int(w & 0x10101010u);
  r.z = int(w & 0x20202020u);
  r.w = int(w & 0x40404040u);
  return r;
}
__device__ __forceinline__ v4i col_bytes(uint32_t x, int h) {
  const uint32_t w = half_word(x, h);
  v4i r;
  r.x = int((w << 3) & 0x40404040u);
  r.y = int((w << 1) & 0x20202020u);
  r.z = int((w >> 1) & 0x10101010u);
  r.w = int((w >> 3) & 0x08080808u);
  return r;
}
// 32 bits as 32 FP4 (E2M1) values: those of a nibble's bits 0, 1, 2 as they
// stand (0.5, 1, 2), bit 3 as 0.5; the columns hold the reciprocals.
__device__ __forceinline__ v8i row_fp4(uint32_t x) {
  v8i r = {};
  r[0] = int(x & 0x11111111u);
  r[1] = int(x & 0x22222222u);
  r[2] = int(x & 0x44444444u);
  r[3] = int((x >> 3) & 0x11111111u);
  return r;
}
__device__ __forceinline__ v8i col_fp4(uint32_t x) {
  v8i r = {};
  r[0] = int((x << 2) & 0x44444444u);
  r[1] = int(x & 0x22222222u);
  r[2] = int((x >> 2) & 0x11111111u);
  r[3] = int((x >> 1) & 0x44444444u);
  return r;
}

__device__ __forceinline__ uint32_t lane_of(uint32_t v, int l) {
  return uint32_t(__builtin_amdgcn_readlane(int(v), l));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, uint32_t(__shfl_xor(int(v), off, kWave)));
  return lane_of(v, 0);
}
// All ones if bit b of x is set.
__device__ __forceinline__ uint32_t bit_mask(uint32_t x, int b) { return uint32_t(int(x << (31 - b)) >> 31); }

// Column of a work item: the lane's own two columns are kb + lane and kb + 64 + lane.
struct Column {
  uint32_t meta = 0, kn = 0, ka = 0;
};

struct RowView {  // one kind of a row's groups
  const uint4* rec;
  const uint32_t* cnt;
  int n, ns;      // groups, and how many lead by type (above the centre)
};

__device__ __forceinline__ Side side_of(const uint4& r) {
  Side k;
  k.m = r.x;
  k.o = (r.y >> 16) & 0xffu;
  k.s = r.y & 0xffu;
  k.h = (unsigned long long)r.z | ((unsigned long long)r.w << 32);
  return k;
}

// The types a window's counters stand for: rows of |m| = p (0: no window) and
// outside counts [oa, ob), those from Rt + 2 on taken as one (r5 <= Rt, so at
// least two outside nodes stay); ol = the last one met.  Counter (o, t, r) is
// number (o - oa) W + t Rs + r, t <= pT, r < Rs = Rt + 1.
struct Window {
  uint32_t p = 0, oa = 0, ob = 0, ol = 0, pT = 0, W = 0;
};

// Reads and clears the counters of one window, classifies each counter once
// per column and adds it with the column's weight.
__device__ __forceinline__ void window_flush(uint32_t* cells, int lane, uint32_t a, const Window& win, uint32_t Rs,
                                             const Column& c0, const Column& c1,
                                             const uint16_t* __restrict__ lut, unsigned long long* hist) {
  const uint32_t p = win.p, oa = win.oa, ol = win.ol, pT = win.pT, W = win.W;
  for (uint32_t o = oa; o <= ol; ++o) {
    const uint32_t rmax = min(o, Rs - 1u);
    for (uint32_t t = 0; t <= pT; ++t) {
      uint32_t* w = cells + ((o - oa) * W + t * Rs) * uint32_t(kMfmaCols) + lane;
      const uint32_t cj = 729u * st3(t) + 27u * st3(p - t);
      uint32_t ck[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const uint32_t ks = (s ? c1.meta : c0.meta) & 0xffu;
        ck[s] = cj + 243u * st3(ks - t) + st3(a + t - p - ks);
      }
      for (uint32_t r = 0; r <= rmax; ++r, w += kMfmaCols) {
        const uint32_t v0 = w[0], v1 = w[kWave];
        if (__ballot((v0 | v1) != 0u) == 0ull) continue;
        w[0] = 0u;
        w[kWave] = 0u;
        const bool disjoint = (t | r) == 0u;
        const uint32_t cr = 81u * st3(r) + 3u * st3(o - r);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const Column& c = s ? c1 : c0;
          const uint32_t v = s ? v1 : v0;
          const uint32_t ko = (c.meta >> 16) & 0xffu;
          const uint32_t wt = disjoint ? (v >> 16) * c.kn : (v & 0xffffu) * c.ka;
          const uint32_t code = ck[s] + cr + 9u * st3(ko - r);
          if (wt) atomicAdd(hist_at(hist, lut[kNumCodes - 1 - code]), (unsigned long long)wt);
        }
      }
    }
  }
}

// What a tile of columns brings to the rows.
struct FullColumns {
  const v4i *bm, *bl, *bh;  // the four column blocks' operands
  v16i cinit;               // LDS address of the lane's column
  const Column &c0, &c1;
  uint32_t pkm, Rt;         // largest |m| (at most 3) and heavy count (at most 7) of a column
  uint32_t dm;              // bit x: row x of a 32 x 32 diagonal block is before the lane's column
};

// Rows [j0, jmax) of the groups by type against the columns, 32 at a time.
// kDiag: j0 = kb, the columns' own position, and only earlier rows count.
template <bool kDiag>
__device__ __forceinline__ void full_rows(const RowView& A, int j0, int jmax, int kb, uint32_t a,
                                          const FullColumns& F, Window& win, uint32_t* cells, int lane,
                                          const uint16_t* __restrict__ lut, unsigned long long* hist) {
  const int h = lane >> 5, c = lane & 31;
  const uint32_t Rt = F.Rt, Rs = Rt + 1u;
  uint4 rn = make_uint4(0, 0, 0, 0);
  if (j0 < jmax) rn = A.rec[j0 + c];
  for (; j0 < jmax; j0 += 32) {
    const uint4 r = rn;
    if (j0 + 32 < jmax) rn = A.rec[j0 + 32 + c];
    const int lim = jmax - j0;
    uint32_t rem = lim >= 32 ? ~0u : (1u << lim) - 1u;
    const uint32_t prow = r.y & 0xffu, om = min((r.y >> 16) & 0xffu, Rt + 2u);
    while (rem) {
      if (win.p == 0u) {
        const int f = __ffs(int(rem)) - 1;
        win.p = lane_of(prow, f);
        win.oa = lane_of(om, f);
        win.pT = min(win.p, F.pkm);
        win.W = (win.pT + 1u) * Rs;
        win.ob = win.oa + uint32_t(kCells) / win.W;
      }
      const uint32_t act = uint32_t(__ballot(prow == win.p && om >= win.oa && om < win.ob)) & rem;
      rem &= ~act;
      if (act) {
        win.ol = lane_of(om, 31 - __clz(int(act)));
        uint32_t wa[16];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const u32x4 w = *reinterpret_cast<const u32x4*>(A.cnt + j0 + 8 * x + 4 * h);
#pragma unroll
          for (int y = 0; y < 4; ++y) wa[4 * x + y] = w[y];
        }
        const bool on = (act >> c) & 1u;
        const uint32_t m = on ? r.x : 0u, hl = on ? r.z : 0u, hh = on ? r.w : 0u;
        v4i am = bytes16<6>((m >> (16 * h)) & 0xffffu);
        if (h && on) am.w |= int(__umul24((om - win.oa) * win.W, 0x0404u) << 16);
        const v4i al = row_bytes(hl, h), ah = row_bytes(hh, h);
        if (act != ~0u) {
          const uint32_t ah4 = act >> (4 * h);
#pragma unroll
          for (int x = 0; x < 16; ++x) wa[x] &= bit_mask(ah4, 8 * (x >> 2) + (x & 3));
        }
        const int rd = kDiag ? (j0 - kb) >> 5 : -1;  // the column block on the diagonal
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (kDiag && q < rd) continue;  // columns before these rows
          v16i d = __builtin_amdgcn_mfma_i32_32x32x32_i8(am, F.bm[q], F.cinit, 0, 0, 0);
          d = __builtin_amdgcn_mfma_i32_32x32x32_i8(al, F.bl[q], d, 0, 0, 0);
          d = __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, F.bh[q], d, 0, 0, 0);
          const uint32_t keep = kDiag && q == rd ? F.dm : ~0u;
#pragma unroll
          for (int x = 0; x < 16; ++x) {
            auto* p = (__attribute__((address_space(3))) uint32_t*)(uintptr_t)uint32_t(d[x]) + 32 * q;
            __hip_atomic_fetch_add(p, kDiag ? wa[x] & bit_mask(keep, x) : wa[x], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
      if (rem) {  // the window's rows are done
        window_flush(cells, lane, a, win, Rs, F.c0, F.c1, lut, hist);
        win.p = 0u;
      }
    }
  }
}

// Columns [kb, kb + 128) of the groups above the centre against the groups
// above it that come before them.
__device__ __forceinline__ void full_tile(const RowView& A, int kb, uint32_t a, uint32_t* cells, int lane,
                                          const uint16_t* __restrict__ lut, unsigned long long* hist) {
  const int h = lane >> 5, c = lane & 31;
  // the four column blocks' operands
  uint4 kr[4];
  uint32_t pk = 0, hk = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = kb + 32 * q + c;
    kr[q] = k < A.n ? A.rec[k] : make_uint4(0, 0, 0, 0);
    pk = max(pk, kr[q].y & 0xffu);
    hk = max(hk, uint32_t(__popc(kr[q].z) + __popc(kr[q].w)));
  }
  const uint32_t pkm = min(wave_max(pk), 3u), Rt = min(wave_max(hk), 7u), Rs = Rt + 1u;
  v4i bm[4], bl[4], bh[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    bm[q] = bytes16<0>((kr[q].x >> (16 * h)) & 0xffffu) * int(8u * Rs);
    bl[q] = col_bytes(kr[q].z, h);
    bh[q] = col_bytes(kr[q].w, h);
    // mask bits 30 and 31 (no node of e_i) carry the row's window slot
    if (h) bm[q].w |= int(0x40400000u);
  }
  Column c0, c1;
  if (kb + lane < A.n) {
    const uint32_t w = A.cnt[kb + lane];
    c0.meta = A.rec[kb + lane].y;
    c0.kn = cnt_all(w);
    c0.ka = cnt_above(w);
  }
  if (kb + kWave + lane < A.n) {
    const uint32_t w = A.cnt[kb + kWave + lane];
    c1.meta = A.rec[kb + kWave + lane].y;
    c1.kn = cnt_all(w);
    c1.ka = cnt_above(w);
  }
  v16i cinit;
  {
    const int base = int(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t*)cells)) + 4 * c;
#pragma unroll
    for (int x = 0; x < 16; ++x) cinit[x] = base;
  }
  // diagonal blocks: the rows of a 32 x 32 block below column c
  uint32_t dm = 0;
#pragma unroll
  for (int x = 0; x < 16; ++x) dm |= (8 * (x >> 2) + 4 * h + (x & 3) < c ? 1u : 0u) << x;

  FullColumns F = {bm, bl, bh, cinit, c0, c1, pkm, Rt, dm};
  Window win;
  full_rows<false>(A, 0, min(A.ns, kb), kb, a, F, win, cells, lane, lut, hist);
  full_rows<true>(A, kb, min(A.ns, kb + kMfmaCols), kb, a, F, win, cells, lane, lut, hist);
  if (win.p) window_flush(cells, lane, a, win, Rs, c0, c1, lut, hist);

  // rows of the rest, lane per pair; and pairs inside a group
#pragma unroll 1
  for (int s = 0; s < 2; ++s) {
    const int k0 = kb + s * kWave, kp = k0 + lane;
    if (k0 >= A.n) break;
    const uint4 rk = kp < A.n ? A.rec[kp] : make_uint4(0, 0, 0, 0);
    const Column& cc = s ? c1 : c0;
    const Side k = side_of(rk);
    const uint32_t aks = a - k.s;
    if (A.ns < k0 + kWave) {
      if (A.ns < k0) gwalk<false, true, true>(A.rec, A.cnt, A.ns, k0, aks, k, cc.kn, cc.ka, kp, lut, hist);
      gwalk<true, false, true>(A.rec, A.cnt, max(A.ns, k0), min(k0 + kWave, A.n), aks, k, cc.kn, cc.ka, kp, lut,
                               hist);
    }
    if (cc.ka >= 2u) {
      const uint32_t code = pair_code(a, k.s, k.o, k, k.s, uint32_t(__popcll(k.h)));
      atomicAdd(hist_at(hist, lut[kNumCodes - 1 - code]), uint64_t(cc.ka) * (cc.ka - 1u) / 2u);
    }
  }
}

// ---------------------------------------------------------------------------
// Open pairs.

constexpr int kMinOpen = 20;  // rows of one class worth a pass over 64 of them

// The lane's own two columns and what is summed for them.
struct OpenColumns {
  Column c0, c1;
  uint32_t m0, l0, h0, m1, l1, h1;  // records
  uint32_t s0, s1;                  // N of the scalar rows of the current class
  uint32_t acc[4];                  // N of the others, by column block and wave half
  uint32_t cur;                     // current class
};

__device__ __forceinline__ void open_end(OpenColumns& C, uint32_t a, int lane, const uint16_t* __restrict__ lut,
                                         unsigned long long* hist) {
  // the two halves hold the same columns: block q's column c is lane c + 32 (q % 2) of set q / 2
  uint32_t s[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    s[q] = C.acc[q] + uint32_t(__shfl_xor(int(C.acc[q]), 32, kWave));
    C.acc[q] = 0u;
  }
  auto k0_of = [](const Column& x) { return 243u * st3(x.meta & 0xffu) + 9u * st3((x.meta >> 16) & 0xffu); };
  const bool h = lane >= 32;
  open_flush(C.cur, C.s0 + (h ? s[1] : s[0]), a - (C.c0.meta & 0xffu), k0_of(C.c0), C.c0.kn, lut, hist);
  open_flush(C.cur, C.s1 + (h ? s[3] : s[2]), a - (C.c1.meta & 0xffu), k0_of(C.c1), C.c1.kn, lut, hist);
  C.s0 = 0u;
  C.s1 = 0u;
}

// The open pairs of the columns with the rows rec[j0 .. n), 64 at a time.
// kDiag: the columns are rows [kb, kb + 128) of the same list, and only earlier
// rows count.
template <bool kDiag>
__device__ __forceinline__ void open_rows(const uint4* __restrict__ rec, const uint32_t* __restrict__ cnt, int j0,
                                          int n, int kb, uint32_t a, const v8i* b1, const v8i* b2, const v8i* b3,
                                          int lane, OpenColumns& C, const uint16_t* __restrict__ lut,
                                          unsigned long long* hist) {
  const int h = lane >> 5, c = lane & 31;
  float magic = 8388608.0f;  // 2^23: the integer stands in the low mantissa bits
  asm volatile("" : "+v"(magic));  // held in registers, not rebuilt for every product
  v16f cinit;
#pragma unroll
  for (int x = 0; x < 16; ++x) cinit[x] = magic;
  asm volatile("" : "+v"(cinit));
  const int s2 = h ? 143 : 127;                         // block scales 2^0 and 2^16
  const u16x2 one = __builtin_bit_cast(u16x2, 0x4b010001u);  // 1 in both halves (2^23's exponent is 0x4b00)
  uint4 rn1 = make_uint4(0, 0, 0, 0), rn2 = rn1;
  if (j0 < n) {
    rn1 = rec[j0 + c];
    rn2 = rec[j0 + 32 + c];
  }
  for (; j0 < n; j0 += 64) {
    const uint32_t cls1 = rn1.y >> 24, cls2 = rn2.y >> 24;
    const v8i a1 = row_fp4(h ? rn1.z : rn1.x), a2 = row_fp4(h ? rn2.x : rn1.w), a3 = row_fp4(h ? rn2.w : rn2.z);
    if (j0 + 64 < n) {
      rn1 = rec[j0 + 64 + c];
      rn2 = rec[j0 + 96 + c];
    }
    const int lim = n - j0;
    uint32_t rem1 = lim >= 32 ? ~0u : (1u << lim) - 1u;
    uint32_t rem2 = lim >= 64 ? ~0u : lim <= 32 ? 0u : (1u << (lim - 32)) - 1u;
    while (rem1 | rem2) {
      const uint32_t cls = rem1 ? lane_of(cls1, __ffs(int(rem1)) - 1) : lane_of(cls2, __ffs(int(rem2)) - 1);
      if (cls != C.cur) {
        open_end(C, a, lane, lut, hist);
        C.cur = cls;
      }
      const uint32_t act1 = uint32_t(__ballot(cls1 == cls)) & rem1, act2 = uint32_t(__ballot(cls2 == cls)) & rem2;
      rem1 &= ~act1;
      rem2 &= ~act2;
      if (__popc(act1) + __popc(act2) < kMinOpen) {  // few rows: one at a time, a lane per column
        uint64_t rows = uint64_t(act1) | (uint64_t(act2) << 32);
        while (rows) {
          const int j = j0 + __builtin_ctzll(rows);
          rows &= rows - 1;
          const uint4 rj = rec[j];
          const uint32_t nj = cnt_all(cnt[j]);
          const uint32_t x0 = and_or(rj.w, C.h0, and_or(rj.z, C.l0, rj.x & C.m0));
          const uint32_t x1 = and_or(rj.w, C.h1, and_or(rj.z, C.l1, rj.x & C.m1));
          if (!kDiag) {
            acc_disjoint(C.s0, x0, nj);
            acc_disjoint(C.s1, x1, nj);
          } else {
            if (x0 == 0u && j < kb + lane) C.s0 += nj;
            if (x1 == 0u && j < kb + kWave + lane) C.s1 += nj;
          }
        }
        continue;
      }
      uint32_t wa[16];  // N of row j and, above, of row j + 32
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const u32x4 w1 = *reinterpret_cast<const u32x4*>(cnt + j0 + 8 * x + 4 * h);
        const u32x4 w2 = *reinterpret_cast<const u32x4*>(cnt + j0 + 32 + 8 * x + 4 * h);
#pragma unroll
        for (int y = 0; y < 4; ++y) wa[4 * x + y] = __builtin_amdgcn_perm(w2[y], w1[y], 0x07060302u);
      }
      if ((act1 & act2) != ~0u) {
        const uint32_t x1 = act1 >> (4 * h), x2 = act2 >> (4 * h);
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const int b = 8 * (x >> 2) + (x & 3);
          wa[x] &= (bit_mask(x1, b) & 0xffffu) | (bit_mask(x2, b) & 0xffff0000u);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (kDiag && j0 >= kb + 32 * q + 32) continue;  // rows after these columns
        v16f d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a1, b1[q], cinit, 4, 4, 0, 127, 0, 127);
        d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a2, b2[q], d, 4, 4, 0, s2, 0, 127);
        d = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a3, b3[q], d, 4, 4, 0, 143, 0, 127);
        uint32_t s = C.acc[q], s1 = 0u;  // two chains of dependent adds
        int jd = j0 + 4 * h - (kb + 32 * q + c);
        if (kDiag) asm volatile("" : "+v"(jd));  // masks formed here, not kept for every column block
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          // max(1 - overlap, 0) of both rows
          const u16x2 z = __builtin_elementwise_sub_sat(one, __builtin_bit_cast(u16x2, __float_as_uint(d[x])));
          uint32_t w = wa[x];
          if (kDiag) {
            const int b = 8 * (x >> 2) + (x & 3);
            w &= (jd + b < 0 ? 0xffffu : 0u) | (jd + b + 32 < 0 ? 0xffff0000u : 0u);
          }
          uint32_t& t = (x & 1) ? s1 : s;
          t = __builtin_amdgcn_udot2(z, __builtin_bit_cast(u16x2, w), t, false);
        }
        C.acc[q] = s + s1;
        __builtin_amdgcn_sched_barrier(0);  // one column block at a time: its accumulators are reused
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The kernels: persistent waves pulling (row, tile) items.

__global__ __launch_bounds__(kPairWaves * kWave, 2) void k_pairs_full(RowGroups G, WorkItems I,
                                                                      const uint16_t* __restrict__ code_to_id3,
                                                                      unsigned long long* out) {
  __shared__ uint16_t lut[kNumCodes];
  __shared__ unsigned long long hist[kFullCopies * kGStride];
  __shared__ uint32_t cells[kPairWaves * kCellWords];
  for (int t = threadIdx.x; t < kNumCodes; t += blockDim.x) lut[t] = uint16_t(code_to_id3[kNumCodes - 1 - t] * 8u);
  for (int t = threadIdx.x; t < kFullCopies * kGStride; t += blockDim.x) hist[t] = 0ull;
  for (int t = threadIdx.x; t < kPairWaves * kCellWords; t += blockDim.x) cells[t] = 0u;
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  unsigned long long* myhist = hist + (lane & (kFullCopies - 1)) * kGStride;
  visit_graphs(
      I,
      [&](int g, const ItemRange& items) {
        int32_t i;
        int tile;
        while (next_item(items, lane, i, tile)) {
          const int64_t gb = G.gbase[i] - G.cap0;
          const uint32_t a = uint32_t(G.edge_ptr[i + 1] - G.edge_ptr[i]);
          const RowView A = {G.rec + gb, G.cnt + gb, G.gna[i], G.elig[i]};
          full_tile(A, tile * kMfmaCols, a, cells + wave * kCellWords, lane, lut, myhist);
        }
      },
      [&](int g) { hist_flush<kFullCopies>(hist, g, out); });
}

// Columns [kb, kb + 128) of the groups with no member above the centre
// against every group before them: open pairs only.
__global__ __launch_bounds__(kPairWaves * kWave, 2) void k_pairs_open(RowGroups G, WorkItems I,
                                                                      const uint16_t* __restrict__ code_to_id3,
                                                                      unsigned long long* out) {
  __shared__ uint16_t lut[kNumCodes];
  __shared__ unsigned long long hist[kOpenCopies * kGStride];
  for (int t = threadIdx.x; t < kNumCodes; t += blockDim.x) lut[t] = uint16_t(code_to_id3[kNumCodes - 1 - t] * 8u);
  for (int t = threadIdx.x; t < kOpenCopies * kGStride; t += blockDim.x) hist[t] = 0ull;
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  const int h = lane >> 5, c = lane & 31;
  unsigned long long* myhist = hist + (lane & (kOpenCopies - 1)) * kGStride;
  visit_graphs(
      I,
      [&](int g, const ItemRange& items) {
        int32_t i;
        int tile;
        while (next_item(items, lane, i, tile)) {
          const int64_t gb = G.gbase[i] - G.cap0, end = G.gbase[i + 1] - G.cap0;
          const int na = G.gna[i], nb = int(G.goff[i + 1] - G.goff[i]) - na, kb = tile * kMfmaCols;
          const uint32_t a = uint32_t(G.edge_ptr[i + 1] - G.edge_ptr[i]);
          const uint4* brec = G.rec + end - nb;
          const uint32_t* bcnt = G.cnt + end - nb;
          OpenColumns C = {};
          v8i b1[4], b2[4], b3[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int k = kb + 32 * q + c;
            const uint4 r = k < nb ? brec[k] : make_uint4(0, 0, 0, 0);
            b1[q] = col_fp4(h ? r.z : r.x);
            b2[q] = col_fp4(h ? r.x : r.w);
            b3[q] = col_fp4(h ? r.w : r.z);
          }
          if (kb + lane < nb) {
            const uint4 r = brec[kb + lane];
            C.c0.meta = r.y;
            C.c0.kn = cnt_all(bcnt[kb + lane]);
            C.m0 = r.x, C.l0 = r.z, C.h0 = r.w;
          }
          if (kb + kWave + lane < nb) {
            const uint4 r = brec[kb + kWave + lane];
            C.c1.meta = r.y;
            C.c1.kn = cnt_all(bcnt[kb + kWave + lane]);
            C.m1 = r.x, C.l1 = r.z, C.h1 = r.w;
          }
#pragma unroll 1
          for (int part = 0; part < 2; ++part)  // the groups above the centre, then the others before these columns
            open_rows<false>(part ? brec : G.rec + gb, part ? bcnt : G.cnt + gb, 0, part ? kb : na, kb, a, b1, b2, b3,
                             lane, C, lut, myhist);
          open_rows<true>(brec, bcnt, kb, min(nb, kb + kMfmaCols), kb, a, b1, b2, b3, lane, C, lut, myhist);
          open_end(C, a, lane, lut, myhist);
        }
      },
      [&](int g) { hist_flush<kOpenCopies>(hist, g, out); });
}

}  // namespace

void launch_sort_groups(int cus, const int32_t* rows, const unsigned long long* nrows, unsigned long long* queue,
                        const RowGroups& G, uint4* rec, uint32_t* cnt, int32_t* elig, hipStream_t s) {
  k_sort_groups<<<unsigned(cus), kSortThreads, 0, s>>>(rows, nrows, queue, G, rec, cnt, elig);
}

void launch_pairs_full(unsigned grid, const RowGroups& G, const WorkItems& I, const uint16_t* code_to_id3,
                       unsigned long long* hist, hipStream_t s) {
  k_pairs_full<<<grid, kPairWaves * kWave, 0, s>>>(G, I, code_to_id3, hist);
}

void launch_pairs_open(unsigned grid, const RowGroups& G, const WorkItems& I, const uint16_t* code_to_id3,
                       unsigned long long* hist, hipStream_t s) {
  k_pairs_open<<<grid, kPairWaves * kWave, 0, s>>>(G, I, code_to_id3, hist);
}
