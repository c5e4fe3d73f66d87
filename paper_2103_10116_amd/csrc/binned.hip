// binned.hip -- y = alpha*A*x + beta*y for irregular matrices in two
// streaming passes, with every random access served from LDS.
//
// A product that gathers x[col] for columns all over a long x is bound by
// the rate of random requests its CUs can keep in the L2 (226e9 gathers/s
// from a 2 MiB slice, 107e9/s from 8 MiB), not by bytes.  Here the entries
// are laid out over a grid of tiles, a tile being the entries of one column
// panel (as many columns as x values fit a CU's LDS) and one row bin
// (consecutive rows), ordered by row within the tile and cut into runs of
// kRun entries, one run a lane:
//   pass 1 (k_bin_mul) walks the tiles panel by panel.  A work-group loads
//     its panel's slice of x into LDS, streams its share of the panel's
//     entries (value and 16-bit column within the panel, the top bit set
//     where a partial sum ends), adds the products of a row within a run and
//     writes these partial sums, bin by bin, those that the lanes of a wave
//     finish in the same step side by side;
//   pass 2 (k_bin_sum) loads one bin's partial sums into LDS (contiguous),
//     picks each row's partials from there in column order by a 16-bit
//     index, adds them by per-lane runs and a segmented scan as the COO
//     kernel does, and writes the bin's rows (with their dot-product
//     partials when a solver asks for them).
// Bytes per entry: V + 2.5 read, and 2T + 2 per partial sum (a row's entries
// that fall into one run make one) against 12 to 16 with gathers, but all of
// them streamed.  No atomics on values: a row's sum has one order.
//
// Power-law rows, 2^20 columns, cold, us (column panels of the merge and COO
// kernels -> this): s = 1.79 (16.9M entries) FP64 129 -> 70, FP32 116 -> 47;
// s = 2.0 (6.4M) FP64 71 -> 41, FP32 49 -> 32.  Pass 1 takes 49 of the 70 us,
// pass 2 the other 21.
#include <algorithm>
#include <initializer_list>
#include <type_traits>
#include <utility>

#include "common.h"

namespace mxs {
namespace {

// x values of one panel: most of a CU's 160 KiB of LDS, and columns that
// leave the top bit of 16 free
constexpr int kSliceBytes = 163840 - 256;
template <typename T>
constexpr int kSlice = kSliceBytes / (int)sizeof(T) < 32768 ? kSliceBytes / (int)sizeof(T) : 32768;
// A run: consecutive entries of a tile added by one lane; 64 runs a chunk,
// one wave each.
constexpr int kRun = 8;
constexpr int kChunk = 64 * kRun;
constexpr int kMulThreads = 1024;
// A bin: kBinThreads threads add kBinRun partial sums each, so at most
// kBinParts of them; at most kBinRows non-empty rows and kBinEntries
// entries.  LDS of pass 2 in FP64: 32 KiB (row sums reuse it), four
// work-groups of 8 waves a CU (2^20 columns, s = 1.79: 70.8 us; 75.4 with 256
// threads, 72.7 with 768).
constexpr int kBinRun = 8;
constexpr int kBinThreads = 512;
constexpr int kBinParts = kBinThreads * kBinRun;  // 4096
constexpr int kBinRows = 1024;
constexpr int kBinEntries = 40960;
constexpr int kMinPanels = 32;
constexpr int kMaxPanels = 160;
constexpr uint16_t kTopBit = 0x8000;

// Panels of equal width whose slices fit LDS, as many as share the CUs out
// evenly where a panel gets two or more work-groups; above num_cus / 2 panels
// the fewest that fit.  At least kMinPanels: a work-group loads its whole
// slice, which on a short x would cost more than its entries (2^18 columns,
// s = 1.79: FP64 27.8 us with 13 panels, 20.5 with 32, 22.6 with 128).
int panel_count(int64_t ncols, size_t xb, int num_cus) {
  const int64_t w = xb == 8 ? kSlice<double> : kSlice<float>;
  const int64_t least = std::max<int64_t>(kMinPanels, (ncols + w - 1) / w);
  const int64_t share = num_cus / least;  // work-groups per panel
  return (int)(share > 1 ? std::max<int64_t>(least, num_cus / share) : least);
}

// most partial sums a row of L entries in at most P panels can make: one per
// run its entries of a panel touch (k_bin_bound counts the same row by row)
int64_t most_parts(int64_t L, int64_t P) {
  const int64_t s = std::min(L, P);
  return std::min(L, (7 * s + 3) / 4 + (L + 7) / 8);
}

// ---- set-up ----------------------------------------------------------------
// Upper bound of each row's partial sums, one wave a row: c entries in one
// panel touch at most 1 + (c + 6) / 8 runs (1 if c = 1).
__global__ __launch_bounds__(256) void k_bin_bound(int64_t n, int W,
                                                   const int32_t* __restrict__ rp,
                                                   const int32_t* __restrict__ col,
                                                   int32_t* __restrict__ bound) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += nw) {
    const int32_t s = rp[i], e = rp[i + 1];
    int starts = 0, single = 0;
    for (int32_t k0 = s; k0 < e; k0 += 64) {
      const int32_t k = k0 + lane;
      const bool on = k < e;
      const int p = on ? col[k] / W : -1;
      const bool first = on && (k == s || col[k - 1] / W != p);
      const bool last = on && (k + 1 == e || col[k + 1] / W != p);
      starts += __popcll(__ballot(first));
      single += __popcll(__ballot(first && last));
    }
    if (lane == 0) {
      const int multi = starts - single, left = e - s - single;
      bound[i] = single + (7 * multi + 3) / 4 + (left + 7) / 8;
    }
  }
}

// One wave lays out one bin, 64 entries in row order at a time.  An entry's
// place in its tile is the number of the tile's entries before it; a partial
// sum ends with a row's last entry in the tile and with each run.  E is the
// raw value word.
struct BinOut {
  uint16_t* acol;
  void* aval;
  int32_t* rbase;   // of each run: partial sums of all tiles before it, the top
                    // bit set for a tile's first run (k_bin_place finishes it)
  int32_t* rbin;    // of each run: the bin's first partial sum
  int32_t* order;   // of each partial sum's last entry: its index in perm, the
                    // top bit set for a row's first
  uint16_t* grank;
  int32_t* rowlist;
};

// WRITE: 0 counts the tiles' entries and partial sums, 1 writes everything,
// 2 the values alone.
template <typename E, int WRITE>
__global__ __launch_bounds__(64) void k_bin_layout(
    int P, int W, const int32_t* __restrict__ brow, const int32_t* __restrict__ bent,
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col, const E* __restrict__ val,
    int32_t* __restrict__ tile_a, int32_t* __restrict__ tile_b,
    const int32_t* __restrict__ bpart, const int32_t* __restrict__ brun,
    const int32_t* __restrict__ brank, BinOut out) {
  __shared__ int32_t ca[kMaxPanels], ce[kMaxPanels];
  __shared__ uint32_t starts[kBinEntries / 32];
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  const int32_t e0 = bent[b], len = bent[b + 1] - e0;
  const uint64_t lt = (uint64_t(1) << lane) - 1, le = lt | (uint64_t(1) << lane);
  int32_t* ta = tile_a + b * P;
  int32_t* tb = tile_b + b * P;
  for (int p = lane; p < P; p += 64) ca[p] = ce[p] = 0;
  for (int q = lane; q * 32 < len; q += 64) starts[q] = 0;
  __syncthreads();
  int rank = 0;
  for (int32_t r0 = brow[b]; r0 < brow[b + 1]; r0 += 64) {
    const int32_t i = r0 + lane;
    const bool on = i < brow[b + 1] && rp[i + 1] > rp[i];
    const uint64_t m = __ballot(on);
    if (on) {
      const int s = rp[i] - e0;
      atomicOr(&starts[s >> 5], 1u << (s & 31));
      if (WRITE == 1) out.rowlist[brank[b] + rank + __popcll(m & lt)] = i;
    }
    rank += __popcll(m);
  }
  __syncthreads();
  rank = -1;           // of the row that the last entry belongs to
  int parts = 0;       // partial sums so far, in row order
  bool has = false;    // the row at hand has a partial sum already
  constexpr int VPL = 16 / (int)sizeof(E);
  for (int k0 = 0; k0 < len; k0 += 64) {
    const int k = k0 + lane;
    const bool on = k < len;
    const int32_t c = on ? col[e0 + k] : 0;
    const int p = c / W;
    const bool start = on && ((starts[k >> 5] >> (k & 31)) & 1u);
    const bool row_end =
        on && (k + 1 == len || ((starts[(k + 1) >> 5] >> ((k + 1) & 31)) & 1u));
    const bool seg_end = on && (row_end || col[e0 + k + 1] / W != p);
    uint64_t same = __ballot(on);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t m = __ballot((p >> bit) & 1);
      same &= (p >> bit) & 1 ? m : ~m;
    }
    const int s = on ? ca[p] + __popcll(same & lt) : 0;
    const bool end = on && (seg_end || s % kRun == kRun - 1);
    const uint64_t eb = __ballot(end), sb = __ballot(start);
    const int q = on ? ce[p] + __popcll(same & lt & eb) : 0;
    const int j = parts + __popcll(eb & lt);
    if (WRITE && on) {
      const int64_t run = (int64_t)ta[p] + s / kRun;
      const int64_t chunk = run / 64, l = run % 64, t = s % kRun;
      reinterpret_cast<E*>(out.aval)[chunk * kChunk + t / VPL * (64 * VPL) + l * VPL + t % VPL] =
          val[e0 + k];
      if (WRITE == 1) {
        out.acol[run * kRun + t] = (uint16_t)(c - p * W) | (end ? kTopBit : 0);
        if (t == 0) {
          out.rbase[run] = (tb[p] + q) | (s == 0 ? INT32_MIN : 0);
          out.rbin[run] = bpart[b];
        }
        if (end) {
          const uint64_t mine = sb & le;  // row starts up to this lane
          const int from = mine ? 63 - __clzll(mine) : 0;
          const bool before =
              (eb & lt & ~((uint64_t(1) << from) - 1)) != 0 || (mine == 0 && has);
          out.order[run * kRun + t] = (brun[b] * kBinRun + j) | (before ? 0 : INT32_MIN);
          if (j % kBinRun == 0)
            out.grank[brun[b] + j / kBinRun] = (uint16_t)(rank + __popcll(sb & le));
        }
      }
    }
    __syncthreads();
    if (on && (same & lt) == 0) {
      ca[p] += __popcll(same);
      ce[p] += __popcll(same & eb);
    }
    __syncthreads();
    has = sb ? (eb >> (63 - __clzll(sb))) != 0 : has || eb != 0;
    rank += __popcll(sb);
    parts += __popcll(eb);
  }
  if (!WRITE)
    for (int p = lane; p < P; p += 64) {
      ta[p] = ca[p];
      tb[p] = ce[p];
    }
}

// The lanes of a chunk whose runs belong to one tile are a piece: r equal over
// the piece and different from its neighbours'.  Its lanes as a mask.
__device__ __forceinline__ uint64_t piece_of(bool first, int lane) {
  const uint64_t le = ~uint64_t(0) >> (63 - lane);
  const uint64_t bnd = __ballot(first || lane == 0);
  const int lo = 63 - __clzll(bnd & le);
  const uint64_t up = bnd & ~le;
  const uint64_t below = up ? (uint64_t(1) << (__ffsll((unsigned long long)up) - 1)) - 1
                            : ~uint64_t(0);
  return below & ~((uint64_t(1) << lo) - 1);
}

// One wave a chunk: the place of each partial sum among its bin's.  Those of
// a piece follow each other step by step (step j: entry j of every run), in
// lane order within a step, so that pass 1's stores are contiguous; rbase
// becomes the piece's first.
__global__ __launch_bounds__(64) void k_bin_place(const uint16_t* __restrict__ acol,
                                                  const int32_t* __restrict__ rbin,
                                                  const int32_t* __restrict__ order,
                                                  int32_t* __restrict__ rbase,
                                                  uint16_t* __restrict__ perm) {
  const int64_t run = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int lane = threadIdx.x;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  const int32_t r = rbase[run];
  const uint64_t piece = piece_of(r < 0, lane);
  const int32_t base = __shfl(r, __ffsll((unsigned long long)piece) - 1, 64) & INT32_MAX;
  const int32_t b0 = rbin[run];
  int32_t at = base;
  for (int j = 0; j < kRun; ++j) {
    const bool end = (acol[run * kRun + j] & kTopBit) != 0;
    const uint64_t m = __ballot(end) & piece;
    if (end) {
      const int32_t o = order[run * kRun + j];
      perm[o & INT32_MAX] = (uint16_t)(at + __popcll(m & lt) - b0) | (o < 0 ? kTopBit : 0);
    }
    at += __popcll(m);
  }
  rbase[run] = base;
}

// ---- pass 1 ----------------------------------------------------------------
// Bound by memory: a chunk's values come as 16-byte words, word w of all its
// lanes side by side; partial sums leave step by step so that the lanes of a
// piece write neighbours (55.5 -> 49.2 us on the s = 1.79 matrix against
// each lane writing its own run's sums one after the other).
template <typename V, typename T>
__global__ __launch_bounds__(kMulThreads) void k_bin_mul(
    const int4* __restrict__ work, const uint16_t* __restrict__ acol,
    const V* __restrict__ aval, const int32_t* __restrict__ rbase, const T* __restrict__ x, int W,
    int64_t ncols, int32_t base, T* __restrict__ prod, const int32_t* __restrict__ skip) {
  __shared__ T xs[kSlice<T>];
  if (skip && *skip) return;
  // panel, first and past-the-last chunk; neighbouring jobs (one panel's) on
  // one XCD, whose L2 then holds their slice of x
  const int4 job = work[xcd_remap(blockIdx.x, gridDim.x)];
  const int64_t c0 = (int64_t)job.x * W;
  const int m = (int)((ncols - c0) < W ? (ncols - c0) : W);
  const int t = threadIdx.x, lane = t & 63;
  constexpr int NW = kRun * (int)sizeof(V) / 16;
  constexpr int S = kMulThreads / 64;
  struct Load {
    uint4 v[NW];
    uint4 c;
    int32_t r;
  };
  const uint4* vw = reinterpret_cast<const uint4*>(aval);
  const uint4* cw = reinterpret_cast<const uint4*>(acol);
  const auto load = [&](int ch, Load& l) {
#pragma unroll
    for (int w = 0; w < NW; ++w) l.v[w] = vw[((int64_t)ch * NW + w) * 64 + lane];
    l.c = cw[(int64_t)ch * 64 + lane];
    l.r = rbase[(int64_t)ch * 64 + lane];
  };
  const auto use = [&](const Load& l) {
    V v[kRun];
    uint16_t c[kRun];
    __builtin_memcpy(v, l.v, sizeof(v));
    __builtin_memcpy(c, &l.c, sizeof(c));
    T g[kRun];
#pragma unroll
    for (int j = 0; j < kRun; ++j) g[j] = xs[c[j] & (kTopBit - 1)];
    const uint64_t piece = piece_of(__shfl_up(l.r, 1, 64) != l.r, lane);
    const uint64_t before = piece & ((uint64_t(1) << lane) - 1);
    int32_t at = l.r - base;
    T sum = 0;
#pragma unroll
    for (int j = 0; j < kRun; ++j) {
      sum += to_acc(v[j]) * g[j];
      const bool end = (c[j] & kTopBit) != 0;
      const uint64_t ends = __ballot(end);
      if (end) {
        prod[at + __popcll(ends & before)] = sum;
        sum = 0;
      }
      at += __popcll(ends & piece);
    }
  };
  int ch = job.y + __builtin_amdgcn_readfirstlane(t >> 6);
  // the wave's next chunk is always on its way, the first one while the slice
  // is loaded (two chunks ahead, or 8 waves with two ahead: no faster)
  Load next{};
  if (ch < job.z) load(ch, next);
  constexpr int U = 8;
  for (int i = t; i < m; i += U * kMulThreads) {
    T g[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * kMulThreads < m) g[u] = x[c0 + i + u * kMulThreads];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * kMulThreads < m) xs[i + u * kMulThreads] = g[u];
  }
  __syncthreads();
  for (; ch < job.z; ch += S) {
    const Load now = next;
    if (ch + S < job.z) load(ch + S, next);
    use(now);
  }
}

// ---- pass 2 ----------------------------------------------------------------
// Bound by the latency of a bin (loads, LDS, scan, stores, one after the
// other), which four work-groups a CU overlap.
// NV = 1: partials of w[i] * y[i] to dpart[b]; NV = 2: also of y[i]^2,
// interleaved; NV = 0: none.
template <typename T, bool SCALED, int NV>
__global__ __launch_bounds__(kBinThreads) void k_bin_sum(
    int64_t b0, const int32_t* __restrict__ bpart, const int32_t* __restrict__ blen,
    const int32_t* __restrict__ brun, const int32_t* __restrict__ brank, int32_t base,
    const uint16_t* __restrict__ perm, const uint16_t* __restrict__ grank,
    const int32_t* __restrict__ rowlist, const T* __restrict__ prod,
    const float* __restrict__ scale, T* __restrict__ y, T alpha, T beta,
    const int32_t* __restrict__ skip, const T* __restrict__ w, double* __restrict__ dpart) {
  constexpr int NW = kBinThreads / 64;
  constexpr int RPT = (kBinRows + kBinThreads - 1) / kBinThreads;
  __shared__ __align__(16) T pl[kBinParts];
  static_assert(kBinRows <= kBinParts, "row sums reuse the partials' LDS");
  T* rs = pl;
  __shared__ T cval[NW];
  __shared__ int crank[NW];
  if (skip && *skip) return;
  const int64_t b = b0 + blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int32_t g0 = bpart[b];
  const int len = blen[b];
  const int32_t q0 = brank[b];
  const int nr = brank[b + 1] - q0;
  const int k0 = t * kBinRun;
  const int m = len - k0 < 0 ? 0 : (len - k0 < kBinRun ? len - k0 : kBinRun);
  // everything this thread reads is asked for before anything is used: its
  // run's slots and the rank of its first row (runs are padded to whole
  // 16-byte words), its share of the partial sums, its rows
  uint16_t ix[kBinRun] = {};
  int r = 0;
  if (m > 0) {
    const uint4 u = *reinterpret_cast<const uint4*>(perm + ((int64_t)brun[b] * kBinRun + k0));
    __builtin_memcpy(ix, &u, sizeof(u));
    r = grank[brun[b] + t];
  }
  constexpr int PER = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(PER)));
  constexpr int NL = kBinParts / PER / kBinThreads;
  const vec* src = reinterpret_cast<const vec*>(prod + (g0 - base));
  const int words = (len + PER - 1) / PER;
  vec pw[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j)
    if (t + j * kBinThreads < words) pw[j] = src[t + j * kBinThreads];
  int32_t row[RPT];
#pragma unroll
  for (int j = 0; j < RPT; ++j)
    row[j] = t + j * kBinThreads < nr ? rowlist[q0 + t + j * kBinThreads] : -1;
#pragma unroll
  for (int j = 0; j < NL; ++j)
    if (t + j * kBinThreads < words) reinterpret_cast<vec*>(pl)[t + j * kBinThreads] = pw[j];
  __syncthreads();
  T pv[kBinRun];
#pragma unroll
  for (int j = 0; j < kBinRun; ++j) pv[j] = pl[ix[j] & (kTopBit - 1)];
  __syncthreads();  // the partials are all in registers
  // as in k_coo: rows inside the run are stored, its first and last rows are
  // joined with the neighbouring lanes' by a segmented scan; a row that
  // began in an earlier wave leaves its part in cval
  const int hrow = r;
  const bool hstart = (ix[0] & kTopBit) != 0;
  const int first = __shfl(hrow, 0, 64);
  const bool first_continues = __shfl((int)hstart, 0, 64) == 0;
  const int next_start = __shfl_down((int)hstart, 1, 64);
  const int next_m = __shfl_down(m, 1, 64);
  const auto emit = [&](int rr, T sum) {
    if (first_continues && rr == first)
      cval[wv] = sum;
    else
      rs[rr] = sum;
  };
  if (lane == 0) crank[wv] = m > 0 && first_continues ? first : -1;
  const bool active = m > 0;
  T vs = 0, hsum = 0, tsum = 0;
  int f = 1;
  bool multi = false, tend = false;
  if (active) {
    T sum = 0;
#pragma unroll
    for (int j = 0; j < kBinRun; ++j) {
      if (j < m) {
        if (j > 0 && (ix[j] & kTopBit)) {
          if (!multi) {
            hsum = sum;
            multi = true;
          } else {
            emit(r, sum);
          }
          ++r;
          sum = 0;
        }
        sum += pv[j];
      }
    }
    tsum = sum;
    tend = lane == 63 || next_m == 0 || next_start;
    if (!multi) hsum = sum;
    vs = tsum;
    f = (multi || hstart) ? 1 : 0;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T ov = __shfl_up(vs, d, 64);
    const int of = __shfl_up(f, d, 64);
    if (lane >= d) {
      if (!f) vs = ov + vs;
      f |= of;
    }
  }
  const T up = __shfl_up(vs, 1, 64);
  const T before = lane > 0 ? up : T(0);
  if (active) {
    if (multi) {
      emit(hrow, hstart ? hsum : before + hsum);
      if (tend) emit(r, tsum);
    } else if (tend) {
      emit(hrow, vs);
    }
  }
  __syncthreads();
  // rows cut between waves: the first wave that continues a row adds the
  // parts of all that do, in wave order
  if (t > 0 && t < NW && crank[t] >= 0 && crank[t - 1] != crank[t]) {
    T s = rs[crank[t]];
    for (int q = t; q < NW && crank[q] == crank[t]; ++q) s += cval[q];
    rs[crank[t]] = s;
  }
  __syncthreads();
  double d0 = 0.0, d1 = 0.0;
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const int32_t i = row[j];
    if (i >= 0) {
      T s = rs[t + j * kBinThreads];
      if (SCALED) s *= (T)scale[i];
      const T out = beta == T(0) ? alpha * s : alpha * s + beta * y[i];
      y[i] = out;
      if constexpr (NV > 0) d0 += (double)w[i] * (double)out;
      if constexpr (NV > 1) d1 += (double)out * (double)out;
    }
  }
  if constexpr (NV > 0) {
    __shared__ double red[2][NW];
    d0 = wave_total(d0);
    if constexpr (NV > 1) d1 = wave_total(d1);
    if (lane == 0) {
      red[0][wv] = d0;
      red[1][wv] = d1;
    }
    __syncthreads();
    if (t < NV) {
      double s = red[t][0];
#pragma unroll
      for (int q = 1; q < NW; ++q) s += red[t][q];
      dpart[b * NV + t] = s;
    }
  }
}

// Cuts `parts` (pointer, bytes) out of one allocation, 256-byte aligned.
using Parts = std::initializer_list<std::pair<void*, size_t>>;  // (T**, bytes)
void carve(void* base, Parts parts) {
  char* at = (char*)base;
  for (const auto& q : parts) {
    *(void**)q.first = at;
    at += (q.second + 255) & ~(size_t)255;
  }
}
size_t carved_bytes(Parts parts) {
  size_t b = 256;
  for (const auto& q : parts) b += (q.second + 255) & ~(size_t)255;
  return b;
}

template <typename T>
bool put(mxs_ctx* ctx, T* d, const std::vector<T>& h) {
  return hipMemcpyAsync(d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice, ctx->stream) ==
         hipSuccess;
}

// runs the layout kernel (write: see there) for values of vb bytes
void layout(mxs_ctx* ctx, const BinPart& B, int write, const int32_t* d_rp,
            const int32_t* d_col, const void* val, size_t vb, int32_t* rbin = nullptr,
            int32_t* order = nullptr) {
  const BinOut o{B.acol, B.aval, B.rbase, rbin, order, B.grank, B.rowlist};
  const auto go = [&](auto word, auto w) {
    using E = decltype(word);
    k_bin_layout<E, decltype(w)::value><<<(unsigned)B.nbins, 64, 0, ctx->stream>>>(
        B.panels, B.width, B.brow, B.bent, d_rp, d_col, (const E*)val, B.tile_a, B.tile_b,
        B.bpart, B.brun, B.brank, o);
  };
  const auto typed = [&](auto w) {
    if (vb == 8)
      go(uint64_t(), w);
    else if (vb == 4)
      go(uint32_t(), w);
    else
      go(uint16_t(), w);
  };
  if (write == 0)
    go(uint64_t(), std::integral_constant<int, 0>());
  else if (write == 1)
    typed(std::integral_constant<int, 1>());
  else
    typed(std::integral_constant<int, 2>());
}

}  // namespace

// Where the two passes beat the gathers.  Measured sides (us, gathers ->
// two passes, FP64 / FP32): power-law rows, s = 1.79, of 32768 columns and
// 0.54M entries 11.4 -> 10.0 / 10.8 -> 9.1, of 2^17 columns 21.5 -> 15.4 /
// 19.7 -> 12.1; below 2^19 entries both are launches (s = 2.0, 50000 columns,
// 0.3M entries 10.7 -> 9.9 / 10.3 -> 9.3) and the set-up costs more than it
// saves.  2^20 rows on 16384 columns, whose x the L1 still serves: 49.9 ->
// 53.3 / 33.3 -> 36.9 with 8 entries a row; on 32768: 52.7 -> 53.2 /
// 39.9 -> 37.8, even in FP64 there.  Also banded rows (24 entries within 20000
// columns of the diagonal, with one long row): 152 -> 88 / 116 -> 58.  The
// callers ask for a row of more than 64 entries besides: shorter rows gain too
// where their columns are scattered, but their set-up, several times that of
// the kernels over row blocks, has not been weighed.  At most kMaxPanels = 160
// panels (3271680 FP64 columns, 5242880 others): with 8 entries a row scattered
// over the columns 2617345 columns (129 panels) take 246 -> 201 / 182 -> 98
// (81 panels), 3271680 (160) 335 -> 269, in FP32 4194305 (129) 290 -> 236 and
// 5242880 (160) 360 -> 337, so more would gain nothing; and a row has to fit a
// bin.
bool bins_fit(const mxs_ctx* ctx, int64_t n, int64_t ncols, int64_t nnz, int64_t max_row,
              mxs_dtype dt) {
  constexpr int64_t kMinCols = 32768, kMinEntries = int64_t(1) << 19;
  if (dt != MXS_F64 && dt != MXS_F32 && dt != MXS_F16_ROWSCALED) return false;
  const size_t xb = dt == MXS_F64 ? 8 : 4;
  if (ncols < kMinCols || nnz < kMinEntries || nnz > INT32_MAX / 2) return false;
  const int P = panel_count(ncols, xb, ctx->num_cus);
  return P <= kMaxPanels && max_row <= kBinEntries && most_parts(max_row, P) <= kBinParts;
}

mxs_status build_bins(mxs_ctx* ctx, mxs_matrix* A, BinPart& B, int64_t n, int64_t ncols,
                      int64_t nnz, const std::vector<int32_t>& rp, const int32_t* d_rp,
                      const int32_t* d_col, const void* d_val, mxs_dtype dt) {
  A->copied = true;
  const size_t vb = value_bytes(dt), xb = dt == MXS_F64 ? 8 : 4;
  const int P = panel_count(ncols, xb, ctx->num_cus);
  const int W = (int)((ncols + P - 1) / P);
  int32_t* d_bound = (int32_t*)ctx->alloc.alloc((size_t)n * 4 + 4);
  void* d_tmp = nullptr;
  std::vector<int32_t> bound((size_t)n);
  mxs_status st = MXS_OK;
  do {
    if (!d_bound) {
      st = fail(ctx, MXS_OOM, "row bins");
      break;
    }
    k_bin_bound<<<(unsigned)std::min<int64_t>((n + 3) / 4, (int64_t)ctx->num_cus * 64), 256, 0,
                  ctx->stream>>>(n, W, d_rp, d_col, d_bound);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(bound.data(), d_bound, (size_t)n * 4, hipMemcpyDeviceToHost,
                       ctx->stream) != hipSuccess ||
        hipStreamSynchronize(ctx->stream) != hipSuccess) {
      st = fail(ctx, MXS_HIP, "row bins: counting failed");
      break;
    }
    // bins: consecutive rows while partial sums, entries and non-empty rows fit
    std::vector<int32_t> brow{0}, bent{0}, brank{0};
    int64_t nr = 0, np = 0;
    for (int64_t i = 0; i < n; ++i) {
      if (bound[(size_t)i] == 0) continue;
      if (nr == kBinRows || np + bound[(size_t)i] > kBinParts ||
          rp[(size_t)i + 1] - bent.back() > kBinEntries) {
        brow.push_back((int32_t)i);
        bent.push_back(rp[(size_t)i]);
        brank.push_back(brank.back() + (int32_t)nr);
        nr = np = 0;
      }
      ++nr;
      np += bound[(size_t)i];
    }
    brow.push_back((int32_t)n);
    bent.push_back((int32_t)nnz);
    brank.push_back(brank.back() + (int32_t)nr);
    const int64_t nb = (int64_t)bent.size() - 1;
    B.panels = P;
    B.width = W;
    B.ncols = ncols;
    const size_t nb4 = (size_t)nb * 4 + 4;
    const Parts first = {{&B.brow, nb4},  {&B.bent, nb4},  {&B.brank, nb4},
                         {&B.bpart, nb4}, {&B.blen, nb4},  {&B.brun, nb4},
                         {&B.tile_a, (size_t)nb * P * 4}, {&B.tile_b, (size_t)nb * P * 4},
                         {&B.rowlist, (size_t)brank.back() * 4}};
    void* mem = mat_alloc(A, carved_bytes(first));
    if (!mem) {
      st = fail(ctx, MXS_OOM, "row bins");
      break;
    }
    carve(mem, first);
    if (!put(ctx, B.brow, brow) || !put(ctx, B.bent, bent) || !put(ctx, B.brank, brank)) {
      st = fail(ctx, MXS_HIP, "row bins: copy failed");
      break;
    }
    // tiles counted on the GPU, placed on the host (P * nb of them)
    std::vector<int32_t> ta((size_t)nb * P), tb((size_t)nb * P), bpart((size_t)nb + 1),
        blen((size_t)nb), brun((size_t)nb + 1);
    B.nbins = nb;
    layout(ctx, B, 0, d_rp, d_col, d_val, vb);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(ta.data(), B.tile_a, ta.size() * 4, hipMemcpyDeviceToHost,
                       ctx->stream) != hipSuccess ||
        hipMemcpyAsync(tb.data(), B.tile_b, tb.size() * 4, hipMemcpyDeviceToHost,
                       ctx->stream) != hipSuccess ||
        hipStreamSynchronize(ctx->stream) != hipSuccess) {
      st = fail(ctx, MXS_HIP, "row bins: counting failed");
      break;
    }
    // partial sums by bin, then panel; a bin starts at a 16-byte boundary
    int64_t g = 0;
    for (int64_t b = 0; b < nb; ++b) {
      bpart[(size_t)b] = (int32_t)g;
      for (int p = 0; p < P; ++p) {
        const int32_t c = tb[(size_t)(b * P + p)];
        tb[(size_t)(b * P + p)] = (int32_t)g;
        g += c;
      }
      blen[(size_t)b] = (int32_t)(g - bpart[(size_t)b]);
      brun[(size_t)b + 1] = brun[(size_t)b] + (blen[(size_t)b] + kBinRun - 1) / kBinRun;
      g = (g + 3) / 4 * 4;
    }
    bpart[(size_t)nb] = (int32_t)g;
    B.parts = g;
    // batches of bins whose partial sums fit the fixed scratch
    const int64_t cap = (int64_t)(kNoAllocScratchBytes / xb);
    B.batch.assign(1, 0);
    for (int64_t b = 0; b < nb; ++b)
      if (bpart[(size_t)b + 1] - bpart[(size_t)B.batch.back()] > cap)
        B.batch.push_back((int32_t)b);
    B.batch.push_back((int32_t)nb);
    const size_t nbatch = B.batch.size() - 1;
    for (size_t q = 0; q < nbatch; ++q)
      B.least = std::max<int64_t>(B.least, bpart[(size_t)B.batch[q + 1]] -
                                               bpart[(size_t)B.batch[q]]);
    // pass 1's order: panel, batch, bin, each panel's share of a batch a whole
    // number of chunks; work lists of about equal shares, one work-group per
    // CU in all: list 0 takes all batches, the others one each
    std::vector<int4> work;
    B.work_at.clear();
    B.batch_base.clear();
    // (a work-group more than the CUs would wait for a whole round: one to
    // each panel, then one at a time to the panel whose share is largest)
    using Span = std::pair<int32_t, int32_t>;  // chunks of one panel
    const auto cut = [&](const std::vector<Span>& s) {
      B.work_at.push_back((int32_t)work.size());
      std::vector<int64_t> k((size_t)P, 0);
      using Share = std::pair<double, int>;
      std::vector<Share> heap;
      int64_t left = ctx->num_cus;
      for (int p = 0; p < P; ++p) {
        const int64_t c = s[(size_t)p].second - s[(size_t)p].first;
        if (c == 0) continue;
        k[(size_t)p] = 1;
        --left;
        heap.push_back({(double)c, p});
      }
      std::make_heap(heap.begin(), heap.end());
      for (; left > 0 && heap.front().first > 1.0; --left) {
        std::pop_heap(heap.begin(), heap.end());
        Share& h = heap.back();
        const int64_t c = s[(size_t)h.second].second - s[(size_t)h.second].first;
        h.first = (double)c / (double)++k[(size_t)h.second];
        std::push_heap(heap.begin(), heap.end());
      }
      for (int p = 0; p < P; ++p) {
        const int64_t f = s[(size_t)p].first, c = s[(size_t)p].second - f;
        for (int64_t q = 0; q < k[(size_t)p]; ++q)
          if (c * (q + 1) / k[(size_t)p] > c * q / k[(size_t)p])
            work.push_back(int4{p, (int)(f + c * q / k[(size_t)p]),
                                (int)(f + c * (q + 1) / k[(size_t)p]), 0});
      }
    };
    std::vector<std::vector<Span>> span(nbatch + 1, std::vector<Span>((size_t)P));
    g = 0;
    for (int p = 0; p < P; ++p) {
      span[0][(size_t)p].first = (int32_t)(g / 64);
      for (size_t q = 0; q < nbatch; ++q) {
        span[q + 1][(size_t)p].first = (int32_t)(g / 64);
        for (int64_t b = B.batch[q]; b < B.batch[q + 1]; ++b) {
          const int32_t c = ta[(size_t)(b * P + p)];
          ta[(size_t)(b * P + p)] = (int32_t)g;
          g += (c + kRun - 1) / kRun;
        }
        g = (g + 63) / 64 * 64;
        span[q + 1][(size_t)p].second = (int32_t)(g / 64);
      }
      span[0][(size_t)p].second = (int32_t)(g / 64);
    }
    for (size_t q = 0; q < (nbatch > 1 ? nbatch + 1 : 1); ++q) cut(span[q]);
    B.work_at.push_back((int32_t)work.size());
    for (size_t q = 0; q < nbatch; ++q) B.batch_base.push_back(bpart[(size_t)B.batch[q]]);
    const int64_t runs = g;
    if (runs * kRun > INT32_MAX) {
      st = fail(ctx, MXS_UNSUPPORTED, "row bins: sizes beyond int32 indices");
      break;
    }
    const size_t acol_b = (size_t)runs * kRun * 2, aval_b = (size_t)runs * kRun * vb,
                 rbase_b = (size_t)runs * 4, perm_b = (size_t)brun.back() * kBinRun * 2;
    const Parts second = {{&B.aval, aval_b}, {&B.acol, acol_b}, {&B.rbase, rbase_b},
                          {&B.perm, perm_b}, {&B.grank, (size_t)brun.back() * 2},
                          {&B.work, work.size() * sizeof(int4)}};
    int32_t *rbin = nullptr, *order = nullptr;
    const Parts tmp = {{&rbin, (size_t)runs * 4}, {&order, (size_t)runs * kRun * 4}};
    mem = mat_alloc(A, carved_bytes(second));
    d_tmp = ctx->alloc.alloc(carved_bytes(tmp));
    if (!mem || !d_tmp) {
      st = fail(ctx, MXS_OOM, "row bins");
      break;
    }
    carve(mem, second);
    carve(d_tmp, tmp);
    if (!put(ctx, B.work, work) || !put(ctx, B.bpart, bpart) || !put(ctx, B.blen, blen) ||
        !put(ctx, B.brun, brun) || !put(ctx, B.tile_a, ta) || !put(ctx, B.tile_b, tb) ||
        hipMemsetAsync(B.acol, 0, acol_b, ctx->stream) != hipSuccess ||
        hipMemsetAsync(B.aval, 0, aval_b, ctx->stream) != hipSuccess ||
        hipMemsetAsync(B.rbase, 0, rbase_b, ctx->stream) != hipSuccess ||
        hipMemsetAsync(B.perm, 0, perm_b, ctx->stream) != hipSuccess ||
        hipMemsetAsync(rbin, 0, (size_t)runs * 4, ctx->stream) != hipSuccess) {
      st = fail(ctx, MXS_HIP, "row bins: copy failed");
      break;
    }
    layout(ctx, B, 1, d_rp, d_col, d_val, vb, rbin, order);
    k_bin_place<<<(unsigned)(runs / 64), 64, 0, ctx->stream>>>(B.acol, rbin, order, B.rbase,
                                                               B.perm);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(ctx->stream) != hipSuccess)
      st = fail(ctx, MXS_HIP, "row bins: set-up failed");
  } while (0);
  (void)hipStreamSynchronize(ctx->stream);
  ctx->alloc.release(d_bound);
  ctx->alloc.release(d_tmp);
  return st;
}

// the current values laid out again
mxs_status refresh_bins(mxs_ctx* ctx, BinPart& B, const int32_t* d_rp, const int32_t* d_col,
                        const void* val, size_t vb) {
  layout(ctx, B, 2, d_rp, d_col, val, vb);
  MXS_HIP_TRY(ctx, hipGetLastError());
  return MXS_OK;
}

namespace {

template <typename V, typename T, bool SCALED>
void bins_typed(mxs_ctx* ctx, const BinPart& B, const float* scale, T alpha, const T* x, T beta,
                T* y, const int32_t* skip, T* prod, size_t prod_bytes, double* dpart, const T* w,
                int nv) {
  // every batch at once when the scratch holds all partial sums
  const bool whole = (size_t)B.parts * sizeof(T) <= prod_bytes;
  const size_t nbatch = B.batch.size() - 1;
  for (size_t q = 0; q < (whole ? 1 : nbatch); ++q) {
    const int32_t b0 = B.batch[q], nb = B.batch[whole ? nbatch : q + 1] - b0;
    const int32_t base = B.batch_base[q];
    const size_t list = whole ? 0 : q + 1;
    const int32_t w0 = B.work_at[list], nwork = B.work_at[list + 1] - w0;
    k_bin_mul<V, T><<<(unsigned)nwork, kMulThreads, 0, ctx->stream>>>(
        B.work + w0, B.acol, (const V*)B.aval, B.rbase, x, B.width, B.ncols, base, prod, skip);
    const auto sum = [&](auto nvc) {
      k_bin_sum<T, SCALED, decltype(nvc)::value><<<(unsigned)nb, kBinThreads, 0, ctx->stream>>>(
          b0, B.bpart, B.blen, B.brun, B.brank, base, B.perm, B.grank, B.rowlist, prod, scale, y,
          alpha, beta, skip, w, dpart);
    };
    if (nv == 2)
      sum(std::integral_constant<int, 2>());
    else if (nv == 1)
      sum(std::integral_constant<int, 1>());
    else
      sum(std::integral_constant<int, 0>());
  }
}

}  // namespace

void launch_bins(mxs_ctx* ctx, const BinPart& B, mxs_dtype dt, const float* scale,
                 const void* alpha, const void* x, const void* beta, void* y,
                 const int32_t* skip, void* prod, size_t prod_bytes, double* dpart,
                 const void* w, int nv) {
  if (dt == MXS_F64)
    bins_typed<double, double, false>(ctx, B, nullptr, *(const double*)alpha, (const double*)x,
                                      *(const double*)beta, (double*)y, skip, (double*)prod,
                                      prod_bytes, dpart, (const double*)w, nv);
  else if (dt == MXS_F32)
    bins_typed<float, float, false>(ctx, B, nullptr, *(const float*)alpha, (const float*)x,
                                    *(const float*)beta, (float*)y, skip, (float*)prod,
                                    prod_bytes, dpart, (const float*)w, nv);
  else
    bins_typed<_Float16, float, true>(ctx, B, scale, *(const float*)alpha, (const float*)x,
                                      *(const float*)beta, (float*)y, skip, (float*)prod,
                                      prod_bytes, dpart, (const float*)w, nv);
}

}  // namespace mxs
