// Tile binning and depth ordering.
//
// The order the renderer needs is, per tile segment, the instances sorted by
// (FP32 depth, Gaussian id).  Jobs of few (view, Gaussian) pairs count and
// fill the tile lists directly and sort each one in registers (the direct
// route below, plan_direct), all of it enqueued before the host has read the
// counts.  Large ones reach the order in two sorts that both use the same
// LDS-resident LSD radix sort (stable, 8- or 9-bit digits; per digit,
// per-partition counts, their scan, then LDS ranking and an LDS-staged
// scatter with those bases; partitions are laid out XCD by XCD, so each of
// the 8 L2s sees a contiguous range).  Both sorts run inside views: the
// elements of view v stay in a range of their own whose start is known
// before the sort, so the digits cover only what varies inside a view:
//   1. the depth keys of the V*n projected Gaussians (only the visible
//      pairs, gathered view by view), on the bits of the visible depth-bit
//      range (a first pass reduces that range together with the instance
//      count, which the host reads back); the key also carries the view
//      above those bits, in 32 bits when it fits, else in the high word of
//      a 64-bit key;
//   2. after emitting every Gaussian's tiles in that depth order (views in
//      order), the instances by their tile index inside the view, on the
//      bits of the largest view's tile count; the last pass turns tile
//      indices into segment ids.
// Stability of (2) keeps the depth order of (1) inside each segment, and
// stability of (1) keeps ascending ids for equal depths, so the result is
// the (segment, depth, id) order -- while the per-instance sort moves only
// ceil(log2(tiles per view)/9) digits of 32-bit keys instead of 5-7 digits
// of 64-bit keys.
#include <algorithm>
#include <cmath>

#include "gs_internal.h"

namespace gs {
namespace {

constexpr int kBlock = 256;
constexpr int kItems = 32;
constexpr int kPart = kBlock * kItems;  // keys per radix-sort partition
constexpr int kCountItems = 8;          // entries per thread in the instance count and scan
constexpr int kCountChunk = kBlock * kCountItems;

__device__ __forceinline__ uint64_t wave_ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

template <int BITS, typename K>
__device__ __forceinline__ uint32_t digit_of(K key, int shift) {
  return (uint32_t)(key >> shift) & ((1u << BITS) - 1u);
}

// Exclusive scan of one value per thread over a 256-thread block.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* s_wave,
                                                         uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t v = x;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(v, off, 64);
    if (lane >= off) v += y;
  }
  if (lane == 63) s_wave[wave] = v;
  __syncthreads();
  uint32_t pre = 0;
  for (int k = 0; k < wave; ++k) pre += s_wave[k];
  if (total) *total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
  __syncthreads();
  return pre + v - x;
}

// Exclusive scan of row[0, n) in place by one block, kIpt consecutive
// values per thread per round; returns the total (to every thread).
template <int kIpt = 16>
__device__ uint32_t block_scan_inplace(uint32_t* __restrict__ row, uint32_t n) {
  __shared__ uint32_t s_wave[4];
  uint32_t carry = 0;
  for (uint32_t b0 = 0; b0 < n; b0 += kBlock * kIpt) {
    const uint32_t e0 = b0 + threadIdx.x * kIpt;
    uint32_t x[kIpt], sum = 0;
#pragma unroll
    for (int i = 0; i < kIpt; ++i) {
      x[i] = e0 + i < n ? row[e0 + i] : 0u;
      sum += x[i];
    }
    uint32_t t;
    uint32_t run = carry + block_exclusive_scan(sum, s_wave, &t);
#pragma unroll
    for (int i = 0; i < kIpt; ++i) {
      if (e0 + i < n) row[e0 + i] = run;
      run += x[i];
    }
    carry += t;
  }
  return carry;
}

// ------------------------------------------------------------ radix sort
// Every sort here orders keys inside views: view v's elements occupy
// [start(v), start(v + 1)) of the array before and after the sort, with
// start(v) = vstart[v * vstride] for v < V and start(V) = n.  Each view's
// range is cut into partitions of at most kPart keys (none straddles two
// views), so the digits only cover the bits that vary inside a view.

__device__ __forceinline__ uint32_t view_start(const uint32_t* __restrict__ vstart,
                                               uint32_t vstride, int V, uint32_t n, int v) {
  return v < V ? vstart[(size_t)v * vstride] : n;
}

// First partition of each view, pfirst[v] (v < V), and the number of
// partitions, pfirst[V].  One block.
__global__ __launch_bounds__(kBlock) void k_part_first(const uint32_t* __restrict__ vstart,
                                                       uint32_t vstride, int V, uint32_t n,
                                                       uint32_t* __restrict__ pfirst) {
  __shared__ uint32_t s_wave[4];
  uint32_t carry = 0;
  for (int v0 = 0; v0 < V; v0 += kBlock) {
    const int v = v0 + (int)threadIdx.x;
    uint32_t np = 0;
    if (v < V) {
      const uint32_t len = view_start(vstart, vstride, V, n, v + 1) -
                           view_start(vstart, vstride, V, n, v);
      np = (len + kPart - 1) / kPart;
    }
    uint32_t tot;
    const uint32_t e = block_exclusive_scan(np, s_wave, &tot);
    if (v < V) pfirst[v] = carry + e;
    carry += tot;
  }
  if (threadIdx.x == 0) pfirst[V] = carry;
}

// Partition p's {view, first element, end, first partition of its view},
// one thread per partition.
__global__ __launch_bounds__(kBlock) void k_part_desc(const uint32_t* __restrict__ vstart,
                                                      uint32_t vstride, int V, uint32_t n,
                                                      const uint32_t* __restrict__ pfirst,
                                                      uint4* __restrict__ desc) {
  const uint32_t p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= pfirst[V]) return;
  int lo = 0, hi = V - 1;  // last view whose first partition is <= p
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pfirst[mid] <= p) lo = mid; else hi = mid - 1;
  }
  const uint32_t pf = pfirst[lo];
  const uint32_t b = view_start(vstart, vstride, V, n, lo) + (p - pf) * (uint32_t)kPart;
  const uint32_t e = view_start(vstart, vstride, V, n, lo + 1);
  desc[p] = make_uint4((uint32_t)lo, b, min(b + (uint32_t)kPart, e), pf);
}

// Partition table access.  With one view the table is not built: partition
// p is [p kPart, min((p + 1) kPart, n1)) of view 0 and there are
// ceil(n1 / kPart) of them (desc and pfirst are then NULL).
struct PartTable {
  const uint4* desc;
  const uint32_t* pfirst;  // V + 1 entries
  uint32_t n1;             // element count when desc is NULL
  int V;
  __device__ __forceinline__ uint32_t count() const {
    return desc ? pfirst[V] : (n1 + kPart - 1) / kPart;
  }
  __device__ __forceinline__ uint4 at(uint32_t p) const {
    if (desc) return desc[p];
    const uint32_t b = p * (uint32_t)kPart;
    return make_uint4(0u, b, min(b + (uint32_t)kPart, n1), 0u);
  }
  __device__ __forceinline__ uint32_t first_of_view(int v) const { return desc ? pfirst[v] : 0u; }
};

// XCD-aware partition of workgroup b: workgroup b runs on XCD b % 8, and
// each XCD takes a contiguous range of partitions, so one L2 merges the
// neighbouring words of the count rows and the adjacent output runs of a
// digit.
__device__ __forceinline__ uint32_t xcd_part(uint32_t pmax) {
  const uint32_t per = (pmax + 7) / 8;
  return (blockIdx.x & 7) * per + (blockIdx.x >> 3);
}

// Per-partition digit counts, digit-major: cnt[d * pmax + p].
template <typename K, int BITS>
__global__ __launch_bounds__(kBlock) void k_part_count(const K* __restrict__ keys, int shift,
                                                       uint32_t pmax, PartTable pt,
                                                       uint32_t* __restrict__ cnt) {
  constexpr int R = 1 << BITS;
  __shared__ uint32_t h[R];
  const uint32_t part = xcd_part(pmax);
  if (part >= pt.count()) return;
  for (int t = threadIdx.x; t < R; t += kBlock) h[t] = 0;
  __syncthreads();
  const uint4 ds = pt.at(part);
  K kk[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = ds.y + (uint32_t)j * kBlock + threadIdx.x;
    kk[j] = i < ds.z ? keys[i] : K(0);
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = ds.y + (uint32_t)j * kBlock + threadIdx.x;
    if (i < ds.z) atomicAdd(&h[digit_of<BITS>(kk[j], shift)], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < R; t += kBlock) cnt[(size_t)t * pmax + part] = h[t];
}

// Exclusive scan of each digit's row of partition counts over all
// partitions (one block per digit); the row total goes to tot[d].
__global__ __launch_bounds__(kBlock) void k_part_scan_rows(uint32_t* __restrict__ cnt,
                                                           uint32_t pmax, PartTable pt,
                                                           uint32_t* __restrict__ tot) {
  const uint32_t t = block_scan_inplace<16>(cnt + (size_t)blockIdx.x * pmax, pt.count());
  if (threadIdx.x == 0) tot[blockIdx.x] = t;
}

// One digit pass with bases from the scans: each wave ranks its keys stably
// by digit with ballots (lanes holding the same digit) and per-wave
// counters in LDS, the block scatters them through LDS into digit order,
// and the global writes come out as runs at (the view's digit start + this
// partition's prefix inside the view); the view's digit starts come from
// the scanned count rows at its first partition and the next view's.  No
// partition waits for another.
// With VALS the values move with the keys; without, the keys carry their
// value in the bits below `shift` of the first pass, and a pass given vout
// splits each key on the way out: value = key & umask to vout, key >> ushift
// to kout.  add (optional, last pass): add[view] is added to every key
// written.
template <typename K, int BITS, bool VALS>
__global__ __launch_bounds__(kBlock) void k_scatter_pass(
    const K* __restrict__ kin, const uint32_t* __restrict__ vin, K* __restrict__ kout,
    uint32_t* __restrict__ vout, int shift, uint32_t pmax, PartTable pt,
    const uint32_t* __restrict__ pbase, const uint32_t* __restrict__ tot,
    const uint32_t* __restrict__ add, int ushift,
    uint32_t umask) {
  constexpr int R = 1 << BITS, DPT = R / kBlock;
  __shared__ uint32_t s_wh[4][R];
  __shared__ uint32_t s_dstart[R];
  __shared__ uint32_t s_gbase[R];
  __shared__ uint32_t s_wave[4];
  __shared__ K s_k[kPart];
  __shared__ uint32_t s_v[VALS ? kPart : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t part = xcd_part(pmax);
  if (part >= pt.count()) return;
  const uint4 ds = pt.at(part);
  const uint32_t view = ds.x, end = ds.z, pf = ds.w;
  for (int t = tid; t < 4 * R; t += kBlock) (&s_wh[0][0])[t] = 0;
  __syncthreads();
  const uint32_t base = ds.y + (uint32_t)wave * 64u * kItems;
  K k[kItems];
  uint32_t val[kItems], rank[kItems], dig[kItems];
  const bool full = end - ds.y == (uint32_t)kPart;
  if (full) {
    const K* kb = kin + base + lane;
#pragma unroll
    for (int j = 0; j < kItems; ++j) k[j] = kb[j * 64];
    if constexpr (VALS) {
      const uint32_t* vb = vin + base + lane;
#pragma unroll
      for (int j = 0; j < kItems; ++j) val[j] = vb[j * 64];
    }
  } else {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const uint32_t idx = base + j * 64 + lane;
      k[j] = idx < end ? kin[idx] : K(0);
      if constexpr (VALS) val[j] = idx < end ? vin[idx] : 0u;
    }
  }
  const uint32_t lower_lo = lane >= 32 ? ~0u : ((1u << lane) - 1u);
  const uint32_t lower_hi = lane <= 32 ? 0u : (~0u >> (64 - lane));
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool valid = full || base + j * 64 + lane < end;
    const uint32_t d = valid ? digit_of<BITS>(k[j], shift) : 0u;
    const uint64_t vmask = wave_ballot(valid);
    uint32_t pl = (uint32_t)vmask, ph = (uint32_t)(vmask >> 32);
    const uint32_t nd = ~d;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const uint32_t flip = (uint32_t)((int32_t)(nd << (31 - b)) >> 31);
      const uint64_t bb = wave_ballot(flip == 0u);
      pl &= (uint32_t)bb ^ flip;
      ph &= (uint32_t)(bb >> 32) ^ flip;
    }
    const uint32_t below = (uint32_t)(__popc(pl & lower_lo) + __popc(ph & lower_hi));
    const uint32_t cnt = (uint32_t)(__popc(pl) + __popc(ph));
    uint32_t prev = 0;
    if (valid) prev = s_wh[wave][d];
    if (valid && below == cnt - 1) s_wh[wave][d] = prev + cnt;
    rank[j] = prev + below;
    dig[j] = d;
  }
  __syncthreads();
  {
    uint32_t run[DPT], tsum = 0;
#pragma unroll
    for (int i = 0; i < DPT; ++i) {
      const int d = tid * DPT + i;
      uint32_t r = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t c = s_wh[w][d];
        s_wh[w][d] = r;
        r += c;
      }
      run[i] = r;
      tsum += r;
    }
    uint32_t dstart = block_exclusive_scan(tsum, s_wave, nullptr);
    // the view's digit starts: its start plus the exclusive scan over the
    // digits of its counts, each the difference of the scanned row at the
    // view's first partition and at the next view's (the row total past
    // the last partition); formed here instead of by a launch of their own
    const uint32_t P = pt.count();
    const uint32_t pnext = pt.desc ? pt.first_of_view((int)view + 1) : P;
    const uint32_t vstart0 = ds.y - (part - pf) * (uint32_t)kPart;
    uint32_t tt[DPT], ts = 0;
#pragma unroll
    for (int i = 0; i < DPT; ++i) {
      const int d = tid * DPT + i;
      const uint32_t* row = pbase + (size_t)d * pmax;
      tt[i] = (pnext < P ? row[pnext] : tot[d]) - row[pf];
      ts += tt[i];
    }
    uint32_t g = vstart0 + block_exclusive_scan(ts, s_wave, nullptr);
#pragma unroll
    for (int i = 0; i < DPT; ++i) {
      const int d = tid * DPT + i;
      const uint32_t* row = pbase + (size_t)d * pmax;
      s_dstart[d] = dstart;
      s_gbase[d] = g + (row[part] - row[pf]) - dstart;
      dstart += run[i];
      g += tt[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if (base + j * 64 + lane < end) {
      const uint32_t lp = s_dstart[dig[j]] + s_wh[wave][dig[j]] + rank[j];
      s_k[lp] = k[j];
      if constexpr (VALS) s_v[lp] = val[j];
    }
  }
  __syncthreads();
  const uint32_t nvalid = end - ds.y;
  const K kadd = add ? (K)add[view] : K(0);
  if constexpr (VALS) {
    for (uint32_t t = tid; t < nvalid; t += kBlock) {
      const K kk = s_k[t];
      const uint32_t g = s_gbase[digit_of<BITS>(kk, shift)] + t;
      kout[g] = kk + kadd;
      vout[g] = s_v[t];
    }
  } else if (vout) {
    for (uint32_t t = tid; t < nvalid; t += kBlock) {
      const K kk = s_k[t];
      const uint32_t g = s_gbase[digit_of<BITS>(kk, shift)] + t;
      kout[g] = (kk >> ushift) + kadd;
      vout[g] = (uint32_t)kk & umask;
    }
  } else {
    for (uint32_t t = tid; t < nvalid; t += kBlock) {
      const K kk = s_k[t];
      kout[s_gbase[digit_of<BITS>(kk, shift)] + t] = kk + kadd;
    }
  }
}

// ------------------------------------------------------------ binning
// Per-view tile geometry from the device cameras, seg_base (V+1) and tx
// (V), one view per thread with a block scan.  One block.
__device__ __forceinline__ void view_info(const gs_camera* __restrict__ cams, int V,
                                          uint32_t* __restrict__ seg_base,
                                          int32_t* __restrict__ txv) {
  __shared__ uint32_t s_wave[4];
  uint32_t carry = 0;
  for (int v0 = 0; v0 < V; v0 += kBlock) {
    const int v = v0 + (int)threadIdx.x;
    uint32_t nt = 0;
    if (v < V) {
      const int tx = tiles_across(cams[v].width), ty = tiles_across(cams[v].height);
      txv[v] = tx;
      nt = (uint32_t)(tx * ty);
    }
    uint32_t tot;
    const uint32_t e = block_exclusive_scan(nt, s_wave, &tot);
    if (v < V) seg_base[v] = carry + e;
    carry += tot;
  }
  if (threadIdx.x == 0) seg_base[V] = carry;
}

// The tile counts and depth bits of Gaussians i0 .. i0 + kCountItems - 1
// of one view (0 past n): two 16-B loads per array when the rows are 16-B
// aligned and the run is whole, else one word at a time.
__device__ __forceinline__ void load_run(const int32_t* __restrict__ tv,
                                         const uint32_t* __restrict__ dv, uint32_t i0, int n,
                                         bool vec, uint32_t (&t)[kCountItems],
                                         uint32_t (&d)[kCountItems]) {
  static_assert(kCountItems == 8, "two 16-B loads per array");
  if (vec && i0 + kCountItems <= (uint32_t)n) {
    const int4 ta = *reinterpret_cast<const int4*>(tv + i0);
    const int4 tb = *reinterpret_cast<const int4*>(tv + i0 + 4);
    const uint4 da = *reinterpret_cast<const uint4*>(dv + i0);
    const uint4 db = *reinterpret_cast<const uint4*>(dv + i0 + 4);
    const int tt[8] = {ta.x, ta.y, ta.z, ta.w, tb.x, tb.y, tb.z, tb.w};
    const uint32_t dd[8] = {da.x, da.y, da.z, da.w, db.x, db.y, db.z, db.w};
#pragma unroll
    for (int j = 0; j < kCountItems; ++j) {
      t[j] = (uint32_t)max(tt[j], 0);
      d[j] = dd[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < kCountItems; ++j) {
      const uint32_t i = i0 + j;
      t[j] = i < (uint32_t)n ? (uint32_t)max(tv[i], 0) : 0u;
      d[j] = t[j] > 0 ? dv[i] : 0u;
    }
  }
}

__device__ __forceinline__ bool rows_aligned(int ld, const void* a, const void* b) {
  return (ld & 3) == 0 && ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0;
}

// Zeroes zero[0, zero_n) over the whole grid (the tile ranges, cleared here
// to save a launch of their own).
__device__ __forceinline__ void grid_zero(uint32_t* __restrict__ zero, size_t zero_n) {
  const size_t nthreads = (size_t)gridDim.x * gridDim.y * kBlock;
  for (size_t z = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kBlock + threadIdx.x;
       z < zero_n; z += nthreads)
    zero[z] = 0u;
}

// What the emission of one (view, Gaussian) pair needs: its first tile in
// the view, id, rectangle width | kSpanFlag, and the per-row spans or the
// bits of 1 / width.
__device__ __forceinline__ uint4 emit_entry(const uint32_t* __restrict__ record_tail, uint32_t id,
                                            uint32_t tiles_per_row) {
  const uint2 ow = *reinterpret_cast<const uint2*>(record_tail);  // origin, width | flag
  const uint32_t spans = record_tail[3];
  return make_uint4((ow.x >> 16) * tiles_per_row + (ow.x & 0xFFFFu), id, ow.y,
                    ow.y & kSpanFlag ? spans : __float_as_uint(1.f / (float)ow.y));
}

// Tile (in the view) of the pair's instance l: row by row over its spans or
// its rectangle.
__device__ __forceinline__ uint32_t entry_tile(const uint4& en, uint32_t tiles_per_row,
                                               uint32_t l) {
  uint32_t dy, dx;
  if (en.z & kSpanFlag) {
    // spans s_r = b_r - a_r per byte; instances before row r: p_r
    const uint32_t m = en.w;
    const uint32_t sp = ((m >> 4) & 0x0F0F0F0Fu) - (m & 0x0F0F0F0Fu);
    const uint32_t p1 = sp & 0xFFu, p2 = p1 + ((sp >> 8) & 0xFFu), p3 = p2 + ((sp >> 16) & 0xFFu);
    dy = (uint32_t)(l >= p1) + (uint32_t)(l >= p2) + (uint32_t)(l >= p3);
    const uint32_t before = dy == 0 ? 0u : (dy == 1 ? p1 : (dy == 2 ? p2 : p3));
    dx = ((m >> (8 * dy)) & 15u) + (l - before);
  } else {
    // l / width: a rectangle has at most 2^24 tiles, so the float quotient
    // is off by at most one
    dy = (uint32_t)((float)l * __uint_as_float(en.w));
    int32_t r = (int32_t)(l - dy * en.z);
    if (r < 0) {
      --dy;
      r += (int32_t)en.z;
    } else if (r >= (int32_t)en.z) {
      ++dy;
      r -= (int32_t)en.z;
    }
    dx = (uint32_t)r;
  }
  return en.x + dy * tiles_per_row + dx;
}

constexpr int kChunkTiles = 8192;  // most tiles of a view of the direct route: its LDS counters
constexpr uint32_t kDirectLongest = 4096;  // keys a sorting workgroup holds

// A sample of each view's Gaussians that tells, before the direct route spends
// anything on a job, whether some tile's list will be too long for its sort:
// then the job belongs to the radix sorts.  Two parts, each beside the work of
// a launch that is there anyway: the sampled pairs' tiles are written out, and
// added up per tile.  gs_bin_sort of crowded jobs in us, all instances counted
// before the route is left / with the sample / radix sorts from the start on:
// 60 k Gaussians at 64x64 135 / 125 / 120, 300 k in a few tiles of 1280x720
// 184 / 170 / 163, 1 M 246 / 220 / 207, 2 M 376 / 319 / 305 (what is left are
// the direct route's launches, which do nothing).  Jobs that stay pay 2-3 us.
// One pair in 64 because a list of 4,097 then has 64 +- 8 pairs in the sample;
// counters of all XCDs in memory in place of one workgroup's took 25-100 us.
// Lists of wide splats need no sample: they are as long as the job is large
// (kDirectCost).
constexpr uint32_t kSampleEvery = 64;     // of all views together one pair in as many,
constexpr uint32_t kSampleLeast = 2048, kSampleMost = 16384;  // within these
constexpr uint32_t kSampleMostTiles = 4;  // of a pair; wider ones spread over many lists
static_assert(kChunkTiles <= 1 << 13, "13 bits per tile of a sampled pair");

struct CrowdSample {
  uint32_t* tiles;    // per sampled pair: two tiles of 13 bits, their number (2 bits), weight
  uint32_t* leave;    // device flag: the job is left to the radix sorts
  bool direct;        // the job takes the direct route unless it is left
  uint32_t views, per_view;  // of the sample; none: no list can be too long
  uint32_t stride;      // Gaussians per sampled one
  uint32_t view_tiles;  // most tiles of a view
  uint32_t limit;       // weighted pairs of one tile from which on it is crowded
};

// Sample k: one Gaussian of stratum k % per_view of view k / per_view, and one
// or two of its tiles, at a random offset.
__device__ __forceinline__ void crowd_sample(const CrowdSample& cs, uint32_t k, int ld,
                                             const gs_camera* __restrict__ cams,
                                             const int32_t* __restrict__ tiles,
                                             const uint32_t* __restrict__ splat_words) {
  if (k >= cs.views * cs.per_view) return;
  const uint32_t v = k / cs.per_view, j = k - v * cs.per_view;
  const uint32_t h = k * 2654435761u;
  const uint32_t i = j * cs.stride + __umulhi(h, cs.stride);
  const size_t at = (size_t)v * ld + i;
  const uint32_t tx = (uint32_t)tiles_across(cams[v].width);
  const uint4 en = emit_entry(splat_words + at * (4 * kSplatF4) + 12, i, tx);
  const uint32_t nt = (uint32_t)max(tiles[at], 0);
  uint32_t out = 0;
  if (nt > 0 && nt <= kSampleMostTiles) {
    const uint32_t l0 = __umulhi(h * 747796405u, nt), l = l0 + nt / 2;
    out = entry_tile(en, tx, l0) & (kChunkTiles - 1);
    out |= (entry_tile(en, tx, l < nt ? l : l - nt) & (kChunkTiles - 1)) << 13;
    out |= min(nt, 2u) << 26 | max(nt / 2, 1u) << 28;
  }
  cs.tiles[k] = out;
}

// One workgroup adds up view v's sample.  The one thread that raises the flag
// tells the host, so nothing else of the call writes that word.
__device__ __forceinline__ void crowd_count(const CrowdSample& cs, uint32_t v,
                                            uint32_t* __restrict__ leave_host) {
  __shared__ uint4 s_four[kChunkTiles / 4];
  uint32_t* s_count = reinterpret_cast<uint32_t*>(s_four);
  const uint32_t fours = (cs.view_tiles + 3) / 4;
  const uint32_t* mine = cs.tiles + (size_t)v * cs.per_view;
  constexpr uint32_t kAhead = 24;
  uint32_t x[kAhead];
  auto load = [&](uint32_t j0) {
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u)
      x[u] = j0 + u * kBlock < cs.per_view ? mine[j0 + u * kBlock] : 0;
  };
  load(threadIdx.x);
  for (uint32_t t = threadIdx.x; t < fours; t += kBlock) s_four[t] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  for (uint32_t j0 = threadIdx.x; j0 < cs.per_view;) {
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) {
      const uint32_t m = (x[u] >> 26) & 3u, w = x[u] >> 28;
      if (m > 0) atomicAdd(&s_count[x[u] & (kChunkTiles - 1)], w);
      if (m > 1) atomicAdd(&s_count[(x[u] >> 13) & (kChunkTiles - 1)], w);
    }
    j0 += kAhead * kBlock;
    load(j0);
  }
  __syncthreads();
  uint32_t most = 0;
  for (uint32_t t = threadIdx.x; t < fours; t += kBlock) {
    const uint4 q = s_four[t];
    most = max(max(most, max(q.x, q.y)), max(q.z, q.w));
  }
  if (__syncthreads_or(most >= cs.limit) && threadIdx.x == 0 && atomicExch(cs.leave, 1u) == 0)
    tell_host(leave_host);
}

// Per chunk of kCountChunk Gaussians of one view (grid x; views on grid y,
// looping past 65535 of them), chunk c = v * gx + blockIdx.x: the
// range of the depth bits of its visible pairs and their instance count,
// part[c] = {min bits, max bits, count lo, count hi}, the number of its
// visible pairs, vis[c], and the count's low word again, icnt[c] (scanned,
// it places each view's instances).  Thread t owns Gaussians 8t .. 8t + 7.
// Workgroups past the chunks' gx columns take the sample.
__global__ __launch_bounds__(kBlock) void k_depth_range(int n, int ld, int V,
                                                        const uint32_t* __restrict__ depth_bits,
                                                        const int32_t* __restrict__ tiles,
                                                        uint4* __restrict__ part,
                                                        uint32_t* __restrict__ vis,
                                                        uint32_t* __restrict__ icnt,
                                                        uint32_t gx, CrowdSample cs,
                                                        const gs_camera* __restrict__ cams,
                                                        const uint32_t* __restrict__ splat_words) {
  __shared__ uint32_t s_min[4], s_max[4], s_cnt[4];
  __shared__ unsigned long long s_sum[4];
  if (blockIdx.x >= gx) {
    const uint32_t b = (blockIdx.x - gx) * gridDim.y + blockIdx.y;
    crowd_sample(cs, b * kBlock + threadIdx.x, ld, cams, tiles, splat_words);
    return;
  }
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *cs.leave = 0u;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool vec = rows_aligned(ld, tiles, depth_bits);
  for (int v = blockIdx.y; v < V; v += gridDim.y) {
    const int32_t* tv = tiles + (size_t)v * ld;
    const uint32_t* dv = depth_bits + (size_t)v * ld;
    const uint32_t i0 = blockIdx.x * (uint32_t)kCountChunk + threadIdx.x * kCountItems;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u, cnt = 0u;
    unsigned long long sum = 0;
    uint32_t t[kCountItems], d[kCountItems];
    load_run(tv, dv, i0, n, vec, t, d);
#pragma unroll
    for (int j = 0; j < kCountItems; ++j) {
      if (t[j] > 0) {
        mn = min(mn, d[j]);
        mx = max(mx, d[j]);
        sum += (unsigned long long)t[j];
        ++cnt;
      }
    }
    for (int off = 32; off >= 1; off >>= 1) {
      mn = min(mn, (uint32_t)__shfl_xor((int)mn, off, 64));
      mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
      sum += __shfl_xor(sum, off, 64);
      cnt += (uint32_t)__shfl_xor((int)cnt, off, 64);
    }
    if (lane == 0) {
      s_min[wave] = mn;
      s_max[wave] = mx;
      s_sum[wave] = sum;
      s_cnt[wave] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      mn = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
      mx = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
      sum = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
      const size_t c = (size_t)v * gx + blockIdx.x;
      part[c] = make_uint4(mn, mx, (uint32_t)sum, (uint32_t)(sum >> 32));
      vis[c] = (s_cnt[0] + s_cnt[1]) + (s_cnt[2] + s_cnt[3]);
      icnt[c] = (uint32_t)sum;
    }
    __syncthreads();
  }
}

// The direct route's time beyond what both routes take grows with the
// instances of its largest chunk, which one workgroup counts and fills (0.92
// ns each), and with all of them (10.5 ns per thousand more than the radix
// sorts).  A job is left where their sum, in the first's units, passes this:
// gs_bin_sort in us, direct / radix, of splats over tens to hundreds of tiles:
// 8 k Gaussians, 90 k instances in the largest chunk, 0.35 M in all 129 / 149;
// 188 k, 0.73 M 226 / 146; 2 k, 6.7 M, 6.7 M 6,340 / 300; 60 k, 80 k, 2.2 M
// 142 / 168; 93 k, 2.6 M 183 / 174; 200 k, 39 k, 3.6 M 149 / 176; 80 k, 7.5 M
// 270 / 218; 15.5 k, 4.4 M 185 / 218; 33 k, 9.4 M 326 / 267.
constexpr uint64_t kDirectCost = 105000, kDirectShare = 125;

// stats = {min bits, max bits, count lo, count hi} over the per-block
// partials of k_depth_range, by one block (device-wide atomics on three
// addresses from every block serialise at the memory side).  Thread 0 gets
// the job's cost on the direct route.
__device__ __forceinline__ uint32_t stats_reduce(const uint4* __restrict__ part, int nb,
                                                 uint32_t* __restrict__ stats) {
  __shared__ uint32_t s_min[4], s_max[4], s_big[4];
  __shared__ unsigned long long s_sum[4];
  uint32_t mn = 0xFFFFFFFFu, mx = 0u, big = 0u;
  unsigned long long sum = 0;
  for (int b = threadIdx.x; b < nb; b += kBlock) {
    const uint4 q = part[b];
    mn = min(mn, q.x);
    mx = max(mx, q.y);
    big = max(big, q.w ? 0xFFFFFFFFu : q.z);
    sum += (unsigned long long)q.z | ((unsigned long long)q.w << 32);
  }
  for (int off = 32; off >= 1; off >>= 1) {
    mn = min(mn, (uint32_t)__shfl_xor((int)mn, off, 64));
    mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
    big = max(big, (uint32_t)__shfl_xor((int)big, off, 64));
    sum += __shfl_xor(sum, off, 64);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    s_min[wave] = mn;
    s_max[wave] = mx;
    s_big[wave] = big;
    s_sum[wave] = sum;
  }
  __syncthreads();
  big = max(max(s_big[0], s_big[1]), max(s_big[2], s_big[3]));
  if (threadIdx.x == 0) {
    sum = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
    stats[0] = min(min(s_min[0], s_min[1]), min(s_min[2], s_min[3]));
    stats[1] = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
    stats[2] = (uint32_t)sum;
    stats[3] = (uint32_t)(sum >> 32);
  }
  return (uint32_t)min((unsigned long long)big + sum / kDirectShare, 0xFFFFFFFFull);
}

// Keys of the visible (view, Gaussian) pairs only, in (view, Gaussian)
// order: chunk c (as in k_depth_range) writes its visible pairs from
// chunk_off[c] on.  KeyOf(v, bits) gives the key; the value is the
// Gaussian id, with the pair's tile count above bit cpack when cpack >= 0.
template <typename K, typename KeyOf>
__device__ __forceinline__ void visible_keys(int n, int ld, int V,
                                             const uint32_t* __restrict__ depth_bits,
                                             const int32_t* __restrict__ tiles,
                                             const uint32_t* __restrict__ chunk_off, KeyOf key,
                                             int cpack, K* __restrict__ keys,
                                             uint32_t* __restrict__ vals) {
  __shared__ uint32_t s_wave[4];
  const bool vec = rows_aligned(ld, tiles, depth_bits);
  for (int v = blockIdx.y; v < V; v += gridDim.y) {
    const int32_t* tv = tiles + (size_t)v * ld;
    const uint32_t* dv = depth_bits + (size_t)v * ld;
    const uint32_t i0 = blockIdx.x * (uint32_t)kCountChunk + threadIdx.x * kCountItems;
    uint32_t c = 0, t[kCountItems], d[kCountItems];
    load_run(tv, dv, i0, n, vec, t, d);
#pragma unroll
    for (int j = 0; j < kCountItems; ++j) c += t[j] > 0 ? 1u : 0u;
    uint32_t r = chunk_off[(size_t)v * gridDim.x + blockIdx.x] +
                 block_exclusive_scan(c, s_wave, nullptr);
#pragma unroll
    for (int j = 0; j < kCountItems; ++j) {
      if (t[j] > 0) {
        keys[r] = key((uint32_t)v, d[j]);
        vals[r] = cpack >= 0 ? (i0 + j) | (t[j] << cpack) : i0 + j;
        ++r;
      }
    }
  }
}

// 32-bit (view, depth) keys when they fit: view << vshift | (bits - min
// bits), vshift the bits of the visible depth-bit range.
__global__ __launch_bounds__(kBlock) void k_depth_keys32(int n, int ld, int V,
                                                         const uint32_t* __restrict__ depth_bits,
                                                         const int32_t* __restrict__ tiles,
                                                         const uint32_t* __restrict__ chunk_off,
                                                         uint32_t dmin, uint32_t vshift,
                                                         int cpack,
                                                         uint32_t* __restrict__ keys,
                                                         uint32_t* __restrict__ vals,
                                                         uint32_t* __restrict__ zero,
                                                         size_t zero_n) {
  grid_zero(zero, zero_n);
  visible_keys<uint32_t>(
      n, ld, V, depth_bits, tiles, chunk_off,
      [=](uint32_t v, uint32_t d) { return (uint32_t)((uint64_t)v << vshift) | (d - dmin); },
      cpack, keys, vals);
}

// View of a depth-sorted key: the high word of a 64-bit key, the bits from
// vshift up of a 32-bit one.
__device__ __forceinline__ uint32_t view_of(uint64_t key, uint32_t) {
  return (uint32_t)(key >> 32);
}
__device__ __forceinline__ uint32_t view_of(uint32_t key, uint32_t vshift) {
  return (uint32_t)((uint64_t)key >> vshift);
}

// 64-bit (view << 32 | bits - min bits) keys otherwise.
__global__ __launch_bounds__(kBlock) void k_depth_keys(int n, int ld, int V,
                                                       const uint32_t* __restrict__ depth_bits,
                                                       const int32_t* __restrict__ tiles,
                                                       const uint32_t* __restrict__ chunk_off,
                                                       uint32_t dmin, int cpack,
                                                       uint64_t* __restrict__ keys,
                                                       uint32_t* __restrict__ vals,
                                                       uint32_t* __restrict__ zero,
                                                       size_t zero_n) {
  grid_zero(zero, zero_n);
  visible_keys<uint64_t>(
      n, ld, V, depth_bits, tiles, chunk_off,
      [=](uint32_t v, uint32_t d) { return ((uint64_t)v << 32) | (d - dmin); }, cpack, keys,
      vals);
}

// Instance count of each depth-sorted entry and the sums per block of
// kBlock entries: from the value's bits above cpack when the count travels
// there (cpack >= 0), else from tiles_touched (kept in cnt for the emit).
template <typename K>
__global__ __launch_bounds__(kBlock) void k_count_reduce(uint32_t N, int ld, uint32_t vshift,
                                                         const K* __restrict__ keys,
                                                         const uint32_t* __restrict__ vals,
                                                         const int32_t* __restrict__ tiles,
                                                         int cpack, uint32_t* __restrict__ cnt,
                                                         uint32_t* __restrict__ chunk_sums) {
  __shared__ uint32_t s_wave[4];
  const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
  uint32_t c = 0;
  if (e < N) {
    if (cpack >= 0) {
      c = vals[e] >> cpack;
    } else {
      const uint32_t v = view_of(keys[e], vshift);
      c = (uint32_t)tiles[(size_t)v * ld + vals[e]];
      cnt[e] = c;
    }
  }
  uint32_t tot;
  block_exclusive_scan(c, s_wave, &tot);
  if (threadIdx.x == 0) chunk_sums[blockIdx.x] = tot;
}

// Exclusive scan of sums[0, nb) in place (one block), 64 values per thread
// per round (one round up to 16,384 values); total to *total.
__global__ __launch_bounds__(kBlock) void k_chunk_scan(uint32_t* __restrict__ sums, uint32_t nb,
                                                       uint32_t* __restrict__ total) {
  const uint32_t t = block_scan_inplace<64>(sums, nb);
  if (threadIdx.x == 0) *total = t;
}

// The end of stage 1 in one launch: block 0 reduces the chunk partials
// into stats[0..3], blocks 1 and 2 scan the visible-pair and instance
// counts per chunk (totals to stats[4] and stats[5]), block 3 lays out the
// views' tiles, and the others, where there are some, add up the sample.
// stats is the context's pinned host memory: the totals need no copy of their
// own, and each of the first three blocks says when its own are there
// (kTotalsReady).
__global__ __launch_bounds__(kBlock) void k_stage1_close(
    const uint4* __restrict__ part, uint32_t* __restrict__ vis, uint32_t* __restrict__ icnt,
    uint32_t nchunk, uint32_t* __restrict__ stats, const gs_camera* __restrict__ cams, int V,
    uint32_t* __restrict__ seg_base, int32_t* __restrict__ txv, CrowdSample cs) {
  if (blockIdx.x > 3) {
    crowd_count(cs, blockIdx.x - 4, stats + kLeaveDirect);
    return;
  }
  if (blockIdx.x == 3) {
    view_info(cams, V, seg_base, txv);
    return;
  }
  if (blockIdx.x == 0) {
    const uint32_t cost = stats_reduce(part, (int)nchunk, stats);
    if (threadIdx.x == 0 && cs.direct && cost > kDirectCost && atomicExch(cs.leave, 1u) == 0)
      tell_host(stats + kLeaveDirect);
  } else {
    uint32_t* a = blockIdx.x == 1 ? vis : icnt;
    // 64 values per thread and round, or 4 where one round of them is enough
    const uint32_t t = nchunk <= 4 * kBlock ? block_scan_inplace<4>(a, nchunk)
                                            : block_scan_inplace<64>(a, nchunk);
    if (threadIdx.x == 0) stats[3 + blockIdx.x] = t;
  }
  if (threadIdx.x == 0) tell_host(stats + kTotalsReady + blockIdx.x);
}

// Emit (tile of the view, Gaussian id) for each tile of each depth-sorted
// entry, row by row over its tile rectangle, or over its per-row spans when
// the record carries them (the rectangle and spans come from the record's
// words 12, 13 and 15); optionally record where each (view, Gaussian)
// starts in this order.  A workgroup takes kBlock consecutive entries, whose
// instances form one contiguous output range, and spreads that range over
// all its threads, four consecutive instances (one 16-B store) at a time,
// so that large and small rectangles balance.  Entries come in depth order,
// so the nearest, largest ones sit together: where one workgroup's range is
// long, gridDim.y workgroups share it (each stages the entries, the first
// writes their bases).  Against 64 entries per wave, each instance found by
// its own search: one 1280x720 view 75 -> 19 us, twelve views 221 -> 106, 2 M
// Gaussians in 8 views 322 -> 181; the 20-view frame (32 M instances), whose
// views hold no large splats, 185 -> 178: what is left there is the random
// 64-B record each entry reads and writes.  It pays with traffic, there 789 ->
// 898 MB counted and 61 k -> 245 k waves, three of four workgroups finding
// nothing to share.  With pack >= 0 each instance is one word, tile << pack |
// id, in seg_out (id_out unused).
constexpr uint32_t kEmitShare = 8192;  // instances from which a range is shared

template <typename K>
__global__ __launch_bounds__(kBlock) void k_emit(uint32_t N, int ld, uint32_t vshift,
                                                 const K* __restrict__ keys,
                                                 const uint32_t* __restrict__ vals,
                                                 const uint32_t* __restrict__ cnt, int cpack,
                                                 const uint32_t* __restrict__ chunk_off,
                                                 const uint32_t* __restrict__ total_of,
                                                 const int32_t* __restrict__ txv,
                                                 uint32_t* __restrict__ seg_out,
                                                 uint32_t* __restrict__ id_out,
                                                 uint32_t* __restrict__ gv_base,
                                                 uint32_t* __restrict__ splat_words,
                                                 int pack) {
  __shared__ uint32_t s_pre[kBlock + 1];
  __shared__ uint4 s_ent[kBlock];  // emit_entry, and its view's tiles per row
  __shared__ uint32_t s_row[kBlock];
  __shared__ uint32_t s_bwave[4];
  const uint32_t base = chunk_off[blockIdx.x];
  const uint32_t end = blockIdx.x + 1 < gridDim.x ? chunk_off[blockIdx.x + 1] : *total_of;
  const uint32_t total = end - base;
  uint32_t part = blockIdx.y, parts = gridDim.y;
  if (total < kEmitShare) {
    if (part > 0) return;
    parts = 1;
  }
  const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
  uint32_t c = 0, g = 0;
  if (e < N) {
    const uint32_t w = vals[e];
    if (cpack >= 0) {
      c = w >> cpack;
      g = w & ((1u << cpack) - 1u);
    } else {
      c = cnt[e];
      g = w;
    }
  }
  const uint32_t pre = block_exclusive_scan(c, s_bwave, nullptr);
  s_pre[threadIdx.x] = pre;
  if (threadIdx.x == 0) s_pre[kBlock] = total;
  if (c > 0) {
    const uint32_t v = view_of(keys[e], vshift);
    uint32_t* rw = splat_words + ((size_t)v * ld + g) * (4 * kSplatF4) + 12;
    const uint32_t tx = (uint32_t)txv[v];
    s_ent[threadIdx.x] = emit_entry(rw, g, tx);
    s_row[threadIdx.x] = tx;
    if (part == 0) {
      if (gv_base) gv_base[(size_t)v * ld + g] = base + pre;
      // record word 14: this pair's first instance in emission order
      rw[2] = base + pre;
    }
  }
  __syncthreads();
  // groups of four instances at aligned output positions (id_out may be the
  // caller's list, aligned to its elements only)
  const bool ids_aligned = (reinterpret_cast<uintptr_t>(id_out) & 15) == 0;
  const uint32_t g_end = (end + 3) / 4;
  for (uint32_t gi = base / 4 + part * kBlock + threadIdx.x; gi < g_end; gi += parts * kBlock) {
    const uint32_t f_end = min(4 * gi + 4, end) - base;
    uint32_t f = 4 * gi >= base ? 4 * gi - base : 0u;
    uint32_t q = 0;  // last entry whose first instance is <= f (it has one)
#pragma unroll
    for (uint32_t step = kBlock / 2; step >= 1; step >>= 1)
      if (s_pre[q + step] <= f) q += step;
    uint32_t out[4], ids[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      // slot k holds instance 4 gi + k; those outside the range are skipped
      const uint32_t j = 4 * gi + (uint32_t)k;
      const bool in = j >= base && j - base < f_end;
      if (in) {
        f = j - base;
        if (f >= s_pre[q + 1]) ++q;  // every entry has an instance
        const uint4 en = s_ent[q];
        const uint32_t tile = entry_tile(en, s_row[q], f - s_pre[q]);
        out[k] = pack >= 0 ? (tile << pack) | en.y : tile;
        ids[k] = en.y;
      }
    }
    if (4 * gi >= base && 4 * gi + 4 <= end && (pack >= 0 || ids_aligned)) {
      *reinterpret_cast<uint4*>(seg_out + 4 * (size_t)gi) =
          make_uint4(out[0], out[1], out[2], out[3]);
      if (pack < 0)
        *reinterpret_cast<uint4*>(id_out + 4 * (size_t)gi) =
            make_uint4(ids[0], ids[1], ids[2], ids[3]);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t j = 4 * gi + (uint32_t)k;
        if (j >= base && j < end) {
          seg_out[j] = out[k];
          if (pack < 0) id_out[j] = ids[k];
        }
      }
    }
  }
}

// ------------------------------------------------ tile lists, direct route
// Every chunk of kCountChunk Gaussians of a view counts its instances per
// tile in LDS and writes that row; the rows are scanned down each tile's
// column and the column totals over the tiles; then each chunk writes its
// instances straight to their lists, and each list is sorted by (depth, id)
// in the registers of one workgroup.  Inside a chunk the order of a list's
// entries is left to LDS atomics; the sort's keys are distinct, so the
// result is the same list.  Against the two radix sorts these are 6 launches
// instead of 22, and two of them, not 17, after the host has read the
// instance count.
constexpr int kChunkThreads = 1024;
static_assert(kCountChunk == 2 * kChunkThreads, "two Gaussians per thread");

struct ChunkPairs {  // a chunk's pairs that have instances, in id order
  uint32_t pre[kCountChunk + 1];  // first instance of each
  uint4 ent[kCountChunk];
  uint32_t tile[kChunkTiles];     // counters or cursors
  uint32_t wave_n[kChunkThreads / 64], wave_c[kChunkThreads / 64];
};

// Stages chunk `chunk` of view v; returns its instance count and the number
// of pairs in `pairs`.  With `bases` each pair's first instance in (view,
// Gaussian) order, from `first` on, is written to its record (word 14) and
// to gv_base.
__device__ __forceinline__ uint32_t stage_chunk(ChunkPairs& sh, int v, uint32_t chunk, int n,
                                                int ld, const int32_t* __restrict__ tiles,
                                                uint32_t tx, bool bases, uint32_t first,
                                                uint32_t* __restrict__ splat_words,
                                                uint32_t* __restrict__ gv_base, uint32_t& pairs) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t i0 = chunk * (uint32_t)kCountChunk + 2 * threadIdx.x;
  const int32_t* tv = tiles + (size_t)v * ld;
  uint32_t c[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) c[k] = i0 + k < (uint32_t)n ? (uint32_t)max(tv[i0 + k], 0) : 0u;
  const uint32_t own_n = (c[0] > 0) + (c[1] > 0), own_c = c[0] + c[1];
  uint32_t in_n = own_n, in_c = own_c;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t yn = __shfl_up(in_n, off, 64), yc = __shfl_up(in_c, off, 64);
    if (lane >= off) {
      in_n += yn;
      in_c += yc;
    }
  }
  if (lane == 63) {
    sh.wave_n[wave] = in_n;
    sh.wave_c[wave] = in_c;
  }
  __syncthreads();
  uint32_t at_n = in_n - own_n, at_c = in_c - own_c, total = 0;
  pairs = 0;
  for (int w = 0; w < kChunkThreads / 64; ++w) {
    if (w < wave) {
      at_n += sh.wave_n[w];
      at_c += sh.wave_c[w];
    }
    pairs += sh.wave_n[w];
    total += sh.wave_c[w];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (c[k] > 0) {
      uint32_t* rw = splat_words + ((size_t)v * ld + i0 + k) * (4 * kSplatF4) + 12;
      sh.pre[at_n] = at_c;
      sh.ent[at_n] = emit_entry(rw, i0 + k, tx);
      if (bases) {
        rw[2] = first + at_c;
        if (gv_base) gv_base[(size_t)v * ld + i0 + k] = first + at_c;
      }
      ++at_n;
      at_c += c[k];
    }
  }
  if (threadIdx.x == 0) sh.pre[pairs] = total;
  return total;
}

// Calls at(tile, id) for every instance of the staged pairs, four
// consecutive ones per thread and search.
template <typename At>
__device__ __forceinline__ void each_instance(const ChunkPairs& sh, uint32_t pairs,
                                              uint32_t total, uint32_t tx, At at) {
  for (uint32_t f0 = 4 * threadIdx.x; f0 < total; f0 += 4 * kChunkThreads) {
    uint32_t q = 0;  // the pair of instance f0
#pragma unroll
    for (uint32_t step = kCountChunk / 2; step >= 1; step >>= 1)
      if (q + step < pairs && sh.pre[q + step] <= f0) q += step;
    uint32_t next = sh.pre[q + 1], base = sh.pre[q];
    uint4 en = sh.ent[q];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t f = f0 + k;
      if (f >= total) break;
      if (f >= next) {  // every staged pair has an instance
        ++q;
        base = next;
        next = sh.pre[q + 1];
        en = sh.ent[q];
      }
      at(entry_tile(en, tx, f - base), en.y);
    }
  }
}

// The chunk of a view that workgroup blockIdx.x takes.  Consecutive
// workgroups go to different XCDs: each XCD takes a contiguous range of the
// view's chunks, so that in k_tile_fill one L2 gathers the words that
// neighbouring chunks write side by side (20-view frame, 32 M instances: 494
// -> 300 us).
__device__ __forceinline__ uint32_t xcd_chunk() {
  const uint32_t xc = blockIdx.x & 7;
  return xc * (gridDim.x >> 3) + min(xc, gridDim.x & 7) + (blockIdx.x >> 3);
}

// rows[chunk of the view][tile]: instances per tile.  Grid: chunks by views.
// Nothing happens in a job that is left, here and in the two kernels behind.
__global__ __launch_bounds__(kChunkThreads) void k_tile_count(
    int n, int ld, int V, const int32_t* __restrict__ tiles, uint32_t* __restrict__ splat_words,
    const uint32_t* __restrict__ seg_base, const int32_t* __restrict__ txv,
    const uint32_t* __restrict__ leave, uint32_t* __restrict__ rows) {
  if (*leave != 0) return;
  __shared__ ChunkPairs sh;
  const uint32_t chunk = xcd_chunk();
  for (int v = blockIdx.y; v < V; v += gridDim.y) {
    const uint32_t sb = seg_base[v], nt = seg_base[v + 1] - sb, tx = (uint32_t)txv[v];
    for (uint32_t t = threadIdx.x; t < nt; t += kChunkThreads) sh.tile[t] = 0u;
    uint32_t pairs;
    const uint32_t total = stage_chunk(sh, v, chunk, n, ld, tiles, tx, false, 0u,
                                       splat_words, nullptr, pairs);
    __syncthreads();
    each_instance(sh, pairs, total, tx,
                  [&](uint32_t tile, uint32_t) { atomicAdd(&sh.tile[tile], 1u); });
    __syncthreads();
    uint32_t* row = rows + (size_t)gridDim.x * sb + (size_t)chunk * nt;
    for (uint32_t t = threadIdx.x; t < nt; t += kChunkThreads) row[t] = sh.tile[t];
    __syncthreads();
  }
}

// Exclusive scan of each tile's column of rows over the view's chunks, in
// place; the column total to counts[seg].  A workgroup takes 64 tiles, its
// 16 waves a sixteenth of the chunks each, kColumnRows of them with their
// loads in flight together (and only once where a wave has no more): 147
// chunks of 3,600 tiles 6.9 -> 5.0 us.
constexpr uint32_t kColumnRows = 16;

__global__ __launch_bounds__(1024) void k_tile_columns(int V, uint32_t nseg, uint32_t chunks,
                                                       const uint32_t* __restrict__ seg_base,
                                                       const uint32_t* __restrict__ leave,
                                                       uint32_t* __restrict__ rows,
                                                       uint32_t* __restrict__ counts) {
  if (*leave != 0) return;
  __shared__ uint32_t s_sum[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t seg = blockIdx.x * 64 + lane;
  const uint32_t per = (chunks + 15) / 16;
  const uint32_t k0 = min((uint32_t)wave * per, chunks), k1 = min(k0 + per, chunks);
  uint32_t* col = nullptr;
  uint32_t nt = 0, sum = 0, x[kColumnRows];
  auto load = [&](uint32_t kb) {
#pragma unroll
    for (uint32_t u = 0; u < kColumnRows; ++u)
      x[u] = kb + u < k1 ? col[(size_t)(kb + u) * nt] : 0u;
  };
  if (seg < nseg) {
    int lo = 0, hi = V - 1;  // last view whose base <= seg
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (seg_base[mid] <= seg) lo = mid; else hi = mid - 1;
    }
    const uint32_t sb = seg_base[lo];
    nt = seg_base[lo + 1] - sb;
    col = rows + (size_t)chunks * sb + (seg - sb);
    for (uint32_t kb = k0; kb < k1; kb += kColumnRows) {
      load(kb);
#pragma unroll
      for (uint32_t u = 0; u < kColumnRows; ++u) sum += x[u];
    }
  }
  s_sum[wave][lane] = sum;
  __syncthreads();
  uint32_t run = 0, total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w == wave) run = total;
    total += s_sum[w][lane];
  }
  if (seg < nseg) {
    for (uint32_t kb = k0; kb < k1; kb += kColumnRows) {
      if (per > kColumnRows) load(kb);
#pragma unroll
      for (uint32_t u = 0; u < kColumnRows; ++u) {
        if (kb + u < k1) col[(size_t)(kb + u) * nt] = run;
        run += x[u];
      }
    }
    if (wave == 0) counts[seg] = total;
  }
}

// Exclusive scan of the tile counts in place, in one workgroup, with their
// sum behind the last, and to *go whether the lists can be filled and sorted:
// at most `capacity` instances, no list above kDirectLongest.  The longest
// list goes to *longest in host memory, and then, when the host may read all
// that this and the kernels before it wrote there, 1 to *ready.
constexpr int kScanBlock = 1024;

__global__ __launch_bounds__(kScanBlock) void k_tile_scan(uint32_t* __restrict__ counts,
                                                          uint32_t nseg, uint64_t capacity,
                                                          const uint32_t* __restrict__ leave,
                                                          uint32_t* __restrict__ longest,
                                                          uint32_t* __restrict__ ready,
                                                          uint32_t* __restrict__ go) {
  if (*leave != 0) {  // the host knows and does not wait for this
    if (threadIdx.x == 0) *go = 0u;
    return;
  }
  __shared__ uint32_t s_wave[kScanBlock / 64], s_max[kScanBlock / 64];
  constexpr uint32_t kPer = 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0, most = 0;
  uint64_t all = 0;
  for (uint32_t b0 = 0; b0 < nseg; b0 += kScanBlock * kPer) {
    const uint32_t e0 = b0 + threadIdx.x * kPer;
    uint32_t x[kPer], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      x[k] = e0 + k < nseg ? counts[e0 + k] : 0u;
      sum += x[k];
      most = max(most, x[k]);
    }
    uint32_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(incl, off, 64);
      if (lane >= off) incl += y;
    }
    __syncthreads();
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t run = carry + incl - sum;
    for (int w = 0; w < kScanBlock / 64; ++w) {
      const uint32_t t = s_wave[w];
      if (w < wave) run += t;
      carry += t;
      all += t;
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      if (e0 + k < nseg) counts[e0 + k] = run;
      run += x[k];
    }
  }
  for (int off = 32; off >= 1; off >>= 1)
    most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
  if (lane == 0) s_max[wave] = most;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kScanBlock / 64; ++w) most = max(most, s_max[w]);
    counts[nseg] = carry;
    *longest = most;
    *go = all <= capacity && most <= kDirectLongest ? 1u : 0u;
    tell_host(ready);
  }
}

// Every instance's Gaussian id to its tile's list, from starts[seg] plus the
// chunk's place in the column on.  Writes the pairs' bases too.  Nothing
// happens without the scan's go-ahead.
__global__ __launch_bounds__(kChunkThreads) void k_tile_fill(
    int n, int ld, int V, const int32_t* __restrict__ tiles,
    const uint32_t* __restrict__ chunk_off, uint32_t* __restrict__ splat_words,
    const uint32_t* __restrict__ seg_base, const int32_t* __restrict__ txv,
    const uint32_t* __restrict__ rows, const uint32_t* __restrict__ starts,
    const uint32_t* __restrict__ go, uint32_t* __restrict__ vals,
    uint32_t* __restrict__ gv_base) {
  if (*go == 0) return;
  __shared__ ChunkPairs sh;
  const uint32_t chunk = xcd_chunk();
  for (int v = blockIdx.y; v < V; v += gridDim.y) {
    const uint32_t sb = seg_base[v], nt = seg_base[v + 1] - sb, tx = (uint32_t)txv[v];
    const uint32_t* row = rows + (size_t)gridDim.x * sb + (size_t)chunk * nt;
    for (uint32_t t = threadIdx.x; t < nt; t += kChunkThreads)
      sh.tile[t] = starts[sb + t] + row[t];
    uint32_t pairs;
    const uint32_t total = stage_chunk(sh, v, chunk, n, ld, tiles, tx, true,
                                       chunk_off[(size_t)v * gridDim.x + chunk],
                                       splat_words, gv_base, pairs);
    __syncthreads();
    each_instance(sh, pairs, total, tx, [&](uint32_t tile, uint32_t id) {
      vals[atomicAdd(&sh.tile[tile], 1u)] = id;
    });
    __syncthreads();
  }
}

// Sort keys: depth bits over id, read as a double.  The bits of a positive
// FP32 number below infinity are the high word of a positive double below
// infinity, so the doubles order as the (depth, id) pairs do, and one
// minimum and one maximum exchange a pair of keys.
__device__ __forceinline__ double list_key(uint32_t depth, uint32_t id) {
  return __hiloint2double((int)depth, (int)id);
}

// One instruction each: fmin and fmax would first quiet signalling NaNs,
// which no key is.
__device__ __forceinline__ double key_min(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double key_max(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  // quad permutes, half-row and row mirrors and the row rotation by 8 are
  // DPP moves; the others go through the LDS crossbar
  if constexpr (MASK == 1)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);
  else if constexpr (MASK == 2)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);
  else if constexpr (MASK == 3)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x1B, 0xF, 0xF, true);
  else if constexpr (MASK == 7)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true);
  else if constexpr (MASK == 8)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true);
  else if constexpr (MASK == 15)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true);
  else
    return (uint32_t)__shfl_xor((int)x, MASK, 64);
}

template <int MASK>
__device__ __forceinline__ double lane_xor(double x) {
  return __hiloint2double((int)lane_xor<MASK>((uint32_t)__double2hiint(x)),
                          (int)lane_xor<MASK>((uint32_t)__double2loint(x)));
}

// One step of the sorting network across threads: key r of a thread meets
// key r (REV: key E - 1 - r) of the thread whose index differs in MASK; the
// lower index keeps the smaller.  Masks of 64 and more exchange through LDS.
template <int E, int T, int MASK, bool REV>
__device__ __forceinline__ void cross_step(double (&k)[E], double* s_keys) {
  const int tid = threadIdx.x;
  const bool upper = (tid & (REV ? (MASK + 1) / 2 : MASK)) != 0;
  double p[E];
  if constexpr (MASK >= 64) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r) s_keys[r * T + tid] = k[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < E; ++r) p[r] = s_keys[(REV ? E - 1 - r : r) * T + (tid ^ MASK)];
  } else {
#pragma unroll
    for (int r = 0; r < E; ++r) p[r] = lane_xor<MASK>(k[REV ? E - 1 - r : r]);
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const double lo = key_min(k[r], p[r]), hi = key_max(k[r], p[r]);
    k[r] = upper ? hi : lo;
  }
}

template <int E, int T, int STRIDE>
__device__ __forceinline__ void merge_down(double (&k)[E], double* s_keys) {
  if constexpr (STRIDE >= E) {
    cross_step<E, T, STRIDE / E, false>(k, s_keys);
    merge_down<E, T, STRIDE / 2>(k, s_keys);
  } else if constexpr (STRIDE >= 1) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      if ((r & STRIDE) == 0) {
        const double a = k[r], b = k[r | STRIDE];
        k[r] = key_min(a, b);
        k[r | STRIDE] = key_max(a, b);
      }
    }
    merge_down<E, T, STRIDE / 2>(k, s_keys);
  }
}

// Bitonic sort of T * E keys, key r of thread t in place t * E + r, each
// merge starting with the mirrored step so that every exchange ascends.
template <int E, int T, int SIZE>
__device__ __forceinline__ void sort_up(double (&k)[E], double* s_keys) {
  if constexpr (SIZE <= T * E) {
    if constexpr (SIZE > E) {
      cross_step<E, T, SIZE / E - 1, true>(k, s_keys);
    } else {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int q = r ^ (SIZE - 1);
        if (r < q) {
          const double a = k[r], b = k[q];
          k[r] = key_min(a, b);
          k[q] = key_max(a, b);
        }
      }
    }
    merge_down<E, T, SIZE / 4>(k, s_keys);
    sort_up<E, T, SIZE * 2>(k, s_keys);
  }
}

template <int E, int T>
__device__ __forceinline__ void sort_list(uint32_t* __restrict__ list, uint32_t count,
                                          const uint32_t* __restrict__ depth,
                                          uint64_t* __restrict__ keys, uint32_t seg,
                                          double* s_keys) {
  double k[E];
  uint32_t id[E];
  // loaded strided (coalesced): the order before the sort does not matter
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t j = (uint32_t)r * T + threadIdx.x;
    id[r] = j < count ? list[j] : 0u;
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t j = (uint32_t)r * T + threadIdx.x;
    k[r] = j < count ? list_key(depth[id[r]], id[r]) : __builtin_inf();
  }
  sort_up<E, T, 2>(k, s_keys);
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t j = threadIdx.x * (uint32_t)E + r;
    if (j < count) {
      list[j] = (uint32_t)__double2loint(k[r]);
      if (keys) keys[j] = ((uint64_t)seg << 32) | (uint32_t)__double2hiint(k[r]);
    }
  }
}

// Sorts each tile's list by (depth, id) and writes its range (0, 0 for an
// empty one).  One workgroup of T threads per tile; lists longer than 16 T
// are left, and with LONG those that one wave sorts.
constexpr uint32_t kShortList = 16 * 64;

template <int T, bool LONG = false>
__global__ __launch_bounds__(T) void k_tile_sort(int V, int ld,
                                                 const uint32_t* __restrict__ starts,
                                                 const uint32_t* __restrict__ seg_base,
                                                 const uint32_t* __restrict__ depth_bits,
                                                 const uint32_t* __restrict__ go,
                                                 uint32_t* __restrict__ vals,
                                                 uint32_t* __restrict__ ranges,
                                                 uint64_t* __restrict__ keys) {
  __shared__ double s_keys[T > 64 ? 16 * T : 1];
  if (*go == 0) return;
  const uint32_t seg = blockIdx.x;
  const uint32_t start = starts[seg], end = starts[seg + 1];
  const uint32_t count = end - start;
  if (LONG && count <= kShortList) return;
  if (threadIdx.x == 0) {
    ranges[2 * (size_t)seg] = count > 0 ? start : 0u;
    ranges[2 * (size_t)seg + 1] = count > 0 ? end : 0u;
  }
  if (count == 0 || count > 16 * T) return;
  int lo = 0, hi = V - 1;  // last view whose base <= seg
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seg_base[mid] <= seg) lo = mid; else hi = mid - 1;
  }
  const uint32_t* depth = depth_bits + (size_t)lo * ld;
  uint32_t* list = vals + start;
  uint64_t* lk = keys ? keys + start : nullptr;
  if constexpr (!LONG) {
    if (count <= T) return sort_list<1, T>(list, count, depth, lk, seg, s_keys);
    if (count <= 2 * T) return sort_list<2, T>(list, count, depth, lk, seg, s_keys);
    if (count <= 4 * T) return sort_list<4, T>(list, count, depth, lk, seg, s_keys);
  }
  if (count <= 8 * T)
    sort_list<8, T>(list, count, depth, lk, seg, s_keys);
  else
    sort_list<16, T>(list, count, depth, lk, seg, s_keys);
}

// Segment boundaries of the sorted segment ids, four per thread (one 16-B
// load; the neighbours across the thread's group come from the adjacent
// lanes, or from memory at the wave's edges).
__global__ __launch_bounds__(kBlock) void k_ranges(uint32_t M, const uint32_t* __restrict__ seg,
                                                   uint32_t* __restrict__ ranges) {
  const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t j0 = 4 * t;
  const int lane = threadIdx.x & 63;
  uint32_t s[4] = {0u, 0u, 0u, 0u};
  if (j0 + 3 < M) {
    const uint4 q = *reinterpret_cast<const uint4*>(seg + j0);
    s[0] = q.x; s[1] = q.y; s[2] = q.z; s[3] = q.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (j0 + i < M) s[i] = seg[j0 + i];
  }
  uint32_t prev = (uint32_t)__shfl_up((int)s[3], 1, 64);
  uint32_t next = (uint32_t)__shfl_down((int)s[0], 1, 64);
  if (lane == 0 && j0 > 0 && j0 - 1 < M) prev = seg[j0 - 1];
  if (lane == 63 && j0 + 4 < M) next = seg[j0 + 4];
  if (j0 >= M) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t j = j0 + i;
    if (j >= M) break;
    const uint32_t before = i == 0 ? prev : s[i - 1];
    const uint32_t after = i == 3 ? next : s[i + 1];
    if (j == 0 || before != s[i]) ranges[2 * (size_t)s[i]] = j;
    if (j == M - 1 || after != s[i]) ranges[2 * (size_t)s[i] + 1] = j + 1;
  }
}

__global__ __launch_bounds__(kBlock) void k_keys64(uint32_t M, int V, int ld,
                                                   const uint32_t* __restrict__ seg,
                                                   const uint32_t* __restrict__ ids,
                                                   const uint32_t* __restrict__ seg_base,
                                                   const uint32_t* __restrict__ depth_bits,
                                                   uint64_t* __restrict__ keys) {
  const uint32_t j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= M) return;
  const uint32_t s = seg[j];
  int lo = 0, hi = V - 1;  // last view whose base <= s
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seg_base[mid] <= s) lo = mid; else hi = mid - 1;
  }
  keys[j] = ((uint64_t)s << 32) | depth_bits[(size_t)lo * ld + ids[j]];
}

__global__ void k_fill_u32(uint32_t* p, uint32_t value, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = value;
}

__global__ void k_fill_f32(float* p, float value, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = value;
}

// ------------------------------------------------------------ host side
inline int bits_for(uint64_t count) {  // bits to hold values 0 .. count-1
  int b = 0;
  while (b < 64 && ((uint64_t)1 << b) < count) ++b;
  return b;
}

// ---------------------------------------------------- usage keep-masks
// Ids beside the usage counts to be sorted (the sort overwrites its input).
__global__ __launch_bounds__(kBlock) void k_usage_pairs(const uint32_t* __restrict__ usage,
                                                        uint32_t n, uint32_t* __restrict__ key,
                                                        uint32_t* __restrict__ id) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  key[i] = usage[i];
  id[i] = i;
}

// rank[id] = position of id in the ordering.
__global__ __launch_bounds__(kBlock) void k_usage_rank(const uint32_t* __restrict__ order,
                                                       uint32_t n, uint32_t* __restrict__ rank) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) rank[order[i]] = i;
}

constexpr int kMaskLevels = 64;
struct MaskDrops {
  uint32_t d[kMaskLevels];
};

// masks[level][texel] = 1 where the texel's Gaussian ranks at or above the
// level's drop count, 0 below it and in the padding.  The ranks are read once
// for all levels of a launch, and the masks come out as whole lines: written
// straight from the ordering they would be scattered bytes.
__global__ __launch_bounds__(kBlock) void k_usage_masks(const uint32_t* __restrict__ rank,
                                                        uint32_t n, size_t texels, int levels,
                                                        MaskDrops drops,
                                                        uint8_t* __restrict__ masks) {
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= texels) return;
  const bool real = t < n;
  const uint32_t r = real ? rank[t] : 0u;
  for (int l = 0; l < levels; ++l) masks[(size_t)l * texels + t] = real && r >= drops.d[l];
}

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Fewest passes with digits of 8 or 9 bits (wider digits cost more per pass
// than they save).
struct DigitPlan {
  int passes;
  int bits;
};
inline DigitPlan plan_digits(int key_bits) {
  if (key_bits <= 0) return {0, 8};
  const int passes = (key_bits + 8) / 9;
  int b = (key_bits + passes - 1) / passes;
  if (b < 8) b = 8;
  return {passes, b};
}
inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

struct Layout {
  size_t dk0, dk1, dv0, dv1, cnt, chunks, segk0, segk1, segv_alt, pcount, dtotal,
      pfirst, pdesc, dparts, vparts, iparts, seg_base, txv, total, bytes;
};

// Bound on the partitions of n keys cut per view (at most one partial
// partition per view).
inline size_t max_parts(size_t n, int V) { return (size_t)cdiv(n, kPart) + (size_t)V; }

Layout make_layout(int V, int ld, int64_t cap, int64_t nseg) {
  (void)nseg;
  Layout L{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes);
    return at;
  };
  const size_t N = (size_t)V * (size_t)ld;
  const size_t pmax = max_parts(std::max(N, (size_t)cap), V);
  constexpr size_t kMaxDigits = 512;
  L.dk0 = take(N * 8);
  L.dk1 = take(N * 8);
  L.dv0 = take(N * 4);
  L.dv1 = take(N * 4);
  L.cnt = take(N * 4);
  L.chunks = take(((size_t)cdiv(N, kBlock) + 1) * 4);
  L.segk0 = take((size_t)cap * 4);
  L.segk1 = take((size_t)cap * 4);
  L.segv_alt = take((size_t)cap * 4);
  // per-partition digit counts of one pass (reused by every pass), the row
  // totals, the partition table
  L.pcount = take(kMaxDigits * pmax * 4);
  L.dtotal = take(kMaxDigits * 4);
  L.pfirst = take(((size_t)V + 1) * 4);
  L.pdesc = take(pmax * 16);
  L.seg_base = take(((size_t)V + 1) * 4);
  L.txv = take((size_t)V * 4);
  L.total = take(16);
  const size_t nchunk = (size_t)V * cdiv((uint64_t)ld, kCountChunk);
  L.dparts = take(nchunk * 16);
  L.vparts = take((nchunk + 1) * 4);
  L.iparts = take((nchunk + 1) * 4);
  L.bytes = o;
  return L;
}

template <typename T>
T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(ws) + off);
}

// Where each view's elements start: vstart[v * vstride] for v < V (the
// chunk scans of stage 1 with stride = chunks per view), n for v = V.
struct ViewStarts {
  const uint32_t* vstart;
  uint32_t vstride;
  int V;
};

// Stable LSD radix sort of (key, value) pairs inside each view on bits
// [shift0, shift0 + BITS * passes), ping-pong between buffer pair 0 and 1.
// First the partition table (none with one view), then per digit pass:
// per-partition digit counts, their exclusive scan per digit over the
// partitions, and the ranking + scatter, which forms its view's digit
// starts from the scanned counts.  Without values
// (v0 == NULL) the keys carry them in their low bits and the last pass
// splits them: key >> shift0 to the key buffer, key & (2^shift0 - 1) to
// vout_last.  add_last (optional): added per view to the keys the last pass
// writes.
struct SortSpec {
  int shift0;
  const uint32_t* add_last;
  uint32_t* vout_last;  // keys-only sorts
};

template <typename K, int BITS>
void radix_passes(K* k0, K* k1, uint32_t* v0, uint32_t* v1, uint32_t n, int passes,
                  const ViewStarts& vs, const SortSpec& sp, void* ws, const Layout& L,
                  hipStream_t s) {
  constexpr int R = 1 << BITS;
  uint32_t* cnt = at<uint32_t>(ws, L.pcount);
  uint32_t* tot = at<uint32_t>(ws, L.dtotal);
  uint32_t* pfirst = at<uint32_t>(ws, L.pfirst);
  uint4* desc = at<uint4>(ws, L.pdesc);
  // one view: partitions follow from their index, no table to build, and
  // the scatter scans the digit totals itself
  const bool one = vs.V == 1;
  const uint32_t pmax = one ? cdiv(n, kPart) : (uint32_t)max_parts(n, vs.V);
  const uint32_t grid = (pmax + 7) / 8 * 8;  // whole XCD rounds
  const PartTable pt{one ? nullptr : desc, one ? nullptr : pfirst, n, vs.V};
  if (!one) {
    hipLaunchKernelGGL(k_part_first, dim3(1), dim3(kBlock), 0, s, vs.vstart, vs.vstride, vs.V, n,
                       pfirst);
    hipLaunchKernelGGL(k_part_desc, dim3(cdiv(pmax, kBlock)), dim3(kBlock), 0, s, vs.vstart,
                       vs.vstride, vs.V, n, pfirst, desc);
  }
  K* kb[2] = {k0, k1};
  uint32_t* vb[2] = {v0, v1};
  const uint32_t umask = sp.shift0 >= 32 ? ~0u : ((1u << sp.shift0) - 1u);
  for (int p = 0; p < passes; ++p) {
    const int src = p & 1;
    const int shift = sp.shift0 + BITS * p;
    const bool last = p == passes - 1;
    hipLaunchKernelGGL((k_part_count<K, BITS>), dim3(grid), dim3(kBlock), 0, s, kb[src], shift,
                       pmax, pt, cnt);
    hipLaunchKernelGGL(k_part_scan_rows, dim3(R), dim3(kBlock), 0, s, cnt, pmax, pt, tot);
    const uint32_t* add = last ? sp.add_last : nullptr;
    if (v0)
      hipLaunchKernelGGL((k_scatter_pass<K, BITS, true>), dim3(grid), dim3(kBlock), 0, s,
                         kb[src], vb[src], kb[src ^ 1], vb[src ^ 1], shift, pmax, pt, cnt, tot,
                         add, 0, 0u);
    else
      hipLaunchKernelGGL((k_scatter_pass<K, BITS, false>), dim3(grid), dim3(kBlock), 0, s,
                         kb[src], nullptr, kb[src ^ 1], last ? sp.vout_last : nullptr, shift,
                         pmax, pt, cnt, tot, add, sp.shift0, umask);
  }
}

// Returns which key buffer holds the result (0 or 1).
template <typename K>
int radix_sort(K* k0, K* k1, uint32_t* v0, uint32_t* v1, uint32_t n, int bits,
               const ViewStarts& vs, const SortSpec& sp, void* ws, const Layout& L,
               hipStream_t s) {
  const DigitPlan dp = plan_digits(bits);
  if (n == 0 || dp.passes == 0) return 0;
  switch (dp.bits) {
    case 8: radix_passes<K, 8>(k0, k1, v0, v1, n, dp.passes, vs, sp, ws, L, s); break;
    default: radix_passes<K, 9>(k0, k1, v0, v1, n, dp.passes, vs, sp, ws, L, s); break;
  }
  return dp.passes & 1;
}

}  // namespace

void launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t s) {
  if (count <= 0) return;
  const int64_t want = (count + 255) / 256;
  const int blocks = (int)std::min<int64_t>(want, 4096);
  StageScope scope(kStFill, s);
  hipLaunchKernelGGL(k_fill_u32, dim3(blocks), dim3(256), 0, s, p, value, (size_t)count);
}

void launch_fill_f32(float* p, float value, int64_t count, hipStream_t s) {
  if (count <= 0) return;
  const int64_t want = (count + 255) / 256;
  const int blocks = (int)std::min<int64_t>(want, 4096);
  StageScope scope(kStFill, s);
  hipLaunchKernelGGL(k_fill_f32, dim3(blocks), dim3(256), 0, s, p, value, (size_t)count);
}

// Workspace of the keep-masks: two (usage, id) buffer pairs, the digit counts
// of one pass and the ranks, which take the place of the pair the sort leaves.
static Layout usage_layout(int n) {
  Layout L{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes);
    return at;
  };
  L.dk0 = take((size_t)n * 4);
  L.dk1 = take((size_t)n * 4);
  L.dv0 = take((size_t)n * 4);
  L.dv1 = take((size_t)n * 4);
  L.pcount = take((size_t)512 * std::max<size_t>(cdiv((uint64_t)n, kPart), 1) * 4);
  L.dtotal = take(512 * 4);
  L.bytes = o;
  return L;
}

size_t usage_masks_workspace_bytes(int n) { return usage_layout(n).bytes; }

hipError_t launch_usage_masks(const uint32_t* usage, int n, size_t texels, const int32_t* drops,
                              int levels, uint8_t* masks, void* ws, hipStream_t s) {
  if (levels == 0 || texels == 0) return hipSuccess;
  const Layout L = usage_layout(n);
  StageScope scope(kStCompact, s);
  uint32_t* k0 = at<uint32_t>(ws, L.dk0);
  uint32_t* v0 = at<uint32_t>(ws, L.dv0);
  uint32_t* v1 = at<uint32_t>(ws, L.dv1);
  const uint32_t blocks = cdiv((uint64_t)n, kBlock);
  if (n > 0) {
    hipLaunchKernelGGL(k_usage_pairs, dim3(blocks), dim3(kBlock), 0, s, usage, (uint32_t)n, k0,
                       v0);
    // equal usage keeps the order of the ids: the sort is stable
    const int which =
        radix_sort<uint32_t>(k0, at<uint32_t>(ws, L.dk1), v0, v1, (uint32_t)n, 32,
                             ViewStarts{nullptr, 0, 1}, SortSpec{0, nullptr, nullptr}, ws, L, s);
    hipLaunchKernelGGL(k_usage_rank, dim3(blocks), dim3(kBlock), 0, s, which ? v1 : v0,
                       (uint32_t)n, k0);
  }
  for (int l = 0; l < levels; l += kMaskLevels) {
    MaskDrops d{};
    const int count = std::min(kMaskLevels, levels - l);
    for (int k = 0; k < count; ++k) d.d[k] = (uint32_t)drops[l + k];
    hipLaunchKernelGGL(k_usage_masks, dim3(cdiv(texels, kBlock)), dim3(kBlock), 0, s, k0,
                       (uint32_t)n, texels, count, d, masks + (size_t)l * texels);
  }
  return hipGetLastError();
}

size_t bin_sort_workspace_bytes(int V, int ld, int64_t cap, int64_t nseg) {
  return make_layout(V, ld, cap, nseg).bytes;
}

namespace {
// The direct route's buffers, in the space of the radix sorts' keys, values
// and instances, which it leaves free: the tile counts (n_segments + 1) and
// the rows of counts, one per chunk of a view.
struct DirectPlan {
  bool possible;
  size_t counts, rows;
};
// Most (view, Gaussian) pairs of the direct route.  All of gs_bin_sort but its
// wait for the host, radix sorts -> direct, in us: 10 k pairs (16 k instances)
// 134 -> 50, 180 k (0.41 M) 190 -> 57, 300 k (1.1 M) 185 -> 78, 480 k (1.3 M)
// 204 -> 79, 1.2 M (6.4 M) 283 -> 204, 1.8 M (9.6 M) 327 -> 271, 3 M (16 M)
// 425 -> 428, 6 M (32 M) 704 -> 851: its lists are written word by word, the
// radix passes write runs.
constexpr int64_t kDirectPairs = 3000000;

// Sampled pairs of one tile from which on a job counts as crowded, with
// `sampled` of a view's n Gaussians: those of a list above kDirectLongest,
// less two standard deviations (none where every Gaussian is sampled).
uint32_t crowd_limit(uint32_t sampled, uint32_t n) {
  const double f = (double)sampled / (double)n, mean = f * (kDirectLongest + 1);
  return std::max(1u, (uint32_t)std::ceil(mean - 2.0 * std::sqrt(mean * (1.0 - f))));
}

DirectPlan plan_direct(const BinSortPlan& p, const Layout& L) {
  DirectPlan d{};
  const int64_t chunks = cdiv((uint64_t)p.n, kCountChunk);
  d.counts = L.dk0;
  d.rows = d.counts + align_up(((size_t)p.n_segments + 1) * 4);
  d.possible = (int64_t)p.n_views * p.n <= kDirectPairs && p.max_tiles <= kChunkTiles &&
               d.rows + (size_t)chunks * (size_t)p.n_segments * 4 <= L.pcount;
  return d;
}
}  // namespace

hipError_t bin_sort_stage1(const BinSortPlan& p, const gs_projected& proj,
                           const gs_camera* cams_dev, void* ws, uint32_t* stats, hipStream_t s) {
  const Layout L = make_layout(p.n_views, p.ld, p.capacity, p.n_segments);
  StageScope scope(kStDepthSort, s);
  // chunks of kCountChunk Gaussians per view; views on grid rows (beyond
  // 65535 they loop)
  const uint32_t gx = cdiv((uint64_t)p.n, kCountChunk);
  const uint32_t gy = std::min<uint32_t>((uint32_t)p.n_views, 65535u);
  const uint32_t nchunk = gx * (uint32_t)p.n_views;
  uint4* part = at<uint4>(ws, L.dparts);
  uint32_t* vis = at<uint32_t>(ws, L.vparts);
  uint32_t* icnt = at<uint32_t>(ws, L.iparts);
  const DirectPlan d = plan_direct(p, L);
  const uint32_t nseg = (uint32_t)p.n_segments;
  uint32_t* leave = at<uint32_t>(ws, L.total) + 1;
  CrowdSample cs{};
  cs.leave = leave;
  cs.direct = d.possible;
  uint32_t sample_blocks = 0;
  if (d.possible && p.n > (int)kDirectLongest) {  // else no list can be longer
    // in the place of the rows of counts, which come later: at most 4 of the
    // 28 bytes that the workspace has per pair up to there
    cs.tiles = at<uint32_t>(ws, d.rows);
    cs.views = (uint32_t)p.n_views;
    const uint32_t pairs = std::min(
        std::max(cs.views * (uint32_t)p.n / kSampleEvery, kSampleLeast), kSampleMost);
    cs.stride = cdiv((uint64_t)cs.views * (uint64_t)p.n, pairs);
    cs.per_view = (uint32_t)p.n / cs.stride;
    cs.view_tiles = (uint32_t)p.max_tiles;
    cs.limit = crowd_limit(cs.per_view, (uint32_t)p.n);
    sample_blocks = cdiv((uint64_t)cs.views * cs.per_view, kBlock);
  }
  hipLaunchKernelGGL(k_depth_range, dim3(gx + cdiv(sample_blocks, gy), gy), dim3(kBlock), 0, s,
                     p.n, p.ld, p.n_views, proj.depth_bits, proj.tiles_touched, part, vis, icnt,
                     gx, cs, cams_dev, reinterpret_cast<const uint32_t*>(proj.splat));
  // the depth-bit range and instance count (stats[0..3]); where each
  // chunk's visible pairs go in the depth sort's input (stats[4] = their
  // number), and where each chunk's instances start in emission order,
  // which keeps the views in order (only read once the host has checked
  // that the total fits 32 bits)
  hipLaunchKernelGGL(k_stage1_close, dim3(4 + cs.views), dim3(kBlock), 0, s, part, vis, icnt,
                     nchunk, stats, cams_dev, p.n_views, at<uint32_t>(ws, L.seg_base),
                     at<int32_t>(ws, L.txv), cs);
  if (d.possible) {
    // the tile counts do not wait for the host
    uint32_t* counts = at<uint32_t>(ws, d.counts);
    uint32_t* rows = at<uint32_t>(ws, d.rows);
    hipLaunchKernelGGL(k_tile_count, dim3(gx, gy), dim3(kChunkThreads), 0, s, p.n, p.ld,
                       p.n_views, proj.tiles_touched, reinterpret_cast<uint32_t*>(proj.splat),
                       at<uint32_t>(ws, L.seg_base), at<int32_t>(ws, L.txv), leave, rows);
    hipLaunchKernelGGL(k_tile_columns, dim3(cdiv(nseg, 64u)), dim3(1024), 0, s, p.n_views, nseg,
                       gx, at<uint32_t>(ws, L.seg_base), leave, rows, counts);
    hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(kScanBlock), 0, s, counts, nseg,
                       (uint64_t)p.capacity, leave, stats + kLongest, stats + kCountsReady,
                       at<uint32_t>(ws, L.total));
  }
  return hipGetLastError();
}

namespace {
// Depth sort of the (view, Gaussian) pairs with keys K inside each view on
// their dbits low bits, instance offsets and emission into (segk0, v0), or
// packed into segk0 alone with pack >= 0; vshift is where a 32-bit key's
// view starts; with cpack >= 0 each pair's tile count rides above bit
// cpack of its value through the sort.  The key gather also clears
// ranges[0, 2 n_segments).
template <typename K>
void depth_count_emit(const BinSortPlan& p, const gs_projected& proj, const Layout& L, void* ws,
                      uint32_t N, uint32_t dmin, uint32_t vshift, int dbits, int cpack,
                      uint32_t* segk0, uint32_t* v0, int pack, uint32_t* gv_base,
                      uint32_t* ranges, hipStream_t s) {
  K* k0 = at<K>(ws, L.dk0);
  K* k1 = at<K>(ws, L.dk1);
  uint32_t* dv0 = at<uint32_t>(ws, L.dv0);
  uint32_t* dv1 = at<uint32_t>(ws, L.dv1);
  int which;
  {
    StageScope scope(kStDepthSort, s);
    // keys of the visible pairs only (the chunk offsets from stage 1)
    const dim3 key_grid(cdiv((uint64_t)p.n, kCountChunk),
                        std::min<uint32_t>((uint32_t)p.n_views, 65535u));
    const uint32_t* vis_off = at<uint32_t>(ws, L.vparts);
    if constexpr (sizeof(K) == 4)
      hipLaunchKernelGGL(k_depth_keys32, key_grid, dim3(kBlock), 0, s, p.n, p.ld, p.n_views,
                         proj.depth_bits, proj.tiles_touched, vis_off, dmin, vshift, cpack, k0,
                         dv0, ranges, (size_t)2 * (size_t)p.n_segments);
    else
      hipLaunchKernelGGL(k_depth_keys, key_grid, dim3(kBlock), 0, s, p.n, p.ld, p.n_views,
                         proj.depth_bits, proj.tiles_touched, vis_off, dmin, cpack, k0, dv0,
                         ranges, (size_t)2 * (size_t)p.n_segments);
    const ViewStarts vs{vis_off, key_grid.x, p.n_views};
    which = radix_sort<K>(k0, k1, dv0, dv1, N, dbits, vs, SortSpec{0, nullptr, nullptr}, ws, L,
                          s);
  }
  const K* sk = which ? k1 : k0;
  const uint32_t* sv = which ? dv1 : dv0;
  uint32_t* cnt = at<uint32_t>(ws, L.cnt);
  uint32_t* chunks = at<uint32_t>(ws, L.chunks);
  const uint32_t nch = cdiv(N, kBlock);
  {
    // instance counts per block of kBlock entries and their scan; the emit
    // finishes the offsets inside its block
    StageScope scope(kStCountScan, s);
    hipLaunchKernelGGL((k_count_reduce<K>), dim3(nch), dim3(kBlock), 0, s, N, p.ld, vshift, sk,
                       sv, proj.tiles_touched, cpack, cnt, chunks);
    hipLaunchKernelGGL(k_chunk_scan, dim3(1), dim3(kBlock), 0, s, chunks, nch,
                       at<uint32_t>(ws, L.total));
  }
  StageScope scope(kStEmit, s);
  // workgroups that may share one range, in us for 1 / 4 / 8: 0.8 k
  // workgroups (one 1280x720 view) 42 / 21 / 19, 9 k (twelve views) 141 / 106
  // / 101, 22 k (2 M Gaussians, 8 views) 220 / 181 / 177; 34 k (44 views) 215
  // / 222 / 235: there the shared ranges hide behind the others and the
  // workgroups that find nothing to share cost more than they give
  const uint32_t parts = nch <= 4096 ? 8u : (nch <= 32768 ? 4u : 1u);
  hipLaunchKernelGGL((k_emit<K>), dim3(nch, parts), dim3(kBlock), 0, s, N, p.ld, vshift, sk, sv,
                     cnt, cpack, chunks, at<uint32_t>(ws, L.total), at<int32_t>(ws, L.txv), segk0,
                     v0, gv_base, reinterpret_cast<uint32_t*>(proj.splat), pack);
}
}  // namespace

namespace {
template <typename Kernel>
void launch_tile_sort(Kernel kernel, int threads, const BinSortPlan& p, const gs_projected& proj,
                      const DirectPlan& d, const Layout& L, const gs_tile_lists& lists, void* ws,
                      hipStream_t s) {
  hipLaunchKernelGGL(kernel, dim3((unsigned)p.n_segments), dim3(threads), 0, s, p.n_views, p.ld,
                     at<uint32_t>(ws, d.counts), at<uint32_t>(ws, L.seg_base), proj.depth_bits,
                     at<uint32_t>(ws, L.total), lists.vals, lists.ranges, lists.keys);
}
}  // namespace

// Most tiles whose lists four waves sort, whatever their length; beyond, one
// wave does up to kShortList.  The sort in us, one wave (and four for long
// lists) -> four: 64 tiles 26.6 -> 12.9, 500 tiles (0.48 M instances) 33.2 ->
// 17.6, 960 tiles 7.3 -> 7.2, 1,200 tiles 7.4 -> 8.3, 3,813 tiles 10.7 -> 14.8.
constexpr int64_t kWideSortTiles = 1024;

// The direct route's fill and sort, enqueued before the host has read the
// counts: the kernels do nothing without the scan's go-ahead.  Beyond
// kWideSortTiles, lists above kShortList follow in stage 2.  The device was
// idle for 25 us of a 187 us view while the host read the counts and came
// back with the rest.
hipError_t bin_sort_ahead(const BinSortPlan& p, const gs_projected& proj,
                          const gs_tile_lists& lists, void* ws, bool* ahead, hipStream_t s) {
  const Layout L = make_layout(p.n_views, p.ld, p.capacity, p.n_segments);
  const DirectPlan d = plan_direct(p, L);
  *ahead = d.possible;
  if (!d.possible) return hipSuccess;
  {
    StageScope scope(kStEmit, s);
    const dim3 grid(cdiv((uint64_t)p.n, kCountChunk),
                    std::min<uint32_t>((uint32_t)p.n_views, 65535u));
    hipLaunchKernelGGL(k_tile_fill, grid, dim3(kChunkThreads), 0, s, p.n, p.ld, p.n_views,
                       proj.tiles_touched, at<uint32_t>(ws, L.iparts),
                       reinterpret_cast<uint32_t*>(proj.splat), at<uint32_t>(ws, L.seg_base),
                       at<int32_t>(ws, L.txv), at<uint32_t>(ws, d.rows),
                       at<uint32_t>(ws, d.counts), at<uint32_t>(ws, L.total), lists.vals,
                       lists.gv_base);
  }
  StageScope scope(kStSegmentSort, s);
  if (p.n_segments <= kWideSortTiles)
    launch_tile_sort(k_tile_sort<256>, 256, p, proj, d, L, lists, ws, s);
  else
    launch_tile_sort(k_tile_sort<64>, 64, p, proj, d, L, lists, ws, s);
  return hipGetLastError();
}

hipError_t bin_sort_stage2(const BinSortPlan& p, const gs_projected& proj, const uint32_t* stats,
                           gs_tile_lists& lists, void* ws, hipStream_t s) {
  const uint32_t dmin = stats[0], dmax = stats[1], M = stats[2], N = stats[4];
  const Layout L = make_layout(p.n_views, p.ld, p.capacity, p.n_segments);
  if (M == 0) {
    launch_fill_u32(lists.ranges, 0u, 2 * p.n_segments, s);
    return hipGetLastError();
  }
  const DirectPlan d = plan_direct(p, L);
  if (d.possible && stats[kLongest] <= kDirectLongest) {  // filled and sorted already
    if (stats[kLongest] <= kShortList || p.n_segments <= kWideSortTiles) return hipSuccess;
    StageScope scope(kStSegmentSort, s);
    launch_tile_sort(k_tile_sort<256, true>, 256, p, proj, d, L, lists, ws, s);
    return hipGetLastError();
  }
  // the tile sort runs inside each view on the bits of its tile index (at
  // least one pass: the last one turns tile indices into segment ids)
  const int sbits = std::max(1, bits_for((uint64_t)p.max_tiles));
  const int spasses = plan_digits(sbits).passes;
  uint32_t* segk0 = at<uint32_t>(ws, L.segk0);
  uint32_t* segk1 = at<uint32_t>(ws, L.segk1);
  uint32_t* alt = at<uint32_t>(ws, L.segv_alt);
  // when a tile index and a Gaussian id fit one word together, the emit
  // writes tile << idbits | id and the tile sort moves those words only
  // (the last pass splits them); otherwise keys and ids move side by side,
  // emitted into the buffer that makes the sorted ids land in lists.vals
  const int idbits = bits_for((uint64_t)p.ld);
  const bool packed = idbits + sbits <= 32;
  uint32_t* v0 = packed ? nullptr : ((spasses & 1) ? alt : lists.vals);
  uint32_t* v1 = packed ? nullptr : ((spasses & 1) ? lists.vals : alt);
  const int pack = packed ? idbits : -1;
  // likewise each pair's tile count (at most the largest view's tiles) rides
  // above its Gaussian id through the depth sort when both fit one word
  const int cpack = idbits + bits_for((uint64_t)p.max_tiles + 1u) <= 32 ? idbits : -1;
  // the depth sort runs inside each view on the bits of the visible depth
  // range; (view, depth) keys are 32-bit when the views fit above those bits
  // (M > 0 means some pair is visible, so dmax >= dmin); only the N visible
  // pairs are sorted
  const int dbits = bits_for((uint64_t)dmax - (uint64_t)dmin + 1u);
  if (((uint64_t)p.n_views << dbits) <= ((uint64_t)1 << 32))
    depth_count_emit<uint32_t>(p, proj, L, ws, N, dmin, (uint32_t)dbits, dbits, cpack, segk0,
                               v0, pack, lists.gv_base, lists.ranges, s);
  else
    depth_count_emit<uint64_t>(p, proj, L, ws, N, dmin, 32u, dbits, cpack, segk0, v0, pack,
                               lists.gv_base, lists.ranges, s);
  int which2;
  {
    StageScope scope(kStSegmentSort, s);
    const ViewStarts vs{at<uint32_t>(ws, L.iparts), cdiv((uint64_t)p.n, kCountChunk), p.n_views};
    const SortSpec sp{packed ? idbits : 0, at<uint32_t>(ws, L.seg_base),
                      packed ? lists.vals : nullptr};
    which2 = radix_sort<uint32_t>(segk0, segk1, v0, v1, M, sbits, vs, sp, ws, L, s);
  }
  const uint32_t* seg_sorted = which2 ? segk1 : segk0;
  StageScope scope(kStRanges, s);
  hipLaunchKernelGGL(k_ranges, dim3(cdiv(cdiv(M, 4u), kBlock)), dim3(kBlock), 0, s, M,
                     seg_sorted, lists.ranges);
  if (lists.keys)
    hipLaunchKernelGGL(k_keys64, dim3(cdiv(M, kBlock)), dim3(kBlock), 0, s, M, p.n_views, p.ld,
                       seg_sorted, lists.vals, at<uint32_t>(ws, L.seg_base), proj.depth_bits,
                       lists.keys);
  return hipGetLastError();
}

}  // namespace gs
