// lut.hip -- device-side build of the guide-to-source lookup table (Sec. 3.1).
//
// LUT[c] = argmin_u |centre(c) - G_S[u]|^2 over all source pixels u, ties to
// the smallest raster index.
//
// 8-bit guides (two or three channels) take a separable exact transform:
// every value tuple a source pixel holds is a site keyed by the smallest
// raster index holding it, and since the squared distance is a sum over
// channels, the (distance, index) minimum over all sites can be taken one
// channel at a time -- first over channel 0 for every fixed value of the
// other channels, then over channel 1, ... -- on the grid of bin centres.
// Keys are uint64 (distance << 32 | index), so the lexicographic minimum is
// the integer minimum, and adding one channel's (weighted) squared distance
// to every key of a line keeps their order.  Each pass takes the minima of a
// line over the values of one channel that hold a site; since a line's
// minimum moves only one way from bin to bin, a few bins are searched over
// the whole line and the others between their neighbours' minima.
//
// 16-bit guides (too many value tuples for a grid) bucket the source pixels
// on a grid whose
// cells are at least twice as wide as a lookup bin (counting sort: count and
// rank, scan, scatter), and each bin then searches square rings of buckets around
// the bucket holding its centre.  After ring k the searched box is known, so
// every unsearched pixel is at least `gap` away along one axis, where gap is
// the distance from the centre to the nearest open side of the box; the
// search ends once the best squared distance is strictly below gap^2 (an
// equal distance further out could still win the raster-index tie).
#include "sb_internal.h"

namespace sb {
namespace {

struct LutGeom {
  int32_t depth;       // guide bits per channel: 8 or 16
  int32_t lut_bits;    // bins per channel = 1 << lut_bits
  int32_t bucket_bits; // buckets per channel = 1 << bucket_bits
  int32_t npix;
};

LutGeom lut_geom(int32_t fmt, int32_t sw, int32_t sh, int32_t lut_bits) {
  LutGeom g;
  g.depth = fmt == SB_GUIDE_U8X2 ? 8 : 16;
  g.lut_bits = lut_bits;
  g.npix = sw * sh;
  // about one bucket per few source pixels, never finer than half a bin
  int32_t side_bits = 0;
  while ((int64_t(1) << (2 * (side_bits + 1))) <= int64_t(g.npix)) ++side_bits;
  int32_t bb = side_bits - 1;
  if (bb > lut_bits - 1) bb = lut_bits - 1;
  if (bb < 1) bb = 1;
  if (bb > g.depth) bb = g.depth;
  g.bucket_bits = bb;
  return g;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct LutWs {
  uint32_t *count;  // nb
  uint32_t *start;  // nb + 1
  uint32_t *uneven; // 1 unless the pixels fill the buckets evenly (see k_lut_scan)
  uint2 *pts;       // npix: {g0 | g1 << 16, raster index}
  uint32_t *rank;   // npix: a pixel's rank in its bucket
  uint32_t *sums;   // the scan's block sums, in pts until the scatter fills it
};

LutWs lut_ws(void *base, const LutGeom &g) {
  size_t nb = size_t(1) << (2 * g.bucket_bits);
  char *p = static_cast<char *>(base);
  LutWs w;
  w.count = reinterpret_cast<uint32_t *>(p);
  p += align256(nb * 4);
  w.start = reinterpret_cast<uint32_t *>(p);
  w.uneven = w.start + nb + 1;
  p += align256((nb + 2) * 4);
  w.pts = reinterpret_cast<uint2 *>(p);
  w.sums = reinterpret_cast<uint32_t *>(p);
  p += align256(size_t(g.npix) * 8);
  w.rank = reinterpret_cast<uint32_t *>(p);
  return w;
}

// ------------------------------------------------ separable (8-bit guides)

constexpr uint64_t kNoKey = ~0ull;
constexpr int32_t kSepTile = 16;  // columns of one pass block
constexpr int32_t kManyLabels = 8;

// f0[value tuple c0 | c1 << 8 (| c2 << 16)] = smallest raster index holding
// it (pre-filled with ~0u); with `labels`, only pixels labelled `want`.  Only
// pixels that may lower an entry take an atomic: not one whose left neighbour
// holds the same value, nor one that already finds a smaller index (a stale
// value of a falling entry only costs an atomic): 512 x 512 normals of a
// sphere, most of them one of few values, 3 us (8.4 with one per pixel).  Where
// more than kManyLabels labels share the pixels (`check` 0) few of a pass's pixels
// are its own and waiting for the entry costs more: 16 tables of 2048 x 2048 noise
// 527 us, 980 with it.
template <int FMT>
__global__ void __launch_bounds__(256) k_sep_sites(const void *guide, int32_t npix, uint32_t *f0,
                                                   const uint8_t *labels, int32_t want,
                                                   int32_t check) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  uint32_t v = ~0u;  // no value
  if (i < uint32_t(npix) && (!labels || labels[i] == want))
    v = FMT == SB_GUIDE_U8X2 ? uint32_t(static_cast<const uint16_t *>(guide)[i])
                             : static_cast<const uint32_t *>(guide)[i] & 0xFFFFFFu;
  const uint32_t left = uint32_t(__shfl_up(int(v), 1, 64));  // every lane takes part
  if (v == ~0u || ((threadIdx.x & 63u) != 0 && v == left)) return;
  if (!check || f0[v] > i) atomicMin(&f0[v], i);
}

// One channel of the minimisation.  The input is [outer][256][inner]: keys,
// or with SITES the site indices of f0 (~0u: none).  The output is
// [outer][nb][inner] keys, or with FINAL the table entries (coordinates;
// where no site exists at all -- a label absent from the exemplar -- the
// entry of `fallback`).  A block takes `ti` columns, adjacent along `inner`
// or, where that is 1, along `outer`: it stages their 256 x ti input keys in
// LDS, lists the channel values that hold a key in any of them, and computes
// the nb x ti minima over that list.
//
// For bins c < c' and values v < v', f_v(c') - f_v'(c') exceeds f_v(c) -
// f_v'(c) (by 2 w (c' - c)(v' - v)): a value that beats a smaller one, or
// ties with it at a smaller index, beats it for good in every later bin, so
// the position of the minimum never falls from bin to bin.  64 / ti bins are
// searched over the whole list, four threads each, then three between every
// two, each only between its neighbours' positions, until every bin is done:
// about 240 candidates per thread at 16 columns instead of 16 x 256.  VALU
// bound (lanes wait for the longest range of their wave): the passes of a
// 512 x 512 three-channel exemplar's 2^24 bins take 134, 133 and 165 us (138,
// 608 and 901 with every bin searched over the whole list); a two-channel
// one's two passes 7 and 9 us (13.4 and 13.7), there the longest thread.
//
// A short list is searched whole for every bin (up to kShortWork candidates a
// thread): the turns from bin to bin would take longer (16 tables of a 64 x 64
// guide with labels 272 us, 234 so).
constexpr int32_t kShortWork = 128;
constexpr uint64_t kFarKey = 0x70000000FFFFFFFFull;  // staged for "no key": beyond every distance

template <bool SITES, bool FINAL>
__global__ __launch_bounds__(256) void k_sep_pass(const void *in, uint64_t *out, uint32_t *lut,
                                                  const uint32_t *fallback, int32_t inner,
                                                  int32_t ti, int32_t lut_bits, int32_t weight,
                                                  int32_t sw) {
  __shared__ uint64_t key[256 * kSepTile];
  __shared__ uint8_t pos[256 * kSepTile];  // list position of a bin's minimum
  __shared__ __attribute__((aligned(4))) uint8_t vlist[256 + 4];
  __shared__ uint32_t wcount[4];
  const int32_t t = threadIdx.x;
  // column j of the block: its first input element, the step between its
  // values there, and its first output element (bins are `inner` apart too)
  const int32_t per_line = inner > 1 ? inner / ti : 1;
  const size_t o0 = inner > 1 ? blockIdx.x / uint32_t(per_line) : size_t(blockIdx.x) * size_t(ti);
  const int32_t i0 = inner > 1 ? int32_t(blockIdx.x % uint32_t(per_line)) * ti : 0;
  const int32_t nb = 1 << lut_bits, sft = 8 - lut_bits;
  for (int32_t e = t; e < 256 * ti; e += 256) {
    // along the fastest index of the input
    const int32_t v = inner > 1 ? e / ti : e & 255, j = inner > 1 ? e - v * ti : e >> 8;
    const size_t src = inner > 1 ? (o0 * 256 + size_t(v)) * size_t(inner) + size_t(i0 + j)
                                 : (o0 + size_t(j)) * 256 + size_t(v);
    uint64_t k;
    if (SITES) {
      const uint32_t idx = static_cast<const uint32_t *>(in)[src];
      k = idx == ~0u ? kFarKey : uint64_t(idx);
    } else {
      k = static_cast<const uint64_t *>(in)[src];
      k = k == kNoKey ? kFarKey : k;
    }
    key[v * kSepTile + j] = k;
  }
  __syncthreads();
  // compact list of the channel values with a key (thread t examines v = t)
  bool any = false;
  for (int32_t j = 0; j < ti; ++j) any |= key[t * kSepTile + j] != kFarKey;
  const uint64_t mask = __ballot(any);
  const int32_t wave = t >> 6, lane = t & 63;
  if (lane == 0) wcount[wave] = uint32_t(__popcll(mask));
  __syncthreads();
  uint32_t base = 0;
  for (int32_t w = 0; w < wave; ++w) base += wcount[w];
  const int32_t count = int32_t(wcount[0] + wcount[1] + wcount[2] + wcount[3]);
  if (any) {
    const int32_t at = int32_t(base) + __popcll(mask & ((1ull << lane) - 1ull));
    vlist[at] = uint8_t(t);
    // a whole search reads four at a time: the last value again is harmless
    if (at == count - 1) vlist[count] = vlist[count + 1] = vlist[count + 2] = uint8_t(t);
  }
  __syncthreads();
  const int32_t half = sft ? 1 << (sft - 1) : 0;
  const int32_t j = t % ti, slot = t / ti, slots = 256 / ti;
  uint64_t best;
  int32_t best_at;
  auto weigh = [&](int32_t centre, int32_t v, int32_t n, uint64_t k) {
    const int32_t d = centre - v;
    const uint64_t cand = k + (uint64_t(uint32_t(__mul24(weight, __mul24(d, d)))) << 32);
    best_at = cand < best ? n : best_at;
    best = cand < best ? cand : best;
  };
  auto emit = [&](int32_t b) {
    const size_t dst = inner > 1 ? (o0 * size_t(nb) + size_t(b)) * size_t(inner) + size_t(i0 + j)
                                 : (o0 + size_t(j)) * size_t(nb) + size_t(b);
    const bool none = best >= kFarKey;
    if (FINAL) {
      const uint32_t idx = uint32_t(best);
      lut[dst] = none ? (fallback ? fallback[dst] : 0u)
                      : pack_xy(idx % uint32_t(sw), idx / uint32_t(sw));
    } else {
      out[dst] = none ? kNoKey : best;
    }
  };
  if (nb * count <= kShortWork * slots) {
    for (int32_t b = slot; b < nb; b += slots) {
      const int32_t centre = (b << sft) + half;
      best = kNoKey, best_at = 0;
      for (int32_t n = 0; n < count; n += 4) {
        const uint32_t v4 = *reinterpret_cast<const uint32_t *>(vlist + n);
        uint64_t k[4];
#pragma unroll
        for (int32_t m = 0; m < 4; ++m)
          k[m] = key[int32_t((v4 >> (8 * m)) & 0xFFu) * kSepTile + j];
#pragma unroll
        for (int32_t m = 0; m < 4; ++m) weigh(centre, int32_t((v4 >> (8 * m)) & 0xFFu), 0, k[m]);
      }
      emit(b);
    }
    return;
  }
  // the first bins, a quarter of the list per thread
  const int32_t firsts = slots / 4, part = slot & 3;
  int32_t step = nb > firsts ? nb / firsts : 1;
  {
    const int32_t b = (slot >> 2) * step, centre = (b << sft) + half;
    best = kNoKey, best_at = 0;
    for (int32_t n = 4 * part; n < count; n += 16) {
      const uint32_t v4 = *reinterpret_cast<const uint32_t *>(vlist + n);
      uint64_t k[4];
#pragma unroll
      for (int32_t m = 0; m < 4; ++m)
        k[m] = key[int32_t((v4 >> (8 * m)) & 0xFFu) * kSepTile + j];
#pragma unroll
      for (int32_t m = 0; m < 4; ++m)
        weigh(centre, int32_t((v4 >> (8 * m)) & 0xFFu), min(n + m, count - 1), k[m]);
    }
#pragma unroll
    for (int32_t x = 1; x <= 2; x <<= 1) {
      const uint64_t k = uint64_t(__shfl_xor((unsigned long long)best, x * ti, 64));
      const int32_t at = __shfl_xor(best_at, x * ti, 64);
      best_at = k < best ? at : best_at;
      best = k < best ? k : best;
    }
    if (part == 0 && b < nb) {
      emit(b);
      pos[b * kSepTile + j] = uint8_t(best_at);
    }
  }
  while (step > 1) {
    __syncthreads();
    const int32_t next = step >= 4 ? step / 4 : 1, per = step / next - 1;  // new bins per gap
    for (int32_t e = slot; e < nb / step * per; e += slots) {
      const int32_t gap = e / per, b = gap * step + (e - gap * per + 1) * next;
      const int32_t centre = (b << sft) + half;
      const int32_t from = pos[gap * step * kSepTile + j];
      const int32_t to = (gap + 1) * step < nb ? int32_t(pos[(gap + 1) * step * kSepTile + j])
                                               : count - 1;
      best = kNoKey, best_at = from;
      for (int32_t n = from; n <= to; n += 2) {
        const int32_t n1 = min(n + 1, to), v0 = vlist[n], v1 = vlist[n1];
        const uint64_t k0 = key[v0 * kSepTile + j], k1 = key[v1 * kSepTile + j];
        weigh(centre, v0, n, k0);
        weigh(centre, v1, n1, k1);
      }
      emit(b);
      pos[b * kSepTile + j] = uint8_t(best_at);
    }
    step = next;
  }
}

// ------------------------------------------------ bucketed (16-bit guides)

__device__ inline void read_guide(const void *g, uint32_t i, uint32_t &c0, uint32_t &c1) {
  const uint32_t v = static_cast<const uint32_t *>(g)[i];
  c0 = v & 0xFFFFu;
  c1 = v >> 16;
}

__global__ void k_fill_u32(uint32_t *p, uint32_t n, uint32_t v) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

// The sort's bucket of source pixel i; a pixel not labelled `want` (with
// `labels`: one per-label table of the segmentation guide) has none.
constexpr uint32_t kNoBucket = ~0u;
__device__ inline uint32_t lut_bucket(const void *guide, uint32_t i, int32_t shift, int32_t bb,
                                      const uint8_t *labels, int32_t want, uint32_t &c0,
                                      uint32_t &c1) {
  if (labels && labels[i] != want) return kNoBucket;
  read_guide(guide, i, c0, c1);
  return ((c1 >> shift) << bb) | (c0 >> shift);
}

// Counting sort over the source pixels, first pass: count[bucket] and every
// pixel's rank in its bucket (the count before it), so the scatter needs no
// second atomic per pixel.  Neighbouring pixels mostly share a bucket (a
// smooth guide), so the lanes of a run of equal buckets take their ranks from
// one atomic of the run's first lane.  Bound by the atomics' rate in L2: 14 us
// for a 2048 x 2048 guide of texture coordinates (one atomic per pixel 70 us,
// and the scatter with its own atomics 141 us against 14).
__global__ void __launch_bounds__(256) k_lut_count(const void *guide, int32_t npix, int32_t shift,
                                                   int32_t bb, uint32_t *count, uint32_t *rank,
                                                   const uint8_t *labels, int32_t want) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  const int32_t lane = int32_t(threadIdx.x & 63u);
  uint32_t c0, c1, b = kNoBucket;
  if (i < uint32_t(npix)) b = lut_bucket(guide, i, shift, bb, labels, want, c0, c1);
  const uint32_t prev = uint32_t(__shfl_up(int(b), 1, 64));  // every lane takes part
  const bool head = lane == 0 || b != prev;
  const uint64_t heads = __ballot(head);
  const uint64_t upto = heads & (~0ull >> (63 - lane));
  const int32_t first = 63 - __clzll((long long)upto);  // bit 0 is always set
  const uint64_t after = lane == 63 ? 0ull : heads >> (lane + 1);
  uint32_t base = 0;
  if (head && b != kNoBucket)
    base = atomicAdd(&count[b], uint32_t(after ? __ffsll((long long)after) : 64 - lane));
  base = uint32_t(__shfl(int(base), first, 64));
  if (b != kNoBucket) rank[i] = base + uint32_t(lane - first);
}

// Exclusive scan of n counts (a power of 4, at least 4) into start[0..n] in
// two passes over blocks of kScanBlock counts: every block's sum, then every
// block adds up the sums before it (at most n / kScanBlock = 1024 of them)
// and scans its own counts: 9 us for 2^20 buckets, launch bound (one
// workgroup scanning all of them took 2.48 ms of the 2.73 ms a 2048 x 2048
// style took).  The second also tells whether the pixels fill the buckets evenly:
// none of them holds more than kFullBucket, and no block has more than half of
// its own empty.
constexpr uint32_t kScanPer = 16, kScanBlock = 256 * kScanPer;
constexpr uint32_t kFullBucket = 32;
// (dword-aligned: the workspace is the caller's)
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ inline uint32_t block_sum(uint32_t v, uint32_t *part) {  // 256 threads
#pragma unroll
  for (int32_t o = 32; o > 0; o >>= 1) v += uint32_t(__shfl_xor(int(v), o, 64));
  if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  return part[0] + part[1] + part[2] + part[3];
}

__global__ void __launch_bounds__(256) k_lut_sums(const uint32_t *count, uint32_t n,
                                                  uint32_t *sums, uint32_t *uneven) {
  __shared__ uint32_t part[4];
  if (blockIdx.x == 0 && threadIdx.x == 0) *uneven = 0u;
  uint32_t s = 0;
#pragma unroll
  for (uint32_t k = 0; k < kScanPer / 4; ++k) {
    const uint32_t i = blockIdx.x * kScanBlock + 4 * (k * 256 + threadIdx.x);
    if (i < n) {
      const u32x4a4 c = *reinterpret_cast<const u32x4a4 *>(count + i);
      s += c.x + c.y + c.z + c.w;
    }
  }
  s = block_sum(s, part);
  if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

__global__ void __launch_bounds__(256) k_lut_scan(const uint32_t *count, const uint32_t *sums,
                                                  uint32_t n, uint32_t *start,
                                                  uint32_t *uneven) {
  __shared__ uint32_t part[4], wsum[4], some[4];
  const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
  uint32_t before = 0;
  for (uint32_t b = t; b < blockIdx.x; b += 256) before += sums[b];
  before = block_sum(before, part);
  // thread t owns counts [kScanPer t, kScanPer (t + 1)) of the block
  const uint32_t i0 = blockIdx.x * kScanBlock + kScanPer * t;
  u32x4a4 c[kScanPer / 4];
  uint32_t s = 0, held = 0, most = 0;
#pragma unroll
  for (uint32_t k = 0; k < kScanPer / 4; ++k) {
    c[k] = u32x4a4{0u, 0u, 0u, 0u};
    if (i0 + 4 * k < n) c[k] = *reinterpret_cast<const u32x4a4 *>(count + i0 + 4 * k);
    s += c[k].x + c[k].y + c[k].z + c[k].w;
#pragma unroll
    for (int j = 0; j < 4; ++j) held += c[k][j] != 0u, most = max(most, c[k][j]);
  }
  uint32_t incl = s;
#pragma unroll
  for (uint32_t o = 1; o < 64; o <<= 1) {
    const uint32_t v = uint32_t(__shfl_up(int(incl), o, 64));
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[wave] = incl;
  // (block_sum's own words are still being read)
  const uint32_t filled = block_sum(held, some);
  const bool full = __any(most > kFullBucket);
  if ((lane == 0 && full) || (t == 0 && 2 * filled < min(n, kScanBlock))) *uneven = 1u;
  uint32_t run = before + incl - s;
  for (uint32_t w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
  for (uint32_t k = 0; k < kScanPer / 4; ++k) {
    if (i0 + 4 * k < n) {
      u32x4a4 v;
      v.x = run;
      v.y = v.x + c[k].x;
      v.z = v.y + c[k].y;
      v.w = v.z + c[k].z;
      run = v.w + c[k].w;
      *reinterpret_cast<u32x4a4 *>(start + i0 + 4 * k) = v;
      if (i0 + 4 * k + 4 == n) start[n] = run;
    }
  }
}

__global__ void __launch_bounds__(256) k_lut_scatter(const void *guide, int32_t npix,
                                                     int32_t shift, int32_t bb,
                                                     const uint32_t *start, const uint32_t *rank,
                                                     uint2 *pts, const uint8_t *labels,
                                                     int32_t want) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= uint32_t(npix)) return;
  uint32_t c0, c1;
  const uint32_t b = lut_bucket(guide, i, shift, bb, labels, want, c0, c1);
  if (b != kNoBucket) pts[start[b] + rank[i]] = make_uint2(c0 | (c1 << 16), i);
}

// Q x Q bins of one bucket, the first of them (cx, cy): one walk over the rings of
// buckets serves them all, so every bucket's bounds and pixels are read once for Q x Q
// bins.  A candidate is distance << 26 | raster index (at most 2^33 and 2^26), so ties
// go to the smallest index by themselves.  Four pixels' loads are in flight together:
// one after another, a long bucket (a guide of few values) takes as many round trips
// as it has pixels (a 512 x 512 guide, half of it constant, at 9 bits 19 ms, 36 so).
template <int Q>
__device__ __forceinline__ void lut_query(const uint32_t *start, const uint2 *pts, uint32_t cx,
                                          uint32_t cy, int32_t lut_bits, int32_t bin_shift,
                                          int32_t bucket_bits, int32_t bucket_shift, int32_t sw,
                                          uint32_t *lut) {
  const uint32_t side = 1u << lut_bits;
  const uint32_t half = bin_shift ? (1u << (bin_shift - 1)) : 0u;
  uint32_t qx[Q], qy[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i)
    qx[i] = ((cx + i) << bin_shift) + half, qy[i] = ((cy + i) << bin_shift) + half;
  const int32_t nb = 1 << bucket_bits;
  const int32_t bw = 1 << bucket_shift;  // bucket width in guide units
  const int32_t bx0 = int32_t(qx[0] >> bucket_shift), by0 = int32_t(qy[0] >> bucket_shift);
  uint64_t best[Q][Q];
#pragma unroll
  for (int j = 0; j < Q; ++j)
#pragma unroll
    for (int i = 0; i < Q; ++i) best[j][i] = ~0ull;
  auto take = [&](const uint2 p) {
    uint32_t dx[Q], dy[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int32_t ex = int32_t(qx[i]) - int32_t(p.x & 0xFFFFu);
      const int32_t ey = int32_t(qy[i]) - int32_t(p.x >> 16);
      dx[i] = uint32_t(ex) * uint32_t(ex), dy[i] = uint32_t(ey) * uint32_t(ey);
    }
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int i = 0; i < Q; ++i)
        best[j][i] = min(best[j][i], ((uint64_t(dx[i]) + dy[j]) << 26) | p.y);
  };
  for (int32_t k = 0;; ++k) {
    const int32_t x0 = bx0 - k, x1 = bx0 + k, y0 = by0 - k, y1 = by0 + k;
    const int32_t ya = y0 > 0 ? y0 : 0, yb = y1 < nb - 1 ? y1 : nb - 1;
    for (int32_t by = ya; by <= yb; ++by) {
      const bool full = (by == y0) || (by == y1);
      const int32_t step = full ? 1 : (x1 - x0);
      for (int32_t bx = x0; bx <= x1; bx += (step > 0 ? step : 1)) {
        if (bx < 0 || bx >= nb) continue;
        const uint32_t b = (uint32_t(by) << bucket_bits) | uint32_t(bx);
        uint32_t e = start[b];
        const uint32_t e1 = start[b + 1];
        for (; e + 4 <= e1; e += 4) {
          const uint2 p0 = pts[e], p1 = pts[e + 1], p2 = pts[e + 2], p3 = pts[e + 3];
          take(p0), take(p1), take(p2), take(p3);
        }
        for (; e < e1; ++e) take(pts[e]);
      }
    }
    // distance from each centre to the nearest side of the searched box that
    // still has buckets beyond it
    bool all = true, more = false;
#pragma unroll
    for (int j = 0; j < Q; ++j)
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        uint32_t gap = ~0u;
        if (x0 > 0) gap = min(gap, qx[i] - uint32_t(x0 * bw) + 1u);
        if (x1 < nb - 1) gap = min(gap, uint32_t((x1 + 1) * bw) - qx[i]);
        if (y0 > 0) gap = min(gap, qy[j] - uint32_t(y0 * bw) + 1u);
        if (y1 < nb - 1) gap = min(gap, uint32_t((y1 + 1) * bw) - qy[j]);
        more |= gap != ~0u;
        all &= best[j][i] != ~0ull && (best[j][i] >> 26) < uint64_t(gap) * gap;
      }
    if (!more || all) break;  // every bucket searched, or every bin's nearest found
  }
#pragma unroll
  for (int j = 0; j < Q; ++j)
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const uint32_t idx = uint32_t(best[j][i]) & 0x3FFFFFFu;
      lut[(cy + j) * side + cx + i] = pack_xy(idx % uint32_t(sw), idx / uint32_t(sw));
    }
}

// The table, a thread per bin or, where that pays, per 2 x 2 bins of one bucket
// (buckets are at least two bins wide from two bits per channel on).  It pays on
// evenly filled buckets (4 M bins of a 2048 x 2048 guide of texture coordinates
// 15.2 us, 19 with one bin a thread): where the pixels crowd in a few, the walks
// are long and a quarter of the threads waits too much for each (a 512 x 512
// guide of constant regions at 9 bits 211 ms, 818 with 2 x 2 bins).
// `fallback` (may be null): when no pixel was bucketed (a label absent from
// the exemplar), copy this table instead.
__global__ void __launch_bounds__(256) k_lut_query(const uint32_t *start, const uint32_t *uneven,
                                                   const uint2 *pts, int32_t lut_bits,
                                                   int32_t bin_shift, int32_t bucket_bits,
                                                   int32_t bucket_shift, int32_t sw, uint32_t *lut,
                                                   const uint32_t *fallback) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (fallback && start[1u << (2 * bucket_bits)] == 0) {
    if (t < 1u << (2 * lut_bits)) lut[t] = fallback[t];
    return;
  }
  if (bucket_bits < lut_bits && *uneven == 0u) {
    const uint32_t across = 1u << (lut_bits - 1);
    if (t < across * across)
      lut_query<2>(start, pts, t % across * 2, t / across * 2, lut_bits, bin_shift, bucket_bits,
                   bucket_shift, sw, lut);
  } else if (t < 1u << (2 * lut_bits)) {
    lut_query<1>(start, pts, t & ((1u << lut_bits) - 1u), t >> lut_bits, lut_bits, bin_shift,
                 bucket_bits, bucket_shift, sw, lut);
  }
}

unsigned blocks_for(uint64_t n, unsigned bs) { return unsigned((n + bs - 1) / bs); }

}  // namespace

namespace {
// Workspace of the separable build: X holds the keys after channel 0; Y
// first the site grid, then (three channels) the keys after channel 1.
struct SepWs {
  uint64_t *x;
  void *y;
};
size_t sep_x_bytes(int32_t nch, int32_t lut_bits) {
  return align256((size_t(1) << (8 * (nch - 1))) * (size_t(1) << lut_bits) * 8);
}
size_t sep_y_bytes(int32_t nch, int32_t lut_bits) {
  const size_t sites = (size_t(1) << (8 * nch)) * 4;
  const size_t keys1 = nch == 3 ? size_t(256) * (size_t(1) << (2 * lut_bits)) * 8 : 0;
  return align256(sites > keys1 ? sites : keys1);
}
}  // namespace

size_t lut_workspace_bytes(int32_t fmt, int32_t sw, int32_t sh, int32_t lut_bits) {
  if (fmt != SB_GUIDE_U16X2) {
    const int32_t nch = fmt_channels(fmt);
    return sep_x_bytes(nch, lut_bits) + sep_y_bytes(nch, lut_bits);
  }
  LutGeom g = lut_geom(fmt, sw, sh, lut_bits);
  size_t nb = size_t(1) << (2 * g.bucket_bits);
  return align256(nb * 4) + align256((nb + 2) * 4) + align256(size_t(g.npix) * 8) +
         align256(size_t(g.npix) * 4);
}

namespace {
// Launch one pass over [outer][256][inner] -> [outer][nb][inner].
template <bool SITES, bool FINAL>
void sep_pass(const void *in, uint64_t *out, uint32_t *lut, const uint32_t *fallback,
              size_t outer, int32_t inner, int32_t lut_bits, int32_t weight, int32_t sw,
              hipStream_t stream) {
  // up to kSepTile columns per block, fewer when that leaves the chip
  // short of blocks (the last pass of a two-channel table has one line of
  // 2^lut_bits columns)
  const size_t cols = outer * size_t(inner), most = inner > 1 ? size_t(inner) : outer;
  int32_t ti = most < size_t(kSepTile) ? int32_t(most) : kSepTile;
  while (ti > 1 && cols / size_t(ti) < 2048) ti >>= 1;
  const size_t blocks = cols / size_t(ti);
  k_sep_pass<SITES, FINAL><<<unsigned(blocks), 256, 0, stream>>>(in, out, lut, fallback, inner,
                                                                  ti, lut_bits, weight, sw);
}

hipError_t build_sep(const void *guide, int32_t fmt, int32_t sw, int32_t sh, int32_t lut_bits,
                     const int32_t *wt, uint32_t *lut, void *workspace, const uint8_t *labels,
                     int32_t want, int32_t nlabels, const uint32_t *fallback,
                     hipStream_t stream) {
  const int32_t nch = fmt_channels(fmt);
  const int32_t nb = 1 << lut_bits, npix = sw * sh;
  uint64_t *x = static_cast<uint64_t *>(workspace);
  char *y = static_cast<char *>(workspace) + sep_x_bytes(nch, lut_bits);
  uint32_t *f0 = reinterpret_cast<uint32_t *>(y);
  const uint32_t nsites = 1u << (8 * nch);
  const int32_t check = nlabels <= kManyLabels;
  k_fill_u32<<<blocks_for(nsites, 256) < 4096 ? blocks_for(nsites, 256) : 4096, 256, 0, stream>>>(
      f0, nsites, ~0u);
  if (fmt == SB_GUIDE_U8X2)
    k_sep_sites<SB_GUIDE_U8X2><<<blocks_for(npix, 256), 256, 0, stream>>>(guide, npix, f0, labels,
                                                                          want, check);
  else
    k_sep_sites<SB_GUIDE_U8X3><<<blocks_for(npix, 256), 256, 0, stream>>>(guide, npix, f0, labels,
                                                                          want, check);
  // channel 0: [v_rest][v0] -> [v_rest][b0]
  sep_pass<true, false>(f0, x, nullptr, nullptr, size_t(1) << (8 * (nch - 1)), 1, lut_bits,
                        wt[0], sw, stream);
  if (nch == 2) {
    // channel 1: [v1][b0] -> [b1][b0], the table
    sep_pass<false, true>(x, nullptr, lut, fallback, 1, nb, lut_bits, wt[1], sw, stream);
  } else {
    uint64_t *k1 = reinterpret_cast<uint64_t *>(y);  // the site grid is no longer needed
    // channel 1: [v2][v1][b0] -> [v2][b1][b0]
    sep_pass<false, false>(x, k1, nullptr, nullptr, 256, nb, lut_bits, wt[1], sw, stream);
    // channel 2: [v2][b1 b0] -> [b2][b1 b0], the table
    sep_pass<false, true>(k1, nullptr, lut, fallback, 1, nb * nb, lut_bits, wt[2], sw, stream);
  }
  return hipGetLastError();
}

// One table: over all source pixels (labels null) or those labelled `want`.
hipError_t build_one(const void *guide, int32_t fmt, int32_t sw, int32_t sh, int32_t lut_bits,
                     const int32_t *wt, uint32_t *lut, void *workspace, const uint8_t *labels,
                     int32_t want, int32_t nlabels, const uint32_t *fallback,
                     hipStream_t stream) {
  if (fmt != SB_GUIDE_U16X2)
    return build_sep(guide, fmt, sw, sh, lut_bits, wt, lut, workspace, labels, want, nlabels,
                     fallback, stream);
  const LutGeom g = lut_geom(fmt, sw, sh, lut_bits);
  const LutWs w = lut_ws(workspace, g);
  const uint32_t nb = 1u << (2 * g.bucket_bits);
  const int32_t shift = g.depth - g.bucket_bits;
  k_fill_u32<<<blocks_for(nb, 256) < 4096 ? blocks_for(nb, 256) : 4096, 256, 0, stream>>>(
      w.count, nb, 0u);
  k_lut_count<<<blocks_for(g.npix, 256), 256, 0, stream>>>(guide, g.npix, shift, g.bucket_bits,
                                                           w.count, w.rank, labels, want);
  // the block sums (at most 1024 words, one per kScanBlock buckets) lie in
  // pts, which holds 8 bytes per pixel and at least one pixel per 4 buckets
  const unsigned sb = blocks_for(nb, kScanBlock);
  k_lut_sums<<<sb, 256, 0, stream>>>(w.count, nb, w.sums, w.uneven);
  k_lut_scan<<<sb, 256, 0, stream>>>(w.count, w.sums, nb, w.start, w.uneven);
  k_lut_scatter<<<blocks_for(g.npix, 256), 256, 0, stream>>>(
      guide, g.npix, shift, g.bucket_bits, w.start, w.rank, w.pts, labels, want);
  const uint64_t nbins = uint64_t(1) << (2 * lut_bits);
  k_lut_query<<<blocks_for(nbins, 256), 256, 0, stream>>>(
      w.start, w.uneven, w.pts, lut_bits, g.depth - lut_bits, g.bucket_bits, shift, sw, lut,
      fallback);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_lut_build(const void *guide, int32_t fmt, int32_t sw, int32_t sh,
                            int32_t lut_bits, const int32_t wt[3], uint32_t *lut,
                            void *workspace, hipStream_t stream) {
  return build_one(guide, fmt, sw, sh, lut_bits, wt, lut, workspace, nullptr, 0, 0, nullptr,
                   stream);
}

hipError_t launch_lut_build_labels(const void *guide, const uint8_t *labels, int32_t fmt,
                                   int32_t sw, int32_t sh, int32_t lut_bits, const int32_t wt[3],
                                   int32_t nlabels, const uint32_t *lut, uint32_t *luts,
                                   void *workspace, hipStream_t stream) {
  const size_t bins = size_t(1) << (fmt_channels(fmt) * lut_bits);
  for (int32_t l = 0; l < nlabels; ++l) {
    const hipError_t e = build_one(guide, fmt, sw, sh, lut_bits, wt, luts + size_t(l) * bins,
                                   workspace, labels, l, nlabels, lut, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace sb
