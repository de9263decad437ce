// search.hip -- guides of 2..8 channels (SB_GUIDE_U8XN / SB_GUIDE_U16XN),
// looked up by an exact nearest-texel search instead of a table: the
// additional guiding channels of Sec. 3.1, for which the paper suggests a
// search tree.
//
//   tree build   texels equal in every channel become one, the one of smallest
//                raster index (k_tree_merge, k_tree_take); of the distinct
//                ones a balanced k-d tree, kept as a complete
//                8-ary tree in level order (see tree_layout): every split is
//                at the median of the widest element (by weight, then by raw
//                range) and hands its left child exactly half of the padded
//                size, so nodes need no links.  Splits of more than
//                kSortBlock texels run over the chip (k_tree_hist,
//                k_tree_split); below that one workgroup sorts its
//                kSortBlock texels in LDS down to runs of eight
//                (k_tree_sort) and k_tree_top joins the runs' boxes.
//   search       groups of G lanes per query, one node per step: the lanes
//                load the node's eight child records (box and smallest
//                coordinate) in one round trip, descend to the nearest and
//                leave the others in LDS; the last level's children are the
//                texels themselves.  A child is skipped only if its box lies
//                strictly farther than the best texel so far (or equally far
//                with no smaller raster index in it), so the result is the
//                exact argmin of sum_k w_k (q_k - g_k)^2, ties to the
//                smallest raster index, for any tree shape.
//   k_seeds_n    eight lanes per padded seed record: the seed and its search.
//   k_assign_blocks_n, k_assign_n
//                the level loop of Algorithm 2 with the many-channel error,
//                per 8 x 8 block or (cells smaller than blocks) per pixel; a
//                pixel no level accepts keeps the nearest candidate its level
//                loop measured.
//   k_fallback_n those pixels' own lookups, each search starting from that
//                candidate.
//   k_tree_query the search of caller-given texels (sb_tree_query).
#include <stdio.h>
#include <string.h>

#include <new>
#include <type_traits>

#include "sb_device.h"

namespace sb {
namespace {

// Texels one workgroup sorts in LDS.
constexpr uint32_t kSortLog = 11, kSortBlock = 1u << kSortLog;
// Texels per workgroup of the splits before that.
constexpr uint32_t kSplitLog = 10, kSplitBlock = 1u << kSplitLog, kSplitThreads = 256;
// Bins of a split's histogram.
constexpr uint32_t kBinsLog = 10, kBins = 1u << kBinsLog;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
// Dword-aligned vectors (global loads need dword alignment only).
typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Squared distances: 8-bit channels fit 32 bits (8 * 127 * 255^2), 16-bit
// ones need 64 (8 * 127 * 65535^2).
template <int D>
struct DistOf {
  typedef uint32_t type;
};
template <>
struct DistOf<16> {
  typedef uint64_t type;
};

// A texel of S bytes: S / (D / 8) elements of D bits.
template <int S>
struct Tx {
  uint32_t w[S / 4];
};

template <int S>
__device__ __forceinline__ Tx<S> load_tx(const void *base, uint32_t i) {
  Tx<S> t;
  if constexpr (S == 4) {
    t.w[0] = glb(static_cast<const uint32_t *>(base))[i];
  } else if constexpr (S == 8) {
    const u32x2 v = glb(static_cast<const u32x2 *>(base))[i];
    t.w[0] = v.x, t.w[1] = v.y;
  } else {
    const u32x4 v = glb(static_cast<const u32x4 *>(base))[i];
    t.w[0] = v.x, t.w[1] = v.y, t.w[2] = v.z, t.w[3] = v.w;
  }
  return t;
}

template <int S>
__device__ __forceinline__ void store_tx(void *base, uint32_t i, const Tx<S> &t) {
  if constexpr (S == 4) {
    glb(static_cast<uint32_t *>(base))[i] = t.w[0];
  } else if constexpr (S == 8) {
    glb(static_cast<u32x2 *>(base))[i] = u32x2{t.w[0], t.w[1]};
  } else {
    glb(static_cast<u32x4 *>(base))[i] = u32x4{t.w[0], t.w[1], t.w[2], t.w[3]};
  }
}

template <int D, int S>
constexpr int kElems = S * 8 / D;

// Element k (compile-time) of a texel.
template <int D, int S, int K>
__device__ __forceinline__ uint32_t elem(const Tx<S> &t) {
  if constexpr (D == 8) return (t.w[K >> 2] >> ((K & 3) * 8)) & 0xFFu;
  else return (t.w[K >> 1] >> ((K & 1) * 16)) & 0xFFFFu;
}

// Weight of element k: byte k of wn (0 past the guide's channels).
template <int K>
__device__ __forceinline__ uint32_t weight(const uint32_t *wn) {
  return (wn[K >> 2] >> ((K & 3) * 8)) & 0xFFu;
}

// Unrolled loop over the elements k = 0..E-1 with k a compile-time constant.
template <int K, int E, class F>
__device__ __forceinline__ void for_elems(F &&f) {
  if constexpr (K < E) {
    f(std::integral_constant<int, K>());
    for_elems<K + 1, E>(f);
  }
}

// sum_k w_k (a_k - b_k)^2.  |a_k - b_k| < 2^16 fits the 24-bit multiply and
// its square fits 32 bits.
template <int D, int S>
__device__ __forceinline__ typename DistOf<D>::type tx_dist(const Tx<S> &a, const Tx<S> &b,
                                                           const uint32_t *wn) {
  typename DistOf<D>::type d = 0;
  for_elems<0, kElems<D, S>>([&](auto k) {
    constexpr int K = decltype(k)::value;
    const int32_t e = int32_t(elem<D, S, K>(a)) - int32_t(elem<D, S, K>(b));
    const uint32_t e2 = uint32_t(__mul24(e, e));
    if constexpr (D == 8) d += __umul24(e2, weight<K>(wn));
    else d += uint64_t(e2) * weight<K>(wn);
  });
  return d;
}

// A texel's elements as 16-bit pairs, so one packed instruction handles two:
// 8-bit texels as the even and the odd bytes of each word.
template <int D, int S>
constexpr int kPairs = kElems<D, S> / 2;
template <int D, int S>
struct Pairs {
  u16x2 p[kPairs<D, S>];
};
template <int D, int S>
__device__ __forceinline__ Pairs<D, S> to_pairs(const Tx<S> &t) {
  Pairs<D, S> r;
#pragma unroll
  for (int k = 0; k < S / 4; ++k) {
    if constexpr (D == 8) {
      r.p[2 * k] = __builtin_bit_cast(u16x2, t.w[k] & 0x00FF00FFu);
      r.p[2 * k + 1] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(0u, t.w[k], 0x0C030C01u));
    } else {
      r.p[k] = __builtin_bit_cast(u16x2, t.w[k]);
    }
  }
  return r;
}
template <int D, int S>
__device__ __forceinline__ Tx<S> from_pairs(const Pairs<D, S> &r) {
  Tx<S> t;
#pragma unroll
  for (int k = 0; k < S / 4; ++k) {
    if constexpr (D == 8)
      t.w[k] = __builtin_bit_cast(uint32_t, r.p[2 * k]) |
               (__builtin_bit_cast(uint32_t, r.p[2 * k + 1]) << 8);
    else t.w[k] = __builtin_bit_cast(uint32_t, r.p[k]);
  }
  return t;
}

// What a search keeps of the style's weights: pairs like a texel's for 8-bit
// guides (the weights are bytes laid out like one), the words for 16-bit ones.
template <int D, int S>
struct Weights {
  uint32_t w[2];
  Pairs<8, 8> p;
  __device__ explicit Weights(const uint32_t *wn) {
    w[0] = wn[0], w[1] = wn[1];
    p = to_pairs<8, 8>(Tx<8>{{wn[0], wn[1]}});
  }
};

// sum_k w_k d_k^2 from q to the nearest point of each of N boxes [lo, hi]
// (their texels where lo = hi): the two saturating differences of an element
// are not both above zero, so their union is its distance to the box.  The
// last pair is left out where its elements carry no weight (five channels
// fill five bytes of eight), a branch of the whole wave.
template <int D, int S, int N>
__device__ __forceinline__ void box_dists(const Pairs<D, S> &q, const Tx<S> *lo, const Tx<S> *hi,
                                          const Weights<D, S> &wt,
                                          typename DistOf<D>::type *acc) {
  constexpr int P = kPairs<D, S>;
  Pairs<D, S> l[N], h[N];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    l[n] = to_pairs<D, S>(lo[n]), h[n] = to_pairs<D, S>(hi[n]);
    acc[n] = 0;
  }
  auto pair = [&](auto k) {
    constexpr int K = decltype(k)::value;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const u16x2 d = __builtin_elementwise_sub_sat(l[n].p[K], q.p[K]) |
                      __builtin_elementwise_sub_sat(q.p[K], h[n].p[K]);
      if constexpr (D == 8) {
        // d <= 255 and w <= 127: their product fits 16 bits
        acc[n] = __builtin_amdgcn_udot2(d, d * wt.p.p[K], acc[n], false);
      } else {
        const uint32_t d0 = d.x, d1 = d.y;
        acc[n] += uint64_t(__umul24(d0, weight<2 * K>(wt.w))) * d0;
        acc[n] += uint64_t(__umul24(d1, weight<2 * K + 1>(wt.w))) * d1;
      }
    }
  };
  for_elems<0, P == 4 ? 3 : P>(pair);
  if constexpr (P == 4) {
    const bool last = D == 8 ? __builtin_bit_cast(uint32_t, wt.p.p[3]) != 0u : wt.w[1] >> 16 != 0u;
    if (last) pair(std::integral_constant<int, 3>());
  }
}

// A distance in 29 bits, weakly monotone (so an order of packed values never
// contradicts the distances'): 8-bit ones are < 2^26, 16-bit ones < 2^42 as
// floats without their two lowest fraction bits.
__device__ __forceinline__ uint32_t pack_dist(uint32_t d) { return d; }
__device__ __forceinline__ uint32_t pack_dist(uint64_t d) {
  const float f = __builtin_fmaf(float(uint32_t(d >> 32)), 4294967296.0f, float(uint32_t(d)));
  return __builtin_bit_cast(uint32_t, f) >> 2;
}

struct TreeRef {
  const void *boxes;
  const uint32_t *keys;
  uint32_t vals;  // bytes from the boxes to the texels
  int32_t levels;
};

TreeRef tree_ref(const void *tree, size_t n, size_t t) {
  const TreeLayout l = tree_layout(n, t);
  const char *b = static_cast<const char *>(tree);
  return TreeRef{b + l.boxes, reinterpret_cast<const uint32_t *>(b + l.keys),
                 uint32_t(l.vals - l.boxes), l.levels};
}

// ... and what only the header tells: the last texel, and the level of the node
// that holds them all (a guide of few values is searched in as many steps as one
// of few texels).
struct TreeView : TreeRef {
  uint32_t last;
  int32_t top;
  __device__ __forceinline__ explicit TreeView(const TreeRef &r) : TreeRef(r) {
    const SB_GLOBAL unsigned char *b = glb(static_cast<const unsigned char *>(boxes));
    last = reinterpret_cast<const SB_GLOBAL uint32_t *>(b - kTreeHeader)[1] - 1u;
    top = levels - max((34 - int32_t(__clz(int(last)))) / 3, 1);
  }
};

// N texels from p on (dword-aligned vectors).
template <int S, int N>
__device__ __forceinline__ void load_run(const SB_GLOBAL unsigned char *p, Tx<S> *t) {
  constexpr int W = S / 4 * N, V = W % 4 == 0 ? 4 : W;  // words, words per load
  typedef uint32_t vec __attribute__((ext_vector_type(V), aligned(4)));
  vec v[W / V];
#pragma unroll
  for (int k = 0; k < W / V; ++k) v[k] = reinterpret_cast<const SB_GLOBAL vec *>(p)[k];
#pragma unroll
  for (int k = 0; k < W; ++k) t[k / (S / 4)].w[k % (S / 4)] = v[k / V][k % V];
}

// Entry e's box, among its siblings' in their parent's record.
template <int S>
__device__ __forceinline__ SB_GLOBAL unsigned char *box_at(void *boxes, uint32_t e) {
  return glb(static_cast<unsigned char *>(boxes)) +
         uint64_t(((e - 1u) >> 3) * uint32_t(16 * S) + ((e - 1u) & 7u) * uint32_t(S));
}
template <int S>
__device__ __forceinline__ void store_box(void *boxes, uint32_t e, const Tx<S> &lo,
                                          const Tx<S> &hi) {
  SB_GLOBAL uint32_t *p = reinterpret_cast<SB_GLOBAL uint32_t *>(box_at<S>(boxes, e));
#pragma unroll
  for (int k = 0; k < S / 4; ++k) p[k] = lo.w[k], p[2 * S + k] = hi.w[k];
}

// v of another lane of the row by the DPP pattern CTRL (every lane of the
// group active).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_from(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_from(uint64_t v) {
  const uint64_t lo = dpp_from<CTRL>(uint32_t(v)), hi = dpp_from<CTRL>(uint32_t(v >> 32));
  return lo | (hi << 32);
}

// v of lane ^ M.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  if constexpr (M == 1) return dpp_from<0xB1>(v);
  else if constexpr (M == 2) return dpp_from<0x4E>(v);
  else if constexpr (M == 3) return dpp_from<0x1B>(v);
  else if constexpr (M == 7) return dpp_from<0x141>(v);   // mirrored halves of a row
  else if constexpr (M == 8) return dpp_from<0x128>(v);   // a row rotated by eight
  else if constexpr (M == 15) return dpp_from<0x140>(v);  // a mirrored row
  else return uint32_t(__shfl_xor(int(v), M, 64));
}

// The least of v over each aligned group of G lanes, in every lane of the
// group (all active): lane ^ 1, lane ^ 2, then the group's two quads (lane
// 7 - i of the group).
template <int G, class T>
__device__ __forceinline__ T group_min(T v) {
  static_assert(G == 2 || G == 4 || G == 8, "groups of 2, 4 or 8 lanes");
  v = min(v, dpp_from<0xB1>(v));
  if constexpr (G >= 4) v = min(v, dpp_from<0x4E>(v));
  if constexpr (G >= 8) v = min(v, dpp_from<0x141>(v));
  return v;
}

// The exact lookup of a texel by an aligned group of G lanes, one tree node
// per step: the source coordinate x | y << 16 of the texel nearest to q under
// the weights, ties to the smallest raster index.  Lane g takes the node's
// children g N .. g N + N - 1 (N = 8 / G): their boxes come in one round
// trip, the nearest child is next and the lanes keep the others' packed
// distances in LDS, one slot per level of the path.  The least distance left
// on each level stays in a register (lane g: levels g N .. g N + N - 1), so
// the deepest level worth going back to is known without looking; nothing is
// kept in scratch memory and there is one dependent round trip per node.
//
// (best, best_key) may start at a real source texel's distance and
// coordinate (a candidate the caller already measured): every subtree that
// could hold a texel at that distance or nearer is still visited, so the
// result is the same, found with fewer steps.
//
// TURN: without one.  Texels that a median could not tell apart lie on both sides,
// so both boxes may hold the lookup of a value the guide has; if the way leaves
// boxes that hold it (packed distance 0) while one is left on the path, it goes
// there at once, up to twice: any texel it came to first would bound the search of
// its neighbourhood by its own distance, which in eight channels of noise is all
// of it (simulated on 43 000 values of a 200 x 200 guide: the longest search 9 nodes
// instead of 129; 65537 lookups 25 us, 177 without).  Only for five 16-bit channels
// and more: with 8-byte texels it saves nothing and makes a lookup's chain longer
// (65536 of five 8-bit channels 68 us, 58 without).
template <int D, int S, int G, bool TURN>
struct Search {
  typedef typename DistOf<D>::type Dist;
  static constexpr int N = 8 / G;
  static constexpr uint32_t kGone = 0xFFFFFFFFu;  // no child
  Pairs<D, S> q;
  Dist best;
  uint32_t best_key, pos, left[N];
  int32_t depth, turns;

  __device__ __forceinline__ void start(const TreeView &tv, const Tx<S> &t, Dist b, uint32_t k) {
    q = to_pairs<D, S>(t);
    best = b, best_key = k;
    pos = 0u, depth = tv.top, turns = 2;
#pragma unroll
    for (int j = 0; j < N; ++j) left[j] = kGone;
  }
  __device__ __forceinline__ static uint32_t least(const uint32_t *pk) {
    uint32_t m = pk[0];
#pragma unroll
    for (int j = 1; j < N; ++j) m = min(m, pk[j]);
    return group_min<G>(m);
  }
  // (d, k) before (e, f), as one comparison where both fit 64 bits
  __device__ __forceinline__ static bool nearer(Dist d, uint32_t k, Dist e, uint32_t f) {
    if constexpr (D == 8) return ((uint64_t(d) << 32) | k) < ((uint64_t(e) << 32) | f);
    else return (d < e) | ((d == e) & (k < f));
  }
  // From a node whose nearest child (m of pk) does not hold q, to the deepest level
  // with a child left that does (every lane of the group takes part): its children
  // and their least, with the child the path came by put back at the nearest
  // distance left under it.
  __device__ __forceinline__ void turn(const uint32_t *slots, uint32_t *pk, uint32_t &m,
                                       int32_t &level) {
    const uint32_t c0 = N * (threadIdx.x & uint32_t(G - 1));
    uint32_t back = 8u;  // 7 - level
#pragma unroll
    for (int j = 0; j < N; ++j) back = left[j] <= 7u ? 7u - c0 - uint32_t(j) : back;
    back = group_min<G>(back);
    if (back == 8u) return;
    level = int32_t(7u - back);
    uint32_t near = m;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const bool under = int32_t(c0) + j > level;
      near = under ? min(near, left[j]) : near;
      left[j] = under ? kGone : left[j];
    }
    near = group_min<G>(near);
    const uint32_t came = (pos >> (3 * (depth - 1 - level))) & 7u;
#pragma unroll
    for (int j = 0; j < N; ++j)
      pk[j] = c0 + uint32_t(j) == came ? (near & ~7u) | came : slots[64 * N * level + j];
    m = least(pk);
    --turns;
  }
  // One node; true when the search is over.  `slots`: the lane's N words of
  // level 0, a level every 64 N words.
  __device__ __forceinline__ bool step(const TreeView &tv, const Weights<D, S> &wt,
                                       uint32_t *slots) {
    const uint32_t c0 = N * (threadIdx.x & uint32_t(G - 1)), node = tree_start(depth) + pos;
    const uint32_t first = 8u * pos + c0;  // the lane's first child on its level
    const uint32_t last = tv.last >> (3 * (tv.levels - 1 - depth));  // that level's last entry
    const bool leaf = depth + 1 == tv.levels;
    // one pair of loads for either kind of children: a texel is its own box
    const uint32_t at = leaf ? tv.vals + first * uint32_t(S) : (node * 16u + c0) * uint32_t(S);
    const SB_GLOBAL unsigned char *base = glb(static_cast<const unsigned char *>(tv.boxes));
    Tx<S> lo[N], hi[N];
    load_run<S, N>(base + uint64_t(at), lo);
    load_run<S, N>(base + uint64_t(leaf ? at : at + 8u * S), hi);
    const SB_GLOBAL uint32_t *keys = glb(tv.keys) + uint64_t(8u * node + 1u + c0);
    Tx<4> key[N];
    if (leaf) load_run<4, N>(reinterpret_cast<const SB_GLOBAL unsigned char *>(keys), key);
    Dist d[N];
    box_dists<D, S, N>(q, lo, hi, wt, d);
    uint32_t pk[N], m = kGone;
    int32_t level = depth;
    if (leaf) {
      Dist dm = ~Dist(0);
      uint32_t km = kNoTreeKey;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const bool in = (first + uint32_t(j) <= last) & nearer(d[j], key[j].w[0], dm, km);
        dm = in ? d[j] : dm, km = in ? key[j].w[0] : km;
      }
      const Dist gd = group_min<G>(dm);
      const uint32_t gk = group_min<G>(dm == gd ? km : kNoTreeKey);
      const bool in = nearer(gd, gk, best, best_key);
      best = in ? gd : best, best_key = in ? gk : best_key;
    } else {
      bool tie = false;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const bool in = (first + uint32_t(j) <= last) & (d[j] <= best);
        pk[j] = in ? (pack_dist(d[j]) << 3) | (c0 + uint32_t(j)) : kGone;
        tie |= in & (d[j] == best);
      }
      if (tie) {  // seldom: as far as the best, worth a visit only for a smaller key
#pragma unroll
        for (int j = 0; j < N; ++j)
          if (pk[j] != kGone && d[j] == best && keys[j] >= best_key) pk[j] = kGone;
      }
      m = least(pk);
      if (TURN && best == ~Dist(0) && m > 7u && turns > 0) turn(slots, pk, m, level);
    }
    if (m == kGone) {
      // back to the deepest level with a child left that is not farther than
      // the best so far
      const uint32_t reach = (pack_dist(best) << 3) | 7u;
      uint32_t back = 8u;  // 7 - level of the deepest
#pragma unroll
      for (int j = 0; j < N; ++j) back = left[j] <= reach ? 7u - c0 - uint32_t(j) : back;
      back = group_min<G>(back);
      if (back == 8u) return true;
      level = int32_t(7u - back);
#pragma unroll
      for (int j = 0; j < N; ++j) pk[j] = slots[64 * N * level + j];
      m = least(pk);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) pk[j] = pk[j] == m ? kGone : pk[j];
#pragma unroll
    for (int j = 0; j < N; ++j) slots[64 * N * level + j] = pk[j];
    const uint32_t rest = least(pk);
#pragma unroll
    for (int j = 0; j < N; ++j) left[j] = uint32_t(level) == c0 + uint32_t(j) ? rest : left[j];
    pos = 8u * (pos >> (3 * (depth - level))) + (m & 7u);
    depth = level + 1;
    return false;
  }
};

// LDS bytes of a 256-thread workgroup's searches (Search::step's slots: one
// level of the path per tree level above the texels).
template <int G>
unsigned stack_bytes(int32_t levels) {
  return unsigned(levels - 1) * 256u * (8u / G) * 4u;
}
template <int G>
__device__ __forceinline__ uint32_t *lane_slots(const TreeView &tv, uint32_t *stack) {
  return stack + (8 / G) * (64u * uint32_t(tv.levels - 1) * (threadIdx.x >> 6) +
                            (threadIdx.x & 63u));
}

template <int D, int S, int G>
__device__ uint32_t tree_search(const TreeView &tv, const Tx<S> &q, const uint32_t *wn,
                                uint32_t *stack) {
  typedef typename DistOf<D>::type Dist;
  const Weights<D, S> wt(wn);
  uint32_t *slots = lane_slots<G>(tv, stack);
  Search<D, S, G, S == 16> s;
  s.start(tv, q, ~Dist(0), kNoTreeKey);
  while (!s.step(tv, wt, slots)) {
  }
  return s.best_key;
}

// ---------------------------------------------------------------- tree build

// Words of a segment's box: every element's lowest value, then the inverse
// of its highest, so that both are minima.
template <int D, int S>
constexpr uint32_t kBoxWords = 2 * kElems<D, S>;

// The distinct texels in the order of the splits so far, and their number.
struct TexelsIn {
  const void *vals;
  const uint32_t *keys, *n;
};

struct SplitArgs {
  TexelsIn in;
  void *vals_out;
  uint32_t *keys_out;
  uint32_t *boxes, *hist, *ctr;  // per segment: kBoxWords, kBins, 4 words
  int32_t level, lg;             // this level's segments hold 2^lg texels
  int32_t last;                  // the children are k_tree_sort's blocks
  uint32_t wn[2];                // build weights (split choice only)
  int32_t channels;
};

// The element a node is split by: the widest by weight, else by raw range; not
// element `but`.
template <int D, int S>
__device__ __forceinline__ int32_t split_axis(const uint32_t *lo, const uint32_t *hi,
                                              const uint32_t *wn, int32_t channels,
                                              int32_t but = -1) {
  int32_t ds = -1, dr = 0;
  uint64_t best_w = 0;
  uint32_t best_r = 0;
#pragma unroll
  for (int k = 0; k < kElems<D, S>; ++k) {
    if (k >= channels || k == but) continue;
    const uint32_t r = hi[k] - lo[k];
    const uint64_t wr = uint64_t(r) * r * ((wn[k >> 2] >> ((k & 3) * 8)) & 0xFFu);
    if (wr > best_w) best_w = wr, ds = k;
    if (r > best_r) best_r = r, dr = k;
  }
  return ds < 0 ? dr : ds;
}

// Element ds (not a compile-time constant) of a texel.
template <int D, int S>
__device__ __forceinline__ uint32_t elem_at(const Tx<S> &t, int32_t ds) {
  constexpr int32_t kLog = D == 8 ? 2 : 1;  // elements per word
  uint32_t w = t.w[0];
#pragma unroll
  for (int k = 1; k < S / 4; ++k) w = (ds >> kLog) == k ? t.w[k] : w;
  return D == 8 ? (w >> ((ds & 3) * 8)) & 0xFFu : (w >> ((ds & 1) * 16)) & 0xFFFFu;
}

template <int D, int S>
struct Box {
  Pairs<D, S> lo, hi;
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < kPairs<D, S>; ++k) lo.p[k] = u16x2{0xFFFF, 0xFFFF}, hi.p[k] = u16x2{0, 0};
  }
  __device__ __forceinline__ void add(const Pairs<D, S> &l, const Pairs<D, S> &h) {
#pragma unroll
    for (int k = 0; k < kPairs<D, S>; ++k) {
      lo.p[k] = __builtin_elementwise_min(lo.p[k], l.p[k]);
      hi.p[k] = __builtin_elementwise_max(hi.p[k], h.p[k]);
    }
  }
  // joined with the box of lane ^ M
  template <int M>
  __device__ __forceinline__ void join() {
    Pairs<D, S> l, h;
#pragma unroll
    for (int k = 0; k < kPairs<D, S>; ++k) {
      l.p[k] = __builtin_bit_cast(u16x2, lane_xor<M>(__builtin_bit_cast(uint32_t, lo.p[k])));
      h.p[k] = __builtin_bit_cast(u16x2, lane_xor<M>(__builtin_bit_cast(uint32_t, hi.p[k])));
    }
    add(l, h);
  }
  // joined over aligned groups of n lanes (a power of two)
  __device__ __forceinline__ void join_lanes(uint32_t n) {
    if (n > 1) join<1>();
    if (n > 2) join<2>();
    if (n > 4) join<7>();
    if (n > 8) join<15>();
    if (n > 16) join<16>();
    if (n > 32) join<32>();
  }
  __device__ __forceinline__ void elems(uint32_t *l, uint32_t *h) const {
    const Tx<S> tl = from_pairs<D, S>(lo), th = from_pairs<D, S>(hi);
    for_elems<0, kElems<D, S>>([&](auto k) {
      constexpr int K = decltype(k)::value;
      l[K] = elem<D, S, K>(tl), h[K] = elem<D, S, K>(th);
    });
  }
  // into a segment's box words, by one lane
  __device__ __forceinline__ void widen(uint32_t *words) const {
    uint32_t l[kElems<D, S>], h[kElems<D, S>];
    elems(l, h);
#pragma unroll
    for (int k = 0; k < kElems<D, S>; ++k) {
      atomicMin(words + k, l[k]);
      atomicMin(words + kElems<D, S> + k, ~h[k]);
    }
  }
};

// Clears what the build accumulates into: words of all ones at a and at b,
// zeros at c.
__global__ void __launch_bounds__(256) k_tree_clear(uint32_t *a, uint32_t na, uint32_t *b,
                                                    uint32_t nb, uint32_t *c, uint32_t nc) {
  const uint32_t step = gridDim.x * 256u, first = blockIdx.x * 256u + threadIdx.x;
  for (uint32_t i = first; i < na; i += step) glb(a)[i] = 0xFFFFFFFFu;
  for (uint32_t i = first; i < nb; i += step) glb(b)[i] = 0xFFFFFFFFu;
  for (uint32_t i = first; i < nc; i += step) glb(c)[i] = 0u;
}

// The table that equal texels meet in, by open addressing: per slot the smallest
// raster index of one value's texels, all ones where empty.
struct MergeArgs {
  const void *guide;
  uint32_t n, sw;
  uint32_t *table;
  uint32_t slots;    // a power of two, at least 3 n
  uint32_t mask[4];  // the channels' bits of a texel's words
  uint8_t *dup;      // per texel: 1 where an equal one has a smaller index
};
constexpr uint32_t kNoTexel = 0xFFFFFFFFu;
constexpr uint32_t kMergeThreads = 1024;

template <int S>
__device__ __forceinline__ bool same_texel(const Tx<S> &a, const Tx<S> &b, const uint32_t *mask) {
  uint32_t x = 0;
#pragma unroll
  for (int k = 0; k < S / 4; ++k) x |= (a.w[k] ^ b.w[k]) & mask[k];
  return x == 0u;
}

// Texels equal in every channel are one to a search, and a tree that holds each
// many times has whole levels of boxes at one distance, all of which a lookup has
// to enter (a constant 512 x 512 guide: 65536 lookups 202 us, 6.4 with one texel).
// So every texel but the first of its value is marked: whenever two equal ones
// meet, the one of larger index.  The texels of a workgroup meet in LDS first (the
// smallest index of each hash's place there, so a texel equal to that one is done):
// a constant region sends one of a workgroup's 1024 to the slot that all of them
// share, where atomics follow one another at 16 ns.  A texel whose place went to
// another value has a second one, from other bits: with one alone, two values that
// share it and fill a guide send half of all texels to one slot (512 x 512 of two
// such values register in 126 us, 1755 with one place).  A probe that finds another
// value's slot goes on by an odd step of the hash; a third of the slots or fewer are
// ever taken, so chains are short.  Bound by them and by the round trips before: 17 us
// for 512 x 512 texels (23 with two thirds taken).
template <int S>
__global__ void __launch_bounds__(kMergeThreads) k_tree_merge(MergeArgs a) {
  __shared__ uint32_t first[2][kMergeThreads];
  const uint32_t tid = threadIdx.x, i = blockIdx.x * kMergeThreads + tid;
  const Tx<S> t = load_tx<S>(a.guide, min(i, a.n - 1u));
  uint32_t h = 0;
#pragma unroll
  for (int k = 0; k < S / 4; ++k) {
    h = (h ^ (t.w[k] & a.mask[k])) * 0x9E3779B1u;  // 2^32 over the golden ratio
    h ^= h >> 15;
  }
  h *= 0x9E3779B1u;
  h ^= h >> 16;
  first[0][tid] = first[1][tid] = kNoTexel;
  __syncthreads();
  const bool in = i < a.n;
  bool dup = false, done = !in;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    uint32_t *place = &first[r][(r ? h >> 4 : h >> 16) % kMergeThreads];
    if (!done) atomicMin(place, i);
    __syncthreads();
    const uint32_t f = *place;
    if (!done && f != i) dup = same_texel<S>(load_tx<S>(a.guide, f), t, a.mask);
    done |= dup | (f == i);
  }
  if (dup) a.dup[i] = 1;
  if (dup || !in) return;
  for (uint32_t s = h;; s += (h >> 12) | 1u) {
    uint32_t *slot = a.table + (s & (a.slots - 1u));
    uint32_t v = atomicCAS(slot, kNoTexel, i);
    if (v == kNoTexel) return;
    if (!same_texel<S>(load_tx<S>(a.guide, v), t, a.mask)) continue;
    v = atomicMin(slot, i);  // the slot is the value's for good, its index falls
    a.dup[max(v, i)] = 1;
    return;
  }
}

// The unmarked texels one after another (in raster order within a workgroup's:
// texels that a split cannot tell apart stay beside their neighbours), with their
// coordinates and (with `box`) the box of them all.
constexpr uint32_t kTakePer = 8;
template <int D, int S>
__global__ void __launch_bounds__(256) k_tree_take(MergeArgs a, void *vals, uint32_t *keys,
                                                   uint32_t *count, uint32_t *box) {
  __shared__ uint32_t words[kBoxWords<D, S>], wave_n[4], base;
  const uint32_t tid = threadIdx.x, wave = tid >> 6;
  if (tid < kBoxWords<D, S>) words[tid] = 0xFFFFFFFFu;
  const uint32_t i0 = (blockIdx.x * 4u + wave) * (64u * kTakePer) + (tid & 63u);
  uint32_t at[kTakePer], n = 0;
  bool has[kTakePer];
  Tx<S> t[kTakePer];
#pragma unroll
  for (uint32_t k = 0; k < kTakePer; ++k) {
    const uint32_t i = min(i0 + 64u * k, a.n - 1u);
    t[k] = load_tx<S>(a.guide, i);
    has[k] = i0 + 64u * k < a.n && glb(a.dup)[i] == 0;
  }
#pragma unroll
  for (uint32_t k = 0; k < kTakePer; ++k) {
    const uint64_t m = __ballot(has[k]);
    at[k] = n + __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
    n += uint32_t(__popcll(m));
  }
  if ((tid & 63u) == 0) wave_n[wave] = n;
  __syncthreads();
  if (tid == 0) base = atomicAdd(count, wave_n[0] + wave_n[1] + wave_n[2] + wave_n[3]);
  __syncthreads();
  uint32_t from = base;
  for (uint32_t w = 0; w < wave; ++w) from += wave_n[w];
  Box<D, S> b;
  b.clear();
#pragma unroll
  for (uint32_t k = 0; k < kTakePer; ++k) {
    if (!has[k]) continue;
    const uint32_t i = i0 + 64u * k;
    store_tx<S>(vals, from + at[k], t[k]);
    glb(keys)[from + at[k]] = ((i / a.sw) << 16) | (i % a.sw);
    const Pairs<D, S> p = to_pairs<D, S>(t[k]);
    b.add(p, p);
  }
  if (!box) return;
  b.join_lanes(64);
  if ((tid & 63u) == 0) b.widen(words);
  __syncthreads();
  if (tid < kBoxWords<D, S>) atomicMin(box + tid, words[tid]);
}

// A level's segment of a workgroup (kSplitBlock texels, so one segment) and
// how it is split.
template <int D, int S>
struct Segment {
  uint32_t id, first, count, half, lo;
  int32_t axis, shift;
  __device__ __forceinline__ Segment(const SplitArgs &a, uint32_t n) {
    const uint32_t seg = blockIdx.x >> (a.lg - int32_t(kSplitLog));
    id = (1u << a.level) - 1u + seg;
    first = seg << a.lg;
    count = min(n - first, 1u << a.lg);
    half = 1u << (a.lg - 1);
    const SB_GLOBAL uint32_t *box = glb(a.boxes) + size_t(id) * kBoxWords<D, S>;
    uint32_t l[kElems<D, S>], h[kElems<D, S>];
#pragma unroll
    for (int k = 0; k < kElems<D, S>; ++k) l[k] = box[k], h[k] = ~box[kElems<D, S> + k];
    axis = split_axis<D, S>(l, h, a.wn, a.channels);
    lo = 0;
    uint32_t range = 0;
#pragma unroll
    for (int k = 0; k < kElems<D, S>; ++k)
      if (k == axis) lo = l[k], range = h[k] - l[k];
    const int32_t bits = 32 - __clz(int(range));
    shift = max(bits - int32_t(kBinsLog), 0);
  }
  // a texel's bin: its value along the axis, in at most kBins steps
  __device__ __forceinline__ uint32_t bin(const Tx<S> &t) const {
    return (elem_at<D, S>(t, axis) - lo) >> shift;
  }
};

constexpr uint32_t kSplitPer = kSplitBlock / kSplitThreads;

// First half of a level's splits: the histogram of every segment's texels
// along its axis.
template <int D, int S>
__global__ void __launch_bounds__(kSplitThreads) k_tree_hist(SplitArgs a) {
  __shared__ uint32_t bins[kBins];
  const uint32_t n = glb(a.in.n)[0];
  if (blockIdx.x * kSplitBlock >= n) return;
  const Segment<D, S> sg(a, n);
  if (sg.count <= sg.half) return;  // all of it goes left
  const uint32_t tid = threadIdx.x;
#pragma unroll
  for (uint32_t k = 0; k < kBins; k += kSplitThreads) bins[k + tid] = 0u;
  __syncthreads();
  const uint32_t i0 = blockIdx.x * kSplitBlock + tid;
  Tx<S> t[kSplitPer];
#pragma unroll
  for (uint32_t k = 0; k < kSplitPer; ++k)
    t[k] = load_tx<S>(a.in.vals, min(i0 + kSplitThreads * k, n - 1));
#pragma unroll
  for (uint32_t k = 0; k < kSplitPer; ++k)
    if (i0 + kSplitThreads * k < n) atomicAdd(&bins[sg.bin(t[k])], 1u);
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < kBins; k += kSplitThreads)
    if (bins[k + tid] != 0u) atomicAdd(a.hist + size_t(sg.id) * kBins + k + tid, bins[k + tid]);
}

// Second half: the texels move to their child's range of the other buffer.
// The median's bin is the one that the left child's last place falls in;
// texels below it go left, above it right, and as many of the bin's own as
// the left child has places for.  Places within a class are dealt to the
// segment's workgroups by three counters (the tree's shape follows from the
// guide up to the order of a bin's texels; a search's result does not depend
// on it).  On the way the children's boxes are taken.
template <int D, int S>
__global__ void __launch_bounds__(kSplitThreads) k_tree_split(SplitArgs a) {
  constexpr uint32_t W = kSplitThreads / 64;
  __shared__ uint32_t part[W], found[3], wave_n[W][3], base[3];
  __shared__ uint32_t box[2 * kBoxWords<D, S>];
  const uint32_t total = glb(a.in.n)[0];
  if (blockIdx.x * kSplitBlock >= total) return;
  const Segment<D, S> sg(a, total);
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  if (tid < 2 * kBoxWords<D, S>) box[tid] = 0xFFFFFFFFu;
  const uint32_t i0 = blockIdx.x * kSplitBlock + tid;
  Tx<S> t[kSplitPer];
  uint32_t key[kSplitPer];
#pragma unroll
  for (uint32_t k = 0; k < kSplitPer; ++k) {
    const uint32_t i = min(i0 + kSplitThreads * k, total - 1);
    t[k] = load_tx<S>(a.in.vals, i);
    key[k] = glb(a.in.keys)[i];
  }
  uint32_t mid = kBins, below = sg.count, same = 0u;  // all left
  if (sg.count > sg.half) {
    const SB_GLOBAL uint32_t *hist = glb(a.hist) + size_t(sg.id) * kBins;
    uint32_t h[kBins / kSplitThreads], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kBins / kSplitThreads; ++k) sum += h[k] = hist[(kBins / kSplitThreads) * tid + k];
    uint32_t incl = sum;
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
      const uint32_t v = uint32_t(__shfl_up(int(incl), o, 64));
      if (lane >= o) incl += v;
    }
    if (lane == 63) part[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (uint32_t w = 0; w < wave; ++w) run += part[w];
#pragma unroll
    for (uint32_t k = 0; k < kBins / kSplitThreads; ++k) {
      if (run <= sg.half && sg.half < run + h[k])
        found[0] = (kBins / kSplitThreads) * tid + k, found[1] = run, found[2] = h[k];
      run += h[k];
    }
    __syncthreads();
    mid = found[0], below = found[1], same = found[2];
  }
  const uint32_t take = sg.half - min(below, sg.half);  // of the median's bin, to the left
  uint32_t rank[kSplitPer], cls[kSplitPer], n[3] = {0u, 0u, 0u};
  const uint64_t under = (1ull << lane) - 1ull;
#pragma unroll
  for (uint32_t k = 0; k < kSplitPer; ++k) {
    const uint32_t b = sg.bin(t[k]);
    // 0 below the median's bin, 1 in it, 2 above, 3 no texel
    cls[k] = i0 + kSplitThreads * k >= total ? 3u : b < mid ? 0u : b == mid ? 1u : 2u;
    rank[k] = 0u;
#pragma unroll
    for (uint32_t c = 0; c < 3; ++c) {
      const uint64_t m = __ballot(cls[k] == c);
      if (cls[k] == c) rank[k] = n[c] + uint32_t(__popcll(m & under));
      n[c] += uint32_t(__popcll(m));
    }
  }
  if (lane < 3) wave_n[wave][lane] = lane == 0 ? n[0] : lane == 1 ? n[1] : n[2];
  __syncthreads();
  if (tid < 3) {
    uint32_t sum = 0;
    for (uint32_t w = 0; w < W; ++w) sum += wave_n[w][tid];
    base[tid] = atomicAdd(a.ctr + size_t(sg.id) * 4 + tid, sum);
  }
  __syncthreads();
  uint32_t at[3];
#pragma unroll
  for (uint32_t c = 0; c < 3; ++c) {
    at[c] = base[c];
    for (uint32_t w = 0; w < wave; ++w) at[c] += wave_n[w][c];
  }
  Box<D, S> left, right;
  left.clear();
  right.clear();
#pragma unroll
  for (uint32_t k = 0; k < kSplitPer; ++k) {
    if (cls[k] == 3u) continue;
    const uint32_t r = rank[k] + (cls[k] == 0u ? at[0] : cls[k] == 1u ? at[1] : at[2]);
    const bool l = cls[k] == 0u || (cls[k] == 1u && r < take);
    const uint32_t place = cls[k] == 0u   ? r
                           : cls[k] == 1u ? (l ? below + r : sg.half + (r - take))
                                          : sg.half + (same - take) + r;
    store_tx<S>(a.vals_out, sg.first + place, t[k]);
    glb(a.keys_out)[sg.first + place] = key[k];
    const Pairs<D, S> p = to_pairs<D, S>(t[k]);
    if (l) left.add(p, p);
    else right.add(p, p);
  }
  if (a.last) return;
  left.join_lanes(64);
  right.join_lanes(64);
  if (lane == 0) {
    left.widen(box);
    right.widen(box + kBoxWords<D, S>);
  }
  __syncthreads();
  // the segment's children are neighbours in the next level
  if (tid < 2 * kBoxWords<D, S>)
    atomicMin(a.boxes + size_t(2u * sg.id + 1u) * kBoxWords<D, S> + tid, box[tid]);
}

struct SortArgs {
  TexelsIn in;
  void *boxes, *vals;
  uint32_t *keys;
  int32_t levels;
  uint32_t wn[2];
  int32_t channels;
};

// Bitonic sorting of kSortBlock keys in ascending segments of 2^lg, thread t
// holding places 4 t .. 4 t + 3: places up to three apart are exchanged in
// registers, within a wave's 256 by lane moves, beyond that through `ky`.
struct Sorter {
  uint32_t v[4];
  __device__ __forceinline__ static void order(uint32_t &a, uint32_t &b) {
    const uint32_t x = min(a, b);
    b = max(a, b), a = x;
  }
  __device__ __forceinline__ void near() {  // places 2, then 1 apart
    order(v[0], v[2]), order(v[1], v[3]);
    order(v[0], v[1]), order(v[2], v[3]);
  }
  // keep the lesser (upper: the greater) of each place and its partner's
  __device__ __forceinline__ void keep(const uint32_t *o, bool upper) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = upper ? max(v[r], o[r]) : min(v[r], o[r]);
  }
  // places J, J / 2 .. 1 apart (J <= 128)
  template <int J>
  __device__ __forceinline__ void merge() {
    if constexpr (J >= 4) {
      uint32_t o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = lane_xor<J / 4>(v[r]);
      keep(o, (threadIdx.x & (J / 4)) != 0);
      merge<J / 2>();
    } else {
      near();
    }
  }
  // runs of K / 2 into runs of K, up to a wave's 256 places
  template <int K>
  __device__ __forceinline__ void stage(uint32_t size) {
    if constexpr (K <= 256) {
      if (K > size) return;
      uint32_t o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = lane_xor<K / 4 - 1>(v[3 - r]);
      keep(o, (threadIdx.x & (K / 8)) != 0);
      merge<K / 4>();
      stage<2 * K>(size);
    }
  }
  __device__ __forceinline__ void far(uint32_t partner, bool flip, bool upper, uint32_t *ky) {
    __syncthreads();
    u32x4 *k4 = reinterpret_cast<u32x4 *>(ky);
    k4[threadIdx.x] = u32x4{v[0], v[1], v[2], v[3]};
    __syncthreads();
    const u32x4 q = k4[partner];
    const uint32_t o[4] = {flip ? q.w : q.x, flip ? q.z : q.y, flip ? q.y : q.z, flip ? q.x : q.w};
    keep(o, upper);
  }
  __device__ __forceinline__ void sort(uint32_t size, uint32_t *ky) {
    const uint32_t t = threadIdx.x;
    order(v[0], v[1]), order(v[2], v[3]);
    order(v[0], v[3]), order(v[1], v[2]);
    order(v[0], v[1]), order(v[2], v[3]);
    stage<8>(size);
    for (uint32_t k = 512; k <= size; k <<= 1) {
      far(t ^ (k / 4 - 1u), true, (t & (k / 8)) != 0, ky);
      for (uint32_t j = k / 4; j >= 256; j >>= 1) far(t ^ (j / 4), false, (t & (j / 4)) != 0, ky);
      merge<128>();
    }
  }
};

// The last kSortLog - 3 splits of kSortBlock texels: at every size 2^lg the
// block's segments take their boxes and axes and are sorted along them (on
// value, value along the next widest element, texel), which leaves each segment's
// halves split at the median.  (A median among texels at one value would deal them
// to both sides with boxes that overlap: 65536 lookups of a guide in eighths of its
// range take 38 us without the second element and 29 with it, its 1080p frame 696
// and 587.)  Then the texels' entries and those of the three levels above them
// are written.  Bound by the chain of exchanges (276 of them, 128 blocks for a
// 512 x 512 style): 35 us; 75 with every exchange through LDS.
template <int D, int S>
__global__ void __launch_bounds__(512) k_tree_sort(SortArgs a) {
  __shared__ Tx<S> tex[kSortBlock];
  __shared__ __attribute__((aligned(16))) uint32_t ky[kSortBlock];
  __shared__ Box<D, S> wbox[8];
  __shared__ uint32_t wkey[8];
  constexpr uint32_t kNone = 0xFFFFFFFFu;  // past the last texel: sorts behind every one
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t n = glb(a.in.n)[0], first = blockIdx.x * kSortBlock;
  if (first >= n) return;
  const uint32_t count = min(n - first, kSortBlock);
#pragma unroll
  for (uint32_t k = 0; k < kSortBlock; k += 512) {
    const uint32_t i = k + tid;
    if (i < count) tex[i] = load_tx<S>(a.in.vals, first + i);
  }
  __syncthreads();
  Sorter st;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) st.v[j] = 4 * tid + j < count ? 4 * tid + j : kNone;
  for (uint32_t lg = kSortLog; lg >= 4; --lg) {
    Box<D, S> b;
    b.clear();
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      if (st.v[j] != kNone) {
        st.v[j] &= kSortBlock - 1u;
        const Pairs<D, S> p = to_pairs<D, S>(tex[st.v[j]]);
        b.add(p, p);
      }
    }
    b.join_lanes(min(1u << (lg - 2), 64u));
    if (lg > 8) {  // the segment's waves
      if (lane == 0) wbox[wave] = b;
      __syncthreads();
      const uint32_t nw = 1u << (lg - 8), w0 = wave & ~(nw - 1u);
      for (uint32_t w = 0; w < nw; ++w) b.add(wbox[w0 + w].lo, wbox[w0 + w].hi);
    }
    uint32_t l[kElems<D, S>], h[kElems<D, S>];
    b.elems(l, h);
    const int32_t axis = split_axis<D, S>(l, h, a.wn, a.channels);
    // texels at one value of the axis by the next widest element
    const int32_t next = split_axis<D, S>(l, h, a.wn, a.channels, axis);
    uint32_t lo = 0, range = 0;
#pragma unroll
    for (int k = 0; k < kElems<D, S>; ++k)
      if (k == next) lo = l[k], range = h[k] - l[k];
    constexpr int32_t kNextBits = D == 8 ? 8 : 4;
    const int32_t shift = max(32 - __clz(int(range)) - kNextBits, 0);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      if (st.v[j] == kNone) continue;
      const Tx<S> t = tex[st.v[j]];
      st.v[j] |= (elem_at<D, S>(t, axis) << (kSortLog + kNextBits)) |
                 (((elem_at<D, S>(t, next) - lo) >> shift) << kSortLog);
    }
    st.sort(1u << lg, ky);
  }
  Box<D, S> b;
  b.clear();
  uint32_t mk = kNoTreeKey;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) {
    const uint32_t v = st.v[j];
    if (v == kNone) continue;
    const Tx<S> t = tex[v & (kSortBlock - 1u)];
    const uint32_t key = glb(a.in.keys)[first + (v & (kSortBlock - 1u))];
    store_tx<S>(a.vals, first + 4 * tid + j, t);
    glb(a.keys)[tree_start(a.levels) + first + 4 * tid + j] = key;
    const Pairs<D, S> p = to_pairs<D, S>(t);
    b.add(p, p);
    mk = min(mk, key);
  }
  // node p of the level `up` above the texels, where it exists
  auto node = [&](int32_t up, uint32_t p) {
    if (up >= a.levels || mk == kNoTreeKey) return;
    const uint32_t e = tree_start(a.levels - up) + p;
    store_box<S>(a.boxes, e, from_pairs<D, S>(b.lo), from_pairs<D, S>(b.hi));
    glb(a.keys)[e] = mk;
  };
  b.template join<1>();
  mk = min(mk, lane_xor<1>(mk));
  if ((lane & 1u) == 0) node(1, (first + 4 * tid) >> 3);
  b.template join<2>(), mk = min(mk, lane_xor<2>(mk));
  b.template join<7>(), mk = min(mk, lane_xor<7>(mk));
  b.template join<15>(), mk = min(mk, lane_xor<15>(mk));
  if ((lane & 15u) == 0) node(2, (first + 4 * tid) >> 6);
  b.template join<16>(), mk = min(mk, lane_xor<16>(mk));
  b.template join<32>(), mk = min(mk, lane_xor<32>(mk));
  if (lane == 0) wbox[wave] = b, wkey[wave] = mk;
  __syncthreads();
  if (lane == 0 && (wave & 1u) == 0) {
    b.add(wbox[wave + 1].lo, wbox[wave + 1].hi);
    mk = min(mk, wkey[wave + 1]);
    node(3, (first + 4 * tid) >> 9);
  }
}

// The levels above k_tree_sort's (one workgroup: at most 2^17 nodes' records
// are read), and the header.
template <int D, int S>
__global__ void __launch_bounds__(1024) k_tree_top(void *boxes, uint32_t *keys, int32_t levels,
                                                   const uint32_t *count, uint32_t *header,
                                                   uint32_t channels) {
  const uint32_t n = glb(count)[0];
  for (int32_t up = 4; up < levels; ++up) {
    const uint32_t kids = uint32_t((uint64_t(n) + (1ull << (3 * up - 3)) - 1) >> (3 * up - 3));
    const uint32_t from = tree_start(levels - up + 1), to = tree_start(levels - up);
    for (uint32_t i = threadIdx.x; 8u * i < kids; i += 1024) {
      Box<D, S> b;
      b.clear();
      uint32_t mk = kNoTreeKey;
      for (uint32_t c = 8 * i; c < min(8 * i + 8, kids); ++c) {
        const SB_GLOBAL unsigned char *p = box_at<S>(boxes, from + c);
        Tx<S> lo, hi;
        load_run<S, 1>(p, &lo);
        load_run<S, 1>(p + 8 * S, &hi);
        b.add(to_pairs<D, S>(lo), to_pairs<D, S>(hi));
        mk = min(mk, glb(keys)[from + c]);
      }
      store_box<S>(boxes, to + i, from_pairs<D, S>(b.lo), from_pairs<D, S>(b.hi));
      glb(keys)[to + i] = mk;
    }
    __syncthreads();
  }
  // (searches read the number of texels)
  if (threadIdx.x == 0) {
    glb(header)[0] = tree_start(levels) + n;
    glb(header)[1] = n;
    glb(header)[2] = S;
    glb(header)[3] = channels;
  }
}

// ------------------------------------------------------------- frame passes

__device__ inline TreeView frame_tree(const FrameArgs &a) {
  return TreeView(TreeRef{a.t_boxes, a.t_keys, a.t_vals, a.t_levels});
}

// Record idx of the padded seed table: the seed of its cell and the
// translation u* - q of the seed's search, eight lanes per record (too few
// records to fill the chip with fewer lanes each, and the pass takes as long
// as its longest search).
template <int D, int S>
__global__ void __launch_bounds__(256) k_seeds_n(FrameArgs a) {
  extern __shared__ uint32_t stack[];
  const uint32_t idx = (blockIdx.x * 256 + threadIdx.x) >> 3, g = threadIdx.x & 7u;
  const Levels &lv = a.lv;
  if (idx >= uint32_t(lv.poffset[lv.count])) return;
  int32_t i = 0;
  while (idx >= uint32_t(lv.poffset[i + 1])) ++i;
  const uint32_t local = idx - uint32_t(lv.poffset[i]), pc = uint32_t(lv.cells_x[i] + 2);
  const int32_t cx = int32_t(local % pc) - 1, cy = int32_t(local / pc) - 1;
  const int32_t ls = lv.log2_spacing[i];
  u32x2 rec = {kNoSeed, 0u};
  if (cx >= 0 && cy >= 0 && cx < lv.cells_x[i] && cy < lv.cells_y[i]) {
    const uint32_t j = cell_jitter(a, ls, lv.cells_x[i], lv.offset[i], a.jhash[i], cx, cy);
    const uint32_t sx = (uint32_t(cx) << ls) + (j & 0xFFFFu);
    const uint32_t sy = (uint32_t(cy) << ls) + (j >> 16);
    if (sx < uint32_t(a.w) && sy < uint32_t(a.h)) {
      const uint32_t at = __umul24(sy, uint32_t(a.w)) + sx;
      const uint32_t u =
          tree_search<D, S, 8>(frame_tree(a), load_tx<S>(a.tgt_guide, at), a.wn, stack);
      rec.x = pack_xy(4 * sx, 4 * sy);
      rec.y = pack_off(int32_t(u & 0xFFFFu) - int32_t(sx), int32_t(u >> 16) - int32_t(sy));
    }
  }
  if (g == 0) seed_table(a)[idx] = rec;
}

// The level loop where every cell holds whole 8 x 8 blocks (finest spacing >=
// 8): a wave takes one block, stages the block's nine seed records of every
// level in LDS, and each lane tests its pixel against two levels at a time,
// both levels' source texels requested together.  Against the loop per pixel
// below, which reads its nine records per level itself, 23 us instead of 32
// for a five-channel 1080p frame.  A pixel no level accepts takes the fallback
// code, and its vote-distance slot the nearest candidate measured (its
// coordinate, or none), from which k_fallback_n starts the pixel's own search.
template <int D, int S>
__global__ void __launch_bounds__(256) k_assign_blocks_n(FrameArgs a) {
  typedef typename DistOf<D>::type Dist;
  constexpr int32_t kStride = 12, kRecs = kStride * SB_MAX_LEVELS;
  __shared__ __attribute__((aligned(16))) uint32_t recs[4][2 * kRecs];
  const int32_t lane = int32_t(threadIdx.x & 63u);
  const int32_t wave = __builtin_amdgcn_readfirstlane(int32_t(threadIdx.x >> 6));
  const uint32_t tiles_x = (uint32_t(a.w) + 15u) / 16u;
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const int32_t bx0 = int32_t((tile % tiles_x) * 16u) + (wave & 1) * 8;
  const int32_t by0 = int32_t((tile / tiles_x) * 16u) + (wave >> 1) * 8;
  if (bx0 >= a.w || by0 >= a.h) return;
  uint32_t *pos = recs[wave], *off = pos + kRecs;
  const Levels &lv = a.lv;
  const int32_t L = lv.count;
  const int32_t x = bx0 + (lane & 7), y = by0 + (lane >> 3);
  const bool in = x < a.w && y < a.h;
  const uint32_t pidx = in ? __umul24(uint32_t(y), uint32_t(a.w)) + uint32_t(x) : 0u;
  const Tx<S> gt = load_tx<S>(a.tgt_guide, pidx);
#pragma unroll
  for (int32_t r = 0; r < 2; ++r) {
    const uint32_t j = uint32_t(lane + 64 * r);
    if (j < uint32_t(9 * L)) {
      const uint32_t i = (j * 57u) >> 9, k = j - 9u * i, kx = (k * 11u) >> 5;  // x outer, y inner
      const int32_t ls = lv.log2_spacing[0] - int32_t(i);
      const int32_t pc = ((a.w - 1) >> ls) + 3;  // cells_x + 2
      int32_t f = lv.poffset[0];
      for (int32_t l = 1; l < L; ++l) f = i >= uint32_t(l) ? lv.poffset[l] : f;
      const u32x2 rec =
          seed_table(a)[f + ((by0 >> ls) + int32_t(k - 3u * kx)) * pc + (bx0 >> ls) + int32_t(kx)];
      pos[kStride * int32_t(i) + int32_t(k)] = rec.x;
      off[kStride * int32_t(i) + int32_t(k)] = rec.y;
    }
  }
  wave_lds_sync();
  const Weights<D, S> wt(a.wn);
  const Pairs<D, S> q = to_pairs<D, S>(gt);
  const ushort2_t p = __builtin_bit_cast(ushort2_t, pack_xy(uint32_t(x), uint32_t(y)));
  const short2_t p4 = __builtin_bit_cast(short2_t, pack_xy(uint32_t(4 * x), uint32_t(4 * y)));
  const ushort2_t last = __builtin_bit_cast(
      ushort2_t, pack_xy(uint32_t(a.sw - 1), uint32_t(a.sh - 1)));
  const ushort2_t row = __builtin_bit_cast(ushort2_t, pack_xy(1u, uint32_t(a.sw)));
  bool done = !in;
  uint32_t seed = 0, level = 0, offset = 0, ckey = 0xFFFFFFFFu;
  Dist cd = ~Dist(0);
  for (int32_t i0 = 0; i0 < L; i0 += 2) {
    if (__all(done)) break;
    uint32_t wq[2], wo[2];
    ushort2_t v[2];
    bool ok[2];
    Tx<S> t[2];
#pragma unroll
    for (int32_t u = 0; u < 2; ++u) {
      const uint32_t *P = pos + kStride * min(i0 + u, L - 1);
      const uint32_t *O = off + kStride * min(i0 + u, L - 1);
      const u32x4 q03 = *reinterpret_cast<const u32x4 *>(P);
      const u32x4 q47 = *reinterpret_cast<const u32x4 *>(P + 4);
      int32_t key = seed_key(P[8], p4, 8);
#pragma unroll
      for (int32_t k = 0; k < 4; ++k) {
        key = min(key, seed_key(q03[k], p4, k));
        key = min(key, seed_key(q47[k], p4, k + 4));
      }
      wq[u] = P[key & 15], wo[u] = O[key & 15];
      // a coordinate below 0 wraps past every exemplar's last texel
      v[u] = p + __builtin_bit_cast(ushort2_t, wo[u]);
      const uint32_t vin =
          __builtin_bit_cast(uint32_t, __builtin_elementwise_min(v[u], last));
      ok[u] = (i0 + u < L) & (key != INT32_MAX) & (vin == __builtin_bit_cast(uint32_t, v[u]));
      const uint32_t at = __builtin_amdgcn_udot2(v[u], row, 0u, false);
      t[u] = load_tx<S>(a.src_guide, ok[u] ? at : 0u);
    }
#pragma unroll
    for (int32_t u = 0; u < 2; ++u) {
      Dist e[1];
      box_dists<D, S, 1>(q, &t[u], &t[u], wt, e);
      const bool take = (!done) & ok[u] & (e[0] < a.threshold);
      seed = take ? wq[u] : seed, level = take ? uint32_t(i0 + u) : level;
      offset = take ? wo[u] : offset;
      done = done | take;
      const uint32_t vkey = __builtin_bit_cast(uint32_t, v[u]);
      const bool better = ok[u] & ((e[0] < cd) | ((e[0] == cd) & (vkey < ckey)));
      cd = better ? e[0] : cd, ckey = better ? vkey : ckey;
    }
  }
  if (!in) return;
  if (done) {
    glb(a.out_chunk)[pidx] = chunk_code(int32_t(level), seed);
    glb(a.offsets)[pidx] = vote_distance(a, offset);
    if (a.out_nnf)
      glb(a.out_nnf)[pidx] =
          __builtin_bit_cast(uint32_t, p + __builtin_bit_cast(ushort2_t, offset));
  } else {
    glb(a.out_chunk)[pidx] = (uint32_t(L) << 26) | (uint32_t(y) << 13) | uint32_t(x);
    glb(a.offsets)[pidx] = ckey;
  }
}

// The level loop per pixel, for finer hierarchies.
constexpr uint32_t kAssignTW = 64, kAssignTH = 16;

template <int D, int S>
__global__ void __launch_bounds__(256) k_assign_n(FrameArgs a) {
  typedef typename DistOf<D>::type Dist;
  const uint32_t tid = threadIdx.x;
  const uint32_t tiles_x = (uint32_t(a.w) + kAssignTW - 1) / kAssignTW;
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const int32_t tx0 = int32_t((tile % tiles_x) * kAssignTW);
  const int32_t ty0 = int32_t((tile / tiles_x) * kAssignTH);
  const Levels &lv = a.lv;
  const int32_t L = lv.count;
  const uint32_t sw = uint32_t(a.sw), sh = uint32_t(a.sh);
#pragma unroll 1
  for (int32_t r = 0; r < int32_t(kAssignTH / 4); ++r) {
    const int32_t x = tx0 + int32_t(tid & 63u), y = ty0 + int32_t(tid >> 6) + 4 * r;
    if (x >= a.w || y >= a.h) continue;
    const uint32_t pidx = __umul24(uint32_t(y), uint32_t(a.w)) + uint32_t(x);
    const Tx<S> gt = load_tx<S>(a.tgt_guide, pidx);
    const short2_t p4 = __builtin_bit_cast(short2_t, pack_xy(uint32_t(4 * x), uint32_t(4 * y)));
    bool done = false;
    Dist cd = ~Dist(0);
    uint32_t ckey = 0xFFFFFFFFu;
    for (int32_t i = 0; i < L && !done; ++i) {
      const int32_t ls = lv.log2_spacing[i], pc = lv.cells_x[i] + 2;
      const SB_GLOBAL u32x2 *top = seed_table(a) + lv.poffset[i] + (y >> ls) * pc + (x >> ls);
      int32_t key = INT32_MAX;
#pragma unroll
      for (int32_t k = 0; k < 9; ++k) key = min(key, seed_key(top[(k % 3) * pc + k / 3].x, p4, k));
      if (key == INT32_MAX) continue;
      const int32_t k = key & 15, kx = (k * 11) >> 5;
      const u32x2 rec = top[(k - 3 * kx) * pc + kx];
      const int32_t vx = x + off_x(rec.y), vy = y + off_y(rec.y);
      if (uint32_t(vx) >= sw || uint32_t(vy) >= sh) continue;
      const uint32_t vidx = __umul24(uint32_t(vy), sw) + uint32_t(vx);
      const Dist e = tx_dist<D, S>(gt, load_tx<S>(a.src_guide, vidx), a.wn);
      if (e < a.threshold) {
        glb(a.out_chunk)[pidx] = chunk_code(i, rec.x);
        glb(a.offsets)[pidx] = vote_distance(a, rec.y);
        if (a.out_nnf) glb(a.out_nnf)[pidx] = pack_xy(uint32_t(vx), uint32_t(vy));
        done = true;
      }
      const uint32_t vkey = pack_xy(uint32_t(vx), uint32_t(vy));
      if (e < cd || (e == cd && vkey < ckey)) cd = e, ckey = vkey;
    }
    if (!done) {
      // no level accepts: the fallback code, and in the vote-distance slot
      // the nearest candidate measured (its coordinate, or none), from
      // which k_fallback_n starts the pixel's own search
      glb(a.out_chunk)[pidx] = (uint32_t(L) << 26) | (uint32_t(y) << 13) | uint32_t(x);
      glb(a.offsets)[pidx] = ckey;
    }
  }
}

// The own lookups of the pixels no level accepted (fallback chunk code).
// Those pixels cluster (whole tiles fall back beside tiles where none does)
// and searches differ in length, so work is dealt as it is taken: a wave
// draws another 8 x 4 tile whenever its list of pixels runs short, and its
// groups of G lanes take the list's next pixels as their searches end (once
// two wait: a search's first load holds up the whole wave).  A search starts
// from the candidate the level loop left in the vote-distance slot (its
// distance measured again here, for the whole tile at once), then the slot
// takes the result's vote distance.
//
// The tiles drawn are counted in the seed table, which has served its purpose
// by now: the offset words of the finest level's empty records left of its
// rows, which the seed pass writes as 0 and nothing reads.  One counter would
// be too few (draws of one word follow one another at 16 ns: 32640 of them
// made the pass take 0.8 ms), so up to 64 counters deal every 64th tile each.
// Without levels there is no table; every pixel falls back then, and the
// waves take every n-th tile.
//
// Bound by VALU issue (64 % of the chip's over the pass, 215 instructions per
// node of a wave's 32 searches) and by the last searches.  The 414 k searches
// of a 1080p frame with five 8-bit channels: 337 us; one search per lane in
// the linked binary tree took 1300.  Fixed 16 x 16 tiles per workgroup 440,
// draws of 8 x 8 370; four lanes per search instead of two 350 (for four
// 16-bit channels 610 k searches in 245, and 320 with four lanes).
constexpr uint32_t kFallbackQueue = 64;  // under 64 / G <= 32 waiting and a tile's 32

template <int D, int S, int G>
__global__ void __launch_bounds__(256) k_fallback_n(FrameArgs a) {
  typedef typename DistOf<D>::type Dist;
  struct Entry {
    uint32_t xy, key;
    Dist dist;
  };
  extern __shared__ uint32_t stack[];
  __shared__ Entry queues[4][kFallbackQueue];
  const uint32_t lane = threadIdx.x & 63u;
  Entry *queue = queues[threadIdx.x >> 6];
  const uint32_t tiles_x = (uint32_t(a.w) + 7u) / 8u;
  const uint32_t tiles = tiles_x * ((uint32_t(a.h) + 3u) / 4u);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * 4u + (threadIdx.x >> 6));
  const int32_t L = a.lv.count;
  uint32_t *drawn = nullptr;
  uint32_t next = wave, stride = gridDim.x * 4u;
  if (L > 0) {
    const uint32_t rows = uint32_t(a.lv.cells_y[L - 1] + 2);
    stride = min(min(rows, 64u), stride);  // counters, each with a wave at least
    next = wave % stride;
    drawn = &a.seeds[a.lv.poffset[L - 1] + int32_t(next) * (a.lv.cells_x[L - 1] + 2)].y;
  }
  uint32_t head = 0, fill = 0;  // the list: places head .. head + fill - 1
  bool more = true;
  const TreeView tv = frame_tree(a);
  const Weights<D, S> wt(a.wn);
  uint32_t *slots = lane_slots<G>(tv, stack);
  Search<D, S, G, false> s;
  s.start(tv, Tx<S>{}, 0, 0u);
  uint32_t xy = 0, pidx = 0;
  bool busy = false;
  for (;;) {
    const uint64_t idle = __ballot(!busy);
    const uint32_t waiting = uint32_t(__popcll(idle)) / G;
    if (waiting >= 2u && (more || fill != 0u)) {
      while (more && fill < waiting) {
        uint32_t tile = next;
        if (drawn) {
          uint32_t t = 0;
          if (lane == 0) t = atomicAdd(drawn, 1u);
          tile += __builtin_amdgcn_readfirstlane(t) * stride;
        } else {
          next += stride;
        }
        more = tile < tiles;
        const uint32_t ty = tile / tiles_x;
        const uint32_t x = (tile - ty * tiles_x) * 8u + (lane & 7u), y = ty * 4u + (lane >> 3);
        const uint32_t at = __umul24(y, uint32_t(a.w)) + x;
        bool need = more && lane < 32u && x < uint32_t(a.w) && y < uint32_t(a.h);
        uint32_t code = 0, ckey = 0;
        Tx<S> gt = {};
        if (need) {
          code = glb(a.out_chunk)[at], ckey = glb(a.offsets)[at];
          gt = load_tx<S>(a.tgt_guide, at);
        }
        need = need && (code >> 26) == uint32_t(L);
        const uint64_t bal = __ballot(need);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
            uint32_t(bal >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(bal), 0u));
        if (need) {
          Dist cd = ~Dist(0);
          if (ckey != 0xFFFFFFFFu) {
            const uint32_t cidx = __umul24(ckey >> 16, uint32_t(a.sw)) + (ckey & 0xFFFFu);
            cd = tx_dist<D, S>(gt, load_tx<S>(a.src_guide, cidx), a.wn);
          }
          queue[(head + fill + below) % kFallbackQueue] = Entry{pack_xy(x, y), ckey, cd};
        }
        fill += uint32_t(__popcll(bal));
      }
      wave_lds_sync();
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
                                uint32_t(idle >> 32),
                                __builtin_amdgcn_mbcnt_lo(uint32_t(idle), 0u)) / G;
      if (!busy && rank < fill) {
        busy = true;
        const Entry en = queue[(head + rank) % kFallbackQueue];
        xy = en.xy;
        pidx = __umul24(xy >> 16, uint32_t(a.w)) + (xy & 0xFFFFu);
        s.start(tv, load_tx<S>(a.tgt_guide, pidx), en.dist, en.key);
      }
      wave_lds_sync();
      const uint32_t took = min(waiting, fill);
      head += took, fill -= took;
    }
    if (__ballot(busy) == 0ull) break;  // (the waiting groups found no pixel left)
    if (busy && s.step(tv, wt, slots)) {
      busy = false;
      if ((lane & uint32_t(G - 1)) == 0) {
        const uint32_t u = s.best_key;
        const uint32_t off = pack_off(int32_t(u & 0xFFFFu) - int32_t(xy & 0xFFFFu),
                                      int32_t(u >> 16) - int32_t(xy >> 16));
        glb(a.offsets)[pidx] = vote_distance(a, off);
        if (a.out_nnf) glb(a.out_nnf)[pidx] = u;
      }
    }
  }
}

// G lanes per query texel.
template <int D, int S, int G>
__global__ void __launch_bounds__(256) k_tree_query(TreeRef tree, const void *q, uint32_t n,
                                                    uint32_t *out, uint32_t w0, uint32_t w1) {
  extern __shared__ uint32_t stack[];
  const uint64_t i = (uint64_t(blockIdx.x) * 256 + threadIdx.x) / G;
  if (i >= n) return;
  const uint32_t wn[2] = {w0, w1};
  const uint32_t u = tree_search<D, S, G>(TreeView(tree), load_tx<S>(q, uint32_t(i)), wn,
                                          stack);
  if ((threadIdx.x & uint32_t(G - 1)) == 0) glb(out)[i] = u;
}

// Lanes per search of the fallback pass (measured there), and up to how many
// queries eight lanes take one rather than four: eight give the shorter chain
// while all searches are on the chip at once (65536 of five channels 58 us,
// 69 with four lanes, 90 with two), four more searches per instruction beyond.
constexpr int kFallbackLanes = 2;
constexpr int64_t kQueryWide = 65536;
// Queries of one launch: a grid has fewer than 2^32 threads.
constexpr int64_t kQueryLaunch = int64_t(1) << 29;
// Workgroups of the fallback pass: what the chip holds.
constexpr unsigned kFallbackGrid = 2048;

// ------------------------------------------------------------------- host

template <int V>
using IC = std::integral_constant<int, V>;

// Calls f(depth, texel bytes) with both as integral constants for the
// guide's format and texel size.
template <class F>
hipError_t with_format(int32_t fmt, int32_t texel, F &&f) {
  if (fmt == SB_GUIDE_U8XN) {
    if (texel == 4) return f(IC<8>(), IC<4>());
    if (texel == 8) return f(IC<8>(), IC<8>());
  } else if (fmt == SB_GUIDE_U16XN) {
    if (texel == 4) return f(IC<16>(), IC<4>());
    if (texel == 8) return f(IC<16>(), IC<8>());
    if (texel == 16) return f(IC<16>(), IC<16>());
  }
  return hipErrorInvalidValue;
}

unsigned blocks_for(uint64_t n, unsigned bs) { return unsigned((n + bs - 1) / bs); }

bool side_ok(int32_t v) { return v >= 1 && v <= SB_MAX_SIDE; }

// The build's workspace: the texels and keys of two consecutive levels of
// splits, the table of distinct texels, per segment of the levels split over the
// chip its box, its histogram and its counters, the number of distinct texels and
// the marks of the others.
struct BuildWs {
  void *vals[2];
  uint32_t *keys[2];
  uint32_t *table, *boxes, *hist, *ctr, *count;
  uint8_t *dup;
  uint32_t slots, box_words, zero_words;  // (zero: hist, ctr, count and dup)
  int32_t splits;                         // levels split over the chip
  size_t total;
};

BuildWs build_ws(char *base, size_t n, size_t t) {
  constexpr size_t kWidest = 16;  // box words of eight elements
  BuildWs w;
  w.splits = 0;
  while ((size_t(kSortBlock) << w.splits) < n) ++w.splits;
  const size_t segs = (size_t(1) << w.splits) - 1;  // at most n / 1024
  size_t slots = 2;
  while (slots < 3 * n) slots *= 2;
  w.slots = uint32_t(slots);
  w.box_words = uint32_t(segs * kWidest);
  w.zero_words = uint32_t(segs * (kBins + 4) + 1 + (n + 3) / 4);
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char *p = base ? base + at : nullptr;
    at += align256(bytes);
    return p;
  };
  for (int k = 0; k < 2; ++k) w.vals[k] = take(n * t);
  for (int k = 0; k < 2; ++k) w.keys[k] = reinterpret_cast<uint32_t *>(take(n * 4));
  // the table and the boxes, cleared to ones in one run, lie one after the other
  char *p = take((slots + w.box_words + w.zero_words) * 4);
  w.total = at;
  w.table = reinterpret_cast<uint32_t *>(p);
  w.boxes = p ? w.table + slots : nullptr;
  w.hist = p ? w.boxes + w.box_words : nullptr;
  w.ctr = p ? w.hist + segs * kBins : nullptr;
  w.count = p ? w.ctr + segs * 4 : nullptr;
  w.dup = reinterpret_cast<uint8_t *>(p ? w.count + 1 : nullptr);
  return w;
}

}  // namespace

bool resolve_weights_n(const uint8_t *in, int32_t channels, uint32_t out[2]) {
  out[0] = out[1] = 0u;
  bool any = false;
  for (int32_t k = 0; in && k < channels; ++k) any |= in[k] != 0;
  for (int32_t k = 0; k < channels; ++k) {
    const uint32_t w = any ? in[k] : 1u;
    if (w > 127u) return false;
    out[k >> 2] |= w << ((k & 3) * 8);
  }
  return true;
}

hipError_t launch_search_frame(const FrameArgs &a, hipEvent_t *ev, hipStream_t stream) {
  const uint32_t records = uint32_t(a.lv.poffset[a.lv.count]);
  const uint32_t tiles = ((uint32_t(a.w) + kAssignTW - 1) / kAssignTW) *
                         ((uint32_t(a.h) + kAssignTH - 1) / kAssignTH);
  const uint32_t btiles = ((uint32_t(a.w) + 15u) / 16u) * ((uint32_t(a.h) + 15u) / 16u);
  return with_format(a.fmt, a.texel, [&](auto d, auto s) -> hipError_t {
    constexpr int D = decltype(d)::value, S = decltype(s)::value;
    if (records > 0)
      k_seeds_n<D, S><<<blocks_for(uint64_t(records) * 8, 256), 256, stack_bytes<8>(a.t_levels),
                        stream>>>(a);
    if (ev) {
      const hipError_t e = hipEventRecord(ev[1], stream);
      if (e != hipSuccess) return e;
    }
    if (a.lv.count > 0 && a.lv.log2_spacing[a.lv.count - 1] >= 3)
      k_assign_blocks_n<D, S><<<btiles, 256, 0, stream>>>(a);
    else
      k_assign_n<D, S><<<tiles, 256, 0, stream>>>(a);
    const uint32_t ftiles = ((uint32_t(a.w) + 7u) / 8u) * ((uint32_t(a.h) + 3u) / 4u);
    const unsigned fblocks = ftiles < 4 * kFallbackGrid ? blocks_for(ftiles, 4) : kFallbackGrid;
    k_fallback_n<D, S, kFallbackLanes>
        <<<fblocks, 256, stack_bytes<kFallbackLanes>(a.t_levels), stream>>>(a);
    return hipGetLastError();
  });
}

}  // namespace sb

using namespace sb;

extern "C" {

int32_t sb_texel_bytes(int32_t fmt, int32_t channels) { return search_texel_bytes(fmt, channels); }

size_t sb_tree_bytes(int32_t fmt, int32_t channels, int32_t sw, int32_t sh) {
  const int32_t t = search_texel_bytes(fmt, channels);
  if (t == 0 || !side_ok(sw) || !side_ok(sh)) return 0;
  return tree_layout(size_t(sw) * size_t(sh), size_t(t)).total;
}

size_t sb_tree_workspace_bytes(int32_t fmt, int32_t channels, int32_t sw, int32_t sh) {
  const int32_t t = search_texel_bytes(fmt, channels);
  if (t == 0 || !side_ok(sw) || !side_ok(sh)) return 0;
  return build_ws(nullptr, size_t(sw) * size_t(sh), size_t(t)).total;
}

int sb_tree_build(const void *guide, int32_t fmt, int32_t channels, int32_t sw, int32_t sh,
                  const uint8_t *weights, void *tree, size_t tree_bytes, void *workspace,
                  size_t workspace_bytes, hipStream_t stream) {
  const int32_t t = search_texel_bytes(fmt, channels);
  if (!guide || !tree || !workspace || t == 0 || !side_ok(sw) || !side_ok(sh)) return SB_EINVAL;
  uint32_t wn[2];
  if (!resolve_weights_n(weights, channels, wn)) return SB_EINVAL;
  const uint32_t n = uint32_t(sw) * uint32_t(sh);
  const TreeLayout l = tree_layout(n, size_t(t));
  if (tree_bytes < l.total) return SB_ENOMEM;
  const BuildWs ws = build_ws(static_cast<char *>(workspace), n, size_t(t));
  if (workspace_bytes < ws.total) return SB_ENOMEM;
  char *tb = static_cast<char *>(tree);
  uint32_t *keys = reinterpret_cast<uint32_t *>(tb + l.keys);
  hipError_t e = with_format(fmt, t, [&](auto d, auto s) -> hipError_t {
    constexpr int D = decltype(d)::value, S = decltype(s)::value;
    const unsigned nblk = blocks_for(n, kSortBlock);
    const uint32_t ones = ws.slots + ws.box_words;
    const uint32_t most = l.entries > ones ? l.entries : ones;
    k_tree_clear<<<blocks_for(most, 256) < 2048 ? blocks_for(most, 256) : 2048, 256, 0, stream>>>(
        keys, l.entries, ws.table, ones, ws.hist, ws.zero_words);
    MergeArgs m = {guide, n, uint32_t(sw), ws.table, ws.slots, {0u, 0u, 0u, 0u}, ws.dup};
    for (int32_t k = 0; k < channels; ++k)
      m.mask[k * D / 32] |= (D == 8 ? 0xFFu : 0xFFFFu) << (k * D % 32);
    k_tree_merge<S><<<blocks_for(n, kMergeThreads), kMergeThreads, 0, stream>>>(m);
    k_tree_take<D, S><<<blocks_for(n, 256 * kTakePer), 256, 0, stream>>>(
        m, ws.vals[1], ws.keys[1], ws.count, ws.splits > 0 ? ws.boxes : nullptr);
    TexelsIn in = {ws.vals[1], ws.keys[1], ws.count};
    for (int32_t lv = 0; lv < ws.splits; ++lv) {
      SplitArgs a;
      a.in = in;
      a.vals_out = ws.vals[lv & 1];
      a.keys_out = ws.keys[lv & 1];
      a.boxes = ws.boxes;
      a.hist = ws.hist;
      a.ctr = ws.ctr;
      a.level = lv;
      a.lg = int32_t(kSortLog) + ws.splits - lv;
      a.last = lv + 1 == ws.splits;
      a.wn[0] = wn[0];
      a.wn[1] = wn[1];
      a.channels = channels;
      k_tree_hist<D, S><<<blocks_for(n, kSplitBlock), kSplitThreads, 0, stream>>>(a);
      k_tree_split<D, S><<<blocks_for(n, kSplitBlock), kSplitThreads, 0, stream>>>(a);
      in.vals = a.vals_out;
      in.keys = a.keys_out;
    }
    const SortArgs a = {in, tb + l.boxes, tb + l.vals, keys, l.levels, {wn[0], wn[1]}, channels};
    k_tree_sort<D, S><<<nblk, 512, 0, stream>>>(a);
    k_tree_top<D, S><<<1, 1024, 0, stream>>>(tb + l.boxes, keys, l.levels, ws.count,
                                             reinterpret_cast<uint32_t *>(tb), uint32_t(channels));
    const hipError_t ec = hipGetLastError();
    if (ec != hipSuccess) return ec;
    // returns with the tree complete and the workspace idle
    return hipStreamSynchronize(stream);
  });
  if (e != hipSuccess) {
    set_hip_error(e, "sb_tree_build");
    return SB_EHIP;
  }
  return SB_OK;
}

int sb_tree_query(const sb_style *style, const void *queries, int64_t n, uint32_t *out,
                  hipStream_t stream) {
  if (!style || !fmt_search(style->fmt) || !style->tree || !queries || !out || n < 0 ||
      n > int64_t(UINT32_MAX) || !side_ok(style->sw) || !side_ok(style->sh))
    return SB_EINVAL;
  const int32_t t = search_texel_bytes(style->fmt, style->channels);
  uint32_t wn[2];
  if (t == 0 || !resolve_weights_n(style->weights, style->channels, wn)) return SB_EINVAL;
  if (n == 0) return SB_OK;
  const TreeRef tree = tree_ref(style->tree, size_t(style->sw) * size_t(style->sh), size_t(t));
  hipError_t e = with_format(style->fmt, t, [&](auto d, auto s) -> hipError_t {
    constexpr int D = decltype(d)::value, S = decltype(s)::value;
    for (int64_t at = 0; at < n; at += kQueryLaunch) {
      const uint32_t m = uint32_t(n - at < kQueryLaunch ? n - at : kQueryLaunch);
      const void *q = static_cast<const char *>(queries) + at * S;
      if (n <= kQueryWide)
        k_tree_query<D, S, 8><<<blocks_for(uint64_t(m) * 8, 256), 256,
                                stack_bytes<8>(tree.levels), stream>>>(tree, q, m, out + at,
                                                                       wn[0], wn[1]);
      else
        k_tree_query<D, S, 4><<<blocks_for(uint64_t(m) * 4, 256), 256,
                                stack_bytes<4>(tree.levels), stream>>>(tree, q, m, out + at,
                                                                       wn[0], wn[1]);
    }
    return hipGetLastError();
  });
  if (e != hipSuccess) {
    set_hip_error(e, "sb_tree_query");
    return SB_EHIP;
  }
  return SB_OK;
}

}  // extern "C"

namespace sb {
// The tree sections a frame of a search-format style reads.
void fill_tree_args(const sb_style *style, FrameArgs *a) {
  const int32_t t = search_texel_bytes(style->fmt, style->channels);
  const TreeRef tree = tree_ref(style->tree, size_t(style->sw) * size_t(style->sh), size_t(t));
  a->t_boxes = tree.boxes;
  a->t_vals = tree.vals;
  a->t_keys = tree.keys;
  a->t_levels = tree.levels;
  a->texel = t;
  resolve_weights_n(style->weights, style->channels, a->wn);
}
}  // namespace sb
