// Backward fused with the sparse SGD update (Algorithms 2-3, fused as the end
// of Section III-A describes), for gfx950, without float atomics.
//
// Input: the look-ups sorted by row key (ties in look-up order), as
// (key << 32 | bag) words.  The sorted list is cut into chunks of C look-ups,
// one per row group of LPR lanes; the row groups of a block walk neighbouring
// chunks.  A row group gathers dY[bag] for each look-up (U row loads in flight
// per lane) and adds it to an FP64 accumulator; when the key changes, the
// finished segment is applied, W[row] <- W[row] - lr * G (the W row was
// requested with the look-up that began it).  A segment that crosses chunks is
// applied by the row group where it begins, which keeps its own sum and the W
// row in registers and, after the block's one barrier, adds the sums that the
// following row groups parked in LDS.  A segment that crosses blocks leaves
// two sums in global memory (slot 2b: block b's part of a segment begun before
// it, slot 2b+1: of one going on past it) and is applied by a second kernel;
// where it may cross very many, a kernel between them adds up groups of blocks.
// Every touched row is read and written exactly once, and its sum is taken in
// an order that positions alone decide (the result is bit-reproducible).
//
// Chunks are short, because a walk is a chain of dependent loads and a small
// call has few of them: with the partial sums in LDS a boundary costs an LDS
// write and read instead of 2 * 8 * E bytes of global memory and a fix-up.
// Measured against chunks of 128 look-ups per wavefront whose crossing
// segments all went through global memory and two more kernels (update of
// plain sums, from a graph): 53K look-ups of E = 128 split rows 45 -> 18 us,
// 59K of E = 64 28 -> 12, 81K of E = 512 111 -> 54, 524K of E = 64 51 -> 42,
// 4.4M of E = 16 179 -> 100, 13.1M of E = 256 1688 -> 1670.
//
// Locality: each XCD owns one contiguous range of blocks, so the dY rows it
// gathers at any time belong to one or two tables, unless eight tables' dY
// would fill more than half of the MALL: then the blocks are walked in
// dispatch order, and all XCDs gather from the dY of the table in progress,
// which the MALL holds.  The W rows, touched once, are read and written with
// non-temporal hints so they do not evict dY.
//
// Sorted positions are unsigned 32-bit: num_indices may be 2^31 - 1, and the
// last block's chunks start at most a block (2^16 look-ups) past it, which
// stays below 2^32.
#include <type_traits>

#include "common.hpp"

namespace embbag {
namespace {

template <class T>
using Global = __attribute__((address_space(1))) T*;

// Element `off` of a row of S at `row`, as a pointer to V.
template <class V, class S>
__device__ __forceinline__ Global<V> at(Global<S> row, int off) {
  return (Global<V>)(row + off);
}

// Row update for FP32 tables: w <- fl(w - lr * G), G in FP64.  A Row is where a
// row of a table lies (kept from its load to its store), a Pre what it holds.
struct Fp32Rows {
  struct Table {
    Global<float> w;
  };
  struct Row {
    Global<float> w;
  };
  struct Pre {
    f4 w;
  };
  template <class D>
  static __device__ __forceinline__ Table table(const D& d, int t) {
    return {(Global<float>)static_cast<float*>(d.w[t])};
  }
  static __device__ __forceinline__ Row row(const Table& t, uint32_t r, uint32_t E) {
    return {t.w + size_t(r) * E};
  }
  static __device__ __forceinline__ Pre load(const Row& r, int c4) {
    return {__builtin_nontemporal_load(at<const f4>(r.w, c4 * 4))};
  }
  static __device__ __forceinline__ void store(const Row& r, int c4, const Pre& p, const d4& g,
                                               double lr) {
    f4 o;
    o.x = float(double(p.w.x) - lr * g.x);
    o.y = float(double(p.w.y) - lr * g.y);
    o.z = float(double(p.w.z) - lr * g.z);
    o.w = float(double(p.w.w) - lr * g.w);
    __builtin_nontemporal_store(o, at<f4>(r.w, c4 * 4));
  }
};

// Row update for split tables (Section VII): recombine hi/lo into the FP32
// weight, apply the FP32 update, split the result again.
struct SplitRows {
  struct Table {
    Global<uint16_t> hi, lo;
  };
  struct Row {
    Global<uint16_t> hi, lo;
  };
  struct Pre {
    u2 hi, lo;
  };
  template <class D>
  static __device__ __forceinline__ Table table(const D& d, int t) {
    return {(Global<uint16_t>)static_cast<uint16_t*>(d.w[t]),
            (Global<uint16_t>)static_cast<uint16_t*>(d.lo[t])};
  }
  static __device__ __forceinline__ Row row(const Table& t, uint32_t r, uint32_t E) {
    const size_t off = size_t(r) * E;
    return {t.hi + off, t.lo + off};
  }
  static __device__ __forceinline__ Pre load(const Row& r, int c4) {
    return {__builtin_nontemporal_load(at<const u2>(r.hi, c4 * 4)),
            __builtin_nontemporal_load(at<const u2>(r.lo, c4 * 4))};
  }
  static __device__ __forceinline__ float upd(uint32_t hi16, uint32_t lo16, double g, double lr) {
    const float w = __uint_as_float((hi16 << 16) | lo16);
    return float(double(w) - lr * g);
  }
  static __device__ __forceinline__ void store(const Row& r, int c4, const Pre& p, const d4& g,
                                               double lr) {
    const uint32_t w0 = __float_as_uint(upd(p.hi.x & 0xFFFFu, p.lo.x & 0xFFFFu, g.x, lr));
    const uint32_t w1 = __float_as_uint(upd(p.hi.x >> 16, p.lo.x >> 16, g.y, lr));
    const uint32_t w2 = __float_as_uint(upd(p.hi.y & 0xFFFFu, p.lo.y & 0xFFFFu, g.z, lr));
    const uint32_t w3 = __float_as_uint(upd(p.hi.y >> 16, p.lo.y >> 16, g.w, lr));
    u2 hi, lo;
    hi.x = (w0 >> 16) | (w1 & 0xFFFF0000u);
    hi.y = (w2 >> 16) | (w3 & 0xFFFF0000u);
    lo.x = (w0 & 0xFFFFu) | (w1 << 16);
    lo.y = (w2 & 0xFFFFu) | (w3 << 16);
    __builtin_nontemporal_store(hi, at<u2>(r.hi, c4 * 4));
    __builtin_nontemporal_store(lo, at<u2>(r.lo, c4 * 4));
  }
};

// Four gradient values of dY row `bag` as loaded (FP32, or BF16 bit patterns);
// BF16 values are widened exactly only when summed, so that the loads of a
// group stay in flight together.
template <bool GBF16>
struct Dy {
  using Raw = typename std::conditional<GBF16, u2, f4>::type;
  static __device__ __forceinline__ Raw load(const void* dY, uint32_t bag, uint32_t E, int c4) {
    if constexpr (!GBF16)
      return *reinterpret_cast<const f4*>(static_cast<const float*>(dY) + size_t(bag) * E + c4 * 4);
    else
      return *reinterpret_cast<const u2*>(static_cast<const uint16_t*>(dY) + size_t(bag) * E +
                                          c4 * 4);
  }
  static __device__ __forceinline__ Raw zero() {
    if constexpr (!GBF16)
      return f4{0.f, 0.f, 0.f, 0.f};
    else
      return u2{0u, 0u};
  }
  static __device__ __forceinline__ f4 value(const Raw& r) {
    if constexpr (!GBF16)
      return r;
    else
      return f4{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xFFFF0000u),
                __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xFFFF0000u)};
  }
};

__device__ __forceinline__ d4 widen(const f4& v) {
  return d4{double(v.x), double(v.y), double(v.z), double(v.w)};
}

// One row group's partial sum in global memory (slot `slot` of E doubles).
template <int CPL>
__device__ __forceinline__ void store_carry(double* carry, int64_t slot, int E, int rl, int lpr,
                                            const d4* acc) {
  double* c = carry + slot * E;
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    const int c4 = rl + j * lpr;
    if (c4 < E / 4) *reinterpret_cast<d4*>(c + c4 * 4) = acc[j];
  }
}

// Look-up coefficients of the gradient sum (Section II's weights a_p): 1 for
// plain sums, the look-up's weight for weighted sums (the weights sorted
// along with the look-ups, so read in sorted order), 1/|bag| for means.
struct PoolDev {
  const float* svals;
  const int32_t* offsets;
};


// Row groups of a block (each walks one chunk).
template <int LPR>
constexpr int kGroups = kBlock / LPR;

template <int LPR, int CPL, class Rows, int MODE, bool GBF16>
__global__ __launch_bounds__(kBlock) void segment_sgd(
    TableDesc d, const uint64_t* __restrict__ sorted, int32_t NS, int32_t C,
    const void* __restrict__ dY, int32_t B, float inv_b, float lr,
    double* __restrict__ carry, const int32_t* __restrict__ flags, uint32_t token, PoolDev pd,
    int32_t in_order) {
  constexpr int NG = kGroups<LPR>;
  __shared__ TableLds tl;
  __shared__ d4 part[NG * LPR * CPL];  // per row group: its first segment's sum, if open
  // whether that segment goes on past the row group's chunk: per row group, or
  // per wavefront and lane
  constexpr bool kMany = NG >= 32;
  __shared__ uint8_t thru[NG];
  __shared__ uint64_t through[kWavesPerBlock];
  if constexpr (LPR < kWave) {
    stage_tables(d, tl);
    __syncthreads();
  }
  const auto& tb = table_view<(LPR < kWave)>(d, tl);
  // A data error, or no sort result for these sizes: no table writes.
  if (flags[0] != 0 || uint32_t(flags[1]) != token) return;
  constexpr int R = kWave / LPR;
  // look-ups in flight per row group: fewer when a wave holds several row
  // groups (their (key, bag) words no longer share scalar registers)
  constexpr int U = CPL == 1 ? (LPR == kWave ? 8 : 4) : (CPL == 2 ? 4 : 2);
  const int E = d.dim;
  const int E4 = E / 4;  // float4 groups per row
  const int lane = lane_id();
  const int rg = lane / LPR, rl = lane % LPR;
  const int blk = int(logical_block(in_order != 0));
  const int grp = wave_id() * R + rg;
  const uint32_t lo = (uint32_t(blk) * NG + uint32_t(grp)) * uint32_t(C);
  const uint32_t hi = lo < uint32_t(NS) ? min(lo + uint32_t(C), uint32_t(NS)) : lo;
  const double lrd = double(lr);
  constexpr bool kW = MODE == kPoolWeighted;

  const uint32_t kprev = lo > 0 && lo < hi ? key_of(sorted[lo - 1]) : kNoKey;
  const uint32_t knext = hi < uint32_t(NS) ? key_of(sorted[hi]) : kNoKey;
  // Software pipeline: the (key, bag) words of the next U look-ups are loaded
  // while the current ones are summed; for the current U look-ups, the dY rows
  // (skipped when a look-up repeats the previous (key, bag) pair: its row is
  // still in registers) and the W rows of the segments that start among them
  // are all requested before the first of them is used.
  // Weighted bags: each look-up's weight is loaded one group ahead, with its
  // word (the weights were sorted along with the look-ups).
  uint64_t pn[U];
  float an[U];
#pragma unroll
  for (int u = 0; u < U; ++u) pn[u] = lo + u < hi ? sorted[lo + u] : 0ull;
  if constexpr (kW) {
#pragma unroll
    for (int u = 0; u < U; ++u) an[u] = lo + u < hi ? pd.svals[lo + u] : 0.f;
  }
  const uint64_t p0 = pn[0];
  // The first segment began before lo (and still is the one being summed).
  const bool before = lo < hi && kprev == key_of(p0);
  bool open = before;
  uint32_t cur = key_of(p0);
  // The table at hand: keys [kfirst, kend).  Keys increase, so it is looked up
  // again only where a walk crosses into the next one, and a row's place is
  // kept from its load to its store: at narrow rows the issue of instructions
  // takes a third of the time (75 -> about 50 per look-up of four row groups;
  // 525K weighted look-ups of E = 100 74 -> 70 us, 81K of E = 512 54 -> 51, 13.1M
  // split of E = 256 1750 -> 1700).
  uint32_t kfirst = 0, kend = 0;
  typename Rows::Table tab;
  auto row_of = [&](uint64_t word) {
    if (key_of(word) >= kend) {
      const int t = table_of_bag(bag_of(word), B, inv_b);
      kfirst = tb.rowbase[t];
      kend = tb.rowbase[t + 1];
      tab = Rows::table(tb, t);
    }
    return Rows::row(tab, key_of(word) - kfirst, E);
  };

  d4 acc[CPL];
  f4 glast[CPL];
  int col[CPL];  // columns past the row's end load its last ones and store nothing
  typename Rows::Row row;
  typename Rows::Pre pre[CPL];
  if (lo < hi) row = row_of(p0);
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    acc[j] = d4{0.0, 0.0, 0.0, 0.0};
    glast[j] = f4{0.f, 0.f, 0.f, 0.f};
    col[j] = min(rl + j * LPR, E4 - 1);
    if (lo < hi && !open) pre[j] = Rows::load(row, col[j]);
  }

  auto apply = [&]() {
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      if (rl + j * LPR < E4) Rows::store(row, col[j], pre[j], acc[j], lrd);
    }
  };
  auto park = [&]() {
#pragma unroll
    for (int j = 0; j < CPL; ++j) part[(grp * CPL + j) * LPR + rl] = acc[j];
  };

  // Look-ups past hi: only in the grid's last blocks.
  const bool ragged = uint64_t(uint32_t(blk) + 1u) * NG * uint32_t(C) > uint32_t(NS);
  // A repeat of the previous look-up's (key, bag) reuses its dY row, where the
  // wavefront is one row group; among several it costs more than the L1 hit.
  constexpr bool kDup = LPR == kWave;
  uint64_t plast = p0;  // look-up before the current group (none before lo: p0 itself)
  for (uint32_t s = lo; s < hi; s += U) {
    uint64_t p[U];
    uint32_t bg[U];
    float aw[U];
    int32_t ob0[U], ob1[U];
    bool dup[U], nseg[U];
    typename Dy<GBF16>::Raw g[U][CPL];
    // At 64 lanes these places are uniform: the compiler keeps them in scalar
    // registers and spills 52 (FP32, plain sums) to 259 (weighted) of those to
    // vector lanes, as against 15 and 71 where a place was formed again at each
    // use.  No call measured was slower for it (E = 256 to 1024, 100K to 6M look-ups,
    // every storage and pooling: 0.97 to 1.00).
    typename Rows::Row wr[U];
    typename Rows::Pre wp[U][CPL];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      p[u] = pn[u];
      if constexpr (kW) aw[u] = an[u];
      bg[u] = bag_of(p[u]);  // bag 0 past hi
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t pq = u == 0 ? plast : p[u - 1];
      const bool valid = !ragged || s + u < hi;
      dup[u] = kDup && p[u] == pq && !(s == lo && u == 0);
      nseg[u] = valid && key_of(p[u]) != key_of(pq);
    }
    if constexpr (MODE == kPoolMean) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        ob0[u] = pd.offsets[bg[u]];
        ob1[u] = pd.offsets[bg[u] + 1];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        if (kDup && dup[u])
          g[u][j] = Dy<GBF16>::zero();
        else
          g[u][j] = Dy<GBF16>::load(dY, bg[u], E, col[j]);
      }
      if (nseg[u]) {
        wr[u] = row_of(p[u]);
#pragma unroll
        for (int j = 0; j < CPL; ++j) wp[u][j] = Rows::load(wr[u], col[j]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) pn[u] = s + U + u < hi ? sorted[s + U + u] : 0ull;
    if constexpr (kW) {
#pragma unroll
      for (int u = 0; u < U; ++u) an[u] = s + U + u < hi ? pd.svals[s + U + u] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (ragged && s + u >= hi) break;
      if (nseg[u]) {
        if (open)
          park();
        else
          apply();
        open = false;
        cur = key_of(p[u]);
        row = wr[u];
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
          acc[j] = d4{0.0, 0.0, 0.0, 0.0};
          pre[j] = wp[u][j];
        }
      }
      double c = 1.0;
      if constexpr (kW) c = double(aw[u]);
      if constexpr (MODE == kPoolMean) c = 1.0 / double(ob1[u] - ob0[u]);
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        if (!kDup || !dup[u]) glast[j] = Dy<GBF16>::value(g[u][j]);
        if constexpr (MODE == kPoolPlain)
          acc[j] += widen(glast[j]);
        else
          acc[j] += c * widen(glast[j]);
      }
    }
    plast = p[U - 1];
  }

  // The chunk's last segment: open at both ends, it is the chunk's only one
  // and parked; ending here, it is applied; begun here and going on, it waits
  // for the partial sums of the row groups that follow.
  const bool last_open = lo < hi && knext == cur;
  const bool whole = open;
  if constexpr (kMany) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(whole && last_open);
    if (lane == 0) through[wave_id()] = m;
  } else if (rl == 0) {
    thru[grp] = whole && last_open;
  }
  if (whole)
    park();
  else if (lo < hi && !last_open)
    apply();
  __syncthreads();
  // Adds the sums that the row groups from k on parked, in order, while the
  // segment goes on; whether it goes on past the block.  Where the row groups are
  // many the chain's end is found first, so that its sums are read several at a
  // time (50K look-ups of E = 4, 256 row groups to a block: an update of 27 us when
  // they were read one by one, 12 so; E = 8 18 and 11).
  auto add_parked = [&](int k) {
    auto add = [&](int i) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[j] += part[(i * CPL + j) * LPR + rl];
    };
    if constexpr (kMany) {
      int w = k / R;
      if (w >= kWavesPerBlock) return true;
      uint64_t ends = ~through[w] & (~0ull << (k % R * LPR));
      while (ends == 0 && ++w < kWavesPerBlock) ends = ~through[w];
      const int last = ends != 0 ? w * R + int(__builtin_ctzll(ends)) / LPR : NG - 1;
#pragma unroll 8
      for (; k <= last; ++k) add(k);
      return ends == 0;
    } else {
      bool on = true;
      for (; on && k < NG; ++k) {
        add(k);
        on = thru[k] != 0;
      }
      return on;
    }
  };
  if (lo < hi && !whole && last_open) {
    if (!add_parked(grp + 1))
      apply();
    else
      store_carry<CPL>(carry, 2 * int64_t(blk) + 1, E, rl, LPR, acc);
  }
  if (grp == 0 && before) {
#pragma unroll
    for (int j = 0; j < CPL; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
    add_parked(0);
    store_carry<CPL>(carry, 2 * int64_t(blk), E, rl, LPR, acc);
  }
}

// Sums over kPre blocks that one segment fills, for segments over very many
// blocks: a fix-up block reads partial sums at one compute unit's 150 GB/s, and
// 4096 of E = 256 are 8 MB.  The sum of an aligned group of kPre blocks from b0 on
// goes to slot 2 * b0 + 1 (a block that a segment fills has no use for it); the
// fix-up knows from the segment's ends alone which groups are full.
constexpr int kPre = 16;

template <int LPR, int CPL>
__global__ __launch_bounds__(kBlock) void segment_presum(
    const uint64_t* __restrict__ sorted, uint32_t span, int32_t nblocks, int32_t E,
    double* __restrict__ carry, const int32_t* __restrict__ flags, uint32_t token) {
  constexpr int R = kWave / LPR;
  constexpr int GU = CPL == 1 ? kPre : (CPL == 2 ? kPre / 2 : kPre / 4);
  const int lane = lane_id(), rg = lane / LPR, rl = lane % LPR;
  const int b0 = ((int(blockIdx.x) * kWavesPerBlock + wave_id()) * R + rg + 1) * kPre;
  if (b0 + kPre >= nblocks) return;  // the look-up after the group has to be in the segment
  const uint32_t first = uint32_t(b0) * span, after = first + kPre * span;
  const uint32_t kf = key_of(sorted[first - 1]), ka = key_of(sorted[after]);
  if (flags[0] != 0 || uint32_t(flags[1]) != token || kf != ka) return;
  d4 acc[CPL];
#pragma unroll
  for (int j = 0; j < CPL; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int u0 = 0; u0 < kPre; u0 += GU) {
    d4 v[GU][CPL];
#pragma unroll
    for (int u = 0; u < GU; ++u) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        const int c4 = rl + j * LPR;
        v[u][j] = c4 < E / 4 ? *reinterpret_cast<const d4*>(carry + 2 * int64_t(b0 + u0 + u) * E + c4 * 4)
                             : d4{0.0, 0.0, 0.0, 0.0};
      }
    }
#pragma unroll
    for (int u = 0; u < GU; ++u) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[j] += v[u][j];
    }
  }
  store_carry<CPL>(carry, 2 * int64_t(b0) + 1, E, rl, LPR, acc);
}

// Threads of a fix-up block.  kBlock of them look after one boundary; a segment
// over many blocks is the work of all, so that one row's partial sums are not a
// long chain of loads.  Narrow rows have row groups enough in kBlock threads,
// and more than 2 float4 groups per lane take registers that 1024 threads have not.
template <int LPR, int CPL>
constexpr int kFixThreads = LPR < 32 ? kBlock : (CPL == 1 ? 4 * kBlock : 2 * kBlock);

// Segments that cross block boundaries: kBlock threads per boundary.  They have
// work if the segment at the boundary begins in the block before it; the segment's
// partial sums are that block's slot 2b+1 and the first slots of the `n`
// blocks that follow and begin inside it.  Row group g adds those of blocks
// g, g + NG, ... in order, and row group 0 adds the row groups' sums in order
// and applies the row once.  Where n is large (at most one of a fix-up block's
// boundaries can be: the segment covers the others) the row groups of the whole
// fix-up block add them so.  The order depends on the positions alone.
// Measured, us per update of 500K look-ups, all of one row / of many rows, with
// row groups of kBlock threads and 4 loads in flight alone: E = 64 34 / 29, E = 128
// 182 / 58, E = 256 196 / 89; so: 26 / 29, 72 / 52, 52 / 86.  64 registers where the
// row groups are few: blocks of 1024 threads then share a compute unit by twos.
template <int LPR, int CPL, class Rows>
__global__ __launch_bounds__((kFixThreads<LPR, CPL>), CPL == 1 && LPR >= 32 ? 8 : 1) void segment_fixup(
    TableDesc d, const uint64_t* __restrict__ sorted, int32_t NS, uint32_t span, int32_t nblocks,
    int32_t B, float inv_b, float lr, const double* __restrict__ carry,
    const int32_t* __restrict__ flags, uint32_t token, bool presummed) {
  constexpr int NG = kGroups<LPR>;
  constexpr int R = kWave / LPR;
  constexpr int Q = kFixThreads<LPR, CPL> / kBlock;  // boundaries of the fix-up block
  constexpr int UF = CPL == 1 ? (LPR < 32 ? 8 : 4) : (CPL == 2 ? 4 : 2);
  // partials per row group up to which a boundary's own row groups add them
  constexpr int US = CPL == 1 ? 4 : (CPL == 2 ? 2 : 1);
  static_assert(US * NG >= Q, "a long segment must cover the fix-up block's other boundaries");
  __shared__ d4 part[Q * NG * LPR * CPL];
  __shared__ int32_t many[Q];  // blocks of the boundary's segment if they are many
  const int lane = lane_id(), wave = wave_id();
  const int rg = lane / LPR, rl = lane % LPR;
  const int q = wave / kWavesPerBlock, grp = wave % kWavesPerBlock * R + rg;
  const int b = int(blockIdx.x) * Q + q;
  // The words at the boundary, requested with the flags.
  const bool real = b + 1 < nblocks;
  const uint32_t lo = uint32_t(b) * span, hi = lo + span;  // hi < NS where real
  const uint64_t wl = real ? sorted[hi - 1] : 0ull, wn = real ? sorted[hi] : ~0ull;
  const uint64_t wb = real && lo > 0 ? sorted[lo - 1] : ~0ull;
  if (flags[0] != 0 || uint32_t(flags[1]) != token) return;
  const int E = d.dim, E4 = E / 4;
  const uint32_t kl = key_of(wl);
  auto slot = [&](int64_t s, d4* v) {
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int c4 = rl + j * LPR;
      v[j] = c4 < E4 ? *reinterpret_cast<const d4*>(carry + s * E + c4 * 4) : d4{0.0, 0.0, 0.0, 0.0};
    }
  };
  d4 acc[CPL];
  typename Rows::Row row;
  typename Rows::Pre pre[CPL];
  auto add_and_apply = [&](const d4* sums, int m) {
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) acc[j] += sums[(k * CPL + j) * LPR + rl];
    }
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int c4 = rl + j * LPR;
      if (c4 < E4) Rows::store(row, c4, pre[j], acc[j], double(lr));
    }
  };
  d4* own = part + q * (NG * LPR * CPL);
  int n = 0;  // the same in every lane of the boundary's wavefronts
  if (key_of(wn) == kl && key_of(wb) != kl) {  // (keys are below 2^31)
    // The partial that row group g adds first, requested before it is known
    // whether its block belongs to the segment.
    d4 sum[CPL];
    if (b + 1 + grp < nblocks) slot(2 * int64_t(b + 1 + grp), sum);
    if (grp == 0) {
      const int ct = table_of_bag(bag_of(wl), B, inv_b);
      row = Rows::row(Rows::table(d, ct), kl - d.rowbase[ct], E);
      slot(2 * int64_t(b) + 1, acc);
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        const int c4 = rl + j * LPR;
        if (c4 < E4) pre[j] = Rows::load(row, c4);
      }
    }
    // n: the blocks from b + 1 on whose first look-up is in the segment (the
    // keys are sorted, so they come first): a look at 64 of them, and if all
    // are, a 64-way search for the last one.
    auto in = [&](int64_t c) {
      return c < nblocks && key_of(sorted[uint32_t(c) * span]) == kl;
    };
    const uint64_t near = __builtin_amdgcn_ballot_w64(in(int64_t(b) + 1 + lane));
    n = __popcll(near);
    if (n == kWave) {
      int first = b + kWave, last = nblocks - 1;  // block `first` is in the segment
      while (first < last) {
        const int step = int((int64_t(last) - first + kWave) / kWave);
        const int64_t c = first + int64_t(lane) * step;
        const uint64_t m = __builtin_amdgcn_ballot_w64(c <= last && in(c));
        first += (63 - __builtin_clzll(m)) * step;
        last = min(first + step - 1, last);
      }
      n = first - b;
    }
    if (n <= US * NG && grp < n) {
      d4 v[US][CPL];
#pragma unroll
      for (int u = 1; u < US; ++u)
        if (grp + u * NG < n) slot(2 * int64_t(b + 1 + grp + u * NG), v[u]);
#pragma unroll
      for (int u = 1; u < US; ++u) {
        if (grp + u * NG < n) {
#pragma unroll
          for (int j = 0; j < CPL; ++j) sum[j] += v[u][j];
        }
      }
#pragma unroll
      for (int j = 0; j < CPL; ++j) own[(grp * CPL + j) * LPR + rl] = sum[j];
    }
  }
  if (int(threadIdx.x) % kBlock == 0) many[q] = n > US * NG ? n : 0;
  __syncthreads();
  if (n > 0 && n <= US * NG && grp == 0) add_and_apply(own, min(n, NG));
  int lb = 0, ln = 0;  // the boundary with many blocks
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    if (many[i] > 0) {
      lb = int(blockIdx.x) * Q + i;
      ln = many[i];
    }
  }
  if (ln == 0) return;  // the same in the whole fix-up block
  __syncthreads();
  // What to add: the blocks up to the first full group, the groups' sums, the
  // blocks after the last of them.
  const int g0 = (lb + kPre) / kPre * kPre;  // first group from block lb + 1 on
  const int groups = presummed && lb + ln > g0 ? (lb + ln - g0) / kPre : 0;
  const int head = groups > 0 ? g0 - (lb + 1) : ln;
  const int items = ln - groups * (kPre - 1);
  auto slot_of = [&](int i) {
    if (i < head) return 2 * int64_t(lb + 1 + i);
    if (i < head + groups) return 2 * int64_t(g0 + (i - head) * kPre) + 1;
    return 2 * int64_t(lb + 1 + i + groups * (kPre - 1));
  };
  const int g = wave * R + rg;
  if (g < items) {
    d4 sum[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) sum[j] = d4{0.0, 0.0, 0.0, 0.0};
    for (int c = g; c < items; c += UF * Q * NG) {
      d4 v[UF][CPL];
#pragma unroll
      for (int u = 0; u < UF; ++u)
        if (c + u * Q * NG < items) slot(slot_of(c + u * Q * NG), v[u]);
#pragma unroll
      for (int u = 0; u < UF; ++u) {
        if (c + u * Q * NG < items) {
#pragma unroll
          for (int j = 0; j < CPL; ++j) sum[j] += v[u][j];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < CPL; ++j) part[(g * CPL + j) * LPR + rl] = sum[j];
  }
  __syncthreads();
  if (b == lb && grp == 0) add_and_apply(part, min(items, Q * NG));
}

#define EMB_GEOM(g, MACRO)           \
  switch (g.lpr) {                   \
    case 1: MACRO(1, 1); break;      \
    case 2: MACRO(2, 1); break;      \
    case 4: MACRO(4, 1); break;      \
    case 8: MACRO(8, 1); break;      \
    case 16: MACRO(16, 1); break;    \
    case 32: MACRO(32, 1); break;    \
    default:                         \
      switch (g.cpl) {               \
        case 1: MACRO(64, 1); break; \
        case 2: MACRO(64, 2); break; \
        case 3: MACRO(64, 3); break; \
        default: MACRO(64, 4); break; \
      }                              \
  }

template <class Rows, int MODE, bool GBF16 = false>
void launch_apply(const TableDesc& d, int32_t B, const void* dY, float lr, const BwdLayout& L,
                  char* ws, uint32_t token, PoolDev pd, hipStream_t st) {
  const uint64_t* sorted = sorted_buffer(L, ws);
  double* carry = reinterpret_cast<double*>(ws + L.off_carry);
  const int32_t* flags = reinterpret_cast<const int32_t*>(ws + L.off_flags);
  const float inv_b = 1.0f / float(B);
  const RowGeom g = row_geom(d.dim);
  const int blocks = int(L.nblocks);
  const uint32_t span = uint32_t(L.chunk) * uint32_t(kBlock / g.lpr);
  const int32_t NS = int32_t(L.ns), C = int32_t(L.chunk);
  const int32_t in_order = apply_in_dispatch_order(blocks, d.num_tables, B, d.dim, GBF16 ? 2 : 4);
  // A launch more (2 us; 5 where a row of E = 1024 fills a group or two) where the
  // blocks' partial sums of one row may be over 4 MB, in updates of 80 us and more.
  // Measured, us per update without / with it, all look-ups of one row and 30% of
  // them: 500K of E = 256 120 / 52 and 105 / 84, of E = 512 218 / 67 and 194 / 146, of
  // E = 1024 398 / 119 and 382 / 298; 250K of E = 256 (1954 blocks) 71 / 31 and 60 / 51,
  // but 51.5 / 53.2 without a hot row, so that the line lies above it.
  const bool presum = blocks > 1024 && int64_t(blocks) * d.dim > (int64_t(1) << 19);
#define EMB_SEG(LL, CC)                                                                        \
  hipLaunchKernelGGL((segment_sgd<LL, CC, Rows, MODE, GBF16>), dim3(blocks), dim3(kBlock), 0, st, \
                     d, sorted, NS, C, dY, B, inv_b, lr, carry, flags, token, pd, in_order);   \
  if (presum)                                                                                  \
    hipLaunchKernelGGL((segment_presum<LL, CC>),                                               \
                       dim3((blocks / kPre + kBlock / LL - 1) / (kBlock / LL)), dim3(kBlock), 0, \
                       st, sorted, span, blocks, d.dim, carry, flags, token);                  \
  if (blocks > 1)                                                                              \
    hipLaunchKernelGGL((segment_fixup<LL, CC, Rows>),                                            \
                     dim3((blocks - 1 + kFixThreads<LL, CC> / kBlock - 1) /                    \
                          (kFixThreads<LL, CC> / kBlock)),                                     \
                     dim3(kFixThreads<LL, CC>), 0, st, d, sorted, NS, span, blocks, B, inv_b,   \
                     lr, carry, flags, token, presum)
  EMB_GEOM(g, EMB_SEG)
#undef EMB_SEG
}

}  // namespace

hipError_t launch_segment_sgd(const TableDesc& d, bool split, int32_t B, const void* dY,
                              bool dy_bf16, float lr, const BwdLayout& L, char* ws,
                              uint32_t token, const PoolArgs& pool, hipStream_t st) {
  if (L.ns == 0) return hipSuccess;
  PoolDev pd{sorted_values(L, ws), pool.offsets};
  if (split && dy_bf16)
    launch_apply<SplitRows, kPoolPlain, true>(d, B, dY, lr, L, ws, token, pd, st);
  else if (split)
    launch_apply<SplitRows, kPoolPlain>(d, B, dY, lr, L, ws, token, pd, st);
  else if (pool.mode == kPoolWeighted)
    launch_apply<Fp32Rows, kPoolWeighted>(d, B, dY, lr, L, ws, token, pd, st);
  else if (pool.mode == kPoolMean)
    launch_apply<Fp32Rows, kPoolMean>(d, B, dY, lr, L, ws, token, pd, st);
  else
    launch_apply<Fp32Rows, kPoolPlain>(d, B, dY, lr, L, ws, token, pd, st);
  return hipGetLastError();
}

}  // namespace embbag
