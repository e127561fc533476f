// Keys and stable sort of a small call's look-ups, in one or two kernels.
//
// A radix sort over the whole list costs nine launches of a few microseconds
// each, whatever the size.  The look-ups of a table are one contiguous range
// already, so here a block sorts 2048 or 4096 look-ups of one table by row
// inside LDS (a tile), every pass of it, and a second kernel merges the tiles
// of a table that has several: each key's place is its own plus, for every
// other tile of the table, the number of that tile's keys before it, found by
// binary search in LDS.  Keys of a tile that is its table's only one go to
// their place at once.  Up to 4096 look-ups in all, a single block sorts them
// by the whole key and nothing is merged.
//
// A tile is one block's work, so that latency bounds it: four dependent loads
// (table edges, bag search, offsets, look-ups) and, per pass of up to 10 bits,
// a few LDS round trips and barriers.  16 wavefronts take 10 us for 512
// look-ups of 25 bits and 15 us for 4096 of 20; the merge 4 us with nothing to
// merge, 6 us for 2 tiles of 4096 per table and 11 us for 7.
//
// The result is that of the radix sort, bit for bit: (key << 32 | bag) words
// in increasing key, ties in look-up order, the weights beside them, the
// status folded into the workspace's flags and the caller's word.
#include "sort_tile.hpp"

namespace embbag {
namespace {

constexpr int kWholeItems = 4;

// WHOLE: one block, the whole list, by the whole key.  Otherwise block b
// sorts the b-th tile of the tables' tiles in order, if there is one.  Every
// block checks `vb` of the offsets.
template <int ITEMS, bool WHOLE>
__global__ __launch_bounds__(kThreads) void tile_sort(
    TableDesc d, const int32_t* __restrict__ I, const int32_t* __restrict__ O, int32_t NS,
    int32_t B, float inv_b, int32_t TB, int32_t vb, uint64_t* __restrict__ out,
    uint32_t* __restrict__ pkeys, uint32_t* __restrict__ pbags, const float* __restrict__ A,
    float* __restrict__ vout, float* __restrict__ vparts, Tile* __restrict__ info,
    int32_t* __restrict__ status, int32_t* __restrict__ flags, int32_t* __restrict__ d_status,
    uint32_t token) {
  constexpr int kTile = ITEMS * kThreads;
  __shared__ uint32_t lbag[kTile];
  __shared__ uint32_t skey[kTile];
  __shared__ uint16_t sidx[kTile];
  // Per-wave digit counts, then each wave's first place for a digit.
  __shared__ __align__(4) uint16_t whist[2][kWaves << kMaxDigitBits];
  __shared__ uint32_t scratch[kWaves];
  __shared__ int32_t krange[2];
  __shared__ int32_t lerr;
  __shared__ uint32_t srows[kMaxTables], srowbase[kMaxTables];
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const int blk = int(blockIdx.x);
  int err = 0;
  if (tid == 0) lerr = 0;
  if (WHOLE && tid < d.num_tables) {
    srows[tid] = d.rows[tid];
    srowbase[tid] = d.rowbase[tid];
  }
  const Tile me = WHOLE ? Tile{0, NS, 0, 1, NS, 0} : find_tile<ITEMS>(O, NS, d.num_tables, B, blk);
  if (!WHOLE && tid == 0) info[blk] = me;
  const int start = me.start, count = me.count, t = me.table;
  const int ipt = max((count + kThreads - 1) / kThreads, 1);
  const int j0 = w * (kWave * ipt) + lane;
  int32_t rv[ITEMS];
  bool valid[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int j = j0 + i * kWave;
    valid[i] = i < ipt && j < count;
    rv[i] = valid[i] ? I[start + j] : 0;
  }
  if constexpr (!WHOLE) {
    const int64_t k0 = int64_t(blk) * vb;
    if (bad_offsets(O, k0, min(k0 + vb, int64_t(TB)), NS, TB)) err = EMBBAG_ERR_OFFSETS;
  }

  if (count > 0) {  // uniform over the block
    for (int i = tid; i < (kWaves << kMaxDigitBits) / 2; i += kThreads)
      reinterpret_cast<uint32_t*>(whist[0])[i] = 0;
    const int lo = WHOLE ? 0 : t * B, hi = WHOLE ? TB - 1 : lo + B - 1;
    if (fill_bags<ITEMS, WHOLE>(O, lo, hi, start, count, NS, TB, lbag, krange)) err = EMBBAG_ERR_OFFSETS;

    uint32_t key[ITEMS], idx[ITEMS];
    const uint32_t span = WHOLE ? d.rowbase[d.num_tables] : d.rows[t];
    const int nbits = 32 - __builtin_clz(max(span - 1u, 1u));
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = j0 + i * kWave;
      key[i] = 0;
      idx[i] = uint32_t(j);
      if (valid[i]) {
        int tt = t;
        if constexpr (WHOLE) tt = table_of_bag(min(lbag[j], uint32_t(TB - 1)), B, inv_b);
        uint32_t r = uint32_t(rv[i]);
        if (r >= (WHOLE ? srows[tt] : d.rows[t])) {
          err = min(err, EMBBAG_ERR_INDEX_RANGE);
          r = 0;
        }
        key[i] = WHOLE ? srowbase[tt] + r : r;
      }
    }
    const int passes = (nbits + kMaxDigitBits - 1) / kMaxDigitBits;
    const int bits = (nbits + passes - 1) / passes;
    for (int p = 0; p < passes; ++p) {
      // the counts of the next pass are cleared while this one ranks
      uint16_t* hist = whist[p & 1];
      uint32_t* clear = reinterpret_cast<uint32_t*>(whist[(p + 1) & 1]);
      if (p + 1 < passes)
        for (int i = tid; i < (kWaves << bits) / 2; i += kThreads) clear[i] = 0;
      uint32_t dig[ITEMS], rank[ITEMS];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        if (p > 0 && i < ipt) {
          key[i] = skey[j0 + i * kWave];
          idx[i] = sidx[j0 + i * kWave];
        }
        dig[i] = (key[i] >> (p * bits)) & ((1u << bits) - 1u);
      }
      rank_digits<ITEMS>(dig, valid, ipt, bits, hist, rank);
      __syncthreads();
      place_digits<true>(bits, hist, scratch);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        if (valid[i]) {
          const uint32_t at = hist[(w << bits) + dig[i]] + rank[i];
          skey[at] = key[i];
          sidx[at] = uint16_t(idx[i]);
        }
      }
      __syncthreads();
    }
    const uint32_t kbase = WHOLE ? 0u : d.rowbase[t];
    for (int j = tid; j < count; j += kThreads) {
      const int from = sidx[j];
      const uint32_t k = kbase + skey[j], bag = min(lbag[from], uint32_t(TB - 1));
      if (WHOLE || me.tiles <= 1) {
        out[start + j] = (uint64_t(k) << 32) | bag;
        if (A != nullptr) vout[start + j] = A[start + from];
      } else {
        pkeys[start + j] = k;
        pbags[start + j] = bag;
        if (A != nullptr) vparts[start + j] = A[start + from];
      }
    }
  }
  __syncthreads();  // lerr is zero
  if (err != 0) atomicMin(&lerr, err);
  __syncthreads();
  if (tid == 0) {
    if constexpr (WHOLE)
      publish(lerr, token, flags, d_status);
    else
      status[blk] = lerr;
  }
}

// kSlices blocks for a tile: each thread takes one key to its place among all
// the tiles of the table.  kAtOnce of them at a time are copied to LDS and
// searched together: a search is a chain of up to 13 dependent reads, a few hundred
// cycles each from the L2 and more past it, where the first kernel's results
// lie.  The last block folds the status words of the first kernel's blocks.
constexpr int kMerge = 512;
constexpr int kAtOnce = 8;
typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));

template <int ITEMS>
__global__ __launch_bounds__(kMerge) void tile_merge(
    const uint32_t* __restrict__ pkeys, const uint32_t* __restrict__ pbags,
    uint64_t* __restrict__ out, const Tile* __restrict__ info,
    const int32_t* __restrict__ status, const float* __restrict__ vparts,
    float* __restrict__ vout, int32_t nblocks, int32_t* __restrict__ flags,
    int32_t* __restrict__ d_status, uint32_t token) {
  constexpr int kTile = ITEMS * kThreads, kSlices = kTile / kMerge;
  __shared__ uint32_t keys[kAtOnce][kTile];
  const int tid = threadIdx.x;
  const int tile = int(blockIdx.x) / kSlices, j = int(blockIdx.x) % kSlices * kMerge + tid;
  if (tile == nblocks) {
    __shared__ int32_t lerr;
    if (tid == 0) lerr = 0;
    __syncthreads();
    int e = 0;
    for (int i = tid; i < nblocks; i += kMerge) e = min(e, status[i]);
    if (e != 0) atomicMin(&lerr, e);
    __syncthreads();
    if (tid == 0) publish(lerr, token, flags, d_status);
    return;
  }
  const Tile me = info[tile];
  if (me.tiles <= 1 || j - tid >= me.count) return;
  const int mine = tile - me.first;
  const int begin = me.start - mine * kTile;  // the table's first look-up
  const bool valid = j < me.count;
  const uint32_t key = valid ? pkeys[me.start + j] : 0u;
  const uint32_t bag = valid ? pbags[me.start + j] : 0u;
  auto size = [&](int o) {
    return o < me.tiles - 1 ? kTile : (o < me.tiles ? me.last : 0);
  };
  int at = j;
  for (int o0 = 0; o0 < me.tiles; o0 += kAtOnce) {
    if (o0 > 0) __syncthreads();
    constexpr int kPer = kTile / 4 / kMerge;
    u4 k[kAtOnce][kPer];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        // (the last words of a table may be read past its end: the bags follow)
        const int q = (i * kMerge + tid) * 4;
        if (q < size(o0 + u))
          k[u][i] = *reinterpret_cast<const u4*>(pkeys + begin + (o0 + u) * kTile + q);
      }
    }
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int n = size(o0 + u);
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int q = (i * kMerge + tid) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) keys[u][q + e] = q + e < n ? k[u][i][e] : kNoKey;
      }
    }
    __syncthreads();
    int pos[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) pos[u] = 0;
    // Keys of an earlier tile go first among equals (keys are below 2^31, and
    // the places past a tile's keys hold kNoKey).
#pragma unroll 1
    for (int step = kTile / 2; step > 0; step >>= 1) {
#pragma unroll
      for (int u = 0; u < kAtOnce; ++u) {
        if (o0 + u < me.tiles)
          pos[u] += keys[u][pos[u] + step - 1] < key + (o0 + u < mine ? 1u : 0u) ? step : 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      if (o0 + u < me.tiles && o0 + u != mine)
        at += pos[u] + (keys[u][pos[u]] < key + (o0 + u < mine ? 1u : 0u) ? 1 : 0);
    }
  }
  if (valid) {
    out[begin + at] = (uint64_t(key) << 32) | bag;
    if (vparts != nullptr) vout[begin + at] = vparts[me.start + j];
  }
}

template <int ITEMS>
hipError_t sort_tiles(const TableDesc& d, int32_t B, const int32_t* I, const int32_t* O,
                      int64_t NS, const BwdLayout& L, char* ws, int32_t* d_status,
                      uint32_t token, const float* A, hipStream_t st) {
  constexpr int kTile = ITEMS * kThreads;
  const int32_t TB = d.num_tables * B, ns = int32_t(NS);
  const float inv_b = B > 0 ? 1.0f / float(B) : 0.0f;
  uint64_t* out = sorted_buffer(L, ws);
  uint32_t* pkeys = reinterpret_cast<uint32_t*>(ws + (L.sorted_in_b ? L.off_a : L.off_b));
  uint32_t* pbags = pkeys + NS;
  float* vout = sorted_values(L, ws);
  float* vparts = reinterpret_cast<float*>(ws + (L.sorted_in_b ? L.off_va : L.off_vb));
  int32_t* flags = reinterpret_cast<int32_t*>(ws + L.off_flags);
  const int blocks = tile_blocks(NS, d.num_tables, kTile);
  Tile* info = reinterpret_cast<Tile*>(ws + L.off_hist);
  int32_t* status = reinterpret_cast<int32_t*>(info + blocks);
  const int32_t vb = (TB + blocks - 1) / blocks;
  hipLaunchKernelGGL((tile_sort<ITEMS, false>), dim3(blocks), dim3(kThreads), 0, st, d, I, O, ns,
                     B, inv_b, TB, vb, out, pkeys, pbags, A, vout, vparts, info, status, flags,
                     d_status, token);
  hipLaunchKernelGGL(tile_merge<ITEMS>, dim3(blocks * (kTile / kMerge) + 1), dim3(kMerge), 0, st,
                     pkeys, pbags, out, info, status, A != nullptr ? vparts : nullptr, vout,
                     blocks, flags, d_status, token);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_sort_small(const TableDesc& d, int32_t B, const int32_t* I, const int32_t* O,
                             int64_t NS, const BwdLayout& L, char* ws, int32_t* d_status,
                             uint32_t token, const float* A, hipStream_t st) {
  if (NS <= kWholeItems * kThreads) {
    const int32_t TB = d.num_tables * B;
    hipLaunchKernelGGL((tile_sort<kWholeItems, true>), dim3(1), dim3(kThreads), 0, st, d, I, O,
                       int32_t(NS), B, B > 0 ? 1.0f / float(B) : 0.0f, TB, TB,
                       sorted_buffer(L, ws), nullptr, nullptr, A, sorted_values(L, ws), nullptr,
                       nullptr, nullptr, reinterpret_cast<int32_t*>(ws + L.off_flags), d_status,
                       token);
    return hipGetLastError();
  }
  // Tiles of 2048 look-ups while the tables have few of them (59K over 8 tables
  // 17 us instead of 20, 53K over 26 13 instead of 15), else of 4096 (81K over
  // 3 tables 24 instead of 25).
  if (NS <= int64_t(d.num_tables) * kAtOnce * 2 * kThreads)
    return sort_tiles<2>(d, B, I, O, NS, L, ws, d_status, token, A, st);
  return sort_tiles<4>(d, B, I, O, NS, L, ws, d_status, token, A, st);
}

}  // namespace embbag
