// Keys and stable sort of a small call's look-ups, in one or two kernels.
//
// A radix sort over the whole list costs nine launches of a few microseconds
// each, whatever the size.  The look-ups of a table are one contiguous range
// already, so here a block sorts up to 4096 look-ups of one table by row
// inside LDS (a tile), every pass of it, and a second kernel merges the tiles
// of a table that has several: each key's place is its own plus, for every
// other tile of the table, the number of that tile's keys before it, found by
// binary search in LDS.  Keys of a tile that is its table's only one go to
// their place at once.  Up to 4096 look-ups in all, a single block sorts them
// by the whole key and nothing is merged.
//
// A tile is one block's work, so that latency bounds it: four dependent loads
// (table edges, bag search, offsets, look-ups) and, per pass of up to 10 bits,
// a few LDS round trips and barriers.  16 wavefronts of 4 keys a lane take
// 10 us for 512 look-ups of 25 bits and 15 us for 4096 of 20; the merge 4 us
// with nothing to merge, 6 us for 2 tiles per table and 11 us for 7.
//
// The result is that of the radix sort, bit for bit: (key << 32 | bag) words
// in increasing key, ties in look-up order, the weights beside them, the
// status folded into the workspace's flags and the caller's word.
#include "common.hpp"

namespace embbag {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kItems = kSmallTile / kThreads;
constexpr int kMaxDigitBits = 10;  // one digit value per thread

// One tile, as the first kernel leaves it for the second.
struct Tile {
  int32_t start, count;  // its look-ups
  int32_t first, tiles;  // block of its table's first tile, tiles of the table
  int32_t last;          // look-ups of the table's last tile (the others are full)
};

// Inclusive scan over a wavefront by lane moves inside the vector unit: shifts
// by 1, 2, 4 and 8 within rows of 16 lanes, then each row's last value to the
// rows after it (through LDS, as __shfl_up goes, a step takes 100 cycles).
__device__ __forceinline__ uint32_t scan_wave(uint32_t v) {
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xF, 0xF, false));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xF, 0xF, false));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xF, 0xF, false));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xF, 0xF, false));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xA, 0xF, false));
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xC, 0xF, false));
  return v;
}

// Exclusive scan of one value per thread over the block.
__device__ __forceinline__ uint32_t scan_block(uint32_t v, uint32_t* scratch) {
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const uint32_t inc = scan_wave(v);
  if (lane == kWave - 1) scratch[w] = inc;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) before += i < w ? scratch[i] : 0u;
  return before + inc - v;
}

__device__ __forceinline__ void publish(int32_t err, uint32_t token, int32_t* flags,
                                        int32_t* d_status) {
  flags[0] = err;
  flags[1] = int32_t(token);
  if (err != 0 && d_status != nullptr) atomicMin(d_status, err);
}

// WHOLE: one block, the whole list, by the whole key.  Otherwise block b
// sorts the b-th tile of the tables' tiles in order, if there is one.  Every
// block checks `vb` of the offsets.
template <bool WHOLE>
__global__ __launch_bounds__(kThreads) void tile_sort(
    TableDesc d, const int32_t* __restrict__ I, const int32_t* __restrict__ O, int32_t NS,
    int32_t B, float inv_b, int32_t TB, int32_t vb, uint64_t* __restrict__ out,
    uint32_t* __restrict__ pkeys, uint32_t* __restrict__ pbags, const float* __restrict__ A,
    float* __restrict__ vout, float* __restrict__ vparts, Tile* __restrict__ info,
    int32_t* __restrict__ status,
    int32_t* __restrict__ flags, int32_t* __restrict__ d_status, uint32_t token) {
  __shared__ uint32_t lbag[kSmallTile];
  __shared__ uint32_t skey[kSmallTile];
  __shared__ uint16_t sidx[kSmallTile];
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

  // The tile: every wavefront finds it for itself from the T + 1 offsets at
  // the tables' edges, one per lane, forced into 0 .. NS and increasing order
  // (offsets that are not are reported below, and the tiles still cover the
  // list once).
  int start = 0, count = NS, t = 0, tiles = 1;
  if constexpr (!WHOLE) {
    const int T = d.num_tables;
    int edge = lane < T ? min(max(O[int64_t(lane) * B], 0), NS) : NS;
    if (lane == 0) edge = 0;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int n = __shfl_up(edge, off, kWave);
      if (lane >= off) edge = max(edge, n);
    }
    int next = __shfl_down(edge, 1, kWave);
    if (lane >= T - 1) next = NS;  // T = 64: no lane holds the last edge
    const int mine = lane < T ? (next - edge + kSmallTile - 1) / kSmallTile : 0;
    const int inc = int(scan_wave(uint32_t(mine)));
    const uint64_t m = __builtin_amdgcn_ballot_w64(inc > blk);
    count = 0;
    if (m != 0) {
      t = int(__builtin_ctzll(m));
      tiles = __builtin_amdgcn_readlane(mine, t);
      const int first = __builtin_amdgcn_readlane(inc, t) - tiles;
      const int at = __builtin_amdgcn_readlane(edge, t), end = __builtin_amdgcn_readlane(next, t);
      start = at + (blk - first) * kSmallTile;
      count = min(kSmallTile, end - start);
      if (tid == 0) info[blk] = Tile{start, count, first, tiles, end - at - (tiles - 1) * kSmallTile};
    } else if (tid == 0) {
      info[blk] = Tile{0, 0, 0, 0, 0};
    }
  }
  // Wavefront w holds the tile's keys [w * 64 * ipt, (w + 1) * 64 * ipt), item
  // i of lane l being the key w * 64 * ipt + i * 64 + l: ranked item by item
  // they keep their order.
  const int ipt = max((count + kThreads - 1) / kThreads, 1);
  const int j0 = w * (kWave * ipt) + lane;
  int32_t rv[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int j = j0 + i * kWave;
    rv[i] = i < ipt && j < count ? I[start + j] : 0;
  }

  // Offsets: O[0] == 0, O non-decreasing, O[TB] == NS, all within [0, NS].
  constexpr int Q = 4;
  auto check = [&](int64_t k, int o, int next) {
    if (o < 0 || o > NS || (k == 0 && o != 0) || next < o || (k + 1 == TB && next != NS))
      err = EMBBAG_ERR_OFFSETS;
  };
  if constexpr (!WHOLE) {
    const int64_t kb0 = int64_t(blk) * vb, kb1 = min(kb0 + vb, int64_t(TB));
    for (int64_t k0 = kb0 + tid; k0 < kb1; k0 += kThreads * Q) {
      int oa[Q], ob[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int64_t k = k0 + q * kThreads;
        oa[q] = k < kb1 ? O[k] : 0;
        ob[q] = k < kb1 ? O[k + 1] : 0;
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int64_t k = k0 + q * kThreads;
        if (k < kb1) check(k, oa[q], ob[q]);
      }
    }
  }

  if (count > 0) {  // uniform over the block
    for (int i = tid; i < kSmallTile; i += kThreads) lbag[i] = 0;
    for (int i = tid; i < (kWaves << kMaxDigitBits) / 2; i += kThreads)
      reinterpret_cast<uint32_t*>(whist[0])[i] = 0;
    // The bags that may hold the tile: all of the table's (of the list's) if
    // they are few, otherwise from the last bag k with
    // O[k] <= the tile's first look-up (wave 0) to the last with O[k] <= its
    // last one (wave 1), 64 bags probed per round.  A bad O still leaves the
    // range inside the table's bags.
    int lo = WHOLE ? 0 : t * B, hi = WHOLE ? TB - 1 : lo + B - 1;
    const bool known = WHOLE || B <= 2 * kThreads;
    if (!known && w < 2) {
      const int x = w == 0 ? start : start + count - 1;
      while (lo < hi) {
        const int step = int((int64_t(hi) - lo + kWave) / kWave);
        const int64_t k = lo + int64_t(lane) * step;
        const uint64_t m = __builtin_amdgcn_ballot_w64(k <= hi && O[k] <= x);
        const int j = m != 0 ? 63 - __builtin_clzll(m) : 0;
        lo = lo + j * step;
        hi = int(min(int64_t(lo) + step - 1, int64_t(hi)));
      }
      if (lane == 0) krange[w] = lo;
    }
    __syncthreads();
    // Bag ids over the tile's look-ups: as many threads per bag as the bags
    // leave, so that a long bag is not one thread's loop.
    {
      const int k0 = known ? lo : krange[0];
      const int nb = max((known ? hi : krange[1]) - k0 + 1, 0);
      int share = 1;
      while (share < kThreads && int64_t(share) * 2 * nb <= kThreads) share *= 2;
      const int lead = tid % share, stride = kThreads / share;
      for (int64_t q0 = tid / share; q0 < nb; q0 += int64_t(stride) * Q) {
        int oa[Q], ob[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int64_t k = q0 + q * stride;
          oa[q] = k < nb ? O[k0 + k] : 0;
          ob[q] = k < nb ? O[k0 + k + 1] : 0;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int64_t k = q0 + q * stride;
          if (k >= nb) break;
          if constexpr (WHOLE) check(k, oa[q], ob[q]);
          const int a = max(oa[q], start) - start, b = min(ob[q], start + count) - start;
          for (int s = a + lead; s < b; s += share) lbag[s] = uint32_t(k0 + k);
        }
      }
    }
    __syncthreads();

    uint32_t key[kItems], idx[kItems];
    int nbits;
    if constexpr (WHOLE)
      nbits = 32 - __builtin_clz(max(d.rowbase[d.num_tables] - 1u, 1u));
    else
      nbits = 32 - __builtin_clz(max(d.rows[t] - 1u, 1u));
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int j = j0 + i * kWave;
      key[i] = 0;
      idx[i] = uint32_t(j);
      if (i < ipt && j < count) {
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
    const int R = 1 << bits;
    const uint64_t below = (1ull << lane) - 1ull;
    for (int p = 0; p < passes; ++p) {
      const int shift = p * bits;
      // the counts of the next pass are cleared while this one ranks
      uint16_t* hist = whist[p & 1];
      uint32_t* clear = reinterpret_cast<uint32_t*>(whist[(p + 1) & 1]);
      if (p + 1 < passes)
        for (int i = tid; i < kWaves * R / 2; i += kThreads) clear[i] = 0;
      if (p > 0) {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
          if (i < ipt) {
            key[i] = skey[j0 + i * kWave];
            idx[i] = sidx[j0 + i * kWave];
          }
        }
      }
      // Lanes whose digit is this lane's: one ballot per bit, every item's at once.
      uint32_t dig[kItems], plo[kItems], phi[kItems];
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        dig[i] = (key[i] >> shift) & uint32_t(R - 1);
        const uint64_t all = __builtin_amdgcn_ballot_w64(i < ipt && j0 + i * kWave < count);
        plo[i] = uint32_t(all);
        phi[i] = uint32_t(all >> 32);
      }
      for (int b = 0; b < bits; ++b) {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
          if (i < ipt) {
            // keep the lanes whose bit b is this lane's (a & ~(b ^ c) per half)
            const int32_t sb = __builtin_amdgcn_sbfe(int32_t(dig[i]), b, 1);  // 0 or -1
            const uint64_t m = __builtin_amdgcn_ballot_w64(sb != 0);
            plo[i] = __builtin_amdgcn_bitop3_b32(plo[i], uint32_t(m), uint32_t(sb), 0x90);
            phi[i] = __builtin_amdgcn_bitop3_b32(phi[i], uint32_t(m >> 32), uint32_t(sb), 0x90);
          }
        }
      }
      uint32_t rank[kItems];
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        if (i < ipt) {
          const uint64_t peers = (uint64_t(phi[i]) << 32) | plo[i];
          const uint32_t lrank = uint32_t(__popcll(peers & below));
          const uint32_t prior = hist[w * R + dig[i]];
          rank[i] = prior + lrank;
          if (j0 + i * kWave < count && lrank == 0)
            hist[w * R + dig[i]] = uint16_t(prior + __popcll(peers));
        }
      }
      __syncthreads();
      // A digit per thread: each wavefront's first place for it.
      uint32_t c[kWaves], run = 0;
      if (tid < R) {
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) c[ww] = hist[ww * R + tid];
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) run += c[ww];
      }
      uint32_t ex = scan_block(run, scratch);
      if (tid < R) {
#pragma unroll
        for (int ww = 0; ww < kWaves; ++ww) {
          hist[ww * R + tid] = uint16_t(ex);
          ex += c[ww];
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        if (i < ipt && j0 + i * kWave < count) {
          const uint32_t at = hist[w * R + dig[i]] + rank[i];
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
      if (WHOLE || tiles <= 1) {
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
// searched together: a search is a chain of 13 dependent reads, a few hundred
// cycles each from the L2 and more past it, where the first kernel's results
// lie.  The last block folds the status words of the first kernel's blocks.
constexpr int kMerge = 512;  // threads: 32 tiles then make 256 blocks
constexpr int kSlices = kSmallTile / kMerge;
constexpr int kAtOnce = 8;
typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));

__global__ __launch_bounds__(kMerge) void tile_merge(
    const uint32_t* __restrict__ pkeys, const uint32_t* __restrict__ pbags,
    uint64_t* __restrict__ out, const Tile* __restrict__ info,
    const int32_t* __restrict__ status, const float* __restrict__ vparts,
    float* __restrict__ vout, int32_t nblocks, int32_t* __restrict__ flags,
    int32_t* __restrict__ d_status, uint32_t token) {
  __shared__ uint32_t keys[kAtOnce][kSmallTile];
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
  const int begin = me.start - mine * kSmallTile;  // the table's first look-up
  const bool valid = j < me.count;
  const uint32_t key = valid ? pkeys[me.start + j] : 0u;
  const uint32_t bag = valid ? pbags[me.start + j] : 0u;
  auto size = [&](int o) {
    return o < me.tiles - 1 ? kSmallTile : (o < me.tiles ? me.last : 0);
  };
  int at = j;
  for (int o0 = 0; o0 < me.tiles; o0 += kAtOnce) {
    if (o0 > 0) __syncthreads();
    constexpr int kPer = kSmallTile / 4 / kMerge;
    u4 k[kAtOnce][kPer];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        // (the last words of a table may be read past its end: the bags follow)
        const int q = (i * kMerge + tid) * 4;
        if (q < size(o0 + u))
          k[u][i] = *reinterpret_cast<const u4*>(pkeys + begin + (o0 + u) * kSmallTile + q);
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
    for (int step = kSmallTile / 2; step > 0; step >>= 1) {
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

}  // namespace

hipError_t launch_sort_small(const TableDesc& d, int32_t B, const int32_t* I, const int32_t* O,
                             int64_t NS, const BwdLayout& L, char* ws, int32_t* d_status,
                             uint32_t token, const float* A, hipStream_t st) {
  const int32_t TB = d.num_tables * B, ns = int32_t(NS);
  const float inv_b = B > 0 ? 1.0f / float(B) : 0.0f;
  uint64_t* out = sorted_buffer(L, ws);
  uint32_t* pkeys = reinterpret_cast<uint32_t*>(ws + (L.sorted_in_b ? L.off_a : L.off_b));
  uint32_t* pbags = pkeys + NS;
  float* vout = sorted_values(L, ws);
  float* vparts = reinterpret_cast<float*>(ws + (L.sorted_in_b ? L.off_va : L.off_vb));
  int32_t* flags = reinterpret_cast<int32_t*>(ws + L.off_flags);
  const int tiles = int((NS + kSmallTile - 1) / kSmallTile);
  if (tiles == 1) {
    hipLaunchKernelGGL(tile_sort<true>, dim3(1), dim3(kThreads), 0, st, d, I, O, ns, B, inv_b, TB,
                       TB, out, nullptr, nullptr, A, vout, nullptr, nullptr, nullptr, flags,
                       d_status, token);
    return hipGetLastError();
  }
  // every table's last tile may be part full
  const int blocks = tiles + d.num_tables;
  Tile* info = reinterpret_cast<Tile*>(ws + L.off_hist);
  int32_t* status = reinterpret_cast<int32_t*>(info + blocks);
  const int32_t vb = (TB + blocks - 1) / blocks;
  hipLaunchKernelGGL(tile_sort<false>, dim3(blocks), dim3(kThreads), 0, st, d, I, O, ns, B, inv_b,
                     TB, vb, out, pkeys, pbags, A, vout, vparts, info, status, flags, d_status, token);
  hipLaunchKernelGGL(tile_merge, dim3(blocks * kSlices + 1), dim3(kMerge), 0, st, pkeys, pbags, out, info,
                     status, A != nullptr ? vparts : nullptr, vout, blocks, flags, d_status, token);
  return hipGetLastError();
}

}  // namespace embbag
