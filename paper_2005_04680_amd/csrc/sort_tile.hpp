// Tiles of one table's look-ups, as the sorts that work table by table cut
// them: a block of kThreads threads per tile, ITEMS keys per thread.
#pragma once

#include "common.hpp"

namespace embbag {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxDigitBits = 10;  // one digit value per thread

// One tile, as the first kernel of a sort leaves it for the next ones.
struct Tile {
  int32_t start, count;  // its look-ups
  int32_t first, tiles;  // block of its table's first tile, tiles of the table
  int32_t last;          // look-ups of the table's last tile (the others are full)
  int32_t table;
};

// Blocks that cover every table's tiles: each table's last may be part full.
inline int tile_blocks(int64_t NS, int32_t T, int tile) { return int((NS + tile - 1) / tile) + T; }

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

// The blk-th of the tables' tiles in order (count 0 if there are fewer).  Every
// wavefront finds it for itself from the T + 1 offsets at the tables' edges,
// one per lane, forced into 0 .. NS and increasing order: offsets that are not
// are reported by check_offsets, and the tiles still cover the list once.
template <int ITEMS>
__device__ __forceinline__ Tile find_tile(const int32_t* O, int32_t NS, int32_t T, int32_t B,
                                          int blk) {
  constexpr int kTile = ITEMS * kThreads;
  const int lane = lane_id();
  int edge = lane < T ? min(max(O[int64_t(lane) * B], 0), NS) : NS;
  if (lane == 0) edge = 0;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int n = __shfl_up(edge, off, kWave);
    if (lane >= off) edge = max(edge, n);
  }
  int next = __shfl_down(edge, 1, kWave);
  if (lane >= T - 1) next = NS;  // T = 64: no lane holds the last edge
  const int mine = lane < T ? (next - edge + kTile - 1) / kTile : 0;
  const int inc = int(scan_wave(uint32_t(mine)));
  const uint64_t m = __builtin_amdgcn_ballot_w64(inc > blk);
  if (m == 0) return Tile{0, 0, 0, 0, 0, 0};
  const int t = int(__builtin_ctzll(m));
  const int tiles = __builtin_amdgcn_readlane(mine, t);
  const int first = __builtin_amdgcn_readlane(inc, t) - tiles;
  const int at = __builtin_amdgcn_readlane(edge, t), end = __builtin_amdgcn_readlane(next, t);
  const int start = at + (blk - first) * kTile;
  return Tile{start, min(kTile, end - start), first, tiles, end - at - (tiles - 1) * kTile, t};
}

// Offsets: O[0] == 0, O non-decreasing, O[TB] == NS, all within [0, NS].
__device__ __forceinline__ bool bad_offset(int64_t k, int o, int next, int32_t NS, int32_t TB) {
  return o < 0 || o > NS || (k == 0 && o != 0) || next < o || (k + 1 == TB && next != NS);
}

constexpr int kOffsetsAtOnce = 4;  // offsets a thread requests before it uses one

// Bags [k0, k1) of the list, whether their offsets are bad.
__device__ __forceinline__ bool bad_offsets(const int32_t* O, int64_t k0, int64_t k1, int32_t NS,
                                            int32_t TB) {
  constexpr int Q = kOffsetsAtOnce;
  bool bad = false;
  for (int64_t b = k0 + threadIdx.x; b < k1; b += kThreads * Q) {
    int oa[Q], ob[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int64_t k = b + q * kThreads;
      oa[q] = k < k1 ? O[k] : 0;
      ob[q] = k < k1 ? O[k + 1] : 0;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int64_t k = b + q * kThreads;
      if (k < k1) bad = bad || bad_offset(k, oa[q], ob[q], NS, TB);
    }
  }
  return bad;
}

// lbag[s - start] = the bag of look-up s, for the tile's look-ups.  Its bags are
// among [lo, hi]: all of those if they are few, otherwise from the last bag k
// with O[k] <= the tile's first look-up (wave 0) to the last with O[k] <= its
// last one (wave 1), 64 bags probed per round.  A bad O still leaves the range
// inside [lo, hi] and the look-ups inside the tile.  Every thread calls it;
// with CHECK the offsets of [lo, hi], which is then taken whole, are checked.
// Ends with a barrier.
template <int ITEMS, bool CHECK>
__device__ __forceinline__ bool fill_bags(const int32_t* O, int lo, int hi, int start, int count,
                                          int32_t NS, int32_t TB, uint32_t* lbag,
                                          int32_t* krange) {
  constexpr int Q = kOffsetsAtOnce;
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  bool bad = false;
  for (int i = tid; i < ITEMS * kThreads; i += kThreads) lbag[i] = 0;
  const bool known = CHECK || hi - lo < 2 * kThreads;
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
  // As many threads per bag as the bags leave, so that a long bag is not one
  // thread's loop; where few of many bags are in the tile (a table of long bags)
  // that is one each, and a wavefront then fills its lanes' long ones together.
  const int k0 = known ? lo : krange[0];
  const int nb = max((known ? hi : krange[1]) - k0 + 1, 0);
  int share = 1;
  while (share < kThreads && int64_t(share) * 2 * nb <= kThreads) share *= 2;
  const int lead = tid % share, stride = kThreads / share;
  for (int64_t q0 = 0; q0 < nb; q0 += int64_t(stride) * Q) {  // uniform over the block
    int oa[Q], ob[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int64_t k = q0 + tid / share + q * stride;
      oa[q] = k < nb ? O[k0 + k] : 0;
      ob[q] = k < nb ? O[k0 + k + 1] : 0;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (q0 + q * stride >= nb) break;  // uniform over the block
      const int64_t k = q0 + tid / share + q * stride;
      if constexpr (CHECK) bad = bad || (k < nb && bad_offset(k, oa[q], ob[q], NS, TB));
      // (both ends forced into the tile before they are moved: a bad offset may
      // be any int; past the last bag both are 0 and give an empty range)
      const int a = min(max(oa[q], start), start + count) - start;
      const int b = min(max(ob[q], start), start + count) - start;
      const uint32_t bag = uint32_t(k0 + k);
      const bool lengthy = share <= 4 && b - a > 128 * share;
      if (!lengthy)
        for (int s = a + lead; s < b; s += share) lbag[s] = bag;
      if (share > 4) continue;
      for (uint64_t m = __builtin_amdgcn_ballot_w64(lengthy && lead == 0); m != 0; m &= m - 1) {
        const int l = int(__builtin_ctzll(m));
        const int from = __builtin_amdgcn_readlane(a, l), to = __builtin_amdgcn_readlane(b, l);
        const uint32_t of = uint32_t(__builtin_amdgcn_readlane(int(bag), l));
        for (int s = from + lane; s < to; s += kWave) lbag[s] = of;
      }
    }
  }
  __syncthreads();
  return bad;
}

// Ranks a tile's keys among the equal digits of their wavefront.  Wavefront w
// holds keys [w * 64 * ipt, (w + 1) * 64 * ipt), item i of lane l being key
// w * 64 * ipt + i * 64 + l: ranked item by item they keep their order.
// hist[w * R + digit], zero before, counts the wavefront's keys of a digit.
template <int ITEMS>
__device__ __forceinline__ void rank_digits(const uint32_t* dig, const bool* valid, int ipt,
                                            int bits, uint16_t* hist, uint32_t* rank) {
  const int lane = lane_id(), row = wave_id() << bits;
  const uint64_t below = (1ull << lane) - 1ull;
  // Lanes whose digit is this lane's: one ballot per bit, every item's at once.
  uint32_t plo[ITEMS], phi[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint64_t all = __builtin_amdgcn_ballot_w64(valid[i]);
    plo[i] = uint32_t(all);
    phi[i] = uint32_t(all >> 32);
  }
  for (int b = 0; b < bits; ++b) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (i < ipt) {
        // keep the lanes whose bit b is this lane's (a & ~(b ^ c) per half)
        const int32_t sb = __builtin_amdgcn_sbfe(int32_t(dig[i]), b, 1);  // 0 or -1
        const uint64_t m = __builtin_amdgcn_ballot_w64(sb != 0);
        plo[i] = __builtin_amdgcn_bitop3_b32(plo[i], uint32_t(m), uint32_t(sb), 0x90);
        phi[i] = __builtin_amdgcn_bitop3_b32(phi[i], uint32_t(m >> 32), uint32_t(sb), 0x90);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (i < ipt) {
      const uint64_t peers = (uint64_t(phi[i]) << 32) | plo[i];
      const uint32_t lrank = uint32_t(__popcll(peers & below));
      const uint32_t prior = hist[row + dig[i]];
      rank[i] = prior + lrank;
      if (valid[i] && lrank == 0) hist[row + dig[i]] = uint16_t(prior + __popcll(peers));
    }
  }
}

// From the wavefronts' counts (after a barrier) to each wavefront's first
// place for a digit among the sorted tile; returns the thread's own digit's
// first place (digit tid < 1 << bits).  A barrier must follow.  KEEP holds the
// counts in registers meanwhile, which saves 16 LDS reads (0.3 us a pass) where
// a second block of the compute unit does not need the registers.
template <bool KEEP>
__device__ __forceinline__ uint32_t place_digits(int bits, uint16_t* hist, uint32_t* scratch) {
  const int tid = threadIdx.x, R = 1 << bits;
  uint32_t c[kWaves], run = 0;
  if (tid < R) {
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww) {
      c[ww] = hist[(ww << bits) + tid];
      run += c[ww];
    }
  }
  const uint32_t first = scan_block(run, scratch);
  if (tid < R) {
    uint32_t ex = first;
    if constexpr (KEEP) {
#pragma unroll
      for (int ww = 0; ww < kWaves; ++ww) {
        hist[(ww << bits) + tid] = uint16_t(ex);
        ex += c[ww];
      }
    } else {
#pragma unroll 4
      for (int ww = 0; ww < kWaves; ++ww) {
        const uint32_t n = hist[(ww << bits) + tid];
        hist[(ww << bits) + tid] = uint16_t(ex);
        ex += n;
      }
    }
  }
  return first;
}

}  // namespace
}  // namespace embbag
