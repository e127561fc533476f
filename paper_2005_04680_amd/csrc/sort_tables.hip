// Keys and stable radix sort of a mid-sized call's look-ups, table by table.
//
// The look-ups of a table are one contiguous range already, so a radix pass
// inside each table needs no digit of the table: digits of up to 10 bits cover
// tables of 2^20 rows in two passes.  A tile (2048, 4096 or 8192 look-ups of one
// table) is a block of 16 wavefronts with a digit per thread.  No kernel scans the
// tiles' counts: each block of the scatter adds up those of its own table by itself
// (16 tiles are 32 KB of 16-bit counts, read from the L2 in one round) while it
// ranks its keys.
//
// Bound by latency: at 524K look-ups over 8 tables (264 blocks) the keys take
// 5 us, a scatter 7 to 10 (the counts' sums, the ranks, four barriers, the store of
// runs of 4 keys), the second pass's counts 4; three passes of 8 bits over the
// whole list took 6 + 3 * (4 + 7) + 2 * 3 in nine launches.
//
// The counts of a table that holds nearly all look-ups are read by as many blocks
// as it has tiles, n^2 * 2 KB of reads from the L2s a pass.  Words of eight counts
// per lane and larger tiles for more look-ups keep that below what the whole
// list's passes take; us per prepare, whole list / words of two counts and tiles
// of at most 4096 / now, one long table among 8 (of 1M rows, the others of 100):
// 520K 39.5 / 52.3 / 39.2, 1.04M 50.9 / 61.1 / 48.8, 2M 59.4 / 132 / 59; with all tables
// of 1M rows 46.8 / 52.6 / 39.0, 65.5 / 61.5 / 48.6, 76.7 / 132 / 58.
//
// The result is that of the whole list's radix sort, bit for bit.
#include "sort_tile.hpp"

namespace embbag {
namespace {

typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// Keys of one tile and its counts of the first digit; `vb` of the offsets.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void table_keys(
    TableDesc d, const int32_t* __restrict__ I, const int32_t* __restrict__ O, int32_t NS,
    int32_t B, int32_t TB, int32_t vb, int32_t bits, uint64_t* __restrict__ out,
    uint16_t* __restrict__ hist, Tile* __restrict__ info, int32_t* __restrict__ status) {
  __shared__ uint32_t lbag[ITEMS * kThreads];
  __shared__ uint32_t lhist[1 << kMaxDigitBits];
  __shared__ int32_t krange[2];
  __shared__ int32_t lerr;
  const int tid = threadIdx.x, blk = int(blockIdx.x);
  int err = 0;
  if (tid == 0) lerr = 0;
  lhist[tid] = 0;
  const Tile me = find_tile<ITEMS>(O, NS, d.num_tables, B, blk);
  if (tid == 0) info[blk] = me;
  const int start = me.start, count = me.count, t = me.table;
  int32_t rv[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int j = i * kThreads + tid;
    rv[i] = j < count ? I[start + j] : 0;
  }
  const int64_t k0 = int64_t(blk) * vb;
  if (bad_offsets(O, k0, min(k0 + vb, int64_t(TB)), NS, TB)) err = EMBBAG_ERR_OFFSETS;
  if (count > 0) {
    if (fill_bags<ITEMS, false>(O, t * B, t * B + B - 1, start, count, NS, TB, lbag, krange))
      err = EMBBAG_ERR_OFFSETS;
    const uint32_t rows = d.rows[t], base = d.rowbase[t], mask = (1u << bits) - 1u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const int j = i * kThreads + tid;
      if (j < count) {
        uint32_t r = uint32_t(rv[i]);
        if (r >= rows) {
          err = min(err, EMBBAG_ERR_INDEX_RANGE);
          r = 0;
        }
        out[start + j] = (uint64_t(base + r) << 32) | min(lbag[j], uint32_t(TB - 1));
        atomicAdd(&lhist[r & mask], 1u);
      }
    }
  }
  __syncthreads();
  if (count > 0 && tid <= int((1u << bits) - 1u))
    hist[(size_t(blk) << bits) + tid] = uint16_t(lhist[tid]);
  if (err != 0) atomicMin(&lerr, err);
  __syncthreads();
  if (tid == 0) status[blk] = lerr;
}

// A tile's counts of the digit at `shift`.  The keys arrive in the previous
// pass's order, so equal digits often come in runs: the first lane of each run
// in a wavefront adds the run's length.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void table_counts(
    TableDesc d, const uint64_t* __restrict__ src, const Tile* __restrict__ info, int32_t shift,
    int32_t bits, uint16_t* __restrict__ hist) {
  __shared__ uint32_t lhist[1 << kMaxDigitBits];
  const int tid = threadIdx.x, lane = lane_id(), blk = int(blockIdx.x);
  const Tile me = info[blk];
  if (me.count <= 0) return;
  lhist[tid] = 0;
  uint32_t kv[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int j = i * kThreads + tid;
    kv[i] = j < me.count ? key_of(src[me.start + j]) : 0u;
  }
  __syncthreads();
  const uint32_t base = d.rowbase[me.table], R = 1u << bits;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t dg =
        i * kThreads + tid < me.count ? ((kv[i] - base) >> shift) & (R - 1u) : R;
    const uint32_t left = __shfl_up(dg, 1, kWave);
    const bool head = lane == 0 || dg != left;
    const uint64_t heads = __builtin_amdgcn_ballot_w64(head);
    if (head && dg < R) {
      const uint64_t after = lane == kWave - 1 ? 0ull : heads >> (lane + 1);
      atomicAdd(&lhist[dg], after ? uint32_t(__builtin_ctzll(after)) + 1u : uint32_t(kWave - lane));
    }
  }
  __syncthreads();
  if (tid < int(R)) hist[(size_t(blk) << bits) + tid] = uint16_t(lhist[tid]);
}

// Stable scatter of a tile by the digit at `shift` inside its table.  A block
// sums the counts of its table's tiles by itself: R 16-bit counts a tile, eight
// per thread, the block's threads taking as many tiles at a time as they span and
// as give each four.  FIRST: one more block folds the status words.  TWO: held to
// 64 registers, so that two blocks share a compute unit, where the blocks are more
// than those (1.7M look-ups in tiles of 4096 64 us instead of 70, 700K in 171
// blocks 36.8 instead of 36.1).  With values in tiles of 4096 the LDS has room for
// one block only.
template <int ITEMS, bool VALS, bool FIRST, bool TWO>
__global__ __launch_bounds__(kThreads, TWO ? 8 : 4) void table_scatter(
    TableDesc d, const uint64_t* __restrict__ src, uint64_t* __restrict__ dst,
    const Tile* __restrict__ info, int32_t shift, int32_t bits,
    const uint16_t* __restrict__ hist, const float* __restrict__ vsrc, float* __restrict__ vdst,
    const int32_t* __restrict__ status, int32_t nblocks, int32_t* __restrict__ flags,
    int32_t* __restrict__ d_status, uint32_t token) {
  constexpr int kTile = ITEMS * kThreads;
  __shared__ uint64_t buf[kTile];
  __shared__ float vbuf[VALS ? kTile : 1];
  __shared__ __align__(4) uint16_t whist[kWaves << kMaxDigitBits];
  __shared__ uint32_t tot[1 << kMaxDigitBits], pre[1 << kMaxDigitBits];
  __shared__ uint32_t scratch[2][kWaves];
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id(), blk = int(blockIdx.x);
  if (FIRST && blk == nblocks) {
    __shared__ int32_t lerr;
    if (tid == 0) lerr = 0;
    __syncthreads();
    int e = 0;
    for (int i = tid; i < nblocks; i += kThreads) e = min(e, status[i]);
    if (e != 0) atomicMin(&lerr, e);
    __syncthreads();
    if (tid == 0) publish(lerr, token, flags, d_status);
    return;
  }
  const Tile me = info[blk];
  if (me.count <= 0) return;
  const int count = me.count, R = 1 << bits;
  const int ipt = (count + kThreads - 1) / kThreads;
  const int j0 = w * (kWave * ipt) + lane;
  uint64_t item[ITEMS];
  float val[VALS ? ITEMS : 1];
  bool valid[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int j = j0 + i * kWave;
    valid[i] = i < ipt && j < count;
    item[i] = valid[i] ? src[me.start + j] : 0ull;
    if constexpr (VALS) val[i] = valid[i] ? vsrc[me.start + j] : 0.f;
  }
  for (int i = tid; i < (kWaves << bits) / 2; i += kThreads)
    reinterpret_cast<uint32_t*>(whist)[i] = 0;
  // Counts of the table's tiles: all (tot) and before this one (pre).
  tot[tid] = 0;
  pre[tid] = 0;
  for (int i = tid; i < (kWaves << bits) / 2; i += kThreads)
    reinterpret_cast<uint32_t*>(whist)[i] = 0;
  __syncthreads();
  {
    constexpr int Q = 4;  // rows requested together
    const int words = R / 8, col = tid & (words - 1), lead = tid / words;
    const int leads = min(kThreads / words, (me.tiles + Q - 1) / Q);  // words <= 128
    const u4* h = reinterpret_cast<const u4*>(hist) + size_t(me.first) * words + col;
    const int mine = blk - me.first;
    if (lead < leads) {
      u4 all_lo{}, all_hi{}, pre_lo{}, pre_hi{};  // of digits 8 col + 0, 2, 4, 6 and 1, 3, 5, 7
      for (int r0 = lead; r0 < me.tiles; r0 += leads * Q) {
        u4 c[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
          c[q] = r0 + q * leads < me.tiles ? h[size_t(r0 + q * leads) * words] : u4{};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const u4 lo = c[q] & 0xFFFFu, hi = c[q] >> 16;
          all_lo += lo;
          all_hi += hi;
          if (r0 + q * leads < mine) {
            pre_lo += lo;
            pre_hi += hi;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (all_lo[i]) atomicAdd(&tot[8 * col + 2 * i], all_lo[i]);
        if (all_hi[i]) atomicAdd(&tot[8 * col + 2 * i + 1], all_hi[i]);
        if (pre_lo[i]) atomicAdd(&pre[8 * col + 2 * i], pre_lo[i]);
        if (pre_hi[i]) atomicAdd(&pre[8 * col + 2 * i + 1], pre_hi[i]);
      }
    }
  }
  const uint32_t base = d.rowbase[me.table];
  uint32_t dig[ITEMS], rank[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) dig[i] = ((key_of(item[i]) - base) >> shift) & uint32_t(R - 1);
  rank_digits<ITEMS>(dig, valid, ipt, bits, whist, rank);
  __syncthreads();
  const uint32_t mine_tot = tid < R ? tot[tid] : 0u;
  const uint32_t to = scan_block(mine_tot, scratch[0]) + (tid < R ? pre[tid] : 0u);
  const uint32_t first = place_digits<!TWO>(bits, whist, scratch[1]);
  __syncthreads();
  // (tot is free: it now holds a digit's place in the table less that in the tile)
  if (tid < R) tot[tid] = to - first;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (valid[i]) {
      const uint32_t at = whist[(w << bits) + dig[i]] + rank[i];
      buf[at] = item[i];
      if constexpr (VALS) vbuf[at] = val[i];
    }
  }
  __syncthreads();
  const int begin = me.start - (blk - me.first) * kTile;
  for (int j = tid; j < count; j += kThreads) {
    const uint64_t it = buf[j];
    const uint32_t g = ((key_of(it) - base) >> shift) & uint32_t(R - 1);
    const uint32_t at = uint32_t(begin) + tot[g] + uint32_t(j);
    dst[at] = it;
    if constexpr (VALS) vdst[at] = vbuf[j];
  }
}

// Counts, tiles and status words of a sort, which share the histograms' place.
size_t scratch_bytes(int64_t NS, int32_t T, int items, int bits) {
  return size_t(tile_blocks(NS, T, items * kThreads)) *
         ((sizeof(uint16_t) << bits) + sizeof(Tile) + sizeof(int32_t));
}

template <int ITEMS>
hipError_t sort_tables(const TableDesc& d, int32_t B, const int32_t* I, const int32_t* O,
                       int64_t NS, const BwdLayout& L, char* ws, int32_t* d_status,
                       uint32_t token, const float* A, int passes, int bits, hipStream_t st) {
  const int32_t TB = d.num_tables * B, ns = int32_t(NS);
  const int blocks = tile_blocks(NS, d.num_tables, ITEMS * kThreads);
  const int32_t vb = (TB + blocks - 1) / blocks;
  uint16_t* hist = reinterpret_cast<uint16_t*>(ws + L.off_hist);
  Tile* info = reinterpret_cast<Tile*>(hist + (size_t(blocks) << bits));
  int32_t* status = reinterpret_cast<int32_t*>(info + blocks);
  int32_t* flags = reinterpret_cast<int32_t*>(ws + L.off_flags);
  // the last pass ends in the first buffer
  uint64_t* src = reinterpret_cast<uint64_t*>(ws + (passes % 2 ? L.off_b : L.off_a));
  uint64_t* dst = reinterpret_cast<uint64_t*>(ws + (passes % 2 ? L.off_a : L.off_b));
  float* vdst = reinterpret_cast<float*>(ws + (passes % 2 ? L.off_va : L.off_vb));
  float* vother = reinterpret_cast<float*>(ws + (passes % 2 ? L.off_vb : L.off_va));
  const bool two = blocks > kNumCu;
  const float* vsrc = A;  // the first pass reads the caller's weights
  hipLaunchKernelGGL(table_keys<ITEMS>, dim3(blocks), dim3(kThreads), 0, st, d, I, O, ns, B, TB, vb, bits,
                     src, hist, info, status);
  for (int p = 0; p < passes; ++p) {
    const int shift = p * bits;
    if (p > 0)
      hipLaunchKernelGGL(table_counts<ITEMS>, dim3(blocks), dim3(kThreads), 0, st, d, src, info, shift,
                         bits, hist);
#define EMB_SCATTER(VALS, FIRST)                                                                 \
  hipLaunchKernelGGL((two ? table_scatter<ITEMS, VALS, FIRST, ITEMS == 4 && !VALS> : table_scatter<ITEMS, VALS, FIRST, false>), dim3(blocks + (FIRST ? 1 : 0)),               \
                     dim3(kThreads), 0, st, d, src, dst, info, shift, bits, hist, vsrc, vdst,    \
                     status, blocks, flags, d_status, token)
    if (A != nullptr && p == 0) EMB_SCATTER(true, true);
    else if (A != nullptr) EMB_SCATTER(true, false);
    else if (p == 0) EMB_SCATTER(false, true);
    else EMB_SCATTER(false, false);
#undef EMB_SCATTER
    uint64_t* t = src;
    src = dst;
    dst = t;
    vsrc = vdst;
    vdst = vother;
    vother = const_cast<float*>(vsrc);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_sort_tables(const TableDesc& d, int32_t B, const int32_t* I, const int32_t* O,
                              int64_t NS, const BwdLayout& L, char* ws, int32_t* d_status,
                              uint32_t token, const float* A, hipStream_t st) {
  uint32_t rows = 2;  // of the largest table: its bits decide the digits
  for (int t = 0; t < d.num_tables; ++t) rows = d.rows[t] > rows ? d.rows[t] : rows;
  const int nbits = 32 - __builtin_clz(rows - 1u);
  const int fewest = (nbits + kMaxDigitBits - 1) / kMaxDigitBits;
  auto digits = [&](int passes) { return (nbits + passes - 1) / passes > 3 ? (nbits + passes - 1) / passes : 3; };
  const size_t room = L.off_tot - L.off_hist;
  auto fits = [&](int items, int passes) {
    return scratch_bytes(NS, d.num_tables, items, digits(passes)) <= room;
  };
  // Tiles of 2048 look-ups while they are at most a block per compute unit (524K
  // over 8 tables 31 us instead of 33, 213K over 26 22 instead of 27) and their
  // counts fit the workspace, of 8192 beyond a block of 4096 per compute unit
  // while they are at most one again, with a table's last half full on average
  // (1.7M look-ups over 26 tables, then over 8: 48 and 50 us instead of 54 and 62;
  // 260 blocks instead of 512 in two halves 78 instead of 58).
  if (NS <= int64_t(kNumCu) * 2 * kThreads && fits(2, fewest))
    return sort_tables<2>(d, B, I, O, NS, L, ws, d_status, token, A, fewest, digits(fewest), st);
  if (NS > int64_t(kNumCu) * 4 * kThreads &&
      NS + int64_t(d.num_tables) * 4 * kThreads <= int64_t(kNumCu) * 8 * kThreads && fits(8, fewest))
    return sort_tables<8>(d, B, I, O, NS, L, ws, d_status, token, A, fewest, digits(fewest), st);
  // A pass more where 10-bit counts do not fit: few look-ups over many tables of
  // which only one is long (62K over 64).
  int passes = fewest;
  while (passes < 4 && !fits(4, passes)) ++passes;
  if (!fits(4, passes)) return hipErrorInvalidValue;
  return sort_tables<4>(d, B, I, O, NS, L, ws, d_status, token, A, passes, digits(passes), st);
}

}  // namespace embbag
