// Which kernel a call takes, as functions of sizes and types alone: host C++
// without HIP, so that the rules can be checked on any machine.  Kernels that
// share a call's range add in the same order, so a rule may look at the group's
// size without changing an owner's bits.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace rwttt {

// READ tiling.  A work item is (group slot, K chunk, column tile).  The chunk
// and tile sizes depend only on the matrix shape, never on the group, so an
// owner's result does not depend on who else is in the group.
constexpr int kReadChunk = 256;       // K rows per work item

constexpr int read_cols_per_lane(int state_bf16) { return state_bf16 ? 8 : 4; }   // 16 B per lane
constexpr int read_tile_n(int state_bf16) { return 64 * read_cols_per_lane(state_bf16); }

// Whether the live state that a call reads (call_bytes) is loaded without the
// non-temporal hint, to stay in the 256 MB last-level cache until the next call
// that reads it.  A serving step visits every owner and layer before it comes back
// to a state, so a context whose live states and W0s (context_bytes) do not fit the
// cache keeps the hint: such loads leave no lines to be pushed out.  A context
// that fits may still share the cache, with other contexts or the rest of a model;
// a large call then loses more than it could win.  In us with / without the hint,
// by the bytes of the states visited in turn:
// * READ of two owners of 2048 x 2048 (42 MB) 13.3 / 10.9 up to 209 MB, 13.4 / 14.6 at
//   330 MB; WRITE of four of 2048 x 2048 with token (67 MB) 30.9 / 27.0 at 225 MB, 31.2 /
//   32.7 at 600 MB;
// * READ of one owner of 9728 x 2560 (149 MB) 27.4 / 25.2 when it is alone, 27.3 /
//   28.8 when two such contexts take turns, 27.4 / 31.6 with four; five of 5000 x
//   1528 (168 MB) 35.1 / 31.1, 36.0 / 36.7, 36.1 / 38.6; WRITE of one of 9728 x 2560
//   with token 47.8 / 44.0, 47.8 / 49.0, 47.8 / 51.3.
// Stores always have the hint: a candidate kept in the cache takes the place of
// a live state (one WRITE of 9728 x 2560, C = 64, 54.6 against 48.1 us).  The GEMM
// keeps it for its live tiles too: its evidence lives in L2 (62.2 against 59.6 us
// for 11 owners of 5448 x 288 bf16, C = 650).
constexpr size_t kCacheContext = 256000000;
constexpr size_t kCacheCall = 48000000;

inline bool stays_cached(size_t call_bytes, size_t context_bytes) {
  return call_bytes <= kCacheCall && context_bytes <= kCacheContext;
}

// ---------------------------------------------------------------------------
// READ
// ---------------------------------------------------------------------------

// Where the two launches are better than one (read_direct_kernel), all with the
// state from HBM, one launch / two in us:
// * a block's column of leaves reaches only about 70 GB/s, so one launch needs few
//   bytes: 11.2 / 14.3 at 512 x 4096 x 4 and 10.6 / 14.4 at 1024 x 2048 x 4 (38 MB),
//   but 16.3 / 14.9 at 1024 x 2048 x 5 (46 MB), 19.0 / 15.6 at 1000 x 3000 x 3 (42 MB);
// * a block of 16 waves takes 1.5 to 2 us of its CU however few rows it has, and
//   one fits a CU (two of bf16 io with fp32 state, the form with the fewest
//   registers), so one launch needs few blocks: bf16 io and state 8.5 / 15.2 at 256 x
//   4096 x 8 (512 blocks), 11.6 / 12.0 at 128 x 14336 x 4 (896), 16.1 / 12.5 at 128 x
//   14336 x 6 (1344), 25.0 / 8.7 at 8 x 14336 x 16 (3584); fp32 14.5 / 10.1 at 64 x
//   14336 x 4 (1792); bf16 io, fp32 state 12.3 / 14.6 at 256 x 2048 x 18 (1152), 12.4 /
//   12.2 at 128 x 14336 x 4 (1792).
constexpr size_t kDirectBytes = 38000000;
constexpr int kDirectRows = 1536;          // at most two leaves per row group
constexpr int kDirectLanes = 8;            // lanes of 16 bytes side by side: a block's columns
constexpr int kDirectBlocks = 1024;
constexpr int kDirectBlocksTwo = 1536;     // where two blocks fit a CU

struct ReadRoute {
  bool direct;               // one launch
  int waves, leaf;           // two launches: waves of a block, rows of a leaf
  bool nt;                   // live state loaded with the non-temporal hint
};

// context_bytes: live states and W0s of all owners and layers
inline ReadRoute read_route(bool io_bf16, bool state_bf16, int d_ff, int d_model, int count,
                            size_t context_bytes) {
  const size_t io = io_bf16 ? 2 : 4, state = state_bf16 ? 2 : 4;
  const size_t bytes = size_t(d_ff) * d_model * (count * state + io);
  ReadRoute r;
  const int tile = kDirectLanes * read_cols_per_lane(state_bf16);
  const int64_t blocks = int64_t((d_model + tile - 1) / tile) * count;
  r.direct = d_ff <= kDirectRows && bytes <= kDirectBytes &&
             blocks <= (io_bf16 && !state_bf16 ? kDirectBlocksTwo : kDirectBlocks);
  r.nt = !stays_cached(bytes, context_bytes);
  // leaves of eight rows where the one launch above must match, and for fp32 io
  // with bf16 state, where they are faster (14.5 against 21.4 us for one owner of
  // 3600 x 1512, 115.6 / 125.6 for eight of 9728 x 2560)
  r.leaf = d_ff <= kDirectRows || io > state ? 8 : 32;
  if (r.leaf == 32) {
    r.waves = count == 1 ? 4 : 8;
    return r;
  }
  // fp32 io with bf16 state needs 138 registers: one block of eight waves fits a CU,
  // or three of four waves, twelve waves.  Past one round of the 256 CUs the smaller
  // blocks are better, unless much of the last column tile is empty.  Eight / four
  // waves, in us: 14.5 / 14.8 at 3600 x 1512, 24.6 / 24.5 at 5000 x 1528 x 4 (239 blocks'
  // worth of columns), 38.8 / 37.5 with five owners, 115.7 / 109.2 at 9728 x 2560 x 8,
  // 260.5 / 239.7 at 14336 x 4096 x 8; 31.2 / 35.9 at 12000 x 520 x 4 and 48.0 / 51.2 with
  // eight.  Four waves forced into 128 registers spill (149 us at 9728 x 2560 x 8).
  const int ktile = read_tile_n(state_bf16), nt = (d_model + ktile - 1) / ktile;
  const bool rounds = size_t(d_ff) * d_model * count > size_t(256) * kReadChunk * ktile;
  r.waves = io > state && d_ff > kDirectRows && rounds && d_model * 4 > nt * ktile * 3 ? 4 : 8;
  return r;
}

// ---------------------------------------------------------------------------
// WRITE
// ---------------------------------------------------------------------------

constexpr int kSTM = 32;                 // streaming kernel: rows per item
constexpr int kSTN = 256;                // columns per tile
constexpr int kSMaxC = 64;               // largest chunk on this path
constexpr int kSParts = 64;              // most row-tile partitions per (owner, column tile)
constexpr int kSSlots = 512;             // blocks of this kernel resident at once (256 CUs x 2)

// Row-tile partitions per (owner, column tile), from the shape alone, so that
// an owner's token partials are added in the same order in any group: as many
// as let one owner's blocks fill one round of the block slots, then the fewest
// that keep the largest partition at the same number of items.
inline int stream_parts(int d_ff, int d_model) {
  const int mt = (d_ff + kSTM - 1) / kSTM;
  const int ntl = (d_model + kSTN - 1) / kSTN;
  const int pmax = std::max(1, std::min(std::min(kSParts, mt), kSSlots / ntl));
  const int items = (mt + pmax - 1) / pmax;
  return (mt + items - 1) / items;
}

// bf16 state and no token: whether the streaming kernel takes the call rather
// than the GEMM, whose 256 x 128 tiles are the better split from one round of
// its 512 block slots up (four owners of 9728 x 2560, C = 32: 83 / 71 us).
// Streaming / GEMM, in us:
// * up to a block of one item a CU the streaming kernel's first rows arrive
//   sooner: 4.5 / 5.6 at 264 x 136, 4.8 / 5.7 at 1000 x 264 x 2, 5.0 / 5.6 at 1024
//   x 1024 x 2, all C = 1; 5.4 / 5.9 at 2048 x 512, C = 64.  Past it 7.5 / 6.4 at
//   512 x 2048 x 4, C = 64, and 7.7 / 5.4 at 5000 x 128 (three items a block);
// * one owner whose blocks fill the slots once, state from HBM and one stage of
//   evidence: 21.2 / 22.2 at 9728 x 2560, 43.4 / 45.1 at 14336 x 4096, C = 16 (the
//   latter 46.4 / 46.0 at C = 48); rows that are no whole 128-byte lines cost the
//   GEMM's narrower tiles more, at every C: 21.0 / 23.8 at 10000 x 2000.
// * few rows leave most of the GEMM's 256 empty.  Up to 32 always: 7.6 / 12.3 at 32 x
//   14336 x 8, C = 1, 27.5 / 41.6 with 32 owners, C = 64, 16.8 / 36.5 at 8 x 14336 x 32.  Up
//   to 64 a limit: 7.8 / 8.4 at 64 x 14336 x 4, C = 64, 13.9 / 14.2 with eight owners, 27.4 /
//   24.7 with 16.  At 72 rows 12.4 / 8.7 at 72 x 14336 x 4.
constexpr size_t kSSmallElems = 2200000;   // 256 blocks of one 32 x 256 item
constexpr size_t kSFewRowsElems = 8000000;

inline bool stream_without_token(int d_ff, int d_model, int count, int chunk, size_t context_bytes) {
  const int parts = stream_parts(d_ff, d_model);
  const size_t elems = size_t(d_ff) * d_model * count;
  if (d_ff <= kSTM || (d_ff <= 2 * kSTM && elems <= kSFewRowsElems)) return true;
  if (parts * kSTM >= d_ff && elems <= kSSmallElems) return true;
  const int blocks = (d_model + kSTN - 1) / kSTN * parts;
  return count == 1 && blocks > kSSlots * 15 / 16 && blocks <= kSSlots &&
         ((context_bytes > kCacheContext && chunk <= 16) || d_model % 64 != 0);
}

constexpr int kRTM = 64;                 // register-operand kernels: rows per wave
constexpr int kRMaxC = 384;              // largest chunk without a fused token on this path
constexpr int kRMinC = 300;              // up to here always on this path, but for one full GEMM round

// With a fused token: against the streaming kernel, whose blocks start with a
// G tile staged through LDS and have few items on a small state, in us: 1000 x
// 4000, C = 20, two owners 15.9 / 19.8, C = 64, eight 59.8 / 72.8; 2496 x 824 x 1,
// C = 64, 11.9 / 12.9; 2000 x 2000 x 6, C = 20, 48.1 / 54.9; 4096 x 1024, C = 16, three
// 26.0 / 27.4, C = 64, eight 59.6 / 60.1.  Outside the rule: few columns are
// padded to 256 (45.9 / 44.7 at 3000 x 296 x 16, C = 64); blocks two waves wide, for
// more rows, win with few owners (26.7 / 31.2 at 6000 x 600 x 3) and lose with many
// (69.6 / 64.3 with eight, 106.0 / 91.8 at 8000 x 1000 x 6), and one wave wide
// lose (137.5 / 118.7 at 14000 x 1400 x 3); bf16 state has half the bytes for the
// same evidence loads (36.8 / 34.5 at 9728 x 2560).  Inside it, rows that are no
// whole 128-byte lines and columns padded by an eighth or more win with one owner
// and lose with many: 10.9 / 12.3 at 2496 x 824 x 1, C = 40, but 43.6 / 39.9 with
// eight owners; 12.8 / 13.6 and 66.0 / 62.4 at 4000 x 904; 11.1 / 12.7 and 48.6 / 46.5 at
// 3000 x 776; 11.0 / 12.3 and 45.1 / 45.4 at 4096 x 520.  The rule looks at the matrix
// alone: the two kernels add a token's rows in different orders.
constexpr size_t kRTokenElems = size_t(4) << 20;

inline bool rows_token(int d_ff, int d_model) {
  return d_ff <= kRTM * kSParts && d_model >= 512 && size_t(d_ff) * d_model <= kRTokenElems;
}

constexpr int kGTM = 256;                // GEMM: rows (d_ff) per tile
constexpr int kGTN = 128;                // columns (d_model) per tile
constexpr int kGColGroups = 2;           // column-tile groups over the XCDs
constexpr int kGRowClasses = 8 / kGColGroups;             // row-tile classes over the XCDs

struct GemmTile {
  int b, mt, nt;             // group slot, row tile, column tile; a tile past the end is idle
};

// Whether the classes below would leave XCDs without a tile: then the tiles are
// dealt to the XCDs one by one.  In us, by classes / one by one, bf16 state: eight
// owners of 256 x 4096, C = 16, 18.4 / 8.1, C = 128 22.4 / 9.9; of 128 x 14336,
// C = 64, 43.8 / 16.6; of 512 x 2048, C = 16, 12.6 / 7.8; of 5000 x 128, C = 16,
// 9.5 / 6.2.  Where every XCD has work the classes keep evidence in its L2: 30.2 /
// 31.9 for eight of 2048 x 2048, C = 128; 7.6 / 8.0 for four of 1000 x 264.
constexpr bool gemm_few_tiles(int mt, int ntl) { return mt < kGRowClasses || ntl < kGColGroups; }

// Block -> tile.  Blocks are dealt to the 8 XCDs round-robin; XCD x takes
// column-tile half x % 2 and the row tiles congruent to x / 2 mod 4, so each Z
// row tile is read by two XCDs and each G column tile by four.  Consecutive
// blocks of an XCD share their Z row tile, and the XCD's G columns (2 MB at C =
// 512) stay in its L2 while the live state streams past them non-temporally.
constexpr GemmTile gemm_tile(unsigned block, int mt, int ntl) {
  if (gemm_few_tiles(mt, ntl)) {
    const int row = int(block) / ntl;
    return {row / mt, row % mt, int(block) % ntl};
  }
  const int xcd = block & 7;
  const int pos = block >> 3;
  const int ntg = (ntl + kGColGroups - 1) / kGColGroups;
  const int mtq = (mt + kGRowClasses - 1) / kGRowClasses;
  const int rest = pos / ntg;
  const int b = rest / mtq;
  return {b, (rest - b * mtq) * kGRowClasses + xcd / kGColGroups, (xcd % kGColGroups) * ntg + pos % ntg};
}

constexpr unsigned gemm_blocks(int count, int mt, int ntl) {
  if (gemm_few_tiles(mt, ntl)) return unsigned(count) * unsigned(mt) * unsigned(ntl);
  const unsigned ntg = unsigned((ntl + kGColGroups - 1) / kGColGroups);
  const unsigned mtq = unsigned((mt + kGRowClasses - 1) / kGRowClasses);
  return unsigned(count) * mtq * ntg * 8u;
}

constexpr int kGSlots = 64;               // GEMM blocks resident at once on an XCD (32 CUs x 2)

// Largest chunk of an fp32 state without a fused token for the register-operand
// kernel, whose time grows by about 3 us for 1000 ranks of a million elements; the
// GEMM's grows half as fast from a higher start, which is the higher the less its
// tiles fill the rounds of its block slots (the XCD with most tiles counts).
// Register operands / GEMM, in us:
// * filled to 0.95 and more, C = 300: 436 / 427 at 14336 x 4096 x 4, 72.7 / 66.6 at 8192 x
//   4096 x 1, but 75.8 / 79.5 at 2048 x 2048 x 8 and 104 / 113 at 6144 x 2048 x 4; C = 384: 494 /
//   443, 82.8 / 69.5, 84.8 / 83.3, 116 / 118, 291 / 258 at 4096 x 4096 x 8;
// * to 0.91: 173 / 162 at 5000 x 1528 x 8, C = 384, 398 / 423 at 9728 x 2560 x 8, C = 320,
//   441 / 442 at 384;
// * less: 153 / 171 at 9728 x 2560 x 3, C = 320, 169 / 177 at 384; 33.0 / 37.6 at 2000 x 2000 x
//   3, 54.0 / 61.8 at 2496 x 824 x 8, C = 384; the exception 136 / 120 at 14336 x 4096 x 1;
// * one round, filled: 36.2 / 33.3 at 4096 x 4096 x 1, C = 192, 36.7 / 38.7 at 8192 x 2048 x 1,
//   37.4 / 36.5 at 2048 x 1024 x 8, C = 200; 43.6 / 41.2 and 44.3 / 39.2 at C = 300.
// Both kernels add in the same order, so the group may be looked at.
inline int rows_max_chunk(int d_ff, int d_model, int count) {
  const int mt = (d_ff + kGTM - 1) / kGTM, ntl = (d_model + kGTN - 1) / kGTN;
  if (gemm_few_tiles(mt, ntl)) return kRMaxC;
  const int64_t most = int64_t(count) * ((mt + kGRowClasses - 1) / kGRowClasses) *
                       ((ntl + kGColGroups - 1) / kGColGroups);
  const int64_t rounds = (most + kGSlots - 1) / kGSlots;
  const double fill = double(d_ff) * d_model * count / (double(rounds) * kGSlots * 8 * kGTM * kGTN);
  if (rounds == 1 && fill >= 0.95) return 220;
  // from kRMinC where the rounds are full to kRMaxC at nine tenths
  return std::min(kRMaxC, kRMinC + int((kRMaxC - kRMinC) * 10 * (1 - fill)));
}

enum class WriteKernel { f32, rows_token, stream, rows, gemm };

struct WriteRoute {
  WriteKernel kernel;
  bool read_first;           // the token is a READ of the group before the update
  int wn;                    // f32: waves of a block side by side
  bool nt;                   // live state loaded with the non-temporal hint
};

inline WriteRoute write_route(bool io_bf16, bool state_bf16, int d_ff, int d_model, int count, int chunk,
                              bool token, size_t context_bytes) {
  WriteRoute r = {WriteKernel::gemm, false, 0, true};
  r.nt = !stays_cached(size_t(d_ff) * d_model * count * (state_bf16 ? 2 : 4), context_bytes);
  if (!io_bf16) {
    r.kernel = WriteKernel::f32;
    // without a token nothing limits the rows of a block
    r.wn = !token || d_ff * 4 <= kReadChunk * kSParts ? 4 : d_ff * 2 <= kReadChunk * kSParts ? 2 : 1;
    return r;
  }
  if (token && chunk <= kSMaxC) {
    r.kernel = !state_bf16 && rows_token(d_ff, d_model) ? WriteKernel::rows_token : WriteKernel::stream;
    return r;
  }
  r.read_first = token;
  if (!state_bf16 && chunk <= rows_max_chunk(d_ff, d_model, count)) r.kernel = WriteKernel::rows;
  if (state_bf16 && chunk <= kSMaxC && stream_without_token(d_ff, d_model, count, chunk, context_bytes)) {
    r.kernel = WriteKernel::stream;
    r.nt = true;             // also in a small context: 4.8 / 5.1 us with / without at 512 x 2048, C = 1
  }
  return r;
}

// ---------------------------------------------------------------------------
// Adapter WRITE
// ---------------------------------------------------------------------------

// Tiles of 16 evidence rows per block of the kernel that forms the products of
// evidence and factors; slices: 1024-element slices of both extents.  A row's sums
// do not depend on it.  One tile while its blocks fit the 256 CUs in one round:
// larger ones only leave CUs idle.  In us, one tile / as below: 10.2 / 15.8 at 2000 x
// 520 x 1, rank 1, C = 129 (27 blocks), 9.0 / 11.0 at 4608 x 304 x 1, C = 100, 11.4 / 13.8 at
// 264 x 136 x 8, rank 20, C = 100, 13.8 / 16.8 at 4608 x 304 x 4 (168 blocks).  Past one
// round 14.4 / 13.0 at 512 x 4096 x 8, rank 16, C = 100 (280 blocks), 16.6 / 15.1 at 14336 x
// 4096 x 4, C = 64 (288), 24.9 / 24.2 at 9728 x 2560 x 4, C = 256 (832).
inline int adapter_pq_tiles(int slices, int chunk, int count, int rank) {
  if (int64_t(slices) * ((chunk + 15) / 16) * count <= 256) return 1;
  return rank <= 16 && chunk > 128 ? 4 : 2;
}

}  // namespace rwttt
