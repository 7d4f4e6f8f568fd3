// gfx950 kernels of the owner-scoped fast-weight READ/WRITE path.
//
// READ  (ApplyState, Section 3 "Read"):   y_r = x_r W0 + x_r dW_r
// WRITE (BoundaryUpdate, Section 3 "Write"): shadow_r = live_r + eta Z_r^T G_r
//
// Both operate on groups of owners, one launch per (group, layer).

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "rwttt_kernels.h"

namespace rwttt {
namespace {

#include "rwttt_device.h"

// ---------------------------------------------------------------------------
// READ
// ---------------------------------------------------------------------------
//
// y_b = x_b W0 + x_b dW_b, as two launches with no cross-block
// synchronisation (one launch for few rows and bytes, below):
//
// 1. read_partial_kernel: one block of eight waves per (group slot b, K chunk of
//    256 rows, column tile).  Each lane owns 16 contiguous bytes of every dW_b
//    row of the tile (4 fp32 or 8 bf16 columns) and the same columns of W0;
//    the waves split the chunk's rows.  Per row it accumulates
//    x[k]*dW[k] and then x[k]*W0[k] into one fp32 accumulator, so the shared
//    W0 term is fused into the same pass.  The W0 tile is the same for every
//    slot: the blocks of all slots for one (chunk, tile) are placed on one XCD
//    (dispatch is round-robin over the 8 XCDs by block index) so that W0 comes
//    from HBM once and is re-read from that XCD's L2.  Which XCD takes a pair
//    rotates with the pair's round of eight: with 10 column tiles a fixed
//    pair % 8 gave the even XCDs only even tiles, whose blocks ran ~7% slower
//    than the odd tiles' (3% once every XCD mixes both: an address effect,
//    not an XCD one), so those XCDs finished last.  dW is streamed with
//    non-temporal loads so it does not evict W0.  The waves' sums are added
//    through LDS as a tree into one partial per (owner, chunk).
//    A wave has 32 rows, four rounds of loads: with four waves of 64 rows a
//    call took 129.3 against 127.9 us (8 owners of 9728 x 2560), 37.6 against
//    36.5 (5 of 5000 x 1528) and 14.4 against 10.7 us (6 of 5496 x 88, fp32),
//    where the chain of rounds is all there is.  More in flight (16 rows at a
//    time, or 16 waves) is slower: 142-147 us for the first.  One owner alone
//    keeps the four-wave block, 64 rows as two leaves of 32, so that the bits
//    are the same: 27.5 against 27.8 us at 9728 x 2560.  So do large calls of bf16
//    state with fp32 io, as eight leaves of 8.
// 2. read_reduce_kernel: y[b, n] = sum over chunks: four contiguous quarters
//    of the chunks, each in chunk order, added in order (as a tree for few
//    rows).
//
// Partials are indexed by owner id, so concurrent reads of disjoint owner sets
// (one per stream) never touch the same workspace bytes.
//
// Every order depends only on the matrix shape and types, so an owner's y is
// bit-identical whatever the group's size, order or other members.  The group
// only chooses between kernels that add in the same order.

struct ReadParams {
  const void* x;
  void* y;
  const void* w0;
  float* part;
  int count, d_ff, d_model, ks, nt, npad;
  int slot_part;             // partial sums indexed by group slot (1) or by owner id (0)
  const void* dw[RWTTT_MAX_GROUP];
  uint32_t row[RWTTT_MAX_GROUP];
  void* tail[RWTTT_MAX_GROUP];     // TailBufferUpdate: row receiving x, or null
};

constexpr int kUnroll = 8;        // rows whose loads are in flight at once; the row count is a multiple

// Fold a stack of 2^n equal-sized sums into their balanced tree: s[i] enters in
// order, pairs are added as soon as both are there.
template <int N, int COLS>
__device__ __forceinline__ void tree_push(float (&stack)[N][COLS], int i, const float (&v)[COLS]) {
  // i is a compile-time constant in every (unrolled) call: level l of the stack
  // is the carry of bit l
  float t[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) t[c] = v[c];
  int l = 0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (!((i >> k) & 1)) break;
#pragma unroll
    for (int c = 0; c < COLS; ++c) t[c] = stack[k][c] + t[c];
    l = k + 1;
  }
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (k == l)
#pragma unroll
      for (int c = 0; c < COLS; ++c) stack[k][c] = t[c];
}

// Balanced tree over N (a power of two) values in index order.
template <int N> __device__ __forceinline__ float tree_sum(float (&v)[N]) {
#pragma unroll
  for (int k = 1; k < N; k *= 2)
#pragma unroll
    for (int i = 0; i + k < N; i += 2 * k) v[i] += v[i + k];
  return v[0];
}

template <typename IO, typename ST, int NW, int LEAF, bool NT>
__global__ void __launch_bounds__(64 * NW) read_partial_kernel(const ReadParams p) {
  constexpr int COLS = 16 / sizeof(ST);
  constexpr int TILE_N = 64 * COLS;
  constexpr int KC = kReadChunk;
  constexpr int RW = KC / NW;
  __shared__ float xs[KC];
  __shared__ float red[NW][TILE_N];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // block -> (XCD, position on that XCD) -> ((chunk, tile) pair, slot).  Round
  // pl of eight pairs is dealt to the XCDs rotated by pl, so that each XCD
  // gets column tiles of both parities even when the tile count is even
  const int xcd = blockIdx.x & 7;
  const int pos = blockIdx.x >> 3;
  const int pl = pos / p.count;
  const int b = pos - pl * p.count;
  const int pair = pl * 8 + ((xcd + pl) & 7);
  if (pair >= p.ks * p.nt) return;
  const int kc = pair / p.nt;
  const int nt = pair - kc * p.nt;
  const int k0 = kc * KC;
  const int kn = min(KC, p.d_ff - k0);
  const int col = nt * TILE_N + lane * COLS;
  const bool col_ok = col < p.d_model;

  for (int k = tid; k < KC; k += 64 * NW)
    xs[k] = k < kn ? Elem<IO>::get(p.x, size_t(p.row[b]) * p.d_ff + k0 + k) : 0.f;
  if (p.tail[b] != nullptr && nt == 0) {
    // TailBufferUpdate: the first column tile's blocks append this chunk of x
    const IO* xr = static_cast<const IO*>(p.x) + size_t(p.row[b]) * p.d_ff + k0;
    IO* tr = static_cast<IO*>(p.tail[b]) + k0;
    for (int k = tid; k < kn; k += 64 * NW) tr[k] = xr[k];
  }
  __syncthreads();

  // leaves of LEAF rows, each a chain from zero, eight rows' loads in flight at
  // once (eight rows are inside or outside the matrix together)
  constexpr int NL = RW / LEAF;
  constexpr int LV = NL == 8 ? 4 : NL == 4 ? 3 : NL;     // log2(NL) + 1
  float stack[LV][COLS];
  const ST* dbase = static_cast<const ST*>(p.dw[b]) + size_t(k0) * p.d_model + col;
  const IO* wbase = static_cast<const IO*>(p.w0) + size_t(k0) * p.d_model + col;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    float acc[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) acc[c] = 0.f;
    const int kend = col_ok ? min(wave * RW + (i + 1) * LEAF, kn) : 0;
    for (int k = wave * RW + i * LEAF; k < kend; k += kUnroll) {
      Packed<ST, COLS> v[kUnroll];
      Packed<IO, COLS> w[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        load_packed<NT>(dbase + size_t(k + u) * p.d_model, v[u]);
        load_packed<false>(wbase + size_t(k + u) * p.d_model, w[u]);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const float xv = xs[k + u];
#pragma unroll
        for (int c = 0; c < COLS; ++c) acc[c] = fmaf(xv, w[u].get(c), fmaf(xv, v[u].get(c), acc[c]));
      }
      if constexpr (LEAF == kUnroll) break;
    }
    tree_push<LV>(stack, i, acc);
  }
#pragma unroll
  for (int c = 0; c < COLS; ++c) red[wave][lane * COLS + c] = stack[LV - 1][c];
  __syncthreads();
  const uint32_t prow = p.slot_part ? uint32_t(b) : p.row[b];
  float* dst = p.part + (size_t(prow) * p.ks + kc) * p.npad + nt * TILE_N;
  for (int j = tid; j < TILE_N; j += 64 * NW) {
    float v[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) v[w] = red[w][j];
    dst[j] = tree_sum<NW>(v);
  }
}

// 64 output columns per block; the four waves each add a contiguous quarter of
// the chunks with all of its loads in flight at once.  Up to 8 chunks: the
// quarters of the next power of two, and everything added as a tree (a READ of
// so few rows may run in read_direct_kernel, which must give the same bits).
// More: each quarter in chunk order, the quarters in order.
constexpr int kRedCols = 64;
constexpr int kRedBatch = 16;
constexpr int kTreeChunks = 8;

template <typename IO, bool TREE>
__global__ void __launch_bounds__(256) read_reduce_kernel(const ReadParams p) {
  __shared__ float qs[4][kRedCols];
  const int b = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = blockIdx.x * kRedCols + lane;
  const int per = !TREE ? (p.ks + 3) / 4 : p.ks > 4 ? 2 : 1;
  const int k0 = wave * per, k1 = min(p.ks, k0 + per);
  float s = 0.f;
  if (n < p.d_model) {
    const uint32_t prow = p.slot_part ? uint32_t(b) : p.row[b];
    const float* q = p.part + size_t(prow) * p.ks * p.npad + n;
    if constexpr (TREE) {
      float a[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) a[u] = k0 + u < k1 ? q[size_t(k0 + u) * p.npad] : 0.f;
      s = a[0] + a[1];
    } else {
      for (int k = k0; k < k1; k += kRedBatch) {
        float a[kRedBatch];
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u) a[u] = k + u < k1 ? q[size_t(k + u) * p.npad] : 0.f;
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u) s += a[u];
      }
    }
  }
  qs[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && n < p.d_model) {
    const float a = qs[0][lane] + qs[1][lane], c = qs[2][lane], d = qs[3][lane];
    Elem<IO>::put(p.y, size_t(p.row[b]) * p.d_model + n, TREE ? a + (c + d) : (a + c) + d);
  }
}

// READ of few rows and bytes, one launch: a block owns a narrow column tile
// (eight lanes of 16 bytes) and all rows, so nothing is left to add across
// blocks.  Its 16 waves x 8 row groups take LEAVES leaves each, whose loads are
// all independent, so a call is one round trip to memory instead of several
// and a second launch: two owners of 256 x 64 fp32 7.4 us (the host's time for
// the call) against 11.2 before, four of 976 x 1920 8.1 against 16.8.  The same
// tree over the same leaves of eight rows as the two launches.
constexpr int kDirectThreads = 1024;
constexpr int kDirectGroups = kDirectThreads / kDirectLanes;
constexpr int kDirectLeaf = kUnroll;
static_assert(kDirectRows <= 2 * kDirectGroups * kDirectLeaf && kDirectRows <= kTreeChunks * kReadChunk, "");

template <typename IO, typename ST, int LEAVES>
__global__ void __launch_bounds__(kDirectThreads) read_direct_kernel(const ReadParams p) {
  constexpr int COLS = 16 / sizeof(ST);
  constexpr int TILE_N = kDirectLanes * COLS;
  constexpr int NW = kDirectThreads / 64;
  constexpr int LV = LEAVES;                             // log2(LEAVES) + 1
  __shared__ float red[NW][TILE_N];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // block -> (XCD, position) -> (column tile, slot): the slots of one tile sit
  // on one XCD, which keeps their W0 columns in its L2
  const int xcd = blockIdx.x & 7;
  const int pos = blockIdx.x >> 3;
  const int pl = pos / p.count;
  const int b = pos - pl * p.count;
  const int nt = pl * 8 + xcd;
  if (nt >= p.nt) return;
  const int cl = lane % kDirectLanes;
  const int cc = min(nt * TILE_N + cl * COLS, p.d_model - COLS);   // past the matrix: not stored
  const IO* x = static_cast<const IO*>(p.x) + size_t(p.row[b]) * p.d_ff;
  const ST* d = static_cast<const ST*>(p.dw[b]) + cc;
  const IO* w0 = static_cast<const IO*>(p.w0) + cc;
  float stack[LV][COLS];
#pragma unroll
  for (int i = 0; i < LEAVES; ++i) {
    const int k = ((tid / kDirectLanes) * LEAVES + i) * kDirectLeaf;
    float acc[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) acc[c] = 0.f;
    if (k < p.d_ff) {
      Packed<ST, COLS> v[kDirectLeaf];
      Packed<IO, COLS> w[kDirectLeaf];
      float xv[kDirectLeaf];
#pragma unroll
      for (int u = 0; u < kDirectLeaf; ++u) {
        xv[u] = Elem<IO>::get(x, k + u);
        load_packed<false>(d + size_t(k + u) * p.d_model, v[u]);
        load_packed<false>(w0 + size_t(k + u) * p.d_model, w[u]);
      }
#pragma unroll
      for (int u = 0; u < kDirectLeaf; ++u)
#pragma unroll
        for (int c = 0; c < COLS; ++c) acc[c] = fmaf(xv[u], w[u].get(c), fmaf(xv[u], v[u].get(c), acc[c]));
    }
    tree_push<LV>(stack, i, acc);
  }
#pragma unroll
  for (int m = kDirectLanes; m < 64; m <<= 1)
#pragma unroll
    for (int c = 0; c < COLS; ++c) stack[LV - 1][c] += __shfl_xor(stack[LV - 1][c], m);
  if (lane < kDirectLanes)
#pragma unroll
    for (int c = 0; c < COLS; ++c) red[wave][cl * COLS + c] = stack[LV - 1][c];
  if (p.tail[b] != nullptr && nt == 0) {
    // TailBufferUpdate: the first column tile's block appends x
    IO* tr = static_cast<IO*>(p.tail[b]);
    for (int k = tid; k < p.d_ff; k += kDirectThreads) tr[k] = x[k];
  }
  __syncthreads();
  const int n = nt * TILE_N + tid;
  if (tid < TILE_N && n < p.d_model) {
    float v[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) v[w] = red[w][tid];
    Elem<IO>::put(p.y, size_t(p.row[b]) * p.d_model + n, tree_sum<NW>(v));
  }
}

// ---------------------------------------------------------------------------
// WRITE: shadow = live + eta Z^T G
// ---------------------------------------------------------------------------

struct WriteParams {
  int count, chunk, d_ff, d_model, mt, ntl;
  int parts, npadw;          // streaming path: row-tile partitions per owner; token partial pitch
  float eta;
  const void* x;             // fused token: [n_owners, d_ff] owner-indexed inputs, or null
  const void* w0;            // fused token: W0 of the layer
  float* tpart;              // fused token: [n_owners][parts][npadw] partial sums
  const void* live[RWTTT_MAX_GROUP];
  void* shadow[RWTTT_MAX_GROUP];
  const void* z[RWTTT_MAX_GROUP];
  const void* g[RWTTT_MAX_GROUP];
  uint32_t row[RWTTT_MAX_GROUP];   // owner id of each group slot
};

// ---------------------------------------------------------------------------
// WRITE, bf16 evidence, small chunk (C <= 64): streaming rank-C update
// ---------------------------------------------------------------------------
//
// For C <= 64 the update moves 2 x |dW| bytes for only 2C flop per element,
// so it is HBM-bound and must stream like a copy: what matters is how many
// bytes each CU keeps in flight.  Each block owns one (group slot, 256-column
// tile, partition) and walks the partition's 32-row items (row tiles part,
// part + P, part + 2P, ...; P fixed by the shape).  The owner's G tile is
// staged once per block into LDS, transposed to rank-contiguous rows.  Per
// item, everything the next item needs from HBM (its live rows, its Z tile,
// and for the token its W0 rows and x values) is requested first; then Z's
// 32 x C tile goes through LDS to rank-contiguous rows, the MFMAs form
// D[m][n] = sum_c Z[c][m] G[c][n], the accumulators go through LDS, and every
// wave reads, updates and stores whole 1 KB rows of the slot.  No load is on
// the critical path of the item that issues it.
//
// For the fused token (the WRITE step's own output, read at version v before
// the candidate is committed) the block also loads the same rows of W0 and
// accumulates x[m] * live[m] + x[m] * W0[m] over its items: the live state is
// read once for both the token and the update.  Per-(owner, partition)
// partials are reduced in partition order by read_reduce_kernel.  The blocks
// of all slots for one (tile, partition) sit on one XCD so that W0 comes from
// HBM once.  The partition of an owner's rows never depends on the group, so
// an owner's token and candidate are bit-identical in any group.

constexpr int kSPitch = kSMaxC + 8;      // bf16 per staged rank row (144 B: 16 rows hit 16 bank groups)

// Rows m0 + 8 wave .. + 7 of a [d_ff, d_model] matrix, 4 columns at ncol.  The
// live state is read once (non-temporal); W0 is read by every slot of the
// group from the same XCD and must stay in its L2 (NT = false).
template <bool NT = true, typename T>
__device__ __forceinline__ void stream_load_rows(const T* base, int d_ff, int d_model, int m0,
                                                 int wave, int ncol, bool ncol_ok,
                                                 Packed<T, 4> (&v)[kSTM / 4]) {
#pragma unroll
  for (int rr = 0; rr < kSTM / 4; ++rr) {
    const int m = m0 + wave * (kSTM / 4) + rr;
    if (m < d_ff && ncol_ok) load_packed<NT>(base + size_t(m) * d_model + ncol, v[rr]);
    else v[rr].zero();
  }
}

// Ranks 2cp, 2cp+1 of eight consecutive rows starting at r0 of a rank-major
// [C][ld] bf16 matrix (threads 0..127: cp = tid / 4, rows r0 + 8 (tid % 4)).
__device__ __forceinline__ void stream_load_pair(const uint16_t* M, int ld, int rows, int chunk,
                                                 int r0, int tid, uint4& a, uint4& b) {
  a = make_uint4(0, 0, 0, 0);
  b = make_uint4(0, 0, 0, 0);
  const int cp = tid >> 2, r = r0 + (tid & 3) * 8, c = 2 * cp;
  if (tid < 128 && r < rows) {
    if (c < chunk) a = *reinterpret_cast<const uint4*>(M + size_t(c) * ld + r);
    if (c + 1 < chunk) b = *reinterpret_cast<const uint4*>(M + size_t(c + 1) * ld + r);
  }
}

// ...and their transpose into rank-contiguous LDS rows dst[row][rank].
__device__ __forceinline__ void stream_store_pair(uint16_t* dst, int tid, int row0, uint4 a,
                                                  uint4 b) {
  if (tid >= 128) return;
  const int cp = tid >> 2, r = row0 + (tid & 3) * 8;
  const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    *reinterpret_cast<uint32_t*>(&dst[(r + 2 * q) * kSPitch + 2 * cp]) = (x[q] & 0xffffu) | (y[q] << 16);
    *reinterpret_cast<uint32_t*>(&dst[(r + 2 * q + 1) * kSPitch + 2 * cp]) = (x[q] >> 16) | (y[q] & 0xffff0000u);
  }
}

template <typename ST, bool TOKEN, bool NT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
write_stream_kernel(const WriteParams p) {
  constexpr int RPW = kSTM / 4;           // epilogue rows per wave
  constexpr int KSMAX = kSMaxC / 16;      // MFMA k-steps
  __shared__ __attribute__((aligned(16))) uint16_t zt[kSTM * kSPitch];
  __shared__ __attribute__((aligned(16))) uint16_t gt[kSTN * kSPitch];
  __shared__ __attribute__((aligned(16))) float out[kSTM * kSTN];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int half = lane >> 5;
  // block -> (XCD, position) -> ((tile, partition) pair, slot)
  const int xcd = blockIdx.x & 7;
  const int pos = blockIdx.x >> 3;
  const int pl = pos / p.count;
  const int b = pos - pl * p.count;
  const int pair = pl * 8 + xcd;
  if (pair >= p.ntl * p.parts) return;
  const int nt = pair / p.parts;
  const int part = pair - nt * p.parts;   // parts <= mt: every partition has an item
  const int n0 = nt * kSTN;
  const int ncol = n0 + lane * 4;
  const bool ncol_ok = ncol < p.d_model;
  const int ksteps = (p.chunk + 15) / 16;
  const float eta = p.eta;
  const ST* live = static_cast<const ST*>(p.live[b]);
  ST* shadow = static_cast<ST*>(p.shadow[b]);
  const uint16_t* Z = static_cast<const uint16_t*>(p.z[b]);
  const uint16_t* G = static_cast<const uint16_t*>(p.g[b]);
  const uint16_t* W0 = static_cast<const uint16_t*>(p.w0);
  const uint16_t* X = static_cast<const uint16_t*>(p.x) + size_t(p.row[b]) * p.d_ff;

  // G tile [C ranks][256 n] -> gt[n][rank], 32 columns per thread pass.
  // Every G request and every request of the first item goes out before
  // any of them is used, so the block's start costs one memory round trip
  // (each use of a value loaded under a lane condition waits for all
  // outstanding loads).
  uint4 ga[kSTN / 32], gb[kSTN / 32];
#pragma unroll
  for (int j = 0; j < kSTN / 32; ++j)
    stream_load_pair(G, p.d_model, p.d_model, p.chunk, n0 + j * 32, tid, ga[j], gb[j]);

  // the first item's operands
  float yacc[4] = {0.f, 0.f, 0.f, 0.f};
  Packed<ST, 4> lv[RPW];
  Packed<uint16_t, 4> wv[RPW];
  uint4 za, zb, xq = make_uint4(0, 0, 0, 0);
  stream_load_rows<NT>(live, p.d_ff, p.d_model, part * kSTM, wave, ncol, ncol_ok, lv);
  stream_load_pair(Z, p.d_ff, p.d_ff, p.chunk, part * kSTM, tid, za, zb);
  if constexpr (TOKEN) {
    stream_load_rows<false>(W0, p.d_ff, p.d_model, part * kSTM, wave, ncol, ncol_ok, wv);
    if (part * kSTM + wave * RPW < p.d_ff)
      xq = *reinterpret_cast<const uint4*>(X + part * kSTM + wave * RPW);
  }
#pragma unroll
  for (int j = 0; j < kSTN / 32; ++j) stream_store_pair(gt, tid, j * 32, ga[j], gb[j]);

  for (int mt = part; mt < p.mt; mt += p.parts) {
    const int m0 = mt * kSTM;
    const int mn = mt + p.parts;
    stream_store_pair(zt, tid, 0, za, zb);
    __syncthreads();
    // the next item's operands load while this one is computed and stored
    Packed<ST, 4> nx[RPW];
    Packed<uint16_t, 4> nw[RPW];
    uint4 nxq = make_uint4(0, 0, 0, 0);
    if (mn < p.mt) {
      stream_load_rows<NT>(live, p.d_ff, p.d_model, mn * kSTM, wave, ncol, ncol_ok, nx);
      stream_load_pair(Z, p.d_ff, p.d_ff, p.chunk, mn * kSTM, tid, za, zb);
      if constexpr (TOKEN) {
        stream_load_rows<false>(W0, p.d_ff, p.d_model, mn * kSTM, wave, ncol, ncol_ok, nw);
        if (mn * kSTM + wave * RPW < p.d_ff)
          nxq = *reinterpret_cast<const uint4*>(X + mn * kSTM + wave * RPW);
      }
    }
    f32x16_t acc[2] = {f32x16_t{}, f32x16_t{}};
#pragma unroll
    for (int s = 0; s < KSMAX; ++s) {
      if (s < ksteps) {
        const int kofs = s * 16 + half * 8;
        const bf16x8_t az = *reinterpret_cast<const bf16x8_t*>(&zt[(lane & 31) * kSPitch + kofs]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bf16x8_t bg = *reinterpret_cast<const bf16x8_t*>(
              &gt[((wave * 2 + i) * 32 + (lane & 31)) * kSPitch + kofs]);
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(az, bg, acc[i], 0, 0, 0);
        }
      }
    }
    // accumulator register 4q+e of lane l holds D[8q + 4(l/32) + e][l % 32]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        out[(8 * (r >> 2) + 4 * half + (r & 3)) * kSTN + (wave * 2 + i) * 32 + (lane & 31)] = acc[i][r];
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr) {
      const int row = wave * RPW + rr;
      const int m = m0 + row;
      if (m < p.d_ff && ncol_ok) {
        float o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = lv[rr].get(c) + eta * out[row * kSTN + lane * 4 + c];
        store_n<4, true>(shadow + size_t(m) * p.d_model + ncol, o);
      }
    }
    if constexpr (TOKEN) {
      // token: x[m] * live[m] + x[m] * W0[m] over this wave's rows, in row order
      const uint32_t xw[4] = {xq.x, xq.y, xq.z, xq.w};
#pragma unroll
      for (int rr = 0; rr < RPW; ++rr) {
        const float xv = (rr & 1) ? bf16_hi(xw[rr >> 1]) : bf16_lo(xw[rr >> 1]);
#pragma unroll
        for (int c = 0; c < 4; ++c) yacc[c] = fmaf(xv, wv[rr].get(c), fmaf(xv, lv[rr].get(c), yacc[c]));
      }
    }
    if (mn < p.mt) {
#pragma unroll
      for (int rr = 0; rr < RPW; ++rr) {
        lv[rr] = nx[rr];
        if constexpr (TOKEN) wv[rr] = nw[rr];
      }
      xq = nxq;
    }
    __syncthreads();
  }

  if constexpr (TOKEN) {
    // the four waves' token sums in wave order -> one partial per (owner, partition)
#pragma unroll
    for (int c = 0; c < 4; ++c) out[wave * kSTN + lane * 4 + c] = yacc[c];
    __syncthreads();
    const float v = ((out[tid] + out[kSTN + tid]) + out[2 * kSTN + tid]) + out[3 * kSTN + tid];
    p.tpart[(size_t(p.row[b]) * p.parts + part) * p.npadw + n0 + tid] = v;
  }
}

// ---------------------------------------------------------------------------
// WRITE, bf16 evidence, bf16 state or large chunk: tiled GEMM
// ---------------------------------------------------------------------------
//
// At C = 512 the update does 2C flop per state element and is near the MFMA
// ridge, so it is organised as a GEMM: D = Z^T G per 256-row (d_ff) x
// 128-column (d_model) tile, four waves of 64 x 128 (2 x 4 MFMA 32x32x16
// blocks, 128 accumulators per lane), two blocks per CU.  The two blocks of
// a CU run independently, so one block's HBM-bound epilogue (read live,
// write shadow) overlaps the other's MFMA main loop.
//
// Operand staging uses no registers: Z and G arrive rank-major and are
// copied as they are, 16 bytes per lane, by buffer loads that write LDS
// directly (lane l of a load lands at LDS offset 16 l).  Ranks are consumed
// in stages of 32 (A: 32 x 256 of Z, B: 32 x 128 of G, 24 KB), three stages
// in flight; each wait names how many newer copies may still be
// outstanding.  The buffer range check turns every 16-byte group outside the
// chunk or the matrix into zeros, so ragged tiles need no other code.  The
// MFMA operands (8 consecutive ranks of one row m or column n) are read back
// with the transposing LDS read ds_read_b64_tr_b16: within each 16-lane
// group, lane i receives element i % 4 of the 8-byte runs addressed by lanes
// 4j + i / 4, so lanes 4j + q address rank row j, columns 4q..4q+3 and two
// such reads give one operand.  The 16-byte groups of rank row r sit in slot
// (group ^ swz(r & 3)), swz = {0, 10, 4, 14}, chosen so that every
// transposing read is free of bank conflicts.
//
// The MFMA is issued as D^T = G^T Z, so the accumulators of a lane hold runs
// of four consecutive columns of one state row.  The epilogue combines them
// with the live rows in that layout (bf16 state: live copied non-temporally
// into the freed stages; fp32 state: a register epilogue through a private LDS region) and
// stores whole rows, rounding to bf16 with the hardware packed convert.

constexpr int kGKC = 32;                                  // ranks per LDS stage
constexpr int kGThreads = 256;                            // 4 waves of 64 x 128
constexpr int kGStageA = kGKC * kGTM;                     // bf16 elements of Z per stage
constexpr int kGStage = kGStageA + kGKC * kGTN;           // 24 KB per stage
constexpr int kGUnitsA = kGStageA * 2 / 1024;             // 1 KB copies of Z per stage (16)
constexpr int kGUnits = kGStage * 2 / 1024;               // 1 KB copies per stage (24)
constexpr int kGCopies = kGUnits / 4;                     // copies per wave per stage (6)

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;

__device__ __forceinline__ int gemm_swz(int r) { return ((r & 3) * 2) ^ ((r & 1) << 3); }

// s_waitcnt with vmcnt(N) and lgkmcnt(0), expcnt left open; no memory access
// moves across it
template <int N>
__device__ __forceinline__ void gemm_wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ void gemm_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

typedef short i16x8_t __attribute__((ext_vector_type(8)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// Buffer descriptor of `bytes` bytes at p: no stride, 32-bit data format
// (accesses at or past `bytes` return zeros and touch no memory).
__device__ __forceinline__ i32x4_t gemm_rsrc(const void* p, int bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return i32x4_t{int(uint32_t(a)), int(uint32_t(a >> 32) & 0xffffu), bytes, 0x00020000};
}

// One 1 KB stage copy: lane l's 16 bytes at byte offset voff of the buffer go
// to LDS at dst + 16 l.  Issued as inline assembly so that the compiler does
// not add its own (conservative) waits for LDS copies: every read of a stage
// is preceded by an explicit vmcnt wait and a barrier.  NT marks the data as
// streamed once (the live state), so that it does not displace the operand
// tiles that the XCD's other blocks still read from L2.
template <bool NT = false>
__device__ __forceinline__ void gemm_copy(uint16_t* dst, uint32_t voff, i32x4_t rsrc) {
  const uint32_t lds = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t*)dst));
  // the descriptor and the LDS address are wave-uniform: keep them in SGPRs
  const i32x4_t r = {__builtin_amdgcn_readfirstlane(rsrc[0]), __builtin_amdgcn_readfirstlane(rsrc[1]),
                     __builtin_amdgcn_readfirstlane(rsrc[2]), __builtin_amdgcn_readfirstlane(rsrc[3])};
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(r) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(voff), "s"(r) : "memory", "m0");
#pragma clang diagnostic pop
}

// One MFMA operand: 8 consecutive ranks (two transposing reads, 4 rank rows
// apart) of the row or column that this lane owns; ROW = LDS row length.
template <int ROW>
__device__ __forceinline__ bf16x8_t gemm_operand(const uint16_t* lds, int off) {
  const i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(lds + off));
  const i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(lds + off + 4 * ROW));
  return __builtin_bit_cast(bf16x8_t, i16x8_t(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)));
}

template <typename ST>
__global__ void __launch_bounds__(kGThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
write_gemm_kernel(const WriteParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t s0[kGStage];
  __shared__ __attribute__((aligned(16))) uint16_t s1[kGStage];
  __shared__ __attribute__((aligned(16))) uint16_t s2[kGStage];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const GemmTile tile = gemm_tile(blockIdx.x, p.mt, p.ntl);
  const int b = tile.b, mt = tile.mt, nt = tile.nt;
  if (nt >= p.ntl || mt >= p.mt || b >= p.count) return;
  const int m0 = mt * kGTM;
  const int n0 = nt * kGTN;
  const uint16_t* Z = static_cast<const uint16_t*>(p.z[b]);
  const uint16_t* G = static_cast<const uint16_t*>(p.g[b]);

  // Stage copies: wave w moves the 1 KB units w, w + 4, w + 8, w + 12 of Z
  // (rank rows 2u, 2u + 1) and w, w + 4 of G (rank rows 4u .. 4u + 3).  Lane
  // l's 16 bytes land at unit offset 16 l, i.e. rank row r, slot s, which
  // holds column group s ^ swz(r).  Byte offsets are relative to the stage's
  // first rank row; a group outside the matrix gets an offset past any range.
  uint32_t voff[kGCopies];
#pragma unroll
  for (int t = 0; t < kGCopies; ++t) {
    const bool za = t < kGUnitsA / 4;
    const int u = wave + 4 * (za ? t : t - kGUnitsA / 4);
    const int r = za ? 2 * u + (lane >> 5) : 4 * u + (lane >> 4);
    const int s = za ? (lane & 31) : (lane & 15);
    const int col = (za ? m0 : n0) + 8 * (s ^ gemm_swz(r));
    const int lim = za ? p.d_ff : p.d_model;
    voff[t] = col < lim ? uint32_t(r * lim + col) * 2u : 0x80000000u;
  }
  auto issue = [&](uint16_t* st, int c0) {
    // rank rows past the chunk fall outside the stage's range: zeros
    const int rows = min(kGKC, p.chunk - c0);
    const i32x4_t zr = gemm_rsrc(Z + size_t(c0) * p.d_ff, rows * p.d_ff * 2);
    const i32x4_t gr = gemm_rsrc(G + size_t(c0) * p.d_model, rows * p.d_model * 2);
#pragma unroll
    for (int t = 0; t < kGCopies; ++t) {
      const bool za = t < kGUnitsA / 4;
      const int u = wave + 4 * (za ? t : t - kGUnitsA / 4);
      gemm_copy(st + (za ? 0 : kGStageA) + u * 512, voff[t], za ? zr : gr);
    }
  };

  // operand read offsets (elements, stage-relative) of this lane's fragments
  const int g4 = lane >> 4;
  const int eps = g4 & 1;
  const int hh = g4 >> 1;
  const int jrow = (lane & 15) >> 2;
  const int q = lane & 3;
  const int sw = gemm_swz(jrow);
  int offa[2], offb[4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
    offa[i] = (8 * hh + jrow) * kGTM + 4 * (q & 1) + (((wave * 8 + i * 4 + 2 * eps + (q >> 1)) ^ sw) << 3);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    offb[j] = kGStageA + (8 * hh + jrow) * kGTN + 4 * (q & 1) + (((j * 4 + 2 * eps + (q >> 1)) ^ sw) << 3);

  f32x16_t acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x16_t{};

  const ST* live = static_cast<const ST*>(p.live[b]);
  ST* shadow = static_cast<ST*>(p.shadow[b]);
  const float eta = p.eta;

  // fp32 state only: the register epilogue's first live rows are requested
  // with the first stages and held through the main loop (a lane owns 8
  // columns of rows (lane >> 4) + 4 rr of each 16-row step)
  const int c8 = (lane & 15) * 8;
  const int ncol = n0 + c8;
  const bool ncol_ok = ncol < p.d_model;
  Packed<ST, 8> lv[4];
  auto row_of = [&](int sp, int rr) { return m0 + wave * 64 + (sp >> 1) * 32 + (sp & 1) * 16 + (lane >> 4) + 4 * rr; };
  auto load_live = [&](int sp) {
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int row = row_of(sp, rr);
      if (row < p.d_ff && ncol_ok)
        load_packed<true>(live + size_t(row) * p.d_model + ncol, lv[rr]);
      else
        lv[rr].zero();
    }
  };

  // bf16 state: wave w's 64 live rows are copied into freed stages as two
  // halves of 32 rows x 128 columns (8 KB each), half 0 during the last
  // stage's MFMAs (into the two stages already consumed), half 1 after it
  uint16_t* reg[2] = {s0, s0};
  auto live_copy = [&](uint16_t* dst, int hf) {
    const int row0 = m0 + wave * 64 + hf * 32;
    const int rows = __builtin_amdgcn_readfirstlane(max(0, min(32, p.d_ff - row0)));   // wave-uniform
    const i32x4_t lr = gemm_rsrc(live + size_t(min(row0, p.d_ff)) * p.d_model, rows * p.d_model * 2);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int r = 4 * t + (lane >> 4);
      const int col = n0 + 8 * ((lane & 15) ^ (r & 15));
      const uint32_t off = col < p.d_model ? uint32_t(r * p.d_model + col) * 2u : 0x80000000u;
      gemm_copy<true>(dst + t * 512, off, lr);
    }
  };

  const int nchunks = (p.chunk + kGKC - 1) / kGKC;
  auto step = [&](uint16_t* cur, uint16_t* nxt, uint16_t* oth, int k) {
    // this wave's copies of chunk k are done once at most those of chunk
    // k + 1 are outstanding; the barrier then covers every wave's copies and
    // frees the stage read in step k - 1 for chunk k + 2
    if (k + 1 < nchunks) gemm_wait_vm<kGCopies>();
    else gemm_wait_vm<0>();
    gemm_barrier();
    if (k + 2 < nchunks) issue(nxt, (k + 2) * kGKC);
    if constexpr (sizeof(ST) == 2) {
      if (k + 1 == nchunks) {
        // nxt and oth were read in the two previous steps: 6 free 8 KB slots
        reg[0] = (wave < 2 ? nxt : oth) + (wave & 1) * 4096;
        reg[1] = wave < 3 ? cur + wave * 4096 : nxt + 2 * 4096;
        live_copy(reg[0], 0);
      }
    }
#pragma unroll
    for (int ks = 0; ks < kGKC / 16; ++ks) {
      bf16x8_t af[2], bf[4];
#pragma unroll
      for (int i = 0; i < 2; ++i) af[i] = gemm_operand<kGTM>(cur, offa[i] + ks * 16 * kGTM);
#pragma unroll
      for (int j = 0; j < 4; ++j) bf[j] = gemm_operand<kGTN>(cur, offb[j] + ks * 16 * kGTN);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[j], af[i], acc[i][j], 0, 0, 0);
    }
  };

  issue(s0, 0);
  if (nchunks > 1) issue(s1, kGKC);
  if constexpr (sizeof(ST) == 4) load_live(0);
  for (int k = 0; k < nchunks; k += 3) {
    step(s0, s2, s1, k);
    if (k + 1 < nchunks) step(s1, s0, s2, k + 1);
    if (k + 2 < nchunks) step(s2, s1, s0, k + 2);
  }
  // every wave is done with the stages after this barrier
  __builtin_amdgcn_s_waitcnt(0xC07F);                      // lgkmcnt(0)
  gemm_barrier();

  if constexpr (sizeof(ST) == 2) {
    // bf16 state.  The MFMA is issued as D^T = G^T Z, so accumulator register
    // 4a+e of block (i, j) holds D[i*32 + l%32][j*32 + 8a + 4(l/32) + e]:
    // four consecutive columns of one row, the layout of the state itself.
    // Each lane reads those 8 bytes of live from the copied half (row r's
    // 16-byte groups sit in slot (group ^ (r & 15)), so the 16 rows of a
    // half-wave hit distinct banks), forms live + eta * D and writes the
    // bf16 result back in place; whole rows are then read back and stored.
    // Loads and stores go through buffer descriptors clipped to the matrix,
    // so ragged tiles need no branches and every wave issues a fixed number
    // of memory instructions.
    live_copy(reg[1], 1);
    const int ml = lane & 31;                              // row of the half this lane updates
    const int h4 = (lane >> 5) * 4;                        // column offset within the 8-column group
    // store side: lane l moves 16 bytes (8 columns) of row 4t + l / 16, so
    // consecutive lanes write consecutive addresses
    const int srow = lane >> 4;
    const int scol = n0 + 8 * (lane & 15);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      // half 0's copies are done once at most half 1's 8 copies are
      // outstanding (loads complete in order); half 1's were waited for
      // before any store was issued, since stores and loads may complete
      // out of order relative to each other
      if (hf == 0) gemm_wait_vm<8>();
      typedef __attribute__((address_space(3))) u32x2_t lds_u32x2_t;
      u32x2_t lt[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int a = 0; a < 4; ++a)
          lt[j][a] = *(const lds_u32x2_t*)(reg[hf] + ml * kGTN + (((4 * j + a) ^ (ml & 15)) << 3) + h4);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const f32x16_t& d = acc[hf][j];
          const float f0 = __uint_as_float(lt[j][a][0] << 16) + eta * d[4 * a + 0];
          const float f1 = __uint_as_float(lt[j][a][0] & 0xffff0000u) + eta * d[4 * a + 1];
          const float f2 = __uint_as_float(lt[j][a][1] << 16) + eta * d[4 * a + 2];
          const float f3 = __uint_as_float(lt[j][a][1] & 0xffff0000u) + eta * d[4 * a + 3];
          *(lds_u32x2_t*)(reg[hf] + ml * kGTN + (((4 * j + a) ^ (ml & 15)) << 3) + h4) =
              u32x2_t{bf16x2_rne(f0, f1), bf16x2_rne(f2, f3)};
        }
      asm volatile("" ::: "memory");
      if (hf == 0) gemm_wait_vm<0>();
      const int row0 = m0 + wave * 64 + hf * 32;
      const int rows = __builtin_amdgcn_readfirstlane(max(0, min(32, p.d_ff - row0)));   // wave-uniform
      const __amdgpu_buffer_rsrc_t sr = __builtin_amdgcn_make_buffer_rsrc(
          shadow + size_t(min(row0, p.d_ff)) * p.d_model, (short)0, rows * p.d_model * 2, 0x00020000);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int r = 4 * t + srow;
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(reg[hf] + r * kGTN + (((lane & 15) ^ (r & 15)) << 3));
        const uint32_t off = scol < p.d_model ? uint32_t(r * p.d_model + scol) * 2u : 0x80000000u;
        __builtin_amdgcn_raw_buffer_store_b128(v, sr, off, 0, 2);        // non-temporal
      }
    }
  } else {
    // fp32 state: each wave passes its own accumulators through a private
    // 8 KB LDS region (16 rows x 128 fp32) in 16-row steps, then every lane
    // updates 8 contiguous columns of 4 rows.  Accumulator register 4a+e of
    // block (i, j) holds D[i*32 + l%32][j*32 + 8a + 4(l/32) + e]: the lanes
    // whose row falls in the step write those 16 bytes.  Row r of a region
    // keeps its 16-byte units XOR (r & 15), so the rows of one write hit
    // distinct banks.  LDS requests of one wave complete in order, so the
    // region needs no barrier.
    float* ep = reinterpret_cast<float*>(wave == 1 ? s1 : wave == 2 ? s2 : s0) + (wave == 3 ? 2048 : 0);
    const int hu = lane >> 5;                              // 16-byte unit within the 8-column group
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
      const int i = sp >> 1;
      const int qh = sp & 1;
      if (((lane & 31) >> 4) == qh) {
        const int rl = (lane & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            const int u = 8 * j + 2 * a + hu;
            *reinterpret_cast<f32x4_t*>(ep + rl * kGTN + ((u ^ rl) << 2)) =
                f32x4_t{acc[i][j][4 * a], acc[i][j][4 * a + 1], acc[i][j][4 * a + 2], acc[i][j][4 * a + 3]};
          }
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int rl = (lane >> 4) + 4 * rr;
        const int u0 = 2 * (lane & 15);
        const f32x4_t a0 = *reinterpret_cast<const f32x4_t*>(ep + rl * kGTN + ((u0 ^ (rl & 15)) << 2));
        const f32x4_t a1 = *reinterpret_cast<const f32x4_t*>(ep + rl * kGTN + (((u0 + 1) ^ (rl & 15)) << 2));
        const float o[8] = {lv[rr].get(0) + eta * a0[0], lv[rr].get(1) + eta * a0[1],
                            lv[rr].get(2) + eta * a0[2], lv[rr].get(3) + eta * a0[3],
                            lv[rr].get(4) + eta * a1[0], lv[rr].get(5) + eta * a1[1],
                            lv[rr].get(6) + eta * a1[2], lv[rr].get(7) + eta * a1[3]};
        const int row = row_of(sp, rr);
        if (row < p.d_ff && ncol_ok) store_n<8, true>(shadow + size_t(row) * p.d_model + ncol, o);
        // this register slot now takes the same row of the next step
        if (sp + 1 < 4) {
          const int nrow = row_of(sp + 1, rr);
          if (nrow < p.d_ff && ncol_ok)
            load_packed<true>(live + size_t(nrow) * p.d_model + ncol, lv[rr]);
          else
            lv[rr].zero();
        }
      }
      asm volatile("" ::: "memory");
    }
  }
}

// ---------------------------------------------------------------------------
// WRITE, fp32 evidence: fp32 matrix instructions (bf16 operands would round Z
// and G)
// ---------------------------------------------------------------------------
//
// The update moves 2 |dW| bytes for 2C fp32 flop per element, so up to about
// C = 100 it is bound by HBM and above by the fp32 matrix rate.  One block of
// eight waves per (group slot, 256 / WN rows, 64 WN columns); a wave owns 32
// rows and 64 columns.  v_mfma_f32_16x16x4_f32 takes its operands as they lie
// in memory: lane (i, q) holds evidence row 4 s + q at state rows 2 i, 2 i + 1
// (8 bytes of Z) and at columns 4 i .. 4 i + 3 (16 bytes of G), which are the
// rows and columns i of 2 x 4 matrices; an accumulator register then belongs to
// one state row, and a lane's four matrices to four consecutive columns of it.
// So nothing goes through LDS, each lane updates 8 whole rows of 16 bytes, and
// the live rows (and for the token W0's) are requested before the evidence.
//
// WN waves side by side make runs of 256 WN bytes per state row: WN = 4, 2 and
// 1 take 126, 132 and 152 us for 8 owners of 12856 x 600, C = 17, and 66, 68 and
// 71 us for two of 9728 x 2560, C = 4 (6.0 TB/s).  The token (x live + x W0, at
// version v) is accumulated from the same live registers into one partial per
// (owner, rows of a block), which read_reduce_kernel adds; the workspace has 64
// such rows per owner, or one per READ chunk of 256 rows, so with a token WN is
// 4 up to 4096 rows, 2 up to 8192 and 1 above.
//
// 4104 x 1032, C = 40, two owners with token (86 MB): 85 us before (a separate
// READ, then one thread per four columns with a load for every fourth
// product), 29 us now (32 when the state comes from HBM); without the token 21 us
// (68 MB).

constexpr int kFThreads = 512;           // 8 waves of 32 rows x 64 columns
static_assert(kFThreads / 64 * 32 == kReadChunk, "WN = 1: one READ chunk per block");

template <typename ST, bool TOKEN, int WN, bool NT>
__global__ void __launch_bounds__(kFThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
write_f32_kernel(const WriteParams p) {
  constexpr int QB = 4;                  // matrix steps (of four evidence rows) per group of loads
  constexpr int WM = 8 / WN;             // waves one above the other
  __shared__ float ysum[WM][64 * WN];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, q4 = lane >> 4;
  // block -> (XCD, position) -> ((rows, columns) pair, slot): the slots of one
  // pair sit on one XCD, so that W0 comes from HBM once
  const int xcd = blockIdx.x & 7;
  const int pos = blockIdx.x >> 3;
  const int pl = pos / p.count;
  const int b = pos - pl * p.count;
  const int pair = pl * 8 + xcd;
  if (pair >= p.mt * p.ntl) return;
  const int mt = pair / p.ntl;
  const int nb = (pair - mt * p.ntl) * 64 * WN;
  const int n0 = nb + (wave % WN) * 64;
  const int mw = (mt * WM + wave / WN) * 32;             // the wave's first row
  const int n = min(n0 + 4 * i16, p.d_model - 4);        // this lane's four columns
  const int m = min(mw + 8 * q4, p.d_ff - 8);            // ... and eight rows, all inside or all outside
  const bool ok = n0 + 4 * i16 < p.d_model && mw + 8 * q4 < p.d_ff;
  const float* Z = static_cast<const float*>(p.z[b]);
  const float* G = static_cast<const float*>(p.g[b]);

  // row r of the eight is register r / 2 of matrix r % 2
  const size_t at = size_t(m) * p.d_model + n;
  const ST* live = static_cast<const ST*>(p.live[b]) + at;
  Packed<ST, 4> lv[8];
  Packed<float, 4> wv[TOKEN ? 8 : 1], xv[TOKEN ? 2 : 1];
#pragma unroll
  for (int r = 0; r < 8; ++r) load_packed<NT>(live + size_t(r) * p.d_model, lv[r]);
  if constexpr (TOKEN) {
    const float* W0 = static_cast<const float*>(p.w0) + at;
    const float* X = static_cast<const float*>(p.x) + size_t(p.row[b]) * p.d_ff + m;
    load_packed<false>(X, xv[0]);
    load_packed<false>(X + 4, xv[1]);
#pragma unroll
    for (int r = 0; r < 8; ++r) load_packed<false>(W0 + size_t(r) * p.d_model, wv[r]);
  }

  // rows 2 i16, 2 i16 + 1 of the wave as the matrices' rows: past the matrix
  // they are copies of real rows whose results are not stored
  const uint32_t zoff = uint32_t(min(mw + 2 * i16, p.d_ff - 2)) * 4u, goff = uint32_t(n) * 4u;
  f32x4_t acc[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[t][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nq = (p.chunk + 3) / 4;
  for (int s0 = 0; s0 < nq; s0 += QB) {
    Packed<float, 2> z[QB];
    Packed<float, 4> g[QB];
    const char* Zs = reinterpret_cast<const char*>(Z + size_t(4 * s0) * p.d_ff);
    const char* Gs = reinterpret_cast<const char*>(G + size_t(4 * s0) * p.d_model);
#pragma unroll
    for (int s = 0; s < QB; ++s) {
      const uint32_t c = uint32_t(min(4 * s + q4, p.chunk - 1 - 4 * s0));
      load_packed<false>(reinterpret_cast<const float*>(Zs + (c * uint32_t(p.d_ff) * 4u + zoff)), z[s]);
      load_packed<false>(reinterpret_cast<const float*>(Gs + (c * uint32_t(p.d_model) * 4u + goff)), g[s]);
    }
#pragma unroll
    for (int s = 0; s < QB; ++s) {
      if (s0 + s >= nq) break;
      const bool in = 4 * (s0 + s) + q4 < p.chunk;       // rows past the chunk: both operands zero
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? z[s].get(t) : 0.f, in ? g[s].get(u) : 0.f,
                                                           acc[t][u], 0, 0, 0);
    }
  }

  ST* shadow = static_cast<ST*>(p.shadow[b]) + at;
  float y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    float o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = lv[r].get(u) + p.eta * acc[r & 1][u][r >> 1];
    if (ok) store_n<4, true>(shadow + size_t(r) * p.d_model, o);
    if constexpr (TOKEN) {
      const float x = xv[r >> 2].get(r & 3);
#pragma unroll
      for (int u = 0; u < 4; ++u) y[u] = fmaf(x, wv[r].get(u), fmaf(x, lv[r].get(u), y[u]));
    }
  }
  if constexpr (TOKEN) {
    // the four quarters' rows, then the waves one above the other, as trees
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v = ok ? y[u] : 0.f;
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (q4 == 0) ysum[wave / WN][(wave % WN) * 64 + 4 * i16 + u] = v;
    }
    __syncthreads();
    if (tid < 64 * WN && nb + tid < p.d_model) {
      float v[WM];
#pragma unroll
      for (int w = 0; w < WM; ++w) v[w] = ysum[w][tid];
#pragma unroll
      for (int k = 1; k < WM; k *= 2)
#pragma unroll
        for (int w = 0; w + k < WM; w += 2 * k) v[w] += v[w + k];
      p.tpart[(size_t(p.row[b]) * p.parts + mt) * p.npadw + nb + tid] = v[0];
    }
  }
}

// ---------------------------------------------------------------------------
// WRITE, bf16 evidence, fp32 state, C <= 384, token apart: register operands
// ---------------------------------------------------------------------------
//
// The fp32 state moves 8 bytes per element for 2C flop, so it is bound by HBM
// over this whole range; what is wanted is a copy that multiplies on the side.
// As in write_f32_kernel nothing goes through LDS and a lane updates whole
// rows: a wave owns 64 rows x 64 columns, a lane (i, q) loads four consecutive
// evidence rows 4 q .. 4 q + 3 of a group of 16 at state rows 4 i .. 4 i + 3 (8
// bytes of Z each) and at columns 4 i .. 4 i + 3 (of G), and byte permutes turn
// these 4 x 4 blocks into the operands (four consecutive ranks of one row or
// column) of 4 x 4 matrices of v_mfma_f32_16x16x16_bf16.  The waves are
// independent; four neighbours of a row of tiles make a block (waves one by
// one: 112 against 104 us below), three blocks fit a CU.
//
// Three owners of 9728 x 2560 (602 MB + evidence), in us, against the streaming
// kernel (C <= 64) and the GEMM that took these calls before: 104 / 117 at C =
// 64, 114 / 155 at 128, 137 / 165 at 256, 168 / 177 at 384.  The evidence loads
// bind then (200 / 188 at 512), so longer chunks stay with the GEMM, and from C =
// 300 on those of calls whose tiles fill its rounds.  One
// owner of 2496 x 824, C = 159: 8.7 / 15.4.  Half as many state rows per wave
// needs nearly twice the loads per product (108, 125, 167 at 64, 128, 256).
// With bf16 state, half the bytes, the GEMM is as fast at C = 16 (78 / 80 us
// for two owners of 14336 x 4096) and faster above (94 / 82 at C = 64).

constexpr int kRThreads = 256;           // 4 waves, neighbours in a row of tiles
constexpr int kRTN = 64;                 // columns per wave

// The product of a wave's 64 rows and 64 columns over the whole chunk: zoff and
// goff are the lane's byte offsets in a row of Z and of G.
__device__ __forceinline__ void rows_product(const WriteParams& p, const uint16_t* Z, const uint16_t* G,
                                             uint32_t zoff, uint32_t goff, int q4, f32x4_t (&acc)[4][4]) {
  constexpr int RS = 16;                 // evidence rows per matrix step
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[t][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < p.chunk; c0 += RS) {
    Packed<uint16_t, 4> z[4], g[4];
    const char* Zs = reinterpret_cast<const char*>(Z + size_t(c0) * p.d_ff);
    const char* Gs = reinterpret_cast<const char*>(G + size_t(c0) * p.d_model);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t c = uint32_t(min(4 * q4 + i, p.chunk - 1 - c0)) * 2u;
      load_packed<false>(reinterpret_cast<const uint16_t*>(Zs + (c * uint32_t(p.d_ff) + zoff)), z[i]);
      load_packed<false>(reinterpret_cast<const uint16_t*>(Gs + (c * uint32_t(p.d_model) + goff)), g[i]);
    }
    if (c0 + RS > p.chunk) {
      // rows past the chunk: both operands zero
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (c0 + 4 * q4 + i >= p.chunk) {
          z[i].zero();
          g[i].zero();
        }
    }
    // value j of four evidence rows in one operand
    auto pick = [](const Packed<uint16_t, 4> (&v)[4], int j) {
      const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
      const int w = j >> 1;
      return __builtin_bit_cast(i16x4_t, u32x2_t{__builtin_amdgcn_perm(v[1].w[w], v[0].w[w], sel),
                                                 __builtin_amdgcn_perm(v[3].w[w], v[2].w[w], sel)});
    };
    i16x4_t az[4], bg[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) az[t] = pick(z, t);
#pragma unroll
    for (int u = 0; u < 4; ++u) bg[u] = pick(g, u);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(az[t], bg[u], acc[t][u], 0, 0, 0);
  }
}

template <bool NT>
__global__ void __launch_bounds__(kRThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
write_rows_kernel(const WriteParams p) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int i16 = lane & 15, q4 = lane >> 4;
  const int b = blockIdx.y;
  // blocks are dealt to the XCDs round-robin: each round of eight is rotated by
  // one, or a power of two of columns would give an XCD always the same ones
  // (30.4 against 24.2 us for two owners of 8192 x 1024)
  const int bx = (int(blockIdx.x) & ~7) | ((int(blockIdx.x) + (int(blockIdx.x) >> 3)) & 7);
  const int tile = bx * (kRThreads / 64) + wave;         // the waves are independent
  const int mt = tile / p.ntl;
  if (mt >= p.mt) return;
  const int m0 = mt * kRTM + 16 * q4;                    // this lane's 16 rows: two runs of eight, each
                                                         // inside or outside the matrix as a whole
  const int n0 = (tile - mt * p.ntl) * kRTN + 4 * i16;
  const bool n_ok = n0 < p.d_model;
  const int n = min(n0, p.d_model - 4);                  // ... and four columns
  const uint16_t* Z = static_cast<const uint16_t*>(p.z[b]);
  const uint16_t* G = static_cast<const uint16_t*>(p.g[b]);

  // the live rows are requested first: row r is register r / 4 of matrix r % 4
  Packed<float, 4> lv[16];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float* live = static_cast<const float*>(p.live[b]) + size_t(min(m0 + 8 * h, p.d_ff - 8)) * p.d_model + n;
#pragma unroll
    for (int r = 0; r < 8; ++r) load_packed<NT>(live + size_t(r) * p.d_model, lv[8 * h + r]);
  }

  const uint32_t zoff = uint32_t(min(mt * kRTM + 4 * i16, p.d_ff - 4)) * 2u, goff = uint32_t(n) * 2u;
  f32x4_t acc[4][4];
  rows_product(p, Z, G, zoff, goff, q4, acc);

#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = lv[r].get(u) + p.eta * acc[r & 3][u][r >> 2];
    if (n_ok && m0 + (r & 8) < p.d_ff)
      store_n<4, true>(static_cast<float*>(p.shadow[b]) + size_t(m0 + r) * p.d_model + n, o);
  }
}

// With a fused token (C <= 64) the waves also load W0's rows, and two blocks fit
// a CU.  A block is four waves side by side and leaves one token partial per
// (owner, 64 rows) in the region of the streaming kernel, whose 64 rows per owner
// end at 4096 matrix rows.
template <bool NT>
__global__ void __launch_bounds__(kRThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
write_rows_token_kernel(const WriteParams p) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int i16 = lane & 15, q4 = lane >> 4;
  // block -> (XCD, position) -> ((rows, columns) pair, slot): the slots of one
  // pair sit on one XCD, so that W0 comes from HBM once.  Rounds of eight are
  // rotated as above
  const int xcd = blockIdx.x & 7;
  const int pos = blockIdx.x >> 3;
  const int pl = pos / p.count;
  const int b = pos - pl * p.count;
  const int pair = pl * 8 + ((xcd + pl) & 7);
  if (pair >= p.mt * p.ntl) return;
  const int mt = pair / p.ntl;
  const int mw = mt * kRTM;                              // the block's first row
  const int n0 = ((pair - mt * p.ntl) * (kRThreads / 64) + wave) * kRTN + 4 * i16;
  const int m0 = mw + 16 * q4;                           // this lane's 16 rows
  const bool n_ok = n0 < p.d_model;
  const int n = min(n0, p.d_model - 4);                  // ... and four columns
  const uint16_t* X = static_cast<const uint16_t*>(p.x) + size_t(p.row[b]) * p.d_ff;
  Packed<float, 4> lv[16];
  Packed<uint16_t, 4> wv[16];
  Packed<uint16_t, 8> xv[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int m = min(m0 + 8 * h, p.d_ff - 8);
    const size_t at = size_t(m) * p.d_model + n;
    load_packed<false>(X + m, xv[h]);
#pragma unroll
    for (int r = 0; r < 8; ++r)
      load_packed<NT>(static_cast<const float*>(p.live[b]) + at + size_t(r) * p.d_model, lv[8 * h + r]);
#pragma unroll
    for (int r = 0; r < 8; ++r)
      load_packed<false>(static_cast<const uint16_t*>(p.w0) + at + size_t(r) * p.d_model, wv[8 * h + r]);
  }
  float y[4] = {0.f, 0.f, 0.f, 0.f};
  f32x4_t acc[4][4];
  rows_product(p, static_cast<const uint16_t*>(p.z[b]), static_cast<const uint16_t*>(p.g[b]),
               uint32_t(min(mw + 4 * i16, p.d_ff - 4)) * 2u, uint32_t(n) * 2u, q4, acc);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = lv[r].get(u) + p.eta * acc[r & 3][u][r >> 2];
    if (n_ok && m0 + (r & 8) < p.d_ff)
      store_n<4, true>(static_cast<float*>(p.shadow[b]) + size_t(m0 + r) * p.d_model + n, o);
  }
  // token: x live + x W0 over this lane's rows, in row order
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float x = xv[r >> 3].get(r & 7);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float t = fmaf(x, wv[r].get(u), fmaf(x, lv[r].get(u), y[u]));
      y[u] = m0 + (r & 8) < p.d_ff ? t : y[u];           // rows past the matrix are copies
    }
  }
  // the four quarters' rows as a tree
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    y[u] += __shfl_xor(y[u], 16);
    y[u] += __shfl_xor(y[u], 32);
  }
  if (q4 == 0 && n_ok) store_n<4>(p.tpart + (size_t(p.row[b]) * p.parts + mt) * p.npadw + n0, y);
}

// ---------------------------------------------------------------------------
// TailBufferUpdate for a WRITE step: its own x row becomes the chunk's last
// ---------------------------------------------------------------------------

struct TailParams {
  int n16;                         // 16-byte units per row
  const uint4* x;                  // owner-indexed rows of n16 units
  uint4* dst[RWTTT_MAX_GROUP];
  uint32_t row[RWTTT_MAX_GROUP];
};

__global__ void __launch_bounds__(256) tail_append_kernel(const TailParams p) {
  const int b = blockIdx.y;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < p.n16) p.dst[b][i] = p.x[size_t(p.row[b]) * p.n16 + i];
}

// ---------------------------------------------------------------------------
// Fork: bulk copy of slots and tails (streaming, non-temporal both ways)
// ---------------------------------------------------------------------------

constexpr int kCopyJobs = 64;

struct CopyParams {
  const u32x4_t* src[kCopyJobs];
  u32x4_t* dst[kCopyJobs];
  size_t n16[kCopyJobs];
};

__global__ void __launch_bounds__(256) copy_kernel(const CopyParams p) {
  const int j = blockIdx.y;
  const size_t n = p.n16[j];
  const u32x4_t* s = p.src[j];
  u32x4_t* d = p.dst[j];
  const size_t stride = size_t(gridDim.x) * 256 * 4;
  for (size_t i = size_t(blockIdx.x) * 256 * 4 + threadIdx.x; i < n; i += stride) {
    u32x4_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + size_t(u) * 256 < n) v[u] = __builtin_nontemporal_load(s + i + size_t(u) * 256);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + size_t(u) * 256 < n) __builtin_nontemporal_store(v[u], d + i + size_t(u) * 256);
  }
}

template <typename IO> void launch_reduce(const ReadParams& p, bool tree, hipStream_t stream) {
  const dim3 grid((p.d_model + kRedCols - 1) / kRedCols, p.count);
  if (tree) hipLaunchKernelGGL((read_reduce_kernel<IO, true>), grid, dim3(256), 0, stream, p);
  else hipLaunchKernelGGL((read_reduce_kernel<IO, false>), grid, dim3(256), 0, stream, p);
}

template <typename IO, typename ST>
hipError_t launch_read_t(const ReadLaunch& L, hipStream_t stream, float* slot_part = nullptr) {
  const ReadGeometry g = read_geometry(L.d_ff, L.d_model, L.state_bf16, L.n_owners);
  ReadParams p;
  p.x = L.x;
  p.y = L.y;
  p.w0 = L.w0;
  p.part = slot_part ? slot_part : static_cast<float*>(L.workspace);
  p.slot_part = slot_part ? 1 : 0;
  p.count = L.count;
  p.d_ff = L.d_ff;
  p.d_model = L.d_model;
  p.ks = g.ks;
  p.nt = g.nt;
  p.npad = g.npad;
  for (int b = 0; b < RWTTT_MAX_GROUP; ++b) {
    p.dw[b] = b < L.count ? L.dw[b] : nullptr;
    p.row[b] = b < L.count ? L.row[b] : 0u;
    p.tail[b] = b < L.count ? L.tail[b] : nullptr;
  }
  const ReadRoute route = read_route(sizeof(IO) == 2, sizeof(ST) == 2, L.d_ff, L.d_model, L.count, L.context_bytes);
  if (route.direct) {
    constexpr int tile = kDirectLanes * read_cols_per_lane(sizeof(ST) == 2);
    p.nt = (L.d_model + tile - 1) / tile;
    const dim3 grid(unsigned((p.nt + 7) / 8 * 8 * L.count));
    if (L.d_ff <= kDirectGroups * kDirectLeaf)
      hipLaunchKernelGGL((read_direct_kernel<IO, ST, 1>), grid, dim3(kDirectThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((read_direct_kernel<IO, ST, 2>), grid, dim3(kDirectThreads), 0, stream, p);
    return hipGetLastError();
  }
  // (chunk, tile) pairs rounded up to a multiple of the 8 XCDs
  const dim3 grid(unsigned((g.ks * g.nt + 7) / 8 * 8) * unsigned(L.count));
  auto run = [&](auto nt) {
    constexpr bool NT = decltype(nt)::value;
    if (route.leaf == kDirectLeaf) {
      // so large a call always has the hint
      static_assert(size_t(256) * kReadChunk * read_tile_n(1) * sizeof(ST) > kCacheCall, "");
      if constexpr (sizeof(IO) > sizeof(ST) && NT) {
        if (route.waves == 4) {
          hipLaunchKernelGGL((read_partial_kernel<IO, ST, 4, kDirectLeaf, NT>), grid, dim3(256), 0, stream, p);
          return;
        }
      }
      hipLaunchKernelGGL((read_partial_kernel<IO, ST, 8, kDirectLeaf, NT>), grid, dim3(512), 0, stream, p);
    } else if constexpr (sizeof(IO) <= sizeof(ST)) {
      if (route.waves == 4)
        hipLaunchKernelGGL((read_partial_kernel<IO, ST, 4, 32, NT>), grid, dim3(256), 0, stream, p);
      else
        hipLaunchKernelGGL((read_partial_kernel<IO, ST, 8, 32, NT>), grid, dim3(512), 0, stream, p);
    }
  };
  if (route.nt) run(std::true_type{});
  else run(std::false_type{});
  launch_reduce<IO>(p, L.d_ff <= kDirectRows, stream);
  return hipGetLastError();
}

template <typename ST>
hipError_t launch_write_t(const WriteLaunch& L, hipStream_t stream) {
  WriteParams p;
  p.count = L.count;
  p.chunk = L.chunk;
  p.d_ff = L.d_ff;
  p.d_model = L.d_model;
  p.eta = L.eta;
  p.parts = 0;
  p.npadw = 0;
  p.x = L.x;
  p.w0 = L.w0;
  p.tpart = nullptr;
  for (int b = 0; b < RWTTT_MAX_GROUP; ++b) {
    const bool in = b < L.count;
    p.live[b] = in ? L.live[b] : nullptr;
    p.shadow[b] = in ? L.shadow[b] : nullptr;
    p.z[b] = in ? L.z[b] : nullptr;
    p.g[b] = in ? L.g[b] : nullptr;
    p.row[b] = in ? L.row[b] : 0u;
  }
  const bool token = L.x != nullptr;
  const WriteRoute route = write_route(L.io_bf16, sizeof(ST) == 2, L.d_ff, L.d_model, L.count, L.chunk, token,
                                       L.context_bytes);
  const ReadGeometry geo = read_geometry(L.d_ff, L.d_model, L.state_bf16, L.n_owners);
  // the fused token's partials, p.parts rows of p.npadw per owner
  auto reduce_token = [&] {
    ReadParams q;
    q.x = nullptr;
    q.y = L.y;
    q.w0 = nullptr;
    q.part = p.tpart;
    q.slot_part = 0;
    q.count = L.count;
    q.d_ff = L.d_ff;
    q.d_model = L.d_model;
    q.ks = p.parts;
    q.nt = p.ntl;
    q.npad = p.npadw;
    for (int b = 0; b < RWTTT_MAX_GROUP; ++b) {
      q.dw[b] = nullptr;
      q.row[b] = b < L.count ? L.row[b] : 0u;
      q.tail[b] = nullptr;
    }
    if (L.io_bf16) launch_reduce<uint16_t>(q, false, stream);
    else launch_reduce<float>(q, false, stream);
  };
  if (route.kernel == WriteKernel::f32) {
    auto run = [&](auto wn, auto nt) {
      constexpr int WN = decltype(wn)::value;
      constexpr bool NT = decltype(nt)::value;
      p.mt = p.parts = (L.d_ff * WN + kReadChunk - 1) / kReadChunk;
      p.ntl = (L.d_model + 64 * WN - 1) / (64 * WN);
      p.npadw = WN == 1 ? geo.npad : geo.tnpad;
      const size_t at = WN == 1 ? 0 : geo.token_offset;
      p.tpart = token ? reinterpret_cast<float*>(static_cast<char*>(L.workspace) + at) : nullptr;
      const dim3 grid(unsigned((p.mt * p.ntl + 7) / 8 * 8) * unsigned(L.count));
      if (token) {
        hipLaunchKernelGGL((write_f32_kernel<ST, true, WN, NT>), grid, dim3(kFThreads), 0, stream, p);
        reduce_token();
      } else {
        hipLaunchKernelGGL((write_f32_kernel<ST, false, WN, NT>), grid, dim3(kFThreads), 0, stream, p);
      }
    };
    auto by_rows = [&](auto nt) {
      if (route.wn == 4) run(std::integral_constant<int, 4>{}, nt);
      else if (route.wn == 2) run(std::integral_constant<int, 2>{}, nt);
      else run(std::integral_constant<int, 1>{}, nt);
    };
    if (route.nt) by_rows(std::true_type{});
    else by_rows(std::false_type{});
    return hipGetLastError();
  }
  if (route.kernel == WriteKernel::rows_token) {
    constexpr int tile = kRThreads / 64 * kRTN;
    p.mt = p.parts = (L.d_ff + kRTM - 1) / kRTM;
    p.ntl = (L.d_model + tile - 1) / tile;
    p.npadw = geo.tnpad;
    p.tpart = reinterpret_cast<float*>(static_cast<char*>(L.workspace) + geo.token_offset);
    const dim3 grid(unsigned((p.mt * p.ntl + 7) / 8 * 8) * unsigned(L.count));
    if (route.nt)
      hipLaunchKernelGGL((write_rows_token_kernel<true>), grid, dim3(kRThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((write_rows_token_kernel<false>), grid, dim3(kRThreads), 0, stream, p);
    reduce_token();
    return hipGetLastError();
  }
  if (route.kernel == WriteKernel::stream) {
    p.mt = (L.d_ff + kSTM - 1) / kSTM;
    p.ntl = (L.d_model + kSTN - 1) / kSTN;
    // partitions of an owner's row tiles: fixed by the shape, never by the group
    p.parts = std::min(stream_parts(L.d_ff, L.d_model), geo.tparts);
    p.npadw = geo.tnpad;
    const dim3 grid(unsigned((p.ntl * p.parts + 7) / 8 * 8) * unsigned(L.count));
    auto run = [&](auto nt) {
      constexpr bool NT = decltype(nt)::value;
      if (token) {
        p.tpart = reinterpret_cast<float*>(static_cast<char*>(L.workspace) + geo.token_offset);
        hipLaunchKernelGGL((write_stream_kernel<ST, true, NT>), grid, dim3(256), 0, stream, p);
        reduce_token();
      } else if constexpr (sizeof(ST) == 2 && NT) {
        hipLaunchKernelGGL((write_stream_kernel<ST, false, NT>), grid, dim3(256), 0, stream, p);
      }
    };
    if (route.nt) run(std::true_type{});
    else run(std::false_type{});
    return hipGetLastError();
  }
  if (route.read_first) {
    // no fused kernel on this path: the token is an ordinary READ of the group at version v
    ReadLaunch R;
    R.io_bf16 = L.io_bf16;
    R.context_bytes = L.context_bytes;
    R.state_bf16 = L.state_bf16;
    R.d_ff = L.d_ff;
    R.d_model = L.d_model;
    R.count = L.count;
    R.n_owners = L.n_owners;
    R.x = L.x;
    R.y = L.y;
    R.w0 = L.w0;
    R.workspace = L.workspace;
    for (int b = 0; b < L.count; ++b) {
      R.dw[b] = L.live[b];
      R.row[b] = L.row[b];
      R.tail[b] = nullptr;
    }
    const hipError_t e = launch_read_t<uint16_t, ST>(R, stream);
    if (e != hipSuccess) return e;
  }
  if (route.kernel == WriteKernel::rows) {
    p.mt = (L.d_ff + kRTM - 1) / kRTM;
    p.ntl = (L.d_model + kRTN - 1) / kRTN;
    constexpr int waves = kRThreads / 64;
    const dim3 grid(unsigned((p.mt * p.ntl + waves - 1) / waves + 7) / 8 * 8, unsigned(L.count));
    if (route.nt)
      hipLaunchKernelGGL((write_rows_kernel<true>), grid, dim3(kRThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((write_rows_kernel<false>), grid, dim3(kRThreads), 0, stream, p);
    return hipGetLastError();
  }
  p.mt = (L.d_ff + kGTM - 1) / kGTM;
  p.ntl = (L.d_model + kGTN - 1) / kGTN;
  const dim3 grid(gemm_blocks(L.count, p.mt, p.ntl));
  hipLaunchKernelGGL((write_gemm_kernel<ST>), grid, dim3(kGThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

ReadGeometry read_geometry(int d_ff, int d_model, int state_bf16, int n_owners) {
  ReadGeometry g;
  const int tile = read_tile_n(state_bf16);
  g.ks = (d_ff + kReadChunk - 1) / kReadChunk;
  g.nt = (d_model + tile - 1) / tile;
  g.npad = g.nt * tile;
  g.part_floats = size_t(n_owners) * g.ks * g.npad;
  // the fused WRITE token's partials follow, also one region per owner
  g.tparts = kSParts;
  g.tnpad = (d_model + kSTN - 1) / kSTN * kSTN;
  g.token_offset = (g.part_floats * sizeof(float) + 255) / 256 * 256;
  g.token_floats = size_t(n_owners) * g.tparts * g.tnpad;
  g.total_bytes = g.token_offset + (g.token_floats * sizeof(float) + 255) / 256 * 256;
  return g;
}

hipError_t launch_read(const ReadLaunch& L, hipStream_t stream) {
  if (L.io_bf16) {
    return L.state_bf16 ? launch_read_t<uint16_t, uint16_t>(L, stream)
                        : launch_read_t<uint16_t, float>(L, stream);
  }
  return L.state_bf16 ? launch_read_t<float, uint16_t>(L, stream)
                      : launch_read_t<float, float>(L, stream);
}

// ---------------------------------------------------------------------------
// READ for callers that cannot allocate device memory
// ---------------------------------------------------------------------------
//
// The split-K partial sums go to a static device array instead of the
// context's workspace, one region per group slot.  Every GPU the library runs
// on holds its own copy of the array until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in): its
// device address is looked up once per device, with that device current, and
// kept.  Every block writes its whole partial tile before the reduce reads it,
// so the array needs no clearing between calls; calls that overlap on one GPU
// share it and race.

static __device__ __align__(256) float scratch[RWTTT_NOALLOC_SCRATCH_BYTES / sizeof(float)];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};   // the array's device address, per device

// The device address of `scratch` on the current device, looked up on the
// first call with that device current.
static hipError_t scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

size_t read_noalloc_bytes(int d_ff, int d_model, int state_bf16, int count) {
  const ReadGeometry g = read_geometry(d_ff, d_model, state_bf16, count);
  return g.part_floats * sizeof(float);
}

hipError_t launch_read_noalloc(const ReadLaunch& L, hipStream_t stream) {
  if (read_noalloc_bytes(L.d_ff, L.d_model, L.state_bf16, L.count) > RWTTT_NOALLOC_SCRATCH_BYTES)
    return hipErrorInvalidValue;
  void* ptr = nullptr;
  const hipError_t e = scratch_address(&ptr);
  if (e != hipSuccess) return e;
  float* part = static_cast<float*>(ptr);
  if (L.io_bf16) {
    return L.state_bf16 ? launch_read_t<uint16_t, uint16_t>(L, stream, part)
                        : launch_read_t<uint16_t, float>(L, stream, part);
  }
  return L.state_bf16 ? launch_read_t<float, uint16_t>(L, stream, part)
                      : launch_read_t<float, float>(L, stream, part);
}

hipError_t launch_tail_append(const TailLaunch& L, hipStream_t stream) {
  TailParams p;
  p.n16 = L.d_ff * (L.io_bf16 ? 2 : 4) / 16;
  p.x = static_cast<const uint4*>(L.x);
  for (int b = 0; b < RWTTT_MAX_GROUP; ++b) {
    p.dst[b] = b < L.count ? static_cast<uint4*>(L.dst[b]) : nullptr;
    p.row[b] = b < L.count ? L.row[b] : 0u;
  }
  hipLaunchKernelGGL(tail_append_kernel, dim3((p.n16 + 255) / 256, L.count), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_copy(const CopyJob* jobs, int n, hipStream_t stream) {
  for (int first = 0; first < n; first += kCopyJobs) {
    const int m = std::min(kCopyJobs, n - first);
    CopyParams p;
    size_t most = 0;
    for (int j = 0; j < kCopyJobs; ++j) {
      const bool in = j < m;
      p.src[j] = in ? static_cast<const u32x4_t*>(jobs[first + j].src) : nullptr;
      p.dst[j] = in ? static_cast<u32x4_t*>(jobs[first + j].dst) : nullptr;
      p.n16[j] = in ? jobs[first + j].bytes / 16 : 0;
      most = std::max(most, p.n16[j]);
    }
    if (most == 0) continue;
    const size_t blocks = std::min<size_t>((most + 1023) / 1024, 2048);
    hipLaunchKernelGGL(copy_kernel, dim3(unsigned(blocks), unsigned(m)), dim3(256), 0, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_write(const WriteLaunch& L, hipStream_t stream) {
  return L.state_bf16 ? launch_write_t<uint16_t>(L, stream) : launch_write_t<float>(L, stream);
}

}  // namespace rwttt
