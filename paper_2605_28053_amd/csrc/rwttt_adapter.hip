// gfx950 kernels of the DeltaAdapterState backend (Section 4.4, backend
// instantiations; Appendix D, the LoRA-style adapter path): each owner's
// request state is a rank-r pair A [d_ff, r], B [r, d_model].
//
// READ  y_r = x_r W0 + (x_r A_r) B_r
// WRITE A' = A + eta Z^T (G B^T),  B' = B + eta (Z A)^T G   (both from the live A, B)
//
// The shared W0 term dominates the READ's bytes; the rank-r terms are tiny.
// Every summation order depends only on the shapes, so an owner's results
// are bit-identical whatever group it is batched in.

#include <algorithm>
#include <type_traits>

#include "rwttt_kernels.h"

namespace rwttt {
namespace {

#include "rwttt_device.h"

constexpr int kAThreads = 512;    // READ partial blocks: 8 waves, two per SIMD
constexpr int kAWaves = kAThreads / 64;
constexpr int kAChunk = 192;      // K rows per READ work item
constexpr int kARows = kAChunk / kAWaves;   // W0 rows per wave, all requested at once
constexpr int kAGroup = 8;        // owners per READ block: W0 is read once for all of them
constexpr int kAURows = kAChunk / 64;   // chunk rows per lane in the u share
constexpr int kARedCols = 64;     // READ reduce: columns per block (four waves split the chunks)
constexpr int kARedLoads = 16;    // READ reduce: partials in flight per lane

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(uint16_t v) { return __uint_as_float(uint32_t(v) << 16); }

// x.lo * w.lo + x.hi * w.hi + acc over packed bf16 pairs (v_dot2c_f32_bf16)
__device__ __forceinline__ float dot2_bf16(uint32_t x, uint32_t w, float acc) {
  typedef __bf16 bf16x2_v __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_v, x), __builtin_bit_cast(bf16x2_v, w),
                                         acc, false);
}

// An empty asm that reads and rewrites four or eight accumulators: the
// arithmetic that produced them cannot move past it.
__device__ __forceinline__ void pin_row(float (&a)[4]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
}
__device__ __forceinline__ void pin_row(float (&a)[8]) {
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]),
               "+v"(a[6]), "+v"(a[7]));
}

// Barrier for data exchanged through LDS: this wave's LDS accesses are
// complete, global loads stay in flight (the compiler waits for those where
// their registers are used).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---------------------------------------------------------------------------
// READ
// ---------------------------------------------------------------------------
//
// 1. adapter_read_partial_kernel: one 512-thread block per (K chunk of 192
//    rows, column tile, group of up to 8 owners); each lane streams 16 bytes
//    of every W0 row of the tile once and applies it to all the block's
//    owners.  The eight waves split the chunk's rows, 24 each.  A wave requests
//    the x values of its own rows (every owner of the group), then the u
//    share's x and A values, then all of its W0 rows, and only then waits:
//    loads of one wave return in order, so x arrives first, and no wave waits
//    for another's x before requesting W0.  Each owner's wave sums are added
//    in wave order into one partial per (owner, chunk, tile).  Owner groups of
//    one (chunk, tile) sit on one XCD (dispatch is round-robin over the 8
//    XCDs).  The chunk's tile blocks also form the owners' chunk shares of
//    u = x A (r values each, ordered two-level sums), owner g in tile
//    g mod (tiles), and the first tile's block appends the x chunk to the
//    owners' tails if asked.
// 2. adapter_read_reduce_kernel: u = sum of the chunks' shares in chunk
//    order; y[n] = (sum of the W0 partials: four contiguous quarters of the
//    chunks, each in chunk order, then the quarters in order) +
//    sum_j u[j] B[j][n], rounded once to the io dtype.

struct AReadParams {
  const void* x;
  void* y;
  const void* w0;
  float* part;        // [n_owners][ks][npad]
  float* upart;       // [n_owners][ks][rank]
  int count, d_ff, d_model, rank, ks, nt, npad;
  const void* state[RWTTT_MAX_GROUP];
  uint32_t row[RWTTT_MAX_GROUP];
  void* tail[RWTTT_MAX_GROUP];
};

template <typename IO, typename ST>
__global__ void __launch_bounds__(kAThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
adapter_read_partial_kernel(const AReadParams p) {
  constexpr int COLS = 16 / sizeof(IO);
  constexpr int TILE_N = 64 * COLS;
  __shared__ float xs[kAChunk][kAGroup];   // x chunk, row-major over owners
  // bf16 io: the same chunk as raw bf16, rows 2m and 2m + 1 of an owner in one word
  __shared__ uint16_t xh[sizeof(IO) == 2 ? kAChunk / 2 : 1][kAGroup][2];
  __shared__ float red[kAGroup][kAWaves][TILE_N];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar indexing
  // block -> (XCD, position) -> ((chunk, tile) pair, owner group)
  const int ngroups = (p.count + kAGroup - 1) / kAGroup;
  const int xcd = blockIdx.x & 7;
  const int pos = blockIdx.x >> 3;
  const int pl = pos / ngroups;
  const int gi = pos - pl * ngroups;
  const int pair = pl * 8 + xcd;
  if (pair >= p.ks * p.nt) return;
  const int kc = pair / p.nt;
  const int nt = pair - kc * p.nt;
  const int k0 = kc * kAChunk;
  const int kn = min(kAChunk, p.d_ff - k0);
  const int col = nt * TILE_N + lane * COLS;
  const bool col_ok = col < p.d_model;
  const int b0 = gi * kAGroup;
  const int ng = min(kAGroup, p.count - b0);

  // 1. requests, in the order they are needed, every one unconditional
  //    (indices clamped into the buffers, unused values zeroed afterwards) so
  //    that no load waits inside a branch.
  uint32_t rows[kAGroup];   // owner rows of the group's slots (block-uniform)
#pragma unroll
  for (int g = 0; g < kAGroup; ++g) rows[g] = p.row[b0 + min(g, ng - 1)];
  // this wave's x values: its 24 rows of every owner of the group (lane l
  // holds value l + 64 t: owner (l + 64 t) / 24, row (l + 64 t) % 24)
  constexpr int XW = kAGroup * kARows / 64;
  const int kw0 = wave * kARows;
  IO xw[XW];
#pragma unroll
  for (int t = 0; t < XW; ++t) {
    const int idx = lane + 64 * t;
    const int g = idx / kARows, k = idx - g * kARows;
    uint32_t r = rows[0];
#pragma unroll
    for (int g2 = 1; g2 < kAGroup; ++g2) r = g == g2 ? rows[g2] : r;
    xw[t] = static_cast<const IO*>(p.x)[size_t(r) * p.d_ff + k0 + min(kw0 + k, kn - 1)];
  }
  // u share (step 2): wave i takes owner nt + i * tiles of the group; its lanes
  // hold rows lane, lane + 64, lane + 128 of the chunk: their x values and
  // their first eight A columns
  const int ug = nt + wave * p.nt;
  const ST* uA = static_cast<const ST*>(p.state[b0 + (ug < ng ? ug : 0)]);
  const uint32_t urow = p.row[b0 + (ug < ng ? ug : 0)];
  IO xu[kAURows];
  float apre[kAURows][8];
#pragma unroll
  for (int r = 0; r < kAURows; ++r)
    xu[r] = static_cast<const IO*>(p.x)[size_t(urow) * p.d_ff + k0 + min(lane + 64 * r, kn - 1)];
  if (ug < ng) {
#pragma unroll
    for (int r = 0; r < kAURows; ++r) {
      const size_t at = size_t(k0 + min(lane + 64 * r, kn - 1)) * p.rank;
#pragma unroll
      for (int j = 0; j < 8; ++j) apre[r][j] = Elem<ST>::get(uA, at + min(j, p.rank - 1));
    }
  } else {
#pragma unroll
    for (int r = 0; r < kAURows; ++r)
#pragma unroll
      for (int j = 0; j < 8; ++j) apre[r][j] = 0.f;
  }
  // then this wave's W0 rows; rows past the chunk repeat its last row (their
  // x is zero); lanes past d_model read column 0 and their sums are dropped
  const IO* wbase = static_cast<const IO*>(p.w0) + size_t(k0) * p.d_model + (col_ok ? col : 0);
  Packed<IO, COLS> w[kARows];
#pragma unroll
  for (int u = 0; u < kARows; ++u)
    load_packed<false>(wbase + size_t(min(kw0 + u, kn - 1)) * p.d_model, w[u]);
  __builtin_amdgcn_sched_barrier(0);   // every request is out before x is waited for
  // the wave stages its own rows of x (no other wave reads them before the
  // block barrier below; LDS requests of one wave complete in order)
#pragma unroll
  for (int t = 0; t < XW; ++t) {
    const int idx = lane + 64 * t;
    const int g = idx / kARows, k = kw0 + idx - (idx / kARows) * kARows;
    const bool ok = g < ng && k < kn;
    xs[k][g] = ok ? to_f32(xw[t]) : 0.f;
    if constexpr (sizeof(IO) == 2) xh[k >> 1][g][k & 1] = ok ? xw[t] : uint16_t(0);
  }

  // 2. u share of this chunk for the wave's owner: sum_k x[k] A[k][j], eight
  //    rank columns per pass: each lane sums its rows in order, then a
  //    butterfly over the wave (every lane ends with the same sum).  The first
  //    pass uses the requested columns and runs while the W0 rows are still
  //    arriving; passes for ranks above eight load theirs at the end.
  float* ur = p.upart + (size_t(p.row[b0 + (ug < ng ? ug : 0)]) * p.ks + kc) * p.rank;
  auto u_pass = [&](int j0, bool loaded) {
    float sj[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sj[j] = 0.f;
#pragma unroll
    for (int r = 0; r < kAURows; ++r) {
      const int k = lane + 64 * r;
      const float xk = k < kn ? to_f32(xu[r]) : 0.f;   // zero past the chunk
      const size_t at = size_t(k0 + min(k, kn - 1)) * p.rank;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = loaded ? apre[r][j] : Elem<ST>::get(uA, at + min(j0 + j, p.rank - 1));
        sj[j] = fmaf(xk, j0 + j < p.rank ? a : 0.f, sj[j]);
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
      for (int j = 0; j < 8; ++j) sj[j] += __shfl_xor(sj[j], m);
    float v = sj[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) v = lane == j ? sj[j] : v;
    if (lane < 8 && j0 + lane < p.rank) ur[j0 + lane] = v;
  };
  if (ug < ng) u_pass(0, true);

  // 3. x W0 over this wave's rows for every owner of the group, rows in order
  float acc[kAGroup][COLS];
#pragma unroll
  for (int g = 0; g < kAGroup; ++g)
#pragma unroll
    for (int c = 0; c < COLS; ++c) acc[g][c] = 0.f;
  if constexpr (sizeof(IO) == 2) {
    // bf16: rows in pairs, one v_dot2 per (owner, column) adds
    // x[2m] W[2m][c] + x[2m+1] W[2m+1][c]; v_perm pairs the two rows' values
    // of a column in one word
#pragma unroll
    for (int m = 0; m < kARows / 2; ++m) {
      const uint32_t* xq = reinterpret_cast<const uint32_t*>(&xh[(kw0 >> 1) + m][0][0]);
      const uint4 xa = *reinterpret_cast<const uint4*>(xq);
      const uint4 xb = *reinterpret_cast<const uint4*>(xq + 4);
      const uint32_t xpair[kAGroup] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
#pragma unroll
      for (int i = 0; i < COLS / 2; ++i) {
        const uint32_t lo = __builtin_amdgcn_perm(w[2 * m + 1].w[i], w[2 * m].w[i], 0x05040100u);
        const uint32_t hi = __builtin_amdgcn_perm(w[2 * m + 1].w[i], w[2 * m].w[i], 0x07060302u);
#pragma unroll
        for (int g = 0; g < kAGroup; ++g) {
          acc[g][2 * i] = dot2_bf16(xpair[g], lo, acc[g][2 * i]);
          acc[g][2 * i + 1] = dot2_bf16(xpair[g], hi, acc[g][2 * i + 1]);
        }
      }
      // one row pair at a time: its x values and paired W0 die before the next
#pragma unroll
      for (int g = 0; g < kAGroup; ++g) pin_row(acc[g]);
    }
  } else {
#pragma unroll
    for (int u = 0; u < kARows; ++u) {
      float xr[kAGroup];
#pragma unroll
      for (int g = 0; g < kAGroup; g += 4) {
        const float4 x4 = *reinterpret_cast<const float4*>(&xs[kw0 + u][g]);
        xr[g] = x4.x; xr[g + 1] = x4.y; xr[g + 2] = x4.z; xr[g + 3] = x4.w;
      }
#pragma unroll
      for (int g = 0; g < kAGroup; ++g)
#pragma unroll
        for (int c = 0; c < COLS; ++c) acc[g][c] = fmaf(xr[g], w[u].get(c), acc[g][c]);
      // one row at a time: the row's products are done here, so its x values
      // and converted W0 die before the next row's are formed
#pragma unroll
      for (int g = 0; g < kAGroup; ++g) pin_row(acc[g]);
    }
  }

  // 4. per owner: the waves' sums in wave order -> one partial per (owner,
  //    chunk, tile), all owners in one pass through LDS
#pragma unroll
  for (int g = 0; g < kAGroup; ++g)
#pragma unroll
    for (int c = 0; c < COLS; c += 4)
      *reinterpret_cast<float4*>(&red[g][wave][lane * COLS + c]) =
          col_ok ? make_float4(acc[g][c], acc[g][c + 1], acc[g][c + 2], acc[g][c + 3])
                 : make_float4(0.f, 0.f, 0.f, 0.f);
  lds_barrier();
  for (int idx = tid; idx < kAGroup * TILE_N / 4; idx += kAThreads) {
    const int g = idx / (TILE_N / 4), j = (idx - g * (TILE_N / 4)) * 4;
    if (g < ng) {
      float4 v = *reinterpret_cast<const float4*>(&red[g][0][j]);
#pragma unroll
      for (int w2 = 1; w2 < kAWaves; ++w2) {
        const float4 t = *reinterpret_cast<const float4*>(&red[g][w2][j]);
        v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
      }
      uint32_t r = rows[0];
#pragma unroll
      for (int g2 = 1; g2 < kAGroup; ++g2) r = g == g2 ? rows[g2] : r;
      *reinterpret_cast<float4*>(p.part + (size_t(r) * p.ks + kc) * p.npad + nt * TILE_N + j) = v;
    }
  }

  if (ug < ng)
    for (int j0 = 8; j0 < p.rank; j0 += 8) u_pass(j0, false);

  // 5. TailBufferUpdate: the first tile's block appends the staged x chunk
  if (nt == 0) {
    for (int g = 0; g < ng; ++g) {
      if (p.tail[b0 + g] == nullptr) continue;
      for (int k = tid; k < kn; k += kAThreads) Elem<IO>::put(p.tail[b0 + g], k0 + k, xs[k][g]);
    }
  }
}

template <typename IO, typename ST>
__global__ void __launch_bounds__(256) adapter_read_reduce_kernel(const AReadParams p) {
  __shared__ float us[8][RWTTT_MAX_RANK];
  __shared__ float u[RWTTT_MAX_RANK];
  __shared__ float qs[4][kARedCols];
  const int b = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = blockIdx.x * kARedCols + lane;
  const int nc = min(n, p.d_model - 1);
  const size_t r = p.row[b];
  const int per = (p.ks + 3) / 4;
  const int k0 = wave * per, k1 = min(p.ks, k0 + per);
  const float* q = p.part + r * p.ks * p.npad + nc;
  const int j = threadIdx.x & 31, qq = threadIdx.x >> 5;
  const ST* Bm = static_cast<const ST*>(p.state[b]) + size_t(p.d_ff) * p.rank;

  // 1. every first-round request at once, unconditional (indices clamped,
  //    unused values dropped below): this lane's W0 partials (its wave's
  //    quarter of the chunks), its x A shares (chunks qq, qq + 8, ...) and the
  //    first eight B values of its column
  float a[kARedLoads], t[8], bv[8];
#pragma unroll
  for (int i = 0; i < kARedLoads; ++i) a[i] = q[size_t(min(k0 + i, p.ks - 1)) * p.npad];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    t[i] = p.upart[(r * p.ks + min(qq + 8 * i, p.ks - 1)) * p.rank + min(j, p.rank - 1)];
#pragma unroll
  for (int i = 0; i < 8; ++i) bv[i] = Elem<ST>::get(Bm, size_t(min(i, p.rank - 1)) * p.d_model + nc);

  // 2. W0 partials: the four waves sum four contiguous quarters of the
  //    chunks, each in chunk order, and the quarters are added in order
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kARedLoads; ++i) s += k0 + i < k1 ? a[i] : 0.f;
  for (int kc = k0 + kARedLoads; kc < k1; kc += 8) {
    float a2[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a2[i] = kc + i < k1 ? q[size_t(kc + i) * p.npad] : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += a2[i];
  }
  qs[wave][lane] = s;
  // u[j] = sum over chunks of the x A shares: eight strided partial sums per
  // rank column (chunks qq, qq + 8, qq + 16, ... in order), then those eight in order
  if (j < p.rank) {
    float su = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) su += qq + 8 * i < p.ks ? t[i] : 0.f;
    for (int kc = qq + 64; kc < p.ks; kc += 64) {
      float t2[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) t2[i] = kc + 8 * i < p.ks ? p.upart[(r * p.ks + kc + 8 * i) * p.rank + j] : 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) su += t2[i];
    }
    us[qq][j] = su;
  }
  lds_barrier();
  if (int(threadIdx.x) < p.rank) {
    float su = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) su += us[i][threadIdx.x];
    u[threadIdx.x] = su;
  }
  lds_barrier();
  if (wave != 0 || n >= p.d_model) return;
  // 3. + u B, rank columns in order
  float lr = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (i < p.rank) lr = fmaf(u[i], bv[i], lr);
  for (int j0 = 8; j0 < p.rank; j0 += 8) {
    float b2[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) b2[i] = j0 + i < p.rank ? Elem<ST>::get(Bm, size_t(j0 + i) * p.d_model + n) : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (j0 + i < p.rank) lr = fmaf(u[j0 + i], b2[i], lr);
  }
  Elem<IO>::put(p.y, r * p.d_model + n, (((qs[0][lane] + qs[1][lane]) + qs[2][lane]) + qs[3][lane]) + lr);
}

// ---------------------------------------------------------------------------
// WRITE
// ---------------------------------------------------------------------------
//
// Both steps are contractions against the fp32 factors and run on the fp32
// matrix instruction v_mfma_f32_16x16x4_f32 (fp32 products, fp32 sums: nothing
// is narrowed).  Their traffic is the evidence, read once by each kernel, and a
// few passes of L2 over the factors and their products with the evidence.  Four
// owners at 9728 x 2560, rank 16, C = 256 (31 MB): 12.9 + 12.7 us, down from 75.2
// + 36.5 us when a block took one evidence row (and read the whole factor slice
// for it) and one thread one value; three owners at 4608 x 304, rank 26, C = 735:
// 37 against 422 us.  What is left is the latency of dependent loads (few
// waves, two launches) and, for large C r, the matrix rate.
//
// 1. adapter_pq_kernel: one 512-thread block per (tile of 16 CT evidence rows
//    c, slice of 1024 columns of G / rows of Z, owner) forms the slice's share of
//    P[c][j] = sum_n G[c][n] B[j][n] or Q[c][j] = sum_k Z[c][k] A[k][j].  Each of
//    the eight waves contracts 128 elements for all 16 CT rows and all rank
//    columns (JT tiles of 16); a lane's 16 bytes of evidence feed eight (bf16)
//    matrix steps.  The waves' sums are added as a tree.  The factor slice is
//    read once per evidence tile: CT = 4 halves that L2 traffic against 2 where
//    rank <= 16 leaves the registers for it and C > 128 the blocks; CT = 1 where
//    its blocks all fit the CUs at once.
// 2. adapter_update_kernel: one block of NW waves per 64 rows k of A or columns
//    n of B, all rank columns: A'[k][j] = A[k][j] + eta sum_c Z[c][k] P[c][j] and
//    B'[j][n] = B[j][n] + eta sum_c Q[c][j] G[c][n].  The waves take contiguous
//    shares of the evidence rows, each sum in c order (four rows per matrix
//    step), then the waves as a tree; the slice shares of P and Q are added in
//    slice order in the register that feeds the matrix step, so the kernel has
//    no staging and no barrier before its last sum.
//
// Every order depends only on the shapes and the chunk.

constexpr int kASlice = 1024;    // columns of G / rows of Z per P / Q block
constexpr int kAUpdRows = 64;    // A rows or B columns per update block
constexpr int kAWWaves = 8;      // waves of a WRITE block
constexpr int kAWThreads = 64 * kAWWaves;

// Sum of N (a power of two) waves' values as a balanced tree.
template <int N, typename F> __device__ __forceinline__ float wave_sum(F v, int first = 0) {
  if constexpr (N == 1) return v(first);
  else return wave_sum<N / 2>(v, first) + wave_sum<N / 2>(v, first + N / 2);
}

struct AWriteParams {
  int count, chunk, d_ff, d_model, rank, max_chunk, sp, sq;   // sp, sq: slices of N, K
  float eta;
  float* P;     // [n_owners][max_chunk][sp][rank] slice shares
  float* Q;     // [n_owners][max_chunk][sq][rank]
  const void* live[RWTTT_MAX_GROUP];
  void* shadow[RWTTT_MAX_GROUP];
  const void* z[RWTTT_MAX_GROUP];
  const void* g[RWTTT_MAX_GROUP];
  uint32_t row[RWTTT_MAX_GROUP];
};

// Element at a 32-bit byte offset from a wave-uniform base: one scalar base and
// one vector register of address instead of 64-bit arithmetic in every lane.
template <typename T> __device__ __forceinline__ const T* at_byte(const void* base, uint32_t off) {
  return reinterpret_cast<const T*>(static_cast<const char*>(base) + off);
}

template <typename IO, typename ST, int JT, int CT>
__global__ void __launch_bounds__(kAWThreads) adapter_pq_kernel(const AWriteParams p) {
  constexpr int KW = kASlice / kAWWaves;   // contracted elements per wave
  constexpr int KG = 32;                   // elements per group of loads: 4 quarter-waves x 8
  constexpr int NG = KW / KG;
  __shared__ float red[kAWWaves][16 * CT][16 * JT + 1];
  const int b = blockIdx.z;
  const int s = blockIdx.x;                // < sp: a P slice; else a Q slice
  const int c0 = int(blockIdx.y) * 16 * CT;
  const bool is_p = s < p.sp;
  const int lim = is_p ? p.d_model : p.d_ff;
  const ST* A = static_cast<const ST*>(p.live[b]);
  const ST* F = is_p ? A + size_t(p.d_ff) * p.rank : A;   // B for P, A for Q
  const IO* E = static_cast<const IO*>(is_p ? p.g[b] : p.z[b]) + size_t(c0) * lim;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, kq = lane >> 4;
  const int i0 = (is_p ? s : s - p.sp) * kASlice + wave * KW;

  // lane (i16, kq) holds elements kb .. kb+7 of evidence row c0 + i16 (+ 16 ci)
  // and of factor column i16 (+ 16 jt); matrix step t contracts the four
  // quarters' element t.  Addresses past the matrix are clamped into it and
  // both operands zeroed (eight elements are in or out together: the extents
  // are multiples of 8); rows past the chunk and columns past the rank only
  // reach sums that are not stored.
  uint32_t eoff[CT], foff[JT];             // byte offsets of element 0 of row / column i16
#pragma unroll
  for (int ci = 0; ci < CT; ++ci)
    eoff[ci] = uint32_t(min(16 * ci + i16, p.chunk - 1 - c0)) * uint32_t(lim) * uint32_t(sizeof(IO));
#pragma unroll
  for (int jt = 0; jt < JT; ++jt)
    foff[jt] = uint32_t(min(16 * jt + i16, p.rank - 1)) * uint32_t(is_p ? p.d_model : 1) * uint32_t(sizeof(ST));

  f32x4_t acc[CT][JT];
#pragma unroll
  for (int ci = 0; ci < CT; ++ci)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) acc[ci][jt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  auto contract = [&](auto isp) {
    constexpr bool IS_P = decltype(isp)::value;
    struct Ops { Packed<IO, 8> e[CT]; Packed<ST, 8> v[IS_P ? JT : 1]; ST f[IS_P ? 1 : JT][8]; };
    auto load = [&](Ops& o, int g) {
      const uint32_t kc = uint32_t(min(i0 + g * KG + 8 * kq, lim - 8));
#pragma unroll
      for (int ci = 0; ci < CT; ++ci)
        load_packed<false>(at_byte<IO>(E, eoff[ci] + kc * uint32_t(sizeof(IO))), o.e[ci]);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        if constexpr (IS_P) {
          load_packed<false>(at_byte<ST>(F, foff[jt] + kc * uint32_t(sizeof(ST))), o.v[jt]);
        } else {
          const uint32_t step = uint32_t(p.rank) * uint32_t(sizeof(ST));
          const char* Ft = reinterpret_cast<const char*>(F);
#pragma unroll
          for (int t = 0; t < 8; ++t) o.f[jt][t] = *at_byte<ST>(Ft + t * step, foff[jt] + kc * step);
        }
      }
    };
    auto mul = [&](const Ops& o, int g) {
      const bool ok = i0 + g * KG + 8 * kq < lim;
      // four short chains from zero (8 products each), added as a tree to the
      // running sum: one chain over the wave's 128 products rounds more often
      // (2.3e-7 against 1.4e-7 from 64 bits at C = 256, 9728 x 2560)
#pragma unroll
      for (int ci = 0; ci < CT; ++ci)
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          f32x4_t h[4];
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            float fv;
            if constexpr (IS_P) fv = o.v[jt].get(t);
            else fv = to_f32(o.f[jt][t]);
            h[t >> 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                ok ? o.e[ci].get(t) : 0.f, ok ? fv : 0.f, (t & 1) ? h[t >> 1] : f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          }
          acc[ci][jt] += (h[0] + h[1]) + (h[2] + h[3]);
        }
    };
    // two sets of operands: a group's loads are in flight while the one before
    // it is multiplied
    Ops o[2];
    load(o[0], 0);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g + 1 < NG) load(o[(g + 1) & 1], g + 1);
      __builtin_amdgcn_sched_barrier(0);
      mul(o[g & 1], g);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if (is_p) contract(std::true_type{});
  else contract(std::false_type{});
  // register q of lane (i16, kq) holds row 4 kq + q, column i16 of a 16 x 16 tile
#pragma unroll
  for (int ci = 0; ci < CT; ++ci)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[wave][16 * ci + 4 * kq + q][16 * jt + i16] = acc[ci][jt][q];
  lds_barrier();
  const int ns = is_p ? p.sp : p.sq, sl = is_p ? s : s - p.sp;
  float* out = (is_p ? p.P : p.Q) + (size_t(p.row[b]) * p.max_chunk + c0) * ns * p.rank;
  const int items = min(16 * CT, p.chunk - c0) * p.rank;
  for (int t = tid; t < items; t += kAWThreads) {
    const int c = t / p.rank, j = t - c * p.rank;
    out[(size_t(c) * ns + sl) * p.rank + j] = wave_sum<kAWWaves>([&](int w) { return red[w][c][j]; });
  }
}

template <typename IO, typename ST, int JT, int NW>
__global__ void __launch_bounds__(64 * NW) adapter_update_kernel(const AWriteParams p) {
  constexpr int QB = 4;                    // matrix steps (of four evidence rows) per group of loads
  constexpr int SB = 3;                    // further slice shares of P or Q in flight
  constexpr int NL = kAUpdRows * 16 * JT / (64 * NW);   // most values a thread finishes
  __shared__ float red[NW][16 * JT][kAUpdRows + 1];
  const int b = blockIdx.y;
  const int na = (p.d_ff + kAUpdRows - 1) / kAUpdRows;
  const bool is_a = int(blockIdx.x) < na;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, cq = lane >> 4;
  const int i0 = (is_a ? int(blockIdx.x) : int(blockIdx.x) - na) * kAUpdRows;
  const int lim = is_a ? p.d_ff : p.d_model;
  const int rows = min(kAUpdRows, lim - i0);
  const int ns = is_a ? p.sp : p.sq;        // A uses P (slices of N); B uses Q (slices of K)
  const float* S = (is_a ? p.P : p.Q) + size_t(p.row[b]) * p.max_chunk * ns * p.rank;
  const IO* E = static_cast<const IO*>(is_a ? p.z[b] : p.g[b]);
  const ST* live = static_cast<const ST*>(p.live[b]) +
                   (is_a ? size_t(i0) * p.rank : size_t(p.d_ff) * p.rank + i0);
  ST* shadow = static_cast<ST*>(p.shadow[b]) + (live - static_cast<const ST*>(p.live[b]));
  // value t of the block: A row i0 + t / r, column t % r (one contiguous run),
  // or B row t / 64, column i0 + t % 64
  const int nv = is_a ? rows * p.rank : kAUpdRows * p.rank;
  auto at_of = [&](int t) {
    return is_a ? uint32_t(t) : uint32_t(t / kAUpdRows) * uint32_t(p.d_model) + uint32_t(min(t % kAUpdRows, rows - 1));
  };
  float lv[NL];
#pragma unroll
  for (int h = 0; h < NL; ++h)
    lv[h] = to_f32(*at_byte<ST>(live, at_of(min(tid + (64 * NW) * h, nv - 1)) * uint32_t(sizeof(ST))));

  f32x4_t acc[4][JT];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) acc[t][jt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // lane (i16, cq) holds evidence row 4 q + cq at columns i0 + 4 i16 .. + 3: row
  // i16 of matrix t is column i0 + 4 i16 + t.  Rows past the chunk are clamped
  // and both operands zeroed.
  const uint32_t ec = uint32_t(min(i0 + 4 * i16, lim - 4)) * uint32_t(sizeof(IO));
  // matrix column i16 of tile jt is rank column JT i16 + jt
  const uint32_t jc = uint32_t(min(JT * i16, p.rank - JT)) * 4u;
  const bool odd = JT * i16 == p.rank - 1;
  const uint32_t spitch = uint32_t(ns) * uint32_t(p.rank) * 4u;
  const int nq = (p.chunk + 3) / 4, per = (nq + NW - 1) / NW;
  const int q1 = min(nq, (wave + 1) * per);
  auto share = [&](const char* Sk, uint32_t off, float (&f)[JT]) {
    if constexpr (JT == 1) {
      f[0] = *at_byte<float>(Sk, off);
    } else {
      // columns 2 i16 and 2 i16 + 1 in one load (4-byte aligned); an odd rank's
      // last lane steps back one column and takes the upper half
      struct __attribute__((packed, aligned(4))) Two { float v[2]; };
      const Two w = *at_byte<Two>(Sk, off);
      f[0] = odd ? w.v[1] : w.v[0];
      f[1] = w.v[1];
    }
  };
  for (int q0 = wave * per; q0 < q1; q0 += QB) {
    Packed<IO, 4> e[QB];
    float f[QB][JT];
    const IO* Eq = E + size_t(4 * q0) * lim;
    const char* Sq = reinterpret_cast<const char*>(S) + size_t(4 * q0) * spitch;
    uint32_t so[QB];
#pragma unroll
    for (int u = 0; u < QB; ++u) {
      const uint32_t c = uint32_t(min(4 * u + cq, p.chunk - 1 - 4 * q0));
      load_packed<false>(at_byte<IO>(Eq, c * uint32_t(lim) * uint32_t(sizeof(IO)) + ec), e[u]);
      so[u] = c * spitch + jc;
      share(Sq, so[u], f[u]);
    }
    for (int sl = 1; sl < ns; sl += SB) {
      float a[SB][QB][JT];
#pragma unroll
      for (int k = 0; k < SB; ++k) {
        const char* Sk = Sq + size_t(min(sl + k, ns - 1)) * p.rank * 4;
#pragma unroll
        for (int u = 0; u < QB; ++u) share(Sk, so[u], a[k][u]);
      }
#pragma unroll
      for (int k = 0; k < SB; ++k)
#pragma unroll
        for (int u = 0; u < QB; ++u)
#pragma unroll
          for (int jt = 0; jt < JT; ++jt) f[u][jt] = sl + k < ns ? f[u][jt] + a[k][u][jt] : f[u][jt];
    }
    // one short chain from zero per group (16 products), added to the running sum
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        f32x4_t h = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < QB; ++u) {
          const bool ok = q0 + u < q1 && 4 * (q0 + u) + cq < p.chunk;
          h = __builtin_amdgcn_mfma_f32_16x16x4f32(ok ? e[u].get(t) : 0.f, ok ? f[u][jt] : 0.f, h, 0, 0, 0);
        }
        acc[t][jt] += h;
      }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[wave][JT * i16 + jt][4 * (4 * cq + q) + t] = acc[t][jt][q];
  lds_barrier();
  const float eta = p.eta;
#pragma unroll
  for (int h = 0; h < NL; ++h) {
    const int t = tid + (64 * NW) * h;
    const int k = is_a ? t / p.rank : t % kAUpdRows, j = is_a ? t - k * p.rank : t / kAUpdRows;
    if (t < nv && k < rows) {
      const float d = wave_sum<NW>([&](int w) { return red[w][j][k]; });
      Elem<ST>::put(shadow, at_of(t), lv[h] + eta * d);
    }
  }
}

template <typename IO, typename ST>
hipError_t launch_adapter_read_t(const AdapterReadLaunch& L, hipStream_t stream) {
  const AdapterGeometry g = adapter_geometry(L.d_ff, L.d_model, L.io_bf16, L.rank, L.n_owners);
  AReadParams p;
  p.x = L.x;
  p.y = L.y;
  p.w0 = L.w0;
  p.part = static_cast<float*>(L.workspace);
  p.upart = reinterpret_cast<float*>(static_cast<char*>(L.workspace) + g.u_offset);
  p.count = L.count;
  p.d_ff = L.d_ff;
  p.d_model = L.d_model;
  p.rank = L.rank;
  p.ks = g.ks;
  p.nt = g.nt;
  p.npad = g.npad;
  for (int b = 0; b < RWTTT_MAX_GROUP; ++b) {
    const bool in = b < L.count;
    p.state[b] = in ? L.state[b] : nullptr;
    p.row[b] = in ? L.row[b] : 0u;
    p.tail[b] = in ? L.tail[b] : nullptr;
  }
  const unsigned pairs8 = unsigned((g.ks * g.nt + 7) / 8 * 8);
  const unsigned groups = unsigned((L.count + kAGroup - 1) / kAGroup);
  hipLaunchKernelGGL((adapter_read_partial_kernel<IO, ST>), dim3(pairs8 * groups),
                     dim3(kAThreads), 0, stream, p);
  hipLaunchKernelGGL((adapter_read_reduce_kernel<IO, ST>), dim3((L.d_model + kARedCols - 1) / kARedCols, L.count),
                     dim3(256), 0, stream, p);
  return hipGetLastError();
}

template <typename IO, typename ST>
hipError_t launch_adapter_write_t(const AdapterWriteLaunch& L, hipStream_t stream) {
  const AdapterGeometry g = adapter_geometry(L.d_ff, L.d_model, L.io_bf16, L.rank, L.n_owners);
  AWriteParams p;
  p.count = L.count;
  p.chunk = L.chunk;
  p.d_ff = L.d_ff;
  p.d_model = L.d_model;
  p.rank = L.rank;
  p.max_chunk = RWTTT_ADAPTER_MAX_CHUNK;
  p.sp = (L.d_model + kASlice - 1) / kASlice;
  p.sq = (L.d_ff + kASlice - 1) / kASlice;
  p.eta = L.eta;
  p.P = reinterpret_cast<float*>(static_cast<char*>(L.workspace) + g.pq_offset);
  p.Q = p.P + size_t(L.n_owners) * RWTTT_ADAPTER_MAX_CHUNK * p.sp * L.rank;
  for (int b = 0; b < RWTTT_MAX_GROUP; ++b) {
    const bool in = b < L.count;
    p.live[b] = in ? L.live[b] : nullptr;
    p.shadow[b] = in ? L.shadow[b] : nullptr;
    p.z[b] = in ? L.z[b] : nullptr;
    p.g[b] = in ? L.g[b] : nullptr;
    p.row[b] = in ? L.row[b] : 0u;
  }
  const unsigned slices = unsigned(p.sp + p.sq), owners = unsigned(L.count);
  const unsigned tiles = unsigned((L.d_ff + kAUpdRows - 1) / kAUpdRows + (L.d_model + kAUpdRows - 1) / kAUpdRows);
  auto pq = [&](auto jt, auto ct) {
    constexpr int JT = decltype(jt)::value, CT = decltype(ct)::value;
    hipLaunchKernelGGL((adapter_pq_kernel<IO, ST, JT, CT>),
                       dim3(slices, unsigned((L.chunk + 16 * CT - 1) / (16 * CT)), owners), dim3(kAWThreads), 0,
                       stream, p);
  };
  auto update = [&](auto jt, auto nw) {
    constexpr int JT = decltype(jt)::value, NW = decltype(nw)::value;
    hipLaunchKernelGGL((adapter_update_kernel<IO, ST, JT, NW>), dim3(tiles, owners), dim3(64 * NW), 0, stream, p);
  };
  using one = std::integral_constant<int, 1>;
  using two = std::integral_constant<int, 2>;
  using four = std::integral_constant<int, 4>;
  using eight = std::integral_constant<int, 8>;
  switch (adapter_pq_tiles(int(slices), L.chunk, L.count, L.rank)) {
    case 1: L.rank > 16 ? pq(two{}, one{}) : pq(one{}, one{}); break;
    case 2: L.rank > 16 ? pq(two{}, two{}) : pq(one{}, two{}); break;
    default: pq(one{}, four{});
  }
  auto by_waves = [&](auto jt) {
    // a wave's group of loads is 16 evidence rows: eight waves have work for
    // each only above 64 (4.9 against 5.6 us at C = 64, one owner, rank 8)
    if (L.chunk <= 64) update(jt, four{});
    else update(jt, eight{});
  };
  if (L.rank > 16) by_waves(two{});
  else by_waves(one{});
  return hipGetLastError();
}

}  // namespace

AdapterGeometry adapter_geometry(int d_ff, int d_model, int io_bf16, int rank, int n_owners) {
  AdapterGeometry g;
  const int tile = 64 * (io_bf16 ? 8 : 4);
  g.ks = (d_ff + kAChunk - 1) / kAChunk;
  g.nt = (d_model + tile - 1) / tile;
  g.npad = g.nt * tile;
  g.part_floats = size_t(n_owners) * g.ks * g.npad;
  auto align = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
  g.u_offset = align(g.part_floats * sizeof(float));
  const size_t u_floats = size_t(n_owners) * g.ks * rank;
  g.pq_offset = g.u_offset + align(u_floats * sizeof(float));
  const int slices = (d_model + kASlice - 1) / kASlice + (d_ff + kASlice - 1) / kASlice;
  const size_t pq_floats = size_t(n_owners) * RWTTT_ADAPTER_MAX_CHUNK * slices * rank;
  g.total_bytes = g.pq_offset + align(pq_floats * sizeof(float));
  return g;
}

hipError_t launch_adapter_read(const AdapterReadLaunch& L, hipStream_t stream) {
  if (L.io_bf16) {
    return L.state_bf16 ? launch_adapter_read_t<uint16_t, uint16_t>(L, stream)
                        : launch_adapter_read_t<uint16_t, float>(L, stream);
  }
  return L.state_bf16 ? launch_adapter_read_t<float, uint16_t>(L, stream)
                      : launch_adapter_read_t<float, float>(L, stream);
}

hipError_t launch_adapter_write(const AdapterWriteLaunch& L, hipStream_t stream) {
  if (L.io_bf16) {
    return L.state_bf16 ? launch_adapter_write_t<uint16_t, uint16_t>(L, stream)
                        : launch_adapter_write_t<uint16_t, float>(L, stream);
  }
  return L.state_bf16 ? launch_adapter_write_t<float, uint16_t>(L, stream)
                      : launch_adapter_write_t<float, float>(L, stream);
}

}  // namespace rwttt
