// Exact per-sample scores of one linear layer (dr_score_exact), the three
// contraction orders of Sec. 4.3 for s_i = <gbar*, g_i> with the mean target
// gradient gbar* = (1/m) sum_j G*_j:
//   DIRECT  materialise each G_i (tile by tile, never stored) and take its
//           inner product with gbar* (update-assembly kernel in score mode,
//           update.hip);
//   PIP     sum_t dy_{i,t}^T gbar* x_{i,t}: a GEMM of the example's token
//           rows with gbar* followed by a dot with the dy rows (pip_kernel;
//           pip_small_kernel for calls of few tiles);
//   GIP     (1/m) sum_j <D_i D*_j^T, X_i X*_j^T>: the two T x T token
//           cross-correlations of every (example, target) pair, multiplied
//           elementwise and summed (gip_kernel).
// gbar* is assembled first from the target rows with weights 1/m (the
// update-assembly kernel); PIP multiplies by it in bf16 as a hi + lo pair
// (two MFMAs, relative rounding ~2^-17 instead of bf16's 2^-9).
//
// Both kernels work on the valid tokens of all examples packed one after
// another (packed position p = cum[i] + t), so a tile is full whatever the
// length mix, and sum its rows per example at the end: a row of the product
// belongs to one token.  Operands are row panels whose reduction index is
// contiguous in memory (token rows of x / dy, rows of gbar*), staged by
// buffer->LDS DMA in 64-wide steps in the swizzled 128-byte-row layout.
// Rows past the last token and columns past a width load as zeros
// (out-of-range buffer offsets), so padding is never read.  Rows are addressed
// by 32-bit offsets from a tile's first example.  A block whose rows lie
// further apart, over a run of empty examples, is taken in pieces, each from
// its own first example (PIECES, where the batch is large enough for that: the
// loop over pieces costs registers that the others need); where full examples
// already would be too far apart, a tile takes rows of one example only
// (`packed` = 0: rows t0 .. of example i, blocks of 256 or 128).
// Partial sums go to fp64 workspace slots and are reduced in a fixed order.

#include "tile256.h"

namespace dr {
namespace {

constexpr int kSThreads = 256;
constexpr int kST = 128;                  // tile rows / columns
constexpr int kSK = 64;                   // reduction step (one 128-byte row)
constexpr int kSPanel = kST * kSK * 2;    // 16 KB

__device__ __forceinline__ int clamp_len(const int* len, int i, int T) {
  int L = len ? len[i] : T;
  return L < 0 ? 0 : (L > T ? T : L);
}

// Row panel of one operand: this lane's four rows (half blocks w, w+4,
// w+8, w+12 of the 128-row panel) as byte offsets, or kOobOffset.
struct PanelRows {
  unsigned off[4];
  int seg[4];
};

__device__ __forceinline__ void issue_panel(__amdgpu_buffer_rsrc_t rs, const PanelRows& pr, unsigned char* dst, int w,
                                            int k0, int K) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int col = k0 + 8 * pr.seg[u];
    const unsigned o = (pr.off[u] == kOobOffset || col >= K) ? kOobOffset : pr.off[u] + (unsigned)(col * 2);
    dma16<kAuxCached>(rs, dst + (w + 4 * u) * 1024, o);
  }
}

// acc[i][j] += A[64 wr + 16 i + .][k] B[64 wc + 16 j + .][k] over k < K for
// NB B panels (summed), A and B given as row panels
template <int NB>
__device__ __forceinline__ void panel_gemm(unsigned char* lds, __amdgpu_buffer_rsrc_t ra, const PanelRows& pa,
                                           const __amdgpu_buffer_rsrc_t (&rb)[NB], const PanelRows& pb, int K,
                                           f32x4 (&acc)[4][4]) {
  constexpr int kStage = (1 + NB) * kSPanel;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1, lr = lane & 15, lg = lane >> 4;
  const int nk = (K + kSK - 1) / kSK;
  auto issue = [&](int t, int st) {
    unsigned char* sb = lds + st * kStage;
    issue_panel(ra, pa, sb, w, t * kSK, K);
#pragma unroll
    for (int b = 0; b < NB; ++b) issue_panel(rb[b], pb, sb + (1 + b) * kSPanel, w, t * kSK, K);
  };
  issue(0, 0);
  for (int t = 0; t < nk; ++t) {
    DR_WAIT_VM(0);
    DR_LDS_SYNC();
    if (t + 1 < nk) issue(t + 1, (t + 1) & 1);
    const unsigned char* sa = lds + (t & 1) * kStage;
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {
      const int seg = 4 * kh + lg;
      u32x4 fa[4], fb[NB][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i] = swz_read(sa + (4 * wr + i) * 2048, lr, seg);
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) fb[b][j] = swz_read(sa + (1 + b) * kSPanel + (4 * wc + j) * 2048, lr, seg);
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = mma_bf16(fa[i], fb[b][j], acc[i][j]);
    }
  }
  DR_LDS_SYNC();   // the ring is free for the next use
}

constexpr int kMaxScoreLayers = 16;

struct ScoreLayer {
  const unsigned char* x;
  const unsigned char* dy;
  long long ldx, lddy;       // elements per token
  long long exx, exdy;       // bytes per example
  const unsigned char* ghi;  // PIP: gbar* as bf16 hi + lo, [d_out][d_in]
  const unsigned char* glo;
  double* part;              // partial sums of this layer
  int d_in, d_out;
  int OB;                    // PIP: 256-column blocks of d_out (128 in pip_small_kernel)
};

struct ScoreArgs {
  ScoreLayer L[kMaxScoreLayers];
  int num_layers;
  int T, n, m;
  int packed;                // rows of a tile: packed positions, or one example's tokens
  int span;                  // packed: examples (empty ones too) that 32-bit offsets reach
  int SB;                    // GIP: 128-row blocks of the target tokens (upper bound)
  const int* len;            // [n + m] or null
  const int* cum;            // [n + 1] token prefix of the general examples, then [m + 1] of the targets
};

// Tile of this workgroup: workgroup b (of a grid of kGridX columns) runs on
// XCD b % 8, which takes runs of 32 tiles.
constexpr int64_t kGridX = (int64_t)1 << 22;    // a launch takes fewer than 2^32 threads per dimension,
constexpr int64_t kGridY = 65535;               // and as many rows
__device__ __forceinline__ long long tile_index() {
  const long long sl = (long long)blockIdx.y * (gridDim.x >> 3) + (blockIdx.x >> 3);
  return ((sl >> 5) * 8 + (blockIdx.x & 7)) * 32 + (sl & 31);
}

// exclusive prefixes of the clamped lengths: block 0 the n general examples,
// block 1 the m targets
__global__ __launch_bounds__(1024) void score_plan_kernel(const int* len, int n, int m, int T, int* cum) {
  __shared__ int wsum[17];
  const int first = blockIdx.x ? n : 0, cnt = blockIdx.x ? m : n;
  int* out = cum + (blockIdx.x ? n + 1 : 0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (cnt + 1023) / 1024;
  const int i0 = tid * per < cnt ? tid * per : cnt, i1 = i0 + per < cnt ? i0 + per : cnt;
  int loc = 0;
  for (int i = i0; i < i1; ++i) loc += clamp_len(len, first + i, T);
  int inc = loc;
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(inc, off, 64);
    if (lane >= off) inc += v;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int w = 0; w < 16; ++w) {
      const int v = wsum[w];
      wsum[w] = run;
      run += v;
    }
    wsum[16] = run;
  }
  __syncthreads();
  int base = wsum[wave] + inc - loc;
  for (int i = i0; i < i1; ++i) {
    out[i] = base;
    base += clamp_len(len, first + i, T);
  }
  if (tid == 0) out[cnt] = wsum[16];
}

// Rows of a tile of ROWS rows: example (relative to e0) and token of each, in LDS.
template <int ROWS>
struct TileRows {
  int cum[ROWS + 1];   // cum[e0 + r] - p0
  int rel[ROWS];       // -1 past the last row
  int tok[ROWS];
};

// position past the last row of row block rt
template <int ROWS>
__device__ __forceinline__ int block_end(const int* cum, int cnt, int rt) {
  const int total = cum[cnt], p0 = rt * ROWS;
  return total - p0 < ROWS ? total : p0 + ROWS;
}

// Fills the table for row block rt of `cnt` examples with prefix `cum`, from
// position p0 of the block on (packed) as far as `span` examples reach: a
// whole 256-thread workgroup; ends with a barrier.  Returns the number of
// valid rows; e0: the example of the first row, e_last: of the last.
template <bool PIECES, int ROWS>
__device__ __forceinline__ int tile_rows(TileRows<ROWS>& tr, const int* cum, const int* len, int first, int cnt, int T,
                                         int packed, int span, int rt, int p0, int& e0, int& e_last) {
  const int tid = threadIdx.x;
  if (!packed) {
    const int TB = (T + ROWS - 1) / ROWS;
    e0 = e_last = rt / TB;
    const int t0 = (rt - e0 * TB) * ROWS, L = clamp_len(len, first + e0, T);
    for (int r = tid; r < ROWS; r += 256) {
      tr.rel[r] = t0 + r < L ? 0 : -1;
      tr.tok[r] = t0 + r;
    }
    if (tid == 0) {
      tr.cum[0] = 0;
      tr.cum[1] = L - t0;
    }
    __syncthreads();
    return L - t0 < ROWS ? L - t0 : ROWS;
  }
  int lo = 0, hi = cnt;   // the last example with cum <= p0 (not empty: p0 is below the total)
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cum[mid] <= p0) lo = mid;
    else hi = mid - 1;
  }
  e0 = lo;
  int end = block_end<ROWS>(cum, cnt, rt);
  if (PIECES && e0 + span < cnt) {
    const int reach = cum[e0 + span];
    end = reach < end ? reach : end;
  }
  const int rows = end - p0;
  // at most ROWS non-empty examples; runs of empty ones can only push an
  // example past the staged prefix, which is then read from memory
  for (int r = tid; r <= ROWS; r += 256) tr.cum[r] = e0 + r <= cnt ? cum[e0 + r] - p0 : 0x7fffffff;
  __syncthreads();
  for (int r = tid; r < ROWS; r += 256) {
    int e = 0, t = 0;
    if (r < rows) {
      while ((e + 1 <= ROWS ? tr.cum[e + 1] : cum[e0 + e + 1] - p0) <= r) ++e;
      t = r - (e <= ROWS ? tr.cum[e] : cum[e0 + e] - p0);
    }
    tr.rel[r] = r < rows ? e : -1;
    tr.tok[r] = t;
  }
  __syncthreads();
  e_last = e0 + tr.rel[rows - 1];
  return rows;
}

// row sums of a tile (rs[h][row], two column halves) -> one partial per
// example of the tile, in slot (row block + example) of a column block: the
// pairs (row block, example) in order step at least one of the two, so the
// slots are distinct (row block alone when it holds rows of one example);
// p0: position of the tile's first row
template <int ROWS>
__device__ __forceinline__ void tile_example_sums(const TileRows<ROWS>& tr, const double (*rs)[ROWS], const int* cum,
                                                  int rows, int packed, int rt, int p0, int e0, int e_last,
                                                  double* part, int stride, int col) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int e = e0 + w; e <= e_last; e += 4) {
    const int r = e - e0;
    int lo = r <= ROWS ? tr.cum[r] : cum[e] - p0, hi = r + 1 <= ROWS ? tr.cum[r + 1] : cum[e + 1] - p0;
    lo = lo > 0 ? lo : 0;
    hi = hi < rows ? hi : rows;
    if (lo >= hi) continue;   // an empty example
    double v = 0.0;
    for (int k = lo + lane; k < hi; k += 64) v += rs[0][k] + rs[1][k];
    v = wave_sum_l63(v);
    if (lane == 63) part[(long long)(packed ? rt + e : rt) * stride + col] = v;
  }
}

// ---------------------------------------------------------------- PIP

// row block rt of 256 tokens x column block ob of 256 outputs of one layer:
// the products of the tokens with gbar* (2 d_in columns: hi and lo of each
// 64-column step in turn), dotted with the dy rows.  Bound by the MFMA rate:
// 2.3 ms for the small block's 2.75 TFLOP (64 examples of 128..512 tokens,
// eight 2048 x 2048 layers), 1.2 PFLOP/s.  128 x 128 tiles of one example
// with both parts of gbar* staged (one workgroup of 96 KB per CU, its DMA
// waited for at every fragment read) took 0.92 ms per layer.  Whole call
// 8.03 -> 2.55 ms.
template <bool PIECES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void pip_kernel(ScoreArgs a) {
  // one LDS object: beside a second one the compiler makes every fragment
  // read wait for all DMA in flight (7.9 instead of 1.9 ms on the small block)
  __shared__ __attribute__((aligned(1024))) unsigned char
      lds[kTileRing + 2 * kTileRows * sizeof(double) + sizeof(TileRows<kTileRows>)];
  double (*rs)[kTileRows] = reinterpret_cast<double (*)[kTileRows]>(lds + kTileRing);
  TileRows<kTileRows>& tr = *reinterpret_cast<TileRows<kTileRows>*>(lds + kTileRing + 2 * kTileRows * sizeof(double));
  const int R = a.packed ? (a.cum[a.n] + kTileRows - 1) / kTileRows : a.n * ((a.T + kTileRows - 1) / kTileRows);
  // each XCD takes runs of 32 tiles: eight column blocks of four row blocks,
  // whose panels its L2 then holds
  long long q = tile_index();
  int li = 0;
  while (li < a.num_layers && q >= (long long)R * a.L[li].OB) {
    q -= (long long)R * a.L[li].OB;
    ++li;
  }
  if (li == a.num_layers) return;
  const ScoreLayer& L = a.L[li];
  const int band = (int)(q / ((long long)R * 8));
  const int wb = L.OB - 8 * band < 8 ? L.OB - 8 * band : 8;
  const int qb = (int)(q - (long long)band * R * 8);
  const int rt = qb / wb, ob = 8 * band + qb % wb;
  if (!a.packed) {
    const int TB = (a.T + kTileRows - 1) / kTileRows, i = rt / TB;
    if ((rt - i * TB) * kTileRows >= clamp_len(a.len, i, a.T)) return;
  }
  for (int p0 = rt * kTileRows, rows;; p0 += rows) {   // one turn, or one per piece
  int e0, e_last;
  rows = tile_rows<PIECES>(tr, a.cum, a.len, 0, a.n, a.T, a.packed, a.span, rt, p0, e0, e_last);
  const int o0 = ob * kTileRows;
  const int d_in = L.d_in, d_out = L.d_out;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1;   // 128-token half, 128-output half
  const int lr = lane & 15, lg = lane >> 4;
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(L.x + (long long)e0 * L.exx, kOobOffset);
  const __amdgpu_buffer_rsrc_t rh = make_rsrc(L.ghi + (long long)o0 * d_in * 2, kOobOffset);
  const __amdgpu_buffer_rsrc_t rl = make_rsrc(L.glo + (long long)o0 * d_in * 2, kOobOffset);
  unsigned offA[8], offB[8];
  int segs[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int hb = w + 4 * u;             // half block: rows 8 hb .. 8 hb + 7
    const int r = 8 * hb + (lane >> 3);
    segs[u] = 8 * swz_seg_of_lane(lane, hb & 1);
    const int rel = tr.rel[r];
    offA[u] = rel >= 0 ? (unsigned)(rel * L.exx + tr.tok[r] * L.ldx * 2) : kOobOffset;
    offB[u] = o0 + r < d_out ? (unsigned)((long long)r * d_in * 2) : kOobOffset;
  }
  auto dma1 = [&](int t, int st, int q) {
    unsigned char* sb = lds + st * kTileStage;
    const int u = q >> 1;
    const int col = (t >> 1) * kTileStepCols + segs[u];
    const bool cok = col < d_in;
    if (q & 1) {
      const unsigned cb = (offB[u] == kOobOffset || !cok) ? kOobOffset : offB[u] + (unsigned)(col * 2);
      dma16<kAuxCached>(t & 1 ? rl : rh, sb + kTilePanel + (w + 4 * u) * 1024, cb);
    } else {
      const unsigned ca = (offA[u] == kOobOffset || !cok) ? kOobOffset : offA[u] + (unsigned)(col * 2);
      dma16<kAuxCached>(ra, sb + (w + 4 * u) * 1024, ca);
    }
  };
  auto rd1 = [&](u32x4* fa, u32x4* fb, const unsigned char* sa, int kh, int q) {
    const int seg = 4 * kh + lg;
    if (q & 1) fb[q >> 1] = swz_read(sa + kTilePanel + (wc * 8 + (q >> 1)) * 2048, lr, seg);
    else fa[q >> 1] = swz_read(sa + (wr * 8 + (q >> 1)) * 2048, lr, seg);
  };
  f32x4 acc[8][8];
  tile256_clear(acc);
  tile256_loop(lds, 2 * ((d_in + kTileStepCols - 1) / kTileStepCols), dma1, rd1, acc);
  // Dot with the dy rows of the tile: the whole tile (256 rows x 512 bytes)
  // goes into the ring by DMA, in the slot order of slot_xor, and the
  // transposing LDS read gives each lane its column of the four rows that one
  // accumulator register quad holds (2-byte loads from memory in that layout
  // took 0.75 ms of 3.2 on the small block).
  DR_WAIT_VM(0);
  DR_LDS_SYNC();   // every wave is done with the ring
  const __amdgpu_buffer_rsrc_t rd = make_rsrc(L.dy + (long long)e0 * L.exdy + o0 * 2LL, kOobOffset);
#pragma unroll 8
  for (int h = 0; h < 32; ++h) {
    const int blk = w + 4 * h, r = 2 * blk + (lane >> 5), u = lane & 31;
    const int col = 16 * ((u >> 1) ^ slot_xor(r)) + 8 * (u & 1);
    const int rel = tr.rel[r];
    dma16<kAuxCached>(rd, lds + blk * 1024,
                      rel >= 0 && o0 + col < d_out
                          ? (unsigned)(rel * L.exdy + tr.tok[r] * L.lddy * 2 + col * 2) : kOobOffset);
  }
  DR_WAIT_VM(0);
  DR_LDS_SYNC();
  const int dq = (lane >> 2) & 3, dr = lane & 3;
  const bool full = o0 + kTileRows <= d_out;
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    const int rrow = wr * 128 + 16 * p + 4 * lg + dq;   // the row this lane addresses
    float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const v4s v = lds_read_tr16(lds + rrow * 512 + (((wc * 8 + j) ^ slot_xor(rrow)) * 32) + dr * 8);
      const bool ok = full || o0 + wc * 128 + 16 * j + lr < d_out;   // else zeros against any product
#pragma unroll
      for (int r = 0; r < 4; ++r)
        d[r] = ok ? fmaf(acc[p][j][r], __uint_as_float((unsigned)(unsigned short)v[r] << 16), d[r]) : d[r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double s = (double)d[r];
      s += dpp_d<0xB1, 0xF>(s);
      s += dpp_d<0x4E, 0xF>(s);
      s += dpp_d<0x141, 0xF>(s);
      s += dpp_d<0x140, 0xF>(s);
      if (lr == 0) rs[wc][wr * 128 + 16 * p + 4 * lg + r] = s;
    }
  }
  __syncthreads();
  tile_example_sums(tr, rs, a.cum, rows, a.packed, rt, p0, e0, e_last, L.part, L.OB, ob);
  if (!PIECES || p0 + rows >= block_end<kTileRows>(a.cum, a.n, rt)) break;
  __syncthreads();   // the next piece's table
  }
}

// row panel of a tile's token rows
__device__ __forceinline__ PanelRows token_panel(const TileRows<kST>& t, long long ex, long long ld) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  PanelRows p;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int hb = w + 4 * u;
    const int r = 8 * hb + (lane >> 3);
    p.seg[u] = swz_seg_of_lane(lane, hb & 1);
    const int rel = t.rel[r];
    p.off[u] = rel >= 0 ? (unsigned)(rel * ex + t.tok[r] * ld * 2) : kOobOffset;
  }
  return p;
}

// The same in tiles of 128 rows of one example x 128 outputs, both parts of
// gbar* staged beside the tokens, where there are too few tiles of either size
// to fill the chip: a tile's own time then counts, and one of 256 x 256 takes
// longer (the whole call, one layer 1024 x 1024, 16 examples of 128 tokens: 61
// us, 92 in 256 x 256 tiles; one of 4096 x 4096, one example of 512: 147, 239).
__global__ __launch_bounds__(kSThreads) void pip_small_kernel(ScoreArgs a) {
  constexpr int kRing = 2 * 3 * kSPanel;
  __shared__ __attribute__((aligned(1024))) unsigned char
      lds[kRing + 2 * kST * sizeof(double) + sizeof(TileRows<kST>)];   // one LDS object, as in pip_kernel
  double (*rs)[kST] = reinterpret_cast<double (*)[kST]>(lds + kRing);
  TileRows<kST>& tr = *reinterpret_cast<TileRows<kST>*>(lds + kRing + 2 * kST * sizeof(double));
  const int TB = (a.T + kST - 1) / kST, R = a.n * TB;
  int q = blockIdx.x, li = 0;
  while (li < a.num_layers && q >= R * a.L[li].OB) {
    q -= R * a.L[li].OB;
    ++li;
  }
  if (li == a.num_layers) return;
  const ScoreLayer& L = a.L[li];
  const int rt = q / L.OB, ob = q - rt * L.OB, o0 = ob * kST;
  if ((rt % TB) * kST >= clamp_len(a.len, rt / TB, a.T)) return;
  int e0, e_last;
  const int rows = tile_rows<false>(tr, a.cum, a.len, 0, a.n, a.T, 0, a.span, rt, 0, e0, e_last);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1, lr = lane & 15, lg = lane >> 4;
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(L.x + (long long)e0 * L.exx, kOobOffset);
  const __amdgpu_buffer_rsrc_t rb[2] = {make_rsrc(L.ghi + (long long)o0 * L.d_in * 2, kOobOffset),
                                        make_rsrc(L.glo + (long long)o0 * L.d_in * 2, kOobOffset)};
  PanelRows pb;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int hb = w + 4 * u, r = 8 * hb + (lane >> 3);
    pb.seg[u] = swz_seg_of_lane(lane, hb & 1);
    pb.off[u] = o0 + r < L.d_out ? (unsigned)((long long)r * L.d_in * 2) : kOobOffset;
  }
  f32x4 acc[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[p][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  panel_gemm<2>(lds, ra, token_panel(tr, L.exx, L.ldx), rb, pb, L.d_in, acc);
  // dot with the dy rows of the tile (valid tokens and outputs only)
  const __bf16* dyb = reinterpret_cast<const __bf16*>(L.dy + (long long)e0 * L.exdy) + o0;
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 64 * wr + 16 * p + 4 * lg + r;
      float d = 0.f;
      if (row < rows) {
        const __bf16* dyr = dyb + (long long)tr.tok[row] * L.lddy;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int o = 64 * wc + 16 * j + lr;
          if (o0 + o < L.d_out) d = fmaf(acc[p][j][r], (float)dyr[o], d);
        }
      }
      double v = (double)d;
      v += dpp_d<0xB1, 0xF>(v);
      v += dpp_d<0x4E, 0xF>(v);
      v += dpp_d<0x141, 0xF>(v);
      v += dpp_d<0x140, 0xF>(v);
      if (lr == 0) rs[wc][row] = v;
    }
  __syncthreads();
  tile_example_sums(tr, rs, a.cum, rows, 0, rt, 0, e0, e_last, L.part, L.OB, ob);
}

// s[l][i] = scale * the sum of the example's partials over its row blocks
// (in order) and the nc column blocks of each, one wave per (layer, example);
// OBS: the layer's own column count
template <int ROWS, bool OBS>
__global__ __launch_bounds__(256) void score_reduce_kernel(ScoreArgs a, float* s, double scale) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), l = blockIdx.y, lane = threadIdx.x & 63;
  if (i >= a.n) return;
  const int len = clamp_len(a.len, i, a.T);
  int stride, nc;   // columns of a slot, and those written
  if (OBS) {
    stride = nc = a.L[l].OB;
  } else {
    stride = a.SB;
    nc = a.SB;
    if (a.packed) nc = (a.cum[a.n + 1 + a.m] + ROWS - 1) / ROWS;
  }
  const int TB = (a.T + ROWS - 1) / ROWS;
  int b0, nb;   // first slot, and how many
  if (a.packed) {
    b0 = a.cum[i] / ROWS + i;
    nb = len > 0 ? (a.cum[i] + len - 1) / ROWS - a.cum[i] / ROWS + 1 : 0;
  } else {
    b0 = i * TB;
    nb = (len + ROWS - 1) / ROWS;
  }
  const double* p = a.L[l].part + (long long)b0 * stride;
  double t = 0.0;
  for (long long k = lane; k < (long long)nb * nc; k += 64) {
    const int blk = (int)(k / nc), c = (int)(k - (long long)blk * nc);
    if (!OBS && !a.packed) {   // column blocks past a target's length hold nothing
      const int j = c / TB;
      if ((c - j * TB) * ROWS >= clamp_len(a.len, a.n + j, a.T)) continue;
    }
    t += p[(long long)blk * stride + c];
  }
  t = wave_sum_l63(t);
  if (lane == 63) s[(long long)l * a.n + i] = (float)(t * scale);
}

// gbar* (fp32) -> bf16 hi + lo (hi = RNE(g), lo = RNE(g - hi))
__global__ void split_kernel(const float* g, long long count, __bf16* hi, __bf16* lo) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  const float v = g[e];
  const __bf16 h = (__bf16)v;
  hi[e] = h;
  lo[e] = (__bf16)(v - (float)h);
}

// ---------------------------------------------------------------- GIP

// 128 general tokens x 128 target tokens of one layer: the row sums of
// (D D*^T) .* (X X*^T).  Rows and columns are packed tokens, so the tile count
// follows the valid tokens (with one tile per pair of examples, 64 examples
// of 32..128 tokens against 8 targets filled 39 % of the products: whole call
// over eight 2048 x 2048 layers 0.67 -> 0.26 ms, all layers in one launch).
template <bool PIECES>
__global__ __launch_bounds__(kSThreads, 2) void gip_kernel(ScoreArgs a) {
  constexpr int kRing = 2 * 2 * kSPanel;
  __shared__ __attribute__((aligned(1024))) unsigned char
      lds[kRing + 2 * kST * sizeof(double) + 2 * sizeof(TileRows<kST>)];   // one LDS object, as in pip_kernel
  double (*rs)[kST] = reinterpret_cast<double (*)[kST]>(lds + kRing);
  TileRows<kST>& tr = *reinterpret_cast<TileRows<kST>*>(lds + kRing + 2 * kST * sizeof(double));
  TileRows<kST>& tc = *(&tr + 1);
  const int TB = (a.T + kST - 1) / kST;
  const int R = a.packed ? (a.cum[a.n] + kST - 1) / kST : a.n * TB;
  const int C = a.packed ? (a.cum[a.n + 1 + a.m] + kST - 1) / kST : a.m * TB;
  // (the column blocks of a row block next to each other)
  long long q = tile_index();
  const long long per = (long long)R * C;
  if (per == 0) return;
  const int li = (int)(q / per);
  if (li >= a.num_layers) return;
  q -= li * per;
  const int rt = (int)(q / C), sb = (int)(q - (long long)rt * C);
  const ScoreLayer& L = a.L[li];
  if (!a.packed) {
    const int i = rt / TB, j = sb / TB;
    if ((rt - i * TB) * kST >= clamp_len(a.len, i, a.T) || (sb - j * TB) * kST >= clamp_len(a.len, a.n + j, a.T)) return;
  }
  const int* tcum = a.cum + a.n + 1;   // the targets' prefix
  for (int p0 = rt * kST, rows;; p0 += rows) {   // one turn each, or one per piece
  int e0, e_last, f0, f_last;
  rows = tile_rows<PIECES>(tr, a.cum, a.len, 0, a.n, a.T, a.packed, a.span, rt, p0, e0, e_last);
  for (int c0 = sb * kST, cols;; c0 += cols) {
  cols = tile_rows<PIECES>(tc, tcum, a.len, a.n, a.m, a.T, a.packed, a.span, sb, c0, f0, f_last);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1, lr = lane & 15, lg = lane >> 4;
  f32x4 dd[4][4], xx[4][4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      dd[p][q4] = f32x4{0.f, 0.f, 0.f, 0.f};
      xx[p][q4] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  {
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(L.dy + (long long)e0 * L.exdy, kOobOffset);
    const __amdgpu_buffer_rsrc_t rb[1] = {make_rsrc(L.dy + (long long)(a.n + f0) * L.exdy, kOobOffset)};
    panel_gemm<1>(lds, ra, token_panel(tr, L.exdy, L.lddy), rb, token_panel(tc, L.exdy, L.lddy), L.d_out, dd);
  }
  {
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(L.x + (long long)e0 * L.exx, kOobOffset);
    const __amdgpu_buffer_rsrc_t rb[1] = {make_rsrc(L.x + (long long)(a.n + f0) * L.exx, kOobOffset)};
    panel_gemm<1>(lds, ra, token_panel(tr, L.exx, L.ldx), rb, token_panel(tc, L.exx, L.ldx), L.d_in, xx);
  }
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float d = 0.f;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        d = 64 * wc + 16 * q4 + lr < cols ? fmaf(dd[p][q4][r], xx[p][q4][r], d) : d;
      double v = (double)d;
      v += dpp_d<0xB1, 0xF>(v);
      v += dpp_d<0x4E, 0xF>(v);
      v += dpp_d<0x141, 0xF>(v);
      v += dpp_d<0x140, 0xF>(v);
      if (lr == 0) {
        double& sum = rs[wc][64 * wr + 16 * p + 4 * lg + r];
        sum = !PIECES || c0 == sb * kST ? v : sum + v;
      }
    }
  if (!PIECES || c0 + cols >= block_end<kST>(tcum, a.m, sb)) break;
  }
  __syncthreads();
  tile_example_sums(tr, rs, a.cum, rows, a.packed, rt, p0, e0, e_last, L.part, a.SB, sb);
  if (!PIECES || p0 + rows >= block_end<kST>(a.cum, a.n, rt)) break;
  __syncthreads();   // the next piece's table
  }
}

__global__ void fill_kernel(float* p, long long count, float v) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) p[e] = v;
}

// ---------------------------------------------------------------- host

struct ScorePlan {
  double tiles;   // of the largest launch (upper bound)
  size_t off_wm, off_g, off_upd, off_hi, off_lo, off_cum, off_part, off_direct, bytes;
};

// Few tiles: with one round of workgroups, and each on rows of one example,
// there is nothing to gain from packing the tokens (nor a prefix to form), and
// PIP takes the smaller tiles: up to one 128 x 128 tile per CU, at T tokens an
// example.  (GIP of 512 tiles, two per CU, gains from packing ragged lengths:
// one layer 4096 x 14336, 4 x 2 examples of T = 1024, 193 us packed, 221 not.)
constexpr double kSmallTiles = 256.0;
bool score_small(const dr_layer* layers, int num_layers, int64_t n, int64_t m, int64_t T, int method) {
  if (method == DR_SCORE_DIRECT) return false;
  const double TB = (double)((T + kST - 1) / kST);
  double tiles = 0.0;
  for (int l = 0; l < num_layers; ++l)
    tiles += (double)n * TB * (method == DR_SCORE_PIP ? (double)((layers[l].d_out + kST - 1) / kST) : (double)m * TB);
  return tiles <= kSmallTiles;
}

// rows of a tile
int64_t score_rows(int method, bool small) { return method == DR_SCORE_PIP && !small ? kTileRows : kST; }

// 128-token column blocks of the m targets (upper bound)
int64_t gip_cols(int64_t m, int64_t T, bool packed) {
  return packed ? (m * T + kST - 1) / kST : m * ((T + kST - 1) / kST);
}

// row blocks over n examples (the most that the lengths allow)
int64_t row_blocks(int64_t n, int64_t T, int64_t rows, bool packed) {
  return packed ? (n * T + rows - 1) / rows : n * ((T + rows - 1) / rows);
}

// (row block, example) slots
int64_t score_slots(int64_t n, int64_t T, int64_t rows, bool packed) {
  return row_blocks(n, T, rows, packed) + (packed ? n : 0);
}

// Layers are taken in groups of at most kMaxScoreLayers consecutive ones: a
// group's gbar* are assembled in one call and its tiles share one launch, so
// that the last round of tiles is a small part of it (eight 2048 x 2048
// layers one at a time: 2.4 rounds of the chip each).  A group's gbar* hold
// at most kGroupElems elements (256 MiB of workspace for PIP), its GIP
// partials, which go with the tokens of both sides, kGroupPartials (256 MiB
// again); or it is one layer.
constexpr int64_t kGroupElems = (int64_t)32 << 20, kGroupPartials = (int64_t)32 << 20;

int group_end(const dr_layer* layers, int num_layers, int first, int64_t n, int64_t m, int64_t T, int method) {
  int64_t g = 0;
  int most = kMaxScoreLayers;
  if (method == DR_SCORE_GIP) {
    double part = 1.0;   // of a layer
    for (int packed = 0; packed < 2; ++packed) {
      const double p = (double)score_slots(n, T, kST, packed) * (double)gip_cols(m, T, packed);
      part = p > part ? p : part;
    }
    const double fit = (double)kGroupPartials / part;
    most = fit >= most ? most : (fit < 1.0 ? 1 : (int)fit);
  }
  int l = first;
  for (; l < num_layers && l - first < most; ++l) {
    g += layers[l].d_out * layers[l].d_in;
    if (method != DR_SCORE_GIP && l > first && g > kGroupElems) break;
  }
  return l;
}

// examples whose rows a 32-bit offset from the first one reaches
int64_t score_span(const dr_layer* layers, int num_layers, int64_t T) {
  int64_t span = (int64_t)1 << 24;
  for (int l = 0; l < num_layers && T > 0; ++l) {
    const int64_t ld = layers[l].ldx > layers[l].lddy ? layers[l].ldx : layers[l].lddy;
    const int64_t e = ((int64_t)kOobOffset - 64) / (T * ld * 2);
    span = e < span ? e : span;
  }
  return span;
}

// Packed tiles address a tile's rows from its first example with 32-bit
// offsets, and positions are 32-bit: possible when the full examples that one
// tile can hold span less than 4 GiB (with empty ones between them the tile is
// taken in pieces).
bool score_packed(const dr_layer* layers, int num_layers, int64_t n, int64_t m, int64_t T, int64_t rows) {
  const int64_t most = n > m ? n : m;
  if (most * T >= ((int64_t)1 << 31) - 2 * rows) return false;
  return score_span(layers, num_layers, T) >= (most < rows ? most : rows);
}

dr_layer target_layer(const dr_layer& L, int64_t n, int64_t T) {
  dr_layer t = L;
  t.x = static_cast<const unsigned char*>(L.x) + n * T * L.ldx * 2;
  t.dy = static_cast<const unsigned char*>(L.dy) + n * T * L.lddy * 2;
  return t;
}

ScorePlan score_plan(const dr_layer* layers, int num_layers, int64_t n, int64_t m, int64_t T, int method) {
  int64_t gmax = 1, partmax = 1;
  double tiles = 0.0;
  size_t updmax = 0, dirmax = 0;
  dr_layer t[kMaxScoreLayers];
  for (int l0 = 0; l0 < num_layers;) {
    const int l1 = group_end(layers, num_layers, l0, n, m, T, method);
    const bool small = score_small(layers + l0, l1 - l0, n, m, T, method);
    const int64_t rows = score_rows(method, small);
    const bool packed = !small && score_packed(layers + l0, l1 - l0, n, m, T, rows);
    const int64_t slots = score_slots(n, T, rows, packed);
    int64_t g = 0, cols = 0;
    for (int l = l0; l < l1; ++l) {
      g += layers[l].d_out * layers[l].d_in;
      t[l - l0] = target_layer(layers[l], n, T);
      cols += method == DR_SCORE_PIP ? (layers[l].d_out + rows - 1) / rows : gip_cols(m, T, packed);
    }
    const int64_t part = slots * cols;
    gmax = g > gmax ? g : gmax;
    partmax = part > partmax ? part : partmax;
    const double nt = (double)row_blocks(n, T, rows, packed) * cols;
    if (method != DR_SCORE_DIRECT) tiles = nt > tiles ? nt : tiles;
    if (method != DR_SCORE_GIP) {
      const size_t u = dr_update_workspace_size(t, l1 - l0, m, T, DR_BF16);
      updmax = u > updmax ? u : updmax;
    }
    if (method == DR_SCORE_DIRECT) {
      for (int l = l0; l < l1; ++l) {
        const size_t d = direct_workspace(layers + l, 1, n);
        dirmax = d > dirmax ? d : dirmax;
      }
    }
    l0 = l1;
  }
  ScorePlan p;
  p.tiles = tiles;
  size_t o = 0;
  p.off_wm = o;     o = align_up(o + (size_t)(m > 0 ? m : 1) * 4, 256);
  p.off_g = o;      if (method != DR_SCORE_GIP) o = align_up(o + (size_t)gmax * 4, 256);
  p.off_upd = o;    if (method != DR_SCORE_GIP) o = align_up(o + updmax, 256);
  p.off_hi = o;     if (method == DR_SCORE_PIP) o = align_up(o + (size_t)gmax * 2, 256);
  p.off_lo = o;     if (method == DR_SCORE_PIP) o = align_up(o + (size_t)gmax * 2, 256);
  p.off_cum = o;    if (method != DR_SCORE_DIRECT) o = align_up(o + (size_t)(n + m + 2) * 4, 256);
  p.off_part = o;   if (method != DR_SCORE_DIRECT) o = align_up(o + (size_t)partmax * 8, 256);
  p.off_direct = o; if (method == DR_SCORE_DIRECT) o = align_up(o + dirmax, 256);
  p.bytes = o;
  return p;
}

dr_status validate_score(const dr_layer* layers, int num_layers, int64_t n, int64_t m, int64_t T, dr_dtype dtype,
                         int method, const float* s) {
  if (dtype != DR_BF16 && dtype != DR_F32) return DR_ERR_DTYPE;
  if (dtype != DR_BF16) return DR_ERR_UNSUPPORTED;
  if (method != DR_SCORE_DIRECT && method != DR_SCORE_GIP && method != DR_SCORE_PIP) return DR_ERR_ARG;
  if (!layers || num_layers < 1 || n < 0 || m < 1 || T < 0) return DR_ERR_ARG;
  if (n + m > (1 << 24) || T > (1 << 20)) return DR_ERR_ARG;
  if (n > 0 && !s) return DR_ERR_ARG;
  for (int l = 0; l < num_layers; ++l) {
    const dr_layer& L = layers[l];
    if (L.d_in < 1 || L.d_out < 1 || L.d_in % 8 || L.d_out % 8) return DR_ERR_ARG;
    if (L.d_in > (1 << 28) || L.d_out > (1 << 28)) return DR_ERR_ARG;
    if (L.ldx < L.d_in || L.lddy < L.d_out || L.ldx % 8 || L.lddy % 8) return DR_ERR_ARG;
    if (T > 0 && (!L.x || !L.dy || !aligned16(L.x) || !aligned16(L.dy))) return DR_ERR_ARG;
    if (T * L.ldx * 2 >= (int64_t)kOobOffset - 64 || T * L.lddy * 2 >= (int64_t)kOobOffset - 64)
      return DR_ERR_UNSUPPORTED;
    if (L.d_out * L.d_in * 2 >= (int64_t)kOobOffset - 64) return DR_ERR_UNSUPPORTED;
  }
  return DR_OK;
}

}  // namespace
}  // namespace dr

extern "C" size_t dr_score_workspace_size(const dr_layer* layers, int num_layers, int64_t n, int64_t m, int64_t T,
                                          dr_dtype dtype, dr_score_method method) {
  if (!layers || num_layers < 1 || n < 0 || m < 1 || T < 0 || dtype != DR_BF16) return 0;
  for (int l = 0; l < num_layers; ++l)
    if (layers[l].d_in < 1 || layers[l].d_out < 1) return 0;
  return dr::score_plan(layers, num_layers, n, m, T, (int)method).bytes;
}

extern "C" dr_status dr_score_exact(const dr_layer* layers, int num_layers, int64_t n, int64_t m, int64_t T,
                                    const int32_t* len, dr_dtype dtype, dr_score_method method, float* s,
                                    void* workspace, size_t ws_bytes, void* stream) {
  using namespace dr;
  dr_status st = validate_score(layers, num_layers, n, m, T, dtype, (int)method, s);
  if (st != DR_OK) return st;
  const ScorePlan pl = score_plan(layers, num_layers, n, m, T, (int)method);
  if (pl.tiles > (double)(kGridX * kGridY)) return DR_ERR_UNSUPPORTED;
  if (!workspace || ws_bytes < pl.bytes) return DR_ERR_WORKSPACE;
  if (n == 0) return DR_OK;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  float* wm = reinterpret_cast<float*>(ws + pl.off_wm);
  float* gstar = reinterpret_cast<float*>(ws + pl.off_g);
  if (method != DR_SCORE_GIP) {
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, hs, wm, (long long)m,
                       1.0f / (float)m);
    if ((st = launch_status()) != DR_OK) return st;
  }
  int* cum = reinterpret_cast<int*>(ws + pl.off_cum);
  bool planned = false;
  for (int l0 = 0; l0 < num_layers;) {
    const int l1 = group_end(layers, num_layers, l0, n, m, T, (int)method), cnt = l1 - l0;
    float* sl = s + (int64_t)l0 * n;
    int64_t goff[kMaxScoreLayers + 1] = {0};
    for (int j = 0; j < cnt; ++j) goff[j + 1] = goff[j] + layers[l0 + j].d_out * layers[l0 + j].d_in;
    if (method != DR_SCORE_GIP) {
      // gbar* = (1/m) sum_j G*_j of the group's layers from the target rows
      dr_layer t[kMaxScoreLayers];
      for (int j = 0; j < cnt; ++j) t[j] = target_layer(layers[l0 + j], n, T);
      st = dr_assemble_update(t, cnt, m, T, len ? len + n : nullptr, DR_BF16, wm, 1, m, nullptr, gstar, goff,
                              ws + pl.off_upd, pl.off_hi - pl.off_upd, stream);
      if (st != DR_OK) return st;
    }
    if (method == DR_SCORE_DIRECT) {
      // one layer at a time: with few tiles an XCD's workgroups then share
      // tiles, whose parts of gbar* its L2 holds (four layers 2048 x 2048 at
      // once 2.58 ms, in turn 2.48)
      const int64_t zero = 0;
      for (int j = 0; j < cnt; ++j) {
        st = direct_scores(layers + l0 + j, 1, n, T, len, gstar + goff[j], &zero, sl + (int64_t)j * n,
                           ws + pl.off_direct, hs);
        if (st != DR_OK) return st;
      }
      l0 = l1;
      continue;
    }
    const bool small = score_small(layers + l0, cnt, n, m, T, (int)method);
    const int64_t rows = score_rows((int)method, small);
    ScoreArgs a = {};
    a.num_layers = cnt;
    a.T = (int)T;
    a.n = (int)n;
    a.m = (int)m;
    a.packed = !small && score_packed(layers + l0, cnt, n, m, T, rows);
    if (a.packed && !planned) {
      hipLaunchKernelGGL(score_plan_kernel, dim3(2), dim3(1024), 0, hs, len, (int)n, (int)m, (int)T, cum);
      if ((st = launch_status()) != DR_OK) return st;
      planned = true;
    }
    a.span = (int)score_span(layers + l0, cnt, T);
    a.SB = (int)gip_cols(m, T, a.packed);
    a.len = len;
    a.cum = cum;
    __bf16* hi = reinterpret_cast<__bf16*>(ws + pl.off_hi);
    __bf16* lo = reinterpret_cast<__bf16*>(ws + pl.off_lo);
    const int64_t slots = score_slots(n, T, rows, a.packed);
    double* part = reinterpret_cast<double*>(ws + pl.off_part);
    int64_t cols = 0;
    for (int j = 0; j < cnt; ++j) {
      const dr_layer& L = layers[l0 + j];
      ScoreLayer& b = a.L[j];
      b.x = static_cast<const unsigned char*>(L.x);
      b.dy = static_cast<const unsigned char*>(L.dy);
      b.ldx = L.ldx;
      b.lddy = L.lddy;
      b.exx = T * L.ldx * 2;
      b.exdy = T * L.lddy * 2;
      b.d_in = (int)L.d_in;
      b.d_out = (int)L.d_out;
      b.OB = (int)((L.d_out + rows - 1) / rows);
      b.ghi = reinterpret_cast<const unsigned char*>(hi + goff[j]);
      b.glo = reinterpret_cast<const unsigned char*>(lo + goff[j]);
      b.part = part;
      const int64_t c = method == DR_SCORE_PIP ? b.OB : a.SB;
      part += slots * c;
      cols += c;
    }
    // tiles over the most row blocks the lengths allow; workgroups past the
    // valid tokens return at once
    const int64_t nt = (row_blocks(n, T, rows, a.packed) * cols + 255) / 256 * 256;
    const dim3 grid((unsigned)(nt < kGridX ? nt : kGridX), (unsigned)((nt + kGridX - 1) / kGridX));
    const bool pieces = a.packed && (n > m ? n : m) > a.span;
    const dim3 rgrid((unsigned)((n + 3) / 4), (unsigned)cnt);
    if (method == DR_SCORE_PIP) {
      hipLaunchKernelGGL(split_kernel, dim3((unsigned)((goff[cnt] + 255) / 256)), dim3(256), 0, hs,
                         (const float*)gstar, (long long)goff[cnt], hi, lo);
      if (nt > 0 && small)
        hipLaunchKernelGGL(pip_small_kernel, grid, dim3(kSThreads), 0, hs, a);
      else if (nt > 0)
        hipLaunchKernelGGL(pieces ? pip_kernel<true> : pip_kernel<false>, grid, dim3(256), 0, hs, a);
      hipLaunchKernelGGL((small ? score_reduce_kernel<kST, true> : score_reduce_kernel<kTileRows, true>), rgrid,
                         dim3(256), 0, hs, a, sl, 1.0);
    } else {
      if (nt > 0)
        hipLaunchKernelGGL(pieces ? gip_kernel<true> : gip_kernel<false>, grid, dim3(kSThreads), 0, hs, a);
      hipLaunchKernelGGL((score_reduce_kernel<kST, false>), rgrid, dim3(256), 0, hs, a, sl, 1.0 / (double)m);
    }
    if ((st = launch_status()) != DR_OK) return st;
    l0 = l1;
  }
  return DR_OK;
}
