// Assembly of the update in full parameter space (dr_assemble_update):
//   U_l = sum_{i < n, w_i != 0} w_i sum_{t < len_i} dy_{i,t} x_{i,t}^T      (d_out x d_in)
// the post-hoc step of Sec. 4.2 that turns the weights of the retained
// examples into the layer updates (top-k weights 1/k on S give the subset
// mean g_S; span or cone weights give u = G^T w of Eq. (proj)).
//
// Kernels
//   update_plan_kernel   one workgroup per example list (one list per
//                        distinct weight row): the examples with w != 0 and
//                        len > 0, their clamped lengths and weights.
//   update_sort_kernel   orders each list by |w| ascending (index breaks
//                        ties) by ranking every entry against all others.
//   update_steps_kernel  whether the weights of a list are all equal, and if
//                        so its token steps.
//   update_list_kernel   the three above in one, for at most 1024 examples.
//   update_tile_kernel   lists of equal weights (top-k, a mean) of larger
//                        calls: one 256 x 256 tile of U per workgroup, 4 waves
//                        of 128 x 128, the examples' tokens one after another.
//   update_bf16_kernel   other lists (and the Direct scorer): the same tile on
//                        8 waves of 128 (d_out) x 64 (d_in), example by
//                        example, tokens through a 2-stage LDS ring in steps of
//                        64.  One fp32 accumulator holds
//                        sum_e (w_e / w_cur) P_e: when the weight changes
//                        from w_cur to w_next it is multiplied by
//                        w_cur / w_next, and by the last weight at the end.
//                        The |w|-ascending order keeps every factor within
//                        [-1, 1] (no overflow whatever the weights).
//                        In both, tokens are staged by buffer->LDS DMA in their
//                        natural token-major layout; the MFMA operands need 8
//                        consecutive tokens per lane, which the gfx950
//                        transposing LDS read (ds_read_b64_tr_b16) delivers
//                        straight from that layout.
//   update_f32_kernel    fp32 inputs: 64 x 64 tiles, 4 waves of 32 x 32,
//                        fp32 MFMA 16x16x4, staged by plain loads; per
//                        example sums added to a second accumulator.
//   update_reduce_kernel when there are fewer tiles than CUs the example
//                        list of a tile is split over `split` workgroups;
//                        their partial tiles are summed in split order.
// Determinism: every sum runs in a fixed order (the sorted list, tokens
// ascending, splits ascending); no atomics.

#include "tile256.h"

namespace dr {
namespace {

constexpr int kMaxUpdLayers = 16;
constexpr int kMaxSplit = 32;

// bf16 tile
constexpr int kBO = 256, kBI = 256, kBK = 64;
constexpr int kBThreads = 512;
constexpr int kBDyBytes = kBK * kBO * 2;   // kBK token rows of 512 bytes
constexpr int kBXBytes = kBK * kBI * 2;
constexpr int kBNH = kBK / 16;             // 1 KB DMA blocks per operand per wave and step
constexpr int kBKK = kBK / 32;             // MFMA reduction slices per step
constexpr int kBStage = kBDyBytes + kBXBytes;
constexpr int kBStages = 2;

// f32 tile
constexpr int kFO = 64, kFI = 64, kFK = 16;
constexpr int kFThreads = 256;
constexpr int kFLd = 80;                   // LDS row stride (floats): the 4 rows of a b32 fragment read hit distinct banks

struct UpdLayerArg {
  const unsigned char* x;
  const unsigned char* dy;
  long long ldx, lddy;   // elements per token
  long long exx, exdy;   // bytes per example (T * ld * element size)
  int d_in, d_out;
  int ti;                // tiles along d_in
  int tile0;             // first tile of this layer within the launch
  int list;              // example list of this layer
  int packed;            // examples of equal weight follow each other in the token steps
  int vec4;              // U rows start 16-byte aligned
  float* U;              // [d_out][d_in]
  const float* gstar;    // score mode: the target-mean gradient [d_out][d_in]
  double* part;          // score mode: partial scores [tiles of the layer][n]
};

// One step of kUK token positions (32 bytes, read by scalar loads): row r is
// token t0 + r of example ex; from row c1 on a token of the next example of
// the list, from row c2 on of the one after; rows past `rows` are empty.
struct UpdStep {
  int ex, t0;
  int geom;         // rows | c1 << 8 | c2 << 16
  int dex1, dex2;   // index of the second and third example, relative to ex
  int pad[3];
};

struct UpdArgs {
  UpdLayerArg L[kMaxUpdLayers];
  int num_layers;
  int ntiles;            // tiles of the launch (all layers)
  int split;             // workgroups per tile along the example list
  int n;                 // list stride (>= 1)
  int nw;                // weighted examples (may be 0)
  const int* ex;         // [lists][n] selected examples, |w| ascending
  const int* exlen;      // [lists][n] their clamped lengths (> 0)
  const float* exw;      // [lists][n] their weights (!= 0)
  const int* cnt;        // [lists] list lengths
  int* pos;              // [lists][2][n + 1] first token position of each example: unpacked, then packed
  int* uniform;          // [lists] 1: all weights of the list are equal
  UpdStep* step;         // [lists][2][max_steps] the token steps of a list of equal weights
  long long max_steps;
  int* uex;              // [lists][n] the same lists before sorting
  int* ulen;
  float* uw;
  float* partial;        // [ntiles * split][tile elements] when split > 1
};

// ------------------------------------------------------------------ plan

struct RowSel {
  int r[kMaxUpdLayers];   // weight row (group) of each layer slot
};

__global__ __launch_bounds__(1024) void update_plan_kernel(const float* w, long long ldw, UpdArgs a,
                                                           const int* len, int T, int list0, RowSel rs) {
  __shared__ int wsum[16];
  __shared__ int base_s;
  const int j = blockIdx.x;                 // layer slot of the launch
  const int list = list0 + j;
  const float* wr = w + (long long)rs.r[j] * ldw;
  int* ex = a.uex + (long long)list * a.n;
  int* exlen = a.ulen + (long long)list * a.n;
  float* exw = a.uw + (long long)list * a.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) base_s = 0;
  __syncthreads();
  for (int b = 0; b < a.nw; b += 1024) {
    const int i = b + tid;
    int L = 0;
    float wi = 0.f;
    if (i < a.nw) {
      wi = wr[i];
      L = len ? len[i] : T;
      L = L < 0 ? 0 : (L > T ? T : L);
    }
    const bool keep = i < a.nw && wi != 0.f && L > 0;
    const unsigned long long m = __ballot(keep);
    const int before = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wave] = __popcll(m);
    __syncthreads();
    int off = base_s;
    for (int v = 0; v < wave; ++v) off += wsum[v];
    if (keep) {
      ex[off + before] = i;
      exlen[off + before] = L;
      exw[off + before] = wi;
    }
    __syncthreads();
    if (tid == 0) {
      int t = 0;
      for (int v = 0; v < 16; ++v) t += wsum[v];
      base_s += t;
    }
    __syncthreads();
  }
  if (tid == 0) const_cast<int*>(a.cnt)[list] = base_s;
}

// Sort key of a weight: |w| as bits, which orders every value, NaNs last (a
// comparison of floats ranks a NaN beside another entry and leaves a hole in
// the list)
__device__ __forceinline__ unsigned weight_key(float w) { return __float_as_uint(w) & 0x7fffffffu; }

// entry i of a list goes to position #{j : (|w_j|, ex_j) < (|w_i|, ex_i)}
__global__ __launch_bounds__(256) void update_sort_kernel(UpdArgs a) {
  __shared__ unsigned kw[256];
  __shared__ int ki[256];
  const int list = blockIdx.y;
  const int cnt = a.cnt[list];
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x * 256 >= cnt) return;
  const long long base = (long long)list * a.n;
  const unsigned wi = i < cnt ? weight_key(a.uw[base + i]) : 0u;
  const int xi = i < cnt ? a.uex[base + i] : 0;
  int rank = 0;
  for (int j0 = 0; j0 < cnt; j0 += 256) {
    __syncthreads();
    const int j = j0 + threadIdx.x;
    kw[threadIdx.x] = j < cnt ? weight_key(a.uw[base + j]) : 0u;
    ki[threadIdx.x] = j < cnt ? a.uex[base + j] : 0;
    __syncthreads();
    const int m = cnt - j0 < 256 ? cnt - j0 : 256;
    for (int q = 0; q < m; ++q) rank += (kw[q] < wi || (kw[q] == wi && ki[q] < xi)) ? 1 : 0;
  }
  if (i < cnt) {
    const_cast<int*>(a.ex)[base + rank] = xi;
    const_cast<int*>(a.exlen)[base + rank] = a.ulen[base + i];
    const_cast<float*>(a.exw)[base + rank] = a.uw[base + i];
  }
}

// Token steps of a list of equal weights (top-k, thresholding, a mean; lists
// of several weights go example by example in update_bf16_kernel).  First the
// position of every example (entry cnt: the end): unpacked, each starts on a
// whole step of kUK tokens; packed, an example of at least kPackLen tokens
// follows the one before it directly (a step then holds tokens of up to
// three), so that a ragged list has one partial step, not one per example.
// Each example is a map x -> (start = fresh ? up(x) : x) + len, up(x) = x
// rounded up to a step; a run of examples is then x -> x + a without a fresh
// start in it, or up(x + a) + b with one (b counts from a whole step on), and
// two runs compose, so a block scan gives every start.  Then the steps
// themselves, one thread each, with everything that update_tile_kernel needs of
// them, so that its main loop has no search and no branch.
constexpr int kUK = 32;   // tokens of a step
constexpr int kPackLen = kUK / 2;
struct PosMap {
  int fresh, a, b;
};
__device__ __forceinline__ int pos_up(int x) { return (x + kUK - 1) & ~(kUK - 1); }
__device__ __forceinline__ PosMap pos_then(PosMap f, PosMap g) {   // g after f
  PosMap r;
  r.fresh = f.fresh | g.fresh;
  r.a = f.fresh ? f.a : f.a + g.a;
  r.b = !f.fresh ? g.b : (g.fresh ? pos_up(f.b + g.a) + g.b : f.b + g.a);
  return r;
}
__device__ __forceinline__ int pos_at(PosMap f) { return f.fresh ? pos_up(f.a) + f.b : f.a; }   // from x = 0

// whether the list's weights are all equal (a whole 1024-thread workgroup;
// the list is in memory)
__device__ __forceinline__ bool list_uniform(const UpdArgs& a, int list, int cnt) {
  __shared__ int differ;
  const float* w = a.exw + (long long)list * a.n;
  if (threadIdx.x == 0) differ = 0;
  __syncthreads();
  bool d = false;
  for (int i = threadIdx.x; i < cnt; i += 1024) d |= w[i] != w[0];
  if (d) differ = 1;
  __syncthreads();
  if (threadIdx.x == 0) a.uniform[list] = !differ;
  return !differ;
}

// its packed or unpacked steps
__device__ __forceinline__ void list_steps(const UpdArgs& a, int list, int cnt, int packed) {
  __shared__ PosMap wmap[16];
  const int* len = a.exlen + (long long)list * a.n;
  const int* ex = a.ex + (long long)list * a.n;
  int* pos = a.pos + ((long long)list * 2 + packed) * (a.n + 1);
  UpdStep* step = a.step + ((long long)list * 2 + packed) * a.max_steps;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (cnt + 1023) / 1024;
  const int i0 = tid * per < cnt ? tid * per : cnt, i1 = i0 + per < cnt ? i0 + per : cnt;
  auto map_of = [&](int i) {
    PosMap m;
    m.fresh = i == 0 || !packed || len[i] < kPackLen;
    m.a = m.fresh ? 0 : len[i];
    m.b = m.fresh ? len[i] : 0;
    return m;
  };
  PosMap loc = {0, 0, 0};
  for (int i = i0; i < i1; ++i) loc = pos_then(loc, map_of(i));
  PosMap inc = loc;
  for (int off = 1; off < 64; off <<= 1) {
    PosMap o;
    o.fresh = __shfl_up(inc.fresh, off, 64);
    o.a = __shfl_up(inc.a, off, 64);
    o.b = __shfl_up(inc.b, off, 64);
    if (lane >= off) inc = pos_then(o, inc);
  }
  __syncthreads();   // (an earlier call's reads of wmap)
  if (lane == 63) wmap[wave] = inc;
  __syncthreads();
  PosMap pre = {0, 0, 0};
  for (int v = 0; v < wave; ++v) pre = pos_then(pre, wmap[v]);
  PosMap o;
  o.fresh = __shfl_up(inc.fresh, 1, 64);
  o.a = __shfl_up(inc.a, 1, 64);
  o.b = __shfl_up(inc.b, 1, 64);
  if (lane > 0) pre = pos_then(pre, o);
  for (int i = i0; i < i1; ++i) {
    const PosMap m = map_of(i);
    const int x = pos_at(pre);
    pos[i] = m.fresh ? pos_up(x) : x;
    pre = pos_then(pre, m);
  }
  if (i1 == cnt && (i0 < cnt || tid == 0)) pos[cnt] = pos_at(pre);
  __syncthreads();
  const int steps = (pos[cnt] + kUK - 1) / kUK;
  for (int q = tid; q < steps; q += 1024) {
    const int p0 = q * kUK;
    int e = 0, hi = cnt - 1;   // the last example that starts at or before p0
    while (e < hi) {
      const int mid = (e + hi + 1) >> 1;
      if (pos[mid] <= p0) e = mid;
      else hi = mid - 1;
    }
    UpdStep st;
    st.ex = ex[e];
    st.t0 = p0 - pos[e];
    st.dex1 = st.dex2 = 0;
    int rows = len[e] - st.t0, c1 = kUK, c2 = kUK;
    if (e + 1 < cnt && pos[e + 1] < p0 + kUK) {
      c1 = pos[e + 1] - p0;
      rows = c1 + len[e + 1];
      st.dex1 = ex[e + 1] - st.ex;
      if (e + 2 < cnt && pos[e + 2] < p0 + kUK) {
        c2 = pos[e + 2] - p0;
        rows = c2 + len[e + 2];
        st.dex2 = ex[e + 2] - st.ex;
      }
    }
    st.geom = (rows < kUK ? rows : kUK) | c1 << 8 | c2 << 16;
    st.pad[0] = st.pad[1] = st.pad[2] = 0;
    step[q] = st;
  }
}

// modes: bit 0 the unpacked steps, bit 1 the packed ones
__global__ __launch_bounds__(1024) void update_steps_kernel(UpdArgs a, int modes) {
  const int list = blockIdx.x, cnt = a.cnt[list];
  if (modes == 0) {
    if (threadIdx.x == 0) a.uniform[list] = 0;
    return;
  }
  if (!list_uniform(a, list, cnt)) return;
  if (modes & 1) list_steps(a, list, cnt, 0);
  if (modes & 2) list_steps(a, list, cnt, 1);
}

// update_plan_kernel, update_sort_kernel and update_steps_kernel in one, for
// at most 1024 examples (three launches less for a call whose products take
// tens of microseconds)
__global__ __launch_bounds__(1024) void update_list_kernel(const float* w, long long ldw, UpdArgs a, const int* len,
                                                           int T, int list0, RowSel rs, int modes) {
  __shared__ int wsum[16];
  __shared__ unsigned kw[1024];
  __shared__ int ki[1024];
  const int list = list0 + blockIdx.x;
  const float* wr = w + (long long)rs.r[blockIdx.x] * ldw;
  const long long base = (long long)list * a.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int L = 0;
  float wi = 0.f;
  if (tid < a.nw) {
    wi = wr[tid];
    L = len ? len[tid] : T;
    L = L < 0 ? 0 : (L > T ? T : L);
  }
  const bool keep = tid < a.nw && wi != 0.f && L > 0;
  const unsigned long long m = __ballot(keep);
  if (lane == 0) wsum[wave] = __popcll(m);
  __syncthreads();
  int at = __popcll(m & ((1ull << lane) - 1ull)), cnt = 0;
  for (int v = 0; v < 16; ++v) {
    at += v < wave ? wsum[v] : 0;
    cnt += wsum[v];
  }
  if (keep) {
    kw[at] = weight_key(wi);
    ki[at] = tid;
  }
  __syncthreads();
  if (keep) {   // to position #{j : (|w_j|, j) < (|w|, i)}
    const unsigned aw = weight_key(wi);
    int rank = 0;
    for (int j = 0; j < cnt; ++j) rank += (kw[j] < aw || (kw[j] == aw && ki[j] < tid)) ? 1 : 0;
    const_cast<int*>(a.ex)[base + rank] = tid;
    const_cast<int*>(a.exlen)[base + rank] = L;
    const_cast<float*>(a.exw)[base + rank] = wi;
  }
  if (tid == 0) {
    const_cast<int*>(a.cnt)[list] = cnt;
    if (modes == 0) a.uniform[list] = 0;
  }
  if (modes == 0) return;
  __syncthreads();
  if (!list_uniform(a, list, cnt)) return;
  if (modes & 1) list_steps(a, list, cnt, 0);
  if (modes & 2) list_steps(a, list, cnt, 1);
}

// which layer / tile / split a workgroup runs.  Workgroup b runs on XCD
// b % 8; each XCD takes a contiguous run of (tile, split) items, so the
// workgroups sharing an L2 share d_out panels of one layer.
__device__ __forceinline__ bool locate(const UpdArgs& a, int& layer, int& to, int& ti, int& s, int& item) {
  const int items = a.ntiles * a.split;
  const int per = (items + 7) >> 3;
  const int k = blockIdx.x >> 3;
  if (k >= per) return false;
  item = (blockIdx.x & 7) * per + k;
  if (item >= items) return false;
  const int tile = item / a.split;
  s = item - tile * a.split;
  layer = 0;
  while (layer + 1 < a.num_layers && a.L[layer + 1].tile0 <= tile) ++layer;
  const int t = tile - a.L[layer].tile0;
  to = t / a.L[layer].ti;
  ti = t - to * a.L[layer].ti;
  return true;
}

// ------------------------------------------------------------------ bf16


// 256 x 256 tiles on eight waves of 128 x 64, one example after another.
// SCORE = false: the update of lists of several weights.  SCORE = true (the Direct scorer of Sec. 4.3):
// every example of the list gets weight 1; at the end of each example its
// tile of G_i is dotted with the same tile of the target-mean gradient and
// the accumulator cleared, so G_i is formed tile by tile and never stored.
template <bool SCORE>
__global__ __launch_bounds__(kBThreads) void update_bf16_kernel(UpdArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kBStages * kBStage];
  int layer, to, ti, s, item;
  if (!locate(a, layer, to, ti, s, item)) return;
  const UpdLayerArg& Lr = a.L[layer];
  const int d_in = Lr.d_in, d_out = Lr.d_out;
  const int o0 = to * kBO, i0 = ti * kBI;
  if (!SCORE && a.uniform[Lr.list]) return;   // update_tile_kernel's
  const int cnt = a.cnt[Lr.list];
  const int e_lo = (int)((long long)s * cnt / a.split), e_hi = (int)((long long)(s + 1) * cnt / a.split);
  const int* ex = a.ex + (long long)Lr.list * a.n;
  const int* exlen = a.exlen + (long long)Lr.list * a.n;
  const float* exw = a.exw + (long long)Lr.list * a.n;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // DMA roles: both tiles have kBK token rows of 512 bytes; wave w fills
  // rows 2j, 2j + 1 for j = w, w + 8, ... of each (1 KB per wave load).
  // Lane l fills 16 bytes: physical slot u / 2, half u % 2 of its row.
  int rrow[kBNH];
  unsigned cdy[kBNH], cx[kBNH];   // byte column inside a token row, or kOobOffset
#pragma unroll
  for (int h = 0; h < kBNH; ++h) {
    const int j = w + 8 * h;
    const int r = 2 * j + (lane >> 5), u = lane & 31;
    const int col = 16 * ((u >> 1) ^ slot_xor(r)) + 8 * (u & 1);
    rrow[h] = r;
    cdy[h] = o0 + col < d_out ? (unsigned)((o0 + col) * 2) : kOobOffset;
    cx[h] = i0 + col < d_in ? (unsigned)((i0 + col) * 2) : kOobOffset;
  }
  const unsigned rowb_dy = (unsigned)(Lr.lddy * 2), rowb_x = (unsigned)(Lr.ldx * 2);

  int ie = e_lo, it = 0, ilen = ie < e_hi ? exlen[ie] : 0;
  auto issue = [&](int st) {
    const unsigned sb = lds_offset(lds) + st * kBStage;
    const unsigned char *rdys, *rxs;
    unsigned o_dy[kBNH], o_x[kBNH];
    if (ie < e_hi) {
      const long long e = ex[ie];
      rdys = Lr.dy + e * Lr.exdy;
      rxs = Lr.x + e * Lr.exx;
#pragma unroll
      for (int h = 0; h < kBNH; ++h) {
        const int t = it + rrow[h];
        o_dy[h] = (t < ilen && cdy[h] != kOobOffset) ? (unsigned)t * rowb_dy + cdy[h] : kOobOffset;
        o_x[h] = (t < ilen && cx[h] != kOobOffset) ? (unsigned)t * rowb_x + cx[h] : kOobOffset;
      }
      it += kBK;
      if (it >= ilen) {
        ++ie;
        it = 0;
        ilen = ie < e_hi ? exlen[ie] : 0;
      }
    } else {
      rdys = Lr.dy;
      rxs = Lr.x;
#pragma unroll
      for (int h = 0; h < kBNH; ++h) o_dy[h] = o_x[h] = kOobOffset;
    }
    // (scores: the tracked form measured 5 % faster, 2.48 against 2.61 ms on
    // four layers of the small block; updates: the other 4 % faster)
    unsigned char* sp = lds + st * kBStage;
#pragma unroll
    for (int h = 0; h < kBNH; ++h) {
      if (SCORE) dma16<kAuxCached>(make_rsrc(rdys, kOobOffset), sp + (w + 8 * h) * 1024, o_dy[h]);
      else dma16_untracked(rdys, sb + (w + 8 * h) * 1024, o_dy[h]);
    }
#pragma unroll
    for (int h = 0; h < kBNH; ++h) {
      if (SCORE) dma16<kAuxCached>(make_rsrc(rxs, kOobOffset), sp + kBDyBytes + (w + 8 * h) * 1024, o_x[h]);
      else dma16_untracked(rxs, sb + kBDyBytes + (w + 8 * h) * 1024, o_x[h]);
    }
  };

  // fragment reads: lane (g, q, r) of the transposing read addresses token
  // row 8g + q (+4 for the second half) and 8-byte piece r of the 16-column
  // block; the block's logical slot is XOR-ed with the row's swizzle.
  const int g = lane >> 4, q = (lane >> 2) & 3, rr = lane & 3;
  const int fx = q | ((g & 1) << 2);
  const int wr = w >> 2, wc = w & 3;   // 128-row half (d_out), 64-column quarter (d_in)
  const unsigned rbase = (unsigned)((8 * g + q) * 512 + rr * 8);
  unsigned offa[8], offb[4];
#pragma unroll
  for (int b = 0; b < 8; ++b) offa[b] = rbase + (unsigned)(((8 * wr + b) ^ fx) * 32);
#pragma unroll
  for (int b = 0; b < 4; ++b) offb[b] = kBDyBytes + rbase + (unsigned)(((4 * wc + b) ^ fx) * 32);

  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  float wlast = 0.f;
  int ce = e_lo, ct = 0, clen = ce < e_hi ? exlen[ce] : 0;
  if (ce < e_hi) {
#pragma unroll
    for (int st = 0; st < kBStages - 1; ++st) issue(st);
    for (int step = 0; ce < e_hi; ++step) {
      DR_WAIT_VM(2 * kBNH * (kBStages - 2));   // this step's loads are done; later steps' may be in flight
      DR_LDS_SYNC();
      issue((step + kBStages - 1) % kBStages);
      const unsigned char* sb0 = lds + (step % kBStages) * kBStage;
#pragma unroll
      for (int kk = 0; kk < kBKK; ++kk) {
        const unsigned char* sb = sb0 + kk * 32 * 512;   // token rows 32 kk .. 32 kk + 31
        u32x4 fa[8], fb[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const v4s lo = lds_read_tr16(sb + offb[b]);
          const v4s hi = lds_read_tr16(sb + offb[b] + 4 * 512);
          fb[b] = u32x4{__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y,
                        __builtin_bit_cast(uint2, hi).x, __builtin_bit_cast(uint2, hi).y};
        }
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const v4s lo = lds_read_tr16(sb + offa[b]);
          const v4s hi = lds_read_tr16(sb + offa[b] + 4 * 512);
          fa[b] = u32x4{__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y,
                        __builtin_bit_cast(uint2, hi).x, __builtin_bit_cast(uint2, hi).y};
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = mma_bf16(fa[i], fb[j], acc[i][j]);
      }
      ct += kBK;
      if (ct >= clen) {
        if constexpr (SCORE) {
          __shared__ double red[kBThreads / 64];
          const int lc = lane & 15;
          float d = 0.f;
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int o = o0 + 128 * wr + 16 * i + 4 * g + r;
              if (o >= d_out) continue;
              const float* grow = Lr.gstar + (long long)o * d_in;
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const int c = i0 + 64 * wc + 16 * j + lc;
                if (c < d_in) d = fmaf(acc[i][j][r], grow[c], d);
              }
            }
          double dd = (double)d;
          for (int off = 32; off > 0; off >>= 1) dd += __shfl_xor(dd, off, 64);
          if (lane == 0) red[w] = dd;
          __syncthreads();
          if (tid == 0) {
            double t = 0.0;
            for (int v = 0; v < kBThreads / 64; ++v) t += red[v];
            Lr.part[(long long)(to * Lr.ti + ti) * a.nw + ex[ce]] = t;
          }
          __syncthreads();
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          ++ce;
          ct = 0;
          clen = ce < e_hi ? exlen[ce] : 0;
        } else {
          const float we = exw[ce];
          ++ce;
          ct = 0;
          clen = ce < e_hi ? exlen[ce] : 0;
          wlast = we;
          if (ce < e_hi) {
            const float wn = exw[ce];
            if (wn != we) {
              const float f = we / wn;   // |f| <= 1 in the sorted order
#pragma unroll
              for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                  for (int r = 0; r < 4; ++r) acc[i][j][r] *= f;
            }
          }
        }
      }
    }
    DR_WAIT_VM(0);
  }
  if constexpr (SCORE) return;

  // C layout: register r of block (i, j) is row 4g + r, column lane % 16
  const int lc = lane & 15;
  if (a.split == 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = o0 + 128 * wr + 16 * i + 4 * g + r;
        if (o >= d_out) continue;
        float* urow = Lr.U + (long long)o * d_in;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = i0 + 64 * wc + 16 * j + lc;
          if (c < d_in) urow[c] = wlast * acc[i][j][r];
        }
      }
  } else {
    float* P = a.partial + (long long)item * (kBO * kBI);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          P[(128 * wr + 16 * i + 4 * g + r) * kBI + 64 * wc + 16 * j + lc] = wlast * acc[i][j][r];
  }
}

// The update of lists of equal weights: one 256 x 256 tile of U per workgroup,
// four waves (one per SIMD) of 128 (d_out) x 128 (d_in) with the accumulators
// in AGPRs, each product an in-place asm MFMA (see tile256.h).  A step is 32
// token rows of 512 bytes of either operand, read as MFMA operands by the
// transposing LDS read; five stages fill the LDS, so that the DMA of a step is
// issued four steps before its reads.  Per step t: wait for step t + 1 (the
// three after it stay in flight) and one barrier, which also frees the stage of
// step t, whose fragments are in registers; then the products of step t with
// the DMA of step t + 5 and the fragment reads of step t + 1 between them.
// Bound by MFMA and by the latency of the DMA's first touch of HBM.  Small
// block, top-32 of 64 (8 layers 2048 x 2048, 0.69 TFLOP): 0.86 ms on eight
// waves of 128 x 64 in steps of 64 tokens padded per example (their fragment
// reads waited for all DMA, and read half as much again per product), 0.71 ms
// here on the benchmark's inputs (0.59 to 0.61 on others of the same size, which
// is not explained; MFMA busy 52 % at 1.9 GHz; 0.51 without any DMA, 0.61 with every read an
// L2 hit), 0.73 with two stages of 64 tokens.  (Several weights would need
// the accumulators rescaled between steps, which makes the compiler spill them.)
constexpr int kUStage = 2 * kUK * 512;   // dy rows, then x rows
constexpr int kUStages = 5;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void update_tile_kernel(UpdArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kUStages * kUStage];
  int layer, to, ti, s, item;
  if (!locate(a, layer, to, ti, s, item)) return;
  const UpdLayerArg& Lr = a.L[layer];
  const int d_in = Lr.d_in, d_out = Lr.d_out;
  const int o0 = to * kBO, i0 = ti * kBI;
  if (!a.uniform[Lr.list]) return;   // update_bf16_kernel's
  const long long lp = (long long)Lr.list * 2 + Lr.packed;
  const int steps = (a.pos[lp * (a.n + 1) + a.cnt[Lr.list]] + kUK - 1) / kUK;
  const int s_lo = (int)((long long)s * steps / a.split), s_hi = (int)((long long)(s + 1) * steps / a.split);
  const int nk = __builtin_amdgcn_readfirstlane(s_hi - s_lo);
  // (constant address space: scalar loads)
  typedef const __attribute__((address_space(4))) UpdStep* StepPtr;
  const StepPtr step = (StepPtr)(a.step + lp * a.max_steps + __builtin_amdgcn_readfirstlane(s_lo));
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // DMA: wave w fills token rows r0 + 8 u, r0 = 2 w + lane / 32, u = 0..3, of
  // both panels (1 KB = two rows each); lane l's 16 bytes are physical slot
  // (l % 32) / 2, half l % 2 of its row, so its column depends on u's parity
  const unsigned rowb_dy = (unsigned)(Lr.lddy * 2), rowb_x = (unsigned)(Lr.ldx * 2);
  const int r0 = 2 * w + (lane >> 5);
  unsigned cdy[2], cx[2];   // byte column inside a token row, or kOobOffset
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int col = 16 * (((lane & 31) >> 1) ^ slot_xor(r0 + 8 * u)) + 8 * (lane & 1);
    cdy[u] = o0 + col < d_out ? (unsigned)((o0 + col) * 2) : kOobOffset;
    cx[u] = i0 + col < d_in ? (unsigned)((i0 + col) * 2) : kOobOffset;
  }
  // the step being issued: this lane's rows as offsets from bdy / bx (from row
  // c1 on those of the next example, from c2 on of the one after: packed lists,
  // whose whole batch spans less than 4 GiB)
  unsigned vdy[4], vx[4];
  const unsigned char* bdy = Lr.dy;
  const unsigned char* bx = Lr.x;
  int geom = -1, dex1 = 0, dex2 = 0, t12 = 0;   // what the offsets were formed for
  const unsigned ex_dy = (unsigned)Lr.exdy, ex_x = (unsigned)Lr.exx;   // (an example spans less than 4 GiB)
  UpdStep nxt = {};                                                    // the next step, loaded a step ahead
  if (nk > 0) {
    const StepPtr p = step;
    nxt = UpdStep{p->ex, p->t0, p->geom, p->dex1, p->dex2, {0, 0, 0}};
  }
  auto place = [&](int t) __attribute__((always_inline)) {
    const UpdStep c = nxt;
    {
      const StepPtr p = step + (t + 1 < nk ? t + 1 : (nk > 0 ? nk - 1 : 0));
      if (nk > 0) nxt = UpdStep{p->ex, p->t0, p->geom, p->dex1, p->dex2, {0, 0, 0}};
    }
    bdy = Lr.dy + (long long)c.ex * Lr.exdy + (long long)c.t0 * rowb_dy;
    bx = Lr.x + (long long)c.ex * Lr.exx + (long long)c.t0 * rowb_x;
    // the offsets change only at the ends of examples: most steps are 32 rows
    // of one example, as the step before
    const int ng = t < nk ? c.geom : 0;
    const int nt = ng >> 8 == (kUK | kUK << 8) ? 0 : c.t0;
    if (ng != geom || nt != t12 || c.dex1 != dex1 || c.dex2 != dex2) {
      geom = ng;
      dex1 = c.dex1;
      dex2 = c.dex2;
      t12 = nt;
      const int rows = ng & 255, c1 = ng >> 8 & 255, c2 = ng >> 16;
      const unsigned t1 = (unsigned)(c1 + c.t0), t2 = (unsigned)(c2 + c.t0);
      const unsigned d1dy = (unsigned)dex1 * ex_dy - t1 * rowb_dy, d1x = (unsigned)dex1 * ex_x - t1 * rowb_x;
      const unsigned d2dy = (unsigned)dex2 * ex_dy - t2 * rowb_dy, d2x = (unsigned)dex2 * ex_x - t2 * rowb_x;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = r0 + 8 * u;
        const unsigned my = r >= c2 ? d2dy : (r >= c1 ? d1dy : 0u), mx = r >= c2 ? d2x : (r >= c1 ? d1x : 0u);
        vdy[u] = r < rows && cdy[u & 1] != kOobOffset ? (unsigned)r * rowb_dy + cdy[u & 1] + my : kOobOffset;
        vx[u] = r < rows && cx[u & 1] != kOobOffset ? (unsigned)r * rowb_x + cx[u & 1] + mx : kOobOffset;
      }
    }
  };
  const unsigned lds0 = lds_offset(lds);
  auto dma1 = [&](int stage, int q) __attribute__((always_inline)) {   // q = 0..7: dy, x rows in turn
    const int u = q >> 1;
    dma16_untracked(q & 1 ? bx : bdy, lds0 + stage + (q & 1) * (kUK * 512) + (w + 4 * u) * 1024,
                    q & 1 ? vx[u] : vdy[u]);
  };

  // fragment reads: lane (g, q, r) of the transposing read addresses token
  // row 8g + q (+4 for the second half) and 8-byte piece r of the 16-column
  // block; the block's logical slot is XOR-ed with the row's swizzle
  const int g = lane >> 4, tq = (lane >> 2) & 3, rr = lane & 3;
  const int fx = tq | ((g & 1) << 2);
  const int wr = w >> 1, wc = w & 1;   // 128-row half (d_out), 128-column half (d_in)
  const unsigned rbase = (unsigned)((8 * g + tq) * 512 + rr * 8);
  // (8 wr + b) ^ fx = 8 wr + (b ^ fx), and no other address bit lies in the slot's
  const unsigned offa = rbase + (unsigned)((8 * wr + fx) * 32);
  const unsigned offb = kUK * 512 + rbase + (unsigned)((8 * wc + fx) * 32);
  auto rd1 = [&](u32x4* fa, u32x4* fb, int stage, int q) __attribute__((always_inline)) {
    const unsigned char* p = lds + stage + ((q & 1 ? offb : offa) ^ (unsigned)((q >> 1) * 32));
    const uint2 lo = __builtin_bit_cast(uint2, lds_read_tr16(p));
    const uint2 hi = __builtin_bit_cast(uint2, lds_read_tr16(p + 4 * 512));
    if (q & 1) fb[q >> 1] = u32x4{lo.x, lo.y, hi.x, hi.y};
    else fa[q >> 1] = u32x4{lo.x, lo.y, hi.x, hi.y};
  };
  f32x4 acc[8][8];
  tile256_clear(acc);
  u32x4 fa0[8], fb0[8], fa1[8], fb1[8];
  static_assert(kUStages == 5, "waits below");
#pragma unroll
  for (int t = 0; t < kUStages; ++t) {
    place(t);
#pragma unroll
    for (int q = 0; q < 8; ++q) dma1(t * kUStage, q);
  }
  DR_WAIT_VM(32);
  DR_LDS_SYNC();
#pragma unroll
  for (int q = 0; q < 16; ++q) rd1(fa0, fb0, 0, q);
  int sc = 0;   // stage of the step being multiplied
  auto run_step = [&](int t, const u32x4* fa, const u32x4* fb, u32x4* na, u32x4* nb) __attribute__((always_inline)) {
    const int sn = sc == (kUStages - 1) * kUStage ? 0 : sc + kUStage;
    place(t + kUStages);
    DR_WAIT_VM(24);
    DR_LDS_SYNC();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      if (q < 8) dma1(sc, q);
      rd1(na, nb, sn, q);
#pragma unroll
      for (int m = 4 * q; m < 4 * q + 4; ++m)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(acc[m & 7][m >> 3]) : "v"(fa[m & 7]), "v"(fb[m >> 3]));
    }
    sc = sn;
  };
  for (int t = 0; t < nk; t += 2) {
    run_step(t, fa0, fb0, fa1, fb1);
    run_step(t + 1, fa1, fb1, fa0, fb0);   // (past the last step: zeros)
  }
  tile256_settle(acc);
  DR_WAIT_VM(0);
  const float wgt = nk > 0 ? a.exw[(long long)Lr.list * a.n] : 0.f;

  // C layout: register r of block (i, j) is row 4g + r, column lane % 16; out
  // in float4 after a 4 x 4 transpose inside each quad of lanes (lane 4 m + c
  // then holds row 4 g + c, columns 4 m .. + 3)
  const int c4 = lane & 3, m4 = (lane >> 2) & 3;
  float* out = a.split == 1 ? Lr.U + (long long)o0 * d_in + i0 : a.partial + (long long)item * (kBO * kBI);
  const long long ld = a.split == 1 ? d_in : kBI;
  const int orows = a.split == 1 ? d_out - o0 : kBO, ocols = a.split == 1 ? d_in - i0 : kBI;
  const bool vec = a.split > 1 || Lr.vec4;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const f32x4 v = quad_transpose(acc[i][j]) * wgt;
      const int row = 128 * wr + 16 * i + 4 * g + c4, col = 128 * wc + 16 * j + 4 * m4;
      if (row >= orows || col >= ocols) continue;   // (widths are multiples of 8)
      float* o = out + row * ld + col;
      if (vec) {
        *reinterpret_cast<f32x4*>(o) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = v[e];
      }
    }
}

// ------------------------------------------------------------------ f32

__global__ __launch_bounds__(kFThreads) void update_f32_kernel(UpdArgs a) {
  __shared__ __attribute__((aligned(16))) float sdy[2][kFK][kFLd];
  __shared__ __attribute__((aligned(16))) float sx[2][kFK][kFLd];
  int layer, to, ti, s, item;
  if (!locate(a, layer, to, ti, s, item)) return;
  const UpdLayerArg& Lr = a.L[layer];
  const int d_in = Lr.d_in, d_out = Lr.d_out;
  const int o0 = to * kFO, i0 = ti * kFI;
  const int cnt = a.cnt[Lr.list];
  const int e_lo = (int)((long long)s * cnt / a.split), e_hi = (int)((long long)(s + 1) * cnt / a.split);
  const int* ex = a.ex + (long long)Lr.list * a.n;
  const int* exlen = a.exlen + (long long)Lr.list * a.n;
  const float* exw = a.exw + (long long)Lr.list * a.n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // staging: thread t loads token row t / 16 (of 16), columns 4 (t % 16) .. +3 of both operands
  const int sr = tid >> 4, sc = 4 * (tid & 15);
  const bool okdy = o0 + sc < d_out, okx = i0 + sc < d_in;
  float4 vdy = make_float4(0.f, 0.f, 0.f, 0.f), vx = vdy;
  int ie = e_lo, it = 0, ilen = ie < e_hi ? exlen[ie] : 0;
  auto fetch = [&]() {
    vdy = make_float4(0.f, 0.f, 0.f, 0.f);
    vx = vdy;
    if (ie < e_hi) {
      const long long e = ex[ie];
      const int t = it + sr;
      if (t < ilen) {
        if (okdy)
          vdy = *reinterpret_cast<const float4*>(Lr.dy + e * Lr.exdy + ((long long)t * Lr.lddy + o0 + sc) * 4);
        if (okx) vx = *reinterpret_cast<const float4*>(Lr.x + e * Lr.exx + ((long long)t * Lr.ldx + i0 + sc) * 4);
      }
      it += kFK;
      if (it >= ilen) {
        ++ie;
        it = 0;
        ilen = ie < e_hi ? exlen[ie] : 0;
      }
    }
  };

  const int wo = w >> 1, wi = w & 1;   // 32 x 32 quarter of the tile
  const int lr = lane & 15, lk = lane >> 4;
  f32x4 acc[2][2], tot[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  int ce = e_lo, ct = 0, clen = ce < e_hi ? exlen[ce] : 0;
  if (ce < e_hi) fetch();
  for (int step = 0; ce < e_hi; ++step) {
    const int b = step & 1;
    *reinterpret_cast<float4*>(&sdy[b][sr][sc]) = vdy;
    *reinterpret_cast<float4*>(&sx[b][sr][sc]) = vx;
    __syncthreads();
    fetch();   // next step's loads in flight during this step's products
#pragma unroll
    for (int kk = 0; kk < kFK / 4; ++kk) {
      const int k = 4 * kk + lk;
      float fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[i] = sdy[b][k][32 * wo + 16 * i + lr];
#pragma unroll
      for (int j = 0; j < 2; ++j) fb[j] = sx[b][k][32 * wi + 16 * j + lr];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mma_f32(fa[i], fb[j], acc[i][j]);
    }
    ct += kFK;
    if (ct >= clen) {
      const float we = exw[ce];
      ++ce;
      ct = 0;
      clen = ce < e_hi ? exlen[ce] : 0;
      if (ce >= e_hi || exw[ce] != we) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) tot[i][j][r] = fmaf(we, acc[i][j][r], tot[i][j][r]);
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  }

  const int g = lane >> 4;
  if (a.split == 1) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = o0 + 32 * wo + 16 * i + 4 * g + r;
        if (o >= d_out) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int c = i0 + 32 * wi + 16 * j + lr;
          if (c < d_in) Lr.U[(long long)o * d_in + c] = tot[i][j][r];
        }
      }
  } else {
    float* P = a.partial + (long long)item * (kFO * kFI);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 2; ++j) P[(32 * wo + 16 * i + 4 * g + r) * kFI + 32 * wi + 16 * j + lr] = tot[i][j][r];
  }
}

// U = sum over splits of the partial tiles, in split order
__global__ __launch_bounds__(256) void update_reduce_kernel(UpdArgs a, int TO, int TI) {
  const int tile = blockIdx.y;
  int layer = 0;
  while (layer + 1 < a.num_layers && a.L[layer + 1].tile0 <= tile) ++layer;
  const UpdLayerArg& Lr = a.L[layer];
  const int t = tile - Lr.tile0, to = t / Lr.ti, ti = t - to * Lr.ti;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= TO * TI) return;
  const int o = to * TO + e / TI, c = ti * TI + e % TI;
  if (o >= Lr.d_out || c >= Lr.d_in) return;
  const float* P = a.partial + (long long)tile * a.split * (TO * TI) + e;
  float v = 0.f;
  for (int s = 0; s < a.split; ++s) v += P[(long long)s * (TO * TI)];
  Lr.U[(long long)o * Lr.d_in + c] = v;
}

// ------------------------------------------------------------------ host

constexpr int64_t kStepBytes = (int64_t)256 << 20;

struct UpdPlan {
  int64_t tiles;     // all layers
  int split;
  size_t off_ex, off_len, off_w, off_uex, off_ulen, off_uw, off_cnt, off_uniform, off_pos, off_step, off_partial, bytes;
  int64_t max_steps;
};

int cu_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                                              hipSuccess || cus < 1)
    cus = 256;
  return cus;
}

void tile_dims(dr_dtype dtype, int& TO, int& TI) {
  TO = dtype == DR_BF16 ? kBO : kFO;
  TI = dtype == DR_BF16 ? kBI : kFI;
}

UpdPlan update_plan(const dr_layer* layers, int num_layers, int64_t n, int64_t T, dr_dtype dtype) {
  UpdPlan p;
  int TO, TI;
  tile_dims(dtype, TO, TI);
  p.tiles = 0;
  for (int l = 0; l < num_layers; ++l)
    p.tiles += ((layers[l].d_out + TO - 1) / TO) * ((layers[l].d_in + TI - 1) / TI);
  // resident workgroups: one bf16 workgroup (128 KB of LDS, 8 waves) or
  // four f32 workgroups per CU
  const int64_t slots = (int64_t)cu_count() * (dtype == DR_BF16 ? 1 : 4);
  int64_t split = 1;
  if (p.tiles < slots && n > 1) {
    split = (slots + p.tiles - 1) / p.tiles;
    if (split > kMaxSplit) split = kMaxSplit;
    if (split > n) split = n;
  }
  p.split = (int)split;
  const size_t nn = (size_t)(n > 0 ? n : 1) * num_layers;
  size_t o = 0;
  p.off_ex = o;      o = align_up(o + nn * 4, 256);
  p.off_len = o;     o = align_up(o + nn * 4, 256);
  p.off_w = o;       o = align_up(o + nn * 4, 256);
  p.off_uex = o;     o = align_up(o + nn * 4, 256);
  p.off_ulen = o;    o = align_up(o + nn * 4, 256);
  p.off_uw = o;      o = align_up(o + nn * 4, 256);
  p.off_cnt = o;     o = align_up(o + (size_t)num_layers * 4, 256);
  // step tables (both modes of every list) within kStepBytes, which also keeps
  // positions in 32 bits; without them every list is update_bf16_kernel's
  p.max_steps = n * ((T + kUK - 1) / kUK) > 0 ? n * ((T + kUK - 1) / kUK) : 1;
  if (dtype != DR_BF16 || p.max_steps > kStepBytes / (int64_t)(2 * sizeof(UpdStep)) / num_layers) p.max_steps = 0;
  p.off_uniform = o; o = align_up(o + (size_t)num_layers * 4, 256);
  p.off_pos = o;     if (p.max_steps > 0) o = align_up(o + (nn + num_layers) * 2 * 4, 256);
  p.off_step = o;    o = align_up(o + (size_t)num_layers * 2 * p.max_steps * sizeof(UpdStep), 256);
  p.off_partial = o;
  if (p.split > 1) o = align_up(o + (size_t)p.tiles * p.split * TO * TI * 4, 256);
  p.bytes = o;
  return p;
}

dr_status validate_update(const dr_layer* layers, int num_layers, int64_t n, int64_t T, dr_dtype dtype,
                          const float* w, int P, int64_t ldw, const int32_t* group_of_layer, const float* U,
                          const int64_t* u_offset) {
  if (dtype != DR_BF16 && dtype != DR_F32) return DR_ERR_DTYPE;
  if (!layers || num_layers < 1 || n < 0 || T < 0 || P < 1) return DR_ERR_ARG;
  if (n > (1 << 24) || T > (1 << 24) || ldw < n) return DR_ERR_ARG;
  if (n > 0 && !w) return DR_ERR_ARG;
  if (!U || !u_offset) return DR_ERR_ARG;
  const int64_t vec = dtype == DR_BF16 ? 8 : 4;
  const int64_t es = dtype == DR_BF16 ? 2 : 4;
  for (int l = 0; l < num_layers; ++l) {
    const dr_layer& L = layers[l];
    if (group_of_layer && (group_of_layer[l] < 0 || group_of_layer[l] >= P)) return DR_ERR_ARG;
    if (u_offset[l] < 0) return DR_ERR_ARG;
    if (L.d_in < 1 || L.d_out < 1 || L.d_in % vec || L.d_out % vec) return DR_ERR_ARG;
    if (L.d_in > (1 << 28) || L.d_out > (1 << 28)) return DR_ERR_ARG;
    if (L.ldx < L.d_in || L.lddy < L.d_out || L.ldx % vec || L.lddy % vec) return DR_ERR_ARG;
    if (n > 0 && T > 0) {
      if (!L.x || !L.dy || !aligned16(L.x) || !aligned16(L.dy)) return DR_ERR_ARG;
      // token rows are addressed with 32-bit offsets inside one example
      if (T * L.ldx * es >= (int64_t)kOobOffset - 64 || T * L.lddy * es >= (int64_t)kOobOffset - 64)
        return DR_ERR_UNSUPPORTED;
    }
  }
  return DR_OK;
}

__global__ void fill_f32_kernel(float* p, long long n, float v) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// s[i] = sum over the layer's tiles of the partial scores (tile order), 0 for empty examples
__global__ void direct_reduce_kernel(const double* part, int tiles, int n, const int* len, int T, float* s) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int L = len ? len[i] : T;
  L = L < 0 ? 0 : (L > T ? T : L);
  double t = 0.0;
  if (L > 0)
    for (int q = 0; q < tiles; ++q) t += part[(long long)q * n + i];
  s[i] = (float)t;
}

}  // namespace

size_t direct_workspace(const dr_layer* layers, int num_layers, int64_t n) {
  const UpdPlan pl = update_plan(layers, num_layers, n, 0, DR_BF16);
  size_t o = align_up(pl.bytes, 256);
  o = align_up(o + (size_t)(n > 0 ? n : 1) * 4, 256);   // unit weights
  for (int l = 0; l < num_layers; ++l) {
    const int64_t tiles = ((layers[l].d_out + kBO - 1) / kBO) * ((layers[l].d_in + kBI - 1) / kBI);
    o = align_up(o + (size_t)tiles * (size_t)(n > 0 ? n : 1) * 8, 256);
  }
  return o;
}

// Direct scores s[l][i] = <gstar_l, G_i^(l)> of the first n examples, for
// bf16 layers whose target-mean gradients sit at gstar + g_off[l]
dr_status direct_scores(const dr_layer* layers, int num_layers, int64_t n, int64_t T, const int32_t* len,
                        const float* gstar, const int64_t* g_off, float* s, void* workspace, hipStream_t hs) {
  const UpdPlan pl = update_plan(layers, num_layers, n, 0, DR_BF16);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  size_t o = align_up(pl.bytes, 256);
  float* ones = reinterpret_cast<float*>(ws + o);
  o = align_up(o + (size_t)(n > 0 ? n : 1) * 4, 256);
  double* part0 = reinterpret_cast<double*>(ws + o);
  if (n == 0) return DR_OK;
  hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, hs, ones, (long long)n, 1.0f);
  dr_status st = launch_status();
  UpdArgs base = {};
  base.split = pl.split;
  base.n = (int)n;
  base.nw = (int)n;
  base.ex = reinterpret_cast<const int*>(ws + pl.off_ex);
  base.exlen = reinterpret_cast<const int*>(ws + pl.off_len);
  base.exw = reinterpret_cast<const float*>(ws + pl.off_w);
  base.uex = reinterpret_cast<int*>(ws + pl.off_uex);
  base.ulen = reinterpret_cast<int*>(ws + pl.off_ulen);
  base.uw = reinterpret_cast<float*>(ws + pl.off_uw);
  base.cnt = reinterpret_cast<const int*>(ws + pl.off_cnt);
  base.uniform = reinterpret_cast<int*>(ws + pl.off_uniform);
  base.pos = reinterpret_cast<int*>(ws + pl.off_pos);
  base.step = reinterpret_cast<UpdStep*>(ws + pl.off_step);
  base.max_steps = pl.max_steps;
  base.partial = reinterpret_cast<float*>(ws + pl.off_partial);
  RowSel rs = {};
  if (st == DR_OK) {
    hipLaunchKernelGGL(update_plan_kernel, dim3(1), dim3(1024), 0, hs, (const float*)ones, (long long)n, base, len,
                       (int)T, 0, rs);
    st = launch_status();
  }
  if (st == DR_OK) {
    hipLaunchKernelGGL(update_sort_kernel, dim3((unsigned)((n + 255) / 256), 1), dim3(256), 0, hs, base);
    st = launch_status();
  }
  double* part = part0;
  for (int first = 0; first < num_layers && st == DR_OK; first += kMaxUpdLayers) {
    const int count = num_layers - first < kMaxUpdLayers ? num_layers - first : kMaxUpdLayers;
    UpdArgs a = base;
    int tiles = 0;
    double* parts[kMaxUpdLayers];
    int ltiles[kMaxUpdLayers];
    for (int j = 0; j < count; ++j) {
      const dr_layer& L = layers[first + j];
      UpdLayerArg& la = a.L[j];
      la.x = static_cast<const unsigned char*>(L.x);
      la.dy = static_cast<const unsigned char*>(L.dy);
      la.ldx = L.ldx;
      la.lddy = L.lddy;
      la.exx = T * L.ldx * 2;
      la.exdy = T * L.lddy * 2;
      la.d_in = (int)L.d_in;
      la.d_out = (int)L.d_out;
      la.ti = (int)((L.d_in + kBI - 1) / kBI);
      la.tile0 = tiles;
      la.list = 0;
      la.U = nullptr;
      la.gstar = gstar + g_off[first + j];
      la.part = part;
      ltiles[j] = (int)(((L.d_out + kBO - 1) / kBO) * la.ti);
      parts[j] = part;
      part = reinterpret_cast<double*>(reinterpret_cast<unsigned char*>(part) +
                                       align_up((size_t)ltiles[j] * (size_t)n * 8, 256));
      tiles += ltiles[j];
    }
    a.num_layers = count;
    a.ntiles = tiles;
    const int items = tiles * pl.split;
    hipLaunchKernelGGL(update_bf16_kernel<true>, dim3((items + 7) / 8 * 8), dim3(kBThreads), 0, hs, a);
    if ((st = launch_status()) != DR_OK) break;
    for (int j = 0; j < count && st == DR_OK; ++j) {
      hipLaunchKernelGGL(direct_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, hs,
                         (const double*)parts[j], ltiles[j], (int)n, len, (int)T, s + (long long)(first + j) * n);
      st = launch_status();
    }
  }
  return st;
}

namespace {
}  // namespace
}  // namespace dr

extern "C" size_t dr_update_workspace_size(const dr_layer* layers, int num_layers, int64_t n, int64_t T,
                                           dr_dtype dtype) {
  if (!layers || num_layers < 1 || n < 0 || T < 0) return 0;
  if (dtype != DR_BF16 && dtype != DR_F32) return 0;
  for (int l = 0; l < num_layers; ++l)
    if (layers[l].d_in < 1 || layers[l].d_out < 1) return 0;
  return dr::update_plan(layers, num_layers, n, T, dtype).bytes;
}

extern "C" dr_status dr_assemble_update(const dr_layer* layers, int num_layers, int64_t n, int64_t T,
                                        const int32_t* len, dr_dtype dtype, const float* w, int P, int64_t ldw,
                                        const int32_t* group_of_layer, float* U, const int64_t* u_offset,
                                        void* workspace, size_t ws_bytes, void* stream) {
  using namespace dr;
  dr_status st = validate_update(layers, num_layers, n, T, dtype, w, P, ldw, group_of_layer, U, u_offset);
  if (st != DR_OK) return st;
  const UpdPlan pl = update_plan(layers, num_layers, n, T, dtype);
  if (!workspace || ws_bytes < pl.bytes) return DR_ERR_WORKSPACE;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  int TO, TI;
  tile_dims(dtype, TO, TI);
  const int64_t es = dtype == DR_BF16 ? 2 : 4;
  const int nstride = n > 0 ? (int)n : 1;
  // one example list per distinct weight row, in order of first use
  int* layer_list = new int[num_layers];
  int* list_row = new int[num_layers];
  int nlists = 0;
  for (int l = 0; l < num_layers; ++l) {
    const int row = group_of_layer ? group_of_layer[l] : 0;
    int q = 0;
    while (q < nlists && list_row[q] != row) ++q;
    if (q == nlists) list_row[nlists++] = row;
    layer_list[l] = q;
  }
  UpdArgs base = {};
  base.split = pl.split;
  base.n = nstride;
  base.nw = (int)n;
  base.ex = reinterpret_cast<const int*>(ws + pl.off_ex);
  base.exlen = reinterpret_cast<const int*>(ws + pl.off_len);
  base.exw = reinterpret_cast<const float*>(ws + pl.off_w);
  base.uex = reinterpret_cast<int*>(ws + pl.off_uex);
  base.ulen = reinterpret_cast<int*>(ws + pl.off_ulen);
  base.uw = reinterpret_cast<float*>(ws + pl.off_uw);
  base.cnt = reinterpret_cast<const int*>(ws + pl.off_cnt);
  base.uniform = reinterpret_cast<int*>(ws + pl.off_uniform);
  base.pos = reinterpret_cast<int*>(ws + pl.off_pos);
  base.step = reinterpret_cast<UpdStep*>(ws + pl.off_step);
  base.max_steps = pl.max_steps;
  base.partial = reinterpret_cast<float*>(ws + pl.off_partial);
  // bf16: a packed step addresses its rows from its first example with 32-bit
  // offsets, and positions are 32-bit: when the whole batch spans less
  auto packed = [&](const dr_layer& L) {
    return n * T * (L.ldx > L.lddy ? L.ldx : L.lddy) * es < (int64_t)kOobOffset - 64;
  };
  // Calls of up to kSmallFlops leave every list to update_bf16_kernel: the
  // second tile kernel's launch, the step tables and the fill of its longer
  // pipeline cost more than its faster loop saves (32 to 64 examples of equal
  // weight, all and half of them: 17 GFLOP 2 to 30 % slower with both, 34 GFLOP
  // 4 %, 69 GFLOP 3 % faster, 137 GFLOP 12 %, 275 GFLOP 19 %, medians of 20 to
  // 56 shapes each).
  constexpr double kSmallFlops = 5e10;
  double flops = 0.0;
  for (int l = 0; l < num_layers; ++l) flops += 2.0 * (double)(n * T) * (double)(layers[l].d_in * layers[l].d_out);
  int modes = 0;
  if (pl.max_steps > 0 && flops > kSmallFlops)
    for (int l = 0; l < num_layers; ++l) modes |= packed(layers[l]) ? 2 : 1;
  for (int first = 0; first < nlists && st == DR_OK; first += kMaxUpdLayers) {
    const int count = nlists - first < kMaxUpdLayers ? nlists - first : kMaxUpdLayers;
    RowSel rs;
    for (int j = 0; j < kMaxUpdLayers; ++j) rs.r[j] = j < count ? list_row[first + j] : 0;
    if (n <= 1024)
      hipLaunchKernelGGL(update_list_kernel, dim3(count), dim3(1024), 0, hs, w, (long long)ldw, base, len, (int)T,
                         first, rs, modes);
    else
      hipLaunchKernelGGL(update_plan_kernel, dim3(count), dim3(1024), 0, hs, w, (long long)ldw, base, len, (int)T,
                         first, rs);
    st = launch_status();
  }
  if (st == DR_OK && n > 1024) {
    hipLaunchKernelGGL(update_sort_kernel, dim3((unsigned)((n + 255) / 256), nlists), dim3(256), 0, hs, base);
    hipLaunchKernelGGL(update_steps_kernel, dim3(nlists), dim3(1024), 0, hs, base, modes);
    st = launch_status();
  }
  for (int first = 0; first < num_layers && st == DR_OK; first += kMaxUpdLayers) {
    const int count = num_layers - first < kMaxUpdLayers ? num_layers - first : kMaxUpdLayers;
    UpdArgs a = base;
    int tiles = 0;
    for (int j = 0; j < count; ++j) {
      const dr_layer& L = layers[first + j];
      UpdLayerArg& la = a.L[j];
      la.x = static_cast<const unsigned char*>(L.x);
      la.dy = static_cast<const unsigned char*>(L.dy);
      la.ldx = L.ldx;
      la.lddy = L.lddy;
      la.exx = T * L.ldx * es;
      la.exdy = T * L.lddy * es;
      la.d_in = (int)L.d_in;
      la.d_out = (int)L.d_out;
      la.ti = (int)((L.d_in + TI - 1) / TI);
      la.tile0 = tiles;
      la.list = layer_list[first + j];
      la.U = U + u_offset[first + j];
      la.packed = packed(L);
      la.vec4 = aligned16(la.U);
      tiles += (int)(((L.d_out + TO - 1) / TO) * la.ti);
    }
    a.num_layers = count;
    a.ntiles = tiles;
    const int items = tiles * pl.split;
    const int grid = (items + 7) / 8 * 8;
    if (dtype == DR_BF16) {
      // each list's tiles are one kernel's work and the other's early exit:
      // which one is known on the device only
      if (modes) hipLaunchKernelGGL(update_tile_kernel, dim3(grid), dim3(256), 0, hs, a);
      hipLaunchKernelGGL(update_bf16_kernel<false>, dim3(grid), dim3(kBThreads), 0, hs, a);
    } else {
      hipLaunchKernelGGL(update_f32_kernel, dim3(grid), dim3(kFThreads), 0, hs, a);
    }
    if ((st = launch_status()) != DR_OK) break;
    if (pl.split > 1) {
      hipLaunchKernelGGL(update_reduce_kernel, dim3((TO * TI + 255) / 256, tiles), dim3(256), 0, hs, a, TO, TI);
      st = launch_status();
    }
  }
  delete[] layer_list;
  delete[] list_row;
  return st;
}
