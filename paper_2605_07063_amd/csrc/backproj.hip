// Back-projection of a sketch-space vector to parameter space
// (dr_back_project): for every layer with first-stage projectors P_in,
// P_out (second stage the identity), the transpose of the factorised
// compressor maps the layer's block x~ of a sketch-space vector to
//   U_l = P_out^T X' P_in,  X' = x~ as [k_out][k_in]     (d_out x d_in)
// (App. C.3, "Backward projection"), never forming Pi^T.  Applied to the
// sketch-space update u~ = G~^T w it gives the parameter-space update of the
// MeSO variant of the layer-wise algorithm.
//
// Up to 16 layers go in one launch (blockIdx.z = layer), so that the small
// per-layer grids fill the chip together.
//   bp_mfma_kernel   aligned bf16 projectors: both products in one kernel, T
//                    kept in LDS as three bf16 planes (see the kernel); else:
//   bp_left_kernel   T = X' P_in   [k_out][d_in] (small, workspace), one
//                    64-column slice of T per workgroup, fp32 MFMA (16x16x4)
//                    with both operands staged in LDS
//   bp_right_kernel  U = P_out^T T, one 64 (d_out) x 256 (d_in) tile per
//                    workgroup: each thread owns 16 rows x 4 columns, so a
//                    float4 of T read from L2 feeds 64 FMAs; the P_out columns
//                    of the tile sit in LDS.  The d_out x d_in fp32 write is
//                    the HBM bound.  (fp32 MFMA has the same peak as fp32
//                    FMA on this chip; staged or not, it measured slower here.)

#include "common.h"

namespace dr {
namespace {

constexpr int kBpLayers = 16;  // layers per launch (blockIdx.z)
constexpr int kBpTile = 64;    // columns of T per workgroup of bp_left_kernel
constexpr int kBpRows = 16;    // bp_right_kernel: rows per wave (4 waves: 64 rows per tile)
constexpr int kBpCols = 256;   // bp_right_kernel: columns per tile (4 per lane)
constexpr int kBpMaxK = 64;
constexpr int kBpLd = 132;     // LDS row stride (floats)

template <typename TP>
__device__ __forceinline__ float ld(const TP* p, long long i) {
  return (float)p[i];
}

struct BpArgs {
  const void* p_in[kBpLayers];
  const void* p_out[kBpLayers];
  const float* x[kBpLayers];   // the layer's block of the sketch-space vector
  float* T[kBpLayers];         // [k_out][d_in] workspace
  float* U[kBpLayers];         // [d_out][d_in] output
  int k_in[kBpLayers], k_out[kBpLayers], d_in[kBpLayers], d_out[kBpLayers];
};

// T[a][c] = sum_b X'[a][b] P_in[b][c] for c in this workgroup's 64 columns;
// a < k_out <= 64 (4 row tiles), 4 column tiles: wave w takes column tile w
// of every row tile.  Rows and columns past k_in / k_out /
// d_in are zero in LDS.
template <typename TP>
__global__ __launch_bounds__(256) void bp_left_kernel(BpArgs g) {
  __shared__ __attribute__((aligned(16))) float xs[kBpMaxK * 68];   // X'[a][b], stride 68
  __shared__ __attribute__((aligned(16))) float ps[kBpMaxK * kBpLd];   // P_in[b][c - c0]
  const int l = blockIdx.z;
  const int k_in = g.k_in[l], k_out = g.k_out[l], d_in = g.d_in[l];
  const int c0 = blockIdx.x * kBpTile;
  if (c0 >= d_in) return;
  const float* x = g.x[l];
  const TP* p_in = static_cast<const TP*>(g.p_in[l]);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lq = lane >> 4;
  {
    // every load of the thread in flight before the LDS writes
    float xv[kBpMaxK * kBpMaxK / 256], pv[kBpMaxK * kBpTile / 256];
#pragma unroll
    for (int u = 0; u < kBpMaxK * kBpMaxK / 256; ++u) {
      const int e = tid + 256 * u, a = e >> 6, b = e & 63;
      xv[u] = (a < k_out && b < k_in) ? x[a * k_in + b] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kBpMaxK * kBpTile / 256; ++u) {
      const int e = tid + 256 * u, b = e / kBpTile, c = e % kBpTile;
      pv[u] = (b < k_in && c0 + c < d_in) ? ld(p_in, (long long)b * d_in + c0 + c) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kBpMaxK * kBpMaxK / 256; ++u) {
      const int e = tid + 256 * u;
      xs[(e >> 6) * 68 + (e & 63)] = xv[u];
    }
#pragma unroll
    for (int u = 0; u < kBpMaxK * kBpTile / 256; ++u) {
      const int e = tid + 256 * u;
      ps[(e / kBpTile) * kBpLd + e % kBpTile] = pv[u];
    }
  }
  __syncthreads();
  f32x4 acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int kq = (k_in + 3) & ~3;
  for (int b0 = 0; b0 < kq; b0 += 4) {
    const float bv = ps[(b0 + lq) * kBpLd + 16 * w + lr];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = mma_f32(xs[(16 * i + lr) * 68 + b0 + lq], bv, acc[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int a = 16 * i + 4 * lq + q, c = c0 + 16 * w + lr;
      if (a >= k_out || c >= d_in) continue;
      const float t = acc[i][q];
      g.T[l][(long long)a * d_in + c] = t;
    }
}

// U[o][c] = sum_a P_out[a][o] T[a][c] for a 64 (d_out) x 256 (d_in) tile:
// wave v owns rows 16 v .. 16 v + 15, lane l columns 4 l .. 4 l + 3; the
// tile's P_out columns sit in LDS (every lane of a wave reads the same four
// 16-byte words per a: broadcasts), T comes from L2 as float4.
template <typename TP>
__global__ __launch_bounds__(256) void bp_right_kernel(BpArgs g) {
  __shared__ __attribute__((aligned(16))) float po[kBpMaxK][kBpRows * 4];
  const int l = blockIdx.z;
  const int k_out = g.k_out[l], d_out = g.d_out[l], d_in = g.d_in[l];
  const TP* p_out = static_cast<const TP*>(g.p_out[l]);
  const float* T = g.T[l];
  float* U = g.U[l];
  const int o0 = blockIdx.y * (kBpRows * 4);
  if (o0 >= d_out || blockIdx.x * kBpCols >= d_in) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int v = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = blockIdx.x * kBpCols + 4 * lane;
  for (int e = tid; e < k_out * kBpRows * 4; e += 256) {
    const int a = e / (kBpRows * 4), r = e % (kBpRows * 4);
    po[a][r] = o0 + r < d_out ? ld(p_out, (long long)a * d_out + o0 + r) : 0.f;
  }
  __syncthreads();
  if (c >= d_in) return;
  float4 acc[kBpRows];
#pragma unroll
  for (int r = 0; r < kBpRows; ++r) acc[r] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int a0 = 0; a0 < k_out; a0 += 8) {   // eight rows of T in flight before the FMAs
    float4 tv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      tv[e] = a0 + e < k_out ? *reinterpret_cast<const float4*>(T + (long long)(a0 + e) * d_in + c)
                             : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (a0 + e >= k_out) break;
      const float4 t = tv[e];
      const float4* pr = reinterpret_cast<const float4*>(&po[a0 + e][kBpRows * v]);
#pragma unroll
      for (int q = 0; q < kBpRows / 4; ++q) {
        const float4 pq = pr[q];
        const float pv[4] = {pq.x, pq.y, pq.z, pq.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float4& A = acc[4 * q + u];
          A.x = fmaf(pv[u], t.x, A.x);
          A.y = fmaf(pv[u], t.y, A.y);
          A.z = fmaf(pv[u], t.z, A.z);
          A.w = fmaf(pv[u], t.w, A.w);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kBpRows; ++r) {
    const int o = o0 + kBpRows * v + r;
    if (o < d_out) *reinterpret_cast<float4*>(U + (long long)o * d_in + c) = acc[r];
  }
}

__device__ __forceinline__ float bf16_val(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
__device__ __forceinline__ float bf16_lo(unsigned h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ float bf16_hi(unsigned h) { return __uint_as_float(h & 0xffff0000u); }

// bf16 projectors (P_out 16-byte aligned, d_in and d_out multiples of 8), both
// products in one kernel: a workgroup takes 128 columns of U and `per` tiles
// of 128 rows.  It makes T = X' P_in of its columns once (fp32 MFMA 16x16x4,
// k_out x 128, P_in and X' staged in LDS) and leaves it in LDS as three bf16
// planes T1 + T2 + T3 = T (each the nearest bf16 to what the previous ones
// leave; the sum is T to about 2^-24).  Then, tile by tile, U = P_out^T (T1 +
// T2 + T3) is one bf16 MFMA contraction over 3 * k_out rows (each product
// exact in fp32, fp32 accumulation): P_out[:, o-tile] goes to LDS beside the
// planes (64 rows of 256 bytes each, 32-byte slots XOR-swizzled per row), all
// read as MFMA operands by the gfx950 transposing read (8 consecutive rows a
// per lane); the next tile's P_out is loaded under the products.  Wave (wr,
// wc) holds a 64 x 64 quarter.  T's columns are the rows of the MFMA tile, so
// a lane ends up with four neighbouring columns of a row of U; 16 rows at a
// time go through 4 KB of LDS of the wave's own, so that a store writes whole
// 256-byte pieces of rows.
// The d_out x d_in fp32 write is the bound, with the start of a workgroup (P_in
// and X' from memory, T) before its first store: 8 layers of 2048 x 2048 in 35
// us and 16 of 4096 x 14336 in 745 us (a fill of U: 21 and 545), 47 and 987
// with T made by a launch of its own, read back by every tile and results
// staged through LDS 128 rows at a time.  Stores straight from the registers
// (64-byte pieces) 39 and 840; one row tile per workgroup 70 and 1700.
constexpr int kBmTile = 128;
constexpr int kBmRow = kBmTile * 2;          // bytes of one staged row
constexpr int kBmSlab = kBpMaxK * kBmRow;    // 16 KB: one operand slab
constexpr int kBmXLd = kBpMaxK + 4;          // X' staging stride (floats)
constexpr int kBmLds = 4 * kBmSlab + 4 * 16 * 64 * 4;   // 80 KB: + 16 x 64 results per wave
constexpr int kBmGroups = 512;               // workgroups that fill the chip (two per CU)
constexpr int kBmMaxPer = 32;                // row tiles per workgroup

__global__ __launch_bounds__(256, 2) void bp_mfma_kernel(BpArgs g, int per) {
  // slab 0: P_out of the row tile; slabs 1..3: the planes of T.  P_in and X'
  // lie there first.
  __shared__ __attribute__((aligned(16))) unsigned char lds[kBmLds];
  const int l = blockIdx.z;
  const int k_in = g.k_in[l], k_out = g.k_out[l], d_out = g.d_out[l], d_in = g.d_in[l];
  const int c0 = blockIdx.x * kBmTile;
  const int tiles = (d_out + kBmTile - 1) / kBmTile;
  const int t0 = blockIdx.y * per, t1 = t0 + per < tiles ? t0 + per : tiles;
  if (t0 >= tiles || c0 >= d_in) return;
  const unsigned short* pg = static_cast<const unsigned short*>(g.p_out[l]);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, g4 = lane >> 4;
  // a 16-byte chunk of the P_out slab per step: row (tid >> 4) + 16 u, columns 8 (tid & 15) ..
  const int pr = tid >> 4, pc = 8 * (tid & 15);
  u32x4 pv[4];
  auto load_p = [&](const unsigned short* src, int k, int x0, int d) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = pr + 16 * u;
      pv[u] = r < k && x0 + pc < d ? *reinterpret_cast<const u32x4*>(src + (long long)r * d + x0 + pc)
                                   : u32x4{0u, 0u, 0u, 0u};
    }
  };
  // T of these 128 columns
  {
    unsigned short* ps = reinterpret_cast<unsigned short*>(lds);        // P_in[b][c - c0], 256 bytes per row
    float* xs = reinterpret_cast<float*>(lds + kBmSlab);                // X'[a][b]
    const float* x = g.x[l];
    float xv[kBpMaxK * kBpMaxK / 256];
    const unsigned short* pi = static_cast<const unsigned short*>(g.p_in[l]);
    if ((reinterpret_cast<uintptr_t>(pi) & 15) == 0) {
      load_p(pi, k_in, c0, d_in);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = pr + 16 * u;
        const bool ok = r < k_in && c0 + pc < d_in;
        const unsigned short* q = pi + (ok ? (long long)r * d_in + c0 + pc : 0);
        // (q[0 .. 7] is inside P_in also where it stands for nothing: d_in >= 8)
#pragma unroll
        for (int v = 0; v < 4; ++v) pv[u][v] = ok ? q[2 * v] | (unsigned)q[2 * v + 1] << 16 : 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < kBpMaxK * kBpMaxK / 256; ++u) {
      const int e = tid + 256 * u, a = e >> 6, b = e & 63;
      xv[u] = (a < k_out && b < k_in) ? x[a * k_in + b] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) *reinterpret_cast<u32x4*>(ps + (pr + 16 * u) * kBmTile + pc) = pv[u];
#pragma unroll
    for (int u = 0; u < kBpMaxK * kBpMaxK / 256; ++u) {
      const int e = tid + 256 * u;
      xs[(e >> 6) * kBmXLd + (e & 63)] = xv[u];
    }
    load_p(pg, k_out, t0 * kBmTile, d_out);   // the first row tile, under T
    __syncthreads();
    f32x4 t[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) t[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int b1 = 0; b1 < k_in; b1 += 16) {   // rows past k_in are zero
#pragma unroll
      for (int b0 = b1; b0 < b1 + 16; b0 += 4) {
        float av[2], bv[4];
#pragma unroll
        for (int i = 0; i < 2; ++i) av[i] = bf16_val(ps[(b0 + g4) * kBmTile + 32 * w + 16 * i + lr]);
#pragma unroll
        for (int j = 0; j < 4; ++j) bv[j] = xs[(16 * j + lr) * kBmXLd + b0 + g4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) t[i][j] = mma_f32(av[i], bv[j], t[i][j]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int a = 16 * j + lr;   // columns 32 w + 16 i + 4 g4 .. + 3 of row a: slot 2 w + i
        unsigned char* at = lds + kBmSlab + a * kBmRow + ((2 * w + i) ^ slot_xor(a)) * 32 + g4 * 8;
        f32x4 v = t[i][j];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const uint2 h = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
          *reinterpret_cast<uint2*>(at + p * kBmSlab) = h;
          v -= f32x4{bf16_lo(h.x), bf16_hi(h.x), bf16_lo(h.y), bf16_hi(h.y)};
        }
      }
  }
  // fragment reads: lane (g4, q, rr) of the transposing read addresses row
  // 8 g4 + q (+4 for the second half) and 8-byte piece rr of a 16-column
  // block; the block's logical slot is XOR-ed with the row's swizzle
  const int q4 = (lane >> 2) & 3, rr = lane & 3;
  const int fx = q4 | ((g4 & 1) << 2);
  const int wr = w >> 1, wc = w & 1;
  const unsigned rbase = (unsigned)((8 * g4 + q4) * kBmRow + rr * 8);
  unsigned offp[4], offt[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) offp[j] = rbase + (unsigned)(((4 * wr + j) ^ fx) * 32);
#pragma unroll
  for (int i = 0; i < 4; ++i) offt[i] = rbase + (unsigned)(((4 * wc + i) ^ fx) * 32);
  auto frag = [&](const unsigned char* base) {
    const v4s lo = lds_read_tr16(base);
    const v4s hi = lds_read_tr16(base + 4 * kBmRow);
    return u32x4{__builtin_bit_cast(uint2, lo).x, __builtin_bit_cast(uint2, lo).y, __builtin_bit_cast(uint2, hi).x,
                 __builtin_bit_cast(uint2, hi).y};
  };
  const int nh = k_out > 32 ? 2 : 1;   // 32-row slices of the sketch index a (rows >= k_out are zero)
  float* U = g.U[l];
  for (int t = t0; t < t1; ++t) {
    const int o0 = t * kBmTile;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = pr + 16 * u, ch = tid & 15;
      *reinterpret_cast<u32x4*>(lds + r * kBmRow + (((ch >> 1) ^ slot_xor(r)) * 32) + (ch & 1) * 16) = pv[u];
    }
    __syncthreads();
    if (t + 1 < t1) load_p(pg, k_out, o0 + kBmTile, d_out);
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int h = 0; h < nh; ++h) {
      u32x4 fp[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) fp[j] = frag(lds + h * 32 * kBmRow + offp[j]);
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        u32x4 ft[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ft[i] = frag(lds + (1 + p) * kBmSlab + h * 32 * kBmRow + offt[i]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = mma_bf16(ft[i], fp[j], acc[i][j]);
      }
    }
    __syncthreads();   // the P_out slab may be replaced
    float* st = reinterpret_cast<float*>(lds + 4 * kBmSlab + w * 4096);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(st + lr * 64 + (((4 * i + g4) ^ lr) * 4)) = acc[i][j];
      // other lanes of the wave read what this one wrote, and write there next
      // (LDS keeps a wave's order; this keeps the compiler to it)
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * i + g4, o = o0 + 64 * wr + 16 * j + r, c = c0 + 64 * wc + 4 * lr;
        const f32x4 v = *reinterpret_cast<const f32x4*>(st + r * 64 + ((lr ^ r) * 4));
        if (o < d_out && c < d_in) *reinterpret_cast<f32x4*>(U + (long long)o * d_in + c) = v;
      }
      asm volatile("" ::: "memory");
    }
  }
}

}  // namespace
}  // namespace dr

extern "C" size_t dr_backproject_workspace_size(const dr_layer* layers, int num_layers) {
  if (!layers || num_layers < 1) return 0;
  // one launch holds up to 16 layers: room for the largest such run of T blocks
  // (aligned bf16 projectors leave it unused: their kernel keeps T in LDS)
  size_t best = 256;
  for (int f = 0; f < num_layers; f += dr::kBpLayers) {
    size_t o = 0;
    for (int l = f; l < num_layers && l < f + dr::kBpLayers; ++l)
      o = dr::align_up(o + (size_t)(layers[l].k_out > 0 ? layers[l].k_out : 0) *
                               (size_t)(layers[l].d_in > 0 ? layers[l].d_in : 0) * sizeof(float), 256);
    best = o > best ? o : best;
  }
  return best;
}

extern "C" dr_status dr_back_project(const dr_layer* layers, int num_layers, dr_dtype dtype, const float* u, float* U,
                                     const int64_t* u_offset, void* workspace, size_t ws_bytes, void* stream) {
  using namespace dr;
  if (dtype != DR_BF16 && dtype != DR_F32) return DR_ERR_DTYPE;
  if (!layers || num_layers < 1 || !u || !U || !u_offset) return DR_ERR_ARG;
  for (int l = 0; l < num_layers; ++l) {
    const dr_layer& L = layers[l];
    if (L.k_in < 1 || L.k_out < 1 || L.k_in > kBpMaxK || L.k_out > kBpMaxK) return DR_ERR_ARG;
    if (L.d_in < 1 || L.d_out < 1 || L.d_in > (1 << 28) || L.d_out > (1 << 28)) return DR_ERR_ARG;
    if (!L.p_in || !L.p_out || L.col_offset < 0 || u_offset[l] < 0) return DR_ERR_ARG;
    if ((L.d_out + 4 * kBpRows - 1) / (4 * kBpRows) > 65535) return DR_ERR_UNSUPPORTED;   // grid rows
    if (L.d_in % 4 || !aligned16(U + u_offset[l])) return DR_ERR_ARG;   // float4 columns and stores
  }
  if (!workspace || ws_bytes < dr_backproject_workspace_size(layers, num_layers)) return DR_ERR_WORKSPACE;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  for (int f = 0; f < num_layers; f += kBpLayers) {
    const int count = num_layers - f < kBpLayers ? num_layers - f : kBpLayers;
    BpArgs g = {};
    int dimax = 1, domax = 1;
    bool mfma = dtype == DR_BF16;
    size_t o = 0;
    long long tiles = 0;
    for (int j = 0; j < count; ++j) {
      const dr_layer& L = layers[f + j];
      g.p_in[j] = L.p_in;
      g.p_out[j] = L.p_out;
      g.x[j] = u + L.col_offset;
      g.T[j] = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + o);
      o = align_up(o + (size_t)L.k_out * (size_t)L.d_in * sizeof(float), 256);
      mfma = mfma && L.d_in % 8 == 0 && L.d_out % 8 == 0 && aligned16(L.p_out);
      g.U[j] = U + u_offset[f + j];
      g.k_in[j] = (int)L.k_in;
      g.k_out[j] = (int)L.k_out;
      g.d_in[j] = (int)L.d_in;
      g.d_out[j] = (int)L.d_out;
      dimax = g.d_in[j] > dimax ? g.d_in[j] : dimax;
      domax = g.d_out[j] > domax ? g.d_out[j] : domax;
      tiles += (long long)((g.d_in[j] + kBmTile - 1) / kBmTile) * ((g.d_out[j] + kBmTile - 1) / kBmTile);
    }
    const dim3 gl((dimax + kBpTile - 1) / kBpTile, 1, count);
    const dim3 gr((dimax + kBpCols - 1) / kBpCols, (domax + 4 * kBpRows - 1) / (4 * kBpRows), count);
    if (mfma) {
      // row tiles per workgroup: as many as leave about two workgroups per CU
      // (T is made once for all of them), the same for each
      const int rows = (domax + kBmTile - 1) / kBmTile;
      const long long want = (tiles + kBmGroups - 1) / kBmGroups;
      int per = want < kBmMaxPer ? (int)want : kBmMaxPer;
      per = per < rows ? per : rows;
      const int parts = (rows + per - 1) / per;
      per = (rows + parts - 1) / parts;
      const dim3 gm((dimax + kBmTile - 1) / kBmTile, (rows + per - 1) / per, count);
      hipLaunchKernelGGL(bp_mfma_kernel, gm, dim3(256), 0, hs, g, per);
    } else if (dtype == DR_BF16) {
      hipLaunchKernelGGL(bp_left_kernel<__bf16>, gl, dim3(256), 0, hs, g);
      hipLaunchKernelGGL(bp_right_kernel<__bf16>, gr, dim3(256), 0, hs, g);
    } else {
      hipLaunchKernelGGL(bp_left_kernel<float>, gl, dim3(256), 0, hs, g);
      hipLaunchKernelGGL(bp_right_kernel<float>, gr, dim3(256), 0, hs, g);
    }
    const dr_status st = launch_status();
    if (st != DR_OK) return st;
  }
  return DR_OK;
}
