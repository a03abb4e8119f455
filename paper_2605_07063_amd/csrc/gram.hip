// Target mean, Gram matrix and alignment scores per parameter group (dr_gram).
//
// Per group p (a column range of the sketch matrix, Sec. 3.3.3):
//   gbar_p = mean of the m target rows            (Sec. 3.2)
//   K_p    = G_p G_p^T                             (redundancy term, Sec. 3.3.2)
//   s_p    = G_p gbar_p,  t2_p = ||gbar_p||^2      (alignment scores)
//
// Kernels
//   target_mean_kernel : gbar in fp32 (fp64 sum over the m rows).
//   gram_tile_kernel   : bf16 rows: one 64x64 tile of K_p over one chunk of
//                        the group's columns (lower-triangle tile pairs only),
//                        bf16 16x16x32 MFMA, fp32 accumulate; operands stream
//                        from memory straight into registers.
//   gram_tile_lds_kernel : fp32 rows, the same tiles and chunks on fp32 MFMA,
//                        operands staged through LDS; the target mean joins
//                        the diagonal tiles as a further row, so s_p and t2_p
//                        come out of the same pass.
//   gram_split_kernel  : fp32 rows, larger problems: 256-row tiles of K_p over one chunk of the
//                        group's columns, each value split into three bf16
//                        parts and each product taken as six bf16 MFMAs.  A
//                        diagonal tile also forms the target mean of its
//                        columns, the scores s_p of its rows and (tile 0)
//                        t2_p, so the same pass yields them.
//   gram_reduce_kernel : sums the chunk partials of a 64x64 tile in fp64 and
//                        writes the lower triangle and its mirror, so K is
//                        exactly symmetric, and for fp32 sketches s_p and
//                        t2_p from the diagonal tiles.
//   score_kernel       : s_p[i] = <G_p[i], gbar_p> and t2_p against the fp32
//                        mean, fp64 accumulation, fixed-order block
//                        reduction: bf16 sketches, and t2_p of fp32 ones
//                        with n = 0.
// Large bf16 problems (at least kBigMinTiles 256x256 lower-triangle tiles):
//   gram_big_kernel    : one 256x256 tile of K_p per workgroup over all of
//                        the group's columns (no split): 64-column steps
//                        stream into a two-stage LDS ring by buffer->LDS DMA,
//                        four waves (one per SIMD) each hold a 128x128 fp32
//                        accumulator in AGPRs (bf16 16x16x32 MFMA); lower-
//                        triangle tiles only, scheduled in 4x8-tile chunks,
//                        one per XCD at a time.  Each tile goes out from
//                        registers in non-temporal float4 stores, also
//                        transposed into the upper triangle, so K is exactly
//                        symmetric without a second pass.
// Small fp32 problems (n + 1 <= 128 rows: the per-step batches):
//   gram_small_kernel  : one workgroup per 128-column chunk of a group forms
//                        the chunk of gbar from the target rows (fp64 sum /
//                        m, as target_mean_kernel) and stages the n + 1
//                        augmented rows in LDS (row stride 132 floats: the
//                        16 rows x 4 columns of an fp32 MFMA operand fall on
//                        distinct banks); the eight waves take the lower
//                        16x16 blocks of the augmented Gram round-robin
//                        (fp32 16x16x4 MFMA) and write chunk partials, a
//                        block's 256 values side by side.
//   gram_small_reduce_kernel : sums the chunk partials (a lane per element, a
//                        fixed order) into K (both triangles), s (row n) and
//                        t2 (element n, n).
// No atomics: results are deterministic.

#include <cmath>
#include <mutex>
#include <type_traits>

#include "tile256.h"

namespace dr {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 64;
constexpr int kMaxGroups = 256;   // groups per launch (more groups -> more launches)
constexpr int kTargetWGs = 1024;
constexpr int kLdsSlots = 256 * 3;   // gram_tile_lds_kernel workgroups resident at once: 256 CUs x 3 (48 KB of LDS each)
constexpr int kSplitSlots = 256;     // gram_split_kernel workgroups resident at once (one per CU)
constexpr int64_t kSplitPartials = (int64_t)44 << 20;   // bytes of its chunk partials

struct GramArgs {
  const unsigned char* G;
  long long ldG;
  int n;
  int rows;                         // rows of the Gram problem: n, or n + 1 with gbar as row n
  const float* gbar;                // [cols] by absolute column (row n when rows == n + 1)
  long long goff[kMaxGroups + 1];   // absolute column offsets of this launch's groups
  int P;
  int NT, pairs, CK, maxchunks;
  float* partial;                   // [P][pairs][maxchunks][kTile*kTile]
  float* K;                         // outputs (the fp32 tile kernels write them themselves
  float* s;                         // when maxchunks == 1); group p of the launch is pbase + p
  float* t2;
  long long pbase;
  int vec4;                         // rows of K start 16-byte aligned
  const float* Gt;                  // fp32 target rows (gram_split_kernel forms their mean itself)
  long long ldGt;
  int m;
};

template <bool BF16>
struct GTr;
template <>
struct GTr<true> {
  static constexpr int ES = 2, EPV = 8, KV = 32;   // KV: columns per 16-byte vector per lane group
};
template <>
struct GTr<false> {
  static constexpr int ES = 4, EPV = 4, KV = 16;
};

template <bool BF16>
__device__ __forceinline__ f32x4 mma_v(u32x4 a, u32x4 b, f32x4 c) {
  if constexpr (BF16) {
    return mma_bf16(a, b, c);
  } else {
    c = mma_f32(__uint_as_float(a.x), __uint_as_float(b.x), c);
    c = mma_f32(__uint_as_float(a.y), __uint_as_float(b.y), c);
    c = mma_f32(__uint_as_float(a.z), __uint_as_float(b.z), c);
    c = mma_f32(__uint_as_float(a.w), __uint_as_float(b.w), c);
    return c;
  }
}

__device__ __forceinline__ void pair_to_tiles(int q, int& I, int& J) {
  int i = (int)((sqrtf(8.f * q + 1.f) - 1.f) * 0.5f);
  while ((i + 1) * (i + 2) / 2 <= q) ++i;
  while (i * (i + 1) / 2 > q) --i;
  I = i;
  J = q - i * (i + 1) / 2;
}

__global__ __launch_bounds__(kThreads, 2) void gram_tile_kernel(GramArgs a) {
  using E = GTr<true>;
  constexpr int NV = 2;              // vectors per row-block per step
  constexpr int STEP = NV * 4 * E::EPV;   // columns per step (4 lane groups)
  const int chunk = blockIdx.x, q = blockIdx.y, p = blockIdx.z;
  const long long g0 = a.goff[p], g1 = a.goff[p + 1];
  const long long c0 = g0 + (long long)chunk * a.CK;
  if (c0 >= g1) return;
  const long long c1 = c0 + a.CK < g1 ? c0 + a.CK : g1;
  int I, J;
  pair_to_tiles(q, I, J);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wr = wave >> 1, wc = wave & 1;

  int rowA[2], rowB[2];
  bool okA[2], okB[2];
  const unsigned char* baseA[2];
  const unsigned char* baseB[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    rowA[b] = I * kTile + wr * 32 + b * 16 + lr;
    rowB[b] = J * kTile + wc * 32 + b * 16 + lr;
    okA[b] = rowA[b] < a.n;
    okB[b] = rowB[b] < a.n;
    baseA[b] = a.G + (long long)rowA[b] * a.ldG * E::ES;
    baseB[b] = a.G + (long long)rowB[b] * a.ldG * E::ES;
  }

  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto load = [&](long long cs, u32x4 (&va)[2][NV], u32x4 (&vb)[2][NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const long long c = cs + (long long)v * 4 * E::EPV + lg * E::EPV;
      const bool cok = c < c1;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // unconditional loads (an entry outside the problem reads the first
        // 16 bytes of the target mean instead, which every call has: G may
        // be empty, and then null; the value is then zeroed), so that the
        // compiler's waits count the loads in flight
        const unsigned char* dummy = reinterpret_cast<const unsigned char*>(a.gbar);
        const bool ea = okA[b] && cok, eb = okB[b] && cok;
        const u32x4 xa = *reinterpret_cast<const u32x4*>(ea ? baseA[b] + c * E::ES : dummy);
        const u32x4 xb = *reinterpret_cast<const u32x4*>(eb ? baseB[b] + c * E::ES : dummy);
        va[b][v] = ea ? xa : u32x4{0u, 0u, 0u, 0u};
        vb[b][v] = eb ? xb : u32x4{0u, 0u, 0u, 0u};
      }
    }
  };

  // DEPTH steps of loads in flight: the operands come from L2 straight
  // into registers, so their latency is what the products wait for; loads
  // past the chunk read zeros (no memory access), whose products add 0
  constexpr int DEPTH = 3;
  u32x4 ba[DEPTH][2][NV], bb[DEPTH][2][NV];
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d) load(c0 + (long long)d * STEP, ba[d], bb[d]);
  for (long long cs = c0; cs < c1; cs += DEPTH * STEP) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      load(cs + (long long)(d + DEPTH - 1) * STEP, ba[(d + DEPTH - 1) % DEPTH], bb[(d + DEPTH - 1) % DEPTH]);
      // the loads go out before this step's products (the scheduler would
      // otherwise move them next to their uses)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mma_v<true>(ba[d][i][v], bb[d][j][v], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  float* out = a.partial + (((long long)p * a.pairs + q) * a.maxchunks + chunk) * (kTile * kTile);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(wr * 32 + i * 16 + lg * 4 + r) * kTile + wc * 32 + j * 16 + lr] = acc[i][j][r];
}


// One 16x16 block of C (lane l holds C[4 (l / 16) + r][l % 16] in element r)
// into K at rows R.., columns C.. and, mirrored, at rows C.., columns R..,
// for an off-diagonal tile inside K with 16-byte aligned rows: every element
// goes out in non-temporal float4 stores.  The mirror is the accumulator as
// it stands (four consecutive rows of one column are four consecutive
// columns of the transposed row); the block itself after a 4 x 4 transpose
// inside each quad of lanes.
__device__ __forceinline__ void big_store_block_fast(float* Kp, int n, int R, int C, f32x4 v, int lane) {
  const int lr = lane & 15, lg = lane >> 4, c = lane & 3, m = lr >> 2;
  __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(Kp + (long long)(C + lr) * n + R + 4 * lg));
  __builtin_nontemporal_store(quad_transpose(v),
                              reinterpret_cast<f32x4*>(Kp + (long long)(R + 4 * lg + c) * n + C + 4 * m));
}

// fp32 rows, n + 1 > 128, where the 256-row tiles below would leave the chip
// idle or spend themselves on a short last tile (lds_tiles_time): 64 x 64
// tile pairs over the n general rows, with the operands staged through LDS.  Per step of 32 columns the workgroup's
// rows are loaded once into registers (16-byte segments), written to a
// three-stage LDS ring in the conflict-free operand layout, and read by the
// four waves as fp32 MFMA fragments; loads run two steps ahead of their LDS
// writes, and the LDS writes one step ahead of the products.  A step's
// products are summed from zero and then added (one chain of MFMAs over a
// chunk had errors of 1.9e-7 to 5.1e-7 against 64 bits).
//   off-diagonal pair (I > J): tile I's 64 rows, then tile J's 64 rows;
//   diagonal pair (I = J): tile I's 64 rows once (they are both operands),
//     then the target mean as a 16-row block whose other rows are zero.
//     Waves (0, 0), (1, 0) and (1, 1) take the tile's lower triangle; wave
//     (0, 1), whose quadrant lies above the diagonal, takes the target mean
//     against the 64 rows (the scores s), and in tile 0 wave (0, 0) also
//     takes the target mean against itself (t2).  Both land in the partial
//     tile's upper triangle, which holds nothing else: s of tile row
//     16 b + l at (16 (b / 2), 32 + 16 (b % 2) + l), t2 at (0, 16).
constexpr int kLS = 32;                          // fp32 columns per step (128-byte rows)
constexpr int kLNS = 3;                          // ring stages
constexpr int kLStage = 2 * kTile * kLS * 4;     // 128 rows of 128 bytes
constexpr int kLMeanRow = kTile;                 // diagonal pairs: the target mean's stage row
constexpr int kKindS = 16, kKindT2 = 17;         // wave tasks beyond the block masks 0..15

__global__ __launch_bounds__(kThreads, 2) void gram_tile_lds_kernel(GramArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kLNS * kLStage];
  const int chunk = blockIdx.x, q = blockIdx.y, p = blockIdx.z;
  const long long g0 = a.goff[p], g1 = a.goff[p + 1];
  const long long c0 = g0 + (long long)chunk * a.CK;
  // with one chunk per group the tile is final and written here, so an
  // empty group still writes its zeros (no steps)
  const bool direct = a.maxchunks == 1;
  if (c0 >= g1 && !direct) return;
  const long long c1 = c0 + a.CK < g1 ? c0 + a.CK : g1;
  const int nsteps = c1 > c0 ? (int)((c1 - c0 + kLS - 1) / kLS) : 0;
  int I, J;
  pair_to_tiles(q, I, J);
  const bool diag = I == J;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int wr = w >> 1, wc = w & 1;
  // loader: segment e = tid + 256 u of a stage is stage row e / 8, segment
  // e % 8 (an off-diagonal pair loads u = 0..3, a diagonal one u = 0..2).
  // An entry outside the problem reads the target mean's first 16 bytes
  // instead and is zeroed at the LDS write, so the loads are unconditional
  // and their waits counted.
  const unsigned char* mean = reinterpret_cast<const unsigned char*>(a.gbar);   // by absolute column
  const unsigned char* src[4];
  bool rok[4];
  int sseg[4];
  unsigned loff[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int e = tid + kThreads * u, R = e >> 3, sg = e & 7;
    if (R < kTile || !diag) {
      const int grow = R < kTile ? I * kTile + R : J * kTile + (R - kTile);
      rok[u] = grow < a.n;
      src[u] = rok[u] ? a.G + (long long)grow * a.ldG * 4 : mean;
    } else {
      rok[u] = R == kLMeanRow;
      src[u] = mean;
    }
    sseg[u] = sg;
    loff[u] = (unsigned)(R * 128 + ((sg ^ ((R >> 1) & 7)) * 16));
  }
  auto seg_ok = [&](int t, int u) { return rok[u] && c0 + (long long)t * kLS + sseg[u] * 4 < c1; };
  // the zeroing happens at the LDS write, so nothing waits for the loads
  // until then
  auto gload = [&](int t, u32x4 (&v)[4], auto nu) {
#pragma unroll
    for (int u = 0; u < decltype(nu)::value; ++u) {
      const long long c = c0 + (long long)t * kLS + sseg[u] * 4;
      v[u] = *reinterpret_cast<const u32x4*>(seg_ok(t, u) ? src[u] + c * 4 : mean);
    }
  };
  auto lstore = [&](int t, const u32x4 (&v)[4], auto nu) {
    unsigned char* sb = lds + (t % kLNS) * kLStage;
#pragma unroll
    for (int u = 0; u < decltype(nu)::value; ++u)
      *reinterpret_cast<u32x4*>(sb + loff[u]) = seg_ok(t, u) ? v[u] : u32x4{0u, 0u, 0u, 0u};
  };
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the wave's products of step t.  Kind 0..15: the 16 x 16 blocks (i, j)
  // whose bit i * 2 + j is set (A block i against B block j); kKindT2: mask
  // 13 plus the target mean against itself into acc[0][1]; kKindS: the
  // target mean against the tile's four 16-row blocks into acc[b / 2][b % 2]
  auto compute = [&](int t, auto kind, auto dg) {
    constexpr int KD = decltype(kind)::value;
    constexpr bool DG = decltype(dg)::value;
    if constexpr (KD != 0) {
      const unsigned char* sb = lds + (t % kLNS) * kLStage;
      const unsigned char* bb = sb + (DG ? 0 : kTile * 128);   // B operand rows
      f32x4 sum[2][2];
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        const int sg = 4 * kh + lg;
        if constexpr (KD == kKindS) {
          const u32x4 fm = swz_read(sb + kLMeanRow * 128, lr, sg);
          u32x4 fb[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) fb[b] = swz_read(sb + 16 * b * 128, lr, sg);
          sum[0][0] = mma_v<false>(fm, fb[0], sum[0][0]);
          sum[0][1] = mma_v<false>(fm, fb[1], sum[0][1]);
          sum[1][0] = mma_v<false>(fm, fb[2], sum[1][0]);
          sum[1][1] = mma_v<false>(fm, fb[3], sum[1][1]);
        } else {
          constexpr int M = KD == kKindT2 ? 13 : KD;
          constexpr bool ra0 = (M & 3) != 0, ra1 = (M & 12) != 0, rb0 = (M & 5) != 0, rb1 = (M & 10) != 0;
          u32x4 fa[2], fb[2];
          if constexpr (ra0) fa[0] = swz_read(sb + (wr * 32) * 128, lr, sg);
          if constexpr (ra1) fa[1] = swz_read(sb + (wr * 32 + 16) * 128, lr, sg);
          if constexpr (rb0) fb[0] = swz_read(bb + (wc * 32) * 128, lr, sg);
          if constexpr (rb1) fb[1] = swz_read(bb + (wc * 32 + 16) * 128, lr, sg);
          if constexpr ((M & 1) != 0) sum[0][0] = mma_v<false>(fa[0], fb[0], sum[0][0]);
          if constexpr ((M & 2) != 0) sum[0][1] = mma_v<false>(fa[0], fb[1], sum[0][1]);
          if constexpr ((M & 4) != 0) sum[1][0] = mma_v<false>(fa[1], fb[0], sum[1][0]);
          if constexpr ((M & 8) != 0) sum[1][1] = mma_v<false>(fa[1], fb[1], sum[1][1]);
          if constexpr (KD == kKindT2) {
            const u32x4 fm = swz_read(sb + kLMeanRow * 128, lr, sg);
            sum[0][1] = mma_v<false>(fm, fm, sum[0][1]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] += sum[i >> 1][i & 1];
    }
  };
  // step t: products from stage t % 3; the data of step t + 2 (loaded two
  // steps ago) into stage (t + 2) % 3, last read at step t - 1; the loads of
  // step t + 4; one barrier
  auto run = [&](auto dg, auto kind) {
    constexpr bool DG = decltype(dg)::value;
    const std::integral_constant<int, DG ? 3 : 4> nu;
    u32x4 va[4], vb[4];
    gload(0, va, nu);
    gload(1, vb, nu);
    lstore(0, va, nu);
    lstore(1, vb, nu);
    gload(2, va, nu);
    gload(3, vb, nu);
    __syncthreads();
    for (int t = 0; t < nsteps; t += 2) {
      compute(t, kind, dg);
      lstore(t + 2, va, nu);
      __builtin_amdgcn_sched_barrier(0);
      gload(t + 4, va, nu);
      __builtin_amdgcn_sched_barrier(0);
      DR_LDS_SYNC();
      compute(t + 1, kind, dg);   // past the last step its stage holds zeros: the products add 0
      lstore(t + 3, vb, nu);
      __builtin_amdgcn_sched_barrier(0);
      gload(t + 5, vb, nu);
      __builtin_amdgcn_sched_barrier(0);
      DR_LDS_SYNC();
    }
  };
  // Blocks the reduction never reads take no products and keep zero
  // accumulators: A rows wholly past row n - 1 (I >= J, so these are the
  // last tile's), and on a diagonal tile the blocks wholly above the
  // diagonal.  The mask is uniform over the wave and is rounded up to the
  // smallest loop variant that contains it (extra products are harmless).
  int live = 0;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int rb = I * kTile + wr * 32 + 16 * i, cb = J * kTile + wc * 32 + 16 * j;
      if (rb < a.n && cb <= rb + 15) live |= 1 << (i * 2 + j);
    }
  using F = std::false_type;
  using T = std::true_type;
  if (!diag) {
    // J < I: every B block lies below the A rows, so live is 0, 3 or 15
    if (live == 0)
      run(F{}, std::integral_constant<int, 0>{});
    else if ((live & ~3) == 0)
      run(F{}, std::integral_constant<int, 3>{});
    else
      run(F{}, std::integral_constant<int, 15>{});
  } else if (wr == 0 && wc == 1) {
    run(T{}, std::integral_constant<int, kKindS>{});
  } else if (I == 0 && wr == 0 && wc == 0) {
    run(T{}, std::integral_constant<int, kKindT2>{});   // its live blocks are within mask 13
  } else if (live == 0) {
    run(T{}, std::integral_constant<int, 0>{});
  } else if ((live & ~1) == 0) {
    run(T{}, std::integral_constant<int, 1>{});
  } else if ((live & ~3) == 0) {
    run(T{}, std::integral_constant<int, 3>{});
  } else if ((live & ~13) == 0) {
    run(T{}, std::integral_constant<int, 13>{});
  } else {
    run(T{}, std::integral_constant<int, 15>{});
  }

  if (direct) {
    // the reduction's writes for a single chunk: K's lower triangle and
    // mirror, and from a diagonal tile the scores and t2 in its upper
    // triangle
    float* Kp = a.K + (a.pbase + p) * (long long)a.n * a.n;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int tr = wr * 32 + i * 16 + lg * 4 + r, tc = wc * 32 + j * 16 + lr;
          const int row = I * kTile + tr, col = J * kTile + tc;
          const float v = acc[i][j][r];
          if (col <= row) {
            if (row < a.n) {
              Kp[(long long)row * a.n + col] = v;
              Kp[(long long)col * a.n + row] = v;
            }
          } else if (diag) {
            if ((tr == 0 || tr == 16) && tc >= 32) {
              const int srow = I * kTile + 2 * tr + (tc - 32);
              if (srow < a.n) a.s[(a.pbase + p) * (long long)a.n + srow] = v;
            } else if (I == 0 && tr == 0 && tc == 16) {
              a.t2[a.pbase + p] = v;
            }
          }
        }
    return;
  }
  float* out = a.partial + (((long long)p * a.pairs + q) * a.maxchunks + chunk) * (kTile * kTile);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(wr * 32 + i * 16 + lg * 4 + r) * kTile + wc * 32 + j * 16 + lr] = acc[i][j][r];
}

// fp32 rows, n + 1 > 128: 256-row tiles on bf16 MFMA.  Each value is split
// into three bf16 parts, x = x0 + x1 + x2, each the nearest bf16 to what the
// previous ones leave (x0 + x1 + x2 holds x to 2^-25), when its 32-column step
// is staged in LDS, and a product takes the six pairs of parts with a + b <= 2:
// every product is exact in fp32, the dropped pairs weigh 2^-25 and less, and
// a step's sum is added to the accumulator by fp32 additions.  Error of K
// against 64 bits: 8e-8 to 9e-8 for 1024 to 229376 columns with shared
// directions; the fp32 MFMA tiles before had 1.9e-7 to 5.1e-7.
//
// Bound: bf16 MFMA at the rate the card's power allows (six products per fp32
// one are 2.6 times the fp32 MFMA rate, which bound the 64 x 64 fp32 tiles
// before).  256 x 229376: 209 -> 102 us, 3.7 us per 32-column step of which
// the products alone take 2.5 (the rest is the loads and splitting that the
// other wave does not cover); 224 groups of 256 x 1024: 219 -> 121 us; 7 groups
// of 1000 x 4096: 435 -> 205 us.  A last row tile of a few rows costs nearly a
// whole one: 20 groups of 300 x 4096 123 -> 134 us.
//
// One workgroup of eight waves (two per SIMD, so that one splits and reads
// while the other multiplies) per tile and column chunk:
//   diagonal tile I: the 256 rows once (they are both operands) and the target
//     mean as a 16-row block (sixteen times the same row).  The lower 64 x 64
//     blocks go one to a wave, the four diagonal ones two to a wave; waves with
//     one block take the target mean against 64 of the rows (the scores), one
//     the mean against itself (t2).
//   off-diagonal tile: 256 rows of row tile I, 128 rows of row tile J < I, one
//     64 x 64 block per wave.
// LDS: per stage three planes of 16-row blocks of 1 KB in fragment order
// (16-byte segment lg of row lr at 16 (16 lg + lr)), so a wave writes and
// reads a block as 1 KB in lane order.  Two stages and one barrier per step:
// the products of step t, and the split of step t + 1 (loaded a step ago)
// followed by the loads of step t + 2.
//
// From a step that holds a value of 2^50 or more (an infinity, or one whose
// partial products could overflow) or a nonzero one below 2^-109 (whose third
// part is below the smallest bf16) on, the chunk is taken on fp32 MFMA straight
// from memory by the same waves: there inf and overflow come out as in fp32
// arithmetic, and tiny values count in full (rows of 1e-36 against targets of
// order one: scores off by 2.5e-5 by their parts, 3e-7 on fp32 MFMA).
constexpr int kPC = 32;                       // fp32 columns per step
constexpr int kPThreads = 512;
constexpr int kPRows = 256, kPCols = 128;     // rows of tile I, rows of an off-diagonal tile's column half
constexpr int kPDiagBlocks = 17, kPOffBlocks = 24;   // 16-row blocks of a stage
constexpr int kPStageMax = 3 * kPOffBlocks * 1024;
constexpr int kPWin = 56;                     // steps whose target mean is in LDS at a time (two windows)
constexpr float kPBig = 1125899906842624.f;   // 2^50
constexpr float kPTiny = 0x1p-109f;           // three parts of eight bits end at 2^-133, the smallest bf16

__device__ const float kZeros4[4] = {0.f, 0.f, 0.f, 0.f};   // read in place of columns past a chunk

struct Planes8 {
  u32x4 p[3];   // eight values, three bf16 parts
};

__device__ __forceinline__ void split2(float a, float b, unsigned& p0, unsigned& p1, unsigned& p2) {
  p0 = pack_bf16(a, b);
  const float a1 = a - __uint_as_float(p0 << 16), b1 = b - __uint_as_float(p0 & 0xffff0000u);
  p1 = pack_bf16(a1, b1);
  p2 = pack_bf16(a1 - __uint_as_float(p1 << 16), b1 - __uint_as_float(p1 & 0xffff0000u));
}

__device__ __forceinline__ Planes8 split8(f32x4 a, f32x4 b) {
  Planes8 r;
  unsigned q[3];
#define DR_SPLIT2(X, Y, F)      \
  split2(X, Y, q[0], q[1], q[2]); \
  r.p[0].F = q[0];              \
  r.p[1].F = q[1];              \
  r.p[2].F = q[2];
  DR_SPLIT2(a.x, a.y, x) DR_SPLIT2(a.z, a.w, y) DR_SPLIT2(b.x, b.y, z) DR_SPLIT2(b.z, b.w, w)
#undef DR_SPLIT2
  return r;
}

__device__ __forceinline__ float abs_max8(f32x4 a, f32x4 b, float m) {   // NaNs are passed over
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a.x), "v"(a.y));
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a.z), "v"(a.w));
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(b.x), "v"(b.y));
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(b.z), "v"(b.w));
  return m;
}

__device__ __forceinline__ float abs_min8(f32x4 a, f32x4 b, float m) {
  asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a.x), "v"(a.y));
  asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(a.z), "v"(a.w));
  asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(b.x), "v"(b.y));
  asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(b.z), "v"(b.w));
  return m;
}

__device__ __forceinline__ bool has_tiny(f32x4 a, f32x4 b) {   // a nonzero value below kPTiny
  bool t = false;
#pragma unroll
  for (int e = 0; e < 4; ++e) t |= (a[e] != 0.f && fabsf(a[e]) < kPTiny) || (b[e] != 0.f && fabsf(b[e]) < kPTiny);
  return t;
}

// c[j] += A B_j^T over one step for NJ blocks: the six part pairs, the smallest
// first, summed from zero and added to c by fp32 additions.  (The bf16 MFMA
// truncates its sums: accumulated in place over a chunk, diagonal entries came
// out 1.3e-6 low.)
template <int NJ, class C>
__device__ __forceinline__ void mma_split(const u32x4 (&a)[3], const u32x4 (*b)[3], C&& c) {
  f32x4 t[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) t[j] = mma_bf16(a[0], b[j][2], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
  for (int j = 0; j < NJ; ++j) t[j] = mma_bf16(a[1], b[j][1], t[j]);
#pragma unroll
  for (int j = 0; j < NJ; ++j) t[j] = mma_bf16(a[2], b[j][0], t[j]);
#pragma unroll
  for (int j = 0; j < NJ; ++j) t[j] = mma_bf16(a[0], b[j][1], t[j]);
#pragma unroll
  for (int j = 0; j < NJ; ++j) t[j] = mma_bf16(a[1], b[j][0], t[j]);
#pragma unroll
  for (int j = 0; j < NJ; ++j) t[j] = mma_bf16(a[0], b[j][0], t[j]);
#pragma unroll
  for (int j = 0; j < NJ; ++j) c(j) += t[j];
}

// The tile and chunk of one workgroup.  NB: 16-row blocks of a stage.
template <bool DIAG>
__device__ __forceinline__ void gram_split_tile(const GramArgs& a, unsigned char* lds, int p, int chunk, int I,
                                                int J2) {
  constexpr int NB = DIAG ? kPDiagBlocks : kPOffBlocks;
  constexpr int NI = DIAG ? 2 : 3;              // 16-row blocks a wave stages (w, w + 8, ...)
  constexpr int kStage = 3 * NB * 1024;
  int* big = reinterpret_cast<int*>(lds + 2 * kPStageMax);   // step + 1 that set it, per stage
  float* gm = reinterpret_cast<float*>(lds + 2 * kPStageMax + 16);   // target mean, two windows of columns
  const long long g0 = a.goff[p], g1 = a.goff[p + 1];
  const long long c0 = g0 + (long long)chunk * a.CK;
  const long long c1 = c0 + a.CK < g1 ? c0 + a.CK : g1;
  const int nsteps = c1 > c0 ? (int)((c1 - c0 + kPC - 1) / kPC) : 0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  // row r of stage block b (rows past n - 1 repeat it: each row of a product
  // depends on its own row of the operand alone, and theirs are not written)
  auto row_ptr = [&](int b, int r) {
    const int row = b < 16 ? I * kPRows + 16 * b + r : J2 * kPCols + 16 * (b - 16) + r;
    return a.G + (long long)(row < a.n ? row : a.n - 1) * a.ldG * 4;
  };
  const int rowsI = a.n - I * kPRows;           // rows of tile I that exist
  // staging: lane (lg, lr) takes columns 8 lg .. + 7 of row lr of its blocks
  // (columns past the chunk: zeros)
  const int width = c1 > c0 ? (int)(c1 - c0) : 0;
  const unsigned char* src[NI];
  bool live16[NI];                              // block w + 8 u has rows (uniform)
#pragma unroll
  for (int u = 0; u < NI; ++u) {
    src[u] = row_ptr(w + 8 * u, lr) + (c0 + 8 * lg) * 4;
    live16[u] = u == 2 || 16 * (w + 8 * u) < rowsI;
  }
  // the target mean of window wd of the chunk's columns (zeros past them)
  // into its half of gm: fp64 sum over the m rows in order
  auto fill_mean = [&](int wd) {
    for (int cc = tid; cc < kPWin * kPC; cc += kPThreads) {
      const int c = wd * kPWin * kPC + cc;
      float g = 0.f;
      if (c < width) {
        const float* gt = a.Gt + c0 + c;
        double acc = 0.0;
        for (int j0 = 0; j0 < a.m; j0 += 8) {
          float x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = gt[(long long)(j0 + u < a.m ? j0 + u : 0) * a.ldGt];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (j0 + u < a.m) acc += (double)x[u];
        }
        g = (float)(acc / (double)a.m);
      }
      gm[(wd & 1) * kPWin * kPC + cc] = g;
    }
  };
  auto gm_at = [&](int t) { return gm + ((t / kPWin & 1) * kPWin + t % kPWin) * kPC; };
  const bool mean_wave = DIAG && w == 3;        // stages the mean's block beside its own
  auto gload = [&](int t, f32x4 (&v)[NI][2]) {
    const int c = t * kPC + 8 * lg;
#pragma unroll
    for (int u = 0; u < NI; ++u) {
      if (!live16[u]) continue;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        // (the cast keeps it a global load: a flat one would also hold up
        // every wait for LDS reads)
        v[u][h] = *(const __attribute__((address_space(1))) f32x4*)(
            c + 4 * h < width ? src[u] + (t * kPC + 4 * h) * 4 : reinterpret_cast<const unsigned char*>(kZeros4));
    }
  };
  auto stage = [&](int t, const f32x4 (&v)[NI][2]) {
    unsigned char* sb = lds + (t & 1) * kStage;
    float m = 0.f, lo = 1.f;
    auto put8 = [&](int b, f32x4 x, f32x4 y) {
      const Planes8 q = split8(x, y);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4*>(sb + (k * NB + b) * 1024 + lane * 16) = q.p[k];
      m = abs_max8(x, y, m);
      lo = abs_min8(x, y, lo);
    };
#pragma unroll
    for (int u = 0; u < NI; ++u)
      if (live16[u]) put8(w + 8 * u, v[u][0], v[u][1]);
    if (mean_wave) {
      const f32x4* g = reinterpret_cast<const f32x4*>(gm_at(t) + 8 * lg);
      put8(16, g[0], g[1]);
    }
    bool odd = m >= kPBig;
    if (__any(lo < kPTiny)) {   // zeros (columns past a chunk, empty rows) or tiny values: look closely
#pragma unroll
      for (int u = 0; u < NI; ++u)
        if (live16[u]) odd |= has_tiny(v[u][0], v[u][1]);
      if (mean_wave) {
        const f32x4* g = reinterpret_cast<const f32x4*>(gm_at(t) + 8 * lg);
        odd |= has_tiny(g[0], g[1]);
      }
    }
    if (__any(odd) && lane == 0) big[t & 1] = t + 1;
  };
  auto frag = [&](const unsigned char* sb, int b, u32x4 (&f)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) f[k] = *reinterpret_cast<const u32x4*>(sb + (k * NB + b) * 1024 + lane * 16);
  };
  // fp32 operand of 16 of the step's columns (half h) from memory
  auto frag32 = [&](int t, int b, int h) {
    const int c = t * kPC + 16 * h + 4 * lg;
    if (DIAG && b == 16) return *reinterpret_cast<const u32x4*>(gm_at(t) + 16 * h + 4 * lg);
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (c < width) v = *reinterpret_cast<const u32x4*>(row_ptr(b, lr) + (c0 + c) * 4);
    return v;
  };

  // the wave's blocks: 64-row blocks ba against bb (diagonal tiles: waves 6,
  // 7 take (0, 0) and (1, 1), (2, 2) and (3, 3)); sblk: the 64-row block whose
  // scores it takes (-1: none)
  int ba, bb, sblk = -1;
  bool two = false;
  if (DIAG) {
    two = w >= 6;
    ba = w < 2 ? 2 : (w < 5 ? 3 : (w == 5 ? 1 : 2 * (w - 6)));
    bb = w == 0 || w == 2 || w == 5 ? 0 : (w == 1 || w == 3 ? 1 : (w == 4 ? 2 : ba));
    sblk = w == 0 ? 2 : (w == 1 ? 1 : (w == 2 ? 3 : (w == 5 ? 0 : -1)));
  } else {
    ba = w >> 1;   // (a short last tile's live blocks then fall on different SIMDs)
    bb = 4 + (w & 1);
  }
  // live 16-row blocks of a 64-row block of tile I
  auto live = [&](int blk) { const int r = rowsI - 64 * blk; return r >= 64 ? 4 : (r > 0 ? (r + 15) / 16 : 0); };
  const int liveA = live(ba);
  // waves with two diagonal blocks keep the first one's lower blocks in acc's
  // lower triangle, the second one's in acc's upper triangle and accs
  f32x4 acc[4][4], accs[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    accs[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto first = [&](int i, int j) -> f32x4& { return acc[i][j]; };
  auto second = [&](int i, int j) -> f32x4& { return i == j ? accs[i] : acc[j][i]; };
  const bool t2_wave = DIAG && I == 0 && w == 4;

  // products of one step.  A wave whose rows end inside its block skips the
  // 16-row blocks past them (FULL = false).
  auto rect = [&](const unsigned char* sb, auto full) {
    u32x4 fb[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j) frag(sb, 4 * bb + j, fb[j]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!decltype(full)::value && i >= liveA) break;
      u32x4 fa[3];
      frag(sb, 4 * ba + i, fa);
      mma_split<4>(fa, fb, [&](int j) -> f32x4& { return acc[i][j]; });
    }
  };
  auto tri = [&](const unsigned char* sb, int blk, auto&& c) {
    u32x4 f[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) frag(sb, 4 * blk + i, f[i]);
    f32x4 t[10];   // the ten lower blocks together: a product's sum takes several MFMAs to come out
    auto pass = [&](int ka, int kb, bool zero) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
          f32x4& x = t[i * (i + 1) / 2 + j];
          x = mma_bf16(f[i][ka], f[j][kb], zero ? f32x4{0.f, 0.f, 0.f, 0.f} : x);
        }
    };
    pass(0, 2, true);
    pass(1, 1, false);
    pass(2, 0, false);
    pass(0, 1, false);
    pass(1, 0, false);
    pass(0, 0, false);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) c(i, j) += t[i * (i + 1) / 2 + j];
  };
  auto scores = [&](const unsigned char* sb) {
    u32x4 fm[3], f[4][3];
    frag(sb, 16, fm);
#pragma unroll
    for (int i = 0; i < 4; ++i) frag(sb, 4 * sblk + i, f[i]);
    mma_split<4>(fm, f, [&](int j) -> f32x4& { return accs[j]; });
  };
  auto mean2 = [&](const unsigned char* sb) {
    u32x4 fm[1][3];
    frag(sb, 16, fm[0]);
    mma_split<1>(fm[0], fm, [&](int) -> f32x4& { return accs[0]; });
  };
  auto slow = [&](int t) {
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
      u32x4 f[4];
      auto tri32 = [&](int blk, auto&& c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f[i] = frag32(t, 4 * blk + i, h);
#pragma unroll
          for (int j = 0; j <= i; ++j) c(i, j) = mma_v<false>(f[i], f[j], c(i, j));
        }
      };
      if (DIAG && two) {
        tri32(ba, first);
        tri32(ba + 1, second);
        continue;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = frag32(t, 4 * bb + j, h);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const u32x4 fa = frag32(t, 4 * ba + i, h);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mma_v<false>(fa, f[j], acc[i][j]);
      }
      if (DIAG) {
        const u32x4 fm = frag32(t, 16, h);
        if (t2_wave) accs[0] = mma_v<false>(fm, fm, accs[0]);
        if (sblk >= 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) accs[i] = mma_v<false>(fm, frag32(t, 4 * sblk + i, h), accs[i]);
        }
      }
    }
  };

  // the two waves of a SIMD (w, w + 4) stage at opposite ends of the step, so
  // that one splits while the other multiplies
  f32x4 v[NI][2];
  if (tid < 2) big[tid] = 0;
  if (DIAG) fill_mean(0);
  __syncthreads();
  gload(0, v);
  stage(0, v);
  gload(1, v);
  int t = 0;
  // the steps until the first with a big value.  One loop per kind of wave:
  // as branches of one loop the compiler moves the accumulators between
  // registers at every join and waits for all loads at its head (184 instead
  // of 132 us for 256 x 229376).
  auto run = [&](auto early, auto&& products) {
    for (; t < nsteps; ++t) {
      DR_LDS_SYNC();   // step t is staged; every wave is done with the other stage
      if (__builtin_amdgcn_readfirstlane(big[t & 1]) == t + 1) break;
      // the next window of the target mean (the half it takes was last read
      // before this barrier, and is next read after a later one)
      if (DIAG && t % kPWin == 0 && t + kPWin < nsteps) fill_mean(t / kPWin + 1);
      if (decltype(early)::value) {
        stage(t + 1, v);   // past the last step zeros, never read
        gload(t + 2, v);
        __builtin_amdgcn_sched_barrier(0);
      }
      products(lds + (t & 1) * kStage);
      if (!decltype(early)::value) {
        __builtin_amdgcn_sched_barrier(0);
        stage(t + 1, v);
        gload(t + 2, v);
      }
    }
  };
  using True = std::true_type;
  using False = std::false_type;
  auto run_rect = [&](auto early) {
    if (liveA == 4) run(early, [&](const unsigned char* sb) { rect(sb, True{}); });
    else run(early, [&](const unsigned char* sb) { rect(sb, False{}); });
  };
  auto run_scores = [&](auto early) {
    if (liveA == 4) run(early, [&](const unsigned char* sb) { rect(sb, True{}); scores(sb); });
    else run(early, [&](const unsigned char* sb) { rect(sb, False{}); scores(sb); });
  };
  if (DIAG && two) {
    run(False{}, [&](const unsigned char* sb) {
      tri(sb, ba, first);
      tri(sb, ba + 1, second);
    });
  } else if (DIAG && sblk >= 0) {
    if (w < 4) run_scores(True{});
    else run_scores(False{});
  } else if (t2_wave) {
    run(False{}, [&](const unsigned char* sb) { rect(sb, False{}); mean2(sb); });
  } else if (w < 4) {
    run_rect(True{});
  } else {
    run_rect(False{});
  }
  for (; t < nsteps; ++t) {          // from that step on
    if (DIAG && t % kPWin == 0) {
      __syncthreads();
      fill_mean(t / kPWin);
      __syncthreads();
    }
    slow(t);
  }

  // out: the reduction's 64 x 64 partial tiles, or with one chunk per group
  // K (lower triangle and mirror), s and t2 themselves
  auto put = [&](int bi, int bj, auto&& c) {
    const int I6 = 4 * I + bi, J6 = DIAG ? 4 * I + bj : 2 * J2 + bj - 4;
    if (I6 >= a.NT) return;
    if (a.maxchunks > 1) {
      float* out = a.partial +
                   (((long long)p * a.pairs + I6 * (I6 + 1) / 2 + J6) * a.maxchunks + chunk) * (kTile * kTile);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (DIAG && two && j > i) continue;   // (the scores live above the diagonal)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int tr = 16 * i + 4 * lg + r, tc = 16 * j + lr;
            if (!(DIAG && two) || tc <= tr) out[tr * kTile + tc] = c(i, j)[r];
          }
        }
      return;
    }
    float* Kp = a.K + (a.pbase + p) * (long long)a.n * a.n;
    const bool fast = a.vec4 && I6 * kTile + kTile <= a.n;   // float4 stores of whole blocks below the diagonal
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = I6 * kTile + 16 * i + 4 * lg + r, col = J6 * kTile + 16 * j + lr;
          if (!(DIAG && two && j >= i) && fast) {
            if (r == 0) big_store_block_fast(Kp, a.n, I6 * kTile + 16 * i, J6 * kTile + 16 * j, c(i, j), lane);
          } else if (!(DIAG && two && j > i) && col <= row && row < a.n) {
            const float v = c(i, j)[r];
            Kp[(long long)row * a.n + col] = v;
            Kp[(long long)col * a.n + row] = v;
          }
        }
  };
  put(ba, bb, first);
  if (DIAG && two) put(ba + 1, ba + 1, second);
  if (DIAG && lane < 16) {   // row 0 of the score blocks: lanes 0 .. 15, register 0
    auto part = [&](int I6) {
      return a.partial + (((long long)p * a.pairs + I6 * (I6 + 1) / 2 + I6) * a.maxchunks + chunk) * (kTile * kTile);
    };
    const int I6 = 4 * I + sblk;
    if (sblk >= 0 && I6 < a.NT) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int row = I6 * kTile + 16 * b + lr;
        if (a.maxchunks > 1)
          part(I6)[16 * (b / 2) * kTile + 32 + 16 * (b % 2) + lr] = accs[b][0];
        else if (row < a.n)
          a.s[(a.pbase + p) * (long long)a.n + row] = accs[b][0];
      }
    }
    if (t2_wave && lane == 0) {
      if (a.maxchunks > 1) part(0)[16] = accs[0][0];
      else a.t2[a.pbase + p] = accs[0][0];
    }
  }
}

// workgroups of a group: T diagonal tiles, then the (I, J2) pairs of row tile
// I and 128-row half J2 < 2 I
__global__ __launch_bounds__(kPThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gram_split_kernel(GramArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kPStageMax + 16 + 2 * kPWin * kPC * 4];
  const int chunk = blockIdx.x, p = blockIdx.z, T = (a.n + kPRows - 1) / kPRows;
  // an empty chunk leaves its partial tiles unwritten (the reduction skips
  // them); with one chunk per group it writes the group's zeros
  if (a.goff[p] + (long long)chunk * a.CK >= a.goff[p + 1] && a.maxchunks > 1) return;
  int q = blockIdx.y;
  if (q < T) {
    gram_split_tile<true>(a, lds, p, chunk, q, 0);
    return;
  }
  q -= T;
  int I = 1;
  while (q >= I * (I + 1)) ++I;
  gram_split_tile<false>(a, lds, p, chunk, I, q - I * (I - 1));
}

// ---------------------------------------------------------------- small fp32

constexpr int kSmCK = 128;           // columns per workgroup
constexpr int kSmLd = kSmCK + 4;     // LDS row stride (floats)
constexpr int kSmMaxRows = 128;      // n + 1 <= 128
constexpr int kSmThreads = 512;      // eight waves share the lower blocks

__global__ __launch_bounds__(kSmThreads) void gram_small_kernel(GramArgs a, const float* Gt, long long ldGt, int m,
                                                              int NRP, int nchunks) {
  __shared__ __attribute__((aligned(16))) float R[kSmMaxRows * kSmLd];
  const int chunk = blockIdx.x, p = blockIdx.y;
  const long long g0 = a.goff[p], g1 = a.goff[p + 1];
  const long long c0 = g0 + (long long)chunk * kSmCK;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = NRP / 16;
  float* out = a.partial + ((long long)p * nchunks + chunk) * NRP * NRP;
  if (c0 >= g1) return;   // (uniform) past the group: the reduction skips this chunk
  const int width = (int)(g1 - c0 < kSmCK ? g1 - c0 : kSmCK);   // a multiple of 4
  // general rows 0 .. n-1 (float4 loads, eight in flight per thread before
  // any store), zero columns past the group
  constexpr int RPP = kSmThreads / (kSmCK / 4);                    // rows per pass
  const int c4 = tid & (kSmCK / 4 - 1), r0 = tid / (kSmCK / 4);
  const bool cok = 4 * c4 < width;
  for (int rb = 0; rb < a.n; rb += 8 * RPP) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = rb + r0 + RPP * u;
      v[u] = (r < a.n && cok) ? *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.G) +
                                                                 (long long)r * a.ldG + c0 + 4 * c4)
                              : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = rb + r0 + RPP * u;
      if (r < a.n) *reinterpret_cast<float4*>(&R[r * kSmLd + 4 * c4]) = v[u];
    }
  }
  // row n: the target mean of this chunk (fp64 sum over the m rows in order,
  // eight loads in flight); rows n + 1 .. NRP - 1: zeros
  if (tid < kSmCK) {
    float gv = 0.f;
    if (tid < width) {
      double acc = 0.0;
      for (int j0 = 0; j0 < m; j0 += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = j0 + u < m ? Gt[(long long)(j0 + u) * ldGt + c0 + tid] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (j0 + u < m) acc += (double)t[u];
      }
      gv = (float)(acc / (double)m);
    }
    R[a.n * kSmLd + tid] = gv;
  }
  for (int e = tid; e < (NRP - a.n - 1) * kSmCK; e += kSmThreads)
    R[(a.n + 1 + e / kSmCK) * kSmLd + e % kSmCK] = 0.f;
  __syncthreads();
  // lower blocks (I, J <= I) round-robin over the waves
  const int lr = lane & 15, lk = lane >> 4, lg = lane >> 4;
  const int nblocks = nb * (nb + 1) / 2;
  for (int q = wave; q < nblocks; q += kSmThreads / 64) {
    int I = 0;
    while ((I + 1) * (I + 2) / 2 <= q) ++I;
    const int J = q - I * (I + 1) / 2;
    const float* ra = &R[(16 * I + lr) * kSmLd + lk];
    const float* rb = &R[(16 * J + lr) * kSmLd + lk];
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int k = 0; k < kSmCK; k += 4) acc = mma_f32(ra[k], rb[k], acc);
    // C layout: register r is row 4 lg + r of the block, column lane % 16
#pragma unroll
    for (int r = 0; r < 4; ++r) out[q * 256 + (4 * lg + r) * 16 + lr] = acc[r];
  }
}

// K (both triangles), s and t2 from the chunk partials: a workgroup takes 64
// neighbouring elements of a 16 x 16 block (four rows), lane by lane; a wave
// sums 16 chunks at a time (a tree in fp64, every load in flight), the waves'
// sums meet in LDS, again as a tree.  A wave's load is 256 contiguous bytes;
// with a wave per element, lanes over the chunks, each load touched 64 lines
// for 4 bytes of each, and most lanes were idle where a group has few chunks.
// The whole Gram, us: one group of 64 x 32768 16.7 -> 12.3, 8 of 64 x 4096 33
// -> 12, one of 127 x 131072 89 -> 52, 200 of 100 x 128 1540 -> 30.  In fp64
// what is left is the error of the chunks' own sums: 64 x 32768 3.1e-8 against
// 64 bits, 4.6e-8 with an fp32 tree, 5.3e-8 with fp32 sums along lanes.
// EL = 16 elements per workgroup, each lane group of 16 on chunks of its own,
// where a launch would have at most 24 blocks and there are 64 chunks or more:
// one group of 16 x 65536 11.6 -> 9.8 us (a wave per element took 10.6), of 32
// x 229376 38 -> 31.  Four groups of 16 x 16384, 48 blocks: 9.2 as it is, 9.6
// with 16 elements.
constexpr int kSrChunks = 16;   // chunks per lane at a time
constexpr int kSrWaves = 16;
template <int EL>
__global__ __launch_bounds__(kSrWaves * 64) void gram_small_reduce_kernel(GramArgs a, int NRP, int nchunks, float* K,
                                                                          float* s, float* t2, long long pbase) {
  constexpr int S = 64 / EL;   // chunk slots of a wave
  __shared__ double part[kSrWaves][64];
  const int p = blockIdx.y, q = blockIdx.x / (256 / EL);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int I = 0;
  while ((I + 1) * (I + 2) / 2 <= q) ++I;
  const int J = q - I * (I + 1) / 2;
  const int e = blockIdx.x % (256 / EL) * EL + lane % EL;   // element of the block
  const int r = 16 * I + (e >> 4), c = 16 * J + (e & 15);
  const long long width = a.goff[p + 1] - a.goff[p];
  const int nvalid = (int)((width + kSmCK - 1) / kSmCK);
  const float* src = a.partial + (long long)p * nchunks * NRP * NRP + q * 256 + e;
  auto tree = [](double (&v)[16]) {
#pragma unroll
    for (int h = 8; h > 0; h >>= 1)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u < h) v[u] += v[u + h];
    return v[0];
  };
  double sum = 0.0;
  for (int ch0 = kSrChunks * (S * wave + lane / EL); ch0 < nvalid; ch0 += kSrChunks * S * nw) {
    float t[kSrChunks];
#pragma unroll
    for (int u = 0; u < kSrChunks; ++u) t[u] = src[(long long)(ch0 + u < nvalid ? ch0 + u : nvalid - 1) * NRP * NRP];
    double v[kSrChunks];
#pragma unroll
    for (int u = 0; u < kSrChunks; ++u) v[u] = ch0 + u < nvalid ? (double)t[u] : 0.0;
    sum += tree(v);
  }
  part[wave][lane] = sum;
  __syncthreads();
  if (wave > 0) return;
  double v[kSrWaves];
#pragma unroll
  for (int u = 0; u < kSrWaves; ++u) v[u] = u < nw ? part[u < nw ? u : 0][lane] : 0.0;
  sum = tree(v);
#pragma unroll
  for (int o = EL; o < 64; o *= 2) sum += __shfl_xor(sum, o, 64);
  if (lane >= EL) return;
  const float acc = (float)sum;
  if (r > a.n || c > r) return;
  if (r < a.n) {
    float* Kp = K + (pbase + p) * (long long)a.n * a.n;
    Kp[(long long)r * a.n + c] = acc;
    Kp[(long long)c * a.n + r] = acc;
  } else if (c < a.n) {
    s[(pbase + p) * (long long)a.n + c] = acc;
  } else {
    t2[pbase + p] = acc;
  }
}

// ---------------------------------------------------------------- large n

constexpr int kBT = kTileRows;             // output tile edge
constexpr int kBK = kTileStepCols;         // bf16 columns per step (128-byte rows)
constexpr int kBPanel = kTilePanel;        // bytes of one operand panel per step (32 KiB)
constexpr int kBStage = kTileStage;        // A and B panels
constexpr int kBigMinTiles = 512;

struct BigArgs {
  const unsigned char* G;
  long long ldG;   // elements
  int n, T, pairs;
  int vec4;        // K rows start 16-byte aligned (n % 4 == 0, K aligned): float4 stores
  long long goff[kMaxGroups + 1];
  float* K;        // [P][n][n] of this launch's groups
};

// a 16 x 16 block into K element by element: rows and columns past n are skipped,
// and in a diagonal tile only the lower triangle (with its mirror above)
__device__ __forceinline__ void big_store_block_masked(float* Kp, int n, bool diag, int R, int C, f32x4 v, int lane) {
  const int lr = lane & 15, lg = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = R + 4 * lg + r, col = C + lr;
    if (row < n && col < n) {
      if (!diag || col <= row) Kp[(long long)row * n + col] = v[r];
      if (!diag || col < row) Kp[(long long)col * n + row] = v[r];
    }
  }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gram_big_kernel(BigArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kTileRing];
  const int p = blockIdx.y;
  // Workgroup i runs on XCD i % 8, and an XCD's 32 CUs take its workgroups
  // in order.  The lower-triangle tiles are grouped in chunks of 4 tile rows
  // x 8 tile columns (bands of 4 rows, 8 columns at a time); XCD x runs
  // chunks x, x + 8, ... one whole chunk at a time, so the 32 concurrent
  // tiles of an XCD read 12 distinct panels through its L2 rather than ~34.
  int I, J;
  {
    const int x = blockIdx.x & 7, sl = blockIdx.x >> 3;
    const int ci = (sl >> 5) * 8 + x, r = sl & 31;
    int band = 0, acc = 0;
    for (;; ++band) {
      if (4 * band >= a.T) return;   // past the last chunk
      const int rows_end = 4 * band + 4 < a.T ? 4 * band + 4 : a.T;
      const int nc = (rows_end + 7) / 8;
      if (ci < acc + nc) break;
      acc += nc;
    }
    I = 4 * band + (r >> 3);
    J = 8 * (ci - acc) + (r & 7);
    if (I >= a.T || J > I) return;
  }
  const long long g0 = a.goff[p], g1 = a.goff[p + 1];
  const int nk = (int)((g1 - g0 + kBK - 1) / kBK);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w >> 1, wc = w & 1;   // 128-row half of A, 128-row half of B
  const int lr = lane & 15, lg = lane >> 4;
  const int rowA0 = I * kBT, rowB0 = J * kBT;
  const int rowsA = a.n - rowA0 < kBT ? a.n - rowA0 : kBT;
  const int rowsB = a.n - rowB0 < kBT ? a.n - rowB0 : kBT;
  const bool diag = I == J;
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.G + (long long)rowA0 * a.ldG * 2, kOobOffset);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(a.G + (long long)rowB0 * a.ldG * 2, kOobOffset);
  // this lane's 8 rows of each panel (half blocks w, w + 4, ..., w + 28) and its segment
  unsigned offA[8], offB[8];
  int segs[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int hb = w + 4 * u;             // half block: rows 8 hb .. 8 hb + 7
    const int r = 8 * hb + (lane >> 3);
    segs[u] = swz_seg_of_lane(lane, hb & 1);
    offA[u] = r < rowsA ? (unsigned)((long long)r * a.ldG * 2) : kOobOffset;
    offB[u] = r < rowsB ? (unsigned)((long long)r * a.ldG * 2) : kOobOffset;
  }
  // DMA q (0..15) of step t into stage st: q even A, q odd B, half block
  // w + 4 (q / 2); steps past the group load zeros (no memory access)
  auto dma1 = [&](int t, int st, int q) {
    unsigned char* sb = lds + st * kBStage;
    const int u = q >> 1;
    const long long col = g0 + (long long)t * kBK + segs[u] * 8;
    const bool cok = col < g1;
    if (q & 1) {
      const unsigned cb = (offB[u] == kOobOffset || !cok) ? kOobOffset : offB[u] + (unsigned)(col * 2);
      dma16<kAuxCached>(rb, sb + kBPanel + (w + 4 * u) * 1024, cb);
    } else {
      const unsigned ca = (offA[u] == kOobOffset || !cok) ? kOobOffset : offA[u] + (unsigned)(col * 2);
      dma16<kAuxCached>(ra, sb + (w + 4 * u) * 1024, ca);
    }
  };
  // fragment read q (0..15) of 32-column half kh: q even A block q / 2, odd B block
  auto rd1 = [&](u32x4* fa, u32x4* fb, const unsigned char* sa, int kh, int q) {
    const int seg = 4 * kh + lg;
    if (q & 1) fb[q >> 1] = swz_read(sa + kBPanel + (wc * 8 + (q >> 1)) * 2048, lr, seg);
    else fa[q >> 1] = swz_read(sa + (wr * 8 + (q >> 1)) * 2048, lr, seg);
  };
  f32x4 acc[8][8];
  tile256_clear(acc);
  tile256_loop(lds, nk, dma1, rd1, acc);

  float* Kp = a.K + (long long)p * a.n * a.n;
  if (a.vec4 && !diag && rowA0 + kBT <= a.n) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        big_store_block_fast(Kp, a.n, rowA0 + wr * 128 + 16 * i, rowB0 + wc * 128 + 16 * j, acc[i][j], lane);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        big_store_block_masked(Kp, a.n, diag, rowA0 + wr * 128 + 16 * i, rowB0 + wc * 128 + 16 * j, acc[i][j], lane);
  }
}

bool gram_use_big(int64_t n, int P, dr_dtype dtype) {
  if (dtype != DR_BF16 || n < 2 * kBT) return false;
  const int64_t T = (n + kBT - 1) / kBT;
  const int gp = P < kMaxGroups ? P : kMaxGroups;
  return T * (T + 1) / 2 * gp >= kBigMinTiles;
}

// ROWS x 256 / ROWS elements of a 64 x 64 tile per workgroup: sums the chunk
// partials in fp64 (each of NP threads per element a run of the chunks, then
// the runs in order) and writes K (lower triangle and its mirror, the latter
// through LDS so that it too goes out in pieces of rows) and, for fp32 rows, s
// and t2 from the upper triangle of the diagonal tiles (where the fp32 tile
// kernels put them).
template <int ROWS, int NP>
__global__ __launch_bounds__(256 * NP) void gram_reduce_kernel(GramArgs a, float* K, float* s, float* t2,
                                                               long long pbase) {
  constexpr int COLS = 256 / ROWS, CB = kTile / COLS;
  __shared__ double red[NP][NP > 1 ? 256 : 1];
  __shared__ float tile[ROWS][COLS + 1];
  const int q = blockIdx.x, p = blockIdx.y;
  const int e = threadIdx.x & 255, part = NP == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const long long width = a.goff[p + 1] - a.goff[p], up = width + a.CK - 1;
  // (a 64-bit division is as long as the sum of a few chunks)
  const int nvalid = a.maxchunks == 1 ? width > 0 : (int)(up >> 32 ? up / a.CK : (unsigned)up / (unsigned)a.CK);
  int I, J;
  pair_to_tiles(q, I, J);
  const int r0 = ROWS * ((int)blockIdx.z / CB), c0 = COLS * ((int)blockIdx.z % CB);
  if (I * kTile + r0 >= a.n) return;   // no rows (nor, below them, scores)
  if (I == J && c0 >= r0 + ROWS && !(a.rows > a.n && r0 % 16 == 0 && r0 <= 16)) return;   // above the diagonal
  const int tr = r0 + e / COLS, tc = c0 + e % COLS;
  const int r = I * kTile + tr, c = J * kTile + tc;
  const bool lower = c <= r && r < a.n;
  // upper triangle of a diagonal tile: the scores (two rows of them) and t2
  int srow = -1;
  if (a.rows > a.n && I == J && c > r) {
    if ((tr == 0 || tr == 16) && tc >= 32) srow = I * kTile + 2 * tr + (tc - 32);
    if (srow >= a.n) srow = -1;
  }
  const bool t2_here = a.rows > a.n && q == 0 && tr == 0 && tc == 16;
  const bool need = lower || srow >= 0 || t2_here;
  double sum = 0.0;
  if (need) {
    int ch = (int)((long long)nvalid * part / NP);
    const int ce = (int)((long long)nvalid * (part + 1) / NP);
    const float* src = a.partial + (((long long)p * a.pairs + q) * a.maxchunks + ch) * (kTile * kTile);
    const unsigned at = tr * kTile + tc;   // (the chunk's address is scalar)
    // every load of a batch in flight before the first addition; the last
    // batch is the smallest that holds what is left
    auto batch = [&](auto count, auto full) {
      constexpr int N = decltype(count)::value;
      constexpr bool FULL = decltype(full)::value;
      float v[N];
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = (src + (FULL || ch + u < ce ? u : 0) * (kTile * kTile))[at];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < N; ++u) sum += FULL || ch + u < ce ? (double)v[u] : 0.0;
      ch += N;
      src += N * (kTile * kTile);
    };
    if constexpr (ROWS == 16) {   // few chunks: little code
      while (ch + 16 <= ce) batch(std::integral_constant<int, 16>{}, std::true_type{});
      while (ch + 4 <= ce) batch(std::integral_constant<int, 4>{}, std::true_type{});
      while (ch < ce) batch(std::integral_constant<int, 1>{}, std::true_type{});
    } else {
      while (ch + 32 <= ce) batch(std::integral_constant<int, 32>{}, std::true_type{});
      if (ch + 16 < ce) batch(std::integral_constant<int, 32>{}, std::false_type{});
      else if (ch + 8 < ce) batch(std::integral_constant<int, 16>{}, std::false_type{});
      else if (ch + 4 < ce) batch(std::integral_constant<int, 8>{}, std::false_type{});
      else if (ch + 1 < ce) batch(std::integral_constant<int, 4>{}, std::false_type{});
      else if (ch < ce) batch(std::integral_constant<int, 1>{}, std::true_type{});
    }
  }
  if (NP > 1) {
    red[part][e] = sum;
    __syncthreads();
    if (part == 0) {
#pragma unroll
      for (int u = 1; u < NP; ++u) sum += red[u][e];
    }
  }
  const float acc = (float)sum;
  float* Kp = K + (pbase + p) * (long long)a.n * a.n;
  if (part == 0) {
    tile[e / COLS][e % COLS] = acc;
    if (lower) Kp[(long long)r * a.n + c] = acc;
    if (srow >= 0) s[(pbase + p) * (long long)a.n + srow] = acc;
    if (t2_here) t2[pbase + p] = acc;
  }
  __syncthreads();
  if (part == 0) {   // mirrored
    const int mr = I * kTile + r0 + e % ROWS, mc = J * kTile + c0 + e / ROWS;
    if (mr < a.n && mc <= mr) Kp[(long long)mc * a.n + mr] = tile[e % ROWS][e / ROWS];
  }
}

// gbar[c] = (1/m) sum_j Gt[j][c] for c in [c_lo, c_hi)
template <bool BF16>
__global__ __launch_bounds__(kThreads) void target_mean_kernel(const unsigned char* Gt, long long ldGt, int m,
                                                               long long c_lo, long long c_hi, float* gbar) {
  const long long c = c_lo + (long long)blockIdx.x * kThreads + threadIdx.x;
  if (c >= c_hi) return;
  auto ld = [&](int j) -> float {
    if constexpr (BF16) {
      const unsigned short h = reinterpret_cast<const unsigned short*>(Gt)[(long long)j * ldGt + c];
      return __uint_as_float((unsigned)h << 16);
    } else {
      return reinterpret_cast<const float*>(Gt)[(long long)j * ldGt + c];
    }
  };
  // rows in batches of 8 loads in flight, summed in row order
  double acc = 0.0;
  int j = 0;
  for (; j + 8 <= m; j += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ld(j + u);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += (double)v[u];
  }
  for (; j < m; ++j) acc += (double)ld(j);
  gbar[c] = (float)(acc / (double)m);
}

// s[p][i] = <G[i][cols_p], gbar[cols_p]> for i < n; row n gives t2[p] = <gbar, gbar>.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void score_kernel(GramArgs a, const float* gbar, float* s, float* t2,
                                                         long long pbase) {
  const int i = blockIdx.x, p = blockIdx.y;
  const long long g0 = a.goff[p], g1 = a.goff[p + 1];
  double acc = 0.0;
  if (i < a.n) {
    // 16-byte loads: group edges are multiples of 8 (bf16) / 4 (fp32)
    // elements and rows are 16-byte aligned
    const unsigned char* row = a.G + (long long)i * a.ldG * GTr<BF16>::ES;
    constexpr int V = GTr<BF16>::EPV;
    for (long long c = g0 + (long long)threadIdx.x * V; c < g1; c += (long long)kThreads * V) {
      const u32x4 q = *reinterpret_cast<const u32x4*>(row + c * GTr<BF16>::ES);
      const float4 g4a = *reinterpret_cast<const float4*>(gbar + c);
      if constexpr (BF16) {
        const float4 g4b = *reinterpret_cast<const float4*>(gbar + c + 4);
        acc += (double)__uint_as_float(q.x << 16) * (double)g4a.x + (double)__uint_as_float(q.x & 0xffff0000u) * (double)g4a.y;
        acc += (double)__uint_as_float(q.y << 16) * (double)g4a.z + (double)__uint_as_float(q.y & 0xffff0000u) * (double)g4a.w;
        acc += (double)__uint_as_float(q.z << 16) * (double)g4b.x + (double)__uint_as_float(q.z & 0xffff0000u) * (double)g4b.y;
        acc += (double)__uint_as_float(q.w << 16) * (double)g4b.z + (double)__uint_as_float(q.w & 0xffff0000u) * (double)g4b.w;
      } else {
        acc += (double)__uint_as_float(q.x) * (double)g4a.x + (double)__uint_as_float(q.y) * (double)g4a.y;
        acc += (double)__uint_as_float(q.z) * (double)g4a.z + (double)__uint_as_float(q.w) * (double)g4a.w;
      }
    }
  } else {
    for (long long c = g0 + threadIdx.x; c < g1; c += kThreads) acc += (double)gbar[c] * (double)gbar[c];
  }
  __shared__ double red[kThreads];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (i < a.n)
      s[(pbase + p) * (long long)a.n + i] = (float)red[0];
    else
      t2[pbase + p] = (float)red[0];
  }
}

struct GramPlan {
  int64_t rows;
  int NT, pairs, CK, maxchunks;
  size_t gbar_bytes, partial_bytes;
  size_t bytes;     // workspace of the call: gbar and the partial tiles, or more (see gram_plan)
  bool lds_tiles;   // fp32 rows: gram_tile_lds_kernel, not gram_split_kernel
  bool small;       // gram_small_kernel path
  int NRP;          // its padded row count
};

bool gram_use_small(int64_t n, dr_dtype dtype) { return dtype == DR_F32 && n >= 1 && n + 1 <= kSmMaxRows; }

// Chunk of gram_tile_lds_kernel: the multiple of 256 columns that keeps the
// launch just within two rounds of kLdsSlots, so that the second round is
// nearly full (the fixed count keeps the chunking, and with it the summation
// order, the same on every device)
int64_t lds_tile_chunk(int64_t maxw, int64_t pairs, int64_t groups) {
  const int64_t all = align_up((size_t)(maxw > 0 ? maxw : 1), 256);
  const int64_t c = align_up((size_t)((maxw * pairs * groups + 2 * kLdsSlots - 1) / (2 * kLdsSlots)), 256);
  return c < 256 ? 256 : (c < all ? c : all);
}

// The fp32 tile kernels' times in us, to within 6.5 % (64 x 64 tiles) and 9.5 %
// (split tiles), fitted to 650 shapes of 128 to 1100 rows, 1 to 224 groups and
// 32 to 229376 columns; the call takes the lesser (the split tiles on a near
// tie), within 0.3 % of the better one on average.  Few columns, few rows and
// short last row tiles leave the split tiles' 256 workgroups idle: one group of
// 256 x 4096 24.5 us split and 18.3 in 64 x 64 tiles, 224 groups of 257 x 256
// 180 and 88, one of 512 x 1024 23.3 and 17.4; but one of 256 x 65536 47 and 71.
// K's own writes count where it is large, and the chunk partials, written and
// read again.
double lds_tiles_time(int64_t n, int64_t pairs, int64_t groups, int64_t maxw) {
  const int64_t ck = lds_tile_chunk(maxw, pairs, groups), chunks = maxw > 0 ? (maxw + ck - 1) / ck : 1;
  const double wgs = (double)(pairs * groups * chunks), rounds = wgs / kLdsSlots;
  const double cols = (double)(ck < maxw ? ck : maxw) * 1e-3;
  double t = 8.5 + cols * (52.0 * (rounds > 1.0 / 3 ? rounds : 1.0 / 3) + 5.1 * std::ceil(rounds));
  t += 0.34 * 4e-6 * (double)(n * n * groups);
  if (chunks > 1) t += 1.5 + 0.63 * 1e-6 * wgs * (kTile * kTile * 4);
  return t;
}

double split_tiles_time(int64_t n, int64_t pairs, int64_t groups, int64_t steps, int64_t chunks) {
  const int64_t T = (n + kPRows - 1) / kPRows;
  // Workgroups are dealt to the eight XCDs in turn: with a multiple of eight
  // per group each XCD gets one kind of tile, and the chip waits for whole
  // rounds of the longest; otherwise short tiles make room for others.
  double rounds = (double)(T * T * groups * chunks) / kSplitSlots;
  rounds = T == 1 || T * T * chunks % 8 == 0 ? std::ceil(rounds) : (rounds > 1.0 ? rounds : 1.0);
  const double rows = n < kPRows ? (double)n / kPRows : 1.0, out = 4e-6 * (double)(n * n * groups);
  double t = 5.6 + rounds * ((double)((steps + chunks - 1) / chunks) * (1.12 + 1.42 * rows) + 1.4 + 5.3 * rows);
  t += 0.16 * out;
  if (chunks > 1) {
    t += 0.45 * 1e-6 * (double)(pairs * groups * chunks * (kTile * kTile * 4)) - 1.1;
  } else if (T > 1) {   // written by elements: a broken 64-row block, rows off 16 bytes
    if (n % 64 && (n - 1) % kPRows >= 64) t += 0.25 * out;
    if (n % 4) t += 0.14 * out;
  }
  return t;
}

// Chunk length: bf16 tiles, a multiple of 256 columns, shrunk until a launch
// has about kTargetWGs workgroups; fp32 tiles, see the two rules; identical for
// every launch of a call.
GramPlan gram_plan(int64_t n, const int64_t* goff, int P, dr_dtype dtype) {
  GramPlan g = {};
  // fp32 sketches: gbar joins as row n, so s and t2 come out of the same
  // pass (the tiles cover the n general rows; the diagonal tiles carry gbar)
  const int64_t rows = dtype == DR_F32 ? n + 1 : n;
  g.NT = (int)((n + kTile - 1) / kTile);
  g.pairs = g.NT * (g.NT + 1) / 2;
  int64_t maxw = 0;
  for (int p = 0; p < P; ++p) maxw = goff[p + 1] - goff[p] > maxw ? goff[p + 1] - goff[p] : maxw;
  const int gp = P < kMaxGroups ? P : kMaxGroups;
  int64_t ck = align_up((size_t)(maxw > 0 ? maxw : 1), 256);
  if (dtype == DR_F32) {
    // split tiles, one workgroup per CU: the chunk count with the least time,
    // rounds of kSplitSlots workgroups times the steps of a chunk and about
    // four more for its prologue and epilogue, and three for the reduction.
    // kSplitSlots is fixed, so the chunking, and with it the summation order,
    // is the same on every device.  Chunks keep at least two steps, and their
    // partial tiles stay within kSplitPartials.  (Weighing a short last row
    // tile less gave more chunks and measured worse: 20 groups of 300 rows x
    // 4096 columns 159 us in six chunks, 134 us in three.)
    const int64_t T = (n + kPRows - 1) / kPRows, wgs = T * T * gp;
    const int64_t steps = (maxw + kPC - 1) / kPC, chunk_bytes = (int64_t)gp * g.pairs * kTile * kTile * 4;
    int64_t best = -1, chunks = 1;
    for (int64_t c = 1; c <= 256 && (c == 1 || (2 * c <= steps && c * chunk_bytes <= kSplitPartials)); ++c) {
      const int64_t cost = (wgs * c + kSplitSlots - 1) / kSplitSlots * ((steps + c - 1) / c + 4) + (c > 1 ? 3 : 0);
      if (best < 0 || cost < best) {
        best = cost;
        chunks = c;
      }
    }
    ck = (steps + chunks - 1) / chunks * kPC;
    if (ck < kPC) ck = kPC;
    g.lds_tiles = n > 0 &&
                  lds_tiles_time(n, g.pairs, gp, maxw) < 0.95 * split_tiles_time(n, g.pairs, gp, steps, chunks);
    if (g.lds_tiles) ck = lds_tile_chunk(maxw, g.pairs, gp);
  } else {
    while (ck > 256 && (int64_t)g.pairs * gp * ((maxw + ck - 1) / ck) < kTargetWGs) ck = align_up((size_t)(ck / 2), 256);
  }
  g.CK = (int)ck;
  g.maxchunks = (int)((maxw + ck - 1) / ck);
  if (g.maxchunks < 1) g.maxchunks = 1;
  g.small = gram_use_small(n, dtype);
  if (g.small) g.lds_tiles = false;
  // fp32 rows: the kernels form gbar in LDS, but for the 64 x 64 tiles (with n = 0 it is the whole work)
  const int64_t gcols = dtype == DR_F32 && n > 0 && !g.lds_tiles ? 0 : goff[P];
  g.gbar_bytes = align_up((size_t)(gcols > 0 ? gcols : 1) * sizeof(float), 256);
  g.partial_bytes = (size_t)gp * g.pairs * g.maxchunks * kTile * kTile * sizeof(float);
  if (rows == 0 || gram_use_big(n, P, dtype) || (dtype == DR_F32 && g.maxchunks == 1)) g.partial_bytes = 0;
  g.rows = rows;
  g.NRP = (int)((n + 1 + 15) / 16 * 16);
  if (g.small) {
    g.maxchunks = (int)((maxw + kSmCK - 1) / kSmCK);
    if (g.maxchunks < 1) g.maxchunks = 1;
    g.partial_bytes = (size_t)gp * g.maxchunks * g.NRP * g.NRP * sizeof(float);
  }
  g.bytes = g.gbar_bytes + g.partial_bytes;
  if (dtype == DR_F32 && n > 0) {
    // The size asked for does not fall below gbar over all columns and, for
    // tiled rows, the chunk partials of gram_tile_lds_kernel: dr_gram_noalloc's
    // limit is stated in it, so that which problems that call refuses does not
    // depend on how the tiles are cut.
    size_t floor = align_up((size_t)(goff[P] > 0 ? goff[P] : 1) * sizeof(float), 256);
    if (g.small) {
      floor += g.partial_bytes;
    } else {
      const int64_t c = lds_tile_chunk(maxw, g.pairs, gp);
      floor += (size_t)gp * g.pairs * (maxw > 0 ? (maxw + c - 1) / c : 1) * kTile * kTile * sizeof(float);
    }
    if (floor > g.bytes) g.bytes = floor;
  }
  return g;
}

dr_status gram_validate(const void* G, int64_t n, int64_t ldG, const void* Gt, int64_t m, int64_t ldGt,
                        dr_dtype dtype, const int64_t* goff, int P, float* K, float* s, float* t2) {
  if (dtype != DR_BF16 && dtype != DR_F32) return DR_ERR_DTYPE;
  if (!goff || P < 1 || n < 0 || m < 1 || n > (1 << 20)) return DR_ERR_ARG;
  if (goff[0] < 0) return DR_ERR_ARG;
  for (int p = 0; p < P; ++p)
    if (goff[p + 1] < goff[p]) return DR_ERR_ARG;
  const int64_t vec = dtype == DR_BF16 ? 8 : 4;
  if (ldGt < goff[P] || ldGt % vec || !Gt || !aligned16(Gt) || !t2) return DR_ERR_ARG;
  if (n > 0) {
    if (ldG < goff[P] || ldG % vec || !G || !aligned16(G) || !K || !s) return DR_ERR_ARG;
    for (int p = 0; p <= P; ++p)
      if (goff[p] % vec) return DR_ERR_ARG;
  }
  return DR_OK;
}

}  // namespace
}  // namespace dr

extern "C" size_t dr_gram_workspace_size(int64_t n, int64_t m, const int64_t* goff, int P, dr_dtype dtype) {
  (void)m;
  if (dtype != DR_BF16 && dtype != DR_F32) return 0;
  if (!goff || P < 1 || n < 0) return 0;
  return dr::gram_plan(n, goff, P, dtype).bytes;
}

namespace dr {
namespace {

// host checks of a call (before any HIP call), then the plan
dr_status gram_check(const void* G, int64_t n, int64_t ldG, const void* Gt, int64_t m, int64_t ldGt, dr_dtype dtype,
                     const int64_t* goff, int P, float* K, float* s, float* t2, GramPlan* plan) {
  dr_status st = gram_validate(G, n, ldG, Gt, m, ldGt, dtype, goff, P, K, s, t2);
  if (st != DR_OK) return st;
  // the large-n kernel addresses a 256-row panel with 32-bit buffer offsets
  if (gram_use_big(n, P, dtype) && (uint64_t)ldG * 2 * (kBT + 1) >= (uint64_t)kOobOffset) return DR_ERR_UNSUPPORTED;
  *plan = gram_plan(n, goff, P, dtype);
  return DR_OK;
}

// enqueue the Gram on hs with the workspace at `workspace` (every byte of
// it that a kernel reads is written earlier in the same call)
dr_status gram_run(const GramPlan& g, const void* G, int64_t n, int64_t ldG, const void* Gt, int64_t m, int64_t ldGt,
                   dr_dtype dtype, const int64_t* goff, int P, float* K, float* s, float* t2, void* workspace,
                   hipStream_t hs) {
  dr_status st = DR_OK;
  const bool bf = dtype == DR_BF16;
  float* gbar = static_cast<float*>(workspace);
  float* partial = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + g.gbar_bytes);

  const long long c_lo = goff[0], c_hi = goff[P];
  if (c_hi > c_lo && (bf || n == 0 || g.lds_tiles)) {   // the other fp32 kernels form gbar inside their chunks
    const int blocks = (int)((c_hi - c_lo + kThreads - 1) / kThreads);
    if (bf)
      hipLaunchKernelGGL(target_mean_kernel<true>, dim3(blocks), dim3(kThreads), 0, hs,
                         static_cast<const unsigned char*>(Gt), (long long)ldGt, (int)m, c_lo, c_hi, gbar);
    else
      hipLaunchKernelGGL(target_mean_kernel<false>, dim3(blocks), dim3(kThreads), 0, hs,
                         static_cast<const unsigned char*>(Gt), (long long)ldGt, (int)m, c_lo, c_hi, gbar);
    if ((st = launch_status()) != DR_OK) return st;
  }

  for (int p0 = 0; p0 < P; p0 += kMaxGroups) {
    const int gp = P - p0 < kMaxGroups ? P - p0 : kMaxGroups;
    GramArgs a = {};
    a.G = static_cast<const unsigned char*>(G);
    a.ldG = ldG;
    a.n = (int)n;
    a.rows = (int)g.rows;
    a.gbar = gbar;
    for (int p = 0; p <= gp; ++p) a.goff[p] = goff[p0 + p];
    a.P = gp;
    a.NT = g.NT;
    a.pairs = g.pairs;
    a.CK = g.CK;
    a.maxchunks = g.maxchunks;
    a.partial = partial;
    a.K = K;
    a.s = s;
    a.t2 = t2;
    a.pbase = p0;
    a.vec4 = n % 4 == 0 && aligned16(K);
    a.Gt = static_cast<const float*>(Gt);
    a.ldGt = ldGt;
    a.m = (int)m;
    if (gram_use_big(n, P, dtype)) {
      BigArgs b = {};
      b.G = static_cast<const unsigned char*>(G);
      b.ldG = ldG;
      b.n = (int)n;
      b.T = (int)((n + kBT - 1) / kBT);
      b.pairs = b.T * (b.T + 1) / 2;
      for (int p = 0; p <= gp; ++p) b.goff[p] = goff[p0 + p];
      b.K = K + (long long)p0 * n * n;
      int chunks = 0;
      for (int band = 0; 4 * band < b.T; ++band) chunks += ((4 * band + 4 < b.T ? 4 * band + 4 : b.T) + 7) / 8;
      b.vec4 = (n % 4 == 0) && aligned16(K);
      hipLaunchKernelGGL(gram_big_kernel, dim3((chunks + 7) / 8 * 256, gp), dim3(256), 0, hs, b);
      if ((st = launch_status()) != DR_OK) return st;
    } else if (g.small) {
      hipLaunchKernelGGL(gram_small_kernel, dim3(g.maxchunks, gp), dim3(kSmThreads), 0, hs, a,
                         static_cast<const float*>(Gt), (long long)ldGt, (int)m, g.NRP, g.maxchunks);
      if ((st = launch_status()) != DR_OK) return st;
      const int nb = g.NRP / 16;
      const bool wide = nb * (nb + 1) * 2 * gp <= 24 && g.maxchunks >= 64;   // (few blocks, many chunks)
      const int el = wide ? 16 : 64, per = kSrChunks * 64 / el;
      const int nw = (g.maxchunks + per - 1) / per;   // 16 chunks per lane, up to 16 waves
      hipLaunchKernelGGL(wide ? gram_small_reduce_kernel<16> : gram_small_reduce_kernel<64>,
                         dim3(nb * (nb + 1) / 2 * (256 / el), gp),
                         dim3(64 * (nw < 1 ? 1 : nw > kSrWaves ? kSrWaves : nw)), 0, hs, a, g.NRP, g.maxchunks, K, s,
                         t2, (long long)p0);
      if ((st = launch_status()) != DR_OK) return st;
    } else if (g.pairs > 0) {
      if (bf) {
        hipLaunchKernelGGL(gram_tile_kernel, dim3(g.maxchunks, g.pairs, gp), dim3(kThreads), 0, hs, a);
      } else if (g.lds_tiles) {
        hipLaunchKernelGGL(gram_tile_lds_kernel, dim3(g.maxchunks, g.pairs, gp), dim3(kThreads), 0, hs, a);
      } else {
        const int T = (int)((n + kPRows - 1) / kPRows);
        hipLaunchKernelGGL(gram_split_kernel, dim3(g.maxchunks, T * T, gp), dim3(kPThreads), 0, hs, a);
      }
      if ((st = launch_status()) != DR_OK) return st;
      if (bf || g.maxchunks > 1) {   // fp32 tiles of a single chunk are written by the tile kernel
        const dim3 rg(g.pairs, gp, kTile * kTile / 256);
        // Rows of 64 where the workgroups are few: a wave's load is then one
        // piece of 256 bytes (one bf16 group of 512 x 4096: 29.5 us, with 16 x
        // 16 blocks 34.0), in four parts where the chunks are many (256 fp32
        // rows x 229376 columns, 256 chunks: 14 us with one).  Where there are
        // many, and few chunks, the writes weigh more: 16 x 16 blocks, whose
        // mirror goes out in pieces of 64 bytes, not 16 (64 groups of 512 x 64:
        // 86 us, 98 in rows).  Up to 16 rows are one such block.
        const int64_t blocks = (int64_t)g.pairs * gp * (kTile * kTile / 256);
        if (g.maxchunks >= 32 && blocks < 512)
          hipLaunchKernelGGL((gram_reduce_kernel<4, 4>), rg, dim3(1024), 0, hs, a, K, s, t2, (long long)p0);
        else if (blocks < 2048 && n > 16)
          hipLaunchKernelGGL((gram_reduce_kernel<4, 1>), rg, dim3(256), 0, hs, a, K, s, t2, (long long)p0);
        else
          hipLaunchKernelGGL((gram_reduce_kernel<16, 1>), rg, dim3(256), 0, hs, a, K, s, t2, (long long)p0);
        if ((st = launch_status()) != DR_OK) return st;
      }
    }
    if (bf) {
      // bf16 sketches: s and t2 against the fp32 target mean in a separate pass
      hipLaunchKernelGGL(score_kernel<true>, dim3(n + 1, gp), dim3(kThreads), 0, hs, a, gbar, s, t2, (long long)p0);
      if ((st = launch_status()) != DR_OK) return st;
    } else if (g.pairs == 0) {
      // fp32 with no general rows: t2 alone
      hipLaunchKernelGGL(score_kernel<false>, dim3(1, gp), dim3(kThreads), 0, hs, a, gbar, s, t2, (long long)p0);
      if ((st = launch_status()) != DR_OK) return st;
    }
  }
  return DR_OK;
}

}  // namespace
}  // namespace dr

extern "C" dr_status dr_gram(const void* G, int64_t n, int64_t ldG, const void* Gt, int64_t m, int64_t ldGt,
                             dr_dtype dtype, const int64_t* goff, int P, float* K, float* s, float* t2,
                             void* workspace, size_t ws_bytes, void* stream) {
  dr::GramPlan g;
  const dr_status st = dr::gram_check(G, n, ldG, Gt, m, ldGt, dtype, goff, P, K, s, t2, &g);
  if (st != DR_OK) return st;
  if (!workspace || ws_bytes < g.bytes) return DR_ERR_WORKSPACE;
  return dr::gram_run(g, G, n, ldG, Gt, m, ldGt, dtype, goff, P, K, s, t2, workspace,
                      reinterpret_cast<hipStream_t>(stream));
}

// ---------------------------------------------------------------------------
// dr_gram_noalloc: the same Gram with its workspace in a fixed device array.
// In host code `scratch` names a host-side stand-in, not device memory: its
// device address is looked up once per device (hipGetSymbolAddress, with
// that device current) and only that address is ever handed to a kernel.
// Each device holds its own copy of the array until the process ends.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[DR_GRAM_NOALLOC_MAX_BYTES];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices];   // device address of `scratch` per device, null until looked up
}  // namespace

extern "C" dr_status dr_gram_noalloc(const void* G, int64_t n, int64_t ldG, const void* Gt, int64_t m, int64_t ldGt,
                                     dr_dtype dtype, const int64_t* goff, int P, float* K, float* s, float* t2,
                                     void* stream) {
  dr::GramPlan g;
  const dr_status st = dr::gram_check(G, n, ldG, Gt, m, ldGt, dtype, goff, P, K, s, t2, &g);
  if (st != DR_OK) return st;
  if (g.bytes > (size_t)DR_GRAM_NOALLOC_MAX_BYTES) return DR_ERR_TOO_LARGE;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchDevices) return DR_ERR_HIP;
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      void* p = nullptr;
      if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DR_ERR_HIP;
      g_scratch_ptr[dev] = p;
    }
    ptr = g_scratch_ptr[dev];
  }
  return dr::gram_run(g, G, n, ldG, Gt, m, ldGt, dtype, goff, P, K, s, t2, ptr, reinterpret_cast<hipStream_t>(stream));
}
