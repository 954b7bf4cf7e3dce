// Steps 2 and 3 of Section 5 in one kernel: the per-position products never leave the CU.
//
// Section 5 gives each core its own images through all three steps and remarks that this lets steps
// 2 and 3 run fused, out of cache.  Here a workgroup has some rows of W_F (output channels) and one block of 64 tiles
// through ALL positions: product_output_kernel four rows, for m = 2; product_output4_kernel 64, for F(4x4,3x3).
#pragma once
#include <type_traits>
#include <utility>

#include "swconv_kernels.hpp"

namespace swconv {

// Where the m x m outputs of a tile go (host-built, one entry per tile of the padded tile range).
struct OutTile {
  uint32_t n;      // image
  uint32_t pix;    // (ty*m)*Wo + tx*m: offset of the tile's first pixel inside an output plane
  uint32_t valid;  // rows (low 16 bits) and columns (high 16 bits) of the tile inside Ho x Wo; 0 = padding tile
  uint32_t pad;
};

constexpr int kFusedWaves = 16;                          // slices (4 rows) of a chunk of rows in the weight packages
constexpr int kFusedRows = kFusedWaves * kSliceRows;     // rows of W_F per chunk

__device__ __forceinline__ void acc_fma(Acc4& y, float c, const Acc4& x) {
  y.a0 = fmaf(c, x.a0, y.a0); y.a1 = fmaf(c, x.a1, y.a1); y.a2 = fmaf(c, x.a2, y.a2); y.a3 = fmaf(c, x.a3, y.a3);
}

// Weight packages: wpk[p][kc][b][w] = one 512-byte batch in the stream layout of the product
// kernel ([q][s] -> (row byte offset in a panel of 64 tiles, weight) of row kc*64 + w*4 + q, step 16 b + s),
// rows in their natural order.  lens[p][kc*16 + w] = steps of that slice (a multiple of 4, at most 16 B).

// ---------------------------------------------------------------------------------------------
// Steps 2 and 3 in one kernel for m = 2, whose M is 9 (F(2x2,5x5)) or 4 times the output.
//
// A workgroup has one slice of one tile block and its NW waves share the positions, P / NW each.  Nothing is staged: a
// wave reads the row of V of a non-zero - 256 bytes a quarter - from the L2 when it multiplies by it, up to
// sixteen steps in flight, or 24 where workgroups have a CU to themselves.  The products of all positions meet in LDS, where four waves, one a row, transform them and
// store the outputs.  The sums are those of the product and the output transform as two kernels, bit for bit.
// What bounds it is the way of the rows: 256 bytes for every non-zero and tile block, without reuse, at 12 TB/s over all
// CUs (32 x 27 x 27, 48 -> 128 channels: 502 MB in 41.8 us), and for the smallest layers two such ways one after the other
// (packages, rows).  24 waves a CU: 16 steps in flight take 64 registers of a lane's 80.  One image of 13 x 13, 256 -> 384
// (96 workgroups, slices of 24 to 44 steps), with 16 steps in flight, each batch waited for before the next, and all three
// batches asked for in front of the lengths: 9.4 us in a rotation of plans that no cache holds and 8.1 repeated; now 8.1 and 7.0.
// Before, a workgroup of 16 waves had 64 rows of a tile block, a panel and weights in LDS and a barrier per position: 44.9
// us for that layer, but 36.8 for one image (now 6.2) and 133 for 64 x 56 x 56, 64 -> 64, F(2x2,3x3) (now 107).
constexpr int kGatherMaxBatches = 3;  // a slice's first two batches are asked for at once, the third by its length

// The lane's four tiles of the rows of steps 4 G .. 4 G + 3: rows of V at `soff`, addressed by the pair's offset, which
// counts 256 bytes a row, times row_scale.
template <int G>
__device__ __forceinline__ Group4 gather_group(__amdgpu_buffer_rsrc_t vr, uint32_t soff, uint32_t row_scale, uint32_t lane_sub,
                                               uint32_t boff) {
  constexpr int I0 = G * kStepGroup;
  auto load = [&](uint32_t off) {
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(vr, (int)(__umul24(off, row_scale) + lane_sub),
                                                                            (int)soff, 0));
  };
  return Group4{load(quarter_bcast<I0 + 0>(boff)), load(quarter_bcast<I0 + 1>(boff)), load(quarter_bcast<I0 + 2>(boff)),
                load(quarter_bcast<I0 + 3>(boff))};
}
template <int G>
__device__ __forceinline__ void multiply_group(const Group4& g, uint32_t bw, Acc4& acc) {
  constexpr int I0 = G * kStepGroup;
  quarter_fma<I0 + 0, true>(acc, bw, g.x0);
  quarter_fma<I0 + 1, false>(acc, bw, g.x1);
  quarter_fma<I0 + 2, false>(acc, bw, g.x2);
  quarter_fma<I0 + 3, false>(acc, bw, g.x3);
}
// The first `steps` (a positive multiple of 4) steps of a batch, the rows of eight or of sixteen steps in flight
// together (as many as there are groups, in four variants, takes registers that cost a third of the waves: 45 -> 57 us).
__device__ __forceinline__ void gather_batch(__amdgpu_buffer_rsrc_t vr, uint32_t soff, uint32_t row_scale, uint32_t lane_sub,
                                             const u32x2_t& b, int steps, Acc4& acc) {
  const Group4 g0 = gather_group<0>(vr, soff, row_scale, lane_sub, b.x), g1 = gather_group<1>(vr, soff, row_scale, lane_sub, b.x);
  if (steps <= 2 * kStepGroup) {
    multiply_group<0>(g0, b.y, acc);
    if (steps > 1 * kStepGroup) multiply_group<1>(g1, b.y, acc);
    return;
  }
  const Group4 g2 = gather_group<2>(vr, soff, row_scale, lane_sub, b.x), g3 = gather_group<3>(vr, soff, row_scale, lane_sub, b.x);
  multiply_group<0>(g0, b.y, acc);
  multiply_group<1>(g1, b.y, acc);
  multiply_group<2>(g2, b.y, acc);
  if (steps > 3 * kStepGroup) multiply_group<3>(g3, b.y, acc);
}

template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// The first `steps` (16 (N - 1) + 4 .. 16 N) steps of N batches as one pipeline, the rows of 24 steps in flight together: for
// workgroups that have a CU to themselves, where nothing else covers the way of the rows and 128 registers are there.  (The
// scheduling barriers keep it so: left to itself the compiler asks for 12 steps' rows at a time, in 67 registers.)
template <int N>
__device__ __forceinline__ void gather_batches(__amdgpu_buffer_rsrc_t vr, uint32_t soff, uint32_t row_scale, uint32_t lane_sub,
                                               const u32x2_t* b, int steps, Acc4& acc) {
  constexpr int kGroups = N * kBatchSteps / kStepGroup, kAhead = 6;
  Group4 g[kGroups];
  auto load = [&](auto i) {
    constexpr int I = decltype(i)::value;
    if constexpr (I < kGroups) g[I] = gather_group<I % 4>(vr, soff, row_scale, lane_sub, b[I / 4].x);
  };
  for_each_index(load, std::make_integer_sequence<int, kAhead>{});
  __builtin_amdgcn_sched_barrier(0);
  for_each_index(
      [&](auto i) {
        constexpr int I = decltype(i)::value;
        if (I <= 4 * (N - 1) || steps > I * kStepGroup) multiply_group<I % 4>(g[I], b[I / 4].y, acc);
        load(std::integral_constant<int, I + kAhead>{});
        __builtin_amdgcn_sched_barrier(0);
      },
      std::make_integer_sequence<int, kGroups>{});
}
template <int B>
__device__ __forceinline__ void gather_slice(__amdgpu_buffer_rsrc_t vr, uint32_t soff, uint32_t row_scale, uint32_t lane_sub,
                                             const u32x2_t (&b)[B], int steps, Acc4& acc) {
  if (steps > 2 * kBatchSteps) {
    if constexpr (B == 3) gather_batches<3>(vr, soff, row_scale, lane_sub, b, steps, acc);
  } else if (steps > kBatchSteps) {
    if constexpr (B >= 2) gather_batches<2>(vr, soff, row_scale, lane_sub, b, steps, acc);
  } else if (steps > 0) {
    gather_batch(vr, soff, row_scale, lane_sub, b[0], steps, acc);
  }
}

// Grid: tile blocks * slices.  B batches a slice.
template <int R, int NW, int B>
__global__ __launch_bounds__(NW * 64, NW == 16 ? 4 : 6) void product_output_kernel(
    const float* __restrict__ V, float* __restrict__ out, const uint32_t* __restrict__ wpk, uint32_t wpk_bytes,
    const uint8_t* __restrict__ lens, const OutTile* __restrict__ otiles, int C, int K, int Tp, int KC,
    int n_slices, uint32_t v_bytes, uint32_t plane, int Wo, uint32_t out_image_stride, uint32_t out_bytes) {
  constexpr int t = R + 1, P = t * t, TB = kTileBlock, PPW = P / NW;
  static_assert(P % NW == 0 && NW >= kSliceRows, "every wave has as many positions; a wave per row afterwards");
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  constexpr uint32_t kParked = 0xfffffff0u;
  __shared__ __attribute__((aligned(16))) float m_lds[P][kSliceRows][TB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane_sub = (uint32_t)(lane & 15) * 16u;
  const int vid = xcd_contiguous_id(blockIdx.x, gridDim.x);  // the slices of a tile block on one XCD: they share its V
  const int tb = vid / n_slices, slice = vid - tb * n_slices;
  const int kc = slice / kFusedWaves, w = slice % kFusedWaves;
  const __amdgpu_buffer_rsrc_t vr = make_rsrc(V, v_bytes), wr = make_rsrc(wpk, wpk_bytes);
  const u32x4_t o = *reinterpret_cast<const u32x4_t*>(otiles + (size_t)tb * TB + lane);  // (n, pix, valid, -)
  // The first two batches come with the lengths, a third where the length says that there is one (parked otherwise: no
  // memory is touched).
  constexpr int kAtOnce = B < 2 ? B : 2;
  u32x2_t b[PPW][B];
  int len[PPW];
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    const int p = wave * PPW + i;
    len[i] = (int)lens[((size_t)p * KC + kc) * kFusedWaves + w];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u)
      b[i][u] = __builtin_amdgcn_raw_buffer_load_b64(wr, lane * 8, (int)(((((uint32_t)p * KC + kc) * B + u) * kFusedWaves + w) * 512u), 0);
  }
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    len[i] = __builtin_amdgcn_readfirstlane(len[i]);
    if constexpr (B > kAtOnce) {
      const uint32_t at = ((((uint32_t)(wave * PPW + i) * KC + kc) * B + kAtOnce) * kFusedWaves + w) * 512u;
      b[i][kAtOnce] =
          __builtin_amdgcn_raw_buffer_load_b64(wr, lane * 8, (int)(len[i] > kAtOnce * kBatchSteps ? at : 0xfffff000u), 0);
    }
  }
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    const int p = wave * PPW + i;
    const uint32_t soff = ((uint32_t)p * C * Tp + (uint32_t)tb * TB) * 4u, scale = (uint32_t)Tp / TB;  // 256 c -> 4 c Tp
    Acc4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (NW == 16) {
      gather_slice(vr, soff, scale, lane_sub, b[i], len[i], acc);
    } else {
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int steps = len[i] - u * kBatchSteps;
        if (steps > 0) gather_batch(vr, soff, scale, lane_sub, b[i][u], steps, acc);
      }
    }
    const f32x4_t m = {acc.a0, acc.a1, acc.a2, acc.a3};
    *reinterpret_cast<f32x4_t*>(&m_lds[p][lane >> 4][(lane & 15) * 4]) = m;
  }
  __syncthreads();
  const int k = slice * kSliceRows + wave;
  if (wave >= kSliceRows || k >= K) return;
  float z[t][t], y[2][2];
#pragma unroll
  for (int i = 0; i < t; ++i)
#pragma unroll
    for (int j = 0; j < t; ++j) z[i][j] = m_lds[i * t + j][wave][lane];
  output_transform<2, R>(z, y);
  const __amdgpu_buffer_rsrc_t orr = make_rsrc(out, out_bytes);
  const int rows = (int)(o.z & 0xffffu), cols = (int)(o.z >> 16);
  const uint32_t at = (o.x * (uint32_t)out_image_stride + (uint32_t)k * plane + o.y) * 4u;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const uint32_t row_at = a < rows ? at + (uint32_t)(a * Wo) * 4u : kParked;
    buffer_store_f32x2<SWCONV_AUX_OUT>(orr, cols > 1 ? row_at : kParked, 0u, y[a][0], y[a][1]);
    buffer_store_f32<SWCONV_AUX_OUT>(orr, cols == 1 ? row_at : kParked, 0u, y[a][0]);
  }
}

// ---------------------------------------------------------------------------------------------
// Steps 2 and 3 in one kernel for F(4x4,3x3) (t = 6, P = 36, 16 outputs per tile and row).
//
// Same decomposition as above - a workgroup of 16 waves owns one 64-tile block and 64 rows of W_F
// through all 36 positions, a wave four rows, a lane one row and four tiles - with the memory side
// rebuilt around the register file: the lane's 4 x 16 output accumulators and the 16 row sums take
// 80 of the 128 vector registers a wave has at 16 waves per CU.
//   - The C x 64 panel of a position goes from memory straight into LDS (16-byte direct loads:
//     the 64 lanes of a load fill 1024 consecutive bytes of LDS = four panel rows), two panel
//     buffers, one barrier per position: the panel of position p + 1 arrives while p is computed.
//     The two buffers are two separate arrays, which is what lets the compiler see that work on
//     one never has to wait for a direct load into the other.
//   - The weights do not pass through LDS: a lane fetches its own (row offset, weight) pairs, 16
//     steps per load.  Two sets of two batch registers in turn: while a position runs on one set,
//     the other receives the first two batches of the next position, a whole position ahead.
//   - Inner loop: the steps of a slice run as one rolling pipeline - the panel read of step s + 4
//     is issued right after the multiply-adds of step s, so a wave always has four LDS reads in
//     flight.  With the waves of a workgroup re-aligned by the barrier of every position, reads
//     issued group by group would leave LDS idle while all waves multiply and the vector ALU idle
//     while all wait.  A unit of the pipeline is two batches (32 steps), written in assembly
//     with fixed registers for the four reads in flight, and left after the slice's last group of
//     four steps.
//   - The fold Y += A^T[.][i] (x) sum_j A^T[.][j] M[(i,j)] runs per position on the lane's four
//     values (column factor) and once per row of positions (row factor).
//   - Epilogue: the 4 x 4 outputs go through LDS (the panels are done with) into the layout of the
//     output rows, one row of W_F at a time per wave, and leave as whole rows with lane-contiguous
//     stores, as in the stand-alone output transform.
// M (36 floats per output tile and row; 16 are stored) never exists in memory.
//
// Requires C % 4 == 0 (a direct load covers four whole rows), C <= 256 (the two panel arrays) and
// an output staging area of at most 2048 floats per wave.  G = ceil(C / 64) direct loads per wave
// and panel; a wave with fewer row groups than G repeats the panel's first group.
// Weight packages: wpk[p][kc][b][wave], B batches per slice and position (B even: whole units);
// lens[p][kc*16 + wave] = steps of the slice (a multiple of 4).

constexpr int kFused4MaxBatches = 14;  // steps of a slice must fit the 8-bit length table
constexpr int kFused4MaxC = 256;       // rows of a panel array
constexpr int kFused4MaxOutArea = kFused4MaxC * kTileBlock / (kFusedWaves / 2);  // floats per wave: eight waves per array

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// The rolling unit of the inner loop (unit_rolling_hi: its reads in flight live in v[112:127]) is
// defined in swconv_kernels.hpp.

// Row a of A^T of F(4,3) at column i: (1, p, p^2, p^3) for the points p = 0, 1, -1, 2, -2 and
// (0, 0, 0, 1) for the point at infinity (i = 5).
__device__ __forceinline__ void at_column(int i, float (&c)[4]) {
  const float pt = i == 1 ? 1.0f : i == 2 ? -1.0f : i == 3 ? 2.0f : i == 4 ? -2.0f : 0.0f;
  c[0] = i < 5 ? 1.0f : 0.0f;
  c[1] = pt;
  c[2] = pt * pt;
  c[3] = pt * pt * pt + (i == 5 ? 1.0f : 0.0f);
}

template <int R, int G>
__global__ __launch_bounds__(kFusedWaves * 64) void product_output4_kernel(
    const float* __restrict__ V, float* __restrict__ out, const uint32_t* __restrict__ wpk, uint32_t wpk_bytes,
    const uint8_t* __restrict__ lens, const TileInfo* __restrict__ tiles, const BlockImage* __restrict__ blocks,
    int KC, int B, int n_wgs, const Geometry g) {
  static_assert(R == 3, "F(4x4,3x3)");
  constexpr int t = R + 3, P = t * t, NW = kFusedWaves, TB = kTileBlock;
  static_assert(P <= 64 && P % 2 == 0, "one lane per position holds the slice length; positions run in pairs");
  static_assert(G >= 1 && (G - 1) * NW * 4 < kFused4MaxC, "G direct loads per wave cover up to 64 G rows");
  __shared__ __attribute__((aligned(1024))) float panel_even[kFused4MaxC * TB];  // panels of the even positions
  __shared__ __attribute__((aligned(1024))) float panel_odd[kFused4MaxC * TB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int quarter = lane >> 4;
  const uint32_t lane_sub = (uint32_t)(lane & 15) * 16u;
  const int vid = xcd_contiguous_id(blockIdx.x, n_wgs);  // the KC workgroups of a tile block are neighbours on one XCD
  const int tb = vid / KC, kc = vid - tb * KC;
  const int C = g.C, Tp = g.Tp;
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(wpk, wpk_bytes), vr = make_rsrc(V, g.v_bytes);

  // the lane's view of its wave's slice lengths: lane l holds the length at position l
  const int spp = KC * NW;
  const int lens_v = lane < P ? (int)lens[(size_t)lane * spp + kc * NW + wave] : 0;

  // Panel loads: load u of wave w moves the row group 16 u + w (rows 4 (16 u + w) .. + 3), or group
  // 0 again where the panel has no such group; lane l fetches piece l % 16 of row l / 16 of them.
  const uint32_t voff = ((uint32_t)(lane >> 4) * (uint32_t)Tp) * 4u + lane_sub;
  int group_of[G];
#pragma unroll
  for (int u = 0; u < G; ++u) group_of[u] = u * NW + wave < C / 4 ? u * NW + wave : 0;
  auto fetch_panel = [&](int p, float* dst) {
    const uint32_t soff = ((uint32_t)p * C * Tp + (uint32_t)tb * TB) * 4u;
#pragma unroll
    for (int u = 0; u < G; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (lds_ptr_t)(dst + group_of[u] * 256), 16, (int)voff,
                                               (int)(soff + (uint32_t)group_of[u] * (uint32_t)Tp * 16u), 0, 0);
  };

  // weight batches of this wave: position p, batch b at ((p KC + kc) B + b) * NW * 512 + wave * 512
  const uint32_t lane8 = (uint32_t)lane * 8u;
  const uint32_t pos_bytes = (uint32_t)KC * B * NW * 512u;
  const uint32_t w0 = ((uint32_t)kc * B * NW + wave) * 512u;
  constexpr uint32_t kBatchStride = NW * 512u;
  auto load_batch = [&](uint32_t byte_off) -> u32x2_t {
    return __builtin_amdgcn_raw_buffer_load_b64(wr, (int)lane8, (int)byte_off, 0);  // past the end: reads 0
  };

  Acc4 y[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) y[a][b] = Acc4{0.0f, 0.0f, 0.0f, 0.0f};
  Acc4 r0 = {0.0f, 0.0f, 0.0f, 0.0f}, r1 = r0, r2 = r0, r3 = r0;  // sum_j A^T[b][j] M[(i,j)], b = 0 .. 3

  // One position: its panel is in `panel`, its first two weight batches in (c0, c1); meanwhile the
  // panel of the next position goes into `other` and its first batches into (n0, n1).
  auto position = [&](int p, const float* panel, float* other, u32x2_t& c0, u32x2_t& c1, u32x2_t& n0, u32x2_t& n1) {
    // every wave has finished position p - 1 (which read the array that is filled next) and has
    // waited for its share of panel p
    __syncthreads();
    const uint32_t cur = (uint32_t)p * pos_bytes + w0;
    const uint32_t nxt = p + 1 < P ? cur + pos_bytes : 0xffff0000u;  // parked past the end after the last position
    if (p + 1 < P) fetch_panel(p + 1, other);
    n0 = load_batch(nxt);
    n1 = load_batch(nxt + kBatchStride);
    // an empty slice runs one group of steps on all-zero pairs: no branch around the pipeline
    const int len = max(__builtin_amdgcn_readlane(lens_v, p), kStepGroup);
    const int units = (len + kUnitSteps - 1) / kUnitSteps;
    const uint32_t lane_base = (uint32_t)(uintptr_t)(lds_ptr_t)panel + lane_sub;
    Acc4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    unit_rolling_hi(lane_base, c0, c1, min(len, kUnitSteps), acc);
    for (int u = 1; u < units; ++u) {  // a slice of more than 32 steps: further batches, fetched as they are needed
      const u32x2_t e0 = load_batch(cur + (uint32_t)(2 * u) * kBatchStride);
      const u32x2_t e1 = load_batch(cur + (uint32_t)(2 * u + 1) * kBatchStride);
      unit_rolling_hi(lane_base, e0, e1, min(len - u * kUnitSteps, kUnitSteps), acc);
    }
    // column j of A^T
    const int j = p % t;
    float cc[4];
    at_column(j, cc);
    acc_fma(r0, cc[0], acc);
    acc_fma(r1, cc[1], acc);
    acc_fma(r2, cc[2], acc);
    acc_fma(r3, cc[3], acc);
    if (j == t - 1) {  // row i of positions is complete: Y[a][b] += A^T[a][i] * r_b
      float rc[4];
      at_column(p / t, rc);
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        acc_fma(y[a][0], rc[a], r0);
        acc_fma(y[a][1], rc[a], r1);
        acc_fma(y[a][2], rc[a], r2);
        acc_fma(y[a][3], rc[a], r3);
      }
      r0 = r1 = r2 = r3 = Acc4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // this wave's share of panel p + 1 is in LDS and the next batches are in their registers (both
    // were asked for a whole position ago)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  };

  fetch_panel(0, panel_even);
  u32x2_t ca0 = load_batch(w0), ca1 = load_batch(w0 + kBatchStride), cb0 = {0u, 0u}, cb1 = {0u, 0u};
  __builtin_amdgcn_s_waitcnt(0x0f70);
  for (int p = 0; p < P; p += 2) {
    position(p, panel_even, panel_odd, ca0, ca1, cb0, cb1);
    position(p + 1, panel_odd, panel_even, cb0, cb1, ca0, ca1);
  }

  // Epilogue.  Every wave has an LDS area laid out like the output rows its tile block covers (the
  // tables of the stand-alone output transform say where a tile's pixels go and which runs of whole
  // rows the block has in each image), eight waves per panel array.  Row by row of W_F: the 16
  // lanes of the row's quarter drop their 4 x 4 outputs there, then all 64 lanes write the runs out
  // with lane-contiguous stores.  LDS executes a wave's operations in order, so inside a wave no
  // barrier is needed.
  __syncthreads();  // every wave is done with the panels
  float* my = (wave < NW / 2 ? panel_even : panel_odd) + (size_t)(wave % (NW / 2)) * g.out_area;
  const TileInfo* ti = tiles + (size_t)tb * TB + (lane & 15) * 4;
  const TileInfo ti0 = ti[0], ti1 = ti[1], ti2 = ti[2], ti3 = ti[3];
  const BlockImage* bi = blocks + (size_t)tb * g.slots;
  const size_t plane = (size_t)g.Ho * g.Wo;
  for (int q = 0; q < kSliceRows; ++q) {
    const int k = kc * kFusedRows + wave * kSliceRows + q;  // wave-uniform
    if (k >= g.K) break;
    if (quarter == q) {
      auto drop = [&](const TileInfo& tile, auto pick) {
        const int y0 = (int16_t)(tile.yx0 & 0xffff), x0 = tile.yx0 >> 16;
        // rows / columns of the tile inside the output (<= 0 for a padding tile, whose y0 is -32768)
        const int rows = y0 == -32768 ? 0 : g.Ho - (y0 + g.pad), cols = g.Wo - (x0 + g.pad);
        float* px = my + tile.out_org;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            if (a < rows && b < cols) px[a * g.Wo + b] = pick(y[a][b]);
      };
      drop(ti0, [](const Acc4& v) { return v.a0; });
      drop(ti1, [](const Acc4& v) { return v.a1; });
      drop(ti2, [](const Acc4& v) { return v.a2; });
      drop(ti3, [](const Acc4& v) { return v.a3; });
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the drops are in LDS before any lane reads them
    for (int sidx = 0; sidx < g.slots; ++sidx) {
      const BlockImage b = bi[sidx];
      if (b.n < 0) continue;
      const float* src = my + b.out_off;
      float* dst = out + (size_t)b.n * g.out_image_stride + k * plane + b.out_elem0;
      // stores past the part's end are dropped by the descriptor: no lane predicate
      const __amdgpu_buffer_rsrc_t orr = make_rsrc(dst, (uint32_t)b.out_span * 4u);
      if (b.whole) {
        for (int e0 = 0; e0 < b.out_span; e0 += 64)
          buffer_store_f32<SWCONV_AUX_OUT>(orr, lane * 4u, e0 * 4u, src[e0 + lane]);
      } else {
        const int row_first = b.out_elem0 / g.Wo;  // wave-uniform
        for (int e0 = 0; e0 < b.out_span; e0 += 64) {
          const int e = e0 + lane;
          const int ry = (int)__umulhi((uint32_t)e, g.wo_magic), x = e - ry * g.Wo;
          const int tl = ((row_first + ry) >> g.m_shift) * g.tw + (x >> g.m_shift);
          const bool mine = tl >= b.t_lo && tl <= b.t_hi;  // a pixel of a tile of this block
          buffer_store_f32<SWCONV_AUX_OUT>(orr, mine ? lane * 4u : 0xfffffff0u, e0 * 4u, src[e]);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads are done before the next row's drops
  }
}

}  // namespace swconv
