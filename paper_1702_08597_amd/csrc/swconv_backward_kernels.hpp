// HIP kernels of the backward pass of the Winograd layer (Section 3, Eq. 5 and Eq. 6) for gfx950.
//
//   dZ  [P][K][Tp]   dL/dZ = A dL/dO~ A^T            (Eq. 5, first line)   - held in the M workspace
//   dW               dL/dW_F(k,c,p) = sum_tau dZ[p][k][tau] V[p][c][tau] at the stored entries (Eq. 5)
//   dV  [P][C][Tp]   dL/dI_F[p] = W_F[p]^T dZ[p]     (Eq. 6, first line): the sparse product kernel of the
//                    forward pass, run on the packed transpose of W_F
//   dI~ [P][C][Tp]   dL/dI~ = B dL/dI_F B^T          (Eq. 6, second line), one t x t patch per (c, tile),
//                    stored position-major like V
//   dI  [N][C][H][W] every pixel sums the patch entries phi maps to it (Eq. 6, third line)
//
// Layouts, tile order and the index tables are those of the forward kernels.
#pragma once
#include "swconv_kernels.hpp"

namespace swconv {

// ---------------------------------------------------------------------------------------------
// Eq. 5, first line.  A wave owns one output channel and 64 consecutive tiles: it copies the rows
// of dL/dO its tiles own into its LDS area with lane-contiguous loads (the staging layout of the
// output transform, read instead of written), every lane gathers its m x m tile - zero where the
// tile reaches past H_o x W_o: those outputs were dropped by psi and carry no gradient -
// transforms it in registers and stores one value per position.
template <int M, int R>
__global__ __launch_bounds__(256) void output_grad_transform_kernel(const float* __restrict__ dout,
                                                                    float* __restrict__ dZ,
                                                                    const TileInfo* __restrict__ tiles,
                                                                    const BlockImage* __restrict__ blocks,
                                                                    const Geometry g) {
  constexpr int t = Wino<M, R>::t;
  extern __shared__ float stage[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = blockIdx.y * 4 + wave;
  const int tau0 = blockIdx.x * 64;
  float* my = stage + wave * g.out_area;
  const BlockImage* bi = blocks + (size_t)blockIdx.x * g.slots;
  const size_t plane = (size_t)g.Ho * g.Wo;
  const TileInfo ti = tiles[tau0 + lane];  // asked for first: it arrives while the rows are staged
  if (k < g.K) {
    auto part = [&](const BlockImage& b) {
      return StagedPart{dout + (size_t)max(b.n, 0) * g.out_image_stride + k * plane + b.out_elem0, b.out_span, b.out_off};
    };
    stage_parts<1>(bi, g.slots, g.out_longest, my, lane, part);
  }
  __syncthreads();
  if (k >= g.K) return;
  float gr[M][M];
  {
    const int y0 = (int16_t)(ti.yx0 & 0xffff), x0 = ti.yx0 >> 16;
    // rows / columns of the tile inside the output (<= 0 for a padding tile, whose y0 is -32768)
    const int rows = y0 == -32768 ? 0 : g.Ho - (y0 + g.pad), cols = g.Wo - (x0 + g.pad);
    const float* px = my + ti.out_org;
#pragma unroll
    for (int a = 0; a < M; ++a)
#pragma unroll
      for (int b = 0; b < M; ++b) {
        const bool inside = a < rows && b < cols;
        const float v = px[inside ? a * g.Wo + b : 0];  // a staged address in any case (a padding tile reads offset 0)
        gr[a][b] = inside ? v : 0.0f;
      }
  }
  float z[t][t];
  output_grad_transform<M, R>(gr, z);
  const __amdgpu_buffer_rsrc_t zr = make_rsrc(dZ, g.m_bytes);
  const uint32_t pstride = (uint32_t)g.K * (uint32_t)g.Tp * 4u;
  uint32_t soff = ((uint32_t)k * g.Tp + tau0) * 4u;
#pragma unroll
  for (int i = 0; i < t; ++i)
#pragma unroll
    for (int j = 0; j < t; ++j) {
      buffer_store_f32<SWCONV_AUX_M>(zr, lane * 4u, soff, z[i][j]);
      soff += pstride;
      asm volatile("" : "+s"(soff));
    }
}

// ---------------------------------------------------------------------------------------------
// Eq. 6, second line.  A wave owns one input channel and 64 consecutive tiles: each lane reads the
// t*t values dL/dI_F(c, tau, :, :) (256 contiguous bytes per wave and position), applies B . B^T in
// registers and stores the t x t patch dL/dI~(c, tau, :, :), again one value per position.
template <int M, int R>
__global__ __launch_bounds__(256) void input_grad_patch_kernel(const float* __restrict__ dV,
                                                               float* __restrict__ patches, const Geometry g) {
  constexpr int t = Wino<M, R>::t;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blockIdx.y * 4 + wave;
  const int tau0 = blockIdx.x * 64;
  if (c >= g.C || tau0 >= g.T) return;
  const __amdgpu_buffer_rsrc_t src = make_rsrc(dV, g.v_bytes), dst = make_rsrc(patches, g.v_bytes);
  const uint32_t row0 = ((uint32_t)c * g.Tp + tau0) * 4u;
  const uint32_t pstride = (uint32_t)g.C * (uint32_t)g.Tp * 4u;
  float f[t][t], d[t][t];
  uint32_t soff = row0;
#pragma unroll
  for (int i = 0; i < t; ++i)
#pragma unroll
    for (int j = 0; j < t; ++j) {
      f[i][j] = buffer_load_f32(src, lane * 4u, soff);
      soff += pstride;
      asm volatile("" : "+s"(soff));
    }
  input_grad_transform<M, R>(f, d);
  soff = row0;
#pragma unroll
  for (int a = 0; a < t; ++a)
#pragma unroll
    for (int b = 0; b < t; ++b) {
      buffer_store_f32<SWCONV_AUX_V>(dst, lane * 4u, soff, d[a][b]);
      soff += pstride;
      asm volatile("" : "+s"(soff));
    }
}

// ---------------------------------------------------------------------------------------------
// Eq. 6, third line, as a gather.  The input plane is cut into m x m cells aligned with the tile
// stride: cell (qy, qx) holds the pixels y = qy*m - pad + ry, x = qx*m - pad + rx.  Every pixel of a
// cell receives from the same tiles (qy - dy, qx - dx), dy, dx in 0 .. (t-1)/m (one tile back for
// the 3x3 filters, two for F(2x2,5x5)), the patch entry (ry + m*dy, rx + m*dx) where that lies
// inside the t x t patch.  A
// thread owns one cell of one (n, c) plane and lanes run over consecutive cells, i.e. consecutive
// tiles, so every patch load of a wave is a contiguous run of one position plane and each patch
// entry is read exactly once; each pixel is written once, its sum taken in ascending tile order.
// Threads run over all cells of all (n, c) planes.
template <int M, int R>
__global__ __launch_bounds__(256) void input_grad_gather_kernel(const float* __restrict__ patches,
                                                                float* __restrict__ din, const Geometry g) {
  constexpr int t = Wino<M, R>::t;
  constexpr int back = (t - 1) / M;  // tiles before its own that still cover a cell, per dimension
  const int cells_y = (g.H - 1 + g.pad) / M + 1, cells_x = (g.W - 1 + g.pad) / M + 1;
  const int cells = cells_y * cells_x;
  const uint32_t idx = blockIdx.x * 256u + threadIdx.x;  // (n, c) plane major, cells of a plane consecutive
  if (idx >= (uint32_t)g.N * g.C * cells) return;
  const int nc = idx / cells, cell = idx - nc * cells;
  const int n = nc / g.C, c = nc - n * g.C;
  const int qy = cell / cells_x, qx = cell - qy * cells_x;
  const __amdgpu_buffer_rsrc_t src = make_rsrc(patches, g.v_bytes);
  const uint32_t pstride = (uint32_t)g.C * (uint32_t)g.Tp;  // floats between positions
  float acc[M][M];
#pragma unroll
  for (int ry = 0; ry < M; ++ry)
#pragma unroll
    for (int rx = 0; rx < M; ++rx) acc[ry][rx] = 0.0f;
  // tiles in ascending order: (qy-back, qx-back), ..., (qy, qx)
#pragma unroll
  for (int dy = back; dy >= 0; --dy) {
    const int ty = qy - dy;
#pragma unroll
    for (int dx = back; dx >= 0; --dx) {
      const int tx = qx - dx;
      if (ty < 0 || ty >= g.th || tx < 0 || tx >= g.tw) continue;
      const uint32_t base = ((uint32_t)c * g.Tp + (uint32_t)(n * g.th + ty) * g.tw + tx) * 4u;
#pragma unroll
      for (int ry = 0; ry < M; ++ry)
#pragma unroll
        for (int rx = 0; rx < M; ++rx) {
          const int a = ry + M * dy, b = rx + M * dx;  // compile-time after unrolling
          if (a < t && b < t) acc[ry][rx] += buffer_load_f32(src, base + (uint32_t)(a * t + b) * pstride * 4u, 0);
        }
    }
  }
  float* plane = din + (size_t)n * g.in_image_stride + (size_t)c * g.H * g.W;
#pragma unroll
  for (int ry = 0; ry < M; ++ry) {
    const int y = qy * M - g.pad + ry;
    if (y < 0 || y >= g.H) continue;
#pragma unroll
    for (int rx = 0; rx < M; ++rx) {
      const int x = qx * M - g.pad + rx;
      if (x >= 0 && x < g.W) plane[y * g.W + x] = acc[ry][rx];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Eq. 5, second line, last step: the per-tile-block partial sums of every stream entry (written by
// the sparse kernel with DOTS) are added over the tile blocks, in ascending order, and go to
// the entry's place in the caller's CSR order; padding entries (index -1) are skipped.
struct PartialSums {
  const float* partial;
  int n_tau_blocks;
  uint32_t stride;             // floats between tile blocks
  const int32_t* entry_index;
  uint32_t n_entries;
  float* dvals;
};
constexpr int kReduceThreads = 256;
__device__ __forceinline__ void reduce_partial_sums(const PartialSums& s, uint32_t block) {
  const uint32_t e = block * (uint32_t)kReduceThreads + threadIdx.x;
  if (e >= s.n_entries) return;
  const int32_t q = s.entry_index[e];
  if (q < 0) return;
  // eight loads in flight, added in ascending order of the tile block
  float sum = 0.0f;
  int tb = 0;
  for (; tb + 8 <= s.n_tau_blocks; tb += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = s.partial[(size_t)(tb + u) * s.stride + e];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += v[u];
  }
  for (; tb < s.n_tau_blocks; ++tb) sum += s.partial[(size_t)tb * s.stride + e];
  s.dvals[q] = sum;
}
__global__ __launch_bounds__(kReduceThreads) void weight_grad_reduce_kernel(PartialSums s) {
  reduce_partial_sums(s, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// Eq. 6, second and third line in one kernel, for images whose planes fit LDS: no patch buffer.
// A wave owns one input channel and a group of G whole images (G = 64 / tiles per image, at least
// 1), whose planes it builds up in LDS.  In passes of 64 consecutive tiles every lane reads the t*t
// values dL/dI_F(c, tau, :, :) and applies B . B^T in registers.  Patches of neighbouring tiles overlap by
// R - 1 pixels (at most m: no patch reaches past its neighbour), and the overlaps are summed where that is cheapest:
//   - columns in registers: a lane takes the last R - 1 columns of the tile to its left from the lane before it
//     (DPP shift by one lane; the pass before hands lane 63's over in scalar registers);
//   - rows through LDS: every tile stores its last R - 1 rows into the plane, then reads what the tile above
//     has stored where its own first R - 1 rows go, adds and stores.
// LDS executes a wave's operations in order, so the sums have a fixed order, and every pixel is stored at least
// once: the planes need no zeroing.  Then the wave writes its planes with lane-contiguous stores.
// LDS was the bound: adding whole patches in four phases of disjoint tiles takes 8 t^2 = 288 LDS instructions a pass
// for F(4x4,3x3), this 32 and the right edge's.  32 images of 56 x 56, 256 channels: 104 -> 78 us (4.3 TB/s; three
// workgroups fit a CU's LDS); 64 of 13 x 13, 384 channels: 21.1 -> 16.2 us; F(4x4,5x5), 32 of 27 x 27, 48 channels, whose
// indices of whole patches overflowed the registers: 10.4 us against 16.5 for the patch and gather kernels.
// PREFETCH: groups of more than one pass ask for the next pass's values before they work on the present one's, at
// t^2 registers that groups of one pass spend on more waves per SIMD.  F(4x4,5x5), with 64 values per lane, spills 53
// to 56 scalar registers into vector lanes (nothing goes to memory).
// Block = 4 waves = 4 channels of the same image group.
// SUMS: the workgroups behind those of the channels (blockIdx.y from ceil(C / 4) on) add up the weight gradient's partial
// sums instead, which the kernel in front of this one has left too: one launch and its ramp less.
struct GradTile {
  int32_t org;  // float offset of pixel (0, 0) of the tile's image inside the wave's LDS area
  int32_t yx0;  // as TileInfo::yx0; y0 = x0 = -32768 for tiles past the last image
};

template <int M, int R, bool PREFETCH, bool SUMS>
__global__ __launch_bounds__(256) void input_grad_kernel(const float* __restrict__ dV, float* __restrict__ din,
                                                         const GradTile* __restrict__ gtiles, int images_per_group,
                                                         const Geometry g, const PartialSums sums) {
  static_assert(kReduceThreads == 256, "the sums' workgroups are this kernel's");
  if constexpr (SUMS) {
    const uint32_t channel_wgs = (uint32_t)(g.C + 3) / 4u;
    if (blockIdx.y >= channel_wgs) return reduce_partial_sums(sums, (blockIdx.y - channel_wgs) * gridDim.x + blockIdx.x);
  }
  constexpr int t = Wino<M, R>::t;
  constexpr int ov = t - M;  // columns (rows) that a patch shares with the next one
  static_assert(ov <= M, "a patch reaches no further than its neighbour");
  extern __shared__ float stage[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blockIdx.y * 4 + wave;
  if (c >= g.C) return;  // no barrier in this kernel: waves are independent
  const int n0 = blockIdx.x * images_per_group;
  const int n_img = min(images_per_group, g.N - n0);
  const int plane = g.H * g.W;
  const int area = images_per_group * plane;
  const int area_padded = (area + 63) / 64 * 64;  // the wave's planes, then one spare float per lane
  float* my = stage + (size_t)wave * (area_padded + 64);
  const int spare = area_padded + lane;  // entries outside the image go here
  const __amdgpu_buffer_rsrc_t src = make_rsrc(dV, g.v_bytes);
  const uint32_t pstride = (uint32_t)g.C * (uint32_t)g.Tp * 4u;
  const int tau0 = n0 * g.tpi, tau_end = tau0 + n_img * g.tpi;
  auto load = [&](int base, float (&f)[t][t], GradTile& gt) {
    const int tau = base + lane;
    // lanes past the group's last tile are parked past the end of the buffer: they read zeros
    const uint32_t voff = tau < tau_end ? ((uint32_t)c * g.Tp + (uint32_t)tau) * 4u : 0xfffffff0u;
    uint32_t soff = 0;
#pragma unroll
    for (int i = 0; i < t; ++i)
#pragma unroll
      for (int j = 0; j < t; ++j) {
        f[i][j] = buffer_load_f32(src, voff, soff);
        soff += pstride;
        asm volatile("" : "+s"(soff));
      }
    gt = gtiles[tau < tau_end ? tau : tau0];
  };
  float carry[t][ov];  // the last columns of the tile before this pass's first one
#pragma unroll
  for (int a = 0; a < t; ++a)
#pragma unroll
    for (int b = 0; b < ov; ++b) carry[a][b] = 0.0f;
  float f[t][t];
  GradTile gt;
  load(tau0, f, gt);
  for (int base = tau0; base < tau_end; base += 64) {
    float d[t][t];
    const GradTile at = gt;
    input_grad_transform<M, R>(f, d);
    if constexpr (PREFETCH)
      if (base + 64 < tau_end) load(base + 64, f, gt);
    const bool live = base + lane < tau_end;
    const int y0 = (int16_t)(at.yx0 & 0xffff), x0 = at.yx0 >> 16;
    const bool left = x0 > -g.pad, above = y0 > -g.pad;  // the tile has a neighbour there
#pragma unroll
    for (int a = 0; a < t; ++a)
#pragma unroll
      for (int b = 0; b < ov; ++b) {
        const int mine = __builtin_bit_cast(int, d[a][M + b]);
        const float from_left = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, carry[a][b]), mine, 0x138, 0xf, 0xf, false));  // wave_shr:1
        d[a][b] += left ? from_left : 0.0f;
        carry[a][b] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(mine, 63));
      }
    // LDS index of an entry; columns M .. t-1 are the next tile's, except behind the last tile of a row
    const bool last_column = x0 + g.pad == (g.tw - 1) * M;
    const int org = at.org + y0 * g.W + x0;
    auto index = [&](int a, int b) -> int {
      const int y = y0 + a, x = x0 + b;
      return live && y >= 0 && y < g.H && x >= 0 && x < g.W ? org + a * g.W + b : spare;
    };
    // whether a column behind the last tile is inside the image (uniform)
    auto edge = [&](int b) { return (g.tw - 1) * M - g.pad + b < g.W; };
    auto store = [&](int a) {
#pragma unroll
      for (int b = 0; b < M; ++b) my[index(a, b)] = d[a][b];
#pragma unroll
      for (int b = M; b < t; ++b)
        if (edge(b)) my[last_column ? index(a, b) : spare] = d[a][b];
    };
#pragma unroll
    for (int a = ov; a < t; ++a) store(a);  // rows of this tile alone, and the first rows of the tile below
    // the reads below see what other lanes stored above: keep the compiler from moving LDS accesses across
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float up[ov][t];
#pragma unroll
    for (int a = 0; a < ov; ++a) {
#pragma unroll
      for (int b = 0; b < M; ++b) up[a][b] = my[index(a, b)];
#pragma unroll
      for (int b = M; b < t; ++b) up[a][b] = edge(b) ? my[last_column ? index(a, b) : spare] : 0.0f;
    }
#pragma unroll
    for (int a = 0; a < ov; ++a) {
#pragma unroll
      for (int b = 0; b < t; ++b) d[a][b] += above ? up[a][b] : 0.0f;
      store(a);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if constexpr (!PREFETCH)
      if (base + 64 < tau_end) load(base + 64, f, gt);
  }
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  for (int i = 0; i < n_img; ++i) {
    const float* from = my + (size_t)i * plane;
    const __amdgpu_buffer_rsrc_t dst =
        make_rsrc(din + (size_t)(n0 + i) * g.in_image_stride + (size_t)c * plane, (uint32_t)plane * 4u);
    // lanes past the plane's end read the plane's last floats and store nothing; whole quads start on 16 bytes of LDS
    if (plane % 4 == 0) {
      for (int e0 = 0; e0 < plane; e0 += 256) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(from + min(e0 + lane * 4, plane - 4));
        __builtin_amdgcn_raw_buffer_store_b128(v, dst, lane * 16, e0 * 4, SWCONV_AUX_OUT);
      }
    } else {
      for (int e0 = 0; e0 < plane; e0 += 64)
        buffer_store_f32<SWCONV_AUX_OUT>(dst, lane * 4u, e0 * 4u, from[min(e0 + lane, plane - 1)]);
    }
  }
}

}  // namespace swconv
