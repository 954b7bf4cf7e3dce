// HIP kernels of the sparse Winograd forward pass (Section 5's three steps) for gfx950.
//
// Layouts in device memory (all fp32):
//   in   [N][C][H][W]            caller's NCHW tensor
//   V    [P][C][Tp]              transformed input, position-major, tiles fastest (Section 5:
//                                "the fastest moving dimension is tiles"); Tp = T rounded up to
//                                the tile-block size, the pad columns hold zeros
//   M    [P][K][Tp]              per-position products
//   out  [N][K][Ho][Wo]
// Lanes of a wavefront map to consecutive tiles tau everywhere, so every V/M access of a wave
// is one contiguous 256-byte segment.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "winograd_transforms.hpp"

// Cache policy of the row stores of V, M and the output (buffer-instruction aux bits: 1 = sc0,
// 16 = sc1): write-through.  A kernel's output (19-28 MB on the AlexNet-sized layers) otherwise stays
// dirty in the 32 MB of L2 and is written back when the kernel ends, after the compute instead of
// under it; measured 38.8 -> 35.4 us per forward on the N=32 conv3 layer.
#ifndef SWCONV_AUX_V
#define SWCONV_AUX_V 17
#endif
#ifndef SWCONV_AUX_M
#define SWCONV_AUX_M 17
#endif
#ifndef SWCONV_AUX_OUT
#define SWCONV_AUX_OUT 17
#endif

namespace swconv {

struct Geometry {
  int N, C, H, W, K, pad;
  int Ho, Wo, th, tw, tpi;  // tpi = th*tw tiles per image
  int T;                    // N*tpi
  int Tp;                   // padded tile count (row pitch of V and M)
  // LDS staging of the transforms: a block of 64 consecutive tiles touches at most `slots` images,
  // and in each of them a run of whole rows; the runs of a block lie one behind the other in the
  // wave's staging area, each rounded up to a multiple of 64 floats; `in_area` / `out_area` =
  // floats of the largest such area over all blocks
  int slots, in_area, out_area;
  int in_longest, out_longest;  // floats of the longest run of an image in any block
  uint32_t v_bytes, m_bytes;  // sizes of the V and M workspaces (both below 4 GiB)
  uint32_t wo_magic;          // ceil(2^32 / Wo): e / Wo == umulhi(e, wo_magic) for every staged element index
  int m_shift;                // log2(m)
  // floats between consecutive images of the input (and dL/dI) and of the output (and dL/dO):
  // C*H*W and K*Ho*Wo for dense tensors, larger when the layer works on a channel group of them
  int64_t in_image_stride, out_image_stride;
};

// V and M are addressed through buffer descriptors: address = base + scalar byte offset (the
// row, wave-uniform) + vector byte offset (the lane), so a row access costs no vector address
// arithmetic.  An access whose vector + scalar offset reaches past `bytes` is dropped by the
// hardware (loads return 0); on gfx950 the scalar offset takes part in that check (measured).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float buffer_load_f32(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}
template <int AUX>
__device__ __forceinline__ void buffer_store_f32(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, (int)voff, (int)soff, AUX);
}
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
template <int AUX>
__device__ __forceinline__ void buffer_store_f32x2(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float x,
                                                   float y) {
  u32x2_t d = {__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y)};
  __builtin_amdgcn_raw_buffer_store_b64(d, r, (int)voff, (int)soff, AUX);
}

// Host-built index tables of the transform kernels (no integer division on the device).
// Per tile (Tp entries; padding tiles have y0 = x0 = -32768 so that every pixel reads as zero):
struct TileInfo {
  int32_t in_org;   // staging-area float offset such that input pixel (y,x) sits at in_org + y*W + x
  int32_t yx0;      // first input row y0 = ty*m - pad (low 16 bits, signed) and column x0 (high 16 bits)
  int32_t ylim;     // first (low 16) and last (high 16) staged input row of the tile's image part
  int32_t out_org;  // staging-area float offset of the tile's first output pixel
};
// Per block of 64 consecutive tiles and image slot (Tp/64 * slots entries): the part of one
// image the block covers.  n < 0 marks an unused slot.
struct BlockImage {
  int32_t n;          // image
  int32_t in_elem0;   // first staged input element inside a channel plane (a whole row start)
  int32_t in_span;    // staged input elements (whole rows)
  int32_t out_elem0;  // first output element of the part inside an output plane (a whole row start)
  int32_t out_span;   // output elements of the part (whole rows)
  int32_t t_lo, t_hi; // first / last tile of the block inside the image (image-local tile index)
  int32_t whole;      // 1 when the part consists of whole tile rows (every pixel of the span is owned)
  int32_t in_off;     // float offset of the part's staged input inside the wave's staging area
  int32_t out_off;    // float offset of the part's output rows inside the wave's staging area
};

// One slice = kSliceRows rows of one position's sparse matrix, rows sorted by length.  32 bytes,
// so a wave fetches a whole descriptor with one scalar load.
struct Slice {
  uint32_t batch0;  // first 512-byte batch of the slice in the packed stream
  int32_t len;      // steps in the slice (one (row offset, weight) pair per row each), a multiple of kStepGroup
  int32_t row0;     // index of its first row in the host's sorted-row table (P * Kp entries)
  int32_t p;        // position
  int32_t k[4];     // output channel of each row, -1 = padding row
};

// One unit of the schedule: a contiguous run of slices of one position, for one tile block.
struct WorkItem {
  int32_t p;
  int32_t tau_block;
  int32_t slice_begin;  // first slice
  int32_t slice_end;    // one past the last slice
};

// What a persistent workgroup needs to start, in one 32-byte scalar load: its range of work
// items, the first of them and where the slices of the second begin.
struct RangeHeader {
  int32_t item_begin, item_end;  // indices into the work-item list; never empty for a launched workgroup
  WorkItem first;                // = items[item_begin]
  int32_t second_slice;          // slice_begin of the item behind it, or its own where there is none
  int32_t pad;
};

constexpr int kSliceRows = 4;    // rows per slice = quarters of a wave
constexpr int kTileBlock = 64;   // tiles per panel row: 16 lanes of a quarter x 4 tiles
constexpr int kBatchSteps = 16;  // steps per 512-byte stream batch (one per lane of a quarter)
constexpr int kStepGroup = 4;    // steps issued together; a slice's length is a multiple of it
constexpr int kPanelPieces = 10; // 16-byte panel pieces a thread holds in registers at most
constexpr int kPanelPieces12 = 7;  // the same in workgroups of 12 waves: two of them per CU, so at most 319 channels
constexpr int kMaxItemSlices = 256;  // slices per work item: their descriptors are staged in LDS, two 16-byte
                                     // pieces each, one piece per thread of the smallest workgroup (512 threads)
constexpr int kMinItemSlices = 8;    // the least the LDS left over by a large panel must hold
constexpr int kXcds = 8;
constexpr int kGroupPieces = 2;  // panel pieces that a wave asks for in front of one slice

// Workgroup ids are dealt round-robin to the 8 XCDs; remap them so that each XCD gets one
// contiguous range of virtual ids (neighbours in the work list then share an L2).
__device__ __forceinline__ int xcd_contiguous_id(int bid, int nblocks) {
  const int per = nblocks / kXcds, rem = nblocks % kXcds;
  const int xcd = bid % kXcds, local = bid / kXcds;
  return xcd * per + (xcd < rem ? xcd : rem) + local;
}

// One image's part of a block's rows: where they lie in the tensor, how many floats, where they go in the
// wave's staging area (a run rounded up to a multiple of 64 floats).
struct StagedPart {
  const float* src;
  int span, off;
};

// Copies the parts of a tile block into the wave's LDS area, with the loads of IG images x EL steps in flight before
// the first LDS write.
// stage_dwords: 64 floats a load.  The descriptor ends with the part: lanes past the end read zeros, and as a run is
// padded to a multiple of 64 floats neither loads nor LDS writes need lane predicates.
template <int IG, int EL, typename Part>
__device__ __forceinline__ void stage_dwords(const BlockImage* bi, int slots, float* my, int lane, Part part) {
  for (int s0 = 0; s0 < slots; s0 += IG) {
    __amdgpu_buffer_rsrc_t src[IG];
    float* dst[IG];
    int span[IG], max_span = 0;
#pragma unroll
    for (int i = 0; i < IG; ++i) {
      const BlockImage b = bi[min(s0 + i, slots - 1)];
      const StagedPart pt = part(b);
      span[i] = s0 + i < slots && b.n >= 0 ? pt.span : 0;
      src[i] = make_rsrc(pt.src, (uint32_t)span[i] * 4u);
      dst[i] = my + pt.off + lane;
      max_span = max(max_span, span[i]);
    }
    for (int e0 = 0; e0 < max_span; e0 += 64 * EL) {
      float buf[IG][EL];
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int u = 0; u < EL; ++u)
          if (e0 + u * 64 < span[i]) buf[i][u] = buffer_load_f32(src[i], (lane + u * 64) * 4u, e0 * 4u);
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int u = 0; u < EL; ++u)
          if (e0 + u * 64 < span[i]) dst[i][e0 + u * 64] = buf[i][u];
    }
  }
}
// stage_quads: 256 floats a load.  A row start is only known to be aligned to a float, which is all that a multi-dword
// buffer load needs.  Every load lies wholly inside or wholly outside its descriptor: that covers the whole quads of
// the span, and the one to three floats that remain come by a dword load.  Lanes past the quads write nothing: the
// next part's run may begin there.
template <int IG, int EL, typename Part>
__device__ __forceinline__ void stage_quads(const BlockImage* bi, int slots, float* my, int lane, Part part) {
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  for (int s0 = 0; s0 < slots; s0 += IG) {
    __amdgpu_buffer_rsrc_t src[IG];
    float* dst[IG];
    int span[IG], max_span = 0;
    float tail[IG];
#pragma unroll
    for (int i = 0; i < IG; ++i) {
      const BlockImage b = bi[min(s0 + i, slots - 1)];
      const StagedPart pt = part(b);
      span[i] = s0 + i < slots && b.n >= 0 ? pt.span : 0;
      src[i] = make_rsrc(pt.src, (uint32_t)(span[i] & ~3) * 4u);
      dst[i] = my + pt.off;
      max_span = max(max_span, span[i]);
      if (span[i] & 3)  // one to three lanes of this are used
        tail[i] = buffer_load_f32(make_rsrc(pt.src, (uint32_t)span[i] * 4u), lane * 4u, (uint32_t)(span[i] & ~3) * 4u);
    }
    for (int e0 = 0; e0 < max_span; e0 += 256 * EL) {
      u32x4_t buf[IG][EL];
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int u = 0; u < EL; ++u)
          if (e0 + u * 256 < span[i])
            buf[i][u] = __builtin_amdgcn_raw_buffer_load_b128(src[i], lane * 16, (e0 + u * 256) * 4, 0);
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int u = 0; u < EL; ++u)
          if (e0 + u * 256 < span[i] && e0 + u * 256 + lane * 4 < (span[i] & ~3))
            *reinterpret_cast<u32x4_t*>(dst[i] + e0 + u * 256 + lane * 4) = buf[i][u];
    }
#pragma unroll
    for (int i = 0; i < IG; ++i)
      if (lane < (span[i] & 3)) dst[i][(span[i] & ~3) + lane] = tail[i];
  }
}
// Which of them: quads where some part of an image is longer than 256 floats.  Up to there the
// four dword loads in flight need one round trip to memory too, and every lane of them carries something (64 images of
// 13 x 13, 384 channels: input transform 12.2 us against 12.6, output gradient transform 14.5 against 15.8; 32 of
// 15 x 15, 256 channels: 7.4 against 7.9; 64 of 7 x 28, 512 channels: 16.3 against 16.8 and 18.2 against 20.1).  Beyond it
// they go to memory in rounds, six in a row for the 26 rows of 56 pixels that a block touches: 32 images of 56 x 56,
// 256 channels: 75 -> 63 us and 69 -> 60 us with quads (5.3 and 5.5 TB/s); 11 of 29 x 23, 131 channels: 10.3 -> 9.8 us.
// The longest part decides, not an average: blocks of F(2x2,5x5) on 27 x 27 reach into a second image now and then, and
// lose 1 us of 14 with dwords.
// (The output gradient transform has a band, 18 to 28 MB of dL/dO, where dwords stay up to 12 % ahead - 62 images of
// 28 x 28, 128 channels: 14.9 against 15.9 us - between sizes where quads are: 5 % at 6, 35 and 50 MB, 8 % at 75 and 100.)
// <2, 4> for blocks of at most two images, <4, 2> for the others: 32 registers either way.
// DWORD_IMAGES: images in flight on the dword path; the output gradient's 13 x 13 planes go faster one by one.
template <int DWORD_IMAGES, typename Part>
__device__ __forceinline__ void stage_parts(const BlockImage* bi, int slots, int longest, float* my, int lane, Part part) {
  if (longest <= 256)
    stage_dwords<DWORD_IMAGES, 4>(bi, slots, my, lane, part);
  else if (slots <= 2)
    stage_quads<2, 4>(bi, slots, my, lane, part);
  else
    stage_quads<4, 2>(bi, slots, my, lane, part);
}

// ---------------------------------------------------------------------------------------------
// Step 1: gather phi + V = B^T d B.  A wave owns one channel and 64 consecutive tiles: it copies
// the input rows those tiles touch into its private LDS area with lane-contiguous (coalesced)
// loads (stage_parts) - each pixel is read from memory once although up to (t/m)^2 tiles use it -
// then every lane gathers its
// t x t tile from LDS (clamped addresses, all reads issued back to back, then selects zero what
// lies outside the image), transforms it in registers and stores one value per position:
// 64 lanes -> 256 contiguous bytes of V[p][c][.], addressed as wave-uniform row + lane.
// Block = 4 waves = 4 channels of the same tile block.
template <int M, int R>
__global__ __launch_bounds__(256) void input_transform_kernel(const float* __restrict__ in, float* __restrict__ V,
                                                              const TileInfo* __restrict__ tiles,
                                                              const BlockImage* __restrict__ blocks,
                                                              const Geometry g) {
  constexpr int t = Wino<M, R>::t;
  extern __shared__ float stage[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = blockIdx.y * 4 + wave;
  const int tau0 = blockIdx.x * 64;
  float* my = stage + wave * g.in_area;
  const BlockImage* bi = blocks + (size_t)blockIdx.x * g.slots;
  const size_t plane = (size_t)g.H * g.W;
  const TileInfo ti = tiles[tau0 + lane];  // asked for first: it arrives while the rows are staged
  if (c < g.C) {
    auto part = [&](const BlockImage& b) {
      return StagedPart{in + (size_t)max(b.n, 0) * g.in_image_stride + c * plane + b.in_elem0, b.in_span, b.in_off};
    };
    stage_parts<4>(bi, g.slots, g.in_longest, my, lane, part);
  }
  __syncthreads();
  if (c >= g.C) return;
  float d[t][t];
  {
    const int y0 = (int16_t)(ti.yx0 & 0xffff), x0 = ti.yx0 >> 16;
    const int y_lo = ti.ylim & 0xffff, y_last = ti.ylim >> 16;
    const float* img = my + ti.in_org;
    int xo[t];
    bool xok[t];
#pragma unroll
    for (int j = 0; j < t; ++j) {
      const int x = x0 + j;
      xok[j] = x >= 0 && x < g.W;
      xo[j] = min(max(x, 0), g.W - 1);
    }
#pragma unroll
    for (int i = 0; i < t; ++i) {
      const float* row = img + min(max(y0 + i, y_lo), y_last) * g.W;  // a staged row in any case
#pragma unroll
      for (int j = 0; j < t; ++j) d[i][j] = row[xo[j]];
    }
    // all t*t reads are issued above; pinning the values here keeps the compiler from turning
    // the selects below into one guarded (and serialised) read each
#pragma unroll
    for (int i = 0; i < t; ++i) {
      if constexpr (t == 8)
        asm volatile("" : "+v"(d[i][0]), "+v"(d[i][1]), "+v"(d[i][2]), "+v"(d[i][3]), "+v"(d[i][4]), "+v"(d[i][5]),
                          "+v"(d[i][6]), "+v"(d[i][7]));
      else if constexpr (t == 6)
        asm volatile("" : "+v"(d[i][0]), "+v"(d[i][1]), "+v"(d[i][2]), "+v"(d[i][3]), "+v"(d[i][4]), "+v"(d[i][5]));
      else
        asm volatile("" : "+v"(d[i][0]), "+v"(d[i][1]), "+v"(d[i][2]), "+v"(d[i][3]));
    }
#pragma unroll
    for (int i = 0; i < t; ++i) {
      const int y = y0 + i;
      const bool yok = y >= 0 && y < g.H;
#pragma unroll
      for (int j = 0; j < t; ++j) d[i][j] = (yok && xok[j]) ? d[i][j] : 0.0f;
    }
  }
  float v[t][t];
  input_transform<M, R>(d, v);
  const __amdgpu_buffer_rsrc_t vr = make_rsrc(V, g.v_bytes);
  const uint32_t row0 = ((uint32_t)c * g.Tp + tau0) * 4u;        // wave-uniform byte offset, position 0
  const uint32_t pstride = (uint32_t)g.C * (uint32_t)g.Tp * 4u;  // bytes between positions
  uint32_t soff = row0;  // one scalar add per store
#pragma unroll
  for (int i = 0; i < t; ++i)
#pragma unroll
    for (int j = 0; j < t; ++j) {
      buffer_store_f32<SWCONV_AUX_V>(vr, lane * 4u, soff, v[i][j]);
      soff += pstride;
      asm volatile("" : "+s"(soff));
    }
}

// ---------------------------------------------------------------------------------------------
// Step 2: M[p] = W_F[p] * V[p] on the plain fp32 ALUs.
//
// Persistent workgroups: the host cuts the sequence of all (position, tile block, slice) units
// into one contiguous, equal-cost range per workgroup; range r is run by the workgroup whose id
// maps to r under xcd_contiguous_id, so neighbouring ranges - which share panels and weights -
// share an XCD's L2.  A range is a short list of work items (runs of slices of one panel).  For an
// item the workgroup stages the C x 64 panel V[p][:, tau_block] in LDS, then the waves draw the
// item's slices from a shared counter, longest first.
//
// Lanes <-> tiles (Section 5: vectorise over tiles), four tiles per lane and four rows per wave:
// a slice has four rows and each quarter of a wave (16 lanes) works on one of them.  Lane (q, s)
// owns row q and the tiles 4s .. 4s+3 of the 64-tile block, so one 16-byte LDS read per lane
// feeds four FMAs, and one LDS address serves four non-zeros x 64 tiles.  LDS delivers such a read per 4.1 clocks
// per CU, whether the quarters read one row or four different ones: 16.3 clocks of a SIMD, the longest part of a step.
// The (row offset, weight) pairs differ between the quarters, so they travel through vector
// memory, 16 steps per load: lane (q, s) fetches the pair of row q, step 16 b + s, and the matrix unit broadcasts
// the pairs of four steps at a time to all lanes of the quarters (swconv_mfma_units.inc).
//
// Stream layout: per slice, batches of 512 bytes; batch b holds [q][s] -> (offset, weight) of row
// q, step 16 b + s; rows shorter than the slice are padded with (0, +0.0f).  A slice's length is
// a multiple of kStepGroup steps.  Panel rows are 64 tiles = 256 bytes.

template <int I>
__device__ __forceinline__ uint32_t quarter_bcast(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + I, 0xf, 0xf, true);  // row_newbcast:I
}

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4v_t __attribute__((ext_vector_type(4)));

// The four accumulators of a lane (its four tiles); separate scalars, so that the inline-asm FMAs
// update them in place.
struct Acc4 {
  float a0, a1, a2, a3;
};

// acc += w * x with w taken from lane I of the lane's quarter.  The broadcast rides on the FMAs
// themselves (DPP operand); the compiler would spend a separate move on it.  `bw` is only ever
// written by a memory load, and FIRST puts two wait states in front, so the rule "two wait states
// between a vector-ALU write of a register and a DPP read of it" holds whatever precedes the group.
template <int I, bool FIRST>
__device__ __forceinline__ void quarter_fma(Acc4& acc, uint32_t bw, const f32x4_t& x) {
#define SWCONV_QFMA(N)                                                                         \
  "v_fmac_f32_dpp %0, %4, %5 row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n"                 \
  "v_fmac_f32_dpp %1, %4, %6 row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n"                 \
  "v_fmac_f32_dpp %2, %4, %7 row_newbcast:" #N " row_mask:0xf bank_mask:0xf\n"                 \
  "v_fmac_f32_dpp %3, %4, %8 row_newbcast:" #N " row_mask:0xf bank_mask:0xf"
#define SWCONV_QFMA_CASE(N)                                                                    \
  if constexpr (I == N) {                                                                      \
    if constexpr (FIRST)                                                                       \
      asm("s_nop 1\n" SWCONV_QFMA(N)                                                           \
          : "+v"(acc.a0), "+v"(acc.a1), "+v"(acc.a2), "+v"(acc.a3)                             \
          : "v"(bw), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));                              \
    else                                                                                       \
      asm(SWCONV_QFMA(N)                                                                       \
          : "+v"(acc.a0), "+v"(acc.a1), "+v"(acc.a2), "+v"(acc.a3)                             \
          : "v"(bw), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));                              \
  }
  SWCONV_QFMA_CASE(0) SWCONV_QFMA_CASE(1) SWCONV_QFMA_CASE(2) SWCONV_QFMA_CASE(3)
  SWCONV_QFMA_CASE(4) SWCONV_QFMA_CASE(5) SWCONV_QFMA_CASE(6) SWCONV_QFMA_CASE(7)
  SWCONV_QFMA_CASE(8) SWCONV_QFMA_CASE(9) SWCONV_QFMA_CASE(10) SWCONV_QFMA_CASE(11)
  SWCONV_QFMA_CASE(12) SWCONV_QFMA_CASE(13) SWCONV_QFMA_CASE(14) SWCONV_QFMA_CASE(15)
#undef SWCONV_QFMA_CASE
#undef SWCONV_QFMA
}

// Four steps' reads.
struct Group4 {
  f32x4_t x0, x1, x2, x3;
};

// The rolling unit of the inner loop (see swconv_rolling_unit.inc): the steps of
// two batches as one pipeline with four reads always in flight, in assembly with the sixteen registers
// of those reads fixed: v[112:127], the top of the 128 registers of the fused F(4x4,3x3) kernel, whose
// other registers are full of accumulators, so that it has none for the broadcasts of the matrix unit.
constexpr int kUnitSteps = 2 * kBatchSteps;
#define SWCONV_UNIT_NAME unit_rolling_hi
#define SWCONV_XR0 112
#define SWCONV_XR1 113
#define SWCONV_XR2 114
#define SWCONV_XR3 115
#define SWCONV_XR4 116
#define SWCONV_XR5 117
#define SWCONV_XR6 118
#define SWCONV_XR7 119
#define SWCONV_XR8 120
#define SWCONV_XR9 121
#define SWCONV_XR10 122
#define SWCONV_XR11 123
#define SWCONV_XR12 124
#define SWCONV_XR13 125
#define SWCONV_XR14 126
#define SWCONV_XR15 127
#include "swconv_rolling_unit.inc"
#undef SWCONV_UNIT_NAME
#undef SWCONV_XR0
#undef SWCONV_XR1
#undef SWCONV_XR2
#undef SWCONV_XR3
#undef SWCONV_XR4
#undef SWCONV_XR5
#undef SWCONV_XR6
#undef SWCONV_XR7
#undef SWCONV_XR8
#undef SWCONV_XR9
#undef SWCONV_XR10
#undef SWCONV_XR11
#undef SWCONV_XR12
#undef SWCONV_XR13
#undef SWCONV_XR14
#undef SWCONV_XR15
#include "swconv_mfma_units.inc"

// ---- dot products (backward pass, Eq. 5 second line): dL/dW_F at the stored entries ----
// The same walk over a packed operand, but every stored entry (row, column) gets the dot product of a
// tensor's row with the panel row of the column over the 64 tiles of the block: the lane multiplies its
// four tiles, the 16 lanes of the quarter are summed with DPP exchanges, and lane i of the quarter ends
// up with the sum of step i, so that after a batch every lane holds the partial sum of "its" stream
// entry and the wave stores 256 contiguous bytes.

// x + (the value of `send` in the lane given by the DPP control): one v_add_f32 with a DPP operand.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x, float send) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), CTRL, 0xf, 0xf, true));
}

// a <- in the lanes of the banks (groups of four lanes of a row of 16) of LO: a + a of the lane given by
// CTRL_LO; in the others: b + b of the lane given by CTRL_HI.  The bank masks of the two instructions do the
// selecting.  Two wait states lie between the vector-ALU write of a register and its read through DPP.
// The sums are written before the b are read: they must not share registers, not even where the compiler knows both
// to hold the same value (the zeros of steps that are not run), hence the early clobbers.
#define SWCONV_FOLD(LO_CTRL, LO, HI_CTRL, HI)                                  \
  asm("s_nop 1\n"                                                              \
      "v_add_f32_dpp %0, %0, %0 " LO_CTRL " row_mask:0xf bank_mask:" LO "\n"    \
      "v_add_f32_dpp %1, %1, %1 " LO_CTRL " row_mask:0xf bank_mask:" LO "\n"    \
      "v_add_f32_dpp %2, %2, %2 " LO_CTRL " row_mask:0xf bank_mask:" LO "\n"    \
      "v_add_f32_dpp %3, %3, %3 " LO_CTRL " row_mask:0xf bank_mask:" LO "\n"    \
      "v_add_f32_dpp %0, %4, %4 " HI_CTRL " row_mask:0xf bank_mask:" HI "\n"    \
      "v_add_f32_dpp %1, %5, %5 " HI_CTRL " row_mask:0xf bank_mask:" HI "\n"    \
      "v_add_f32_dpp %2, %6, %6 " HI_CTRL " row_mask:0xf bank_mask:" HI "\n"    \
      "v_add_f32_dpp %3, %7, %7 " HI_CTRL " row_mask:0xf bank_mask:" HI           \
      : "+&v"(a0), "+&v"(a1), "+&v"(a2), "+&v"(a3)                             \
      : "v"(b0), "v"(b1), "v"(b2), "v"(b3))
__device__ __forceinline__ void fold_bit3(float& a0, float& a1, float& a2, float& a3, float b0, float b1, float b2, float b3) {
  SWCONV_FOLD("row_ror:8", "0x3", "row_ror:8", "0xc");  // partner lane ^ 8
}
__device__ __forceinline__ void fold_bit2(float& a0, float& a1, float& a2, float& a3, float b0, float b1, float b2, float b3) {
  SWCONV_FOLD("row_shl:4", "0x5", "row_shr:4", "0xa");  // partner lane ^ 4
}
#undef SWCONV_FOLD

// The first `steps` steps of one batch; returns, in lane (q, i), the partial sum of row q, step i
// (0 for steps that were not run).  Every lane first collects its share of all 16 steps; the 16
// lanes of a quarter then add them up in a transposing butterfly: in the stage with partner
// lane ^ 8 (then ^ 4, ^ 2, ^ 1) a lane keeps the half of its values whose step has the lane's own
// bit 3 (2, 1, 0) and adds the partner's values for that half, so 8 + 4 + 2 + 1 sums leave the total
// of step i in lane i: 33 instructions, as the bank masks of DPP select for free in the first two
// stages, against 45 with selects in all four and 80 for a reduction step by step.
__device__ __forceinline__ float product_dots_batch(const f32x4_t& lane_base4, float one, const u32x2_t& b, int steps,
                                                    const f32x4_t& z, int lane_in_quarter, Acc4& acc) {
  float d[kBatchSteps];
  unit_dots(lane_base4, one, b, min(steps, kBatchSteps), z, d, acc);
  fold_bit3(d[0], d[1], d[2], d[3], d[8], d[9], d[10], d[11]);
  fold_bit3(d[4], d[5], d[6], d[7], d[12], d[13], d[14], d[15]);
  fold_bit2(d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7]);
  const bool b1 = lane_in_quarter & 2, b0 = lane_in_quarter & 1;
  float g[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) g[i] = dpp_add<0x4E>(b1 ? d[i + 2] : d[i], b1 ? d[i] : d[i + 2]);  // quad_perm [2,3,0,1]: lane ^ 2
  return dpp_add<0xB1>(b0 ? g[1] : g[0], b0 ? g[0] : g[1]);                                       // quad_perm [1,0,3,2]: lane ^ 1
}

// One pass over a packed operand A with panels of V: Mbuf[p] = A[p] * V[p] (forward step 2; on the packed
// transpose the backward pass's dL/dI_F, Eq. 6 first line).
// With DOTS, on the transpose, the same pass makes dL/dW_F (Eq. 5 second line) too:
// partial[tau_block][stream entry] = the entry's dot product of its row of `zrows` (I_F) with its column's row
// of V (dL/dZ) over that tile block; `partial_stride` entries per block.  An entry's dot product does not
// depend on which of the two tensors is the panel, so dL/dZ, the weights and every LDS value are read once for
// both gradients.
//
// EARLY (16 waves, one workgroup per CU): the next item's panel is asked for while this one is worked on, kGroupPieces
// of a thread's pieces in front of each of the wave's first slices, since nothing else on the CU covers its way from
// memory.  Vector-memory results come back in issue order and the stream batches use the same path; the pieces are few
// at a time and the batches two to four ahead, so that a batch is seldom waited for because of a piece.  Workgroups of
// 12 waves have no registers for that (80 each); two of them share a CU, so one computes while the other loads.
// LONG: slices may have more than kUnitSteps steps.  Then four batches are on their way (two units), else two: a
// slice of a few steps would fetch 2 KB to use the first 512 bytes (11 x 29 x 23, 131 -> 187 channels at 7 %: 9.6
// against 10.3 us).
// What it takes (us, before: DPP broadcasts, panel pieces written to LDS by 4-byte words because the array's declared
// alignment was that of a float, the panel asked for behind an item's last slice, and a draw of a slice 25 instructions
// longer): 64 x 13 x 13, 384 -> 384 at 10 %: 42.1 -> 36; 384 -> 256 at 30 %: 67 -> 57 (38 TFLOP/s); 32 x 13 x 13,
// 256 -> 384: 18.8 -> 16.5; 32 x 56 x 56, 256 -> 256: 142 -> 129, and of 132 there remained 118 without the inner loop (V and M
// go through memory).  Both gradients in one pass: 69 -> 61.5, 222 -> 204 (56 x 56), 30.1 -> 27.
// Tried and not kept: a wave of its own that loads panels straight into one of two LDS buffers, one barrier an item
// (15 waves compute): 16.0 for 16.8 and 9.1 for 9.7 us on the two small layers, 135 for 132 and 220 for 205 on the
// 56 x 56 one; drawing a slice under the unit in front instead of before it: 17.2 for 16.6.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds_at(uint32_t byte) {
  return (__attribute__((address_space(3))) T*)(uintptr_t)byte;
}

template <int NWAVES, int PIECES, bool DOTS, bool LONG>
__global__ __launch_bounds__(NWAVES * 64, NWAVES == 12 ? 6 : 4) void spmm_kernel(
    const float* __restrict__ V, float* __restrict__ Mbuf, const uint32_t* __restrict__ stream, uint32_t stream_bytes,
    const Slice* __restrict__ slices, int n_slices, const WorkItem* __restrict__ items,
    const RangeHeader* __restrict__ ranges, int n_wgs, int C, int K, int Tp, uint32_t m_bytes,
    const float* __restrict__ zrows, float* __restrict__ partial, uint32_t partial_stride) {
  constexpr int NT = NWAVES * 64;
  constexpr int TB = kTileBlock;
  constexpr bool EARLY = NWAVES == 16;
  constexpr int kBatchRegs = !DOTS && LONG ? 4 : 2;
  typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
  // LDS: the slice counter (64 bytes; at offset 0, where the appending draw can address it), the panel [C][64], then the
  // descriptors of the item's slices
  extern __shared__ __attribute__((aligned(16))) float panel[];
  // byte addresses in LDS (opaque: the array's address as a symbol costs an addition per access)
  uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)panel;
  asm volatile("" : "+s"(lds0));
  const uint32_t panel0 = lds0 + 64u, desc0 = panel0 + (uint32_t)C * (TB * 4u);
  int drawn_before = -NWAVES;  // draws of the items before, less the first slices, which are not drawn
  // the thread's index, opaque: what is formed from it is formed where it is used instead of held in registers that the
  // inner loop needs
  auto thread_index = [&]() -> uint32_t {
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  };
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RangeHeader hdr = ranges[xcd_contiguous_id(blockIdx.x, n_wgs)];
  const int quarter = lane >> 4;
  const uint32_t lane_sub = (uint32_t)(lane & 15) * 16u;  // byte offset of the lane's four tiles in a row
  const __amdgpu_buffer_rsrc_t mr = make_rsrc(Mbuf, m_bytes), zr = make_rsrc(zrows, m_bytes);
  const __amdgpu_buffer_rsrc_t sr = make_rsrc(stream, stream_bytes);
  const __amdgpu_buffer_rsrc_t dr = make_rsrc(slices, (uint32_t)n_slices * (uint32_t)sizeof(Slice));
  const uint32_t lane8 = (uint32_t)lane * 8u;

  // Panel staging: thread i moves the 16-byte pieces i, i + NT, ... of a panel, through registers.  The descriptors
  // of the item's slices (32 bytes each, at most kMaxItemSlices) are staged the same way, one 16-byte piece per
  // thread: drawing a slice then costs an LDS atomic and an LDS read, and no scalar-memory load -
  // which shares its counter with the LDS reads of the inner loop - is in flight while it runs.
  constexpr int rows_per_piece = NT / (TB / 4);
  const uint32_t piece_stride = (uint32_t)rows_per_piece * (uint32_t)Tp * 4u;
  // the panel's rows as a buffer of their own: what reaches past the last one reads 0 and touches no memory
  auto panel_rsrc = [&](const WorkItem& w) {
    const uint32_t at = (uint32_t)w.p * ((uint32_t)C * (uint32_t)Tp) + (uint32_t)w.tau_block * TB;  // of less than 2^30 floats
    return make_rsrc(V + at, ((uint32_t)(C - 1) * (uint32_t)Tp + TB) * 4u);
  };
  u32x4_t piece[PIECES], desc_piece;
  auto load_batch = [&](uint32_t byte_off) -> u32x2_t {
    return __builtin_amdgcn_raw_buffer_load_b64(sr, (int)lane8, (int)byte_off, 0);  // past the end: reads 0
  };

  // A slice as the loop holds it: stream position and length in scalar registers, the output
  // channel of the lane's quarter in a vector register (-1 = padding row).
  struct Cur {
    uint32_t base;  // byte offset of the slice's first batch
    int len;        // steps
    int k;          // per lane
  };
  // The wave's first slice of an item, from the descriptors in memory (clamped: unconditional, in bounds).  Its four
  // channels are taken from scalar registers at once: left to itself the compiler loads each in a branch of its quarter,
  // three latencies one after the other in front of every item's barrier (forward passes of 32 x 13 x 13, 256 -> 384:
  // 29.4 -> 28.1 us; 64 x 13 x 13, 384 -> 384: 73.2 -> 71.5).
  auto first_index = [&](int slice_begin) { return min(slice_begin + wave, n_slices - 1); };
  auto take_slice = [&](const Slice& sl) -> Cur {
    int k0 = sl.k[0], k1 = sl.k[1], k2 = sl.k[2], k3 = sl.k[3];
    asm volatile("" : "+s"(k0), "+s"(k1), "+s"(k2), "+s"(k3));
    const uint32_t q = (thread_index() >> 4) & 3u;
    return Cur{sl.batch0 * 512u, sl.len, q == 0 ? k0 : q == 1 ? k1 : q == 2 ? k2 : k3};
  };
  auto row_offset = [&](int p, int tau0, int k) -> uint32_t {  // quarters of padding rows are parked beyond the buffer
    return k >= 0 ? (((uint32_t)p * K + (uint32_t)k) * Tp + tau0) * 4u + (thread_index() & 15u) * 16u : 0xfffffff0u;
  };
  auto load_z = [&](int p, int tau0, int k) -> f32x4_t {
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(zr, (int)row_offset(p, tau0, k), 0, 0));
  };
  // Group g of an item's requests: the descriptors with the first, kGroupPieces panel pieces each.
  constexpr int kGroups = (PIECES + kGroupPieces - 1) / kGroupPieces;
  auto request_group = [&](int g, const WorkItem& w, __amdgpu_buffer_rsrc_t vr) {
    const uint32_t tid = thread_index();
    const uint32_t voff0 = ((tid / (TB / 4)) * (uint32_t)Tp + (tid % (TB / 4)) * 4u) * 4u;
    if (g == 0)
      desc_piece = __builtin_amdgcn_raw_buffer_load_b128(
          dr, (int)((int)tid < 2 * (w.slice_end - w.slice_begin) ? tid * 16u : 0xfffffff0u),
          (int)((uint32_t)w.slice_begin * (uint32_t)sizeof(Slice)), 0);
#pragma unroll
    for (int u = g * kGroupPieces; u < (g + 1) * kGroupPieces; ++u)
      if (u < PIECES)
        piece[u] = __builtin_amdgcn_raw_buffer_load_b128(vr, (int)voff0, (int)((uint32_t)u * piece_stride), 0);
  };

  // Start of the first item: the panel pieces and the descriptor piece, then the wave's first slice descriptor and
  // its first two batches, which arrive right behind the panel.
  WorkItem it = hdr.first;
  Cur cur;
  {
    const __amdgpu_buffer_rsrc_t first_panel = panel_rsrc(it);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) request_group(g, it, first_panel);
  }
  cur.k = (int)__builtin_amdgcn_raw_buffer_load_b32(dr, quarter * 4 + 16, first_index(it.slice_begin) * (int)sizeof(Slice), 0);
  // the scalar loads depend on the header only: one latency in front of the first batches and the first barrier
  WorkItem it_next = items[min(hdr.item_begin + 1, hdr.item_end - 1)];
  WorkItem it_after = items[min(hdr.item_begin + 2, hdr.item_end - 1)];
  Slice next_slice = slices[first_index(hdr.second_slice)];
  cur.base = slices[first_index(it.slice_begin)].batch0 * 512u;
  cur.len = slices[first_index(it.slice_begin)].len;
  asm volatile(""
               : "+s"(cur.base), "+s"(cur.len), "+s"(it_next.slice_begin), "+s"(it_after.slice_begin), "+s"(next_slice.batch0));
  u32x2_t b0 = load_batch(cur.base), b1 = load_batch(cur.base + 512u);
  u32x2_t b2 = {0u, 0u}, b3 = {0u, 0u};
  if constexpr (kBatchRegs == 4) b2 = load_batch(cur.base + 1024u), b3 = load_batch(cur.base + 1536u);
  f32x4_t lane_base4;
  lane_base4[0] = lane_base4[1] = lane_base4[2] = lane_base4[3] = __uint_as_float(panel0 + lane_sub);
  float one = 1.0f;
  asm volatile("" : "+v"(lane_base4), "+v"(one));
  // dot products: the lane's four tiles of the row of its quarter (zeros for a padding row)
  f32x4_t z_cur = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (DOTS) z_cur = load_z(it.p, it.tau_block * TB, cur.k);

  // The panel and the descriptors go to LDS.
  auto stage_item = [&](int n_item_slices) {
    const uint32_t tid = thread_index(), tid16 = tid * 16u;
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
      if ((int)tid < C * (TB / 4) - u * NT) *lds_at<u32x4_t>(panel0 + tid16 + (uint32_t)u * (NT * 16u)) = piece[u];
    }
    if ((int)tid < 2 * n_item_slices) *lds_at<u32x4_t>(desc0 + tid16) = desc_piece;
  };
  // The first item's staging stands in front of the loop: a wait in a loop is as strict as its strictest way in, and
  // inside it these writes also waited for the batches behind the pieces, in every first item (the second workgroup of a CU
  // had its panel in LDS 3.0 us after the launch began instead of 2.2: 64 x 20 x 20, 24 -> 48 channels).
  stage_item(it.slice_end - it.slice_begin);
  // (used behind their conditional writes too, the pieces are asked for in front of them and not inside)
#pragma unroll
  for (int u = 0; u < PIECES; ++u) asm volatile("" ::"v"(piece[u]));
  asm volatile("" ::"v"(desc_piece));
  if (thread_index() == 0) *lds_at<int>(lds0) = 0;
  Cur next_first = take_slice(next_slice);
  __syncthreads();

  for (int item = hdr.item_begin;; ++item) {
    const int tau0 = it.tau_block * TB;
    const int n_item_slices = it.slice_end - it.slice_begin;
    // dot products: this tile block's row of the partial-sum buffer, one float per stream entry
    const __amdgpu_buffer_rsrc_t pr =
        make_rsrc(DOTS ? partial + (size_t)it.tau_block * partial_stride : nullptr, DOTS ? partial_stride * 4u : 0u);
    const bool has_next = item + 1 < hdr.item_end;
    if (!has_next) next_first.base = 0xfffff000u;

    // Waves take slices dynamically, longest first: the first one by wave number, every further
    // one from a counter in LDS.  The next slice is drawn before the current one is computed.
    // Returns whether another one was drawn.
    auto run_slice = [&]() -> bool {
      const int drawn = __builtin_amdgcn_ds_append(lds_at<int>(lds0));  // adds 64, one per lane
      Acc4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
      Cur nxt;
      bool more;
      auto take_drawn = [&]() {
        const int i_next = (__builtin_amdgcn_readfirstlane(drawn) >> 6) - drawn_before;
        more = i_next < n_item_slices;
        const uint32_t d = desc0 + 32u * (uint32_t)min(i_next, n_item_slices - 1);  // clamped: stays inside the staged part
        const u32x2_t d_head = *lds_at<u32x2_t>(d);  // all lanes read the same 8 bytes
        const int d_k = *lds_at<int>(d + 16u + (uint32_t)quarter * 4u);
        nxt.base = more ? (uint32_t)__builtin_amdgcn_readfirstlane((int)d_head.x) * 512u : next_first.base;
        nxt.len = more ? __builtin_amdgcn_readfirstlane((int)d_head.y) : next_first.len;
        nxt.k = more ? d_k : next_first.k;
      };
      const int len = cur.len;
      // Batch registers in turn: a register is refilled right after its batch is consumed, unconditionally, with the
      // batch kBatchRegs ahead - or, when the slice has no such batch, with the batch of the same register of the NEXT
      // slice: the one drawn, or the wave's first of the next item (parked past the end of the stream when there is
      // none: reads 0, touches no memory).
      auto refill = [&](int j) -> u32x2_t {
        return load_batch(LONG && j * kBatchSteps < len ? cur.base + (uint32_t)j * 512u
                                                        : nxt.base + (uint32_t)(j & (kBatchRegs - 1)) * 512u);
      };
      // The first batches stand in front of the loop: what the wave has requested between them and their use
      // (panel pieces, a row store) then need not arrive first - a wait in a loop is as strict as its strictest way in.
      f32x4_t z_next = {0.0f, 0.0f, 0.0f, 0.0f};
      if constexpr (DOTS) {
        take_drawn();
        z_next = more ? load_z(it.p, tau0, nxt.k) : load_z(it_next.p, it_next.tau_block * TB, nxt.k);
        auto consume = [&](const u32x2_t& b, int j) {
          const float r = product_dots_batch(lane_base4, one, b, len - j * kBatchSteps, z_cur, lane & 15, acc);
          buffer_store_f32<SWCONV_AUX_M>(pr, lane * 4u, cur.base / 2u + (uint32_t)j * 256u, r);
        };
        if (len > 0) consume(b0, 0);
        b0 = refill(2);
        if (len > kBatchSteps) consume(b1, 1);
        b1 = refill(3);
        for (int j = 2; j * kBatchSteps < len; j += 2) {
          consume(b0, j);
          b0 = refill(j + 2);
          if ((j + 1) * kBatchSteps < len) consume(b1, j + 1);
          b1 = refill(j + 3);
        }
      } else {
        auto consume = [&](const u32x2_t& x, const u32x2_t& y, int j) {
          unit_mfma(lane_base4, one, x, y, min(len - j * kBatchSteps, kUnitSteps), acc);
        };
        take_drawn();
        if (len > 0) consume(b0, b1, 0);
        b0 = refill(kBatchRegs);
        b1 = refill(kBatchRegs + 1);
        if constexpr (LONG) {
          if (len > kUnitSteps) consume(b2, b3, 2);
          b2 = refill(6);
          b3 = refill(7);
          for (int j = 4; j * kBatchSteps < len; j += 4) {
            consume(b0, b1, j);
            b0 = refill(j + 4);
            b1 = refill(j + 5);
            if ((j + 2) * kBatchSteps < len) consume(b2, b3, j + 2);
            b2 = refill(j + 6);
            b3 = refill(j + 7);
          }
        }
      }
      const u32x4v_t result = {__float_as_uint(acc.a0), __float_as_uint(acc.a1), __float_as_uint(acc.a2),
                               __float_as_uint(acc.a3)};
      __builtin_amdgcn_raw_buffer_store_b128(result, mr, (int)row_offset(it.p, tau0, cur.k), 0, SWCONV_AUX_M);
      cur = nxt;
      z_cur = z_next;
      return more;
    };
    auto skip_item = [&]() {  // nothing to do here: on to the next item's first slice
      cur = next_first;
      b0 = load_batch(cur.base);
      b1 = load_batch(cur.base + 512u);
      if constexpr (kBatchRegs == 4) b2 = load_batch(cur.base + 1024u), b3 = load_batch(cur.base + 1536u);
      if constexpr (DOTS) z_cur = load_z(it_next.p, it_next.tau_block * TB, cur.k);
    };
    bool more = wave < n_item_slices;
    const __amdgpu_buffer_rsrc_t next_panel = panel_rsrc(it_next);
    if constexpr (EARLY) {
      if (!more) skip_item();
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        if (has_next) request_group(g, it_next, next_panel);
        if (more) more = run_slice();
      }
      while (more) more = run_slice();
    } else if (more) {
      // The item's first batches have arrived: on the way round the loop the youngest request is then the row store of the
      // slice before, and no slice waits for it (the wait in the loop was vmcnt(0) and is vmcnt(1); a write-through store
      // takes 600 clocks).
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      while (run_slice()) {
      }
    } else {
      skip_item();
    }
    if (!has_next) break;
    drawn_before += n_item_slices;  // a slice, a draw
    if constexpr (!EARLY) {
#pragma unroll
      for (int g = 0; g < kGroups; ++g) request_group(g, it_next, next_panel);
    }
    it = it_next;
    it_next = it_after;
    // scalar loads: they arrive while the panel is written
    it_after = items[min(item + 3, hdr.item_end - 1)];
    next_slice = slices[first_index(it_next.slice_begin)];
    __syncthreads();  // every wave is done with the previous panel and descriptors
    stage_item(it.slice_end - it.slice_begin);
    next_first = take_slice(next_slice);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Step 3: Y = A^T z A + scatter psi.  A wave owns one output channel and 64 consecutive tiles:
// each lane reads its t*t values of M (256 contiguous bytes per wave and position), transforms
// them in registers and drops its m x m outputs into the wave's LDS area laid out like the output
// rows; the wave then writes those rows out with lane-contiguous stores (whole image planes when
// the block covers whole images).  Pixels of tiles that belong to a neighbouring block are
// skipped.  Block = 4 waves = 4 output channels of the same tile block.
template <int M, int R>
__global__ __launch_bounds__(256) void output_transform_kernel(const float* __restrict__ Mbuf,
                                                               float* __restrict__ out,
                                                               const TileInfo* __restrict__ tiles,
                                                               const BlockImage* __restrict__ blocks,
                                                               const Geometry g) {
  constexpr int t = Wino<M, R>::t;
  extern __shared__ float stage[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = blockIdx.y * 4 + wave;
  const int tau0 = blockIdx.x * 64;
  if (tau0 >= g.T) return;  // whole block is padding (uniform for the block)
  float* my = stage + wave * g.out_area;
  const TileInfo ti = tiles[tau0 + lane];  // asked for before the t*t loads below, used after them
  if (k < g.K) {
    const __amdgpu_buffer_rsrc_t mr = make_rsrc(Mbuf, g.m_bytes);
    const uint32_t row0 = ((uint32_t)k * g.Tp + tau0) * 4u;        // wave-uniform byte offset, position 0
    const uint32_t pstride = (uint32_t)g.K * (uint32_t)g.Tp * 4u;  // bytes between positions
    float z[t][t];
    uint32_t soff = row0;  // one scalar add per load
#pragma unroll
    for (int i = 0; i < t; ++i)
#pragma unroll
      for (int j = 0; j < t; ++j) {
        z[i][j] = buffer_load_f32(mr, lane * 4u, soff);
        soff += pstride;
        asm volatile("" : "+s"(soff));
      }
    float y[M][M];
    output_transform<M, R>(z, y);
    const int y0 = (int16_t)(ti.yx0 & 0xffff), x0 = ti.yx0 >> 16;
    // rows / columns of the tile inside the output (<= 0 for a padding tile, whose y0 is -32768)
    const int rows = y0 == -32768 ? 0 : g.Ho - (y0 + g.pad), cols = g.Wo - (x0 + g.pad);
    float* px = my + ti.out_org;
#pragma unroll
    for (int a = 0; a < M; ++a)
#pragma unroll
      for (int b = 0; b < M; ++b)
        if (a < rows && b < cols) px[a * g.Wo + b] = y[a][b];
  }
  __syncthreads();
  if (k >= g.K) return;
  const BlockImage* bi = blocks + (size_t)blockIdx.x * g.slots;
  const size_t plane = (size_t)g.Ho * g.Wo;
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
}

}  // namespace swconv
