// First layer of an ImageNet-style network in 16-bit data: 7 x 7 / stride 2 / pad 3 convolution of an NCHW image with at most 3
// channels, channels-last output, optionally with the 3 x 3 / stride 2 / pad 1 max-pool behind it in the same kernel.
//
// The strips of conv_stem7_split_kernel.hpp on numbers as they are: the image in planes [channel][16 rows as a ring][columns], a reduction of
// (channel, window row) units of 8 columns (147 of 192 terms real), weights in registers for good, two conv rows and one barrier a
// step, the next four image rows on their way meanwhile, rows pooled across lanes and steps in registers before they are rounded (the
// maximum of rounded numbers is the rounded maximum).
//
// What bounds it: the vector work around the MFMAs (per row and filter block 4 sums' bias, clamp and maxima): with the pool, 64
// filters at 224x224, batch 32, the vector ALU is busy 72 % of the cycles in which a unit has work, the matrix pipes 24.
// Measured with the pool, 16 x 16 blocks of outputs (conv_stem7_block_kernel.hpp) / this kernel (us): 64 filters at 224x224, batch 32 30.4 / 24.9, 8 10.3 /
// 10.3, 1 7.9 / 4.5; 64 at 64x64, batch 16 7.9 / 4.8; 10 at 96x96, batch 33 7.1 / 6.5.  Few filters leave the rows' addresses and reads to few
// products, 17 to 32 of them 16 to a wavefront: 32 at 224x224, batch 8 6.9 / 8.1, batch 12 8.0 / 10.0 (two strips side by side with all
// filters in each wavefront at batch 8: 9.8; one wavefront a work-group with all of them 9.0).  There the blocks run (stem7_blocks in api.hip).
//
// The output's pixels hold a multiple of four filters (Cop).
#pragma once
#include "conv_split_kernel.hpp"
#include "strip_index.hpp"

namespace cprune {

// POOL 0: the layer alone; 1: with the pool
template <typename T, int MB, int POOL>
__global__ __launch_bounds__(128, MB == 1 ? 5 : 4) void conv_stem7_kernel(StemArgs a) {
  static_assert(sizeof(T) == 2, "16-bit data");
  constexpr int NT = 128, NR = kStem7Rounds;
  constexpr int STEP = POOL ? 14 : 16;          // conv columns, or image column pairs, from strip to strip
  constexpr int PAIRS = 19;                     // column pairs a strip needs: 2 * 15 + 8 columns
  constexpr int PITCH = 21;                     // dwords (column pairs) per staged row
  constexpr int FIRST = POOL ? 11 : 9;          // image rows under the first step
  __shared__ uint32_t sP[3 * 16 * PITCH];

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 15, g4 = lane >> 4;

  int tile;
  {
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int q = G >> 3, rem = G & 7;
    tile = xcd * q + (xcd < rem ? xcd : rem) + local;
  }
  const StripAt strip = strip_at(tile, a.tiles_x, a.tiles_y, a.magic_x, a.magic_y);
  const int n = strip.group, tx = strip.tx, ty = strip.ty;
  const int o0 = ((int)blockIdx.y * 2 + wave) * (MB * 16);
  const int p_end = POOL ? a.Hp : (a.Ho + 1) >> 1;            // steps of the whole map
  const int p0 = ty * a.band, p1 = min(p0 + a.band, p_end);
  const int cx = STEP * tx - (POOL ? 1 : 0) + r;        // the lane's conv column
  const int ix0 = 2 * (cx - r) - 4;                           // image column of staged column 0

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);

  // ---- staging: item = (row, channel, column pair); row iy lives in ring row (iy + 8) & 15 ----
  struct Item { int off, lds, row; bool c0, c1; };            // byte offset in image row 0; dword of ring row 0
  auto item = [&](int idx, int rows) CPRUNE_INLINE -> Item {
    const int rc = idx / PAIRS, pair = idx - rc * PAIRS;
    const int row = rc / 3, c = rc - row * 3;
    const int ix = ix0 + 2 * pair;
    const bool in = row < rows && c < a.C;
    return Item{((n * a.C + c) * a.H * a.W + ix) * 2, c * (16 * PITCH) + pair, row < rows ? row : -1,
                in && (unsigned)ix < (unsigned)a.W, in && (unsigned)(ix + 1) < (unsigned)a.W};
  };
  auto load_item = [&](const Item& it, int iy, uint32_t (&v)[2]) CPRUNE_INLINE {
    const bool in = (unsigned)iy < (unsigned)a.H;
    const unsigned off = (unsigned)(it.off + iy * a.W * 2);
    v[0] = Elem<T>::load(xr, in & it.c0 ? off : kOutOfRange, 0);
    v[1] = Elem<T>::load(xr, in & it.c1 ? off + 2u : kOutOfRange, 0);
  };
  auto store_item = [&](const Item& it, int iy, const uint32_t (&v)[2]) CPRUNE_INLINE {
    if (it.row < 0) return;
    sP[it.lds + ((iy + 8) & 15) * PITCH] = v[0] | v[1] << 16;
  };

  // ---- the first rows, then the weights, on their way together ----
  const int iy_first = 4 * p0 + 6 - FIRST;
  {
    constexpr int U = (FIRST * 3 * PAIRS + NT - 1) / NT;
    Item it[U];
    uint32_t v[U][2];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      it[j] = item(t + NT * j, FIRST);
      load_item(it[j], iy_first + it[j].row, v[j]);
    }
#pragma unroll
    for (int j = 0; j < U; ++j) store_item(it[j], iy_first + it[j].row, v[j]);
  }
  uint4 wt[MB][NR];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NR; ++j)
      wt[i][j] = load_b128(wr, o0 + i * 16 < a.O ? (unsigned)(((o0 >> 4) + i) * NR + j) * 1024u + (unsigned)lane * 16u : kOutOfRange, 0);
  float4_t bias[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) bias[i] = load_bias4(a.bias, a.O, o0 + i * 16 + 4 * g4);

  constexpr int U = (4 * 3 * PAIRS + NT - 1) / NT;            // items of a later step
  Item it[U];
#pragma unroll
  for (int j = 0; j < U; ++j) it[j] = item(t + NT * j, 4);

  // the lane's unit of each round: window row, dword of its channel's plane
  int unit_row[NR], unit_lds[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int q = min(4 * j + g4, 20), c = q / 7;
    unit_row[j] = q - c * 7;
    unit_lds[j] = c * (16 * PITCH) + r;
  }
  // Units past the last, of the last round, are zeros: behind their zero weights a finite number would do, an infinity not.  (As a row of zeros
  // in LDS they cost 2-3 % of a 3.6 us launch, as these selects 1.)
  const bool real = 4 * (NR - 1) + g4 <= 20;

  // conv row cy: sums of the lane's pixel
  auto multiply = [&](int cy, float4_t (&out)[MB]) CPRUNE_INLINE {
#pragma unroll
    for (int i = 0; i < MB; ++i) out[i] = bias[i];
    uint4 x[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) __builtin_memcpy(&x[j], sP + unit_lds[j] + ((2 * cy + 5 + unit_row[j]) & 15) * PITCH, 16);    // (2 cy - 3 + row) + 8
    uint4& q = x[NR - 1];
    q.x = real ? q.x : 0u; q.y = real ? q.y : 0u; q.z = real ? q.z : 0u; q.w = real ? q.w : 0u;
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int i = 0; i < MB; ++i) out[i] = mfma_split<T>(wt[i][j], x[j], out[i]);
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) out[i][q] = apply_act(out[i][q], a.act);
  };
  // the largest of three neighbouring columns, in the lane of the first (an activated value is never NaN)
  const bool col_ok = (unsigned)cx < (unsigned)a.Wo;
  auto across = [&](float4_t (&v)[MB]) CPRUNE_INLINE {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float c0 = col_ok ? v[i][q] : -__builtin_inff();
        auto next = [&](auto d) CPRUNE_INLINE {
          return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, c0), 0x100 + decltype(d)::value, 0xf, 0xf, true));
        };
        v[i][q] = fmaxf(fmaxf(c0, next(std::integral_constant<int, 1>{})), next(std::integral_constant<int, 2>{}));
      }
  };
  auto store = [&](void* map, int y, int x, int w, int h, bool lane_ok, const float4_t (&v)[MB]) CPRUNE_INLINE {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int o = o0 + i * 16 + 4 * g4;
      if (lane_ok & (x < w) & (o < a.Cop)) *(uint2*)((T*)map + ((size_t)(n * h + y) * w + x) * a.Cop + o) = narrow4<T>(v[i]);
    }
  };

  __syncthreads();
  float4_t carry[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) carry[i] = (float4_t){-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
  if (POOL && p0 > 0 && o0 < a.O) {
    multiply(2 * p0 - 1, carry);
  }
  for (int p = p0; p < p1; ++p) {
    const bool more = p + 1 < p1;
    uint32_t v[U][2];
    if (more) {
#pragma unroll
      for (int j = 0; j < U; ++j) load_item(it[j], 4 * p + 6 + it[j].row, v[j]);
    }
    if (o0 < a.O) {
      float4_t top[MB], s[MB];                   // the first row of the step, and the largest of the window's; the second row
      multiply(2 * p, top);
      const bool second = 2 * p + 1 < a.Ho;
      if (second) multiply(2 * p + 1, s);
      if constexpr (POOL != 0) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            top[i][q] = fmaxf(carry[i][q], second ? fmaxf(top[i][q], s[i][q]) : top[i][q]);
            carry[i][q] = s[i][q];
          }
        across(top);
        store(a.y, p, 7 * tx + (r >> 1), a.Wp, a.Hp, ((r & 1) == 0) & (r < 14), top);
      } else {
        store(a.y, 2 * p, cx, a.Wo, a.Ho, true, top);
        if (second) store(a.y, 2 * p + 1, cx, a.Wo, a.Ho, true, s);
      }
    }
    if (more) {
#pragma unroll
      for (int j = 0; j < U; ++j) store_item(it[j], 4 * p + 6 + it[j].row, v[j]);
    }
    __syncthreads();
  }
}

template <typename T>
inline int launch_stem7(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a) {
#define CPRUNE_STEM7(MB_, POOL_)                                                                        \
  if (mb == MB_ && pool == POOL_) {                                                                     \
    hipLaunchKernelGGL((conv_stem7_kernel<T, MB_, POOL_>), grid, dim3(128), 0, s, a);                   \
    return CPRUNE_OK;                                                                                   \
  }
  CPRUNE_STEM7(1, 0) CPRUNE_STEM7(1, 1) CPRUNE_STEM7(2, 0) CPRUNE_STEM7(2, 1)
#undef CPRUNE_STEM7
  return CPRUNE_ERR_UNSUPPORTED;
}

}  // namespace cprune
