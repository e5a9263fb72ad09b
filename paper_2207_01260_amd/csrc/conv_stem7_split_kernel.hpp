// First layer of an ImageNet-style network in fp32: 7 x 7 / stride 2 / pad 3 convolution of an NCHW image with at most 3
// channels on the 16-bit matrix cores, channels-last output, optionally with the 3 x 3 / stride 2 / pad 1 max-pool behind
// it in the same kernel.
//
// Every number is cut into three bf16 parts and six of the nine products are multiplied (conv_split_kernel.hpp has the
// error and the range of that).  What decides the layout is the gather of the windows: the image is cut once, while it is
// staged, into planes [part][channel][16 rows as a ring][columns], and the reduction is a list of (channel, window row)
// units of 8 columns, the first of them a column left of the window that meets a zero weight.  A lane's operand of a unit
// is then 16 consecutive bytes of a plane; 21 units make 6 rounds of 32 terms, 147 of 192 real.  (Four-channel pixels,
// as conv_stem7_block_kernel.hpp has them, take 7.)
//   weights   a wavefront holds those of its MB 16-filter blocks in registers for good: 6 rounds x 3 parts, 144 registers at
//             two blocks.  The two wavefronts of a work-group take the two halves of a filter tile on the same pixels.
//   pixels    a work-group walks down a strip of 16 conv columns, two conv rows a step; four new image rows a step are
//             loaded a step ahead, cut and stored into ring rows that nobody reads meanwhile: one barrier a step.
//   pool      a finished row is reduced over its neighbouring lanes (DPP) and over the step's two rows in registers; the
//             odd row is carried to the next step.  Strips then advance by 14 columns (7 pooled ones), and a band of rows
//             begins with the row above it.  The conv map, the largest tensor of such a network, is written only where it is
//             asked for (a timed handle keeps it readable), each of its pixels by the strip and the band that own it, and
//             never read again.
//
// Measured, 64 filters at 224x224 (us), the first-layer kernel on the fp32 instruction and the pool behind it / this kernel and the pool
// behind it / with the pool and the conv map / with the pool alone: batch 32 120 / 91 / 69 / 60-65, 8 40 / 29 / 25 / 22.5, 1 15.6 / 9.5 / 9.5 /
// 8.6.  The MFMAs of batch 32 take 27 us at full rate (147 of 192 terms and 14 of 16 columns real); two wavefronts per SIMD hide the rest in
// part: cutting, addresses, the sums' look and the pool (counters: matrix pipes busy 52 %, vector ALU 46, LDS 8, waiting 34).  The conv map is 103 MB, 20 us at the copy rate (streaming
// stores: the same time).  Error against 64 bits 7.4e-8, on the fp32 instruction 2.1e-7.
#pragma once
#include "conv_split_kernel.hpp"
#include "strip_index.hpp"

namespace cprune {

// POOL 0: the layer alone; 1: with the pool; 2: with the pool, and the conv map written as well
template <int MB, int POOL>
__global__ __launch_bounds__(128, 2) void conv_stem7_split_kernel(StemArgs a) {
  constexpr int NT = 128, NR = kStem7Rounds;
  constexpr int PAIRS = 19;                     // column pairs a strip needs: 2 * 15 + 8 columns
  constexpr int PITCH = 21;                     // dwords (column pairs) per staged row
  constexpr int PLANE = 3 * 16 * PITCH;         // dwords per part
  constexpr int FIRST = POOL ? 11 : 9;          // image rows under the first step
  __shared__ uint32_t sP[3 * PLANE];

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
  const int cx = POOL ? 14 * tx - 1 + r : 16 * tx + r;        // the lane's conv column
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
    return Item{((n * a.C + c) * a.H * a.W + ix) * 4, c * (16 * PITCH) + pair, row < rows ? row : -1,
                in && (unsigned)ix < (unsigned)a.W, in && (unsigned)(ix + 1) < (unsigned)a.W};
  };
  auto load_item = [&](const Item& it, int iy, uint32_t (&v)[2]) CPRUNE_INLINE {
    const bool in = (unsigned)iy < (unsigned)a.H;
    const unsigned off = (unsigned)(it.off + iy * a.W * 4);
    v[0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xr, (int)(in & it.c0 ? off : kOutOfRange), 0, 0);
    v[1] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(xr, (int)(in & it.c1 ? off + 4u : kOutOfRange), 0, 0);
  };
  auto store_item = [&](const Item& it, int iy, const uint32_t (&v)[2]) CPRUNE_INLINE {
    if (it.row < 0) return;
    uint32_t h, m, l;
    split3(v[0], v[1], h, m, l);
    uint32_t* const d = sP + it.lds + ((iy + 8) & 15) * PITCH;
    d[0] = h; d[PLANE] = m; d[2 * PLANE] = l;
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
  uint4 wt[MB][NR][3];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        wt[i][j][p] = load_b128(wr, o0 + i * 16 < a.O ? (unsigned)((((o0 >> 4) + i) * NR + j) * 3 + p) * 1024u + (unsigned)lane * 16u
                                                      : kOutOfRange, 0);
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
    const int q = min(4 * j + g4, 20), c = q / 7;             // (units past the last meet zero weights)
    unit_row[j] = q - c * 7;
    unit_lds[j] = c * (16 * PITCH) + r;
  }

  // conv row cy: sums of the lane's pixel
  auto multiply = [&](int cy, float4_t (&out)[MB]) CPRUNE_INLINE {
    float4_t big[MB], small[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) big[i] = small[i] = (float4_t){0.f, 0.f, 0.f, 0.f};
    uint4 x[2][3];
    auto fetch = [&](int j, uint4 (&f)[3]) CPRUNE_INLINE {
      const uint32_t* const src = sP + unit_lds[j] + ((2 * cy + 5 + unit_row[j]) & 15) * PITCH;    // (2 cy - 3 + row) + 8
#pragma unroll
      for (int p = 0; p < 3; ++p) __builtin_memcpy(&f[p], src + p * PLANE, 16);
    };
    fetch(0, x[0]);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      if (j + 1 < NR) fetch(j + 1, x[(j + 1) & 1]);
      const uint4 (&b)[3] = x[j & 1];
      auto term = [&](int pw, int px, float4_t (&d)[MB]) CPRUNE_INLINE {
#pragma unroll
        for (int i = 0; i < MB; ++i) d[i] = mfma_split<float>(wt[i][j][pw], b[px], d[i]);
      };
      term(0, 2, small); term(0, 0, big); term(2, 0, small); term(1, 1, small); term(0, 1, small); term(1, 0, small);
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) out[i] = big[i] + small[i];

    // data that three parts do not hold shows in the sums (see conv_split_kernel): then once more on the fp32 instruction
    constexpr uint32_t kInf = 0x7f800000u, kSmall = (127u - 50u) << 23;
    uint32_t odd = 0;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) odd = max(odd, (__float_as_uint(out[i][q]) << 1) - (kSmall << 1));
    if (__any(odd >= (kInf - kSmall) << 1)) {
      uint32_t top = 0, low = ~0u;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t mag = __float_as_uint(out[i][q]) & 0x7fffffffu;
          top = max(top, mag);
          low = min(low, mag - 1);      // (zero goes to the other end)
        }
      if (__any(top >= kInf || low < kSmall - 1)) {
        const __amdgpu_buffer_rsrc_t ww = make_rsrc(a.w_raw, a.w_raw_bytes);
        const int terms = a.C * 49;
#pragma unroll
        for (int i = 0; i < MB; ++i) out[i] = (float4_t){0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < terms; k0 += 4) {
          const int k = k0 + g4, c = k / 49, uv = k - c * 49, u = uv / 7, v = uv - u * 7;
          const int iy = 2 * cy - 3 + u, ix = 2 * cx - 3 + v;
          const bool in = (k < terms) & ((unsigned)iy < (unsigned)a.H) & ((unsigned)ix < (unsigned)a.W);
          const float xv = __uint_as_float(Elem<float>::load(xr, in ? (unsigned)(((n * a.C + c) * a.H + iy) * a.W + ix) * 4u : kOutOfRange, 0));
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            const int o = o0 + i * 16 + r;
            const float wv = __uint_as_float(Elem<float>::load(ww, (k < terms) & (o < a.O) ? (unsigned)(o * terms + k) * 4u : kOutOfRange, 0));
            out[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, xv, out[i], 0, 0, 0);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) out[i][q] = apply_act(out[i][q] + bias[i][q], a.act);
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
      if (lane_ok & (x < w) & (o < a.Cop)) *(float4_t*)((float*)map + ((size_t)(n * h + y) * w + x) * a.Cop + o) = v[i];
    }
  };

  __syncthreads();
  float4_t carry[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) carry[i] = (float4_t){-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
  if (POOL && p0 > 0 && o0 < a.O) {
    multiply(2 * p0 - 1, carry);
    across(carry);
  }
  for (int p = p0; p < p1; ++p) {
    const bool more = p + 1 < p1;
    uint32_t v[U][2];
    if (more) {
#pragma unroll
      for (int j = 0; j < U; ++j) load_item(it[j], 4 * p + 6 + it[j].row, v[j]);
    }
#pragma unroll
    for (int z = 0; z < 2; ++z) {
      const int cy = 2 * p + z;
      if (cy < a.Ho && o0 < a.O) {
        float4_t s[MB];
        multiply(cy, s);
        if constexpr (POOL == 2) store(a.y_map, cy, cx, a.Wo, a.Ho, (r > 0) & (r < 15), s);      // (14 columns are the strip's own)
        if constexpr (POOL != 0) {
          across(s);
          if (z == 0) {
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
              for (int q = 0; q < 4; ++q) carry[i][q] = fmaxf(carry[i][q], s[i][q]);
          } else {
            float4_t m[MB];
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
              for (int q = 0; q < 4; ++q) m[i][q] = fmaxf(carry[i][q], s[i][q]);
            store(a.y, p, 7 * tx + (r >> 1), a.Wp, a.Hp, ((r & 1) == 0) & (r < 14), m);
#pragma unroll
            for (int i = 0; i < MB; ++i) carry[i] = s[i];
          }
        } else {
          store(a.y, cy, cx, a.Wo, a.Ho, true, s);
        }
      } else if (POOL && o0 < a.O) {
        store(a.y, p, 7 * tx + (r >> 1), a.Wp, a.Hp, ((r & 1) == 0) & (r < 14), carry);
      }
    }
    if (more) {
#pragma unroll
      for (int j = 0; j < U; ++j) store_item(it[j], 4 * p + 6 + it[j].row, v[j]);
    }
    __syncthreads();
  }
}

inline int launch_stem7_split(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a) {
#define CPRUNE_STEM7S(MB_, POOL_)                                                                       \
  if (mb == MB_ && pool == POOL_) {                                                                     \
    hipLaunchKernelGGL((conv_stem7_split_kernel<MB_, POOL_>), grid, dim3(128), 0, s, a);                \
    return CPRUNE_OK;                                                                                   \
  }
  CPRUNE_STEM7S(1, 0) CPRUNE_STEM7S(1, 1) CPRUNE_STEM7S(1, 2) CPRUNE_STEM7S(2, 0) CPRUNE_STEM7S(2, 1) CPRUNE_STEM7S(2, 2)
#undef CPRUNE_STEM7S
  return CPRUNE_ERR_UNSUPPORTED;
}

}  // namespace cprune
