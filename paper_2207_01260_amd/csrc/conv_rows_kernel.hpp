// 3x3 / stride 1 / pad 1 convolution of 16-bit data, channels-last, without LDS in the main loop.
//
// At 16x16x32 MFMAs the tiled kernels spend their time on the way of the operands: global memory -> registers -> LDS ->
// registers, with one or two barriers per chunk of channels, for MFMAs that take 16 cycles each.  Here a WAVEFRONT owns a
// strip of 16 columns x R output rows of one image (of two or four images side by side on maps of at most 8 or 4
// columns) and MB blocks of 16 filters, and keeps the operands in registers:
//   activations  an input row of the strip is one 16-byte load per lane and chunk of 32 channels, and as loaded the B operand
//                of 16 pixels x 32 channels for the middle column of the window; the operands of the left and the right column
//                are the same registers shifted by a lane (DPP; the strip's edge columns come with a load of two
//                lanes, or are zero).  Every row is used for the three output rows it touches: 9 x MB MFMAs per load.
//   weights      the nine taps of a chunk, MB blocks each, in registers, read once per chunk in operand order (launch_repack_wave);
//                those of the next chunk are asked for as soon as the last row has used the present ones.  The four
//                wavefronts of a work-group take neighbouring strips of the same filters, so that three of four reads hit
//                the vector cache.
// Rows outside the image are left out, not multiplied.  KS > 1: KS wavefronts share a strip and split its chunks (few strips,
// many channels); their sums meet in LDS at the end, in order.  Optional 2x2 max-pool behind the activation.
//
// Measured, the best other kernel / this one (us): fp16 at batch 64: 209 -> 197 at 8x8 12.2 / 7.8, 360 -> 360 at 4x4 10.1 / 6.6, 56 ->
// 56 at 32x32 with the pool 9.9 / 9.0; bf16 at batch 32: 512 -> 411 at 7x7 19.2 / 10.5, 173 -> 256 at 14x14 13.6 / 10.0, 128 -> 85 at
// 28x28 12.9 / 11.1, 40 -> 64 at 56x56 14.1 / 14.5 (the patch kernel stays there).  What bounds it: some 5 us of launch, first loads
// and stores; alone on its SIMD a wavefront takes 1.3 us per chunk of 2 blocks x 8 rows, 1.0 us of it MFMA issue, the
// rest the wait for the weights of the next chunk, which are asked for 300 clocks before their use (a second set of
// registers for them would leave one wavefront per SIMD).
#pragma once
#include "conv_nhwc_kernel.hpp"

namespace cprune {

struct RowsArgs {
  const void* x;        // [n][h][w][cp]
  const void* w;        // launch_repack_wave
  const float* bias;
  const void* res;
  void* y;              // [n][h][w][cop], pooled: [n][h / 2][w / 2][cop]
  int N, H, W, O, Cp, Cop;
  int tiles_y, tiles_x, tiles_m;   // strips of a map, filter tiles
  int strips;                      // of the whole batch
  int lane_shift;                  // lanes per image: 1 << lane_shift
  unsigned magic_m, magic_x, magic_y;
  unsigned x_bytes, w_bytes, y_bytes;
  int nchunk;                      // chunks of 32 channels
  int act, pool;
};

template <typename T, int MB, int R, int KS, bool HALO>
__global__ __launch_bounds__(KS == 8 ? 512 : 256, 2) void conv_rows_kernel(RowsArgs a) {
  static_assert(sizeof(T) == 2 && R % 2 == 0, "16-bit data, pairs of rows");
  constexpr int NS = KS >= 4 ? 1 : 4 / KS;       // strips of a work-group
  constexpr int ROWS = R + 2;
  constexpr int PF = R == 8 ? 5 : MB <= 2 ? 6 : 3;   // rows asked for ahead
  constexpr int SLOTS = KS > 4 ? 4 : KS;
  static_assert(ROWS % PF == 0, "ring of rows");
  __shared__ __attribute__((aligned(16))) float4_t xch[KS > 1 ? NS * SLOTS * R * MB * 64 : 1];

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int slice = wave % KS, sub = wave / KS;
  const int r = lane & 15, g4 = lane >> 4;

  int tile;
  {
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int q = G >> 3, rem = G & 7;
    tile = xcd * q + (xcd < rem ? xcd : rem) + local;
  }
  const int group = (int)fast_div((unsigned)tile, a.magic_m);      // of NS strips
  const int tile_m = tile - group * a.tiles_m;
  const int o0 = tile_m * (MB * 16);
  const int strip = group * NS + sub;
  const int q_x = (int)fast_div((unsigned)strip, a.magic_x);
  const int tx = strip - q_x * a.tiles_x;
  const int grp = (int)fast_div((unsigned)q_x, a.magic_y);
  const int ty = q_x - grp * a.tiles_y;
  const int lr = r & ((1 << a.lane_shift) - 1);
  const int img = (grp << (4 - a.lane_shift)) + (r >> a.lane_shift);
  const int cx = tx * 16 + lr;
  const int iy0 = ty * R - 1;
  const bool live = strip < a.strips;
  const bool col_ok = live & (img < a.N) & (cx < a.W);

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);
  const int row_bytes = a.W * a.Cp * 2;
  const int x_off = ((img * a.H + iy0) * a.W + cx) * a.Cp * 2 + g4 * 16;
  // HALO: the columns beside the strip, fetched by its edge lanes; otherwise neighbours exist inside an image only
  const int hx = r == 0 ? cx - 1 : cx + 1;
  const bool h_ok = HALO && live && img < a.N && (r == 0 || r == 15) && (unsigned)hx < (unsigned)a.W;
  const int h_off = x_off + (r == 0 ? -a.Cp * 2 : a.Cp * 2);
  const unsigned ml = lr > 0 ? ~0u : 0u, mr = lr < (1 << a.lane_shift) - 1 ? ~0u : 0u;

  uint4 pre[PF], hal[HALO ? PF : 1];
  auto load_row = [&](int c, int i, int slot) {
    const bool in = ((unsigned)(iy0 + i) < (unsigned)a.H) & (c * 32 + g4 * 8 < a.Cp);
    pre[slot] = load_b128(xr, in & col_ok ? (unsigned)(x_off + i * row_bytes) : kOutOfRange, (unsigned)c * 64u);
    if constexpr (HALO) hal[slot] = load_b128(xr, in & h_ok ? (unsigned)(h_off + i * row_bytes) : kOutOfRange, (unsigned)c * 64u);
  };
  uint4 wt[3][3][MB];
  auto load_taps = [&](int c, int u) {
    const unsigned past = c < a.nchunk ? 0u : kOutOfRange;
#pragma unroll
    for (int v = 1; v < 4; ++v)                    // (in the order of their use)
#pragma unroll
      for (int m = 0; m < MB; ++m)
        wt[u][v % 3][m] = load_b128(wr, o0 + m * 16 < a.O ? past | (unsigned)lane * 16u : kOutOfRange,
                                    (unsigned)(((tile_m * MB + m) * a.nchunk + c) * 9 + u * 3 + v % 3) * 1024u);
  };
  // (in the order in which the loop asks for them, so that the waits at its head count the same loads on both ways in)
#pragma unroll
  for (int i = ROWS - PF; i < ROWS; ++i) {
    load_row(slice, i + PF - ROWS, i % PF);
    __builtin_amdgcn_sched_barrier(0);
    if (i >= R - 1) load_taps(slice, i - (R - 1));
    __builtin_amdgcn_sched_barrier(0);
  }

  float4_t acc[R][MB];
#pragma unroll
  for (int y = 0; y < R; ++y)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[y][m] = (float4_t){0.f, 0.f, 0.f, 0.f};

  auto shifted = [&](const uint4& x, const uint4& edge, auto left_tag) -> uint4 {
    constexpr bool left = decltype(left_tag)::value;
    constexpr int ctrl = left ? 0x111 : 0x101;       // row_shr:1 (the lane takes its left neighbour's) / row_shl:1
    auto one = [&](unsigned v, unsigned e) -> unsigned {
      if constexpr (HALO) return (unsigned)__builtin_amdgcn_update_dpp((int)e, (int)v, ctrl, 0xf, 0xf, false);
      else return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true) & (left ? ml : mr);
    };
    return make_uint4(one(x.x, edge.x), one(x.y, edge.y), one(x.z, edge.z), one(x.w, edge.w));
  };

  for (int c = slice; c < a.nchunk; c += KS) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const uint4 x = pre[i % PF], edge = hal[HALO ? i % PF : 0];
      if ((unsigned)(iy0 + i) < (unsigned)a.H) {
        const uint4 b[3] = {shifted(x, edge, std::true_type{}), x, shifted(x, edge, std::false_type{})};
#pragma unroll
        for (int v = 1; v != 4; ++v)               // the middle column first: its operand needs no shift
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            if (i - u < 0 || i - u >= R) continue;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
              if constexpr (std::is_same<T, _Float16>::value)
                acc[i - u][m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, wt[u][v % 3][m]),
                                                                      __builtin_bit_cast(half8_t, b[v % 3]), acc[i - u][m], 0, 0, 0);
              else
                acc[i - u][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wt[u][v % 3][m]),
                                                                       __builtin_bit_cast(bf16x8_t, b[v % 3]), acc[i - u][m], 0, 0, 0);
            }
          }
      }
      if (i + PF < ROWS) load_row(c, i + PF, i % PF);
      else load_row(c + KS, i + PF - ROWS, i % PF);
      if (i >= R - 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (i == R - 1 + u) load_taps(c + KS, u);
    }
  }

  // ---- bias, shortcut, activation, store: four filters of a pixel, or of the maximum of a 2x2 window ----
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res, a.res ? a.y_bytes : 0u);
  const float lo = a.act == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi = a.act == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  auto at = [&](int y, int m) -> unsigned {
    const int oy = ty * R + y, o = o0 + m * 16 + 4 * g4;
    const bool ok = col_ok & (oy < a.H) & (o < a.Cop);
    if (a.pool) return ok & ((cx & 1) == 0) ? (unsigned)(((img * (a.H >> 1) + (oy >> 1)) * (a.W >> 1) + (cx >> 1)) * a.Cop + o) * 2u : kOutOfRange;
    return ok ? (unsigned)(((img * a.H + oy) * a.W + cx) * a.Cop + o) * 2u : kOutOfRange;
  };
  auto widen = [&](uint2 q) -> float4_t {
    const T* h = reinterpret_cast<const T*>(&q);
    return (float4_t){Elem<T>::to_f32(h[0]), Elem<T>::to_f32(h[1]), Elem<T>::to_f32(h[2]), Elem<T>::to_f32(h[3])};
  };
  typedef unsigned int uint32x2_t __attribute__((ext_vector_type(2)));
  auto load_res = [&](unsigned off) -> uint2 {
    const uint32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(rr, (int)off, 0, 0);
    return make_uint2(v.x, v.y);
  };
  auto clamp4 = [&](float4_t v) -> float4_t {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = __builtin_amdgcn_fmed3f(v[q], lo, hi);
    return v;
  };
  auto store = [&](unsigned off, float4_t v) {
    if (off == kOutOfRange) return;
    T h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = Elem<T>::from_f32(v[q]);
    *(uint2*)((char*)a.y + off) = *(const uint2*)h;
  };
  // rows y and y + 1 of the sums -> the window's maximum (the activation is monotone), in its two lanes
  auto window = [&](float4_t s0, float4_t s1) -> float4_t {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float v = fmaxf(s0[q], s1[q]);
      const float w = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));
      s0[q] = fmaxf(v, w);       // 0xB1: lanes 1, 0, 3, 2 of each four
    }
    return s0;
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const float4_t bias = load_bias4(a.bias, a.O, o0 + m * 16 + 4 * g4);
      uint2 res[R];
      if (a.res) {
#pragma unroll
        for (int y = 0; y < R; ++y) res[y] = load_res(at(y, m));
      }
#pragma unroll
      for (int y = 0; y < R; y += 2) {
        if (a.pool) {
          store(at(y, m), window(clamp4(acc[y][m] + bias), clamp4(acc[y + 1][m] + bias)));
        } else {
#pragma unroll
          for (int z = y; z < y + 2; ++z) {
            float4_t v = acc[z][m] + bias;
            if (a.res) v += widen(res[z]);
            store(at(z, m), clamp4(v));
          }
        }
      }
    }
  } else {
    // the upper half of the wavefronts hands over to the lower one until SLOTS are left; their sums are added in order,
    // the units (a pair of rows, a filter block) shared by all wavefronts of the strip
    constexpr int SLOT = R * MB * 64;
    float4_t* const mine = xch + sub * (SLOTS * SLOT) + lane;
    int nw = KS;
#pragma unroll
    for (int level = KS; level > SLOTS; level >>= 1) {
      const int hw = level >> 1;
      if (slice >= hw && slice < level) {
#pragma unroll
        for (int q = 0; q < R * MB; ++q) mine[(slice - hw) * SLOT + q * 64] = acc[q / MB][q % MB];
      }
      __syncthreads();
      if (slice < hw) {
#pragma unroll
        for (int q = 0; q < R * MB; ++q) acc[q / MB][q % MB] += mine[slice * SLOT + q * 64];
      }
      __syncthreads();
      nw = hw;
    }
    if (slice < nw) {
#pragma unroll
      for (int q = 0; q < R * MB; ++q) mine[slice * SLOT + q * 64] = acc[q / MB][q % MB];
    }
    __syncthreads();
    for (int q = slice; q < R / 2 * MB; q += KS) {
      const int y = 2 * (q / MB), m = q % MB;
      const float4_t bias = load_bias4(a.bias, a.O, o0 + m * 16 + 4 * g4);
      uint2 res[2];
      if (a.res) { res[0] = load_res(at(y, m)); res[1] = load_res(at(y + 1, m)); }
      float4_t s[2];
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const float4_t* const src = mine + ((y + z) * MB + m) * 64;
        s[z] = src[0];
#pragma unroll
        for (int w = 1; w < SLOTS; ++w) s[z] += src[w * SLOT];
        s[z] += bias;
        if (a.res) s[z] += widen(res[z]);
        s[z] = clamp4(s[z]);
      }
      if (a.pool) store(at(y, m), window(s[0], s[1]));
      else { store(at(y, m), s[0]); store(at(y + 1, m), s[1]); }
    }
  }
}

// Variants: id, 16-filter blocks, rows of a strip, wavefronts that share a strip
#define CPRUNE_ROWS_LIST(X) \
  X(0, 2, 8, 1) X(1, 2, 8, 2) X(2, 2, 8, 4)                          \
  X(3, 2, 4, 1) X(4, 2, 4, 2) X(5, 2, 4, 4) X(6, 2, 4, 8)            \
  X(7, 3, 4, 1) X(8, 4, 4, 1) X(9, 1, 8, 1)                          \
  X(10, 1, 4, 2) X(11, 1, 4, 4) X(12, 1, 4, 8)

constexpr int kNumRows = 13;

template <typename T>
inline int launch_rows(int id, dim3 grid, hipStream_t s, const RowsArgs& a) {
#define CPRUNE_ROWS_CASE(ID, MB_, R_, KS_)                                                                           \
  case ID:                                                                                                           \
    if (a.tiles_x > 1) hipLaunchKernelGGL((conv_rows_kernel<T, MB_, R_, KS_, true>), grid, dim3(KS_ == 8 ? 512 : 256), 0, s, a); \
    else hipLaunchKernelGGL((conv_rows_kernel<T, MB_, R_, KS_, false>), grid, dim3(KS_ == 8 ? 512 : 256), 0, s, a);  \
    break;
  switch (id) { CPRUNE_ROWS_LIST(CPRUNE_ROWS_CASE) default: return CPRUNE_ERR_UNSUPPORTED; }
#undef CPRUNE_ROWS_CASE
  return CPRUNE_OK;
}

int launch_conv_rows_f16(int id, dim3 grid, hipStream_t s, const RowsArgs& a);
int launch_conv_rows_bf16(int id, dim3 grid, hipStream_t s, const RowsArgs& a);

}  // namespace cprune
