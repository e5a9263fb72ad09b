// 3x3 / stride 2 / pad 1 convolution, channels-last, without LDS in the main loop: the row-strip kernel (conv_rows_kernel.hpp) at
// stride 2, in 16-bit data and in fp32 on three bf16 parts (conv_split_kernel.hpp has the error and the range of that).  A strip is
// 16 output columns x R output rows; an input row is two operands, its even columns (the window's middle) and its odd ones (the
// window's right; shifted by a lane its left).  Even rows serve one output row, odd ones two.  Strips of a map wider than 16
// overlap by a column, whose left neighbour lies in the strip before.
//
// The layer that halves a residual network's map has a 1x1 / stride 2 layer beside it on the same input, whose operand is the
// middle tap's.  Its filter tiles can be work-groups of the same launch: alone they are a launch of some three microseconds of
// little work, which nothing overlaps.
//
// Measured, bf16 (us), the best other kernel / this one: batch 32, 64 -> 67 at 56x56 12.4 / 12.2, 256 -> 158 at 14x14 10.1 / 7.5; one image,
// 128 -> 173 at 28x28 5.2 / 3.9, 256 -> 158 7.6 / 4.3; with the 1x1 layer beside it (two launches / one): batch 32, 64 -> 67 and 128 at 56x56
// 20.0 / 15.8, 128 -> 173 and 256 17.7 / 15.0, 256 -> 158 and 512 16.5 / 12.6; one image 8.0 / 4.0, 9.6 / 5.3, 12.5 / 4.4; 45 random layers, timed
// choice 1.33 times as fast as before, fp32 1.13.  What bounds it: loads: 2 R + 1 rows of two operands and nine taps a chunk, a
// kilobyte each from the vector cache, for 9 R MFMAs per filter block, which is why two and three blocks per wavefront win at batch 32 (counters there,
// bf16: wavefronts waiting for memory 46-51 % of their cycles, matrix pipes busy 13-15 %); in fp32 also cutting, four operands per output row.  Four blocks (a wavefront per SIMD) were never the fastest.
#pragma once
#include "conv_rows_kernel.hpp"

namespace cprune {

struct RowsS2Args : RowsArgs {
  int Hi, Wi;                      // the input map
  int tiles_m1;                    // filter tiles of the 3x3 layer; those behind them are the 1x1 layer's
  const void* w2;                  // launch_pack_split, whole chunks
  const float* bias2;
  void* y2;
  const void* w2_raw;              // fp32: [o][cp]
  int O2, Cop2, act2;
  unsigned w2_bytes, y2_bytes, w2_raw_bytes;
};

// Numbers of 8 channels of a pixel as they come from memory, and as operands
template <typename T> struct RawRow { uint4 q[sizeof(T) / 2]; };
template <typename T> struct Operand { uint4 p[SplitParts<T>::value]; };

template <typename T>
__device__ __forceinline__ Operand<T> to_operand(const RawRow<T>& v) {
  if constexpr (sizeof(T) == 2) return Operand<T>{{v.q[0]}};
  else {
    uint32_t h[4], m[4], l[4];
    split3(v.q[0].x, v.q[0].y, h[0], m[0], l[0]); split3(v.q[0].z, v.q[0].w, h[1], m[1], l[1]);
    split3(v.q[1].x, v.q[1].y, h[2], m[2], l[2]); split3(v.q[1].z, v.q[1].w, h[3], m[3], l[3]);
    return Operand<T>{{make_uint4(h[0], h[1], h[2], h[3]), make_uint4(m[0], m[1], m[2], m[3]), make_uint4(l[0], l[1], l[2], l[3])}};
  }
}

template <typename T, int MB, int R, int KS>
__global__ __launch_bounds__(KS == 8 ? 512 : 256, 2) void conv_rows_s2_kernel(RowsS2Args a) {
  constexpr int ES = (int)sizeof(T), P = SplitParts<T>::value, NQ = ES / 2;
  constexpr int ROWS = 2 * R + 1;                           // input rows of a strip
  constexpr int PF = P == 1 ? 3 : 2;                        // rows asked for ahead
  constexpr int STEPS = (ROWS + PF - 1) / PF * PF;          // (a whole number of turns of their ring)
  static_assert(R % 2 == 0, "pairs of rows");
  const RowsAt at = rows_at<MB, KS>(a);
  const int lane = at.lane, r = at.r, g4 = at.g4, slice = at.slice, img = at.img, cx = at.cx;
  const int iy0 = 2 * at.ty * R - 1;
  const bool second = at.tile_m >= a.tiles_m1;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const int row_bytes = a.Wi * a.Cp * ES;
  const int x_off = ((img * a.Hi + iy0) * a.Wi + 2 * cx) * a.Cp * ES + g4 * (8 * ES);
  const bool odd_ok = at.col_ok & (2 * cx + 1 < a.Wi);
  auto load_pixel = [&](int c, int i, bool odd, RawRow<T>& v) CPRUNE_INLINE {
    const bool in = ((unsigned)(iy0 + i) < (unsigned)a.Hi) & (odd ? odd_ok : at.col_ok);
    const int off = x_off + i * row_bytes + (odd ? a.Cp * ES : 0);
#pragma unroll
    for (int e = 0; e < NQ; ++e) {
      const bool ch = c * 32 + g4 * 8 + e * (16 / ES) < a.Cp;
      v.q[e] = load_b128(xr, in & ch ? (unsigned)(off + c * (32 * ES) + e * 16) : kOutOfRange, 0);
    }
  };

  float4_t acc[R][MB], small[P == 3 ? R : 1][MB];
#pragma unroll
  for (int y = 0; y < R; ++y)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[y][m] = small[P == 3 ? y : 0][m] = (float4_t){0.f, 0.f, 0.f, 0.f};
  // product pw * px of the parts, into the sum of its size
  auto product = [&](const uint4& w, const uint4& x, int pw, int px, int y, int m) CPRUNE_INLINE {
    float4_t& d = pw + px == 0 ? acc[y][m] : small[P == 3 ? y : 0][m];
    d = mfma_split<T>(w, x, d);
  };
  constexpr int NPROD = P == 3 ? 6 : 1;
  constexpr int kW[6] = {0, 0, 2, 1, 0, 1}, kX[6] = {P == 3 ? 2 : 0, 0, 0, 1, 1, 0};

  RowsArgs f = a;                  // (what the sums' end needs)
  int o0 = at.o0;
  const void* w_raw = a.w_raw;
  unsigned w_raw_bytes = a.w_raw_bytes;
  int taps = 9;
  if (!second) {
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);
    uint4 wt[3][3][MB][P];
    auto load_taps = [&](int c, int u) CPRUNE_INLINE {
      const bool past = c >= a.nchunk;
#pragma unroll
      for (int v = 0; v < 3; ++v)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int p = 0; p < P; ++p)
            wt[u][v][m][p] = load_b128(wr, past | (o0 + m * 16 >= a.O) ? kOutOfRange :
                                       (unsigned)((((at.tile_m * MB + m) * a.nchunk + c) * 9 + u * 3 + v) * P + p) * 1024u + (unsigned)lane * 16u, 0);
    };
    RawRow<T> pre[PF][2];
    // the loads of step i of chunk c: the row PF steps on, and the taps that step has used for the last time
    auto ask = [&](int c, int i) CPRUNE_INLINE {
      const int row = (i + PF) % STEPS, cr = i + PF < STEPS ? c : c + KS;
      if (row < ROWS) {
        load_pixel(cr, row, false, pre[i % PF][0]);
        load_pixel(cr, row, true, pre[i % PF][1]);
      }
      if (i >= 2 * R - 2 && i <= 2 * R) load_taps(c + KS, i - (2 * R - 2));
      __builtin_amdgcn_sched_barrier(0);
    };
    // (in the order in which the loop asks for them, so that the waits at its head count the same loads on both ways in)
    constexpr int BEGIN = STEPS - PF < 2 * R - 2 ? STEPS - PF : 2 * R - 2;
#pragma unroll
    for (int i = BEGIN; i < STEPS; ++i) ask(slice - KS, i);
    const unsigned ml = at.lr > 0 ? ~0u : 0u;
    auto left_of = [&](const Operand<T>& x) CPRUNE_INLINE -> Operand<T> {
      auto one = [&](unsigned v) -> unsigned { return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true) & ml; };
      Operand<T> s;
#pragma unroll
      for (int p = 0; p < P; ++p) s.p[p] = make_uint4(one(x.p[p].x), one(x.p[p].y), one(x.p[p].z), one(x.p[p].w));
      return s;
    };
    for (int c = slice; c < a.nchunk; c += KS) {
#pragma unroll
      for (int i = 0; i < STEPS; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        if (i < ROWS && (unsigned)(iy0 + i) < (unsigned)a.Hi) {
          const Operand<T> even = to_operand(pre[i % PF][0]);
          auto column = [&](const Operand<T>& b, int v) CPRUNE_INLINE {
#pragma unroll
            for (int k = 0; k < NPROD; ++k)
#pragma unroll
              for (int u = 0; u < 3; ++u) {
                if ((i - u) % 2 != 0 || i < u || (i - u) / 2 >= R) continue;
#pragma unroll
                for (int m = 0; m < MB; ++m) product(wt[u][v][m][kW[k]], b.p[kX[k]], kW[k], kX[k], (i - u) / 2, m);
              }
          };
          column(even, 1);
          const Operand<T> odd = to_operand(pre[i % PF][1]);
          column(odd, 2);
          column(left_of(odd), 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        ask(c, i);
      }
    }
  } else {
    // the 1x1 layer: even columns of the middle rows
    o0 = (at.tile_m - a.tiles_m1) * (MB * 16);
    f.bias = a.bias2; f.res = nullptr; f.y = a.y2; f.O = a.O2; f.Cop = a.Cop2; f.act = a.act2; f.y_bytes = a.y2_bytes;
    w_raw = a.w2_raw; w_raw_bytes = a.w2_raw_bytes; taps = 1;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w2, a.w2_bytes);
    uint4 w0[MB][P], w1[MB][P];
    RawRow<T> x0[R], x1[R];
    auto ask = [&](int c, uint4 (&w)[MB][P], RawRow<T> (&x)[R]) CPRUNE_INLINE {
      const bool past = c >= a.nchunk;
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int p = 0; p < P; ++p)
          w[m][p] = load_b128(wr, past | (o0 + m * 16 >= a.O2) ? kOutOfRange :
                              (unsigned)(((o0 / 16 + m) * a.nchunk + c) * P + p) * 1024u + (unsigned)lane * 16u, 0);
#pragma unroll
      for (int y = 0; y < R; ++y) load_pixel(c, 2 * y + 1, false, x[y]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto run = [&](const uint4 (&w)[MB][P], const RawRow<T> (&x)[R]) CPRUNE_INLINE {
#pragma unroll
      for (int y = 0; y < R; ++y) {
        const Operand<T> b = to_operand(x[y]);
#pragma unroll
        for (int k = 0; k < NPROD; ++k)
#pragma unroll
          for (int m = 0; m < MB; ++m) product(w[m][kW[k]], b.p[kX[k]], kW[k], kX[k], y, m);
      }
    };
    ask(slice, w0, x0);
    for (int c = slice; c < a.nchunk; c += 2 * KS) {
      ask(c + KS, w1, x1);
      run(w0, x0);
      ask(c + 2 * KS, w0, x0);
      run(w1, x1);                               // (past the last chunk: zeros)
    }
  }

  if constexpr (P == 3) {
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
      for (int m = 0; m < MB; ++m) acc[y][m] += small[y][m];
    // data that three parts do not hold shows in the sums (see conv_split_kernel): then the slice once more on the fp32
    // instruction, operands straight from memory
    constexpr uint32_t kInf = 0x7f800000u, kSmall = (127u - 50u) << 23;
    uint32_t top = 0, low = ~0u;
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t mag = __float_as_uint(acc[y][m][q]) & 0x7fffffffu;
          top = max(top, mag);
          low = min(low, mag - 1);      // (zero goes to the other end)
        }
    if (__any(top >= kInf || low < kSmall - 1)) {
      const __amdgpu_buffer_rsrc_t ww = make_rsrc(w_raw, w_raw_bytes);
#pragma unroll
      for (int y = 0; y < R; ++y)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[y][m] = (float4_t){0.f, 0.f, 0.f, 0.f};
      for (int c = slice; c < a.nchunk; c += KS)
        for (int tap = 0; tap < taps; ++tap) {
          const int u = taps == 1 ? 1 : tap / 3, v = taps == 1 ? 1 : tap - u * 3, ix = 2 * cx + v - 1;
          const bool col = at.col_ok & ((unsigned)ix < (unsigned)a.Wi);
          for (int ch = c * 32 + g4; ch < c * 32 + 32; ch += 4) {
            const bool real = ch < a.Cp;
            float wv[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
              const int o = o0 + m * 16 + r;
              wv[m] = __uint_as_float(Elem<float>::load(ww, real & (o < f.O) ? (unsigned)((o * taps + tap) * a.Cp + ch) * 4u : kOutOfRange, 0));
            }
#pragma unroll
            for (int y = 0; y < R; ++y) {
              const int iy = 2 * (at.ty * R + y) + u - 1;
              const bool in = real & col & ((unsigned)iy < (unsigned)a.Hi);
              const float xv = __uint_as_float(Elem<float>::load(xr, in ? (unsigned)(((img * a.Hi + iy) * a.Wi + ix) * a.Cp + ch) * 4u : kOutOfRange, 0));
#pragma unroll
              for (int m = 0; m < MB; ++m) acc[y][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[m], xv, acc[y][m], 0, 0, 0);
            }
          }
        }
    }
  }
  RowsAt end = at;
  end.o0 = o0;
  rows_finish<T, MB, R, KS>(f, end, acc);
}

// Variants: id, 16-filter blocks, output rows of a strip, wavefronts that share a strip (fp32: those of one block and at most four rows)
#define CPRUNE_ROWS_S2_LIST(X) \
  X(0, 1, 8, 1) X(1, 1, 8, 2) X(2, 1, 8, 4) X(3, 2, 8, 1) X(4, 2, 8, 2) X(5, 2, 4, 1) X(6, 2, 4, 2) X(7, 2, 4, 4) \
  X(8, 1, 4, 1) X(9, 1, 4, 2) X(10, 1, 4, 4) X(11, 1, 4, 8) X(12, 1, 2, 2) X(13, 1, 2, 4) X(14, 1, 2, 8) \
  X(15, 3, 4, 1) X(16, 3, 4, 2) X(17, 3, 4, 4)

constexpr int kNumRowsS2 = 18;

template <typename T>
inline int launch_rows_s2(int id, dim3 grid, hipStream_t s, const RowsS2Args& a) {
#define CPRUNE_ROWS_S2_CASE(ID, MB_, R_, KS_)                                                                        \
  case ID:                                                                                                           \
    if constexpr (sizeof(T) == 2 || (MB_ == 1 && R_ <= 4)) {                                                         \
      hipLaunchKernelGGL((conv_rows_s2_kernel<T, MB_, R_, KS_>), grid, dim3(KS_ == 8 ? 512 : 256), 0, s, a);         \
      return CPRUNE_OK;                                                                                              \
    }                                                                                                                \
    break;
  switch (id) { CPRUNE_ROWS_S2_LIST(CPRUNE_ROWS_S2_CASE) default: break; }
#undef CPRUNE_ROWS_S2_CASE
  return CPRUNE_ERR_UNSUPPORTED;
}

int launch_conv_rows_s2_f32(int id, dim3 grid, hipStream_t s, const RowsS2Args& a);
int launch_conv_rows_s2_f16(int id, dim3 grid, hipStream_t s, const RowsS2Args& a);
int launch_conv_rows_s2_bf16(int id, dim3 grid, hipStream_t s, const RowsS2Args& a);

}  // namespace cprune
