// 3x3 / stride 1 / pad 1 convolution in the boundary's layout (NCHW, OIHW weights): the row strips of conv_rows_kernel.hpp on tensors
// as a caller has them, in 16-bit data and in fp32 on three bf16 parts (conv_split_kernel.hpp has the error and the range of that).
//   activations  a lane's operand is 8 channels of one column: eight loads of a number each, 16 lanes on 16 consecutive columns of a
//                plane.  As in the fp32 row strips a row is cut while the row before it is multiplied, its left and right
//                columns are the same registers shifted by a lane, and strips of a map wider than 16 overlap by two columns.
//   weights      nothing is packed beforehand: the wavefronts of a work-group that work on the same slice of the channels read a chunk's
//                weights as they lie (two channels' nine taps per thread, consecutive in memory), cut them and leave them in
//                LDS in operand order; each takes its nine taps from there into registers for all rows of its strip.
// KS > 1: KS wavefronts share a strip and split its chunks; their sums meet in LDS at the end, in order.
//
// Measured, the best other kernel (the split kernel with its packing launch, or the general one) / this one (us): fp32 128 -> 83 at 56x56,
// batch 8, 44 / 35.5 (135 TFLOP/s); 64 -> 45 at 32x32, one image, 10.4 / 6.6; 205 -> 13 at 110x110, batch 9, 68 / 46; bf16 128 -> 83 24 / 17.3;
// 64 -> 45 10.6 / 4.9; 322 -> 167 at 44x44, one image, 26 / 16.  What bounds it: one image, launch and a chain of loads, LDS, MFMAs and stores;
// large layers in fp32 cutting and the matrix pipes (128 -> 83: a third of the rate of six bf16 products; counters: vector ALU busy 59 %, matrix
// pipes 51, waiting 19), in 16-bit data the eight loads of a number per row and chunk (vector ALU 40 %, matrix pipes 16, waiting 35).  16-bit weights
// of an odd channel count come as whole dwords shifted into place: a load per number (eighteen a thread) made 495 -> 276 at 41x41 48 us, now 28.
#pragma once
#include "conv_rows_s2_kernel.hpp"

namespace cprune {

template <typename T, int MB, int R, int KS>
__global__ __launch_bounds__(256, 2) void conv_rows_nchw_kernel(RowsArgs a) {
  constexpr int ES = (int)sizeof(T), P = SplitParts<T>::value;
  constexpr int ROWS = R + 2, PF = 2;
  constexpr int TAP = P * 1024;                  // bytes of one tap of a filter block in LDS: [part][lane][16]
  constexpr int NT = 256 / KS;                   // threads that stage a slice's weights
  constexpr int NI = MB * 256 / NT;              // (filter, pair of channels) items per thread
  static_assert(KS <= 4 && ROWS % PF == 0, "four wavefronts; ring of rows");
  constexpr int SUMS = KS > 1 ? (4 / KS) * (KS - 1) * R * MB * 1024 : 0, WEIGHTS = KS * MB * 9 * TAP;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SUMS > WEIGHTS ? SUMS : WEIGHTS];
  const RowsAt at = rows_at<MB, KS>(a);
  const int lane = at.lane, r = at.r, g4 = at.g4, slice = at.slice, o0 = at.o0, lr = at.lr, img = at.img, cx = at.cx;
  const int C = a.Cp, hw = a.H * a.W;
  const int iy0 = at.ty * R - 1;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);

  // ---- weights: memory -> registers -> LDS ----
  unsigned char* const w_lds = smem + slice * (MB * 9 * TAP);
  const int st = at.sub * 64 + lane;             // this thread among those of its slice
  constexpr int WV = ES == 4 ? 18 : 10;          // dwords of two channels' taps (16-bit: those they lie in)
  uint32_t wv[NI][WV];
  // 16-bit data: from the 4-byte boundary in front of the weights to the one behind them (a dword of which a half is there is read whole)
  const unsigned w_shift = ES == 4 ? 0u : (unsigned)(uintptr_t)a.w & 2u;
  const __amdgpu_buffer_rsrc_t wd = make_rsrc((const char*)a.w - w_shift, (a.w_bytes + w_shift + 3u) & ~3u);
  // (which item: filter of the tile, pair of channels of the chunk)
  auto filter_of = [&](int j) CPRUNE_INLINE { return (st + j * NT) >> 4; };
  auto load_weights = [&](int c) CPRUNE_INLINE {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int o = o0 + filter_of(j), ch = c * 32 + (st & 15) * 2;
      const unsigned off = (unsigned)((o * C + ch) * 9) * ES;
      const bool ok0 = (o < a.O) & (ch < C), ok1 = (o < a.O) & (ch + 1 < C);
      if constexpr (ES == 4) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {            // every load lies inside one channel's taps
          const unsigned at_h = (h ? ok1 : ok0) ? off + h * 36u : kOutOfRange;
          const uint4 q0 = load_b128(wr, at_h, 0), q1 = load_b128(wr, at_h == kOutOfRange ? kOutOfRange : at_h + 16u, 0);
          wv[j][h * 9] = q0.x; wv[j][h * 9 + 1] = q0.y; wv[j][h * 9 + 2] = q0.z; wv[j][h * 9 + 3] = q0.w;
          wv[j][h * 9 + 4] = q1.x; wv[j][h * 9 + 5] = q1.y; wv[j][h * 9 + 6] = q1.z; wv[j][h * 9 + 7] = q1.w;
          wv[j][h * 9 + 8] = Elem<float>::load(wr, at_h == kOutOfRange ? kOutOfRange : at_h + 32u, 0);
        }
      } else {
        const unsigned from = (off + w_shift) & ~3u;      // one channel's taps lie in the first five dwords, whichever half they begin in
        const uint4 q0 = load_b128(wd, ok0 ? from : kOutOfRange, 0), q1 = load_b128(wd, ok1 ? from + 20u : kOutOfRange, 0);
        wv[j][0] = q0.x; wv[j][1] = q0.y; wv[j][2] = q0.z; wv[j][3] = q0.w;
        wv[j][4] = Elem<float>::load(wd, ok0 ? from + 16u : kOutOfRange, 0);
        wv[j][5] = q1.x; wv[j][6] = q1.y; wv[j][7] = q1.z; wv[j][8] = q1.w;
        wv[j][9] = Elem<float>::load(wd, ok1 && ((off + w_shift) & 2u) ? from + 36u : kOutOfRange, 0);
      }
    }
  };
  auto store_weights = [&](int w_chunk) CPRUNE_INLINE {      // (what load_weights(w_chunk) has asked for)
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int f = filter_of(j), pr = st & 15;
      unsigned char* const d = w_lds + (f >> 4) * (9 * TAP) + ((pr >> 2) * 16 + (f & 15)) * 16 + (pr & 3) * 4;
      uint32_t h[9];                             // 16-bit data: halves 0 .. 17 in place, without what lies behind the last channel
      if constexpr (ES == 2) {
        const unsigned half = ((unsigned)((o0 + f) * C + w_chunk * 32 + pr * 2) * 18u + w_shift) & 2u;
        const bool two = w_chunk * 32 + pr * 2 + 1 < C;
#pragma unroll
        for (int k = 0; k < 9; ++k) h[k] = __builtin_amdgcn_alignbit(wv[j][k + 1], wv[j][k], half * 8);
        if (!two) {
          h[4] &= 0xffffu;
#pragma unroll
          for (int k = 5; k < 9; ++k) h[k] = 0;
        }
      }
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        uint32_t p[3];
        if constexpr (ES == 4) split3(wv[j][tap], wv[j][9 + tap], p[0], p[1], p[2]);
        else {                                   // halves tap and 9 + tap of the 18
          const uint32_t lo = tap & 1 ? h[tap >> 1] >> 16 : h[tap >> 1] & 0xffffu;
          const uint32_t hi = (9 + tap) & 1 ? h[(9 + tap) >> 1] & 0xffff0000u : h[(9 + tap) >> 1] << 16;
          p[0] = lo | hi;
        }
#pragma unroll
        for (int q = 0; q < P; ++q) *(uint32_t*)(d + tap * TAP + q * 1024) = p[q];
      }
    }
  };
  uint4 wt[3][3][MB][P];
  auto load_taps = [&](int u) CPRUNE_INLINE {
#pragma unroll
    for (int v = 1; v < 4; ++v)                  // (in the order of their use)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int p = 0; p < P; ++p) wt[u][v % 3][m][p] = *(const uint4*)(w_lds + (m * 9 + u * 3 + v % 3) * TAP + p * 1024 + lane * 16);
  };

  // ---- activations ----
  struct Raw { uint32_t q[ES == 4 ? 8 : 4]; };
  const int x_off = (((img * C + g4 * 8) * a.H + iy0) * a.W + cx) * ES;
  auto load_row = [&](int c, int i, Raw& v) CPRUNE_INLINE {
    const bool in = ((unsigned)(iy0 + i) < (unsigned)a.H) & at.col_ok;
    const unsigned off = in ? (unsigned)(x_off + i * a.W * ES) : kOutOfRange;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t t = Elem<T>::load(xr, off | ((unsigned)(c * 32 + g4 * 8 + e >= C) << 31), (unsigned)(min(c * 32 + e, C - 1) * hw) * ES);
      if constexpr (ES == 4) v.q[e] = t;
      else if (e & 1) v.q[e >> 1] |= t << 16;
      else v.q[e >> 1] = t;
    }
  };
  auto cut = [&](const Raw& v) CPRUNE_INLINE -> Operand<T> {
    if constexpr (ES == 4)
      return to_operand<float>(RawRow<float>{{make_uint4(v.q[0], v.q[1], v.q[2], v.q[3]), make_uint4(v.q[4], v.q[5], v.q[6], v.q[7])}});
    else return Operand<T>{{make_uint4(v.q[0], v.q[1], v.q[2], v.q[3])}};
  };
  const unsigned ml = lr > 0 ? ~0u : 0u, mr = lr < (1 << a.lane_shift) - 1 ? ~0u : 0u;
  auto shifted = [&](const Operand<T>& x, auto left_tag) CPRUNE_INLINE -> Operand<T> {
    constexpr bool left = decltype(left_tag)::value;
    constexpr int ctrl = left ? 0x111 : 0x101;       // row_shr:1 (the lane takes its left neighbour's) / row_shl:1
    auto one = [&](unsigned v) -> unsigned { return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true) & (left ? ml : mr); };
    Operand<T> s;
#pragma unroll
    for (int p = 0; p < P; ++p) s.p[p] = make_uint4(one(x.p[p].x), one(x.p[p].y), one(x.p[p].z), one(x.p[p].w));
    return s;
  };

  float4_t acc[R][MB], small[P == 3 ? R : 1][MB];
#pragma unroll
  for (int y = 0; y < R; ++y)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[y][m] = small[P == 3 ? y : 0][m] = (float4_t){0.f, 0.f, 0.f, 0.f};
  constexpr int NPROD = P == 3 ? 6 : 1;
  constexpr int kW[6] = {0, 0, 2, 1, 0, 1}, kX[6] = {P == 3 ? 2 : 0, 0, 0, 1, 1, 0};

  // every wavefront makes the same number of turns (they share barriers); one past its slice's last chunk multiplies zeros
  const int turns = (a.nchunk + KS - 1) / KS;
  Raw pre[PF];
  load_weights(slice);
  load_row(slice, 0, pre[0]);
  load_row(slice, 1, pre[1]);
  store_weights(slice);
  load_weights(slice + KS);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u) load_taps(u);
  Operand<T> x = cut(pre[0]);
  load_row(slice, 2, pre[0]);

  for (int turn = 0; turn < turns; ++turn) {
    const int c = slice + turn * KS;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i == 1 && turn + 1 < turns) {
        __syncthreads();                         // everyone has the present taps in registers
        store_weights(c + KS);
        load_weights(c + 2 * KS);
        __syncthreads();
      }
      const int slot = (i + 1) % PF;
      Operand<T> nx;
      auto cut_next = [&](auto apart) CPRUNE_INLINE {
        Raw q = pre[slot];
        if constexpr (decltype(apart)::value) {      // (opaque: otherwise the compiler moves what both branches do before them)
#pragma unroll
          for (int k = 0; k < (ES == 4 ? 8 : 4); ++k) asm("" : "+v"(q.q[k]));
        }
        nx = cut(q);
      };
      if ((unsigned)(iy0 + i) < (unsigned)a.H) {
        auto column = [&](const Operand<T>& b, int v) CPRUNE_INLINE {
#pragma unroll
          for (int k = 0; k < NPROD; ++k)
#pragma unroll
            for (int u = 0; u < 3; ++u) {
              if (i - u < 0 || i - u >= R) continue;
#pragma unroll
              for (int m = 0; m < MB; ++m) {
                float4_t& d = kW[k] + kX[k] == 0 ? acc[i - u][m] : small[P == 3 ? i - u : 0][m];
                d = mfma_split<T>(wt[u][v][m][kW[k]], b.p[kX[k]], d);
              }
            }
        };
        column(x, 1);
        column(shifted(x, std::false_type{}), 2);
        column(shifted(x, std::true_type{}), 0);
        cut_next(std::false_type{});
        if constexpr (P == 3) {
          // vector operations between the MFMAs, not in front of them
#pragma unroll
          for (int k = 0; k < 54; ++k) {
            if (k >= 18 * ((i < 2 ? i + 1 : 3) - (i >= R ? i - R + 1 : 0))) break;
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
          }
        }
      } else {
        cut_next(std::true_type{});
      }
      x = nx;
      __builtin_amdgcn_sched_barrier(0);
      if (i + 3 < ROWS) load_row(c, i + 3, pre[slot]);
      else load_row(c + KS, i + 3 - ROWS, pre[slot]);
      if (i >= R - 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (i == R - 1 + u) load_taps(u);        // (behind the last chunk: the present ones again, which nothing uses)
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
#pragma unroll
      for (int y = 0; y < R; ++y)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[y][m] = (float4_t){0.f, 0.f, 0.f, 0.f};
      for (int c = slice; c < a.nchunk; c += KS)
        for (int tap = 0; tap < 9; ++tap) {
          const int u = tap / 3, ix = cx + tap - u * 3 - 1;
          const bool col = at.live & (img < a.N) & ((unsigned)ix < (unsigned)a.W);
          for (int ch = c * 32 + g4; ch < c * 32 + 32; ch += 4) {
            const bool real = ch < C;
            float wf[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
              const int o = o0 + m * 16 + r;
              wf[m] = __uint_as_float(Elem<float>::load(wr, real & (o < a.O) ? (unsigned)((o * C + ch) * 9 + tap) * 4u : kOutOfRange, 0));
            }
#pragma unroll
            for (int y = 0; y < R; ++y) {
              const int iy = at.ty * R + y + u - 1;
              const bool in = real & col & ((unsigned)iy < (unsigned)a.H);
              const float xv = __uint_as_float(Elem<float>::load(xr, in ? (unsigned)(((img * C + ch) * a.H + iy) * a.W + ix) * 4u : kOutOfRange, 0));
#pragma unroll
              for (int m = 0; m < MB; ++m) acc[y][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[m], xv, acc[y][m], 0, 0, 0);
            }
          }
        }
    }
  }

  if constexpr (KS > 1) {
    // the other slices' wavefronts hand their sums to the first, which adds them in order
    constexpr int SLOT = R * MB * 64;
    float4_t* const mine = (float4_t*)smem + at.sub * ((KS - 1) * SLOT) + lane;
    __syncthreads();                             // (the weights' place)
    if (slice > 0) {
#pragma unroll
      for (int q = 0; q < R * MB; ++q) mine[(slice - 1) * SLOT + q * 64] = acc[q / MB][q % MB];
    }
    __syncthreads();
    if (slice > 0) return;
#pragma unroll
    for (int k = 1; k < KS; ++k)
#pragma unroll
      for (int q = 0; q < R * MB; ++q) acc[q / MB][q % MB] += mine[(k - 1) * SLOT + q * 64];
  }
  // bias, shortcut, activation; a lane stores its column of four filters' planes
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res, a.res ? a.y_bytes : 0u);
  const float lo = a.act == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f, hi = a.act == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int o = o0 + m * 16 + 4 * g4;
    const float4_t bias = load_bias4(a.bias, a.O, o);
#pragma unroll
    for (int y = 0; y < R; y += 2) {
      unsigned off[2][4];
      float s[2][4];
#pragma unroll
      for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int oy = at.ty * R + y + z;
          off[z][q] = at.out_ok & (oy < a.H) & (o + q < a.O) ? (unsigned)(((img * a.O + o + q) * a.H + oy) * a.W + cx) * ES : kOutOfRange;
          s[z][q] = acc[y + z][m][q] + bias[q];
          if (a.res) {
            const uint32_t v = Elem<T>::load(rr, off[z][q], 0);
            if constexpr (ES == 4) s[z][q] += __uint_as_float(v);
            else s[z][q] += Elem<T>::to_f32(__builtin_bit_cast(T, (uint16_t)v));
          }
        }
#pragma unroll
      for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (off[z][q] != kOutOfRange) *(T*)((char*)a.y + off[z][q]) = Elem<T>::from_f32(fminf(fmaxf(s[z][q], lo), hi));
    }
  }
}

// Variants: id, 16-filter blocks, rows of a strip, wavefronts that share a strip (fp32: those of one block, at most six rows and two
// wavefronts: eight rows spill 63 registers)
#define CPRUNE_ROWS_NCHW_LIST(X) \
  X(0, 1, 8, 1) X(1, 1, 4, 1) X(2, 1, 4, 2) X(3, 1, 2, 1) X(4, 1, 2, 2) X(5, 2, 8, 1) X(6, 2, 4, 1) X(7, 2, 4, 2) X(8, 1, 2, 4) \
  X(9, 1, 6, 1) X(10, 2, 6, 1)

constexpr int kNumRowsNchw = 11;

template <typename T>
inline int launch_rows_nchw(int id, dim3 grid, hipStream_t s, const RowsArgs& a) {
#define CPRUNE_ROWS_NCHW_CASE(ID, MB_, R_, KS_)                                                                      \
  case ID:                                                                                                           \
    if constexpr (sizeof(T) == 2 || (MB_ == 1 && R_ <= 6 && KS_ <= 2)) {                                                        \
      hipLaunchKernelGGL((conv_rows_nchw_kernel<T, MB_, R_, KS_>), grid, dim3(256), 0, s, a);                        \
      return CPRUNE_OK;                                                                                              \
    }                                                                                                                \
    break;
  switch (id) { CPRUNE_ROWS_NCHW_LIST(CPRUNE_ROWS_NCHW_CASE) default: break; }
#undef CPRUNE_ROWS_NCHW_CASE
  return CPRUNE_ERR_UNSUPPORTED;
}

int launch_conv_rows_nchw_f32(int id, dim3 grid, hipStream_t s, const RowsArgs& a);
int launch_conv_rows_nchw_f16(int id, dim3 grid, hipStream_t s, const RowsArgs& a);
int launch_conv_rows_nchw_bf16(int id, dim3 grid, hipStream_t s, const RowsArgs& a);

}  // namespace cprune
