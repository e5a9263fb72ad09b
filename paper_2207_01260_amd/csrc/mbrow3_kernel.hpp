// Inverted-residual blocks in fp32: mbrow_kernel.hpp's strips (a wavefront runs expansion, depthwise layer and projection of 16 columns x
// R output rows in registers) with both matrix products on three bf16 parts per number (conv_split_kernel.hpp has the error of that).
//
// Why: v_mfma_f32_16x16x4_f32 shares the vector ALU.  Measured on one SIMD, it takes 13.7 ns alone, 19 with one vector operation behind it
// and 21 / 23 / 25 with two to four; v_mfma_f32_16x16x32_bf16 7.5 ns alone or with two, 8.9 with three.  In a kernel that spends as many
// clocks on the depthwise window as on the products the fp32 instruction makes the two take turns.
//
// 16 channels are three MFMAs of 32: a lane's eight places of the reduction are its four channels twice, so that
//   (wm, wh) x (m, m)  =  wm m + wh m,      (wm, wh) x (h, h)  =  wm h + wh h,      (wh, wl) x (l, h)  =  wh l + wl h
// are the six products of conv_split_kernel, and what the depthwise layer leaves in a lane (four channels of a pixel), cut, is the
// projection's operand without a move between lanes.  The strip's input is cut once, while it is staged; weights come packed as
// operands from launch_pack_parts.  The projection's 16 terms are summed by themselves and
// added to the row's sum by the vector ALU, one rounding of that per 16 terms; with the three MFMAs on the sum itself 300 and more terms were 5-14 % further
// from the exact result than on the fp32 instruction.
//
// What bounds it: vector operations, some hundred a row and chunk (36 window products, 20 moves and clamps, 26 to cut the finished row), beside
// 9-30 MFMAs; two wavefronts per SIMD; weights of the next chunk from L2 some 500 clocks ahead; launch, staging and stores.
// Counters over MobileNetV2's 13 launches at batch 64: vector ALU busy 53 % of the cycles in which a unit has work (image form 77), matrix pipes 22, wavefronts waiting
// for memory or a barrier 32 % of their cycles and to issue 23.  Measured, batch 64,
// fp32 instruction / this kernel (us): 24 -> 86 -> 32 at 56x56 stride 2 24.8 / 22.6; 32 -> 92 -> 32 at 28x28 17.5 / 14.0; 32 -> 115 -> 64 stride 2
// 14.8 / 12.2; 64 -> 330 -> 64 at 14x14 23.8 / 20; 64 -> 196 -> 96 21.7 (apart) / 18.8; 96 -> 385 -> 96 36.7 / 34 (depthwise and projection); 16 -> 50 ->
// 24 at 112x112 stride 2 42.5 / 39.5; 24 -> 65 -> 24 at 56x56 34.6 / 34; image -> 32 -> 16 64 / 58; MobileNetV2 542 -> 494.  Error against 64 bits: 24 -> 65 -> 24 1.5e-7 /
// 1.1e-7, 64 -> 330 -> 64 2.7e-7 / 1.7e-7.  Left to the compiler's order of the row's operations the same kernel gained nothing (24 -> 65 -> 24 38.6).
//
// Numbers three parts do not hold send the strip's wavefronts through mbrow3_slow, the same steps on the fp32 instruction: where an input, or
// without an expansion a depthwise result, is from the limit up that launch_parts_limit puts behind the packed weights (infinities and
// NaN always are, whatever the block's weights), and where a sum at the end is not finite, or not zero and below 2^-50.  Within the limit
// what numbers below 2^-110 lose stays below the last place of every sum from 2^-50 up (parts_limit.hpp); numbers below 2^-133, all denormal,
// count as zero, and a sum that comes out as zero is not made again.  Projections of fewer than 16 terms without an expansion always go that way:
// the instruction rounds those less than what parts leave out (3 -> 4 -> 24: 6.5e-8 / 7.3e-8); expansions of few terms are no worse on
// parts (3 -> 40 -> 24 8.7e-8 / 7.4e-8, 1 -> 40 -> 24 9.0e-8 / 7.5e-8, whole blocks against 64 bits).
#pragma once
#include "conv_split_kernel.hpp"
#include "mbrow_kernel.hpp"

namespace cprune {

typedef unsigned long long ulong2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

// the larger of two pairs of magnitudes of bf16 numbers
__device__ __forceinline__ unsigned max_bf16x2(unsigned seen, unsigned h) {
  return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, seen), __builtin_bit_cast(ushort2_t, h & 0x7fff7fffu)));
}

// f(0) ... f(N - 1), the index a constant of its own type (loops that the compiler would have to unroll before it can choose are too large for
// it); f(A) ... f(B - 1)
template <int A, int... I, typename F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F&& f) { (f(std::integral_constant<int, A + I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void each(F&& f) { each_of<0>(std::make_integer_sequence<int, N>{}, f); }
template <int A, int B, typename F>
__device__ __forceinline__ void each_from(F&& f) { each_of<A>(std::make_integer_sequence<int, B - A>{}, f); }

// Weights of 16 rows x 16 channels, operands as they lie in memory: (wh, wl), (wm, wh) or, twice, (wh, wl), (wm, wm), (wh, wh).  Either
// the numbers are doubled (four moves a product) or the weights (a third of their registers more).
template <bool TWICE> struct PartsA { uint4 q[TWICE ? 3 : 2]; };
constexpr int parts_unit(bool twice) { return twice ? 3072 : 2048; }

template <bool TWICE>
__device__ __forceinline__ PartsA<TWICE> load_parts(__amdgpu_buffer_rsrc_t rsrc, unsigned invalid, int lane, unsigned unit) {
  PartsA<TWICE> w;
#pragma unroll
  for (int t = 0; t < (TWICE ? 3 : 2); ++t) w.q[t] = load_b128(rsrc, invalid | (unsigned)lane * 16u, unit * parts_unit(TWICE) + t * 1024u);
  return w;
}

// Four numbers of a lane, cut: (l, h), and (h, m) or m
template <bool TWICE> struct PartsB { uint4 lh; typename std::conditional<TWICE, uint4, uint2>::type m; };

// + one of the three products, the small ones first
template <int P, bool TWICE>
__device__ __forceinline__ float4_t mma_part(const PartsA<TWICE>& w, const PartsB<TWICE>& x, const float4_t& acc) {
  if constexpr (P == 0) return mfma_split<float>(w.q[0], x.lh, acc);
  else if constexpr (TWICE) return mfma_split<float>(w.q[P], x.m, acc);
  else if constexpr (P == 1) return mfma_split<float>(w.q[1], make_uint4(x.m.x, x.m.y, x.m.x, x.m.y), acc);
  else return mfma_split<float>(w.q[1], make_uint4(x.lh.z, x.lh.w, x.lh.z, x.lh.w), acc);
}

// The wavefront's share of the strip on the fp32 instruction, operands straight from memory; replaces the sums of `mine` lanes.
template <int S, int MB, int R, bool EXP, bool IMG>
__device__ __forceinline__ void mbrow3_slow(const MbArgs& a, const MbAt& at, bool mine, float4_t (&acc)[R][MB]) {
  constexpr int K = 3;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const float lo_e = a.act_e == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f, hi_e = a.act_e == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  const float lo_d = a.act_dw == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f, hi_d = a.act_dw == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  const float* const we = (const float*)a.we_raw;
  const float* const wp = (const float*)a.wp_raw;
  const float* const wd = (const float*)a.wdw;
  const int terms = IMG ? a.Cpi * 9 : a.Cpi;
  // four channels of a row's 16 pixels at column offset s: expanded, or read
  auto row = [&](int c, int iy, int s) -> float4_t {
    const int ix = at.cj * S + s;
    const bool in = (unsigned)iy < (unsigned)a.H;
    if constexpr (!EXP) {
      const bool ok = in & (at.img < a.N) & (ix < a.W) & (c * 16 + at.g4 * 4 < a.Cpe);
      const uint4 q = load_b128(xr, ok ? (unsigned)(((at.img * a.H + iy) * a.W + ix) * a.Cpe + c * 16 + at.g4 * 4) * 4u : kOutOfRange, 0);
      return __builtin_bit_cast(float4_t, q);
    } else {
      float4_t e = load_bias4(a.be, a.Ce, c * 16 + at.g4 * 4);
#pragma unroll 1
      for (int k0 = 0; k0 < terms; k0 += 4) {
        const int k = k0 + at.g4, ch = c * 16 + at.r;
        const float w = k < terms && ch < a.Ce ? we[(long)ch * terms + k] : 0.0f;
        unsigned off = kOutOfRange;
        if constexpr (IMG) {
          const int pc = k / 9, pu = (k - pc * 9) / 3, pv = k - pc * 9 - pu * 3, y = 2 * iy - 1 + pu, x = 2 * ix - 1 + pv;
          if (k < terms && in && at.img < a.N && (unsigned)y < (unsigned)a.Hi && (unsigned)x < (unsigned)a.Wi)
            off = (unsigned)(((at.img * a.Cpi + pc) * a.Hi + y) * a.Wi + x) * 4u;
        } else {
          if (k < terms && in && at.img < a.N && ix < a.W) off = (unsigned)(((at.img * a.H + iy) * a.W + ix) * a.Cpi + k) * 4u;
        }
        e = __builtin_amdgcn_mfma_f32_16x16x4f32(w, __uint_as_float(Elem<float>::load(xr, off, 0)), e, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = in ? __builtin_amdgcn_fmed3f(e[q], lo_e, hi_e) : 0.0f;
      return e;
    }
  };
#pragma unroll 1
  for (int y = 0; y < R; ++y) {
    float4_t sum[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) sum[m] = load_bias4(a.bp, at.wave == 0 ? a.O : 0, at.o0 + m * 16 + 4 * at.g4);
#pragma unroll 1
    for (int c = at.wave; c < a.nchunk; c += at.ks) {
      const int ch = c * 16 + at.g4 * 4;
      float4_t d = load_bias4(a.bdw, a.Ce, ch);
#pragma unroll 1
      for (int u = 0; u < K; ++u) {
        const int iy = at.iy0 + y * S + u;
        const float4_t e0 = row(c, iy, 0), e1 = S == 2 ? row(c, iy, S - 1) : e0;
        auto tap = [&](int v) -> float4_t {
          float4_t w = {0.f, 0.f, 0.f, 0.f};
          if (ch < a.Cpe && (unsigned)(at.cj * S + v - K / 2) < (unsigned)a.W) w = *(const float4_t*)(wd + (u * K + v) * a.Cpe + ch);
          return w;
        };
#pragma unroll
        for (int v = 0; v < K; ++v) {
          const float4_t w = tap(v);
          const int col = v - K / 2;               // from the lane's own (even) column
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float x;
            if (S == 1) x = col < 0 ? row_shift<-1>(e0[q]) : col == 0 ? e0[q] : row_shift<1>(e0[q]);
            else x = col < 0 ? row_shift<-1>(e1[q]) : col == 0 ? e0[q] : e1[q];
            d[q] = fmaf(x, w[q], d[q]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) d[q] = __builtin_amdgcn_fmed3f(d[q], lo_d, hi_d);
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const int o = at.o0 + m * 16 + at.r;
        float4_t w = {0.f, 0.f, 0.f, 0.f};
        if (o < a.O && ch < a.Cpe) w = *(const float4_t*)(wp + (long)o * a.Cpe + ch);
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q], d[q], sum[m], 0, 0, 0);
      }
    }
#pragma unroll
    for (int z = 0; z < R; ++z)
      if (z == y) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[z][m][q] = mine ? sum[m][q] : acc[z][m][q];
      }
  }
}

// A staged pixel (XH units of 8 channels): l, h and m of four channels together, or (the weights not doubled: 16-byte reads) l and h of all
// channels, then m; and what turns the pixels' banks.  Bytes of a pixel; of a row of the staged image, one part.
constexpr int mbrow3_pixel(int xh) { return xh * 48 + (xh & 1 ? 0 : 16); }
constexpr int kImageRow = 72;                  // 33 columns and one more, 4-byte aligned pairs
constexpr int mbrow3_rows(int s, int r) { return (r - 1) * s + 3; }
constexpr int mbrow3_strip_bytes(int s, int xh, int r, bool img) {
  return img ? 3 * 3 * (2 * mbrow3_rows(s, r) + 1) * kImageRow : xh ? mbrow3_rows(s, r) * 16 * s * mbrow3_pixel(xh) : 0;
}

template <int S, int MB, int XH, int R, bool IMG>
__global__ __launch_bounds__(512, 2) void mbrow3_kernel(MbArgs a) {
  constexpr int K = 3, PAD = 1;
  constexpr int ROWS = mbrow3_rows(S, R);   // input rows of a strip
  constexpr int CW = 16 * S;                   // input columns of a strip
  constexpr int XP = mbrow3_pixel(XH);
  constexpr bool EXP = XH > 0;
  constexpr int XR = IMG ? 3 : (XH + 1) / 2;   // rounds of 16 channels (IMG: of four window rows of four columns)
  constexpr int IROWS = 2 * ROWS + 1, IPLANE = 3 * IROWS * kImageRow;     // IMG: rows of a channel, bytes of a part
  constexpr bool TE = mbrow3_twice(S, XH, IMG);   // the expansion's weights are doubled
  constexpr int NE = 3 * XR * S;               // MFMAs that expand a row
  constexpr int FLAGS = mbrow3_strip_bytes(S, XH, R, IMG);

  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const MbAt at = mbrow_at<3, S, MB, R>(a);
  const int t = threadIdx.x, lane = at.lane, ks = at.ks, wave = at.wave, r = at.r, g4 = at.g4, o0 = at.o0;
  const bool two = at.two;
  const int n0 = at.n0, j0 = at.j0, img = at.img, cj = at.cj, iy0 = at.iy0;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t er = make_rsrc(a.we, a.we_bytes);
  const __amdgpu_buffer_rsrc_t pr = make_rsrc(a.wp, a.wp_bytes);
  const __amdgpu_buffer_rsrc_t dr = make_rsrc(a.wdw, a.wdw_bytes);

  unsigned odd = 0;                            // numbers that three parts do not hold: bit 0, or 1 for the second of two images
  const unsigned limit = EXP ? *(const unsigned*)((const unsigned char*)a.we + a.we_bytes) : *(const unsigned*)((const unsigned char*)a.wp + a.wp_bytes);
  if constexpr (EXP) {
    const int nthr = ks * 64;
    unsigned seen = 0, seen2 = 0;
    if constexpr (IMG) {
      // the image under the strip's windows, [part][channel][row][column], zeros outside; two columns an item
      constexpr int ITEMS = 3 * IROWS * 17, U = 8;
      for (int b0 = t; b0 < ITEMS; b0 += nthr * U) {
        uint32_t v[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b0 + u * nthr;
          const int row = idx / 17, ix = 2 * j0 - 1 + 2 * (idx - row * 17);
          const int c = row / IROWS, iy = 2 * iy0 - 1 + row - c * IROWS;
          const bool in = (idx < ITEMS) & (c < a.Cpi) & ((unsigned)iy < (unsigned)a.Hi);
          const unsigned off = (unsigned)(((n0 * a.Cpi + c) * a.Hi + iy) * a.Wi + ix) * 4u;
          v[u][0] = Elem<float>::load(xr, in & ((unsigned)ix < (unsigned)a.Wi) ? off : kOutOfRange, 0);
          v[u][1] = Elem<float>::load(xr, in & ((unsigned)(ix + 1) < (unsigned)a.Wi) ? off + 4u : kOutOfRange, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b0 + u * nthr;
          uint32_t h, m, l;
          split3(v[u][0], v[u][1], h, m, l);
          seen = max_bf16x2(seen, h);
          if (idx < ITEMS) {
            unsigned char* const dst = lds + (idx / 17) * kImageRow + (idx % 17) * 4;
            *(uint32_t*)dst = l; *(uint32_t*)(dst + IPLANE) = h; *(uint32_t*)(dst + 2 * IPLANE) = m;
          }
        }
      }
    } else {
      // the strip's block input: zeros outside the image and past the last channel.  A period of rows is a whole number of items (four
      // channels of a pixel) per lane, which then differ by rows only.
      constexpr int XQ = XH * 2, PER = (S * XH) & 1 ? 2 : 1, SLOTS = PER * S * XH / 2, TURNS = (ROWS + PER - 1) / PER;
      int g_off[SLOTS], l_off[SLOTS], m_off[SLOTS];
      bool live[SLOTS], second[SLOTS];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        const int idx = k * 64 + lane, i = idx / (CW * XQ), rest = idx - i * (CW * XQ), cc = rest / XQ, q = rest - cc * XQ;
        second[k] = two & (cc >= 8 * S);
        const int im = second[k] ? n0 + 1 : n0, ix = two ? cc % (8 * S) : j0 * S + cc;
        live[k] = (ix < a.W) & (im < a.N) & (q * 4 < a.Cpi);
        g_off[k] = (((im * a.H + iy0 + i) * a.W + ix) * a.Cpi + q * 4) * 4;
        l_off[k] = (i * CW + cc) * XP + q * (TE ? 24 : 16);
        m_off[k] = (i * CW + cc) * XP + (TE ? q * 24 + 16 : XH * 32 + q * 8);
      }
      constexpr int U = SLOTS >= 8 ? 1 : 8 / SLOTS;       // turns in flight
      for (int g0 = wave; g0 < TURNS; g0 += ks * U) {
        uint4 v[U][SLOTS];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < SLOTS; ++k) {
            const int row = (g0 + u * ks) * PER, i = PER == 1 ? 0 : (k * 64 + lane) / (CW * XQ);
            const bool in = live[k] & (row + i < ROWS) & ((unsigned)(iy0 + row + i) < (unsigned)a.H);
            v[u][k] = load_b128(xr, in ? (unsigned)(g_off[k] + row * a.W * a.Cpi * 4) : kOutOfRange, 0);
          }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < SLOTS; ++k) {
            const int row = (g0 + u * ks) * PER, i = PER == 1 ? 0 : (k * 64 + lane) / (CW * XQ);
            uint32_t h0, m0, l0, h1, m1, l1;
            split3(v[u][k].x, v[u][k].y, h0, m0, l0); split3(v[u][k].z, v[u][k].w, h1, m1, l1);
            const unsigned top = max_bf16x2(h0 & 0x7fff7fffu, h1);
            seen = max_bf16x2(seen, second[k] ? 0u : top);
            seen2 = max_bf16x2(seen2, second[k] ? top : 0u);
            if (row + i < ROWS) {
              unsigned char* const dst = lds + row * (CW * XP);
              if constexpr (TE) {
                *(uint2*)(dst + l_off[k]) = make_uint2(l0, l1);
                *(uint2*)(dst + l_off[k] + 8) = make_uint2(h0, h1);
              } else {
                *(uint4*)(dst + l_off[k]) = make_uint4(l0, l1, h0, h1);
              }
              *(uint2*)(dst + m_off[k]) = make_uint2(m0, m1);
            }
          }
      }
    }
    auto beyond = [&](unsigned v) -> bool { return ((v & 0xffffu) >= limit) | ((v >> 16) >= limit); };
    odd = (__any(beyond(seen)) ? 1u : 0u) | (__any(beyond(seen2)) ? 2u : 0u);
    if (lane == 0) *(unsigned*)(lds + FLAGS + wave * 4) = odd;
  }

  // depthwise weights: byte offset of the lane's channels, out of range for taps outside the image
  unsigned w_off[K];
#pragma unroll
  for (int v = 0; v < K; ++v) w_off[v] = (unsigned)(cj * S + v - PAD) < (unsigned)a.W ? (unsigned)(g4 * 16) : kOutOfRange;
  // XH = 0: byte offset of the lane's pixel(s) in row 0 of the strip
  int x_base[S];
  if constexpr (!EXP) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int ix = cj * S + s;
      x_base[s] = (img < a.N && ix < a.W) ? (((img * a.H + iy0) * a.W + ix) * a.Cpe + g4 * 4) * 4 : -1;
    }
  }
  const bool x_ok0 = (img < a.N) & (cj * S < a.W), x_ok1 = (img < a.N) & (cj * S + 1 < a.W);

  const float lo_e = a.act_e == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi_e = a.act_e == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  const float lo_d = a.act_dw == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi_d = a.act_dw == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();

  // the projection's bias opens the sums (of the strip's first wavefront)
  float4_t acc[R][MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) acc[0][m] = load_bias4(a.bp, wave == 0 ? a.O : 0, o0 + m * 16 + 4 * g4);
#pragma unroll
  for (int y = 1; y < R; ++y)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[y][m] = acc[0][m];

  uint4 pre[EXP ? 1 : ROWS][S];                // XH = 0: the rows of a chunk, asked for one chunk ahead
  auto load_row = [&](int c, int i) CPRUNE_INLINE {
    const int iy = iy0 + i;
    const bool in = ((unsigned)iy < (unsigned)a.H) & (c * 16 + g4 * 4 < a.Cpe);
#pragma unroll
    for (int s = 0; s < S; ++s)
      pre[EXP ? 0 : i][s] = load_b128(xr, in & (s ? x_ok1 : x_ok0) ? (unsigned)(x_base[s] + i * a.W * a.Cpe * 4) : kOutOfRange,
                                      (unsigned)c * 64u);
  };
  if constexpr (!EXP) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) load_row(wave, i);
  }
  // the lane's operands of input row i, column offset s, round j
  const unsigned char* const xl = lds + S * r * XP + g4 * (TE ? 24 : 16);
  const unsigned char* const xm = lds + S * r * XP + XH * 32 + g4 * 8;
  const int half = XH & 1 ? (g4 & 1) - g4 : 0;       // an odd last round: the lanes past it read (finite) numbers of others, their weights are zero
  int i_off[IMG ? XR : 1];                           // IMG: the lane's window row of a round
  if constexpr (IMG) {
#pragma unroll
    for (int j = 0; j < XR; ++j) {
      const int p = 4 * j + g4, c = p / 3;           // (channel, window row); the weights past the last are zero
      i_off[j] = (p < a.Cpi * 3 ? (c * IROWS + p - c * 3) * kImageRow : 0) + r * 4;
    }
  }
  // (h is read twice: copied it would have to be waited for)
  int again = S * r * XP + g4 * 24;
  asm("" : "+v"(again));
  const unsigned char* const xl2 = lds + again;
  auto operand = [&](int i, int s, int j) CPRUNE_INLINE -> PartsB<TE> {
    PartsB<TE> x;
    if constexpr (IMG) {
      const int off = i_off[j] + 2 * i * kImageRow;
      auto word = [&](int part) -> uint2 { return make_uint2(*(const uint32_t*)(lds + off + part * IPLANE), *(const uint32_t*)(lds + off + part * IPLANE + 4)); };
      const uint2 l = word(0), h = word(1);
      x.lh = make_uint4(l.x, l.y, h.x, h.y);
      x.m = word(2);
    } else {
      const int last = (XH & 1) && j == XR - 1 ? half : 0, px = (i * CW + s) * XP;
      if constexpr (TE) {
        const int off = px + j * 96 + last * 24;
        const uint2 *const p = (const uint2*)(xl + off), *const p2 = (const uint2*)(xl2 + off);
        const uint2 l = p[0], h = p[1], h2 = p2[1], m = p2[2];
        x.lh = make_uint4(l.x, l.y, h.x, h.y);
        x.m = make_uint4(h2.x, h2.y, m.x, m.y);
      } else {
        x.lh = *(const uint4*)(xl + px + j * 64 + last * 16);
        x.m = *(const uint2*)(xm + px + j * 32 + last * 8);
      }
    }
    return x;
  };
  // Weights of one chunk of 16 expanded channels, carried in registers: those of the next are asked for as soon as the last row
  // has used the present ones.
  uint4 wq[K][K];
  PartsA<TE> ae[EXP ? XR : 1];
  PartsA<false> ap[MB];
  float4_t be, bd;
  auto load_taps = [&](int c, int u) CPRUNE_INLINE {
    const unsigned inval = (unsigned)(c * 16 + g4 * 4 >= a.Cpe) << 31;
#pragma unroll
    for (int v = 0; v < K; ++v) wq[u][v] = load_b128(dr, w_off[v] | inval, (unsigned)(((u * K + v) * a.Cpe + c * 16) * 4));
  };
  auto load_expand = [&](int c) CPRUNE_INLINE {
    if constexpr (EXP) {
      const unsigned off = c < a.nchunk ? 0u : kOutOfRange;
#pragma unroll
      for (int j = 0; j < XR; ++j) ae[j] = load_parts<TE>(er, off, lane, (unsigned)(c * XR + j));
      be = load_bias4(a.be, a.Ce, c * 16 + g4 * 4);
    }
  };
  auto load_project = [&](int c) CPRUNE_INLINE {
    const unsigned off = c < a.nchunk ? 0u : kOutOfRange;
#pragma unroll
    for (int m = 0; m < MB; ++m)
      ap[m] = load_parts<false>(pr, o0 + m * 16 < a.O ? off : kOutOfRange, lane, (unsigned)((blockIdx.y * MB + m) * a.nchunk + c));
  };
  // operands of the rounds ahead: a row's, or (registers) the next three or four
  constexpr int SX = EXP ? S * XR : 1, RING = SX <= 4 ? SX : SX % 4 ? 3 : 4;
  static_assert(SX % RING == 0, "whole turns a row");
  PartsB<TE> xb[RING];
  uint32_t top_d = 0;                          // XH = 0: the largest depthwise result (of negative ones any counts as larger)
  load_expand(wave);
  bd = load_bias4(a.bdw, a.Ce, wave * 16 + g4 * 4);
#pragma unroll
  for (int u = 0; u < K; ++u) load_taps(wave, u);
  load_project(wave);
  if constexpr (EXP) {
    __syncthreads();
    odd = 0;
    for (int w = 0; w < ks; ++w) odd |= *(const unsigned*)(lds + FLAGS + w * 4);
    odd = __builtin_amdgcn_readfirstlane(odd);
#pragma unroll
    for (int f = 0; f < RING; ++f) xb[f] = operand(0, f / XR, f % XR);
  }

  for (int c = wave; c < a.nchunk; c += ks) {
    const int cn = c + ks;
    float4_t wd[K][K];
#pragma unroll
    for (int u = 0; u < K; ++u)
#pragma unroll
      for (int v = 0; v < K; ++v) wd[u][v] = __builtin_bit_cast(float4_t, wq[u][v]);
    float4_t dacc[R];
#pragma unroll
    for (int y = 0; y < R; ++y) dacc[y] = bd;
    bd = load_bias4(a.bdw, a.Ce, cn * 16 + g4 * 4);
    float4_t e[S];
    PartsB<false> fin = {};                    // the finished output row, cut
    // Step i: row i is expanded while the row before it is multiplied into its output rows; the output row that this completes is
    // cut while the one that the step before completed is projected; the operands of row i + 1 are read.  All of it is written in the
    // order it is to run in, a few vector operations behind each MFMA: left alone the compiler puts the MFMAs of a sum, which wait
    // for each other, in a row, and reads from LDS right before their use.
    each<ROWS + 2>([&](auto i_tag) CPRUNE_INLINE {
      constexpr int i = decltype(i_tag)::value, ir = i - 1;            // ir: the row that is multiplied
      constexpr int done = ir - (K - 1), y_done = done / S;            // output row it completes
      constexpr bool dw = i > 0 && i <= ROWS, completes = dw && done >= 0 && done % S == 0;
      constexpr int was = done - 1, y_was = was / S;                   // ... that the step before completed
      constexpr bool expand = EXP && i < ROWS, project = was >= 0 && was % S == 0;
      constexpr int TP = project ? 3 * MB : 0, T = TP + (expand ? NE : 0);        // MFMAs of the step
      PartsB<false> nf = fin;
      // the step's vector operations in units, a window row of a channel, then the cut of two channels: those behind MFMA t
      constexpr int NU = 4 * K + 2;
      auto work = [&](auto t_tag) CPRUNE_INLINE {
        constexpr int t = decltype(t_tag)::value, Q = T ? T : 1;
        each_from<(t * NU + Q - 1) / Q, ((t + 1) * NU + Q - 1) / Q>([&](auto n_tag) CPRUNE_INLINE {
          constexpr int n = decltype(n_tag)::value;
          if constexpr (n < 4 * K) {
            constexpr int q = n / K, u = n % K, y = (ir - u) / S;
            if constexpr (dw && (ir - u) % S == 0 && ir >= u && y < R) {
              float d = dacc[y][q];
              if constexpr (S == 1) {
                d = fmaf(row_shift<-1>(e[0][q]), wd[u][PAD - 1][q], d);
                d = fmaf(e[0][q], wd[u][PAD][q], d);
                d = fmaf(row_shift<1>(e[0][q]), wd[u][PAD + 1][q], d);
              } else {
                d = fmaf(row_shift<-1>(e[S - 1][q]), wd[u][PAD - 1][q], d);
                d = fmaf(e[0][q], wd[u][PAD][q], d);
                d = fmaf(e[S - 1][q], wd[u][PAD + 1][q], d);
              }
              dacc[y][q] = d;
            }
          } else if constexpr (completes) {
            constexpr int p = n - 4 * K;
            uint32_t h, m, l;
            const uint32_t d0 = __float_as_uint(__builtin_amdgcn_fmed3f(dacc[y_done][2 * p], lo_d, hi_d));
            const uint32_t d1 = __float_as_uint(__builtin_amdgcn_fmed3f(dacc[y_done][2 * p + 1], lo_d, hi_d));
            split3(d0, d1, h, m, l);
            if constexpr (!EXP) top_d = max(max(top_d, d0), d1);
            if constexpr (p == 0) { nf.lh.x = l; nf.lh.z = h; nf.m.x = m; }
            else { nf.lh.y = l; nf.lh.w = h; nf.m.y = m; }
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      };
      __builtin_amdgcn_sched_barrier(0);
      // up to four filter blocks product by product, more (registers) block by block, a block's sum added while the next one's is multiplied
      constexpr bool BY_BLOCK = MB > 4;
      float4_t sum[BY_BLOCK ? 2 : MB];
      if constexpr (project) {
        each<3 * MB>([&](auto t_tag) CPRUNE_INLINE {
          constexpr int t = decltype(t_tag)::value, m = BY_BLOCK ? t / 3 : t % MB, p = BY_BLOCK ? t % 3 : t / MB, z = BY_BLOCK ? m & 1 : m;
          if constexpr (p == 0) sum[z] = (float4_t){0.f, 0.f, 0.f, 0.f};
          sum[z] = mma_part<p>(ap[m], fin, sum[z]);
          if constexpr (BY_BLOCK && p == 1 && m > 0) acc[y_was][m - 1] += sum[(m - 1) & 1];
          work(t_tag);
        });
      }
      float4_t en[S];
      if constexpr (expand) {
        const bool in = (unsigned)(iy0 + i) < (unsigned)a.H;
        const float lo = in ? lo_e : 0.0f, hi = in ? hi_e : 0.0f;      // a row outside the image: zeros
        constexpr int nxt = i + 1 < ROWS ? i + 1 : 0;                  // (behind the last row the first one's operands, for the next chunk)
        each<S * XR>([&](auto sj) CPRUNE_INLINE {
          constexpr int s = sj.value / XR, j = sj.value % XR;
          if constexpr (j == 0) en[s] = be;
          each<3>([&](auto p) CPRUNE_INLINE {
            en[s] = mma_part<p.value>(ae[j], xb[sj.value % RING], en[s]);
            if constexpr (p.value == 2) {
              constexpr int f = (sj.value + RING) % SX;
              xb[sj.value % RING] = operand(sj.value + RING < SX ? i : nxt, f / XR, f % XR);
            }
            work(std::integral_constant<int, TP + sj.value * 3 + p.value>{});
          });
        });
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int q = 0; q < 4; ++q) en[s][q] = __builtin_amdgcn_fmed3f(en[s][q], lo, hi);
      } else if constexpr (i < ROWS) {
#pragma unroll
        for (int s = 0; s < S; ++s) en[s] = __builtin_bit_cast(float4_t, pre[i][s]);
        load_row(cn, i);                       // (past the last chunk: zeros, without a branch)
      }
      if constexpr (T == 0) work(std::integral_constant<int, 0>{});
      if constexpr (project) {
#pragma unroll
        for (int m = BY_BLOCK ? MB - 1 : 0; m < MB; ++m) acc[y_was][m] += sum[BY_BLOCK ? m & 1 : m];
      }
      fin = nf;
      if constexpr (i < ROWS) {
#pragma unroll
        for (int s = 0; s < S; ++s) e[s] = en[s];
      }
      if constexpr (i == ROWS - 1) load_expand(cn);
      if constexpr (ir >= (R - 1) * S && ir < (R - 1) * S + K) load_taps(cn, ir - (R - 1) * S);
      if constexpr (i == ROWS + 1) load_project(cn);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
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
  const bool bad = top >= kInf || low < kSmall - 1 || (!EXP && top_d >= limit), second = two && r >= 8;
  odd |= (__any(bad && !second) ? 1u : 0u) | (__any(bad && second) ? 2u : 0u);
  if (odd) mbrow3_slow<S, MB, R, EXP, IMG>(a, at, odd >> (second ? 1 : 0) & 1u, acc);

  mbrow_finish<float, R, MB>(a, at, lds, acc);
}

// LDS of a work-group: the strip's input and a word per wavefront, later the sums of `slots` wavefronts
template <int S, int MB, int XH, int R, bool IMG>
inline int launch_mbrow3_rows(dim3 grid, int ks, hipStream_t s, MbArgs a) {
  constexpr int strip = mbrow3_strip_bytes(S, XH, R, IMG) + (XH ? 32 : 0);
  constexpr int slot = R * MB * 1024;
  static_assert(strip <= 160 * 1024 && 4 * slot <= 160 * 1024, "LDS budget");
  a.slots = ks > 4 ? 4 : ks;
  const int red = ks > 1 ? a.slots * slot : 0;
  const int bytes = strip > red ? strip : red;
  if (bytes > 65536) {   // more than the default 64 KiB has to be asked for once
    static std::atomic<bool> raised{false};
    if (!raised.load(std::memory_order_relaxed)) {
      CPRUNE_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&mbrow3_kernel<S, MB, XH, R, IMG>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
      raised.store(true, std::memory_order_relaxed);
    }
  }
  hipLaunchKernelGGL((mbrow3_kernel<S, MB, XH, R, IMG>), grid, dim3(64 * ks), bytes, s, a);
  return CPRUNE_OK;
}

template <int S, int MB, int XH, bool IMG = false>
inline int launch_mbrow3_one(int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  constexpr int R0 = mbrow3_strip_rows(S, MB, XH, 0), R1 = mbrow3_strip_rows(S, MB, XH, 1);
  if (R0 == R1 || !low) return launch_mbrow3_rows<S, MB, XH, R0, IMG>(grid, ks, s, a);
  return launch_mbrow3_rows<S, MB, XH, R1, IMG>(grid, ks, s, a);
}

// (MB, XH) pairs that are built; XH = 0: depthwise + projection only.  mbrow_form picks one of them (tiles of 128 filters: mbrow_kernel.hpp).
template <int S>
inline int launch_mbrow3_ks(int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
#define CPRUNE_MBROW(MB_, XH_) \
  if (mb == MB_ && xh == XH_) return launch_mbrow3_one<S, MB_, XH_>(low, grid, ks, s, a);
  CPRUNE_MBROW(1, 0) CPRUNE_MBROW(2, 0) CPRUNE_MBROW(4, 0) CPRUNE_MBROW(6, 0)
  CPRUNE_MBROW(2, 2) CPRUNE_MBROW(2, 3) CPRUNE_MBROW(2, 4)
  CPRUNE_MBROW(4, 4) CPRUNE_MBROW(4, 8) CPRUNE_MBROW(6, 8) CPRUNE_MBROW(6, 12)
#undef CPRUNE_MBROW
  return CPRUNE_ERR_UNSUPPORTED;
}

// (a template, so that its kernels are compiled where it is called)
template <typename T>
inline int launch_mbrow3(int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  if (a.Hi > 0) {      // the image form: 9 (channel, window row) pairs of four columns in three rounds
    if (stride != 1) return CPRUNE_ERR_UNSUPPORTED;
    if (mb == 1) return launch_mbrow3_one<1, 1, 4, true>(low, grid, ks, s, a);
    if (mb == 2) return launch_mbrow3_one<1, 2, 4, true>(low, grid, ks, s, a);
    return CPRUNE_ERR_UNSUPPORTED;
  }
  return stride == 1 ? launch_mbrow3_ks<1>(mb, xh, low, grid, ks, s, a) : launch_mbrow3_ks<2>(mb, xh, low, grid, ks, s, a);
}

}  // namespace cprune
