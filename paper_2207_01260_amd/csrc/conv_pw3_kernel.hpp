// 1x1 convolution, channels-last, stride 1 or 2, on the 16-bit matrix cores: an fp32 number cut into three bf16 parts, six of the
// nine products multiplied (conv_split_kernel.hpp has the error and the range of that), 16-bit data as it is.
//
// A matrix product of short reductions (three to thirty rounds of 32 channels) on few pixels: what the split kernel for any window
// loses on it is two barriers, a table walk and a wait for the chunk per round.  Here a work-group of four wavefronts owns NB * 16 pixels
// and up to 4 * MB 16-filter blocks, dealt evenly.  A chunk of two rounds (16-bit data: four) is cut once, while it is stored to LDS ([round][part][pixel][64
// bytes]: every store and operand read is 1 KiB of consecutive memory), and read by all four wavefronts; there are two buffers,
// so one barrier per chunk, and the chunk behind them is on its way in registers.  Weights, packed in whole rounds
// (launch_pack_split), go from memory to registers a round ahead.  DEEP: two chunks on their way and weights a chunk ahead, for long
// reductions of few work-groups, which wait for nothing else; the registers cost a wavefront or two per SIMD, and a layer of a
// chunk or two gains nothing from them.
//
// Measured, the best other kernel / this one (us): 96 -> 385 at 14x14, batch 64, 19.7 / 12.1; 160 -> 829 at 7x7 16.0 / 9.5; 829 -> 320 at
// 7x7 29 / 15, 320 -> 1280 31 / 18 (143 TFLOP/s); stride 2, batch 32: 64 -> 128 at 56x56 12.1 / 7.7, 256 -> 512 at 14x14 10.6 / 6.5; 90
// random layers of 0.01-4 GFLOP, timed choice before / now 1.29 times on average, untimed 1.50.  Deep or not: 739 -> 58 at 28x28
// stride 2, batch 30, 9.6 / 12.3; 29 -> 232 at 56x56, batch 28, 32.0 / 23.8.  bf16, 80 random layers: timed choice 1.23 times as fast as before,
// untimed 1.44 (865 -> 78 at 56x56 stride 2, batch 28, 12 us; 16 -> 292 at 56x56, batch 55, stays on the short-reduction kernel, 35.5 / 40.9).  What bounds it: launch, first loads and stores (some 4 us);
// 96 -> 385 moves 24 MB, 5 us at the copy rate.  Counters, fp32: matrix pipes busy 16-26 %, 320 -> 1280 44, wavefronts waiting for memory or the
// barrier 37-60 % of their cycles; bf16 5 and 59.
#pragma once
#include "conv_rows_s2_kernel.hpp"

namespace cprune {

struct Pw3Args {
  const void* x;        // [n][h][w][cp]
  const void* w;        // launch_pack_split, whole rounds
  const void* w_raw;    // [o][cp]
  const float* bias;
  const void* res;
  void* y;              // [p][cop]
  int P, H, W, Ho, Wo, O, Cp, Cop;
  int stride;
  int tiles_m, blk_base, blk_rem;      // as SplitArgs
  int rounds;
  unsigned x_bytes, w_bytes, w_raw_bytes, y_bytes;
  unsigned magic_m, magic_wo, magic_ho;
  int act;
};

// Variants: id, 16-filter blocks per wavefront, 16-pixel blocks of a work-group, deep (16-bit data: always)
#define CPRUNE_PW3_LIST(X) \
  X(0, 1, 2, 0) X(1, 2, 2, 0) X(2, 1, 4, 0) X(3, 2, 4, 0) X(4, 1, 2, 1) X(5, 2, 2, 1) \
  X(6, 1, 4, 1) X(7, 2, 4, 1)

constexpr int kNumPw3 = 8;      // (fp32: the first six)

template <typename T, int MB, int NB, bool DEEP>
__global__ __launch_bounds__(256, 2) void conv_pw3_kernel(Pw3Args a) {
  constexpr int ES = (int)sizeof(T), P = SplitParts<T>::value, NQ = ES / 2;
  constexpr int RC = P == 3 ? 2 : 4;           // rounds of a chunk
  constexpr int PT = NB * 16;
  constexpr int NI = PT * 4 * RC / 256;        // staging items (8 channels of a pixel) per thread
  constexpr int PART = PT * 64, ROUND = P * PART, BUF = RC * ROUND;
  static_assert(NI >= 1 && NI * 256 == PT * 4 * RC, "staging items");
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * BUF];

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
  const int tile_p = (int)fast_div((unsigned)tile, a.magic_m), tile_m = tile - tile_p * a.tiles_m;
  const SplitShare share = split_share(tile_m, (wave + tile_p) & 3, 4, a.blk_base, a.blk_rem);   // (the long shares rotate)
  const int nblk = share.count, o0 = share.first * 16;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);
  // byte offset of pixel p's channels
  auto pixel = [&](int p) CPRUNE_INLINE -> unsigned {
    int at = p;
    if (a.stride != 1) {
      const int q = (int)fast_div((unsigned)p, a.magic_wo), n = (int)fast_div((unsigned)q, a.magic_ho);
      at = (n * a.H + (q - n * a.Ho) * a.stride) * a.W + (p - q * a.Wo) * a.stride;
    }
    return p < a.P ? (unsigned)(at * a.Cp) * ES : kOutOfRange;
  };

  // ---- staging ----
  unsigned x_off[NI];
  int x_ch[NI], x_lds[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int idx = t + 256 * j, g = idx & 3, px = (idx >> 2) % PT, rd = idx / (4 * PT);
    x_off[j] = pixel(tile_p * PT + px) + (unsigned)(rd * 32 + g * 8) * ES;
    x_ch[j] = rd * 32 + g * 8;
    x_lds[j] = rd * ROUND + px * 64 + g * 16;
  }
  auto gload = [&](int c, RawRow<T> (&raw)[NI]) CPRUNE_INLINE {
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < NQ; ++e)
        raw[j].q[e] = load_b128(xr, c * (RC * 32) + x_ch[j] + e * (16 / ES) < a.Cp ? x_off[j] + (unsigned)(c * (RC * 32 * ES) + e * 16) : kOutOfRange, 0);
  };
  auto lds_store = [&](int buf, const RawRow<T> (&raw)[NI]) CPRUNE_INLINE {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const Operand<T> v = to_operand(raw[j]);
#pragma unroll
      for (int p = 0; p < P; ++p) *(uint4*)(smem + buf * BUF + x_lds[j] + p * PART) = v.p[p];
    }
  };

  const unsigned w_blk = (unsigned)a.rounds * (P * 1024u);
  const unsigned w_base = (unsigned)split_weight_block(share.first, a.blk_base * a.tiles_m + a.blk_rem) * w_blk;
  auto load_weights = [&](auto mbc, int round, uint4 (&f)[MB][P]) CPRUNE_INLINE {
    const unsigned at = w_base + (unsigned)split_weight_round(round, a.rounds) * (P * 1024u);
#pragma unroll
    for (int i = 0; i < decltype(mbc)::value; ++i)
#pragma unroll
      for (int p = 0; p < P; ++p) f[i][p] = load_b128(wr, (unsigned)lane * 16u + p * 1024u, at + i * w_blk);
  };

  float4_t big[MB][NB], small[P == 3 ? MB : 1][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) big[i][j] = small[P == 3 ? i : 0][j] = (float4_t){0.f, 0.f, 0.f, 0.f};
  const unsigned char* const b_at = smem + r * 64 + g4 * 16;
  // consecutive MFMAs on different sums: the scheduler by itself issues each block's chain back to back
  auto multiply = [&](auto mbc, const uint4 (&f)[MB][P], int off) CPRUNE_INLINE {
    constexpr int MBC = decltype(mbc)::value;
    constexpr int JS = 2;
#pragma unroll
    for (int j0 = 0; j0 < NB; j0 += JS) {
      uint4 b[JS][P];
#pragma unroll
      for (int j = 0; j < JS; ++j)
#pragma unroll
        for (int p = 0; p < P; ++p) b[j][p] = *(const uint4*)(b_at + off + p * PART + (j0 + j) * 1024);
      auto term = [&](int pw, int px) CPRUNE_INLINE {
#pragma unroll
        for (int j = 0; j < JS; ++j)
#pragma unroll
          for (int i = 0; i < MBC; ++i) {
            float4_t& d = pw + px == 0 ? big[i][j0 + j] : small[P == 3 ? i : 0][j0 + j];
            d = mfma_split<T>(f[i][pw], b[j][px], d);
          }
      };
      if constexpr (P == 3) {
        term(0, 2); term(0, 0); term(2, 0); term(1, 1); term(0, 1); term(1, 0);
      } else {
        term(0, 0);
      }
    }
  };

  const int nchunk = (a.rounds + RC - 1) / RC;
  auto main_loop = [&](auto mbc) CPRUNE_INLINE {
    uint4 w0[DEEP ? RC : 1][MB][P], w1[DEEP ? RC : 1][MB][P];
    RawRow<T> raw0[NI], raw1[NI];
    if constexpr (DEEP) {
      gload(0, raw1);
#pragma unroll
      for (int q = 0; q < RC; ++q) load_weights(mbc, q, w0[q]);
      gload(1, raw0);                          // (past the last channel: zeros)
      lds_store(0, raw1);
      gload(2, raw1);
      __syncthreads();
      // chunk c, its weights at hand; the raw chunk c + 1 goes to LDS, its place to chunk c + 3
      auto step = [&](int c, const uint4 (&w)[RC][MB][P], uint4 (&next)[RC][MB][P], RawRow<T> (&raw)[NI]) CPRUNE_INLINE {
        const int at = (c & 1) * BUF;
#pragma unroll
        for (int q = 0; q < RC; ++q) load_weights(mbc, RC * c + RC + q, next[q]);
#pragma unroll
        for (int q = 0; q < RC; ++q)
          if (q == 0 || RC * c + q < a.rounds) multiply(mbc, w[q], at + q * ROUND);
        if (c + 1 < nchunk) {
          lds_store((c + 1) & 1, raw);
          gload(c + 3, raw);
          __syncthreads();
        }
      };
      for (int c = 0; c < nchunk; c += 2) {
        step(c, w0, w1, raw0);
        if (c + 1 < nchunk) step(c + 1, w1, w0, raw1);
      }
    } else {
      gload(0, raw0);
      load_weights(mbc, 0, w0[0]);
      lds_store(0, raw0);
      gload(1, raw0);
      __syncthreads();
      for (int c = 0; c < nchunk; ++c) {
        const int at = (c & 1) * BUF;
        load_weights(mbc, RC * c + 1, w1[0]);
        multiply(mbc, w0[0], at);
        load_weights(mbc, RC * c + 2, w0[0]);
        if (RC * c + 1 < a.rounds) multiply(mbc, w1[0], at + ROUND);
        if (c + 1 < nchunk) {
          lds_store((c + 1) & 1, raw0);
          gload(c + 2, raw0);
          __syncthreads();
        }
      }
    }
  };
  if (MB >= 2 && nblk >= 2) main_loop(std::integral_constant<int, MB >= 2 ? 2 : 1>{});
  else main_loop(std::integral_constant<int, 1>{});        // (a wavefront without a block stages, and stores nothing)
  if (nblk == 0) return;

  float4_t bias[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) bias[i] = load_bias4(a.bias, i < nblk ? a.O : 0, o0 + i * 16 + 4 * g4);
  if constexpr (P == 3) {
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) big[i][j] += small[i][j];

  // data that three parts do not hold shows in the sums (see conv_split_kernel): then once more on the fp32 instruction
  constexpr uint32_t kInf = 0x7f800000u, kSmall = (127u - 50u) << 23;
  uint32_t odd = 0;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) odd = max(odd, (__float_as_uint(big[i][j][q]) << 1) - (kSmall << 1));
  if (__any(odd >= (kInf - kSmall) << 1)) {
    uint32_t top = 0, low = ~0u;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t mag = __float_as_uint(big[i][j][q]) & 0x7fffffffu;
          top = max(top, mag);
          low = min(low, mag - 1);      // (zero goes to the other end)
        }
    if (__any(top >= kInf || low < kSmall - 1)) {
      const __amdgpu_buffer_rsrc_t ww = make_rsrc(a.w_raw, a.w_raw_bytes);
      unsigned px[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) px[j] = pixel(tile_p * PT + j * 16 + r);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) big[i][j] = (float4_t){0.f, 0.f, 0.f, 0.f};
      for (int c0 = 0; c0 < a.Cp; c0 += 4) {       // (the stride is a multiple of four channels)
        const unsigned at = (unsigned)(c0 + g4) * 4u;
        float wv[MB], xv[NB];
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const int o = o0 + i * 16 + r;
          wv[i] = __uint_as_float(Elem<float>::load(ww, (i < nblk) & (o < a.O) ? (unsigned)(o * a.Cp) * 4u + at : kOutOfRange, 0));
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) xv[j] = __uint_as_float(Elem<float>::load(xr, px[j] == kOutOfRange ? kOutOfRange : px[j] + at, 0));
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) big[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i], xv[j], big[i][j], 0, 0, 0);
      }
    }
  }
  }

  // bias, shortcut (a block's loads before its stores), activation, four filters of a pixel per store
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res, a.res ? a.y_bytes : 0u);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int p = tile_p * PT + j * 16 + r;
    unsigned off[MB];
    float4_t s[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int o = o0 + i * 16 + 4 * g4;
      off[i] = (p < a.P) & (i < nblk) & (o < a.Cop) ? (unsigned)(p * a.Cop + o) * ES : kOutOfRange;
      s[i] = big[i][j] + bias[i];
      if (a.res) {
        if constexpr (ES == 4) {
          const uint4 q = load_b128(rr, off[i], 0);
          s[i] += __builtin_bit_cast(float4_t, q);
        } else {
          s[i] += widen4<T>(load_b64(rr, off[i], 0));
        }
      }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      if (off[i] == kOutOfRange) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) s[i][q] = apply_act(s[i][q], a.act);
      if constexpr (ES == 4) *(float4_t*)((char*)a.y + off[i]) = s[i];
      else *(uint2*)((char*)a.y + off[i]) = narrow4<T>(s[i]);
    }
  }
}

template <typename T>
inline int launch_pw3(int id, dim3 grid, hipStream_t s, const Pw3Args& a) {
#define CPRUNE_PW3_CASE(ID, MB_, NB_, DEEP_) \
  case ID:                                                                                                                 \
    if constexpr (sizeof(T) == 4 ? !(NB_ == 4 && DEEP_) : DEEP_ != 0) {                                                  \
      hipLaunchKernelGGL((conv_pw3_kernel<T, MB_, NB_, DEEP_ != 0>), grid, dim3(256), 0, s, a);                          \
      return CPRUNE_OK;                                                                                                    \
    }                                                                                                                      \
    break;
  switch (id) { CPRUNE_PW3_LIST(CPRUNE_PW3_CASE) default: break; }
#undef CPRUNE_PW3_CASE
  return CPRUNE_ERR_UNSUPPORTED;
}

int launch_conv_pw3_f32(int id, dim3 grid, hipStream_t s, const Pw3Args& a);
int launch_conv_pw3_f16(int id, dim3 grid, hipStream_t s, const Pw3Args& a);
int launch_conv_pw3_bf16(int id, dim3 grid, hipStream_t s, const Pw3Args& a);

}  // namespace cprune
