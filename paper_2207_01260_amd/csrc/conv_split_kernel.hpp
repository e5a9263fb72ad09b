// Dense convolution, any window up to 7x7 and stride up to 2, on the 16-bit matrix cores for fp32 data too.
//
// v_mfma_f32_16x16x4_f32 multiplies at 157 TFLOP/s, v_mfma_f32_16x16x32_bf16 at 2.5 PFLOP/s.  An fp32 number of ordinary
// size is exactly the sum of three bf16 numbers (its 24 significant bits cut into three runs of eight), so an fp32 product
// is the sum of nine bf16 products, each exact in fp32; the three smallest are left out and the six others accumulated in
// fp32, at 2.7 times the fp32 instruction's rate.  Weights are cut and packed once (launch_pack_split), activations while
// they are staged into LDS (some six vector operations per element, against 9 x 6 multiplies per filter).  Both are cut
// by rounding to nearest: a second part is then at most 2^-8 of the number and a third 2^-16, what is left out at most 2^-23
// of a product (5.7e-9 in the 2-norm; by truncation 1.8e-8), and it has no sign of its own, so it does not add up over
// the layers of a network.  A sum is rounded twice per 32 terms, by the fp32 instruction at every term: at 16 terms the
// error is 3.3e-8 against 7.5e-8, at 24 3.7e-8 against 9.0e-8, at 2304 0.2 to 0.4 of it; a single product is 2.6e-8 off where
// one rounding is 2.5e-8, so sums of fewer than 16 terms stay on the fp32 instruction (split_supports).
// What three bf16 numbers cannot hold (infinities, numbers that round to one, numbers below 2^-110 whose last part falls
// off the end of the range) shows in the sums: such a sum is not finite, or too small for what was lost to be below its own
// last place.  A wavefront that finds one multiplies its block again with the fp32 instruction (`again` below).
// 16-bit data runs the same kernel with one part per number.
//
// A work-group owns MT = WM * MB * 16 filters and a block of th x tw pixels of ni images, at most PT = WN * NB * 16
// pixels; which block is the host's choice per map (split_plan): pixels are numbered by division, so the block need
// not be a power of two and an odd map wastes little.  Per chunk of 32 input channels the patch the block's windows
// touch is staged once ([pixel][8-channel group][part][16 bytes], 16 bytes of pad per pixel so that the pixels of a
// read rotate through the banks).  The reduction of a chunk is a list of (tap, 8-channel group) units, four per MFMA
// round, one per 16-lane quarter; the LDS offset of a unit comes from a table in LDS.  A last chunk of one to three
// groups therefore costs no padded rounds: channel counts cost in steps of 8, not 32.  Weight fragments go straight
// from memory to registers, packed in the order of the rounds (a wavefront's load is 1 KiB of consecutive memory), one
// round ahead; the next chunk's activations are in flight while this one is multiplied.  WK wavefronts can share one
// block and take every WK-th round (few blocks, long reductions); their sums meet in LDS at the end, in order.
//
// Measured, fp32 channels-last, best variant against the best fp32-instruction kernel: 56 -> 56 at 32x32, batch 64, 42.4
// -> 26.5 us; 40 -> 64 at 56x56, batch 32, 54.1 -> 35.0 us; 128 -> 85 at 28x28 56.8 -> 37.0 us; 512 -> 411 at 7x7
// 72.2 -> 52.0 us; 360 -> 360 at 4x4, batch 64, 25.4 -> 26.2 us (the independent-wavefront kernel stays there);
// stride 2, 128 -> 173 at 28x28, 34.8 -> 25.1 us.  What bounds it:
// of the 32 us of 85 -> 128 at 28x28 the matrix pipes need 14; operand reads, weight reads and staging cost 5-8 %
// each when left out alone; 8 us are launch, first loads and stores, which the two or three work-groups of a unit,
// started together, do not hide from each other.
#pragma once
#include <atomic>
#include "conv_nhwc_kernel.hpp"
#include "split_index.hpp"

// every lambda of the kernel: one that is not inlined takes the arrays it captures into scratch memory
#define CPRUNE_INLINE __attribute__((always_inline))

namespace cprune {

struct SplitArgs {
  const void* x;        // NCHW or channels-last
  const void* w;        // packed by launch_pack_split
  const void* w_raw;    // fp32: the weights as they are, [o][c][taps] or channels-last [o][taps][C]
  const float* bias;
  const void* res;
  void* y;              // the layout of x
  int N, H, W, Ho, Wo, O, C;   // C: input channels (channels-last: their stride, pad channels zero)
  int Cop;              // channels-last: channel stride of y
  int stride, pad, kw, taps;
  int th, tw, ni, ph, pw;      // pixel block of a work-group; its input patch
  int tiles_n, tiles_y, tiles_x, tiles_m;
  int blk_base, blk_rem;       // 16-filter blocks per filter tile: blk_base, and one more in the first blk_rem
  int nfull, rounds_last, rtot;  // chunks of 32 channels; rounds of the last, partial one (0: none); rounds in all
  int groups_last;               // 8-channel groups of the last chunk
  unsigned x_bytes, w_bytes, w_raw_bytes;
  unsigned magic_s, magic_m, magic_x, magic_y;      // tile decode (as PatchArgs)
  unsigned magic_pp, magic_pw;                      // patch pixel -> (image, row, column)
  unsigned magic_thw, magic_tw;                     // output pixel of the block -> (image, row, column); pooled: windows
  unsigned magic_np;                                // staging item -> (group, patch pixel), NCHW
  int m_major, act, pool, vec_out;
  int off_patch;        // LDS offset of the patch behind the tables
};

constexpr int kSplitTab = 128;   // LDS: 64 bytes of zeros, 64 that take the writes of threads without an item, then
                                 // the two offset tables (full chunk, last chunk), then the patch

template <typename T> struct SplitParts { static constexpr int value = sizeof(T) == 4 ? 3 : 1; };

typedef float float2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// two numbers as three pairs of bf16 numbers, each the nearest to what the ones before it leave
__device__ __forceinline__ void split3(uint32_t u0, uint32_t u1, uint32_t& h, uint32_t& m, uint32_t& l) {
  const float2_t x = {__uint_as_float(u0), __uint_as_float(u1)};
  h = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
  const float r0 = x[0] - __uint_as_float(h << 16), r1 = x[1] - __uint_as_float(h & 0xffff0000u);
  m = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t){r0, r1}, bf16x2_t));
  const float s0 = r0 - __uint_as_float(m << 16), s1 = r1 - __uint_as_float(m & 0xffff0000u);
  l = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2_t){s0, s1}, bf16x2_t));
}

template <typename T>
__device__ __forceinline__ float4_t mfma_split(const uint4& a, const uint4& b, const float4_t& c) {
  if constexpr (std::is_same<T, _Float16>::value)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

template <typename T, bool NCHW, int WM, int WN, int WK, int MB, int NB, int NIB>
__global__ __launch_bounds__(256, MB * NB <= 4 && NIB <= 4 ? 3 : 2) void conv_split_kernel(SplitArgs a) {
  constexpr int ES = (int)sizeof(T);
  constexpr int P = SplitParts<T>::value;
  constexpr int UNIT = P * 16;            // bytes of one 8-channel group of a pixel
  constexpr int BROW = 4 * UNIT + 16;
  constexpr int NV = ES == 4 ? 8 : 4;     // dwords of a staged item held in registers
  static_assert(WM * WN * WK == 4, "four wavefronts");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  int* const tab = (int*)(smem + kSplitTab);

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wk = wave / (WM * WN), wmn = wave % (WM * WN);
  const int wn = wmn % WN;
  const int r = lane & 15, g4 = lane >> 4;

  // tile decode; each XCD (own L2) gets one contiguous stretch of the tile order
  int tile;
  {
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int q = G >> 3, rem = G & 7;
    tile = xcd * q + (xcd < rem ? xcd : rem) + local;
  }
  // (which wavefronts get a tile's first blocks rotates from work-group to work-group, so that where the blocks do not
  // divide evenly the longer and the shorter shares meet on every SIMD of a unit)
  const int wm = (wmn / WN + (tile >> 1)) % WM;
  const int tiles_s = a.tiles_n * a.tiles_y * a.tiles_x;
  const int q_s = (int)fast_div((unsigned)tile, a.magic_s), q_m = (int)fast_div((unsigned)tile, a.magic_m);
  const int tile_m = a.m_major ? q_s : tile - q_m * a.tiles_m;
  const int rest = a.m_major ? tile - q_s * tiles_s : q_m;
  const int q_x = (int)fast_div((unsigned)rest, a.magic_x);
  const int q_y = (int)fast_div((unsigned)q_x, a.magic_y);
  const int tx0 = (rest - q_x * a.tiles_x) * a.tw;
  const int ty0 = (q_x - q_y * a.tiles_y) * a.th;
  const int n0 = q_y * a.ni;
  const SplitShare share = split_share(tile_m, wm, WM, a.blk_base, a.blk_rem);
  const int nblk = share.count;           // 16-filter blocks of this wavefront
  const int o0 = share.first * 16;        // its first filter

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);

  // ---- weights: one round of this wavefront's filter blocks ----
  const unsigned a_blk = (unsigned)a.rtot * (P * 1024u);
  const unsigned a_base = (unsigned)split_weight_block(share.first, a.blk_base * a.tiles_m + a.blk_rem) * a_blk;
  auto load_weights = [&](auto mbc, int round, uint4 (&f)[MB][P]) CPRUNE_INLINE {
    const int rg = split_weight_round(round, a.rtot);
#pragma unroll
    for (int i = 0; i < decltype(mbc)::value; ++i)
#pragma unroll
      for (int p = 0; p < P; ++p)
        f[i][p] = load_b128(wr, (unsigned)lane * 16u + p * 1024u, a_base + i * a_blk + (unsigned)rg * (P * 1024u));
  };
  uint4 a0[MB][P], a1[MB][P];

  // ---- staging items: (patch pixel, 8-channel group) ----
  const int npp = a.ph * a.pw, npatch = a.ni * npp;
  const int hw = a.H * a.W;
  unsigned b_off[NIB];
  int b_lds[NIB], b_ch[NIB];
#pragma unroll
  for (int j = 0; j < NIB; ++j) {
    const int idx = t + 256 * j;
    int g, pp;
    if constexpr (NCHW) {
      g = (int)fast_div((unsigned)idx, a.magic_np);
      pp = idx - g * npatch;
    } else {
      g = idx & 3;
      pp = idx >> 2;
    }
    const bool item = pp < npatch && g < 4;
    const int img = (int)fast_div((unsigned)pp, a.magic_pp), pr = pp - img * npp;
    const int py = (int)fast_div((unsigned)pr, a.magic_pw), px = pr - py * a.pw;
    const int iy = ty0 * a.stride + py - a.pad, ix = tx0 * a.stride + px - a.pad, n = n0 + img;
    const bool inside = item && n < a.N && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
    if constexpr (NCHW)
      b_off[j] = inside ? (unsigned)((n * a.C + g * 8) * hw + iy * a.W + ix) * ES : kOutOfRange;
    else
      b_off[j] = inside ? (unsigned)(((n * a.H + iy) * a.W + ix) * a.C + g * 8) * ES : kOutOfRange;
    b_lds[j] = item ? a.off_patch + pp * BROW + g * UNIT : 64;
    b_ch[j] = g * 8;
  }
  uint32_t breg[NIB][NV];
  auto gload = [&](int c) CPRUNE_INLINE {
    const int c0 = c * 32;
#pragma unroll
    for (int j = 0; j < NIB; ++j) {
      if constexpr (NCHW) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const unsigned voff = b_off[j] | ((unsigned)(c0 + b_ch[j] + e >= a.C) << 31);
          const uint32_t v = Elem<T>::load(xr, voff, (unsigned)(min(c0 + e, a.C - 1) * hw) * ES);
          if constexpr (ES == 4) breg[j][e] = v;
          else if (e & 1) breg[j][e >> 1] |= v << 16;
          else breg[j][e >> 1] = v;
        }
      } else {
        constexpr int EPI = 16 / ES;      // elements per 16-byte load
#pragma unroll
        for (int e = 0; e < 8; e += EPI) {
          const unsigned voff = b_off[j] | ((unsigned)(c0 + b_ch[j] + e >= a.C) << 31);
          const uint4 v = load_b128(xr, voff + e * ES, (unsigned)(c0 * ES));
          breg[j][e * ES / 4] = v.x; breg[j][e * ES / 4 + 1] = v.y;
          breg[j][e * ES / 4 + 2] = v.z; breg[j][e * ES / 4 + 3] = v.w;
        }
      }
    }
  };
  auto lds_store = [&]() CPRUNE_INLINE {
    if constexpr (P == 1) {
#pragma unroll
      for (int j = 0; j < NIB; ++j) *(uint4*)(smem + b_lds[j]) = make_uint4(breg[j][0], breg[j][1], breg[j][2], breg[j][3]);
    } else {
#pragma unroll
      for (int j = 0; j < NIB; ++j) {
        uint4* const dst = (uint4*)(smem + b_lds[j]);
        uint32_t h[4], m[4], l[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) split3(breg[j][2 * e], breg[j][2 * e + 1], h[e], m[e], l[e]);
        dst[0] = make_uint4(h[0], h[1], h[2], h[3]);
        dst[1] = make_uint4(m[0], m[1], m[2], m[3]);
        dst[2] = make_uint4(l[0], l[1], l[2], l[3]);
      }
    }
  };
  gload(0);

  // ---- offset tables: unit u of a chunk = (tap u / groups, group u % groups); -1 past the last unit ----
  if (t < 32) ((int*)smem)[t] = 0;
  for (int i = t; i < (a.taps + a.rounds_last) * 4; i += 256) {
    const bool last = i >= a.taps * 4;
    const int u = last ? i - a.taps * 4 : i;
    const int ng = last ? a.groups_last : 4;
    const int tap = u / ng, g = u - tap * ng;
    const int ty = tap / a.kw;
    tab[i] = tap < a.taps ? (ty * a.pw + tap - ty * a.kw) * BROW + g * UNIT : -1;
  }

  // ---- this lane's pixels: patch position of the window's first tap ----
  int b_frag[NB];
  auto pixel_of = [&](int j, int& img, int& ty, int& tx) CPRUNE_INLINE {   // column j of this wavefront
    const int id = (wn * NB + j) * 16 + r;
    if (a.pool) {   // four consecutive pixels are one 2x2 window
      const int win = id >> 2, wpi = (a.th * a.tw) >> 2;
      img = (int)fast_div((unsigned)win, a.magic_thw);
      const int wr_ = win - img * wpi;
      const int wy = (int)fast_div((unsigned)wr_, a.magic_tw);
      ty = 2 * wy + ((id >> 1) & 1);
      tx = 2 * (wr_ - wy * (a.tw >> 1)) + (id & 1);
    } else {
      img = (int)fast_div((unsigned)id, a.magic_thw);
      const int ir = id - img * a.th * a.tw;
      ty = (int)fast_div((unsigned)ir, a.magic_tw);
      tx = ir - ty * a.tw;
    }
  };
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    int img, ty, tx;
    pixel_of(j, img, ty, tx);
    b_frag[j] = a.off_patch + (img < a.ni ? (img * npp + ty * a.stride * a.pw + tx * a.stride) * BROW : 0);
  }

  float4_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = (float4_t){0.f, 0.f, 0.f, 0.f};

  // pixel columns are multiplied JS at a time; two such sets of operands are held: the one in use and the next one
  constexpr int JS = (NB >= 8 && MB == 1) ? 4 : (NB >= 4 && MB <= 2 ? 2 : 1), NSET = NB / JS;
  static_assert(NSET >= 2 && NB % JS == 0, "two operand sets");
  uint4 bf[2][JS][P];
  auto read_set = [&](int set, int off) CPRUNE_INLINE {
#pragma unroll
    for (int j = 0; j < JS; ++j) {
      const uint4* const src = (const uint4*)(smem + (off < 0 ? 0 : b_frag[set * JS + j] + off));
#pragma unroll
      for (int p = 0; p < P; ++p) bf[set & 1][j][p] = src[p];
    }
  };
  // The five small products of a round are added up among themselves, so that their sum is rounded at its own size, and
  // meet the running sum once: two roundings of it per 32 terms, where the fp32 instruction makes 32.  They do so
  // while the next set is multiplied.  The barriers keep consecutive MFMAs on different accumulators: left alone the
  // scheduler issues each block's chain back to back and waits out every result (56 -> 56 filters at 32x32, batch 64:
  // 28.1 us without, 25.7 us with them).
  float4_t small[MB][JS];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < JS; ++j) small[i][j] = (float4_t){0.f, 0.f, 0.f, 0.f};
  auto add_small = [&](auto mbc, int set) CPRUNE_INLINE {
    constexpr int MBC = decltype(mbc)::value;
#pragma unroll
    for (int j = 0; j < JS; ++j)
#pragma unroll
      for (int i = 0; i < MBC; ++i) acc[i][set * JS + j] += small[i][j];
  };
  // one round at offset `off`, its first two operand sets read; leaves the first two of the round at `next_off`
  auto round = [&](auto mbc, const uint4 (&f)[MB][P], int off, int next_off) CPRUNE_INLINE {
    constexpr int MBC = decltype(mbc)::value;
#pragma unroll
    for (int set = 0; set < NSET; ++set) {
      const int j0 = set * JS;
      const uint4 (&b)[JS][P] = bf[set & 1];
      if constexpr (P == 3) {
        float4_t sum[MB][JS];
#pragma unroll
        for (int j = 0; j < JS; ++j)
#pragma unroll
          for (int i = 0; i < MBC; ++i) sum[i][j] = mfma_split<T>(f[i][0], b[j][2], (float4_t){0.f, 0.f, 0.f, 0.f});
        __builtin_amdgcn_sched_barrier(0x6);
        add_small(mbc, (set + NSET - 1) % NSET);
        auto term = [&](int pa, int pb) CPRUNE_INLINE {
#pragma unroll
          for (int j = 0; j < JS; ++j)
#pragma unroll
            for (int i = 0; i < MBC; ++i) sum[i][j] = mfma_split<T>(f[i][pa], b[j][pb], sum[i][j]);
          __builtin_amdgcn_sched_barrier(0x6);
        };
        term(2, 0);
#pragma unroll
        for (int j = 0; j < JS; ++j)
#pragma unroll
          for (int i = 0; i < MBC; ++i) acc[i][j0 + j] = mfma_split<T>(f[i][0], b[j][0], acc[i][j0 + j]);
        __builtin_amdgcn_sched_barrier(0x6);
        term(1, 1); term(0, 1); term(1, 0);
#pragma unroll
        for (int j = 0; j < JS; ++j)
#pragma unroll
          for (int i = 0; i < MBC; ++i) small[i][j] = sum[i][j];
      } else {
#pragma unroll
        for (int j = 0; j < JS; ++j)
#pragma unroll
          for (int i = 0; i < MBC; ++i) acc[i][j0 + j] = mfma_split<T>(f[i][0], b[j][0], acc[i][j0 + j]);
      }
      if (set + 2 < NSET) read_set(set + 2, off);
      else read_set(set + 2 - NSET, next_off);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  const int nchunk = a.nfull + (a.rounds_last ? 1 : 0);
  auto main_loop = [&](auto mbc) CPRUNE_INLINE {
    constexpr int MBC = decltype(mbc)::value;
    load_weights(mbc, wk, a0);
    for (int c = 0; c < nchunk; ++c) {
      __syncthreads();            // everyone is done reading the previous chunk (and the tables are written)
      lds_store();
      __syncthreads();
      const bool full = c < a.nfull;
      const int R = full ? a.taps : a.rounds_last;
      const int* const tb = tab + (full ? 0 : a.taps * 4) + g4;
      const int rg0 = c * a.taps;
      auto next_rg = [&](int q) CPRUNE_INLINE { return split_next_round(q, wk, WK, R, rg0, a.taps); };
      if (wk >= R) {
        if (c + 1 < nchunk) gload(c + 1);
        continue;
      }
      auto tab_at = [&](int q) CPRUNE_INLINE { return tb[(q < R ? q : R - 1) * 4]; };
      int off0 = tab_at(wk), off1 = tab_at(wk + WK);
      read_set(0, off0);
      read_set(1, off0);
      int q = wk;
      // the first round asks for the second one's weights before it asks for the next chunk's activations: loads
      // return in order, and a wait for weights asked for behind them waits for them too
      load_weights(mbc, next_rg(q), a1);
      if (c + 1 < nchunk) gload(c + 1);
      auto step = [&](const uint4 (&f)[MB][P], int qq) CPRUNE_INLINE {
        const int nxt = tab_at(qq + 2 * WK);
        round(mbc, f, off0, off1);
        off0 = off1;
        off1 = nxt;
      };
      step(a0, q);
      q += WK;
      for (; q + WK < R; q += 2 * WK) {
        load_weights(mbc, next_rg(q), a0);
        step(a1, q);
        load_weights(mbc, next_rg(q + WK), a1);
        step(a0, q + WK);
      }
      if (q < R) {
        load_weights(mbc, next_rg(q), a0);
        step(a1, q);
      } else {
#pragma unroll
        for (int i = 0; i < MBC; ++i)
#pragma unroll
          for (int p = 0; p < P; ++p) a0[i][p] = a1[i][p];
      }
    }
    if constexpr (P == 3) add_small(mbc, NSET - 1);
  };
  // The wavefront's whole reduction once more, four terms at a time on the fp32 instruction, operands straight from
  // memory: for data that three parts do not hold only, because it is slow (every wavefront of 128 -> 83 filters at 56x56, batch
  // 8: 44 -> 200 us, of 512 -> 411 at 7x7, batch 32: 71 -> 550-630 us).
  auto again = [&]() CPRUNE_INLINE {
    const __amdgpu_buffer_rsrc_t ww = make_rsrc(a.w_raw, a.w_raw_bytes);
    const unsigned step = NCHW ? (unsigned)hw * 4u : 4u, row = (unsigned)(a.taps * a.C) * 4u;
    const unsigned wtap = NCHW ? 4u : (unsigned)a.C * 4u, wchan = NCHW ? (unsigned)a.taps * 4u : 4u;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = (float4_t){0.f, 0.f, 0.f, 0.f};
    for (int tap = 0; tap < a.taps; ++tap) {
      const int u = tap / a.kw;
      unsigned px[NB];      // this lane's pixels under the tap, channel 0
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        int img, ty, tx;
        pixel_of(j, img, ty, tx);
        const int n = n0 + img, iy = (ty0 + ty) * a.stride - a.pad + u, ix = (tx0 + tx) * a.stride - a.pad + tap - u * a.kw;
        const bool inside = img < a.ni && n < a.N && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
        const int pix = NCHW ? n * a.C * hw + iy * a.W + ix : ((n * a.H + iy) * a.W + ix) * a.C;
        px[j] = inside ? (unsigned)pix * 4u : kOutOfRange;
      }
      for (int c0 = 0; c0 < a.C; c0 += 4) {
        const int c = c0 + g4;
        const bool real = c < a.C;
        float wv[MB], xv[NB];
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const int o = o0 + i * 16 + r;
          const bool have = real && i < nblk && o < a.O;
          wv[i] = __uint_as_float(Elem<float>::load(ww, have ? o * row + tap * wtap + c * wchan : kOutOfRange, 0));
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) xv[j] = __uint_as_float(Elem<float>::load(xr, real ? px[j] + c * step : kOutOfRange, 0));
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i], xv[j], acc[i][j], 0, 0, 0);
      }
    }
  };
  // compiled once per block count, as the other kernels' main loops (a wavefront without a block runs the shortest one
  // and stores nothing)
  if (MB >= 3 && nblk >= 3) main_loop(std::integral_constant<int, MB >= 3 ? 3 : 1>{});
  else if (MB >= 2 && nblk >= 2) main_loop(std::integral_constant<int, MB >= 2 ? 2 : 1>{});
  else main_loop(std::integral_constant<int, 1>{});
  if constexpr (WK > 1) {
    // the wavefronts that share a block hand their sums to the first, which adds them in order
    __syncthreads();
    float4_t* const red = (float4_t*)smem + (size_t)wmn * (MB * NB * 64) + lane;
    constexpr int STEP = WM * WN * MB * NB * 64;
    if (wk > 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) red[(wk - 1) * STEP + (i * NB + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (wk > 0) return;
#pragma unroll
    for (int k = 1; k < WK; ++k)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] += red[(k - 1) * STEP + (i * NB + j) * 64];
  }
  if (nblk == 0) return;

  if constexpr (P == 3) {
    // Every infinity and every number that rounds to one makes a sum infinite or NaN (its first part is infinite, the
    // second infinite of the other sign or NaN).  A number under 2^-110 loses at most 2^-134 (half of bf16's last bit; the
    // instruction keeps denormal operands: 1e-36 keeps 14 bits), times the other operand in its product: below half the last place
    // of sums from 2^-50 up while the terms of a sum times that operand stay under 2^59.  (Sums of ordinary numbers that
    // come out smaller, but not zero, are one in 10^15.)
    constexpr uint32_t kInf = 0x7f800000u, kSmall = (127u - 50u) << 23;
    // (first a look that takes one and a half operations per sum and cannot tell zeros from small numbers)
    uint32_t odd = 0;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) odd = max(odd, (__float_as_uint(acc[i][j][v]) << 1) - (kSmall << 1));
    if (__any(odd >= (kInf - kSmall) << 1)) {
      uint32_t top = 0, low = ~0u;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const uint32_t mag = __float_as_uint(acc[i][j][v]) & 0x7fffffffu;
            top = max(top, mag);
            low = min(low, mag - 1);      // (zero goes to the other end)
          }
      if (__any(top >= kInf || low < kSmall - 1)) again();
    }
  }

  // ---- epilogue: a lane holds filters o .. o + 3 of its pixel ----
  ConvArgs e;
  e.bias = a.bias; e.res = a.res; e.y = a.y; e.O = a.O; e.Cop = a.Cop; e.act = a.act; e.vec_out = a.vec_out; e.pool4 = 0;
  float4_t bias4[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) bias4[i] = load_bias4(a.bias, a.O, o0 + i * 16 + 4 * g4);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    int img, ty, tx;
    pixel_of(j, img, ty, tx);
    const int n = n0 + img, oy = ty0 + ty, ox = tx0 + tx;
    const bool inside = img < a.ni && ty < a.th && n < a.N && oy < a.Ho && ox < a.Wo;
    if constexpr (NCHW) {
      if (!inside) continue;
      T* const yg = (T*)a.y;
      const T* const rg = (const T*)a.res;
      const size_t howo = (size_t)a.Ho * a.Wo;
      const size_t pix = (size_t)n * a.O * howo + (size_t)oy * a.Wo + ox;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (i >= nblk) break;
          const int o = o0 + i * 16 + 4 * g4 + v;
          if (o < a.O) {
            const size_t off = pix + (size_t)o * howo;
            float val = acc[i][j][v] + bias4[i][v];
            if (rg) val += Elem<T>::to_f32(rg[off]);
            yg[off] = Elem<T>::from_f32(apply_act(val, a.act));
          }
        }
    } else if (!a.pool) {
      if (!inside) continue;
#pragma unroll
      for (int i = 0; i < MB; ++i)
        if (i < nblk) nhwc_store4<T>(e, acc[i][j], (n * a.Ho + oy) * a.Wo + ox, o0 + i * 16 + 4 * g4, bias4[i]);
    } else {
      // the activation is monotone: the maximum of a window's four activated values, in lanes r ^ 1, r ^ 2, r ^ 3
      ConvArgs ep = e;
      ep.act = CPRUNE_ACT_NONE;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        float4_t m;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float x = apply_act(acc[i][j][v] + bias4[i][v], a.act);
          x = fmaxf(x, __shfl_xor(x, 1, 64));
          m[v] = fmaxf(x, __shfl_xor(x, 2, 64));
        }
        if (inside && (r & 3) == 0 && i < nblk)
          nhwc_store4<T>(ep, m, (n * (a.Ho >> 1) + (oy >> 1)) * (a.Wo >> 1) + (ox >> 1), o0 + i * 16 + 4 * g4,
                         (float4_t){0.f, 0.f, 0.f, 0.f});
      }
    }
  }
}

template <typename T, bool NCHW>
inline int launch_split(int id, dim3 grid, size_t lds, hipStream_t s, const SplitArgs& a) {
#define CPRUNE_SPLIT_CASE(ID, WM_, WN_, WK_, MB_, NB_, NIB_)                                                  \
  case ID: {                                                                                                  \
    static std::atomic<bool> raised{false};   /* more than the default 64 KiB of LDS has to be asked for once */ \
    if (lds > 65536 && !raised.load(std::memory_order_relaxed)) {                                             \
      CPRUNE_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_split_kernel<T, NCHW, WM_, WN_, WK_, MB_, NB_, NIB_>), \
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));            \
      raised.store(true, std::memory_order_relaxed);                                                          \
    }                                                                                                         \
    hipLaunchKernelGGL((conv_split_kernel<T, NCHW, WM_, WN_, WK_, MB_, NB_, NIB_>), grid, dim3(256), lds, s, a); \
    break;                                                                                                    \
  }
  switch (id) { CPRUNE_SPLIT_LIST(CPRUNE_SPLIT_CASE) default: return CPRUNE_ERR_UNSUPPORTED; }
#undef CPRUNE_SPLIT_CASE
  return CPRUNE_OK;
}

int launch_conv_split_f32(int id, bool nchw, dim3 grid, size_t lds, hipStream_t s, const SplitArgs& a);
int launch_conv_split_f16(int id, dim3 grid, size_t lds, hipStream_t s, const SplitArgs& a);    // NCHW only
int launch_conv_split_bf16(int id, dim3 grid, size_t lds, hipStream_t s, const SplitArgs& a);

}  // namespace cprune
