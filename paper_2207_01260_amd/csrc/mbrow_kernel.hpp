// Inverted-residual blocks (MobileNetV2, MnasNet), channels-last: the depthwise k x k layer and the 1x1 projection
// behind it in one kernel, with or without the 1x1 expansion in front of them.  The expanded channels are the ones the
// method prunes and the block's largest tensor by far; here they are read once and never written (XH = 0), or never
// reach memory at all (XH > 0).
//
// What bounds such a kernel is not arithmetic but the hand-over between its three steps: through LDS every step is a
// chain write -> barrier -> read.  Here a WAVEFRONT runs all three steps in registers.  It owns a strip of 16 columns x R
// output rows of one image (a map of at most 8 lanes per row packs two images) and walks over the expanded channels in
// chunks of 64 bytes per pixel, over the strip's input rows inside a chunk:
//   expansion   one 16 x 16 MFMA block: rows = 16 expanded channels, columns = the 16 pixels of the row.  Its result
//               layout (lane = pixel r + 16 * g, registers = channels 4 g .. 4 g + 3) is what the next steps need.
//   depthwise   a row is multiplied into the K output rows it touches; the horizontal neighbours come from the
//               neighbouring lanes (DPP row shifts inside the 16 lanes, part of the FMA).  Stride 2 holds even and odd
//               columns in two registers.  Taps outside the image have zero weights (per lane, loaded once a chunk).
//   projection  a finished row is, as it stands, the B operand of 16 pixels x 16 (32) channels.
// No LDS access, no barrier and no conversion lies between the steps.  LDS holds the block input of the strip (read as
// the expansion's B operand once per chunk); KS wavefronts of a work-group share a strip and split its chunks, their sums
// meet in LDS at the end, in order.  Weights come from L2 in operand order, once per chunk and wavefront.
// IMG: the layer in front of the depthwise one is the network's first, a 3x3 / stride 2 layer on an NCHW image of at most 3
// channels; the image is staged, and a lane gathers its terms of a window from there.
// Neighbouring strips overlap by the window's halo: 14 of 16 columns (k = 3) and R of R + k - 1 rows are new.
//
// Values handed from step to step are rounded to the activation type, as the separate layers store them.
//
// fp32 with 3x3 windows and up to 96 filters runs mbrow3_kernel.hpp instead, the same strips on three bf16 parts.
//
// Measured (expansion + depthwise + projection, us): the layers apart or with the depthwise layer fused through LDS, the
// faster of both / this kernel.  MnasNet bf16 at batch 16: 16 -> 38 -> 24, 112x112: 20 / 10; 24 -> 58 -> 24 at 56x56: 15 / 8.3; image 3 -> 32 -> 16
// 20.3 / 16 (the windows' gather from LDS).  Without window weights as fp32 and operands
// a row ahead / with them (mbrow_wide, mbrow_read_ahead): 32 -> 92 -> 32 at 28x28 batch 64 11.0 / 10.1, 64 -> 330 -> 64 at 14x14 13.1 / 12.5.
// Counters over MnasNet's launches in bf16 at batch 16: 3x3 vector ALU busy 53 % of the cycles in which a unit has work, matrix pipes 4, waiting for memory or a barrier 34 % of
// the wave cycles; 5x5 36, 3 and 42.
//  In fp32 the matrix instruction bounds it, which takes turns with the vector ALU (mbrow3_kernel.hpp).
#pragma once
#include <atomic>
#include "conv_nhwc_kernel.hpp"

namespace cprune {

// lane l of each row of 16 takes lane l + D of that row, zero past the row's end
template <int D>
__device__ __forceinline__ float row_shift(float v) {
  if constexpr (D == 0) return v;
  else {
    constexpr int ctrl = D > 0 ? 0x100 + D : 0x110 - D;      // row_shl / row_shr
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xf, 0xf, true));
  }
}

// Where a wavefront works.
struct MbAt {
  int lane, r, g4, wave, ks;       // wavefront of the strip's ks
  int o0;                          // first filter of the projection tile
  int tx, ty, n0, img;             // strip, its first image, the lane's image
  int j0, lr, cj, iy0;             // first output column of the strip, the lane's place in its image's columns, its output column; input row 0
  bool two, lane_out;              // two images side by side; the lane's column is one that this strip stores
};

template <int K, int S, int MB, int R>
__device__ __forceinline__ MbAt mbrow_at(const MbArgs& a) {
  constexpr int HL = mbrow_halo_left(K, S), HR = mbrow_halo_right(K, S);
  MbAt p;
  p.lane = threadIdx.x & 63;
  p.ks = (int)blockDim.x >> 6;
  p.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  p.r = p.lane & 15; p.g4 = p.lane >> 4;
  int tile;
  {
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int q = G >> 3, rem = G & 7;
    tile = xcd * q + (xcd < rem ? xcd : rem) + local;
  }
  p.o0 = blockIdx.y * (MB * 16);
  const StripAt strip = strip_at(tile, a.tiles_x, a.tiles_y, a.magic_x, a.magic_y);
  p.tx = strip.tx; p.ty = strip.ty;
  p.two = a.ipt == 2;
  p.n0 = p.two ? 2 * strip.group : strip.group;
  p.j0 = p.tx * (16 - HL - HR);
  p.lr = p.two ? (p.r & 7) : p.r;
  p.img = p.two ? p.n0 + (p.r >> 3) : p.n0;
  p.cj = p.j0 + p.lr;
  p.iy0 = p.ty * R * S - K / 2;
  p.lane_out = (p.img < a.N) & (p.cj < a.Wo) & ((p.tx == 0) | (p.lr >= HL)) & ((p.tx == a.tiles_x - 1) | (p.lr < 16 - HR));
  return p;
}

// Shortcut (all loads before the first store), activation, store of four filters of one pixel; where several wavefronts share the
// strip, behind the sum of theirs.
template <typename T, int R, int MB>
__device__ __forceinline__ void mbrow_finish(const MbArgs& a, const MbAt& at, unsigned char* lds, float4_t (&acc)[R][MB]) {
  constexpr int ES = (int)sizeof(T);
  const int lane = at.lane, ks = at.ks, wave = at.wave, g4 = at.g4;
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res, a.res ? a.y_bytes : 0u);
  const float lo_o = a.act_out == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi_o = a.act_out == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  auto out_at = [&](int y, int m) -> unsigned {
    const int oy = at.ty * R + y, o = at.o0 + m * 16 + 4 * g4;
    return at.lane_out & (oy < a.Ho) & (o < a.Cop) ? (unsigned)(((at.img * a.Ho + oy) * a.Wo + at.cj) * a.Cop + o) * ES : kOutOfRange;
  };
  auto load_res = [&](unsigned off) -> float4_t {
    if constexpr (ES == 4) {
      const uint4 q = load_b128(rr, off, 0);
      return __builtin_bit_cast(float4_t, q);
    } else {
      return widen4<T>(load_b64(rr, off, 0));
    }
  };
  auto store = [&](unsigned off, float4_t v) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = __builtin_amdgcn_fmed3f(v[q], lo_o, hi_o);
    if (off == kOutOfRange) return;
    if constexpr (ES == 4) *(float4_t*)((char*)a.y + off) = v;
    else *(uint2*)((char*)a.y + off) = narrow4<T>(v);
  };
  if (ks == 1) {
    constexpr int GROUP = MB > 4 ? 2 : 16 / MB;       // rows whose shortcuts are in flight together
#pragma unroll
    for (int y0 = 0; y0 < R; y0 += GROUP) {
      if (a.res) {
        float4_t res[GROUP][MB];
#pragma unroll
        for (int y = 0; y < GROUP; ++y)
#pragma unroll
          for (int m = 0; m < MB; ++m)
            if (y0 + y < R) res[y][m] = load_res(out_at(y0 + y, m));
#pragma unroll
        for (int y = 0; y < GROUP; ++y)
#pragma unroll
          for (int m = 0; m < MB; ++m)
            if (y0 + y < R) acc[y0 + y][m] += res[y][m];
      }
#pragma unroll
      for (int y = 0; y < GROUP; ++y)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          if (y0 + y < R) store(out_at(y0 + y, m), acc[y0 + y][m]);
    }
    return;
  }

  // the sums of the wavefronts meet in LDS: the upper half hands over to the lower one until a.slots of them are left,
  // whose sums are then added in order, the (row, filter block) units shared by all wavefronts
  constexpr int SLOT = R * MB * 64;
  float4_t* const xch = (float4_t*)lds;
  int nw = ks;
  while (nw > a.slots) {
    const int hw = nw >> 1;
    __syncthreads();
    if (wave >= hw && wave < nw) {
      float4_t* const dst = xch + (wave - hw) * SLOT + lane;
#pragma unroll
      for (int y = 0; y < R; ++y)
#pragma unroll
        for (int m = 0; m < MB; ++m) dst[(y * MB + m) * 64] = acc[y][m];
    }
    __syncthreads();
    if (wave < hw) {
      const float4_t* const src = xch + wave * SLOT + lane;
#pragma unroll
      for (int y = 0; y < R; ++y)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[y][m] += src[(y * MB + m) * 64];
    }
    nw = hw;
  }
  __syncthreads();
  if (wave < nw) {
    float4_t* const dst = xch + wave * SLOT + lane;
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
      for (int m = 0; m < MB; ++m) dst[(y * MB + m) * 64] = acc[y][m];
  }
  __syncthreads();
  constexpr int UNITS = R * MB;
  for (int q0 = wave; q0 < UNITS; q0 += 4 * ks) {
    float4_t res[4];
    unsigned off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = q0 + j * ks;
      off[j] = q < UNITS ? out_at(q / MB, q % MB) : kOutOfRange;
      if (a.res) res[j] = load_res(off[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int q = q0 + j * ks;
      if (q >= UNITS) break;
      float4_t s = xch[q * 64 + lane];
      for (int w = 1; w < nw; ++w) s += xch[w * SLOT + q * 64 + lane];
      if (a.res) s += res[j];
      store(off[j], s);
    }
  }
}

// What a strip with a 3x3 window has registers for beside its sums, 4 R MB of them.  Wide (16-bit data): the window's weights come as fp32 (widened
// where they are used they are a tenth of the vector operations; waiting for that they are 18 registers fewer); without an expansion the input
// rows of a chunk lie in registers too.  Reading ahead: the expansion's operands of a row are read from LDS while the row before it
// is multiplied, 4 a round.  Neither / ahead / wide / both, us, expanded to 86-400 channels, 56x56, batch 8: bf16 24 -> 32 9.7 / 9.4 / 9.3 / 9.2, stride 2 8.7 / 8.3 /
// 8.6 / 8.1, 64 -> 96 low 18.7 / 17.9 / 17.7 / 16.8; 64 -> 64 tall 16.0 / 17.6 / 16.1 / 16.7; 160 -> 128 tall 37.7 / 43 / 41 / 48, stride 2 17.5 / 18.5 / 17.9 / 19.7; fp16
// 64 -> 64 tall 14.5 / 14.2 / 16.4 / 16.9, 96 -> 96 tall 31 / 33 / 40 / 40, low 24.0 / 22.9 / 23.2 / 24.2.  Depthwise and projection alone, narrow / wide: bf16 64 filters
// tall 9.3 / 11.1, low 8.0 / 7.8, stride 2 tall 7.1 / 7.8, 128 9.8 / 9.5; fp16 64 tall 9.1 / 12.0, low 7.9 / 7.9, stride 2 tall 7.7 / 11.0, 128 stride 2 6.4 / 7.7.  fp32
// 96 -> 128 (of 128 filters only), not ahead / ahead: low 66.5 / 65.0, tall 86 / 88, stride 2 36.6 / 38.0.  5x5 windows have no room for either (40 -> 88 -> 40 at 28x28 12.5 / 13.3
// with both).
// At 112x112, batch 64, the chip full, a third wavefront on a SIMD counts: fp16 64 -> 32 stride 2 tall 70 neither / 81 ahead / 85 wide, 24 -> 32 low 33 / 32 / 32, both 34,
// 64 -> 64 low 81 / 90 / 94; the image form with 16 filters at 224x224, batch 64, fp16 tall 45.5 / 45.1 / 52.3 / 52.2, low 57.6 / 57.8 / 57.0 / 57.3, bf16 tall 53.7 / 53.2 /
// 52.5 / 52.4, low 59.7 / 59.5 / 57.6 / 57.1.
template <typename T>
constexpr bool mbrow_wide(int k, int s, int mb, int xh, int r, bool image) {
  if (sizeof(T) != 2 || k != 3) return false;
  const int sums = 4 * r * mb, rows = (r - 1) * s + k;
  if (std::is_same<T, __bf16>::value) return xh ? mb < 8 : sums + 4 * rows * s <= 120;
  if (image) return (mb == 1) == (r <= 4);               // (the others have three wavefronts without, two with)
  return xh && s == 1 && mb <= 4 && sums <= 64;          // (fp16 forms spill where those of bf16 do not)
}
template <typename T>
constexpr bool mbrow_read_ahead(int k, int s, int mb, int xh, int r, bool image) {
  if (k != 3 || xh == 0) return false;
  const bool low = 4 * r * mb <= 72;
  if (sizeof(T) == 4) return low && s == 1;
  if (std::is_same<T, __bf16>::value) return (xh <= 2 || low) && !(mb == 8 && s == 2);
  return (mb <= 4 || low) && !image && !(s == 2 && xh == 4 && r * mb == 8);      // (those two: 165 registers without, 170 with)
}

template <typename T, int K, int S, int MB, int XH, int R, bool IMG>
__global__ __launch_bounds__(512, 2) void mbrow_kernel(MbArgs a) {
  constexpr int ES = (int)sizeof(T);
  constexpr int EPI = 16 / ES;
  constexpr int PAD = K / 2;
  constexpr int ROWS = (R - 1) * S + K;        // input rows of a strip
  constexpr int CW = 16 * S;                   // input columns of a strip
  constexpr int NH = ES == 4 ? 1 : 2;          // blocks of 16 channels in a chunk
  constexpr int XQ = XH * 2;                   // 16-byte pieces of a staged pixel
  constexpr int XP = XH * 32 + 16;             // bytes per staged pixel
  constexpr int XR = XH / 2;                   // whole 64-byte rounds of the expansion's reduction
  constexpr bool EXP = XH > 0;
  constexpr int IROWS = 2 * ROWS + 1, IPITCH = mbrow_image_pitch(ES);   // IMG: rows and row pitch of the staged image

  constexpr bool AHEAD = !(EXP && K == 5 && ES == 2);   // window weights asked for one block ahead (there they do not fit)
  constexpr bool W32 = ES == 4 || mbrow_wide<T>(K, S, MB, XH, R, IMG), READ_AHEAD = mbrow_read_ahead<T>(K, S, MB, XH, R, IMG);

  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int HL = mbrow_halo_left(K, S), HR = mbrow_halo_right(K, S);
  // (mbrow_at's lines: through its result 5x5 forms spilled up to twice as much, bf16 24 -> 64 at 28x28, batch 32 15.5 / 16.5 us, and all were 2 % slower)
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int ks = (int)blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 15, g4 = lane >> 4;

  int tile;
  {
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int q = G >> 3, rem = G & 7;
    tile = xcd * q + (xcd < rem ? xcd : rem) + local;
  }
  const int o0 = blockIdx.y * (MB * 16);
  const StripAt strip = strip_at(tile, a.tiles_x, a.tiles_y, a.magic_x, a.magic_y);
  const int tx = strip.tx, ty = strip.ty, grp = strip.group;
  const bool two = a.ipt == 2;
  const int n0 = two ? 2 * grp : grp;
  const int j0 = tx * (16 - HL - HR);
  const int lr = two ? (r & 7) : r;
  const int img = two ? n0 + (r >> 3) : n0;
  const int cj = j0 + lr;                      // the lane's output column
  const int iy0 = ty * R * S - PAD;
  const bool lane_out = (img < a.N) & (cj < a.Wo) & ((tx == 0) | (lr >= HL)) & ((tx == a.tiles_x - 1) | (lr < 16 - HR));
  MbAt at;                                     // for mbrow_finish
  at.lane = lane; at.r = r; at.g4 = g4; at.wave = wave; at.ks = ks; at.o0 = o0;
  at.tx = tx; at.ty = ty; at.n0 = n0; at.img = img; at.j0 = j0; at.lr = lr; at.cj = cj; at.iy0 = iy0;
  at.two = two; at.lane_out = lane_out;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t er = make_rsrc(a.we, a.we_bytes);
  const __amdgpu_buffer_rsrc_t pr = make_rsrc(a.wp, a.wp_bytes);
  const __amdgpu_buffer_rsrc_t dr = W32 && ES == 2 ? make_rsrc(a.wdw32, 2 * a.wdw_bytes) : make_rsrc(a.wdw, a.wdw_bytes);

  if constexpr (EXP) {
    // the strip's block input: zeros outside the image and past the last channel
    const int nthr = ks * 64;
    if constexpr (IMG) {
      // the image under the strip's windows, [channel][row][column], zeros outside; all loads of a batch in flight together
      constexpr int ITEMS = 3 * IROWS * 33, U = 16;
      for (int b0 = t; b0 < ITEMS; b0 += nthr * U) {
        typename Elem<T>::raw_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b0 + u * nthr;
          const int row = idx / 33, ix = 2 * j0 - 1 + idx - row * 33;
          const int c = row / IROWS, iy = 2 * iy0 - 1 + row - c * IROWS;
          const bool in = (idx < ITEMS) & (c < a.Cpi) & ((unsigned)iy < (unsigned)a.Hi) & ((unsigned)ix < (unsigned)a.Wi);
          v[u] = Elem<T>::load(xr, in ? (unsigned)(((n0 * a.Cpi + c) * a.Hi + iy) * a.Wi + ix) * ES : kOutOfRange, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b0 + u * nthr;
          if (idx < ITEMS) ((typename Elem<T>::raw_t*)lds)[(idx / 33) * IPITCH + idx % 33] = v[u];
        }
      }
    } else {
    constexpr int ITEMS = ROWS * CW * XQ;
    auto stage = [&](auto u_tag) {
      constexpr int U = decltype(u_tag)::value;       // loads in flight per thread
      for (int b0 = t; b0 < ITEMS; b0 += nthr * U) {
        uint4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b0 + u * nthr;
          const int px = idx / XQ, q = idx - px * XQ;
          const int i = px / CW, cc = px - i * CW;
          const int im = two ? n0 + cc / (8 * S) : n0;
          const int ix = two ? cc % (8 * S) : j0 * S + cc;
          const int iy = iy0 + i;
          const bool in = (idx < ITEMS) & ((unsigned)iy < (unsigned)a.H) & (ix < a.W) & (im < a.N) & (q * EPI < a.Cpi);
          v[u] = load_b128(xr, in ? (unsigned)(((im * a.H + iy) * a.W + ix) * a.Cpi + q * EPI) * ES : kOutOfRange, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idx = b0 + u * nthr;
          if (idx < ITEMS) *(uint4*)&lds[(idx / XQ) * XP + (idx % XQ) * 16] = v[u];
        }
      }
    };
    constexpr int ONE = (ITEMS + 63) / 64;
    if (ks == 1) stage(std::integral_constant<int, (ONE > 20 ? 20 : ONE)>{});
    else stage(std::integral_constant<int, 10>{});
    }
  }

  // depthwise weights: byte offset of the lane's channels, out of range for taps outside the image
  unsigned w_off[K];
#pragma unroll
  for (int v = 0; v < K; ++v)
    w_off[v] = (unsigned)(cj * S + v - PAD) < (unsigned)a.W ? (unsigned)(g4 * 4 * NH * (W32 ? 4 : ES)) : kOutOfRange;
  // XH = 0: byte offset of the lane's pixel(s) in row 0 of the strip
  int x_base[S];
  if constexpr (!EXP) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int ix = cj * S + s;
      x_base[s] = (img < a.N && ix < a.W) ? (((img * a.H + iy0) * a.W + ix) * a.Cpe + g4 * EPI) * ES : -1;
    }
  }
  const bool x_ok0 = (img < a.N) & (cj * S < a.W), x_ok1 = (img < a.N) & (cj * S + 1 < a.W);

  const float lo_e = a.act_e == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi_e = a.act_e == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  const float lo_d = a.act_dw == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi_d = a.act_dw == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();

  // the projection's bias opens the sums (of the strip's first wavefront)
  float4_t bias[MB], acc[R][MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) bias[m] = load_bias4(a.bp, wave == 0 ? a.O : 0, o0 + m * 16 + 4 * g4);
#pragma unroll
  for (int y = 0; y < R; ++y)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[y][m] = bias[m];

  uint4 pre[EXP ? 1 : ROWS][S];                // XH = 0: the rows of a chunk, asked for one chunk ahead
  auto load_row = [&](int c, int i) {
    const int iy = iy0 + i;
    const bool in = ((unsigned)iy < (unsigned)a.H) & (c * 4 * EPI + g4 * EPI < a.Cpe);
#pragma unroll
    for (int s = 0; s < S; ++s)
      pre[EXP ? 0 : i][s] = load_b128(xr, in & (s ? x_ok1 : x_ok0) ? (unsigned)(x_base[s] + i * a.W * a.Cpe * ES) : kOutOfRange,
                                      (unsigned)c * 64u);
  };
  if constexpr (!EXP) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) load_row(wave, i);
  }
  const unsigned char* xl = lds + S * r * XP + g4 * 16;
  // IMG: where the lane's terms of a window lie in the staged image, k = (channel, row, column); terms past the last are zero
  int i_off[IMG ? XR * EPI : 1];
  bool i_ok[IMG ? XR * EPI : 1];
  if constexpr (IMG) {
#pragma unroll
    for (int q = 0; q < XR * EPI; ++q) {
      const int k = (q / EPI) * 4 * EPI + g4 * EPI + q % EPI, c = k / 9, u = (k - c * 9) / 3;
      i_ok[q] = k < a.Cpi * 9;
      i_off[q] = i_ok[q] ? (c * IROWS + u) * IPITCH + k - c * 9 - u * 3 + 2 * r : 0;
    }
  }
  auto window = [&](int i, int j) -> uint4 {
    T v[EPI];
#pragma unroll
    for (int e = 0; e < EPI; ++e) {
      const T w = ((const T*)lds)[2 * i * IPITCH + i_off[IMG ? j * EPI + e : 0]];
      v[e] = i_ok[IMG ? j * EPI + e : 0] ? w : (T)0.0f;
    }
    return *(const uint4*)v;
  };
  // Weights of one block of 16 channels (chunk c, block h), carried in registers: those of the next block are asked for as
  // soon as the last row has used the present ones.
  typedef typename std::conditional<W32, uint4, uint2>::type Quad;     // four channels
  Quad wq[K][K];
  uint4 ae[EXP ? XR : 1], ap[MB];
  uint2 ae_last;
  float4_t be, bd;
  auto first_channel = [&](int c, int h) -> int { return c * 16 * NH + g4 * 4 * NH + h * 4; };   // the lane's four
  auto load_taps = [&](int c, int h, int u) {
    const unsigned inval = (unsigned)(first_channel(c, h) >= a.Cpe) << 31;
#pragma unroll
    for (int v = 0; v < K; ++v) {
      const unsigned soff = (unsigned)(((u * K + v) * a.Cpe + c * 16 * NH + h * 4) * (W32 ? 4 : ES));
      if constexpr (W32) wq[u][v] = load_b128(dr, w_off[v] | inval, soff);
      else wq[u][v] = load_b64(dr, w_off[v] | inval, soff);
    }
  };
  auto load_expand = [&](int c, int h) {
    if constexpr (EXP) {
      const unsigned off = c < a.nchunk ? 0u : kOutOfRange, base = (unsigned)(c * NH + h) * (XH * 512u);
#pragma unroll
      for (int j = 0; j < XR; ++j) ae[j] = load_b128(er, off | (unsigned)lane * 16u, base + j * 1024u);
      if constexpr (XH & 1) ae_last = load_b64(er, off | (unsigned)lane * 8u, base + XR * 1024u);
      be = load_bias4(a.be, a.Ce, first_channel(c, h));
    }
  };
  auto load_project = [&](int c) {
    const unsigned off = c < a.nchunk ? 0u : kOutOfRange;
#pragma unroll
    for (int m = 0; m < MB; ++m)
      ap[m] = load_b128(pr, o0 + m * 16 < a.O ? off | (unsigned)lane * 16u : kOutOfRange,
                        (unsigned)((blockIdx.y * MB + m) * a.nchunk + c) * 1024u);
  };
  load_expand(wave, 0);
  bd = load_bias4(a.bdw, a.Ce, first_channel(wave, 0));
  if constexpr (AHEAD) {
#pragma unroll
    for (int u = 0; u < K; ++u) load_taps(wave, 0, u);
  }
  load_project(wave);
  if constexpr (EXP) __syncthreads();
  uint4 xb[S][READ_AHEAD ? XR : 1];            // operands of the row that is expanded next
  auto operands = [&](int i) {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int j = 0; j < XR; ++j) {
        if constexpr (IMG) xb[s][j] = window(i, j);
        else xb[s][j] = *(const uint4*)&xl[(i * CW + s) * XP + j * 64];
      }
  };
  if constexpr (READ_AHEAD) operands(0);

  for (int c = wave; c < a.nchunk; c += ks) {
    uint2 bq[ES == 4 ? 1 : R];                 // 16-bit data: finished rows of the chunk's first half
    auto half = [&](auto h_tag) {
      constexpr int h = decltype(h_tag)::value;
      const int cn = h == NH - 1 ? c + ks : c, hn = h == NH - 1 ? 0 : h + 1;      // the next block
      if constexpr (!AHEAD) {
#pragma unroll
        for (int u = 0; u < K; ++u) load_taps(c, h, u);
      }
      float4_t wd[K][K];
#pragma unroll
      for (int u = 0; u < K; ++u)
#pragma unroll
        for (int v = 0; v < K; ++v) {
          if constexpr (W32) wd[u][v] = __builtin_bit_cast(float4_t, wq[u][v]);
          else wd[u][v] = widen4<T>(wq[u][v]);
        }
      float4_t dacc[R];
#pragma unroll
      for (int y = 0; y < R; ++y) dacc[y] = bd;
      bd = load_bias4(a.bdw, a.Ce, first_channel(cn, hn));
      float4_t e[S];
      // step i: row i is expanded while the row before it is multiplied into its output rows.  The scheduler may mix
      // these two, but not reach further (it would hold every row's operands at once).
#pragma unroll
      for (int i = 0; i <= ROWS; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        float4_t en[S];
        if (EXP && i < ROWS) {
          const bool in = (unsigned)(iy0 + i) < (unsigned)a.H;
          const float lo = in ? lo_e : 0.0f, hi = in ? hi_e : 0.0f;     // a row outside the image: zeros
#pragma unroll
          for (int s = 0; s < S; ++s) {
            float4_t ev = be;
#pragma unroll
            for (int j = 0; j < XR; ++j) {
              uint4 b;
              if constexpr (READ_AHEAD) b = xb[s][j];
              else if constexpr (IMG) b = window(i, j);
              else b = *(const uint4*)&xl[(i * CW + s) * XP + j * 64];
              float4_t d[1][1] = {{ev}};
              const uint4 aa[1] = {ae[j]}, bb[1] = {b};
              mma_slab<T, 1, 1, 1>(aa, bb, d);
              ev = d[0][0];
            }
            if constexpr (XH & 1) {
              const uint2 b = *(const uint2*)&xl[(i * CW + s) * XP + XR * 64 - g4 * 8];
              ev = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(ae_last.x), __uint_as_float(b.x), ev, 0, 0, 0);
              ev = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(ae_last.y), __uint_as_float(b.y), ev, 0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) ev[q] = __builtin_amdgcn_fmed3f(ev[q], lo, hi);
            if constexpr (ES == 2) ev = widen4<T>(narrow4<T>(ev));
            en[s] = ev;
          }
          if constexpr (READ_AHEAD) operands(i + 1 < ROWS ? i + 1 : 0);
        } else if (i < ROWS) {
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const uint4 q = pre[i][s];
            if constexpr (ES == 4) en[s] = __builtin_bit_cast(float4_t, q);
            else en[s] = widen4<T>(h ? make_uint2(q.z, q.w) : make_uint2(q.x, q.y));
          }
          if constexpr (h == NH - 1) {
            load_row(c + ks, i);             // (past the last chunk: zeros, without a branch)
          }
        }
        if (i > 0) {
          const int ir = i - 1;
#pragma unroll
          for (int u = 0; u < K; ++u) {
            if ((ir - u) % S != 0 || ir < u || (ir - u) / S >= R) continue;
            const int y = (ir - u) / S;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float d = dacc[y][q];
              if constexpr (S == 1) {
                if constexpr (K == 5) d = fmaf(row_shift<-2>(e[0][q]), wd[u][0][q], d);
                d = fmaf(row_shift<-1>(e[0][q]), wd[u][PAD - 1][q], d);
                d = fmaf(e[0][q], wd[u][PAD][q], d);
                d = fmaf(row_shift<1>(e[0][q]), wd[u][PAD + 1][q], d);
                if constexpr (K == 5) d = fmaf(row_shift<2>(e[0][q]), wd[u][K - 1][q], d);
              } else {
                if constexpr (K == 5) d = fmaf(row_shift<-1>(e[0][q]), wd[u][0][q], d);
                d = fmaf(row_shift<-1>(e[S - 1][q]), wd[u][PAD - 1][q], d);
                d = fmaf(e[0][q], wd[u][PAD][q], d);
                d = fmaf(e[S - 1][q], wd[u][PAD + 1][q], d);
                if constexpr (K == 5) d = fmaf(row_shift<1>(e[0][q]), wd[u][K - 1][q], d);
              }
              dacc[y][q] = d;
            }
          }
          if (ir >= K - 1 && (ir - (K - 1)) % S == 0) {            // output row y is complete
            const int y = (ir - (K - 1)) / S;
            float4_t o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = __builtin_amdgcn_fmed3f(dacc[y][q], lo_d, hi_d);
            uint4 bo;
            if constexpr (ES == 4) bo = __builtin_bit_cast(uint4, o);
            else {
              const uint2 p = narrow4<T>(o);
              if constexpr (h == 0) bq[y] = p;
              else bo = make_uint4(bq[y].x, bq[y].y, p.x, p.y);
            }
            if constexpr (h == NH - 1) {
              const uint4 bb[1] = {bo};
              float4_t d[MB][1];
#pragma unroll
              for (int m = 0; m < MB; ++m) d[m][0] = acc[y][m];
              mma_slab<T, MB, 1, MB>(ap, bb, d);
#pragma unroll
              for (int m = 0; m < MB; ++m) acc[y][m] = d[m][0];
            }
          }
        }
        if (i < ROWS) {
#pragma unroll
          for (int s = 0; s < S; ++s) e[s] = en[s];
        }
        if (i == ROWS - 1) load_expand(cn, hn);
#pragma unroll
        for (int u = 0; u < K; ++u)
          if (AHEAD && i - 1 == (R - 1) * S + u) load_taps(cn, hn, u);
        if (i == ROWS && h == NH - 1) load_project(cn);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    half(std::integral_constant<int, 0>{});
    if constexpr (NH == 2) half(std::integral_constant<int, 1>{});
  }

  mbrow_finish<T, R, MB>(a, at, lds, acc);
}

// LDS of a work-group: the strip's input, later the sums of `slots` wavefronts
template <typename T, int K, int S, int MB, int XH, int R, bool IMG>
inline int launch_mbrow_rows(dim3 grid, int ks, hipStream_t s, MbArgs a) {
  constexpr int strip = IMG ? 3 * (2 * (R + 2) + 1) * mbrow_image_pitch((int)sizeof(T)) * (int)sizeof(T)
                            : ((R - 1) * S + K) * 16 * S * (XH ? XH * 32 + 16 : 0);
  constexpr int slot = R * MB * 1024;
  static_assert(strip <= 160 * 1024 && 4 * slot <= 160 * 1024, "LDS budget");
  a.slots = ks > 4 ? 4 : ks;
  const int red = ks > 1 ? a.slots * slot : 0;
  const int bytes = strip > red ? strip : red;
  if (bytes > 65536) {   // more than the default 64 KiB has to be asked for once
    static std::atomic<bool> raised{false};
    if (!raised.load(std::memory_order_relaxed)) {
      CPRUNE_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&mbrow_kernel<T, K, S, MB, XH, R, IMG>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
      raised.store(true, std::memory_order_relaxed);
    }
  }
  hipLaunchKernelGGL((mbrow_kernel<T, K, S, MB, XH, R, IMG>), grid, dim3(64 * ks), bytes, s, a);
  return CPRUNE_OK;
}

template <typename T, int K, int S, int MB, int XH, bool IMG = false>
inline int launch_mbrow_one(int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  constexpr int R0 = mbrow_rows(K, S, MB, 0), R1 = mbrow_rows(K, S, MB, 1);
  if (R0 == R1 || !low) return launch_mbrow_rows<T, K, S, MB, XH, R0, IMG>(grid, ks, s, a);
  return launch_mbrow_rows<T, K, S, MB, XH, R1, IMG>(grid, ks, s, a);
}

// (MB, XH) pairs that are built; XH = 0: depthwise + projection only.  mbrow_form picks one of them.
template <typename T, int K, int S>
inline int launch_mbrow_ks(int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
#define CPRUNE_MBROW(MB_, XH_) \
  if (mb == MB_ && xh == XH_) return launch_mbrow_one<T, K, S, MB_, XH_>(low, grid, ks, s, a);
  if constexpr (sizeof(T) == 4 && K == 3) {      // (up to 96 filters: mbrow3_kernel.hpp)
    CPRUNE_MBROW(8, 0) CPRUNE_MBROW(8, 12)
    return CPRUNE_ERR_UNSUPPORTED;
  } else {
  CPRUNE_MBROW(1, 0) CPRUNE_MBROW(2, 0) CPRUNE_MBROW(4, 0) CPRUNE_MBROW(6, 0) CPRUNE_MBROW(8, 0)
  if constexpr (sizeof(T) == 4) {
    CPRUNE_MBROW(2, 2) CPRUNE_MBROW(2, 3) CPRUNE_MBROW(2, 4)
    CPRUNE_MBROW(4, 4) CPRUNE_MBROW(4, 8) CPRUNE_MBROW(6, 8) CPRUNE_MBROW(6, 12) CPRUNE_MBROW(8, 12)
  } else {
    CPRUNE_MBROW(2, 2) CPRUNE_MBROW(2, 4) CPRUNE_MBROW(4, 2) CPRUNE_MBROW(4, 4) CPRUNE_MBROW(6, 4)
    CPRUNE_MBROW(6, 6) CPRUNE_MBROW(8, 10)
  }
  return CPRUNE_ERR_UNSUPPORTED;
  }
#undef CPRUNE_MBROW
}

// The image form: 27 terms in one 32-byte unit per 8 (16) numbers.
template <typename T>
inline int launch_mbrow_image(int mb, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  constexpr int XH = sizeof(T) == 4 ? 4 : 2;
  if (mb == 1) return launch_mbrow_one<T, 3, 1, 1, XH, true>(low, grid, ks, s, a);
  if (mb == 2) return launch_mbrow_one<T, 3, 1, 2, XH, true>(low, grid, ks, s, a);
  return CPRUNE_ERR_UNSUPPORTED;
}

template <typename T>
inline int launch_mbrow(int k, int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a) {
  if constexpr (sizeof(T) == 2) {      // (fp32: mbrow3_kernel.hpp)
    if (a.Hi > 0) return k == 3 && stride == 1 ? launch_mbrow_image<T>(mb, low, grid, ks, s, a) : CPRUNE_ERR_UNSUPPORTED;
  }
  if (k == 3 && stride == 1) return launch_mbrow_ks<T, 3, 1>(mb, xh, low, grid, ks, s, a);
  if (k == 3 && stride == 2) return launch_mbrow_ks<T, 3, 2>(mb, xh, low, grid, ks, s, a);
  if (k == 5 && stride == 1) return launch_mbrow_ks<T, 5, 1>(mb, xh, low, grid, ks, s, a);
  if (k == 5 && stride == 2) return launch_mbrow_ks<T, 5, 2>(mb, xh, low, grid, ks, s, a);
  return CPRUNE_ERR_UNSUPPORTED;
}

}  // namespace cprune
