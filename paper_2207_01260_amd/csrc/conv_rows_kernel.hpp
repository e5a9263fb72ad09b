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
// registers for them would leave one wavefront per SIMD).  Counters over whole launches (ResNet-18, batch 32): matrix pipes busy 24-33 % of
// the cycles their units have work, wavefronts waiting for memory or the sums' barrier 26-38 % and to issue 28-46 %.
#pragma once
#include "conv_split_kernel.hpp"

namespace cprune {

struct RowsArgs {
  const void* x;        // [n][h][w][cp]
  const void* w;        // launch_repack_wave
  const float* bias;
  const void* res;
  void* y;              // [n][h][w][cop], pooled: [n][h / 2][w / 2][cop]
  int N, H, W, O, Cp, Cop;         // H, W: the output map
  int tiles_y, tiles_x, tiles_m;   // strips of a map, filter tiles
  int strips;                      // of the whole batch
  int lane_shift;                  // lanes per image: 1 << lane_shift
  int step;                        // columns from strip to strip: 16, or 14 (12 with a pool) where strips overlap (fp32), 15 at stride 2
  int m_major;                     // 0: filter tiles run fastest; otherwise slowest, and the work-groups of one filter tile
  unsigned magic_m, magic_x, magic_y;   // (magic_m: of m_major where that is set)
  unsigned x_bytes, w_bytes, y_bytes;
  int nchunk;                      // chunks of 32 channels
  int act, pool;
  const void* w_raw;               // fp32: [o][9][cp], and its size
  unsigned w_raw_bytes;
};

// What lies beside a strip's outer lanes: nothing that counts (zeros), columns fetched by its edge lanes, or, where several
// images share the 16 lanes, another image.
enum RowsEdge { kEdgeZero = 0, kEdgeLoad = 1, kEdgeImage = 2 };

// Where a wavefront works.
struct RowsAt {
  int lane, r, g4, slice, sub;     // slice of the reduction, strip of the work-group
  int tile_m, o0;                  // filter tile, its first filter
  int ty, tx, lr, img, cx;         // strip; the lane's place in its image's columns, image, column
  bool live, col_ok, out_ok;       // the strip exists; the lane has a pixel; one that this strip stores
};

template <int MB, int KS>
__device__ __forceinline__ RowsAt rows_at(const RowsArgs& a) {
  constexpr int NS = KS >= 4 ? 1 : 4 / KS;       // strips of a work-group
  RowsAt p;
  const int t = threadIdx.x;
  p.lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  p.slice = wave % KS; p.sub = wave / KS;
  p.r = p.lane & 15; p.g4 = p.lane >> 4;
  int tile;
  {
    const int G = gridDim.x;
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int q = G >> 3, rem = G & 7;
    tile = xcd * q + (xcd < rem ? xcd : rem) + local;
  }
  const int major = (int)fast_div((unsigned)tile, a.magic_m), minor = tile - major * (a.m_major ? a.m_major : a.tiles_m);
  const int group = a.m_major ? minor : major;                     // of NS strips
  p.tile_m = a.m_major ? major : minor;
  p.o0 = p.tile_m * (MB * 16);
  const int strip = group * NS + p.sub;
  const int q_x = (int)fast_div((unsigned)strip, a.magic_x);
  p.tx = strip - q_x * a.tiles_x;
  const int grp = (int)fast_div((unsigned)q_x, a.magic_y);
  p.ty = q_x - grp * a.tiles_y;
  p.lr = p.r & ((1 << a.lane_shift) - 1);
  p.img = (grp << (4 - a.lane_shift)) + (p.r >> a.lane_shift);
  p.cx = p.tx * a.step + p.lr;
  p.live = strip < a.strips;
  p.col_ok = p.live & (p.img < a.N) & (p.cx < a.W);
  // columns whose neighbours, or pool windows, lie in the strip before and behind (at stride 2 only the one before is missed)
  const int before = (17 - a.step) >> 1, behind = (16 - a.step) >> 1;
  p.out_ok = p.col_ok & ((p.tx == 0) | (p.lr >= before)) & ((p.tx == a.tiles_x - 1) | (p.lr < 16 - behind));
  return p;
}

// Sums of KS wavefronts, bias, shortcut, activation, store: four filters of a pixel, or of the maximum of a 2x2 window.
template <typename T, int MB, int R, int KS>
__device__ __forceinline__ void rows_finish(const RowsArgs& a, const RowsAt& p, float4_t (&acc)[R][MB]) {
  constexpr int ES = (int)sizeof(T);
  constexpr int NS = KS >= 4 ? 1 : 4 / KS;
  constexpr int SLOTS = KS > 4 ? 4 : KS;
  __shared__ __attribute__((aligned(16))) float4_t xch[KS > 1 ? NS * SLOTS * R * MB * 64 : 1];
  typedef typename std::conditional<ES == 4, uint4, uint2>::type Quad;     // four numbers
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.res, a.res ? a.y_bytes : 0u);
  const float lo = a.act == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi = a.act == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  auto at = [&](int y, int m) -> unsigned {
    const int oy = p.ty * R + y, o = p.o0 + m * 16 + 4 * p.g4;
    const bool ok = p.out_ok & (oy < a.H) & (o < a.Cop);
    if (a.pool) return ok & ((p.cx & 1) == 0) ? (unsigned)(((p.img * (a.H >> 1) + (oy >> 1)) * (a.W >> 1) + (p.cx >> 1)) * a.Cop + o) * ES : kOutOfRange;
    return ok ? (unsigned)(((p.img * a.H + oy) * a.W + p.cx) * a.Cop + o) * ES : kOutOfRange;
  };
  auto widen = [&](Quad q) -> float4_t {
    if constexpr (ES == 4) return __builtin_bit_cast(float4_t, q);
    else {
      const T* h = reinterpret_cast<const T*>(&q);
      return (float4_t){Elem<T>::to_f32(h[0]), Elem<T>::to_f32(h[1]), Elem<T>::to_f32(h[2]), Elem<T>::to_f32(h[3])};
    }
  };
  typedef unsigned int uint32x2_t __attribute__((ext_vector_type(2)));
  auto load_res = [&](unsigned off) -> Quad {
    if constexpr (ES == 4) return load_b128(rr, off, 0);
    else {
      const uint32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(rr, (int)off, 0, 0);
      return make_uint2(v.x, v.y);
    }
  };
  auto clamp4 = [&](float4_t v) -> float4_t {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = __builtin_amdgcn_fmed3f(v[q], lo, hi);
    return v;
  };
  auto store = [&](unsigned off, float4_t v) {
    if (off == kOutOfRange) return;
    if constexpr (ES == 4) *(float4_t*)((char*)a.y + off) = v;
    else {
      T h[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = Elem<T>::from_f32(v[q]);
      *(uint2*)((char*)a.y + off) = *(const uint2*)h;
    }
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
      const float4_t bias = load_bias4(a.bias, a.O, p.o0 + m * 16 + 4 * p.g4);
      Quad res[R];
      if (a.res) {
#pragma unroll
        for (int y = 0; y < R; ++y) res[y] = load_res(at(y, m));
      }
#pragma unroll
      for (int y = 0; y < R; y += 2) {
        if (R % 2 == 0 && a.pool) {
          store(at(y, m), window(clamp4(acc[y][m] + bias), clamp4(acc[y + (R % 2 == 0)][m] + bias)));
        } else {
#pragma unroll
          for (int z = y; z < y + 2 && z < R; ++z) {
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
    float4_t* const mine = xch + p.sub * (SLOTS * SLOT) + p.lane;
    int nw = KS;
#pragma unroll
    for (int level = KS; level > SLOTS; level >>= 1) {
      const int hw = level >> 1;
      if (p.slice >= hw && p.slice < level) {
#pragma unroll
        for (int q = 0; q < R * MB; ++q) mine[(p.slice - hw) * SLOT + q * 64] = acc[q / MB][q % MB];
      }
      __syncthreads();
      if (p.slice < hw) {
#pragma unroll
        for (int q = 0; q < R * MB; ++q) acc[q / MB][q % MB] += mine[p.slice * SLOT + q * 64];
      }
      __syncthreads();
      nw = hw;
    }
    if (p.slice < nw) {
#pragma unroll
      for (int q = 0; q < R * MB; ++q) mine[p.slice * SLOT + q * 64] = acc[q / MB][q % MB];
    }
    __syncthreads();
    for (int q = p.slice; q < (R + 1) / 2 * MB; q += KS) {
      const int y = 2 * (q / MB), m = q % MB;
      const float4_t bias = load_bias4(a.bias, a.O, p.o0 + m * 16 + 4 * p.g4);
      Quad res[2];
      const bool two = R % 2 == 0 || y + 1 < R;
      if (a.res) { res[0] = load_res(at(y, m)); if (two) res[1] = load_res(at(y + 1, m)); }
      float4_t s[2];
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const float4_t* const src = mine + ((y + (two ? z : 0)) * MB + m) * 64;
        s[z] = src[0];
#pragma unroll
        for (int w = 1; w < SLOTS; ++w) s[z] += src[w * SLOT];
        s[z] += bias;
        if (a.res) s[z] += widen(res[two ? z : 0]);
        s[z] = clamp4(s[z]);
      }
      if (R % 2 == 0 && a.pool) store(at(y, m), window(s[0], s[1]));
      else { store(at(y, m), s[0]); if (two) store(at(y + 1, m), s[1]); }
    }
  }
}

template <typename T, int MB, int R, int KS, int EDGE>
__global__ __launch_bounds__(KS == 8 ? 512 : 256, 2) void conv_rows_kernel(RowsArgs a) {
  static_assert(sizeof(T) == 2, "16-bit data");
  constexpr bool HALO = EDGE == kEdgeLoad;
  constexpr int ROWS = R + 2;
  constexpr int PF = R == 8 ? 5 : R == 7 || MB > 2 ? 3 : 6;   // rows asked for ahead
  static_assert(ROWS % PF == 0, "ring of rows");
  const RowsAt at = rows_at<MB, KS>(a);
  const int lane = at.lane, r = at.r, g4 = at.g4, slice = at.slice, tile_m = at.tile_m, o0 = at.o0, lr = at.lr, img = at.img, cx = at.cx;
  const int iy0 = at.ty * R - 1;
  const bool live = at.live, col_ok = at.col_ok;

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
      else if constexpr (EDGE == kEdgeImage) return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true) & (left ? ml : mr);
      else return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true);
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

  rows_finish<T, MB, R, KS>(a, at, acc);
}

// The same for fp32 data: every number is cut into three bf16 parts and six of the nine products are multiplied (as in
// conv_split_kernel, whose notes on error and range hold here too), weights packed by launch_pack_split in whole chunks of 32
// channels.  A row is cut in registers once per wavefront: some 70 vector operations beside 54 MFMAs per 16 filters and
// output rows it touches.  The first product of a pair has an accumulator of its
// own and the five small ones share another, over the whole reduction: one rounding of the sum per 32 terms.  Strips of a
// map wider than 16 overlap by two columns (14 of 16 are stored; four with a pool): edge columns of their own would have to be cut as well.
//
// Measured, the best other kernel / this one (us), batch 32: 512 -> 411 at 7x7 52 / 38, 173 -> 256 at 14x14 36.2 / 28.6, 256 -> 87 26 /
// 19.6, 128 -> 85 at 28x28 38.5 / 30.1, 64 -> 28 at 56x56 26.5 / 22.9, 40 -> 64 33.5 / 38.8 (a second chunk of 8 real channels of 32); batch
// 64: 209 -> 197 at 8x8 25.6 / 19.9, 360 -> 360 at 4x4 25.4 / 20.0, 56 -> 56 at 32x32 25.5 / 31 (strips of 14 waste a third).  Alone
// on its SIMD a wavefront takes 3.7 us per chunk of 8 rows, 2.9 of it MFMA issue; the rest is the wait for the next chunk's
// weights.  Cutting a row in front of its MFMAs instead of between those of the row before: 4.4 us.  Counters over whole launches (ResNet-18,
// batch 32): matrix pipes busy 46-61 %, vector ALU 40-50 %, wavefronts waiting for memory 17-23 % and to issue 27-44 %.
template <int R, int KS, bool IMAGES>
__global__ __launch_bounds__(KS == 8 ? 512 : 256, 2) void conv_split_rows_kernel(RowsArgs a) {
  constexpr int ROWS = R + 2, PF = R == 7 ? 3 : 2;
  static_assert(ROWS % PF == 0, "ring of rows");
  const RowsAt at = rows_at<1, KS>(a);
  const int lane = at.lane, r = at.r, g4 = at.g4, slice = at.slice, o0 = at.o0, lr = at.lr, img = at.img, cx = at.cx;
  const int iy0 = at.ty * R - 1;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);
  const int row_bytes = a.W * a.Cp * 4;
  const int x_off = ((img * a.H + iy0) * a.W + cx) * a.Cp * 4 + g4 * 32;
  const unsigned ml = lr > 0 ? ~0u : 0u, mr = lr < (1 << a.lane_shift) - 1 ? ~0u : 0u;

  uint4 pre[PF][2];
  auto load_row = [&](int c, int i, int slot) {
    const bool in = (unsigned)(iy0 + i) < (unsigned)a.H;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const bool ch = c * 32 + g4 * 8 + e * 4 < a.Cp;
      pre[slot][e] = load_b128(xr, in & ch & at.col_ok ? (unsigned)(x_off + i * row_bytes + e * 16) : kOutOfRange, (unsigned)c * 128u);
    }
  };
  uint4 wt[3][3][3];               // window row, column, part
  auto load_taps = [&](int c, int u) {
    const unsigned past = c < a.nchunk ? 0u : kOutOfRange;
#pragma unroll
    for (int v = 1; v < 4; ++v)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        wt[u][v % 3][p] = load_b128(wr, past | (unsigned)lane * 16u, (unsigned)(((at.tile_m * a.nchunk + c) * 9 + u * 3 + v % 3) * 3 + p) * 1024u);
  };
  float4_t acc[R][1], small[R];
#pragma unroll
  for (int y = 0; y < R; ++y) acc[y][0] = small[y] = (float4_t){0.f, 0.f, 0.f, 0.f};

  struct Cut { uint4 p[3]; };
  auto cut = [&](const uint4 (&q)[2]) -> Cut {
    uint32_t h[4], m[4], l[4];
    split3(q[0].x, q[0].y, h[0], m[0], l[0]); split3(q[0].z, q[0].w, h[1], m[1], l[1]);
    split3(q[1].x, q[1].y, h[2], m[2], l[2]); split3(q[1].z, q[1].w, h[3], m[3], l[3]);
    return Cut{{make_uint4(h[0], h[1], h[2], h[3]), make_uint4(m[0], m[1], m[2], m[3]), make_uint4(l[0], l[1], l[2], l[3])}};
  };
  auto shifted = [&](const Cut& x, auto left_tag) -> Cut {
    constexpr bool left = decltype(left_tag)::value;
    constexpr int ctrl = left ? 0x111 : 0x101;
    auto one = [&](unsigned v) -> unsigned {
      const unsigned n = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true);
      return IMAGES ? n & (left ? ml : mr) : n;
    };
    Cut s;
#pragma unroll
    for (int p = 0; p < 3; ++p) s.p[p] = make_uint4(one(x.p[p].x), one(x.p[p].y), one(x.p[p].z), one(x.p[p].w));
    return s;
  };

  // Row i + 1 is cut while row i is multiplied; its place in the ring of raw rows then takes row i + 1 + PF.  (What the loop
  // finds in flight is asked for here in the order of its last steps, so that the waits at its head count the same loads.)
  load_row(slice, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_taps(slice, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_row(slice, 1, 1);
  __builtin_amdgcn_sched_barrier(0);
  load_taps(slice, 1);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (PF == 3) load_row(slice, 2, 2);
  Cut x = cut(pre[0]);
  load_row(slice, PF, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_taps(slice, 2);
  __builtin_amdgcn_sched_barrier(0);

  for (int c = slice; c < a.nchunk; c += KS) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const int slot = (i + 1) % PF;
      Cut nx;
      auto cut_next = [&](auto apart) {
        uint4 q[2] = {pre[slot][0], pre[slot][1]};
        if constexpr (decltype(apart)::value) {      // (opaque: otherwise the compiler moves what both branches do before them)
#pragma unroll
          for (int k = 0; k < 2; ++k) asm("" : "+v"(q[k].x), "+v"(q[k].y), "+v"(q[k].z), "+v"(q[k].w));
        }
        nx = cut(q);
      };
      if ((unsigned)(iy0 + i) < (unsigned)a.H) {
        auto column = [&](const Cut& b, int v) {
          auto term = [&](int pw, int px, bool big) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
              if (i - u < 0 || i - u >= R) continue;
              float4_t& d = big ? acc[i - u][0] : small[i - u];
              d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wt[u][v][pw]), __builtin_bit_cast(bf16x8_t, b.p[px]),
                                                          d, 0, 0, 0);
            }
          };
          term(0, 2, false); term(0, 0, true); term(2, 0, false); term(1, 1, false); term(0, 1, false); term(1, 0, false);
        };
        column(x, 1);
        column(shifted(x, std::false_type{}), 2);
        column(shifted(x, std::true_type{}), 0);
        cut_next(std::false_type{});
        // vector operations between the MFMAs, not in front of them
        constexpr int hits = 3;
#pragma unroll
        for (int k = 0; k < 18 * hits; ++k) {
          if (k >= 18 * ((i < 2 ? i + 1 : hits) - (i >= R ? i - R + 1 : 0))) break;
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        }
      } else {
        cut_next(std::true_type{});
      }
      x = nx;
      __builtin_amdgcn_sched_barrier(0);
      if (i + 1 + PF < ROWS) load_row(c, i + 1 + PF, slot);
      else load_row(c + KS, i + 1 + PF - ROWS, slot);
      if (i >= R - 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (i == R - 1 + u) load_taps(c + KS, u);
    }
  }
#pragma unroll
  for (int y = 0; y < R; ++y) acc[y][0] += small[y];

  // data that three parts do not hold shows in the sums (see conv_split_kernel): then the slice once more on the fp32
  // instruction, operands straight from memory
  constexpr uint32_t kInf = 0x7f800000u, kSmall = (127u - 50u) << 23;
  uint32_t odd = 0;
#pragma unroll
  for (int y = 0; y < R; ++y)
#pragma unroll
    for (int q = 0; q < 4; ++q) odd = max(odd, (__float_as_uint(acc[y][0][q]) << 1) - (kSmall << 1));
  if (__any(odd >= (kInf - kSmall) << 1)) {
    uint32_t top = 0, low = ~0u;
#pragma unroll
    for (int y = 0; y < R; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t mag = __float_as_uint(acc[y][0][q]) & 0x7fffffffu;
        top = max(top, mag);
        low = min(low, mag - 1);      // (zero goes to the other end)
      }
    if (__any(top >= kInf || low < kSmall - 1)) {
      const __amdgpu_buffer_rsrc_t ww = make_rsrc(a.w_raw, a.w_raw_bytes);
#pragma unroll
      for (int y = 0; y < R; ++y) acc[y][0] = (float4_t){0.f, 0.f, 0.f, 0.f};
      for (int c = slice; c < a.nchunk; c += KS)
        for (int tap = 0; tap < 9; ++tap) {
          const int u = tap / 3, ix = cx + tap - u * 3 - 1;
          const bool col = at.live & (img < a.N) & ((unsigned)ix < (unsigned)a.W);
          for (int ch = c * 32 + g4; ch < c * 32 + 32; ch += 4) {
            const bool real = ch < a.Cp;
            const float wv = __uint_as_float(Elem<float>::load(ww, real & (o0 + r < a.O) ? (unsigned)(((o0 + r) * 9 + tap) * a.Cp + ch) * 4u : kOutOfRange, 0));
#pragma unroll
            for (int y = 0; y < R; ++y) {
              const int iy = at.ty * R + y + u - 1;
              const bool in = real & col & ((unsigned)iy < (unsigned)a.H);
              const float xv = __uint_as_float(Elem<float>::load(xr, in ? (unsigned)(((img * a.H + iy) * a.W + ix) * a.Cp + ch) * 4u : kOutOfRange, 0));
              acc[y][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, xv, acc[y][0], 0, 0, 0);
            }
          }
        }
    }
  }
  rows_finish<float, 1, R, KS>(a, at, acc);
}

// Variants: id, 16-filter blocks, rows of a strip, wavefronts that share a strip (fp32: those of one block)
#define CPRUNE_ROWS_LIST(X) \
  X(0, 2, 8, 1) X(1, 2, 8, 2) X(2, 2, 8, 4)                          \
  X(3, 2, 4, 1) X(4, 2, 4, 2) X(5, 2, 4, 4) X(6, 2, 4, 8)            \
  X(7, 3, 4, 1) X(8, 4, 4, 1) X(9, 1, 8, 1)                          \
  X(10, 1, 4, 2) X(11, 1, 4, 4) X(12, 1, 4, 8)                       \
  X(13, 1, 8, 2) X(14, 1, 8, 4) X(15, 1, 4, 1)

constexpr int kNumRows = 16;

// Strips of seven rows (no fused pool): the maps of ImageNet networks are 7 x 2^n high.  Eight rows compute an eighth too much on 7 and 14, and
// on 56 x 56 at batch 32 leave 2.6 wavefronts to a SIMD where seven give exactly three of an eighth less.  The ring of nine input rows is three
// deep.  Eight rows -> seven, us, the best of each at batch 32: fp32 64->40 at 56x56 31.7 -> 29.5, 85->128 at 28x28 30.4 -> 28.2, 173->256 at
// 14x14 29.2 -> 26.7, 512->411 at 7x7 34.0 -> 32.8; bf16 14.4 -> 12.9, 11.9 -> 9.8, 9.1 -> 8.4, 10.5 -> 9.6.  They lose on powers of two (fp32
// 209->197 at 8x8, batch 64: 20.0 -> over 23.8; 56->55 at 16x16 9.4 -> 12.0), so both stay and a handle times both; without timing the choice
// is among the sixteen above, as before.  Counters, ResNet-18 at batch 32: fp32 matrix pipes busy 59 %, vector ALU 48 %, waiting for memory 19 % and to issue 42;
// bf16 28, 23, 35 and 33.
#define CPRUNE_ROWS7_LIST(X) X(0, 1, 7, 1) X(1, 1, 7, 2) X(2, 1, 7, 4) X(3, 2, 7, 1) X(4, 2, 7, 2) X(5, 2, 7, 4)

constexpr int kNumRows7 = 6;

inline RowsEdge rows_edge(const RowsArgs& a) {
  return a.lane_shift < 4 ? kEdgeImage : a.tiles_x > 1 && a.step == 16 ? kEdgeLoad : kEdgeZero;
}

template <typename T>
inline int launch_rows(int id, dim3 grid, hipStream_t s, const RowsArgs& a) {
  const RowsEdge edge = rows_edge(a);
#define CPRUNE_ROWS_CASE(ID, MB_, R_, KS_)                                                                           \
  case ID: {                                                                                                         \
    const dim3 block(KS_ == 8 ? 512 : 256);                                                                          \
    if (edge == kEdgeLoad) hipLaunchKernelGGL((conv_rows_kernel<T, MB_, R_, KS_, kEdgeLoad>), grid, block, 0, s, a); \
    else if (edge == kEdgeImage) hipLaunchKernelGGL((conv_rows_kernel<T, MB_, R_, KS_, kEdgeImage>), grid, block, 0, s, a); \
    else hipLaunchKernelGGL((conv_rows_kernel<T, MB_, R_, KS_, kEdgeZero>), grid, block, 0, s, a);                   \
    break;                                                                                                           \
  }
  switch (id) { CPRUNE_ROWS_LIST(CPRUNE_ROWS_CASE) default: break; }
  if (id < kNumRows) return CPRUNE_OK;
  switch (id - kNumRows) { CPRUNE_ROWS7_LIST(CPRUNE_ROWS_CASE) default: return CPRUNE_ERR_UNSUPPORTED; }
#undef CPRUNE_ROWS_CASE
  return CPRUNE_OK;
}

// (a template like the other: its kernels are compiled where it is called, not in every file that includes this one)
template <typename T>
inline int launch_rows3(int id, dim3 grid, hipStream_t s, const RowsArgs& a) {
#define CPRUNE_ROWS_CASE(ID, MB_, R_, KS_)                                                                           \
  case ID:                                                                                                           \
    if constexpr (MB_ == 1 && std::is_same<T, float>::value) {                                                       \
      const dim3 block(KS_ == 8 ? 512 : 256);                                                                        \
      if (a.lane_shift < 4) hipLaunchKernelGGL((conv_split_rows_kernel<R_, KS_, true>), grid, block, 0, s, a);       \
      else hipLaunchKernelGGL((conv_split_rows_kernel<R_, KS_, false>), grid, block, 0, s, a);                       \
      return CPRUNE_OK;                                                                                              \
    }                                                                                                                \
    break;
  if (id < kNumRows)
    switch (id) { CPRUNE_ROWS_LIST(CPRUNE_ROWS_CASE) default: break; }
  else
    switch (id - kNumRows) { CPRUNE_ROWS7_LIST(CPRUNE_ROWS_CASE) default: break; }
#undef CPRUNE_ROWS_CASE
  return CPRUNE_ERR_UNSUPPORTED;
}

int launch_conv_rows_f32(int id, dim3 grid, hipStream_t s, const RowsArgs& a);
int launch_conv_rows_f16(int id, dim3 grid, hipStream_t s, const RowsArgs& a);
int launch_conv_rows_bf16(int id, dim3 grid, hipStream_t s, const RowsArgs& a);

}  // namespace cprune
