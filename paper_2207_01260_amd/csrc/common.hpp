// Shared host-side declarations of the library's translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bfloat16.h>
#include <stdint.h>
#include <stddef.h>

#include "cprune.h"
#include "split_index.hpp"
#include "strip_index.hpp"

namespace cprune {

void set_last_hip_error(hipError_t e);

#define CPRUNE_HIP_TRY(expr)                         \
  do {                                               \
    hipError_t _e = (expr);                          \
    if (_e != hipSuccess) {                          \
      ::cprune::set_last_hip_error(_e);              \
      return CPRUNE_ERR_DEVICE;                      \
    }                                                \
  } while (0)

// Launch status check that does not synchronise.
#define CPRUNE_LAUNCH_CHECK() CPRUNE_HIP_TRY(hipGetLastError())

inline size_t dtype_size(int dt) { return dt == CPRUNE_F32 ? 4 : 2; }
inline bool dtype_ok(int dt) { return dt == CPRUNE_F32 || dt == CPRUNE_F16 || dt == CPRUNE_BF16; }
inline bool act_ok(int a) { return a == CPRUNE_ACT_NONE || a == CPRUNE_ACT_RELU || a == CPRUNE_ACT_RELU6; }

inline int conv_out_dim(int in, int k, int stride, int pad) { return (in + 2 * pad - k) / stride + 1; }

// ---- dense conv variants -------------------------------------------------
struct TileVariant {
  int wm, wn;   // waves along output channels / pixels (wm * wn == 4)
  int mb, nb;   // 16x16 MFMA blocks per wave along channels / pixels
  int kq;       // MFMA rounds (64 bytes of k per row each) per slab
  int sched;    // scheduling mode: 0 = one tile per work-group, n = runs for n * 256 groups,
                // -1 = 3x3 spatial-patch kernel (one th x tw pixel block per work-group),
                // -2 = reduction-split kernel (16 filters x nb pixel blocks per work-group),
                // -3 = short-reduction 1x1 kernel (persistent groups, filter tile resident in LDS),
                // -4 = independent-wavefront 3x3 kernel (16 filters x wn * nb 4x4 pixel blocks x ks slices of
                //      the reduction per work-group; wn * ks wavefronts of nb blocks each)
  int th = 0, tw = 0, ni = 1, patch_id = -1;
  int blk32 = 0;  // patch kernels: 1 = 32x32 MFMA blocks (patch_id then indexes that kernel's list)
  int ks = 1;     // patch kernels on 16x16 blocks: wave groups per tile; split kernel: wavefronts that share a block
  int kwaves = 0; // reduction-split kernel: wavefronts that share one tile's reduction (patch_id indexes its list)
  int split = 0;  // 1 (with sched = -1): split kernel, any window and stride, fp32 as three bf16 parts
  int rows = 0;   // 1 (with sched = -1): row-strip kernel, 3x3 layers of a handle (2: in the boundary's layout); th = rows of a strip, ks = wavefronts that
                  // share one (patch_id indexes its list)
  int pw3 = 0;    // 1, 2 (deep) (with sched = -1): 1x1 kernel on the 16-bit matrix cores, layers of a handle (patch_id indexes its list)
  int nib = 0;    // split kernel: staging items per thread (patch_id indexes its list)
  int nr = 0;     // short-reduction 1x1 kernel: 64-byte rounds of the reduction its filter tile holds
  int stride = 1; // spatial-patch kernel on 16x16 blocks: the window stride it is built for (patch_id then indexes the
                  // stride-2 list)
  int tile_m() const { return wm * mb * 16; }
  // Filters of the box the variant is pruned by.  A wavefront of the row-strip kernel holds one to four 16-filter blocks and a SIMD
  // two wavefronts; a block less in one of two leaves the layer the time of the other, so one block is never a step: 3x3 on 128
  // channels at 56x56, batch 8, fp32, 128 / 112 / 96 filters on 8 rows 39.4 / 37.7 / 36.6 us, 8 rows shared by two 41.5 / 40.7 / 31.5, 4 rows
  // 43.9 / 42.7 / 33.7; bf16 on 4 rows 21.5 / 21.1 / 16.9.  At stride 2 fp32, batch 32, 4 rows, 128 / 112 / 96 / 80 / 64 filters 80 / 76 / 58 / 59 / 40,
  // batch 8, 2 rows shared by two 28.1 / 27.6 / 21.9 / 21.6 / 15.5; in the boundary's layout, batch 8, 4 rows 56 / 50 / 40 / 40 / 28.
  // Strips of seven rows come out even at 128 filters there (two wavefronts to each SIMD), and a single block shows: 128 / 112 / 96 / 64 filters
  // 36.2 / 33.2 / 32.6 / 21.0, shared by two 38.1 / 35.4 / 28.2 / 20.5: a box of one.
  int step_m() const { return rows && mb == 1 && th != 7 ? 32 : tile_m(); }
  int tile_p() const { return wn * nb * 16; }
};
int num_variants();
const TileVariant& variant(int id);

// Memory layout a dense conv runs in.  nhwc = 0: NCHW activations / OIHW weights (the
// boundary's layout).  nhwc = 1: channels-last inside a network handle, channel strides
// cp_in / cp_out in elements (counts rounded up to one 16-byte vector, except a final
// dense output), weights [c_out][kh][kw][cp_in].
// A 1x1 / stride 2 layer that runs in the launch of a 3x3 / stride 2 / pad 1 layer on the same input (row-strip kernel at stride 2).
struct ConvPair {
  const void* w;        // launch_pack_split, whole chunks
  const void* w_raw;    // [o][cp_in]
  const float* bias;
  void* y;
  int c_out, cp_out, act;
};
struct ConvLayout {
  int nhwc = 0;
  int cp_in = 0;
  int cp_out = 0;
  int nhwc_out = 0;  // with nhwc = 0: NCHW input and OIHW weights (the boundary's layout) but a channels-last
                     // output of channel stride cp_out: the first layer of a network handle
  const void* w_wave = nullptr;  // the weights once more, in the order of the independent-wavefront 3x3
                                 // kernel (launch_repack_wave); that kernel, and the row-strip kernel in 16-bit
                                 // data, run only where this is set
  const void* w_rows = nullptr;  // the weights once more as [16-row tile][64-byte round of the reduction][lane][16
                                 // bytes] (launch_repack_rows): the reduction-split kernel reads these when set
  const void* w_split = nullptr; // channels-last fp32: the weights cut and packed for the split kernel
                                 // (launch_pack_split), which runs only where this is set; a call in the boundary's
                                 // layout packs its weights into the caller's scratch
  const void* w_rows3 = nullptr; // channels-last fp32 3x3 / pad 1, and 1x1 layers of any type: cut and packed in whole chunks of 32 channels
                                 // for the row-strip kernel (the 1x1 kernel), which runs such a layer only where this is set
  const ConvPair* pair = nullptr;
  int pool = 0;  // 1: channels-last 3x3 layer with a 2x2/2 max-pool fused behind the activation (patch kernels);
                 // 2: rows are (channel, position of a 2x2 map) and each group of four rows is reduced to its
                 //    maximum behind the activation; cp_out is the stride of the pooled output
};
inline int round_up_vec(int c, int dt) { const int v = dt == CPRUNE_F32 ? 4 : 8; return (c + v - 1) / v * v; }

int validate_conv_desc(const cprune_conv_desc* d);
bool variant_supports(const cprune_conv_desc& d, int v, const ConvLayout& lay = ConvLayout());
size_t conv_ws_bytes(const cprune_conv_desc& d, int v, const ConvLayout& lay = ConvLayout());
// ws_limit: scratch bytes the chosen variant may need
int heuristic_variant(const cprune_conv_desc& d, const ConvLayout& lay = ConvLayout(), size_t ws_limit = SIZE_MAX);
size_t variant_ws_bytes(const cprune_conv_desc& d, int v, const ConvLayout& lay);   // of a variant that runs the layer
// Estimated clocks of a variant: of the general kernel on a layer it runs, of the split and the row-strip kernel (-1 where
// they do not run the layer); -1 for the others.
int best_split_variant(const cprune_conv_desc& d, const ConvLayout& lay, double* cost);   // the cheapest; -1: none runs it
int best_pw3_variant(const cprune_conv_desc& d, const ConvLayout& lay, double* cost);     // and of the 1x1 kernel on three parts
int best_rows_variant(const cprune_conv_desc& d, const ConvLayout& lay, double* cost);    // likewise of the row-strip kernel
double variant_cost(const cprune_conv_desc& d, int v, const ConvLayout& lay);
int cached_or_heuristic_variant(const cprune_conv_desc& d, bool* timed, const ConvLayout& lay = ConvLayout());
void remember_variant(const cprune_conv_desc& d, int v, const ConvLayout& lay = ConvLayout());

// Launchers (no argument validation: callers have validated).
int launch_conv_dense(const cprune_conv_desc& d, const void* x, const void* w, const float* bias,
                      const void* residual, void* y, int v, void* ws, hipStream_t s,
                      const ConvLayout& lay = ConvLayout());
int launch_conv_depthwise(const cprune_conv_desc& d, const void* x, const void* w,
                          const float* bias, const void* residual, void* y, hipStream_t s);
int launch_maxpool(const void* x, int n, int c, int h, int w, int k, int stride, int pad, int dt,
                   void* y, hipStream_t s);
int launch_gavgpool(const void* x, int n, int c, int hw, int dt, void* y, hipStream_t s);

// Channels-last layers of the network handle (cp = channel stride in elements).
int launch_depthwise_nhwc(const cprune_conv_desc& d, int cp, const void* x, const void* w_khwc,
                          const float* bias, const void* residual, void* y, hipStream_t s);
int launch_maxpool_nhwc(const void* x, int n, int cp, int h, int w, int k, int stride, int pad, int dt,
                        void* y, hipStream_t s);
int launch_gavgpool_nhwc(const void* x, int n, int cp, int hw, int dt, void* y, hipStream_t s);
int launch_nchw_to_nhwc(const void* x, int n, int c, int hw, int cp, int dt, void* y, hipStream_t s);
int launch_nhwc_to_nchw(const void* x, int n, int c, int hw, int cp, int dt, void* y, hipStream_t s);
// w [o][c][khw] -> [o][khw][cp] (zero pad); depthwise: o = 1 and c = channels gives [khw][cp]
int launch_repack_weights(const void* w, int o, int c, int khw, int cp, int dt, void* y, hipStream_t s);
// 3x3 / stride 1 / pad 1 on a 2x2 map as one matrix over the whole map: w [o][c][3][3] ->
// [rows][4 * cp_in], column (input pixel, channel), row (output pixel, channel) with channel
// stride cp_out, or (channel, output pixel) when rows_by_channel; bias [o] -> [4 * cp_out] alike
// w [o][9][cp] (channels-last 3x3 weights) -> the operand order of the independent-wavefront 3x3 kernel:
// [filter tile of 16][64-byte channel chunk][tap][lane][16 bytes], zero padded; wave_packed_bytes: its size
size_t wave_packed_bytes(int o, int cp, int dt);
int launch_repack_wave(const void* w_khwc, int o, int cp, int dt, void* y, hipStream_t s);
// w [rows][k], k contiguous -> the operand order of the reduction-split kernel, zero padded; rows_packed_bytes: size
size_t rows_packed_bytes(int rows, int k, int dt);
int launch_repack_rows(const void* w, int rows, int k, int dt, void* y, hipStream_t s);
// weights [o][taps][c] (khwc = 1) or [o][c][taps] -> the operand order of the split kernel: [filter tile of 16][round]
// [part][lane][16 bytes]; an fp32 weight as three bf16 parts, 16-bit weights as they are; zeros past the last filter
// and channel.  split_packed_bytes: size of the packed weights
// (whole: the last chunk of 32 channels packed like the others, zero padded; otherwise its groups only)
size_t split_packed_bytes(int o, int c, int taps, int dt, bool whole = false);
int launch_pack_split(const void* w, int o, int c, int taps, int khwc, int dt, void* y, hipStream_t s, bool whole = false);
int launch_repack_map2x2(const void* w, const float* bias, int o, int c, int cp_in, int cp_out,
                         int rows_by_channel, int dt, void* w_out, float* bias_out, hipStream_t s);

// Inverted-residual blocks, channels-last: depthwise k x k (+ bias + activation) and the 1x1 convolution behind it in one
// kernel, with (xh > 0) or without the 1x1 expansion in front of them.
struct MbArgs {
  const void* x;        // xh > 0: [n][h][w][cpi] block input; xh = 0: [n][h][w][cpe] expanded activations
  const void* we;       // expansion weights from launch_pack_expand, or null
  const float* be;      // [ce] or null
  const void* wdw;      // [k][k][cpe] depthwise weights (folded)
  const float* wdw32;   // 16-bit data, 3x3: the same as fp32, for the forms that read them so
  const float* bdw;     // [ce] or null
  const void* wp;       // [o][cpe] projection weights from launch_repack_rows
  const float* bp;      // [o] or null
  const void* res;      // [n][ho][wo][cop] shortcut or null
  void* y;              // [n][ho][wo][cop]
  int N, H, W, Ho, Wo, Cpi, Ce, Cpe, O, Cop;
  int Hi, Wi;           // image form (x is the NCHW image of cpi channels, H x W the first layer's map): its size, otherwise 0
  int act_e, act_dw, act_out;
  int tiles_y, tiles_x; // strips of a map
  int ipt;              // images side by side in the 16 columns of a strip: 1 or 2
  unsigned magic_x, magic_y;   // strip_magic of tiles_x and tiles_y
  unsigned x_bytes, we_bytes, wp_bytes, wdw_bytes, y_bytes;
  int nchunk;           // 64-byte chunks of expanded channels
  const void *we_raw, *wp_raw;   // fp32: the weights as they are, [ce][terms] and [o][cpe]
  int slots;            // wavefronts whose sums fit the exchange area (set by the launcher)
};

// Output rows a wavefront owns (k in {3, 5}, stride in {1, 2}, mb filter blocks): about as many as its registers hold beside the
// window's weights, multiples or halves of 7 where possible (the maps of the evaluated networks are 7 x 2^n); low = 1: about
// half as many, for maps whose tall strips leave units idle.  Some forms hold more than fit and spill: 7 of the 37 fp32 forms (all 5x5), 22 of the
// 75 bf16 and 9 of the 75 fp16 ones, by 1 to 84 registers, most where the window is 5x5 (its widened weights are 100
// registers) or a tall strip has 48 filters and more.  Timing chooses among tall and low all the same.
constexpr int mbrow_rows(int k, int s, int mb, int low) {
  if (s == 1 && k == 3) return mb <= 4 ? (low ? 4 : 7) : mb == 6 ? (low ? 3 : 5) : (low ? 2 : 3);
  if (s == 1) return mb <= 2 ? (low ? 2 : 4) : 2;
  if (k == 3) return mb <= 4 ? (low ? 2 : 4) : 2;
  return mb <= 4 ? 2 : 1;
}
// Whether fp32 strips multiply on three bf16 parts (mbrow3_kernel.hpp).  5x5 windows not (their 100 registers of weights leave too few: 24 -> 60 ->
// 40 at 56x56 stride 2, batch 48, 34.2 us on the fp32 instruction, 41.8 on parts, 80 -> 300 -> 80 at 14x14 46 / 118), nor tiles of 128
// filters (96 -> 280 -> 160 at 14x14 stride 2, depthwise and projection, 22.4 / 26.5).
constexpr bool mbrow_parts(int k, int mb) { return k == 3 && mb <= 6; }
// Likewise there: eight registers of weights a filter block and not four, so that tall strips of 64 filters do not fit (5 of the 37 forms spill).
constexpr int mbrow3_strip_rows(int s, int mb, int xh, int low) {
  if (s == 1) return mb <= 2 ? (low ? 4 : 7) : mb == 4 ? (low && xh > 4 ? 2 : 4) : mb == 6 && !xh ? 3 : 2;
  return mb <= 2 ? (low ? 2 : 4) : 2;
}
// elements from row to row of the staged image: 33 columns and what turns the rows' banks
constexpr int mbrow_image_pitch(int es) { return es == 4 ? 35 : 38; }
// columns at the left / right end of a strip whose window reaches into the neighbouring strip
constexpr int mbrow_halo_left(int k, int s) { return s == 1 ? k / 2 : 1; }
constexpr int mbrow_halo_right(int k, int s) { return s == 1 ? k / 2 : k == 5 ? 1 : 0; }
// The smallest built form for c_out filters and an input of cp_in channels (0: no expansion): mb 16-filter blocks and xh
// 32-byte units of a pixel's input.  false: none (c_out above 128 with an expansion, or too many input channels).
bool mbrow_form(int dt, int c_out, int cp_in, int* mb, int* xh);
// The image form: a 3x3 / stride 2 / pad 1 first layer on at most 3 channels, a 3x3 / stride 1 depthwise layer on a map
// wider than 8, up to 32 filters.
bool mbrow_image_form(int dt, int c_out, int* mb, int* xh);
// grid = (strips, filter tiles), ks in {1, 2, 4, 8} wavefronts that share a strip.
// CPRUNE_ERR_UNSUPPORTED for other combinations.
int launch_mbrow_f32(int k, int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a);
int launch_mbrow3_f32(int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a);
int launch_mbrow_f16(int k, int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a);
int launch_mbrow_bf16(int k, int stride, int mb, int xh, int low, dim3 grid, int ks, hipStream_t s, const MbArgs& a);
// expansion weights [ce][cp] -> the operand order of that kernel, [block of 16 channels][xh 32-byte units], zero padded
size_t expand_packed_bytes(int ce, int xh, int dt);
int launch_pack_expand(const void* w, int ce, int cp, int xh, int dt, void* y, hipStream_t s);
// numbers of a 16-bit type as fp32
int launch_widen(const void* x, long count, int dt, float* y, hipStream_t s);
// fp32 weights [rows][terms] -> three bf16 parts in the operand order of mbrow3_kernel, [tile of 16 rows][round of 16 terms][operand], zero
// padded to `rounds`; image: terms (channel, window row, window column) in rounds of four window rows of four columns.  Behind them
// the word of launch_parts_limit.
// The expansion's operands for xh 32-byte units of input are three a round, with each part twice where a round's weights are used for few.
constexpr bool mbrow3_twice(int stride, int xh, bool image) { return stride == 1 && xh <= 4 && !image; }
size_t parts_packed_bytes(int rows, int rounds, bool twice);
int launch_pack_parts(const void* w, int rows, int terms, int rounds, bool twice, bool image, void* y, hipStream_t s);
// The numbers from which on a strip of that kernel runs on the fp32 instruction, written to *limit: with an expansion the upper half of
// the smallest such input, without one the bits of the smallest such depthwise result.
struct PartsLimits {
  const float *we, *wd, *wp;       // [ce][terms] or null, [9][cpe], [o][cpe]
  const float *be, *bd;            // [ce] or null
  int ce, terms, cpe, o, act_e, act_d;
  unsigned* limit;
};
int launch_parts_limit(const PartsLimits& p, hipStream_t s);

// The depthwise 5x5 layer and the 1x1 convolution behind it through local memory, an 8 x 8 block of output pixels per work-group.
struct DwProjArgs {
  const void* x;        // [n][h][w][cpe], expanded activations
  const void* wdw;      // [k][k][cpe] depthwise weights (folded)
  const float* bdw;     // [ce] depthwise bias or null
  const void* wp;       // [o][cpe] projection weights (folded)
  const float* bp;      // [o] projection bias or null
  const void* res;      // [n][ho][wo][cop] or null
  void* y;              // [n][ho][wo][cop]
  int N, H, W, Ho, Wo, Ce, Cpe, O, Cop;
  int pad, act_dw, act_out;
  int tiles_y, tiles_x, tiles_m;
  unsigned x_bytes, wp_bytes, wdw_bytes;
  int vec_out;
};
// k = 5, stride in {1, 2}, mb in {2, 4, 8} (16-filter blocks per tile), ks in {1, 2} (groups of four wavefronts per work-group
// that split the channel chunks); grid = one work-group per (image, 8x8 output block, filter tile).
// CPRUNE_ERR_UNSUPPORTED for other combinations.
int launch_dwproj_f32(int k, int stride, int mb, int ks, dim3 grid, hipStream_t s, const DwProjArgs& a);
int launch_dwproj_f16(int k, int stride, int mb, int ks, dim3 grid, hipStream_t s, const DwProjArgs& a);
int launch_dwproj_bf16(int k, int stride, int mb, int ks, dim3 grid, hipStream_t s, const DwProjArgs& a);

// The first two layers of a network in one kernel: both 3x3 / stride 1 / pad 1, the first on the NCHW image
// (at most 3 channels) with c1 <= 32 filters, the second dense and channels-last.  d2 / lay2 describe the second
// layer (c_in = c1, cp_in = its channel stride in w2 <= 32, pool = 0 / 1); w1_packed from launch_repack_stem
// with 32 rows; y as for that layer.  CPRUNE_ERR_UNSUPPORTED outside these limits.
bool conv_stem2_supported(const cprune_conv_desc& d2, const ConvLayout& lay2, int c_in, int c1);
int launch_conv_stem2(const cprune_conv_desc& d2, const ConvLayout& lay2, const void* x_nchw, int c_in,
                      const void* w1_packed, const float* b1, int c1, int act1, const void* w2, const float* b2,
                      void* y, hipStream_t s);

// First-layer convolution: NCHW input with at most 3 channels, OIHW weights, channels-last output.
struct StemArgs {
  const void* x;        // [n][c][h][w]
  const void* w;        // [tiles_m * 16 * mb][kp] packed by launch_repack_stem: k = (c, u, v) padded with
                        // zeros to kp, rows beyond o zero
  const float* bias;    // [o] or null
  void* y;              // [n][ho][wo][cop]
  int N, C, H, W, Ho, Wo, O, Cop;
  int pad, act;
  int tiles_y, tiles_x, tiles_m;
  unsigned magic_x, magic_y;   // strip_magic of tiles_x, tiles_y
  int vec_out;
  int Hp = 0, Wp = 0;   // 7x7 / stride 2 kernels with the 3x3 / stride 2 / pad 1 max-pool inside: the pooled map; y is
                        // then [n][hp][wp][cop] and tiles_y, tiles_x count bands of its rows x 7 columns
  void* y_map = nullptr;   // fp32 7x7 / stride 2 kernel with the pool inside: the conv map as well (pool = 2)
  int band = 0;         // 7x7 / stride 2 kernels: pairs of conv rows a work-group walks over
  const void* w_raw = nullptr;          // ... fp32: the weights as they are, [o][c][7][7]
  unsigned x_bytes = 0, w_bytes = 0, w_raw_bytes = 0;
};
// (k, stride) in {(3, 1), (3, 2), (7, 2)}, mb in {2, 4} (16-filter blocks per tile); grid.x = workers
// that share the (image, 8x16 output block) list round-robin, grid.y = filter tiles.
// CPRUNE_ERR_UNSUPPORTED for other windows.  stem_packed_k: padded row length in elements.
int stem_packed_k(int k, int dt);
int launch_repack_stem(const void* w, int o, int ktot, int rows, int kp, int dt, void* y, hipStream_t s);
int launch_conv_stem_f32(int k, int stride, int mb, dim3 grid, hipStream_t s, const StemArgs& a);
int launch_conv_stem_f16(int k, int stride, int mb, dim3 grid, hipStream_t s, const StemArgs& a);
int launch_conv_stem_bf16(int k, int stride, int mb, dim3 grid, hipStream_t s, const StemArgs& a);
// 7x7 / stride 2 / pad 3 first layer, fp32 on three bf16 parts: reduction ordered (channel, window row, 8 columns: zero, then the window's),
// weights [16-filter block][6 rounds][part][lane][16 bytes] from launch_pack_stem7.  mb in {1, 2} blocks per wavefront, two wavefronts per
// work-group; grid.x = (image, band of rows, strip), grid.y = tiles of 32 mb filters; pool = 1 runs the 3x3 / stride 2 / pad 1 max-pool too
// (StemArgs::Hp, Wp), 2 (fp32) stores the conv map as well.
constexpr int kStem7Rounds = 6;
inline size_t stem7_packed_bytes(int o, int dt) { return (size_t)((o + 15) / 16) * kStem7Rounds * (dt == CPRUNE_F32 ? 3 : 1) * 1024; }
int launch_pack_stem7(const void* w, int o, int c, int dt, void* y, hipStream_t s);
int launch_conv_stem7_f16(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a);
int launch_conv_stem7_bf16(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a);
int launch_conv_stem7_f32(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a);
// The same layer in 16-bit data, 16 x 16 conv outputs a work-group, reduction ordered (window row, 8 window columns, 4 channels):
// weights [rows][224] from launch_repack_stem7 (k = u * 32 + (v + 1) * 4 + c; zero for column slot 0, channel slot 3, channels beyond c and
// rows beyond o).  mb in {2, 4}; pool = 1 runs the max-pool too; tiles_y, tiles_x count blocks of the map, or 7 x 7 blocks of the pooled one;
// grid.x = workers sharing the (image, block) list, grid.y = filter tiles.
constexpr int kStem7K = 224;
int launch_repack_stem7(const void* w, int o, int c, int rows, int dt, void* y, hipStream_t s);
int launch_conv_stem7_block_f16(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a);
int launch_conv_stem7_block_bf16(int mb, int pool, dim3 grid, hipStream_t s, const StemArgs& a);

}  // namespace cprune
