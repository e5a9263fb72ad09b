// Host side of the dense convolution: the variant table (tile x scheduling
// mode), what each variant supports and needs, and the launch.
#include "conv_ksplit_kernel.hpp"
#include "conv_pw_kernel.hpp"
#include "conv_wave_kernel.hpp"
#include "conv_stem2_kernel.hpp"
#include "conv_patch32_kernel.hpp"
#include "conv_split_kernel.hpp"
#include "conv_rows_kernel.hpp"
#include "conv_pw3_kernel.hpp"
#include "conv_rows_s2_kernel.hpp"
#include "conv_rows_nchw_kernel.hpp"

#include <algorithm>
#include <cmath>

namespace cprune {
namespace {

const TileVariant kTiles[] = {
#define CPRUNE_TILE_ROW(ID, WM_, WN_, MB_, NB_, KQ_) {WM_, WN_, MB_, NB_, KQ_, 1},
    CPRUNE_TILE_LIST(CPRUNE_TILE_ROW)
#undef CPRUNE_TILE_ROW
};
static_assert(sizeof(kTiles) / sizeof(kTiles[0]) == kNumTiles, "tile table");
// Scheduling modes: 0 = one output tile per work-group; n > 0 = the (tile, slab)
// work line is cut into equal runs for n * 256 resident work-groups.
const int kScheds[] = {0, 1, 2, 3, 4, 6, 8};
constexpr int kNumScheds = sizeof(kScheds) / sizeof(kScheds[0]);
constexpr int kMinUnitsPerGroup = 4;
constexpr long kMaxKsplitGroups = 8192;
constexpr int kMaxWaveMap = 32;
constexpr long kSplitMinTerms = 16;

unsigned magic_for(unsigned d) {
  if (d <= 1) return 0;
  return (unsigned)((0x100000000ull + d - 1) / d);
}

int slab_k(int dt, int kq) { return (dt == CPRUNE_F32 ? 16 : 32) * kq; }

struct Plan {
  int tiles_m, tiles_p, slabs, units, units_per_wg, groups;
  bool fixup;
};

Plan make_plan(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay) {
  Plan p;
  const int ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  const long P = (long)d.n * ho * wo;
  const int K = (lay.nhwc ? lay.cp_in : d.c_in) * d.kh * d.kw;
  const int kt = slab_k(d.dtype, tv.kq);
  p.tiles_m = (d.c_out + tv.tile_m() - 1) / tv.tile_m();
  p.tiles_p = (int)((P + tv.tile_p() - 1) / tv.tile_p());
  p.slabs = (K + kt - 1) / kt;
  const long units = (long)p.tiles_m * p.tiles_p * p.slabs;
  p.units = (int)units;
  if (tv.sched == 0) {
    p.units_per_wg = p.slabs;
    p.groups = p.tiles_m * p.tiles_p;
    p.fixup = false;
  } else {
    long g = (long)tv.sched * 256;
    const long cap = (units + kMinUnitsPerGroup - 1) / kMinUnitsPerGroup;
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    p.units_per_wg = (int)((units + g - 1) / g);
    p.groups = (int)((units + p.units_per_wg - 1) / p.units_per_wg);
    p.fixup = (p.units_per_wg % p.slabs) != 0;
  }
  return p;
}

// Rough cost in clocks of the general kernel's tiles, whole or cut into equal runs.  A unit holds `occ` work-groups (local
// memory); a slab costs a group its matrix instructions times the groups it shares them with, and no less than the round
// trip of its operands; groups come in rounds; cut tiles pay a second launch and their pieces.  (Cutting always, with the
// largest reuse per operand, gave a layer with a short reduction a dozen groups in all: 13 -> 36 filters, 1x1 at 49x49,
// batch 4, bf16 57 us, now 16 us; timed choice 15.7.)  Scaled to the clocks of split_cost, which it is compared with: over
// 209 layers with windows of 3 to 7 that the scale was not taken from, the cheaper estimate loses 1.0 % (fp32 channels-last),
// 0.9 % (fp32 in the boundary's layout) and 3.0 % (bf16 there) to the better of the two on average, always the split kernel 2.6,
// 4.6 and 3.1 % and up to two times (a fully connected layer on a 7x7 map, 256 -> 1000, batch 32, 65.8 us; the general kernel 33.5).
double tile_cost(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay) {
  const Plan p = make_plan(d, tv, lay);
  const bool f32 = d.dtype == CPRUNE_F32;
  const long mt = tv.tile_m(), pt = tv.tile_p();
  const double run = p.units_per_wg, slabs = p.slabs, groups = p.groups;
  const double rows = std::min((double)tv.mb, std::ceil((double)d.c_out / 16.0 / tv.wm));   // filter blocks that exist
  const double mfma = rows * tv.nb * tv.kq * (f32 ? 128.0 : 16.0);
  const double bytes = (double)(mt + pt) * 64 * tv.kq;
  const double occ = std::max(1.0, std::min(4.0, std::floor(160.0 * 1024 / (2.0 * (mt + pt) * (64 * tv.kq + 16)))));
  const double held = std::min(occ, std::ceil(groups / 256.0));
  const double slab = std::max(900.0 + bytes / 16.0, held * std::max(mfma, bytes / 16.0));
  const double store = 2000.0 + (double)(mt * pt) / 8.0;
  return (f32 ? 1.7 : 2.0) * (std::ceil(groups / (256.0 * occ)) * (run * slab + std::ceil(run / slabs) * store) +
                              (p.fixup ? 9000.0 + 120.0 * slabs / run : 0.0));
}

// The pixel block a work-group of a split variant owns on a map: as few blocks as possible, and among equal ones the
// smaller patch.  Whole images (several, if they fit) or th x tw pixels of one; a fused pool needs even sizes.
struct SplitPlan {
  int th, tw, ni, ph, pw, tiles_n, tiles_y, tiles_x;
  size_t lds;
  int off_patch;
};

bool split_plan(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay, SplitPlan* out) {
  const int ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  const int pt = tv.tile_p(), parts = d.dtype == CPRUNE_F32 ? 3 : 1, even = lay.pool ? 2 : 1;
  const int taps = d.kh * d.kw;
  int rounds_last;
  split_rounds(lay.nhwc ? lay.cp_in : d.c_in, taps, nullptr, nullptr, &rounds_last);
  const int off_patch = kSplitTab + (taps + rounds_last) * 16;
  const size_t red = (size_t)(tv.ks - 1) * tv.wm * tv.wn * tv.mb * tv.nb * 1024;
  double best = -1.0;
  auto consider = [&](int ni, int th, int tw) {
    SplitPlan p;
    p.th = th; p.tw = tw; p.ni = ni;
    p.ph = (th - 1) * d.stride + d.kh; p.pw = (tw - 1) * d.stride + d.kw;
    const long npatch = (long)ni * p.ph * p.pw;
    if ((long)ni * th * tw > pt || npatch > 64L * tv.nib) return;
    p.tiles_n = (d.n + ni - 1) / ni; p.tiles_y = (ho + th - 1) / th; p.tiles_x = (wo + tw - 1) / tw;
    p.off_patch = off_patch;
    p.lds = (size_t)off_patch + (size_t)npatch * (64 * parts + 16);
    if (p.lds < red) p.lds = red;
    if (p.lds > 160 * 1024) return;
    const double cost = (double)p.tiles_n * p.tiles_y * p.tiles_x * (pt + 0.25 * (double)npatch);
    if (best < 0.0 || cost < best) { best = cost; *out = p; }
  };
  if ((long)ho * wo <= pt)
    for (int ni = (int)(pt / ((long)ho * wo)); ni >= 1; --ni)
      if (ni <= d.n) consider(ni, ho, wo);
  // every width that some number of blocks per row gives, the widest first
  for (int tw = (wo + even - 1) / even * even, nx; tw > 0; nx = tw > even ? (wo + tw - even - 1) / (tw - even) : 0,
           tw = nx ? ((wo + nx - 1) / nx + even - 1) / even * even : 0) {
    if (tw > pt / even) continue;
    int th = pt / tw < ho ? pt / tw : ho;                              // rows that fit the block ...
    const int pw = (tw - 1) * d.stride + d.kw;
    const int ph_max = 64 * tv.nib / pw;                               // ... and whose patch fits the staging items
    if (ph_max < d.kh) continue;
    if ((ph_max - d.kh) / d.stride + 1 < th) th = (ph_max - d.kh) / d.stride + 1;
    th = th / even * even;
    if (th < 1) continue;
    const int ny = (ho + th - 1) / th;
    consider(1, ((ho + ny - 1) / ny + even - 1) / even * even, tw);
  }
  return best >= 0.0;
}

// Whether the split kernel runs a layer, as far as that does not depend on the variant.
bool split_layer(const cprune_conv_desc& d, const ConvLayout& lay) {
  if (lay.nhwc ? !(d.dtype == CPRUNE_F32 && lay.w_split) : lay.nhwc_out != 0) return false;
  if (lay.pool == 2 || (lay.pool && ((d.h | d.w) & 1 || d.stride != 1)) || d.stride > 2) return false;
  // fp32 sums of a few terms are less exact in parts than on the fp32 instruction (conv_split_kernel.hpp)
  if (d.dtype == CPRUNE_F32 && (long)d.c_in * d.kh * d.kw < kSplitMinTerms) return false;
  const int ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  if (!lay.nhwc && (long)ho * wo < 16) return false;   // a map of a few pixels is a matrix product: the general kernel
  return split_packed_bytes(d.c_out, lay.nhwc ? lay.cp_in : d.c_in, d.kh * d.kw, d.dtype) < ((size_t)1 << 31);
}

// multiply-high divisions in the tile decode: exact while groups x divisor < 2^32
bool split_groups_fit(const cprune_conv_desc& d, const TileVariant& tv, const SplitPlan& p) {
  const long tiles_s = (long)p.tiles_n * p.tiles_y * p.tiles_x;
  const long groups = tiles_s * ((d.c_out + tv.tile_m() - 1) / tv.tile_m());
  return groups * tiles_s < (1L << 32) && groups < (1L << 31);
}

// Whether a split variant runs a layer, and the plan it runs by.
bool split_supports(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay, SplitPlan* plan) {
  return split_layer(d, lay) && split_plan(d, tv, lay, plan) && split_groups_fit(d, tv, *plan);
}

// Rough cost in clocks of a split variant on a layer, for choosing among them untimed: the matrix-pipe time of the
// work-groups a compute unit gets, plus per group the staging of its chunks and the fixed start and end, which overlap
// between the two or three groups a unit holds (the kernel's launch bound).  Constants from timings of all variants on twenty
// layers.
double split_cost(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay, const SplitPlan& p) {
  int nfull, groups_last, rounds_last;
  const int rtot = split_rounds(lay.nhwc ? lay.cp_in : d.c_in, d.kh * d.kw, &nfull, &groups_last, &rounds_last);
  const double groups = (double)p.tiles_n * p.tiles_y * p.tiles_x * ((d.c_out + tv.tile_m() - 1) / tv.tile_m());
  const int occ = tv.mb * tv.nb <= 4 && tv.nib <= 4 ? 3 : 2;
  const double mfma = std::ceil((double)rtot / tv.ks) * tv.mb * tv.nb * (d.dtype == CPRUNE_F32 ? 6 : 1) * 18.0;
  const double chunks = nfull + (rounds_last ? 1 : 0);
  const double npatch = (double)p.ni * p.ph * p.pw;
  const double wait = (double)rtot / tv.ks * 250.0;   // operand latency of a round that nothing else hides
  const double fixed = 5000.0 + chunks * (1500.0 + 8.0 * npatch) + wait;
  return std::ceil(groups / 256.0) * mfma + std::ceil(groups / (256.0 * occ)) * fixed;
}

int launch_split_conv(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay, const void* x,
                      const void* w, const float* bias, const void* residual, void* y, void* ws, hipStream_t s) {
  SplitPlan p;
  if (!split_supports(d, tv, lay, &p)) return CPRUNE_ERR_UNSUPPORTED;
  SplitArgs a;
  const size_t es = dtype_size(d.dtype);
  a.C = lay.nhwc ? lay.cp_in : d.c_in;
  a.taps = d.kh * d.kw; a.kw = d.kw;
  a.rtot = split_rounds(a.C, a.taps, &a.nfull, &a.groups_last, &a.rounds_last);
  a.w_bytes = (unsigned)split_packed_bytes(d.c_out, a.C, a.taps, d.dtype);
  if (lay.nhwc) {
    a.w = lay.w_split;
  } else {
    const int rc = launch_pack_split(w, d.c_out, d.c_in, a.taps, 0, d.dtype, ws, s);
    if (rc != CPRUNE_OK) return rc;
    a.w = ws;
  }
  a.w_raw = w; a.w_raw_bytes = (unsigned)((size_t)d.c_out * a.C * a.taps * es);
  a.x = x; a.bias = bias; a.res = residual; a.y = y;
  a.N = d.n; a.H = d.h; a.W = d.w; a.O = d.c_out;
  a.Ho = conv_out_dim(d.h, d.kh, d.stride, d.pad); a.Wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  a.Cop = lay.cp_out; a.vec_out = (lay.cp_out % 4) == 0 ? 1 : 0;
  a.stride = d.stride; a.pad = d.pad;
  a.th = p.th; a.tw = p.tw; a.ni = p.ni; a.ph = p.ph; a.pw = p.pw;
  a.tiles_n = p.tiles_n; a.tiles_y = p.tiles_y; a.tiles_x = p.tiles_x;
  a.tiles_m = (d.c_out + tv.tile_m() - 1) / tv.tile_m();
  const int blocks = (d.c_out + 15) / 16;
  a.blk_base = blocks / a.tiles_m; a.blk_rem = blocks % a.tiles_m;
  a.x_bytes = (unsigned)((size_t)d.n * a.C * d.h * d.w * es);
  a.pool = lay.pool; a.act = d.act;
  a.m_major = a.w_bytes > a.x_bytes ? 1 : 0;
  const int tiles_s = p.tiles_n * p.tiles_y * p.tiles_x, div = lay.pool ? 2 : 1;
  a.magic_s = magic_for((unsigned)tiles_s); a.magic_m = magic_for((unsigned)a.tiles_m);
  a.magic_x = magic_for((unsigned)p.tiles_x); a.magic_y = magic_for((unsigned)p.tiles_y);
  a.magic_pp = magic_for((unsigned)(p.ph * p.pw)); a.magic_pw = magic_for((unsigned)p.pw);
  a.magic_thw = magic_for((unsigned)(p.th * p.tw / (div * div))); a.magic_tw = magic_for((unsigned)(p.tw / div));
  a.magic_np = magic_for((unsigned)(p.ni * p.ph * p.pw));
  a.off_patch = p.off_patch;
  const dim3 grid((unsigned)((long)tiles_s * a.tiles_m));
  int rc;
  if (d.dtype == CPRUNE_F32) rc = launch_conv_split_f32(tv.patch_id, !lay.nhwc, grid, p.lds, s, a);
  else if (d.dtype == CPRUNE_F16) rc = launch_conv_split_f16(tv.patch_id, grid, p.lds, s, a);
  else rc = launch_conv_split_bf16(tv.patch_id, grid, p.lds, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

}  // namespace

constexpr int kFirstSplit = kNumTiles * kNumScheds + kNumPatch + kNumPatch32 + kNumKsplit + kNumPw + kNumWave + kNumPatchS2;
constexpr int kFirstRows = kFirstSplit + kNumSplit;
constexpr int kFirstPw3 = kFirstRows + kNumRows;
constexpr int kFirstRowsS2 = kFirstPw3 + kNumPw3;
constexpr int kFirstRowsNchw = kFirstRowsS2 + kNumRowsS2;
constexpr int kFirstRows7 = kFirstRowsNchw + kNumRowsNchw;
constexpr int kNumVariants = kFirstRows7 + kNumRows7;
int num_variants() { return kNumVariants; }

namespace {
struct VariantTable {
  TileVariant table[kNumVariants];
  VariantTable() {
#define CPRUNE_PATCH_ROW(ID, MB_, TH_, TW_, NI_, KQ_, KS_)                                 \
    {                                                                         \
      TileVariant& pv = table[kNumTiles * kNumScheds + ID];                   \
      pv.wm = 1; pv.wn = 4; pv.mb = MB_; pv.nb = (TH_ * TW_ * NI_) / 64; pv.kq = KQ_; pv.ni = NI_; \
      pv.sched = -1; pv.th = TH_; pv.tw = TW_; pv.patch_id = ID; pv.ks = KS_; \
    }
    CPRUNE_PATCH_LIST(CPRUNE_PATCH_ROW)
#undef CPRUNE_PATCH_ROW
#define CPRUNE_PATCH32_ROW(ID, MB2_, NB2_, WPX_, TH_, TW_, NI_, KQ_)                       \
    {                                                                                      \
      TileVariant& pv = table[kNumTiles * kNumScheds + kNumPatch + ID];                    \
      pv.wm = 1; pv.wn = WPX_; pv.mb = 2 * MB2_; pv.nb = 2 * NB2_; pv.kq = KQ_; pv.ni = NI_; \
      pv.sched = -1; pv.th = TH_; pv.tw = TW_; pv.patch_id = ID; pv.blk32 = 1;             \
    }
    CPRUNE_PATCH32_LIST(CPRUNE_PATCH32_ROW)
#undef CPRUNE_PATCH32_ROW
#define CPRUNE_KSPLIT_ROW(ID, NB_, KW_)                                                    \
    {                                                                                      \
      TileVariant& kv = table[kNumTiles * kNumScheds + kNumPatch + kNumPatch32 + ID];      \
      kv.wm = 1; kv.wn = 1; kv.mb = 1; kv.nb = NB_; kv.kq = 1; kv.sched = -2;              \
      kv.patch_id = ID; kv.kwaves = KW_;                                                   \
    }
    CPRUNE_KSPLIT_LIST(CPRUNE_KSPLIT_ROW)
#undef CPRUNE_KSPLIT_ROW
#define CPRUNE_PW_ROW(ID, MB_, NR_)                                                        \
    {                                                                                      \
      TileVariant& kv = table[kNumTiles * kNumScheds + kNumPatch + kNumPatch32 + kNumKsplit + ID]; \
      kv.wm = 1; kv.wn = 4; kv.mb = MB_; kv.nb = 1; kv.kq = NR_; kv.sched = -3;            \
      kv.patch_id = ID; kv.nr = NR_;                                                       \
    }
    CPRUNE_PW_LIST(CPRUNE_PW_ROW)
#undef CPRUNE_PW_ROW
#define CPRUNE_WAVE_ROW(ID, NP_, NB_, KS_)                                                 \
    {                                                                                      \
      TileVariant& kv = table[kNumTiles * kNumScheds + kNumPatch + kNumPatch32 + kNumKsplit + kNumPw + ID]; \
      kv.wm = 1; kv.wn = NP_; kv.mb = 1; kv.nb = NB_; kv.kq = 1; kv.sched = -4;            \
      kv.th = 4; kv.tw = 4; kv.patch_id = ID; kv.ks = KS_;                                 \
    }
    CPRUNE_WAVE_LIST(CPRUNE_WAVE_ROW)
#undef CPRUNE_WAVE_ROW
    // (new families go behind the existing ones, so that stored variant numbers keep their meaning)
#define CPRUNE_PATCH_S2_ROW(ID, MB_, TH_, TW_, KQ_)                                        \
    {                                                                                      \
      TileVariant& pv = table[kNumTiles * kNumScheds + kNumPatch + kNumPatch32 + kNumKsplit + kNumPw + kNumWave + ID]; \
      pv.wm = 1; pv.wn = 4; pv.mb = MB_; pv.nb = (TH_ * TW_) / 64; pv.kq = KQ_; pv.ni = 1;  \
      pv.sched = -1; pv.th = TH_; pv.tw = TW_; pv.patch_id = ID; pv.stride = 2;            \
    }
    CPRUNE_PATCH_S2_LIST(CPRUNE_PATCH_S2_ROW)
#undef CPRUNE_PATCH_S2_ROW
#define CPRUNE_SPLIT_ROW(ID, WM_, WN_, WK_, MB_, NB_, NIB_)                                \
    {                                                                                      \
      TileVariant& kv = table[kFirstSplit + ID];                                            \
      kv.wm = WM_; kv.wn = WN_; kv.mb = MB_; kv.nb = NB_; kv.kq = 1; kv.sched = -1; kv.split = 1;         \
      kv.patch_id = ID; kv.ks = WK_; kv.nib = NIB_;                                        \
    }
    CPRUNE_SPLIT_LIST(CPRUNE_SPLIT_ROW)
#undef CPRUNE_SPLIT_ROW
#define CPRUNE_ROWS_ROW(ID, MB_, R_, KS_)                                                  \
    {                                                                                      \
      TileVariant& kv = table[kFirstRows + ID];                                            \
      kv.wm = 1; kv.wn = KS_ >= 4 ? 1 : 4 / KS_; kv.mb = MB_; kv.nb = R_; kv.kq = 1; kv.sched = -1; kv.rows = 1; \
      kv.th = R_; kv.tw = 16; kv.patch_id = ID; kv.ks = KS_;                               \
    }
    CPRUNE_ROWS_LIST(CPRUNE_ROWS_ROW)
#undef CPRUNE_ROWS_ROW
#define CPRUNE_PW3_ROW(ID, MB_, NB_, DEEP_)                                                \
    {                                                                                      \
      TileVariant& kv = table[kFirstPw3 + ID];                                             \
      kv.wm = 4; kv.wn = 1; kv.mb = MB_; kv.nb = NB_; kv.kq = 2; kv.sched = -1; kv.pw3 = 1 + DEEP_; kv.patch_id = ID; \
    }
    CPRUNE_PW3_LIST(CPRUNE_PW3_ROW)
#undef CPRUNE_PW3_ROW
#define CPRUNE_ROWS_S2_ROW(ID, MB_, R_, KS_)                                               \
    {                                                                                      \
      TileVariant& kv = table[kFirstRowsS2 + ID];                                          \
      kv.wm = 1; kv.wn = KS_ >= 4 ? 1 : 4 / KS_; kv.mb = MB_; kv.nb = R_; kv.kq = 1; kv.sched = -1; kv.rows = 1; \
      kv.th = R_; kv.tw = 16; kv.patch_id = ID; kv.ks = KS_; kv.stride = 2;                \
    }
    CPRUNE_ROWS_S2_LIST(CPRUNE_ROWS_S2_ROW)
#undef CPRUNE_ROWS_S2_ROW
#define CPRUNE_ROWS_NCHW_ROW(ID, MB_, R_, KS_)                                             \
    {                                                                                      \
      TileVariant& kv = table[kFirstRowsNchw + ID];                                        \
      kv.wm = 1; kv.wn = 4 / KS_; kv.mb = MB_; kv.nb = R_; kv.kq = 1; kv.sched = -1; kv.rows = 2; \
      kv.th = R_; kv.tw = 16; kv.patch_id = ID; kv.ks = KS_;                               \
    }
    CPRUNE_ROWS_NCHW_LIST(CPRUNE_ROWS_NCHW_ROW)
#undef CPRUNE_ROWS_NCHW_ROW
#define CPRUNE_ROWS7_ROW(ID, MB_, R_, KS_)                                                 \
    {                                                                                      \
      TileVariant& kv = table[kFirstRows7 + ID];                                           \
      kv.wm = 1; kv.wn = KS_ >= 4 ? 1 : 4 / KS_; kv.mb = MB_; kv.nb = R_; kv.kq = 1; kv.sched = -1; kv.rows = 1; \
      kv.th = R_; kv.tw = 16; kv.patch_id = kNumRows + ID; kv.ks = KS_;                    \
    }
    CPRUNE_ROWS7_LIST(CPRUNE_ROWS7_ROW)
#undef CPRUNE_ROWS7_ROW
    for (int t = 0; t < kNumTiles; ++t)
      for (int s = 0; s < kNumScheds; ++s) {
        table[t * kNumScheds + s] = kTiles[t];
        table[t * kNumScheds + s].sched = kScheds[s];
      }
  }
};
}  // namespace

const TileVariant& variant(int id) {
  static const VariantTable vt;   // built once, on first use, whichever thread gets there first
  return vt.table[id];
}

// (the plan is a search over block shapes, the same for variants with equal pixel blocks and staging items: five for 13 variants)
int best_split_variant(const cprune_conv_desc& d, const ConvLayout& lay, double* cost) {
  if (!split_layer(d, lay)) return -1;
  SplitPlan plan[kNumSplit];
  bool have[kNumSplit];
  int best_v = -1;
  for (int id = 0; id < kNumSplit; ++id) {
    const int v = kFirstSplit + id;
    const TileVariant& tv = variant(v);
    int same = 0;
    while (same < id && !(variant(v - id + same).tile_p() == tv.tile_p() && variant(v - id + same).nib == tv.nib)) ++same;
    if (same < id) { plan[id] = plan[same]; have[id] = have[same]; }
    else have[id] = split_plan(d, tv, lay, &plan[id]);
    if (!have[id] || !split_groups_fit(d, tv, plan[id])) continue;
    const double c = split_cost(d, tv, lay, plan[id]);
    if (best_v < 0 || c < *cost) { *cost = c; best_v = v; }
  }
  return best_v;
}

// Strips of the row-strip kernel on a layer: 16 columns x th rows of one image's output, or of two (four) images of at most 8 (4)
// columns.
static RowsArgs rows_tiles(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay) {
  RowsArgs a;
  a.H = conv_out_dim(d.h, 3, tv.stride, 1); a.W = conv_out_dim(d.w, 3, tv.stride, 1);
  a.lane_shift = a.W <= 4 ? 2 : a.W <= 8 ? 3 : 4;
  const int ipt = 16 >> a.lane_shift;
  a.tiles_x = (a.W + 15) / 16;
  a.step = 16;
  if (a.tiles_x > 1 && (tv.stride == 2 || tv.rows == 2 || d.dtype == CPRUNE_F32)) {
    a.step = tv.stride == 2 ? 15 : lay.pool ? 12 : 14;
    a.tiles_x = (a.W - 16 + a.step - 1) / a.step + 1;
  }
  a.tiles_y = (a.H + tv.th - 1) / tv.th;
  a.tiles_m = (d.c_out + tv.tile_m() - 1) / tv.tile_m();
  a.strips = (d.n + ipt - 1) / ipt * a.tiles_y * a.tiles_x;
  return a;
}

// Whether the work-groups of a layer in a handle run filter tile by filter tile.  Each XCD owns a contiguous stretch of them; the other
// way round (strips slowest) all eight read all weights, which, cut in parts, are the larger operand of the small maps.  Below 3 MB an
// XCD's L2 holds them with its pixels and the order does not matter (fp32, 209 -> 197 at 8x8, 2.2 MB: 20.4 us either way) or costs 1-2 %
// (bf16 284 -> 360 at 4x4, 1.8 MB); above: fp32 411 -> 512 at 7x7 b32 37.4 -> 32.7 us, 512 -> 411 38.0 -> 34.4, 360 -> 360 at 4x4 b64 19.9 ->
// 17.4, 284 -> 360 17.3 -> 15.3; bf16 512 -> 411 10.75 -> 10.45.  Not with the 1x1 layer's (shorter) work-groups behind: they would all be one XCD's.
static bool rows_m_major(const RowsArgs& a, long groups_s, bool pair) {
  return !pair && a.w_bytes > (3u << 20) && a.w_bytes > a.x_bytes && groups_s * a.tiles_m * groups_s < (1L << 32);
}

// Clocks of a row-strip variant, to choose among them untimed: a wavefront's chunks, 16 clocks per MFMA (six for one in fp32) and
// what a wavefront alone on its SIMD waits per chunk, or the whole layer's on 1024 SIMDs where that is longer; the meeting of the
// sums.  On 72 random layers (maps 4 to 56, batch 1-64) its choice takes 3 % longer than the best of the variants on average, 17 % at
// most, in bf16, 0.4 % on average in fp32.
static double rows_cost(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay) {
  const RowsArgs p = rows_tiles(d, tv, lay);
  const bool f32 = d.dtype == CPRUNE_F32;
  if (tv.rows == 2) {
    // in the boundary's layout: a chunk of a wavefront alone on its SIMD, and of one among many (from timings of all variants on 60
    // random layers a type)
    const double chunks = (d.c_in + 31) / 32, turns = std::ceil(chunks / tv.ks), r = tv.th, mb = tv.mb;
    const double alone = f32 ? 1800.0 * r + 2200.0 : r * (150.0 + 850.0 * mb) + 600.0;
    const double busy = f32 ? 1250.0 * r + 3300.0 : (r * (850.0 * mb - 250.0) + 1250.0) * (tv.ks == 4 ? 1.5 : 1.0);
    const double load = (double)p.strips * p.tiles_m * tv.ks / 1024.0;      // wavefronts of a SIMD
    return std::max(turns * alone, (load < 4.0 ? std::ceil(load) : load + 0.5) * turns * busy) + (tv.ks > 1 ? 1200.0 : 0.0);
  }
  const double waves = (double)p.strips * p.tiles_m * tv.ks;
  const double chunks = ((lay.cp_in + 31) / 32 + tv.ks - 1) / tv.ks;
  const double mma = (f32 ? 864.0 : 144.0) * tv.mb * std::min(tv.th, p.H);
  if (tv.stride == 2) {
    // every row is two operands (fp32: of two loads, and cut), weights are shared by the work-group's strips; a kilobyte each from the
    // vector cache, which four SIMDs share at 64 bytes a clock
    const double rows = 2 * std::min(tv.th, p.H) + 1, parts = f32 ? 3.0 : 1.0;
    const double load = (rows * (f32 ? 4.0 : 2.0) + 9.0 * parts * tv.mb / tv.wn) * 64.0, cut = f32 ? 352.0 * rows : 0.0;
    return std::max(chunks * (mma + cut + (f32 ? 1500.0 : 500.0)), waves / 1024.0 * chunks * (std::max(mma, load) + 0.4 * cut + 300.0)) +
           (tv.ks > 1 && !f32 ? 160.0 * tv.mb * tv.th : 0.0) + 500.0 * std::ceil(waves / 1024.0);
  }
  return std::max(chunks * (mma + (f32 ? 4000.0 : 500.0)), waves / 1024.0 * chunks * (mma + 300.0)) +
         (tv.ks > 1 && !f32 ? 160.0 * tv.mb * tv.th : 0.0) + 500.0 * std::ceil(waves / 1024.0);
}

int best_rows_variant(const cprune_conv_desc& d, const ConvLayout& lay, double* cost) {
  int best_v = -1;
  const int first = !lay.nhwc ? kFirstRowsNchw : d.stride == 1 ? kFirstRows : kFirstRowsS2;
  const int count = !lay.nhwc ? kNumRowsNchw : d.stride == 1 ? kNumRows : kNumRowsS2;
  for (int v = first; v < first + count; ++v) {
    if (!variant_supports(d, v, lay)) continue;
    const double c = rows_cost(d, variant(v), lay);
    if (best_v < 0 || c < *cost) { *cost = c; best_v = v; }
  }
  return best_v;
}

// Work-groups of the 1x1 kernel on three parts along pixels and filters.
static long pw3_groups(const cprune_conv_desc& d, const TileVariant& tv, long* tiles_m) {
  const long P = (long)d.n * conv_out_dim(d.h, 1, d.stride, 0) * conv_out_dim(d.w, 1, d.stride, 0);
  *tiles_m = (d.c_out + tv.tile_m() - 1) / tv.tile_m();
  return (P + tv.tile_p() - 1) / tv.tile_p() * *tiles_m;
}

// Clocks of one of its variants, to choose among them: as split_cost, constants from timings of all variants on 160 random layers.
static double pw3_cost(const cprune_conv_desc& d, const TileVariant& tv, const ConvLayout& lay) {
  long tiles_m;
  const double groups = (double)pw3_groups(d, tv, &tiles_m), rounds = (lay.cp_in + 31) / 32;
  const double blocks = std::ceil((d.c_out + 15) / 16 / (double)tiles_m / 4.0);      // of a tile's longest share
  const bool deep = tv.pw3 == 2, f32 = d.dtype == CPRUNE_F32;
  const int occ = !f32 ? (tv.nb > 2 ? (tv.mb == 1 ? 4 : 3) : tv.mb == 1 ? 6 : 4) : tv.nb > 2 ? (tv.mb == 1 ? 3 : 2) : tv.mb == 1 ? (deep ? 4 : 6) : deep ? 2 : 4;
  const double held = std::max(1.0, std::min((double)occ, groups / 256.0));      // work-groups of a unit hide each other's waits
  return std::ceil(groups / 256.0) * rounds * blocks * tv.nb * (f32 ? 108.0 : 40.0) +
         std::ceil(groups / (256.0 * occ)) * ((deep ? 5500.0 : 5000.0) + rounds * (!f32 ? 300.0 : deep ? 650.0 : 850.0) / held);
}

int best_pw3_variant(const cprune_conv_desc& d, const ConvLayout& lay, double* cost) {
  int best_v = -1;
  for (int v = kFirstPw3; v < kFirstPw3 + kNumPw3; ++v) {
    if (!variant_supports(d, v, lay)) continue;
    const double c = pw3_cost(d, variant(v), lay);
    if (best_v < 0 || c < *cost) { *cost = c; best_v = v; }
  }
  return best_v;
}

double variant_cost(const cprune_conv_desc& d, int v, const ConvLayout& lay) {
  const TileVariant& tv = variant(v);
  if (tv.pw3) return variant_supports(d, v, lay) ? pw3_cost(d, tv, lay) : -1.0;
  SplitPlan p;
  if (tv.split) return split_supports(d, tv, lay, &p) ? split_cost(d, tv, lay, p) : -1.0;
  if (tv.rows) return variant_supports(d, v, lay) ? rows_cost(d, tv, lay) : -1.0;
  return tv.sched >= 0 ? tile_cost(d, tv, lay) : -1.0;
}

bool variant_supports(const cprune_conv_desc& d, int v, const ConvLayout& lay) {
  if (v < 0 || v >= num_variants()) return false;
  if (d.groups != 1) return false;
  const TileVariant& tv = variant(v);
  if (tv.split) {
    SplitPlan p;
    return split_supports(d, tv, lay, &p);
  }
  if (tv.rows) {
    // 3x3 / pad 1 at the variant's stride in a handle, or (rows = 2) at stride 1 in the boundary's layout; wavefronts share a strip only while there is a chunk for each, and not where strips
    // alone fill the chip several times
    if (tv.rows == 2) {
      if (lay.nhwc || lay.nhwc_out || lay.pool || !(d.kh == 3 && d.kw == 3 && d.stride == 1 && d.pad == 1)) return false;
      // the kernel addresses its output (and shortcut) with 31-bit byte offsets; a call bounds it in elements only
      if ((size_t)d.n * d.c_out * d.h * d.w * dtype_size(d.dtype) >= ((size_t)1 << 31)) return false;
      const RowsArgs p = rows_tiles(d, tv, lay);
      const long groups = (long)((p.strips + tv.wn - 1) / tv.wn) * p.tiles_m;
      if (d.dtype == CPRUNE_F32 && ((long)d.c_in * 9 < kSplitMinTerms || tv.mb > 1 || tv.th > 6 || tv.ks > 2)) return false;
      if (tv.ks > 1 && tv.ks > (d.c_in + 31) / 32) return false;
      return groups * p.tiles_m < (1L << 32) && ((long)p.strips + 4) * p.tiles_x < (1L << 32) &&
             ((long)p.strips / p.tiles_x + 4) * p.tiles_y < (1L << 32);
    }
    if (!(lay.nhwc && (d.dtype == CPRUNE_F32 ? lay.w_rows3 && tv.mb == 1 && (tv.stride == 1 || tv.th <= 4) : lay.w_wave != nullptr) && d.kh == 3 && d.kw == 3 &&
          d.stride == tv.stride && d.pad == 1)) return false;
    if (lay.pool == 2 || (lay.pool && (((d.h | d.w) & 1) || tv.stride != 1 || (tv.th & 1)))) return false;
    if (lay.cp_out & 3) return false;      // four filters per store: not a dense map of logits
    const RowsArgs p = rows_tiles(d, tv, lay);
    const long waves = (long)p.strips * p.tiles_m;
    if (d.dtype == CPRUNE_F32) {
      if ((long)d.c_in * 9 < kSplitMinTerms) return false;      // as the split kernel
      if (split_packed_bytes(d.c_out, lay.cp_in, 9, d.dtype, true) >= ((size_t)1 << 31)) return false;
    }
    if (tv.ks > 1 && (tv.ks > (lay.cp_in + 31) / 32 || waves * tv.ks > 8192)) return false;
    // multiply-high divisions of the tile decode: exact while groups x divisor < 2^32
    const long tiles_m = p.tiles_m + (lay.pair ? (lay.pair->c_out + tv.tile_m() - 1) / tv.tile_m() : 0);
    const long groups = (long)((p.strips + tv.wn - 1) / tv.wn) * tiles_m;
    return groups * tiles_m < (1L << 32) && ((long)p.strips + 4) * p.tiles_x < (1L << 32) &&
           ((long)p.strips / p.tiles_x + 4) * p.tiles_y < (1L << 32);
  }
  if (tv.pw3) {
    // 1x1 / stride 1 or 2 in a handle; fp32 sums of at least 16 terms, as the split kernel; four filters per store
    const bool f32 = d.dtype == CPRUNE_F32;
    if (!(lay.nhwc && lay.w_rows3 && d.kh == 1 && d.kw == 1 && d.pad == 0 && d.stride <= 2)) return false;
    if (lay.pool || (lay.cp_out & 3) || (f32 && d.c_in < kSplitMinTerms)) return false;
    if (f32 ? tv.nb == 4 && tv.pw3 == 2 : tv.pw3 != 2) return false;      // (built: see CPRUNE_PW3_LIST)
    if (split_packed_bytes(d.c_out, lay.cp_in, 1, d.dtype, true) >= ((size_t)1 << 31)) return false;
    // multiply-high divisions of the decode: exact while dividend x divisor < 2^32
    long tiles_m;
    const long groups = pw3_groups(d, tv, &tiles_m);
    const long P = groups / tiles_m * tv.tile_p(), side = std::max(conv_out_dim(d.h, 1, d.stride, 0), conv_out_dim(d.w, 1, d.stride, 0));
    return groups * tiles_m < (1L << 32) && P * side < (1L << 32);
  }
  if (tv.sched == -4) {
    // 3x3 / stride 1 / pad 1 on small maps (every wavefront fetches its own weights: with many pixels the
    // tiled kernels, which share them through LDS, are the ones to use)
    if (!(lay.nhwc && lay.w_wave && d.kh == 3 && d.kw == 3 && d.stride == 1 && d.pad == 1)) return false;
    if (lay.pool == 2 || (lay.pool && ((d.h | d.w) & 1))) return false;
    if (!(d.h >= 3 && d.w >= 3 && d.h <= kMaxWaveMap && d.w <= kMaxWaveMap)) return false;
    // multiply-high divisions in the group decode: exact while groups x divisor < 2^32
    const long blocks = (long)d.n * ((d.h + 3) / 4) * ((d.w + 3) / 4);
    const long tiles_n = (blocks + tv.wn * tv.nb - 1) / (tv.wn * tv.nb);
    const long groups = tiles_n * ((d.c_out + 15) / 16);
    return groups * tiles_n < (1L << 32) && (blocks + 16) * 16 < (1L << 32);
  }
  if (tv.sched == -3) {
    // 1x1 / stride 1, no pool; exactly one (mb, nr) pair serves a shape: the smallest filter tile that
    // holds min(c_out, 128) filters and the smallest round count that holds the reduction
    if (!lay.nhwc || lay.pool || !(d.kh == 1 && d.kw == 1 && d.stride == 1 && d.pad == 0)) return false;
    const int rounds = (int)(((long)lay.cp_in * (long)dtype_size(d.dtype) + 63) / 64);
    const int nr = rounds <= 4 ? rounds : (rounds <= 6 ? 6 : 0);
    const int mb = d.c_out <= 32 ? 2 : (d.c_out <= 64 ? 4 : 8);
    return tv.nr == nr && tv.mb == mb;
  }
  if (tv.sched == -2) {
    // the reduction of a pixel is one contiguous run: 1x1 / stride 1, or a window that covers the whole map
    const bool pointwise = d.kh == 1 && d.kw == 1 && d.stride == 1 && d.pad == 0;
    const bool whole_map = d.pad == 0 && d.kh == d.h && d.kw == d.w;
    if (!lay.nhwc || !(pointwise || whole_map)) return false;
    if (lay.pool == 1 || (lay.pool == 2 && (d.c_out & 3))) return false;
    // made for few pixels: with many, the tiled kernels reuse their operands and this one does not
    const long P = (long)d.n * conv_out_dim(d.h, d.kh, d.stride, d.pad) * conv_out_dim(d.w, d.kw, d.stride, d.pad);
    const long groups = ((d.c_out + 15) / 16) * ((P + tv.tile_p() - 1) / tv.tile_p());
    return groups <= kMaxKsplitGroups;
  }
  if (tv.sched < 0) {
    if (!(lay.nhwc && d.kh == 3 && d.kw == 3 && d.stride == tv.stride && d.pad == 1)) return false;
    if (lay.pool == 2 || (lay.pool && ((d.h | d.w) & 1)) || (lay.pool && tv.stride != 1)) return false;
    const int ho = conv_out_dim(d.h, 3, d.stride, 1), wo = conv_out_dim(d.w, 3, d.stride, 1);   // = h, w at stride 1
    // multi-image tiles are for maps that fit one tile; single-image tiles for the rest
    if (tv.ni > 1 ? !(ho <= tv.th && wo <= tv.tw) : !(ho * 2 > tv.th && wo * 2 > tv.tw)) return false;
    // the kernels decode their tile with multiply-high divisions, exact while groups x divisor < 2^32
    const long tiles_s = (long)((d.n + tv.ni - 1) / tv.ni) * ((ho + tv.th - 1) / tv.th) * ((wo + tv.tw - 1) / tv.tw);
    const long groups = tiles_s * ((d.c_out + tv.tile_m() - 1) / tv.tile_m());
    return groups * tiles_s < (1L << 32);
  }
  if (lay.pool == 1) return false;                // only the patch kernels fuse a spatial pool
  if (lay.pool && lay.nhwc_out && !lay.nhwc) return false;
  if (lay.pool == 2 && !(lay.nhwc && (d.c_out & 3) == 0)) return false;
  const int ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  const long P = (long)d.n * ho * wo;
  const long K = (long)(lay.nhwc ? lay.cp_in : d.c_in) * d.kh * d.kw;
  const long kt = slab_k(d.dtype, tv.kq);
  const long units = ((d.c_out + tv.tile_m() - 1) / tv.tile_m()) * ((P + tv.tile_p() - 1) / tv.tile_p()) * ((K + kt - 1) / kt);
  return units < (1L << 30);
}

size_t variant_ws_bytes(const cprune_conv_desc& d, int v, const ConvLayout& lay) {
  const TileVariant& tv = variant(v);
  if (tv.split && !lay.nhwc) return split_packed_bytes(d.c_out, d.c_in, d.kh * d.kw, d.dtype);
  if (tv.sched < 0) return 0;
  const Plan p = make_plan(d, tv, lay);
  return p.fixup ? (size_t)2 * p.groups * tv.tile_m() * tv.tile_p() * sizeof(float) : 0;
}

size_t conv_ws_bytes(const cprune_conv_desc& d, int v, const ConvLayout& lay) {
  if (d.groups != 1) return 0;
  if (v >= 0) {
    return variant_supports(d, v, lay) ? variant_ws_bytes(d, v, lay) : 0;
  }
  // the most any variant needs: cut tiles, or (all alike) the packed weights of the split kernel
  size_t best = 0;
  bool split = false;
  for (int i = 0; i < num_variants(); ++i) {
    const TileVariant& tv = variant(i);
    if (tv.split ? lay.nhwc || split : tv.sched <= 0) continue;
    const size_t b = conv_ws_bytes(d, i, lay);
    if (tv.split && b) split = true;
    if (b > best) best = b;
  }
  return best;
}

int launch_conv_dense(const cprune_conv_desc& d, const void* x, const void* w, const float* bias,
                      const void* residual, void* y, int v, void* ws, hipStream_t s, const ConvLayout& lay) {
  const TileVariant& tv = variant(v);
  const size_t es = dtype_size(d.dtype);
  if (tv.split) return launch_split_conv(d, tv, lay, x, w, bias, residual, y, ws, s);
  if (tv.rows) {
    RowsS2Args a;
    (RowsArgs&)a = rows_tiles(d, tv, lay);
    if (tv.rows == 2) {
      a.x = x; a.w = w; a.bias = bias; a.res = residual; a.y = y;
      a.N = d.n; a.O = d.c_out; a.Cp = d.c_in; a.Cop = d.c_out;
      a.x_bytes = (unsigned)((size_t)d.n * d.c_in * d.h * d.w * es);
      a.w_bytes = (unsigned)((size_t)d.c_out * d.c_in * 9 * es);
      a.y_bytes = (unsigned)((size_t)d.n * d.c_out * d.h * d.w * es);
      a.w_raw = nullptr; a.w_raw_bytes = 0;
      a.nchunk = (d.c_in + 31) / 32; a.act = d.act; a.pool = 0; a.m_major = 0;
      a.magic_m = magic_for((unsigned)a.tiles_m); a.magic_x = magic_for((unsigned)a.tiles_x); a.magic_y = magic_for((unsigned)a.tiles_y);
      const dim3 grid((unsigned)((a.strips + tv.wn - 1) / tv.wn * a.tiles_m));
      const int rc = d.dtype == CPRUNE_F32 ? launch_conv_rows_nchw_f32(tv.patch_id, grid, s, a) :
                     d.dtype == CPRUNE_F16 ? launch_conv_rows_nchw_f16(tv.patch_id, grid, s, a) : launch_conv_rows_nchw_bf16(tv.patch_id, grid, s, a);
      if (rc != CPRUNE_OK) return rc;
      CPRUNE_LAUNCH_CHECK();
      return CPRUNE_OK;
    }
    a.x = x; a.w = lay.w_wave; a.bias = bias; a.res = residual; a.y = y;
    a.N = d.n; a.O = d.c_out; a.Cp = lay.cp_in; a.Cop = lay.cp_out;
    a.Hi = d.h; a.Wi = d.w;
    a.x_bytes = (unsigned)((size_t)d.n * lay.cp_in * d.h * d.w * es);
    a.w_bytes = (unsigned)wave_packed_bytes(d.c_out, lay.cp_in, d.dtype);
    if (d.dtype == CPRUNE_F32) {
      a.w = lay.w_rows3;
      a.w_bytes = (unsigned)split_packed_bytes(d.c_out, lay.cp_in, 9, d.dtype, true);
    }
    a.w_raw = w;
    a.w_raw_bytes = (unsigned)((size_t)d.c_out * 9 * lay.cp_in * es);
    a.y_bytes = (unsigned)((size_t)d.n * lay.cp_out * a.H * a.W * es);
    a.nchunk = (lay.cp_in + 31) / 32;
    a.act = d.act; a.pool = lay.pool;
    a.tiles_m1 = a.tiles_m;
    if (lay.pair) {
      const ConvPair& q = *lay.pair;
      a.tiles_m += (q.c_out + tv.tile_m() - 1) / tv.tile_m();
      a.w2 = q.w; a.w2_raw = q.w_raw; a.bias2 = q.bias; a.y2 = q.y; a.O2 = q.c_out; a.Cop2 = q.cp_out; a.act2 = q.act;
      a.w2_bytes = (unsigned)split_packed_bytes(q.c_out, lay.cp_in, 1, d.dtype, true);
      a.w2_raw_bytes = (unsigned)((size_t)q.c_out * lay.cp_in * es);
      a.y2_bytes = (unsigned)((size_t)d.n * q.cp_out * a.H * a.W * es);
    }
    const int groups_s = (a.strips + tv.wn - 1) / tv.wn;
    a.m_major = rows_m_major(a, groups_s, lay.pair != nullptr) ? groups_s : 0;
    a.magic_m = magic_for((unsigned)(a.m_major ? a.m_major : a.tiles_m)); a.magic_x = magic_for((unsigned)a.tiles_x); a.magic_y = magic_for((unsigned)a.tiles_y);
    const dim3 grid((unsigned)(groups_s * a.tiles_m));
    int rc;
    if (tv.stride == 2)
      rc = d.dtype == CPRUNE_F32 ? launch_conv_rows_s2_f32(tv.patch_id, grid, s, a) :
           d.dtype == CPRUNE_F16 ? launch_conv_rows_s2_f16(tv.patch_id, grid, s, a) : launch_conv_rows_s2_bf16(tv.patch_id, grid, s, a);
    else
      rc = d.dtype == CPRUNE_F32 ? launch_conv_rows_f32(tv.patch_id, grid, s, a) :
           d.dtype == CPRUNE_F16 ? launch_conv_rows_f16(tv.patch_id, grid, s, a) : launch_conv_rows_bf16(tv.patch_id, grid, s, a);
    if (rc != CPRUNE_OK) return rc;
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  if (tv.pw3) {
    Pw3Args a;
    a.x = x; a.w = lay.w_rows3; a.w_raw = w; a.bias = bias; a.res = residual; a.y = y;
    a.H = d.h; a.W = d.w; a.Ho = conv_out_dim(d.h, 1, d.stride, 0); a.Wo = conv_out_dim(d.w, 1, d.stride, 0);
    a.P = d.n * a.Ho * a.Wo; a.O = d.c_out; a.Cp = lay.cp_in; a.Cop = lay.cp_out; a.stride = d.stride;
    long tiles_m;
    const long groups = pw3_groups(d, tv, &tiles_m);
    const int blocks = (d.c_out + 15) / 16;
    a.tiles_m = (int)tiles_m; a.blk_base = blocks / a.tiles_m; a.blk_rem = blocks % a.tiles_m;
    a.rounds = (lay.cp_in + 31) / 32;
    a.x_bytes = (unsigned)((size_t)d.n * lay.cp_in * d.h * d.w * es);
    a.w_bytes = (unsigned)split_packed_bytes(d.c_out, lay.cp_in, 1, d.dtype, true);
    a.w_raw_bytes = (unsigned)((size_t)d.c_out * lay.cp_in * es);
    a.y_bytes = (unsigned)((size_t)a.P * lay.cp_out * es);
    a.magic_m = magic_for((unsigned)a.tiles_m); a.magic_wo = magic_for((unsigned)a.Wo); a.magic_ho = magic_for((unsigned)a.Ho);
    a.act = d.act;
    const dim3 grid((unsigned)groups);
    const int rc = d.dtype == CPRUNE_F32 ? launch_conv_pw3_f32(tv.patch_id, grid, s, a) :
                   d.dtype == CPRUNE_F16 ? launch_conv_pw3_f16(tv.patch_id, grid, s, a) : launch_conv_pw3_bf16(tv.patch_id, grid, s, a);
    if (rc != CPRUNE_OK) return rc;
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  if (tv.sched == -4) {
    PatchArgs pa;
    pa.x = x; pa.w = lay.w_wave; pa.bias = bias; pa.res = residual; pa.y = y;
    pa.N = d.n; pa.H = d.h; pa.W = d.w; pa.O = d.c_out; pa.Cp = lay.cp_in; pa.Cop = lay.cp_out;
    pa.pool = lay.pool;
    pa.tiles_y = (d.h + 3) / 4;
    pa.tiles_x = (d.w + 3) / 4;
    const long blocks = (long)d.n * pa.tiles_y * pa.tiles_x;
    pa.tiles_n = (int)((blocks + tv.wn * tv.nb - 1) / (tv.wn * tv.nb));   // groups along the block list
    pa.tiles_m = (d.c_out + 15) / 16;
    pa.x_bytes = (unsigned)((size_t)d.n * lay.cp_in * d.h * d.w * es);
    pa.w_bytes = (unsigned)wave_packed_bytes(d.c_out, lay.cp_in, d.dtype);
    pa.act = d.act;
    pa.vec_out = (lay.cp_out % 4) == 0 ? 1 : 0;
    pa.m_major = pa.w_bytes > pa.x_bytes ? 1 : 0;
    pa.magic_s = magic_for((unsigned)pa.tiles_n); pa.magic_m = magic_for((unsigned)pa.tiles_m);
    pa.magic_x = magic_for((unsigned)pa.tiles_x); pa.magic_y = magic_for((unsigned)pa.tiles_y);
    pa.magic_xy = magic_for((unsigned)(pa.tiles_x * pa.tiles_y));
    dim3 grid((unsigned)(pa.tiles_n * pa.tiles_m));
    int rc;
    if (d.dtype == CPRUNE_F32) rc = launch_conv_wave_f32(tv.patch_id, grid, s, pa);
    else if (d.dtype == CPRUNE_F16) rc = launch_conv_wave_f16(tv.patch_id, grid, s, pa);
    else rc = launch_conv_wave_bf16(tv.patch_id, grid, s, pa);
    if (rc != CPRUNE_OK) return rc;
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  if (tv.sched == -3) {
    ConvArgs a;
    a.x = x; a.w = w; a.bias = bias; a.res = residual; a.y = y; a.partial = nullptr;
    a.N = d.n; a.C = d.c_in; a.H = d.h; a.W = d.w; a.O = d.c_out; a.KH = 1; a.KW = 1; a.stride = 1; a.pad = 0;
    a.Ho = d.h; a.Wo = d.w;
    a.K = lay.cp_in; a.Cp = lay.cp_in; a.Cop = lay.cp_out;
    a.vec_out = (lay.cp_out % 4) == 0 ? 1 : 0;
    a.pool4 = 0; a.nhwc_out = 0;
    a.HoWo = d.h * d.w;
    a.P = d.n * a.HoWo;
    a.x_bytes = (unsigned)((size_t)a.P * lay.cp_in * es);
    a.w_bytes = (unsigned)((size_t)d.c_out * lay.cp_in * es);
    a.act = d.act;
    a.tiles_m = (d.c_out + tv.tile_m() - 1) / tv.tile_m();
    a.tiles_p = (a.P + 63) / 64;
    // persistent groups: as many as stay resident (LDS decides, at most 8 per compute unit), shared between
    // the filter tiles; each walks over its share of the pixel tiles
    const long lds = (long)tv.tile_m() * (tv.nr * 64 + 16);
    long per_cu = (160 * 1024) / lds;
    per_cu = per_cu > 8 ? 8 : (per_cu < 1 ? 1 : per_cu);
    long workers = 256 * per_cu / a.tiles_m;
    workers = workers < 1 ? 1 : (workers > a.tiles_p ? a.tiles_p : workers);
    dim3 grid((unsigned)workers, (unsigned)a.tiles_m);
    if (d.dtype == CPRUNE_F32) launch_conv_pw_f32(tv.patch_id, grid, s, a);
    else if (d.dtype == CPRUNE_F16) launch_conv_pw_f16(tv.patch_id, grid, s, a);
    else launch_conv_pw_bf16(tv.patch_id, grid, s, a);
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  if (tv.sched == -2) {
    ConvArgs a;
    a.x = x; a.w = w; a.bias = bias; a.res = residual; a.y = y; a.partial = nullptr;
    a.N = d.n; a.C = d.c_in; a.H = d.h; a.W = d.w; a.O = d.c_out; a.KH = d.kh; a.KW = d.kw;
    a.stride = d.stride; a.pad = d.pad;
    a.Ho = conv_out_dim(d.h, d.kh, d.stride, d.pad);
    a.Wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
    a.K = lay.cp_in * d.kh * d.kw;
    a.Cp = lay.cp_in; a.Cop = lay.cp_out;
    a.vec_out = (lay.cp_out % 4) == 0 ? 1 : 0;
    a.pool4 = lay.pool == 2 ? 1 : 0;
    a.nhwc_out = 0;
    a.HoWo = a.Ho * a.Wo;
    a.P = d.n * a.HoWo;
    a.x_bytes = (unsigned)((size_t)d.n * lay.cp_in * d.h * d.w * es);
    a.w_bytes = (unsigned)((size_t)d.c_out * a.K * es);
    a.act = d.act;
    a.tiles_m = (d.c_out + 15) / 16;
    a.tiles_p = (a.P + tv.tile_p() - 1) / tv.tile_p();
    a.magic_tp = magic_for((unsigned)a.tiles_p);   // at most kMaxKsplitGroups groups: exact
    if (lay.w_rows) {
      a.w = lay.w_rows;
      a.w_bytes = (unsigned)rows_packed_bytes(d.c_out, a.K, d.dtype);
      a.w_packed = 1;
    }
    dim3 grid((unsigned)(a.tiles_m * a.tiles_p));
    if (d.dtype == CPRUNE_F32) launch_conv_ksplit_f32(tv.patch_id, grid, s, a);
    else if (d.dtype == CPRUNE_F16) launch_conv_ksplit_f16(tv.patch_id, grid, s, a);
    else launch_conv_ksplit_bf16(tv.patch_id, grid, s, a);
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  if (tv.sched < 0) {
    PatchArgs pa;
    pa.x = x; pa.w = w; pa.bias = bias; pa.res = residual; pa.y = y;
    pa.N = d.n; pa.H = d.h; pa.W = d.w; pa.O = d.c_out; pa.Cp = lay.cp_in; pa.Cop = lay.cp_out;
    pa.tiles_n = (d.n + tv.ni - 1) / tv.ni;
    pa.pool = lay.pool;
    pa.Ho = conv_out_dim(d.h, 3, d.stride, 1); pa.Wo = conv_out_dim(d.w, 3, d.stride, 1);   // = h, w at stride 1
    pa.tiles_y = (pa.Ho + tv.th - 1) / tv.th;
    pa.tiles_x = (pa.Wo + tv.tw - 1) / tv.tw;
    pa.tiles_m = (d.c_out + tv.tile_m() - 1) / tv.tile_m();
    pa.x_bytes = (unsigned)((size_t)d.n * lay.cp_in * d.h * d.w * es);
    pa.w_bytes = (unsigned)((size_t)d.c_out * 9 * lay.cp_in * es);
    pa.act = d.act;
    pa.vec_out = (lay.cp_out % 4) == 0 ? 1 : 0;
    pa.m_major = pa.w_bytes > pa.x_bytes ? 1 : 0;
    pa.magic_s = magic_for((unsigned)(pa.tiles_n * pa.tiles_y * pa.tiles_x)); pa.magic_m = magic_for((unsigned)pa.tiles_m);
    pa.magic_x = magic_for((unsigned)pa.tiles_x); pa.magic_y = magic_for((unsigned)pa.tiles_y);
    pa.magic_xy = 0;
    dim3 pgrid((unsigned)(pa.tiles_n * pa.tiles_y * pa.tiles_x * pa.tiles_m));
    if (tv.stride == 2) {
      if (d.dtype == CPRUNE_F32) launch_conv_patch_s2_f32(tv.patch_id, pgrid, s, pa);
      else if (d.dtype == CPRUNE_F16) launch_conv_patch_s2_f16(tv.patch_id, pgrid, s, pa);
      else launch_conv_patch_s2_bf16(tv.patch_id, pgrid, s, pa);
    } else if (tv.blk32) {
      if (d.dtype == CPRUNE_F32) launch_conv_patch32_f32(tv.patch_id, pgrid, s, pa);
      else if (d.dtype == CPRUNE_F16) launch_conv_patch32_f16(tv.patch_id, pgrid, s, pa);
      else launch_conv_patch32_bf16(tv.patch_id, pgrid, s, pa);
    } else if (d.dtype == CPRUNE_F32) launch_conv_patch_f32(tv.patch_id, pgrid, s, pa);
    else if (d.dtype == CPRUNE_F16) launch_conv_patch_f16(tv.patch_id, pgrid, s, pa);
    else launch_conv_patch_bf16(tv.patch_id, pgrid, s, pa);
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  const Plan p = make_plan(d, tv, lay);
  ConvArgs a;
  a.x = x; a.w = w; a.bias = bias; a.res = residual; a.y = y; a.partial = (float*)ws;
  a.N = d.n; a.C = d.c_in; a.H = d.h; a.W = d.w; a.O = d.c_out; a.KH = d.kh; a.KW = d.kw;
  a.stride = d.stride; a.pad = d.pad;
  a.Ho = conv_out_dim(d.h, d.kh, d.stride, d.pad);
  a.Wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  a.K = (lay.nhwc ? lay.cp_in : d.c_in) * d.kh * d.kw;
  a.Cp = lay.cp_in;
  a.Cop = lay.cp_out;
  a.magic_cp = magic_for((unsigned)lay.cp_in);
  a.vec_out = (lay.cp_out % 4) == 0 ? 1 : 0;
  a.pool4 = lay.pool == 2 ? 1 : 0;
  a.nhwc_out = (!lay.nhwc && lay.nhwc_out) ? 1 : 0;
  a.HoWo = a.Ho * a.Wo;
  a.P = d.n * a.HoWo;
  a.HW = d.h * d.w;
  a.KHW = d.kh * d.kw;
  a.magic_khw = magic_for((unsigned)a.KHW);
  a.magic_kw = magic_for((unsigned)a.KW);
  a.x_bytes = (unsigned)((size_t)d.n * (lay.nhwc ? lay.cp_in : d.c_in) * d.h * d.w * es);
  a.w_bytes = (unsigned)((size_t)d.c_out * a.K * es);
  a.act = d.act;
  a.tiles_m = p.tiles_m;
  a.tiles_p = p.tiles_p;
  a.slabs = p.slabs;
  a.units = p.units;
  a.units_per_wg = p.units_per_wg;
  dim3 grid((unsigned)p.groups);
  const int tile = v / kNumScheds;  // implicit-GEMM variants come first in the table
  if (lay.nhwc) {
    if (d.dtype == CPRUNE_F32) launch_conv_nhwc_f32(tile, grid, s, a, p.fixup);
    else if (d.dtype == CPRUNE_F16) launch_conv_nhwc_f16(tile, grid, s, a, p.fixup);
    else launch_conv_nhwc_bf16(tile, grid, s, a, p.fixup);
  } else {
    if (d.dtype == CPRUNE_F32) launch_conv_f32(tile, grid, s, a, p.fixup);
    else if (d.dtype == CPRUNE_F16) launch_conv_f16(tile, grid, s, a, p.fixup);
    else launch_conv_bf16(tile, grid, s, a, p.fixup);
  }
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

bool conv_stem2_supported(const cprune_conv_desc& d2, const ConvLayout& lay2, int c_in, int c1) {
  if (!(c_in >= 1 && c_in <= 3 && c1 >= 1 && c1 <= 32 && d2.c_in == c1 && lay2.cp_in <= 32)) return false;
  if (!(lay2.nhwc && d2.groups == 1 && d2.kh == 3 && d2.kw == 3 && d2.stride == 1 && d2.pad == 1)) return false;
  if (d2.has_residual || lay2.pool == 2 || (lay2.pool && ((d2.h | d2.w) & 1))) return false;
  const long tiles = (long)d2.n * ((d2.h + 7) / 8) * ((d2.w + 15) / 16);
  const int mb = d2.c_out <= 16 ? 1 : (d2.c_out <= 32 ? 2 : 4);
  const long groups = tiles * ((d2.c_out + mb * 16 - 1) / (mb * 16));
  return groups * tiles < (1L << 32);   // multiply-high tile decode
}

int launch_conv_stem2(const cprune_conv_desc& d2, const ConvLayout& lay2, const void* x_nchw, int c_in,
                      const void* w1_packed, const float* b1, int c1, int act1, const void* w2, const float* b2,
                      void* y, hipStream_t s) {
  if (!conv_stem2_supported(d2, lay2, c_in, c1)) return CPRUNE_ERR_UNSUPPORTED;
  const size_t es = dtype_size(d2.dtype);
  const int mb = d2.c_out <= 16 ? 1 : (d2.c_out <= 32 ? 2 : 4);
  Stem2Args a;
  a.x = x_nchw; a.w1 = w1_packed; a.b1 = b1; a.C = c_in; a.C1 = c1; a.Cp1 = lay2.cp_in; a.act1 = act1;
  PatchArgs& pa = a.p;
  pa.x = nullptr; pa.w = w2; pa.bias = b2; pa.res = nullptr; pa.y = y;
  pa.N = d2.n; pa.H = d2.h; pa.W = d2.w; pa.O = d2.c_out; pa.Cp = lay2.cp_in; pa.Cop = lay2.cp_out;
  pa.tiles_n = d2.n;
  pa.pool = lay2.pool;
  pa.tiles_y = (d2.h + 7) / 8;
  pa.tiles_x = (d2.w + 15) / 16;
  pa.tiles_m = (d2.c_out + mb * 16 - 1) / (mb * 16);
  pa.x_bytes = 0;
  pa.w_bytes = (unsigned)((size_t)d2.c_out * 9 * lay2.cp_in * es);
  pa.act = d2.act;
  pa.vec_out = (lay2.cp_out % 4) == 0 ? 1 : 0;
  pa.m_major = 0;
  pa.magic_s = 0; pa.magic_xy = 0;
  pa.magic_m = magic_for((unsigned)pa.tiles_m);
  pa.magic_x = magic_for((unsigned)pa.tiles_x); pa.magic_y = magic_for((unsigned)pa.tiles_y);
  dim3 grid((unsigned)(pa.tiles_n * pa.tiles_y * pa.tiles_x * pa.tiles_m));
  int rc;
  if (d2.dtype == CPRUNE_F32) rc = launch_conv_stem2_f32(mb, grid, s, a);
  else if (d2.dtype == CPRUNE_F16) rc = launch_conv_stem2_f16(mb, grid, s, a);
  else rc = launch_conv_stem2_bf16(mb, grid, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

bool mbrow_form(int dt, int c_out, int cp_in, int* mb, int* xh) {
  static const int f32[][2] = {{2, 2}, {2, 3}, {2, 4}, {4, 4}, {4, 8}, {6, 8}, {6, 12}, {8, 12}};
  static const int half[][2] = {{2, 2}, {2, 4}, {4, 2}, {4, 4}, {6, 4}, {6, 6}, {8, 10}};
  *xh = 0;
  if (cp_in == 0) {
    *mb = c_out <= 16 ? 1 : c_out <= 32 ? 2 : c_out <= 64 ? 4 : c_out <= 96 ? 6 : 8;
    return true;
  }
  const int need = (cp_in * (int)dtype_size(dt) + 31) / 32;
  const int count = dt == CPRUNE_F32 ? 8 : 7;
  for (int i = 0; i < count; ++i) {
    const int* f = dt == CPRUNE_F32 ? f32[i] : half[i];
    if (f[0] * 16 >= c_out && f[1] >= need) { *mb = f[0]; *xh = f[1]; return true; }
  }
  return false;
}

bool mbrow_image_form(int dt, int c_out, int* mb, int* xh) {
  *mb = c_out <= 16 ? 1 : 2;
  *xh = dt == CPRUNE_F32 ? 4 : 2;
  return c_out <= 32;
}

}  // namespace cprune
