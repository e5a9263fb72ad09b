// C-ABI entry points: argument validation, the per-shape variant cache and
// on-device selection, the single-layer calls and the network handle.
#include "common.hpp"

#include <map>
#include <mutex>
#include <vector>
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>

namespace cprune {

static thread_local hipError_t g_last_hip_error = hipSuccess;
void set_last_hip_error(hipError_t e) { g_last_hip_error = e; }

// ---- descriptor validation ---------------------------------------------------
int validate_conv_desc(const cprune_conv_desc* d) {
  if (!d) return CPRUNE_ERR_INVALID_ARG;
  if (d->n < 1 || d->c_in < 1 || d->h < 1 || d->w < 1 || d->c_out < 1) return CPRUNE_ERR_INVALID_ARG;
  if (d->kh < 1 || d->kw < 1 || d->stride < 1 || d->pad < 0) return CPRUNE_ERR_INVALID_ARG;
  if (!dtype_ok(d->dtype) || !act_ok(d->act)) return CPRUNE_ERR_INVALID_ARG;
  if (d->has_residual != 0 && d->has_residual != 1) return CPRUNE_ERR_INVALID_ARG;
  if (d->groups < 1) return CPRUNE_ERR_INVALID_ARG;
  if (d->h + 2 * d->pad < d->kh || d->w + 2 * d->pad < d->kw) return CPRUNE_ERR_INVALID_ARG;
  if (d->groups != 1 && !(d->groups == d->c_in && d->c_out == d->c_in)) return CPRUNE_ERR_UNSUPPORTED;
  if (d->kh > 7 || d->kw > 7) return CPRUNE_ERR_UNSUPPORTED;
  if (d->pad >= d->kh || d->pad >= d->kw) return CPRUNE_ERR_UNSUPPORTED;  // every window holds a real element
  const long ho = conv_out_dim(d->h, d->kh, d->stride, d->pad), wo = conv_out_dim(d->w, d->kw, d->stride, d->pad);
  const long lim = 1L << 31;
  if (d->groups == 1) {  // the dense kernel addresses x and w with 31-bit byte offsets
    const long es = (long)dtype_size(d->dtype);
    if ((long)d->n * d->c_in * d->h * d->w * es >= lim) return CPRUNE_ERR_UNSUPPORTED;
    if ((long)d->c_out * d->c_in * d->kh * d->kw * es >= lim) return CPRUNE_ERR_UNSUPPORTED;
  }
  if ((long)d->n * d->c_in * d->h * d->w >= lim || (long)d->n * d->c_out * ho * wo >= lim) return CPRUNE_ERR_UNSUPPORTED;
  if ((long)d->c_out * (d->c_in / d->groups) * d->kh * d->kw >= lim) return CPRUNE_ERR_UNSUPPORTED;
  if ((long)d->c_in * d->kh * d->kw * d->kh * d->kw >= lim) return CPRUNE_ERR_UNSUPPORTED;  // exact magic division
  return CPRUNE_OK;
}

// ---- variant cache -------------------------------------------------------------
typedef std::array<int, 18> DescKey;
static DescKey key_of(const cprune_conv_desc& d, const ConvLayout& lay) {
  return DescKey{d.n, d.c_in, d.h, d.w, d.c_out, d.kh, d.kw, d.stride, d.pad, d.groups, d.dtype, d.act,
                 d.has_residual, lay.nhwc, lay.cp_in, lay.cp_out, lay.pool, lay.nhwc_out};
}
static std::mutex g_cache_mutex;
static std::map<DescKey, int> g_cache;
// Untimed choices of the boundary's layout, as cprune_cached_tile gives them (the Python entry asks it before each call, to size the
// scratch): the estimates take 4-6 us of the caller's thread, a look here 0.2.  They depend on the shape alone; at most kMaxChoices are
// kept.  A call with variant -1 chooses among what its scratch allows, and makes the estimates itself.
static std::map<DescKey, int> g_choices;
constexpr size_t kMaxChoices = 1024;
// likewise the variant a pair of layers in one launch runs, or -1 where the layers apart were faster
static std::map<std::array<int, 21>, int> g_pairs;

void remember_variant(const cprune_conv_desc& d, int v, const ConvLayout& lay) {
  std::lock_guard<std::mutex> lock(g_cache_mutex);
  g_cache[key_of(d, lay)] = v;
}

// Whether a choice considers the split kernel: inside a handle always; in the boundary's layout from 0.3 GFLOP up where
// variants are timed and from 0.6 untimed, because there the weights are packed on every call, by a launch of its own (4-8 us of
// the device, 3 us of the caller's thread, which bounds calls of under 20 us).  Timed, device time of this kernel / the best
// other, whole call: nine layers of 0.002-0.06 GFLOP 7.5-10.9 / 7.8-12.1 us, 17-19 / 14-17; 0.22 (89 -> 21 at 33x33 b6 bf16)
// 11.0 / 13.4, 17.8 / 15; 0.24 (28 -> 11 at 58x58 b13 fp32), whole call 16.2 / 14.4; 0.27 14.9 / 16.8, 16.9 / 17; three of 0.30-0.39
// 13.0-16.5 / 17.7-34, 17-18 / 18-34.  Untimed, 128 -> 83 filters at 56x56, batch 8, 74 -> 44 us in fp32 and 38 -> 22 us in bf16;
// on 232 layers under 0.8 GFLOP a line at 0.6 loses 5.5 % of the device time to the better kernel on average, one at 0.2 4.3 %,
// always the general kernel 7.1 %, always this one 14 %.
static bool split_pays(const cprune_conv_desc& d, const ConvLayout& lay, double line) {
  const long ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  return lay.nhwc || 2.0 * (double)d.n * ho * wo * d.c_out * d.c_in * d.kh * d.kw >= line;
}

// Whether an untimed layer takes the row-strip kernel where it runs (3x3 layers).  In the boundary's layout: see there; in a handle, 16-bit data: always (on 72 random
// layers 2.35 times as fast as the general kernel, at least 1.15 times).  fp32, against the split kernel: from 0.2 GFLOP up on maps one
// strip wide and 0.3 on wider ones whose strips are well filled (56 of 4 x 16 columns, not 32 of 3 x 16 or, with a pool, 56 of 5 x
// 16) and whose chunks of 32 channels are not mostly padding as well; there 1.12 times as fast on average (63 random layers of 28 to 400 us),
// 0.95 times at worst; the layers left out by the fill alone 0.9-1.07 times, and below the lines 0.7-1.2 times.  Stride 2 in fp32: from
// four chunks of channels up, on maps of two strips at most, to 1 GFLOP, and long chains from 0.2 (200 random layers, before / now: 73 met
// the line of 2 GFLOP and any chain, 1.12 times as fast on average, 17 of them slower: 181 -> 265 at 20x20, batch 14, 16.8 / 24.1, 683 -> 94 at
// 14x14, one image, 14.1 / 17.2; now 55, 1.20 times, 0.81 at worst); with one to
// three chunks 0.6-1.1 times: 18 -> 44 at 28x28, batch 2, 4.6 / 7.7 us; 16-bit data always (200 random layers: 1.74 times, 0.80 at worst).  A layer without the split kernel's copy (a smaller batch in a
// handle whose full batch runs row strips) has the general kernel's fp32 instruction in its place, and always takes them:
// ResNet-18 built for 32, 2 and 1 images 213 -> 198 and 269 -> 190 us, VGG-16 built for 64, 8 images 173 -> 141.
static bool rows_pay(const cprune_conv_desc& d, const ConvLayout& lay) {
  if (!lay.nhwc) {
    // no more than 5.5 GFLOP (45 -> 364 at 42x42, batch 29, fp32 105 / 121 us; in 16-bit data 10 from 64 channels up: 105 -> 60 at 43x43, batch
    // 30, bf16 26 / 20), few channels (fp32 4 -> 110 at 44x44, batch 5, 7.9 / 9.6), or, in fp32, a long chain of chunks under a small layer (247 ->
    // 13 at 8x8, batch 29, 13.8 / 15.6; 141 -> 13 at 12x12, one image, 10.3 / 12.2).  Over 1 GFLOP (16-bit 2) also none whose chunks of 32 channels are
    // padding to more than a tenth (16-bit three tenths): the split kernel counts channels in eights (8 -> 326 at 94x77, batch 9, fp32 68 / 90;
    // bf16 33 -> 285 at 97x101, batch 2, 21 / 25).  350 random layers a type, the kernels there were before / the untimed choice: fp32 1.20 times
    // the time on average, 0.81 at worst, bf16 1.42 and 0.93; 130 random layers a type: the untimed choice is 1.06 times the time of the timed one on average.
    const double flops = 18.0 * d.n * d.h * d.w * (double)d.c_out * d.c_in;
    const int padded = (d.c_in + 31) / 32 * 32;
    if (d.dtype != CPRUNE_F32) return d.c_in >= 4 && flops <= (d.c_in >= 64 ? 1e10 : 5.5e9) && (flops <= 2e9 || 10 * d.c_in >= 7 * padded);
    return d.c_in >= 8 && flops <= 5.5e9 && (flops <= 1e9 || 10 * d.c_in >= 9 * padded) &&
           (d.c_in <= 128 || flops >= (d.c_in <= 192 ? 2e7 : 4e8));
  }
  if (d.dtype != CPRUNE_F32 || !lay.w_split) return true;
  if (d.stride == 2) {
    const long ho = conv_out_dim(d.h, 3, 2, 1), wo = conv_out_dim(d.w, 3, 2, 1);
    const double flops = 18.0 * d.n * ho * wo * (double)d.c_out * d.c_in;
    return lay.cp_in >= 112 && wo <= 32 && (lay.cp_in <= 384 || flops >= 2e8) && flops <= 1e9;
  }
  const double flops = 18.0 * d.n * d.h * d.w * (double)d.c_out * d.c_in;
  if (d.w <= 16) return flops >= 2e8;
  const int step = lay.pool ? 12 : 14, strips = (d.w - 16 + step - 1) / step + 1;      // (as rows_tiles has them)
  const double cols = d.w / (16.0 * strips), chans = lay.cp_in / (32.0 * ((lay.cp_in + 31) / 32));
  return flops >= 3e8 && cols >= 0.85 && cols * chans >= 0.6;
}

// Untimed choice: the row-strip kernel where it pays; otherwise the cheapest by variant_cost among the general kernel's tiles,
// whole or cut into equal runs, and, for windows of more than one tap, the split kernel's variants where it pays, for 1x1 layers of a
// handle those of the 1x1 kernel on the 16-bit matrix cores (90 random fp32 layers: 1.50 times as fast as the general kernel's choice on
// average, none slower, 1.16 times the time of the timed choice; 80 in bf16: 1.44 and 1.12 times).
int heuristic_variant(const cprune_conv_desc& d, const ConvLayout& lay, size_t ws_limit) {
  double best = -1.0;
  const int rows = rows_pay(d, lay) ? best_rows_variant(d, lay, &best) : -1;
  if (rows >= 0) return rows;
  best = -1.0;
  int best_v = d.kh * d.kw > 1 ? (split_pays(d, lay, 6e8) ? best_split_variant(d, lay, &best) : -1) : best_pw3_variant(d, lay, &best);
  if (best_v < 0 || variant_ws_bytes(d, best_v, lay) > ws_limit) { best = -1.0; best_v = 0; }
  for (int v = 0; v < num_variants(); ++v) {
    const TileVariant& tv = variant(v);
    if (!(tv.sched == 0 || tv.sched == 2 || tv.sched == 4) || !variant_supports(d, v, lay)) continue;
    const double cost = variant_cost(d, v, lay);
    if (cost >= 0.0 && (best < 0.0 || cost < best) && variant_ws_bytes(d, v, lay) <= ws_limit) { best = cost; best_v = v; }
  }
  if (best < 0.0)  // none of those (a fused pool needs a patch kernel): first that runs
    for (int v = 0; v < num_variants(); ++v)
      if (variant_supports(d, v, lay)) return v;
  return best_v;
}

// The variant timed for exactly this shape and layout, or -1; also -1 where it does not run here: the key does not say
// which packed copies of its weights a handle's layer has.
static int timed_variant(const cprune_conv_desc& d, const ConvLayout& lay) {
  int v = -1;
  {
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    auto it = g_cache.find(key_of(d, lay));
    if (it != g_cache.end()) v = it->second;
  }
  return v >= 0 && variant_supports(d, v, lay) ? v : -1;
}

int cached_or_heuristic_variant(const cprune_conv_desc& d, bool* timed, const ConvLayout& lay) {
  const int v = timed_variant(d, lay);
  if (timed) *timed = v >= 0;
  if (v >= 0) return v;
  if (lay.nhwc || lay.nhwc_out) return heuristic_variant(d, lay);
  const DescKey key = key_of(d, lay);
  {
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    auto it = g_choices.find(key);
    if (it != g_choices.end()) return it->second;
  }
  const int choice = heuristic_variant(d, lay);
  std::lock_guard<std::mutex> lock(g_cache_mutex);
  if (g_choices.size() >= kMaxChoices) g_choices.clear();
  g_choices[key] = choice;
  return choice;
}

static int conv_dispatch(const cprune_conv_desc& d, const void* x, const void* w, const float* bias,
                         const void* residual, void* y, int v, void* ws, size_t ws_bytes, hipStream_t s,
                         const ConvLayout& lay = ConvLayout()) {
  if (d.groups != 1)
    return lay.nhwc ? launch_depthwise_nhwc(d, lay.cp_in, x, w, bias, residual, y, s)
                    : launch_conv_depthwise(d, x, w, bias, residual, y, s);
  if (v < 0) {
    // a timed choice needs the scratch it was timed with, except that a caller without room for packed weights gets a
    // kernel that packs none; an untimed choice takes what scratch there is
    const size_t have = ws ? ws_bytes : 0;
    v = timed_variant(d, lay);
    if (v < 0 || (variant(v).split && variant_ws_bytes(d, v, lay) > have)) v = heuristic_variant(d, lay, have);
  }
  const bool split = variant(v).split;      // (its launch finds out by itself whether it runs the layer)
  if (!split && !variant_supports(d, v, lay)) return CPRUNE_ERR_UNSUPPORTED;
  const size_t need = variant_ws_bytes(d, v, lay);
  if (need > 0 && (!ws || ws_bytes < need))
    return split && !variant_supports(d, v, lay) ? CPRUNE_ERR_UNSUPPORTED : CPRUNE_ERR_WORKSPACE;
  return launch_conv_dense(d, x, w, bias, residual, y, v, ws, s, lay);
}

// Times every supported variant on the given buffers; returns the fastest.  Two stages: every
// variant briefly, then the few best again with more repetitions, so that a short disturbance
// (another process's burst, a clock change) during one measurement does not decide the choice.
static int select_tile_impl(const cprune_conv_desc& d, const void* x, const void* w, const float* bias,
                            const void* residual, void* y, void* ws, size_t ws_bytes, int warmup,
                            int iters, int* variant_out, float* best_ms_out, float* all_ms_out,
                            hipStream_t s, const ConvLayout& lay = ConvLayout()) {
  hipEvent_t e0, e1;
  CPRUNE_HIP_TRY(hipEventCreate(&e0));
  hipError_t ee = hipEventCreate(&e1);
  if (ee != hipSuccess) { hipEventDestroy(e0); set_last_hip_error(ee); return CPRUNE_ERR_DEVICE; }
  int rc = CPRUNE_OK;
  // fastest of `passes` timed passes of `n` launches each, per launch
  auto time_variant = [&](int v, int n, int passes, float* ms_out) -> int {
    float ms = 0.0f;
    for (int pass = 0; pass < passes; ++pass) {
      int r = CPRUNE_OK;
      hipError_t e = hipEventRecord(e0, s);
      for (int i = 0; i < n && r == CPRUNE_OK; ++i) r = conv_dispatch(d, x, w, bias, residual, y, v, ws, ws_bytes, s, lay);
      if (r != CPRUNE_OK) return r;
      if (e == hipSuccess) e = hipEventRecord(e1, s);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      float t = 0.0f;
      if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
      if (e != hipSuccess) { set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
      t /= (float)n;
      if (pass == 0 || t < ms) ms = t;
    }
    *ms_out = ms;
    return CPRUNE_OK;
  };
  std::vector<std::pair<float, int>> timed;
  int supported = d.groups == 1 ? 0 : 1;   // variants that can run the shape (timed or not)
  const int nv = d.groups == 1 ? num_variants() : 1;
  for (int v = 0; v < nv && rc == CPRUNE_OK; ++v) {
    if (all_ms_out) all_ms_out[v] = -1.0f;
    if (d.groups == 1) {
      if (!variant_supports(d, v, lay)) continue;
      ++supported;
      if (variant(v).split && !split_pays(d, lay, 3e8)) continue;
      if (conv_ws_bytes(d, v, lay) > ws_bytes) continue;  // not timed: the caller's scratch cannot run it
    }
    for (int i = 0; i < warmup && rc == CPRUNE_OK; ++i) rc = conv_dispatch(d, x, w, bias, residual, y, v, ws, ws_bytes, s, lay);
    if (rc != CPRUNE_OK) break;
    float ms = 0.0f;
    rc = time_variant(v, iters, 2, &ms);
    if (rc != CPRUNE_OK) break;
    if (all_ms_out) all_ms_out[v] = ms;
    timed.emplace_back(ms, v);
  }
  if (rc == CPRUNE_OK && timed.size() > 1) {
    std::sort(timed.begin(), timed.end());
    const size_t finalists = timed.size() < 4 ? timed.size() : 4;
    for (size_t k = 0; k < finalists && rc == CPRUNE_OK; ++k) {
      float ms = 0.0f;
      rc = time_variant(timed[k].second, 3 * iters, 3, &ms);
      if (rc != CPRUNE_OK) break;
      timed[k].first = ms;
      if (all_ms_out) all_ms_out[timed[k].second] = timed[k].first;
    }
    std::sort(timed.begin(), timed.begin() + finalists);
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  if (rc != CPRUNE_OK) return rc;
  if (timed.empty()) return supported ? CPRUNE_ERR_WORKSPACE : CPRUNE_ERR_UNSUPPORTED;
  const int best_v = timed[0].second;
  if (d.groups == 1) remember_variant(d, best_v, lay);
  if (variant_out) *variant_out = best_v;
  if (best_ms_out) *best_ms_out = timed[0].first;
  return CPRUNE_OK;
}

}  // namespace cprune

using namespace cprune;

extern "C" const char* cprune_status_string(int status) {
  switch (status) {
    case CPRUNE_OK: return "ok";
    case CPRUNE_ERR_INVALID_ARG: return "invalid argument";
    case CPRUNE_ERR_UNSUPPORTED: return "unsupported configuration";
    case CPRUNE_ERR_WORKSPACE: return "workspace too small";
    case CPRUNE_ERR_DEVICE: return "HIP call failed";
    case CPRUNE_ERR_NOT_TUNED: return "shape not tuned";
    default: return "unknown status";
  }
}

extern "C" int cprune_last_hip_error(void) { return (int)g_last_hip_error; }

extern "C" int cprune_num_tile_variants(void) { return num_variants(); }

extern "C" int cprune_tile_variant_info(int v, int* tile_m, int* tile_p, int* sched) {
  if (v < 0 || v >= num_variants()) return CPRUNE_ERR_INVALID_ARG;
  const TileVariant& tv = variant(v);
  if (tile_m) *tile_m = tv.step_m();
  if (tile_p) *tile_p = tv.tile_p();
  if (sched) *sched = tv.sched;
  return CPRUNE_OK;
}

extern "C" int cprune_tile_variant_name(int v, int channels_last, cprune_dtype dtype, char* buf, size_t buf_bytes) {
  if (v < 0 || v >= num_variants() || !buf || buf_bytes < 1 || !dtype_ok(dtype)) return CPRUNE_ERR_INVALID_ARG;
  const TileVariant& tv = variant(v);
  const char* t = dtype == CPRUNE_F32 ? "float" : dtype == CPRUNE_F16 ? "_Float16" : "__bf16";
  int n;
  if (tv.sched >= 0)
    n = snprintf(buf, buf_bytes, "%s<%s, %d, %d, %d, %d, %d>", channels_last ? "conv_nhwc_kernel" : "conv_igemm_kernel", t,
                 tv.wm, tv.wn, tv.mb, tv.nb, tv.kq);
  else if (tv.split)
    n = snprintf(buf, buf_bytes, "conv_split_kernel<%s, %s, %d, %d, %d, %d, %d, %d>", t, channels_last ? "false" : "true", tv.wm,
                 tv.wn, tv.ks, tv.mb, tv.nb, tv.nib);
  else if (tv.rows == 1 && tv.stride == 1 && channels_last && dtype == CPRUNE_F32)
    n = snprintf(buf, buf_bytes, "conv_split_rows_kernel<%d, %d>", tv.th, tv.ks);
  else if (tv.rows == 2)
    n = snprintf(buf, buf_bytes, "conv_rows_nchw_kernel<%s, %d, %d, %d>", t, tv.mb, tv.th, tv.ks);
  else if (tv.rows && tv.stride == 2)
    n = snprintf(buf, buf_bytes, "conv_rows_s2_kernel<%s, %d, %d, %d>", t, tv.mb, tv.th, tv.ks);
  else if (tv.pw3)
    n = snprintf(buf, buf_bytes, "conv_pw3_kernel<%s, %d, %d, %s>", t, tv.mb, tv.nb, tv.pw3 == 2 ? "true" : "false");
  else if (tv.rows)
    n = snprintf(buf, buf_bytes, "conv_rows_kernel<%s, %d, %d, %d>", t, tv.mb, tv.th, tv.ks);
  else if (tv.sched == -4)
    n = snprintf(buf, buf_bytes, "conv_wave_kernel<%s, %d, %d, %d>", t, tv.wn, tv.nb, tv.ks);
  else if (tv.sched == -3)
    n = snprintf(buf, buf_bytes, "conv_pw_kernel<%s, %d, %d>", t, tv.mb, tv.nr);
  else if (tv.sched == -2)
    n = snprintf(buf, buf_bytes, "conv_ksplit_kernel<%s, %d, %d>", t, tv.nb, tv.kwaves);
  else if (tv.blk32)
    n = snprintf(buf, buf_bytes, "conv_patch32_kernel<%s, %d, %d, %d, %d, %d, %d, %d>", t, tv.mb / 2, tv.nb / 2, tv.wn, tv.th,
                 tv.tw, tv.ni, tv.kq);
  else if (tv.stride == 2)
    n = snprintf(buf, buf_bytes, "conv_patch_s2_kernel<%s, %d, %d, %d, %d>", t, tv.mb, tv.th, tv.tw, tv.kq);
  else
    n = snprintf(buf, buf_bytes, "conv_patch_kernel<%s, %d, %d, %d, %d, %d, %d>", t, tv.mb, tv.th, tv.tw, tv.ni, tv.kq, tv.ks);
  return (n < 0 || (size_t)n >= buf_bytes) ? CPRUNE_ERR_INVALID_ARG : CPRUNE_OK;
}

extern "C" size_t cprune_conv_workspace_bytes(const cprune_conv_desc* desc, int v) {
  if (validate_conv_desc(desc) != CPRUNE_OK) return 0;
  if (v >= num_variants()) return 0;
  return conv_ws_bytes(*desc, v);
}

extern "C" int cprune_conv2d_bn_relu(const cprune_conv_desc* desc, const void* x, const void* w,
                                     const float* bias, const void* residual, void* y, int tile_variant,
                                     void* ws, size_t ws_bytes, void* stream) {
  int rc = validate_conv_desc(desc);
  if (rc != CPRUNE_OK) return rc;
  if (!x || !w || !y) return CPRUNE_ERR_INVALID_ARG;
  if ((desc->has_residual != 0) != (residual != nullptr)) return CPRUNE_ERR_INVALID_ARG;
  if (tile_variant < -1 || tile_variant >= num_variants()) return CPRUNE_ERR_INVALID_ARG;
  return conv_dispatch(*desc, x, w, bias, residual, y, tile_variant, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" int cprune_select_tile(const cprune_conv_desc* desc, const void* x, const void* w,
                                  const float* bias, const void* residual, void* y, void* ws,
                                  size_t ws_bytes, int warmup, int iters, int* variant_out,
                                  float* best_ms_out, float* all_ms_out, void* stream) {
  int rc = validate_conv_desc(desc);
  if (rc != CPRUNE_OK) return rc;
  if (!x || !w || !y || !variant_out) return CPRUNE_ERR_INVALID_ARG;
  if ((desc->has_residual != 0) != (residual != nullptr)) return CPRUNE_ERR_INVALID_ARG;
  if (warmup < 0 || iters < 1) return CPRUNE_ERR_INVALID_ARG;
  return select_tile_impl(*desc, x, w, bias, residual, y, ws, ws ? ws_bytes : 0, warmup, iters, variant_out,
                          best_ms_out, all_ms_out, (hipStream_t)stream);
}

extern "C" void cprune_clear_tile_cache(void) {
  std::lock_guard<std::mutex> lock(g_cache_mutex);
  g_cache.clear();
  g_choices.clear();
  g_pairs.clear();
}

extern "C" int cprune_cached_tile(const cprune_conv_desc* desc, int* variant_out, int* was_timed_out) {
  int rc = validate_conv_desc(desc);
  if (rc != CPRUNE_OK) return rc;
  if (!variant_out) return CPRUNE_ERR_INVALID_ARG;
  if (desc->groups != 1) return CPRUNE_ERR_UNSUPPORTED;
  bool timed = false;
  *variant_out = cached_or_heuristic_variant(*desc, &timed);
  if (was_timed_out) *was_timed_out = timed ? 1 : 0;
  return CPRUNE_OK;
}

extern "C" int cprune_maxpool2d(const void* x, int n, int c, int h, int w, int k, int stride, int pad,
                                cprune_dtype dtype, void* y, void* stream) {
  if (!x || !y || n < 1 || c < 1 || h < 1 || w < 1 || k < 1 || stride < 1 || pad < 0) return CPRUNE_ERR_INVALID_ARG;
  if (!dtype_ok(dtype) || h + 2 * pad < k || w + 2 * pad < k) return CPRUNE_ERR_INVALID_ARG;
  if (pad >= k) return CPRUNE_ERR_UNSUPPORTED;
  if ((long)n * c * h * w >= (1L << 31)) return CPRUNE_ERR_UNSUPPORTED;
  return launch_maxpool(x, n, c, h, w, k, stride, pad, dtype, y, (hipStream_t)stream);
}

extern "C" int cprune_global_avgpool(const void* x, int n, int c, int h, int w, cprune_dtype dtype,
                                     void* y, void* stream) {
  if (!x || !y || n < 1 || c < 1 || h < 1 || w < 1 || !dtype_ok(dtype)) return CPRUNE_ERR_INVALID_ARG;
  if ((long)n * c * h * w >= (1L << 31)) return CPRUNE_ERR_UNSUPPORTED;
  return launch_gavgpool(x, n, c, h * w, dtype, y, (hipStream_t)stream);
}

static cprune_conv_desc fc_desc(int n, int f, int c_out, int act, int dtype) {
  cprune_conv_desc d;
  d.n = n; d.c_in = f; d.h = 1; d.w = 1; d.c_out = c_out; d.kh = 1; d.kw = 1; d.stride = 1; d.pad = 0;
  d.groups = 1; d.dtype = dtype; d.act = act; d.has_residual = 0;
  return d;
}

extern "C" size_t cprune_fc_workspace_bytes(int n, int f, int c_out, cprune_dtype dtype) {
  if (n < 1 || f < 1 || c_out < 1 || !dtype_ok(dtype)) return 0;
  cprune_conv_desc d = fc_desc(n, f, c_out, CPRUNE_ACT_NONE, dtype);
  return conv_ws_bytes(d, -1);
}

extern "C" int cprune_fc(const void* x, const void* w, const float* bias, int n, int f, int c_out,
                         cprune_act act, cprune_dtype dtype, void* y, void* ws, size_t ws_bytes,
                         void* stream) {
  if (n < 1 || f < 1 || c_out < 1 || !x || !w || !y) return CPRUNE_ERR_INVALID_ARG;
  if (!dtype_ok(dtype) || !act_ok(act)) return CPRUNE_ERR_INVALID_ARG;
  cprune_conv_desc d = fc_desc(n, f, c_out, act, dtype);
  int rc = validate_conv_desc(&d);
  if (rc != CPRUNE_OK) return rc;
  // the remembered or heuristic variant, or its one-tile-per-group twin when the
  // caller's scratch is too small for cut tiles
  int v = cached_or_heuristic_variant(d, nullptr);
  if (conv_ws_bytes(d, v) > (ws ? ws_bytes : 0)) {
    int twin = -1;
    for (int i = 0; i < num_variants(); ++i)
      if (variant_supports(d, i) && variant(i).sched == 0 && variant(i).tile_m() == variant(v).tile_m() &&
          variant(i).tile_p() == variant(v).tile_p()) { twin = i; break; }
    if (twin < 0) return CPRUNE_ERR_WORKSPACE;
    v = twin;
  }
  return launch_conv_dense(d, x, w, bias, nullptr, y, v, ws, (hipStream_t)stream);
}

// ---- network handle ------------------------------------------------------------
// Inside a handle everything is channels-last: activations [n][h][w][cp], dense weights
// [c_out][kh][kw][cp], depthwise weights [kh][kw][cp], with cp the channel count rounded up
// to one 16-byte vector (pad channels are zero and stay zero through every layer).  The
// boundary stays NCHW: a dense first layer with few input channels reads the caller's tensor
// as it is (any other reader gets a converted copy); activations are converted on the way out.
// What a work-group of a depthwise layer inside its 1x1 reader's kernel owns: strips of a map (mbrow_kernel.hpp), or, 5x5 windows
// only, 8 x 8 output pixels (dwproj_kernel.hpp).
enum DwTile { kTallStrips = 0, kLowStrips = 1, kPixelBlocks = 2 };

struct NetLayer {
  cprune_layer_desc d;
  int h_in, w_in, h_out, w_out;
  int cp_in = 0, cp_out = 0;  // channel strides of the input / output buffers
  void* w = nullptr;
  float* b = nullptr;
  void* act = nullptr;        // [max_batch][h_out][w_out][cp_out]
  size_t per_image = 0;       // elements per image of the output buffer
  int variant = -1;           // dense conv / fc: variant for max_batch
  bool timed = false;         // ... chosen by timing or pinned, not estimated
  std::vector<int> at_batch;  // dense conv / fc: variant chosen for a smaller batch, by batch (-1: not yet)
  bool fused_pool = false;    // conv: the 2x2 max-pool that follows runs in its epilogue; act is the pooled map
  bool alias = false;         // max-pool folded into its producer: no kernel, act is the producer's buffer
  bool map2x2 = false;        // 3x3 / stride 1 / pad 1 conv on a 2x2 map, run as one matrix over the whole map
  int fuse_dw = -1;           // 1x1 conv: index of the depthwise layer computed inside its kernel, or -1
  int dw_ks = 0;              // ... and how many wavefronts share a strip there (1, 2, 4, 8; 0: not timed), or a pixel block (4, 8)
  int dw_tile = kLowStrips;   // ... and what a work-group owns (DwTile)
  bool fused_away = false;    // depthwise conv that runs inside its consumer's kernel (no launch, no activation)
  float* w_dw32 = nullptr;    // ... 16-bit data, 3x3: its weights as fp32, for the strip kernel
  int dw_reader = -1;         // depthwise conv that may run inside the 1x1 conv dw_reader's kernel
  int fuse_block = -1;        // 1x1 conv with fuse_dw set: index of the 1x1 expansion in front of that depthwise
                              // layer when the whole block (expansion, depthwise, this projection) is one kernel
  int block_ks = 0;           // ... and how many wavefronts share a strip there
  int block_low = 1;          // ... and whether its strips are the low ones
  int block_expand = -1;      // depthwise conv: the expansion layer that may join it and dw_reader in one kernel
  void* w_expand = nullptr;   // expansion of such a block: weights once more, in that kernel's operand order
  void* w_proj = nullptr;     // 1x1 conv that may run behind a depthwise layer in one kernel: weights in its operand order
  int pair = -1;              // 3x3 / stride 2 conv: index of the 1x1 / stride 2 layer on the same input that runs in its launch, or -1
  int pair_by = -1;           // that 1x1 layer: index of the 3x3 layer whose launch it runs in now, or -1
  int pair_with = -1;         // 3x3 layer: the 1x1 layer that could run in its launch
  int pair_variant = -1;      // ... variant of the pair at max_batch
  bool pinned = false;        // the caller has named the variant
  std::vector<int> pair_at;   // ... and at a smaller batch (-1: not yet)
  int fuse_stem = -1;         // 3x3 conv: index of the first layer (on the image) computed inside its kernel, or -1
  int stem_reader = -1;       // first layer that may run inside the 3x3 conv stem_reader's kernel
  void* w_stem = nullptr;     // weights packed for the first-layer kernel
  void* w_rows = nullptr;     // layer the reduction-split kernel can run: weights once more, in its operand order
  void* w_wave = nullptr;     // 3x3 / stride 1 / pad 1 layer: weights once more, packed for the independent-wavefront kernel
                              // (small maps) and, in 16-bit data, the row-strip kernel
  void* w_split = nullptr;    // fp32 dense layer: weights once more, cut and packed for the split kernel
  void* w_rows3 = nullptr;    // fp32 3x3 / pad 1 layer, or 1x1 layer of any type: likewise, for the row-strip (the 1x1) kernel
  bool stem = false;          // nchw_in layer that runs the first-layer kernel (whole reduction in LDS)
  void* w_stem7b = nullptr;   // ... 16-bit data, up to 48 filters or a dense last map: packed for its kernel in 16 x 16 blocks
  void* w_stem7 = nullptr;    // 7x7 / stride 2 / pad 3 first layer: weights packed for the kernel made for it
  int stem7 = 0;              // 1: that kernel runs the layer; 2: and the 3x3 / stride 2 max-pool pool3 with it; 3 (fp32): the same,
                              // and the conv map is stored too
  int pool3 = -1;             // the max-pool that can run inside that kernel (the layer's only reader), or -1
  bool in_producer = false;   // max-pool computed inside its producer's kernel: no launch, its buffer is written there
  int stem_ok = 0;            // that kernel exists for the layer's window and stride
  bool nchw_in = false;       // dense conv on the network input: reads the caller's NCHW tensor and its own
                              // OIHW weights, writes channels-last (no layout conversion pass)
};

struct GraphKey {
  int n; const void* x; void* logits;
  bool operator<(const GraphKey& o) const {
    if (n != o.n) return n < o.n;
    if (x != o.x) return x < o.x;
    return logits < o.logits;
  }
};

struct cprune_net {
  std::vector<NetLayer> layers;
  int in_c, in_h, in_w, in_cp, max_batch, dtype;
  std::vector<void*> allocs;
  void* x_cl = nullptr;       // the network input, channels-last
  bool tuned = false;         // forms and variants were timed at creation
  bool convert_input = true;  // false when every reader of the input takes the caller's NCHW tensor itself
  void* ws = nullptr;
  size_t ws_bytes = 0;
  struct GraphEntry { hipGraphExec_t exec; uint64_t last_use; };
  std::map<GraphKey, GraphEntry> graphs;   // at most kMaxGraphs: the least recently used one makes room
  uint64_t graph_clock = 0;
  hipStream_t capture_stream = nullptr;  // graphs are recorded here (the caller's may be the null stream)
  int last_n = 0;
};

// A fully connected layer is a convolution whose kernel covers its whole input map.
static cprune_conv_desc layer_conv_desc(const cprune_net& net, const NetLayer& L, int n) {
  cprune_conv_desc d;
  d.n = n; d.c_in = L.d.c_in; d.c_out = L.d.c_out; d.dtype = net.dtype; d.act = L.d.act;
  d.has_residual = L.d.residual >= 0 ? 1 : 0;
  d.h = L.h_in; d.w = L.w_in;
  if (L.map2x2) {
    // channels-last, a 2x2 map of cp channels is one vector of 4 * cp values per image
    d.c_in = 4 * L.cp_in; d.c_out = 4 * round_up_vec(L.d.c_out, net.dtype);
    d.h = d.w = 1; d.kh = d.kw = 1; d.stride = 1; d.pad = 0; d.groups = 1;
    return d;
  }
  if (L.d.kind == CPRUNE_LAYER_FC) {
    d.kh = L.h_in; d.kw = L.w_in; d.stride = 1; d.pad = 0; d.groups = 1;
  } else {
    d.kh = d.kw = L.d.k; d.stride = L.d.stride; d.pad = L.d.pad; d.groups = L.d.groups;
  }
  return d;
}

static ConvLayout layer_layout(const NetLayer& L) {
  ConvLayout lay;
  lay.nhwc = 1; lay.cp_in = L.cp_in; lay.cp_out = L.cp_out; lay.pool = L.fused_pool ? 1 : 0;
  lay.w_wave = L.w_wave;
  lay.w_rows = L.w_rows;
  lay.w_split = L.w_split;
  lay.w_rows3 = L.w_rows3;
  if (L.nchw_in) { lay.nhwc = 0; lay.nhwc_out = 1; lay.cp_in = 0; return lay; }
  if (L.map2x2) {
    lay.cp_in = 4 * L.cp_in;
    if (L.fused_pool) lay.pool = 2;   // rows ordered (channel, pixel); cp_out stays the pooled map's stride
    else lay.cp_out = 4 * L.cp_out;
  }
  return lay;
}

// 3x3 / stride 1 or 2 / pad 1 on a map of its own: what the row-strip and, at stride 1, the independent-wavefront kernels run.
static bool strips_layer(const cprune_net& net, const NetLayer& L) {
  return L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1 && L.d.k == 3 && L.d.stride <= 2 && L.d.pad == 1 && !L.map2x2 && !L.nchw_in &&
         wave_packed_bytes(L.d.c_out, L.cp_in, net.dtype) < ((size_t)1 << 31);      // 31-bit offsets in the kernels
}

// ... on a map that the independent-wavefront kernel takes: it keeps the copy that kernel reads
static bool wave_layer(const cprune_net& net, const NetLayer& L) {
  return strips_layer(net, L) && L.d.stride == 1 && L.h_in >= 3 && L.w_in >= 3 && L.h_in <= 32 && L.w_in <= 32;
}

// The other copies of a dense layer's weights are made only for a layer that runs the kernel that reads them (while variants are
// timed, for every layer that could): fp32, cut and packed for the split, the row-strip and the 1x1 kernel, each 1.5 times the weights or
// more; 16-bit data, the 1x1 kernel's, and the row-strip kernel's copy on maps that are not the independent-wavefront kernel's, as large as the weights.
static ConvLayout layout_if_packed(const cprune_net& net, const NetLayer& L) {
  ConvLayout lay = layer_layout(L);      // (only whether the copies are set matters to a choice)
  if (net.dtype == CPRUNE_F32 && !L.nchw_in) lay.w_split = lay.w_rows3 = L.w;
  if (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1 && L.d.k == 1 && !L.nchw_in) lay.w_rows3 = L.w;
  if (net.dtype != CPRUNE_F32 && !lay.w_wave && strips_layer(net, L)) lay.w_wave = L.w;
  return lay;
}

// the copy variant v reads, if it reads one
static int pack_for(cprune_net* net, NetLayer& L, int v, hipStream_t s) {
  const bool f32 = net->dtype == CPRUNE_F32, pw = variant(v).pw3, rows = variant(v).rows || pw;
  if (!rows && !(f32 && variant(v).split)) return CPRUNE_OK;
  void*& slot = !rows ? L.w_split : f32 || pw ? L.w_rows3 : L.w_wave;
  if (slot) return CPRUNE_OK;
  const cprune_conv_desc d = layer_conv_desc(*net, L, net->max_batch);
  const int cp = layer_layout(L).cp_in, taps = d.kh * d.kw;
  const bool split = f32 || pw;
  void* copy = nullptr;
  CPRUNE_HIP_TRY(hipMalloc(&copy, split ? split_packed_bytes(d.c_out, cp, taps, net->dtype, rows) : wave_packed_bytes(d.c_out, cp, net->dtype)));
  net->allocs.push_back(copy);
  slot = copy;
  return split ? launch_pack_split(L.w, d.c_out, cp, taps, 1, net->dtype, copy, s, rows) : launch_repack_wave(L.w, d.c_out, cp, net->dtype, copy, s);
}

// gives back what variant v (-1: none) does not read (nothing that reads it is in flight)
static void drop_copies(cprune_net* net, NetLayer& L, int v) {
  for (void** slot : {&L.w_split, &L.w_rows3, &L.w_wave}) {
    if (!*slot || (v >= 0 && (slot == &L.w_split ? variant(v).split : variant(v).rows || variant(v).pw3))) continue;
    if (slot == &L.w_wave && wave_layer(*net, L)) continue;
    net->allocs.erase(std::find(net->allocs.begin(), net->allocs.end(), *slot));
    hipFree(*slot);
    *slot = nullptr;
  }
}

// The opening of the ImageNet networks, which has kernels of its own.
// (fp32: not as a last layer whose map lies dense in the caller's buffer, which its kernel stores four filters at a time)
static bool stem7_layer(const NetLayer& L, int dtype) {
  return L.nchw_in && L.d.c_in <= 3 && L.d.k == 7 && L.d.stride == 2 && L.d.pad == 3 && L.d.residual < 0 &&
         !(dtype == CPRUNE_F32 && (L.cp_out & 3));
}

constexpr size_t kMaxGraphs = 8;

static void drop_graphs(cprune_net* net) {
  for (auto& g : net->graphs) hipGraphExecDestroy(g.second.exec);
  net->graphs.clear();
}

static void net_free(cprune_net* net) {
  drop_graphs(net);
  if (net->capture_stream) hipStreamDestroy(net->capture_stream);
  for (void* p : net->allocs) hipFree(p);
  delete net;
}

// The first-layer kernel on the caller's NCHW input.
static int net_run_stem(cprune_net* net, int i, int n, const void* x, void* dst, hipStream_t s) {
  const NetLayer& L = net->layers[i];
  StemArgs a;
  a.x = x; a.w = L.w_stem; a.bias = L.b; a.y = dst;
  a.N = n; a.C = L.d.c_in; a.H = L.h_in; a.W = L.w_in; a.Ho = L.h_out; a.Wo = L.w_out;
  a.O = L.d.c_out; a.Cop = L.cp_out; a.pad = L.d.pad; a.act = L.d.act;
  const int mb = L.d.c_out <= 32 ? 2 : 4;
  a.tiles_y = (a.Ho + 7) / 8; a.tiles_x = (a.Wo + 15) / 16; a.tiles_m = (a.O + mb * 16 - 1) / (mb * 16);
  a.vec_out = (a.Cop % 4) == 0 ? 1 : 0;
  a.magic_x = strip_magic(a.tiles_x); a.magic_y = strip_magic(a.tiles_y);
  const long ptiles = (long)n * a.tiles_y * a.tiles_x;
  // as many workers as stay resident: LDS per work-group = weight tile + patch + offset table
  const int es = (int)dtype_size(net->dtype), kp = stem_packed_k(L.d.k, net->dtype);
  const int ph = 7 * L.d.stride + L.d.k, pwp = (15 * L.d.stride + L.d.k + 3) / 4 * 4;
  const long lds = (long)mb * 16 * (kp * es + 16) + 3L * ph * pwp * es + kp * 4;
  long per_cu = (160 * 1024) / lds;
  per_cu = per_cu > 8 ? 8 : (per_cu < 1 ? 1 : per_cu);
  // a small weight tile costs little to stage: then one pixel block per work-group keeps more of them in flight
  const bool light = (long)mb * 16 * (kp * es + 16) < 8192;
  const long workers = (light || ptiles < 256 * per_cu) ? ptiles : 256 * per_cu;
  dim3 grid((unsigned)workers, (unsigned)a.tiles_m);
  int rc;
  if (net->dtype == CPRUNE_F32) rc = launch_conv_stem_f32(L.d.k, L.d.stride, mb, grid, s, a);
  else if (net->dtype == CPRUNE_F16) rc = launch_conv_stem_f16(L.d.k, L.d.stride, mb, grid, s, a);
  else rc = launch_conv_stem_bf16(L.d.k, L.d.stride, mb, grid, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

constexpr int kStem7BlockFilters = 48;
static int stem7_block_tile(int c_out) { return c_out <= 32 ? 32 : 64; }

// Whether the 16-bit 7x7 / stride 2 first layer runs in 16 x 16 blocks of conv outputs rather than in strips.  Blocks take rounds of the work-groups that
// fit the chip (three per CU, two above 32 filters), whatever a round holds; strips take what their steps take.  Both times (us) as fitted to 20
// sizes each from 64x64 to 448x448, batch 2 to 256, in bf16; choosing so is at most 6 % over the better one there (16 filters without the pool, 24 and 32 images, where blocks would be the better), in most 0.  Blocks / strips, with the
// pool, 32 filters at 224x224: batch 3 5.8 / 5.6, 4 5.8 / 6.1, 8 6.9 / 8.1, 12 8.0 / 10.0, 16 13.1 / 11.9, 24 13.2 / 15.9, 64 34.7 / 31.0; 16 filters, batch 8 6.5 /
// 6.6, 12 7.4 / 7.9, 16 11.6 / 9.4; 48, batch 8 9.6 / 10.0, 12 15.8 / 12.6; without it, 16 filters, batch 12 6.1 / 7.4, 32 12.4 / 13.1; 32, batch 12 8.1 / 9.3,
// 32 19.6 / 17.3; 48, batch 8 8.6 / 9.3, 12 13.9 / 12.0.  64 filters, batch 8: 10.3 / 10.3 with the pool, 11.3 / 10.6 without.
static bool stem7_blocks(const StemArgs& a, bool pool) {
  if (a.Cop & 3) return true;                  // a last layer's dense map: strips store four filters at a time
  if (a.O > kStem7BlockFilters) return false;
  struct Times { double one, more, first, round, strips, step; };      // one group per CU, each further one; several rounds; strips: fixed, per 1000 steps
  constexpr double kNever = 1e9;
  static const Times times[2][3] = {
    {{4.92, 0.5, 0.0, kNever, 3.21, 0.95}, {5.85, 0.95, 0.0, kNever, 3.05, 1.32}, {7.1, 1.3, 0.0, kNever, 3.5, 1.75}},
    {{5.5, 0.9, 2.63, 4.42, 4.0, 0.69}, {5.75, 1.05, 2.07, 5.32, 4.12, 1.04}, {7.6, 1.9, 0.0, kNever, 4.9, 1.42}}};
  const Times& t = times[pool][(a.O - 1) / 16];
  const long h = pool ? a.Hp : a.Ho, w = pool ? a.Wp : a.Wo, side = pool ? 7 : 16;
  const long blocks = a.N * ((h + side - 1) / side) * ((w + side - 1) / side), steps = a.N * ((w + side - 1) / side) * (pool ? h : (h + 1) / 2);
  const long resident = 256 * (a.O <= 32 ? 3 : 2);
  const double in_blocks = blocks <= resident ? t.one + t.more * ((blocks + 255) / 256 - 1) : t.first + t.round * ((blocks + resident - 1) / resident);
  return in_blocks < t.strips + t.step * 1e-3 * steps;
}

static int net_run_stem7_blocks(const NetLayer& L, int dtype, int pool, StemArgs a, hipStream_t s) {
  const int tile = stem7_block_tile(a.O), side = pool ? 7 : 16;
  a.w = L.w_stem7b;
  a.tiles_m = (a.O + tile - 1) / tile;
  a.tiles_y = ((pool ? a.Hp : a.Ho) + side - 1) / side;
  a.tiles_x = ((pool ? a.Wp : a.Wo) + side - 1) / side;
  a.vec_out = (a.Cop % 4) == 0 ? 1 : 0;
  a.magic_x = strip_magic(a.tiles_x); a.magic_y = strip_magic(a.tiles_y);
  const long blocks = (long)a.N * a.tiles_y * a.tiles_x;
  // as many workers as stay resident: weight tile + patch (+ the conv block the pool reads)
  const long lds = tile * (kStem7K * 2L + 16) + 37L * 320 + (pool ? 256L * (tile * 2 + 16) : 16L), resident = 256 * (160 * 1024 / lds);
  const dim3 grid((unsigned)(blocks < resident ? blocks : resident), (unsigned)a.tiles_m);
  const int rc = dtype == CPRUNE_F16 ? launch_conv_stem7_block_f16(tile / 16, pool, grid, s, a) : launch_conv_stem7_block_bf16(tile / 16, pool, grid, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

// The 7x7 / stride 2 first-layer kernel on the caller's NCHW input, with or without the max-pool behind it.  A work-group walks over a band
// of rows and repeats the row above it for the pool; the bands are those for which the rounds of work-groups that fit the chip (two wavefronts each;
// two, in 16-bit data four, on a SIMD) take the fewest steps, a work-group's start and its repeated row counted as one step and a fifth.  64 filters at
// 224x224 in fp32 (us), as many bands as fit one round / this rule: batch 32 60 / 60, 33 76 / 69; one image 9.0 / 8.6.
static int net_run_stem7(cprune_net* net, int i, int n, const void* x, void* dst, hipStream_t s) {
  const NetLayer& L = net->layers[i];
  const bool f32 = net->dtype == CPRUNE_F32;
  const int pool = L.stem7 >= 2 ? L.stem7 - 1 : 0;
  const size_t es = dtype_size(net->dtype);
  StemArgs a;
  a.x = x; a.w = L.w_stem7; a.bias = L.b; a.y = dst;
  a.N = n; a.C = L.d.c_in; a.H = L.h_in; a.W = L.w_in; a.Ho = L.h_out; a.Wo = L.w_out;
  a.O = L.d.c_out; a.Cop = L.cp_out; a.pad = L.d.pad; a.act = L.d.act;
  if (pool) {
    const NetLayer& P = net->layers[L.pool3];
    a.y = P.act; a.Hp = P.h_out; a.Wp = P.w_out; a.Cop = P.cp_out;
    if (pool == 2) a.y_map = dst;
  }
  if (!f32 && stem7_blocks(a, pool)) return net_run_stem7_blocks(L, net->dtype, pool, a, s);
  const int mb = a.O <= 32 ? 1 : 2;
  a.tiles_m = (a.O + 32 * mb - 1) / (32 * mb);
  a.tiles_x = pool ? (a.Wp + 6) / 7 : (a.Wo + 15) / 16;
  const long strips = (long)n * a.tiles_x * a.tiles_m, steps = pool ? a.Hp : (a.Ho + 1) / 2, resident = f32 ? 1024 : mb == 1 ? 2560 : 2048;
  double best = 0.0;
  // (each length of a band once, with the fewest bands of it: 14 of the 56 numbers of bands at 224x224)
  for (long bands = 1; bands <= steps;) {
    const long band = (steps + bands - 1) / bands;
    const double cost = ((strips * bands + resident - 1) / resident) * (band + 1.2);
    if (bands == 1 || cost < best) { best = cost; a.band = (int)band; }
    bands = band > 1 ? (steps + band - 2) / (band - 1) : steps + 1;
  }
  a.tiles_y = (int)((steps + a.band - 1) / a.band);
  a.magic_x = strip_magic(a.tiles_x); a.magic_y = strip_magic(a.tiles_y);
  a.w_raw = L.w;
  a.x_bytes = (unsigned)((size_t)n * a.C * a.H * a.W * es);
  a.w_bytes = (unsigned)stem7_packed_bytes(a.O, net->dtype);
  a.w_raw_bytes = (unsigned)((size_t)a.O * a.C * 49 * es);
  const dim3 grid((unsigned)((long)n * a.tiles_y * a.tiles_x), (unsigned)a.tiles_m);
  const int rc = f32 ? launch_conv_stem7_f32(mb, pool, grid, s, a) :
                 net->dtype == CPRUNE_F16 ? launch_conv_stem7_f16(mb, pool, grid, s, a) : launch_conv_stem7_bf16(mb, pool, grid, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

// First layer L.fuse_stem and the 3x3 layer i in one kernel: reads the caller's NCHW image.
static int net_run_stem2(cprune_net* net, int i, int n, const void* x, void* dst, hipStream_t s) {
  const NetLayer& L = net->layers[i];
  const NetLayer& F = net->layers[L.fuse_stem];
  const cprune_conv_desc d2 = layer_conv_desc(*net, L, n);
  return launch_conv_stem2(d2, layer_layout(L), x, F.d.c_in, F.w_stem, F.b, F.d.c_out, F.d.act, L.w, L.b, dst, s);
}

// Whether the strips of depthwise layer D and the 1x1 layer P multiply on three bf16 parts, in every form.
static bool block_parts(int dtype, const NetLayer& D, const NetLayer& P) {
  int mb = 0, xh = 0;
  return dtype == CPRUNE_F32 && mbrow_form(dtype, P.d.c_out, 0, &mb, &xh) && mbrow_parts(D.d.k, mb);
}

// Rows of a strip.
static int block_rows(int dtype, const NetLayer& D, const NetLayer& P, int mb, int xh, int low) {
  return block_parts(dtype, D, P) ? mbrow3_strip_rows(D.d.stride, mb, xh, low) : mbrow_rows(D.d.k, D.d.stride, mb, low);
}

// Strips of r rows of a map in the inverted-residual kernel.
static void mbrow_tiles(const NetLayer& D, int r, MbArgs* a) {
  const int hl = mbrow_halo_left(D.d.k, D.d.stride), hr = mbrow_halo_right(D.d.k, D.d.stride), step = 16 - hl - hr;
  // two images side by side where an image with the columns its windows reach past the right edge fits eight lanes
  const int last = D.d.stride == 1 ? D.w_in + hr : D.w_out + 1;
  a->ipt = last <= 8 ? 2 : 1;
  a->tiles_x = a->ipt == 2 || D.w_out <= 16 ? 1 : (D.w_out - hl - hr + step - 1) / step;
  a->tiles_y = (D.h_out + r - 1) / r;
}

// Wavefronts that share a strip at n images, where none were timed: doubled from `ks` while the strips leave most of the chip idle
// (1024 SIMDs) and every wavefront still has a chunk.  Timed with 1 / 2 / 4 / 8: MobileNetV2 at batch 64, 32 -> 92 -> 32 at 28x28, 896
// strips 18.8 / 17.6 / 21.0 / 35.3 us; 64 -> 330 -> 64 at 14x14, 256 strips 43 / 43 / 26.8 / 26.2.
static int mbrow_auto_ks(const MbArgs& a, int n, int tiles_m, int ks) {
  const long strips = (long)((n + a.ipt - 1) / a.ipt) * a.tiles_y * a.tiles_x * tiles_m;
  while (ks < 8 && strips * ks < 1024 && 2 * ks <= a.nchunk) ks *= 2;
  return ks;
}

// Depthwise layer P.fuse_dw and the 1x1 layer i in one kernel, reading the depthwise layer's input; with the expansion
// P.fuse_block in it as well, reading the expansion's input.
static bool mbrow_form_of(const cprune_net& net, const NetLayer& P, const NetLayer* E, int* mb, int* xh) {
  if (E && E->nchw_in) return mbrow_image_form(net.dtype, P.d.c_out, mb, xh);
  return mbrow_form(net.dtype, P.d.c_out, E ? E->cp_in : 0, mb, xh);
}

// Three parts: rounds of the expansion's reduction in three parts (four window rows a round on the image)
static int expand_rounds(const NetLayer& E, int xh) { return E.nchw_in ? 3 : (xh + 1) / 2; }

static int net_run_mbrow(cprune_net* net, int i, int n, const void* x, void* dst, hipStream_t s) {
  const NetLayer& P = net->layers[i];
  const NetLayer& D = net->layers[P.fuse_dw];
  const NetLayer* E = P.fuse_block >= 0 ? &net->layers[P.fuse_block] : nullptr;
  const size_t es = dtype_size(net->dtype);
  int mb = 0, xh = 0;
  if (!mbrow_form_of(*net, P, E, &mb, &xh)) return CPRUNE_ERR_UNSUPPORTED;
  const bool image = E && E->nchw_in;
  MbArgs a;
  a.x = image ? x : net->layers[E ? E->d.input : D.d.input].act;
  a.Hi = image ? E->h_in : 0; a.Wi = image ? E->w_in : 0;
  a.we = E ? E->w_expand : nullptr; a.be = E ? E->b : nullptr;
  a.wdw = D.w; a.wdw32 = D.w_dw32; a.bdw = D.b; a.wp = P.w_proj; a.bp = P.b;
  a.res = P.d.residual >= 0 ? net->layers[P.d.residual].act : nullptr;
  a.y = dst;
  a.N = n; a.H = D.h_in; a.W = D.w_in; a.Ho = D.h_out; a.Wo = D.w_out;
  a.Cpi = image ? E->d.c_in : E ? E->cp_in : 0; a.Ce = D.d.c_out; a.Cpe = D.cp_in; a.O = P.d.c_out; a.Cop = P.cp_out;
  a.act_e = E ? E->d.act : CPRUNE_ACT_NONE; a.act_dw = D.d.act; a.act_out = P.d.act;
  const int low = E ? P.block_low : P.dw_tile != kTallStrips;
  mbrow_tiles(D, block_rows(net->dtype, D, P, mb, xh, low), &a);
  a.magic_x = strip_magic(a.tiles_x); a.magic_y = strip_magic(a.tiles_y);
  a.x_bytes = (unsigned)((size_t)n * (image ? (size_t)a.Hi * a.Wi : (size_t)a.H * a.W) * (E ? a.Cpi : a.Cpe) * es);
  const bool parts = block_parts(net->dtype, D, P);
  a.nchunk = (int)((a.Cpe * es + 63) / 64);
  a.we_raw = E ? E->w : nullptr; a.wp_raw = P.w;
  a.we_bytes = !E ? 0u : (unsigned)(parts ? parts_packed_bytes(a.Ce, expand_rounds(*E, xh), mbrow3_twice(D.d.stride, xh, image)) : expand_packed_bytes(a.Ce, xh, net->dtype));
  a.wp_bytes = (unsigned)(parts ? parts_packed_bytes(a.O, a.nchunk, false) : rows_packed_bytes(a.O, a.Cpe, net->dtype));
  a.wdw_bytes = (unsigned)((size_t)D.d.k * D.d.k * a.Cpe * es);
  a.y_bytes = (unsigned)((size_t)n * a.Ho * a.Wo * a.Cop * es);
  a.slots = 0;
  const int tiles_m = (a.O + mb * 16 - 1) / (mb * 16);
  const dim3 grid((unsigned)((n + a.ipt - 1) / a.ipt * a.tiles_y * a.tiles_x), (unsigned)tiles_m);
  int ks = E ? P.block_ks : P.dw_tile == kPixelBlocks ? 0 : P.dw_ks;     // the timed choice holds at the full batch
  if (!ks || n < net->max_batch) ks = mbrow_auto_ks(a, n, tiles_m, ks ? ks : 1);
  int rc;
  if (net->dtype == CPRUNE_F32) rc = launch_mbrow_f32(D.d.k, D.d.stride, mb, xh, low, grid, ks, s, a);
  else if (net->dtype == CPRUNE_F16) rc = launch_mbrow_f16(D.d.k, D.d.stride, mb, xh, low, grid, ks, s, a);
  else rc = launch_mbrow_bf16(D.d.k, D.d.stride, mb, xh, low, grid, ks, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

// Likewise without an expansion and on pixel blocks.
static DwProjArgs dwproj_tiles(const NetLayer& P, const NetLayer& D, int* mb) {
  DwProjArgs a;
  *mb = P.d.c_out <= 32 ? 2 : (P.d.c_out <= 64 ? 4 : 8);
  a.tiles_y = (D.h_out + 7) / 8; a.tiles_x = (D.w_out + 7) / 8; a.tiles_m = (P.d.c_out + *mb * 16 - 1) / (*mb * 16);
  return a;
}

static long dwproj_groups(const NetLayer& P, const NetLayer& D, int n) {
  int mb = 0;
  const DwProjArgs a = dwproj_tiles(P, D, &mb);
  return (long)n * a.tiles_y * a.tiles_x * a.tiles_m;
}

// What an untimed 5x5 half runs on: pixel blocks in 16-bit data and at stride 2 (fp32: onto maps of at least 28 columns), from 512
// work-groups up.  Time of pixel blocks / strips there: f16 0.53-0.82, bf16 0.46-0.93 from 1024 work-groups up, 0.7-1.05 from 512
// (f16 28x28 1.2-1.3); fp32 at stride 2 0.62-1.02, onto smaller maps 1.1-1.4; fp32 at stride 1 0.8-1.5; below 512 work-groups 1.0-1.6.
static int dw_tile_untimed(const NetLayer& P, const NetLayer& D, int max_batch, int dtype) {
  const bool blocks = D.d.k == 5 && (dtype != CPRUNE_F32 || (D.d.stride == 2 && D.w_out >= 28)) && dwproj_groups(P, D, max_batch) >= 512;
  return blocks ? kPixelBlocks : kLowStrips;
}

static int net_run_dwproj(cprune_net* net, int i, int n, void* dst, hipStream_t s) {
  const NetLayer& P = net->layers[i];
  const NetLayer& D = net->layers[P.fuse_dw];
  const size_t es = dtype_size(net->dtype);
  int mb = 0;
  DwProjArgs a = dwproj_tiles(P, D, &mb);
  a.x = net->layers[D.d.input].act;
  a.wdw = D.w; a.bdw = D.b; a.wp = P.w; a.bp = P.b;
  a.res = P.d.residual >= 0 ? net->layers[P.d.residual].act : nullptr;
  a.y = dst;
  a.N = n; a.H = D.h_in; a.W = D.w_in; a.Ho = D.h_out; a.Wo = D.w_out;
  a.Ce = D.d.c_out; a.Cpe = D.cp_in; a.O = P.d.c_out; a.Cop = P.cp_out;
  a.pad = D.d.pad; a.act_dw = D.d.act; a.act_out = P.d.act;
  a.x_bytes = (unsigned)((size_t)n * a.H * a.W * a.Cpe * es);
  a.wp_bytes = (unsigned)((size_t)a.O * a.Cpe * es);
  a.wdw_bytes = (unsigned)((size_t)D.d.k * D.d.k * a.Cpe * es);
  a.vec_out = (a.Cop % 4) == 0 ? 1 : 0;
  const dim3 grid((unsigned)(n * a.tiles_y * a.tiles_x * a.tiles_m));
  const int ks = P.dw_ks > 4 ? 2 : 1;
  int rc;
  if (net->dtype == CPRUNE_F32) rc = launch_dwproj_f32(D.d.k, D.d.stride, mb, ks, grid, s, a);
  else if (net->dtype == CPRUNE_F16) rc = launch_dwproj_f16(D.d.k, D.d.stride, mb, ks, grid, s, a);
  else rc = launch_dwproj_bf16(D.d.k, D.d.stride, mb, ks, grid, s, a);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

// Which blocks cprune_net_fuse_block may turn into one kernel at the caller's wish: up to 128 projection filters and layers
// whose weights, input patch (8 x 8 outputs with the halo) and chunk tiles stay within the 160 KiB of a compute unit.
// Blocks beyond that are one kernel only where cprune_net_create timed them so.
static bool block_on_request(const cprune_net& net, const NetLayer& E, const NetLayer& D, const NetLayer& P) {
  const size_t es = dtype_size(net.dtype);
  if (P.d.c_out > 128) return false;
  const size_t filters = P.d.c_out <= 32 ? 32 : P.d.c_out <= 64 ? 64 : 128;
  const size_t ph = 7 * D.d.stride + D.d.k, patch = (ph * ph + 31) / 32 * 32, kk = (size_t)D.d.k * D.d.k;
  const size_t in = (E.cp_in * es + 63) / 64 * 64, chunks = (D.cp_in * es + 63) / 64, cc = 64 / es;
  if (patch * in / 16 > 2560) return false;
  const size_t lds = patch * (in + 16) + 2 * (patch + 64) * 80 + chunks * (cc * (in + 16) + filters * 80 + kk * 64 + 2 * cc * 4);
  return lds <= 160 * 1024;
}

// The one layer that reads `layer`, as its input; -1: none or several.
static int only_reader(const cprune_net& net, int layer) {
  int reader = -1, readers = 0;
  for (int j = 0; j < (int)net.layers.size(); ++j) {
    if (net.layers[j].d.input == layer) { reader = j; ++readers; }
    if (net.layers[j].d.residual == layer) readers += 2;
  }
  return readers == 1 ? reader : -1;
}

// Whether the layer that depthwise layer i reads can join it and its 1x1 reader in one kernel: a 1x1 expansion, or the network's
// first layer (3x3 / stride 2 on the image), that nobody else reads; and the kernel's form for it.
static bool block_joins(const cprune_net& net, int i, int* mb, int* xh) {
  const NetLayer& D = net.layers[i];
  const NetLayer& E = net.layers[D.d.input];
  const NetLayer& P = net.layers[D.dw_reader];
  const cprune_layer_desc& ed = E.d;
  if (ed.kind != CPRUNE_LAYER_CONV || ed.groups != 1 || ed.residual >= 0 || E.fused_pool || E.cp_out != D.cp_in ||
      only_reader(net, D.d.input) != i)
    return false;
  if (E.nchw_in)
    return ed.c_in <= 3 && ed.k == 3 && ed.stride == 2 && ed.pad == 1 && !E.fused_away && E.stem_reader < 0 && D.d.k == 3 &&
           D.d.stride == 1 && D.w_in > 8 && mbrow_image_form(net.dtype, P.d.c_out, mb, xh);
  return ed.k == 1 && ed.stride == 1 && ed.pad == 0 && ed.input >= 0 && !E.map2x2 && E.fuse_dw < 0 &&
         E.cp_out == round_up_vec(ed.c_out, net.dtype) && mbrow_form(net.dtype, P.d.c_out, E.cp_in, mb, xh);
}

// Behind packed weights of three parts: the limit of the block's strips (with the expansion E, or none).
static int pack_parts_limit(const NetLayer* E, const NetLayer& D, const NetLayer& P, void* copy, size_t bytes, hipStream_t s) {
  PartsLimits p;
  p.we = E ? (const float*)E->w : nullptr; p.wd = (const float*)D.w; p.wp = (const float*)P.w;
  p.be = E ? E->b : nullptr; p.bd = D.b;
  p.ce = D.d.c_out; p.terms = !E ? 0 : E->nchw_in ? E->d.c_in * 9 : E->cp_in; p.cpe = P.cp_in; p.o = P.d.c_out;
  p.act_e = E ? E->d.act : CPRUNE_ACT_NONE; p.act_d = D.d.act;
  p.limit = (unsigned*)((unsigned char*)copy + bytes);
  return launch_parts_limit(p, s);
}

static int pack_expansion(cprune_net* net, NetLayer& E, const NetLayer& D, const NetLayer& P, int xh, hipStream_t s) {
  if (E.w_expand) return CPRUNE_OK;
  void* copy = nullptr;
  const int terms = E.nchw_in ? E.d.c_in * 9 : E.cp_in;
  const bool parts = block_parts(net->dtype, D, P), twice = mbrow3_twice(D.d.stride, xh, E.nchw_in);
  CPRUNE_HIP_TRY(hipMalloc(&copy, parts ? parts_packed_bytes(E.d.c_out, expand_rounds(E, xh), twice) + 16 : expand_packed_bytes(E.d.c_out, xh, net->dtype)));
  net->allocs.push_back(copy);
  E.w_expand = copy;
  if (parts) {
    const int rc = launch_pack_parts(E.w, E.d.c_out, terms, expand_rounds(E, xh), twice, E.nchw_in, copy, s);
    return rc == CPRUNE_OK ? pack_parts_limit(&E, D, P, copy, parts_packed_bytes(E.d.c_out, expand_rounds(E, xh), twice), s) : rc;
  }
  return launch_pack_expand(E.w, E.d.c_out, terms, xh, net->dtype, copy, s);
}

// The variant a layer of a handle for larger batches runs at n images, where none was timed for that shape.  Without a timed
// (or pinned) choice for the full batch: the estimate for n.  Otherwise the full batch's choice, which the timing of all
// kernels stands behind, unless n is at most 7/8 of the full batch, the choice has an estimate and another tile of the same
// kernel costs a tenth less by it: tiles chosen for many images leave most units idle at a few.  Graph replays in us, keeping
// the choice always / by this rule: ResNet-18 fp32, 2 of 32 images 368 / 224, 24 of 32 609 / 566, bf16 2 of 32 199 / 200; VGG-16 fp32, 1 of 64
// 157 / 136, 40 of 64 182 / 182, fp16 37 of 64 97 / 98; MobileNetV2 fp32, 4 of 64 444 / 401.  Estimating always, which knows two of
// the kernels only, gave 222 us for VGG-16 fp16, 37 of 64.
static int choose_at_batch(const cprune_net* net, const NetLayer& L, const cprune_conv_desc& d, const ConvLayout& lay) {
  if (!(L.timed && L.variant >= 0 && variant_supports(d, L.variant, lay) && conv_ws_bytes(d, L.variant, lay) <= net->ws_bytes))
    return heuristic_variant(d, lay, net->ws_bytes);
  const double kept = variant_cost(d, L.variant, lay);
  if (kept < 0.0 || 8 * d.n > 7 * net->max_batch) return L.variant;
  int best_v = -1;
  double best = 0.0;
  if (variant(L.variant).split) {
    best_v = best_split_variant(d, lay, &best);
  } else if (variant(L.variant).rows) {
    best_v = best_rows_variant(d, lay, &best);
  } else if (variant(L.variant).pw3) {
    best_v = best_pw3_variant(d, lay, &best);
  } else {
    for (int v = 0; v < num_variants(); ++v) {
      const TileVariant& tv = variant(v);
      if (!(tv.sched == 0 || tv.sched == 2 || tv.sched == 4) || !variant_supports(d, v, lay)) continue;
      const double cost = variant_cost(d, v, lay);
      if ((best_v < 0 || cost < best) && variant_ws_bytes(d, v, lay) <= net->ws_bytes) { best = cost; best_v = v; }
    }
  }
  return best_v >= 0 && best < 0.9 * kept ? best_v : L.variant;
}

static int layer_variant_at(const cprune_net* net, NetLayer& L, const cprune_conv_desc& d, const ConvLayout& lay, int n) {
  if (n == net->max_batch) return L.variant;
  const int timed = timed_variant(d, lay);
  if (timed >= 0 && variant_ws_bytes(d, timed, lay) <= net->ws_bytes) return timed;
  if (L.at_batch.empty()) L.at_batch.assign(net->max_batch, -1);
  if (L.at_batch[n] < 0) L.at_batch[n] = choose_at_batch(net, L, d, lay);
  return L.at_batch[n];
}

// The layout and the second layer of a pair (3x3 layer L and the 1x1 layer beside it).
static ConvPair pair_of(const cprune_net* net, const NetLayer& L) {
  const NetLayer& S = net->layers[L.pair_with];
  return ConvPair{S.w_rows3, S.w, S.b, S.act, S.d.c_out, S.cp_out, S.d.act};
}

static ConvLayout pair_layout(const NetLayer& L, const ConvPair* pair) {
  ConvLayout lay = layer_layout(L);
  lay.pair = pair;
  return lay;
}

static int net_run_pair(cprune_net* net, NetLayer& L, int n, const void* src, hipStream_t s) {
  const ConvPair pair = pair_of(net, L);
  const ConvLayout lay = pair_layout(L, &pair);
  const cprune_conv_desc d = layer_conv_desc(*net, L, n);
  int v = L.pair_variant;
  if (8 * n <= 7 * net->max_batch) {       // as choose_at_batch
    if (L.pair_at.empty()) L.pair_at.assign(net->max_batch, -1);
    if (L.pair_at[n] < 0) {
      double cost = 0.0;
      const int best = best_rows_variant(d, lay, &cost);
      L.pair_at[n] = best >= 0 && cost < 0.9 * variant_cost(d, v, lay) ? best : v;
    }
    v = L.pair_at[n];
  }
  const void* res = L.d.residual >= 0 ? net->layers[L.d.residual].act : nullptr;
  return launch_conv_dense(d, src, L.w, L.b, res, L.act, v, net->ws, s, lay);
}

static int net_run_layer(cprune_net* net, int i, int n, const void* x, void* out_override, hipStream_t s) {
  NetLayer& L = net->layers[i];
  const void* src = L.d.input < 0 ? (L.nchw_in ? x : net->x_cl) : net->layers[L.d.input].act;
  void* dst = out_override ? out_override : L.act;
  if (L.fused_away || L.pair_by >= 0) return CPRUNE_OK;
  if (L.pair >= 0) return net_run_pair(net, L, n, src, s);
  if (L.fuse_dw >= 0) {
    // (a smaller batch of few pixel blocks runs on strips, which more wavefronts can share)
    const bool blocks = L.fuse_block < 0 && L.dw_tile == kPixelBlocks &&
                        (n == net->max_batch || dwproj_groups(L, net->layers[L.fuse_dw], n) >= 256);
    return blocks ? net_run_dwproj(net, i, n, dst, s) : net_run_mbrow(net, i, n, x, dst, s);
  }
  if (L.fuse_stem >= 0) return net_run_stem2(net, i, n, x, dst, s);
  if (L.stem7) return net_run_stem7(net, i, n, src, dst, s);
  if (L.stem) return net_run_stem(net, i, n, src, dst, s);
  switch (L.d.kind) {
    case CPRUNE_LAYER_CONV:
    case CPRUNE_LAYER_FC: {
      cprune_conv_desc d = layer_conv_desc(*net, L, n);
      const ConvLayout lay = layer_layout(L);
      const void* res = L.d.residual >= 0 ? net->layers[L.d.residual].act : nullptr;
      int v = -1;
      if (d.groups == 1) v = layer_variant_at(net, L, d, lay, n);
      return conv_dispatch(d, src, L.w, L.b, res, dst, v, net->ws, net->ws_bytes, s, lay);
    }
    case CPRUNE_LAYER_MAXPOOL:
      if (L.alias || L.in_producer) return CPRUNE_OK;
      return launch_maxpool_nhwc(src, n, L.cp_in, L.h_in, L.w_in, L.d.k, L.d.stride, L.d.pad, net->dtype, dst, s);
    case CPRUNE_LAYER_GAVGPOOL:
      return launch_gavgpool_nhwc(src, n, L.cp_in, L.h_in * L.w_in, net->dtype, dst, s);
  }
  return CPRUNE_ERR_INVALID_ARG;
}

// Device time of running the given layers one after the other, as they are configured right now:
// the faster of two timed passes of six repetitions each, after one untimed pass.  What the
// create-time choices between two forms of the same layers are decided by.
static int time_layers(cprune_net* net, const int* layers, int n_layers, int batch, const void* x, hipStream_t s,
                       float* ms_out) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  CPRUNE_HIP_TRY(hipEventCreate(&e0));
  hipError_t e = hipEventCreate(&e1);
  if (e != hipSuccess) { hipEventDestroy(e0); set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
  int rc = CPRUNE_OK;
  float best = 0.f;
  for (int pass = 0; pass < 3 && rc == CPRUNE_OK && e == hipSuccess; ++pass) {
    e = hipEventRecord(e0, s);
    for (int it = 0; it < 6 && rc == CPRUNE_OK; ++it)
      for (int k = 0; k < n_layers && rc == CPRUNE_OK; ++k) rc = net_run_layer(net, layers[k], batch, x, nullptr, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float t = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
    if (pass == 1 || (pass == 2 && t < best)) best = t;
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  if (rc != CPRUNE_OK) return rc;
  if (e != hipSuccess) { set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
  *ms_out = best;
  return CPRUNE_OK;
}

// Times the given layers, the last of which runs as one kernel with those before it: with tall and low strips and with the
// wavefronts per strip that the rule for untimed layers names, or twice as many (strips = false: not); 5x5 halves of 256 work-groups and more
// on pixel blocks as well.  Leaves the fastest in *low (DwTile) and *ks, its time in *best (infinite, and both untouched: none timed).
static int time_mbrow(cprune_net* net, const int* layers, int n_layers, bool strips, int* low, int* ks, float* best, hipStream_t s) {
  const NetLayer& P = net->layers[layers[n_layers - 1]];
  const NetLayer& D = net->layers[P.fuse_dw];
  int mb = 0, xh = 0, best_low = *low, best_ks = *ks;
  *best = __builtin_inff();
  auto take = [&](int tile, int k) -> int {
    float ms = 0.f;
    *low = tile; *ks = k;
    const int rc = time_layers(net, layers, n_layers, net->max_batch, net->x_cl, s, &ms);
    if (rc == CPRUNE_OK && ms < *best) { *best = ms; best_ks = k; best_low = tile; }
    return rc;
  };
  mbrow_form_of(*net, P, P.fuse_block >= 0 ? &net->layers[P.fuse_block] : nullptr, &mb, &xh);
  for (int l = 0; l < 2 && strips; ++l) {
    if (l && block_rows(net->dtype, D, P, mb, xh, 0) == block_rows(net->dtype, D, P, mb, xh, 1)) break;
    MbArgs a;
    mbrow_tiles(D, block_rows(net->dtype, D, P, mb, xh, l), &a);
    a.nchunk = (int)((D.cp_in * dtype_size(net->dtype) + 63) / 64);
    const int k0 = mbrow_auto_ks(a, net->max_batch, (P.d.c_out + mb * 16 - 1) / (mb * 16), 1);
    for (int k = k0; k <= 8 && k <= 2 * k0; k *= 2) {
      const int rc = take(l, k);
      if (rc != CPRUNE_OK) return rc;
    }
  }
  const long groups = dwproj_groups(P, D, net->max_batch);
  if (P.fuse_block < 0 && D.d.k == 5 && groups >= 256) {
    const int rc = take(kPixelBlocks, groups <= 320 ? 8 : 4);
    if (rc != CPRUNE_OK) return rc;
  }
  *low = best_low; *ks = best_ks;
  return CPRUNE_OK;
}

static void set_pair(cprune_net* net, NetLayer& L, bool on) {
  NetLayer& S = net->layers[L.pair_with];
  L.pair = on ? L.pair_with : -1;
  S.pair_by = on ? (int)(&L - net->layers.data()) : -1;
}

// The copies a pair reads are those of the row-strip and of the 1x1 kernel.
static int any_pw3() {
  int v = 0;
  while (!variant(v).pw3) ++v;
  return v;
}

static int pack_pair(cprune_net* net, NetLayer& L, int rows_variant, hipStream_t s) {
  const int rc = pack_for(net, L, rows_variant, s);
  return rc != CPRUNE_OK ? rc : pack_for(net, net->layers[L.pair_with], any_pw3(), s);
}

// Whether an untimed pair (3x3 layer d, 1x1 layer S) runs in one launch: up to 0.3 GFLOP in fp32, 0.6 in 16-bit data.  250 random pairs a
// type, the layers apart / in one launch, untimed choices both: below the line 1.43 times the time on average (0.91 at worst), 16-bit
// 1.50 (0.88); above it 0.92 (0.41: 256 -> 56 and 440 at 40x40, batch 6, 22.5 / 51 us), 16-bit 0.92 (0.49): there the 1x1 kernel by
// itself has the better tiles.  Which variant runs is the 3x3 layer's estimate; with the 1x1 layer's tiles counted in it the choice was no
// better (1.01 times the time of the best variant both ways, 16-bit 1.06 and 1.06-1.08).
static bool pair_pays(const cprune_conv_desc& d, const NetLayer& S) {
  const long ho = conv_out_dim(d.h, 3, 2, 1), wo = conv_out_dim(d.w, 3, 2, 1);
  return 2.0 * d.n * ho * wo * d.c_in * (9.0 * d.c_out + S.d.c_out) <= (d.dtype == CPRUNE_F32 ? 3e8 : 6e8);
}

// Layer i, if it is the 3x3 / stride 2 / pad 1 layer that halves a residual network's map, takes the 1x1 / stride 2 layer on the same input
// into its launch.
static int make_pair(cprune_net* net, int i, bool tune, hipStream_t s) {
  NetLayer& L = net->layers[i];
  const int nl = (int)net->layers.size();
  if (!(strips_layer(*net, L) && L.d.stride == 2 && L.d.input >= 0 && i != nl - 1 && L.cp_out == round_up_vec(L.d.c_out, net->dtype))) return CPRUNE_OK;
  if (L.fused_away || L.fuse_dw >= 0 || L.fuse_stem >= 0) return CPRUNE_OK;
  int with = -1;
  for (int j = 0; j < nl - 1 && with < 0; ++j) {
    const NetLayer& S = net->layers[j];
    if (S.d.kind != CPRUNE_LAYER_CONV || S.d.groups != 1 || S.d.input != L.d.input || S.d.k != 1 || S.d.stride != 2 || S.d.pad != 0) continue;
    if (S.d.residual >= 0 || S.fused_away || S.fuse_dw >= 0 || S.pair_by >= 0 || S.cp_out != round_up_vec(S.d.c_out, net->dtype)) continue;
    if (S.h_out != L.h_out || S.w_out != L.w_out || (net->dtype == CPRUNE_F32 && S.d.c_in < 16)) continue;      // (as the other kernels on parts)
    bool late = true;                                    // its readers come behind layer i, where it is computed
    for (int k = 0; k <= i; ++k) late &= net->layers[k].d.input != j && net->layers[k].d.residual != j;
    if (late) with = j;
  }
  if (with < 0) return CPRUNE_OK;
  NetLayer& S = net->layers[with];
  const bool f32 = net->dtype == CPRUNE_F32;
  const size_t b1 = split_packed_bytes(S.d.c_out, S.cp_in, 1, net->dtype, true);
  const size_t b3 = f32 ? split_packed_bytes(L.d.c_out, L.cp_in, 9, net->dtype, true) : wave_packed_bytes(L.d.c_out, L.cp_in, net->dtype);
  if (b1 >= ((size_t)1 << 31) || b3 >= ((size_t)1 << 31)) return CPRUNE_OK;
  L.pair_with = with;
  const cprune_conv_desc d = layer_conv_desc(*net, L, net->max_batch);
  std::array<int, 21> key;
  {
    const DescKey k = key_of(d, layer_layout(L));
    std::copy(k.begin(), k.end(), key.begin());
    key[18] = S.d.c_out; key[19] = S.d.act; key[20] = S.cp_out;
  }
  int known = -2;
  if (tune) {
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    auto it = g_pairs.find(key);
    if (it != g_pairs.end()) known = it->second;
  }
  if (known == -1 || (!tune && !pair_pays(d, S))) return CPRUNE_OK;
  if (!tune && !(L.variant >= 0 && variant(L.variant).rows)) return CPRUNE_OK;
  int v3 = 0;
  while (!(variant(v3).rows == 1 && variant(v3).stride == 2)) ++v3;
  int rc = pack_pair(net, L, v3, s);
  if (rc != CPRUNE_OK) return rc;
  const ConvPair pair = pair_of(net, L);
  const ConvLayout lay = pair_layout(L, &pair);
  int best_v = known >= 0 ? known : -1;
  if (known < 0 && !tune) {
    double cost = 0.0;
    best_v = best_rows_variant(d, lay, &cost);
  } else if (known < 0) {
    const int apart[2] = {with, i};
    float best = 0.f;
    rc = time_layers(net, apart, 2, net->max_batch, net->x_cl, s, &best);
    std::vector<std::pair<float, int>> timed;
    auto time_pair = [&](int v, float* ms) -> int {
      L.pair_variant = v;
      set_pair(net, L, true);
      const int r = time_layers(net, &i, 1, net->max_batch, net->x_cl, s, ms);
      set_pair(net, L, false);
      return r;
    };
    for (int v = 0; v < num_variants() && rc == CPRUNE_OK; ++v) {
      if (!(variant(v).rows && variant(v).stride == 2) || !variant_supports(d, v, lay)) continue;
      timed.emplace_back(0.f, v);
      rc = time_pair(v, &timed.back().first);
    }
    std::sort(timed.begin(), timed.end());
    for (size_t k = 0; k < timed.size() && k < 3 && rc == CPRUNE_OK; ++k) {      // the fastest once more, and the layers apart between them
      float ms = 0.f, two = 0.f;
      rc = time_pair(timed[k].second, &ms);
      timed[k].first = std::min(timed[k].first, ms);
      if (rc == CPRUNE_OK) rc = time_layers(net, apart, 2, net->max_batch, net->x_cl, s, &two);
      if (rc == CPRUNE_OK) best = std::min(best, two);
    }
    for (const auto& t : timed)
      if (t.first < best) { best = t.first; best_v = t.second; }
    if (rc != CPRUNE_OK) return rc;
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    g_pairs[key] = best_v;
  }
  L.pair_variant = best_v;
  if (best_v >= 0) set_pair(net, L, true);
  CPRUNE_HIP_TRY(hipStreamSynchronize(s));      // (copies may still be on their way)
  drop_copies(net, L, best_v >= 0 ? best_v : L.variant);
  drop_copies(net, S, best_v >= 0 ? any_pw3() : S.variant);
  return CPRUNE_OK;
}

// The last layer writes straight into the caller's buffer when its map is 1x1 (its
// channel stride is then the dense channel count); otherwise its buffer is converted.
static int net_enqueue(cprune_net* net, const void* x, int n, void* logits, hipStream_t s) {
  const int nl = (int)net->layers.size();
  int rc = CPRUNE_OK;
  if (net->convert_input) rc = launch_nchw_to_nhwc(x, n, net->in_c, net->in_h * net->in_w, net->in_cp, net->dtype, net->x_cl, s);
  if (rc != CPRUNE_OK) return rc;
  const NetLayer& last = net->layers[nl - 1];
  const bool direct = last.h_out * last.w_out == 1;
  for (int i = 0; i < nl; ++i) {
    rc = net_run_layer(net, i, n, x, (i == nl - 1 && direct) ? logits : nullptr, s);
    if (rc != CPRUNE_OK) return rc;
  }
  if (!direct)
    rc = launch_nhwc_to_nchw(last.act, n, last.d.c_out, last.h_out * last.w_out, last.cp_out, net->dtype, logits, s);
  return rc;
}

extern "C" int cprune_net_create(const cprune_layer_desc* layers, int n_layers, int in_c, int in_h,
                                 int in_w, int max_batch, cprune_dtype dtype, int tune, void* stream,
                                 cprune_net** out) {
  if (!layers || !out || n_layers < 1 || in_c < 1 || in_h < 1 || in_w < 1 || max_batch < 1) return CPRUNE_ERR_INVALID_ARG;
  if (!dtype_ok(dtype)) return CPRUNE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  cprune_net* net = new cprune_net();
  net->in_c = in_c; net->in_h = in_h; net->in_w = in_w; net->max_batch = max_batch; net->dtype = dtype; net->tuned = tune != 0;
  net->in_cp = round_up_vec(in_c, dtype);
  net->layers.resize(n_layers);
  const size_t es = dtype_size(dtype);
  const long lim = 1L << 31;
  int rc = CPRUNE_OK;
  // shapes and validation
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    L.d = layers[i];
    const cprune_layer_desc& d = L.d;
    if (d.input < -1 || d.input >= i || d.residual < -1 || d.residual >= i) { rc = CPRUNE_ERR_INVALID_ARG; break; }
    int c, h, w;
    if (d.input < 0) { c = in_c; h = in_h; w = in_w; L.cp_in = net->in_cp; }
    else { const NetLayer& S = net->layers[d.input]; c = S.d.c_out; h = S.h_out; w = S.w_out; L.cp_in = S.cp_out; }
    L.h_in = h; L.w_in = w;
    if (d.kind == CPRUNE_LAYER_FC) {
      if (d.c_in != c || d.c_out < 1 || !d.weight || !act_ok(d.act) || d.residual >= 0) { rc = CPRUNE_ERR_INVALID_ARG; break; }
      if (h > 7 || w > 7) { rc = CPRUNE_ERR_UNSUPPORTED; break; }
      L.h_out = L.w_out = 1;
    } else if (d.kind == CPRUNE_LAYER_GAVGPOOL) {
      if (d.c_in != c || d.c_out != c) { rc = CPRUNE_ERR_INVALID_ARG; break; }
      L.h_out = L.w_out = 1;
    } else if (d.kind == CPRUNE_LAYER_MAXPOOL || d.kind == CPRUNE_LAYER_CONV) {
      if (d.c_in != c || d.k < 1 || d.stride < 1 || d.pad < 0 || h + 2 * d.pad < d.k || w + 2 * d.pad < d.k) { rc = CPRUNE_ERR_INVALID_ARG; break; }
      L.h_out = conv_out_dim(h, d.k, d.stride, d.pad);
      L.w_out = conv_out_dim(w, d.k, d.stride, d.pad);
      if (d.kind == CPRUNE_LAYER_MAXPOOL) {
        if (d.c_out != c || d.pad >= d.k) { rc = CPRUNE_ERR_INVALID_ARG; break; }
      } else if (!d.weight) { rc = CPRUNE_ERR_INVALID_ARG; break; }
    } else { rc = CPRUNE_ERR_INVALID_ARG; break; }
    if (d.kind == CPRUNE_LAYER_CONV || d.kind == CPRUNE_LAYER_FC) {
      cprune_conv_desc cd = layer_conv_desc(*net, L, max_batch);
      rc = validate_conv_desc(&cd);
      if (rc != CPRUNE_OK) break;
    }
    // pools keep their input's stride; a final 1x1 map is written dense for the caller
    const bool last_dense = (i == n_layers - 1) && L.h_out * L.w_out == 1;
    if (d.kind == CPRUNE_LAYER_MAXPOOL || d.kind == CPRUNE_LAYER_GAVGPOOL) L.cp_out = L.cp_in;
    else L.cp_out = last_dense ? d.c_out : round_up_vec(d.c_out, dtype);
    if (last_dense && L.cp_out != d.c_out) { rc = CPRUNE_ERR_UNSUPPORTED; break; }  // a pool cannot end a net densely
    if (d.residual >= 0) {
      const NetLayer& R = net->layers[d.residual];
      if (d.kind != CPRUNE_LAYER_CONV || R.d.c_out != d.c_out || R.h_out != L.h_out || R.w_out != L.w_out ||
          R.cp_out != L.cp_out) { rc = CPRUNE_ERR_INVALID_ARG; break; }
    }
    L.per_image = (size_t)L.cp_out * L.h_out * L.w_out;
    if ((long)L.per_image * max_batch * (long)es >= lim || (long)L.cp_in * h * w * max_batch * (long)es >= lim) { rc = CPRUNE_ERR_UNSUPPORTED; break; }
  }
  if (rc != CPRUNE_OK) { net_free(net); return rc; }

  // A 3x3 / stride 1 / pad 1 conv on a 2x2 map reads the whole input map for every output pixel:
  // it runs as one matrix product per image, 4/9 of the multiply-adds of the nine-tap form
  // (the other 5/9 would multiply padding).
  for (int i = 0; i < n_layers; ++i) {
    NetLayer& L = net->layers[i];
    const cprune_layer_desc& d = L.d;
    if (d.kind == CPRUNE_LAYER_CONV && d.groups == 1 && d.k == 3 && d.stride == 1 && d.pad == 1 &&
        L.h_in == 2 && L.w_in == 2 && L.cp_out == round_up_vec(d.c_out, dtype))
      L.map2x2 = true;
  }

  // A 2x2 / stride 2 max-pool whose only producer is a plain 3x3 stride-1 conv that nobody
  // else reads runs in that conv's epilogue: one launch and one round trip through HBM less.
  for (int i = 0; i < n_layers; ++i) {
    NetLayer& Pl = net->layers[i];
    const cprune_layer_desc& pd = Pl.d;
    if (pd.kind != CPRUNE_LAYER_MAXPOOL || pd.k != 2 || pd.stride != 2 || pd.pad != 0 || pd.input < 0) continue;
    NetLayer& Cv = net->layers[pd.input];
    const cprune_layer_desc& cd = Cv.d;
    if (cd.kind != CPRUNE_LAYER_CONV || cd.groups != 1 || cd.k != 3 || cd.stride != 1 || cd.pad != 1 || cd.residual >= 0) continue;
    if ((Cv.h_out & 1) || (Cv.w_out & 1) || i == n_layers - 1) continue;
    bool shared = false;
    for (int j = 0; j < n_layers; ++j)
      if (j != i && (net->layers[j].d.input == pd.input || net->layers[j].d.residual == pd.input)) shared = true;
    if (shared) continue;
    // only where some variant can run the layer with the pool in its epilogue (none can on e.g. a 2 x 18 map)
    Cv.fused_pool = true;
    const cprune_conv_desc fd = layer_conv_desc(*net, Cv, max_batch);
    const ConvLayout fl = layer_layout(Cv);
    bool runnable = false;
    for (int v = 0; v < num_variants() && !runnable; ++v) runnable = variant_supports(fd, v, fl);
    if (!runnable) { Cv.fused_pool = false; continue; }
    Cv.per_image = (size_t)Cv.cp_out * Pl.h_out * Pl.w_out;
    Pl.alias = true;
  }

  // A dense conv on the network input reads the caller's NCHW tensor directly (its few input
  // channels gain nothing from the channels-last vector loads) and writes channels-last.
  net->convert_input = false;
  for (int i = 0; i < n_layers; ++i) {
    NetLayer& L = net->layers[i];
    if (L.d.input >= 0) continue;
    if (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1 && L.d.c_in <= 4 && !L.fused_pool && !L.map2x2 &&
        L.d.residual < 0 && L.cp_out == round_up_vec(L.d.c_out, dtype))
      L.nchw_in = true;
    else
      net->convert_input = true;
  }

  auto dev_alloc = [&](size_t bytes, void** p) -> int {
    hipError_t e = hipMalloc(p, bytes ? bytes : 16);
    if (e != hipSuccess) { set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
    net->allocs.push_back(*p);
    return CPRUNE_OK;
  };
  // weights (repacked channels-last), biases, activations, scratch
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    const cprune_layer_desc& d = L.d;
    if (L.map2x2) {
      const int cpo = round_up_vec(d.c_out, dtype);
      const size_t nw = (size_t)16 * cpo * L.cp_in;
      if ((long)nw * (long)es >= lim) { rc = CPRUNE_ERR_UNSUPPORTED; break; }
      rc = dev_alloc(nw * es, &L.w);
      if (rc == CPRUNE_OK) rc = dev_alloc((size_t)4 * cpo * sizeof(float), (void**)&L.b);
      if (rc != CPRUNE_OK) break;
      rc = launch_repack_map2x2(d.weight, d.bias, d.c_out, d.c_in, L.cp_in, cpo, L.fused_pool ? 1 : 0, dtype, L.w, L.b, s);
      if (rc != CPRUNE_OK) break;
      cprune_conv_desc cd = layer_conv_desc(*net, L, max_batch);
      size_t need = conv_ws_bytes(cd, -1, layer_layout(L));
      if (need > net->ws_bytes) net->ws_bytes = need;
    } else if (L.nchw_in) {
      const size_t nw = (size_t)d.c_out * d.c_in * d.k * d.k;
      rc = dev_alloc(nw * es, &L.w);
      if (rc != CPRUNE_OK) break;
      hipError_t e = hipMemcpyAsync(L.w, d.weight, nw * es, hipMemcpyDeviceToDevice, s);
      if (e == hipSuccess && d.bias) {
        rc = dev_alloc((size_t)d.c_out * sizeof(float), (void**)&L.b);
        if (rc != CPRUNE_OK) break;
        e = hipMemcpyAsync(L.b, d.bias, (size_t)d.c_out * sizeof(float), hipMemcpyDeviceToDevice, s);
      }
      if (e != hipSuccess) { set_last_hip_error(e); rc = CPRUNE_ERR_DEVICE; break; }
      cprune_conv_desc cd = layer_conv_desc(*net, L, max_batch);
      size_t need = conv_ws_bytes(cd, -1, layer_layout(L));
      if (need > net->ws_bytes) net->ws_bytes = need;
    } else if (d.kind == CPRUNE_LAYER_CONV || d.kind == CPRUNE_LAYER_FC) {
      const int khw = d.kind == CPRUNE_LAYER_FC ? L.h_in * L.w_in : d.k * d.k;
      const bool dw = d.kind == CPRUNE_LAYER_CONV && d.groups != 1;
      const size_t nw = (size_t)(dw ? 1 : d.c_out) * khw * L.cp_in;
      if ((long)nw * (long)es >= lim) { rc = CPRUNE_ERR_UNSUPPORTED; break; }
      rc = dev_alloc(nw * es, &L.w);
      if (rc != CPRUNE_OK) break;
      rc = launch_repack_weights(d.weight, dw ? 1 : d.c_out, d.c_in, khw, L.cp_in, dtype, L.w, s);
      if (rc != CPRUNE_OK) break;
      if (d.bias) {
        rc = dev_alloc((size_t)d.c_out * sizeof(float), (void**)&L.b);
        if (rc != CPRUNE_OK) break;
        hipError_t e = hipMemcpyAsync(L.b, d.bias, (size_t)d.c_out * sizeof(float), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) { set_last_hip_error(e); rc = CPRUNE_ERR_DEVICE; break; }
      }
      if (!dw) {
        cprune_conv_desc cd = layer_conv_desc(*net, L, max_batch);
        size_t need = conv_ws_bytes(cd, -1, layer_layout(L));
        if (need > net->ws_bytes) net->ws_bytes = need;
      }
    }
    if (L.alias) { L.act = net->layers[d.input].act; continue; }
    const size_t abytes = L.per_image * max_batch * es;
    rc = dev_alloc(abytes, &L.act);
    if (rc != CPRUNE_OK) break;
    hipError_t e = hipMemsetAsync(L.act, 0, abytes, s);
    if (e != hipSuccess) { set_last_hip_error(e); rc = CPRUNE_ERR_DEVICE; break; }
  }
  if (rc == CPRUNE_OK && net->ws_bytes) rc = dev_alloc(net->ws_bytes, &net->ws);
  if (rc == CPRUNE_OK) {
    size_t ib = (size_t)max_batch * net->in_cp * in_h * in_w * es;
    rc = dev_alloc(ib, &net->x_cl);
    if (rc == CPRUNE_OK) {
      hipError_t e = hipMemsetAsync(net->x_cl, 0, ib, s);
      if (e != hipSuccess) { set_last_hip_error(e); rc = CPRUNE_ERR_DEVICE; }
    }
  }
  // 3x3 layers on small maps: a second copy of the weights in the operand order of the kernels made for them
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    if (!wave_layer(*net, L)) continue;
    rc = dev_alloc(wave_packed_bytes(L.d.c_out, L.cp_in, dtype), &L.w_wave);
    if (rc == CPRUNE_OK) rc = launch_repack_wave(L.w, L.d.c_out, L.cp_in, dtype, L.w_wave, s);
  }
  // layers the reduction-split kernel can run (1x1 / stride 1, fully connected, 2x2 maps as one matrix; few
  // pixels): likewise a copy in its operand order
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    if (!(L.d.kind == CPRUNE_LAYER_FC || (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1)) || L.nchw_in) continue;
    const cprune_conv_desc cd = layer_conv_desc(*net, L, max_batch);
    const ConvLayout lay = layer_layout(L);
    bool any = false;
    for (int v = 0; v < num_variants() && !any; ++v) any = variant(v).sched == -2 && variant_supports(cd, v, lay);
    if (!any) continue;
    const int k = lay.cp_in * cd.kh * cd.kw;
    if (rows_packed_bytes(cd.c_out, k, dtype) >= ((size_t)1 << 31)) continue;   // the kernel then reads the row layout
    rc = dev_alloc(rows_packed_bytes(cd.c_out, k, dtype), &L.w_rows);
    if (rc == CPRUNE_OK) rc = launch_repack_rows(L.w, cd.c_out, k, dtype, L.w_rows, s);
  }
  // variant per dense layer
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    if (!(L.d.kind == CPRUNE_LAYER_FC || (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1))) continue;
    cprune_conv_desc cd = layer_conv_desc(*net, L, max_batch);
    ConvLayout lay = layout_if_packed(*net, L);
    bool timed = false;
    int v = cached_or_heuristic_variant(cd, &timed, lay);
    for (int k = 0; k < num_variants() && rc == CPRUNE_OK; ++k)
      if (tune && !timed ? variant_supports(cd, k, lay) : k == v) rc = pack_for(net, L, k, s);
    if (rc != CPRUNE_OK) break;
    lay = layer_layout(L);
    if (tune && !timed) {
      const void* src = L.d.input < 0 ? net->x_cl : net->layers[L.d.input].act;
      const void* res = L.d.residual >= 0 ? net->layers[L.d.residual].act : nullptr;
      rc = select_tile_impl(cd, src, L.w, L.b, res, L.act, net->ws, net->ws_bytes, 2, 6, &v, nullptr, nullptr, s, lay);
    }
    L.variant = v;
    L.timed = timed || tune;
    if (rc == CPRUNE_OK) drop_copies(net, L, v);
  }
  // A first layer with an image-like input (<= 3 channels; 3x3 or 7x7 window) has a kernel of its
  // own that keeps the whole reduction in LDS; with tune != 0 it is timed against the chosen variant
  // of the general kernel, otherwise it is taken.
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    const cprune_layer_desc& d = L.d;
    if (!L.nchw_in || d.c_in > 3 || d.pad != d.k / 2) continue;
    if (!((d.k == 3 && (d.stride == 1 || d.stride == 2)) || (d.k == 7 && d.stride == 2))) continue;
    L.stem_ok = 1;
    {
      const int mb = d.c_out <= 32 ? 2 : 4;
      const int rows = (d.c_out + mb * 16 - 1) / (mb * 16) * (mb * 16);
      const int kp = stem_packed_k(d.k, dtype);
      rc = dev_alloc((size_t)rows * kp * es, &L.w_stem);
      if (rc == CPRUNE_OK) rc = launch_repack_stem(L.w, d.c_out, d.c_in * d.k * d.k, rows, kp, dtype, L.w_stem, s);
      if (rc != CPRUNE_OK) break;
    }
    bool use = true;
    if (tune && !(dtype == CPRUNE_F32 && stem7_layer(L, dtype))) {
      float ms[2] = {0.f, 0.f};
      for (int form = 0; form < 2 && rc == CPRUNE_OK; ++form) {   // 0: general kernel, 1: first-layer kernel
        L.stem = form == 1;
        rc = time_layers(net, &i, 1, max_batch, net->x_cl, s, &ms[form]);
      }
      use = ms[1] < ms[0];
    }
    L.stem = use;
    if (use) L.variant = -1;
  }

  // 7x7 / stride 2 / pad 3 on the image (the first layer of the ImageNet networks): a kernel whose
  // reduction order makes every MFMA operand one LDS read, and which can run the 3x3 / stride 2 / pad 1 max-pool
  // behind the layer as well when nobody else reads the conv map.  With tune != 0 the three forms (as decided so far;
  // that kernel; that kernel with the pool) are timed and the fastest kept; otherwise the most fused one is taken.  In fp32 nothing
  // is timed: a timed handle takes the kernel with the pool inside and the conv map stored as well, an untimed one the kernel alone; a
  // caller that can do without the conv map asks for form 2.  With the general kernels' fp32 instruction / kernel and pool apart / one
  // kernel and the conv map / one kernel (us): 64 filters at 224x224, 32 images 121 / 91 / 69 / 62, 1 15.6 / 9.5 / 9.5 / 8.6; 96, 8 images 56 /
  // 44 / 36 / 32; 64 at 16x16, 128 images 14.7 / 9.5 / 9.4 / 8.9; 31 sizes in all: one kernel and the map at most the time of the fp32
  // instruction (8.6 / 8.6 at worst) and, to 0.4 us, of the two apart, except 10 filters at 29x96, 33 images 7.7 / 8.6, and 92 at 22x255, 9 images 11.3 / 14.2.
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& L = net->layers[i];
    const cprune_layer_desc& d = L.d;
    if (!stem7_layer(L, dtype)) continue;
    rc = dev_alloc(stem7_packed_bytes(d.c_out, dtype), &L.w_stem7);
    if (rc == CPRUNE_OK) rc = launch_pack_stem7(L.w, d.c_out, d.c_in, dtype, L.w_stem7, s);
    if (rc == CPRUNE_OK && dtype != CPRUNE_F32 && (d.c_out <= kStem7BlockFilters || (L.cp_out & 3))) {
      const int rows = (d.c_out + stem7_block_tile(d.c_out) - 1) / stem7_block_tile(d.c_out) * stem7_block_tile(d.c_out);
      rc = dev_alloc((size_t)rows * kStem7K * es, &L.w_stem7b);
      if (rc == CPRUNE_OK) rc = launch_repack_stem7(L.w, d.c_out, d.c_in, rows, dtype, L.w_stem7b, s);
    }
    if (rc != CPRUNE_OK) break;
    int reader = -1, readers = 0;
    for (int j = 0; j < n_layers; ++j) {
      if (net->layers[j].d.input == i) { reader = j; ++readers; }
      if (net->layers[j].d.residual == i) readers += 2;
    }
    if (readers == 1 && reader != n_layers - 1) {
      const cprune_layer_desc& pd = net->layers[reader].d;
      if (pd.kind == CPRUNE_LAYER_MAXPOOL && pd.k == 3 && pd.stride == 2 && pd.pad == 1) L.pool3 = reader;
    }
    auto set_form = [&](int form) {
      L.stem7 = form;
      if (L.pool3 >= 0) net->layers[L.pool3].in_producer = form >= 2;
    };
    const int n_forms = L.pool3 >= 0 ? 3 : 2;
    int best = dtype != CPRUNE_F32 ? n_forms - 1 : tune && L.pool3 >= 0 ? 3 : 1;
    if (tune && dtype != CPRUNE_F32) {
      const int pair[2] = {i, L.pool3};
      float ms[3] = {0.f, 0.f, 0.f};
      for (int form = 0; form < n_forms && rc == CPRUNE_OK; ++form) {
        set_form(form);
        rc = time_layers(net, pair, L.pool3 >= 0 ? 2 : 1, max_batch, net->x_cl, s, &ms[form]);
      }
      best = 0;
      for (int form = 1; form < n_forms; ++form)
        if (ms[form] < ms[best]) best = form;
    }
    set_form(best);
    if (best) L.variant = -1;
  }

  // A first layer (3x3 / stride 1, at most 32 filters) whose only reader is another 3x3 / stride 1 conv can run
  // inside that conv's kernel: the largest activation of a VGG-style network is then never written.  With
  // tune != 0 both forms are timed and the faster kept; otherwise only cprune_net_fuse_first_layers turns it on.
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& F = net->layers[i];
    if (!(F.stem_ok && F.nchw_in && F.d.k == 3 && F.d.stride == 1 && F.d.pad == 1 && F.d.residual < 0 && !F.fused_pool)) continue;
    int reader = -1, readers = 0;
    for (int j = 0; j < n_layers; ++j) {
      if (net->layers[j].d.input == i) { reader = j; ++readers; }
      if (net->layers[j].d.residual == i) readers += 2;
    }
    if (readers != 1 || i == n_layers - 1) continue;
    NetLayer& L = net->layers[reader];
    if (!(L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1 && L.d.residual < 0 && !L.map2x2 && !L.nchw_in)) continue;
    if (!conv_stem2_supported(layer_conv_desc(*net, L, max_batch), layer_layout(L), F.d.c_in, F.d.c_out)) continue;
    F.stem_reader = reader;
    bool fuse = false;
    if (tune) {
      const int pair[2] = {i, reader};
      float ms[2] = {0.f, 0.f};
      for (int form = 0; form < 2 && rc == CPRUNE_OK; ++form) {   // 0: layers apart as decided so far, 1: one kernel
        F.fused_away = form == 1;
        L.fuse_stem = form == 1 ? i : -1;
        rc = time_layers(net, pair, 2, max_batch, net->x_cl, s, &ms[form]);
      }
      fuse = ms[1] < ms[0];
    }
    F.fused_away = fuse;
    L.fuse_stem = fuse ? i : -1;
    if (fuse) L.variant = -1;
  }

  // A depthwise conv whose only reader is a 1x1 conv can run inside that conv's kernel: the
  // expanded activations are then read once and never written.  When its input is a 1x1 expansion that nobody
  // else reads, the whole inverted-residual block can be one kernel, and they never reach memory at all.  With
  // tune != 0 the forms are timed and the fastest kept; otherwise a pair is fused on large maps (enough
  // 8x8 pixel blocks to fill the chip) and only cprune_net_fuse_block turns a whole block into one kernel.
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) {
    NetLayer& D = net->layers[i];
    const cprune_layer_desc& dd = D.d;
    if (!(dd.kind == CPRUNE_LAYER_CONV && dd.groups != 1 && dd.input >= 0 && dd.residual < 0)) continue;
    if (!((dd.k == 3 || dd.k == 5) && (dd.stride == 1 || dd.stride == 2) && dd.pad == dd.k / 2)) continue;
    const int reader = only_reader(*net, i);
    if (reader < 0 || i == n_layers - 1) continue;
    NetLayer& P = net->layers[reader];
    const cprune_layer_desc& pd = P.d;
    if (!(pd.kind == CPRUNE_LAYER_CONV && pd.groups == 1 && pd.k == 1 && pd.stride == 1 && pd.pad == 0)) continue;
    if (P.cp_out != round_up_vec(pd.c_out, dtype) || P.nchw_in || P.map2x2 || P.fused_pool) continue;
    D.dw_reader = reader;
    P.dw_tile = dw_tile_untimed(P, D, max_batch, dtype);
    if (dtype != CPRUNE_F32 && dd.k == 3) {
      const long count = (long)9 * D.cp_in;
      void* copy = nullptr;
      rc = dev_alloc((size_t)count * 4, &copy);
      D.w_dw32 = (float*)copy;
      if (rc == CPRUNE_OK) rc = launch_widen(D.w, count, dtype, D.w_dw32, s);
      if (rc != CPRUNE_OK) break;
    }
    if (block_parts(dtype, D, P)) {
      const int rounds = (P.cp_in + 15) / 16;
      rc = dev_alloc(parts_packed_bytes(pd.c_out, rounds, false) + 16, &P.w_proj);
      if (rc == CPRUNE_OK) rc = launch_pack_parts(P.w, pd.c_out, P.cp_in, rounds, false, false, P.w_proj, s);
      if (rc == CPRUNE_OK) rc = pack_parts_limit(nullptr, D, P, P.w_proj, parts_packed_bytes(pd.c_out, rounds, false), s);
      if (rc != CPRUNE_OK) break;
    } else if (P.w_rows) {
      P.w_proj = P.w_rows;
    } else {
      rc = dev_alloc(rows_packed_bytes(pd.c_out, P.cp_in, dtype), &P.w_proj);
      if (rc == CPRUNE_OK) rc = launch_repack_rows(P.w, pd.c_out, P.cp_in, dtype, P.w_proj, s);
      if (rc != CPRUNE_OK) break;
    }

    NetLayer& E = net->layers[dd.input];
    int mb = 0, xh = 0;
    bool block = block_joins(*net, i, &mb, &xh);
    const bool on_request = block && !E.nchw_in && block_on_request(*net, E, D, P);
    block = block && (on_request || tune);       // (the first layer in the expansion's place: only where timed as faster)
    if (block) {
      rc = pack_expansion(net, E, D, P, xh, s);
      if (rc != CPRUNE_OK) break;
      if (on_request) D.block_expand = dd.input;
    }

    auto set_form = [&](int form) {      // 0: three layers, 1: the depthwise layer inside the projection, 2: one kernel
      D.fused_away = form > 0;
      P.fuse_dw = form > 0 ? i : -1;
      if (block) E.fused_away = form == 2;
      P.fuse_block = form == 2 ? dd.input : -1;
    };
    const long groups = (long)max_batch * ((D.h_out + 7) / 8) * ((D.w_out + 7) / 8) * ((pd.c_out + 127) / 128);
    int form = groups >= 512 ? 1 : 0;
    if (tune) {
      const int layers_of[3] = {dd.input, i, reader};
      const int* timed = block ? layers_of : layers_of + 1;
      const int n_timed = block ? 3 : 2;
      float best = 0.f, ms = 0.f;
      bool ahead = false;
      set_form(0);
      rc = time_layers(net, timed, n_timed, max_batch, net->x_cl, s, &best);
      form = 0;
      if (rc == CPRUNE_OK && block) {
        set_form(2);
        rc = time_mbrow(net, timed, n_timed, true, &P.block_low, &P.block_ks, &ms, s);
        ahead = ms < 0.8f * best;      // (the depthwise half on strips is not timed then)
        if (ms < best) { form = 2; best = ms; }
      }
      if (rc == CPRUNE_OK) {
        set_form(1);
        rc = time_mbrow(net, timed, n_timed, !ahead, &P.dw_tile, &P.dw_ks, &ms, s);
        if (ms < best) form = 1;
      }
    }
    set_form(form);
    if (form) P.variant = -1;
    if (form == 2) E.variant = -1;
  }
  for (int i = 0; i < n_layers && rc == CPRUNE_OK; ++i) rc = make_pair(net, i, tune != 0, s);
  if (rc == CPRUNE_OK) {
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) { set_last_hip_error(e); rc = CPRUNE_ERR_DEVICE; }
  }
  if (rc != CPRUNE_OK) { net_free(net); return rc; }
  for (NetLayer& L : net->layers)
    if (L.variant < 0) drop_copies(net, L, -1);      // runs inside another kernel
  *out = net;
  return CPRUNE_OK;
}

extern "C" int cprune_net_forward(cprune_net* net, const void* x, int n, void* logits, int use_graph,
                                  void* stream) {
  if (!net || !x || !logits) return CPRUNE_ERR_INVALID_ARG;
  if (n < 1 || n > net->max_batch) return CPRUNE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  net->last_n = n;
  if (!use_graph) return net_enqueue(net, x, n, logits, s);
  GraphKey key{n, x, logits};
  auto it = net->graphs.find(key);
  if (it == net->graphs.end()) {
    if (!net->capture_stream) CPRUNE_HIP_TRY(hipStreamCreateWithFlags(&net->capture_stream, hipStreamNonBlocking));
    hipStream_t cs = net->capture_stream;
    hipGraph_t graph = nullptr;
    CPRUNE_HIP_TRY(hipStreamBeginCapture(cs, hipStreamCaptureModeRelaxed));
    int rc = net_enqueue(net, x, n, logits, cs);
    hipError_t e = hipStreamEndCapture(cs, &graph);
    if (rc != CPRUNE_OK) { if (graph) hipGraphDestroy(graph); return rc; }
    if (e != hipSuccess) { set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
    hipGraphExec_t exec = nullptr;
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    hipGraphDestroy(graph);
    if (e != hipSuccess) { set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
    if (net->graphs.size() >= kMaxGraphs) {
      // make room: the least recently replayed graph goes, once nothing can still be running it
      auto victim = net->graphs.begin();
      for (auto g = net->graphs.begin(); g != net->graphs.end(); ++g)
        if (g->second.last_use < victim->second.last_use) victim = g;
      hipError_t se = hipDeviceSynchronize();
      hipGraphExecDestroy(victim->second.exec);
      net->graphs.erase(victim);
      if (se != hipSuccess) { hipGraphExecDestroy(exec); set_last_hip_error(se); return CPRUNE_ERR_DEVICE; }
    }
    it = net->graphs.emplace(key, cprune_net::GraphEntry{exec, 0}).first;
  }
  it->second.last_use = ++net->graph_clock;
  CPRUNE_HIP_TRY(hipGraphLaunch(it->second.exec, s));
  return CPRUNE_OK;
}

extern "C" int cprune_net_layer_times(cprune_net* net, const void* x, int n, int iters, float* ms_out,
                                      void* stream) {
  if (!net || !x || !ms_out || iters < 1) return CPRUNE_ERR_INVALID_ARG;
  if (n < 1 || n > net->max_batch) return CPRUNE_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const int nl = (int)net->layers.size();
  hipEvent_t e0 = nullptr, e1 = nullptr;
  CPRUNE_HIP_TRY(hipEventCreate(&e0));
  hipError_t ec = hipEventCreate(&e1);
  if (ec != hipSuccess) { hipEventDestroy(e0); set_last_hip_error(ec); return CPRUNE_ERR_DEVICE; }
  net->last_n = n;
  int rc = CPRUNE_OK;
  if (net->convert_input) rc = launch_nchw_to_nhwc(x, n, net->in_c, net->in_h * net->in_w, net->in_cp, net->dtype, net->x_cl, s);
  // layer by layer, in order (so every layer finds its inputs): `iters` launches back to
  // back between two events, which is how the layer runs inside a forward pass
  for (int i = 0; i < nl && rc == CPRUNE_OK; ++i) {
    ms_out[i] = 0.0f;
    rc = net_run_layer(net, i, n, x, nullptr, s);   // untimed first run
    if (rc != CPRUNE_OK || net->layers[i].alias || net->layers[i].fused_away || net->layers[i].in_producer ||
        net->layers[i].pair_by >= 0) continue;
    hipError_t e = hipEventRecord(e0, s);
    for (int it = 0; it < iters && rc == CPRUNE_OK && e == hipSuccess; ++it) rc = net_run_layer(net, i, n, x, nullptr, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e != hipSuccess) { set_last_hip_error(e); rc = CPRUNE_ERR_DEVICE; break; }
    ms_out[i] = ms / (float)iters;
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  return rc;
}

extern "C" int cprune_net_copy_activation(cprune_net* net, int layer, int n, void* dst, size_t dst_bytes,
                                          void* stream) {
  if (!net || !dst || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  if (n < 1 || n > net->max_batch) return CPRUNE_ERR_INVALID_ARG;
  const NetLayer& L = net->layers[layer];
  if (L.fused_pool || L.stem7 == 2) return CPRUNE_ERR_UNSUPPORTED;  // only the pooled map exists: ask for the pool layer
  if (L.fused_away) return CPRUNE_ERR_UNSUPPORTED;  // computed inside its consumer's kernel, never stored
  const size_t bytes = (size_t)L.d.c_out * L.h_out * L.w_out * n * dtype_size(net->dtype);
  if (dst_bytes < bytes) return CPRUNE_ERR_INVALID_ARG;
  return launch_nhwc_to_nchw(L.act, n, L.d.c_out, L.h_out * L.w_out, L.cp_out, net->dtype, dst, (hipStream_t)stream);
}

extern "C" int cprune_net_output_shape(const cprune_net* net, int* c_out, int* h_out, int* w_out) {
  if (!net || !c_out || !h_out || !w_out) return CPRUNE_ERR_INVALID_ARG;
  const NetLayer& L = net->layers.back();
  *c_out = L.d.c_out; *h_out = L.h_out; *w_out = L.w_out;
  return CPRUNE_OK;
}

extern "C" int cprune_net_layer_variant(const cprune_net* net, int layer, int* variant_out) {
  if (!net || !variant_out || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  const NetLayer& L = net->layers[layer];
  *variant_out = L.pair_by >= 0 ? -1 : L.pair >= 0 ? L.pair_variant : L.variant;
  return CPRUNE_OK;
}

extern "C" int cprune_net_task_table(const cprune_net* net, int* task_of_layer, int* n_tasks_out) {
  if (!net || !task_of_layer || !n_tasks_out) return CPRUNE_ERR_INVALID_ARG;
  std::map<DescKey, int> ids;
  for (size_t i = 0; i < net->layers.size(); ++i) {
    const NetLayer& L = net->layers[i];
    if (!(L.d.kind == CPRUNE_LAYER_FC || (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1))) { task_of_layer[i] = -1; continue; }
    const DescKey key = key_of(layer_conv_desc(*net, L, net->max_batch), layer_layout(L));
    auto it = ids.find(key);
    if (it == ids.end()) it = ids.emplace(key, (int)ids.size()).first;
    task_of_layer[i] = it->second;
  }
  *n_tasks_out = (int)ids.size();
  return CPRUNE_OK;
}

extern "C" int cprune_net_task_key(const cprune_net* net, int layer, int32_t* key_out) {
  if (!net || !key_out || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  const NetLayer& L = net->layers[layer];
  if (!(L.d.kind == CPRUNE_LAYER_FC || (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1))) return CPRUNE_ERR_INVALID_ARG;
  const DescKey key = key_of(layer_conv_desc(*net, L, net->max_batch), layer_layout(L));
  static_assert(std::tuple_size<DescKey>::value == CPRUNE_TASK_KEY_INTS, "key length is part of the ABI");
  for (size_t i = 0; i < key.size(); ++i) key_out[i] = key[i];
  return CPRUNE_OK;
}

static int restore_variant(cprune_net* net, NetLayer& L) {
  if (L.variant >= 0 || L.stem || L.stem7) return CPRUNE_OK;
  const int v = cached_or_heuristic_variant(layer_conv_desc(*net, L, net->max_batch), &L.timed, layout_if_packed(*net, L));
  const int rc = pack_for(net, L, v, nullptr);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  L.variant = v;
  L.at_batch.clear();
  return CPRUNE_OK;
}

extern "C" int cprune_net_fuse_first_layers(cprune_net* net, int enable) {
  if (!net) return CPRUNE_ERR_INVALID_ARG;
  int first = -1;
  for (int i = 0; i < (int)net->layers.size(); ++i)
    if (net->layers[i].stem_reader >= 0) { first = i; break; }
  if (first < 0) return CPRUNE_ERR_UNSUPPORTED;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  drop_graphs(net);
  NetLayer& F = net->layers[first];
  NetLayer& L = net->layers[F.stem_reader];
  F.fused_away = enable != 0;
  L.fuse_stem = enable ? first : -1;
  if (enable) L.variant = -1;
  else return restore_variant(net, L);
  return CPRUNE_OK;
}

extern "C" int cprune_net_first_layer_form(cprune_net* net, int form) {
  if (!net || form < 0 || form > 2) return CPRUNE_ERR_INVALID_ARG;
  int first = -1;
  for (int i = 0; i < (int)net->layers.size(); ++i)
    if (net->layers[i].w_stem7) { first = i; break; }
  if (first < 0) return CPRUNE_ERR_UNSUPPORTED;
  NetLayer& L = net->layers[first];
  if (form == 2 && L.pool3 < 0) return CPRUNE_ERR_UNSUPPORTED;
  if (net->dtype == CPRUNE_F32 && (form == 1 || L.pool3 < 0)) return CPRUNE_ERR_UNSUPPORTED;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  drop_graphs(net);
  L.stem7 = form;
  if (L.pool3 >= 0) net->layers[L.pool3].in_producer = form == 2;
  if (form) L.variant = -1;
  else return restore_variant(net, L);
  return CPRUNE_OK;
}

extern "C" int cprune_net_fuse_depthwise(cprune_net* net, int layer, int enable) {
  if (!net || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  NetLayer& D = net->layers[layer];
  if (D.dw_reader < 0) return CPRUNE_ERR_UNSUPPORTED;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  drop_graphs(net);
  NetLayer& P = net->layers[D.dw_reader];
  if (enable && P.fused_away) {        // the reader is the expansion of a later block's kernel: out of there first
    for (NetLayer& Q : net->layers)
      if (Q.fuse_block == D.dw_reader) Q.fuse_block = -1;
    P.fused_away = false;
  }
  if (P.fuse_block >= 0) {             // leaves the one-kernel block form either way
    NetLayer& E = net->layers[P.fuse_block];
    E.fused_away = false;
    P.fuse_block = -1;
    const int rc = restore_variant(net, E);
    if (rc != CPRUNE_OK) return rc;
  }
  D.fused_away = enable != 0;
  P.fuse_dw = enable ? layer : -1;
  if (enable) P.variant = -1;
  else return restore_variant(net, P);
  return CPRUNE_OK;
}

extern "C" int cprune_net_fuse_block(cprune_net* net, int layer, int enable) {
  if (!net || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  NetLayer& D = net->layers[layer];
  if (D.dw_reader < 0) return CPRUNE_ERR_UNSUPPORTED;
  NetLayer& P = net->layers[D.dw_reader];
  if (D.block_expand < 0 && (enable || P.fuse_block < 0)) return CPRUNE_ERR_UNSUPPORTED;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  drop_graphs(net);
  NetLayer& E = net->layers[D.d.input];
  if (enable) {
    if (E.fuse_dw >= 0) {              // the expansion runs an earlier depthwise layer inside its own kernel: apart first
      if (E.fuse_block >= 0) return CPRUNE_ERR_UNSUPPORTED;
      net->layers[E.fuse_dw].fused_away = false;
      E.fuse_dw = -1;
    }
    E.fused_away = true; D.fused_away = true;
    P.fuse_dw = layer; P.fuse_block = D.d.input;
    P.variant = -1; E.variant = -1;
  } else if (P.fuse_block >= 0) {      // back to the depthwise + projection pair in one kernel, expansion on its own
    E.fused_away = false;
    P.fuse_block = -1;
    const int rc = restore_variant(net, E);
    if (rc != CPRUNE_OK) return rc;
  }
  return CPRUNE_OK;
}

extern "C" int cprune_net_block_form(cprune_net* net, int layer, int form, int tile, int wavefronts) {
  if (!net || layer < 0 || layer >= (int)net->layers.size() || form < 0 || form > 2 || tile < 0 || tile > 2) return CPRUNE_ERR_INVALID_ARG;
  if (wavefronts != 1 && wavefronts != 2 && wavefronts != 4 && wavefronts != 8) return CPRUNE_ERR_INVALID_ARG;
  NetLayer& D = net->layers[layer];
  if (D.dw_reader < 0) return CPRUNE_ERR_UNSUPPORTED;
  NetLayer& P = net->layers[D.dw_reader];
  NetLayer& E = net->layers[D.d.input];
  int mb = 0, xh = 0;
  if (P.fused_away) return CPRUNE_ERR_UNSUPPORTED;      // itself inside a later block's kernel
  if (form && tile == kPixelBlocks && (form != 1 || D.d.k != 5 || wavefronts < 4)) return CPRUNE_ERR_UNSUPPORTED;
  const bool joined = P.fuse_block >= 0;
  if (form == 2 && !joined && !block_joins(*net, layer, &mb, &xh)) return CPRUNE_ERR_UNSUPPORTED;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  drop_graphs(net);
  if (form == 2 && !joined) {
    const int rc = pack_expansion(net, E, D, P, xh, nullptr);
    if (rc != CPRUNE_OK) return rc;
    CPRUNE_HIP_TRY(hipDeviceSynchronize());
  }
  D.fused_away = form > 0;
  P.fuse_dw = form > 0 ? layer : -1;
  P.fuse_block = form == 2 ? D.d.input : -1;
  if (form == 1) { P.dw_tile = tile; P.dw_ks = wavefronts; }
  if (form == 2) { P.block_low = tile; P.block_ks = wavefronts; }
  if (form == 2 || joined) E.fused_away = form == 2;
  if (form == 2) E.variant = -1;
  else if (joined) {
    const int rc = restore_variant(net, E);
    if (rc != CPRUNE_OK) return rc;
  }
  if (form) P.variant = -1;
  else return restore_variant(net, P);
  return CPRUNE_OK;
}

extern "C" int cprune_net_layer_fused(const cprune_net* net, int layer, int* fused_out) {
  if (!net || !fused_out || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  *fused_out = net->layers[layer].fused_away || net->layers[layer].pair_by >= 0 ? 1 : 0;
  return CPRUNE_OK;
}

extern "C" int cprune_net_set_layer_variant(cprune_net* net, int layer, int variant) {
  if (!net || layer < 0 || layer >= (int)net->layers.size()) return CPRUNE_ERR_INVALID_ARG;
  NetLayer& L = net->layers[layer];
  if (!(L.d.kind == CPRUNE_LAYER_FC || (L.d.kind == CPRUNE_LAYER_CONV && L.d.groups == 1))) return CPRUNE_ERR_INVALID_ARG;
  if (L.fuse_dw >= 0 || L.fuse_stem >= 0 || L.fused_away) return CPRUNE_ERR_INVALID_ARG;   // runs inside a fused kernel: no variants
  if (L.pair >= 0 || (L.pair_with >= 0 && !net->tuned && !net->layers[L.pair_with].pinned && net->layers[L.pair_with].pair_by < 0)) {
    // a variant of the kernel that runs pairs keeps the pair; any other means a launch of its own.  In an untimed handle it also makes
    // the pair, unless the 1x1 layer has been given a variant of its own: how the choices of a timed handle are applied to another
    NetLayer& S = net->layers[L.pair_with];
    const ConvPair pair = pair_of(net, L);
    ConvLayout lay = pair_layout(L, &pair);
    lay.w_wave = lay.w_rows3 = L.w;                    // (only whether they are set matters here)
    if (variant >= 0 && variant < num_variants() && cprune::variant(variant).rows &&
        variant_supports(layer_conv_desc(*net, L, net->max_batch), variant, lay)) {
      const int rc = pack_pair(net, L, variant, nullptr);
      if (rc != CPRUNE_OK) return rc;
      CPRUNE_HIP_TRY(hipDeviceSynchronize());
      drop_graphs(net);
      set_pair(net, L, true);
      drop_copies(net, L, variant);
      drop_copies(net, S, any_pw3());
      L.pair_variant = L.variant = variant;      // (for this layer alone too, when the pair ends: the same copy)
      L.pair_at.clear();
      L.timed = true;
      L.at_batch.clear();
      return CPRUNE_OK;
    }
  }
  if (L.stem) L.stem = false;                          // a pinned variant means the general kernel
  if (L.stem7) {
    if (L.pool3 >= 0) net->layers[L.pool3].in_producer = false;
    L.stem7 = 0;
  }
  const cprune_conv_desc cd = layer_conv_desc(*net, L, net->max_batch);
  const ConvLayout lay = layout_if_packed(*net, L);
  if (!variant_supports(cd, variant, lay)) return CPRUNE_ERR_UNSUPPORTED;
  if (conv_ws_bytes(cd, variant, lay) > net->ws_bytes) return CPRUNE_ERR_WORKSPACE;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  drop_graphs(net);
  // (the other layer of a pair that ends here runs its own variant, whose copy the pair may not have read)
  NetLayer* const other = L.pair >= 0 ? &net->layers[L.pair] : L.pair_by >= 0 ? &net->layers[L.pair_by] : nullptr;
  int rc = pack_for(net, L, variant, nullptr);
  if (rc == CPRUNE_OK && other) rc = pack_for(net, *other, other->variant, nullptr);
  if (rc != CPRUNE_OK) return rc;
  CPRUNE_HIP_TRY(hipDeviceSynchronize());
  if (other) {
    set_pair(net, L.pair >= 0 ? L : *other, false);
    drop_copies(net, *other, other->variant);
  }
  drop_copies(net, L, variant);
  L.variant = variant;
  L.pinned = true;
  L.timed = true;
  L.at_batch.clear();
  return CPRUNE_OK;
}

extern "C" int cprune_net_destroy(cprune_net* net) {
  if (!net) return CPRUNE_ERR_INVALID_ARG;
  hipError_t e = hipDeviceSynchronize();
  net_free(net);
  if (e != hipSuccess) { set_last_hip_error(e); return CPRUNE_ERR_DEVICE; }
  return CPRUNE_OK;
}
