// Bandwidth-bound layers of the evaluated networks: depthwise convolution
// (MobileNetV2's 3x3 stage between the pruned 1x1 expansion and projection),
// max pooling and global average pooling.  No contraction across channels, so
// these are plain coalesced kernels: consecutive lanes take consecutive output
// columns of one (image, channel) plane.
#include "conv_split_kernel.hpp"
#include "parts_limit.hpp"

namespace cprune {
namespace {

template <typename T> __device__ __forceinline__ float ld(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void st(T* p, float v) { *p = (T)v; }

// an activation is a clamp with uniform bounds: a max and a min per element, no branches
__device__ __forceinline__ float act_f(float v, int act) {
  const float lo = act == CPRUNE_ACT_NONE ? -__builtin_inff() : 0.0f;
  const float hi = act == CPRUNE_ACT_RELU6 ? 6.0f : __builtin_inff();
  return fminf(fmaxf(v, lo), hi);
}

// grid.x = n*c planes, grid.y slices the output plane; weights of the plane's
// channel are read once into registers (k <= 7).
template <typename T, int K>
__global__ __launch_bounds__(256) void depthwise_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                        const float* __restrict__ bias,
                                                        const T* __restrict__ res, T* __restrict__ y,
                                                        int c, int h, int wd, int ho, int wo, int stride,
                                                        int pad, int act) {
  const int plane = blockIdx.x;
  const int ch = plane % c;
  float wk[K * K];
#pragma unroll
  for (int i = 0; i < K * K; ++i) wk[i] = ld(w + (long)ch * K * K + i);
  const float b = bias ? bias[ch] : 0.0f;
  const T* xp = x + (long)plane * h * wd;
  const long obase = (long)plane * ho * wo;
  const int total = ho * wo;
  for (int e = blockIdx.y * 256 + threadIdx.x; e < total; e += gridDim.y * 256) {
    int oy = e / wo, ox = e - oy * wo;
    int iy0 = oy * stride - pad, ix0 = ox * stride - pad;
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < K; ++u) {
      int iy = iy0 + u;
      if ((unsigned)iy >= (unsigned)h) continue;
#pragma unroll
      for (int v = 0; v < K; ++v) {
        int ix = ix0 + v;
        if ((unsigned)ix < (unsigned)wd) acc += ld(xp + (long)iy * wd + ix) * wk[u * K + v];
      }
    }
    acc += b;
    if (res) acc += ld(res + obase + e);
    st(y + obase + e, act_f(acc, act));
  }
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_kernel(const T* __restrict__ x, T* __restrict__ y, int h,
                                                      int wd, int ho, int wo, int k, int stride,
                                                      int pad) {
  const int plane = blockIdx.x;
  const T* xp = x + (long)plane * h * wd;
  const int total = ho * wo;
  for (int e = blockIdx.y * 256 + threadIdx.x; e < total; e += gridDim.y * 256) {
    int oy = e / wo, ox = e - oy * wo;
    int iy0 = oy * stride - pad, ix0 = ox * stride - pad;
    float m = 0.0f;
    bool have = false;
    for (int u = 0; u < k; ++u) {
      int iy = iy0 + u;
      if ((unsigned)iy >= (unsigned)h) continue;
      for (int v = 0; v < k; ++v) {
        int ix = ix0 + v;
        if ((unsigned)ix >= (unsigned)wd) continue;
        float val = ld(xp + (long)iy * wd + ix);
        if (!have || val > m) { m = val; have = true; }
      }
    }
    st(y + (long)plane * total + e, m);
  }
}

// One wavefront per (image, channel) plane: strided partial sums, then a
// shuffle tree; 4 planes per work-group.
template <typename T>
__global__ __launch_bounds__(256) void gavgpool_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                       int planes, int hw) {
  const int plane = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (plane >= planes) return;
  const int lane = threadIdx.x & 63;
  const T* xp = x + (long)plane * hw;
  float s = 0.0f;
  for (int i = lane; i < hw; i += 64) s += ld(xp + i);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) st(y + plane, s / (float)hw);
}

// ---- channels-last twins used inside the network handle ------------------------
// One thread per output element, consecutive threads on consecutive channels of a
// pixel (the contiguous direction of [n][h][w][cp]); pad channels carry zeros.

template <typename T>
__global__ __launch_bounds__(256) void maxpool_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                           long total, int cp, int h, int wd, int ho, int wo,
                                                           int k, int stride, int pad) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int c = (int)(i % cp);
  long pix = i / cp;
  const int ox = (int)(pix % wo); pix /= wo;
  const int oy = (int)(pix % ho);
  const long n = pix / ho;
  const int iy0 = oy * stride - pad, ix0 = ox * stride - pad;
  float m = 0.0f;
  bool have = false;
  for (int u = 0; u < k; ++u) {
    const int iy = iy0 + u;
    if ((unsigned)iy >= (unsigned)h) continue;
    for (int v = 0; v < k; ++v) {
      const int ix = ix0 + v;
      if ((unsigned)ix >= (unsigned)wd) continue;
      const float val = ld(x + ((n * h + iy) * wd + ix) * cp + c);
      if (!have || val > m) { m = val; have = true; }
    }
  }
  st(y + i, m);
}

template <typename T> struct VecOf;
template <> struct VecOf<float> { static constexpr int V = 4; };
template <> struct VecOf<_Float16> { static constexpr int V = 8; };
template <> struct VecOf<__bf16> { static constexpr int V = 8; };

template <typename T, int V>
__device__ __forceinline__ void unpack16(const uint4& q, float (&f)[V]) {
  if constexpr (V == 4) {
    f[0] = __uint_as_float(q.x); f[1] = __uint_as_float(q.y); f[2] = __uint_as_float(q.z); f[3] = __uint_as_float(q.w);
  } else {
    const T* h = reinterpret_cast<const T*>(&q);
#pragma unroll
    for (int i = 0; i < 8; ++i) f[i] = (float)h[i];
  }
}

// 16 channel vectors x 16 slices of the map per work-group; the slices' sums meet in LDS, in order.  (One thread per
// channel walked the whole map: 49 loads one behind the other, 6.3 us at 7x7 whatever the batch; now 2.8 us.)
template <typename T>
__global__ __launch_bounds__(256) void gavgpool_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y, int vblocks, int cp,
                                                            int hw) {
  constexpr int V = VecOf<T>::V;
  __shared__ float part[16][16][V + 1];
  const int n = blockIdx.x / vblocks, vb = blockIdx.x - n * vblocks;
  const int lane = threadIdx.x & 15, slice = threadIdx.x >> 4;
  const int c0 = (vb * 16 + lane) * V;
  float s[V];
#pragma unroll
  for (int e = 0; e < V; ++e) s[e] = 0.0f;
  if (c0 < cp) {
    const T* const xp = x + (size_t)n * hw * cp + c0;
#pragma unroll 4
    for (int p = slice; p < hw; p += 16) {
      float in[V];
      unpack16<T, V>(*reinterpret_cast<const uint4*>(xp + (size_t)p * cp), in);
#pragma unroll
      for (int e = 0; e < V; ++e) s[e] += in[e];
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) part[slice][lane][e] = s[e];
  __syncthreads();
  const int c = threadIdx.x / V, e = threadIdx.x % V;   // channel vb * 16 * V + threadIdx.x of the group
  if (threadIdx.x < 16 * V && vb * 16 * V + (int)threadIdx.x < cp) {
    float sum = part[0][c][e];
#pragma unroll
    for (int k = 1; k < 16; ++k) sum += part[k][c][e];
    st(y + (size_t)n * cp + vb * 16 * V + threadIdx.x, sum / (float)hw);
  }
}

template <typename T, int K>
__global__ __launch_bounds__(256) void depthwise_nhwc_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                             const float* __restrict__ bias,
                                                             const T* __restrict__ res, T* __restrict__ y,
                                                             long total, int c_real, int cp, int h, int wd,
                                                             int ho, int wo, int stride, int pad, int act) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int c = (int)(i % cp);
  long pix = i / cp;
  const int ox = (int)(pix % wo); pix /= wo;
  const int oy = (int)(pix % ho);
  const long n = pix / ho;
  const int iy0 = oy * stride - pad, ix0 = ox * stride - pad;
  float acc = 0.0f;
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int iy = iy0 + u;
    if ((unsigned)iy >= (unsigned)h) continue;
#pragma unroll
    for (int v = 0; v < K; ++v) {
      const int ix = ix0 + v;
      if ((unsigned)ix < (unsigned)wd)
        acc += ld(x + ((n * h + iy) * wd + ix) * cp + c) * ld(w + (u * K + v) * cp + c);
    }
  }
  if (bias && c < c_real) acc += bias[c];
  if (res) acc += ld(res + i);
  st(y + i, act_f(acc, act));
}

// Channels-last max-pool on 16-byte channel vectors (one output pixel and vector per thread).  A window position outside
// the image reads the nearest one inside, which is in the window too (pad < k): the K * K loads need no branches and are
// in flight together (K = 0: any other window).  3x3 / stride 2 on 64 channels at 112x112, batch 32, fp32 28.4 -> 26.9 us.
template <typename T, int K>
__global__ __launch_bounds__(256) void maxpool_nhwc_vec_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                               unsigned total, int cp, int h, int wd, int ho,
                                                               int wo, int k, int stride, int pad) {
  constexpr int V = VecOf<T>::V;
  const unsigned idx = blockIdx.x * 256u + threadIdx.x;
  if (idx >= total) return;
  const unsigned nvec = (unsigned)cp / V;
  const int c0 = (int)(idx % nvec) * V;
  unsigned r = idx / nvec;
  const int ox = (int)(r % (unsigned)wo); r /= (unsigned)wo;
  const int oy = (int)(r % (unsigned)ho);
  const int n = (int)(r / (unsigned)ho);
  auto at = [&](int u, int v) -> uint4 {
    const int iy = min(max(oy * stride - pad + u, 0), h - 1), ix = min(max(ox * stride - pad + v, 0), wd - 1);
    return *reinterpret_cast<const uint4*>(x + ((size_t)(n * h + iy) * wd + ix) * cp + c0);
  };
  float m[V];
  if constexpr (K > 0) {
    uint4 raw[K * K];
#pragma unroll
    for (int i = 0; i < K * K; ++i) raw[i] = at(i / K, i % K);
    unpack16<T, V>(raw[0], m);
#pragma unroll
    for (int i = 1; i < K * K; ++i) {
      float in[V];
      unpack16<T, V>(raw[i], in);
#pragma unroll
      for (int e = 0; e < V; ++e) m[e] = fmaxf(m[e], in[e]);
    }
  } else {
    unpack16<T, V>(at(0, 0), m);
    for (int u = 0; u < k; ++u)
      for (int v = 0; v < k; ++v) {
        float in[V];
        unpack16<T, V>(at(u, v), in);
#pragma unroll
        for (int e = 0; e < V; ++e) m[e] = fmaxf(m[e], in[e]);
      }
  }
  uint4 q;
  if constexpr (V == 4) {
    q.x = __float_as_uint(m[0]); q.y = __float_as_uint(m[1]); q.z = __float_as_uint(m[2]); q.w = __float_as_uint(m[3]);
  } else {
    T* hq = reinterpret_cast<T*>(&q);
#pragma unroll
    for (int e = 0; e < 8; ++e) hq[e] = (T)m[e];
  }
  *reinterpret_cast<uint4*>(y + (size_t)idx * V) = q;
}

// Channels-last depthwise, vectorised: a thread owns one vector of V channels of TX neighbouring output pixels of a row.
// Consecutive lanes take consecutive vectors, so every access is a coalesced 16-byte (5x5 on 16-bit data: 8-byte) load
// or store; each input column loaded serves every output of the run whose window covers it ((TX - 1) * S + K loads per
// row for TX outputs instead of TX * K), each window row's weights are read with it.  Every load is unconditional (outside the image it is
// out of the buffer's range and reads as zero, and so do the weights of a window row outside: a row that is not there
// adds nothing, whatever its weights): behind branches each would be waited for before the next is issued, and on small
// maps that chain is the kernel's whole time.  Batch 16, bf16: 3x3 on 854 channels at 7x7 5.6 -> 3.5 us.
// What bounds it on larger batches is the first-level cache: 3x3 with TX = 7 reads 4.3 vectors per output, with TX = 2
// 10.5 (829 channels at 7x7, batch 64, fp32: 9.1 -> 6.3 us, 3.4 TB/s of input and output).  A 5x5 window unrolled whole
// holds so many rows at once that one or two wavefronts fit a SIMD and runs of four spill; so its rows go round a loop
// with the next row requested while this one is used, and 16-bit data takes four channels per thread instead of eight:
// 900 channels at 7x7, batch 256: fp32 57 -> 30 us, bf16 47 -> 22 us; 374 at 14x14, batch 16, bf16: 7.8 -> 6.5 us.
template <typename T, int K> struct DwVec { static constexpr int V = K == 5 ? 4 : VecOf<T>::V; };
template <int BYTES> struct DwRaw { typedef uint4 type; };
template <> struct DwRaw<8> { typedef uint2 type; };

__device__ __forceinline__ void dw_load(__amdgpu_buffer_rsrc_t r, unsigned off, uint4& q) { q = load_b128(r, off, 0); }
__device__ __forceinline__ void dw_load(__amdgpu_buffer_rsrc_t r, unsigned off, uint2& q) { q = load_b64(r, off, 0); }
template <typename T, int V> __device__ __forceinline__ void dw_unpack(const uint4& q, float (&f)[V]) { unpack16<T, V>(q, f); }
template <typename T, int V> __device__ __forceinline__ void dw_unpack(const uint2& q, float (&f)[V]) {
  const T* h = reinterpret_cast<const T*>(&q);
#pragma unroll
  for (int e = 0; e < V; ++e) f[e] = (float)h[e];
}

template <typename T, int K, int S, int TX>
__global__ __launch_bounds__(256) void depthwise_nhwc_vec_kernel(const T* __restrict__ x, unsigned x_bytes, const T* __restrict__ w,
                                                                 const float* __restrict__ bias,
                                                                 const T* __restrict__ res, T* __restrict__ y,
                                                                 unsigned total, int c_real, int cp, int h, int wd,
                                                                 int ho, int wo, int xblocks, int pad, int act) {
  constexpr int V = DwVec<T, K>::V;
  constexpr int ES = (int)sizeof(T);
  constexpr int NIN = (TX - 1) * S + K;
  constexpr int AHEAD = K == 5 ? 2 : 1;   // sets of row registers
  typedef typename DwRaw<V * ES>::type raw_t;
  const unsigned idx = blockIdx.x * 256u + threadIdx.x;
  if (idx >= total) return;
  const unsigned nvec = (unsigned)cp / V;
  const unsigned cv = idx % nvec;
  unsigned r = idx / nvec;
  const int xb = (int)(r % (unsigned)xblocks); r /= (unsigned)xblocks;
  const int oy = (int)(r % (unsigned)ho);
  const int n = (int)(r / (unsigned)ho);
  const int c0 = (int)cv * V;

  const __amdgpu_buffer_rsrc_t xr = make_rsrc(x, x_bytes), wr = make_rsrc(w, (unsigned)(K * K * cp) * ES);
  float4_t bv[V / 4];   // requested first: at the end they would be waited for in full
#pragma unroll
  for (int i = 0; i < V / 4; ++i) bv[i] = load_bias4(bias, c_real, c0 + 4 * i);
  float acc[TX][V];
#pragma unroll
  for (int t = 0; t < TX; ++t)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[t][e] = 0.0f;

  const int ox0 = xb * TX;
  const int ix_base = ox0 * S - pad;
  unsigned col[NIN];   // byte offset of a window column inside its row, out of range outside the image
#pragma unroll
  for (int j = 0; j < NIN; ++j)
    col[j] = (unsigned)(ix_base + j) < (unsigned)wd ? (unsigned)((ix_base + j) * cp + c0) * ES : kOutOfRange;
  raw_t raw[AHEAD][NIN], wraw[AHEAD][K];
  auto request = [&](int u, int b) {
    const int iy = oy * S - pad + u;
    const bool inside = (unsigned)iy < (unsigned)h;
    const unsigned row = inside ? (unsigned)((n * h + iy) * wd * cp) * ES : 0u;
    const unsigned out = inside ? 0u : kOutOfRange;
#pragma unroll
    for (int j = 0; j < NIN; ++j) dw_load(xr, (col[j] | out) + row, raw[b][j]);
#pragma unroll
    for (int v = 0; v < K; ++v) dw_load(wr, (unsigned)((u * K + v) * cp + c0) * ES | out, wraw[b][v]);
  };
  auto use = [&](int b) {
    float wk[K][V];
#pragma unroll
    for (int v = 0; v < K; ++v) dw_unpack<T, V>(wraw[b][v], wk[v]);
#pragma unroll
    for (int j = 0; j < NIN; ++j) {
      float in[V];
      dw_unpack<T, V>(raw[b][j], in);
#pragma unroll
      for (int t = 0; t < TX; ++t) {
        const int v = j - t * S;
        if (v >= 0 && v < K) {
#pragma unroll
          for (int e = 0; e < V; ++e) acc[t][e] += in[e] * wk[v][e];
        }
      }
    }
  };
  if constexpr (AHEAD == 1) {
#pragma unroll
    for (int u = 0; u < K; ++u) { request(u, 0); use(0); }
  } else {
    request(0, 0);
#pragma unroll 1
    for (int u = 0; u + 2 < K; u += 2) { request(u + 1, 1); use(0); request(u + 2, 0); use(1); }
    use(0);
  }
#pragma unroll
  for (int t = 0; t < TX; ++t) {
    const int ox = ox0 + t;
    if (ox >= wo) break;
    const size_t off = ((size_t)(n * ho + oy) * wo + ox) * cp + c0;
    float o[V];
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = acc[t][e] + bv[e / 4][e % 4];
    if (res) {
      float rv[V];
      dw_unpack<T, V>(*reinterpret_cast<const raw_t*>(res + off), rv);
#pragma unroll
      for (int e = 0; e < V; ++e) o[e] += rv[e];
    }
    raw_t q;
    if constexpr (ES == 4) {
      q.x = __float_as_uint(act_f(o[0], act)); q.y = __float_as_uint(act_f(o[1], act));
      q.z = __float_as_uint(act_f(o[2], act)); q.w = __float_as_uint(act_f(o[3], act));
    } else {
      T* hq = reinterpret_cast<T*>(&q);
#pragma unroll
      for (int e = 0; e < V; ++e) hq[e] = (T)act_f(o[e], act);
    }
    *reinterpret_cast<raw_t*>(y + off) = q;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void nchw_to_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                           long total, int c, int hw, int cp) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int ch = (int)(i % cp);
  const long pix = i / cp;
  const long n = pix / hw;
  const int p = (int)(pix - n * hw);
  T v = (T)0.0f;
  if (ch < c) v = x[(n * c + ch) * hw + p];
  y[i] = v;
}

template <typename T>
__global__ __launch_bounds__(256) void nhwc_to_nchw_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                           long total, int c, int hw, int cp) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;  // index into dense [n][c][hw]
  if (i >= total) return;
  const int p = (int)(i % hw);
  const long nc = i / hw;
  const int ch = (int)(nc % c);
  const long n = nc / c;
  y[i] = x[(n * hw + p) * cp + ch];
}

// [o][c][khw] -> [o][khw][cp], zero in the pad channels
template <typename T>
__global__ __launch_bounds__(256) void repack_weights_kernel(const T* __restrict__ w, T* __restrict__ y,
                                                             long total, int c, int khw, int cp) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int ch = (int)(i % cp);
  const long ot = i / cp;
  const int tpos = (int)(ot % khw);
  const long o = ot / khw;
  T v = (T)0.0f;
  if (ch < c) v = w[(o * c + ch) * khw + tpos];
  y[i] = v;
}

// [o][9][cp] -> the order in which the independent-wavefront 3x3 kernel's lanes fetch their MFMA
// operands: [filter tile of 16][64-byte channel chunk][tap][lane = quad * 16 + filter][16 bytes], so
// that one wavefront-wide load reads 1 KiB of consecutive memory; zero past the last filter / channel
template <typename T>
__global__ __launch_bounds__(256) void repack_wave_kernel(const T* __restrict__ w, T* __restrict__ y, long total,
                                                          int o_count, int cp, int nchunk) {
  constexpr int EPI = 16 / (int)sizeof(T);
  const long i = (long)blockIdx.x * 256 + threadIdx.x;   // one element of the output
  if (i >= total) return;
  const int e = (int)(i % EPI);
  long q = i / EPI;
  const int lane = (int)(q & 63); q >>= 6;
  const int tap = (int)(q % 9); q /= 9;
  const int chunk = (int)(q % nchunk);
  const long tm = q / nchunk;
  const long o = tm * 16 + (lane & 15);
  const int ch = chunk * 4 * EPI + (lane >> 4) * EPI + e;
  T v = (T)0.0f;
  if (o < o_count && ch < cp) v = w[(o * 9 + tap) * cp + ch];
  y[i] = v;
}

// [rows][k] (k contiguous) -> the order in which the reduction-split kernel's lanes fetch their MFMA
// operands: [16-row tile][64-byte round of k][lane = quad * 16 + row][16 bytes]; zero past the last row / k
template <typename T>
__global__ __launch_bounds__(256) void repack_rows_kernel(const T* __restrict__ w, T* __restrict__ y, long total,
                                                          int rows, int k, int rounds) {
  constexpr int EPI = 16 / (int)sizeof(T);
  const long i = (long)blockIdx.x * 256 + threadIdx.x;   // one element of the output
  if (i >= total) return;
  const int e = (int)(i % EPI);
  long q = i / EPI;
  const int lane = (int)(q & 63); q >>= 6;
  const int rnd = (int)(q % rounds);
  const long tm = q / rounds;
  const long row = tm * 16 + (lane & 15);
  const int kk = rnd * 4 * EPI + (lane >> 4) * EPI + e;
  T v = (T)0.0f;
  if (row < rows && kk < k) v = w[row * k + kk];
  y[i] = v;
}

// Expansion weights [ce][cp] -> the order in which the inverted-residual kernel's lanes fetch them, [block of 16 channels][xh
// 32-byte units of the reduction]: whole 64-byte rounds as [lane = quad * 16 + row][16 bytes], an odd last unit (fp32) as
// [lane][8 bytes].  In 16-bit data two blocks share 32 channels, four at a time, so that a lane's results of both are
// eight consecutive channels.  Zero past the last channel.
template <typename T>
__global__ __launch_bounds__(256) void pack_expand_kernel(const T* __restrict__ w, T* __restrict__ y, long total, int ce, int cp,
                                                          int xh) {
  constexpr int ES = (int)sizeof(T), EPI = 16 / ES;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;   // one element of the output
  if (i >= total) return;
  const int per = xh * (512 / ES);
  const int blk = (int)(i / per), off = (int)(i % per);
  const int whole = (xh / 2) * (1024 / ES);
  int lane, k;
  if (off < whole) {
    const int rnd = off / (1024 / ES), q = off % (1024 / ES);
    lane = q / EPI;
    k = rnd * 4 * EPI + (lane >> 4) * EPI + q % EPI;
  } else {
    const int q = off - whole;
    lane = q / (EPI / 2);
    k = (xh / 2) * 4 * EPI + (lane >> 4) * (EPI / 2) + q % (EPI / 2);
  }
  const int row = lane & 15;
  const int ch = ES == 4 ? blk * 16 + row : (blk >> 1) * 32 + (row >> 2) * 8 + (blk & 1) * 4 + (row & 3);
  y[i] = (ch < ce && k < cp) ? w[(long)ch * cp + k] : (T)0.0f;
}

// fp32 weights [rows][terms] -> the operands of mbrow3_kernel: [tile of 16 rows][round of 16 terms][operand][lane = quad * 16 + row], of four
// terms (wh, wl), (wm, wh) or, twice, (wh, wl), (wm, wm), (wh, wh).  image: a round is four window rows (channel, row) of four
// columns, the last of them zero.
__global__ __launch_bounds__(256) void pack_parts_kernel(const float* __restrict__ w, uint4* __restrict__ y, int total, int rows, int terms,
                                                         int rounds, int twice, int image) {
  const int i = blockIdx.x * 256 + threadIdx.x;          // one lane of one round
  if (i >= total) return;
  const int lane = i & 63, unit = i >> 6, rnd = unit % rounds, row = unit / rounds * 16 + (lane & 15);
  float v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int p = rnd * 4 + (lane >> 4), k = image ? p * 3 + q : p * 4 + q;
    v[q] = row < rows && k < terms && !(image && q == 3) ? w[(long)row * terms + k] : 0.0f;
  }
  uint32_t h[2], m[2], l[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) split3(__float_as_uint(v[2 * q]), __float_as_uint(v[2 * q + 1]), h[q], m[q], l[q]);
  uint4* const dst = y + (size_t)unit * (twice ? 192 : 128) + lane;
  dst[0] = make_uint4(h[0], h[1], l[0], l[1]);
  dst[64] = twice ? make_uint4(m[0], m[1], m[0], m[1]) : make_uint4(m[0], m[1], h[0], h[1]);
  if (twice) dst[128] = make_uint4(h[0], h[1], h[0], h[1]);
}

template <typename T>
__global__ __launch_bounds__(256) void widen_kernel(const T* __restrict__ x, float* __restrict__ y, long count) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < count) y[i] = (float)x[i];
}

// What the strips of mbrow3_kernel may meet before they have to run on the fp32 instruction, from a block's weights (one work-group; the
// bounds are derived at PartsLimits).
__global__ __launch_bounds__(256) void parts_limit_kernel(PartsLimits p) {
  __shared__ unsigned s_top[4][5], s_small[4][2];
  // largest magnitude as bits (infinities and NaN above all numbers); whether there is one below 2^-110 that is not zero
  unsigned top[5] = {0, 0, 0, 0, 0}, small[2] = {0, 0};
  auto scan = [&](const float* w, long n, unsigned& most, unsigned* low) {
    for (long i = threadIdx.x; w && i < n; i += 256) {
      const unsigned mag = __float_as_uint(w[i]) & 0x7fffffffu;
      most = max(most, mag);
      if (low) *low |= mag - 1 < ((127u - 110u) << 23) - 1 ? 1u : 0u;
    }
  };
  scan(p.we, (long)p.ce * p.terms, top[0], &small[0]);
  scan(p.wd, (long)9 * p.cpe, top[1], nullptr);
  scan(p.wp, (long)p.o * p.cpe, top[2], &small[1]);
  scan(p.be, p.ce, top[3], nullptr);
  scan(p.bd, p.ce, top[4], nullptr);
  for (int step = 32; step; step >>= 1) {
    for (unsigned& v : top) v = max(v, (unsigned)__shfl_xor((int)v, step));
    for (unsigned& v : small) v |= (unsigned)__shfl_xor((int)v, step);
  }
  if ((threadIdx.x & 63) == 0) {
    for (int i = 0; i < 5; ++i) s_top[threadIdx.x >> 6][i] = top[i];
    for (int i = 0; i < 2; ++i) s_small[threadIdx.x >> 6][i] = small[i];
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < 4; ++w) {
    for (int i = 0; i < 5; ++i) top[i] = max(top[i], s_top[w][i]);
    for (int i = 0; i < 2; ++i) small[i] |= s_small[w][i];
  }
  *p.limit = parts_limit(p, __uint_as_float(top[0]), __uint_as_float(top[1]), __uint_as_float(top[2]), __uint_as_float(top[3]),
                         __uint_as_float(top[4]), small[0], small[1]);
}

// Weights -> the operand order of the split kernel: [filter tile of 16][round][part][lane = quarter * 16 + filter]
// [8 channels].  A round holds four (tap, 8-channel group) units, one per quarter.
template <typename T>
__global__ __launch_bounds__(256) void pack_split_kernel(const T* __restrict__ w, uint4* __restrict__ y, int total,
                                                         int o_count, int c_count, int taps, int khwc, int nfull,
                                                         int groups_last, int rtot) {
  constexpr int P = sizeof(T) == 4 ? 3 : 1;
  const int i = blockIdx.x * 256 + threadIdx.x;    // one lane of one round of one filter tile
  if (i >= total) return;
  const int lane = i & 63;
  const int rg = (i >> 6) % rtot, tm = (i >> 6) / rtot;
  const int o = tm * 16 + (lane & 15);
  const bool full = rg < nfull * taps;
  const int chunk = full ? rg / taps : nfull;
  const int u = (rg - chunk * taps) * 4 + (lane >> 4);
  const int ng = full ? 4 : groups_last;
  const int tap = u / ng, c0 = chunk * 32 + (u - tap * ng) * 8;
  uint32_t part[P][4];
  T vals[8];
  const bool row = o < o_count && tap < taps && c0 < c_count;
  const size_t step = khwc ? 1 : taps;
  const T* const src = w + (row ? (khwc ? ((size_t)o * taps + tap) * c_count + c0 : ((size_t)o * c_count + c0) * taps + tap) : 0);
#pragma unroll
  for (int e = 0; e < 8; ++e) vals[e] = src[row && c0 + e < c_count ? e * step : 0];   // (all eight in flight at once)
#pragma unroll
  for (int e = 0; e < 8; ++e) vals[e] = row && c0 + e < c_count ? vals[e] : (T)0.0f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (P == 1)
      part[0][e] = (uint32_t)__builtin_bit_cast(uint16_t, vals[2 * e]) | (uint32_t)__builtin_bit_cast(uint16_t, vals[2 * e + 1]) << 16;
    else
      split3(__float_as_uint(vals[2 * e]), __float_as_uint(vals[2 * e + 1]), part[0][e], part[1][e], part[2][e]);
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    y[((size_t)(i >> 6) * P + p) * 64 + lane] = make_uint4(part[p][0], part[p][1], part[p][2], part[p][3]);
}

// Every input pixel of a 2x2 map lies inside the 3x3 window (pad 1) of every output pixel, so
// the layer is one dense matrix from the whole input map to the whole output map: the tap that
// links input pixel (iy, ix) to output pixel (oy, ox) is (iy - oy + 1, ix - ox + 1).
template <typename T>
__global__ __launch_bounds__(256) void repack_map2x2_kernel(const T* __restrict__ w, const float* __restrict__ bias,
                                                            T* __restrict__ y, float* __restrict__ bias_out, int o_count,
                                                            int c, int cp_in, int cp_out, int rows_by_channel) {
  const long total = (long)16 * cp_out * cp_in;
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int col = (int)(i % (4 * cp_in));
  const int row = (int)(i / (4 * cp_in));
  const int pi = col / cp_in, ch = col % cp_in;
  const int po = rows_by_channel ? (row & 3) : row / cp_out;
  const int o = rows_by_channel ? (row >> 2) : row % cp_out;
  T v = (T)0.0f;
  if (o < o_count && ch < c) {
    const int u = (pi >> 1) - (po >> 1) + 1, t = (pi & 1) - (po & 1) + 1;
    v = w[((long)o * c + ch) * 9 + u * 3 + t];
  }
  y[i] = v;
  if (col == 0) bias_out[row] = (bias && o < o_count) ? bias[o] : 0.0f;
}

// [o][ktot] -> [rows][kp], zero beyond ktot and beyond the last filter
template <typename T>
__global__ __launch_bounds__(256) void repack_stem_kernel(const T* __restrict__ w, T* __restrict__ y, long total,
                                                          int o_count, int ktot, int kp) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int k = (int)(i % kp);
  const long o = i / kp;
  T v = (T)0.0f;
  if (o < o_count && k < ktot) v = w[o * ktot + k];
  y[i] = v;
}

// OIHW 7x7 weights -> [rows][224]: k = u * 32 + (v + 1) * 4 + c (window row, window column shifted by one slot,
// channel), zero elsewhere
template <typename T>
__global__ __launch_bounds__(256) void repack_stem7_kernel(const T* __restrict__ w, T* __restrict__ y, long total,
                                                           int o_count, int c_count) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int k = (int)(i % kStem7K);
  const long o = i / kStem7K;
  const int u = k >> 5, slot = (k >> 2) & 7, c = k & 3;
  T v = (T)0.0f;
  if (o < o_count && c < c_count && slot >= 1) v = w[((o * c_count + c) * 7 + u) * 7 + (slot - 1)];
  y[i] = v;
}

// OIHW 7x7 weights -> [16-filter block][round][part (fp32: of three)][lane = quarter * 16 + filter][8 columns]: unit 4 * round + quarter =
// (channel, window row), its columns a zero and the window row's seven
template <typename T>
__global__ __launch_bounds__(256) void pack_stem7_kernel(const T* __restrict__ w, uint4* __restrict__ y, int total, int o_count, int c_count) {
  const int i = blockIdx.x * 256 + threadIdx.x;      // one lane of one round of one block
  if (i >= total) return;
  const int lane = i & 63, round = (i >> 6) % kStem7Rounds, block = (i >> 6) / kStem7Rounds;
  const int o = block * 16 + (lane & 15), q = 4 * round + (lane >> 4), c = q / 7, u = q - c * 7;
  const bool row = o < o_count && c < c_count;
  const T* const src = w + (row ? ((o * c_count + c) * 7 + u) * 7 : 0);
  T v[8];
  v[0] = (T)0.0f;
#pragma unroll
  for (int e = 0; e < 7; ++e) v[e + 1] = row ? src[e] : (T)0.0f;
  if constexpr (sizeof(T) == 2) {
    uint4 all;
    __builtin_memcpy(&all, v, 16);
    y[(size_t)(i >> 6) * 64 + lane] = all;
  } else {
    uint32_t part[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split3(__float_as_uint(v[2 * e]), __float_as_uint(v[2 * e + 1]), part[0][e], part[1][e], part[2][e]);
#pragma unroll
    for (int p = 0; p < 3; ++p) y[((size_t)(i >> 6) * 3 + p) * 64 + lane] = make_uint4(part[p][0], part[p][1], part[p][2], part[p][3]);
  }
}

inline dim3 blocks_for(long total) { return dim3((unsigned)((total + 255) / 256)); }

int plane_slices(int total) {
  int s = (total + 1023) / 1024;
  return s < 1 ? 1 : (s > 64 ? 64 : s);
}

template <typename T>
int depthwise_dispatch(const cprune_conv_desc& d, const void* x, const void* w, const float* bias,
                       const void* res, void* y, hipStream_t s) {
  const int ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  dim3 grid((unsigned)(d.n * d.c_in), (unsigned)plane_slices(ho * wo));
#define GO(K)                                                                                     \
  hipLaunchKernelGGL((depthwise_kernel<T, K>), grid, dim3(256), 0, s, (const T*)x, (const T*)w,  \
                     bias, (const T*)res, (T*)y, d.c_in, d.h, d.w, ho, wo, d.stride, d.pad, d.act)
  switch (d.kh) {
    case 1: GO(1); break;
    case 3: GO(3); break;
    case 5: GO(5); break;
    case 7: GO(7); break;
    default: return CPRUNE_ERR_UNSUPPORTED;
  }
#undef GO
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

}  // namespace

int launch_conv_depthwise(const cprune_conv_desc& d, const void* x, const void* w, const float* bias,
                          const void* residual, void* y, hipStream_t s) {
  if (d.kh != d.kw) return CPRUNE_ERR_UNSUPPORTED;
  if (d.dtype == CPRUNE_F32) return depthwise_dispatch<float>(d, x, w, bias, residual, y, s);
  if (d.dtype == CPRUNE_F16) return depthwise_dispatch<_Float16>(d, x, w, bias, residual, y, s);
  return depthwise_dispatch<__bf16>(d, x, w, bias, residual, y, s);
}

int launch_maxpool(const void* x, int n, int c, int h, int w, int k, int stride, int pad, int dt,
                   void* y, hipStream_t s) {
  const int ho = conv_out_dim(h, k, stride, pad), wo = conv_out_dim(w, k, stride, pad);
  dim3 grid((unsigned)(n * c), (unsigned)plane_slices(ho * wo));
  if (dt == CPRUNE_F32)
    hipLaunchKernelGGL(maxpool_kernel<float>, grid, dim3(256), 0, s, (const float*)x, (float*)y, h, w,
                       ho, wo, k, stride, pad);
  else if (dt == CPRUNE_F16)
    hipLaunchKernelGGL(maxpool_kernel<_Float16>, grid, dim3(256), 0, s, (const _Float16*)x,
                       (_Float16*)y, h, w, ho, wo, k, stride, pad);
  else
    hipLaunchKernelGGL(maxpool_kernel<__bf16>, grid, dim3(256), 0, s, (const __bf16*)x, (__bf16*)y, h,
                       w, ho, wo, k, stride, pad);
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_gavgpool(const void* x, int n, int c, int hw, int dt, void* y, hipStream_t s) {
  const int planes = n * c;
  dim3 grid((unsigned)((planes + 3) / 4));
  if (dt == CPRUNE_F32)
    hipLaunchKernelGGL(gavgpool_kernel<float>, grid, dim3(256), 0, s, (const float*)x, (float*)y,
                       planes, hw);
  else if (dt == CPRUNE_F16)
    hipLaunchKernelGGL(gavgpool_kernel<_Float16>, grid, dim3(256), 0, s, (const _Float16*)x,
                       (_Float16*)y, planes, hw);
  else
    hipLaunchKernelGGL(gavgpool_kernel<__bf16>, grid, dim3(256), 0, s, (const __bf16*)x, (__bf16*)y,
                       planes, hw);
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

#define CPRUNE_BY_DTYPE(DT, CALL)                      \
  do {                                                  \
    if ((DT) == CPRUNE_F32) { typedef float T; CALL; }  \
    else if ((DT) == CPRUNE_F16) { typedef _Float16 T; CALL; } \
    else { typedef __bf16 T; CALL; }                    \
  } while (0)

int launch_maxpool_nhwc(const void* x, int n, int cp, int h, int w, int k, int stride, int pad, int dt,
                        void* y, hipStream_t s) {
  const int ho = conv_out_dim(h, k, stride, pad), wo = conv_out_dim(w, k, stride, pad);
  const long total = (long)n * ho * wo * cp;
  const int vec = dt == CPRUNE_F32 ? 4 : 8;
  if (cp % vec == 0 && total / vec < (1L << 32)) {
    const long tv = total / vec;
#define CPRUNE_POOL(K)                                                                                               \
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL((maxpool_nhwc_vec_kernel<T, K>), blocks_for(tv), dim3(256), 0, s, (const T*)x, \
                                         (T*)y, (unsigned)tv, cp, h, w, ho, wo, k, stride, pad))
    if (k == 2) { CPRUNE_POOL(2); }
    else if (k == 3) { CPRUNE_POOL(3); }
    else { CPRUNE_POOL(0); }
#undef CPRUNE_POOL
    CPRUNE_LAUNCH_CHECK();
    return CPRUNE_OK;
  }
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(maxpool_nhwc_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)x,
                                         (T*)y, total, cp, h, w, ho, wo, k, stride, pad));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_gavgpool_nhwc(const void* x, int n, int cp, int hw, int dt, void* y, hipStream_t s) {
  const int per_block = 16 * (dt == CPRUNE_F32 ? 4 : 8), vblocks = (cp + per_block - 1) / per_block;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(gavgpool_nhwc_kernel<T>, dim3((unsigned)(n * vblocks)), dim3(256), 0, s,
                                         (const T*)x, (T*)y, vblocks, cp, hw));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

// Outputs per thread.  A long run loads less per output, a short one leaves more threads: with few vectors of output
// (`vecs` = pixels times channel vectors) the kernel's time is one thread's, with many it is the loads'.  Sevens, made
// for the widths 7, 14, 28 and 56, only where they leave little undone at the row's end
// (400 at 15x15, bf16: 8.2 us in fours, 10.1 in sevens; 200 at 20x20: 8.1 and 7.5), and not on input rows over 40 KB, where window rows
// lie too many threads apart (584 at 28x28, batch 33, fp32, 64 KB, fours / sevens 29 / 36; 5x5 on 598 at 56x56, batch 3, 19 / 25; 5x5 on
// 16-bit data has no such case: 310 at 112x112, batch 4, 69 KB, 33 / 31).  At stride 2 fours from where they are
// well over a work-group a unit (110 at 64x64, batch 10, fp32, 280k vectors, 1.1 groups, twos / fours 5.2 / 6.8).  800 random layers a
// type, window and stride: 1.00-1.02 times the best run's time on average.  us for runs of 1 / 2 / 4 / 7, batch
// 64 unless said:
//   3x3, fp32:  829 at 7x7 (652k) 11.2 / 9.1 / 6.9 / 6.3; 374 at 14x14, batch 16 (301k) 5.1 / 4.4 / 4.3 / 4.1;
//               829 at 7x7, batch 16 (163k) 3.9 / 3.5 / 3.3 / 3.9; 400 at 14x14, batch 4 (78k) 3.0 / 2.7 / 3.1 / 3.7
//   3x3, bf16:  500 at 14x14 (803k) 10.8 / 11.1 / 9.7 / 7.9; 300 at 14x14 (477k) 7.5 / 6.7 / 7.2 / 7.0
//   3x3 / stride 2, fp32: 500 to 7x7 (401k) 8.8 / 7.7 / 6.6 / 5.3; 400 to 8x8 (410k) 8.1 / 7.4 / 6.0 / 6.9;
//               70 to 28x28, batch 16 (251k) 4.6 / 4.0 / 4.7 / 4.6
//   5x5, fp32:  374 at 14x14, batch 16 (301k) 9.6 / 7.2 / 6.7 / 5.6; 829 at 7x7, batch 16 (163k) 6.4 / 5.3 / 4.4 / 5.3;
//               400 at 14x14, batch 4 (78k) 4.8 / 3.7 / 4.2 / 5.1; 900 at 7x7, batch 4 (45k) 3.4 / 3.6 / 4.1 / 5.1
//   5x5, bf16:  374 at 14x14, batch 16 (301k) 9.1 / 7.3 / 7.0 / 6.5; 900 at 7x7, batch 4 (45k) 3.4 / 4.1 / 5.1 / 6.3
//   5x5 / stride 2, bf16: 300 to 11x11, batch 48 (441k) 12.3 / 9.8 / 7.9 / 10.4; 374 to 7x7, batch 16 (75k) 4.8 / 4.4 / 5.6 / 7.0
static int depthwise_run(long vecs, int wo, int k, int stride, bool f32, size_t row_bytes) {
  const int by7 = (wo + 6) / 7 * 7, by4 = (wo + 3) / 4 * 4;
  bool sevens = stride == 1 ? by7 * 5 <= by4 * 6 : k == 3 && f32 && wo % 7 == 0;
  if (row_bytes > 40 * 1024 && (f32 || k == 3)) sevens = false;
  const long full = k == 3 && (stride == 2 || !f32) ? 384 : 128;   // thousands of vectors
  if (sevens && vecs >= (k == 3 && stride == 1 && !f32 ? 512L : 256L) * 1024) return 7;
  if (vecs >= full * 1024) return 4;
  return vecs >= 64L * 1024 ? 2 : 1;
}

template <typename T>
static int depthwise_nhwc_dispatch(const cprune_conv_desc& d, int cp, const void* x, const void* w,
                                   const float* bias, const void* res, void* y, hipStream_t s) {
  const int ho = conv_out_dim(d.h, d.kh, d.stride, d.pad), wo = conv_out_dim(d.w, d.kw, d.stride, d.pad);
  constexpr int V = VecOf<T>::V;
  // vectorised kernel: 3x3 and 5x5 at stride 1 or 2, channel stride a whole number of vectors
  if ((d.kh == 3 || d.kh == 5) && (d.stride == 1 || d.stride == 2) && cp % V == 0) {
    const long per_row = (long)d.n * ho * (cp / (d.kh == 5 ? DwVec<T, 5>::V : V));
    const int tx = depthwise_run(per_row * wo, wo, d.kh, d.stride, sizeof(T) == 4, (size_t)d.w * cp * sizeof(T));
    const int xblocks = (wo + tx - 1) / tx;
    const long total = per_row * xblocks;
    const size_t xb = (size_t)d.n * d.h * d.w * cp * sizeof(T);
    if (total < (1L << 32) && xb < ((size_t)1 << 31)) {
      const unsigned x_bytes = (unsigned)xb;
#define GOV(K, S, TX)                                                                                           \
      hipLaunchKernelGGL((depthwise_nhwc_vec_kernel<T, K, S, TX>), blocks_for(total), dim3(256), 0, s, (const T*)x, x_bytes, \
                         (const T*)w, bias, (const T*)res, (T*)y, (unsigned)total, d.c_in, cp, d.h, d.w, ho, wo,  \
                         xblocks, d.pad, d.act)
      const int key = d.kh * 100 + d.stride * 10 + tx;
      switch (key) {
        case 311: GOV(3, 1, 1); break;
        case 312: GOV(3, 1, 2); break;
        case 314: GOV(3, 1, 4); break;
        case 317: GOV(3, 1, 7); break;
        case 321: GOV(3, 2, 1); break;
        case 322: GOV(3, 2, 2); break;
        case 324: GOV(3, 2, 4); break;
        case 327: if constexpr (sizeof(T) == 4) { GOV(3, 2, 7); } break;      // (16-bit data: 290-940 bytes of scratch a lane)
        case 511: GOV(5, 1, 1); break;
        case 512: GOV(5, 1, 2); break;
        case 514: GOV(5, 1, 4); break;
        case 517: GOV(5, 1, 7); break;
        case 521: GOV(5, 2, 1); break;
        case 522: GOV(5, 2, 2); break;
        case 524: GOV(5, 2, 4); break;
      }
#undef GOV
      CPRUNE_LAUNCH_CHECK();
      return CPRUNE_OK;
    }
  }
  const long total = (long)d.n * ho * wo * cp;
#define GO(K)                                                                                          \
  hipLaunchKernelGGL((depthwise_nhwc_kernel<T, K>), blocks_for(total), dim3(256), 0, s, (const T*)x,   \
                     (const T*)w, bias, (const T*)res, (T*)y, total, d.c_in, cp, d.h, d.w, ho, wo,     \
                     d.stride, d.pad, d.act)
  switch (d.kh) {
    case 1: GO(1); break;
    case 3: GO(3); break;
    case 5: GO(5); break;
    case 7: GO(7); break;
    default: return CPRUNE_ERR_UNSUPPORTED;
  }
#undef GO
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_depthwise_nhwc(const cprune_conv_desc& d, int cp, const void* x, const void* w, const float* bias,
                          const void* residual, void* y, hipStream_t s) {
  if (d.kh != d.kw) return CPRUNE_ERR_UNSUPPORTED;
  if (d.dtype == CPRUNE_F32) return depthwise_nhwc_dispatch<float>(d, cp, x, w, bias, residual, y, s);
  if (d.dtype == CPRUNE_F16) return depthwise_nhwc_dispatch<_Float16>(d, cp, x, w, bias, residual, y, s);
  return depthwise_nhwc_dispatch<__bf16>(d, cp, x, w, bias, residual, y, s);
}

int launch_nchw_to_nhwc(const void* x, int n, int c, int hw, int cp, int dt, void* y, hipStream_t s) {
  const long total = (long)n * hw * cp;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(nchw_to_nhwc_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)x,
                                         (T*)y, total, c, hw, cp));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_nhwc_to_nchw(const void* x, int n, int c, int hw, int cp, int dt, void* y, hipStream_t s) {
  const long total = (long)n * c * hw;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(nhwc_to_nchw_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)x,
                                         (T*)y, total, c, hw, cp));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_repack_weights(const void* w, int o, int c, int khw, int cp, int dt, void* y, hipStream_t s) {
  const long total = (long)o * khw * cp;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(repack_weights_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w,
                                         (T*)y, total, c, khw, cp));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

size_t wave_packed_bytes(int o, int cp, int dt) {
  const int cc = dt == CPRUNE_F32 ? 16 : 32;   // channels per 64-byte chunk
  return (size_t)((o + 15) / 16) * ((cp + cc - 1) / cc) * 9 * 1024;
}

int launch_repack_wave(const void* w_khwc, int o, int cp, int dt, void* y, hipStream_t s) {
  const int cc = dt == CPRUNE_F32 ? 16 : 32;
  const int nchunk = (cp + cc - 1) / cc;
  const long total = (long)(wave_packed_bytes(o, cp, dt) / dtype_size(dt));
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(repack_wave_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w_khwc,
                                         (T*)y, total, o, cp, nchunk));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

size_t rows_packed_bytes(int rows, int k, int dt) {
  const size_t per_round = 64 / dtype_size(dt);
  return (size_t)((rows + 15) / 16) * ((k + per_round - 1) / per_round) * 1024;
}

int launch_repack_rows(const void* w, int rows, int k, int dt, void* y, hipStream_t s) {
  const int per_round = (int)(64 / dtype_size(dt));
  const int rounds = (k + per_round - 1) / per_round;
  const long total = (long)(rows_packed_bytes(rows, k, dt) / dtype_size(dt));
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(repack_rows_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, (T*)y,
                                         total, rows, k, rounds));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

size_t expand_packed_bytes(int ce, int xh, int dt) {
  const int cc = (int)(64 / dtype_size(dt));   // channels per chunk
  return (size_t)((ce + cc - 1) / cc) * (cc / 16) * xh * 512;
}

int launch_pack_expand(const void* w, int ce, int cp, int xh, int dt, void* y, hipStream_t s) {
  const long total = (long)(expand_packed_bytes(ce, xh, dt) / dtype_size(dt));
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(pack_expand_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, (T*)y,
                                         total, ce, cp, xh));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_widen(const void* x, long count, int dt, float* y, hipStream_t s) {
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(widen_kernel<T>, blocks_for(count), dim3(256), 0, s, (const T*)x, y, count));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

size_t parts_packed_bytes(int rows, int rounds, bool twice) { return (size_t)((rows + 15) / 16) * rounds * (twice ? 3072 : 2048); }

int launch_pack_parts(const void* w, int rows, int terms, int rounds, bool twice, bool image, void* y, hipStream_t s) {
  const int total = (rows + 15) / 16 * rounds * 64;
  hipLaunchKernelGGL(pack_parts_kernel, blocks_for(total), dim3(256), 0, s, (const float*)w, (uint4*)y, total, rows, terms, rounds, twice ? 1 : 0,
                     image ? 1 : 0);
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_parts_limit(const PartsLimits& p, hipStream_t s) {
  hipLaunchKernelGGL(parts_limit_kernel, dim3(1), dim3(256), 0, s, p);
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

size_t split_packed_bytes(int o, int c, int taps, int dt, bool whole) {
  return (size_t)((o + 15) / 16) * split_rounds(whole ? (c + 31) / 32 * 32 : c, taps, nullptr, nullptr, nullptr) * (dt == CPRUNE_F32 ? 3072 : 1024);
}

int launch_pack_split(const void* w, int o, int c, int taps, int khwc, int dt, void* y, hipStream_t s, bool whole) {
  int nfull, groups_last, rounds_last;
  const int rtot = split_rounds(whole ? (c + 31) / 32 * 32 : c, taps, &nfull, &groups_last, &rounds_last);
  const long total = (long)((o + 15) / 16) * rtot * 64;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(pack_split_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, (uint4*)y,
                                         (int)total, o, c, taps, khwc, nfull, groups_last, rtot));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int stem_packed_k(int k, int dt) {
  const int rk = dt == CPRUNE_F32 ? 16 : 32;   // k per 64-byte MFMA round
  return (3 * k * k + rk - 1) / rk * rk;
}

int launch_repack_stem(const void* w, int o, int ktot, int rows, int kp, int dt, void* y, hipStream_t s) {
  const long total = (long)rows * kp;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(repack_stem_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, (T*)y,
                                         total, o, ktot, kp));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_repack_stem7(const void* w, int o, int c, int rows, int dt, void* y, hipStream_t s) {
  const long total = (long)rows * kStem7K;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(repack_stem7_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, (T*)y,
                                         total, o, c));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_pack_stem7(const void* w, int o, int c, int dt, void* y, hipStream_t s) {
  const int total = (o + 15) / 16 * kStem7Rounds * 64;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(pack_stem7_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, (uint4*)y, total, o, c));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

int launch_repack_map2x2(const void* w, const float* bias, int o, int c, int cp_in, int cp_out,
                         int rows_by_channel, int dt, void* w_out, float* bias_out, hipStream_t s) {
  const long total = (long)16 * cp_out * cp_in;
  CPRUNE_BY_DTYPE(dt, hipLaunchKernelGGL(repack_map2x2_kernel<T>, blocks_for(total), dim3(256), 0, s, (const T*)w, bias,
                                         (T*)w_out, bias_out, o, c, cp_in, cp_out, rows_by_channel));
  CPRUNE_LAUNCH_CHECK();
  return CPRUNE_OK;
}

}  // namespace cprune
