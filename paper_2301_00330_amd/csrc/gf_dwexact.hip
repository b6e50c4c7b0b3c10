// Vanilla back-propagation (Sec. 3.1) of depthwise layers: every (image, channel) plane is a
// small 2-D problem of its own.  Undilated layers of stride 1 or 2, whose padded plane fits LDS, take one pass for both
// gradients (dw_exact_onepass_k and dw_exact_stride2_k below).  The others: a block stages a run of whole planes in LDS with coalesced
// 16-byte loads (NCHW planes of consecutive channels are one contiguous stream) and all tap
// arithmetic runs from LDS.  Both kernels move each tensor through HBM once.
//   input gradient   g_x[h, w]  = sum_taps theta[c, u, v] * g_y[(h + p - u d) / s, (w + p - v d) / s]
//   weight gradient  g_theta[c, u, v] = sum_{n, i, j} x[i s - p + u d, j s - p + v d] * g_y[i, j]
// The weight gradient is formed per plane (fixed-order sums) and the planes of a channel are
// added over n by the finalize kernel.
#include "gf_internal.h"
#include "gf_mma.h"
#include <algorithm>

namespace gf {

namespace {

constexpr int kThreads = 256;
constexpr int kLdsBudget = 56 * 1024;

struct DwExactArgs {
  const void* x;
  const void* w;
  const void* gy;
  void* gx;
  float* part;   // [N, C, K * K]
  int C, H, W, Hy, Wy, K, s, p, dl;
  int planes, ppb;
  // stride-1 kernels: the staged operand sits in a zero frame of `halo` pixels (PH x PW per plane)
  int halo, PH, PW;
  FastDiv d_hw, d_w, d_hwy, d_wy, d_c;
};

// copy elements [e0, e1) of a tensor to LDS with 16-byte loads; returns the LDS pointer of
// element e0 (the image starts `shift` bytes into `buf`, which needs (e1 - e0) * sizeof(T) + 32 bytes)
template <class T>
__device__ __forceinline__ T* stage_run(const void* base, long e0, long e1, unsigned char* buf, int tid) {
  const long byte0 = e0 * (long)sizeof(T), byte1 = e1 * (long)sizeof(T);
  const long a0 = byte0 & ~15L;   // the tensor base is 16-byte aligned
  const int span = (int)(byte1 - a0);
  const int nvec = span >> 4;
  const uint4* src = reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(base) + a0);
  uint4* dst = reinterpret_cast<uint4*>(buf);
  for (int v = tid; v < nvec; v += 4 * kThreads) {
    // four loads in flight per lane; past-the-end indices are clamped and rewritten
    uint4 rg[4];
    int idx[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) idx[k] = min(v + k * kThreads, nvec - 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) rg[k] = load_stream16(src + idx[k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[idx[k]] = rg[k];
  }
  const int tail0 = nvec << 4;   // fewer than 16 trailing bytes: the run ends where the tensor ends
  const int ntail = (span - tail0) / (int)sizeof(T);
  if (tid < ntail)
    reinterpret_cast<T*>(buf + tail0)[tid] =
        reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(src) + tail0)[tid];
  return reinterpret_cast<T*>(buf + (int)(byte0 - a0));
}

// The same run of whole planes [pl0, pl0 + npl) of an [*, H, W] tensor, but laid out in LDS as
// [npl][PH][PW] with the plane at row `top`, column `left` of a zero frame, so that the tap loops
// need no bounds checks.  `buf` must have been cleared (the frame) before the call.
template <class T>
__device__ __forceinline__ void stage_padded(const void* base, int pl0, int npl, int H, int W, int top, int left,
                                             int PH, int PW, const FastDiv& d_hw, const FastDiv& d_w, T* buf,
                                             int tid) {
  constexpr int VE = 16 / (int)sizeof(T);
  const int HW = H * W;
  const long e0 = (long)pl0 * HW, e1 = e0 + (long)npl * HW;
  const long byte0 = e0 * (long)sizeof(T), byte1 = e1 * (long)sizeof(T);
  const long a0 = byte0 & ~15L;
  const int lead = (int)((byte0 - a0) / (long)sizeof(T));   // elements of the first vector that precede the run
  const int nvec = (int)((byte1 - a0) >> 4);                // whole vectors that end inside the run
  const uint4* src = reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(base) + a0);
  const int count = npl * HW;
  auto put = [&](int e, T val) {   // e: element index relative to the run
    const int pl = (int)d_hw.div((uint32_t)e);
    const int rem = e - pl * HW;
    const int h = (int)d_w.div((uint32_t)rem);
    buf[(pl * PH + h + top) * PW + rem - h * W + left] = val;
  };
  for (int v = tid; v < nvec; v += 4 * kThreads) {
    uint4 rg[4];
    int idx[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) idx[k] = min(v + k * kThreads, nvec - 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) rg[k] = load_stream16(src + idx[k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (v + k * kThreads >= nvec) continue;
      const T* el = reinterpret_cast<const T*>(&rg[k]);
#pragma unroll
      for (int i = 0; i < VE; ++i) {
        const int e = idx[k] * VE + i - lead;
        if (e >= 0) put(e, el[i]);
      }
    }
  }
  // elements behind the last whole vector (the run ends where the tensor may end)
  const int tail0 = nvec * VE - lead;
  if (tid < count - tail0 && tail0 + tid >= 0) put(tail0 + tid, static_cast<const T*>(base)[e0 + tail0 + tid]);
}

// ---------------------------------------------------------------------------
// input gradient: the block's planes one after the other (WAVE: small planes, a wave per plane);
// the K x K taps of the plane's channel sit in registers, K and the stride S are compile-time
// (S = 0: any stride, with divisions)
// ---------------------------------------------------------------------------
template <class T, int K, int S, bool WAVE>
__global__ __launch_bounds__(kThreads) void dw_exact_dgrad_k(DwExactArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pl0 = blockIdx.x * a.ppb;
  const int npl = min(a.ppb, a.planes - pl0);
  const int HW = a.H * a.W, HWy = a.Hy * a.Wy;
  const int in_bytes = ((a.ppb * HWy * (int)sizeof(T) + 32) + 15) & ~15;
  const T* gys = stage_run<T>(a.gy, (long)pl0 * HWy, (long)(pl0 + npl) * HWy, smem, tid);
  // the g_x image of the same planes, laid out as in memory (16-byte phase of its first element kept)
  const long obyte0 = (long)pl0 * HW * (long)sizeof(T);
  const long oa0 = obyte0 & ~15L;
  const int oshift = (int)(obyte0 - oa0);
  T* gxs = reinterpret_cast<T*>(smem + in_bytes + oshift);
  const T* w = static_cast<const T*>(a.w);
  __syncthreads();
  const int first = WAVE ? wave : 0, step = WAVE ? kThreads / 64 : 1;
  const int t0 = WAVE ? lane : tid, tstep = WAVE ? 64 : kThreads;
  const int s = S ? S : a.s;
  for (int pl = first; pl < npl; pl += step) {
    const int gpl = pl0 + pl;
    const int c = gpl - (int)a.d_c.div((uint32_t)gpl) * a.C;
    float wk[K * K];
#pragma unroll
    for (int t = 0; t < K * K; ++t) wk[t] = to_f32(w[(long)c * (K * K) + t]);
    const T* src = gys + pl * HWy;
    T* dst = gxs + pl * HW;
    for (int e = t0; e < HW; e += tstep) {
      const int h = (int)a.d_w.div((uint32_t)e);
      const int ww = e - h * a.W;
      int ri[K], cj[K];   // source row offset / column per tap, -1 where the tap does not reach a g_y pixel
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int nh = h + a.p - u * a.dl;
        const int i = S == 1 ? nh : nh / s;
        ri[u] = (nh >= 0 && i * s == nh && i < a.Hy) ? i * a.Wy : -1;
        const int nw = ww + a.p - u * a.dl;
        const int j = S == 1 ? nw : nw / s;
        cj[u] = (nw >= 0 && j * s == nw && j < a.Wy) ? j : -1;
      }
      float acc = 0.f;
#pragma unroll
      for (int u = 0; u < K; ++u)
#pragma unroll
        for (int v = 0; v < K; ++v) {
          const bool ok = (ri[u] | cj[v]) >= 0;
          const float g = to_f32(src[ok ? ri[u] + cj[v] : 0]);
          acc += ok ? wk[u * K + v] * g : 0.f;
        }
      dst[e] = from_f32<T>(acc);
    }
  }
  __syncthreads();
  // store the image: whole 16-byte vectors, then the partial vectors at both ends, which the
  // neighbouring blocks share, element by element
  T* out = static_cast<T*>(a.gx);
  const long e0 = (long)pl0 * HW;
  const int span = oshift + npl * HW * (int)sizeof(T);
  const int nvec = span >> 4;
  unsigned char* img = smem + in_bytes;
  unsigned char* dstb = reinterpret_cast<unsigned char*>(out) + oa0;
  for (int v = tid + (oshift ? 1 : 0); v < nvec; v += kThreads)
    store_stream16(dstb + ((long)v << 4), *reinterpret_cast<const uint4*>(img + (v << 4)));
  if (oshift) {
    const int nhead = min((16 - oshift) / (int)sizeof(T), npl * HW);
    if (tid < nhead) out[e0 + tid] = gxs[tid];
  }
  {
    const int tail0 = nvec << 4;
    const int ntail = (span - tail0) / (int)sizeof(T);
    const int efirst = (tail0 - oshift) / (int)sizeof(T);
    if (tid < ntail && efirst + tid >= 0) out[e0 + efirst + tid] = gxs[efirst + tid];
  }
}

// stride 1: g_y staged in a zero frame, no bounds checks in the tap loop
template <class T, int K, bool WAVE>
__global__ __launch_bounds__(kThreads) void dw_exact_dgrad_s1_k(DwExactArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pl0 = blockIdx.x * a.ppb;
  const int npl = min(a.ppb, a.planes - pl0);
  const int HW = a.H * a.W;
  const int pad_elems = a.ppb * a.PH * a.PW;
  const int in_bytes = (pad_elems * (int)sizeof(T) + 15) & ~15;
  T* gys = reinterpret_cast<T*>(smem);
  for (int i = tid; i < (in_bytes >> 4); i += kThreads) reinterpret_cast<uint4*>(smem)[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  stage_padded<T>(a.gy, pl0, npl, a.Hy, a.Wy, a.halo, a.halo, a.PH, a.PW, a.d_hwy, a.d_wy, gys, tid);
  const long obyte0 = (long)pl0 * HW * (long)sizeof(T);
  const long oa0 = obyte0 & ~15L;
  const int oshift = (int)(obyte0 - oa0);
  T* gxs = reinterpret_cast<T*>(smem + in_bytes + oshift);
  const T* w = static_cast<const T*>(a.w);
  __syncthreads();
  const int first = WAVE ? wave : 0, step = WAVE ? kThreads / 64 : 1;
  const int t0 = WAVE ? lane : tid, tstep = WAVE ? 64 : kThreads;
  int off[K * K];   // tap (u, v) reads g_y[h + p - u d][w + p - v d]
#pragma unroll
  for (int u = 0; u < K; ++u)
#pragma unroll
    for (int v = 0; v < K; ++v) off[u * K + v] = (a.p + a.halo - u * a.dl) * a.PW + a.p + a.halo - v * a.dl;
  for (int pl = first; pl < npl; pl += step) {
    const int gpl = pl0 + pl;
    const int c = gpl - (int)a.d_c.div((uint32_t)gpl) * a.C;
    float wk[K * K];
#pragma unroll
    for (int t = 0; t < K * K; ++t) wk[t] = to_f32(w[(long)c * (K * K) + t]);
    const T* src = gys + pl * a.PH * a.PW;
    T* dst = gxs + pl * HW;
    for (int e = t0; e < HW; e += tstep) {
      const int h = (int)a.d_w.div((uint32_t)e);
      const int ww = e - h * a.W;
      const T* q = src + h * a.PW + ww;
      float acc = 0.f;
#pragma unroll
      for (int t = 0; t < K * K; ++t) acc += wk[t] * to_f32(q[off[t]]);
      dst[e] = from_f32<T>(acc);
    }
  }
  __syncthreads();
  T* out = static_cast<T*>(a.gx);
  const long e0 = (long)pl0 * HW;
  const int span = oshift + npl * HW * (int)sizeof(T);
  const int nvec = span >> 4;
  unsigned char* img = smem + in_bytes;
  unsigned char* dstb = reinterpret_cast<unsigned char*>(out) + oa0;
  for (int v = tid + (oshift ? 1 : 0); v < nvec; v += kThreads)
    store_stream16(dstb + ((long)v << 4), *reinterpret_cast<const uint4*>(img + (v << 4)));
  if (oshift) {
    const int nhead = min((16 - oshift) / (int)sizeof(T), npl * HW);
    if (tid < nhead) out[e0 + tid] = gxs[tid];
  }
  {
    const int tail0 = nvec << 4;
    const int ntail = (span - tail0) / (int)sizeof(T);
    const int efirst = (tail0 - oshift) / (int)sizeof(T);
    if (tid < ntail && efirst + tid >= 0) out[e0 + efirst + tid] = gxs[efirst + tid];
  }
}

// stride 1: x staged in a zero frame of p pixels, no bounds checks in the tap loop
template <class T, int K, bool WAVE>
__global__ __launch_bounds__(kThreads) void dw_exact_wgrad_s1_k(DwExactArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float red[kThreads / 64][K * K];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pl0 = blockIdx.x * a.ppb;
  const int npl = min(a.ppb, a.planes - pl0);
  const int HWy = a.Hy * a.Wy;
  const int pad_elems = a.ppb * a.PH * a.PW;
  const int x_bytes = (pad_elems * (int)sizeof(T) + 15) & ~15;
  T* xs = reinterpret_cast<T*>(smem);
  for (int i = tid; i < (x_bytes >> 4); i += kThreads) reinterpret_cast<uint4*>(smem)[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  stage_padded<T>(a.x, pl0, npl, a.H, a.W, a.halo, a.halo, a.PH, a.PW, a.d_hw, a.d_w, xs, tid);
  const T* gys = stage_run<T>(a.gy, (long)pl0 * HWy, (long)(pl0 + npl) * HWy, smem + x_bytes, tid);
  __syncthreads();
  const int first = WAVE ? wave : 0, step = WAVE ? kThreads / 64 : 1;
  const int t0 = WAVE ? lane : tid, tstep = WAVE ? 64 : kThreads;
  int off[K * K];   // tap (u, v) of output (i, j) reads x[i - p + u d][j - p + v d]; the frame is p wide
#pragma unroll
  for (int u = 0; u < K; ++u)
#pragma unroll
    for (int v = 0; v < K; ++v) off[u * K + v] = (u * a.dl) * a.PW + v * a.dl;
  for (int pl = first; pl < npl; pl += step) {
    const T* xp = xs + pl * a.PH * a.PW;
    const T* gp = gys + pl * HWy;
    float acc[K * K];
#pragma unroll
    for (int t = 0; t < K * K; ++t) acc[t] = 0.f;
    for (int e = t0; e < HWy; e += tstep) {
      const int i = (int)a.d_wy.div((uint32_t)e);
      const int j = e - i * a.Wy;
      const float g = to_f32(gp[e]);
      const T* q = xp + i * a.PW + j;
#pragma unroll
      for (int t = 0; t < K * K; ++t) acc[t] += to_f32(q[off[t]]) * g;
    }
#pragma unroll
    for (int t = 0; t < K * K; ++t)
      for (int m = 32; m > 0; m >>= 1) acc[t] += __shfl_xor(acc[t], m, 64);
    float* dst = a.part + (long)(pl0 + pl) * (K * K);
    if constexpr (WAVE) {
      if (lane == 0) {
#pragma unroll
        for (int t = 0; t < K * K; ++t) dst[t] = acc[t];
      }
    } else {
      if (lane == 0) {
#pragma unroll
        for (int t = 0; t < K * K; ++t) red[wave][t] = acc[t];
      }
      __syncthreads();
      if (tid < K * K) {
        float sm = 0.f;
        for (int k = 0; k < kThreads / 64; ++k) sm += red[k][tid];
        dst[tid] = sm;
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// weight gradient: K x K accumulators per lane, one plane after the other; WAVE: small planes,
// every wave owns whole planes (no block barrier in the reduction)
// ---------------------------------------------------------------------------
template <class T, int K, bool WAVE>
__global__ __launch_bounds__(kThreads) void dw_exact_wgrad_k(DwExactArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float red[kThreads / 64][K * K];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int pl0 = blockIdx.x * a.ppb;
  const int npl = min(a.ppb, a.planes - pl0);
  const int HW = a.H * a.W, HWy = a.Hy * a.Wy;
  const int x_bytes = ((a.ppb * HW * (int)sizeof(T) + 32) + 15) & ~15;
  const T* xs = stage_run<T>(a.x, (long)pl0 * HW, (long)(pl0 + npl) * HW, smem, tid);
  const T* gys = stage_run<T>(a.gy, (long)pl0 * HWy, (long)(pl0 + npl) * HWy, smem + x_bytes, tid);
  __syncthreads();
  const int first = WAVE ? wave : 0, step = WAVE ? kThreads / 64 : 1;
  const int t0 = WAVE ? lane : tid, tstep = WAVE ? 64 : kThreads;
  for (int pl = first; pl < npl; pl += step) {
    const T* xp = xs + pl * HW;
    const T* gp = gys + pl * HWy;
    float acc[K * K];
#pragma unroll
    for (int t = 0; t < K * K; ++t) acc[t] = 0.f;
    for (int e = t0; e < HWy; e += tstep) {
      const int i = (int)a.d_wy.div((uint32_t)e);
      const int j = e - i * a.Wy;
      const float g = to_f32(gp[e]);
      const int hb = i * a.s - a.p, wb = j * a.s - a.p;
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int h = hb + u * a.dl;
        const bool okh = h >= 0 && h < a.H;
#pragma unroll
        for (int v = 0; v < K; ++v) {
          const int ww = wb + v * a.dl;
          const bool ok = okh && ww >= 0 && ww < a.W;
          const float xv = to_f32(xp[ok ? h * a.W + ww : 0]);
          acc[u * K + v] += ok ? xv * g : 0.f;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < K * K; ++t)
      for (int m = 32; m > 0; m >>= 1) acc[t] += __shfl_xor(acc[t], m, 64);
    float* dst = a.part + (long)(pl0 + pl) * (K * K);
    if constexpr (WAVE) {
      if (lane == 0) {
#pragma unroll
        for (int t = 0; t < K * K; ++t) dst[t] = acc[t];
      }
    } else {
      if (lane == 0) {
#pragma unroll
        for (int t = 0; t < K * K; ++t) red[wave][t] = acc[t];
      }
      __syncthreads();
      if (tid < K * K) {
        float s = 0.f;
        for (int k = 0; k < kThreads / 64; ++k) s += red[k][tid];
        dst[tid] = s;
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Both gradients of a stride-1, undilated layer in one pass over x, g_y and g_x (bound by HBM).  With the offset of a
// tap moved from x to g_y,
//   g_x[h, w] = sum_taps theta[u, v] * g_y[h + p - u, w + p - v],   g_theta[u, v] = sum_{h, w} x[h, w] * g_y[h + p - u, w + p - v],
// the two products read the same window of g_y and x only at the pixel itself: g_y is staged in a zero frame in LDS (as
// floats), x and g_x go between memory and registers.  A lane owns kQ pixels of a row, whose window is
// K rows of whole 16-byte LDS reads.  A block keeps one channel and walks its planes in `npb` images, `ipp` of them at a
// time, so the K x K sums stay in registers until the end and the launch that adds the slabs has npb times less to
// read.  Blocks of one XCD (block index mod 8) take neighbouring channels, whose planes share cache lines.
// Measured, both gradients, against the two launches below (us; x, g_y and g_x from memory):
//   fp32  144 channels, 56 x 56, n = 32: 79 -> 41 (4.2 TB/s)   576, 14 x 14, n = 128: 144 -> 47   960, 7 x 7, n = 128: 110 -> 24
//         192, 28 x 28, n = 32: 44 -> 17   72, 28 x 28, 5 x 5 taps, n = 32: 42 -> 17   16, 7 x 7, n = 1: 13 -> 9.6
//   bf16  144, 56 x 56, n = 64: 133 -> 64    96, 112 x 112, n = 64: 280 -> 184    144, 65 x 65, n = 32: 92 -> 52
// bf16 is bound by vector instructions (18 multiply-adds per pixel, the same as in fp32 on half the bytes).
// ---------------------------------------------------------------------------
constexpr int kQ = 4;

struct DwBothArgs {
  const void* x;
  const void* w;
  const void* gy;
  void* gx;      // null: not wanted
  float* part;   // [slabs][C][K * K]; null: g_theta not wanted
  int N, C, H, W, Hy, Wy, p, npb, ipp, blocks;
  int PH, PW;    // frame: H + K - 1 rows; columns: whole groups of kQ and the window of the last one
  int hr, hc;    // g_y stands at that row and column of it
  int groups;    // of kQ pixels per row (stride 2: of a pair of rows)
  int rows;      // stride 2: pairs of rows
  FastDiv d_wy, d_grp, d_vec, d_tail, d_items, d_c;
};

template <class T> struct __attribute__((packed, aligned(sizeof(T)))) Quad { T v[kQ]; };

// g_y of ni images of a channel into their frames
template <class T>
__device__ __forceinline__ void stage_frames(const DwBothArgs& a, const T* gy, int ni, float* fr, int tid) {
  constexpr int VE = 16 / (int)sizeof(T);
  const int HWy = a.Hy * a.Wy, FR = a.PH * a.PW, nvec = HWy / VE, ntail = HWy - nvec * VE;
  const long cHWy = (long)a.C * HWy;
  const bool whole = a.Wy % VE == 0;   // no vector runs over the end of a row
  const int vecs = ni * nvec;
  for (int v0 = tid; v0 < vecs; v0 += 4 * kThreads) {   // four loads of a lane in flight, clamped
    uint4 rg[4];
    int im[4], ve[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = min(v0 + k * kThreads, vecs - 1);
      im[k] = (int)a.d_vec.div((uint32_t)v);
      ve[k] = (v - im[k] * nvec) * VE;
      rg[k] = load_vec<T>(gy + im[k] * cHWy + ve[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (v0 + k * kThreads >= vecs) continue;
      const int row = (int)a.d_wy.div((uint32_t)ve[k]);
      int col = ve[k] - row * a.Wy;
      float* d = fr + im[k] * FR + (row + a.hr) * a.PW + col + a.hc;
      const T* el = reinterpret_cast<const T*>(&rg[k]);
      if (whole) {
#pragma unroll
        for (int i = 0; i < VE; ++i) d[i] = to_f32(el[i]);
      } else {
#pragma unroll
        for (int i = 0; i < VE; ++i) {
          *d++ = to_f32(el[i]);
          if (++col == a.Wy) { col = 0; d += a.PW - a.Wy; }
        }
      }
    }
  }
  for (int t = tid; t < ni * ntail; t += kThreads) {   // the last elements of the planes
    const int im = (int)a.d_tail.div((uint32_t)t), e = nvec * VE + t - im * ntail;
    const int row = (int)a.d_wy.div((uint32_t)e), col = e - row * a.Wy;
    fr[im * FR + (row + a.hr) * a.PW + col + a.hc] = to_f32(gy[im * cHWy + e]);
  }
}

// the block's sums: slab z of channel c
template <int K>
__device__ __forceinline__ void put_taps(const DwBothArgs& a, float (&aw)[K * K], float (&red)[kThreads / 64][K * K], int z, int c) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int t = 0; t < K * K; ++t)
    for (int m = 32; m > 0; m >>= 1) aw[t] += __shfl_xor(aw[t], m, 64);
  if (lane == 0) {
#pragma unroll
    for (int t = 0; t < K * K; ++t) red[wave][t] = aw[t];
  }
  __syncthreads();
  if (tid < K * K) {
    float sm = 0.f;
    for (int k = 0; k < kThreads / 64; ++k) sm += red[k][tid];
    a.part[((long)z * a.C + c) * (K * K) + tid] = sm;
  }
}

template <class T, int K>
__global__ __launch_bounds__(kThreads, K == 3 ? 7 : 3) void dw_exact_onepass_k(DwBothArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float red[kThreads / 64][K * K];
  constexpr int WN = (kQ + K - 1 + 3) / 4;   // window: WN 16-byte reads per row
  float* fr = reinterpret_cast<float*>(smem);
  const int tid = threadIdx.x;
  const int idx = (int)(blockIdx.x & 7) * (gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (idx >= a.blocks) return;   // (uniform)
  const int z = (int)a.d_c.div((uint32_t)idx), c = idx - z * a.C;
  const int n0 = z * a.npb, n1 = min(n0 + a.npb, a.N);
  const int HW = a.H * a.W, HWy = a.Hy * a.Wy, FR = a.PH * a.PW;
  for (int i = tid; i < a.ipp * FR / 4; i += kThreads) reinterpret_cast<uint4*>(smem)[i] = make_uint4(0, 0, 0, 0);
  float wk[K * K], aw[K * K];
#pragma unroll
  for (int t = 0; t < K * K; ++t) {
    wk[t] = a.gx ? to_f32(static_cast<const T*>(a.w)[c * (K * K) + t]) : 0.f;
    aw[t] = 0.f;
  }
  const int items = a.H * a.groups;
  const long cHW = (long)a.C * HW, cHWy = (long)a.C * HWy;
  for (int n = n0; n < n1; n += a.ipp) {
    const int ni = min(a.ipp, n1 - n);
    const T* gy = static_cast<const T*>(a.gy) + n * cHWy + (long)c * HWy;
    const T* x = static_cast<const T*>(a.x) + n * cHW + (long)c * HW;
    T* gx = static_cast<T*>(a.gx) + n * cHW + (long)c * HW;
    __syncthreads();   // the frames are cleared / the planes before have been read
    stage_frames<T>(a, gy, ni, fr, tid);
    __syncthreads();
    for (int g = tid; g < ni * items; g += kThreads) {
      const int im = (int)a.d_items.div((uint32_t)g), gr = g - im * items;
      const int h = (int)a.d_grp.div((uint32_t)gr), w0 = (gr - h * a.groups) * kQ;
      const long o = im * cHW + h * a.W + w0;
      const int cnt = min(kQ, a.W - w0);
      Quad<T> xq = {};
      if (!a.part) {
      } else if (cnt == kQ) {
        xq = *reinterpret_cast<const Quad<T>*>(x + o);
      } else {
#pragma unroll
        for (int e = 0; e < kQ; ++e)
          if (e < cnt) xq.v[e] = x[o + e];
      }
      float win[K][4 * WN];
      const float* src = fr + im * FR + h * a.PW + w0;
#pragma unroll
      for (int u = 0; u < K; ++u)
#pragma unroll
        for (int k = 0; k < WN; ++k) {
          const float4 q = *reinterpret_cast<const float4*>(src + u * a.PW + 4 * k);
          win[u][4 * k] = q.x; win[u][4 * k + 1] = q.y; win[u][4 * k + 2] = q.z; win[u][4 * k + 3] = q.w;
        }
      if (a.part) {
        float xv[kQ];
#pragma unroll
        for (int e = 0; e < kQ; ++e) xv[e] = to_f32(xq.v[e]);
#pragma unroll
        for (int u = 0; u < K; ++u)
#pragma unroll
          for (int v = 0; v < K; ++v)
#pragma unroll
            for (int e = 0; e < kQ; ++e) aw[u * K + v] += xv[e] * win[K - 1 - u][e + K - 1 - v];
      }
      if (a.gx) {
        float acc[kQ];
#pragma unroll
        for (int e = 0; e < kQ; ++e) acc[e] = 0.f;
#pragma unroll
        for (int u = 0; u < K; ++u)
#pragma unroll
          for (int v = 0; v < K; ++v)
#pragma unroll
            for (int e = 0; e < kQ; ++e) acc[e] += wk[u * K + v] * win[K - 1 - u][e + K - 1 - v];
        if (cnt == kQ) {
          Quad<T> out;
#pragma unroll
          for (int e = 0; e < kQ; ++e) out.v[e] = from_f32<T>(acc[e]);
          *reinterpret_cast<Quad<T>*>(gx + o) = out;
        } else {
#pragma unroll
          for (int e = 0; e < kQ; ++e)
            if (e < cnt) gx[o + e] = from_f32<T>(acc[e]);
        }
      }
    }
  }
  if (!a.part) return;
  // The zeros of the frame, and of x past the end of a row, meet every tap, also the ones that do not read there; with an
  // infinity or a NaN on the other side that is a NaN.  Where the sums of the block are not all finite, they are
  // formed again from what lies inside the map.
  float fin = 0.f;
#pragma unroll
  for (int t = 0; t < K * K; ++t) fin = __builtin_fmaf(aw[t], 0.f, fin);
  if (__syncthreads_or(fin != 0.f)) {
#pragma unroll
    for (int t = 0; t < K * K; ++t) aw[t] = 0.f;
    for (int n = n0; n < n1; ++n) {
      const T* gy = static_cast<const T*>(a.gy) + n * cHWy + (long)c * HWy;
      const T* x = static_cast<const T*>(a.x) + n * cHW + (long)c * HW;
      for (int e = tid; e < HW; e += kThreads) {
        const int h = e / a.W, w = e - h * a.W;
        const float xv = to_f32(x[e]);
#pragma unroll
        for (int u = 0; u < K; ++u)
#pragma unroll
          for (int v = 0; v < K; ++v) {
            const int i = h + a.p - u, j = w + a.p - v;
            if (i >= 0 && i < a.Hy && j >= 0 && j < a.Wy) aw[u * K + v] += xv * to_f32(gy[i * a.Wy + j]);
          }
      }
    }
  }
  put_taps<K>(a, aw, red, z, c);
}

// The same for stride 2 (undilated).  With A = h + p, B = w + p, a pixel of x or g_x meets the taps of its parity,
//   u = A mod 2 + 2 m, v = B mod 2 + 2 l,   at g_y[A / 2 - m, B / 2 - l],
// so a lane owns two rows A = 2 a, 2 a + 1 of four columns B = 4 b ..: every tap is multiplied with every g_y pixel of a
// window of (K + 1) / 2 rows and (K + 3) / 2 columns once per product, and nothing is divided or tested per tap.  In the two
// launches above a tap costs divisions by the stride and a test, and the weight gradient a shuffle tree per plane.
// Measured, both gradients, the two launches / one pass (us):
//   fp32  576 channels, 14 x 14, n = 128 (130 MB): 201 / 66   96, 112 x 112, n = 32: 697 / 92   144, 56 x 56, n = 32: 101 / 47
//         72, 56 x 56, 5 x 5 taps, n = 32: 96 / 30   576, 15 x 17, n = 8: 17.4 / 12.2   8, 200 x 200, n = 2: 55 / 36   16, 7 x 7, n = 1: 10.2 / 6.2
//   bf16  138 / 42   150 / 60   89 / 31   98 / 30   18.2 / 11.2   63 / 33   10.3 / 6.7
// Errors against 64-bit sums: g_theta 0.81 .. 1.04 of the former ones, g_x 0.82 .. 0.98 (fp32).  What is left of the time on
// small maps is the chain staging -> barrier -> x -> store that a block walks per group of images.  (x of the pieces at the
// ends of a row element by element: bf16 46, 68, 31 and 33 us for the first four, fp32 69, 90, 48 and 37.)
// One gradient alone takes the same pass, so that it has the same bits as beside the other.  300 layers (16 - 576 channels, 7 x 7 -
// 112 x 112, n = 1 - 64, both kernel sizes and types), two launches / one pass, in the mean: both gradients 2.5, g_w 1.46, g_x 2.2
// times as fast.  Slower alone: g_w of few large planes, a block or less per CU, and where few blocks leave several slabs (bf16,
// 16 channels, 112 x 112, n = 16 10.7 / 14.8; 96, n = 4 12.2 / 15.3; 16, 28 x 28, n = 16 5.4 / 7.7), g_x of the smallest calls (3.1 / 3.6).
template <class T, int K>
__global__ __launch_bounds__(kThreads, K == 3 ? 7 : 3) void dw_exact_stride2_k(DwBothArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float red[kThreads / 64][K * K];
  constexpr int M = (K + 1) / 2;
  float* fr = reinterpret_cast<float*>(smem);
  const int tid = threadIdx.x;
  const int idx = (int)(blockIdx.x & 7) * (gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (idx >= a.blocks) return;   // (uniform)
  const int z = (int)a.d_c.div((uint32_t)idx), c = idx - z * a.C;
  const int n0 = z * a.npb, n1 = min(n0 + a.npb, a.N);
  const int HW = a.H * a.W, HWy = a.Hy * a.Wy, FR = a.PH * a.PW;
  for (int i = tid; i < a.ipp * FR / 4; i += kThreads) reinterpret_cast<uint4*>(smem)[i] = make_uint4(0, 0, 0, 0);
  float wk[K * K], aw[K * K];
#pragma unroll
  for (int t = 0; t < K * K; ++t) {
    if constexpr (sizeof(T) == 2) wk[t] = a.gx ? __uint_as_float(static_cast<const uint16_t*>(a.w)[c * (K * K) + t]) : 0.f;   // (the bits, so far)
    else wk[t] = a.gx ? static_cast<const float*>(a.w)[c * (K * K) + t] : 0.f;
    aw[t] = 0.f;
  }
  bool finite_w = true;   // (uniform) else the frame's zeros would not be neutral in g_x
  const int items = a.rows * a.groups;
  const long cHW = (long)a.C * HW, cHWy = (long)a.C * HWy;
  for (int n = n0; n < n1; n += a.ipp) {
    const int ni = min(a.ipp, n1 - n);
    const T* x = static_cast<const T*>(a.x) + n * cHW + (long)c * HW;
    T* gx = static_cast<T*>(a.gx) + n * cHW + (long)c * HW;
    __syncthreads();   // the frames are cleared / the planes before have been read
    stage_frames<T>(a, static_cast<const T*>(a.gy) + n * cHWy + (long)c * HWy, ni, fr, tid);
    __syncthreads();
    if (n == n0) {   // here, not ahead of the loop: the loads of g_y would wait for those of the kernel
      float wfin = 0.f;
#pragma unroll
      for (int t = 0; t < K * K; ++t) {
        if constexpr (sizeof(T) == 2) wk[t] = __uint_as_float(__float_as_uint(wk[t]) << 16);
        wfin = __builtin_fmaf(wk[t], 0.f, wfin);
      }
      finite_w = wfin == 0.f;
    }
    for (int g = tid; g < ni * items; g += kThreads) {
      const int im = (int)a.d_items.div((uint32_t)g), gr = g - im * items;
      const int ar = (int)a.d_grp.div((uint32_t)gr), bc = gr - ar * a.groups;
      // first pixel; the first row and up to three columns may lie before the map, the last ones past it
      const int h0 = 2 * (ar + (a.p >> 1)) - a.p, w0 = 4 * (bc + (a.p >> 2)) - a.p;
      const bool full = w0 >= 0 && w0 + kQ <= a.W;
      Quad<T> xq[2] = {};
      if (a.part) {
#pragma unroll
        for (int dr = 0; dr < 2; ++dr) {
          const int h = h0 + dr;
          if (h < 0 || h >= a.H) continue;
          const T* xp = x + im * cHW + h * a.W;
          if (a.W >= kQ) {   // (uniform) one load inside the row, shifted
            const int wc = min(max(w0, 0), a.W - kQ), sh = w0 - wc;
            const Quad<T> q = *reinterpret_cast<const Quad<T>*>(xp + wc);
#pragma unroll
            for (int e = 0; e < kQ; ++e)
#pragma unroll
              for (int f = 0; f < kQ; ++f)
                if (e + sh == f) xq[dr].v[e] = q.v[f];
          } else {
#pragma unroll
            for (int e = 0; e < kQ; ++e)
              if (w0 + e >= 0 && w0 + e < a.W) xq[dr].v[e] = xp[w0 + e];
          }
        }
      }
      float win[M][4];   // win[m'][l']: g_y[a - (M - 1) + m', 2 b - (M - 1) + l']
      const float* src = fr + im * FR + ar * a.PW + 2 * bc;
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float2 q = *reinterpret_cast<const float2*>(src + m * a.PW + 2 * k);
          win[m][2 * k] = q.x; win[m][2 * k + 1] = q.y;
        }
      if (a.part) {
#pragma unroll
        for (int u = 0; u < K; ++u)
#pragma unroll
          for (int v = 0; v < K; ++v)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              aw[u * K + v] += to_f32(xq[u & 1].v[2 * j + (v & 1)]) * win[M - 1 - (u >> 1)][M - 1 - (v >> 1) + j];
      }
      if (a.gx) {
        float acc[2][kQ];
#pragma unroll
        for (int e = 0; e < kQ; ++e) acc[0][e] = acc[1][e] = 0.f;
        if (finite_w) {
#pragma unroll
          for (int u = 0; u < K; ++u)
#pragma unroll
            for (int v = 0; v < K; ++v)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                acc[u & 1][2 * j + (v & 1)] += wk[u * K + v] * win[M - 1 - (u >> 1)][M - 1 - (v >> 1) + j];
        } else {
          const int i0 = ar + (a.p >> 1), j0 = 2 * (bc + (a.p >> 2));
#pragma unroll
          for (int u = 0; u < K; ++u)
#pragma unroll
            for (int v = 0; v < K; ++v)
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                const int i = i0 - (u >> 1), jj = j0 + j - (v >> 1);
                if (i >= 0 && i < a.Hy && jj >= 0 && jj < a.Wy)
                  acc[u & 1][2 * j + (v & 1)] += wk[u * K + v] * win[M - 1 - (u >> 1)][M - 1 - (v >> 1) + j];
              }
        }
#pragma unroll
        for (int dr = 0; dr < 2; ++dr) {
          const int h = h0 + dr;
          if (h < 0 || h >= a.H) continue;
          T* gp = gx + im * cHW + h * a.W + w0;
          if (full) {
            Quad<T> out;
#pragma unroll
            for (int e = 0; e < kQ; ++e) out.v[e] = from_f32<T>(acc[dr][e]);
            *reinterpret_cast<Quad<T>*>(gp) = out;
          } else {
#pragma unroll
            for (int e = 0; e < kQ; ++e)
              if (w0 + e >= 0 && w0 + e < a.W) gp[e] = from_f32<T>(acc[dr][e]);
          }
        }
      }
    }
  }
  if (!a.part) return;
  // (as above: sums that are not finite are formed again from what lies inside the map)
  float fin = 0.f;
#pragma unroll
  for (int t = 0; t < K * K; ++t) fin = __builtin_fmaf(aw[t], 0.f, fin);
  if (__syncthreads_or(fin != 0.f)) {
#pragma unroll
    for (int t = 0; t < K * K; ++t) aw[t] = 0.f;
    for (int n = n0; n < n1; ++n) {
      const T* gy = static_cast<const T*>(a.gy) + n * cHWy + (long)c * HWy;
      const T* x = static_cast<const T*>(a.x) + n * cHW + (long)c * HW;
      for (int e = tid; e < HWy; e += kThreads) {
        const int i = e / a.Wy, j = e - i * a.Wy;
        const float gv = to_f32(gy[e]);
#pragma unroll
        for (int u = 0; u < K; ++u)
#pragma unroll
          for (int v = 0; v < K; ++v) {
            const int h = 2 * i - a.p + u, w = 2 * j - a.p + v;
            if (h >= 0 && h < a.H && w >= 0 && w < a.W) aw[u * K + v] += to_f32(x[h * a.W + w]) * gv;
          }
      }
    }
  }
  put_taps<K>(a, aw, red, z, c);
}

bool shape_ok(const Geom& g) {
  if (g.Cg != 1 || g.Og != 1 || g.Ci != g.Co) return false;   // depthwise
  if (g.Kh != g.Kw) return false;
  return true;
}

// planes per block: as many as fit the budget, few enough for ~1024 blocks
int planes_per_block(const Geom& g, long per_plane) {
  long ppb = (kLdsBudget - 96) / per_plane;
  const long planes = (long)g.N * g.Ci;
  if (ppb > planes / 1024) ppb = planes / 1024;
  if (ppb < 1) ppb = 1;
  if (ppb > 64) ppb = 64;
  return (int)ppb;
}

DwExactArgs make_args(const Geom& g) {
  DwExactArgs a = {};
  a.C = g.Ci; a.H = g.H; a.W = g.W; a.Hy = g.Hy; a.Wy = g.Wy; a.K = g.Kh; a.s = g.s; a.p = g.p; a.dl = g.dl;
  a.planes = g.N * g.Ci;
  a.d_hw = FastDiv((uint32_t)(g.H * g.W));
  a.d_w = FastDiv((uint32_t)g.W);
  a.d_hwy = FastDiv((uint32_t)(g.Hy * g.Wy));
  a.d_wy = FastDiv((uint32_t)g.Wy);
  a.d_c = FastDiv((uint32_t)g.Ci);
  return a;
}

}  // namespace

// LDS bytes per plane of the two kernels (stride 1: the staged operand carries its zero frame)
static int dgrad_halo(const Geom& g) { const int h = (g.Kh - 1) * g.dl - g.p; return g.s == 1 && h > 0 ? h : 0; }
static long dgrad_per_plane(const Geom& g) {
  const int h = dgrad_halo(g);
  return ((long)(g.Hy + 2 * h) * (g.Wy + 2 * h) + (long)g.H * g.W) * g.b;
}
static long wgrad_per_plane(const Geom& g) {
  const int h = g.s == 1 ? g.p : 0;
  return ((long)(g.H + 2 * h) * (g.W + 2 * h) + (long)g.Hy * g.Wy) * g.b;
}

bool dw_exact_dgrad_ok(const Geom& g) {
  if (!shape_ok(g) || (g.Kh != 3 && g.Kh != 5 && g.Kh != 7)) return false;
  return dgrad_per_plane(g) + 96 <= kLdsBudget;
}

bool dw_exact_wgrad_ok(const Geom& g) {
  if (!shape_ok(g) || (g.Kh != 3 && g.Kh != 5)) return false;
  return wgrad_per_plane(g) + 96 <= kLdsBudget;
}

size_t ws_dw_exact_wgrad(const Geom& g) { return (size_t)g.N * g.Ci * g.KK * sizeof(float); }

template <class T, int K, int S>
static hipError_t dgrad_launch_s(DwExactArgs& a, bool wave, size_t lds, hipStream_t st) {
  const dim3 grid(cdiv(a.planes, a.ppb)), block(kThreads);
  if constexpr (S == 1) {
    if (wave) GF_LAUNCH((dw_exact_dgrad_s1_k<T, K, true>), grid, block, lds, st, a);
    else GF_LAUNCH((dw_exact_dgrad_s1_k<T, K, false>), grid, block, lds, st, a);
  } else {
    if (wave) GF_LAUNCH((dw_exact_dgrad_k<T, K, S, true>), grid, block, lds, st, a);
    else GF_LAUNCH((dw_exact_dgrad_k<T, K, S, false>), grid, block, lds, st, a);
  }
  return hipGetLastError();
}

template <class T, int K>
static hipError_t dgrad_launch_k(DwExactArgs& a, bool wave, size_t lds, hipStream_t st) {
  if (a.s == 1) return dgrad_launch_s<T, K, 1>(a, wave, lds, st);
  if (a.s == 2) return dgrad_launch_s<T, K, 2>(a, wave, lds, st);
  return dgrad_launch_s<T, K, 0>(a, wave, lds, st);
}

template <class T>
static hipError_t dgrad_launch_t(DwExactArgs& a, bool wave, size_t lds, hipStream_t st) {
  if (a.K == 3) return dgrad_launch_k<T, 3>(a, wave, lds, st);
  if (a.K == 5) return dgrad_launch_k<T, 5>(a, wave, lds, st);
  return dgrad_launch_k<T, 7>(a, wave, lds, st);
}

hipError_t launch_dw_exact_dgrad(const Geom& g, const void* w, const void* g_y, void* g_x, hipStream_t st) {
  DwExactArgs a = make_args(g);
  a.w = w; a.gy = g_y; a.gx = g_x;
  a.ppb = planes_per_block(g, dgrad_per_plane(g));
  const bool wave = g.H * g.W <= 256 && a.ppb >= 4;
  a.halo = dgrad_halo(g);
  a.PH = g.Hy + 2 * a.halo;
  a.PW = g.Wy + 2 * a.halo;
  const int in_bytes = g.s == 1 ? ((a.ppb * a.PH * a.PW * g.b + 15) & ~15)
                                : (((a.ppb * g.Hy * g.Wy * g.b + 32) + 15) & ~15);
  const int out_bytes = ((a.ppb * g.H * g.W * g.b + 32) + 15) & ~15;
  const size_t lds = (size_t)in_bytes + out_bytes;
  if (g.dtype == GF_BF16) return dgrad_launch_t<bf16_t>(a, wave, lds, st);
  return dgrad_launch_t<float>(a, wave, lds, st);
}

template <class T, int K>
static hipError_t wgrad_launch(DwExactArgs& a, bool wave, size_t lds, hipStream_t st) {
  const dim3 grid(cdiv(a.planes, a.ppb)), block(kThreads);
  if (a.s == 1) {
    if (wave) GF_LAUNCH((dw_exact_wgrad_s1_k<T, K, true>), grid, block, lds, st, a);
    else GF_LAUNCH((dw_exact_wgrad_s1_k<T, K, false>), grid, block, lds, st, a);
  } else {
    if (wave) GF_LAUNCH((dw_exact_wgrad_k<T, K, true>), grid, block, lds, st, a);
    else GF_LAUNCH((dw_exact_wgrad_k<T, K, false>), grid, block, lds, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_dw_exact_wgrad(const Geom& g, const void* x, const void* g_y, float* g_w, void* ws,
                                 hipStream_t st) {
  DwExactArgs a = make_args(g);
  a.x = x; a.gy = g_y; a.part = static_cast<float*>(ws);
  a.ppb = planes_per_block(g, wgrad_per_plane(g));
  const bool wave = g.Hy * g.Wy <= 256 && a.ppb >= 4;
  a.halo = g.s == 1 ? g.p : 0;
  a.PH = g.H + 2 * a.halo;
  a.PW = g.W + 2 * a.halo;
  const int x_bytes = g.s == 1 ? ((a.ppb * a.PH * a.PW * g.b + 15) & ~15)
                               : (((a.ppb * g.H * g.W * g.b + 32) + 15) & ~15);
  const int y_bytes = ((a.ppb * g.Hy * g.Wy * g.b + 32) + 15) & ~15;
  const size_t lds = (size_t)x_bytes + y_bytes;
  hipError_t e;
  if (g.dtype == GF_BF16)
    e = g.Kh == 3 ? wgrad_launch<bf16_t, 3>(a, wave, lds, st) : wgrad_launch<bf16_t, 5>(a, wave, lds, st);
  else
    e = g.Kh == 3 ? wgrad_launch<float, 3>(a, wave, lds, st) : wgrad_launch<float, 5>(a, wave, lds, st);
  if (e != hipSuccess) return e;
  // g_theta[c, t] = sum over n of part[n, c, t]
  return launch_finalize(a.part, g_w, g.Ci * g.KK, g.N, 1, 1.f, st);
}

// One pass for both gradients (or either): stride 1 or 2, no dilation, padding below the kernel size, the frame of one plane in
// LDS.  rows x groups: a lane's pieces of a plane.
struct Frame { int PH, PW, hr, hc, rows, groups; size_t bytes; };
static Frame both_frame(const Geom& g) {
  Frame f;
  if (g.s == 1) {
    f.hr = f.hc = g.Kh - 1 - g.p;
    f.rows = g.H;
    f.groups = cdiv(g.W, kQ);
    f.PH = g.H + g.Kh - 1;
    f.PW = f.groups * kQ + (g.Kh + 2) / 4 * 4;   // the window of the last group ends on a 16-byte boundary
  } else {
    const int m = (g.Kh + 1) / 2, a0 = g.p >> 1, b0 = g.p >> 2;   // window rows; first pair of rows, group of columns
    f.hr = m - 1 - a0;
    f.hc = m - 1 - 2 * b0;
    f.rows = ((g.H + g.p - 1) >> 1) - a0 + 1;
    f.groups = ((g.W + g.p - 1) >> 2) - b0 + 1;
    f.PH = (f.rows + m - 1 + 1) & ~1;            // (an even number: frames of 16 bytes each)
    f.PW = 2 * f.groups + 2;                     // the last group's window of four
  }
  f.bytes = (size_t)f.PH * f.PW * sizeof(float);
  return f;
}

bool dw_exact_onepass_ok(const Geom& g) {
  if (g.g == 1 || !shape_ok(g) || (g.Kh != 3 && g.Kh != 5) || g.s > 2 || g.dl != 1 || g.p >= g.Kh) return false;
  return both_frame(g).bytes <= 60 * 1024 && (long)g.N * g.Ci < (1L << 30);
}

template <class T>
static void launch_both(const DwBothArgs& a, int K, int s, size_t lds, hipStream_t st) {
  const dim3 grid((a.blocks + 7) & ~7), block(kThreads);
  if (s == 2) {
    if (K == 3) GF_LAUNCH((dw_exact_stride2_k<T, 3>), grid, block, lds, st, a);
    else GF_LAUNCH((dw_exact_stride2_k<T, 5>), grid, block, lds, st, a);
  } else {
    if (K == 3) GF_LAUNCH((dw_exact_onepass_k<T, 3>), grid, block, lds, st, a);
    else GF_LAUNCH((dw_exact_onepass_k<T, 5>), grid, block, lds, st, a);
  }
}

hipError_t launch_dw_exact_onepass(const Geom& g, const void* x, const void* w, const void* g_y, float* g_w, void* g_x,
                                void* ws, hipStream_t st) {
  DwBothArgs a = {};
  a.x = x; a.w = w; a.gy = g_y; a.gx = g_x; a.part = g_w ? static_cast<float*>(ws) : nullptr;
  a.N = g.N; a.C = g.Ci; a.H = g.H; a.W = g.W; a.Hy = g.Hy; a.Wy = g.Wy; a.p = g.p;
  const Frame f = both_frame(g);
  a.PH = f.PH; a.PW = f.PW; a.hr = f.hr; a.hc = f.hc; a.rows = f.rows; a.groups = f.groups;
  a.d_wy = FastDiv((uint32_t)g.Wy); a.d_grp = FastDiv((uint32_t)a.groups);
  const int VE = 16 / g.b, HWy = g.Hy * g.Wy, items = f.rows * f.groups;
  a.d_vec = FastDiv((uint32_t)std::max(HWy / VE, 1)); a.d_tail = FastDiv((uint32_t)std::max(HWy % VE, 1));
  a.d_items = FastDiv((uint32_t)items); a.d_c = FastDiv((uint32_t)g.Ci);
  // images at a time: about two groups of pixels per lane (g_x alone on a chip that is not full: one); images per block: what fills the last round of blocks best
  // (a block costs about a pass beside its passes; seven or three blocks per CU by registers)
  const int per_lane = !g_w && (long)g.Ci * g.N * items <= 512L * kThreads ? 1 : 2;
  a.ipp = std::max(1, std::min({g.N, per_lane * kThreads / items, (int)(24 * 1024 / f.bytes)}));
  a.ipp = cdiv(g.N, cdiv(g.N, a.ipp));
  const size_t lds = f.bytes * a.ipp;
  const long slots = 256L * std::min<long>(g.Kh == 5 ? 3 : 7, 160 * 1024 / (lds + 512));
  const int passes = cdiv(g.N, a.ipp);
  double best = 0;
  int k = 1;
  for (int q = 1; q <= 16 && q <= passes; ++q) {
    const double t = cdiv((long)g.Ci * cdiv(passes, q), slots) * (q + 1.0);
    if (q == 1 || t < best) { best = t; k = q; }
  }
  a.npb = k * a.ipp;
  const int nz = cdiv(passes, k);
  a.blocks = nz * g.Ci;
  if (g_w && nz == 1) a.part = g_w;   // one slab is the result: no launch to add slabs (2.8 us)
  if (g.dtype == GF_BF16) launch_both<bf16_t>(a, g.Kh, g.s, lds, st);
  else launch_both<float>(a, g.Kh, g.s, lds, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !g_w || nz == 1) return e;
  return launch_finalize(a.part, g_w, g.Ci * g.KK, nz, 1, 1.f, st);
}

}  // namespace gf
