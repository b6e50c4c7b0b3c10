// Gradient filtering on signed 8-bit codes (Supp. H combines the method with 8-bit gradient
// quantisation).  The reduced maps gy_u and x_u and the kernel sum are held as codes with one step
// size per tensor (round half to even, clipped to +-127); Eq. 5 and Eq. 3 then are integer
// contractions, which are exact, and the integer is scaled once by the product of the two step
// sizes and 1/s^2.  Dense layers with enough channels run on the matrix cores (gf_dense.hip); here:
//
//  * kernel_sum_q8_k   -- codes of the spatial kernel sum (text after Eq. 3)
//  * q8_wgrad_pair_k   -- Eq. 5 (groups, depthwise, few channels): one
//                         block per (c_o, c_i) pair, v_dot4_i32_i8 on 32-bit words where the plane
//                         allows it, 64-bit sums
//  * q8_dgrad_tile_k   -- Eq. 3 for planes that are multiples of four codes: a lane owns four patches
//                         of four (or one) input channels and walks the group's c_o; stores the
//                         full-resolution pixel runs itself where the patch rows allow
//  * q8_dgrad_k        -- Eq. 3 for the other planes: one lane per (n, c_i, patch)
//    both write the reduced map (storage type), or, where they cannot store full resolution
//    themselves, an fp32 map that the expansion kernels of the floating-point path replicate
#include "gf_internal.h"

#include <algorithm>

namespace gf {

namespace {

constexpr int kThreads = 256;

template <class T>
__global__ __launch_bounds__(kThreads) void kernel_sum_q8_k(const T* w, int8_t* w_q, int pairs, int KK, float inv) {
  const int e = blockIdx.x * kThreads + threadIdx.x;
  if (e < pairs) w_q[e] = q8_code(kernel_sum_of(w, e, KK), inv);
}

// ---------------------------------------------------------------------------
// Eq. 5, any layer: block = one (c_o, c_i') pair
// ---------------------------------------------------------------------------
struct Q8PairArgs {
  const int8_t* gyq;
  const int8_t* xq;
  float* g_w;
  int N, Ci, Co, Cg, Og, P, KK;
  float scale;
  FastDiv d_per;   // words (P / 4) or codes (P) per plane
};

// V4: the plane is a multiple of four codes, so rows are read as 32-bit words and multiplied with
// v_dot4_i32_i8.  A lane adds at most 1024 words into an int32 before it moves on to 64 bits.
template <bool V4>
__global__ __launch_bounds__(kThreads) void q8_wgrad_pair_k(Q8PairArgs a) {
  __shared__ long long red[kThreads / 64];
  const int pair = blockIdx.x;
  const int co = pair / a.Cg, cl = pair - co * a.Cg;
  const int ci = (co / a.Og) * a.Cg + cl;
  const int8_t* gbase = a.gyq + (long)co * a.P;
  const int8_t* xbase = a.xq + (long)ci * a.P;
  const long gs = (long)a.Co * a.P, xs = (long)a.Ci * a.P;   // image strides
  const int per = V4 ? a.P / 4 : a.P;                        // words / codes per plane
  const int tot = a.N * per;                                 // < 2^31 (host)
  long long s = 0;
  int i = threadIdx.x;
  while (i < tot) {
    int acc = 0;
#pragma unroll 4
    for (int u = 0; u < 1024; ++u) {
      if (i >= tot) break;
      const int n = (int)a.d_per.div((uint32_t)i);
      const int q = i - n * per;
      if (V4) {
        const int gv = reinterpret_cast<const int*>(gbase + n * gs)[q];
        const int xv = reinterpret_cast<const int*>(xbase + n * xs)[q];
        acc = __builtin_amdgcn_sdot4(gv, xv, acc, false);
      } else {
        acc += (int)gbase[n * gs + q] * (int)xbase[n * xs + q];
      }
      i += kThreads;
    }
    s += acc;
  }
  for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int k = 0; k < kThreads / 64; ++k) t += red[k];
    const float v = (float)t * a.scale;
    for (int k = 0; k < a.KK; ++k) a.g_w[(long)pair * a.KK + k] = v;
  }
}

// ---------------------------------------------------------------------------
// Eq. 3: dst[n, ci, p] = float(sum over the group's c_o of gy_q[n, co, p] * w_q[co, cl]) * scale
// ---------------------------------------------------------------------------
struct Q8DgradArgs {
  const int8_t* gyq;
  const int8_t* wq;
  void* dst;
  int N, Ci, Co, Cg, Og, P;
  long total;   // N * Ci * P
  float scale;
  FastDiv d_p, d_ci;
};

template <class D>
__global__ __launch_bounds__(kThreads) void q8_dgrad_k(Q8DgradArgs a) {
  const long e = (long)blockIdx.x * kThreads + threadIdx.x;
  if (e >= a.total) return;
  const int plane = (int)a.d_p.div((uint32_t)e);   // n * Ci + ci   (total < 2^31, checked on the host)
  const int p = (int)e - plane * a.P;
  const int n = (int)a.d_ci.div((uint32_t)plane);
  const int ci = plane - n * a.Ci;
  const int grp = ci / a.Cg, cl = ci - grp * a.Cg;
  const int8_t* gp = a.gyq + ((long)n * a.Co + (long)grp * a.Og) * a.P + p;
  const int8_t* wp = a.wq + (long)grp * a.Og * a.Cg + cl;
  int acc = 0;   // Og * 127^2 < 2^31 for Og <= 133 000 (checked on the host)
  for (int ol = 0; ol < a.Og; ++ol) acc += (int)gp[(long)ol * a.P] * (int)wp[(long)ol * a.Cg];
  static_cast<D*>(a.dst)[e] = from_f32<D>((float)acc * a.scale);
}

// The same for planes that are multiples of four codes: a lane owns four patches of CT input
// channels (CT = 4 needs group widths that are multiples of four; CT = 1 is for layers with so few
// input channels that 4 x 4 tiles would leave most of the chip idle).  Per c_o it reads one word of
// gy_q (four patches) and one word (or one code) of w_q and adds the 4 CT products.
struct Q8DgradTileArgs {
  const int8_t* gyq;
  const int8_t* wq;
  void* dst;
  int N, Ci, Co, Cg, Og, P;
  int total;   // N * (Ci / CT) * (P / 4)
  float scale;
  FastDiv d_p4, d_ct;
  // full-resolution store (RX > 0): the four patches of a lane lie in one patch row (4 | W_p)
  int H, W, Wq;   // Wq = W_p / 4
  FastDiv d_wq;
};

__device__ __forceinline__ int code_of(int word, int k) { return (int)(int8_t)(word >> (8 * k)); }

// SPLIT (1 or 4) neighbouring lanes share a tile and take every SPLIT-th c_o (integer sums, so the
// order does not matter); it shortens the chain of dependent loads when the tiles are few.
// RX > 0: instead of the reduced map, every pixel of the RX x RX input-side patches receives its
// patch's value (rounded once to the storage type, then replicated), as 16-byte runs of pixels.
template <class D, int CT, int SPLIT, int RX>
__global__ __launch_bounds__(kThreads) void q8_dgrad_tile_k(Q8DgradTileArgs a) {
  const int lane_id = blockIdx.x * kThreads + threadIdx.x;
  if (lane_id >= a.total * SPLIT) return;
  const int e = lane_id / SPLIT, sub = lane_id - e * SPLIT;
  const int P4 = a.P >> 2, CN = a.Ci / CT;
  const int planes = (int)a.d_p4.div((uint32_t)e);   // n * CN + c
  const int q = e - planes * P4;
  const int n = (int)a.d_ct.div((uint32_t)planes);
  const int ci0 = (planes - n * CN) * CT;
  const int grp = ci0 / a.Cg, cl0 = ci0 - grp * a.Cg;   // CT | Cg: the lane's channels share a group
  const int8_t* gp = a.gyq + ((long)n * a.Co + (long)grp * a.Og) * a.P + 4 * q;
  const int8_t* wp = a.wq + (long)grp * a.Og * a.Cg + cl0;
  int acc[CT][4];
#pragma unroll
  for (int i = 0; i < CT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0;
#pragma unroll 4
  for (int ol = sub; ol < a.Og; ol += SPLIT) {
    const int gv = *reinterpret_cast<const int*>(gp + (long)ol * a.P);
    int gc[4], wc[CT];
#pragma unroll
    for (int k = 0; k < 4; ++k) gc[k] = code_of(gv, k);
    if constexpr (CT == 4) {
      const int wv = *reinterpret_cast<const int*>(wp + (long)ol * a.Cg);
#pragma unroll
      for (int k = 0; k < 4; ++k) wc[k] = code_of(wv, k);
    } else {
      wc[0] = (int)wp[(long)ol * a.Cg];
    }
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] += wc[i] * gc[j];
  }
  if constexpr (SPLIT > 1) {
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        for (int m = SPLIT >> 1; m > 0; m >>= 1) acc[i][j] += __shfl_xor(acc[i][j], m, 64);
    if (sub != 0) return;
  }
#pragma unroll
  for (int i = 0; i < CT; ++i) {
    D v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = from_f32<D>((float)acc[i][j] * a.scale);
    if constexpr (RX == 0) {
      D* d = static_cast<D*>(a.dst) + ((long)n * a.Ci + ci0 + i) * a.P + 4 * q;
      if constexpr (sizeof(D) == 4) *reinterpret_cast<uint4*>(d) = *reinterpret_cast<const uint4*>(v);
      else *reinterpret_cast<uint2*>(d) = *reinterpret_cast<const uint2*>(v);
    } else {
      constexpr int VE = 16 / (int)sizeof(D);     // pixels per 16-byte run
      constexpr int NV = 4 * RX / VE;             // runs per pixel row of the lane's four patches
      const int hp = (int)a.d_wq.div((uint32_t)q);
      const int wq = q - hp * a.Wq;
      const int h0 = hp * RX, rows = min(RX, a.H - h0);
      __attribute__((aligned(16))) D px[4 * RX];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < RX; ++k) px[j * RX + k] = v[j];
      D* d = static_cast<D*>(a.dst) + (((long)n * a.Ci + ci0 + i) * a.H + h0) * a.W + wq * 4 * RX;
      // one run per lane and row: a wave's store covers whole lines, which is what the streaming
      // store wants; with several runs per lane each instruction writes parts of lines (plain stores)
      for (int row = 0; row < rows; ++row)
#pragma unroll
        for (int k = 0; k < NV; ++k) {
          if constexpr (NV == 1) store_stream16(d + (long)row * a.W, *reinterpret_cast<const uint4*>(px));
          else *reinterpret_cast<uint4*>(d + (long)row * a.W + k * VE) = *reinterpret_cast<const uint4*>(px + k * VE);
        }
    }
  }
}

template <class D, int RX>
static hipError_t q8_tile_launch(Q8DgradTileArgs& a, int ct, bool split, hipStream_t st) {
  const dim3 block(kThreads), grid(cdiv((long)a.total * (split ? 4 : 1), kThreads));
  if (ct == 4 && split) GF_LAUNCH((q8_dgrad_tile_k<D, 4, 4, RX>), grid, block, 0, st, a);
  else if (ct == 4) GF_LAUNCH((q8_dgrad_tile_k<D, 4, 1, RX>), grid, block, 0, st, a);
  else if (split) GF_LAUNCH((q8_dgrad_tile_k<D, 1, 4, RX>), grid, block, 0, st, a);
  else GF_LAUNCH((q8_dgrad_tile_k<D, 1, 1, RX>), grid, block, 0, st, a);
  return hipGetLastError();
}

// the tile kernel can store full resolution itself when a lane's four patches share a patch row and
// the pixel runs are whole 16-byte vectors
static bool q8_dgrad_full_ok(const Geom& g) {
  return g.P % 4 == 0 && g.Wp % 4 == 0 && (g.rx == 2 || g.rx == 4) && g.W == g.Wp * g.rx;
}

// full: dst is g_x at full resolution (only when q8_dgrad_full_ok), else the reduced map
template <class D>
static hipError_t q8_dgrad_launch(const Geom& g, const int8_t* gy_q, const int8_t* w_q, float fscale, void* dst,
                                  bool full, hipStream_t st) {
  if (g.P % 4 == 0) {
    // 4 x 4 tiles (fewest instructions per product) where the group width allows; when they are too
    // few to fill the chip and the channel sum is long, four lanes share a tile
    const int ct = g.Cg % 4 == 0 ? 4 : 1;
    Q8DgradTileArgs a;
    a.gyq = gy_q; a.wq = w_q; a.dst = dst;
    a.N = g.N; a.Ci = g.Ci; a.Co = g.Co; a.Cg = g.Cg; a.Og = g.Og; a.P = g.P;
    a.total = (int)((long)g.N * (g.Ci / ct) * (g.P / 4));
    a.scale = fscale;
    a.d_p4 = FastDiv((uint32_t)(g.P / 4));
    a.d_ct = FastDiv((uint32_t)(g.Ci / ct));
    a.H = g.H; a.W = g.W; a.Wq = g.Wp / 4 > 0 ? g.Wp / 4 : 1;
    a.d_wq = FastDiv((uint32_t)a.Wq);
    const bool split = g.Og >= 32 && a.total < 128 * 1024;
    if (full && g.rx == 2) return q8_tile_launch<D, 2>(a, ct, split, st);
    if (full) return q8_tile_launch<D, 4>(a, ct, split, st);
    return q8_tile_launch<D, 0>(a, ct, split, st);
  }
  Q8DgradArgs a;
  a.gyq = gy_q; a.wq = w_q; a.dst = dst;
  a.N = g.N; a.Ci = g.Ci; a.Co = g.Co; a.Cg = g.Cg; a.Og = g.Og; a.P = g.P;
  a.total = (long)g.N * g.Ci * g.P;
  a.scale = fscale;
  a.d_p = FastDiv((uint32_t)g.P);
  a.d_ci = FastDiv((uint32_t)g.Ci);
  GF_LAUNCH(q8_dgrad_k<D>, dim3(cdiv(a.total, kThreads)), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_kernel_sum_q8(const Geom& g, const void* w, float inv_delta, int8_t* w_q, hipStream_t st) {
  const int pairs = g.Co * g.Cg;
  const dim3 grid(cdiv(pairs, kThreads)), block(kThreads);
  if (g.dtype == GF_BF16)
    GF_LAUNCH(kernel_sum_q8_k<bf16_t>, grid, block, 0, st, static_cast<const bf16_t*>(w), w_q, pairs, g.KK, inv_delta);
  else
    GF_LAUNCH(kernel_sum_q8_k<float>, grid, block, 0, st, static_cast<const float*>(w), w_q, pairs, g.KK, inv_delta);
  return hipGetLastError();
}

size_t ws_bwd_weight_q8(const Geom& g) { return dense_q8_ok(g) ? ws_dense_q8(g, true, false, false, false) : 0; }

hipError_t launch_bwd_weight_q8(const Geom& g, const int8_t* x_q, const int8_t* gy_q, float scale, float* g_w,
                                void* ws, hipStream_t st) {
  if (dense_q8_ok(g))
    return launch_dense_q8(g, gy_q, 0.f, x_q, nullptr, 0.f, scale, scale, nullptr, g_w, nullptr, false, ws, st);
  const float fscale = scale / ((float)g.s * (float)g.s);
  Q8PairArgs a;
  a.gyq = gy_q; a.xq = x_q; a.g_w = g_w;
  a.N = g.N; a.Ci = g.Ci; a.Co = g.Co; a.Cg = g.Cg; a.Og = g.Og; a.P = g.P; a.KK = g.KK;
  a.scale = fscale;
  const bool v4 = g.P % 4 == 0;
  a.d_per = FastDiv((uint32_t)(v4 ? g.P / 4 : g.P));
  if (v4) GF_LAUNCH(q8_wgrad_pair_k<true>, dim3(g.Co * g.Cg), dim3(kThreads), 0, st, a);
  else GF_LAUNCH(q8_wgrad_pair_k<false>, dim3(g.Co * g.Cg), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

// Dense layers: the two-product launch where the caller brings its workspace.  Else the input gradient at full
// resolution goes through an fp32 reduced map in the workspace, the reduced one (and patch rows the kernel can store)
// needs none.  Integer sums: the same results, bit for bit.
size_t ws_bwd_input_q8(const Geom& g, bool reduced_out) {
  if (dense_q8_ok(g)) return ws_dense_q8(g, false, true, reduced_out, false);
  return ws_bwd_input_q8_least(g, reduced_out);
}
size_t ws_bwd_input_q8_least(const Geom& g, bool reduced_out) {
  if (reduced_out || q8_dgrad_full_ok(g)) return 0;
  return (size_t)g.N * g.Ci * g.P * sizeof(float);
}

bool q8_shape_ok(const Geom& g) {
  // 64-bit sums where they are long; the int32 sums of q8_dgrad_k and q8_wgrad_pair_k stay in range
  return g.r > 1 && g.Og <= kMaxTerms32 && (long)(g.P / kThreads + 1) <= kMaxTerms32;
}

hipError_t launch_bwd_input_q8(const Geom& g, const int8_t* gy_q, const int8_t* w_q, float scale, void* g_x,
                               bool reduced_out, void* ws, size_t ws_bytes, hipStream_t st) {
  if (dense_q8_ok(g) && ws_bytes >= ws_bwd_input_q8(g, reduced_out))
    return launch_dense_q8(g, gy_q, 0.f, nullptr, w_q, 0.f, scale, scale, nullptr, nullptr, g_x, reduced_out, ws, st);
  const float fscale = scale / ((float)g.s * (float)g.s);
  if (reduced_out || q8_dgrad_full_ok(g))
    return g.dtype == GF_BF16 ? q8_dgrad_launch<bf16_t>(g, gy_q, w_q, fscale, g_x, !reduced_out, st)
                              : q8_dgrad_launch<float>(g, gy_q, w_q, fscale, g_x, !reduced_out, st);
  hipError_t e = q8_dgrad_launch<float>(g, gy_q, w_q, fscale, ws, false, st);
  if (e != hipSuccess) return e;
  return launch_expand_f32(g, static_cast<const float*>(ws), g_x, st);
}

}  // namespace gf
