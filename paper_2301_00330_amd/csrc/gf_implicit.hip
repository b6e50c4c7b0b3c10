// Vanilla back-propagation (Sec. 3.1) of dense convolutions as implicit GEMMs on the MFMA cores
// of gfx950:
//
//   weight gradient  g_th[co, ci, t] = sum_{n, k} g_y[n, co, k] * xs[n, ci, k + dW(t)]      (k: output pixel)
//   input gradient   g_x[n, ci, j]   = sum_{t, co} th[co, ci, t] * g_y[n, co, j + dD(t)]   (j: input pixel)
//
// Stride 1, output map as wide as the input map ("same" padding): the pixel a tap reads is
// the flattened pixel index plus a constant,
//   dW(t) = (u d - p) W + (v d - p),   dD(t) = (p - u d) W_y + (p - v d),   t = (u, v),
// wherever the tap stays inside the image; where it leaves it the factor is a zero of the
// padding.  So no column tensor is built: the shifted operand is read straight from the
// tensor with 16-byte loads at 2- or 4-byte alignment, and a byte table [tap][8 pixels] says
// which of the eight elements are padding.  Planes are addressed as if they held 8 *
// ceil(HW / 8) pixels, so that a vector never straddles two images; the surplus positions
// are masked like padding.
//
// Stride s > 1: x is first split into its s x s phase planes xq[a, b][n, ci, i, j] =
// x[n, ci, s i + a, s j + b], stored with the row pitch W_y of the output map.  Tap (u, v) of
// output pixel (i, j) reads x[s i + u d - p, s j + v d - p], which is one fixed phase plane at
// (i, j) plus a constant: the same kernels run with a per-tap offset that includes the phase
// plane.  The input gradient is computed phase by phase (each phase of g_x receives the taps
// whose parity matches, so no multiplication is wasted on the zeros of a zero-inserted g_y)
// into phase planes that the last launch interleaves into g_x.
//
// Three launches: set-up (tables, kernel tap-major, phase planes), both products (xgemm_k: the first blocks of the
// grid are weight-gradient tiles, the rest input-gradient tiles; neither product alone fills the chip on small maps,
// where a block waits for its loads most of the time), and the last one (slab sums, tap-major to tap-minor, interleave).
// Inside xgemm_k: the pipeline of gf_gemm.h on 64 x 64, 128 x 64 or 128 x 128 tiles.  A wave of the largest reads four
// operand fragments from LDS per four matrix instructions, one of the smallest four per two, and LDS is what bounds bf16
// (a 64 x 64 x 64 step moves 48 KB through it, 384 clocks, for 128 clocks of matrix instructions).  Measured, both
// products, against separate kernels per product before (us, tensors of three rotating sets):
//   bf16  256 -> 256, 14 x 14, n = 64: 112 -> 74     512 -> 512, 7 x 7: 121 -> 79     256 -> 512, stride 2: 90 -> 63
//         256 -> 256, 64 x 64, n = 8, dilation 12: 162 -> 146 (528 TFLOP/s)
//   fp32  512 -> 512, 30 x 40, n = 8: 968 -> 636 (142 TFLOP/s)     128 -> 128, 28 x 28, n = 32: 177 -> 114 (130 TFLOP/s)
//         256 -> 512, 14 x 14, n = 4, stride 2: 132 -> 52
// (fp32 sums every 16 or 32 k from zero and changes the sign from chunk to chunk, see mul_all: 2 - 8 % of these times.)
// bf16 layers of kernels larger than 1 x 1 with enough channels take the same three steps on staged operands (sgemm_k, below).
#include "gf_gemm.h"

#include <algorithm>
#include <numeric>

namespace gf {

namespace {

constexpr double kPlainWgradMinFlops = 6e9;  // below, the tiles of the merged filtered launch are faster

// AND words of an element mask (bit e keeps element e)
template <class T>
__device__ __forceinline__ u32x4_t bit_mask(uint32_t m) {
  u32x4_t w;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (sizeof(T) == 4) {
      w[i] = (uint32_t)((int)(m << (31 - i)) >> 31);
    } else {
      const uint32_t lo = (uint32_t)((int)(m << (31 - 2 * i)) >> 31), hi = (uint32_t)((int)(m << (30 - 2 * i)) >> 31);
      w[i] = (lo & 0xffffu) | (hi & 0xffff0000u);
    }
  }
  return w;
}

// mask bits of the vector that starts at pixel q (a multiple of VE) from the table byte of its group of eight pixels
template <class T>
__device__ __forceinline__ uint32_t vec_mask(uint32_t byte, int q) {
  return sizeof(T) == 2 ? byte : (byte >> (q & 4)) & 0xfu;
}

// ---------------------------------------------------------------------------
// Set-up.  With e = u d - p, f = v d - p (tap offsets on the input side) and, for stride s,
// a = e mod s, b = f mod s (the phase plane the tap reads), Hq = ceil(H / s), Wq = W_y:
//   tapw[t]        = phase(a, b) * N Ci Hq Wq + floor(e / s) * Wq + floor(f / s)
//   tabw[t][k / 8] bit i: output pixel k + i exists and tap t of it reads inside the image
//   per phase ph = (a, b) of g_x, the taps with (a + p - u d) and (b + p - v d) divisible by s:
//   tapd[ph][kk]   = {t, ((a + p - u d) / s) * W_y + (b + p - v d) / s},  ntap[ph] of them
//   tabd[ph][t][j / 8] bit i: position j + i of the phase plane exists and that tap reaches it
//                             from an output pixel inside the map
// ---------------------------------------------------------------------------
struct PrepArgs {
  uint8_t* tabw;
  uint8_t* tabd;
  int* tapw;    // [KK]
  int2* tapd;   // [s*s][KK]
  int* ntap;    // [s*s]
  int N, Ci, H, W, Hy, Wy, Hq, Wq, Kw, KK, s, d, p, nvw, nvd;
  int* tickets;   // zeroed for the slab sums of the input gradient
  int ntickets;
};

__device__ __forceinline__ int floor_div(int a, int b) { return (a >= 0) ? a / b : -((-a + b - 1) / b); }

__device__ __forceinline__ void prep_tables(const PrepArgs& a, int block) {
  const int e0 = block * kT + threadIdx.x;
  const int nph = a.s * a.s;
  const int nmax = a.nvw > a.nvd * nph ? a.nvw : a.nvd * nph;
  if (block == 0 && (int)threadIdx.x < nph) {  // tap list of one phase of g_x
    const int ph = threadIdx.x, pa = ph / a.s, pb = ph - pa * a.s;
    int cnt = 0;
    for (int t = 0; t < a.KK; ++t) {
      const int u = t / a.Kw, v = t - u * a.Kw;
      const int ea = pa + a.p - u * a.d, eb = pb + a.p - v * a.d;
      const int qa = floor_div(ea, a.s), qb = floor_div(eb, a.s);
      if (qa * a.s == ea && qb * a.s == eb) a.tapd[ph * a.KK + cnt++] = make_int2(t, qa * a.Wy + qb);
    }
    a.ntap[ph] = cnt;
  }
  if (e0 < a.ntickets) a.tickets[e0] = 0;
  if (e0 >= a.KK * nmax) return;
  const int t = e0 / nmax, g = e0 - t * nmax;
  const int u = t / a.Kw, v = t - u * a.Kw;
  const int e = u * a.d - a.p, f = v * a.d - a.p;
  if (g == 0) {
    const int qe = floor_div(e, a.s), qf = floor_div(f, a.s);
    const int ph = (e - qe * a.s) * a.s + (f - qf * a.s);
    a.tapw[t] = ph * (a.N * a.Ci * a.Hq * a.Wq) + qe * a.Wq + qf;
  }
  if (g < a.nvw) {
    uint32_t m = 0;
    for (int i = 0; i < 8; ++i) {
      const int k = g * 8 + i;
      if (k >= a.Hy * a.Wy) break;
      const int hy = k / a.Wy, wy = k - hy * a.Wy;
      const int hs = hy * a.s + e, ws = wy * a.s + f;
      if (hs >= 0 && hs < a.H && ws >= 0 && ws < a.W) m |= 1u << i;
    }
    a.tabw[t * a.nvw + g] = (uint8_t)m;
  }
  if (g < a.nvd * nph) {
    const int ph = g / a.nvd, gg = g - ph * a.nvd;
    const int pa = ph / a.s, pb = ph - pa * a.s;
    const int ea = pa + a.p - u * a.d, eb = pb + a.p - v * a.d;
    const int qa = floor_div(ea, a.s), qb = floor_div(eb, a.s);
    uint32_t m = 0;
    if (qa * a.s == ea && qb * a.s == eb) {
      for (int i = 0; i < 8; ++i) {
        const int j = gg * 8 + i;
        if (j >= a.Hq * a.Wq) break;
        const int h = j / a.Wq, w = j - h * a.Wq;
        const int hs = h + qa, ws = w + qb;
        if (hs >= 0 && hs < a.Hy && ws >= 0 && ws < a.Wy) m |= 1u << i;
      }
    }
    a.tabd[(ph * a.KK + t) * a.nvd + gg] = (uint8_t)m;
  }
}

// One set-up launch.  Blocks [0, tab_blocks): tables and tap lists.  Then w_blocks blocks write the kernel tap-major
// with rows of c_i padded to whole vectors (zeros), wt[(t Co + co) Cip + ci] = w[(co Ci + ci) KK + t] (input gradient
// only): a block takes kWPairs consecutive c_i of one c_o, one contiguous run of w, through LDS.  Then the phase
// planes of x (weight gradient of a strided layer only), a vector per lane.
constexpr int kWPairs = 128;
constexpr int kWTaps = 16;   // taps a pass of a block holds in LDS

template <class T>
__global__ __launch_bounds__(kT) void prep_k(PrepArgs a, int tab_blocks, int w_blocks, const T* w, T* wt, int Co, int Cip,
                                             const T* x, T* xq) {
  int b = blockIdx.x;
  const int tid = threadIdx.x;
  if (b < tab_blocks) {
    prep_tables(a, b);
    return;
  }
  b -= tab_blocks;
  if (b < w_blocks) {
    __shared__ T run[kWPairs * (kWTaps + 1)];
    const int per_co = (Cip + kWPairs - 1) / kWPairs;
    const int co = b / per_co, ci0 = (b - co * per_co) * kWPairs;
    const int nc = min(kWPairs, a.Ci - ci0), ncp = min(kWPairs, Cip - ci0);
    const T* src = w + ((long)co * a.Ci + ci0) * a.KK;
    for (int t0 = 0; t0 < a.KK; t0 += kWTaps) {
      const int nt = min(kWTaps, a.KK - t0);
      if (t0) __syncthreads();
      const int total = nc * nt;
      for (int e0 = tid; e0 < total; e0 += 4 * kT) {   // four loads in flight
        T v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int e = min(e0 + k * kT, total - 1);
          const int c = e / nt, t = e - c * nt;
          v[k] = src[c * a.KK + t0 + t];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int e = e0 + k * kT;
          if (e < total) {
            const int c = e / nt, t = e - c * nt;
            run[t * (kWPairs + 8) + c] = v[k];
          }
        }
      }
      __syncthreads();
      for (int e = tid; e < nt * ncp; e += kT) {
        const int t = e / ncp, c = e - t * ncp;
        wt[((long)(t0 + t) * Co + co) * Cip + ci0 + c] = c < nc ? run[t * (kWPairs + 8) + c] : from_f32<T>(0.f);
      }
    }
    return;
  }
  b -= w_blocks;
  // phase planes: plane = (ph * N + n) * Ci + ci of PQ elements each, as one flat stream
  constexpr int VE = El<T>::VE;
  const int PQ = a.Hq * a.Wq;
  const int total = a.s * a.s * a.N * a.Ci * PQ;
  const int e0 = (b * kT + tid) * VE;
  if (e0 >= total) return;
  const int plane = e0 / PQ, pos = e0 - plane * PQ;
  int i = pos / a.Wq, j = pos - i * a.Wq;
  int ph = plane / (a.N * a.Ci), nc = plane - ph * (a.N * a.Ci);
  int pa = ph / a.s, pb = ph - pa * a.s;
  T v[VE];
  int idx[VE];
#pragma unroll
  for (int k = 0; k < VE; ++k) {
    const int h = i * a.s + pa, ww = j * a.s + pb;
    idx[k] = (e0 + k < total && h < a.H && ww < a.W) ? (nc * a.H + h) * a.W + ww : -1;
    if (++j == a.Wq) {
      j = 0;
      if (++i == a.Hq) {
        i = 0;
        if (++nc == a.N * a.Ci) {
          nc = 0;
          if (++pb == a.s) { pb = 0; ++pa; }
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < VE; ++k) v[k] = x[max(idx[k], 0)];
#pragma unroll
  for (int k = 0; k < VE; ++k) v[k] = idx[k] >= 0 ? v[k] : from_f32<T>(0.f);
  if (e0 + VE <= total) {
    __attribute__((aligned(16))) T o[VE];
#pragma unroll
    for (int k = 0; k < VE; ++k) o[k] = v[k];
    *reinterpret_cast<uint4*>(xq + e0) = *reinterpret_cast<const uint4*>(o);
  } else {
    for (int k = 0; e0 + k < total; ++k) xq[e0 + k] = v[k];
  }
}

// ---------------------------------------------------------------------------
// both products
// ---------------------------------------------------------------------------
constexpr int kTapsLds = 128;

struct XArgs {
  int N, Ci, Co, KK;
  const void* gy;
  int HWy, tot_gy;        // plane of g_y, elements
  // weight gradient: part[z][t][co][ci] = sum over the K chunks of slab z
  const void* x;          // x, or its phase planes
  float* part;
  const uint8_t* tabw;    // null: plain contraction of two maps of the same size
  const int* tapw;        // per tap: offset of the element of the x operand that output pixel 0 reads
  int HW, tot_x;          // plane of the x operand (a phase plane for strided layers)
  int qv, kvecs, nvw;     // vectors per padded plane of g_y, N * qv, table bytes per tap
  int nchunks, cpz, nz, tx, tiles, R, xcd_slabs, nW;
  // input gradient
  const void* wt;         // [KK][Co][Cip]
  void* gx;               // g_x, or its phase planes [s*s][N][Ci][PQ]
  const uint8_t* tabd;
  const int2* tapd;       // [phase][KK]: {tap, offset of the g_y element that position 0 reads}
  const int* ntap;        // [phase]
  int Cip, PQ, qd, nvd;   // padded c_i, plane of the output, vectors per padded plane, table bytes per tap and phase
  int d_tm, d_tn, nck, nD;
  int d_nz, d_its, d_grp, d_ngrp;   // K slabs of a tile, steps (tap, chunk) per slab, grouping of the slab sum
  float* partD;
  int* tickD;
  int d_first;            // the input-gradient blocks lead the grid
  FastDiv d_qv, d_qd, d_r, d_tiles, d_tx;
  // staged operands (stage_k): rows of 32 channels, one per pixel of g_y / x and one of zeros at the end
  const void* gt;         // [Cop / 32][N PY + 1][32]
  const void* xt;         // [Cix / 32][N H W + 1][32]
  const void* wr;         // [KK][Cop / 32][Ci][32]
  const int4* taps;       // [phase][KK]: {tap, row and column offset of the g_y pixel that position 0 reads}
  int Cop, Cix, H, W, Hy, Wy, Wq, Kw, s, d, p;
  FastDiv d_py, d_wy, d_wq;
};

template <class T, int TM, int TN>
struct XTile {
  static constexpr bool SPLIT = is_split<T>();
  static constexpr int TERMS = terms_of<T>();
  static constexpr int KB = El<T>::KB, VE = El<T>::VE;
  static constexpr int BM = 64 * TM, BN = 64 * TN;
  static constexpr int RW = SPLIT ? 64 + 16 : 128 + 16;   // weight gradient: bytes of one K-major row of a term
  static constexpr int WA = BM * RW, WB = BN * RW;
  static constexpr int DA = KB * BM * El<T>::EB, DB = KB * BN * El<T>::EB;  // input gradient: [k][columns]
  static constexpr int kW = TERMS * (WA + WB), kD = TERMS * (DA + DB);
  static constexpr int SC = BN + VE;                        // element stride of the staged result
  static constexpr int kE = 64 * SC * (int)sizeof(T);
  static constexpr int kOp = kW > kD ? kW : kD;
  static constexpr int kBytes = kOp > kE ? kOp : kE;
};

// One register set.  oa / ob: what this lane's offsets started from; off: a load had to be moved into its tensor;
// keep: elements of the vector inside the plane of g_y; mb: table byte of the shifted operand; k0: first row of k
// (weight gradient: pixel of the vector).  Nothing here is computed from a load before stage(): that would wait for it.
template <int LA, int LB>
struct XSet {
  u32x4_t a[LA], b[LB];
  int oa, ob, off, keep, k0;
  uint32_t mb;
};

// register sets of the K loop
template <class T, int TM, int TN> constexpr int xsets_of() { return TM * TN == 1 && !__is_same(T, raw_f32) ? 4 : 2; }

// acc += g_y[rows m0 ..][chunk] * x[rows n0 .., moved by the tap][chunk]^T over the chunks of a K slab
template <class T, int TM, int TN>
__device__ __forceinline__ void xw_mainloop(const XArgs& a, int t, int m0, int n0, int kc0, int kc1, unsigned char* smem,
                                            f32x16 (&acc)[TM][TN], uint32_t& low) {
  using X = XTile<T, TM, TN>;
  constexpr int VE = X::VE, LA = 2 * TM, LB = 2 * TN;
  typedef XSet<LA, LB> Set;
  const int delta = a.tapw ? a.tapw[t] : 0;
  unsigned char* As = smem;
  unsigned char* Bs = smem + X::TERMS * X::WA;
  const T* gy = static_cast<const T*>(a.gy);
  const T* x = static_cast<const T*>(a.x);
  const int tid = lane_id<T>(), lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int vi = tid & 7, row0 = tid >> 3;   // this lane's vector of the chunk, first row
  int rowa[LA], rowb[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) rowa[i] = min(m0 + row0 + 32 * i, a.Co - 1) * a.HWy;
#pragma unroll
  for (int i = 0; i < LB; ++i) rowb[i] = min(n0 + row0 + 32 * i, a.Ci - 1) * a.HW + delta;
  const int cop = a.Co * a.HWy, cip = a.Ci * a.HW;
  const int hi_a = a.tot_gy - VE, hi_b = a.tot_x - VE;
  const uint8_t* tab = a.tabw ? a.tabw + (long)t * a.nvw : nullptr;
  // this lane's position in K (see w_mainloop in gf_dense.hip)
  const int dn = (int)a.d_qv.div(8u), dpv = 8 - dn * a.qv;
  int kv = kc0 * 8 + vi;
  int n = (int)a.d_qv.div((uint32_t)min(kv, a.kvecs - 1));
  int pv = min(kv, a.kvecs - 1) - n * a.qv;
  auto fetch = [&](Set& s, int kc) __attribute__((always_inline)) {
    const int q = pv * VE;
    s.oa = n * cop + q; s.ob = n * cip + q; s.off = 0;
    s.keep = kv < a.kvecs ? a.HWy - q : 0;
    s.mb = tab ? tab[q >> 3] : 0xffu;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int o = s.oa + rowa[i], oc = min(o, hi_a);
      s.off |= o ^ oc;
      s.a[i] = load16<T, true>(gy + oc);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int o = s.ob + rowb[i], oc = min(max(o, 0), hi_b);
      s.off |= o ^ oc;
      s.b[i] = load16<T, true>(x + oc);
    }
    s.k0 = q;
    if (kc + 1 < kc1) {   // (uniform)
      kv += 8;
      n += dn; pv += dpv;
      if (pv >= a.qv) { pv -= a.qv; ++n; }
      if (kv >= a.kvecs) { n = a.N - 1; pv = a.qv - 1; }   // past the last image: its last vector, masked
    }
  };
  auto stage = [&](Set& s, int, auto neg) __attribute__((always_inline)) {
    if (s.off) {   // first or last rows of the tensors only: shift the moved vectors back
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int o = s.oa + rowa[i];
        s.a[i] = shifted<T>(s.a[i], min(o - min(o, hi_a), VE));
      }
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int o = s.ob + rowb[i];
        s.b[i] = shifted<T>(s.b[i], min(max(o - min(max(o, 0), hi_b), -VE), VE));
      }
    }
    // both operands: what the tap does not read must not meet an infinity on the other side either
    const u32x4_t m = keep_mask<T>(s.keep) & bit_mask<T>(vec_mask<T>(s.mb, s.k0));
    auto put = [&](unsigned char* tile, int term_bytes, int row, const u32x4_t& v, auto sign) __attribute__((always_inline)) {
      if constexpr (X::SPLIT) {
        uint2 w[3];
        split3<decltype(sign)::value>(v, w, low);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(tile + k * term_bytes + row * X::RW + vi * 8) = w[k];
      } else {
        *reinterpret_cast<u32x4_t*>(tile + row * X::RW + vi * 16) = v;
      }
    };
#pragma unroll
    for (int i = 0; i < LA; ++i) put(As, X::WA, row0 + 32 * i, s.a[i] & m, neg);
#pragma unroll
    for (int i = 0; i < LB; ++i) put(Bs, X::WB, row0 + 32 * i, s.b[i] & m, std::false_type());
  };
  auto mul = [&](auto neg) __attribute__((always_inline)) {
    typename El<T>::acc s;
    const int r = lane & 31, kg = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < El<T>::KS; ++ks) {
      uint4 fa[TM][X::TERMS], fb[TN][X::TERMS];
#pragma unroll
      for (int u = 0; u < X::TERMS; ++u) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          fa[i][u] = *reinterpret_cast<const uint4*>(As + u * X::WA + (64 * i + 32 * wm + r) * X::RW + ks * 32 + kg * 16);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          fb[j][u] = *reinterpret_cast<const uint4*>(Bs + u * X::WB + (64 * j + 32 * wn + r) * X::RW + ks * 32 + kg * 16);
      }
      mul_all<T, decltype(neg)::value>(fa, fb, acc, s, ks);
    }
  };
  k_loop<xsets_of<T, TM, TN>(), Set>(kc0, kc1, fetch, stage, mul);
}

// ---------------------------------------------------------------------------
// Staged operands (bf16, kernels larger than 1 x 1).  stage_k writes g_y, x and the kernel once more in planes of 32
// channels, channels innermost, so that every 16 bytes a tap reads are aligned and whole: no masks -- a pixel outside the image
// is the row of zeros -- and the loads go straight to LDS (global_load_lds_dwordx4), four buffers of 32 k, a barrier per buffer.
//   weight gradient: K = pixels; both operands are rows of k = pixel and go through the transposing reads
//   input gradient:  K = (tap, c_o); both operands are K-major rows of 32 c_o
// xgemm_k on the same maps spends its steps on masks, unaligned loads and the way through registers into LDS, and splits each
// image's planes of 8 ceil(HW / 8) pixels; here a step is loads, transposing or plain reads of LDS and matrix instructions, of
// which none alone bounds it (256 -> 256, 14 x 14, n = 64: 54 us; with the matrix instructions left out 39, with the loads 49).
// Both gradients, xgemm_k / staged, whole call (us, three rotating sets; the staging launch 6 - 8 of it, prep_k took 7 - 11):
//   256 -> 256, 14 x 14, n = 64: 74 / 54    512 -> 512, 7 x 7: 81 / 57    256 -> 512, stride 2: 63 / 46
//   64 -> 64, 8 x 8, n = 1: 18 / 14    256 -> 256, 60 x 80, n = 8: 176 / 124; 64 x 64, dilation 12: 148 / 117
//   512 -> 512, 32 x 32, n = 8: 160 / 112    5 x 5, 64 -> 64, 56 x 56, n = 16: 81 / 59
//   128 -> 256, 60 x 80, n = 128: 1131 / 935    512 -> 512, 30 x 40, n = 128: 2240 / 1652 (1.03 PFLOP/s)
// Also timed, first layer above: four waves of 64 x 64 and two buffers of 64 k 54.6 (the three first layers 55 / 48 / 59, with
// eight waves 55 / 45 / 56), 128 x 64 tiles 70, the operands of step k + 1 read during step k 55.
// ---------------------------------------------------------------------------
struct StageJob {   // src [N][C][PX] -> dst [Cp / 32][N PX + 1][32], channels past C and the last row zero; kernel: see stage_k
  const void* src;
  void* dst;
  int N, C, PX, Cp, pb, cb, blocks;   // blocks of 64 pixels per image, of 64 channels, all
};
struct StageArgs {
  StageJob job[3];
  int4* taps;
  int* ntap;
  int* tickets;
  int ntickets, KK, Kw, s, d, p;
};

// A block transposes 64 channels x 64 pixels: a lane loads eight pixels of two channels and writes eight channel pairs, in an
// order of 16-byte units within a pixel's row that spreads them over the banks.
__global__ __launch_bounds__(kT) void stage_k(StageArgs a) {
  __shared__ __attribute__((aligned(16))) uint32_t tile[64 * 32];
  int b = blockIdx.x;
  const int tid = threadIdx.x;
  if (b == 0) {   // tap lists of the phases, tickets, rows of zeros
    const int nph = a.s * a.s;
    if (a.taps && tid < nph) {
      const int pa = tid / a.s, pb = tid - pa * a.s;
      int cnt = 0;
      for (int t = 0; t < a.KK; ++t) {
        const int u = t / a.Kw, v = t - u * a.Kw;
        const int ea = pa + a.p - u * a.d, eb = pb + a.p - v * a.d;
        const int qa = floor_div(ea, a.s), qb = floor_div(eb, a.s);
        if (qa * a.s == ea && qb * a.s == eb) a.taps[tid * a.KK + cnt++] = make_int4(t, qa, qb, 0);
      }
      a.ntap[tid] = cnt;
    }
    for (int i = tid; i < a.ntickets; i += kT) a.tickets[i] = 0;
    for (int j = 0; j < 3; ++j) {
      const StageJob& q = a.job[j];
      if (!q.blocks) continue;
      uint32_t* z = static_cast<uint32_t*>(q.dst);
      const long rows = (long)q.N * q.PX + 1;
      if (j < 2)
        for (int i = tid; i < q.Cp / 2; i += kT) z[((i >> 4) * rows + rows - 1) * 16 + (i & 15)] = 0;
    }
    return;
  }
  b -= 1;
  int j = 0;
  while (j < 2 && b >= a.job[j].blocks) b -= a.job[j++].blocks;   // (uniform)
  const StageJob q = a.job[j];
  const int c64 = b % q.cb, rest = b / q.cb;
  const int n = rest / q.pb, p0 = (rest - n * q.pb) * 64;
  const int pv = tid & 7, cp = tid >> 3;   // eight pixels, channel pair
  const int px = p0 + pv * 8, c = c64 * 64 + cp * 2;
  const bf16_t* src = static_cast<const bf16_t*>(q.src);
  uint32_t v[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bf16_t* s = src + ((long)n * q.C + min(c + h, q.C - 1)) * q.PX;
    if (px + 8 <= q.PX) {
      const uint4 w = load_vec<bf16_t>(s + px);
      v[h][0] = w.x; v[h][1] = w.y; v[h][2] = w.z; v[h][3] = w.w;
    } else {
      uint16_t e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = __builtin_bit_cast(uint16_t, s[min(px + i, q.PX - 1)]);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[h][i] = (uint32_t)e[2 * i] | ((uint32_t)e[2 * i + 1] << 16);
    }
    if (c + h >= q.C)
#pragma unroll
      for (int i = 0; i < 4; ++i) v[h][i] = 0;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t lo = v[0][i >> 1] >> (16 * (i & 1)) & 0xffffu, hi = v[1][i >> 1] >> (16 * (i & 1)) & 0xffffu;
    tile[(pv * 8 + i) * 32 + (((cp >> 2) ^ pv) << 2 | (cp & 3))] = lo | hi << 16;
  }
  __syncthreads();
  bf16_t* dst = static_cast<bf16_t*>(q.dst);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = i * 32 + (tid >> 3), un = tid & 7;
    if (p0 + r >= q.PX) continue;
    const int plane = c64 * 2 + (un >> 2);
    long row;
    if (j < 2) {
      row = plane * ((long)q.N * q.PX + 1) + (long)n * q.PX + p0 + r;
    } else {   // "pixels" are (c_i, tap): [tap][c_o / 32][c_i][32]
      const int ci = (p0 + r) / a.KK, t = p0 + r - ci * a.KK;
      row = ((long)t * (q.Cp >> 5) + plane) * (q.PX / a.KK) + ci;
    }
    const uint4 u = *reinterpret_cast<const uint4*>(tile + r * 32 + ((un ^ (r >> 3)) << 2));
    *reinterpret_cast<uint4*>(dst + row * 32 + (un & 3) * 8) = u;
  }
}

// 16 bytes per lane from base + off to LDS, lane i to lds + 16 i (both uniform).  Behind the compiler's back: it would wait for
// every such load at the next read of LDS; the loops below wait themselves.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (m0 is reserved: the compiler sets it where an instruction needs it, and must do so again after this)
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ uint32_t lds_of(const unsigned char* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const unsigned char*)p;
}
// Block tile of 64 TM x 64 TN, NT lanes: waves of 32 x 32 TNW, WN of them side by side.  Eight waves on the largest tile: their
// address arithmetic and reads of LDS hide behind each other's matrix instructions (four waves of 64 x 64: one per SIMD and
// block, 1100 clocks for a step of 256 clocks of matrix instructions).
template <int TM, int TN>
struct STile {
  static constexpr int BM = 64 * TM, BN = 64 * TN;
  static constexpr int NT = TM * TN == 4 ? 512 : 256;
  static constexpr int WN = TM > TN ? 1 : 2, TNW = BN / (32 * WN);
  static constexpr int A = 4096 * TM, B = 4096 * TN, kStage = A + B;   // a buffer of 32 k
  static constexpr int LA = A / (16 * NT), LB = B / (16 * NT);         // 16-byte loads of a lane
  static constexpr int SC = BN + 8;                                     // element stride of the staged result
  static constexpr int kOp = 4 * kStage, kE = BM * SC * 2;
  static constexpr int kBytes = kOp > kE ? kOp : kE;
  static_assert(BM == 32 * (NT / 64 / WN), "the waves cover the tile");
  static_assert(kOp <= 65536, "16-bit LDS addresses of the loads");
};

// Steps [0, n) of 32 k through four buffers: three are on their way or read while the fourth is filled.  A step waits until this
// wave's loads of its buffer have landed (those of at most two later buffers are still out) and its reads of the last one
// are done; after the barrier the same holds for all waves.  The operands are read before the next loads are issued (their
// address arithmetic then covers the latency of LDS).
template <int LOADS, class F, class R, class M>
__device__ __forceinline__ void stage_loop(int n, F&& fetch, R&& read, M&& mul) {
  fetch(0);
  if (n > 1) fetch(1);   // (uniform)
  if (n > 2) fetch(2);
  for (int k = 0; k < n; ++k) {
    if (k + 2 < n) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LOADS) : "memory");
    else if (k + 1 < n) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    read(k & 3);
    if (k + 3 < n) fetch(k + 3 & 3);
    mul();
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The operand of one MFMA from a plane of 32 k x 32 channels -- lane: channel lane % 32, k = 16 ks + 8 (lane / 32) .. + 7 --
// with transposing reads (see frag_tr); four rows of 64 bytes are read together, all banks once.
__device__ __forceinline__ uint4 frag_plane(const unsigned char* plane, int ks, int lane) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const unsigned char* p = plane + (ks * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2)) * 64 + (lane & 16) * 2 + 8 * (lane & 3);
  const uint2 a = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
  const uint2 b = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * 64)));
  return make_uint4(a.x, a.y, b.x, b.y);
}

// A pixel of g_y in a walk over all pixels in steps of 32, and the row of x under a tap, by additions only.
struct PixelWalk {
  int q, hs, ws, xr;   // pixel; row and column of x; row of the staged x
};

// acc += g_y[pixels][c_o]^T * x[pixels moved by tap t][c_i] over the chunks of 64 pixels of a K slab
template <int TM, int TN>
__device__ __forceinline__ void sw_mainloop(const XArgs& a, int t, int m0, int n0, int kc0, int kc1, unsigned char* smem,
                                            f32x16 (&acc)[1][STile<TM, TN>::TNW]) {
  using S = STile<TM, TN>;
  constexpr int LA = S::LA, LB = S::LB;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WN, wn = wave % S::WN;
  const int u = t / a.Kw, e = u * a.d - a.p, f = (t - u * a.Kw) * a.d - a.p;
  const int K = a.N * a.HWy, zg = K, zx = a.N * a.H * a.W;
  // LDS: planes of 32 channels x 32 k; all of a lane's loads lie in row tid / 4 % 32, planes tid / 128 + (NT / 128) i
  uint32_t ca[LA], cb[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i)
    ca[i] = (uint32_t)min(m0 / 32 + (tid >> 7) + S::NT / 128 * i, a.Cop / 32 - 1) * (uint32_t)(zg + 1) * 64u + (tid & 3) * 16;
#pragma unroll
  for (int i = 0; i < LB; ++i)
    cb[i] = (uint32_t)min(n0 / 32 + (tid >> 7) + S::NT / 128 * i, a.Cix / 32 - 1) * (uint32_t)(zx + 1) * 64u + (tid & 3) * 16;
  const uint32_t lds0 = lds_of(smem) + wave * 1024;
  // 32 pixels on: dh rows and dw columns (and dn images), then the wraps
  const int dn = (int)a.d_py.div(32u), dr = 32 - dn * a.HWy, dh = (int)a.d_wy.div((uint32_t)dr), dw = dr - dh * a.Wy;
  const int step_x = (dn * a.H + dh * a.s) * a.W + dw * a.s, wrap_w = a.s * (a.W - a.Wy), wrap_h = (a.H - a.Hy * a.s) * a.W;
  const int end_w = a.Wy * a.s + f, end_h = a.Hy * a.s + e;
  PixelWalk p;
  {
    p.q = kc0 * 64 + (tid >> 2 & 31);
    const int n = (int)a.d_py.div((uint32_t)p.q), r = p.q - n * a.HWy;
    const int h = (int)a.d_wy.div((uint32_t)r), w = r - h * a.Wy;
    p.hs = h * a.s + e; p.ws = w * a.s + f;
    p.xr = (n * a.H + p.hs) * a.W + p.ws;
  }
  auto fetch = [&](int buf) __attribute__((always_inline)) {
    const uint32_t lds = lds0 + buf * S::kStage;
    const bool ok = p.q < K && (uint32_t)p.hs < (uint32_t)a.H && (uint32_t)p.ws < (uint32_t)a.W;
    const uint32_t g = (uint32_t)(ok ? p.q : zg) * 64u, x = (uint32_t)(ok ? p.xr : zx) * 64u;
#pragma unroll
    for (int i = 0; i < LA; ++i) dma16(a.gt, g + ca[i], lds + i * (16 * S::NT));
#pragma unroll
    for (int i = 0; i < LB; ++i) dma16(a.xt, x + cb[i], lds + S::A + i * (16 * S::NT));
    p.q += 32; p.ws += dw * a.s; p.hs += dh * a.s; p.xr += step_x;
    if (p.ws >= end_w) { p.ws -= a.Wy * a.s; p.hs += a.s; p.xr += wrap_w; }
    if (p.hs >= end_h) { p.hs -= a.Hy * a.s; p.xr += wrap_h; }
  };
  uint4 fa[2], fb[2][S::TNW];
  auto read = [&](int buf) __attribute__((always_inline)) {
    const unsigned char* As = smem + buf * S::kStage;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      fa[ks] = frag_plane(As + wm * 2048, ks, lane);
#pragma unroll
      for (int j = 0; j < S::TNW; ++j) fb[ks][j] = frag_plane(As + S::A + (S::WN * j + wn) * 2048, ks, lane);
    }
  };
  auto mul = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < S::TNW; ++j) acc[0][j] = mma32(fa[ks], fb[ks][j], acc[0][j]);
  };
  stage_loop<LA + LB>(2 * (kc1 - kc0), fetch, read, mul);
}

// acc += w[rows m0 ..][steps] * g_y[columns of the tile, moved by the tap][steps]^T over steps (tap of the phase, 64 c_o)
template <int TM, int TN>
__device__ __forceinline__ void sd_mainloop(const XArgs& a, int m0, int tni, int it0, int iters, unsigned char* smem,
                                            const int4* taps, f32x16 (&acc)[1][STile<TM, TN>::TNW]) {
  using S = STile<TM, TN>;
  constexpr int LA = S::LA, LB = S::LB, RP = S::NT / 4;   // RP: rows between a lane's loads
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WN, wn = wave % S::WN;
  const int row0 = tid >> 2;                                  // rows row0 + RP i
  const uint32_t unit = 16 * ((tid & 3) ^ (row0 >> 2 & 3));   // the lane's 16 bytes of the 64 of a row
  const uint32_t lds0 = lds_of(smem) + wave * 1024;
  const int zg = a.N * a.HWy, np = a.Cop >> 5;                // planes of 32 c_o
  uint32_t offa[LA], offb[LB];
  int ph[LB], pw[LB], pn[LB];   // pixel of a column
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int jp = tni * S::BN + row0 + RP * i;
    const int n = (int)a.d_qd.div((uint32_t)(jp >> 3)), q = jp - n * a.qd * 8;
    ph[i] = (int)a.d_wq.div((uint32_t)q);
    pw[i] = q - ph[i] * a.Wq;
    pn[i] = n < a.N && q < a.PQ ? n * a.Hy : -1;
  }
  int kk = 2 * it0 / np, kc = 2 * it0 - kk * np;   // tap of the list and plane the next fetch takes
  bool new_tap = true;
  auto fetch = [&](int buf) __attribute__((always_inline)) {
    if (new_tap) {   // (uniform)
      const int t = __builtin_amdgcn_readfirstlane(taps[kk].x), qa = __builtin_amdgcn_readfirstlane(taps[kk].y);
      const int qb = __builtin_amdgcn_readfirstlane(taps[kk].z);
#pragma unroll
      for (int i = 0; i < LA; ++i) offa[i] = (uint32_t)(t * np * a.Ci + min(m0 + row0 + RP * i, a.Ci - 1)) * 64u + unit;
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int h = ph[i] + qa, w = pw[i] + qb;
        const bool ok = pn[i] >= 0 && (uint32_t)h < (uint32_t)a.Hy && (uint32_t)w < (uint32_t)a.Wy;
        offb[i] = (uint32_t)(ok ? (pn[i] + h) * a.Wy + w : zg) * 64u + unit;
      }
    }
    const uint32_t lds = lds0 + buf * S::kStage;
    const uint32_t ka = (uint32_t)(kc * a.Ci) * 64u, kb = (uint32_t)kc * (uint32_t)(zg + 1) * 64u;
#pragma unroll
    for (int i = 0; i < LA; ++i) dma16(a.wr, offa[i] + ka, lds + i * (16 * S::NT));
#pragma unroll
    for (int i = 0; i < LB; ++i) dma16(a.gt, offb[i] + kb, lds + S::A + i * (16 * S::NT));
    new_tap = ++kc == np;
    if (new_tap) { kc = 0; ++kk; }
  };
  uint4 fa[2], fb[2][S::TNW];
  auto read = [&](int buf) __attribute__((always_inline)) {
    const unsigned char* As = smem + buf * S::kStage;
    const int r = lane & 31, kg = lane >> 5, x = r >> 2 & 3;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int o = r * 64 + ((2 * ks + kg) ^ x) * 16;
      fa[ks] = *reinterpret_cast<const uint4*>(As + 32 * wm * 64 + o);
#pragma unroll
      for (int j = 0; j < S::TNW; ++j) fb[ks][j] = *reinterpret_cast<const uint4*>(As + S::A + 32 * (S::WN * j + wn) * 64 + o);
    }
  };
  auto mul = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < S::TNW; ++j) acc[0][j] = mma32(fa[ks], fb[ks][j], acc[0][j]);
  };
  stage_loop<LA + LB>(2 * (iters - it0), fetch, read, mul);
}

// weight-gradient block L: K slab, tap and tile (see xwgrad_block)
struct WTileAt {
  int z, t, m0, n0;
};
__device__ __forceinline__ WTileAt wtile_at(const XArgs& a, int L, int bm, int bn) {
  WTileAt w;
  int rest;
  // The hardware hands consecutive blocks to the eight XCDs in turn; with eight or more K slabs block L works on
  // slab (L % 8) + 8 * (..), so that all taps and tiles of a slab share one XCD's L2 and each XCD touches an eighth
  // of x and g_y.
  if (a.xcd_slabs) {
    const int idx = L >> 3;
    const int zl = (int)a.d_r.div((uint32_t)idx);
    w.z = (L & 7) + 8 * zl;
    rest = idx - zl * a.R;
  } else {
    w.z = (int)a.d_r.div((uint32_t)L);
    rest = L - w.z * a.R;
  }
  w.t = (int)a.d_tiles.div((uint32_t)rest);
  const int tile = rest - w.t * a.tiles;
  const int by = (int)a.d_tx.div((uint32_t)tile), bx = tile - by * a.tx;
  w.m0 = by * bm;
  w.n0 = bx * bn;
  return w;
}

template <int TM, int TN>
__global__ __launch_bounds__((STile<TM, TN>::NT), 4) void sgemm_k(XArgs a) {
  using S = STile<TM, TN>;
  struct Lds {   // (the operands first: the loads address the first 64 KB)
    __attribute__((aligned(16))) unsigned char op[S::kBytes];
    int4 taps[kTapsLds];
    int flag;
  };
  __shared__ Lds lds;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / S::WN, wn = wave % S::WN;
  f32x16 acc[1][S::TNW];
  zero_acc(acc);
  int L = blockIdx.x;
  if (a.d_first ? L >= a.nD : L < a.nW) {
    if (a.d_first) L -= a.nD;
    const WTileAt w = wtile_at(a, L, S::BM, S::BN);
    if (w.z >= a.nz) return;   // (uniform)
    sw_mainloop<TM, TN>(a, w.t, w.m0, w.n0, w.z * a.cpz, min(w.z * a.cpz + a.cpz, a.nchunks), lds.op, acc);
    float* dst = a.part + ((long)w.z * a.KK + w.t) * a.Co * a.Ci;
#pragma unroll
    for (int j = 0; j < S::TNW; ++j) {
      const int ci = w.n0 + 32 * (S::WN * j + wn) + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int co = w.m0 + 32 * wm + acc_row(lane, v);
        if (co < a.Co && ci < a.Ci) dst[(long)co * a.Ci + ci] = acc[0][j][v];
      }
    }
    return;
  }
  // input gradient: rows c_i of one column tile (positions of the padded planes, counted over the batch) of one phase
  if (!a.d_first) L -= a.nW;
  const int per_ph = a.d_tm * a.d_tn;
  const int tile = L / a.d_nz, z = L - tile * a.d_nz;
  const int ph = tile / per_ph, rest = tile - ph * per_ph;
  const int tni = rest / a.d_tm, tmi = rest - tni * a.d_tm;   // row tiles of one column tile run side by side
  const int m0 = tmi * S::BM;
  const int ntap = a.ntap[ph], nck = a.Cop >> 6;
  const int it0 = z * a.d_its, iters = min(ntap * nck, it0 + a.d_its);   // steps of this slab
  if (tid < min(ntap, kTapsLds)) lds.taps[tid] = a.taps[(long)ph * a.KK + tid];
  __syncthreads();
  if (it0 < iters) sd_mainloop<TM, TN>(a, m0, tni, it0, iters, lds.op, lds.taps, acc);
  if (a.d_nz > 1 && !reduce_slabs<1, S::TNW, S::NT>(acc, a.partD + (long)tile * (a.d_nz + a.d_ngrp) * (4096 * TM * TN), z,
                                                    a.tickD + tile * (1 + a.d_ngrp), a.d_nz, a.d_grp, a.d_ngrp, &lds.flag,
                                                    a.Ci - m0 - 32 * wm, 64 * S::TNW))   // (all column tiles of the wave)
    return;
  // through LDS (rounded once to the storage type), out as 16-byte runs of pixels
  bf16_t* Cs = reinterpret_cast<bf16_t*>(lds.op);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < S::TNW; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      Cs[(32 * wm + acc_row(lane, v)) * S::SC + 32 * (S::WN * j + wn) + (lane & 31)] = from_f32<bf16_t>(acc[0][j][v]);
  __syncthreads();
  constexpr int VB = S::BN / 8;
  const int jv = tni * VB + tid % VB;               // this lane's column vector
  const int nimg = (int)a.d_qd.div((uint32_t)jv), q = (jv - nimg * a.qd) * 8;
  if (nimg >= a.N || q >= a.PQ) return;
  bf16_t* out = static_cast<bf16_t*>(a.gx) + ((long)(ph * a.N + nimg) * a.Ci + m0) * a.PQ + q;
  const int nr = min(S::BM, a.Ci - m0);
#pragma unroll 4
  for (int row = tid / VB; row < nr; row += S::NT / VB) {
    bf16_t* d = out + (long)row * a.PQ;
    const bf16_t* src = Cs + row * S::SC + tid % VB * 8;
    if (q + 8 <= a.PQ) {
      const uint4 val = *reinterpret_cast<const uint4*>(src);
      Unal<bf16_t> o;
      o.w[0] = val.x; o.w[1] = val.y; o.w[2] = val.z; o.w[3] = val.w;
      *reinterpret_cast<Unal<bf16_t>*>(d) = o;
    } else {
      for (int e = 0; q + e < a.PQ; ++e) d[e] = src[e];
    }
  }
}

template <class T, int TM, int TN>
__device__ __forceinline__ void xwgrad_block(const XArgs& a, int L, unsigned char* smem) {
  using X = XTile<T, TM, TN>;
  static_assert(XTile<raw_f32, TM, TN>::kOp <= X::kBytes || !is_split<T>(), "the second pass works in the same LDS");
  const WTileAt w = wtile_at(a, L, X::BM, X::BN);
  const int z = w.z, t = w.t, m0 = w.m0, n0 = w.n0;
  if (z >= a.nz) return;  // uniform for the block
  const int kc0 = z * a.cpz, kc1 = min(kc0 + a.cpz, a.nchunks);
  f32x16 acc[TM][TN];
  uint32_t low = 0;
  zero_acc(acc);
  xw_mainloop<T, TM, TN>(a, t, m0, n0, kc0, kc1, smem, acc, low);
  if constexpr (is_split<T>()) {
    if (split_failed(acc, low)) {
      zero_acc(acc);
      xw_mainloop<raw_f32, TM, TN>(a, t, m0, n0, kc0, kc1, smem, acc, low);
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  float* dst = a.part + ((long)z * a.KK + t) * a.Co * a.Ci;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int ci = n0 + 64 * j + 32 * wn + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int co = m0 + 64 * i + 32 * wm + acc_row(lane, v);
        if (co < a.Co && ci < a.Ci) dst[(long)co * a.Ci + ci] = acc[i][j][v];
      }
    }
}

// acc += w[steps][rows m0 ..]^T * g_y[steps][columns of the tile, moved by the tap] over steps (tap of the phase, chunk of c_o)
template <class T, int TM, int TN>
__device__ __forceinline__ void xd_mainloop(const XArgs& a, int ph, int m0, int tni, int it0, int iters, unsigned char* smem,
                                            const int2* taps_lds, f32x16 (&acc)[TM][TN], uint32_t& low) {
  using X = XTile<T, TM, TN>;
  constexpr int VE = X::VE, KB = X::KB, LA = 2 * TM, LB = 2 * TN;
  constexpr int VA = X::BM / VE, VB = X::BN / VE;   // vectors per row of k
  static_assert(kT % VB == 0, "a lane keeps its column vector");
  typedef XSet<LA, LB> Set;
  const int2* taps = a.tapd + (long)ph * a.KK;
  const uint8_t* tab = a.tabd + (long)ph * a.KK * a.nvd;
  const int tid = lane_id<T>(), lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  unsigned char* As = smem;
  unsigned char* Bs = smem + X::TERMS * X::DA;
  const T* gy = static_cast<const T*>(a.gy);
  const T* wt = static_cast<const T*>(a.wt);
  const int jv = tni * VB + tid % VB;               // this lane's column vector
  const int nimg = (int)a.d_qd.div((uint32_t)jv);
  const int q = (jv - nimg * a.qd) * VE;
  const bool img = nimg < a.N;
  const int colbase = min(nimg, a.N - 1) * a.Co * a.HWy + q;
  const int hi = a.tot_gy - VE;
  int ca[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) ca[i] = min(m0 + (tid + i * kT) % VA * VE, a.Cip - VE);
  int kk = it0 / a.nck, kc = it0 - kk * a.nck;   // tap of the list and chunk of c_o the next fetch takes
  int2 tap = make_int2(0, 0);
  bool new_tap = true;
  auto fetch = [&](Set& s, int it) __attribute__((always_inline)) {
    if (new_tap) {   // (uniform)
      // (two loads that the compiler cannot merge into one of a selected address: a flat load would wait for every
      // load in flight)
      if (kk < kTapsLds) {
        tap.x = __builtin_amdgcn_readfirstlane(taps_lds[kk].x);
        tap.y = __builtin_amdgcn_readfirstlane(taps_lds[kk].y);
      } else {
        const int2 g = taps[kk];
        tap.x = __builtin_amdgcn_readfirstlane(g.x);
        tap.y = __builtin_amdgcn_readfirstlane(g.y);
      }
    }
    s.k0 = kc * KB;
    s.mb = tab[tap.x * a.nvd + (q >> 3)];
    s.ob = colbase + tap.y + s.k0 * a.HWy;
    s.off = 0;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int k = min(s.k0 + (tid + i * kT) / VA, a.Co - 1);
      s.a[i] = load16<T, false>(wt + ((long)tap.x * a.Co + k) * a.Cip + ca[i]);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int o = s.ob + (tid + i * kT) / VB * a.HWy, oc = min(max(o, 0), hi);
      s.off |= o ^ oc;
      s.b[i] = load16<T, true>(gy + oc);
    }
    if (it + 1 < iters) {   // (uniform)
      new_tap = ++kc == a.nck;
      if (new_tap) { kc = 0; ++kk; }
    } else {
      new_tap = false;
    }
  };
  auto stage = [&](Set& s, int, auto neg) __attribute__((always_inline)) {
    if (s.off) {   // first or last rows of g_y only: shift the moved vectors back
#pragma unroll
      for (int i = 0; i < LB; ++i) {
        const int o = s.ob + (tid + i * kT) / VB * a.HWy;
        s.b[i] = shifted<T>(s.b[i], min(max(o - min(max(o, 0), hi), -VE), VE));
      }
    }
    const u32x4_t m = bit_mask<T>(img ? vec_mask<T>(s.mb, q) : 0u);
#pragma unroll
    for (int i = 0; i < LB; ++i) s.b[i] &= m;
    if (s.k0 + KB > a.Co) {   // rows past c_o (the last chunk of a tap only)
#pragma unroll
      for (int i = 0; i < LA; ++i)
        if (s.k0 + (tid + i * kT) / VA >= a.Co) s.a[i] = u32x4_t{0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < LB; ++i)
        if (s.k0 + (tid + i * kT) / VB >= a.Co) s.b[i] = u32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int i = 0; i < LA; ++i) put_row<T, X::BM, decltype(neg)::value>(As, (tid + i * kT) / VA, (tid + i * kT) % VA, s.a[i], low);
#pragma unroll
    for (int i = 0; i < LB; ++i) put_row<T, X::BN>(Bs, (tid + i * kT) / VB, tid % VB, s.b[i], low);
  };
  auto mul = [&](auto neg) __attribute__((always_inline)) {
    typename El<T>::acc s;
#pragma unroll
    for (int ks = 0; ks < El<T>::KS; ++ks) {
      uint4 fa[TM][X::TERMS], fb[TN][X::TERMS];
#pragma unroll
      for (int u = 0; u < X::TERMS; ++u) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i][u] = frag_tr<T, X::BM>(As + u * X::DA, ks, 64 * i + 32 * wm, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j][u] = frag_tr<T, X::BN>(Bs + u * X::DB, ks, 64 * j + 32 * wn, lane);
      }
      mul_all<T, decltype(neg)::value>(fa, fb, acc, s, ks);
    }
  };
  k_loop<xsets_of<T, TM, TN>(), Set>(it0, iters, fetch, stage, mul);
}

// rows c_i of one column tile (64 TN positions of the padded planes, counted over the batch) of one phase
template <class T, int TM, int TN>
__device__ __forceinline__ void xdgrad_block(const XArgs& a, int L, unsigned char* smem, int2* taps_lds, int* s_flag) {
  using X = XTile<T, TM, TN>;
  constexpr int VE = X::VE, VB = X::BN / VE;
  const int per_ph = a.d_tm * a.d_tn;
  const int tile = L / a.d_nz, z = L - tile * a.d_nz;
  const int ph = tile / per_ph, rest = tile - ph * per_ph;
  const int tni = rest / a.d_tm, tmi = rest - tni * a.d_tm;   // row tiles of one column tile run side by side
  const int m0 = tmi * X::BM;
  const int ntap = a.ntap[ph];
  const int it0 = z * a.d_its, iters = min(ntap * a.nck, it0 + a.d_its);   // steps of this slab
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  if (tid < min(ntap, kTapsLds)) taps_lds[tid] = a.tapd[(long)ph * a.KK + tid];
  __syncthreads();
  f32x16 acc[TM][TN];
  uint32_t low = 0;
  zero_acc(acc);
  if (it0 < iters) xd_mainloop<T, TM, TN>(a, ph, m0, tni, it0, iters, smem, taps_lds, acc, low);
  if constexpr (is_split<T>()) {
    if (split_failed(acc, low)) {
      zero_acc(acc);
      xd_mainloop<raw_f32, TM, TN>(a, ph, m0, tni, it0, iters, smem, taps_lds, acc, low);
    }
  }
  if (a.d_nz > 1 && !reduce_slabs<TM, TN>(acc, a.partD + (long)tile * (a.d_nz + a.d_ngrp) * (4096 * TM * TN), z,
                                          a.tickD + tile * (1 + a.d_ngrp), a.d_nz, a.d_grp, a.d_ngrp, s_flag,
                                          a.Ci - m0 - 32 * wm, 64 * TN))
    return;

  const int jv = tni * VB + tid % VB;               // this lane's column vector
  const int nimg = (int)a.d_qd.div((uint32_t)jv);
  const int q = (jv - nimg * a.qd) * VE;
  const bool img = nimg < a.N;
  // 64 rows at a time through LDS (rounded once to the storage type), out as 16-byte runs of pixels
  T* Cs = reinterpret_cast<T*>(smem);
  T* out = static_cast<T*>(a.gx) + (long)ph * a.N * a.Ci * a.PQ;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m1 = m0 + 64 * i;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        Cs[(32 * wm + acc_row(lane, v)) * X::SC + 64 * j + 32 * wn + (lane & 31)] = from_f32<T>(acc[i][j][v]);
    __syncthreads();
    // the lane's column vector is the one of its operand loads
    if (img && q < a.PQ) {
#pragma unroll 4
      for (int row = tid / VB; row < 64; row += kT / VB) {
        if (m1 + row >= a.Ci) break;
        T* d = out + ((long)nimg * a.Ci + m1 + row) * a.PQ + q;
        const T* src = Cs + row * X::SC + tid % VB * VE;
        if (q + VE <= a.PQ) {
          const uint4 val = *reinterpret_cast<const uint4*>(src);
          Unal<T> o;
          o.w[0] = val.x; o.w[1] = val.y; o.w[2] = val.z; o.w[3] = val.w;
          *reinterpret_cast<Unal<T>*>(d) = o;
        } else {
          for (int e = 0; q + e < a.PQ; ++e) d[e] = src[e];
        }
      }
    }
  }
}

template <class T, int TM, int TN>
__global__ __launch_bounds__(kT, TM * TN == 4 ? 2 : 3) void xgemm_k(XArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[XTile<T, TM, TN>::kBytes];
  __shared__ int2 taps_lds[kTapsLds];
  __shared__ int s_flag;
  const int b = blockIdx.x;
  if (a.d_first ? b < a.nD : b >= a.nW) xdgrad_block<T, TM, TN>(a, a.d_first ? b : b - a.nW, smem, taps_lds, &s_flag);
  else xwgrad_block<T, TM, TN>(a, a.d_first ? b - a.nD : b, smem);
}

// ---------------------------------------------------------------------------
// last launch: g_w[pair][t] = sum_z part[z][t][pair] (blocks of 64 pairs), then g_x from its phase planes
// ---------------------------------------------------------------------------
struct FinalArgs {
  const float* part;
  float* g_w;
  int pairs, KK, nz, w_blocks;
  const void* gxq;
  void* gx;
  int NC, H, W, Hq, Wq, s, ppb;
  FastDiv d_w, d_h, d_s;
};

__device__ __forceinline__ int cdiv_dev(int a, int b) { return (a + b - 1) / b; }

constexpr int kFinTaps = 9;   // taps a pass of a block holds

// where the VE pixels from e0 on (over planes of H x W) stand in `planes` planes of every phase
template <int VE>
__device__ __forceinline__ void interleave_offsets(const FinalArgs& a, int e0, int planes, int (&at)[VE]) {
  const int PQ = a.Hq * a.Wq;
  const int r0 = (int)a.d_w.div((uint32_t)e0);
  int w = e0 - r0 * a.W;
  int pl = (int)a.d_h.div((uint32_t)r0), h = r0 - pl * a.H;
#pragma unroll
  for (int k = 0; k < VE; ++k) {
    const int hs = (int)a.d_s.div((uint32_t)h), ws = (int)a.d_s.div((uint32_t)w);
    at[k] = (((h - hs * a.s) * a.s + w - ws * a.s) * planes + pl) * PQ + hs * a.Wq + ws;
    if (++w == a.W) {
      w = 0;
      if (++h == a.H) { h = 0; ++pl; }
    }
  }
}

template <class T, int VE>
__device__ __forceinline__ void put_run(T* dst, int e0, int total, const T (&v)[VE]) {
  if (e0 + VE <= total) {
    *reinterpret_cast<uint4*>(dst + e0) = *reinterpret_cast<const uint4*>(v);
  } else {
#pragma unroll
    for (int k = 0; k < VE; ++k)
      if (e0 + k < total) dst[e0 + k] = v[k];
  }
}

template <class T>
__global__ __launch_bounds__(kT) void xfinal_k(FinalArgs a) {
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < a.w_blocks) {
    // Lane (g, e): the slabs z = g, g + 4, ... of pair e, all taps of a pass in flight; the four sums of a value are
    // then added in index order (the result does not depend on scheduling) and the values leave tap-minor as one run.
    __shared__ float red[4][kFinTaps][64 + 1];
    const int e = tid & 63, g = tid >> 6;
    const int p0 = blockIdx.x * 64, np = min(64, a.pairs - p0);
    const float* src = a.part + p0 + min(e, np - 1);
    const long ts = a.pairs, zs = (long)a.KK * a.pairs;
    for (int t0 = 0; t0 < a.KK; t0 += kFinTaps) {
      const int nt = min(kFinTaps, a.KK - t0);
      float s[kFinTaps];
#pragma unroll
      for (int t = 0; t < kFinTaps; ++t) s[t] = 0.f;
#pragma unroll 2
      for (int z = g; z < a.nz; z += 4) {
        float v[kFinTaps];
#pragma unroll
        for (int t = 0; t < kFinTaps; ++t) v[t] = src[z * zs + (t0 + min(t, nt - 1)) * ts];
#pragma unroll
        for (int t = 0; t < kFinTaps; ++t) s[t] += v[t];
      }
      if (t0) __syncthreads();
#pragma unroll
      for (int t = 0; t < kFinTaps; ++t) red[g][t][e] = s[t];
      __syncthreads();
      for (int i = tid; i < np * nt; i += kT) {
        const int pe = i / nt, t = i - pe * nt;
        a.g_w[(long)(p0 + pe) * a.KK + t0 + t] = ((red[0][t][pe] + red[1][t][pe]) + red[2][t][pe]) + red[3][t][pe];
      }
    }
    return;
  }
  // g_x[n, ci, h, w] = gxq[phase(h mod s, w mod s)][n, ci, h / s, w / s].  Small planes: a block stages ppb consecutive
  // planes of every phase -- one contiguous run each, at element alignment -- and writes their pixels as one aligned run (a
  // gather of two-byte elements from memory took 15 us for 12.8 MB).
  constexpr int VE = El<T>::VE;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* lds = reinterpret_cast<T*>(smem);
  const int PQ = a.Hq * a.Wq, HW = a.H * a.W, nph = a.s * a.s;
  const int pl0 = ((int)blockIdx.x - a.w_blocks) * a.ppb, np = min(a.ppb, a.NC - pl0);
  const T* gxq = static_cast<const T*>(a.gxq);
  T* gx = static_cast<T*>(a.gx);
  if (a.ppb == 0) {   // large planes: a vector per lane, gathered from the phase planes
    const int e0 = (((int)blockIdx.x - a.w_blocks) * kT + tid) * VE, total = a.NC * HW;
    if (e0 >= total) return;
    int at[VE];
    interleave_offsets<VE>(a, e0, a.NC, at);
    __attribute__((aligned(16))) T v[VE];
#pragma unroll
    for (int k = 0; k < VE; ++k) v[k] = gxq[e0 + k < total ? at[k] : at[0]];
    put_run(gx, e0, total, v);
    return;
  }
  const int run = np * PQ, runv = cdiv_dev(run, VE);
  for (int i = tid; i < nph * runv; i += kT) {
    const int ph = i / runv, v = i - ph * runv;
    const long o = ((long)ph * a.NC + pl0) * PQ;
    if (v * VE + VE <= run) {
      const uint4 q = load_vec<T>(gxq + o + v * VE);
      const u32x4_t w = {q.x, q.y, q.z, q.w};
      T* d = lds + ph * a.ppb * PQ + v * VE;
#pragma unroll
      for (int k = 0; k < VE; ++k) {
        if constexpr (sizeof(T) == 4) d[k] = __uint_as_float(w[k]);
        else d[k] = __builtin_bit_cast(T, (uint16_t)(w[k >> 1] >> (16 * (k & 1))));
      }
    } else {
      for (int k = v * VE; k < run; ++k) lds[ph * a.ppb * PQ + k] = gxq[o + k];
    }
  }
  __syncthreads();
  const int total = np * HW;
  T* dst = gx + (long)pl0 * HW;   // (host: ppb * H * W is a multiple of VE)
  for (int e0 = tid * VE; e0 < total; e0 += kT * VE) {
    int at[VE];
    interleave_offsets<VE>(a, e0, a.ppb, at);
    __attribute__((aligned(16))) T v[VE];
#pragma unroll
    for (int k = 0; k < VE; ++k) v[k] = lds[min(at[k], nph * a.ppb * PQ - 1)];
    put_run(dst, e0, total, v);
  }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

int up8(int v) { return (v + 7) / 8 * 8; }

// Geometry of the implicit GEMMs: PQ = plane of the x operand / of the g_x output (the phase
// plane Hq x Wq for strided layers, the image itself for stride 1), PY = plane of g_y.
struct XGeo {
  int s, nph, Hq, Wq, PQ, PY;
};

XGeo make_xgeo(const Geom& g) {
  XGeo q;
  q.s = g.s;
  q.nph = g.s * g.s;
  q.Hq = g.s == 1 ? g.H : (g.H + g.s - 1) / g.s;
  q.Wq = g.s == 1 ? g.W : g.Wy;
  q.PQ = q.Hq * q.Wq;
  q.PY = g.Hy * g.Wy;
  return q;
}

// largest |tap offset| in flattened pixels of a plane of pitch Wq
long max_shift(const Geom& g, const XGeo& q) {
  const long a = g.p, b = (long)g.dl * ((g.Kh > g.Kw ? g.Kh : g.Kw) - 1) - g.p;
  return ((a > b ? a : b) / g.s + 1) * (q.Wq + 1);
}

// K slabs of a layer: kFull as many as are fastest; kSlim no more than take a smaller workspace -- of the input gradient (fp32) from 16
// steps on only, of the weight gradient fewer beside them.
enum Form { kFull, kSlim };

struct XPlan {
  bool staged;
  int Cop, Cix;   // channels of a staged row
  size_t off_gt, off_xt, off_wr;
  size_t off_tabw, off_tabd, off_taps, off_tick, off_wt, off_xq, off_gxq, off_part, off_pd, total;
  int nvw, nvd, tm, tn, Cip, ntickets;
  int d_nz, d_its, d_grp, d_ngrp, d_first;
  int qv, nchunks, nz, cpz, w_tm, w_tn, qd, d_tm, d_tn;
};

// taps of the phase that has most of them: taps of one phase are s / gcd(dilation, s) apart
int most_taps(const Geom& g) {
  const int step = g.s / std::gcd(g.dl, g.s);
  return cdiv(g.Kh, step) * cdiv(g.Kw, step);
}

// Tile sides in units of 64: 128 x 128 where every block slot of the chip has at least eight steps of such tiles (two
// blocks per CU: registers), 128 x 64 below that, and 64 x 64 where a side of the layer has no more than 64 channels.
// An input gradient alone has its few channels in K: 128 x 128 (c_i, pixels) from 384 such tiles on, where K is one slab
// with either tile (bf16: the bits of the call for both; fp32: 16 instead of 32 k before a sum goes to the total).
// 64 x 64 / 128 x 128 in us, 3 x 3: 512 -> 64 channels, 48 x 48, n = 40 bf16 160 / 103, fp32 453 / 358; 192 -> 64,
// 120 x 160, n = 8 107 / 87, 303 / 298; 320 -> 40, 33 x 33, n = 16 (408 tiles) 31.9 / 28.6, 68.8 / 67.3; 128 -> 64,
// 60 x 80, n = 8 (300) 28.5 / 25.2, 62 / 63.5; 192 -> 64, 30 x 40, n = 8 (150) 18.4 / 21.4, 34 / 50.
void tile_shape(const Geom& g, const XGeo& q, bool want_gw, int* tm, int* tn, long* slots) {
  const bool wide = g.Co > 64 && g.Ci > 64;
  const long w_steps = (long)cdiv(g.Co, 128) * cdiv(g.Ci, 128) * g.KK * cdiv((long)g.N * up8(q.PY), g.b == 2 ? 64 : 32);
  *tm = wide ? 2 : 1;
  *tn = wide && w_steps >= 4 * 512 ? 2 : 1;
  if (!want_gw && !wide && g.Ci > 64 && (long)cdiv(g.Ci, 128) * cdiv((long)g.N * up8(q.PQ), 128) * q.nph >= 384) *tm = *tn = 2;
  *slots = *tn == 2 ? 512 : 768;
}
// Chunks per slab for about z slabs.  Slabs go to the XCDs in turn (each L2 then keeps its own part of the maps), so
// from eight on their number is a multiple of eight where the chunks allow it.
int slab_chunks(int nchunks, long z) {
  if (z >= 6) {
    const long z8 = std::max(8L, (z + 2) / 8 * 8);
    if (cdiv(nchunks, cdiv(nchunks, z8)) % 8 == 0) z = z8;
  }
  return cdiv(nchunks, z);
}
// Slabs dealt to the XCDs: also a number that is no multiple of eight while no XCD gets more than a tenth above its share (its
// last round of block numbers is partly empty).  64 -> 64 channels, 200 x 200, n = 4, 87 slabs: both gradients 94 -> 69 us,
// 120 x 160, n = 8 (86): 90 -> 65; 128 -> 128, 60 x 80, n = 8 (50): 59 -> 51.
// 280 layers of all calls that split K (vanilla of both types, bf16 weight gradients of 6 GFLOP and more): 0.89 .. 1.28, mean 1.004.
bool deal_slabs(int nz) { return 10 * (cdiv(nz, 8) * 8) <= 11 * nz; }
XPlan make_plan(const Geom& g, bool want_gw, bool want_gx, bool staged, Form form) {
  const XGeo q = make_xgeo(g);
  const int VE = 16 / g.b;
  XPlan p = {};
  p.nvw = up8(q.PY) / 8;
  p.nvd = up8(q.PQ) / 8;
  long slots;
  tile_shape(g, q, want_gw, &p.tm, &p.tn, &slots);
  p.Cip = cdiv(g.Ci, VE) * VE;
  p.qv = up8(q.PY) / VE;
  p.staged = staged;
  p.Cop = (g.Co + 63) / 64 * 64;
  p.Cix = (g.Ci + 63) / 64 * 64;
  p.nchunks = staged ? cdiv((long)g.N * q.PY, 64) : cdiv((long)g.N * p.qv, 8);
  p.w_tm = cdiv(g.Co, 64 * p.tm);
  p.w_tn = cdiv(g.Ci, 64 * p.tn);
  p.qd = up8(q.PQ) / VE;
  p.d_tm = cdiv(g.Ci, 64 * p.tm);
  p.d_tn = cdiv((long)g.N * p.qd, 64 * p.tn / VE);
  // Steps (64 or 32 k each) of the two products.  The chip holds about slots blocks; a step of the larger tile counts
  // double.  Input gradient: K = (tap, c_o) is split (slab sums inside the launch) only where its tiles leave most
  // of the chip idle.  Weight gradient: as many slabs as the slots the input gradient leaves can take in one go.
  const long d_tiles = (long)p.d_tm * p.d_tn * q.nph, w_tiles = (long)p.w_tm * p.w_tn * g.KK;
  const int taps = cdiv(g.KK, q.nph);                     // per phase, about
  const int d_steps = taps * cdiv(g.Co, g.b == 2 ? 64 : 32), d_most = most_taps(g) * cdiv(g.Co, g.b == 2 ? 64 : 32);
  p.d_nz = 1;
  // Twice the slabs where a block has 16 steps and more and half the slots take them; fp32, whose steps take twice as long: also from
  // 8 steps on where a quarter of the slots does, from 4 where an eighth does.  Both gradients in us, 16 steps / this rule: 256 -> 88, 3 x 3,
  // 6 x 6, n = 2 37.9 / 25.9; 154 -> 88, 5 x 5, n = 1 38.5 / 26.9; 216 -> 144, 15 x 15, stride 2, n = 2 42.9 / 26.8; 250 random layers: the 82
  // that change 1.18 times as fast in the mean, 0.96 at the least.  With 8 steps up to half the slots: 64 -> 32, 25 x 25, n = 19 33 / 40.
  // bf16 from 8 steps on where a sixteenth takes them: 41 layers 1.05 in the mean, but ten of them 0.88 - 0.95; not taken.  Nor under
  // 16 output channels, whose steps are mostly padding: 8 of 4 x 4, n = 2 would bring 128 KB of slabs to 3 KB of tensors.
  auto worth = [&](int steps, long blocks) { return steps >= 16 && blocks <= slots / 2; };
  auto worth_f32 = [&](int steps, long blocks) { return (steps >= 8 && blocks <= slots / 4) || (steps >= 4 && blocks <= slots / 8); };
  while (p.d_nz < 64 && worth(d_steps / p.d_nz, d_tiles * p.d_nz * 2)) p.d_nz *= 2;
  const int nz16 = p.d_nz;
  if (form == kFull && g.b == 4 && g.Co >= 16)
    while (p.d_nz < 64 && (worth(d_steps / p.d_nz, d_tiles * p.d_nz * 2) || worth_f32(d_steps / p.d_nz, d_tiles * p.d_nz * 2))) p.d_nz *= 2;
  p.d_its = p.d_nz == 1 ? d_most : cdiv(d_steps, p.d_nz);
  // phases with more taps than the average need more slabs (counted up to the taps of the whole kernel, most of them were
  // empty: 208 -> 104, 5 x 5, 20 x 20, stride 2, n = 10, fp32 98 -> 56 us; 152 -> 488, 10 x 10, n = 12, bf16 47 -> 36)
  if (p.d_nz > 1) p.d_nz = cdiv(d_most, p.d_its);
  groups_for(p.d_nz, &p.d_grp, &p.d_ngrp);
  p.ntickets = p.d_nz > 1 ? (int)(d_tiles * (1 + p.d_ngrp)) : 0;
  // Both products at once where the slots the input gradient leaves take the weight gradient with blocks of about its
  // length; else several rounds, with weight-gradient blocks of about half the launch.
  // (kSlim counts the blocks of the input gradient up to the taps of the whole kernel: fewer slabs are left for g_w)
  long d_blocks = d_tiles * p.d_nz, d_len = p.d_nz == 1 ? d_steps : p.d_its;
  if (form != kFull) {
    d_len = cdiv(d_steps, nz16);
    d_blocks = d_tiles * (nz16 == 1 ? 1 : cdiv(g.KK * cdiv(g.Co, g.b == 2 ? 64 : 32), (int)d_len));
  }
  const long per_slot = (w_tiles * p.nchunks + d_blocks * d_len) / slots;
  long z = (slots - d_blocks) / w_tiles;
  if (z < 1 || cdiv(p.nchunks, z) > 1.2 * std::max(d_len, per_slot)) z = cdiv(p.nchunks, std::max(per_slot / 2, 8L));
  const long most = p.nchunks / 4 > 0 ? p.nchunks / 4 : 1;   // at least four chunks per block
  z = std::min(z, most);
  p.cpz = slab_chunks(p.nchunks, z);
  p.nz = cdiv(p.nchunks, p.cpz);
  p.d_first = (p.d_nz == 1 ? d_steps : p.d_its) > p.cpz ? 1 : 0;   // the longer blocks start first
  size_t off = 0;
  if (staged) {
    p.off_taps = off; off += align256(sizeof(int4) * (size_t)q.nph * g.KK + sizeof(int) * q.nph);
    p.off_tick = off; off += align256(sizeof(int) * (size_t)p.ntickets);
    p.off_gt = off; off += align256(((size_t)g.N * q.PY + 1) * p.Cop * g.b);
    p.off_xt = off; if (want_gw) off += align256(((size_t)g.N * g.H * g.W + 1) * p.Cix * g.b);
    p.off_wr = off; if (want_gx) off += align256(((size_t)g.Ci * g.KK + 1) * p.Cop * g.b);
    p.off_gxq = off; if (want_gx && g.s > 1) off += align256((size_t)q.nph * g.N * g.Ci * q.PQ * g.b);
    p.off_part = off; if (want_gw) off += align256((size_t)p.nz * g.KK * g.Co * g.Ci * sizeof(float));
    p.off_pd = off;
    if (want_gx && p.d_nz > 1) off += align256((size_t)d_tiles * (p.d_nz + p.d_ngrp) * 4096 * p.tm * p.tn * sizeof(float));
    p.total = off;
    return p;
  }
  p.off_tabw = off; off += align256((size_t)g.KK * p.nvw);
  p.off_tabd = off; off += align256((size_t)q.nph * g.KK * p.nvd);
  p.off_taps = off; off += align256(sizeof(int) * ((size_t)g.KK + 2 * (size_t)q.nph * g.KK + q.nph));
  p.off_tick = off; off += align256(sizeof(int) * (size_t)p.ntickets);
  p.off_wt = off;
  if (want_gx) off += align256((size_t)g.KK * g.Co * p.Cip * g.b);
  p.off_xq = off;
  if (want_gw && g.s > 1) off += align256((size_t)q.nph * g.N * g.Ci * q.PQ * g.b);
  p.off_gxq = off;
  if (want_gx && g.s > 1) off += align256((size_t)q.nph * g.N * g.Ci * q.PQ * g.b);
  p.off_part = off;
  if (want_gw) off += align256((size_t)p.nz * g.KK * g.Co * g.Ci * sizeof(float));
  p.off_pd = off;
  if (want_gx && p.d_nz > 1) off += align256((size_t)d_tiles * (p.d_nz + p.d_ngrp) * 4096 * p.tm * p.tn * sizeof(float));
  p.total = off;
  return p;
}
size_t plan_bytes(const Geom& g, bool want_gw, bool want_gx, bool staged, Form form) { return make_plan(g, want_gw, want_gx, staged, form).total; }
// The form a call on the maps themselves takes with all the workspace it asks for: kSlim where only that keeps both gradients within the library's own
// scratch.  The one-call entry, which returns the same bits there, and in fp32, where the slabs of g_x differ, all others whatever
// they ask for.  Layers that cannot come near it are not planned twice: an upper bound of the weight-gradient slabs (a slab has four
// chunks), the repacked tensors and half the block slots' tiles of g_x.
Form form_of(const Geom& g) {
  if (g.b == 2 && !g.own_scratch) return kFull;
  const XGeo q = make_xgeo(g);
  const double wel = (double)g.KK * g.Co * (g.Ci + 7), slabs = 4 + (double)g.N * up8(q.PY) * g.b / (4 * 128);
  const double tiles = 27e6 * most_taps(g) / cdiv(g.KK, q.nph);
  if (4 * wel * (1 + slabs) + 8. * q.nph * g.N * g.Ci * q.PQ + (double)g.KK * (q.PY + q.nph * (q.PQ + 64)) + tiles <= GF_STATIC_SCRATCH_BYTES) return kFull;
  return plan_bytes(g, true, true, false, kFull) > GF_STATIC_SCRATCH_BYTES && plan_bytes(g, true, true, false, kSlim) <= GF_STATIC_SCRATCH_BYTES ? kSlim : kFull;
}

// planes a block of the interleave stages: a multiple of VE (runs start on vector boundaries), about 16 KB, and
// enough blocks for the chip; 0 where that many planes do not fit LDS (from 56 x 56 on): gathered from memory (64 ->
// 128 channels, 112 x 112, stride 2, n = 8, both gradients: 53 us in bf16, 109 in fp32; through a column tensor 370, 568)
int interleave_planes(const Geom& g, const XGeo& q) {
  const int VE = 16 / g.b;
  const long plane = (long)q.nph * q.PQ * g.b;
  if (VE * plane > 48 * 1024) return 0;
  long ppb = 16 * 1024 / (VE * plane) * VE;
  while (ppb > VE && (long)g.N * g.Ci / ppb < 1024) ppb -= VE;
  return (int)(ppb < VE ? VE : ppb);
}

// Calls whose operands are staged: bf16, kernels larger than 1 x 1, channels that fill most of the rows they are padded to
// (64), offsets of staged rows within 32 bits; not where the copies alone would take a call out of the library's own scratch.
// Not either where the copies cost a weight gradient alone more than the products gain: 128 x 128 tiles, few operations per
// element, maps past 64 MiB.  3 x 3, unstaged / staged in us: 128 -> 128, 60 x 80, n = 32 (79 MB) 81 / 86, n = 128 270 / 319;
// 96 -> 96, 112 x 112, n = 128 629 / 783; 128 -> 256, 60 x 80, n = 128 552 / 594; but 128 -> 128, 28 x 28, n = 64 43.7 / 42.2,
// 256 -> 256, 60 x 80, n = 128 1613 / 1210; 5 x 5, 128 -> 128, 56 x 56, n = 64 275 / 237.  With planes of whole vectors either
// form returns the same weight gradient, with others K is cut into other chunks; there gf_conv_bwd_exact, gf_conv_bwd_weight and the
// chained entry, with the workspace gf_workspace_bytes names, take the same form whichever gradients they are asked for (57 x 81, n = 64, both gradients 274 / 269).  The one-call entry, which
// returns the same bits on the library's scratch, keeps the unstaged form where only that fits (256 -> 256, 57 x 57, n = 32: 37 MB,
// staged 138), with any workspace: its g_w may then differ from theirs in the order of the sums, its g_x does not.
bool staged_ok(const Geom& g, bool want_gx) {
  if (g.dtype != GF_BF16 || g.KK == 1 || g.KK > kTapsLds) return false;
  const XGeo q = make_xgeo(g);
  const long cop = (g.Co + 63) / 64 * 64, cix = (g.Ci + 63) / 64 * 64, lim = (1L << 31) - 4096;
  if (4 * g.Co < 3 * cop || 4 * g.Ci < 3 * cix) return false;
  if (((long)g.N * q.PY + 1) * cop * 2 > lim || ((long)g.N * g.H * g.W + 1) * cix * 2 > lim ||
      ((long)g.Ci * g.KK + 1) * cop * 2 > lim)
    return false;
  if (g.s == 1 && g.Co > 64 && g.Ci > 64 && (long)g.KK * g.Co * g.Ci <= 800L * (g.Co + g.Ci) &&
      ((long)g.N * q.PY * g.Co + (long)g.N * g.H * g.W * g.Ci) * 2 >= (64L << 20) && !(want_gx && q.PY % 8 == 0))
    return false;
  return !g.own_scratch || plan_bytes(g, true, true, true, kFull) <= GF_STATIC_SCRATCH_BYTES ||
         plan_bytes(g, true, true, false, form_of(g)) > GF_STATIC_SCRATCH_BYTES;
}

// the product launch and the last one (x: the map itself or its phase planes; staged layers: in the workspace)
template <class T>
hipError_t implicit_products(const Geom& g, const XGeo& q, const XPlan& p, const void* x, const void* g_y, float* g_w, void* g_x,
                             char* wsb, hipStream_t st) {
  const bool want_gw = g_w != nullptr, want_gx = g_x != nullptr;
  constexpr int VE = El<T>::VE;
  int2* tapd = reinterpret_cast<int2*>(wsb + p.off_taps);   // 8-byte aligned: first in the region
  int* tapw = reinterpret_cast<int*>(tapd + (size_t)q.nph * g.KK);
  // ---- both products
  XArgs a = {};
  a.N = g.N; a.Ci = g.Ci; a.Co = g.Co; a.KK = g.KK;
  a.gy = g_y; a.HWy = q.PY; a.tot_gy = g.N * g.Co * q.PY;
  a.x = x;
  a.part = reinterpret_cast<float*>(wsb + p.off_part);
  a.tabw = reinterpret_cast<uint8_t*>(wsb + p.off_tabw); a.tapw = tapw;
  a.HW = q.PQ; a.tot_x = q.nph * g.N * g.Ci * q.PQ;
  a.qv = p.qv; a.kvecs = g.N * p.qv; a.nvw = p.nvw;
  a.nchunks = p.nchunks; a.cpz = p.cpz; a.nz = p.nz;
  a.tx = p.w_tn; a.tiles = p.w_tm * p.w_tn; a.R = a.tiles * g.KK;
  a.xcd_slabs = deal_slabs(p.nz) ? 1 : 0;
  a.nW = !want_gw ? 0 : a.xcd_slabs ? 8 * a.R * cdiv(p.nz, 8) : a.R * p.nz;
  a.wt = wsb + p.off_wt; a.gx = g.s > 1 ? static_cast<void*>(wsb + p.off_gxq) : g_x;
  a.tabd = reinterpret_cast<uint8_t*>(wsb + p.off_tabd); a.tapd = tapd;
  a.ntap = p.staged ? reinterpret_cast<int*>(wsb + p.off_taps + sizeof(int4) * (size_t)q.nph * g.KK) : tapw + g.KK;
  a.Cip = p.Cip; a.PQ = q.PQ; a.qd = p.qd; a.nvd = p.nvd;
  a.d_tm = p.d_tm; a.d_tn = p.d_tn; a.nck = cdiv(g.Co, El<T>::KB);   // (a staged row's chunks are as many)
  a.nD = want_gx ? p.d_tm * p.d_tn * q.nph * p.d_nz : 0;
  a.d_nz = p.d_nz; a.d_its = p.d_its; a.d_grp = p.d_grp; a.d_ngrp = p.d_ngrp; a.d_first = p.d_first;
  a.partD = reinterpret_cast<float*>(wsb + p.off_pd); a.tickD = reinterpret_cast<int*>(wsb + p.off_tick);
  a.d_qv = FastDiv((uint32_t)p.qv); a.d_qd = FastDiv((uint32_t)p.qd);
  a.d_r = FastDiv((uint32_t)a.R); a.d_tiles = FastDiv((uint32_t)a.tiles); a.d_tx = FastDiv((uint32_t)a.tx);
  if (p.staged) {
    a.gt = wsb + p.off_gt; a.xt = wsb + p.off_xt; a.wr = wsb + p.off_wr;
    a.taps = reinterpret_cast<const int4*>(wsb + p.off_taps);
    a.Cop = p.Cop; a.Cix = p.Cix;
    a.H = g.H; a.W = g.W; a.Hy = g.Hy; a.Wy = g.Wy; a.Wq = q.Wq; a.Kw = g.Kw; a.s = g.s; a.d = g.dl; a.p = g.p;
    a.d_py = FastDiv((uint32_t)q.PY); a.d_wy = FastDiv((uint32_t)g.Wy); a.d_wq = FastDiv((uint32_t)q.Wq);
  }
  const dim3 grid(a.nW + a.nD);
  if (p.staged) {
    if (p.tn == 2) GF_LAUNCH((sgemm_k<2, 2>), grid, dim3(STile<2, 2>::NT), 0, st, a);
    else if (p.tm == 2) GF_LAUNCH((sgemm_k<2, 1>), grid, dim3(STile<2, 1>::NT), 0, st, a);
    else GF_LAUNCH((sgemm_k<1, 1>), grid, dim3(STile<1, 1>::NT), 0, st, a);
  } else if (p.tn == 2) GF_LAUNCH((xgemm_k<T, 2, 2>), grid, dim3(kT), 0, st, a);
  else if (p.tm == 2) GF_LAUNCH((xgemm_k<T, 2, 1>), grid, dim3(kT), 0, st, a);
  else GF_LAUNCH((xgemm_k<T, 1, 1>), grid, dim3(kT), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // ---- slab sums, interleave
  const bool inter = want_gx && g.s > 1;
  if (!want_gw && !inter) return e;
  FinalArgs f = {};
  f.part = a.part; f.g_w = g_w; f.pairs = g.Co * g.Ci; f.KK = g.KK; f.nz = p.nz;
  if (want_gw && g.KK == 1) {   // many slabs, few values: more lanes per value
    e = launch_finalize(a.part, g_w, f.pairs, p.nz, 1, 1.f, st);
    if (e != hipSuccess || !inter) return e;
  }
  f.w_blocks = want_gw && g.KK > 1 ? cdiv(f.pairs, 64) : 0;
  f.gxq = wsb + p.off_gxq; f.gx = g_x;
  f.NC = g.N * g.Ci; f.H = g.H; f.W = g.W; f.Hq = q.Hq; f.Wq = q.Wq; f.s = g.s;
  f.d_w = FastDiv((uint32_t)g.W); f.d_h = FastDiv((uint32_t)g.H); f.d_s = FastDiv((uint32_t)g.s);
  size_t lds = 0;
  int i_blocks = 0;
  if (inter) {
    f.ppb = interleave_planes(g, q);
    lds = f.ppb ? (size_t)q.nph * f.ppb * q.PQ * sizeof(T) + 16 : 0;
    i_blocks = f.ppb ? cdiv(f.NC, f.ppb) : cdiv(cdiv((long)f.NC * g.H * g.W, VE), kT);
  }
  GF_LAUNCH(xfinal_k<T>, dim3(f.w_blocks + i_blocks), dim3(kT), lds, st, f);
  return hipGetLastError();
}

template <class T>
hipError_t implicit_t(const Geom& g, const void* x, const void* w, const void* g_y, float* g_w, void* g_x,
                      void* ws, const XPlan& p, hipStream_t st) {
  const bool want_gw = g_w != nullptr, want_gx = g_x != nullptr;
  const XGeo q = make_xgeo(g);
  constexpr int VE = El<T>::VE;
  char* wsb = static_cast<char*>(ws);
  if (p.staged) {
    StageArgs t = {};
    t.taps = want_gx ? reinterpret_cast<int4*>(wsb + p.off_taps) : nullptr;
    t.ntap = reinterpret_cast<int*>(wsb + p.off_taps + sizeof(int4) * (size_t)q.nph * g.KK);
    t.tickets = reinterpret_cast<int*>(wsb + p.off_tick); t.ntickets = want_gx ? p.ntickets : 0;
    t.KK = g.KK; t.Kw = g.Kw; t.s = g.s; t.d = g.dl; t.p = g.p;
    auto job = [](const void* src, void* dst, int N, int C, int PX, int Cp) {
      return StageJob{src, dst, N, C, PX, Cp, cdiv(PX, 64), Cp / 64, N * cdiv(PX, 64) * (Cp / 64)};
    };
    t.job[0] = job(g_y, wsb + p.off_gt, g.N, g.Co, q.PY, p.Cop);
    if (want_gw) t.job[1] = job(x, wsb + p.off_xt, g.N, g.Ci, g.H * g.W, p.Cix);
    if (want_gx) t.job[2] = job(w, wsb + p.off_wr, 1, g.Co, g.Ci * g.KK, p.Cop);   // [c_o][c_i taps] -> [c_i taps][c_o]
    GF_LAUNCH(stage_k, dim3(1 + t.job[0].blocks + t.job[1].blocks + t.job[2].blocks), dim3(kT), 0, st, t);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : implicit_products<T>(g, q, p, nullptr, g_y, g_w, g_x, wsb, st);
  }
  int2* tapd = reinterpret_cast<int2*>(wsb + p.off_taps);   // 8-byte aligned: first in the region
  int* tapw = reinterpret_cast<int*>(tapd + (size_t)q.nph * g.KK);
  int* ntap = tapw + g.KK;
  // ---- set-up
  PrepArgs t;
  t.tabw = reinterpret_cast<uint8_t*>(wsb + p.off_tabw);
  t.tabd = reinterpret_cast<uint8_t*>(wsb + p.off_tabd);
  t.tapw = tapw; t.tapd = tapd; t.ntap = ntap;
  t.N = g.N; t.Ci = g.Ci; t.H = g.H; t.W = g.W; t.Hy = g.Hy; t.Wy = g.Wy; t.Hq = q.Hq; t.Wq = q.Wq;
  t.Kw = g.Kw; t.KK = g.KK; t.s = g.s; t.d = g.dl; t.p = g.p; t.nvw = p.nvw; t.nvd = p.nvd;
  t.tickets = reinterpret_cast<int*>(wsb + p.off_tick); t.ntickets = want_gx ? p.ntickets : 0;
  const int nmax = p.nvw > p.nvd * q.nph ? p.nvw : p.nvd * q.nph;
  const int tab_blocks = cdiv(std::max((long)g.KK * nmax, (long)t.ntickets), kT);
  const int w_blocks = want_gx ? g.Co * cdiv(p.Cip, kWPairs) : 0;
  const int x_blocks = (want_gw && g.s > 1) ? cdiv(cdiv((long)q.nph * g.N * g.Ci * q.PQ, VE), kT) : 0;
  GF_LAUNCH(prep_k<T>, dim3(tab_blocks + w_blocks + x_blocks), dim3(kT), 0, st, t, tab_blocks, w_blocks,
            static_cast<const T*>(w), reinterpret_cast<T*>(wsb + p.off_wt), g.Co, p.Cip, static_cast<const T*>(x),
            reinterpret_cast<T*>(wsb + p.off_xq));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return implicit_products<T>(g, q, p, g.s > 1 ? static_cast<const void*>(wsb + p.off_xq) : x, g_y, g_w, g_x, wsb, st);
}
// K slabs of the plain contraction part[z][co][ci] = sum_{n, p} a[n, co, p] * b[n, ci, p] over maps of P pixels
void plain_plan(const Geom& g, int* nz, int* cpz, int* nchunks) {
  *nchunks = cdiv((long)g.N * cdiv(g.P, 16 / g.b), 8);
  const long tiles = (long)cdiv(g.Co, 128) * cdiv(g.Ci, 128);
  const long z = std::max(1L, std::min(512 / tiles, (long)*nchunks / 4));
  *cpz = slab_chunks(*nchunks, z);
  *nz = cdiv(*nchunks, *cpz);
}

template <class T>
hipError_t plain_wgrad_t(const Geom& g, const void* x_u, const void* gy_u, float* part, int* nz_out,
                         hipStream_t st) {
  XArgs a = {};
  a.gy = gy_u; a.x = x_u; a.part = part;
  a.N = g.N; a.Ci = g.Ci; a.Co = g.Co; a.KK = 1;
  a.HW = g.P; a.HWy = g.P;
  a.qv = cdiv(g.P, El<T>::VE); a.kvecs = g.N * a.qv;
  plain_plan(g, &a.nz, &a.cpz, &a.nchunks);
  a.tx = cdiv(g.Ci, 128);
  a.tiles = a.tx * cdiv(g.Co, 128);
  a.R = a.tiles;
  a.xcd_slabs = deal_slabs(a.nz) ? 1 : 0;
  a.tot_x = g.N * g.Ci * g.P;
  a.tot_gy = g.N * g.Co * g.P;
  a.nW = a.xcd_slabs ? 8 * a.R * cdiv(a.nz, 8) : a.R * a.nz;
  a.d_qv = FastDiv((uint32_t)a.qv); a.d_qd = FastDiv(1u);
  a.d_r = FastDiv((uint32_t)a.R); a.d_tiles = FastDiv((uint32_t)a.tiles); a.d_tx = FastDiv((uint32_t)a.tx);
  *nz_out = a.nz;
  GF_LAUNCH((xgemm_k<T, 2, 2>), dim3(a.nW), dim3(kT), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// The filtered weight gradient (Eq. 5) of a large dense layer is the same contraction with one
// tap and no padding: these are the 128 x 128 tiles of the exact weight gradient on x_u and gy_u.
bool plain_wgrad_ok(const Geom& g) {
  const long lim = 2147483647L;
  if (g.g != 1 || g.Co < 128 || g.Ci < 128) return false;
  if ((long)g.N * g.Ci * g.P + 1024 >= lim || (long)g.N * g.Co * g.P + 1024 >= lim) return false;
  if ((long)g.N * up8(g.P) + 1024 >= lim || (long)g.N * g.Ci * g.P < 16 || (long)g.N * g.Co * g.P < 16) return false;
  return 2.0 * g.Co * g.Ci * g.N * g.P >= kPlainWgradMinFlops;
}

int plain_wgrad_splits(const Geom& g) {
  int nz, cpz, nch;
  plain_plan(g, &nz, &cpz, &nch);
  return nz;
}

hipError_t launch_plain_wgrad(const Geom& g, const void* x_u, const void* gy_u, float* part, int* nz_out,
                              hipStream_t st) {
  return g.dtype == GF_BF16 ? plain_wgrad_t<bf16_t>(g, x_u, gy_u, part, nz_out, st)
                            : plain_wgrad_t<float>(g, x_u, gy_u, part, nz_out, st);
}

// Dense layers whose tap offsets are constant in flattened pixels: stride 1 with W_y == W, or stride s with ceil(W / s) <= W_y
// (phase planes of pitch W_y); every index (plus the largest tap offset) below 2^31.
bool implicit_ok(const Geom& g) {
  const int ve = 16 / g.b;
  if (g.g != 1 || is_depthwise_layer(g) || g.KK > 1024 || g.s > 4) return false;
  if (g.s == 1 ? g.Wy != g.W : (g.W + g.s - 1) / g.s > g.Wy) return false;
  const XGeo q = make_xgeo(g);
  const long lim = 2147483647L;
  const long pqp = up8(q.PQ), pyp = up8(q.PY);
  const long reach = max_shift(g, q) + 1024;
  const long tx = (long)q.nph * g.N * g.Ci * q.PQ, ty = (long)g.N * g.Co * q.PY;
  if (tx < ve || ty < ve) return false;
  if (tx + reach + pqp >= lim || ty + reach + pyp >= lim) return false;
  if ((long)g.N * g.Ci * g.H * g.W >= lim) return false;
  if ((long)g.N * pqp + 1024 >= lim || (long)g.N * pyp + 1024 >= lim) return false;
  if ((long)g.KK * g.Co * g.Ci >= lim) return false;
  if (cdiv(g.Ci, 64) > 65535 || cdiv(g.Co, 64) > 65535) return false;
  if ((long)cdiv(g.Ci, 64) * cdiv(g.Co, 64) * g.KK * 8 * 130 >= lim) return false;  // one-dimensional grid
  return true;
}

// A 1 x 1 stride-1 layer without padding has no taps to shift: its maps are reduced maps of one-pixel patches, and the
// two-product launch of the filtered path computes both gradients from them, or where few channels meet many pixels one pass
// over the maps (gf_pixel.hip).
static bool plain_pointwise(const Geom& g, Geom* e) {
  if (g.KK != 1 || g.s != 1 || g.p != 0) return false;
  // (bf16 from 6 GFLOP per product on: 128-row tiles, 140 against 183 us for 2048 -> 256 channels, 64 x 64, N = 8)
  if (g.dtype == GF_BF16 && g.Co > 64 && g.Ci > 64 && 2.0 * g.Co * g.Ci * g.N * g.H * g.W >= kPlainWgradMinFlops) return false;
  *e = g;
  e->r = 2;            // (not vanilla: the map itself is what is contracted)
  e->rx = 1;
  e->Hp = g.H; e->Wp = g.W; e->P = g.H * g.W;
  return gemm_maps_ok(*e);
}

// The forms of a call, best first: f(staged, form) of each until it returns true
template <class F>
static void each_form(const Geom& g, bool want_gx, F&& f) {
  const bool staged = staged_ok(g, want_gx);
  if (staged && f(true, kFull)) return;
  const Form form = form_of(g);
  if (f(false, form) || (form == kFull && f(false, kSlim))) return;
  if (staged) f(true, kSlim);
}

size_t ws_implicit(const Geom& g, bool want_gw, bool want_gx) {
  Geom e;
  if (plain_pointwise(g, &e)) return pointwise_ok(e) ? ws_pointwise(e, want_gw) : ws_dense(e, want_gw, want_gx, true, false);
  size_t total = 0;
  each_form(g, want_gx, [&](bool staged, Form form) {
    total = plan_bytes(g, want_gw, want_gx, staged, form);
    return true;
  });
  return total;
}

// Layers of the one pass over the maps take the two products, layers on staged operands the maps themselves, and layers whose K is cut into
// many slabs fewer, with a workspace that only those fit: the copies are many times the rest (512 -> 512, 30 x 40, n = 128: 357 MB and 42).
// Either changes the order of the sums: of g_w, and in fp32 of g_x (bf16: the slabs of g_x are the same in all forms).
size_t ws_implicit_least(const Geom& g, bool want_gw, bool want_gx) {
  Geom e;
  if (plain_pointwise(g, &e)) return std::min(ws_implicit(g, want_gw, want_gx), ws_dense(e, want_gw, want_gx, true, false));
  size_t least = ~(size_t)0;
  each_form(g, want_gx, [&](bool staged, Form form) {
    least = std::min(least, plan_bytes(g, want_gw, want_gx, staged, form));
    return false;
  });
  return least;
}

// g_w and / or g_x (either may be null): one set-up launch, then the GEMM launches
hipError_t launch_implicit(const Geom& g, const void* x, const void* w, const void* g_y, float* g_w, void* g_x,
                           void* ws, size_t ws_bytes, hipStream_t st) {
  Geom e;
  const bool gw = g_w != nullptr, gx = g_x != nullptr;
  if (plain_pointwise(g, &e)) {
    if (pointwise_ok(e) && ws_bytes >= ws_implicit(g, gw, gx)) return launch_pointwise(e, g_y, x, w, g_w, g_x, ws, st);
    return launch_dense(e, g_y, false, x, w, nullptr, g_w, g_x, true, nullptr, ws, st);
  }
  hipError_t rc = hipErrorInvalidValue;   // (a workspace under ws_implicit_least: the entries refuse it)
  each_form(g, gx, [&](bool staged, Form form) {
    const XPlan p = make_plan(g, gw, gx, staged, form);
    if (ws_bytes < p.total) return false;
    rc = g.dtype == GF_BF16 ? implicit_t<bf16_t>(g, x, w, g_y, g_w, g_x, ws, p, st) : implicit_t<float>(g, x, w, g_y, g_w, g_x, ws, p, st);
    return true;
  });
  return rc;
}

}  // namespace gf
