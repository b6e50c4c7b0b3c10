// Both gradients of a pointwise layer with few channels on one side, in ONE pass over the maps:
//   g_w[co][ci]     = sum_{n, p} gy[n][co][p] x[n][ci][p]
//   g_x[n][ci][p]   = sum_co     w[co][ci]    gy[n][co][p]
// for fp32 1 x 1 stride-1 layers without the filter.
//
// Bound: memory, if every map is touched once.  As two products on 64 x 64 tiles (dense_gemm_k) such a layer reads gy
// twice, splits every fp32 operand once per tile that uses it and multiplies 64 columns of which 24 exist: 17 000 chunks of
// 64 x 64 x 32 for 24 -> 144 channels, 56 x 56, n = 32, which take a CU 0.6 us each.  Here a block walks over runs of
// KB pixels of ALL channels (128 bytes a row), splits each value once on its way into LDS and multiplies it from there
// twice: rows [channel][pixel] are K-major for the weight gradient and rows of k for the input gradient (transposing
// reads).  The weight gradient stays in registers until the block's last run; a slab per block, added by
// a launch of their own.  The kernel's fragments are split once per block.
#include "gf_gemm.h"

#include <algorithm>

namespace gf {

namespace {

constexpr int KB = El<float>::KB, VE = El<float>::VE;   // pixels of a run, of a 16-byte vector

struct PixArgs {
  int N, Ci, Co, PX;
  int cpi, chunks;            // runs of KB pixels per image, all
  int tot_gy, tot_x;
  const float *gy, *x, *w;
  float* part;                // [block][Co][Ci]; null: no weight gradient
  float* gx;                  // null: no input gradient
  FastDiv d_cpi;
};

// MT, NC: tiles of 32 output and input channels, one of them 1
template <int MT, int NC>
struct PixTile {
  static constexpr int RW = 64 + 16;                 // bytes of a row of a term: eight rows read together cover all banks
  static constexpr int RAW_RW = 128 + 16;            // ... of the values as they are
  static constexpr int ROWS = 32 * (MT + NC), kTerm = ROWS * RW;
  static constexpr int S = 33;                       // element stride of the staged sums
  static_assert(RAW_RW <= 3 * RW, "the second pass works in the same LDS");
  static constexpr int kOp = 3 * kTerm, kSum = 4 * 32 * S * 4;
  static constexpr bool EXPAND = MT > 1;             // the waves share K = c_o of the input gradient, else its tiles of c_i
  static constexpr int WT = (MT * NC + 3) / 4;       // weight-gradient tiles of a wave
  static constexpr int DT = EXPAND ? 1 : (NC + 3) / 4;            // input-gradient tiles of a wave
  static constexpr int KW = EXPAND ? (2 * MT + 3) / 4 : 2;        // its steps of 16 c_o
};

// one run's vectors of a lane
template <int RV>
struct PixSet {
  u32x4_t v[RV];
  int keep, n, p0, off;   // elements inside the plane, image, first pixel; off: a load had to be moved into its tensor
};

struct PixLow { uint32_t gy, x, w; };   // what the splits of the operands left (see split3)

// Runs [c0, c1): acc = the block's share of the weight gradient, g_x written.  RAW: the values as they are and
// v_mfma_f32_32x32x2_f32 -- the second pass of a block that met operands which three bf16 terms do not hold (split_failed):
// infinities, NaN, values past the largest bf16 or below 2^-110.  It forms only the gradients that such an operand enters.
// Both gradients with one value in 10^6 of g_y below 2^-110 / with none, us: 24 -> 144, 56 x 56, n = 32 50 / 33, 144 -> 24 55 / 41
// (dense_gemm_k 69 and 64; a product per lane and step instead of matrix instructions 812 and 562); g_x alone 32 / 21 and
// 30 / 20 (dense_gemm_k 28 and 28); one kernel value below 2^-110: 50 and 59 (64 and 49, a tile that has the value; 1175 and 1036).
template <int MT, int NC, bool RAG, bool RAW>
__device__ __forceinline__ void pixel_pass(const PixArgs& a, unsigned char* smem, int c0, int c1,
                                           bool want_w, bool want_d, f32x16 (&acc)[1][PixTile<MT, NC>::WT], PixLow& low, float& bad) {
  using L = PixTile<MT, NC>;
  constexpr int RV = MT + NC;                  // vectors of a lane per run
  constexpr int RW = RAW ? L::RAW_RW : L::RW;  // bytes of a row in LDS
  float* sums = reinterpret_cast<float*>(smem + L::kOp);
  const int tid = lane_id<typename std::conditional<RAW, raw_f32, float>::type>(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int vi = tid & 7, row0 = tid >> 3, r = lane & 31, kg = lane >> 5;
  const int wtiles = L::EXPAND ? (a.Co + 31) >> 5 : (a.Ci + 31) >> 5, nks = (a.Co + 15) >> 4;

  PixSet<RV> set;   // the next run, on its way
  auto fetch = [&](PixSet<RV>& s, int c) __attribute__((always_inline)) {
    const int n = s.n = (int)a.d_cpi.div((uint32_t)c);
    s.p0 = (c - n * a.cpi) * KB;
    const int p = s.p0 + vi * VE;
    s.keep = a.PX - p;
    const int q = RAG ? p : min(p, a.PX - VE);
    if constexpr (RAG) s.off = 0;
#pragma unroll
    for (int i = 0; i < RV; ++i) {
      const bool g = i < MT;
      if (!g && !want_w) break;   // (uniform)
      int o = (g ? n * a.Co + min(row0 + 32 * i, a.Co - 1) : n * a.Ci + min(row0 + 32 * (i - MT), a.Ci - 1)) * a.PX + q;
      if constexpr (RAG) {
        const int hi = (g ? a.tot_gy : a.tot_x) - VE;
        s.off |= o > hi;
        o = min(o, hi);
      }
      s.v[i] = load16<float, RAG>((g ? a.gy : a.x) + o);
    }
  };
  auto stage = [&](PixSet<RV>& s, uint32_t flip) __attribute__((always_inline)) {
    const u32x4_t m = keep_mask<float>(RAG ? s.keep : s.keep > 0 ? VE : 0);
#pragma unroll
    for (int i = 0; i < RV; ++i) {
      const bool g = i < MT;
      if (!g && !want_w) break;
      const int c = row0 + 32 * (g ? i : i - MT);
      if (8 * wave + 32 * (g ? i : i - MT) >= (g ? a.Co : a.Ci)) continue;   // (uniform for the wave)
      if constexpr (RAG) {
        if (s.off) {   // the vector at the very end of a tensor
          const int cc = min(c, (g ? a.Co : a.Ci) - 1), hi = (g ? a.tot_gy : a.tot_x) - VE;
          s.v[i] = shifted<float>(s.v[i], max(0, (s.n * (g ? a.Co : a.Ci) + cc) * a.PX + s.p0 + vi * VE - hi));
        }
      }
      if (c >= (g ? a.Co : a.Ci)) continue;
      u32x4_t u = s.v[i] & m;
      if (g) u ^= flip;
      unsigned char* d = smem + (row0 + 32 * i) * RW;
      if constexpr (RAW) {
        *reinterpret_cast<u32x4_t*>(d + vi * 16) = u;
      } else {
        uint2 t[3];
        split3<false>(u, t, g ? low.gy : low.x);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(d + k * L::kTerm + vi * 8) = t[k];
      }
    }
  };
  // rows of channels that do not exist: zeros, once
  for (int i = tid; i < (RAW ? 1 : 3) * L::ROWS * 8; i += kT) {
    const int row = i / 8 % L::ROWS, c = row < 32 * MT ? row : row - 32 * MT;
    if (c < (row < 32 * MT ? a.Co : a.Ci)) continue;
    if constexpr (RAW) *reinterpret_cast<uint4*>(smem + row * RW + i % 8 * 16) = make_uint4(0, 0, 0, 0);
    else *reinterpret_cast<uint2*>(smem + i / 8 / L::ROWS * L::kTerm + row * RW + i % 8 * 8) = make_uint2(0, 0);
  }
  if (c0 < c1) fetch(set, c0);

  // The kernel's fragments: lane holds c_i = lane % 32, c_o = 16 ks + 8 (lane / 32) .. + 7.  Where the waves share K, every
  // other one takes -w and is subtracted (the lean of the instruction's sums cancels, see mul_all).
  const int back = 3 - wave;   // the order of the waves here: wave 0 has a weight-gradient tile more
  constexpr int NF = RAW ? 2 : 3;   // vectors of a fragment: eight values, or their terms
  uint4 fw[L::DT][L::KW][NF];
#pragma unroll
  for (int i = 0; i < L::DT; ++i)
#pragma unroll
    for (int k = 0; k < L::KW; ++k) {
      const int ci = (L::EXPAND ? 0 : back + 4 * i) * 32 + r, co = (L::EXPAND ? back + 4 * k : k) * 16 + 8 * kg;
      __attribute__((aligned(16))) float e[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float val = want_d ? a.w[min(co + j, a.Co - 1) * a.Ci + min(ci, a.Ci - 1)] : 0.f;
        e[j] = ci < a.Ci && co + j < a.Co ? (L::EXPAND && (back & 1) ? -val : val) : 0.f;
      }
      if constexpr (RAW) {
#pragma unroll
        for (int t = 0; t < 2; ++t) fw[i][k][t] = reinterpret_cast<const uint4*>(e)[t];
      } else {
        uint2 t0[3], t1[3];
        split3<false>(reinterpret_cast<const u32x4_t*>(e)[0], t0, low.w);
        split3<false>(reinterpret_cast<const u32x4_t*>(e)[1], t1, low.w);
#pragma unroll
        for (int t = 0; t < 3; ++t) fw[i][k][t] = make_uint4(t0[t].x, t0[t].y, t1[t].x, t1[t].y);
      }
    }

  if (want_w) zero_acc(acc);
  auto terms = [&](const uint4 (&fa)[3], const uint4 (&fb)[3], f32x16 s) __attribute__((always_inline)) {   // smallest products first
    s = mma32(fa[2], fb[0], s);
    s = mma32(fa[0], fb[2], s);
    s = mma32(fa[1], fb[1], s);
    s = mma32(fa[1], fb[0], s);
    s = mma32(fa[0], fb[1], s);
    return mma32(fa[0], fb[0], s);
  };
  auto mul_raw = [&](uint32_t x, uint32_t y, f32x16 s) __attribute__((always_inline)) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x), __uint_as_float(y), s, 0, 0, 0);
  };
  auto wgrad = [&](float sign) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < L::WT; ++i) {
      const int q = wave + 4 * i;
      if (q >= wtiles) break;   // (uniform for the wave)
      const int ra = L::EXPAND ? 32 * q : 0, rb = 32 * MT + (L::EXPAND ? 0 : 32 * q);
      f32x16 s;
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
      for (int ks = 0; ks < (RAW ? 4 : 2); ++ks) {
        if constexpr (RAW) {
          const u32x4_t fa = *reinterpret_cast<const u32x4_t*>(smem + (ra + r) * RW + ks * 32 + kg * 16);
          const u32x4_t fb = *reinterpret_cast<const u32x4_t*>(smem + (rb + r) * RW + ks * 32 + kg * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) s = mul_raw(fa[e], fb[e], s);
        } else {
          uint4 fa[3], fb[3];
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            fa[t] = *reinterpret_cast<const uint4*>(smem + t * L::kTerm + (ra + r) * RW + ks * 32 + kg * 16);
            fb[t] = *reinterpret_cast<const uint4*>(smem + t * L::kTerm + (rb + r) * RW + ks * 32 + kg * 16);
          }
          s = terms(fa, fb, s);
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[0][i][e] = __builtin_fmaf(s[e], sign, acc[0][i][e]);
    }
  };
  // 16 c_o x 32 pixels of gy, transposed on the way (as they are: lane = pixel, eight rows)
  auto frag_gy = [&](uint4 (&fb)[NF], int ks) __attribute__((always_inline)) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
#pragma unroll
    for (int t = 0; t < NF; ++t) {
      if constexpr (RAW) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(smem + (ks * 16 + 8 * kg + 4 * t) * RW) + r;
        fb[t] = make_uint4(p[0], p[RW / 4], p[2 * RW / 4], p[3 * RW / 4]);
      } else {
        const unsigned char* p = smem + t * L::kTerm + (ks * 16 + 8 * kg + ((lane & 15) >> 2)) * RW + (lane & 16) * 2 + 8 * (lane & 3);
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
        const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * RW)));
        fb[t] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
    }
  };
  auto mul_frag = [&](const uint4 (&fa)[NF], const uint4 (&fb)[NF], f32x16 s) __attribute__((always_inline)) {
    if constexpr (!RAW) return terms(fa, fb, s);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s = mul_raw(fa[t].x, fb[t].x, s);
      s = mul_raw(fa[t].y, fb[t].y, s);
      s = mul_raw(fa[t].z, fb[t].z, s);
      s = mul_raw(fa[t].w, fb[t].w, s);
    }
    return s;
  };
  // a finished vector of g_x: row ci from pixel p on
  auto finish = [&](f32x4 f, int nn, int ci, int p, float sign) __attribute__((always_inline)) {
    if (ci >= a.Ci || p >= a.PX) return;
    float* d = a.gx + ((long)nn * a.Ci + ci) * a.PX + p;
    f *= sign;
    if (!RAG) {
      store_stream16(d, __builtin_bit_cast(uint4, f));
    } else if (p + VE <= a.PX) {
      const uint4 q = __builtin_bit_cast(uint4, f);
      *reinterpret_cast<Unal<float>*>(d) = Unal<float>{{q.x, q.y, q.z, q.w}};
    } else {
#pragma unroll
      for (int e = 0; e < VE; ++e)
        if (p + e < a.PX) d[e] = f[e];
    }
  };
  // One copy of the step, with a sign that changes at run time: the code of a block that lives for six runs is fetched more
  // often than it is repeated (13 KB; with copies for the two signs and for the ends, 24 - 31 KB, 144 -> 24 channels took 38 - 41 us instead of 36; a
  // second run on its way in registers changed nothing).
#pragma unroll 1
  for (int c = c0; c < c1; ++c) {   // odd runs of the whole layer are multiplied with the sign changed (see mul_all)
    const int nn = set.n, pp = set.p0;
    const float sign = c & 1 ? -1.f : 1.f;
    stage(set, (uint32_t)c << 31);
    lds_barrier();
    if (c + 1 < c1) fetch(set, c + 1);
    if (want_w) wgrad(sign);
    if constexpr (L::EXPAND) {
      if (want_d) {
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
        // (uniform for the wave: steps past c_o; their rows may lie past the operands)
        uint4 fb[L::KW][NF];
#pragma unroll
        for (int k = 0; k < L::KW; ++k)
          if (back + 4 * k < nks) frag_gy(fb[k], back + 4 * k);
        if constexpr (RAW) {
#pragma unroll
          for (int k = 0; k < L::KW; ++k)
            if (back + 4 * k < nks) s = mul_frag(fw[0][k], fb[k], s);
        } else {
          auto all = [&](int ta, int tb) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < L::KW; ++k)
              if (back + 4 * k < nks) s = mma32(fw[0][k][ta], fb[k][tb], s);
          };
          all(2, 0); all(0, 2); all(1, 1); all(1, 0); all(0, 1); all(0, 0);   // smallest products first
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          bad = __builtin_fmaf(s[e], 0.f, bad);
          sums[(wave * 32 + acc_row(lane, e)) * L::S + r] = s[e];
        }
      }
      lds_barrier();
      if (want_d) {
        f32x4 f;
        const float* src = sums + row0 * L::S + vi * VE;
#pragma unroll
        for (int e = 0; e < VE; ++e)   // waves 0 and 2 took -w
          f[e] = (src[3 * 32 * L::S + e] - src[2 * 32 * L::S + e]) + (src[32 * L::S + e] - src[e]);
        finish(f, nn, row0, pp + vi * VE, sign);
      }
    } else {
      if (want_d) {
#pragma unroll
        for (int i = 0; i < L::DT; ++i) {
          const int tile = back + 4 * i;
          if (tile >= wtiles) break;   // (uniform for the wave)
          f32x16 s;
#pragma unroll
          for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            if (k >= nks) break;
            uint4 fb[NF];
            frag_gy(fb, k);
            s = mul_frag(fw[i][k], fb, s);
          }
          float* cs = sums + wave * 32 * L::S;   // (this wave's own: no barrier)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            bad = __builtin_fmaf(s[e], 0.f, bad);
            cs[acc_row(lane, e) * L::S + r] = s[e];
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          constexpr int PV = 32 / VE;   // vectors of a row of the tile
#pragma unroll
          for (int h = 0; h < 32 * PV / 64; ++h) {
            const int row = (lane + 64 * h) / PV, col = (lane + 64 * h) % PV * VE;
            f32x4 f;
#pragma unroll
            for (int e = 0; e < VE; ++e) f[e] = cs[row * L::S + col + e];
            finish(f, nn, tile * 32 + row, pp + col, sign);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
      }
      lds_barrier();
    }
  }
}

template <int MT, int NC, bool RAG>
__global__ __launch_bounds__(kT, 2) void pointwise_k(PixArgs a) {
  using L = PixTile<MT, NC>;
  __shared__ __attribute__((aligned(16))) unsigned char smem[L::kOp + L::kSum];
  const int c0 = (int)((long)blockIdx.x * a.chunks / gridDim.x), c1 = (int)((long)(blockIdx.x + 1) * a.chunks / gridDim.x);
  f32x16 acc[1][L::WT];
  zero_acc(acc);
  PixLow low = {0, 0, 0};
  float bad = 0.f;
  pixel_pass<MT, NC, RAG, false>(a, smem, c0, c1, a.part != nullptr, a.gx != nullptr, acc, low, bad);
  const bool again_w = a.part && split_failed(acc, low.gy | low.x);   // (uniform)
  const bool again_d = a.gx && __syncthreads_or(((low.gy | low.w) & 0xffffu) != 0 || bad != 0.f);
  if (again_w || again_d) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stores of g_x so far, of every wave, before the second ones
    __syncthreads();
    pixel_pass<MT, NC, RAG, true>(a, smem, c0, c1, again_w, again_d, acc, low, bad);
  }
  if (a.part) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31;
    float* d = a.part + (long)blockIdx.x * a.Co * a.Ci;
#pragma unroll
    for (int i = 0; i < L::WT; ++i) {
      const int q = wave + 4 * i;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int co = (L::EXPAND ? 32 * q : 0) + acc_row(lane, e), ci = (L::EXPAND ? 0 : 32 * q) + r;
        if (co < a.Co && ci < a.Ci) d[co * a.Ci + ci] = acc[0][i][e];
      }
    }
  }
}

// g_w = sum of the slabs, in 64 bits: 512 of them, added in 32, would round as often as the runs themselves.
// 16 values per block, 16 lanes per value with their loads in flight together.
__global__ __launch_bounds__(kT) void pixel_slabs_k(const float* part, float* g_w, int pairs, int nz) {
  __shared__ double red[16][17];
  const int o = threadIdx.x & 15, zg = threadIdx.x >> 4, e = blockIdx.x * 16 + o;
  double s = 0.;
  if (e < pairs) {
    for (int z = zg; z < nz; z += 8 * 16) {
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = part[(long)min(z + 16 * k, nz - 1) * pairs + e];   // clamped: always issued
#pragma unroll
      for (int k = 0; k < 8; ++k) s += z + 16 * k < nz ? (double)v[k] : 0.;
    }
  }
  red[zg][o] = s;
  __syncthreads();
  if (zg == 0 && e < pairs) {
    double t = 0.;
#pragma unroll
    for (int k = 0; k < 16; ++k) t += red[k][o];
    g_w[e] = (float)t;
  }
}

struct PixPlan { int cpi, chunks, blocks; };

// two blocks per CU, what LDS holds; 384, 640, 768 and 1024 blocks: 35, 40, 41 and 40 us where 512 take 31 (24 -> 144, 56 x 56,
// n = 32)
PixPlan make_plan(const Geom& g) {
  PixPlan p;
  p.cpi = cdiv(g.P, KB);
  p.chunks = g.N * p.cpi;
  p.blocks = std::min(p.chunks, 512);
  return p;
}

template <int MT, int NC>
void launch_tile(const PixArgs& a, int blocks, hipStream_t st) {
  if constexpr (MT > 1) {   // (planes of whole vectors otherwise: pointwise_ok)
    if (a.PX % VE != 0) {
      GF_LAUNCH((pointwise_k<MT, NC, true>), dim3(blocks), dim3(kT), 0, st, a);
      return;
    }
  }
  GF_LAUNCH((pointwise_k<MT, NC, false>), dim3(blocks), dim3(kT), 0, st, a);
}

}  // namespace

// Layers the pass above takes: fp32, at most 32 channels on one side and 33 to 192 on the other, and enough pixels for a
// few runs per block -- whichever gradients are asked for, so that each has the same bits alone and beside the other.  g: the
// layer with its pixels as P, sizes as gemm_maps_ok wants them.  Both gradients, g_w alone, g_x alone in us, dense_gemm_k / one pass
// (buffers rotating over 600 MB):
//   24 -> 144, 56 x 56, n = 32 48 / 32, 40 / 25, 26 / 21; 3 -> 64, 112 x 112, n = 16 41 / 28, 37 / 22, 25 / 19; 32 -> 192, 64 x 64,
//   n = 24 50 / 40, 40 / 30, 30 / 24; n = 12 (1536 runs) 30 / 27, 20 / 22, 18 / 14; 3 -> 40 17 / 12, 13 / 11, 7.8 / 7.0
//   planes at any alignment: 24 -> 144, 57 x 55, n = 32 50 / 36, 43 / 27, 28 / 25; 3 -> 192, 47 x 49, n = 30 (2160 runs) 39 / 30, 34 / 25, 24 / 21
// and on the other side
//   24 -> 144, 28 x 28, n = 32 (800) 17.0 / 20.5; 144 -> 24 18.0 / 21.4; 96 -> 32, 39 x 41, n = 32 (1600) 24.9 / 24.5;
//   32 -> 32, 80 x 80, n = 16 21.7 / 22.4; bf16, whose products need no split: 144 -> 24, 56 x 56, n = 32 27 / 31
// Many channels on the input side: a run of g_x is 128 bytes of each row.  Where rows do not start on lines or half lines every
// line is written in two pieces, 5 us apart, while 64 blocks of an XCD move more than its L2 holds: planes of 16 k pixels only.
//   144 -> 24, 56 x 56, n = 32 47 / 40, 39 / 26, 27 / 19; 28 x 28, n = 128, 144 -> 16 49 / 43, 41 / 26, 28 / 21; 96 -> 32 41 / 33, 34 / 22, 21 / 16
//   57 x 56 (3192 pixels), n = 32, 144 -> 24 49 / 59, 40 / 28, 28 / 37; 192 -> 16 52 / 74, 40 / 30, 31 / 49; 57 x 55 55 / 80 (192 -> 24)
// Not with 161 or more of them for more than 16 outputs either, whose waves have two tiles and two steps of each: 192 -> 32,
// 64 x 64, n = 12 30 / 35, 21 / 23, 15 / 15, n = 24 48 / 49, 40 / 31, 29 / 21; 28 x 28, n = 128 53 / 59; 192 -> 16, 64 x 64, n = 12 29 / 26,
// 19 / 19, 15 / 13.  Up to 64 of them, which are a tile there as here, from twice the runs on: 40 -> 16, 64 x 64, n = 12 14.3 / 12.7,
// 11.8 / 11.5, 6.4 / 7.3; 48 x 48, n = 22 14.9 / 13.8, 13.0 / 12.0, 7.1 / 8.1; 56 x 56, n = 32 (3136) 20 / 17, 17 / 15, 10.9 / 10.5.
bool pointwise_ok(const Geom& g) {
  const int mt = cdiv(g.Co, 32), nc = cdiv(g.Ci, 32);
  if (g.dtype != GF_F32 || std::min(mt, nc) != 1 || std::max(mt, nc) < 2 || std::max(mt, nc) > 6) return false;
  if (nc > 1 && (g.P % 16 != 0 || (nc > 5 && g.Co > 16))) return false;
  return make_plan(g).chunks >= (nc == 2 ? 3072 : g.P % VE == 0 ? 1536 : 2048);
}

size_t ws_pointwise(const Geom& g, bool want_w) {
  // (never 0: a caller that passes no workspace is told so)
  return std::max<size_t>(want_w ? (size_t)make_plan(g).blocks * g.Co * g.Ci * sizeof(float) : 0, 256);
}

hipError_t launch_pointwise(const Geom& g, const void* gy, const void* x, const void* w, float* g_w, void* g_x, void* ws,
                            hipStream_t st) {
  const PixPlan p = make_plan(g);
  PixArgs a = {};
  a.N = g.N; a.Ci = g.Ci; a.Co = g.Co; a.PX = g.P;
  a.cpi = p.cpi; a.chunks = p.chunks;
  a.tot_gy = g.N * g.Co * g.P; a.tot_x = g.N * g.Ci * g.P;
  a.gy = static_cast<const float*>(gy); a.x = static_cast<const float*>(x); a.w = static_cast<const float*>(w);
  a.part = g_w ? static_cast<float*>(ws) : nullptr;
  a.gx = static_cast<float*>(g_x);
  a.d_cpi = FastDiv((uint32_t)p.cpi);
  const int mt = cdiv(g.Co, 32), nc = cdiv(g.Ci, 32);
  if (mt > 5) launch_tile<6, 1>(a, p.blocks, st);
  else if (mt > 4) launch_tile<5, 1>(a, p.blocks, st);
  else if (mt > 2) launch_tile<4, 1>(a, p.blocks, st);
  else if (mt > 1) launch_tile<2, 1>(a, p.blocks, st);
  else if (nc > 5) launch_tile<1, 6>(a, p.blocks, st);
  else if (nc > 4) launch_tile<1, 5>(a, p.blocks, st);
  else if (nc > 2) launch_tile<1, 4>(a, p.blocks, st);
  else launch_tile<1, 2>(a, p.blocks, st);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !g_w) return e;
  const int pairs = g.Co * g.Ci;
  GF_LAUNCH(pixel_slabs_k, dim3(cdiv(pairs, 16)), dim3(kT), 0, st, a.part, g_w, pairs, p.blocks);
  return hipGetLastError();
}

}  // namespace gf
