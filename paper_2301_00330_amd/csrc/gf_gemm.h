// Building blocks of the two-product GEMM kernels (gf_dense.hip: filtered backward, gf_implicit.hip: vanilla BP):
// 256-lane blocks, four waves in a 2 x 2 arrangement on 64 TM x 64 TN tiles, v_mfma_f32_32x32x16_bf16, operands
// global -> registers -> LDS -> registers; fp32 operands as three bf16 terms; signed 8-bit codes with
// v_mfma_i32_32x32x32_i8, whose fragments are the same 16 bytes with twice the k.
#pragma once

#include "gf_internal.h"
#include "gf_mma.h"

#include <type_traits>

namespace gf {

constexpr int kT = 256;

template <class T> struct El;
// elements per 128-byte chunk / 16-byte vector, matrix steps per chunk, bytes of an element (of a term) in LDS, accumulator
template <> struct El<float> { static constexpr int KB = 32, VE = 4, KS = 2, EB = 2; typedef f32x16 acc; };
template <> struct El<bf16_t> { static constexpr int KB = 64, VE = 8, KS = 4, EB = 2; typedef f32x16 acc; };
// fp32 operands multiplied as they are, v_mfma_f32_32x32x2_f32 (a tile's second pass: see split_failed)
struct raw_f32 { float v; };
template <> struct El<raw_f32> { static constexpr int KB = 32, VE = 4, KS = 4, EB = 4; typedef f32x16 acc; };
template <> struct Unal<raw_f32> : Unal<float> {};
template <> struct El<int8_t> { static constexpr int KB = 128, VE = 16, KS = 4, EB = 1; typedef i32x16 acc; };

// the lane's number in the block; in a second pass as a value of its own, so that nothing derived from it is kept in
// registers through the first
template <class T>
__device__ __forceinline__ int lane_id() {
  int t = threadIdx.x;
  if (__is_same(T, raw_f32)) asm volatile("" : "+v"(t));
  return t;
}

template <class T> constexpr bool is_split() { return __is_same(T, float); }
template <class T> constexpr int terms_of() { return is_split<T>() ? 3 : 1; }   // bf16 terms of an operand

// Accumulators of a wave: TM x TN tiles of 32 x 32; row of such a tile that element v of lane
// `lane` holds (the column is lane % 32).  Tile (i, j) of wave (wm, wn) covers rows 64 i + 32 wm .. of the block
// tile and columns 64 j + 32 wn .., so 64 consecutive rows are complete per i.
__device__ __forceinline__ int acc_row(int lane, int v) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

template <class A, int TM, int TN>
__device__ __forceinline__ void zero_acc(A (&acc)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
}

// Four fp32 values as three bf16 terms, x = t0 + t1 + t2 exactly: every term is the nearest bf16 of what the
// earlier ones leave (|t1| <= 2^-8 |x|, |t2| <= 2^-16 |x|), both remainders are exact in fp32, and the second
// has at most 8 significant bits.  A product x y is taken as the six term products of order <= 2; the three
// that are dropped stay below 2^-23 |x y| (2^-24 at most and 2^-27 rms over random operands): the size of one
// rounding of the fp32 accumulation.  One packed
// conversion per pair of values and term, two shifts / masks and two subtractions per pair and remainder.
// The split is not exact for every value.  Below about 2^-110 the last term reaches under the smallest bf16: the
// second remainder then has bits set below the upper 16, and `low` collects them (one instruction per pair).  An
// infinity, a NaN or a value that rounds past the largest bf16 (3.39e38) leaves inf - inf in the remainders, and every sum it
// enters is not finite.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
template <bool NEG>   // the terms of -x (a sign modifier of the instructions)
__device__ __forceinline__ void split3(const u32x4_t& v, uint2 (&t)[3], uint32_t& low) {
  f32x2_t a = {__uint_as_float(v.x), __uint_as_float(v.y)}, b = {__uint_as_float(v.z), __uint_as_float(v.w)};
  if (NEG) { a = -a; b = -b; }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    // one packed conversion per pair (round to nearest even)
    const uint32_t pa = __builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf16x2_t));
    const uint32_t pb = __builtin_bit_cast(uint32_t, __builtin_convertvector(b, bf16x2_t));
    t[k] = make_uint2(pa, pb);
    if (k < 2) {
      a.x -= bf_lo(pa); a.y -= bf_hi(pa);
      b.x -= bf_lo(pb); b.y -= bf_hi(pb);
    }
  }
  low |= __float_as_uint(a.x) | __float_as_uint(a.y);
  low |= __float_as_uint(b.x) | __float_as_uint(b.y);
  asm volatile("" : "+v"(low));   // now: else the remainders stay in registers
}

// True in all lanes of a block if a product of one of its lanes may not be what fp32 operands give: the block then takes
// its K slab again with fp32 matrix instructions (raw_f32).  One look at the accumulators per block and slab.
template <int TM, int TN>
__device__ __forceinline__ bool split_failed(const f32x16 (&acc)[TM][TN], uint32_t low) {
  float s = 0.f;   // x * 0 is 0, or NaN for an infinity or a NaN
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) s = __builtin_fmaf(acc[i][j][v], 0.f, s);
  return __syncthreads_or((low & 0xffffu) != 0 || s != 0.f) != 0;
}

// Barrier between the waves of a block that orders LDS traffic only.  __syncthreads() also waits
// for every global load in flight (its fence covers all address spaces), which would end the
// prefetch of the next chunk at every barrier: measured 1.7 us per chunk instead of 0.4.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// K loop over chunks [kc0, kc1): register set -> LDS, barrier, the load of a later chunk into the freed set,
// matrix instructions, barrier.  A global load takes 1.5 - 2 us here, several chunks of work, so NS - 1 chunks are
// in flight in registers beside the one in LDS; the sets have fixed roles per step (arrays indexed at run time
// would live in scratch memory).  Whole rounds of NS steps without a branch inside (the compiler then knows how many
// loads are in flight at every wait; with conditional steps it drains all of them at the loop head), then the
// chunks that are left, already on their way.  fetch(set, kc) clamps kc itself.  stage and mul are told whether the
// chunk is an odd one (see mul_all).
template <int NS, class Set, class F, class S, class M>
__device__ __forceinline__ void k_loop(int kc0, int kc1, F&& fetch, S&& stage, M&& mul) {
  static_assert(NS == 2 || NS == 4, "register sets");
  auto step = [&](Set& cur, Set& nxt, int kc, bool more, auto neg) __attribute__((always_inline)) {
    stage(cur, kc, neg);
    lds_barrier();
    if (more) fetch(nxt, kc + NS - 1);
    mul(neg);
    lds_barrier();
  };
  constexpr std::integral_constant<bool, false> pos{};
  constexpr std::integral_constant<bool, true> neg{};
  Set s0, s1;
  fetch(s0, kc0);
  int kc = kc0;
  if constexpr (NS == 2) {
    for (; kc + 2 <= kc1; kc += 2) {
      step(s0, s1, kc, true, pos);
      step(s1, s0, kc + 1, true, neg);
    }
    if (kc < kc1) step(s0, s1, kc, false, pos);
  } else {
    Set s2, s3;
    fetch(s1, kc0 + 1);
    fetch(s2, kc0 + 2);
    for (; kc + 4 <= kc1; kc += 4) {
      step(s0, s3, kc, true, pos);
      step(s1, s0, kc + 1, true, neg);
      step(s2, s1, kc + 2, true, pos);
      step(s3, s2, kc + 3, true, neg);
    }
    if (kc < kc1) step(s0, s3, kc, false, pos);
    if (kc + 1 < kc1) step(s1, s0, kc + 1, false, neg);
    if (kc + 2 < kc1) step(s2, s1, kc + 2, false, pos);
  }
}

// 16 bytes: aligned, or (RAG) at element alignment
template <class T, bool RAG>
__device__ __forceinline__ u32x4_t load16(const T* p) {
  if constexpr (!RAG) return *reinterpret_cast<const u32x4_t*>(p);
  const uint4 v = load_vec<T>(p);
  return u32x4_t{v.x, v.y, v.z, v.w};
}
template <class T>
__device__ __forceinline__ u32x4_t shifted(const u32x4_t& v, int sh) {
  const uint4 r = realign<T>(make_uint4(v.x, v.y, v.z, v.w), sh);
  return u32x4_t{r.x, r.y, r.z, r.w};
}
// AND words that keep the first `keep` elements of a vector
template <class T>
__device__ __forceinline__ u32x4_t keep_mask(int keep) {
  u32x4_t m;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (sizeof(T) == 4) m[i] = i < keep ? 0xffffffffu : 0u;
    else if (sizeof(T) == 1) m[i] = keep >= 4 * i + 4 ? 0xffffffffu : keep <= 4 * i ? 0u : (1u << (8 * (keep - 4 * i))) - 1u;
    else m[i] = 2 * i + 1 < keep ? 0xffffffffu : 2 * i < keep ? 0x0000ffffu : 0u;
  }
  return m;
}

// s += the six term products of two fp32 operands, smallest first
__device__ __forceinline__ void add_products(const uint4 (&fa)[3], const uint4 (&fb)[3], f32x16& s) {
  s = mma32(fa[2], fb[0], s);
  s = mma32(fa[0], fb[2], s);
  s = mma32(fa[1], fb[1], s);
  s = mma32(fa[1], fb[0], s);
  s = mma32(fa[0], fb[1], s);
  s = mma32(fa[0], fb[0], s);
}

// Matrix step ks of a chunk, all tiles.  fp32: the term products are summed from zero -- those of a whole chunk of 32 k
// for a single tile, of 16 k otherwise (a sum per tile would not fit the registers; two tiles of a filtered input gradient are taken
// one after the other instead, d_mainloop of gf_dense.hip) -- and then added to the accumulator
// with one rounding; straight into the accumulator they would round it 24 times per chunk.  And the instruction takes
// the sum of eight products down to a multiple of about 2^-23 of the largest one, towards minus infinity: with 35e6
// products per output every weight gradient came out 0.4 below values of 5e3.  So every other chunk is multiplied with
// the sign of its first operand changed and subtracted, and the lean cancels.  Error of g_w against 64-bit sums, 60 random
// layers: 0.55 (vanilla) and 0.69 (filtered) of what fp32 matrix instructions gave, g_x 0.41 and 0.60; before these two
// measures g_w stood at 1.18.  They cost 2 - 3 % of a matrix-bound layer, 8 % on 128 x 128 tiles (vanilla, 256 channels, 59 x
// 65, n = 2: 169 -> 185 us).  Straight into an accumulator that changes its sign with the chunk: no faster (188 us), and
// g_w at 1.08 and 1.15.
template <class T, bool NEG, int TM, int TN>
__device__ __forceinline__ void mul_all(const uint4 (&fa)[TM][terms_of<T>()], const uint4 (&fb)[TN][terms_of<T>()],
                                        typename El<T>::acc (&acc)[TM][TN], typename El<T>::acc& s, int ks) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if constexpr (is_split<T>()) {
        if (TM * TN > 1 || ks == 0)
#pragma unroll
          for (int v = 0; v < 16; ++v) s[v] = 0.f;
        add_products(fa[i], fb[j], s);
        if (TM * TN > 1 || ks == El<T>::KS - 1) {
          if (NEG) acc[i][j] -= s;
          else acc[i][j] += s;
          // here: left to the end of a round of steps, the sums would stay in registers of their own
          asm volatile("" : "+v"(acc[i][j]));
        } else {
          __builtin_amdgcn_sched_barrier(0);
        }
      } else if constexpr (__is_same(T, raw_f32)) {
        const u32x4_t x = {fa[i][0].x, fa[i][0].y, fa[i][0].z, fa[i][0].w}, y = {fb[j][0].x, fb[j][0].y, fb[j][0].z, fb[j][0].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(x[e]), __uint_as_float(y[e]), acc[i][j], 0, 0, 0);
      } else {
        acc[i][j] = mma32(fa[i][0], fb[j][0], acc[i][j]);
      }
    }
}

// Rows of k in LDS: C columns, in blocks of 32 (64 bytes; codes: 32) whose order within the row depends on k, so that
// the four rows (codes: eight) that a transposing read takes together fall into different banks.
template <class T, int C>
__device__ __forceinline__ int swz(int k) {
  if (El<T>::EB == 4 || C == 32) return 0;
  const int r = El<T>::EB == 2 ? k : k >> 1;
  return C == 64 ? (r >> 1) & 1 : r & 3;
}

// vector cv of row k into such a tile (fp32: into the three term tiles)
template <class T, int C, bool NEG = false>
__device__ __forceinline__ void put_row(unsigned char* tile, int k, int cv, const u32x4_t& v, uint32_t& low) {
  constexpr int VE = El<T>::VE, VPB = 32 / VE;   // vectors per block of 32 columns
  constexpr int EB = El<T>::EB;
  unsigned char* d = tile + k * (C * EB) + (((cv / VPB) ^ swz<T, C>(k)) * VPB + cv % VPB) * (VE * EB);
  if constexpr (is_split<T>()) {
    uint2 t[3];
    split3<NEG>(v, t, low);
#pragma unroll
    for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(d + q * (El<T>::KB * C * 2)) = t[q];
  } else {
    *reinterpret_cast<u32x4_t*>(d) = v;
  }
}

// the operand of one MFMA -- lane: column c0 + lane % 32, k = 16 ks + 8 (lane / 32) .. + 7, codes: 32 ks + 16 (lane / 32)
// .. + 15; fp32 as it is: 8 ks + 4 (lane / 32) .. + 3 -- from such a tile.  ds_read_b64_tr_b16: sixteen lanes read a block of 4 x 16 and each gets one column of
// four, lanes 4 r .. 4 r + 3 pointing to row r; ds_read_b64_tr_b8: 8 x 16, columns of eight, lanes 2 r and 2 r + 1.
template <class T, int C>
__device__ __forceinline__ uint4 frag_tr(const unsigned char* tile, int ks, int c0, int lane) {
  uint2 a, b;
  if constexpr (El<T>::EB == 4) {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(tile) + (ks * 8 + 4 * (lane >> 5)) * C + c0 + (lane & 31);
    return make_uint4(p[0], p[C], p[2 * C], p[3 * C]);
  } else if constexpr (El<T>::EB == 2) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const int k = ks * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int in_blk = (lane & 16) + 4 * (lane & 3);       // column within the block of 32
    const unsigned char* p = tile + k * (C * 2) + (((c0 >> 5) ^ swz<T, C>(k)) * 32 + in_blk) * 2;   // k and k + 4 share the order
    a = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
    b = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * C * 2)));
  } else {
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) i32x2 lds_i32x2;
    const int k = ks * 32 + 16 * (lane >> 5) + ((lane & 15) >> 1);
    const int in_blk = (lane & 16) + 8 * (lane & 1);
    const unsigned char* p = tile + k * C + ((c0 >> 5) ^ swz<T, C>(k)) * 32 + in_blk;               // k and k + 8 share it
    a = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)p));
    b = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)(p + 8 * C)));
  }
  return make_uint4(a.x, a.y, b.x, b.y);
}

// Slab data crosses XCDs inside one launch.  Every XCD has an L2 of its own, and a device-wide
// release / acquire fence writes back resp. invalidates that whole L2, which every block of the grid
// would pay (measured: 5 - 8 x the run time of the whole launch).  The slabs therefore move with
// relaxed device-scope atomic stores and loads, which go through to the memory side and never
// leave a stale or dirty line in an L2; the ticket is a device-scope atomic as well, and every wave
// waits for its stores to be acknowledged (s_waitcnt vmcnt(0)) before the barrier ahead of the ticket.
// A workgroup-scope release fence is not enough there: inside one work-group it orders nothing that
// leaves the CU, compiles to no wait for stores, and the block with the last ticket then now and then
// added slabs that were still on their way.
template <class V>   // float or int
__device__ __forceinline__ void slab_store(float* p, V x, V y) {
  const uint64_t v = (uint64_t)__builtin_bit_cast(uint32_t, x) | ((uint64_t)__builtin_bit_cast(uint32_t, y) << 32);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t slab_load(const float* p) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// element pair q of the lane's 16 of tile (i, j): slab[((i TN + j) 8 + q) 512 + 2 lane]
// (mw, nw: rows and columns of the matrix from this wave's first ones on; tiles wholly outside are left out)
template <int TM, int TN, int NT = kT, class A>
__device__ __forceinline__ void put_slab(const A (&acc)[TM][TN], float* slab, int mw, int nw) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      if (64 * i < mw && 64 * j < nw)   // (uniform for the wave)
#pragma unroll
      for (int q = 0; q < 8; ++q)
        slab_store(slab + (((i * TN + j) * 8 + q) * NT + threadIdx.x) * 2, acc[i][j][2 * q], acc[i][j][2 * q + 1]);
}

// one block's ticket of `count`: true in the block that takes the last one (all stores made before it are complete)
__device__ __forceinline__ bool last_ticket(int* ticket, int count, int* s_flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores have reached the memory side ...
  __syncthreads();                                    // ... and so have the other waves'
  if (threadIdx.x == 0) {
    const bool last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == count - 1;
    if (last) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
    *s_flag = last;
  }
  __syncthreads();
  const bool last = *s_flag != 0;
  __syncthreads();
  return last;
}

// acc = slab 0 + slab 1 + ... in slab order, a few slabs' loads in flight at a time.  Integer slabs are added in 64
// bits; a final sum leaves as the bits of the nearest float.
template <int TM, int TN, int NT = kT, class A>
__device__ __forceinline__ void sum_slabs(A (&acc)[TM][TN], const float* slabs, int nz, int mw, int nw, bool final) {
  constexpr int SZ = 16 * NT * TM * TN, ZB = 4;
  constexpr bool INT = __is_same(A, i32x16);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {   // 16 floats per lane and pass
      if (64 * i >= mw || 64 * j >= nw) continue;
      typename std::conditional<INT, long long, float>::type s[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = 0;
      const float* p0 = slabs + ((i * TN + j) * 8 * NT + threadIdx.x) * 2;
      for (int z0 = 0; z0 < nz; z0 += ZB) {
        uint64_t t[ZB][8];
#pragma unroll
        for (int zz = 0; zz < ZB; ++zz)
#pragma unroll
          for (int q = 0; q < 8; ++q) t[zz][q] = slab_load(p0 + (long)min(z0 + zz, nz - 1) * SZ + q * (2 * NT));   // clamped: always issued
#pragma unroll
        for (int zz = 0; zz < ZB; ++zz)
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if (z0 + zz < nz) {
              typedef typename std::conditional<INT, int, float>::type V;
              s[2 * q] += __builtin_bit_cast(V, (uint32_t)t[zz][q]);
              s[2 * q + 1] += __builtin_bit_cast(V, (uint32_t)(t[zz][q] >> 32));
            }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        if constexpr (INT) acc[i][j][e] = final ? __float_as_int((float)s[e]) : (int)s[e];
        else acc[i][j][e] = s[e];
      }
    }
}

// The partial tile of this block goes to slab z of its tile, in the order the lanes hold it (every store and load
// is one contiguous 1 KB run per wave).  Slabs are summed in groups of `grp`: the block that completes a group adds
// it into the group's own slab, the block that completes the last group adds those (one level where there is one
// group: a block adds a slab of 16 KB in 0.2 - 0.4 us, so 128 slabs one after the other would take longer than the
// launch).  True in that block, with acc = the sum.  tickets: one for the tile, one per group.
template <int TM, int TN, int NT = kT, class A>
__device__ __forceinline__ bool reduce_slabs(A (&acc)[TM][TN], float* slabs, int z, int* tickets, int nz, int grp,
                                             int ngrp, int* s_flag, int mw, int nw) {
  constexpr long SZ = 16 * NT * TM * TN;
  const int gi = z / grp, in_grp = min(grp, nz - gi * grp);
  put_slab<TM, TN, NT>(acc, slabs + z * SZ, mw, nw);
  if (!last_ticket(tickets + 1 + gi, in_grp, s_flag)) return false;
  sum_slabs<TM, TN, NT>(acc, slabs + gi * grp * SZ, in_grp, mw, nw, ngrp == 1);
  if (ngrp == 1) return true;
  float* sums = slabs + nz * SZ;
  put_slab<TM, TN, NT>(acc, sums + gi * SZ, mw, nw);
  if (!last_ticket(tickets, ngrp, s_flag)) return false;
  sum_slabs<TM, TN, NT>(acc, sums, ngrp, mw, nw, true);
  return true;
}

// slabs per group of the two-level sum: up to 16 slabs are added by one block
inline void groups_for(int nz, int* grp, int* ngrp) {
  int g = nz;
  if (nz > 16) {
    g = 4;
    while (g * g < nz) ++g;
  }
  *grp = g;
  *ngrp = cdiv(nz, g);
}

}  // namespace gf
