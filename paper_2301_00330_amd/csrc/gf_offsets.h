// Offsets of operand loads, as plain integer arithmetic: usable in host code, where their bounds are tested.
#pragma once

#ifdef __HIPCC__
#define GF_HD __host__ __device__ __forceinline__
#else
#define GF_HD inline
#endif

namespace gf {

// Element offsets of one lane's vector in the K chunks of an operand with k as the slow index (rows of `stride`
// elements; the vector stands at column offset `base` in row `row` of every chunk of `kb` rows).  Rows past the last
// one are read at the last one, whose values the caller clears: in a tensor of few rows the offset of a row that
// does not exist can pass 2^31 (8 channels, 6000 x 6000 pixels, chunks of 64: row 63 would start at 2.3e9).  Only the
// last chunk has such rows, so it gets an offset of its own and every other chunk costs one addition.
struct RowOffsets {
  int inner, last;   // of the vector in a chunk whose rows all exist, in the last chunk; both without the chunk's own rows

  GF_HD void set(int base, int row, int rows, int kb, int stride) {
    const int tail = rows - (rows - 1) / kb * kb;   // rows of the last chunk
    inner = base + (row < rows ? row : rows - 1) * stride;
    last = base + (row < tail ? row : tail - 1) * stride;
  }
  // in the chunk that starts at row k0 (of any lane of the block: k0 is uniform)
  GF_HD int at(int k0, int rows, int kb, int stride) const { return (k0 + kb > rows ? last : inner) + k0 * stride; }
};

}  // namespace gf
