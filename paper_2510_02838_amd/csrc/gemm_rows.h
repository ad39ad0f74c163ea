// Row arithmetic of the matrix products, in plain C++ so that the host can check it.
#pragma once
#if defined(__HIPCC__)
#define DIT_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define DIT_HOST_DEVICE inline
#endif

namespace dit {

// The row of the output (and of the rotary table) that row m of a product of M rows belongs to: m itself without a map.
// The last tile's rows from M on are never stored, but their rotary pairs are read: they take those of row M - 1.
DIT_HOST_DEVICE int dest_row(const int* map, int m, int M) {
  const int c = m < M ? m : M - 1;
  return map ? map[c] : c;
}

}  // namespace dit
