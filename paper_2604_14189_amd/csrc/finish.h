// Work split of the kernels that finish a gradient (all physics): padded cells
// summed into the model cells that they repeat.
#pragma once

#include "internal.h"

namespace sweep {

// Model cells of the finishing kernels, which sum the padded cells that repeat a
// model cell: one for an inner cell, up to (P + 1)^2 for one on the model's
// border. Blocks [0, finish_inner_blocks) take a thread per model cell and leave
// the border to the waves of the others, one per border cell, whose lanes share
// the padded cells (float64 sums, added by a fixed tree).
inline __host__ __device__ int finish_inner_blocks(int nx, int nz) {
  return (int)(((size_t)nx * nz + 255) / 256);
}
inline __host__ __device__ int finish_border_cells(int nx, int nz) {
  return (nz > 1 ? 2 : 1) * nx + (nz > 2 ? nz - 2 : 0) * (nx > 1 ? 2 : 1);
}
inline dim3 finish_grid(int nx, int nz) {
  return dim3(finish_inner_blocks(nx, nz) + (finish_border_cells(nx, nz) + 3) / 4);
}
// Model cell of this thread (256 per block) and its share (lane of nl) of the
// padded cells; false where there is none.
__device__ __forceinline__ bool finish_cell(int nx, int nz, int& ii, int& jj, int& lane, int& nl) {
  const int nb = finish_inner_blocks(nx, nz);
  if ((int)blockIdx.x < nb) {
    const size_t m = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (m >= (size_t)nx * nz) return false;
    jj = (int)(m / nx);
    ii = (int)(m - (size_t)jj * nx);
    lane = 0;
    nl = 1;
    return ii > 0 && ii < nx - 1 && jj > 0 && jj < nz - 1;
  }
  int w = ((int)blockIdx.x - nb) * 4 + (int)(threadIdx.x >> 6);
  if (w >= finish_border_cells(nx, nz)) return false;
  lane = threadIdx.x & 63;
  nl = 64;
  if (w < nx) {
    ii = w;
    jj = 0;
  } else if ((w -= nx) < nx && nz > 1) {
    ii = w;
    jj = nz - 1;
  } else {
    w -= nx;
    jj = 1 + (nx > 1 ? w >> 1 : w);
    ii = nx > 1 && (w & 1) ? nx - 1 : 0;
  }
  return true;
}
// Sum over the nl lanes that share a model cell (all of them active).
__device__ __forceinline__ double finish_sum(double v, int nl) {
  for (int d = nl >> 1; d > 0; d >>= 1) v += __shfl_xor(v, d);
  return v;
}

}  // namespace sweep
