// The chain rule of every gradient call: the gradient with respect to the
// index-space entries (fixed voxel index -> continuous moving index, formed by
// the call's preparation from the caller's physical mm matrices), which the
// backward sweep accumulates, becomes the gradient with respect to the
// caller's physical entries.
#include "common.h"

namespace gemi {

// With y_r = (sum_c P[r][c] x_c + P[r][3] - morg[r]) / msp[r] and the fixed
// voxel's position x_c = forg[c] + fsp[c] i_c, the moving index depends on
// P[r][c] through M[r][c] = P[r][c] fsp[c] / msp[r] and
// M[r][3] = (... + P[r][c] forg[c] ...) / msp[r]:
//   dMI/dP[r][c] = (dMI/dM[r][c] fsp[c] + dMI/dM[r][3] forg[c]) / msp[r],
//   dMI/dP[r][3] = dMI/dM[r][3] / msp[r].
__global__ void grad_physical_kernel(double* __restrict__ G, int64_t rows, Geometry g) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < rows;
       k += (int64_t)gridDim.x * blockDim.x) {
    double* row = G + 12 * k;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const double gt = row[4 * r + 3];
#pragma unroll
      for (int c = 0; c < 3; ++c) row[4 * r + c] = (row[4 * r + c] * g.fsp[c] + gt * g.forg[c]) / g.msp[r];
      row[4 * r + 3] = gt / g.msp[r];
    }
  }
}

__global__ __launch_bounds__(256) void sample_layout_kernel(const double* __restrict__ P, int64_t n, Geometry g,
                                                            double row_weight, double limit,
                                                            uint32_t* __restrict__ records) {
  __shared__ double sum[256];
  const int64_t used = n < 256 ? n : 256;
  double rise = 0.0;
  if ((int64_t)threadIdx.x < used) {
    double m[12];
    compose_index_matrix(P + 12 * ((int64_t)threadIdx.x * n / used), g, m);
    rise = row_weight * fabs(m[4]) + fabs(m[8]);
    if (!(rise < 65536.0)) rise = 0.0;  // a rejected matrix
  }
  sum[threadIdx.x] = rise;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) sum[threadIdx.x] += sum[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) *records = sum[0] > limit * (double)used ? 1u : 0u;
}

hipError_t launch_sample_layout(const double* P, int64_t n, const Geometry& g, double row_weight, double limit,
                                uint32_t* records, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sample_layout_kernel, dim3(1), dim3(256), 0, s, P, n, g, row_weight, limit, records);
  return hipGetLastError();
}

static unsigned grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

hipError_t launch_grad_physical(double* grad, int64_t rows, const Geometry& g, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(grad_physical_kernel, dim3(grid_for(rows)), dim3(256), 0, s, grad, rows, g);
  return hipGetLastError();
}

}  // namespace gemi
