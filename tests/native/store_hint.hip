// One store of a row of y, for a look at what it compiles to.
#include "spmv_impl.h"

extern "C" __global__ void store_row(double *y, const int32_t *perm, int64_t n, bool keep, const double *v) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < n) sell::dev::put_row(y, perm, p, keep, v[p]);
}
