// One-launch contraction of small FP64 tensors (see contract.hip).
#pragma once
#include <hip/hip_runtime.h>

namespace tci {

constexpr int CONTRACT_MAX_BONDS = 8;
constexpr int CONTRACT_MAX_K = 64;                 // summed terms per element
constexpr long long CONTRACT_MAX_WORK = 1 << 17;   // multiply-adds

// c (row-major over its nc bonds) = sum over ns summed bonds of a b.  A bond of
// c advances a by sa and b by sb elements (one of the two is 0), a summed bond
// by ta and tb.
struct ContractArgs {
  int nc, ns, nout, k;
  int cdim[CONTRACT_MAX_BONDS], sa[CONTRACT_MAX_BONDS], sb[CONTRACT_MAX_BONDS];
  int sdim[CONTRACT_MAX_BONDS], ta[CONTRACT_MAX_BONDS], tb[CONTRACT_MAX_BONDS];
};

// dtype F64 or C128; 1 <= k <= CONTRACT_MAX_K, nout >= 1; c overlaps neither operand.
hipError_t contract_small(int dtype, const void* a, const void* b, void* c, const ContractArgs& g, hipStream_t s);

}  // namespace tci
