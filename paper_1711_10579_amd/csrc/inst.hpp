// Access to instance descriptors and Newton states in the kernels.
#pragma once

#include "blk.hpp"
#include "device.hpp"

namespace pfd {

// Descriptor of instance `slot` of a batch.  A batch of one passes the
// descriptor's own address, marked by its low bit: the kernels of a single
// solve last a few dependent memory round trips, and this takes the table
// (and, where the slot comes from a work item, the item) out of that chain.
__device__ inline const PF_AS1 Inst& inst_at(const Inst* const* insts, int slot) {
  const uintptr_t p = (uintptr_t)insts;
  if (p & 1) return *(const PF_AS1 Inst*)(p - 1);
  return *gp(gp(insts)[slot]);
}

// its Newton state, at a fixed place beside the descriptor
__device__ inline PF_AS1 Red* red_of(const PF_AS1 Inst& I) {
  return (PF_AS1 Red*)((const PF_AS1 char*)&I - kRedOffset);
}

}  // namespace pfd
