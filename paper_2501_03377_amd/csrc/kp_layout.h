// Index arithmetic of the packed operators, shared by the host packing and the
// kernels (plain C++).
#pragma once

#include <stdint.h>

namespace kp {

// The folded FP64 and FP32 operators (kp_fold.hip) are blocks of 16 k x 16
// columns, ordered by group, column fragment and k-block: the block's number,
// and the 16-byte units before it (units: of a block).  An operator of 2^31
// units (FP64: more than 65536 points) has 34 GB, one of 2^32 blocks 9 TB, so
// the number takes 32 bits and only the offset 64.
constexpr uint32_t fold_block(uint32_t q, uint32_t jf, uint32_t kb, uint32_t nf, uint32_t nkb) {
  return (q * nf + jf) * nkb + kb;
}
constexpr uint64_t fold_units(uint32_t block, uint32_t units) { return (uint64_t)block * units; }

}  // namespace kp
