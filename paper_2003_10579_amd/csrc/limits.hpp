// Limits of addresses that the kernels share, as plain host arithmetic (no HIP), so that a test can compile it by itself.
#pragma once
#include <stdint.h>

namespace ssgd {

// The steady-state kernels of the linear models gather rows through one buffer descriptor that spans the sample matrix:
// the row's place is the scalar offset, a lane's column the vector offset.  Such a load is out of range, and gives zeros,
// from vector offset >= size - scalar offset on, so a lane that must read zeros whatever the row needs a vector offset at
// or past the size itself.  (2^31 is not that for a matrix of more than 2 GiB: the lane would read the data 2 GiB further
// on.)  The last of the four words of the load does not wrap either.
constexpr uint32_t kPastMatrix = 0xFFFFFFF0u;
inline bool one_descriptor_spans(uint64_t N, uint64_t d) { return N * d * 4u <= kPastMatrix; }

}  // namespace ssgd
