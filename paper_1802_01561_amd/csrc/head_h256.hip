// Fused output layer + V-trace kernels for hidden size 256.
#include "head_impl.hpp"

namespace vtrace {

void launch_head_h256(const HeadArgs& a, hipStream_t st, unsigned nwg) { launch_head_h<256>(a, st, nwg); }

}  // namespace vtrace
