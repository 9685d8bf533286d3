// Fused output layer + V-trace kernels for hidden size 64.
#include "head_impl.hpp"

namespace vtrace {

void launch_head_h64(const HeadArgs& a, hipStream_t st, unsigned nwg) { launch_head_h<64>(a, st, nwg); }

}  // namespace vtrace
