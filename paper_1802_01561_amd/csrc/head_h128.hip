// Fused output layer + V-trace kernels for hidden size 128.
#include "head_impl.hpp"

namespace vtrace {

void launch_head_h128(const HeadArgs& a, hipStream_t st, unsigned nwg) { launch_head_h<128>(a, st, nwg); }

}  // namespace vtrace
