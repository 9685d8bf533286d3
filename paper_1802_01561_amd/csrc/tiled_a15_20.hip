// Tiled V-trace kernel instantiations for A = 15, 16, 17, 19, 20 (fp32 or bf16
// logits); the kernel is in tiled_impl.hpp.
#include "tiled_impl.hpp"

namespace vtrace {

hipError_t launch_tiled_a15_20(const StepArgs& a, LogitsType lt, int lanes, Mode mode, hipStream_t st,
                               int64_t* num_workgroups, bool allow_multi) {
  switch (a.A) {
    case 15: return launch_any<15>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 16: return launch_any<16>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 17: return launch_any<17>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 19: return launch_any<19>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 20: return launch_any<20>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    default: return hipErrorNotSupported;
  }
}

}  // namespace vtrace
