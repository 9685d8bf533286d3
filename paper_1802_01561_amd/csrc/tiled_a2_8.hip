// Tiled V-trace kernel instantiations for A = 2, 3, 4, 5, 6, 7, 8 (fp32 or bf16
// logits); the kernel is in tiled_impl.hpp.
#include "tiled_impl.hpp"

namespace vtrace {

hipError_t launch_tiled_a2_8(const StepArgs& a, LogitsType lt, int lanes, Mode mode, hipStream_t st,
                             int64_t* num_workgroups, bool allow_multi) {
  switch (a.A) {
    case 2: return launch_any<2>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 3: return launch_any<3>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 4: return launch_any<4>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 5: return launch_any<5>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 6: return launch_any<6>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 7: return launch_any<7>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    case 8: return launch_any<8>(a, lt, lanes, mode, st, num_workgroups, allow_multi);
    default: return hipErrorNotSupported;
  }
}

}  // namespace vtrace
