// The plain (ungrouped) instantiations of the FP32 MFMA GEMM kernel.
#include "gemm_kernel.hpp"

namespace cpra {
namespace gemmk {

void launch_plain(bool a_t, bool b_t, int cfg, LaunchArgs& args, hipStream_t stream) {
  if (!a_t && b_t) launch_any<false, true, 0>(cfg, args, stream);
  else if (!a_t && !b_t) launch_any<false, false, 0>(cfg, args, stream);
  else if (a_t && !b_t) launch_any<true, false, 0>(cfg, args, stream);
  else launch_any<true, true, 0>(cfg, args, stream);
}

}  // namespace gemmk
}  // namespace cpra
