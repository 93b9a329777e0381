// The TN (weight gradient) and TT instantiations of the split GEMM: plain and by
// graph K ranges; and the dispatch over the layouts.
#include "gemm_split.hpp"

namespace cpra {
namespace gemmk {

void launch_split(int mode, bool a_t, bool b_t, int cfg, LaunchArgs& args, hipStream_t stream) {
  if (!a_t) {
    if (b_t) launch_split_nt(mode, cfg, args, stream);
    else launch_split_nn(mode, cfg, args, stream);
  } else if (mode == 2) {
    launch_split_any<true, false, 2>(cfg, args, stream);
  } else if (b_t) {
    launch_split_any<true, true, 0>(cfg, args, stream);
  } else {
    launch_split_any<true, false, 0>(cfg, args, stream);
  }
}

}  // namespace gemmk
}  // namespace cpra
