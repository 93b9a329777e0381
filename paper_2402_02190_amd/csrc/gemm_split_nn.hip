// The NN instantiations of the split GEMM: plain and by graph rows.
#include "gemm_split.hpp"

namespace cpra {
namespace gemmk {

void launch_split_nn(int mode, int cfg, LaunchArgs& args, hipStream_t stream) {
  if (mode == 1) launch_split_any<false, false, 1>(cfg, args, stream);
  else launch_split_any<false, false, 0>(cfg, args, stream);
}

}  // namespace gemmk
}  // namespace cpra
