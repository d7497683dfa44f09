// Wave-bin kernels: numeric pass, float values summed in input order (SPKADD_FLAG_ORDERED).
#include "wave_kernels.h"

namespace spk {

hipError_t launch_pipe_ord_f32(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s) {
  return launch_pipe_t<true, float, ACC_ORDERED>(bin, acc, a, list, n, n_cu, s);
}

}  // namespace spk
