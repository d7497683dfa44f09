// Wave-bin kernels: numeric pass, double values.
#include "wave_kernels.h"

namespace spk {

hipError_t launch_pipe_f64(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s) {
  return launch_pipe_t<true, double>(bin, acc, a, list, n, n_cu, s);
}

}  // namespace spk
