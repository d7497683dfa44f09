// Host side of the wave-bin kernels of the plain (one SpKAdd) launch.
#include "wave_kernels.h"

namespace spk {

bool wave_pipe_ok(int k, int alpha_num_q, int acc) {
  return alpha_num_q == 512 && k <= (acc == ACC_HASH ? 64 : 128);
}

void lds_layout_pipe(int bin, bool numeric, int vbytes, int ts_max, int acc, int rows, int k, KArgs& a) {
  pipe_layout(wave_bin_E(bin), numeric, vbytes, ts_max, acc, rows, k > 64 ? 2 : 1, a);
}

hipError_t launch_wave_pipe(int bin, bool numeric, bool f64, int acc, const KArgs& a, const int* d_list, int nunits,
                            int n_cu, hipStream_t s) {
  if (nunits <= 0) return hipSuccess;
  if (!numeric) return launch_pipe_sym(bin, acc, a, d_list, nunits, n_cu, s);
  if (acc & ACC_ORDERED)
    return f64 ? launch_pipe_ord_f64(bin, acc & 3, a, d_list, nunits, n_cu, s)
               : launch_pipe_ord_f32(bin, acc & 3, a, d_list, nunits, n_cu, s);
  return f64 ? launch_pipe_f64(bin, acc, a, d_list, nunits, n_cu, s)
             : launch_pipe_f32(bin, acc, a, d_list, nunits, n_cu, s);
}

}  // namespace spk
