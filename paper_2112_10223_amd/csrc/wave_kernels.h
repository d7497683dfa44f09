// Wave-bin kernels of the plain (one SpKAdd) launch and their launcher, instantiated per
// pass and value type (wave_sym.hip, wave_num_f32.hip, wave_num_f64.hip and, with values
// summed in input order, wave_ord_f32.hip, wave_ord_f64.hip: one translation unit each,
// so that they compile side by side).  The device code is in
// wave_device.h.
#pragma once
#include "wave_device.h"

namespace spk {

template <int E, bool NUM, typename V, int ACC, int KC>
__global__ __launch_bounds__(64 * PIPE_WAVES_PER_BLOCK) void k_wave_pipe(KArgs a, const int* __restrict__ list,
                                                                        int nunits) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = lane_id(), w = threadIdx.x >> 6;
  // Units are dealt out with stride G (all wavefronts of the launch): at any time
  // the wavefronts of one XCD (consecutive gw after the remap) work on neighbouring
  // columns, whose input rows share cache lines, instead of each wavefront walking a
  // column range of its own (too many partly used lines for the L2).
  const int G = (int)gridDim.x * PIPE_WAVES_PER_BLOCK;
  const int gw = xcd_remap(blockIdx.x, gridDim.x) * PIPE_WAVES_PER_BLOCK + w;
  if (gw >= nunits) return;  // no block-wide barriers in this kernel
  const int nu = (nunits - gw + G - 1) / G;  // <= upw <= 64
  const int ucol = lane < nu ? list[gw + lane * G] : 0;
  run_pipe<E, NUM, V, ACC, KC>(a, smem + w * a.slice_bytes, nu, ucol);
}

// Workgroups of a kernel that a CU's registers hold (512 per lane and SIMD, in steps of
// 8; a workgroup puts one wavefront on each SIMD).
template <typename F>
int register_blocks(F kernel) {
  hipFuncAttributes fa{};
  if (hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kernel)) != hipSuccess || fa.numRegs <= 0) {
    (void)hipGetLastError();
    return 4;
  }
  const int w = 512 / ((fa.numRegs + 7) & ~7);
  return w < 1 ? 1 : w > 8 ? 8 : w;
}

// The launch fills the CUs with resident wavefronts and each takes an equal share of the
// units, at most 64.  With more than four workgroups on a CU a wavefront of a short launch
// would get one or two units, and nothing of the next one in flight while it works: as
// many as LDS and registers hold only where each then still has three units (two at
// E = 1).  Numeric fp32, 4,000 rows, at most four / all: u = 128, 6,000 columns 11.7 /
// 14.9 us, 16,000 16.8 / 20.1, 64,000 37.2 / 36.4; u = 192, 6,000 columns 14.4 / 18.4,
// 65,536 rows, 130,000 columns 128.8 / 127.4; u = 32, 8,000 columns 8.4 / 9.4, 16,000
// 10.6 / 10.6, 130,000 40.3 / 36.1.
template <int E, bool NUM, typename V, int ACC, int KC>
hipError_t launch_pipe_k(const KArgs& a_in, const int* list, int n, int n_cu, hipStream_t s) {
  static_assert(PIPE_WAVES_PER_BLOCK == 4, "register_blocks counts one wavefront per SIMD");
  static const int by_regs = register_blocks(k_wave_pipe<E, NUM, V, ACC, KC>);
  KArgs a = a_in;
  const size_t lds = (size_t)a.slice_bytes * PIPE_WAVES_PER_BLOCK;
  int bpc = (int)((size_t)max_lds_bytes() / lds);
  if (bpc > by_regs) bpc = by_regs;
  if (bpc < 1) bpc = 1;
  const long long per_block = (long long)n_cu * PIPE_WAVES_PER_BLOCK;
  if (bpc > 4 && n <= per_block * bpc * (E == 1 ? 1 : 2)) bpc = 4;
  const long long resident = per_block * bpc;
  const long long upw = (n + resident - 1) / resident;
  a.upw = (int)(upw < 1 ? 1 : upw > 64 ? 64 : upw);
  const int waves = (n + a.upw - 1) / a.upw;
  const unsigned blocks = (unsigned)((waves + PIPE_WAVES_PER_BLOCK - 1) / PIPE_WAVES_PER_BLOCK);
  k_wave_pipe<E, NUM, V, ACC, KC><<<blocks, 64 * PIPE_WAVES_PER_BLOCK, lds, s>>>(a, list, n);
  return hipGetLastError();
}

// ORD: ACC_ORDERED or 0 (hash tables: only 0).
template <int E, bool NUM, typename V, int ORD>
hipError_t launch_pipe_e(int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s) {
  if (a.k > 64) {
    if (acc == ACC_BITMAP) return launch_pipe_k<E, NUM, V, ACC_BITMAP | ORD, 2>(a, list, n, n_cu, s);
    if (acc == ACC_RANKED) return launch_pipe_k<E, NUM, V, ACC_RANKED | ORD, 2>(a, list, n, n_cu, s);
    return hipErrorInvalidValue;
  }
  if (acc == ACC_BITMAP) return launch_pipe_k<E, NUM, V, ACC_BITMAP | ORD, 1>(a, list, n, n_cu, s);
  if (acc == ACC_RANKED) return launch_pipe_k<E, NUM, V, ACC_RANKED | ORD, 1>(a, list, n, n_cu, s);
  if constexpr (ORD == 0) return launch_pipe_k<E, NUM, V, ACC_HASH, 1>(a, list, n, n_cu, s);
  return hipErrorInvalidValue;
}

template <bool NUM, typename V, int ORD = 0>
hipError_t launch_pipe_t(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s) {
  switch (bin) {
    case BIN_W1: return launch_pipe_e<1, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W2: return launch_pipe_e<2, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W3: return launch_pipe_e<3, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W4: return launch_pipe_e<4, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W5: return launch_pipe_e<5, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W6: return launch_pipe_e<6, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W8: return launch_pipe_e<8, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W10: return launch_pipe_e<10, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W12: return launch_pipe_e<12, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    case BIN_W16: return launch_pipe_e<16, NUM, V, ORD>(acc, a, list, n, n_cu, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_pipe_sym(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s);
hipError_t launch_pipe_f32(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s);
hipError_t launch_pipe_f64(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s);
hipError_t launch_pipe_ord_f32(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s);
hipError_t launch_pipe_ord_f64(int bin, int acc, const KArgs& a, const int* list, int n, int n_cu, hipStream_t s);

}  // namespace spk
