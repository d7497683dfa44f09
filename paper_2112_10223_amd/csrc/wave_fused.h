// The symbolic pass of the wave bins in one launch (wave_fused.hip).  Not part of
// the public ABI.
#pragma once
#include "internal.h"

namespace spk {

// Per wave bin (index bin - BIN_W1): accumulator (ACC_*), bitmap rows of 256 words
// (ACC_BITMAP) and symbolic table slots (ACC_HASH); the kernel derives each bin's LDS
// layout from them.
struct WaveBinTable {
  int acc[NWAVE_BINS];
  int bm_nq[NWAVE_BINS];
  int ts[NWAVE_BINS];
};

// Wavefronts per SIMD of the fused launch: its registers are held to that.  Its longest
// columns would take 136 (145 with two inputs per lane) and leave three; held to 128 it
// spills 4 (15), in the bodies of the bins E = 16 alone.
constexpr int SYM_FUSED_WAVES = 4;

// Counts the distinct rows of every column of the wave bins.  The bins' column
// lists and offsets are read on the device (d_list, d_binoff as the binning kernels
// leave them), so the host needs no bin count to launch it.  a.slice_bytes is the
// largest slice of any wave bin; blocks is the grid (resident blocks of four
// wavefronts).
hipError_t launch_wave_sym_fused(const KArgs& a, const WaveBinTable& t, const int* d_list, const int* d_binoff,
                                 unsigned blocks, hipStream_t s);

}  // namespace spk
