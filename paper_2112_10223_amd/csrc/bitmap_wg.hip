// Workgroup bitmap accumulator for row windows (Section III-B, Algorithms 7-8) and
// workgroup columns, on a bitmap of the unit's rows, ranked where they are spread
// wide (bitmap_wg_device.h).  Symbolic (Algorithm 6): an OR that finds its bit clear
// counts a new row.  Numeric (Algorithm 5): OR with return marks each row's first
// entry, a block-wide popcount prefix over pairs of words gives rank(row) = the row's
// position in the sorted output, the first entry stores (row, value) at its rank in
// an LDS staging area and later entries add by compare-and-swap; the unit is then
// written out coalesced.  No hash table and no sort: the bitmap is the "partitioned
// SPA" the paper proposes for row-partitioned accumulation, with a rank in place of a
// dense value array.
//
// Bound by latency (three dependent loads and the barriers of a unit), which the units
// resident on a CU hide: four workgroups of 512 threads, two of 1024.
#include "bitmap_wg_device.h"

namespace spk {

template <int NT, int EW, bool NUM, bool WIN, typename V>
__global__ __launch_bounds__(NT, 8) void k_bitmap_wg(KArgs a, const int* __restrict__ list, int nunits) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int red[bitmap_wg_reds(NT)];
  const int unit = xcd_remap(blockIdx.x, gridDim.x);
  if (unit >= nunits) return;  // uniform over the block
  int j, blo = 0, rlo = 0, rhi = a.m;
  if (WIN) {
    const int4 w = a.wrec[unit];
    j = w.x;
    rlo = w.y;
    rhi = w.z;
    blo = w.w;
  } else {
    j = list[unit];
  }
  bitmap_wg_unit<NT, EW, NUM, WIN, V>(a, smem, red, unit, j, blo, rlo, rhi);
}

// ---- host side ----

// LDS of a unit of at most cap entries (in registers; regs of them at most) or, for a
// window with more, cap rows; span: rows of the widest unit.  The low bitmap (a word per
// entry, or one bit per row for up to that many bits) and its prefix, then the top bitmap
// (a bit per 32 rows, at most 20 per entry: 1.3 million rows at cap = 2048) and its
// prefix; the symbolic pass needs the low prefix only when there are more levels.  The
// staging area overlays all of them (every rank is read before the first store), but not
// the bitmap of cap rows and its prefix at the start, which the windows with more entries
// than registers read while they add.
void lds_layout_bitmap_wg(bool numeric, int vbytes, int k, int cap, int regs, int span, KArgs& a) {
  auto align16 = [](int x) { return (x + 15) & ~15; };
  const int low = (32 * cap + 1023) & ~1023;
  int topb = (20 * cap + 1023) & ~1023;
  const long long blocks = ((long long)span + 31) / 32;
  const bool more = blocks > topb;  // than two levels
  if (!more) topb = span > low ? (int)((blocks + 1023) & ~1023LL) : 0;
  a.wg_low_bits = low;
  a.wg_top_bits = topb;
  a.off_bm = 0;
  a.off_pre = align16(low / 8);
  a.off_top = a.off_pre + (numeric || more ? align16(low / 32) : 0);
  int off = a.off_top + align16(topb / 8) + align16(topb / 32);
  a.off_dpre = (cap + 255) / 256 * 32;
  a.off_bvals = a.off_dpre + align16((cap + 255) / 256 * 8);
  a.off_brows = a.off_bvals + align16(cap * vbytes);
  const int staged = a.off_brows + align16(cap * 4);
  if (numeric && staged > off) off = staged;
  a.off_P = off;
  off = align16(off + (k + 1) * 4);
  a.off_adj = a.off_adjv = off;
  off = align16(off + k * (numeric ? 16 : 8));
  a.off_mark = off;  // segment-start mask and its prefix
  const int words = (regs / 64 + 63) / 64 * 64;
  off += words * (8 + 4);
  a.slice_bytes = align16(off);
  a.wg_cap = cap;
}

// Threads of the kernel that takes units of up to cap entries.
int bitmap_wg_threads(int bin, int cap) {
  if (bin == BIN_G1) return G1_THREADS;
  return bin == BIN_G3 || cap > G2_THREADS * BITMAP_WG_EW ? G3_THREADS : G2_THREADS;
}

template <bool NUM, typename V>
static hipError_t launch_bw(int bin, const KArgs& a, const int* list, int n, hipStream_t s) {
  const size_t lds = (size_t)a.slice_bytes;
  constexpr int EW = BITMAP_WG_EW;
  const int nt = bitmap_wg_threads(bin, a.wg_cap);
  if (nt == G1_THREADS)
    k_bitmap_wg<G1_THREADS, EW, NUM, false, V><<<n, nt, lds, s>>>(a, list, n);
  else if (bin == BIN_WIN && nt == G2_THREADS)
    k_bitmap_wg<G2_THREADS, EW, NUM, true, V><<<n, nt, lds, s>>>(a, list, n);
  else if (bin == BIN_WIN)
    k_bitmap_wg<G3_THREADS, EW, NUM, true, V><<<n, nt, lds, s>>>(a, list, n);
  else if (nt == G2_THREADS)
    k_bitmap_wg<G2_THREADS, EW, NUM, false, V><<<n, nt, lds, s>>>(a, list, n);
  else
    k_bitmap_wg<G3_THREADS, EW, NUM, false, V><<<n, nt, lds, s>>>(a, list, n);
  return hipGetLastError();
}

hipError_t launch_bitmap_wg(int bin, bool numeric, bool f64, const KArgs& a, const int* d_list, int nunits,
                            hipStream_t s) {
  if (nunits <= 0) return hipSuccess;
  if (bin != BIN_G1 && bin != BIN_G2 && bin != BIN_G3 && bin != BIN_WIN) return hipErrorInvalidValue;
  if (!numeric) return launch_bw<false, float>(bin, a, d_list, nunits, s);
  return f64 ? launch_bw<true, double>(bin, a, d_list, nunits, s) : launch_bw<true, float>(bin, a, d_list, nunits, s);
}

}  // namespace spk
