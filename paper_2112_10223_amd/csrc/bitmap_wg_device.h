// Device body of the workgroup bitmap accumulator (bitmap_wg.hip: plain units;
// batch_fused.hip: the workgroup-sized columns of batched runs).
#pragma once
#include "wave_device.h"

namespace spk {

// Exclusive scan over the NT threads of a block, in one barrier: `scratch` holds NT / 64
// values and may be written again only after another barrier.
template <int NT>
__device__ __forceinline__ int block_scan1(int x, int* scratch, int& total) {
  constexpr int NW = NT / 64;
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int incl = wave_scan_add(x);
  if (lane == 63) scratch[w] = incl;
  __syncthreads();
  const int sums = wave_scan_add(lane < NW ? scratch[lane] : 0);  // every wavefront scans the NW totals
  total = readlane(sums, 63);
  return readlane(sums, w) - readlane(incl, 63) + incl - x;
}

// Exclusive popcount prefix per pair of words of a bitmap of ngrp pairs (of which the
// words up to a multiple of 8 are clear) into pw.  A thread takes four consecutive pairs
// of a tile of 4 NT: two 16-byte reads, one 8-byte write (pair by pair, lanes 32 bytes
// apart conflict in the LDS banks eight to one).  The bitmap is complete (a barrier) on
// entry and pw on return.  Returns the set bits.
template <int NT>
__device__ __forceinline__ int block_bitmap_prefix(const unsigned* bm, unsigned short* pw, int ngrp, int* scratch) {
  const uint4* bm4 = reinterpret_cast<const uint4*>(bm);
  int carry = 0;
  for (int base = 0; base < ngrp; base += 4 * NT) {  // (uniform)
    if (base > 0) __syncthreads();  // (the scratch of the tile before)
    const int g = base + 4 * (int)threadIdx.x;
    uint4 x = make_uint4(0u, 0u, 0u, 0u), y = x;
    if (g < ngrp) {
      x = bm4[g >> 1];
      y = bm4[(g >> 1) + 1];
    }
    const int c0 = __popc(x.x) + __popc(x.y), c1 = c0 + __popc(x.z) + __popc(x.w);
    const int c2 = c1 + __popc(y.x) + __popc(y.y), c3 = c2 + __popc(y.z) + __popc(y.w);
    int total = 0;
    const int run = carry + block_scan1<NT>(c3, scratch, total);
    if (g < ngrp)
      reinterpret_cast<uint2*>(pw)[g >> 2] = make_uint2((unsigned)run | ((unsigned)(run + c0) << 16),
                                                        (unsigned)(run + c1) | ((unsigned)(run + c2) << 16));
    carry += total;
  }
  __syncthreads();
  return carry;
}

// Keeps the compiler from starting the entries of a thread (loops over t) more than four
// at a time: their addresses and table words would only take registers, and with them
// resident workgroups.
__device__ __forceinline__ void in_fours(int t) {
  if (t > 0 && t % 4 == 0) __builtin_amdgcn_sched_barrier(0);
}

// Set bits below bit r.
__device__ __forceinline__ int bitmap_rank(const unsigned* bm, const unsigned short* pw, int r) {
  const uint2 pr = reinterpret_cast<const uint2*>(bm)[r >> 6];
  const unsigned odd = 0u - (unsigned)((r >> 5) & 1);
  const unsigned word = pr.x ^ ((pr.x ^ pr.y) & odd);
  return (int)pw[r >> 6] + (int)((unsigned)__popc(pr.x) & odd) + __popc(word & ((1u << (r & 31)) - 1u));
}

// Segments of a unit for its first wavefront: the exclusive prefix P of the segment
// lengths and the addresses of input i's entries in pr[i] (shifted so that the entry's
// number in the unit addresses them); for a unit of at most REGS entries the non-empty
// segments only, in order, with their starts as bits of a mask over the entries (mask
// words, then the starts before each word).  Returns u.
template <int REGS, bool NUM, typename V>
__device__ __forceinline__ int build_segments(const KArgs& a, int j, bool win, int blo, int* P, long long* adj,
                                              unsigned long long* smask) {
  constexpr int WPL = (REGS / 64 + 63) / 64;  // mask words per lane
  const int lane = lane_id();
  int carry = 0, nz = 0;
#pragma unroll
  for (int c = 0; c < WPL; ++c) smask[WPL * lane + c] = 0ull;
  wave_sync();
  for (int base = 0; base < a.k; base += 64) {
    const int i = base + lane;
    int s = 0, e = 0;
    const int* rp = nullptr;
    const V* vp = nullptr;
    if (i < a.k) {
      // the row / value pointers are fetched together with the segment bounds
      rp = a.ri[i];
      if (NUM) vp = (const V*)a.va[i];
      if (win) {
        s = a.bpos[(long long)blo * a.k + i];
        e = max(a.bpos[(long long)(blo + 1) * a.k + i], s);  // (only an unsorted input could invert them)
      } else if (a.cpt) {
        const int* c = a.cpt + (long long)j * cpt_stride(a.k) + i;
        s = c[0];
        e = c[cpt_stride(a.k)];
      } else {
        const int* c = a.cp[i];
        s = c[j];
        e = c[j + 1];
      }
    }
    const int len = e - s;
    const int incl = wave_scan_add(len);
    const int ex = carry + incl - len;
    const uint64_t some = ballot(len > 0);
    if (len > 0) {
      const int o = nz + mbcnt(some);
      const long long ar = (long long)(rp + s) - 4LL * ex;
      if constexpr (NUM)
        reinterpret_cast<longlong2*>(adj)[o] = make_longlong2(ar, (long long)(vp + s) - (long long)sizeof(V) * ex);
      else
        adj[o] = ar;
      P[o] = ex;
      if (ex < REGS) atomicOr(&smask[ex >> 6], 1ull << (ex & 63));
    }
    nz += __popcll(some);
    carry += readlane(incl, 63);
  }
  wave_sync();
  int* mpre = reinterpret_cast<int*>(smask + 64 * WPL);
  int cw = 0, c0 = 0;
#pragma unroll
  for (int c = 0; c < WPL; ++c) {
    const int x = __popcll(smask[WPL * lane + c]);
    if (c == 0) c0 = x;
    cw += x;
  }
  const int before = wave_scan_add(cw) - cw;
  mpre[WPL * lane] = before;
  if constexpr (WPL == 2) mpre[WPL * lane + 1] = before + c0;
  if (lane == 0) P[a.k] = nz;  // (the number of non-empty segments)
  return carry;
}

// One unit (a column, or a row window when WIN) of the unit's row range [rlo, rhi):
// the whole workgroup of NT threads.  `red` holds 2 NT / 64 + 1 ints of workgroup-shared
// scratch; `smem` the layout of lds_layout_bitmap_wg.
//
// A unit's entries sit in registers, EW per thread (a window with more of them holds at
// most wg_cap rows: refinement only stops splitting a window above wg_cap entries once
// it is that narrow; its entries are read twice).  A range of at most wg_low_bits rows
// takes one bit per row.  A wider one is ranked first: a top bitmap marks the non-empty
// blocks of 32^L rows, and a block's rank replaces its number, which leaves at most
// wg_cap blocks of 32^(L-1) rows each divided again, down to one word per 32-row block.
// So the bitmap that gives the ranks has at most one word per entry, however wide the
// range: the LDS, its clearing and its prefix are bound by the unit's entries.
template <int NT, int EW, bool NUM, bool WIN, typename V>
__device__ __forceinline__ void bitmap_wg_unit(const KArgs& a, unsigned char* smem, int* red, int unit, int j, int blo,
                                               int rlo, int rhi) {
  constexpr int REGS = NT * EW;
  constexpr int WPL = (REGS / 64 + 63) / 64;
  const int tid = threadIdx.x;
  const int span = rhi - rlo;
  unsigned* bm = reinterpret_cast<unsigned*>(smem);
  unsigned short* pw = reinterpret_cast<unsigned short*>(smem + a.off_pre);  // set bits below each word pair
  unsigned* top = reinterpret_cast<unsigned*>(smem + a.off_top);
  int* P = reinterpret_cast<int*>(smem + a.off_P);
  long long* adj = reinterpret_cast<long long*>(smem + a.off_adj);
  unsigned long long* smask = reinterpret_cast<unsigned long long*>(smem + a.off_mark);
  const int* mpre = reinterpret_cast<const int*>(smask + 64 * WPL);
  int* red0 = red;
  int* red1 = red + NT / 64;
  int& info = red[2 * (NT / 64)];
  // the unit's output place (numeric), read now so that it arrives with the segment table
  int cnt = 0, o0 = 0;
  if (NUM) {
    if (WIN) {
      cnt = a.win_cnt[unit];
      o0 = a.colptr_c[j] + a.win_off[unit];
    } else {
      o0 = a.colptr_c[j];
      cnt = a.colptr_c[j + 1] - o0;
    }
  }
  if (tid < 64) {
    const int u0 = build_segments<REGS, NUM, V>(a, j, WIN, blo, P, adj, smask);
    if (tid == 0) info = u0;
  }
  // levels (uniform): the top one covers the range in blocks of 2^sh rows
  int sh = 0;
  if (span > a.wg_low_bits) {
    sh = 5;
    while ((span - 1) >> sh >= a.wg_top_bits) sh += 5;
  }
  {
    uint4* bm4 = reinterpret_cast<uint4*>(bm);
    const int low4 = 2 * ((min(span, a.wg_low_bits) + 255) >> 8);
    for (int w = tid; w < low4; w += NT) bm4[w] = make_uint4(0u, 0u, 0u, 0u);
    if (sh > 0) {
      uint4* top4 = reinterpret_cast<uint4*>(top);
      const int n4 = 2 * ((((span - 1) >> sh) + 256) >> 8);
      for (int w = tid; w < n4; w += NT) top4[w] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  __syncthreads();
  const int u = info;
  if (u <= REGS) {
    if (u <= 0) {  // (uniform) an empty window
      if (!NUM && tid == 0) {
        if (WIN) a.win_cnt[unit] = 0;
        else a.colcnt[j] = 0;
      }
      if (NUM && cnt != 0 && tid == 0) atomicOr(a.err, ERR_COUNT);
      return;
    }
    // A wavefront skips the groups of 64 entries past the unit's end (live: its groups);
    // in the group that holds the end, the places past it take the unit's last entry: no
    // load is masked off.
    const int wf = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int live = (u - wf + NT - 1) / NT;  // (at most EW; none when not positive)
    int rows[EW], vr[EW];
    V vals[EW];
    // (the 64 lanes' entries of one t share a mask word: lane t of the wavefront holds it)
    const int mw = min((tid >> 6) + (NT / 64) * min(lane_id(), EW - 1), 64 * WPL - 1);
    const unsigned long long sw = smask[mw];
    const int swl = (int)(unsigned)sw, swh = (int)(unsigned)(sw >> 32), spre = mpre[mw];
#pragma unroll
    for (int t = 0; t < EW; ++t) {
      in_fours(t);
      rows[t] = rlo;
      if constexpr (NUM) vals[t] = V(0);
      if (t >= live) continue;
      const int e = min(tid + NT * t, u - 1);
      // the segments that start at or before the entry, minus one (a place past the end
      // counts them all)
      const unsigned long long S =
          ((unsigned long long)(unsigned)readlane(swh, t) << 32) | (unsigned long long)(unsigned)readlane(swl, t);
      const int sg = readlane(spre, t) + (int)(S & 1ull) + mbcnt(S >> 1) - 1;
      if constexpr (NUM) {
        const longlong2 pr = reinterpret_cast<const longlong2*>(adj)[sg];
        rows[t] = gload<int>(pr.x + 4LL * e);
        vals[t] = gload<V>(pr.y + (long long)sizeof(V) * e);
      } else {
        rows[t] = gload<int>(adj[sg] + 4LL * e);
      }
    }
    bool bad = false;
#pragma unroll
    for (int t = 0; t < EW; ++t) {
      const unsigned r = (unsigned)rows[t] - (unsigned)rlo;
      bad |= r >= (unsigned)span;  // a row outside the unit's range: invalid input
      vr[t] = (int)min(r, (unsigned)(span - 1));
    }
    if (bad) atomicOr(a.err, ERR_INPUT);
    forget_derived<EW>(vr);
    unsigned bits = (unsigned)span;  // of the bitmap that the rows' bits (vr) index (up to 2^31 after ranking)
    bool fresh = true;  // the low bitmap is still clear
    unsigned* lb = top;
    for (; sh > 0; sh -= 5) {  // (uniform)
      unsigned short* lp = lb == top ? reinterpret_cast<unsigned short*>(smem + a.off_top + a.wg_top_bits / 8) : pw;
      const int ngrp = (int)((((bits - 1u) >> sh) + 64u) >> 6);
      if (lb != top) {
        for (int w = tid; w < 8 * ((ngrp + 3) >> 2); w += NT) lb[w] = 0u;
        __syncthreads();
        fresh = false;
      }
#pragma unroll
      for (int t = 0; t < EW; ++t) {
        in_fours(t);
        if (t < live) (void)or_bit(lb, vr[t] >> sh, tid + NT * t < u);
      }
      __syncthreads();
      forget_derived<EW>(vr);
      const int blocks = block_bitmap_prefix<NT>(lb, lp, ngrp, red0);
#pragma unroll
      for (int t = 0; t < EW; ++t) {
        in_fours(t);
        if (t < live) vr[t] = (bitmap_rank(lb, lp, vr[t] >> sh) << sh) | (vr[t] & ((1 << sh) - 1));
      }
      bits = (unsigned)blocks << sh;
      forget_derived<EW>(vr);
      if (lb != top) __syncthreads();  // (the next level clears this one's words)
      lb = bm;
    }
    const int ngrp = (int)((bits + 63u) >> 6);
    if (!fresh) {
      for (int w = tid; w < 8 * ((ngrp + 3) >> 2); w += NT) bm[w] = 0u;
      __syncthreads();
    }
    if constexpr (!NUM) {
      int newc = 0;
#pragma unroll
      for (int t = 0; t < EW; ++t) {
        in_fours(t);
        // (a copy past the end finds its row's bit clear at most once, and then in place of
        // the entry itself: no mask, which cost more than the one group's conflicts)
        if (t < live)
          newc += 1 - (int)__builtin_amdgcn_ubfe(atomicOr(&bm[vr[t] >> 5], 1u << (vr[t] & 31)), (unsigned)(vr[t] & 31), 1u);
      }
      int total = 0;
      (void)block_scan1<NT>(newc, red1, total);
      if (tid == 0) {
        if (WIN) a.win_cnt[unit] = total;
        else a.colcnt[j] = total;
      }
      return;
    } else {
      bool first[EW];
#pragma unroll
      for (int t = 0; t < EW; ++t) {
        in_fours(t);
        first[t] = false;
        if (t >= live) continue;
        const bool in = tid + NT * t < u;
        first[t] = or_bit(bm, vr[t], in) == 0u && in;
      }
      __syncthreads();
      forget_derived<EW>(vr);
      const int c = block_bitmap_prefix<NT>(bm, pw, ngrp, red1);
      if (c != cnt || c > a.wg_cap) {  // (uniform)
        if (tid == 0) atomicOr(a.err, ERR_COUNT);
        return;
      }
#pragma unroll
      for (int t = 0; t < EW; ++t) {
        in_fours(t);
        if (t < live) vr[t] = bitmap_rank(bm, pw, vr[t]);
      }
      __syncthreads();  // the staging area overlays the bitmaps
      forget_derived<EW>(vr);
      V* bv = reinterpret_cast<V*>(smem + a.off_bvals);
      int* br = reinterpret_cast<int*>(smem + a.off_brows);
      // first entries store at their rank, then the others add
#pragma unroll
      for (int t = 0; t < EW; ++t)
        if (first[t]) {
          bv[vr[t]] = vals[t];
          br[vr[t]] = rows[t];
        }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < EW; ++t)
        if (tid + NT * t < u && !first[t]) lds_add_cas<V>(&bv[vr[t]], vals[t]);
      __syncthreads();
      int* outr = a.out_r + o0;
      V* outv = (V*)a.out_v + o0;
      for (int e = tid; e < c; e += NT) {
        gstore_nt<int>((long long)(outr + e), br[e]);
        gstore_nt<V>((long long)(outv + e), bv[e]);
      }
    }
    return;
  }
  // more entries than registers (a window of at most wg_cap rows): one bit per row
  if (span > a.wg_cap) {  // (uniform; excluded by the window split)
    if (tid == 0) atomicOr(a.err, ERR_COUNT);
    return;
  }
  const int nseg = P[a.k];
  int ktop = 0;  // largest power of two <= nseg - 1
  while ((ktop << 1) <= nseg - 1) ktop = ktop ? ktop << 1 : 1;
  if (nseg <= 1) ktop = 0;
  unsigned short* dpw = reinterpret_cast<unsigned short*>(smem + a.off_dpre);
  int newc = 0;
  bool bad = false;
  for (int cb = 0; cb < u; cb += REGS) {
    int rows[EW];
#pragma unroll
    for (int t = 0; t < EW; ++t) {
      const int e = min(cb + tid + NT * t, u - 1);
      const int sg = seg_of(P, nseg, ktop, e);
      const long long ar = NUM ? reinterpret_cast<const longlong2*>(adj)[sg].x : adj[sg];
      rows[t] = gload<int>(ar + 4LL * e);
    }
#pragma unroll
    for (int t = 0; t < EW; ++t) {
      const unsigned r = (unsigned)rows[t] - (unsigned)rlo;
      bad |= r >= (unsigned)span;
      const unsigned x = min(r, (unsigned)(span - 1));
      newc += 1 - (int)__builtin_amdgcn_ubfe(atomicOr(&bm[x >> 5], 1u << (x & 31)), x & 31, 1u);
    }
  }
  if (bad) atomicOr(a.err, ERR_INPUT);
  if (!NUM) {
    int total = 0;
    (void)block_scan1<NT>(newc, red1, total);
    if (tid == 0) {
      if (WIN) a.win_cnt[unit] = total;
      else a.colcnt[j] = total;
    }
    return;
  }
  __syncthreads();
  const int c = block_bitmap_prefix<NT>(bm, dpw, (span + 63) >> 6, red1);
  if (c != cnt || c > a.wg_cap) {  // (uniform)
    if (tid == 0) atomicOr(a.err, ERR_COUNT);
    return;
  }
  // every entry adds into a zeroed staging area, which lies after this bitmap and its prefix
  V* bv = reinterpret_cast<V*>(smem + a.off_bvals);
  int* br = reinterpret_cast<int*>(smem + a.off_brows);
  for (int s = tid; s < c; s += NT) bv[s] = V(0);
  __syncthreads();
  for (int cb = 0; cb < u; cb += REGS) {
#pragma unroll
    for (int t = 0; t < EW; ++t) {
      const int e = cb + tid + NT * t;
      if (e < u) {
        const longlong2 pr = reinterpret_cast<const longlong2*>(adj)[seg_of(P, nseg, ktop, e)];
        const int row = gload<int>(pr.x + 4LL * e);
        const V v = gload<V>(pr.y + (long long)sizeof(V) * e);
        const unsigned r = (unsigned)row - (unsigned)rlo;
        if (r < (unsigned)span) {
          const int rk = bitmap_rank(bm, dpw, (int)r);
          br[rk] = row;  // every entry of a row writes the same row
          lds_add_cas<V>(&bv[rk], v);
        }
      }
    }
  }
  __syncthreads();
  int* outr = a.out_r + o0;
  V* outv = (V*)a.out_v + o0;
  for (int e = tid; e < c; e += NT) {
    gstore_nt<int>((long long)(outr + e), br[e]);
    gstore_nt<V>((long long)(outv + e), bv[e]);
  }
}

}  // namespace spk
