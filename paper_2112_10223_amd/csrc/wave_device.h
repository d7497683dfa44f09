// Device code of the wave-bin kernels: one wavefront per column, with a
// per-wavefront pipeline over its columns.  Included by the plain launch
// (wave_kernels.hip) and the batched launch (batch_kernels.hip).
//
// Wavefront gw of a launch of G wavefronts takes the bin's units gw, gw + G,
// gw + 2G, ... (at most 64).  While it accumulates one column in LDS, the column
// pointers of the column after next and the row (and value) loads of the next
// column are already in flight.  Two register sets alternate, and the loop is
// unrolled by two so that no register copy forces a wait.  Each lane keeps the base
// pointers of its KC inputs for the whole run: input lane for k <= 64 (KC = 1), inputs
// 2 lane and 2 lane + 1 for k <= 128 (KC = 2).
//
// Three accumulators, chosen per launch:
//  * hash (Algorithms 5 and 6): linear-probing LDS tables with compare-and-swap
//    claims; the numeric table is then compacted, bucketed by the top 8 bits of
//    (row - min row) and ranked inside each bucket, which sorts the column;
//  * bitmap: one bit per row of the matrix in LDS (the dense accumulator of
//    Algorithm 4 with the value array indexed by rank); the rank of a row among
//    the set bits is its output position, so the column comes out sorted with no
//    probing and no sort;
//  * ranked bitmap: the same over the non-empty 64-row blocks only, for matrices too
//    tall for a bitmap of all their rows.  A bitmap over the blocks gives each
//    non-empty block its rank, and the row's bit is rank(block) * 64 + row % 64: at
//    most 64 bits per entry, whatever the matrix's height.  It takes the place of the
//    hash tables, whose probing, compaction, bucket sort and larger slices (9.8 KiB a
//    wavefront at E = 8 against 5) cost more LDS instructions: 16 inputs of 1,000,003 x
//    150,001 with 12 rows per column, fp32: numeric 502 -> 178 us, symbolic 252 -> 131.
//    Where the bitmap over all rows fits, that one is faster (65,536 rows, E = 10:
//    numeric 169 against 199 us, symbolic 72 against 126).
// In every case the sorted column is written out coalesced.
#pragma once
#include "hash_common.h"

namespace spk {

// Levels of the ranked bitmap of an m-row matrix: the top level marks blocks of
// 2^shift rows (shift a multiple of 6) in nq rows of 8192 bits, at most RK_TOP_ROWS.
// The levels below it hold at most 64 sub-blocks of each of a column's at most 64 E
// non-empty blocks: rk_low_rows(E) rows of 8192 bits.
__host__ __device__ constexpr int rk_low_rows(int E) { return (E + 1) / 2; }
__host__ __device__ inline void rk_levels(int m, int& shift, int& nq) {
  shift = 6;
  while ((((long long)m + (1LL << shift) - 1) >> shift) > 8192LL * RK_TOP_ROWS) shift += 6;
  const long long blocks = ((long long)m + (1LL << shift) - 1) >> shift;
  nq = (int)((blocks + 8191) / 8192);
  if (nq < 1) nq = 1;
}

// KiB of the symbolic segment table: start mask (at most 128 bytes) and row pointers.
__host__ __device__ constexpr int sym_meta_rows(int KC) { return KC; }

// Entries of a lane whose table lookups are in flight together.  Up to E = 10 all of
// them; above, the registers they hold cost resident wavefronts.  With the ranked
// bitmap that starts at E = 10 (129 registers and three wavefronts per SIMD, 126 and four
// in groups of five: 96 -> 76 us on 32,768 columns of 480 entries).
__host__ __device__ constexpr int lookup_group(int E, bool ranked) {
  return E <= 8 ? E : E == 10 ? (ranked ? 5 : 10) : 4;
}

// Entry addresses of one unit.  The non-empty segments (inputs with entries in the
// column) are numbered in order, and each sets the bit of its start position in a
// 64 E-bit start mask.  The segment of position p is (#starts at positions <= p)
// - 1: per chunk of 64 positions, the starts of earlier chunks (a scalar count)
// plus mbcnt over the chunk's mask word.  Lanes past the end take the unit's last
// entry (every unit has u > 0), so no load is masked off.
template <int E, bool NUM, typename V, int ACC>
__device__ __forceinline__ void issue_unit_loads(const KArgs& a, unsigned char* base, const long long* adj, int u,
                                                 int (&rows)[E], V (&vals)[E]) {
  const int lane = lane_id();
  // lane t holds the start mask's word t
  const unsigned long long sw =
      reinterpret_cast<const unsigned long long*>(base + a.off_mark)[E == 16 ? lane & 15 : min(lane, E - 1)];
  const int swl = (int)(unsigned)sw, swh = (int)(unsigned)(sw >> 32);
  int before = -1;  // starts in earlier chunks, minus one
  // (addresses of a few entries at a time: more of them would only cost registers)
  constexpr int CH = lookup_group(E, (ACC & 3) == ACC_RANKED);
#pragma unroll
  for (int t0 = 0; t0 < E; t0 += CH) {
  if (t0 > 0) __builtin_amdgcn_sched_barrier(0);
  long long ar[CH], av[CH];
#pragma unroll
  for (int t = 0; t < CH; ++t) {
    // (readlane returns int: go through unsigned so the low word is not sign-extended)
    const unsigned hi = (unsigned)readlane(swh, t0 + t), lo = (unsigned)readlane(swl, t0 + t);
    const unsigned long long S = ((unsigned long long)hi << 32) | (unsigned long long)lo;
    const int seg = before + (int)(S & 1ull) + mbcnt(S >> 1);
    before += __popcll(S);
    if constexpr (NUM) {  // (rows, values) pointer pairs: one 16-byte read
      const longlong2 pr = reinterpret_cast<const longlong2*>(adj)[seg];
      ar[t] = pr.x;
      av[t] = pr.y;
    } else {
      ar[t] = adj[seg];
    }
  }
#pragma unroll
  for (int t = 0; t < CH; ++t) {
    const int e = min(lane + 64 * (t0 + t), u - 1);
    rows[t0 + t] = gload<int>(ar[t] + 4LL * e);
    if (NUM) vals[t0 + t] = gload<V>(av[t] + (long long)sizeof(V) * e);
  }
  }
}

// Column pointers of unit column j: a lane reads colptr_i[j], colptr_i[j+1] of its
// inputs i; lanes 0 and 1 also read colptr(B)[j], colptr(B)[j+1] for the numeric pass.
// Places past the last input hold its pointer and so repeat its reads.
// cpp holds the places of column 0, a.cpt's columns being cpt_stride(k) ints apart.
template <bool NUM, int KC>
__device__ __forceinline__ void issue_meta_loads(const KArgs& a, const long long (&cpp)[KC], int j, int (&s)[KC],
                                                 int (&e)[KC], int& cc) {
  const int lane = lane_id();
  const long long stride = a.cpt ? 4LL * cpt_stride(a.k) : 4LL;
  const long long at = stride * j;
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    s[c] = gload<int>(cpp[c] + at);
    e[c] = gload<int>(cpp[c] + at + stride);
  }
  if (NUM) cc = gload<int>((long long)(a.colptr_c + j + (lane & 1)));
}

// Segment table of a unit from its column pointers: the base pointers of the
// non-empty segments, shifted so that entry index (position in the unit) addresses
// them, in segment order, and the start mask.  Returns u.
template <int E, bool NUM, typename V, int KC>
__device__ __forceinline__ int build_unit_meta(const KArgs& a, unsigned char* base, const long long (&rip)[KC],
                                               const long long (&vap)[KC], const int (&s)[KC], const int (&e)[KC],
                                               long long* adj) {
  const int lane = lane_id();
  int len[KC], tot = 0, ord = 0;
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    len[c] = lane * KC + c < a.k ? e[c] - s[c] : 0;
    tot += len[c];
    ord += mbcnt(ballot(len[c] > 0));  // non-empty segments of the lanes below
  }
  const int incl = wave_scan_add(tot);
  unsigned* sb = reinterpret_cast<unsigned*>(base + a.off_mark);
  if (lane < 2 * E) sb[lane] = 0u;
  wave_sync();
  int ex = incl - tot;
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    if (len[c] > 0) {
      // numeric: (rows, values) pointer pairs in the 16-byte slots of adj
      if constexpr (NUM)
        reinterpret_cast<longlong2*>(adj)[ord] =
            make_longlong2(rip[c] + 4LL * (s[c] - ex), vap[c] + (long long)sizeof(V) * (s[c] - ex));
      else
        adj[ord] = rip[c] + 4LL * (s[c] - ex);
      atomicOr(&sb[ex >> 5], 1u << (ex & 31));
      ++ord;
    }
    ex += len[c];
  }
  return readlane(incl, 63);
}


// Coalesced write-out of an output column staged in LDS (rows br[0..c), values
// bv[0..c), rows ascending) at offset o0 of rowidx(B) / values(B).  Lanes past the
// end repeat the last entry's store (same address, same value).  With c == 0 (a failed
// unit) every lane stores into the write sink instead.  The base
// pointers are the same for the whole wavefront, so only the offsets are per lane.
template <int E, typename V>
__device__ __forceinline__ void write_column(const KArgs& a, int o0, int c, const int* br, const V* bv) {
  const int lane = lane_id();
  const bool live = c > 0;
  int* ob = live ? a.out_r + o0 : reinterpret_cast<int*>((char*)a.dummy + 2048);
  V* ov = live ? (V*)a.out_v + o0 : reinterpret_cast<V*>((char*)a.dummy + 2048 + 64);
  const int last = live ? c - 1 : 0;
  // every staged entry is read before the first store (one LDS round trip)
  int rr[E];
  V vv[E];
#pragma unroll
  for (int t = 0; t < E; ++t) {
    const int q = min(64 * t + lane, last);
    rr[t] = br[q];
    vv[t] = bv[q];
  }
  // uniform base (in scalar registers) + zero-extended 32-bit offset: no 64-bit
  // address arithmetic per lane
  const unsigned long long sob = uniform_u64((unsigned long long)ob);
  const unsigned long long sov = uniform_u64((unsigned long long)ov);
#pragma unroll
  for (int t = 0; t < E; ++t) {
    const unsigned q = (unsigned)min(64 * t + lane, last);
    gstore_nt<int>((long long)(sob + (unsigned long long)(q * 4u)), rr[t]);
    gstore_nt<V>((long long)(sov + (unsigned long long)(q * (unsigned)sizeof(V))), vv[t]);
  }
}

// Algorithms 5 and 6 on E entries per lane of a wavefront-private table, with
// linear probing.  Every entry of the wavefront probes at once, one step per round:
// a lane's E compare-and-swaps are in flight together, and the wavefront waits for
// its longest probe sequence once rather than once per index t.  A row's probe
// sequence depends only on the row, so concurrent inserts of the same row meet in
// the same slot.  NUM: once every row has its slot, the lanes whose claims created
// slots store their values (plain stores), then the lanes that found their row
// already there add with a compare-and-swap loop.  SYM counts first claims.
// Returns this lane's new keys.
template <int E, bool NUM, typename V>
__device__ __forceinline__ int insert_batch(int* K, V* Vt, int TS, int mode, int u, const int (&rows)[E],
                                            const V (&vals)[E], int* err) {
  const int lane = lane_id();
  // per entry: slot in the low 16 bits (TS <= 2048), state above: 0 probing,
  // 1 claimed the slot, 2 found its row there, 3 no entry
  constexpr int SH = 16, MASK = (1 << SH) - 1;
  int code[E];
#pragma unroll
  for (int t = 0; t < E; ++t) code[t] = hash_slot(rows[t], TS, mode) | ((lane + 64 * t < u ? 0 : 3) << SH);
  for (int probe = 0; probe < TS; ++probe) {
    bool pending = false;
#pragma unroll
    for (int t = 0; t < E; ++t) {
      if ((code[t] >> SH) == 0) {
        const int sl = code[t] & MASK;
        const int old = atomicCAS(&K[sl], -1, rows[t]);
        if (old == -1) code[t] = sl | (1 << SH);
        else if (old == rows[t]) code[t] = sl | (2 << SH);
        else {
          code[t] = sl + 1 == TS ? 0 : sl + 1;
          pending = true;
        }
      }
    }
    if (ballot(pending) == 0) break;  // (uniform)
  }
  int newc = 0;
#pragma unroll
  for (int t = 0; t < E; ++t) {
    if ((code[t] >> SH) == 0) atomicOr(err, ERR_PROBE);  // a full table: sized wrong
    newc += (code[t] >> SH) == 1 ? 1 : 0;
  }
  if (NUM) {
#pragma unroll
    for (int t = 0; t < E; ++t)
      if ((code[t] >> SH) == 1) Vt[code[t] & MASK] = vals[t];
    wave_sync();
#pragma unroll
    for (int t = 0; t < E; ++t)
      if ((code[t] >> SH) == 2) lds_add_cas<V>(&Vt[code[t] & MASK], vals[t]);
    wave_sync();
  }
  return newc;
}

// Numeric work of one unit: table, accumulation, compaction, bucket-rank sort,
// write-out.  The key and value arrays have 64 extra sink slots after ts_max; lanes
// without an entry write there, so no store is predicated.
template <int E, typename V>
__device__ __forceinline__ void num_unit(const KArgs& a, unsigned char* base, int u, int cnt, int o0, const int (&rows)[E],
                                         const V (&vals)[E]) {
  constexpr int NCH = 2 * E;  // 64-slot table chunks at load factor 1/2
  constexpr int RANK_UNROLL = 4;
  const int lane = lane_id();
  int* K = (int*)base;
  V* Vt = (V*)(base + (a.ts_max + 64) * 4);
  int* hist = (int*)(base + a.off_hist);  // 256 buckets + sink
  const int sink = a.ts_max + lane;
  int TS = slots_for(cnt, a.alpha_q);
  if (TS > NCH * 64) TS = NCH * 64;
#pragma unroll
  for (int c = 0; c < NCH; ++c) K[64 * c + lane] = -1;
  reinterpret_cast<int4*>(hist)[lane] = make_int4(0, 0, 0, 0);
  wave_sync();
  insert_batch<E, true, V>(K, Vt, TS, a.hash_mode, u, rows, vals, a.err);
  wave_sync();
  // compaction of the valid slots to A = [0, nc), slot order
  int kk[NCH];
  V vv[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    kk[c] = K[64 * c + lane];
    vv[c] = Vt[64 * c + lane];
  }
  int nc = 0, mn = INT_MAX, mx = -1;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const bool ok = kk[c] != -1;
    const uint64_t m = ballot(ok);
    const int dst = ok ? nc + mbcnt(m) : sink;
    K[dst] = kk[c];
    Vt[dst] = vv[c];
    nc += __popcll(m);
    mn = min(mn, ok ? kk[c] : INT_MAX);
    mx = max(mx, ok ? kk[c] : -1);
  }
  if (nc != cnt) {
    if (lane == 0) atomicOr(a.err, ERR_COUNT);
    nc = 0;  // write nothing for this unit
  }
  if (a.unsorted) {  // (uniform) table order
    wave_sync();
    write_column<E, V>(a, o0, nc, K, Vt);
    return;
  }
  mn = wave_total_min(mn);
  mx = wave_total_max(mx);
  const int bits = mx >= mn ? ceil_log2(mx - mn + 1) : 0;
  const int sh = bits > 8 ? bits - 8 : 0;
  wave_sync();
  // bucket histogram of A (bucket = top 8 bits of key - mn)
  int ka[E], dg[E];
  V va[E];
#pragma unroll
  for (int c = 0; c < E; ++c) {
    const int p = 64 * c + lane;
    ka[c] = K[p];
    va[c] = Vt[p];
    dg[c] = p < nc ? (ka[c] - mn) >> sh : 256;
    atomicAdd(&hist[dg[c]], 1);
  }
  wave_sync();
  {
    const int4 h = reinterpret_cast<int4*>(hist)[lane];
    const int tot = h.x + h.y + h.z + h.w;
    const int ex = wave_scan_add(tot) - tot;
    wave_sync();
    reinterpret_cast<int4*>(hist)[lane] = make_int4(ex, ex + h.x, ex + h.x + h.y, ex + h.x + h.y + h.z);
  }
  wave_sync();
  // scatter into buckets, B = [half, half + nc)
  const int half = NCH * 32;
#pragma unroll
  for (int c = 0; c < E; ++c) {
    const int pos = atomicAdd(&hist[dg[c]], 1);
    const int dst = dg[c] < 256 ? half + pos : sink;
    K[dst] = ka[c];
    Vt[dst] = va[c];
  }
  wave_sync();
  // rank inside the bucket (rows are unique), final order into A
#pragma unroll
  for (int c = 0; c < E; ++c) {
    const int p = 64 * c + lane;
    const bool ok = p < nc;
    const int key = K[half + p];
    const V val = Vt[half + p];
    const int d = ok ? (key - mn) >> sh : 0;
    const int be = ok ? hist[d] : 0;
    const int bs = (ok && d) ? hist[d - 1] : 0;
    // the first RANK_UNROLL members of the bucket without a loop, the rest in one
    int r = 0;
#pragma unroll
    for (int q = 0; q < RANK_UNROLL; ++q) {
      const int x = K[half + min(bs + q, NCH * 64 - 1)];
      r += (bs + q < be && x < key) ? 1 : 0;
    }
    if (ballot(be - bs > RANK_UNROLL) != 0)
      for (int q = bs + RANK_UNROLL; q < be; ++q) r += K[half + q] < key;
    const int dst = ok ? bs + r : sink;
    K[dst] = key;
    Vt[dst] = val;
  }
  wave_sync();
  write_column<E, V>(a, o0, nc, K, Vt);
}

// ---------------------------------------------------------------------------
// Bitmap accumulator for dense columns: a row-indexed bitmap in LDS (the sparse
// accumulator of Algorithm 4, with the dense array replaced by one bit per row and
// the value array indexed by rank).  Symbolic: OR the rows in, count the bits.
// Numeric: OR the rows in (the atomic OR's old word tells which entry came first),
// prefix-popcount the bitmap, and use rank(row) = #set bits below it as the output
// position.  That gives sorted output with no hash probing and no sort.  A first
// entry stores its row and value at that position; a later entry of the same row
// adds with compare-and-swap.
// The bitmap holds bm_nq x 256 words (bm_nq x 8192 rows).
// ---------------------------------------------------------------------------
// Exclusive popcount prefix per pair of words of an nq x 256 word bitmap into pw32 (two
// 16-bit prefixes per word; counts stay <= 1024).  Lane handles the 4 words (2 pairs)
// of group q*64 + lane.  Two bitmap rows share one scan, one in each 16-bit half: no
// partial sum exceeds the column's distinct rows, so the halves never carry into each
// other.  Returns the number of set bits.
__device__ __forceinline__ int bitmap_prefix(const uint4* bm4, unsigned* pw32, int nq) {
  const int lane = lane_id();
  int carry = 0;
  for (int q = 0; q < nq; q += 2) {
    const bool two = q + 1 < nq;
    const uint4 x = bm4[q * 64 + lane];
    const uint4 y = two ? bm4[(q + 1) * 64 + lane] : make_uint4(0u, 0u, 0u, 0u);
    const int x01 = __popc(x.x) + __popc(x.y), nx = x01 + __popc(x.z) + __popc(x.w);
    const int y01 = __popc(y.x) + __popc(y.y), ny = y01 + __popc(y.z) + __popc(y.w);
    const int packed = nx | (ny << 16);
    const int incl = wave_scan_add(packed);
    const int ex = incl - packed;
    const int tot = readlane(incl, 63);
    const int px = carry + (ex & 0xffff);
    carry += tot & 0xffff;
    const int py = carry + (ex >> 16);
    carry += tot >> 16;
    pw32[q * 64 + lane] = (unsigned)px | ((unsigned)(px + x01) << 16);
    if (two) pw32[(q + 1) * 64 + lane] = (unsigned)py | ((unsigned)(py + y01) << 16);
  }
  return carry;
}

// Ranks of E set bits (bit numbers r): the set bits below each.  A group's lookups are
// issued before the first is used (one LDS round trip).  (The word is
// picked by masking, not by a select: a select between two array elements is turned
// into an indexed scratch access.)
// BLOCKS: the bits are those of the blocks r >> sh, and rk gets the block's rank in
// place of its number (r and rk may be the same array).
template <int E, bool RANKED, bool BLOCKS = false>
__device__ __forceinline__ void bitmap_ranks(const unsigned* bm, const unsigned short* pw, const int (&r)[E],
                                             int (&rk)[E], int sh = 0) {
  constexpr int CH = lookup_group(E, RANKED);
#pragma unroll
  for (int t0 = 0; t0 < E; t0 += CH) {
    if (t0 > 0) __builtin_amdgcn_sched_barrier(0);
    unsigned plo[CH], phi[CH], pp[CH];
#pragma unroll
    for (int t = 0; t < CH; ++t) {
      const int w = r[t0 + t] >> (BLOCKS ? sh + 5 : 5);
      const uint2 pr = reinterpret_cast<const uint2*>(bm)[w >> 1];
      plo[t] = pr.x;
      phi[t] = pr.y;
      pp[t] = pw[w >> 1];
    }
#pragma unroll
    for (int t = 0; t < CH; ++t) {
      const int x = BLOCKS ? r[t0 + t] >> sh : r[t0 + t];
      const unsigned odd = 0u - (unsigned)((x >> 5) & 1);  // all ones for the second word of the pair
      const unsigned word = plo[t] ^ ((plo[t] ^ phi[t]) & odd);
      const int below = (int)pp[t] + (int)((unsigned)__popc(plo[t]) & odd) + __popc(word & ((1u << (x & 31)) - 1u));
      rk[t0 + t] = BLOCKS ? (below << sh) | (r[t0 + t] & ((1 << sh) - 1)) : below;
    }
  }
}

// Between the passes over a unit's entries: keeps the compiler from carrying word
// addresses, bits and masks of every entry from one pass to the next instead of forming
// them again (registers, and with them resident wavefronts).
template <int EW>
__device__ __forceinline__ void forget_derived(int (&vr)[EW]) {
#pragma unroll
  for (int t = 0; t < EW; ++t) asm volatile("" : "+v"(vr[t]));
}

// ORs bit r into the bitmap; returns its word before, masked to the bit.  A lane past
// the end (in false) ORs nothing, into a word of its own: 64 lanes at the copies' one
// word would take the LDS 64 turns (row windows with such groups skipped: R-MAT scale
// 20, 64 inputs, symbolic 2314 -> 1195 us).
__device__ __forceinline__ unsigned or_bit(unsigned* bm, int r, bool in) {
  const unsigned bit = in ? 1u << (r & 31) : 0u;
  return atomicOr(&bm[in ? r >> 5 : lane_id()], bit) & bit;
}

// Ranked bitmap: the rows of a unit (lanes past the end hold a copy of its last row)
// as bit numbers below 4096 E in the rows' order.  The top level marks the non-empty
// blocks of 2^rk_shift rows; a block's rank replaces its number, which leaves at most
// 64 E blocks.  While blocks are larger than 64 rows, they are divided into 64 again
// and ranked again.  A row outside the matrix (invalid input) counts as its last.
template <int E>
__device__ __forceinline__ void rank_rows(const KArgs& a, unsigned char* base, int u, const int (&rows)[E],
                                          int (&vr)[E]) {
  const int lane = lane_id();
  uint4* bm4 = reinterpret_cast<uint4*>(base);
  unsigned* bm = reinterpret_cast<unsigned*>(base);
  wave_sync();  // (the segment table read before shares the region)
#pragma unroll
  for (int t = 0; t < E; ++t) vr[t] = (int)min((unsigned)rows[t], (unsigned)max(a.m, 1) - 1u);
  int nq = a.rk_nq;
  for (int sh = a.rk_shift; sh > 0; sh -= 6) {  // (uniform)
    unsigned short* pw = reinterpret_cast<unsigned short*>(base + nq * 1024);
    for (int q = 0; q < nq; ++q) bm4[q * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
#pragma unroll
    for (int t = 0; t < E; ++t) {
      (void)or_bit(bm, vr[t] >> sh, lane + 64 * t < u);
    }
    wave_sync();
    forget_derived<E>(vr);
    bitmap_prefix(bm4, reinterpret_cast<unsigned*>(pw), nq);
    wave_sync();
    bitmap_ranks<E, true, true>(bm, pw, vr, vr, sh);
    forget_derived<E>(vr);
    wave_sync();
    nq = rk_low_rows(E);
  }
}

// ORs the rows' bits (vr) into the bitmap; returns the bits this lane found clear.
template <int E>
__device__ __forceinline__ int count_new(unsigned* bm, int u, const int (&vr)[E]) {
  const int lane = lane_id();
  int newc = 0;
#pragma unroll
  for (int t = 0; t < E; ++t) {
    const bool in = lane + 64 * t < u;
    newc += (or_bit(bm, vr[t], in) == 0u && in) ? 1 : 0;
  }
  return newc;
}

// Symbolic: OR the rows in; an OR that finds its bit clear counts a new row.  The
// bitmap is all zero on entry (cleared at the start of the run) and is left all
// zero: the words the unit touched are cleared again.
template <int E>
__device__ __forceinline__ int bm_sym_unit(const KArgs& a, unsigned char* base, int u, const int (&rows)[E]) {
  const int lane = lane_id();
  unsigned* bm = reinterpret_cast<unsigned*>(base + a.off_bm);
  const int newc = count_new<E>(bm, u, rows);
  wave_sync();
#pragma unroll
  for (int t = 0; t < E; ++t) bm[lane + 64 * t < u ? rows[t] >> 5 : lane] = 0u;
  wave_sync();
  return wave_total_add(newc);
}

// Entries of a column up to which the symbolic pass of the ranked bitmap counts in a hash
// table instead (columns of at most 64 entries): the levels of a bitmap cost the same for
// every column, probing and clearing a table of 64 or 128 slots grows with its entries.
// 150,000 columns, plan and symbolic pass in us, levels / tables: m = 2^20, u = 4 104.8 /
// 99.7, u = 20 105.3 / 116.6; m = 2^21, u = 10 119.9 / 104.6, u = 20 119.5 / 116.5, u = 32
// 119.7 / 127.3; m = 2^24, u = 10 115.6 / 105.7, u = 20 114.9 / 116.9; m = 2^28, u = 20 129.8 /
// 116.8, u = 32 130.0 / 127.2, u = 48 133.4 / 136.1.
__host__ __device__ inline int rk_short(int shift, int nq) {
  return shift == 6 ? (nq > 1 ? 5 * nq : 0) : 12 * (shift / 6 - 1) + 5 * nq;
}
constexpr int RK_SHORT_MOST = 24 + 5 * RK_TOP_ROWS;
static_assert(2 * RK_SHORT_MOST <= 128, "a short column's table has at most 128 slots");

// Symbolic: the distinct rows of a unit of at most RK_SHORT_MOST entries.
__device__ __forceinline__ int short_sym_unit(const KArgs& a, unsigned char* base, int u, const int (&rows)[1]) {
  const int lane = lane_id();
  int* T = reinterpret_cast<int*>(base);
  wave_sync();  // (the segment table read before shares the region)
  T[lane] = -1;
  T[64 + lane] = -1;
  wave_sync();
  const float none[1] = {0.f};
  const int newc = insert_batch<1, false, float>(T, nullptr, u <= 32 ? 64 : 128, 0, u, rows, none, a.err);
  wave_sync();
  return wave_total_add(newc);
}

// Symbolic over the ranked bitmap (cleared for every unit).
template <int E>
__device__ __forceinline__ int rk_sym_unit(const KArgs& a, unsigned char* base, int u, const int (&rows)[E]) {
  const int lane = lane_id();
  uint4* bm4 = reinterpret_cast<uint4*>(base);
  int vr[E];
  rank_rows<E>(a, base, u, rows, vr);
#pragma unroll
  for (int q = 0; q < rk_low_rows(E); ++q) bm4[q * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
  wave_sync();
  const int newc = count_new<E>(reinterpret_cast<unsigned*>(base), u, vr);
  wave_sync();
  return wave_total_add(newc);
}

// RK: over the ranked bitmap, whose levels all start at the slice's base.
// ORD (SPKADD_FLAG_ORDERED): every value is the sequential sum of its terms in input
// order.  A unit's entries are numbered input by input, 64 of them at a time in
// ascending groups, so only entries of one group can meet in a slot out of order: of
// the lanes still to add, the lowest of each slot (an LDS minimum) adds, until none is
// left (one round for a group without equal rows, at most 64).  A slot's first term is
// stored as it is (adding it to a zero would quiet a signalling NaN): a slot untouched
// before a group can only be so in the group's first round.  A row outside the matrix (invalid input)
// is reported and counts as the last of the bitmap: every rank stays below 64 E, where a
// lane reads back the minimum it took part in.  (A rank past the LDS, whose reads give 0,
// would leave the lanes above 0 adding for ever.)
template <int E, typename V, bool RK, bool ORD>
__device__ __forceinline__ void bm_num_unit(const KArgs& a, unsigned char* base, int u, int cnt, int o0,
                                            const int (&rows)[E], const V (&vals)[E]) {
  const int lane = lane_id();
  uint4* bm4 = reinterpret_cast<uint4*>(base + a.off_bm);
  unsigned* bm = reinterpret_cast<unsigned*>(bm4);
  unsigned short* pw = reinterpret_cast<unsigned short*>(base + a.off_pre);  // set bits below each word pair
  V* bv = reinterpret_cast<V*>(base + a.off_bvals);  // may overlay the bitmap (used after the ranks)
  // rows follow the 64 (E + 1) staged values (a.off_brows; a constant distance, so
  // one address serves both)
  int* br = reinterpret_cast<int*>(reinterpret_cast<unsigned char*>(bv) + 64 * (E + 1) * sizeof(V));
  const int nq = RK ? rk_low_rows(E) : a.bm_nq;
  int vr[E];  // the bits of the rows
  if constexpr (ORD) {
    bool bad = false;
#pragma unroll
    for (int t = 0; t < E; ++t) bad |= (unsigned)rows[t] >= (unsigned)a.m;
    if (bad) atomicOr(a.err, ERR_INPUT);
  }
  if constexpr (RK) {
    rank_rows<E>(a, base, u, rows, vr);
  } else {
#pragma unroll
    for (int t = 0; t < E; ++t) vr[t] = ORD ? (int)min((unsigned)rows[t], (unsigned)(8192 * nq) - 1u) : rows[t];
    if constexpr (ORD) forget_derived<E>(vr);
  }
  for (int q = 0; q < nq; ++q) bm4[q * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
  wave_sync();
  bool first[E];
#pragma unroll
  for (int t = 0; t < E; ++t) {
    const bool in = lane + 64 * t < u;
    first[t] = or_bit(bm, vr[t], in) == 0u && in;
  }
  wave_sync();
  if constexpr (RK || ORD) forget_derived<E>(vr);  // (the other bitmap is faster without, at the same residency)
  int c = bitmap_prefix(bm4, reinterpret_cast<unsigned*>(pw), nq);
  if (c != cnt) {
    if (lane == 0) atomicOr(a.err, ERR_COUNT);
    c = 0;
  }
  wave_sync();
  // rank(row) = set bits below it = output position; the first entry of a row puts
  // the row and its value there, later entries of the row add their values
  int rk[E];
  bitmap_ranks<E, RK>(bm, pw, vr, rk);
  if constexpr (RK || ORD) forget_derived<E>(rk);
  wave_sync();  // the bitmap is read for the last time above
  if constexpr (ORD) {
    // (the rows' places hold the adding lane or a slot's state until the rows are stored)
    constexpr int FREE = 64, UNTOUCHED = 65;
#pragma unroll
    for (int t = 0; t < E; ++t) br[64 * t + lane] = UNTOUCHED;
    wave_sync();
#pragma unroll
    for (int t = 0; t < E; ++t) {
      bool todo = lane + 64 * t < u;
      int state = br[rk[t]];
      // (uniform; every round ends its lowest lane's turn)
      for (int round = 0; round < 64 && ballot(todo) != 0; ++round) {
        if (todo) atomicMin(&br[rk[t]], lane);
        wave_sync();
        const bool mine = todo && br[rk[t]] == lane;
        wave_sync();
        if (mine) {
          bv[rk[t]] = state == UNTOUCHED ? vals[t] : bv[rk[t]] + vals[t];
          br[rk[t]] = FREE;
          todo = false;
        }
        state = FREE;
        wave_sync();
      }
    }
#pragma unroll
    for (int t = 0; t < E; ++t)
      if (lane + 64 * t < u) br[rk[t]] = RK ? rows[t] : vr[t];
    wave_sync();
  } else {
    // entries that are not first write into per-lane sink slots 64 E + lane
#pragma unroll
    for (int t = 0; t < E; ++t) {
      const int d = first[t] ? rk[t] : 64 * E + lane;
      bv[d] = vals[t];
      br[d] = rows[t];
    }
    wave_sync();
#pragma unroll
    for (int t = 0; t < E; ++t)
      if (lane + 64 * t < u && !first[t]) lds_add_cas<V>(&bv[rk[t]], vals[t]);
    wave_sync();
  }
  write_column<E, V>(a, o0, c, br, bv);
  if (RK) wave_sync();  // (the next unit's segment table shares the region)
}

// Marks the entry registers of a unit as needed here.  Called before the next
// unit's loads are issued: the compiler then waits for these loads with the
// previous unit's stores still in flight (stores count in vmcnt on this target,
// and a wait placed after newer loads would also wait for them).
template <int E, bool NUM, typename V>
__device__ __forceinline__ void require_loaded(const int (&rows)[E], const V (&vals)[E]) {
#pragma unroll
  for (int t = 0; t < E; ++t) {
    asm volatile("" ::"v"(rows[t]));
    if constexpr (NUM) asm volatile("" ::"v"(vals[t]));
  }
}

// Stores into the write sink as many store instructions as one pipeline step
// issues, so that the pipeline loop is entered with the same memory-counter history
// as its back edge (loads, then one unit's stores).  Otherwise the compiler merges
// the two histories at the loop head into a wait for every outstanding store.
template <int E, bool NUM, typename V>
__device__ __forceinline__ void prime_stores(const KArgs& a) {
  const int lane = lane_id();
  const long long dmy = (long long)a.dummy + 2048 + 8LL * lane;
  // (the empty asm statements keep the compiler from merging the repeated stores)
  if constexpr (NUM) {
#pragma unroll
    for (int t = 0; t < E; ++t) {
      gstore<int>(dmy, 0);
      asm volatile("" ::: "memory");
      gstore<V>(dmy, V(0));
      asm volatile("" ::: "memory");
    }
  } else {
    gstore<int>(dmy, 0);
  }
}

// The symbolic bitmap shares its LDS with the segment table (mark and pointers, at the
// slice's start), which is zeroed again once the unit's loads are issued.
template <int KC>
__device__ __forceinline__ void clear_meta(const KArgs& a, unsigned char* base) {
  wave_sync();
#pragma unroll
  for (int q = 0; q < sym_meta_rows(KC); ++q)
    reinterpret_cast<uint4*>(base)[q * 64 + lane_id()] = make_uint4(0u, 0u, 0u, 0u);
  wave_sync();
}

template <int E, bool NUM, typename V>
struct UnitRegs {
  int rows[E];
  V vals[E];
  int u, j, cnt, o0;
};

// One pipeline step: finish the metadata of unit t+1, start loads for units t+2
// (pointers) and t+1 (entries), then process unit t.
// Every step runs the same instruction sequence, so the compiler keeps the next unit's
// loads in flight (after the last unit the loads are of that unit again, unused).  The
// loop leaves after either step: replaying the last unit into the write sink to fill up
// an even count had every wavefront of the chip store to one cache line (16 inputs of
// 1,000,003 x 150,001: odd counts 258 us, even ones 162).
template <int E, bool NUM, typename V, int ACC, int KC>
__device__ __forceinline__ void pipe_step(const KArgs& a, unsigned char* base, int t, int nu, int ucol,
                                          const long long (&cpp)[KC], const long long (&rip)[KC],
                                          const long long (&vap)[KC], int (&ms)[KC], int (&me)[KC], int& mc,
                                          UnitRegs<E, NUM, V>& cur, UnitRegs<E, NUM, V>& nxt) {
  const int lane = lane_id();
  require_loaded<E, NUM, V>(cur.rows, cur.vals);
  {
    // one segment table: a unit's pointers are read into registers in the step
    // that writes them
    long long* adj = (long long*)(base + a.off_adj);
    nxt.j = readlane(ucol, min(t + 1, nu - 1));
    nxt.u = build_unit_meta<E, NUM, V, KC>(a, base, rip, vap, ms, me, adj);
    if (NUM) {
      nxt.o0 = readlane(mc, 0);
      nxt.cnt = readlane(mc, 1) - nxt.o0;
    }
    issue_meta_loads<NUM, KC>(a, cpp, readlane(ucol, min(t + 2, nu - 1)), ms, me, mc);
    wave_sync();
    issue_unit_loads<E, NUM, V, ACC>(a, base, adj, nxt.u, nxt.rows, nxt.vals);
    if constexpr (!NUM && ACC == ACC_BITMAP) clear_meta<KC>(a, base);
  }
  if constexpr (NUM && ACC != ACC_HASH) {
    bm_num_unit<E, V, (ACC & 3) == ACC_RANKED, (ACC & ACC_ORDERED) != 0>(a, base, cur.u, cur.cnt, cur.o0, cur.rows, cur.vals);
  } else if constexpr (NUM) {
    num_unit<E, V>(a, base, cur.u, cur.cnt, cur.o0, cur.rows, cur.vals);
  } else if constexpr (ACC != ACC_HASH) {
    int cnt;
    if constexpr (ACC == ACC_BITMAP) {
      cnt = bm_sym_unit<E>(a, base, cur.u, cur.rows);
    } else if constexpr (E == 1) {
      if (cur.u <= a.rk_short) cnt = short_sym_unit(a, base, cur.u, cur.rows);  // (uniform)
      else cnt = rk_sym_unit<E>(a, base, cur.u, cur.rows);
    } else {
      cnt = rk_sym_unit<E>(a, base, cur.u, cur.rows);
    }
    // one unconditional store instruction: every lane writes the count to its place (one
    // request; write-sink slots for the other lanes would be lines shared by the whole chip)
    gstore<int>((long long)(a.colcnt + cur.j), cnt);
    wave_sync();
  } else {
    int* T = (int*)base;
    int TS = slots_for(cur.u, a.alpha_q);
    if (TS > a.ts_max) TS = a.ts_max;
    for (int s = lane; s < TS; s += 64) T[s] = -1;
    wave_sync();
    const int newc = insert_batch<E, false, V>(T, nullptr, TS, a.hash_mode, cur.u, cur.rows, cur.vals, a.err);
    const int cnt = wave_total_add(newc);
    gstore<int>((long long)(a.colcnt + cur.j), cnt);
    wave_sync();
  }
}

// The pipeline over one wavefront's units: nu <= 64 unit column ids, lane t of
// ucol holding unit t.  Every unit has entries (u > 0).
template <int E, bool NUM, typename V, int ACC, int KC>
__device__ __forceinline__ void run_pipe(const KArgs& a, unsigned char* base, int nu, int ucol) {
  const int lane = lane_id();
  long long cpp[KC], rip[KC], vap[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const int li = min(lane * KC + c, a.k - 1);
    cpp[c] = a.cpt ? (long long)(a.cpt + li) : (long long)a.cp[li];
    rip[c] = (long long)a.ri[li];
    vap[c] = NUM ? (long long)a.va[li] : 0;
  }

  UnitRegs<E, NUM, V> A, B;
  int ms[KC], me[KC], mc = 0;
  // prologue: metadata and entry loads of unit 0, pointers of unit 1
  issue_meta_loads<NUM, KC>(a, cpp, readlane(ucol, 0), ms, me, mc);
  {
    long long* adj = (long long*)(base + a.off_adj);
    A.u = build_unit_meta<E, NUM, V, KC>(a, base, rip, vap, ms, me, adj);
    A.j = readlane(ucol, 0);
    if (NUM) {
      A.o0 = readlane(mc, 0);
      A.cnt = readlane(mc, 1) - A.o0;
    }
    issue_meta_loads<NUM, KC>(a, cpp, readlane(ucol, min(1, nu - 1)), ms, me, mc);
    wave_sync();
    issue_unit_loads<E, NUM, V, ACC>(a, base, adj, A.u, A.rows, A.vals);
  }
  if constexpr (!NUM && ACC == ACC_BITMAP) {  // the symbolic bitmap starts all zero and stays so
    wave_sync();
    uint4* bm4 = reinterpret_cast<uint4*>(base + a.off_bm);
    for (int q = 0; q < a.bm_nq; ++q) bm4[q * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
  }
  prime_stores<E, NUM, V>(a);
  for (int t = 0;;) {
    pipe_step<E, NUM, V, ACC, KC>(a, base, t, nu, ucol, cpp, rip, vap, ms, me, mc, A, B);
    if (++t >= nu) break;  // (uniform)
    pipe_step<E, NUM, V, ACC, KC>(a, base, t, nu, ucol, cpp, rip, vap, ms, me, mc, B, A);
    if (++t >= nu) break;
  }
}

// LDS layout of one wavefront's slice (bytes) for accumulator acc, kc inputs per lane.
// `rows` is the number of bitmap rows of 8192 bits (ACC_BITMAP) or the matrix's height
// (ACC_RANKED).  Region 1: the hash table (keys + 64 sink slots, then values and the
// 256-bucket histogram) or the bitmap (nq x 1 KiB) with its pair prefix (nq x 256 B);
// for the numeric bitmap the rows and values staged by rank overlay the bitmap when
// they fit in it.  Then the start mask (E 64-bit words) and the segment pointer table.
// The ranked bitmap keeps nothing in LDS from one unit to the next, and the segment
// table of the next unit is read (its loads issued) before this unit's accumulation
// starts: its levels, staging and segment table all share one region.
__host__ __device__ inline void pipe_layout(int E, bool numeric, int vbytes, int ts_max, int acc, int rows, int kc,
                                            KArgs& a) {
  const int adj_bytes = kc * 64 * (numeric ? 16 : 8);  // (rows, values) pointer pairs, or row pointers
  const int mark_bytes = (8 * E + 15) & ~15;
  a.ts_max = ts_max;
  a.bm_nq = a.rk_nq = a.rk_shift = a.rk_short = 0;
  if (acc == ACC_RANKED) {
    int shift = 0, nq = 0;
    rk_levels(rows, shift, nq);
    a.rk_shift = (short)shift;
    a.rk_nq = (short)nq;
    a.rk_short = (short)rk_short(shift, nq);
    const int low = rk_low_rows(E);
    a.off_bm = 0;
    a.off_pre = low * 1024;
    a.off_bvals = 0;
    a.off_brows = 64 * (E + 1) * vbytes;
    // (the symbolic pass needs no prefix of its last level)
    int bytes = low * (numeric || a.rk_shift > 6 ? 1280 : 1024);
    if (bytes < 1280 * a.rk_nq) bytes = 1280 * a.rk_nq;
    const int staged = numeric ? 64 * (E + 1) * (vbytes + 4) : 0;
    if (staged > bytes) bytes = staged;
    a.off_mark = 0;
    a.off_P = a.off_adj = a.off_adjv = mark_bytes;
    if (mark_bytes + adj_bytes > bytes) bytes = mark_bytes + adj_bytes;
    a.off_hist = 0;
    a.slice_bytes = (bytes + 15) & ~15;
    return;
  }
  const int bm_nq = acc == ACC_BITMAP ? rows : 0;
  int hash_bytes = (ts_max + 64) * 4;
  if (numeric) hash_bytes += (ts_max + 64) * vbytes + 272 * 4;
  int bm_bytes = 0;
  a.bm_nq = bm_nq;
  if (bm_nq > 0) {
    a.off_bm = 0;
    a.off_pre = bm_nq * 256 * 4;
    const int staged = 64 * (E + 1) * (vbytes + 4);  // 64 E positions + 64 sink slots
    a.off_bvals = staged <= a.off_pre ? 0 : a.off_pre + bm_nq * 256;
    a.off_brows = a.off_bvals + 64 * (E + 1) * vbytes;
    bm_bytes = !numeric ? a.off_pre : staged <= a.off_pre ? a.off_pre + bm_nq * 256 : a.off_brows + 64 * (E + 1) * 4;
  }
  int off = bm_nq > 0 ? bm_bytes : hash_bytes;
  off = (off + 15) & ~15;
  a.off_hist = ((ts_max + 64) * 4 + (ts_max + 64) * vbytes + 15) & ~15;  // used by the hash layout only
  if (!numeric && bm_nq > 0) {
    // the segment table is zeroed again after it is read, and shares the bitmap
    a.off_mark = 0;
    a.off_P = a.off_adj = a.off_adjv = mark_bytes;
    const int meta = sym_meta_rows(kc) * 1024;
    a.slice_bytes = off > meta ? off : meta;
    return;
  }
  if (numeric && bm_nq > 0 && mark_bytes + adj_bytes <= bm_nq * 256) {
    // The start mask and the segment table of the next unit are read (its loads
    // issued) before this unit writes its prefix words, and written again only after
    // the unit's ranks are read: they share the prefix region.
    a.off_mark = a.off_pre;
    a.off_P = a.off_adj = a.off_pre + mark_bytes;
    a.off_adjv = a.off_adj;
    a.slice_bytes = off;
    return;
  }
  a.off_mark = off;
  off += mark_bytes;
  a.off_P = a.off_adj = off;
  a.off_adjv = a.off_adj;  // (inside the pairs)
  off += adj_bytes;
  a.slice_bytes = (off + 15) & ~15;
}

}  // namespace spk
