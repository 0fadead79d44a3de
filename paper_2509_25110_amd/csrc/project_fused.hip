// Projection product with the Bessel tiles generated in LDS (gCAMB paper,
// Sec. 2.1 Eq. 2-3; per k the tau sum is Delta_k[l][c] = sum_n J_k[l][n] S_k[n][c]
// with J_k[l][n] = w_n j_l(k chi_n)), in two kernels per chunk of k rows:
//
// jseed_kernel (FP64, one lane per tau node): the node's top row R (below the
//   MFMA band cut ltop_mfma) and the pair w (j_R, j_{R+1}) (node_top_pair),
//   then ONE descending sweep that
//   leaves, at the top row of every 32-row segment at or below R, the pair
//   (w j_T, w j_{T+1}), T = min(R, segment top), in a seed table; also 1/x
//   and R per node and the largest R of every chunk of 64 nodes.  Nothing of
//   J itself is stored.
//
// tile_list_kernel (batches of many tiles): the (k row, TM-row l tile, TN-column
//   tile) items that hold data, as one list per XCD.
//
// fused_gemm_kernel (as many workgroups as the device holds, each taking tiles from the lists, or
//   one per possible tile): the tau axis advances in chunks of 64 nodes, visiting only the
//   chunks whose largest R reaches the tile (two ballots over the chunk table), and the sources,
//   seeds and R of the next such chunk are loaded while the matrix cores work on the current
//   one.  Per chunk every wave regenerates one 32-row segment of the l tile for the 64 nodes
//   from the seeds (FP64 recurrence in registers, one lane per node, rounded to FP32 -- or split
//   into bf16 hi/lo -- as it is written to LDS), the S columns of the tile are staged in LDS,
//   and the matrix cores multiply the two.  The recurrence runs with the same coefficient
//   cadence as the Bessel-table kernel (coefficient (2l+1)/x formed exactly at the rows 16b + 15
//   and 16b + 7 above lmin, stepped by -2/x in between), so the generated values are those of
//   the table, and the products are accumulated in the same order as the table-based kernels
//   (32-node blocks in increasing order; within a block the same fragment layout).
//
// Data per chunk row kc (workspace):
//   rtop[kc * ntp + n]                 R (absolute l) or -1 (no row in band)
//   nix[kc * ntp + n]                  1 / x (0 where R < 0)
//   seed[(kc * nseg + s) * ntp + n]    (w j_T, w j_{T+1}), T = min(R, lmin + 32 s + 31),
//                                      written for segments with lmin + 32 s <= R
//   cmax[kc * (ntp / 64) + c]          max of rtop over nodes 64 c .. 64 c + 63
//   rowtop[kc]                         max of the row's cmax
//   items, queue                       with lists: the tiles with data, per XCD, and the heads
// ntp = nodes padded to a multiple of 64 (at most 8192, so at most 128 chunks).
//
// What bounds it (48 models, 3 sources, l <= 5000, 8000 k, 3000 nodes; 84 to 102 columns a row):
// in FP32 the matrix cores, 19 ms of the products' 31 at their peak rate; the rest is what two
// workgroups a CU leave uncovered of the generation and staging.  One step of it was 51 ms, and
//   54.1 -> 51.2 ms  column blocks dealt to the waves in turn; no S staged past the columns in use
//   51.2 -> 41.1     tile lists and staying workgroups; rows above the band neither written nor
//                    read
//   41.1 -> 40.4     every wave takes all column blocks and two row blocks (2 x 2 waves with
//                    half of each had 2 of 4 column blocks idle at 96 of 128 columns)
//   40.4 -> 35.1     S and seed loads without tests or selects: the compiler had waited for them
//                    before the products (vmcnt(0)) instead of after
//   35.1 -> 33.3     a tile's column limits by one load; list heads on lines of their own
//   33.3 -> 33.1     128-row tiles with 8 waves, 4 on a SIMD, half of the column blocks each
// (the matrix cores busy 0.68 of the largest launch, 0.50 before).  7 models in split-BF16x3
// (9 to 21 columns): 3.46 -> 1.50 -> 1.47 ms; 256 models: 170 -> 143 -> 136 ms in FP32,
// 100 -> 74 -> 68 ms in split-BF16x3 (the last figure of each from the 8 waves).
// Slower: S fragments from device memory straight to the lanes, no S in LDS (79 ms: each wave
// loads them all, in half-used lines).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "bessel_dev.hpp"
#include "los_internal.hpp"

namespace los {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16;

constexpr int KB = 64;  // tau nodes per LDS chunk
constexpr int kQueueStride = 64;  // ints from one list's (head, length) to the next

__device__ inline int wave_max_int(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// Smallest set bit >= from of the 128-bit mask (a1:a0), or -1.
__device__ inline int next_chunk(uint64_t a0, uint64_t a1, int from) {
  if (from < 64) {
    const uint64_t m = a0 & (~0ull << from);
    if (m) return __ffsll((unsigned long long)m) - 1;
    from = 64;
  }
  if (from < 128) {
    const uint64_t m = a1 & (~0ull << (from - 64));
    if (m) return 64 + __ffsll((unsigned long long)m) - 1;
  }
  return -1;
}

// ------------------------------------------------------------------ seeds

__global__ __launch_bounds__(256) void jseed_kernel(FusedArgs a) {
  const int ki = blockIdx.y;
  const int64_t i = a.row_index ? a.row_index[a.k0 + ki] : a.k0 + ki;
  const int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (n >= a.ntp) return;
  int R = -1;
  double ix = 0.0, cur = 0.0, nxt = 0.0;
  if (n < a.ntau) {
    const double x = a.k[i] * (a.tau0 - a.tau[n]);
    const double wt = a.w[n];
    if (x >= kXTiny && wt != 0.0) {
      ix = 1.0 / x;
      R = node_top_pair(x, ix, wt, a.lmin, a.lmax, ltop_mfma_of(x), cur, nxt);
    }
  }
  // every lane of the wave is here (ntp is a multiple of 64): the wave's 64
  // nodes are chunk n / 64
  const int cm = wave_max_int(R);
  if ((threadIdx.x & 63) == 0) a.cmax[(int64_t)ki * (a.ntp / KB) + (n / KB)] = cm;
  const int64_t nb = (int64_t)ki * a.ntp + n;
  a.rtop[nb] = R;
  a.nix[nb] = R >= 0 ? ix : 0.0;
  if (R < 0) return;
  double2 *sd = a.seed + (int64_t)ki * a.nseg * a.ntp + n;
  const double d2 = ix + ix;
  // 16-row blocks b from R's block down to block 1; the pair at the top of
  // block b is stored when b is odd (a segment top) or b is R's own block.
  const int bR = (R - a.lmin) >> 4;
  for (int b = bR; b >= 1; --b) {
    if ((b & 1) || b == bR) sd[(int64_t)(b >> 1) * a.ntp] = make_double2(cur, nxt);
    if (b == 1) break;
    const int lbase = a.lmin + 16 * b;
    double t = 0.0;
#pragma unroll
    for (int r = 15; r >= 0; --r) {
      if (r == 15 || r == 7) t = (double)(2 * (lbase + r) + 1) * ix;
      const double pv = rec_step(t, cur, nxt);
      nxt = cur;
      cur = pv;
      t -= d2;
    }
  }
  if (bR == 0) sd[0] = make_double2(cur, nxt);
}

// ------------------------------------------------------------------ tile lists

// Last 16-row l block that column c0 of plan row r, the largest l_max from there on, needs.
__device__ inline int last_block(const FusedArgs &a, int64_t r, int c0) {
  const int last = a.nlb - 1;
  return a.col_lmax ? min(last, (a.col_lmax[a.col_off[r] + c0] - a.lmin) >> 4) : last;
}

// XCD x takes the rows of rank x, x + 8, ... (rank 0 = largest k, the most work): rows of the
// lists before list x.
__device__ inline int64_t list_base(int x, int kcount) {
  return (int64_t)x * (kcount / 8) + min(x, kcount % 8);
}

// The tiles with anything to compute, as one list per XCD (workgroup x): largest k first; within
// a row the l tiles of one column tile follow each other (they read the same S columns, kept in
// that XCD's L2).  Also the row's band top, and the lists' heads and lengths for the product's
// workgroups.  Launching a workgroup per possible tile instead left most of the chip idle where
// few tiles hold data (48 models, 3 sources, l <= 5000: the 900 smallest k, one full tile each,
// 1.38 ms; now 0.56 ms).  Transposed products only: untransposed, every tile has zeros to write.
__global__ __launch_bounds__(256) void tile_list_kernel(FusedArgs a, int tm, int tn, int tiles_m,
                                                        int tiles_n, int kcount, int places) {
  __shared__ int s_sum[4];
  const int x = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nch = (int)(a.ntp / KB);
  const int rows = (kcount - x + 7) / 8;
  int2 *out = a.items + list_base(x, kcount) * tiles_m * tiles_n;
  int done = 0;
  for (int i0 = 0; i0 < rows; i0 += 256) {
    const bool in = i0 + tid < rows;
    const int ki = kcount - 1 - (x + 8 * (i0 + tid));
    int n = 0, top = -1, ncol = 0;
    if (in) {
      const int *cm = a.cmax + (int64_t)ki * nch;
      for (int c = 0; c < nch; ++c) top = max(top, cm[c]);
      a.rowtop[ki] = top;
      ncol = a.col_cnt ? a.col_cnt[a.k0 + ki] : a.ncol;
      if (top >= a.lmin)
        for (int c0 = 0; c0 < ncol; c0 += tn)
          n += min(last_block(a, a.k0 + ki, c0), (top - a.lmin) >> 4) / (tm / 16) + 1;
    }
    int incl = n;  // inclusive sum over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    __syncthreads();  // the previous round's sums are read
    if (lane == 63) s_sum[w] = incl;
    __syncthreads();
    int at = done + incl - n;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (u < w) at += s_sum[u];
      done += s_sum[u];
    }
    if (n > 0)
      for (int c0 = 0; c0 < ncol; c0 += tn) {
        const int m = min(last_block(a, a.k0 + ki, c0), (top - a.lmin) >> 4) / (tm / 16) + 1;
        for (int u = 0; u < m; ++u) out[at++] = make_int2((int)((unsigned)u << 16 | ki), c0 / tn);
      }
  }
  if (tid == 0) {
    a.queue[kQueueStride * x] = places;
    a.queue[kQueueStride * x + 1] = done;
  }
}

// ------------------------------------------------------------------ product

template <int PREC>
struct LdsLayout;
template <>
struct LdsLayout<1> {  // FP32 rows of KB + 4 floats (272 bytes: 16 consecutive rows hit 16 bank groups)
  static constexpr int LD = KB + 4;
  static constexpr size_t bytes(int tm, int tn) { return sizeof(float) * (size_t)(tm + tn) * LD; }
};
template <>
struct LdsLayout<2> {  // bf16 hi and lo rows of KB + 8 (144 bytes: 16 rows hit 16 bank groups)
  static constexpr int LD = KB + 8;
  static constexpr size_t bytes(int tm, int tn) { return 2 * sizeof(u16) * (size_t)(tm + tn) * LD; }
};

__device__ inline u16 bf16_bits(__bf16 v) { return __builtin_bit_cast(u16, v); }

// x rounded to FP32, as a value the compiler may not look through: the bf16
// split that follows must round this FP32 value (as the table pipeline does),
// not x itself (a direct FP64 -> bf16 rounding differs in rare ties).
__device__ inline float f32_opaque(double x) {
  float v = (float)x;
  asm("" : "+v"(v));
  return v;
}

// One LDS stage: the J tile [TM][LD] and the S tile [TN][LD] (FP32), or hi and
// lo copies of each (bf16), starting at byte offset `base` of the shared memory.
template <int PREC, int TM, int TN>
struct Stage {
  float *Jf, *Sf;
  u16 *Jh, *Jl, *Sh, *Sl;
  __device__ Stage(unsigned char *base) {
    constexpr int LD = LdsLayout<PREC>::LD;
    Jf = (float *)base;
    Sf = Jf + TM * LD;
    Jh = (u16 *)base;
    Jl = Jh + TM * LD;
    Sh = Jl + TM * LD;
    Sl = Sh + TN * LD;
  }
};

// A workgroup's tile.
struct Tile {
  int ki, tm, ncol, c0, lb0, lb_last, tile_lo, top_cap;
  int nblk;  // 16-column blocks of the tile that need one of its rows (the first nblk)
  int64_t r, sbase, dbase;
};

// The tile (chunk row ki, l tile tm, column tile tn) of the list.  need: in lane j, the last
// 16-row block (relative to the tile) that column block j needs, from the l_max of its first
// column (columns are ordered by l_max, largest first, within a row); -1 where there is none.
// (One load for all blocks: block after block they made 16 us of each 200 us tile.)
template <int TM, int TN>
__device__ inline void tile_at(const FusedArgs &a, int ki, int tm, int tn, int lane, Tile &t,
                               int &need) {
  t.ki = ki;
  t.r = a.k0 + t.ki;
  t.lb0 = tm * (TM / 16);
  t.tm = tm;
  t.tile_lo = 16 * t.lb0;  // first row of the tile (l - lmin)
  t.ncol = a.col_cnt ? __builtin_amdgcn_readfirstlane(a.col_cnt[t.r]) : a.ncol;
  t.c0 = tn * TN;
  const int64_t off = a.col_off ? a.col_off[t.r] : 0;
  t.sbase = a.col_off ? off * a.s_cstride : t.r * a.s_kstride;
  t.dbase = a.col_off ? (off - a.col_base) * a.ldd : t.r * (int64_t)a.nl * t.ncol;
  need = -1;
  const int c = t.c0 + 16 * lane;
  if (lane < TN / 16 && c < t.ncol)
    need = (a.col_lmax ? min(a.nlb - 1, (a.col_lmax[off + c] - a.lmin) >> 4) : a.nlb - 1) - t.lb0;
  t.nblk = (int)__popcll(__ballot(need >= 0));
  t.lb_last = t.lb0 + __builtin_amdgcn_readfirstlane(need);
  t.top_cap = 16 * t.lb_last + 15 - t.tile_lo;  // last tile row any column needs
}

// Without lists every possible tile is a workgroup, dealt to the XCDs as the lists are; those past
// the row's columns or their l_max (y = -1) have nothing to do.  An XCD deals its workgroups to 4
// shader engines in turn: with an even number of tiles a row the same ones got every row's full
// tiles, unless the order turns with the row (l <= 2500, 4000 k, 3000 nodes, 3 sources: 3.36 -> 2.86
// ms, l <= 1000, 3000 k, 500 nodes: 490 -> 278 us; a kernel of its own, without the lists' loop: 2.79
// ms and 262 us, l <= 3000, 1500 k, 300 nodes 263 -> 239).
template <int TM, int TN>
__device__ inline int2 direct_tile(const FusedArgs &a, int per_row, int tiles_m, int kcount) {
  const int x = blockIdx.x & 7, s = blockIdx.x >> 3;
  const int row = s / per_row, pos = (s + (per_row & 1 ? 0 : row >> 1)) % per_row;
  const int ki = kcount - 1 - x - 8 * row, u = pos % tiles_m, tn = pos / tiles_m;
  if (ki < 0) return make_int2(0, -1);
  const int64_t r = a.k0 + ki;
  if (tn * TN >= (a.col_cnt ? a.col_cnt[r] : a.ncol) || u * (TM / 16) > last_block(a, r, tn * TN))
    return make_int2(0, -1);
  return make_int2((int)((unsigned)u << 16 | ki), tn);
}

// A workgroup's tiles from the lists (thread 0 only).  The first is its own: workgroup 8 s + x of
// the launch has place s of list x.  The rest of list x, from place gridDim.x / 8 on, and then of
// the other lists, are taken as they come.  A list's head is read before it is raised, and each
// has a cache line of its own: some hundred workgroups raising one line's heads at the end made
// 300 us.
__device__ inline int2 first_tile(const FusedArgs &a, int64_t per_row, int kcount, int &from) {
  const int x = blockIdx.x & 7, s = blockIdx.x >> 3;
  if (s < a.queue[kQueueStride * x + 1]) return a.items[list_base(x, kcount) * per_row + s];
  from = 8;  // list x has no more than one tile for each of its workgroups
  return make_int2(0, -1);
}

__device__ inline int2 next_tile(const FusedArgs &a, int64_t per_row, int kcount, int &from) {
  for (; from < 8; ++from) {
    const int y = (blockIdx.x + from) & 7;
    int *head = a.queue + kQueueStride * y;
    const int len = head[1];
    if (len <= (int)gridDim.x / 8 ||
        __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= len)
      continue;
    const int q = atomicAdd(head, 1);
    if (q < len) return a.items[list_base(y, kcount) * per_row + q];
  }
  return make_int2(0, -1);
}

// Active chunks: those whose largest top row reaches the tile's first row, as
// a 128-bit mask (the same in every wave), and the lane's entries of the
// chunk table (chunk_top reads them back).
struct Chunks {
  int cm0, cm1;
  uint64_t act0, act1;
};

__device__ inline Chunks active_chunks(const FusedArgs &a, const Tile &t, int lane) {
  const int nch = (int)(a.ntp / KB);  // <= 128
  const int *cmr = a.cmax + (int64_t)t.ki * nch;
  const int thr = a.lmin + t.tile_lo;
  Chunks ch;
  ch.cm0 = lane < nch ? cmr[lane] : -1;
  ch.cm1 = lane + 64 < nch ? cmr[lane + 64] : -1;
  ch.act0 = __ballot(ch.cm0 >= thr);
  ch.act1 = __ballot(ch.cm1 >= thr);
  return ch;
}

// The last tile row that holds data in chunk c (its largest R, capped).
__device__ inline int chunk_top(const FusedArgs &a, const Tile &t, const Chunks &ch, int c) {
  const int cmax = __shfl(c < 64 ? ch.cm0 : ch.cm1, c & 63, 64);
  return __builtin_amdgcn_readfirstlane(min(cmax - a.lmin - t.tile_lo, t.top_cap));  // uniform
}

// The S tile [TN columns][KB nodes] moves in 16-byte pieces, NTH threads.
template <int TN, int NTH>
struct SPieces {
  static constexpr int SP = TN * KB / 4;
  static constexpr int SPT = (SP + NTH - 1) / NTH;  // per thread (the last round may be partial)
};

// One chunk's inputs as one producing thread holds them: R, seed pair and 1/x
// of the lane's node (for the wave's segment) and the thread's S pieces.
template <int SPT>
struct ChunkIn {
  int R = -1;
  double2 sd = make_double2(0.0, 0.0);
  double nx = 0.0;
  f4 sv[SPT];
};

// What a producing wave needs to regenerate its segment and stage S.
struct Producer {
  int seg_hi;         // l - lmin of the segment's top row
  bool seg_ok;        // the segment exists (sg < nseg)
  int64_t rowb;       // chunk row offset in the per-node tables
  const double2 *seedp;
};

__device__ inline Producer producer_of(const FusedArgs &a, const Tile &t, int sg) {
  Producer p;
  p.seg_ok = sg < a.nseg;
  p.seg_hi = 32 * sg + 31;
  p.rowb = (int64_t)t.ki * a.ntp;
  p.seedp = a.seed + ((int64_t)t.ki * a.nseg + (p.seg_ok ? sg : a.nseg - 1)) * a.ntp;
  return p;
}

typedef f4 f4_any __attribute__((aligned(4)));  // a 16-byte load at any float

// No load here waits for another or is tested, and no value is touched, so that all are in
// flight until gen_segment and store_s take them: columns past the blocks in use read the last
// one (their products are not stored), and pieces that reach past tau the last four nodes
// (those past it meet zeros in J, and a non-finite value has reached the sums from its own
// node already).  TINY: fewer than 4 nodes, element by element.
template <int TN, int NTH, bool TINY>
__device__ inline void load_chunk_in(const FusedArgs &a, const Tile &t, const Producer &p, int c,
                                     int lane, int pt, ChunkIn<SPieces<TN, NTH>::SPT> &in) {
  constexpr int SPT = SPieces<TN, NTH>::SPT;
  const int n = c * KB + lane;
  in.R = a.rtop[p.rowb + n];
  in.nx = a.nix[p.rowb + n];
  in.sd = p.seedp[n];  // read whatever the node's R; used only below R
  const int last = (int)a.ntau - 1;
  const int ns = c * KB + pt * 4 % KB;  // the piece's first node, and its column
  const int cs = t.c0 + pt * 4 / KB, clast = min(t.c0 + 16 * t.nblk, t.ncol) - 1;
#pragma unroll
  for (int q = 0; q < SPT; ++q) {
    const float *src =
        a.S + t.sbase + (int64_t)min(cs + q * (NTH * 4 / KB), clast) * a.s_cstride;
    if (TINY) {
#pragma unroll
      for (int u = 0; u < 4; ++u) in.sv[q][u] = src[min(ns + u, last)];
    } else {
      in.sv[q] = *(const f4_any *)(src + min(ns, last - 3));
    }
  }
}

// Regenerate the 32 rows of a segment (tile rows tr_base .. tr_base + 31) for
// the lane's node, zeros above its R.  No branch per row: a node live only in
// the lower 16-row block enters the recurrence there from its seed, and rows
// above a node's R run the recurrence on zeros.
template <int PREC, int TM, int TN, int SPT>
__device__ inline void gen_segment(const FusedArgs &a, const Producer &p, const ChunkIn<SPT> &in,
                                   int tr_base, int lane, const Stage<PREC, TM, TN> &sm) {
  constexpr int LD = LdsLayout<PREC>::LD;
  const int Rrel = in.R - a.lmin;                       // < 0 when the node has no row
  const bool liveA = in.R >= 0 && Rrel >= p.seg_hi;       // live through the upper 16 rows
  const bool liveB = in.R >= 0 && Rrel >= p.seg_hi - 16;  // live in the lower 16 rows
  const double ix = liveB ? in.nx : 0.0;
  const double d2 = ix + ix;
  double cur = liveA ? in.sd.x : 0.0, nxt = liveA ? in.sd.y : 0.0;
#pragma unroll
  for (int half = 1; half >= 0; --half) {
    if (half == 0) {
      cur = liveA ? cur : (liveB ? in.sd.x : 0.0);
      nxt = liveA ? nxt : (liveB ? in.sd.y : 0.0);
    }
    const int hi_row = p.seg_hi - 16 * (1 - half);  // l - lmin of the block's top row
    const int tr0 = tr_base + 16 * half;            // tile row of the block's bottom row
    double tt = 0.0;
#pragma unroll
    for (int rr = 15; rr >= 0; --rr) {
      if (rr == 15 || rr == 7) tt = (double)(2 * (a.lmin + hi_row - 15 + rr) + 1) * ix;
      const float v = PREC == 1 ? (float)cur : f32_opaque(cur);
      const double pv = rec_step(tt, cur, nxt);
      nxt = cur;
      cur = pv;
      tt -= d2;
      const int row = tr0 + rr;
      if (PREC == 1) {
        sm.Jf[row * LD + lane] = v;
      } else {
        const __bf16 h = (__bf16)v;
        sm.Jh[row * LD + lane] = bf16_bits(h);
        sm.Jl[row * LD + lane] = bf16_bits((__bf16)(v - (float)h));
      }
    }
  }
}

// The thread's S pieces into the stage (FP32, or split into bf16 hi and lo).
// Pieces that cross the end of tau (over nodes past it, 1 to 3; 0: none in this chunk) were
// read from the last four nodes and are shifted here, those from node `edge` on.
template <int PREC, int TM, int TN, int NTH>
__device__ inline void store_s(ChunkIn<SPieces<TN, NTH>::SPT> &in, int nblk, int over, int edge,
                               int pt, const Stage<PREC, TM, TN> &sm) {
  if (over > 0) {  // uniform
    const bool cross = pt * 4 % KB >= edge;
    for (int o = 0; o < over; ++o)
#pragma unroll
      for (int q = 0; q < SPieces<TN, NTH>::SPT; ++q) {
        const f4 v = in.sv[q];
        in.sv[q] = cross ? f4{v[1], v[2], v[3], v[3]} : v;
      }
  }
  constexpr int LD = LdsLayout<PREC>::LD;
  constexpr int SP = SPieces<TN, NTH>::SP, SPT = SPieces<TN, NTH>::SPT;
#pragma unroll
  for (int q = 0; q < SPT; ++q) {
    if (q * NTH >= nblk * 4 * KB || (SP % NTH != 0 && q * NTH + pt >= SP)) break;
    const int e = (q * NTH + pt) * 4;
    const int col = e / KB, nn = e % KB;
    if (PREC == 1) {
      *(f4 *)(sm.Sf + col * LD + nn) = in.sv[q];
    } else {
      const f4 v4 = in.sv[q];
      u16 hh[4], ll[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const __bf16 h = (__bf16)v4[u];
        hh[u] = bf16_bits(h);
        ll[u] = bf16_bits((__bf16)(v4[u] - (float)h));
      }
      *(uint2 *)(sm.Sh + col * LD + nn) = make_uint2(hh[0] | ((unsigned)hh[1] << 16),
                                                     hh[2] | ((unsigned)hh[3] << 16));
      *(uint2 *)(sm.Sl + col * LD + nn) = make_uint2(ll[0] | ((unsigned)ll[1] << 16),
                                                     ll[2] | ((unsigned)ll[3] << 16));
    }
  }
}

// Products of one 32-node block of a wave's row blocks 0 .. M - 1 with a column block.
template <int PREC>
struct Frag;
template <>
struct Frag<1> {
  float v[8];
  __device__ void load(const float *hi, const float *, int ofs) {
    const float4 a = *(const float4 *)(hi + ofs), b = *(const float4 *)(hi + ofs + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};
template <>
struct Frag<2> {
  bf8 h, l;
  __device__ void load(const u16 *hi, const u16 *lo, int ofs) {
    h = *(const bf8 *)(hi + ofs);
    l = *(const bf8 *)(lo + ofs);
  }
};

template <int M>
__device__ __forceinline__ void products(f4 (&acc)[2], const Frag<1> (&a)[2], const Frag<1> &b) {
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int i = 0; i < M; ++i)
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].v[e], b.v[e], acc[i], 0, 0, 0);
}
template <int M>
__device__ __forceinline__ void products(f4 (&acc)[2], const Frag<2> (&a)[2], const Frag<2> &b) {
#pragma unroll
  for (int i = 0; i < M; ++i)
    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].l, b.h, acc[i], 0, 0, 0);
#pragma unroll
  for (int i = 0; i < M; ++i)
    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].h, b.l, acc[i], 0, 0, 0);
#pragma unroll
  for (int i = 0; i < M; ++i)
    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].h, b.h, acc[i], 0, 0, 0);
}

// One chunk's products for one wave: its row blocks are wr and wr + WR of the
// tile (those with data: 16 wr <= top_tr), its column blocks in turn; the two
// 32-node blocks of the chunk in increasing order.  Every accumulator sees its
// terms in the same order whichever wave owns it.  A wave holds the fragments
// of its rows and streams the columns', each read one block ahead.
template <int PREC, int TM, int TN, int WR, int WC, int NB>
__device__ inline void mfma_chunk(f4 (&acc)[NB][2], const int (&njb)[2], int wr, int wc,
                                  int top_tr, int g, int r16, const Stage<PREC, TM, TN> &sm) {
  constexpr int LD = LdsLayout<PREC>::LD;
  const int n0 = 16 * wr <= top_tr ? njb[0] : 0;
  const int n1 = 16 * (wr + WR) <= top_tr ? njb[1] : 0;  // <= n0
  if (n0 == 0) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int kofs = r16 * LD + 32 * h + 8 * g;
    Frag<PREC> fa[2], fb[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int ofs = 16 * (wr + WR * i) * LD + kofs;
      if constexpr (PREC == 1) fa[i].load(sm.Jf, nullptr, ofs);
      else fa[i].load(sm.Jh, sm.Jl, ofs);
    }
    auto load_b = [&](int j) {
      const int ofs = 16 * (WC * j + wc) * LD + kofs;
      if constexpr (PREC == 1) fb[j & 1].load(sm.Sf, nullptr, ofs);
      else fb[j & 1].load(sm.Sh, sm.Sl, ofs);
    };
    load_b(0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j < n0) {  // uniform
        if (j + 1 < NB) load_b(j + 1);
        if (j < n1) products<2>(acc[j], fa, fb[j & 1]);
        else products<1>(acc[j], fa, fb[j & 1]);
      }
    }
  }
}

// Accumulators to Delta: lane holds rows 4g + v of each 16-row block, column
// r16 of each column block.  Transposed (batch): columns of ldd >= 16 nlb
// floats, a multiple of 32, so a lane's four rows are one 16-byte store and 64
// bytes of a column go out together; blocks above the row's band (last_blk)
// and column blocks whose models stop below are not written, nor read later.
template <int WR, int WC, int NB>
__device__ inline void store_acc(const FusedArgs &a, const Tile &t, const f4 (&acc)[NB][2],
                                 const int (&njb)[2], int last_blk, int wr, int wc, int g,
                                 int r16) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int blk = t.lb0 + wr + WR * i;
    if (blk > last_blk) break;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int cc = t.c0 + 16 * (WC * j + wc) + r16;
      if (cc >= t.ncol) continue;
      if (a.dtrans) {
        if (j < njb[i])
          *(f4 *)(a.delta + t.dbase + (int64_t)cc * a.ldd + blk * 16 + 4 * g) = acc[j][i];
        continue;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = blk * 16 + 4 * g + v;
        if (row < a.nl) a.delta[t.dbase + (int64_t)row * t.ncol + cc] = acc[j][i][v];
      }
    }
  }
}

// A workgroup multiplies a (k row, 32 WR-row l tile, 16 NB WC-column tile) at a time with WR x WC
// waves: per active chunk the first WR waves regenerate one 32-row segment each, the threads
// stage S, and after a barrier wave (wr, wc) multiplies its row blocks wr and wr + WR
// (interleaved, so that the waves share a tile's partly filled upper blocks) by every WC-th
// column block from wc on; the next chunk's inputs load meanwhile.  The waves of one wr are on
// one SIMD (w and w + 4), so that any number of column blocks is shared evenly.
// LISTS: the workgroups stay and take tiles from the lists until these are empty; the list
// position of the next tile is fetched during the current one.  Otherwise each has one tile.
template <int PREC, int WR, int WC, int NB, bool TINY, bool LISTS>
__global__ __launch_bounds__(64 * WR * WC, WC == 2 ? 4 : 1) void fused_gemm_kernel(FusedArgs a, int per_row,
                                                                  int tiles_m, int kcount) {
  constexpr int NT = 64 * WR * WC, TM = 32 * WR, TN = 16 * NB * WC;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int2 s_item;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform
  const int g = lane >> 4, r16 = lane & 15;
  const int wr = w % WR, wc = w / WR;
  const Stage<PREC, TM, TN> sm(smem);
  // S pieces that cross the end of tau: in the last chunk, by `tail` nodes
  const int tail = TINY ? 0 : (int)(-a.ntau & 3), ctail = (int)(a.ntau / KB);
  int from = 0;
  int2 item = make_int2(0, -1);
  if (!LISTS || tid == 0) {
    if constexpr (LISTS) item = first_tile(a, per_row, kcount, from);
    else item = direct_tile<TM, TN>(a, per_row, tiles_m, kcount);
  }
  for (;;) {
    if constexpr (LISTS) {
      if (tid == 0) s_item = item;
      __syncthreads();
    }
    const unsigned mk = __builtin_amdgcn_readfirstlane(LISTS ? s_item.x : item.x);
    const int tn = __builtin_amdgcn_readfirstlane(LISTS ? s_item.y : item.y);
    if (tn < 0) return;
    const int ki = mk & 0xffff;
    if (LISTS && tid == 0) item = next_tile(a, per_row, kcount, from);
    Tile t;
    int need;
    tile_at<TM, TN>(a, ki, mk >> 16, tn, lane, t, need);
    const Producer p = producer_of(a, t, t.tm * WR + wr);
    const Chunks ch = active_chunks(a, t, lane);
    int last_blk = t.lb_last;
    if (a.dtrans) {
      int top;
      if (LISTS) {
        top = a.rowtop[ki];
      } else {  // no list kernel has left it: the row's first tile does
        top = wave_max_int(max(ch.cm0, ch.cm1));
        if (t.tm == 0 && tn == 0 && tid == 0) a.rowtop[ki] = top;
      }
      last_blk = min(last_blk, (top - a.lmin) >> 4);
    }

    f4 acc[NB][2];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j][0] = acc[j][1] = f4{0.f, 0.f, 0.f, 0.f};
    // column blocks whose models reach the wave's row blocks (the first njb[i]); the others'
    // products are skipped
    const int njb[2] = {((int)__popcll(__ballot(need >= wr)) + WC - 1 - wc) / WC,
                        ((int)__popcll(__ballot(need >= wr + WR)) + WC - 1 - wc) / WC};

    ChunkIn<SPieces<TN, NT>::SPT> in;
    int c = next_chunk(ch.act0, ch.act1, 0);
    if (c >= 0) load_chunk_in<TN, NT, TINY>(a, t, p, c, lane, tid, in);
    if (LISTS) __syncthreads();  // s_item is read
    while (c >= 0) {
      const int top_tr = chunk_top(a, t, ch, c);
      if (wc == 0 && p.seg_ok && 32 * wr <= top_tr) gen_segment(a, p, in, 32 * wr, lane, sm);
      store_s<PREC, TM, TN, NT>(in, t.nblk, c == ctail ? tail : 0, (int)a.ntau % KB / 4 * 4, tid,
                               sm);
      __syncthreads();
      // the next active chunk's inputs are in flight while the matrix cores run
      const int cn = next_chunk(ch.act0, ch.act1, c + 1);
      // (after the last the same again: a load under a condition would be waited for here)
      load_chunk_in<TN, NT, TINY>(a, t, p, cn >= 0 ? cn : c, lane, tid, in);
      // FP32: the wave's products go ahead of the other workgroup's segment
      // generation on the SIMD (1 % on C4; nothing for split-BF16x3)
      if constexpr (PREC == 1) __builtin_amdgcn_s_setprio(1);
      mfma_chunk<PREC, TM, TN, WR, WC, NB>(acc, njb, wr, wc, top_tr, g, r16, sm);
      if constexpr (PREC == 1) __builtin_amdgcn_s_setprio(0);
      __syncthreads();
      c = cn;
    }
    store_acc<WR, WC, NB>(a, t, acc, njb, last_blk, wr, wc, g, r16);
    if (!LISTS) return;
  }
}

// Per kernel and device: the large-LDS limit (a per-device function attribute) is set and the
// number of workgroups that the device holds at once is read on the first launch.  Threads that
// race here store the same values.
struct Resident {
  std::atomic<int> n[64] = {};
};

template <typename K>
hipError_t resident_blocks(K kern, int threads, size_t lds, Resident &r, int &n) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  n = r.n[dev].load();
  if (n > 0) return hipSuccess;
  if (lds > 64 * 1024) {
    e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
    if (e != hipSuccess) return e;
  }
  int cus = 0, per_cu = 0;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, threads, lds);
  if (e != hipSuccess) return e;
  n = (std::max(1, cus * per_cu) + 7) / 8 * 8;  // XCD = block index % 8
  r.n[dev].store(n);
  return hipSuccess;
}

template <int PREC, int WR, int WC, int NB, bool TINY = false>
hipError_t launch_fused_t(const FusedArgs &a, int kcount, int max_ncol, hipStream_t s) {
  constexpr int TM = 32 * WR, TN = 16 * NB * WC;
  const int tiles_m = (a.nlb * 16 + TM - 1) / TM, tiles_n = (max_ncol + TN - 1) / TN;
  if (kcount < 1 || max_ncol < 1 || kcount > 65535 || tiles_m > 65535) return hipErrorInvalidValue;
  const size_t lds = LdsLayout<PREC>::bytes(TM, TN);
  auto kern = fused_gemm_kernel<PREC, WR, WC, NB, TINY, true>;
  static Resident resident;
  int blocks = 0;
  hipError_t e = resident_blocks(kern, 64 * WR * WC, lds, resident, blocks);
  if (e != hipSuccess) return e;
  const int64_t tiles = (int64_t)kcount * tiles_m * tiles_n;
  // Lists or a workgroup per possible tile?  A tile from a list costs some 4 us of its own (heads
  // and items are read one after the other) and the list kernel 3 to 8: lists pay where many of
  // many tiles are empty.  Time with lists over without: 1 model of 60 k (60 tiles) 1.05, 200 of
  // 200 k (1000) 1.15, 2 of 400 k (1600) 1.05, 40 of 400 k, l <= 3500 (11 000) 0.98, 20 of 3000 k
  // (48 000) 0.90.  Untransposed every tile is written: 60 x 4000 x 4096 nodes 1.04, 2500 x 4000
  // x 3000 1.14, 3000 x 1500 x 300 1.66.
  if (a.dtrans && tiles > 2 * blocks) {
    hipLaunchKernelGGL(tile_list_kernel, dim3(8), dim3(256), 0, s, a, TM, TN, tiles_m, tiles_n,
                       kcount, blocks / 8);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else {
    const int64_t direct = (int64_t)(kcount + 7) / 8 * 8 * tiles_m * tiles_n;
    // (a launch counts its threads in 32 bits; at most 4 columns: always enough)
    if (direct * (64 * WR * WC) >= (int64_t)1 << 32) return hipErrorInvalidValue;
    blocks = (int)direct;
    kern = fused_gemm_kernel<PREC, WR, WC, NB, TINY, false>;
    static Resident attributes;  // (the large-LDS limit of this kernel)
    int unused = 0;
    e = resident_blocks(kern, 64 * WR * WC, lds, attributes, unused);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * WR * WC), lds, s, a,
                     tiles_m * tiles_n, tiles_m, kcount);
  return hipGetLastError();
}

// Registers spilled: with lists, 128 x 128 tiles 1 (the price of 4 waves a SIMD); 256 x 256 1 in FP32
// and 73 (296 bytes a lane) in split-BF16x3, where the batch tuner times it all the same and finds
// it 3 times slower on C4.
template <int PREC>
hipError_t launch_fused_p(const FusedArgs &a, int shape, int kcount, int max_ncol,
                          hipStream_t s) {
  if (a.ntau < 4) return launch_fused_t<PREC, 4, 1, 1, true>(a, kcount, max_ncol, s);
  switch (shape) {
    case 0:
    case 2: return launch_fused_t<PREC, 8, 1, 8>(a, kcount, max_ncol, s);   // 256 x 128
    case 1: return launch_fused_t<PREC, 4, 2, 4>(a, kcount, max_ncol, s);   // 128 x 128
    case 3: return launch_fused_t<PREC, 8, 1, 16>(a, kcount, max_ncol, s);  // 256 x 256
    case 4: return launch_fused_t<PREC, 8, 1, 1>(a, kcount, max_ncol, s);   // 256 x 16
    case 5: return launch_fused_t<PREC, 4, 1, 1>(a, kcount, max_ncol, s);   // 128 x 16
    case 6: return launch_fused_t<PREC, 4, 2, 2>(a, kcount, max_ncol, s);   // 128 x 64
    case 7: return launch_fused_t<PREC, 4, 2, 1>(a, kcount, max_ncol, s);   // 128 x 32
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

FusedShape fused_shape_at(int i) {
  static const FusedShape shapes[kFusedShapeCount] = {
      {256, 128}, {128, 128}, {256, 128}, {256, 256}, {256, 16}, {128, 16},
      {128, 64},  {128, 32}};
  return shapes[i];
}

// Tiles of a row at most: 128 rows by 16 columns is the smallest tile.
static size_t row_tiles(int nseg, int max_ncol) {
  return (size_t)((nseg + 3) / 4) * (size_t)((max_ncol + 15) / 16);
}

size_t fused_seed_bytes_per_row(int nseg, int64_t ntp, int max_ncol) {
  return (size_t)ntp * (sizeof(int) + sizeof(double) + sizeof(double2) * (size_t)nseg) +
         sizeof(int) * (size_t)(ntp / KB + 1) + sizeof(int2) * row_tiles(nseg, max_ncol);
}

void fused_workspace_at(FusedArgs &a, void *ws, int kcount, int max_ncol) {
  char *p = (char *)ws;
  a.queue = (int *)p;
  p += kFusedFixedBytes;
  a.seed = (double2 *)p;
  p += sizeof(double2) * (size_t)a.nseg * a.ntp * kcount;
  a.nix = (double *)p;
  p += sizeof(double) * (size_t)a.ntp * kcount;
  a.items = (int2 *)p;
  p += sizeof(int2) * row_tiles(a.nseg, max_ncol) * kcount;
  a.rtop = (int *)p;
  p += sizeof(int) * (size_t)a.ntp * kcount;
  a.cmax = (int *)p;
  p += sizeof(int) * (size_t)(a.ntp / KB) * kcount;
  a.rowtop = (int *)p;
}

hipError_t jseed_launch(const FusedArgs &a, int kcount, hipStream_t s) {
  dim3 grid((unsigned)((a.ntp + 255) / 256), (unsigned)kcount);
  hipLaunchKernelGGL(jseed_kernel, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t fused_gemm_launch(const FusedArgs &a, int prec, int shape, int kcount, int max_ncol,
                             hipStream_t s) {
  if (prec == 1) return launch_fused_p<1>(a, shape, kcount, max_ncol, s);
  if (prec == 2) return launch_fused_p<2>(a, shape, kcount, max_ncol, s);
  return hipErrorInvalidValue;
}

}  // namespace los
