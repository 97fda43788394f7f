// psl_dev.h -- device state and device helpers of libpsl (gfx950, wave64).
//
// Layout in HBM (one presolver handle):
//   CSR   rp[m+1] i32, ci[N] i32, va[N] f64              (input, read-only)
//   CSC   cp[n+1] i32, ri[N] i32, cva[N] f64             (built at ingest)
//   rows  lhs/rhs[m] f64, row_on[m] u8, row_code[m] u8, row_out[m] 16 B
//   cols  bnd[n] double2 (lb, ub), bkey[2n] i64 (order-mapped accumulators of
//         the round's best lb / ub, both largest key first), src[2n] i32, col_len[n] i32, c[n] f64
//   bins  bins[m] {row, start, len} (rows grouped by CSR length: those of the
//         ingest all rows, ascending within a bin; a selection's the rows to
//         sweep, ascending within a tile of rows, the tiles in any order)
// A column is removed exactly when lb == ub: a fixed column keeps lb = ub = v,
// and every active column has ub - lb > fix_tol * max(1, |lb|) >= 0 once a
// round has run, so the sweep learns a column's state from its bounds alone.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define PSL_BLOCK 256
#define PSL_WAVE 64

namespace psl {

enum : uint8_t {
  REC_FIX_COL = 1, REC_EMPTY_COL = 2, REC_EMPTY_ROW = 3, REC_REDUNDANT_ROW = 4,
  REC_SINGLETON_ROW = 5, REC_BOUND_CHANGE = 6, REC_PARALLEL_ROW = 7, REC_LEADER_SIDES = 8,
  REC_DUAL_FIX = 9, REC_FREE_SINGLETON = 10, REC_PARALLEL_COL = 11, REC_LEADER_BOUNDS = 12,
  REC_FORCING_ROW = 13, REC_DOUBLETON_ROW = 14, REC_DOMINATED_COL = 15
};

// row decision codes written by the sweep for the current round
enum : uint8_t { RC_KEEP = 0, RC_EMPTY = 1, RC_REDUNDANT = 2, RC_SINGLETON = 3, RC_FORCE_MIN = 4, RC_FORCE_MAX = 5 };

// column decision bits of a round
enum : uint8_t {
  CC_LB = 1, CC_UB = 2, CC_FIX = 4, CC_EMPTY = 8, CC_UNBOUNDED = 16, CC_INFEAS = 32,
  CC_LBFIN = 64, CC_UBFIN = 128  // set at emission: lb (ub) went from infinite to finite
};
// a dual fixing sets both CC_FIX and CC_EMPTY (never set together otherwise)
#define CC_DUALFIX (CC_FIX | CC_EMPTY)

// row length bins: rows of <= 4 / <= 8 / <= 16 entries by 4- / 8- / 16-lane
// groups (the 8-lane bin is optional: its bound is 4 or 8), rows of <= 64 /
// <= 256 / <= 512 entries by one wavefront (1 / 4 / 8 contiguous positions per
// lane), longer rows split into workgroup chunks
enum { BIN_G4 = 0, BIN_G8 = 1, BIN_G16 = 2, BIN_W1 = 3, BIN_W4 = 4, BIN_W8 = 5, BIN_LONG = 6, NBINS = 7 };

#define PASS_LEN 2048      // positions per workgroup pass (256 lanes x 8)
#define LONG_MAX_CHUNKS 512
#define LONG_MAX_PASSES 64   // rows up to 512 chunks x 64 passes x 2048 positions

struct Record {
  uint8_t type, side;
  uint16_t round;
  int32_t i, j, k;
  double v[4];
};
static_assert(sizeof(Record) == 48, "record layout");

struct RowOut {      // what the sweep leaves for a removed row's record
  double v0, v1;     // (activity, -) / (min act, max act) / (a_ij, -)
  int32_t j, pad;
};

struct Cand {        // a candidate bound that may be the round's final value
  int32_t js;        // 2*j + side (side 1 = upper)
  int32_t pos;       // CSR position of the entry (its row and coefficient)
  double t;
};

struct LongChunk {   // one workgroup's slice of a long row: npass passes of PASS_LEN
  int32_t row, first;  // row index, first CSR position (relative to row start)
  int32_t lrow, npass; // index of the long row, passes per chunk
  int32_t cand_off;    // start of its candidate region (after the other bins')
  int32_t id;          // index of its partial statistics (stable under filtering)
};

struct BinEnt {      // one row of a bin list
  int32_t row, start, len, pad;
};

// Candidate regions: every sweep workgroup appends to its own region of the
// candidate buffer (an LDS counter, no global atomics). A region holds two
// candidates per position the workgroup can visit.

struct LongPart {    // partial statistics of one chunk (an aligned subtree)
  double smin, smax;
  int32_t nmin, nmax, L, tiny;  // tiny: active entries with |a| < coef_tol
};

struct LongRow {     // per long row
  int32_t row, chunk0, nchunk, npass;
};

// Batched presolve: K LPs form one block-diagonal LP (the rows and columns of
// LP k are contiguous, its entries use the shifted column indices). Every LP
// keeps its own round count and stopping state, so its records and reduced
// problem are those of presolving it alone.
struct LpFlags {     // per LP, cleared before every round
  int32_t infeasible, unbounded, merged, pad;
};

struct LpOut {       // per LP: nonzero when the last round gave it records (cleared per round)
  int32_t total, pad;
};

// A count of a row selection, on a cache line of its own (every workgroup of
// the selection adds to it).
struct SelCnt {
  int32_t v, pad[15];
};
// counts of a selection: rows per bin, long-row chunks, nonzeros
enum { SEL_CHUNKS = NBINS, SEL_NNZ = NBINS + 1, SEL_N = NBINS + 2 };

// Rows and nonzeros swept so far in the run, spread over cache lines.
#define SWEPT_SLOTS 16
struct Swept {
  unsigned long long rows, nnz;
  int64_t pad[6];
};

struct Flags {
  int32_t infeasible, unbounded, error, merged;
  int32_t round_total, vlist_count, rows_removed;
  int32_t fin_cols;        // columns of the round with a bound that became finite
  int32_t mode;            // the next round's selection mode (bit 0: touched rows
                           // only, bit 1: inert rows skipped), set with the decisions
  int64_t error_pos;
  int32_t lead_count;      // parallel pass: leaders whose merged sides add locks
  int32_t fs_picks;        // the last round with a free singleton candidate
  int32_t fs_rows;         // chunks of long eliminated rows listed
  int32_t fs_claims;       // chunks of long substituting rows listed
  int32_t dbl_count;       // doubleton-equality candidates listed
  int32_t dbl_applied;     // a doubleton substitution was applied this pass
  int32_t n_dense, bins[NBINS];  // ingest: columns in dense_cols; rows of each bin
  // rounds queued ahead of the host: a round's kernels do nothing when its
  // number is above stop_at, which the last round's control sets
  int32_t stop_at, rounds_done;
  int64_t rec_base;                  // first record of the running round
  int64_t rec_at, rec_cap;           // next free record; records the buffer holds
  int64_t sum_rows, sum_nnz, sum_cols;  // swept so far in the run: rows, nonzeros, columns at most
  uint64_t stamp[3];       // clock at the round's long-row statistics, sweep, decisions
  uint64_t ticks[3];       // clock ticks of those phases so far in the run
  SelCnt sel[2][SEL_N];    // counts of the full view / of the rounds' selections
  Swept swept[SWEPT_SLOTS];  // (direct sweeps)
};

struct Cfg {
  double feas_tol, fix_tol, min_improve, par_tol, inf_value, coef_tol;
  int32_t dual_fix;        // lock-based dual fixing on
  int32_t free_sing;       // zero-cost free column singletons eliminated
  int32_t forcing;         // forcing rows on
};

struct HashSlot {
  unsigned long long key;
  unsigned int leader;   // (inequality << 31) | row, minimised
  unsigned int pad;
};

struct Dev {
  int32_t m, n;
  int64_t nnz;
  const int32_t *rp, *ci;
  const double *va;
  const int32_t *cp, *ri;
  const double *cva;
  double *lhs, *rhs;
  double2 *bnd;
  long long *bkey;
  int32_t *src;
  double *c;                   // costs (a working copy: substitutions change them)
  unsigned long long *owner;   // free singletons: per column the lowest claim, (~round << 32) | row,
                               // so a claim of the current round beats an older one (reset per run)
  uint8_t *fs_bad;             // per row: a long substituting row lost a column
  int32_t *col_len;
  uint8_t *row_on, *row_code, *col_code;
  uint8_t *dirty;          // rows touched by a column change: the mark (round_mark) of
                           // the round after it, so that no mark needs clearing
  uint8_t *dirty_tile;     // per 1024 rows, the same for some row of it (the row
                           // selection skips the other tiles when it takes
                           // marked rows only)
  const int32_t *rowid1;   // row of CSR position p at index p + 1 (built at ingest)
  int2 *rinf;              // per row: infinite min / max contributions at its last
                           // sweep, lowered as bounds of its columns become finite
  int32_t *dense_cols;     // columns of more than 4096 entries (listed at ingest)
  int32_t *n_dense;
  uint8_t *touch;          // columns whose decision may change this round
  unsigned long long *locks;  // dual fixing: per column, the alive rows keeping it
                              // from decreasing (low 32 bits) / increasing (high)
  // free singletons: per column and side, -1 = infinite input bound not changed,
  // r >= 0 = infinite input bound tightened only from row r, -2 = otherwise
  int32_t *lsrc, *usrc;
  uint8_t *fs_flag;        // column to check for a free singleton this round
  int32_t *fs_pick;        // per row: lowest candidate column (INT32_MAX: none)
  const uint32_t *colid;   // column of each position of the transposed copy
  RowOut *row_out;
  Cand *cand;
  int32_t *cand_cnt;   // candidates written per sweep workgroup
  Flags *flags;
  int32_t *cnt, *off;
  Record *rec;
  // the rows a launch takes: lists in fixed places (bin b's from bin_off[b], room
  // for every row of the bin), their lengths in sel
  const BinEnt *bins;
  int32_t bin_off[NBINS + 1];
  const SelCnt *sel;
  int32_t look_first;          // some column has more than MARK_DENSE entries
  int32_t direct;              // the lists hold every row (those of the ingest): a
                               // kernel tests each row itself, sel is not used
  const LongChunk *lchunk;
  const LongChunk *chunks0;    // chunk table of all long rows (built at ingest)
  LongPart *lpart;
  LongRow *lrow;
  int32_t nlong, nchunks;      // long rows and their chunks (of all rows)
  // the decision tiles' sums: per 64 tiles the records, the columns with a bound
  // made finite and the tiles done (fields of a word), groups of 64 tiles
  // done, and the records before each
  unsigned long long *super;
  int32_t *super_done, *super_off;
  // batched presolve (K LPs); with K == 1 every row and column is in LP 0
  // and none of these arrays is read
  int32_t K;
  const int32_t *row_lp, *col_lp;     // LP of each row / column
  const int32_t *lp_row0, *lp_col0;   // [K+1] first row / column of each LP
  uint8_t *lp_ok;                     // [K] LP still presolving (its rows stay in the bins;
                                      // cleared here when the LP stops)
  uint8_t *lp_run;                    // [K] lp_ok at the start of the round, kept through it
  const int32_t *lp_round;            // [K] the LP's own number of the current round
  int32_t *lp_round_next;             // the same after the round, written by its control
  LpFlags *lpf;                       // [K]
  LpOut *lpo;                         // [K]
  Cfg cfg;
};

__device__ __forceinline__ int row_lp_of(const Dev& d, int i) { return d.K > 1 ? d.row_lp[i] : 0; }
__device__ __forceinline__ int col_lp_of(const Dev& d, int j) { return d.K > 1 ? d.col_lp[j] : 0; }
// round number written into a record of LP lp
__device__ __forceinline__ int round_of(const Dev& d, int lp, int round) { return d.K > 1 ? d.lp_round[lp] : round; }
// the round with launch number seq is not run: an earlier one ended the rounds
__device__ __forceinline__ bool round_over(const Dev& d, int seq) { return seq > d.flags->stop_at; }

// the mark of rows to sweep in the round with launch number seq, 1 .. 255 (a
// mark left from 255 rounds before only sweeps its row once more)
__device__ __forceinline__ uint8_t round_mark(int seq) { return (uint8_t)(1 + (unsigned)seq % 255u); }

// rows of bin b in the lists (at most)
__device__ __forceinline__ int bin_rows_listed(const Dev& d, int b) {
  return d.direct ? d.bin_off[b + 1] - d.bin_off[b] : d.sel[b].v;
}
__device__ __forceinline__ int chunks_listed(const Dev& d) { return d.direct ? d.nchunks : d.sel[SEL_CHUNKS].v; }
// (direct lists hold rows of every LP) the row's LP is still presolving; for
// kernels beside which none stops an LP
__device__ __forceinline__ bool row_lp_on(const Dev& d, int i) {
  return !d.direct || d.K == 1 || d.lp_ok[d.row_lp[i]] != 0;
}
// ... was presolving when the round began: for the sweep, whose workgroups stop
// LPs while others still read their rows. All rows of an LP take part in the
// round that stops it, as where the LP is alone.
__device__ __forceinline__ bool row_lp_swept(const Dev& d, int i) {
  return !d.direct || d.K == 1 || d.lp_run[d.row_lp[i]] != 0;
}

// A value the compiler has to have loaded here: loads written before it are
// in flight together instead of each behind the branch that first needs it.
template <class T>
__device__ __forceinline__ void hold(T x) {
  asm volatile("" : : "v"(x));
}
// The kernel's first argument, its Dev, read again where it is used: for code
// that few wavefronts reach. Its pointers otherwise stay in scalar registers
// from the kernel's start, and when those run out every use anywhere pays for
// the reload from a vector lane.
__device__ __forceinline__ const Dev& cold_dev() {
  unsigned long long a = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return *(const Dev*)(const __attribute__((address_space(4))) Dev*)a;
}
// an LP that stops leaves the next selection at once
__device__ __forceinline__ void flag_infeasible(const Dev& d, int lp) {
  atomicOr(&d.flags->infeasible, 1);
  if (d.K > 1) {
    atomicOr(&d.lpf[lp].infeasible, 1);
    d.lp_ok[lp] = 0;
  }
}
__device__ __forceinline__ void flag_unbounded(const Dev& d, int lp) {
  atomicOr(&d.flags->unbounded, 1);
  if (d.K > 1) {
    atomicOr(&d.lpf[lp].unbounded, 1);
    d.lp_ok[lp] = 0;
  }
}

// ---------------------------------------------------------------------------
// scalar helpers (IEEE double; the library is built with -ffp-contract=off)
// ---------------------------------------------------------------------------

__device__ __forceinline__ double pos0(double x) { return x == 0.0 ? 0.0 : x; }
__device__ __forceinline__ double mx1(double x) {
  double a = fabs(x);
  return a > 1.0 ? a : 1.0;
}
__device__ __forceinline__ bool is_inf(double x) { return __builtin_isinf(x); }

// the locks one row puts on a column with coefficient a (down in the low
// word, up in the high word): a > 0 with a finite lhs (a < 0: rhs) keeps the
// column from decreasing, a > 0 with a finite rhs (a < 0: lhs) from increasing
__device__ __forceinline__ unsigned long long lock_bits(double a, double lhs, double rhs) {
  unsigned long long lf = is_inf(lhs) ? 0ull : 1ull, rf = is_inf(rhs) ? 0ull : 1ull;
  return a > 0 ? (lf | (rf << 32)) : (rf | (lf << 32));
}

// a row removal takes column j (coefficient a, the row's sides lhs / rhs) out
// of that row; a column left in no row is decided this round, and with dual
// fixing so is every column that lost a row (it may have lost its last lock);
// a column left in one row is checked for a free singleton
__device__ __forceinline__ void drop_col(const Dev& d, int j, double a, double lhs, double rhs) {
  int left = atomicSub(&d.col_len[j], 1) - 1;
  if (d.cfg.dual_fix) {
    atomicAdd(&d.locks[j], 0ull - lock_bits(a, lhs, rhs));  // the counts never go below 0
    d.touch[j] = 1;
  } else if (left == 0) {
    d.touch[j] = 1;
  }
  if (d.cfg.free_sing && left == 1) d.fs_flag[j] = 1;  // now in one row: a candidate
}

// A row whose every finite side has at least two infinite contributions on
// the side's residual, and that cannot be redundant, gives no candidate, no
// removal and no infeasibility: sweeping it changes nothing.
__device__ __forceinline__ bool row_inert(int2 c, double lhs, double rhs) {
  bool lo_inf = is_inf(lhs), up_inf = is_inf(rhs);
  bool prop = (!up_inf && c.x <= 1) || (!lo_inf && c.y <= 1);
  bool redundant_possible = (lo_inf || c.x == 0) && (up_inf || c.y == 0);
  return !prop && !redundant_possible;
}

__device__ __forceinline__ double tol_of(const Cfg& c, double x) { return c.feas_tol * mx1(x); }

// order-preserving map double <-> int64 (an involution); -0 never occurs
__device__ __forceinline__ long long dkey(double x) {
  long long b = __double_as_longlong(x);
  return b >= 0 ? b : (b ^ 0x7FFFFFFFFFFFFFFFLL);
}
__device__ __forceinline__ double dunkey(long long k) {
  return __longlong_as_double(k >= 0 ? k : (k ^ 0x7FFFFFFFFFFFFFFFLL));
}

// the order reversed: an upper bound's key grows as the bound falls, so both
// sides' accumulators take the largest key
__device__ __forceinline__ long long ukey(double x) { return ~dkey(x); }
__device__ __forceinline__ double unukey(long long k) { return dunkey(~k); }

// contribution of coefficient a on [lb, ub] to the min / max activity
__device__ __forceinline__ void contrib(double a, double lb, double ub, double& tmin,
                                       bool& imin, double& tmax, bool& imax) {
  double bmin = a > 0 ? lb : ub;
  double bmax = a > 0 ? ub : lb;
  imin = is_inf(bmin);
  imax = is_inf(bmax);
  tmin = imin ? 0.0 : pos0(a * bmin);
  tmax = imax ? 0.0 : pos0(a * bmax);
}

// ---------------------------------------------------------------------------
// wave helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return threadIdx.x & (PSL_WAVE - 1); }

__device__ __forceinline__ unsigned long long lanemask_lt() {
  int l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// One step of a butterfly whose lanes hold equal values over aligned groups of
// S lanes: each lane's value of the neighbouring group. Within 16 lanes a
// data-parallel move of the vector unit (a mirror reaches the other half as
// well as an exchange does, its lanes being equal); across 16 and 32 lanes the
// swaps of rows, whose two results are this and the other group's value in an
// order that a commutative sum does not see. No LDS access: a shuffle is one,
// of about 60 cycles, for each 32 bits and step.
template <int S>
__device__ __forceinline__ void lane_pair(unsigned x, unsigned& a, unsigned& b) {
  if constexpr (S <= 8) {
    constexpr int ctrl = S == 1 ? 0xB1 : S == 2 ? 0x4E : S == 4 ? 0x141 : 0x140;
    a = x;
    b = (unsigned)__builtin_amdgcn_mov_dpp((int)x, ctrl, 0xF, 0xF, true);
  } else if constexpr (S == 16) {
    auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    a = r[0];
    b = r[1];
  } else {
    auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    a = r[0];
    b = r[1];
  }
}

template <int S>
__device__ __forceinline__ void lane_pair64(unsigned long long x, unsigned long long& a, unsigned long long& b) {
  unsigned al, ah, bl, bh;
  lane_pair<S>((unsigned)x, al, bl);
  lane_pair<S>((unsigned)(x >> 32), ah, bh);
  a = ((unsigned long long)ah << 32) | al;
  b = ((unsigned long long)bh << 32) | bl;
}

// Sum over aligned groups of G lanes by a butterfly. fl(a + b) is
// commutative, so both partners compute the same node and after log2(G)
// steps every lane of the group holds the pairwise tree over its G lanes.
template <int G, int S = 1>
__device__ __forceinline__ double group_sum(double x) {
  if constexpr (S < G) {
    unsigned long long a, b;
    lane_pair64<S>((unsigned long long)__double_as_longlong(x), a, b);
    return group_sum<G, 2 * S>(__longlong_as_double((long long)a) + __longlong_as_double((long long)b));
  } else {
    return x;
  }
}

template <int G, int S = 1>
__device__ __forceinline__ unsigned long long group_sum_u64(unsigned long long x) {
  if constexpr (S < G) {
    unsigned long long a, b;
    lane_pair64<S>(x, a, b);
    return group_sum_u64<G, 2 * S>(a + b);
  } else {
    return x;
  }
}

template <int G, int S = 1>
__device__ __forceinline__ int group_sum_int(int x) {
  if constexpr (S < G) {
    unsigned a, b;
    lane_pair<S>((unsigned)x, a, b);
    return group_sum_int<G, 2 * S>((int)(a + b));
  } else {
    return x;
  }
}

template <int G>
__device__ __forceinline__ unsigned long long group_mask() {
  if constexpr (G == 64) return ~0ull;
  else return ((1ull << G) - 1) << (lane_id() & ~(G - 1));
}

// Pairwise tree over v[0..n) padded with +0 to the next power of two,
// in place (used for pass and chunk sums held in LDS).
__device__ __forceinline__ double tree_inplace(double* v, int n) {
  if (n <= 0) return 0.0;
  int p = 1;
  while (p < n) p <<= 1;
  for (int w = 1; w < p; w <<= 1)
    for (int i = 0; i + w < n; i += 2 * w) v[i] = v[i] + v[i + w];
  return v[0];
}

// candidate-region sizes (entries) of the sweep bins, per workgroup
// Row blocks (of 256 threads' rows) one workgroup of a bin sweeps in turn:
// short rows give a wavefront little work, so their workgroups take several.
// With the direct lists (one: an LP of at most 5e5 nonzeros) the chip has more
// room than there are row blocks and a workgroup takes one: the chains of four
// blocks one after another were the launch's time (2000 rows: 16.5 us a sweep,
// 8.0 with one block; a presolve 1.64 and 1.28 ms). Selected lists keep four:
// with one block a wavefront has fewer gathers in flight (1e7 rows: 77 ms with
// four, 90 with one; a 4096-LP batch 77 and 88 ms).
__host__ __device__ __forceinline__ int bin_rep(int bin, int one) {
  return one ? 1 : bin <= BIN_G16 ? 4 : bin == BIN_W1 ? 2 : 1;
}

// rows of a row block of the bin
__host__ __device__ __forceinline__ int bin_rows(int bin) {
  return bin == BIN_G4 ? 64 : bin == BIN_G8 ? 32 : bin == BIN_G16 ? 16 : 4;
}

__host__ __device__ __forceinline__ int64_t cand_region(int bin, int one) {
  // 2 candidates x (rows per workgroup x longest row of the bin)
  int len = bin == BIN_G4 ? 4 : bin == BIN_G8 ? 8 : bin == BIN_G16 ? 16 : bin == BIN_W1 ? 64 : bin == BIN_W4 ? 256 : 512;
  return 2 * (int64_t)bin_rep(bin, one) * bin_rows(bin) * len;
}

// SplitMix64 output function for state x (Steele, Lea & Flood 2014).
__device__ __forceinline__ unsigned long long splitmix(unsigned long long x) {
  unsigned long long z = x + 0x9E3779B97F4A7C15ULL;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// sign, exponent and top 32 mantissa bits, rounded to nearest
__device__ __forceinline__ unsigned long long quantize(double v) {
  unsigned long long b = (unsigned long long)__double_as_longlong(v);
  unsigned long long sign = b >> 63;
  unsigned long long mag = b & 0x7FFFFFFFFFFFFFFFULL;
  return ((mag + (1ULL << 19)) >> 20) | (sign << 63);
}

// exclusive scan of one int per thread across a block of NT threads
template <int NT>
__device__ __forceinline__ int block_excl_scan_n(int v, int* total) {
  __shared__ int wsum[NT / PSL_WAVE];
  int lane = lane_id(), w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < PSL_WAVE; o <<= 1) {
    int y = __shfl_up(x, o, PSL_WAVE);
    if (lane >= o) x += y;
  }
  if (lane == PSL_WAVE - 1) wsum[w] = x;
  __syncthreads();
  int pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < NT / PSL_WAVE; ++k) {
    int s = wsum[k];
    if (k < w) pre += s;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + x - v;
}

// the same across the 256-thread block
__device__ __forceinline__ int block_excl_scan(int v, int* total) { return block_excl_scan_n<PSL_BLOCK>(v, total); }


}  // namespace psl
