// ingest.hip -- validation, canonicalisation, the transposed copy of A, row
// binning and the input fixings ("round 0").
//
// The paper keeps A together with its transpose (section 3.2, "Internal data
// structures"). The transpose is built here by a stable radix sort of the CSR
// positions by column, so the rows of every column come out ascending.
#include <algorithm>

#include "psl_kern.h"
#include "sweep.h"

namespace psl {

enum : int32_t {
  ERR_ROWPTR = 1, ERR_COLIDX = 2, ERR_COEF = 4, ERR_SIDE = 8, ERR_BOUND = 16, ERR_COST = 32
};

__device__ __forceinline__ void report(const Dev& d, int32_t bit, int64_t pos) {
  atomicOr(&d.flags->error, bit);
  atomicMin((long long*)&d.flags->error_pos, (long long)pos);
}

__device__ __forceinline__ double canon_inf(double v, double inf_value) {
  if (v >= inf_value) return __builtin_huge_val();
  if (v <= -inf_value) return -__builtin_huge_val();
  return pos0(v);
}

// the arrays of an LP in device memory, one row of workgroups each
__global__ void __launch_bounds__(PSL_BLOCK) k_copy_in(CopyIn c) {
  const InSeg g = c.seg[blockIdx.y];
  const int64_t t = (int64_t)blockIdx.x * PSL_BLOCK + threadIdx.x, step = (int64_t)gridDim.x * PSL_BLOCK;
  int64_t done = 0;
  if ((((uintptr_t)g.src | (uintptr_t)g.dst) & 15) == 0) {
    done = g.words / 4;
    const uint4* src = reinterpret_cast<const uint4*>(g.src);
    uint4* dst = reinterpret_cast<uint4*>(g.dst);
    for (int64_t i = t; i < done; i += step) dst[i] = src[i];
    done *= 4;
  }
  for (int64_t i = done + t; i < g.words; i += step) g.dst[i] = g.src[i];
}

void launch_copy_in(const CopyIn& c, hipStream_t s) {
  int64_t w = 0;
  for (const InSeg& g : c.seg) w = g.words > w ? g.words : w;
  int64_t blocks = (w + 4 * PSL_BLOCK - 1) / (4 * PSL_BLOCK);
  if (blocks == 0) return;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(k_copy_in, dim3((unsigned)blocks, IN_SEGS), dim3(PSL_BLOCK), 0, s, c);
}

// bin of a row of len entries
__device__ __forceinline__ int bin_of_len(int len, int t_long, int t_g8) {
  return len <= 4 ? BIN_G4 : len <= t_g8 ? BIN_G8 : len <= 16 ? BIN_G16 : len > t_long ? BIN_LONG
       : len <= 64 ? BIN_W1 : len <= 256 ? BIN_W4 : BIN_W8;
}

// Rows and columns, in tiles of 1024 of each: the checks, the stored sides and
// bounds, and each tile's rows per bin (hist[bin * tiles + tile], from whose
// scan k_bin_fill lists them). The launches of the ingest are queued without a
// look at the errors found, so each of them stays inside its arrays whatever
// the input holds.
#define ING_TILE 1024
__global__ void __launch_bounds__(PSL_BLOCK) k_check(Dev d, const double* lb_in, const double* ub_in, double* c_mut,
                                                     int32_t t_long, int32_t t_g8, int32_t* hist, int tiles) {
  __shared__ int c[NBINS];
  if (threadIdx.x < NBINS) c[threadIdx.x] = 0;
  __syncthreads();
  const double iv = d.cfg.inf_value;
  const int64_t base = (int64_t)blockIdx.x * ING_TILE + threadIdx.x;
#pragma unroll
  for (int k = 0; k < ING_TILE / PSL_BLOCK; ++k) {
    const int64_t i = base + k * PSL_BLOCK;
    int bin = -1;
    if (i < d.m) {
      int32_t a = d.rp[i], b = d.rp[i + 1];
      if ((i == 0 && a != 0) || a < 0 || b < a || (int64_t)b > d.nnz || (i == d.m - 1 && (int64_t)b != d.nnz))
        report(d, ERR_ROWPTR, i);
      double l = d.lhs[i], r = d.rhs[i];
      if (__builtin_isnan(l) || __builtin_isnan(r) || l >= iv || r <= -iv) report(d, ERR_SIDE, i);
      d.lhs[i] = canon_inf(l, iv);
      d.rhs[i] = canon_inf(r, iv);
      bin = bin_of_len(b - a, t_long, t_g8);
    }
#pragma unroll
    for (int q = 0; q < NBINS; ++q) {
      int cnt = __popcll(__ballot(bin == q));
      if (lane_id() == 0 && cnt) atomicAdd(&c[q], cnt);
    }
    if (i < d.n) {
      double l = lb_in[i], u = ub_in[i], cost = c_mut[i];
      if (__builtin_isnan(l) || __builtin_isnan(u) || l >= iv || u <= -iv) report(d, ERR_BOUND, i);
      if (!__builtin_isfinite(cost)) report(d, ERR_COST, i);
      d.bnd[i] = make_double2(canon_inf(l, iv), canon_inf(u, iv));
      c_mut[i] = pos0(cost);
    }
  }
  __syncthreads();
  if (threadIdx.x < NBINS && (int)blockIdx.x < tiles) hist[threadIdx.x * tiles + blockIdx.x] = c[threadIdx.x];
}

// the bins' lists, rows ascending in each, and the bins' sizes
__global__ void __launch_bounds__(PSL_BLOCK) k_bin_fill(Dev d, int32_t t_long, int32_t t_g8, const int32_t* off,
                                                        int tiles, BinEnt* bins) {
  __shared__ int at[NBINS], wcnt[PSL_BLOCK / PSL_WAVE][NBINS];
  const int w = threadIdx.x >> 6;
  if (threadIdx.x < NBINS) {
    const int q = threadIdx.x;
    at[q] = off[q * tiles + blockIdx.x];
    if (blockIdx.x == 0) d.flags->bins[q] = (q + 1 < NBINS ? off[(q + 1) * tiles] : d.m) - off[q * tiles];
  }
  for (int k = 0; k < ING_TILE / PSL_BLOCK; ++k) {
    const int64_t i = (int64_t)blockIdx.x * ING_TILE + k * PSL_BLOCK + threadIdx.x;
    int a = 0, len = 0, bin = -1, below = 0;
    if (i < d.m) {
      a = d.rp[i];
      len = d.rp[i + 1] - a;
      bin = bin_of_len(len, t_long, t_g8);
    }
#pragma unroll
    for (int q = 0; q < NBINS; ++q) {
      unsigned long long m = __ballot(bin == q);
      if (bin == q) below = __popcll(m & lanemask_lt());
      if (lane_id() == 0) wcnt[w][q] = __popcll(m);
    }
    __syncthreads();
    if (bin >= 0) {
      int p = at[bin] + below;
      for (int v = 0; v < w; ++v) p += wcnt[v][bin];
      bins[p] = BinEnt{(int32_t)i, a, len, 0};
    }
    __syncthreads();
    if (threadIdx.x < NBINS)
      for (int v = 0; v < PSL_BLOCK / PSL_WAVE; ++v) at[threadIdx.x] += wcnt[v][threadIdx.x];
    __syncthreads();
  }
}

// last row i < m with rp[i] <= p, given rp[0] <= p < rp[m] (rp ascends), by the
// wavefront: 64 probes a step
__device__ __forceinline__ int row_of_pos(const int32_t* rp, int m, int p) {
  int lo = 0, hi = m;
  while (hi - lo > 1) {
    const int step = (hi - lo + PSL_WAVE - 1) / PSL_WAVE;
    const int64_t at = (int64_t)lo + (int64_t)(lane_id() + 1) * step;
    const int c = __popcll(__ballot(at < hi && rp[at < hi ? at : lo] <= p));
    lo += c * step;
    hi = hi - lo > step ? lo + step : hi;
  }
  return lo;
}

// Per tile of 2048 positions: the rows of the positions (rowid1), the checks of
// the entries, and the counts of the first transposition pass (digits of the
// column under mask; 0: none). The tile's first and last rows are searched, the
// rows' starts between them marked in LDS and carried over their positions by a
// running maximum. Also sets cp to -1 for the transposition.
// One launch where a fill, a count per row, a scan, the checks and the pass's
// counts were up to seven (1e7 rows, 9.7e7 entries: 1.16 ms together, 0.65 now,
// of it 0.25 for the 1.5 GB it reads and writes).
#define POS_TILE RX_TILE
#define POS_ITEMS (POS_TILE / PSL_BLOCK)
__global__ void __launch_bounds__(PSL_BLOCK) k_positions(Dev d, int32_t* rowid1, int32_t* cp, uint32_t mask,
                                                         int32_t* hist, int tiles) {
  __shared__ int mk[POS_TILE];
  __shared__ int digit[256];
  __shared__ int ends[2], wmax[PSL_BLOCK / PSL_WAVE];
  const int t = threadIdx.x, w = t >> 6;
  for (int64_t j = (int64_t)blockIdx.x * PSL_BLOCK + t; j <= d.n; j += (int64_t)gridDim.x * PSL_BLOCK) cp[j] = -1;
  if (blockIdx.x == 0 && t == 0) rowid1[0] = 0;
  const int64_t p0 = (int64_t)blockIdx.x * POS_TILE;
  if (p0 >= d.nnz) return;
  const int cnt = (int)(d.nnz - p0 < POS_TILE ? d.nnz - p0 : POS_TILE);
  // rows can be searched when their pointers passed the check
  const bool rows_ok = d.m > 0 && !(d.flags->error & ERR_ROWPTR);
  const bool check = !(d.flags->error & (ERR_ROWPTR | ERR_SIDE | ERR_BOUND | ERR_COST));
  digit[t] = 0;
#pragma unroll
  for (int k = 0; k < POS_ITEMS; ++k) mk[k * PSL_BLOCK + t] = 0;
  if (w < 2 && rows_ok) {
    const int r = row_of_pos(d.rp, d.m, (int)(w == 0 ? p0 : p0 + cnt - 1));
    if (lane_id() == 0) ends[w] = r;
  }
  __syncthreads();
  const int r0 = rows_ok ? ends[0] : 0, r1 = rows_ok ? ends[1] : 0;
  const bool whole = rows_ok && (int64_t)d.rp[r0] == p0;  // the tile starts with a row
  // (a tile between which many empty rows lie is searched position by position)
  const bool walk = r1 - r0 <= 16 * POS_TILE;
  if (walk) {
    for (int r = r0 + 1 + t; r <= r1; r += PSL_BLOCK) {
      const int s = d.rp[r];
      if (d.rp[r + 1] > s) mk[s - p0] = r;
    }
    if (t == 0) mk[0] = r0;
    __syncthreads();
    int v[POS_ITEMS], run = 0;
#pragma unroll
    for (int k = 0; k < POS_ITEMS; ++k) {
      const int x = mk[t * POS_ITEMS + k];
      run = x > run ? x : run;
      v[k] = run;
    }
    int pre = run;
#pragma unroll
    for (int o = 1; o < PSL_WAVE; o <<= 1) {
      const int x = __shfl_up(pre, o, PSL_WAVE);
      if (lane_id() >= o && x > pre) pre = x;
    }
    if (lane_id() == PSL_WAVE - 1) wmax[w] = pre;
    __syncthreads();
    pre = __shfl_up(pre, 1, PSL_WAVE);
    if (lane_id() == 0) pre = 0;
    for (int q = 0; q < w; ++q) pre = wmax[q] > pre ? wmax[q] : pre;
#pragma unroll
    for (int k = 0; k < POS_ITEMS; ++k) mk[t * POS_ITEMS + k] = v[k] > pre ? v[k] : pre;
  } else {
    for (int k = t; k < cnt; k += PSL_BLOCK) {
      int lo = r0, hi = r1 + 1;
      while (hi - lo > 1) {
        const int mid = lo + (hi - lo) / 2;
        if ((int64_t)d.rp[mid] <= p0 + k) lo = mid;
        else hi = mid;
      }
      mk[k] = lo;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < POS_ITEMS; ++k) {
    const int q = k * PSL_BLOCK + t;
    if (q >= cnt) continue;
    const int64_t p = p0 + q;
    const int row = mk[q], j = d.ci[p];
    rowid1[p + 1] = row;
    if (mask) atomicAdd(&digit[(uint32_t)j & mask], 1);
    if (check) {
      const bool first = q == 0 ? whole : mk[q - 1] != row;
      if (j < 0 || j >= d.n || (!first && d.ci[p - 1] >= j)) report(d, ERR_COLIDX, p);
      const double a = d.va[p];
      if (!__builtin_isfinite(a) || a == 0.0) report(d, ERR_COEF, p);
    }
  }
  __syncthreads();
  if (mask && (uint32_t)t <= mask) hist[(int64_t)t * tiles + blockIdx.x] = digit[t];
}

// column bits and passes of the transposition
static int csc_bits(const Dev& d) {
  int bits = 0;
  while (bits < 31 && ((int64_t)1 << bits) < (int64_t)d.n) ++bits;
  return bits;
}

void launch_checks(const Dev& d, const double* lb_in, const double* ub_in, double* c_mut, const int32_t* thresholds,
                   BinEnt* bins, IngestScratch& sc, hipStream_t s) {
  const int64_t t = d.m > d.n ? d.m : d.n;
  const int tiles = (int)(((int64_t)d.m + ING_TILE - 1) / ING_TILE);
  if (t > 0)
    hipLaunchKernelGGL(k_check, dim3((unsigned)((t + ING_TILE - 1) / ING_TILE)), dim3(PSL_BLOCK), 0, s, d, lb_in,
                       ub_in, c_mut, thresholds[0], thresholds[2], sc.ws, tiles);
  if (tiles > 0) {
    scan_excl(sc.ws, sc.ws, (int64_t)NBINS * tiles, nullptr, sc.ws + (int64_t)NBINS * tiles, s);
    hipLaunchKernelGGL(k_bin_fill, dim3(tiles), dim3(PSL_BLOCK), 0, s, d, thresholds[0], thresholds[2],
                       (const int32_t*)sc.ws, tiles, bins);
  }
  // the first pass's digits, as build_csc splits them
  const int bits = csc_bits(d), passes = (bits + 7) / 8, per = passes ? (bits + passes - 1) / passes : 0;
  const int64_t pt = (d.nnz + POS_TILE - 1) / POS_TILE;
  // and enough workgroups for cp where the columns are many and the positions few
  // (1.5e7 columns, 2000 entries: 2.13 ms an ingest with the one of the positions)
  const int64_t ct = std::min<int64_t>(((int64_t)d.n + POS_TILE) / POS_TILE, 2048);
  hipLaunchKernelGGL(k_positions, dim3((unsigned)std::max(pt, ct)), dim3(PSL_BLOCK), 0, s, d, sc.rowid1,
                     (int32_t*)d.cp, passes ? (1u << per) - 1u : 0u, sc.ws, (int)pt);
}

// ---------------------------------------------------------------------------
// transposed copy
// ---------------------------------------------------------------------------
__global__ void k_csc_gather(Dev d, const int32_t* perm, const int32_t* rowid1, int32_t* ri, double* cva) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < d.nnz; q += (int64_t)gridDim.x * blockDim.x) {
    int p = perm ? perm[q] : (int)q;
    ri[q] = rowid1[p + 1];
    cva[q] = d.va[p];
  }
}

// cp from the column-sorted keys: position q starts every column in
// (keys[q-1], keys[q]] (keys[-1] = -1, keys[nnz] = n), so empty columns get
// the next column's start. A thread writes at most the last COLPTR_RUN
// entries of its run (always cp[keys[q]], the start of a nonempty column, and
// cp[n]); longer runs of empty columns, e.g. a block of columns that appear in
// no row, are left at -1 (cp is filled with -1 before) and resolved per column
// in k_col_len, so no thread loops over a long run.
#define COLPTR_RUN 64
__global__ void k_col_ptr(Dev d, const uint32_t* keys, int32_t* cp) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *d.n_dense = 0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q <= d.nnz; q += (int64_t)gridDim.x * blockDim.x) {
    int64_t prev = q > 0 ? (int64_t)keys[q - 1] : -1;
    int64_t cur = q < d.nnz ? (int64_t)keys[q] : (int64_t)d.n;
    // valid keys are < n; clamped, so that no store leaves cp for others
    prev = prev < (int64_t)d.n ? prev : (int64_t)d.n;
    cur = cur < (int64_t)d.n ? cur : (int64_t)d.n;
    int64_t j0 = cur - prev > COLPTR_RUN ? cur - COLPTR_RUN : prev;
    for (int64_t j = j0 + 1; j <= cur; ++j) cp[j] = (int32_t)q;
  }
}

// first position whose key is >= j (keys ascend): the start of column j
__device__ __forceinline__ int32_t col_start(const uint32_t* keys, int64_t nnz, int64_t j) {
  int64_t lo = 0, hi = nnz;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    if ((int64_t)keys[mid] < j) lo = mid + 1;
    else hi = mid;
  }
  return (int32_t)lo;
}

// column lengths; entries of cp a long run left at -1 get the start of the
// next nonempty column by a search over the keys (cp[n] is always written)
__global__ void k_col_len(Dev d, const uint32_t* keys, int32_t* cp, int32_t* col_len) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d.n) return;
  int32_t a = cp[j], b = cp[j + 1];
  if (a < 0) {
    a = col_start(keys, d.nnz, j);
    cp[j] = a;
  }
  if (b < 0) b = col_start(keys, d.nnz, j + 1);  // written by thread j + 1
  col_len[j] = b - a;
  // the columns of more than MARK_DENSE entries (order irrelevant; of a valid
  // input they fit the list)
  if (b - a > MARK_DENSE && !d.flags->error) d.dense_cols[atomicAdd(d.n_dense, 1)] = (int32_t)j;
}

// Stable transpose by LSD radix passes over the column index (at most 8 bits
// a pass, the bits split evenly), moving row and value with each key; the
// last pass writes the transposed copy itself. vtmp: nnz doubles of scratch.
// counted: k_positions left the first pass's counts in the workspace and cp
// at -1.
// Returns the column of every position of the transposed copy (the sorted
// keys), which compaction uses.
const uint32_t* build_csc(const Dev& d, int32_t* cp, int32_t* ri, double* cva, int32_t* col_len, IngestScratch& sc,
                          double* vtmp, bool counted, hipStream_t s) {
  int bits = csc_bits(d);
  int passes = (bits + 7) / 8;
  const uint32_t* kin = (const uint32_t*)d.ci;
  if (passes == 0) {
    // at most one column: the transposed copy is the CSR order
    if (d.nnz > 0) {
      int64_t blocks = (d.nnz + PSL_BLOCK - 1) / PSL_BLOCK;
      if (blocks > 16384) blocks = 16384;
      hipLaunchKernelGGL(k_csc_gather, dim3((unsigned)blocks), dim3(PSL_BLOCK), 0, s, d, (const int32_t*)nullptr,
                         sc.rowid1, ri, cva);
    }
  } else {
    int per = (bits + passes - 1) / passes;
    const int32_t* rin = nullptr;
    const double* vin = d.va;
    uint32_t* kb[2] = {sc.k0, sc.k1};
    int32_t* rb[2] = {sc.v0, sc.v1};
    for (int pass = 0, shift = 0; pass < passes; ++pass, shift += per) {
      int b = bits - shift < per ? bits - shift : per;
      bool last = pass == passes - 1;
      // the values end in cva after an odd number of hops from it
      double* vout = ((passes - 1 - pass) % 2 == 0) ? cva : vtmp;
      int32_t* rout = last ? ri : rb[pass & 1];
      uint32_t* kout = kb[pass & 1];
      radix_pass_payload(kin, rin, sc.rowid1, vin, kout, rout, vout, d.nnz, shift, b, counted && pass == 0,
                         sc.ws, s);
      kin = kout;
      rin = rout;
      vin = vout;
    }
  }
  if (!counted) fill_i32(cp, -1, d.n + 1, s);
  {
    int64_t blocks = (d.nnz + 1 + PSL_BLOCK - 1) / PSL_BLOCK;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_col_ptr, dim3((unsigned)blocks), dim3(PSL_BLOCK), 0, s, d, kin, cp);
  }
  if (d.n > 0)
    hipLaunchKernelGGL(k_col_len, dim3((d.n + PSL_BLOCK - 1) / PSL_BLOCK), dim3(PSL_BLOCK), 0, s, d, kin, cp,
                       col_len);
  return kin;
}

// ---------------------------------------------------------------------------
// the chunk table of long rows
// ---------------------------------------------------------------------------
// passes per chunk: the requested size, doubled until the row has at most
// LONG_MAX_CHUNKS chunks (chunk sizes stay powers of two times PASS_LEN)
__global__ void k_long_count(Dev d, int npass0, int32_t* cnt, int32_t* cnt2) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.nlong) return;
  BinEnt be = d.bins[d.bin_off[BIN_LONG] + k];
  int row = be.row;
  int64_t len = be.len;
  int64_t np = npass0;
  while ((len + np * PASS_LEN - 1) / (np * PASS_LEN) > LONG_MAX_CHUNKS) np *= 2;
  if (np > LONG_MAX_PASSES) {
    atomicOr(&d.flags->error, 64);  // row too long for the chunk table
    np = LONG_MAX_PASSES;
  }
  int nch = (int)((len + np * PASS_LEN - 1) / (np * PASS_LEN));
  d.lrow[k] = LongRow{row, 0, nch, (int32_t)np};
  cnt[k] = nch;
  cnt2[k] = 2 * (int)len;  // candidate entries of the row's chunks
}

__global__ void k_long_fill(Dev d, const int32_t* off, const int32_t* uoff, LongChunk* chunks) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.nlong) return;
  LongRow lr = d.lrow[k];
  lr.chunk0 = off[k];
  d.lrow[k] = lr;
  for (int c = 0; c < lr.nchunk; ++c)
    chunks[lr.chunk0 + c] = LongChunk{lr.row, c * lr.npass * PASS_LEN, k, lr.npass,
                                      uoff[k] + 2 * c * lr.npass * PASS_LEN, lr.chunk0 + c};
}

void build_long_chunks(const Dev& d, int npass0, LongChunk* chunks, int32_t* cnt, int32_t* cnt2, int32_t* totals,
                       int32_t* ws, hipStream_t s) {
  unsigned blocks = (unsigned)((d.nlong + PSL_BLOCK - 1) / PSL_BLOCK);
  hipLaunchKernelGGL(k_long_count, dim3(blocks), dim3(PSL_BLOCK), 0, s, d, npass0, cnt, cnt2);
  scan_excl(cnt, cnt, d.nlong, totals, ws, s);
  scan_excl(cnt2, cnt2, d.nlong, totals + 1, ws, s);
  hipLaunchKernelGGL(k_long_fill, dim3(blocks), dim3(PSL_BLOCK), 0, s, d, (const int32_t*)cnt, (const int32_t*)cnt2,
                     chunks);
}

// ---------------------------------------------------------------------------
// row selection: the rows a round sweeps, as bin lists and long-row chunks
// ---------------------------------------------------------------------------
// One pass over the rows in tiles, four a thread (striped, so the loads
// coalesce). A row is kept when it is active, its LP still presolving and, by
// the mode, marked / not inert; the row data of a row is read only when its
// cheap tests pass, so a selection of few marked rows reads about a byte per
// row. A tile's kept rows are counted per bin by ballots and take their place
// in the bins' lists with one atomic add per bin: a tile's rows stay together
// and in row order, whose place in the list is of no consequence (candidates
// fold by maximum and minimum, their sources by the lowest position). A tile
// is 1024 rows, 4096 from SEL_BIG rows on: the adds to one count take 10 ns each
// (1e6 rows: 24 us a selection with 977 tiles, 15 with 245).
#define SEL_ITEMS 4
#define SEL_BIG (1 << 18)

struct SelArgs {
  int mode;             // -1: the device's (bit 0: marked rows only; bit 1: inert rows skipped)
  int t_long, t_g8;     // bin thresholds of the ingest
  int seq;              // launch number of the round before
};

// index of long row `row` in d.lrow (ascending rows; the row is long)
__device__ __forceinline__ int long_row_index(const Dev& d, int row) {
  int lo = 0, hi = d.nlong - 1;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (d.lrow[mid].row < row) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

template <int BS>
__global__ void __launch_bounds__(BS) k_select(Dev d, SelArgs a, BinEnt* out, LongChunk* cout, SelCnt* cnt) {
  constexpr int W = BS / PSL_WAVE;
  constexpr int MARKS = BS * SEL_ITEMS / 1024;  // tiles of the marks in one of ours
  __shared__ int wc[SEL_ITEMS][NBINS][W];       // per item row and bin: each wavefront's rows
  __shared__ int at[NBINS];
  __shared__ int wz[W];
  const int tile = blockIdx.x;
  const bool next = a.mode < 0;
  const int w = threadIdx.x >> 6;
  const int64_t t0 = (int64_t)tile * BS * SEL_ITEMS + threadIdx.x;
  const uint8_t mark = round_mark(a.seq + 1);
  // the tile's marks
  bool marked = false;
#pragma unroll
  for (int k = 0; k < MARKS; ++k) {
    int64_t x = (int64_t)tile * MARKS + k;
    if (x <= d.m / 1024) marked = marked || d.dirty_tile[x] == mark;
  }
  const int mode = next ? d.flags->mode : a.mode;
  if ((next && round_over(d, a.seq)) || ((mode & 1) && !marked)) return;
  // level by level for all items, without branches around the loads (a row
  // that fails the cheap tests reads row 0's data, which is cached)
  bool keep[SEL_ITEMS];
#pragma unroll
  for (int k = 0; k < SEL_ITEMS; ++k) {
    int64_t i = t0 + k * BS, ii = i < d.m ? i : 0;
    uint8_t on = d.row_on[ii], dt = d.dirty[ii];
    keep[k] = i < d.m && on != 0 && (!(mode & 1) || dt == mark);
  }
  int r0[SEL_ITEMS], len[SEL_ITEMS], lpi[SEL_ITEMS];
  int2 rf[SEL_ITEMS];
  double lh[SEL_ITEMS], rh[SEL_ITEMS];
#pragma unroll
  for (int k = 0; k < SEL_ITEMS; ++k) {
    int64_t jj = keep[k] ? t0 + k * BS : 0;
    r0[k] = d.rp[jj];
    len[k] = d.rp[jj + 1] - r0[k];
    lpi[k] = d.K > 1 ? d.row_lp[jj] : 0;
    if (mode & 2) {
      rf[k] = d.rinf[jj];
      lh[k] = d.lhs[jj];
      rh[k] = d.rhs[jj];
    }
  }
  int bin[SEL_ITEMS], pre[SEL_ITEMS];
  int z = 0;
#pragma unroll
  for (int k = 0; k < SEL_ITEMS; ++k) {
    if (d.K > 1) keep[k] = keep[k] && d.lp_ok[lpi[k]] != 0;
    if (mode & 2) keep[k] = keep[k] && !row_inert(rf[k], lh[k], rh[k]);
    bin[k] = keep[k] ? bin_of_len(len[k], a.t_long, a.t_g8) : -1;
    z += keep[k] ? len[k] : 0;
    pre[k] = 0;
#pragma unroll
    for (int b = 0; b < NBINS; ++b) {
      unsigned long long bal = __ballot(bin[k] == b);
      if (bin[k] == b) pre[k] = __popcll(bal & lanemask_lt());
      if (lane_id() == 0) wc[k][b][w] = __popcll(bal);
    }
  }
#pragma unroll
  for (int o = 1; o < PSL_WAVE; o <<= 1) z += __shfl_xor(z, o, PSL_WAVE);
  if (lane_id() == 0) wz[w] = z;
  __syncthreads();
  // one thread per bin: the exclusive prefix of every (item row, wavefront)
  // count in row order, then the tile's place in the bin's list
  if (threadIdx.x < NBINS) {
    int run = 0;
#pragma unroll
    for (int k = 0; k < SEL_ITEMS; ++k)
      for (int v = 0; v < W; ++v) {
        int x = wc[k][threadIdx.x][v];
        wc[k][threadIdx.x][v] = run;
        run += x;
      }
    at[threadIdx.x] = run ? atomicAdd(&cnt[threadIdx.x].v, run) : 0;
  } else if (threadIdx.x == PSL_WAVE) {
    int s = 0;
    for (int v = 0; v < W; ++v) s += wz[v];
    if (s) atomicAdd(&cnt[SEL_NNZ].v, s);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < SEL_ITEMS; ++k) {
    if (!keep[k]) continue;
    const int i = (int)(t0 + k * BS), b = bin[k];
    out[d.bin_off[b] + at[b] + wc[k][b][w] + pre[k]] = BinEnt{i, r0[k], len[k], 0};
    if (b == BIN_LONG) {
      LongRow lr = d.lrow[long_row_index(d, i)];
      int c0 = atomicAdd(&cnt[SEL_CHUNKS].v, lr.nchunk);
      for (int c = 0; c < lr.nchunk; ++c) cout[c0 + c] = d.chunks0[lr.chunk0 + c];
    }
  }
}

static void launch_select(const Dev& d, const SelArgs& a, BinEnt* out, LongChunk* cout, SelCnt* cnt, hipStream_t s) {
  if (d.m == 0) return;
  if (d.m >= SEL_BIG) {
    int T = (d.m + 1024 * SEL_ITEMS - 1) / (1024 * SEL_ITEMS);
    hipLaunchKernelGGL(k_select<1024>, dim3(T), dim3(1024), 0, s, d, a, out, cout, cnt);
  } else {
    int T = (d.m + PSL_BLOCK * SEL_ITEMS - 1) / (PSL_BLOCK * SEL_ITEMS);
    hipLaunchKernelGGL(k_select<PSL_BLOCK>, dim3(T), dim3(PSL_BLOCK), 0, s, d, a, out, cout, cnt);
  }
}

void select_all(const Dev& d, int t_long, int t_g8, BinEnt* out, LongChunk* cout, SelCnt* cnt, hipStream_t s) {
  fill_i32(&cnt[0].v, 0, (int64_t)SEL_N * (sizeof(SelCnt) / sizeof(int32_t)), s);
  launch_select(d, SelArgs{0, t_long, t_g8, 0}, out, cout, cnt, s);
}

void select_next(const Dev& d, int t_long, int t_g8, BinEnt* out, LongChunk* cout, SelCnt* cnt, int seq,
                 hipStream_t s) {
  launch_select(d, SelArgs{-1, t_long, t_g8, seq}, out, cout, cnt, s);
}

__global__ void k_rounds_begin(Dev d, int64_t rec_at, int64_t rec_cap) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k == 0) {
    d.flags->rec_at = rec_at;
    d.flags->rec_cap = rec_cap;
    d.flags->stop_at = 0x7FFFFFFF;
  }
  if (d.K > 1 && k < d.K) {
    d.lpf[k] = LpFlags{0, 0, 0, 0};
    d.lpo[k] = LpOut{0, 0};
    d.lp_run[k] = d.lp_ok[k];
  }
}

void launch_rounds_begin(const Dev& d, int64_t rec_at, int64_t rec_cap, hipStream_t s) {
  hipLaunchKernelGGL(k_rounds_begin, dim3((d.K + PSL_BLOCK - 1) / PSL_BLOCK), dim3(PSL_BLOCK), 0, s, d, rec_at,
                     rec_cap);
}

// ---------------------------------------------------------------------------
// state initialisation and round 0 (input fixings, crossed bounds / sides)
// ---------------------------------------------------------------------------
// (the run's start also copies the costs: it works on a copy, since
// free-singleton substitutions change it and postsolve wants the input's)
__global__ void k_init_state(Dev d, int64_t supers, const double* c_in, double* c_run) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < d.m) {
    d.row_on[t] = 1;
    d.row_code[t] = RC_KEEP;
    d.dirty[t] = 0;
    d.fs_pick[t] = 0x7FFFFFFF;
  }
  if (t <= d.m / 1024) d.dirty_tile[t] = 0;
  if (t < d.n) {
    double2 b = d.bnd[t];
    if (c_run) c_run[t] = c_in[t];
    d.touch[t] = 1;    // the first round decides every column
    d.fs_flag[t] = 1;  // and checks every column for a free singleton
    d.owner[t] = ~0ull;
    d.lsrc[t] = is_inf(b.x) ? -1 : -2;
    d.usrc[t] = is_inf(b.y) ? -1 : -2;
    d.bkey[2 * t] = dkey(b.x);
    d.bkey[2 * t + 1] = ukey(b.y);
    d.src[2 * t] = 0x7FFFFFFF;
    d.src[2 * t + 1] = 0x7FFFFFFF;
    d.col_code[t] = 0;
  }
  if (t == 0) {
    Flags f;
    f.n_dense = d.flags->n_dense;  // of the ingest
    for (int b = 0; b < NBINS; ++b) f.bins[b] = d.flags->bins[b];
    f.infeasible = f.unbounded = f.error = f.merged = 0;
    f.round_total = f.vlist_count = f.rows_removed = 0;
    f.fin_cols = f.mode = f.lead_count = f.fs_picks = f.fs_rows = f.fs_claims = 0;
    f.error_pos = 0x7FFFFFFFFFFFFFFFLL;
    f.dbl_count = f.dbl_applied = 0;
    f.stop_at = 0x7FFFFFFF;
    f.rounds_done = 0;
    f.rec_base = f.rec_at = f.rec_cap = 0;
    for (int k = 0; k < SWEPT_SLOTS; ++k) f.swept[k].rows = f.swept[k].nnz = 0;
    f.sum_rows = f.sum_nnz = f.sum_cols = 0;
    for (int k = 0; k < 3; ++k) f.stamp[k] = f.ticks[k] = 0;
    for (int k = 0; k < 2; ++k)
      for (int b = 0; b < SEL_N; ++b) f.sel[k][b].v = 0;
    *d.flags = f;
  }
  if (t < supers) {
    d.super[t] = 0;
    d.super_done[t] = 0;
  }
}

// Variable locks of every column from the alive rows (dual fixing): one bit
// per position of the transposed copy for each direction, scanned, and each
// column's count read off as the difference of the scans at its ends.
__global__ void k_lock_bits(Dev d, int32_t* dn, int32_t* up) {
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q <= d.nnz; q += stride) {
    unsigned long long b = 0;
    if (q < d.nnz) {
      int i = d.ri[q];
      if (d.row_on[i]) b = lock_bits(d.cva[q], d.lhs[i], d.rhs[i]);
    }
    dn[q] = (int32_t)(b & 1ull);
    up[q] = (int32_t)(b >> 32);
  }
}

__global__ void k_lock_cols(Dev d, const int32_t* dn, const int32_t* up) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d.n) return;
  int q0 = d.cp[j], q1 = d.cp[j + 1];
  unsigned long long down = (unsigned)(dn[q1] - dn[q0]), upc = (unsigned)(up[q1] - up[q0]);
  d.locks[j] = down | (upc << 32);
}

void init_locks(const Dev& d, int32_t* dn, int32_t* up, int32_t* ws, hipStream_t s) {
  if (d.n == 0) return;
  int64_t blocks = (d.nnz + 1 + PSL_BLOCK - 1) / PSL_BLOCK;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_lock_bits, dim3((unsigned)blocks), dim3(PSL_BLOCK), 0, s, d, dn, up);
  scan_excl(dn, dn, d.nnz + 1, nullptr, ws, s);
  scan_excl(up, up, d.nnz + 1, nullptr, ws, s);
  hipLaunchKernelGGL(k_lock_cols, dim3((unsigned)((d.n + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d,
                     (const int32_t*)dn, (const int32_t*)up);
}

void launch_init_state(const Dev& d, const double* c_in, double* c_run, hipStream_t s) {
  int64_t t = d.m > d.n ? d.m : d.n;
  int64_t supers = (int64_t)decide_supers(d.m, d.n);
  if (t < supers) t = supers;
  hipLaunchKernelGGL(k_init_state, dim3((unsigned)((t + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d, supers,
                     c_in, c_run);
}

__global__ void k_round0_count(Dev d) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t m = d.m, n = d.n;
  if (t < m) {
    d.cnt[t] = 0;
    double l = d.lhs[t], r = d.rhs[t];
    if (!is_inf(l) && !is_inf(r) && l > r + tol_of(d.cfg, r)) flag_infeasible(d, row_lp_of(d, (int)t));
    return;
  }
  if (t >= m + n) return;
  int j = (int)(t - m);
  double2 b = d.bnd[j];
  int k = 0;
  if (!is_inf(b.x) && !is_inf(b.y)) {
    if (b.x > b.y + tol_of(d.cfg, b.y)) flag_infeasible(d, col_lp_of(d, j));
    if (b.y - b.x <= d.cfg.fix_tol * mx1(b.x)) k = 1;
  }
  d.cnt[t] = k;
}

__global__ void k_round0_emit(Dev d, int64_t base) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t m = d.m, n = d.n;
  if (t < m || t >= m + n) return;
  int j = (int)(t - m);
  double2 b = d.bnd[j];
  if (is_inf(b.x) || is_inf(b.y) || !(b.y - b.x <= d.cfg.fix_tol * mx1(b.x))) return;
  Record r;
  r.type = REC_FIX_COL;
  r.side = 0;
  r.round = 0;
  r.i = -1;
  r.j = j;
  r.k = -1;
  r.v[0] = b.x;
  r.v[1] = d.c[j];
  r.v[2] = 0.0;
  r.v[3] = 0.0;
  d.rec[base + d.off[t]] = r;
  d.bnd[j] = make_double2(b.x, b.x);
  d.bkey[2 * (int64_t)j + 1] = ukey(b.x);
}

void launch_round0_count(const Dev& d, hipStream_t s) {
  int64_t t = (int64_t)d.m + d.n;
  if (t == 0) return;
  hipLaunchKernelGGL(k_round0_count, dim3((unsigned)((t + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d);
}

void launch_round0_emit(const Dev& d, int64_t base, hipStream_t s) {
  int64_t t = (int64_t)d.m + d.n;
  if (t == 0) return;
  hipLaunchKernelGGL(k_round0_emit, dim3((unsigned)((t + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d,
                     base);
}

}  // namespace psl
