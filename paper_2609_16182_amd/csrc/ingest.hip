// ingest.hip -- validation, canonicalisation, the transposed copy of A, row
// binning and the input fixings ("round 0").
//
// The paper keeps A together with its transpose (section 3.2, "Internal data
// structures"). The transpose is built here by a stable radix sort of the CSR
// positions by column, so the rows of every column come out ascending.
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

__global__ void k_check_rows(Dev d) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.m) return;
  int32_t a = d.rp[i], b = d.rp[i + 1];
  if ((i == 0 && a != 0) || a < 0 || b < a || (int64_t)b > d.nnz || (i == d.m - 1 && (int64_t)b != d.nnz))
    report(d, ERR_ROWPTR, i);
  double l = d.lhs[i], r = d.rhs[i];
  double iv = d.cfg.inf_value;
  if (__builtin_isnan(l) || __builtin_isnan(r) || l >= iv || r <= -iv) report(d, ERR_SIDE, i);
  d.lhs[i] = canon_inf(l, iv);
  d.rhs[i] = canon_inf(r, iv);
}

__global__ void k_check_cols(Dev d, const double* lb_in, const double* ub_in, double* c_mut) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d.n) return;
  double l = lb_in[j], u = ub_in[j], c = c_mut[j];
  double iv = d.cfg.inf_value;
  if (__builtin_isnan(l) || __builtin_isnan(u) || l >= iv || u <= -iv) report(d, ERR_BOUND, j);
  if (!__builtin_isfinite(c)) report(d, ERR_COST, j);
  d.bnd[j] = make_double2(canon_inf(l, iv), canon_inf(u, iv));
  c_mut[j] = pos0(c);
}

// rowid1[e] counts the rows ending at position e; its exclusive scan then
// gives, at index p + 1, the row holding CSR position p.
__global__ void k_row_ends(Dev d, int32_t* cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.m) return;
  atomicAdd(&cnt[d.rp[i + 1]], 1);
}

__global__ void k_check_entries(Dev d, const int32_t* rowid1) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < d.nnz; p += (int64_t)gridDim.x * blockDim.x) {
    int row = rowid1[p + 1];
    int j = d.ci[p];
    if (j < 0 || j >= d.n || (p > d.rp[row] && d.ci[p - 1] >= j)) report(d, ERR_COLIDX, p);
    double a = d.va[p];
    if (!__builtin_isfinite(a) || a == 0.0) report(d, ERR_COEF, p);
  }
}

void launch_check_rows(const Dev& d, hipStream_t s) {
  if (d.m == 0) return;
  hipLaunchKernelGGL(k_check_rows, dim3((d.m + PSL_BLOCK - 1) / PSL_BLOCK), dim3(PSL_BLOCK), 0, s, d);
}

void check_cols(const Dev& d, const double* lb_in, const double* ub_in, double* c_mut, hipStream_t s) {
  if (d.n == 0) return;
  hipLaunchKernelGGL(k_check_cols, dim3((d.n + PSL_BLOCK - 1) / PSL_BLOCK), dim3(PSL_BLOCK), 0, s, d, lb_in, ub_in,
                     c_mut);
}

void build_rowid(const Dev& d, IngestScratch& sc, hipStream_t s) {
  fill_i32(sc.rowid1, 0, d.nnz + 1, s);
  if (d.m > 0)
    hipLaunchKernelGGL(k_row_ends, dim3((d.m + PSL_BLOCK - 1) / PSL_BLOCK), dim3(PSL_BLOCK), 0, s, d, sc.rowid1);
  scan_excl(sc.rowid1, sc.rowid1, d.nnz + 1, nullptr, sc.ws, s);
}

void launch_check_entries(const Dev& d, const int32_t* rowid1, hipStream_t s) {
  if (d.nnz == 0) return;
  int64_t blocks = (d.nnz + PSL_BLOCK - 1) / PSL_BLOCK;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(k_check_entries, dim3((unsigned)blocks), dim3(PSL_BLOCK), 0, s, d, rowid1);
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
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q <= d.nnz; q += (int64_t)gridDim.x * blockDim.x) {
    int64_t prev = q > 0 ? (int64_t)keys[q - 1] : -1;
    int64_t cur = q < d.nnz ? (int64_t)keys[q] : (int64_t)d.n;
    // keys were validated (< n); clamped all the same so no store leaves cp
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
}

// Stable transpose by LSD radix passes over the column index (at most 8 bits
// a pass, the bits split evenly), moving row and value with each key; the
// last pass writes the transposed copy itself. vtmp: nnz doubles of scratch.
// Returns the column of every position of the transposed copy (the sorted
// keys), which compaction uses.
const uint32_t* build_csc(const Dev& d, int32_t* cp, int32_t* ri, double* cva, int32_t* col_len, IngestScratch& sc,
                          double* vtmp, hipStream_t s) {
  int bits = 0;
  while (bits < 31 && ((int64_t)1 << bits) < (int64_t)d.n) ++bits;
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
      radix_pass_payload(kin, rin, sc.rowid1, vin, kout, rout, vout, d.nnz, shift, b, sc.ws, s);
      kin = kout;
      rin = rout;
      vin = vout;
    }
  }
  fill_i32(cp, -1, d.n + 1, s);
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
// row bins by CSR length, and the chunk table of long rows
// ---------------------------------------------------------------------------
// bin of every row, and the bin sizes (counted per wavefront by ballots, per
// workgroup in LDS, then one global add per workgroup and bin)
__global__ void k_bin_keys(Dev d, int32_t t_long, int32_t t_g8, uint32_t* keys, int32_t* counts) {
  __shared__ int c[NBINS];
  if (threadIdx.x < NBINS) c[threadIdx.x] = 0;
  __syncthreads();
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x; i0 < d.m; i0 += stride) {
    int64_t i = i0 + threadIdx.x;
    int b = -1;
    if (i < d.m) {
      int len = d.rp[i + 1] - d.rp[i];
      b = len <= 4 ? BIN_G4 : len <= t_g8 ? BIN_G8 : len <= 16 ? BIN_G16 : len > t_long ? BIN_LONG
        : len <= 64 ? BIN_W1 : len <= 256 ? BIN_W4 : BIN_W8;
      keys[i] = (uint32_t)b;
    }
#pragma unroll
    for (int k = 0; k < NBINS; ++k) {
      int cnt = __popcll(__ballot(b == k));
      if (lane_id() == 0 && cnt) atomicAdd(&c[k], cnt);
    }
  }
  __syncthreads();
  if (threadIdx.x < NBINS && c[threadIdx.x]) atomicAdd(&counts[threadIdx.x], c[threadIdx.x]);
}

__global__ void k_bin_fill(Dev d, const int32_t* rows, BinEnt* bins) {
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.m) return;
  int row = rows[k];
  int a = d.rp[row], b = d.rp[row + 1];
  bins[k] = BinEnt{row, a, b - a, 0};
}

void build_bins(const Dev& d, const int32_t* thresholds, BinEnt* bins, int32_t* counts, IngestScratch& sc,
                hipStream_t s) {
  fill_i32(counts, 0, NBINS, s);
  if (d.m == 0) return;
  unsigned blocks = (unsigned)((d.m + PSL_BLOCK - 1) / PSL_BLOCK);
  unsigned kb = blocks < 1024 ? blocks : 1024;
  hipLaunchKernelGGL(k_bin_keys, dim3(kb), dim3(PSL_BLOCK), 0, s, d, thresholds[0], thresholds[2], sc.k0, counts);
  radix_pass(sc.k0, nullptr, sc.k1, sc.v0, d.m, 0, 3, sc.ws, s);
  hipLaunchKernelGGL(k_bin_fill, dim3(blocks), dim3(PSL_BLOCK), 0, s, d, (const int32_t*)sc.v0, bins);
}

// ---------------------------------------------------------------------------
// filtering of the bin lists and the chunk list down to the active rows
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
  if (d.nlong == 0) {
    fill_i32(totals, 0, 2, s);
    return;
  }
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
// is 1024 rows, 4096 from SEL_BIG rows on (fewer adds to each count).
#define SEL_ITEMS 4
#define SEL_BIG (1 << 20)

struct SelArgs {
  int mode;             // -1: the device's (bit 0: marked rows only; bit 1: inert rows skipped)
  int t_long, t_g8;     // bin thresholds of the ingest
  int seq;              // launch number of the round before
};

// bin of a row of len entries (the bins of the ingest)
__device__ __forceinline__ int bin_of_len(int len, int t_long, int t_g8) {
  return len <= 4 ? BIN_G4 : len <= t_g8 ? BIN_G8 : len <= 16 ? BIN_G16 : len > t_long ? BIN_LONG
       : len <= 64 ? BIN_W1 : len <= 256 ? BIN_W4 : BIN_W8;
}

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
  }
}

void launch_rounds_begin(const Dev& d, int64_t rec_at, int64_t rec_cap, hipStream_t s) {
  hipLaunchKernelGGL(k_rounds_begin, dim3((d.K + PSL_BLOCK - 1) / PSL_BLOCK), dim3(PSL_BLOCK), 0, s, d, rec_at,
                     rec_cap);
}

// the columns of more than MARK_DENSE entries (order irrelevant)
__global__ void k_dense_cols(Dev d) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d.n) return;
  if (d.cp[j + 1] - d.cp[j] > MARK_DENSE) d.dense_cols[atomicAdd(d.n_dense, 1)] = (int32_t)j;
}

void list_dense_cols(const Dev& d, hipStream_t s) {
  fill_i32(d.n_dense, 0, 1, s);
  if (d.n > 0)
    hipLaunchKernelGGL(k_dense_cols, dim3((unsigned)((d.n + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d);
}

// ---------------------------------------------------------------------------
// state initialisation and round 0 (input fixings, crossed bounds / sides)
// ---------------------------------------------------------------------------
__global__ void k_init_state(Dev d, int64_t supers) {
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
    f.infeasible = f.unbounded = f.error = f.merged = 0;
    f.cand_count = f.round_total = f.vlist_count = f.rows_removed = 0;
    f.fin_cols = f.mode = f.lead_count = f.fs_total = f.fs_rows = f.fs_claims = 0;
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

void launch_init_state(const Dev& d, hipStream_t s) {
  int64_t t = d.m > d.n ? d.m : d.n;
  int64_t supers = (int64_t)decide_supers(d.m, d.n);
  if (t < supers) t = supers;
  hipLaunchKernelGGL(k_init_state, dim3((unsigned)((t + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d, supers);
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
