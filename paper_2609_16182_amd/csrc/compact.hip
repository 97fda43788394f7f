// compact.hip -- emission of the reduced LP (section 3.3): kept rows x kept
// columns in their original order, sides shifted by the removed columns'
// constant contribution (canonical pairwise sum over the row, computed by the
// sweep in compaction mode), the removed columns' cost terms folded into the
// objective offset, and both the CSR and the transposed copy.
//
// Output positions are ranks among keep flags, of the rows, the columns, the
// CSR positions and the transposed copy's positions, so the kept entries keep
// their order in both layouts. The flags are bits: 64 and the kept ones before
// them in their tile of 2048 to a word, the tiles' counts of all four in one
// array whose scan gives the tiles' places. (With an int per position, flags,
// scans and gathers took 4.6 ms for 9.7e7 entries, 3.2 now;
// 2000 rows: 15 launches, 7 now.) In a batch the LPs are blocks of one LP, so
// each LP's kept rows, columns and entries are contiguous in these ranks.
#include "bits.h"
#include "psl_kern.h"
#include "sweep.h"

namespace psl {

#define CMP_TILE PW_TILE  // the columns' tiles are also those of their cost terms' sum
#define CMP_ITEMS (CMP_TILE / PSL_BLOCK)
#define CMP_WORDS (CMP_TILE / 64)

// Words and count of a tile from the lanes' flags: item k * 256 + thread of the
// tile has flag k; size items in all.
struct TileBits {
  unsigned long long bits[CMP_WORDS];
  int total;
};
__device__ __forceinline__ void tile_bits(const bool (&f)[CMP_ITEMS], TileBits& sh, RankWord* words, int64_t size,
                                          int64_t tile, int32_t* count) {
  const int t = threadIdx.x, w = t >> 6;
#pragma unroll
  for (int k = 0; k < CMP_ITEMS; ++k) {
    const unsigned long long m = __ballot(f[k]);
    if (lane_id() == 0) sh.bits[k * (PSL_BLOCK / 64) + w] = m;
  }
  __syncthreads();
  if (t < CMP_WORDS) {  // half a wavefront
    const unsigned long long m = sh.bits[t];
    int pre = __popcll(m);
    const int own = pre;
#pragma unroll
    for (int o = 1; o < CMP_WORDS; o <<= 1) {
      const int x = __shfl_up(pre, o, CMP_WORDS);
      if (t >= o) pre += x;
    }
    const int64_t at = tile * CMP_WORDS + t;
    if (at <= size / 64) words[at] = RankWord{m, pre - own, 0};
    if (t == CMP_WORDS - 1) *count = pre;
  }
}

// kept items before item i, i < size of the section whose first tile is t0
__device__ __forceinline__ int rank_in(const CompactScratch& c, const RankWord* words, int t0, int64_t i) {
  return c.tile_off[t0 + i / CMP_TILE] - c.tile_off[t0] + tile_rank_of(words, i);
}
// the same for i <= size
__device__ __forceinline__ int rank_to(const CompactScratch& c, const RankWord* words, int t0, int64_t i) {
  return i % CMP_TILE ? rank_in(c, words, t0, i) : c.tile_off[t0 + i / CMP_TILE] - c.tile_off[t0];
}

// kept rows and columns, the removed columns' cost terms (K > 1) or their tile
// sums (K = 1)
__global__ void __launch_bounds__(PSL_BLOCK) k_cmp_flags(Dev d, CompactScratch c) {
  __shared__ TileBits sh;
  __shared__ double terms[CMP_TILE];
  bool f[CMP_ITEMS];
  const int t = threadIdx.x;
  if (blockIdx.x == 0 && t == 0) c.tile_off[c.tiles] = 0;
  if ((int)blockIdx.x < c.t_col) {
    const int64_t i0 = (int64_t)blockIdx.x * CMP_TILE + t;
#pragma unroll
    for (int k = 0; k < CMP_ITEMS; ++k) f[k] = i0 + k * PSL_BLOCK < d.m && d.row_on[i0 + k * PSL_BLOCK] != 0;
    tile_bits(f, sh, c.rbits, d.m, blockIdx.x, c.tile_off + blockIdx.x);
    return;
  }
  const int64_t tile = (int64_t)blockIdx.x - c.t_col, j0 = tile * CMP_TILE + t;
#pragma unroll
  for (int k = 0; k < CMP_ITEMS; ++k) {
    const int64_t j = j0 + k * PSL_BLOCK;
    double term = 0.0;
    f[k] = false;
    if (j < d.n) {
      const double2 b = d.bnd[j];
      f[k] = b.x != b.y;
      term = f[k] ? 0.0 : pos0(d.c[j] * b.x);
      if (d.K > 1) c.terms[j] = term;
    }
    terms[k * PSL_BLOCK + t] = term;
  }
  tile_bits(f, sh, c.cbits, d.n, tile, c.tile_off + blockIdx.x);
  if (d.K > 1) return;
  __syncthreads();
  const double sum = tile_sum(terms, d.n - tile * CMP_TILE);
  if (t == 0) c.terms[tile] = sum;
}

// kept positions of both layouts (a position is kept when its row and its
// column are): in CSR order the row is monotone and the column random, in
// the transposed copy the other way round; the bits looked up are L2-resident
__global__ void __launch_bounds__(PSL_BLOCK) k_cmp_positions(Dev d, CompactScratch c) {
  __shared__ TileBits sh;
  const bool csr = (int)blockIdx.x < c.t_csc - c.t_csr;
  const int64_t tile = csr ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - (c.t_csc - c.t_csr);
  const int64_t p0 = tile * CMP_TILE + threadIdx.x;
  int major[CMP_ITEMS], minor[CMP_ITEMS];
#pragma unroll
  for (int k = 0; k < CMP_ITEMS; ++k) {
    const int64_t p = p0 + k * PSL_BLOCK < d.nnz ? p0 + k * PSL_BLOCK : 0;
    major[k] = csr ? c.rowid1[p + 1] : (int)c.colid[p];
    minor[k] = csr ? d.ci[p] : d.ri[p];
  }
  bool f[CMP_ITEMS];
#pragma unroll
  for (int k = 0; k < CMP_ITEMS; ++k)
    f[k] = p0 + k * PSL_BLOCK < d.nnz && bit_of(csr ? c.rbits : c.cbits, major[k]) &&
           bit_of(csr ? c.cbits : c.rbits, minor[k]);
  tile_bits(f, sh, csr ? c.ebits : c.qbits, d.nnz, tile, c.tile_off + c.t_csr + blockIdx.x);
}

// Batched presolve: each LP's reduced problem is numbered from 0 (its rows,
// columns and positions start at the LP's bases in c.lpr) and its row and
// column pointer arrays get one end entry each, at lpr.rb + k and lpr.cb + k.
// Also the totals, of a single LP the objective offset (from the cost terms'
// sum, null: no column), and the rows' and columns' ranks in all, which the
// gather looks up at random (with the tile's place as a second look-up it took
// 2.39 ms for 9.7e7 entries, 1.97 now).
__global__ void k_cmp_lpbase(Dev d, CompactScratch c, Reduced r, const double* sum, double off) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (64 * (int64_t)k < d.m)
    c.rbits[k].all = c.tile_off[k / CMP_WORDS] - c.tile_off[0] + c.rbits[k].pre;
  if (64 * (int64_t)k < d.n)
    c.cbits[k].all = c.tile_off[c.t_col + k / CMP_WORDS] - c.tile_off[c.t_col] + c.cbits[k].pre;
  if (k > d.K) return;
  auto base = [&](int q) {
    int i0 = d.K > 1 ? d.lp_row0[q] : (q ? d.m : 0);
    int j0 = d.K > 1 ? d.lp_col0[q] : (q ? d.n : 0);
    LpRed b;
    b.rb = rank_to(c, c.rbits, 0, i0);
    b.cb = rank_to(c, c.cbits, c.t_col, j0);
    b.eb = rank_to(c, c.ebits, c.t_csr, d.rp[i0]);
    b.qb = rank_to(c, c.qbits, c.t_csc, d.cp[j0]);
    return b;
  };
  LpRed b = base(k);
  c.lpr[k] = b;
  if (k < d.K) {
    LpRed e = base(k + 1);
    r.row_ptr[e.rb + k] = e.eb - b.eb;
    r.col_ptr[e.cb + k] = e.qb - b.qb;
  } else {
    c.totals[0] = b.rb;
    c.totals[1] = b.cb;
    c.totals[2] = c.tile_off[c.t_csc] - c.tile_off[c.t_csr];
    c.totals[3] = c.tile_off[c.tiles] - c.tile_off[c.t_csc];
    if (d.K == 1) c.offset[0] = pos0(off + (sum ? *sum : 0.0));
  }
}

// kept entries of the CSR (new column ids from the column bits) and of the
// transposed copy (new row ids from the row bits)
__global__ void __launch_bounds__(PSL_BLOCK) k_cmp_gather(Dev d, CompactScratch c, Reduced r) {
  const bool csr = (int)blockIdx.x < c.t_csc - c.t_csr;
  const int64_t tile = csr ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - (c.t_csc - c.t_csr);
  const int64_t p0 = tile * CMP_TILE + threadIdx.x;
  const RankWord* words = csr ? c.ebits : c.qbits;
  const int32_t* minor = csr ? d.ci : d.ri;
  const double* val = csr ? d.va : d.cva;
  const RankWord* ids = csr ? c.cbits : c.rbits;
  const int at = c.tile_off[c.t_csr + blockIdx.x] - c.tile_off[csr ? c.t_csr : c.t_csc];
  const unsigned long long below = lanemask_lt();
  int j[CMP_ITEMS], pos[CMP_ITEMS];
  double a[CMP_ITEMS];
#pragma unroll
  for (int k = 0; k < CMP_ITEMS; ++k) {
    const int64_t p = p0 + k * PSL_BLOCK;
    pos[k] = -1;
    j[k] = 0;
    a[k] = 0.0;
    if (p < d.nnz) {
      const RankWord w = words[p >> 6];
      if (w.bits >> lane_id() & 1) pos[k] = at + w.pre + __popcll(w.bits & below);
      j[k] = minor[p];
      a[k] = val[p];
    }
  }
#pragma unroll
  for (int k = 0; k < CMP_ITEMS; ++k) {
    if (pos[k] < 0) continue;
    int id = rank_of(ids, j[k]);
    if (d.K > 1) id -= csr ? c.lpr[d.col_lp[j[k]]].cb : c.lpr[d.row_lp[j[k]]].rb;
    (csr ? r.col_idx : r.row_idx)[pos[k]] = id;
    (csr ? r.val : r.cval)[pos[k]] = a[k];
  }
}

__global__ void k_cmp_fill(Dev d, CompactScratch c, Reduced r) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t m = d.m, n = d.n;
  if (t < m) {
    int i = (int)t;
    if (!d.row_on[i]) return;
    int lp = row_lp_of(d, i);
    LpRed b = c.lpr[lp];
    int ri = rank_of(c.rbits, i);
    double k = d.row_out[i].v0;  // constant of the removed columns
    double l = d.lhs[i], u = d.rhs[i];
    double nl = is_inf(l) ? l : pos0(l - k);
    double nu = is_inf(u) ? u : pos0(u - k);
    int p0 = rank_to(c, c.ebits, c.t_csr, d.rp[i]), p1 = rank_to(c, c.ebits, c.t_csr, d.rp[i + 1]);
    int len = p1 - p0;
    r.row_map[ri] = i - (d.K > 1 ? d.lp_row0[lp] : 0);
    r.lhs[ri] = nl;
    r.rhs[ri] = nu;
    r.row_ptr[ri + lp] = p0 - b.eb;
    r.row_class[ri] = len == 1 ? 1 : len == 2 ? (nl == nu ? 2 : 3) : 0;
    return;
  }
  if (t >= m + n) return;
  int j = (int)(t - m);
  double2 b = d.bnd[j];
  if (b.x == b.y) return;
  int lp = col_lp_of(d, j);
  LpRed cb = c.lpr[lp];
  int rj = rank_of(c.cbits, j);
  int q0 = rank_to(c, c.qbits, c.t_csc, d.cp[j]), q1 = rank_to(c, c.qbits, c.t_csc, d.cp[j + 1]);
  int len = q1 - q0;
  r.col_map[rj] = j - (d.K > 1 ? d.lp_col0[lp] : 0);
  r.lb[rj] = b.x;
  r.ub[rj] = b.y;
  r.c[rj] = d.c[j];
  r.col_ptr[rj + lp] = q0 - cb.qb;
  bool fr = is_inf(b.x) && is_inf(b.y);
  r.col_class[rj] = len == 1 ? (fr ? 1 : 2) : len == 2 ? 3 : 0;
}

int64_t compact_tiles(int64_t m, int64_t n, int64_t nnz) {
  auto t = [](int64_t x) { return (x + CMP_TILE - 1) / CMP_TILE; };
  return t(m) + t(n) + 2 * t(nnz);
}

void compact(const Dev& d, const CompactScratch& scratch, const Reduced& r, double obj_offset, hipStream_t s) {
  CompactScratch c = scratch;
  c.t_col = (int)compact_tiles(d.m, 0, 0);
  c.t_csr = (int)compact_tiles(d.m, d.n, 0);
  c.tiles = (int)compact_tiles(d.m, d.n, d.nnz);
  c.t_csc = c.t_csr + (c.tiles - c.t_csr) / 2;
  const int col_tiles = c.t_csr - c.t_col;
  hipLaunchKernelGGL(k_cmp_flags, dim3(c.t_csr > 0 ? c.t_csr : 1), dim3(PSL_BLOCK), 0, s, d, c);
  if (d.nnz > 0)
    hipLaunchKernelGGL(k_cmp_positions, dim3(c.tiles - c.t_csr), dim3(PSL_BLOCK), 0, s, d, c);
  scan_excl(c.tile_off, c.tile_off, (int64_t)c.tiles + 1, nullptr, c.ws, s);
  const double* sum = nullptr;
  if (d.K > 1) {
    segmented_pairwise_sum(c.terms, c.seg, c.seg_host, d.K, c.lp_off_in, c.offset, c.pws, s);
  } else if (col_tiles == 1) {
    sum = c.terms;
  } else if (col_tiles > 1) {  // the tree above the tiles
    pairwise_sum(c.terms, col_tiles, c.pws, c.pws + 1, s);
    sum = c.pws;
  }
  const int64_t words = std::max<int64_t>((std::max(d.m, d.n) + 63) / 64, d.K + 1);
  hipLaunchKernelGGL(k_cmp_lpbase, dim3((unsigned)((words + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d, c, r, sum,
                     obj_offset);
  if (d.nnz > 0)
    hipLaunchKernelGGL(k_cmp_gather, dim3(c.tiles - c.t_csr), dim3(PSL_BLOCK), 0, s, d, c, r);
  int64_t t = (int64_t)d.m + d.n;
  if (t < 1) t = 1;
  hipLaunchKernelGGL(k_cmp_fill, dim3((unsigned)((t + PSL_BLOCK - 1) / PSL_BLOCK)), dim3(PSL_BLOCK), 0, s, d, c, r);
}

}  // namespace psl
