// sweep.hip -- one propagation round (section 3.1, "Bound tightening" and
// "Length-based load balancing"; section 3.2, "Internal data structures").
//
// Round semantics (Jacobi): every test reads the bounds as they were when the
// round started (bnd); tightenings are combined in bkey with order-free
// atomic maxima of order-mapped int64 keys; the source row of a final bound
// is the lowest row whose candidate equals it (resolved from a candidate list
// after the sweep). Activities are canonical pairwise trees over the row's CSR
// positions (leaves padded with +0 to a power of two), so every aligned
// power-of-two grouping of positions -- C contiguous positions per lane, a
// butterfly over G lanes, four wavefronts, chunk partials -- gives the same
// bits, whatever bin a row falls in.
//
// Bins (by CSR length; the order of the rows in a bin is of no consequence):
//   G4  <= 4     4-lane groups, 1 position per lane
//   G8  <= 8     8-lane groups, 1 position per lane
//   G16 <= 16    16-lane groups, 1 position per lane
//   W1  <= 64    one wavefront, 1 position per lane
//   W4  <= 256   one wavefront, 4 contiguous positions per lane
//   W8  <= 512   one wavefront, 8 contiguous positions per lane
//   LONG         chunks of npass * 2048 positions, one workgroup each:
//                k_long_stats writes chunk partials, then k_sweep combines
//                them in tree order and propagates chunk by chunk.
// Each row is handled in one pass with its elements kept in registers.
//
// What bounds it: misses of the L2, one 128 B line for each gathered 16 B bound
// (1e7 rows, every row swept: 96e6 gathers in 1.9 ms, 5.0e10/s; a plain gather
// of that size reaches 5.6e10/s), and below that the vector memory unit's
// stalls on lines in flight. Against a version with branches per condition, LDS
// shuffles and a look at the accumulators (a 4096-LP batch, every row swept: 310
// vector and 244 scalar instructions for each 64 positions, 2.2 ms) this one has
// 275 and 130 and takes 1.87 ms; its later rounds 1.67 -> 1.37 ms.
#include "psl_kern.h"
#include "sweep.h"

namespace psl {


struct El {
  int j;
  double a, lb, ub;
  bool v;
};

// Elements at positions s0 + base + k (k < C) of a row, valid when on and
// base + k < len. All loads are issued before any is used, without branches
// between them (an invalid element reads position 0, which exists whenever
// the matrix has an entry), so a lane has C gathers in flight at once.
template <int C>
__device__ __forceinline__ void load_els(const Dev& d, int64_t s0, int len, int base, bool on, El (&e)[C]) {
  int j[C];
  double a[C];
  double2 b[C];
  bool v[C];
#pragma unroll
  for (int k = 0; k < C; ++k) {
    v[k] = on && base + k < len;
    j[k] = 0;
    a[k] = 0.0;
    b[k] = make_double2(0.0, 0.0);
  }
  if (d.nnz > 0) {
#pragma unroll
    for (int k = 0; k < C; ++k) {
      int64_t p = v[k] ? s0 + base + k : 0;
      j[k] = d.ci[p];
      a[k] = d.va[p];
    }
#pragma unroll
    for (int k = 0; k < C; ++k) b[k] = d.bnd[j[k]];
  }
#pragma unroll
  for (int k = 0; k < C; ++k) {
    e[k].v = v[k];
    e[k].j = v[k] ? j[k] : 0;
    e[k].a = v[k] ? a[k] : 0.0;
    e[k].lb = v[k] ? b[k].x : 0.0;
    e[k].ub = v[k] ? b[k].y : 0.0;
  }
}

__device__ __forceinline__ bool el_active(const El& e) { return e.v && e.lb != e.ub; }

// activity terms of one element and its packed counts
// (bit 0: infinite min contribution, bit 10: infinite max, bit 20: active)
// (straight-line: an invalid element holds a = lb = ub = 0 and so gives +0
// terms and no counts)
template <int MODE>
__device__ __forceinline__ void el_terms(const El& e, double& tmin, double& tmax, int& cnt) {
  tmin = tmax = 0.0;
  cnt = 0;
  bool act = e.v && e.lb != e.ub;
  if (MODE == MODE_ROUND) {
    bool imin, imax;
    contrib(e.a, e.lb, e.ub, tmin, imin, tmax, imax);
    cnt = (imin ? 1 : 0) | (imax ? 1 << 10 : 0) | (act ? 1 << 20 : 0);
  } else {
    // compaction: constant of the removed columns; active-entry count
    tmin = act ? 0.0 : pos0(e.a * e.lb);
    cnt = act ? 1 << 20 : 0;
  }
}

__device__ __forceinline__ int cnt_min(int c) { return c & 1023; }
__device__ __forceinline__ int cnt_max(int c) { return (c >> 10) & 1023; }
__device__ __forceinline__ int cnt_act(int c) { return c >> 20; }

// pairwise tree over C values held in registers (C a power of two)
template <int C>
__device__ __forceinline__ double lane_tree(double (&x)[C]) {
#pragma unroll
  for (int w = 1; w < C; w <<= 1)
#pragma unroll
    for (int i = 0; i < C; i += 2 * w) x[i] = x[i] + x[i + w];
  return x[0];
}

// load C contiguous positions [base, base + C) of a row and reduce them
template <int C, int MODE>
__device__ __forceinline__ void lane_stats(const Dev& d, int64_t s0, int len, int base, El (&e)[C], double& smin,
                                           double& smax, int& cnt) {
  double a[C], b[C];
  cnt = 0;
  load_els<C>(d, s0, len, base, true, e);
#pragma unroll
  for (int k = 0; k < C; ++k) {
    int c;
    el_terms<MODE>(e[k], a[k], b[k], c);
    cnt += c;
  }
  smin = lane_tree<C>(a);
  smax = lane_tree<C>(b);
}

struct RowDec {
  uint8_t code;
  bool infeasible, prop, single;
  int force;  // forcing row: 1 at its min activity (= rhs), 2 at its max (= lhs)
};

// Row decisions from the round's statistics. any_tiny: the row has an active
// entry with |a| < coef_tol (such a row is never forcing: its column could
// move far within the tolerance).
__device__ __forceinline__ RowDec decide_row(const Cfg& c, double lhs, double rhs, int L, int nmin, int nmax,
                                             double minact, double maxact, bool any_tiny) {
  // Without branches, as prop_el: all conditions are evaluated (those of an
  // infinite side compare to a NaN or an infinity and are masked out).
  RowDec r{RC_KEEP, false, false, false, 0};
  const bool fl = !is_inf(lhs), fr = !is_inf(rhs), empty = L == 0;
  const bool n0 = nmin == 0, x0 = nmax == 0;
  const double tl = tol_of(c, lhs), tr = tol_of(c, rhs);
  const bool lo_ok = !fl | (n0 & (minact >= lhs - tl));
  const bool up_ok = !fr | (x0 & (maxact <= rhs + tr));
  const bool leaves = lo_ok & up_ok;
  const bool beyond = (n0 & fr & (minact > rhs + tr)) | (x0 & fl & (maxact < lhs - tl));
  if (leaves) r.code = empty ? RC_EMPTY : RC_REDUNDANT;
  r.infeasible = !leaves & (empty | beyond);
  // A side gives an entry a bound only when the residual activity on that side
  // is finite, i.e. with at most one infinite contribution (the entry's own);
  // with none on either side the row yields no candidate and is not re-read.
  // (A row with one active column has at most one infinite contribution per
  // side, so it always propagates on its finite sides.)
  r.prop = !leaves & !empty & ((fr & (nmin <= 1)) | (fl & (nmax <= 1)));
  r.single = !leaves & (L == 1);
  // Forcing rows (at least two active columns): the finite min activity
  // reaching rhs (or the max reaching lhs) within tol leaves every active
  // column at the bound of that contribution; the row leaves and those
  // bounds become candidates.
  if (c.forcing && !leaves && !r.infeasible && L >= 2 && !any_tiny) {
    if (nmin == 0 && !is_inf(rhs) && minact >= rhs - tol_of(c, rhs)) r.force = 1;
    else if (nmax == 0 && !is_inf(lhs) && maxact <= lhs + tol_of(c, lhs)) r.force = 2;
    if (r.force) r.code = r.force == 1 ? RC_FORCE_MIN : RC_FORCE_MAX;
  }
  return r;
}

__device__ __forceinline__ bool is_forcing(uint8_t code) { return code == RC_FORCE_MIN || code == RC_FORCE_MAX; }

struct RowStat {
  double minact, maxact;
  int nmin, nmax;
};

// Implied bounds of one active entry from the residual activity (the row's
// activity with the entry's own contribution taken out). Side 0 uses rhs and
// the residual min, side 1 lhs and the residual max; a > 0 turns side 0 into an
// upper bound, a < 0 into a lower bound. cap = false when a finite side yields
// no bound (it matters for rows with one active column, which are removed only
// when every finite side became a bound).
__device__ __forceinline__ void prop_el(const Cfg& c, bool on, const El& e, double lhs, double rhs, const RowStat& st,
                                        bool single, int force, bool& cap, bool& hlo, double& tlo, bool& hup,
                                        double& tup) {
  // without branches: a wavefront's lanes take every path between them, and
  // each branch costs its mask's scalar work; only the divisions are skipped
  const bool fr = !is_inf(rhs), fl = !is_inf(lhs), pos = e.a > 0;
  const bool tiny = fabs(e.a) < c.coef_tol;
  double tmin, tmax;
  bool imin, imax;
  contrib(e.a, e.lb, e.ub, tmin, imin, tmax, imax);
  const bool h0 = fr & ((st.nmin == 0) | ((st.nmin == 1) & imin));
  const bool h1 = fl & ((st.nmax == 0) | ((st.nmax == 1) & imax));
  double t0 = 0.0, t1 = 0.0;
  on = on & !((force == 0) & tiny);
  const double r0 = rhs - (st.nmin == 0 ? st.minact - tmin : st.minact);
  const double r1 = lhs - (st.nmax == 0 ? st.maxact - tmax : st.maxact);
  if (on & h0) t0 = pos0(r0 / e.a);
  if (on & h1) t1 = pos0(r1 / e.a);
  const bool v0 = h0 & (fabs(t0) < c.inf_value), v1 = h1 & (fabs(t1) < c.inf_value);
  cap = !tiny & (v0 | !fr) & (v1 | !fl);
  tup = pos ? t0 : t1;
  tlo = pos ? t1 : t0;
  const double u = e.ub, l = e.lb;
  const double du = c.min_improve * mx1(u), dl = c.min_improve * mx1(l);
  const bool qu = is_inf(u) | (tup < (single ? u : u - du));
  const bool ql = is_inf(l) | (tlo > (single ? l : l + dl));
  hup = on & (pos ? v0 : v1) & qu;
  hlo = on & (pos ? v1 : v0) & ql;
  if (c.forcing && force) {
    // a forcing row: the column's other bound moves onto the forced one
    // (min side: a > 0 at lb, a < 0 at ub; max side the other way round)
    const bool up = (force == 1) == pos;
    cap = true;
    hup = on && up && l < u;
    hlo = on && !up && u > l;
    tup = l;
    tlo = u;
  }
}

struct CandSink {  // this workgroup's candidate region and its LDS counter
  Cand* list;
  int32_t* counter;
};

// Fold qualifying candidates into the round's accumulators and list them; a
// candidate that another one beats is found not to be the final bound when the
// sources are taken. Nothing is read back, so no wavefront waits for memory
// here; in an LP with long columns (d.look_first) the accumulators are read first,
// since a beaten candidate's atomic waits for all others on that address. The
// look is the whole LP's: 1e6 power-law rows, with many long columns, take 4.41
// ms a presolve with it and 4.77 without; 1e7 rows with 20 long columns of 1.5e7
// 72.7 and 72.0, so a few of them pay for it; a 4096-LP batch without any, which
// has no look, 71.4 with one and 70.7.
// Most lanes have one side at most, so one atomic and one store serve both.
// Must be reached by every lane of the wavefront.
__device__ __forceinline__ void commit_cands(const Dev& d, const CandSink& sk, int pos, int j, bool hlo, double tlo,
                                             bool hup, double tup) {
  if (__ballot(hlo | hup) == 0) return;
  long long* const k = &d.bkey[2 * (int64_t)j];
  const long long klo = dkey(tlo), kup = ukey(tup);
  bool alo = hlo, aup = hup;
  if (d.look_first && (hlo | hup)) {
    const longlong2 cur = *reinterpret_cast<const longlong2*>(k);  // may be stale (wider): only costs an atomic
    hlo = hlo & (klo >= cur.x);
    hup = hup & (kup >= cur.y);
    alo = hlo & (klo > cur.x);
    aup = hup & (kup > cur.y);
  }
  const unsigned long long one = __ballot(hlo | hup), two = __ballot(hlo & hup);
  if (one == 0) return;
  const int n1 = __popcll(one);
  int base = 0;
  if (lane_id() == 0) base = atomicAdd(sk.counter, n1 + (int)__popcll(two));
  if (alo | aup) atomicMax(alo ? k : k + 1, alo ? klo : kup);
  if (alo & aup) atomicMax(k + 1, kup);
  base = __builtin_amdgcn_readfirstlane(base);
  const unsigned long long below = lanemask_lt();
  if (hlo | hup) {
    d.touch[j] = 1;
    sk.list[base + __popcll(one & below)] = hlo ? Cand{2 * j, pos, tlo} : Cand{2 * j + 1, pos, tup};
  }
  if (hlo & hup) sk.list[base + n1 + __popcll(two & below)] = Cand{2 * j + 1, pos, tup};
}

__device__ __forceinline__ RowOut row_out_of(uint8_t code, const RowStat& st) {
  RowOut o;
  o.j = -1;
  o.pad = 0;
  if (code == RC_EMPTY || code == RC_FORCE_MIN) {
    o.v0 = st.minact;
    o.v1 = 0.0;
  } else if (code == RC_FORCE_MAX) {
    o.v0 = st.maxact;
    o.v1 = 0.0;
  } else {
    o.v0 = st.nmin ? -__builtin_huge_val() : st.minact;
    o.v1 = st.nmax ? __builtin_huge_val() : st.maxact;
  }
  return o;
}

// propagate the C register-held elements of a lane; tracks the one active
// element of a row with L == 1 and whether some entry left a side unbounded
template <int C>
__device__ __forceinline__ void lane_prop(const Dev& d, const CandSink& sk, int64_t p0, bool prop, const El (&e)[C],
                                          double lhs, double rhs,
                                          const RowStat& st, bool single, int force, bool& uncap, bool& mine,
                                          int& aj, double& aa) {
#pragma unroll
  for (int k = 0; k < C; ++k) {
    bool act = prop && el_active(e[k]);
    bool cap, hlo, hup;
    double tlo, tup;
    prop_el(d.cfg, act, e[k], lhs, rhs, st, single, force, cap, hlo, tlo, hup, tup);
    commit_cands(d, sk, (int)(p0 + k), e[k].j, hlo, tlo, hup, tup);
    if (act && !cap) uncap = true;
    if (act) {
      mine = true;
      aj = e[k].j;
      aa = e[k].a;
    }
  }
}

// the same, loading the elements again in groups of (at most) four, so that
// wide lanes do not keep C elements live while each group's gathers are in
// flight together
#define STREAM_GROUP 4
template <int C>
__device__ __forceinline__ void lane_prop_stream(const Dev& d, const CandSink& sk, bool prop, int64_t s0,
                                                 int len, int base, double lhs, double rhs, const RowStat& st,
                                                 bool single, int force, bool& uncap, bool& mine, int& aj,
                                                 double& aa) {
  constexpr int GS = C < STREAM_GROUP ? C : STREAM_GROUP;
#pragma unroll 1
  for (int g = 0; g < C; g += GS) {
    El e[GS];
    load_els<GS>(d, s0, len, base + g, prop, e);
#pragma unroll
    for (int k = 0; k < GS; ++k) {
      bool act = el_active(e[k]);
      bool cap, hlo, hup;
      double tlo, tup;
      prop_el(d.cfg, act, e[k], lhs, rhs, st, single, force, cap, hlo, tlo, hup, tup);
      commit_cands(d, sk, (int)(s0 + base + g + k), e[k].j, hlo, tlo, hup, tup);
      if (act && !cap) uncap = true;
      if (act) {
        mine = true;
        aj = e[k].j;
        aa = e[k].a;
      }
    }
  }
}

template <int C>
__device__ __forceinline__ void lane_drop_stream(const Dev& d, bool on, int64_t s0, int len, int base, double lhs,
                                                 double rhs) {
  constexpr int GS = C < STREAM_GROUP ? C : STREAM_GROUP;
#pragma unroll 1
  for (int g = 0; g < C; g += GS) {
    El e[GS];
    load_els<GS>(d, s0, len, base + g, on, e);
#pragma unroll
    for (int k = 0; k < GS; ++k)
      if (el_active(e[k])) drop_col(d, e[k].j, e[k].a, lhs, rhs);
  }
}

template <int C>
__device__ __forceinline__ void lane_drop(const Dev& d, const El (&e)[C], double lhs, double rhs) {
#pragma unroll
  for (int k = 0; k < C; ++k)
    if (el_active(e[k])) drop_col(d, e[k].j, e[k].a, lhs, rhs);
}

// ---------------------------------------------------------------------------
// rows of at most G*C entries: one G-lane group per row, C positions per lane
// ---------------------------------------------------------------------------

// a round's sweep: what its workgroups know of the round, and what they count
struct RoundArgs {
  int mode;       // bit 0: marked rows only; bit 1: inert rows skipped (direct lists)
  uint8_t mark;   // the round's mark
  int32_t* rows;  // LDS: rows and nonzeros swept (direct lists)
  int32_t* nnz;
};

// a lane's part of its row in a row block
template <int C>
struct RowIn {
  bool on;       // the row is swept
  int len;
  int64_t s0;
  double lhs, rhs;
  El e[C];
};

// a lane's row of a list, and whether it is swept
struct RowOf {
  bool vr, on;
  int row, start, len;
  double lhs, rhs;
};

// First level of a list's loads: the entry of the lane's row. A lane beyond the
// bin's last row (cap rows at most) reads that one's entry, so the load does
// not wait for the list's length.
__device__ __forceinline__ BinEnt row_entry(const Dev& d, int bin, int cap, int gid) {
  return d.bins[d.bin_off[bin] + (gid < cap ? gid : cap - 1)];
}

__device__ __forceinline__ void row_take(const BinEnt& be, bool vr, RowOf& r) {
  r.vr = vr;
  r.row = vr ? be.row : 0;
  r.start = vr ? be.start : 0;
  r.len = vr ? be.len : 0;
}

// Second level: the row's sides and flags, beside the positions (columns and
// coefficients); the third level, the bounds, is issued by load_els or by the
// caller. A row of the direct lists is swept when it is active, of an LP that was
// presolving when the round began and, by the mode, marked / not inert.
template <int MODE, bool DIR>
__device__ __forceinline__ void row_data(const Dev& d, const RoundArgs& ra, RowOf& r) {
  r.lhs = d.lhs[r.row];
  r.rhs = d.rhs[r.row];
  if (MODE == MODE_COMPACT) {
    r.on = r.vr && d.row_on[r.row] != 0;
  } else if (DIR) {
    uint8_t on = d.row_on[r.row], dt = d.dirty[r.row];
    int2 rf = d.rinf[r.row];
    r.on = r.vr && on != 0 && (!(ra.mode & 1) || dt == ra.mark) && row_lp_swept(d, r.row) &&
           (!(ra.mode & 2) || !row_inert(rf, r.lhs, r.rhs));
  } else {
    r.on = r.vr;  // selected
  }
}

// Outcome of a swept row for its lane: code and infinite-contribution counts.
struct RowRes {
  uint32_t w;
  __device__ __forceinline__ static uint32_t pack(uint8_t code, int nmin, int nmax) {
    return (uint32_t)code | (uint32_t)nmin << 8 | (uint32_t)nmax << 18;
  }
};
__device__ __forceinline__ void row_store(const Dev& d, int row, uint32_t w) {
  d.rinf[row] = make_int2((int)(w >> 8) & 1023, (int)(w >> 18));
  d.row_code[row] = (uint8_t)w;
}

// Statistics, decisions, candidates and removals of the row block's rows from
// the loaded inputs (elements of inactive rows are cleared here). Lane `from`
// holds the lane's row number. Returns the row's packed outcome.
template <int G, int C, int MODE>
__device__ __forceinline__ uint32_t row_block(const Dev& d, const CandSink& sk, RowIn<C>& in, bool vr, int row_of,
                                              int from) {
  const bool on = in.on;
  const int len = in.len;
  const int64_t s0 = in.s0;
  int gl = threadIdx.x & (G - 1);
  El(&e)[C] = in.e;
  double smin, smax;
  int cnt = 0;
  {
    double a[C], b[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
      if (!on) e[k] = El{0, 0.0, 0.0, 0.0, false};
      int c;
      el_terms<MODE>(e[k], a[k], b[k], c);
      cnt += c;
    }
    smin = lane_tree<C>(a);
    smax = lane_tree<C>(b);
  }
  RowStat st;
  st.minact = group_sum<G>(smin);
  st.maxact = group_sum<G>(smax);
  cnt = group_sum_int<G>(cnt);
  st.nmin = cnt_min(cnt);
  st.nmax = cnt_max(cnt);
  int L = cnt_act(cnt);
  if (MODE == MODE_COMPACT) {
    const int row = __shfl(row_of, from, PSL_WAVE);
    if (vr && gl == 0) {
      d.row_out[row].v0 = st.minact;
      d.row_out[row].j = on ? L : 0;
    }
    return 0;
  }
  const double lhs = on ? in.lhs : 0.0, rhs = on ? in.rhs : 0.0;
  bool tiny = false;
#pragma unroll
  for (int k = 0; k < C; ++k) tiny = tiny || (el_active(e[k]) && fabs(e[k].a) < d.cfg.coef_tol);
  bool any_tiny = (__ballot(tiny) & group_mask<G>()) != 0;
  RowDec dec = decide_row(d.cfg, lhs, rhs, L, st.nmin, st.nmax, st.minact, st.maxact, any_tiny);
  bool prop = on && dec.prop;
  bool uncap = false, mine = false;
  int aj = 0;
  double aa = 0.0;
  int force = on ? dec.force : 0;
  if (C == 1) lane_prop<C>(d, sk, s0 + gl * C, prop, e, lhs, rhs, st, dec.single, force, uncap, mine, aj, aa);
  else  // reload (L1/L2 hits) instead of keeping C elements live through the sums
    lane_prop_stream<C>(d, sk, prop, s0, len, gl * C, lhs, rhs, st, dec.single, force, uncap, mine, aj, aa);
  bool captured = (__ballot(uncap) & group_mask<G>()) == 0;
  uint8_t code = RC_KEEP;
  if (on) {
    code = dec.code;
    if (prop && dec.single && !dec.infeasible && captured) code = RC_SINGLETON;
  }
  if (__ballot(code != RC_KEEP || (on && dec.infeasible)) != 0) {
    // a row of the wavefront leaves, or cannot be met
    const Dev& cd = cold_dev();
    const int row = __shfl(row_of, from, PSL_WAVE);
    if (on && dec.infeasible && gl == 0) flag_infeasible(cd, row_lp_of(cd, row));
    if (on && gl == 0 && (code == RC_EMPTY || code == RC_REDUNDANT || is_forcing(code)))
      cd.row_out[row] = row_out_of(code, st);
    if (code == RC_SINGLETON && mine) {
      cd.row_out[row] = RowOut{aa, 0.0, aj, 0};
      drop_col(cd, aj, aa, lhs, rhs);
    }
    if (code == RC_REDUNDANT || is_forcing(code)) {
      if (C == 1) lane_drop<C>(cd, e, lhs, rhs);
      else lane_drop_stream<C>(cd, on, s0, len, gl * C, lhs, rhs);
    }
  }
  return RowRes::pack(code, st.nmin, st.nmax);
}

// rows and nonzeros that are swept (direct lists), of rows held one by a lane
template <int MODE, bool DIR>
__device__ __forceinline__ void count_swept(const RoundArgs& ra, bool on, int len) {
  if (MODE != MODE_ROUND || !DIR) return;
  unsigned long long m = __ballot(on);
  int z = group_sum_int<PSL_WAVE>(on ? len : 0);
  if (lane_id() == 0 && m) {
    atomicAdd(ra.rows, (int)__popcll(m));
    atomicAdd(ra.nnz, z);
  }
}

// The workgroup's REP row blocks of a bin with one position per lane: a
// wavefront takes REP * 64 / G consecutive rows of the list. One lane reads a
// row's entry, sides and flags and stores its outcome, for all blocks with one
// load or store each, and the lanes of the row's group take them from it: the
// vector memory unit needs 17 cycles for any 8- or 16-byte load of a wavefront
// (37 where the lanes' lines differ, as the bounds'), also where four or more
// lanes read one row's, and it was 80% busy when each block made its own. The
// positions' loads of all blocks are issued, level by level, before any block
// is processed, so a lane has REP rows' gathers in flight together.
template <int G, int MODE, int REP, bool DIR>
__device__ __forceinline__ void sweep_rows(const Dev& d, const CandSink& sk, RoundArgs ra, bool over, int bin,
                                           int lblock) {
  constexpr int RW = PSL_WAVE / G, NR = REP * RW;  // rows of a block's wavefront; of all blocks'
  static_assert(NR <= PSL_WAVE, "one row per lane");
  const int cap = d.bin_off[bin + 1] - d.bin_off[bin];
  const int lane = lane_id(), gl = lane & (G - 1);
  const int first = (lblock * (PSL_BLOCK / PSL_WAVE) + (int)(threadIdx.x >> 6)) * NR;
  const BinEnt be = row_entry(d, bin, cap, first + (lane < NR ? lane : NR - 1));
  const int count = DIR ? cap : d.sel[bin].v;
  hold(be.row);
  if (over || first >= count) return;  // uniform over the wavefront
  RowOf r;
  row_take(be, lane < NR && first + lane < count, r);
  int j[REP];
  double a[REP];
#pragma unroll
  for (int k = 0; k < REP; ++k) {
    const int from = k * RW + lane / G;
    const int s0 = __shfl(r.start, from, PSL_WAVE), len = __shfl(r.len, from, PSL_WAVE);
    const int64_t p = gl < len ? (int64_t)s0 + gl : 0;
    j[k] = d.ci[p];
    a[k] = d.va[p];
  }
  row_data<MODE, DIR>(d, ra, r);
  const unsigned long long on = __ballot(r.on);
  double2 bb[REP];
#pragma unroll
  for (int k = 0; k < REP; ++k) {
    bb[k] = make_double2(0.0, 0.0);
    if (!DIR || (on >> (k * RW + lane / G) & 1)) bb[k] = d.bnd[j[k]];
  }
  count_swept<MODE, DIR>(ra, r.on, r.len);
  uint32_t res = 0;
#pragma unroll
  for (int k = 0; k < REP; ++k) {
    if (first + k * RW >= count) break;  // uniform over the wavefront
    if (DIR && MODE == MODE_ROUND && ((on >> (k * RW)) & (RW == 64 ? ~0ull : (1ull << RW) - 1)) == 0) continue;
    const int from = k * RW + lane / G;
    RowIn<1> in;
    in.on = (on >> from) & 1;
    in.s0 = __shfl(r.start, from, PSL_WAVE);
    in.len = __shfl(r.len, from, PSL_WAVE);
    in.lhs = __shfl(r.lhs, from, PSL_WAVE);
    in.rhs = __shfl(r.rhs, from, PSL_WAVE);
    const bool v = gl < in.len;
    in.e[0] = El{v ? j[k] : 0, v ? a[k] : 0.0, v ? bb[k].x : 0.0, v ? bb[k].y : 0.0, v};
    const bool vr = first + from < count;
    const uint32_t w = row_block<G, 1, MODE>(d, sk, in, vr, r.row, from);
    const uint32_t x = __shfl(w, (lane & (RW - 1)) * G, PSL_WAVE);
    if (lane / RW == k) res = x;
  }
  if (MODE == MODE_ROUND && r.on) row_store(d, r.row, res);
}

// one row of a wavefront at a time, C positions per lane
template <int C, int MODE, bool DIR>
__device__ __forceinline__ void sweep_wide_row(const Dev& d, const CandSink& sk, RoundArgs ra, bool over, int bin,
                                               int lblock) {
  const int cap = d.bin_off[bin + 1] - d.bin_off[bin];
  const int lane = lane_id();
  const int gid = lblock * (PSL_BLOCK / PSL_WAVE) + (int)(threadIdx.x >> 6);
  const int count = DIR ? cap : d.sel[bin].v;
  if (over || gid >= count) return;  // uniform over the wavefront
  RowOf r;
  row_take(row_entry(d, bin, cap, gid), true, r);
  row_data<MODE, DIR>(d, ra, r);
  if (DIR && MODE == MODE_ROUND && !r.on) return;
  count_swept<MODE, DIR>(ra, r.on && lane == 0, r.len);
  RowIn<C> in;
  in.on = r.on;
  in.s0 = r.start;
  in.len = r.len;
  in.lhs = r.lhs;
  in.rhs = r.rhs;
  load_els<C>(d, in.s0, in.len, lane * C, true, in.e);
  const uint32_t w = row_block<PSL_WAVE, C, MODE>(d, sk, in, true, r.row, lane);
  if (MODE == MODE_ROUND && r.on && lane == 0) row_store(d, r.row, w);
}

// ---------------------------------------------------------------------------
// long rows: workgroup passes of 2048 positions (8 contiguous per thread)
// ---------------------------------------------------------------------------

// sums of one pass: (w0 + w1) + (w2 + w3) over the wavefront butterflies
template <int MODE>
__device__ __forceinline__ void pass_stats(const Dev& d, int64_t s0, int len, int base, El (&e)[8], double* wl,
                                           int* il, double& psmin, double& psmax, int& nmin, int& nmax, int& L) {
  double a, b;
  int c;
  lane_stats<8, MODE>(d, s0, len, base + (int)threadIdx.x * 8, e, a, b, c);
  a = group_sum<PSL_WAVE>(a);
  b = group_sum<PSL_WAVE>(b);
  c = group_sum_int<PSL_WAVE>(c);
  int w = threadIdx.x >> 6;
  if (lane_id() == 0) {
    wl[w] = a;
    wl[4 + w] = b;
    il[w] = c;
  }
  __syncthreads();
  psmin = (wl[0] + wl[1]) + (wl[2] + wl[3]);
  psmax = (wl[4] + wl[5]) + (wl[6] + wl[7]);
  nmin = nmax = L = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    nmin += cnt_min(il[k]);
    nmax += cnt_max(il[k]);
    L += cnt_act(il[k]);
  }
  __syncthreads();
}

// Is long row `row` (active) swept this round, from the direct lists? Every
// workgroup of the row's chunks takes the same answer: the counts its inert
// test reads are rewritten by the sweep with the values they have, and the
// LP's state is the one at the round's start.
__device__ __forceinline__ bool long_swept(const Dev& d, int row, RoundSeq rs) {
  int mode = rs.full ? 0 : d.flags->mode;
  return (!(mode & 1) || d.dirty[row] == round_mark(rs.seq)) && row_lp_swept(d, row) &&
         (!(mode & 2) || !row_inert(d.rinf[row], d.lhs[row], d.rhs[row]));
}

// partial statistics of one chunk (its passes combined in tree order)
template <int MODE>
__global__ void __launch_bounds__(PSL_BLOCK) k_long_stats(Dev d, RoundSeq rs) {
  if (MODE == MODE_ROUND) {
    if (round_over(d, rs.seq)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) d.flags->stamp[0] = wall_clock64();
  }
  if ((int)blockIdx.x >= chunks_listed(d)) return;
  __shared__ double ps[2 * LONG_MAX_PASSES];
  __shared__ double wl[8];
  __shared__ int il[4];
  LongChunk ch = d.lchunk[blockIdx.x];
  int row = ch.row;
  if (!d.row_on[row]) return;
  if (MODE == MODE_ROUND && d.direct && !long_swept(d, row, rs)) return;
  int64_t s0 = d.rp[row];
  int len = d.rp[row + 1] - (int)s0;
  int tmin = 0, tmax = 0, tl = 0;
  int np = ch.npass;
  bool tiny = false;  // an active entry with |a| < coef_tol (forcing rows)
  for (int p = 0; p < np; ++p) {
    El e[8];
    double a, b;
    int x, y, z;
    pass_stats<MODE>(d, s0, len, ch.first + p * PASS_LEN, e, wl, il, a, b, x, y, z);
    if (threadIdx.x == 0) {
      ps[p] = a;
      ps[LONG_MAX_PASSES + p] = b;
    }
    tmin += x;
    tmax += y;
    tl += z;
#pragma unroll
    for (int k = 0; k < 8; ++k) tiny = tiny || (el_active(e[k]) && fabs(e[k].a) < d.cfg.coef_tol);
  }
  int any_tiny = __syncthreads_or(tiny ? 1 : 0);
  if (threadIdx.x == 0) {
    LongPart pt;
    pt.smin = tree_inplace(ps, np);
    pt.smax = tree_inplace(ps + LONG_MAX_PASSES, np);
    pt.nmin = tmin;
    pt.nmax = tmax;
    pt.L = tl;
    pt.tiny = any_tiny ? 1 : 0;
    d.lpart[ch.id] = pt;
  }
}

// row totals from the chunk partials: one wavefront, 8 chunks per lane
__device__ __forceinline__ void long_totals(const Dev& d, const LongRow& lr, RowStat& st, int& L, int& tiny) {
  double a[8], b[8];
  int n0 = 0, n1 = 0, n2 = 0, n3 = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    int c = lane_id() * 8 + k;
    a[k] = b[k] = 0.0;
    if (c < lr.nchunk) {
      LongPart pt = d.lpart[lr.chunk0 + c];
      a[k] = pt.smin;
      b[k] = pt.smax;
      n0 += pt.nmin;
      n1 += pt.nmax;
      n2 += pt.L;
      n3 += pt.tiny;
    }
  }
  st.minact = group_sum<PSL_WAVE>(lane_tree<8>(a));
  st.maxact = group_sum<PSL_WAVE>(lane_tree<8>(b));
  st.nmin = group_sum_int<PSL_WAVE>(n0);
  st.nmax = group_sum_int<PSL_WAVE>(n1);
  L = group_sum_int<PSL_WAVE>(n2);
  tiny = group_sum_int<PSL_WAVE>(n3);
}

// decisions and propagation over one chunk of a long row
__device__ __forceinline__ void sweep_long_chunk(const Dev& d, const CandSink& sk, const RoundArgs& ra, RoundSeq rs,
                                                 int chunk, double* lds) {
  LongChunk ch = d.lchunk[chunk];
  int row = ch.row;
  if (!d.row_on[row]) {
    if (ch.first == 0 && threadIdx.x == 0) d.row_code[row] = RC_KEEP;
    return;
  }
  LongRow lr = d.lrow[ch.lrow];
  if (d.direct) {
    if (!long_swept(d, row, rs)) return;
    if (ch.first == 0 && threadIdx.x == 0) {
      atomicAdd(ra.rows, 1);
      atomicAdd(ra.nnz, d.rp[row + 1] - d.rp[row]);
    }
  }
  int* li = (int*)(lds + 2);
  if (threadIdx.x < PSL_WAVE) {
    RowStat st;
    int L, tiny;
    long_totals(d, lr, st, L, tiny);
    if (threadIdx.x == 0) {
      lds[0] = st.minact;
      lds[1] = st.maxact;
      li[0] = st.nmin;
      li[1] = st.nmax;
      li[2] = L;
      li[3] = tiny;
    }
  }
  __syncthreads();
  RowStat st;
  st.minact = lds[0];
  st.maxact = lds[1];
  st.nmin = li[0];
  st.nmax = li[1];
  int L = li[2];
  int64_t s0 = d.rp[row];
  int len = d.rp[row + 1] - (int)s0;
  double lhs = d.lhs[row], rhs = d.rhs[row];
  RowDec dec = decide_row(d.cfg, lhs, rhs, L, st.nmin, st.nmax, st.minact, st.maxact, li[3] != 0);
  if (ch.first == 0 && threadIdx.x == 0) d.rinf[row] = make_int2(st.nmin, st.nmax);
  bool uncap = false, mine = false;
  int aj = 0;
  double aa = 0.0;
  for (int p = 0; p < ch.npass; ++p) {
    int base = ch.first + p * PASS_LEN + (int)threadIdx.x * 8;
    if (dec.prop)
      lane_prop_stream<8>(d, sk, true, s0, len, base, lhs, rhs, st, dec.single, dec.force, uncap, mine, aj, aa);
    if (dec.code == RC_REDUNDANT || is_forcing(dec.code)) lane_drop_stream<8>(d, true, s0, len, base, lhs, rhs);
  }
  if (dec.prop && dec.single && !dec.infeasible) {
    // the one active entry decides whether its row becomes bounds
    if (mine) {
      if (!uncap) {
        d.row_code[row] = RC_SINGLETON;
        d.row_out[row] = RowOut{aa, 0.0, aj, 0};
        drop_col(d, aj, aa, lhs, rhs);
      } else {
        d.row_code[row] = RC_KEEP;
      }
    }
  } else if (ch.first == 0 && threadIdx.x == 0) {
    d.row_code[row] = dec.code;
    if (dec.infeasible) flag_infeasible(d, row_lp_of(d, row));
    if (dec.code == RC_EMPTY || dec.code == RC_REDUNDANT || is_forcing(dec.code))
      d.row_out[row] = row_out_of(dec.code, st);
  }
}

__device__ __forceinline__ int long_first_block(const SweepGrid& g) {
  int b = 0;
  for (int k = 0; k < BIN_LONG; ++k) b += g.nb[k];
  return b;
}

// Three launches per sweep, by register need: (0) 4/8/16/64-lane group bins
// with one position per lane, (1) wavefront bins with 4 or 8 positions per
// lane, (2) long-row chunks. Workgroups keep one global numbering across the
// launches (candidate regions and counts are indexed by it).
enum { KIND_SHORT = 0, KIND_WIDE = 1, KIND_LONG = 2, KIND_ALL = 3 };

template <int MODE, int KIND, bool DIR>
__global__ void __launch_bounds__(PSL_BLOCK) k_sweep(Dev d, SweepGrid g, int base, RoundSeq rs) {
  __shared__ double lds[8];
  __shared__ int32_t lcount, lrows, lnnz;
  if (threadIdx.x == 0) lcount = lrows = lnnz = 0;
  __syncthreads();
  const bool over = MODE == MODE_ROUND && round_over(d, rs.seq);
  RoundArgs ra{0, 0, &lrows, &lnnz};
  if (MODE == MODE_ROUND) {
    ra.mode = rs.full ? 0 : d.flags->mode;
    ra.mark = round_mark(rs.seq);
  }
  int gb = blockIdx.x + base;  // global workgroup number
  if (MODE == MODE_ROUND && gb == 0 && threadIdx.x == 0 && !over) {
    unsigned long long t = wall_clock64();
    d.flags->stamp[1] = t;
    if (g.nb[BIN_LONG] == 0) d.flags->stamp[0] = t;
  }
  int b = gb;
  int bin;
  int64_t start = cand_region_start(g, b, bin);
  int lfb = long_first_block(g);
  if (MODE == MODE_ROUND && (KIND == KIND_LONG || KIND == KIND_ALL) && gb >= lfb) {
    // a chunk of a long row
    int chunk = gb - lfb;
    if (!over && chunk < chunks_listed(d)) {
      CandSink sk{d.cand + g.long_base + (int64_t)d.lchunk[chunk].cand_off, &lcount};
      sweep_long_chunk(d, sk, ra, rs, chunk, lds);
    }
  } else {
    CandSink sk{d.cand + start, &lcount};
    if (KIND != KIND_WIDE && b < g.nb[BIN_G4]) {
      sweep_rows<4, MODE, DIR ? 1 : 4, DIR>(d, sk, ra, over, BIN_G4, b);
    } else if (KIND != KIND_WIDE && (b -= g.nb[BIN_G4]) < g.nb[BIN_G8]) {
      sweep_rows<8, MODE, DIR ? 1 : 4, DIR>(d, sk, ra, over, BIN_G8, b);
    } else if (KIND != KIND_WIDE && (b -= g.nb[BIN_G8]) < g.nb[BIN_G16]) {
      sweep_rows<16, MODE, DIR ? 1 : 4, DIR>(d, sk, ra, over, BIN_G16, b);
    } else if (KIND != KIND_WIDE && (b -= g.nb[BIN_G16]) < g.nb[BIN_W1]) {
      sweep_rows<64, MODE, DIR ? 1 : 2, DIR>(d, sk, ra, over, BIN_W1, b);
    } else if (KIND != KIND_SHORT) {
      b -= KIND == KIND_WIDE ? g.nb[BIN_G4] + g.nb[BIN_G8] + g.nb[BIN_G16] + g.nb[BIN_W1] : g.nb[BIN_W1];
      if (b < g.nb[BIN_W4]) sweep_wide_row<4, MODE, DIR>(d, sk, ra, over, BIN_W4, b);
      else sweep_wide_row<8, MODE, DIR>(d, sk, ra, over, BIN_W8, b - g.nb[BIN_W4]);
    }
  }
  if (MODE == MODE_ROUND && !over) {
    __syncthreads();
    if (threadIdx.x == 0) {
      d.cand_cnt[gb] = lcount;
      if (DIR && lrows) {
        atomicAdd(&d.flags->swept[gb % SWEPT_SLOTS].rows, (unsigned long long)lrows);
        atomicAdd(&d.flags->swept[gb % SWEPT_SLOTS].nnz, (unsigned long long)lnnz);
      }
    }
  }
}

// compaction: a long row's constant and active length from its partials
__global__ void __launch_bounds__(PSL_BLOCK) k_long_finish_compact(Dev d) {
  int k = blockIdx.x * (PSL_BLOCK / PSL_WAVE) + (threadIdx.x >> 6);
  if (k >= d.nlong) return;
  LongRow lr = d.lrow[k];
  bool on = d.row_on[lr.row] != 0;
  RowStat st;
  int L = 0;
  int tiny = 0;
  if (on) long_totals(d, lr, st, L, tiny);
  else st.minact = 0.0;
  if (lane_id() == 0) {
    d.row_out[lr.row].v0 = st.minact;
    d.row_out[lr.row].j = on ? L : 0;
  }
}

// ---------------------------------------------------------------------------
// source rows of the final bounds
// ---------------------------------------------------------------------------
// the candidate region of sweep workgroup b
__device__ __forceinline__ void sources(const Dev& d, const SweepGrid& g, int b) {
  int n = d.cand_cnt[b];
  if (n == 0) return;
  int bin;
  int64_t start = cand_region_start(g, b, bin);
  if (start < 0) start = g.long_base + (int64_t)d.lchunk[b - long_first_block(g)].cand_off;
  const Cand* list = d.cand + start;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    Cand c = list[i];
    const long long k = d.bkey[c.js];
    if (c.t == (c.js & 1 ? unukey(k) : dunkey(k))) atomicMin(&d.src[c.js], c.pos);
  }
}

// ---------------------------------------------------------------------------
// decisions per column, record counts per row and column
// ---------------------------------------------------------------------------
__device__ __forceinline__ double empty_value(double c, double lo, double up) {
  if (c > 0) return lo;
  if (c < 0) return up;
  return lo > 0 ? lo : (up < 0 ? up : 0.0);
}

// decision of an active or removed column from the round's accumulators:
// code bits, and the number of records it gives
// Dual fixing (a lock-based dual reduction): when no alive row keeps column
// j from moving towards the bound its cost prefers (c > 0: down, c < 0: up;
// c = 0: either, with a finite bound, lower first), some optimal solution has
// it there; an infinite such bound means the LP is unbounded if feasible.
// Returns true with the value (possibly infinite) and side (0 lower, 1 upper).
__device__ __forceinline__ bool dual_fix_of(double c, double lo, double up, unsigned long long locks, double& v,
                                            int& side) {
  bool free_down = (locks & 0xFFFFFFFFull) == 0, free_up = (locks >> 32) == 0;
  side = 0;
  v = lo;
  if (c > 0) return free_down;
  side = 1;
  v = up;
  if (c < 0) return free_up;
  if (free_down && !is_inf(lo)) {
    side = 0;
    v = lo;
    return true;
  }
  return free_up && !is_inf(up);
}

__device__ __forceinline__ uint8_t col_decide(const Dev& d, int j, int& k) {
  k = 0;
  double2 b = d.bnd[j];
  longlong2 key = *reinterpret_cast<const longlong2*>(&d.bkey[2 * (int64_t)j]);
  int left = d.col_len[j];
  hold(left);
  if (b.x == b.y) return 0;
  double lo = dunkey(key.x);
  double up = unukey(key.y);
  uint8_t code = 0;
  if (lo != b.x) {
    code |= CC_LB;
    ++k;
  }
  if (up != b.y) {
    code |= CC_UB;
    ++k;
  }
  bool fin = !is_inf(lo) && !is_inf(up);
  bool lfin = !is_inf(lo), ufin = !is_inf(up);  // the new bounds
  if (fin && lo > up + tol_of(d.cfg, up)) code |= CC_INFEAS;
  if (fin && up - lo <= d.cfg.fix_tol * mx1(lo)) {
    code |= CC_FIX;
    ++k;
  } else if (left == 0) {
    double v = empty_value(d.c[j], lo, up);
    if (is_inf(v)) {
      code |= CC_UNBOUNDED;
    } else {
      code |= CC_EMPTY;
      lfin = ufin = true;
      ++k;
    }
  } else if (d.cfg.dual_fix) {
    double v;
    int side;
    if (dual_fix_of(d.c[j], lo, up, d.locks[j], v, side)) {
      if (is_inf(v)) {
        code |= CC_UNBOUNDED;
      } else {
        code |= CC_DUALFIX;
        lfin = ufin = true;
        ++k;
      }
    }
  }
  // bounds that become finite lower the infinite-contribution counts of the
  // column's rows (applied by the marks)
  if (is_inf(b.x) && lfin) code |= CC_LBFIN;
  if (is_inf(b.y) && ufin) code |= CC_UBFIN;
  if (code & CC_INFEAS) flag_infeasible(d, col_lp_of(d, j));
  if (code & CC_UNBOUNDED) flag_unbounded(d, col_lp_of(d, j));
  return code;
}

// Decision tiles: the rows in tiles of DEC_TILE, then the columns in tiles of
// DEC_TILE (index order, so the records keep the order rows, then columns).
// A lane loads the codes of DEC_ITEMS consecutive indices as one word (the
// arrays are 256-byte aligned and padded, so a word starting below the end
// stays inside them); the indices with work (touched columns, indices with
// records) are then compacted per wavefront in LDS and dealt out to its lanes,
// so the lanes stay busy whether few or all indices have work, and a tile
// costs four wavefronts instead of one per 64 indices.
#define DEC_ITEMS 4
#define DEC_BLOCK 256
#define DEC_TILE (DEC_BLOCK * DEC_ITEMS)
#define DEC_WAVES (DEC_BLOCK / PSL_WAVE)
#define DEC_WAVE_ITEMS (PSL_WAVE * DEC_ITEMS)
// an index has at most 3 records (a row 1; a column: each bound side and one
// of fixed, empty or dual-fixed), so a lane's count fits in 4 bits
static_assert(3 * DEC_ITEMS < 16, "record counts per lane must fit in 4 bits");
static_assert(DEC_BLOCK == PSL_BLOCK, "block scans");
static_assert(DEC_ITEMS == 4, "a lane's codes are one 32-bit word");

// prefix (lanes below) and total of per-lane counts 0..15 across the
// wavefront, from one ballot per bit
__device__ __forceinline__ void wave_small_scan(int v, int& pre, int& tot) {
  unsigned long long below = (1ull << lane_id()) - 1ull;
  unsigned long long b0 = __ballot(v & 1), b1 = __ballot(v & 2), b2 = __ballot(v & 4), b3 = __ballot(v & 8);
  pre = __popcll(b0 & below) + 2 * __popcll(b1 & below) + 4 * __popcll(b2 & below) + 8 * __popcll(b3 & below);
  tot = __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2) + 8 * __popcll(b3);
}

// bytes of a lane's word that hold indices below the end (rem of them)
__device__ __forceinline__ uint32_t valid_bytes(int64_t rem) {
  return rem >= 4 ? 0xFFFFFFFFu : (1u << (8 * (int)rem)) - 1u;
}

// the codes' word of a lane: 4 consecutive indices from i0 (a multiple of 4)
__device__ __forceinline__ uint32_t code_word(const uint8_t* a, int64_t i0) {
  return reinterpret_cast<const uint32_t*>(a)[i0 >> 2];
}

// records of a column with decision code `code`
__device__ __forceinline__ int col_recs(uint32_t code) {
  return (code & CC_LB ? 1 : 0) + (code & CC_UB ? 1 : 0) + (code & (CC_FIX | CC_EMPTY) ? 1 : 0);
}

// The tiles' record counts are summed per 64 tiles with atomic adds whose
// results are awaited, so that the workgroup that finishes the last tile sees
// every sum without a fence: it scans the few sums of 64 (a tile's offset is
// then one of them plus at most 63 tile counts) and sets the next round's mode.
// Column tiles start at a multiple of 64, so the rows removed are the records
// before the first of them.
#define SUPER 64

static int64_t row_supers(int64_t m) { return ((m + DEC_TILE - 1) / DEC_TILE + SUPER - 1) / SUPER; }

// tiles, with the row tiles filled up to a multiple of SUPER; at least one
// column tile (the last workgroup's work is done in any case)
int64_t decide_tiles(int64_t m, int64_t n) {
  int64_t ct = (n + DEC_TILE - 1) / DEC_TILE;
  return SUPER * row_supers(m) + (ct > 0 ? ct : 1);
}

size_t decide_supers(int64_t m, int64_t n) { return (size_t)((decide_tiles(m, n) + SUPER - 1) / SUPER + 1); }

struct TileGrid {
  int nsrc;       // workgroups of the sweep (their candidate regions come first)
  int row_tiles;  // tiles of rows
  int col0;       // first column tile (a multiple of SUPER)
  int tiles;      // col0 + the column tiles
};

// the next round's selection mode from this round's totals
__device__ __forceinline__ int round_mode(const Dev& d, const RoundMode& rm, int changed, int fin_cols) {
  bool incr = rm.allow && (int64_t)changed * rm.incr_factor < (int64_t)d.n;
  bool counts = (int64_t)fin_cols * rm.count_factor < (int64_t)d.n;
  return (incr ? 1 : 0) | (counts ? 2 : 0);
}

// fields of a word of the sums
#define SUP_REC(v) ((int)((v) & 0xFFFFFFull))
#define SUP_FIN(v) ((int)((v) >> 24 & 0xFFFFFull))
#define SUP_TILES(v) ((int)((v) >> 44))
static_assert(3ull * DEC_TILE * SUPER < (1ull << 24), "records of 64 tiles");

// the sums of 64 tiles scanned, the round's totals, the next mode (one
// workgroup)
__device__ __forceinline__ void decide_totals(const Dev& d, const TileGrid& tg, const RoundMode& rm) {
  int ns = (tg.tiles + SUPER - 1) / SUPER, rs = tg.col0 / SUPER;
  int run = 0, fin = 0, removed = 0;
  for (int k0 = 0; k0 < ns; k0 += DEC_BLOCK) {
    int k = k0 + (int)threadIdx.x;
    unsigned long long v = 0;
    if (k < ns) {
      v = __hip_atomic_load(&d.super[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      atomicExch(&d.super[k], 0ull);
    }
    int c = SUP_REC(v), f = SUP_FIN(v), tot, ftot, rtot;
    int pre = block_excl_scan(c, &tot);
    if (k < ns) d.super_off[k] = run + pre;
    block_excl_scan(f, &ftot);
    block_excl_scan(k < rs ? c : 0, &rtot);
    run += tot;
    fin += ftot;
    removed += rtot;
  }
  if (threadIdx.x == 0) {
    *d.super_done = 0;
    Flags& F = *d.flags;
    F.round_total = run;
    F.rows_removed = removed;
    F.fin_cols = fin;
    F.mode = round_mode(d, rm, run - removed, fin);
    F.rec_base = F.rec_at;
    if (!d.direct) {
      int64_t rows = 0, nnz = d.sel[SEL_NNZ].v;
#pragma unroll
      for (int b = 0; b < NBINS; ++b) rows += d.sel[b].v;
      F.sum_rows += rows;
      F.sum_nnz += nnz;
      F.sum_cols += nnz < d.n ? nnz : d.n;
    }
  }
}

// Sources of the final bounds, and beside them the column decisions of the
// touched columns (untouched ones cannot change: an active column with
// unchanged bounds and rows is neither fixed nor empty), and the record count
// of each tile.
__global__ void __launch_bounds__(DEC_BLOCK) k_decide(Dev d, SweepGrid g, TileGrid tg, RoundMode rm, int seq,
                                                      int32_t* tile_sum) {
  const bool over = round_over(d, seq);
  if (blockIdx.x == 0 && threadIdx.x == 0 && !over) {
    unsigned long long t = wall_clock64();
    d.flags->stamp[2] = t;
    if (tg.nsrc == 0) d.flags->stamp[0] = d.flags->stamp[1] = t;  // no row to sweep
  }
  if ((int)blockIdx.x < tg.nsrc) {
    if (!over) sources(d, g, blockIdx.x);
    return;
  }
  __shared__ int list[DEC_TILE];
  __shared__ int wtot[DEC_WAVES], wfin[DEC_WAVES];
  __shared__ int last;
  int w = threadIdx.x >> 6, lane = lane_id();
  int* wl = list + w * DEC_WAVE_ITEMS;
  int t = (int)blockIdx.x - tg.nsrc;
  const bool rows = t < tg.row_tiles;
  const int tile = rows ? t : tg.col0 + (t - tg.row_tiles);
  const int64_t i0 = (int64_t)(rows ? tile : tile - tg.col0) * DEC_TILE + (int64_t)threadIdx.x * DEC_ITEMS;
  const int64_t lim = rows ? d.m : d.n;
  uint32_t traw = 0, cw = 0, vm = 0;  // touched, codes
  if (i0 < lim) {
    vm = valid_bytes(lim - i0);
    cw = code_word(rows ? d.row_code : d.col_code, i0) & vm;
    if (!rows) traw = code_word(d.touch, i0);
  }
  hold(cw);
  hold(traw);
  if (over) return;
  int c = 0, nt = 0, ntot = 0, fin = 0;
  if (rows) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (((cw >> (8 * b)) & 0xFFu) != RC_KEEP) {
        ++c;
        if (d.K > 1) d.lpo[d.row_lp[i0 + b]].total = 1;  // the LP changes this round
      }
  } else {
    uint32_t tw = traw & vm;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      bool touched = ((tw >> (8 * b)) & 0xFFu) != 0;
      nt += touched;
      // a code left from an earlier round of an untouched column
      if (!touched && ((cw >> (8 * b)) & 0xFFu)) d.col_code[i0 + b] = 0;
    }
    if (tw) reinterpret_cast<uint32_t*>(d.touch)[i0 >> 2] = traw & ~vm;
    // the touched columns of the wavefront, in LDS, dealt out to its lanes
    int pre;
    wave_small_scan(nt, pre, ntot);
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if ((tw >> (8 * b)) & 0xFFu) wl[pre++] = (int)(i0 + b);
  }
  __syncthreads();
  for (int e = lane; e < ntot; e += PSL_WAVE) {
    int j = wl[e];
    int kk;
    uint8_t code = col_decide(d, j, kk);
    d.col_code[j] = code;
    c += kk;
    fin += (code & (CC_LBFIN | CC_UBFIN)) != 0;
    if (kk && d.K > 1) d.lpo[d.col_lp[j]].total = 1;
  }
  // the tile's counts: wavefront totals by ballots, summed by thread 0
  int pre_w, tot_w, fin_w;
  wave_small_scan(c, pre_w, tot_w);
  wave_small_scan(fin, pre_w, fin_w);
  if (lane == 0) {
    wtot[w] = tot_w;
    wfin[w] = fin_w;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0, ftot = 0;
#pragma unroll
    for (int k = 0; k < DEC_WAVES; ++k) {
      tot += wtot[k];
      ftot += wfin[k];
    }
    tile_sum[tile] = tot;
    int sp = tile / SUPER;
    int end = rows ? tg.row_tiles : tg.tiles;  // tiles of this 64 that exist
    int members = (end < (sp + 1) * SUPER ? end : (sp + 1) * SUPER) - sp * SUPER;
    last = 0;
    // the second add is issued once the first has returned
    unsigned long long o =
        atomicAdd(&d.super[sp], (unsigned long long)tot | ((unsigned long long)ftot << 24) | (1ull << 44));
    if (SUP_TILES(o) == members - 1) last = atomicAdd(d.super_done, 1) == (tg.tiles + SUPER - 1) / SUPER - 1;
  }
  __syncthreads();
  if (last) decide_totals(d, tg, rm);
}

__device__ __forceinline__ Record mkrec(uint8_t type, uint8_t side, int round, int i, int j, int k, double v0,
                                        double v1, double v2, double v3) {
  Record r;
  r.type = type;
  r.side = side;
  r.round = (uint16_t)round;
  r.i = i;
  r.j = j;
  r.k = k;
  r.v[0] = v0;
  r.v[1] = v1;
  r.v[2] = v2;
  r.v[3] = v3;
  return r;
}

__device__ __forceinline__ void emit_row(const Dev& d, int i, int round, Record* r) {
  uint8_t code = d.row_code[i];
  RowOut o = d.row_out[i];
  if (code == RC_EMPTY) *r = mkrec(REC_EMPTY_ROW, 0, round, i, -1, -1, o.v0, d.lhs[i], d.rhs[i], 0.0);
  else if (code == RC_REDUNDANT) *r = mkrec(REC_REDUNDANT_ROW, 0, round, i, -1, -1, o.v0, o.v1, d.lhs[i], d.rhs[i]);
  else if (is_forcing(code))
    *r = mkrec(REC_FORCING_ROW, code == RC_FORCE_MAX ? 1 : 0, round, i, -1, -1, o.v0, d.lhs[i], d.rhs[i], 0.0);
  else *r = mkrec(REC_SINGLETON_ROW, 0, round, i, o.j, -1, o.v0, d.lhs[i], d.rhs[i], 0.0);
  d.row_on[i] = 0;
  d.row_code[i] = RC_KEEP;
}

// the records and new state of a column with decision code `code`
__device__ __forceinline__ void emit_col(const Dev& d, int j, uint8_t code, int round, Record* r) {
  double2 b = d.bnd[j];
  double lo = dunkey(d.bkey[2 * (int64_t)j]);
  double up = unukey(d.bkey[2 * (int64_t)j + 1]);
  // the source of a changed bound is the CSR position of the lowest row's
  // candidate equal to it (positions of one column ascend with the row); a
  // changed bound always has one
  if (code & CC_LB) {
    int q = d.src[2 * (int64_t)j];
    bool ok = q >= 0 && q < d.nnz;
    int k = ok ? d.rowid1[q + 1] : -1;
    *r++ = mkrec(REC_BOUND_CHANGE, 0, round, -1, j, k, b.x, lo, ok ? d.va[q] : __builtin_nan(""), 0.0);
    if (d.cfg.free_sing) {
      int ls = d.lsrc[j];
      d.lsrc[j] = ls == -1 || ls == k ? k : -2;  // a bound from one row only keeps it implied by that row
    }
  }
  if (code & CC_UB) {
    int q = d.src[2 * (int64_t)j + 1];
    bool ok = q >= 0 && q < d.nnz;
    int k = ok ? d.rowid1[q + 1] : -1;
    *r++ = mkrec(REC_BOUND_CHANGE, 1, round, -1, j, k, b.y, up, ok ? d.va[q] : __builtin_nan(""), 0.0);
    if (d.cfg.free_sing) {
      int us = d.usrc[j];
      d.usrc[j] = us == -1 || us == k ? k : -2;
    }
  }
  double nlo = lo, nup = up;
  if ((code & CC_DUALFIX) == CC_DUALFIX) {
    // the locks have not changed since the decision
    double v;
    int side;
    dual_fix_of(d.c[j], lo, up, d.locks[j], v, side);
    *r++ = mkrec(REC_DUAL_FIX, (uint8_t)side, round, -1, j, -1, v, d.c[j], 0.0, 0.0);
    nlo = nup = v;
  } else if (code & CC_FIX) {
    *r++ = mkrec(REC_FIX_COL, 0, round, -1, j, -1, lo, d.c[j], 0.0, 0.0);
    nlo = nup = lo;
  } else if (code & CC_EMPTY) {
    double v = empty_value(d.c[j], lo, up);
    *r++ = mkrec(REC_EMPTY_COL, 0, round, -1, j, -1, v, d.c[j], 0.0, 0.0);
    nlo = nup = v;
  }
  d.bnd[j] = make_double2(nlo, nup);
  d.bkey[2 * (int64_t)j] = dkey(nlo);
  d.bkey[2 * (int64_t)j + 1] = ukey(nup);
  d.src[2 * (int64_t)j] = 0x7FFFFFFF;
  d.src[2 * (int64_t)j + 1] = 0x7FFFFFFF;
}

// ---------------------------------------------------------------------------
// marks for the next round
// ---------------------------------------------------------------------------
// Rows of the columns whose bounds changed (or that were fixed) this round,
// from the transposed copy; their infinite-contribution counts follow the
// bounds that became finite. The wavefront that emitted its columns' records
// walks their entries; columns of more than MARK_DENSE entries (listed once at
// ingest) are walked by every workgroup of a second launch.
#define MARK_SHORT 16
#define MARK_MASK (CC_LB | CC_UB | CC_FIX)

// One entry (q, row i) of a changed column: mark the row (when the next
// round sweeps dirty rows only), and (with count) lower its infinite-
// contribution counts when the column's lb / ub became finite.
__device__ __forceinline__ void mark_entry(const Dev& d, int64_t q, int code, bool mark, bool count, uint8_t with) {
  int i = d.ri[q];
  if (mark) {
    d.dirty[i] = with;
    if (!d.direct) d.dirty_tile[i >> 10] = with;
  }
  if (count && (code & (CC_LBFIN | CC_UBFIN))) {
    bool pos = d.cva[q] > 0;
    bool lbf = (code & CC_LBFIN) != 0, ubf = (code & CC_UBFIN) != 0;
    if ((lbf && pos) || (ubf && !pos)) atomicSub(&d.rinf[i].x, 1);  // min contribution now finite
    if ((lbf && !pos) || (ubf && pos)) atomicSub(&d.rinf[i].y, 1);  // max contribution now finite
  }
}

// columns the marking pass walks: changed ones when rows are marked, those
// with a bound that became finite when counts are kept
__device__ __forceinline__ bool mark_col(int code, int mode) {
  return ((mode & 1) && (code & MARK_MASK)) || ((mode & 2) && (code & (CC_LBFIN | CC_UBFIN)));
}

// exclusive prefix (lanes below) and total of per-lane values 0..31 across
// the wavefront, from one ballot per bit
__device__ __forceinline__ void wave_scan5(int v, int& pre, int& tot) {
  unsigned long long below = lanemask_lt();
  pre = tot = 0;
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    unsigned long long m = __ballot((v >> b) & 1);
    pre += __popcll(m & below) << b;
    tot += __popcll(m) << b;
  }
}

// marks of the wavefront's columns wl[0 .. n) (any of them with records)
__device__ __forceinline__ void mark_cols(const Dev& d, const int* wl, int n, int mode, uint8_t with) {
  int lane = lane_id();
  for (int c0 = 0; c0 < n; c0 += PSL_WAVE) {
    int q0 = 0, q1 = 0, code = 0;
    if (c0 + lane < n) {
      int j = wl[c0 + lane];
      code = d.col_code[j];
      if (mark_col(code, mode)) {
        q0 = d.cp[j];
        q1 = d.cp[j + 1];
      }
    }
    int len = q1 - q0;
    // short columns: the entries of the lanes' columns, concatenated in
    // column order, one per lane (a column's entries are contiguous, so the
    // row-index loads of a step touch a few lines, and no lane walks a
    // column alone)
    int sl = len <= MARK_SHORT ? len : 0;
    int pre, tot;
    wave_scan5(sl, pre, tot);
    for (int e0 = 0; e0 < tot; e0 += PSL_WAVE) {
      int e = e0 + lane;
      // the entry's column: the last lane whose prefix is <= e
      int lo = 0, hi = PSL_WAVE - 1;
#pragma unroll
      for (int it = 0; it < 6; ++it) {
        int mid = (lo + hi + 1) >> 1;
        bool le = __shfl(pre, mid, PSL_WAVE) <= e;
        lo = le ? mid : lo;
        hi = le ? hi : mid - 1;
      }
      int q = __shfl(q0, lo, PSL_WAVE) + (e - __shfl(pre, lo, PSL_WAVE));
      int cl = __shfl(code, lo, PSL_WAVE);
      if (e < tot) mark_entry(d, q, cl, mode & 1, mode & 2, with);
    }
    // longer ones: the wavefront walks them one after another
    unsigned long long mask = __ballot(len > MARK_SHORT && len <= MARK_DENSE);
    while (mask) {
      int l = __ffsll((long long)mask) - 1;
      mask &= mask - 1;
      int a = __shfl(q0, l, PSL_WAVE), b = __shfl(q1, l, PSL_WAVE), cl = __shfl(code, l, PSL_WAVE);
      for (int q = a + lane; q < b; q += PSL_WAVE) mark_entry(d, q, cl, mode & 1, mode & 2, with);
    }
  }
}

// every workgroup lists the changed dense columns (in slices of 1024, checked
// in parallel) and walks a grid-strided share of their entries
__global__ void __launch_bounds__(PSL_BLOCK) k_mark_dense(Dev d, int seq) {
  __shared__ int32_t list[1024];
  __shared__ int32_t cnt;
  if (round_over(d, seq)) return;
  int mode = d.flags->mode;
  const uint8_t with = round_mark(seq + 1);
  if (mode == 0) return;
  int nd = *d.n_dense;
  for (int k0 = 0; k0 < nd; k0 += 1024) {
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    for (int k = k0 + threadIdx.x; k < nd && k < k0 + 1024; k += PSL_BLOCK) {
      int j = d.dense_cols[k];
      if (mark_col(d.col_code[j], mode)) list[atomicAdd(&cnt, 1)] = j;
    }
    __syncthreads();
    int nc = cnt;
    for (int c = 0; c < nc; ++c) {
      int j = list[c];
      int code = d.col_code[j];
      int64_t q1 = d.cp[j + 1];
      for (int64_t q = d.cp[j] + (int64_t)blockIdx.x * PSL_BLOCK + threadIdx.x; q < q1;
           q += (int64_t)gridDim.x * PSL_BLOCK)
        mark_entry(d, q, code, mode & 1, mode & 2, with);
    }
    __syncthreads();
  }
}

// The round's control (one workgroup; sweep.h, RoundCtl). d.lp_round: the
// number of the LP's running round while it propagates, minus its last one once
// it does not.
// A round that is not run only hands the numbers on.
// The one workgroup goes over all LPs, so a thread has the loads of CTL_LPS of them
// in flight together (one after another, 200000 LPs of one row took 16.7 ms a pass;
// 15.5 so).
#define CTL_LPS 8
__device__ __forceinline__ void round_control(const Dev& d, const RoundCtl& ctl, bool over, int seq) {
  __shared__ int go_on;
  Flags& f = *d.flags;
  if (over) {
    if (d.K > 1)
      for (int k0 = threadIdx.x; k0 < d.K; k0 += CTL_LPS * blockDim.x) {
        int r[CTL_LPS];
#pragma unroll
        for (int q = 0; q < CTL_LPS; ++q) r[q] = d.lp_round[k0 + q * (int)blockDim.x < d.K ? k0 + q * (int)blockDim.x : k0];
#pragma unroll
        for (int q = 0; q < CTL_LPS; ++q)
          if (k0 + q * (int)blockDim.x < d.K) d.lp_round_next[k0 + q * (int)blockDim.x] = r[q];
      }
    return;
  }
  if (threadIdx.x == 0) go_on = d.K == 1 && !f.infeasible && !f.unbounded && f.round_total != 0;
  __syncthreads();
  if (d.K > 1) {
    bool any = false;
    for (int k0 = threadIdx.x; k0 < d.K; k0 += CTL_LPS * blockDim.x) {
      int r[CTL_LPS], total[CTL_LPS];
      LpFlags f[CTL_LPS];
      uint8_t ok[CTL_LPS];
#pragma unroll
      for (int q = 0; q < CTL_LPS; ++q) {
        const int k = k0 + q * (int)blockDim.x < d.K ? k0 + q * (int)blockDim.x : k0;
        r[q] = d.lp_round[k];
        f[q] = d.lpf[k];
        total[q] = d.lpo[k].total;
        ok[q] = d.lp_ok[k];
      }
#pragma unroll
      for (int q = 0; q < CTL_LPS; ++q) {
        const int k = k0 + q * (int)blockDim.x;
        if (k >= d.K) break;
        if (r[q] > 0) {
          const bool more = !f[q].infeasible && !f[q].unbounded && total[q] != 0;
          d.lpo[k].total = 0;
          r[q] = more ? r[q] + 1 : -r[q];
          any = any || more;
        }
        d.lp_round_next[k] = r[q];
        d.lp_run[k] = ok[q];
      }
    }
    if (any) go_on = 1;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (d.direct) {
    int64_t rows = 0, nnz = 0;
    for (int k = 0; k < SWEPT_SLOTS; ++k) {
      rows += f.swept[k].rows;
      nnz += f.swept[k].nnz;
    }
    int64_t z = nnz - f.sum_nnz;
    f.sum_cols += z < d.n ? z : d.n;
    f.sum_rows = rows;
    f.sum_nnz = nnz;
  }
  f.rounds_done += 1;
  f.rec_at = f.rec_base + f.round_total;
  unsigned long long now = wall_clock64();
  f.ticks[0] += f.stamp[1] - f.stamp[0];
  f.ticks[1] += f.stamp[2] - f.stamp[1];
  f.ticks[2] += now - f.stamp[2];
  if (!go_on || (!ctl.last && f.rec_at + ctl.need > f.rec_cap)) f.stop_at = seq;
}

// Rounds with free singletons: the control after them (the first workgroup), and
// the picks of the long rows they took (the chunks listed), all of whose chunks
// are done.
__global__ void __launch_bounds__(PSL_BLOCK) k_round_control(Dev d, RoundCtl ctl, const int32_t* list, int seq) {
  const bool over = round_over(d, seq);
  const int nc = over || d.flags->fs_picks != seq ? 0 : d.flags->fs_rows;
  for (int k = blockIdx.x * PSL_BLOCK + threadIdx.x; k < nc; k += gridDim.x * PSL_BLOCK) {
    int p0 = list[k];
    int i = d.rowid1[p0 + 1];
    if (p0 == d.rp[i]) d.fs_pick[i] = 0x7FFFFFFF;  // the row's first chunk
  }
  if (blockIdx.x == 0) round_control(d, ctl, over, seq);
}

// Records of the round in index order: a tile's offset is the sum of the tiles
// before its 64 (scanned) and of the tiles before it among them; the position
// of an index's records inside the tile comes from the counts of the indices
// before it (ballots inside the wavefront, the wavefronts' totals through LDS).
// The indices with records are compacted per wavefront and dealt out to its
// lanes, each writing its index's records at that position; a wavefront of
// columns then marks their rows for the next round. The last workgroup is the
// round's control. Also clears the next selection's counts.
__global__ void __launch_bounds__(DEC_BLOCK) k_decide_emit(Dev d, const int32_t* tile_sum, TileGrid tg, RoundCtl ctl,
                                                           int round, int seq) {
  const bool over = round_over(d, seq);
  const bool rows = (int)blockIdx.x < tg.row_tiles;
  const int tile = rows ? (int)blockIdx.x : tg.col0 + ((int)blockIdx.x - tg.row_tiles);
  if (tile == tg.tiles) {
    if (ctl.by_emit) round_control(d, ctl, over, seq);
    return;
  }
  if (!over && !d.direct && blockIdx.x == 0 && threadIdx.x < SEL_N) d.flags->sel[1][threadIdx.x].v = 0;
  __shared__ int list[DEC_TILE], lpos[DEC_TILE];
  __shared__ int wtot[DEC_WAVES];
  int w = threadIdx.x >> 6, lane = lane_id();
  // one level of loads: the tile's count, the codes, the tile's offset
  const int tsum = tile_sum[tile];
  const int mode = d.flags->mode;
  const int64_t t0 = (int64_t)(rows ? tile : tile - tg.col0) * DEC_TILE + (int64_t)threadIdx.x * DEC_ITEMS;
  const int64_t lim = rows ? d.m : d.n;
  uint32_t cw = 0;
  if (t0 < lim) cw = code_word(rows ? d.row_code : d.col_code, t0) & valid_bytes(lim - t0);
  int before = lane < (tile & (SUPER - 1)) ? tile_sum[(tile & ~(SUPER - 1)) + lane] : 0;
  const int64_t base = d.flags->rec_base + d.super_off[tile / SUPER];
  hold(cw);
  hold(before);
  hold(base);
  if (over || tsum == 0) return;  // a tile without records
  uint32_t cnt4 = 0;  // the records of the lane's 4 indices, a byte each
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    uint32_t code = (cw >> (8 * b)) & 0xFFu;
    cnt4 |= (uint32_t)(rows ? code != RC_KEEP : col_recs(code)) << (8 * b);
  }
  int c = 0, ni = 0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    int k = (cnt4 >> (8 * b)) & 0xFF;
    c += k;
    ni += k != 0;
  }
  int pre, tot_w, ipre, itot;
  wave_small_scan(c, pre, tot_w);
  wave_small_scan(ni, ipre, itot);
  if (lane == 0) wtot[w] = tot_w;
  before = group_sum_int<PSL_WAVE>(before);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < DEC_WAVES; ++k) pre += k < w ? wtot[k] : 0;
  int* wl = list + w * DEC_WAVE_ITEMS;
  int* wp = lpos + w * DEC_WAVE_ITEMS;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    int k = (cnt4 >> (8 * b)) & 0xFF;
    if (k) {
      wl[ipre] = (int)(t0 + b);
      wp[ipre] = pre;
      ++ipre;
      pre += k;
    }
  }
  __syncthreads();
  Record* r0 = d.rec + base + before;
  for (int e = lane; e < itot; e += PSL_WAVE) {
    int x = wl[e];
    Record* r = r0 + wp[e];
    if (rows) emit_row(d, x, round_of(d, row_lp_of(d, x), round), r);
    else emit_col(d, x, d.col_code[x], round_of(d, col_lp_of(d, x), round), r);
  }
  if (!rows && mode != 0) mark_cols(d, wl, itot, mode, round_mark(seq + 1));
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void launch_long_stats(const Dev& d, int mode, int chunks, RoundSeq rs, hipStream_t s) {
  if (chunks == 0) return;
  if (mode == MODE_ROUND) hipLaunchKernelGGL(k_long_stats<MODE_ROUND>, dim3(chunks), dim3(PSL_BLOCK), 0, s, d, rs);
  else hipLaunchKernelGGL(k_long_stats<MODE_COMPACT>, dim3(chunks), dim3(PSL_BLOCK), 0, s, d, rs);
}

template <int MODE, bool DIR>
static void sweep_launches(const Dev& d, const SweepGrid& g, bool split, RoundSeq rs, hipStream_t s) {
  int n_short = g.nb[BIN_G4] + g.nb[BIN_G8] + g.nb[BIN_G16] + g.nb[BIN_W1];
  int n_wide = g.nb[BIN_W4] + g.nb[BIN_W8];
  int n_long = MODE == MODE_ROUND ? g.nb[BIN_LONG] : 0;
  dim3 blk(PSL_BLOCK);
  // Without wide and long rows the short kind's kernel alone: it holds none of
  // their code, and its pointers stay in scalar registers (a presolve of 523 rows
  // 1.28 ms with the kernel of all kinds, 1.24 with this; 31337 rows 1.06 and
  // 1.04; a 4096-LP batch 71.4 and 70.6). With such rows they run beside each other.
  if (!split && n_wide + n_long > 0) {
    int total = n_short + n_wide + n_long;
    if (total) hipLaunchKernelGGL((k_sweep<MODE, KIND_ALL, DIR>), dim3(total), blk, 0, s, d, g, 0, rs);
    return;
  }
  if (n_short) hipLaunchKernelGGL((k_sweep<MODE, KIND_SHORT, DIR>), dim3(n_short), blk, 0, s, d, g, 0, rs);
  if (n_wide) hipLaunchKernelGGL((k_sweep<MODE, KIND_WIDE, DIR>), dim3(n_wide), blk, 0, s, d, g, n_short, rs);
  if (n_long)
    hipLaunchKernelGGL((k_sweep<MODE, KIND_LONG, DIR>), dim3(n_long), blk, 0, s, d, g, n_short + n_wide, rs);
}

void launch_sweep(const Dev& d, const SweepGrid& g, int mode, RoundSeq rs, hipStream_t s) {
  if (mode == MODE_COMPACT) {
    if (d.direct) sweep_launches<MODE_COMPACT, true>(d, g, true, rs, s);
    else sweep_launches<MODE_COMPACT, false>(d, g, true, rs, s);
    if (d.nlong > 0)
      hipLaunchKernelGGL(k_long_finish_compact, dim3((d.nlong + 3) / 4), dim3(PSL_BLOCK), 0, s, d);
  } else {
    if (d.direct) sweep_launches<MODE_ROUND, true>(d, g, mode == 2, rs, s);
    else sweep_launches<MODE_ROUND, false>(d, g, mode == 2, rs, s);
  }
}

// every long row's removed-column constant and active length (row_out), from
// the compaction-mode chunk partials
void launch_long_consts(const Dev& d, hipStream_t s) {
  if (d.nlong == 0) return;
  launch_long_stats(d, MODE_COMPACT, d.nchunks, RoundSeq{0, 1}, s);
  hipLaunchKernelGGL(k_long_finish_compact, dim3((d.nlong + 3) / 4), dim3(PSL_BLOCK), 0, s, d);
}

// the round's sources, decisions, records and marks; the record total goes to
// d.flags->round_total
void launch_decide(const Dev& d, const SweepGrid& g, const RoundMode& rm, const RoundCtl& ctl, bool dense, int round,
                   int seq, int32_t* tile_sum, hipStream_t s) {
  TileGrid tg;
  tg.nsrc = 0;
  for (int b = 0; b < NBINS; ++b) tg.nsrc += g.nb[b];
  tg.row_tiles = (int)(((int64_t)d.m + DEC_TILE - 1) / DEC_TILE);
  tg.col0 = (int)(SUPER * row_supers(d.m));
  tg.tiles = (int)decide_tiles(d.m, d.n);
  int nt = tg.row_tiles + tg.tiles - tg.col0;
  hipLaunchKernelGGL(k_decide, dim3((unsigned)(tg.nsrc + nt)), dim3(DEC_BLOCK), 0, s, d, g, tg, rm, seq, tile_sum);
  hipLaunchKernelGGL(k_decide_emit, dim3((unsigned)(nt + 1)), dim3(DEC_BLOCK), 0, s, d, (const int32_t*)tile_sum, tg,
                     ctl, round, seq);
  if (dense) hipLaunchKernelGGL(k_mark_dense, dim3(512), dim3(PSL_BLOCK), 0, s, d, seq);
}

void launch_control(const Dev& d, const RoundCtl& ctl, const int32_t* fs_list, int seq, hipStream_t s) {
  hipLaunchKernelGGL(k_round_control, dim3(32), dim3(PSL_BLOCK), 0, s, d, ctl, fs_list, seq);
}

int long_max_passes() { return LONG_MAX_PASSES; }

}  // namespace psl
