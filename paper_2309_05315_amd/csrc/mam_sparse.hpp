// Device code of the iterations between the first and the last of a call
// (short columns): plans kept as -b plus their few active entries.
//
// Step 2 of Alg. 1 writes theta'_rs = pi_hat_rs - b^(m)_r, and pi_hat is 0 at
// every inactive entry, so between two iterations a plan column is the
// vector nbv_m = (T)(-b^(m)), common to its measure, except at its patches:
// the active rows, with their stored values.  Inside one call only the
// patches are kept; the bound theta is read by the first iteration (the
// column kernel's SPARSE form) and written back once, when the call returns
// (sparse_write_kernel).  Values are the ones the dense kernels store, and
// the threshold's sums take the column kernel's order, so the iterates are
// the dense path's bit for bit.
//
// Finding the active entries without reading R rows.  An unpatched entry has
//   w_r = base_r - c_r / rho,  base_r = nbv_r + 2 b_r  (per measure).
// With lambda_C the threshold of Prop. 3 of a set C of entries, adding
// entries only raises it: rows outside C whose w is at most lambda_C are
// inactive, and if that is every row then lambda_C is the column's
// threshold.  Two upper bounds of w settle that:
//
//  * In time, one lane per column.  C = the patches (the last active set).
//    V = the largest w outside C when the column was last looked at; since
//    then each w of the measure rose by at most the sum of the iterations'
//    largest rises of base (drift G_m, kept by the close kernel), so
//    V + (G_now - G_then) bounds them all.  (Every sum G is rounded up, so a
//    call of any length keeps the bound; a margin of 2^-46 of the magnitudes
//    covers the rounding at the two ends.)
//    Base moves slowly, so few columns per iteration are looked at again: 11 to
//    14% in the first 20 iterations of a solve, then 0.6 to 1.4% on the 64x64
//    workload and up to 5% on smaller grids.
//  * In space, 16 lanes per open column, four columns per wave.  Over a block
//    of 64 rows w <= max base - min c / rho, by the same fused multiply-add as
//    w itself, so rounding (monotone) keeps the bound exact.  Blocks whose
//    bound exceeds lambda_C are evaluated, rows above lambda_C join C, and
//    the rest gives the new V.  Blocks a little below lambda_C (16 times the
//    last drift) are evaluated too: a V taken from their bound would open the
//    column again at once.  The minima of every cost column are taken once
//    per call (cost_min_kernel), the maxima of base by the close kernel.
//  * A column with more than kPatch candidates, or with an entry at its
//    threshold (kTie), is taken by a whole wave over all its rows, in the
//    column kernel's rounds from its stored threshold, and stored dense in
//    theta while it has more than kPatch active entries (count -1).
//
// What bounds it: a column costs some 40 bytes (q, V, count, one patch, a
// cost and a b) where a dense iteration streams R rows of theta twice and of
// the cost once, so the kernel is a chain of three dependent memory accesses
// (tile, column, cost and b at the patch; two more for an open column) and
// not bandwidth: its waves wait for 72% of their cycles on the 64x64 workload
// (10.9 us), 66% on 256 problems (54 us), and the close kernel's for 64% and 70%.
#pragma once

#include "mam_kernels.hpp"

namespace mam {

static_assert(kPatch == 16, "one patch per lane of a 16-lane group");
constexpr int kBlkRows = 64;    // rows per block of the bounds
constexpr int kSparseMaxM = 96;   // measures the close kernel holds in LDS (1.5 KiB each in FP64)

// One problem as the sparse iterations see it.
template <typename T>
struct SpProb {
  T* theta;
  const T* cost;
  const T* q;
  const int32_t* cidx;
  unsigned long long* acc;  // M x R fixed-point sums of pi_hat (zero between iterations)
  const double* fx;         // M scales 2^E_m, then M inverse scales
  int64_t ld, cost_ld;
  int64_t tcols;            // columns (stride of the patch slots)
  int32_t R, Rp;            // rows; rows padded to kBlkRows (stride of nbv and eb)
  int32_t cost_mode, nblk, nblkp;  // blocks; padded to 4 (stride of cmin, dblk and drift)
  int32_t relaxed, balanced;  // balanced: gamma = inf, t = 1
  int32_t ntl, vecl, vpt;   // column kernel's shape: log2 threads, log2 vector width, values per thread
  int32_t M, vec_cost, vec_theta;  // vec_*: 16-byte accesses allowed
  int32_t ncost;            // cost columns
  double rho, inv_rho, gamma;
  double* pm;               // M x R
  double* pm_prev;
  double* p;                // R
  double* p_prev;
  const double* aw;
  const double* Sd;
  double* d2w;              // partial sums of d^2 over 64 rows
  double* d2part;           // partial sums of d^2 over 256 rows (the dense kernels')
  double* lam;
  double* t_out;            // t of the last iteration, then (finite gamma) of the next
  const int64_t* col_off;
  T* nbv;                   // M x Rp, (T)(-b) of the last iteration
  double* eb;               // M x Rp, b of the next iteration
  double* bb;               // M x Rp, base of the next iteration
  double* dblk;             // M x nblkp, largest base of each block
  double* drift;            // 2 x M x nblkp, largest rise of base in each block, by parity
  double* G;                // M, sum of the rises before the current one
  int32_t* par;             // parity of the current rise: [1] for the column kernel, which copies it to [0]
                            // for the close kernel, which sets [1] (no kernel reads a word that it writes)
  T* cmin;                  // ncost x nblkp, least cost of each block
  int32_t* cnt;             // patches of each column, -1 = stored dense in theta
  int32_t* prow;            // kPatch x tcols
  T* pval;                  // kPatch x tcols
  double* vg;               // largest w outside a column's patches, less the drift then (inf: not known)
  int32_t* wide;            // one per plan: what the write-back of the call has noted (sparse_write_kernel)
};

struct SpTile {
  int32_t prob, m, j0;
  int32_t n;  // columns; bit 16: the problem's first tile of the launch
};

struct SpRows {
  int32_t prob, blk;
};

struct SpCost {
  int32_t prob, c0, n, pad;
};

template <typename T>
struct SpArgs {
  const SpProb<T>* probs;
  const SpTile* tiles;
  int32_t ntiles;
  const int32_t* stop;
  uint8_t* rec;     // as ColArgs::rec; the words are zero before the launch
  int64_t rec_ld;
};

// Tables written by the host before the launch and never by a kernel: read
// through the constant address space, so uniform entries take scalar loads.
template <typename U>
using ConstPtr = const __attribute__((address_space(4))) U*;
template <typename U>
__device__ __forceinline__ ConstPtr<U> cptr(const U* p) {
  return (ConstPtr<U>)(uint64_t)p;
}

// A measure's rises so far plus the next one, no less than the exact sum: the
// rise is a rounded difference, and the sum is rounded too (late in a run
// rises are below half an ulp of G, and rounded to nearest they would all be
// lost).  The kernels that form it use this one expression.
__device__ __forceinline__ double drift_sum(double g, double rise) {
  const double s = g + (rise + fabs(rise) * 0x1p-40);
  return s + fabs(s) * 0x1p-52;
}

// Maxima of results of arithmetic: one instruction each (max_arith).
struct OpMaxA {
  static constexpr double id() { return -__builtin_huge_val(); }
  __device__ static double f(double a, double b) { return max_arith(a, b); }
};

template <class Op>
__device__ __forceinline__ double row16_reduce(double v) {
  v = Op::f(v, dpp_move<0xb1, 0xf>(v, Op::id()));
  v = Op::f(v, dpp_move<0x4e, 0xf>(v, Op::id()));
  v = Op::f(v, dpp_move<0x141, 0xf>(v, Op::id()));
  v = Op::f(v, dpp_move<0x140, 0xf>(v, Op::id()));
  return v;
}

// A lane's four consecutive rows of a cost column, rows past the end as
// +inf (their w is -inf).  Vector accesses stay inside the column: its
// stride is a multiple of the vector there.
template <typename T>
__device__ __forceinline__ void load_cost4(const T* __restrict__ col, int r0, int R, bool vec, T (&c)[4]) {
  if (vec) {
    if constexpr (sizeof(T) == 4) {
      if (r0 < R) load_vec<T, 4>(col + r0, c);
    } else {
      T a[2] = {}, b[2] = {};
      if (r0 < R) load_vec<T, 2>(col + r0, a);
      if (r0 + 2 < R) load_vec<T, 2>(col + r0 + 2, b);
      c[0] = a[0];
      c[1] = a[1];
      c[2] = b[0];
      c[3] = b[1];
    }
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (r0 + v < R) c[v] = col[r0 + v];
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (r0 + v >= R) c[v] = (T)__builtin_huge_val();
}

template <typename T>
__device__ __forceinline__ void load_row4(const T* __restrict__ p, T (&x)[4]) {
  if constexpr (sizeof(T) == 4) {
    load_vec<T, 4>(p, x);
  } else {
    T a[2], b[2];
    load_vec<T, 2>(p, a);
    load_vec<T, 2>(p + 2, b);
    x[0] = a[0];
    x[1] = a[1];
    x[2] = b[0];
    x[3] = b[1];
  }
}

// Least cost of every block of 64 rows, per cost column: 16 lanes per block,
// one wave per column.  Once per call (the cost may have been rebuilt in
// place between two calls): one read of the cost.
template <typename T>
__global__ void __launch_bounds__(256)
cost_min_kernel(const SpProb<T>* __restrict__ probs, const SpCost* __restrict__ tasks, const int32_t* __restrict__ stop) {
  if (stop != nullptr && *stop != 0) return;
  const SpCost tk = tasks[blockIdx.x];
  const ConstPtr<SpProb<T>> P = cptr(probs) + uniform_i(tk.prob);
  if (blockIdx.x == 0 && threadIdx.x == 0) *gptr(P->wide) = 0;
  const int lane = threadIdx.x & 63, l = lane & 15, g = lane >> 4;
  const int wv = uniform_i((int)(threadIdx.x >> 6));
  const int R = P->R, nblk = P->nblk;
  const bool vec = P->vec_cost != 0;
  for (int i = wv; i < tk.n; i += 4) {
    const int64_t cc = uniform_i(tk.c0) + i;
    const T* const col = gptr(P->cost) + cc * P->cost_ld;
    T* const cm = gptr(P->cmin) + cc * P->nblkp;
    for (int b0 = 0; b0 < nblk; b0 += 16) {
      T c[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) load_cost4<T>(col, (b0 + u * 4 + g) * kBlkRows + l * 4, R, vec, c[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int blk = b0 + u * 4 + g;
        const double v = row16_reduce<OpMin>(fmin(fmin((double)c[u][0], (double)c[u][1]),
                                                  fmin((double)c[u][2], (double)c[u][3])));
        if (l == 0 && blk < nblk) cm[blk] = (T)v;
      }
    }
  }
}

// t^k from the partial sums over 64 rows, added as the close kernels of the
// dense path add them (four waves of a 256-row block in order, then the
// blocks by a wave reduction).
__device__ __forceinline__ double damping_t64(const double* d2w, int nblk, double rho, double gam, int lane) {
  double d2 = 0.0;
  if (lane * 4 < nblk) {
    d2 = d2w[lane * 4];
#pragma unroll
    for (int k = 1; k < 4; ++k) d2 += lane * 4 + k < nblk ? d2w[lane * 4 + k] : 0.0;
  }
  d2 = wave_reduce<OpSum>(d2);
  return (__builtin_isinf(gam) || rho * sqrt(d2) <= gam) ? 1.0 : gam / (rho * sqrt(d2));
}

// Active-set bit of row r in the record of column j.
__device__ __forceinline__ void set_mask_bit(uint8_t* rec, int64_t rec_ld, int64_t j, int r, int ntl, int vecl,
                                             int vpt) {
  const int v = r & ((1 << vecl) - 1), q = r >> vecl;
  const int tid = q & ((1 << ntl) - 1), k = ((q >> ntl) << vecl) + v;
  const int byte = vpt <= 8 ? tid : tid * 2 + (k >> 3);
  unsigned* const w = reinterpret_cast<unsigned*>(gptr(rec) + j * rec_ld + (byte & ~3));
  atomicOr(w, 1u << (((byte & 3) << 3) + (k & 7)));
}

// S = (x + y) + z or x + (y + z) for three active entries of a column,
// whichever the column kernel's reduction takes: entries of one thread by row,
// then the lanes of a wave as a binary tree over the lane number, then the
// waves in turn.
__device__ __forceinline__ double sum3(double w0, int r0, double w1, int r1, double w2, int r2, int ntl, int vecl) {
  const int msk = (1 << ntl) - 1;
  int k0 = (((r0 >> vecl) & msk) << 13) | r0, k1 = (((r1 >> vecl) & msk) << 13) | r1,
      k2 = (((r2 >> vecl) & msk) << 13) | r2;
  auto order = [](int& ka, double& wa, int& kb, double& wb) {
    const bool s = kb < ka;
    const int k = s ? ka : kb;
    const double w = s ? wa : wb;
    ka = s ? kb : ka;
    wa = s ? wb : wa;
    kb = k;
    wb = w;
  };
  order(k0, w0, k1, w1);
  order(k1, w1, k2, w2);
  order(k0, w0, k1, w1);
  const int x = (k0 >> 13) ^ (k1 >> 13), y = (k1 >> 13) ^ (k2 >> 13);
  const bool right = (y >> 6) == 0 && ((x >> 6) != 0 || x > y);
  return right ? w0 + (w1 + w2) : (w0 + w1) + w2;
}

__device__ __forceinline__ double shfl_d(double v, int src) {
  return __hiloint2double(__shfl(__double2hiint(v), src), __shfl(__double2loint(v), src));
}

// Entries at the threshold.  With w_r = lambda within rounding the set that a
// threshold is formed over is not unique: the column kernel's depends on the
// round that settled the column, and with it the last bit of lambda (and the
// recorded set).  On data of few binary digits (integer costs, equal weights)
// such bits decide where mass goes, so these columns are left to the whole
// wave, which repeats the column kernel's rounds.  Everywhere else the set is
// unique and its sum, taken in the column kernel's order, gives the same bits.
// The margin covers the rounding of a sum of kPatch entries within tau of
// lambda.  The largest entry is always in the set, unless lambda = w_max - tau
// rounds to w_max; it is 0 then either way, and it is in the recorded set only
// if the float bounds of the column kernel's certificate hold with equality.
constexpr double kTie = 0x1p-46;
template <bool REC>
__device__ __forceinline__ bool top_unsure(double top, double lam) {
  return REC && top == lam && (double)(float)top == top;
}

// Entries of a thread that a whole wave takes at a time (a thread of the
// column kernel holds up to 16; 8 keep the kernel at 128 registers, four
// waves per SIMD).
constexpr int kWholeRows = 8;

template <typename T, bool REC>
__global__ void __launch_bounds__(256, 4)
sparse_column_kernel(SpArgs<T> a) {
  __shared__ double s_w[4][64], s_b[4][64], s_pw[4][3][64], s_pb[4][3][64], s_pl[4][64];
  __shared__ int s_r[4][64], s_pr[4][3][64];

  const int wv = uniform_i((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int wid = blockIdx.x * 4 + wv;
  const int stopv = a.stop != nullptr ? *gptr(a.stop) : 0;
  if (wid >= a.ntiles) return;
  const ConstPtr<SpTile> tk = cptr(a.tiles) + wid;
  const ConstPtr<SpProb<T>> P = cptr(a.probs) + tk->prob;
  const int m = tk->m, n = tk->n & 0xffff;
  const bool first = (tk->n >> 16) != 0;
  const int64_t j0 = tk->j0;
  if (uniform_i(stopv) != 0) return;

  const int R = P->R, nblk = P->nblk, nblkp = P->nblkp, cost_mode = P->cost_mode;
  const int ntl = P->ntl, vecl = P->vecl;
  const int64_t tc = P->tcols, cost_ld = P->cost_ld;
  const double inv_rho = P->inv_rho;
  const bool relaxed = P->relaxed != 0;
  const T* const cost = gptr(P->cost);
  const T* const qv = gptr(P->q);
  const double* const eb = gptr(P->eb) + (int64_t)m * P->Rp;
  const T* const nbv = gptr(P->nbv) + (int64_t)m * P->Rp;
  const double* const dblk = gptr(P->dblk) + (int64_t)m * nblkp;
  int32_t* const cntv = gptr(P->cnt);
  int32_t* const prow = gptr(P->prow);
  T* const pval = gptr(P->pval);
  double* const vgv = gptr(P->vg);
  double* const lamv = gptr(P->lam);
  unsigned long long* const acc = gptr(P->acc) + (int64_t)m * R;
  const double fxm = gptr(P->fx)[m];
  const int64_t off_m = cost_mode == MAM_COST_SHARED ? cptr(P->col_off)[m] : 0;

  // ---- one lane per column ----
  const bool have = lane < n;
  const int64_t j = j0 + (have ? lane : 0);
  const int par = uniform_i(gptr(P->par)[1]);
  const int64_t cc = cost_mode == MAM_COST_INDEXED ? (int64_t)gptr(P->cidx)[j] : j - off_m;
  const double tau = (double)qv[j];
  const int cnt = have ? cntv[j] : 0;
  const double vg = vgv[j];
  constexpr int NL = 3;  // patches a lane takes
  int row[NL];
  double val[NL];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    row[k] = prow[k * tc + j];
    val[k] = (double)pval[k * tc + j];
  }
  row[2] = 0;
  val[2] = 0.0;
  // the drift up to this iteration (rounded up)
  const double* const dr = gptr(P->drift) + ((int64_t)par * P->M + m) * nblkp;
  double delta = lane < nblk ? dr[lane] : -__builtin_huge_val();
  if (lane + 64 < nblk) delta = max_arith(delta, dr[lane + 64]);
  const double G0 = gptr(P->G)[m];
  if (first && lane == 0) {
    gptr(P->par)[0] = par;
    gptr(P->t_out)[0] = P->balanced ? 1.0 : gptr(P->t_out)[1];
  }
  if (__ballot(cnt > 2) != 0ull) {
    row[2] = prow[2 * tc + j];
    val[2] = (double)pval[2 * tc + j];
  }
  const bool lanes_take = cnt >= 1 && cnt <= NL;
  const T* const ccol = cost + cc * cost_ld;
  double b[NL], w[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    b[k] = 0.0;
    w[k] = -__builtin_huge_val();
    if (__ballot(lanes_take && cnt > k) != 0ull) {
      const bool on = lanes_take && cnt > k;
      if (!on) row[k] = 0;
      const double c = (double)ccol[row[k]];
      b[k] = eb[row[k]];
      if (on) w[k] = __builtin_fma(-c, inv_rho, val[k] + 2.0 * b[k]);
    }
  }
  delta = wave_reduce<OpMaxA>(delta);
  const double G = drift_sum(G0, delta);
  // threshold of the patches alone
  double hi = max_arith(w[0], w[1]), mid = fmin(w[0], w[1]);
  const double lo2 = fmin(hi, w[2]);
  hi = max_arith(hi, w[2]);
  const double lo = fmin(mid, lo2);
  mid = max_arith(mid, lo2);
  double lam = hi - tau;
  if (mid > lam) {
    lam = (hi + mid - tau) / 2.0;
    if (lo > lam) lam = (sum3(w[0], row[0], w[1], row[1], w[2], row[2], ntl, vecl) - tau) / 3.0;
  }
  const double lout = relaxed ? max_arith(lam, 0.0) : lam;
  const double eps = (fabs(lam) + tau) * kTie;
  const bool tie = fabs(mid - lam) <= eps || fabs(lo - lam) <= eps || top_unsure<REC>(hi, lam);
  const bool ok = lanes_take && !tie && vg + G + ((fabs(vg) + fabs(G)) * kTie + eps) <= lout;
  unsigned long long open = __ballot(have && cnt != 0 && !ok);
  if (have && ok) {
    bool in[NL];
    int na = 0;
    double nv[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      in[k] = w[k] > lout;
      na += in[k] ? 1 : 0;
      nv[k] = -b[k];
      if (in[k]) {
        const double ph = max_arith(w[k] - lout, 0.0);
        nv[k] = ph - b[k];
        atomicAdd(acc + row[k], to_fixed(ph, fxm));
        if constexpr (REC) set_mask_bit(a.rec, a.rec_ld, j, row[k], ntl, vecl, P->vpt);
      }
    }
    lamv[j] = lam;
    if (na == cnt) {
      pval[j] = (T)nv[0];
      if (cnt > 1) pval[tc + j] = (T)nv[1];
      if (cnt > 2) pval[2 * tc + j] = (T)nv[2];
    } else {
      // entries that became inactive leave the list, with their w (at least
      // their w without a patch) in V; without any active entry the largest
      // stays, as a witness with pi_hat = 0
      double vn = vg;
      int pos = 0;
      bool kept = false;
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        if (k < cnt) {
          const bool keep = na ? in[k] : (!kept && w[k] == hi);
          if (keep) {
            kept = true;
            prow[pos * tc + j] = row[k];
            pval[pos * tc + j] = (T)nv[k];
            ++pos;
          } else {
            vn = max_arith(vn, w[k] - G);
          }
        }
      }
      if (pos != cnt) cntv[j] = pos;
      vgv[j] = vn;
    }
  }
  if (open == 0ull) return;

  // ---- columns left open: 16 lanes each, four at a time ----
  const int l = lane & 15, g = lane >> 4, gs = g * 16;
  const bool vec = P->vec_cost != 0;
  // the measure's block maxima: 64 blocks a round, four to a lane (a second
  // round's are read with every column: held, they spill the FP64 kernel's
  // registers to memory that every column then waits for)
  const int nh = nblk > 64 ? 2 : 1;
  double db[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) db[i] = -__builtin_huge_val();
  if (l * 4 < nblkp) load_row4<double>(dblk + l * 4, db);
  // the lanes' patches, for the groups
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    s_pr[wv][k][lane] = row[k];
    s_pw[wv][k][lane] = w[k];
    s_pb[wv][k][lane] = b[k];
  }
  s_pl[wv][lane] = lam;
  wave_lds_sync();
  const unsigned long long freshes = __ballot(vg == __builtin_huge_val());
  const double rise = 16.0 * max_arith(delta, 0.0);
  double* const lw = s_w[wv] + gs;
  double* const lb = s_b[wv] + gs;
  int* const lr = s_r[wv] + gs;
  unsigned long long whole = 0ull;  // columns for a whole wave
  auto group_bits = [&](bool c) -> unsigned { return (unsigned)(__ballot(c) >> gs) & 0xffffu; };
  // threshold of the group's entries (one per lane, -inf for none) for mass
  // tq: Newton steps from the set of all of them (below the root), which is
  // the active set as often as not
  auto simplex16 = [&](double x, double tq, unsigned& set) -> double {
    double lm = -1.7e308;
    int last = -1;
    bool run = true;
    set = 0u;
    for (int it = 0; it < kPatch + 2; ++it) {
      const bool in = run && x > lm;
      const unsigned bits = group_bits(in);
      const int na = __popc(bits);
      if (run) {
        set = bits;
        run = na != last && na != 0;  // na = 0: the largest less tq rounded to itself, nothing active
        last = na;
      }
      if (__ballot(run) == 0ull) break;
      const double S = row16_reduce<OpSum>(in ? x : 0.0);
      if (run) lm = (S - tq) / (double)na;
    }
    return lm;
  };
  // columns (of the tile) whose group has cond, as a mask
  auto columns_where = [&](int mine, bool cond) -> unsigned long long {
    unsigned long long d = 0ull;
    const unsigned long long c = __ballot(cond);
    if (c != 0ull) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int mk = __builtin_amdgcn_readlane(mine, k * 16);
        if (mk >= 0 && ((c >> (k * 16)) & 1ull)) d |= 1ull << mk;
      }
    }
    return d;
  };
  while (open != 0ull) {
    int mine = -1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (open != 0ull) {
        const int s = __builtin_ctzll(open);
        open &= open - 1;
        if (g == k) mine = s;
      }
    }
    const int src = mine >= 0 ? mine : 0;
    // every lane shuffles: a source lane may belong to a group without a column
    const int ncol = __shfl(cnt, src);
    const int n0 = mine >= 0 ? ncol : 0;
    const bool dense0 = n0 < 0;
    whole |= columns_where(mine, dense0);
    bool live = mine >= 0 && !dense0;
    if (__ballot(live) == 0ull) continue;
    const int64_t jj = j0 + src;
    const int64_t c2 = (int64_t)__shfl((int)cc, src);
    const double tq = shfl_d(tau, src);
    const bool fresh = live && ((freshes >> src) & 1ull);
    const bool many = live && n0 > NL;  // more patches than a lane takes
    const bool any_many = __ballot(many) != 0ull;
    const T* const col = cost + c2 * cost_ld;
    // block bounds of the column
    double ub[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) ub[h][i] = -__builtin_huge_val();
      if (h < nh && h * 64 + l * 4 < nblkp) {
        T c4[4];
        double d4[4];
        load_row4<T>(gptr(P->cmin) + c2 * nblkp + h * 64 + l * 4, c4);
        if (h > 0) load_row4<double>(dblk + h * 64 + l * 4, d4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (h * 64 + l * 4 + i < nblk) ub[h][i] = __builtin_fma(-(double)c4[i], inv_rho, h > 0 ? d4[i] : db[i]);
      }
    }
    // its patches: entry l in lane l, the rows of the first three in every lane
    const bool has = live && l < n0;
    int er = 0, r3[NL];
    double ew = -__builtin_huge_val(), ebr = 0.0;
#pragma unroll
    for (int k = 0; k < NL; ++k) r3[k] = live && !many && k < n0 ? s_pr[wv][k][src] : -1;
    double lc = s_pl[wv][src];
    unsigned set = 0u;
    if (has && !many) {
      er = s_pr[wv][l][src];
      ew = s_pw[wv][l][src];
      ebr = s_pb[wv][l][src];
    }
    int nmax = 0;  // list entries to go through beyond the first three
    if (any_many) {
      if (has && many) {
        er = prow[l * tc + jj];
        ebr = eb[er];
        ew = __builtin_fma(-(double)col[er], inv_rho, (double)pval[l * tc + jj] + 2.0 * ebr);
      }
      const double lc16 = simplex16(ew, tq, set);
      if (many) lc = lc16;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int y = __builtin_amdgcn_readlane(many ? n0 : 0, k * 16);
        nmax = y > nmax ? y : nmax;
      }
    }
    if (!many) set = group_bits(has && ew > lc);
    lr[l] = has ? er : -1;
    lw[l] = ew;
    lb[l] = ebr;
    wave_lds_sync();
    const double lcr = relaxed ? max_arith(lc, 0.0) : lc;
    // a column that is here for its many patches only
    const double vgs = shfl_d(vg, src);
    const bool settled = many && vgs + G + (fabs(vgs) + fabs(G) + fabs(lc) + tq) * kTie <= lcr;
    const bool look = live && !settled;
    // entries this far below the candidates' threshold cannot be active (the
    // margin covers the rounding of a threshold over a larger set)
    double lim = lcr - (fabs(lcr) + tq) * kTie;

    // w of a lane's four rows of block blk; patched rows and rows past the
    // end as -inf
    auto scan = [&](int blk, bool on, double (&x)[4], double (&bb)[4]) {
      const int r0 = on ? blk * kBlkRows + l * 4 : 0;
      T nb4[4], c[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) c[v] = (T)0;
      load_cost4<T>(col, r0, R, vec, c);
      load_row4<T>(nbv + r0, nb4);
      load_row4<double>(eb + r0, bb);
      int skip = on ? 0 : 15;
#pragma unroll
      for (int k = 0; k < NL; ++k)
        if ((r3[k] & ~3) == r0) skip |= 1 << (r3[k] & 3);
      for (int e = 0; e < nmax; ++e) {
        const int re = lr[e];
        if (many && e < n0 && (re & ~3) == r0) skip |= 1 << (re & 3);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool use = r0 + v < R && !((skip >> v) & 1);
        x[v] = use ? __builtin_fma(-(double)c[v], inv_rho, (double)nb4[v] + 2.0 * bb[v]) : -__builtin_huge_val();
      }
    };

    if (__ballot(fresh) != 0ull) {
      // the candidates are those of a dense iteration, or a stand-in: raise
      // the limit with the block of the largest bound
      double um = -__builtin_huge_val();
      int ui = 0;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (ub[h][i] > um) {
            um = ub[h][i];
            ui = h * 64 + l * 4 + i;
          }
      const double gm0 = row16_reduce<OpMaxA>(um);
      const unsigned eq = group_bits(um == gm0);
      const int blk = __shfl(ui, gs + (eq ? __builtin_ctz(eq) : 0));
      double x[4], bb[4];
      scan(blk, fresh, x, bb);
      const double gm = row16_reduce<OpMaxA>(max_arith(max_arith(x[0], x[1]), max_arith(x[2], x[3])));
      double l1 = gm - tq;
      if (relaxed) l1 = max_arith(l1, 0.0);
      if (fresh && l1 > lcr) lim = l1 - (fabs(l1) + tq) * kTie;
    }

    // blocks to evaluate: by their bound, and those with a patch (their bound
    // is that of the patched row as often as not)
    const double flag = lim - rise;
    double vm = -__builtin_huge_val();  // this lane's bound of w outside the candidates
    unsigned fm = 0u;
    auto must = [&](int r) {
      if (look && r >= 0 && ((r >> 8) & 15) == l) fm |= 1u << (((r >> 12) << 2) | ((r >> 6) & 3));
    };
#pragma unroll
    for (int k = 0; k < NL; ++k) must(r3[k]);
    for (int e = 0; e < nmax; ++e) must(many && e < n0 ? lr[e] : -1);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (look && ub[h][i] > flag) fm |= 1u << (h * 4 + i);
        if (look && !((fm >> (h * 4 + i)) & 1u)) vm = max_arith(vm, ub[h][i]);
      }
    int nc = live ? n0 : 0;  // candidates so far
    for (;;) {
      const unsigned long long any = __ballot(fm != 0u);
      if (any == 0ull) break;
      const unsigned own = (unsigned)(any >> gs) & 0xffffu;
      const bool bon = own != 0u;
      const int ol = bon ? __builtin_ctz(own) : 0;
      const int fb = fm ? __builtin_ctz(fm) : 0;
      const int bk = __shfl((fb >> 2) * 64 + l * 4 + (fb & 3), gs + ol);
      if (bon && l == ol) fm &= fm - 1u;
      double x[4], bb[4];
      scan(bk, bon, x, bb);
      bool hit = false;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool hv = x[v] > lim;
        hit |= hv;
        if (!hv) vm = max_arith(vm, x[v]);
      }
      if (__ballot(hit) != 0ull) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const bool hv = x[v] > lim;
          const unsigned bits = group_bits(hv);
          if (hv) {
            const int at = nc + __popc(bits & ((1u << l) - 1u));
            if (at < kPatch) {
              lr[at] = bk * kBlkRows + l * 4 + v;
              lw[at] = x[v];
              lb[at] = bb[v];
            }
          }
          nc += __popc(bits);
        }
      }
    }
    // too many candidates: the whole wave takes the column below
    whole |= columns_where(mine, nc > kPatch);
    if (nc > kPatch) live = false;
    const bool grew = live && nc > n0;
    double lm = lc;
    if (__ballot(grew) != 0ull) {
      wave_lds_sync();
      if (grew && l >= n0 && l < nc) {
        er = lr[l];
        ew = lw[l];
        ebr = lb[l];
      }
      unsigned set2;
      const double l2 = simplex16(live ? ew : -__builtin_huge_val(), tq, set2);
      if (grew) {
        lm = l2;
        set = set2;
      }
    }
    const bool cand = live && l < nc;
    // three and more active entries (but for the lanes' own sums): their sum
    // in the column kernel's order.  Entries sorted by thread, then row;
    // neighbours are joined where the level at which they meet (0 in one
    // thread, 1 + the highest lane bit they differ in, 7 between waves) is
    // below that on the left and not above that on the right: rows of a
    // thread in turn, lanes as a binary tree, waves in turn.
    const bool tree = live && (grew || many) && __popc(set) > 2;
    if (__ballot(tree) != 0ull) {
      const bool on = tree && ((set >> l) & 1u);
      const int tid = (er >> vecl) & ((1 << ntl) - 1);
      const int key = (tid << 13) | er;  // R <= 8192
      wave_lds_sync();
      lr[l] = key;
      wave_lds_sync();
      int rank = 0;
#pragma unroll
      for (int e = 0; e < kPatch; ++e) rank += ((set >> e) & 1u) && lr[e] < key ? 1 : 0;
      wave_lds_sync();
      if (on) {
        lr[rank] = tid;
        lw[rank] = ew;
      }
      const int total = __popc(set);
      int na = tree ? total : 0;
      auto level = [](int x, int y) -> int {
        const int d = x ^ y;
        return d > 63 ? 7 : (d ? 32 - __builtin_clz(d) : 0);
      };
      while (__ballot(na > 1) != 0ull) {
        wave_lds_sync();
        const int kc = lr[l], kp = lr[l > 0 ? l - 1 : 0], kn = lr[l < 15 ? l + 1 : 15], k2 = lr[l < 14 ? l + 2 : 15];
        const double sc = lw[l], sn = lw[l < 15 ? l + 1 : 15];
        const int lv = level(kc, kn);
        const bool join = l + 1 < na && (l == 0 || lv < level(kp, kc)) && (l + 2 >= na || lv <= level(kn, k2));
        const unsigned jb = group_bits(join);
        const bool gone = ((jb << 1) >> l) & 1u;
        wave_lds_sync();
        if (l < na && !gone) {
          const int at = l - __popc(jb & ((1u << l) - 1u));
          lr[at] = kc;
          lw[at] = join ? sc + sn : sc;
        }
        na -= __popc(jb);
      }
      wave_lds_sync();
      const double S = lw[0];
      if (tree) lm = (S - tq) / (double)total;
    }
    // entries at the threshold, but for the largest (there is none larger)
    const double gap = ew - lm, eps = (fabs(lm) + tq) * kTie;
    const bool near = cand && fabs(gap) <= eps;
    bool tie = false;
    if (__ballot(near) != 0ull) {
      tie = live && __popc(group_bits(near)) > (group_bits(cand && gap > eps) != 0u ? 0 : 1);
      if constexpr (REC)
        tie = tie || (live && group_bits(cand && gap > 0.0) == 0u && group_bits(cand && top_unsure<REC>(ew, lm)) != 0u);
      whole |= columns_where(mine, tie);
    }
    if (live && !tie) {
      const double lo16 = relaxed ? max_arith(lm, 0.0) : lm;
      const bool in = cand && (relaxed ? ew > lo16 : ((set >> l) & 1u) != 0u);
      unsigned bits = group_bits(in);
      double nv = -ebr;
      if (in) {
        const double ph = max_arith(ew - lo16, 0.0);
        nv = ph - ebr;
        atomicAdd(acc + er, to_fixed(ph, fxm));
        if constexpr (REC) set_mask_bit(a.rec, a.rec_ld, jj, er, ntl, vecl, P->vpt);
      }
      if (bits == 0u) {
        // nothing active: the largest entry stays as a witness (pi_hat = 0)
        const double top = row16_reduce<OpMaxA>(cand ? ew : -__builtin_huge_val());
        const unsigned eq = group_bits(cand && ew == top);
        bits = eq & (0u - eq);
        if (bits == 0u) bits = 1u;
      }
      const bool keep = ((bits >> l) & 1u) != 0u;
      if (keep) {
        const int pos = __popc(bits & ((1u << l) - 1u));
        prow[pos * tc + jj] = er;
        pval[pos * tc + jj] = (T)nv;
      } else if (cand) {
        vm = max_arith(vm, ew);
      }
      vm = row16_reduce<OpMaxA>(vm);
      if (l == 0) {
        cntv[jj] = __popc(bits);
        vgv[jj] = max_arith(vm - G, settled ? vgs : -1e300);
        lamv[jj] = lm;
      }
    }
    wave_lds_sync();
  }

  // ---- columns taken by the whole wave, in the column kernel's order ----
  while (whole != 0ull) {
    const int s = __builtin_ctzll(whole);
    whole &= whole - 1;
    const int64_t jj = j0 + s;
    const int n0 = uniform_i(__shfl(cnt, s));
    const bool dense0 = n0 < 0;
    const int np = dense0 ? 0 : n0;
    const int64_t c2 = (int64_t)uniform_i(__shfl((int)cc, s));
    const double tq = uniform_d(shfl_d(tau, s));
    T* const th = gptr(P->theta) + jj * P->ld;
    const T* const col = cost + c2 * cost_ld;
    if (lane < np) {
      s_r[wv][lane] = prow[lane * tc + jj];
      s_w[wv][lane] = (double)pval[lane * tc + jj];
    }
    wave_lds_sync();
    const int nt = 1 << ntl, vpt = P->vpt;
    const int nwave = nt > 64 ? nt / 64 : 1;
    constexpr int KW = kWholeRows;
    double x[KW], bx[KW];
    int rx[KW];
    // w (and b) of entries k0 .. k0 + KW - 1 of this lane's thread of wave v;
    // -inf past the end
    auto rows_of = [&](int v, int k0) {
      const int tid = v * 64 + lane;
      T tv[KW], cv[KW];
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        const int k = k0 + i;
        const int r = ((((k >> vecl) << ntl) + tid) << vecl) + (k & ((1 << vecl) - 1));
        rx[i] = k < vpt && tid < nt && r < R ? r : -1;
        const int rr = rx[i] >= 0 ? rx[i] : 0;
        tv[i] = dense0 ? th[rr] : nbv[rr];
        cv[i] = col[rr];
        bx[i] = eb[rr];
      }
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        double t = (double)tv[i];
        for (int e = 0; e < np; ++e)
          if (s_r[wv][e] == rx[i]) t = s_w[wv][e];
        x[i] = rx[i] >= 0 ? __builtin_fma(-(double)cv[i], inv_rho, t + 2.0 * bx[i]) : -__builtin_huge_val();
      }
    };
    // one round of the column kernel: the entries above bound, their sum in
    // its order, the least of them and the largest of the others
    auto count = [&](double bound, double* sum, double* least, double* most) -> int {
      double S = 0.0, lo = __builtin_huge_val(), hi = -__builtin_huge_val();
      int c = 0;
      for (int v = 0; v < nwave; ++v) {
        double y = 0.0;
        for (int k0 = 0; k0 < vpt; k0 += KW) {
          rows_of(v, k0);
#pragma unroll
          for (int i = 0; i < KW; ++i) {
            const bool in = x[i] > bound;
            y += in ? x[i] : 0.0;
            c += in ? 1 : 0;
            lo = fmin(lo, in ? x[i] : __builtin_huge_val());
            hi = fmax(hi, in ? -__builtin_huge_val() : x[i]);
          }
        }
        S += wave_reduce<OpSum>(y);
      }
      for (int o = 32; o; o >>= 1) c += __shfl_xor(c, o);
      *sum = S;
      *least = wave_reduce<OpMin>(lo);
      *most = wave_reduce<OpMax>(hi);
      return uniform_i(c);
    };
    // its rounds, from the stored threshold (lset: the bound whose set, of na
    // entries, gives lm).  A round depends on lm and the last count alone, so
    // one that finds both as they were two rounds ago starts a cycle of two,
    // and an even number of rounds can be left out.
    double lm = uniform_d(lamv[jj]), lset = lm, lm1 = lm, lm2 = __builtin_nan(""), S, least, most;
    int na = 0, last = -1, last1 = -1, last2 = -2;
    bool settled = false;
    for (int it = 0;; ++it) {
      if (lm == lm2 && last == last2 && it < R + 4) it += (R + 3 - it) & ~1;
      lm2 = lm1;
      last2 = last1;
      lm1 = lm;
      last1 = last;
      settled = settled || it >= R + 4;
      if (settled) {
        if (!relaxed || na == 0) break;
        lset = max_arith(lset, max_arith(lm, 0.0));  // of the entries that it took, those above 0
      }
      na = count(settled ? lset : lm, &S, &least, &most);
      if (settled) break;
      if (na == 0) {
        settled = lm == lm && last >= 0;
        if (lm != lm) {
          lm = most - tq;
          last = 0x7fffffff;
        } else if (!settled) {
          lm = __builtin_nan("");
        }
        continue;
      }
      lset = lm;
      lm = (S - tq) / (double)na;
      settled = na == last || ((double)float_down(least) >= lm && (double)float_up(most) <= lm);
      last = na;
    }
    const double lo2 = relaxed ? max_arith(lm, 0.0) : lm;
    // the new values; a row's w is formed before its value is stored
    // (nothing active: a row of the largest w stays as a witness)
    int pos = 0;
    double vm = -__builtin_huge_val();
    const bool dense = na > kPatch;
    for (int v = 0; v < nwave; ++v)
      for (int k0 = 0; k0 < vpt; k0 += KW) {
        rows_of(v, k0);
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          const int r = rx[i];
          const bool in = r >= 0 && na != 0 && x[i] > lset;
          double ph = 0.0;
          if (in) {
            ph = max_arith(x[i] - lo2, 0.0);
            atomicAdd(acc + r, to_fixed(ph, fxm));
            if constexpr (REC) set_mask_bit(a.rec, a.rec_ld, jj, r, ntl, vecl, vpt);
          }
          const T nv = (T)(in ? ph - bx[i] : -bx[i]);
          if (dense) {
            if (r >= 0) th[r] = nv;
          } else {
            const bool wit = na == 0 && pos == 0 && r >= 0 && x[i] == most;
            const unsigned long long top = __ballot(wit);
            const bool keep = in || (wit && lane == __builtin_ctzll(top));
            const unsigned long long bits = __ballot(keep);
            if (keep) {
              const int at = pos + __popcll(bits & ((1ull << lane) - 1ull));
              prow[at * tc + jj] = r;
              pval[at * tc + jj] = nv;
            } else {
              vm = max_arith(vm, x[i]);
            }
            pos += __popcll(bits);
          }
        }
      }
    vm = wave_reduce<OpMaxA>(vm);
    if (lane == 0) {
      cntv[jj] = dense ? -1 : pos;
      // rows read from theta need not be -b of the last iteration: V not known
      vgv[jj] = dense || dense0 ? __builtin_huge_val() : max_arith(vm - G, -1e300);
      lamv[jj] = lm;
    }
    wave_lds_sync();
  }
}

// What the next sparse iteration reads of measure m in a block of 64 rows
// (lane = row): b, and the block's largest base = nbv + 2b and its largest
// rise since the last iteration (reset: the measure's first sparse
// iteration, nothing to compare with).
template <typename T>
__device__ __forceinline__ void sparse_next(const ConstPtr<SpProb<T>> P, int m, int blk, int lane, bool in, double b,
                                            double nb, double last, int wpar, bool reset) {
  const int64_t o = (int64_t)m * P->Rp + blk * 64 + lane;
  const double base = nb + 2.0 * b;
  const double up = reset ? 0.0 : base - last;
  gptr(P->bb)[o] = base;
  gptr(P->eb)[o] = b;
  const double mx = wave_reduce<OpMaxA>(in ? base : -__builtin_huge_val());
  const double dx = wave_reduce<OpMaxA>(in ? up : -__builtin_huge_val());
  if (lane == 0) {
    gptr(P->dblk)[(int64_t)m * P->nblkp + blk] = mx;
    gptr(P->drift)[((int64_t)wpar * P->M + m) * P->nblkp + blk] = dx;
  }
}

// The rise that the iteration used joins the sums (one wave, measure m).
template <typename T>
__device__ __forceinline__ void sparse_absorb(const ConstPtr<SpProb<T>> P, int m, int lane, int rpar, bool reset) {
  const double* const dr = gptr(P->drift) + ((int64_t)rpar * P->M + m) * P->nblkp;
  const double g = gptr(P->G)[m];
  double d = lane < P->nblk ? dr[lane] : -__builtin_huge_val();
  if (lane + 64 < P->nblk) d = fmax(d, dr[lane + 64]);
  d = wave_reduce<OpMax>(d);
  if (lane == 0) gptr(P->G)[m] = reset ? 0.0 : drift_sum(g, d);
}

// How an iteration updated measure m: 0 not at all (bundles), 1 yes, 2 as
// its first sparse iteration.  mode: the first iteration of a call, or one after it.
constexpr int kSpFirst = 1, kSpNext = 2;

// Steps 3 and 1 of a block of 64 rows, all measures: the new marginals from
// the fixed-point sums, p, the partial sum of d^2, nbv = (T)(-b) of the
// iteration that ended and, with gamma = inf (t = 1), what the next sparse
// iteration reads.  Wave w of the workgroup takes measures w, w + W, ...; wave
// 0 sums p and d^2 in the order m = 0, 1, ... from LDS (every wave summing p
// by itself read 16 times as much LDS, and the divisions of d^2 were one
// wave's: 8.8 us at 1024 rows and 50 measures with a finite gamma, 7.2 us now).
// upd: null, or per measure how the iteration updated it.
template <typename T>
__global__ void __launch_bounds__(1024)
sparse_close_kernel(const SpProb<T>* __restrict__ probs, const SpRows* __restrict__ tasks, int save_prev,
                    const uint8_t* __restrict__ upd, int mode, const int32_t* __restrict__ stop) {
  extern __shared__ double sp_lds[];
  __shared__ double s_p[64];
  const int stopv = stop != nullptr ? *gptr(stop) : 0;
  const ConstPtr<SpRows> tk = cptr(tasks) + blockIdx.x;
  const ConstPtr<SpProb<T>> P = cptr(probs) + tk->prob;
  if (uniform_i(stopv) != 0) return;
  const int blk = tk->blk;
  const int lane = threadIdx.x & 63, wv = uniform_i((int)(threadIdx.x >> 6));
  const int W = blockDim.x >> 6;
  const int R = P->R, M = P->M, Rp = P->Rp;
  const bool balanced = P->balanced != 0;
  double* const sv = sp_lds;                                    // [M][64] new marginals
  double* const sl = sp_lds + (size_t)M * 64;                   // [M][64] base of the iteration that ended
  T* const sn = reinterpret_cast<T*>(sp_lds + (size_t)2 * M * 64);  // [M][64] -b
  const int r = blk * 64 + lane;
  const bool in = r < R;
  const int rr = in ? r : R - 1;
  double* const pm = gptr(P->pm);
  double* const p = gptr(P->p);
  unsigned long long* const acc = gptr(P->acc);
  T* const nbv = gptr(P->nbv);
  const ConstPtr<double> aw = cptr(P->aw), Sd = cptr(P->Sd), fxinv = cptr(P->fx) + M;
  const double t = balanced ? 1.0 : uniform_d(*gptr(P->t_out));
  const int rpar = mode == kSpNext ? uniform_i(gptr(P->par)[0]) : 0;
  const double pold = p[rr];
  auto updated = [&](int m) -> int { return upd != nullptr ? (int)upd[m] : 1; };
  constexpr int U = 4;
  for (int m0 = wv; m0 < M; m0 += W * U) {
    double old[U], last[U];
    unsigned long long ac[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * W < M ? m0 + u * W : wv;
      const int64_t o = (int64_t)m * R + rr;
      old[u] = pm[o];
      ac[u] = acc[o];
      last[u] = balanced ? gptr(P->bb)[(int64_t)m * Rp + rr] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * W;
      if (m < M) {
        const int64_t o = (int64_t)m * R + rr;
        double v = old[u];
        T nb;
        if (updated(m) != 0) {
          const double Sm = Sd[m];
          const double b = t * (pold - old[u]) / Sm;
          v = (double)ac[u] * fxinv[m] - Sm * b;
          nb = (T)(-b);
          if (in) {
            acc[o] = 0ull;
            pm[o] = v;
            nbv[(int64_t)m * Rp + r] = nb;
          }
        } else {
          nb = nbv[(int64_t)m * Rp + rr];
        }
        if (save_prev && in) gptr(P->pm_prev)[o] = old[u];
        sv[m * 64 + lane] = v;
        sl[m * 64 + lane] = last[u];
        sn[m * 64 + lane] = nb;
      }
    }
  }
  if (blk == 0 && balanced) {
    for (int m = wv; m < M; m += W) sparse_absorb<T>(P, m, lane, rpar, mode != kSpNext || updated(m) == 2);
    if (threadIdx.x == 0) gptr(P->par)[1] = rpar ^ 1;
  }
  __syncthreads();
  double pr = 0.0;
  if (wv == 0) {
#pragma unroll 8
    for (int m = 0; m < M; ++m) pr += aw[m] * sv[m * 64 + lane];
    s_p[lane] = pr;
    if (in) {
      if (save_prev) gptr(P->p_prev)[r] = pold;
      p[r] = pr;
    }
  }
  __syncthreads();
  pr = s_p[lane];
  if (!balanced) {  // (sl is free)
    for (int m = wv; m < M; m += W) {
      const double e = pr - sv[m * 64 + lane];
      sl[m * 64 + lane] = e * e / Sd[m];
    }
    __syncthreads();
    if (wv == 0) {
      double d2 = 0.0;
      if (in) {
#pragma unroll 8
        for (int m = 0; m < M; ++m) d2 += sl[m * 64 + lane];
      }
      d2 = wave_sum(d2);
      if (lane == 0) gptr(P->d2w)[blk] = d2;
    }
    return;  // sparse_next_kernel, once d^2 is complete
  }
  for (int m = wv; m < M; m += W)
    sparse_next<T>(P, m, blk, lane, in, (pr - sv[m * 64 + lane]) / Sd[m], (double)sn[m * 64 + lane],
                   sl[m * 64 + lane], rpar ^ 1, mode != kSpNext || updated(m) == 2);
}

// The last part of the close of problems with a finite gamma: t^{k+1} needs
// every block's part of d^2, so it is a launch of its own; it also publishes
// t^{k+1}.  The measures of a block are dealt over gridDim.y workgroups, one
// measure to a wave: with all of them in one workgroup, as in the close
// kernel, a wave took four in turn and 1024 rows x 50 measures 6.4 us on 16
// workgroups (4.2 us now).
template <typename T>
__global__ void __launch_bounds__(1024)
sparse_next_kernel(const SpProb<T>* __restrict__ probs, const SpRows* __restrict__ tasks,
                   const uint8_t* __restrict__ upd, int mode, const int32_t* __restrict__ stop) {
  const int stopv = stop != nullptr ? *gptr(stop) : 0;
  const ConstPtr<SpRows> tk = cptr(tasks) + blockIdx.x;
  const ConstPtr<SpProb<T>> P = cptr(probs) + tk->prob;
  if (uniform_i(stopv) != 0 || P->balanced != 0) return;
  const int blk = tk->blk;
  const int lane = threadIdx.x & 63, wv = uniform_i((int)(threadIdx.x >> 6));
  const int W = blockDim.x >> 6;
  const int R = P->R, M = P->M, Rp = P->Rp;
  const double t = damping_t64(gptr(P->d2w), P->nblk, P->rho, P->gamma, lane);
  const int rpar = mode == kSpNext ? uniform_i(gptr(P->par)[0]) : 0;
  const int r = blk * 64 + lane;
  const bool in = r < R;
  const int rr = in ? r : R - 1;
  const ConstPtr<double> Sd = cptr(P->Sd);
  const double pr = gptr(P->p)[rr];
  for (int m = (int)blockIdx.y * W + wv; m < M; m += W * (int)gridDim.y) {
    const bool reset = mode != kSpNext || (upd != nullptr && upd[m] == 2);
    const double b = t * (pr - gptr(P->pm)[(int64_t)m * R + rr]) / Sd[m];
    sparse_next<T>(P, m, blk, lane, in, b, (double)gptr(P->nbv)[(int64_t)m * Rp + rr],
                   gptr(P->bb)[(int64_t)m * Rp + rr], rpar ^ 1, reset);
    if (blk == 0) sparse_absorb<T>(P, m, lane, rpar, reset);
  }
  if (blk == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    gptr(P->par)[1] = rpar ^ 1;
    gptr(P->t_out)[1] = t;
  }
}

// The 256-row partial sums of d^2 that the dense kernels read, from the
// close kernel's 64-row ones (added in the dense kernels' order).
template <typename T>
__global__ void __launch_bounds__(256)
sparse_d2_kernel(const SpProb<T>* __restrict__ probs, const int32_t* __restrict__ stop) {
  if (stop != nullptr && *gptr(stop) != 0) return;
  const SpProb<T>& P = probs[blockIdx.x];
  const double* const w = gptr(P.d2w);
  for (int i = threadIdx.x; i * 4 < P.nblk; i += 256) {
    double s = w[i * 4];
    for (int k = 1; k < 4; ++k) s += i * 4 + k < P.nblk ? w[i * 4 + k] : 0.0;
    gptr(P.d2part)[i] = s;
  }
}

// The plans back into theta: nbv with the patches in place (columns stored
// dense are there already).  A workgroup takes one tile; a thread holds 16
// bytes or two times 16 of nbv and walks the tile's columns.  note: null, or a
// word of host memory for the most rows that a tile holds in columns stored
// dense, under the plan's tag (the host looks at it before the next call and
// never waits for it; a tile that meets another's note may leave the smaller).
template <typename T>
__global__ void __launch_bounds__(256)
sparse_write_kernel(const SpProb<T>* __restrict__ probs, const SpTile* __restrict__ tiles,
                    const int32_t* __restrict__ stop, unsigned long long* __restrict__ note, unsigned tag) {
  __shared__ int32_t s_n[64], s_r[64][kPatch];
  __shared__ T s_v[64][kPatch];
  if (stop != nullptr && *gptr(stop) != 0) return;
  const ConstPtr<SpTile> tk = cptr(tiles) + blockIdx.x;
  const ConstPtr<SpProb<T>> P = cptr(probs) + tk->prob;
  const int m = tk->m, n = tk->n & 0xffff;
  const int64_t j0 = tk->j0, tc = P->tcols, ld = P->ld;
  for (int i = threadIdx.x; i < n * kPatch; i += 256) {
    const int e = i / n, c = i - e * n;
    const int cn = gptr(P->cnt)[j0 + c];
    if (e == 0) s_n[c] = cn;
    if (e < cn) {
      s_r[c][e] = gptr(P->prow)[e * tc + j0 + c];
      s_v[c][e] = gptr(P->pval)[e * tc + j0 + c];
    }
  }
  __syncthreads();
  const int R = P->R;
  if (note != nullptr && threadIdx.x < 64) {
    const int rows = __popcll(__ballot((int)threadIdx.x < n && s_n[threadIdx.x] < 0)) * R;
    if (threadIdx.x == 0 && rows > 0 && atomicMax(gptr(P->wide), rows) < rows)
      __hip_atomic_store(note, (unsigned long long)tag << 32 | (unsigned)rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  const bool vec = P->vec_theta != 0;
  const T* const nbv = gptr(P->nbv) + (int64_t)m * P->Rp;
  T* const theta = gptr(P->theta);
  // 1024 rows at a time, 16 bytes per thread and store, neighbouring threads
  // on neighbouring vectors (32 contiguous bytes per thread instead, two
  // half-line stores, took 2.15 ms for 3.2 GB of FP64 plans)
  constexpr int VN = VecOf<T>::N, H = 4 / VN;
  for (int c0 = 0; c0 < R; c0 += 1024) {
    T nb[H][VN];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int r = c0 + (h * 256 + (int)threadIdx.x) * VN;
      if (r < R) load_vec<T, VN>(nbv + r, nb[h]);  // nbv is padded to whole blocks
    }
    for (int c = 0; c < n; ++c) {
      const int cn = s_n[c];
      if (cn < 0) continue;
      T* const col = theta + (j0 + c) * ld;
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int r = c0 + (h * 256 + (int)threadIdx.x) * VN;
        T x[VN];
#pragma unroll
        for (int k = 0; k < VN; ++k) x[k] = nb[h][k];
        for (int e = 0; e < cn; ++e) {
          const int d = s_r[c][e] - r;
          if (d >= 0 && d < VN) {
            const T v = s_v[c][e];
#pragma unroll
            for (int k = 0; k < VN; ++k) x[k] = d == k ? v : x[k];
          }
        }
        if (vec && r + VN <= R) {
          store_vec_nt<T, VN>(col + r, x);
        } else {
#pragma unroll
          for (int k = 0; k < VN; ++k)
            if (r + k < R) col[r + k] = x[k];
        }
      }
    }
  }
}

}  // namespace mam
