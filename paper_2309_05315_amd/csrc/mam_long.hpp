// Device code of MAM for long plan columns: R beyond what one workgroup
// holds in registers.  The free-support formulation (Theorem c: measures on
// one K^d grid with alpha_m = 1/M) has R = ((K-1)M+1)^d candidate support
// points, 349,281 for M = 10 images of 60 x 60 pixels.
//
// A column is cut into row tiles of RB = 256*VPT rows; inside a tile each of
// the four waves of a workgroup owns an interleaved quarter of the rows (a
// sub-tile).  Thread tid holds rows rb*RB + ((k/VEC)*256 + tid)*VEC + k%VEC,
// k < VPT.  One iteration of Alg. 1 is three kernels plus the marginal and
// averaging kernels of the short path:
//
//   scan       per (column, sub-tile): w = theta + 2b - c/rho, the sub-tile's
//              maximum w_loc, and the entries with w > w_loc - q_s (at most
//              E of them kept, in fixed slots).  An entry left out has
//              w <= w_loc - q_s <= w_max - q_s <= lambda (one entry of a
//              projection onto Delta_R(q_s) carries at most q_s, Prop. 3), so
//              it is inactive.
//   threshold  per column (one wave): the exact threshold of Prop. 3 from the
//              kept entries of the sub-tiles with w_loc > w_max - q_s (no other
//              sub-tile can hold an active entry).  Newton steps on the
//              piecewise-linear root with an exactness certificate; every step
//              is kept >= w_max - q_s, so the left-out entries stay below it.
//   write      per (column, sub-tile): theta' = -b everywhere, patched with
//              max(w - lambda, 0) - b at the kept entries above lambda (none
//              unless w_loc > lambda), and the tile's row-sum partials (fixed
//              order, no atomics).
//
// The sub-tile headers and slots are the only cross-workgroup exchange: theta
// and c are read once and theta written once per iteration.  A sub-tile with
// more than E candidates is recomputed from theta and c where it is needed
// (threshold rounds, and the write pass before theta is overwritten).  Every
// sum has a fixed order: results are bitwise reproducible.
//
// With the sparse store an iteration of a call after its first has three more
// kernels' worth of choices to make, so that work follows the active entries
// and not T x R:
//
//   base       per (measure, row): 2b and the common value + 2b
//   limit      per column: a lower bound of its threshold from its last active
//              entries, and from it the sub-tiles that can hold an active one
//              (their bound: least cost, largest common value + 2b)
//   scan       the (column, sub-tile) pairs left, from a work list; candidates
//              above the bound only
//
// Ten 40 x 40 images (R = 152,881, 16,000 columns, FP32), per iteration:
// scanning every sub-tile 2.9 ms scan, 0.24 ms threshold, 0.28 ms write; now
// 13 us base, 41 us limit, 71 us scan, 32 us threshold, 45 us write.  About
// three of a column's 152 sub-tiles are scanned, two of them for their
// patches.  20 iterations of a call: 63 -> 14.5 ms, of which 7.8 ms are the
// start's fill, the first scan and the write-back: 9.8 GB each.
#pragma once

#include <utility>

#include "mam_kernels.hpp"

namespace mam {

constexpr int LNT = 256;  // threads per workgroup of the tile kernels (4 waves)

template <typename T>
struct LongArgs {
  T* theta;
  const T* cost;
  const T* q;
  const int32_t* cidx;
  int64_t ld, cost_ld;
  int32_t R, cost_mode, M, nrb;  // nrb: row tiles per column
  int32_t cap, warm;             // candidate slots per sub-tile; warm starts on
  int32_t relaxed, pad0;         // columns projected onto {u >= 0, sum u <= q_s}
  double rho, inv_rho, gamma;
  double* t;                     // damping t^k of the iteration (set by damping_kernel)
  const double* p;               // R, averaged marginal
  const double* pm;              // M x R marginals
  const double* d2part;          // ceil(R/256) partial sums of d^2
  int32_t nb, pad;
  const double* Sd;              // S^m as double
  const int64_t* col_off;        // M+1
  // work items (row tile, measure, column range), in schedule order
  const int32_t* it_rb;
  const int32_t* it_m;
  const int64_t* it_j0;
  const int64_t* it_j1;
  const int64_t* it_poff;        // offset of the item's RB row-sum partials
  const int32_t* wg_it;          // items of workgroup w: [wg_it[w], wg_it[w+1])
  // per (column j, sub-tile s = rb*4 + wave), index h = j*nrb*4 + s
  double* hmax;                  // the sub-tile's maximum of w
  int32_t* hcnt;                 // its candidates (entries with w > hmax - q_s)
  int32_t* crow;                 // h*cap + e: row of candidate e < min(hcnt, cap)
  double* cw;                    //            its w
  double* lam;                   // T: threshold (previous one in, new one out)
  double* partial;
  const int32_t* stop;           // early-exit flag, or null
  int64_t T_cols;
  // grid cost (cost_mode MAM_COST_GRID): row r is point (i0, i1) of an
  // n0 x n1 grid (last axis fastest; gdim 1: i0 = r, gn1 = 1 and a second
  // axis of origin and spacing 0) with coordinates go[k] + i_k * gh[k], and
  // cost column s is the point gz[s*gdim ..]: c_rs = sum_k (x_rk - z_sk)^2,
  // rounded to the storage type
  int32_t gdim, gn1;
  double go[2], gh[2];
  const double* gz;
  // sparse store (MAM_FLAG_SPARSE_STORE): between iterations the plans are
  // held per (column j, sub-tile s) either as the dense rows in theta
  // (pcnt[s*T + j] < 0) or as pcnt[s*T + j] >= 0 patches (row, value), in
  // slots h*cap + e with h = j*nsub + s, over the value nbv[par][m][r] that
  // every other entry of measure m's row r holds
  int32_t sparse, pad1;
  int32_t* spar;                 // [0] par: which half of nbv holds the stored plans; [1] all of them dense;
                                 // [2] entries of the work list
  int32_t* pcnt;
  int32_t* prow;                 // h*cap + e: row of patch e
  T* pval;                       //            its value
  T* nbv;                        // 2 x M x R
  // diagnostics of the iteration (the DIAG instances): per column j,
  // ldiag[4j..4j+3] = <c_s, pi_hat_s>, the column's measure residual, its
  // threshold rounds and active entries; per write workgroup w,
  // wdiag[w*DIAG_STRIDE + 2] = max |theta' - theta| over its entries (dense
  // store only)
  double* ldiag;
  double* wdiag;
  // sparse store: what the scan can leave out (see long_limit_kernel)
  T* cmin;                       // nsub x ncost: least cost of each sub-tile, per cost column
  int64_t ncost, c_first;        // cost columns; the first one of a cost_min launch
  double* limit;                 // T: a lower bound of the column's threshold (-inf: none)
  int32_t* wit;                  // T: a row of the column's largest w, or -1
  unsigned long long* smask;     // T x nmask words: the sub-tiles the scan looked at (the others have no header)
  unsigned long long* gmask;     // nsub x ngrp words: the same by sub-tile, for groups of 64 columns
  int32_t nmask, ngrp;
  // per (measure m, tile rb, slot k, thread tid) at ((m*nrb + rb)*VPT + k)*256
  // + tid: 2 b of the slot's row and the common value + 2 b (-inf past R);
  // and per (m, sub-tile) the largest of the latter
  double* b2v;
  double* basev;
  double* bmax;                  // M x nsub
  // work list of the sparse-store scan, spar[2] entries: sub-tile, group of 64
  // columns, and which of them
  int32_t* wsub;
  int32_t* wgrp;
  unsigned long long* wcol;
  int32_t* colm;                 // T: measure of the column
};

// Columns of an entry of the sparse-store scan's work list (a group of 64 is
// up to eight of them).
constexpr int kScanCols = 8;

// Waves of a workgroup of long_limit_kernel.
constexpr int kLimitWaves = 16;

// Coordinate k of grid index i: origin + i * spacing, each operation rounded
// (no fused multiply-add).
template <typename T>
__device__ __forceinline__ double grid_coord(const LongArgs<T>& a, int k, int i) {
#pragma clang fp contract(off)
  return a.go[k] + (double)i * a.gh[k];
}

// The grid cost of the point (x0, x1) and the column's point (z0, z1),
// evaluated in the order of its definition (each product and sum rounded, no
// fused multiply-add), then rounded to the storage type as a stored cost
// would be.  On a one-dimensional grid x1 = z1 = 0, so the second term is +0
// and c = d0^2 exactly.
template <typename T>
__device__ __forceinline__ double grid_cost_xy(double x0, double x1, double z0, double z1) {
#pragma clang fp contract(off)
  const double d0 = x0 - z0, d1 = x1 - z1;
  const double c = d0 * d0 + d1 * d1;
  return (double)(T)c;
}

// The column's point (z0, z1) of cost column j (z1 = 0 on a 1-D grid).
template <typename T>
__device__ __forceinline__ void grid_point(const LongArgs<T>& a, int64_t j, int64_t off_m, double* z0, double* z1) {
  const double* z = gptr(a.gz) + (j - off_m) * a.gdim;
  *z0 = z[0];
  *z1 = a.gdim == 2 ? z[1] : 0.0;
}

template <typename T>
__device__ __forceinline__ double grid_cost(const LongArgs<T>& a, int r, double z0, double z1) {
  const int i0 = r / a.gn1;
  return grid_cost_xy<T>(grid_coord(a, 0, i0), grid_coord(a, 1, r - i0 * a.gn1), z0, z1);
}

template <typename T>
__device__ __forceinline__ const T* long_cost_col(const LongArgs<T>& a, int64_t j, int64_t off_m) {
  int64_t cc;
  if (a.cost_mode == MAM_COST_INDEXED) cc = a.cidx[j];
  else if (a.cost_mode == MAM_COST_SHARED) cc = j - off_m;
  else cc = j;
  return a.cost + cc * a.cost_ld;
}

// The value of v in lane l (l wave-uniform).
__device__ __forceinline__ double read_lane(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float read_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// w = theta + 2b - c/rho (FP64) from 2b: one expression with one fused
// multiply-add, so the scan, threshold and write kernels form the same value
// for an entry.
__device__ __forceinline__ double long_w(double th, double b2, double c, double inv_rho) {
  return __builtin_fma(-c, inv_rho, th + b2);
}

// b^(m)_r = t (p_r - p^(m)_r) / S^m: every kernel forms it with this one
// expression, so all of them see the same value.
__device__ __forceinline__ double long_b(double t, const double* p, const double* pmm, int r, double Sm) {
  return t * (p[r] - pmm[r]) / Sm;
}

// Thread tt of the tile at rbase owns rows rbase + ((k/VEC)*LNT + tt)*VEC + k%VEC,
// k < VPT; row offset rr = r - rbase is slot k of thread (rr/VEC) % LNT.
__device__ __forceinline__ int slot_owner(int rr, int vec) { return (rr / vec) % LNT; }
__device__ __forceinline__ int slot_of(int rr, int vec) { return (rr / (vec * LNT)) * vec + rr % vec; }

// Sparse store: apply the pc <= cap patches (lane e holds row pr and value
// pv of patch e) to the values th of thread tt's rows, in patch order.
template <typename T, int VPT, int VEC>
__device__ __forceinline__ void apply_patches(int pc, int pr, T pv, int rbase, int tt, T (&th)[VPT]) {
  for (int e = 0; e < pc; ++e) {
    const int rr = __builtin_amdgcn_readlane(pr, e) - rbase;
    const T v = read_lane(pv, e);
    if (slot_owner(rr, VEC) == tt) {
      const int k = slot_of(rr, VEC);
#pragma unroll
      for (int kk = 0; kk < VPT; ++kk)
        if (kk == k) th[kk] = v;
    }
  }
}

// The stored plan values of thread tt's rows of the tile at rbase in column j
// (sub-tile si, measure m), 0 at rows past R: the dense rows, or the
// measure's common values with the sub-tile's patches.
template <typename T, int VPT, int VEC>
__device__ void stored_rows(const LongArgs<T>& a, int64_t j, int si, int rbase, int tt, int m, int par,
                            T (&th)[VPT]) {
  const int R = a.R;
  const int64_t h = j * (a.nrb * 4) + si;
  const int pc = a.sparse ? uniform_i(gptr(a.pcnt)[(int64_t)si * a.T_cols + j]) : -1;
  const T* __restrict__ src = pc < 0 ? gptr(a.theta) + j * a.ld : gptr(a.nbv) + ((size_t)par * a.M + m) * R;
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int r = rbase + ((k / VEC) * LNT + tt) * VEC + (k % VEC);
    th[k] = r < R ? src[r] : T(0);
  }
  if (pc > 0) {
    const int lane = threadIdx.x & 63;
    const int pr = lane < pc ? gptr(a.prow)[h * a.cap + lane] : 0;
    const T pv = lane < pc ? gptr(a.pval)[h * a.cap + lane] : T(0);
    apply_patches<T, VPT, VEC>(pc, pr, pv, rbase, tt, th);
  }
}

// The candidates of one sub-tile's column: entries w > thr of the wave's
// lanes into the slots at h*cap, in slot-major order inside the wave (position
// = candidates of earlier slots + earlier lanes of this slot; rows past R have
// w = -inf and are never candidates).  Returns their number.  With none (q_s
// below the rounding of w, or the bound), slot 0 names a row of the maximum,
// for long_limit_kernel.
template <typename T, int VPT, typename Row>
__device__ __forceinline__ int keep_candidates(const LongArgs<T>& a, int64_t h, const double (&w)[VPT],
                                               Row&& row, double mx, double thr, bool any) {
  int32_t* const crow = gptr(a.crow) + h * a.cap;
  double* const cw = gptr(a.cw) + h * a.cap;
  int n = 0;
  if (any) {
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      const bool sel = w[k] > thr;
      const unsigned long long bal = __ballot(sel);
      if (sel) {
        const int pos = n + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
        if (pos < a.cap) {
          crow[pos] = row(k);
          cw[pos] = w[k];
        }
      }
      n += __popcll(bal);
    }
    if (n == 0) {
#pragma unroll
      for (int k = 0; k < VPT; ++k)
        if (w[k] == mx) crow[0] = row(k);
    }
  }
  return n;
}

// ---- scan: w, sub-tile maxima, candidates -------------------------------
// The dense plans: every iteration of the dense store, the first one of a
// call with the sparse store (spar[1]).  GRID: the cost is formed from the
// row's grid point and the column's point instead of being read (only theta
// is streamed).
template <typename T, int VPT, int VEC, bool GRID>
__global__ void __launch_bounds__(LNT)
long_scan_kernel(LongArgs<T> a) {
  constexpr int NCH = VPT / VEC, RB = LNT * VPT;
  // columns in flight per wave: two where the registers allow it at two
  // waves per SIMD (FP32 tiles of 16 values in vectors), else one
  constexpr int PF = (sizeof(T) == 4 && VPT == 16 && VEC > 1) ? 2 : 1;
  static_assert(VPT % VEC == 0 && VPT <= 16, "tile shape");
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  if (a.sparse && uniform_i(gptr(a.spar)[1]) == 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = uniform_i(tid >> 6);
  const int R = a.R, nsub = a.nrb * 4;
  const double t = uniform_d(*gptr(a.t)), inv_rho = a.inv_rho;
  const T* const theta = gptr(a.theta);
  const T* const qv = gptr(a.q);
  const int ib = uniform_i(a.wg_it[blockIdx.x]), ie = uniform_i(a.wg_it[blockIdx.x + 1]);
  for (int it = ib; it < ie; ++it) {
    const int rb = uniform_i(a.it_rb[it]), m = uniform_i(a.it_m[it]);
    const int64_t j0 = uniform_l(a.it_j0[it]), j1 = uniform_l(a.it_j1[it]);
    const double Sm = uniform_d(gptr(a.Sd)[m]);
    const int64_t off_m = uniform_l(gptr(a.col_off)[m]);
    const double* __restrict__ pmm = gptr(a.pm) + (size_t)m * R;
    const double* __restrict__ pv = gptr(a.p);
    const int rbase = rb * RB;
    int row[VPT];
    // 2 b_r, or -inf for rows past R: their w is then -inf (theta and c are
    // finite), below every threshold, without a select per entry
    double b2[VPT];
    double gx0[GRID ? VPT : 1], gx1[GRID ? VPT : 1];  // grid coordinates of the rows
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      row[k] = rbase + ((k / VEC) * LNT + tid) * VEC + (k % VEC);
      b2[k] = row[k] < R ? 2.0 * long_b(t, pv, pmm, row[k], Sm) : -__builtin_huge_val();
      if constexpr (GRID) {
        const int i0 = row[k] / a.gn1;
        gx0[k] = grid_coord(a, 0, i0);
        gx1[k] = grid_coord(a, 1, row[k] - i0 * a.gn1);
      }
    }
    // raw theta and c (or the column's point) of the next PF columns in
    // flight while one is scanned: PF buffers, used in turn
    T rt[PF][VPT], rc[PF][GRID ? 1 : VPT], rq[PF];
    double rz[PF][2];
    auto issue = [&](auto S, int64_t j) {
      constexpr int s = decltype(S)::value;
      const T* __restrict__ thp = theta + j * a.ld;
      rq[s] = qv[j];
      if constexpr (GRID) grid_point(a, j, off_m, &rz[s][0], &rz[s][1]);
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int r0 = row[c * VEC] < R ? row[c * VEC] : rbase;  // rows past R read the tile's first (masked)
        T tv[VEC];
        load_vec_nt<T, VEC>(thp + r0, tv);
#pragma unroll
        for (int v = 0; v < VEC; ++v) rt[s][c * VEC + v] = tv[v];
        if constexpr (!GRID) {
          T cv[VEC];
          load_vec<T, VEC>(long_cost_col(a, j, off_m) + r0, cv);
#pragma unroll
          for (int v = 0; v < VEC; ++v) rc[s][c * VEC + v] = cv[v];
        }
      }
    };
    // scan column j from buffer S; with NEXT, load column min(j + PF, j1 - 1)
    // into that buffer (past the item's end it loads its last column again:
    // unconditional loads keep the buffers in place across iterations)
    auto column = [&](auto S, auto NEXT, int64_t j) {
      constexpr int s = decltype(S)::value;
      double w[VPT];
      double mx = -__builtin_huge_val();
      const double z0 = uniform_d(rz[s][0]), z1 = uniform_d(rz[s][1]);
#pragma unroll
      for (int k = 0; k < VPT; ++k) {
        double c;
        if constexpr (GRID) c = grid_cost_xy<T>(gx0[k], gx1[k], z0, z1);
        else c = (double)rc[s][k];
        w[k] = long_w((double)rt[s][k], b2[k], c, inv_rho);
        mx = fmax(mx, w[k]);
      }
      const double tau = uniform_d((double)rq[s]);
      if constexpr (decltype(NEXT)::value) issue(S, j + PF < j1 ? j + PF : j1 - 1);
      mx = wave_max(mx);
      const int64_t h = j * nsub + rb * 4 + wv;
      const int n = keep_candidates<T, VPT>(a, h, w, [&](int k) { return row[k]; }, mx, mx - tau, tau > 0.0);
      if (lane == 0) {
        gptr(a.hmax)[h] = mx;
        gptr(a.hcnt)[h] = n;
      }
    };
    using YES = std::true_type;
    using NO = std::false_type;
    // buffer i holds column j + i (clamped to the item's last column)
    static_for<PF>([&](auto I) { issue(I, j0 + I < j1 ? j0 + I : j1 - 1); });
    int64_t j = j0;
    for (; j + PF - 1 < j1; j += PF) static_for<PF>([&](auto I) { column(I, YES{}, j + I); });
    static_for<PF - 1>([&](auto I) {
      if (j + I < j1) column(I, NO{}, j + I);
    });
  }
}

// The sparse plans: the columns of the work list (long_limit_kernel), an
// entry being up to kScanCols columns of one sub-tile and group of 64 that
// long_limit_kernel did not rule out.  An unpatched entry of a sparse
// sub-tile has theta = the common value, so theta + 2b is a per-row constant
// ('base', formed once per iteration) and w costs one fused multiply-add.
// Waves take the entries in turn: the columns left gather in the few
// sub-tiles that carry the barycenter, and with fixed shares of the columns
// the waves of those took 0.32 ms of an iteration on 40 x 40 images.  Which
// wave scans a column changes nothing: its header and slots are its own.
template <typename T, int VPT, int VEC, bool GRID>
__global__ void __launch_bounds__(LNT, 3)
long_scan_sparse_kernel(LongArgs<T> a) {
  constexpr int RB = LNT * VPT;
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  const int lane = threadIdx.x & 63;
  const int R = a.R, cap = a.cap, nsub = a.nrb * 4;
  const double inv_rho = a.inv_rho;
  const int count = uniform_i(gptr(a.spar)[2]), step = (int)gridDim.x * 4;
  for (int i = (int)blockIdx.x * 4 + uniform_i((int)(threadIdx.x >> 6)); i < count; i += step) {
    const int si = uniform_i(gptr(a.wsub)[i]);
    const int64_t jlo = (int64_t)uniform_i(gptr(a.wgrp)[i]) * 64;
    unsigned long long todo = (unsigned long long)uniform_l((int64_t)gptr(a.wcol)[i]);
    const int rb = si >> 2, tid = (si & 3) * 64 + lane, rbase = rb * RB;
    // lane l: measure, patch count, weight, bound and point of column jlo + l
    const int64_t jl = jlo + lane < a.T_cols ? jlo + lane : a.T_cols - 1;
    const int ml = gptr(a.colm)[jl], pcl = gptr(a.pcnt)[(int64_t)si * a.T_cols + jl];
    const double tl = (double)gptr(a.q)[jl], ll = gptr(a.limit)[jl];
    const int64_t offl = gptr(a.col_off)[ml];
    double zl0 = 0.0, zl1 = 0.0;
    if constexpr (GRID) grid_point(a, jl, offl, &zl0, &zl1);
    int m = -1;
    constexpr int NCH = VPT / VEC;
    double base[VPT];
    size_t o = 0;
    auto row = [&](int k) { return rbase + ((k / VEC) * LNT + tid) * VEC + (k % VEC); };
    // grid indices of each vector's first row (all rows' coordinates would be
    // 64 registers, and with them one wave per SIMD)
    int gi0[GRID ? NCH : 1], gi1[GRID ? NCH : 1];
    if constexpr (GRID) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        gi0[c] = row(c * VEC) / a.gn1;
        gi1[c] = row(c * VEC) - gi0[c] * a.gn1;
      }
    }
    // one column ahead: its costs and, in lane e, row and parts of w of patch e
    T rc[GRID ? 1 : VPT], pvv = T(0), pcv = T(0);
    int pr = 0;
    double pb2 = 0.0;
    auto issue = [&](int l) {
      const int64_t j = jlo + l, h = j * nsub + si;
      const int np = __builtin_amdgcn_readlane(pcl, l);
      if (lane < np) {
        pr = gptr(a.prow)[h * cap + lane];
        pvv = gptr(a.pval)[h * cap + lane];
        const size_t om = ((size_t)__builtin_amdgcn_readlane(ml, l) * a.nrb + rb) * VPT * LNT;
        pb2 = gptr(a.b2v)[om + slot_of(pr - rbase, VEC) * LNT + slot_owner(pr - rbase, VEC)];
        if constexpr (!GRID) pcv = long_cost_col(a, j, gptr(a.col_off)[__builtin_amdgcn_readlane(ml, l)])[pr];
      }
      if constexpr (!GRID) {
        const T* const cp = long_cost_col(a, j, uniform_l(gptr(a.col_off)[__builtin_amdgcn_readlane(ml, l)]));
#pragma unroll
        for (int c = 0; c < VPT / VEC; ++c) {
          T cv[VEC];
          load_vec<T, VEC>(cp + (row(c * VEC) < R ? row(c * VEC) : rbase), cv);
#pragma unroll
          for (int v = 0; v < VEC; ++v) rc[c * VEC + v] = cv[v];
        }
      }
    };
    issue(__builtin_ctzll(todo));
    while (todo != 0ull) {
      const int l = __builtin_ctzll(todo);
      const int64_t j = jlo + l;
      todo &= todo - 1ull;
      if (__builtin_amdgcn_readlane(ml, l) != m) {
        m = __builtin_amdgcn_readlane(ml, l);
        o = ((size_t)m * a.nrb + rb) * VPT * LNT + tid;
#pragma unroll
        for (int k = 0; k < VPT; ++k) base[k] = gptr(a.basev)[o + k * LNT];
      }
      const double z0 = read_lane(zl0, l), z1 = read_lane(zl1, l), tau = read_lane(tl, l), lim = read_lane(ll, l);
      const int np = __builtin_amdgcn_readlane(pcl, l), prs = pr;
      const double pw = lane < np ? long_w((double)pvv, pb2, GRID ? grid_cost(a, pr, z0, z1) : (double)pcv, inv_rho) : 0.0;
      double w[VPT], mx = -__builtin_huge_val();
      // f(k, c) for every slot's cost
      auto costs = [&](auto&& f) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          int i0 = GRID ? gi0[c] : 0, i1 = GRID ? gi1[c] : 0;
          // (keeps the compiler from holding every row's coordinates over the
          // columns after all)
          if constexpr (GRID) asm volatile("" : "+v"(i0), "+v"(i1));
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            if constexpr (GRID) {
              f(c * VEC + v, grid_cost_xy<T>(grid_coord(a, 0, i0), grid_coord(a, 1, i1), z0, z1));
              const bool wrap = ++i1 == a.gn1;
              i0 += wrap ? 1 : 0;
              i1 = wrap ? 0 : i1;
            } else {
              f(c * VEC + v, (double)rc[c * VEC + v]);
            }
          }
        }
      };
      if (np >= 0) {
        costs([&](int kk, double c) { w[kk] = __builtin_fma(-c, inv_rho, base[kk]); });
        // the patched rows
        for (int e = 0; e < np; ++e) {
          const int rr = __builtin_amdgcn_readlane(prs, e) - rbase;
          const double v = read_lane(pw, e);
          const int kp = slot_owner(rr, VEC) == tid ? slot_of(rr, VEC) : -1;
#pragma unroll
          for (int kk = 0; kk < VPT; ++kk) w[kk] = kk == kp ? v : w[kk];
        }
      } else {
        const T* const thp = gptr(a.theta) + j * a.ld;
        costs([&](int kk, double c) {
          w[kk] = long_w((double)thp[row(kk) < R ? row(kk) : rbase], gptr(a.b2v)[o + kk * LNT], c, inv_rho);
        });
      }
#pragma unroll
      for (int kk = 0; kk < VPT; ++kk) mx = fmax(mx, w[kk]);
      const int64_t h = j * nsub + si;
      if (todo != 0ull) issue(__builtin_ctzll(todo));
      mx = wave_max(mx);
      // (an entry at or below the column's bound is inactive too)
      const int n = keep_candidates<T, VPT>(a, h, w, row, mx, fmax(mx - tau, lim), tau > 0.0);
      if (lane == 0) {
        gptr(a.hmax)[h] = mx;
        gptr(a.hcnt)[h] = n;
      }
    }
  }
}

// x of the lanes in bal, the i-th of them moved to lane (first + i) mod 64.
__device__ __forceinline__ double rank_lane(unsigned long long bal, int first, double x) {
  const int lane = threadIdx.x & 63;
  const int up = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
  const int to = ((bal >> lane) & 1ull) ? first + up : first + __popcll(bal) + lane - up;  // a permutation
  const int lo = __builtin_amdgcn_ds_permute((to & 63) * 4, __double2loint(x));
  const int hi = __builtin_amdgcn_ds_permute((to & 63) * 4, __double2hiint(x));
  return __hiloint2double(hi, lo);
}

// ---- threshold: one wave per column -------------------------------------
// Only sub-tiles with w_loc > w_max - q_s are visited, in index order; inside
// one, lane e takes kept entry e, or (more than E candidates) lane l
// recomputes the VPT values of thread 64*wave + l of the tile.  The entries
// above the threshold are dealt to the lanes by their rank in the column and
// summed in a fixed tree: the sum depends on which entries are active and not
// on which others were kept.
template <typename T, int VPT, int VEC, bool DIAG, bool SP>
__global__ void __launch_bounds__(256)
long_threshold_kernel(LongArgs<T> a) {
  constexpr int RB = LNT * VPT, LW = 256;
  __shared__ double s_list[4][LW];
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  const int lane = threadIdx.x & 63;
  const int64_t j = (int64_t)blockIdx.x * 4 + uniform_i(threadIdx.x >> 6);
  if (j >= a.T_cols) return;  // whole waves; no barriers below
  const int R = a.R, cap = a.cap, nsub = a.nrb * 4;
  const double tau = uniform_d((double)gptr(a.q)[j]);
  double* const lamv = gptr(a.lam);
  if (!(tau > 0.0)) {
    if (lane == 0) {
      lamv[j] = __builtin_huge_val();  // q_s = 0: the column is 0
      if constexpr (DIAG) {
        double* const dj = gptr(a.ldiag) + j * 4;
        dj[0] = dj[1] = dj[2] = dj[3] = 0.0;
      }
    }
    return;
  }
  const double* __restrict__ hm = gptr(a.hmax) + j * nsub;
  const int32_t* __restrict__ hc = gptr(a.hcnt) + j * nsub;
  const double* __restrict__ cwj = gptr(a.cw) + j * nsub * (int64_t)cap;
  double wmx = -__builtin_huge_val();
  // sparse store: only the sub-tiles that the scan looked at have a header
  const unsigned long long* const smk = SP ? gptr(a.smask) + j * a.nmask : nullptr;
  auto looked = [&](int s) -> bool { return s < nsub && (smk == nullptr || ((smk[s >> 6] >> (s & 63)) & 1ull)); };
  for (int s = lane; s < nsub; s += 64)
    if (looked(s)) wmx = fmax(wmx, hm[s]);
  wmx = wave_max(wmx);
  // the root is >= w_max - tau, and >= the column's bound, below which the
  // sparse-store scan keeps no entry
  const double lo = SP ? fmax(wmx - tau, uniform_d(gptr(a.limit)[j])) : wmx - tau;
  // an overflowed sub-tile is recomputed from theta and c: the column's
  // measure and b
  int m = 0;
  while (m + 1 < a.M && gptr(a.col_off)[m + 1] <= j) ++m;
  const double t = uniform_d(*gptr(a.t));
  const double Sm = gptr(a.Sd)[m];
  const int64_t off_m = gptr(a.col_off)[m];
  const double* __restrict__ pmm = gptr(a.pm) + (size_t)m * R;
  const double* __restrict__ pv = gptr(a.p);
  const int par = SP ? uniform_i(*gptr(a.spar)) : 0;
  const T* __restrict__ cp = long_cost_col(a, j, off_m);
  double z0 = 0.0, z1 = 0.0;
  if (a.gdim) grid_point(a, j, off_m, &z0, &z1);
  auto costv = [&](int r) { return a.gdim ? grid_cost(a, r, z0, z1) : (double)cp[r]; };
  auto visit = [&](auto&& f) {
    for (int s0 = 0; s0 < nsub; s0 += 64) {
      const int s = s0 + lane;
      unsigned long long rel = __ballot(looked(s) && hm[s < nsub ? s : 0] > lo);
      while (rel) {
        const int si = s0 + __builtin_ctzll(rel);
        rel &= rel - 1;
        const int n = uniform_i(hc[si]);
        if (n <= cap) {
          const bool in = lane < n;
          f(in, in ? cwj[(int64_t)si * cap + lane] : 0.0,
            in ? gptr(a.crow)[(j * nsub + si) * (int64_t)cap + lane] : 0);
        } else {
          const int rbase = (si >> 2) * RB, tt = (si & 3) * 64 + lane;
          T th[VPT];
          stored_rows<T, VPT, VEC>(a, j, si, rbase, tt, m, par, th);
#pragma unroll
          for (int k = 0; k < VPT; ++k) {
            const int r = rbase + ((k / VEC) * LNT + tt) * VEC + (k % VEC);
            const int rl = r < R ? r : rbase;
            // (long_base_kernel's 2 b with the sparse store)
            const double b2 = SP ? gptr(a.b2v)[(((size_t)m * a.nrb + (si >> 2)) * VPT + k) * LNT + tt]
                                       : 2.0 * long_b(t, pv, pmm, rl, Sm);
            f(r < R, long_w((double)th[k], b2, costv(rl), a.inv_rho), r);
          }
        }
      }
    }
  };
  // The kept entries of every sub-tile that counts, in order, in LDS: lane l
  // copies those of sub-tile s0 + l.  Columns with more than LW of them, or
  // with an overflowed sub-tile, read them again in every round.
  double* const list = s_list[threadIdx.x >> 6];
  int nlist = 0, wrow = -1;
  for (int s0 = 0; s0 < nsub && nlist <= LW; s0 += 64) {
    const int s = s0 + lane;
    const bool rel = looked(s) && hm[s < nsub ? s : 0] > lo;
    const int n = rel ? hc[s] : 0;
    if (__ballot(n > cap) != 0ull) {
      nlist = LW + 1;
      break;
    }
    if (__ballot(rel) == 0ull) continue;
    int off = n;  // inclusive prefix sum over the lanes
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const int v = __shfl_up(off, d);
      if (lane >= d) off += v;
    }
    const int tot = __builtin_amdgcn_readlane(off, 63);
    off += nlist - n;
    nlist += tot;
    if (nlist > LW) break;
    const int64_t h0 = (int64_t)(s < nsub ? s : 0) * cap;
    for (int e0 = 0; __ballot(e0 < n) != 0ull; e0 += 4) {
      double x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = e0 + u < n ? cwj[h0 + e0 + u] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e0 + u < n) {
          list[off + e0 + u] = x[u];
          if (x[u] == wmx) wrow = gptr(a.crow)[j * nsub * (int64_t)cap + h0 + e0 + u];
        }
    }
  }
  wave_lds_sync();
  const double lprev = lamv[j];
  double lam = (a.warm && lprev == lprev && lprev > lo) ? lprev : lo;
  // a list made in a round holds the entries above that round's threshold
  // lfrom; mxout is the largest of the others
  double lfrom = -__builtin_huge_val(), mxout = -__builtin_huge_val();
  int nprev = -1, nrounds = 0, nact = 0;
  for (int round = 0; round < R + 4; ++round) {
    double S = 0.0, mnA = __builtin_huge_val(), mxN = mxout;
    int n = 0;
    const bool all = nlist > LW;  // every entry, read again
    if (all) {
      // each 64 entries above lam go through the list's LDS to the lanes
      visit([&](bool in, double x, int r) {
        if (in && x == wmx) wrow = r;
        const bool act = in && x > lam;
        const unsigned long long bal = __ballot(act);
        mnA = fmin(mnA, act ? x : __builtin_huge_val());
        mxN = fmax(mxN, in && !act ? x : -__builtin_huge_val());
        if (act) {
          const int pos = n + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
          list[pos & (LW - 1)] = x;
        }
        const int n0 = n & ~63;
        n += __popcll(bal);
        if ((n & ~63) != n0) {
          wave_lds_sync();
          S += list[(n0 & (LW - 1)) + lane];
          wave_lds_sync();
        }
      });
      wave_lds_sync();
      if (lane < (n & 63)) S += list[((n & ~63) & (LW - 1)) + lane];
    } else {
      for (int i = 0; i < nlist; i += 64) {
        const double x = list[i + lane < nlist ? i + lane : 0];
        const bool act = i + lane < nlist && x > lam;
        const unsigned long long bal = __ballot(act);
        mnA = fmin(mnA, act ? x : __builtin_huge_val());
        mxN = fmax(mxN, i + lane < nlist && !act ? x : -__builtin_huge_val());
        if (bal == 0ull) continue;
        const double y = rank_lane(bal, n, x);
        if (((lane - n) & 63) < __popcll(bal)) S += y;
        n += __popcll(bal);
      }
    }
    ++nrounds;
    S = wave_sum(S);
    mnA = wave_reduce<OpMin>(mnA);
    mxN = wave_max(mxN);
    if (n == 0) {
      if (lam > lo) {  // a warm start at or above w_max: restart from the bound
        lam = lo;
        nprev = -1;
        continue;
      }
      // w_max - tau rounded to w_max (tau below half an ulp): the column is 0
      lam = __builtin_huge_val();
      break;
    }
    const double ln = (S - tau) / (double)n;
    if (ln >= lo && (n == nprev || (mnA >= ln && mxN <= ln))) {
      // the set above lam is exactly the active set
      lam = ln;
      nact = n;
      break;
    }
    nprev = n;
    if (all && n <= LW) {  // they fit: the list from here on
      nlist = n;
      lfrom = lam;
      mxout = mxN;
    }
    lam = fmax(ln, lo);
    if (lam < lfrom) {  // (a warm start above the threshold): entries are missing
      nlist = LW + 1;
      lfrom = mxout = -__builtin_huge_val();
    }
  }
  // relaxed columns: max(w - max(lam, 0), 0) is the projection onto
  // {u >= 0, sum u <= q_s} (the write pass patches only entries above it)
  if (a.relaxed) lam = fmax(lam, 0.0);
  if (lane == 0) lamv[j] = lam;
  if (SP) {
    // the row of the column's maximum, for long_limit_kernel: a kept entry,
    // or (q_s below the rounding of w) slot 0 of a sub-tile that kept none
    const unsigned long long has = __ballot(wrow >= 0);
    if (has) {
      wrow = __builtin_amdgcn_readlane(wrow, __builtin_ctzll(has));
    } else {
      for (int s0 = 0; s0 < nsub; s0 += 64) {
        const int s = s0 + lane;
        const unsigned long long at = __ballot(looked(s) && hm[s < nsub ? s : 0] == wmx);
        if (at == 0ull) continue;
        const int si = s0 + __builtin_ctzll(at);
        if (uniform_i(hc[si]) == 0) wrow = uniform_i(gptr(a.crow)[(j * nsub + si) * (int64_t)cap]);
        break;
      }
    }
    if (lane == 0) gptr(a.wit)[j] = wrow;
  }
  if constexpr (DIAG) {
    // the column's pi_hat = max(w - lam, 0) at the same entries and in the
    // same arithmetic as the write pass: its sum against q_s and against the
    // cost (fixed order: sub-tiles in order, lanes by the wave sum)
    double cs = 0.0, wc = 0.0;
    if (lam < __builtin_huge_val()) {
      visit([&](bool in, double x, int r) {
        if (in && x > lam) {
          const double ph = fmax(x - lam, 0.0);
          cs += ph;
          wc += costv(r) * ph;
        }
      });
    }
    cs = wave_sum(cs);
    wc = wave_sum(wc);
    if (lane == 0) {
      double* const dj = gptr(a.ldiag) + j * 4;
      dj[0] = wc;
      dj[1] = a.relaxed ? fmax(cs - tau, 0.0) : fabs(cs - tau);
      dj[2] = (double)nrounds;
      dj[3] = (double)(lam < __builtin_huge_val() ? nact : 0);
    }
  }
}

// ---- write: theta' and the tile's row-sum partials ----------------------
// Usually a column's sub-tile is stored as -b in whole vectors, and the few
// kept entries above lambda are then patched by the thread that owns the
// row (its own earlier store to the same address comes first).  An
// overflowed sub-tile above lambda is done vector by vector instead: theta
// and c are read, w formed, and the patched vector stored in one go.  The
// thresholds and sub-tile headers of 256 columns at a time are loaded into
// LDS together (one column per thread), so no column waits on memory for
// them.  Dynamic LDS: VPT*256 doubles of row-sum patches (each row owned by
// one thread: no atomics).
template <typename T, int VPT, int VEC, bool DIAG>
__global__ void __launch_bounds__(LNT)
long_write_kernel(LongArgs<T> a) {
  constexpr int NCH = VPT / VEC, RB = LNT * VPT;
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  double dth = 0.0;  // DIAG, dense store: max |theta' - theta| of this thread's entries
  extern __shared__ double lds_dyn[];
  double* fix = lds_dyn;  // [VPT][256]
  constexpr int WB = 128;  // columns whose thresholds and headers are staged at once
  __shared__ double s_lam[WB], s_max[4][WB];
  __shared__ int s_cnt[4][WB];
  const int tid = threadIdx.x;
  const int wv = uniform_i(tid >> 6);
  const int R = a.R, cap = a.cap, nsub = a.nrb * 4;
  const double t = uniform_d(*gptr(a.t)), inv_rho = a.inv_rho;
  T* const theta = gptr(a.theta);
  const double* const hm = gptr(a.hmax);
  const int32_t* const hc = gptr(a.hcnt);
  const int32_t* const crow = gptr(a.crow);
  const double* const cw = gptr(a.cw);
  const double* const lamv = gptr(a.lam);
  const bool sparse = a.sparse != 0;
  const int par = sparse ? uniform_i(*gptr(a.spar)) : 0;
  // Sparse store.  A sub-tile that the scan left out of a column keeps its
  // patch count of 0, so only the columns of gmask's set bits need work, in
  // order and 64 at a time: lane l takes column l's header, compares its kept
  // entries with the threshold and stores the patches; the updates then go to
  // the row sums in column order, those of one row one after the other.
  // (Taken one column at a time, each with its own chain of loads, the 40 x 40
  // images took 0.27 ms: the patches gather in few tiles.)
  constexpr int LP = 256;  // updates of a batch
  __shared__ int s_col[4][128], s_slot[4][LP];
  __shared__ double s_upd[4][LP];
  auto write_sparse = [&](auto&& column, int rb, int64_t j0, int64_t j1, int rbase, double tt, double Sm,
                          const double* pv, const double* pmm) {
    const int lane = tid & 63, sub = rb * 4 + wv;
    int* const col = s_col[wv];
    int* const slot = s_slot[wv];
    double* const upd = s_upd[wv];
    auto batch = [&](int nc) {
      const bool in = lane < nc;
      const int64_t j = in ? col[lane] : j0;
      const int64_t h = j * nsub + sub;
      const double lam = lamv[j];
      const double lmax = in ? hm[h] : -__builtin_huge_val();
      const bool act = lmax > lam;
      const int n = act ? hc[h] : 0;
      int32_t* const pcj = gptr(a.pcnt) + (int64_t)sub * a.T_cols + j;
      if (in && !act) *pcj = 0;
      int kept = 0;
      const bool over = __ballot(n > cap) != 0ull;
      if (!over)
        for (int e0 = 0; __ballot(e0 < n) != 0ull; e0 += 4) {
          double x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = e0 + u < n ? cw[h * cap + e0 + u] : -__builtin_huge_val();
#pragma unroll
          for (int u = 0; u < 4; ++u) kept += x[u] > lam ? 1 : 0;
        }
      int off = kept;
#pragma unroll
      for (int d = 1; d < 64; d *= 2) {
        const int v = __shfl_up(off, d);
        if (lane >= d) off += v;
      }
      const int tot = __builtin_amdgcn_readlane(off, 63);
      if (over || tot > LP) {
        for (unsigned long long am = __ballot(act); am != 0ull; am &= am - 1ull) {
          const int l = __builtin_ctzll(am);
          column((int64_t)__builtin_amdgcn_readlane((int)j, l), read_lane(lam, l), read_lane(lmax, l),
                 __builtin_amdgcn_readlane(n, l));
        }
        return;
      }
      off -= kept;
      int pos = 0;
      for (int e0 = 0; __ballot(e0 < n) != 0ull; e0 += 4) {
        double x[4], b[4];
        int r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          x[u] = e0 + u < n ? cw[h * cap + e0 + u] : -__builtin_huge_val();
          r[u] = x[u] > lam ? crow[h * cap + e0 + u] : rbase;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = long_b(tt, pv, pmm, r[u], Sm);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (x[u] > lam) {
            const double d = fmax(x[u] - lam, 0.0);  // theta' - (-b) before rounding
            gptr(a.prow)[h * cap + pos] = r[u];
            gptr(a.pval)[h * cap + pos] = (T)(d - b[u]);
            const int rr = r[u] - rbase;
            slot[off + pos] = slot_of(rr, VEC) * LNT + slot_owner(rr, VEC);
            upd[off + pos] = d;
            ++pos;
          }
      }
      if (act) *pcj = kept;
      wave_lds_sync();
      for (int i0 = 0; i0 < tot; i0 += 64) {
        const int ni = tot - i0 < 64 ? tot - i0 : 64;
        const int sl = lane < ni ? slot[i0 + lane] : -1 - lane;
        int before = 0;  // earlier updates of the same row
        for (int l = 0; l + 1 < ni; ++l)
          before += (lane > l && __builtin_amdgcn_readlane(sl, l) == sl) ? 1 : 0;
        for (int k = 0; __ballot(lane < ni && before >= k) != 0ull; ++k) {
          if (lane < ni && before == k) fix[sl] += upd[i0 + lane];
          wave_lds_sync();
        }
      }
      wave_lds_sync();
    };
    int nc = 0;
    const int64_t g1 = (j1 + 63) >> 6;
    for (int64_t g0 = j0 >> 6; g0 < g1; g0 += 64) {
      unsigned long long word = g0 + lane < g1 ? gptr(a.gmask)[(int64_t)sub * a.ngrp + g0 + lane] : 0ull;
      for (unsigned long long some = __ballot(word != 0ull); some != 0ull; some &= some - 1ull) {
        const int l = __builtin_ctzll(some);
        const int64_t j = ((g0 + l) << 6) + lane;
        const unsigned long long w = (unsigned long long)__double_as_longlong(read_lane(__longlong_as_double((long long)word), l));
        const unsigned long long bits = __ballot(((w >> lane) & 1ull) && j >= j0 && j < j1);
        if ((bits >> lane) & 1ull)
          col[nc + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bits >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((unsigned)bits, 0u))] = (int)j;
        nc += __popcll(bits);
        wave_lds_sync();
        if (nc >= 64) {
          batch(64);
          nc -= 64;
          const int v = lane < nc ? col[64 + lane] : 0;
          wave_lds_sync();
          if (lane < nc) col[lane] = v;
          wave_lds_sync();
        }
      }
    }
    if (nc > 0) batch(nc);
    wave_lds_sync();
  };
  const int ib = uniform_i(a.wg_it[blockIdx.x]), ie = uniform_i(a.wg_it[blockIdx.x + 1]);
  for (int it = ib; it < ie; ++it) {
    const int rb = uniform_i(a.it_rb[it]), m = uniform_i(a.it_m[it]);
    const int64_t j0 = uniform_l(a.it_j0[it]), j1 = uniform_l(a.it_j1[it]);
    const double Sm = uniform_d(gptr(a.Sd)[m]);
    const int64_t off_m = uniform_l(gptr(a.col_off)[m]);
    const double* __restrict__ pmm = gptr(a.pm) + (size_t)m * R;
    const double* __restrict__ pv = gptr(a.p);
    const int rbase = rb * RB;
    const int sub = rb * 4 + wv;
    auto row = [&](int k) { return rbase + ((k / VEC) * LNT + tid) * VEC + (k % VEC); };
    // b of slot k's row (sparse store: half the 2 b that long_base_kernel left)
    const size_t o2 = ((size_t)m * a.nrb + rb) * VPT * LNT + tid;
    auto b_of = [&](int k) {
      const double v = sparse ? 0.5 * gptr(a.b2v)[o2 + k * LNT] : long_b(t, pv, pmm, row(k) < R ? row(k) : rbase, Sm);
      return row(k) < R ? v : 0.0;
    };
    T nb[VPT];  // -b rounded to the storage type: every inactive entry's new value
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      nb[k] = (T)(-b_of(k));
      fix[k * LNT + tid] = 0.0;  // each thread touches only its own slots
    }
    // sparse store: the tile's new common values of measure m, written once
    // (by the item that starts at the measure's first column) into the half
    // of nbv the stored plans do not use yet
    if (sparse && j0 == off_m) {
      T* __restrict__ nbn = gptr(a.nbv) + ((size_t)(par ^ 1) * a.M + m) * R;
#pragma unroll
      for (int k = 0; k < VPT; ++k)
        if (row(k) < R) nbn[row(k)] = nb[k];
    }
    const T* __restrict__ nbo = sparse ? gptr(a.nbv) + ((size_t)par * a.M + m) * R : nullptr;
    auto column = [&](int64_t j, double lam, double lmax, int n) {
      T* __restrict__ thp = theta + j * a.ld;
      const bool some = lmax > lam;  // some entry of this sub-tile is active
      const int64_t h = j * nsub + sub;
      int32_t* const pcj = sparse ? gptr(a.pcnt) + (int64_t)sub * a.T_cols + j : nullptr;
      if (some && n > cap) {
        // more candidates than slots: vector by vector, w from theta and c
        // (one vector at a time, so this rare path holds few registers); the
        // stored plans of a sparse sub-tile are the common values and its
        // patches, and the sub-tile is dense in theta afterwards
        const T* __restrict__ cp = long_cost_col(a, j, off_m);
        double z0 = 0.0, z1 = 0.0;
        if (a.gdim) grid_point(a, j, off_m, &z0, &z1);
        const int pc = sparse ? uniform_i(*pcj) : -1;
        const int lane = tid & 63;
        const int pr = lane < pc ? gptr(a.prow)[h * cap + lane] : 0;
        const T pvv = lane < pc ? gptr(a.pval)[h * cap + lane] : T(0);
        // stored values tv, b and w of vector c (w = -inf past R)
        auto vec_w = [&](int c, T (&tv)[VEC], double (&bk)[VEC], double (&w)[VEC]) {
          const int r0 = rbase + (c * LNT + tid) * VEC;
          const int rl = r0 < R ? r0 : rbase;  // rows past R read the tile's first (masked)
          if (pc < 0) {
            load_vec<T, VEC>(thp + rl, tv);
          } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) tv[v] = r0 + v < R ? nbo[r0 + v] : T(0);
            for (int e = 0; e < pc; ++e) {
              const int rr = __builtin_amdgcn_readlane(pr, e) - rbase;
              const T val = read_lane(pvv, e);
              if (slot_owner(rr, VEC) == tid && slot_of(rr, VEC) / VEC == c) {
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                  if (v == rr % VEC) tv[v] = val;
              }
            }
          }
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            const int rv = r0 + v < R ? r0 + v : rbase;
            bk[v] = sparse ? 0.5 * gptr(a.b2v)[o2 + (c * VEC + v) * LNT] : long_b(t, pv, pmm, rv, Sm);
            const double cc = a.gdim ? grid_cost(a, rv, z0, z1) : (double)cp[rv];
            w[v] = r0 + v < R ? long_w((double)tv[v], 2.0 * bk[v], cc, inv_rho) : -__builtin_huge_val();
          }
        };
        if (sparse) {
          // no more active entries than slots (the usual case: the slots ran
          // out of candidates, not of active entries): patches
          int na = 0;
#pragma unroll 1
          for (int c = 0; c < NCH; ++c) {
            T tv[VEC];
            double bk[VEC], w[VEC];
            vec_w(c, tv, bk, w);
#pragma unroll
            for (int v = 0; v < VEC; ++v) na += __popcll(__ballot(w[v] > lam));
          }
          if (na <= cap) {
            int pos = 0;
#pragma unroll 1
            for (int c = 0; c < NCH; ++c) {
              T tv[VEC];
              double bk[VEC], w[VEC];
              vec_w(c, tv, bk, w);
#pragma unroll
              for (int v = 0; v < VEC; ++v) {
                const unsigned long long bal = __ballot(w[v] > lam);
                if (w[v] > lam) {
                  const int e = pos + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
                  const double ph = fmax(w[v] - lam, 0.0);
                  gptr(a.prow)[h * cap + e] = row(c * VEC + v);
                  gptr(a.pval)[h * cap + e] = (T)(ph - bk[v]);
                  fix[(c * VEC + v) * LNT + tid] += ph;
                }
                pos += __popcll(bal);
              }
            }
            if (lane == 0) *pcj = na;
            return;
          }
        }
#pragma unroll 1
        for (int c = 0; c < NCH; ++c) {
          const int r0 = rbase + (c * LNT + tid) * VEC;
          T tv[VEC], out[VEC];
          double bk[VEC], w[VEC];
          vec_w(c, tv, bk, w);
#pragma unroll
          for (int v = 0; v < VEC; ++v) {
            out[v] = T(0);  // rows past R are not stored
            if (r0 + v < R) {
              out[v] = (T)(-bk[v]);  // the entry's value when inactive (nb of its slot)
              if (w[v] > lam) {
                const double ph = fmax(w[v] - lam, 0.0);
                out[v] = (T)(ph - bk[v]);
                fix[(c * VEC + v) * LNT + tid] += ph;  // theta' - (-b) before rounding
              }
            }
          }
          if constexpr (DIAG) {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
              if (r0 + v < R) dth = fmax(dth, fabs((double)out[v] - (double)tv[v]));
          }
          if (r0 + VEC <= R) {
            store_vec_nt<T, VEC>(thp + r0, out);
          } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
              if (r0 + v < R) thp[r0 + v] = out[v];
          }
        }
        if (sparse && lane == 0) *pcj = -1;
        return;
      }
      // DIAG, dense store: the entries' old values, and which of them the
      // patches below overwrite
      T old[VPT];
      unsigned pmask = 0u;
      if constexpr (DIAG) {
        if (!sparse) {
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            const int r0 = row(c * VEC);
            T ov[VEC];
            if (r0 + VEC <= R) {
              load_vec<T, VEC>(thp + r0, ov);
            } else {
#pragma unroll
              for (int v = 0; v < VEC; ++v) ov[v] = r0 + v < R ? thp[r0 + v] : T(0);
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) old[c * VEC + v] = ov[v];
          }
        }
      }
      if (!sparse) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const int r0 = row(c * VEC);
          T out[VEC];
#pragma unroll
          for (int v = 0; v < VEC; ++v) out[v] = nb[c * VEC + v];
          if (r0 + VEC <= R) {
            store_vec_nt<T, VEC>(thp + r0, out);
          } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
              if (r0 + v < R) thp[r0 + v] = out[v];
          }
        }
      }
      if (some) {
        // the kept entries above lambda (n <= cap <= 64): lane e reads entry
        // e and forms its patch, all at once; then, in entry order, the
        // owner of each row stores it (or, with the sparse store, the
        // patches are kept in slots) and adds it to the row sum
        const int e = tid & 63;
        const double xe = e < n ? cw[h * cap + e] : -__builtin_huge_val();
        const int re = e < n ? crow[h * cap + e] : rbase;
        const bool keep = xe > lam;
        const double bk = keep ? long_b(t, pv, pmm, re, Sm) : 0.0;
        const double dfix = fmax(xe - lam, 0.0);  // theta' - (-b) before rounding
        const T val = (T)(dfix - bk);
        unsigned long long sel = __ballot(keep);
        if (sparse) {
          const int pos = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(sel >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((unsigned)sel, 0u));
          if (keep) {
            gptr(a.prow)[h * cap + pos] = re;
            gptr(a.pval)[h * cap + pos] = val;
          }
          if (e == 0) *pcj = __popcll(sel);
        }
        while (sel != 0ull) {
          const int l = __builtin_ctzll(sel);
          sel &= sel - 1ull;
          const int rr = __builtin_amdgcn_readlane(re, l) - rbase;
          if (slot_owner(rr, VEC) == tid) {
            if (!sparse) thp[rbase + rr] = read_lane(val, l);
            fix[slot_of(rr, VEC) * LNT + tid] += read_lane(dfix, l);
            if constexpr (DIAG) {
              if (!sparse) {
                const int sl = slot_of(rr, VEC);
                const double nv = (double)read_lane(val, l);
#pragma unroll
                for (int k = 0; k < VPT; ++k)
                  if (k == sl) dth = fmax(dth, fabs(nv - (double)old[k]));
                pmask |= 1u << sl;
              }
            }
          }
        }
      }
      if constexpr (DIAG) {
        // every other entry of the sub-tile became -b
        if (!sparse) {
#pragma unroll
          for (int k = 0; k < VPT; ++k)
            if (row(k) < R && !((pmask >> k) & 1u)) dth = fmax(dth, fabs((double)nb[k] - (double)old[k]));
        }
      }
    };
    if (sparse) {
      write_sparse(column, rb, j0, j1, rbase, t, Sm, pv, pmm);
    } else {
      for (int64_t jb = j0; jb < j1; jb += WB) {
        // thresholds and this tile's four sub-tile headers of WB columns
        __syncthreads();  // the previous block's readers are done
        if (tid < WB && jb + tid < j1) {
          const int64_t jj = jb + tid;
          s_lam[tid] = lamv[jj];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            s_max[q][tid] = hm[jj * nsub + rb * 4 + q];
            s_cnt[q][tid] = hc[jj * nsub + rb * 4 + q];
          }
        }
        __syncthreads();
        const int64_t je = jb + WB < j1 ? jb + WB : j1;
        for (int64_t j = jb; j < je; ++j)
          column(j, uniform_d(s_lam[j - jb]), uniform_d(s_max[wv][j - jb]), uniform_i(s_cnt[wv][j - jb]));
      }
    }
    // the item's row sums: (#columns) * (-b) plus the patches, in double
    // from the unrounded updates (as in the short column kernel: the stored
    // -b of the inactive entries would add the same rounding error from
    // every column of the measure)
    const double ncols = (double)(j1 - j0);
    double* __restrict__ part = gptr(a.partial) + uniform_l(a.it_poff[it]);
#pragma unroll
    for (int k = 0; k < VPT; ++k)
      if (row(k) < R) part[row(k) - rbase] = fix[k * LNT + tid] - ncols * b_of(k);
  }
  if constexpr (DIAG) {
    __shared__ double sh_dth[4];
    const double m = wave_max(dth);
    if ((tid & 63) == 0) sh_dth[tid >> 6] = m;
    __syncthreads();
    if (tid == 0)
      gptr(a.wdiag)[(size_t)blockIdx.x * DIAG_STRIDE + 2] =
          sparse ? __builtin_nan("") : fmax(fmax(sh_dth[0], sh_dth[1]), fmax(sh_dth[2], sh_dth[3]));
  }
}

// Row sums of the plans into the item partials (initialisation).  OWN: the
// plans are the library's own start, (T)(q_s/R) in every row of column s, so
// every row of an item has the same sum, taken over its columns in the same
// order without reading the plans (9.8 GB of them took 8.0 ms).
template <typename T, bool OWN>
__global__ void __launch_bounds__(256)
long_rowsum_kernel(LongArgs<T> a, int rows_per_tile) {
  const int ib = a.wg_it[blockIdx.x], ie = a.wg_it[blockIdx.x + 1];
  for (int it = ib; it < ie; ++it) {
    const int rbase = a.it_rb[it] * rows_per_tile;
    const int rend = rbase + rows_per_tile < a.R ? rbase + rows_per_tile : a.R;
    if constexpr (OWN) {
      constexpr int U = 16;
      const int64_t j0 = a.it_j0[it], j1 = a.it_j1[it];
      double s = 0.0;
      for (int64_t j = j0; j < j1; j += U) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = (double)(T)((double)a.q[j + u < j1 ? j + u : j0] / (double)a.R);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (j + u < j1) s += x[u];
      }
      for (int r = rbase + threadIdx.x; r < rend; r += 256) a.partial[a.it_poff[it] + (r - rbase)] = s;
      continue;
    }
    for (int r = rbase + threadIdx.x; r < rend; r += 256) {
      double s = 0.0;
      for (int64_t j = a.it_j0[it]; j < a.it_j1[it]; ++j) s += (double)a.theta[j * a.ld + r];
      a.partial[a.it_poff[it] + (r - rbase)] = s;
    }
  }
}

// ---- sparse store: what the scan can leave out ---------------------------
// Least cost of every (sub-tile, cost column), once per call: the cost of a
// call does not change.  A workgroup takes one row tile and 16 cost columns.
template <typename T, int VPT, int VEC, bool GRID>
__global__ void __launch_bounds__(LNT)
long_cost_min_kernel(LongArgs<T> a) {
  constexpr int RB = LNT * VPT;
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform_i(tid >> 6);
  const int R = a.R, rb = blockIdx.x, rbase = rb * RB;
  int row[VPT];
  double gx0[GRID ? VPT : 1], gx1[GRID ? VPT : 1];
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    row[k] = rbase + ((k / VEC) * LNT + tid) * VEC + (k % VEC);
    if constexpr (GRID) {
      const int i0 = row[k] / a.gn1;
      gx0[k] = grid_coord(a, 0, i0);
      gx1[k] = grid_coord(a, 1, row[k] - i0 * a.gn1);
    }
  }
  const int64_t c0 = a.c_first + (int64_t)blockIdx.y * 16;
  const int64_t c1 = c0 + 16 < a.ncost ? c0 + 16 : a.ncost;
  for (int64_t c = c0; c < c1; ++c) {
    double z0 = 0.0, z1 = 0.0;
    if constexpr (GRID) grid_point(a, c, 0, &z0, &z1);
    double mn = __builtin_huge_val();
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      double v;
      if constexpr (GRID) v = grid_cost_xy<T>(gx0[k], gx1[k], z0, z1);
      else v = (double)a.cost[c * a.cost_ld + (row[k] < R ? row[k] : rbase)];
      if (row[k] < R) mn = fmin(mn, v);
    }
    mn = wave_reduce<OpMin>(mn);
    if (lane == 0) gptr(a.cmin)[(int64_t)(rb * 4 + wv) * a.ncost + c] = (T)mn;
  }
}

// A lower bound of every column's threshold for the iteration to come.  With
// the sums taken over the column's patches alone (its last active entries),
// (sum w - q_s)/n is one Newton step of Prop. 3 from below, hence at most the
// threshold of those entries, hence at most the column's; so is w - q_s of any
// single entry.  A column without patches (no active entry, or a sub-tile that
// overflowed its slots) uses the row of its last maximum, whose stored value
// is at least the one read here.  A margin of 2^-40 of the magnitudes covers the rounding.  One
// thread per (column, 1/kLimitWaves of the sub-tiles), 64 columns per workgroup:
// the counts are stored with the column index fastest.  Then the sub-tiles of
// each column to scan, as masks and as the scan's work list.
template <typename T, int VPT, int VEC>
__global__ void __launch_bounds__(64 * kLimitWaves)
long_limit_kernel(LongArgs<T> a) {
  constexpr int RB = LNT * VPT;
  __shared__ double s_top[kLimitWaves][64], s_sum[kLimitWaves][64];
  __shared__ int s_n[kLimitWaves][64];
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  const int lane = threadIdx.x & 63, q = uniform_i((int)(threadIdx.x >> 6));
  const int64_t j = (int64_t)blockIdx.x * 64 + lane;
  const bool in = j < a.T_cols;
  const int nsub = a.nrb * 4;
  const bool dense = uniform_i(gptr(a.spar)[1]) != 0;  // everything is scanned
  if (in)
    for (int k = q; k < a.nmask; k += kLimitWaves) gptr(a.smask)[j * a.nmask + k] = dense ? ~0ull : 0ull;
  if (dense)
    for (int s = threadIdx.x; s < nsub; s += 64 * kLimitWaves) gptr(a.gmask)[(int64_t)s * a.ngrp + blockIdx.x] = ~0ull;
  double top = -__builtin_huge_val(), sum = 0.0;
  int n = 0, m = 0;
  double z0 = 0.0, z1 = 0.0;
  int64_t off_m = 0;
  if (in) {
    while (m + 1 < a.M && gptr(a.col_off)[m + 1] <= j) ++m;
    off_m = gptr(a.col_off)[m];
    if (a.gdim) grid_point(a, j, off_m, &z0, &z1);
  }
  const double* const b2m = gptr(a.b2v) + (size_t)m * a.nrb * VPT * LNT;
  auto w_of = [&](int r, T v) -> double {
    const double c = a.gdim ? grid_cost(a, r, z0, z1) : (double)long_cost_col(a, j, off_m)[r];
    const int rr = r % RB;
    const double b2 = b2m[((size_t)(r / RB) * VPT + slot_of(rr, VEC)) * LNT + slot_owner(rr, VEC)];
    return long_w((double)v, b2, c, a.inv_rho);
  };
  constexpr int U = 8;
  const int s1 = nsub * (q + 1) / kLimitWaves;
  for (int s0 = dense ? s1 : nsub * q / kLimitWaves; s0 < s1; s0 += U) {
    int pc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) pc[u] = in && s0 + u < s1 ? gptr(a.pcnt)[(int64_t)(s0 + u) * a.T_cols + j] : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t h = j * nsub + s0 + u;
      for (int e = 0; e < pc[u]; ++e) {
        const double w = w_of(gptr(a.prow)[h * a.cap + e], gptr(a.pval)[h * a.cap + e]);
        top = fmax(top, w);
        sum += w;
        ++n;
      }
    }
  }
  s_top[q][lane] = top;
  s_sum[q][lane] = sum;
  s_n[q][lane] = n;
  __syncthreads();
  if (q == 0) {
    for (int k = 1; k < kLimitWaves; ++k) {
      top = fmax(top, s_top[k][lane]);
      sum += s_sum[k][lane];
      n += s_n[k][lane];
    }
    const double tau = in ? (double)gptr(a.q)[j] : 0.0;
    double lim = -__builtin_huge_val();
    if (n > 0) {
      lim = fmax(top - tau, (sum - tau) / (double)n);
    } else if (in) {
      const int r = gptr(a.wit)[j];
      if (r >= 0 && r < a.R) {
        const int par = *gptr(a.spar);
        const int si = r / RB * 4 + (slot_owner(r % RB, VEC) >> 6);
        const bool th = gptr(a.pcnt)[(int64_t)si * a.T_cols + j] < 0;
        lim = w_of(r, th ? gptr(a.theta)[j * a.ld + r] : gptr(a.nbv)[((size_t)par * a.M + m) * a.R + r]) - tau;
      }
    }
    // a column of weight 0 is 0 whatever its w
    lim = tau > 0.0 ? lim - (fabs(lim) + tau) * 0x1p-40 : __builtin_huge_val();
    if (in) {
      gptr(a.limit)[j] = lim;
      gptr(a.colm)[j] = m;
    }
    s_top[0][lane] = lim;
  }
  __syncthreads();
  if (dense) return;
  // The sub-tiles to scan: those with a patch or dense, and those whose bound
  // of w (by the multiply-add that forms w) exceeds the column's bound.
  const double lim = s_top[0][lane];
  const int64_t cc = !in ? 0
                     : a.cost_mode == MAM_COST_INDEXED ? (int64_t)a.cidx[j]
                     : a.cost_mode == MAM_COST_PER_COLUMN ? j : j - off_m;
  const double* const bm = gptr(a.bmax) + (int64_t)m * nsub;
  for (int s0 = nsub * q / kLimitWaves; s0 < s1; s0 += 64) {  // lane l keeps the word of sub-tile s0 + l
    unsigned long long word = 0ull;
    unsigned long long mine = 0ull;  // this column's sub-tiles
    const int ns = s1 - s0 < 64 ? s1 - s0 : 64;
    for (int u0 = 0; u0 < ns; u0 += U) {
      int pc[U];
      double bd[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = u0 + u < ns ? s0 + u0 + u : s0;
        pc[u] = in ? gptr(a.pcnt)[(int64_t)s * a.T_cols + j] : 0;
        bd[u] = __builtin_fma(-(double)gptr(a.cmin)[(int64_t)s * a.ncost + cc], a.inv_rho, bm[s]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool go = in && u0 + u < ns && (pc[u] != 0 || !(bd[u] <= lim));
        const unsigned long long b = __ballot(go);
        if (lane == u0 + u) word = b;
        if (go) mine |= 1ull << (u0 + u);
      }
    }
    if (in && mine != 0ull) {
      const int k = s0 >> 6, sh = s0 & 63;
      unsigned long long* const mk = gptr(a.smask) + j * a.nmask + k;
      atomicOr(mk, mine << sh);
      if (sh != 0 && (mine >> (64 - sh)) != 0ull) atomicOr(mk + 1, mine >> (64 - sh));
    }
    if (lane < ns) gptr(a.gmask)[(int64_t)(s0 + lane) * a.ngrp + blockIdx.x] = word;
    const int nc = (__popcll(word) + kScanCols - 1) / kScanCols;
    int off = nc;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const int v = __shfl_up(off, d);
      if (lane >= d) off += v;
    }
    const int tot = __builtin_amdgcn_readlane(off, 63);
    int first = 0;
    if (lane == 0 && tot > 0) first = atomicAdd(gptr(a.spar) + 2, tot);
    first = uniform_i(first) + off - nc;
    for (int c = 0; c < nc; ++c) {
      unsigned long long rest = word;
      for (int k = 0; k < kScanCols; ++k) rest &= rest - 1ull;  // 0 stays 0
      gptr(a.wsub)[first + c] = s0 + lane;
      gptr(a.wgrp)[first + c] = (int32_t)blockIdx.x;
      gptr(a.wcol)[first + c] = word & ~rest;
      word = rest;
    }
  }
}

// ---- sparse store: the per-row terms -------------------------------------
// 2 b and the common value + 2 b of every row, once per iteration for the scan
// and write kernels: formed in each of their workgroups they were most of the
// time of both (two dependent loads and a division per row, at 16 rows a
// thread; the scan of ten 40 x 40 images 0.36 ms).
template <typename T, int VPT, int VEC>
__global__ void __launch_bounds__(LNT)
long_base_kernel(LongArgs<T> a) {
  if (a.stop != nullptr && uniform_i(*gptr(a.stop)) != 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform_i(tid >> 6);
  const int rb = blockIdx.x, m = blockIdx.y, R = a.R, rbase = rb * LNT * VPT;
  const int par = uniform_i(*gptr(a.spar));
  if (rb == 0 && m == 0 && tid == 0) gptr(a.spar)[2] = 0;
  const double t = uniform_d(*gptr(a.t)), Sm = uniform_d(gptr(a.Sd)[m]);
  const double* const pmm = gptr(a.pm) + (size_t)m * R;
  const T* const nbm = gptr(a.nbv) + ((size_t)par * a.M + m) * R;
  const size_t o = ((size_t)m * a.nrb + rb) * VPT * LNT + tid;
  double mx = -__builtin_huge_val();
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int r = rbase + ((k / VEC) * LNT + tid) * VEC + (k % VEC), rl = r < R ? r : rbase;
    const double b2 = r < R ? 2.0 * long_b(t, gptr(a.p), pmm, rl, Sm) : -__builtin_huge_val();
    const double bs = (double)nbm[rl] + b2;
    gptr(a.b2v)[o + k * LNT] = b2;
    gptr(a.basev)[o + k * LNT] = bs;
    mx = fmax(mx, bs);
  }
  mx = wave_max(mx);
  if (lane == 0) gptr(a.bmax)[((int64_t)m * a.nrb + rb) * 4 + wv] = mx;
}

// ---- sparse store: write-back --------------------------------------------
// Write the stored plans back into theta: every sparse sub-tile is stored as
// its common values (whole vectors) and then its patches (each by the thread
// owning the row, after its own store), and marked dense.
template <typename T, int VPT, int VEC>
__global__ void __launch_bounds__(LNT)
long_materialize_kernel(LongArgs<T> a) {
  constexpr int NCH = VPT / VEC, RB = LNT * VPT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = uniform_i(tid >> 6);
  const int R = a.R, cap = a.cap, nsub = a.nrb * 4;
  const int par = uniform_i(*gptr(a.spar));
  T* const theta = gptr(a.theta);
  if (blockIdx.x == 0 && tid == 0) gptr(a.spar)[1] = 1;  // (read by no other workgroup of this kernel)
  const int ib = uniform_i(a.wg_it[blockIdx.x]), ie = uniform_i(a.wg_it[blockIdx.x + 1]);
  for (int it = ib; it < ie; ++it) {
    const int rb = uniform_i(a.it_rb[it]), m = uniform_i(a.it_m[it]);
    const int64_t j0 = uniform_l(a.it_j0[it]), j1 = uniform_l(a.it_j1[it]);
    const int rbase = rb * RB;
    const T* __restrict__ nbm = gptr(a.nbv) + ((size_t)par * a.M + m) * R;
    T nb[VPT];
#pragma unroll
    for (int k = 0; k < VPT; ++k) {
      const int r = rbase + ((k / VEC) * LNT + tid) * VEC + (k % VEC);
      nb[k] = r < R ? nbm[r] : T(0);
    }
    for (int64_t j = j0; j < j1; ++j) {
      const int64_t h = j * nsub + rb * 4 + wv;
      int32_t* const pcj = gptr(a.pcnt) + (int64_t)(rb * 4 + wv) * a.T_cols + j;
      const int pc = uniform_i(*pcj);
      if (pc < 0) continue;
      T* __restrict__ thp = theta + j * a.ld;
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const int r0 = rbase + (c * LNT + tid) * VEC;
        T out[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) out[v] = nb[c * VEC + v];
        if (r0 + VEC <= R) {
          store_vec_nt<T, VEC>(thp + r0, out);
        } else {
#pragma unroll
          for (int v = 0; v < VEC; ++v)
            if (r0 + v < R) thp[r0 + v] = out[v];
        }
      }
      if (pc > 0) {
        const int pr = lane < pc ? gptr(a.prow)[h * cap + lane] : 0;
        const T pvv = lane < pc ? gptr(a.pval)[h * cap + lane] : T(0);
        for (int e = 0; e < pc; ++e) {
          const int r = __builtin_amdgcn_readlane(pr, e);
          const T val = read_lane(pvv, e);
          if (slot_owner(r - rbase, VEC) == tid) thp[r] = val;
        }
      }
      if (lane == 0) *pcj = -1;
    }
  }
}

}  // namespace mam
