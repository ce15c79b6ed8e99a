// Column-kernel instance lookup.  The instances are compiled in separate
// translation units (one per element type and diagnostics mode) so the
// build runs in parallel.
#pragma once

#include "mam_kernels.hpp"

namespace mam {

template <typename T>
using ColFn = void (*)(ColArgs<T>);

// Returns the instance for (threads per column, values per thread, vector
// width, columns in flight, diagnostics) or nullptr if none exists.
// Instances: 64 threads with 1-16 values per thread, 128-1024 threads with
// 4-16; columns in flight 1, 2, 4 for vector loads without diagnostics,
// otherwise 1.
template <typename T, int KC>
ColFn<T> pick_column_kc(int nt, int vpt, int vec, int stream);
template <typename T>
ColFn<T> pick_column_diag(int nt, int vpt, int vec);

// First iteration of a sparse call, 64 or more threads per column.
template <typename T>
ColFn<T> pick_column_sparse(int nt, int vpt, int vec);
extern template ColFn<float> pick_column_sparse<float>(int, int, int);
extern template ColFn<double> pick_column_sparse<double>(int, int, int);

// Kernels of the sparse iterations (mam_sparse.hpp).
template <typename T> struct SpArgs;
struct SpTile;
struct SpRows;
struct SpCost;
template <typename T>
struct SparseFns {
  void (*column)(SpArgs<T>) = nullptr;
  void (*column_rec)(SpArgs<T>) = nullptr;  // records the active sets
  void (*close)(const SpProb<T>*, const SpRows*, int, const uint8_t*, int, const int32_t*) = nullptr;
  void (*next)(const SpProb<T>*, const SpRows*, const uint8_t*, int, const int32_t*) = nullptr;
  void (*write)(const SpProb<T>*, const SpTile*, const int32_t*, unsigned long long*, unsigned) = nullptr;
  void (*d2)(const SpProb<T>*, const int32_t*) = nullptr;
  void (*cost_min)(const SpProb<T>*, const SpCost*, const int32_t*) = nullptr;
};
template <typename T>
SparseFns<T> pick_sparse();
extern template SparseFns<float> pick_sparse<float>();
extern template SparseFns<double> pick_sparse<double>();

// Sub-wave instance (16 or 32 lanes per column, one column in flight, no
// diagnostics) or nullptr.  sparse: the first iteration of a sparse call.
template <typename T>
ColFn<T> pick_subwave(int nt, int vpt, int vec, int stream, bool sparse);
extern template ColFn<float> pick_subwave<float>(int, int, int, int, bool);
extern template ColFn<double> pick_subwave<double>(int, int, int, int, bool);

// The kernel of the first iteration of a sparse call: theta read, patches
// stored (one column in flight, so a schedule's block of any size fits).
template <typename T>
inline ColFn<T> pick_first(int nt, int vpt, int vec) {
  return nt < 64 ? pick_subwave<T>(nt, vpt, vec, 0, true) : pick_column_sparse<T>(nt, vpt, vec);
}

template <typename T>
inline ColFn<T> pick_column(int nt, int vpt, int vec, int kc, int diag, int stream) {
  if (nt < 64) return (diag || kc != 1) ? nullptr : pick_subwave<T>(nt, vpt, vec, stream, false);
  if (diag) return pick_column_diag<T>(nt, vpt, vec);
  switch (kc) {
    case 1: return pick_column_kc<T, 1>(nt, vpt, vec, stream);
    case 2: return pick_column_kc<T, 2>(nt, vpt, vec, stream);
    case 4: return pick_column_kc<T, 4>(nt, vpt, vec, stream);
    default: return nullptr;
  }
}

// Long-column tile kernels for (values per thread, vector width, grid
// cost); null members if no instance exists.
template <typename T> struct LongArgs;
template <typename T>
struct LongFns {
  void (*scan)(LongArgs<T>) = nullptr;
  void (*thresh)(LongArgs<T>) = nullptr;
  void (*write)(LongArgs<T>) = nullptr;
  void (*rowsum)(LongArgs<T>, int) = nullptr;
  void (*rowsum_q)(LongArgs<T>, int) = nullptr;  // of the library's own start, from q
  void (*materialize)(LongArgs<T>) = nullptr;  // sparse store write-back
  void (*scan_sparse)(LongArgs<T>) = nullptr;  // sparse-store scan
  void (*thresh_diag)(LongArgs<T>) = nullptr;  // with the iteration's diagnostics
  void (*thresh_sparse)(LongArgs<T>) = nullptr;
  void (*thresh_sparse_diag)(LongArgs<T>) = nullptr;
  void (*write_diag)(LongArgs<T>) = nullptr;
  void (*cost_min)(LongArgs<T>) = nullptr;     // sparse store: least cost of every sub-tile
  void (*base)(LongArgs<T>) = nullptr;         // sparse store: 2b and common value + 2b of every row
  void (*limit)(LongArgs<T>) = nullptr;        // sparse store: lower bounds of the thresholds
};
template <typename T>
LongFns<T> pick_long(int vpt, int vec, bool grid);
extern template LongFns<float> pick_long<float>(int, int, bool);
extern template LongFns<double> pick_long<double>(int, int, bool);

// Reverse-mode column kernel for (mask bytes per lane, columns per wave at
// a time); nullptr if none exists.
struct AdjArgs;
using AdjFn = void (*)(AdjArgs);
AdjFn pick_adjoint(int lane_bytes, int kc);

extern template ColFn<float> pick_column_kc<float, 1>(int, int, int, int);
extern template ColFn<float> pick_column_kc<float, 2>(int, int, int, int);
extern template ColFn<float> pick_column_kc<float, 4>(int, int, int, int);
extern template ColFn<double> pick_column_kc<double, 1>(int, int, int, int);
extern template ColFn<double> pick_column_kc<double, 2>(int, int, int, int);
extern template ColFn<double> pick_column_kc<double, 4>(int, int, int, int);
extern template ColFn<float> pick_column_diag<float>(int, int, int);
extern template ColFn<double> pick_column_diag<double>(int, int, int);

}  // namespace mam
