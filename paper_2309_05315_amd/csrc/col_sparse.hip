// Kernels of the sparse iterations (mam_sparse.hpp) for both element types.
#include "mam_dispatch.hpp"
#include "mam_sparse.hpp"

namespace mam {

template <typename T>
SparseFns<T> pick_sparse() {
  SparseFns<T> f;
  f.column = &sparse_column_kernel<T, false>;
  f.column_rec = &sparse_column_kernel<T, true>;
  f.close = &sparse_close_kernel<T>;
  f.next = &sparse_next_kernel<T>;
  f.write = &sparse_write_kernel<T>;
  f.d2 = &sparse_d2_kernel<T>;
  f.cost_min = &cost_min_kernel<T>;
  return f;
}
template SparseFns<float> pick_sparse<float>();
template SparseFns<double> pick_sparse<double>();

}  // namespace mam
