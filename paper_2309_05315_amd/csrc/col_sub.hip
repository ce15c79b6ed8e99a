// Instances of the sub-wave column kernel: 16 or 32 lanes per column, 1-16
// values per lane, vector loads of 16 bytes when a lane holds at least one
// vector, plain or streaming (non-temporal) plans; and the first iteration of
// a sparse call (theta is read once: streaming).
#include "mam_dispatch.hpp"
#include "mam_sparse.hpp"
#include "mam_subwave.hpp"

namespace mam {

template <typename T, int NT, int VPT>
ColFn<T> pick_sub_vec(int vec, int stream, bool sparse) {
  constexpr int VN = VecOf<T>::N;
  if (sparse) {
    if constexpr (VPT >= VN) {
      if (vec == VN) return &subwave_kernel<T, NT, VPT, VN, true, true>;
    }
    return vec == 1 ? &subwave_kernel<T, NT, VPT, 1, false, true> : nullptr;
  }
  if constexpr (VPT >= VN) {
    if (vec == VN) return stream ? &subwave_kernel<T, NT, VPT, VN, true> : &subwave_kernel<T, NT, VPT, VN, false>;
  }
  if (vec == 1) return stream ? &subwave_kernel<T, NT, VPT, 1, true> : &subwave_kernel<T, NT, VPT, 1, false>;
  return nullptr;
}

template <typename T, int NT>
ColFn<T> pick_sub_vpt(int vpt, int vec, int stream, bool sparse) {
  switch (vpt) {
    case 1: return pick_sub_vec<T, NT, 1>(vec, stream, sparse);
    case 2: return pick_sub_vec<T, NT, 2>(vec, stream, sparse);
    case 4: return pick_sub_vec<T, NT, 4>(vec, stream, sparse);
    case 8: return pick_sub_vec<T, NT, 8>(vec, stream, sparse);
    case 16: return pick_sub_vec<T, NT, 16>(vec, stream, sparse);
    default: return nullptr;
  }
}

template <typename T>
ColFn<T> pick_subwave(int nt, int vpt, int vec, int stream, bool sparse) {
  if (nt == 16) return pick_sub_vpt<T, 16>(vpt, vec, stream, sparse);
  if (nt == 32) return pick_sub_vpt<T, 32>(vpt, vec, stream, sparse);
  return nullptr;
}

template ColFn<float> pick_subwave<float>(int, int, int, int, bool);
template ColFn<double> pick_subwave<double>(int, int, int, int, bool);

}  // namespace mam
