// Launch of the 3-D column kernels (FP32, FP64 and bf16 storage).
#include "kron.h"
#include "kron_cols.hpp"
#include "kron_launch.hpp"

namespace kron {
namespace {

template <class M, int N, bool kTrans>
void launch_cols3d(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
                   const typename M::io_t* X, typename M::io_t* Y, int64_t batch, hipStream_t stream) {
  using S = Col3D<M, N, kTrans>;
  auto k = kron3d_cols_kernel<S>;
  const int64_t tiles = (batch + S::P - 1) / S::P;
  constexpr int per_cu = col3d_shape<N, typename M::io_t>().per_cu;
  const bool few = per_cu > 0 && batch * S::E * (int64_t)sizeof(typename M::io_t) >= kColLong;
  const int64_t cap = (int64_t)device_cus() * (few ? per_cu : occupancy_blocks(k, S::kThreads));
  hipLaunchKernelGGL(k, dim3((unsigned)(tiles < cap ? tiles : cap)), dim3(S::kThreads), 0, stream, A, B, C, X, Y,
                     batch, tiles);
}

template <class M>
int cols3d_n(int n, const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
             const typename M::io_t* X, typename M::io_t* Y, int64_t batch, hipStream_t s, bool trans) {
  int rc = -1;
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if (n != N) return;
    if constexpr (!kHasCols<M, N>) {
      return;
    } else if constexpr (std::is_same_v<M, ModeBF16>) {
      rc = 0;
      launch_cols3d<M, N, false>(A, B, C, X, Y, batch, s);  // no transposed entry point
    } else {
      rc = 0;
      if (trans) launch_cols3d<M, N, true>(A, B, C, X, Y, batch, s);
      else launch_cols3d<M, N, false>(A, B, C, X, Y, batch, s);
    }
  });
  return rc;
}

}  // namespace

bool has_cols3d(int mode, int n) {
  bool has = false;
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if (n == N) has = mode == KRON_MODE_F32   ? kHasCols<ModeF32, N>
                      : mode == KRON_MODE_F64 ? kHasCols<ModeF64, N>
                                              : mode == KRON_MODE_BF16 && kHasCols<ModeBF16, N>;
  });
  return has;
}

int cols3d(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
           hipStream_t s, bool trans) {
  return cols3d_n<ModeF32>(n, A, B, C, X, Y, batch, s, trans);
}
int cols3d(int n, const double* A, const double* B, const double* C, const double* X, double* Y, int64_t batch,
           hipStream_t s, bool trans) {
  return cols3d_n<ModeF64>(n, A, B, C, X, Y, batch, s, trans);
}
int cols3d(int n, const uint16_t* A, const uint16_t* B, const uint16_t* C, const uint16_t* X, uint16_t* Y,
           int64_t batch, hipStream_t s, bool trans) {
  return cols3d_n<ModeBF16>(n, A, B, C, X, Y, batch, s, trans);
}

}  // namespace kron
