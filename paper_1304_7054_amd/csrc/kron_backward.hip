// Launch of the backward kernels (FP32 and FP64).
#include "kron.h"
#include "kron_backward.hpp"
#include "kron_launch.hpp"

namespace kron {

// Partial sums a call may leave in its workspace: a fixed function of the
// batch and the device.
int64_t grad_waves(int dim, int n, int64_t batch) {
  const int64_t q = 16 / n;
  const int64_t ops = dim == 3 ? q * q * q : q * q;
  const int64_t ntiles = (batch + ops - 1) / ops;
  const int64_t cap = (int64_t)device_cus() * 8;
  int64_t w = ntiles < cap ? ntiles : cap;
  w = (w + 3) / 4 * 4;
  return w < 4 ? 4 : w;
}

size_t grad_workspace_bytes(int dim, int n, int64_t batch, int elem_bytes) {
  return (size_t)grad_waves(dim, n, batch) * 3 * 256 * (size_t)elem_bytes;
}

namespace {

// The workgroup count is a fixed function of the batch and the device, so the
// summation order (and the result) is the same on every call.
template <typename T, int Dim, int N>
void launch_backward(const T* A, const T* B, const T* C, const T* X, const T* dY, T* dX, T* dA, T* dB, T* dC,
                     int64_t batch, void* ws, hipStream_t stream) {
  using S = Bwd<T, Dim, N>;
  const int which = (dA ? 1 : 0) | (dB ? 2 : 0) | (dC ? 4 : 0);
  T* part = static_cast<T*>(ws);
  int64_t nblocks = 0;
  if (batch > 0) {
    auto k = kron_backward_kernel<S>;
    const int64_t tiles = (batch + S::P - 1) / S::P;
    const int64_t cap = std::min((int64_t)device_cus() * occupancy_blocks(k, S::kThreads), grad_waves(Dim, N, batch));
    nblocks = std::min(tiles, cap);
    hipLaunchKernelGGL(k, dim3((unsigned)nblocks), dim3(S::kThreads), 0, stream, A, B, C, X, dY, dX, part, batch, tiles,
                       which);
  }
  hipLaunchKernelGGL((kron_backward_sum_kernel<T, N>), dim3(Dim * N * N), dim3(256), 0, stream, part, nblocks, dA, dB,
                     dC);
}

template <typename T, int Dim>
int backward_n(int n, const T* A, const T* B, const T* C, const T* X, const T* dY, T* dX, T* dA, T* dB, T* dC,
               int64_t batch, void* ws, hipStream_t s) {
  int rc = -1;
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if (n != N) return;
    launch_backward<T, Dim, N>(A, B, C, X, dY, dX, dA, dB, dC, batch, ws, s);
    rc = 0;
  });
  return rc;
}

}  // namespace

int backward(int dim, int n, const float* A, const float* B, const float* C, const float* X, const float* dY,
             float* dX, float* dA, float* dB, float* dC, int64_t batch, void* ws, hipStream_t s) {
  return dim == 2 ? backward_n<float, 2>(n, A, B, C, X, dY, dX, dA, dB, nullptr, batch, ws, s)
                  : backward_n<float, 3>(n, A, B, C, X, dY, dX, dA, dB, dC, batch, ws, s);
}
int backward(int dim, int n, const double* A, const double* B, const double* C, const double* X, const double* dY,
             double* dX, double* dA, double* dB, double* dC, int64_t batch, void* ws, hipStream_t s) {
  return dim == 2 ? backward_n<double, 2>(n, A, B, C, X, dY, dX, dA, dB, nullptr, batch, ws, s)
                  : backward_n<double, 3>(n, A, B, C, X, dY, dX, dA, dB, dC, batch, ws, s);
}

}  // namespace kron
