// Host-side launch of the forward kernels: n dispatch, alignment choice and
// grid size.  Included by one translation unit per precision mode.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <mutex>
#include <type_traits>
#include <unordered_map>

#include "kron_kernels.hpp"
#include "kron_staged.hpp"
#include "kron_runtime.hpp"

namespace kron {

// Resident workgroups per CU for a kernel, queried once per kernel (keyed by
// its address: kernels of one signature must not share the value).
inline int occupancy_blocks_of(const void* kernel, int threads = kBlock) {
  static std::mutex mu;
  static std::unordered_map<const void*, int> cache;
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(kernel);
  if (it != cache.end()) return it->second;
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1) nb = 1;
  cache.emplace(kernel, nb);
  return nb;
}

template <typename K>
int occupancy_blocks(K kernel, int threads = kBlock) {
  return occupancy_blocks_of(reinterpret_cast<const void*>(kernel), threads);
}

// Workgroups to launch: enough to cover the work, at most `per_cu` (or the
// occupancy limit when per_cu <= 0) on every CU.
inline unsigned grid_blocks(int64_t waves_needed, int occ, int per_cu) {
  const int64_t need = (waves_needed + kBlock / kWave - 1) / (kBlock / kWave);
  const int64_t cap = (int64_t)device_cus() * (per_cu > 0 ? per_cu : occ);
  int64_t g = need < cap ? need : cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

inline bool aligned_to(const void* p, int bytes) { return (reinterpret_cast<uintptr_t>(p) % bytes) == 0; }

template <class M, int N, bool kTrans, bool kVec, int kTiles>
void launch2d_k(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* X,
                typename M::io_t* Y, int64_t batch, int64_t ntiles, int per_cu, hipStream_t stream) {
  auto k = kron2d_kernel<M, N, kVec, kTrans, kTiles>;
  const int64_t waves = (ntiles + kTiles - 1) / kTiles;
  hipLaunchKernelGGL(k, dim3(grid_blocks(waves, occupancy_blocks(k), per_cu)), dim3(kBlock), 0, stream, A, B, X, Y,
                     batch, ntiles);
}

template <class M, int N, bool kTrans, bool kVec>
void launch2d_v(int variant, const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* X,
                typename M::io_t* Y, int64_t batch, int64_t ntiles, int per_cu, hipStream_t stream) {
  switch (variant) {
    case 1:
      launch2d_k<M, N, kTrans, kVec, 8>(A, B, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 2:
      launch2d_k<M, N, kTrans, kVec, 2>(A, B, X, Y, batch, ntiles, per_cu, stream);
      break;
    default:
      launch2d_k<M, N, kTrans, kVec, 4>(A, B, X, Y, batch, ntiles, per_cu, stream);
  }
}

// Element strides of one array: s1 between columns (2-D) or along the middle
// index (3-D), s2 along the slowest index (3-D), sp between operands.
struct Strides {
  int64_t s1, s2, sp;
};

// Rows that 16-byte vectors can take.
inline bool vec_strides(const Strides& s, const void* base) {
  return s.s1 % 4 == 0 && s.s2 % 4 == 0 && s.sp % 4 == 0 && reinterpret_cast<uintptr_t>(base) % 16 == 0;
}

// The strided action on columns in LDS (kron_strided_cols.hip) of prepared
// factors; false, with nothing launched, where the general kernel is used:
// operands so far apart that offsets in a tile need more than 32 bits, and
// n = 16 with rows for 16-byte vectors (but for FP64 3-D without beta), whose
// tiles waste nothing and contract in the order of the packed call's kernel, so
// that the results equal it to the last bit (3-D FP32 padded by 4, 671 MB of X:
// 413 us, columns 449; padded by 1, 128 MiB: 93, columns 56), or FP32
// beyond 320 MiB (3-D padded by 1, 512 MiB: 337, columns 365; 256: 179, 150).
bool strided_cols(int dim, int n, const float* A, const float* B, const float* C, const float* X, const Strides& xs,
                  float* Y, const Strides& ys, int64_t batch, float beta, bool transx, hipStream_t stream);
bool strided_cols(int dim, int n, const double* A, const double* B, const double* C, const double* X,
                  const Strides& xs, double* Y, const Strides& ys, int64_t batch, double beta, bool transx,
                  hipStream_t stream);

// Modes and sizes that have a column kernel (kron_cols.hip), by measurement
// over 1 GiB of operands (old: the best of the other variants):
//   FP32, n < 16 (at n = 16 one operand fills a 16-slot tile, in registers):
//     3.1 .. 4.9 -> 4.6 .. 6.0 TB/s (n = 10: 3.87 -> 5.31; n = 7: 3.87 -> 5.24);
//   FP64, every n: 2.6 .. 4.6 -> 4.5 .. 6.1 TB/s (n = 12: 3.01 -> 5.42; n = 16:
//     4.60 -> 5.53);
//   bf16 storage, the sizes whose tiles waste most slots: 2.2 .. 3.4 -> 3.4 ..
//     4.0 TB/s; at the others the staged tiles' K = 32 products need fewer
//     matrix cycles than FP32 ones (n = 12: 4.3 against 3.7 TB/s).
template <class M, int N>
constexpr bool kHasCols = std::is_same_v<M, ModeF64> || (std::is_same_v<M, ModeF32> && N < 16) ||
                          (std::is_same_v<M, ModeBF16> && (N == 3 || (N >= 5 && N <= 11 && N != 8)));

// Sizes that read their tiles through LDS: every n but 16 (an FP64 3-D
// slice is up to 32 KiB per wavefront, 128 KiB per workgroup).
template <class M, int N, int Dim>
constexpr bool kStageable = N != 16;

// 2-D variants: tiles kept in flight per wavefront, 0 -> 4, 1 -> 8, 2 -> 2;
// 3 -> tiles staged through LDS (n != 16), 4 -> the same with two LDS slices
// per wavefront and each span's copy-out issued after the next span's
// operands are committed (n = 16 runs variant 0).
template <class M, int N, bool kTrans>
int launch2d_n(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* X,
               typename M::io_t* Y, int64_t batch, hipStream_t stream, int mode) {
  using io_t = typename M::io_t;
  constexpr int64_t ops = (int64_t)Geo<N>::Q * Geo<N>::Q;
  const int64_t ntiles = (batch + ops - 1) / ops;
  const LaunchShape sh = launch_shape(mode, 2, N);
  if constexpr (kStageable<M, N, 2>) {
    if (sh.variant == 3 || sh.variant == 4) {
      auto k = sh.variant == 4 ? kron2d_staged_kernel<M, N, kTrans, true> : kron2d_staged_kernel<M, N, kTrans, false>;
      constexpr int kT = Staged2D<M, N, kTrans>::kT;
      const int64_t waves = (ntiles + kT - 1) / kT;
      hipLaunchKernelGGL(k, dim3(grid_blocks(waves, occupancy_blocks(k), sh.blocks_per_cu)), dim3(kBlock), 0,
                         stream, A, B, X, Y, batch, ntiles);
      return 0;
    }
  }
  if constexpr (Geo<N>::kVec) {
    if (aligned_to(X, Mem<io_t>::kAlign) && aligned_to(Y, Mem<io_t>::kAlign)) {
      launch2d_v<M, N, kTrans, true>(sh.variant, A, B, X, Y, batch, ntiles, sh.blocks_per_cu, stream);
      return 0;
    }
  }
  launch2d_v<M, N, kTrans, false>(sh.variant, A, B, X, Y, batch, ntiles, sh.blocks_per_cu, stream);
  return 0;
}

template <class M, int N, bool kTrans, bool kVec, bool kPipe, bool kContig, int kWindow>
void launch3d_k(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
                const typename M::io_t* X, typename M::io_t* Y, int64_t batch, int64_t ntiles, int per_cu,
                hipStream_t stream) {
  auto k = kron3d_kernel<M, N, kVec, kTrans, kPipe, kContig, kWindow>;
  hipLaunchKernelGGL(k, dim3(grid_blocks(ntiles, occupancy_blocks(k), per_cu)), dim3(kBlock), 0, stream, A, B, C, X,
                     Y, batch, ntiles);
}

template <class M, int N, bool kTrans, bool kVec>
void launch3d_v(int variant, const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
                const typename M::io_t* X, typename M::io_t* Y, int64_t batch, int64_t ntiles, int per_cu,
                hipStream_t stream) {
  switch (variant) {
    case 1:
      launch3d_k<M, N, kTrans, kVec, true, false, 0>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 2:
      launch3d_k<M, N, kTrans, kVec, false, true, 0>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 3:
      launch3d_k<M, N, kTrans, kVec, true, true, 0>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 4:
      launch3d_k<M, N, kTrans, kVec, false, true, 2>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 5:
      launch3d_k<M, N, kTrans, kVec, false, true, 4>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 6:
      launch3d_k<M, N, kTrans, kVec, true, true, 2>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 7:
      launch3d_k<M, N, kTrans, kVec, true, true, 4>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      break;
    case 9:
    case 10:
      if constexpr (N == 16 && kVec) {
        auto k = variant == 9 ? kron3d_stream_kernel<M, kTrans, 2> : kron3d_stream_kernel<M, kTrans, 4>;
        hipLaunchKernelGGL(k, dim3(grid_blocks(ntiles, occupancy_blocks(k), per_cu)), dim3(kBlock), 0, stream, A, B,
                           C, X, Y, ntiles);
      } else {
        // same stage order (contiguous rows), slab window 2
        launch3d_k<M, N, kTrans, kVec, false, true, 2>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
      }
      break;
    default:
      launch3d_k<M, N, kTrans, kVec, false, false, 0>(A, B, C, X, Y, batch, ntiles, per_cu, stream);
  }
}

// 3-D variants: 0 plain, 1 next tile prefetched, 2 contiguous 1 KiB rows
// (operand slabs along the slow axis, a second lane-group exchange),
// 3 = 1 + 2, 4/5 contiguous rows with a window of 2/4 slab loads in flight,
// 6/7 = 4/5 with the next tile's first slabs requested before stage 3,
// 8 = tiles staged through LDS (n != 16; n = 16 falls back to variant 0), 9/10 = n = 16 with the result stores
// interleaved with the next tile's loads and stages 1-2, window 2/4 (other
// sizes and unaligned arrays run variant 4, the same stage order), 11 = 8
// with two LDS slices per wavefront where they fit and each tile's copy-out
// issued after the next tile's operands are committed (n = 16: variant 0).
// Workgroups per CU -1: the column kernels.
template <class M, int N, bool kTrans>
int launch3d_n(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
               const typename M::io_t* X, typename M::io_t* Y, int64_t batch, hipStream_t stream, int mode) {
  using io_t = typename M::io_t;
  constexpr int64_t ops = (int64_t)Geo<N>::Q * Geo<N>::Q * Geo<N>::Q;
  const int64_t ntiles = (batch + ops - 1) / ops;
  const LaunchShape sh = launch_shape(mode, 3, N);
  if constexpr (kHasCols<M, N>) {
    if (sh.blocks_per_cu < 0) return cols3d(N, A, B, C, X, Y, batch, stream, kTrans);
  }
  if constexpr (kStageable<M, N, 3>) {
    if (sh.variant == 8 || sh.variant == 11) {
      auto k = sh.variant == 11 ? kron3d_staged_kernel<M, N, kTrans, true> : kron3d_staged_kernel<M, N, kTrans, false>;
      hipLaunchKernelGGL(k, dim3(grid_blocks(ntiles, occupancy_blocks(k), sh.blocks_per_cu)), dim3(kBlock), 0,
                         stream, A, B, C, X, Y, batch, ntiles);
      return 0;
    }
  }
  if constexpr (Geo<N>::kVec) {
    if (aligned_to(X, Mem<io_t>::kAlign) && aligned_to(Y, Mem<io_t>::kAlign)) {
      launch3d_v<M, N, kTrans, true>(sh.variant, A, B, C, X, Y, batch, ntiles, sh.blocks_per_cu, stream);
      return 0;
    }
  }
  launch3d_v<M, N, kTrans, false>(sh.variant, A, B, C, X, Y, batch, ntiles, sh.blocks_per_cu, stream);
  return 0;
}

// kron_ex_kernel (beta != 0, or 2-D operands read transposed): the vector
// path when X and Y are aligned, a persistent grid sized by occupancy.
template <class M, int Dim, int N, bool kBeta, bool kTX>
void launch_ex_k(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
                 const typename M::io_t* X, typename M::io_t* Y, int64_t batch, typename M::io_t beta,
                 hipStream_t stream) {
  using io_t = typename M::io_t;
  constexpr int64_t Q = Geo<N>::Q;
  constexpr int64_t ops = Dim == 2 ? Q * Q : Q * Q * Q;
  const int64_t ntiles = (batch + ops - 1) / ops;
  const int64_t waves = Dim == 2 ? (ntiles + 3) / 4 : ntiles;  // 2-D: four tiles per wavefront step
  auto run = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(grid_blocks(waves, occupancy_blocks(k), 0)), dim3(kBlock), 0, stream, A, B, C, X, Y,
                       batch, ntiles, beta);
  };
  if constexpr (Geo<N>::kVec) {
    if (aligned_to(X, Mem<io_t>::kAlign) && aligned_to(Y, Mem<io_t>::kAlign)) {
      run(kron_ex_kernel<M, N, true, Dim, kBeta, kTX>);
      return;
    }
  }
  run(kron_ex_kernel<M, N, false, Dim, kBeta, kTX>);
}

template <class M, int Dim, int N>
int launch_ex_n(const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
                const typename M::io_t* X, typename M::io_t* Y, int64_t batch, typename M::io_t beta, bool transx,
                hipStream_t stream) {
  const bool has_beta = beta != typename M::io_t(0);
  if constexpr (Dim == 2) {
    if (transx) {
      if (has_beta) launch_ex_k<M, 2, N, true, true>(A, B, C, X, Y, batch, beta, stream);
      else launch_ex_k<M, 2, N, false, true>(A, B, C, X, Y, batch, beta, stream);
      return 0;
    }
  }
  if (!has_beta || transx) return -2;  // nothing this kernel adds: the caller runs the plain kernels
  launch_ex_k<M, Dim, N, true, false>(A, B, C, X, Y, batch, beta, stream);
  return 0;
}

#define KRON_N_CASES(F) \
  F(1) F(2) F(3) F(4) F(5) F(6) F(7) F(8) F(9) F(10) F(11) F(12) F(13) F(14) F(15) F(16)

template <class M, bool kTrans>
int launch2d(int n, const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* X,
             typename M::io_t* Y, int64_t batch, hipStream_t stream, int mode) {
  switch (n) {
#define KRON_CASE(NN) \
  case NN:            \
    return launch2d_n<M, NN, kTrans>(A, B, X, Y, batch, stream, mode);
    KRON_N_CASES(KRON_CASE)
#undef KRON_CASE
    default:
      return -1;
  }
}

template <class M, int Dim>
int launch_ex(int n, const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
              const typename M::io_t* X, typename M::io_t* Y, int64_t batch, typename M::io_t beta, bool transx,
              hipStream_t stream) {
  switch (n) {
#define KRON_CASE(NN) \
  case NN:            \
    return launch_ex_n<M, Dim, NN>(A, B, C, X, Y, batch, beta, transx, stream);
    KRON_N_CASES(KRON_CASE)
#undef KRON_CASE
    default:
      return -1;
  }
}

// n in [NLO, NHI] (one translation unit per range keeps builds parallel)
template <class M, bool kTrans, int NN, int NHI>
int launch3d_range(int n, const typename M::io_t* A, const typename M::io_t* B, const typename M::io_t* C,
                   const typename M::io_t* X, typename M::io_t* Y, int64_t batch, hipStream_t stream, int mode) {
  if constexpr (NN > NHI) {
    return -1;
  } else {
    if (n == NN) return launch3d_n<M, NN, kTrans>(A, B, C, X, Y, batch, stream, mode);
    return launch3d_range<M, kTrans, NN + 1, NHI>(n, A, B, C, X, Y, batch, stream, mode);
  }
}

}  // namespace kron
