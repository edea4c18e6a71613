// Strided storage: the mode products of the column kernels with the strides only
// where the operands enter and leave (n < 16; n = 16 where the general kernel's
// 16-byte rows do not apply or, FP64 3-D, are the slower ones).
//
// A workgroup holds P operands packed in LDS (the image of the backward
// kernels) and works on one column per lane, so that no lane, product or
// access is spent on padding a tile axis to 16 slots, and a NaN stays in its
// operand.  3-D: the slow-axis columns are read from memory into the registers
// of the first product, consecutive lanes along the fast and middle axes; 2-D:
// op(X) is read in memory order, because a slow-axis column's neighbours end
// after n elements.  The results leave LDS in memory order.  A tile's offsets
// are 32 bits wide; operands further apart take the general kernel.  What bounds
// it is memory, the result's lines being written in part: their gaps stay as
// they were.  128 MiB of X, general kernel before and this one now: FP32 2-D
// n = 10 padded by 4 141 -> 56 us, 3-D n = 5 padded by 2 157 -> 53, FP64 3-D
// n = 3 312 -> 52; 1 MiB 21 -> 16 us, FP64 3-D n = 1 58 -> 18.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kron.h"
#include "kron_backward.hpp"
#include "kron_launch.hpp"

namespace kron {
namespace {

constexpr unsigned kNear = 1u << 29;  // elements; offsets stay below it, and their bytes in FP64 below 2^32

// The result's bytes, gaps included, up to which its lines wait in the last
// cache for their neighbours; beyond, stores that bypass it are faster (n = 10
// padded by 4, FP32 3-D: 128 MiB 56 us, bypassing 70; 256 MiB 162 and 135).
constexpr int64_t kCached = (int64_t)160 << 20;

// Wavefronts per SIMD that the registers are held to, without spills.
template <class S>
constexpr int per_simd() {
  if (sizeof(typename S::io_t) == 8) return S::N <= 8 ? 3 : 2;
  return S::N <= 8 ? 4 : S::N <= 11 ? 3 : 2;
}

template <class S, bool kBeta, bool kTX>
__global__ __launch_bounds__(S::kThreads) __attribute__((amdgpu_waves_per_eu(per_simd<S>()))) void
kron_strided_cols_kernel(const typename S::io_t* __restrict__ A, const typename S::io_t* __restrict__ B,
                         const typename S::io_t* __restrict__ C, const typename S::io_t* __restrict__ X, Strides xs,
                         typename S::io_t* __restrict__ Y, Strides ys, int64_t batch, int64_t ntiles,
                         typename S::io_t beta, bool longer) {
  using T = typename S::io_t;
  using Tiles = BwdTiles<S>;
  constexpr int N = S::N, P = S::P, NC = S::NC, kE = S::kE, Dim = S::Dim, E = S::E, kT = S::kThreads;
  __shared__ __attribute__((aligned(16))) T lds[S::kImage];
  const Tiles tl;
  const int lane = threadIdx.x & 63;
  const typename S::template Factor<false> fA(A, lane), fB(B, lane);
  const unsigned x1 = (unsigned)xs.s1, x2 = (unsigned)xs.s2, xp = (unsigned)xs.sp;
  const unsigned y1 = (unsigned)ys.s1, y2 = (unsigned)ys.s2, yp = (unsigned)ys.sp;
  // element e of a tile, in memory order, in a strided array
  auto place = [](int e, unsigned s1, unsigned s2, unsigned sp) {
    const unsigned row = e / N % N, in = e % N;
    if constexpr (Dim == 3) return (unsigned)(e / E) * sp + (unsigned)(e / (N * N) % N) * s2 + row * s1 + in;
    return (unsigned)(e / E) * sp + row * s1 + in;
  };
  auto count_of = [&](int64_t t) {
    const int64_t rem = batch - t * P;
    return (int)(rem < P ? rem : P) * E;
  };
  auto copy_out = [&](int64_t t) {
    T* const Yt = Y + t * P * ys.sp;
    const int count = count_of(t);
    T v[S::NE];
#pragma unroll
    for (int i = 0; i < S::NE; ++i) {
      const int e = tl.tid + kT * i;
      if (e < count) {
        if constexpr (kBeta) v[i] = in_global(Yt)[place(e, y1, y2, yp)];
      }
    }
#pragma unroll
    for (int i = 0; i < S::NE; ++i) {
      const int e = tl.tid + kT * i;
      if (e < count) {
        const T y = in_lds(lds)[Tiles::flat(e)];
        if constexpr (kBeta) v[i] = y + beta * v[i];
        else v[i] = y;
      }
    }
    // two loops: the compiler would merge the two kinds of store of one
    if (longer) {
#pragma unroll
      for (int i = 0; i < S::NE; ++i) {
        const int e = tl.tid + kT * i;
        if (e < count) __builtin_nontemporal_store(v[i], in_global(Yt) + place(e, y1, y2, yp));
      }
      asm volatile("");
    } else {
#pragma unroll
      for (int i = 0; i < S::NE; ++i) {
        const int e = tl.tid + kT * i;
        if (e < count) in_global(Yt)[place(e, y1, y2, yp)] = v[i];
      }
    }
  };
  T z[NC][kE] = {};
  int64_t t = blockIdx.x;
  if constexpr (Dim == 3) {
    const typename S::template Factor<false> fC(C, lane);
    T x[NC][kE] = {};
    auto load = [&](int64_t tt) {
      const T* const Xt = X + tt * P * xs.sp;
      const int64_t rem = batch - tt * P;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (tl.ok[c] && tl.op0[c] < rem) {
          const unsigned off = (unsigned)tl.op0[c] * xp + (unsigned)tl.row0[c] * x1 + (unsigned)tl.col0[c];
#pragma unroll
          for (int s = 0; s < kE; ++s)
            if (tl.has(s)) x[c][s] = in_global(Xt)[off + (unsigned)(tl.k0 + S::kd * s) * x2];
        }
    };
    if (t < ntiles) load(t);
    for (; t < ntiles; t += gridDim.x) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int s = 0; s < kE; ++s) z[c][s] = x[c][s];
      fA.template apply<NC>(z);
      if (t + gridDim.x < ntiles) load(t + gridDim.x);
      lds_barrier();  // the previous tile's results have left LDS
      tl.template put<2>(lds, z);
      lds_barrier();
      tl.template get<1>(lds, z);
      fB.template apply<NC>(z);
      tl.template put<1>(lds, z);
      lds_barrier();
      tl.template get<0>(lds, z);
      fC.template apply<NC>(z);
      tl.template put<0>(lds, z);
      lds_barrier();
      copy_out(t);
    }
  } else {
    T x[S::NE] = {};
    auto load = [&](int64_t tt) {
      const T* const Xt = X + tt * P * xs.sp;
      const int count = count_of(tt);
#pragma unroll
      for (int i = 0; i < S::NE; ++i) {
        const int e = tl.tid + kT * i;
        if (e < count) x[i] = in_global(Xt)[place(e, x1, 0, xp)];
      }
    };
    if (t < ntiles) load(t);
    for (; t < ntiles; t += gridDim.x) {
      const int count = count_of(t);
      lds_barrier();  // the previous tile's results have left LDS
#pragma unroll
      for (int i = 0; i < S::NE; ++i) {
        const int e = tl.tid + kT * i;
        if (e < count) in_lds(lds)[kTX ? S::at(e / E, e % N, e / N % N) : Tiles::flat(e)] = x[i];
      }
      lds_barrier();
      if (t + gridDim.x < ntiles) load(t + gridDim.x);
      tl.template get<1>(lds, z);
      fA.template apply<NC>(z);
      tl.template put<1>(lds, z);
      lds_barrier();
      tl.template get<0>(lds, z);
      fB.template apply<NC>(z);
      tl.template put<0>(lds, z);
      lds_barrier();
      copy_out(t);
    }
  }
}

// Whether the offsets inside a tile of `ops` operands fit 32 bits.
bool near(int dim, int n, int ops, const Strides& s) {
  const int64_t parts[3] = {s.s1, dim == 3 ? s.s2 : 0, s.sp};
  const int times[3] = {n, n, ops};
  int64_t room = kNear - n;
  for (int i = 0; i < 3; ++i) {
    if (parts[i] > kNear || parts[i] * times[i] > room) return false;
    room -= parts[i] * times[i];
  }
  return true;
}

template <typename T, int Dim, int N>
bool launch(const T* A, const T* B, const T* C, const T* X, const Strides& xs, T* Y, const Strides& ys, int64_t batch,
            T beta, bool transx, hipStream_t stream) {
  using S = Bwd<T, Dim, N>;
  if (!near(Dim, N, S::P, xs) || !near(Dim, N, S::P, ys)) return false;
  const int64_t ntiles = (batch + S::P - 1) / S::P;
  const int64_t bytes = batch * ys.sp * (int64_t)sizeof(T);
  if (N == 16 && sizeof(T) == 4 && bytes > 2 * kCached) return false;
  auto run = [&](auto k) {
    const int64_t cap = (int64_t)device_cus() * occupancy_blocks(k, S::kThreads);
    hipLaunchKernelGGL(k, dim3((unsigned)std::min(ntiles, cap)), dim3(S::kThreads), 0, stream, A, B, C, X, xs, Y, ys,
                       batch, ntiles, beta, bytes > kCached);
  };
  const bool has_beta = beta != T(0);
  if constexpr (Dim == 2) {
    if (transx) {
      if (has_beta) run(kron_strided_cols_kernel<S, true, true>);
      else run(kron_strided_cols_kernel<S, false, true>);
      return true;
    }
  }
  if (has_beta) run(kron_strided_cols_kernel<S, true, false>);
  else run(kron_strided_cols_kernel<S, false, false>);
  return true;
}

template <typename T>
bool dispatch(int dim, int n, const T* A, const T* B, const T* C, const T* X, const Strides& xs, T* Y, const Strides& ys,
         int64_t batch, T beta, bool transx, hipStream_t stream) {
  // FP64 3-D without beta: the packed call runs on columns too, so these equal
  // it, and are the faster ones (padded by 4: 32 KiB 14.3 us general, 15.0 here;
  // 64 MiB 61 and 33, 1 GiB 872 and 698).  With beta the packed call runs on
  // register tiles, in the general kernel's order.
  const bool columns = sizeof(T) == 8 && dim == 3 && beta == T(0);
  if (n == 16 && !columns && vec_strides(xs, X) && vec_strides(ys, Y)) return false;
  bool done = false;
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if (n != N) return;
    done = dim == 2 ? launch<T, 2, N>(A, B, C, X, xs, Y, ys, batch, beta, transx, stream)
                    : launch<T, 3, N>(A, B, C, X, xs, Y, ys, batch, beta, false, stream);
  });
  return done;
}

}  // namespace

bool strided_cols(int dim, int n, const float* A, const float* B, const float* C, const float* X, const Strides& xs,
                  float* Y, const Strides& ys, int64_t batch, float beta, bool transx, hipStream_t stream) {
  return dispatch(dim, n, A, B, C, X, xs, Y, ys, batch, beta, transx, stream);
}
bool strided_cols(int dim, int n, const double* A, const double* B, const double* C, const double* X,
                  const Strides& xs, double* Y, const Strides& ys, int64_t batch, double beta, bool transx,
                  hipStream_t stream) {
  return dispatch(dim, n, A, B, C, X, xs, Y, ys, batch, beta, transx, stream);
}

}  // namespace kron
