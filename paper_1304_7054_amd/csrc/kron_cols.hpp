// Column kernels: 3-D operands through workgroup tiles in LDS (FP32 n < 16, FP64
// every n, bf16 storage the sizes whose register tiles waste most).
//
// A mode product is a small matrix applied to every column (fibre) of the
// operand along one axis.  A workgroup holds P whole operands, packed back to
// back in LDS as they are in memory, so that their P * n^2 columns along any
// axis are one dense sequence; every lane takes one column into n registers,
// applies the factor and puts the n results back in place.  The columns of
// several operands fill the 64 lanes without padding, and the factor is the
// only operand padded (to a multiple of four rows), where a 16-slot tile axis
// pads both the factor and the data to 16.
//
// The product of one column per lane runs on the 4x4x1 FP32 matrix
// instruction: 16 blocks of four lanes, each block multiplying four rows of
// the factor by its four columns.  With the broadcast control (cbsz = 4) one
// block's factor values serve all 16 blocks, so a single register holds 16
// (row block, k) steps of the factor, selected by an immediate; the data
// operand is simply element k of every lane's column, and register r of the
// accumulator is row r of every lane's result.  Nothing crosses columns, so a
// NaN or Inf stays in its operand and no tile is ever redone.
#pragma once

#include <type_traits>
#include <utility>

#include "kron_staged.hpp"

namespace kron {

// Workgroup barrier that orders LDS accesses only: the global loads and
// stores in flight are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Compile-time loop: f(integral_constant<int, 0>) .. f(integral_constant<int, K - 1>).
template <int... I, class F>
__host__ __device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int K, class F>
__host__ __device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, K>{}, static_cast<F&&>(f));
}

// How a wavefront holds columns and applies a factor to them.  Each lane holds
// kE elements of each of its columns; kLanes columns lie side by side in the
// wavefront.  x[c] <- M x[c] for the lane's NC columns (M^T with kTrans).

// FP32 and bf16 storage: one column per lane, the 4x4x1 instruction.  Step
// (row block rb, index k) of the factor sits in lanes 4b .. 4b + 3 of register
// v, where 16 v + b = n * rb + k; lane 4b + i holds M(4 rb + i, k).
template <int N, bool kTrans, typename io_t, int kKind>
struct ColFactor {
  static constexpr int kE = N, kLanes = 64;
  static constexpr int kRB = (N + 3) / 4;
  static constexpr int kRegs = (kRB * N + 15) / 16;
  float v[kRegs];

  __device__ __forceinline__ ColFactor(const io_t* M, int lane) {
    const int b = lane >> 2, i = lane & 3;
#pragma unroll
    for (int r = 0; r < kRegs; ++r) {
      const int step = 16 * r + b, row = 4 * (step / N) + i, k = step % N;
      float x = 0.f;
      if (step < kRB * N && row < N) x = widen(in_global(M)[kTrans ? k + N * row : row + N * k]);
      v[r] = x;
    }
  }

  template <int NC>
  __device__ __forceinline__ void apply(float (&x)[NC][kE]) const {
    f32x4 y[NC][kRB];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb) y[c][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    static_for<N>([&](auto kk) {
      static_for<kRB>([&](auto rr) {
        constexpr int k = decltype(kk)::value, rb = decltype(rr)::value, step = rb * N + k;
#pragma unroll
        for (int c = 0; c < NC; ++c)
          y[c][rb] = __builtin_amdgcn_mfma_f32_4x4x1f32(v[step / 16], x[c][k], y[c][rb], 4, step % 16, 0);
      });
    });
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int k = 0; k < N; ++k) x[c][k] = y[c][k / 4][k % 4];
  }
};

// FP64, n <= 8: one column per lane.  The vector unit's FP64 FMA rate equals
// the matrix rate, so the product is plain FMAs with the factor entries in
// scalar registers, and neither rows nor columns are padded.  The entries are
// read again for every product, as scalar loads that hit the constant cache.
constexpr int kColScalar = 1;
template <int N, bool kTrans>
struct ColFactor<N, kTrans, double, kColScalar> {
  static constexpr int kE = N, kLanes = 64;
  const double* M;

  __device__ __forceinline__ ColFactor(const double* M_, int) : M(M_) {}

  template <int NC>
  __device__ __forceinline__ void apply(double (&x)[NC][kE]) const {
    typedef const __attribute__((address_space(4))) double* const_ptr;
    uint64_t bits = reinterpret_cast<uint64_t>(M);
    asm volatile("" : "+s"(bits));  // keeps the loads inside the tile loop: all three factors would not fit
    const_ptr m = (const_ptr)bits;
    double y[NC][N];
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const double f = m[kTrans ? k + N * i : i + N * k];
#pragma unroll
        for (int c = 0; c < NC; ++c) y[c][i] = k == 0 ? f * x[c][k] : __builtin_fma(f, x[c][k], y[c][i]);
      }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int k = 0; k < N; ++k) x[c][k] = y[c][k];
  }
};

// FP64, n > 8: the scalar registers no longer hold a useful part of a factor,
// and the padding of the 16x16x4 instruction (16 rows, n rounded up to four
// indices) is small.  16 columns per wavefront step: lane (L, g) holds
// elements g, g + 4, .. of column L, which is both the instruction's data
// operand and its result layout.
constexpr int kColMatrix = 2;
template <int N, bool kTrans>
struct ColFactor<N, kTrans, double, kColMatrix> {
  static constexpr int kE = (N + 3) / 4, kLanes = 16;
  double v[kE];

  __device__ __forceinline__ ColFactor(const double* M, int lane) {
    const int row = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < kE; ++s) {
      const int k = 4 * s + g;
      v[s] = row < N && k < N ? in_global(M)[kTrans ? k + N * row : row + N * k] : 0.0;
    }
  }

  template <int NC>
  __device__ __forceinline__ void apply(double (&x)[NC][kE]) const {
    f64x4 y[NC];
#pragma unroll
    for (int s = 0; s < kE; ++s)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (s == 0) y[c] = f64x4{0.0, 0.0, 0.0, 0.0};
        y[c] = mfma_f64(v[s], x[c][s], y[c]);
      }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int s = 0; s < kE; ++s) x[c][s] = y[c][s];
  }
};

// FP32 on the 16x16x4 instruction: lane (L, g) holds elements 4g .. 4g + 3 of
// column L, again both operand and result.
template <int N, bool kTrans>
struct ColFactor<N, kTrans, float, kColMatrix> {
  static_assert(N == 16, "every lane's four elements exist");
  static constexpr int kE = 4, kLanes = 16;
  float v[kE];

  __device__ __forceinline__ ColFactor(const float* M, int lane) {
    const int row = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < kE; ++s) v[s] = in_global(M)[kTrans ? 4 * g + s + N * row : row + N * (4 * g + s)];
  }

  template <int NC>
  __device__ __forceinline__ void apply(float (&x)[NC][kE]) const {
    f32x4 y[NC];
#pragma unroll
    for (int s = 0; s < kE; ++s)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (s == 0) y[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        y[c] = mfma_f32(v[s], x[c][s], y[c]);
      }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int s = 0; s < kE; ++s) x[c][s] = y[c][s];
  }
};

template <int N, typename io_t>
constexpr int col_kind() {
  return sizeof(io_t) != 8 ? 0 : N <= 8 ? kColScalar : kColMatrix;
}

// Operands per workgroup tile and wavefronts per workgroup, the fastest of a
// sweep at 1 GiB of operands: the tile's columns fill the lanes (n = 10: 400 of
// 448), and tiles stay near 16 KiB, so that several workgroups per CU hide each
// other's barriers.  per_cu (0: as many as are resident) is the workgroups per
// CU for operands of kColLong bytes and more, where a few long streams suit the
// memory better (1 GiB, FP64 n = 4: 358 us with 2, 451 with all 8; FP32 n = 7:
// 414 with 1, 431 with all 4); below, as many as fit (256 MiB, FP64 n = 4: 82
// and 81 us; FP32 n = 7: 118 and 86; 16 MiB: 10.8 and 7.7).
constexpr int64_t kColLong = (int64_t)512 << 20;
struct ColShape {
  int ops, waves, per_cu;
};

template <int N, typename io_t>
constexpr ColShape col3d_shape() {
  constexpr ColShape s4[17] = {{0, 0, 0},  {512, 4, 0}, {128, 4, 4}, {56, 4, 4}, {16, 4, 4}, {10, 4, 4},
                               {14, 4, 2}, {15, 6, 1},  {8, 4, 2},   {6, 4, 3},  {4, 7, 3},  {4, 8, 1},
                               {2, 5, 2},  {1, 3, 4},   {1, 4, 4},   {1, 4, 4},  {0, 0, 0}};
  constexpr ColShape s8[17] = {{0, 0, 0}, {512, 4, 4}, {64, 4, 4}, {28, 4, 3}, {16, 4, 2}, {10, 4, 2},
                               {7, 4, 2}, {10, 8, 1},  {4, 4, 0},  {3, 4, 3},  {1, 2, 0},  {1, 2, 4},
                               {1, 3, 4}, {1, 4, 4},   {1, 7, 2},  {1, 8, 4},  {1, 8, 4}};
  constexpr int per2[17] = {0, 0, 0, 0, 0, 0, 0, 4, 0, 4, 3, 4, 0, 0, 0, 0, 0};  // bf16: the FP32 tiles
  if (sizeof(io_t) == 8) return s8[N];
  if (sizeof(io_t) == 2) return ColShape{s4[N].ops, s4[N].waves, per2[N]};
  return s4[N];
}

template <class M, int N, bool kTrans, int P_ = col3d_shape<N, typename M::io_t>().ops,
          int W_ = col3d_shape<N, typename M::io_t>().waves, int kKind = col_kind<N, typename M::io_t>()>
struct Col3D {
  using io_t = typename M::io_t;
  using elem_t = std::conditional_t<sizeof(io_t) == 8, double, float>;
  using Factor = ColFactor<N, kTrans, io_t, kKind>;
  static constexpr int kN = N;
  static constexpr int P = P_;
  static constexpr int kThreads = 64 * W_;
  static constexpr int E = N * N * N;
  static constexpr int kCols = P * N * N;
  static constexpr int kE = Factor::kE;
  static constexpr int kStep = Factor::kLanes * W_;  // columns a workgroup holds per c
  static constexpr int NC = (kCols + kStep - 1) / kStep;
  // n = 4 and 8: planes of n^2 elements at a pitch that spreads the rows of a
  // middle-axis read over the banks (flat, every row of n = 8 starts in bank 0)
  static constexpr int kPad = N == 8 ? 8 : N == 4 ? 4 : 0;
  // n = 16: rows of 16 at a pitch of 18, for the reads along the fast axis
  static constexpr int RP = N == 16 ? 18 : N;
  static constexpr int PL = N * RP + kPad;
  // Odd n: a tile can start anywhere between two 16-byte boundaries of Y, and
  // is moved by up to a vector in LDS so that its output vectors are aligned
  // there too.  Even n: tiles start on a boundary whenever Y does.
  static constexpr bool kShift = N % 2 == 1;
  static constexpr int kLds = P * N * PL + 4;
  // element of the tile (in memory order) -> LDS offset
  __device__ static constexpr int at(int e) {
    return RP == N && kPad == 0 ? e : (e / (N * N)) * PL + ((e / N) % N) * RP + e % N;
  }
};

// A workgroup's column kernel: its factors, the places of its columns, and the
// tile loop.  The products run slow axis first, each in place.
//
// The slow-axis columns come from memory straight into the registers that the
// first product reads (consecutive lanes, consecutive addresses), the next
// tile's while the current one is in LDS; through 16-byte vectors and LDS
// instead, one more pass over LDS, every size measured slower (FP32 n = 10:
// 4.7 against 5.2 TB/s).  The results leave LDS as 16-byte vectors.  What
// bounds it is the six passes over LDS per element and, from n = 12 on, the
// matrix cores, both a little below the time of the memory traffic.
template <class S>
struct ColTiles {
  using io_t = typename S::io_t;
  using elem_t = typename S::elem_t;
  using Factor = typename S::Factor;
  static constexpr int P = S::P, NC = S::NC, E = S::E, PL = S::PL, RP = S::RP, kT = S::kThreads, kE = S::kE, N = S::kN;
  static constexpr bool kMat = Factor::kLanes == 16;
  static constexpr int V = 16 / (int)sizeof(io_t), W = 16 / (int)sizeof(elem_t);  // a vector in memory, in LDS
  // element s of a lane's column is element k0 + kd * s of the column
  static constexpr int kd = kMat ? 4 : 1;
  // fast-axis columns: their elements are consecutive, in vectors where n allows
  static constexpr int F = kMat ? 1 : N % W == 0 ? W : N % 2 == 0 ? 2 : 1;
  typedef io_t vec_t __attribute__((ext_vector_type(V)));
  typedef elem_t wide_t __attribute__((ext_vector_type(W)));
  typedef elem_t fast_t __attribute__((ext_vector_type(F)));

  const Factor fA, fB, fC;
  const int tid, k0;
  // this lane's columns on each axis: LDS offset of element k0 (the slow-axis
  // column's offset in memory is ga); operand P: no column
  int la[NC], lb[NC], lc[NC], ga[NC], pa[NC];
  elem_t x[NC][kE], z[NC][kE];

  __device__ __forceinline__ ColTiles(const io_t* A, const io_t* B, const io_t* C)
      : fA(A, threadIdx.x & 63),
        fB(B, threadIdx.x & 63),
        fC(C, threadIdx.x & 63),
        tid(threadIdx.x),
        k0(kMat ? (threadIdx.x & 63) >> 4 : 0) {
    const int q0 = kMat ? 16 * (tid >> 6) + (tid & 15) : tid;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int q = q0 + S::kStep * c, p = q / (N * N), r = q % (N * N);
      ga[c] = p * E + r + k0 * N * N;
      pa[c] = q < S::kCols ? p : P;
      la[c] = p * N * PL + S::at(r) + k0 * PL;
      lb[c] = (q / N) * PL + q % N + k0 * RP;
      lc[c] = (q / N) * PL + (q % N) * RP + k0;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int s = 0; s < kE; ++s) x[c][s] = z[c][s] = 0;
  }

  // whether the column has element k0 + kd * s
  __device__ __forceinline__ bool has(int s) const { return !kMat || N % 4 == 0 || s + 1 < kE || k0 + kd * s < N; }

  __device__ __forceinline__ void load(const io_t* X, int64_t t, int64_t batch) {
    const io_t* Xt = X + t * (int64_t)(P * E);
    const int64_t rem = batch - t * P;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (pa[c] < P && pa[c] < rem) {
#pragma unroll
        for (int s = 0; s < kE; ++s)
          if (has(s)) x[c][s] = widen(in_global(Xt)[ga[c] + kd * s * N * N]);
      }
  }

  __device__ __forceinline__ void get(const elem_t* lds, const int (&base)[NC], int stride) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (pa[c] < P) {
#pragma unroll
        for (int s = 0; s < kE; ++s) z[c][s] = has(s) ? in_lds(lds)[base[c] + kd * s * stride] : elem_t(0);
      }
  }
  __device__ __forceinline__ void put(elem_t* lds, const int (&base)[NC], int stride) const {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (pa[c] < P) {
#pragma unroll
        for (int s = 0; s < kE; ++s)
          if (has(s)) in_lds(lds)[base[c] + kd * s * stride] = z[c][s];
      }
  }
  __device__ __forceinline__ void get_fast(const elem_t* lds) {
    if constexpr (F == 1) {
      get(lds, lc, 1);
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (pa[c] < P) {
#pragma unroll
          for (int s = 0; s < kE / F; ++s) {
            const fast_t v = in_lds(reinterpret_cast<const fast_t*>(lds + lc[c]))[s];
#pragma unroll
            for (int j = 0; j < F; ++j) z[c][F * s + j] = v[j];
          }
        }
    }
  }
  __device__ __forceinline__ void put_fast(elem_t* lds) const {
    if constexpr (F == 1) {
      put(lds, lc, 1);
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (pa[c] < P) {
#pragma unroll
          for (int s = 0; s < kE / F; ++s) {
            fast_t v;
#pragma unroll
            for (int j = 0; j < F; ++j) v[j] = z[c][F * s + j];
            in_lds(reinterpret_cast<fast_t*>(lds + lc[c]))[s] = v;
          }
        }
    }
  }

  // Tiles t, t + step, .. below tend of a batch (the same for the whole
  // workgroup); lds: S::kLds elements, 16-byte aligned.
  __device__ __forceinline__ void run(const io_t* X, io_t* Y, int64_t batch, int64_t t, int64_t tend, int64_t step,
                                      elem_t* slice) {
    if (t < tend) load(X, t, batch);
    for (; t < tend; t += step) {
      const int64_t rem = batch - t * P;
      io_t* Yt = Y + t * (int64_t)(P * E);
      const int count = (int)(rem < P ? rem : P) * E;
      const int head = head_elems(Yt, count);
      elem_t* lds = slice;
      if constexpr (S::kShift) lds += (16 - head) & (W - 1);
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int s = 0; s < kE; ++s) z[c][s] = x[c][s];
      fA.template apply<NC>(z);
      if (t + step < tend) load(X, t + step, batch);
      lds_barrier();  // the previous tile's results have left LDS
      put(lds, la, PL);
      lds_barrier();
      get(lds, lb, RP);
      fB.template apply<NC>(z);
      put(lds, lb, RP);
      lds_barrier();
      get_fast(lds);
      fC.template apply<NC>(z);
      put_fast(lds);
      lds_barrier();
      copy_out(Yt, lds, count, head);
    }
  }

  // Results out: 16-byte vectors from the first 16-byte boundary of Y on.
  __device__ __forceinline__ void copy_out(io_t* Yt, const elem_t* lds, int count, int head) const {
    const int nv = (count - head) / V, done = head + nv * V;
    for (int i = tid; i < nv; i += kT) {
      vec_t o;
      if (S::kShift || head == 0) {  // aligned in LDS too
        const wide_t* src = reinterpret_cast<const wide_t*>(lds + S::at(head + V * i));
#pragma unroll
        for (int w = 0; w < V / W; ++w) {
          const wide_t v = in_lds(src)[w];
#pragma unroll
          for (int j = 0; j < W; ++j) o[W * w + j] = narrow<io_t>(v[j]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) o[j] = narrow<io_t>(in_lds(lds)[S::at(head + V * i + j)]);
      }
      __builtin_nontemporal_store(o, in_global(reinterpret_cast<vec_t*>(Yt + head)) + i);
    }
    if (tid < head + count - done) {
      const int e = tid < head ? tid : done + tid - head;
      __builtin_nontemporal_store(narrow<io_t>(in_lds(lds)[S::at(e)]), in_global(Yt) + e);
    }
  }
};

// At least two wavefronts per SIMD (at most 256 registers): the compiler then
// keeps the matrix results in vector registers.  With accumulation registers
// it pairs LDS stores wrongly: FP32 n = 8 stores rows 4 and 5 of a plane as
// ds_write2_b32 at elements 8 and 40, not 32 and 40, the byte offset 128 divided
// by 4 twice.  A host test holds every kernel that writes columns to none.
template <class S>
__global__ __launch_bounds__(S::kThreads) __attribute__((amdgpu_waves_per_eu(2))) void kron3d_cols_kernel(
    const typename S::io_t* __restrict__ A, const typename S::io_t* __restrict__ B,
    const typename S::io_t* __restrict__ C, const typename S::io_t* __restrict__ X, typename S::io_t* __restrict__ Y,
    int64_t batch, int64_t ntiles) {
  __shared__ __attribute__((aligned(16))) typename S::elem_t lds[S::kLds];
  ColTiles<S> tiles(A, B, C);
  tiles.run(X, Y, batch, blockIdx.x, ntiles, gridDim.x, lds);
}

}  // namespace kron
