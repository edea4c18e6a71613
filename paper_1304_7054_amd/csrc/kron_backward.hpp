// The whole backward of a batch with shared factors in one pass: dX and the
// partial sums of dA, dB (, dC), FP32 and FP64, any n.
//
// A workgroup holds P operands of X and of D = dY in LDS (the column layout of
// kron_cols.hpp).  Every factor gradient pairs X, transformed on some axes,
// with D, transformed on the others, and contracts all columns along the
// factor's own axis:
//   3-D  D1 = C^T on the fast axis of D, D2 = B^T on the middle axis of D1,
//        X1 = A on the slow axis of X, X2 = B on the middle axis of X1:
//        dA(i, a) = sum D2(i, ..) X(a, ..)      over the slow-axis columns
//        dB(j, b) = sum D1(j, ..) X1(b, ..)     over the middle-axis columns
//        dC(k, c) = sum D(k, ..) X2(c, ..)      over the fast-axis columns
//        dX = A^T on the slow axis of D2
//   2-D  D1 = B^T on the fast axis of D, X1 = A on the slow axis of X:
//        dA(i, u) = sum D1(i, ..) X(u, ..),  dB(j, v) = sum D(j, ..) X1(v, ..),
//        dX = A^T on the slow axis of D1
// so the chains of X and of D serve all gradients and dX: five products and
// three contractions in 3-D, where separate gradients take nine and three.
// Three LDS images (X, D and a work image) suffice, because X1 and D1 wait in
// registers while the work image holds D2.
//
// A contraction from n = 9 on takes four columns per 16x16x4 instruction: lane
// (L, g) reads element L of column g of both images.  Its rows and columns
// beyond n hold values that no result uses, so only missing columns are masked.
// Up to n = 4 and 8 that wastes most of the products (n^2 / 256 of them count),
// and the smaller forms below take their place: with every gradient and dX at
// 128 MiB of X, FP32 3-D n = 2 took 679 us a training step and now takes 150,
// FP32 3-D n = 5 229 us a backward and now 144, FP64 3-D n = 5 204 and now 99.
#pragma once

#include "kron_cols.hpp"

namespace kron {

// Operands per tile, wavefronts per workgroup, and wavefronts per SIMD the
// registers are held to.  At 512 MiB of X, FP32 3-D n = 16: three workgroups of
// four wavefronts fit a CU (408 us; two of eight: 430).  At 128 MiB: FP32 3-D
// n = 5 to 8 at 3 a SIMD, because at 5 the sums spill (n = 8: 101 against
// 333 us); FP64 2-D at 3 a SIMD on tiles that let three or more workgroups
// share a CU (n = 8: 185 to 90 us, n = 12: 148 to 111, n = 16: 176 to 99).
// Twice and four times the operands for n <= 4: up to three times slower.
struct BwdShape {
  int ops, waves, per_simd;
};

template <int Dim, int N, typename T>
constexpr BwdShape bwd_shape() {
  constexpr int f3[17] = {0, 256, 64, 28, 16, 10, 7, 5, 4, 3, 2, 2, 1, 1, 1, 1, 1};
  constexpr int w3[17] = {0, 4, 4, 4, 4, 4, 4, 4, 4, 4, 4, 4, 3, 3, 4, 4, 4};
  constexpr int d3[17] = {0, 256, 64, 28, 16, 10, 7, 5, 4, 1, 1, 1, 1, 1, 1, 1, 1};
  constexpr int v3[17] = {0, 4, 4, 4, 4, 4, 4, 4, 4, 4, 4, 4, 5, 6, 7, 8, 8};
  if (Dim == 3) {
    if (sizeof(T) == 8) return BwdShape{d3[N], v3[N], 2};
    return BwdShape{f3[N], w3[N], N <= 4 ? 5 : N <= 8 ? 3 : N <= 12 ? 4 : 3};
  }
  if (sizeof(T) == 8) return BwdShape{N <= 4 ? 256 / N : N <= 8 || N > 12 ? 128 / N : 64 / N, N <= 4 || N > 8 ? 4 : 2, 3};
  return BwdShape{N < 16 ? 256 / N : 8, 4, N >= 12 && N < 16 ? 3 : 4};
}

template <typename T, int Dim_, int N_>
struct Bwd {
  using io_t = T;
  static constexpr int Dim = Dim_, N = N_;
  static constexpr int P = bwd_shape<Dim, N, T>().ops, kWaves = bwd_shape<Dim, N, T>().waves;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kKind = N == 16 ? kColMatrix : col_kind<N, T>();
  template <bool kTrans>
  using Factor = ColFactor<N, kTrans, T, kKind>;
  static constexpr bool kMat = Factor<false>::kLanes == 16;
  static constexpr int kE = Factor<false>::kE, kd = kMat && sizeof(T) == 8 ? 4 : 1;
  static constexpr int E = Dim == 3 ? N * N * N : N * N;
  static constexpr int NP = Dim == 3 ? P * N : P;  // planes of n rows
  static constexpr int kCols = NP * N;             // columns along any axis
  static constexpr int NC = (kCols + Factor<false>::kLanes * kWaves - 1) / (Factor<false>::kLanes * kWaves);
  static constexpr int NE = (P * E + kThreads - 1) / kThreads;  // elements per thread (2-D loads)
  // n = 16: row b of a plane holds its groups of four at (group ^ (b / 4)), so
  // that neither a read along the rows nor one down them meets a bank twice;
  // with padded rows instead, three images of two workgroups fill a CU, so
  // three.  Planes at pitches that spread the slow-axis reads.
  static constexpr int kMinWaves = bwd_shape<Dim, N, T>().per_simd;
  static constexpr int PL = N == 16 ? 276 : N * N + (N == 8 ? 8 : N == 4 || N == 12 ? 4 : 0);
  static constexpr int kImage = NP * PL;
  // FP64 n = 4 and 8: row b holds element c at (c ^ b); the reads of a row per
  // lane met 16 of the 64 banks otherwise (2-D n = 8 at 128 MiB: 255 us).
  __device__ static constexpr int swz(int row) {
    return N == 16 ? 4 * (row >> 2) : sizeof(T) == 8 && (N == 4 || N == 8) ? row : 0;
  }
  __device__ static constexpr int at(int plane, int row, int col) { return plane * PL + row * N + (col ^ swz(row)); }
};

template <class S>
struct BwdTiles {
  using T = typename S::io_t;
  static constexpr int N = S::N, P = S::P, NC = S::NC, kE = S::kE, kd = S::kd, PL = S::PL, kT = S::kThreads;
  using acc_t = std::conditional_t<sizeof(T) == 8, f64x4, f32x4>;
  typedef T regs_t[NC][kE];
  // n <= 4: a lane sums the outer products of its own columns, n * n sums a
  // gradient; a 16x16x4 instruction would use n^3 / 1024 of its products.
  static constexpr bool kOwn = N <= 4;
  struct own_t {
    T v[N * N];
  };
  // n = 5 to 8: 4x4x1 (FP64: 4x4x4) instructions, 16 columns each, two by two
  // for the entries, where a 16x16x4 takes four columns of at most half its
  // rows.  Lane i of a column holds elements 2i and 2i + 1; v[ti][tj] holds
  // entries (2r + ti, 2j + tj), j being the lane mod 4 and r the register
  // (FP64: the lane over 16), for the column groups of the other lane bits.
  static constexpr bool kQuad = N > 4 && N <= 8;
  struct quad_t {
    std::conditional_t<sizeof(T) == 8, T, f32x4> v[2][2];
  };
  using sum_t = std::conditional_t<kOwn, own_t, std::conditional_t<kQuad, quad_t, acc_t>>;

  const int tid, wave, k0, q0;
  int plane1[NC], fast1[NC];  // column q as (plane, position) of the middle and fast axes
  int op0[NC], row0[NC], col0[NC];  // 3-D slow-axis column: operand, row, position
  bool ok[NC];

  __device__ __forceinline__ BwdTiles()
      : tid(threadIdx.x),
        wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)),
        k0(S::kMat ? ((threadIdx.x & 63) >> 4) * (kd == 4 ? 1 : 4) : 0),
        q0(S::kMat ? 16 * (threadIdx.x >> 6) + (threadIdx.x & 15) : threadIdx.x) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int q = q0 + (S::kMat ? 16 : 64) * S::kWaves * c;
      ok[c] = q < S::kCols;
      plane1[c] = q / N;
      fast1[c] = q % N;
      op0[c] = q / (N * N);
      row0[c] = q / N % N;
      col0[c] = q % N;
    }
  }

  __device__ __forceinline__ static int lane() { return threadIdx.x & 63; }
  __device__ __forceinline__ bool has(int s) const { return !S::kMat || N % 4 == 0 || s + 1 < kE || k0 + kd * s < N; }

  // LDS offset of element s of column c along an axis: 0 the fast one, 1 the
  // one above it (3-D: middle, 2-D: slow), 2 the 3-D slow one.
  template <int kAxis>
  __device__ __forceinline__ int where(int c, int s) const {
    const int k = k0 + kd * s;
    if constexpr (kAxis == 0) return plane1[c] * PL + fast1[c] * N + (k ^ S::swz(fast1[c]));
    if constexpr (kAxis == 1) return plane1[c] * PL + k * N + (fast1[c] ^ S::swz(k));
    return (op0[c] * N + k) * PL + row0[c] * N + (col0[c] ^ S::swz(row0[c]));
  }
  template <int kAxis>
  __device__ __forceinline__ void get(const T* img, regs_t& z) const {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (ok[c]) {
        if constexpr (kAxis == 0 && N % 4 == 0 && sizeof(T) == 4) {
#pragma unroll
          for (int s = 0; s < kE; s += 4) {
            const f32x4 v = *in_lds(reinterpret_cast<const f32x4*>(img + where<0>(c, s)));
#pragma unroll
            for (int j = 0; j < 4; ++j) z[c][s + j] = v[j];
          }
        } else {
#pragma unroll
          for (int s = 0; s < kE; ++s) z[c][s] = has(s) ? in_lds(img)[where<kAxis>(c, s)] : T(0);
        }
      }
  }
  template <int kAxis>
  __device__ __forceinline__ void put(T* img, const regs_t& z) const {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (ok[c]) {
        if constexpr (kAxis == 0 && N % 4 == 0 && sizeof(T) == 4) {
#pragma unroll
          for (int s = 0; s < kE; s += 4)
            *in_lds(reinterpret_cast<f32x4*>(img + where<0>(c, s))) = f32x4{z[c][s], z[c][s + 1], z[c][s + 2], z[c][s + 3]};
        } else {
#pragma unroll
          for (int s = 0; s < kE; ++s)
            if (has(s)) in_lds(img)[where<kAxis>(c, s)] = z[c][s];
        }
      }
  }

  // sum += sum over the columns of the tile's first `planes` planes (3-D slow
  // axis: rows) of U(i, column) V(j, column), for all i and j.
  // Up to n = 8 every column goes straight to a running sum: a lane's (n <= 4), or
  // that of one of a wavefront's 16 column groups.
  template <int kAxis>
  __device__ __forceinline__ void contract(const T* U, const T* V, int planes, own_t& sum) const {
    regs_t u, v;
    get<kAxis>(U, u);
    get<kAxis>(V, v);
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (ok[c] && (kAxis == 2 ? op0[c] * N : plane1[c]) < planes) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int j = 0; j < N; ++j) sum.v[i * N + j] += u[c][i] * v[c][j];
      }
  }
  template <int kAxis>
  __device__ __forceinline__ void contract(const T* U, const T* V, int planes, quad_t& sum) const {
    const int i = threadIdx.x & 3, k0 = min(2 * i, N - 1), k1 = min(2 * i + 1, N - 1);
#pragma unroll
    for (int r = 0; r < (S::kCols + 16 * S::kWaves - 1) / (16 * S::kWaves); ++r) {
      const int q = 16 * (S::kWaves * r + wave) + (lane() >> 2);
      // element k of column q
      auto at = [&](int k) {
        if constexpr (kAxis == 0) return S::at(q / N, q % N, k);
        else if constexpr (kAxis == 1) return S::at(q / N, k, q % N);
        else return S::at(q / (N * N) * N + k, q / N % N, q % N);
      };
      T u[2] = {0, 0}, v[2] = {0, 0};
      if (q < planes * N) {
        u[0] = in_lds(U)[at(k0)];
        u[1] = in_lds(U)[at(k1)];
        v[0] = in_lds(V)[at(k0)];
        v[1] = in_lds(V)[at(k1)];
      }
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          if constexpr (sizeof(T) == 8)
            sum.v[a][b] = __builtin_amdgcn_mfma_f64_4x4x4f64(u[a], v[b], sum.v[a][b], 0, 0, 0);
          else
            sum.v[a][b] = __builtin_amdgcn_mfma_f32_4x4x1f32(u[a], v[b], sum.v[a][b], 0, 0, 0);
    }
  }
  // n > 8: the wavefronts take planes in turn.  A tile's columns are summed by
  // themselves first, in two chains that keep the matrix pipe fed, so that the
  // running sum grows by one rounding per tile instead of one per column.
  template <int kAxis>
  __device__ __forceinline__ void contract(const T* U, const T* V, int planes, acc_t& sum) const {
    acc_t acc[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
    add_columns<kAxis>(U, V, planes, acc);
    sum += acc[0] + acc[1];
  }
  template <int kAxis>
  __device__ __forceinline__ void add_columns(const T* U, const T* V, int planes, acc_t (&acc)[2]) const {
    const int l = threadIdx.x & 63, g = l >> 4, L = (l & 15) < N ? (l & 15) : N - 1;
    constexpr int G = (N + 3) / 4;
    if constexpr (N == 16 && kAxis != 0) {
      // columns 4g .. 4g + 3 of a row are consecutive: one vector per image
      typedef T vec_t __attribute__((ext_vector_type(4)));
      for (int r = wave; r < planes; r += S::kWaves) {
        const int e = kAxis == 1 ? S::at(r, L, 4 * g) : r / N * (N * PL) + S::at(L, r % N, 4 * g);
        const vec_t u = *in_lds(reinterpret_cast<const vec_t*>(U + e)), v = *in_lds(reinterpret_cast<const vec_t*>(V + e));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (sizeof(T) == 8) acc[j & 1] = mfma_f64(u[j], v[j], acc[j & 1]);
          else acc[j & 1] = mfma_f32(u[j], v[j], acc[j & 1]);
        }
      }
      return;
    }
    int lane[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
      if constexpr (kAxis == 0) lane[j] = (4 * j + g < N ? 4 * j + g : 0) * N + (L ^ S::swz(4 * j + g));
      else if constexpr (kAxis == 1) lane[j] = L * N + ((4 * j + g) ^ S::swz(L));
      else lane[j] = L * PL;
    }
    for (int r = wave; r < planes; r += S::kWaves) {
      int off, sw = 0;
      if constexpr (kAxis == 2) {
        const int p = r / N, b = r % N;
        off = p * N * PL + b * N;
        sw = S::swz(b);
      } else {
        off = r * PL;
      }
#pragma unroll
      for (int j = 0; j < G; ++j) {
        int e = lane[j] + off;
        if constexpr (kAxis == 2) e += (4 * j + g) ^ sw;
        T u, v;
        if (N % 4 != 0 && j == G - 1) {
          const bool in = 4 * j + g < N;
          u = in ? in_lds(U)[e] : T(0);
          v = in ? in_lds(V)[e] : T(0);
        } else {
          u = in_lds(U)[e];
          v = in_lds(V)[e];
        }
        if constexpr (sizeof(T) == 8) acc[j & 1] = mfma_f64(u, v, acc[j & 1]);
        else acc[j & 1] = mfma_f32(u, v, acc[j & 1]);
      }
    }
  }

  // 3-D: the slow-axis columns of tile t of an array
  __device__ __forceinline__ void load_cols(const T* A, int64_t t, int64_t batch, regs_t& z) const {
    const T* At = A + t * (int64_t)(P * S::E);
    const int64_t rem = batch - t * P;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (ok[c] && op0[c] < rem) {
#pragma unroll
        for (int s = 0; s < kE; ++s)
          if (has(s)) z[c][s] = in_global(At)[op0[c] * S::E + (k0 + kd * s) * N * N + row0[c] * N + col0[c]];
      }
  }
  __device__ __forceinline__ void store_cols(T* A, int64_t t, int64_t batch, const regs_t& z) const {
    T* At = A + t * (int64_t)(P * S::E);
    const int64_t rem = batch - t * P;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (ok[c] && op0[c] < rem) {
#pragma unroll
        for (int s = 0; s < kE; ++s)
          if (has(s)) in_global(At)[op0[c] * S::E + (k0 + kd * s) * N * N + row0[c] * N + col0[c]] = z[c][s];
      }
  }
  // 2-D: the tile's elements in memory order, consecutive lanes
  __device__ __forceinline__ void load_flat(const T* A, int64_t t, int count, T (&r)[S::NE]) const {
#pragma unroll
    for (int i = 0; i < S::NE; ++i) {
      const int e = tid + kT * i;
      if (e < count) r[i] = in_global(A + t * (int64_t)(P * S::E))[e];
    }
  }
  __device__ __forceinline__ static int flat(int e) { return S::at(e / (N * N), e / N % N, e % N); }
};

// LDS elements of a workgroup: the images, or at the end the sums of the
// wavefronts, or one factor's of the lanes.
template <class S>
constexpr int backward_lds() {
  using Tiles = BwdTiles<S>;
  constexpr int kRed = Tiles::kOwn    ? S::kThreads * S::N * S::N
                       : Tiles::kQuad ? S::kThreads * 16
                                      : S::kWaves * S::Dim * 256;
  return 3 * S::kImage > kRed ? 3 * S::kImage : kRed;
}

// Workgroup `block` of `nblocks`: its tiles and its partial sums.  `which` bit
// f asks for factor f's gradient, of at least one; dX may be null.  Partials:
// ws[(block * 3 + f) * 256 + row * 16 + col].
//
// The tests of `which` always hold.  They part loads, LDS writes and products
// into blocks that the compiler schedules by themselves; without them FP64 3-D
// n = 8 takes 84 us for dA alone, 63 with (128 MiB of X), n = 10 220 and 209
// for everything.
template <class S>
__device__ __forceinline__ void backward_block(
    typename S::io_t* const lds, const typename S::io_t* __restrict__ A, const typename S::io_t* __restrict__ B,
    const typename S::io_t* __restrict__ C, const typename S::io_t* __restrict__ X,
    const typename S::io_t* __restrict__ dY, typename S::io_t* __restrict__ dX, typename S::io_t* __restrict__ ws,
    const int64_t batch, const int which, const unsigned block, const unsigned nblocks) {
  using T = typename S::io_t;
  using Tiles = BwdTiles<S>;
  constexpr int N = S::N, P = S::P, NC = S::NC, kE = S::kE, Dim = S::Dim, kWaves = S::kWaves;
  const int64_t ntiles = (batch + P - 1) / P;
  T* const ix = lds;
  T* const id = lds + S::kImage;
  T* const iw = lds + 2 * S::kImage;
  const Tiles tl;
  const int lane = threadIdx.x & 63;
  typename Tiles::sum_t acc[Dim] = {};
  const bool wa = which & 1, wb = which & 2, wc = which & 4;
  const typename S::template Factor<false> fA(A, lane);
  const typename S::template Factor<true> tA(A, lane), tB(B, lane);
  T z[NC][kE] = {}, x1[NC][kE] = {};
  if constexpr (Dim == 3) {
    const typename S::template Factor<false> fB(B, lane);
    const typename S::template Factor<true> tC(C, lane);
    T x[NC][kE] = {}, d[NC][kE] = {}, d1[NC][kE] = {};
    int64_t t = block;
    if (t < ntiles) {
      if (which) tl.load_cols(X, t, batch, x);
      tl.load_cols(dY, t, batch, d);
    }
    for (; t < ntiles; t += nblocks) {
      const int64_t rem = batch - t * P;
      const int planes = (int)(rem < P ? rem : P) * N;
      lds_barrier();  // every wavefront is done with the previous tile's images
      tl.template put<2>(id, d);
      if (which) {
        tl.template put<2>(ix, x);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int s = 0; s < kE; ++s) x1[c][s] = x[c][s];
        fA.template apply<NC>(x1);
      }
      lds_barrier();
      if (t + nblocks < ntiles) {
        if (which) tl.load_cols(X, t + nblocks, batch, x);
        tl.load_cols(dY, t + nblocks, batch, d);
      }
      // dC alone takes D as it is (FP64, 128 MiB of X: n = 13 140 us with D1, 117
      // without).  Up to n = 8 and in FP32 it is not bound by the products, and
      // the test costs the other gradients up to 5 % (FP32 n = 2).
      if (sizeof(T) == 4 || N <= 8 || wa || wb || dX) {
        tl.template get<0>(id, d1);
        tC.template apply<NC>(d1);
        tl.template put<0>(iw, d1);
        lds_barrier();
      }
      if (wa || dX) {
        tl.template get<1>(iw, z);
        tB.template apply<NC>(z);
        tl.template put<1>(iw, z);
        lds_barrier();
        if (wa) tl.template contract<2>(iw, ix, planes, acc[0]);
        if (dX) {
          tl.template get<2>(iw, z);
          tA.template apply<NC>(z);
          tl.store_cols(dX, t, batch, z);
        }
        if (!(wb || wc)) continue;
        lds_barrier();
        if (wb) tl.template put<0>(iw, d1);
      }
      tl.template put<2>(ix, x1);
      lds_barrier();
      if (wb) tl.template contract<1>(iw, ix, planes, acc[1]);
      if (wc) {
        tl.template get<1>(ix, z);
        fB.template apply<NC>(z);
        lds_barrier();
        tl.template put<1>(ix, z);
        lds_barrier();
        tl.template contract<0>(id, ix, planes, acc[2]);
      }
    }
  } else {
    T x[S::NE] = {}, d[S::NE] = {};
    auto count_of = [&](int64_t t) {
      const int64_t rem = batch - t * P;
      return (int)(rem < P ? rem : P) * S::E;
    };
    int64_t t = block;
    if (t < ntiles) {
      if (which) tl.load_flat(X, t, count_of(t), x);
      tl.load_flat(dY, t, count_of(t), d);
    }
    for (; t < ntiles; t += nblocks) {
      const int count = count_of(t), planes = count / S::E;
      lds_barrier();  // every wavefront is done with the previous tile's images
#pragma unroll
      for (int i = 0; i < S::NE; ++i) {
        const int e = tl.tid + S::kThreads * i;
        if (e < count) {
          in_lds(id)[Tiles::flat(e)] = d[i];
          if (which) in_lds(ix)[Tiles::flat(e)] = x[i];
        }
      }
      lds_barrier();
      const int64_t tn = t + nblocks;
      if (tn < ntiles) {
        if (which) tl.load_flat(X, tn, count_of(tn), x);
        tl.load_flat(dY, tn, count_of(tn), d);
      }
      if (wa || dX) {
        tl.template get<0>(id, z);
        tB.template apply<NC>(z);
        tl.template put<0>(iw, z);
      }
      if (wb) {
        tl.template get<1>(ix, x1);
        fA.template apply<NC>(x1);
      }
      lds_barrier();
      if (wa) tl.template contract<1>(iw, ix, planes, acc[0]);
      if (dX) {
        tl.template get<1>(iw, z);
        tA.template apply<NC>(z);
      }
      lds_barrier();
      if (dX) tl.template put<1>(iw, z);
      if (wb) tl.template put<1>(ix, x1);
      lds_barrier();
      if (wb) tl.template contract<0>(id, ix, planes, acc[1]);
      if (dX) {
        T* dXt = dX + t * (int64_t)(P * S::E);
        for (int e = tl.tid; e < count; e += S::kThreads) in_global(dXt)[e] = in_lds(iw)[Tiles::flat(e)];
      }
    }
  }
  if constexpr (Tiles::kOwn) {
    // 16 lanes an entry: each sums every sixteenth of the lanes' sums
    static_assert(S::kThreads >= 16 * N * N, "16 lanes an entry");
#pragma unroll
    for (int f = 0; f < Dim; ++f) {
      lds_barrier();
#pragma unroll
      for (int e = 0; e < N * N; ++e) in_lds(lds)[e * S::kThreads + tl.tid] = acc[f].v[e];
      lds_barrier();
      const int e = tl.tid >> 4;
      T sum = 0;
      if (e < N * N) {
#pragma unroll
        for (int i = 0; i < S::kThreads; i += 16) sum += in_lds(lds)[e * S::kThreads + (tl.tid & 15) + i];
      }
#pragma unroll
      for (int h = 8; h > 0; h >>= 1) sum += __shfl_xor(sum, h);
      if (e < N * N && (tl.tid & 15) == 0) ws[((int64_t)block * 3 + f) * 256 + e / N * 16 + e % N] = sum;
    }
  } else if constexpr (Tiles::kQuad) {
    // kWaves lanes an entry: each sums one wavefront's column groups
#pragma unroll
    for (int f = 0; f < Dim; ++f) {
      constexpr int R = sizeof(T) == 8 ? 1 : 4;  // registers a tile of entries
      lds_barrier();
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          T* const to = lds + (v * R + r) * S::kThreads + tl.tid;
          if constexpr (R == 1) *in_lds(to) = acc[f].v[v >> 1][v & 1];
          else *in_lds(to) = acc[f].v[v >> 1][v & 1][r];
        }
      lds_barrier();
      const int w = tl.tid % kWaves, e = tl.tid / kWaves, tile = e >> 4, i = e >> 2 & 3, j = e & 3;
      const T* const from = lds + (R == 1 ? tile * S::kThreads + 16 * i : (4 * tile + i) * S::kThreads) + 64 * w + j;
      T sum = 0;
#pragma unroll
      for (int b = 0; b < 4 * R; ++b) sum += in_lds(from)[4 * b];
#pragma unroll
      for (int h = 1; h < kWaves; h <<= 1) sum += __shfl_xor(sum, h);
      const int row = 2 * i + (tile >> 1), col = 2 * j + (tile & 1);
      if (w == 0) ws[((int64_t)block * 3 + f) * 256 + row * 16 + col] = sum;
    }
  } else {
    // the wavefronts' partials, summed in wavefront order through LDS
    lds_barrier();
    const int g = lane >> 4, L = lane & 15;
#pragma unroll
    for (int f = 0; f < Dim; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        in_lds(lds)[(tl.wave * Dim + f) * 256 + (sizeof(T) == 8 ? g + 4 * r : 4 * g + r) * 16 + L] = acc[f][r];
    lds_barrier();
    for (int e = tl.tid; e < Dim * 256; e += S::kThreads) {
      T sum = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sum += in_lds(lds)[w * Dim * 256 + e];
      ws[(int64_t)block * 3 * 256 + e] = sum;
    }
  }
}

template <class S>
__global__ __launch_bounds__(S::kThreads) __attribute__((amdgpu_waves_per_eu(S::kMinWaves))) void kron_backward_kernel(
    const typename S::io_t* A, const typename S::io_t* B, const typename S::io_t* C, const typename S::io_t* X,
    const typename S::io_t* dY, typename S::io_t* dX, typename S::io_t* ws, int64_t batch, int which) {
  __shared__ __attribute__((aligned(16))) typename S::io_t lds[backward_lds<S>()];
  backward_block<S>(lds, A, B, C, X, dY, dX, ws, batch, which, blockIdx.x, gridDim.x);
}

// The groups of one launch, in its kernel arguments (so that a captured launch
// keeps them).  A group's workgroups are consecutive, from `first` on.
constexpr int kBwdGroups = 32;
struct BwdGroup {
  const void *A, *B, *C, *X, *dY;
  void *dX, *ws, *out[3];
  int64_t batch;
  int n, which;
  unsigned first, blocks;  // of the tile kernel
  unsigned row, rows;      // of the sum kernel
};
template <int K>
struct BwdTable {
  int count, pad;
  BwdGroup g[K];
};
static_assert(sizeof(BwdTable<kBwdGroups>) <= 4096 - 256, "kernel arguments");
typedef const __attribute__((address_space(4))) BwdTable<kBwdGroups>* bwd_table_t;

// Sizes that share a launch: those that keep as many wavefronts on a SIMD and
// need about the same LDS, because the launch's registers and LDS are the
// largest of its sizes.
constexpr int kBwdClasses = 3;
template <typename T, int Dim>
constexpr int bwd_class(int n) {
  if (sizeof(T) == 8) return n <= 8 ? 0 : n <= 12 ? 1 : 2;
  if (Dim == 3) return n <= 8 ? 0 : n <= 12 ? 1 : 2;
  return n <= 8 ? 0 : n <= 11 || n == 16 ? 1 : 2;
}
template <typename T, int Dim, int kClass>
struct BwdClass {
  int lds = 0, threads = 0, per_simd = 8;
  constexpr BwdClass() { add(std::make_integer_sequence<int, KRON_MAX_N>{}); }
  template <int... i>
  constexpr void add(std::integer_sequence<int, i...>) {
    (one<i + 1>(), ...);
  }
  template <int N>
  constexpr void one() {
    if (bwd_class<T, Dim>(N) != kClass) return;
    using S = Bwd<T, Dim, N>;
    if (backward_lds<S>() > lds) lds = backward_lds<S>();
    if (S::kThreads > threads) threads = S::kThreads;
    if (S::kMinWaves < per_simd) per_simd = S::kMinWaves;
  }
};

// One launch over groups of one type, dimension and class.  Every group gets
// the workgroups, tiles and sums of its own launch, hence its results.  30
// groups (n = 2 .. 16, 2-D and 3-D, 500,000 operands, 2.1 GB): 740 us, on eight
// streams with a launch and a sum each 878; 2,000 operands 137 us, then 442.
template <typename T, int Dim, int kClass>
__global__ __launch_bounds__((BwdClass<T, Dim, kClass>().threads))
    __attribute__((amdgpu_waves_per_eu(BwdClass<T, Dim, kClass>().per_simd))) void kron_backward_grouped_kernel(
        BwdTable<kBwdGroups>) {
  __shared__ __attribute__((aligned(16))) T lds[BwdClass<T, Dim, kClass>().lds];
  // the table in place: a by-value copy indexed at run time would go to scratch
  const bwd_table_t tab = (bwd_table_t)__builtin_amdgcn_kernarg_segment_ptr();
  int g = 0;
  while (g + 1 < tab->count && blockIdx.x >= tab->g[g + 1].first) ++g;
  const auto* d = &tab->g[g];
  const int n = d->n;
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if constexpr (bwd_class<T, Dim>(N) == kClass) {
      using S = Bwd<T, Dim, N>;
      if (n != N || threadIdx.x >= S::kThreads) return;
      backward_block<S>(lds, (const T*)d->A, (const T*)d->B, (const T*)d->C, (const T*)d->X, (const T*)d->dY,
                        (T*)d->dX, (T*)d->ws, d->batch, d->which, blockIdx.x - d->first, d->blocks);
    }
  });
}

// dM(i, j) = sum of entry (i, j) over the partial tiles, in a fixed order in
// FP64: one workgroup per row i of each factor, so that a partial is read in
// whole rows of 16; 64 lanes share an entry, lane p sums partials p, p + 64, ..
// and a fixed-shape tree finishes.  Column-major (i + n*j).
template <typename T, int K>
__global__ __launch_bounds__(1024) void kron_backward_sum_kernel(BwdTable<K>) {
  const bwd_table_t tab = (bwd_table_t)__builtin_amdgcn_kernarg_segment_ptr();
  int g = 0;
  while (g + 1 < tab->count && blockIdx.x >= tab->g[g + 1].row) ++g;
  const auto* d = &tab->g[g];
  const int n = d->n, row = blockIdx.x - d->row, f = row / n, i = row % n;
  T* const out = (T*)d->out[f];
  if (out == nullptr) return;
  const int j = threadIdx.x & 15, p = threadIdx.x >> 4;
  const T* const ws = (const T*)d->ws + f * 256 + i * 16 + j;
  const int64_t nparts = d->blocks;
  double s = 0.0;
  if (j < n) {
#pragma unroll 8
    for (int64_t w = p; w < nparts; w += 64) s += (double)in_global(ws)[w * 768];
  }
  __shared__ double red[1024];
  red[threadIdx.x] = s;
  __syncthreads();
#pragma unroll
  for (int h = 512; h >= 16; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x < (unsigned)n) out[i + n * threadIdx.x] = (T)red[threadIdx.x];
}

}  // namespace kron
