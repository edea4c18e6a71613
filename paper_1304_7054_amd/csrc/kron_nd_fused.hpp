// Several mode products of the general action in one kernel.
//
// A workgroup holds P whole operands (or, when an operand is too large, P
// slices of the fastest indices) in LDS and applies the factors one after the
// other, in place where the factor is square (a wavefront has read its columns
// before it writes them) and between two LDS images otherwise, so that memory sees the operands once in and
// once out instead of once each way per dimension.  Sizes are runtime values:
// any extents whose images and factors fit (nd_fuse in kron_nd.hip).
//
// Every product is tiles of 16 output rows by 16 columns on the 16x16x4
// matrix instruction.  A column is one fibre along the contracted index, with
// all other indices of all P operands flattened, so columns are never padded;
// lane (L, g) reads elements 4s + g of column L.  Rows of the fastest index
// sit at a pitch that lets 16 columns be read side by side without meeting an
// LDS bank twice.  The factors are laid out in LDS as the fragments that the
// instruction takes: once, or, with factors per operand, those of every operand
// of the tile, whose blocks of columns then hold one operand's only.
#pragma once

#include "kron_cols.hpp"

namespace kron {

// q = x / d for x < 2^31, by multiplication with a rounded-up reciprocal
// (Granlund and Montgomery, Division by invariant integers, 1994, figure 4.1).
struct FastDiv {
  uint32_t d, m, s;
  __device__ __forceinline__ uint32_t div(uint32_t x) const { return (__umulhi(x, m) + x) >> s; }
};
inline FastDiv fast_div(uint32_t d) {
  uint32_t s = 0;
  while (s < 31 && (1u << s) < d) ++s;
  const uint64_t m = ((((uint64_t)1 << s) - d) << 32) / d + 1;
  return FastDiv{d, (uint32_t)m, s};
}

constexpr int kFuseMax = 8;

// Whose factors a tile has: the batch's, each operand's own, or those of the one
// operand that it is, or has slices of.
enum FusedFactors { kFusedShared, kFusedOwn, kFusedOne };

// One product: columns c = (u, w) with w < post; element k of a column is at
// u * in_u + where(w) + k * in_s, where(w) = (w / fast) * pitch + w % fast.
struct FusedStage {
  int n, m, ks, rb;       // contracted and produced extent; steps of 4, blocks of 16
  int cols;               // columns per operand
  int in_u, in_s, out_u, out_s, pitch;
  int in, out;            // LDS offsets of the images (the same one when m == n)
  FastDiv post, fast;
  FastDiv frags, steps;   // fragments of the factor: rb * ks, and ks
  int fac;                // LDS offset of the factor's fragments
  int tab;                // first entry of the tile's columns in the offset table
  const void* F;
  int64_t ldfp;           // elements between operands' factors (0: shared)
  int ld, op;             // as in NdPass
};

// Operand storage: dense (stride[0] < 0), or an element stride per index
// (fastest first) and between operands, up to three indices.
struct FusedArray {
  int64_t stride[3], sp;
  int elems, pitch;       // elements per operand; pitch of its rows in LDS
  FastDiv ext[3];         // extents, fastest first
};

struct FusedArgs {
  const void* X;
  void* Y;
  int nstage, ops;        // products; operands per tile
  int64_t batch, ntiles;
  int64_t per;            // slices per operand (the operand of slice i is i / per)
  int img_x, img_y;       // LDS offsets of the first and the last image
  int table;              // bytes before the offset table (-1: no room for one)
  int per_operand;        // factors change with the operand: a tile's slices are of one, or its operands whole
  int facs;               // LDS elements of one operand's fragments
  int conjx;
  FusedArray x, y;
  FusedStage st[kFuseMax];
};

template <typename T, bool kC>
struct FusedElem {
  using type = T;
};
template <typename T>
struct FusedElem<T, true> {
  typedef T type __attribute__((ext_vector_type(2)));
};

// Global offset of element e of the tile's operands (e = operand * elems + index).
__device__ __forceinline__ int64_t fused_offset(const FusedArray& a, FastDiv elems, uint32_t e) {
  if (a.stride[0] < 0) return e;
  const uint32_t p = elems.div(e);
  uint32_t i = e - p * elems.d;
  int64_t off = (int64_t)p * a.sp;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const uint32_t q = j < 2 ? a.ext[j].div(i) : 0;
    off += (int64_t)(j < 2 ? i - q * a.ext[j].d : i) * a.stride[j];
    i = q;
  }
  return off;
}

// Where column c starts in a product's images: input low, output high.
__device__ __forceinline__ uint32_t fused_column(const FusedStage& st, uint32_t c) {
  const uint32_t u = st.post.div(c), w = c - u * st.post.d, wr = st.fast.div(w);
  const uint32_t wo = wr * st.pitch + (w - wr * st.fast.d);
  return (u * st.in_u + wo) | (u * st.out_u + wo) << 16;
}

// One product of a tile by one wavefront of four: kCB blocks of 16 columns at a
// time, their kKS steps of four elements in registers (st.ks == kKS).  kVar:
// `sets` operands have factors of their own, facs elements apart, and ncols
// columns each; else all ncols columns of the tile share one.
template <typename T, bool kC, int kKS, int kCB, bool kVar>
__device__ __forceinline__ void fused_stage(const FusedStage& st, typename FusedElem<T, kC>::type* base,
                                            const uint32_t* tab, int sets, int ncols, int facs, int wave, int lane) {
  using elem_t = typename FusedElem<T, kC>::type;
  using acc_t = std::conditional_t<sizeof(T) == 8, f64x4, f32x4>;
  auto mma = [](T a, T b, acc_t c) {
    if constexpr (sizeof(T) == 8) return mfma_f64(a, b, c);
    else return mfma_f32(a, b, c);
  };
  const int L = lane & 15, g = lane >> 4;
  const elem_t* in = base + st.in;
  elem_t* out = base + st.out;
  const int in_s = st.in_s, out_s = st.out_s;
  const bool last_in = 4 * (kKS - 1) + g < st.n;  // whether the last step's element exists
  const elem_t* fac = base + st.fac + lane;
  int first = 0;  // the set's first column
  for (int c0 = 16 * kCB * wave;; c0 += 16 * kCB * 4) {
    if constexpr (kVar) {
      while (c0 >= ncols && sets > 0) {
        c0 -= (ncols + 16 * kCB - 1) / (16 * kCB) * (16 * kCB);
        first += ncols;
        fac += facs;
        --sets;
      }
      if (sets == 0) break;
    } else {
      if (c0 >= ncols) break;
    }
    T x[kCB][kKS], xi[kC ? kCB : 1][kC ? kKS : 1];
    elem_t* dst[kCB];
    bool ok[kCB];
#pragma unroll
    for (int b = 0; b < kCB; ++b) {
      // lanes past the last column read it again and write nothing
      const int cw = c0 + 16 * b + L;
      ok[b] = cw < ncols;
      const uint32_t c = (ok[b] ? cw : ncols - 1) + first;
      const uint32_t at = tab ? in_lds(tab)[st.tab + c] : fused_column(st, c);
      const elem_t* top = in + (at & 0xffff);
      const elem_t* col = top + g * in_s;
      // where the last step's element does not exist, the column's first one in
      // its place: beyond the last column the image ends
      const elem_t* tail = last_in ? col + 4 * (kKS - 1) * in_s : top;
      dst[b] = out + (at >> 16) + (sizeof(T) == 8 ? g : 4 * g) * out_s;
#pragma unroll
      for (int s = 0; s < kKS; ++s) {
        const elem_t v = s + 1 < kKS ? in_lds(col)[4 * s * in_s] : *in_lds(tail);
        if constexpr (kC) {
          x[b][s] = v[0];
          xi[b][s] = v[1];
        } else {
          x[b][s] = v;
        }
      }
      x[b][kKS - 1] = last_in ? x[b][kKS - 1] : T(0);
      if constexpr (kC) xi[b][kKS - 1] = last_in ? xi[b][kKS - 1] : T(0);
    }
    for (int rb = 0; rb < st.rb; ++rb) {
      acc_t dr[kCB], di[kC ? kCB : 1];
#pragma unroll
      for (int b = 0; b < kCB; ++b) {
        dr[b] = acc_t{0, 0, 0, 0};
        if constexpr (kC) di[b] = acc_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int s = 0; s < kKS; ++s) {
        const elem_t f = in_lds(fac)[(rb * kKS + s) * 64];
#pragma unroll
        for (int b = 0; b < kCB; ++b) {
          if constexpr (kC) {
            dr[b] = mma(f[0], x[b][s], dr[b]);
            dr[b] = mma(-f[1], xi[b][s], dr[b]);
            di[b] = mma(f[0], xi[b][s], di[b]);
            di[b] = mma(f[1], x[b][s], di[b]);
          } else {
            dr[b] = mma(f, x[b][s], dr[b]);
          }
        }
      }
      const int rows = st.m - 16 * rb;  // rows left, this block's first being row 0
#pragma unroll
      for (int b = 0; b < kCB; ++b)
        if (ok[b]) {
          elem_t* o = dst[b] + 16 * rb * out_s;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int step = sizeof(T) == 8 ? 4 * r : r;
            if (rows >= 16 || (sizeof(T) == 8 ? g : 4 * g) + step < rows) {
              if constexpr (kC) in_lds(o)[step * out_s] = elem_t{dr[b][r], di[b][r]};
              else in_lds(o)[step * out_s] = dr[b][r];
            }
          }
        }
    }
  }
}

// Wavefronts per SIMD the registers are held to, by measurement (256 MiB and
// more of operands; two fewer or more cost 5 to 30 %).  kKS: the largest
// product's steps of four contracted indices.
template <typename T, bool kC, int kKS>
constexpr int fused_waves() {
  if (kKS > 8) return 2;
  if (kC) return kKS > 4 ? 3 : sizeof(T) == 8 ? 5 : 4;
  return sizeof(T) == 4 ? 5 : kKS <= 4 ? 4 : 3;
}

template <typename T, bool kC, int kKS, int kCB, bool kBeta, int kVar>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(fused_waves<T, kC, kKS>()))) void kron_nd_fused_kernel(
    FusedArgs P, FastDiv xe, FastDiv ye, T ar, T ai, T br, T bi) {
  using elem_t = typename FusedElem<T, kC>::type;
  constexpr int kS = kC ? 2 : 1;
  constexpr int V = 16 / (int)sizeof(elem_t);  // elements of a 16-byte vector
  typedef T vec_t __attribute__((ext_vector_type(16 / sizeof(T))));
  extern __shared__ __attribute__((aligned(16))) unsigned char fused_lds[];
  elem_t* const base = reinterpret_cast<elem_t*>(fused_lds);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the fragments of every factor of `count` operands: (row block, step) by lane
  auto load_factors = [&](int64_t operand, int count) {
    for (int q = 0; q < P.nstage; ++q) {
      const FusedStage st = P.st[q];
      const T* F = static_cast<const T*>(st.F) + operand * st.ldfp * kS;
      for (int e = tid; e < count * (int)st.frags.d * 64; e += 256) {
        const uint32_t f = e >> 6, op = kVar == kFusedOwn ? st.frags.div(f) : 0, h = f - op * st.frags.d, rb = st.steps.div(h);
        const int i = 16 * rb + (e & 15), k = 4 * (h - rb * st.steps.d) + ((e >> 4) & 3);
        T re = 0, im = 0;
        if (i < st.m && k < st.n) {
          const int64_t o = (st.op == 0 ? i + (int64_t)st.ld * k : k + (int64_t)st.ld * i) + op * st.ldfp;
          re = in_global(F)[kS * o];
          if constexpr (kC) im = st.op == 2 ? -in_global(F)[kS * o + 1] : in_global(F)[kS * o + 1];
        }
        const int to = st.fac + (int)(op * P.facs + h * 64) + lane;
        if constexpr (kC) in_lds(base)[to] = elem_t{re, im};
        else in_lds(base)[to] = re;
      }
    }
  };
  if constexpr (kVar == kFusedShared) load_factors(0, 1);
  // where each column of a full tile starts in the images, for every product
  uint32_t* const tab = P.table < 0 ? nullptr : reinterpret_cast<uint32_t*>(fused_lds + P.table);
  if (tab) {
    for (int q = 0; q < P.nstage; ++q) {
      const FusedStage st = P.st[q];
      for (int c = tid; c < P.ops * st.cols; c += 256) in_lds(tab)[st.tab + c] = fused_column(st, c);
    }
  }
  const bool xvec = P.x.stride[0] < 0 && P.x.ext[0].d % V == 0 && (reinterpret_cast<uintptr_t>(P.X) & 15) == 0;
  const bool yvec = P.y.stride[0] < 0 && P.y.ext[0].d % V == 0 && (reinterpret_cast<uintptr_t>(P.Y) & 15) == 0;
  // a vector of packed operands, from element e on, into the first image
  auto place = [&](elem_t* img, uint32_t e, vec_t v) {
    if constexpr (kC) {
      if (P.conjx) {
#pragma unroll
        for (int i = 1; i < 16 / (int)sizeof(T); i += 2) v[i] = -v[i];
      }
    }
    const uint32_t row = P.x.ext[0].div(e);
    *in_lds(reinterpret_cast<vec_t*>(img + row * P.x.pitch + (e - row * P.x.ext[0].d))) = v;
  };
  // a workgroup's tiles; slices of an operand with its own factors one after the
  // other, so that the factors are read once per operand
  int64_t t = blockIdx.x, end = P.ntiles, step = gridDim.x, loaded = -1;
  if (kVar == kFusedOne && P.per > 1) {
    const int64_t share = (P.ntiles + gridDim.x - 1) / gridDim.x;
    t = blockIdx.x * share;
    end = t + share < P.ntiles ? t + share : P.ntiles;
    step = 1;
  }
  for (; t < end; t += step) {
    const int64_t rem = P.batch - t * P.ops;
    const int nops = (int)(rem < P.ops ? rem : P.ops);
    const elem_t* X = static_cast<const elem_t*>(P.X) + t * P.ops * (P.x.stride[0] < 0 ? P.x.elems : P.x.sp);
    elem_t* Y = static_cast<elem_t*>(P.Y) + t * P.ops * (P.y.stride[0] < 0 ? P.y.elems : P.y.sp);
    if constexpr (kVar == kFusedOwn) load_factors(t * P.ops, nops);
    if constexpr (kVar == kFusedOne) {
      const int64_t operand = P.per > 1 ? t * P.ops / P.per : t;
      if (operand != loaded) load_factors(operand, 1);
      loaded = operand;
    }
    {
      elem_t* img = base + P.img_x;
      const int count = nops * P.x.elems;
      if (xvec) {
        for (int v0 = tid; v0 < count / V; v0 += 4 * 256) {
          vec_t r[4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (v0 + 256 * j < count / V) r[j] = __builtin_nontemporal_load(in_global(reinterpret_cast<const vec_t*>(X)) + v0 + 256 * j);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (v0 + 256 * j < count / V) place(img, V * (v0 + 256 * j), r[j]);
        }
      } else {
        for (int e0 = tid; e0 < count; e0 += 4 * 256) {
          elem_t r[4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (e0 + 256 * j < count) r[j] = in_global(X)[fused_offset(P.x, xe, e0 + 256 * j)];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (e0 + 256 * j < count) {
              const uint32_t e = e0 + 256 * j, row = P.x.ext[0].div(e);
              if constexpr (kC) {
                if (P.conjx) r[j][1] = -r[j][1];
              }
              in_lds(img)[row * P.x.pitch + (e - row * P.x.ext[0].d)] = r[j];
            }
        }
      }
    }
    lds_barrier();
    for (int q = 0; q < P.nstage; ++q) {
      const FusedStage st = P.st[q];
      static_for<kKS>([&](auto i) {
        constexpr int kSteps = decltype(i)::value + 1;
        if (st.ks == kSteps) fused_stage<T, kC, kSteps, kSteps <= 8 ? kCB : 1, kVar == kFusedOwn>(
              st, base, tab, nops, kVar == kFusedOwn ? st.cols : nops * st.cols, P.facs, wave, lane);
      });
      lds_barrier();
    }
    const elem_t* img = base + P.img_y;
    const int count = nops * P.y.elems;
    auto scaled = [&](elem_t v, const elem_t* old) {
      if constexpr (kC) {
        elem_t o = elem_t{ar * v[0] - ai * v[1], ar * v[1] + ai * v[0]};
        if constexpr (kBeta) {
          const elem_t y = *in_global(old);
          o[0] += br * y[0] - bi * y[1];
          o[1] += br * y[1] + bi * y[0];
        }
        return o;
      } else {
        elem_t o = ar * v;
        if constexpr (kBeta) o += br * *in_global(old);
        return o;
      }
    };
    if (yvec) {
      for (int v = tid; v < count / V; v += 256) {
        const uint32_t e = V * v, row = P.y.ext[0].div(e);
        const elem_t* src = img + row * P.y.pitch + (e - row * P.y.ext[0].d);
        vec_t o;
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const elem_t z = scaled(in_lds(src)[j], Y + e + j);
          if constexpr (kC) {
            o[2 * j] = z[0];
            o[2 * j + 1] = z[1];
          } else {
            o[j] = z;
          }
        }
        __builtin_nontemporal_store(o, in_global(reinterpret_cast<vec_t*>(Y)) + v);
      }
    } else {
      for (uint32_t e = tid; e < (uint32_t)count; e += 256) {
        const uint32_t row = P.y.ext[0].div(e);
        elem_t* dst = Y + fused_offset(P.y, ye, e);
        *in_global(dst) = scaled(in_lds(img)[row * P.y.pitch + (e - row * P.y.ext[0].d)], dst);
      }
    }
    lds_barrier();  // the images are free for the next tile
  }
}

}  // namespace kron
