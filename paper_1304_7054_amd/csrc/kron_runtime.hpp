// Host runtime shared by the translation units of libkron: device facts,
// launch tuning table and the per-mode launch entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>
#include <vector>

struct kron_group;

namespace kron {

// Compute units of the current device (cached per device ordinal).
int device_cus();

// Launch shape for (mode, dim, n): workgroups per CU (0 = as many as are
// resident at once) and kernel variant; (-1, 0) = the column kernels.  Defaults come from a table measured
// on MI355X; kron_set_launch / kron_autotune replace them.
struct LaunchShape {
  int blocks_per_cu;
  int variant;
};
LaunchShape launch_shape(int mode, int dim, int n);
int set_launch_shape(int mode, int dim, int n, int blocks_per_cu, int variant);

// Forward launches of each precision mode, defined in kron_<mode>.hip.
// Return 0, or -1 for an n outside 1..16.
int fwd2d_f32(int n, const float* A, const float* B, const float* X, float* Y, int64_t batch, hipStream_t s,
              bool trans);
int fwd3d_f32(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
              hipStream_t s, bool trans);
int fwd2d_f64(int n, const double* A, const double* B, const double* X, double* Y, int64_t batch, hipStream_t s,
              bool trans);
int fwd3d_f64(int n, const double* A, const double* B, const double* C, const double* X, double* Y,
              int64_t batch, hipStream_t s, bool trans);
int fwd2d_bf16x3(int n, const float* A, const float* B, const float* X, float* Y, int64_t batch, hipStream_t s);
int fwd3d_bf16x3(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                 hipStream_t s);
int fwd2d_bf16x6(int n, const float* A, const float* B, const float* X, float* Y, int64_t batch, hipStream_t s);
int fwd3d_bf16x6(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                 hipStream_t s);
int fwd2d_bf16(int n, const uint16_t* A, const uint16_t* B, const uint16_t* X, uint16_t* Y, int64_t batch,
               hipStream_t s);
int fwd3d_bf16(int n, const uint16_t* A, const uint16_t* B, const uint16_t* C, const uint16_t* X, uint16_t* Y,
               int64_t batch, hipStream_t s);

// 3-D launches split by n range (kron_<mode>_3d_lo/hi.hip).
int fwd3d_f32_lo(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                hipStream_t s, bool trans);
int fwd3d_f32_hi(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                hipStream_t s, bool trans);
int fwd3d_f64_lo(int n, const double* A, const double* B, const double* C, const double* X, double* Y, int64_t batch,
                hipStream_t s, bool trans);
int fwd3d_f64_hi(int n, const double* A, const double* B, const double* C, const double* X, double* Y, int64_t batch,
                hipStream_t s, bool trans);
int fwd3d_bf16x3_lo(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                hipStream_t s);
int fwd3d_bf16x3_hi(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                hipStream_t s);
int fwd3d_bf16x6_lo(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                hipStream_t s);
int fwd3d_bf16x6_hi(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
                hipStream_t s);
int fwd3d_bf16_lo(int n, const uint16_t* A, const uint16_t* B, const uint16_t* C, const uint16_t* X, uint16_t* Y, int64_t batch,
                hipStream_t s);
int fwd3d_bf16_hi(int n, const uint16_t* A, const uint16_t* B, const uint16_t* C, const uint16_t* X, uint16_t* Y, int64_t batch,
                hipStream_t s);

// 3-D column kernels (kron_cols.hip) of the modes and sizes that have one.
// cols3d returns 0, or -1 without one.
bool has_cols3d(int mode, int n);
int cols3d(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
           hipStream_t s, bool trans);
int cols3d(int n, const double* A, const double* B, const double* C, const double* X, double* Y, int64_t batch,
           hipStream_t s, bool trans);
int cols3d(int n, const uint16_t* A, const uint16_t* B, const uint16_t* C, const uint16_t* X, uint16_t* Y,
           int64_t batch, hipStream_t s, bool trans);

// Y <- K(op(X)) + beta Y (kron_ex_<mode>.hip) for beta != 0 or, in 2-D,
// transposed operands (transx); alpha and op on the factors are already in
// the factors.  Return 0, -1 for an n outside 1..16, or -2 when beta == 0
// and !transx (the plain kernels cover that case).
int ex2d_f32(int n, const float* A, const float* B, const float* X, float* Y, int64_t batch, float beta, bool transx,
             hipStream_t s);
int ex3d_f32(int n, const float* A, const float* B, const float* C, const float* X, float* Y, int64_t batch,
             float beta, hipStream_t s);
int ex2d_f64(int n, const double* A, const double* B, const double* X, double* Y, int64_t batch, double beta,
             bool transx, hipStream_t s);
int ex3d_f64(int n, const double* A, const double* B, const double* C, const double* X, double* Y, int64_t batch,
             double beta, hipStream_t s);

// alpha op(F_0), op(F_1)[, op(F_2)] (leading dimensions ld, transposed where
// tmask has the factor's bit) written dense to out, n^2 elements each.
void prepare_factors(int n, int nf, const float* const* F, const int* ld, unsigned tmask, float alpha, float* out,
                     hipStream_t stream);
void prepare_factors(int n, int nf, const double* const* F, const int* ld, unsigned tmask, double alpha, double* out,
                     hipStream_t stream);

// Grouped launch (kron_grouped.hip).
size_t grouped_workspace_bytes(const struct kron_group* g, int ngroups);
int grouped_prepare(const struct kron_group* g, int ngroups, void* ws, size_t ws_bytes, hipStream_t stream);
int grouped_launch(const void* ws, hipStream_t stream);

// The backward with at least one factor gradient (kron_backward.hip): dX (may
// be null) and the factor gradients (null ones are skipped; dC only in 3-D) in
// one pass over X and dY.  ws holds grad_workspace_bytes().
int64_t grad_partials(int dim, int n, int64_t batch);
size_t grad_workspace_bytes(int dim, int n, int64_t batch, int elem_bytes);
int backward(const struct kron_group_grad& d, void* ws, hipStream_t stream);
// The same for each of several groups (descriptor, workspace), in few launches.
void backward_grouped(const std::vector<std::pair<const struct kron_group_grad*, void*>>& groups, hipStream_t stream);

}  // namespace kron
