// Launch of the backward kernels (FP32 and FP64).
#include <algorithm>
#include <utility>
#include <vector>

#include "kron.h"
#include "kron_backward.hpp"
#include "kron_launch.hpp"

namespace kron {

// Workgroups a call may have, each with one partial sum of every gradient in the
// workspace: a fixed function of the batch and the device.  One for (16 / n)^dim
// operands and a multiple of four, at most eight a CU; at n <= 4 that is fewer
// than there are tiles in a small batch (3-D n = 2, 1 MiB of X: 64 for 512).
int64_t grad_partials(int dim, int n, int64_t batch) {
  const int64_t q = 16 / n;
  const int64_t ops = dim == 3 ? q * q * q : q * q;
  const int64_t ntiles = (batch + ops - 1) / ops;
  const int64_t cap = (int64_t)device_cus() * 8;
  int64_t w = ntiles < cap ? ntiles : cap;
  w = (w + 3) / 4 * 4;
  return w < 4 ? 4 : w;
}

size_t grad_workspace_bytes(int dim, int n, int64_t batch, int elem_bytes) {
  return (size_t)grad_partials(dim, n, batch) * 3 * 256 * (size_t)elem_bytes;
}

namespace {

// Workgroups of a group's tiles.  A fixed function of the batch and the
// device, so the summation order (and the result) is the same on every call.
template <typename T, int Dim, int N>
unsigned backward_blocks(int64_t batch) {
  using S = Bwd<T, Dim, N>;
  const int64_t tiles = (batch + S::P - 1) / S::P;
  const int64_t cap = std::min((int64_t)device_cus() * occupancy_blocks(kron_backward_kernel<S>, S::kThreads),
                               grad_partials(Dim, N, batch));
  return (unsigned)std::min(tiles, cap);
}

template <typename T>
BwdGroup group_of(const kron_group_grad_t& d, void* ws) {
  BwdGroup g{};
  g.A = d.A, g.B = d.B, g.C = d.C, g.X = d.X, g.dY = d.dY, g.dX = d.dX, g.ws = ws;
  g.out[0] = d.dA, g.out[1] = d.dB, g.out[2] = d.dim == 3 ? d.dC : nullptr;
  for (int f = 0; f < 3; ++f) g.which |= g.out[f] ? 1 << f : 0;
  g.batch = d.count;
  g.n = d.n;
  g.rows = (unsigned)(d.dim * d.n);
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if (d.n == N) g.blocks = d.dim == 2 ? backward_blocks<T, 2, N>(d.count) : backward_blocks<T, 3, N>(d.count);
  });
  return g;
}

template <typename T, int K>
void launch_sum(BwdTable<K>& tab, hipStream_t stream) {
  unsigned rows = 0;
  for (int i = 0; i < tab.count; ++i) {
    tab.g[i].row = rows;
    rows += tab.g[i].rows;
  }
  hipLaunchKernelGGL((kron_backward_sum_kernel<T, K>), dim3(rows), dim3(1024), 0, stream, tab);
}

template <typename T, int Dim, int kClass>
void launch_class(const BwdTable<kBwdGroups>& tab, unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL((kron_backward_grouped_kernel<T, Dim, kClass>), dim3(blocks),
                     dim3(BwdClass<T, Dim, kClass>().threads), 0, stream, tab);
}

template <typename T>
int run_one(const BwdGroup& g, int dim, hipStream_t stream) {
  static_for<KRON_MAX_N>([&](auto i) {
    constexpr int N = decltype(i)::value + 1;
    if (g.n != N || g.blocks == 0) return;
    auto go = [&](auto k, int threads) {
      hipLaunchKernelGGL(k, dim3(g.blocks), dim3(threads), 0, stream, (const T*)g.A, (const T*)g.B, (const T*)g.C,
                         (const T*)g.X, (const T*)g.dY, (T*)g.dX, (T*)g.ws, g.batch, g.which);
    };
    if (dim == 2) go(kron_backward_kernel<Bwd<T, 2, N>>, Bwd<T, 2, N>::kThreads);
    else go(kron_backward_kernel<Bwd<T, 3, N>>, Bwd<T, 3, N>::kThreads);
  });
  BwdTable<1> tab;
  tab.count = 1;
  tab.g[0] = g;
  launch_sum<T>(tab, stream);
  return 0;
}

template <typename T>
void run_groups(std::vector<std::pair<const kron_group_grad_t*, void*>>& groups, hipStream_t stream) {
  // the groups with the longest workgroups first, so that short ones end a launch
  std::vector<BwdGroup> all;
  std::vector<int> dims, order;
  std::vector<double> cost;
  for (auto& [d, ws] : groups) {
    all.push_back(group_of<T>(*d, ws));
    dims.push_back(d->dim);
    order.push_back((int)order.size());
    double e = (double)d->count / std::max(1u, all.back().blocks);
    for (int k = 0; k < d->dim; ++k) e *= d->n;
    cost.push_back(e);
  }
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
  for (int dim = 3; dim >= 2; --dim)
    static_for<kBwdClasses>([&](auto c) {
      constexpr int kClass = kBwdClasses - 1 - decltype(c)::value;
      BwdTable<kBwdGroups> tab;
      tab.count = 0;
      unsigned blocks = 0;
      auto flush = [&] {
        if (tab.count == 0) return;
        if (dim == 2) launch_class<T, 2, kClass>(tab, blocks, stream);
        else launch_class<T, 3, kClass>(tab, blocks, stream);
        tab.count = 0;
        blocks = 0;
      };
      for (int i : order) {
        if (dims[i] != dim || all[i].blocks == 0) continue;
        if ((dim == 2 ? bwd_class<T, 2>(all[i].n) : bwd_class<T, 3>(all[i].n)) != kClass) continue;
        tab.g[tab.count] = all[i];
        tab.g[tab.count++].first = blocks;
        blocks += all[i].blocks;
        if (tab.count == kBwdGroups) flush();
      }
      flush();
    });
  for (size_t at = 0; at < all.size(); at += kBwdGroups) {
    BwdTable<kBwdGroups> tab;
    tab.count = (int)std::min(all.size() - at, (size_t)kBwdGroups);
    std::copy_n(all.begin() + at, tab.count, tab.g);
    launch_sum<T>(tab, stream);
  }
}

}  // namespace

int backward(const kron_group_grad_t& d, void* ws, hipStream_t stream) {
  return d.mode == KRON_MODE_F32 ? run_one<float>(group_of<float>(d, ws), d.dim, stream)
                                 : run_one<double>(group_of<double>(d, ws), d.dim, stream);
}

void backward_grouped(const std::vector<std::pair<const kron_group_grad_t*, void*>>& groups, hipStream_t stream) {
  for (int mode : {KRON_MODE_F32, KRON_MODE_F64}) {
    std::vector<std::pair<const kron_group_grad_t*, void*>> mine;
    for (auto& g : groups)
      if (g.first->mode == mode) mine.push_back(g);
    if (mine.empty()) continue;
    if (mode == KRON_MODE_F32) run_groups<float>(mine, stream);
    else run_groups<double>(mine, stream);
  }
}

}  // namespace kron
