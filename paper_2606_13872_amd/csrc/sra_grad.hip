// The matrix kernels of the SRA backward on gfx950: dK/dV (sra_dkv.h) and dQ (sra_dq.h), and the sums
// of split items. Their work items do not depend on one another, so a launch of few items runs both
// kinds together (sra_grad_kernel): one launch less, and the one kind fills the compute units that
// the other's last round leaves idle. A long launch runs the two kernels one after the other: each
// kind's items are then ordered so that those resident on an XCD share rows through its L2, and a
// last round is worth little. One launch and split items: 480p, 5 heads 11.8 -> 10.7 ms; 8 heads of
// 1,280 + 1,024 tokens, d = 64, 111 -> 47 us.
#include "sra_dkv.h"
#include "sra_dq.h"

namespace sra {

template <int D, bool kOneStride>
__global__ void __launch_bounds__(kDkvWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1)))
sra_dkv_kernel(BwdArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[DkvLds<D>::kBytes];
  const WorkItem it = a.items[blockIdx.x];
  if (it.stream < 0) return;
  dkv_item<D, kOneStride>(a, it, lds);
}

template <int D, bool kOneStride>
__global__ void __launch_bounds__(kDqWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1)))
sra_dq_kernel(BwdArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kDqLdsBytes<D>];
  const WorkItem it = a.items[blockIdx.x];
  if (it.stream < 0) return;
  dq_item<D, kOneStride>(a, it, lds);
}

// Both kinds: bit 1 of an item's stream marks a dQ item.
template <int D, bool kOneStride>
__global__ void __launch_bounds__(kDkvWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1)))
sra_grad_kernel(BwdArgs a) {
  static_assert(kDkvWaves == kDqWaves, "one block size");
  constexpr uint32_t kBytes = DkvLds<D>::kBytes > kDqLdsBytes<D> ? DkvLds<D>::kBytes : kDqLdsBytes<D>;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kBytes];
  const WorkItem it = a.items[blockIdx.x];
  if (it.stream < 0) return;
  if (it.stream & 2) dq_item<D, kOneStride>(a, it, lds);
  else dkv_item<D, kOneStride>(a, it, lds);
}

// Sums of the split items' pieces, in piece order: items [0, n_kv) dK and dV, the others dQ.
// D / 4 threads per row. Bound by reading the partial sums; a few microseconds behind a launch that ends
// earlier by more (the scheduler's replay).
template <int D>
__global__ void __launch_bounds__(kThreads) sra_grad_combine_kernel(BwdArgs a, const CombineItem* items, int n_kv) {
  constexpr int TPR = D / 4, RPB = kThreads / TPR;
  const CombineItem it = items[blockIdx.x];
  const int r = blockIdx.y * RPB + threadIdx.x / TPR, sub = threadIdx.x % TPR;
  if (r >= it.len) return;
  const bool kv = int(blockIdx.x) < n_kv;
  const int64_t out = (int64_t(it.start + r) * a.heads + it.head) * D + 4 * sub;
  auto sum = [&](const float* p, int64_t slot, float scale, __bf16* dst) {
    floatx4 x = *reinterpret_cast<const floatx4*>(p);
    for (int i = 1; i < it.n; ++i) x += *reinterpret_cast<const floatx4*>(p + i * slot);
    bf16x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = (__bf16)(x[e] * scale);
    *reinterpret_cast<bf16x4*>(dst + out) = y;
  };
  if (kv) {
    constexpr int64_t slot = int64_t(2) * kDkvKeyTile * D;
    const float* p = a.part_kv + it.slot0 * slot + r * D + 4 * sub;
    sum(p, slot, a.scale, a.dk[it.stream]);
    sum(p + kDkvKeyTile * D, slot, 1.f, a.dv[it.stream]);
  } else {
    constexpr int64_t slot = int64_t(kDqQueryTile) * D;
    sum(a.part_q + it.slot0 * slot + r * D + 4 * sub, slot, a.scale, a.dq[it.stream]);
  }
}

template <int D, bool kOneStride>
static void launch_kind(GradKind kind, const BwdArgs& a, int n_items, hipStream_t stream) {
  const dim3 grid(n_items), block(kDkvWaves * 64);
  if (kind == GradKind::kDkv) hipLaunchKernelGGL((sra_dkv_kernel<D, kOneStride>), grid, block, 0, stream, a);
  else if (kind == GradKind::kDq) hipLaunchKernelGGL((sra_dq_kernel<D, kOneStride>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((sra_grad_kernel<D, kOneStride>), grid, block, 0, stream, a);
}

hipError_t launch_grad(GradKind kind, const BwdArgs& a, int n_items, int head_dim, hipStream_t stream) {
  if (n_items <= 0) return hipSuccess;
  const bool one = a.in_stride[0] == a.in_stride[1];
  if (head_dim == 128) {
    if (one) launch_kind<128, true>(kind, a, n_items, stream);
    else launch_kind<128, false>(kind, a, n_items, stream);
  } else {
    if (one) launch_kind<64, true>(kind, a, n_items, stream);
    else launch_kind<64, false>(kind, a, n_items, stream);
  }
  return hipGetLastError();
}

hipError_t launch_grad_combine(const BwdArgs& a, const CombineItem* items, int n_kv, int n, int head_dim,
                               hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  static_assert(kDkvKeyTile == kDqQueryTile, "one grid for both kinds");
  const dim3 grid(n, kDqQueryTile * (head_dim / 4) / kThreads);
  if (head_dim == 128)
    hipLaunchKernelGGL(sra_grad_combine_kernel<128>, grid, dim3(kThreads), 0, stream, a, items, n_kv);
  else
    hipLaunchKernelGGL(sra_grad_combine_kernel<64>, grid, dim3(kThreads), 0, stream, a, items, n_kv);
  return hipGetLastError();
}

}  // namespace sra
