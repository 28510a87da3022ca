// Backward attention, dQ kernel (gfx950); the per-workgroup body is in
// bwd_dq.hpp.
#include "bwd_dq.hpp"

namespace fck {

// Head dim 64: -D held in registers leaves two waves per SIMD, without it the
// four-heads tile runs three. It gains on many workgroups (64/16 heads over 64K
// tokens 1163 -> 1110 us, 32/8 over 32K 254 -> 247) and loses on few (32/8 over 16K
// 110 -> 118; D subtracted per score, 122); the other tiles, at or over the
// three-wave limit without it, are faster with -D held (8/8 heads over 32K 109
// against 112 us, 16/8 95 against 97).
template <int D, int HPW>
__global__ __launch_bounds__(256, D == 64 && HPW == 4 ? 3 : 2) void attn_bwd_dq_kernel(DqParams p) {
  __shared__ __attribute__((aligned(16))) char smem[DqLds<D>::bytes];
  dq_tile<D, HPW, D == 64 && HPW != 4>(p, blockIdx.x, smem);
}

template <int D>
static hipError_t launch_dq_d(const DqParams& p, int hpw, hipStream_t s) {
  const dim3 grid(unsigned(p.n_items) * p.hkv * p.head_chunks), block(256);
  switch (hpw) {
    case 1: hipLaunchKernelGGL((attn_bwd_dq_kernel<D, 1>), grid, block, 0, s, p); break;
    case 2: hipLaunchKernelGGL((attn_bwd_dq_kernel<D, 2>), grid, block, 0, s, p); break;
    case 4: hipLaunchKernelGGL((attn_bwd_dq_kernel<D, 4>), grid, block, 0, s, p); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_bwd_dq(const DqParams& p, int d, int heads_per_tile, hipStream_t s) {
  if (p.n_items == 0) return hipSuccess;
  if (d == 64) return launch_dq_d<64>(p, heads_per_tile, s);
  if (d == 128) return launch_dq_d<128>(p, heads_per_tile, s);
  return hipErrorInvalidValue;
}

}  // namespace fck
