// Launches of the dQ pass by itself (bwd_dq.hpp holds the work of a workgroup).
#include "bwd_dq.hpp"

namespace helix {

template <int D, bool CAUSAL, int ROWS>
__global__ void __launch_bounds__(ROWS == 64 ? 256 : 512) __attribute__((amdgpu_waves_per_eu(2)))
bwd_dq_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
              const __bf16* __restrict__ dO, const float* __restrict__ lse2, const float* __restrict__ neg_delta,
              __bf16* __restrict__ dq, BwdMaps maps, int BH, int H, int S, int T, float scale) {
  if constexpr (ROWS == 256) dq_whole_rows<D, CAUSAL>(blockIdx.x, q, k, v, dO, lse2, neg_delta, dq, maps, BH, H, S, T, scale);
  else dq_split_rows<D, CAUSAL, ROWS / 32>(blockIdx.x, q, k, v, dO, lse2, neg_delta, dq, maps, BH, H, S, T, scale);
}

template <int D, bool CAUSAL>
static hipError_t launch_dq_pipe_t(const void* q, const void* k, const void* v, const void* dO,
                                   const float* lse2, const float* neg_delta, void* dq, const BwdMaps& maps,
                                   int B, int H, int S, float scale, hipStream_t stream) {
  const int BH = B * H;
  const Rows rows = dq_rows(gradient_tiles(D, BH, S, CAUSAL));
  const int T = tiles(S, rows);
  const unsigned grid = (unsigned)grid_blocks(BH, T);
  const size_t lds = rows == Rows::k256 ? kDqWholeLds<D> : DqSplit<D>::LDS;
  auto kern = rows == Rows::k64 ? bwd_dq_kernel<D, CAUSAL, 64> : rows == Rows::k128 ? bwd_dq_kernel<D, CAUSAL, 128> : bwd_dq_kernel<D, CAUSAL, 256>;
  static unsigned long long configured[3] = {};   // per template instantiation and kernel
  hipError_t e = allow_dynamic_lds(kern, lds, configured[(int)rows]);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(rows == Rows::k64 ? 256 : 512), lds, stream, (const __bf16*)q, (const __bf16*)k, (const __bf16*)v,
                     (const __bf16*)dO, lse2, neg_delta, (__bf16*)dq, maps, BH, H, S, T, scale);
  return hipGetLastError();
}

hipError_t launch_bwd_dq(const void* q, const void* k, const void* v, const void* dO,
                         const float* lse2, const float* neg_delta, void* dq, const BwdMaps& maps,
                         int B, int H, int S, int D, float scale, bool causal, hipStream_t stream) {
  if (D == 128) return causal ? launch_dq_pipe_t<128, true>(q, k, v, dO, lse2, neg_delta, dq, maps, B, H, S, scale, stream)
                              : launch_dq_pipe_t<128, false>(q, k, v, dO, lse2, neg_delta, dq, maps, B, H, S, scale, stream);
  return causal ? launch_dq_pipe_t<64, true>(q, k, v, dO, lse2, neg_delta, dq, maps, B, H, S, scale, stream)
                : launch_dq_pipe_t<64, false>(q, k, v, dO, lse2, neg_delta, dq, maps, B, H, S, scale, stream);
}

}  // namespace helix
