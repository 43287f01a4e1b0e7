// Extend (chunked prefill) attention over the paged cache: kernel entry
// points.  The algorithms live in extend_body.h.
#include "extend_body.h"

namespace pa {
namespace {

template <int G>
__global__ void __launch_bounds__(64 * mfma::kWaves) __attribute__((amdgpu_waves_per_eu(2, 8)))
extend_mfma_kernel(const ExtendParams p) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[extend::kLdsBytes];
  extend::extend_body<G>(p, blockIdx.x, (lds_u8_t*)smem);
}

template <int G>
__global__ void __launch_bounds__(64 * mfma::kWaves) __attribute__((amdgpu_waves_per_eu(2, 8)))
extend_split_kernel(const ExtendParams p) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[extend::kSplitLdsBytes];
  extend::extend_split_body<G>(p, blockIdx.x, (lds_u8_t*)smem);
}

template <int G>
hipError_t launch_t(ExtendParams p, hipStream_t stream) {
  auto grid_of = [&](int rows_per_wg) {
    p.groups = (int32_t)(((int64_t)p.max_chunk * G + rows_per_wg - 1) / rows_per_wg);
    return (int64_t)p.batch * p.groups * p.num_kv_heads;
  };
  const dim3 blk(64 * mfma::kWaves);
  // The split form while its workgroups, weighed by the tokens a chunk's
  // average row sees against the longest context, are all resident at once
  // (two per CU), or while they are at most twice the 128-row form's, whose
  // tiles are then mostly empty.  128-row / split form, chunks over their
  // contexts, 32 heads over 8: one of 256 over 2560 (256 split workgroups)
  // 65.8 / 27.7 us, 512 over 2816 (512) 72.6 / 45.9, 1000 over 3304 (1000)
  // 83.5 / 92.7; four of 128 over 640 (512) 22.5 / 16.3, eight (1024) 24.3 /
  // 30.0; 128 of 16 over 1040 (2048, twice the others) 93.2 / 79.9; one head
  // of 8, the whole context of 4096 (1024, half as many weighed) 98.7 / 81.2;
  // 128 single tokens over 2049, 64 heads over 8 (equal counts) 156 / 66.6.
  const int64_t split = grid_of(kSharedTileRows);
  const int64_t rows = grid_of(kExtendRowsPerWg);
  if (rows > 0x7fffffffLL) return hipErrorInvalidValue;
  if (split <= 0x7fffffffLL && (split * (2 * (int64_t)p.max_ctx - p.max_chunk) <= 2 * 512 * (int64_t)p.max_ctx ||
                                split <= 2 * rows)) {
    grid_of(kSharedTileRows);
    hipLaunchKernelGGL(extend_split_kernel<G>, dim3((unsigned)split), blk, 0, stream, p);
  } else {
    hipLaunchKernelGGL(extend_mfma_kernel<G>, dim3((unsigned)rows), blk, 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_extend(const ExtendParams& p, int group, hipStream_t stream) {
  if (group == 4) return launch_t<4>(p, stream);
  if (group == 8) return launch_t<8>(p, stream);
  return hipErrorInvalidValue;
}

}  // namespace pa
