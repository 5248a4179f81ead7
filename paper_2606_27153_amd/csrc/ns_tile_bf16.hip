// The bf16 small-tile kernels, every stage (see ns_gemm.h for why they have a
// translation unit of their own).
#include "ns_tile_kernel.h"

namespace muon {

int launch_tile_bf16(int32_t exec, int32_t stage, unsigned grid, const GemmArgs& g, hipStream_t st) {
  switch (exec) {
    case EX_128_RING3: return launch_tile<__bf16, 128, 3>(stage, grid, g, st);
    case EX_128_RING2: return launch_tile<__bf16, 128, 2>(stage, grid, g, st);
    case EX_64_RING3: return launch_tile<__bf16, 64, 3>(stage, grid, g, st);
    default: return -1;
  }
}

int launch_multi_bf16(unsigned grid, const MultiArgs& m, hipStream_t st) {
  return launch_multi<__bf16>(grid, m, st);
}

}  // namespace muon
