// Stand-alone cell binning of one frame: the binning body of bin.h by z
// layers, 1024 threads a workgroup (the PPPM step runs the same body as extra
// workgroups of its first mesh launch instead).
#include "bin.h"

namespace cpm {

constexpr int BIN_THREADS = 1024;

__global__ __launch_bounds__(BIN_THREADS) void k_bin_sites(BinArgs a) {
  extern __shared__ __align__(16) int lds[];
  bin_layers_block<BIN_THREADS>(a, blockIdx.x, gridDim.x, lds);
}

size_t bin_lds_bytes(int n_site, int n_cells) { return bin_body_lds<BIN_THREADS>(n_site, n_cells); }

void launch_bin_sites(hipStream_t s, const BinArgs& a) {
  hipLaunchKernelGGL(k_bin_sites, dim3(bin_layer_wgs(a.cell)), dim3(BIN_THREADS),
                     bin_layers_lds<BIN_THREADS>(a.n_site, a.cell), s, a);
}

}  // namespace cpm
