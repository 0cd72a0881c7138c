// Instantiations of the paired launch of a layer's two adjoint products (TN
// wrt the weights, NT wrt the input) of bf16 networks: register-staged
// configuration 3, direct-to-LDS configurations 10 and 12.
#include "gemm_xl.hpp"

namespace dlvm {
namespace gemm {

bool pair_config(int dtype, int cfg_tn, int cfg_nt) {
  // (6, 7, 8 and 23 have the same number of waves, so any two of them share a launch)
  auto eight = [](int c) { return (c >= 6 && c <= 8) || c == 23; };
  if (eight(cfg_tn) && eight(cfg_nt)) return true;
  if (cfg_tn != cfg_nt) return false;
  if (cfg_tn == 9) return true;
  if (dtype == F32) return cfg_tn >= 20 && cfg_tn <= 22;
  return cfg_tn == 3 || cfg_tn == 10 || cfg_tn == 12;
}

namespace {

template <typename T, typename TO2>
hipError_t launch_reg_pair(const Params& p1, const Params& p2, int n1, unsigned grid,
                           hipStream_t s) {
  launch_kernel((dlvm_gemm_pair_kernel<T, TO2, 32, 32, 1, 1, 4, 4>), dim3(grid), dim3(256), s,
                  p1, p2, n1);
  return hipGetLastError();
}

template <typename TO2>
hipError_t launch_async_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg,
                             hipStream_t s) {
  if (cfg == 10)
    launch_kernel((dlvm_gemm_async_pair_kernel<TO2, 256, 256, 64, 2, 4, 2>), dim3(grid),
                  dim3(512), s, p1, p2, n1);
  else
    launch_kernel((dlvm_gemm_async_pair_kernel<TO2, 128, 128, 64, 2, 2, 4>), dim3(grid),
                  dim3(256), s, p1, p2, n1);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int out_dtype2, int cfg,
                       hipStream_t s) {
  if (cfg >= kAsyncFirst) {
    if (out_dtype2 == F32) return launch_async_pair<float>(p1, p2, n1, grid, cfg, s);
    return launch_async_pair<bf16_t>(p1, p2, n1, grid, cfg, s);
  }
  if (out_dtype2 == F32) return launch_reg_pair<bf16_t, float>(p1, p2, n1, grid, s);
  return launch_reg_pair<bf16_t, bf16_t>(p1, p2, n1, grid, s);
}

}  // namespace gemm
}  // namespace dlvm
