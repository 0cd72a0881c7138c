// Instantiations of the large float32 products for the three layouts.
#include "gemm_f32.hpp"

namespace dlvm {
namespace gemm {

namespace {

template <bool AK, bool BKM, bool VEC, int EPI, bool PH2>
hipError_t launch_f32_layout(const Params& p, int cfg, unsigned grid, hipStream_t s) {
  switch (cfg) {
    case 20:
      launch_kernel((dlvm_gemm_f32_kernel<AK, BKM, 128, 128, 2, 2, 2, VEC, EPI, PH2>), dim3(grid), dim3(256), s, p);
      break;
    case 21:
      launch_kernel((dlvm_gemm_f32_kernel<AK, BKM, 64, 64, 2, 2, 3, VEC, EPI, PH2>), dim3(grid), dim3(256), s, p);
      break;
    case 22:
      launch_kernel((dlvm_gemm_f32_kernel<AK, BKM, 128, 64, 2, 2, 3, VEC, EPI, PH2>), dim3(grid), dim3(256), s, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool VEC>
hipError_t launch_f32_vec(const Params& p, Layout layout, int cfg, unsigned grid, hipStream_t s) {
  switch (layout) {
    case Layout::NN:
      if (p.A2 != nullptr) return launch_f32_layout<true, false, VEC, EPI_STORE, true>(p, cfg, grid, s);
      if (p.partials != nullptr) return launch_f32_layout<true, false, VEC, EPI_CHAIN, false>(p, cfg, grid, s);
      return launch_f32_layout<true, false, VEC, EPI_STORE, false>(p, cfg, grid, s);
    case Layout::NT:
      return launch_f32_layout<true, true, VEC, EPI_DACT, false>(p, cfg, grid, s);
    case Layout::TN:
      return launch_f32_layout<false, false, VEC, EPI_DW, false>(p, cfg, grid, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_f32(const Params& p, Layout layout, int cfg, unsigned grid, bool vec, hipStream_t s) {
  return vec ? launch_f32_vec<true>(p, layout, cfg, grid, s) : launch_f32_vec<false>(p, layout, cfg, grid, s);
}

}  // namespace gemm
}  // namespace dlvm
