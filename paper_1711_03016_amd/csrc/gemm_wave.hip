// Instantiations of the float32 products whose waves share the contraction,
// for the three layouts, and the paired adjoint launches of float32 products.
#include "gemm_f32.hpp"
#include "gemm_wave.hpp"

namespace dlvm {
namespace gemm {

namespace {

template <bool AK, bool BKM, int EPI, bool PH2>
hipError_t launch_wave_layout(const Params& p, int cfg, unsigned grid, hipStream_t s) {
  switch (cfg) {
    case 6:
      launch_kernel((dlvm_gemm_wave_kernel<AK, BKM, 1, 1, 8, 4, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    case 7:
      launch_kernel((dlvm_gemm_wave_kernel<AK, BKM, 1, 2, 8, 4, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    case 8:
      launch_kernel((dlvm_gemm_wave_kernel<AK, BKM, 2, 2, 8, 3, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    case 9:
      launch_kernel((dlvm_gemm_wave_kernel<AK, BKM, 4, 4, 4, 2, EPI, PH2>), dim3(grid), dim3(256), s, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wave(const Params& p, Layout layout, int cfg, unsigned grid, hipStream_t s) {
  if (p.partials != nullptr) return hipErrorInvalidValue;  // (no chain epilogue here)
  switch (layout) {
    case Layout::NN:
      if (p.A2 != nullptr) return launch_wave_layout<true, false, EPI_STORE, true>(p, cfg, grid, s);
      return launch_wave_layout<true, false, EPI_STORE, false>(p, cfg, grid, s);
    case Layout::NT:
      return launch_wave_layout<true, true, EPI_DACT, false>(p, cfg, grid, s);
    case Layout::TN:
      return launch_wave_layout<false, false, EPI_DW, false>(p, cfg, grid, s);
  }
  return hipErrorInvalidValue;
}

namespace {

template <int AB1, int BB1, int D1>
hipError_t launch_wave_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg_nt,
                            hipStream_t s) {
  switch (cfg_nt) {
    case 6:
      launch_kernel((dlvm_gemm_wave_pair_kernel<AB1, BB1, D1, 1, 1, 4, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
      break;
    case 7:
      launch_kernel((dlvm_gemm_wave_pair_kernel<AB1, BB1, D1, 1, 2, 4, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
      break;
    default:
      launch_kernel((dlvm_gemm_wave_pair_kernel<AB1, BB1, D1, 2, 2, 3, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
      break;
  }
  return hipGetLastError();
}

template <bool VEC>
hipError_t launch_lds_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg,
                           hipStream_t s) {
  switch (cfg) {
    case 20:
      launch_kernel((dlvm_gemm_f32_pair_kernel<128, 128, 2, 2, 2, VEC>), dim3(grid), dim3(256), s, p1, p2, n1);
      break;
    case 22:
      launch_kernel((dlvm_gemm_f32_pair_kernel<128, 64, 2, 2, 3, VEC>), dim3(grid), dim3(256), s, p1, p2, n1);
      break;
    default:
      launch_kernel((dlvm_gemm_f32_pair_kernel<64, 64, 2, 2, 3, VEC>), dim3(grid), dim3(256), s, p1, p2, n1);
      break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_f32_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg_tn,
                           int cfg_nt, bool vec, hipStream_t s) {
  if (!pair_config(F32, cfg_tn, cfg_nt)) return hipErrorInvalidValue;
  switch (cfg_tn) {
    case 6: return launch_wave_pair<1, 1, 4>(p1, p2, n1, grid, cfg_nt, s);
    case 7: return launch_wave_pair<1, 2, 4>(p1, p2, n1, grid, cfg_nt, s);
    case 8: return launch_wave_pair<2, 2, 3>(p1, p2, n1, grid, cfg_nt, s);
    case 9:
      launch_kernel((dlvm_gemm_wave_pair_kernel<4, 4, 2, 4, 4, 2, 4>), dim3(grid), dim3(256), s, p1, p2, n1);
      return hipGetLastError();
    default:
      return vec ? launch_lds_pair<true>(p1, p2, n1, grid, cfg_tn, s)
                 : launch_lds_pair<false>(p1, p2, n1, grid, cfg_tn, s);
  }
}

}  // namespace gemm
}  // namespace dlvm
