// Instantiations of the products whose waves share the contraction, for the three
// layouts, and the paired adjoint launches on them and on the large float32 tiles.
#include "gemm_f32.hpp"
#include "gemm_wave.hpp"

namespace dlvm {
namespace gemm {

namespace {

// Waves of the 64 x 64 tile (configuration 9). bf16 is bound by the loads in flight of
// the one tile a compute unit has (1024 x 1024 x 4096 wrt the weights: 23.1 us with 4
// waves, 21.2 with 8); float32 tiles are several to a unit, and 8 waves' partial tiles
// would leave LDS for one (2048 x 1024 x 768: 34.6 us with 4 waves, 38.3 with 8).
//
// Between it and 32 x 32 (8) stands 32 x 64 (23): forward 1000 x 500 x 784 in bf16 has 256
// such tiles, one to a compute unit, and takes 7.1 us (8: 512 tiles, 8.2; 9: 128 tiles,
// 10.5); float32 777 x 1001 x 2049 wrt the weights 41.4 (8: 45.2; 9: 40.0).
template <typename T> constexpr int kNW9 = sizeof(T) == 2 ? 8 : 4;

template <typename T, typename TO, bool AK, bool BKM, int EPI, bool PH2>
hipError_t launch_wave_layout(const Params& p, int cfg, unsigned grid, hipStream_t s) {
  switch (cfg) {
    case 6:
      launch_kernel((dlvm_gemm_wave_kernel<T, TO, AK, BKM, 1, 1, 8, 4, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    case 7:
      launch_kernel((dlvm_gemm_wave_kernel<T, TO, AK, BKM, 1, 2, 8, 4, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    case 8:
      launch_kernel((dlvm_gemm_wave_kernel<T, TO, AK, BKM, 2, 2, 8, 3, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    case 9:
      launch_kernel((dlvm_gemm_wave_kernel<T, TO, AK, BKM, 4, 4, kNW9<T>, 2, EPI, PH2>), dim3(grid),
                    dim3(64 * kNW9<T>), s, p);
      break;
    case 23:
      launch_kernel((dlvm_gemm_wave_kernel<T, TO, AK, BKM, 2, 4, 8, 3, EPI, PH2>), dim3(grid), dim3(512), s, p);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, typename TO>
hipError_t launch_wave_typed(const Params& p, Layout layout, int cfg, unsigned grid, hipStream_t s) {
  switch (layout) {
    case Layout::NN:
      if (p.A2 != nullptr) return launch_wave_layout<T, TO, true, false, EPI_STORE, true>(p, cfg, grid, s);
      if constexpr (std::is_same<T, float>::value) {
        if (p.partials != nullptr) return launch_wave_layout<T, TO, true, false, EPI_CHAIN, false>(p, cfg, grid, s);
      }
      return launch_wave_layout<T, TO, true, false, EPI_STORE, false>(p, cfg, grid, s);
    case Layout::NT:
      return launch_wave_layout<T, TO, true, true, EPI_DACT, false>(p, cfg, grid, s);
    case Layout::TN:
      return launch_wave_layout<T, float, false, false, EPI_DW, false>(p, cfg, grid, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_wave(const Params& p, Layout layout, int dtype, int out_dtype, int cfg, unsigned grid,
                       hipStream_t s) {
  if (p.mask != nullptr || (p.partials != nullptr && (dtype != F32 || p.splits > 1)))
    return hipErrorInvalidValue;  // (no such epilogue here)
  if (dtype == F32) return launch_wave_typed<float, float>(p, layout, cfg, grid, s);
  if (out_dtype == F32) return launch_wave_typed<bf16_t, float>(p, layout, cfg, grid, s);
  return launch_wave_typed<bf16_t, bf16_t>(p, layout, cfg, grid, s);
}

hipError_t launch_wave_xent(const Params& p, int dtype, hipStream_t s) {
  if (p.N > 32 || p.lda2 > (p.N <= 16 ? 16 : 32) || p.splits > 1 || p.tiles_n != 1) return hipErrorInvalidValue;
  const dim3 g(p.tiles_m), b(512);
  if (dtype == F32) {
    if (p.N <= 16)
      launch_kernel((dlvm_gemm_wave_kernel<float, float, true, false, 1, 1, 8, 4, EPI_XENT, false>), g, b, s, p);
    else
      launch_kernel((dlvm_gemm_wave_kernel<float, float, true, false, 1, 2, 8, 4, EPI_XENT, false>), g, b, s, p);
  } else {
    if (p.N <= 16)
      launch_kernel((dlvm_gemm_wave_kernel<bf16_t, float, true, false, 1, 1, 8, 4, EPI_XENT, false>), g, b, s, p);
    else
      launch_kernel((dlvm_gemm_wave_kernel<bf16_t, float, true, false, 1, 2, 8, 4, EPI_XENT, false>), g, b, s, p);
  }
  return hipGetLastError();
}

namespace {

template <typename T, typename TO2, int AB1, int BB1, int D1>
hipError_t launch_wave_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg_nt,
                            hipStream_t s) {
  switch (cfg_nt) {
    case 6:
      launch_kernel((dlvm_gemm_wave_pair_kernel<T, TO2, AB1, BB1, D1, 1, 1, 4, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
      break;
    case 7:
      launch_kernel((dlvm_gemm_wave_pair_kernel<T, TO2, AB1, BB1, D1, 1, 2, 4, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
      break;
    case 23:
      launch_kernel((dlvm_gemm_wave_pair_kernel<T, TO2, AB1, BB1, D1, 2, 4, 3, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
      break;
    default:
      launch_kernel((dlvm_gemm_wave_pair_kernel<T, TO2, AB1, BB1, D1, 2, 2, 3, 8>), dim3(grid), dim3(512), s, p1, p2, n1);
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

namespace {
template <typename T, typename TO2>
hipError_t launch_wave_pair_typed(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg_tn,
                                  int cfg_nt, hipStream_t s) {
  switch (cfg_tn) {
    case 6: return launch_wave_pair<T, TO2, 1, 1, 4>(p1, p2, n1, grid, cfg_nt, s);
    case 7: return launch_wave_pair<T, TO2, 1, 2, 4>(p1, p2, n1, grid, cfg_nt, s);
    case 8: return launch_wave_pair<T, TO2, 2, 2, 3>(p1, p2, n1, grid, cfg_nt, s);
    case 23: return launch_wave_pair<T, TO2, 2, 4, 3>(p1, p2, n1, grid, cfg_nt, s);
    default:
      launch_kernel((dlvm_gemm_wave_pair_kernel<T, TO2, 4, 4, 2, 4, 4, 2, kNW9<T>>), dim3(grid),
                    dim3(64 * kNW9<T>), s, p1, p2, n1);
      return hipGetLastError();
  }
}
}  // namespace

hipError_t launch_wave_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int dtype,
                            int out_dtype2, int cfg_tn, int cfg_nt, hipStream_t s) {
  if (!pair_config(dtype, cfg_tn, cfg_nt)) return hipErrorInvalidValue;
  if (dtype == F32) return launch_wave_pair_typed<float, float>(p1, p2, n1, grid, cfg_tn, cfg_nt, s);
  if (out_dtype2 == F32) return launch_wave_pair_typed<bf16_t, float>(p1, p2, n1, grid, cfg_tn, cfg_nt, s);
  return launch_wave_pair_typed<bf16_t, bf16_t>(p1, p2, n1, grid, cfg_tn, cfg_nt, s);
}

hipError_t launch_f32_pair(const Params& p1, const Params& p2, int n1, unsigned grid, int cfg, bool vec,
                           hipStream_t s) {
  if (!pair_config(F32, cfg, cfg)) return hipErrorInvalidValue;
  return vec ? launch_lds_pair<true>(p1, p2, n1, grid, cfg, s) : launch_lds_pair<false>(p1, p2, n1, grid, cfg, s);
}

}  // namespace gemm
}  // namespace dlvm
