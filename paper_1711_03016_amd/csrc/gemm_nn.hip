// Instantiations of the dense-layer product for the NN layout (forward products: bias + activation
// epilogue).
#include "gemm_xl.hpp"

namespace dlvm {
namespace gemm {

hipError_t launch_nn(const Params& p, int dtype, int out_dtype, int cfg, unsigned grid, bool va,
                     bool vb, hipStream_t s) {
  if (p.A2 != nullptr) {  // a two-phase contraction: the kernels that choose A per k-tile
    if (dtype == F32) return launch_f32_far<true, false, EPI_STORE, true>(p, cfg, grid, s);
    if (cfg >= kAsyncFirst) {
      if (out_dtype == F32) return launch_async<float, true, false, EPI_STORE, true>(p, cfg, grid, s);
      return launch_async<bf16_t, true, false, EPI_STORE, true>(p, cfg, grid, s);
    }
    if (out_dtype == F32)
      return launch_vec<bf16_t, float, true, false, EPI_STORE, true>(p, cfg, grid, va, vb, s);
    return launch_vec<bf16_t, bf16_t, true, false, EPI_STORE, true>(p, cfg, grid, va, vb, s);
  }
  if (p.partials != nullptr) return hipErrorInvalidValue;  // (the chain runs on 6-9 and 20-23)
  if (dtype == F32) {  // (16-byte loads of both operands, or element loads of both: the same sums)
    if (va && vb) return launch_cfg<float, float, true, false, true, true, EPI_STORE>(p, cfg, grid, s);
    return launch_cfg<float, float, true, false, false, false, EPI_STORE>(p, cfg, grid, s);
  }
  if (cfg >= kAsyncFirst) {
    if (out_dtype == F32) return launch_bf16<float, true, false, EPI_STORE>(p, cfg, grid, s);
    return launch_bf16<bf16_t, true, false, EPI_STORE>(p, cfg, grid, s);
  }
  if (out_dtype == F32) return launch_vec<bf16_t, float, true, false, EPI_STORE>(p, cfg, grid, va, vb, s);
  return launch_vec<bf16_t, bf16_t, true, false, EPI_STORE>(p, cfg, grid, va, vb, s);
}

}  // namespace gemm
}  // namespace dlvm
