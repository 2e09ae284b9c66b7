// The tiled GEMM's fp32 kernels (gemm_tile_kernel.hiph), in a file of their own because they take long to compile.
#include "gemm_tile_kernel.hiph"

namespace lora {

hipError_t init_gemm_tile_f32() { return init_tiles<float>(); }

hipError_t launch_gemm_tile_f32(const GemmArgs &a, int variant, hipStream_t stream, const KernelTimer *timer) {
    return launch_variant<float>(a, variant, stream, timer);
}

}  // namespace lora
