// The tiled GEMM's bf16 kernels (gemm_tile_kernel.hiph), its launch by data type, and the launch that sums a GEMM split along K.
#include "gemm_tile_kernel.hiph"

namespace lora {
namespace {

// The second launch of a GEMM split along K: one thread = 8 consecutive columns of one row; the splits' partials are
// requested together and summed in split order, the adapter term of rows with an adapter is added, Y is rounded once.
template <typename E>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(SplitReduceArgs p) {
    if (p.plan.scalars[kScStatus] != 0) return;
    const int n8 = (p.N + 7) >> 3;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)p.T * n8) return;
    const int row = (int)(idx / n8), n = (int)(idx % n8) * 8;
    const bool has = p.D != nullptr && p.plan.row_adapter[row] >= 0 && row_ext_rank(p.plan.row_ext[row]) > 0;
    constexpr int kMaxSplit = 8;
    chunk_t q[kMaxSplit][2];
    const float *src = p.P + (int64_t)row * p.ldp + n;  // (rows are ldp >= N rounded up to 8 floats long: whole pieces are readable)
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s) {
        const float *ps = src + (int64_t)min(s, p.split_k - 1) * p.T * p.ldp;
        q[s][0] = load_chunk(ps);
        q[s][1] = load_chunk(ps + 4);
    }
    const float *dsrc = has ? p.D + (int64_t)row * p.ldd + n : src;
    const chunk_t d0 = load_chunk(dsrc), d1 = load_chunk(dsrc + 4);
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s) {
        if (s < p.split_k) {
            v[0] += __uint_as_float(q[s][0].x);
            v[1] += __uint_as_float(q[s][0].y);
            v[2] += __uint_as_float(q[s][0].z);
            v[3] += __uint_as_float(q[s][0].w);
            v[4] += __uint_as_float(q[s][1].x);
            v[5] += __uint_as_float(q[s][1].y);
            v[6] += __uint_as_float(q[s][1].z);
            v[7] += __uint_as_float(q[s][1].w);
        }
    }
    if (has) {
        v[0] += __uint_as_float(d0.x);
        v[1] += __uint_as_float(d0.y);
        v[2] += __uint_as_float(d0.z);
        v[3] += __uint_as_float(d0.w);
        v[4] += __uint_as_float(d1.x);
        v[5] += __uint_as_float(d1.y);
        v[6] += __uint_as_float(d1.z);
        v[7] += __uint_as_float(d1.w);
    }
    E *y = static_cast<E *>(p.Y) + (int64_t)row * p.ldy + n;
    if (n + 7 < p.N) {
        store8(y, v);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (n + e < p.N) store1(y + e, v[e]);
    }
}

}  // namespace

hipError_t init_gemm_tile_kernels() {
    const hipError_t e = init_tiles<__bf16>();
    return e == hipSuccess ? init_gemm_tile_f32() : e;
}

hipError_t launch_gemm_tile(const GemmArgs &a, int dtype, int variant, hipStream_t stream, const KernelTimer *timer) {
    return dtype == 1 ? launch_variant<__bf16>(a, variant, stream, timer) : launch_gemm_tile_f32(a, variant, stream, timer);
}

hipError_t launch_splitk_reduce(const SplitReduceArgs &a, int dtype, hipStream_t stream, const KernelTimer *timer) {
    if (a.T <= 0 || a.N <= 0) return hipSuccess;
    if (a.split_k < 1 || a.split_k > 8 || a.P == nullptr || a.Y == nullptr || a.ldp < a.N || (a.ldp & 7) != 0 ||
        (a.D != nullptr && (a.ldd < a.N || (a.ldd & 7) != 0)))
        return hipErrorInvalidValue;
    const long threads = (long)a.T * ((a.N + 7) / 8);
    const dim3 grid((unsigned)((threads + 255) / 256));
    if (dtype == 1) return launch_kernel(splitk_reduce_kernel<__bf16>, grid, dim3(256), 0, stream, timer, a);
    return launch_kernel(splitk_reduce_kernel<float>, grid, dim3(256), 0, stream, timer, a);
}

}  // namespace lora
