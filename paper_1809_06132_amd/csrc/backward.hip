// Soft-argmin backward pass (the kernels themselves are in backward_impl.h):
// the forms for levels of fronto planes only, the zero and pose-reduce
// kernels, and the lookup of a form by window, source count, image format,
// image-gradient request and plane families.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "backward_impl.h"

namespace psw {

// the image gradients of up to four sources, one launch (blockIdx.y: source)
__global__ void zero_kernel(float *p0, float *p1, float *p2, float *p3, int64_t n0, int64_t n1, int64_t n2, int64_t n3) {
    float *const p = blockIdx.y == 0 ? p0 : blockIdx.y == 1 ? p1 : blockIdx.y == 2 ? p2 : p3;
    const int64_t n = blockIdx.y == 0 ? n0 : blockIdx.y == 1 ? n1 : blockIdx.y == 2 ? n2 : n3;
    if (!p) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

// Sum of the workgroups' pose partial sums: workgroup c adds column c, each of
// its 256 threads a strided share of the rows, then a fixed tree (the same
// order every time).  Bound by the latency of its reads: four of a thread's are
// in flight, next to its neighbours' in memory.
__global__ __launch_bounds__(256) void pose_reduce_kernel(const double *__restrict__ gpart, int n_rows,
                                                          double *__restrict__ gpose) {
    __shared__ double part[256 / kWave];
    const int t = threadIdx.x;
    const double *col = gpart + (int64_t)blockIdx.x * n_rows;
    double acc = 0.0;
    for (int r = t; r < n_rows; r += 1024) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = r + 256 * k < n_rows ? col[r + 256 * k] : 0.0;
        acc += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int o = kWave / 2; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, kWave);
    if (t % kWave == 0) part[t / kWave] = acc;
    __syncthreads();
    if (t == 0) gpose[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

}  // namespace psw

extern "C" {
const void *psw_backward_ground_kernel(int win, int n_src, int img, int image_grads);   // backward_ground.hip

const void *psw_zero_kernel() { return (const void *)&psw::zero_kernel; }
const void *psw_pose_reduce_kernel() { return (const void *)&psw::pose_reduce_kernel; }

const void *psw_backward_kernel(int win, int n_src, int img, int image_grads, int ground) {
    if (ground) return psw_backward_ground_kernel(win, n_src, img, image_grads);
#define PSW_B(W, I, G)                                                                      \
    if (win == W && img == I && (image_grads != 0) == G) {                                  \
        if (n_src == 1) return (const void *)&psw::backward_kernel<W, 1, I, G, false>;     \
        if (n_src == 2) return (const void *)&psw::backward_kernel<W, 2, I, G, false>;     \
        if (n_src == 3) return (const void *)&psw::backward_kernel<W, 3, I, G, false>;     \
        if (n_src == 4) return (const void *)&psw::backward_kernel<W, 4, I, G, false>;     \
    }
    PSW_B(5, 0, true) PSW_B(7, 0, true) PSW_B(9, 0, true) PSW_B(5, 1, true) PSW_B(7, 1, true) PSW_B(9, 1, true)
    PSW_B(5, 0, false) PSW_B(7, 0, false) PSW_B(9, 0, false) PSW_B(5, 1, false) PSW_B(7, 1, false)
    PSW_B(9, 1, false)
#undef PSW_B
    return nullptr;
}

int psw_backward_tile_rows() { return psw::Backward<5, 1, 0, true, false>::TYO; }
int psw_backward_threads(int image_grads) {
    return image_grads ? psw::Backward<5, 1, 0, true, false>::NW * psw::kWave : psw::Backward<5, 1, 0, false, false>::NW * psw::kWave;
}

size_t psw_backward_lds(int win, int n_src, int image_grads) {
#define PSW_L(W, G)                                                          \
    if (win == W && (image_grads != 0) == G) {                               \
        if (n_src == 1) return psw::Backward<W, 1, 0, G, false>::lds_bytes();       \
        if (n_src == 2) return psw::Backward<W, 2, 0, G, false>::lds_bytes();       \
        if (n_src == 3) return psw::Backward<W, 3, 0, G, false>::lds_bytes();       \
        if (n_src == 4) return psw::Backward<W, 4, 0, G, false>::lds_bytes();       \
    }
    PSW_L(5, true) PSW_L(7, true) PSW_L(9, true) PSW_L(5, false) PSW_L(7, false) PSW_L(9, false)
#undef PSW_L
    return 0;
}
}
