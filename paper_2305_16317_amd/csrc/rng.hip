// Up-front noise of Algorithm 1 (prior point and the noise of every step)
// from the counter-based draws of philox.h: one thread turns one 128-bit
// counter block into four normals.
#include "pd_internal.h"
#include "philox.h"

namespace pd {
namespace {

// Values v of quad q (those below count) into out.
__device__ __forceinline__ void store_quad(const float (&v)[4], int64_t q, int64_t count, float* __restrict__ out) {
    const int64_t base = 4 * q;
    if (base + 3 < count && (count & 3) == 0) {
        *reinterpret_cast<float4*>(out + base) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (base + e < count) out[base + e] = v[e];
    }
}

__global__ __launch_bounds__(256) void k_normals(uint64_t seed, uint32_t rng_stream, int64_t count,
                                                 float* __restrict__ out) {
    const int64_t nq = (count + 3) / 4;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nq; q += step) {
        float v[4];
        normals4(seed, rng_stream, q, v);
        store_quad(v, q, count, out);
    }
}

// The prior (stream 0, BD values into x0) in grid row 0 and the noise (stream
// 1) of step i, times scale[i], in row i + 1 (rows past the grid's 65535 are
// taken in turn); the first block also starts the Picard loop when has_init is
// set.  BD a multiple of four (WHOLE): a quad lies in one step and the scale is
// the row's.  Else the noise is one run of quads shared by the rows, each value
// finding its step by a division.  On 1000 steps of 4x96x96: 74 us, 153
// with four 64-bit divisions a quad and the math library's functions.
template <bool WHOLE>
__global__ __launch_bounds__(256) void k_sample_setup(uint64_t seed, int64_t BD, float* __restrict__ x0, int64_t T,
                                                      const float* __restrict__ scale, float* __restrict__ noise,
                                                      PicardInit init, int has_init) {
    if (has_init && blockIdx.x == 0 && blockIdx.y == 0) picard_init_body(init);
    const int64_t nq = (BD + 3) / 4, step = (int64_t)gridDim.x * blockDim.x;
    const int64_t q0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float v[4];
    if (blockIdx.y == 0)
        for (int64_t q = q0; q < nq; q += step) {
            normals4(seed, 0, q, v);
            store_quad(v, q, BD, x0);
        }
    if (!noise) return;
    if constexpr (WHOLE) {
        for (int64_t r = blockIdx.y; r <= T; r += gridDim.y) {
            if (r == 0) continue;
            const float sc = scale[r - 1];
            for (int64_t q = q0; q < nq; q += step) {
                normals4(seed, 1, (r - 1) * nq + q, v);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = sc * v[e];
                store_quad(v, (r - 1) * nq + q, T * BD, noise);
            }
        }
    } else {
        const int64_t count = T * BD, all = (count + 3) / 4;
        for (int64_t q = blockIdx.y * step + q0; q < all; q += step * gridDim.y) {
            normals4(seed, 1, q, v);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * q + e < count) v[e] = scale[(4 * q + e) / BD] * v[e];
            store_quad(v, q, count, noise);
        }
    }
}

}  // namespace

void launch_normals(uint64_t seed, uint32_t rng_stream, int64_t count, float* out, hipStream_t s) {
    if (count <= 0) return;
    const int64_t nq = (count + 3) / 4;
    int64_t blocks = (nq + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_normals, dim3((unsigned)blocks), dim3(256), 0, s, seed, rng_stream, count, out);
    PD_HIP(hipGetLastError());
}

void launch_sample_setup(uint64_t seed, int64_t BD, float* x0, int64_t T, const float* scale, float* noise,
                         const PicardInit* init, hipStream_t s) {
    int64_t blocks = ((BD + 3) / 4 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    const int64_t rows = noise ? (T + 1 < 65535 ? T + 1 : 65535) : 1;
    const PicardInit none{};
    const dim3 grid((unsigned)blocks, (unsigned)rows), block(256);
    if (BD % 4 == 0)
        hipLaunchKernelGGL(k_sample_setup<true>, grid, block, 0, s, seed, BD, x0, T, scale, noise,
                           init ? *init : none, init ? 1 : 0);
    else
        hipLaunchKernelGGL(k_sample_setup<false>, grid, block, 0, s, seed, BD, x0, T, scale, noise,
                           init ? *init : none, init ? 1 : 0);
    PD_HIP(hipGetLastError());
}

}  // namespace pd
