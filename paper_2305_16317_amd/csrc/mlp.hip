// Dense layers of the synthetic MLP denoiser on the matrix cores: one block
// per output tile (the tile itself is computed in linear_tile.h).  A layer is
// bound by the loads of its busiest compute unit and by the latency around
// them, so the launch picks the tile by the rows and features it has.
#include "eps_out.h"
#include "linear_tile.h"
#include "mlp.h"

namespace pd {
namespace {

__device__ __forceinline__ TileRows tile_rows_of(const RowSrc& src, const HiddenBuf& in, int64_t D) {
    return TileRows{(src.active ? *src.active : src.max_groups) * src.group, src.max_groups * src.group, in, &src, D,
                    nullptr, 0, nullptr};
}

// The largest tile is held to the registers of four waves per SIMD, two blocks
// per compute unit: with one block a forward of 1024 rows takes 94 us, with two 81.
constexpr int tile_waves(int rt, int ct) { return rt * ct == 4 ? 4 : kLinWaves / 4; }

template <int RT, int CT, LinearIn IN, bool SPLIT>
__global__ __launch_bounds__(kLinThreads) __attribute__((amdgpu_waves_per_eu(tile_waves(RT, CT))))
void k_linear(LinearArgs a, RowSrc src, HiddenBuf in, int64_t D, HiddenBuf out) {
    __shared__ LinearLds<RT, CT> lds;
    hidden_tile<RT, CT, IN, SPLIT>(a, tile_rows_of(src, in, D), out, blockIdx.y * RT, blockIdx.x * CT, lds);
}

// The last layer: epsilon, row-major, or the step that follows it.  With h,
// each output's Euler prediction in the window (Heun's first stage).
template <int RT, int CT, bool SPLIT, bool PREDICT>
__global__ __launch_bounds__(kLinThreads) __attribute__((amdgpu_waves_per_eu(tile_waves(RT, CT))))
void k_linear_out(LinearArgs a, RowSrc src, HiddenBuf in, HeunPredictArgs h, EpsOut out) {
    __shared__ LinearLds<RT, CT> lds;
    const int mt0 = blockIdx.y * RT, nt0 = blockIdx.x * CT;
    const TileRows rows = tile_rows_of(src, in, 0);
    const int M = rows.M, N = a.N;
    linear_tile<RT, CT, IN_HIDDEN, SPLIT>(
        a, rows, mt0, nt0, lds, [&](int tile, float e) {
            const int row = 16 * (mt0 + tile / CT) + ((threadIdx.x >> 2) & 15);
            const int n = 16 * (nt0 + tile % CT) + 4 * ((threadIdx.x >> 6) & 3) + (threadIdx.x & 3);
            if (row >= M || n >= N) return;
            if constexpr (!PREDICT) {
                eps_out(out, (int64_t)row * N + n, e);
            } else {
                out.y[(int64_t)row * N + n] = e;
                const LoopState cur = *h.st;
                const int j = row / src.group, b = row % src.group;
                const int m = cur.t + j;
                const int64_t BD = (int64_t)src.group * N;
                const int64_t c = (int64_t)b * N + n;
                const float x = h.ring[(int64_t)((m <= cur.f ? m : cur.f) % h.ring_slots) * BD + c];
                h.xt[(int64_t)j * BD + c] = __fadd_rn(x, drift(h.A[m], x, h.B[m], e));
            }
        });
}

// Weights [N][K] -> packed fragments (layout in linear_tile.h), one block per
// 16 features and layer (blockIdx.y); with `split`, also the exponent of each
// feature's power of two.  *nonfinite is set when a weight is infinite or NaN.
// Bound by the latency of its loads: whole rows in 16-byte pieces, several in
// flight, 11 us for a layer of 1024 x 1024, so that the layers go together.
__global__ __launch_bounds__(256) void k_pack_linear(PackLayers layers, int32_t* nonfinite) {
    __shared__ uint32_t s_max[16];
    const PackLayer& a = layers.at[blockIdx.y];
    const float* __restrict__ W = a.w;
    float* __restrict__ out = a.out;
    int32_t* __restrict__ wexp = a.wexp;
    const int N = a.N, K = a.K;
    const bool split = wexp != nullptr;
    const int nt = blockIdx.x, tid = threadIdx.x, i = tid & 15;
    if (16 * nt >= N) return;                    // uniform over the block
    const int n = 16 * nt + i;
    const lin_f4 zero = {0.f, 0.f, 0.f, 0.f};
    {   // 16 neighbouring threads a feature
        const int r = tid >> 4, nr = 16 * nt + r;
        uint32_t mr = 0;
        if (nr < N) {
            const lin_f4* row = reinterpret_cast<const lin_f4*>(W + (int64_t)nr * K);
#pragma unroll 8
            for (int k4 = i; k4 < K / 4; k4 += 16) {
                const lin_f4 v = row[k4];
                // the conversion matters: of a vector's element itself bit_cast reads
                // the vector's first
#pragma unroll
                for (int u = 0; u < 4; ++u) mr = umax32(mr, __builtin_bit_cast(uint32_t, (float)v[u]) & 0x7fffffffu);
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) mr = umax32(mr, (uint32_t)__shfl_xor((int)mr, o, 16));
        if (i == 0) s_max[r] = mr;
    }
    __syncthreads();
    const uint32_t m = s_max[i];
    if (m >= 0x7f800000u) *nonfinite = 1;        // every writer stores the same value
    int e = m > 0 && m < 0x7f800000u ? (int)(m >> 23) - 127 : 0;
    e = e < -126 ? -126 : e;
    // w 2^(14 - e) in [2^14, 2^15) for the feature's largest weight, in two exact
    // steps (2^(14 - e) alone may exceed the float range)
    const int sh = 14 - e;
    const float f1 = __builtin_bit_cast(float, (uint32_t)(sh / 2 + 127) << 23);
    const float f2 = __builtin_bit_cast(float, (uint32_t)(sh - sh / 2 + 127) << 23);
    if (split && tid < 16 && n < N) wexp[n] = -sh;
    const int KC = (K + 31) / 32;
    float* dst = out + (int64_t)nt * KC * 512;   // 2 KB per chunk
    // thread: feature i, inputs 32 c + 16 (u / 4) + 4 g + u % 4 of lane i + 16 g
#pragma unroll 4
    for (int q = tid >> 4; q < KC * 4; q += 16) {
        const int c = q >> 2, g = q & 3, lane = i + 16 * g;
        float w[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = 32 * c + 16 * h + 4 * g;     // K is a multiple of four
            const lin_f4 v = n < N && k < K ? *reinterpret_cast<const lin_f4*>(W + (int64_t)n * K + k) : zero;
#pragma unroll
            for (int u = 0; u < 4; ++u) w[4 * h + u] = v[u];
        }
        if (split) {
            lin_h8 p0, p1;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float s = w[u] * f1 * f2;
                p0[u] = (_Float16)s;
                // zero only where the weight is, for its products with infinities
                // (the second part takes the difference back)
                if (p0[u] == (_Float16)0.f && w[u] != 0.f) p0[u] = (_Float16)__builtin_copysignf(0x1p-24f, w[u]);
                p1[u] = (_Float16)(s - (float)p0[u]);
            }
            reinterpret_cast<lin_h8*>(dst)[(c * 2) * 64 + lane] = p0;
            reinterpret_cast<lin_h8*>(dst)[(c * 2 + 1) * 64 + lane] = p1;
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                reinterpret_cast<lin_f4*>(dst)[(c * 2 + h) * 64 + lane] =
                    lin_f4{w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]};
        }
    }
}

// The tile of a launch, in 16 x 16 blocks.  A block loads RT row tiles and CT
// feature tiles whole (64 KB each at 1024 inputs), so the busiest compute unit
// takes in rounds x (RT + CT) of them; ties go to the smaller tile (more
// blocks, less to add up).  Four layers of 1024 (160 in and out), us: one row
// 19.4 as 1 x 1 and 21.9 as 1 x 2; 100 rows 28.8, 26.3, 30.7 as 2 x 2; 160 rows
// 35.5, 37.5, 31.1; 320 rows 49, 51, 41; 777 rows 97, 98, 60.  Larger tiles
// (2 x 4, 4 x 4) have one block per unit, whose phases nothing overlaps: 64 and
// 63 us at 777 rows.
struct TileChoice {
    int rt, ct;
};
TileChoice choose_tile(int64_t rows, int N) {
    static constexpr TileChoice kTiles[] = {{1, 1}, {1, 2}, {2, 2}};
    const int64_t MT = (rows + 15) / 16, NT = (N + 15) / 16, cus = device_cus();
    TileChoice best{1, 1};
    int64_t cost = INT64_MAX;
    for (const TileChoice& t : kTiles) {
        const int64_t blocks = ((MT + t.rt - 1) / t.rt) * ((NT + t.ct - 1) / t.ct);
        const int64_t c = (blocks + cus - 1) / cus * (t.rt + t.ct);
        if (c < cost) {
            cost = c;
            best = t;
        }
    }
    return best;
}

// f(rows per tile, features per tile as integral constants, grid)
template <class F>
void with_tile(int64_t rows, int N, F&& f) {
    const TileChoice t = choose_tile(rows, N);
    auto go = [&](auto rt, auto ct) {
        constexpr int RT = decltype(rt)::value, CT = decltype(ct)::value;
        f(rt, ct, dim3((unsigned)((N + 16 * CT - 1) / (16 * CT)), (unsigned)((rows + 16 * RT - 1) / (16 * RT))));
    };
    using std::integral_constant;
    if (t.rt == 2) go(integral_constant<int, 2>{}, integral_constant<int, 2>{});
    else if (t.ct == 2) go(integral_constant<int, 1>{}, integral_constant<int, 2>{});
    else go(integral_constant<int, 1>{}, integral_constant<int, 1>{});
}

void check_sizes(const LinearArgs& a) {
    if ((a.K % 4) != 0 || (a.N % 4) != 0) fail(PD_ERR_UNSUPPORTED, "mlp layer sizes must be multiples of 4");
}

template <LinearIn IN>
void launch_hidden(const LinearArgs& a, const RowSrc& rows, const HiddenBuf& in, int64_t D, const HiddenBuf& out,
                   hipStream_t s) {
    const int64_t M = (int64_t)rows.max_groups * rows.group;
    if (M == 0) return;
    check_sizes(a);
    with_tile(M, a.N, [&](auto rt, auto ct, dim3 grid) {
        constexpr int RT = decltype(rt)::value, CT = decltype(ct)::value;
        const dim3 block(kLinThreads);
        if (a.wexp) hipLaunchKernelGGL((k_linear<RT, CT, IN, true>), grid, block, 0, s, a, rows, in, D, out);
        else hipLaunchKernelGGL((k_linear<RT, CT, IN, false>), grid, block, 0, s, a, rows, in, D, out);
    });
    PD_HIP(hipGetLastError());
}

template <bool PREDICT>
void launch_out(const LinearArgs& a, const HiddenBuf& in, const RowSrc& rows, const HeunPredictArgs& h,
                const EpsOut& out, hipStream_t s) {
    const int64_t M = (int64_t)rows.max_groups * rows.group;
    if (M == 0) return;
    check_sizes(a);
    with_tile(M, a.N, [&](auto rt, auto ct, dim3 grid) {
        constexpr int RT = decltype(rt)::value, CT = decltype(ct)::value;
        const dim3 block(kLinThreads);
        if (a.wexp) hipLaunchKernelGGL((k_linear_out<RT, CT, true, PREDICT>), grid, block, 0, s, a, rows, in, h, out);
        else hipLaunchKernelGGL((k_linear_out<RT, CT, false, PREDICT>), grid, block, 0, s, a, rows, in, h, out);
    });
    PD_HIP(hipGetLastError());
}

}  // namespace

size_t hidden_floats(int64_t rows, int width) {
    const int64_t nt4 = ((width + 15) / 16 + 3) / 4 * 4;
    return (size_t)(rows * width + rows * nt4 + 3) / 4 * 4;
}
HiddenBuf hidden_buf(float* p, int64_t rows, int width) {
    return HiddenBuf{p, reinterpret_cast<uint32_t*>(p + rows * width)};
}

size_t packed_linear_floats(int N, int K) { return (size_t)((N + 15) / 16) * ((K + 31) / 32) * 512; }

void launch_pack_linear(const PackLayers& layers, int count, int32_t* nonfinite, hipStream_t s) {
    int n = 0;
    for (int i = 0; i < count; ++i) n = layers.at[i].N > n ? layers.at[i].N : n;
    hipLaunchKernelGGL(k_pack_linear, dim3((unsigned)((n + 15) / 16), (unsigned)count), dim3(256), 0, s, layers,
                       nonfinite);
    PD_HIP(hipGetLastError());
}

void launch_linear_first(const LinearArgs& a, const RowSrc& src, int64_t D, const HiddenBuf& out, hipStream_t s) {
    launch_hidden<IN_GATHER>(a, src, HiddenBuf{}, D, out, s);
}

void launch_linear_hidden(const LinearArgs& a, const HiddenBuf& in, const RowSrc& rows, const HiddenBuf& out,
                          hipStream_t s) {
    launch_hidden<IN_HIDDEN>(a, rows, in, 0, out, s);
}

void launch_linear_out(const LinearArgs& a, const HiddenBuf& in, const RowSrc& rows, const EpsOut& out,
                       hipStream_t s) {
    launch_out<false>(a, in, rows, HeunPredictArgs{}, out, s);
}

void launch_linear_out_predict(const LinearArgs& a, const HiddenBuf& in, const RowSrc& rows, const HeunPredictArgs& h,
                               float* y, hipStream_t s) {
    launch_out<true>(a, in, rows, h, eps_store(y), s);
}

}  // namespace pd
