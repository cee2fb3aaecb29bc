// One output tile of a dense layer y = act(x W^T + bias) (or + shift[n_row]
// for the first layer, which carries b1 + e_n) of the synthetic MLP denoiser.
// Shared by the layer kernels (mlp.hip) and the Picard update with the next
// iteration's first layer (picard.hip).
//
// Layers are computed transposed, out^T = W x^T: the MFMA's M dimension is the
// output feature and its N dimension the row.  A tile is RT x CT blocks of
// 16 rows x 16 features; the block's kLinWaves waves each take a contiguous
// run of the 32-input reduction chunks of the whole tile, so every weight and
// input of the tile is loaded once per block, and the partial tiles are added
// through LDS in wave order (the same order for every tile shape: a row's
// result does not depend on how many rows there are).
//
// What bounds it: at the policy's sizes a layer is a few microseconds of
// latency (launch, first loads, reduction) around the tile's loads, which one
// compute unit takes in at 64 B a cycle.  So operands lie in memory exactly as
// the lanes take them: lane l = i + 16 g of a chunk c holds inputs
// k = 32 c + 16 q + 4 g + e (q = 0, 1; e = 0..3) of feature or row i,
//   weights  [feature tile][c][q or part][lane][16 B]
//   hidden   [row tile][k / 4][row][4]     (k / 4 = 8 c + 4 q + g)
// and a wave's load is 1 KB (weights) or four runs of 256 B (rows), all of
// them in flight before anything is waited for.  An accumulator holds, in lane
// j + 16 g and register e, feature 4 g + e of row j: the hidden layout's own
// four floats, so the next layer reads what this one stores.
// On one MI355X a forward of the 160-1024-1024-1024-160 policy network over 777
// rows went from 140 to 60 us, over 320 from 72 to 41, over 100 from 34 to 26 and
// over one from 21.5 to 20 (row-major operands on fp32 MFMA before).
//
// Split products (SPLIT): a weight of feature n is held as 2^wexp[n] (w0 + w1),
// two fp16 parts with the feature's largest weight in [2^14, 2^15); an input row
// x as x S = x0 + x1 in fp16 with S = 2^-xexp the power of two that puts the
// row's largest value in [2^14, 2^15).  w0 x0, and w0 x1 + w1 x0 in a sum of
// their own (2^-11 as large, so that their roundings do not count), then keep
// about 22 bits of every product of values within 2^-16 of the largest, and
// 2^-39 of the largest below; w1 x1 is left out.  Every fp16 product is exact in
// the MFMA's fp32 accumulator, and one such chunk of 32 inputs rounds the large sum
// once: against float64 a forward of the policy is 2.5e-7 off, 4.0e-7 with fp32
// MFMA and 3.2e-7 with one sum for all three products, at a fifth of the matrix
// time.  What is left is the split of the weights, which stays the same along
// a chain: with a third part, held exactly, 100-step samples were another 8 %
// closer to float64, for half as much again to load (a forward of 1024 rows 98 us
// for 80).  The row's largest value comes from the producing layer, one maximum
// per row and 16-feature tile (rmax); the first layer takes it from its own loads.
// Layers with few inputs and models with a non-finite weight run on fp32 MFMA.
#pragma once

#include "pd_internal.h"

namespace pd {

constexpr int kLinWaves = 8;              // waves per block, splitting the reduction
constexpr int kLinThreads = kLinWaves * 64;

// GELU(u) = u Phi(u) = max(u, 0) - |u| Q(|u|), Q(t) = erfc(t / sqrt 2) / 2 =
// exp(-t^2 / 2) G(t), with G (a scaled erfcx, smooth and slowly falling) as 1/2
// and a polynomial of degree 8 in w = 0.29 t / (1 + 0.29 t): least squares
// reweighted towards the largest relative error, 3.1e-8 on [0, 6].  One
// reciprocal, one exponential and no branch, where u (1 + erff(u / sqrt 2)) / 2
// took both of erff's branches.  Distance to float64 over normal u of
// deviation 0.3, 1 and 3: 4.0e-8, 2.9e-8 and 2.2e-8, and with erff 4.1e-8, 3.9e-8 and 3.0e-8.
// +inf gives inf, -inf and NaN give NaN (as the product with 1 + erf does).
__device__ __forceinline__ float gelu_exact(float u) {
    const float t = __builtin_fabsf(u > 30.f ? 30.f : u);
    const float w = t * 0.29f * __builtin_amdgcn_rcpf(__builtin_fmaf(t, 0.29f, 1.0f));
    float g = 0.0398590082f;
    g = __builtin_fmaf(g, w, -0.123180827f);
    g = __builtin_fmaf(g, w, 0.0589313836f);
    g = __builtin_fmaf(g, w, 0.160809925f);
    g = __builtin_fmaf(g, w, 0.0255656515f);
    g = __builtin_fmaf(g, w, -0.883300482f);
    g = __builtin_fmaf(g, w, 1.59700807f);
    g = __builtin_fmaf(g, w, -1.37566304f);
    g = __builtin_fmaf(g, w, 0.5f);
    const float e = __builtin_amdgcn_exp2f(t * t * -0.72134752f);   // log2(e) / 2
    return __builtin_fmaf(-t, e * g, u > 0.f ? u : 0.f);
}

// Barrier for LDS traffic only: global loads and stores issued before it may
// still be in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef float lin_f4 __attribute__((ext_vector_type(4)));
typedef _Float16 lin_h8 __attribute__((ext_vector_type(8)));
typedef uint32_t lin_u4 __attribute__((ext_vector_type(4)));

// Row tile mt of a hidden buffer of M rows: rows of the tile (the last tile is
// stored without padding).
__device__ __forceinline__ int tile_rows(int M, int mt) { return min(16, M - 16 * mt); }
// First float of row (16 mt + j)'s run in a hidden buffer of width K; input k
// sits at + (k / 4) tile_rows * 4 + k % 4
__device__ __forceinline__ int64_t hidden_row(int K, int mt, int j) { return (int64_t)mt * 16 * K + 4 * j; }
// Word of the maximum of row j of row tile mt over feature tile nt (NT of
// them): [mt][nt / 4][row][nt % 4]
__device__ __forceinline__ int64_t rmax_word(int NT, int mt, int rows, int nt, int j) {
    return (int64_t)mt * 16 * ((NT + 3) / 4 * 4) + ((int64_t)(nt >> 2) * rows + j) * 4 + (nt & 3);
}

__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }

// LDS of a tile.  The maxima are bits of |x| (unsigned order: NaN above inf
// above every number).
template <int RT, int CT>
struct LinearLds {
    float part[kLinWaves][RT * CT][256];
    uint32_t mx[kLinWaves][16 * RT];
    int xexp[16 * RT];                     // 1 / S = 2^xexp of the tile's rows
    uint32_t pm[RT * CT][4][16];           // maxima of the tile's outputs, per 4 features
};

// One chunk's operands of a lane: inputs 16 q + 4 g + e of each row tile; the
// two 16-byte halves (fp32) or parts (fp16) of each feature tile's weights.
template <int RT, int CT>
struct LinearChunk {
    lin_f4 x[RT][2];
    lin_f4 w[CT][2];
};

struct SplitX {
    lin_h8 x0, x1;
};
__device__ __forceinline__ SplitX split_row(const lin_f4& a, const lin_f4& b, float S, bool nonfinite) {
    lin_u4 p0, p1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float v0 = q < 2 ? a[2 * q] : b[2 * q - 4], v1 = q < 2 ? a[2 * q + 1] : b[2 * q - 3];
        const float h0 = v0 * S, h1 = v1 * S;                 // exact: a power of two
        uint32_t u, w;
        float d0, d1;
        asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(u) : "v"(h0), "v"(h1));
        asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(d0) : "v"(v0), "v"(S), "v"(u));
        asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(d1) : "v"(v1), "v"(S), "v"(u));
        asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(w) : "v"(d0), "v"(d1));
        p0[q] = u;
        p1[q] = w;
    }
    SplitX s;
    s.x0 = __builtin_bit_cast(lin_h8, p0);
    s.x1 = __builtin_bit_cast(lin_h8, p1);
    if (nonfinite) {
        // an infinite or NaN input goes to the second part alone, which meets
        // only the weights' leading parts: its products are those of the value
        // itself (a weight's leading part is zero only where the weight is)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t bits = (p0[i >> 1] >> (16 * (i & 1))) & 0x7fff;
            if (bits >= 0x7c00) {
                s.x1[i] = s.x0[i];
                s.x0[i] = (_Float16)0.f;
            }
        }
    }
    return s;
}

// Where a tile's input rows come from.
enum LinearIn {
    IN_HIDDEN,     // a hidden buffer of Mmax rows
    IN_GATHER,     // the window's ring slots or a [rows][D] batch (the first layer)
    IN_LDS,        // the tile's 16 rows in LDS (the first layer after a scan in the same block)
};
struct TileRows {
    int M, Mmax;               // active rows, and rows of the launch's buffers
    HiddenBuf in;              // IN_HIDDEN
    const RowSrc* src;         // IN_GATHER
    int64_t D;                 // IN_GATHER: values of a row
    const float* x;            // IN_LDS: row j at x + j xs
    int xs;
    const int* n;              // IN_LDS: network timestep of row j
};

// The tile of row tiles mt0.. and feature tiles nt0..; every thread of the
// block calls it, and emit(tile, u) is then called for the block's outputs: u
// the pre-activation of row j = (tid / 4) % 16 and feature 4 g + e, g =
// (tid / 64) % 4, e = tid % 4, of the 16 x 16 block (row tile mt0 + tile / CT,
// feature tile nt0 + tile % CT), which is the same for the whole wave (the row
// or feature may lie past the end: nothing is stored for those).  Returns false, with
// nothing emitted, when no row of the tile is active.  Rows and inputs past the
// end are clamped (to the last active row where rows are gathered, else to the
// last row of the buffer), loaded and count for nothing.
template <int RT, int CT, LinearIn IN, bool SPLIT, class Emit>
__device__ __forceinline__ bool linear_tile(const LinearArgs& a, const TileRows& rows, int mt0, int nt0,
                                            LinearLds<RT, CT>& lds, Emit&& emit) {
    static_assert(RT == 1 || RT == 2, "the row maxima are shared out over 512 threads");
    static_assert(IN != IN_LDS || RT == 1, "one row tile in LDS");
    constexpr bool GATHER = IN == IN_GATHER;
    typedef LinearChunk<RT, CT> Chunk;
    const int tid = threadIdx.x, lane = tid & 63, j = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = rows.M, Mmax = rows.Mmax;
    const int K = a.K, N = a.N, K4 = K / 4;
    const int KC = (K + 31) / 32, NT = (N + 15) / 16;
    // gathered rows need the loop state first: only the active groups' slots
    // are set (past them a slot may never have been written)
    if constexpr (IN != IN_HIDDEN) {
        if (16 * mt0 >= M) return false;                      // uniform over the block
    }
    const int Mread = IN == IN_HIDDEN ? Mmax : M;

    // the input rows' largest values, read first (loads return in order)
    uint32_t mrow = 0;
    if constexpr (SPLIT && IN == IN_HIDDEN) {
        constexpr int PARTS = kLinThreads / (16 * RT);
        const int r = tid % (16 * RT), part = tid / (16 * RT);
        const int row = min(16 * mt0 + r, Mmax - 1), mt = row >> 4;
        const int NTi = (K + 15) / 16, nr = tile_rows(Mmax, mt);
        for (int n4 = part; n4 < (NTi + 3) / 4; n4 += PARTS) {
            const lin_u4 v = *reinterpret_cast<const lin_u4*>(rows.in.rmax + rmax_word(NTi, mt, nr, 4 * n4, row & 15));
#pragma unroll
            for (int e = 0; e < 4; ++e) mrow = umax32(mrow, 4 * n4 + e < NTi ? v[e] : 0u);
        }
    }

    // this lane's row of each row tile; in a hidden buffer the tile (the same
    // pointer in every lane), the bytes from there to the row and those from one of
    // its input groups of four to the next (32 and 24 bits: a width of 2^26 would
    // have weights past any memory)
    const float* xp[RT];
    uint32_t xo[RT], xs[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int row = min(16 * (mt0 + rt) + j, Mread - 1);
        if constexpr (GATHER) {
            const RowSrc& src = *rows.src;
            const int gr = row / src.group, b = row % src.group;
            const int64_t sl = src.slot ? src.slot[gr] : gr;
            xp[rt] = src.base + sl * src.slot_stride + (int64_t)b * rows.D;
        } else if constexpr (IN == IN_LDS) {
            xp[rt] = rows.x + j * rows.xs;
        } else {
            const int mt = min(mt0 + rt, (Mmax - 1) >> 4);    // row / 16, the same in every lane
            xp[rt] = rows.in.h + hidden_row(K, mt, 0);
            xs[rt] = 16u * tile_rows(Mmax, mt);
            xo[rt] = 16u * (row & 15);
        }
    }
    const lin_f4* wp[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
        wp[ct] = static_cast<const lin_f4*>(a.w) + (int64_t)min(nt0 + ct, NT - 1) * KC * 128;

    const int per = (KC + kLinWaves - 1) / kLinWaves;
    const int c_begin = wave * per, c_end = min(c_begin + per, KC);
    auto load = [&](int c) -> Chunk {
        Chunk ch;
        c = min(c, KC - 1);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int q = 0; q < 2; ++q) ch.w[ct][q] = (wp[ct] + (int64_t)c * 128 + q * 64)[(uint32_t)lane];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int k4 = min(8 * c + 4 * q + g, K4 - 1);
                if constexpr (IN == IN_HIDDEN)
                    ch.x[rt][q] = *reinterpret_cast<const lin_f4*>(reinterpret_cast<const char*>(xp[rt]) +
                                                                   (xo[rt] + __umul24(k4, xs[rt])));
                else
                    ch.x[rt][q] = *reinterpret_cast<const lin_f4*>(xp[rt] + 4 * (int64_t)k4);
            }
        return ch;
    };

    // U chunks at a time, in two register sets: at 1024 inputs the small tiles
    // have all four chunks of a wave in flight at once
    constexpr int U = RT + CT <= 3 ? 2 : 1;
    Chunk A[U], B[U];
#pragma unroll
    for (int u = 0; u < U; ++u) A[u] = load(c_begin + u);
#pragma unroll
    for (int u = 0; u < U; ++u) B[u] = load(c_begin + U + u);

    // epilogue operands, fetched before the products
    constexpr int E = (RT * CT * 256 + kLinThreads - 1) / kLinThreads;   // outputs per thread
    float addv[E];
    int wev[E];
    // the 16 x 16 block of a thread's i-th output is the same for its whole
    // wave: kept in scalar registers, with all addresses that follow from it
    const int upper = __builtin_amdgcn_readfirstlane(tid >> 8);
    const int o = tid & 255, oj = (o >> 2) & 15, on = 4 * (o >> 6) + (o & 3);
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int tile = min(2 * i + upper, RT * CT - 1);
        // two feature tiles: the same one for all of a thread's outputs
        const int n = min(16 * (nt0 + (CT == 2 ? upper : tile % CT)) + on, N - 1);
        const int row = min(16 * (mt0 + tile / CT) + oj, Mread - 1);
        if constexpr (GATHER) {
            const int gr = rows.src->group == 1 ? row : row / rows.src->group;
            addv[i] = a.shift[(int64_t)row_timestep(*rows.src, gr) * N + n];
        } else if constexpr (IN == IN_LDS) {
            addv[i] = a.shift[(int64_t)rows.n[row - 16 * mt0] * N + n];
        } else {
            addv[i] = a.bias[n];
        }
        wev[i] = SPLIT ? a.wexp[n] : 0;
    }
    // the loads above stay ahead of this exit (they need no loop state)
    asm volatile("" ::: "memory");
    if (16 * mt0 >= M) return false;                          // uniform over the block

    float S[RT];
    bool nonfinite = false;
    if constexpr (SPLIT) {
        if constexpr (IN != IN_HIDDEN) {
            // this wave's chunks of each row, from the registers that hold the
            // first ones (clamped inputs repeat one of the row)
            uint32_t m[RT];
            auto take = [&](const Chunk& ch) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        m[rt] = umax32(m[rt], __builtin_bit_cast(uint32_t, (float)ch.x[rt][u / 4][u % 4]) & 0x7fffffffu);
            };
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) m[rt] = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) take(A[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) take(B[u]);
            for (int c = c_begin + 2 * U; c < c_end; ++c) take(load(c));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                m[rt] = umax32(m[rt], __shfl_xor(m[rt], 16, 64));
                m[rt] = umax32(m[rt], __shfl_xor(m[rt], 32, 64));
                if (g == 0) lds.mx[wave][16 * rt + j] = m[rt];
            }
        } else {
            if constexpr (RT == 1) mrow = umax32(mrow, __shfl_xor(mrow, 16, 64));
            mrow = umax32(mrow, __shfl_xor(mrow, 32, 64));
            if (lane < 16 * RT) lds.mx[wave][lane] = mrow;
        }
        lds_barrier();
        uint32_t m[RT];
        auto all_waves = [&] {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                m[rt] = lds.mx[0][16 * rt + j];
#pragma unroll
                for (int v = 1; v < kLinWaves; ++v) m[rt] = umax32(m[rt], lds.mx[v][16 * rt + j]);
                // (rows past the active ones may never have been written)
                nonfinite |= m[rt] >= 0x7f800000u && 16 * (mt0 + rt) + j < M;
            }
        };
        all_waves();
        nonfinite = __ballot(nonfinite) != 0;                 // the same in every wave
        if (nonfinite) {
            // rare: the inputs are read once more for the largest finite value
            // of each row, which scales the finite ones beside a non-finite one
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) m[rt] = 0;
            for (int c = c_begin; c < c_end; ++c) {
                const Chunk ch = load(c);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const uint32_t v = __builtin_bit_cast(uint32_t, (float)ch.x[rt][u / 4][u % 4]) & 0x7fffffffu;
                        m[rt] = umax32(m[rt], v < 0x7f800000u ? v : 0u);
                    }
            }
            lds_barrier();                                    // every wave has read the maxima
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                m[rt] = umax32(m[rt], __shfl_xor(m[rt], 16, 64));
                m[rt] = umax32(m[rt], __shfl_xor(m[rt], 32, 64));
                if (g == 0) lds.mx[wave][16 * rt + j] = m[rt];
            }
            lds_barrier();
            all_waves();
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            // S = 2^(14 - e), e the exponent of the largest finite value; a row
            // of zeros takes 1
            int e = m[rt] > 0 ? (int)(m[rt] >> 23) - 127 : 14;
            e = e < -112 ? -112 : e;                          // S at most 2^126
            S[rt] = __builtin_bit_cast(float, (uint32_t)(14 - e + 127) << 23);
            if (wave == 0 && g == 0) lds.xexp[16 * rt + j] = e - 14;
        }
    }

    // split: the two small products have accumulators of their own (acl)
    lin_f4 acc[RT][CT], acl[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = acl[rt][ct] = lin_f4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](Chunk& ch, int c) {
        if (8 * c + 8 > K4) {                                 // inputs past K (the last chunk of a ragged K)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (8 * c + 4 * q + g >= K4)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) ch.x[rt][q] = lin_f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if constexpr (SPLIT) {
                const SplitX s = split_row(ch.x[rt][0], ch.x[rt][1], S[rt], nonfinite);
#pragma unroll
                for (int p = 0; p < 3; ++p)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        // the main product between the two small ones, so that
                        // none waits for the one before
                        lin_f4& to = p == 1 ? acc[rt][ct] : acl[rt][ct];
                        to = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(lin_h8, ch.w[ct][p == 2 ? 1 : 0]),
                                                                    p == 0 ? s.x1 : s.x0, to, 0, 0, 0);
                    }
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(ch.w[ct][u / 4][u % 4], ch.x[rt][u / 4][u % 4],
                                                                           acc[rt][ct], 0, 0, 0);
            }
        }
    };
    for (int c = c_begin; c < c_end; c += 2 * U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c + u < c_end) compute(A[u], c + u);
            if (c + 2 * U + u < c_end) A[u] = load(c + 2 * U + u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c + U + u < c_end) compute(B[u], c + U + u);
            if (c + 3 * U + u < c_end) B[u] = load(c + 3 * U + u);
        }
    }

    // partial tiles, 1 KB per wave and 16 x 16 block: conflict-free 16-byte
    // writes and 4-byte reads
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
            *reinterpret_cast<lin_f4*>(&lds.part[wave][rt * CT + ct][4 * lane]) =
                SPLIT ? acc[rt][ct] + acl[rt][ct] : acc[rt][ct];
    lds_barrier();
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const int tile = 2 * i + upper;
        if (tile < RT * CT) {                                 // uniform over the wave
            float sum = lds.part[0][tile][o];
#pragma unroll
            for (int v = 1; v < kLinWaves; ++v) sum += lds.part[v][tile][o];
            // both scales at once: one of them alone may leave the float range
            if constexpr (SPLIT) sum = __builtin_ldexpf(sum, lds.xexp[16 * (tile / CT) + oj] + wev[i]);
            emit(tile, sum + addv[i]);
        }
    }
    return true;
}

// A hidden layer's tile: GELU into the next layer's input layout, and the
// maximum of each row over each 16-feature tile.
template <int RT, int CT, LinearIn IN, bool SPLIT>
__device__ __forceinline__ void hidden_tile(const LinearArgs& a, const TileRows& in, const HiddenBuf& out, int mt0,
                                            int nt0, LinearLds<RT, CT>& lds) {
    const int M = in.M, N = a.N;
    const int j = (threadIdx.x >> 2) & 15, g = (threadIdx.x >> 6) & 3, e = threadIdx.x & 3;
    const bool any = linear_tile<RT, CT, IN, SPLIT>(a, in, mt0, nt0, lds, [&](int tile, float u) {
        const float v = gelu_exact(u);
        const int mt = mt0 + tile / CT, nt = nt0 + tile % CT, rows = tile_rows(in.Mmax, mt);
        const bool valid = j < M - 16 * mt && 4 * g + e < N - 16 * nt;
        if (valid) (out.h + hidden_row(N, mt, 0) + (int64_t)nt * 16 * rows)[(g * rows + j) * 4 + e] = v;
        // largest of the quad's four features
        uint32_t m = valid ? __builtin_bit_cast(uint32_t, v) & 0x7fffffffu : 0u;
        m = umax32(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xb1, 0xf, 0xf, false));
        m = umax32(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4e, 0xf, 0xf, false));
        if (e == 0) lds.pm[tile][g][j] = m;
    });
    if (!any) return;
    lds_barrier();
    const int NT = (N + 15) / 16;
    for (int i = threadIdx.x; i < RT * CT * 16; i += kLinThreads) {
        const int tile = i >> 4, r = i & 15;
        const int mt = mt0 + tile / CT, nt = nt0 + tile % CT;
        if (16 * mt + r < M && nt < NT) {
            const uint32_t m = umax32(umax32(lds.pm[tile][0][r], lds.pm[tile][1][r]),
                                      umax32(lds.pm[tile][2][r], lds.pm[tile][3][r]));
            out.rmax[rmax_word(NT, mt, tile_rows(in.Mmax, mt), nt, r)] = m;
        }
    }
}

}  // namespace pd
