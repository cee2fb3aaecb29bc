// Picard update, error check and window slide of Algorithm 1 on the device.
//
// The window x_t .. x_{t+p} lives in a ring of p+1 trajectory slots,
// slot(m) = m mod (p+1) (p+2 for the multistep drift, which also keeps
// x_{t-1}).  The frontier f is the highest index that holds a computed
// point; every point past f equals x_f (the new points of Algorithm 1 are
// copies of the window's last point), so they are read from slot(f) and
// never copied.  The loop state (t, k, f, p_eff) stays on the device: the
// finalize step of one iteration writes the row descriptors (ring slot and
// network timestep of every window point) that the next iteration's denoiser
// and scan read, so no host round trip is needed between iterations; it also
// copies the state into mapped host memory for the host's batch decisions.
#include <type_traits>

#include "eps_out.h"
#include "linear_tile.h"
#include "pd_internal.h"

namespace pd {
namespace {

// Waves per scan block, split along the window: 8 for windows of up to 64
// points, 16 above (up to 8 rows per wave, so windows up to 128 points).  At
// 64 points and 4 x 4 x 96 x 96 columns, 8 waves of 8 rows took 20.8 us per
// launch against 25.3 us for 16 waves of 4; 16 rows per wave spill.
constexpr int kScanMaxRows = 8;
constexpr int kMaxWindow = 16 * kScanMaxRows;

// Columns per lane of the scan: four (one 16-byte access per row) when the
// sample size allows it, else one.
inline int scan_vec(int64_t D) { return D % 4 == 0 ? 4 : 1; }

template <int VEC>
struct Cols;
template <>
struct Cols<1> {
    typedef float type;
    typedef double sum;
};
template <>
struct Cols<4> {
    typedef float type __attribute__((ext_vector_type(4)));
    typedef double sum __attribute__((ext_vector_type(4)));
};
template <int VEC>
__device__ __forceinline__ float& col_at(typename Cols<VEC>::type& v, int c) {
    if constexpr (VEC == 1) return v;
    else return reinterpret_cast<float*>(&v)[c];
}
template <int VEC>
__device__ __forceinline__ double& sum_at(typename Cols<VEC>::sum& v, int c) {
    if constexpr (VEC == 1) return v;
    else return reinterpret_cast<double*>(&v)[c];
}
template <int VEC>
__device__ __forceinline__ float col_at(const typename Cols<VEC>::type& v, int c) {
    if constexpr (VEC == 1) return v;
    else return v[c];
}

// Sum over aligned groups of N lanes (N a power of two <= 64); every lane of
// a group ends with the group's sum.  Groups up to 16 lanes reduce with DPP
// lane moves inside a row (quad swaps, then the 8- and 16-lane mirrors), with
// no LDS traffic; wider groups finish with a cross-row shuffle.
template <int N>
__device__ __forceinline__ float group_sum(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                             0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                             0xF, 0xF, false));
    };
    if constexpr (N >= 2) v += dpp(v, std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
    if constexpr (N >= 4) v += dpp(v, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
    if constexpr (N >= 8) v += dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
    if constexpr (N >= 16) v += dpp(v, std::integral_constant<int, 0x140>{}); // row_mirror
    if constexpr (N >= 32) v += __shfl_xor(v, 16, 64);
    if constexpr (N >= 64) v += __shfl_xor(v, 32, 64);
    return v;
}

// Heun's method, window side (rows j < p_eff of the current window):
// predict:  xt[j] = x_{t+j} + (A x_{t+j} + B eps[j])      (the Euler step)
// The scan then takes (eps[j] + eps2[j]) / 2 in place of eps[j] for every step
// but the last, so that its A x + B eps is A x + (B / 2)(eps + eps2) rounded
// exactly as written (halving is exact).
__global__ __launch_bounds__(256) void k_heun_predict(const LoopState* __restrict__ st,
                                                      const float* __restrict__ ring,
                                                      const float* __restrict__ eps,
                                                      const float* __restrict__ Atab,
                                                      const float* __restrict__ Btab, int p,
                                                      int64_t BD, float* __restrict__ xt) {
    const int pe = st->p_eff;
    const int t = st->t, f = st->f, P1 = p + 1;
    const int64_t n = (int64_t)pe * BD;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(i / BD);
        const int64_t c = i - (int64_t)j * BD;
        const int m = t + j;
        const float x = ring[(int64_t)((m <= f ? m : f) % P1) * BD + c];
        xt[i] = __fadd_rn(x, drift(Atab[m], x, Btab[m], eps[i]));
    }
}

// The sequential sampler's step apart from the denoiser: a run with timed
// launches reports the two by themselves.
__global__ __launch_bounds__(256) void k_eps_step(EpsOut out, const float* __restrict__ eps, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        eps_out(out, i, eps[i]);
}

// The stride is known: record it, slide the window and write the next
// iteration's row descriptors.  cur is the loop state as the iteration found
// it.  mt / mt2 (or nullptr: read the tables) hold model_t[t + i] /
// model_t_next[t + i] for i < 2p, which covers every index read here (the
// next window starts at t + stride <= t + p_eff).  Thread 0 rewrites the loop
// state.
__device__ void slide_window(const FinalizeArgs& a, int stride, int bad, const LoopState& cur,
                             const int* mt, const int* mt2) {
    LoopState* st = a.st;
    const int p = a.p, T = a.T;
    const int t = cur.t, k = cur.k, pe = cur.p_eff, rows_now = cur.nrows;
    const int fn = t + pe, tn = t + stride;
    const int pn = bad ? 0 : (p < T - tn ? p : T - tn);
    auto model_t = [&](int m) { return mt ? mt[m - t] : a.model_t[m]; };
    auto model_t_next = [&](int m) { return mt2 ? mt2[m - t] : a.model_t_next[m]; };
    // next batch: [the point before the window, for the multistep drift] then
    // the window's points
    const int hn = (a.history && tn >= 1 && pn > 0) ? 1 : 0;
    if (threadIdx.x == 0) {
        a.trace[k] = stride;
        LoopState v = cur;
        if (k == 0) v.first_stride = stride;
        v.k = k + 1;
        // network evaluations: Heun evaluates twice per point but the last
        // step; with a history row the batch had one row more than the window
        v.evals += a.nrow2 ? 2 * pe - (t + pe == T ? 1 : 0) : rows_now;
        v.f = fn;
        v.t = bad ? T : tn;
        v.p_eff = pn > 0 ? pn : 0;
        if (bad) v.status = PD_ERR_NUMERIC;
        v.nrows = pn > 0 ? pn + hn : 0;
        *st = v;
        if (hn) {
            a.slot[0] = (tn - 1) % a.ring_slots;     // tn - 1 < fn: a computed point
            a.nrow[0] = model_t(tn - 1);
        }
        mirror_state(v, a.st_host);
    }
    for (int j = threadIdx.x; j < pn; j += blockDim.x) {
        const int m = tn + j;
        a.slot[hn + j] = (m < fn ? m : fn) % a.ring_slots;
        a.nrow[hn + j] = model_t(m);
        if (a.nrow2) a.nrow2[j] = model_t_next(m);
    }
}

// The iteration that reaches T copies x_T out, so the host needs no copy launch:
// its new points are this block's own stores (waited for here) or were made
// visible to it by kernel order.  The condition is uniform over the block.
__device__ void finalize_apply(const FinalizeArgs& a, int stride, int bad, const LoopState& cur, const int* mt,
                               const int* mt2) {
    slide_window(a, stride, bad, cur, mt, mt2);
    if (!bad && cur.t + stride >= a.T) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        for (int64_t i = threadIdx.x; i < a.BD; i += blockDim.x) a.x_out[i] = a.xT[i];
    }
}

// Tolerance of window offset o >= 1 (Algorithm 1's stride test compares the
// error with it; sigma^2 = 0 allows no change at all).
__device__ __forceinline__ float offset_tol(const FinalizeArgs& a, int t, int o) {
    const float s2 = a.tol_var[t + o + a.tol_offset];
    return (s2 == 0.f) ? 0.f : a.tau2 * s2;
}

// One block: reduce the partials of every (offset, sample), apply the stride
// rule, slide the window and prepare the next iteration's row descriptors.
// cur is the loop state as the iteration found it; thread 0 rewrites it at
// the end.
__device__ void finalize_body(const FinalizeArgs& a, int nblk, const LoopState& cur) {
    const int pe = cur.p_eff;
    if (pe <= 0) return;
    const int t = cur.t, p = a.p;
    __shared__ int s_stride, s_bad;
    if (threadIdx.x == 0) {
        s_stride = pe;
        s_bad = 0;
    }
    __syncthreads();
    constexpr int kTeam = 16;
    const int team = threadIdx.x / kTeam, tl = threadIdx.x % kTeam;
    const int nteams = blockDim.x / kTeam;
    for (int pair = team; pair < pe * a.batch; pair += nteams) {
        const int o = pair / a.batch, b = pair % a.batch;
        const float tol = o >= 1 ? offset_tol(a, t, o) : 0.f;    // in flight with the sums
        const float* src = a.partials + ((int64_t)b * p + o) * nblk;
        // 8 independent loads per step keep the team's reads in flight together
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int i0 = 0; i0 < nblk; i0 += 8 * kTeam) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + u * kTeam + tl;
                acc[u] += i < nblk ? src[i] : 0.f;
            }
        }
        float s = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
        s = group_sum<kTeam>(s);
        bool fails = false, bad = false;
        if (tl == 0) {
            if (o == 0) {
                bad = s != 0.f;
            } else {
                const float err = s / a.err_div;
                bad = !isfinite(err);
                fails = !(err <= tol);
            }
        }
        // lanes hold pairs in increasing order: the wave's first failing
        // lane has its smallest failing offset, and one lane per wave votes
        const uint64_t fm = __ballot(fails), bm = __ballot(bad);
        const int lane = threadIdx.x & 63;
        if (fm && lane == __ffsll((unsigned long long)fm) - 1) atomicMin(&s_stride, o);
        if (bm && lane == __ffsll((unsigned long long)bm) - 1) atomicOr(&s_bad, 1);
    }
    __syncthreads();
    finalize_apply(a, s_stride, s_bad, cur, nullptr, nullptr);
}

// The finalize step of a multi-block scan (kernel order makes every block's
// partials visible to it).
__global__ __launch_bounds__(1024) void k_picard_finalize(FinalizeArgs a, int nblk) {
    const LoopState cur = *a.st;
    finalize_body(a, nblk, cur);
}

// One block: cpb <= 64 * VEC consecutive columns of one sample b (a multiple
// of VEC, from picard_scan_cols), all window rows,
// split over NW waves (rows [w*ch, (w+1)*ch) per wave, ch <= R).  Each row's
// drift plus noise is summed along the rows inside each wave, the wave totals are
// exchanged through LDS, and the new points x^{k+1}_{t+j+1} = x_t + sum (y + z)
// are written back to the ring, rounded once each from x_t and the totals of the
// waves before, in double, plus the wave's own sum: 16 policy samples of 100 steps
// are 1.00e-7 from float64, 1.28e-7 with sums of drift and noise of their own in
// float32, at the same time.  All loads use clamped, always-valid
// indices and no branches, so a wave's rows are in flight together; the drift
// coefficients of a wave's rows come in one vector load and are broadcast
// with readlane.  The squared differences against the old points are summed
// per lane over its columns, transposed through LDS and reduced per window
// offset into per-block partial sums partials[b][o][blk]; offset 0 (never
// tested) carries the count of non-finite points in the window's last row
// (a non-finite point in any other row makes its error non-finite).  With
// DPM, a second-order step's drift also adds R x_{i-1} + S eps_{i-1}: the
// previous row's point and epsilon, or for a wave's first row the ones
// before it (for the window's first row, the history row x_{t-1} that the
// batch evaluated first).
template <int NW, int R, int VEC, bool NOISE, bool DPM>
__global__ __launch_bounds__(NW * 64) void k_picard_scan(
    const LoopState* __restrict__ st, float* ring, const float* __restrict__ eps,
    const float* __restrict__ noise, const float* __restrict__ Atab,
    const float* __restrict__ Btab, const float* __restrict__ Rtab,
    const float* __restrict__ Stab, int p, int batch, int64_t D, float* __restrict__ partials,
    FinalizeArgs fin, int fuse_finalize, int cpb, const float* __restrict__ eps2) {
    typedef typename Cols<VEC>::type V;
    const LoopState cur = *st;
    const int pe = cur.p_eff;
    if (pe <= 0) return;
    const int t = cur.t, f = cur.f;
    // the wave index is uniform: keep it (and every row index derived from
    // it) in scalar registers
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y, blk = blockIdx.x, nblk = gridDim.x;
    // lane l covers columns [blk cpb + l VEC, + VEC) of the block's cpb (D and
    // cpb are multiples of VEC)
    const int64_t d = (int64_t)blk * cpb + (int64_t)lane * VEC;
    const bool valid = lane * VEC < cpb && d < D;
    const int64_t slotsz = (int64_t)batch * D;
    const int64_t col = (int64_t)b * D + (valid ? d : 0);
    const int P1 = fin.ring_slots;
    // DPM-Solver: eps row 0 holds the point before the window (once t >= 1)
    const int hist = DPM ? cur.nrows - pe : 0;
    const int ch = (pe + NW - 1) / NW;
    const int j0 = min(w * ch, pe), j1 = min(j0 + ch, pe);
    const int nr = j1 - j0;

    // a single-block grid finalizes the iteration itself, from LDS: its
    // tolerances and the timesteps of the next window are fetched now, with
    // the window's data
    __shared__ int s_mt[2 * kMaxWindow], s_mt2[2 * kMaxWindow];
    __shared__ float s_err[kMaxWindow];
    float ftol = 0.f;
    int mt_i = 0, mt2_i = 0;   // stored to LDS once the window's loads have arrived
    const bool has_mt = fuse_finalize && (int)threadIdx.x < 2 * p && t + (int)threadIdx.x < fin.T;
    if (fuse_finalize) {
        const int i = threadIdx.x;
        if (i >= 1 && i < pe) ftol = offset_tol(fin, t, i);
        if (has_mt) {
            mt_i = fin.model_t[t + i];
            if (fin.nrow2) mt2_i = fin.model_t_next[t + i];
        }
    }

    // wave totals and first old points, then (after a barrier) the
    // per-row squared differences of every lane
    __shared__ union {
        struct {
            V tot[NW][64];
            V first[NW][64];
        } x;
        float d2[NW * R][65];
    } sh;

    // ---- every read of this block's ring columns is consumed before the
    // first barrier; the writes all come after it (the ring slots overlap).
    const V anchor = *reinterpret_cast<const V*>(ring + (int64_t)(t % P1) * slotsz + col);
    const int slot_f = f % P1;
    const int jt = min(j0 + (lane < R ? lane : R - 1), pe - 1);   // lane r: row j0 + r
    const float ta = Atab[t + jt], tb = Btab[t + jt];
    float tr = 0.f, ts = 0.f;
    V xp = V(0.f), ep = V(0.f);   // DPM-Solver: x and eps of the step before row j0
    if constexpr (DPM) {
        tr = Rtab[t + jt];
        ts = Stab[t + jt];
        const int mp = max(t + j0 - 1, 0);           // clamped (step 0 is first order)
        xp = *reinterpret_cast<const V*>(ring + (int64_t)(mp <= f ? mp % P1 : slot_f) * slotsz + col);
        ep = *reinterpret_cast<const V*>(eps + (int64_t)max(j0 - 1 + hist, 0) * slotsz + col);
    }
    V xo[R], y[R], z[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = min(j0 + r, pe - 1);            // clamped: always a window row
        const int m = t + j;
        const int sl = m <= f ? m % P1 : slot_f;      // points past f equal x_f
        xo[r] = *reinterpret_cast<const V*>(ring + (int64_t)sl * slotsz + col);
        y[r] = *reinterpret_cast<const V*>(eps + (int64_t)(j + hist) * slotsz + col);
        if (eps2 != nullptr && m + 1 < fin.T) {
            // Heun: the mean of the two evaluations, for every step but the
            // chain's last (which keeps its Euler drift)
            const V e2 = *reinterpret_cast<const V*>(eps2 + (int64_t)j * slotsz + col);
#pragma unroll
            for (int c = 0; c < VEC; ++c)
                col_at<VEC>(y[r], c) = __fmul_rn(__fadd_rn(col_at<VEC>(y[r], c), col_at<VEC>(e2, c)), 0.5f);
        }
        if constexpr (NOISE) z[r] = *reinterpret_cast<const V*>(noise + (int64_t)m * slotsz + col);
    }
    // steps (drift and noise) replace eps in y; rows past the wave's range count
    // as zero
    V acc_y = V(0.f);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float ca = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ta), r));
        const float cb = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tb), r));
        const bool in = r < nr;
        float cr = 0.f, cs = 0.f;
        if constexpr (DPM) {
            cr = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tr), r));
            cs = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ts), r));
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const float e = col_at<VEC>(y[r], c);
            float v = drift(ca, col_at<VEC>(xo[r], c), cb, e);
            if constexpr (DPM) {
                // second-order steps add R x_{m-1} + S eps_{m-1}, in that order
                const float v2 = __fadd_rn(__fadd_rn(v, __fmul_rn(cr, col_at<VEC>(xp, c))),
                                           __fmul_rn(cs, col_at<VEC>(ep, c)));
                v = cr != 0.f ? v2 : v;
                col_at<VEC>(xp, c) = col_at<VEC>(xo[r], c);
                col_at<VEC>(ep, c) = e;
            }
            if constexpr (NOISE) v = __fadd_rn(v, col_at<VEC>(z[r], c));
            col_at<VEC>(y[r], c) = in ? v : 0.f;
            col_at<VEC>(acc_y, c) = __fadd_rn(col_at<VEC>(acc_y, c), col_at<VEC>(y[r], c));
        }
    }
    sh.x.tot[w][lane] = acc_y;
    sh.x.first[w][lane] = xo[0];   // x^k_{t+j0}: the previous wave's old point past its range
    if (has_mt) {
        s_mt[threadIdx.x] = mt_i;
        s_mt2[threadIdx.x] = mt2_i;
    }
    // every ring value this wave read has been consumed above, so the ring
    // writes after the next barrier cannot overtake a read
    lds_barrier();
    // the point this wave's rows start from, in double: x_t and the totals of the
    // waves before it, four at a time in flight
    typename Cols<VEC>::sum from;
#pragma unroll
    for (int c = 0; c < VEC; ++c) sum_at<VEC>(from, c) = (double)col_at<VEC>(anchor, c);
    for (int v0 = 0; v0 < w; v0 += 4) {
        V a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = sh.x.tot[min(v0 + u, NW - 1)][lane];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (v0 + u >= w) break;
#pragma unroll
            for (int c = 0; c < VEC; ++c) sum_at<VEC>(from, c) += (double)col_at<VEC>(a[u], c);
        }
    }
    const V next_old = (w + 1 < NW) ? sh.x.first[w + 1][lane] : V(0.f);
    lds_barrier();

    // ---- new points, their squared differences, and the writes
    V sy = V(0.f);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r;
        const bool in = r < nr;
        // error of window offset o = j + 1: x^{k+1}_{t+j+1} against x^k_{t+j+1}
        const V xold = (r + 1 < R && r + 1 < nr) ? xo[r + 1 < R ? r + 1 : r] : next_old;
        V xn;
        float acc = 0.f;
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            col_at<VEC>(sy, c) = __fadd_rn(col_at<VEC>(sy, c), col_at<VEC>(y[r], c));
            const float v = (float)(sum_at<VEC>(from, c) + (double)col_at<VEC>(sy, c));
            col_at<VEC>(xn, c) = v;
            if (j + 1 < pe) {
                const float dl = __fsub_rn(v, col_at<VEC>(xold, c));
                acc += dl * dl;
            } else {
                acc += isfinite(v) ? 0.f : 1.f;     // last row: count non-finite points
            }
        }
        if (in && valid) *reinterpret_cast<V*>(ring + (int64_t)((t + j + 1) % P1) * slotsz + col) = xn;
        sh.d2[w * R + r][lane] = (in && valid) ? acc : 0.f;
    }
    lds_barrier();
    // row q of the NW * R (wave, row) pairs is summed by 64 / R threads
    constexpr int TPR = 64 / R;
    const int q = threadIdx.x / TPR, part = threadIdx.x % TPR;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 64 / TPR; ++i) s += sh.d2[q][part + TPR * i];
    s = group_sum<TPR>(s);
    const int qw = q / R, qr = q % R;
    const int q0 = min(qw * ch, pe), nq = min(q0 + ch, pe) - q0;
    if (!fuse_finalize) {
        if (part == 0 && qr < nq) {
            const int jq = q0 + qr;
            partials[((int64_t)b * p + (jq + 1 < pe ? jq + 1 : 0)) * nblk + blk] = s;
        }
        return;     // the finalize step follows as its own launch
    }
    // one block, one sample: the sums are the errors' numerators; the stride
    // test and the slide follow here (the same arithmetic as the separate
    // finalize step, whose sum over one partial is that partial)
    if (part == 0 && qr < nq) {
        const int jq = q0 + qr;
        s_err[jq + 1 < pe ? jq + 1 : 0] = s;
    }
    lds_barrier();
    // thread o tests offset o; each wave records its first failing offset
    __shared__ int s_wfail[NW], s_wbad[NW];
    {
        const int o = threadIdx.x;
        bool fails = false, bad = false;
        if (o == 0) {
            bad = s_err[0] != 0.f;
        } else if (o < pe) {
            const float err = s_err[o] / fin.err_div;
            bad = !isfinite(err);
            fails = !(err <= ftol);
        }
        const uint64_t fm = __ballot(fails), bm = __ballot(bad);
        if (lane == 0) {
            s_wfail[w] = fm ? w * 64 + __ffsll((unsigned long long)fm) - 1 : pe;
            s_wbad[w] = bm != 0;
        }
    }
    lds_barrier();
    int stride = pe, bad = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        stride = min(stride, s_wfail[v]);
        bad |= s_wbad[v];
    }
    finalize_apply(fin, stride, bad, cur, s_mt, fin.nrow2 ? s_mt2 : nullptr);
}


// The scan, stride and slide of one sample's window, and the first layer of the
// next iteration, in one launch: every block of the first layer's grid works out
// the whole update for itself (the same additions in the same order, so the
// same stride), and takes its 16 rows of the new window from its own registers.
// Nothing is exchanged between blocks: the old window and the loop state are
// read from one pair of buffers and the new ones written to the other, each
// block storing its share of the new points and the first one the rest.  Each
// block reads the whole window, epsilon and noise: with 224 blocks (100 points of
// 160, width 1024) 43 MB go through the caches an iteration, which is free where
// nothing else runs and is taken from other streams where something does.
//
// Bound by latency, as the launches it replaces were: two round trips for the
// loop state and the window (at most 96 points of 256 values, 192 KB at 100
// points of 160), a few barriers, and the tile.  At 100 points of 160 and width
// 1024 it takes 11.6 us, apart 8.2 and 5.7 and a launch gap of about 1; at 15
// points 7.9, apart 4.2 and 4.9 and the gap.
//
// Threads: C4 = D / 4 column groups of four by row groups of ch consecutive
// window rows (at least four, so that few totals are added up).  The points are
// rounded as in the scan, from the totals of other row groups: 100-step policy
// samples are 0.85e-7 from float64, 1.04e-7 with float32 sums, at the same time.
constexpr int kFusedRows = 128, kFusedCols = 256;
template <int CT, int R, bool NOISE, bool DPM>
__global__ __launch_bounds__(kLinThreads) void k_scan_first(ScanFirstArgs s, FinalizeArgs fin, LinearArgs l1,
                                                            HiddenBuf out) {
    typedef Cols<4>::type V;
    __shared__ LinearLds<1, CT> lds;
    __shared__ V s_ty[kLinThreads];
    __shared__ float s_d2[kFusedRows][kFusedCols / 4 + 1];
    __shared__ __attribute__((aligned(16))) float s_x[16][kFusedCols + 4];
    __shared__ float s_A[kFusedRows], s_B[kFusedRows], s_R[kFusedRows], s_S[kFusedRows], s_err[kFusedRows];
    __shared__ int s_mt[2 * kFusedRows], s_mt2[2 * kFusedRows], s_n[16];
    __shared__ int s_wfail[kLinWaves], s_wbad[kLinWaves];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bid = blockIdx.x + gridDim.x * blockIdx.y, nb = gridDim.x * gridDim.y;
    const LoopState cur = *s.st;
    const int pe = cur.p_eff;
    if (pe <= 0) {                                   // the loop has ended: pass its state on
        if (bid == 0 && tid == 0) *fin.st = cur;
        return;
    }
    const int t = cur.t, f = cur.f, P1 = fin.ring_slots, T = fin.T;
    const int D = (int)s.D, C4 = D / 4;
    const int groups = kLinThreads / C4;
    int ch = (pe + groups - 1) / groups;             // <= R: the launch covers a full window
    ch = ch < 4 ? 4 : ch;
    const int rg = tid / C4, col = 4 * (tid - rg * C4);
    const int j0 = min(rg * ch, pe), nr = rg < groups ? min(j0 + ch, pe) - j0 : 0;
    const int hist = DPM ? cur.nrows - pe : 0;
    // ring slots by wrapping additions from x_t's
    const int slot_t = t % P1;
    auto slot_at = [&](int o) {                      // slot of point t + o, 0 <= o < P1
        const int v = slot_t + o;
        return v >= P1 ? v - P1 : v;
    };
    auto old_point = [&](int j) {                    // window row j: points past f equal x_f
        return *reinterpret_cast<const V*>(s.ring_in + (int64_t)slot_at(min(j, f - t)) * D + col);
    };

    // ---- the window, every load in flight together
    V anchor = V(0.f), xnext = V(0.f), xp = V(0.f), ep = V(0.f);
    V xo[R], y[R], z[R], e2[R];
    if (nr > 0) {
        anchor = old_point(0);
        xnext = old_point(min(j0 + nr, pe - 1));
        if constexpr (DPM) {
            // the step before row j0 (for the window's first row x_{t-1}; at t = 0
            // there is none and its coefficients are zero)
            const int o = t + j0 > 0 ? j0 - 1 : 0;
            const int sl = o < 0 ? (slot_t == 0 ? P1 - 1 : slot_t - 1) : slot_at(min(o, f - t));
            xp = *reinterpret_cast<const V*>(s.ring_in + (int64_t)sl * D + col);
            ep = *reinterpret_cast<const V*>(s.eps + (int64_t)max(j0 - 1 + hist, 0) * D + col);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r < ch) {                            // uniform
                const int j = min(j0 + r, pe - 1);
                xo[r] = old_point(j);
                y[r] = *reinterpret_cast<const V*>(s.eps + (int64_t)(j + hist) * D + col);
                if (s.eps2 != nullptr) e2[r] = *reinterpret_cast<const V*>(s.eps2 + (int64_t)j * D + col);
                if constexpr (NOISE) z[r] = *reinterpret_cast<const V*>(s.noise + (int64_t)(t + j) * D + col);
            }
        }
    }
    // the tile's weights are brought near while the scan runs
    lin_f4 warm[2 * CT];
#pragma unroll
    for (int i = 0; i < 2 * CT; ++i) {
        const int KC = (l1.K + 31) / 32, NT = (l1.N + 15) / 16;
        const int nt = min((int)blockIdx.x * CT + i / 2, NT - 1);
        warm[i] = static_cast<const lin_f4*>(l1.w)[((int64_t)nt * KC + min(w, KC - 1)) * 128 + (i & 1) * 64 + lane];
    }
    float ftol = 0.f;
    if (tid < pe) {
        s_A[tid] = s.A[t + tid];
        s_B[tid] = s.B[t + tid];
        if constexpr (DPM) {
            s_R[tid] = s.R[t + tid];
            s_S[tid] = s.S[t + tid];
        }
        if (tid >= 1) ftol = offset_tol(fin, t, tid);
    }
    if (tid < 2 * fin.p && t + tid < T) {
        s_mt[tid] = fin.model_t[t + tid];
        if (fin.nrow2) s_mt2[tid] = fin.model_t_next[t + tid];
    }
    lds_barrier();

    // ---- steps (drift and noise) replace eps in y; each thread's total
    V ty = V(0.f);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r < nr) {
            const int j = j0 + r;
            const float ca = s_A[j], cb = s_B[j];
            float cr = 0.f, cs = 0.f;
            if constexpr (DPM) {
                cr = s_R[j];
                cs = s_S[j];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // Heun: the mean of the two evaluations but at the chain's last step
                if (s.eps2 != nullptr && t + j + 1 < T) y[r][c] = __fmul_rn(__fadd_rn(y[r][c], e2[r][c]), 0.5f);
                const float e = y[r][c];
                float v = drift(ca, xo[r][c], cb, e);
                if constexpr (DPM) {
                    const float v2 = __fadd_rn(__fadd_rn(v, __fmul_rn(cr, xp[c])), __fmul_rn(cs, ep[c]));
                    v = cr != 0.f ? v2 : v;
                    xp[c] = xo[r][c];
                    ep[c] = e;
                }
                if constexpr (NOISE) v = __fadd_rn(v, z[r][c]);
                y[r][c] = v;
                ty[c] = __fadd_rn(ty[c], v);
            }
        }
    }
    s_ty[tid] = ty;
    lds_barrier();
    // the point this thread's rows start from, in double: x_t and the totals of
    // the rows before, four at a time in flight
    Cols<4>::sum from;
#pragma unroll
    for (int c = 0; c < 4; ++c) from[c] = (double)anchor[c];
    if (nr > 0)
        for (int v0 = 0; v0 < rg; v0 += 4) {
            V a4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) a4[u] = s_ty[min(v0 + u, rg) * C4 + col / 4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (v0 + u < rg)
#pragma unroll
                    for (int c = 0; c < 4; ++c) from[c] += (double)a4[u][c];
        }

    // ---- new points (in y) and their squared differences
    V sy = V(0.f);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r < nr) {
            const int j = j0 + r;
            const V xold = (r + 1 < R && r + 1 < nr) ? xo[r + 1 < R ? r + 1 : r] : xnext;
            float acc = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                sy[c] = __fadd_rn(sy[c], y[r][c]);
                const float v = (float)(from[c] + (double)sy[c]);
                y[r][c] = v;
                if (j + 1 < pe) {
                    const float dl = __fsub_rn(v, xold[c]);
                    acc += dl * dl;
                } else {
                    acc += isfinite(v) ? 0.f : 1.f;  // last row: count non-finite points
                }
            }
            s_d2[j][col / 4] = acc;
        }
    }
    lds_barrier();
    {
        const int q = tid >> 2, part = tid & 3;      // four threads a row
        float sum = 0.f;
        if (q < pe)
            for (int i = part; i < C4; i += 4) sum += s_d2[q][i];
        sum = group_sum<4>(sum);
        if (part == 0 && q < pe) s_err[q + 1 < pe ? q + 1 : 0] = sum;
    }
    lds_barrier();
    {
        bool fails = false, bad = false;
        if (tid == 0) {
            bad = s_err[0] != 0.f;
        } else if (tid < pe) {
            const float err = s_err[tid] / fin.err_div;
            bad = !isfinite(err);
            fails = !(err <= ftol);
        }
        const uint64_t fm = __ballot(fails), bm = __ballot(bad);
        if (lane == 0) {
            s_wfail[w] = fm ? w * 64 + __ffsll((unsigned long long)fm) - 1 : pe;
            s_wbad[w] = bm != 0;
        }
    }
    lds_barrier();
    int stride = pe, bad = 0;
#pragma unroll
    for (int v = 0; v < kLinWaves; ++v) {
        stride = min(stride, s_wfail[v]);
        bad |= s_wbad[v];
    }

    // ---- the new window: rows i are points first + i (the history row first)
    const int tn = t + stride;
    const int pn = bad ? 0 : min(fin.p, T - tn);
    const int hn = (DPM && tn >= 1 && pn > 0) ? 1 : 0;
    const int M = pn > 0 ? pn + hn : 0, mt0 = blockIdx.y, i0 = 16 * mt0;
    const int back = stride - hn + i0;               // row i0's point is t + back (>= t)
    if (rg == 0) {
        if (bid == 0) *reinterpret_cast<V*>(s.ring_out + (int64_t)slot_t * D + col) = anchor;
        if (back == 0) *reinterpret_cast<V*>(&s_x[0][col]) = anchor;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r < nr) {
            const int j = j0 + r;                    // the point t + j + 1
            if (j == bid || (j >= nb && j % nb == bid)) *reinterpret_cast<V*>(s.ring_out + (int64_t)slot_at(j + 1) * D + col) = y[r];
            int i = j + 1 - back;
            if (i >= 0 && i < 16) *reinterpret_cast<V*>(&s_x[i][col]) = y[r];
            if (j == pe - 1) {                       // points past the window's last repeat it
                for (i = max(i + 1, 0); i < 16; ++i) *reinterpret_cast<V*>(&s_x[i][col]) = y[r];
                if (bid == 0 && !bad && tn >= T)     // a caller's pointer: aligned to a float
#pragma unroll
                    for (int c = 0; c < 4; ++c) fin.x_out[col + c] = y[r][c];
            }
        }
    }
    if (tid < 16) {
        const int n = i0 + tid < M ? s_mt[back + tid] : 0;
        s_n[tid] = n < 0 ? 0 : (n > s.n_max ? s.n_max : n);
    }
    if (bid == 0) slide_window(fin, stride, bad, cur, s_mt, fin.nrow2 ? s_mt2 : nullptr);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 2 * CT; ++i) asm volatile("" ::"v"(warm[i]));
    if (i0 >= M) return;                             // uniform over the block
    hidden_tile<1, CT, IN_LDS, false>(
        l1, TileRows{M, s.rows_max, HiddenBuf{}, nullptr, 0, &s_x[0][0], kFusedCols + 4, s_n}, out, mt0,
        blockIdx.x * CT, lds);
}

}  // namespace

// A block covers at most 64 lanes x VEC columns.  When the grid takes more
// than one block, the columns are shared out evenly over the fewest rounds of
// one block per compute unit that the 64-lane limit allows (a multiple of VEC
// per block), so that no unit streams twice the data of another: at
// 4x96x96 and one sample, 256 blocks of 144 columns instead of 144 of 256.
int picard_scan_cols(int64_t D, int batch) {
    const int vec = scan_vec(D);
    const int64_t full = 64 * (int64_t)vec;
    const int64_t blocks = (D + full - 1) / full * batch;
    const int64_t cus = device_cus();
    // one block keeps the fused finalize; a grid under half the units gains nothing
    if (blocks <= 1 || 2 * blocks < cus) return (int)full;
    const int64_t rounds = (blocks + cus - 1) / cus;
    int64_t per = (D * batch + rounds * cus - 1) / (rounds * cus);   // columns per block
    per = (per + vec - 1) / vec * vec;
    return (int)(per < full ? per : full);
}
int picard_partial_blocks(int64_t D, int batch) {
    const int64_t cols = picard_scan_cols(D, batch);
    return (int)((D + cols - 1) / cols);
}

static unsigned stream_blocks(int64_t n) {
    const int64_t b = (n + 255) / 256;
    return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

void launch_heun_predict(const LoopState* st, const float* ring, const float* eps, const float* A,
                         const float* B, int p, int64_t BD, float* xt, hipStream_t s) {
    hipLaunchKernelGGL(k_heun_predict, dim3(stream_blocks((int64_t)p * BD)), dim3(256), 0, s, st,
                       ring, eps, A, B, p, BD, xt);
    PD_HIP(hipGetLastError());
}

void launch_eps_step(const EpsOut& out, const float* eps, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_eps_step, dim3(stream_blocks(n)), dim3(256), 0, s, out, eps, n);
    PD_HIP(hipGetLastError());
}

template <int NW, int R, int VEC>
static bool launch_scan(const LoopState* st, float* ring, const float* eps, const float* noise,
                        const float* A, const float* B, const float* Rt, const float* St, int p,
                        int batch, int64_t D, float* partials, const FinalizeArgs& fin,
                        const float* eps2, hipStream_t s) {
    const int cpb = picard_scan_cols(D, batch);
    const dim3 grid((unsigned)picard_partial_blocks(D, batch), (unsigned)batch);
    const int fuse = grid.x * grid.y == 1;   // one block: the finalize works from LDS
    const dim3 block(NW * 64);
    if (Rt)      // DPM-Solver integrates the noise-free chain
        hipLaunchKernelGGL((k_picard_scan<NW, R, VEC, false, true>), grid, block, 0, s, st, ring, eps,
                           noise, A, B, Rt, St, p, batch, D, partials, fin, fuse, cpb, eps2);
    else if (noise)
        hipLaunchKernelGGL((k_picard_scan<NW, R, VEC, true, false>), grid, block, 0, s, st, ring, eps,
                           noise, A, B, Rt, St, p, batch, D, partials, fin, fuse, cpb, eps2);
    else
        hipLaunchKernelGGL((k_picard_scan<NW, R, VEC, false, false>), grid, block, 0, s, st, ring, eps,
                           noise, A, B, Rt, St, p, batch, D, partials, fin, fuse, cpb, eps2);
    PD_HIP(hipGetLastError());
    return fuse != 0;
}

bool launch_picard_scan(const LoopState* st, float* ring, const float* eps, const float* noise,
                        const float* A, const float* B, const float* R, const float* S, int p,
                        int batch, int64_t D, float* partials, const FinalizeArgs& fin,
                        const float* eps2, hipStream_t s) {
    if (p > kMaxWindow) fail(PD_ERR_UNSUPPORTED, "window larger than 128 points");
    if (R && noise) fail(PD_ERR_INVALID_ARG, "the multistep drift is for the noise-free chain");
    if (R && eps2) fail(PD_ERR_INVALID_ARG, "the multistep and Heun drifts do not combine");
    const bool v4 = scan_vec(D) == 4;
#define PD_SCAN(NW, RR)                                                                          \
    return v4 ? launch_scan<NW, RR, 4>(st, ring, eps, noise, A, B, R, S, p, batch, D, partials, \
                                       fin, eps2, s)                                             \
              : launch_scan<NW, RR, 1>(st, ring, eps, noise, A, B, R, S, p, batch, D, partials, \
                                       fin, eps2, s);
    if (p > 64) PD_SCAN(16, 8)
    const int ch = (p + 7) / 8;      // rows per wave at a full window, 8 waves
    if (ch <= 1) PD_SCAN(8, 1)
    if (ch <= 2) PD_SCAN(8, 2)
    if (ch <= 4) PD_SCAN(8, 4)
    PD_SCAN(8, 8)
#undef PD_SCAN
}

// Rows of a window of p points that a thread takes; up to twelve fit its registers.
static int scan_first_rows(int p, int64_t D) {
    const int groups = kLinThreads / (int)(D / 4);
    return (p + groups - 1) / groups;
}
bool scan_first_fits(int p, int batch, int64_t D, const LinearArgs& l1) {
    return batch == 1 && p >= 1 && p <= kFusedRows && D >= 4 && D <= kFusedCols && D % 4 == 0 && l1.K == D &&
           l1.N % 4 == 0 && l1.wexp == nullptr && scan_first_rows(p, D) <= 12;
}

template <int CT, int R>
static void launch_scan_first_t(const ScanFirstArgs& a, const FinalizeArgs& fin, const LinearArgs& l1,
                                const HiddenBuf& out, hipStream_t s) {
    const dim3 grid((unsigned)((l1.N + 16 * CT - 1) / (16 * CT)), (unsigned)((a.rows_max + 15) / 16)), block(kLinThreads);
    if (a.R) hipLaunchKernelGGL((k_scan_first<CT, R, false, true>), grid, block, 0, s, a, fin, l1, out);
    else if (a.noise) hipLaunchKernelGGL((k_scan_first<CT, R, true, false>), grid, block, 0, s, a, fin, l1, out);
    else hipLaunchKernelGGL((k_scan_first<CT, R, false, false>), grid, block, 0, s, a, fin, l1, out);
    PD_HIP(hipGetLastError());
}

void launch_scan_first(const ScanFirstArgs& a, const FinalizeArgs& fin, const LinearArgs& l1, const HiddenBuf& out,
                       hipStream_t s) {
    if (!scan_first_fits(fin.p, fin.batch, a.D, l1) || a.rows_max != fin.p + fin.history || (a.R != nullptr) != (fin.history != 0))
        fail(PD_ERR_UNSUPPORTED, "fused scan and first layer: sizes");
    if (a.R && (a.noise || a.eps2)) fail(PD_ERR_INVALID_ARG, "the multistep drift is for the noise-free chain");
    const int ch = scan_first_rows(fin.p, a.D);
    // one 16 x 16 block per unit while there are units, then two features tiles a block
    const bool one = (int64_t)((a.rows_max + 15) / 16) * ((l1.N + 15) / 16) <= device_cus();
#define PD_FUSED(R) return one ? launch_scan_first_t<1, R>(a, fin, l1, out, s) : launch_scan_first_t<2, R>(a, fin, l1, out, s)
    if (ch <= 4) PD_FUSED(4);
    if (ch <= 8) PD_FUSED(8);
    PD_FUSED(12);
#undef PD_FUSED
}

void launch_picard_finalize(const FinalizeArgs& fin, hipStream_t s) {
    hipLaunchKernelGGL(k_picard_finalize, dim3(1), dim3(1024), 0, s, fin,
                       picard_partial_blocks(fin.D, fin.batch));
    PD_HIP(hipGetLastError());
}

}  // namespace pd
