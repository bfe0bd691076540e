// Preparation kernels of compression: state reset, exact min/max of the field,
// the absolute error bound (Sec. 3.1 Eq. "general", Sec. 6.1.4) and the
// sampled-block tuner (Sec. 5.1.3).
#include "hiz_internal.h"

#include <type_traits>

namespace hiz {

// ---------------------------------------------------------------------------
// Error bound: eps = eb (ABS) or eb * (max - min) (REL), formed in FP64 and
// rounded down to FP32 so that it never exceeds the requested bound.
// ---------------------------------------------------------------------------
__device__ inline float bound_of(double e)
{
    float f = (float)e;
    if ((double)f > e)
        f = nextafterf(f, 0.0f);
    return f;
}
__device__ inline double tune_scale_of(float f)
{
    return f > 0.0f ? 65536.0 / (2.0 * (double)f) : 65536.0;
}
__device__ inline void store_bound(FieldState *st, double e)
{
    const float f = bound_of(e);
    st->eps = f;
    st->two_eb = f * 2.0f;
    st->inv = 1.0f / st->two_eb;
    st->tune_scale = tune_scale_of(f);
}
// REL, behind the launch that found the extremes: the bound in FP64. False: the
// field is constant.
__device__ inline bool rel_bound(const Job &J, uint32_t kmn, uint32_t kmx, double &e)
{
    const double range = (double)fkey_inv(kmx) - (double)fkey_inv(kmn);
    e = J.eb * range;
    return range != 0.0;
}
__device__ inline void store_rel_bound(const Job &J, FieldState *st, uint32_t kmn, uint32_t kmx)
{
    st->kmin = kmn;
    st->kmax = kmx;
    st->vmin = fkey_inv(kmn);
    st->vmax = fkey_inv(kmx);
    double e;
    if (rel_bound(J, kmn, kmx, e))
        store_bound(st, e);
    else
        atomicOr(&st->flags, (uint32_t)ST_CONST);
}
__device__ inline void store_cfg(FieldState *st, int l, int sp, int sc, int pm)
{
    st->cfg[l][0] = (uint8_t)sp;
    st->cfg[l][1] = (uint8_t)sc;
    st->cfg[l][2] = (uint8_t)pm;
}

// ---------------------------------------------------------------------------
// Reset of per-field state and look-back flags (a fill kernel rather than
// hipMemsetAsync so that the sequence can be captured in a HIP graph). The Job
// table is read from pinned host memory and copied to the device on the way,
// which saves the call a copy of its own (each one some 5 us on the stream).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_init_compress(const Job *__restrict__ h_jobs,
                                                       Job *__restrict__ d_jobs, Counters *cnt)
{
    __shared__ Job J;
    copy_job(J, h_jobs, d_jobs);
    FieldState *st = J.st;
    const uint32_t t = threadIdx.x;
    if (blockIdx.x == 0) {
        st->hist[t] = 0;
        if (t < kLevels * kCands)
            (&st->tune_err[0][0])[t] = 0;
        if (t == 0) {
            st->flags = 0u;
            st->n_out = 0;
            st->payload_words = 0;
            st->total_bytes = 0;
            st->zeros_seen = 0;
            st->tuned = 0;
            if (J.mode != 1)
                store_bound(st, J.eb);
        }
        // without a sample to measure: the configuration asked for, or the
        // default one; with one, the tuner's last workgroup stores its choice
        if (t < kLevels) {
            const uint8_t *cf = J.cfg_forced[t];
            if (J.n_tune != 0)
                store_cfg(st, t, 0, 0, 0);
            else if (J.tune)
                store_cfg(st, t, 1, 0, 0);
            else
                store_cfg(st, t, cf[0], cf[1], cf[2]);
        }
        if (blockIdx.y == 0 && t < sizeof(Counters) / 4)
            reinterpret_cast<uint32_t *>(cnt)[t] = 0u;
    }
    for (uint64_t i = blockIdx.x * 256ull + t; i < J.n_groups; i += 256ull * gridDim.x) {
        J.lb_a[i] = 0;
        J.lb_b[i] = 0;
    }
    // look-back words of the last stages' chunks and of the outlier units
    for (uint64_t i = blockIdx.x * 256ull + t; i < J.n_lc; i += 256ull * gridDim.x)
        J.lb_c[i] = 0;
    const uint64_t nd = J.n_ou > J.n_lc ? J.n_ou : J.n_lc;
    for (uint64_t i = blockIdx.x * 256ull + t; i < nd; i += 256ull * gridDim.x)
        J.lb_d[i] = 0;
}

void launch_init_compress(const Job *h_jobs, Job *d_jobs, int njobs, uint64_t max_chunks,
                          Counters *cnt, hipStream_t s)
{
    // (each workgroup reads its Job over the host link: 1024 of them, or one a field)
    uint64_t gx = cdiv(max_chunks, 256);
    if (gx > 1024 / (uint64_t)njobs)
        gx = 1024 / (uint64_t)njobs;
    if (gx < 1)
        gx = 1;
    hipLaunchKernelGGL(k_init_compress, dim3((uint32_t)gx, njobs), dim3(256), 0, s, h_jobs, d_jobs,
                       cnt);
}

// ---------------------------------------------------------------------------
// Exact min/max (REL mode): ordered 32-bit keys, so the result does not depend
// on the order of reduction; NaN/Inf raise a flag. A workgroup keeps its extremes
// over all its units of a field and stores them in the slot of the first of
// them, which is below the grid's size: a field has min(units, grid) slots, and
// whoever needs the bound reduces those. (Atomics on two words of the field
// instead: 100 x 500 x 500 59 us, this way 29.)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_minmax(const Job *__restrict__ jobs, int njobs,
                                                uint64_t total)
{
    __shared__ uint32_t red[8];
    const uint32_t t = threadIdx.x;
    int cur = -1;
    uint64_t slot = 0;
    uint32_t kmn = 0xffffffffu, kmx = 0u;
    bool bad = false;
    auto flush = [&]() {
        if (__any(bad) && (t & 63) == 0)
            atomicOr(&jobs[cur].st->flags, (uint32_t)ST_NONFINITE);
        block_minmax(kmn, kmx, red);
        if (t == 0)
            gstore_u2(gmem(jobs[cur].mm_part) + slot, make_uint2(kmn, kmx));
        kmn = 0xffffffffu;
        kmx = 0u;
        bad = false;
        __syncthreads(); // red is free again
    };
    for (uint64_t u = blockIdx.x; u < total; u += gridDim.x) {
        const int ji = find_job<WK_MM>(jobs, njobs, u);
        if (ji != cur) {
            if (cur >= 0)
                flush();
            cur = ji;
            slot = u - jobs[ji].mm_begin;
        }
        const Job &J = jobs[ji];
        const uint64_t lu = u - J.mm_begin;
        const uint64_t lo = lu * kMmUnit;
        const uint64_t hi = min(lo + kMmUnit, J.N);
        HIZ_GLOBAL const float *f = gmem(J.field);
        const bool vec = ((reinterpret_cast<uintptr_t>(f) & 15u) == 0) && (hi - lo == kMmUnit);
        if (vec) {
            // all 16 loads of a thread in flight before any is used: one
            // memory round trip per unit; streamed (the field is larger than
            // the caches, so nothing of it would be found there later)
            HIZ_GLOBAL const float *fb = f + lo;
            constexpr int K = (int)(kMmUnit / 4 / 256);
            float4 q4[K];
#pragma unroll
            for (int k = 0; k < K; k++)
                q4[k] = gload_f4_nt(fb + 4 * (k * 256 + t));
#pragma unroll
            for (int k = 0; k < K; k++) {
                const float4 q = q4[k];
                float e[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    bad |= !isfinite(e[i]);
                    uint32_t key = fkey(e[i]);
                    kmn = min(kmn, key);
                    kmx = max(kmx, key);
                }
            }
        } else {
            for (uint64_t i = lo + t; i < hi; i += 256) {
                float e = f[i];
                bad |= !isfinite(e);
                uint32_t key = fkey(e);
                kmn = min(kmn, key);
                kmx = max(kmx, key);
            }
        }
    }
    if (cur >= 0)
        flush();
}

uint32_t minmax_grid(uint64_t total, int cus)
{
    return (uint32_t)(total < 8ull * cus ? total : 8ull * cus);
}

void launch_minmax(const Job *d_jobs, int njobs, uint64_t total, uint32_t grid, hipStream_t s)
{
    if (total == 0)
        return;
    hipLaunchKernelGGL(k_minmax, dim3(grid), dim3(256), 0, s, d_jobs, njobs, total);
}

// The bound of REL fields whose configuration is not measured (the tuner's
// launch forms it for the others).
__global__ __launch_bounds__(256) void k_eps(const Job *__restrict__ jobs, uint32_t mm_grid)
{
    __shared__ uint32_t red[8];
    const Job &J = jobs[blockIdx.x];
    if (J.mode != 1 || J.n_tune != 0 || (J.st->flags & ST_NONFINITE))
        return;
    uint32_t kmn, kmx;
    reduce_partials(J.mm_part, min(J.n_mm, (uint64_t)mm_grid), kmn, kmx, red);
    if (threadIdx.x == 0)
        store_rel_bound(J, J.st, kmn, kmx);
}

void launch_eps(const Job *d_jobs, int njobs, uint32_t mm_grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_eps, dim3(njobs), dim3(256), 0, s, d_jobs, mm_grid);
}

// ---------------------------------------------------------------------------
// Tuner (Sec. 5.1.3). Full 17^3 blocks with 0.2 % of the volume are sampled at
// even spacing. Every level is tested with the 21 candidates {LIN, CUB, NAT}
// x {MD, SEQ over the 6 dimension orders}, predicting from ORIGINAL values; the
// candidate with the smallest aggregated |x - p| wins per level (ties: lower
// index). Each |x - p| is counted in units of 2*eps/65536, rounded and capped
// at 2^36, and summed as a 64-bit integer, so the totals are exact and do not
// depend on the reduction order.
//
// Work balance follows the paper's idea of giving the expensive fine levels
// more thread blocks: per sample, one block tests strides 8 and 4, two
// blocks share stride 2 and six share stride 1. Unlike the paper, each block
// tests all 21 candidates on its share of targets, because the candidates
// reuse the same per-axis stencils: a sequential candidate predicts a target by
// one axis's stencil, the last of its odd axes in the candidate's order. So a
// target costs three splines' errors along each of its odd axes and, with more
// than one, of their combination; they are added up apart for each class of
// targets (which axes are odd) and handed out to the candidates once per class.
// A wave takes 64 targets of one class at a time; had each class been spread over
// the workgroup, its part of it (85 targets of stride 1) would leave two thirds of
// the lanes idle. What bounds the kernel is the latency of one workgroup: loads,
// three of those units, the sums. With all 21 errors formed per target, and the
// bound and the choice left to launches of their own, the three took 39 us at 64^3,
// 53 at 512^3 and 41 for a 1800 x 3600 field; this way one takes 20, 26 and 20.
// ---------------------------------------------------------------------------
constexpr int kTuneParts = 9;

// 1-D spline stencil (Sec. 5.1.2): Lagrange weights at the midpoint from the
// samples at -3s, -s, +s, +3s; lower orders where samples are missing. With
// all four samples, spline 2 is the natural cubic spline through them (zero
// second derivative at the outer samples): weights (-3, 23, 23, -3) / 40.
__device__ __forceinline__ float stencil_1d(float a, float b, float c, float d, bool pa, bool pc,
                                            bool pd, int spline, int &rank)
{
    const bool cub = spline != 0;
    if (cub && pa && pc && pd) {
        rank = 4;
        if (spline == 2)
            return ((b + c) * 23.0f - (a + d) * 3.0f) / 40.0f;
        return ((b + c) * 9.0f - (a + d)) * 0.0625f;
    }
    if (cub && pc && pd) {
        rank = 3;
        return ((b * 3.0f + c * 6.0f) - d) * 0.125f;
    }
    if (cub && pa && pc) {
        rank = 3;
        return ((b * 6.0f + c * 3.0f) - a) * 0.125f;
    }
    if (pc) {
        rank = 2;
        return (b + c) * 0.5f;
    }
    if (pa) {
        rank = 1;
        return b * 1.5f - a * 0.5f;
    }
    rank = 0;
    return b;
}

// Mean of the predictions of maximal rank, combined in x, y, z order.
__device__ __forceinline__ float md_combine(const float p[3], const int r[3], int mask)
{
    int best = -1;
    for (int k = 0; k < 3; k++)
        if ((mask >> k) & 1)
            best = max(best, r[k]);
    bool u0 = (mask & 1) && r[0] == best, u1 = (mask & 2) && r[1] == best,
         u2 = (mask & 4) && r[2] == best;
    int m = (int)u0 + (int)u1 + (int)u2;
    float first = u0 ? p[0] : (u1 ? p[1] : p[2]);
    float second = u0 ? (u1 ? p[1] : p[2]) : p[2];
    if (m == 1)
        return first;
    if (m == 2)
        return (first + second) * 0.5f;
    return ((p[0] + p[1]) + p[2]) / 3.0f;
}

// |x - p| in units of 1 / scale, rounded and capped at 2^36, as the integer held
// in the low bits of 2^52 + it: sums of n terms carry n times 2^52's bits
// (kTermBias), taken off at the end. A NaN counts as the cap.
constexpr uint64_t kTermBias = 0x4330000000000000ull;
__device__ __forceinline__ uint64_t tune_term(float x, float p, double scale)
{
    const double w = fmin((double)fabsf(x - p) * scale, 68719476736.0);
    return (uint64_t)__double_as_longlong(trunc(w + 0.5) + 4503599627370496.0);
}

// Sum over the wave with DPP moves (the result in lane 63).
__device__ __forceinline__ uint64_t wave_sum_dpp64(uint64_t v)
{
    auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
        constexpr int c = decltype(ctrl)::value, r = decltype(rows)::value;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, c, r, 0xf, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), c, r, 0xf, false);
        v += ((uint64_t)hi << 32) | lo;
    };
    step(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{}); // row_shr 1
    step(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{}); // row_bcast 15
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{}); // row_bcast 31
    return v;
}

// Add the 21 candidates' error sums of class M's targets on the stride-s grid of
// a block held in LDS (strides 17*17, 17, 1) whose extent on axis k is E[k] (17,
// or 1 on a flat axis); of the targets in order, those from n g0 / parts up to
// n (g0 + 1) / parts.
template <int M>
__device__ __forceinline__ void tune_class(const float *__restrict__ blk, const int E[3], int s,
                                           int &unit, int &base, int waves, double scale,
                                           uint64_t acc[kCands])
{
    const int K = 8 / s; // odd multiples of s in a block; even ones: one more
    int n[3];
    for (int k = 0; k < 3; k++)
        n[k] = (M >> k) & 1 ? (E[k] == 1 ? 0 : K) : (E[k] == 1 ? 1 : K + 1);
    const int total = n[0] * n[1] * n[2];
    constexpr bool MULTI = (M & (M - 1)) != 0;
    uint64_t one[3][3] = {}, md[3] = {}; // [spline][axis]; multi-dimensional
    int terms = 0;
    const int end = base + (total + 63) / 64;
    if (unit >= end) {
        base = end;
        return;
    }
    for (; unit < end; unit += waves) {
        const int g = 64 * (unit - base) + (int)(threadIdx.x & 63);
        if (g >= total)
            continue;
        const int iz = g % n[2], r = g / n[2], iy = r % n[1], ix = r / n[1];
        const int t[3] = {(2 * ix + (M & 1)) * s, (2 * iy + ((M >> 1) & 1)) * s,
                          (2 * iz + (M >> 2)) * s};
        const int st[3] = {kSide * kSide, kSide, 1};
        const int li = (t[0] * kSide + t[1]) * kSide + t[2];
        const float x = blk[li];
        float p[3][3];
        int rk[3][3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            if (!((M >> k) & 1))
                continue;
            const bool pa = t[k] - 3 * s >= 0, pc = t[k] + s <= E[k] - 1, pd = t[k] + 3 * s <= E[k] - 1;
            const float b = blk[li - s * st[k]];
            const float a = pa ? blk[li - 3 * s * st[k]] : 0.0f;
            const float c = pc ? blk[li + s * st[k]] : 0.0f;
            const float d = pd ? blk[li + 3 * s * st[k]] : 0.0f;
#pragma unroll
            for (int sp = 0; sp < 3; sp++) {
                p[sp][k] = stencil_1d(a, b, c, d, pa, pc, pd, sp, rk[sp][k]);
                one[sp][k] += tune_term(x, p[sp][k], scale);
            }
        }
        if constexpr (MULTI)
#pragma unroll
            for (int sp = 0; sp < 3; sp++)
                md[sp] += tune_term(x, md_combine(p[sp], rk[sp], M), scale);
        terms++;
    }
    base = end;
    const uint64_t bias = (uint64_t)terms * kTermBias;
    constexpr int first = (M & 1) ? 0 : ((M & 2) ? 1 : 2);
#pragma unroll
    for (int sp = 0; sp < 3; sp++) {
        acc[7 * sp] += (MULTI ? md[sp] : one[sp][first]) - bias;
        // SEQ over the orders (x,y,z) (x,z,y) (y,x,z) (y,z,x) (z,x,y) (z,y,x)
        constexpr int perm[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
#pragma unroll
        for (int q = 0; q < 6; q++) {
            const int axis = (M >> perm[q][2]) & 1 ? perm[q][2]
                                                   : ((M >> perm[q][1]) & 1 ? perm[q][1] : perm[q][0]);
            acc[7 * sp + 1 + q] += one[sp][axis] - bias;
        }
    }
}
// The targets of a level, in units of a class's 64 (base: the first of a class),
// dealt out to `waves` waves of which this is the one numbered `unit`.
__device__ void tune_level(const float *__restrict__ blk, const int E[3], int s, int unit, int waves,
                           double scale, uint64_t acc[kCands])
{
    int base = 0;
    tune_class<7>(blk, E, s, unit, base, waves, scale, acc);
    tune_class<6>(blk, E, s, unit, base, waves, scale, acc);
    tune_class<5>(blk, E, s, unit, base, waves, scale, acc);
    tune_class<3>(blk, E, s, unit, base, waves, scale, acc);
    tune_class<4>(blk, E, s, unit, base, waves, scale, acc);
    tune_class<2>(blk, E, s, unit, base, waves, scale, acc);
    tune_class<1>(blk, E, s, unit, base, waves, scale, acc);
}

__device__ void tune_flush(FieldState *st, int level, uint64_t acc[kCands], uint64_t *red)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int c = 0; c < kCands; c++) {
        const uint64_t v = wave_sum_dpp64(acc[c]);
        if (lane == 63)
            red[wave * kCands + c] = v;
        acc[c] = 0;
    }
    __syncthreads();
    if (threadIdx.x < kCands) {
        uint64_t v = 0;
        for (int w = 0; w < nw; w++)
            v += red[w * kCands + threadIdx.x];
        if (v)
            atomicAdd((unsigned long long *)&st->tune_err[level][threadIdx.x],
                      (unsigned long long)v);
    }
    __syncthreads();
}

// Per-level argmin by one wave: each lane holds one candidate's error of every
// level, and a wave argmin takes the smallest, the lower candidate on equal
// errors (the first in candidate order).
__device__ void pick(FieldState *st)
{
    static_assert(kCands <= 64, "one lane per candidate");
    const int lane = threadIdx.x & 63;
    uint64_t err[kLevels];
#pragma unroll
    for (int l = 0; l < kLevels; l++)
        err[l] = lane < kCands ? lb_load(&st->tune_err[l][lane]) : ~0ull;
#pragma unroll
    for (int l = 0; l < kLevels; l++) {
        uint64_t e = err[l];
        int c = lane;
        for (int o = 32; o > 0; o >>= 1) {
            const uint64_t e2 = shfl64(e, lane ^ o);
            const int c2 = __shfl_xor(c, o, 64);
            if (e2 < e || (e2 == e && c2 < c)) {
                e = e2;
                c = c2;
            }
        }
        const int r = c % 7;
        if (lane == 0)
            store_cfg(st, l, c / 7, r == 0 ? 0 : 1, r == 0 ? 0 : r - 1);
    }
}

__global__ __launch_bounds__(256) void k_tune(const Job *__restrict__ jobs, int njobs,
                                              uint64_t total, uint32_t mm_grid)
{
    __shared__ float blk[kSide * kSide * kSide];
    __shared__ uint64_t red[4 * kCands];
    const uint64_t u = blockIdx.x;
    if (u >= total)
        return;
    const Job &J = jobs[find_job<WK_TUNE>(jobs, njobs, u)];
    FieldState *st = J.st;
    if (st->flags & ST_NONFINITE)
        return;
    const uint64_t lu = u - J.tune_begin;
    const uint64_t j = (uint32_t)lu / (uint32_t)kTuneParts; // (a launch has fewer than 2^32 units)
    const int part = (int)((uint32_t)lu - (uint32_t)j * kTuneParts);
    // (divisions in 32 bits where they do)
    auto div = [](uint64_t a, uint64_t b) __attribute__((always_inline)) -> uint64_t {
        return (a | b) >> 32 ? a / b : (uint64_t)((uint32_t)a / (uint32_t)b);
    };
    const uint64_t n_full = (uint64_t)J.n_full[0] * J.n_full[1] * J.n_full[2];
    const uint64_t idx = div((2 * j + 1) * n_full, 2 * (uint64_t)J.n_samples);
    const uint64_t row = div(idx, J.n_full[2]), ba = div(row, J.n_full[1]);
    const uint64_t bc = idx - row * J.n_full[2], bb = row - ba * J.n_full[1];
    const uint64_t dy = J.dims[1], dz = J.dims[2];
    // a full block spans 17 points per axis, 1 on a flat axis (2-D / 1-D fields)
    const int E[3] = {J.dims[0] == 1 ? 1 : kSide, J.dims[1] == 1 ? 1 : kSide,
                      J.dims[2] == 1 ? 1 : kSide};
    // all of a thread's loads in flight before the first is written to LDS
    constexpr int IB = (kSide * kSide * kSide + 255) / 256;
    float e[IB];
    HIZ_GLOBAL const float *f0 =
        gmem(J.field) + ((ba * kAnchor) * dy + bb * kAnchor) * dz + bc * kAnchor;
#pragma unroll
    for (int k = 0; k < IB; k++) {
        const int i = threadIdx.x + 256 * k;
        const int z = i % kSide, r = i / kSide, y = r % kSide, x = r / kSide;
        const bool in = x < E[0] && y < E[1] && z < E[2]; // (past the block's last point: x = 17)
        e[k] = f0[in ? (x * dy + y) * dz + z : 0];
    }
    // a REL field's bound: every workgroup forms it, the first one stores it
    double scale;
    if (J.mode == 1) {
        uint32_t *red32 = reinterpret_cast<uint32_t *>(red);
        uint32_t kmn, kmx;
        reduce_partials(J.mm_part, min(J.n_mm, (uint64_t)mm_grid), kmn, kmx, red32);
        if (threadIdx.x == 0) {
            red32[0] = kmn;
            red32[1] = kmx;
            if (lu == 0)
                store_rel_bound(J, st, kmn, kmx);
        }
        __syncthreads();
        double b;
        if (!rel_bound(J, red32[0], red32[1], b))
            return;
        scale = tune_scale_of(bound_of(b));
    } else {
        scale = st->tune_scale;
    }
#pragma unroll
    for (int k = 0; k < IB; k++) {
        const int i = threadIdx.x + 256 * k;
        if (k < IB - 1 || i < kSide * kSide * kSide)
            blk[i] = e[k];
    }
    __syncthreads();
    uint64_t acc[kCands];
#pragma unroll
    for (int c = 0; c < kCands; c++)
        acc[c] = 0;
    // stride 8 and 4 in one part, stride 2 in two, stride 1 in six
    const int l0 = part == 0 ? 0 : (part <= 2 ? 2 : 3), l1 = part == 0 ? 1 : l0;
#pragma unroll 1
    for (int l = l0; l <= l1; l++) {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int p = part == 0 ? 0 : part <= 2 ? part - 1 : part - 3;
        const int parts = part == 0 ? 1 : part <= 2 ? 2 : 6;
        tune_level(blk, E, 8 >> l, 4 * p + wave, 4 * parts, scale, acc);
        tune_flush(st, l, acc, red);
    }
    // The field's last workgroup picks: every workgroup's sums are in place
    // (its wave 0 has waited for its atomics) before it counts itself.
    if (threadIdx.x >= 64)
        return;
    drain_memory();
    int last = 0;
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(&st->tuned, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
               (uint32_t)J.n_tune - 1;
    if (__builtin_amdgcn_readfirstlane(last))
        pick(st);
}

void launch_tune(const Job *d_jobs, int njobs, uint64_t total, uint32_t mm_grid, hipStream_t s)
{
    if (total == 0)
        return;
    hipLaunchKernelGGL(k_tune, dim3((uint32_t)total), dim3(256), 0, s, d_jobs, njobs, total,
                       mm_grid);
}

// ---------------------------------------------------------------------------
// Constant-field decompression: every element gets the stored value.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fill(float *out, uint64_t n, float v)
{
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += 256ull * gridDim.x)
        out[i] = v;
}

void launch_fill(float *out, uint64_t n, float v, hipStream_t s)
{
    uint64_t g = cdiv(n, 256);
    if (g > 4096)
        g = 4096;
    if (g < 1)
        g = 1;
    hipLaunchKernelGGL(k_fill, dim3((uint32_t)g), dim3(256), 0, s, out, n, v);
}

// ---------------------------------------------------------------------------
// The first bytes of every job's state, written to pinned host memory.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gather_results(const Job *__restrict__ jobs, int njobs,
                                                        uint32_t *__restrict__ dst)
{
    constexpr int W = kResultBytes / 4;
    const uint64_t i = blockIdx.x * 256ull + threadIdx.x;
    if (i >= (uint64_t)njobs * W)
        return;
    const int j = (int)(i / W), w = (int)(i % W);
    dst[i] = reinterpret_cast<const uint32_t *>(jobs[j].st)[w];
}

void launch_gather_results(const Job *d_jobs, int njobs, void *h_dst, hipStream_t s)
{
    const uint64_t n = (uint64_t)njobs * (kResultBytes / 4);
    hipLaunchKernelGGL(k_gather_results, dim3((uint32_t)cdiv(n, 256)), dim3(256), 0, s, d_jobs,
                       njobs, static_cast<uint32_t *>(h_dst));
}

// The first kOffChunks bytes (or all, if fewer) of n streams, kOffChunks apart, to
// pinned memory; tab: n {address, size}, in pinned memory too.
__global__ __launch_bounds__(128) void k_gather_headers(const uint64_t *__restrict__ tab,
                                                        uint8_t *__restrict__ dst)
{
    const uint64_t n = min(tab[2 * blockIdx.x + 1], (uint64_t)kOffChunks);
    HIZ_GLOBAL const uint8_t *src = gmem(reinterpret_cast<const uint8_t *>(tab[2 * blockIdx.x]));
    dst += (uint64_t)kOffChunks * blockIdx.x;
    if (n == kOffChunks && (reinterpret_cast<uintptr_t>(src) & 3) == 0) {
        if (threadIdx.x < kOffChunks / 4)
            reinterpret_cast<uint32_t *>(dst)[threadIdx.x] =
                reinterpret_cast<HIZ_GLOBAL const uint32_t *>(src)[threadIdx.x];
    } else {
        for (uint64_t i = threadIdx.x; i < n; i += 128)
            dst[i] = src[i];
    }
}

void launch_gather_headers(const uint64_t *h_tab, int n, void *h_dst, hipStream_t s)
{
    hipLaunchKernelGGL(k_gather_headers, dim3(n), dim3(128), 0, s, h_tab, static_cast<uint8_t *>(h_dst));
}

} // namespace hiz
