// Level-wise spline interpolation over 17^3 blocks (Sec. 5.1.1-5.1.2), fused
// with linear-scaling quantization and the code histogram (compression) or
// with reconstruction from codes (decompression).
//
// GPU design. A workgroup owns a tile of TZ consecutive blocks along z
// (1 x 1 x TZ blocks, 17 x 17 x (16*TZ+1) points with the shared +1 faces) and
// walks all four levels on it in LDS; every target of a sub-step is
// independent of the others in that sub-step, so the workgroup sweeps a
// sub-step in parallel and synchronizes between sub-steps. Targets on the face
// shared by two blocks of a tile are computed once: their stencils never leave
// the face, so they equal what each block would compute alone, and z-stencils
// stop at the block's own faces exactly as in a lone block.
//
// Layout. The eight parity classes of a point's coordinates are kept apart
// (struct Tile), each dense, so four consecutive targets of a class along z,
// and the samples of their x- and y-stencils, are whole 16-byte pieces of LDS:
// the stride-1 level (7 of every 8 points) works on quads of four targets per
// lane, every sample of a quad one LDS read where a layout in plain z order
// needs four. The lanes of such a read cover consecutive 16-byte pieces, so no
// two lanes of a pass meet in a bank. The class of even coordinates is the
// lattice on which the coarser levels run. A thread owns the same two-by-two
// rows of eight z through the whole tile: it loads them (32 bytes per row),
// quantizes their odd-lattice targets, keeps the codes in registers and stores
// whole 8-byte pieces, so codes need no LDS and 39 KB of values leave room for
// four workgroups per compute unit.
//
// Workgroups are persistent: each walks tiles of the contiguous eighth of the
// list that its XCD (blockIdx % 8) owns, so neighbouring tiles that share halo
// faces are read through the same L2. The code histogram is kept in LDS for a
// tile, in registers across the tiles of a field.
// What bounds it: instruction issue and LDS latency of the levels, at four waves
// per SIMD (LDS holds four tiles per compute unit); the traffic alone would take
// 134 us each way at 512^3. The 128 registers that four waves leave hold all that
// k_reconstruct and the flat tiles need. k_predict spills: 41 to 44 registers, 56 to
// 68 bytes of scratch per lane, by tile depth. At 512^3 that is 113 of its 257 MiB
// written and 119 of its 693 MiB read; with three waves per SIMD it spills nothing
// and takes 467 us instead of 432.
// Measured at 512^3 (linear splines), with all levels in this kernel: k_predict
// 438 us, k_reconstruct 308 us; 16 M points with odd sides (cubic): 108 and 83
// us. With plain rows in LDS, lines along an axis per thread and the coarse
// levels in a kernel of their own it took 655 and 594, 308 and 287 us.
#include "hiz_internal.h"

#include <type_traits>

namespace hiz {

// A tile of NX x 16 x 16 TZ owned points (NX = 16, or 1 for flat fields of a
// single x plane) with its +1 faces, in LDS. Class c of a point has bit 0, 1, 2
// set where its x, y, z is odd; a point's place in its class is (x / 2, y / 2,
// z / 2). Class c is an array of rows of KZ words along z, 9 rows (y even) or 8
// (y odd) per x; class 0 (the lattice) has rows of LP words, the far z face its
// word KZ. The far z face of classes 1, 2, 3 is an array of its own per class.
template <int TZ, int NX> struct Tile {
    static constexpr bool FLAT = NX == 1;
    static constexpr int SX = FLAT ? 1 : kSide; // planes along x
    static constexpr int KZ = 8 * TZ;           // points of a class row without the far face
    static constexpr int LP = KZ + 4;           // pitch of a lattice row (KZ + 1 used)
    static constexpr int NQ = 2 * TZ;           // quads of a row
    // places along x and y of class c
    static constexpr int nx(int c) { return (c & 1) ? (FLAT ? 0 : 8) : (FLAT ? 1 : 9); }
    static constexpr int ny(int c) { return (c & 2) ? 8 : 9; }
    static constexpr int pitch(int c) { return c == 0 ? LP : KZ; }
    static constexpr int base(int c) { return c == 0 ? 0 : base(c - 1) + nx(c - 1) * ny(c - 1) * pitch(c - 1); }
    static constexpr int face(int c) { return c <= 1 ? base(8) : face(c - 1) + nx(c - 1) * ny(c - 1); }
    static constexpr int NV = face(4);
    static constexpr int OX = FLAT ? 1 : 8;          // owned lattice points along x
    static constexpr int LXS = 9 * LP;               // lattice words from one x to the next
    static constexpr int NT = (FLAT ? 8 : 64) * NQ;  // threads: one per owned row group and quad
    static constexpr int NW = NT / 64;
    // rows on the far x and y faces: 17 of even x and y (9 along y at x = 16,
    // 8 along x at y = 16), 8 with y odd, 8 with x odd; in a flat tile one
    static constexpr int NE = (FLAT ? 1 : 33) * NQ;
    // rows of the far z face, those holding targets of the stride-1 level first
    static constexpr int NR = SX * kSide;
    static constexpr int IF = (NR + NT - 1) / NT;
    static_assert(NT >= 64 && NT % 64 == 0 && NE <= NT, "one face-row quad per thread");
    // word of place (x, y, z) in class c; of far-face place (x, y) in class 1, 2 or 3
    template <int C> static __device__ __forceinline__ int word(int x, int y, int z)
    {
        return base(C) + (x * ny(C) + y) * pitch(C) + z;
    }
    template <int C> static __device__ __forceinline__ int fword(int x, int y)
    {
        return C == 0 ? (x * 9 + y) * LP + KZ : face(C) + x * ny(C) + y;
    }
};

struct Geo {
    int ex, ey, ez;       // tile extents (<= 17, 17, 16*TZ+1)
    int ownx, owny, ownz; // owned extents
};

__device__ __forceinline__ float unif(float v) { return __uint_as_float(uni32(__float_as_uint(v))); }
// The i-th of three values (passed by value: a choice between members would
// put the struct that holds them into memory).
__device__ __forceinline__ uint32_t pick(int i, uint32_t a, uint32_t b, uint32_t c)
{
    return i == 0 ? a : (i == 1 ? b : c);
}
// Bound and level configuration of the current field, the same for all lanes.
struct FieldQ {
    float eps, two_eb, inv;
    uint32_t cfg0, cfg1, cfg2; // the 12 configuration bytes, {spline, scheme, order} per level
    uint32_t use0, use1, use2; // stride-1 level: the axes of class c in pass p, at bit 4 c of use p
    __device__ __forceinline__ int spline(int l) const { return byte(3 * l); }
    __device__ __forceinline__ bool md(int l) const { return byte(3 * l + 1) == 0; }
    __device__ __forceinline__ int order(int l) const { return byte(3 * l + 2); }
    __device__ __forceinline__ int byte(int i) const
    {
        // read anew where it is used, not kept unpacked across the tile loop
        const uint32_t w = uni32(pick(i >> 2, cfg0, cfg1, cfg2));
        return (int)(w >> (8 * (i & 3))) & 255;
    }
};
// ---------------------------------------------------------------------------
// Stencils (Sec. 5.1.2)
// ---------------------------------------------------------------------------
// x / 3 and x / 40 correctly rounded: the product with the rounded reciprocal,
// corrected once by its exact remainder. Equal to the division for every
// finite x (3), and for every |x| at or above 2^-120 (40): compared on all
// floats.
__device__ __forceinline__ float div3(float x)
{
    const float y = 1.0f / 3.0f, q = x * y;
    return __builtin_fmaf(__builtin_fmaf(-3.0f, q, x), y, q);
}
__device__ __forceinline__ float div40(float x)
{
    const float y = 1.0f / 40.0f, q = x * y;
    return __builtin_fmaf(__builtin_fmaf(-40.0f, q, x), y, q);
}

// Four-sample midpoint values of the cubic splines: Lagrange (-1, 9, 9, -1) / 16,
// or (nat, the same for the wave) the natural cubic spline through the samples,
// zero second derivative at the outer two, (-3, 23, 23, -3) / 40.
template <int N>
__device__ __forceinline__ void mid(const float (&a)[N], const float (&b)[N], const float (&c)[N],
                                    const float (&d)[N], bool nat, float (&p)[N])
{
    if (nat) {
        bool tiny = false;
#pragma unroll
        for (int j = 0; j < N; j++) {
            const float x = (b[j] + c[j]) * 23.0f - (a[j] + d[j]) * 3.0f;
            p[j] = div40(x);
            tiny |= fabsf(x) < 0x1p-120f;
        }
        if (__builtin_expect(__any(tiny), 0)) {
#pragma unroll
            for (int j = 0; j < N; j++)
                p[j] = ((b[j] + c[j]) * 23.0f - (a[j] + d[j]) * 3.0f) / 40.0f;
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; j++)
            p[j] = ((b[j] + c[j]) * 9.0f - (a[j] + d[j])) * 0.0625f;
    }
}

// Which samples of a 1-D stencil exist besides b = v(t-s): a = v(t-3s),
// c = v(t+s), d = v(t+3s).
struct Has {
    bool a, c, d;
};

// 1-D spline stencil: the spline's midpoint value (CUB: cubic or natural
// cubic; else linear); where samples are missing the order drops to quadratic
// (one side), linear, linear extrapolation or copy. Missing samples are never
// selected. stencil_low: what is left when the cubic does not apply.
template <bool CUB, bool FULL>
__device__ __forceinline__ float stencil_low(float a, float b, float c, float d, const Has &h)
{
    if constexpr (CUB) {
        const float vqr = ((b * 3.0f + c * 6.0f) - d) * 0.125f;
        const float vql = ((b * 6.0f + c * 3.0f) - a) * 0.125f;
        if constexpr (FULL) // a block's targets lack at most one sample
            return h.d ? vqr : vql;
        const float vl = (b + c) * 0.5f;
        const float ve = b * 1.5f - a * 0.5f;
        return h.c && h.d ? vqr : (h.c && h.a ? vql : (h.c ? vl : (h.a ? ve : b)));
    } else {
        const float vl = (b + c) * 0.5f;
        if constexpr (FULL)
            return vl;
        const float ve = b * 1.5f - a * 0.5f;
        return h.c ? vl : (h.a ? ve : b);
    }
}
// N targets whose samples exist alike. FULL: c exists, and a or d.
template <bool CUB, bool FULL, int N>
__device__ __forceinline__ void stencils(const float (&a)[N], const float (&b)[N],
                                         const float (&c)[N], const float (&d)[N], const Has &h,
                                         bool nat, float (&p)[N])
{
    if (CUB && h.a && h.c && h.d) {
        mid(a, b, c, d, nat, p);
    } else {
#pragma unroll
        for (int j = 0; j < N; j++)
            p[j] = stencil_low<CUB, FULL>(a[j], b[j], c[j], d[j], h);
    }
}
template <bool CUB>
__device__ __forceinline__ float stencil(float a, float b, float c, float d, const Has &h, bool nat)
{
    const float a1[1] = {a}, b1[1] = {b}, c1[1] = {c}, d1[1] = {d};
    float p[1];
    stencils<CUB, false>(a1, b1, c1, d1, h, nat, p);
    return p[0];
}
// Its rank: 4 cubic, 3 quadratic, 2 linear, 1 extrapolation, 0 copy.
template <bool CUB> __device__ __forceinline__ int rank_of(const Has &h)
{
    if (CUB && h.c && (h.a || h.d))
        return h.a && h.d ? 4 : 3;
    return h.c ? 2 : (h.a ? 1 : 0);
}

// Multi-dimensional combination: the predictions of the highest rank, averaged
// in x, y, z order.
__device__ __forceinline__ float combine2(float p, int rp, float q, int rq)
{
    return rp == rq ? (p + q) * 0.5f : (rp > rq ? p : q);
}
__device__ __forceinline__ float combine3(float px, int rx, float py, int ry, float pz, int rz)
{
    const int best = max(rx, max(ry, rz));
    const bool ux = rx == best, uy = ry == best, uz = rz == best;
    if (ux && uy && uz)
        return div3((px + py) + pz);
    if (ux && uy)
        return (px + py) * 0.5f;
    if (uz && (ux || uy))
        return ((ux ? px : py) + pz) * 0.5f;
    return ux ? px : (uy ? py : pz);
}

// ---------------------------------------------------------------------------
// Linear-scaling quantization (code = 128 + q, |q| <= 127; else outlier code 0
// with the exact value kept) of n targets: xv their values, p their
// predictions; xv receives the reconstruction (the exact value of an outlier),
// b the code in its low byte, XOR 0x80.
//  - q = round-half-even((x - p) / (2 eps)): the sum with 1.5 * 2^23 rounds to
//    an integer held in the low bits, and taking 1.5 * 2^23 off again gives q
//    as a float (+0 for zero). Past 2^22 the sum is no longer that integer,
//    but stays out of range all the same.
//  - The bound holds after FP32 rounding: |x - x'| <= eps in exact arithmetic.
//    FP32 subtraction rounds monotonically and eps is an FP32 number, so the
//    rounded difference decides unless it equals eps; only then (for a lane of
//    the wave) is the difference formed in FP64, where it is exact.
// ---------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void quantize(float (&xv)[N], const float (&p)[N], uint32_t (&b)[N],
                                         const FieldQ &f)
{
    float xr[N], s[N];
    bool ok[N], eq = false;
#pragma unroll
    for (int j = 0; j < N; j++) {
        const float t = (xv[j] - p[j]) * f.inv + 12582912.0f;
        const float q = t - 12582912.0f;
        b[j] = __float_as_uint(t);
        xr[j] = p[j] + q * f.two_eb;
        s[j] = fabsf(xv[j] - xr[j]);
        const bool in = fabsf(q) <= 127.0f;
        ok[j] = in && s[j] < f.eps;
        eq |= in && s[j] == f.eps;
    }
    if (__builtin_expect(__any(eq), 0)) {
#pragma unroll
        for (int j = 0; j < N; j++)
            if (s[j] == f.eps && fabsf(__uint_as_float(b[j]) - 12582912.0f) <= 127.0f)
                ok[j] = fabs((double)xv[j] - (double)xr[j]) <= (double)f.eps;
    }
#pragma unroll
    for (int j = 0; j < N; j++) {
        xv[j] = ok[j] ? xr[j] : xv[j];
        b[j] = ok[j] ? b[j] : 0x80u;
    }
}
// Low bytes of four words, XOR 0x80 each.
__device__ __forceinline__ uint32_t pack_codes(const uint32_t (&b)[4])
{
    const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
    return (lo | hi) ^ 0x80808080u;
}
// Value of code c (1..255) at prediction p.
__device__ __forceinline__ float dequantize(float p, uint32_t c, const FieldQ &f)
{
    return p + ((float)c - 128.0f) * f.two_eb;
}

// ---------------------------------------------------------------------------
// Sub-steps. A class of points is the set c of axes (1 x, 2 y, 4 z) on which
// the coordinate is an odd multiple of the level's stride. In a sub-step of a
// level (pass 0..2) class c is interpolated along the axes use_axes(c), 0: not
// in this pass. MD: 1-D, then 2-D, then 3-D targets, along all their odd axes.
// SEQ(order): pass j interpolates along the j-th axis of the order every
// target whose last odd axis (in that order) is that axis.
// ---------------------------------------------------------------------------
struct Pass {
    bool md;
    int pass;
    int a0, a1, a2; // SEQ: the order's axes as bits
    int axis;       // SEQ: this pass's
    __device__ __forceinline__ int use(int c) const
    {
        if (md)
            return __builtin_popcount(c) == pass + 1 ? c : 0;
        const int later = pass == 0 ? a1 | a2 : (pass == 1 ? a2 : 0);
        return (c & axis) && !(c & later) ? axis : 0;
    }
    // the classes of this pass, four bits each
    __device__ __forceinline__ uint32_t classes() const
    {
        if (md)
            return pass == 0 ? 0x421u : (pass == 1 ? 0x653u : 0x7u);
        return (uint32_t)(pass == 0 ? a0
                                    : (pass == 1 ? a1 | (a0 | a1) << 4
                                                 : a2 | (a0 | a2) << 4 | (a1 | a2) << 8 | 7 << 12));
    }
};
__device__ __forceinline__ Pass make_pass(bool md, int order, int pass)
{
    // the axes (0 x, 1 y, 2 z) of the six orders, two bits each, six per order
    constexpr uint64_t kOrders = (0ull | 1ull << 2 | 2ull << 4) | (0ull | 2ull << 2 | 1ull << 4) << 6 |
                                 (1ull | 0ull << 2 | 2ull << 4) << 12 |
                                 (1ull | 2ull << 2 | 0ull << 4) << 18 |
                                 (2ull | 0ull << 2 | 1ull << 4) << 24 |
                                 (2ull | 1ull << 2 | 0ull << 4) << 30;
    const uint32_t o = (uint32_t)(kOrders >> (6 * order)) & 63u;
    Pass P;
    P.md = md;
    P.pass = pass;
    P.a0 = 1 << (o & 3u);
    P.a1 = 1 << ((o >> 2) & 3u);
    P.a2 = 1 << (o >> 4);
    P.axis = pass == 0 ? P.a0 : (pass == 1 ? P.a1 : P.a2);
    return P;
}

__device__ __forceinline__ FieldQ load_field(const FieldState *st, bool compress)
{
    FieldQ f;
    f.eps = unif(st->eps);
    f.two_eb = unif(st->two_eb);
    f.inv = compress ? unif(st->inv) : 0.f;
    const uint32_t *c = reinterpret_cast<const uint32_t *>(&st->cfg[0][0]);
    f.cfg0 = uni32(c[0]);
    f.cfg1 = uni32(c[1]);
    f.cfg2 = uni32(c[2]);
    auto use = [&](int pass) __attribute__((always_inline)) {
        const Pass S = make_pass(f.md(3), f.order(3), pass);
        uint32_t u = 0;
        for (int i = 1; i < 8; i++)
            u |= (uint32_t)S.use(i) << (4 * i);
        return uni32(u);
    };
    f.use0 = use(0);
    f.use1 = use(1);
    f.use2 = use(2);
    return f;
}

__device__ __forceinline__ void lds_read4(const float *p, float (&o)[4])
{
    const float4 v = *reinterpret_cast<const float4 *>(p);
    o[0] = v.x;
    o[1] = v.y;
    o[2] = v.z;
    o[3] = v.w;
}
__device__ __forceinline__ void lds_write4(float *p, float x, float y, float z, float w)
{
    *reinterpret_cast<float4 *>(p) = make_float4(x, y, z, w);
}

// ---------------------------------------------------------------------------
// Stride-1 level: predictions of the quad q of class C's row (xh, yh), along
// the axes U (C, or one of its axes). FULL: the tile has all its points (every
// +1 face), so a target always has its +s neighbour. The neighbours of a place
// p along an axis are the places p (-s), p + 1 (+s), p - 1 (-3s) and p + 2
// (+3s) of the class that is even on that axis. The axes are kept from
// overlapping, so that one axis's samples are in registers at a time.
// ---------------------------------------------------------------------------
template <int TZ, int NX, int C, bool CUB, bool FULL>
__device__ __forceinline__ void predict_quad(const float *__restrict__ v, int xh, int yh, int q,
                                             const Geo &g, int U, bool nat, float (&p)[4])
{
    using T = Tile<TZ, NX>;
    float px[4], py[4], pz[4];
    int rx = 0, ry = 0, rz[4];
    if ((C & 1) && (U & 1)) {
        constexpr int D = C & 6, ST = T::ny(D) * T::pitch(D);
        const float *s = v + T::template word<D>(xh, yh, 4 * q);
        const Has h = {xh >= 1, FULL || 2 * xh + 2 < g.ex, FULL ? xh <= 6 : 2 * xh + 4 < g.ex};
        float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4], c[4], d[4] = {0.f, 0.f, 0.f, 0.f};
        lds_read4(s, b);
        lds_read4(s + ST, c);
        if (CUB || !FULL)
            lds_read4(h.a ? s - ST : s, a);
        if (CUB)
            lds_read4(h.d ? s + 2 * ST : s, d);
        rx = rank_of<CUB>(h);
        stencils<CUB, FULL>(a, b, c, d, h, nat, px);
        if (CUB)
            asm volatile("" ::: "memory");
    }
    if ((C & 2) && (U & 2)) {
        constexpr int D = C & 5, ST = T::pitch(D);
        const float *s = v + T::template word<D>(xh, yh, 4 * q);
        const Has h = {yh >= 1, FULL || 2 * yh + 2 < g.ey, FULL ? yh <= 6 : 2 * yh + 4 < g.ey};
        float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4], c[4], d[4] = {0.f, 0.f, 0.f, 0.f};
        lds_read4(s, b);
        lds_read4(s + ST, c);
        if (CUB || !FULL)
            lds_read4(h.a ? s - ST : s, a);
        if (CUB)
            lds_read4(h.d ? s + 2 * ST : s, d);
        ry = rank_of<CUB>(h);
        stencils<CUB, FULL>(a, b, c, d, h, nat, py);
        if (CUB)
            asm volatile("" ::: "memory");
    }
    if ((C & 4) && (U & 4)) {
        // samples: places k - 1 .. k + 2 of target k = 4 q + j; eight targets
        // to a block, so even quads start one and odd quads end one
        constexpr int D = C & 3;
        const float *e = v + T::template word<D>(xh, yh, 4 * q);
        float e4[4];
        lds_read4(e, e4);
        const bool lastq = D != 0 && q == T::NQ - 1;
        const float up = *(lastq ? v + T::template fword<D>(xh, yh) : e + 4);
        float dn = 0.f, up2 = 0.f;
        if (CUB || !FULL)
            dn = e[q > 0 ? -1 : 0];
        if (CUB)
            up2 = e[(q & 1) ? 0 : 5];
        const float a4[4] = {dn, e4[0], e4[1], e4[2]}, c4[4] = {e4[1], e4[2], e4[3], up},
                    d4[4] = {e4[2], e4[3], up, up2};
        const int z0 = 8 * q + 1, hi = min((z0 & ~15) + 16, g.ez - 1);
        float m[4];
        if (CUB)
            mid(a4, e4, c4, d4, nat, m);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int z = z0 + 2 * j;
            Has h;
            h.a = j > 0 || (q & 1);
            h.c = FULL || z + 1 <= hi;
            h.d = FULL ? (j < 3 || !(q & 1)) : z + 3 <= hi;
            rz[j] = rank_of<CUB>(h);
            pz[j] = CUB && h.a && h.c && h.d ? m[j]
                                             : stencil_low<CUB, FULL>(a4[j], e4[j], c4[j], d4[j], h);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
        if constexpr (C == 1)
            p[j] = px[j];
        else if constexpr (C == 2)
            p[j] = py[j];
        else if constexpr (C == 4)
            p[j] = pz[j];
        else if (U == C) {
            if constexpr (C == 3)
                p[j] = combine2(px[j], rx, py[j], ry);
            else if constexpr (C == 5)
                p[j] = combine2(px[j], rx, pz[j], rz[j]);
            else if constexpr (C == 6)
                p[j] = combine2(py[j], ry, pz[j], rz[j]);
            else
                p[j] = combine3(px[j], rx, py[j], ry, pz[j], rz[j]);
        } else {
            p[j] = (C & 1) && (U & 1) ? px[j] : ((C & 2) && (U & 2) ? py[j] : pz[j]);
        }
    }
}

// Keeps what is computed from v from being moved out of the tile loop, where
// every address would hold a register across all tiles.
__device__ __forceinline__ void opaque(int &v) { asm volatile("" : "+v"(v)); }

// A thread's place in the tile: quad q of the rows at (ix, iy) of every class,
// the same quad of a far-face row at (fx, fy) of class fc (0: even x and y, 1: x
// odd, 2: y odd; 3: none), and far z face points (x / 2, y / 2 and class in four
// bits each; class 15: none). Kept packed across tiles (PlaceBits), taken
// apart where it is used.
template <int TZ, int NX> struct Place {
    using T = Tile<TZ, NX>;
    int q, ix, iy, fx, fy, fc;
    int frow[T::IF];
};
template <int TZ, int NX> struct PlaceBits {
    using T = Tile<TZ, NX>;
    int t, far;
    int frow[T::IF];
    __device__ __forceinline__ explicit PlaceBits(int thread) : t(thread)
    {
        const int r = t / T::NQ;
        if (T::FLAT)
            far = 0 | 8 << 4 | (r == 0 ? 0 : 3) << 8;
        else if (r < 9)
            far = 8 | r << 4;
        else if (r < 17)
            far = (r - 9) | 8 << 4;
        else if (r < 25)
            far = 8 | (r - 17) << 4 | 2 << 8;
        else
            far = ((r - 25) & 7) | 8 << 4 | (r < 33 ? 1 : 3) << 8;
#pragma unroll
        for (int k = 0; k < T::IF; k++) {
            const int i = t + T::NT * k;
            int x, y, c;
            if (T::FLAT) {
                x = 0;
                y = i < 8 ? i : i - 8;
                c = i < 8 ? 2 : 0;
            } else if (i < 72) {
                x = i / 8;
                y = i % 8;
                c = 2;
            } else if (i < 144) {
                x = (i - 72) / 9;
                y = (i - 72) % 9;
                c = 1;
            } else if (i < 208) {
                x = (i - 144) / 8;
                y = (i - 144) % 8;
                c = 3;
            } else {
                x = (i - 208) / 9;
                y = (i - 208) % 9;
                c = 0;
            }
            frow[k] = x | (y << 4) | ((i < T::NR ? c : 15) << 8);
        }
    }
    // opaque copies: nothing computed from them is moved out of the tile loop
    __device__ __forceinline__ Place<TZ, NX> get() const
    {
        int a = t, b = far;
        opaque(a);
        opaque(b);
        Place<TZ, NX> p;
        p.q = a % T::NQ;
        p.iy = (a / T::NQ) % 8;
        p.ix = a / (8 * T::NQ);
        p.fx = b & 15;
        p.fy = (b >> 4) & 15;
        p.fc = b >> 8;
#pragma unroll
        for (int k = 0; k < T::IF; k++) {
            p.frow[k] = frow[k];
            opaque(p.frow[k]);
        }
        return p;
    }
};
// Full coordinates and word of a far z face point.
struct FacePoint {
    int xh, yh, c, x, y;
    __device__ __forceinline__ explicit FacePoint(int r)
        : xh(r & 15), yh((r >> 4) & 15), c(r >> 8), x(2 * (r & 15) + ((r >> 8) & 1)),
          y(2 * ((r >> 4) & 15) + ((r >> 9) & 1))
    {
    }
};
template <int TZ, int NX> __device__ __forceinline__ int face_word(const FacePoint &p)
{
    using T = Tile<TZ, NX>;
    return p.c == 0 ? T::template fword<0>(p.xh, p.yh)
                    : (p.c == 1 ? T::template fword<1>(p.xh, p.yh)
                                : (p.c == 2 ? T::template fword<2>(p.xh, p.yh)
                                            : T::template fword<3>(p.xh, p.yh)));
}

// The prediction of a point of the far z face along axes U (x and y only).
template <int TZ, int NX, bool CUB>
__device__ __forceinline__ float predict_face(const float *__restrict__ v, const FacePoint &P,
                                              const Geo &g, int U, bool nat)
{
    using T = Tile<TZ, NX>;
    float px = 0.f, py = 0.f;
    int rx = -1, ry = -1;
    if (U & 1) {
        // the class that is even on x: 0 or 2
        const float *s = v + ((P.c & 2) ? T::template fword<2>(P.xh, P.yh) : T::template fword<0>(P.xh, P.yh));
        const int st = (P.c & 2) ? 8 : T::LXS;
        const Has h = {P.x >= 3, P.x + 1 < g.ex, P.x + 3 < g.ex};
        rx = rank_of<CUB>(h);
        px = stencil<CUB>(s[h.a ? -st : 0], s[0], s[h.c ? st : 0], s[h.d ? 2 * st : 0], h, nat);
    }
    if (U & 2) {
        const float *s = v + ((P.c & 1) ? T::template fword<1>(P.xh, P.yh) : T::template fword<0>(P.xh, P.yh));
        const int st = (P.c & 1) ? 1 : T::LP;
        const Has h = {P.y >= 3, P.y + 1 < g.ey, P.y + 3 < g.ey};
        ry = rank_of<CUB>(h);
        py = stencil<CUB>(s[h.a ? -st : 0], s[0], s[h.c ? st : 0], s[h.d ? 2 * st : 0], h, nat);
    }
    return combine2(px, rx, py, ry);
}

// The codes of a thread's rows: words of four codes per class (class 0, the
// lattice, only for the stores), its face-row quads (even and odd z) and
// far-face points.
template <int TZ, int NX> struct RowCodes {
    uint32_t own[8];
    uint32_t fe, fo;
    uint32_t face[Tile<TZ, NX>::IF];
};

// One class of the stride-1 level: the quads of the thread's own row and, for
// the classes that the far x and y faces hold, of its face row.
template <int TZ, int NX, int C, bool CUB, bool FULL, bool COMP>
__device__ __forceinline__ void level1_class(float *__restrict__ v, const PlaceBits<TZ, NX> &P0,
                                             RowCodes<TZ, NX> &rc, const Geo &g, int U, bool keep,
                                             bool nat, const FieldQ &f)
{
    using T = Tile<TZ, NX>;
    constexpr bool ODDZ = (C & 4) != 0;
    constexpr bool FACES = (C & 3) != 3 && !(T::FLAT && (C & 3) != 0);
#pragma unroll 1
    for (int e = 0; e < (FACES ? 2 : 1); e++) {
        const Place<TZ, NX> P = P0.get();
        const int xh = e == 0 ? P.ix : P.fx, yh = e == 0 ? P.iy : P.fy, q = P.q;
        bool on = e == 0 || P.fc == (C & 3);
        if (!FULL)
            on = on && 2 * xh + (C & 1) < g.ex && 2 * yh + ((C >> 1) & 1) < g.ey && 8 * q < g.ez;
        if (!on)
            continue;
        float p[4], xv[4];
        predict_quad<TZ, NX, C, CUB, FULL>(v, xh, yh, q, g, U, nat, p);
        float *dst = v + T::template word<C>(xh, yh, 4 * q);
        lds_read4(dst, xv);
        if constexpr (COMP) {
            uint32_t b[4];
            quantize(xv, p, b, f);
            if (keep)
                lds_write4(dst, xv[0], xv[1], xv[2], xv[3]);
            if (e == 0)
                rc.own[C] = pack_codes(b);
        } else {
            // code 0: the exact outlier value already in place is kept
            const uint32_t w = e == 0 ? rc.own[C] : (ODDZ ? rc.fo : rc.fe);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint32_t c = (w >> (8 * j)) & 255u;
                const float y4 = dequantize(p[j], c, f);
                xv[j] = c != 0 ? y4 : xv[j];
            }
            lds_write4(dst, xv[0], xv[1], xv[2], xv[3]);
        }
    }
}

template <int TZ, int NX, bool CUB, bool FULL, bool COMP>
__device__ __forceinline__ void level1(float *__restrict__ v, const PlaceBits<TZ, NX> &P0,
                                       RowCodes<TZ, NX> &rc, const Geo &g, const FieldQ &f)
{
    using T = Tile<TZ, NX>;
    const bool nat = f.spline(3) == 2;
#pragma unroll 1
    for (int pass = 0; pass < 3; pass++) {
        const uint32_t use = pick(pass, f.use0, f.use1, f.use2);
        // compression: no later sub-step reads the last one's targets
        const bool keep = pass < 2;
#define HIZ_CLASS(C)                                                                              \
    if constexpr (!(T::FLAT && ((C)&1)))                                                          \
        if (const int U = (int)(use >> (4 * C)) & 7)                                                               \
            level1_class<TZ, NX, C, CUB, FULL, COMP>(v, P0, rc, g, U, keep, nat, f);
        HIZ_CLASS(4)
        HIZ_CLASS(2)
        HIZ_CLASS(6)
        HIZ_CLASS(1)
        HIZ_CLASS(5)
        HIZ_CLASS(3)
        HIZ_CLASS(7)
#undef HIZ_CLASS
        // the far z face's own targets: even z, so along x and y only
        const int U1 = (use >> 4) & 7, U2 = (use >> 8) & 7, U3 = (use >> 12) & 7;
        if (g.ez == 16 * TZ + 1 && (U1 | U2 | U3)) {
#pragma unroll
            for (int k = 0; k < T::IF; k++) {
                int fr = P0.frow[k];
                opaque(fr);
                const FacePoint F(fr);
                const int U = F.c == 1 ? U1 : (F.c == 2 ? U2 : (F.c == 3 ? U3 : 0));
                if (U == 0 || F.x >= g.ex || F.y >= g.ey)
                    continue;
                float p[1] = {predict_face<TZ, NX, CUB>(v, F, g, U, nat)};
                float *dst = v + face_word<TZ, NX>(F);
                if constexpr (COMP) {
                    float xv[1] = {*dst};
                    uint32_t b[1];
                    quantize(xv, p, b, f);
                    *dst = xv[0];
                } else {
                    const uint32_t code = rc.face[k] & 255u;
                    if (code != 0)
                        *dst = dequantize(p[0], code, f);
                }
            }
        }
        if (pass < 2)
            lds_barrier();
    }
}

// ---------------------------------------------------------------------------
// Levels of stride 8, 4 and 2 on the lattice of even points (half the
// coordinates: strides 4, 2, 1; a line's samples exist on the lattice exactly
// when they exist in the tile), one target per lane. lc: codes of the lattice
// points: of the owned ones in compression (a word per thread: KZ bytes for
// each of the 8 x 8 (x, y), the anchors' bytes free for codes that nobody
// needs), at their lattice words in decompression.
// ---------------------------------------------------------------------------
// The prediction along one axis: A the target's word, st the words from one
// sample's place to the next (the samples are one st either side, and three).
template <bool CUB, bool FULL>
__device__ __forceinline__ float predict_axis(const float *__restrict__ v, int A, int st,
                                              const Has &h, bool nat, int &rank)
{
    const float b = v[A - st], c = v[FULL || h.c ? A + st : A - st];
    float a = 0.f, d = 0.f;
    if (CUB || !FULL)
        a = v[h.a ? A - 3 * st : A - st];
    if (CUB)
        d = v[h.d ? A + 3 * st : A - st];
    rank = rank_of<CUB>(h);
    return stencil<CUB>(a, b, c, d, h, nat);
}
// The value at lattice word A; ci: where its code is.
template <bool COMP>
__device__ __forceinline__ void coarse_value(float *__restrict__ v, uint8_t *__restrict__ lc, int A,
                                             int ci, float pred, const FieldQ &f)
{
    float xv[1] = {v[A]}, p[1] = {pred};
    if constexpr (COMP) {
        uint32_t b[1];
        quantize(xv, p, b, f);
        v[A] = xv[0];
        lc[ci] = (uint8_t)(b[0] ^ 0x80u);
    } else {
        // code 0: the exact outlier value already in place is kept
        const uint32_t code = lc[ci];
        const float y = dequantize(pred, code, f);
        v[A] = code != 0 ? y : xv[0];
    }
}

// Which targets a thread takes in each pass of the three levels depends on the
// field's configuration alone, so each is worked out once per field by every
// workgroup and kept across its tiles (15 words per thread; k_predict has no
// registers left for all of them): targets i = t, t + NT, ... of the pass's classes
// one after the other, as a tile with all its points has them. Bits 0..11: the target's lattice
// word (0, an anchor: no target); 12..14: its class, or the one axis used; from
// bit 15 on, per axis used, whether the samples three steps before and after
// exist; 21..31: where its code goes in compression.
template <int TZ, int NX> struct CoarsePlan {
    using T = Tile<TZ, NX>;
    // targets per thread and pass on the level of stride 2 (the coarser levels: one)
    static constexpr int slots(int pass) { return pass == 1 && !T::FLAT ? 2 : 3; }
    uint32_t d0[3], d1[3], d2[3][3];

    // a / b for 0 <= a < 2^12, 0 < b <= 64: (a + 1/2) / b is at least 1 / 128 off a
    // whole number, far more than the two roundings
    static __device__ __forceinline__ int small_div(int a, int b)
    {
        return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
    }
    static __device__ __forceinline__ uint32_t target(bool md, int order, int l, int pass, int i)
    {
        const int lh = 2 - l;
        const Pass S = make_pass(md, order, pass);
        const int mx = T::FLAT ? 1 : (8 >> lh) + 1, my = (8 >> lh) + 1, mz = (T::KZ >> lh) + 1;
        // the class this target lies in, and its number there: the same steps for
        // every lane, so that counts stay scalar, and no integer division (a lane
        // at a time through the search, with two of them, a workgroup took 3 us
        // longer per field: 64^3 k_predict 38 us, this way 35; 24 fields of sides
        // 32..160 168, this way 158)
        int c = 0, r = -1, first = 0;
        for (uint32_t list = S.classes(); list; list >>= 4) {
            const int k = list & 7;
            const int n = ((mx + 1 - (k & 1)) >> 1) * ((my + 1 - ((k >> 1) & 1)) >> 1) *
                          ((mz + 1 - (k >> 2)) >> 1);
            if (i >= first && i < first + n) {
                c = k;
                r = i - first;
            }
            first += n;
        }
        if (r < 0)
            return 0;
        const int ny = (my + 1 - ((c >> 1) & 1)) >> 1, nz = (mz + 1 - (c >> 2)) >> 1;
        const int xy = small_div(r, nz), kx = small_div(xy, ny);
        // places on the level's grid
        const int q[3] = {2 * kx + (c & 1), 2 * (xy - kx * ny) + ((c >> 1) & 1),
                          2 * (r - xy * nz) + (c >> 2)};
        const int u = S.md ? c : S.axis;
        uint32_t d = (uint32_t)((q[0] * T::LXS + q[1] * T::LP + q[2]) << lh) | (uint32_t)u << 12;
        const int x = q[0] << lh, y = q[1] << lh, z = q[2] << lh;
        if (x < 8 && y < 8 && z < T::KZ)
            d |= (uint32_t)((x * 8 + y) * T::KZ + z) << 21;
        int bit = 15;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            if (!((u >> k) & 1))
                continue;
            const int in = q[k] & ((8 >> lh) - 1); // in its block
            d |= (uint32_t)(in >= 3) << bit | (uint32_t)(in + 3 <= (8 >> lh)) << (bit + 1);
            bit += 2;
        }
        return d;
    }
    __device__ __forceinline__ void make(const FieldQ &f, int t)
    {
        // one loop over all targets, so that the search above is there once
#pragma unroll 1
        for (int n = 0; n < 15; n++) {
            const int l = n < 3 ? 0 : (n < 6 ? 1 : 2), pass = n < 6 ? n % 3 : (n - 6) % 3,
                      k = n < 6 ? 0 : (n - 6) / 3;
            const uint32_t d = target(f.md(l), f.order(l), l, pass, t + T::NT * k);
#pragma unroll
            for (int p = 0; p < 3; p++) {
                d0[p] = n == p ? d : d0[p];
                d1[p] = n == 3 + p ? d : d1[p];
#pragma unroll
                for (int j = 0; j < 3; j++)
                    d2[p][j] = n == 6 + 3 * j + p ? d : d2[p][j];
            }
        }
    }
};

// Lattice coordinates of a target and the last lattice points of its tile: which
// samples exist in a tile that lacks points follows from these.
struct LatticePoint {
    int x, y, z, lx, ly, lz;
    __device__ __forceinline__ bool inside() const { return x <= lx && y <= ly && z <= lz; }
    __device__ __forceinline__ Has has(int axis, int h) const
    {
        if (axis == 4) {
            const int zb = z & 7, hi = min(8, lz - (z & ~7));
            return Has{zb >= 3 * h, zb + h <= hi, zb + 3 * h <= hi};
        }
        const int c = axis == 1 ? x : y, l = axis == 1 ? lx : ly;
        return Has{c >= 3 * h, c + h <= l, c + 3 * h <= l};
    }
};

// One planned target interpolated along AX axes; lh: log2 of the lattice step.
template <int TZ, int NX, int AX, bool CUB, bool FULL>
__device__ __forceinline__ float coarse_predict(const float *__restrict__ v, uint32_t d, int lh,
                                                const LatticePoint &L, bool nat)
{
    using T = Tile<TZ, NX>;
    const int A = d & 0xfff, c = (d >> 12) & 7;
    // samples of the k-th axis used
    auto has = [&](int k, int axis) __attribute__((always_inline)) {
        return FULL ? Has{((d >> (15 + 2 * k)) & 1) != 0, true, ((d >> (16 + 2 * k)) & 1) != 0}
                    : L.has(axis, 1 << lh);
    };
    int r0, r1, r2;
    if constexpr (AX == 1) {
        const int st = (c == 1 ? T::LXS : (c == 2 ? T::LP : 1)) << lh;
        return predict_axis<CUB, FULL>(v, A, st, has(0, c), nat, r0);
    } else if constexpr (AX == 2) {
        const float p =
            predict_axis<CUB, FULL>(v, A, (c == 6 ? T::LP : T::LXS) << lh, has(0, c == 6 ? 2 : 1), nat, r0);
        const float q =
            predict_axis<CUB, FULL>(v, A, (c == 3 ? T::LP : 1) << lh, has(1, c == 3 ? 2 : 4), nat, r1);
        return combine2(p, r0, q, r1);
    } else {
        const float p = predict_axis<CUB, FULL>(v, A, T::LXS << lh, has(0, 1), nat, r0);
        const float q = predict_axis<CUB, FULL>(v, A, T::LP << lh, has(1, 2), nat, r1);
        const float s = predict_axis<CUB, FULL>(v, A, 1 << lh, has(2, 4), nat, r2);
        return combine3(p, r0, q, r1, s, r2);
    }
}
template <int TZ, int NX, int AX, bool FULL, bool COMP>
__device__ __forceinline__ void coarse_target(float *__restrict__ v, uint8_t *__restrict__ lc,
                                              uint32_t d, int lh, bool cub, bool nat, const Geo &g,
                                              const FieldQ &f)
{
    using T = Tile<TZ, NX>;
    const int A = d & 0xfff;
    bool on = A != 0;
    LatticePoint L{};
    if constexpr (!FULL) {
        const int r = A / T::LP;
        L = LatticePoint{r / 9, r % 9, A % T::LP, (g.ex - 1) >> 1, (g.ey - 1) >> 1, (g.ez - 1) >> 1};
        on = on && L.inside();
    }
    if (on) {
        const float p = cub ? coarse_predict<TZ, NX, AX, true, FULL>(v, d, lh, L, nat)
                            : coarse_predict<TZ, NX, AX, false, FULL>(v, d, lh, L, nat);
        coarse_value<COMP>(v, lc, A, COMP ? (int)(d >> 21) : A, p, f);
    }
}
// N targets of a pass: in the multi-dimensional scheme along pass + 1 axes.
template <int TZ, int NX, int PASS, int N, bool FULL, bool COMP>
__device__ __forceinline__ void coarse_pass(float *__restrict__ v, uint8_t *__restrict__ lc,
                                            const uint32_t (&d)[N], int l, const Geo &g,
                                            const FieldQ &f)
{
    const int spline = f.spline(l), lh = 2 - l;
    if (PASS == 0 || !f.md(l)) {
#pragma unroll
        for (int k = 0; k < N; k++)
            coarse_target<TZ, NX, 1, FULL, COMP>(v, lc, d[k], lh, spline != 0, spline == 2, g, f);
    } else {
        // three axes: one class, at most NT targets
#pragma unroll
        for (int k = 0; k < (PASS == 2 ? 1 : N); k++)
            coarse_target<TZ, NX, PASS + 1, FULL, COMP>(v, lc, d[k], lh, spline != 0, spline == 2, g, f);
    }
    lds_barrier();
}

template <int TZ, int NX, bool FULL, bool COMP>
__device__ __forceinline__ void coarse_levels(float *__restrict__ v, uint8_t *__restrict__ lc,
                                              const CoarsePlan<TZ, NX> &C, const Geo &g,
                                              const FieldQ &f)
{
    uint32_t p0[1] = {C.d0[0]}, p1[1] = {C.d0[1]}, p2[1] = {C.d0[2]};
#pragma unroll 1
    for (int l = 0; l < 2; l++) {
        coarse_pass<TZ, NX, 0, 1, FULL, COMP>(v, lc, p0, l, g, f);
        coarse_pass<TZ, NX, 1, 1, FULL, COMP>(v, lc, p1, l, g, f);
        coarse_pass<TZ, NX, 2, 1, FULL, COMP>(v, lc, p2, l, g, f);
        p0[0] = C.d1[0];
        p1[0] = C.d1[1];
        p2[0] = C.d1[2];
    }
    constexpr int S1 = CoarsePlan<TZ, NX>::slots(1);
    uint32_t q1[S1];
#pragma unroll
    for (int k = 0; k < S1; k++)
        q1[k] = C.d2[1][k];
    coarse_pass<TZ, NX, 0, 3, FULL, COMP>(v, lc, C.d2[0], 2, g, f);
    coarse_pass<TZ, NX, 1, S1, FULL, COMP>(v, lc, q1, 2, g, f);
    coarse_pass<TZ, NX, 2, 3, FULL, COMP>(v, lc, C.d2[2], 2, g, f);
}

// All four levels of a tile.
template <int TZ, int NX, bool FULL, bool COMP>
__device__ __forceinline__ void walk_levels(float *__restrict__ v, uint8_t *__restrict__ lc,
                                            const PlaceBits<TZ, NX> &P0, RowCodes<TZ, NX> &rc,
                                            const CoarsePlan<TZ, NX> &C, const Geo &g,
                                            const FieldQ &f)
{
    coarse_levels<TZ, NX, FULL, COMP>(v, lc, C, g, f);
    if (f.spline(3) != 0)
        level1<TZ, NX, true, FULL, COMP>(v, P0, rc, g, f);
    else
        level1<TZ, NX, false, FULL, COMP>(v, P0, rc, g, f);
}

// ---------------------------------------------------------------------------
// Tiles
// ---------------------------------------------------------------------------
struct TilePos {
    uint64_t base;  // field index of the tile's first point
    uint64_t sx, dz;
    uint32_t bx, by, bz;
    Geo g;
    bool whole; // every piece of eight along z that starts in the tile ends in the field
};
template <int TZ> __device__ __forceinline__ TilePos tile_pos(const Job &J, uint64_t lt)
{
    // a launch holds fewer than 2^32 tiles: 32-bit division
    const uint32_t l = (uint32_t)lt;
    const uint32_t tz = l % J.ntz, r = l / J.ntz;
    TilePos P;
    P.by = r % J.nb[1];
    P.bx = r / J.nb[1];
    P.bz = tz * TZ;
    const uint64_t ox = (uint64_t)P.bx * kAnchor, oy = (uint64_t)P.by * kAnchor,
                   oz = (uint64_t)P.bz * kAnchor;
    const uint64_t dy = J.dims[1];
    P.dz = J.dims[2];
    P.sx = dy * P.dz;
    P.base = (ox * dy + oy) * P.dz + oz;
    Geo &g = P.g;
    g.ex = (int)min<uint64_t>(kSide, J.dims[0] - ox);
    g.ey = (int)min<uint64_t>(kSide, dy - oy);
    g.ez = (int)min<uint64_t>(16 * TZ + 1, P.dz - oz);
    g.ownx = min(g.ex, 16);
    g.owny = min(g.ey, 16);
    g.ownz = min(g.ez, 16 * TZ);
    P.whole = P.base + (uint64_t)(g.ex - 1) * P.sx + (uint64_t)(g.ey - 1) * P.dz + 16 * TZ <= J.N;
    return P;
}
template <int TZ, int NX> __device__ __forceinline__ bool tile_full(const Geo &g)
{
    return g.ex == Tile<TZ, NX>::SX && g.ey == kSide && g.ez == 16 * TZ + 1;
}

// Tiles of a workgroup. Each XCD (workgroups are dealt to the eight XCDs
// round-robin by blockIdx) owns a contiguous eighth of the list, so tiles that
// share halo faces meet in the same L2, and its W workgroups take W neighbouring
// tiles at a time. From one such round to the next a workgroup's place shifts by
// about 0.38 W: places a whole number of rows apart (W is often a multiple of
// the tiles along z) hold the slower tiles, cut by the field's far end, in
// every round, and without the shift the same workgroups would take them all
// (512^3: 448 us of k_reconstruct against 326). Claiming tiles from a counter
// balances no better and costs small launches a round trip per workgroup and
// exhausted eighth (16 M points: 90 us against 123).
struct TileWalk {
    uint64_t lo;            // the group's first tile
    uint32_t n, w, at, round; // its tiles and workgroups; this workgroup's place, start of the round
    __device__ __forceinline__ bool done() const { return round + at >= n; }
    __device__ __forceinline__ uint64_t tile() const { return lo + round + at; }
    __device__ __forceinline__ void step()
    {
        round += w;
        at += (w * 98 >> 8) | 1;
        at = at >= w ? at - w : at;
    }
};
__device__ __forceinline__ TileWalk tile_walk(uint64_t lo, uint64_t hi)
{
    const int lg = (gridDim.x & 7) == 0 ? 3 : 0;
    const uint64_t x = lg ? blockIdx.x & 7 : 0;
    TileWalk t;
    t.lo = lo + ((hi - lo) * x >> lg);
    t.n = (uint32_t)(lo + ((hi - lo) * (x + 1) >> lg) - t.lo);
    t.w = gridDim.x >> lg;
    t.at = blockIdx.x >> lg;
    t.round = 0;
    return t;
}

// Unaligned pieces: rows start at any multiple of four bytes (values) or at
// any byte (codes).
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u2_any __attribute__((ext_vector_type(2), aligned(1)));

// Eight consecutive values at field index `off`; past the field's end (points
// that no tile holds) its last value. whole: the same for the wave.
__device__ __forceinline__ void load_row8(float (&e)[8], HIZ_GLOBAL const float *p, uint64_t off,
                                          bool whole, uint64_t N)
{
    if (whole) {
        const f4_any a = *(HIZ_GLOBAL const f4_any *)(p + off);
        const f4_any b = *(HIZ_GLOBAL const f4_any *)(p + off + 4);
        e[0] = a.x;
        e[1] = a.y;
        e[2] = a.z;
        e[3] = a.w;
        e[4] = b.x;
        e[5] = b.y;
        e[6] = b.z;
        e[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < 8; j++)
            e[j] = p[min(off + j, N - 1)];
    }
}
// A row's eight values into its two classes (D: the class of even z).
template <int TZ, int NX, int D>
__device__ __forceinline__ void put_row8(float *v, int xh, int yh, int q, const float (&e)[8])
{
    using T = Tile<TZ, NX>;
    lds_write4(v + T::template word<D>(xh, yh, 4 * q), e[0], e[2], e[4], e[6]);
    lds_write4(v + T::template word<(D | 4)>(xh, yh, 4 * q), e[1], e[3], e[5], e[7]);
}
// The same for a far-face row of class P.fc.
template <int TZ, int NX>
__device__ __forceinline__ void put_face8(float *v, const Place<TZ, NX> &P, const float (&e)[8])
{
    if (P.fc == 0)
        put_row8<TZ, NX, 0>(v, P.fx, P.fy, P.q, e);
    if constexpr (NX != 1) {
        if (P.fc == 1)
            put_row8<TZ, NX, 1>(v, P.fx, P.fy, P.q, e);
        else if (P.fc == 2)
            put_row8<TZ, NX, 2>(v, P.fx, P.fy, P.q, e);
    }
}
// Calls f(class) for the thread's own rows: classes 0, 2 (and 1, 3).
template <int NX, typename F> __device__ __forceinline__ void own_rows(F &&f)
{
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 2>{});
    if constexpr (NX != 1) {
        f(std::integral_constant<int, 1>{});
        f(std::integral_constant<int, 3>{});
    }
}
// Field index of a thread's own row of class 0; the row of class D follows at
// + (D & 1) * sx + (D >> 1) * dz.
template <int TZ, int NX>
__device__ __forceinline__ uint64_t own_offset(const TilePos &tp, const Place<TZ, NX> &P)
{
    return tp.base + (uint64_t)(2 * P.ix) * tp.sx + (uint64_t)(2 * P.iy) * tp.dz + 8 * P.q;
}
template <int D> __device__ __forceinline__ uint64_t row_step(const TilePos &tp)
{
    return ((D & 1) ? tp.sx : 0) + ((D & 2) ? tp.dz : 0);
}
template <int TZ, int NX>
__device__ __forceinline__ uint64_t face_offset(const TilePos &tp, const Place<TZ, NX> &P)
{
    return tp.base + (uint64_t)(2 * P.fx + (P.fc & 1)) * tp.sx +
           (uint64_t)(2 * P.fy + ((P.fc >> 1) & 1)) * tp.dz + 8 * P.q;
}
// Whether the thread's own row of class D, its face row, lie in the extents.
template <int TZ, int NX, int D>
__device__ __forceinline__ bool own_in(const Place<TZ, NX> &P, int ex, int ey)
{
    return 2 * P.ix + (D & 1) < ex && 2 * P.iy + (D >> 1) < ey;
}
template <int TZ, int NX>
__device__ __forceinline__ bool face_in(const Place<TZ, NX> &P, const Geo &g)
{
    return P.fc != 3 && 2 * P.fx + (P.fc & 1) < g.ex && 2 * P.fy + (P.fc >> 1) < g.ey && 8 * P.q < g.ez;
}

// A tile's values as a thread holds them ahead of their use.
template <int TZ, int NX> struct TileRegs {
    using T = Tile<TZ, NX>;
    float own[4][8]; // by class
    float ext[8];
    float face[T::IF];
};
template <int TZ, int NX>
__device__ __forceinline__ void tile_fetch(TileRegs<TZ, NX> &r, const Job &J, const TilePos &tp,
                                           const Place<TZ, NX> &P)
{
    using T = Tile<TZ, NX>;
    HIZ_GLOBAL const float *src = gmem(J.field);
    const bool full = tile_full<TZ, NX>(tp.g);
    const bool zin = 8 * P.q < tp.g.ez;
    const uint64_t o0 = own_offset(tp, P);
    own_rows<NX>([&](auto d) __attribute__((always_inline)) {
        constexpr int D = decltype(d)::value;
        if (full || (zin && own_in<TZ, NX, D>(P, tp.g.ex, tp.g.ey)))
            load_row8(r.own[D], src, o0 + row_step<D>(tp), tp.whole, J.N);
    });
    if (face_in(P, tp.g))
        load_row8(r.ext, src, face_offset(tp, P), tp.whole, J.N);
    if (tp.g.ez == 16 * TZ + 1) {
#pragma unroll
        for (int k = 0; k < T::IF; k++) {
            const FacePoint F(P.frow[k]);
            if (F.c != 15 && F.x < tp.g.ex && F.y < tp.g.ey)
                r.face[k] = src[tp.base + F.x * tp.sx + F.y * tp.dz + 16 * TZ];
        }
    }
}

// ---------------------------------------------------------------------------
// Compression: predict + quantize + histogram, persistent over tiles. A tile's
// values are loaded when its turn comes, the three other workgroups of the
// compute unit at work meanwhile: held ahead of time in registers (42 more) they
// make it spill that much more (512^3: 784 us; at three waves per SIMD 541;
// without 435).
// ---------------------------------------------------------------------------
template <int TZ, int NX>
__global__ __launch_bounds__((Tile<TZ, NX>::NT), 4) void k_predict(const Job *__restrict__ jobs,
                                                                 int njobs, uint64_t lo,
                                                                 uint64_t hi)
{
    using T = Tile<TZ, NX>;
    __shared__ __align__(16) float v[T::NV];
    __shared__ __align__(4) uint8_t lc[T::OX * 8 * T::KZ];
    // a tile's histogram: two 16-bit counts per word (a tile holds at most
    // 16384 codes), taken over into registers after each tile. Code k shares a
    // word with k + 128, so that the frequent codes around 128 lie in words of
    // their own (k beside k + 1: 1800 x 3600 203 us instead of 117).
    __shared__ uint32_t hist[128];
    __shared__ uint32_t red[2 * T::NW < 8 ? 8 : 2 * T::NW];
    constexpr int HW = T::NT >= 128 ? 1 : 2; // histogram words per thread
    const int t = threadIdx.x;
    uint32_t cnt[HW][2];
#pragma unroll
    for (int k = 0; k < HW; k++) {
        cnt[k][0] = cnt[k][1] = 0;
        if (t + k * T::NT < 128)
            hist[t + k * T::NT] = 0;
    }
    // after a barrier behind a tile's counting
    auto take_hist = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < HW; k++)
            if (t + k * T::NT < 128) {
                const uint32_t n = hist[t + k * T::NT];
                hist[t + k * T::NT] = 0;
                cnt[k][0] += n & 0xffffu;
                cnt[k][1] += n >> 16;
            }
    };
    auto flush = [&](int job) __attribute__((always_inline)) {
        unsigned long long *h = (unsigned long long *)jobs[job].st->hist;
#pragma unroll
        for (int k = 0; k < HW; k++)
#pragma unroll
            for (int b = 0; b < 2; b++) {
                if (cnt[k][b])
                    atomicAdd(&h[t + k * T::NT + 128 * b], (unsigned long long)cnt[k][b]);
                cnt[k][b] = 0;
            }
    };
    auto count = [&](uint32_t code) __attribute__((always_inline)) {
        atomicAdd(&hist[code & 127], 1u << (16 * (code >> 7)));
    };
    const PlaceBits<TZ, NX> P0(t);
    TileWalk w = tile_walk(lo, hi);
    TileRegs<TZ, NX> r;
    FieldQ f;
    int cur = -1;
    bool skip = false;
    CoarsePlan<TZ, NX> plan;
    for (; !w.done(); w.step()) {
        const uint64_t u = w.tile();
        lds_barrier(); // every wave is done with the previous tile's values and codes
        take_hist();
        const int ji = find_job<WK_TILE>(jobs, njobs, u);
        const Job &J = jobs[ji];
        if (ji != cur) {
            if (cur >= 0)
                flush(cur);
            cur = ji;
            // The waves have to agree, or their barriers pair up wrongly from
            // here on, into the next field's tiles. With a relative bound the
            // flags are final; with an absolute one this launch sets them while
            // other waves would read them, so the field is walked to its end
            // (values that are not finite become outliers of a result that is
            // then refused).
            skip = J.mode != 0 && (uni32(J.st->flags) & (ST_CONST | ST_NONFINITE)) != 0;
            f = load_field(J.st, true);
            plan.make(f, t);
        }
        if (skip)
            continue;
        const TilePos tp = tile_pos<TZ>(J, u - J.tile_begin);
        const Geo &g = tp.g;
        const bool full = tile_full<TZ, NX>(g);
        const Place<TZ, NX> P = P0.get();
        tile_fetch(r, J, tp, P);
        // the tile (with its +1 faces) into LDS
        own_rows<NX>([&](auto d) __attribute__((always_inline)) {
            constexpr int D = decltype(d)::value;
            put_row8<TZ, NX, D>(v, P.ix, P.iy, P.q, r.own[D]);
        });
        put_face8(v, P, r.ext);
#pragma unroll
        for (int k = 0; k < T::IF; k++) {
            const FacePoint F(P.frow[k]);
            if (F.c != 15)
                v[face_word<TZ, NX>(F)] = r.face[k];
        }
        // anchors: local (0, 0, 16j), stored raw (the levels never write them)
        if (P.ix == 0 && P.iy == 0 && (P.q & 1) == 0 && 8 * P.q < g.ownz) {
            const uint64_t ai = ((uint64_t)tp.bx * J.nb[1] + tp.by) * J.nb[2] + tp.bz + (P.q >> 1);
            const uint64_t off = J.off_anchors + 4 * ai;
            if (off + 4 <= J.cap)
                *reinterpret_cast<HIZ_GLOBAL float *>(gmem(J.stream) + off) = r.own[0][0];
        }
        if (J.mode == 0) {
            // ABS mode: exact extremes of the owned points, for the header
            uint32_t kmn = 0xffffffffu, kmx = 0u;
            bool bad = false;
            own_rows<NX>([&](auto d) __attribute__((always_inline)) {
                constexpr int D = decltype(d)::value;
                const bool in = own_in<TZ, NX, D>(P, g.ownx, g.owny);
#pragma unroll
                for (int j = 0; j < 8; j++)
                    if (in && 8 * P.q + j < g.ownz) {
                        bad |= !isfinite(r.own[D][j]);
                        const uint32_t key = fkey(r.own[D][j]);
                        kmn = min(kmn, key);
                        kmx = max(kmx, key);
                    }
            });
            if (__any(bad) && (t & 63) == 0)
                atomicOr(&J.st->flags, (uint32_t)ST_NONFINITE);
            block_minmax(kmn, kmx, red);
            if (t == 0)
                gstore_u2(gmem(J.mm_part) + (u - J.tile_begin), make_uint2(kmn, kmx));
        }
        lds_barrier();
        RowCodes<TZ, NX> rc;
        if (full)
            walk_levels<TZ, NX, true, true>(v, lc, P0, rc, plan, g, f);
        else
            walk_levels<TZ, NX, false, true>(v, lc, P0, rc, plan, g, f);
        // codes of owned points -> global, histogram in LDS
        rc.own[0] = *reinterpret_cast<const uint32_t *>(lc + (P.ix * 8 + P.iy) * T::KZ + 4 * P.q);
        if (P.ix == 0 && P.iy == 0 && (P.q & 1) == 0)
            rc.own[0] = (rc.own[0] & ~255u) | 128u; // an anchor's slot
        const int nz = min(8, g.ownz - 8 * P.q);
        const uint64_t o0 = own_offset(tp, P);
        own_rows<NX>([&](auto d) __attribute__((always_inline)) {
            constexpr int D = decltype(d)::value;
            if (!full && (nz <= 0 || !own_in<TZ, NX, D>(P, g.ownx, g.owny)))
                return;
            // even and odd z interleaved
            const uint32_t c[2] = {__builtin_amdgcn_perm(rc.own[D | 4], rc.own[D], 0x05010400u),
                                   __builtin_amdgcn_perm(rc.own[D | 4], rc.own[D], 0x07030602u)};
            HIZ_GLOBAL uint8_t *dst = gmem(J.codes) + o0 + row_step<D>(tp);
            if (full || nz == 8) {
                u2_any o;
                o.x = c[0];
                o.y = c[1];
                *(HIZ_GLOBAL u2_any *)dst = o;
#pragma unroll
                for (int j = 0; j < 8; j++)
                    count((c[j >> 2] >> (8 * (j & 3))) & 255u);
            } else {
#pragma unroll 1
                for (int j = 0; j < nz; j++) {
                    const uint32_t code = ((j < 4 ? c[0] : c[1]) >> (8 * (j & 3))) & 255u;
                    dst[j] = (uint8_t)code;
                    count(code);
                }
            }
        });
    }
    lds_barrier();
    take_hist();
    if (cur >= 0)
        flush(cur);
}

// ---------------------------------------------------------------------------
// Decompression: rebuild the tile from codes, anchors and outliers,
// persistent over tiles.
// ---------------------------------------------------------------------------
// A tile's codes as a thread holds them ahead of their use: eight per own row
// and face row, far-face points, and one anchor of the tile region.
template <int TZ, int NX> struct CodeRegs {
    using T = Tile<TZ, NX>;
    static constexpr int NA = (T::FLAT ? 2 : 4) * (TZ + 1);
    uint32_t own[4][2];
    uint32_t ext[2];
    uint32_t face[T::IF];
    float anchor;
};
// Eight consecutive codes; past the field's end its last code.
__device__ __forceinline__ void load_codes8(uint32_t (&c)[2], HIZ_GLOBAL const uint8_t *p,
                                            uint64_t off, bool whole, uint64_t N)
{
    if (whole) {
        const u2_any a = *(HIZ_GLOBAL const u2_any *)(p + off);
        c[0] = a.x;
        c[1] = a.y;
    } else {
        c[0] = c[1] = 0;
#pragma unroll
        for (int j = 0; j < 8; j++)
            c[j >> 2] |= (uint32_t)p[min(off + j, N - 1)] << (8 * (j & 3));
    }
}
// Anchor i of the tile region: x, y from its low bits, z above them.
template <int NX> __device__ __forceinline__ void anchor_at(int i, int &x, int &y, int &z)
{
    x = NX == 1 ? 0 : i & 1;
    y = NX == 1 ? i & 1 : (i >> 1) & 1;
    z = NX == 1 ? i >> 1 : i >> 2;
}
template <int TZ, int NX>
__device__ __forceinline__ void code_fetch(CodeRegs<TZ, NX> &r, const Job &J, const TilePos &tp,
                                           const Place<TZ, NX> &P)
{
    using T = Tile<TZ, NX>;
    const Geo &g = tp.g;
    HIZ_GLOBAL const uint8_t *src = gmem(J.codes);
    const bool full = tile_full<TZ, NX>(g);
    const bool zin = 8 * P.q < g.ez;
    const uint64_t o0 = own_offset(tp, P);
    // points outside the tile count as no outliers
    own_rows<NX>([&](auto d) __attribute__((always_inline)) {
        constexpr int D = decltype(d)::value;
        r.own[D][0] = r.own[D][1] = 0x80808080u;
        if (full || (zin && own_in<TZ, NX, D>(P, g.ex, g.ey)))
            load_codes8(r.own[D], src, o0 + row_step<D>(tp), tp.whole, J.N);
    });
    r.ext[0] = r.ext[1] = 0x80808080u;
    if (face_in(P, g))
        load_codes8(r.ext, src, face_offset(tp, P), tp.whole, J.N);
#pragma unroll
    for (int k = 0; k < T::IF; k++) {
        const FacePoint F(P.frow[k]);
        r.face[k] = 0x80u;
        if (F.c != 15 && g.ez == 16 * TZ + 1 && F.x < g.ex && F.y < g.ey)
            r.face[k] = src[tp.base + F.x * tp.sx + F.y * tp.dz + 16 * TZ];
    }
    // anchors of the tile region: every coordinate a multiple of 16
    int x, y, z;
    anchor_at<NX>((int)threadIdx.x, x, y, z);
    if ((int)threadIdx.x < CodeRegs<TZ, NX>::NA && 16 * x < g.ex && 16 * y < g.ey && 16 * z < g.ez) {
        const uint64_t ai = ((uint64_t)(tp.bx + x) * J.nb[1] + (tp.by + y)) * J.nb[2] + tp.bz + z;
        r.anchor = reinterpret_cast<HIZ_GLOBAL const float *>(gmem(J.stream) + J.off_anchors)[ai];
    }
}

// whether a 32-bit word holds a zero byte
__device__ __forceinline__ bool has_zero_byte(uint32_t w)
{
    return ((w - 0x01010101u) & ~w & 0x80808080u) != 0;
}

template <int TZ, int NX>
__global__ __launch_bounds__((Tile<TZ, NX>::NT), 4) void k_reconstruct(const Job *__restrict__ jobs,
                                                                     int njobs, uint64_t lo,
                                                                     uint64_t hi)
{
    using T = Tile<TZ, NX>;
    __shared__ __align__(16) float v[T::NV];
    __shared__ __align__(4) uint8_t lc[T::base(1)]; // codes of the lattice, at its words
    const int t = threadIdx.x;
    const PlaceBits<TZ, NX> P0(t);
    TileWalk w = tile_walk(lo, hi);
    CodeRegs<TZ, NX> r;
    FieldQ f;
    int cur = -1;
    CoarsePlan<TZ, NX> plan;
    int ji = 0;
    TilePos tp;
    auto fetch = [&](uint64_t u) __attribute__((always_inline)) {
        ji = find_job<WK_TILE>(jobs, njobs, u);
        tp = tile_pos<TZ>(jobs[ji], u - jobs[ji].tile_begin);
        code_fetch(r, jobs[ji], tp, P0.get());
    };
    if (!w.done())
        fetch(w.tile());
    while (!w.done()) {
        const Job &J = jobs[ji];
        if (ji != cur) {
            cur = ji;
            f = load_field(J.st, false);
            plan.make(f, t);
        }
        const Geo g = tp.g;
        const bool full = tile_full<TZ, NX>(g);
        HIZ_GLOBAL float *out = gmem(J.out);
        const Place<TZ, NX> P = P0.get();
        const uint64_t o0 = own_offset(tp, P), sx = tp.sx, dz = tp.dz;
        lds_barrier(); // every wave is done with the previous tile's values
        // Rows that hold a zero code: their outliers' exact values were
        // scattered into the output beforehand; the whole row piece is taken
        // over (what it holds at other points is overwritten by the levels).
        // Codes of the lattice go to LDS, the others stay in registers.
        auto put_lattice = [&](int xh, int yh, uint32_t c) __attribute__((always_inline)) {
            *reinterpret_cast<uint32_t *>(lc + T::template word<0>(xh, yh, 4 * P.q)) = c;
        };
        RowCodes<TZ, NX> rc;
        own_rows<NX>([&](auto d) __attribute__((always_inline)) {
            constexpr int D = decltype(d)::value;
            if (has_zero_byte(r.own[D][0]) || has_zero_byte(r.own[D][1])) {
                float e[8];
                load_row8(e, out, o0 + row_step<D>(tp), tp.whole, J.N);
                put_row8<TZ, NX, D>(v, P.ix, P.iy, P.q, e);
            }
            rc.own[D] = __builtin_amdgcn_perm(r.own[D][1], r.own[D][0], 0x06040200u);
            rc.own[D | 4] = __builtin_amdgcn_perm(r.own[D][1], r.own[D][0], 0x07050301u);
        });
        put_lattice(P.ix, P.iy, rc.own[0]);
        rc.fe = __builtin_amdgcn_perm(r.ext[1], r.ext[0], 0x06040200u);
        rc.fo = __builtin_amdgcn_perm(r.ext[1], r.ext[0], 0x07050301u);
        if (has_zero_byte(r.ext[0]) || has_zero_byte(r.ext[1])) {
            float e[8];
            load_row8(e, out, face_offset(tp, P), tp.whole, J.N);
            put_face8(v, P, e);
        }
        if (P.fc == 0)
            put_lattice(P.fx, P.fy, rc.fe);
#pragma unroll
        for (int k = 0; k < T::IF; k++) {
            const FacePoint F(P.frow[k]);
            rc.face[k] = r.face[k];
            if (F.c != 15 && r.face[k] == 0)
                v[face_word<TZ, NX>(F)] = out[tp.base + F.x * tp.sx + F.y * tp.dz + 16 * TZ];
            if (F.c == 0)
                lc[T::template fword<0>(F.xh, F.yh)] = (uint8_t)r.face[k];
        }
        lds_barrier();
        {
            int x, y, z;
            anchor_at<NX>(t, x, y, z);
            if (t < CodeRegs<TZ, NX>::NA)
                v[T::template word<0>(8 * x, 8 * y, 8 * z)] = r.anchor;
        }
        // the next tile's loads fly while this tile's levels run
        w.step();
        if (!w.done())
            fetch(w.tile());
        lds_barrier();
        if (full)
            walk_levels<TZ, NX, true, false>(v, lc, P0, rc, plan, g, f);
        else
            walk_levels<TZ, NX, false, false>(v, lc, P0, rc, plan, g, f);
        // the thread's own rows, all written by itself or before a barrier
        const int nz = min(8, g.ownz - 8 * P.q);
        own_rows<NX>([&](auto d) __attribute__((always_inline)) {
            constexpr int D = decltype(d)::value;
            if (!full && (nz <= 0 || !own_in<TZ, NX, D>(P, g.ownx, g.owny)))
                return;
            const float *se = v + T::template word<D>(P.ix, P.iy, 4 * P.q);
            const float *so = v + T::template word<(D | 4)>(P.ix, P.iy, 4 * P.q);
            HIZ_GLOBAL float *dst = out + o0 + ((D & 1) ? sx : 0) + ((D & 2) ? dz : 0);
            if (full || nz == 8) {
                float e[4], o[4];
                lds_read4(se, e);
                lds_read4(so, o);
                f4_any a, b;
                a.x = e[0];
                a.y = o[0];
                a.z = e[1];
                a.w = o[1];
                b.x = e[2];
                b.y = o[2];
                b.z = e[3];
                b.w = o[3];
                *(HIZ_GLOBAL f4_any *)dst = a;
                *(HIZ_GLOBAL f4_any *)(dst + 4) = b;
            } else {
#pragma unroll 1
                for (int j = 0; j < nz; j++)
                    dst[j] = (j & 1) ? so[j >> 1] : se[j >> 1];
            }
        });
    }
}

// ---------------------------------------------------------------------------
// Launches: one per tile kind (tiles of 1, 2 or 4 blocks, and the flat tiles
// of fields of a single x plane, which take four blocks along z).
// ---------------------------------------------------------------------------
template <typename F> static void with_kind(int kind, F &&f)
{
    if (kind == kFlatKind)
        f(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
    else if (kind == 0)
        f(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
    else if (kind == 1)
        f(std::integral_constant<int, 2>{}, std::integral_constant<int, 16>{});
    else
        f(std::integral_constant<int, 4>{}, std::integral_constant<int, 16>{});
}

void launch_predict(const Job *d_jobs, int njobs, uint64_t lo, uint64_t hi, int kind, int grid,
                    hipStream_t s)
{
    if (hi <= lo)
        return;
    with_kind(kind, [&](auto tz, auto nx) {
        constexpr int TZ = decltype(tz)::value, NX = decltype(nx)::value;
        hipLaunchKernelGGL((k_predict<TZ, NX>), dim3(grid), dim3(Tile<TZ, NX>::NT), 0, s, d_jobs,
                           njobs, lo, hi);
    });
}

void launch_reconstruct(const Job *d_jobs, int njobs, uint64_t lo, uint64_t hi, int kind, int grid,
                        hipStream_t s)
{
    if (hi <= lo)
        return;
    with_kind(kind, [&](auto tz, auto nx) {
        constexpr int TZ = decltype(tz)::value, NX = decltype(nx)::value;
        hipLaunchKernelGGL((k_reconstruct<TZ, NX>), dim3(grid), dim3(Tile<TZ, NX>::NT), 0, s,
                           d_jobs, njobs, lo, hi);
    });
}

int predict_blocks_per_cu(int kind)
{
    int n = 0;
    with_kind(kind, [&](auto tz, auto nx) {
        constexpr int TZ = decltype(tz)::value, NX = decltype(nx)::value;
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_predict<TZ, NX>, Tile<TZ, NX>::NT, 0);
    });
    return n > 0 ? n : 1;
}

int reconstruct_blocks_per_cu(int kind)
{
    int n = 0;
    with_kind(kind, [&](auto tz, auto nx) {
        constexpr int TZ = decltype(tz)::value, NX = decltype(nx)::value;
        (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_reconstruct<TZ, NX>, Tile<TZ, NX>::NT, 0);
    });
    return n > 0 ? n : 1;
}

} // namespace hiz
