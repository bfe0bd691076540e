// Bitwise-redundancy lossless stages (Sec. 5.2.3), code reordering by
// interpolation level (Sec. 5.1.4, Eq. reorder) and the row-major outlier
// list of compression when the lossless stage does not see the codes in
// row-major order.
//
// Stages. A stage stream is cut into chunks of kLcChunk bytes; one workgroup
// runs one chunk through every stage of its pipeline in LDS (two ping-pong
// buffers) and stores the result, or the raw chunk when the result is not
// smaller. Chunk offsets in the stream come from a decoupled look-back over
// chunks claimed in order. Per stage, with symbol width k bytes:
//  - TCMS_k: (w << 1) ^ (w >> (8k-1)), arithmetic shift, on each k-byte word
//    (two's complement to magnitude-sign);
//  - BIT_1: bit shuffle: output plane p holds bit p of every byte, byte 8j+i
//    giving bit i of the plane's byte j (an 8x8 bit transpose per group);
//  - RRE_k / RZE_k: a bitmap marks the words that differ from the word before
//    (0 before the first) / that are nonzero, and only those are kept. The
//    stage writes its input length (u16), the bitmap compressed recursively
//    (a bitmap of at most 8 bytes as it is; a longer one as the bitmap of its
//    bytes that differ from the byte before, compressed the same way, then
//    those bytes), the kept words and the bytes after the last whole word.
// Each stage is a pass of the workgroup over its chunk in 16-byte pieces, one
// scan over all pieces and bitmap levels, and a compaction out of registers;
// TCMS is done on the way in or out of its neighbour. What bounds the kernels is
// the instructions of those passes and, per chunk, the latency of a claim, of the
// look-back and of some five barriers; four workgroups per compute unit (36 KB
// of LDS each) fill in for each other. 256^3: throughput mode 134 -> 35 us
// encoding and 87 -> 39 decoding, ratio mode 108 -> 30 and 44 -> 24, the first
// figure for loops over single bytes with a scan per bitmap level.
#include "hiz_internal.h"

namespace hiz {

constexpr int kLcThreads = 256;
constexpr int kLcWaves = kLcThreads / 64;
constexpr int kPiece = 16;                         // bytes a thread handles at a time
constexpr int kRound = kPiece * kLcThreads;        // bytes of one round of the workgroup
constexpr int kRounds = kLcChunk / kRound;         // rounds of a chunk
// Longest stream between two stages: RRE_4 of a whole chunk, nothing left out
// (2 + 512 + 64 + 8 bytes in front of the words).
constexpr int kLcMid = kLcChunk + 2 + kLcChunk / 32 + kLcChunk / 256 + 8;
constexpr int kMidRounds = (kLcMid + kRound - 1) / kRound;
// Bitmap levels of up to kLcMid marks: level 0, and each level's byte marks
// (level 3 has at most 8 bytes).
constexpr int kBm0 = (kLcMid + 7) / 8, kBm1 = (kBm0 + 7) / 8, kBm2 = (kBm1 + 7) / 8;
static_assert((kBm2 + 7) / 8 <= 8 && kBm1 <= 2 * kLcThreads && kBm2 <= 64, "four bitmap levels");
constexpr int kBmOff[4] = {0, (kBm0 + 31) & ~15, ((kBm0 + 31) & ~15) + ((kBm1 + 31) & ~15),
                           ((kBm0 + 31) & ~15) + ((kBm1 + 31) & ~15) + ((kBm2 + 31) & ~15)};
constexpr int kBmBytes = kBmOff[3] + 16;

// 36 KB, so that four workgroups fit on a compute unit.
struct LcShared {
    alignas(16) uint8_t a[kLcChunk + 2 * kPiece];              // a chunk's stored form
    alignas(16) uint8_t b[(kLcMid + 2 * kPiece) & ~15];        // between two stages
    alignas(16) uint8_t bm[kBmBytes];
    alignas(16) uint32_t part[5][kLcWaves];
    int pos; // decoder: bytes read so far, -1: more than there are
    uint32_t id;
    uint64_t base, zbase;
};
static_assert(sizeof(LcShared) <= 40960, "four workgroups per compute unit");

typedef uint32_t u4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u4_lds __attribute__((ext_vector_type(4)));

// LDS accesses of one wave stay in this order (the LDS itself keeps it).
__device__ __forceinline__ void wave_order() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ uint32_t pick4(const uint32_t (&w)[4], int i)
{
    return i == 0 ? w[0] : i == 1 ? w[1] : i == 2 ? w[2] : w[3];
}

// ---- small primitives --------------------------------------------------------

// Exclusive prefix of v over the workgroup; `total` gets the sum.
__device__ inline int wg_excl_scan(int v, int *tmp, int &total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int incl = (int)wave_incl_scan_dpp((uint32_t)v);
    if (lane == 63)
        tmp[wv] = incl;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kLcWaves; w++) {
        const int x = tmp[w];
        before += w < wv ? x : 0;
        total += x;
    }
    __syncthreads();
    return before + incl - v;
}

// N counters of at most 1024 per wave at once: `before` gets each one's
// exclusive prefix over the workgroup, `total` its sum. One barrier; the next
// use of `part` has to be behind another.
template <int N>
__device__ __forceinline__ void scan_counters(const uint32_t (&c)[N], uint32_t (&before)[N],
                                              uint32_t (&total)[N], LcShared &S)
{
    constexpr int P = (N + 1) / 2;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t in[P];
#pragma unroll
    for (int p = 0; p < P; p++) {
        const uint32_t v = c[2 * p] | (2 * p + 1 < N ? c[2 * p + 1] << 16 : 0u);
        const uint32_t x = wave_incl_scan_dpp(v);
        if (lane == 63)
            S.part[p][wv] = x;
        in[p] = x - v;
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < P; p++) {
        uint32_t b = in[p], s = 0;
        // (a workgroup's sum of one counter is at most 4096: it fits its half)
#pragma unroll
        for (int w = 0; w < kLcWaves; w++) {
            const uint32_t x = S.part[p][w];
            b += w < wv ? x : 0u;
            s += x;
        }
        before[2 * p] = b & 0xffffu;
        total[2 * p] = s & 0xffffu;
        if (2 * p + 1 < N) {
            before[2 * p + 1] = b >> 16;
            total[2 * p + 1] = s >> 16;
        }
    }
}

// One bit per byte of x, set where the byte is not zero.
__device__ __forceinline__ uint32_t nonzero4(uint32_t x)
{
    const uint32_t t = (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) >> 7 & 0x01010101u;
    return t * 0x01020408u >> 24;
}
__device__ __forceinline__ uint32_t nonzero8(uint64_t x)
{
    return nonzero4((uint32_t)x) | nonzero4((uint32_t)(x >> 32)) << 4;
}

// 8x8 bit transpose: byte i of v, bit p -> byte p of the result, bit i.
__device__ inline uint64_t transpose8(uint64_t x)
{
    uint64_t t;
    t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
    x ^= t ^ (t << 7);
    t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
    x ^= t ^ (t << 14);
    t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
    x ^= t ^ (t << 28);
    return x;
}

// TCMS of every byte of x, of a 64-bit word, and back.
__device__ __forceinline__ uint32_t tcms1(uint32_t x)
{
    return (x << 1 & 0xfefefefeu) ^ (x >> 7 & 0x01010101u) * 255u;
}
__device__ __forceinline__ uint32_t tcms1_inv(uint32_t x)
{
    return (x >> 1 & 0x7f7f7f7fu) ^ (x & 0x01010101u) * 255u;
}
__device__ __forceinline__ uint64_t tcms8(uint64_t w)
{
    return (w << 1) ^ (uint64_t)((int64_t)w >> 63);
}
__device__ __forceinline__ uint64_t tcms8_inv(uint64_t w) { return (w >> 1) ^ (0ull - (w & 1)); }
// The 64-bit words of the piece at byte i of a stream of n bytes; bytes past the
// last whole word stay.
template <bool INV> __device__ __forceinline__ void tcms8_piece(uint4 &x, int i, int n)
{
    uint64_t lo = x.x | (uint64_t)x.y << 32, hi = x.z | (uint64_t)x.w << 32;
    if (i + 8 <= n)
        lo = INV ? tcms8_inv(lo) : tcms8(lo);
    if (i + 16 <= n)
        hi = INV ? tcms8_inv(hi) : tcms8(hi);
    x = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// Transpose of a 4x4 byte matrix held as four words.
__device__ __forceinline__ void transpose_bytes(uint32_t (&w)[4])
{
    const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u); // w0.0 w1.0 w0.1 w1.1
    const uint32_t b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u); // w0.2 w1.2 w0.3 w1.3
    const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
    const uint32_t d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    w[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    w[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    w[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    w[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// Bytes of the bitmap levels of m marks; `top` is the last level.
struct Bitmap {
    int nb[4], top;
    __device__ explicit Bitmap(int m)
    {
        nb[0] = (m + 7) / 8;
#pragma unroll
        for (int l = 1; l < 4; l++)
            nb[l] = (nb[l - 1] + 7) / 8;
        top = nb[0] <= 8 ? 0 : nb[1] <= 8 ? 1 : nb[2] <= 8 ? 2 : 3;
    }
    __device__ int top_bytes() const
    {
        return top == 0 ? nb[0] : top == 1 ? nb[1] : top == 2 ? nb[2] : nb[3];
    }
    __device__ static int top_off(int top)
    {
        return top == 0 ? kBmOff[0] : top == 1 ? kBmOff[1] : top == 2 ? kBmOff[2] : kBmOff[3];
    }
};
// The low `n` of 8 (or more) mark bits.
__device__ __forceinline__ uint32_t low_bits(int n) { return n >= 31 ? ~0u : (1u << max(n, 0)) - 1u; }

// ---- RRE / RZE --------------------------------------------------------------

// Marks of level bytes 8q..8q+7 (of n) that differ from the byte before.
__device__ __forceinline__ uint32_t level_marks(const uint8_t *src, int q, int n)
{
    const uint64_t w = *reinterpret_cast<const uint64_t *>(src + 8 * q);
    const uint64_t before = q ? src[8 * q - 1] : 0;
    return nonzero8(w ^ (w << 8 | before)) & low_bits(n - 8 * q);
}
// The marked bytes of the eight at src, in order, to dst.
__device__ __forceinline__ void keep8(uint8_t *dst, const uint8_t *src, uint32_t marks)
{
    const uint64_t w = *reinterpret_cast<const uint64_t *>(src);
#pragma unroll
    for (int k = 0; k < 8; k++)
        if (marks >> k & 1)
            *dst++ = (uint8_t)(w >> (8 * k));
}

// RRE_K (ZERO = false) / RZE_K (ZERO = true) of n bytes into out, R rounds of
// the workgroup at most. Thread t takes the 16 bytes at 4096 r + 16 t in round
// r: fetch(r, x, before) gives them and, for RRE, the word before. What a thread
// keeps stays in its registers until one scan over all rounds and bitmap levels
// has told where everything goes. Returns the length; one of at least `limit`
// is not written.
template <int K, bool ZERO, int R, class FETCH>
__device__ int st_reduce(FETCH fetch, int n, uint8_t *out, int limit, LcShared &S)
{
    constexpr int E = kPiece / K; // words of a piece
    const int t = threadIdx.x;
    const int m = n / K;
    const Bitmap B(m);
    uint8_t *bm0 = S.bm + kBmOff[0], *bm1 = S.bm + kBmOff[1], *bm2 = S.bm + kBmOff[2],
            *bm3 = S.bm + kBmOff[3];
    uint4 x[R];
    uint32_t marks[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = kRound * r + kPiece * t;
        marks[r] = 0;
        if (i < n) {
            uint32_t before = 0;
            fetch(r, x[r], before);
            const uint4 v = x[r];
            if (K == 4) {
                marks[r] = (uint32_t)(v.x != before) | (uint32_t)(v.y != v.x) << 1 |
                           (uint32_t)(v.z != v.y) << 2 | (uint32_t)(v.w != v.z) << 3;
            } else if (ZERO) {
                marks[r] = nonzero4(v.x) | nonzero4(v.y) << 4 | nonzero4(v.z) << 8 |
                           nonzero4(v.w) << 12;
            } else {
                marks[r] = nonzero4(v.x ^ __builtin_amdgcn_alignbyte(v.x, before, 3)) |
                           nonzero4(v.y ^ __builtin_amdgcn_alignbyte(v.y, v.x, 3)) << 4 |
                           nonzero4(v.z ^ __builtin_amdgcn_alignbyte(v.z, v.y, 3)) << 8 |
                           nonzero4(v.w ^ __builtin_amdgcn_alignbyte(v.w, v.z, 3)) << 12;
            }
            marks[r] &= low_bits(m - i / K);
        }
        if (K == 4) {
            const uint32_t odd = (uint32_t)__shfl_xor((int)marks[r], 1, 64);
            if (!(t & 1) && i < n)
                bm0[i / 32] = (uint8_t)(marks[r] | odd << 4);
        } else if (i < n) {
            *reinterpret_cast<uint16_t *>(bm0 + i / 8) = (uint16_t)marks[r];
        }
    }
    __syncthreads();
    // level 1 by the workgroup, levels 2 and 3 (34 and 5 bytes at most) by wave 0
    uint32_t c[4 + R];
#pragma unroll
    for (int k = 0; k < 4; k++)
        c[k] = 0;
    uint32_t lm[4] = {0, 0, 0, 0}; // marks of this thread's bytes: level 2, 1, 0 and 0 again
    if (B.top > 0) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = t + kLcThreads * h;
            if (q < B.nb[1]) {
                lm[2 + h] = level_marks(bm0, q, B.nb[0]);
                bm1[q] = (uint8_t)lm[2 + h];
            }
        }
        __syncthreads();
        if (t < 64 && B.top > 1) {
            if (t < B.nb[2]) {
                lm[1] = level_marks(bm1, t, B.nb[1]);
                bm2[t] = (uint8_t)lm[1];
            }
            wave_order();
            if (B.top > 2 && t < B.nb[3]) {
                lm[0] = level_marks(bm2, t, B.nb[2]);
                bm3[t] = (uint8_t)lm[0];
            }
            wave_order();
        }
    }
#pragma unroll
    for (int k = 0; k < 4; k++)
        c[k] = __popc(lm[k]);
#pragma unroll
    for (int r = 0; r < R; r++)
        c[4 + r] = __popc(marks[r]);
    uint32_t o[4 + R], total[4 + R];
    scan_counters<4 + R>(c, o, total, S);
    const int nt = B.top_bytes();
    int len = 2 + nt;
#pragma unroll
    for (int k = 0; k < 4 + R; k++) {
        const int w = k < 4 ? 1 : K;
        o[k] = (uint32_t)len + w * o[k];
        len += w * (int)total[k];
    }
    const int tail = n - m * K;
    if (len + tail >= limit)
        return len + tail;
    if (t < 64) {
        if (t == 0) {
            out[0] = (uint8_t)(n & 255);
            out[1] = (uint8_t)(n >> 8);
        }
        if (t < nt)
            out[2 + t] = S.bm[Bitmap::top_off(B.top) + t];
        if (lm[0])
            keep8(out + o[0], bm2 + 8 * t, lm[0]);
        if (lm[1])
            keep8(out + o[1], bm1 + 8 * t, lm[1]);
    }
    if (lm[2])
        keep8(out + o[2], bm0 + 8 * t, lm[2]);
    if (lm[3])
        keep8(out + o[3], bm0 + 8 * (t + kLcThreads), lm[3]);
#pragma unroll
    for (int r = 0; r < R; r++) {
        const uint32_t w[4] = {x[r].x, x[r].y, x[r].z, x[r].w};
        uint8_t *p = out + o[4 + r];
#pragma unroll
        for (int k = 0; k < E; k++)
            if (marks[r] >> k & 1) {
                if (K == 4) {
#pragma unroll
                    for (int b = 0; b < 4; b++)
                        p[b] = (uint8_t)(w[k] >> (8 * b));
                } else {
                    *p = (uint8_t)(w[k / 4] >> (8 * (k & 3)));
                }
                p += K;
            }
        // bytes past the last whole word
        if (K > 1) {
            const int i = kRound * r + kPiece * t, e = m * K - i;
            if (tail && e >= 0 && e < kPiece)
                for (int b = 0; b < tail; b++)
                    out[len + b] = (uint8_t)(pick4(w, e / 4) >> (8 * b));
        }
    }
    __syncthreads();
    return len + tail;
}

// Eight level bytes from their marks: kept bytes at src, `r` of them before.
__device__ __forceinline__ uint64_t spread8(const uint8_t *src, uint32_t r, uint32_t marks)
{
    uint64_t v = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        r += marks >> k & 1;
        const uint32_t e = src[(int)r - 1]; // (with r = 0 a byte of the length or a bitmap)
        v |= (uint64_t)(r ? e : 0u) << (8 * k);
    }
    return v;
}
// A bitmap level of at most 512 bytes from the marks of the level above, by one
// wave; false: fewer than the marked bytes are left at pos.
__device__ __forceinline__ bool restore_level(const uint8_t *a, int avail, int &pos,
                                              const uint8_t *marks, uint8_t *dst, int n)
{
    const int t = threadIdx.x & 63;
    const uint32_t mk = 8 * t < n ? marks[t] & low_bits(n - 8 * t) : 0u;
    const uint32_t c = __popc(mk), incl = wave_incl_scan_dpp(c);
    const int total = __builtin_amdgcn_readlane((int)incl, 63);
    if (total > avail - pos)
        return false;
    if (8 * t < n)
        *reinterpret_cast<uint64_t *>(dst + 8 * t) = spread8(a + pos, incl - c, mk);
    pos += total;
    return true;
}

// Inverse of st_reduce on a[0..avail): put(r, x) takes the 16 bytes at
// 4096 r + 16 t (past the end zeros). want >= 0: the length has to be that.
// Returns the length, or -1 with nothing put: the stream is not one of
// st_reduce's. Every count is checked against what is left before it is read.
template <int K, bool ZERO, int R, class PUT>
__device__ int st_restore(const uint8_t *a, int avail, int want, PUT put, LcShared &S)
{
    constexpr int E = kPiece / K;
    const int t = threadIdx.x;
    if (avail < 2)
        return -1;
    const int n = a[0] | a[1] << 8;
    if (n > R * kRound || n > kLcMid || (want >= 0 && n != want))
        return -1;
    const int m = n / K, tail = n - m * K;
    const Bitmap B(m);
    uint8_t *bm0 = S.bm + kBmOff[0], *bm1 = S.bm + kBmOff[1], *bm2 = S.bm + kBmOff[2],
            *bm3 = S.bm + kBmOff[3];
    const int nt = B.top_bytes();
    if (2 + nt > avail)
        return -1;
    // levels above 0 by wave 0
    if (t < 64) {
        if (t < nt)
            S.bm[Bitmap::top_off(B.top) + t] = a[2 + t];
        wave_order();
        int pos = 2 + nt;
        bool ok = true;
        if (B.top > 2)
            ok = restore_level(a, avail, pos, bm3, bm2, B.nb[2]);
        wave_order();
        if (ok && B.top > 1)
            ok = restore_level(a, avail, pos, bm2, bm1, B.nb[1]);
        if (t == 0)
            S.pos = ok ? pos : -1;
    }
    __syncthreads();
    int pos = __builtin_amdgcn_readfirstlane(S.pos);
    if (pos < 0)
        return -1;
    if (B.top > 0) {
        uint32_t mk[2], c[2], o[2], total[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = t + kLcThreads * h;
            mk[h] = q < B.nb[1] ? bm1[q] & low_bits(B.nb[0] - 8 * q) : 0u;
            c[h] = __popc(mk[h]);
        }
        scan_counters<2>(c, o, total, S);
        if ((int)(total[0] + total[1]) > avail - pos)
            return -1;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int q = t + kLcThreads * h;
            if (q < B.nb[1])
                *reinterpret_cast<uint64_t *>(bm0 + 8 * q) =
                    spread8(a + pos, o[h] + (h ? total[0] : 0u), mk[h]);
        }
        pos += (int)(total[0] + total[1]);
        __syncthreads();
    }
    uint32_t mk[R], c[R], o[R], total[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = kRound * r + kPiece * t;
        mk[r] = 0;
        if (i < n) {
            mk[r] = K == 4 ? (uint32_t)bm0[i / 32] >> (4 * (t & 1)) & 15u
                           : *reinterpret_cast<const uint16_t *>(bm0 + i / 8);
            mk[r] &= low_bits(m - i / K);
        }
        c[r] = __popc(mk[r]);
    }
    scan_counters<R>(c, o, total, S);
    int kept = 0;
#pragma unroll
    for (int r = 0; r < R; r++) {
        o[r] += (uint32_t)kept;
        kept += (int)total[r];
    }
    if (pos + K * kept + tail != avail)
        return -1;
    const uint8_t *src = a + pos;
    const uint32_t sh = (uint32_t)(pos & 3);
    const uint32_t *src4 = reinterpret_cast<const uint32_t *>(src - sh);
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = kRound * r + kPiece * t;
        if (i >= n)
            continue;
        uint32_t w[4] = {0, 0, 0, 0};
        int k0 = (int)o[r] - 1; // the kept word an unmarked first one repeats
#pragma unroll
        for (int k = 0; k < E; k++) {
            const bool mark = mk[r] >> k & 1;
            k0 += mark;
            const bool has = (ZERO ? mark : k0 >= 0) && i / K + k < m;
            const int j = has ? k0 : 0;
            if (K == 4) {
                const uint32_t e = __builtin_amdgcn_alignbyte(src4[j + 1], src4[j], sh);
                w[k] = has ? e : 0u;
            } else {
                w[k / 4] |= (has ? (uint32_t)src[j] : 0u) << (8 * (k & 3));
            }
        }
        if (K > 1) {
            const int e = m * K - i;
            if (tail && e >= 0 && e < kPiece)
#pragma unroll
                for (int k = 0; k < 4; k++)
                    if (k == e / 4)
                        for (int b = 0; b < tail; b++)
                            w[k] |= (uint32_t)src[K * kept + b] << (8 * b);
        }
        put(r, make_uint4(w[0], w[1], w[2], w[3]));
    }
    __syncthreads();
    return n;
}

// ---- TCMS_1 and BIT_1 -------------------------------------------------------

// TCMS_1 then BIT_1 of the n bytes at src (16-byte aligned) into b, four groups of eight bytes a
// thread at a time: their planes' bytes are written as words. zero[r] gets a
// bit for each zero byte of the thread's 32 in round r.
constexpr int kBitRounds = kLcChunk / (32 * kLcThreads);
__device__ void st_planes(HIZ_GLOBAL const uint8_t *src, int n, uint8_t *b,
                          uint32_t (&zero)[kBitRounds])
{
    const int t = threadIdx.x, g = n / 8;
    uint4 v[kBitRounds][2];
#pragma unroll
    for (int r = 0; r < kBitRounds; r++) {
        const int i = 32 * (kLcThreads * r + t);
        if (i + 32 <= n) {
            v[r][0] = gload_u4(src + i);
            v[r][1] = gload_u4(src + i + 16);
        }
    }
#pragma unroll
    for (int r = 0; r < kBitRounds; r++) {
        const int i = 32 * (kLcThreads * r + t);
        zero[r] = 0;
        if (i + 32 <= n) {
            uint32_t w[8] = {v[r][0].x, v[r][0].y, v[r][0].z, v[r][0].w,
                             v[r][1].x, v[r][1].y, v[r][1].z, v[r][1].w};
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int q = 0; q < 8; q++)
                zero[r] |= (nonzero4(w[q]) ^ 15u) << (4 * q);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const uint64_t x =
                    transpose8(tcms1(w[2 * q]) | (uint64_t)tcms1(w[2 * q + 1]) << 32);
                lo[q] = (uint32_t)x;
                hi[q] = (uint32_t)(x >> 32);
            }
            if ((g & 3) == 0) {
                transpose_bytes(lo);
                transpose_bytes(hi);
#pragma unroll
                for (int p = 0; p < 4; p++) {
                    *reinterpret_cast<uint32_t *>(b + p * g + i / 8) = lo[p];
                    *reinterpret_cast<uint32_t *>(b + (p + 4) * g + i / 8) = hi[p];
                }
            } else {
#pragma unroll
                for (int p = 0; p < 8; p++)
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        b[p * g + i / 8 + q] = (uint8_t)((p < 4 ? lo[q] : hi[q]) >> (8 * (p & 3)));
            }
        } else if (i < n) {
            // the chunk's last bytes: whole groups, then bytes that stay
            for (int k = 0; k < n - i; k++) {
                const uint32_t e = src[i + k];
                zero[r] |= (uint32_t)(e == 0) << k;
                if (i + k >= 8 * g)
                    b[i + k] = (uint8_t)tcms1(e);
            }
            for (int j = i / 8; j < g; j++) {
                uint64_t x = 0;
                for (int k = 0; k < 8; k++)
                    x |= (uint64_t)(uint8_t)tcms1(src[8 * j + k]) << (8 * k);
                x = transpose8(x);
                for (int p = 0; p < 8; p++)
                    b[p * g + j] = (uint8_t)(x >> (8 * p));
            }
        }
    }
    __syncthreads();
}

// The inverse, from b to dst (16-byte aligned); returns how many of the
// thread's bytes are zero.
__device__ int st_planes_inv(const uint8_t *b, int n, HIZ_GLOBAL uint8_t *dst)
{
    const int t = threadIdx.x, g = n / 8;
    int zeros = 0;
#pragma unroll
    for (int r = 0; r < kBitRounds; r++) {
        const int i = 32 * (kLcThreads * r + t);
        if (i + 32 <= n) {
            uint32_t lo[4], hi[4], w[8];
            if ((g & 3) == 0) {
#pragma unroll
                for (int p = 0; p < 4; p++) {
                    lo[p] = *reinterpret_cast<const uint32_t *>(b + p * g + i / 8);
                    hi[p] = *reinterpret_cast<const uint32_t *>(b + (p + 4) * g + i / 8);
                }
                transpose_bytes(lo);
                transpose_bytes(hi);
            } else {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    lo[q] = hi[q] = 0;
#pragma unroll
                    for (int p = 0; p < 4; p++) {
                        lo[q] |= (uint32_t)b[p * g + i / 8 + q] << (8 * p);
                        hi[q] |= (uint32_t)b[(p + 4) * g + i / 8 + q] << (8 * p);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const uint64_t x = transpose8(lo[q] | (uint64_t)hi[q] << 32);
                w[2 * q] = tcms1_inv((uint32_t)x);
                w[2 * q + 1] = tcms1_inv((uint32_t)(x >> 32));
                zeros += 8 - __popc(nonzero4(w[2 * q])) - __popc(nonzero4(w[2 * q + 1]));
            }
            gstore_u4(dst + i, make_uint4(w[0], w[1], w[2], w[3]));
            gstore_u4(dst + i + 16, make_uint4(w[4], w[5], w[6], w[7]));
        } else if (i < n) {
            for (int j = i / 8; j < g; j++) {
                uint64_t x = 0;
                for (int p = 0; p < 8; p++)
                    x |= (uint64_t)b[p * g + j] << (8 * p);
                x = transpose8(x);
                for (int k = 0; k < 8; k++) {
                    const uint8_t e = (uint8_t)tcms1_inv((uint32_t)(x >> (8 * k)) & 255u);
                    zeros += e == 0;
                    dst[8 * j + k] = e;
                }
            }
            for (int k = max(i, 8 * g); k < n; k++) {
                const uint8_t e = (uint8_t)tcms1_inv(b[k]);
                zeros += e == 0;
                dst[k] = e;
            }
        }
    }
    return zeros;
}

// n bytes from LDS (16-byte aligned) or from global memory (any alignment).
template <class SRC> __device__ void copy_out(HIZ_GLOBAL uint8_t *dst, SRC src, int n)
{
    for (int i = kPiece * threadIdx.x; i < n; i += kRound) {
        if (i + kPiece <= n)
            *reinterpret_cast<HIZ_GLOBAL u4_any *>(dst + i) = src.piece(i);
        else
            for (int k = i; k < n; k++)
                dst[k] = src.byte(k);
    }
}
struct FromLds {
    const uint8_t *p;
    __device__ u4_any piece(int i) const { return *reinterpret_cast<const u4_lds *>(p + i); }
    __device__ uint8_t byte(int i) const { return p[i]; }
};
struct FromGlobal {
    HIZ_GLOBAL const uint8_t *p;
    __device__ u4_any piece(int i) const { return *reinterpret_cast<HIZ_GLOBAL const u4_any *>(p + i); }
    __device__ uint8_t byte(int i) const { return p[i]; }
};

// Stage-stream input of compression: the code sequence (throughput mode) or
// the Huffman payload's bytes (ratio mode).
__device__ inline uint64_t lc_input_bytes(const Job &J, const FieldState *st)
{
    return J.pipe == PIPE_TP ? J.N : 4 * st->payload_words;
}

// Stream offsets of the stage sections: the chunk-size table and the data.
__device__ inline void lc_offsets(const Job &J, const FieldState *st, uint64_t n_lc,
                                  uint64_t &o_sizes, uint64_t &o_data)
{
    if (J.pipe == PIPE_TP) {
        o_sizes = kOffChunks;
        o_data = st->off_payload;
    } else {
        o_sizes = align16(st->off_oval + 4 * st->n_out);
        o_data = align16(o_sizes + 4 * n_lc);
    }
}

// The 16 bytes at i of n in global memory (16-byte aligned), zeros past the end.
__device__ __forceinline__ uint4 load_piece(HIZ_GLOBAL const uint8_t *src, int i, int n)
{
    if (i + kPiece <= n)
        return gload_u4(src + i);
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < kPiece; k++)
        w[k / 4] |= (i + k < n ? (uint32_t)src[i + k] : 0u) << (8 * (k & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// ---- compression: one workgroup per chunk -----------------------------------
// Chunks of every job of the launch, throughput and ratio mode alike.
__global__ __launch_bounds__(kLcThreads, 4) void k_lc_encode(const Job *__restrict__ jobs,
                                                             int njobs, uint64_t total,
                                                             Counters *cnt)
{
    __shared__ LcShared S;
    const int t = threadIdx.x;
    // One field: as many workgroups claim as there are chunks. (A payload is
    // sized for 32 bits a code, and most of the launch has no chunk; claims, on
    // one word, are made one after the other: 256^3 ratio mode 53 us, 30
    // without.)
    if (njobs == 1 && blockIdx.x >= cdiv(lc_input_bytes(jobs[0], jobs[0].st), kLcChunk))
        return;
    if (t == 0)
        S.id = atomicAdd(&cnt->lc_next, 1u);
    __syncthreads();
    const uint64_t id = uni32(S.id);
    if (id >= total)
        return;
    const Job &J = jobs[find_job<WK_LC>(jobs, njobs, id)];
    const bool tp = J.pipe == PIPE_TP;
    FieldState *st = J.st;
    if (st->flags & (ST_CONST | ST_NONFINITE))
        return; // every chunk of this field returns here: nobody waits on it
    const uint64_t c = id - J.lc_begin;
    const uint64_t n_in = lc_input_bytes(J, st);
    const uint64_t n_lc = cdiv(n_in, kLcChunk);
    if (c >= n_lc)
        return; // past the end of a payload shorter than its bound
    const uint64_t lo = c * kLcChunk;
    const int n = (int)min<uint64_t>(kLcChunk, n_in - lo);
    HIZ_GLOBAL const uint8_t *src = tp ? gmem(J.seq) + lo : gmem(J.hpay) + lo;
    // outliers of a row-major code chunk (throughput mode, codes not reordered)
    const bool outl = tp && !J.reorder;
    uint32_t zero[kBitRounds], zbefore[kBitRounds], ztotal[kBitRounds];
    uint32_t zt = 0;
    int len;
    if (tp) {
        st_planes(src, n, S.b, zero);
        if (outl) {
            uint32_t zc[kBitRounds];
#pragma unroll
            for (int r = 0; r < kBitRounds; r++)
                zc[r] = __popc(zero[r]);
            static_assert(kBitRounds == 2 && 64 * 32 <= 4096, "two counters");
            scan_counters<kBitRounds>(zc, zbefore, ztotal, S);
            zbefore[1] += ztotal[0];
            zt = ztotal[0] + ztotal[1];
        }
        len = st_reduce<1, false, kRounds>(
            [&](int r, uint4 &x, uint32_t &before) __attribute__((always_inline)) {
                const int i = kRound * r + kPiece * t;
                x = *reinterpret_cast<const uint4 *>(S.b + i);
                before = i ? *reinterpret_cast<const uint32_t *>(S.b + i - 4) : 0u;
            },
            n, S.a, n, S);
    } else {
        const int n1 = st_reduce<4, false, kRounds>(
            [&](int r, uint4 &x, uint32_t &before) __attribute__((always_inline)) {
                const int i = kRound * r + kPiece * t;
                x = load_piece(src, i, n);
                before = i ? *reinterpret_cast<HIZ_GLOBAL const uint32_t *>(src + i - 4) : 0u;
            },
            n, S.b, kLcMid + 1, S);
        // TCMS_8 on the way into RZE_1
        len = st_reduce<1, true, kMidRounds>(
            [&](int r, uint4 &x, uint32_t &) __attribute__((always_inline)) {
                const int i = kRound * r + kPiece * t;
                x = *reinterpret_cast<const uint4 *>(S.b + i);
                tcms8_piece<false>(x, i, n1);
            },
            n1, S.a, n, S);
    }
    const bool raw = len >= n;
    if (raw)
        len = n;
    // offsets: stored bytes by wave 0, outliers by wave 1
    if (t < 64) {
        const uint64_t b = lookback(J.lb_c, c, (uint64_t)len);
        if (t == 0)
            S.base = b;
    } else if (t < 128 && outl) {
        const uint64_t b = lookback(J.lb_d, c, (uint64_t)zt);
        if (t == 64)
            S.zbase = b;
    }
    __syncthreads();
    uint64_t o_sizes, o_data;
    lc_offsets(J, st, n_lc, o_sizes, o_data);
    const uint64_t cap = J.cap;
    HIZ_GLOBAL uint8_t *out = gmem(J.stream);
    const uint64_t dst = o_data + S.base;
    const int room = dst >= cap ? 0 : (int)min<uint64_t>((uint64_t)len, cap - dst);
    if (raw)
        copy_out(out + dst, FromGlobal{src}, room);
    else
        copy_out(out + dst, FromLds{S.a}, room);
    if (outl) {
        const int ib = J.idx_bytes;
        const uint64_t oidx = st->off_oidx, oval = st->off_oval;
#pragma unroll
        for (int r = 0; r < kBitRounds; r++) {
            uint64_t z = S.zbase + zbefore[r];
            for (uint32_t m = zero[r]; m; m &= m - 1) {
                const uint64_t gi = lo + 32 * (kLcThreads * r + t) + (__ffs((int)m) - 1);
                if (oidx + (z + 1) * ib <= cap) {
                    if (ib == 4)
                        reinterpret_cast<HIZ_GLOBAL uint32_t *>(out + oidx)[z] = (uint32_t)gi;
                    else
                        reinterpret_cast<HIZ_GLOBAL uint64_t *>(out + oidx)[z] = gi;
                }
                if (oval + (z + 1) * 4 <= cap)
                    reinterpret_cast<HIZ_GLOBAL float *>(out + oval)[z] = gmem(J.field)[gi];
                z++;
            }
        }
        if (c == n_lc - 1 && t == 0 && S.zbase + zt != st->n_out)
            atomicOr(&st->flags, (uint32_t)ST_CORRUPT);
    }
    if (t == 0) {
        if (o_sizes + 4 * (c + 1) <= cap)
            reinterpret_cast<HIZ_GLOBAL uint32_t *>(out + o_sizes)[c] = (uint32_t)len;
        if (c == n_lc - 1) {
            const uint64_t lc_bytes = S.base + len;
            const uint64_t total_bytes = o_data + lc_bytes;
            st->lc_bytes = lc_bytes;
            st->total_bytes = total_bytes;
            if (H_NLC + 8 <= cap) {
                *reinterpret_cast<HIZ_GLOBAL uint64_t *>(out + H_LCBYTES) = lc_bytes;
                *reinterpret_cast<HIZ_GLOBAL uint64_t *>(out + H_NLC) = n_lc;
                *reinterpret_cast<HIZ_GLOBAL uint64_t *>(out + H_TOTAL) = total_bytes;
            }
            if (total_bytes > cap)
                atomicOr(&st->flags, (uint32_t)ST_OVERFLOW);
        }
    }
    // zero the alignment gaps around the ratio mode's sections (< 16 bytes each)
    if (!tp && c == 0 && t < 32) {
        const uint64_t a0 = t < 16 ? st->off_oval + 4 * st->n_out : o_sizes + 4 * n_lc;
        const uint64_t a1 = t < 16 ? o_sizes : o_data;
        const uint64_t g = a0 + (t & 15);
        if (g < a1 && g < cap)
            out[g] = 0;
    }
}

// ---- decompression: one workgroup per chunk ---------------------------------
__global__ __launch_bounds__(kLcThreads, 4) void k_lc_decode(const Job *__restrict__ jobs,
                                                             int njobs, uint64_t total,
                                                             Counters *cnt)
{
    __shared__ LcShared S;
    const int t = threadIdx.x;
    if (t == 0)
        S.id = atomicAdd(&cnt->lc_next, 1u);
    __syncthreads();
    const uint64_t id = uni32(S.id);
    if (id >= total)
        return;
    const Job &J = jobs[find_job<WK_LC>(jobs, njobs, id)];
    const bool tp = J.pipe == PIPE_TP;
    FieldState *st = J.st;
    const uint64_t c = id - J.lc_begin;
    const uint64_t n_raw = tp ? J.N : 4 * J.payload_words;
    const uint64_t lo = c * kLcChunk;
    const int n = (int)min<uint64_t>(kLcChunk, n_raw - lo);
    HIZ_GLOBAL const uint8_t *in = gmem(J.stream);
    const uint32_t size = reinterpret_cast<HIZ_GLOBAL const uint32_t *>(in + J.off_lcsizes)[c];
    if (t < 64) {
        const uint64_t b = lookback(J.lb_c, c, (uint64_t)size);
        if (t == 0)
            S.base = b;
    }
    __syncthreads();
    const uint64_t base = uni64(S.base);
    bool bad = size > (uint32_t)n || base + size > J.lc_bytes ||
               (c == J.n_lc - 1 && base + size != J.lc_bytes);
    HIZ_GLOBAL uint8_t *dst = tp ? gmem(J.seq) + lo : gmem(J.hpay) + lo;
    int zeros = 0; // code-0 count, checked against the outlier count
    if (!bad) {
        HIZ_GLOBAL const uint8_t *src = in + J.off_lcdata + base;
        if (size == (uint32_t)n) { // stored as it is
            copy_out(dst, FromGlobal{src}, n);
            if (tp) {
                for (int i = kPiece * t; i < n; i += kRound) {
                    if (i + kPiece <= n) {
                        const u4_any v = *reinterpret_cast<HIZ_GLOBAL const u4_any *>(src + i);
                        zeros += 16 - __popc(nonzero4(v.x)) - __popc(nonzero4(v.y)) -
                                 __popc(nonzero4(v.z)) - __popc(nonzero4(v.w));
                    } else {
                        for (int k = i; k < n; k++)
                            zeros += src[k] == 0;
                    }
                }
            }
        } else {
            for (int i = kPiece * t; i < (int)size; i += kRound) {
                if (i + kPiece <= (int)size)
                    *reinterpret_cast<u4_lds *>(S.a + i) =
                        *reinterpret_cast<HIZ_GLOBAL const u4_any *>(src + i);
                else
                    for (int k = i; k < (int)size; k++)
                        S.a[k] = src[k];
            }
            __syncthreads();
            if (tp) {
                bad = st_restore<1, false, kRounds>(
                          S.a, (int)size, n,
                          [&](int r, const uint4 &x) __attribute__((always_inline)) {
                              *reinterpret_cast<uint4 *>(S.b + kRound * r + kPiece * t) = x;
                          },
                          S) < 0;
                if (!bad)
                    zeros = st_planes_inv(S.b, n, dst);
            } else {
                // the length of what RRE_4 gave is in front of it
                const int n1 = st_restore<1, true, kMidRounds>(
                    S.a, (int)size, -1,
                    [&](int r, uint4 x) __attribute__((always_inline)) {
                        const int i = kRound * r + kPiece * t;
                        tcms8_piece<true>(x, i, S.a[0] | S.a[1] << 8);
                        *reinterpret_cast<uint4 *>(S.b + i) = x;
                    },
                    S);
                bad = n1 < 0 || st_restore<4, false, kRounds>(
                                    S.b, n1, n,
                                    [&](int r, const uint4 &x) __attribute__((always_inline)) {
                                        const int i = kRound * r + kPiece * t;
                                        if (i + kPiece <= n) {
                                            gstore_u4(dst + i, x);
                                        } else {
                                            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                                            for (int k = 0; k < kPiece; k++)
                                                if (i + k < n)
                                                    dst[i + k] = (uint8_t)(w[k / 4] >> (8 * (k & 3)));
                                        }
                                    },
                                    S) < 0;
            }
        }
    }
    if (bad) {
        if (t == 0)
            atomicOr(&st->flags, (uint32_t)ST_CORRUPT);
        for (int i = t; i < n; i += kLcThreads)
            dst[i] = 0;
        return;
    }
    if (tp) {
        for (int o = 32; o > 0; o >>= 1)
            zeros += __shfl_xor(zeros, o, 64);
        if ((t & 63) == 0 && zeros)
            atomicAdd((unsigned long long *)&st->zeros_seen, (unsigned long long)zeros);
    }
}

// ---- reordering by interpolation level (Sec. 5.1.4, Eq. reorder) -----------
// Level of a point: the largest l <= 4 with 2^l dividing every coordinate.
// Its index: points of coarser levels first (their count is the product of
// ceil(d / 2^(l+1)) over the axes), then the point's rank in row-major order
// among the level-l points, found on the grid of multiples of 2^l (sizes
// ceil(d / 2^l)) as its row-major index minus the coarser points before it.
// The anchor level is plain row-major order on the anchor grid.
__device__ inline uint64_t level_index(const Job &J, uint64_t x, uint64_t y, uint64_t z)
{
    const uint64_t any = x | y | z;
    const int l = any ? min(4, (int)__builtin_ctzll(any)) : 4;
    const uint64_t r = (1ull << l) - 1;
    const uint64_t Dy = (J.dims[1] + r) >> l, Dz = (J.dims[2] + r) >> l;
    const uint64_t xs = x >> l, ys = y >> l, zs = z >> l;
    uint64_t I = (xs * Dy + ys) * Dz + zs;
    if (l == 4)
        return I;
    const uint64_t r1 = (2ull << l) - 1;
    const uint64_t coarser = ((J.dims[0] + r1) >> (l + 1)) * ((J.dims[1] + r1) >> (l + 1)) *
                             ((J.dims[2] + r1) >> (l + 1));
    const uint64_t hy = (Dy + 1) >> 1, hz = (Dz + 1) >> 1;
    I -= ((xs + 1) >> 1) * hy * hz;
    if (!(xs & 1)) {
        I -= ((ys + 1) >> 1) * hz;
        if (!(ys & 1))
            I -= (zs + 1) >> 1;
    }
    return coarser + I;
}

// inverse = false: seq[I(x,y,z)] = codes[x,y,z]; inverse = true: the reverse.
// Threads take 16 consecutive z of a row, blockIdx.y is the job. In a row whose
// x and y are multiples of 2^l (and not both of 2^(l+1)) all multiples of 2^l
// along z are of level l and consecutive in the sequence; of the points between
// them, each finer level's are consecutive too. So a piece of 16 is one unaligned
// access of the row and one of the sequence per level, at most five, where single
// codes were 16: 256^3 codes 52 -> 18 us
// out, 52 -> 19 back.
typedef uint32_t u2_any __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u1_any __attribute__((aligned(1)));
typedef uint16_t h1_any __attribute__((aligned(1)));

template <bool INV>
__global__ __launch_bounds__(256) void k_reorder(const Job *__restrict__ jobs, int njobs)
{
    const Job &J = jobs[blockIdx.y];
    if (!J.reorder || (J.st->flags & (ST_CONST | ST_NONFINITE)))
        return;
    const uint64_t dz = J.dims[2];
    const uint64_t q = (dz + 15) / 16; // pieces per row
    const uint64_t n = J.dims[0] * J.dims[1] * q;
    HIZ_GLOBAL uint8_t *codes = gmem(J.codes);
    HIZ_GLOBAL uint8_t *seq = gmem(J.seq);
    for (uint64_t u = blockIdx.x * 256ull + threadIdx.x; u < n; u += 256ull * gridDim.x) {
        uint64_t row, x;
        if (n < 1ull << 32) { // (32-bit divisions where they do)
            row = (uint32_t)u / (uint32_t)q;
            x = (uint32_t)row / (uint32_t)J.dims[1];
        } else {
            row = u / q;
            x = row / J.dims[1];
        }
        const uint64_t z0 = (u - row * q) * 16, y = row - x * J.dims[1];
        const uint64_t g = row * dz + z0;
        if (dz - z0 < 16) {
            for (int k = 0; k < (int)(dz - z0); k++) {
                const uint64_t I = level_index(J, x, y, z0 + k);
                if (INV)
                    codes[g + k] = seq[I];
                else
                    seq[I] = codes[g + k];
            }
            continue;
        }
        // this piece's first code of level l in the sequence: at z0 when the
        // row's points are all of levels >= l, else at the first odd multiple
        const uint64_t xy = x | y;
        const int lr = xy ? min(4, (int)__builtin_ctzll(xy)) : 4;
        auto at = [&](int l) __attribute__((always_inline)) {
            return seq + level_index(J, x, y, lr == l ? z0 : z0 + (1ull << l));
        };
        if (!INV) {
            const u4_any w = *reinterpret_cast<HIZ_GLOBAL const u4_any *>(codes + g);
            if (lr == 0) {
                *reinterpret_cast<HIZ_GLOBAL u4_any *>(at(0)) = w;
                continue;
            }
            u2_any o, e;
            o.x = __builtin_amdgcn_perm(w.y, w.x, 0x07050301u);
            o.y = __builtin_amdgcn_perm(w.w, w.z, 0x07050301u);
            e.x = __builtin_amdgcn_perm(w.y, w.x, 0x06040200u);
            e.y = __builtin_amdgcn_perm(w.w, w.z, 0x06040200u);
            *reinterpret_cast<HIZ_GLOBAL u2_any *>(at(0)) = o;
            if (lr == 1) {
                *reinterpret_cast<HIZ_GLOBAL u2_any *>(at(1)) = e;
                continue;
            }
            const uint32_t f = __builtin_amdgcn_perm(e.y, e.x, 0x06040200u);
            *reinterpret_cast<HIZ_GLOBAL u1_any *>(at(1)) =
                __builtin_amdgcn_perm(e.y, e.x, 0x07050301u);
            if (lr == 2) {
                *reinterpret_cast<HIZ_GLOBAL u1_any *>(at(2)) = f;
                continue;
            }
            *reinterpret_cast<HIZ_GLOBAL h1_any *>(at(2)) =
                (uint16_t)((f >> 8 & 0xffu) | (f >> 16 & 0xff00u));
            const uint32_t h = (f & 0xffu) | (f >> 8 & 0xff00u);
            if (lr == 3) {
                *reinterpret_cast<HIZ_GLOBAL h1_any *>(at(3)) = (uint16_t)h;
                continue;
            }
            *at(3) = (uint8_t)(h >> 8);
            *at(4) = (uint8_t)h;
        } else {
            u4_any w;
            if (lr == 0) {
                w = *reinterpret_cast<HIZ_GLOBAL const u4_any *>(at(0));
            } else {
                const u2_any o = *reinterpret_cast<HIZ_GLOBAL const u2_any *>(at(0));
                u2_any e;
                if (lr == 1) {
                    e = *reinterpret_cast<HIZ_GLOBAL const u2_any *>(at(1));
                } else {
                    const uint32_t o1 = *reinterpret_cast<HIZ_GLOBAL const u1_any *>(at(1));
                    uint32_t f;
                    if (lr == 2) {
                        f = *reinterpret_cast<HIZ_GLOBAL const u1_any *>(at(2));
                    } else {
                        const uint32_t o2 = *reinterpret_cast<HIZ_GLOBAL const h1_any *>(at(2));
                        uint32_t h;
                        if (lr == 3)
                            h = *reinterpret_cast<HIZ_GLOBAL const h1_any *>(at(3));
                        else
                            h = (uint32_t)*at(4) | (uint32_t)*at(3) << 8;
                        f = __builtin_amdgcn_perm(o2, h, 0x05010400u);
                    }
                    e.x = __builtin_amdgcn_perm(o1, f, 0x05010400u);
                    e.y = __builtin_amdgcn_perm(o1, f, 0x07030602u);
                }
                w.x = __builtin_amdgcn_perm(o.x, e.x, 0x05010400u);
                w.y = __builtin_amdgcn_perm(o.x, e.x, 0x07030602u);
                w.z = __builtin_amdgcn_perm(o.y, e.y, 0x05010400u);
                w.w = __builtin_amdgcn_perm(o.y, e.y, 0x07030602u);
            }
            *reinterpret_cast<HIZ_GLOBAL u4_any *>(codes + g) = w;
        }
    }
}

// max_pieces: the most pieces of 16 codes of a row that a field has (rows of fewer
// codes are one each).
void launch_reorder(const Job *d_jobs, int njobs, uint64_t max_pieces, bool inverse, hipStream_t s)
{
    if (njobs == 0 || max_pieces == 0)
        return;
    uint64_t g = cdiv(max_pieces, 256);
    if (g > 16384)
        g = 16384;
    if (inverse)
        hipLaunchKernelGGL(k_reorder<true>, dim3((uint32_t)g, njobs), dim3(256), 0, s, d_jobs,
                           njobs);
    else
        hipLaunchKernelGGL(k_reorder<false>, dim3((uint32_t)g, njobs), dim3(256), 0, s, d_jobs,
                           njobs);
}

// ---- outliers of the row-major code array -----------------------------------
// Units of kLcChunk codes, claimed in order: count the code-0 points, take
// the outlier slot by look-back, write (index, exact value) ascending.
__global__ __launch_bounds__(256) void k_outliers(const Job *__restrict__ jobs, int njobs,
                                                  uint64_t total, Counters *cnt)
{
    __shared__ int s_scan[8];
    __shared__ uint32_t s_id;
    __shared__ uint64_t s_base;
    const int t = threadIdx.x;
    if (t == 0)
        s_id = atomicAdd(&cnt->ou_next, 1u);
    __syncthreads();
    const uint64_t id = s_id;
    if (id >= total)
        return;
    const Job &J = jobs[find_job<WK_OU>(jobs, njobs, id)];
    FieldState *st = J.st;
    if (st->flags & (ST_CONST | ST_NONFINITE))
        return;
    const uint64_t u = id - J.ou_begin;
    const uint64_t lo = u * kLcChunk;
    const int n = (int)min<uint64_t>(kLcChunk, J.N - lo);
    HIZ_GLOBAL const uint8_t *codes = gmem(J.codes) + lo;
    // 64 codes per thread, in a chunk's whole pieces 16 at a time (the code array
    // starts at a multiple of 256 bytes)
    constexpr int per = kLcChunk / 256;
    uint32_t w[per / 4];
    const int i0 = t * per;
    int z = 0;
    if (i0 + per <= n) {
#pragma unroll
        for (int k = 0; k < per / 16; k++) {
            const uint4 v = gload_u4(codes + i0 + 16 * k);
            w[4 * k] = v.x;
            w[4 * k + 1] = v.y;
            w[4 * k + 2] = v.z;
            w[4 * k + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < per / 4; k++) {
            w[k] = 0;
            for (int b = 0; b < 4; b++) {
                const int i = i0 + 4 * k + b;
                w[k] |= (uint32_t)(i < n ? codes[i] : 1u) << (8 * b);
            }
        }
    }
    // bit k of zero[h]: code 32 h + k is an outlier's
    uint32_t zero[per / 32];
#pragma unroll
    for (int h = 0; h < per / 32; h++) {
        zero[h] = 0;
#pragma unroll
        for (int k = 0; k < 8; k++)
            zero[h] |= (nonzero4(w[8 * h + k]) ^ 15u) << (4 * k);
        z += __popc(zero[h]);
    }
    int zt;
    const int zb = wg_excl_scan(z, s_scan, zt);
    if (t < 64) {
        const uint64_t b = lookback(J.lb_d, u, (uint64_t)zt);
        if (t == 0)
            s_base = b;
    }
    __syncthreads();
    uint64_t slot = s_base + zb;
    if (z) {
        const uint64_t cap = J.cap;
        const int ib = J.idx_bytes;
        HIZ_GLOBAL uint8_t *out = gmem(J.stream);
        const uint64_t oidx = st->off_oidx, oval = st->off_oval;
#pragma unroll
        for (int h = 0; h < per / 32; h++) {
            for (uint32_t m = zero[h]; m; m &= m - 1) {
                const uint64_t gi = lo + i0 + 32 * h + (__ffs((int)m) - 1);
                if (oidx + (slot + 1) * ib <= cap) {
                    if (ib == 4)
                        reinterpret_cast<HIZ_GLOBAL uint32_t *>(out + oidx)[slot] = (uint32_t)gi;
                    else
                        reinterpret_cast<HIZ_GLOBAL uint64_t *>(out + oidx)[slot] = gi;
                }
                if (oval + (slot + 1) * 4 <= cap)
                    reinterpret_cast<HIZ_GLOBAL float *>(out + oval)[slot] = gmem(J.field)[gi];
                slot++;
            }
        }
    }
    if (t == 0 && u == J.n_ou - 1 && s_base + zt != st->n_out)
        atomicOr(&st->flags, (uint32_t)ST_CORRUPT);
}

void launch_outliers(const Job *d_jobs, int njobs, uint64_t total, Counters *cnt, hipStream_t s)
{
    if (total == 0)
        return;
    hipLaunchKernelGGL(k_outliers, dim3((uint32_t)total), dim3(256), 0, s, d_jobs, njobs, total,
                       cnt);
}

void launch_lc_encode(const Job *d_jobs, int njobs, uint64_t total, Counters *cnt, hipStream_t s)
{
    if (total == 0)
        return;
    hipLaunchKernelGGL(k_lc_encode, dim3((uint32_t)total), dim3(kLcThreads), 0, s, d_jobs, njobs,
                       total, cnt);
}

void launch_lc_decode(const Job *d_jobs, int njobs, uint64_t total, Counters *cnt, hipStream_t s)
{
    if (total == 0)
        return;
    hipLaunchKernelGGL(k_lc_decode, dim3((uint32_t)total), dim3(kLcThreads), 0, s, d_jobs, njobs,
                       total, cnt);
}

} // namespace hiz
