// Transform-domain blind rotation at N = 1024 (the third schedule of the
// int8 path's rotation, same words as the other two).
//
// A negacyclic product of gadget digits u with a key polynomial K is exact
// integer arithmetic mod 2^32, so any exact way to compute the integers will
// do.  Here each product goes through a complex transform of N/2 points in
// double precision: the polynomial x is folded to z_j = x_j + i x_{j+N/2}
// (X^{N/2} = i at the 512 points used), the points are those of X^512 = i,
// and nine levels split X^m = e^(i theta) into X^{m/2} = +- e^(i theta/2).  A
// CMux step with L live slots then costs (L + 1) ell forward and 2 (L + 1)
// inverse transforms and (4 L + 4) ell N/2 complex multiply-adds instead of
// (8 L + 8) ell N^2 int8 operations, and each gate's accumulator stays in LDS.
// Three kernels: several gates per compute unit (fft_lean_kernel), one
// (fft_gate_kernel), and several compute units per gate (fft_team_kernel, the
// only one whose workgroups wait for each other, and only for those that run).
//
// Exactness.  A key coefficient is split K = 2^16 K_hi + K_lo with signed
// 16-bit halves; every accumulated product sum is then an integer below
// 2^37 in magnitude, and the double result is within 0.021 of it for every
// input, so rounding to the nearest integer recovers it.  With u = 2^-53: a
// forward butterfly's output carries a relative error (2-norm of the pair) of
// at most 4u (table entries u each, one rounding per fused multiply-add), nine
// levels 37u; an inverse one's 5u where it is scaled (subtraction, tangent,
// multiply-add, cosine, product), else 3u, seven and two levels and the final
// scale (4u) 45u; the sum of P products of transforms 2 sqrt(2) P u.  With M =
// sum over the P products of |u|_2 |K|_2 <= P (2^7 sqrt(N)) (2^15 sqrt(N)) =
// P 2^32, forward errors of digits and keys reach a result coefficient through
// Cauchy-Schwarz as 37u M each, the products' as 2 sqrt(2) P u M, and the
// inverse's 45u times the 2-norm of the result, at most sqrt(N) M.  For the
// largest P, (k + 1) ell = 27 at 8 parties: 27 2^-21 (74 + 76 + 32 * 45) =
// 0.0205.  Unsplit keys would be bounded by 2^16 times as much, so the split
// (twice the inverse transforms and products) is what makes the rounding
// exact for every key and ciphertext and not only for likely ones.  The
// rounding adds 1.5 2^52: the sum's low word is the integer mod 2^32.
//
// Butterflies are six fused multiply-adds (b (1 + i t) scaled by c, twiddle
// c (1 + i t): the cosine/tangent form of the fast Fourier transform's
// butterflies for fused multiply-adds, Linzer and Feig 1993).  A wave runs levels 1-8 of one transform with 8 points per
// lane: three levels in registers, two across lane bits 5 and 4
// (v_permlane32_swap, v_permlane16_swap), one exchange through LDS, three in
// registers.  Level 9 is done by the thread that owns the two frequencies and
// multiplies them with the keys, which are stored in that order.
//
// What bounds it: LDS and vector instruction issue together.  Measured on
// MI355X a ds_write_b128 takes 13 cycles of a compute unit's LDS and a
// ds_read_b128 5.5, so LDS traffic, not arithmetic, bounded the first form
// with every exchange through LDS (1024 gates: 33 ms, 17 ms with the
// exchanges taken out); the permutes replace one of three exchanges.
// Conflict-free words (struct Lane): a read's 16-lane phases, lanes with one
// parity of bits 2-4, hit 16 different 16-byte columns, a write's 8
// consecutive lanes 8.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>
#include <vector>

#include "mk_device_common.h"

namespace mk {

#define MK_HIP(call, what)                               \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) return hip_fail(e_, what); \
    } while (0)

namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

constexpr int kN = 1024;             // ring dimension
constexpr int kH = kN / 2;           // complex points of a transform
constexpr int kParts = 2;            // 16-bit halves of a key coefficient
constexpr int kPoly = kParts * kH;   // complex words of one transformed key polynomial
constexpr int kEll = 3;              // largest gadget length
constexpr double kMagic = 6755399441055744.0;   // 1.5 * 2^52

// Twiddle table (complex words of (cos, tan) pairs): levels 4 and 5 by lane /
// 16, four each; levels 6-8, four entries of 64 lanes; level 9 by thread.
constexpr int kTabP = 0, kTabQ = 16, kTab9 = kTabQ + 256;
// The same for transforms by a wave pair: levels 3 and 4 by lane / 16, two
// each; levels 5 and 6, 16 entries each; levels 7 and 8, 128 each.
constexpr int kTab2 = kTab9 + 256, kTab2Q = 8, kTab2R = kTab2Q + 32, kTab2Words = kTab2R + 256;
constexpr int kTabWords = kTab2 + kTab2Words;

struct Cx {
    double r, i;
};
struct Tw {
    double c, t;   // cos and tan of the twiddle's angle
};

// Angles pi/4; pi/8; pi/16, 5 pi/16
constexpr Tw kTwA[4] = {
    {0.70710678118654752440, 1.0},
    {0.92387953251128675613, 0.41421356237309504880},
    {0.98078528040323044913, 0.19891236737965800691},
    {0.55557023301960222474, 1.49660576266548901760},
};

template <bool ODD>
__device__ __forceinline__ void bf_fwd(Cx &a, Cx &b, double c, double t) {
    const double p = __builtin_fma(-t, b.i, b.r), q = __builtin_fma(t, b.r, b.i);
    if constexpr (!ODD) {
        b.r = __builtin_fma(-c, p, a.r);
        b.i = __builtin_fma(-c, q, a.i);
        a.r = __builtin_fma(c, p, a.r);
        a.i = __builtin_fma(c, q, a.i);
    } else {
        b.r = __builtin_fma(c, q, a.r);
        b.i = __builtin_fma(-c, p, a.i);
        a.r = __builtin_fma(-c, q, a.r);
        a.i = __builtin_fma(c, p, a.i);
    }
}

template <bool ODD, bool SCALE>
__device__ __forceinline__ void bf_inv(Cx &a, Cx &b, double c, double t) {
    const double dr = a.r - b.r, di = a.i - b.i;
    a.r += b.r;
    a.i += b.i;
    const double x = __builtin_fma(t, di, dr), y = __builtin_fma(-t, dr, di);
    b.r = ODD ? y : x;
    b.i = ODD ? -x : y;
    if constexpr (SCALE) {
        b.r *= c;
        b.i *= c;
    }
}

template <class TW>
__device__ __forceinline__ void radix8_fwd(Cx (&x)[8], TW tw) {
    {
        const Tw w = tw(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) bf_fwd<false>(x[r], x[r + 4], w.c, w.t);
    }
    {
        const Tw w = tw(1);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            bf_fwd<false>(x[r], x[r + 2], w.c, w.t);
            bf_fwd<true>(x[r + 4], x[r + 6], w.c, w.t);
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const Tw w = tw(2 + h);
        bf_fwd<false>(x[4 * h], x[4 * h + 1], w.c, w.t);
        bf_fwd<true>(x[4 * h + 2], x[4 * h + 3], w.c, w.t);
    }
}

// Hides a lane index from loop-invariant code motion: the LDS addresses formed
// from it are formed where they are used instead of living across a whole
// step in registers.
__device__ __forceinline__ int here(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}

__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Barrier that orders LDS accesses only (loads of keys stay in flight).
__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS is addressed by byte offsets from the start of the workgroup's block, so
// that a word's exclusive-or pattern is one instruction away from its address.
extern __shared__ __align__(16) unsigned char smem[];
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(3))) d2 lds_d2;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ lds_byte *lds_at(uint32_t off) { return (lds_byte *)smem + off; }
__device__ __forceinline__ Cx ld(uint32_t off) {
    const d2 v = *(lds_d2 *)lds_at(off);
    return {v.x, v.y};
}
__device__ __forceinline__ void st(uint32_t off, const Cx &v) { *(lds_d2 *)lds_at(off) = d2{v.r, v.i}; }
__device__ __forceinline__ uint32_t ldw(uint32_t off) { return *(lds_u32 *)lds_at(off); }
__device__ __forceinline__ void stw(uint32_t off, uint32_t v) { *(lds_u32 *)lds_at(off) = v; }
__device__ __forceinline__ void addw(uint32_t off, uint32_t v) {
    __hip_atomic_fetch_add((lds_u32 *)lds_at(off), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
constexpr uint32_t kBufBytes = kH * 16;   // one transform
constexpr uint32_t kRowBytes = kN * 4;    // one polynomial
constexpr size_t kLdsBytes = 160 * 1024;  // of a compute unit

// Exchanges the register pair's bit with lane bit 5 (W = 32) or 4 (W = 16).
template <int W>
__device__ __forceinline__ void swap_word(uint32_t &a, uint32_t &b) {
    if constexpr (W == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    }
}
template <int W>
__device__ __forceinline__ void swap_bit(double &a, double &b) {
    uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32), yl = (uint32_t)y, yh = (uint32_t)(y >> 32);
    swap_word<W>(xl, yl);
    swap_word<W>(xh, yh);
    a = __builtin_bit_cast(double, (uint64_t)xh << 32 | xl);
    b = __builtin_bit_cast(double, (uint64_t)yh << 32 | yl);
}
template <int W>
__device__ __forceinline__ void swap_bit(Cx &a, Cx &b) {
    swap_bit<W>(a.r, b.r);
    swap_bit<W>(a.i, b.i);
}

// LDS bytes of point j = (j8 .. j0) of a transform for this lane's two
// layouts.  Packed, so that they can stay in two registers.
struct Lane {
    uint32_t e, h;   // exchange (outer | inner << 16) and hand-over (inner)
    __device__ __forceinline__ explicit Lane(int l) {
        // outer: lane (j8 j7 j3 j2 j1 j0), registers (j5 j4 j6)
        const int o8 = l >> 5, o7 = (l >> 4) & 1;
        const int outer = (l >> 4) * 128 + ((l & 15) ^ ((o8 ^ o7) << 3) ^ (o7 << 2));
        // inner: lane (j4 j5 j8 j7 j6 j0), registers (j3 j2 j1)
        const int j0 = l & 1, j6 = (l >> 1) & 1, j7 = (l >> 2) & 1, j8 = (l >> 3) & 1, j5 = (l >> 4) & 1, j4 = l >> 5;
        const int b5 = j8 * 16 + j7 * 8 + j6 * 4 + j5 * 2 + j4;
        const int inner = b5 * 16 + (j0 ^ ((j8 ^ j7) << 3) ^ (j7 << 2) ^ (j6 << 1));
        e = (uint32_t)outer * 16 | (uint32_t)inner << 20;
        h = (uint32_t)(j0 * 256 + (b5 >> 1) * 16 + ((j4 ^ j8) << 3) + (j7 * 4 + j6 * 2 + j0)) * 16;
    }
    __device__ __forceinline__ Lane here() const {   // see here(int)
        Lane v = *this;
        asm volatile("" : "+v"(v.e), "+v"(v.h));
        return v;
    }
    // register r of the outer layout, of the inner one, and its hand-over word,
    // in the buffer at `buf` (a multiple of 4 KB)
    __device__ __forceinline__ uint32_t outer(uint32_t buf, int r) const {
        const uint32_t b = buf + (e & 0xFFFFu);
        return ((r & 1) ? (b ^ 32u) + 1024u : b) + (uint32_t)((r >> 2) * 512 + ((r >> 1) & 1) * 256);
    }
    __device__ __forceinline__ uint32_t inner(uint32_t buf, int r) const { return (buf + (e >> 16)) ^ (uint32_t)(32 * r); }
    __device__ __forceinline__ uint32_t hand(uint32_t buf, int r) const { return (buf + h) ^ (uint32_t)(16 * r); }
};
// Hand-over word of thread c = (j8 .. j1), j0 = 0 (j0 = 1: 256 + (word ^ 1))
__device__ __forceinline__ int owner_word(int c) {
    return (c & ~15) | ((((c >> 3) ^ (c >> 7)) & 1) << 3) | ((c & 7) ^ (((c >> 6) & 1) << 2) ^ (((c >> 5) & 1) << 1));
}

// Levels 1 .. 8 of a transform by one wave.  x[r]: point 64 r + lane; the
// result goes to `buf` in hand-over order.
__device__ __forceinline__ void fwd_levels(Cx (&x)[8], int l, const Lane &at, uint32_t buf, const d2 *tab) {
    d2 tp[4], tq[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) tp[i] = tab[kTabP + (l >> 4) * 4 + i];
    radix8_fwd(x, [](int i) { return kTwA[i]; });
#pragma unroll
    for (int i = 0; i < 4; ++i) tq[i] = tab[kTabQ + 64 * i + l];
#pragma unroll
    for (int r = 0; r < 4; ++r) swap_bit<32>(x[r], x[r + 4]);
#pragma unroll
    for (int j7 = 0; j7 < 2; ++j7) {   // level 4
        bf_fwd<false>(x[2 * j7], x[2 * j7 + 4], tp[j7].x, tp[j7].y);
        bf_fwd<true>(x[2 * j7 + 1], x[2 * j7 + 5], tp[j7].x, tp[j7].y);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        swap_bit<16>(x[r], x[r + 2]);
        swap_bit<16>(x[r + 4], x[r + 6]);
    }
#pragma unroll
    for (int j6 = 0; j6 < 2; ++j6) {   // level 5
        bf_fwd<false>(x[j6], x[j6 + 2], tp[2 + j6].x, tp[2 + j6].y);
        bf_fwd<true>(x[j6 + 4], x[j6 + 6], tp[2 + j6].x, tp[2 + j6].y);
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) st(at.outer(buf, r), x[r]);
    wave_fence();
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = ld(at.inner(buf, r));
    radix8_fwd(x, [&](int i) { return Tw{tq[i].x, tq[i].y}; });
    wave_fence();
#pragma unroll
    for (int r = 0; r < 8; ++r) st(at.hand(buf, r), x[r]);
}

// Digit (24 - sh) / 8 of the coefficients y, FLIP: y still has its bias.
template <bool FLIP>
__device__ __forceinline__ void wave_fwd(uint32_t y, int sh, int lane, const Lane &lane_at, uint32_t buf, const d2 *tab) {
    const int l = here(lane);
    const Lane at = lane_at.here();
    const uint32_t yl = y + 4u * (uint32_t)l;
    Cx x[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        uint32_t a = ldw(yl + 256u * r), b = ldw(yl + 256u * r + kRowBytes / 2);
        if constexpr (FLIP) {
            a ^= 0x80808080u;
            b ^= 0x80808080u;
        }
        x[r].r = (double)(int)__builtin_amdgcn_sbfe(a, sh, 8);
        x[r].i = (double)(int)__builtin_amdgcn_sbfe(b, sh, 8);
    }
    fwd_levels(x, l, at, buf, tab);
}

__device__ __forceinline__ uint32_t round_word(double x, double s) {
    const double v = __builtin_fma(x, s, kMagic);
    return (uint32_t)__builtin_bit_cast(uint64_t, v);
}

// ------------------------------------------- transforms by a wave pair ----
//
// For short latency: 128 lanes hold four points each, the exchange through LDS
// is between the two waves, and every transform has two halves with a
// workgroup barrier between them.  Per wave half the arithmetic and half the
// LDS words of a transform by one wave: where compute units have few
// transforms at a time one takes 2.2k cycles instead of 2.8k (team kernel, one
// gate at 2 parties 8.2 -> 7.6 ms), with nine at a time they are bound by
// instruction issue either way (gate kernel, 9.4 -> 8.9 ms at 2 parties).  A wave's inner and hand-over words are
// the same half of the buffer (j8), so neither wave overwrites words that the
// other has yet to read.

struct Lane2 {
    uint32_t e, h;   // exchange (outer | inner << 16) and hand-over (inner)
    uint32_t io;     // words: of y (packed order) | of an accumulator << 16
    __device__ __forceinline__ Lane2(int l, int w) {
        {   // outer: lane (j8 j7 j3 j2 j1 j0), wave j4, registers (j6 j5)
            const int j7 = (l >> 4) & 1;
            e = 16u * (uint32_t)((l >> 4) * 128 + w * 16 + ((l & 15) ^ (j7 << 1)));
            // before the permutes: lane (j6 j5 j3 j2 j1 j0), registers (j8 j7)
            io = 4u * (uint32_t)(w * 64 + l) | (4u * (uint32_t)((l >> 4) * 32 + w * 16 + (l & 15))) << 16;
        }
        {   // inner: lane (j2 j1 j5 j6 j7 j0), wave j8, registers (j4 j3); after
            // the permutes lane (j4 j3 j5 j6 j7 j0), registers (j2 j1)
            const int j0 = l & 1, j7 = (l >> 1) & 1, j6 = (l >> 2) & 1, j5 = (l >> 3) & 1, x4 = (l >> 4) & 1, x5 = l >> 5;
            const int b4 = w * 8 + j7 * 4 + j6 * 2 + j5;
            e |= 16u * (uint32_t)(b4 * 32 + ((j5 << 3) ^ ((x5 ^ j6) << 2) ^ ((x4 ^ j7) << 1) ^ j0)) << 16;
            h = 16u * (uint32_t)(w * 256 + j0 * 128 + (b4 & 7) * 16 + ((x5 ^ j6) << 3) + ((x4 ^ j6) << 2) + (j7 << 1) + j0);
        }
    }
    __device__ __forceinline__ Lane2 here() const {
        Lane2 v = *this;
        asm volatile("" : "+v"(v.e), "+v"(v.h), "+v"(v.io));
        return v;
    }
    __device__ __forceinline__ uint32_t outer(uint32_t buf, int r) const {   // r = (j6 j5)
        return ((buf + (e & 0xFFFFu)) ^ (uint32_t)((r & 1) * 128 + (r >> 1) * 64)) + (uint32_t)((r >> 1) * 1024 + (r & 1) * 512);
    }
    __device__ __forceinline__ uint32_t inner(uint32_t buf, int r) const {   // r = (j4 j3)
        return ((buf + (e >> 16)) ^ (uint32_t)((r & 1) * 128)) + (uint32_t)((r >> 1) * 256);
    }
    __device__ __forceinline__ uint32_t hand(uint32_t buf, int r) const { return (buf + h) ^ (uint32_t)(16 * r); }   // (j2 j1)
};
// Byte of coefficient m in y's order (j4 above j6)
__device__ __forceinline__ uint32_t packed_byte(int m) {
    return 4u * (uint32_t)((m & ~0x70) | ((m & 0x10) << 2) | ((m & 0x60) >> 1));
}
// Hand-over word of thread c = (j8 .. j1), j0 = 0 (j0 = 1: 128 + (word ^ 1))
__device__ __forceinline__ int owner_word2(int c) {
    const int j7 = (c >> 6) & 1, j6 = (c >> 5) & 1;
    return ((c & 128) << 1) | ((c & 127) ^ (j7 << 1) ^ (j6 << 2) ^ (j6 << 3));
}

// Coefficients from y, in y's order; FLIP: they still have their bias.
template <bool FLIP>
struct FromY {
    uint32_t y;
    __device__ __forceinline__ void operator()(const Lane2 &at, int r, uint32_t &a, uint32_t &b) const {
        const uint32_t yl = y + (at.io & 0xFFFFu);
        a = ldw(yl + 512u * r);
        b = ldw(yl + 512u * r + kRowBytes / 2);
        if constexpr (FLIP) {
            a ^= 0x80808080u;
            b ^= 0x80808080u;
        }
    }
};
// `words(at, r, a, b)`: biased coefficients 128 r + .. and 512 + 128 r + ..
template <class Words>
__device__ __forceinline__ void pair_fwd_a(Words words, int sh, int lane, const Lane2 &lane_at, uint32_t buf, const d2 *tab2) {
    const int l = here(lane);
    const Lane2 at = lane_at.here();
    const d2 t3 = tab2[(l >> 4) * 2], t4 = tab2[(l >> 4) * 2 + 1];
    Cx x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        uint32_t a, b;
        words(at, r, a, b);
        x[r].r = (double)(int)__builtin_amdgcn_sbfe(a, sh, 8);
        x[r].i = (double)(int)__builtin_amdgcn_sbfe(b, sh, 8);
    }
    bf_fwd<false>(x[0], x[2], kTwA[0].c, kTwA[0].t);
    bf_fwd<false>(x[1], x[3], kTwA[0].c, kTwA[0].t);
    bf_fwd<false>(x[0], x[1], kTwA[1].c, kTwA[1].t);
    bf_fwd<true>(x[2], x[3], kTwA[1].c, kTwA[1].t);
    swap_bit<32>(x[0], x[2]);
    swap_bit<32>(x[1], x[3]);
    bf_fwd<false>(x[0], x[2], t3.x, t3.y);
    bf_fwd<true>(x[1], x[3], t3.x, t3.y);
    swap_bit<16>(x[0], x[1]);
    swap_bit<16>(x[2], x[3]);
    bf_fwd<false>(x[0], x[1], t4.x, t4.y);
    bf_fwd<true>(x[2], x[3], t4.x, t4.y);
#pragma unroll
    for (int r = 0; r < 4; ++r) st(at.outer(buf, r), x[r]);
}
__device__ __forceinline__ void pair_fwd_b(int lane, int w, const Lane2 &lane_at, uint32_t buf, const d2 *tab2) {
    const int l = here(lane);
    const Lane2 at = lane_at.here();
    Cx x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = ld(at.inner(buf, r));
    const d2 *tq = tab2 + kTab2Q + w * 8 + ((l >> 1) & 7), *tr = tab2 + kTab2R + w * 64 + l;
    const d2 t5 = tq[0], t6 = tq[16], t7 = tr[0], t8 = tr[128];
    bf_fwd<false>(x[0], x[2], t5.x, t5.y);
    bf_fwd<false>(x[1], x[3], t5.x, t5.y);
    bf_fwd<false>(x[0], x[1], t6.x, t6.y);
    bf_fwd<true>(x[2], x[3], t6.x, t6.y);
    swap_bit<32>(x[0], x[2]);
    swap_bit<32>(x[1], x[3]);
    bf_fwd<false>(x[0], x[2], t7.x, t7.y);
    bf_fwd<true>(x[1], x[3], t7.x, t7.y);
    swap_bit<16>(x[0], x[1]);
    swap_bit<16>(x[2], x[3]);
    bf_fwd<false>(x[0], x[1], t8.x, t8.y);
    bf_fwd<true>(x[2], x[3], t8.x, t8.y);
    wave_fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) st(at.hand(buf, r), x[r]);
}
__device__ __forceinline__ void pair_inv_a(int lane, int w, const Lane2 &lane_at, uint32_t buf, const d2 *tab2) {
    const int l = here(lane);
    const Lane2 at = lane_at.here();
    Cx x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = ld(at.hand(buf, r));
    const d2 *tq = tab2 + kTab2Q + w * 8 + ((l >> 1) & 7), *tr = tab2 + kTab2R + w * 64 + l;
    const d2 t5 = tq[0], t6 = tq[16], t7 = tr[0], t8 = tr[128];
    bf_inv<false, true>(x[0], x[1], t8.x, t8.y);
    bf_inv<true, true>(x[2], x[3], t8.x, t8.y);
    swap_bit<16>(x[0], x[1]);
    swap_bit<16>(x[2], x[3]);
    bf_inv<false, true>(x[0], x[2], t7.x, t7.y);
    bf_inv<true, true>(x[1], x[3], t7.x, t7.y);
    swap_bit<32>(x[0], x[2]);
    swap_bit<32>(x[1], x[3]);
    bf_inv<false, true>(x[0], x[1], t6.x, t6.y);
    bf_inv<true, true>(x[2], x[3], t6.x, t6.y);
    bf_inv<false, true>(x[0], x[2], t5.x, t5.y);
    bf_inv<false, true>(x[1], x[3], t5.x, t5.y);
    wave_fence();
#pragma unroll
    for (int r = 0; r < 4; ++r) st(at.inner(buf, r), x[r]);
}
// Where an inverse's words go: added to an accumulator row or (packed) to y, or
// stored in y.
struct Add {
    uint32_t dst;
    bool packed;
    __device__ __forceinline__ void operator()(const Lane2 &at, int r, uint32_t a, uint32_t b) const {
        const uint32_t dl = dst + (packed ? at.io & 0xFFFFu : at.io >> 16);
        addw(dl + 512u * r, a);
        addw(dl + 512u * r + kRowBytes / 2, b);
    }
};
struct SetY {
    uint32_t dst;
    __device__ __forceinline__ void operator()(const Lane2 &at, int r, uint32_t a, uint32_t b) const {
        const uint32_t dl = dst + (at.io & 0xFFFFu);
        stw(dl + 512u * r, a);
        stw(dl + 512u * r + kRowBytes / 2, b);
    }
};

template <class Out>
__device__ __forceinline__ void pair_inv_b(uint32_t buf, Out out, int sh, int lane, const Lane2 &lane_at, const d2 *tab2) {
    const int l = here(lane);
    const Lane2 at = lane_at.here();
    Cx x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = ld(at.outer(buf, r));
    const d2 t3 = tab2[(l >> 4) * 2], t4 = tab2[(l >> 4) * 2 + 1];
    bf_inv<false, true>(x[0], x[1], t4.x, t4.y);
    bf_inv<true, true>(x[2], x[3], t4.x, t4.y);
    swap_bit<16>(x[0], x[1]);
    swap_bit<16>(x[2], x[3]);
    bf_inv<false, true>(x[0], x[2], t3.x, t3.y);
    bf_inv<true, true>(x[1], x[3], t3.x, t3.y);
    swap_bit<32>(x[0], x[2]);
    swap_bit<32>(x[1], x[3]);
    bf_inv<false, false>(x[0], x[1], kTwA[1].c, kTwA[1].t);
    bf_inv<true, false>(x[2], x[3], kTwA[1].c, kTwA[1].t);
    bf_inv<false, false>(x[0], x[2], kTwA[0].c, kTwA[0].t);
    bf_inv<false, false>(x[1], x[3], kTwA[0].c, kTwA[0].t);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double s = (1.0 / kH) * ((r & 1) ? kTwA[1].c : 1.0) * ((r & 2) ? kTwA[0].c : 1.0);
        out(at, r, round_word(x[r].r, s) << sh, round_word(x[r].i, s) << sh);
    }
}

__device__ __forceinline__ void mac(Cx &s, const Cx &u, const d2 &k) {
    s.r = __builtin_fma(u.r, k.x, __builtin_fma(-u.i, k.y, s.r));
    s.i = __builtin_fma(u.r, k.y, __builtin_fma(u.i, k.x, s.i));
}

// Words of consecutive transformed key polynomials [poly][part][j0][256]
// through a wave-uniform descriptor: one vector offset for all loads.
struct KeyBlock {
    __amdgpu_buffer_rsrc_t r;
    uint32_t lane;
    __device__ __forceinline__ KeyBlock(const d2 *base, int polys, int word)
        : r(__builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, polys * kPoly * 16, 0x00020000)),
          lane(16u * (uint32_t)word) {}
    __device__ __forceinline__ d2 operator()(int w) const {
        const u4 v = __builtin_amdgcn_raw_buffer_load_b128(r, lane, 16 * w, 0);
        return __builtin_bit_cast(d2, v);
    }
};

// ------------------------------------------------------------- upload ----

__global__ __launch_bounds__(256) void fft_key_kernel(const uint32_t *__restrict__ ext, const d2 *__restrict__ tab,
                                                      d2 *__restrict__ out) {
    const size_t poly = blockIdx.x;
    const uint32_t *K = ext + poly * 2 * kN + kN;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    if (wave < kParts) {   // part 0: low 16 bits (signed), part 1: the rest
        const int l = tid & 63;
        auto part = [&](int m) {
            const uint32_t w = K[m];
            const int lo = (int16_t)(w & 0xFFFFu);
            return (double)(wave ? (int)(int16_t)((w - (uint32_t)lo) >> 16) : lo);
        };
        Cx x[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) x[r] = {part(l + 64 * r), part(l + 64 * r + kH)};
        fwd_levels(x, l, Lane(l), wave * kBufBytes, tab);
    }
    __syncthreads();
    const d2 t9 = tab[kTab9 + tid];
    const uint32_t at0 = 16u * owner_word(tid), at1 = 4096u + (at0 ^ 16u);
    for (int p = 0; p < kParts; ++p) {
        Cx a = ld(p * kBufBytes + at0), b = ld(p * kBufBytes + at1);
        bf_fwd<false>(a, b, t9.x, t9.y);
        out[poly * kPoly + p * kH + tid] = d2{a.r, a.i};
        out[poly * kPoly + p * kH + 256 + tid] = d2{b.r, b.i};
    }
}

// ----------------------------------------------------------- rotation ----

struct FftArgs {
    int k, n, ell, G, st0, st1;
    uint32_t offset;
    const uint32_t *abar;   // [G][kn+1]
    uint32_t *acc;          // [G][k+1][N]
    const d2 *bk;           // [k][n][3][ell][part][j0][256]
    const d2 *evk;          // [k+1][ell][part][j0][256]
    const d2 *tab;
    // teams (fft_team_kernel)
    uint64_t *xch;          // boxes [G][members][2][N]
    uint32_t *form;         // [G]: members that run, kApart (form_team)
    uint32_t *status;
    int members, nx, form_polls;
};

// Set in a gate's word: its team did not form, one workgroup runs the steps.
constexpr uint32_t kApart = 1u << 31;

// Accumulators of one gate: X^-b v, 0, .. at the start, else the rows saved before.
template <int T>
__device__ __forceinline__ void load_acc(const FftArgs &a, int g, const uint32_t *abar, uint32_t acc) {
    const int words = (a.k + 1) * kN;
    for (int idx = threadIdx.x; idx < words; idx += T) {
        uint32_t v = 0;
        if (a.st0 > 0) {
            v = a.acc[(size_t)g * words + idx];
        } else if (idx < kN) {
            const int s = idx + (int)abar[0];
            const uint32_t tv = (s & (kN - 1)) < kN / 2 ? 0xE0000000u : 0x20000000u;
            v = (s & kN) ? 0u - tv : tv;
        }
        stw(acc + 4u * idx, v);
    }
}

// X^-shift c - c into y, biased for digit extraction.
template <int T, bool PACKED>
__device__ __forceinline__ void rotate(uint32_t c, int shift, uint32_t offset, int tid, uint32_t y) {
#pragma unroll
    for (int i = 0; i < kN / T; ++i) {
        const int m = tid + T * i, s = m + shift;
        const uint32_t src = ldw(c + 4u * (uint32_t)(s & (kN - 1))), rot = (s & kN) ? 0u - src : src;
        stw(y + (PACKED ? packed_byte(m) : 4u * m), (rot - ldw(c + 4u * m) + offset) ^ 0x80808080u);
    }
}

// Rotation amounts of the next 64 steps, one per lane: a load per step would
// have to wait for the key loads in flight before it.
struct Shifts {
    const uint32_t *abar;   // of step 0
    int end, lane;
    uint32_t v;
    __device__ __forceinline__ int operator()(int step, int first) {
        const int i = (step - first) & 63;
        if (i == 0) v = abar[min(step + lane, end - 1)];
        return (int)__builtin_amdgcn_readlane(v, i);
    }
};

// The thread's two frequencies of the transform in `buf`, and back.
struct Owner {
    uint32_t at0, at1;
    double c, t;
    // hand-over words of j0 = 0 and, `apart` words on, of j0 = 1
    __device__ __forceinline__ Owner(int c_, int word, int apart, const d2 *tab)
        : at0(16u * (uint32_t)word), at1(16u * (uint32_t)(apart + (word ^ 1))) {
        const d2 v = tab[kTab9 + c_];
        c = v.x;
        t = v.y;
    }
    __device__ __forceinline__ void get(uint32_t buf, Cx &u, Cx &v) const {
        u = ld(buf + at0);
        v = ld(buf + at1);
        bf_fwd<false>(u, v, c, t);
    }
    __device__ __forceinline__ void put(uint32_t buf, const Cx (&s)[2]) const {
        Cx p = s[0], q = s[1];
        bf_inv<false, true>(p, q, c, t);
        st(buf + at0, p);
        st(buf + at1, q);
    }
};

// Several gates per compute unit (four up to two parties): what one gate's
// workgroup cannot use of a compute unit another's does.  Forward transforms
// by single waves, the digits of a slot at a time; inverse ones, of which there
// are two at a time, by wave pairs, so that all four waves have work (against
// single waves 768 gates at 4 parties 63.8 -> 62.0 ms, 2600 at 2 78.8 -> 77.8).
// Vector instructions issue about 60 % of the time; the rest is the latency of
// LDS and of the keys, which 128 registers leave no room to fetch ahead.
// Measured (MI355X, 2 parties): 1024 gates 31.0 ms.
constexpr int kLeanT = 256;
constexpr int kLeanBufs = 3;

template <int ELL>
__global__ __launch_bounds__(kLeanT, 4) void fft_lean_kernel(FftArgs a) {
    constexpr int ell = ELL;
    const int K1 = a.k + 1, tid = threadIdx.x;
    // LDS: accumulators [K1][N], y [N], transforms [kLeanBufs][H]
    const uint32_t acc = 0, y = K1 * kRowBytes, buf = y + kRowBytes;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid & 63;
    const int g = blockIdx.x;
    const uint32_t *abar = a.abar + (size_t)g * (a.k * a.n + 1);
    const d2 *tab = a.tab;
    const Owner own(tid, owner_word(tid), 256, tab);
    const Lane at(l);
    const int pair = wave >> 1, w2 = wave & 1;
    const Lane2 at2(l, w2);
    const d2 *tab2 = tab + kTab2;
    const Owner back(tid, owner_word2(tid), 128, tab);   // for inverse transforms
    load_acc<kLeanT>(a, g, abar, acc);
    int shift = a.st0 < a.st1 ? (int)abar[1 + a.st0] : 0;
    int turn = (int)(blockIdx.x >> 3) + (int)(blockIdx.x >> 8);
    __syncthreads();
    for (int step = a.st0; step < a.st1; ++step) {
        const int party = step / a.n, bit = step - party * a.n;
        const int next_shift = step + 1 < a.st1 ? (int)abar[2 + step] : 0;
        const KeyBlock kd(a.bk + ((size_t)party * a.n + bit) * 3 * ell * kPoly, 3 * ell, tid), ke(a.evk, K1 * ell, tid);
        auto rot = [&](int j) { rotate<kLeanT, false>(acc + j * kRowBytes, shift, a.offset, here(tid), y); };
        // products of the ell transforms with two key polynomials each
        auto madd = [&](const KeyBlock &k0, int p0, Cx (&c0)[kParts][2], const KeyBlock &k1, int p1, Cx (&c1)[kParts][2]) {
            lds_sync();
#pragma unroll 1
            for (int d = 0; d < ell; ++d) {
                d2 x0[kParts][2], x1[kParts][2];
#pragma unroll
                for (int p = 0; p < kParts; ++p)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        x0[p][s] = k0((p0 + d) * kPoly + p * kH + s * 256);
                        x1[p][s] = k1((p1 + d) * kPoly + p * kH + s * 256);
                    }
                Cx u, v;
                own.get(buf + d * kBufBytes, u, v);
#pragma unroll
                for (int p = 0; p < kParts; ++p) {
                    mac(c0[p][0], u, x0[p][0]);
                    mac(c0[p][1], v, x0[p][1]);
                    mac(c1[p][0], u, x1[p][0]);
                    mac(c1[p][1], v, x1[p][1]);
                }
            }
        };
        // digit by digit round the waves
        auto forward = [&](auto flip) {
            const int v = (wave - turn) & 3;
            turn += ell;
            if (v < ell) wave_fwd<decltype(flip)::value>(y, 24 - 8 * v, l, at, buf + v * kBufBytes, tab);
        };
        // transforms in buffers b0 and b1, a wave pair each
        auto inverse = [&](int b0, int b1, uint32_t dst) {   // low and high part
            const uint32_t b = buf + (pair ? b1 : b0) * kBufBytes;
            pair_inv_a(l, w2, at2, b, tab2);
            lds_sync();
            pair_inv_b(b, Add{dst, false}, 16 * pair, l, at2, tab2);
        };
        Cx w[kParts][2] = {};
        rot(party > 0 ? 1 : 0);
        for (int j = 1; j <= party; ++j) {   // slots without a stage-2 part
            lds_sync();
            forward(std::false_type{});
            Cx cT[kParts][2] = {};
            madd(ke, j * ell, w, kd, 0, cT);
            lds_sync();
            back.put(buf, cT[0]);
            back.put(buf + kBufBytes, cT[1]);
            rot(j < party ? j + 1 : 0);
            lds_sync();
            inverse(0, 1, acc + j * kRowBytes);
        }
        lds_sync();
        forward(std::false_type{});
        Cx cA[kParts][2] = {}, cB[kParts][2] = {};
        madd(ke, 0, w, kd, 0, cA);
        rot(1 + party);
        lds_sync();
        forward(std::false_type{});
        madd(ke, (1 + party) * ell, w, kd, 0, cB);
        for (int i = tid; i < kN; i += kLeanT) stw(y + 4u * i, a.offset);
        lds_sync();
        back.put(buf, w[0]);
        back.put(buf + kBufBytes, w[1]);
        lds_sync();
        inverse(0, 1, y);
        lds_sync();
        forward(std::true_type{});
        madd(kd, ell, cA, kd, 2 * ell, cB);
        lds_sync();
        back.put(buf, cA[0]);
        back.put(buf + kBufBytes, cA[1]);
        back.put(buf + 2 * kBufBytes, cB[0]);
        lds_sync();
        inverse(0, 1, acc);
        lds_sync();
        back.put(buf, cB[1]);
        lds_sync();
        inverse(2, 0, acc + (1 + party) * kRowBytes);
        shift = next_shift;
        lds_sync();
    }
    __syncthreads();
    for (int idx = tid; idx < K1 * kN; idx += kLeanT) a.acc[(size_t)g * K1 * kN + idx] = ldw(acc + 4u * idx);
}

size_t fft_lean_lds(int k) { return (size_t)(k + 2) * kN * 4 + (size_t)kLeanBufs * kH * 16; }

// One gate per compute unit.  Bound by the serial chain of a step (rotate,
// digits forward, products, V back, forward, products, back: 18k cycles at two
// parties), half of it instruction issue of the first transforms and products.
// A word's two key parts are two threads', so that the keys of a step fit
// registers and can be loaded a phase before their use, in small groups between
// the transforms' halves: a wave that meets a full memory pipe stalls, whatever
// it wanted to do next.  Measured (2 / 4 parties, up to 256 gates): 8.8 / 22.3
// ms; 9.4 / 22.7 with transforms by single waves and keys loaded in one go.
constexpr int kGateT = 512;           // threads: part tid / 256 of word tid % 256
constexpr int kGateP = kGateT / 128;  // wave pairs
constexpr int kSlots = 3;             // slots whose digits are transformed together
constexpr int kFwd = kSlots * kEll;   // buffers of digit transforms
constexpr int kGateBufs = kFwd + 4;   // and of inverse transforms

// LEFT: behind a team launch, the gates that it left.
template <int ELL, bool LEFT>
__global__ __launch_bounds__(kGateT, 2) void fft_gate_kernel(FftArgs a) {
    constexpr int ell = ELL;
    const int K1 = a.k + 1, tid = threadIdx.x;
    // LDS: accumulators [K1][N], y [kSlots][N], transforms [kGateBufs][H],
    // twiddles [kTab2Words]
    const uint32_t acc = 0, y = K1 * kRowBytes, buf = y + kSlots * kRowBytes;
    d2 *tab = reinterpret_cast<d2 *>(smem + buf + kGateBufs * kBufBytes);
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid & 63;
    const int part = __builtin_amdgcn_readfirstlane(tid / 256);
    const int g = blockIdx.x;
    if constexpr (LEFT) {
        const uint32_t f = __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.form + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        __syncthreads();
        if (tid == 0) __hip_atomic_store(a.form + g, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!(f & kApart)) return;
    }
    const uint32_t *abar = a.abar + (size_t)g * (a.k * a.n + 1);
    const Owner own(tid & 255, owner_word2(tid & 255), 128, a.tab);
    const int pair = wave >> 1, w2 = wave & 1;
    const Lane2 at(l, w2);
    const int word = part * kH + (tid & 255);
    if (tid < kTab2Words) tab[tid] = a.tab[kTab2 + tid];
    load_acc<kGateT>(a, g, abar, acc);
    int shift = a.st0 < a.st1 ? (int)abar[1 + a.st0] : 0;
    __syncthreads();
    const KeyBlock ke(a.evk, K1 * ell, word);
    // keys [digit][j0]: d of the step, b of the first three slots
    d2 xd[ell][2], xe[kSlots][ell][2];
    auto load_d = [&](int step) {
        const KeyBlock kd(a.bk + (size_t)step * 3 * ell * kPoly, 3 * ell, word);
#pragma unroll
        for (int d = 0; d < ell; ++d)
#pragma unroll
                for (int s = 0; s < 2; ++s) xd[d][s] = kd(d * kPoly + s * 256);
    };
    auto load_e = [&](d2 (&x)[ell][2], int j) {
#pragma unroll
        for (int d = 0; d < ell; ++d)
#pragma unroll
                for (int s = 0; s < 2; ++s) x[d][s] = ke((j * ell + d) * kPoly + s * 256);
    };
    if (a.st0 < a.st1) {
        load_d(a.st0);
        load_e(xe[0], 0);
    }
    for (int step = a.st0; step < a.st1; ++step) {
        const int party = step / a.n;
        const int next = min(step + 1, a.st1 - 1);
        auto rot = [&](int row, int j) { rotate<kGateT, true>(acc + j * kRowBytes, shift, a.offset, here(tid), y + row * kRowBytes); };
        Cx w[2] = {}, cA[2] = {}, cB[2] = {}, cT[2][2] = {};
        auto madd = [&](int i, const d2 (&x0)[2], Cx (&c0)[2], const d2 (&x1)[2], Cx (&c1)[2]) {
            Cx u, v;
            own.get(buf + i * kBufBytes, u, v);
            mac(c0[0], u, x0[0]);
            mac(c0[1], v, x0[1]);
            mac(c1[0], u, x1[0]);
            mac(c1[1], v, x1[1]);
        };
        // slots 0, 1 + party and the first of the slots 1 .. party, which get
        // no stage-2 part; then those by twos
        rot(0, 0);
        rot(1, 1 + party);
        if (party > 0) rot(2, 1);
        lds_sync();
        const int nf = (party > 0 ? 3 : 2) * ell;
        for (int t = pair; t < nf; t += kGateP)
            pair_fwd_a(FromY<false>{y + (t / ell) * kRowBytes}, 24 - 8 * (t % ell), l, at, buf + t * kBufBytes, tab);
        load_e(xe[1], 1 + party);
        lds_sync();
        for (int t = pair; t < nf; t += kGateP) pair_fwd_b(l, w2, at, buf + t * kBufBytes, tab);
        if (party > 0) load_e(xe[2], 1);
        lds_sync();
#pragma unroll
        for (int d = 0; d < ell; ++d)
            {
                madd(d, xe[0][d], w, xd[d], cA);
                madd(ell + d, xe[1][d], w, xd[d], cB);
                if (party > 0) madd(2 * ell + d, xe[2][d], w, xd[d], cT[0]);
            }
        int done = 1;                  // slots 1 .. done are transformed;
        int nT = party > 0 ? 1 : 0;    // the last nT of them wait for their inverse
        while (done < party) {
            const int cnt = min(2, party - done), j0 = done + 1;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (i < nT) {
                    own.put(buf + (kFwd + 2 * i + part) * kBufBytes, cT[i]);
                    cT[i][0] = cT[i][1] = {0.0, 0.0};
                }
            for (int i = 0; i < cnt; ++i) rot(i, j0 + i);
            lds_sync();
            const int mf = cnt * ell, mi = nT * kParts, jT = done + 1 - nT;
            for (int t = pair; t < mf + mi; t += kGateP) {
                if (t < mf) pair_fwd_a(FromY<false>{y + (t / ell) * kRowBytes}, 24 - 8 * (t % ell), l, at, buf + t * kBufBytes, tab);
                else pair_inv_a(l, w2, at, buf + (kFwd + t - mf) * kBufBytes, tab);
            }
            lds_sync();
            for (int t = pair; t < mf + mi; t += kGateP) {
                if (t < mf) pair_fwd_b(l, w2, at, buf + t * kBufBytes, tab);
                else pair_inv_b(buf + (kFwd + t - mf) * kBufBytes, Add{acc + (jT + (t - mf) / 2) * kRowBytes, false}, 16 * ((t - mf) & 1), l, at, tab);
            }
            d2 xo[2][ell][2];
            load_e(xo[0], j0);
            if (cnt > 1) load_e(xo[1], j0 + 1);
            lds_sync();
#pragma unroll
            for (int d = 0; d < ell; ++d)
                {
                    madd(d, xo[0][d], w, xd[d], cT[0]);
                    if (cnt > 1) madd(ell + d, xo[1][d], w, xd[d], cT[1]);
                }
            done += cnt;
            nT = cnt;
        }
        // w, and the last slots without a stage-2 part
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (i < nT) own.put(buf + (kFwd + 2 * i + part) * kBufBytes, cT[i]);
        const int bw = nT == 2 ? 2 * ell : kFwd + 2;   // free buffers
        own.put(buf + (bw + part) * kBufBytes, w);
        for (int i = tid; i < kN; i += kGateT) stw(y + 4u * i, a.offset);
        lds_sync();
        // transforms: w low, w high, then the slots'
        const int ni = 2 + nT * kParts;
        for (int t = pair; t < ni; t += kGateP) pair_inv_a(l, w2, at, buf + (t < 2 ? bw + t : kFwd + t - 2) * kBufBytes, tab);
        d2 x0[ell][2], x1[ell][2];
        const KeyBlock kf(a.bk + ((size_t)step * 3 + 1) * ell * kPoly, 2 * ell, word);
        auto load_f = [&](int part_of) {
#pragma unroll
            for (int d = 0; d < ell; ++d)
                if (d == part_of)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        x0[d][s] = kf(d * kPoly + s * 256);
                        x1[d][s] = kf((ell + d) * kPoly + s * 256);
                    }
        };
        load_f(0);
        lds_sync();
        for (int t = pair; t < ni; t += kGateP)
            pair_inv_b(buf + (t < 2 ? bw + t : kFwd + t - 2) * kBufBytes, Add{t < 2 ? y : acc + (done + 1 - nT + (t - 2) / 2) * kRowBytes, t < 2}, 16 * (t & 1), l, at, tab);
        load_f(1);
        lds_sync();
        if (pair < ell) pair_fwd_a(FromY<true>{y}, 24 - 8 * pair, l, at, buf + pair * kBufBytes, tab);
        load_f(2);
        lds_sync();
        if (pair < ell) pair_fwd_b(l, w2, at, buf + pair * kBufBytes, tab);
        lds_sync();
        const int next_shift = (int)abar[1 + next];
#pragma unroll
        for (int d = 0; d < ell; ++d)
            madd(d, x0[d], cA, x1[d], cB);
        own.put(buf + (kFwd + part) * kBufBytes, cA);
        own.put(buf + (kFwd + 2 + part) * kBufBytes, cB);
        lds_sync();
        pair_inv_a(l, w2, at, buf + (kFwd + pair) * kBufBytes, tab);
        load_d(next);
        lds_sync();
        pair_inv_b(buf + (kFwd + pair) * kBufBytes, Add{acc + (pair < 2 ? 0 : 1 + party) * kRowBytes, false}, 16 * (pair & 1), l, at, tab);
        load_e(xe[0], 0);
        shift = __builtin_amdgcn_readfirstlane(next_shift);
        lds_sync();
    }
    __syncthreads();
    for (int idx = tid; idx < K1 * kN; idx += kGateT) a.acc[(size_t)g * K1 * kN + idx] = ldw(acc + 4u * idx);
}

size_t fft_gate_lds(int k) {
    return (size_t)(k + 1 + kSlots) * kN * 4 + (size_t)(kGateBufs * kH + kTab2Words) * 16;
}

// A team of workgroups per gate, for batches that leave compute units idle.
// Members 0 and 1 own the slots with a stage-2 part (0 and 1 + party), helpers
// up to three of the slots 1 .. party each (members 0 and 1 what is left): a
// member rotates, transforms and multiplies its own slots, turns its own sum of
// products into its part of V (an integer, so the parts add exactly), and
// publishes it.  Members 0 and 1 add the parts up and run stage 2 of their
// slot.  Nothing else is exchanged, once per step; helpers need no V, so they
// run up to a step ahead.  A launch ends with a party, since slots then change
// hands.
//
// A published word is 64 bits, value and step number, written and read
// atomically at device scope: it is either not there yet or complete, and no
// other ordering is needed.  A box has two sides by the step's parity.  Members
// 0 and 1 publish step s only after reading step s - 1, so whoever has seen
// their step s may overwrite the side of step s - 1 (their own words for
// members 0 and 1, which read every step; `passed` for helpers).
//
// A team's blocks are nx apart, hence on one XCD and next to each other in its
// dispatch order, and the team size is chosen so that all are resident at once
// on an idle device.  On a busy one other streams' work can keep a member's
// compute unit for any time, so nobody waits for a workgroup that may not run:
// members count themselves in when they start (form_team), and one that has
// seen its team incomplete for kFormPolls marks the gate, at which those
// already there and those to come leave it to a launch of fft_gate_kernel that
// follows every team launch (its other blocks end at once).  A complete team
// holds its compute units until it ends, so its waits end too; they are bounded
// all the same (kSpinLimit: the status word is set, the member waits no more
// and goes on publishing).
//
// Bound by the latency of four transforms (2.2k cycles each), two rounds of
// products (1.2k) and the exchange (2.2-3k, of which a load is 1.1k).  Measured
// (ms, one workgroup per gate / here): one gate at 2, 4, 8 parties 8.8 / 7.3,
// 22.3 / 15.7, 64 / 30.7; 64 gates at 8 parties 64 / 35.4.
struct Team {
    int m, helpers, party;
    __device__ __forceinline__ int slots() const {
        const int q = min(party, kSlots * helpers);   // helpers' slots
        if (m >= 2) return (q - (m - 2) + helpers - 1) / helpers;
        return 1 + (party - q - m + 1) / 2;
    }
    __device__ __forceinline__ int slot(int i) const {
        if (m >= 2) return 1 + (m - 2) + i * helpers;
        return i == 0 ? m * (1 + party) : 1 + kSlots * helpers + m + 2 * (i - 1);
    }
    __device__ __forceinline__ bool owns(int j) const {
        for (int i = 0; i < slots(); ++i)
            if (slot(i) == j) return true;
        return m == 0 && j > 1 + party;   // rows still zero
    }
};

// What a team exchanges: a value and its tag in one 64-bit word, so that a word
// is either not there yet or complete.
struct Box {
    uint64_t *p;
    __device__ __forceinline__ static uint64_t get(uint64_t *q) {
        // read where atomics are done: 64 gates at 8 parties 37.7 -> 36.7 ms
        // against a device-scope load
        return __hip_atomic_fetch_or(q, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ static void put(uint64_t *q, uint32_t v, uint32_t tag) {
        __hip_atomic_store(q, (uint64_t)tag << 32 | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ u4 load(uint32_t off) const {
        const uint64_t v = get(p + off / 8), u = get(p + off / 8 + 1);
        return u4{(uint32_t)v, (uint32_t)(v >> 32), (uint32_t)u, (uint32_t)(u >> 32)};
    }
    __device__ __forceinline__ void store(uint32_t off, u4 v) const {
        put(p + off / 8, v.x, v.y);
        put(p + off / 8 + 1, v.z, v.w);
    }
};
constexpr int kMaxMembers = 5;
constexpr uint32_t kBoxBytes = kN * 8;   // (value, tag) words of one member and parity

constexpr uint32_t kSpinLimit = 1u << 23;   // polls of about a microsecond
// Polls before a member gives its team up: about 0.2 ms, many times what an idle
// device takes to start a launch's workgroups, little beside a party's steps.
constexpr int kFormPolls = 256;

// One thread of each member: whether all `members` run.  The gate's word counts
// them; kApart is set only while some are missing, so all see the same answer.
__device__ __forceinline__ bool form_team(uint32_t *word, uint32_t members, int polls) {
    uint32_t v = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    for (int i = 0; v < members; ++i) {
        if (i < polls) {
            __builtin_amdgcn_s_sleep(1);
            v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (__hip_atomic_compare_exchange_strong(word, &v, v | kApart, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT)) {
            return false;
        }   // else v is the word's new value: one more member or kApart
    }
    return v == members;
}

template <int ELL>
__global__ __launch_bounds__(kGateT, 2) void fft_team_kernel(FftArgs a) {
    constexpr int ell = ELL;
    const int K1 = a.k + 1, tid = threadIdx.x;
    // LDS as in fft_gate_kernel
    const uint32_t acc = 0, y = K1 * kRowBytes, buf = y + kSlots * kRowBytes;
    d2 *tab = reinterpret_cast<d2 *>(smem + buf + kGateBufs * kBufBytes);
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid & 63;
    const int part = __builtin_amdgcn_readfirstlane(tid / 256);
    // blocks go round the XCDs: a team's members share an L2
    const int x = blockIdx.x % a.nx, b = blockIdx.x / a.nx;
    const int g = x + a.nx * (b / a.members);
    const int party = a.st0 / a.n;
    const Team team{b % a.members, a.members - 2, party};
    if (g >= a.G) return;
    const int ns = team.slots();
    if (ns <= 0) return;
    const int helpers = min(party, a.members - 2);   // that own a slot
    const int members = 2 + helpers;
    const bool helper = team.m >= 2;
    const uint32_t *abar = a.abar + (size_t)g * (a.k * a.n + 1);
    const int pair = wave >> 1, w2 = wave & 1;
    const Owner own(tid & 255, owner_word2(tid & 255), 128, a.tab);
    const Lane2 at(l, w2);
    const int word = part * kH + (tid & 255);
    if (tid < kTab2Words) tab[tid] = a.tab[kTab2 + tid];
    load_acc<kGateT>(a, g, abar, acc);
    __syncthreads();
    if (tid == 0) stw(y, form_team(a.form + g, (uint32_t)members, a.form_polls));
    __syncthreads();
    const bool formed = ldw(y) != 0;
    __syncthreads();
    if (!formed) return;
    const KeyBlock ke(a.evk, K1 * ell, word);
    d2 xd[ell][2], xe[kSlots][ell][2], xf[ell][2];
    auto load = [&](d2 (&v)[ell][2], const KeyBlock &k, int poly) {
#pragma unroll
        for (int d = 0; d < ell; ++d)
#pragma unroll
            for (int s = 0; s < 2; ++s) v[d][s] = k((poly + d) * kPoly + s * 256);
    };
    auto keys = [&](int step) { return KeyBlock(a.bk + (size_t)step * 3 * ell * kPoly, 3 * ell, word); };
    load(xd, keys(a.st0), 0);
    load(xe[0], ke, team.slot(0) * ell);
    Shifts shifts{abar + 1, a.st1, l, 0};
    bool dead = false;   // a member gave up waiting: the status word says so
    auto give_up = [&]() {
        dead = true;
        __hip_atomic_fetch_or(a.status, kStatusTimeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const Box box{a.xch + (size_t)g * a.members * 2 * kN};
    auto at_box = [&](int member, uint32_t tag) { return (uint32_t)(2 * member + (int)(tag & 1)) * kBoxBytes; };
    auto passed = [&](uint32_t tag) {   // members 0 and 1 have published `tag`
        for (uint32_t spin = 0; !dead; ++spin) {
            const uint64_t v = __hip_atomic_load(box.p + at_box(0, tag) / 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t u = __hip_atomic_load(box.p + at_box(1, tag) / 8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t)(v >> 32) == tag && (uint32_t)(u >> 32) == tag) break;
            if (spin == kSpinLimit) give_up();
            __builtin_amdgcn_s_sleep(1);
        }
    };
    for (int step = a.st0; step < a.st1; ++step) {
        const int shift = shifts(step, a.st0);
        const uint32_t tag = (uint32_t)step + 1;
#pragma unroll
        for (int i = 0; i < kSlots; ++i)
            if (i < ns) rotate<kGateT, true>(acc + team.slot(i) * kRowBytes, shift, a.offset, here(tid), y + i * kRowBytes);
        lds_sync();
        Cx w[2] = {}, c[kSlots][2] = {};
        auto madd = [&](int i, const d2 (&x0)[2], Cx (&c0)[2], const d2 (&x1)[2], Cx (&c1)[2]) {
            Cx u, v;
            own.get(buf + i * kBufBytes, u, v);
            mac(c0[0], u, x0[0]);
            mac(c0[1], v, x0[1]);
            mac(c1[0], u, x1[0]);
            mac(c1[1], v, x1[1]);
        };
        for (int t = pair; t < ns * ell; t += kGateP)
            pair_fwd_a(FromY<false>{y + (t / ell) * kRowBytes}, 24 - 8 * (t % ell), l, at, buf + t * kBufBytes, tab);
        lds_sync();
        for (int t = pair; t < ns * ell; t += kGateP) pair_fwd_b(l, w2, at, buf + t * kBufBytes, tab);
        if (ns > 1) load(xe[1], ke, team.slot(1) * ell);
        if (ns > 2) load(xe[2], ke, team.slot(2) * ell);
        lds_sync();
#pragma unroll
        for (int i = 0; i < kSlots; ++i)
            if (i < ns)
#pragma unroll
                for (int d = 0; d < ell; ++d) madd(i * ell + d, xe[i][d], w, xd[d], c[i]);
        // w, and the slots without a stage-2 part
        const int first = helper ? 0 : 1;
        const int bt = ns < kSlots ? ns * ell : 0;
        if (ns == kSlots) lds_sync();   // their transforms take the digits' place
        own.put(buf + (kGateBufs - 2 + part) * kBufBytes, w);
#pragma unroll
        for (int i = 0; i < kSlots; ++i)
            if (i >= first && i < ns) own.put(buf + (bt + 2 * (i - first) + part) * kBufBytes, c[i]);
        lds_sync();
        // tasks: w low, w high, then the slots'
        const int ni = 2 + 2 * (ns - first);
        auto at_inv = [&](int t) { return buf + (t < 2 ? kGateBufs - 2 + t : bt + t - 2) * kBufBytes; };
        for (int t = pair; t < ni; t += kGateP) pair_inv_a(l, w2, at, at_inv(t), tab);
        if (!helper) load(xf, keys(step), (1 + team.m) * ell);
        lds_sync();
        for (int t = pair; t < ni; t += kGateP) {
            if (t < 2) pair_inv_b(at_inv(t), SetY{y + t * kRowBytes}, 16 * t, l, at, tab);
            else pair_inv_b(at_inv(t), Add{acc + team.slot(first + t / 2 - 1) * kRowBytes, false}, 16 * (t & 1), l, at, tab);
        }
        lds_sync();
        // this member's part of V
        const uint32_t mine = y + 8u * tid;
        uint32_t v0 = ldw(mine) + ldw(mine + kRowBytes), v1 = ldw(mine + 4u) + ldw(mine + kRowBytes + 4u);
        if (helper && step > a.st0) passed(tag - 1);   // the box is free once its readers are a step on
        box.store(at_box(team.m, tag) + 16u * tid, u4{v0, tag, v1, tag});
        if (helper) {
            load(xd, keys(min(step + 1, a.st1 - 1)), 0);
            lds_sync();
            continue;
        }
        {
            u4 in[kMaxMembers - 1];
            for (uint32_t spin = 0; !dead; ++spin) {
                bool all = true;
#pragma unroll
                for (int o = 0; o < kMaxMembers - 1; ++o)
                    if (o < members - 1) in[o] = box.load(at_box(o == 0 ? 1 - team.m : 1 + o, tag) + 16u * tid);
#pragma unroll
                for (int o = 0; o < kMaxMembers - 1; ++o)
                    if (o < members - 1) all &= in[o].y == tag && in[o].w == tag;
                if (all) break;
                if (spin == kSpinLimit) give_up();
            }
#pragma unroll
            for (int o = 0; o < kMaxMembers - 1; ++o)
                if (o < members - 1) {
                    v0 += in[o].x;
                    v1 += in[o].z;
                }
        }
        stw(mine, v0 + a.offset);
        stw(mine + 4u, v1 + a.offset);
        lds_sync();
        if (pair < ell) pair_fwd_a(FromY<true>{y}, 24 - 8 * pair, l, at, buf + pair * kBufBytes, tab);
        lds_sync();
        if (pair < ell) pair_fwd_b(l, w2, at, buf + pair * kBufBytes, tab);
        lds_sync();
#pragma unroll
        for (int d = 0; d < ell; ++d) {
            Cx u, v;
            own.get(buf + d * kBufBytes, u, v);
            mac(c[0][0], u, xf[d][0]);
            mac(c[0][1], v, xf[d][1]);
        }
        own.put(buf + (kFwd + part) * kBufBytes, c[0]);
        lds_sync();
        if (pair < 2) pair_inv_a(l, w2, at, buf + (kFwd + pair) * kBufBytes, tab);
        load(xd, keys(min(step + 1, a.st1 - 1)), 0);
        lds_sync();
        if (pair < 2)
            pair_inv_b(buf + (kFwd + pair) * kBufBytes, Add{acc + team.slot(0) * kRowBytes, false}, 16 * pair, l, at, tab);
        lds_sync();
    }
    __syncthreads();
    for (int j = 0; j < K1; ++j)
        if (team.owns(j))
            for (int i = tid; i < kN; i += kGateT) a.acc[((size_t)g * K1 + j) * kN + i] = ldw(acc + j * kRowBytes + 4u * i);
}

__global__ void fft_clear_kernel(uint64_t *p, size_t words) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < words) p[i] = 0;
}

}  // namespace

static bool fft_supported(const mk_params &P) { return P.N == kN && P.bk_ell <= kEll; }

// Automatic schedule, unless the caller forces something that only the int8
// kernels have (GEMM tile shapes, team sizes): at N = 1024 the transforms are
// faster at every batch size and party count (ms, int8 kernels / here: one
// gate 34 / 7.3, 256 gates 45 / 8.9, 1024 gates 86 / 31.4 at 2 parties; 1024
// gates 199 / 89 at 4 parties; 64 gates 180 / 35 at 8 parties).
bool use_fft(const mk_ctx *ctx) {
    const DeviceKeys &D = ctx->dev;
    return D.fft_bk && D.rot_kind == MK_ROT_AUTO && !D.team_rows && D.force_tiles[0] < 0 && D.force_tiles[1] < 0;
}

// Transforms the uploaded keys (extended form [-K | K]) and builds the twiddle
// table; nothing for parameter sets this schedule does not run, nor where the
// device has no room for them (the int8 kernels then run, as with neither).
int fft_upload(mk_ctx *ctx, hipStream_t s) {
    const mk_params &P = ctx->p;
    DeviceKeys &D = ctx->dev;
    if (!fft_supported(P)) return MK_OK;
    const size_t bk_polys = (size_t)P.k * P.n * 3 * P.bk_ell, evk_polys = (size_t)(P.k + 1) * P.bk_ell;
    std::vector<d2> tab(kTabWords);
    void **bufs[3] = {&D.fft_evk, &D.fft_tab, &D.fft_bk};
    const size_t bytes[3] = {evk_polys * kPoly * sizeof(d2), tab.size() * sizeof(d2), bk_polys * kPoly * sizeof(d2)};
    for (int i = 0; i < 3; ++i)
        if (hipMalloc(bufs[i], bytes[i]) != hipSuccess) {
            (void)hipGetLastError();   // or the next launch would report it
            *bufs[i] = nullptr;
            for (int j = 0; j < i; ++j) {
                (void)hipFree(*bufs[j]);
                *bufs[j] = nullptr;
            }
            return MK_OK;
        }
    // angle of block `b` at level lv (1 .. 9): X^m = e^(i theta) splits at
    // X^(m/2) = +- e^(i theta/2)
    auto entry = [](int lv, int b) {
        long double f = 0.25L;
        for (int i = lv - 2; i >= 0; --i) f = f / 2 + (((b >> i) & 1) ? 0.5L : 0.0L);
        f *= 3.141592653589793238462643383279502884L;
        return d2{(double)cosl(f), (double)tanl(f)};
    };
    for (int q = 0; q < 4; ++q)   // q = (j8 j7)
        for (int i = 0; i < 2; ++i) {
            tab[kTabP + 4 * q + i] = entry(4, 4 * (q >> 1) + 2 * i);
            tab[kTabP + 4 * q + 2 + i] = entry(5, 4 * q + 2 * i);
        }
    for (int l = 0; l < 64; ++l) {
        const int b5 = ((l >> 3) & 1) * 16 + ((l >> 2) & 1) * 8 + ((l >> 1) & 1) * 4 + ((l >> 4) & 1) * 2 + (l >> 5);
        tab[kTabQ + l] = entry(6, b5);
        tab[kTabQ + 64 + l] = entry(7, 2 * b5);
        tab[kTabQ + 128 + l] = entry(8, 4 * b5);
        tab[kTabQ + 192 + l] = entry(8, 4 * b5 + 2);
    }
    for (int c = 0; c < 256; ++c) tab[kTab9 + c] = entry(9, c);
    for (int q = 0; q < 4; ++q) {   // q = (j8 j7)
        tab[kTab2 + 2 * q] = entry(3, 2 * (q >> 1));
        tab[kTab2 + 2 * q + 1] = entry(4, 2 * q);
    }
    for (int w = 0; w < 2; ++w)
        for (int l = 0; l < 64; ++l) {   // lane (j4 j3 j5 j6 j7 j0), wave j8
            const int b4 = w * 8 + ((l >> 1) & 1) * 4 + ((l >> 2) & 1) * 2 + ((l >> 3) & 1);
            const int q = w * 8 + ((l >> 1) & 7);
            tab[kTab2 + kTab2Q + q] = entry(5, b4);
            tab[kTab2 + kTab2Q + 16 + q] = entry(6, 2 * b4);
            tab[kTab2 + kTab2R + w * 64 + l] = entry(7, 4 * b4 + 2 * (l >> 5));
            tab[kTab2 + kTab2R + 128 + w * 64 + l] = entry(8, 8 * b4 + 4 * (l >> 5) + 2 * ((l >> 4) & 1));
        }
    MK_HIP(hipMemcpyAsync(D.fft_tab, tab.data(), tab.size() * sizeof(d2), hipMemcpyHostToDevice, s), "transform tables");
    hipLaunchKernelGGL(fft_key_kernel, dim3((unsigned)bk_polys), dim3(256), kParts * kBufBytes, s, D.bk_ext, (const d2 *)D.fft_tab,
                       (d2 *)D.fft_bk);
    MK_HIP(hipGetLastError(), "bootstrapping key transform launch");
    hipLaunchKernelGGL(fft_key_kernel, dim3((unsigned)evk_polys), dim3(256), kParts * kBufBytes, s, D.evk_ext, (const d2 *)D.fft_tab,
                       (d2 *)D.fft_evk);
    MK_HIP(hipGetLastError(), "evaluation key transform launch");
    MK_HIP(hipStreamSynchronize(s), "key transform sync");
    return MK_OK;
}

template <class Kernel>
static int launch_kernel(Kernel kern, int blocks, int threads, size_t lds, const FftArgs &a, hipStream_t s) {
    MK_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
           "transform rotation LDS attribute");
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), lds, s, a);
    MK_HIP(hipGetLastError(), "transform rotation launch");
    return MK_OK;
}
template <int ELL>
static int launch_ell(const FftArgs &a, bool lean, hipStream_t s) {
    if (a.members) {
        const int blocks = a.nx * a.members * ((a.G + a.nx - 1) / a.nx);
        if (int rc = launch_kernel(fft_team_kernel<ELL>, blocks, kGateT, fft_gate_lds(a.k), a, s)) return rc;
        return launch_kernel(fft_gate_kernel<ELL, true>, a.G, kGateT, fft_gate_lds(a.k), a, s);
    }
    if (lean) return launch_kernel(fft_lean_kernel<ELL>, a.G, kLeanT, fft_lean_lds(a.k), a, s);
    return launch_kernel(fft_gate_kernel<ELL, false>, a.G, kGateT, fft_gate_lds(a.k), a, s);
}

static size_t box_words(size_t count, int members) { return count * members * 2 * kN; }
// 64-bit words of a team launch's scratch: boxes, then a 32-bit word per gate.
static size_t team_words(size_t count, int members) { return box_words(count, members) + (count + 1) / 2; }

static int useful_members(const mk_params &P) { return std::min(2 + (P.k - 1 + kSlots - 1) / kSlots, kMaxMembers); }

// Bytes that the teams of a rotation of up to `count` gates need: they are no
// more workgroups than compute units.
size_t fft_team_scratch(const mk_ctx *ctx, size_t count) {
    const DeviceKeys &D = ctx->dev;
    if (!D.fft_bk || D.num_xcd <= 0) return 0;
    const size_t cus = (size_t)std::max(1, D.num_cus);
    return box_words(1, 1) * 8 * std::min(count * useful_members(ctx->p), cus) + (std::min(count, cus) + 1) / 2 * 8;
}

// Workgroups per gate (0: one, fft_gate_kernel or fft_lean_kernel): as many as
// have work and as an XCD's compute units hold for its share of the gates (a
// workgroup takes a compute unit's LDS).  Measured (MI355X, ms, one workgroup /
// team): 70 gates at 2 parties 8.8 / 7.5; 64 at 4 22.3 / 15.9; 80 at 8 (teams
// of 3) 64 / 38.
static int team_members(const mk_ctx *ctx, size_t count) {
    const mk_params &P = ctx->p;
    const DeviceKeys &D = ctx->dev;
    if (!count || D.num_xcd <= 0 || D.num_cus < D.num_xcd) return 0;
    const size_t rows = (count + D.num_xcd - 1) / D.num_xcd, fit = (size_t)(D.num_cus / D.num_xcd) / rows;
    const int m = (int)std::min<size_t>(fit, useful_members(P));
    return m >= 2 ? m : 0;
}

// Whether a team of `members` runs a party's steps.  Helpers take three slots
// each, members 0 and 1 at most two more; without helpers a team gains only
// while there is nothing for them (128 gates at 2 parties, two members for both
// 8.7 ms, for the first alone 8.4, one workgroup 8.7).
static bool team_runs(int members, int party) {
    return party <= kSlots * (members - 2) + (members > 2 ? 2 * (kSlots - 1) : 0);
}

// Gates first .. first + count - 1 of a batch on one kernel (a team's parties on
// fft_team_kernel, the others on fft_gate_kernel).
static int launch_part(mk_ctx *ctx, FftArgs a, size_t first, size_t count, bool lean, int members, int steps, hipStream_t s) {
    if (!count) return MK_OK;
    const int n = a.n;
    a.G = (int)count;
    a.abar += first * ((size_t)a.k * n + 1);
    a.acc += first * (size_t)(a.k + 1) * kN;
    a.members = 0;
    if (members) {
        const size_t words = team_words(count, members);
        int rc = MK_OK;
        a.xch = (uint64_t *)team_scratch_for(ctx, count, s, &rc);
        if (rc) return rc;
        if (a.xch) {
            hipLaunchKernelGGL(fft_clear_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, a.xch, words);
            MK_HIP(hipGetLastError(), "transform team clear");
            a.members = members;
            a.form = (uint32_t *)(a.xch + box_words(count, members));
            a.form_polls = ctx->dev.team_wait < 0 ? kFormPolls : ctx->dev.team_wait;
        }
    }
    // During a capture a launch ends where the stream-ordered steps (four kernels
    // each, to which the few that really run are not added) would end a graph
    // piece, so pieces stay as long as documented.  The count stays a multiple of
    // four, so rounding the steps up takes no piece past the largest size, and
    // keep_room leaves it the kernels that end the level.
    for (int st = 0; st < steps || st == 0; st = std::max(a.st1, 1)) {
        const int room = capture_room(ctx);
        a.st0 = st;
        a.st1 = room == INT_MAX ? steps : std::min(steps, st + (room + 3) / 4);
        if (a.members && !team_runs(a.members, st / n)) a.members = 0;
        if (a.members) a.st1 = std::min(a.st1, (st / n + 1) * n);   // a team's slots change with the party
        int rc = a.ell == 3 ? launch_ell<3>(a, lean, s) : a.ell == 2 ? launch_ell<2>(a, lean, s) : launch_ell<1>(a, lean, s);
        if (!rc) rc = capture_checkpoint(ctx, s, 4 * (a.st1 - a.st0), true);
        if (rc) return rc;
    }
    return MK_OK;
}

int launch_br_fft(mk_ctx *ctx, const uint32_t *abar, uint32_t *acc, size_t count, int steps, hipStream_t s) {
    const mk_params &P = ctx->p;
    DeviceKeys &D = ctx->dev;
    FftArgs a = {};
    a.k = P.k; a.n = P.n; a.ell = P.bk_ell;
    a.offset = decomp_offset(P.bk_ell);
    a.abar = abar; a.acc = acc;
    a.bk = (const d2 *)D.fft_bk; a.evk = (const d2 *)D.fft_evk; a.tab = (const d2 *)D.fft_tab;
    a.nx = D.num_xcd; a.status = D.status;
    StageTimer t1(ctx, 1, s);
    StageTimer t4(ctx, 4, s);
    // Which kernel: see team_members for several compute units per gate; one
    // gate per compute unit at a time, or several.  Measured on MI355X (256
    // compute units), fft_gate_kernel / fft_lean_kernel, ms: 2 parties 256 gates
    // 8.9 / 16.9, 512 gates 17.4 / 21.2, 1024 gates 34.9 / 31.4; 4 parties 256
    // gates 22.3 / 41, 512 gates 44.9 / 50, 768 gates 67 / 63; 8 parties (two
    // lean workgroups fit a compute unit) 256 gates 64 / 116, 512 gates 128 / 143.
    // What full rounds leave over runs as a batch of that size would, instead of
    // one more round on a few compute units.  Measured, one launch / parts: 300
    // gates at 2 parties 18.0 / 16.5, at 4 44.7 / 38.4, at 8 128 / 97.  After the
    // lean kernel's rounds up to one gate per compute unit does from 3 parties on
    // (1024 gates at 3 parties 56.9 / 56.1, 800 at 4 89 / 80, 1024 89 / 85); at 2,
    // where its workgroups drift apart more, it does not (1100 gates 40.3 / 41.3).
    // At 3 parties the lean kernel wins from 600 gates on (44.4 / 41.3; 513 gates
    // 41.5 / 42.4); at 6 and 7 it loses at 513, 768 and 1024 gates (1024: 162 /
    // 168, 207 / 214).  At 5 it would gain from 600 gates on (92.6 / 85.3, 1024
    // 123 / 116 with parts) and lose at 513 (81 / 86); it is not used there.
    const size_t cus = (size_t)std::max(1, D.num_cus);
    size_t lean = P.k <= 4 && count > 2 * cus ? count : 0;
    const size_t round = cus * std::min<size_t>(4, kLdsBytes / fft_lean_lds(P.k));
    if (P.k > 2 && lean > round && lean % round <= cus) lean -= lean % round;
    const size_t rest = count - lean;
    const int members = rest ? team_members(ctx, rest % cus) : 0;
    const size_t team = members ? rest % cus : 0;
    int rc = launch_part(ctx, a, 0, lean, true, 0, steps, s);
    if (!rc) rc = launch_part(ctx, a, lean, rest - team, false, 0, steps, s);
    if (!rc) rc = launch_part(ctx, a, count - team, team, false, members, steps, s);
    return rc;
}

}  // namespace mk

using namespace mk;

extern "C" {

int mk_set_team_wait(mk_ctx *ctx, int polls) {
    if (!ctx || polls < -1) return fail(MK_EINVAL, "mk_set_team_wait: bad argument");
    ctx->dev.team_wait = polls;
    return MK_OK;
}

}  // extern "C"
