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
// (8 L + 8) ell N^2 int8 operations, and each gate's accumulator stays in one
// workgroup's LDS, so no workgroup ever waits for another.
//
// Exactness.  A key coefficient is split K = 2^16 K_hi + K_lo with signed
// 16-bit halves; every accumulated product sum is then an integer below
// 2^37 in magnitude, and the double result is within 0.02 of it for every
// input, so rounding to the nearest integer recovers it.  With u = 2^-53: a
// butterfly's output carries a relative error (2-norm of the pair) of at
// most 4u (table entries u each, one rounding per fused multiply-add), nine
// levels 37u; the sum of P products of transforms 2 sqrt(2) P u.  With M = sum
// over the P products of |u|_2 |K|_2 <= P (2^7 sqrt(N)) (2^15 sqrt(N)) = P 2^32,
// forward errors of digits and keys reach a result coefficient through
// Cauchy-Schwarz as 37u M each, the products' as 2 sqrt(2) P u M, and the
// inverse's 37u times the 2-norm of the result, at most sqrt(N) M.  For the
// largest P, (k + 1) ell = 27 at 8 parties: 27 2^-21 (74 + 76 + 32 * 37) =
// 0.018.  Unsplit keys would be bounded by 2^16 times as much, so the split
// (twice the inverse transforms and products) is what makes the rounding
// exact for every key and ciphertext and not only for likely ones.  The
// rounding adds 1.5 2^52: the sum's low word is the integer mod 2^32.
//
// Butterflies are six fused multiply-adds (b (1 + i t) scaled by c, twiddle
// c (1 + i t)).  A wave runs levels 1-8 of one transform with 8 points per
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
constexpr int kTabP = 0, kTabQ = 16, kTab9 = kTabQ + 256, kTabWords = kTab9 + 256;

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

// LAST: the two outermost levels leave their cosines out (the caller scales)
template <bool LAST, class TW>
__device__ __forceinline__ void radix8_inv(Cx (&x)[8], TW tw) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const Tw w = tw(2 + h);
        bf_inv<false, true>(x[4 * h], x[4 * h + 1], w.c, w.t);
        bf_inv<true, true>(x[4 * h + 2], x[4 * h + 3], w.c, w.t);
    }
    {
        const Tw w = tw(1);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            bf_inv<false, !LAST>(x[r], x[r + 2], w.c, w.t);
            bf_inv<true, !LAST>(x[r + 4], x[r + 6], w.c, w.t);
        }
    }
    {
        const Tw w = tw(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) bf_inv<false, !LAST>(x[r], x[r + 4], w.c, w.t);
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

// Levels 8 .. 1 of an inverse transform by one wave, from hand-over order;
// every coefficient, rounded and shifted left by `sh`, is added to dst.
__device__ __forceinline__ void wave_inv(uint32_t buf, uint32_t dst, int sh, int lane, const Lane &lane_at, const d2 *tab) {
    const int l = here(lane);
    const Lane at = lane_at.here();
    const uint32_t dl = dst + 4u * (uint32_t)l;
    d2 tp[4], tq[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) tq[i] = tab[kTabQ + 64 * i + l];
    Cx x[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = ld(at.hand(buf, r));
#pragma unroll
    for (int i = 0; i < 4; ++i) tp[i] = tab[kTabP + (l >> 4) * 4 + i];
    radix8_inv<false>(x, [&](int i) { return Tw{tq[i].x, tq[i].y}; });
    wave_fence();
#pragma unroll
    for (int r = 0; r < 8; ++r) st(at.inner(buf, r), x[r]);
    wave_fence();
#pragma unroll
    for (int r = 0; r < 8; ++r) x[r] = ld(at.outer(buf, r));
#pragma unroll
    for (int j6 = 0; j6 < 2; ++j6) {   // level 5
        bf_inv<false, true>(x[j6], x[j6 + 2], tp[2 + j6].x, tp[2 + j6].y);
        bf_inv<true, true>(x[j6 + 4], x[j6 + 6], tp[2 + j6].x, tp[2 + j6].y);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        swap_bit<16>(x[r], x[r + 2]);
        swap_bit<16>(x[r + 4], x[r + 6]);
    }
#pragma unroll
    for (int j7 = 0; j7 < 2; ++j7) {   // level 4
        bf_inv<false, true>(x[2 * j7], x[2 * j7 + 4], tp[j7].x, tp[j7].y);
        bf_inv<true, true>(x[2 * j7 + 1], x[2 * j7 + 5], tp[j7].x, tp[j7].y);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) swap_bit<32>(x[r], x[r + 4]);
    radix8_inv<true>(x, [](int i) { return kTwA[i]; });
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const double s = (1.0 / kH) * ((r & 2) ? kTwA[1].c : 1.0) * ((r & 4) ? kTwA[0].c : 1.0);
        addw(dl + 256u * r, round_word(x[r].r, s) << sh);
        addw(dl + 256u * r + kRowBytes / 2, round_word(x[r].i, s) << sh);
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
};

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
template <int T>
__device__ __forceinline__ void rotate(uint32_t c, int shift, uint32_t offset, int tid, uint32_t y) {
#pragma unroll
    for (int i = 0; i < kN / T; ++i) {
        const int m = tid + T * i, s = m + shift;
        const uint32_t src = ldw(c + 4u * (uint32_t)(s & (kN - 1))), rot = (s & kN) ? 0u - src : src;
        stw(y + 4u * m, (rot - ldw(c + 4u * m) + offset) ^ 0x80808080u);
    }
}

// The thread's two frequencies of the transform in `buf`, and back.
struct Owner {
    uint32_t at0, at1;
    double c, t;
    __device__ __forceinline__ Owner(int c_, const d2 *tab)
        : at0(16u * owner_word(c_)), at1(4096u + (16u * owner_word(c_) ^ 16u)) {
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
    const Owner own(tid, tab);
    const Lane at(l);
    load_acc<kLeanT>(a, g, abar, acc);
    int shift = a.st0 < a.st1 ? (int)abar[1 + a.st0] : 0;
    int turn = (int)(blockIdx.x >> 3) + (int)(blockIdx.x >> 8);
    __syncthreads();
    for (int step = a.st0; step < a.st1; ++step) {
        const int party = step / a.n, bit = step - party * a.n;
        const int next_shift = step + 1 < a.st1 ? (int)abar[2 + step] : 0;
        const KeyBlock kd(a.bk + ((size_t)party * a.n + bit) * 3 * ell * kPoly, 3 * ell, tid), ke(a.evk, K1 * ell, tid);
        auto rot = [&](int j) { rotate<kLeanT>(acc + j * kRowBytes, shift, a.offset, here(tid), y); };
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
        // this wave's task of a round of `tasks`: rounds follow each other around
        // the waves
        auto next = [&](int tasks) {
            const int v = (wave - turn) & 3;
            turn += tasks;
            return v;
        };
        auto forward = [&](auto flip) {
            const int v = next(ell);
            if (v < ell) wave_fwd<decltype(flip)::value>(y, 24 - 8 * v, l, at, buf + v * kBufBytes, tab);
        };
        auto inverse = [&](int tasks, uint32_t dst) {   // low and high part
            const int v = next(tasks);
            if (v < tasks) wave_inv(buf + v * kBufBytes, dst, 16 * v, l, at, tab);
        };
        Cx w[kParts][2] = {};
        rot(party > 0 ? 1 : 0);
        for (int j = 1; j <= party; ++j) {   // slots without a stage-2 part
            lds_sync();
            forward(std::false_type{});
            Cx cT[kParts][2] = {};
            madd(ke, j * ell, w, kd, 0, cT);
            lds_sync();
            own.put(buf, cT[0]);
            own.put(buf + kBufBytes, cT[1]);
            rot(j < party ? j + 1 : 0);
            lds_sync();
            inverse(2, acc + j * kRowBytes);
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
        own.put(buf, w[0]);
        own.put(buf + kBufBytes, w[1]);
        lds_sync();
        inverse(2, y);
        lds_sync();
        forward(std::true_type{});
        madd(kd, ell, cA, kd, 2 * ell, cB);
        lds_sync();
        own.put(buf, cA[0]);
        own.put(buf + kBufBytes, cA[1]);
        own.put(buf + 2 * kBufBytes, cB[0]);
        lds_sync();
        {
            const int v = next(3);
            if (v < 3) wave_inv(buf + v * kBufBytes, acc + (v < 2 ? 0 : 1 + party) * kRowBytes, v == 1 ? 16 : 0, l, at, tab);
        }
        lds_sync();
        own.put(buf, cB[1]);
        lds_sync();
        if (next(1) == 0) wave_inv(buf, acc + (1 + party) * kRowBytes, 16, l, at, tab);
        shift = next_shift;
        lds_sync();
    }
    __syncthreads();
    for (int idx = tid; idx < K1 * kN; idx += kLeanT) a.acc[(size_t)g * K1 * kN + idx] = ldw(acc + 4u * idx);
}

size_t fft_lean_lds(int k) { return (size_t)(k + 2) * kN * 4 + (size_t)kLeanBufs * kH * 16; }

// One gate per compute unit.
constexpr int kGateT = 512;           // threads: part tid / 256 of word tid % 256
constexpr int kGateW = kGateT / 64;   // waves
constexpr int kSlots = 3;             // slots whose digits are transformed together
constexpr int kFwd = kSlots * kEll;   // buffers of digit transforms
constexpr int kGateBufs = kFwd + 4;   // and of inverse transforms

template <int ELL, bool MANY>
__global__ __launch_bounds__(kGateT, 2) void fft_gate_kernel(FftArgs a) {
    constexpr int ell = ELL;
    const int K1 = a.k + 1, tid = threadIdx.x;
    // LDS: accumulators [K1][N], y [kSlots][N], transforms [kGateBufs][H],
    // twiddles [kTab9]
    const uint32_t acc = 0, y = K1 * kRowBytes, buf = y + kSlots * kRowBytes;
    d2 *tab = reinterpret_cast<d2 *>(smem + buf + kGateBufs * kBufBytes);
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid & 63;
    const int part = __builtin_amdgcn_readfirstlane(tid / 256);
    const int g = blockIdx.x;
    const uint32_t *abar = a.abar + (size_t)g * (a.k * a.n + 1);
    const Owner own(tid & 255, a.tab);
    const Lane at(l);
    const int word = part * kH + (tid & 255);
    if (tid < kTab9) tab[tid] = a.tab[tid];
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
    auto load_step = [&](int step) {
        const int party = step / a.n;
        load_d(step);
        load_e(xe[0], 0);
        load_e(xe[1], 1 + party);
    };
    if (a.st0 < a.st1) load_step(a.st0);
    for (int step = a.st0; step < a.st1; ++step) {
        const int party = step / a.n;
        const int next_shift = step + 1 < a.st1 ? (int)abar[2 + step] : 0;
        auto rot = [&](int row, int j) { rotate<kGateT>(acc + j * kRowBytes, shift, a.offset, here(tid), y + row * kRowBytes); };
        Cx w[2] = {}, cA[2] = {}, cB[2] = {}, cT[2][2] = {};
        auto madd = [&](int i, const d2 (&x0)[2], Cx (&c0)[2], const d2 (&x1)[2], Cx (&c1)[2]) {
            Cx u, v;
            own.get(buf + i * kBufBytes, u, v);
            mac(c0[0], u, x0[0]);
            mac(c0[1], v, x0[1]);
            mac(c1[0], u, x1[0]);
            mac(c1[1], v, x1[1]);
        };
        // touch the next step's keys, so that they are in this XCD's L2 by
        // then (the keys of 4 parties and more exceed every cache)
        uint32_t touched[3];
        {
            const uint32_t bytes = 3u * ell * kPoly * 16u;
            const int nxt = min(step + 1, a.st1 - 1);
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(a.bk + (size_t)nxt * 3 * ell * kPoly), (short)0, (int)bytes, 0x00020000);
#pragma unroll
            for (int i = 0; i < 3; ++i)
                touched[i] = __builtin_amdgcn_raw_buffer_load_b32(r, 128u * (tid + kGateT * i), 0, 0);
        }
        // slots 0, 1 + party and the first of the slots 1 .. party, which get
        // no stage-2 part; then those by twos
        rot(0, 0);
        rot(1, 1 + party);
        if (party > 0) rot(2, 1);
        lds_sync();
        for (int t = wave; t < (party > 0 ? 3 : 2) * ell; t += kGateW)
            wave_fwd<false>(y + (t / ell) * kRowBytes, 24 - 8 * (t % ell), l, at, buf + t * kBufBytes, tab);
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
        while (MANY && done < party) {
            const int cnt = min(2, party - done), j0 = done + 1;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (i < nT) {
                    own.put(buf + (kFwd + 2 * i + part) * kBufBytes, cT[i]);
                    cT[i][0] = cT[i][1] = {0.0, 0.0};
                }
            for (int i = 0; i < cnt; ++i) rot(i, j0 + i);
            lds_sync();
            const int nf = cnt * ell, ni = nT * kParts, jT = done + 1 - nT;
            for (int t = wave; t < nf + ni; t += kGateW) {
                if (t < nf) wave_fwd<false>(y + (t / ell) * kRowBytes, 24 - 8 * (t % ell), l, at, buf + t * kBufBytes, tab);
                else wave_inv(buf + (kFwd + t - nf) * kBufBytes, acc + (jT + (t - nf) / 2) * kRowBytes, 16 * ((t - nf) & 1), l, at, tab);
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
        if (wave < 2) {
            wave_inv(buf + (bw + wave) * kBufBytes, y, 16 * wave, l, at, tab);
        } else if (wave < 2 + nT * kParts) {
            const int t = wave - 2;
            wave_inv(buf + (kFwd + t) * kBufBytes, acc + (done + 1 - nT + t / 2) * kRowBytes, 16 * (t & 1), l, at, tab);
        }
        d2 x0[ell][2], x1[ell][2];
        auto load_f = [&]() {
            const KeyBlock kf(a.bk + ((size_t)step * 3 + 1) * ell * kPoly, 2 * ell, word);
#pragma unroll
            for (int d = 0; d < ell; ++d)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        x0[d][s] = kf(d * kPoly + s * 256);
                        x1[d][s] = kf((ell + d) * kPoly + s * 256);
                    }
        };
        
        lds_sync();
        if (wave < ell) wave_fwd<true>(y, 24 - 8 * wave, l, at, buf + wave * kBufBytes, tab);
        load_f();
        lds_sync();
#pragma unroll
        for (int d = 0; d < ell; ++d)
            madd(d, x0[d], cA, x1[d], cB);
        own.put(buf + (kFwd + part) * kBufBytes, cA);
        own.put(buf + (kFwd + 2 + part) * kBufBytes, cB);
        lds_sync();
        if (wave < 4)
            wave_inv(buf + (kFwd + wave) * kBufBytes, acc + (wave < 2 ? 0 : 1 + party) * kRowBytes, 16 * (wave & 1), l, at, tab);
        load_step(min(step + 1, a.st1 - 1));
        asm volatile("" : : "v"(touched[0]), "v"(touched[1]), "v"(touched[2]));
        shift = next_shift;
        lds_sync();
    }
    __syncthreads();
    for (int idx = tid; idx < K1 * kN; idx += kGateT) a.acc[(size_t)g * K1 * kN + idx] = ldw(acc + 4u * idx);
}

size_t fft_gate_lds(int k) {
    return (size_t)(k + 1 + kSlots) * kN * 4 + (size_t)(kGateBufs * kH + kTab9) * 16;
}

}  // namespace

static bool fft_supported(const mk_params &P) { return P.N == kN && P.bk_ell <= kEll; }

// Automatic schedule, unless the caller forces something that only the int8
// kernels have (GEMM tile shapes, team sizes): at N = 1024 the transforms are
// faster at every batch size and party count (ms, int8 kernels / here: one
// gate 34 / 9.5, 256 gates 45 / 9.5, 1024 gates 86 / 32.4 at 2 parties; 1024
// gates 199 / 89 at 4 parties; 64 gates 180 / 61 at 8 parties).
bool use_fft(const mk_ctx *ctx) {
    const DeviceKeys &D = ctx->dev;
    return D.fft_bk && D.rot_kind == MK_ROT_AUTO && !D.team_rows && D.force_tiles[0] < 0 && D.force_tiles[1] < 0;
}

// Transforms the uploaded keys (extended form [-K | K]) and builds the twiddle
// table; nothing for parameter sets this schedule does not run.
int fft_upload(mk_ctx *ctx, hipStream_t s) {
    const mk_params &P = ctx->p;
    DeviceKeys &D = ctx->dev;
    if (!fft_supported(P)) return MK_OK;
    const size_t bk_polys = (size_t)P.k * P.n * 3 * P.bk_ell, evk_polys = (size_t)(P.k + 1) * P.bk_ell;
    if (hipMalloc(&D.fft_bk, bk_polys * kPoly * sizeof(d2)) != hipSuccess) {
        D.fft_bk = nullptr;
        return fail(MK_ENOMEM, "device allocation failed: transformed bootstrapping key");
    }
    if (hipMalloc(&D.fft_evk, evk_polys * kPoly * sizeof(d2)) != hipSuccess) {
        D.fft_evk = nullptr;
        return fail(MK_ENOMEM, "device allocation failed: transformed evaluation key");
    }
    std::vector<d2> tab(kTabWords);
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
    if (hipMalloc(&D.fft_tab, tab.size() * sizeof(d2)) != hipSuccess) {
        D.fft_tab = nullptr;
        return fail(MK_ENOMEM, "device allocation failed: transform tables");
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
static int launch_kernel(Kernel kern, int threads, size_t lds, const FftArgs &a, hipStream_t s) {
    MK_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
           "transform rotation LDS attribute");
    hipLaunchKernelGGL(kern, dim3((unsigned)a.G), dim3(threads), lds, s, a);
    MK_HIP(hipGetLastError(), "transform rotation launch");
    return MK_OK;
}
template <int ELL>
static int launch_ell(const FftArgs &a, bool lean, hipStream_t s) {
    if (lean) return launch_kernel(fft_lean_kernel<ELL>, kLeanT, fft_lean_lds(a.k), a, s);
    if (a.k > 2) return launch_kernel(fft_gate_kernel<ELL, true>, kGateT, fft_gate_lds(a.k), a, s);
    return launch_kernel(fft_gate_kernel<ELL, false>, kGateT, fft_gate_lds(a.k), a, s);
}

int launch_br_fft(mk_ctx *ctx, const uint32_t *abar, uint32_t *acc, size_t count, int steps, hipStream_t s) {
    const mk_params &P = ctx->p;
    DeviceKeys &D = ctx->dev;
    FftArgs a;
    a.k = P.k; a.n = P.n; a.ell = P.bk_ell; a.G = (int)count;
    a.st0 = 0; a.st1 = steps;
    a.offset = decomp_offset(P.bk_ell);
    a.abar = abar; a.acc = acc;
    a.bk = (const d2 *)D.fft_bk; a.evk = (const d2 *)D.fft_evk; a.tab = (const d2 *)D.fft_tab;
    StageTimer t1(ctx, 1, s);
    StageTimer t4(ctx, 4, s);
    // Which kernel: one gate per compute unit at a time, or several.  Measured
    // on MI355X (256 compute units), fft_gate_kernel / fft_lean_kernel, ms: 2
    // parties 256 gates 9.4 / 16.9, 512 gates 18.4 / 21.2, 1024 gates 36.8 /
    // 32.4; 4 parties 256 gates 22.7 / 41, 512 gates 45 / 50, 1024 gates 91 /
    // 89; 8 parties (two lean workgroups fit a compute unit) 256 gates 61 / 116,
    // 512 gates 122 / 143.
    const size_t cus = (size_t)std::max(1, D.num_cus);
    const bool lean = P.k <= 4 && count > 2 * cus;
    // During a capture a launch ends where the stream-ordered steps (four kernels
    // each) would end a graph piece, so pieces stay as long as documented.
    for (int st = 0; st < steps || st == 0; st = std::max(a.st1, 1)) {
        const int room = capture_room(ctx);
        a.st0 = st;
        a.st1 = room == INT_MAX ? steps : std::min(steps, st + (room + 3) / 4);
        int rc = P.bk_ell == 3   ? launch_ell<3>(a, lean, s)
                 : P.bk_ell == 2 ? launch_ell<2>(a, lean, s)
                                 : launch_ell<1>(a, lean, s);
        if (!rc) rc = capture_checkpoint(ctx, s, 4 * (a.st1 - a.st0));
        if (rc) return rc;
    }
    return MK_OK;
}

}  // namespace mk
