// Negacyclic products of the CMux by complex FFTs in double precision, exact.
//
// A real polynomial d of Z[X]/(X^1024 + 1) is held as the complex polynomial
// z_j = d_j + i d_(j+512), j < 512, of C[X]/(X^512 - i) (X^512 = i is one of
// the two square roots of X^1024 = -1; the other is its conjugate and carries
// nothing new).  A product there is a product of values at the 512 roots of
// X^512 = i.
//
// Exactness.  Key words (signed 32-bit) are split k = 2^16 k_hi + k_lo into
// signed halves, |k_hi|, |k_lo| <= 2^15, and each half gets its own product
// V_hi, V_lo with the digits, |digit| <= 2^9.  Every coefficient of the sum
// over four rows is an integer below 4 * 1024 * 2^9 * 2^15 = 2^36, and
// rounding the computed real number to the nearest integer recovers it.  With
// u = 2^-53, to first order in u, z and k the polynomials of a row's digits and
// of a key half (|z| <= 2^14, |k| <= 2^20 in the Euclidean norm), X and K their
// exact values at the 512 roots (|X| = 512^(1/2) |z|, likewise K) and B the sum
// of |z| |k| over the rows, at most 2^36:
//  - A butterfly r = a + w b, s = 2 a - r (see butterfly()) computes r to
//    u (|a| + 2 |b| + |r|): two roundings per component and one of w.  s adds
//    u |s|.  Both errors together are at most 5.46 u of the norm of (a, b), that is
//    3.9 u of the norm of (r, s); the digits' first level, on sums of integers,
//    and twiddles of 1 and -i less.
//  - Forward, nine levels: the computed spectra are within 36 u |X| and 36 u |K|
//    of the exact ones (roots and constants are correctly rounded).  By Cauchy
//    and Schwarz the products of a row are then within 72 u |X| |K| = 512 * 72 u
//    |z| |k|, summed over the roots.
//  - Multiply-add: at most 16 roundings per component, each of a partial sum below
//    the sum of the |X_p| |K_p| over the rows: 512 * 24 u B summed over the roots.
//  - Every coefficient is the sum of 512 products S_p with weights of magnitude
//    1/512 (exact, in the key), so that it inherits at most 96 u B of these.
//  - Inverse: every intermediate value is a sum of its own leaves with such
//    weights, so those of one level are together at most the sum of the
//    |S_p| / 512, which is at most B; a butterfly's outputs are within
//    4 u (|a| + |b|); and each coefficient gets each level's errors once from
//    every node, with weights of magnitude one: 4 u B per level.  A product with
//    a rounded factor (the factors between the group kernel's two transforms, a
//    twist) adds 3 u B.  Group kernel: nine levels and two products, 42 u B.
//    Narrow kernel: eight levels, one product and the join of the halves (4 u B),
//    39 u B.
// Altogether at most 138 u B <= 138 * 2^-17 < 0.0011, where 0.5 would be needed
// to round wrongly, for any key and any digits.  The result V_lo + 2^16 V_hi mod
// 2^32 is therefore the definition's, bit for bit.
//
// Transforms.  Forward: Cooley-Tukey on the ring, X^(2m) - w^2 splitting into
// (X^m - w)(X^m + w), i.e. (a, b) -> (a + w b, a - w b); a node is named by
// the path of its splits (first split = most significant bit), which is also
// its position in place.  With E(k) = exp(i pi k / 1024), the node of path c
// (l bits, c_0 first) below a root X^M - E(2 n) splits with
//   w = E(n / 2^l + (1024 / 2^l) (c_0 + 2 c_1 + 4 c_2 + ...)),
// so the two children of one node split with w and i w: only every second
// twiddle is stored.  Leaf p (9 path bits) is the root E(1 + 4 brv9(p)).
// Inverse: decimation in time from that bit-reversed order, (e, o) ->
// (e + w o, e - w o) with w = exp(-2 pi i j / (2 h)) at span h, then the twist
// E(-j) / 512 of output j.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace fhe {
namespace dev {
namespace fft {

struct alignas(16) cd {
    double x, y;
};

// cos(pi k / 32), k = 0..16, and by symmetry any k.
constexpr double kCos[17] = {1.0,
                             0.9951847266721968862448,
                             0.9807852804032304491262,
                             0.9569403357322088649358,
                             0.9238795325112867561282,
                             0.8819212643483550297128,
                             0.8314696123025452370788,
                             0.7730104533627369608109,
                             0.7071067811865475244008,
                             0.6343932841636454982152,
                             0.5555702330196022247428,
                             0.4713967368259976485564,
                             0.3826834323650897717285,
                             0.2902846772544623676362,
                             0.1950903220161282678483,
                             0.0980171403295606019942,
                             0.0};
constexpr double cos32(int k) {
    k = ((k % 64) + 64) % 64;
    if (k > 32) k = 64 - k;
    return k <= 16 ? kCos[k] : -kCos[32 - k];
}
constexpr double sin32(int k) { return cos32(k - 16); }

constexpr int brv(int x, int bits) {
    int r = 0;
    for (int b = 0; b < bits; ++b)
        if (x & (1 << b)) r |= 1 << (bits - 1 - b);
    return r;
}

template <int B, int E, class F>
__device__ __forceinline__ void unroll(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        unroll<B + 1, E>(f);
    }
}

// (a, b) -> (a + w b, a - w b), six fused multiply-adds: the second output is
// 2 a minus the first.
__device__ __forceinline__ void butterfly(cd& a, cd& b, double wr, double wi) {
    const double r = __builtin_fma(-wi, b.y, __builtin_fma(wr, b.x, a.x));
    const double i = __builtin_fma(wi, b.x, __builtin_fma(wr, b.y, a.y));
    b.x = __builtin_fma(2.0, a.x, -r);
    b.y = __builtin_fma(2.0, a.y, -i);
    a.x = r;
    a.y = i;
}

// The same with w = exp(i pi K / 32) known at compile time.
template <int K>
__device__ __forceinline__ void butterfly_c(cd& a, cd& b) {
    constexpr int k = ((K % 64) + 64) % 64;
    if constexpr (k == 0) {
        const cd t = a;
        a.x = t.x + b.x;
        a.y = t.y + b.y;
        b.x = t.x - b.x;
        b.y = t.y - b.y;
    } else if constexpr (k == 48) {  // w = -i
        const cd t = a, o = b;
        a.x = t.x + o.y;
        a.y = t.y - o.x;
        b.x = t.x - o.y;
        b.y = t.y + o.x;
    } else {
        butterfly(a, b, cos32(k), sin32(k));
    }
}

// Forward on R registers below the root n = 256 (X^512 = i), whose twiddles
// are the same for every lane, from level FROM on.
template <int R, int FROM = 0>
__device__ __forceinline__ void forward_root(cd (&x)[R]) {
    constexpr int L = __builtin_ctz(R);
    unroll<FROM, L>([&](auto l_) {
        constexpr int l = decltype(l_)::value, m = R >> (l + 1);
        unroll<0, (1 << l)>([&](auto c_) {
            constexpr int c = decltype(c_)::value;
            constexpr int k = (256 >> l) + (1024 >> l) * brv(c, l);
            static_assert(k % 32 == 0, "twiddle outside the constants");
            unroll<0, m>([&](auto j_) {
                constexpr int j = decltype(j_)::value;
                butterfly_c<k / 32>(x[2 * m * c + j], x[2 * m * c + j + m]);
            });
        });
    });
}

// Forward on R registers below a lane's own root; w[2^(l-1) + (c >> 1)] (w[0]
// at level 0) is the twiddle of node c of level l, even c.
template <int R, class W>
__device__ __forceinline__ void forward_lane(cd (&x)[R], W&& w) {
    constexpr int L = __builtin_ctz(R);
    unroll<0, L>([&](auto l_) {
        constexpr int l = decltype(l_)::value, m = R >> (l + 1);
        unroll<0, (l == 0 ? 1 : 1 << (l - 1))>([&](auto d_) {
            constexpr int d = decltype(d_)::value;
            const cd t = w(std::integral_constant<int, (l == 0 ? 0 : (1 << (l - 1)) + d)>{});
            unroll<0, (l == 0 ? 1 : 2)>([&](auto s_) {
                constexpr int c = 2 * d + decltype(s_)::value;
                unroll<0, m>([&](auto j_) {
                    constexpr int j = decltype(j_)::value;
                    if constexpr (decltype(s_)::value == 0)
                        butterfly(x[2 * m * c + j], x[2 * m * c + j + m], t.x, t.y);
                    else
                        butterfly(x[2 * m * c + j], x[2 * m * c + j + m], -t.y, t.x);
                });
            });
        });
    });
}

// Inverse on R registers in bit-reversed order, natural order out, twiddles
// the same for every lane.
template <int R>
__device__ __forceinline__ void inverse_root(cd (&x)[R]) {
    constexpr int L = __builtin_ctz(R);
    unroll<0, L>([&](auto l_) {
        constexpr int h = 1 << decltype(l_)::value;
        unroll<0, R / 2>([&](auto k_) {
            constexpr int k = decltype(k_)::value, j = k % h, u = (k / h) * 2 * h + j;
            butterfly_c<-32 * j / h>(x[u], x[u + h]);
        });
    });
}

// Nearest integer of v (|v| < 2^50) mod 2^32: adding 1.5 * 2^52 leaves the
// integer in the low mantissa bits.
__device__ __forceinline__ uint32_t round_word(double v) {
    return (uint32_t)__builtin_bit_cast(uint64_t, v + 6755399441055744.0);
}

}  // namespace fft
}  // namespace dev
}  // namespace fhe
