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
// rounding the computed real number to the nearest integer recovers it: with
// u = 2^-53, a butterfly of two fused multiply-adds per component (see
// butterfly()) adds an error of at most 5.8 u of its outputs' Euclidean norm
// (twiddles are correctly rounded; the digits' first level, on sums of
// integers, less), so nine levels add 52 u, in the digits' transform, in the
// key's and in the inverse alike; the multiply-add over four rows and the final
// twist add less than 16 u.  The Euclidean norms are at most 2^9 * 2^5 (digits)
// and 2^15 * 2^5 (key half) per row, and a coefficient of a product is at most
// the product of the norms: the error is below
// 4 * 2^14 * 2^20 * 172 u = 172 * 2^-17 < 0.0014, where 0.5 would be
// needed to round wrongly.  The result V_lo + 2^16 V_hi mod 2^32 is therefore
// the definition's, bit for bit.
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
