// gfx950 kernels of TFHE gate bootstrapping.
//
// CMux i (TFHE blind rotation): D = X^abar_i ACC - ACC; the two gadget digits
// of its two polynomials (four digit rows) are multiplied by BK_i and summed
// into the two columns of ACC, all modulo 2^32 and X^1024 + 1.  The negacyclic
// products are exact in either of two arithmetics:
//
//   arith 1 (default): complex FFTs of 512 points in double precision with the
//   key words split in two 16-bit halves, which keeps every product
//   coefficient below 2^36 and its rounding exact (the bound is in fft.h).
//
//   arith 0: an NTT over Z_p, p = 2^64 - 2^32 + 1.  Digits are in [-512, 511]
//   and key words are read as signed 32-bit, so every coefficient of a summed
//   product is below 4 * 1024 * 2^9 * 2^31 = 2^52 < p/2 in magnitude and lifts
//   back to Z/2^32 exactly.
//
// Both equal the schoolbook definition bit for bit.
//
// Work layout of arith 0: one wavefront (64 lanes) bootstraps one gate; its
// accumulator (two polynomials of 1024 uint32) lives in LDS.  Lane l = 32h + t
// (half h, t < 32) transforms polynomial data of coefficients m = t + 32*q,
// held in register q (q < 32).  A 1024-point negacyclic
// NTT is split 32 x 32: a 32-point negacyclic transform in registers over q
// (root psi^32 = 8, so every twiddle is a power of two: shifts only), one
// general twiddle psi^(t(2j+1)) per value, a transpose through LDS, and a
// 32-point cyclic transform in registers (root psi^64 = 2^6).  After it, lane
// (h, t) register q holds frequency k = t + 32*brv5(q).  The inverse runs the
// same steps backwards; N^-1 is folded into its twiddles.  Each half extracts
// its own gadget digit (half h -> digit h) of polynomial hp = 0, 1 in two
// passes, transforms it, swaps it with the other half (v_permlane32_swap),
// and half h accumulates output column h against BK_i in the NTT domain.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <type_traits>

#include "fhe_internal.h"
#include "fft.h"
#include "goldilocks.h"
#include "kernels.h"

namespace fhe {
namespace dev {
namespace {

constexpr int N = 1024;
constexpr int NW = 501;            // LWE sample words
constexpr int NLWE = 500;
constexpr uint32_t kDecompOffset = 0x80200800u;  // 2^31 + 2^21 + 2^11

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

__host__ __device__ constexpr int brv5(int x) {
    return ((x & 1) << 4) | ((x & 2) << 2) | (x & 4) | ((x & 8) >> 2) | ((x & 16) >> 4);
}

// ---------------------------------------------------------------------------
// 32-point transforms in registers.
// ---------------------------------------------------------------------------

// Negacyclic forward, root psi2 = 8 (order 64), natural in, bit-reversed out:
// out[q] = sum_i x[i] psi2^(i (2 brv5(q) + 1)).  Merged Cooley-Tukey.
__device__ __forceinline__ void ntt32_neg_fwd(uint64_t (&x)[32]) {
    static_for<0, 5>([&](auto L) {
        constexpr int m = 1 << decltype(L)::value;
        constexpr int t = 16 >> decltype(L)::value;
        static_for<0, m>([&](auto I) {
            constexpr int i = decltype(I)::value;
            constexpr int S = 3 * brv5(m + i);
            static_for<0, t>([&](auto J) {
                constexpr int j = 2 * i * t + decltype(J)::value;
                const uint64_t U = x[j];
                const uint64_t V = gl::mul_pow2<S>(x[j + t]);
                x[j] = gl::add(U, V);
                x[j + t] = gl::sub(U, V);
            });
        });
    });
}

// Cyclic forward, root w = 2^6 (order 32), natural in, bit-reversed out.
// Decimation in frequency.
__device__ __forceinline__ void ntt32_cyc_fwd(uint64_t (&x)[32]) {
    static_for<0, 5>([&](auto L) {
        constexpr int ln = 16 >> decltype(L)::value;
        static_for<0, 16 / ln>([&](auto B) {
            constexpr int st = 2 * ln * decltype(B)::value;
            static_for<0, ln>([&](auto J) {
                constexpr int j = decltype(J)::value;
                constexpr int S = 6 * j * (16 / ln);
                const uint64_t U = x[st + j], V = x[st + j + ln];
                x[st + j] = gl::add(U, V);
                x[st + j + ln] = gl::mul_pow2<S>(gl::sub(U, V));
            });
        });
    });
}

// Inverse of ntt32_cyc_fwd without the 1/32: bit-reversed in, natural out.
// w^-s = -2^(96-s).
__device__ __forceinline__ void ntt32_cyc_inv(uint64_t (&x)[32]) {
    static_for<0, 5>([&](auto L) {
        constexpr int ln = 1 << decltype(L)::value;
        static_for<0, 16 / ln>([&](auto B) {
            constexpr int st = 2 * ln * decltype(B)::value;
            static_for<0, ln>([&](auto J) {
                constexpr int j = decltype(J)::value;
                constexpr int S = 6 * j * (16 / ln);
                const uint64_t U = x[st + j], V = x[st + j + ln];
                if constexpr (S == 0) {
                    x[st + j] = gl::add(U, V);
                    x[st + j + ln] = gl::sub(U, V);
                } else {
                    const uint64_t W = gl::mul_pow2<96 - S>(V);
                    x[st + j] = gl::sub(U, W);
                    x[st + j + ln] = gl::add(U, W);
                }
            });
        });
    });
}

// Inverse of ntt32_neg_fwd without the 1/32: bit-reversed in, natural out.
// Gentleman-Sande; psi2^-e = -2^(96-e), so (U - V) psi2^-e = (V - U) 2^(96-e).
__device__ __forceinline__ void ntt32_neg_inv(uint64_t (&x)[32]) {
    static_for<0, 5>([&](auto L) {
        constexpr int t = 1 << decltype(L)::value;
        constexpr int h = 16 >> decltype(L)::value;
        static_for<0, h>([&](auto I) {
            constexpr int i = decltype(I)::value;
            constexpr int E = 3 * brv5(h + i);
            static_for<0, t>([&](auto J) {
                constexpr int j = 2 * t * i + decltype(J)::value;
                const uint64_t U = x[j], V = x[j + t];
                x[j] = gl::add(U, V);
                x[j + t] = gl::mul_pow2<96 - E>(gl::sub(V, U));
            });
        });
    });
}

// Scheduling fence: keeps the compiler from hoisting the loads of later
// chunks above it, which bounds the registers held by loads in flight.
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Orders the wave's LDS traffic: LDS operations of one wavefront execute in
// issue order, so a compiler-level barrier is all a wave-private exchange
// needs.
typedef __attribute__((address_space(3))) uint32_t lds_u32;

// Word t of an LDS array as an LDS address the optimiser cannot see through,
// so that the 32 reads at t + 32 q share one base register held in the loop
// (otherwise it hoists a base per pair of reads and spills them).
__device__ __forceinline__ const lds_u32* lds_column(const uint32_t* a, int t) {
    const lds_u32* p = (const lds_u32*)(a + t);
    asm volatile("" : "+v"(p));
    return p;
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 32 x 32 transpose of 64-bit values through this half's 4 KB tile of
// 32-bit words, one word of each value at a time.  Element (row, col) sits at
// row*32 + (col ^ row), which keeps both the row writes and the column reads
// free of bank conflicts.  Before: register k holds (row wr(k), col t); after:
// register k holds (row t, col rd(k)).
template <class WR, class RD>
__device__ __forceinline__ void transpose32(uint64_t (&x)[32], uint32_t* tile, int t, WR wr, RD rd) {
    uint32_t lo[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) tile[wr(k) * 32 + (t ^ wr(k))] = (uint32_t)x[k];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) lo[k] = tile[t * 32 + (rd(k) ^ t)];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) tile[wr(k) * 32 + (t ^ wr(k))] = (uint32_t)(x[k] >> 32);
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 32; ++k) x[k] = ((uint64_t)tile[t * 32 + (rd(k) ^ t)] << 32) | lo[k];
    wave_lds_sync();
}

// Full 1024-point forward negacyclic NTT of this half's polynomial.
__device__ __forceinline__ void ntt1024_fwd(uint64_t (&x)[32], uint32_t* tile,
                                            const uint64_t* twf, int t) {
    ntt32_neg_fwd(x);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        sched_fence();
#pragma unroll
        for (int q = 8 * c; q < 8 * c + 8; ++q) x[q] = gl::mul(x[q], twf[q * 32 + t]);
    }
    sched_fence();
    transpose32(x, tile, t, [](int q) { return brv5(q); }, [](int r) { return r; });
    ntt32_cyc_fwd(x);
}

// Inverse of ntt1024_fwd including N^-1 (folded in twi).
__device__ __forceinline__ void ntt1024_inv(uint64_t (&x)[32], uint32_t* tile,
                                            const uint64_t* twi, int t) {
    ntt32_cyc_inv(x);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        sched_fence();
#pragma unroll
        for (int r = 8 * c; r < 8 * c + 8; ++r) x[r] = gl::mul(x[r], twi[r * 32 + t]);
    }
    sched_fence();
    transpose32(x, tile, t, [](int r) { return r; }, [](int q) { return brv5(q); });
    ntt32_neg_inv(x);
}

// Value of the other half's lane with the same t.
__device__ __forceinline__ uint32_t partner32(uint32_t v, int h) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return h ? r[0] : r[1];
}

__device__ __forceinline__ uint64_t partner64(uint64_t v, int h) {
    const uint32_t lo = partner32((uint32_t)v, h);
    const uint32_t hi = partner32((uint32_t)(v >> 32), h);
    return ((uint64_t)hi << 32) | lo;
}

// Per-wave LDS, as views into the block's arrays: the accumulator (two
// polynomials of 1024 words) and one 32 x 32 transpose tile of 32-bit words
// per half.  16 KB.
struct WaveLds {
    uint32_t (&acc)[2][1024];
    uint32_t (&tile)[2][32 * 32];
};

// Shared-memory footprint of a block of WPB one-wave gates: twiddles plus one
// accumulator and one pair of tiles per wave (WPB = 4: 80 KB, so two blocks
// fit a CU's 160 KB, i.e. two waves per SIMD).
template <int WPB>
struct BlockLds {
    uint64_t twf[32 * 32];
    uint64_t twi[32 * 32];
    uint32_t acc[WPB][2][1024];
    uint32_t tile[WPB][2][32 * 32];
};

// Shared memory of one gate bootstrapped by two waves (56 KB): wave w runs
// pass w of every CMux; wave 1 hands its multiply-accumulate result to wave 0
// through `part`, and wave 0 finishes the step.
struct PairLds {
    uint64_t twf[32 * 32];
    uint64_t twi[32 * 32];
    uint32_t acc[2][1024];
    uint32_t tile[2][2][32 * 32];  // [wave][half]
    uint64_t part[32][64];         // [register q][lane]
};

// Pass HP of a CMux step: D = X^ai ACC_HP - ACC_HP (a = ACC_HP), this half's
// gadget digit of it (half h extracts digit h), its forward NTT, then the
// multiply-accumulate against BK_i rows (2HP + h) and (2HP + 1 - h), column h,
// added to mac when ACCUM (else stored).  tile: this half's transpose tile;
// bk_i: BK_i in the kernel layout [hp][q][sel][64 lanes].  PREFETCH issues
// the 64 key loads before the digit extraction so that their latency hides
// behind the forward NTT (128 more registers live across it).
template <int HP, bool ACCUM, bool PREFETCH>
__device__ __forceinline__ void cmux_pass(const uint32_t* a, uint32_t* tile, int ai,
                                          const uint64_t* __restrict__ bk_i,
                                          const uint64_t* twf, int lane, uint64_t (&mac)[32]) {
    const int h = lane >> 5, t = lane & 31;
    const int shift = 22 - 10 * h;
    uint64_t b_pre[PREFETCH ? 64 : 1];
    if constexpr (PREFETCH) {
        const uint64_t* bkp = bk_i + (size_t)HP * (32 * 2 * 64) + lane;
#pragma unroll
        for (int k = 0; k < 64; ++k) b_pre[k] = bkp[k * 64];
    }
    uint64_t x[32];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        sched_fence();
#pragma unroll
        for (int q = 8 * c; q < 8 * c + 8; ++q) {
            const int m = t + 32 * q;
            const int s = (m - ai) & 2047;
            const uint32_t v = a[s & 1023];
            const uint32_t rot = (s & 1024) ? 0u - v : v;
            const uint32_t D = rot - a[m];
            const int32_t dg = (int32_t)(((D + kDecompOffset) >> shift) & 1023u) - 512;
            x[q] = gl::from_i64(dg);
        }
    }
    sched_fence();
    ntt1024_fwd(x, tile, twf, t);
    const uint64_t* bkp = bk_i + (size_t)HP * (32 * 2 * 64) + lane;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        sched_fence();
#pragma unroll
        for (int q = 4 * c; q < 4 * c + 4; ++q) {
            const uint64_t other = partner64(x[q], h);
            uint64_t b_own, b_oth;
            if constexpr (PREFETCH) {
                b_own = b_pre[q * 2 + 0];
                b_oth = b_pre[q * 2 + 1];
            } else {
                b_own = bkp[(q * 2 + 0) * 64];
                b_oth = bkp[(q * 2 + 1) * 64];
            }
            const uint64_t v = gl::add(gl::mul(x[q], b_own), gl::mul(other, b_oth));
            mac[q] = ACCUM ? gl::add(mac[q], v) : v;
        }
    }
    sched_fence();
}

// Inverse NTT of the two output columns (half h: column h) and ACC += their
// lift to Z/2^32.
__device__ __forceinline__ void cmux_finish(uint32_t (&acc)[2][1024], uint32_t* tile,
                                            uint64_t (&mac)[32], const uint64_t* twi, int lane) {
    const int h = lane >> 5, t = lane & 31;
    ntt1024_inv(mac, tile, twi, t);
    uint32_t* mine = acc[h];
#pragma unroll
    for (int q = 0; q < 32; ++q) mine[t + 32 * q] += gl::lift32(mac[q]);
}

// One CMux step on this wave's accumulator W.acc:
//   ACC += BK_i [x] (X^ai ACC - ACC).
__device__ __forceinline__ void cmux_step(WaveLds& W, int ai, const uint64_t* __restrict__ bk_i,
                                          const uint64_t* twf, const uint64_t* twi, int lane) {
    const int h = lane >> 5;
    uint64_t mac[32];
    cmux_pass<0, false, false>(W.acc[0], W.tile[h], ai, bk_i, twf, lane, mac);
    cmux_pass<1, true, false>(W.acc[1], W.tile[h], ai, bk_i, twf, lane, mac);
    cmux_finish(W.acc, W.tile[h], mac, twi, lane);
    wave_lds_sync();
}

// ---------------------------------------------------------------------------
// The same CMux with its products by complex FFTs in double precision (fft.h):
// four digit rows r = 2 hp + digit forward, four outputs o = 2 c + half back
// (column c, key half), 512 complex points each.
// ---------------------------------------------------------------------------

using fft::cd;

// The key's transform, on one wavefront (64 lanes x 8 registers, 512 = 8 x 8 x
// 8): coefficient j = lane + 64 reg before, leaf
// p = 8 lane + reg after.  Between the passes the registers are exchanged with
// the lanes' upper, then lower three bits through the wave's own 9 KB of LDS;
// the strides of 72 and 9 sixteen-byte slots spread the sixteen lanes that
// read together over all 64 banks.
constexpr int kExSlots = 576;

// A lane's twiddles of passes 2 and 3.
struct LaneTwiddles {
    cd f2[4], f3[4];
};

__device__ __forceinline__ cd conj_root(const cd* __restrict__ roots, int k) {
    const cd e = roots[k & 2047];
    return {e.x, -e.y};
}

__device__ __forceinline__ int brv3(int x) { return ((x & 1) << 2) | (x & 2) | ((x >> 2) & 1); }

__device__ __forceinline__ void load_forward_twiddles(LaneTwiddles& W, const cd* __restrict__ roots, int lane) {
    const int n2 = 32 + 128 * brv3(lane >> 3);
    const int n3 = 4 + 16 * brv3(lane >> 3) + 128 * brv3(lane & 7);
    W.f2[0] = roots[n2], W.f2[1] = roots[n2 / 2], W.f2[2] = roots[n2 / 4], W.f2[3] = roots[n2 / 4 + 256];
    W.f3[0] = roots[n3], W.f3[1] = roots[n3 / 2], W.f3[2] = roots[n3 / 4], W.f3[3] = roots[n3 / 4 + 256];
}

// Exchanges through the wave's slots: registers written at base + stride k,
// read at base + stride k.
template <int WS, int RS>
__device__ __forceinline__ void wave_exchange(cd (&x)[8], cd* wbase, const cd* rbase) {
#pragma unroll
    for (int k = 0; k < 8; ++k) wbase[WS * k] = x[k];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = rbase[RS * k];
    wave_lds_sync();
}

__device__ __forceinline__ void fft512_forward(cd (&x)[8], cd* ex, const LaneTwiddles& W, int lane) {
    const int hi = lane >> 3, lo = lane & 7;
    fft::forward_root<8>(x);
    wave_exchange<72, 8>(x, ex + lane, ex + hi * 72 + lo);
    fft::forward_lane<8>(x, [&](auto k) { return W.f2[decltype(k)::value]; });
    wave_exchange<9, 1>(x, ex + hi * 72 + lo, ex + hi * 72 + 9 * lo);
    fft::forward_lane<8>(x, [&](auto k) { return W.f3[decltype(k)::value]; });
}

__device__ __forceinline__ void mac(cd& o, const cd& k, const cd& x) {
    o.x = __builtin_fma(-k.y, x.y, __builtin_fma(k.x, x.x, o.x));
    o.y = __builtin_fma(k.y, x.x, __builtin_fma(k.x, x.y, o.y));
}

// Barrier for data exchanged through LDS alone: key loads in flight stay in
// flight (__syncthreads would wait for them).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void lds_add(uint32_t* p, uint32_t v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---------------------------------------------------------------------------
// One gate on eight wavefronts, two per digit row (and per output): wave
// (row, half) keeps the half of the ring X^512 - i = (X^256 - w)(X^256 + w),
// w = E(256), i.e. 256 of a row's leaves, four registers per lane.  The four
// waves of a polynomial share its digit words; both waves of a row fold its
// digits by the first split, and the other eight levels are four passes of two
// levels in registers.  Registers and lane bits are exchanged between the
// passes: bits 5, 4 by v_permlane32/16_swap, bits 3, 2 by moves within rows of
// 16 lanes, bits 1, 0 through the wave's slots in LDS.  The last level of the
// inverse joins the two halves through LDS.
// ---------------------------------------------------------------------------

constexpr int kNarrowSlots = 320;
constexpr int kPad = 64;  // words before each accumulator polynomial: -ACC[960 + k]

// LEAN: two gates per compute unit, in half of the LDS and 128 registers.  The
// spectra stay in the waves' exchange slots (one more barrier), the twiddles of
// passes 3 and 4 in LDS, and two rows of keys instead of four in registers.
template <bool LEAN>
struct alignas(16) NarrowLds {
    uint32_t acc[2][kPad + 1024];
    uint32_t tail[kPad];  // (makes the padded view below end inside the struct)
    uint4 digits[2][4][64];  // digit words of coefficients lane + 64 (4 part + word)
    cd ex[8][kNarrowSlots];
    cd spec[LEAN ? 1 : 8][LEAN ? 1 : 256];
    cd tw[2][256];                       // [half]: E(-j), E(-5 j)
    cd fwd[LEAN ? 2 : 1][LEAN ? 4 : 1][64];  // [half]: f3, f4 of NarrowTwiddles
    cd inv[LEAN ? 4 : 1][64];                // i3, i4
    // The spectrum of a wave, 256 leaves.
    __device__ __forceinline__ cd* spectrum(int wave) {
        if constexpr (LEAN)
            return ex[wave];
        else
            return spec[wave];
    }
    // The accumulator polynomials behind their pads.
    __device__ __forceinline__ uint32_t (&view())[2][kPad + 1024] {
        return *reinterpret_cast<uint32_t (*)[2][kPad + 1024]>(&acc[0][kPad]);
    }
};

struct NarrowTwiddles {
    cd f1[2];                     // pass 1, the same for the whole wave
    cd f2[2], f3[2], f4[2];       // forward passes 2..4
    cd i2[2], i3[2], i4[2];       // inverse passes 2..4 (conjugates)
};

template <bool LEAN>
__device__ __forceinline__ void load_narrow_twiddles(NarrowLds<LEAN>& S, NarrowTwiddles& T,
                                                     const cd* __restrict__ roots, int wave, int half, int lane) {
    const int p2 = half + 2 * ((lane >> 5) & 1) + 4 * ((lane >> 4) & 1);
    const int p3 = p2 + 8 * ((lane >> 3) & 1) + 16 * ((lane >> 2) & 1);
    const int p4 = p3 + 32 * ((lane >> 1) & 1) + 64 * (lane & 1);
    T.f1[0] = roots[128 + 512 * half], T.f1[1] = roots[64 + 256 * half];
    T.f2[0] = roots[32 + 128 * p2], T.f2[1] = roots[16 + 64 * p2];
    T.f3[0] = roots[8 + 32 * p3], T.f3[1] = roots[4 + 16 * p3];
    T.f4[0] = roots[2 + 8 * p4], T.f4[1] = roots[1 + 4 * p4];
    T.i2[0] = conj_root(roots, 256 * (lane & 3)), T.i2[1] = conj_root(roots, 128 * (lane & 3));
    T.i3[0] = conj_root(roots, 64 * (lane & 15)), T.i3[1] = conj_root(roots, 32 * (lane & 15));
    T.i4[0] = conj_root(roots, 16 * lane), T.i4[1] = conj_root(roots, 8 * lane);
    if constexpr (LEAN) {
        if (wave < 2) {
            S.fwd[half][0][lane] = T.f3[0], S.fwd[half][1][lane] = T.f3[1];
            S.fwd[half][2][lane] = T.f4[0], S.fwd[half][3][lane] = T.f4[1];
            S.inv[0][lane] = T.i3[0], S.inv[1][lane] = T.i3[1];
            S.inv[2][lane] = T.i4[0], S.inv[3][lane] = T.i4[1];
        }
    }
    for (int j = lane; j < 256; j += 64)
        if (wave < 2) S.tw[half][j] = conj_root(roots, half ? 5 * j : j);
}

__device__ __forceinline__ double with_words(uint32_t lo, uint32_t hi) {
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Exchanges the register bit that tells a from b with lane bit 5 (ROW16: 4).
template <bool ROW16>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    if constexpr (ROW16) {
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        a = with_words(l[0], h[0]);
        b = with_words(l[1], h[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        a = with_words(l[0], h[0]);
        b = with_words(l[1], h[1]);
    }
}

// Register bits (1, 0) <-> lane bits (5, 4).
__device__ __forceinline__ void exchange_high(cd (&x)[4]) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        lane_swap<false>(x[k].x, x[k + 2].x);
        lane_swap<false>(x[k].y, x[k + 2].y);
    }
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        lane_swap<true>(x[k].x, x[k + 1].x);
        lane_swap<true>(x[k].y, x[k + 1].y);
    }
}

// The same with lane bit 3 (N = 8) or 2 (N = 4), by moves within rows of 16.
template <int N>
__device__ __forceinline__ void row_swap(double& a, double& b) {
    constexpr int kUpper = N == 8 ? 0xC : 0xA;  // banks of four lanes that have the bit
    uint32_t x[2] = {(uint32_t)__builtin_bit_cast(uint64_t, a), (uint32_t)(__builtin_bit_cast(uint64_t, a) >> 32)};
    uint32_t y[2] = {(uint32_t)__builtin_bit_cast(uint64_t, b), (uint32_t)(__builtin_bit_cast(uint64_t, b) >> 32)};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t old = x[k];
        x[k] = (uint32_t)__builtin_amdgcn_update_dpp((int)x[k], (int)y[k], 0x110 + N, 0xF, kUpper, false);
        y[k] = (uint32_t)__builtin_amdgcn_update_dpp((int)y[k], (int)old, 0x100 + N, 0xF, 0xF ^ kUpper, false);
    }
    a = with_words(x[0], x[1]);
    b = with_words(y[0], y[1]);
}

// Register bits (1, 0) <-> lane bits (3, 2).
__device__ __forceinline__ void exchange_mid(cd (&x)[4]) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        row_swap<8>(x[k].x, x[k + 2].x);
        row_swap<8>(x[k].y, x[k + 2].y);
    }
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        row_swap<4>(x[k].x, x[k + 1].x);
        row_swap<4>(x[k].y, x[k + 1].y);
    }
}

// Two levels on four registers below a node: w[0] splits it, w[1] its even
// child (the odd child's twiddle is i w[1]).
__device__ __forceinline__ void forward4(cd (&x)[4], const cd (&w)[2]) {
    fft::butterfly(x[0], x[2], w[0].x, w[0].y);
    fft::butterfly(x[1], x[3], w[0].x, w[0].y);
    fft::butterfly(x[0], x[1], w[1].x, w[1].y);
    fft::butterfly(x[2], x[3], -w[1].y, w[1].x);
}

__device__ __forceinline__ void inverse4(cd (&x)[4], const cd (&w)[2]) {
    fft::butterfly(x[0], x[1], w[0].x, w[0].y);
    fft::butterfly(x[2], x[3], w[0].x, w[0].y);
    fft::butterfly(x[0], x[2], w[1].x, w[1].y);
    fft::butterfly(x[1], x[3], w[1].y, -w[1].x);
}

template <int WS, int RS>
__device__ __forceinline__ void exchange_low(cd (&x)[4], cd* wbase, const cd* rbase) {
#pragma unroll
    for (int k = 0; k < 4; ++k) wbase[WS * k] = x[k];
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = rbase[RS * k];
    wave_lds_sync();
}

// Key words of row r, output o, half, register j, lane (narrow layout).
__device__ __forceinline__ void load_narrow_keys(cd (&k)[4], const cd* __restrict__ key, int r, int o, int half,
                                                 int lane) {
    const cd* p = key + (((r * 4 + o) * 2 + half) * 4) * 64 + lane;
#pragma unroll
    for (int j = 0; j < 4; ++j) k[j] = p[64 * j];
}

// One CMux step of wave (row, half).  ka[k]: the step's keys of row (row + k)
// mod 4; k = 0, 1 are loaded a step ahead (from `next`), k = 2, 3 during the
// forward transform (LEAN: into the registers of 0 and 1 once those are used).
// Four barriers: digits written, spectra written, halves joined, ACC updated
// (LEAN: one more, spectra read).
template <bool LEAN>
__device__ __forceinline__ void narrow_step(NarrowLds<LEAN>& S, int ai, const cd* __restrict__ cur,
                                            const cd* __restrict__ next, cd (&ka)[LEAN ? 2 : 4][4],
                                            const NarrowTwiddles& T, int row, int half, int lane) {
    cd* ex = S.ex[2 * row + half];
    const int u = lane >> 2, v = lane & 3;
    cd* e3a = ex + 20 * u + v;      // bits 1, 0: stride 5 by register,
    cd* e3b = ex + 20 * u + 5 * v;  // stride 1 after the exchange
    cd x[4];
    {
        // D = X^ai ACC - ACC, four words per lane and wave: the four waves of
        // a polynomial share them through LDS.  Coefficient lane + 64 e reads
        // block (e - ai / 64) mod 16 at lane - ai mod 64 (the pad serves
        // negative ones), negated when (e - ai / 64) mod 32 >= 16, the same
        // for the whole wave.
        const int hp = row >> 1, part = 2 * (row & 1) + half;
        const uint32_t* a = S.view()[hp];
        const lds_u32* am = lds_column(a + 256 * part, lane);
        const uint32_t rot = (uint32_t)(uintptr_t)(const lds_u32*)a + 4 * (uint32_t)(lane - (ai & 63));
        const uint32_t first = (4u * part - ((uint32_t)ai >> 6)) << 8;
        uint32_t w[4], own[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w[e] = *(const lds_u32*)(uintptr_t)(rot + ((first + 256u * e) & 0xF00u));
            own[e] = am[64 * e];
        }
        uint32_t z[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t sgn = (uint32_t)((int32_t)((first + 256u * e) << 19) >> 31);
            z[e] = ((w[e] ^ sgn) + (kDecompOffset - sgn - own[e])) ^ 0x80200000u;
        }
        S.digits[hp][part][lane] = make_uint4(z[0], z[1], z[2], z[3]);
        lds_barrier();  // digit words written; every wave has read ACC
        const int shift = 22 - 10 * (row & 1);
        int32_t d[16];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint4 q = S.digits[hp][e][lane];
            d[4 * e + 0] = (int32_t)__builtin_amdgcn_sbfe((int32_t)q.x, shift, 10);
            d[4 * e + 1] = (int32_t)__builtin_amdgcn_sbfe((int32_t)q.y, shift, 10);
            d[4 * e + 2] = (int32_t)__builtin_amdgcn_sbfe((int32_t)q.z, shift, 10);
            d[4 * e + 3] = (int32_t)__builtin_amdgcn_sbfe((int32_t)q.w, shift, 10);
        }
        // first split: a + w b or a - w b with w = (1 + i) / sqrt 2
        const double c = half ? -fft::kCos[8] : fft::kCos[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k].x = __builtin_fma(c, (double)(d[k + 4] - d[k + 12]), (double)d[k]);
            x[k].y = __builtin_fma(c, (double)(d[k + 4] + d[k + 12]), (double)d[k + 8]);
        }
    }
    if constexpr (!LEAN) load_narrow_keys(ka[2], cur, (row + 2) & 3, row, half, lane);
    sched_fence();
    forward4(x, T.f1);
    exchange_high(x);
    forward4(x, T.f2);
    exchange_mid(x);
    if constexpr (LEAN) {
        const cd w3[2] = {S.fwd[half][0][lane], S.fwd[half][1][lane]};
        forward4(x, w3);
        exchange_low<5, 1>(x, e3a, e3b);
        const cd w4[2] = {S.fwd[half][2][lane], S.fwd[half][3][lane]};
        forward4(x, w4);
    } else {
        load_narrow_keys(ka[3], cur, (row + 3) & 3, row, half, lane);
        sched_fence();
        forward4(x, T.f3);
        exchange_low<5, 1>(x, e3a, e3b);
        forward4(x, T.f4);
    }
    cd* mine = S.spectrum(2 * row + half);
#pragma unroll
    for (int j = 0; j < 4; ++j) mine[64 * j + lane] = x[j];
    lds_barrier();  // spectra written
    cd out[4];
    auto mac_row = [&](int k, const cd (&keys)[4], const cd (&s)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (k == 0) out[j] = {0.0, 0.0};
            mac(out[j], keys[j], s[j]);
        }
    };
    auto read_row = [&](int k, cd (&s)[4]) {
        const cd* p = S.spectrum(2 * ((row + k) & 3) + half);
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = p[64 * j + lane];
    };
    mac_row(0, ka[0], x);
    if constexpr (LEAN) {
        cd s1[4], s2[4], s3[4];
        load_narrow_keys(ka[0], cur, (row + 2) & 3, row, half, lane);
        read_row(1, s1);
        mac_row(1, ka[1], s1);
        load_narrow_keys(ka[1], cur, (row + 3) & 3, row, half, lane);
        read_row(2, s2);
        read_row(3, s3);
        lds_barrier();  // spectra read
        mac_row(2, ka[0], s2);
        mac_row(3, ka[1], s3);
    } else {
        cd s1[4], s2[4], s3[4];
        read_row(1, s1);
        read_row(2, s2);
        read_row(3, s3);
        mac_row(1, ka[1], s1);
        mac_row(2, ka[2], s2);
        mac_row(3, ka[3], s3);
    }
    sched_fence();
    fft::inverse_root<4>(out);
    exchange_low<1, 5>(out, e3b, e3a);
    load_narrow_keys(ka[0], next, (row + 0) & 3, row, half, lane);
    sched_fence();
    inverse4(out, T.i2);
    exchange_mid(out);
    if constexpr (LEAN) {
        const cd w3[2] = {S.inv[0][lane], S.inv[1][lane]};
        inverse4(out, w3);
        exchange_high(out);
        const cd w4[2] = {S.inv[2][lane], S.inv[3][lane]};
        inverse4(out, w4);
    } else {
        inverse4(out, T.i3);
        exchange_high(out);
        inverse4(out, T.i4);
    }
    load_narrow_keys(ka[1], next, (row + 1) & 3, row, half, lane);
    sched_fence();
    // last level and twist: with e = E(-j) even_j and o = E(-5 j) odd_j, the
    // outputs are e + o at j = lane + 64 q and (e - o) E(-256) at j + 256
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const cd f = S.tw[half][64 * q + lane], y = out[q];
        out[q] = {__builtin_fma(f.x, y.x, -(f.y * y.y)), __builtin_fma(f.x, y.y, f.y * y.x)};
        ex[64 * q + lane] = out[q];
    }
    lds_barrier();
    const cd* other = S.ex[2 * row + (half ^ 1)];
    const int o = row;
    uint32_t* accw = &S.view()[o >> 1][lane + 256 * half];
    uint32_t w[8];
    if (half == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const cd y = other[64 * q + lane];
            w[q] = fft::round_word(out[q].x + y.x);
            w[q + 4] = fft::round_word(out[q].y + y.y);
        }
    } else {
        constexpr double c = fft::kCos[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const cd y = other[64 * q + lane];
            const double dx = y.x - out[q].x, dy = y.y - out[q].y;
            w[q] = fft::round_word(c * (dx + dy));
            w[q + 4] = fft::round_word(c * (dy - dx));
        }
    }
    const int sh = 16 * (o & 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        lds_add(accw + 64 * q, w[q] << sh);
        lds_add(accw + 64 * q + 512, w[q + 4] << sh);
    }
    if (half == 1) lds_add(&S.acc[o >> 1][lane], 0u - (w[7] << sh));
    lds_barrier();  // ACC updated; spectra free
}

// Gate constants: phase offset kappa and input signs (TFHE +-1/8 encoding)
// of the two-input codes 0..9.
__device__ __forceinline__ void gate_consts(uint32_t op, uint32_t& kappa, int32_t& s1, int32_t& s2) {
    constexpr uint32_t mu = kMu;
    switch (op) {
    case FHE_AND:   kappa = 0u - mu;      s1 = 1;  s2 = 1;  break;
    case FHE_NAND:  kappa = mu;           s1 = -1; s2 = -1; break;
    case FHE_OR:    kappa = mu;           s1 = 1;  s2 = 1;  break;
    case FHE_NOR:   kappa = 0u - mu;      s1 = -1; s2 = -1; break;
    case FHE_XOR:   kappa = 2u * mu;      s1 = 2;  s2 = 2;  break;
    case FHE_XNOR:  kappa = 0u - 2u * mu; s1 = -2; s2 = -2; break;
    case FHE_ANDNY: kappa = 0u - mu;      s1 = -1; s2 = 1;  break;
    case FHE_ANDYN: kappa = 0u - mu;      s1 = 1;  s2 = -1; break;
    case FHE_ORNY:  kappa = mu;           s1 = -1; s2 = 1;  break;
    default:        kappa = mu;           s1 = 1;  s2 = -1; break;  // FHE_ORYN
    }
}

// Value (+1 true, -1 false) of a symmetric two-input code with k of its two
// inputs true; 0 for a code that is not symmetric (compound gates take
// AND, NAND, OR, NOR, XOR, XNOR).
__device__ __forceinline__ int32_t sym_value(uint32_t op, int k) {
    switch (op) {
    case FHE_AND:  return k == 2 ? 1 : -1;
    case FHE_NAND: return k == 2 ? -1 : 1;
    case FHE_OR:   return k >= 1 ? 1 : -1;
    case FHE_NOR:  return k >= 1 ? -1 : 1;
    case FHE_XOR:  return k == 1 ? 1 : -1;
    case FHE_XNOR: return k == 1 ? -1 : 1;
    default:       return 0;
    }
}

// What gate g of a batch computes (uniform over the wave).
struct GateMode {
    uint32_t op0, op1;  // code; second code of a compound gate
    bool compound;      // two symmetric gates from one rotation
    bool three;         // MAJ / XOR3 with a third input
    bool valid;
};

__device__ __forceinline__ GateMode gate_mode(const GateIO& io, uint32_t g) {
    GateMode m{0u, 0u, false, false, true};
    if (io.tv) return m;  // programmable bootstrapping: no gate code
    uint32_t op;
    bool has3;
    if (io.desc) {
        op = io.desc[g].x;
        has3 = io.desc3 != nullptr;
        m.compound = (op & kCompoundFlag) != 0;
    } else {
        op = io.ops ? io.ops[g] : io.op_const;
        has3 = io.in2 != nullptr;
        m.compound = io.ops1 != nullptr;
    }
    if (m.compound) {
        m.op0 = op & 0xFFu;
        m.op1 = io.desc ? (op >> 8) & 0xFFu : io.ops1[g];
        m.valid = sym_value(m.op0, 0) != 0 && sym_value(m.op1, 0) != 0 && (!io.desc || op < 2 * kCompoundFlag);
        return m;
    }
    m.op0 = op;
    m.three = has3 && (op == FHE_MAJ || op == FHE_XOR3);
    m.valid = op <= FHE_ORYN || m.three;
    return m;
}

__device__ __forceinline__ uint32_t* wire_ptr(const GateIO& io, uint32_t w) {
    return io.region[w >> 30] + (size_t)(w & 0x3FFFFFFFu) * NW;
}

// Input samples of gate g; c3 is null unless the gate takes three inputs.
__device__ __forceinline__ void gate_operands(const GateIO& io, uint32_t g, const GateMode& m,
                                              const uint32_t*& c1, const uint32_t*& c2, const uint32_t*& c3) {
    c3 = nullptr;
    if (io.desc) {
        const uint4 d = io.desc[g];
        c1 = wire_ptr(io, d.y);
        c2 = wire_ptr(io, d.z);
        if (m.three) c3 = wire_ptr(io, io.desc3[g]);
    } else {
        c1 = io.in0 + (size_t)g * NW;
        c2 = io.in1 + (size_t)g * NW;
        if (m.three) c3 = io.in2 + (size_t)g * NW;
    }
}

__device__ __forceinline__ uint32_t* gate_output(const GateIO& io, uint32_t g) {
    return io.desc ? wire_ptr(io, io.desc[g].w) : io.out + (size_t)g * NW;
}

// Output of key-switched sample k: gate k, or with pair slots output k & 1
// of gate k >> 1 (null for the unused second slot of a single gate).
__device__ __forceinline__ uint32_t* ks_output(const GateIO& io, uint32_t k) {
    if (!io.pair_slots) return gate_output(io, k);
    const uint32_t g = k >> 1;
    if ((k & 1) == 0) return gate_output(io, g);
    if (io.desc) return (io.desc[g].x & kCompoundFlag) ? wire_ptr(io, io.desc3[g]) : nullptr;
    return io.ops1 ? io.out1 + (size_t)g * NW : nullptr;
}

template <int THREADS, class L>
__device__ __forceinline__ void load_twiddles(L& S, const uint64_t* twf, const uint64_t* twi) {
    for (int k = threadIdx.x; k < 1024; k += THREADS) {
        S.twf[k] = twf[k];
        S.twi[k] = twi[k];
    }
    __syncthreads();
}

// Gate linear combination and modulus switch to Z_2N.  Lane l keeps abar of
// words l + 64k in ab[k]; returns bbar (uniform).  Two-input codes: (0,
// kappa) + s1 c1 + s2 c2; MAJ: c1 + c2 + c3; XOR3: -2 (c1 + c2 + c3);
// compound gates: c1 + c2; programmable bootstrapping: c1 itself.
__device__ __forceinline__ int gate_prologue(const GateIO& io, uint32_t g, int lane, uint32_t (&ab)[8]) {
    const GateMode m = gate_mode(io, g);
    const uint32_t *c1, *c2, *c3;
    gate_operands(io, g, m, c1, c2, c3);
    uint32_t kappa = 0;
    int32_t s1 = 1, s2 = 1, s3 = 0;
    if (io.tv) {
        s2 = 0;
    } else if (m.three) {
        s1 = s2 = s3 = m.op0 == FHE_MAJ ? 1 : -2;
    } else if (!m.compound) {
        gate_consts(m.op0, kappa, s1, s2);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int w = lane + 64 * k;
        uint32_t v = 0;
        if (w < NW) {
            v = (uint32_t)s1 * c1[w] + (uint32_t)s2 * c2[w];
            if (c3) v += (uint32_t)s3 * c3[w];
            if (w == NLWE) v += kappa;
        }
        ab[k] = (v + (1u << 20)) >> 21;
    }
    return __builtin_amdgcn_readlane(ab[7], NLWE - 448);
}

// Constant test vector of gate g: mu = 1/8 for the gates, 1/16 for compound
// gates (their two outputs are weighted sums of two extractions).
__device__ __forceinline__ uint32_t gate_mu(const GateIO& io, uint32_t g) {
    return gate_mode(io, g).compound ? kMu >> 1 : kMu;
}

// Test-vector rotation: ACC = (0, X^(2N - bbar) v), v = mu (1 + X + ... +
// X^(N-1)).  Lane l = 32h + t writes coefficients t + 32q of polynomial h.
// With a test vector tv (programmable bootstrapping): ACC = (0, X^c tv),
// coefficient m = tv[j] for j = (m - c) mod 2N < N, else -tv[j - N].
template <int S>
__device__ __forceinline__ void acc_init(uint32_t (&acc)[2][S], int bbar, int h, int t,
                                         const uint32_t* __restrict__ tv, uint32_t mu) {
    const int c = (2 * N - bbar) & (2 * N - 1);
    if (tv) {
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            const int m = t + 32 * q;
            const int j = (m - c) & (2 * N - 1);
            const uint32_t v = tv[j & (N - 1)];
            acc[h][m] = h == 0 ? 0u : (j < N ? v : 0u - v);
        }
        return;
    }
    const int cm = c & (N - 1);
    const uint32_t neg = (c >= N) ? 1u : 0u;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const int m = t + 32 * q;
        const uint32_t sgn = (m >= cm) ? neg : 1u - neg;  // 1 -> -mu
        acc[h][m] = h == 0 ? 0u : (sgn ? 0u - mu : mu);
    }
}

// An extracted sample as key switching reads it: word q of 512 holds the 16
// bits kept of a'_2q (low half) and a'_(2q+1), i.e. eight base-4 digits each;
// word 512 is b'.  Slots are kSampleWords apart.
__device__ __forceinline__ uint32_t kept_bits(uint32_t a) { return (a + (1u << 15)) >> 16; }
__device__ __forceinline__ uint32_t pack_kept(uint32_t even, uint32_t odd) {
    return kept_bits(even) | kept_bits(odd) << 16;
}

// Sample extraction of coefficient 0: a'_0 = a_0, a'_m = -a_(N-m), b' = b_0,
// by THREADS threads with index `tid`.
template <int THREADS, int S>
__device__ __forceinline__ void sample_extract(const uint32_t (&acc)[2][S], uint32_t* o, int tid) {
    for (int q = tid; q < N / 2; q += THREADS)
        o[q] = pack_kept(q == 0 ? acc[0][0] : 0u - acc[0][N - 2 * q], 0u - acc[0][N - 2 * q - 1]);
    if (tid == 0) o[N / 2] = acc[1][0];
}

// Compound gate outputs.  The accumulator was rotated from the test vector
// 1/16 by the phase of c1 + c2 (-1/4, 0, +1/4 for k = 0, 1, 2 true inputs);
// the extractions of coefficients 3N/4 (E1) and N/4 (E2) then encrypt
// (E1, E2) = (+,-), (+,+), (-,+) x 1/16 for k = 0, 1, 2.  A symmetric gate
// with values g0, g1, g2 (+-1, units of 1/8) is the sample
// (g1 - g2) E1 + (g1 - g0) E2 + (0, (g0 + g2)/16).  Extraction of
// coefficient m: a'_j = a_(m-j) for j <= m, -a_(N+m-j) for j > m, b' = b_m.
template <int THREADS, int S>
__device__ __forceinline__ void compound_extract(const uint32_t (&acc)[2][S], uint32_t op0, uint32_t op1,
                                                 uint32_t* o0, uint32_t* o1, int tid) {
    constexpr int m1 = 3 * N / 4, m2 = N / 4;
    const int32_t a0 = sym_value(op0, 0), a1 = sym_value(op0, 1), a2 = sym_value(op0, 2);
    const int32_t b0 = sym_value(op1, 0), b1 = sym_value(op1, 1), b2 = sym_value(op1, 2);
    const uint32_t x0 = (uint32_t)(a1 - a2), y0 = (uint32_t)(a1 - a0);
    const uint32_t x1 = (uint32_t)(b1 - b2), y1 = (uint32_t)(b1 - b0);
    for (int q = tid; q < N / 2; q += THREADS) {
        uint32_t v0[2], v1[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int j = 2 * q + s;
            const uint32_t e1 = j <= m1 ? acc[0][m1 - j] : 0u - acc[0][N + m1 - j];
            const uint32_t e2 = j <= m2 ? acc[0][m2 - j] : 0u - acc[0][N + m2 - j];
            v0[s] = x0 * e1 + y0 * e2;
            v1[s] = x1 * e1 + y1 * e2;
        }
        o0[q] = pack_kept(v0[0], v0[1]);
        o1[q] = pack_kept(v1[0], v1[1]);
    }
    if (tid == 0) {
        const uint32_t e1 = acc[1][m1], e2 = acc[1][m2];
        o0[N / 2] = x0 * e1 + y0 * e2 + (uint32_t)(a0 + a2) * (kMu >> 1);
        o1[N / 2] = x1 * e1 + y1 * e2 + (uint32_t)(b0 + b2) * (kMu >> 1);
    }
}

// After the blind rotation: the extracted sample(s) of gate g into its
// slot(s) of big; an invalid code gives all-zero samples (which key-switch
// to the all-zero output) and is reported through io.err.
template <int THREADS, int S>
__device__ __forceinline__ void gate_epilogue(const GateIO& io, uint32_t g, const uint32_t (&acc)[2][S],
                                              uint32_t* __restrict__ big, int tid) {
    const GateMode m = gate_mode(io, g);
    uint32_t* o = big + (size_t)(io.pair_slots ? 2 * g : g) * kSampleWords;
    if (!m.valid) {
        const int words = (io.pair_slots ? 2 : 1) * kSampleWords;
        for (int j = tid; j < words; j += THREADS) o[j] = 0u;
        if (tid == 0 && io.err)
            __hip_atomic_store(io.err, 0x100u | (m.op0 & 0xFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    if (m.compound)
        compound_extract<THREADS>(acc, m.op0, m.op1, o, o + kSampleWords, tid);
    else
        sample_extract<THREADS>(acc, o, tid);
}

// ---------------------------------------------------------------------------
// Kernels.
// ---------------------------------------------------------------------------

// Gate linear combination + modulus switch, test-vector rotation, 500 CMux,
// sample extraction.  One wave per gate, WPB gates per block; the register
// budget allows two waves per SIMD.
template <int WPB>
__global__ __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_blind_rotate(
    DeviceKeys K, GateIO io, uint32_t* __restrict__ big, uint32_t count) {
    __shared__ BlockLds<WPB> S;
    load_twiddles<64 * WPB>(S, K.twf, K.twi);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t g = blockIdx.x * WPB + wave;
    if (g >= count) return;

    const int h = lane >> 5, t = lane & 31;
    uint32_t ab[8];
    const int bbar = gate_prologue(io, g, lane, ab);
    WaveLds W{S.acc[wave], S.tile[wave]};
    acc_init(W.acc, bbar, h, t, io.tv, gate_mu(io, g));
    wave_lds_sync();

    // Blind rotation.  abar_i = 0 would give D = 0 and leave ACC unchanged,
    // so every step runs unconditionally.
    const uint64_t* bk = K.bkd;
#pragma unroll 1
    for (int i = 0; i < NLWE; ++i) {
        const int ai = __builtin_amdgcn_readlane(ab[0], i & 63);
        cmux_step(W, ai, bk, S.twf, S.twi, lane);
        bk += 2 * 32 * 2 * 64;
        if ((i & 63) == 63) {
#pragma unroll
            for (int r = 0; r < 7; ++r) ab[r] = ab[r + 1];
        }
    }
    gate_epilogue<64>(io, g, W.acc, big, lane);
}

// The same computation with two waves per gate (one gate per block), for
// latency: wave w runs pass w of each CMux (digits of ACC_w, their forward
// NTTs and multiply-accumulate) concurrently; wave 0 then adds wave 1's
// partial sums, runs the inverse NTTs and updates ACC while wave 1 waits.
// The critical path of a CMux drops from two passes plus the inverse to one
// pass plus the inverse; the issued work stays the same.
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_blind_rotate_pair(
    DeviceKeys K, GateIO io, uint32_t* __restrict__ big, uint32_t count) {
    __shared__ PairLds S;
    load_twiddles<128>(S, K.twf, K.twi);
    const uint32_t g = blockIdx.x;
    if (g >= count) return;  // uniform over the block
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, h = lane >> 5, t = lane & 31;

    uint32_t ab[8];
    const int bbar = gate_prologue(io, g, lane, ab);
    if (wave == 0) acc_init(S.acc, bbar, h, t, io.tv, gate_mu(io, g));
    __syncthreads();

    const uint64_t* bk = K.bkd;
#pragma unroll 1
    for (int i = 0; i < NLWE; ++i) {
        const int ai = __builtin_amdgcn_readlane(ab[0], i & 63);
        uint64_t mac[32];
        if (wave == 0) {
            cmux_pass<0, false, true>(S.acc[0], S.tile[0][h], ai, bk, S.twf, lane, mac);
        } else {
            cmux_pass<1, false, true>(S.acc[1], S.tile[1][h], ai, bk, S.twf, lane, mac);
#pragma unroll
            for (int q = 0; q < 32; ++q) S.part[q][lane] = mac[q];
        }
        __syncthreads();  // part written; both waves done reading ACC
        if (wave == 0) {
#pragma unroll
            for (int q = 0; q < 32; ++q) mac[q] = gl::add(mac[q], S.part[q][lane]);
            cmux_finish(S.acc, S.tile[0][h], mac, S.twi, lane);
        }
        __syncthreads();  // ACC updated; part free
        bk += 2 * 32 * 2 * 64;
        if ((i & 63) == 63) {
#pragma unroll
            for (int r = 0; r < 7; ++r) ab[r] = ab[r + 1];
        }
    }
    gate_epilogue<128>(io, g, S.acc, big, threadIdx.x);
}

// Blind rotation with FFT products on eight wavefronts per gate, for batches
// that leave compute units with one gate (LEAN = false: one gate 1.42 ms, 256
// gates 1.47 ms) or two (LEAN: 512 gates 2.72 ms, 300 gates 2.56).  A step of
// one gate takes 6,700 cycles, a chain of LDS round trips and four barriers
// around 495 VALU per wave; two waves per SIMD fill each other's gaps.  With
// two gates LDS is busy 70% of the time, most of it writes (64 B per clock).
// Both exchanges of lane bits 3 to 0 through LDS: one gate 1.53 ms and 512 gates
// 3.08, where this form took 1.40 and 2.86 (bits 1 and 0 by moves as well, which
// need selects: 1.46 and 2.96).  The 128 KB of key
// per step and gate are 2,000 cycles of the vector memory path, so the loads
// are spread over the step: all in one place they cost 0.3 ms.  Four wavefronts
// per gate, one per row: 2.06 and 4.2 ms; two: 2.54 and 3.3.  The integer NTTs
// modulo two primes that these replace: 3.2 ms (one gate) and 4.6 (512).
// STEP: one CMux with K.bkn instead of the whole bootstrap, on the accumulator at
// big ([2][N], in place), rotated by `first`.
template <bool LEAN, bool STEP>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(LEAN ? 4 : 2, LEAN ? 4 : 2)))
void k_blind_rotate_narrow(DeviceKeys K, GateIO io, uint32_t* __restrict__ big, uint32_t first, uint32_t count) {
    __shared__ NarrowLds<LEAN> S;
    static_assert(!LEAN || 2 * sizeof(NarrowLds<LEAN>) <= 160 * 1024, "two gates per compute unit");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = wave >> 1, half = wave & 1;
    const int lane = threadIdx.x & 63, h = lane >> 5, t = lane & 31;
    const uint32_t g = first + blockIdx.x;
    if (!STEP && g >= count) return;  // uniform over the block
    NarrowTwiddles T;
    load_narrow_twiddles(S, T, K.roots, wave, half, lane);
    uint32_t ab[8];
    const int bbar = STEP ? 0 : gate_prologue(io, g, lane, ab);
    uint32_t (&acc)[2][kPad + 1024] = S.view();
    if (wave == 0) {
        if constexpr (STEP)
            for (int k = lane; k < 2 * N; k += 64) acc[k / N][k % N] = big[k];
        else
            acc_init(acc, bbar, h, t, io.tv, gate_mu(io, g));
        wave_lds_sync();
#pragma unroll
        for (int p = 0; p < 2; ++p) S.acc[p][lane] = 0u - acc[p][960 + lane];
    }
    const cd* key = K.bkn;
    cd ka[LEAN ? 2 : 4][4];
#pragma unroll
    for (int k = 0; k < 2; ++k) load_narrow_keys(ka[k], key, (row + k) & 3, row, half, lane);
    __syncthreads();
    if constexpr (STEP) {
        narrow_step(S, (int)first, key, key, ka, T, row, half, lane);
        for (int k = threadIdx.x; k < 2 * N; k += 512) big[k] = acc[k / N][k % N];
        return;
    }
#pragma unroll 1
    for (int b = 0; b < NLWE; b += 64) {
#pragma unroll 1
        for (int i = 0; i < 64 && b + i < NLWE; ++i) {
            const int ai = __builtin_amdgcn_readlane(ab[0], i);
            const cd* next = b + i + 1 < NLWE ? key + kKeyStep : key;
            narrow_step(S, ai, key, next, ka, T, row, half, lane);
            key = next;
        }
#pragma unroll
        for (int r = 0; r < 7; ++r) ab[r] = ab[r + 1];
    }
    gate_epilogue<512>(io, g, acc, big, threadIdx.x);
}

// Blind rotation with FFT products for wide batches: groups of four gates on
// four wavefronts.  Wave w extracts and finishes gate w, and in between holds
// a quarter of the spectrum of all four gates, so that each key value loaded
// serves four gates (a wave per gate would stream 128 KB of key per step and
// gate through a 64 B per clock cache, more than half the time of the
// arithmetic) and the multiply-add over the rows is a matrix product.  The f64
// matrix instructions run at the rate of the VALU and not beside it: they
// save exchanges, not arithmetic.
// Lane layouts (32 complex registers):
//   A: lane (polynomial hp or column c, t): registers (digit or half, q),
//      coefficient pair t + 32 q of gate w;
//   B: lane (row r or output o, b, gate n): registers t, node Q = 4 w + b of
//      the first four levels (block Q of 32 leaves).
// 512 = 16 x 32 points need one exchange between them, through LDS, first all
// real, then all imaginary parts (64 KB, so that two groups fit a compute
// unit): value (Q, r, n, t) in row 64 (Q / 4) + 16 r + 4 (Q % 4) + n, column t.
// Between the steps the accumulators are in registers and pass through the
// same LDS to be read rotated.
//
// Bound by issue: about 2,220 VALU (1,830 of them f64 at 4.6-5.1 cycles) and
// 128 matrix instructions of 16 cycles per wave and step, 12,500 of the 15,000
// cycles that a step takes per wave at two waves per SIMD; LDS is busy a third
// of the time, its writes (64 B per clock) most of it.  16,384 gates in 51 ms,
// 2,048 in 7.0 ms, 1,024 (one wave per SIMD) in 4.5 ms.  With a masked address
// and a sign of its own for each rotated word, and the first level in doubles:
// 2,310 VALU, 52.0 ms (with the reads spread among the arithmetic 53.7).  The
// integer NTTs modulo two 28-bit primes that this replaces issued 6,570 VALU per
// wave and step: 100, 12.5 and 8.1 ms.
constexpr int kRowBytes = 32 * 8 + 16;  // 16-byte skew: lanes of layout B read 16 rows at once

struct alignas(16) GroupLds {
    char buf[256 * kRowBytes];  // also the accumulators, each wave's in its own rows, during the extraction
    cd tabf[16][16];            // twiddle k of block Q (forward levels 5..9)
    cd tabi[32][16];            // inverse factor of coefficient t, block Q
};
static_assert(2 * sizeof(GroupLds) <= 160 * 1024, "two groups per compute unit");

// An accumulator polynomial to be read rotated by any amount at fixed offsets
// from one address: ACC, then -ACC.  (The skew sends the lanes' two polynomials
// to different banks.)
constexpr int kAccWords = 2 * N + 32;
static_assert(2 * kAccWords * 4 <= 64 * kRowBytes, "accumulators fit the wave's own rows");

constexpr int kStaged = 12;  // key loads of a step that go through LDS
constexpr int KW = 8;        // window of the others, in registers
static_assert(kStaged % 4 == 0 && kStaged * 1024 <= 64 * kRowBytes, "staged keys fit the wave's own rows");
// (The group kernel's only shared object starts at LDS address 0.)
static_assert(offsetof(GroupLds, buf) + 3 * 64 * kRowBytes + kStaged * 1024 <= 65536, "and below 64 KB of LDS");

// Starts the copy of 1 KB of key (the lanes' 16 bytes at byte offset `off`)
// from memory to LDS byte address `dst`, which must be below 64 KB (M0 holds
// its low 16 bits).  M0 is declared as written, so that no pass keeps a value of
// its own in it across the copy; it is a reserved register, which the compiler
// warns of because it would not save one either.  The compiler does not
// count the copy: the reader waits for every load (vmcnt(0)) before it reads the
// bytes.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_key_lds(const cd* __restrict__ src, uint32_t off, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 ::"s"(dst), "v"(off), "s"(src) : "m0", "memory");
}
#pragma clang diagnostic pop

// STEP: one CMux with K.bkc instead of the whole bootstrap, on four accumulators
// at big ([4][2][N], in place), rotated by `count`.
template <bool STEP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_blind_rotate_group(DeviceKeys K, GateIO io, uint32_t* __restrict__ big, uint32_t count) {
    __shared__ GroupLds S;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, h = lane >> 5, t = lane & 31;
    {
        const int Q = threadIdx.x & 15, f = threadIdx.x >> 4;  // twiddle f: level l, even node c = 2 d
        const int l = f == 0 ? 0 : f == 1 ? 1 : f < 4 ? 2 : f < 8 ? 3 : 4;
        const int d = f < 2 ? 0 : f - (1 << (l - 1));
        int s = 0;  // c_0 + 2 c_1 + ... of the l - 1 leading path bits
        for (int b = 0; b < l - 1; ++b) s |= ((d >> (l - 2 - b)) & 1) << b;
        const int n = 16 + 64 * fft::brv(Q, 4);
        S.tabf[f][Q] = K.roots[((n >> l) + (1024 >> l) * s) & 2047];
    }
    for (int k = threadIdx.x; k < 512; k += 256) {
        const int Q = k & 15, m = k >> 4;
        S.tabi[m][Q] = conj_root(K.roots, m * (1 + 4 * fft::brv(Q, 4)));
    }
    char* buf = S.buf;
    char* own = buf + 64 * kRowBytes * w;  // this wave's own rows
    uint32_t (&accl)[2][kAccWords] = *reinterpret_cast<uint32_t (*)[2][kAccWords]>(own);
    const uint32_t g = blockIdx.x * 4 + w;
    const bool live = STEP || g < count;  // a missing gate's wave still serves the others' spectrum
    uint32_t ab[8] = {}, acc[32] = {};
    if constexpr (STEP) {
#pragma unroll
        for (int e = 0; e < 32; ++e) acc[e] = big[(2 * w + h) * N + t + 32 * e];
    } else if (live) {
        const int bbar = gate_prologue(io, g, lane, ab);
        acc_init(accl, bbar, h, t, io.tv, gate_mu(io, g));
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < 32; ++e) acc[e] = accl[h][t + 32 * e];
    }
    __syncthreads();

    const int b = (lane >> 2) & 3;
    char* colA = buf + (32 * h + w) * kRowBytes + 8 * t;       // layout A: this lane's column
    char* rowB = buf + (64 * w + lane) * kRowBytes;            // layout B: this lane's row
    const cd* tf = &S.tabf[0][4 * w + b];
    const cd* ti = &S.tabi[0][4 * w + b];
    const cd* keyw = K.bkc + 64 * w;  // this wave's keys of the step
    const cd* key = keyw + lane;
    const uint32_t lane16 = 16 * lane;
    const uint32_t kslot = (uint32_t)(uintptr_t)(const lds_u32*)(const uint32_t*)own;
    const char* kread = own + 16 * lane;
    uint32_t* accw = &accl[h][t];
    auto col_at = [&](auto d, auto q) -> double& {
        constexpr int Q = decltype(q)::value;
        return *reinterpret_cast<double*>(colA + (64 * (Q >> 2) + 16 * decltype(d)::value + 4 * (Q & 3)) * kRowBytes);
    };
#pragma unroll 1
    for (int i = 0; i < (STEP ? 1 : NLWE); ++i) {
        const int ai = STEP ? (int)count : __builtin_amdgcn_readlane(ab[0], i & 63);
        cd x[2][16], y[32];
        // digits of D = X^ai ACC - ACC, both of each coefficient.  X^ai ACC is
        // the words of (ACC, -ACC) from (-ai) mod N on, or their negatives, for
        // every lane alike; the fences keep all reads ahead of the arithmetic.
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            accw[32 * e] = acc[e];
            accw[32 * e + N] = 0u - acc[e];
        }
        wave_lds_sync();
        {
            const uint32_t sgn = (uint32_t)((int32_t)((uint32_t)(-ai) << 21) >> 31), off = kDecompOffset - sgn;
            const uint32_t* rot = accw + (-ai & (N - 1));
            uint32_t v[32];
#pragma unroll
            for (int e = 0; e < 32; ++e) v[e] = rot[32 * e];
            sched_fence();
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint32_t z[4];  // top bit of each digit's field flipped: the signed 10-bit fields are the digits
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    z[q] = ((v[k + 8 * q] ^ sgn) + (off - acc[k + 8 * q])) ^ 0x80200000u;
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    int32_t g[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) g[q] = (int32_t)__builtin_amdgcn_sbfe((int32_t)z[q], 22 - 10 * d, 10);
                    // first level: (a, b) -> a +- b (1 + i) / sqrt 2, the sums in integers
                    constexpr double c = fft::kCos[8];
                    const double re = (double)g[0], im = (double)g[2];
                    const double br = (double)(g[1] - g[3]), bi = (double)(g[1] + g[3]);
                    x[d][k] = {__builtin_fma(c, br, re), __builtin_fma(c, bi, im)};
                    x[d][k + 8] = {__builtin_fma(-c, br, re), __builtin_fma(-c, bi, im)};
                }
            }
            sched_fence();
        }
        fft::forward_root<16, 1>(x[0]);
        fft::forward_root<16, 1>(x[1]);
        lds_barrier();  // every wave has read its accumulator
        static_for<0, 2>([&](auto d) { static_for<0, 16>([&](auto q) { col_at(d, q) = x[d][q].x; }); });
        lds_barrier();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const cd v = *reinterpret_cast<const cd*>(rowB + 16 * k);
            y[2 * k].x = v.x;
            y[2 * k + 1].x = v.y;
        }
        lds_barrier();
        static_for<0, 2>([&](auto d) { static_for<0, 16>([&](auto q) { col_at(d, q) = x[d][q].y; }); });
        lds_barrier();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const cd v = *reinterpret_cast<const cd*>(rowB + 16 * k);
            y[2 * k].y = v.x;
            y[2 * k + 1].y = v.y;
        }
        lds_barrier();  // every wave has read the imaginary parts
        // The multiply-add wants its 32 KB of key a memory latency (1,000
        // cycles under this load) early and has registers for eight of its 32
        // loads: the first twelve wait in the wave's own rows, idle until the
        // inverse exchange, while the transform runs (12 staged and a window
        // of 8: 13.65 ms at 4,096 gates; a window of 4 and none staged, 14.0;
        // all staged, 14.1; a window of 8 and none staged spills more, 14.8).
        // This form keeps nine registers in scratch; a step stores one word of
        // them and reads three.
#pragma unroll
        for (int k = 0; k < kStaged; ++k) load_key_lds(keyw + k * 256, lane16, kslot + 1024 * k);
        fft::forward_lane<32>(y, [&](auto k) { return tf[16 * decltype(k)::value]; });
        // out_o = sum over rows of K_(r, o) x_r, per leaf: matrix products of
        // 4 outputs x 4 rows x 4 gates, four leaves (b) per instruction
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        cd kr[KW];
#pragma unroll
        for (int k = 0; k < KW; ++k) kr[k] = key[(kStaged + k) * 256];
        sched_fence();
        static_for<0, 8>([&](auto C_) {
            constexpr int c = 4 * decltype(C_)::value;
            cd kb[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (c < kStaged) kb[k] = *reinterpret_cast<const cd*>(kread + 1024 * (c + k));
                else kb[k] = kr[(c + k - kStaged) % KW];
            }
            double re[4], im[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) re[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(kb[k].x, y[c + k].x, 0.0, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) im[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(kb[k].x, y[c + k].y, 0.0, 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) re[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(kb[k].y, y[c + k].y, re[k], 0, 0, 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) im[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(kb[k].y, y[c + k].x, im[k], 0, 0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                y[c + k] = {re[k], im[k]};
                if constexpr (c >= kStaged && c + KW < 32) kr[(c + k - kStaged) % KW] = key[(c + k + KW) * 256];
            }
            sched_fence();
        });
        keyw += kKeyStep;
        key += kKeyStep;
        fft::inverse_root<32>(y);
#pragma unroll
        for (int m = 1; m < 32; ++m) {
            const cd f = ti[16 * m];
            y[m] = {__builtin_fma(f.x, y[m].x, -(f.y * y[m].y)), __builtin_fma(f.x, y[m].y, f.y * y[m].x)};
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) *reinterpret_cast<cd*>(rowB + 16 * k) = {y[2 * k].x, y[2 * k + 1].x};
        lds_barrier();
        static_for<0, 2>([&](auto d) { static_for<0, 16>([&](auto q) { x[d][q].x = col_at(d, q); }); });
        lds_barrier();
#pragma unroll
        for (int k = 0; k < 16; ++k) *reinterpret_cast<cd*>(rowB + 16 * k) = {y[2 * k].y, y[2 * k + 1].y};
        lds_barrier();
        static_for<0, 2>([&](auto d) { static_for<0, 16>([&](auto q) { x[d][q].y = col_at(d, q); }); });
        fft::inverse_root<16>(x[0]);
        fft::inverse_root<16>(x[1]);
        static_for<0, 16>([&](auto q_) {
            constexpr int q = decltype(q_)::value;
            constexpr double cr = fft::cos32(q), ci = -fft::sin32(q);  // twist of coefficient pair t + 32 q
            uint32_t re[2], im[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const cd v = x[s][q];
                re[s] = fft::round_word(q == 0 ? v.x : __builtin_fma(cr, v.x, -(ci * v.y)));
                im[s] = fft::round_word(q == 0 ? v.y : __builtin_fma(cr, v.y, ci * v.x));
            }
            acc[q] += re[0] + (re[1] << 16);
            acc[q + 16] += im[0] + (im[1] << 16);
        });
        lds_barrier();  // every wave has read its imaginary parts
        if ((i & 63) == 63) {
#pragma unroll
            for (int r = 0; r < 7; ++r) ab[r] = ab[r + 1];
        }
    }
    if constexpr (STEP) {
#pragma unroll
        for (int e = 0; e < 32; ++e) big[(2 * w + h) * N + t + 32 * e] = acc[e];
        return;
    }
    if (!live) return;
#pragma unroll
    for (int e = 0; e < 32; ++e) accl[h][t + 32 * e] = acc[e];
    wave_lds_sync();
    gate_epilogue<64>(io, g, accl, big, lane);
}

// BK -> the FFT domain, scaled by 1/512 (the inverse transform's factor; a
// power of two, exact), in the kernels' layouts: one wave per polynomial (CMux i, row
// r, column c) transforms its low and its high signed half words.
//   bkn[i][r][o][leaf / 256][leaf % 4][leaf % 256 / 4] (k_blind_rotate_narrow);
//   bkc[i][leaf % 32][leaf / 128][16 r + 4 (leaf / 32 % 4) + o] (k_blind_rotate_group).
__global__ __launch_bounds__(kBlockThreads) void k_bk_prepare_fft(const uint32_t* __restrict__ bk, cd* __restrict__ bkc,
                                                                  cd* __restrict__ bkn, const cd* __restrict__ roots,
                                                                  uint32_t npolys) {
    __shared__ cd ex[kWavesPerBlock][kExSlots];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t poly = blockIdx.x * kWavesPerBlock + wave;
    if (poly >= npolys) return;
    LaneTwiddles T;
    load_forward_twiddles(T, roots, lane);
    const uint32_t i = poly / 8, r = (poly / 2) % 4, c = poly % 2;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        cd x[8];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t k = bk[(size_t)poly * N + lane + 64 * e];
            const int32_t lo = (int16_t)k, hi = (int32_t)(k - (uint32_t)lo) >> 16;
            const double v = s == 0 ? lo : hi;
            if (e < 8)
                x[e & 7].x = v;
            else
                x[e & 7].y = v;
        }
        fft512_forward(x, ex[wave], T, lane);
        const uint32_t o = 2 * c + s;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const cd v = {x[j].x * (1.0 / 512), x[j].y * (1.0 / 512)};
            const uint32_t leaf = 8 * lane + j;
            if (bkn) bkn[(size_t)i * kKeyStep + ((r * 4 + o) * 8 + 4 * (leaf / 256) + leaf % 4) * 64 + leaf % 256 / 4] = v;
            if (bkc) bkc[(size_t)i * kKeyStep + ((leaf % 32) * 4 + leaf / 128) * 64 + 16 * r + 4 * (leaf / 32 % 4) + o] = v;
        }
    }
}

// Key switching N -> n: out = (0, b') - sum_{i,j} KSK[i][j][d_ij], d_ij the
// j-th base-4 digit of the 16 bits kept of a'_i.
//
// As a matrix product on the int8 matrix cores: a gate's row of A holds, for
// each of the 8,192 digits and each value v = 1, 2, 3, the byte [d == v]; B
// holds the key-switching rows as four signed byte limbs per word
// (w = s0 + 2^8 s1 + 2^16 s2 + 2^24 s3 mod 2^32).  Each limb's sum is at most
// 8,192 * 128 = 2^20 in magnitude, exact in the 32-bit accumulators, and the
// limbs recombine modulo 2^32: the words are those of the row sums.  The
// product does four times the additions of the gathers it replaces, on units
// with 128 times the rate, and reads every key row once per 32 or 64 gates
// instead of once per use.
//
// One instruction multiplies 32 gates x 32 digits of one value v x 8 words (32
// limb columns, column 4 word + limb).  Its k order is lane half h, byte t:
// digit field at bit 8 (t / 4) + 2 (t % 4) of sample word 256 h + kc, so that a
// lane builds its A operand from one sample word: the flags of a value are
// bits 0, 2, 4, 6 of each byte, which a 24-bit product with 1 + 2^6 + 2^12 +
// 2^18 spreads to the low bits of four bytes.  B is stored in operand order.
// A workgroup takes MT x 32 gates and NF x 8 words and splits the 256 steps kc
// over KW waves, whose sums meet in LDS.
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

template <int MT, int NF, int KW>
__global__ __launch_bounds__(64 * KW) void k_key_switch(DeviceKeys K, GateIO io, const uint32_t* __restrict__ big,
                                                        uint32_t count) {
    __shared__ uint32_t red[32 * MT][8 * NF];
    constexpr int kThreads = 64 * KW, kGates = 32 * MT, kSteps = 256 / KW;
    const int lane = threadIdx.x & 63, kw = threadIdx.x >> 6, h = lane >> 5;
    const uint32_t gate0 = blockIdx.x / (64 / NF) * kGates, frag0 = blockIdx.x % (64 / NF) * NF;
    for (int k = threadIdx.x; k < kGates * 8 * NF; k += kThreads) (&red[0][0])[k] = 0u;
    __syncthreads();

    const uint32_t* arow[MT];  // this lane's half of its gates' sample words
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const uint32_t g = gate0 + 32 * m + (lane & 31);
        arow[m] = big + (size_t)(g < count ? g : count - 1) * kSampleWords + 256 * h + kSteps * kw;
    }
    const v4i* bp = reinterpret_cast<const v4i*>(K.ksb) + ((size_t)frag0 * 256 + kSteps * kw) * 3 * 64 + lane;
    v16i acc[MT][NF];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][f][r] = 0;
    v4i bn[3][NF];
    auto load_b = [&](int kc) {
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int f = 0; f < NF; ++f) bn[v][f] = bp[((size_t)f * 256 + kc) * 192 + v * 64];
    };
    load_b(0);
#pragma unroll 1
    for (int kc = 0; kc < kSteps; kc += 4) {
        uint4 aw[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) aw[m] = *reinterpret_cast<const uint4*>(arow[m] + kc);
        static_for<0, 4>([&](auto U) {
            constexpr int u = decltype(U)::value;
            v4i b[3][NF];
#pragma unroll
            for (int v = 0; v < 3; ++v)
#pragma unroll
                for (int f = 0; f < NF; ++f) b[v][f] = bn[v][f];
            load_b(kc + u + 1 < kSteps ? kc + u + 1 : kc + u);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const uint32_t w = u == 0 ? aw[m].x : u == 1 ? aw[m].y : u == 2 ? aw[m].z : aw[m].w;
                const uint32_t lo = w & 0x55555555u, hi = (w >> 1) & 0x55555555u;
                const uint32_t both = lo & hi;
                const uint32_t flags[3] = {lo ^ both, hi ^ both, both};
#pragma unroll
                for (int v = 0; v < 3; ++v) {
                    v4i a;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        a[c] = (int)(__umul24((flags[v] >> (8 * c)) & 0xFFu, 0x41041u) & 0x01010101u);
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        acc[m][f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[v][f], acc[m][f], 0, 0, 0);
                }
            }
        });
    }

    // limbs of a word are in four neighbouring lanes: shift, add over the
    // quad, and lane `limb` adds the rows r with r % 4 == limb to LDS
    const int limb = lane & 3, word = (lane >> 2) & 7;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                uint32_t v = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    uint32_t x = (uint32_t)acc[m][f][4 * a + r] << (8 * limb);
                    x += (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
                    x += (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
                    v = limb == r ? x : v;
                }
                lds_add(&red[32 * m + 8 * a + 4 * h + limb][8 * f + word], v);
            }
    __syncthreads();
    for (int k = threadIdx.x; k < kGates * 8 * NF; k += kThreads) {
        const uint32_t g = gate0 + k / (8 * NF), w = 8 * frag0 + k % (8 * NF);
        if (g >= count || w >= NW) continue;
        uint32_t* o = ks_output(io, g);
        if (!o) continue;  // unused second slot of a single gate
        o[w] = (w == NLWE ? big[(size_t)g * kSampleWords + N / 2] : 0u) - (&red[0][0])[k];
    }
}

// KSK [N][t][4][501] -> operand B of k_key_switch, bytes
// [8-word group][kc][v][lane][t]: lane = 32 h + 4 word + limb, digit field at
// bit p = 8 (t / 4) + 2 (t % 4) of sample word 256 h + kc.
__global__ __launch_bounds__(256) void k_ksk_prepare(const uint32_t* __restrict__ ksk, uint8_t* __restrict__ ksb) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t block = blockIdx.x * 4 + (threadIdx.x >> 6);  // [group][kc][v]
    const uint32_t v = block % 3, kc = block / 3 % 256, group = block / 768;
    const uint32_t w = 8 * group + ((lane >> 2) & 7), limb = lane & 3, q = 256 * (lane >> 5) + kc;
    uint32_t out[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        uint32_t packed = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t p = 8 * c + 2 * b;
            const uint32_t i = 2 * q + (p >> 4), j = 7 - (p & 15) / 2;
            uint32_t x = w < NW ? ksk[((size_t)(i * kKsT + j) * kKsBase + v + 1) * NW + w] : 0u;
            for (uint32_t l = 0; l < limb; ++l) x = (x - (uint32_t)(int32_t)(int8_t)x) >> 8;
            packed |= (x & 0xFFu) << (8 * b);
        }
        out[c] = packed;
    }
    reinterpret_cast<uint4*>(ksb)[(size_t)block * 64 + lane] = make_uint4(out[0], out[1], out[2], out[3]);
}

// BK (uint32 [n][4][2][N]) -> NTT domain in the layout cmux_step reads:
// bkd[i][hp][q][sel][lane], lane = 32c + t, for row r = 2hp + digit, column c:
// sel = 0 when digit == c (the half's own digit), 1 otherwise.
__global__ __launch_bounds__(kBlockThreads) void k_bk_prepare(const uint32_t* __restrict__ bk,
                                                              uint64_t* __restrict__ bkd,
                                                              const uint64_t* __restrict__ twf,
                                                              uint32_t npolys) {
    __shared__ uint64_t stw[32 * 32];
    __shared__ uint32_t tiles[kWavesPerBlock][2][32 * 32];
    for (int k = threadIdx.x; k < 1024; k += kBlockThreads) stw[k] = twf[k];
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int h = lane >> 5, t = lane & 31;
    const uint32_t base = 2 * (blockIdx.x * kWavesPerBlock + wave);
    if (base >= npolys) return;
    const uint32_t poly = base + h;  // npolys is even
    uint64_t x[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) x[q] = gl::from_i64((int32_t)bk[(size_t)poly * N + t + 32 * q]);
    ntt1024_fwd(x, &tiles[wave][h][0], stw, t);
    const uint32_t i = poly / 8, r = (poly / 2) % 4, c = poly % 2;
    const uint32_t hp = r >> 1, digit = r & 1, sel = (digit == c) ? 0 : 1;
    uint64_t* dst = bkd + (size_t)i * (2 * 32 * 2 * 64) + (size_t)hp * (32 * 2 * 64) + 32 * c + t;
#pragma unroll
    for (int q = 0; q < 32; ++q) dst[(q * 2 + sel) * 64] = gl::canon(x[q]);
}

// One CMux on acc[2][N] in global memory with the NTT products (single wave).
__global__ __launch_bounds__(64) void k_debug_cmux(DeviceKeys K, const uint64_t* __restrict__ bk_i,
                                                   int32_t abar, uint32_t* __restrict__ accg) {
    __shared__ BlockLds<1> S;
    WaveLds W{S.acc[0], S.tile[0]};
    for (int k = threadIdx.x; k < 1024; k += 64) {
        S.twf[k] = K.twf[k];
        S.twi[k] = K.twi[k];
    }
    for (int k = threadIdx.x; k < 2 * N; k += 64) W.acc[k / N][k % N] = accg[k];
    __syncthreads();
    cmux_step(W, abar, bk_i, S.twf, S.twi, threadIdx.x);
    __syncthreads();
    for (int k = threadIdx.x; k < 2 * N; k += 64) accg[k] = W.acc[k / N][k % N];
}

// Issue-rate probe of one VALU instruction class (the roofline's peak per
// class): every lane runs 16 independent chains of the instruction (eight
// for the swap, which writes two registers), 64 instructions per
// iteration.  Only arithmetic instructions, no memory access but the final
// store of each lane's sum into out[global thread index].
template <int OP>
__global__ __launch_bounds__(256) void k_valu_probe(uint32_t* __restrict__ out, int iters) {
    uint32_t a[16];
    uint64_t w[16];
    const uint32_t b = threadIdx.x * 3u + 1u, c = threadIdx.x ^ 5u;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        a[k] = threadIdx.x + k;
        w[k] = (uint64_t)threadIdx.x * (k + 1);
    }
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                if constexpr (OP == 0) asm volatile("v_add_u32 %0, %0, %1" : "+v"(a[k]) : "v"(b));
                if constexpr (OP == 1) asm volatile("v_mul_lo_u32 %0, %0, %1" : "+v"(a[k]) : "v"(b));
                if constexpr (OP == 2)
                    asm volatile("v_mad_i64_i32 %0, vcc, %1, %2, %0" : "+v"(w[k]) : "v"(b), "v"(c) : "vcc");
                if constexpr (OP == 3) asm volatile("v_mul_hi_u32 %0, %0, %1" : "+v"(a[k]) : "v"(b));
                if constexpr (OP == 4) asm volatile("v_bfe_i32 %0, %0, %1, 10" : "+v"(a[k]) : "v"(c));
                if constexpr (OP == 5)  // eight disjoint register pairs, each swapped twice per pass
                    asm volatile("v_permlane32_swap_b32 %0, %1" : "+v"(a[k & 7]), "+v"(a[8 + (k & 7)]));
            }
        }
    }
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += a[k] + (uint32_t)w[k] + (uint32_t)(w[k] >> 32);
    out[blockIdx.x * blockDim.x + threadIdx.x] = sum;
}

}  // namespace

hipError_t launch_valu_probe(int op, uint32_t* out, uint32_t blocks, int iters, hipStream_t s) {
    switch (op) {
    case 0: hipLaunchKernelGGL(k_valu_probe<0>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case 1: hipLaunchKernelGGL(k_valu_probe<1>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case 2: hipLaunchKernelGGL(k_valu_probe<2>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case 3: hipLaunchKernelGGL(k_valu_probe<3>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case 4: hipLaunchKernelGGL(k_valu_probe<4>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case 5: hipLaunchKernelGGL(k_valu_probe<5>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_bk_prepare(const uint32_t* bk, uint64_t* bkd, const uint64_t* twf,
                             uint32_t n_lwe, hipStream_t s) {
    const uint32_t npolys = n_lwe * 8;
    const uint32_t waves = npolys / 2;
    const uint32_t blocks = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
    hipLaunchKernelGGL(k_bk_prepare, dim3(blocks), dim3(kBlockThreads), 0, s, bk, bkd, twf, npolys);
    return hipGetLastError();
}

// How many gates at the end of a wide batch of `count` run on the narrow kernel
// after the groups.  Groups fill the chip in rounds of eight gates per compute
// unit; a last round of up to four per unit still takes 4.4 ms and one of more
// 7.0 ms, and leaves most of the chip idle when it is short.  The narrow kernel
// does one gate per unit in 1.5 ms and two in 2.7 (256 units; blind rotation, ms,
// all groups / with a tail):
//   rest up to 2 per unit:     2,049 gates 11.3 / 8.9, 2,560 gates 11.0 / 9.7,
//                              16,385 gates 56.2 / 53.5
//   rest over 4, to 5 per unit: 1,025 to 1,280 gates 7.1 / 5.9
// With three per unit the narrow kernel takes 4.26 ms itself and with four 5.35,
// and past 5 per unit the two parts (4.4 + 2.7) take as long as one round.
static uint32_t narrow_tail(uint32_t count, uint32_t cus) {
    const uint32_t rest = count % (8 * cus);
    if (count > rest && rest <= 2 * cus) return rest;
    if (rest > 4 * cus && rest <= 5 * cus) return rest - 4 * cus;
    return 0;
}

hipError_t launch_blind_rotate(const DeviceKeys& K, const GateIO& io, uint32_t* big,
                               uint32_t count, LaunchConfig cfg, uint32_t cus, hipStream_t s) {
    if (count == 0) return hipSuccess;
    auto launch = [&](auto kernel, uint32_t gates, uint32_t threads) {
        hipLaunchKernelGGL(kernel, dim3((count + gates - 1) / gates), dim3(threads), 0, s, K, io, big, count);
        return hipGetLastError();
    };
    // gates first .. count - 1, one per block
    auto launch_narrow = [&](uint32_t first, bool lean) {
        const dim3 grid(count - first), block(512);
        if (lean)
            hipLaunchKernelGGL((k_blind_rotate_narrow<true, false>), grid, block, 0, s, K, io, big, first, count);
        else
            hipLaunchKernelGGL((k_blind_rotate_narrow<false, false>), grid, block, 0, s, K, io, big, first, count);
        return hipGetLastError();
    };
    if (cfg.arith == 1) {
        switch (cfg.waves_per_gate) {
        // groups of four gates, whatever cfg.gates_per_group (a wave per gate, which
        // shares no key loads, was dropped: 18.7 ms for one gate, a group 4.4)
        case 1: {
            const uint32_t tail = narrow_tail(count, cus);
            if (tail) {
                hipLaunchKernelGGL(k_blind_rotate_group<false>, dim3((count - tail) / 4), dim3(256), 0, s, K, io, big,
                                   count - tail);
                const hipError_t e = hipGetLastError();
                return e == hipSuccess ? launch_narrow(count - tail, tail > cus) : e;
            }
            return launch(k_blind_rotate_group<false>, 4, 256);
        }
        case 2: return launch_narrow(0, true);
        case 4: return launch_narrow(0, false);
        default: return hipErrorInvalidValue;
        }
    }
    if (cfg.arith != 0) return hipErrorInvalidValue;
    if (cfg.waves_per_gate == 2) return launch(k_blind_rotate_pair, 1, 128);
    if (cfg.waves_per_gate != 1) return hipErrorInvalidValue;
    switch (cfg.gates_per_group) {
    case 1: return launch(k_blind_rotate<1>, 1, 64);
    case 2: return launch(k_blind_rotate<2>, 2, 128);
    case 4: return launch(k_blind_rotate<4>, 4, 256);
    case 8: return launch(k_blind_rotate<8>, 8, 512);
    default: return hipErrorInvalidValue;
    }
}

template <int MT, int NF, int KW>
static hipError_t launch_key_switch_shape(const DeviceKeys& K, const GateIO& io, const uint32_t* big, uint32_t count,
                                          hipStream_t s) {
    constexpr uint32_t gates = 32 * MT;
    hipLaunchKernelGGL((k_key_switch<MT, NF, KW>), dim3(64 / NF * ((count + gates - 1) / gates)), dim3(64 * KW), 0, s,
                       K, io, big, count);
    return hipGetLastError();
}

hipError_t launch_key_switch(const DeviceKeys& K, const GateIO& io, const uint32_t* big,
                             uint32_t count, hipStream_t s) {
    if (count == 0) return hipSuccess;
    // Few gates: every workgroup streams its columns of B once, so more and
    // narrower column groups (and fewer gates per instruction) fill more
    // compute units.  Many gates: more columns per workgroup share the A
    // operands, which cost 41 VALU per 3 x 4 operand words.  us per launch at
    // 128 / 256 / 512 / 1,024 / 16,384 gates (the row gathers this replaces:
    // 145 / 145 / 280 / 440 / 8,500):
    //   <1, 1, 16>  18 / 31 / 56 / 106 / 1,609
    //   <2, 1, 16>  23 / 24 / 43 /  80 / 1,187
    //   <2, 2, 16>  30 / 30 / 34 /  65 /   918
    //   <2, 4,  8>  49 / 47 / 48 /  56 /   808   (0.41 of the int8 rate)
    // Four waves on four gate groups that share B through L1 instead of the
    // split over steps: 998 at 16,384.  (<2, 2, 16> keeps one register in scratch.)
    if (count <= 128) return launch_key_switch_shape<1, 1, 16>(K, io, big, count, s);
    if (count <= 256) return launch_key_switch_shape<2, 1, 16>(K, io, big, count, s);
    if (count <= 512) return launch_key_switch_shape<2, 2, 16>(K, io, big, count, s);
    return launch_key_switch_shape<2, 4, 8>(K, io, big, count, s);
}

hipError_t launch_ksk_prepare(const uint32_t* ksk, uint8_t* ksb, hipStream_t s) {
    hipLaunchKernelGGL(k_ksk_prepare, dim3(64 * 256 * 3 / 4), dim3(256), 0, s, ksk, ksb);
    return hipGetLastError();
}

hipError_t launch_debug_cmux(const DeviceKeys& K, LaunchConfig cfg, int32_t abar, uint32_t* acc, hipStream_t s) {
    const GateIO io{};
    const uint32_t ai = (uint32_t)abar;
    if (cfg.arith == 0)
        hipLaunchKernelGGL(k_debug_cmux, dim3(1), dim3(64), 0, s, K, K.bkd, abar, acc);
    else if (cfg.waves_per_gate == 1)
        hipLaunchKernelGGL(k_blind_rotate_group<true>, dim3(1), dim3(256), 0, s, K, io, acc, ai);
    else if (cfg.waves_per_gate == 2)
        hipLaunchKernelGGL((k_blind_rotate_narrow<true, true>), dim3(1), dim3(512), 0, s, K, io, acc, ai, 0u);
    else
        hipLaunchKernelGGL((k_blind_rotate_narrow<false, true>), dim3(1), dim3(512), 0, s, K, io, acc, ai, 0u);
    return hipGetLastError();
}

hipError_t launch_bk_prepare_fft(const uint32_t* bk, fft::cd* bkc, fft::cd* bkn, const fft::cd* roots,
                                 uint32_t n_lwe, hipStream_t s) {
    const uint32_t npolys = n_lwe * 8;
    const uint32_t blocks = (npolys + kWavesPerBlock - 1) / kWavesPerBlock;
    hipLaunchKernelGGL(k_bk_prepare_fft, dim3(blocks), dim3(kBlockThreads), 0, s, bk, bkc, bkn, roots, npolys);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace fhe
