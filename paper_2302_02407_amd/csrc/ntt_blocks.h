// Register blocks of the radix-2 negacyclic transforms shared by the two-launch kernels, the column conversion and the small-ring kernels:
// four butterfly stages on 16 points, or two on 4 points, held by one thread (Harvey butterflies, lazy ranges).
#pragma once
#include <type_traits>

#include "modarith.h"

#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)   // loads above it are issued before the arithmetic below it

// A butterfly is counted in instructions: on gfx950 the 32-bit multiplies, multiply-adds, v_lshl_add_u64, carries and the FP64 instructions all
// issue at one per lane and cycle, and what other instructions there are among them at the same, so what costs is how many there are.  A wavefront by
// itself issues one in five cycles; a scalar instruction between two vector ones costs it some 20 more, a wait state 4.  The product
// enters the sum through the multiply-adds' own addend (X + w*Y - h*2q accumulated in one chain), and the difference is
// 2X + 5q minus that sum: two instructions for the quotient h, 7 for the sum (split_acc), 3 for the difference, and 3 for a factor's second
// word where it is not the same for the whole wavefront (scalar instructions there).  With a quotient of two words it were 16, a
// product formed on its own and then added and subtracted takes 20.  (tests/test_butterfly_instructions.py counts them.)
//
// Ranges are kept in units of q and known when the code is compiled: a product is below 5q whatever its factor, a forward stage therefore
// adds that to the bound of every point, an inverse stage doubles it.  What multiplies a factor has to stay
// below 2^63.  Classes of moduli, a template parameter W of everything here, one for each direction (he_internal.h):
//   0  narrow: never reduced.  Forward: 17 stages from below 5q end below 90q; inverse: a pass ends below 640q.
//   1  up to 2^63 / 13: points stay below 13q, which takes one conditional subtraction of two instructions (csub_min) a forward butterfly.
//   2  the others (below 2^60): below 8q, two of them.
//   3  W_NEAR, moduli near a multiple of 2^32 (near_acc, modarith.h): signed points, never reduced.  Forward: below 22q at the end (16q above 2^58),
//      NEAR_ROWS between the passes; inverse: a pass ends below 512q.  What they need at the start: he_internal.h.
#define NEAR_ROWS 14
// multiples of q that make any forward result positive, which together stay below 2^64
__device__ __forceinline__ u64 near_bias(u64 q) { return q * (q > 1ull << 58 ? 16 : 24); }
__device__ constexpr int w_lim(int W) { return W == W_NEAR ? NEAR_ROWS : W == 1 ? 13 : 8; }         // sums and products' operands (W > 0)
__device__ constexpr int w_half(int W) { return w_lim(W) / 2; }            // inverse: points between stages (W = 1, 2)
__device__ constexpr int w_start(int W) { return W == 1 || W == 2 ? w_half(W) : 2; }      // inverse: what a pass starts with
// f(std::integral_constant<int, W>, v) for the class W of bits `mi` of c; v: what the loads of a class follow from.  Keeps the loads of the
// branches apart: merged above them (they look alike) they would stay live across all of it, 240 registers instead of 109.  (A chain of
// branches: on the class as one number the compiler makes a tree of them, with ten registers more in the rescale's columns.)
template <class F>
__device__ __forceinline__ void by_class(const ModClasses& c, uint32_t mi, uint32_t v, F&& f) {
    if ((c.b[0] & c.b[1]) >> mi & 1u) {
        asm("; near" : "+s"(v));
        f(std::integral_constant<int, W_NEAR>(), v);
    } else if (!((c.b[0] | c.b[1]) >> mi & 1u)) {
        asm("; narrow" : "+s"(v));
        f(std::integral_constant<int, 0>(), v);
    } else if (!(c.b[1] >> mi & 1u)) {
        asm("; wide" : "+s"(v));
        f(std::integral_constant<int, 1>(), v);
    } else {
        asm("; widest" : "+s"(v));
        f(std::integral_constant<int, 2>(), v);
    }
}
// what the butterflies need of a modulus, in scalar registers
struct StageQ {
    u64 n2q, q5;
    __device__ __forceinline__ explicit StageQ(u64 q) : n2q(opaque_s(0 - 2 * q)), q5(opaque_s(5 * q)) {}
};
// x < b*q to below half of that, rounded up
__device__ __forceinline__ void halve(u64& x, int& b, u64 q) {
    const int h = (b + 1) / 2;
    x = csub_min(x, q * (u64)h);
    b = h;
}
// Two butterflies of a near modulus, with a factor each
template <bool UNI>
__device__ __forceinline__ void ct_near2(u64& x0, u64& y0, ulonglong2 f0, u64& x1, u64& y1, ulonglong2 f1, const NearQ& n) {
    u64 s0, s1;
    near_acc2<UNI>(s0, x0, y0, f0, s1, x1, y1, f1, n);
    y0 = (x0 << 1) - s0;
    y1 = (x1 << 1) - s1;
    x0 = s0;
    x1 = s1;
}
template <bool UNI>
__device__ __forceinline__ void gs_near2(u64& x0, u64& y0, ulonglong2 f0, u64& x1, u64& y1, ulonglong2 f1, const NearQ& n) {
    u64 d0, d1;
    sub2(d0, x0, y0, d1, x1, y1);
    x0 = x0 + y0;
    x1 = x1 + y1;
    near_acc2<UNI, true>(y0, 0, d0, f0, y1, 0, d1, f1, n);
}
// One factor on K pairs of points X(k), Y(k) below b*q; returns the bound of the results.
template <int W, bool UNI, int K, class PX, class PY>
__device__ __forceinline__ int ct_stage(int b, PX&& X, PY&& Y, u64 w, u64 a, u64 q) {
    if constexpr (W == W_NEAR) {
        const NearQ n(q);
#pragma unroll
        for (int k = 0; k + 1 < K; k += 2) ct_near2<UNI>(X(k), Y(k), make_ulonglong2(w, a), X(k + 1), Y(k + 1), make_ulonglong2(w, a), n);
        static_assert(K % 2 == 0, "");
        return b + 1;
    }
    const StageQ sq(q);
    const u64 wh = split_factor<UNI>(w, a, sq.n2q);
    int after = b;
#pragma unroll
    for (int k = 0; k < K; k++) {
        u64 &x = X(k), &y = Y(k);
        int bx = b;
#pragma unroll
        for (int r = 0; r < 2; r++) if (W && bx + 5 > w_lim(W)) halve(x, bx, q);
        // The compiler puts what comes out of an instruction it does not know last in a sum: a halved x was added behind the multiply-adds, in an
        // instruction of its own, unless y passes one later.  384 limbs forward, N = 2^16: 57-bit primes 149 -> 144 us, just below 2^60 158 -> 154.
        if (bx < b) asm("" : "+v"(y));
        const u64 S = split_acc(x, y, w, a, wh, sq.n2q);
        y = (x + x + sq.q5) - S;
        x = S;
        after = bx + 5;
    }
    return after;
}
// Inverse butterflies of one factor on K pairs of points below b*q; returns the bound of the results.  Wide moduli: twice the bound of what
// goes in stays within w_lim, so sums (and, of the widest, products) are halved where the next stage would leave it.
template <int W, bool UNI, int K, class PX, class PY>
__device__ __forceinline__ int gs_stage(int b, PX&& X, PY&& Y, u64 w, u64 a, u64 q) {
    if constexpr (W == W_NEAR) {
        const NearQ n(q);
#pragma unroll
        for (int k = 0; k + 1 < K; k += 2) gs_near2<UNI>(X(k), Y(k), make_ulonglong2(w, a), X(k + 1), Y(k + 1), make_ulonglong2(w, a), n);
        static_assert(K % 2 == 0, "");
        return 2 * b;
    }
    const StageQ sq(q);
    const u64 wh = split_factor<UNI>(w, a, sq.n2q);
    int after = b;
#pragma unroll
    for (int k = 0; k < K; k++) {
        u64 &x = X(k), &y = Y(k);
        int bx = 2 * b, by = 5;
        const u64 d = (x + q * (u64)b) - y;
        x = x + y;
        y = split_acc(0, d, w, a, wh, sq.n2q);
        if (W && 2 * bx > w_lim(W)) halve(x, bx, q);
        if (W && 2 * by > w_lim(W)) halve(y, by, q);
        after = bx > by ? bx : by;
    }
    return after;
}

// a pointer to constant memory, which no store can change: loads through it stay scalar after stores and after ieee_off()
typedef const __attribute__((address_space(4))) u64* const_u64;
// a modulus' constants, in scalar registers
__device__ __forceinline__ ModConst mod_const(const ModConst* mc, uint32_t mi) {
    const const_u64 p = (const_u64)(uintptr_t)uni64((u64)(mc + mi));
    ModConst m = {};
    m.q = p[offsetof(ModConst, q) / 8];
    m.mu = p[offsetof(ModConst, mu) / 8];
    m.ninv = p[offsetof(ModConst, ninv) / 8];
    m.ninv_sh = p[offsetof(ModConst, ninv_sh) / 8];
    m.ninv_w = p[offsetof(ModConst, ninv_w) / 8];
    m.ninv_w_sh = p[offsetof(ModConst, ninv_w_sh) / 8];
    m.near_s = p[offsetof(ModConst, near_s) / 8];
    m.near_s_sh = p[offsetof(ModConst, near_s_sh) / 8];
    m.near_w = p[offsetof(ModConst, near_w) / 8];
    m.near_w_sh = p[offsetof(ModConst, near_w_sh) / 8];
    m.one_sh = p[offsetof(ModConst, one_sh) / 8];
    const u64 v = p[offsetof(ModConst, bits) / 8];
    m.bits = (uint32_t)v; m.rec = (uint32_t)(v >> 32);
    return m;
}
// Results of a forward transform (W_NEAR: signed) as positive numbers below 2^7 q
template <int W>
__device__ __forceinline__ u64 fwd_positive(u64 x, u64 q) { return W == W_NEAR ? x + near_bias(q) : x; }
// Results where the caller takes them below 2q of narrow moduli and canonical of others (q or 0 is taken off: no branch between the points)
template <int W>
__device__ __forceinline__ u64 fwd_lazy(u64 x, const ModConst& m) {
    const u64 v = reduce_lazy<7>(fwd_positive<W>(x, m.q), m.q, m.bits, m.rec);
    return W == W_NEAR ? csub_min(v, m.q > (1ull << 63) / 96 ? m.q : 0) : v;
}
// Points of up to 2^7 q for the first forward pass of a modulus that needs them centred, below q in magnitude
template <int W, int N>
__device__ __forceinline__ void fwd_centre(u64 (&x)[N], const ModConst& m) {
    if (W != W_NEAR || m.q <= 1ull << 58) return;
#pragma unroll
    for (int k = 0; k < N; k++) x[k] = reduce_lazy<7>(x[k], m.q, m.bits, m.rec) - m.q;
}
// What an inverse pass ends with, below 2q (narrow and near moduli)
template <int W>
__device__ __forceinline__ u64 inv_end(u64 x, const ModConst& m) { return reduce_lazy<10>(W == W_NEAR ? x + (m.q << 9) : x, m.q, m.bits, m.rec); }

// The last inverse stage's products, which carry the output scaling (any operand an inverse pass has), and what makes them canonical.
template <int W>
__device__ __forceinline__ u64 inv_scaled(u64 y, u64 w, u64 w_sh, u64 q) { return W == W_NEAR ? near_acc<true>(q, y, make_ulonglong2(w, w_sh), NearQ(q)) : shoup_lazy4(y, w, w_sh, q); }
template <int W>
__device__ __forceinline__ u64 inv_canonical(u64 x, u64 q) { return W == W_NEAR ? csub_min(x, q) : csub_min(csub_min(x, 2 * q), q); }
// Whether a forward transform's results go into a ModDown's difference (accumulator below 6q, less the result, plus the bias, below 2^63) as they are
template <int W>
__device__ __forceinline__ bool fwd_raw(const ModConst& m) { return (W == 0 && m.bits <= 55) || (W == W_NEAR && m.bits <= 57); }
template <int W>
__device__ __forceinline__ u64 fwd_raw_bias(u64 q) { return W == W_NEAR ? near_bias(q) : q << 7; }

// Register blocks of four stages on 16 points.  Stage u pairs (k, k + (8>>u)); the twiddle of the pair's group g =
// k >> (4-u) is tw[(1 << (s0+u)) + (G << u) + g], G = group of the 16 points at stage s0, kept at index (1 << u) - 1 + g.
// A factor and its companion lie next to each other, one 16-byte load.  Loading is separate from use: a pass that
// fetched its factors where it needs them spent 40 of 104 us (row pass, 384 limbs) waiting for them.
template <int U0, int U1>
__device__ __forceinline__ void tw_load(ulonglong2 (&w)[15], const ulonglong2* __restrict__ tw, uint32_t s0, uint32_t G) {
#pragma unroll
    for (int u = U0; u < U1; u++) {
        const ulonglong2* p = tw + ((1u << (s0 + u)) + (G << u));
#pragma unroll
        for (int g = 0; g < (1 << u); g++) w[(1 << u) - 1 + g] = p[g];
    }
}
// The same through constant memory: scalar loads where s0 and G are the same for the wavefront.
typedef u64 v2u64 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) v2u64* ctw_t;
template <int U0, int U1>
__device__ __forceinline__ void tw_load_c(ulonglong2 (&w)[15], ctw_t tw, uint32_t s0, uint32_t G) {
#pragma unroll
    for (int u = U0; u < U1; u++) {
        ctw_t p = tw + ((1u << (s0 + u)) + (G << u));
#pragma unroll
        for (int g = 0; g < (1 << u); g++) { const v2u64 v = p[g]; w[(1 << u) - 1 + g] = make_ulonglong2(v.x, v.y); }
    }
}
// The same for the last four stages of the two-launch transforms, whose tables keep one factor of every group after the
// other (ctx.hip, tw_pos); G of 2^s0 groups.
template <int U0, int U1>
__device__ __forceinline__ void tw_load_last(ulonglong2 (&w)[15], const ulonglong2* __restrict__ tw, uint32_t s0, uint32_t G) {
    tw += (1u << s0) + G;
#pragma unroll
    for (int u = U0; u < U1; u++)
#pragma unroll
        for (int g = 0; g < (1 << u); g++) w[(1 << u) - 1 + g] = tw[(size_t)((1u << u) - 1u + g) << s0];
}
// Forward stages U0 .. U1-1 on points below b*q, the bound of the results replaces it; UNI: the factors are the same for the whole
// wavefront.
template <int W, int U0, int U1, bool UNI = false>
__device__ __forceinline__ void fwd_stages(u64 (&x)[16], const ulonglong2 (&w)[15], u64 q, int& b) {
#pragma unroll
    for (int u = U0; u < U1; u++) {
        const int dist = 8 >> u;
        int after = b;
#pragma unroll
        for (int g = 0; g < (1 << u); g++) {
            const ulonglong2 f = w[(1 << u) - 1 + g];
            auto X = [&](int k) -> u64& { return x[g * 2 * dist + k]; };
            auto Y = [&](int k) -> u64& { return x[g * 2 * dist + dist + k]; };
            if (u == 0) after = ct_stage<W, UNI, 8>(b, X, Y, f.x, f.y, q);
            else if (u == 1) after = ct_stage<W, UNI, 4>(b, X, Y, f.x, f.y, q);
            else if (u == 2) after = ct_stage<W, UNI, 2>(b, X, Y, f.x, f.y, q);
            else if constexpr (W != W_NEAR) after = ct_stage<W, UNI, 1>(b, X, Y, f.x, f.y, q);
            else if (g & 1) {                            // two factors at a time
                const ulonglong2 e = w[(1 << u) - 2 + g];
                ct_near2<UNI>(x[2 * g - 2], x[2 * g - 1], e, x[2 * g], x[2 * g + 1], f, NearQ(q));
                after = b + 1;
            }
        }
        b = after;
    }
}
// Inverse stages U1-1 down to U0, likewise.
template <int W, int U0, int U1, bool UNI = false>
__device__ __forceinline__ void inv_stages(u64 (&x)[16], const ulonglong2 (&w)[15], u64 q, int& b) {
#pragma unroll
    for (int u = U1 - 1; u >= U0; u--) {
        const int dist = 8 >> u;
        int after = b;
#pragma unroll
        for (int g = 0; g < (1 << u); g++) {
            const ulonglong2 f = w[(1 << u) - 1 + g];
            auto X = [&](int k) -> u64& { return x[g * 2 * dist + k]; };
            auto Y = [&](int k) -> u64& { return x[g * 2 * dist + dist + k]; };
            if (u == 0) after = gs_stage<W, UNI, 8>(b, X, Y, f.x, f.y, q);
            else if (u == 1) after = gs_stage<W, UNI, 4>(b, X, Y, f.x, f.y, q);
            else if (u == 2) after = gs_stage<W, UNI, 2>(b, X, Y, f.x, f.y, q);
            else if constexpr (W != W_NEAR) after = gs_stage<W, UNI, 1>(b, X, Y, f.x, f.y, q);
            else if (g & 1) {                            // two factors at a time
                const ulonglong2 e = w[(1 << u) - 2 + g];
                gs_near2<UNI>(x[2 * g - 2], x[2 * g - 1], e, x[2 * g], x[2 * g + 1], f, NearQ(q));
                after = 2 * b;
            }
        }
        b = after;
    }
}

// Two forward / inverse stages on 4 register points of NX rows (same pairing and twiddle indexing as the 16-point blocks), factors
// r = {w0, a0, w1, a1, w2, a2}.  ONE: only the first of the two stages.
template <int W, bool UNI, int NX, bool ONE = false>
__device__ __forceinline__ void fwd_block2_x(u64 (&x)[NX][4], const u64 (&r)[6], u64 q, int& b) {
    b = ct_stage<W, UNI, 2 * NX>(b, [&](int k) -> u64& { return x[k >> 1][k & 1]; }, [&](int k) -> u64& { return x[k >> 1][2 + (k & 1)]; }, r[0], r[1], q);
    if (ONE) return;
    if constexpr (W == W_NEAR) {
#pragma unroll
        for (int c = 0; c < NX; c++) ct_near2<UNI>(x[c][0], x[c][1], make_ulonglong2(r[2], r[3]), x[c][2], x[c][3], make_ulonglong2(r[4], r[5]), NearQ(q));
        b += 1;
    } else {
        const int after = ct_stage<W, UNI, NX>(b, [&](int k) -> u64& { return x[k][0]; }, [&](int k) -> u64& { return x[k][1]; }, r[2], r[3], q);
        ct_stage<W, UNI, NX>(b, [&](int k) -> u64& { return x[k][2]; }, [&](int k) -> u64& { return x[k][3]; }, r[4], r[5], q);
        b = after;
    }
}
template <int W, bool UNI, int NX, bool ONE = false>
__device__ __forceinline__ void inv_block2_x(u64 (&x)[NX][4], const u64 (&r)[6], u64 q, int& b) {
    if constexpr (!ONE && W == W_NEAR) {
#pragma unroll
        for (int c = 0; c < NX; c++) gs_near2<UNI>(x[c][0], x[c][1], make_ulonglong2(r[2], r[3]), x[c][2], x[c][3], make_ulonglong2(r[4], r[5]), NearQ(q));
        b *= 2;
    } else if constexpr (!ONE) {
        const int after = gs_stage<W, UNI, NX>(b, [&](int k) -> u64& { return x[k][0]; }, [&](int k) -> u64& { return x[k][1]; }, r[2], r[3], q);
        gs_stage<W, UNI, NX>(b, [&](int k) -> u64& { return x[k][2]; }, [&](int k) -> u64& { return x[k][3]; }, r[4], r[5], q);
        b = after;
    }
    b = gs_stage<W, UNI, 2 * NX>(b, [&](int k) -> u64& { return x[k >> 1][k & 1]; }, [&](int k) -> u64& { return x[k >> 1][2 + (k & 1)]; }, r[0], r[1], q);
}
template <int W, bool UNI = false, bool ONE = false>
__device__ __forceinline__ void fwd_block2_r(u64 (&x)[4], const u64 (&r)[6], u64 q, int& b) {
    fwd_block2_x<W, UNI, 1, ONE>(reinterpret_cast<u64 (&)[1][4]>(x), r, q, b);
}
template <int W, bool UNI = false, bool ONE = false>
__device__ __forceinline__ void inv_block2_r(u64 (&x)[4], const u64 (&r)[6], u64 q, int& bound) {
    inv_block2_x<W, UNI, 1, ONE>(reinterpret_cast<u64 (&)[1][4]>(x), r, q, bound);
}
// the three twiddles of such a block and their companions
__device__ __forceinline__ void tw_block2(u64 (&r)[6], const ulonglong2* tw, uint32_t s0, uint32_t G) {
    const uint32_t b0 = (1u << s0) + G, b1 = (2u << s0) + 2 * G;
    const ulonglong2 w0 = tw[b0], w1 = tw[b1], w2 = tw[b1 + 1];
    r[0] = w0.x; r[1] = w0.y; r[2] = w1.x; r[3] = w1.y; r[4] = w2.x; r[5] = w2.y;
}
// lanes of one wavefront exchange through LDS: its own accesses are in order, the compiler has to keep them so
__device__ __forceinline__ void wave_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Position in bit-reversed order that the Galois map X -> X^g takes the value of position j from.
__device__ __forceinline__ uint32_t galois_pos(uint32_t j, uint32_t g, uint32_t logN) {
    const uint32_t k = __brev(j) >> (32 - logN);
    const uint32_t kp = (g * k + ((g - 1) >> 1)) & ((1u << logN) - 1u);
    return __brev(kp) >> (32 - logN);
}

// ---------------------------------------------------------------- rows with 4 points per thread
// In the last block (four neighbours a lane) lane t takes points 4T .. 4T+3, T = row4_last(t): 16 lanes then read factors that lie
// side by side (tw_pos), where T = t made every quad of lanes read from four places.
__device__ __forceinline__ uint32_t row4_last(uint32_t t) { return ((t & 15u) << 2) | (t >> 4); }
// Factors of the four two-stage blocks of row b for thread t of 64 (b the same for the whole wavefront).
__device__ __forceinline__ void tw_row4(u64 (&w)[4][6], const ulonglong2* __restrict__ tw, uint32_t lc, uint32_t b, uint32_t t) {
    const uint32_t bu = __builtin_amdgcn_readfirstlane(b);
    const const_u64 f0 = (const_u64)(uintptr_t)uni64((u64)(tw + ((1u << lc) + bu))), f1 = (const_u64)(uintptr_t)uni64((u64)(tw + ((2u << lc) + 2 * bu)));
    w[0][0] = f0[0]; w[0][1] = f0[1];                    // the same for the whole row (scalar registers)
#pragma unroll
    for (int i = 0; i < 4; i++) w[0][2 + i] = f1[i];
    tw_block2(w[1], tw, lc + 2, 4 * b + (t >> 4));
    const uint32_t NG = 1u << (lc + 4), T = row4_last(t), g = T & 3u;           // the last four stages' order: tw_pos
    const ulonglong2 *p = tw + NG + 16 * b + (t >> 2), *l = tw + NG + 16 * b + (T >> 2);
    const ulonglong2 v[6] = {p[0], p[NG], p[2 * NG], l[(3 + g) * NG], l[(7 + 2 * g) * NG], l[(8 + 2 * g) * NG]};
#pragma unroll
    for (int i = 0; i < 6; i++) { w[2 + i / 3][2 * (i % 3)] = v[i].x; w[2 + i / 3][2 * (i % 3) + 1] = v[i].y; }
}
// LDS words of a row of 256 points shared by 64 threads (256 words): point e lies at e ^ 6*e5 ^ 24*e6 ^ 2*e7 (e5, e6, e7: its bits),
// so that every access below, 8 bytes a lane in the first three blocks and 16 in the others, falls on 64 different banks per
// half or quarter wavefront.  Pairs of points stay pairs, in order.
__device__ __forceinline__ uint32_t row4_word(uint32_t e) { return e ^ ((e >> 5 & 1u) * 6u) ^ ((e >> 6 & 1u) * 24u) ^ ((e >> 6 & 2u)); }
struct Row4 {
    uint32_t b0, b1, b2, b3;                             // words of thread t's first point in blocks 0 .. 3
    __device__ __forceinline__ explicit Row4(uint32_t t)
        : b0(row4_word(t)), b1(row4_word((t >> 4 << 6) | (t & 15u))), b2(row4_word((t >> 2 << 4) | (t & 3u))), b3(row4_word(4 * row4_last(t))) {}
    __device__ __forceinline__ uint32_t at(int i, int k) const {     // i < 3
        if (i == 0) return (b0 ^ ((k & 1 ? 24u : 0u) ^ (k & 2 ? 2u : 0u))) + 64u * k;
        if (i == 1) return (b1 ^ ((k & 1 ? 16u : 0u) ^ (k & 2 ? 6u : 0u))) + (k & 2 ? 32u : 0u);
        return b2 ^ (4u * k);
    }
    __device__ __forceinline__ void load(int i, u64 (&x)[4], const u64* s) const {
        if (i < 3) {
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = s[at(i, k)];
        } else {
            const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(s + b3), u = *reinterpret_cast<const ulonglong2*>(s + (b3 ^ 2u));
            x[0] = v.x; x[1] = v.y; x[2] = u.x; x[3] = u.y;
        }
    }
    __device__ __forceinline__ void store(int i, const u64 (&x)[4], u64* s) const {
        if (i < 3) {
#pragma unroll
            for (int k = 0; k < 4; k++) s[at(i, k)] = x[k];
        } else {
            *reinterpret_cast<ulonglong2*>(s + b3) = make_ulonglong2(x[0], x[1]);
            *reinterpret_cast<ulonglong2*>(s + (b3 ^ 2u)) = make_ulonglong2(x[2], x[3]);
        }
    }
};
// The eight stages of NX rows at once, 64 threads to a row: values 64k + t in, 4T + k out (forward, T = row4_last(t); W > 0: inputs below
// w_lim), the other way round (inverse: inputs below 2q, results below 2q, W > 0: below w_half).  s: 256 LDS words for each row,
// `stride` apart, on a multiple of 16 bytes.  A block's values are written where they were read, so a lane waits for no other between
// the two.
template <int W, int NX>
__device__ __forceinline__ void row4_fwd(u64 (&x)[NX][4], const u64 (&w)[4][6], u64* s, uint32_t stride, const Row4& at, u64 q) {
    int b = w_lim(W);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (i) {
            wave_exchange();
#pragma unroll
            for (int c = 0; c < NX; c++) at.load(i, x[c], s + c * stride);
        }
        if (i == 0) fwd_block2_x<W, true, NX>(x, w[i], q, b);             // its factors are the same for the whole row
        else fwd_block2_x<W, false, NX>(x, w[i], q, b);
        if (i < 3) {
#pragma unroll
            for (int c = 0; c < NX; c++) at.store(i, x[c], s + c * stride);
        }
    }
}
template <int W, int NX>
__device__ __forceinline__ void row4_inv(u64 (&x)[NX][4], const u64 (&w)[4][6], u64* s, uint32_t stride, const Row4& at, u64 q, const ModConst& m) {
    int bound = 2;                                       // narrow: 2, 10, 40, 160, at the end 640
#pragma unroll
    for (int i = 3; i >= 0; i--) {
        if (i < 3) {
            wave_exchange();
#pragma unroll
            for (int c = 0; c < NX; c++) at.load(i, x[c], s + c * stride);
        }
        if (i == 0) inv_block2_x<W, true, NX>(x, w[i], q, bound);         // its factors are the same for the whole row
        else inv_block2_x<W, false, NX>(x, w[i], q, bound);
        if (i) {
#pragma unroll
            for (int c = 0; c < NX; c++) at.store(i, x[c], s + c * stride);
        }
    }
    if (W == 0 || W == W_NEAR) {
#pragma unroll
        for (int c = 0; c < NX; c++)
#pragma unroll
            for (int k = 0; k < 4; k++) x[c][k] = inv_end<W>(x[c][k], m);
    }
}
