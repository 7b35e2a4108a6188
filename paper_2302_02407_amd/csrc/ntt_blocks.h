// Register blocks of the radix-2 negacyclic transforms shared by the two-launch kernels, the column conversion and the small-ring kernels:
// four butterfly stages on 16 points, or two on 4 points, held by one thread (Harvey butterflies, lazy ranges).
#pragma once
#include "modarith.h"

#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)   // loads above it are issued before the arithmetic below it

// A butterfly is counted in instructions: on gfx950 the 32-bit multiplies, v_mad_u64_u32 and v_lshl_add_u64 all issue at
// one per lane and cycle (28-35 T/s measured), so what costs is how many there are.  The product enters the sum through
// the multiply-adds' own addend (X + w*Y - h*q accumulated in one chain with -q as the factor), and the difference is
// 2X + c*q minus that sum.  Narrow moduli: two instructions for the quotient h, 7 for the sum, 3 for the difference (split_acc), and
// 3 for a factor's second word where it is not the same for the whole wavefront (scalar instructions there).  Wide ones: 5, 8 and 3
// with Shoup's companion.  A product formed on its own and then added and subtracted takes 20.
//
// Which moduli are narrow stands at narrow_fwd / narrow_inv (he_internal.h); their factors are stored with h_tw_split's companion, the
// others' with Shoup's (ctx.hip).
//
// Ranges are kept in units of q and known when the code is compiled: a twiddle product is below 5q (narrow) or 4q (wide) whatever
// its factor, a forward stage therefore adds that to the bound of every point, an inverse stage adds the bounds of its two points.  A
// conditional subtraction is made only where the next sum would leave 64 bits: nowhere for narrow moduli (forward: 17 stages
// from below 5q end below 90q; inverse: a pass ends below 640q), every other forward stage and a few inverse points for wide ones
// (below 2^60, so that 16q fits).
__device__ __forceinline__ void ct_bfly(u64& X, u64& Y, u64 w, u64 w_sh, u64 q, u64 q4) {
    const u64 S = shoup_acc(X, Y, w, w_sh, q);
    Y = (X + X + q4) - S;
    X = S;
}
// what the narrow butterflies need of a modulus, in scalar registers
struct NarrowQ {
    u64 n2q, q5;
    __device__ __forceinline__ explicit NarrowQ(u64 q) : n2q(opaque_s(0 - 2 * q)), q5(opaque_s(5 * q)) {}
};
__device__ __forceinline__ void ct_bfly_n(u64& X, u64& Y, u64 w, u64 a, u64 wh, const NarrowQ& n) {
    const u64 S = split_acc(X, Y, w, a, wh, n.n2q);
    Y = (X + X + n.q5) - S;
    X = S;
}
// One factor on K pairs of points (X[i], Y[i]), stage n of a block.  Wide moduli: X brought below 8q first in every other stage
// (inputs below 16q).
template <bool WIDE, bool UNI, int K, class PX, class PY>
__device__ __forceinline__ void ct_stage(int n, PX&& X, PY&& Y, u64 w, u64 a, u64 q) {
    if (WIDE) {
#pragma unroll
        for (int k = 0; k < K; k++) {
            if ((n & 1) == 0) X(k) = csub_u(X(k), 8 * q);
            ct_bfly(X(k), Y(k), w, a, q, 4 * q);
        }
    } else {
        const NarrowQ nq(q);
        const u64 wh = split_factor<UNI>(w, a, nq.n2q);
#pragma unroll
        for (int k = 0; k < K; k++) ct_bfly_n(X(k), Y(k), w, a, wh, nq);
    }
}

// Inverse butterflies of one factor on K pairs of points below bx*q and by*q; the bounds of the results replace them.  They are
// constants of the unrolled code.
template <bool WIDE, bool UNI, int K, class PX, class PY, class BX, class BY>
__device__ __forceinline__ void gs_stage(PX&& PX_, PY&& PY_, BX&& bx_, BY&& by_, u64 w, u64 a, u64 q) {
    const NarrowQ nq(q);
    const u64 wh = WIDE ? 0 : split_factor<UNI>(w, a, nq.n2q);
#pragma unroll
    for (int k = 0; k < K; k++) {
        u64 &X = PX_(k), &Y = PY_(k);
        int &bx = bx_(k), &by = by_(k);
        if (WIDE) {
#pragma unroll
            for (int r = 0; r < 3; r++) {                // at most three steps are ever needed; constants once unrolled
                if (bx + by <= 16) continue;
                if (bx >= by) { const int b = bx > 8 ? 8 : 4; X = csub_u(X, q * b); bx = b; }
                else { const int b = by > 8 ? 8 : 4; Y = csub_u(Y, q * b); by = b; }
            }
        }
        const u64 d = (X + q * (u64)by) - Y;
        X = X + Y;
        Y = WIDE ? shoup_lazy4(d, w, a, q) : split_acc(0, d, w, a, wh, nq.n2q);
        bx += by;
        by = WIDE ? 4 : 5;
    }
}
// Every point of a register block below 4q again (wide moduli, before an exchange mixes the points).
template <int N>
__device__ __forceinline__ void settle4(u64 (&x)[N], int (&b)[N], u64 q) {
#pragma unroll
    for (int k = 0; k < N; k++) {
        if (b[k] > 8) x[k] = csub_u(x[k], q * 8);
        if (b[k] > 4) x[k] = csub_u(x[k], q * 4);
        b[k] = 4;
    }
}
// Bound of every point of narrow inverse blocks of n stages that start below b*q: sums double it, a product is below 5q and may be
// doubled by the stages behind its own.
__device__ constexpr int narrow_after(int b, int n) { return (b << n) > (5 << n) / 2 ? b << n : (5 << n) / 2; }

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
// Forward stages U0 .. U1-1; UNI: the factors are the same for the whole wavefront.  Wide moduli: inputs and results below 16q.
template <bool WIDE, int U0, int U1, bool UNI = false>
__device__ __forceinline__ void fwd_stages(u64 (&x)[16], const ulonglong2 (&w)[15], u64 q) {
#pragma unroll
    for (int u = U0; u < U1; u++) {
        const int dist = 8 >> u;
#pragma unroll
        for (int g = 0; g < (1 << u); g++) {
            const ulonglong2 f = w[(1 << u) - 1 + g];
            auto X = [&](int k) -> u64& { return x[g * 2 * dist + k]; };
            auto Y = [&](int k) -> u64& { return x[g * 2 * dist + dist + k]; };
            if (u == 0) ct_stage<WIDE, UNI, 8>(u - U0, X, Y, f.x, f.y, q);
            else if (u == 1) ct_stage<WIDE, UNI, 4>(u - U0, X, Y, f.x, f.y, q);
            else if (u == 2) ct_stage<WIDE, UNI, 2>(u - U0, X, Y, f.x, f.y, q);
            else ct_stage<WIDE, UNI, 1>(u - U0, X, Y, f.x, f.y, q);
        }
    }
}
// Inverse stages U1-1 down to U0, bounds b per point.
template <bool WIDE, int U0, int U1, bool UNI = false>
__device__ __forceinline__ void inv_stages(u64 (&x)[16], int (&b)[16], const ulonglong2 (&w)[15], u64 q) {
#pragma unroll
    for (int u = U1 - 1; u >= U0; u--) {
        const int dist = 8 >> u;
#pragma unroll
        for (int g = 0; g < (1 << u); g++) {
            const ulonglong2 f = w[(1 << u) - 1 + g];
            auto X = [&](int k) -> u64& { return x[g * 2 * dist + k]; };
            auto Y = [&](int k) -> u64& { return x[g * 2 * dist + dist + k]; };
            auto BX = [&](int k) -> int& { return b[g * 2 * dist + k]; };
            auto BY = [&](int k) -> int& { return b[g * 2 * dist + dist + k]; };
            if (u == 0) gs_stage<WIDE, UNI, 8>(X, Y, BX, BY, f.x, f.y, q);
            else if (u == 1) gs_stage<WIDE, UNI, 4>(X, Y, BX, BY, f.x, f.y, q);
            else if (u == 2) gs_stage<WIDE, UNI, 2>(X, Y, BX, BY, f.x, f.y, q);
            else gs_stage<WIDE, UNI, 1>(X, Y, BX, BY, f.x, f.y, q);
        }
    }
}
// the largest bound of a block holds for all of its points once an exchange has mixed them
template <int N>
__device__ __forceinline__ void bounds_all(int (&b)[N], int v) {
#pragma unroll
    for (int k = 0; k < N; k++) b[k] = v;
}

// Two forward / inverse stages on 4 register points of NX rows (same pairing and twiddle indexing as the 16-point blocks), factors
// r = {w0, a0, w1, a1, w2, a2}.  ONE: only the first of the two stages.  Ranges as above.
template <bool WIDE, bool UNI, int NX, bool ONE = false>
__device__ __forceinline__ void fwd_block2_x(u64 (&x)[NX][4], const u64 (&r)[6], u64 q) {
    ct_stage<WIDE, UNI, 2 * NX>(0, [&](int k) -> u64& { return x[k >> 1][k & 1]; }, [&](int k) -> u64& { return x[k >> 1][2 + (k & 1)]; }, r[0], r[1], q);
    if (ONE) return;
    ct_stage<WIDE, UNI, NX>(1, [&](int k) -> u64& { return x[k][0]; }, [&](int k) -> u64& { return x[k][1]; }, r[2], r[3], q);
    ct_stage<WIDE, UNI, NX>(1, [&](int k) -> u64& { return x[k][2]; }, [&](int k) -> u64& { return x[k][3]; }, r[4], r[5], q);
}
// Inverse: inputs below bound*q.  Narrow: results below narrow_after(bound, 2 or 1 stages) * q; wide: bound 4, results below 4q.
template <bool WIDE, bool UNI, int NX, bool ONE = false>
__device__ __forceinline__ void inv_block2_x(u64 (&x)[NX][4], const u64 (&r)[6], u64 q, int bound) {
    int b[NX][4];
#pragma unroll
    for (int i = 0; i < NX; i++)
#pragma unroll
        for (int k = 0; k < 4; k++) b[i][k] = WIDE ? 4 : bound;
    if (!ONE) {
        gs_stage<WIDE, UNI, NX>([&](int k) -> u64& { return x[k][0]; }, [&](int k) -> u64& { return x[k][1]; },
                                [&](int k) -> int& { return b[k][0]; }, [&](int k) -> int& { return b[k][1]; }, r[2], r[3], q);
        gs_stage<WIDE, UNI, NX>([&](int k) -> u64& { return x[k][2]; }, [&](int k) -> u64& { return x[k][3]; },
                                [&](int k) -> int& { return b[k][2]; }, [&](int k) -> int& { return b[k][3]; }, r[4], r[5], q);
    }
    gs_stage<WIDE, UNI, 2 * NX>([&](int k) -> u64& { return x[k >> 1][k & 1]; }, [&](int k) -> u64& { return x[k >> 1][2 + (k & 1)]; },
                                [&](int k) -> int& { return b[k >> 1][k & 1]; }, [&](int k) -> int& { return b[k >> 1][2 + (k & 1)]; }, r[0], r[1], q);
    if (WIDE) {
#pragma unroll
        for (int i = 0; i < NX; i++) settle4(x[i], b[i], q);
    }
}
template <bool WIDE, bool UNI = false, bool ONE = false>
__device__ __forceinline__ void fwd_block2_r(u64 (&x)[4], const u64 (&r)[6], u64 q) {
    fwd_block2_x<WIDE, UNI, 1, ONE>(reinterpret_cast<u64 (&)[1][4]>(x), r, q);
}
template <bool WIDE, bool UNI = false, bool ONE = false>
__device__ __forceinline__ void inv_block2_r(u64 (&x)[4], const u64 (&r)[6], u64 q, int bound) {
    inv_block2_x<WIDE, UNI, 1, ONE>(reinterpret_cast<u64 (&)[1][4]>(x), r, q, bound);
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
// a pointer to constant memory, which no store can change: loads through it stay scalar after stores
typedef const __attribute__((address_space(4))) u64* const_u64;
// what the row kernels need of a modulus, in scalar registers
__device__ __forceinline__ ModConst mod_const(const ModConst* mc, uint32_t mi) {
    const const_u64 p = (const_u64)(uintptr_t)uni64((u64)(mc + mi));
    ModConst m = {};
    m.q = p[offsetof(ModConst, q) / 8];
    m.mu = p[offsetof(ModConst, mu) / 8];
    const u64 v = p[offsetof(ModConst, bits) / 8];
    m.bits = (uint32_t)v; m.rec = (uint32_t)(v >> 32);
    return m;
}
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
// The eight stages of NX rows at once, 64 threads to a row: values 64k + t in, 4T + k out (forward, T = row4_last(t)), the other way round
// (inverse; narrow moduli: inputs below 2q, results below 2q; wide: below 4q).  s: 256 LDS words for each row, `stride` apart, on
// a multiple of 16 bytes.  A block's values are written where they were read, so a lane waits for no other between the two.
template <bool WIDE, int NX>
__device__ __forceinline__ void row4_fwd(u64 (&x)[NX][4], const u64 (&w)[4][6], u64* s, uint32_t stride, const Row4& at, u64 q) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (i) {
            wave_exchange();
#pragma unroll
            for (int c = 0; c < NX; c++) at.load(i, x[c], s + c * stride);
        }
        if (i == 0) fwd_block2_x<WIDE, true, NX>(x, w[i], q);            // its factors are the same for the whole row
        else fwd_block2_x<WIDE, false, NX>(x, w[i], q);
        if (i < 3) {
#pragma unroll
            for (int c = 0; c < NX; c++) at.store(i, x[c], s + c * stride);
        }
    }
}
template <bool WIDE, int NX>
__device__ __forceinline__ void row4_inv(u64 (&x)[NX][4], const u64 (&w)[4][6], u64* s, uint32_t stride, const Row4& at, u64 q, const ModConst& m) {
    int bound = 2;                                       // narrow: 2, 10, 40, 160, at the end 640
#pragma unroll
    for (int i = 3; i >= 0; i--) {
        if (i < 3) {
            wave_exchange();
#pragma unroll
            for (int c = 0; c < NX; c++) at.load(i, x[c], s + c * stride);
        }
        if (i == 0) inv_block2_x<WIDE, true, NX>(x, w[i], q, bound);     // its factors are the same for the whole row
        else inv_block2_x<WIDE, false, NX>(x, w[i], q, bound);
        bound = narrow_after(bound, 2);
        if (i) {
#pragma unroll
            for (int c = 0; c < NX; c++) at.store(i, x[c], s + c * stride);
        }
    }
    if (!WIDE) {
#pragma unroll
        for (int c = 0; c < NX; c++)
#pragma unroll
            for (int k = 0; k < 4; k++) x[c][k] = reduce_lazy<10>(x[c][k], q, m.bits, m.rec);
    }
}
