// Device-side 64-bit modular arithmetic for gfx950.
//
// gfx950 has no 64x64->128 multiply; wide products are built from 32x32->64 multiply-adds
// (v_mad_u64_u32), which issue at the same rate as fp64 FMA on this chip, so the cost model is
// "count the 32-bit multiplies".  Twiddle-like multiplications by a constant known in advance
// use Shoup's precomputed quotient; sums of products are accumulated in 128 bits and reduced
// once with a Barrett step.
#pragma once
#include "he_internal.h"

__device__ __forceinline__ u64 mulhi64(u64 a, u64 b) { return __umul64hi(a, b); }

// Two adjacent residues of a buffer that the caller gave, which is aligned to a residue and no further: 8 bytes, as the type
// says, so that nothing is concluded from 16.  Still one 16-byte access, which global memory takes at any multiple of 4.
typedef ulonglong2 pair64 __attribute__((aligned(8)));
#define LOAD2(p) (*reinterpret_cast<const pair64*>(p))
#define STORE2(p) (*reinterpret_cast<pair64*>(p))
// The same past the caches' usual replacement: data that is read once (operands of sums larger than the caches) or that is no faster
// for its reader where it would stay (the results of a key switch or a rescale) does not take the place of what is read again.
typedef u64 stream64 __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ ulonglong2 load2_stream(const u64* p) {
    const stream64 v = __builtin_nontemporal_load(reinterpret_cast<const stream64*>(p));
    return make_ulonglong2(v.x, v.y);
}
__device__ __forceinline__ void store2_stream(u64* p, u64 a, u64 b) { __builtin_nontemporal_store((stream64){a, b}, reinterpret_cast<stream64*>(p)); }

// w*y mod q in [0, 2q) for any y < 2^64, given w < q and w_sh = floor(w*2^64/q)  (Shoup).
__device__ __forceinline__ u64 shoup_lazy(u64 y, u64 w, u64 w_sh, u64 q) {
    u64 h = mulhi64(w_sh, y);
    return w * y - h * q;
}

// x >= q ? x - q : x for x < q + 2^63.  The sign of the difference, spread over a word, masks the q that is added back:
// four instructions with no carry flag for the uniform form (the subtraction is an addition of -q, which the compiler
// must not turn back into a borrow chain), against compare, two selects, subtract with borrow and the wait states a flag
// needs.  csub takes any q, csub_u a q that is the same for the whole wavefront.
__device__ __forceinline__ u64 mask_add(u64 d, u64 q) { return d + (q & (u64)((int64_t)d >> 63)); }
__device__ __forceinline__ u64 csub(u64 x, u64 q) { return mask_add(x - q, q); }
__device__ __forceinline__ u64 neg_u(u64 q) {
    u64 n = 0 - q;
    asm("" : "+s"(n));
    return n;
}
// a value that is the same for the whole wavefront, in scalar registers (loads after a store come back in vector ones)
__device__ __forceinline__ u64 uni64(u64 v) {
    return ((u64)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
}
__device__ __forceinline__ u64 csub_u(u64 x, u64 q) { return mask_add(x + neg_u(q), q); }

// x >= q ? x - q : x for x < 2^63 in two instructions: the smaller of x and the difference, taken as doubles, which order bit patterns
// below 2^63 as the integers they are.  Where the difference is negative, clearing its sign leaves 2^63 - (q - x), which is above x
// or not a number, and the minimum of a number and none is the number.  For signalling ones that holds with the wavefront's IEEE mode
// off: kernels that use this start with ieee_off().  Nothing in the source ties the two together, so the build refuses an object with a
// kernel that has the one and not, before its first branch, the other (build.py).  q: the same for the whole wavefront.
__device__ __forceinline__ void ieee_off() { asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 9, 1), 0"); }
__device__ __forceinline__ u64 csub_min(u64 x, u64 q) {
    u64 r;
    asm("v_min_f64 %0, |%1|, %2" : "=v"(r) : "v"(x + neg_u(q)), "v"(x));
    return r;
}

// the same value in scalar registers, from which nothing is concluded about its factors
__device__ __forceinline__ u64 opaque_s(u64 v) {
    asm("" : "+s"(v));
    return v;
}
// s with h added to its upper word: as one 32-bit addition, which the compiler would widen to 64 bits and a move
__device__ __forceinline__ u64 add_upper(u64 s, u64 h) {
    uint32_t r;
    asm("v_add_u32 %0, %1, %2" : "=v"(r) : "v"((uint32_t)(s >> 32)), "v"((uint32_t)h));
    return ((u64)r << 32) | (uint32_t)s;
}

// High word of a*b from three 32x32 products (the low*low product and the carries out of the
// middle column are dropped): never above the true value, at most 2 below it.  The last 32-bit term is added by a
// multiply-add with the factor 1, which takes it as it is; written as an addition it is widened to a register pair first,
// two moves per product (16-output convolution at level 5: 651 -> 638 us).
__device__ __forceinline__ u64 mulhi64_approx(u64 a, u64 b) {
    const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b, bh = (uint32_t)(b >> 32);
    u64 r = (u64)ah * bh + __umulhi(ah, bl), carry;
    asm("v_mad_u64_u32 %0, %1, %2, 1, %3" : "=v"(r), "=s"(carry) : "v"(__umulhi(al, bh)), "v"(r));
    return r;
}

// a + b + c as one instruction.  Opaque on purpose: sums of 32-bit products written in C become 64-bit multiply-adds with
// moves around them (7 instructions instead of 6 for the high word below, 12 where nothing is added first).
__device__ __forceinline__ uint32_t add3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// a * b + c as one instruction where the compiler sees a shift
__device__ __forceinline__ u64 mad_wide(uint32_t a, uint32_t b, uint32_t c) {
    u64 r, carry;
    asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(r), "=s"(carry) : "v"(a), "s"(b), "v"((u64)c));
    return r;
}

// x + (w*y mod q), the product in [0, 4q): Shoup's product with the approximate quotient above (one multiply fewer and
// no carry chain; the quotient is at most 2 short, each unit adds q to the remainder).  One multiply-add chain modulo
// 2^64 with x as its first addend and -q as the quotient's factor: two wide multiply-adds for the low columns, four
// 32-bit products for the high word.
__device__ __forceinline__ u64 shoup_acc(u64 x, u64 y, u64 w, u64 w_sh, u64 q) {
    const u64 h = mulhi64_approx(w_sh, y), nq = 0 - q;
    const uint32_t w0 = (uint32_t)w, w1 = (uint32_t)(w >> 32), y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
    const uint32_t h0 = (uint32_t)h, h1 = (uint32_t)(h >> 32), n0 = (uint32_t)nq, n1 = (uint32_t)(nq >> 32);
    u64 s = (u64)w0 * y0 + x;
    s += (u64)h0 * n0;
    const uint32_t hi = add3(add3((uint32_t)(s >> 32), w0 * y1, w1 * y0), h0 * n1, h1 * n0);
    return ((u64)hi << 32) | (uint32_t)s;
}

// ---- products by a factor known in advance, in nine instructions (narrow moduli of the two-launch transforms)
// w*y = w*y0 + w'*y1 with y = y0 + 2^32 y1 and w' = 2^32 w mod q: the quotient of the sum then fits one word and takes two multiply-adds,
// h = (a0*y0 + a1*y1) / 2^32, where the quotient of a 64-bit y is two words of three products.  (a0, a1) are the words of floor(w * 2^63 / q)
// (h_companion): one bit less than Shoup's companion, so that the sum of the two products fits 64 bits for every y below 2^63, at
// the price of a quotient that counts in units of 2q.  w' is 2^32 w - a0 * 2q, below 2q; a1 / 2^31 is then w' / q up to rounding.
// Error of the quotient in units of q: below 2 for a0 (y0 / 2^31), 1 for a1 (y1 / 2^31), 2 for the division: results below 5q.

// w' of a factor; n2q = -2q.  UNI: factor and modulus are the same for the whole wavefront (scalar instructions).
template <bool UNI>
__device__ __forceinline__ u64 split_factor(u64 w, u64 a, u64 n2q) {
    const uint32_t a0 = (uint32_t)(a >> 32);
    if (UNI) return (w << 32) + (u64)a0 * n2q;
    u64 h = (u64)a0 * (uint32_t)(n2q >> 32) + w;
    asm("" : "+v"(h));
    return add_upper((u64)a0 * (uint32_t)n2q, h);
}
// x + (w*y mod q), the product below 5q, for y below 2^63.  Both words are chains of multiply-adds: the upper one's carries are
// dropped with its upper half.
__device__ __forceinline__ u64 split_acc(u64 x, u64 y, u64 w, u64 a, u64 wh, u64 n2q) {
    const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
    const uint32_t h = (uint32_t)(((u64)(uint32_t)(a >> 32) * y0 + (u64)(uint32_t)a * y1) >> 32);
    u64 s = (u64)(uint32_t)w * y0 + x;
    s += (u64)(uint32_t)wh * y1;
    s += (u64)h * (uint32_t)n2q;
    u64 u = (u64)(uint32_t)(w >> 32) * y0;
    u += (u64)(uint32_t)(wh >> 32) * y1;
    u += (u64)h * (uint32_t)(n2q >> 32);
    asm("" : "+v"(u));
    return add_upper(s, u);
}

// ---- products by a factor known in advance, in nine instructions and nothing to prepare (moduli near a multiple of 2^32)
// Values are signed here.  With y = y0 + 2^32 y1, A = 2^32 w and B = 2^64 w mod q the sum A y0 + B y1 is 2^32 w y mod q, and one step of
// Montgomery's reduction (Math. Comp. 44, 1985) divides it by 2^32: m = -sum/q mod 2^32, (sum + m q) / 2^32.  All words are balanced: the low word
// of y, of a factor and of q is a signed number, the upper one rounded to match (y1 is the upper word of y + 2^31).  So the low words' sum A0 y0 +
// B0 y1 + m q0 stays in 63 bits where q0 is small (near_fwd, near_inv: he_internal.h), and the result is below q/4 + q |y| / 2^65 + q/2 in
// magnitude.  A factor's table entry is (A, B), so none of its words has to be worked out (split_factor: three instructions), bounds grow by less than
// q a stage instead of 5q, and 60-bit special primes need no conditional subtractions.  Butterflies of four stages on 16 points, instructions and
// rate (10^12/s): forward 13.4 -> 12, 2.52 -> 2.69, inverse 14.4 -> 12, 2.36 -> 2.73; at 60 bits forward 15.4 -> 12, 2.22 -> 2.81.
struct NearQ {
    int32_t q0, q1, qi;              // balanced words of q, -1/q mod 2^32
    u64 half;                        // 2^31
    __device__ __forceinline__ explicit NearQ(u64 q) : q0((int32_t)(uint32_t)q), q1((int32_t)(uint32_t)((q + 0x80000000ull) >> 32)), half(opaque_s(0x80000000ull)) {
        uint32_t v = 3u * (uint32_t)q ^ 2u;              // 1/q to 5 bits, then 10, 20, 40
#pragma unroll
        for (int i = 0; i < 3; i++) v *= 2u - (uint32_t)q * v;
        qi = (int32_t)(0u - v);
    }
};
// r = x + (w*y mod q); ZERO: without x.  UNI: the factor is the same for the whole wavefront.  One block of instructions (near_acc2: two products): the
// compiler would take the factors' words as 64-bit numbers, keep their signs in registers of their own and multiply the long way (1.6 instead of
// 2.7 * 10^12 butterflies/s), and it puts wait states between blocks that follow each other.  What words have to be named of lies in v[2:3].
#define NEAR_WORDS(F, f) F((uint32_t)f.x), F((uint32_t)(f.x >> 32)), F((uint32_t)f.y), F((uint32_t)(f.y >> 32))
#define NEAR_PRODUCT(R, A0, A1, B0, B1, YL, Y, START)          \
    "v_lshl_add_u64 v[2:3], " Y ", 0, %[half]\n\t"             \
    "v_mad_i64_i32 " R ", %[c], " B1 ", v3, " START "\n\t"     \
    "v_mad_i64_i32 v[2:3], %[c], " B0 ", v3, 0\n\t"            \
    "v_mad_i64_i32 " R ", %[c], " A1 ", " YL ", " R "\n\t"     \
    "v_mad_i64_i32 v[2:3], %[c], " A0 ", " YL ", v[2:3]\n\t"   \
    "v_mul_lo_u32 %[m], v2, %[qi]\n\t"                         \
    "v_mad_i64_i32 v[2:3], %[c], %[m], %[q0], v[2:3]\n\t"      \
    "v_mad_i64_i32 " R ", %[c], %[m], %[q1], " R "\n\t"        \
    "v_mad_i64_i32 " R ", %[c], v3, 1, " R "\n\t"
template <bool UNI, bool ZERO = false>
__device__ __forceinline__ u64 near_acc(u64 x, u64 y, ulonglong2 f, const NearQ& n) {
    u64 r, carry;
    uint32_t m;
#define NEAR_ASM(START, F)                                                                                                           \
    asm(NEAR_PRODUCT("%0", "%3", "%4", "%5", "%6", "%7", "%8", START)                                                                 \
        : "=&v"(r), [m] "=&v"(m), [c] "=&s"(carry)                                                                                   \
        : NEAR_WORDS(F, f), "v"((uint32_t)y), "v"(y), "v"(x), [qi] "s"(n.qi), [q0] "s"(n.q0), [q1] "s"(n.q1), [half] "s"(n.half)      \
        : "v2", "v3")
    if (ZERO) x = y;                                     // not used
    if (UNI && ZERO) NEAR_ASM("0", "s");
    if (UNI && !ZERO) NEAR_ASM("%9", "s");
    if (!UNI && ZERO) NEAR_ASM("0", "v");
    if (!UNI && !ZERO) NEAR_ASM("%9", "v");
#undef NEAR_ASM
    return r;
}
template <bool UNI, bool ZERO = false>
__device__ __forceinline__ void near_acc2(u64& r0, u64 x0, u64 y0, ulonglong2 f0, u64& r1, u64 x1, u64 y1, ulonglong2 f1, const NearQ& n) {
    u64 s0, s1, carry;
    uint32_t m;
#define NEAR_ASM(START0, START1, F)                                                                                                  \
    asm(NEAR_PRODUCT("%0", "%4", "%5", "%6", "%7", "%12", "%14", START0) NEAR_PRODUCT("%1", "%8", "%9", "%10", "%11", "%13", "%15", START1)   \
        : "=&v"(s0), "=&v"(s1), [m] "=&v"(m), [c] "=&s"(carry)                                                                       \
        : NEAR_WORDS(F, f0), NEAR_WORDS(F, f1), "v"((uint32_t)y0), "v"((uint32_t)y1), "v"(y0), "v"(y1), "v"(x0), "v"(x1),             \
          [qi] "s"(n.qi), [q0] "s"(n.q0), [q1] "s"(n.q1), [half] "s"(n.half)                                                         \
        : "v2", "v3")
    if (ZERO) x0 = y0, x1 = y1;                          // not used
    if (UNI && ZERO) NEAR_ASM("0", "0", "s");
    if (UNI && !ZERO) NEAR_ASM("%16", "%17", "s");
    if (!UNI && ZERO) NEAR_ASM("0", "0", "v");
    if (!UNI && !ZERO) NEAR_ASM("%16", "%17", "v");
#undef NEAR_ASM
    r0 = s0;
    r1 = s1;
}
// Differences of two pairs of 64-bit numbers.  A borrow may be read two instructions after it is written; the compiler, which
// keeps all of them in the same flag, waits that long for each.
__device__ __forceinline__ u64 join32(uint32_t lo, uint32_t hi) { return ((u64)hi << 32) | lo; }
__device__ __forceinline__ void sub2(u64& d0, u64 a0, u64 b0, u64& d1, u64 a1, u64 b1) {
    uint32_t l0, h0, l1, h1;
    u64 c;
    asm("v_sub_co_u32 %0, vcc, %5, %6\n\t"
        "v_sub_co_u32 %2, %4, %9, %10\n\t"
        "s_nop 0\n\t"
        "v_subb_co_u32 %1, vcc, %7, %8, vcc\n\t"
        "v_subb_co_u32 %3, %4, %11, %12, %4"
        : "=&v"(l0), "=&v"(h0), "=&v"(l1), "=&v"(h1), "=&s"(c)
        : "v"((uint32_t)a0), "v"((uint32_t)b0), "v"((uint32_t)(a0 >> 32)), "v"((uint32_t)(b0 >> 32)), "v"((uint32_t)a1), "v"((uint32_t)b1),
          "v"((uint32_t)(a1 >> 32)), "v"((uint32_t)(b1 >> 32))
        : "vcc");
    d0 = join32(l0, h0);
    d1 = join32(l1, h1);
}

// w*y mod q in [0, 4q)
__device__ __forceinline__ u64 shoup_lazy4(u64 y, u64 w, u64 w_sh, u64 q) { return shoup_acc(0, y, w, w_sh, q); }

// canonical w*y mod q
__device__ __forceinline__ u64 shoup_mul(u64 y, u64 w, u64 w_sh, u64 q) { return csub(shoup_lazy(y, w, w_sh, q), q); }

// x mod q for x < 2^(bits+63), mu = floor(2^(bits+63)/q): quotient estimate is at most 2 low.
__device__ __forceinline__ u64 barrett128(u128 x, u64 q, u64 mu, uint32_t bits) {
    u64 x1 = (u64)(x >> (bits - 1));
    u64 qh = mulhi64(x1, mu);
    u64 r = (u64)x - qh * q;
    r = csub(r, 2 * q);
    return csub(r, q);
}

// Same with the three-product quotient and no final correction: result in [0, 5q), congruent to x.
__device__ __forceinline__ u64 barrett128_lazy(u128 x, u64 q, u64 mu, uint32_t bits) {
    u64 x1 = (u64)(x >> (bits - 1));
    u64 qh = mulhi64_approx(x1, mu);
    return (u64)x - qh * q;
}

// x mod q for a single word x (any value), through the same Barrett constant.
__device__ __forceinline__ u64 barrett64(u64 x, u64 q, u64 mu, uint32_t bits) { return barrett128((u128)x, q, mu, bits); }

__device__ __forceinline__ u64 addmod(u64 a, u64 b, u64 q) { return csub(a + b, q); }
__device__ __forceinline__ u64 submod(u64 a, u64 b, u64 q) { return a >= b ? a - b : a + q - b; }

__device__ __forceinline__ u64 mulmod(u64 a, u64 b, const ModConst& m) { return barrett128((u128)a * b, m.q, m.mu, m.bits); }

// Sum of products of values below 2^60 (or below 2^61 with a factor that small primes keep low), halves of 30 bits summed
// in three 64-bit words that the multiply-adds feed directly: 4 instructions per product besides the splitting, where a
// 128-bit sum takes 14.  a0 and a2 take below 2^60 per product of canonical residues, a1 below 2^61:
// 8 products fit (a1 reaches 16 (2^30 - 1)^2, with a0's carries below 2^64), 16 of residues of at most 59 bits (high halves below 2^29).
#define SPLIT_H 30
struct SplitSum {
    u64 a0, a1, a2;
};
__device__ __forceinline__ void split_mac(SplitSum& s, u64 d, u64 k) {
    const uint32_t M = (1u << SPLIT_H) - 1;
    const uint32_t d0 = (uint32_t)d & M, d1 = (uint32_t)(d >> SPLIT_H), k0 = (uint32_t)k & M, k1 = (uint32_t)(k >> SPLIT_H);
    s.a0 += (u64)d0 * k0;
    s.a1 += (u64)d0 * k1;
    s.a1 += (u64)d1 * k0;
    s.a2 += (u64)d1 * k1;
}
__device__ __forceinline__ u128 split_value(const SplitSum& s) {
    return (u128)s.a0 + ((u128)s.a1 << SPLIT_H) + ((u128)s.a2 << (2 * SPLIT_H));
}
// Congruent to the sums (below 2^(bits+63)), below 6q.  From 32 bits the quotient is taken from a sum's top, a2 * 2^(61-bits) +
// (a1 + a0 / 2^30) / 2^(bits-31), at most 1.5 below the sum / 2^(bits-1), and the remainder from the sum's low word: 17
// instructions, where putting the 128-bit sum together first takes 30.
template <int H = SPLIT_H>
__device__ __forceinline__ u64 split_reduce_top(const SplitSum& s, const ModConst& m) {
    const u64 a1 = s.a1 + (s.a0 >> H);
    const u64 qh = mulhi64_approx((s.a2 << (2 * H + 1 - m.bits)) + (a1 >> (m.bits - H - 1)), m.mu);
    return s.a0 + (s.a1 << H) + (s.a2 << (2 * H)) - qh * m.q;
}
template <int N>
__device__ __forceinline__ void split_reduce(u64 (&v)[N], const SplitSum (&s)[N], const ModConst& m) {
    if (m.bits >= 32) {
#pragma unroll
        for (int i = 0; i < N; i++) v[i] = split_reduce_top(s[i], m);
    } else {
#pragma unroll
        for (int i = 0; i < N; i++) v[i] = barrett128_lazy(split_value(s[i]), m.q, m.mu, m.bits);
    }
}
__device__ __forceinline__ u64 split_reduce(const SplitSum& s, const ModConst& m) {
    return m.bits >= 32 ? split_reduce_top(s, m) : barrett128_lazy(split_value(s), m.q, m.mu, m.bits);
}

// v mod q for v below 2^LOGV * 2^bits (and below 2^64): the quotient from the top 32 bits of v and rec =
// floor(2^(bits+31) / q), at most one too small.  The lazy form stops before the correction: below 2q.
template <int LOGV>
__device__ __forceinline__ u64 reduce_lazy(u64 v, u64 q, uint32_t bits, uint32_t rec) {
    const uint32_t sh = bits > 32 - LOGV ? bits - (32 - LOGV) : 0;
    const uint32_t qh = __umulhi((uint32_t)(v >> sh), rec) >> (bits - 1 - sh);
    return v - (u64)qh * q;
}
template <int LOGV>
__device__ __forceinline__ u64 reduce_full(u64 v, u64 q, uint32_t bits, uint32_t rec) {
    return csub(reduce_lazy<LOGV>(v, q, bits, rec), q);
}
// the same for a q of the whole wavefront, after ieee_off()
template <int LOGV>
__device__ __forceinline__ u64 reduce_min(u64 v, u64 q, uint32_t bits, uint32_t rec) {
    return csub_min(reduce_lazy<LOGV>(v, q, bits, rec), q);
}
