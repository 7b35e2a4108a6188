// Internal declarations shared by the translation units of the library (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../../include/he_mi355x.h"

typedef unsigned long long u64;
typedef unsigned __int128 u128;

#define HE_MAX_MODULI 64        // nq + np
#define HE_MAX_LAUNCH_LIMBS 512 // limbs described by one kernel-argument list

// Moduli whose points are never reduced inside the transforms of N = 2^13 and more (products: split_acc, modarith.h) on
// the way: every product's operand has to stay below 2^63, and points reach 90q in 17 forward stages that start below 5q, 640q in
// eight inverse ones (ntt_blocks.h).  Any other modulus is wide and takes conditional subtractions, more of them the widest ones.
// 384 limbs, N = 2^16, primes just below each power or line (in brackets: with products of sixteen instructions, which take any operand
// and had their lines at 2^57 and 2^54): forward 2^54 142 us (147), 2^56.4 144 (147), 2^57 152 (148), 2^59.3 152 (158), 2^60 159 (159); inverse
// 2^53.6 144 (154), 2^54 150 (154), 2^59.3 151 (161), 2^60 157 (160).  The primes from 2^56.4 to 2^57 are the ones that lost, in one
// direction.  With narrow forward up to 2^57.3, their rows brought below 13q first, they took 149, and every other class paid for the
// branch in the row passes: one rotation at level 5 53.6 -> 55.2, a product 59.3 -> 61.1, rescale 26.7 -> 27.5.
static inline bool narrow_fwd(u64 q) { return q <= (1ull << 63) / 96; }       // all of 56 bits, and up to 2^56.4
static inline bool narrow_inv(u64 q) { return q <= (1ull << 63) / 640; }      // all of 53 bits, and up to 2^53.6
static inline bool widest(u64 q) { return q > (1ull << 63) / 13; }            // above 2^59.29
// Moduli whose low word is near 0 as a signed number, as it is of primes near a power of two.  The products of near_acc (modarith.h) ask for
// |operand| / 2 + 2^62 + |low word| 2^31 below 2^63 and are below (3/4 + |operand| / 2^65) q.  Points are not reduced on the way (checked below):
//   forward, up to 2^58: 5q at the start, less than q more with every stage, 17 stages: below 22q;
//   forward, up to 2^59.003 with at most 16 stages, the special primes that are taken above 2^59: 1.5q at the start (whoever writes points for
//   the first pass centres them, near_top), operands below 14.6q < 2^63 - 2^58, which is what low words below 2^26 leave, results below 15.6q
//   (made positive by 16q, near_bias: ntt_blocks.h);
//   inverse: doubled by each of eight stages from 2q, below 512q.
// The lines are where these ranges end.  384 limbs, N = 2^16, primes with small low words (in brackets: such primes in the other classes):
// forward 2^54 134.6 us (134.4), just below 2^58 135.6 (142.9), just above 136.1 (143.3), just above 2^59 136.5 (143.4); inverse 2^54 135.8 (145.5),
// just below 2^53.896 135.6 (149.6).  24 limbs: forward 23.3 (23.5) at 2^54, 23.4 (24.2) below 2^58, 23.8 (24.2) above 2^59; inverse 23.5 (25.0).  Outside
// the class, now that it is there (in brackets before): inverse just above 2^53.9 150.2 (149.8), forward at 1.2 * 2^59 143.0 (143.7), just below 2^60
// 153.6 (151.3).  What it costs other moduli is the jump over its code, which comes first in every kernel, an instruction fetch of some 0.3 us a
// launch: one rotation at level 5 53.5 us (52.0) with narrow ciphertext primes, where the near ones take 51.
static inline bool near_word(u64 q, int64_t most) { return (int32_t)(uint32_t)q < most && (int32_t)(uint32_t)q > -most; }
#define NEAR_WORD (1ll << 27)
#define NEAR_TOP_WORD (1ll << 26)
#define NEAR_FWD (1ull << 58)
#define NEAR_TOP ((1ull << 59) + (1ull << 50))
#define NEAR_INV ((1ull << 63) / 550)        // 2^53.896
static inline bool near_top(u64 q) { return q > NEAR_FWD; }
static inline bool near_fwd(u64 q, uint32_t logN) {
    return near_top(q) ? logN <= 16 && q <= NEAR_TOP && near_word(q, NEAR_TOP_WORD) : near_word(q, NEAR_WORD);
}
static inline bool near_inv(u64 q) { return near_word(q, NEAR_WORD) && q <= NEAR_INV; }
// The ranges above: what points below b*q become in `stages` stages, in units of q; -1 where a product's operand leaves its range
constexpr bool near_takes(double operand, double q, double word) { return operand * q / 2 + 0x1p62 + word * 0x1p31 < 0x1p63; }
constexpr double near_forward(double b, double q, double word, int stages) {
    for (int i = 0; i < stages; i++) {
        if (!near_takes(b, q, word)) return -1;
        b += 0.75 + b * q * 0x1p-65;
    }
    return b;
}
constexpr double near_inverse(double b, double q, double word, int stages) {
    for (int i = 0; i < stages; i++) {
        b *= 2;
        if (!near_takes(b, q, word)) return -1;
    }
    return b;
}
static_assert(near_forward(5, NEAR_FWD, NEAR_WORD, 17) > 5 && near_forward(5, NEAR_FWD, NEAR_WORD, 17) < 22, "");
static_assert(near_forward(1.5, NEAR_TOP, NEAR_TOP_WORD, 15) < 14.6 && near_forward(1.5, NEAR_TOP, NEAR_TOP_WORD, 16) > 1.5 && near_forward(1.5, NEAR_TOP, NEAR_TOP_WORD, 16) < 15.6, "");
static_assert(14.6 * NEAR_TOP < 0x1p63 - 0x1p58 && near_forward(1.5, NEAR_TOP, NEAR_TOP_WORD, 17) > 16, "17 stages end beyond what near_bias makes positive");
static_assert(near_inverse(2, NEAR_INV, NEAR_WORD, 8) == 512 && near_inverse(2, NEAR_INV, NEAR_WORD, 9) < 0, "");
// The classes (ntt_blocks.h), and those of all moduli of a context, bit by bit (a kernel's argument: the branch to a class waits for no load of the
// modulus' constants)
#define W_NEAR 3
static inline uint32_t class_fwd(u64 q, uint32_t logN) { return near_fwd(q, logN) ? W_NEAR : narrow_fwd(q) ? 0 : widest(q) ? 2 : 1; }
static inline uint32_t class_inv(u64 q) { return near_inv(q) ? W_NEAR : narrow_inv(q) ? 0 : widest(q) ? 2 : 1; }
// W of a modulus in the row kernels of key switches (ksrows.hip), for both directions; what is near for the inverse is so for the forward
static inline uint32_t ks_width(u64 q, uint32_t logN) {
    if (near_fwd(q, logN)) return near_inv(q) ? 4 : 5;
    return (uint32_t)!narrow_inv(q) + (uint32_t)!narrow_fwd(q) + (uint32_t)widest(q);
}
struct ModClasses {
    u64 b[2];
    void set(uint32_t mi, uint32_t w) { for (int i = 0; i < 2; i++) b[i] |= (u64)(w >> i & 1u) << mi; }
};

// Per-modulus constants, resident on the device (array indexed by modulus index).
struct ModConst {
    u64 q;          // the prime
    u64 q2;         // 2q
    u64 mu;         // floor(2^(bits+63) / q): Barrett constant for inputs < 2^(bits+63)
    u64 ninv;       // N^-1 mod q
    u64 ninv_sh;    // Shoup companion floor(ninv * 2^64 / q)
    u64 ninv_w;     // N^-1 * psi^-(N/2): scaling folded into the twiddle of the last inverse stage
    u64 ninv_w_sh;
    u64 near_s, near_s_sh, near_w, near_w_sh;    // ninv and ninv_w as factors of near_acc (two-launch transforms)
    u64 one_sh;     // floor(2^64 / q): Shoup companion of the constant 1 (a quotient step for any 64-bit value)
    uint32_t bits;  // bit length of q
    uint32_t rec;   // floor(2^(bits+31) / q): 32-bit reciprocal for small quotients
    double qinv;    // 1 / q
};

#define HE_FP64_BITS 45   // products modulo such primes are exact in FP64 with the ranges smallring.hip keeps

// Modulus index of each limb of a launch, passed by value in the kernel arguments.
struct LimbList {
    uint8_t mod[HE_MAX_LAUNCH_LIMBS];
};

// Optional per-limb output scaling of an inverse transform (replaces the plain N^-1).
struct ScaleList {
    u64 s[HE_MAX_MODULI];
    u64 s_sh[HE_MAX_MODULI];
    u64 w[HE_MAX_MODULI];      // s * psi^-(N/2) mod q (the last inverse stage's twiddle, pre-scaled)
    u64 w_sh[HE_MAX_MODULI];
};

// One target modulus of a conversion on the matrix cores (colconv.hip; filled by conv_operand in keyswitch.hip).  A wavefront loads one as
// eight bytes a lane and four of the rest a lane; from LDS it is read sixteen at a time.
struct alignas(16) ConvOperand {
    uint8_t dig[512];
    int32_t bias[8];
    u64 nq;            // -q modulo 2^64
    uint32_t rec, bits;
    uint32_t centre;   // added to a value's upper word for its quotient: results in [0, 2q), or in [-q, q + 2^32)
    uint32_t unused[3];
};

struct ProfSpan {
    hipEvent_t e0, e1;
    uint32_t limbs;   // limbs transformed by the launch between the two events
    uint32_t digit_limbs; // raised-digit limbs a pass that carries the key-switch inner product has to read
    uint32_t kind;        // he_profile_t::pass_ms index: 0 fwd column or conversion with its columns, 1 fwd row, 2 fwd row +
                          // inner product/epilogue, 3 inv row, 4 inv row + inner product, 5 inv column
};

struct he_ctx {
    uint32_t logN, N, nq, np, dnum, alpha, M; // M = nq + np
    bool srf;          // small ring whose moduli all have at most HE_FP64_BITS bits: FP64 kernels (smallring.hip)
    hipStream_t stream;
    int device;
    u64 mod[HE_MAX_MODULI];
    u64 psi[HE_MAX_MODULI];
    u64 itw1[HE_MAX_MODULI];    // psi^-(N/2), the single twiddle of inverse stage 0
    ModConst h_mc[HE_MAX_MODULI];
    ModClasses cls_fwd, cls_inv;
    u64 ks_width[3];            // of all moduli, bit by bit
    // device tables
    ModConst* d_mc;    // [M]
    ulonglong2* d_tw;  // [M][N]  psi^bitrev(i) and its companion (h_companion), one 16-byte load
    ulonglong2* d_itw; // [M][N]  psi^-bitrev(i), likewise
    double *d_ftw, *d_fitw; // [M][N] the same factors for the FP64 kernels, in their order (ctx.hip, ftw_pos); null elsewhere
    // basis-conversion tables (keyswitch.hip); present when np > 0
    u64* d_up_hat;     // [dnum][alpha][alpha][M]: (Q_j/q_i) mod m for digit j holding sz limbs, [j][sz-1][i][m]
    std::vector<u64> h_up_invhat; // [dnum][alpha][alpha]: ((Q_j/q_i)^-1 mod q_i), [j][sz-1][i]
    u64* d_dn_hat;     // [np][M]: (P/p_t) mod m  (only m < nq used)
    std::vector<u64> h_dn_invhat; // [np]: (P/p_t)^-1 mod p_t
    // the same constants as operands of the matrix instruction (colconv.hip): [dnum][alpha][M] and [M], null where that path
    // does not apply
    ConvOperand *d_up_op, *d_dn_op;
    u64* d_pinv;       // [nq] P^-1 mod q_r
    std::vector<u64> h_pinv;      // the same on the host
    u64* d_pinv_sh;    // [nq] companions (h_companion)
    // rescale tables: q_l^-1 mod q_r for r < l, [nq][nq]
    u64* d_qlinv;
    std::vector<u64> h_qlinv;
    u64* d_qlinv_sh;
    // workspace (grown on demand)
    u64* d_ws;
    size_t ws_bytes;
    std::map<uint32_t, const u64*> evk; // Galois element -> device key
    he_counters_t cnt;
    bool prof_on;                       // time every transform launch with an event pair
    std::vector<ProfSpan> prof_events;
    uint64_t prof_key_limbs;            // key limbs the inner products had to read while timing was on (one pass per key per chunk)
    std::string err;
};

// ---- host helpers (ctx.hip)
int32_t he_fail(he_ctx* ctx, int32_t code, const char* fmt, ...);
int32_t he_ensure_ws(he_ctx* ctx, size_t bytes);
u64 h_mulmod(u64 a, u64 b, u64 m);
u64 h_powmod(u64 a, u64 e, u64 m);
u64 h_invmod(u64 a, u64 m);
u64 h_shoup(u64 w, u64 m);
u64 h_companion(uint32_t logN, u64 w, u64 m);
uint32_t h_galois_of_step(const he_ctx* ctx, int32_t step);

// Rings whose limb does not fit one work group's LDS: two launches per transform (ntt2p.hip)
static inline bool two_pass(const he_ctx* c) { return c->logN > 12; }

// Every extern "C" body runs inside he_guard: no C++ exception (a failed host allocation in a
// std::vector / std::map / std::string) crosses the C ABI; it comes back as HE_ERR_ALLOC.
void he_fail_nothrow(he_ctx* ctx, const char* msg) noexcept;
template <class F>
static inline int32_t he_guard(const he_ctx* ctx, const char* who, F&& body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc&) {
        he_fail_nothrow(const_cast<he_ctx*>(ctx), who);
        return HE_ERR_ALLOC;
    } catch (...) {
        he_fail_nothrow(const_cast<he_ctx*>(ctx), who);
        return HE_ERR_ALLOC;
    }
}

#define HE_HIP(ctx, call)                                                                            \
    do {                                                                                             \
        hipError_t e__ = (call);                                                                     \
        if (e__ != hipSuccess) return he_fail(ctx, HE_ERR_HIP, "%s: %s", #call, hipGetErrorString(e__)); \
    } while (0)

int32_t he_noalloc_init_device(he_ctx* ctx, int device);   // noalloc.hip: address of the static scratch on this GPU

// ---- internal device-work launchers (all enqueue on ctx->stream, none synchronises)
#define HE_MAX_SEGS 16      // distinct source allocations one transform launch can read from
#define HE_MAX_KS_JOBS 16   // key-switch jobs whose ModDown runs in one set of launches

// Epilogue of ModDown fused into the last pass of the forward transform of the converted p-part
// (separate kernel on the generic path).  The launch covers J jobs x 2 components x L1 limbs:
// limb i -> job i/(2*L1), component (i/L1)&1, limb r = i%L1;
//   out_c[r] = (acc_c[r] - ntt) * P^-1  (+ c0[r] gathered by the Galois map of g for component 0)
//              (+ self_c[r], ungathered: the ciphertext itself for a rotate-and-sum step, the
//                 tensor-product parts d0, d1 for a relinearisation).
struct ModDownEpilogue {
    const u64* acc;      // [J][2][R][N]
    const u64* pinv;     // [nq]
    const u64* pinv_sh;
    uint32_t R, L1;
    const u64* c0[HE_MAX_KS_JOBS];      // [L1][N] or nullptr (plain key switch)
    const u64* self0[HE_MAX_KS_JOBS];   // [L1][N] or nullptr: added to out0 as is
    const u64* self1[HE_MAX_KS_JOBS];   // [L1][N] or nullptr: added to out1 as is
    u64* out0[HE_MAX_KS_JOBS];
    u64* out1[HE_MAX_KS_JOBS];
    uint32_t g[HE_MAX_KS_JOBS];
    // small rings only (smallring.hip), whose kernel computes the accumulator itself: sum_j digit_j (gathered by the Galois map) *
    // evk_j, digit j's own limbs taken from the switched polynomial
    uint32_t beta, alpha, M;
    const u64* raised[HE_MAX_KS_JOBS];  // [beta][R][N]
    const u64* own[HE_MAX_KS_JOBS];     // [L1][N]
    const u64* evk[HE_MAX_KS_JOBS];     // [dnum][2][M][N]
};

// Row passes of key switches, or of one sum of rotations, with the inner products in them (ksrows.hip).  Special primes: mid
// [J][2][k][N] receives the inverse rows of the inner products; q-limbs: mid [J][2][L1][N] holds the converted part in the state the
// forward column pass leaves it, outputs as in ModDownEpilogue.  Digits are transformed already (done) or in the state the column
// pass leaves them.
#define KS_ROW_PRODUCTS 7           // products in one sum (modarith.h)
struct KsRows {
    const u64* raised[HE_MAX_KS_JOBS];  // [beta][R][N], by job (sum: by term, as own, evk and g)
    const u64* own[HE_MAX_KS_JOBS];     // [L1][N]
    const u64* evk[HE_MAX_KS_JOBS];     // [dnum][2][M][N]
    const u64* c0[HE_MAX_KS_JOBS];
    const u64* self0[HE_MAX_KS_JOBS];
    const u64* self1[HE_MAX_KS_JOBS];
    u64* out0[HE_MAX_KS_JOBS];
    u64* out1[HE_MAX_KS_JOBS];
    u64* next[HE_MAX_KS_JOBS];          // receives the inverse rows of out1 (null: not wanted)
    uint32_t g[HE_MAX_KS_JOBS];
    u64* mid;
    const u64* pinv;     // [nq]
    const u64* pinv_sh;
    uint32_t J, n_terms, beta, alpha, R, M, L1, k, nq;
    uint32_t sum;                       // one output (J = 1), the sum over n_terms terms; else n_terms = 1
    uint32_t done;                      // the digits' rows are transformed already
    uint32_t count_up, count_down;      // whether the digits' / the ModDown's transforms are counted with these rows
    // set by the launch
    uint32_t logN;
    u64 width[3];        // ks_width
    const ModConst* mc;
    const ulonglong2 *tw, *itw;
};
int32_t launch_ks_rows(he_ctx* ctx, KsRows& a, bool special);

// One batched transform launch (both passes).  Limb i is read at seg[src_seg[i]] + src_limb[i]*N
// by the first pass and lives at dst + i*N afterwards; mod_idx[i] == 0xFF leaves limb i alone.
struct TransformDesc {
    bool fwd;
    const u64* seg[HE_MAX_SEGS];
    uint32_t n_seg;
    u64* dst;
    uint32_t n;                  // <= HE_MAX_LAUNCH_LIMBS
    const uint32_t* mod_idx;     // [n]
    const uint8_t* src_seg;      // [n] or nullptr (all segment 0)
    const uint16_t* src_limb;    // [n] (< 4096) or nullptr (identity)
    const ScaleList* scale;      // inverse only: limb i is multiplied by scale[i % scale_period]
    uint32_t scale_period;       //   (must include N^-1); nullptr = plain N^-1
    const ModDownEpilogue* ep;   // forward only, or nullptr
    bool lazy_out;               // forward only: outputs may stay below 2q for narrow moduli
                                 // (internal buffers whose consumers allow for it)
    uint32_t only_pass;          // two-launch transforms: 0 = both passes; 1 = the first pass only (inverse: rows, reading the
                                 // sources; forward: columns); 2 = the second pass only, in place at dst
    uint32_t rescale_from;       // two-launch transforms, forward only: l + 1 when the sources are coefficient-form limbs of
                                 // modulus l and limb i (modulus r) transforms ((t + h) mod q_l) mod q_r - (h mod q_r),
                                 // h = floor(q_l / 2): the rounding term of Rescale, negated; 0 = sources as they are
};

// Basis conversion with the column passes around it (colconv.hip).  Set s (a digit of ModUp; the special primes of ModDown):
// sources src + rep*src_stride + i*N (i < ns, moduli mod0 + i, output scaling sc entry sc0 + i) in the state the inverse
// row pass leaves them; target t has modulus mod[t] and is written, in the state the forward column pass leaves it, at
// dst + rep*dst_stride + limb[t]*N.  op: conversion constants per modulus.
// The arrays of bytes start at multiples of 8 and are read eight at a time: a scalar load of a narrower field could be split
// into a base and an offset register that are each misaligned, whose low bits the hardware drops one by one.
#define CC_MAX_SETS 8
struct ColConvSet {
    const u64* src;
    u64* dst;
    const ConvOperand* op;     // [modulus]
    uint32_t ns, mod0, sc0, nt;
    uint8_t limb[HE_MAX_MODULI], mod[HE_MAX_MODULI];
};
struct ColConv {
    ColConvSet set[CC_MAX_SETS];
    size_t src_stride, dst_stride;
    ModClasses fwd, inv;
    uint32_t n_sets;
    uint32_t share;            // targets of a work group of those that share a tile (set by the launch)
};
int32_t launch_col_conv(he_ctx* ctx, ColConv& cc, const ScaleList& sc, uint32_t reps, uint32_t limb_passes);
// Column passes of Rescale (rescale.hip): src [n][N] holds the dropped limbs (modulus `level`) in the state the inverse row pass
// leaves them, dst [n][level][N] receives the negated rounding terms in the state the forward column pass leaves them.
struct RescaleCols {
    const u64* src;
    u64* dst;
    uint32_t level, parts, share;      // work groups that share a tile's moduli, `share` each (set by the launch)
    ModClasses fwd, inv;
};
bool rescale_cols_pays(const he_ctx* ctx, uint32_t n, uint32_t level);
int32_t launch_rescale_cols(he_ctx* ctx, const u64* src, u64* dst, uint32_t n, uint32_t level);
// fills w / w_sh of entry i from s (modulus index mi)
void scale_entry(const he_ctx* c, ScaleList& sc, uint32_t i, uint32_t mi, u64 s);
int32_t launch_transform(he_ctx* ctx, const TransformDesc& d);
int32_t launch_transform2p(he_ctx* ctx, const TransformDesc& d);   // N = 2^13 .. 2^17 (ntt2p.hip)
int32_t probe_butterfly_rates(he_ctx* ctx, u64* d_out, uint32_t groups, double rate_out[3]);   // ntt2p.hip
int32_t launch_moddown_final(he_ctx* ctx, const u64* conv, uint32_t n_jobs, const ModDownEpilogue& ep);

// in-place conveniences
int32_t launch_ntt(he_ctx* ctx, u64* d, const uint32_t* mod_idx, uint32_t n);
int32_t launch_intt(he_ctx* ctx, u64* d, const uint32_t* mod_idx, uint32_t n, const ScaleList* scale);
int32_t launch_automorph_ntt(he_ctx* ctx, const u64* in, u64* out, uint32_t n_limbs, uint32_t g);
struct AffineConst {
    u64 mul[HE_MAX_MODULI], add[HE_MAX_MODULI];
};
int32_t launch_affine(he_ctx* ctx, const u64* ct, uint32_t level, const AffineConst& k, u64* out);   // out may alias ct
// Inverse rows that a launch takes along of polynomials it forms (out null: none), and what they need
struct RowsOut {
    u64* out;                            // [polynomials][limbs][N]
    const ulonglong2* itw;
    ModClasses inv;
};
static inline RowsOut rows_out(const he_ctx* ctx, u64* out) { return {out, ctx->d_itw, ctx->cls_inv}; }
// tensor squares of mul*u, n ciphertexts, and tensor products: d = [d0][d1][d2], each [level+1][N].  rows: receives the inverse rows of every d2 (null: not wanted)
int32_t launch_square_lift(he_ctx* ctx, const u64* u, uint32_t n, uint32_t level, const u64* mul, u64* d, u64* rows);
int32_t launch_tensor(he_ctx* ctx, const u64* a, const u64* b, uint32_t level, u64* d, u64* rows);
int32_t launch_automorph_coef(he_ctx* ctx, const u64* in, u64* out, const uint32_t* mod_idx, uint32_t n, uint32_t g);

// key switching engine (keyswitch.hip)
int32_t ks_init_tables(he_ctx* ctx);
void ks_free_tables(he_ctx* ctx);
struct KsSrc {
    const u64* c0;   // [level+1][N] or nullptr (plain key switch: nothing rotated is added to out0)
    const u64* c1;   // [level+1][N]: the polynomial that is raised and switched
    const u64* s0;   // [level+1][N] or nullptr: addends for jobs with add_self
    const u64* s1;
};
struct KsJob {
    uint32_t src;        // index into the sources
    uint32_t g;          // Galois element applied to the raised digits and to c0 (1 = none)
    const u64* evk;      // key used
    u64* out0;           // [level+1][N]
    u64* out1;
    uint32_t add_self;   // out0 += src.s0, out1 += src.s1 (rotate-and-sum step, relinearisation)
};
// Runs every job: one ModUp per source, then inner product + ModDown per job, batched.
// src_rows: ks_engine_src_rows holds the sources' inverse rows already; raised: their raised digits, which
// the call takes from there; raised_next: where the raised digits of the second components of its results go (sr_moddown_raises), for as many jobs,
// one a source and all under one key, as one launch set takes.  rows: [n_src][level+1][N] outside the engine's workspace, the sources' inverse
// rows; rows_next: receives those of the second components of its results, one job a source (both: ks_engine_next_rows; may be the same).
int32_t ks_engine(he_ctx* ctx, uint32_t level, const KsSrc* srcs, uint32_t n_src, const KsJob* jobs, uint32_t n_jobs, bool src_rows = false,
                  const u64* raised = nullptr, u64* raised_next = nullptr, u64* rows = nullptr, u64* rows_next = nullptr);
// Whether the engine raises all sources and runs all jobs at once; raised digits of n sources: ks_raised_elems
bool ks_engine_at_once(const he_ctx* ctx, uint32_t level, uint32_t n_src, uint32_t n_jobs);
size_t ks_raised_elems(const he_ctx* c, uint32_t level, uint32_t n);
// Where the inverse rows of the sources [n_src][level+1][N] go (in a workspace that is large enough), if the engine can start from them: its
// conversion does the columns, and it raises all sources at once.  Null otherwise.
u64* ks_engine_src_rows(const he_ctx* ctx, uint32_t level, uint32_t n_src, uint32_t n_jobs);
bool ks_engine_next_rows(const he_ctx* ctx, uint32_t level, uint32_t n_src, uint32_t n_jobs);
size_t ks_engine_ws_elems(const he_ctx* c, uint32_t level, uint32_t n_src, uint32_t n_jobs);
// Sum of rotations with one ModDown for the whole sum.  Terms with g == 1 are added as they are (evk unused).
#define HE_MAX_SUM_TERMS 49
struct KsSumTerm {
    const u64* c0;   // [level+1][N]
    const u64* c1;
    uint32_t g;
    const u64* evk;
};
size_t ks_rotate_sum_ws_elems(const he_ctx* c, uint32_t level, uint32_t n_rot);
int32_t ks_rotate_sum_deferred(he_ctx* c, uint32_t level, const KsSumTerm* terms, uint32_t n_terms, u64* out0, u64* out1, u64* ws, bool src_rows = false);
// The same for a sum of n_rot rotations of different ciphertexts, whose ws is the start of the workspace.
u64* ks_rotate_sum_src_rows(const he_ctx* c, uint32_t level, uint32_t n_rot);
// sum over T shared (Galois element, key) terms of the rotations of each of J ciphertexts, one ModUp and one ModDown per
// ciphertext; srcs[j] = {c0_j, c1_j, addend0_j or null, addend1_j or null} (keyswitch.hip)
size_t ks_hoisted_sum_ws_elems(const he_ctx* c, uint32_t level, uint32_t J, uint32_t T);
int32_t ks_hoisted_sum(he_ctx* c, uint32_t level, const KsSrc* srcs, uint32_t J, const uint32_t* gs, const u64* const* evks, uint32_t T,
                       u64* const* out0, u64* const* out1, u64* ws);
// Hoisted inner products kept over the raised basis, and the ModDown of stored accumulators (keyswitch.hip)
size_t ks_raised_products_ws_elems(const he_ctx* c, uint32_t level);
int32_t ks_raised_products(he_ctx* c, uint32_t level, const u64* c1, const uint32_t* gs, const u64* const* evks, uint32_t n, u64* acc, u64* ws);
size_t ks_moddown_stored_ws_elems(const he_ctx* c, uint32_t level, uint32_t J);
int32_t ks_moddown_stored(he_ctx* c, uint32_t level, uint32_t J, u64* acc, const u64* const* add0, const u64* const* add1,
                          u64* const* out0, u64* const* out1, u64* ws);
// Latency path for rings whose limb fits one work group's LDS (smallring.hip)
bool small_ring_path(const he_ctx* c, uint32_t level);
int32_t sr_modup(he_ctx* c, const KsSrc* srcs, uint32_t cb, uint32_t level, u64* raised);
// raised_next [J][beta][R][N] or null: in the same launch, the ModUp of the second components it leaves
bool sr_moddown_raises(const he_ctx* c, uint32_t level);
int32_t sr_moddown(he_ctx* c, uint32_t level, uint32_t J, const ModDownEpilogue& ep, u64* raised_next = nullptr);
// Rescale of n ciphertexts at `level` and, in the same launch, the ModUp of the second components it leaves, to raised [n][beta][R][N]
bool sr_rescale_raises(const he_ctx* c, uint32_t level, uint32_t n);
int32_t sr_rescale_modup(he_ctx* c, const u64* const* cts, u64* const* outs, uint32_t n, uint32_t level, u64* raised);
int32_t sr_rescale(he_ctx* c, const u64* const* cts, u64* const* outs, uint32_t n, uint32_t level);
size_t rescale_ws_elems(const he_ctx* c, uint32_t level, uint32_t n);
int32_t rescale_batch(he_ctx* ctx, const u64* const* cts, u64* const* outs, uint32_t n, uint32_t level, u64* ws);
