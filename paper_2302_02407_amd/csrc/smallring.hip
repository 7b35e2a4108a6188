// Latency path for rings whose limb fits one work group's LDS (N <= 2^12, 32 KiB): a key switch in two launches
// and a rescale in one.  At these sizes a call is bound by the chain of dependent launches and, inside a launch,
// by the chain of dependent memory round trips, not by arithmetic.  So each work group produces one OUTPUT limb
// from start to finish, recomputing what it shares with its neighbours instead of exchanging it through memory,
// and issues every global load it will need before it starts computing: operands at the top of the kernel,
// each transform's twiddle table one transform ahead (into registers, then into LDS, where the stages read it).
//   ModUp    (hybrid key switching, paper Appendix: evaluation keys, dnum): work group (source, digit j, target
//            limb r) inverse-transforms the digit's <= 4 limbs in LDS, accumulates the basis conversion to r in
//            registers, transforms forward and writes raised_j[r];
//   ModDown  work group (job, component, q-limb r) forms the inner products of limb r and of every special-prime
//            limb from the operands it loaded (digits gathered by the Galois map), inverse-transforms the
//            special-prime ones in LDS, accumulates the conversion to r, transforms forward and writes
//            (acc - conv) * P^-1 (+ rotated c0) (+ addend);
//   Rescale  (Section 2.1) work group (ciphertext, component, limb r) inverse-transforms the dropped limb,
//            forms the correction term modulo q_r, transforms it forward and writes (c_r + delta) * q_l^-1.
// The arithmetic is the engine's (same digits, same conversion without overflow correction, same ModDown without
// rounding term), so the results are the same bits as the multi-launch path that larger rings and wider digits take.
#include "modarith.h"
#include "ntt_blocks.h"

#define SR_THREADS 1024
#define SR_PTS 4          // points per thread: 1024 threads x 4 = the largest limb (2^12)
#define SR_MAX_SRC 4      // limbs per digit and special primes this path handles
#define SR_LDS (4096 + 256)

// LDS position of element i: one spare slot per 16 spreads the strided accesses of the late stages over the banks.
__device__ __forceinline__ uint32_t sp(uint32_t i) { return i + (i >> 4); }

// A twiddle table (N factors and their Shoup companions) on its way from memory to LDS: fetched into registers
// while the previous transform still uses the LDS copy, committed once that transform is done.
struct TwRegs { u64 w[SR_PTS], s[SR_PTS]; };

__device__ __forceinline__ void tw_fetch(TwRegs& r, const ulonglong2* __restrict__ tw, uint32_t N) {
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        if (e < N) { const ulonglong2 v = tw[e]; r.w[p] = v.x; r.s[p] = v.y; }
    }
}
__device__ __forceinline__ void tw_commit(const TwRegs& r, ulonglong2* twl, uint32_t N) {
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        if (e < N) twl[e] = make_ulonglong2(r.w[p], r.s[p]);
    }
}

// Two stages on 4 points, factors with Shoup's companion from the LDS table.  Forward: wide moduli below 16q in and out, others up by 8q.
// Inverse: below 4q in and out, for any modulus below 2^60.
__device__ __forceinline__ void sr_ct(u64& X, u64& Y, u64 w, u64 w_sh, u64 q) {
    const u64 S = shoup_acc(X, Y, w, w_sh, q);
    Y = (X + X + 4 * q) - S;
    X = S;
}
__device__ __forceinline__ void sr_gs(u64& X, u64& Y, u64 bq, u64 w, u64 w_sh, u64 q) {
    const u64 d = (X + bq) - Y;
    X = X + Y;
    Y = shoup_lazy4(d, w, w_sh, q);
}
template <bool WIDE>
__device__ __forceinline__ void sr_fwd2(u64 (&x)[4], const ulonglong2* tw, uint32_t s0, uint32_t G, u64 q) {
    u64 r[6];
    tw_block2(r, tw, s0, G);
    if (WIDE) { x[0] = csub_u(x[0], 8 * q); x[1] = csub_u(x[1], 8 * q); }
    sr_ct(x[0], x[2], r[0], r[1], q);
    sr_ct(x[1], x[3], r[0], r[1], q);
    sr_ct(x[0], x[1], r[2], r[3], q);
    sr_ct(x[2], x[3], r[4], r[5], q);
}
__device__ __forceinline__ void sr_inv2(u64 (&x)[4], const ulonglong2* tw, uint32_t s0, uint32_t G, u64 q) {
    u64 r[6];
    tw_block2(r, tw, s0, G);
    sr_gs(x[0], x[1], 4 * q, r[2], r[3], q);
    sr_gs(x[2], x[3], 4 * q, r[4], r[5], q);
    sr_gs(x[0], x[2], 8 * q, r[0], r[1], q);
    sr_gs(x[1], x[3], 4 * q, r[0], r[1], q);
    x[0] = csub_u(csub_u(x[0], 8 * q), 4 * q);
    x[1] = csub_u(x[1], 4 * q);
}

// Forward transform of the whole limb in LDS (decimation in time, psi folded into the twiddles; natural order in,
// bit-reversed out): register blocks of two stages on 4 points per thread with one LDS exchange between blocks,
// then one radix-2 stage when logN is odd.  Twiddles from the LDS table.  Inputs below 4q, results canonical.
// Ends with a barrier.
template <bool WIDE>
__device__ __forceinline__ void lds_ntt_fwd_t(u64* sm, const ulonglong2* twl, const ModConst& m, uint32_t logN) {
    const u64 q = m.q, q2 = 2 * q;
    const uint32_t N = 1u << logN, nb = logN >> 1;
    // the blocks leave values below 52q (never reduced) or, for the widest moduli, below 16q
    for (uint32_t blk = 0; blk < nb; blk++) {
        const uint32_t s0 = 2 * blk, log_span = logN - s0 - 2, span = 1u << log_span;
        for (uint32_t tid = threadIdx.x; tid < (N >> 2); tid += SR_THREADS) {
            const uint32_t G = tid >> log_span, off = tid & (span - 1), base = (G << (logN - s0)) + off;
            u64 x[4];
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = sm[sp(base + (k << log_span))];
            sr_fwd2<WIDE>(x, twl, s0, G, q);
            if (blk + 1 == nb) {
#pragma unroll
                for (int k = 0; k < 4; k++) x[k] = reduce_full<7>(x[k], q, m.bits, m.rec);
            }
#pragma unroll
            for (int k = 0; k < 4; k++) sm[sp(base + (k << log_span))] = x[k];
        }
        __syncthreads();
    }
    if (logN & 1u) {
        const uint32_t s = logN - 1;
        for (uint32_t b = threadIdx.x; b < (N >> 1); b += SR_THREADS) {
            const uint32_t e0 = sp(2 * b), e1 = sp(2 * b + 1), k = (1u << s) + b;
            const u64 x = sm[e0];
            const u64 v = shoup_lazy(sm[e1], twl[k].x, twl[k].y, q);
            sm[e0] = csub(csub(x + v, q2), q);
            sm[e1] = csub(csub(x - v + q2, q2), q);
        }
        __syncthreads();
    }
}
__device__ __forceinline__ void lds_ntt_fwd(u64* sm, const ulonglong2* twl, const ModConst& m, uint32_t logN) {
    if (m.bits > 57) lds_ntt_fwd_t<true>(sm, twl, m, logN);
    else lds_ntt_fwd_t<false>(sm, twl, m, logN);
}

// Inverse transform in LDS (bit-reversed in, natural out): the last stage as a radix-2 stage first when logN is
// odd, then the register blocks from the highest stages down; every value times `scale` (which carries N^-1) as
// the last block stores it.  Inputs canonical, results canonical.  Ends with a barrier.
__device__ __forceinline__ void lds_ntt_inv(u64* sm, const ulonglong2* twl, const ModConst& m, uint32_t logN, u64 scale,
                                            u64 scale_sh) {
    const u64 q = m.q, q2 = 2 * q;
    const uint32_t N = 1u << logN, nb = logN >> 1;
    if (logN & 1u) {
        const uint32_t s = logN - 1;
        for (uint32_t b = threadIdx.x; b < (N >> 1); b += SR_THREADS) {
            const uint32_t e0 = sp(2 * b), e1 = sp(2 * b + 1), k = (1u << s) + b;
            const u64 x = sm[e0], y = sm[e1];
            sm[e0] = csub(x + y, q2);
            sm[e1] = shoup_lazy(x - y + q2, twl[k].x, twl[k].y, q);
        }
        __syncthreads();
    }
    for (uint32_t blk = nb; blk-- > 0;) {
        const uint32_t s0 = 2 * blk, log_span = logN - s0 - 2, span = 1u << log_span;
        for (uint32_t tid = threadIdx.x; tid < (N >> 2); tid += SR_THREADS) {
            const uint32_t G = tid >> log_span, off = tid & (span - 1), base = (G << (logN - s0)) + off;
            u64 x[4];
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = sm[sp(base + (k << log_span))];
            sr_inv2(x, twl, s0, G, q);
            if (blk == 0) {
#pragma unroll
                for (int k = 0; k < 4; k++) x[k] = csub(shoup_lazy(x[k], scale, scale_sh, q), q);
            }
#pragma unroll
            for (int k = 0; k < 4; k++) sm[sp(base + (k << log_span))] = x[k];
        }
        __syncthreads();
    }
}

__device__ __forceinline__ uint32_t galois_src_sr(uint32_t j, uint32_t g, uint32_t logN) {
    uint32_t k = __brev(j) >> (32 - logN);
    uint32_t kp = (g * k + ((g - 1) >> 1)) & ((1u << logN) - 1);
    return __brev(kp) >> (32 - logN);
}

struct SrTables {
    const ModConst* mc;
    const ulonglong2 *tw, *itw;   // [M][N]: factor, Shoup companion
    const double *ftw, *fitw;     // [M][N]: the factors in the FP64 kernels' order (ctx.hip, ftw_pos), where those run
    uint32_t logN;
};

// ---------------------------------------------------------------- ModUp
struct SrUpArgs {
    const u64* c1[HE_MAX_KS_JOBS]; // sources [L1][N], NTT form
    u64* raised;               // [n_src][beta][R][N]; a digit's own limbs are left unwritten
    const u64* hat;            // conversion constants [digit][size-1][modulus][i padded to aw]
    u64 scale[HE_MAX_MODULI];  // per source limb: N^-1 * (Q_j/q_i)^-1 mod q_i, and its Shoup companion
    u64 scale_sh[HE_MAX_MODULI];
    uint32_t L1, R, beta, alpha, M, nq, level, aw, n_out;   // n_out = output limbs per source
    uint8_t oj[512], orr[512]; // output o of a source: digit, raised-basis limb
};

__global__ __launch_bounds__(SR_THREADS) void sr_modup_kernel(SrUpArgs a, SrTables tb) {
    __shared__ u64 sm[SR_LDS];
    __shared__ ulonglong2 twl[4096];
    const uint32_t N = 1u << tb.logN;
    const uint32_t s = blockIdx.x / a.n_out, o = blockIdx.x % a.n_out;
    const uint32_t j = a.oj[o], r = a.orr[o];
    const uint32_t lo = j * a.alpha, sz = min(a.alpha, a.L1 - lo);
    const uint32_t mr = r <= a.level ? r : a.nq + (r - a.level - 1);
    const ModConst m = tb.mc[mr];
    const u64* hat = a.hat + ((size_t)(j * a.alpha + (sz - 1)) * a.M + mr) * a.aw;
    // every operand first: the digit's limbs (points e = threadIdx.x + 1024 p), the first table
    u64 in[SR_MAX_SRC][SR_PTS];
    u64 h[SR_MAX_SRC];
#pragma unroll
    for (uint32_t i = 0; i < SR_MAX_SRC; i++) {
        const u64* src = a.c1[s] + ((size_t)(lo + (i < sz ? i : 0)) << tb.logN);
        h[i] = i < sz ? hat[i] : 0;
#pragma unroll
        for (uint32_t p = 0; p < SR_PTS; p++) {
            const uint32_t e = threadIdx.x + SR_THREADS * p;
            in[i][p] = (i < sz && e < N) ? src[e] : 0;
        }
    }
    TwRegs tr;
    tw_fetch(tr, tb.itw + ((size_t)lo << tb.logN), N);
    u128 acc[SR_PTS] = {};
#pragma unroll
    for (uint32_t i = 0; i < SR_MAX_SRC; i++) {
        if (i < sz) {
            const uint32_t mi = lo + i;
            const ModConst mq = tb.mc[mi];
#pragma unroll
            for (uint32_t p = 0; p < SR_PTS; p++) {
                const uint32_t e = threadIdx.x + SR_THREADS * p;
                if (e < N) sm[sp(e)] = in[i][p];
            }
            tw_commit(tr, twl, N);
            __syncthreads();
            // the table of the next transform travels while this one runs
            if (i + 1 < sz) tw_fetch(tr, tb.itw + ((size_t)(mi + 1) << tb.logN), N);
            else tw_fetch(tr, tb.tw + ((size_t)mr << tb.logN), N);
            lds_ntt_inv(sm, twl, mq, tb.logN, a.scale[mi], a.scale_sh[mi]);
#pragma unroll
            for (uint32_t p = 0; p < SR_PTS; p++) {
                const uint32_t e = threadIdx.x + SR_THREADS * p;
                if (e < N) acc[p] += (u128)sm[sp(e)] * h[i];
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        if (e < N) sm[sp(e)] = barrett128(acc[p], m.q, m.mu, m.bits);
    }
    tw_commit(tr, twl, N);
    __syncthreads();
    lds_ntt_fwd(sm, twl, m, tb.logN);
    u64* dst = a.raised + ((size_t)((s * a.beta + j) * a.R + r) << tb.logN);
    for (uint32_t e = threadIdx.x; e < N; e += SR_THREADS) dst[e] = sm[sp(e)];
}

// A launch whose first work groups rescale or bring down, and whose others raise what comes of it: per source limb of the ModUp (d Q_j/q_i)^-1
// mod q_i, d = q_l or P
struct SrRaise {
    uint32_t first;
    u64 factor[HE_MAX_MODULI];
};

// ---------------------------------------------------------------- inner product + ModDown
struct SrDownArgs {
    const u64* dn_hat;         // [M][pw]: (P/p_t) mod modulus
    u64 scale[SR_MAX_SRC];     // N^-1 * (P/p_t)^-1 mod p_t and Shoup companions
    u64 scale_sh[SR_MAX_SRC];
    uint32_t k, nq, level, pw;
};

__global__ __launch_bounds__(SR_THREADS) void sr_moddown_kernel(ModDownEpilogue ep, SrDownArgs a, SrTables tb) {
    __shared__ u64 sm[SR_LDS];
    __shared__ ulonglong2 twl[4096];
    const uint32_t N = 1u << tb.logN, L1 = ep.L1, R = ep.R, beta = ep.beta;
    const uint32_t pc = blockIdx.x / L1, r = blockIdx.x - pc * L1, job = pc >> 1, comp = pc & 1u;
    const ModConst m = tb.mc[r];
    const uint32_t g = ep.g[job];
    const u64* raised = ep.raised[job];
    const u64* evk = ep.evk[job];
    TwRegs tr;
    tw_fetch(tr, tb.itw + ((size_t)a.nq << tb.logN), N);
    uint32_t src[SR_PTS];
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        src[p] = (e < N && g != 1) ? galois_src_sr(e, g, tb.logN) : e;
    }
    // every inner product first, so that all operand loads are in flight together: limb r of the accumulator (digit
    // j's own limbs come from the switched polynomial itself), the epilogue's addends, the special-prime limbs
    const uint32_t own_j = r / ep.alpha;
    const u64* own = ep.own[job] + ((size_t)r << tb.logN);
    const u64* c0 = (comp == 0 && ep.c0[job]) ? ep.c0[job] + ((size_t)r << tb.logN) : nullptr;
    const u64* self = comp ? ep.self1[job] : ep.self0[job];
    u64 aq[SR_PTS], add0[SR_PTS], add1[SR_PTS], pl[SR_MAX_SRC][SR_PTS];
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        aq[p] = add0[p] = add1[p] = 0;
        if (e < N) {
            u128 sum = 0;
            for (uint32_t j = 0; j < beta; j++) {
                const u64 d = j == own_j ? own[src[p]] : raised[((size_t)(j * R + r) << tb.logN) + src[p]];
                sum += (u128)d * evk[((size_t)((j * 2 + comp) * ep.M + r) << tb.logN) + e];
            }
            aq[p] = barrett128(sum, m.q, m.mu, m.bits);
            if (c0) add0[p] = c0[src[p]];
            if (self) add1[p] = self[((size_t)r << tb.logN) + e];
        }
    }
#pragma unroll
    for (uint32_t t = 0; t < SR_MAX_SRC; t++) {
        const uint32_t mt = a.nq + (t < a.k ? t : 0);
        const ModConst mp = tb.mc[mt];
#pragma unroll
        for (uint32_t p = 0; p < SR_PTS; p++) {
            const uint32_t e = threadIdx.x + SR_THREADS * p;
            pl[t][p] = 0;
            if (t < a.k && e < N) {
                u128 sum = 0;
                for (uint32_t j = 0; j < beta; j++)
                    sum += (u128)raised[((size_t)(j * R + L1 + t) << tb.logN) + src[p]] *
                           evk[((size_t)((j * 2 + comp) * ep.M + mt) << tb.logN) + e];
                pl[t][p] = barrett128(sum, mp.q, mp.mu, mp.bits);
            }
        }
    }
    u128 acc[SR_PTS] = {};
#pragma unroll
    for (uint32_t t = 0; t < SR_MAX_SRC; t++) {
        if (t < a.k) {
            const uint32_t mt = a.nq + t;
            const ModConst mp = tb.mc[mt];
#pragma unroll
            for (uint32_t p = 0; p < SR_PTS; p++) {
                const uint32_t e = threadIdx.x + SR_THREADS * p;
                if (e < N) sm[sp(e)] = pl[t][p];
            }
            tw_commit(tr, twl, N);
            __syncthreads();
            if (t + 1 < a.k) tw_fetch(tr, tb.itw + ((size_t)(mt + 1) << tb.logN), N);
            else tw_fetch(tr, tb.tw + ((size_t)r << tb.logN), N);
            lds_ntt_inv(sm, twl, mp, tb.logN, a.scale[t], a.scale_sh[t]);
            const u64 h = a.dn_hat[(size_t)r * a.pw + t];
#pragma unroll
            for (uint32_t p = 0; p < SR_PTS; p++) {
                const uint32_t e = threadIdx.x + SR_THREADS * p;
                if (e < N) acc[p] += (u128)sm[sp(e)] * h;
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        if (e < N) sm[sp(e)] = barrett128(acc[p], m.q, m.mu, m.bits);
    }
    tw_commit(tr, twl, N);
    __syncthreads();
    lds_ntt_fwd(sm, twl, m, tb.logN);
    u64* out = (comp ? ep.out1[job] : ep.out0[job]) + ((size_t)r << tb.logN);
    const u64 pinv = ep.pinv[r], pinv_sh = ep.pinv_sh[r];
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        if (e < N) {
            u64 v = shoup_mul(submod(aq[p], sm[sp(e)], m.q), pinv, pinv_sh, m.q);
            if (c0) v = addmod(v, add0[p], m.q);
            if (self) v = addmod(v, add1[p], m.q);
            out[e] = v;
        }
    }
}

// ---------------------------------------------------------------- rescale
struct SrRescaleArgs {
    const u64* ct[HE_MAX_KS_JOBS];   // [2][level+1][N]
    u64* out[HE_MAX_KS_JOBS];        // [2][level][N]
    const u64 *qlinv, *qlinv_sh;     // q_level^-1 mod q_r
    uint32_t level;
};

__global__ __launch_bounds__(SR_THREADS) void sr_rescale_kernel(SrRescaleArgs a, SrTables tb) {
    __shared__ u64 sm[SR_LDS];
    __shared__ ulonglong2 twl[4096];
    const uint32_t N = 1u << tb.logN, level = a.level;
    const uint32_t jc = blockIdx.x / level, r = blockIdx.x - jc * level, job = jc >> 1, comp = jc & 1u;
    const ModConst ml = tb.mc[level], mr = tb.mc[r];
    const u64* top = a.ct[job] + ((size_t)(comp * (level + 1) + level) << tb.logN);
    const u64* in = a.ct[job] + ((size_t)(comp * (level + 1) + r) << tb.logN);
    const u64 qlinv = a.qlinv[r], qlinv_sh = a.qlinv_sh[r];
    TwRegs tr;
    tw_fetch(tr, tb.itw + ((size_t)level << tb.logN), N);
    u64 cr[SR_PTS];
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        cr[p] = 0;
        if (e < N) { sm[sp(e)] = top[e]; cr[p] = in[e]; }
    }
    tw_commit(tr, twl, N);
    __syncthreads();
    tw_fetch(tr, tb.tw + ((size_t)r << tb.logN), N);
    lds_ntt_inv(sm, twl, ml, tb.logN, ml.ninv, ml.ninv_sh);
    const u64 h = ml.q >> 1, hr = barrett64(h, mr.q, mr.mu, mr.bits);
    for (uint32_t e = threadIdx.x; e < N; e += SR_THREADS) {
        const u64 t = addmod(sm[sp(e)], h, ml.q);
        sm[sp(e)] = submod(hr, barrett64(t, mr.q, mr.mu, mr.bits), mr.q);
    }
    tw_commit(tr, twl, N);
    __syncthreads();
    lds_ntt_fwd(sm, twl, mr, tb.logN);
    u64* out = a.out[job] + ((size_t)(comp * level + r) << tb.logN);
#pragma unroll
    for (uint32_t p = 0; p < SR_PTS; p++) {
        const uint32_t e = threadIdx.x + SR_THREADS * p;
        if (e < N) out[e] = shoup_mul(addmod(cr[p], sm[sp(e)], mr.q), qlinv, qlinv_sh, mr.q);
    }
}

// ---------------------------------------------------------------- moduli of at most 45 bits: FP64
// One double holds any value below 2^53, so a twiddle product modulo q is h = y*w, l = y*w - h (exact by FMA), b = h/q
// rounded to an integer, d = (h - b*q) + l: seven FP64 instructions (16 multiply-adds in 64-bit integers), all at full rate
// and five deep where the integer chain is fifteen deep: these launches run two wavefronts per SIMD at most, so the
// depth is what they wait for.  Every step is exact on integers: h - b*q is a multiple of 1 below 2^53, and only the choice of b depends on a rounding.
//   With |y| < 2^49 and moduli below 2^45 the quotient is within 1/2 + 2^-3 of h/q, so |d| < 0.63 q.
//   Forward: a stage adds 0.63 q; inputs below 2q end below 10q < 2^49.  Inverse: three stages turn values below q into
//   sums below 8q < 2^48, then the sums are brought below 0.63 q again.
// A limb is 8 points per thread in register blocks of 3 stages (512 threads at N = 2^12: 2 wavefronts per SIMD, 256
// registers, nothing spilled).  Block b of thread t = G*R + r, R = N/8^(b+1), holds points G*8R + k*R + r; the last block, where
// LN is no multiple of 3, the 8 points 8t + k and only its last stages.  From block 1 on a wavefront holds the same
// 512 points in every block, so one barrier per transform is left; transformed limbs are read and written at 8t + k.
// N = 2^12, one 40-bit limb per digit, one special prime (three digits): ModUp 9.6 us, ModDown 14.6, rescale 8.6, where the integer
// kernels above take 20, 29 and 20; what is left is the operands (a compute unit takes 64 bytes a cycle: 400 KB in 2.6 us), inner
// products of 1.8 us a limb, and transforms of 2.4 to 3.0 us, a compute unit's FP64 rate.
#pragma clang fp contract(off)
#define SRF_LDS(LN) ((1 << (LN)) + (1 << ((LN) - 3)))
#define SRF_DIG 3                  // digits whose operands are requested together
#define EACH8(k) _Pragma("unroll") for (int k = 0; k < 8; k++)

struct FMod { double q, qi; u64 n; };
__device__ __forceinline__ FMod f_mod(const ModConst& m) { return {(double)m.q, m.qinv, m.q}; }
__device__ __forceinline__ double f_of(u64 v) { return __longlong_as_double((long long)(v | 0x4330000000000000ull)) - 4503599627370496.0; }   // v < 2^52
__device__ __forceinline__ double f_round(double v) { return (v + 6755399441055744.0) - 6755399441055744.0; }                              // |v| < 2^51
__device__ __forceinline__ double f_mul(double y, double w, const FMod& m) {
    const double h = y * w, l = __builtin_fma(y, w, -h);
    const double b = __builtin_fma(h, m.qi, 6755399441055744.0) - 6755399441055744.0;
    return __builtin_fma(-b, m.q, h) + l;
}
__device__ __forceinline__ double f_red(double x, const FMod& m) { return __builtin_fma(-f_round(x * m.qi), m.q, x); }
__device__ __forceinline__ u64 f_canon(double d, const FMod& m) {                      // |d| < q
    const long long i = __double_as_longlong(d + 6755399441055744.0) - 0x4338000000000000ll;
    return (u64)(i + ((i >> 63) & (long long)m.n));
}
__device__ __forceinline__ double f_nonneg(double d, const FMod& m) { return d < 0 ? d + m.q : d; }

template <int LN>
struct Srf {
    static constexpr uint32_t N = 1u << LN, T = N / 8;
    static constexpr int NB = (LN + 2) / 3, U0 = 3 * NB - LN;      // blocks; first stage of the last one
    static __device__ __forceinline__ uint32_t word(uint32_t e) { return e + (e >> 3); }
    static constexpr uint32_t R(int b) { return b + 1 < NB ? N >> (3 * b + 3) : 1; }
    static __device__ __forceinline__ uint32_t pos(int b, uint32_t t, uint32_t k) { return word(t / R(b) * (8 * R(b)) + k * R(b) + t % R(b)); }
    static constexpr int s0(int b) { return b + 1 < NB ? 3 * b : LN - 3; }
    static constexpr int u0(int b) { return b + 1 < NB ? 0 : U0; }
};
// The 8W points of a wavefront (W lanes; half of one at N = 2^8) between memory and its transform: read and written in pairs at
// 2l + 2W*i of lane l, so that every access is one run of 16 W bytes, and turned into the transform's order in LDS.  A Galois
// map takes aligned runs of 2^m positions to aligned runs, so a wavefront's points come from the points of one wavefront:
// digits and rotated addends are read as they lie and permuted there too, with no barrier.  What a lane reads for itself at
// 8t + k (or gathers) is 64 lines an instruction in the first-level cache, which takes one a cycle; with all of it read that way
// ModUp took 10.7 us instead of 9.6, ModDown 18.2 instead of 14.6, rescale 9.9 instead of 8.6.
template <int LN>
struct SrfRow {
    using G = Srf<LN>;
    static constexpr uint32_t W = G::T < 64 ? G::T : 64, S = 8 * W;
    uint32_t l, wb;                                    // lane, the wavefront's first point
    __device__ __forceinline__ explicit SrfRow(uint32_t t) : l(t % W), wb(t / W * S) {}
    static __device__ __forceinline__ uint32_t at(uint32_t e) { return e ^ ((e >> 5 & 3u) << 1); }      // 16-byte accesses to different banks
    template <class V>
    __device__ __forceinline__ V* words(double* sm) const { return reinterpret_cast<V*>(sm + G::word(wb)); }
    __device__ __forceinline__ void load(u64 (&v)[8], const u64* __restrict__ p) const {                // p: the wavefront's first point
#pragma unroll
        for (int i = 0; i < 4; i++) { const ulonglong2 u = LOAD2(p + 2 * l + 2 * W * i); v[2 * i] = u.x; v[2 * i + 1] = u.y; }
    }
    __device__ __forceinline__ void store(u64* p, const u64 (&v)[8]) const {
#pragma unroll
        for (int i = 0; i < 4; i++) STORE2(p + 2 * l + 2 * W * i) = make_ulonglong2(v[2 * i], v[2 * i + 1]);
    }
    // values in pairs <-> values at 8t + k, through the wavefront's words of LDS
    template <class V>
    __device__ __forceinline__ void pairs_in(const V (&v)[8], double* sm) const {
#pragma unroll
        for (int i = 0; i < 4; i++) { V* w = words<V>(sm) + at(2 * l + 2 * W * i); w[0] = v[2 * i]; w[1] = v[2 * i + 1]; }
        wave_exchange();
    }
    template <class V>
    __device__ __forceinline__ void to_own(V (&v)[8], double* sm) const {
        pairs_in(v, sm);
#pragma unroll
        for (int i = 0; i < 4; i++) { const V* w = words<V>(sm) + at(8 * l + 2 * i); v[2 * i] = w[0]; v[2 * i + 1] = w[1]; }
        wave_exchange();
    }
    template <class V>
    __device__ __forceinline__ void to_pairs(V (&v)[8], double* sm) const {
        wave_exchange();
#pragma unroll
        for (int i = 0; i < 4; i++) { V* w = words<V>(sm) + at(8 * l + 2 * i); w[0] = v[2 * i]; w[1] = v[2 * i + 1]; }
        wave_exchange();
#pragma unroll
        for (int i = 0; i < 4; i++) { const V* w = words<V>(sm) + at(2 * l + 2 * W * i); v[2 * i] = w[0]; v[2 * i + 1] = w[1]; }
    }
};
// Where the Galois image of a wavefront's points comes from: its first point, and the words of the lane's pairs in it.
template <int LN>
struct SrfGalois {
    uint32_t first, src[4];
    __device__ __forceinline__ SrfGalois(const SrfRow<LN>& row, uint32_t g) {
        using Q = SrfRow<LN>;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t s = galois_src_sr(row.wb + 2 * row.l + 2 * Q::W * i, g, LN);
            first = __builtin_amdgcn_readfirstlane(s & ~(Q::S - 1));
            src[i] = Q::at(s & (Q::S - 1));
        }
    }
    __device__ __forceinline__ void apply(u64 (&v)[8], const SrfRow<LN>& row, double* sm) const {
        row.pairs_in(v, sm);
        const u64* w = row.template words<u64>(sm);
#pragma unroll
        for (int i = 0; i < 4; i++) { v[2 * i] = w[src[i]]; v[2 * i + 1] = w[src[i] ^ 1u]; }             // aligned pairs come from aligned pairs
        wave_exchange();
    }
};
// Factors of a transform's blocks.
template <int LN>
struct SrfTw { double w[Srf<LN>::NB][7]; };
template <int LN, int B>
__device__ __forceinline__ void srf_tw(double (&w)[7], const double* __restrict__ tw, uint32_t t) {
    const uint32_t G = t / Srf<LN>::R(B);
#pragma unroll
    for (int u = Srf<LN>::u0(B); u < 3; u++)
#pragma unroll
        for (int g = 0; g < (1 << u); g++) w[(1 << u) - 1 + g] = tw[(1u << (Srf<LN>::s0(B) + u)) + (g << Srf<LN>::s0(B)) + G];
}
// block 0's are the same for every thread: scalar loads, through a pointer to constant memory
typedef const __attribute__((address_space(4))) double* const_f64;
template <int LN>
__device__ __forceinline__ void srf_tw0(double (&w)[7], const double* tw) {
    const const_f64 p = (const_f64)(uintptr_t)tw;
#pragma unroll
    for (int i = 0; i < 7; i++) w[i] = p[1 + i];
}
template <int LN, int B = 1>
__device__ __forceinline__ void srf_tw_all(SrfTw<LN>& w, const double* __restrict__ tw, uint32_t t) {
    if (B == 1) srf_tw0<LN>(w.w[0], tw);
    srf_tw<LN, B>(w.w[B], tw, t);
    if constexpr (B + 1 < Srf<LN>::NB) srf_tw_all<LN, B + 1>(w, tw, t);
}
// block B's points -> block D's
template <int LN, int B, int D>
__device__ __forceinline__ void srf_move(double (&x)[8], double* sm, uint32_t t) {
    asm("" : "+v"(t));                             // the words are worked out here, not kept in registers
    EACH8(k) sm[Srf<LN>::pos(B, t, k)] = x[k];
    if (B == 0 || D == 0) __syncthreads();
    else wave_exchange();
    EACH8(k) x[k] = sm[Srf<LN>::pos(D, t, k)];
}
// In: strided points (block 0's) below 2q in size.  Out: points 8t + k, not reduced (below 10q).
template <int LN, int B = 0>
__device__ __forceinline__ void srf_fwd(double (&x)[8], SrfTw<LN>& tw, const double* __restrict__ table, double* sm, uint32_t t, const FMod& m) {
    double w[7];
#pragma unroll
    for (int i = (1 << Srf<LN>::u0(B)) - 1; i < 7; i++) w[i] = tw.w[B][i];
#pragma unroll
    for (int u = Srf<LN>::u0(B); u < 3; u++) {
        const int dist = 4 >> u;
        double d[4];
#pragma unroll
        for (int p = 0; p < 4; p++) d[p] = f_mul(x[p / dist * 2 * dist + p % dist + dist], w[(1 << u) - 1 + p / dist], m);
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const int a = p / dist * 2 * dist + p % dist;
            x[a + dist] = x[a] - d[p];
            x[a] = x[a] + d[p];
        }
    }
    if constexpr (B + 1 < Srf<LN>::NB) {
        srf_move<LN, B, B + 1>(x, sm, t);
        srf_fwd<LN, B + 1>(x, tw, table, sm, t, m);
    }
}
// In: points 8t + k below q in size.  Out: strided points times scale (which carries N^-1), in [0, q).  The factors of the
// transform after this one (next) are requested as soon as this one has used its own.
template <int LN, int B = Srf<LN>::NB - 1>
__device__ __forceinline__ void srf_inv(double (&x)[8], SrfTw<LN>& tw, const double* __restrict__ table, const double* __restrict__ next, double scale,
                                        double* sm, uint32_t t, const FMod& m) {
    double w[7];
#pragma unroll
    for (int i = (1 << Srf<LN>::u0(B)) - 1; i < 7; i++) w[i] = tw.w[B][i];
    if (B > 0) srf_tw<LN, B>(tw.w[B], next, t);
    else srf_tw0<LN>(tw.w[0], next);
#pragma unroll
    for (int u = 2; u >= Srf<LN>::u0(B); u--) {
        const int dist = 4 >> u;
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const int a = p / dist * 2 * dist + p % dist;
            const double d = x[a] - x[a + dist];
            x[a] = x[a] + x[a + dist];
            x[a + dist] = d;
        }
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const int a = p / dist * 2 * dist + p % dist + dist;
            x[a] = f_mul(x[a], w[(1 << u) - 1 + p / dist], m);
        }
    }
    if constexpr (B > 0) {
        const int dist = 4 >> Srf<LN>::u0(B);
#pragma unroll
        for (int p = 0; p < 4; p++) { const int a = p / dist * 2 * dist + p % dist; x[a] = f_red(x[a], m); }
        srf_move<LN, B, B - 1>(x, sm, t);
        srf_inv<LN, B - 1>(x, tw, table, next, scale, sm, t, m);
    } else {
        EACH8(k) x[k] = f_nonneg(f_mul(x[k], scale, m), m);
    }
}
// sum of x_i * h_i over the limbs of a conversion: the last one's digits in x, the others in keep.  Below 2q in size.
template <int LN>
__device__ __forceinline__ void srf_convert(double (&x)[8], const double* keep, const u64* h, uint32_t n, uint32_t t, const FMod& m) {
    double s[8];
    const double hl = f_of(h[n - 1]);
    EACH8(k) s[k] = f_mul(x[k], hl, m);
    for (uint32_t i = 0; i + 1 < n; i++) {
        const double hi = f_of(h[i]);
        EACH8(k) s[k] += f_mul(keep[i * Srf<LN>::N + t + k * Srf<LN>::T], hi, m);
    }
    EACH8(k) x[k] = n > 1 ? f_red(s[k], m) : s[k];
}

template <int LN>
__global__ __launch_bounds__(Srf<LN>::T, 2) void srf_modup_kernel(SrUpArgs a, SrTables tb) {
    using G = Srf<LN>;
    __shared__ __attribute__((aligned(16))) double sm[SRF_LDS(LN)];
    __shared__ double keep[(SR_MAX_SRC - 1) * G::N];
    const uint32_t t = threadIdx.x;
    const SrfRow<LN> row(t);
    const uint32_t s = blockIdx.x / a.n_out, o = blockIdx.x % a.n_out;
    const uint32_t j = a.oj[o], r = a.orr[o];
    const uint32_t lo = j * a.alpha, sz = min(a.alpha, a.L1 - lo);
    const uint32_t mr = r <= a.level ? r : a.nq + (r - a.level - 1);
    const u64* c1 = a.c1[s] + ((size_t)lo << LN) + row.wb;
    const double *itw = tb.fitw + ((size_t)lo << LN), *ftw = tb.ftw + ((size_t)mr << LN);
    u64 in[8];
    SrfTw<LN> w;
    row.load(in, c1);
    srf_tw_all<LN>(w, itw, t);
    const FMod m = f_mod(tb.mc[mr]);
    const u64* hat = a.hat + ((size_t)(j * a.alpha + (sz - 1)) * a.M + mr) * a.aw;
    double x[8];
    for (uint32_t i = 0; i < sz; i++) {
        const bool last = i + 1 == sz;
        if (i) __syncthreads();                    // the words of the transform before have been read
        row.to_own(in, sm);
        EACH8(k) x[k] = f_of(in[k]);
        if (!last) row.load(in, c1 += G::N);
        srf_inv<LN>(x, w, itw, last ? ftw : itw + G::N, f_of(a.scale[lo + i]), sm, t, f_mod(tb.mc[lo + i]));
        itw += G::N;
        if (!last) { EACH8(k) keep[i * G::N + t + k * G::T] = x[k]; }
    }
    srf_convert<LN>(x, keep, hat, sz, t, m);
    srf_fwd<LN>(x, w, ftw, sm, t, m);
    u64* dst = a.raised + ((size_t)((s * a.beta + j) * a.R + r) << LN) + row.wb;
    EACH8(k) in[k] = f_canon(f_red(x[k], m), m);
    row.to_pairs(in, sm);
    row.store(dst, in);
}

// One limb's inner product at the wavefront's pairs.  The operands of the first SRF_DIG digits are requested together, and a
// transform ahead of their use.
struct SrfOps { u64 d[SRF_DIG][8], kv[SRF_DIG][8]; };
struct SrfInner {
    const u64 *raised, *own, *key;     // this limb's digits (own: of digit own_j, null elsewhere) and key rows
    uint32_t own_j;
};
template <int LN>
__device__ __forceinline__ void srf_digit(u64 (&d)[8], u64 (&kv)[8], const SrfInner& in, uint32_t j, size_t ds, size_t ks, const SrfRow<LN>& row, const SrfGalois<LN>& ga) {
    row.load(d, (j == in.own_j ? in.own : in.raised + j * ds) + ga.first);
    row.load(kv, in.key + j * ks + row.wb);
}
template <int LN>
__device__ __forceinline__ void srf_request(SrfOps& o, const SrfInner& in, uint32_t beta, size_t ds, size_t ks, const SrfRow<LN>& row, const SrfGalois<LN>& ga) {
#pragma unroll
    for (uint32_t j = 0; j < SRF_DIG; j++)
        if (j < beta) srf_digit(o.d[j], o.kv[j], in, j, ds, ks, row, ga);
}
// |result| < q; o holds the first SRF_DIG digits.  The wavefront's words of sm are overwritten.
template <int LN>
__device__ __forceinline__ void srf_inner(double (&out)[8], SrfOps& o, const SrfInner& in, uint32_t beta, size_t ds, size_t ks, const SrfRow<LN>& row,
                                          const SrfGalois<LN>& ga, double* sm, const FMod& m) {
    ga.apply(o.d[0], row, sm);
    EACH8(k) out[k] = f_mul(f_of(o.d[0][k]), f_of(o.kv[0][k]), m);
#pragma unroll
    for (uint32_t j = 1; j < SRF_DIG; j++)
        if (j < beta) {
            ga.apply(o.d[j], row, sm);
            EACH8(k) out[k] += f_mul(f_of(o.d[j][k]), f_of(o.kv[j][k]), m);
        }
    for (uint32_t j = SRF_DIG; j < beta; j++) {
        u64 d[8], kv[8];
        srf_digit(d, kv, in, j, ds, ks, row, ga);
        ga.apply(d, row, sm);
        EACH8(k) out[k] += f_mul(f_of(d[k]), f_of(kv[k]), m);
    }
    EACH8(k) out[k] = f_red(out[k], m);
}

template <int LN>
__device__ __forceinline__ void srf_moddown(const ModDownEpilogue& ep, const SrDownArgs& a, const SrTables& tb, double* sm, double* keep) {
    using G = Srf<LN>;
    const uint32_t L1 = ep.L1, R = ep.R, beta = ep.beta, t = threadIdx.x;
    const SrfRow<LN> row(t);
    const uint32_t pc = blockIdx.x / L1, r = blockIdx.x - pc * L1, job = pc >> 1, comp = pc & 1u;
    const SrfGalois<LN> ga(row, ep.g[job]);
    const size_t ds = (size_t)R << LN, ks = (size_t)(2 * ep.M) << LN, ro = (size_t)r << LN;
    const u64* raised = ep.raised[job];
    const u64* evk = ep.evk[job] + ((size_t)(comp * ep.M) << LN);
    const double *itw = tb.fitw + ((size_t)a.nq << LN), *ftw = tb.ftw + ro;
    SrfTw<LN> w;
    SrfOps o;
    SrfInner in = {raised + ((size_t)L1 << LN), nullptr, evk + ((size_t)a.nq << LN), 0xFFFFFFFFu};
    srf_request(o, in, beta, ds, ks, row, ga);
    srf_tw_all<LN>(w, itw, t);
    const FMod m = f_mod(tb.mc[r]);
    double x[8];
    for (uint32_t i = 0; i < a.k; i++) {
        const bool last = i + 1 == a.k;
        const FMod mp = f_mod(tb.mc[a.nq + i]);
        if (i) __syncthreads();                    // the words of the transform before have been read
        srf_inner(x, o, in, beta, ds, ks, row, ga, sm, mp);
        row.to_own(x, sm);
        // next: another special-prime limb, or after them limb r
        if (last) in = {raised + ro, ep.own[job] + ro, evk + ro, r / ep.alpha};
        else { in.raised += G::N; in.key += G::N; }
        srf_request(o, in, beta, ds, ks, row, ga);
        srf_inv<LN>(x, w, itw, last ? ftw : itw + G::N, f_of(a.scale[i]), sm, t, mp);
        itw += G::N;
        if (!last) { EACH8(k) keep[i * G::N + t + k * G::T] = x[k]; }
    }
    srf_convert<LN>(x, keep, a.dn_hat + (size_t)r * a.pw, a.k, t, m);
    __syncthreads();                               // the words of the inverse transform have been read
    double aq[8];
    srf_inner(aq, o, in, beta, ds, ks, row, ga, sm, m);
    // the addends travel while the forward transform runs
    const u64* c0 = comp == 0 ? ep.c0[job] : nullptr;
    const u64* self = comp ? ep.self1[job] : ep.self0[job];
    u64 add0[8], add1[8];
    EACH8(k) add0[k] = add1[k] = 0;
    if (c0) row.load(add0, c0 + ro + ga.first);
    if (self) row.load(add1, self + ro + row.wb);
    __syncthreads();                               // the forward transform writes everybody's words
    srf_fwd<LN>(x, w, ftw, sm, t, m);
    row.to_pairs(x, sm);
    wave_exchange();
    if (c0) ga.apply(add0, row, sm);
    u64* out = (comp ? ep.out1[job] : ep.out0[job]) + ro + row.wb;
    const double pinv = f_of(ep.pinv[r]);
    EACH8(k) {
        const double v = f_mul(aq[k] - x[k], pinv, m) + (f_of(add0[k]) + f_of(add1[k]));     // below 3q in size
        add0[k] = f_canon(f_red(v, m), m);
    }
    row.store(out, add0);
}

template <int LN>
__global__ __launch_bounds__(Srf<LN>::T, 2) void srf_moddown_kernel(ModDownEpilogue ep, SrDownArgs a, SrTables tb) {
    __shared__ __attribute__((aligned(16))) double sm[SRF_LDS(LN)];
    __shared__ double keep[(SR_MAX_SRC - 1) * Srf<LN>::N];
    srf_moddown<LN>(ep, a, tb, sm, keep);
}
// ModDown and the ModUp of the second components it leaves, side by side: coefficients of a digit's limb are those of sum / P + addend less
// those of the converted part / P, so a digit needs the special primes' inverse transforms (as every ModDown work group does) and its own, and
// not the results.  A layer of N = 2^12 with two steps 79.6 -> 74.9 us (ModDown 14.7 and ModUp 9.6 one after the other).  Digits and special primes of together at most four
// limbs, which LDS holds; of a digit's limbs only the first is asked for ahead (all of them spill).
template <int LN>
__global__ __launch_bounds__(Srf<LN>::T, 2) void srf_moddown_modup_kernel(ModDownEpilogue ep, SrDownArgs a, SrUpArgs u, SrRaise f, SrTables tb) {
    using G = Srf<LN>;
    __shared__ __attribute__((aligned(16))) double sm[SRF_LDS(LN)];
    __shared__ double keep[(SR_MAX_SRC - 1) * G::N];       // the special primes' limbs, then the digit's but the last
    if (blockIdx.x < f.first) {
        srf_moddown<LN>(ep, a, tb, sm, keep);
        return;
    }
    const uint32_t t = threadIdx.x, b = blockIdx.x - f.first, job = b / u.n_out, o = b - job * u.n_out, beta = ep.beta;
    const SrfRow<LN> row(t);
    const uint32_t j = u.oj[o], r = u.orr[o], lo = j * u.alpha, sz = min(u.alpha, u.L1 - lo);
    const uint32_t mr = r <= u.level ? r : u.nq + (r - u.level - 1);
    const SrfGalois<LN> ga(row, ep.g[job]);
    const size_t ds = (size_t)ep.R << LN, ks = (size_t)(2 * ep.M) << LN;
    const u64 *raised = ep.raised[job], *evk = ep.evk[job] + ((size_t)ep.M << LN), *self = ep.self1[job];
    const double *itw = tb.fitw + ((size_t)a.nq << LN), *ftw = tb.ftw + ((size_t)mr << LN);
    SrfTw<LN> w;
    SrfOps ops;
    SrfInner in = {raised + ((size_t)ep.L1 << LN), nullptr, evk + ((size_t)a.nq << LN), 0xFFFFFFFFu};
    srf_request(ops, in, beta, ds, ks, row, ga);
    srf_tw_all<LN>(w, itw, t);
    double x[8];
    for (uint32_t i = 0; i < a.k; i++) {
        const bool last = i + 1 == a.k;
        const FMod mp = f_mod(tb.mc[a.nq + i]);
        if (i) __syncthreads();                            // the words of the transform before have been read
        srf_inner(x, ops, in, beta, ds, ks, row, ga, sm, mp);
        row.to_own(x, sm);
        // next: another special-prime limb, or after them the digit's first
        if (last) in = {raised + ((size_t)lo << LN), ep.own[job] + ((size_t)lo << LN), evk + ((size_t)lo << LN), j};
        else { in.raised += G::N; in.key += G::N; }
        srf_request(ops, in, beta, ds, ks, row, ga);
        srf_inv<LN>(x, w, itw, last ? tb.fitw + ((size_t)lo << LN) : itw + G::N, f_of(a.scale[i]), sm, t, mp);
        itw += G::N;
        EACH8(k) keep[i * G::N + t + k * G::T] = x[k];
    }
    itw = tb.fitw + ((size_t)lo << LN);
    double* digit = keep + a.k * G::N;
    for (uint32_t i = 0; i < sz; i++) {
        const bool last = i + 1 == sz;
        const uint32_t q = lo + i;
        const FMod mi = f_mod(tb.mc[q]);
        const double pinv = f_of(ep.pinv[q]), c = f_of(f.factor[q]);
        if (i) {
            in.raised += G::N; in.own += G::N; in.key += G::N;
            srf_request(ops, in, beta, ds, ks, row, ga);
        }
        __syncthreads();                                   // the words of the transform before have been read
        srf_inner(x, ops, in, beta, ds, ks, row, ga, sm, mi);
        u64 add[8];
        EACH8(k) add[k] = 0;
        if (self) row.load(add, self + ((size_t)q << LN) + row.wb);
        EACH8(k) x[k] = f_red(f_mul(x[k], pinv, mi) + f_of(add[k]), mi);
        row.to_own(x, sm);
        srf_inv<LN>(x, w, itw, last ? ftw : itw + G::N, f_of(u.scale[q]), sm, t, mi);
        itw += G::N;
        double v[8];
        EACH8(k) v[k] = keep[(a.k - 1) * G::N + t + k * G::T];
        srf_convert<LN>(v, keep, a.dn_hat + (size_t)q * a.pw, a.k, t, mi);
        EACH8(k) x[k] = f_nonneg(f_red(x[k] - f_mul(v[k], c, mi), mi), mi);
        if (!last) { EACH8(k) digit[i * G::N + t + k * G::T] = x[k]; }
    }
    const FMod m = f_mod(tb.mc[mr]);
    srf_convert<LN>(x, digit, u.hat + ((size_t)(j * u.alpha + (sz - 1)) * u.M + mr) * u.aw, sz, t, m);
    srf_fwd<LN>(x, w, ftw, sm, t, m);
    u64* dst = u.raised + ((size_t)((job * u.beta + j) * u.R + r) << LN) + row.wb;
    u64 out[8];
    EACH8(k) out[k] = f_canon(f_red(x[k], m), m);
    row.to_pairs(out, sm);
    row.store(dst, out);
}

template <int LN>
__device__ __forceinline__ void srf_rescale(const SrRescaleArgs& a, const SrTables& tb, double* sm) {
    const uint32_t level = a.level, t = threadIdx.x;
    const SrfRow<LN> row(t);
    const uint32_t jc = blockIdx.x / level, r = blockIdx.x - jc * level, job = jc >> 1, comp = jc & 1u;
    const u64* top = a.ct[job] + ((size_t)(comp * (level + 1) + level) << LN) + row.wb;
    const u64* in = a.ct[job] + ((size_t)(comp * (level + 1) + r) << LN) + row.wb;
    const double *itw = tb.fitw + ((size_t)level << LN), *ftw = tb.ftw + ((size_t)r << LN);
    u64 tp[8], cr[8];
    SrfTw<LN> w;
    row.load(tp, top);
    srf_tw_all<LN>(w, itw, t);
    row.load(cr, in);
    const FMod ml = f_mod(tb.mc[level]), m = f_mod(tb.mc[r]);
    const double qlinv = f_of(a.qlinv[r]), h = f_of(ml.n >> 1);
    double x[8];
    row.to_own(tp, sm);
    EACH8(k) x[k] = f_of(tp[k]);
    srf_inv<LN>(x, w, itw, ftw, f_of(tb.mc[level].ninv), sm, t, ml);
    EACH8(k) {                                       // (h mod q_r) - ((x + h mod q_l) mod q_r), below 2q_r in size
        const double v = x[k] + h;
        x[k] = f_red(h, m) - f_red(v < ml.q ? v : v - ml.q, m);
    }
    srf_fwd<LN>(x, w, ftw, sm, t, m);
    row.to_pairs(x, sm);
    u64* out = a.out[job] + ((size_t)(comp * level + r) << LN) + row.wb;
    EACH8(k) cr[k] = f_canon(f_mul(f_of(cr[k]) + x[k], qlinv, m), m);
    row.store(out, cr);
}
template <int LN>
__global__ __launch_bounds__(Srf<LN>::T, 2) void srf_rescale_kernel(SrRescaleArgs a, SrTables tb) {
    __shared__ __attribute__((aligned(16))) double sm[SRF_LDS(LN)];
    srf_rescale<LN>(a, tb, sm);
}
// Rescale and the ModUp of the second components it leaves, side by side: the digits' coefficients are (c_i + correction) / q_l of the inputs'
// coefficients, so a digit needs the dropped limb's inverse transform besides its own and not the rescaled limbs.  u: for the level below.  A layer
// of N = 2^12 with two steps 83.6 -> 79.6 us, with four outputs and one tap 60.7 -> 56.1 (8.5 us of rescale and 9.6 of ModUp, 13.7 side by side).
template <int LN>
__global__ __launch_bounds__(Srf<LN>::T, 2) void srf_rescale_modup_kernel(SrRescaleArgs a, SrUpArgs u, SrRaise f, SrTables tb) {
    using G = Srf<LN>;
    __shared__ __attribute__((aligned(16))) double sm[SRF_LDS(LN)];
    __shared__ double keep[(SR_MAX_SRC - 1) * G::N];
    if (blockIdx.x < f.first) {
        srf_rescale<LN>(a, tb, sm);
        return;
    }
    const uint32_t t = threadIdx.x, b = blockIdx.x - f.first, s = b / u.n_out, o = b - s * u.n_out, level = a.level;
    const SrfRow<LN> row(t);
    const uint32_t j = u.oj[o], r = u.orr[o], lo = j * u.alpha, sz = min(u.alpha, u.L1 - lo);
    const uint32_t mr = r <= u.level ? r : u.nq + (r - u.level - 1);
    const u64 *c1 = a.ct[s] + ((size_t)(level + 1) << LN) + row.wb, *limb = c1 + ((size_t)lo << LN);
    const double *top = tb.fitw + ((size_t)level << LN), *itw = tb.fitw + ((size_t)lo << LN), *ftw = tb.ftw + ((size_t)mr << LN);
    u64 in[8];
    SrfTw<LN> w;
    row.load(in, c1 + ((size_t)level << LN));
    srf_tw_all<LN>(w, top, t);
    const FMod m = f_mod(tb.mc[mr]), ml = f_mod(tb.mc[level]);
    const double h = f_of(ml.n >> 1);
    const u64* hat = u.hat + ((size_t)(j * u.alpha + (sz - 1)) * u.M + mr) * u.aw;
    double x[8], v[8];
    row.to_own(in, sm);
    EACH8(k) x[k] = f_of(in[k]);
    row.load(in, limb);
    srf_inv<LN>(x, w, top, itw, f_of(tb.mc[level].ninv), sm, t, ml);
    EACH8(k) { const double y = x[k] + h; v[k] = y < ml.q ? y : y - ml.q; }
    for (uint32_t i = 0; i < sz; i++) {
        const bool last = i + 1 == sz;
        const FMod mi = f_mod(tb.mc[lo + i]);
        __syncthreads();                           // the words of the transform before have been read
        row.to_own(in, sm);
        EACH8(k) x[k] = f_of(in[k]);
        if (!last) row.load(in, limb += G::N);
        srf_inv<LN>(x, w, itw, last ? ftw : itw + G::N, f_of(u.scale[lo + i]), sm, t, mi);
        itw += G::N;
        const double hi = f_red(h, mi), c = f_of(f.factor[lo + i]);
        EACH8(k) x[k] = f_nonneg(f_red(x[k] + f_mul(hi - f_red(v[k], mi), c, mi), mi), mi);
        if (!last) { EACH8(k) keep[i * G::N + t + k * G::T] = x[k]; }
    }
    srf_convert<LN>(x, keep, hat, sz, t, m);
    srf_fwd<LN>(x, w, ftw, sm, t, m);
    u64* dst = u.raised + ((size_t)((s * u.beta + j) * u.R + r) << LN) + row.wb;
    EACH8(k) in[k] = f_canon(f_red(x[k], m), m);
    row.to_pairs(in, sm);
    row.store(dst, in);
}
#pragma clang fp contract(on)

// ---------------------------------------------------------------- host
static SrTables sr_tables(const he_ctx* c) { return {c->d_mc, c->d_tw, c->d_itw, c->d_ftw, c->d_fitw, c->logN}; }

// FP64 kernels where every modulus of the context allows them (their values stay exact up to 45 bits), else the integer ones
#define SR_LAUNCH(NAME, GRID, ...)                                                                                             \
    do {                                                                                                                       \
        if (!c->srf) hipLaunchKernelGGL(sr_##NAME, GRID, dim3(SR_THREADS), 0, c->stream, __VA_ARGS__);                         \
        else SRF_LAUNCH(NAME, GRID, __VA_ARGS__);                                                                              \
    } while (0)
#define SRF_LAUNCH(NAME, GRID, ...)                                                                                            \
    do {                                                                                                                       \
        if (c->logN == 12) hipLaunchKernelGGL(srf_##NAME<12>, GRID, dim3(Srf<12>::T), 0, c->stream, __VA_ARGS__);         \
        else if (c->logN == 11) hipLaunchKernelGGL(srf_##NAME<11>, GRID, dim3(Srf<11>::T), 0, c->stream, __VA_ARGS__);         \
        else if (c->logN == 10) hipLaunchKernelGGL(srf_##NAME<10>, GRID, dim3(Srf<10>::T), 0, c->stream, __VA_ARGS__);         \
        else if (c->logN == 9) hipLaunchKernelGGL(srf_##NAME<9>, GRID, dim3(Srf<9>::T), 0, c->stream, __VA_ARGS__);            \
        else hipLaunchKernelGGL(srf_##NAME<8>, GRID, dim3(Srf<8>::T), 0, c->stream, __VA_ARGS__);                              \
    } while (0)

bool small_ring_path(const he_ctx* c, uint32_t level) {
    const uint32_t beta = (level + c->alpha) / c->alpha;
    return c->logN <= 12 && c->alpha <= SR_MAX_SRC && c->np >= 1 && c->np <= SR_MAX_SRC && beta <= 8 && beta * (level + 1 + c->np) <= 512;
}

// all but the sources
static void sr_up_args(const he_ctx* c, uint32_t level, u64* raised, SrUpArgs& a) {
    const uint32_t L1 = level + 1, R = L1 + c->np, al = c->alpha, beta = (level + al) / al;
    a.raised = raised; a.hat = c->d_up_hat;
    a.L1 = L1; a.R = R; a.beta = beta; a.alpha = al; a.M = c->M; a.nq = c->nq; a.level = level; a.aw = (al + 7u) & ~7u;
    for (uint32_t i = 0; i < L1; i++) {
        const uint32_t j = i / al, lo = j * al, hi = (j + 1) * al < L1 ? (j + 1) * al : L1, sz = hi - lo;
        a.scale[i] = h_mulmod(c->h_mc[i].ninv, c->h_up_invhat[(size_t)(j * al + (sz - 1)) * al + (i - lo)], c->mod[i]);
        a.scale_sh[i] = h_shoup(a.scale[i], c->mod[i]);
    }
    a.n_out = 0;
    for (uint32_t j = 0; j < beta; j++) {
        const uint32_t lo = j * al, hi = (j + 1) * al < L1 ? (j + 1) * al : L1;
        for (uint32_t r = 0; r < R; r++) {
            if (r >= lo && r < hi) continue;
            a.oj[a.n_out] = (uint8_t)j; a.orr[a.n_out] = (uint8_t)r; a.n_out++;
        }
    }
}
int32_t sr_modup(he_ctx* c, const KsSrc* srcs, uint32_t cb, uint32_t level, u64* raised) {
    const uint32_t L1 = level + 1;
    SrUpArgs a;
    if (cb > HE_MAX_KS_JOBS) return he_fail(c, HE_ERR_BADARG, "small-ring ModUp: more than %d sources", HE_MAX_KS_JOBS);
    for (uint32_t s = 0; s < HE_MAX_KS_JOBS; s++) a.c1[s] = srcs[s < cb ? s : 0].c1;
    sr_up_args(c, level, raised, a);
    SR_LAUNCH(modup_kernel, dim3(cb * a.n_out), a, sr_tables(c));
    HE_HIP(c, hipGetLastError());
    // logical transform counts (each work group repeats the inverse transforms of its digit)
    c->cnt.intt_limbs += (uint64_t)cb * L1;
    c->cnt.ntt_limbs += (uint64_t)cb * a.n_out;
    c->cnt.modup += cb;
    return HE_OK;
}

bool sr_moddown_raises(const he_ctx* c, uint32_t level) { return c->srf && small_ring_path(c, level) && c->alpha + c->np <= SR_MAX_SRC; }
int32_t sr_moddown(he_ctx* c, uint32_t level, uint32_t J, const ModDownEpilogue& ep, u64* raised_next) {
    const uint32_t L1 = level + 1, k = c->np;
    SrDownArgs a;
    a.dn_hat = c->d_dn_hat; a.k = k; a.nq = c->nq; a.level = level; a.pw = (k + 7u) & ~7u;
    for (uint32_t t = 0; t < k; t++) {
        const u64 p = c->mod[c->nq + t];
        a.scale[t] = h_mulmod(c->h_mc[c->nq + t].ninv, c->h_dn_invhat[t], p);
        a.scale_sh[t] = h_shoup(a.scale[t], p);
    }
    if (raised_next) {
        if (!sr_moddown_raises(c, level)) return he_fail(c, HE_ERR_BADARG, "ModDown with ModUp: bad shape");
        SrUpArgs u;
        SrRaise f;
        sr_up_args(c, level, raised_next, u);
        f.first = J * 2 * L1;
        for (uint32_t i = 0; i < L1; i++) {
            const u64 q = c->mod[i];
            f.factor[i] = h_mulmod(h_mulmod(u.scale[i], c->N % q, q), c->h_pinv[i], q);
        }
        SRF_LAUNCH(moddown_modup_kernel, dim3(f.first + J * u.n_out), ep, a, u, f, sr_tables(c));
        c->cnt.intt_limbs += (uint64_t)J * L1;
        c->cnt.ntt_limbs += (uint64_t)J * u.n_out;
        c->cnt.modup += J;
    } else SR_LAUNCH(moddown_kernel, dim3(J * 2 * L1), ep, a, sr_tables(c));
    HE_HIP(c, hipGetLastError());
    c->cnt.intt_limbs += (uint64_t)J * 2 * k;
    c->cnt.ntt_limbs += (uint64_t)J * 2 * L1;
    c->cnt.moddown += J;
    return HE_OK;
}

int32_t sr_rescale(he_ctx* c, const u64* const* cts, u64* const* outs, uint32_t n, uint32_t level) {
    for (uint32_t b0 = 0; b0 < n; b0 += HE_MAX_KS_JOBS) {
        const uint32_t nb = n - b0 < HE_MAX_KS_JOBS ? n - b0 : HE_MAX_KS_JOBS;
        SrRescaleArgs a;
        for (uint32_t i = 0; i < nb; i++) { a.ct[i] = cts[b0 + i]; a.out[i] = outs[b0 + i]; }
        a.qlinv = c->d_qlinv + (size_t)level * c->nq; a.qlinv_sh = c->d_qlinv_sh + (size_t)level * c->nq; a.level = level;
        SR_LAUNCH(rescale_kernel, dim3(nb * 2 * level), a, sr_tables(c));
        HE_HIP(c, hipGetLastError());
        c->cnt.intt_limbs += (uint64_t)2 * nb;
        c->cnt.ntt_limbs += (uint64_t)2 * nb * level;
        c->cnt.rescale += nb;
    }
    return HE_OK;
}

bool sr_rescale_raises(const he_ctx* c, uint32_t level, uint32_t n) { return c->srf && level && n <= HE_MAX_KS_JOBS && small_ring_path(c, level - 1); }
int32_t sr_rescale_modup(he_ctx* c, const u64* const* cts, u64* const* outs, uint32_t n, uint32_t level, u64* raised) {
    if (!sr_rescale_raises(c, level, n) || n == 0) return he_fail(c, HE_ERR_BADARG, "rescale with ModUp: bad shape");
    SrRescaleArgs a;
    SrUpArgs u;
    SrRaise f;
    for (uint32_t i = 0; i < n; i++) { a.ct[i] = cts[i]; a.out[i] = outs[i]; }
    a.qlinv = c->d_qlinv + (size_t)level * c->nq; a.qlinv_sh = c->d_qlinv_sh + (size_t)level * c->nq; a.level = level;
    sr_up_args(c, level - 1, raised, u);
    f.first = 2 * n * level;
    for (uint32_t i = 0; i < level; i++) {
        const u64 q = c->mod[i];
        u.scale[i] = h_mulmod(u.scale[i], c->h_qlinv[(size_t)level * c->nq + i], q);
        f.factor[i] = h_mulmod(u.scale[i], c->N % q, q);
    }
    SRF_LAUNCH(rescale_modup_kernel, dim3(f.first + n * u.n_out), a, u, f, sr_tables(c));
    HE_HIP(c, hipGetLastError());
    c->cnt.intt_limbs += (uint64_t)n * (2 + level);
    c->cnt.ntt_limbs += (uint64_t)n * (2 * level + u.n_out);
    c->cnt.rescale += n;
    c->cnt.modup += n;
    return HE_OK;
}
