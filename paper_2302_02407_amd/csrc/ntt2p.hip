// Two-launch negacyclic NTT / iNTT (ring of paper Section 2.1) for rings whose limb does not fit one work group:
// N = 2^13 .. 2^17.
//
// The limb is viewed as 2^LC rows of 256 (row-major, LC = logN - 8).  A transform is two launches:
//   forward : column pass (stages 0 .. LC-1, row distance 2^(LC-1) .. 1), row pass (stages LC .. LC+7);
//   inverse : row pass (stages LC+7 .. LC), column pass (stages LC-1 .. 0) with the output scaling.
// Inside a pass every thread keeps 16 points of one sub-transform in registers and runs up to 4 butterfly stages on
// them, then the threads of the sub-transform exchange points through LDS and run the others: one LDS round trip
// replaces eight (two for the 9-stage columns of N = 2^17).  Points are held either "strided" (thread t holds t + k*16 of
// a row, t + k*2^(LC-4) of a column) or "contiguous" (16t + j).
//
// What bounds a pass is how far loads run ahead of arithmetic.  A row pass needs 240 bytes of twiddles per thread for 128
// bytes of points; fetched where they are used they cost 40 us of 104 (384 limbs, N = 2^16, measured with the factors
// taken out), so they are requested a block ahead, as the registers of the previous block's factors come free: 81 us,
// where a copy of the same limbs through LDS takes 61.  The second block's factors are every thread's own; kept one of every
// thread after the other (ctx.hip, tw_pos) a load covers 8 cache lines where a thread's own side by side made it 64:
// inverse row pass of 384 limbs 124 -> 102 us, forward 110 -> 105.
//
// Arithmetic: ntt_blocks.h.  Forward values are never reduced inside a transform for narrow moduli (16 or 17 stages end
// below 90q); a small-quotient step makes them canonical at the end.
#include <algorithm>

#include "modarith.h"
#include "ntt_blocks.h"

#define P2_THREADS 256

// Limbs of a launch, sorted by modulus: destination limb (bits 0-8), modulus (9-14), source segment (27-30) and limb in it
// (15-26).  One 32-bit word per limb, so that a work group gets all of it in one scalar load, and
// branches to the code of its modulus' class before it loads anything else (a branch between the loads and their use
// doubles the registers that are live across it).
struct LimbTab {
    const u64* seg[HE_MAX_SEGS];
    uint32_t e[HE_MAX_LAUNCH_LIMBS];
};
#define TAB_NONE 0xFFFFFFFFu
struct P2Args {
    u64* dst;
    const ModConst* mc;
    const ulonglong2* tw;     // [M][N] forward or inverse twiddles
    uint32_t logN;
    uint32_t lazy;            // forward, last pass: outputs may stay below 2q
    uint32_t rs_mod;          // forward, first pass reading the Rescale rounding term: modulus index of the dropped limb
    uint32_t log_chunk;       // row passes, see row_decode
    ModClasses cls;           // of this direction
};
__device__ __forceinline__ uint32_t tab_dst(uint32_t e) { return e & 511u; }
__device__ __forceinline__ uint32_t tab_mod(uint32_t e) { return (e >> 9) & 63u; }
__device__ __forceinline__ const u64* tab_src(const LimbTab& tab, uint32_t e, uint32_t logN) {
    return tab.seg[(e >> 27) & 15u] + ((size_t)((e >> 15) & 0xFFFu) << logN);
}

// Work order of the row passes.  Their twiddles depend on (modulus, tile), so limbs that share a modulus should run the same
// tile back to back on the same XCD (one L2 per XCD; workgroups are handed to the 8 XCDs round-robin).  The table is
// padded with TAB_NONE to a multiple of the chunk size C = 1 << log_chunk; the linear work index
// L = (chunk_of_limbs*tiles + tile)*C + j walks the C limbs of a chunk for one tile, and
// workgroup id -> L keeps each run of C consecutive L on one XCD.
template <int LANES>
__device__ __forceinline__ uint32_t row_decode(const LimbTab& tab, const P2Args& a, uint32_t& tile) {
    const uint32_t lc = a.log_chunk, idx = blockIdx.x, lt = a.logN - (LANES == 16 ? 12 : 10);
    const uint32_t xcd = idx & 7u, slot = idx >> 3;
    const uint32_t L = ((((slot >> lc) << 3) + xcd) << lc) | (slot & ((1u << lc) - 1u));
    const uint32_t pchunk = L >> (lt + lc), rem = L & ((1u << (lt + lc)) - 1u);
    tile = rem >> lc;
    return __builtin_amdgcn_readfirstlane(tab.e[(pchunk << lc) + (rem & ((1u << lc) - 1u))]);
}

// ---------------------------------------------------------------- column passes
// Tile of a column pass: all 2^LC rows of C = 4096 / 2^LC adjacent columns.  LDS position of (row, column): one spare row
// per 16 keeps the row groups that a wavefront reads back at once on different banks (with 32 or more columns a half
// wavefront stays inside one row).
template <int LC>
struct Col {
    static constexpr int LCOLS = 12 - LC, C = 1 << LCOLS, LT = LC - 4, T = 1 << LT;   // T threads share a column
    static constexpr int U0 = LC < 8 ? 8 - LC : 0;                                   // first stage of the second block
    static constexpr int LDS = C >= 32 ? 4096 : 4096 + 256;
    static __device__ __forceinline__ uint32_t pos(uint32_t r, uint32_t cl) { return (C >= 32 ? r : r + (r >> 4)) * C + cl; }
};

// RS: the source is the coefficient form of the limb that Rescale drops (modulus ml); what is transformed is the negated
// rounding term ((v + h) mod q_l) mod q - (h mod q), h = floor(q_l / 2), of this limb's modulus m.
template <int LC, bool RS, int W>
__device__ __forceinline__ void col_fwd(const P2Args& a, const LimbTab& tab, uint32_t e, uint32_t tile, u64* sm) {
    using G = Col<LC>;
    const uint32_t mi = tab_mod(e), logN = LC + 8;
    const u64* src = tab_src(tab, e, logN);
    const ulonglong2* tw = a.tw + ((size_t)mi << logN);
    const uint32_t t = threadIdx.x >> G::LCOLS, cl = threadIdx.x & (G::C - 1), c = tile * G::C + cl;
    u64 x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = (src + ((size_t)k << (G::LT + 8)))[t * 256 + c];
    ulonglong2 w1[15], w2[15];                           // w1: the same for the whole limb (scalar registers)
    if (LC <= 8) tw_load<G::U0, 4>(w2, tw, LC - 4, t);
    else tw_load<0, 4>(w2, tw, 4, t >> 1);
    tw_load_c<0, 4>(w1, (ctw_t)(uintptr_t)tw, 0, 0);
    const ModConst m = mod_const(a.mc, mi), ml = RS ? mod_const(a.mc, a.rs_mod) : m;
    u64* dst = a.dst + ((size_t)tab_dst(e) << logN);
    const u64 q = m.q;
    if (RS) {
        const u64 h = ml.q >> 1, hr = barrett64(h, q, m.mu, m.bits);
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = shoup_lazy4(addmod(x[k], h, ml.q), 1, m.one_sh, q) + (q - hr);      // below 5q
    }
    fwd_centre<W>(x, m);
    int b = 5;
    fwd_stages<W, 0, 4, true>(x, w1, q, b);
#pragma unroll
    for (int k = 0; k < 16; k++) sm[G::pos(t + (k << G::LT), cl)] = x[k];
    __syncthreads();
    if (LC <= 8) {
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = sm[G::pos(16 * t + j, cl)];
        fwd_stages<W, G::U0, 4>(x, w2, q, b);
    } else {
        // nine stages: rows 32G + e + 2j for stages 4..7 (t = 2G + e), then contiguous rows for stage 8
        const uint32_t r0 = (t >> 1) * 32 + (t & 1);
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = sm[G::pos(r0 + 2 * j, cl)];
        fwd_stages<W, 0, 4>(x, w2, q, b);
        ulonglong2 w3[15];
        tw_load<3, 4>(w3, tw, 5, t);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; j++) sm[G::pos(r0 + 2 * j, cl)] = x[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = sm[G::pos(16 * t + j, cl)];
        fwd_stages<W, 3, 4>(x, w3, q, b);
    }
#pragma unroll
    for (int j = 0; j < 16; j++) (dst + j * 256)[t * 4096 + c] = x[j];
}

template <int LC, bool RS>
__global__ __launch_bounds__(P2_THREADS, 4) void ntt_col_fwd_kernel(P2Args a, LimbTab tab) {
    ieee_off();
    using G = Col<LC>;
    __shared__ u64 sm[G::LDS];
    const uint32_t tile = blockIdx.x & (G::T - 1), e = __builtin_amdgcn_readfirstlane(tab.e[blockIdx.x >> G::LT]);
    by_class(a.cls, tab_mod(e), e, [&](auto W, uint32_t v) { col_fwd<LC, RS, W>(a, tab, v, tile, sm); });
}

// Inverse column stages and output scaling: inputs below 2q (wide moduli: w_half), results canonical.  Stage 0 (one twiddle for the whole limb)
// carries the scaling: the sum is multiplied by the scale, the difference by scale * twiddle.  Narrow moduli: bounds
// 2 -> 40 (N = 2^17: 80, reduced) -> 320 -> 640 (products that take any value, Shoup's).
template <int LC, bool CUSTOM_SCALE, bool AHEAD, int W>
__device__ __forceinline__ void col_inv(const P2Args& a, uint32_t e, uint32_t tile, u64* sm, const ScaleList& sc, uint32_t scale_period) {
    using G = Col<LC>;
    const uint32_t mi = tab_mod(e), logN = LC + 8, limb = tab_dst(e);
    u64* data = a.dst + ((size_t)limb << logN);
    const ulonglong2* tw = a.tw + ((size_t)mi << logN);
    const uint32_t t = threadIdx.x >> G::LCOLS, cl = threadIdx.x & (G::C - 1), c = tile * G::C + cl;
    u64 x[16];
#pragma unroll
    for (int j = 0; j < 16; j++) x[j] = (data + j * 256)[t * 4096 + c];
    ulonglong2 w1[15], w2[15];
    if (LC <= 8) tw_load<G::U0, 4>(w2, tw, LC - 4, t);
    else if (AHEAD) tw_load<0, 4>(w2, tw, 4, t >> 1);
    const ModConst m = mod_const(a.mc, mi);
    const uint32_t si = CUSTOM_SCALE ? limb % scale_period : 0;
    constexpr bool NEAR = W == W_NEAR;
    const u64 cs = CUSTOM_SCALE ? sc.s[si] : NEAR ? m.near_s : m.ninv, cs_sh = CUSTOM_SCALE ? sc.s_sh[si] : NEAR ? m.near_s_sh : m.ninv_sh;
    const u64 cw = CUSTOM_SCALE ? sc.w[si] : NEAR ? m.near_w : m.ninv_w, cw_sh = CUSTOM_SCALE ? sc.w_sh[si] : NEAR ? m.near_w_sh : m.ninv_w_sh;
    const u64 q = m.q;
    int bound = w_start(W);
    if (LC <= 8) {
        inv_stages<W, G::U0, 4>(x, w2, q, bound);
#pragma unroll
        for (int j = 0; j < 16; j++) sm[G::pos(16 * t + j, cl)] = x[j];
    } else {
        ulonglong2 w3[15];
        tw_load<3, 4>(w3, tw, 5, t);
        inv_stages<W, 3, 4>(x, w3, q, bound);
        if (!AHEAD) {
            SCHED_FENCE();
            tw_load<0, 4>(w2, tw, 4, t >> 1);
        }
        const uint32_t r0 = (t >> 1) * 32 + (t & 1);
#pragma unroll
        for (int j = 0; j < 16; j++) sm[G::pos(16 * t + j, cl)] = x[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = sm[G::pos(r0 + 2 * j, cl)];
        inv_stages<W, 0, 4>(x, w2, q, bound);
        if (W == 0 || W == W_NEAR) {
            bound = 2;
#pragma unroll
            for (int j = 0; j < 16; j++) x[j] = inv_end<W>(x[j], m);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; j++) sm[G::pos(r0 + 2 * j, cl)] = x[j];
    }
    tw_load_c<1, 4>(w1, (ctw_t)(uintptr_t)tw, 0, 0);     // the same for the whole limb (scalar registers)
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = sm[G::pos(t + (k << G::LT), cl)];
    inv_stages<W, 1, 4, true>(x, w1, q, bound);
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const u64 X = x[k], Y = x[k + 8];
        x[k] = inv_scaled<W>(X + Y, cs, cs_sh, q);
        x[k + 8] = inv_scaled<W>(W == W_NEAR ? X - Y : (X + q * (u64)bound) - Y, cw, cw_sh, q);
    }
#pragma unroll
    for (int k = 0; k < 16; k++) (data + ((size_t)k << (G::LT + 8)))[t * 256 + c] = inv_canonical<W>(x[k], q);
}

// AHEAD: N = 2^17 (LC = 9), the middle block's factors are asked for with the first block's, for which four wavefronts to a SIMD have no
// registers (8 bytes spilled a lane).  For launches that do not fill four: 8 limbs 13.4 us, 13.9 with the factors behind the first block;
// 192 limbs 118.5 and 108.5, 96 limbs 66 and 62.
template <int LC, bool CUSTOM_SCALE, bool AHEAD = false>
__global__ __launch_bounds__(P2_THREADS, AHEAD ? 3 : 4) void ntt_col_inv_kernel(P2Args a, LimbTab tab, ScaleList sc, uint32_t scale_period) {
    ieee_off();
    using G = Col<LC>;
    __shared__ u64 sm[G::LDS];
    const uint32_t tile = blockIdx.x & (G::T - 1), e = __builtin_amdgcn_readfirstlane(tab.e[blockIdx.x >> G::LT]);
    by_class(a.cls, tab_mod(e), e, [&](auto W, uint32_t v) { col_inv<LC, CUSTOM_SCALE, AHEAD, W>(a, v, tile, sm, sc, scale_period); });
}

// ---------------------------------------------------------------- forward row pass
// Pass B: workgroup = 16 consecutive rows (256-point blocks); tid = blk*16 + t.  A row stays inside 16 lanes of one wavefront,
// so its exchanges need no barrier and the wavefronts run apart.
// EPI: whether the pass ends in the ModDown (or Rescale) epilogue, with the accumulator read from memory.  Its results go past the
// caches' usual replacement: a merge of 16 ciphertexts with its rescale 163.3 -> 161.7 us, and, where the call's next launch reads them,
// 16 channels with a hoisted sum at level 12 1203 -> 1191, at level 5 628 -> 625; other layers within 0.3 % either way.
// LANES: threads that share a row, 16 points each in two register blocks of four stages or, for small launches, 4 points each
// in four blocks of two (see launch_transform2p).
template <int W, bool EPI, int LANES>
__device__ __forceinline__ void row_fwd(const P2Args& a, uint32_t e, uint32_t tile, u64* sm, const ModDownEpilogue& ep) {
    const uint32_t mi = tab_mod(e), limb = tab_dst(e), logN = a.logN, lc = logN - 8;
    const ulonglong2* tw = a.tw + ((size_t)mi << logN);
    constexpr int DP = 2 * LANES;
    const uint32_t blk = threadIdx.x / LANES, t = threadIdx.x % LANES, b = tile * (P2_THREADS / LANES) + blk;
    u64* row = a.dst + ((size_t)limb << logN) + (size_t)b * 256;
    u64* s = sm + blk * 272;
    const ModConst m = mod_const(a.mc, mi);
    const u64 q = m.q;
    constexpr int PTS = 256 / LANES;
    u64 x[PTS];
    if constexpr (LANES == 16) {
        ulonglong2 w1[15], w2[15];
        tw_load<0, 4>(w1, tw, lc, b);
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = row[t + 16 * k];
        SCHED_FENCE();
        int bound = w_lim(W);
        fwd_stages<W, 0, 3>(x, w1, q, bound);
        SCHED_FENCE();
        tw_load_last<0, 3>(w2, tw, lc + 4, 16 * b + t);      // into the registers that the first three stages' factors leave
        SCHED_FENCE();
        fwd_stages<W, 3, 4>(x, w1, q, bound);
        SCHED_FENCE();
        tw_load_last<3, 4>(w2, tw, lc + 4, 16 * b + t);
        SCHED_FENCE();
#pragma unroll
        for (int k = 0; k < 16; k++) s[t + 17 * k] = x[k];
        wave_exchange();
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = s[17 * t + j];
        fwd_stages<W, 0, 4>(x, w2, q, bound);
    } else {
        u64 w[4][6];
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = row[t + 64 * k];
        tw_row4(w, tw, lc, b, t);
        row4_fwd<W, 1>(reinterpret_cast<u64 (&)[1][4]>(x), w, s, 272, Row4(t), q);
    }
    if (!EPI) {
        if ((W == 0 || W == W_NEAR) && a.lazy) {
#pragma unroll
            for (int j = 0; j < PTS; j++) x[j] = fwd_lazy<W>(x[j], m);
        } else {
#pragma unroll
            for (int j = 0; j < PTS; j++) x[j] = reduce_min<7>(fwd_positive<W>(x[j], q), q, m.bits, m.rec);
        }
        if constexpr (LANES == 16) {
            wave_exchange();
#pragma unroll
            for (int j = 0; j < 16; j++) s[17 * t + j] = x[j];
            wave_exchange();
#pragma unroll
            for (int k = 0; k < 16; k++) row[t + 16 * k] = s[t + 17 * k];
        } else {
            const Row4 at(t);
            wave_exchange();
            at.store(3, x, s);
            wave_exchange();
            const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(s + row4_word(2 * t)), u = *reinterpret_cast<const ulonglong2*>(s + row4_word(128 + 2 * t));
            STORE2(row + 2 * t) = v;
            STORE2(row + 128 + 2 * t) = u;
        }
        return;
    }
    // out = (acc - ntt) * P^-1 + sigma(c0) + self: the product is below 5q whatever its factor, so the transform value may
    // stay as it is where what makes it positive (fwd_raw_bias: 128q, near moduli 24q) plus the accumulator (below 6q) fits 63 bits, else below
    // 2q; the sum is below 7q
    const bool raw = fwd_raw<W>(m);
    if (!raw) {
#pragma unroll
        for (int j = 0; j < PTS; j++) x[j] = reduce_lazy<7>(fwd_positive<W>(x[j], q), q, m.bits, m.rec);
    }
    wave_exchange();
    const uint32_t e0 = LANES == 16 ? 16 * t : 4 * row4_last(t);       // x[j] = point e0 + j of the row
#pragma unroll
    for (int j = 0; j < PTS; j++) s[e0 + j + ((e0 + j) >> 4)] = x[j];
    const u64 bias = raw ? fwd_raw_bias<W>(q) : 2 * q;
    const uint32_t pc = limb / ep.L1, r = limb - pc * ep.L1, job = pc >> 1, comp = pc & 1u, row0 = b * 256;
    const u64 pinv = uni64(ep.pinv[r]), pinv_sh = uni64(ep.pinv_sh[r]), n2q = opaque_s(0 - 2 * q), pinv_h = split_factor<true>(pinv, pinv_sh, n2q);
    const size_t ro = (size_t)r << logN;
    u64* out = (comp ? ep.out1[job] : ep.out0[job]) + ro;
    const u64* c0p = comp == 0 ? ep.c0[job] : nullptr;
    const u64* sp = comp ? ep.self1[job] : ep.self0[job];
    const bool has_c0 = c0p != nullptr, has_self = sp != nullptr;
    const u64* c0 = has_c0 ? c0p + ro : nullptr;
    const u64* self = has_self ? sp + ro : nullptr;
    wave_exchange();
    const u64* acc = ep.acc + ((size_t)(pc * ep.R + r) << logN);
    const uint32_t g = ep.g[job];
    // an aligned pair of positions takes its rotated addends from an aligned pair, in order or swapped: one 16-byte load
    ulonglong2 av[PTS / 2];
#pragma unroll
    for (int p = 0; p < PTS / 2; p++) av[p] = LOAD2(acc + row0 + 2 * t + DP * p);
#pragma unroll
    for (int p = 0; p < PTS / 2; p++) {
        const uint32_t pos = row0 + 2 * t + DP * p, e = pos - row0, l = e + (e >> 4);
        ulonglong2 add = has_self ? LOAD2(self + pos) : make_ulonglong2(0, 0);
        if (has_c0) {
            const uint32_t src = g == 1 ? pos : galois_pos(pos, g, logN);
            const ulonglong2 c = LOAD2(c0 + (src & ~1u));
            add.x += src & 1u ? c.y : c.x;
            add.y += src & 1u ? c.x : c.y;
        }
        ulonglong2 o;
        o.x = reduce_min<7>(split_acc(add.x, av[p].x + bias - s[l], pinv, pinv_sh, pinv_h, n2q), q, m.bits, m.rec);
        o.y = reduce_min<7>(split_acc(add.y, av[p].y + bias - s[l + 1], pinv, pinv_sh, pinv_h, n2q), q, m.bits, m.rec);
        store2_stream(out + pos, o.x, o.y);
    }
}

template <bool EPI, int LANES>
__global__ __launch_bounds__(P2_THREADS, 4) void ntt_row_fwd_kernel(P2Args a, LimbTab tab, ModDownEpilogue ep) {
    ieee_off();
    __shared__ alignas(16) u64 sm[P2_THREADS / LANES * 272];         // 16 groups of 17: conflict-free both ways
    uint32_t tile;
    const uint32_t e = row_decode<LANES>(tab, a, tile);
    if (e == TAB_NONE) return;
    by_class(a.cls, tab_mod(e), e, [&](auto W, uint32_t v) { row_fwd<W, EPI, LANES>(a, v, tile, sm, ep); });
}

// ---------------------------------------------------------------- inverse row pass
// Stages LC+7 .. LC+4 on contiguous points, exchange, stages LC+3 .. LC on strided points: inputs below 2q, results below
// 2q (wide moduli: w_half).  Narrow moduli: bounds 2 -> 40 after the first block, -> 640 after the second, one quotient step at the end.
// LANES as in row_fwd.
template <int W, int LANES>
__device__ __forceinline__ void row_inv(const P2Args& a, const LimbTab& tab, uint32_t e, uint32_t tile, u64* sm) {
    const uint32_t mi = tab_mod(e), limb = tab_dst(e), logN = a.logN, lc = logN - 8;
    const ModConst m = mod_const(a.mc, mi);
    const ulonglong2* tw = a.tw + ((size_t)mi << logN);
    constexpr int DP = 2 * LANES, PTS = 256 / LANES;
    const uint32_t blk = threadIdx.x / LANES, t = threadIdx.x % LANES, b = tile * (P2_THREADS / LANES) + blk;
    u64* out = a.dst + ((size_t)limb << logN) + (size_t)b * 256;
    u64* s = sm + blk * 272;
    u64 x[PTS], w4[4][6];                                // w4: LANES == 64
    ulonglong2 w2[15];                                   // LANES == 16
    const u64* in = tab_src(tab, e, logN) + (size_t)b * 256;
    if constexpr (LANES == 16) {
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = in[t + 16 * k];
        tw_load_last<0, 4>(w2, tw, lc + 4, 16 * b + t);
        SCHED_FENCE();
#pragma unroll
        for (int k = 0; k < 16; k++) s[t + 17 * k] = x[k];
    } else {
        const ulonglong2 v = LOAD2(in + 2 * t), u = LOAD2(in + 128 + 2 * t);
        tw_row4(w4, tw, lc, b, t);
        *reinterpret_cast<ulonglong2*>(s + row4_word(2 * t)) = v;
        *reinterpret_cast<ulonglong2*>(s + row4_word(128 + 2 * t)) = u;
        wave_exchange();
        Row4(t).load(3, x, s);
    }
    const u64 q = m.q;
    if constexpr (LANES == 16) {
        wave_exchange();
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = s[17 * t + j];
        ulonglong2 w1[15];
        int bound = 2;
        inv_stages<W, 2, 4>(x, w2, q, bound);
        SCHED_FENCE();
        tw_load<2, 4>(w1, tw, lc, b);                        // into the registers that the first two stages' factors leave
        SCHED_FENCE();
        inv_stages<W, 0, 2>(x, w2, q, bound);
        SCHED_FENCE();
        tw_load<0, 2>(w1, tw, lc, b);
        SCHED_FENCE();
        wave_exchange();
#pragma unroll
        for (int j = 0; j < 16; j++) s[17 * t + j] = x[j];
        wave_exchange();
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = s[t + 17 * k];
        inv_stages<W, 0, 4>(x, w1, q, bound);
        if (W == 0 || W == W_NEAR) {
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = inv_end<W>(x[k], m);
        }
#pragma unroll
        for (int k = 0; k < 16; k++) out[t + 16 * k] = x[k];
    } else {
        row4_inv<W, 1>(reinterpret_cast<u64 (&)[1][4]>(x), w4, s, 272, Row4(t), q, m);
#pragma unroll
        for (int k = 0; k < 4; k++) out[t + 64 * k] = x[k];
    }
}

template <int LANES>
__global__ __launch_bounds__(P2_THREADS, 4) void ntt_row_inv_kernel(P2Args a, LimbTab tab) {
    ieee_off();
    __shared__ alignas(16) u64 sm[P2_THREADS / LANES * 272];
    uint32_t tile;
    const uint32_t e = row_decode<LANES>(tab, a, tile);
    if (e == TAB_NONE) return;
    by_class(a.cls, tab_mod(e), e, [&](auto W, uint32_t v) { row_inv<W, LANES>(a, tab, v, tile, sm); });
}

// ---------------------------------------------------------------- row passes of several limbs of one modulus
// Plain row passes where a launch holds many limbs of each modulus (a batch of polynomials, the digits of several key
// switches): a wavefront takes ONE row of 4 limbs at a time, 16 lanes each, and goes on with the same row of the next 4.
// The first block's factors are then the same for the wavefront (scalar registers), the second block's are loaded once for
// the whole run instead of once per limb.  384 limbs, N = 2^16, against the passes above: forward 105 -> 95 us, inverse
// 102 -> 95, near what the points alone take (403 MB, 82 us at copy rate).  Asking for the next four limbs' points ahead
// costs a third of the wavefronts and gave 110.
struct RunTab {
    uint32_t r[HE_MAX_LAUNCH_LIMBS / 4 + HE_MAX_MODULI];     // first entry of LimbTab (bits 0-8), limbs (9-13), modulus (14-19)
};
// what entry 4*it + i of the run gives for lane quarter i (the last entry's again where the run has fewer)
template <class F>
__device__ __forceinline__ auto run_pick(const LimbTab& tab, uint32_t first, uint32_t n, uint32_t it, uint32_t quarter, F&& f) {
    const auto v0 = f(tab.e[first + min(4 * it, n - 1)]), v1 = f(tab.e[first + min(4 * it + 1, n - 1)]);
    const auto v2 = f(tab.e[first + min(4 * it + 2, n - 1)]), v3 = f(tab.e[first + min(4 * it + 3, n - 1)]);
    return quarter & 2 ? (quarter & 1 ? v3 : v2) : (quarter & 1 ? v1 : v0);
}
// the first block's factors into scalar registers
__device__ __forceinline__ void run_tw1(ulonglong2 (&w)[15], const ulonglong2* tw, uint32_t s0, uint32_t b) {
#pragma unroll
    for (int u = 0; u < 4; u++)
#pragma unroll
        for (int g = 0; g < (1 << u); g++) {
            const const_u64 p = (const_u64)(uintptr_t)uni64((u64)(tw + ((1u << (s0 + u)) + (b << u) + g)));
            w[(1 << u) - 1 + g] = make_ulonglong2(p[0], p[1]);
        }
}
// The loop over a run uses the factors again and again: without this the compiler keeps the upper words of all of them in
// registers of their own besides (30 more, which then spill).
__device__ __forceinline__ void run_keep(ulonglong2 (&w)[15]) {
#pragma unroll
    for (int i = 0; i < 15; i++) asm("" : "+v"(w[i].x), "+v"(w[i].y));
}
template <int W, bool LAZY>
__device__ __forceinline__ void row_run_fwd(const P2Args& a, const LimbTab& tab, uint32_t run, uint32_t b, u64* sm) {
    const uint32_t first = run & 511u, n = (run >> 9) & 31u, logN = a.logN, lc = logN - 8, mi = tab_mod(tab.e[first]);
    const uint32_t quarter = (threadIdx.x >> 4) & 3u, t = threadIdx.x & 15u;
    const ulonglong2* tw = a.tw + ((size_t)mi << logN);
    u64* s = sm + (threadIdx.x >> 4) * 272;
    u64 x[16];
    ulonglong2 w1[15], w2[15];
    auto dst = [&](uint32_t e) { return tab_dst(__builtin_amdgcn_readfirstlane(e)); };
    u64* base = a.dst + b * 256u + t;
    run_tw1(w1, tw, lc, b);
    tw_load_last<0, 4>(w2, tw, lc + 4, 16 * b + t);
    const ModConst m = mod_const(a.mc, mi);
    const u64 q = m.q;
    for (uint32_t it = 0;; it++) {
        const uint32_t dl = run_pick(tab, first, n, it, quarter, dst);
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = base[((size_t)dl << logN) + 16 * k];
        SCHED_FENCE();
        int bound = w_lim(W);
        fwd_stages<W, 0, 4, true>(x, w1, q, bound);
#pragma unroll
        for (int k = 0; k < 16; k++) s[t + 17 * k] = x[k];
        wave_exchange();
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = s[17 * t + j];
        SCHED_FENCE();
        run_keep(w2);
        fwd_stages<W, 0, 4>(x, w2, q, bound);
        SCHED_FENCE();
        if ((W == 0 || W == W_NEAR) && LAZY) {
#pragma unroll
            for (int j = 0; j < 16; j++) x[j] = fwd_lazy<W>(x[j], m);
        } else {
#pragma unroll
            for (int j = 0; j < 16; j++) x[j] = reduce_min<7>(fwd_positive<W>(x[j], q), q, m.bits, m.rec);
        }
        wave_exchange();
#pragma unroll
        for (int j = 0; j < 16; j++) s[17 * t + j] = x[j];
        wave_exchange();
        if (4 * it + quarter < n) {
#pragma unroll
            for (int k = 0; k < 16; k++) base[((size_t)dl << logN) + 16 * k] = s[t + 17 * k];
        }
        if (4 * (it + 1) >= n) return;
        wave_exchange();
    }
}
template <int W>
__device__ __forceinline__ void row_run_inv(const P2Args& a, const LimbTab& tab, uint32_t run, uint32_t b, u64* sm) {
    const uint32_t first = run & 511u, n = (run >> 9) & 31u, logN = a.logN, lc = logN - 8, mi = tab_mod(tab.e[first]);
    const uint32_t quarter = (threadIdx.x >> 4) & 3u, t = threadIdx.x & 15u;
    const ulonglong2* tw = a.tw + ((size_t)mi << logN);
    u64* s = sm + (threadIdx.x >> 4) * 272;
    u64 x[16];
    ulonglong2 w1[15], w2[15];
    const uint32_t at = b * 256u + t;
    auto dst = [&](uint32_t e) { return tab_dst(__builtin_amdgcn_readfirstlane(e)); };
    auto src = [&](uint32_t e) { return uni64((u64)tab_src(tab, e, logN)); };
    tw_load_last<0, 4>(w2, tw, lc + 4, 16 * b + t);
    run_tw1(w1, tw, lc, b);
    const ModConst m = mod_const(a.mc, mi);
    const u64 q = m.q;
    for (uint32_t it = 0;; it++) {
        const u64* in = (const u64*)run_pick(tab, first, n, it, quarter, src) + at;
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = in[16 * k];
        const uint32_t dl = run_pick(tab, first, n, it, quarter, dst);
#pragma unroll
        for (int k = 0; k < 16; k++) s[t + 17 * k] = x[k];
        wave_exchange();
        SCHED_FENCE();
#pragma unroll
        for (int j = 0; j < 16; j++) x[j] = s[17 * t + j];
        int bound = 2;
        run_keep(w2);
        inv_stages<W, 0, 4>(x, w2, q, bound);
        SCHED_FENCE();
        wave_exchange();
#pragma unroll
        for (int j = 0; j < 16; j++) s[17 * t + j] = x[j];
        wave_exchange();
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = s[t + 17 * k];
        inv_stages<W, 0, 4, true>(x, w1, q, bound);
        if (W == 0 || W == W_NEAR) {
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = inv_end<W>(x[k], m);
        }
        if (4 * it + quarter < n) {
            u64* out = a.dst + ((size_t)dl << logN) + at;
#pragma unroll
            for (int k = 0; k < 16; k++) out[16 * k] = x[k];
        }
        if (4 * (it + 1) >= n) return;
        wave_exchange();
    }
}
// work group: 4 adjacent rows of one run
template <bool FWD, bool LAZY>
__global__ __launch_bounds__(P2_THREADS, 4) void ntt_row_run_kernel(P2Args a, LimbTab tab, RunTab runs) {
    ieee_off();
    __shared__ u64 sm[16 * 272];
    const uint32_t lb = a.logN - 10, b = (blockIdx.x & ((1u << lb) - 1u)) * 4u + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t run = __builtin_amdgcn_readfirstlane(runs.r[blockIdx.x >> lb]);
    by_class(a.cls, run >> 14 & 63u, run, [&](auto W, uint32_t v) {
        if constexpr (FWD) row_run_fwd<W, LAZY>(a, tab, v, b, sm);
        else row_run_inv<W>(a, tab, v, b, sm);
    });
}

// ---------------------------------------------------------------- butterfly-rate probe
// The vector-ALU roof of the transforms, measured rather than derived: the register blocks of the passes
// above (four stages on 16 points, twiddles from a 256-entry table that stays in the first-level cache)
// run back to back with no other memory traffic, for the class of the modulus.  Values wrap around after a few rounds; the timing
// does not depend on them.
template <bool FWD, int W>
__global__ __launch_bounds__(P2_THREADS) void bfly_probe_kernel(const ulonglong2* __restrict__ tw, u64 q,
                                                                 u64* __restrict__ out, uint32_t rounds) {
    ieee_off();
    const uint32_t t = threadIdx.x & 15;
    ulonglong2 w[15];
    u64 x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = (u64)(blockIdx.x * P2_THREADS + threadIdx.x) * 16 + k;
    for (uint32_t r = 0; r < rounds; r++) {
        tw_load<0, 4>(w, tw, 4, t);
        int b = FWD ? w_lim(W) : w_half(W);
        if (FWD) fwd_stages<W, 0, 4>(x, w, q, b);
        else inv_stages<W, 0, 4>(x, w, q, b);
    }
    u64 v = 0;
#pragma unroll
    for (int k = 0; k < 16; k++) v ^= x[k];
    out[blockIdx.x * P2_THREADS + threadIdx.x] = v;
}

int32_t probe_butterfly_rates(he_ctx* ctx, u64* d_out, uint32_t groups, double rate_out[3]) {
    static void (*const probes[2][4])(const ulonglong2*, u64, u64*, uint32_t) = {
        {bfly_probe_kernel<false, 0>, bfly_probe_kernel<false, 1>, bfly_probe_kernel<false, 2>, bfly_probe_kernel<false, W_NEAR>},
        {bfly_probe_kernel<true, 0>, bfly_probe_kernel<true, 1>, bfly_probe_kernel<true, 2>, bfly_probe_kernel<true, W_NEAR>}};
    const uint32_t rounds = 64;                          // 32 butterflies per thread per round
    uint32_t narrow = 0, wide = ctx->M;
    for (uint32_t i = 0; i < ctx->M; i++) if (!narrow_fwd(ctx->mod[i])) { wide = i; break; }
    hipEvent_t e0, e1;
    HE_HIP(ctx, hipEventCreate(&e0));
    HE_HIP(ctx, hipEventCreate(&e1));
    for (int which = 0; which < 3; which++) {
        const uint32_t mi = which == 2 ? wide : narrow;
        rate_out[which] = 0.0;
        if (mi >= ctx->M) continue;
        const bool fwd = which != 1;
        const ulonglong2* tw = (fwd ? ctx->d_tw : ctx->d_itw) + (size_t)mi * ctx->N;
        const u64 q = ctx->mod[mi];
        void (*const kernel)(const ulonglong2*, u64, u64*, uint32_t) = probes[fwd][fwd ? class_fwd(q, ctx->logN) : class_inv(q)];
        for (int rep = 0; rep < 2; rep++) {              // the first launch warms up
            HE_HIP(ctx, hipEventRecord(e0, ctx->stream));
            hipLaunchKernelGGL(kernel, dim3(groups), dim3(P2_THREADS), 0, ctx->stream, tw, q, d_out, rounds);
            HE_HIP(ctx, hipGetLastError());
            HE_HIP(ctx, hipEventRecord(e1, ctx->stream));
            HE_HIP(ctx, hipEventSynchronize(e1));
        }
        float ms = 0.f;
        HE_HIP(ctx, hipEventElapsedTime(&ms, e0, e1));
        rate_out[which] = (double)groups * P2_THREADS * 32.0 * rounds / (ms * 1e-3);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return HE_OK;
}

// ---------------------------------------------------------------- host
#define COL_DISPATCH(K, SECOND, ...)                                                                              \
    switch (ctx->logN - 8) {                                                                                         \
    case 5: hipLaunchKernelGGL((K<5, SECOND>), __VA_ARGS__); break;                                                  \
    case 6: hipLaunchKernelGGL((K<6, SECOND>), __VA_ARGS__); break;                                                  \
    case 7: hipLaunchKernelGGL((K<7, SECOND>), __VA_ARGS__); break;                                                  \
    case 8: hipLaunchKernelGGL((K<8, SECOND>), __VA_ARGS__); break;                                                  \
    default: hipLaunchKernelGGL((K<9, SECOND>), __VA_ARGS__); break;                                                 \
    }
int32_t launch_transform2p(he_ctx* ctx, const TransformDesc& d) {
    const uint32_t n = d.n, logN = ctx->logN;
    const bool fwd = d.fwd;
    if (d.rescale_from && (!fwd || d.rescale_from > ctx->M || d.only_pass == 2))
        return he_fail(ctx, HE_ERR_BADARG, "transform: the Rescale rounding term is read by the first pass of a forward transform");
    // live limbs sorted by modulus (stable counting sort)
    LimbTab tab;
    uint32_t count[HE_MAX_MODULI] = {0}, start[HE_MAX_MODULI], live = 0, distinct = 0;
    for (uint32_t s = 0; s < HE_MAX_SEGS; s++) tab.seg[s] = s < d.n_seg ? d.seg[s] : d.seg[0];
    for (uint32_t i = 0; i < n; i++) {
        if (d.mod_idx[i] == 0xFFu) continue;
        if (d.mod_idx[i] >= ctx->M) return he_fail(ctx, HE_ERR_BADARG, "transform: modulus index %u out of range", d.mod_idx[i]);
        count[d.mod_idx[i]]++;
    }
    for (uint32_t m = 0; m < ctx->M; m++) { start[m] = live; live += count[m]; distinct += count[m] != 0; }
    if (live == 0) return HE_OK;
    for (uint32_t i = 0; i < n; i++) {
        const uint32_t mi = d.mod_idx[i];
        if (mi == 0xFFu) continue;
        const uint32_t seg = d.src_seg ? d.src_seg[i] : 0, lim = d.src_limb ? d.src_limb[i] : i;
        if (seg >= HE_MAX_SEGS || seg >= d.n_seg || lim >= 4096) return he_fail(ctx, HE_ERR_BADARG, "transform: source limb out of range");
        tab.e[start[mi]++] = i | (mi << 9) | (lim << 15) | (seg << 27);
    }
    // Plain row passes by runs of one modulus: fours of limbs, up to 16 in a run, shorter runs where the launch would not
    // fill the chip four times over.  Where more than a quarter of the lanes would have no limb, one limb at a time.
    RunTab runs;
    uint32_t n_runs = 0, fours = 0;
    for (uint32_t m = 0; m < ctx->M; m++) fours += (count[m] + 3) / 4;
    const bool by_runs = live >= 3 * fours;
    if (by_runs) {
        uint32_t piece = 16;
        const uint32_t groups = ctx->N >> 10;               // work groups per run
        while (piece > 4 && (live / piece) * groups < 4 * 768) piece >>= 1;
        for (uint32_t m = 0, at = 0; m < ctx->M; at += count[m++])
            for (uint32_t i = 0; i < count[m]; i += piece)
                runs.r[n_runs++] = (at + i) | (std::min(piece, count[m] - i) << 9) | (m << 14);
    }
    P2Args a;
    a.dst = d.dst; a.mc = ctx->d_mc;
    a.tw = fwd ? ctx->d_tw : ctx->d_itw;
    a.logN = logN;
    a.cls = fwd ? ctx->cls_fwd : ctx->cls_inv;
    a.lazy = (fwd && d.lazy_out) ? 1u : 0u;
    a.rs_mod = d.rescale_from ? d.rescale_from - 1 : 0;
    uint32_t lc = 0;
    while (lc < 4 && (2u << lc) * distinct <= live) lc++;      // chunk <= average group size, at most 16
    a.log_chunk = lc;
    // the work index of a workgroup runs over whole groups of 8 chunks x tiles: with the 2 tiles of the smallest ring the
    // limbs are padded so that every index a launch can form lies inside the table
    const uint32_t tiles = ctx->N >> 12, unit = std::max<uint32_t>(1u << lc, tiles < 8 ? (8u / tiles) << lc : 0u);
    const uint32_t padded = (live + unit - 1) / unit * unit;
    if (padded > HE_MAX_LAUNCH_LIMBS) return he_fail(ctx, HE_ERR_BADARG, "transform: too many limbs in one launch");
    for (uint32_t i = live; i < padded; i++) tab.e[i] = TAB_NONE;
    // A row is shared by 64 threads instead of 16 while 16 would make at most 4 wavefronts per SIMD, about what the chip holds at
    // once: such a launch is as long as one wavefront's chain of loads and butterflies, which is a fourth as long on four
    // times the wavefronts.  One rotation at level 5: 65 us with 16 threads, 55 with 64; at level 11 of N = 2^15 70 and 57.
    // With the line at 2048 two rotations at level 11 take 131.5 us instead of 129.1 and one at level 20 of the six-digit
    // set 187 instead of 182; at 8192 a block of layers takes 1255 instead of 1251, at 16384 that rotation 186 again.  Eight
    // at level 5 take 220 instead of 215 because their smallest launch falls under the line.
    const bool wide_rows = live * (ctx->N >> 10) <= 4096;
    const dim3 block(P2_THREADS), grid_cols(live * tiles), grid_rows(padded * tiles * (wide_rows ? 4 : 1));
    for (int pass = 0; pass < 2; pass++) {
        if (d.only_pass && d.only_pass != (uint32_t)pass + 1) continue;
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (ctx->prof_on) {
            HE_HIP(ctx, hipEventCreate(&e0));
            HE_HIP(ctx, hipEventCreate(&e1));
            HE_HIP(ctx, hipEventRecord(e0, ctx->stream));
        }
        if (fwd && pass == 0) {
            if (d.rescale_from) { COL_DISPATCH(ntt_col_fwd_kernel, true, grid_cols, block, 0, ctx->stream, a, tab) }
            else { COL_DISPATCH(ntt_col_fwd_kernel, false, grid_cols, block, 0, ctx->stream, a, tab) }
        } else if (fwd) {
            ModDownEpilogue none = {};
            if (d.ep && wide_rows) hipLaunchKernelGGL((ntt_row_fwd_kernel<true, 64>), grid_rows, block, 0, ctx->stream, a, tab, *d.ep);
            else if (d.ep) hipLaunchKernelGGL((ntt_row_fwd_kernel<true, 16>), grid_rows, block, 0, ctx->stream, a, tab, *d.ep);
            else if (by_runs && !wide_rows && a.lazy) hipLaunchKernelGGL((ntt_row_run_kernel<true, true>), dim3(n_runs * (ctx->N >> 10)), block, 0, ctx->stream, a, tab, runs);
            else if (by_runs && !wide_rows) hipLaunchKernelGGL((ntt_row_run_kernel<true, false>), dim3(n_runs * (ctx->N >> 10)), block, 0, ctx->stream, a, tab, runs);
            else if (wide_rows) hipLaunchKernelGGL((ntt_row_fwd_kernel<false, 64>), grid_rows, block, 0, ctx->stream, a, tab, none);
            else hipLaunchKernelGGL((ntt_row_fwd_kernel<false, 16>), grid_rows, block, 0, ctx->stream, a, tab, none);
        } else if (pass == 0) {
            if (by_runs && !wide_rows) hipLaunchKernelGGL((ntt_row_run_kernel<false, false>), dim3(n_runs * (ctx->N >> 10)), block, 0, ctx->stream, a, tab, runs);
            else if (wide_rows) hipLaunchKernelGGL((ntt_row_inv_kernel<64>), grid_rows, block, 0, ctx->stream, a, tab);
            else hipLaunchKernelGGL((ntt_row_inv_kernel<16>), grid_rows, block, 0, ctx->stream, a, tab);
        } else {
            const bool ahead = logN == 17 && grid_cols.x < 1024;     // four work groups to a compute unit: 25 limbs 23.5 us with it, 24.5 without, 32 both 26.9, 48 34.4 and 33.6
            const ScaleList none = {};
            if (ahead && d.scale) hipLaunchKernelGGL((ntt_col_inv_kernel<9, true, true>), grid_cols, block, 0, ctx->stream, a, tab, *d.scale, d.scale_period);
            else if (ahead) hipLaunchKernelGGL((ntt_col_inv_kernel<9, false, true>), grid_cols, block, 0, ctx->stream, a, tab, none, 1u);
            else if (d.scale) { COL_DISPATCH(ntt_col_inv_kernel, true, grid_cols, block, 0, ctx->stream, a, tab, *d.scale, d.scale_period) }
            else { COL_DISPATCH(ntt_col_inv_kernel, false, grid_cols, block, 0, ctx->stream, a, tab, none, 1u) }
        }
        HE_HIP(ctx, hipGetLastError());
        if (ctx->prof_on) {
            HE_HIP(ctx, hipEventRecord(e1, ctx->stream));
            const uint32_t kind = fwd ? (pass == 0 ? 0u : (d.ep ? 2u : 1u)) : (pass == 0 ? 3u : 5u);
            ctx->prof_events.push_back({e0, e1, live, 0u, kind});
        }
    }
    if (fwd) ctx->cnt.ntt_limbs += live; else ctx->cnt.intt_limbs += live;
    return HE_OK;
}
