// Basis conversion with its column passes: inverse column pass of the sources -> conversion -> forward column pass of every
// target, in one launch (N = 2^13 .. 2^16, at most 8 sources).
//
// The three steps work on columns of the 2^LC x 256 view, so a work group takes a tile of 1024 points (C = 1024 / 2^LC
// columns) of all its limbs through them and neither the coefficient-form sources nor the converted limbs ever reach
// memory.  Separate kernels moved 24 + 24 + 24 + 72 + 72 + 72 limbs for one ModUp at the benchmark's top level, this one 24
// + 72, and the conversion alone took 17 % of a rotation.
//
// One wavefront owns one limb during the transforms (16 points per lane), so that an exchange stays inside the wavefront and
// needs no barrier.  The conversion is a contraction - every target residue is a fixed linear combination of the same 8
// source residues - and runs on the matrix cores: with y_i = sum_a u_(i,a) 2^(8a) the bytes of source i,
//     sum_i y_i * hat_i = sum_(i,a) u_(i,a) * V_(i,a)  (mod q),   V_(i,a) = hat_i * 2^(8a) mod q, centred,
// is a product over k = (source, byte), 64 of them, whose right factors split into 8 signed base-256 digits b:
// v_mfma_i32_16x16x64_i8 with the digits as rows and 16 points as columns.  A source residue in memory order IS the operand
// (each byte minus 128, which the constant term returns).  Two instructions give 16 points x 4 targets x 8 digits, laid
// out so that a lane gets the 8 digit sums of one (point, target); they are put together and reduced below 2q in 16
// vector instructions, where the vector-unit form of the same sum takes 68 (baseconv_kernel).
//
// What bounds it is vector issue: 4828 instructions per wavefront for 8 + 24 limbs (counters; 5969 with products of eleven and more
// instructions, sums put together in 22 and operands fetched one by one), 4 cycles each, fill 0.62 of the issue slots at 2.4 GHz
// and 0.73 of those at the 2.05 GHz that the clock has under this load; 2.75 TB/s move and wavefronts wait 0.41 of their cycles.
// Sets of sixteen, 24 limbs and eight special primes: 311 us a launch so, 261 to 267 now; with the tiles' accesses side by
// side (wrong results, a probe) 240, without stores 209, and the instructions alone are some 185.
// Small launches are chains (level 5, tiles of 256 points, in cycles of a work group): sources asked for at 2900 after a start of
// 5700, 500 of waiting, 4600 until they are transformed (3500 of them issue), 2700 at the barrier and 2500 in the conversion.
// Asking for the round's list before the sources takes one rotation at level 5 from 57.3 to 56.8 us, with six digits at level 6 from
// 61.0 to 59.6; asking for the operands themselves as well gave nothing.
#include <algorithm>

#include "modarith.h"
#include "ntt_blocks.h"

#define CC_THREADS 512
#define CC_WAVES 8
#define CC_REGION 1088            // LDS words of one limb's tile: 16 runs of 64, 4 spare words after each

typedef int v4i __attribute__((ext_vector_type(4)));
static_assert(alignof(ConvOperand) % alignof(v4i) == 0 && offsetof(ConvOperand, bias) % alignof(v4i) == 0, "read as v4i");

// Word of (run k, lane): a lane that holds rows t + k*T of column cl keeps them at run k, lane t*C + cl.
__device__ __forceinline__ uint32_t cc_word(uint32_t k, uint32_t lane) { return 68 * k + lane; }
// Row r of column cl.
template <int LC>
__device__ __forceinline__ uint32_t cc_row(uint32_t r, uint32_t cl) {
    constexpr uint32_t LT = LC - 4, LCOLS = 10 - LC;
    return cc_word(r >> LT, ((r & ((1u << LT) - 1u)) << LCOLS) + cl);
}
// Factors of the second register block (rows 16t .. 16t+15): 2^LC - 16 entries of the table in a row, which a wavefront reads once, side by side,
// and keeps in its LDS region.  Read from memory where they are used, the four or more lanes of a row group each asked for the same
// 16 bytes fifteen times over, as much work for the memory pipeline as the points themselves: without those loads (uniform factors, wrong
// results) the conversions of 240 rotations took 8449 us instead of 8947.
template <int LC>
struct CcFactors {
    static constexpr int N = LC >= 8 ? 4 : LC == 7 ? 2 : 1;       // loads of 64 entries from the table's first
    static constexpr uint32_t LAST = 1u << (LC - 1);              // first entry of the last stage, whose eight a row group are one apart from the next eight
    v2u64 v[N];
    static __device__ __forceinline__ uint32_t word(uint32_t k, uint32_t lane) {
        if (64 * k >= LAST) return 64 * k + (64 * k - LAST) / 8 + lane + (lane >> 3);
        return 64 * k + lane + (64 * k + 63 >= LAST && lane >= LAST ? (lane - LAST) >> 3 : 0);
    }
    __device__ __forceinline__ void load(ctw_t tw, uint32_t lane) {
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = (tw + 64 * k)[lane];
    }
    __device__ __forceinline__ void put(u64* reg, uint32_t lane) const {
#pragma unroll
        for (int k = 0; k < N; k++) reinterpret_cast<v2u64*>(reg)[word(k, lane)] = v[k];
    }
    // factors G0 .. G1-1 of stage LC-4+u for rows 16t .. 16t+15
    template <int G0, int G1>
    static __device__ __forceinline__ void get(ulonglong2 (&w)[15], const u64* reg, int u, uint32_t t) {
        const v2u64* p = reinterpret_cast<const v2u64*>(reg) + (u == 3 ? 9 * t : t << u);
#pragma unroll
        for (int g = G0; g < G1; g++) { const v2u64 f = p[(1u << (LC - 4 + u)) + g]; w[(1 << u) - 1 + g] = make_ulonglong2(f.x, f.y); }
    }
    template <int U0>
    static __device__ __forceinline__ void first(ulonglong2 (&w)[15], const u64* reg, uint32_t t) {       // the stages before the last
        if (U0 < 1) get<0, 1>(w, reg, 0, t);
        if (U0 < 2) get<0, 2>(w, reg, 1, t);
        if (U0 < 3) get<0, 4>(w, reg, 2, t);
    }
};
// Inverse column stages of one source limb, output scaling, canonical residues into the limb's LDS region.
template <int LC, int W>
__device__ __forceinline__ void cc_source(u64* reg, const u64* src, const ColConv& cc, const ScaleList& sc, uint32_t mi, uint32_t si,
                                          uint32_t lane, uint32_t c0, const ModConst* mc, const ulonglong2* itw) {
    constexpr int LT = LC - 4, LCOLS = 10 - LC, U0 = 8 - LC;
    const uint32_t t = lane >> LCOLS, cl = lane & ((1u << LCOLS) - 1u), c = c0 + cl;
    const ctw_t tw = (ctw_t)(uintptr_t)(itw + ((size_t)mi << (LC + 8)));
    u64 x[16];
    ulonglong2 w1[15], w2[15];
    CcFactors<LC> f;
    f.load(tw, lane);
#pragma unroll
    for (int j = 0; j < 16; j++) x[j] = (src + j * 256)[t * 4096 + c];
    const const_u64 mp = (const_u64)(uintptr_t)(mc + mi);
    const u64 q = uni64(mp[0]);
    const u64 cs = sc.s[si], cs_sh = sc.s_sh[si], cw = sc.w[si], cw_sh = sc.w_sh[si];
    int bound = w_start(W);
    f.put(reg, lane);
    wave_exchange();
    f.template first<U0>(w2, reg, t);
    f.template get<0, 8>(w2, reg, 3, t);
    inv_stages<W, U0, 4>(x, w2, q, bound);
    wave_exchange();
#pragma unroll
    for (int j = 0; j < 16; j++) reg[cc_row<LC>(16 * t + j, cl)] = x[j];
    tw_load_c<1, 4>(w1, tw, 0, 0);
    wave_exchange();
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = reg[cc_word(k, lane)];
    inv_stages<W, 1, 4, true>(x, w1, q, bound);
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const u64 X = x[k], Y = x[k + 8];
        x[k] = inv_scaled<W>(X + Y, cs, cs_sh, q);
        x[k + 8] = inv_scaled<W>(W == W_NEAR ? X - Y : (X + q * (u64)bound) - Y, cw, cw_sh, q);
    }
    // each byte less 128, as the signed operand of the matrix instruction
#pragma unroll
    for (int k = 0; k < 16; k++) reg[cc_word(k, lane)] = inv_canonical<W>(x[k], q) ^ 0x8080808080808080ull;
    (void)LT;
}

// Forward column stages of one target limb from its LDS region (below 2q, or centred) to memory.
// `before`: what goes ahead of the stores, for which later loads wait.
template <int LC, int W, class Before>
__device__ __forceinline__ void cc_target(u64* reg, u64* dst, uint32_t mi, const ulonglong2 (&w1)[15], uint32_t lane, uint32_t c0, const ModConst* mc, const ulonglong2* ftw,
                                          Before&& before) {
    constexpr int LCOLS = 10 - LC, U0 = 8 - LC;
    const uint32_t t = lane >> LCOLS, cl = lane & ((1u << LCOLS) - 1u), c = c0 + cl;
    const ctw_t tw = (ctw_t)(uintptr_t)(ftw + ((size_t)mi << (LC + 8)));
    const const_u64 mp = (const_u64)(uintptr_t)(mc + mi);
    const u64 q = uni64(mp[0]);
    ulonglong2 w2[15];
    CcFactors<LC> f;
    f.load(tw, lane);
    u64 x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = reg[cc_word(k, lane)];
    int b = 2;
    fwd_stages<W, 0, 4, true>(x, w1, q, b);
    wave_exchange();
#pragma unroll
    for (int k = 0; k < 16; k++) reg[cc_word(k, lane)] = x[k];
    wave_exchange();
#pragma unroll
    for (int j = 0; j < 16; j++) x[j] = reg[cc_row<LC>(16 * t + j, cl)];
    wave_exchange();
    f.put(reg, lane);
    wave_exchange();
    f.template first<U0>(w2, reg, t);
    // the last stage's eight factors come in two halves, each into the registers that earlier factors leave: with the
    // source bytes that stay for the next targets there is no room for all of them
    if (U0 < 2) fwd_stages<W, (U0 < 2 ? U0 : 2), 2>(x, w2, q, b);
    SCHED_FENCE();
    f.template get<0, 4>(w2, reg, 3, t);
    SCHED_FENCE();
    if (U0 < 3) fwd_stages<W, (U0 < 2 ? 2 : U0), (U0 < 3 ? 3 : U0)>(x, w2, q, b);
    SCHED_FENCE();
    f.template get<4, 8>(w2, reg, 3, t);
    SCHED_FENCE();
    fwd_stages<W, 3, 4>(x, w2, q, b);
    before();
#pragma unroll
    for (int j = 0; j < 16; j++) (dst + j * 256)[t * 4096 + c] = x[j];
}

// ---------------------------------------------------------------- tiles of 256 points, 4 per lane
// For launches that leave the chip mostly idle: a fourth of the butterflies in a row and four times the work groups.  Point
// e = row * C + column of the tile; block i runs stages 2i and 2i + 1 (with odd LC the last block only its first), where lane
// t holds points c4_point(i, t, k).
__device__ __forceinline__ uint32_t c4_point(int i, uint32_t t, int k) {
    const uint32_t ls = 6 - 2 * i;
    return ((t >> ls) << (ls + 2)) + (t & ((1u << ls) - 1u)) + ((uint32_t)k << ls);
}
__device__ __forceinline__ uint32_t c4_word(uint32_t e) { return e + (e >> 4); }
template <int LC>
struct C4 {
    static constexpr int LCOLS = 8 - LC, NB = (LC + 1) / 2;
    static __device__ __forceinline__ uint32_t at(uint32_t e, uint32_t c0) { return ((e >> LCOLS) << 8) + c0 + (e & ((1u << LCOLS) - 1u)); }
};
template <int LC>
__device__ __forceinline__ void c4_factors(u64 (&w)[4][6], const ulonglong2* tw, uint32_t t) {
#pragma unroll
    for (int i = 0; i < C4<LC>::NB; i++) tw_block2(w[i], tw, 2 * i, t >> (6 - 2 * i));
}
template <int LC, int W>
__device__ __forceinline__ void c4_source(u64* reg, const u64* src, const ScaleList& sc, uint32_t mi, uint32_t si, uint32_t t, uint32_t c0,
                                          const ModConst* mc, const ulonglong2* itw) {
    using G = C4<LC>;
    u64 x[4], w[4][6];
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = src[G::at(c4_point(G::NB - 1, t, k), c0)];
    c4_factors<LC>(w, itw + ((size_t)mi << (LC + 8)), t);
    const u64 q = uni64(mc[mi].q), cs = sc.s[si], cs_sh = sc.s_sh[si];
    int bound = w_start(W);                            // narrow rows arrive below 2q: 2, 10, 40, 160, at the end 640
#pragma unroll
    for (int i = G::NB - 1; i >= 0; i--) {
        if (i + 1 < G::NB) {
            wave_exchange();
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] = reg[c4_word(c4_point(i, t, k))];
        }
        if (2 * i + 1 >= LC) inv_block2_r<W, false, true>(x, w[i], q, bound);
        else if (i == 0) inv_block2_r<W, true>(x, w[i], q, bound);         // its factors are the same for the whole limb
        else inv_block2_r<W>(x, w[i], q, bound);
#pragma unroll
        for (int k = 0; k < 4; k++)
            reg[c4_word(c4_point(i, t, k))] = i ? x[k] : csub_min(W == W_NEAR ? near_acc<true>(q, x[k], make_ulonglong2(cs, cs_sh), NearQ(q)) : shoup_lazy(x[k], cs, cs_sh, q), q) ^ 0x8080808080808080ull;
    }
}
template <int LC, int W, class Before>
__device__ __forceinline__ void c4_target(u64* reg, u64* dst, uint32_t mi, const u64 (&w)[4][6], uint32_t t, uint32_t c0, const ModConst* mc, Before&& before) {
    using G = C4<LC>;
    const u64 q = uni64(mc[mi].q);
    u64 x[4];
    int b = 2;
#pragma unroll
    for (int i = 0; i < G::NB; i++) {
        if (i) wave_exchange();
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = reg[c4_word(c4_point(i, t, k))];
        if (2 * i + 1 >= LC) fwd_block2_r<W, false, true>(x, w[i], q, b);
        else if (i == 0) fwd_block2_r<W, true>(x, w[i], q, b);                // its factors are the same for the whole limb
        else fwd_block2_r<W>(x, w[i], q, b);
        if (i + 1 < G::NB) {
#pragma unroll
            for (int k = 0; k < 4; k++) reg[c4_word(c4_point(i, t, k))] = x[k];
        }
    }
    before();
#pragma unroll
    for (int k = 0; k < 4; k++) dst[G::at(c4_point(G::NB - 1, t, k), c0)] = x[k];
}

// The lane's number: what follows from it is worked out anew, not kept in registers
__device__ __forceinline__ uint32_t lane_again() {
    uint32_t l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
    return l;
}

// grid: (parts * tiles, sets, repetitions), so that nothing has to be divided, or loaded first, to find the set.  Work groups go to the
// XCDs round-robin: each XCD gets neighbouring tiles of a group, so that the tiles that share a memory line are read and written
// through one L2.
template <int LC, int PTS>
__global__ __launch_bounds__(CC_THREADS, 4) void col_conv_kernel(ColConv cc, ScaleList sc, const ModConst* mc, const ulonglong2* ftw,
                                                                 const ulonglong2* itw) {
    ieee_off();
    constexpr int LCOLS = (PTS == 16 ? 10 : 8) - LC, TPX = (256 >> LCOLS) / 8;       // tiles of a group per XCD
    constexpr int REGION = PTS == 16 ? CC_REGION : 272, NB = PTS / 2;                // LDS words of a limb's tile, blocks of 16 points per wavefront
    __shared__ __attribute__((aligned(16))) u64 lds[CC_WAVES * REGION];
    __shared__ ConvOperand ops[CC_WAVES];                                              // of a round's targets
    auto point = [](uint32_t w, int b, uint32_t p16) {
        return PTS == 16 ? cc_word(2 * w + (b >> 2), 16 * (b & 3) + p16) : c4_word(32 * w + 16 * b + p16);
    };
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t slot = blockIdx.x >> 3, tile = (blockIdx.x & 7u) * TPX + slot % TPX, rep = blockIdx.z, c0 = tile << LCOLS;
    const ColConvSet& st = cc.set[blockIdx.y];
    u64* reg = lds + w * REGION;
    const uint32_t tb = slot / TPX * cc.share, nt = min(st.nt, tb + cc.share);
    // the first round's list is asked for before the sources: everything else of the round waits for it
    u64 mods = uni64(*reinterpret_cast<const u64*>(st.mod + tb)), lims = uni64(*reinterpret_cast<const u64*>(st.limb + tb));
    // this wavefront's part of the next round's operands on its way to LDS; a target beyond the list: the round's first
    u64 op_dig;
    uint32_t op_rest;
    auto op_load = [&](uint32_t t0) {
        const uint32_t m = t0 + w < nt ? (uint32_t)(mods >> (8 * w)) & 255u : (uint32_t)mods & 255u;
        const ConvOperand* p = st.op + m;
        const uint32_t l = lane_again();
        op_dig = reinterpret_cast<const u64*>(p)[l];
        op_rest = reinterpret_cast<const uint32_t*>(p)[128 + (l & 15u)];
    };
    auto op_store = [&]() {
        const uint32_t l = lane_again();
        reinterpret_cast<u64*>(ops + w)[l] = op_dig;
        if (l < 16) reinterpret_cast<uint32_t*>(ops + w)[128 + l] = op_rest;
    };
    op_load(tb);
    // 4 points: all factors, of the first round's target ahead of the sources (small launches have the registers, and a round each)
    u64 w4[4][6];
    auto factors4 = [&](uint32_t t0) {
        const uint32_t m = t0 + w < nt ? (uint32_t)(mods >> (8 * w)) & 255u : (uint32_t)mods & 255u;
        c4_factors<LC>(w4, ftw + ((size_t)m << (LC + 8)), lane_again());
    };
    if (PTS == 4) factors4(tb);
    if (w < st.ns) {
        const u64* src = st.src + (size_t)rep * cc.src_stride + ((size_t)w << (LC + 8));
        const uint32_t mi = st.mod0 + w;
        by_class(cc.inv, mi, mi, [&](auto W, uint32_t m) {
            if constexpr (PTS == 4) c4_source<LC, W>(reg, src, sc, m, st.sc0 + w, lane, c0, mc, itw);
            else cc_source<LC, W>(reg, src, cc, sc, m, st.sc0 + w, lane, c0, mc, itw);
        });
    }
    op_store();
    __syncthreads();
    // this wavefront's eighth of the points of every source; lane group g = lane / 16 holds sources 2g, 2g+1 of 16
    // points, in memory order the bytes k = 16g .. 16g+15 of the contraction
    v4i frag[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const uint32_t g = lane >> 4, word = point(w, b, lane & 15);
        const u64 y0 = 2 * g < st.ns ? lds[(2 * g) * REGION + word] : 0;
        const u64 y1 = 2 * g + 1 < st.ns ? lds[(2 * g + 1) * REGION + word] : 0;
        frag[b] = v4i{(int)(uint32_t)y0, (int)(uint32_t)(y0 >> 32), (int)(uint32_t)y1, (int)(uint32_t)(y1 >> 32)};
    }
    for (uint32_t t0 = tb; t0 < nt; t0 += CC_WAVES) {
        uint32_t ln = lane_again();
        const uint32_t g = ln >> 4, p16 = ln & 15;
        // this wavefront's target and the factors of its first block, which arrive during the conversion
        const bool have = t0 + w < nt;
        const uint32_t mi = have ? (uint32_t)(mods >> (8 * w)) & 255u : (uint32_t)mods & 255u, li = (uint32_t)(lims >> (8 * w)) & 255u;
        ulonglong2 w1[15];                                   // 16 points per lane
        if constexpr (PTS == 16) tw_load_c<0, 4>(w1, (ctw_t)(uintptr_t)(ftw + ((size_t)mi << (LC + 8))), 0, 0);
        else if (t0 != tb) factors4(t0);
        __syncthreads();                                     // the regions are free (operands read, last targets done)
        // four targets (s) at a time: lane group g works on target t0 + 4s + g and this lane supplies row lane % 16 = (target (lane
        // % 16) / 4, digit lane % 4) of the left factor
#pragma unroll
        for (int s = 0; s < 2; s++) {
            if (t0 + 4 * s >= nt) break;
            const v4i* A = reinterpret_cast<const v4i*>(ops[4 * s + (p16 >> 2)].dig + (p16 & 3) * 64 + g * 16);
            const v4i* K = reinterpret_cast<const v4i*>(ops[4 * s + g].bias);
            const v4i a0 = A[0], a1 = A[16], k0 = K[0], k1 = K[1], mk = K[2];      // digits 0..3, digits 4..7 (256 bytes on); -q, rec, bits
            const uint32_t centre = (uint32_t)K[3].x;
            const uint32_t n0 = (uint32_t)mk.x, n1 = (uint32_t)mk.y, rec = (uint32_t)mk.z, bits = (uint32_t)mk.w;
            // quotient of a value below 2^(bits+14) from its 32 bits above bit 32 + sh (sh at most 10)
            const uint32_t sh = bits > 50 ? bits - 50 : 0, e = bits - 33 - sh, up = 16 - sh;
            u64* out = lds + (4 * s + g) * REGION;
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const v4i d0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, frag[b], k0, 0, 0, 0);
                const v4i d1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, frag[b], k1, 0, 0, 0);
                // p01 and p23 are positive (conv_operand), the upper two of either sign; the value is lo + 2^32 * (p45 + 2^16 p67)
                const int p01 = d0.x + (d0.y << 8), p23 = d0.z + (d0.w << 8), p45 = d1.x + (d1.y << 8), p67 = d1.z + (d1.w << 8);
                const u64 lo = mad_wide((uint32_t)p23, 65536u, (uint32_t)p01);
                const int top = (int)add3((uint32_t)p45, (uint32_t)(lo >> 32), centre);
                const uint32_t qh = __umulhi(((uint32_t)p67 << up) + (uint32_t)(top >> sh), rec) >> e;
                const u64 v = (u64)qh * n0 + lo;
                const uint32_t vh = add3((uint32_t)(v >> 32), ((uint32_t)p67 << 16) + (uint32_t)p45, qh * n1);
                out[point(w, b, p16)] = ((u64)vh << 32) | (uint32_t)v;       // a target beyond the list: a region that nobody reads
            }
        }
        __syncthreads();
        // The next round's operands are asked for here and put down before this round's results are stored: loads behind the stores
        // would wait for them, which took a fourth of a wavefront's time.
        const bool more = t0 + CC_WAVES < nt;
        if (more) {
            mods = uni64(*reinterpret_cast<const u64*>(st.mod + t0 + CC_WAVES));
            lims = uni64(*reinterpret_cast<const u64*>(st.limb + t0 + CC_WAVES));
            op_load(t0 + CC_WAVES);
        }
        auto before = [&]() { if (more) op_store(); };
        ln = lane_again();
        if (have) {
            u64* dst = st.dst + (size_t)rep * cc.dst_stride + ((size_t)li << (LC + 8));
            by_class(cc.fwd, mi, mi, [&](auto W, uint32_t m) {
                if constexpr (PTS == 4) c4_target<LC, W>(reg, dst, m, w4, ln, c0, mc, before);
                else cc_target<LC, W>(reg, dst, m, w1, ln, c0, mc, ftw, before);
            });
        }
    }
}

int32_t launch_col_conv(he_ctx* ctx, ColConv& cc, const ScaleList& sc, uint32_t reps, uint32_t limb_passes) {
    const uint32_t groups = cc.n_sets * reps, LC = ctx->logN - 8;
    if (groups == 0) return HE_OK;
    if (LC < 5 || LC > 8 || cc.n_sets > CC_MAX_SETS) return he_fail(ctx, HE_ERR_BADARG, "column conversion: bad shape");
    uint32_t rounds = 1;
    for (uint32_t s = 0; s < cc.n_sets; s++) {
        const ColConvSet& st = cc.set[s];
        rounds = std::max(rounds, (st.nt + CC_WAVES - 1) / CC_WAVES);
        if (st.ns == 0 || st.ns > CC_WAVES || st.nt == 0 || st.nt > HE_MAX_MODULI || st.mod0 + st.ns > ctx->M || st.sc0 + st.ns > HE_MAX_MODULI ||
            !st.src || !st.dst || !st.op)
            return he_fail(ctx, HE_ERR_BADARG, "column conversion: bad group %u", s);
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventCreate(&e0));
        HE_HIP(ctx, hipEventCreate(&e1));
        HE_HIP(ctx, hipEventRecord(e0, ctx->stream));
    }
    const uint32_t tiles16 = 1u << (LC - 2);
    // Tiles of 256 points while the rounds of all 1024-point tiles would not give every second compute unit a work group (the
    // sources of a tile are at most 8, one phase, and are not counted).  One rotation at level 5 of N = 2^16: 63.0 us with the
    // large tiles, 55.3 with the small ones; at level 5 of 2^14 44.6 and 35.2, at level 2 of 2^13 36.1 and 30.2.  With the line at
    // 192 three rotations at level 5 take 106.2 us instead of 101.3 and eight at level 2 of 2^13 44.1 instead of 41.4; at 256 one at
    // level 11 takes 93.5 instead of 84.8.  At 64 one at level 5 takes 56.9.
    const bool small = groups * tiles16 * rounds <= 128;
    const uint32_t work = groups * tiles16 * (small ? 4 : 1);
    // While every compute unit has at most one work group, the rounds of a tile run side by side, each with the inverse pass of
    // its own: a ciphertext product and its rescale at level 11 takes 127 us instead of 136, one rotation at level 15 92 instead of
    // 104.  Up to two work groups per compute unit, where the tiles alone are 192 or 256, one rotation at level 23 takes 140.0 us
    // instead of 130.1, at level 19 132.0 instead of 122.7, two at level 11 124.1 instead of 115.7, a product at level 23 208.4 instead of
    // 198.5; nothing measured was faster so by more than the runs differ.
    const uint32_t parts = std::max(1u, std::min(rounds, 256 / work));
    cc.share = (rounds + parts - 1) / parts * CC_WAVES;
    const dim3 grid(tiles16 * (small ? 4 : 1) * ((rounds * CC_WAVES + cc.share - 1) / cc.share), cc.n_sets, reps), block(CC_THREADS);
#define CC_LAUNCH(LC_)                                                                                                                        \
    case LC_:                                                                                                                                 \
        if (small) hipLaunchKernelGGL((col_conv_kernel<LC_, 4>), grid, block, 0, ctx->stream, cc, sc, ctx->d_mc, ctx->d_tw, ctx->d_itw);        \
        else hipLaunchKernelGGL((col_conv_kernel<LC_, 16>), grid, block, 0, ctx->stream, cc, sc, ctx->d_mc, ctx->d_tw, ctx->d_itw);             \
        break;
    switch (LC) { CC_LAUNCH(5) CC_LAUNCH(6) CC_LAUNCH(7) CC_LAUNCH(8) }
    HE_HIP(ctx, hipGetLastError());
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventRecord(e1, ctx->stream));
        ctx->prof_events.push_back({e0, e1, limb_passes, 0u, 0u});
    }
    return HE_OK;
}
