// The row passes of key switches, N = 2^13 .. 2^17: the inner product and the transforms of ModDown around it, a wavefront per
// row, and before them the last eight stages of the digits whose source serves one job or one term of a sum of rotations.
//
// The Galois map takes whole rows of the 2^LC x 256 view to whole rows: k' = g*k + (g-1)/2 and the row of a position is the
// low LC bits of k (bit-reversed order).  So row b of an inner product needs exactly one row of every digit, row sigma(b), and
// that row can be transformed where it is used: it is read once in the state the column pass leaves it and permuted in LDS,
// where a transform launch of its own wrote and read back 72 of some 580 limb moves of a key switch at the benchmark's top
// level, and both components read it again.  Digits that several jobs use are transformed once instead (ntt2p.hip) and come
// here complete (DONE); fifteen rotations of each of three sources at level 18 of N = 2^16 (45 key switches) took 1782 us so, where
// sums formed inside the transforms of each component, which read every digit twice, took 1910.
//
//   special primes: rows of the digits -> products with both components of the key -> inverse rows of both sums;
//   q-limbs:        rows of the digits -> products -> rows of both converted components -> (acc - conv) * P^-1 + addends.
//
// What bounds it (cards differ by a few percent): bytes and issue together for the q-limbs (sixteen key switches at level 23 of N = 2^16
// in 415 us, 1.6 GiB moved at 4.2 TB/s, vector issue 0.67 of the slots at 2.4 GHz, 0.79 of those at the 2.05 GHz the clock has
// under this load; 4.5 TB/s and 0.58 or 0.68 where the digits are complete), vector issue for the special primes (161 us, 0.72 or
// 0.84: their 60-bit ranges take a conditional subtraction every other stage).  Nine-instruction products and two-instruction
// subtractions took 8 % of the instructions and 1 % of the time.  A key switch of a batch takes 26 + 10 us in these two launches where rows
// of the digits, sums with inverse rows and sums with the ModDown took 18 + 9 + 26.  A row is shared by a whole wavefront, 4 points
// a lane, because then the sums of both components stay in registers (8 sums of three words) and every product is formed once from
// digits that both components share.  With two wavefronts to a row, a component each, a batch of 240 (in sets of eight) took 24.9 ms
// instead of 19.4 (twice the preparation and twice the misses of the key rows in the first-level cache); three wavefronts to a SIMD
// instead of four 20.1.  Reading a digit back in the Galois map's order (KrRow::src) is not free of bank conflicts: 0.30 to 0.33 of the
// LDS cycles of these kernels, which issue an LDS instruction for every 17 to 21 vector ones.
//
// No kernel may spill registers, and the build refuses one that does (build.py): a build of the work-group form with 84 bytes of scratch a
// lane gave wrong sums, other ones each time, wherever two work groups shared a compute unit; the same code without spills gave
// right ones.  Why is not known.
//
// Digits and converted components are read once, in whole lines; they and the results go past the caches' usual replacement, so
// that the key's rows and the next launches' sources stay.  Calls whose results nobody reads: one key switch at level 23 149.9 -> 143.3
// us, eight hoisted ones at level 5 174.4 -> 165.9, 28 of N = 2^15 at level 11 579 -> 562, 240 of a batch 18.91 -> 18.72 ms.  In a layer
// the next launch reads the results; there it is about even, for small ciphertexts a little worse and for large ones better.  As streams /
// stored the usual way wherever the call itself reads them: 16 channels in the paper's order, 8 outputs, level 5 1016 / 1018 us on one
// card, 1125 / 1115 on another, 1050 / 1033 on a third, level 8 1289 / 1290, 14 2024 / 2043, 23 3376 / 3410 and 3550 / 3580; 16 outputs at
// level 5 1709 / 1720; its hoisted form at level 5 656 / 658; reordered layer, a ModDown per rotation, level 5 305 / 306, 20 967 / 974;
// five rotate-and-sum rounds of one ciphertext at level 5 279 / 277, of 16 at level 11 3158 / 3179.  Choosing by a flag of the launch
// costs one rotation at level 5 0.7 of its 57.5 us, so there is none.
//
// Work order: jobs (they come sorted by key) are the fastest index, then rows of the source; each XCD works on every eighth (limb,
// row), so that jobs under one key, whose rows of the key and of the factors are then one row too, and jobs of one source find
// them in that XCD's L2.  In the order of the results' rows jobs of one source shared only the factors: the rotations of three
// sources above 1686 us, so 1675.
#include <algorithm>

#include "modarith.h"
#include "ntt_blocks.h"

#define KR_WAVES 4
#define KR_THREADS (KR_WAVES * 64)
// Up to this many rows in a launch, one for each SIMD, a work group takes a row and spreads its digits over the wavefronts: the
// launch is then as long as one row's chain of transforms.  One rotation at level 2 of N = 2^13 (32 and 96 rows): 34.7 us with a
// wavefront to a row, 29.5 with a work group; level 5 of 2^14 39.5 and 34.8.  At 2048 one at level 5 of 2^16 (2048 and 1536
// rows) takes 59.9 instead of 56.6, six ciphertexts by eight amounts at 2^14 352 instead of 329.
#define KR_GROUP_ROWS 1024
// Digits that are transformed already leave a wavefront so little to do that up to this many rows each component gets one of its
// own, which transforms the converted component while the first digit is on its way.  The launches are then two rounds of
// wavefronts at most.  Four rotations of one source at level 5 of N = 2^14 46.2 us with one wavefront to a row, 42.1 so; two at
// level 11 of 2^16 (4096 and 6144 rows) 119.7 and 116.4; at 16384 eight rotations at level 5 of 2^16 (16384 and 12288 rows) 174.6
// instead of 171.2.
#define KR_HALF_ROWS 8192

// A lane works on points 4T .. 4T+3 of a row (row4_last) in the last block of a transform and on points 2t, 2t+1, 128+2t, 129+2t
// elsewhere, so that whatever it reads from memory there lies side by side.
__device__ __forceinline__ void kr_load(u64 (&x)[4], const u64* row, uint32_t t) {
    const ulonglong2 v = LOAD2(row + 2 * t), u = LOAD2(row + 128 + 2 * t);
    x[0] = v.x; x[1] = v.y; x[2] = u.x; x[3] = u.y;
}
// LDS words of point 2t and of the values that the lane's four points take from row bs
struct KrRow {
    uint32_t pos, src[4], bs;
    __device__ __forceinline__ explicit KrRow(uint32_t t) : pos(row4_word(2 * t)), src{}, bs(0) {}
    __device__ __forceinline__ void map(uint32_t row0, uint32_t t, uint32_t g, uint32_t logN) {
#pragma unroll
        for (int p = 0; p < 2; p++) {
            const uint32_t v = galois_pos(row0 + 2 * t + 128 * p, g, logN);
            src[2 * p] = row4_word(v & 255u);
            src[2 * p + 1] = src[2 * p] ^ 1u;            // aligned pairs come from aligned pairs
            bs = __builtin_amdgcn_readfirstlane(v >> 8);
        }
    }
    __device__ __forceinline__ void put(u64* buf, const u64 (&x)[4]) const {
        *reinterpret_cast<ulonglong2*>(buf + pos) = make_ulonglong2(x[0], x[1]);
        *reinterpret_cast<ulonglong2*>(buf + (pos ^ 2u) + 128) = make_ulonglong2(x[2], x[3]);
    }
    __device__ __forceinline__ void get(u64 (&x)[4], const u64* buf) const {
        const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(buf + pos), u = *reinterpret_cast<const ulonglong2*>(buf + (pos ^ 2u) + 128);
        x[0] = v.x; x[1] = v.y; x[2] = u.x; x[3] = u.y;
    }
};

// The row b with sigma_g(b) = bs.  Exponents of a row agree in their low `rows` bits, and 2k' + 1 = g (2k + 1).
__device__ __forceinline__ uint32_t kr_row_from(uint32_t bs, uint32_t g, uint32_t rows) {
    uint32_t inv = g;                                    // right in its low 3 bits, then 6, 12, 24
#pragma unroll
    for (int i = 0; i < 3; i++) inv *= 2 - g * inv;
    return __brev((inv * (2 * (__brev(bs) >> (32 - rows)) + 1)) >> 1) >> (32 - rows);
}

// W: 0 = narrow in both directions (ntt_blocks.h), 1 = only forward, 2 = in neither, 3 = the widest, 4 = near a multiple of 2^32 in both
// directions, 5 = only forward.
__device__ constexpr int kr_fwd(int W) { return W >= 4 ? W_NEAR : W < 2 ? 0 : W - 1; }      // classes of the transforms
__device__ constexpr int kr_inv(int W) { return W == 4 ? W_NEAR : W == 0 ? 0 : W == 3 ? 2 : 1; }

//
// Both components of the inner products of row b of limb r for one (source, key) term, added to the sums s; `spill`
// empties them when they hold KS_ROW_PRODUCTS products.  Digits enter as the row transform leaves them where W = 0 or 4 (below 90q <
// 2^60.2, 4: 46q: 31-bit high halves; seven products with key values below q, together below 2^117, fit the sums and split_reduce), else below
// 2q (1, 5) or canonical (2, 3).  5 reaches furthest: digits below 2^60.003 and keys of 2^59.003, of which seven products stay below 10.6 * 2^60 in
// the middle sum and below 2^121.9 together, where 2^(bits + 63) is 2^123.  buf: a row for each digit, of which
// digits j0, j0 + step .. are worked on (j0 < beta).  AHEAD: the next digit's row and the own one are asked for ahead of their turn.
template <int W, bool SP, bool AHEAD, class Spill>
__device__ __forceinline__ void ks_row_products(const KsRows& a, uint32_t id, uint32_t r, uint32_t b, uint32_t t, u64* buf, const ModConst& m, const Row4& at,
                                                KrRow& kr, SplitSum (&s)[2][4], uint32_t j0, uint32_t step, Spill&& spill) {
    const uint32_t logN = a.logN, mi = SP ? a.nq + r : r, row0 = b * 256;
    const size_t ro = (size_t)(SP ? a.L1 + r : r) << logN, dig_stride = (size_t)a.R << logN, comp_stride = (size_t)a.M << logN;
    const uint32_t own_j = SP ? 0xFFFFFFFFu : r / a.alpha;
    kr.map(row0, t, a.g[id], logN);
    const u64* row = a.raised[id] + ro + (size_t)kr.bs * 256;
    const u64* key = a.evk[id] + ((size_t)mi << logN) + row0;
    u64 own[4], kb[2][4], ka[2][4], w[4][6], x[1][4];
    const bool owns = !SP && own_j % step == j0;
    const u64* own_row = owns ? a.own[id] + ro + (size_t)kr.bs * 256 : nullptr;
    if (AHEAD && owns) kr_load(own, own_row, t);
    uint32_t j = j0 == own_j ? j0 + step : j0;
    if (j < a.beta) {
#pragma unroll
        for (int k = 0; k < 4; k++) x[0][k] = __builtin_nontemporal_load(&(row + j * dig_stride)[t + 64 * k]);
        tw_row4(w, a.tw + ((size_t)mi << logN), logN - 8, kr.bs, t);
#pragma unroll 1
        while (true) {
            const uint32_t jn = j + step == own_j ? j + 2 * step : j + step;
            u64 nx[4];
            if (AHEAD && jn < a.beta) {
#pragma unroll
                for (int k = 0; k < 4; k++) nx[k] = __builtin_nontemporal_load(&(row + jn * dig_stride)[t + 64 * k]);
            }
            SCHED_FENCE();
            if (!AHEAD && kr_fwd(W) != W_NEAR) {         // the factors' second words (near moduli have none) are formed anew, not kept in registers
#pragma unroll
                for (int i = 0; i < 18; i++) asm("" : "+v"(w[1 + i / 6][i % 6]));
            }
            row4_fwd<kr_fwd(W), 1>(x, w, buf + 256 * j, 256, at, m.q);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                x[0][k] = fwd_positive<kr_fwd(W)>(x[0][k], m.q);
                if (W == 1 || W == 5) x[0][k] = reduce_lazy<7>(x[0][k], m.q, m.bits, m.rec);
                if (W == 2 || W == 3) x[0][k] = reduce_min<7>(x[0][k], m.q, m.bits, m.rec);
            }
            wave_exchange();
            at.store(3, x[0], buf + 256 * j);
            if (jn >= a.beta) break;
            j = jn;
#pragma unroll
            for (int k = 0; k < 4; k++) x[0][k] = AHEAD ? nx[k] : __builtin_nontemporal_load(&(row + jn * dig_stride)[t + 64 * k]);
        }
    }
    if (!AHEAD && owns) kr_load(own, own_row, t);
    const size_t step_stride = 2 * step * comp_stride;
    key += 2 * j0 * comp_stride;
    kr_load(kb[0], key, t);
    kr_load(ka[0], key + comp_stride, t);
    if (owns) kr.put(buf + 256 * own_j, own);
    wave_exchange();
    auto digit = [&](const u64 (&b4)[4], const u64 (&a4)[4], u64 (&nb)[4], u64 (&na)[4]) {
        key += step_stride;
        if (j + step < a.beta) {
            kr_load(nb, key, t);
            kr_load(na, key + comp_stride, t);
        }
        u64 d[4];
#pragma unroll
        for (int k = 0; k < 4; k++) d[k] = buf[256 * j + kr.src[k]];
        SCHED_FENCE();
        spill();
#pragma unroll
        for (int k = 0; k < 4; k++) {
            split_mac(s[0][k], d[k], b4[k]);
            split_mac(s[1][k], d[k], a4[k]);
        }
        j += step;
    };
#pragma unroll 1
    for (j = j0; j < a.beta;) {
        digit(kb[0], ka[0], kb[1], ka[1]);
        if (j < a.beta) digit(kb[1], ka[1], kb[0], ka[0]);
    }
    wave_exchange();
}

// The same from digits that are transformed already (below 2q, canonical for wide moduli), for components c0 .. c0+NX-1.
// buf: two rows.  `first` runs while the first digit is on its way.
template <bool SP, int NX, class Spill, class First>
__device__ __forceinline__ void ks_row_products_done(const KsRows& a, uint32_t id, uint32_t r, uint32_t b, uint32_t t, u64* buf, KrRow& kr,
                                                     SplitSum (&s)[NX][4], uint32_t c0, Spill&& spill, First&& first) {
    const uint32_t logN = a.logN, mi = SP ? a.nq + r : r, row0 = b * 256, own_j = SP ? 0xFFFFFFFFu : r / a.alpha;
    const size_t ro = (size_t)(SP ? a.L1 + r : r) << logN, dig_stride = (size_t)a.R << logN, comp_stride = (size_t)a.M << logN;
    kr.map(row0, t, a.g[id], logN);
    const u64* row = a.raised[id] + ro + (size_t)kr.bs * 256;
    const u64* own = SP ? row : a.own[id] + ro + (size_t)kr.bs * 256;
    const u64* key = a.evk[id] + ((size_t)mi << logN) + row0 + c0 * comp_stride;
    u64 d[2][4], kv[2][NX][4];
    auto load = [&](uint32_t j, int n) {
        kr_load(d[n], j == own_j ? own : row + j * dig_stride, t);
#pragma unroll
        for (int c = 0; c < NX; c++) kr_load(kv[n][c], key + (2 * j + c) * comp_stride, t);
    };
    auto digit = [&](uint32_t j, int n) {
        kr.put(buf + 256 * n, d[n]);
        if (j + 1 < a.beta) load(j + 1, 1 - n);
        wave_exchange();
        u64 v[4];
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = buf[256 * n + kr.src[k]];
        SCHED_FENCE();
        spill();
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int c = 0; c < NX; c++) split_mac(s[c][k], v[k], kv[n][c][k]);
    };
    load(0, 0);
    SCHED_FENCE();
    first();
#pragma unroll 1
    for (uint32_t j = 0; j < a.beta; j += 2) {
        digit(j, 0);
        if (j + 1 < a.beta) digit(j + 1, 1);
    }
    wave_exchange();
}

// What follows the sums v of components c0 .. c0+NX-1 (below 6q; special primes: below 2q): inverse rows of the special primes, or
// rows of the converted components and the ModDown's last step.  w, cv: factors and input of the transform; buf: NX rows.
template <int W, int NX>
__device__ __forceinline__ void ks_row_special(const KsRows& a, uint32_t job, uint32_t c0, uint32_t r, uint32_t b, uint32_t t, u64* buf, const ModConst& m,
                                               const Row4& at, const KrRow& kr, const u64 (&w)[4][6], u64 (&v)[NX][4]) {
#pragma unroll
    for (int c = 0; c < NX; c++) kr.put(buf + 256 * c, v[c]);
    wave_exchange();
#pragma unroll
    for (int c = 0; c < NX; c++) at.load(3, v[c], buf + 256 * c);
    wave_exchange();
    row4_inv<kr_inv(W), NX>(v, w, buf, 256, at, m.q, m);
    u64* out = a.mid + ((size_t)((2 * job + c0) * a.k + r) << a.logN) + b * 256;
#pragma unroll
    for (int c = 0; c < NX; c++)
#pragma unroll
        for (int k = 0; k < 4; k++) (out + ((size_t)(c * a.k) << a.logN))[t + 64 * k] = v[c][k];
}
template <int NX>
__device__ __forceinline__ void ks_row_converted(u64 (&cv)[NX][4], const KsRows& a, uint32_t job, uint32_t c0, uint32_t r, uint32_t b, uint32_t t) {
    const u64* conv = a.mid + ((size_t)((2 * job + c0) * a.L1 + r) << a.logN) + b * 256;
#pragma unroll
    for (int c = 0; c < NX; c++)
#pragma unroll
        for (int k = 0; k < 4; k++) cv[c][k] = __builtin_nontemporal_load(&(conv + ((size_t)(c * a.L1) << a.logN))[t + 64 * k]);
}
// addends: the Galois image of c0 (row bs), and values that are added as they are
template <int NX>
struct KrAdd {
    u64 add[NX][4], rot[4];
    bool rotated;
    __device__ __forceinline__ void load(const KsRows& a, uint32_t job, uint32_t c0, uint32_t r, uint32_t b, uint32_t t, uint32_t bs) {
        const size_t qo = (size_t)r << a.logN;
        const u64* rp = c0 == 0 ? a.c0[job] : nullptr;
        rotated = rp != nullptr;
        if (rotated) kr_load(rot, rp + qo + (size_t)bs * 256, t);
#pragma unroll
        for (int c = 0; c < NX; c++) {
            const u64* self = c0 + c ? a.self1[job] : a.self0[job];
#pragma unroll
            for (int k = 0; k < 4; k++) add[c][k] = 0;
            if (self) kr_load(add[c], self + qo + b * 256, t);
        }
    }
};
// rows of the converted components, in the order of the sums
template <int W, int NX>
__device__ __forceinline__ void ks_row_transformed(u64 (&cv)[NX][4], u64* buf, const ModConst& m, const Row4& at, const KrRow& kr, const u64 (&w)[4][6]) {
    SCHED_FENCE();
    row4_fwd<kr_fwd(W), NX>(cv, w, buf, 256, at, m.q);
    const bool raw = fwd_raw<kr_fwd(W)>(m);
    wave_exchange();
#pragma unroll
    for (int c = 0; c < NX; c++) {
        if (!raw) {
#pragma unroll
            for (int k = 0; k < 4; k++) cv[c][k] = reduce_lazy<7>(fwd_positive<kr_fwd(W)>(cv[c][k], m.q), m.q, m.bits, m.rec);
        }
        at.store(3, cv[c], buf + 256 * c);
    }
    wave_exchange();
#pragma unroll
    for (int c = 0; c < NX; c++) kr.get(cv[c], buf + 256 * c);
    wave_exchange();
}
// Inverse rows of a result's second component, where it is what the next key switch raises: the row is in LDS already, and its digits are used
// once (not DONE: no registers or branch there).  A step of a rotate-and-sum loses the launch it began with.  us before/now, N = 2^16: layer of 16 channels,
// 8 outputs, level 5, 993/950, with its taps deferred and 3 outputs at level 6 831/809, block at level 6 1490/1453; at level 23, where the rows fill the
// vector units, 3268/3258.  In the kernel of small launches a branch for it cost one rotation 51.9 -> 52.7, so that has two forms (NEXT).
template <int W>
__device__ __forceinline__ void ks_row_next(const KsRows& a, uint32_t job, uint32_t r, uint32_t b, uint32_t t, u64* buf, const ModConst& m, const KrRow& kr, const u64 (&o)[4]) {
    u64 w[4][6], x[1][4];
    kr.put(buf, o);
    SCHED_FENCE();
    asm("" : "+v"(t));                                   // what follows from the lane is worked out anew, not kept in registers
    const Row4 at(t);
    tw_row4(w, a.itw + ((size_t)r << a.logN), a.logN - 8, b, t);
    wave_exchange();
    at.load(3, x[0], buf);
    wave_exchange();
    row4_inv<kr_inv(W), 1>(x, w, buf, 256, at, m.q, m);
    u64* out = a.next[job] + ((size_t)r << a.logN) + b * 256;
#pragma unroll
    for (int k = 0; k < 4; k++) out[t + 64 * k] = x[0][k];
}
template <int W, int NX, bool NEXT>
__device__ __forceinline__ void ks_row_down(const KsRows& a, uint32_t job, uint32_t c0, uint32_t r, uint32_t b, uint32_t t, u64* buf, const ModConst& m,
                                            const KrRow& kr, u64 (&cv)[NX][4], const u64 (&v)[NX][4], KrAdd<NX>& ad) {
    const uint32_t row0 = b * 256;
    const size_t qo = (size_t)r << a.logN;
    // out = (acc - conv) * P^-1 + addends: the product is below 5q whatever its factor, so the transform value may stay as it is
    // where what it can be plus the accumulator (below 6q) fits 63 bits, else below 2q; the sum is below 7q
    const bool raw = fwd_raw<kr_fwd(W)>(m);
    const u64 bias = raw ? fwd_raw_bias<kr_fwd(W)>(m.q) : 2 * m.q, pinv = ((const_u64)(uintptr_t)a.pinv)[r], pinv_sh = ((const_u64)(uintptr_t)a.pinv_sh)[r];
    const u64 n2q = opaque_s(0 - 2 * m.q), pinv_h = split_factor<true>(pinv, pinv_sh, n2q);
    if (ad.rotated) {
        kr.put(buf, ad.rot);
        wave_exchange();
#pragma unroll
        for (int k = 0; k < 4; k++) ad.add[0][k] += buf[kr.src[k]];
    }
#pragma unroll
    for (int c = 0; c < NX; c++) {
        u64* out = (c0 + c ? a.out1[job] : a.out0[job]) + qo + row0 + 2 * t;
        u64 o[4];
#pragma unroll
        for (int k = 0; k < 4; k++)
            o[k] = reduce_min<7>(split_acc(ad.add[c][k], v[c][k] + bias - cv[c][k], pinv, pinv_sh, pinv_h, n2q), m.q, m.bits, m.rec);
        store2_stream(out, o[0], o[1]);
        store2_stream(out + 128, o[2], o[3]);
        if (NEXT && c0 + c == 1 && a.next[job]) ks_row_next<W>(a, job, r, b, t, buf, m, kr, o);
    }
}
// v = (v + sums) below 2q, the sums empty again
template <int NX>
__device__ __forceinline__ void kr_flush(u64 (&v)[NX][4], SplitSum (&s)[NX][4], const ModConst& m) {
#pragma unroll
    for (int c = 0; c < NX; c++) {
        u64 p[4];
        split_reduce(p, s[c], m);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            v[c][k] = reduce_lazy<7>(v[c][k] + p[k], m.q, m.bits, m.rec);
            s[c][k] = SplitSum{0, 0, 0};
        }
        SCHED_FENCE();
    }
}

// One wavefront: row b of limb r for one job.  MANY: more than KS_ROW_PRODUCTS digits.
template <int W, bool SP, bool MANY, bool DONE>
__device__ __forceinline__ void ks_row(const KsRows& a, uint32_t job, uint32_t r, uint32_t b, uint32_t t, u64* buf) {
    const uint32_t mi = SP ? a.nq + r : r, lc = a.logN - 8;
    const ModConst m = mod_const(a.mc, mi);
    KrRow kr(t);
    u64 w[4][6], v[2][4] = {}, cv[2][4];
    SplitSum s[2][4] = {};
    uint32_t pending = 0;
    auto spill = [&]() {
        if (MANY && pending == KS_ROW_PRODUCTS) { kr_flush(v, s, m); pending = 0; }
        pending++;
    };
    if constexpr (DONE) ks_row_products_done<SP, 2>(a, job, r, b, t, buf, kr, s, 0, spill, []() {});
    else ks_row_products<W, SP, true>(a, job, r, b, t, buf, m, Row4(t), kr, s, 0, 1, spill);
    SCHED_FENCE();
    if (MANY) kr_flush(v, s, m);
    else split_reduce(v[0], s[0], m);
    SCHED_FENCE();
    asm("" : "+v"(t));                                   // what follows from the lane is worked out anew, not kept in registers
    if (!SP) ks_row_converted(cv, a, job, 0, r, b, t);
    tw_row4(w, (SP ? a.itw : a.tw) + ((size_t)mi << a.logN), lc, b, t);
    SCHED_FENCE();
    if (!MANY) split_reduce(v[1], s[1], m);
    SCHED_FENCE();
    if (SP) {
        if (!MANY) {
#pragma unroll
            for (int i = 0; i < 8; i++) v[i / 4][i % 4] = reduce_lazy<7>(v[i / 4][i % 4], m.q, m.bits, m.rec);
        }
        ks_row_special<W, 2>(a, job, 0, r, b, t, buf, m, Row4(t), kr, w, v);
    } else {
        KrAdd<2> ad;
        ad.load(a, job, 0, r, b, t, kr.bs);
        ks_row_transformed<W, 2>(cv, buf, m, Row4(t), kr, w);
        ks_row_down<W, 2, !DONE>(a, job, 0, r, b, t, buf, m, kr, cv, v, ad);
    }
}
// One wavefront: one component of that, from digits that are transformed already.  buf: two rows.
template <int W, bool SP>
__device__ __forceinline__ void ks_row_half(const KsRows& a, uint32_t job, uint32_t c, uint32_t r, uint32_t b, uint32_t t, u64* buf) {
    const uint32_t mi = SP ? a.nq + r : r;
    const ModConst m = mod_const(a.mc, mi);
    KrRow kr(t);
    u64 w[4][6], v[1][4] = {}, cv[1][4];
    SplitSum s[1][4] = {};
    KrAdd<1> ad;
    if (!SP) ks_row_converted(cv, a, job, c, r, b, t);
    tw_row4(w, (SP ? a.itw : a.tw) + ((size_t)mi << a.logN), a.logN - 8, b, t);
    ks_row_products_done<SP, 1>(a, job, r, b, t, buf, kr, s, c, []() {}, [&]() {
        if (SP) return;
        ks_row_transformed<W, 1>(cv, buf, m, Row4(t), kr, w);
        asm("" : "+v"(t));                               // what follows from the lane is worked out anew, not kept in registers
        ad.load(a, job, c, r, b, t, kr.bs);
    });
    SCHED_FENCE();
    kr_flush(v, s, m);
    if (SP) ks_row_special<W, 1>(a, job, c, r, b, t, buf, m, Row4(t), kr, w, v);
    else ks_row_down<W, 1, false>(a, job, c, r, b, t, buf, m, kr, cv, v, ad);
}
// A work group of nw wavefronts: row b of limb r, the terms (SUM) or the digits spread over the wavefronts; the first two then take
// a component each.  buf: LDS of the work group, max(beta, 2) rows a wavefront.
template <int W, bool SP, bool SUM, bool DONE, bool NEXT>
__device__ __forceinline__ void ks_row_group(const KsRows& a, uint32_t job, uint32_t r, uint32_t b, uint32_t wave, uint32_t nw, uint32_t t, u64* buf) {
    const uint32_t mi = SP ? a.nq + r : r, lc = a.logN - 8;
    const ModConst m = mod_const(a.mc, mi);
    KrRow kr(t);
    const uint32_t per_wave = 256 * (DONE ? 2u : max(a.beta, 2u));
    u64* part = buf + per_wave * wave;                   // the wavefront's digits, then its two sums
    u64 v[2][4] = {};
    SplitSum s[2][4] = {};
    uint32_t pending = 0;
    auto spill = [&]() {
        if (SUM && pending == KS_ROW_PRODUCTS) { kr_flush(v, s, m); pending = 0; }
        pending++;
    };
    if (SUM) {
#pragma unroll 1
        for (uint32_t i = wave; i < a.n_terms; i += nw) {
            asm("" : "+v"(t));                           // what follows from the lane is worked out anew, not kept in registers
            if constexpr (DONE) ks_row_products_done<SP, 2>(a, i, r, b, t, part, kr, s, 0, spill, []() {});
            else ks_row_products<W, SP, false>(a, i, r, b, t, part, m, Row4(t), kr, s, 0, 1, spill);
        }
    } else if (wave < a.beta) {
        ks_row_products<W, SP, false>(a, job, r, b, t, part, m, Row4(t), kr, s, wave, nw, spill);
    }
    SCHED_FENCE();
    kr_flush(v, s, m);
#pragma unroll
    for (int c = 0; c < 2; c++) kr.put(part + 256 * c, v[c]);
    SCHED_FENCE();
    asm("" : "+v"(t));
    u64 w[4][6], cv[1][4], sum[1][4] = {};
    KrAdd<1> ad;
    if (wave < 2) {
        if (!SUM) kr.map(b * 256, t, a.g[job], a.logN);
        if (!SP) {
            ks_row_converted(cv, a, job, wave, r, b, t);
            ad.load(a, job, wave, r, b, t, kr.bs);
        }
        tw_row4(w, (SP ? a.itw : a.tw) + ((size_t)mi << a.logN), lc, b, t);
    }
    __syncthreads();
    if (wave >= 2) return;
#pragma unroll 1
    for (uint32_t i = 0; i < nw; i++) {
        u64 o[4];
        kr.get(o, buf + per_wave * i + 256 * wave);
#pragma unroll
        for (int k = 0; k < 4; k++) sum[0][k] += o[k];
    }
#pragma unroll
    for (int k = 0; k < 4; k++) sum[0][k] = reduce_lazy<7>(sum[0][k], m.q, m.bits, m.rec);
    u64* mine = buf + 256 * wave;                        // a sum that only this wavefront has read
    wave_exchange();
    if (SP) ks_row_special<W, 1>(a, job, wave, r, b, t, mine, m, Row4(t), kr, w, sum);
    else {
        ks_row_transformed<W, 1>(cv, mine, m, Row4(t), kr, w);
        ks_row_down<W, 1, NEXT>(a, job, wave, r, b, t, mine, m, kr, cv, sum, ad);
    }
}

// W of a modulus (ks_width, he_internal.h), from the argument list: the branch waits for no load of its constants.  (Near or not first: on the
// number put together from its bits the compiler orders the bodies so that one rotation of other moduli at level 5 takes 54.1 us instead of 53.5.)
__device__ __forceinline__ uint32_t kr_width(const KsRows& a, uint32_t mi) {
    const uint32_t low = (uint32_t)(a.width[0] >> mi & 1u);
    if (a.width[2] >> mi & 1u) return low ? 5 : 4;
    return low + 2 * (uint32_t)(a.width[1] >> mi & 1u);
}
template <int W>
__device__ __forceinline__ uint32_t kr_pin(uint32_t v) {     // keeps the widths' loads apart (by_class, ntt_blocks.h)
    if (W == 0) asm("; narrow" : "+s"(v));
    else if (W == 1) asm("; narrow forward" : "+s"(v));
    else if (W == 2) asm("; wide" : "+s"(v));
    else if (W == 4) asm("; near" : "+s"(v));
    else if (W == 5) asm("; near forward" : "+s"(v));
    else asm("; widest" : "+s"(v));
    return v;
}

// A wavefront per (limb, row, job), jobs fastest; each XCD works on every eighth (limb, row).
template <bool SP, bool MANY, bool DONE>
__global__ __launch_bounds__(KR_THREADS, MANY ? 3 : 4) void ks_rows_kernel(KsRows a) {
    ieee_off();
    extern __shared__ __attribute__((aligned(16))) u64 sm[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rows = a.logN - 8;
    const uint32_t item = (blockIdx.x >> 3) * KR_WAVES + wave, un = item / a.J, job = item - un * a.J;
    const uint32_t u = un * 8 + (blockIdx.x & 7u), r = u >> rows;
    if (r >= (SP ? a.k : a.L1)) return;
    const uint32_t b = kr_row_from(u & ((1u << rows) - 1u), a.g[job], rows);
    u64* buf = sm + wave * (256 * (DONE ? 2u : max(a.beta, 2u)));
    const uint32_t width = kr_width(a, SP ? a.nq + r : r), t = threadIdx.x & 63u;
    if (width == 4) ks_row<4, SP, MANY, DONE>(a, job, kr_pin<4>(r), b, t, buf);
    else if (width == 5) ks_row<5, SP, MANY, DONE>(a, job, kr_pin<5>(r), b, t, buf);
    else if (width == 0) ks_row<0, SP, MANY, DONE>(a, job, kr_pin<0>(r), b, t, buf);
    else if (width == 1) ks_row<1, SP, MANY, DONE>(a, job, kr_pin<1>(r), b, t, buf);
    else if (width == 2) ks_row<2, SP, MANY, DONE>(a, job, kr_pin<2>(r), b, t, buf);
    else ks_row<3, SP, MANY, DONE>(a, job, kr_pin<3>(r), b, t, buf);
}
// A wavefront per (limb, row, job, component).
template <bool SP>
__global__ __launch_bounds__(KR_THREADS, 4) void ks_rows_half_kernel(KsRows a) {
    ieee_off();
    __shared__ __attribute__((aligned(16))) u64 sm[KR_WAVES * 512];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rows = a.logN - 8, t = threadIdx.x & 63u;
    const uint32_t at = (blockIdx.x >> 3) * KR_WAVES + wave, item = at >> 1, un = item / a.J, job = item - un * a.J;
    const uint32_t u = un * 8 + (blockIdx.x & 7u), r = u >> rows;
    if (r >= (SP ? a.k : a.L1)) return;
    const uint32_t b = kr_row_from(u & ((1u << rows) - 1u), a.g[job], rows);
    u64* buf = sm + 512 * wave;
    const uint32_t width = kr_width(a, SP ? a.nq + r : r);
    if (width == 4) ks_row_half<4, SP>(a, job, at & 1u, kr_pin<4>(r), b, t, buf);
    else if (width == 5) ks_row_half<5, SP>(a, job, at & 1u, kr_pin<5>(r), b, t, buf);
    else if (width == 0) ks_row_half<0, SP>(a, job, at & 1u, kr_pin<0>(r), b, t, buf);
    else if (width == 1) ks_row_half<1, SP>(a, job, at & 1u, kr_pin<1>(r), b, t, buf);
    else if (width == 2) ks_row_half<2, SP>(a, job, at & 1u, kr_pin<2>(r), b, t, buf);
    else ks_row_half<3, SP>(a, job, at & 1u, kr_pin<3>(r), b, t, buf);
}
// A work group per (limb, row) of a sum, or per (limb, row, job).
template <bool SP, bool SUM, bool DONE, bool NEXT = false>
__global__ __launch_bounds__(KR_THREADS, SUM && DONE ? 2 : 3) void ks_rows_group_kernel(KsRows a) {
    ieee_off();
    extern __shared__ __attribute__((aligned(16))) u64 sm[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6, rows = a.logN - 8, t = threadIdx.x & 63u;
    const uint32_t item = blockIdx.x >> 3, un = item / a.J, job = item - un * a.J;
    const uint32_t u = un * 8 + (blockIdx.x & 7u), r = u >> rows, b = u & ((1u << rows) - 1u);
    const uint32_t width = kr_width(a, SP ? a.nq + r : r);
    if (width == 4) ks_row_group<4, SP, SUM, DONE, NEXT>(a, job, kr_pin<4>(r), b, wave, nw, t, sm);
    else if (width == 5) ks_row_group<5, SP, SUM, DONE, NEXT>(a, job, kr_pin<5>(r), b, wave, nw, t, sm);
    else if (width == 0) ks_row_group<0, SP, SUM, DONE, NEXT>(a, job, kr_pin<0>(r), b, wave, nw, t, sm);
    else if (width == 1) ks_row_group<1, SP, SUM, DONE, NEXT>(a, job, kr_pin<1>(r), b, wave, nw, t, sm);
    else if (width == 2) ks_row_group<2, SP, SUM, DONE, NEXT>(a, job, kr_pin<2>(r), b, wave, nw, t, sm);
    else ks_row_group<3, SP, SUM, DONE, NEXT>(a, job, kr_pin<3>(r), b, wave, nw, t, sm);
}

int32_t launch_ks_rows(he_ctx* ctx, KsRows& a, bool special) {
    const uint32_t limbs = special ? a.k : a.L1, units = limbs << (ctx->logN - 8);
    if (a.J == 0 || a.J > HE_MAX_KS_JOBS || a.n_terms == 0 || a.n_terms > HE_MAX_KS_JOBS || (a.sum && a.J != 1) || (!a.sum && a.n_terms != 1) ||
        a.beta == 0 || a.beta > 8 || ctx->logN < 13 || ctx->logN > 17 || limbs == 0 || limbs > HE_MAX_MODULI)
        return he_fail(ctx, HE_ERR_BADARG, "key-switch rows: bad shape");
    if (a.next[0] && (a.sum || a.done)) return he_fail(ctx, HE_ERR_BADARG, "key-switch rows: inverse rows of sums or from complete digits");
    a.mc = ctx->d_mc; a.tw = ctx->d_tw; a.itw = ctx->d_itw; a.logN = ctx->logN;
    for (int b = 0; b < 3; b++) a.width[b] = ctx->ks_width[b];
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventCreate(&e0));
        HE_HIP(ctx, hipEventCreate(&e1));
        HE_HIP(ctx, hipEventRecord(e0, ctx->stream));
    }
    const uint32_t n_rows = units * a.J;
    const bool many = a.beta > KS_ROW_PRODUCTS;
    const bool group = a.sum || (!a.done && n_rows <= KR_GROUP_ROWS), half = !a.sum && a.done && !many && n_rows <= KR_HALF_ROWS;
    const uint32_t nw = group ? std::max(2u, std::min<uint32_t>(KR_WAVES, a.sum ? a.n_terms : a.beta)) : KR_WAVES;
    const dim3 grid(group ? n_rows : 8 * ((n_rows / 8 * (half ? 2 : 1) + KR_WAVES - 1) / KR_WAVES)), block(64 * nw);
    const size_t lds = half ? 0 : (size_t)nw * 256 * (a.done ? 2u : std::max(a.beta, 2u)) * sizeof(u64);       // at most 64 KiB
#define KR_LAUNCH(...) hipLaunchKernelGGL((__VA_ARGS__), grid, block, lds, ctx->stream, a)
#define KR_DISPATCH(SP)                                                                                                             \
    do {                                                                                                                            \
        if (a.sum && a.done) KR_LAUNCH(ks_rows_group_kernel<SP, true, true>);                                                       \
        else if (a.sum) KR_LAUNCH(ks_rows_group_kernel<SP, true, false>);                                                           \
        else if (half) KR_LAUNCH(ks_rows_half_kernel<SP>);                                                                          \
        else if (group && a.next[0]) KR_LAUNCH(ks_rows_group_kernel<SP, false, false, !SP>);                                        \
        else if (group) KR_LAUNCH(ks_rows_group_kernel<SP, false, false>);                                                          \
        else if (many && a.done) KR_LAUNCH(ks_rows_kernel<SP, true, true>);                                                         \
        else if (many) KR_LAUNCH(ks_rows_kernel<SP, true, false>);                                                                  \
        else if (a.done) KR_LAUNCH(ks_rows_kernel<SP, false, true>);                                                                \
        else KR_LAUNCH(ks_rows_kernel<SP, false, false>);                                                                           \
    } while (0)
    if (special) KR_DISPATCH(true);
    else KR_DISPATCH(false);
    HE_HIP(ctx, hipGetLastError());
    const uint32_t sources = a.sum ? a.n_terms : a.J, sums = 2 * a.J * limbs;
    const uint32_t digits = a.done ? 0 : sources * (special ? a.beta * a.k : (a.beta - 1) * a.L1);      // transformed here
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventRecord(e1, ctx->stream));
        ctx->prof_events.push_back({e0, e1, digits + sums, a.done ? sources * a.beta * limbs : 0u, special ? 4u : 2u});
    }
    // transforms whose column pass was a launch of its own are counted there
    if (a.count_up) ctx->cnt.ntt_limbs += digits;
    if (a.count_down) (special ? ctx->cnt.intt_limbs : ctx->cnt.ntt_limbs) += sums;
    return HE_OK;
}
