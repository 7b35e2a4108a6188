// Column passes of Rescale in one launch, N = 2^13 .. 2^17: the dropped limb's inverse columns, and for every other modulus the
// forward columns of the negated rounding term ((v + h) mod q_l) mod q - (h mod q), h = floor(q_l / 2), of its coefficients v.
//
// Separate passes wrote the coefficients of two limbs and read each of them back for every modulus, in two launches that leave the
// chip mostly idle: 6.7 and 11.3 us after a product at level 11 of N = 2^16, 13.8 in one.  What bounds it is a wavefront's chain, load -
// eight stages - eight stages for each of its moduli, so a tile has 1024 points with 4 to a lane: all but one exchange stay inside a
// wavefront and the memory's runs are 32 bytes (a tile to a wavefront, 256 points, has runs of 8 bytes at N = 2^16: 123 us where
// this takes 117).
#include <algorithm>

#include "modarith.h"
#include "ntt_blocks.h"

#define RS_THREADS 256
#define RS_LDS 1088

// Point e = row * C + column of a tile of 1024 points (C = 1024 / 2^LC columns); 4 points a lane.  Block 0 (stages 0 and 1) has
// points thread + 256 k; what follows stays inside the 256 points of a wavefront, whose block i >= 1 runs stages 2i and 2i + 1 (with
// odd LC the last one only its first).
template <int LC>
struct RsTile {
    static constexpr int LCOLS = 10 - LC, NB = (LC + 1) / 2;
    uint32_t wave, t;
    __device__ __forceinline__ uint32_t point(int i, int k) const {
        if (i == 0) return wave * 64 + t + 256 * k;
        const uint32_t ls = 8 - 2 * i;
        return wave * 256 + ((t >> ls) << (ls + 2)) + (t & ((1u << ls) - 1u)) + ((uint32_t)k << ls);
    }
    static __device__ __forceinline__ uint32_t word(uint32_t e) { return e + (e >> 4); }
    static __device__ __forceinline__ uint32_t at(uint32_t e, uint32_t c0) { return ((e >> LCOLS) << 8) + c0 + (e & ((1u << LCOLS) - 1u)); }
    // the first two blocks' are the same for the wavefront (scalar registers)
    __device__ __forceinline__ void factors(u64 (&w)[NB][6], const ulonglong2* tw) const {
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const uint32_t b0 = (1u << (2 * i)) + (i ? wave : 0), b1 = 2 * b0;
            const const_u64 p0 = (const_u64)(uintptr_t)uni64((u64)(tw + b0)), p1 = (const_u64)(uintptr_t)uni64((u64)(tw + b1));
            w[i][0] = p0[0]; w[i][1] = p0[1];
            w[i][2] = p1[0]; w[i][3] = p1[1]; w[i][4] = p1[2]; w[i][5] = p1[3];
        }
#pragma unroll
        for (int i = 2; i < NB; i++) tw_block2(w[i], tw, 2 * i, (wave << (2 * i - 2)) + (t >> (8 - 2 * i)));
    }
    __device__ __forceinline__ void load(u64 (&x)[4], const u64* buf, int i) const {
#pragma unroll
        for (int k = 0; k < 4; k++) x[k] = buf[word(point(i, k))];
    }
    __device__ __forceinline__ void store(u64* buf, const u64 (&x)[4], int i) const {
#pragma unroll
        for (int k = 0; k < 4; k++) buf[word(point(i, k))] = x[k];
    }
    // points of the last block to points of the first: below 2q and 640q (narrow moduli), below w_half before and after (others)
    template <int W>
    __device__ __forceinline__ void inverse(u64 (&x)[4], u64* buf, const u64 (&w)[NB][6], u64 q, const ModConst& m) const {
        int bound = w_start(W);
#pragma unroll
        for (int i = NB - 1; i >= 0; i--) {
            if (i + 1 < NB) {
                if (i) wave_exchange();
                else __syncthreads();
                load(x, buf, i);
            }
            if ((W == 0 || W == W_NEAR) && LC == 9 && i == 0) {            // nine stages: the last two would leave the range
#pragma unroll
                for (int k = 0; k < 4; k++) x[k] = inv_end<W>(x[k], m);
                bound = 2;
            }
            if (2 * i + 1 >= LC) inv_block2_r<W, false, true>(x, w[i], q, bound);
            else if (i < 2) inv_block2_r<W, true>(x, w[i], q, bound);
            else inv_block2_r<W>(x, w[i], q, bound);
            if (i) store(buf, x, i);
        }
    }
    // points of the first block below 5q to points of the last
    template <int W>
    __device__ __forceinline__ void forward(u64 (&x)[4], u64* buf, const u64 (&w)[NB][6], u64 q) const {
        int b = 5;
#pragma unroll
        for (int i = 0; i < NB; i++) {
            if (i) {
                if (i > 1) wave_exchange();
                else __syncthreads();
                load(x, buf, i);
            }
            if (2 * i + 1 >= LC) fwd_block2_r<W, false, true>(x, w[i], q, b);
            else if (i < 2) fwd_block2_r<W, true>(x, w[i], q, b);
            else fwd_block2_r<W>(x, w[i], q, b);
            if (i + 1 < NB) store(buf, x, i);
        }
    }
};

// A work group takes a tile of one dropped limb through `share` moduli; the coefficients stay in registers.  Two buffers in
// turn, so that one barrier a transform is enough: whoever writes a buffer again has passed the barrier of the transform between,
// which every wavefront reaches after its last access to that buffer.
template <int LC>
__global__ __launch_bounds__(RS_THREADS, 4) void rescale_cols_kernel(RescaleCols rc, const ModConst* mc, const ulonglong2* ftw, const ulonglong2* itw) {
    ieee_off();
    using G = RsTile<LC>;
    constexpr uint32_t TPX = 1u << (LC - 5);             // tiles of a limb per XCD
    __shared__ u64 lds[2 * RS_LDS];
    G g{(uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63u};
    const uint32_t slot = blockIdx.x >> 3, tile = (blockIdx.x & 7u) * TPX + slot % TPX, gp = slot / TPX, limb = gp / rc.parts;
    const uint32_t c0 = tile << G::LCOLS, r0 = (gp - limb * rc.parts) * rc.share, r1 = min(rc.level, r0 + rc.share);
    const u64* src = rc.src + ((size_t)limb << (LC + 8));
    u64 x[4], w[G::NB][6];
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = src[G::at(g.point(G::NB - 1, k), c0)];
    g.factors(w, itw + ((size_t)rc.level << (LC + 8)));
    const ModConst ml = mod_const(mc, rc.level);
    const u64 h = ml.q >> 1;
    by_class(rc.inv, rc.level, 0, [&](auto W, uint32_t) {
        g.template inverse<W>(x, lds + RS_LDS, w, ml.q, ml);
        if (W == W_NEAR) {                               // positive, as the product below takes them
#pragma unroll
            for (int k = 0; k < 4; k++) x[k] += ml.q << 9;
        }
    });
    g.factors(w, ftw + ((size_t)r0 << (LC + 8)));
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = csub_min(csub_min(shoup_lazy(x[k], ml.ninv, ml.ninv_sh, ml.q), ml.q) + h, ml.q);
#pragma unroll 1
    for (uint32_t r = r0;;) {
        asm("" : "+v"(g.t));                             // what follows from the lane is worked out anew, not kept in registers
        const ModConst m = mod_const(mc, r);
        const u64 q = m.q;
        u64 y[4], *buf = lds + ((r - r0) & 1u) * RS_LDS;
        // Below 5q as they are where the dropped prime is at most 4q, that is for primes of one width: no quotient of four values (thirteen
        // instructions each, some 40 of a transform's 400).  A product and its rescale at level 11 of N = 2^16 116.8 -> 115.1 us.
        if (ml.q <= 4 * q) {
            const u64 up = 2 * q - (h < q ? h + q : h);  // h is below 2q
#pragma unroll
            for (int k = 0; k < 4; k++) y[k] = x[k] + up;
        } else {
            const u64 one_sh = m.one_sh, up = uni64(q - barrett64(h, q, m.mu, m.bits));
#pragma unroll
            for (int k = 0; k < 4; k++) y[k] = shoup_lazy4(x[k], 1, one_sh, q) + up;      // below 5q
        }
        by_class(rc.fwd, r, 0, [&](auto W, uint32_t) {
            fwd_centre<W>(y, m);
            g.template forward<W>(y, buf, w, q);
        });
        u64* dst = rc.dst + ((size_t)(limb * rc.level + r) << (LC + 8));
        if (++r < r1) g.factors(w, ftw + ((size_t)r << (LC + 8)));
#pragma unroll
        for (int k = 0; k < 4; k++) dst[G::at(g.point(G::NB - 1, k), c0)] = y[k];
        if (r >= r1) return;
    }
}

// Where the two column passes are one launch: while they are short enough that the launch saved counts more than the order of the
// writes.  A tile's points are runs of 32 bytes that go to every modulus in turn, where the separate passes (ntt2p.hip) write runs
// of 128 bytes, modulus after modulus.  Product and rescale at level 2 of N = 2^13 48.9 us with separate passes, 43.7 with one; at
// level 11 of 2^16 (1408 by this measure) 122.0 and 117.4, at level 12 of 2^17 (3072) 266.4 and 264.0; a block of layers (up to 6144)
// 1191 and 1176; eight outputs at level 8 of 2^16 (8192) 749.6 and 749 to 753, at level 16 (16384) the same, at level 23 (23552)
// 2301 and 2310.
bool rescale_cols_pays(const he_ctx* ctx, uint32_t n, uint32_t level) { return (uint64_t)n * level * (ctx->N >> 10) < 8192; }
int32_t launch_rescale_cols(he_ctx* ctx, const u64* src, u64* dst, uint32_t n, uint32_t level) {
    if (n == 0) return HE_OK;
    if (ctx->logN < 13 || ctx->logN > 17 || level == 0 || level >= ctx->nq) return he_fail(ctx, HE_ERR_BADARG, "rescale columns: bad shape");
    RescaleCols rc = {src, dst, level, 0, 0, ctx->cls_fwd, ctx->cls_inv};
    // The moduli of a tile are shared out, each share with the inverse columns of its own, while that makes at most three work groups
    // per compute unit: a rescale after a product at level 11 of N = 2^16 117.4 us with up to 768 or 1024, 120.4 with 2048, 123.6 with
    // 256 (a build with more registers); at level 23 206.6, 206.8, 208.8 and 225.
    const uint32_t groups = n * (ctx->N >> 10), parts = std::min(level, std::max(1u, 768 / groups));
    rc.share = (level + parts - 1) / parts;
    rc.parts = (level + rc.share - 1) / rc.share;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventCreate(&e0));
        HE_HIP(ctx, hipEventCreate(&e1));
        HE_HIP(ctx, hipEventRecord(e0, ctx->stream));
    }
    const dim3 grid(groups * rc.parts), block(RS_THREADS);
    switch (ctx->logN - 8) {
    case 5: hipLaunchKernelGGL(rescale_cols_kernel<5>, grid, block, 0, ctx->stream, rc, ctx->d_mc, ctx->d_tw, ctx->d_itw); break;
    case 6: hipLaunchKernelGGL(rescale_cols_kernel<6>, grid, block, 0, ctx->stream, rc, ctx->d_mc, ctx->d_tw, ctx->d_itw); break;
    case 7: hipLaunchKernelGGL(rescale_cols_kernel<7>, grid, block, 0, ctx->stream, rc, ctx->d_mc, ctx->d_tw, ctx->d_itw); break;
    case 8: hipLaunchKernelGGL(rescale_cols_kernel<8>, grid, block, 0, ctx->stream, rc, ctx->d_mc, ctx->d_tw, ctx->d_itw); break;
    default: hipLaunchKernelGGL(rescale_cols_kernel<9>, grid, block, 0, ctx->stream, rc, ctx->d_mc, ctx->d_tw, ctx->d_itw); break;
    }
    HE_HIP(ctx, hipGetLastError());
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventRecord(e1, ctx->stream));
        ctx->prof_events.push_back({e0, e1, n * (1 + level), 0u, 0u});
    }
    return HE_OK;
}
