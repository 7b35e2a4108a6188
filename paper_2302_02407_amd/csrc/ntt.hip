// Batched negacyclic NTT / iNTT over RNS limbs (ring Z_q[X]/(X^N+1), paper Section 2.1).
//
// Forward: decimation-in-time butterflies with the 2N-th root folded into the twiddles
// (natural-order coefficients in, bit-reversed evaluations out); inverse: the mirrored
// decimation-in-frequency network.  Butterflies keep residues lazily reduced (forward in
// [0,4q), inverse in [0,2q)) and multiply by twiddles with Shoup's precomputed quotients;
// only the last pass canonicalises.
//
// This file serves rings up to N = 2^12: the whole limb (at most 32 KiB) staged in LDS, one launch.  Larger rings take two
// launches (ntt2p.hip).
#include "modarith.h"

#define NTT_THREADS 1024
#define NTT_MAX_N 4096

struct NttArgs {
    u64* data;
    const ModConst* mc;
    const ulonglong2* tw;   // [M][N] forward or inverse table
    uint32_t logN;
};

// Where limb i is read: segment (limb[i] >> 12) at limb offset (limb[i] & 0xFFF); the result lands at data + i*N.
struct TileSrc {
    const u64* seg[HE_MAX_SEGS];
    uint16_t limb[HE_MAX_LAUNCH_LIMBS];
};

template <bool FWD, bool CUSTOM_SCALE>
__global__ __launch_bounds__(NTT_THREADS) void ntt_limb_kernel(NttArgs a, LimbList ll, ScaleList sc, uint32_t scale_period, TileSrc ts) {
    __shared__ u64 sm[NTT_MAX_N];
    const uint32_t limb = blockIdx.x, N = 1u << a.logN;
    const uint32_t mi = ll.mod[limb];
    if (mi == 0xFFu) return; // limb marked "leave untouched" (uniform for the whole workgroup)
    const ModConst m = a.mc[mi];
    const u64 q = m.q, q2 = m.q2;
    u64* base = a.data + (size_t)limb * N;
    const ulonglong2* tw = a.tw + (size_t)mi * N;
    const uint32_t sl = ts.limb[limb];
    const u64* in = ts.seg[sl >> 12] + (size_t)(sl & 0xFFFu) * N;
    for (uint32_t e = threadIdx.x; e < N; e += NTT_THREADS) sm[e] = in[e];
    __syncthreads();
    const uint32_t half = N >> 1;
    for (uint32_t i = 0; i < a.logN; i++) {
        const uint32_t s = FWD ? i : a.logN - 1 - i, log_t = a.logN - 1 - s, t = 1u << log_t;
        for (uint32_t b = threadIdx.x; b < half; b += NTT_THREADS) {
            const uint32_t g = b >> log_t, e0 = (g << (log_t + 1)) + (b & (t - 1)), e1 = e0 + t;
            const ulonglong2 w = tw[(1u << s) + g];
            const u64 x = sm[e0], y = sm[e1];
            if (FWD) {
                const u64 u = csub(x, q2), v = shoup_lazy(y, w.x, w.y, q);
                sm[e0] = u + v;
                sm[e1] = u - v + q2;
            } else {
                sm[e0] = csub(x + y, q2);
                sm[e1] = shoup_lazy(x - y + q2, w.x, w.y, q);
            }
        }
        __syncthreads();
    }
    const u64 scale = CUSTOM_SCALE ? sc.s[limb % scale_period] : m.ninv, scale_sh = CUSTOM_SCALE ? sc.s_sh[limb % scale_period] : m.ninv_sh;
    for (uint32_t e = threadIdx.x; e < N; e += NTT_THREADS) {
        const u64 v = sm[e];
        base[e] = FWD ? csub(csub(v, q2), q) : csub(shoup_lazy(v, scale, scale_sh, q), q);
    }
}

template <bool FWD>
static int32_t run_transform(he_ctx* ctx, u64* d, const uint32_t* mod_idx, uint32_t n, const ScaleList* scale, uint32_t scale_period,
                             const TileSrc& ts) {
    LimbList ll;
    uint32_t live = 0;
    for (uint32_t i = 0; i < n; i++) {
        if (mod_idx[i] == 0xFFu) { ll.mod[i] = 0xFF; continue; } // internal marker: skip this limb
        if (mod_idx[i] >= ctx->M) return he_fail(ctx, HE_ERR_BADARG, "transform: modulus index %u out of range", mod_idx[i]);
        ll.mod[i] = (uint8_t)mod_idx[i];
        live++;
    }
    ScaleList sc;
    if (scale) sc = *scale;
    const NttArgs a = {d, ctx->d_mc, FWD ? ctx->d_tw : ctx->d_itw, ctx->logN};
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventCreate(&e0));
        HE_HIP(ctx, hipEventCreate(&e1));
        HE_HIP(ctx, hipEventRecord(e0, ctx->stream));
    }
    if (scale) hipLaunchKernelGGL((ntt_limb_kernel<FWD, true>), dim3(n), dim3(NTT_THREADS), 0, ctx->stream, a, ll, sc, scale_period ? scale_period : 1u, ts);
    else hipLaunchKernelGGL((ntt_limb_kernel<FWD, false>), dim3(n), dim3(NTT_THREADS), 0, ctx->stream, a, ll, sc, 1u, ts);
    HE_HIP(ctx, hipGetLastError());
    if (ctx->prof_on) {
        HE_HIP(ctx, hipEventRecord(e1, ctx->stream));
        ctx->prof_events.push_back({e0, e1, live, 0u, FWD ? 1u : 3u});
    }
    if (FWD) ctx->cnt.ntt_limbs += live; else ctx->cnt.intt_limbs += live;
    return HE_OK;
}

// Small rings: the ModDown epilogue runs as its own kernel.
static int32_t launch_transform_generic(he_ctx* ctx, const TransformDesc& d) {
    if (d.rescale_from) return he_fail(ctx, HE_ERR_BADARG, "transform: the Rescale rounding term is only read by two-launch transforms");
    TileSrc ts;
    for (uint32_t s = 0; s < HE_MAX_SEGS; s++) ts.seg[s] = s < d.n_seg ? d.seg[s] : d.seg[0];
    for (uint32_t i = 0; i < d.n; i++) {
        uint32_t seg = d.src_seg ? d.src_seg[i] : 0, lim = d.src_limb ? d.src_limb[i] : i;
        if (seg >= HE_MAX_SEGS || seg >= d.n_seg || lim >= 4096) return he_fail(ctx, HE_ERR_BADARG, "transform: source limb out of range");
        ts.limb[i] = (uint16_t)((seg << 12) | lim);
    }
    int32_t rc = d.fwd ? run_transform<true>(ctx, d.dst, d.mod_idx, d.n, nullptr, 1, ts)
                       : run_transform<false>(ctx, d.dst, d.mod_idx, d.n, d.scale, d.scale_period, ts);
    if (rc != HE_OK) return rc;
    if (d.fwd && d.ep) return launch_moddown_final(ctx, d.dst, d.n / (2 * d.ep->L1), *d.ep);
    return HE_OK;
}

int32_t launch_transform(he_ctx* ctx, const TransformDesc& d) {
    if (d.n == 0) return HE_OK;
    if (d.n > HE_MAX_LAUNCH_LIMBS) return he_fail(ctx, HE_ERR_BADARG, "transform: too many limbs in one launch");
    if (d.scale && (d.scale_period == 0 || d.scale_period > HE_MAX_MODULI)) return he_fail(ctx, HE_ERR_BADARG, "transform: bad scale period");
    return two_pass(ctx) ? launch_transform2p(ctx, d) : launch_transform_generic(ctx, d);
}

int32_t launch_ntt(he_ctx* ctx, u64* d, const uint32_t* mod_idx, uint32_t n) {
    TransformDesc t = {};
    t.fwd = true; t.seg[0] = d; t.n_seg = 1; t.dst = d; t.n = n; t.mod_idx = mod_idx;
    return launch_transform(ctx, t);
}
int32_t launch_intt(he_ctx* ctx, u64* d, const uint32_t* mod_idx, uint32_t n, const ScaleList* scale) {
    TransformDesc t = {};
    t.fwd = false; t.seg[0] = d; t.n_seg = 1; t.dst = d; t.n = n; t.mod_idx = mod_idx;
    t.scale = scale; t.scale_period = scale ? n : 0;
    return launch_transform(ctx, t);
}

extern "C" {

int32_t he_ntt(he_ctx* ctx, uint64_t* d_data, const uint32_t* h_mod_idx, uint32_t n_limbs) {
    return he_guard(ctx, "he_ntt: host allocation failed", [&]() -> int32_t {
    if (!ctx) return HE_ERR_BADARG;
    if (n_limbs == 0) return HE_OK;
    if (!d_data || !h_mod_idx) return he_fail(ctx, HE_ERR_BADARG, "he_ntt: null argument");
    for (uint32_t i = 0; i < n_limbs; i++)
        if (h_mod_idx[i] >= ctx->M) return he_fail(ctx, HE_ERR_BADARG, "he_ntt: modulus index %u out of range", h_mod_idx[i]);
    for (uint32_t o = 0; o < n_limbs; o += HE_MAX_LAUNCH_LIMBS) {
        uint32_t n = n_limbs - o < HE_MAX_LAUNCH_LIMBS ? n_limbs - o : HE_MAX_LAUNCH_LIMBS;
        int32_t rc = launch_ntt(ctx, (u64*)d_data + (size_t)o * ctx->N, h_mod_idx + o, n);
        if (rc != HE_OK) return rc;
    }
    return HE_OK;
    });
}

int32_t he_intt(he_ctx* ctx, uint64_t* d_data, const uint32_t* h_mod_idx, uint32_t n_limbs) {
    return he_guard(ctx, "he_intt: host allocation failed", [&]() -> int32_t {
    if (!ctx) return HE_ERR_BADARG;
    if (n_limbs == 0) return HE_OK;
    if (!d_data || !h_mod_idx) return he_fail(ctx, HE_ERR_BADARG, "he_intt: null argument");
    for (uint32_t i = 0; i < n_limbs; i++)
        if (h_mod_idx[i] >= ctx->M) return he_fail(ctx, HE_ERR_BADARG, "he_intt: modulus index %u out of range", h_mod_idx[i]);
    for (uint32_t o = 0; o < n_limbs; o += HE_MAX_LAUNCH_LIMBS) {
        uint32_t n = n_limbs - o < HE_MAX_LAUNCH_LIMBS ? n_limbs - o : HE_MAX_LAUNCH_LIMBS;
        int32_t rc = launch_intt(ctx, (u64*)d_data + (size_t)o * ctx->N, h_mod_idx + o, n, nullptr);
        if (rc != HE_OK) return rc;
    }
    return HE_OK;
    });
}

} // extern "C"
