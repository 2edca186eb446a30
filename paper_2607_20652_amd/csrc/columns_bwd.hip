// Decode-backward of plans that decode through parent columns, for gfx950.
#include "columns.hpp"

namespace dpb {
namespace {

// Gradient rows of a column-backward wave, their column bitmaps and score
// tile: the bytes of the region that the decode reuses.
__host__ __device__ inline unsigned col_act_rows(const DevPlan& P, bool g_bf16)
{
    return align16u((unsigned)P.wave_tokens * (g_bf16 ? P.prow : P.dp) * 4u);
}
__host__ __device__ inline unsigned col_act_bytes(const DevPlan& P, bool g_bf16)
{
    return col_act_rows(P, g_bf16) + align16u(16u * P.cws * 4u) + 16u * 16u * 4u;
}

// The backward of plans that decode through parent columns (P.wave_tokens =
// 16 / CPT): grad_coef as in decode_bwd2_kernel, then the column decode of it.
template <int CPT, int NG, bool G_BF16, bool GX_BF16>
__global__ __launch_bounds__(kColThreads, 4) void col_bwd_kernel(ColPlan C, DevPlan P, const int32_t* __restrict__ idx,
                                                                 const void* __restrict__ g, int64_t T,
                                                                 float* __restrict__ grad_coef, void* grad_x,
                                                                 const float* __restrict__ add_gc, const void* add_gx,
                                                                 const float2* __restrict__ stats)
{
    constexpr int TPW = col_tpw(CPT);
    extern __shared__ __align__(16) unsigned char smem[];
    col_load_shared(C, smem);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const unsigned act_bytes = col_act_bytes(P, G_BF16);
    ColWave W = col_wave(C, smem, CPT, act_bytes, wave, lane);
    Wave S{};
    {
        const ColLayout L = col_layout(C, CPT, act_bytes);
        unsigned char* b = smem + col_shared_bytes(C) + (unsigned)wave * L.bytes;
        S.idx = W.idx;
        S.coef = W.coef;
        S.route = (int32_t*)(b + L.route);
        S.pairs = (uint32_t*)(b + L.act);
        S.gf = (float*)(b + L.act);
        S.cw = (uint32_t*)(b + L.act + col_act_rows(P, G_BF16));
        S.score = (float*)(b + L.act + col_act_rows(P, G_BF16) + align16u(16u * P.cws * 4u));
    }
    const int nslots = TPW * C.k, d = C.d, dp = C.dp;
    const int64_t ngroups = (T + TPW - 1) / TPW, gstride = (int64_t)gridDim.x * kColWaves;
    // the next group's indices are requested while this group is processed
    const bool pf = nslots <= 64 * CodeFetch::kWords;
    int32_t nidx[CodeFetch::kWords];
    auto live_slots = [&](int64_t grp) { return (int)min((int64_t)TPW, T - grp * TPW) * C.k; };
    auto fetch = [&](int64_t grp) {
        const int n = live_slots(grp);
        const int32_t* pi = idx + grp * nslots;
#pragma unroll
        for (int e = 0; e < CodeFetch::kWords; ++e) {
            const int i = e * 64 + lane;
            nidx[e] = i < n ? pi[i] : -1;
        }
    };
    int64_t grp = (int64_t)blockIdx.x * kColWaves + wave;
    if (pf && grp < ngroups) fetch(grp);
    for (; grp < ngroups; grp += gstride) {
        const int64_t t0 = grp * TPW;
        W.ntok = S.ntok = (int)min((int64_t)TPW, T - t0);
        // values derived from the lane index are recomputed for each group:
        // hoisted out of this loop they would take the registers of a wave
        W.lane = lane;
        __asm__ volatile("" : "+v"(W.lane));
        const int ln = S.lane = W.lane;
        const int n = live_slots(grp);
        if (pf) {
#pragma unroll
            for (int e = 0; e < CodeFetch::kWords; ++e) {
                const int i = e * 64 + ln;
                if (i < nslots) W.idx[i] = nidx[e];
            }
            if (grp + gstride < ngroups) fetch(grp + gstride);
        } else {
            for (int i = ln; i < nslots; i += 64) W.idx[i] = i < n ? idx[grp * nslots + i] : -1;
        }
        if constexpr (G_BF16) {
            load_pairs(P, ln, W.ntok, TPW, (const uint16_t*)g, t0, S.pairs);
        } else {
            const float* gfp = (const float*)g;
            for (int tt = 0; tt < TPW; ++tt)
                for (int iota = ln; iota < dp; iota += 64)
                    S.gf[tt * dp + iota] = (tt < W.ntok && iota < d) ? gfp[(t0 + tt) * d + iota] : 0.f;
        }
        wave_sync();
        col_parents<CPT>(C, W);
        wave_sync();
        // routes of the leaf slots; coefficients of basis slots (g at their
        // coordinate) and padding
        for (int i = ln; i < nslots; i += 64) {
            const int tt = item_token<TPW>(i, C.k), s = i - tt * C.k;
            const int32_t c = W.idx[i];
            float v = 0.f;
            if (c >= 0 && c < d) v = g_at<G_BF16>(P, S, tt, c);
            W.coef[i] = v;
            S.route[i] = s >= C.sbL && c >= d ? col_route<CPT>(C, W, tt, (uint32_t)c) : -1;
        }
        wave_sync();
        // grad_coef of routed slots: child scores of each parent column
        // against g; every other hashed slot directly
        score_level<G_BF16>(P, S, P.levels - 1);
        direct_scores<G_BF16, NG>(P, S);
        wave_sync();
        if (add_gc) {
            for (int i = ln; i < n; i += 64) W.coef[i] += add_gc[t0 * C.k + i];
            wave_sync();
        }
        for (int i = ln; i < n; i += 64) grad_coef[t0 * C.k + i] = W.coef[i];
        if (stats) {
            // standardized coefficients z = (s - mu) r: dz/dx = r phi
            wave_sync();
            const int32_t nfeat_sh = P.level_bits[P.levels - 1];
            for (int i = ln; i < n; i += 64) {
                const int32_t c = W.idx[i];
                if (c >= 0 && (c >> nfeat_sh) == 0) W.coef[i] *= stats[c].y;
            }
            wave_sync();
        }
        // grad_x = decode(idx, grad_coef) (+ add_gx); the scoring buffers are dead now
        col_alpha<CPT>(C, W, W.coef, [&](int tt, int s) { return S.route[tt * C.k + s]; });
        col_decode<CPT, NG, GX_BF16>(C, W, W.coef, t0, grad_x, add_gx);
    }
}

}  // namespace

template <int CPT, int NG, bool GB, bool XB>
static void launch_colb_v(const ColPlan& C, const DevPlan& P, size_t lds, hipStream_t stream, const int32_t* idx,
                          const void* g, int64_t T, float* gc, void* gx, BwdExtra ex)
{
    allow_lds(col_bwd_kernel<CPT, NG, GB, XB>, lds);
    hipLaunchKernelGGL((col_bwd_kernel<CPT, NG, GB, XB>), col_grid(T, col_tpw(CPT), lds, 4, 1), dim3(kColThreads), lds,
                       stream, C, P, idx, g, T, gc, gx, ex.gc, ex.gx, ex.stats);
}

template <int CPT, bool GB, bool XB>
static void launch_colb_ng(int ng, const ColPlan& C, const DevPlan& P, size_t lds, hipStream_t stream,
                           const int32_t* idx, const void* g, int64_t T, float* gc, void* gx, BwdExtra ex)
{
    switch (ng) {
    case 3: launch_colb_v<CPT, 3, GB, XB>(C, P, lds, stream, idx, g, T, gc, gx, ex); break;
    case 4: launch_colb_v<CPT, 4, GB, XB>(C, P, lds, stream, idx, g, T, gc, gx, ex); break;
    case 5: launch_colb_v<CPT, 5, GB, XB>(C, P, lds, stream, idx, g, T, gc, gx, ex); break;
    case 6: launch_colb_v<CPT, 6, GB, XB>(C, P, lds, stream, idx, g, T, gc, gx, ex); break;
    default: launch_colb_v<CPT, 8, GB, XB>(C, P, lds, stream, idx, g, T, gc, gx, ex); break;
    }
}

// The column backward of the plan, if it takes it (false: nothing launched).
template <bool GB, bool XB>
static bool launch_colb(const DevPlan& Pp, const int32_t* idx, const void* g, int64_t T, float* gc, void* gx,
                           BwdExtra ex, hipStream_t stream)
{
    const int cpt = col_cpt(Pp);
    if (!cpt) return false;
    DevPlan P = Pp;
    P.wave_tokens = col_tpw(cpt);
    const ColPlan C = col_plan(P, cpt);
    const size_t lds =
        col_shared_bytes(C) + (size_t)kColWaves * col_layout(C, cpt, col_act_bytes(P, GB)).bytes;
    if (lds > (size_t)kLdsBudget) return false;
    const int ng = ng_variant(P);
    if (cpt == 4) launch_colb_ng<4, GB, XB>(ng, C, P, lds, stream, idx, g, T, gc, gx, ex);
    else if (cpt == 8) launch_colb_ng<8, GB, XB>(ng, C, P, lds, stream, idx, g, T, gc, gx, ex);
    else launch_colb_ng<16, GB, XB>(ng, C, P, lds, stream, idx, g, T, gc, gx, ex);
    return true;
}

bool launch_col_bwd(const DevPlan& P, const int32_t* idx, const void* g, bool g_bf16, int64_t T, float* grad_coef,
                    void* grad_x, bool gx_bf16, BwdExtra ex, hipStream_t stream)
{
    if (g_bf16)
        return gx_bf16 ? launch_colb<true, true>(P, idx, g, T, grad_coef, grad_x, ex, stream)
                       : launch_colb<true, false>(P, idx, g, T, grad_coef, grad_x, ex, stream);
    return gx_bf16 ? launch_colb<false, true>(P, idx, g, T, grad_coef, grad_x, ex, stream)
                   : launch_colb<false, false>(P, idx, g, T, grad_coef, grad_x, ex, stream);
}

}  // namespace dpb
