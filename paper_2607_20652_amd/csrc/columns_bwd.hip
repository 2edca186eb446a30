// Decode-backward of codes of at most 254 slots (columns.hpp), for gfx950.
#include "columns.hpp"

namespace dpb {
namespace {

// Gradient rows of a column-backward wave, their column bitmaps and score
// tile: the bytes of the region that the decode reuses.
__host__ __device__ inline unsigned col_act_rows(const DevPlan& P, bool g_bf16)
{
    return align16u((unsigned)P.wave_tokens * (g_bf16 ? P.prow : P.dp) * 4u);
}
// The score tile (and the direct reductions' list) of a plan without leaf
// columns shares the bitmaps' space: it has no scores, and lists after them.
__host__ __device__ inline unsigned col_act_bitmaps(const DevPlan& P, int cpt)
{
    const unsigned b = align16u(16u * P.cws * 4u);
    return cpt ? b : b > 1024u ? b : 1024u;
}
__host__ __device__ inline unsigned col_act_bytes(const DevPlan& P, int cpt, bool g_bf16)
{
    return col_act_rows(P, g_bf16) + col_act_bitmaps(P, cpt) + (cpt ? 1024u : 0u);
}

// The smallest fp32 magnitude (bits) that rounds to an infinite bf16.
constexpr uint32_t kBf16Inf = 0x7F7F8000u;

// Unscaled sums of one block of sixteen columns phi~_p (.) g against the
// level's sixteen generators (LEAF: `s`, the child scores, lane rows 4 kq ..)
// and against ones (`o`, the column's own <phi~_p, g>, the same in every row).
// Building the columns is the cost (8 vector instructions per 32 coordinates
// of sixteen columns); the second product rides on them.
template <bool G_BF16, bool LEAF>
__device__ __forceinline__ void column_products(const DevPlan& P, const Wave& S, int trow, f32x4& s, f32x4& o)
{
    constexpr int SB = 6;   // fragments requested together
    const int lane = S.lane, kq = lane >> 4, nchunk = P.nchunk, l = P.levels - 1;
    const u32x4* Ap = (const u32x4*)P.gamma_pair + P.gamma_off[l] + lane;
    const uint32_t* cwp = S.cw + (lane & 15) * P.cws;
    const uint32_t* prow = S.pairs + trow * P.prow + kq * 4;
    const float* frow = S.gf + trow * P.dp;
    const u32x4 one = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    s = o = f32x4{0.f, 0.f, 0.f, 0.f};
    int c0 = 0;
    for (; c0 + SB <= nchunk; c0 += SB) {
        u32x4 a[SB];
        uint32_t wd[SB];
#pragma unroll
        for (int e = 0; e < SB; ++e) {
            if constexpr (LEAF) a[e] = Ap[(int64_t)(c0 + e) * 64];
            wd[e] = cwp[c0 + e];
        }
#pragma unroll
        for (int e = 0; e < SB; ++e) score_chunk2<G_BF16, LEAF, true>(kq, a[e], one, wd[e], prow, frow, c0 + e, s, o);
    }
    for (; c0 < nchunk; ++c0) {
        u32x4 a = one;
        if constexpr (LEAF) a = Ap[(int64_t)c0 * 64];
        score_chunk2<G_BF16, LEAF, true>(kq, a, one, cwp[c0], prow, frow, c0, s, o);
    }
}

// grad_coef of the leaf slots (child scores of their parent's column), the
// leaf parents and, with bf16 gradients, the summed slots, each from columns
// on the matrix cores: 0.5 vector instructions per slot and chunk against 1
// in direct_scores.  (fp32 gradients: the exact split costs more than the
// direct reductions, so the summed slots are left to those.)  Measured, us:
// 65,536 tokens d 768 k 96 304 -> 299, 8,192 tokens d 768 k 56 37 -> 35,
// 16,381 tokens d 1024 k 144 191 -> 187, 20,000 tokens d 200 k 16 31 -> 27,
// 8,192 tokens d 768 k 56 in fp32 85 -> 74.  An fp32 gradient whose high
// term is infinite has no such split (inf - inf in the second term): the
// parents of a token that holds one are reduced directly, which gives the
// signed infinity, or the finite sum of a value beyond the largest bf16.
template <int CPT, bool G_BF16>
__device__ __forceinline__ void col_scores(const ColPlan& C, const DevPlan& P, const Wave& S)
{
    constexpr int TPW = col_tpw(CPT);
    const int lane = S.lane, col = lane & 15, kq = lane >> 4, k = C.k;
    f32x4 s, o;
    if constexpr (CPT > 0) {   // the leaf parents: column tt CPT + q
        const int tt = col / CPT, q = col & (CPT - 1);
        const int32_t p = q < C.KP ? S.idx[tt * k + C.sbP + q] : -1;
        if (!G_BF16 || __ballot(p >= 0)) {   // no parent: no leaf has a route (fp32 measured slower with the branch)
            index_bitmaps(P, lane, p, P.nt, S.cw);
            wave_sync();
            column_products<G_BF16, true>(P, S, tt, s, o);
#pragma unroll
            for (int i = 0; i < 4; ++i) S.score[col * 16 + kq * 4 + i] = s[i] * C.rsd;
            if (kq == 0 && p >= C.d) S.coef[tt * k + C.sbP + q] = o[0] * C.rsd;
            wave_sync();
            for (int i = lane; i < TPW * C.KL; i += 64) {
                const int t2 = item_token<TPW>(i, C.KL), at = t2 * k + C.sbL + i - t2 * C.KL, rt = S.route[at];
                if (rt >= 0) S.coef[at] = S.score[(t2 * CPT + (rt >> 16)) * 16 + (rt & 0xFFFF)];
            }
        }
    }
    if constexpr (G_BF16) {
        for (int i0 = 0; i0 < TPW * C.ns; i0 += 16) {
            const int i = i0 + col, tt = min(item_token<TPW>(i, C.ns), TPW - 1);
            const int at = tt * k + C.ss + i - tt * C.ns;
            const int32_t c = i < TPW * C.ns ? S.idx[at] : -1;
            if (!__ballot(c >= C.d)) continue;   // basis slots and padding
            wave_sync();
            index_bitmaps(P, lane, c, P.nt, S.cw);
            wave_sync();
            column_products<G_BF16, false>(P, S, tt, s, o);
            if (kq == 0 && c >= C.d) S.coef[at] = o[0] * C.rsd;
        }
    }
    wave_sync();
}

// The backward over columns (P.wave_tokens = col_tpw(CPT)): grad_coef as in decode_bwd2_kernel, then the column decode of it.
template <int CPT, int NG, bool G_BF16, bool GX_BF16>
__global__ __launch_bounds__(kColThreads, col_bwd_waves(CPT, G_BF16)) void col_bwd_kernel(ColPlan C, DevPlan P, const int32_t* __restrict__ idx,
                                                                 const void* __restrict__ g, int64_t T,
                                                                 float* __restrict__ grad_coef, void* grad_x,
                                                                 const float* __restrict__ add_gc, const void* add_gx,
                                                                 const float2* __restrict__ stats)
{
    constexpr int TPW = col_tpw(CPT);
    extern __shared__ __align__(16) unsigned char smem[];
    col_load_shared(C, smem);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const unsigned act_bytes = col_act_bytes(P, CPT, G_BF16);
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
        S.score = (float*)(b + L.act + col_act_rows(P, G_BF16) + (CPT ? col_act_bitmaps(P, CPT) : 0u));
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
    // and so are its bf16 gradient rows for two and four tokens a wave, where
    // four pieces of 512 coordinates hold them (65,536 tokens d 768 285 -> 274
    // us, 20,000 tokens d 200 26.6 -> 23.2; one token a wave measured slower
    // with it: d 1024 N 2^24 183 -> 186, pt_large_2l 82 -> 103)
    constexpr bool kRows = G_BF16 && TPW > 1;
    constexpr int kPieces = 4, PPT = kPieces / TPW;
    const bool pfg = kRows && d <= 512 * PPT && (d & 7) == 0;
    u32x4 ng[kPieces];
    auto fetch_g = [&](int64_t gp) {
#pragma unroll
        for (int e = 0; e < kPieces; ++e) {
            const int o = (e % PPT) * 512 + lane * 8;
            const int64_t t = gp * TPW + e / PPT;
            ng[e] = (o < d && t < T) ? *(const u32x4*)((const uint16_t*)g + t * d + o) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    int64_t grp = (int64_t)blockIdx.x * kColWaves + wave;
    if (pf && grp < ngroups) fetch(grp);
    if (pfg && grp < ngroups) fetch_g(grp);
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
        } else {
            for (int i = ln; i < nslots; i += 64) W.idx[i] = i < n ? idx[grp * nslots + i] : -1;
        }
        uint32_t nosplit = 0;   // tokens with a gradient value that has no three-term split
        if (kRows && pfg) {
#pragma unroll
            for (int e = 0; e < kPieces; ++e) {
                const int o = (e % PPT) * 512 + ln * 8;
                if (o < dp) store_pair_piece(ln, ng[e], o, S.pairs + (e / PPT) * P.prow);
            }
        } else if constexpr (G_BF16) {
            load_pairs(P, ln, W.ntok, TPW, (const uint16_t*)g, t0, S.pairs);
        } else {
            const float* gfp = (const float*)g;
            for (int tt = 0; tt < TPW; ++tt) {
                uint32_t top = 0;
                for (int iota = ln; iota < dp; iota += 64) {
                    const float v = (tt < W.ntok && iota < d) ? gfp[(t0 + tt) * d + iota] : 0.f;
                    S.gf[tt * dp + iota] = v;
                    top = max(top, __float_as_uint(v) & 0x7FFFFFFFu);
                }
                nosplit |= (uint32_t)(__ballot(top >= kBf16Inf) != 0) << tt;
            }
        }
        wave_sync();
        col_parents<CPT>(C, W);
        wave_sync();
        // routes of the leaf slots; coefficients of basis slots (g at their
        // coordinate) and padding
        bool direct = false;
        for (int i = ln; i < nslots; i += 64) {
            const int tt = item_token<TPW>(i, C.k), s = i - tt * C.k;
            const int32_t c = W.idx[i];
            float v = 0.f;
            if (c >= 0 && c < d) v = g_at<G_BF16>(P, S, tt, c);
            W.coef[i] = v;
            int rt = -1;
            if (s >= C.sbL) rt = c >= d ? col_route<CPT>(C, W, tt, (uint32_t)c) : -1;
            else if ((s >= C.sbP || (G_BF16 && s >= C.ss)) && !((nosplit >> tt) & 1u)) rt = 0;   // a column of its own
            S.route[i] = rt;
            direct |= c >= d && rt < 0;
        }
        const uint64_t left = __ballot(direct);
        wave_sync();
        // grad_coef of hashed slots: leaf slots, their parents and the summed
        // slots as columns, whatever is left directly
        col_scores<CPT, G_BF16>(C, P, S);
        if (left) {
            direct_scores<G_BF16, NG>(P, S);
            wave_sync();
        }
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
        // requested here, after the scoring's table reads: memory waits are in
        // issue order, and the decode's set-up reads no memory
        if (grp + gstride < ngroups) {
            if (pf) fetch(grp + gstride);
            if (kRows && pfg) fetch_g(grp + gstride);
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
    hipLaunchKernelGGL((col_bwd_kernel<CPT, NG, GB, XB>), col_grid(T, col_tpw(CPT), lds, col_bwd_waves(CPT, GB), 1), dim3(kColThreads), lds,
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
    DevPlan P = Pp;
    auto lds_bytes = [&](int cpt) {
        P.wave_tokens = col_tpw(cpt);
        const ColPlan C = col_plan(P, cpt);
        return col_shared_bytes(C) + (size_t)kColWaves * col_layout(C, cpt, col_act_bytes(P, cpt, GB)).bytes;
    };
    const int cpt = col_choose(Pp, lds_bytes);
    if (cpt < 0) return false;
    const size_t lds = lds_bytes(cpt);   // leaves its tokens a wave in P
    const ColPlan C = col_plan(P, cpt);
    if (lds > (size_t)kLdsBudget) return false;
    const int ng = ng_variant(P);
    if (cpt == 0) launch_colb_ng<0, GB, XB>(ng, C, P, lds, stream, idx, g, T, gc, gx, ex);
    else if (cpt == 4) launch_colb_ng<4, GB, XB>(ng, C, P, lds, stream, idx, g, T, gc, gx, ex);
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
