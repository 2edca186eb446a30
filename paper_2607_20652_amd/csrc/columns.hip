// Decode through parent columns (columns.hpp) for gfx950.
#include "columns.hpp"

namespace dpb {
namespace {

template <int CPT, int NG, bool OUT_BF16>
__global__ __launch_bounds__(kColThreads, col_decode_waves(CPT)) void col_decode_kernel(ColPlan C, const int32_t* __restrict__ idx,
                                                                    const float* __restrict__ coef, int64_t T,
                                                                    void* __restrict__ y)
{
    constexpr int TPW = col_tpw(CPT);
    extern __shared__ __align__(16) unsigned char smem[];
    col_load_shared(C, smem);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    ColWave W = col_wave(C, smem, CPT, 0, wave, lane);
    const int nslots = TPW * C.k;
    const int64_t ngroups = (T + TPW - 1) / TPW, gstride = (int64_t)gridDim.x * kColWaves;
    // the next group's code is requested while this group is decoded
    const bool pf = nslots <= 64 * CodeFetch::kWords;
    CodeFetch N;
    auto live_slots = [&](int64_t grp) { return (int)min((int64_t)TPW, T - grp * TPW) * C.k; };
    auto fetch = [&](int64_t grp) {
        const int n = live_slots(grp);
        const int32_t* pi = idx + grp * nslots;
        const float* pc = coef + grp * nslots;
#pragma unroll
        for (int e = 0; e < CodeFetch::kWords; ++e) {
            const int i = e * 64 + lane;
            N.i[e] = i < n ? pi[i] : -1;
            N.c[e] = i < n ? pc[i] : 0.f;
        }
    };
    int64_t grp = (int64_t)blockIdx.x * kColWaves + wave;
    if (pf && grp < ngroups) fetch(grp);
    for (; grp < ngroups; grp += gstride) {
        W.ntok = (int)min((int64_t)TPW, T - grp * TPW);
        // values derived from the lane index are recomputed for each group:
        // hoisted out of this loop they would take the registers of a wave
        W.lane = lane;
        __asm__ volatile("" : "+v"(W.lane));
        if (pf) {
#pragma unroll
            for (int e = 0; e < CodeFetch::kWords; ++e) {
                const int i = e * 64 + lane;
                if (i < nslots) {
                    W.idx[i] = N.i[e];
                    W.coef[i] = N.c[e];
                }
            }
            if (grp + gstride < ngroups) fetch(grp + gstride);
        } else {
            const int n = live_slots(grp);
            for (int i = lane; i < nslots; i += 64) {
                W.idx[i] = i < n ? idx[grp * nslots + i] : -1;
                W.coef[i] = i < n ? coef[grp * nslots + i] : 0.f;
            }
        }
        wave_sync();
        col_parents<CPT>(C, W);
        col_alpha<CPT>(C, W, W.coef, [&](int tt, int s) {
            const int32_t c = W.idx[tt * C.k + s];
            return c >= C.d ? col_route<CPT>(C, W, tt, (uint32_t)c) : -1;
        });
        col_decode<CPT, NG, OUT_BF16>(C, W, W.coef, grp * TPW, y, nullptr);
    }
}

}  // namespace

template <int CPT, int NG, bool OB>
static void launch_col_v(const ColPlan& C, size_t lds, hipStream_t stream, const int32_t* idx, const float* coef,
                         int64_t T, void* y)
{
    allow_lds(col_decode_kernel<CPT, NG, OB>, lds);
    hipLaunchKernelGGL((col_decode_kernel<CPT, NG, OB>), col_grid(T, col_tpw(CPT), lds, col_decode_waves(CPT), 1), dim3(kColThreads), lds,
                       stream, C, idx, coef, T, y);
}

template <int CPT, bool OB>
static void launch_col_ng(int ng, const ColPlan& C, size_t lds, hipStream_t stream, const int32_t* idx,
                          const float* coef, int64_t T, void* y)
{
    switch (ng) {
    case 3: launch_col_v<CPT, 3, OB>(C, lds, stream, idx, coef, T, y); break;
    case 4: launch_col_v<CPT, 4, OB>(C, lds, stream, idx, coef, T, y); break;
    case 5: launch_col_v<CPT, 5, OB>(C, lds, stream, idx, coef, T, y); break;
    case 6: launch_col_v<CPT, 6, OB>(C, lds, stream, idx, coef, T, y); break;
    default: launch_col_v<CPT, 8, OB>(C, lds, stream, idx, coef, T, y); break;
    }
}

// The column decode of the plan, if it takes it (false: nothing launched).
template <bool OB>
static bool launch_col(const DevPlan& P, const int32_t* idx, const float* coef, int64_t T, void* y, hipStream_t stream)
{
    auto lds_bytes = [&](int cpt) {
        const ColPlan C = col_plan(P, cpt);
        return col_shared_bytes(C) + (size_t)kColWaves * col_layout(C, cpt, 0).bytes;
    };
    const int cpt = col_choose(P, lds_bytes);
    if (cpt < 0) return false;
    const ColPlan C = col_plan(P, cpt);
    const size_t lds = lds_bytes(cpt);
    if (lds > (size_t)kLdsBudget) return false;
    const int ng = ng_variant(P);
    if (cpt == 0) launch_col_ng<0, OB>(ng, C, lds, stream, idx, coef, T, y);
    else if (cpt == 4) launch_col_ng<4, OB>(ng, C, lds, stream, idx, coef, T, y);
    else if (cpt == 8) launch_col_ng<8, OB>(ng, C, lds, stream, idx, coef, T, y);
    else launch_col_ng<16, OB>(ng, C, lds, stream, idx, coef, T, y);
    return true;
}

bool launch_col_decode(const DevPlan& P, const int32_t* idx, const float* coef, int64_t T, void* y, bool y_bf16,
                       hipStream_t stream)
{
    return y_bf16 ? launch_col<true>(P, idx, coef, T, y, stream) : launch_col<false>(P, idx, coef, T, y, stream);
}

}  // namespace dpb
