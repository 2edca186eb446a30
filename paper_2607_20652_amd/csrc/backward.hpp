// The gradient to the coefficients, shared by the backward kernels: a wave's
// LDS regions, the child scores of the last level on the matrix cores, and
// the direct reductions of the other hashed slots.
#pragma once

#include "scoring.hpp"

namespace dpb {

struct Wave {
    int lane;
    int64_t t0;
    int ntok;
    int32_t* idx;     // [TPW][k]
    float* coef;      // [TPW][k]
    int32_t* route;   // [TPW][k]: (parent slot << 16) | j (| kClaimed when decoded by its column), or -1
    int32_t* par;     // [16] parent index of each column row
    float* alpha;     // [16][dpad] column coefficients
    int32_t* claim;   // [16][dpad] lowest slot claiming (row, j)
    int32_t* fri;     // [fr_cap] indices of the table-decoded slots
    float* frc;       // [fr_cap] their coefficients (0 for basis and padding slots)
    uint32_t* frv;    // [fr_cap / 32][8][16] slot-parity tables (256-byte aligned)
    float* frt;       // [fr_cap / 4][16] signed coefficient sums
    void* pb;         // [TPW][dp] sign bits of the leaf level's parents (pb_bytes each)
    float* y;         // [TPW][dp] output accumulator (fp32)
    uint32_t* pairs;  // [TPW][prow] g as signed bf16 pairs, interleaved halves
    float* gf;        // [TPW][dp] fp32 g (fp32 activations)
    uint32_t* cw;     // [16][cws] column sign bitmaps
    float* score;     // [16][16] scores of one column block and generator tile
    const uint32_t* mask;  // [dp] row masks (shared)
    const uint32_t* gtab;  // generator hash tables (shared): (g_j, j) pairs
    const uint32_t* gens;  // generators (shared)
};

// g at coordinate iota of token tt, from the LDS copy.
template <bool G_BF16>
__device__ __forceinline__ float g_at(const DevPlan& P, const Wave& W, int tt, int iota)
{
    if constexpr (G_BF16) return pair_value(P, W.pairs, tt, iota);
    else return W.gf[tt * P.dp + iota];
}

// Child scores of the parent columns of level l against the wave's g,
// written to the coefficients of the slots routed to them.
template <bool G_BF16>
__device__ void score_level(const DevPlan& P, const Wave& W, int l)
{
    const int k = P.k_tot, TPW = P.wave_tokens, lane = W.lane;
    const int CPT = P.cpt[l], csh = P.cpt_shift[l], Kp = P.active[l - 1], Kl = P.active[l];
    const int ncol = TPW * CPT, NB = (ncol + 15) >> 4, sbp = P.slot_base[l - 1], sbl = P.slot_base[l];
    const ActTile A{W.pairs, W.gf};
    const int col = lane & 15, kq = lane >> 4;
    for (int nb = 0; nb < NB; ++nb) {
        // (bf16: the fixed-offset form takes this kernel from 168 registers, three
        // waves per SIMD, to 170 or 210; 16,381 tokens d 768 k 288 169 us
        // without it and 218 with, in fp32 501 and 277)
        column_bitmaps<!G_BF16>(P, lane, W.ntok, csh, nb, W.idx + sbp, k, Kp, P.nt, W.cw);
        wave_sync();
        const int r = nb * 16 + col, tt = r >> csh, q = r & (CPT - 1);
        const bool valid = r < ncol && tt < W.ntok && q < Kp && W.idx[tt * k + sbp + q] >= 0;
        const int trow = valid ? tt : 0;
        for (int mb = 0; mb < P.mblocks[l]; ++mb) {
            const f32x4 acc = mfma_scores<G_BF16>(P, lane, l, mb, trow, A, W.cw);
#pragma unroll
            for (int i = 0; i < 4; ++i) W.score[col * 16 + kq * 4 + i] = acc[i] * P.rsd;
            wave_sync();
            // slots routed to a column of this block and a generator of this tile
            for (int tt2 = 0; tt2 < W.ntok; ++tt2)
                for (int s = sbl + lane; s < sbl + Kl; s += 64) {
                    const int rt = W.route[tt2 * k + s];
                    if (rt < 0) continue;
                    const int r2 = (tt2 << csh) + (rt >> 16), j = rt & 0xFFFF;
                    if ((r2 >> 4) == nb && (j >> 4) == mb) W.coef[tt2 * k + s] = W.score[(r2 & 15) * 16 + (j & 15)];
                }
            wave_sync();
        }
    }
}

typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

// c + a.lo b.lo + a.hi b.hi for bf16 pairs.  The operands are taken as plain
// words: a bit cast of a vector element (pq.y) reads element 0 with this
// compiler.
__device__ __forceinline__ float dot2u(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, a), __builtin_bit_cast(bf16x2v, b), c, false);
}

// +-1 bf16 pair carrying bits 15 and 31 of R as its signs
__device__ __forceinline__ uint32_t unit_pair(uint32_t R)
{
    return __builtin_amdgcn_bitop3_b32(R, 0x80008000u, 0x3F803F80u, 0xEA);   // (R & signs) | one
}

// grad_coef of the hashed slots that route nowhere: the scaled sum over the
// coordinates of g(iota) (-1)^{parity(M_iota & c)} for slot index c, with
// one lane per slot while 64 or more remain, then 2, 4 or 8 lanes per slot
// (each taking every 2nd, 4th or 8th chunk) in rounds of 32, 16 and 8 slots,
// so that the lanes stay busy (48 slots: 32 at two lanes, then 16 at four,
// 18 chunk steps instead of 24).  The slot's signs over the 32
// coordinates of chunk w form one word, the XOR of one nibble-table word per
// 4-bit group of c (parity is linear in the index bits).  bf16 g: dword o of
// the chunk holds coordinates o and o + 16, which meet the +-1 pair made from
// word bits o and o + 16 in a two-element dot product (fp32 accumulation).
template <bool G_BF16, int NG>
__device__ void direct_scores(const DevPlan& P, const Wave& W)
{
    static_assert(NG <= kNtGroupsPadded, "nibble groups beyond the padded tables");
    const int k = P.k_tot, n = W.ntok * k, lane = W.lane, nchunk = P.nchunk, d = P.d;
    int32_t* list = (int32_t*)W.score;   // 256 entries
    const uint64_t below = (1ull << lane) - 1;
    for (int w0 = 0; w0 < n; w0 += 256) {
        int m = 0;
        for (int b = w0; b < min(n, w0 + 256); b += 64) {
            const int i = b + lane;
            const bool act = i < n && W.idx[i] >= d && W.route[i] < 0;
            const uint64_t bal = __ballot(act);
            if (act) list[m + __popcll(bal & below)] = i;
            m += __popcll(bal);
        }
        wave_sync();
        for (int r0 = 0; r0 < m;) {
            const int rem = m - r0;
            const int sh = rem >= 64 ? 0 : rem >= 32 ? 1 : rem >= 16 ? 2 : 3;   // 2^sh lanes per slot
            const int mr = min(64 >> sh, rem);
            const int r = lane & ((64 >> sh) - 1), part = lane >> (6 - sh);
            const bool valid = r < mr;
            const int item = list[r0 + (valid ? r : 0)];
            const int tt = item / k;
            const uint32_t c = (uint32_t)W.idx[item];
            float acc0 = 0.f, acc1 = 0.f;
            // the nibble-table words of the next chunk are requested before
            // this chunk is summed (the device tables hold at least NG groups,
            // zero words past nt_groups)
            uint32_t toff[NG], tw[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) toff[g] = 4u * ((uint32_t)(g * nchunk * 16) + ((c >> (4 * g)) & 15u));
            const unsigned char* ntb = (const unsigned char*)P.nt;   // byte offsets: 32-bit address arithmetic
            auto fetch_words = [&](int w) {
#pragma unroll
                for (int g = 0; g < NG; ++g) tw[g] = *(const uint32_t*)(ntb + (toff[g] + (uint32_t)(w * 64)));
            };
            auto fold_words = [&]() {
                uint32_t v = 0;
#pragma unroll
                for (int g = 0; g < NG; ++g) v ^= tw[g];
                return v;
            };
            fetch_words(min(part, nchunk - 1));
            for (int w = part; w < nchunk; w += 1 << sh) {
                const uint32_t word = fold_words();
                fetch_words(min(w + (1 << sh), nchunk - 1));
                // keeps the compiler from sinking those loads to their use
                __asm__ volatile("" ::: "memory");
                if constexpr (G_BF16) {
                    const u32x4* pr = (const u32x4*)(W.pairs + tt * P.prow + w * 16);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const u32x4 pq = pr[q];
                        const int o = 4 * q;
                        acc0 = dot2u(pq.x, unit_pair(word << (15 - o)), acc0);
                        acc1 = dot2u(pq.y, unit_pair(word << (14 - o)), acc1);
                        acc0 = dot2u(pq.z, unit_pair(word << (13 - o)), acc0);
                        acc1 = dot2u(pq.w, unit_pair(word << (12 - o)), acc1);
                    }
                } else {
                    const float* gr = W.gf + tt * P.dp + 32 * w;
#pragma unroll
                    for (int b = 0; b < 32; b += 2) {
                        acc0 += __uint_as_float(__float_as_uint(gr[b]) ^ ((word << (31 - b)) & 0x80000000u));
                        acc1 += __uint_as_float(__float_as_uint(gr[b + 1]) ^ ((word << (30 - b)) & 0x80000000u));
                    }
                }
            }
            float acc = acc0 + acc1;
            for (int off = 64 >> sh; off < 64; off <<= 1) acc += __shfl_xor(acc, off, 64);
            if (valid && part == 0) W.coef[item] = P.rsd * acc;
            r0 += mr;
        }
        wave_sync();   // the list is rewritten by the next window
    }
}

struct BwdExtra {
    const float* gc;
    const void* gx;
    const float2* stats;
};

// Kernel variants: index groups NG in {3, 4, 5, 6, 8} (a larger NG than the
// plan needs is exact: the extra table rows are zero) and the width of the
// leaf parents' sign bits.
inline int ng_variant(const DevPlan& P)
{
    return P.nt_groups <= 3 ? 3 : P.nt_groups <= 6 ? P.nt_groups : 8;
}

// Column decode and backward (columns.hip, columns_bwd.hip): false when the
// plan is not theirs, and nothing was launched.
bool launch_col_decode(const DevPlan& P, const int32_t* idx, const float* coef, int64_t T, void* y, bool y_bf16,
                       hipStream_t stream);
bool launch_col_bwd(const DevPlan& P, const int32_t* idx, const void* g, bool g_bf16, int64_t T, float* grad_coef,
                    void* grad_x, bool gx_bf16, BwdExtra ex, hipStream_t stream);

}  // namespace dpb
