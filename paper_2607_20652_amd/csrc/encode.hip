// Encoder for gfx950: the top-down beam search of §2.2.
//
// A wave owns `wave_tokens` tokens (16 / CPT, CPT = parent columns per
// token rounded up to a power of two); their activations stay in LDS in the
// interleaved-halves layout of scoring.hpp.
//
//  * Level 0 (§2.1 Eq. 2: scoring a basis feature is a coordinate read):
//    each token's lanes take the maximum key over their coordinates; the
//    K_0-th largest lane maximum tau bounds the answer from below (the K_0
//    largest lane maxima are distinct keys >= tau), so only the few keys >= tau
//    are ranked exactly.  With bf16 activations a key is 32 bits: the bf16
//    magnitude above the complemented coordinate.
//  * With standardization statistics (mu, r = 1/sigma per feature, §2.2
//    "Score Standardization") every score s becomes z = (s - mu) r before it
//    is keyed: level 0 then uses 64-bit keys of fp32 z, and each child's
//    (mu, r) is gathered from the statistics table.
//  * Levels l >= 1: the children of every active parent are scored on the
//    matrix cores (§2.2 child-scoring equation); the 64-bit keys (|s| desc,
//    index asc, see device_common.hpp) are sorted by a bitonic network laid
//    over the MFMA output layout, unrolled at compile time, with DPP and
//    swizzle lane exchanges; a child reached from several parents has
//    bit-identical keys (same products, same reduction), so it appears as
//    adjacent duplicates and is kept once; the first K_l survivors are emitted
//    in order.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "scoring.hpp"

namespace dpb {
namespace {

constexpr int kEncWaves = 4;
constexpr int kEncThreads = 64 * kEncWaves;

struct EncLayout {
    unsigned act, cw, par, list, cnt, bytes;
    int kmaxp;   // row stride of par
    int listn;   // keys per token in list
};

__host__ __device__ inline int pow2_ceil(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

__host__ __device__ inline int enc_r(const DevPlan& P)
{
    int mb = 1;
    for (int l = 1; l < P.levels; ++l) mb = P.mblocks[l] > mb ? P.mblocks[l] : mb;
    return 4 * pow2_ceil(mb);
}

__host__ __device__ inline EncLayout enc_layout_with(const DevPlan& P, bool act_bf16, int listn)
{
    EncLayout L;
    const int TPW = P.wave_tokens;
    L.listn = listn;
    L.kmaxp = P.kmax;
    unsigned off = 0;
    L.act = off;
    off = align16u(off + (act_bf16 ? TPW * P.prow * 4 : TPW * P.dp * 4));
    L.cw = off;   off = align16u(off + 16 * P.cws * 4);
    L.par = off;  off = align16u(off + TPW * L.kmaxp * 4);
    L.list = off; off = align16u(off + TPW * listn * 8);
    L.cnt = off;  off = align16u(off + TPW * 4);
    L.bytes = off;
    return L;
}

// The least a wave needs: level-0 candidates, the K_0 lanes whose maximum
// reaches tau, each with all its keys; listn counts 64-bit words per token.
// Plain bf16 keys are 32 bits (2 ND per lane, two to a word); standardized
// and fp32 keys are 64.
inline EncLayout enc_layout_least(const DevPlan& P, bool act_bf16, bool std)
{
    const int LPT = 64 / P.wave_tokens;
    const int ND = (P.dp / 2 + LPT - 1) / LPT;  // activation dwords per lane at level 0
    return enc_layout_with(P, act_bf16,
                           (act_bf16 && !std) ? P.active[0] * ND
                                              : P.active[0] * (act_bf16 ? 2 * ND : (P.d + LPT - 1) / LPT));
}

// Shared LDS of an encoder workgroup: nibble tables, generators and, with
// standardization, the level-0 statistics.
__host__ __device__ inline unsigned enc_shared_bytes(const DevPlan& P, bool std)
{
    return align16u(P.nt_groups * 16 * P.nchunk * 4) + align16u(P.gens_total * 4) + (std ? align16u(P.d * 8) : 0u);
}

// The layout in use: where the LDS holds it, lists of one key per lane (the
// beam levels' selection).
inline EncLayout enc_layout(const DevPlan& P, bool act_bf16, bool std)
{
    const EncLayout least = enc_layout_least(P, act_bf16, std);
    const int lanes = 64 / P.wave_tokens;
    const EncLayout L = enc_layout_with(P, act_bf16, least.listn > lanes ? least.listn : lanes);
    return enc_shared_bytes(P, std) + kEncWaves * L.bytes <= (unsigned)kLdsBudget ? L : least;
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src)
{
    const uint32_t hi = (uint32_t)__shfl((int)(v >> 32), src, 64);
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, 64);
    return ((uint64_t)hi << 32) | lo;
}

// The value of the lane whose index differs by the bits of M.
template <int M, typename K>
__device__ __forceinline__ K xlane_mask(K v, int x32addr)
{
    auto one = [&](uint32_t w) -> uint32_t {
        if constexpr (M == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, false);
        else if constexpr (M == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, false);
        else if constexpr (M < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)w, (M << 10) | 0x1F);
        else return (uint32_t)__builtin_amdgcn_ds_bpermute(x32addr ^ ((M ^ 32) << 2), (int)w);
    };
    if constexpr (sizeof(K) == 8) return ((uint64_t)one((uint32_t)(v >> 32)) << 32) | one((uint32_t)v);
    else return one(v);
}

// Lane bits of position bit B, and of position bits 0 .. B (see sort_desc).
template <bool MFMA_LAYOUT, int B>
constexpr int lane_bit() { return MFMA_LAYOUT ? (B < 2 ? (16 << B) : (1 << (B - 2))) : (1 << B); }
template <bool MFMA_LAYOUT, int B>
constexpr int lane_bits()
{
    if constexpr (B < 0) return 0;
    else return lane_bit<MFMA_LAYOUT, B>() | lane_bits<MFMA_LAYOUT, B - 1>();
}

// One exchange with the lanes at mask M: the lane with position bit B clear
// keeps the larger keys.  FLIP: against the other lane's registers in reverse.
template <int R, int M, int B, bool FLIP, typename K>
__device__ __forceinline__ void sort_lanes(K (&v)[R], int lanepos, int x32addr)
{
    const bool lower = !((lanepos >> B) & 1);
    K o[R];
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] = xlane_mask<M>(v[FLIP ? R - 1 - r : r], x32addr);
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = ((o[r] > v[r]) == lower) ? o[r] : v[r];
}

template <int R, bool MFMA_LAYOUT, int JS, typename K>
__device__ __forceinline__ void sort_halves(K (&v)[R], int lanepos, int x32addr)
{
    constexpr int LR = R == 1 ? 0 : R == 2 ? 1 : R == 4 ? 2 : R == 8 ? 3 : 4;
    if constexpr (JS >= 0) {
        if constexpr (JS >= LR) {
            sort_lanes<R, lane_bit<MFMA_LAYOUT, JS - LR>(), JS - LR, false>(v, lanepos, x32addr);
        } else {
            constexpr int j = 1 << JS;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r & j) continue;
                const K a = v[r], c = v[r | j];
                v[r] = key_max(a, c);
                v[r | j] = key_min(a, c);
            }
        }
        sort_halves<R, MFMA_LAYOUT, JS - 1>(v, lanepos, x32addr);
    }
}

template <int R, int NB, bool MFMA_LAYOUT, int KS, typename K>
__device__ __forceinline__ void sort_merge(K (&v)[R], int lanepos, int x32addr)
{
    constexpr int LR = R == 1 ? 0 : R == 2 ? 1 : R == 4 ? 2 : R == 8 ? 3 : 4;
    if constexpr (KS <= LR + NB) {
        if constexpr (KS > LR) {
            sort_lanes<R, lane_bits<MFMA_LAYOUT, KS - LR - 1>(), KS - LR - 1, true>(v, lanepos, x32addr);
        } else {
            constexpr int mirror = (1 << KS) - 1;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if ((r ^ mirror) < r) continue;
                const K a = v[r], c = v[r ^ mirror];
                v[r] = key_max(a, c);
                v[r ^ mirror] = key_min(a, c);
            }
        }
        sort_halves<R, MFMA_LAYOUT, KS - 2>(v, lanepos, x32addr);
        sort_merge<R, NB, MFMA_LAYOUT, KS + 1>(v, lanepos, x32addr);
    }
}

// Descending bitonic sort of one token's R * 2^NB keys: element e =
// lanepos * R + r lives in register r of the lane at position lanepos.  In
// the MFMA layout lanepos = q * 4 + kq (q = lane bits 0.., kq = lane bits
// 4, 5); otherwise lanepos bit b is lane bit b.  Each merge first compares an
// element with its mirror image in the block, so every block is sorted
// descending and no comparison's direction depends on the lane: a
// compare-exchange within a lane is one maximum and one minimum (the form with
// alternating directions took five instructions for 64-bit keys).
template <int R, int NB, bool MFMA_LAYOUT, typename K>
__device__ __forceinline__ void sort_desc(K (&v)[R], int lanepos, int x32addr)
{
    sort_merge<R, NB, MFMA_LAYOUT, 1>(v, lanepos, x32addr);
}

// Emits the first K distinct keys of each token straight from the sorted
// registers of the MFMA layout (position lanepos * R + r): duplicates are
// adjacent, the predecessor of register 0 comes from the lane at lanepos - 1,
// and ranks are prefix counts in lanepos order.  Writes slots [sb, sb + K)
// and records them as the next parents.
template <int R, int CPT>
__device__ __forceinline__ void emit_mfma(const DevPlan& P, const uint64_t (&key)[R], int lane, int lanepos, int ct,
                                          int prev_addr, uint64_t before_mask, uint64_t token_mask, int64_t t0,
                                          int ntok, int K, int sb, int32_t* par, int kmaxp, int32_t* out_idx,
                                          float* out_coef)
{
    (void)lane;
    const int k_tot = P.k_tot;
    const uint32_t ph = (uint32_t)__builtin_amdgcn_ds_bpermute(prev_addr, (int)(uint32_t)(key[R - 1] >> 32));
    const uint32_t pl = (uint32_t)__builtin_amdgcn_ds_bpermute(prev_addr, (int)(uint32_t)key[R - 1]);
    uint64_t prev = lanepos > 0 ? (((uint64_t)ph << 32) | pl) : 0ull;
    int kept = 0, cnt = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool k = key[r] != 0ull && key[r] != prev;
        kept |= (int)k << r;
        cnt += (int)k;
        prev = key[r];
    }
    int before = 0, total = 0;
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const uint64_t m = __ballot((cnt >> b) & 1);
        before += (int)__popcll(m & before_mask) << b;
        total += (int)__popcll(m & token_mask) << b;
    }
    const bool live = ct < ntok;
    int rank = before;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (((kept >> r) & 1) && rank < K) {
            const uint32_t ci = key_index(key[r]);
            par[ct * kmaxp + rank] = (int32_t)ci;
            if (live) {
                out_idx[(t0 + ct) * k_tot + sb + rank] = (int32_t)ci;
                out_coef[(t0 + ct) * k_tot + sb + rank] = key_value(key[r]);
            }
        }
        rank += (kept >> r) & 1;
    }
    for (int r = total + lanepos; r < K; r += 4 * CPT) {
        par[ct * kmaxp + r] = -1;
        if (live) {
            out_idx[(t0 + ct) * k_tot + sb + r] = -1;
            out_coef[(t0 + ct) * k_tot + sb + r] = 0.f;
        }
    }
}

// Level 0, bf16 activations: 32-bit keys (|x| bf16 bits << 16 | 0xFFFF - iota).
// Lane li of token tt reads the interleaved dwords e = li + LPT m; dword e
// holds coordinates 32 (e >> 4) + (e & 15) (low half) and that + 16.
// Coordinates past d hold zeros, so their keys sort below every real key.
template <int LPT, int LLP>
__device__ void level0_bf16(const DevPlan& P, int lane, int64_t t0, int ntok, const uint32_t* pairs, uint64_t* list,
                            int listn, int* cnt, int32_t* par, int kmaxp, int32_t* out_idx, float* out_coef,
                            int x32addr)
{
    const int tt = lane >> LLP, li = lane & (LPT - 1), K0 = P.active[0], dp2 = P.dp / 2;
    const uint32_t* row = pairs + tt * P.prow;
    const int lo0 = 32 * (li >> 4) + (li & 15);  // coordinate of the low half of dword li
    constexpr uint32_t STEP = 2 * LPT;           // coordinate step per dword row
    uint32_t best = 0;
    {
        uint32_t c = 0xFFFFu - (uint32_t)lo0;
        for (int e = li; e < dp2; e += LPT, c -= STEP) {
            const uint32_t D = row[e];
            const uint32_t klo = ((D << 16) & 0x7FFF0000u) | c, khi = (D & 0x7FFF0000u) | (c - 16u);
            best = max(best, max(klo, khi));
        }
    }
    uint32_t sv[1] = {best};
    sort_desc<1, LLP, false>(sv, li, x32addr);
    const uint32_t tau = (uint32_t)__shfl((int)sv[0], (lane & ~(LPT - 1)) + K0 - 1, 64);
    if (li == 0) cnt[tt] = 0;
    wave_sync();
    uint32_t* lst = (uint32_t*)(list + tt * listn);
    {
        uint32_t c = 0xFFFFu - (uint32_t)lo0;
        for (int e = li; e < dp2; e += LPT, c -= STEP) {
            const uint32_t D = row[e];
            const uint32_t klo = ((D << 16) & 0x7FFF0000u) | c, khi = (D & 0x7FFF0000u) | (c - 16u);
            if (klo >= tau) lst[atomicAdd(&cnt[tt], 1)] = klo;
            if (khi >= tau) lst[atomicAdd(&cnt[tt], 1)] = khi;
        }
    }
    wave_sync();
    const int n = cnt[tt];
    const bool live = tt < ntok;
    for (int e = li; e < n; e += LPT) {
        const uint32_t ke = lst[e];
        int rank = 0;
        for (int f = 0; f < n; ++f) rank += lst[f] > ke;
        if (rank < K0) {
            const uint32_t iota = 0xFFFFu - (ke & 0xFFFFu);
            par[tt * kmaxp + rank] = (int32_t)iota;
            if (live) {
                out_idx[(t0 + tt) * P.k_tot + rank] = (int32_t)iota;
                out_coef[(t0 + tt) * P.k_tot + rank] = pair_value(P, pairs, tt, (int)iota);
            }
        }
    }
}

// Level 0, fp32 activations: 64-bit keys over natural-order coordinates.
template <int LPT, int LLP>
__device__ void level0_f32(const DevPlan& P, int lane, int64_t t0, int ntok, const float* xf, uint64_t* list,
                           int listn, int* cnt, int32_t* par, int kmaxp, int32_t* out_idx, float* out_coef,
                           int x32addr)
{
    const int tt = lane >> LLP, li = lane & (LPT - 1), K0 = P.active[0], d = P.d, dp = P.dp;
    const float* row = xf + tt * dp;
    uint64_t best = 0;
    for (int iota = li; iota < d; iota += LPT) best = max(best, make_key(row[iota], (uint32_t)iota));
    uint64_t sv[1] = {best};
    sort_desc<1, LLP, false>(sv, li, x32addr);
    const uint64_t tau = shfl_u64(sv[0], (lane & ~(LPT - 1)) + K0 - 1);
    if (li == 0) cnt[tt] = 0;
    wave_sync();
    uint64_t* lst = list + tt * listn;
    for (int iota = li; iota < d; iota += LPT) {
        const uint64_t kk = make_key(row[iota], (uint32_t)iota);
        if (kk >= tau) lst[atomicAdd(&cnt[tt], 1)] = kk;
    }
    wave_sync();
    const int n = cnt[tt];
    const bool live = tt < ntok;
    for (int e = li; e < n; e += LPT) {
        const uint64_t ke = lst[e];
        int rank = 0;
        for (int f = 0; f < n; ++f) rank += lst[f] > ke;
        if (rank < K0) {
            const uint32_t iota = key_index(ke);
            par[tt * kmaxp + rank] = (int32_t)iota;
            if (live) {
                out_idx[(t0 + tt) * P.k_tot + rank] = (int32_t)iota;
                out_coef[(t0 + tt) * P.k_tot + rank] = key_value(ke);
            }
        }
    }
}

// Level 0 on standardized scores z = (x - mu) r (§2.2 "Score
// Standardization"), in fp32: 64-bit keys over the coordinates, as level0_f32,
// with the level-0 statistics staged in LDS (st0).  With bf16 activations lane
// li reads the interleaved dwords e = li + LPT m (coordinates 32 (e >> 4) +
// (e & 15) and that + 16); coordinates past d get key 0.
template <int LPT, int LLP, bool X_BF16>
__device__ void level0_std(const DevPlan& P, int lane, int64_t t0, int ntok, const uint32_t* pairs, const float* xf,
                           const float2* st0, uint64_t* list, int listn, int* cnt, int32_t* par, int kmaxp,
                           int32_t* out_idx, float* out_coef, int x32addr)
{
    const int tt = lane >> LLP, li = lane & (LPT - 1), K0 = P.active[0], d = P.d;
    auto zkey = [&](float x, int iota) -> uint64_t {
        if (iota >= d) return 0ull;
        const float2 st = st0[iota];
        return make_key((x - st.x) * st.y, (uint32_t)iota);
    };
    uint64_t best = 0;
    if constexpr (X_BF16) {
        const uint32_t* row = pairs + tt * P.prow;
        for (int e = li; e < P.dp / 2; e += LPT) {
            const uint32_t D = row[e];
            const int lo = 32 * (e >> 4) + (e & 15);
            best = max(best, max(zkey(bf16_bits_to_f32(D & 0xFFFFu), lo), zkey(bf16_bits_to_f32(D >> 16), lo + 16)));
        }
    } else {
        const float* row = xf + tt * P.dp;
        for (int iota = li; iota < d; iota += LPT) best = max(best, zkey(row[iota], iota));
    }
    uint64_t sv[1] = {best};
    sort_desc<1, LLP, false>(sv, li, x32addr);
    const uint64_t tau = shfl_u64(sv[0], (lane & ~(LPT - 1)) + K0 - 1);
    if (li == 0) cnt[tt] = 0;
    wave_sync();
    uint64_t* lst = list + tt * listn;
    if constexpr (X_BF16) {
        const uint32_t* row = pairs + tt * P.prow;
        for (int e = li; e < P.dp / 2; e += LPT) {
            const uint32_t D = row[e];
            const int lo = 32 * (e >> 4) + (e & 15);
            const uint64_t klo = zkey(bf16_bits_to_f32(D & 0xFFFFu), lo), khi = zkey(bf16_bits_to_f32(D >> 16), lo + 16);
            if (klo >= tau && klo != 0ull) lst[atomicAdd(&cnt[tt], 1)] = klo;
            if (khi >= tau && khi != 0ull) lst[atomicAdd(&cnt[tt], 1)] = khi;
        }
    } else {
        const float* row = xf + tt * P.dp;
        for (int iota = li; iota < d; iota += LPT) {
            const uint64_t kk = zkey(row[iota], iota);
            if (kk >= tau) lst[atomicAdd(&cnt[tt], 1)] = kk;
        }
    }
    wave_sync();
    const int n = cnt[tt];
    const bool live = tt < ntok;
    for (int e = li; e < n; e += LPT) {
        const uint64_t ke = lst[e];
        int rank = 0;
        for (int f = 0; f < n; ++f) rank += lst[f] > ke;
        if (rank < K0) {
            const uint32_t iota = key_index(ke);
            par[tt * kmaxp + rank] = (int32_t)iota;
            if (live) {
                out_idx[(t0 + tt) * P.k_tot + rank] = (int32_t)iota;
                out_coef[(t0 + tt) * P.k_tot + rank] = key_value(ke);
            }
        }
    }
}

// The variants for bf16 input with one block of sixteen parent columns per
// level and plain scores (one or two tokens per wave) are held to 128
// registers, four waves per SIMD: both fit without spilling.  The two-token
// variant gains from it only because its level-0 list holds 32-bit keys at
// half the 64-bit size, so that four workgroups fit the LDS of a CU.
template <bool X_BF16, int CPT, int R, bool STD>
__global__ __launch_bounds__(kEncThreads, (X_BF16 && (CPT == 16 || CPT == 8) && R == 4 && !STD) ? 4 : 1) void encode3_kernel(DevPlan P, int listn, const void* __restrict__ xin, int64_t T,
                                                              const float2* __restrict__ stats,
                                                              int32_t* __restrict__ out_idx,
                                                              float* __restrict__ out_coef)
{
    constexpr int TPW = 16 / CPT, LPT = 64 / TPW;
    constexpr int CB = CPT == 4 ? 2 : CPT == 8 ? 3 : 4;  // log2 CPT
    constexpr int NB = CB + 2;                            // lane bits of a token in the MFMA layout
    constexpr int LLP = LPT == 16 ? 4 : LPT == 32 ? 5 : 6;
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t* s_nt = (uint32_t*)smem;
    uint32_t* s_gens = (uint32_t*)(smem + align16u(P.nt_groups * 16 * P.nchunk * 4));
    float2* s_st0 = (float2*)(smem + enc_shared_bytes(P, false));   // level-0 statistics (STD)
    for (int i = threadIdx.x; i < P.nt_groups * 16 * P.nchunk; i += kEncThreads) s_nt[i] = P.nt[i];
    for (int i = threadIdx.x; i < P.gens_total; i += kEncThreads) s_gens[i] = P.gens[i];
    if constexpr (STD)
        for (int i = threadIdx.x; i < P.d; i += kEncThreads) s_st0[i] = stats[i];
    __syncthreads();

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int d = P.d, dp = P.dp;
    const int x32 = (lane ^ 32) << 2;
    const EncLayout EL = enc_layout_with(P, X_BF16, listn);
    unsigned char* wb = smem + enc_shared_bytes(P, STD) + (unsigned)wave * EL.bytes;
    uint32_t* pairs = (uint32_t*)(wb + EL.act);
    float* xf = (float*)(wb + EL.act);
    uint32_t* cw = (uint32_t*)(wb + EL.cw);
    int32_t* par = (int32_t*)(wb + EL.par);
    uint64_t* list = (uint64_t*)(wb + EL.list);
    int* cnt = (int*)(wb + EL.cnt);
    const ActTile A{pairs, xf};

    const int col = lane & 15, kq = lane >> 4, ct = col >> CB, q = col & (CPT - 1), lanepos = q * 4 + kq;
    // lanepos order inside a token: lanes of positions below mine, all lanes of my token, lane of lanepos - 1
    uint64_t before_mask = 0, token_mask = 0;
    for (int q2 = 0; q2 < CPT; ++q2)
        for (int k2 = 0; k2 < 4; ++k2) {
            const uint64_t bit = 1ull << (ct * CPT + q2 + 16 * k2);
            token_mask |= bit;
            if (q2 * 4 + k2 < lanepos) before_mask |= bit;
        }
    const int prev_addr = (kq > 0 ? lane - 16 : lane + 47) << 2;

    const int64_t ngroups = (T + TPW - 1) / TPW;
    const int64_t gstride = (int64_t)gridDim.x * kEncWaves;
    // bf16 rows of two tokens with d <= 1024 (d a multiple of 8): the next
    // group's rows are requested while this group is encoded
    const bool pf = X_BF16 && TPW == 2 && d <= 1024 && (d & 7) == 0;
    u32x4 nx[4];
    auto fetch = [&](int64_t gp) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int tt = e >> 1, o = (e & 1) * 512 + lane * 8;
            const int64_t t = gp * TPW + tt;
            nx[e] = (o < d && t < T) ? *(const u32x4*)((const uint16_t*)xin + t * d + o) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    int64_t grp = (int64_t)blockIdx.x * kEncWaves + wave;
    if (pf && grp < ngroups) fetch(grp);
    for (; grp < ngroups; grp += gstride) {
        const int64_t t0 = grp * TPW;
        const int ntok = (int)min((int64_t)TPW, T - t0);

        if (pf) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = (e & 1) * 512 + lane * 8;
                if (o < dp) store_pair_piece(lane, nx[e], o, pairs + (e >> 1) * P.prow);
            }
            if (grp + gstride < ngroups) fetch(grp + gstride);
        } else if constexpr (X_BF16) {
            load_pairs(P, lane, ntok, TPW, (const uint16_t*)xin, t0, pairs);
        } else {
            const float* xs = (const float*)xin;
            for (int tt = 0; tt < TPW; ++tt)
                for (int iota = lane; iota < dp; iota += 64)
                    xf[tt * dp + iota] = (tt < ntok && iota < d) ? xs[(t0 + tt) * d + iota] : 0.f;
        }
        wave_sync();

        // ---- level 0
        if constexpr (STD)
            level0_std<LPT, LLP, X_BF16>(P, lane, t0, ntok, pairs, xf, s_st0, list, EL.listn, cnt, par, EL.kmaxp,
                                         out_idx, out_coef, x32);
        else if constexpr (X_BF16)
            level0_bf16<LPT, LLP>(P, lane, t0, ntok, pairs, list, EL.listn, cnt, par, EL.kmaxp, out_idx,
                                  out_coef, x32);
        else
            level0_f32<LPT, LLP>(P, lane, t0, ntok, xf, list, EL.listn, cnt, par, EL.kmaxp, out_idx, out_coef, x32);
        wave_sync();

        // ---- levels l >= 1
        for (int l = 1; l < P.levels; ++l) {
            const int Kp = P.active[l - 1], Dl = P.delta[l];
            column_bitmaps(P, lane, ntok, CB, 0, par, EL.kmaxp, Kp, s_nt, cw);
            wave_sync();
            const int32_t p = (ct < ntok && q < Kp) ? par[ct * EL.kmaxp + q] : -1;
            const bool valid = p >= 0;
            const int trow = valid ? ct : 0;
            const uint32_t* gens = s_gens + P.gens_off[l];
            // standardization statistics of this lane's children, gathered
            // during the last batch of the first tile's scoring (read
            // unconditionally at an index that is always a feature: a
            // generator of the level when there is no parent)
            float2 stv[R];
            auto gather = [&]() {
                if constexpr (STD) {
#pragma unroll
                    for (int e = 0; e < R; ++e) {
                        const int j = 16 * (e >> 2) + 4 * kq + (e & 3);
                        const float2 v = stats[(valid ? (uint32_t)p : 0u) ^ gens[min(j, Dl - 1)]];
                        stv[e] = (valid && j < Dl) ? v : make_float2(0.f, 1.f);
                    }
                }
            };
            uint64_t keys[R];
#pragma unroll
            for (int mb = 0; mb < R / 4; ++mb) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                // batches of 6 chunks: faster here than 4, 8 or 12
                if (mb == 0) acc = mfma_scores<X_BF16, 6>(P, lane, l, mb, trow, A, cw, gather);
                else if (mb < P.mblocks[l]) acc = mfma_scores<X_BF16, 6>(P, lane, l, mb, trow, A, cw);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = 16 * mb + 4 * kq + i;
                    const bool ok = valid && j < Dl;
                    const uint32_t c = ok ? (uint32_t)p ^ gens[j] : 0u;
                    float sc = acc[i] * P.rsd;
                    if constexpr (STD) sc = (sc - stv[4 * mb + i].x) * stv[4 * mb + i].y;
                    keys[4 * mb + i] = ok ? make_sort_key(sc, c) : 0ull;
                }
            }
            // Levels that keep few of their candidates (K_l <= 2 CPT, the beam
            // levels): the K_l-th largest lane maximum tau bounds the answer (at
            // least K_l keys reach it); the keys with a magnitude >= tau are
            // listed (at most one per lane of the token), each lane counts
            // the listed keys above its own, and the key goes to that place of
            // the list.  Equal keys (a child reached from two parents)
            // share a place and leave the next one empty, so the distinct keys
            // are the occupied places in order.  A token with fewer than K_l
            // distinct ones although not all are listed takes the K_l-th
            // distinct lane maximum for tau and lists again; one with more
            // listed keys than lanes sorts all its keys.  (Sorting the list
            // as 64-bit keys and ranking by ballots took 270 vector instructions a
            // level, this takes about 150; with the sort of fixed directions:
            // 65,536 tokens d 768 268 -> 238 us, 16,384 tokens d 1024 N 2^24
            // 188 -> 171, standardized 367 -> 331.)
            const int Kl = P.active[l];
            bool done = false;
            if (Kl <= 2 * CPT && EL.listn >= 4 * CPT) {
                uint32_t mg[R], top[1] = {0u};
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    mg[r] = (uint32_t)(keys[r] >> 32);
                    top[0] = max(top[0], mg[r]);
                }
                uint64_t* tl = list + ct * EL.listn;
                sort_desc<1, NB, true>(top, lanepos, x32);
                // the lane at position K_l - 1 of my token
                const int at = Kl - 1, src = ct * CPT + (at >> 2) + 16 * (at & 3);
                uint32_t tau = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)top[0]);
                for (bool again = false;; again = true) {
                    uint32_t z = 0;
                    __asm__ volatile("" : "+v"(z));   // not kept in registers across the levels
                    const uint64_t none = ((uint64_t)z << 32) | z;
                    tl[lanepos] = none;
                    if (lanepos == 0) cnt[ct] = 0;
                    uint32_t hits = 0u;
#pragma unroll
                    for (int r = 0; r < R; ++r) hits |= (uint32_t)(keys[r] != 0ull && mg[r] >= tau) << r;
                    wave_sync();
                    int pos = hits ? atomicAdd(&cnt[ct], (int)__popc(hits)) : 0;
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if ((hits >> r) & 1u) {
                            if (pos < 4 * CPT) tl[pos] = keys[r];
                            ++pos;
                        }
                    wave_sync();
                    const int n = cnt[ct];
                    if (__ballot(n > 4 * CPT)) break;
                    const uint64_t e = tl[lanepos];
                    int above = 0;
                    for (int f = 0; __ballot(f < n); f += 4) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) above += (int)(tl[f + u] > e);
                    }
                    wave_sync();
                    tl[lanepos] = none;
                    wave_sync();
                    if (e != 0ull) tl[above] = e;
                    wave_sync();
                    const uint64_t k = tl[lanepos];
                    const uint64_t full = __ballot(k != 0ull);
                    const int rank = (int)__popcll(full & before_mask), total = (int)__popcll(full & token_mask);
                    if (!__ballot(total < Kl && tau != 0u)) {
                        int32_t* pr = par + ct * EL.kmaxp;
                        const bool live = ct < ntok;
                        const int64_t o = (t0 + ct) * P.k_tot + P.slot_base[l];
                        if (k != 0ull && rank < Kl) {
                            const uint32_t ci = key_index(k);
                            pr[rank] = (int32_t)ci;
                            if (live) {
                                out_idx[o + rank] = (int32_t)ci;
                                out_coef[o + rank] = key_value(k);
                            }
                        }
                        for (int r = total + lanepos; r < Kl; r += 4 * CPT) {
                            pr[r] = -1;
                            if (live) {
                                out_idx[o + r] = -1;
                                out_coef[o + r] = 0.f;
                            }
                        }
                        done = true;
                        break;
                    }
                    if (again) break;
                    // the K_l-th distinct lane maximum (equal ones are neighbours), 0 if there is none
                    const uint32_t prev = (uint32_t)__builtin_amdgcn_ds_bpermute(prev_addr, (int)top[0]);
                    const bool kept = top[0] != 0u && (lanepos == 0 || top[0] != prev);
                    const int drank = (int)__popcll(__ballot(kept) & before_mask);
                    const uint64_t owner = __ballot(kept && drank == Kl - 1) & token_mask;
                    const uint32_t dtau =
                        (uint32_t)__builtin_amdgcn_ds_bpermute((int)__builtin_ctzll(owner | (1ull << 63)) << 2, (int)top[0]);
                    tau = owner ? dtau : 0u;
                    wave_sync();
                }
                wave_sync();
            }
            if (!done) {
                sort_desc<R, NB, true>(keys, lanepos, x32);
                emit_mfma<R, CPT>(P, keys, lane, lanepos, ct, prev_addr, before_mask, token_mask, t0, ntok, Kl,
                                  P.slot_base[l], par, EL.kmaxp, out_idx, out_coef);
            }
            wave_sync();
        }
    }
}

// ---------------------------------------------------------------------------
// Wide encoder: levels that score many children per parent (the paper's own
// hierarchies score 256, App. G Table 6).  Level 0 runs one wave per token.
// Each level l >= 1 is then a GEMM and a selection over chunks of tokens:
//  * wide_gemm_kernel: the scores of all K_{l-1} x Delta_l children of the
//    chunk's tokens, S[(t, q)][j] = <gamma_j, phi~_{p_tq} (.) x_t> (§2.2
//    child-scoring equation), as 16x16x32 bf16 MFMAs over a workgroup tile of
//    all generator rows x 128 (token, parent) columns.  A fragments (exact
//    +-1) are built from per-generator sign bitmaps held in LDS, B fragments
//    from the token rows and the parents' sign bitmaps (nibble tables), as in
//    the narrow encoder.  Its epilogue computes each token's threshold (the
//    K_l-th largest distinct magnitude among the lanes' maxima; distinct
//    magnitudes are distinct children) and writes only the (candidate, z)
//    entries at or above it to the workspace (with standardization it first
//    takes z = (s - mu) r with each candidate's gathered statistics); tokens
//    with too many entries and shapes it does not cover get the full scores.
//  * wide_select_kernel: one wave per token; AbsTopK with deduplication (a
//    child reached from several parents has bit-identical keys): the listed
//    entries, or the candidates above the same threshold found from the full
//    scores, are sorted as 64-bit keys by a bitonic network and the first K
//    distinct ones emitted; too many hits fall back to an exact extraction
//    (K rounds of a wave maximum below the previous key).
constexpr int kWideCols = 128;     // (token, parent) columns of a GEMM workgroup
constexpr int kWideList = 1024;    // collected keys per token
constexpr int kSeg = 16;           // keys per lane segment (64 kSeg = kWideList)
constexpr int kSegStride = kSeg + 1;
static_assert(64 * kSeg == kWideList && kSeg < 32, "segments fill the list; counts fit five bits");
constexpr int kWideThreads = 256;
static_assert(kWideThreads % kWideCols == 0, "column bitmaps: whole columns per thread group");
// (the fused epilogue keeps a lane's hits of one column tile, 4 MT <= 32 values, in one word)

template <bool X_BF16, bool STD>
__global__ __launch_bounds__(kWideThreads) void wide_level0_kernel(DevPlan P, const void* __restrict__ xin, int64_t T,
                                                                   const float2* __restrict__ stats,
                                                                   int32_t* __restrict__ out_idx,
                                                                   float* __restrict__ out_coef)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, d = P.d, dp = P.dp;
    const int ND = (dp / 2 + 63) / 64;
    const int listn = P.active[0] * (X_BF16 ? 2 * ND : (d + 63) / 64);
    const unsigned act_b = align16u(X_BF16 ? P.prow * 4 : dp * 4);
    const unsigned per_wave = act_b + align16u(listn * 8) + align16u((P.active[0] + 1) * 4) + 16;
    float2* st0 = (float2*)smem;
    unsigned char* wb = smem + (STD ? align16u(d * 8) : 0u) + wave * per_wave;
    uint32_t* pairs = (uint32_t*)wb;
    float* xf = (float*)wb;
    uint64_t* list = (uint64_t*)(wb + act_b);
    int32_t* par = (int32_t*)(wb + act_b + align16u(listn * 8));
    int* cnt = (int*)(wb + act_b + align16u(listn * 8) + align16u((P.active[0] + 1) * 4));
    if constexpr (STD) {
        for (int i = threadIdx.x; i < d; i += kWideThreads) st0[i] = stats[i];
        __syncthreads();
    }
    const int x32 = (lane ^ 32) << 2;
    for (int64_t t = (int64_t)blockIdx.x * 4 + wave; t < T; t += (int64_t)gridDim.x * 4) {
        if constexpr (X_BF16) {
            load_pairs(P, lane, 1, 1, (const uint16_t*)xin, t, pairs);
        } else {
            const float* xs = (const float*)xin;
            for (int iota = lane; iota < dp; iota += 64) xf[iota] = iota < d ? xs[t * d + iota] : 0.f;
        }
        wave_sync();
        if constexpr (STD)
            level0_std<64, 6, X_BF16>(P, lane, t, 1, pairs, xf, st0, list, listn, cnt, par, 0, out_idx, out_coef, x32);
        else if constexpr (X_BF16)
            level0_bf16<64, 6>(P, lane, t, 1, pairs, list, listn, cnt, par, 0, out_idx, out_coef, x32);
        else
            level0_f32<64, 6>(P, lane, t, 1, xf, list, listn, cnt, par, 0, out_idx, out_coef, x32);
        wave_sync();
    }
}

// Exclusive prefix over the wave of per-lane counts below 2^BITS.
template <int BITS>
__device__ __forceinline__ int wave_prefix(int cnt, int lane, int& total)
{
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int before = 0;
    total = 0;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint64_t m = __ballot((cnt >> b) & 1);
        before += (int)__popcll(m & below) << b;
        total += (int)__popcll(m) << b;
    }
    return before;
}
__device__ __forceinline__ int wave_prefix5(int cnt, int lane, int& total) { return wave_prefix<5>(cnt, lane, total); }

// LDS of a GEMM workgroup: generator bitmaps, the tokens' rows, column bitmaps.
__host__ __device__ inline unsigned wide_gemm_lds(const DevPlan& P, int l, bool x_bf16)
{
    const int TT = kWideCols / P.cpt[l];
    return align16u(P.gpad[l] * P.cws * 4) + align16u(TT * (x_bf16 ? P.prow : P.dp) * 4) +
           align16u(kWideCols * P.cws * 4) + align16u(kWideCols * 4);
}

// Whether level l's GEMM selects in its epilogue: 16 to 64 parent columns per
// token (whole tokens per 64-column wave tile) and a token's score region can
// hold the kWideList (candidate, z) entries plus the discard entry after them.
// The fused epilogue reuses the staging LDS: the lane maxima, thresholds and
// counts below kWideEpiZ, then each wave's z values of one column tile.
constexpr unsigned kWideEpiZ = 8192;
__host__ __device__ inline unsigned wide_epi_lds(int MT) { return kWideEpiZ + 4u * 64u * (4u * MT + 4u) * 4u; }

__host__ __device__ inline bool wide_fused(const DevPlan& P, int l)
{
    const int MT = (P.delta[l] > 32 ? P.delta[l] : 32) / 32;
    return P.cpt[l] >= 16 && P.cpt[l] <= 64 && P.active[l - 1] * P.delta[l] >= 2 * (kWideList + 1) &&
           wide_gemm_lds(P, l, true) - align16u(kWideCols * 4) >= wide_epi_lds(MT);
}

// max(m, |a|, |b|); a NaN among them gives NaN.
__device__ __forceinline__ float max3_abs(float m, float a, float b)
{
    return __builtin_elementwise_maximum(m, __builtin_elementwise_maximum(__builtin_fabsf(a), __builtin_fabsf(b)));
}

// hm shifted left by four, a bit per value: |v| >= tau or unordered.  Two
// instructions a value (compare, add with carry); each carry is read at
// least two instructions after its compare, which gfx950 asks for.
__device__ __forceinline__ uint32_t shift_in_not_less(uint32_t hm, f32x4 v, float tau)
{
    uint64_t c0, c1, c2, c3;
    __asm__("v_cmp_nlt_f32 %1, abs(%5), %9\n\t"
            "v_cmp_nlt_f32 %2, abs(%6), %9\n\t"
            "v_cmp_nlt_f32 %3, abs(%7), %9\n\t"
            "v_cmp_nlt_f32 %4, abs(%8), %9\n\t"
            "v_addc_co_u32 %0, vcc, %0, %0, %1\n\t"
            "v_addc_co_u32 %0, vcc, %0, %0, %2\n\t"
            "v_addc_co_u32 %0, vcc, %0, %0, %3\n\t"
            "v_addc_co_u32 %0, vcc, %0, %0, %4"
            : "+v"(hm), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
            : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(tau)
            : "vcc");
    return hm;
}

// Set bits of m in lanes below this one.
__device__ __forceinline__ int lanes_below(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Scores of tokens [t0 + TT blockIdx.x, ...) of a chunk of ntok tokens at level
// l into scores[(t - t0) K_{l-1} + q][j] (t0-relative tokens).  MT = 16-row
// tiles per wave: waves (wr, wc) cover rows 16 MT wr .. and columns 64 wc ..
// FUSE: instead of all scores, each token's region receives the (candidate,
// z) entries at or above a threshold tau computed here from the lanes'
// largest magnitude keys (the selection's first pass), and counts[t - t0]
// their number; a token with more than kWideList entries gets its full scores
// and its count says so.  STD (with FUSE): every score is standardized here,
// z = (s - mu) r with the candidate's statistics (§2.2 "Score
// Standardization"), so that the threshold, the lists and any full scores
// hold z.
template <bool X_BF16, int MT, bool FUSE, bool STD>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(2))) void wide_gemm_kernel(DevPlan P, int l, const void* __restrict__ xin,
                                                                 int64_t t0, int64_t ntok,
                                                                 const int32_t* __restrict__ idx,
                                                                 const float2* __restrict__ stats,
                                                                 float* __restrict__ scores,
                                                                 int* __restrict__ counts)
{
    static_assert(FUSE || !STD, "standardized scores only with the fused epilogue");
    extern __shared__ __align__(16) unsigned char smem[];
    const int KP = P.active[l - 1], KC = P.cpt[l], D = P.delta[l], nchunk = P.nchunk, d = P.d, dp = P.dp;
    const int csh = P.cpt_shift[l];   // KC = 2^csh
    const int TT = kWideCols >> csh;
    const int64_t tb = (int64_t)blockIdx.x * TT;
    const int nt_tok = (int)min((int64_t)TT, ntok - tb);
    uint32_t* s_gb = (uint32_t*)smem;   // row stride cws (odd): the 16 rows of a fragment on 16 banks
    unsigned char* p1 = smem + align16u(P.gpad[l] * P.cws * 4);
    uint32_t* pairs = (uint32_t*)p1;
    float* xf = (float*)p1;
    uint32_t* cw = (uint32_t*)(p1 + align16u(TT * (X_BF16 ? P.prow : dp) * 4));
    int32_t* s_pidx = (int32_t*)((unsigned char*)cw + align16u(kWideCols * P.cws * 4));   // parent of each column
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

    {   // generator bitmaps: already in the LDS layout (row stride cws), 16-byte copies
        const u32x4* gsrc = (const u32x4*)(P.gbits + P.gbits_off[l]);
        u32x4* gdst = (u32x4*)s_gb;
        for (int i = threadIdx.x; i < P.gpad[l] * P.cws / 4; i += kWideThreads) gdst[i] = gsrc[i];
    }
    for (int tt = wave; tt < TT; tt += 4) {
        if constexpr (X_BF16) {
            load_pairs(P, lane, tt < nt_tok ? 1 : 0, 1, (const uint16_t*)xin, t0 + tb + tt, pairs + tt * P.prow);
        } else {
            const float* xs = (const float*)xin;
            for (int iota = lane; iota < dp; iota += 64)
                xf[tt * dp + iota] = (tt < nt_tok && iota < d) ? xs[(t0 + tb + tt) * d + iota] : 0.f;
        }
    }
    // parents' sign bitmaps: one nibble-table word per 4-bit group of the index;
    // lanes take consecutive columns of one word, so a table read touches one
    // 64-byte row of the table
    {
        const int col = threadIdx.x & (kWideCols - 1), tt = col >> csh, q = col & (KC - 1);
        const int32_t p = (tt < nt_tok && q < KP) ? idx[(t0 + tb + tt) * P.k_tot + P.slot_base[l - 1] + q] : -1;
        if (threadIdx.x < kWideCols) s_pidx[col] = p;
        // the loads of a word are independent and wait once; only the index's
        // own groups are read, two folded per instruction
        const uint32_t pu = p >= 0 ? (uint32_t)p : 0u;
        const unsigned char* ntb = (const unsigned char*)P.nt;
        auto words = [&](auto groups) {
            constexpr int NG = groups.value;
            uint32_t toff[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) toff[g] = 4u * ((uint32_t)(g * nchunk * 16) + ((pu >> (4 * g)) & 15u));
#pragma unroll 4
            for (int w = threadIdx.x / kWideCols; w < nchunk; w += kWideThreads / kWideCols) {
                uint32_t t[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) t[g] = *(const uint32_t*)(ntb + toff[g] + (uint32_t)w * 64u);
                uint32_t word = __builtin_amdgcn_bitop3_b32(t[0], t[1], t[2], 0x96);
#pragma unroll
                for (int g = 3; g + 1 < NG; g += 2) word = __builtin_amdgcn_bitop3_b32(word, t[g], t[g + 1], 0x96);
                if constexpr (NG % 2 == 0) word ^= t[NG - 1];
                cw[col * P.cws + w] = p >= 0 ? word : 0u;
            }
        };
        if (P.nt_groups <= 3) words(std::integral_constant<int, 3>{});
        else if (P.nt_groups == 4) words(std::integral_constant<int, 4>{});
        else if (P.nt_groups == 5) words(std::integral_constant<int, 5>{});
        else words(std::integral_constant<int, kNtGroupsPadded>{});
    }
    __syncthreads();

    const int wr = wave >> 1, wc = wave & 1, c16 = lane & 15, kq = lane >> 4;
    f32x4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[mt][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int rowbase = wr * 16 * MT + c16;
    int bcol[4], btok[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        bcol[n] = wc * 64 + n * 16 + c16;
        btok[n] = bcol[n] >> csh;
    }
    // the LDS words of chunk c + 1 are requested before chunk c is computed
    // (two register sets, used in turn)
    struct Words {
        uint32_t a[MT], b[4];
    };
    auto fetch = [&](int c, Words& W) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) W.a[mt] = s_gb[(rowbase + 16 * mt) * P.cws + c];
#pragma unroll
        for (int n = 0; n < 4; ++n) W.b[n] = cw[bcol[n] * P.cws + c];
    };
    // A dword i: bf16 +-1 pair with the signs at coordinates 4kq + i and 16 + 4kq + i of the chunk
    auto afrag = [&](uint32_t w) -> bf16x8 {
        const uint32_t R = rotl32(w, 15u - 4u * (uint32_t)kq);
        u32x4 a;
        a.x = __builtin_amdgcn_bitop3_b32(R, 0x80008000u, 0x3F803F80u, 0xEA);   // (R & M) | one
        a.y = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_alignbit(R, R, 1), 0x80008000u, 0x3F803F80u, 0xEA);
        a.z = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_alignbit(R, R, 2), 0x80008000u, 0x3F803F80u, 0xEA);
        a.w = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_alignbit(R, R, 3), 0x80008000u, 0x3F803F80u, 0xEA);
        return __builtin_bit_cast(bf16x8, a);
    };
    auto compute = [&](int c, const Words& W) {
        // fp32 activations: each value split exactly into three bf16 terms
        u32x4 bh[4], bm[4], bl[4];
#pragma unroll
        for (int n = 0; n < 4; ++n)
            split_column(xf + btok[n] * dp + 32 * c + 4 * kq, rotl32(W.b[n], 15u - 4u * (uint32_t)kq), bh[n], bm[n], bl[n]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const bf16x8 av = afrag(W.a[mt]);
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                acc[mt][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bh[n]),
                                                                     acc[mt][n], 0, 0, 0);
                acc[mt][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bm[n]),
                                                                     acc[mt][n], 0, 0, 0);
                acc[mt][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, bl[n]),
                                                                     acc[mt][n], 0, 0, 0);
            }
        }
    };
    if constexpr (X_BF16) {
        // Vector instructions and matrix products of the k-loop are balanced
        // (96 of 4 cycles against 32 of 16 per chunk at MT = 8), so they have
        // to overlap within a wave: behind every product (mt, n) of chunk c
        // stand two of the eight instructions that build the next row operand
        // and its share of those that build the column operands of chunk
        // c + 1, and the LDS words of chunk c + 2 are requested as the words
        // they replace are used up.  The order is pinned: left alone, the
        // compiler builds each operand in one piece between products.
        constexpr int NS = 4 * MT, BPS = 32 / NS;   // slots per chunk, column instructions per slot
        u32x4 pd[4], bf[2][4], av[2];
        uint32_t bw[4], aw[2][MT], RB, RA, tb, ta;
        const int rot = 15 - 4 * kq;
        auto fetch_col = [&](int c, int n) {
            bw[n] = cw[bcol[n] * P.cws + c];
            pd[n] = *(const u32x4*)(pairs + btok[n] * P.prow + c * 16 + kq * 4);
        };
        auto fetch_row = [&](int c, int mt, uint32_t (&a)[MT]) { a[mt] = s_gb[(rowbase + 16 * mt) * P.cws + c]; };
        // instruction k of the eight that build a column operand (of sign word
        // w and pairs p), and two (k = 0..3) of the eight of a row operand
        auto col_op = [&](int k, uint32_t w, const u32x4& p, u32x4& o) {
            switch (k) {
            case 0: RB = rotl32(w, (uint32_t)rot); break;
            case 1: o.x = p.x ^ (RB & 0x80008000u); break;
            case 2: tb = __builtin_amdgcn_alignbit(RB, RB, 1); break;
            case 3: o.y = p.y ^ (tb & 0x80008000u); break;
            case 4: tb = __builtin_amdgcn_alignbit(RB, RB, 2); break;
            case 5: o.z = p.z ^ (tb & 0x80008000u); break;
            case 6: tb = __builtin_amdgcn_alignbit(RB, RB, 3); break;
            default: o.w = p.w ^ (tb & 0x80008000u); break;
            }
        };
        auto row_op = [&](int k, uint32_t w, u32x4& o) {
            if (k == 0) RA = rotl32(w, (uint32_t)rot);
            ta = k == 0 ? RA : __builtin_amdgcn_alignbit(RA, RA, k);
            const uint32_t u = __builtin_amdgcn_bitop3_b32(ta, 0x80008000u, 0x3F803F80u, 0xEA);   // (R & M) | one
            if (k == 0) o.x = u;
            else if (k == 1) o.y = u;
            else if (k == 2) o.z = u;
            else o.w = u;
        };
        // one chunk: cur = its column operands, a = its row words, an = those
        // of the next chunk (its first row operand is built here)
        auto chunk = [&](int c, u32x4 (&cur)[4], u32x4 (&next)[4], uint32_t (&a)[MT], uint32_t (&an)[MT]) {
            const int cf = c + 2;   // past the last chunk: words of the next row, never used
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    acc[mt][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, av[mt & 1]), __builtin_bit_cast(bf16x8, cur[n]), acc[mt][n], 0, 0, 0);
                    // the row operand is done two slots before it is used
                    const uint32_t w = mt + 1 < MT ? a[mt + 1 < MT ? mt + 1 : 0] : an[0];
                    if (n == 0) row_op(0, w, av[(mt + 1) & 1]);
                    if (n < 3) row_op(n + 1, w, av[(mt + 1) & 1]);
                    const int first = n == 0 ? 0 : n - 1, count = n == 0 ? 0 : n == 3 ? 2 : 1;   // of the tile's four shares
#pragma unroll
                    for (int u = 0; u < 2 * BPS; ++u) {
                        const int k = (4 * mt + first) * BPS + u;
                        if (u < count * BPS) {
                            col_op(k & 7, bw[k >> 3], pd[k >> 3], next[k >> 3]);
                            if ((k & 7) == 7) fetch_col(cf, k >> 3);
                        }
                    }
                    if (n == 3) fetch_row(cf, mt, a);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if constexpr (MT & 1) av[0] = av[1];
        };
#pragma unroll
        for (int n = 0; n < 4; ++n) fetch_col(0, n);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            fetch_row(0, mt, aw[0]);
            fetch_row(min(1, nchunk - 1), mt, aw[1]);
        }
#pragma unroll
        for (int n = 0; n < 4; ++n) {
#pragma unroll
            for (int k = 0; k < 8; ++k) col_op(k, bw[n], pd[n], bf[0][n]);
            fetch_col(min(1, nchunk - 1), n);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) row_op(k, aw[0][0], av[0]);
        int c = 0;
        for (; c + 1 < nchunk; c += 2) {
            chunk(c, bf[0], bf[1], aw[0], aw[1]);
            chunk(c + 1, bf[1], bf[0], aw[1], aw[0]);
        }
        if (c < nchunk) chunk(c, bf[0], bf[1], aw[0], aw[1]);
    } else {
        Words w0, w1;
        fetch(0, w0);
        for (int c = 0; c < nchunk; c += 2) {
            if (c + 1 < nchunk) fetch(c + 1, w1);
            compute(c, w0);
            if (c + 2 < nchunk) fetch(c + 2, w0);
            if (c + 1 < nchunk) compute(c + 1, w1);
        }
    }
    // scores (times 1/sqrt d; standardized in place already with STD) of the
    // live (token, parent) columns and generator rows
    const bool all_rows = 32 * MT == D;   // else rows from D on are padding
    const float osc = STD ? 1.f : P.rsd;
    auto store_scores = [&](int n) {
        const int col = wc * 64 + n * 16 + c16, tt = col >> csh, q = col & (KC - 1);
        if (tt >= nt_tok || q >= KP) return;
        float* dst = scores + ((tb + tt) * KP + q) * D + wr * 16 * MT + 4 * kq;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (all_rows || wr * 16 * MT + 16 * mt + 4 * kq < D) {
                const f32x4 v = acc[mt][n];
                *(float4*)(dst + 16 * mt) = make_float4(v[0] * osc, v[1] * osc, v[2] * osc, v[3] * osc);
            }
        }
    };
    if constexpr (!FUSE) {
#pragma unroll
        for (int n = 0; n < 4; ++n) store_scores(n);
    } else {
        const int K = P.active[l], x32 = (lane ^ 32) << 2;
        const int tpw = 64 >> csh;   // tokens in a wave's 64 columns: 4, 2 or 1
        int32_t pid[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) pid[n] = s_pidx[bcol[n]];
        __syncthreads();   // the staging LDS is free from here on
        // with standardization z = (s - mu) r in place (s = acc / sqrt d), the
        // statistics of child p XOR g_row gathered at an index that is always a
        // feature (generator of a clamped row, parent 0 for padding columns)
        if constexpr (STD) {
            const uint32_t* gl = P.gens + P.gens_off[l];
            uint32_t gv[MT][4];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) gv[mt][i] = gl[min(wr * 16 * MT + 16 * mt + 4 * kq + i, D - 1)];
            // a batch is one row tile against the four column tiles: its
            // generators are neighbours in value
            uint32_t pu[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) pu[n] = pid[n] >= 0 ? (uint32_t)pid[n] : 0u;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float2 st[4][4];
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i) st[n][i] = stats[pu[n] ^ gv[mt][i]];
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[mt][n][i] = (acc[mt][n][i] * P.rsd - st[n][i].x) * st[n][i].y;
            }
        }
        // The threshold and the hits are taken on |acc|: plain scores are
        // scaled only where they are written (a multiplication by 1/sqrt d per
        // value, and a magnitude key of it, were a third of this epilogue).
        // Padding rows count as 0, whole padding columns as no candidates.
        if (!all_rows) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool pad = wr * 16 * MT + 16 * mt + 4 * kq + i >= D;
#pragma unroll
                    for (int n = 0; n < 4; ++n) acc[mt][n][i] = pad ? 0.f : acc[mt][n][i];
                }
        }
        uint32_t* s_top = (uint32_t*)smem;             // [TT][2 row halves][64 lanes]
        float* s_tau = (float*)(s_top + TT * 128);     // [TT]
        int* s_cnt = (int*)(s_tau + TT);              // [TT]
        // each lane's largest magnitude per column tile, two values an
        // instruction (a NaN stays one), then per token of this wave
        uint32_t top[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            float m = 0.f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const f32x4 v = acc[mt][n];
                m = max3_abs(m, v[0], v[1]);
                m = max3_abs(m, v[2], v[3]);
            }
            top[n] = pid[n] >= 0 ? __float_as_uint(m) & 0x7FFFFFFFu : 0u;
        }
        uint32_t* tp = s_top + (((wc * 64) >> csh) * 2 + wr) * 64 + lane;   // 128 words from token to token
        if (tpw == 4) {
#pragma unroll
            for (int n = 0; n < 4; ++n) tp[n * 128] = top[n];
        } else if (tpw == 2) {
            tp[0] = max(top[0], top[1]);
            tp[128] = max(top[2], top[3]);
        } else {
            tp[0] = max(max(top[0], top[1]), max(top[2], top[3]));
        }
        if ((int)threadIdx.x < TT) s_cnt[threadIdx.x] = 0;
        __syncthreads();
        // tau of each token: the K-th largest distinct magnitude among its 128
        // lane maxima.  Four units in the last place below it are listed too,
        // so that unequal |acc| that the scaling rounds to one magnitude stay
        // together (the smaller index wins among them).  Fewer than K distinct
        // maxima, a NaN, or magnitudes so small that the scaled ones lose
        // bits list everything.
        for (int tt = wave; tt < TT; tt += 4) {
            uint32_t v[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) v[r] = s_top[tt * 128 + lane * 2 + r];
            sort_desc<2, 6, false>(v, lane, x32);
            uint32_t prev = (uint32_t)__shfl((int)v[1], (lane + 63) & 63, 64);
            if (lane == 0) prev = 0u;
            const bool k0 = v[0] != 0u && v[0] != prev, k1 = v[1] != 0u && v[1] != v[0];
            const uint64_t b0 = __ballot(k0), b1 = __ballot(k1);
            const int rank = lanes_below(b0) + lanes_below(b1);
            const uint64_t h0 = __ballot(k0 && rank == K - 1), h1 = __ballot(k1 && rank + (int)k0 == K - 1);
            uint32_t tau = 0u;
            if (h0) tau = (uint32_t)__builtin_amdgcn_readlane((int)v[0], __builtin_ctzll(h0));
            else if (h1) tau = (uint32_t)__builtin_amdgcn_readlane((int)v[1], __builtin_ctzll(h1));
            const uint32_t most = (uint32_t)__builtin_amdgcn_readfirstlane((int)v[0]);
            constexpr uint32_t kSmall = 0x0D800000u;   // 2^-100
            tau = (most > 0x7F800000u || tau < kSmall) ? 0u : tau - 4u;
            if (lane == 0) s_tau[tt] = __uint_as_float(tau);
        }
        __syncthreads();
        // list the candidates at or above tau in the token's region: a bit
        // per value says which are listed (two instructions each), one LDS
        // atomic per lane with hits reserves their places (the order of the
        // list is of no account), and a tile's values go through the wave's LDS
        // rows so that each lane visits only its hits
        float* zrow = (float*)(smem + kWideEpiZ) + (wave * 64 + lane) * (4 * MT + 4);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int tt = bcol[n] >> csh, q = bcol[n] & (KC - 1);
            const float tau = s_tau[tt];
            uint64_t* lst = (uint64_t*)(scores + (tb + tt) * KP * D);
            uint32_t hm = 0u;   // bit 4 MT - 1 - (4 mt + i): value (mt, i) is listed
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) hm = shift_in_not_less(hm, acc[mt][n], tau);
            if (!all_rows) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (wr * 16 * MT + 16 * mt + 4 * kq + i >= D) hm &= ~(1u << (4 * MT - 1 - (4 * mt + i)));
            }
            if (pid[n] < 0) hm = 0u;
            if (!__ballot(hm != 0u)) continue;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const f32x4 v = acc[mt][n];
                *(float4*)(zrow + 4 * mt) = make_float4(v[0], v[1], v[2], v[3]);
            }
            int pos = hm ? atomicAdd(&s_cnt[tt], (int)__popc(hm)) : 0;
            const uint32_t f0 = (uint32_t)(q * D + wr * 16 * MT + 4 * kq);
            while (hm) {
                const int b = 4 * MT - 1 - (31 - __builtin_clz(hm));
                hm &= ~(0x80000000u >> __builtin_clz(hm));
                const uint32_t f = f0 + 16u * (uint32_t)(b >> 2) + (uint32_t)(b & 3);
                if (pos < kWideList) lst[pos] = ((uint64_t)f << 32) | __float_as_uint(zrow[b] * osc);
                ++pos;
            }
        }
        __syncthreads();
        // a token with too many entries gets its full scores instead
#pragma unroll
        for (int n = 0; n < 4; ++n)
            if (s_cnt[bcol[n] >> csh] > kWideList) store_scores(n);
        if ((int)threadIdx.x < nt_tok) counts[tb + threadIdx.x] = s_cnt[threadIdx.x];
    }
}

// Sorts the n <= 64 R keys of the list (0-padded) and emits the first K
// distinct ones of the token into slots [sb, sb + K); returns how many.
template <int R>
__device__ __forceinline__ int wide_emit(const DevPlan& P, const uint64_t* lst, int n, int K, int lane, int x32,
                                         int64_t t, int sb, int32_t* out_idx, float* out_coef)
{
    uint64_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = lane * R + r;
        v[r] = e < n ? lst[e] : 0ull;
    }
    sort_desc<R, 6, false>(v, lane, x32);
    uint64_t prev = shfl_u64(v[R - 1], (lane + 63) & 63);
    if (lane == 0) prev = 0ull;
    int kept = 0, cnt = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool k = v[r] != 0ull && v[r] != prev;
        kept |= (int)k << r;
        cnt += (int)k;
        prev = v[r];
    }
    int total = 0;
    int rank = wave_prefix5(cnt, lane, total);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (((kept >> r) & 1) && rank < K) {
            out_idx[t * P.k_tot + sb + rank] = (int32_t)key_index(v[r]);
            out_coef[t * P.k_tot + sb + rank] = key_value(v[r]);
        }
        rank += (kept >> r) & 1;
    }
    return total;
}

// counts (plain scores only): the GEMM listed counts[t - t0] <= kWideList
// (candidate, z) entries at or above the threshold in the token's region; more
// means the region holds the full scores.  Without counts the region always
// holds the full scores.
template <bool STD>
__global__ __launch_bounds__(kWideThreads) void wide_select_kernel(DevPlan P, int l, int64_t t0, int64_t ntok,
                                                                   const float* __restrict__ scores,
                                                                   const int* __restrict__ counts,
                                                                   const float2* __restrict__ stats,
                                                                   int32_t* __restrict__ out_idx,
                                                                   float* __restrict__ out_coef)
{
    __shared__ uint64_t s_list[4][64 * kSegStride];
    __shared__ int32_t s_par[4][128];
    __shared__ uint32_t s_gen[256];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, x32 = (lane ^ 32) << 2;
    const int KP = P.active[l - 1], D = P.delta[l], K = P.active[l], n = KP * D, sb = P.slot_base[l];
    const int dsh = 31 - __builtin_clz((unsigned)D);
    for (int j = threadIdx.x; j < D; j += kWideThreads) s_gen[j] = P.gens[P.gens_off[l] + j];
    __syncthreads();
    // chunk-relative token (wave-uniform: scalar, so score addresses are 32-bit offsets)
    const int64_t tl = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + wave);
    if (tl >= ntok) return;
    const int64_t t = t0 + tl;
    for (int q = lane; q < KP; q += 64) s_par[wave][q] = out_idx[t * P.k_tot + P.slot_base[l - 1] + q];
    wave_sync();
    // live parent slots as a bit set (padding parents have no children)
    uint64_t live[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int q = 64 * h + lane;
        live[h] = __ballot(q < KP && s_par[wave][q] >= 0);
    }
    const float* src = scores + tl * (int64_t)n;

    // candidate f is child s_gen[f mod D] of parent slot f / D
    auto child_index = [&](int f) -> uint32_t { return (uint32_t)s_par[wave][f >> dsh] ^ s_gen[f & (D - 1)]; };
    auto is_live = [&](int f) -> bool {
        const int q = f >> dsh;
        const uint64_t lw = q < 64 ? live[0] : live[1];
        return f < n && ((lw >> (q & 63)) & 1ull);
    };
    // standardized score of a live candidate
    auto z_of = [&](int f, float v) -> float {
        if constexpr (STD) {
            const float2 st = stats[child_index(f)];
            v = (v - st.x) * st.y;
        }
        return v;
    };
    // magnitude key |z| bits + 1, 0 for padding: distinct values mean distinct children
    auto mkey = [](bool ok, float z) -> uint32_t { return ok ? (__float_as_uint(z) & 0x7FFFFFFFu) + 1u : 0u; };
    // this lane's candidates are streamed from the workspace eight at a time
    // (unconditional, clamped loads: one wait per round)
    constexpr int B = 8;
    const int rounds = (n + 64 * B - 1) / (64 * B);
    auto load_round = [&](int rd, float (&v)[B]) {
#pragma unroll
        for (int b = 0; b < B; ++b)
            v[b] = *(const float*)((const char*)src + 4u * (uint32_t)min((rd * B + b) * 64 + lane, n - 1));
    };

    uint64_t* lst = s_list[wave];
    int nl = kWideList + 1;
    const int listed = counts ? counts[tl] : kWideList + 1;
    if (listed <= kWideList) {
        // the GEMM's list: full keys of its entries
        const uint64_t* ent = (const uint64_t*)src;
        for (int e = lane; e < listed; e += 64) {
            const uint64_t en = ent[e];
            lst[e] = make_sort_key(__uint_as_float((uint32_t)en), child_index((int)(en >> 32)));
        }
        wave_sync();
        nl = listed;
    } else {
        // threshold tau: the K-th largest distinct magnitude key among the lanes'
        // top two.  At least K distinct children have mkey >= tau, so the top K
        // distinct (|z|, index) keys are all among the candidates with mkey >= tau.
        uint32_t top0 = 0u, top1 = 0u;
        for (int rd = 0; rd < rounds; ++rd) {
            float v[B];
            load_round(rd, v);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int f = (rd * B + b) * 64 + lane;
                const bool ok = is_live(f);
                const uint32_t m = mkey(ok, ok ? z_of(f, v[b]) : 0.f);
                const bool gt0 = m > top0, gt1 = m > top1 && m != top0;
                top1 = gt0 ? top0 : (gt1 ? m : top1);
                top0 = gt0 ? m : top0;
            }
        }
        constexpr int M = 2;
        uint32_t top[M] = {top0, top1};
        sort_desc<M, 6, false>(top, lane, x32);
        uint32_t prev = (uint32_t)__shfl((int)top[M - 1], (lane + 63) & 63, 64);
        if (lane == 0) prev = 0u;
        int kept = 0, cnt = 0;
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const bool kk = top[r] != 0u && top[r] != prev;
            kept |= (int)kk << r;
            cnt += (int)kk;
            prev = top[r];
        }
        int total = 0;
        int rank = wave_prefix5(cnt, lane, total);
        uint32_t tau_l = 0u;
#pragma unroll
        for (int r = 0; r < M; ++r) {
            if (((kept >> r) & 1) && rank == K - 1) tau_l = top[r];
            rank += (kept >> r) & 1;
        }
        // one lane holds tau when at least K distinct magnitudes were seen; else take every live candidate
        uint32_t tau = 1u;
        const uint64_t hb = __ballot(tau_l != 0u);
        if (hb) tau = (uint32_t)__shfl((int)tau_l, __builtin_ctzll(hb), 64);

        // collect (f, z) of the candidates with mkey >= tau: each lane appends to
        // its own segment of kSeg entries (every candidate is stored, at the
        // lane's next free entry, so the pass has no branches and no cross-lane
        // steps; entry kSeg takes what does not fit).  The segments are then
        // packed into one list of full keys.  A lane with more than kSeg hits
        // sends the token to the exact extraction below.
        int mine_n = 0;
        for (int rd = 0; rd < rounds; ++rd) {
            float v[B];
            load_round(rd, v);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int f = (rd * B + b) * 64 + lane;
                const bool ok = is_live(f);
                const float z = ok ? z_of(f, v[b]) : 0.f;
                lst[lane * kSegStride + min(mine_n, kSeg)] = ((uint64_t)(uint32_t)f << 32) | __float_as_uint(z);
                mine_n += (int)(mkey(ok, z) >= tau);
            }
        }
        wave_sync();
        if (!__ballot(mine_n > kSeg)) {
            uint64_t mine[kSeg];
#pragma unroll
            for (int j = 0; j < kSeg; ++j) {
                mine[j] = 0ull;
                if (j < mine_n) {
                    const uint64_t en = lst[lane * kSegStride + j];
                    mine[j] = make_sort_key(__uint_as_float((uint32_t)en), child_index((int)(en >> 32)));
                }
            }
            const int pre = wave_prefix5(mine_n, lane, nl);
            wave_sync();
#pragma unroll
            for (int j = 0; j < kSeg; ++j)
                if (j < mine_n) lst[pre + j] = mine[j];
        }
        wave_sync();
    }
    int emitted;
    if (nl <= 64) emitted = wide_emit<1>(P, lst, nl, K, lane, x32, t, sb, out_idx, out_coef);
    else if (nl <= 128) emitted = wide_emit<2>(P, lst, nl, K, lane, x32, t, sb, out_idx, out_coef);
    else if (nl <= 256) emitted = wide_emit<4>(P, lst, nl, K, lane, x32, t, sb, out_idx, out_coef);
    else if (nl <= 512) emitted = wide_emit<8>(P, lst, nl, K, lane, x32, t, sb, out_idx, out_coef);
    else if (nl <= kWideList) emitted = wide_emit<16>(P, lst, nl, K, lane, x32, t, sb, out_idx, out_coef);
    else {
        // exact extraction: K rounds of the largest key below the previous one
        uint64_t last = ~0ull;
        emitted = 0;
        for (int r = 0; r < K; ++r) {
            uint64_t best = 0ull;
            for (int rd = 0; rd < rounds; ++rd) {
                float v[B];
                load_round(rd, v);
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const int f = (rd * B + b) * 64 + lane;
                    const bool ok = is_live(f);
                    const uint64_t k = ok ? make_sort_key(z_of(f, v[b]), child_index(f)) : 0ull;
                    best = (k < last && k > best) ? k : best;
                }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const uint64_t o = shfl_u64(best, lane ^ off);
                best = o > best ? o : best;
            }
            if (best == 0ull) break;
            if (lane == 0) {
                out_idx[t * P.k_tot + sb + r] = (int32_t)key_index(best);
                out_coef[t * P.k_tot + sb + r] = key_value(best);
            }
            last = best;
            ++emitted;
        }
    }
    for (int r = emitted + lane; r < K; r += 64) {
        out_idx[t * P.k_tot + sb + r] = -1;
        out_coef[t * P.k_tot + sb + r] = 0.f;
    }
}

}  // namespace

// Whether the standardized encoder's workgroup fits the LDS budget.
bool encode2_std_supported(const DevPlan& P)
{
    const size_t lds = enc_shared_bytes(P, true) + (size_t)kEncWaves * enc_layout_least(P, false, false).bytes;
    return encode2_supported(P) && lds <= (size_t)kLdsBudget;
}

bool encode2_supported(const DevPlan& P)
{
    const int TPW = P.wave_tokens, LPT = 64 / TPW;
    if (P.active[0] > LPT || enc_r(P) > 16 || P.d > 65535) return false;
    for (int l = 1; l < P.levels; ++l)
        if (P.cpt[l] > 16 || TPW * P.cpt[l] > 16) return false;
    if (16 / TPW != 4 && 16 / TPW != 8 && 16 / TPW != 16) return false;
    const size_t lds = enc_shared_bytes(P, false) + (size_t)kEncWaves * enc_layout_least(P, false, false).bytes;
    return lds <= (size_t)kLdsBudget;
}

hipError_t launch_encode2(const DevPlan& P, const void* x, bool x_bf16, int64_t T, const float* stats, int32_t* idx,
                          float* coef, hipStream_t stream)
{
    const float2* st = (const float2*)stats;
    const EncLayout EL = enc_layout(P, x_bf16, stats != nullptr);
    const int listn = EL.listn;
    const size_t lds = enc_shared_bytes(P, stats != nullptr) + (size_t)kEncWaves * EL.bytes;
    const int64_t groups = (T + P.wave_tokens - 1) / P.wave_tokens;
    const int64_t need = (groups + kEncWaves - 1) / kEncWaves;
    const int cus = device_cus();
    const int per_cu = (int)std::max<size_t>(1, (160 * 1024) / std::max<size_t>(lds, 1));
    const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(need, (int64_t)cus * std::min(per_cu, 8) * 4)));
    const int R = enc_r(P), CPT = 16 / P.wave_tokens;
#define DPB_ENC(XB, CV, RV)                                                                                        \
    do {                                                                                                           \
        if (st) {                                                                                                  \
            allow_lds(encode3_kernel<XB, CV, RV, true>, lds);                                                      \
            hipLaunchKernelGGL((encode3_kernel<XB, CV, RV, true>), grid, dim3(kEncThreads), lds, stream, P, listn, x, T, \
                               st, idx, coef);                                                                     \
        } else {                                                                                                   \
            allow_lds(encode3_kernel<XB, CV, RV, false>, lds);                                                     \
            hipLaunchKernelGGL((encode3_kernel<XB, CV, RV, false>), grid, dim3(kEncThreads), lds, stream, P, listn, x, T, \
                               st, idx, coef);                                                                     \
        }                                                                                                          \
    } while (0)
#define DPB_ENC_R(XB, CV)                    \
    do {                                     \
        if (R == 4) DPB_ENC(XB, CV, 4);      \
        else if (R == 8) DPB_ENC(XB, CV, 8); \
        else DPB_ENC(XB, CV, 16);            \
    } while (0)
    if (x_bf16) {
        if (CPT == 4) DPB_ENC_R(true, 4);
        else if (CPT == 8) DPB_ENC_R(true, 8);
        else DPB_ENC_R(true, 16);
    } else {
        if (CPT == 4) DPB_ENC_R(false, 4);
        else if (CPT == 8) DPB_ENC_R(false, 8);
        else DPB_ENC_R(false, 16);
    }
#undef DPB_ENC_R
#undef DPB_ENC
    return hipGetLastError();
}

// Tokens per pass of the wide encoder (bounds its workspace).
constexpr int64_t kWideChunkTokens = 16384;

static int wide_max_cands(const DevPlan& P)
{
    int m = 0;
    for (int l = 1; l < P.levels; ++l) m = std::max(m, P.active[l - 1] * P.delta[l]);
    return m;
}

static unsigned wide_level0_lds(const DevPlan& P, bool x_bf16, bool std)
{
    const int ND = (P.dp / 2 + 63) / 64;
    const int listn = P.active[0] * (x_bf16 ? 2 * ND : (P.d + 63) / 64);
    const unsigned per_wave = align16u(x_bf16 ? P.prow * 4 : P.dp * 4) + align16u(listn * 8) +
                              align16u((P.active[0] + 1) * 4) + 16;
    return (std ? align16u(P.d * 8) : 0u) + 4 * per_wave;
}

bool encode_wide_supported(const DevPlan& P, bool x_bf16)
{
    if (P.levels < 2 || P.active[0] > 64 || P.d > 4096) return false;
    if (wide_level0_lds(P, x_bf16, true) > (unsigned)kLdsBudget) return false;
    for (int l = 1; l < P.levels; ++l) {
        const int D = P.delta[l];
        if (D < 16 || D > 256 || (D & (D - 1)) || P.cpt[l] > 128 || P.active[l] > 128) return false;
        if (P.active[l - 1] * D > 64 * 128) return false;
        if (wide_gemm_lds(P, l, x_bf16) > (unsigned)kLdsBudget) return false;
    }
    return true;
}

// Workspace: per chunk token, the scores (or the GEMM's list) of its
// candidates, then one count per chunk token.
static size_t wide_scores_bytes(const DevPlan& P, int64_t ch)
{
    return ((size_t)ch * wide_max_cands(P) * 4 + 255) & ~(size_t)255;
}

static size_t wide_chunk_bytes(const DevPlan& P, int64_t ch)
{
    return ch > 0 ? wide_scores_bytes(P, ch) + (((size_t)ch * 4 + 255) & ~(size_t)255) : 0;
}

size_t encode_wide_workspace_bytes(const DevPlan& P, int64_t T)
{
    return wide_chunk_bytes(P, std::min<int64_t>(T, kWideChunkTokens));
}

// counts != nullptr: the fused epilogue (lists instead of scores); STD: it
// standardizes the scores with `st`.
template <bool XB, bool FUSE, bool STD>
static void launch_wide_gemm(const DevPlan& P, int l, const void* x, int64_t c0, int64_t nc, const int32_t* idx,
                             const float2* st, float* scores, int* counts, hipStream_t stream)
{
    const int TT = kWideCols / P.cpt[l];
    const dim3 grid((unsigned)((nc + TT - 1) / TT));
    const size_t lds = wide_gemm_lds(P, l, XB);
    const int MT = std::max(32, P.delta[l]) / 32;
#define DPB_WG(M)                                                                                             \
    do {                                                                                                      \
        allow_lds(wide_gemm_kernel<XB, M, FUSE, STD>, lds);                                                   \
        hipLaunchKernelGGL((wide_gemm_kernel<XB, M, FUSE, STD>), grid, dim3(kWideThreads), lds, stream, P, l, x, c0, \
                           nc, idx, st, scores, counts);                                                      \
    } while (0)
    if (MT == 1) DPB_WG(1);
    else if (MT == 2) DPB_WG(2);
    else if (MT == 4) DPB_WG(4);
    else DPB_WG(8);
#undef DPB_WG
}

template <bool STD>
static void launch_wide_select(const DevPlan& P, int l, int64_t c0, int64_t nc, const float* scores,
                               const int* counts, const float2* st, int32_t* idx, float* coef, hipStream_t stream)
{
    const dim3 grid((unsigned)((nc + 3) / 4));
    hipLaunchKernelGGL((wide_select_kernel<STD>), grid, dim3(kWideThreads), 0, stream, P, l, c0, nc, scores, counts,
                       st, idx, coef);
}

hipError_t launch_encode_wide(const DevPlan& P, const void* x, bool x_bf16, int64_t T, const float* stats,
                              int32_t* idx, float* coef, void* ws, hipStream_t stream, int64_t chunk)
{
    const float2* st = (const float2*)stats;
    {
        const int cus = device_cus();
        const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>((T + 3) / 4, (int64_t)cus * 8)));
        const size_t lds = wide_level0_lds(P, x_bf16, st != nullptr);
#define DPB_W0(XB, SD)                                                                                        \
    do {                                                                                                      \
        allow_lds(wide_level0_kernel<XB, SD>, lds);                                                           \
        hipLaunchKernelGGL((wide_level0_kernel<XB, SD>), grid, dim3(kWideThreads), lds, stream, P, x, T, st, idx, \
                           coef);                                                                             \
    } while (0)
        if (x_bf16 && st) DPB_W0(true, true);
        else if (x_bf16) DPB_W0(true, false);
        else if (st) DPB_W0(false, true);
        else DPB_W0(false, false);
#undef DPB_W0
    }
    float* scores = (float*)ws;
    if (chunk <= 0) chunk = kWideChunkTokens;
    int* counts = (int*)((char*)ws + wide_scores_bytes(P, std::min<int64_t>(T, chunk)));
    for (int64_t c0 = 0; c0 < T; c0 += chunk) {
        const int64_t nc = std::min<int64_t>(chunk, T - c0);
        for (int l = 1; l < P.levels; ++l) {
            // the fused epilogue standardizes in place (its lists and scores hold z);
            // otherwise the selection standardizes the full scores
            const bool fuse = wide_fused(P, l);
            if (fuse) {
                if (x_bf16 && st) launch_wide_gemm<true, true, true>(P, l, x, c0, nc, idx, st, scores, counts, stream);
                else if (x_bf16) launch_wide_gemm<true, true, false>(P, l, x, c0, nc, idx, st, scores, counts, stream);
                else if (st) launch_wide_gemm<false, true, true>(P, l, x, c0, nc, idx, st, scores, counts, stream);
                else launch_wide_gemm<false, true, false>(P, l, x, c0, nc, idx, st, scores, counts, stream);
                launch_wide_select<false>(P, l, c0, nc, scores, counts, nullptr, idx, coef, stream);
            } else {
                if (x_bf16) launch_wide_gemm<true, false, false>(P, l, x, c0, nc, idx, st, scores, nullptr, stream);
                else launch_wide_gemm<false, false, false>(P, l, x, c0, nc, idx, st, scores, nullptr, stream);
                if (st) launch_wide_select<true>(P, l, c0, nc, scores, nullptr, st, idx, coef, stream);
                else launch_wide_select<false>(P, l, c0, nc, scores, nullptr, st, idx, coef, stream);
            }
        }
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Encoder workspace without allocation: the wide encoder's scratch taken from
// a file-scope device array instead of a caller's buffer.  Each device holds
// its own copy; its address is looked up once per device with that device
// current (scratch_setup) and passed to the kernels like a workspace.  Tokens
// go through in passes sized to the array.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxScratchDevices] = {};
}  // namespace

void* scratch_setup(int device)
{
    if (device < 0 || device >= kMaxScratchDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch[device]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) == hipSuccess) g_scratch[device] = ptr;
        else (void)hipGetLastError();
    }
    return g_scratch[device];
}

int64_t static_chunk_tokens(const DevPlan& P)
{
    // the largest pass (a multiple of 256 tokens, at most the usual chunk) whose workspace fits
    int64_t ch = kWideChunkTokens;
    while (ch >= kStaticMinChunk && wide_chunk_bytes(P, ch) > kStaticScratchBytes) ch -= 256;
    return ch >= kStaticMinChunk ? ch : 0;
}

}  // namespace dpb
