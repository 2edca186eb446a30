// Column decode: y = sum_s coef_s phi_{c_s} for codes of at most 254 slots, the
// last level through parent columns where the plan has them, straight from
// registers to the output rows.
//
// A wave takes TPW = 16 / CPT tokens (CPT parent columns per token, a power
// of two); each token owns LPT = 64 / TPW lanes, and a lane owns the
// coordinate pair 2 LPT m + 2 (lane mod LPT) + {0, 1} in step m.  In a step
// the lane
//  * folds one word U per coordinate, bit b = parity(M_iota & x_b) for the 32
//    listed indices x_b of its token (App. A.4, packed-parity equation: parity
//    is linear in the row mask, so U is the XOR of one table row per 4-bit
//    group of M_iota);
//  * sums the listed coefficients from 16-entry tables of signed sums, four
//    slots at a time;
//  * takes Gamma^T alpha of the last level's columns from 16x16x16 bf16 MFMAs
//    (alpha split into two bf16 terms for bf16 output, exactly into three for
//    fp32); the accumulator starts at the parents' own coefficients, since
//    phi~_p (.) (a_p + Gamma^T alpha_p) is the parent slot and its children
//    together (§2.2 factorization equation);
//  * multiplies its four columns by the parents' signs, +-1 as fp16 halves
//    (v_fma_mix_f32: sign and sum in one instruction; +-1 is exact), and sums
//    the columns of a token across lanes with the row-swap permutes, which
//    leave each lane the sums of its own coordinates;
//  * writes the pair.
// Vector issue and LDS latency bound it.  Nothing of the row goes through LDS,
// so a wave holds 7 KB (d 768, k 96) instead of 11.5 and the kernels are held
// to 128 registers: four waves per SIMD instead of three, and a quarter fewer
// vector instructions.  Measured against the row-in-LDS decode
// it replaced here: 65,536 tokens d 768 k 96: 195 -> 137 us; 16,384 tokens
// d 1024 k 144: 211 -> 87 us; 8,192 tokens d 768 k 56: 33 -> 19 us; the
// backward 367 -> 304, 285 -> 191 and 55 -> 37 us.  (Five waves per SIMD
// measured slower, 157 us; the groups no longer divide evenly.)
// The bits of U that carry parents sit in the low nibbles of the two
// half-words, parent 2i at bit i and parent 2i + 1 at bit 16 + i: one shift
// brings the signs of two parents to bits 15 and 31.
//
// Basis slots mark their coordinate in a byte map; the lane that owns a marked
// coordinate adds the slot's coefficient before it writes.  Hashed slots
// that fit nowhere else (a leaf that routes to no parent, a hashed index in a
// level-0 slot: codes the encoder does not produce) are added one by one up
// to sixteen a token, through the tables beyond (col_pass).
#pragma once

#include <algorithm>
#include <type_traits>

#include "backward.hpp"

namespace dpb {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Everything the column decode needs of a plan, passed by value.
struct ColPlan {
    int d, dp;
    int steps;             // coordinate steps: ceil(dp / (2 LPT))
    int mstride;           // bytes of marks per token: 2 LPT steps
    int k;                 // code width
    int K0;                // level-0 slots
    int KP, sbP;           // leaf parents: count, first slot
    int KL, sbL;           // leaf slots: count, first slot
    int ss, ns;            // summed slots (levels 1 .. L - 3): first, count
    int words;             // words of 32 listed indices per token
    float rsd;
    uint32_t hmask;        // generator hash of the last level: h(x) = (x ^ (x >> hshift)) & hmask
    int hshift;
    const uint32_t* gtab;  // its hmask + 1 pairs (g_j, j)
    const uint32_t* masks; // [dp] row masks
    const void* gamma_t;   // [dp / 16][64] x 4 bf16 (leaf level)
};

constexpr int kColWaves = 4;
constexpr int kColThreads = 64 * kColWaves;
// Waves per SIMD the kernels are held to by registers.  (The decode to fp32
// with sixteen columns and more than 24 index bits keeps four of its registers
// in scratch for it; with three waves, 16,381 tokens d 1024 N 2^28 103 -> 109 us.)
constexpr int col_decode_waves(int cpt) { return cpt ? 4 : 8; }
constexpr int col_bwd_waves(int cpt, bool g_bf16) { return cpt == 0 && g_bf16 ? 5 : 4; }   // (five in fp32: 60 us for 53)
constexpr int kColMaxSlots = 254;   // a mark holds slot + 1 in a byte

// CPT = 0: a plan without leaf columns.  One token per wave, every hashed slot
// is summed through the tables, and the matrix cores take no part in a step.
// Against the row-in-LDS kernels, us: decode of 16,384 tokens pt_small_3l
// 93 -> 76, 8,192 tokens pt_large_2l 58 -> 36, 20,000 tokens d 64 k 48
// 37 -> 15; backward 236 -> 177, 109 -> 82, and 20,000 tokens d 256 k 64
// 98 -> 52.
// Nibbles of each half-word of word 0 that hold parent bits, and the listed
// indices that leaves.
__host__ __device__ constexpr int col_parent_nibbles(int cpt) { return cpt == 16 ? 2 : cpt ? 1 : 0; }
__host__ __device__ constexpr int col_word0_slots(int cpt) { return 32 - 8 * col_parent_nibbles(cpt); }
__host__ __device__ constexpr int col_tpw(int cpt) { return cpt ? 16 / cpt : 1; }

// LDS of a column wave (byte offsets inside its region).  `act` is the first
// byte of a region of act_bytes that the caller uses before the decode (the
// backward's gradient rows); tables, marks and lists live there too.
struct ColLayout {
    unsigned idx, coef, route, par, pc, tab, scr, xs, bas, mark, act, bytes;
};

// act_bytes != 0 (the backward) also reserves the slots' routes.
__host__ __device__ inline ColLayout col_layout(const ColPlan& C, int cpt, unsigned act_bytes)
{
    const int tpw = col_tpw(cpt);
    ColLayout L;
    unsigned off = 0;
    L.act = off;
    L.tab = off;  off += (unsigned)(tpw * C.words) * 1024u;      // 256-byte aligned; alpha uses its first 1 KB
    L.scr = off;  off += 512u;
    L.xs = off;   off = align16u(off + (unsigned)(tpw * C.k) * 2u);
    L.bas = off;  off = align16u(off + (unsigned)(tpw * (C.k + 1)) * 4u);
    L.mark = off; off = align16u(off + (unsigned)(tpw * C.mstride));
    if (off < act_bytes) off = align16u(act_bytes);
    L.idx = off;  off = align16u(off + (unsigned)(tpw * C.k) * 4u);
    L.coef = off; off = align16u(off + (unsigned)(tpw * C.k) * 4u);
    L.route = off;
    if (act_bytes) off = align16u(off + (unsigned)(tpw * C.k) * 4u);
    L.par = off;  off += 16u * 8u;
    L.pc = off;   off += 16u * 4u;
    L.bytes = (off + 255u) & ~255u;
    return L;
}

// LDS shared by a workgroup: per coordinate the row mask's even and odd
// nibbles as table offsets (4 x nibble g in byte g / 2), then the hash table.
__host__ __device__ inline unsigned col_mask_bytes(const ColPlan& C) { return (unsigned)C.mstride * 8u; }
__host__ __device__ inline unsigned col_shared_bytes(const ColPlan& C)
{
    return (col_mask_bytes(C) + (C.hmask + 1u) * 8u + 255u) & ~255u;
}

struct ColWave {
    int lane;
    int ntok;
    int32_t* idx;      // [TPW][k]
    float* coef;       // [TPW][k]
    u32x2* par;        // [16] leaf parents: (index or ~0, 8 h(index))
    float* pc;         // [16] their coefficients (0 for basis and padding parents)
    unsigned char* tab;
    uint32_t* scr;
    uint16_t* xs;      // [TPW][k] slots added one by one
    float* bas;        // [TPW][k + 1] basis coefficients by mark (0: none)
    unsigned char* mark;
    const u32x4* mask; // (shared) per coordinate pair
    const unsigned char* gtab;   // (shared)
};

__device__ inline ColWave col_wave(const ColPlan& C, unsigned char* smem, int cpt, unsigned act_bytes, int wave,
                                   int lane)
{
    const ColLayout L = col_layout(C, cpt, act_bytes);
    unsigned char* b = smem + col_shared_bytes(C) + (unsigned)wave * L.bytes;
    ColWave W;
    W.lane = lane;
    W.ntok = 0;
    W.idx = (int32_t*)(b + L.idx);
    W.coef = (float*)(b + L.coef);
    W.par = (u32x2*)(b + L.par);
    W.pc = (float*)(b + L.pc);
    W.tab = b + L.tab;
    W.scr = (uint32_t*)(b + L.scr);
    W.xs = (uint16_t*)(b + L.xs);
    W.bas = (float*)(b + L.bas);
    W.mark = b + L.mark;
    W.mask = (const u32x4*)smem;
    W.gtab = smem + col_mask_bytes(C);
    return W;
}

__device__ inline void col_load_shared(const ColPlan& C, unsigned char* smem)
{
    uint32_t* m = (uint32_t*)smem;
    for (int i = threadIdx.x; i < C.mstride; i += kColThreads) {
        const uint32_t M = i < C.dp ? C.masks[i] : 0u;
        m[2 * i] = (M << 2) & 0x3C3C3C3Cu;
        m[2 * i + 1] = (M >> 2) & 0x3C3C3C3Cu;
    }
    uint32_t* g = (uint32_t*)(smem + col_mask_bytes(C));
    for (int i = threadIdx.x; i < 2 * ((int)C.hmask + 1); i += kColThreads) g[i] = C.gtab[i];
    __syncthreads();
}

typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) float lds_f32;
__device__ __forceinline__ uint32_t lds_addr(const void* p)
{
    return (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)p;
}
__device__ __forceinline__ uint32_t lds_ld(uint32_t a) { return *(const lds_u32*)(size_t)a; }
__device__ __forceinline__ float lds_ldf(uint32_t a) { return *(const lds_f32*)(size_t)a; }

// Bit transpose inside each 32-lane half: lane s of a half holds x_s on
// entry; on exit lane b holds the word whose bit s is bit b of x_s.  The five
// exchanges run on the vector ALU (a chain of LDS-path swizzles was slower).
__device__ __forceinline__ uint32_t transpose32(uint32_t x, int lane)
{
    uint32_t o;
    o = lane_xor<16>(x);
    x = (lane & 16) ? ((x & 0xFFFF0000u) | ((o >> 16) & 0x0000FFFFu)) : ((x & 0x0000FFFFu) | ((o & 0x0000FFFFu) << 16));
    o = lane_xor<8>(x);
    x = (lane & 8) ? ((x & 0xFF00FF00u) | ((o >> 8) & 0x00FF00FFu)) : ((x & 0x00FF00FFu) | ((o & 0x00FF00FFu) << 8));
    o = lane_xor<4>(x);
    x = (lane & 4) ? ((x & 0xF0F0F0F0u) | ((o >> 4) & 0x0F0F0F0Fu)) : ((x & 0x0F0F0F0Fu) | ((o & 0x0F0F0F0Fu) << 4));
    o = lane_xor<2>(x);
    x = (lane & 2) ? ((x & 0xCCCCCCCCu) | ((o >> 2) & 0x33333333u)) : ((x & 0x33333333u) | ((o & 0x33333333u) << 2));
    o = lane_xor<1>(x);
    x = (lane & 1) ? ((x & 0xAAAAAAAAu) | ((o >> 1) & 0x55555555u)) : ((x & 0x55555555u) | ((o & 0x55555555u) << 1));
    return x;
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Token of item i when every token has n items and there are TPW tokens.
template <int TPW>
__device__ __forceinline__ int item_token(int i, int n)
{
    int t = 0;
#pragma unroll
    for (int u = 1; u < TPW; ++u) t += (int)(i >= u * n);
    return t;
}

// The leaf parents' indices and hashes into W.par (needs W.idx).
template <int CPT>
__device__ __forceinline__ void col_parents(const ColPlan& C, const ColWave& W)
{
    if constexpr (CPT == 0) return;
    else if (W.lane < 16) {
        const int tt = W.lane / CPT, q = W.lane & (CPT - 1);
        const int32_t p = q < C.KP ? W.idx[tt * C.k + C.sbP + q] : -1;
        const uint32_t u = p >= 0 ? (uint32_t)p : ~0u;
        W.par[W.lane] = u32x2{u, ((u ^ (u >> C.hshift)) & C.hmask) << 3};
    }
}

// Parent slot and generator of leaf index c among its token's parents, the
// first matching parent in slot order: (q << 16) | j, or -1.  The hash is
// linear over XOR, so the probe for parent q is at h(c) ^ h(parent q).
// Parent ~0 (none) never matches: generators are below 2^30.
template <int CPT>
__device__ __forceinline__ int col_route(const ColPlan& C, const ColWave& W, int tt, uint32_t c)
{
    const uint32_t hc = ((c ^ (c >> C.hshift)) & C.hmask) << 3;
    constexpr int B = CPT < 8 ? (CPT ? CPT : 1) : 8;
    int rt = -1;
#pragma unroll
    for (int q0 = CPT - B; q0 >= 0; q0 -= B) {
        u32x2 p[B], e[B];
#pragma unroll
        for (int u = 0; u < B; ++u) p[u] = W.par[tt * CPT + q0 + u];
#pragma unroll
        for (int u = 0; u < B; ++u) e[u] = *(const u32x2*)(W.gtab + (hc ^ p[u].y));
        // descending q: the lowest matching parent is kept.  An empty entry
        // is (0, -1): it matches c = parent, which is no child, and gives -1
#pragma unroll
        for (int u = B - 1; u >= 0; --u) rt = (e[u].x ^ p[u].x) == c ? (int)(e[u].y | (uint32_t)((q0 + u) << 16)) : rt;
    }
    return rt;
}

// The bf16 terms of the columns' coefficients as MFMA A operands: lane
// (row, kq) holds generators 4 kq .. 4 kq + 3 of column row.  THREE: a third
// term, which makes the split exact.
struct ColFrag {
    bf16x4 hi, lo, third;
};

template <bool THREE>
__device__ __forceinline__ ColFrag col_frag(const float* alpha, int lane)
{
    const float4 a = *(const float4*)(alpha + (lane & 15) * 16 + 4 * (lane >> 4));
    auto low = [](uint32_t w) { return __uint_as_float(w << 16); };
    auto high = [](uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); };
    ColFrag F;
    const uint32_t h0 = pack_bf16x2(a.x, a.y), h1 = pack_bf16x2(a.z, a.w);
    const float r0 = a.x - low(h0), r1 = a.y - high(h0), r2 = a.z - low(h1), r3 = a.w - high(h1);
    const uint32_t m0 = pack_bf16x2(r0, r1), m1 = pack_bf16x2(r2, r3);
    F.hi = __builtin_bit_cast(bf16x4, (u32x2){h0, h1});
    F.lo = __builtin_bit_cast(bf16x4, (u32x2){m0, m1});
    F.third = F.lo;
    if constexpr (THREE)
        F.third = __builtin_bit_cast(bf16x4, (u32x2){pack_bf16x2(r0 - low(m0), r1 - high(m0)),
                                                     pack_bf16x2(r2 - low(m1), r3 - high(m1))});
    return F;
}

// Tables of each word of 32 listed indices: sign words (row v of group g =
// bits parity(x_b & (v << 4g))) and signed sums of four coefficients (row v
// of group i, times 1/sqrt d).  Two words (32 lanes each) per round.
// slot(tt, w, b, sum) gives the code slot of bit b of word w of token tt (-1:
// none) and whether its coefficient is summed here.
template <int CPT, int NG, typename Slot>
__device__ __forceinline__ void col_tables(const ColPlan& C, const ColWave& W, const float* cf, Slot slot)
{
    constexpr int TPW = col_tpw(CPT);
    const int lane = W.lane, b = lane & 31, v = lane & 15;
    const uint32_t x0 = -(uint32_t)(v & 1), x1 = -(uint32_t)((v >> 1) & 1), x2 = -(uint32_t)((v >> 2) & 1),
                   x3 = -(uint32_t)((v >> 3) & 1);
    const int units = TPW * C.words;
    for (int u0 = 0; u0 < units; u0 += 2) {
        const int unit = min(u0 + (lane >> 5), units - 1);
        const int tt = TPW == 1 ? 0 : item_token<TPW>(unit, C.words);
        const int w = unit - tt * C.words;
        bool sum = true;
        const int s = slot(tt, w, b, sum);
        const int at = tt * C.k + max(s, 0);
        const int32_t c = s >= 0 ? W.idx[at] : 0;
        W.scr[64 + lane] = __float_as_uint(sum && s >= 0 && c >= C.d ? cf[at] : 0.f);
        W.scr[lane] = transpose32((uint32_t)max(c, 0), lane);
        wave_sync();
        unsigned char* tb = W.tab + unit * 1024;
        const int gh = (lane >> 4) & 1;
#pragma unroll
        for (int g0 = 0; g0 < NG; g0 += 2) {
            const int g = g0 + gh;
            const u32x4 e = *(const u32x4*)(W.scr + (lane & 32) + 4 * g);
            const uint32_t V = ((e.x & x0) ^ (e.y & x1)) ^ ((e.z & x2) ^ (e.w & x3));
            *(uint32_t*)(tb + g * 64 + v * 4) = V;
        }
#pragma unroll
        for (int g0 = 0; g0 < 8; g0 += 2) {
            const int g = g0 + gh;
            const u32x4 e = *(const u32x4*)(W.scr + 64 + (lane & 32) + 4 * g);
            const uint32_t sg = 0x80000000u;
            const float t0 = __uint_as_float(e.x ^ (x0 & sg)) + __uint_as_float(e.y ^ (x1 & sg));
            const float t1 = __uint_as_float(e.z ^ (x2 & sg)) + __uint_as_float(e.w ^ (x3 & sg));
            *(float*)(tb + 512 + g * 64 + v * 4) = C.rsd * (t0 + t1);
        }
        wave_sync();
    }
}

// The tables of the plan's own list: a parent in the low bits of the
// half-words of word 0, else a summed slot.
template <int CPT, int NG>
__device__ __forceinline__ void col_list_tables(const ColPlan& C, const ColWave& W, const float* cf)
{
    constexpr int PN = col_parent_nibbles(CPT);
    col_tables<CPT, NG>(C, W, cf, [&](int, int w, int b, bool& sum) {
        const int hb = b & 15, hi = b >> 4;
        int i = 32 * w + b - 32 + col_word0_slots(CPT);   // summed slot of words 1 ..
        if (w == 0) {
            i = (16 - 4 * PN) * hi + hb - 4 * PN;
            sum = hb >= 4 * PN;
            const int q = 2 * hb + hi;
            if (!sum) return hb < CPT / 2 && q < C.KP ? C.sbP + q : -1;
        }
        return i < C.ns ? C.ss + i : -1;
    });
}

// The sign word of a coordinate (its row mask's even and odd nibbles as table
// offsets) from the tables at vb.
template <int NG>
__device__ __forceinline__ uint32_t col_word(uint32_t vb, uint32_t even, uint32_t odd)
{
    uint32_t r[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)
        r[g] = lds_ld(__builtin_amdgcn_perm(vb, (g & 1) ? odd : even, 0x07060500u | (uint32_t)(g >> 1)) +
                      (uint32_t)(g * 64));
    uint32_t x = xor3(r[0], r[1], r[2]);
    if constexpr (NG == 4) x ^= r[3];
    if constexpr (NG >= 5) x = xor3(x, r[3], r[4]);
    if constexpr (NG == 6) x ^= r[5];
    if constexpr (NG == 8) x = xor3(x, r[5], r[6]) ^ r[7];
    return x;
}

// t plus the signed coefficients of a whole word of slots, eight groups of
// four from the sums at tb, with the signs of word x.
__device__ __forceinline__ float col_word_sum(uint32_t tb, uint32_t x, float t)
{
    const uint32_t e4 = (x << 2) & 0x3C3C3C3Cu, o4 = (x >> 2) & 0x3C3C3C3Cu;
#pragma unroll
    for (int n = 0; n < 8; ++n)
        t += lds_ldf(__builtin_amdgcn_perm(tb, (n & 1) ? o4 : e4, 0x07060500u | (uint32_t)(n >> 1)) +
                     (uint32_t)(n * 64));
    return t;
}

// Unlisted slots of a token up to which they are added one by one: about ten
// vector instructions a slot and step, against a table set-up per pass and
// one instruction a slot.  Decode of 16,381 tokens d 768 k 96, us, one by one
// and in passes: 8 slots 55 and 69, 16 slots 67 and 68, 32 slots 84 and 65; at
// d 4096 k 80 (one workgroup a CU, where the set-ups' latency shows) 32 slots
// 685 and 785.  Without leaf columns all of them are added one by one: they are
// hashed indices on level 0 alone.
constexpr int col_few(int cpt) { return cpt ? 16 : 1 << 30; }

// Unlisted slots of a wave's tokens: the most of a token that has its added
// one by one, the most of the others (bits of `big`).  Each token's way, and so
// the order of its sums, is its own count's alone.
struct Unlisted {
    int few, many;
    uint32_t big;
};

// Marks the basis slots' coordinates with slot + 1 and keeps their
// coefficients by mark in W.bas (a coordinate held by several slots gathers
// their coefficients, in slot order, in the marked one); lists the slots that
// fit nowhere else in W.xs and returns how many of them there are.  (Leaf slots
// that went into their parent's column hold a negative index by now.)
template <int CPT>
__device__ __forceinline__ Unlisted col_marks(const ColPlan& C, const ColWave& W, const float* cf)
{
    constexpr int TPW = col_tpw(CPT);
    const int lane = W.lane, k = C.k;
    for (int o = lane * 16; o < TPW * C.mstride; o += 1024) *(u32x4*)(W.mark + o) = u32x4{0u, 0u, 0u, 0u};
    if (lane < TPW) W.bas[lane * (k + 1)] = 0.f;
    wave_sync();
    auto is_extra = [&](int32_t c, int s) { return c >= C.d && (s < C.K0 ? s < C.sbP : s >= C.sbL); };
    uint64_t extras = 0;
    for (int i0 = 0; i0 < TPW * k; i0 += 64) {
        const int i = i0 + lane, tt = item_token<TPW>(i, k), s = i - tt * k;
        const int32_t c = i < TPW * k ? W.idx[i] : -1;
        const bool basis = c >= 0 && c < C.d;
        extras |= __ballot(is_extra(c, s));
        if (!__ballot(basis)) continue;
        unsigned char* m = W.mark + tt * C.mstride + c;
        float* bas = W.bas + tt * (k + 1) + 1;
        const float a = basis ? cf[i] : 0.f;
        const bool fresh = basis && *m == 0;   // not marked by an earlier block
        if (fresh) {
            *m = (unsigned char)(s + 1);   // of several slots any one
            bas[s] = a;
        }
        wave_sync();
        const int owner = basis ? (int)*m - 1 : s;
        if (__ballot(owner != s)) {
            // a repeated coordinate: its slots are added in slot order
            if (fresh && owner == s) bas[s] = 0.f;
            for (uint64_t left = __ballot(basis); left; left &= left - 1) {
                if (lane == __builtin_ctzll(left)) bas[owner] += a;
                wave_sync();
            }
        }
        wave_sync();
    }
    Unlisted U{0, 0, 0u};
    if (!extras) return U;
    for (int tt = 0; tt < TPW; ++tt) {
        int n = 0;
        for (int s0 = 0; s0 < k; s0 += 64) {
            const int s = s0 + lane;
            const bool extra = s < k && is_extra(W.idx[tt * k + s], s);
            const uint64_t ball = __ballot(extra);
            if (extra) W.xs[tt * k + n + (int)__popcll(ball & ((1ull << lane) - 1ull))] = (uint16_t)s;
            n += (int)__popcll(ball);
        }
        for (int i = n + lane; i < k; i += 64) W.xs[tt * k + i] = 0xFFFF;   // no slot
        if (n > col_few(CPT)) {
            U.many = max(U.many, n);
            U.big |= 1u << tt;
        } else {
            U.few = max(U.few, n);
        }
    }
    wave_sync();
    return U;
}

// Index and scaled coefficient of the 64 / TPW slots of W.xs from number i0
// on, zero past the last and for the tokens of `big`, where the tables'
// scratch is free by now.
template <int CPT>
__device__ __forceinline__ void col_stage_few(const ColPlan& C, const ColWave& W, const float* cf, int i0, uint32_t big)
{
    constexpr int cap = 64 / col_tpw(CPT);
    const int lane = W.lane, i = i0 + (lane & (cap - 1)), tt = lane / cap;
    const int s = i < C.k && !((big >> tt) & 1u) ? W.xs[tt * C.k + i] : 0xFFFF;
    const int at = tt * C.k + (s == 0xFFFF ? 0 : s);
    const float a = s == 0xFFFF ? 0.f : C.rsd * cf[at];
    ((u32x2*)W.scr)[lane] = u32x2{(uint32_t)W.idx[at], __float_as_uint(a)};
    wave_sync();
}

constexpr int kColPass = 4;   // coordinate steps of a pass

// Sums of the slots of W.xs of U's big tokens over the steps from m0 on,
// as many words of them at a time as the plan's tables have room for.  The
// tables are built anew for each pass, the plan's own after them: room for
// both would take a workgroup a CU from every code.  A code of 64 leaves and
// no parent, 16,381 tokens d 768, us: decode 254 one by one, 77 here (108 in
// the row-in-LDS kernels); backward 344, 139 (174).
template <int CPT, int NG>
__device__ __forceinline__ void col_pass(const ColPlan& C, const ColWave& W, const float* cf, Unlisted U, int m0,
                                         float (&ex)[2 * kColPass])
{
    constexpr int LPT = 64 / col_tpw(CPT), PS = kColPass;
    const uint32_t vb = lds_addr(W.tab) + (uint32_t)(W.lane / LPT * C.words) * 1024u;
    const u32x4* mk = W.mask + (W.lane & (LPT - 1));
#pragma unroll
    for (int u = 0; u < 2 * PS; ++u) ex[u] = 0.f;
    for (int i0 = 0; i0 < U.many; i0 += 32 * C.words) {
        col_tables<CPT, NG>(C, W, cf, [&](int tt, int w, int b, bool&) {
            const int i = i0 + 32 * w + b, s = i < C.k && ((U.big >> tt) & 1u) ? W.xs[tt * C.k + i] : 0xFFFF;
            return s == 0xFFFF ? -1 : s;
        });
        for (int w = 0; w < min(C.words, (U.many - i0 + 31) / 32); ++w) {
#pragma unroll
            for (int u = 0; u < PS; ++u) {
                const u32x4 sm = mk[min(m0 + u, C.steps - 1) * LPT];
                const uint32_t v = vb + (uint32_t)w * 1024u;
                const uint32_t x[2] = {col_word<NG>(v, sm.x, sm.y), col_word<NG>(v, sm.z, sm.w)};
                float r[2][8];   // all sixteen requested before the first is added
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const uint32_t e4 = (x[e] << 2) & 0x3C3C3C3Cu, o4 = (x[e] >> 2) & 0x3C3C3C3Cu;
#pragma unroll
                    for (int n = 0; n < 8; ++n)
                        r[e][n] = lds_ldf(__builtin_amdgcn_perm(v + 512u, (n & 1) ? o4 : e4, 0x07060500u | (uint32_t)(n >> 1)) +
                                          (uint32_t)(n * 64));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int n = 0; n < 8; ++n) ex[2 * u + e] += r[e][n];
            }
        }
        wave_sync();
    }
}

// The coordinate steps: G0 four-slot groups of word 0 are summed.  out (and
// the optional add, which may alias it) are the rows of the wave's tokens,
// row stride d.  nx staged slots are added one by one; with PASS only the steps
// of a pass from m0 on are taken, on top of its sums ex.
template <int CPT, int NG, bool OUT_BF16, int G0, bool PASS = false>
__device__ __forceinline__ void col_steps(const ColPlan& C, const ColWave& W, const float* cf, const ColFrag& F,
                                          f32x4 c0, int nx, int64_t row0, void* out, const void* add, int m0 = 0,
                                          float* ex = nullptr)
{
    constexpr int TPW = col_tpw(CPT), LPT = 64 / TPW, NP = LPT / 16;   // NP 16-column blocks per pair half
    constexpr int PN = col_parent_nibbles(CPT);
    const int lane = W.lane, row = lane & 15, kq = lane >> 4, ll = lane & (LPT - 1);
    const int tt = lane / LPT;
    const uint32_t vb = lds_addr(W.tab) + (uint32_t)(tt * C.words) * 1024u, tb = vb + 512u;
    const u32x4* mk = W.mask + ll;
    const unsigned char* mark = W.mark + tt * C.mstride + 2 * ll;
    const int sh0 = CPT ? 15 - 2 * (kq & (CPT / 4 - 1)) : 0;
    // B operands: coordinates 2 LPT m + 32 p + 2 row + {0, 1}, generators 4 kq .. (16 bytes hold both).
    // Addresses here and of the rows are a scalar base plus a 32-bit lane offset.
    const char* bfr = (const char*)C.gamma_t;
    const int blocks2 = C.dp / 32;                       // pairs of 16-coordinate blocks
    const uint32_t boff = 16u * (uint32_t)((row >> 3) * 32 + (row & 7) + 8 * kq);   // block, column pair, generators
    auto fetch = [&](int m, u32x4 (&B)[NP]) {
        if constexpr (CPT == 0) return;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            B[p] = *(const u32x4*)(bfr + (size_t)(1024u * (uint32_t)min(m * NP + p, blocks2 - 1)) + boff);
    };
    const int lim = tt < W.ntok ? C.d - 2 * ll : 0;     // coordinates left of this lane's first
    constexpr uint32_t ES = OUT_BF16 ? 2 : 4;
    char* orow = (char*)out + row0 * C.d * ES;
    const char* arow = (const char*)add + row0 * C.d * ES;
    const uint32_t ooff = (uint32_t)(tt * C.d + 2 * ll) * ES;
    const bool even = (C.d & 1) == 0;
    const float* bas = W.bas + tt * (C.k + 1);
    u32x4 B[NP];
    const int mend = PASS ? min(m0 + kColPass, C.steps) : C.steps;
    fetch(PASS ? m0 : 0, B);
    for (int m = PASS ? m0 : 0; m < mend; ++m) {
        const u32x4 sm = mk[m * LPT];
        const uint32_t mw = *(const uint16_t*)(mark + m * 2 * LPT);
        const float b0 = bas[mw & 255u], b1 = bas[mw >> 8];   // basis coefficients (mark 0: none)
        const uint32_t s0[2] = {sm.x, sm.z}, s1[2] = {sm.y, sm.w};
        // columns: products of both coordinates of every block
        f32x4 acc[2][NP];
#pragma unroll
        for (int p = 0; p < (CPT ? NP : 0); ++p) {
            const bf16x4 g0 = __builtin_bit_cast(bf16x4, (u32x2){B[p].x, B[p].y});
            const bf16x4 g1 = __builtin_bit_cast(bf16x4, (u32x2){B[p].z, B[p].w});
            acc[0][p] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(F.hi, g0, c0, 0, 0, 0);
            acc[1][p] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(F.hi, g1, c0, 0, 0, 0);
            acc[0][p] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(F.lo, g0, acc[0][p], 0, 0, 0);
            acc[1][p] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(F.lo, g1, acc[1][p], 0, 0, 0);
            if constexpr (!OUT_BF16) {
                acc[0][p] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(F.third, g0, acc[0][p], 0, 0, 0);
                acc[1][p] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(F.third, g1, acc[1][p], 0, 0, 0);
            }
        }
        fetch(m + 1 < C.steps ? m + 1 : m, B);
        // sign words and coefficient sums of the two coordinates
        uint32_t U[2];
        float t[2] = {b0, b1};
        if constexpr (PASS) {
            t[0] += ex[0];
            t[1] += ex[1];
#pragma unroll
            for (int u = 0; u + 2 < 2 * kColPass; ++u) ex[u] = ex[u + 2];
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) U[e] = col_word<NG>(vb, s0[e], s1[e]);
        if constexpr (G0 > 0) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t e4 = (U[e] << 2) & 0x3C3C3C3Cu, o4 = (U[e] >> 2) & 0x3C3C3C3Cu;
#pragma unroll
                for (int i = 0; i < G0; ++i) {
                    const int n = PN + i + (i >= 4 - PN ? PN : 0);   // nibble of group i
                    t[e] += lds_ldf(__builtin_amdgcn_perm(tb, (n & 1) ? o4 : e4, 0x07060500u | (uint32_t)(n >> 1)) +
                                    (uint32_t)(n * 64));
                }
            }
        }
        for (int w = 1; w < C.words; ++w) {
            const uint32_t v = vb + (uint32_t)w * 1024u;
#pragma unroll
            for (int e = 0; e < 2; ++e) t[e] = col_word_sum(v + 512u, col_word<NG>(v, s0[e], s1[e]), t[e]);
        }
        // the parents' signs on this lane's four columns, then the token's columns summed
        float y[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if constexpr (CPT == 0) {
                y[e] = t[e];
                continue;
            }
            uint32_t Up[NP];
            if constexpr (NP == 1) {
                Up[0] = U[e];
            } else if constexpr (NP == 2) {
                const auto s = __builtin_amdgcn_permlane16_swap(U[e], U[e], false, false);
                Up[0] = s[0];
                Up[1] = s[1];
            } else {
                const auto h = __builtin_amdgcn_permlane32_swap(U[e], U[e], false, false);
                const auto a = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
                const auto b = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
                Up[0] = a[0];
                Up[1] = a[1];
                Up[2] = b[0];
                Up[3] = b[1];
            }
            float v[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const uint32_t Ra = Up[p] << sh0, Rb = Up[p] << (sh0 - 1);
                const f16x2 sa = __builtin_bit_cast(f16x2, __builtin_amdgcn_bitop3_b32(Ra, 0x80008000u, 0x3C003C00u, 0xEA));
                const f16x2 sb = __builtin_bit_cast(f16x2, __builtin_amdgcn_bitop3_b32(Rb, 0x80008000u, 0x3C003C00u, 0xEA));
                const f32x4 q = acc[e][p];
                float x = __builtin_fmaf((float)sa.x, q[0], 0.f);
                x = __builtin_fmaf((float)sa.y, q[1], x);
                x = __builtin_fmaf((float)sb.x, q[2], x);
                v[p] = __builtin_fmaf((float)sb.y, q[3], x);
            }
            float leaf;
            if constexpr (NP == 1) {
                leaf = v[0];
            } else {
                auto swap_sum = [](float a, float b, auto lanes32) {
                    if constexpr (lanes32.value) {
                        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
                        return __uint_as_float(s[0]) + __uint_as_float(s[1]);
                    } else {
                        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
                        return __uint_as_float(s[0]) + __uint_as_float(s[1]);
                    }
                };
                if constexpr (NP == 2) {
                    leaf = swap_sum(v[0], v[1], std::false_type{});
                } else {
                    const float a = swap_sum(v[0], v[2], std::true_type{}), b = swap_sum(v[1], v[3], std::true_type{});
                    leaf = swap_sum(a, b, std::false_type{});
                }
            }
            y[e] = __builtin_fmaf(C.rsd, leaf, t[e]);
        }
        if (nx) {
            // slots added one by one: sign = parity of the row mask and the index
            const uint32_t M0 = (s0[0] >> 2) | (s1[0] << 2), M1 = (s0[1] >> 2) | (s1[1] << 2);
            auto add_slot = [&](uint32_t c, float a) {
                y[0] += signed_by_parity(a, M0 & c);
                y[1] += signed_by_parity(a, M1 & c);
            };
            const u32x2* few = (const u32x2*)W.scr + tt * (64 / TPW);
            constexpr int cap = 64 / TPW;
            for (int i0 = 0; i0 < nx; i0 += cap) {
                if (CPT == 0 && nx > cap) {   // more than the scratch holds
                    wave_sync();
                    col_stage_few<CPT>(C, W, cf, i0, 0u);
                }
                for (int i = 0; i < min(nx - i0, cap); i += 4) {
                    u32x2 q[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) q[u] = few[i + u];
#pragma unroll
                    for (int u = 0; u < 4; ++u) add_slot(q[u].x, __uint_as_float(q[u].y));
                }
                if (CPT > 0) break;   // col_few of them at most
            }
        }
        if (m * 2 * LPT < lim) {
            const size_t mo = (size_t)((uint32_t)(m * 2 * LPT) * ES);
            const bool second = m * 2 * LPT + 1 < lim;
            char* o = orow + mo + ooff;
            const char* ad = arow + mo + ooff;
            if (even) {
                if constexpr (OUT_BF16) {
                    if (add) {
                        const uint32_t q = *(const uint32_t*)ad;
                        y[0] += bf16_bits_to_f32(q & 0xFFFFu);
                        y[1] += bf16_bits_to_f32(q >> 16);
                    }
                    *(uint32_t*)o = pack_bf16x2(y[0], y[1]);
                } else {
                    if (add) {
                        const float2 q = *(const float2*)ad;
                        y[0] += q.x;
                        y[1] += q.y;
                    }
                    *(float2*)o = make_float2(y[0], y[1]);
                }
            } else {
                if (add) {
                    y[0] += load_act<OUT_BF16>(ad, 0);
                    if (second) y[1] += load_act<OUT_BF16>(ad, 1);
                }
                store_act<OUT_BF16>(o, 0, y[0]);
                if (second) store_act<OUT_BF16>(o, 1, y[1]);
            }
        }
    }
}

// Decode of the wave's tokens from W.idx and coefficients cf (W.par set,
// alpha = the leaf coefficients by (column, generator) in W.tab).
template <int CPT, int NG, bool OUT_BF16>
__device__ __forceinline__ void col_decode(const ColPlan& C, const ColWave& W, const float* cf, int64_t row0, void* out,
                                           const void* add)
{
    const int lane = W.lane;
    ColFrag F{};
    f32x4 c0{};
    if constexpr (CPT > 0) {
        if (lane < 16) {
            const int tt = lane / CPT, q = lane & (CPT - 1);
            const uint32_t p = W.par[lane].x;
            W.pc[lane] = p != ~0u && p >= (uint32_t)C.d ? cf[tt * C.k + C.sbP + q] : 0.f;
        }
        wave_sync();
        F = col_frag<!OUT_BF16>((const float*)W.tab, lane);
        c0 = *(const f32x4*)(W.pc + 4 * (lane >> 4));
        wave_sync();
    }
    constexpr int MG = col_word0_slots(CPT) / 4;   // groups of word 0
    col_list_tables<CPT, NG>(C, W, cf);
    const Unlisted U = col_marks<CPT>(C, W, cf);
    const int nx = U.few;
    if (CPT > 0 && U.many) {
        // the tables hold the unlisted slots of a few steps and the listed ones
        // of the same steps in turn
        ColWave V = W;
        for (int m0 = 0; m0 < C.steps; m0 += kColPass) {
            float ex[2 * kColPass];
            __asm__ volatile("" : "+v"(V.lane));   // nothing of this path is worked out before it
            col_pass<CPT, NG>(C, V, cf, U, m0, ex);
            __asm__ volatile("" : "+v"(V.lane));
            col_list_tables<CPT, NG>(C, V, cf);
            if (nx) col_stage_few<CPT>(C, V, cf, 0, U.big);
            __asm__ volatile("" : "+v"(V.lane));
            col_steps<CPT, NG, OUT_BF16, MG, true>(C, V, cf, F, c0, nx, row0, out, add, m0, ex);
            wave_sync();
        }
        return;
    }
    if (nx) col_stage_few<CPT>(C, W, cf, 0, 0u);
    wave_sync();
    const int g0 = min(C.ns, col_word0_slots(CPT));
    if (g0 == 0) col_steps<CPT, NG, OUT_BF16, 0>(C, W, cf, F, c0, nx, row0, out, add);
    else if (g0 <= 8) col_steps<CPT, NG, OUT_BF16, 2>(C, W, cf, F, c0, nx, row0, out, add);
    else if (MG == 4 || g0 <= 16) col_steps<CPT, NG, OUT_BF16, 4>(C, W, cf, F, c0, nx, row0, out, add);
    else if (MG == 6 || g0 <= 24) col_steps<CPT, NG, OUT_BF16, MG < 6 ? 4 : 6>(C, W, cf, F, c0, nx, row0, out, add);
    else col_steps<CPT, NG, OUT_BF16, MG>(C, W, cf, F, c0, nx, row0, out, add);
    wave_sync();
}

// Clears alpha (to -0: a cell that still reads -0 holds nothing, and -0 adds
// nothing), then adds each routed leaf coefficient to its cell and takes the
// slot off the list (a negative index).  An index listed several times
// gathers its slots in slot order: two slots give the same sum in either
// order, and a cell that three or more go to sends the group through the adds
// again, one slot after another.
// route(tt, s) gives the route of a leaf slot.
template <int CPT, typename Route>
__device__ __forceinline__ void col_alpha(const ColPlan& C, const ColWave& W, const float* cf, Route route)
{
    if constexpr (CPT == 0) return;
    constexpr int TPW = col_tpw(CPT);
    static_assert(TPW * kColMaxSlots <= 64 * 32, "a bit per round of 64 leaf slots");
    float* alpha = (float*)W.tab;
    const int n = TPW * C.KL;
    auto slot = [&](int i) {
        const int tt = item_token<TPW>(i, C.KL);
        return tt * C.k + C.sbL + i - tt * C.KL;
    };
    auto taken = [](float old) { return (uint32_t)(__float_as_uint(old) != 0x80000000u); };
    float none = -0.f;
    __asm__ volatile("" : "+v"(none));   // four registers of it would be kept across the groups
    *(float4*)(alpha + 4 * W.lane) = make_float4(none, none, none, none);
    wave_sync();
    uint32_t again = 0, bit = 1;   // a bit per round: this lane's cell already held something
    float old = -0.f;              // looked at a round later, when it has arrived
    for (int i = W.lane; i < n; i += 64) {
        const int tt = item_token<TPW>(i, C.KL), at = slot(i);
        const int rt = route(tt, at - tt * C.k);
        again |= taken(old) * (bit >> 1);
        old = -0.f;
        if (rt >= 0) {
            const int cell = (tt * CPT + (rt >> 16)) * 16 + (rt & 0xFFFF);
            old = atomicAdd(&alpha[cell], cf[at]);
            W.idx[at] = -2 - cell;
        } else {
            W.idx[at] = max(W.idx[at], -1);
        }
        bit <<= 1;
    }
    again |= taken(old) * (bit >> 1);
    if (__ballot(again != 0)) {
        int lane = W.lane;
        __asm__ volatile("" : "+v"(lane));   // nothing of this path is worked out before it
        if (lane < 8) W.scr[lane] = 0;
        wave_sync();
        bool third = false;
        for (int i = lane; again; i += 64, again >>= 1)
            if (again & 1u) {
                const int cell = -2 - W.idx[slot(i)];
                third |= ((atomicOr(&W.scr[cell >> 5], 1u << (cell & 31)) >> (cell & 31)) & 1u) != 0;
            }
        if (__ballot(third)) {
            wave_sync();
            *(float4*)(alpha + 4 * lane) = make_float4(0.f, 0.f, 0.f, 0.f);
            wave_sync();
            for (int i0 = 0; i0 < n; i0 += 64) {
                const int i = i0 + lane, at = slot(min(i, n - 1));
                const int cell = i < n ? -2 - W.idx[at] : -1;
                for (uint64_t left = __ballot(cell >= 0); left; left &= left - 1) {
                    if (lane == __builtin_ctzll(left)) alpha[cell] += cf[at];
                    wave_sync();
                }
            }
        }
    }
    wave_sync();
}

// A group's codes on their way to LDS (the next group's are requested while
// this one is processed).
struct CodeFetch {
    static constexpr int kWords = 4;   // per lane and array: groups of up to 256 slots are prefetched
    int32_t i[kWords];
    float c[kWords];
};

// Parent columns per token of the column decode: the last level's where it
// decodes through them, else 0 (every hashed slot through the tables); -1 for
// codes wider than a mark, which the row-in-LDS kernels of codes.hip take.
inline int col_cpt(const DevPlan& P)
{
    const int L1 = P.levels - 1;
    if (P.k_tot > kColMaxSlots) return -1;
    if (!P.leaf_columns || P.gtab_total <= 0 || P.cpt[L1] < 4 || P.cpt[L1] > 16) return 0;
    return P.cpt[L1];
}

inline ColPlan col_plan(const DevPlan& P, int cpt)
{
    const int L1 = P.levels - 1, lpt = 64 / col_tpw(cpt);
    ColPlan C{};
    C.d = P.d;
    C.dp = P.dp;
    C.steps = (P.dp + 2 * lpt - 1) / (2 * lpt);
    C.mstride = 2 * lpt * C.steps;
    C.k = P.k_tot;
    C.K0 = P.active[0];
    C.ss = P.active[0];
    C.sbP = C.sbL = P.k_tot;
    C.gtab = P.gtab;
    C.masks = P.masks;
    C.rsd = P.rsd;
    if (cpt) {
        C.KP = P.active[L1 - 1];
        C.sbP = P.slot_base[L1 - 1];
        C.KL = P.active[L1];
        C.sbL = P.slot_base[L1];
        C.hmask = (1u << P.gtab_bits[L1]) - 1u;
        C.hshift = P.gtab_shift[L1];
        C.gtab = P.gtab + 2 * (size_t)P.gtab_off[L1];
        C.gamma_t = (const char*)P.gamma_t + 8 * P.gamma_t_off[L1];
    }
    C.ns = std::max(0, C.sbP - C.K0);
    C.words = 1 + (std::max(0, C.ns - col_word0_slots(cpt)) + 31) / 32;
    return C;
}

// The parent columns per token a kernel takes for the plan (lds(cpt): bytes of
// its workgroup).  A wave of several tokens holds all their rows.  Where a CU
// has room for one such workgroup only, and for two or more without leaf
// columns, the plan goes without them unless they save it table words; where
// it has room for none, it goes without them in any case (else the row-in-LDS
// kernels would take it).
// Backward of 16,381 tokens in bf16, us, with and without: d 1024 K 32,32,4,12
// 324 and 102, d 2048 K 4,4,8 168 and 101, d 3000 K 8,8,16 347 and 287; a word
// more without: d 2048 K 4,4,32 178 and 224; one workgroup either way: d 4096
// K 8,8,16 418 and 564.
template <typename Lds>
inline int col_choose(const DevPlan& P, Lds lds)
{
    const int cpt = col_cpt(P);
    if (cpt <= 0 || lds(cpt) <= (size_t)kLdsBudget / 2) return cpt;
    if (lds(cpt) > (size_t)kLdsBudget) return 0;
    return lds(0) <= (size_t)kLdsBudget / 2 && col_plan(P, 0).words <= col_plan(P, cpt).words ? 0 : cpt;
}

// Persistent grid over groups of `tpw` tokens: `rounds` times the workgroups
// that `lds` lets the chip hold, at most `waves` waves per SIMD of them.
inline dim3 col_grid(int64_t T, int tpw, size_t lds, int waves, int rounds)
{
    const int64_t groups = (T + tpw - 1) / tpw, need = (groups + kColWaves - 1) / kColWaves;
    const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(waves, (160 * 1024) / lds));
    return dim3((unsigned)std::max<int64_t>(1, std::min(need, (int64_t)device_cus() * per_cu * rounds)));
}

}  // namespace dpb
