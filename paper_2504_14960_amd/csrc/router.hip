// a1. Router: logits = x W_g^T (+ bias), softmax over experts, top-K gating
// (Eq. 2 and Eq. 3, Section 3.1.1; router paragraph of Section 3.3).
//
// bf16 path: one workgroup owns 16*MB tokens and all experts.  Its four waves
// split the hidden dimension; each wave streams its slices of the token rows
// with fully coalesced 16-byte loads, parks them in a wave-private LDS region
// and re-reads them in MFMA operand order (16x16x32 bf16, fp32 accumulate).
// The router weight is small and stays in L2; its fragments are read straight
// from global memory.  Partial sums are folded in a fixed wave order, so the
// logits are bit-reproducible.  Selection is done by groups of lanes, one
// group per token, with butterfly reductions on (value desc, index asc) keys.
// With few tokens the same work is spread over more workgroups (router_logits_kernel; the selection in the same launch for up
// to 16 experts, else one of its own); with many tokens and 17 to 128 experts the logits are computed in tiles of tokens and
// experts (router_tile_kernel).
#include "common.h"

namespace moe {

namespace {

__device__ __forceinline__ bool ranks_before(float a, int ia, float b, int ib) {
    return (a > b) || (a == b && ia < ib);
}

// One token per group of G lanes (G a power of two, <= 64); lane `lig` of the
// group holds the logits of experts lig + j*G, j < VPL.  Lane k of the group
// writes slot k.
template <int VPL>
__device__ __forceinline__ void select_topk(const float (&vin)[VPL], int lig, int G, int E, int K,
                                            int renorm, bool valid, int32_t* idx_out,
                                            float* gate_out) {
    float v[VPL];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        const int e = lig + j * G;
        float x = vin[j];
        x = (x != x) ? -INFINITY : x;  // NaN ranks last
        v[j] = (e < E) ? x : -INFINITY;
        m = fmaxf(m, v[j]);
    }
    for (int off = G >> 1; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, G));
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        const int e = lig + j * G;
        if (e < E) z += expf(v[j] - m);
    }
    for (int off = G >> 1; off > 0; off >>= 1) z += __shfl_xor(z, off, G);

    uint32_t taken = 0;
    float my_gate = 0.f, gsum = 0.f;
    int my_idx = 0;
    for (int k = 0; k < K; ++k) {
        float bv = -INFINITY;
        int be = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
            const int e = lig + j * G;
            if (e < E && !((taken >> j) & 1u) && ranks_before(v[j], e, bv, be)) {
                bv = v[j];
                be = e;
            }
        }
        for (int off = G >> 1; off > 0; off >>= 1) {
            const float ov = __shfl_xor(bv, off, G);
            const int oe = __shfl_xor(be, off, G);
            if (ranks_before(ov, oe, bv, be)) {
                bv = ov;
                be = oe;
            }
        }
        if (be < E && (be & (G - 1)) == lig) taken |= 1u << (be / G);
        const float p = expf(bv - m) / z;
        gsum += p;
        if (lig == k) {
            my_gate = p;
            my_idx = be;
        }
    }
    if (renorm) my_gate /= gsum;
    if (valid && lig < K) {
        idx_out[lig] = my_idx;
        gate_out[lig] = my_gate;
    }
}

__host__ __device__ inline int group_lanes(int E) {
    int g = 1;
    while (g < E && g < 64) g <<= 1;
    return g;
}

// Selection for `ntok` tokens whose logits sit in `rows` (row stride `ld`, LDS
// or global), spread over the 4 waves of the workgroup.
template <int VPL>
__device__ __forceinline__ void select_block(const float* rows, int ld, int ntok, int t0, int T,
                                             int E, int K, int renorm, int32_t* topk_idx,
                                             float* topk_gate) {
    const int G = group_lanes(E);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
    const int per_wave = 64 / G;
    const int lig = lane & (G - 1), grp = lane / G;
    for (int base = wave * per_wave; base < ntok; base += nwaves * per_wave) {
        const int lt = base + grp;
        const bool valid = lt < ntok && (t0 + lt) < T;
        float v[VPL];
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
            const int e = lig + j * G;
            v[j] = (valid && e < E) ? rows[(size_t)lt * ld + e] : -INFINITY;
        }
        const size_t o = (size_t)(t0 + (valid ? lt : 0)) * K;
        select_topk<VPL>(v, lig, G, E, K, renorm, valid, topk_idx + o, topk_gate + o);
    }
}

__device__ __forceinline__ void select_dispatch(const float* rows, int ld, int ntok, int t0, int T,
                                                int E, int K, int renorm, int32_t* topk_idx,
                                                float* topk_gate) {
    if (E <= 64)
        select_block<1>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
    else if (E <= 128)
        select_block<2>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
    else
        select_block<4>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
}

// Selection with L lanes per token (K <= KSEL <= 8, L in {1, 2, 4, 8}).  Lane
// `sub` of a token walks its block of ceil(E/L) consecutive logits (with an odd
// row stride the lanes of a wave then hit distinct LDS banks), keeping its KSEL
// best in a sorted register list (insertion by compare-and-swap on the key
// (value desc, index asc), so equal logits keep the lower index first).  The L
// lists are then merged pairwise across lanes: the element-wise better of my
// list and the partner's reversed list is a bitonic sequence holding the KSEL
// best of both, and log2(KSEL) compare-exchange stages sort it; both partners
// end with the same list.  A second walk gives the softmax denominator.
// L = 1 needs no cross-lane traffic at all; L = 8 gives 8192 tokens of a
// 64-expert layer 1024 waves of work instead of 128.
// `rows` must be LDS (row stride `ld`, odd => conflict-free).
template <int KSEL, int L>
__device__ __forceinline__ void select_lanes(const float* rows, int ld, int ntok, int t0, int T, int E,
                                             int K, int renorm, int32_t* topk_idx, float* topk_gate) {
    const int sub = threadIdx.x % L;
    const int tpb = blockDim.x / L;  // tokens per pass of the workgroup
    for (int base = 0; base < ntok; base += tpb) {
        const int lt = base + threadIdx.x / L;
        const bool valid = lt < ntok && t0 + lt < T;  // same for the L lanes of a token
        const float* r = rows + (size_t)(valid ? lt : 0) * ld;
        float lv[KSEL];
        int le[KSEL];
#pragma unroll
        for (int j = 0; j < KSEL; ++j) {
            lv[j] = -INFINITY;
            le[j] = 0x7fffffff;
        }
        const int e_begin = sub * ((E + L - 1) / L), e_end = min(E, e_begin + (E + L - 1) / L);
        for (int e = e_begin; e < e_end; ++e) {
            float cv = r[e];
            cv = (cv != cv) ? -INFINITY : cv;  // NaN ranks last
            int ce = e;
#pragma unroll
            for (int j = 0; j < KSEL; ++j) {
                const bool b = ranks_before(cv, ce, lv[j], le[j]);
                const float tv = b ? lv[j] : cv;
                const int te = b ? le[j] : ce;
                lv[j] = b ? cv : lv[j];
                le[j] = b ? ce : le[j];
                cv = tv;
                ce = te;
            }
        }
#pragma unroll
        for (int off = 1; off < L; off <<= 1) {
            float pv[KSEL];
            int pe[KSEL];
#pragma unroll
            for (int j = 0; j < KSEL; ++j) {
                pv[j] = __shfl_xor(lv[j], off, 64);
                pe[j] = __shfl_xor(le[j], off, 64);
            }
#pragma unroll
            for (int j = 0; j < KSEL; ++j) {
                const bool b = ranks_before(pv[KSEL - 1 - j], pe[KSEL - 1 - j], lv[j], le[j]);
                lv[j] = b ? pv[KSEL - 1 - j] : lv[j];
                le[j] = b ? pe[KSEL - 1 - j] : le[j];
            }
#pragma unroll
            for (int d = KSEL / 2; d > 0; d >>= 1)
#pragma unroll
                for (int j = 0; j < KSEL; ++j)
                    if ((j & d) == 0) {
                        const bool b = ranks_before(lv[j + d], le[j + d], lv[j], le[j]);
                        const float tv = lv[j];
                        const int te = le[j];
                        lv[j] = b ? lv[j + d] : tv;
                        le[j] = b ? le[j + d] : te;
                        lv[j + d] = b ? tv : lv[j + d];
                        le[j + d] = b ? te : le[j + d];
                    }
        }
        const float m = lv[0];
        float z = 0.f;
        for (int e = e_begin; e < e_end; ++e) {
            float v = r[e];
            v = (v != v) ? -INFINITY : v;
            z += expf(v - m);
        }
#pragma unroll
        for (int off = 1; off < L; off <<= 1) z += __shfl_xor(z, off, 64);
        float gsum = 0.f;
#pragma unroll
        for (int k = 0; k < KSEL; ++k)
            if (k < K) gsum += expf(lv[k] - m) / z;
        // lane `sub` writes the slots sub, sub + L, ...
#pragma unroll
        for (int k = 0; k < KSEL; ++k)
            if (k < K && (k % L) == sub && valid) {
                const size_t o = (size_t)(t0 + lt) * K;
                const float p = expf(lv[k] - m) / z;
                topk_idx[o + k] = le[k];
                topk_gate[o + k] = renorm ? p / gsum : p;
            }
    }
}

// lanes per token of the register-list selection: about 8 logits per lane
__host__ __device__ inline int lanes_per_token(int E) { return E >= 64 ? 8 : E >= 32 ? 4 : E >= 16 ? 2 : 1; }

template <int KSEL>
__device__ __forceinline__ void select_lanes_for(const float* rows, int ld, int ntok, int t0, int T, int E,
                                                 int K, int renorm, int32_t* topk_idx, float* topk_gate) {
    switch (lanes_per_token(E)) {
        case 8: select_lanes<KSEL, 8>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate); break;
        case 4: select_lanes<KSEL, 4>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate); break;
        case 2: select_lanes<KSEL, 2>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate); break;
        default: select_lanes<KSEL, 1>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate); break;
    }
}

// K <= 8: register lists; larger K: one lane group per token.
__device__ __forceinline__ void select_tokens(const float* rows, int ld, int ntok, int t0, int T, int E,
                                              int K, int renorm, int32_t* topk_idx, float* topk_gate) {
    if (K <= 2)
        select_lanes_for<2>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
    else if (K <= 4)
        select_lanes_for<4>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
    else if (K <= 8)
        select_lanes_for<8>(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
    else
        select_dispatch(rows, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
}

// ------------------------------------------------------------------ bf16 / MFMA
template <int MB, int NB>
__global__ __launch_bounds__(256) void router_bf16_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, const float* __restrict__ bias,
    float* __restrict__ logits, int T, int H, int E, int K, int renorm,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate) {
    constexpr int TOK = 16 * MB;      // tokens per workgroup
    // MFMA k-steps per slice: 8 token loads in flight per lane where the weight
    // fragments of a slice (KSTEPS * NB of them, kept in registers) allow it
    constexpr int KSTEPS = (8 / MB < ((16 / NB) > 1 ? (16 / NB) : 1)) ? 8 / MB : ((16 / NB) > 1 ? (16 / NB) : 1);
    constexpr int KC = 32 * KSTEPS;   // hidden elements per slice
    constexpr int LPR = KC / 8;       // lanes covering one row slice
    constexpr int KCP = KC + 8;       // padded LDS row (elements)
    constexpr int RPI = 64 / LPR;     // rows per load instruction
    constexpr int NLD = TOK / RPI;    // token loads per lane per slice
    constexpr int EP = 16 * NB;       // experts padded to the MFMA N size
    __shared__ __attribute__((aligned(16))) bf16_t xs[4][TOK][KCP];
    __shared__ float red[TOK][EP + 1];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = blockIdx.x * TOK;
    const int nchunks = (H + KC - 1) / KC;

    f32x4 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int lrow = lane / LPR, lcol = (lane % LPR) * 8;
    const int fr = lane & 15, fg = lane >> 4;  // fragment row / k-group
    // both the token slice and the matching router-weight fragments of the NEXT
    // slice are requested before the current slice is multiplied, so neither the
    // HBM nor the L2 round trip sits in front of an MFMA
    u32x4 xr[NLD], wr[KSTEPS][NB];
    auto load_chunk = [&](int c) {
        const int k = c * KC + lcol;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int t = t0 + i * RPI + lrow;
            u32x4 v = u32x4{0u, 0u, 0u, 0u};
            if (t < T && k < H) v = *reinterpret_cast<const u32x4*>(x + (size_t)t * H + k);
            xr[i] = v;
        }
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
            const int kw = c * KC + s * 32 + fg * 8;
#pragma unroll
            for (int b2 = 0; b2 < NB; ++b2) {
                const int e = b2 * 16 + fr;
                u32x4 v = u32x4{0u, 0u, 0u, 0u};
                if (e < E && kw < H) v = *reinterpret_cast<const u32x4*>(w + (size_t)e * H + kw);
                wr[s][b2] = v;
            }
        }
    };

    // workgroups start at different slices of the hidden dimension: the rows of x
    // and of the router weight lie a whole row apart, so workgroups that walk the
    // slices in step would all ask the same few memory channels at a time
    const int rot = (int)((blockIdx.x * 7u) % (unsigned)nchunks);
    auto slice_of = [&](int c) { const int cc = c + rot; return cc >= nchunks ? cc - nchunks : cc; };
    if (wave < nchunks) load_chunk(slice_of(wave));
    for (int c = wave; c < nchunks; c += 4) {
        bf16x8 bfrag[KSTEPS][NB];
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            *reinterpret_cast<u32x4*>(&xs[wave][i * RPI + lrow][lcol]) = xr[i];
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s)
#pragma unroll
            for (int b2 = 0; b2 < NB; ++b2) bfrag[s][b2] = __builtin_bit_cast(bf16x8, wr[s][b2]);
        if (c + 4 < nchunks) load_chunk(slice_of(c + 4));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
#pragma unroll
            for (int a = 0; a < MB; ++a) {
                const u32x4 av = *reinterpret_cast<const u32x4*>(&xs[wave][a * 16 + fr][s * 32 + fg * 8]);
                const bf16x8 afrag = __builtin_bit_cast(bf16x8, av);
#pragma unroll
                for (int b2 = 0; b2 < NB; ++b2)
                    acc[a][b2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afrag, bfrag[s][b2], acc[a][b2], 0, 0, 0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // fold the four partial sums in wave order 0,1,2,3 (fixed => reproducible)
    for (int ww = 0; ww < 4; ++ww) {
        if (wave == ww) {
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float* p = &red[a * 16 + fg * 4 + r][b * 16 + fr];
                        *p = (ww == 0) ? acc[a][b][r] : (*p + acc[a][b][r]);
                    }
        }
        __syncthreads();
    }
    // bias, write logits
    for (int i = threadIdx.x; i < TOK * E; i += 256) {
        const int lt = i / E, e = i - lt * E;
        float v = red[lt][e];
        if (bias) v += bias[e];
        red[lt][e] = v;
        if (t0 + lt < T) logits[(size_t)(t0 + lt) * E + e] = v;
    }
    __syncthreads();
    select_tokens(&red[0][0], EP + 1, TOK, t0, T, E, K, renorm, topk_idx, topk_gate);
}

// ------------------------------------------------------------------ bf16 / MFMA, many experts and few tokens
// A compute unit reads about 40 bytes per nanosecond here, whatever is in flight, and the kernel above has one workgroup
// read the whole router weight: 64 experts x 3584 is 460 KB, 11 us for a single token.  So with few tokens the experts
// are spread over workgroups too (blockIdx.y): a workgroup forms the logits of at most 16 MB tokens (tb of them used)
// and 16 experts (eg used), and the selection, which needs all experts of a token, is a launch of its own
// (topk_rank_kernel).  The 16 waves split the hidden dimension, U steps of 64 elements in flight each; operands go
// straight from memory to the matrix instruction's registers (lane group j holds bytes 32 j .. 32 j + 31 of a 128-byte
// step of both, so whole lines are asked for; the order inside a step plays no part in a dot product).  The partial
// sums are added in wave order (fixed => reproducible).
// SELECT (E <= 16: a workgroup holds all logits of its tokens): the selection as well, sixteen lanes per token.
// PLAN (one workgroup, tb <= kPlanTokens tokens): the dispatch too, whose own launch is as long as its work then.  A lane of the
// first wave holds an assignment (at most 4 tokens x 16 experts): its row is the number of kept ones of lower experts and of its
// own expert's lower assignments.  The token rows are requested before the plan is made.  Maps as launch_permute's, bit for bit.
constexpr int kSplitWaves = 16, kPlanTokens = 4;

struct Dispatch {
    int32_t *counts, *offsets, *row_of_assign, *assign_of_row, *one_expert;
    uint8_t* x_perm;
    int capacity, r_max;
};

template <int MB, bool SELECT, bool PLAN = false>
__global__ __launch_bounds__(kSplitWaves * 64) void router_logits_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, const float* __restrict__ bias,
    float* __restrict__ logits, int T, int H, int E, int tb, int eg, int K, int renorm,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate, Dispatch d) {
    static_assert(SELECT || !PLAN, "the dispatch follows the selection");
    constexpr int LD = 20;                     // row of a partial tile: the four lane groups of a store hit different banks
    constexpr int U = MB == 1 ? 4 : 3;         // steps in flight
    static_assert(MB == 1 || !SELECT, "the lanes that sum a token's logits are the first turn's");
    __shared__ float part[kSplitWaves][16 * MB][LD];
    __shared__ int sel[PLAN ? 64 : 1];         // the expert of an assignment, then its row
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = blockIdx.x * tb, e0 = blockIdx.y * eg;
    const int fr = lane & 15, fg = lane >> 4;
    const int nsteps = (H + 63) / 64;
    // rows and experts past the workgroup's repeat its last one (the same lines) and are never stored
    const bf16_t* xrow[MB];
#pragma unroll
    for (int a = 0; a < MB; ++a) xrow[a] = x + (size_t)min(t0 + min(a * 16 + fr, tb - 1), T - 1) * H;
    const bf16_t* const wrow = w + (size_t)min(e0 + min(fr, eg - 1), E - 1) * H;
    f32x4 acc[MB];
#pragma unroll
    for (int a = 0; a < MB; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = wave; s0 < nsteps; s0 += U * kSplitWaves) {
        u32x4 xa[U][MB][2], wa[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int k = (s0 + u * kSplitWaves) * 64 + fg * 16 + p * 8;
                const bool in = k < H;         // H is a multiple of 8: a piece is in or out as a whole
                wa[u][p] = u32x4{0u, 0u, 0u, 0u};
                if (in) wa[u][p] = *reinterpret_cast<const u32x4*>(wrow + k);
#pragma unroll
                for (int a = 0; a < MB; ++a) {
                    xa[u][a][p] = u32x4{0u, 0u, 0u, 0u};
                    if (in) xa[u][a][p] = *reinterpret_cast<const u32x4*>(xrow[a] + k);
                }
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int a = 0; a < MB; ++a)
                    acc[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[u][a][p]),
                                                                     __builtin_bit_cast(bf16x8, wa[u][p]), acc[a], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][a * 16 + fg * 4 + r][fr] = acc[a][r];
    const int row_bytes = 2 * H, at = 16 * (int)threadIdx.x;   // PLAN: a row has at most 16 bytes for every thread
    u32x4 mine[PLAN ? kPlanTokens : 1];
    if constexpr (PLAN)
#pragma unroll
        for (int t = 0; t < kPlanTokens; ++t)
            if (t < T && at < row_bytes) mine[t] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(x) + (size_t)t * row_bytes + at);
    __syncthreads();
    for (int i = threadIdx.x; i < 16 * MB * 16; i += kSplitWaves * 64) {
        const int lt = i >> 4, le = i & 15;
        if (lt >= tb || le >= eg || t0 + lt >= T || e0 + le >= E) continue;
        float v = part[0][lt][le];
#pragma unroll
        for (int ww = 1; ww < kSplitWaves; ++ww) v += part[ww][lt][le];
        if (bias) v += bias[e0 + le];
        logits[(size_t)(t0 + lt) * E + e0 + le] = v;
        if (SELECT) part[0][lt][le] = (v != v) ? -INFINITY : v;   // NaN ranks last; read back by its own wave's lanes only
    }
    if constexpr (SELECT) {
        // the sixteen lanes that summed a token's logits select its experts: the rank of an expert is the number of experts in
        // front of it (value descending, index ascending), as in topk_rank_kernel
        const int lt = threadIdx.x >> 4, le = lane & 15;
        if (lt < tb && t0 + lt < T) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const float v = le < E ? part[0][lt][le] : -INFINITY;
            float m = v;
            int rank = 0;
            for (int e = 0; e < E; ++e) {
                const float s = part[0][lt][e];
                rank += e < le ? s >= v : s > v;
                m = fmaxf(m, s);
            }
            float p = le < E ? expf(v - m) : 0.f, z = p;
            for (int off = 8; off > 0; off >>= 1) z += __shfl_xor(z, off, 16);
            p = p / z;
            const bool chosen = le < E && rank < K;
            float gsum = chosen ? p : 0.f;
            if (renorm)
                for (int off = 8; off > 0; off >>= 1) gsum += __shfl_xor(gsum, off, 16);
            if (chosen) {
                topk_idx[(size_t)(t0 + lt) * K + rank] = le;
                topk_gate[(size_t)(t0 + lt) * K + rank] = renorm ? p / gsum : p;
                if constexpr (PLAN) sel[lt * K + rank] = le;
            }
        }
    }
    if constexpr (PLAN) {
        __syncthreads();
        const int A = T * K;
        if (wave == 0) {
            const int e = lane < A ? sel[lane] : -1, limit = d.capacity > 0 ? d.capacity : A;
            const uint64_t below = lane == 0 ? 0ull : ~0ull >> (64 - lane);
            int row = -1, total = 0, count = 0, end = 0;
            for (int q = 0; q < E; ++q) {
                const uint64_t peers = __ballot(e == q);
                const int n = min(__popcll(peers), limit), rank = __popcll(peers & below);
                if (e == q && rank < limit && total + rank < d.r_max) row = total + rank;   // r_max holds all rows that are kept
                total += n;
                if (lane == q) {
                    count = n;
                    end = total;
                }
            }
            sel[lane] = row;
            if (lane < E) {
                d.counts[lane] = count;
                d.offsets[lane + 1] = end;
            }
            if (lane == 0) {
                d.offsets[0] = 0;
                if (d.one_expert != nullptr) {
                    d.one_expert[0] = 0;
                    d.one_expert[1] = T;
                }
            }
            if (lane < A) d.row_of_assign[lane] = row;
            if (row >= 0) d.assign_of_row[row] = lane;
            for (int r = total + lane; r < d.r_max; r += 64) d.assign_of_row[r] = -1;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < kPlanTokens; ++t)
            if (t < T && at < row_bytes)
                for (int k = 0; k < K; ++k) {
                    const int row = sel[t * K + k];
                    if (row >= 0) *reinterpret_cast<u32x4*>(d.x_perm + (size_t)row * row_bytes + at) = mine[t];
                }
    }
}

// ------------------------------------------------------------------ bf16 / MFMA, many experts and many tokens
// TM tokens x TE experts a workgroup, both operands through one ring of LDS stages (64 elements of the TM + TE rows, direct
// global-to-LDS loads, rows swizzled as in the grouped GEMMs).  What bounds it is what a compute unit takes in, (TM + TE) rows
// for TM x TE logits, so both sides are tall; router_bf16_kernel reads all experts for 16 to 64 tokens.  The four waves
// share the 32 x 32 blocks, or split a stage's contraction where there are fewer than four (the partial sums are added in
// wave order).  SELECT: TE >= E, and the workgroup selects for its tokens.  H is a multiple of 64.
template <int TM, int TE>
constexpr int router_tile_stages() {
    constexpr int per = (TM + TE) / 32, fit = 144 * 1024 / ((TM + TE) * 128);
    return fit < 8 ? fit : per * 6 < 64 ? 8 : 63 / per + 2;
}

template <int TM, int TE, bool SELECT>
__global__ __launch_bounds__(256) void router_tile_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, const float* __restrict__ bias,
    float* __restrict__ logits, int T, int H, int E, int K, int renorm,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate) {
    constexpr int PER = (TM + TE) / 32;                 // direct loads per thread and stage: 32 rows each
    constexpr int STAGE = (TM + TE) * 128;
    constexpr int S = router_tile_stages<TM, TE>();
    constexpr int NTE = TE / 32, NT = TM / 32 * NTE;    // 32 x 32 blocks
    constexpr int KS = NT >= 4 ? 1 : 4 / NT;            // waves that share a block's contraction
    constexpr int BPW = NT >= 4 ? NT / 4 : 1;           // blocks per wave, of the same tokens
    constexpr int LD = TE + 1;
    static_assert(S >= 3 && (S - 2) * PER < 64 && BPW <= NTE && TM * LD * 4 <= S * STAGE, "ring");
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * TM, e0 = blockIdx.y * TE;
    const int block = KS == 1 ? wave * BPW : wave % NT, ks = KS == 1 ? 0 : wave / NT;
    const int tm = block / NTE, te = block % NTE;

    // load q covers rows 32 q .. 32 q + 31 of the stage: the tokens, then the experts (the last one again past the end)
    const uint8_t* src[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int row = 32 * q + (tid >> 3);
        const bf16_t* r = 32 * q < TM ? x + (size_t)min(t0 + row, T - 1) * H : w + (size_t)min(e0 + row - TM, E - 1) * H;
        src[q] = reinterpret_cast<const uint8_t*>(r) + 16 * ((tid & 7) ^ lds_swizzle(row));
    }
    const int nst = H / 64;
    const int rot = (int)(((blockIdx.x + blockIdx.y * 5u) * 7u) % (unsigned)nst);   // see router_bf16_kernel
    auto issue = [&](int slot, int s) {
        int sr = s + rot;
        sr = sr >= nst ? sr - nst : sr;
        const size_t k = s >= nst ? 0 : (size_t)sr * 128;   // past the last stage: the first again, never used
#pragma unroll
        for (int q = 0; q < PER; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[q] + k),
                                             (__attribute__((address_space(3))) void*)(smem + slot * STAGE + (q * 32 + wave * 8) * 128),
                                             16, 0, 0);
    };
    // A logit is the sum of several separate sums (at least 4, 16 for the smallest tile), as in the kernels for fewer tokens: one
    // sum over the whole row doubles the error (20882 tokens, 5760 x 128, against 64 bits: one sum 4.7e-7, so 1.6e-7; the kernel for
    // fewer experts 2.3e-7).
    constexpr int Q = 4 / KS;                                       // of a stage's four steps, this wave's
    constexpr int U = KS > 1 ? 4 : BPW == 1 ? 2 : 1;                // stages that follow one another in sums of their own
    f32x16 acc[U][Q][BPW];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int b = 0; b < BPW; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[u][q][b][v] = 0.f;
    const int fr = lane & 31, fk = lane >> 5, sw = lds_swizzle(fr);
    const uint8_t* const xrow = smem + (tm * 32 + fr) * 128;
    const uint8_t* const wrow = smem + (TM + te * 32 + fr) * 128;
#pragma unroll
    for (int d = 0; d < S - 1; ++d) issue(d, d);
    int slot = 0, fill = S - 1;
    for (int s0 = 0; s0 < nst; s0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u >= nst) break;
            // this wave's loads of the stage have landed, its reads of the stage before are in registers
            constexpr int W = (S - 2) * PER;
            __builtin_amdgcn_s_waitcnt((W & 0xF) | ((W >> 4) << 14) | 0x70);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            issue(fill, s0 + u + S - 1);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int c = ((2 * (ks * Q + q) + fk) ^ sw) * 16;
                const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xrow + slot * STAGE + c));
#pragma unroll
                for (int b = 0; b < BPW; ++b) {
                    const bf16x8 e = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wrow + slot * STAGE + b * 4096 + c));
                    acc[u][q][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(e, a, acc[u][q][b], 0, 0, 0);
                }
            }
            slot = slot + 1 == S ? 0 : slot + 1;
            fill = fill + 1 == S ? 0 : fill + 1;
        }
    }
    // pairwise: the sums of a stage's steps, then those of successive stages
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
#pragma unroll
        for (int d = 1; d < Q; d *= 2)
#pragma unroll
            for (int q = 0; q < Q; q += 2 * d)
#pragma unroll
                for (int u = 0; u < U; ++u) acc[u][q][b] += acc[u][q + d][b];
#pragma unroll
        for (int d = 1; d < U; d *= 2)
#pragma unroll
            for (int u = 0; u < U; u += 2 * d) acc[u][0][b] += acc[u + d][0][b];
    }
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): nothing lands in the ring any more
    __syncthreads();
    // a lane holds token 32 tm + fr and, of each block, experts 8 q + 4 fk + 0 .. 3
    float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        if (ks == kk) {
#pragma unroll
            for (int b = 0; b < BPW; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float* p = red + (tm * 32 + fr) * LD + (te + b) * 32 + 8 * (v >> 2) + 4 * fk + (v & 3);
                    *p = kk == 0 ? acc[0][0][b][v] : *p + acc[0][0][b][v];
                }
        }
        __syncthreads();
    }
    const int cols = min(TE, E - e0);
    for (int i = tid; i < TM * cols; i += 256) {
        const int lt = i / cols, e = i - lt * cols;
        float v = red[lt * LD + e];
        if (bias) v += bias[e0 + e];
        if (SELECT) red[lt * LD + e] = v;
        if (t0 + lt < T) logits[(size_t)(t0 + lt) * E + e0 + e] = v;
    }
    if constexpr (SELECT) {
        __syncthreads();
        select_tokens(red, LD, TM, t0, T, E, K, renorm, topk_idx, topk_gate);
    }
}

// Selection by rank, one wave per token: lane l holds the logits of experts l, l + 64, ..; the rank of an expert is the
// number of experts in front of it (value descending, index ascending), counted against every logit in turn, and the
// experts of rank < K write the slots.  No sorted lists, so the chain of dependent instructions is short: what counts
// when there are too few tokens to fill the chip (7 us of the list form's time at 64 experts was that chain).
// E <= 64 VPL.
template <int VPL>
__global__ __launch_bounds__(256) void topk_rank_kernel(const float* __restrict__ logits, int T, int E, int K,
                                                        int renorm, int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_gate) {
    const int lane = threadIdx.x & 63;
    const int t = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (t >= T) return;
    float v[VPL];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        const int e = lane + 64 * j;
        const float l = e < E ? logits[(size_t)t * E + e] : -INFINITY;
        v[j] = (l != l) ? -INFINITY : l;   // NaN ranks last
        m = fmaxf(m, v[j]);
    }
    int rank[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) rank[j] = 0;
#pragma unroll
    for (int q = 0; q < VPL; ++q)
#pragma unroll
        for (int i0 = 0; i0 < 64; i0 += 16) {
            if (64 * q + i0 >= E) break;   // uniform; the padding up to the next multiple of 16 ranks behind everything
#pragma unroll
            for (int i = i0; i < i0 + 16; ++i) {
                const float s = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v[q]), i));
#pragma unroll
                for (int j = 0; j < VPL; ++j) {
                    const bool lower = j > q || (j == q && lane > i);   // expert 64 q + i has the lower index
                    rank[j] += lower ? s >= v[j] : s > v[j];
                }
            }
        }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    float p[VPL], z = 0.f;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        p[j] = lane + 64 * j < E ? expf(v[j] - m) : 0.f;
        z += p[j];
    }
    for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off, 64);
    float gsum = 0.f;
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        p[j] = p[j] / z;
        if (lane + 64 * j < E && rank[j] < K) gsum += p[j];
    }
    if (renorm)
        for (int off = 32; off > 0; off >>= 1) gsum += __shfl_xor(gsum, off, 64);
#pragma unroll
    for (int j = 0; j < VPL; ++j) {
        const int e = lane + 64 * j;
        if (e < E && rank[j] < K) {
            topk_idx[(size_t)t * K + rank[j]] = e;
            topk_gate[(size_t)t * K + rank[j]] = renorm ? p[j] / gsum : p[j];
        }
    }
}

// ------------------------------------------------------------------ fp32 / VALU
// A wave forms the logits of TW tokens; lanes stride the hidden dimension, eight experts at a time: their weight loads
// are in flight together, and the eight sums are folded across the wave in ten shuffles (three halving steps that leave
// lane l with the sum of expert l mod 8 over an eighth of the wave, then three ordinary ones).  WT waves share a
// token's experts, eight at a time in turn.  A sum's order is the same at every TW and WT.
// With few tokens a chain of loads bounds it (a block of experts waits for the block before it: WT waves walk E / 8 WT of
// them), with many the weight's way from the caches (TW tokens share a load).  Further steps of the hidden dimension in
// flight in a wave came out slower (256 x 828 x 16: 8.1 us for 7.5).
template <int TW, int WT>
__global__ __launch_bounds__(256) void router_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    float* __restrict__ logits, int T, int H, int E, int K, int renorm,
    int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate) {
    constexpr int EB = 8, NT = 4 / WT * TW;
    __shared__ float red[NT][kMaxExperts + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = blockIdx.x * NT, slot = wave / WT * TW;
    const int t = t0 + slot;
    if (t < T) {
        const float* xr[TW];
#pragma unroll
        for (int u = 0; u < TW; ++u) xr[u] = x + (size_t)min(t + u, T - 1) * H;
        for (int e0 = wave % WT * EB; e0 < E; e0 += EB * WT) {
            float s[TW][EB];
#pragma unroll
            for (int u = 0; u < TW; ++u)
#pragma unroll
                for (int j = 0; j < EB; ++j) s[u][j] = 0.f;
            for (int h = lane * 4; h < H; h += 256) {
                f32x4 a[TW], b[EB];
#pragma unroll
                for (int u = 0; u < TW; ++u) a[u] = *reinterpret_cast<const f32x4*>(xr[u] + h);
#pragma unroll
                for (int j = 0; j < EB; ++j) b[j] = *reinterpret_cast<const f32x4*>(w + (size_t)min(e0 + j, E - 1) * H + h);
#pragma unroll
                for (int u = 0; u < TW; ++u)
#pragma unroll
                    for (int j = 0; j < EB; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q) s[u][j] = fmaf(a[u][q], b[j][q], s[u][j]);
            }
#pragma unroll
            for (int u = 0; u < TW; ++u) {
#pragma unroll
                for (int n = EB / 2; n > 0; n >>= 1) {
                    const bool up = lane & n;   // this lane keeps the upper half of the values it still holds
#pragma unroll
                    for (int j = 0; j < n; ++j) {
                        const float keep = up ? s[u][j + n] : s[u][j], give = up ? s[u][j] : s[u][j + n];
                        s[u][j] = keep + __shfl_xor(give, n, 64);
                    }
                }
                float v = s[u][0];
#pragma unroll
                for (int off = EB; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
                const int e = e0 + lane;
                if (lane < EB && e < E && t + u < T) {
                    if (bias) v += bias[e];
                    red[slot + u][e] = v;
                    logits[(size_t)(t + u) * E + e] = v;
                }
            }
        }
    }
    __syncthreads();
    select_tokens(&red[0][0], kMaxExperts + 1, NT, t0, T, E, K, renorm, topk_idx, topk_gate);
}

// ------------------------------------------------------------------ selection only
constexpr int kTopkTileFloats = 12288;

// tokens per tile of the selection-only kernel: one pass of the workgroup
__host__ __device__ inline int topk_tile_tokens(int E, int K) {
    if (K <= 8) return 256 / lanes_per_token(E);
    const int fit = kTopkTileFloats / (E | 1);
    return fit > 256 ? 256 : fit;
}

__global__ __launch_bounds__(256) void topk_only_kernel(const float* __restrict__ logits, int T,
                                                        int E, int K, int renorm,
                                                        int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_gate) {
    // a tile of tokens is copied to LDS with coalesced loads (row stride odd),
    // then selected from there
    __shared__ float tile[kTopkTileFloats];
    const int ld = E | 1;
    const int per_block = topk_tile_tokens(E, K);
    for (int t0 = blockIdx.x * per_block; t0 < T; t0 += gridDim.x * per_block) {
        const int ntok = min(per_block, T - t0);
        const float* src = logits + (size_t)t0 * E;
        for (int i = threadIdx.x; i < ntok * E; i += 256) {
            const int lt = i / E, e = i - lt * E;
            tile[lt * ld + e] = src[i];
        }
        __syncthreads();
        select_tokens(tile, ld, ntok, t0, T, E, K, renorm, topk_idx, topk_gate);
        __syncthreads();
    }
}

template <int MB, int NB>
void launch_bf16(const void* x, const void* w, const float* bias, float* logits, int T, int H, int E,
                 int K, int renorm, int32_t* idx, float* gate, hipStream_t s) {
    const int grid = (T + 16 * MB - 1) / (16 * MB);
    hipLaunchKernelGGL((router_bf16_kernel<MB, NB>), dim3(grid), dim3(256), 0, s,
                       static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w), bias, logits, T,
                       H, E, K, renorm, idx, gate);
}

template <int TM, int TE, bool SELECT>
void launch_tile(const void* x, const void* w, const float* bias, float* logits, int T, int H, int E, int K, int renorm,
                 int32_t* idx, float* gate, hipStream_t s) {
    constexpr int smem = router_tile_stages<TM, TE>() * (TM + TE) * 128;
    auto kern = router_tile_kernel<TM, TE, SELECT>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), smem);
    hipLaunchKernelGGL(kern, dim3((T + TM - 1) / TM, (E + TE - 1) / TE), dim3(256), smem, s, static_cast<const bf16_t*>(x),
                       static_cast<const bf16_t*>(w), bias, logits, T, H, E, K, renorm, idx, gate);
}

}  // namespace

// Where the experts are spread over workgroups (one launch before / logits + selection after, us, H = 3584):
// (inside the layer, 64 tokens of the Qwen2 shape: 33 / 10)
//   64 experts:  1 token 23.1 / 7.2, 64 tokens 24.4 / 9.0, 500 tokens 24.7 / 11.6, 2048 tokens 26.9 / 18.7, 4096 27.8 / 31.6
//   128 experts x 2048:  1 token 31.3 / 8.6, 2048 tokens 37.1 / 24.8, 4096 tokens 36.6 / 41.5
// Inside a layer with a small expert FFN (us of the layer; 64 and 2048 tokens):
//   8 experts x 1024  26.1 / 26.4, 45.2 / 46.3     12 x 1000  27.7 / 26.4, 49.5 / 48.4     8 x 3072  35.1 / 33.7, 74.0 / 73.5
//   8 x 3584          38.4 / 36.3, 90.5 / 91.2      8 x 4096  40.9 / 38.3, 98.0 / 96.6    64 x 512   33.5 / 27.4, 64.2 / 58.6
// The line lies at 64 KB of router weight, from where on the two launches are ahead for every number of tokens; below, down to
// some 24 KB, they are by up to 3 us for most.
constexpr int kSplitMaxTokens = 2048, kSplitMinWeights = 32768;
// Up to 16 experts, logits and selection in one launch of the split kernel (us, H x experts; the kernel for many tokens / logits +
// selection / so): 4096 x 8, 1 token 8.3 / 6.7 / 5.8, 64 tokens 8.6 / 7.3 / 6.2, 2048 11.2 / 10.5 / 7.9, 4096 14.2 / - / 9.5, 8192
// 21.2 / - / 19.3; 6144 x 8, 8192 tokens 25.2 / - / 27.9; 1000 x 12, 777 tokens 7.1 / 6.3 / 4.2; 1600 x 16, 11500 14.8 / - / 15.3.
// With a large router weight few tokens are better off with the experts spread (logits + selection / so: 6 tokens, 6144 x 16 1.5 us
// less; 4096 x 16, 1 token 6.6 / 7.2, 64 tokens 7.4 / 7.8, 130 8.2 / 7.9; 5376 x 12, 1 token 7.4 / 7.9, 64 tokens 8.6 / 8.5; 7168 x 8,
// 1 token 7.8 / 8.0, 8 tokens 9.2 / 8.5; 16384 x 4, 30 tokens 15.5 / 13.4): of more than eight experts up to 64 tokens from 57344
// weights on, of any number up to 512 tokens from 65536.
constexpr int kOneBlockMaxTokens = 4096;
static bool one_block_pays(int T, int H, int E) {
    return T <= kOneBlockMaxTokens && (T > 512 || (long long)E * H <= (T <= 64 && E > 8 ? 57344 : 65536));
}
// router_tile_kernel, from so many logits on (us in the layer, the kernels before / so): 2048 tokens, 6144 x 64 24.8 / 19.8, 1400,
// 5248 x 128 34.4 / 15.5, 1473, 4096 x 60 16.4 / 12.3, 3684, 6784 x 64 53 / 25 + 7 for the selection, 4164, 5248 x 64 44 / 32, 20882,
// 5760 x 128 239 / 127 + 24; 905, 4032 x 64 10.9 / 11.8.
// Not for up to 64 experts from 32768 tokens on, where router_bf16_kernel takes 64 tokens a workgroup (alone): 32768 tokens, 2048 x 64
// 46 / 57, 4096 x 64 72 / 74, 7168 x 64 132 / 117; 40000, 4096 x 64 113 / 123; 49152, 4096 x 32 87 / 89; 65536, 2048 x 48 71 / 82,
// 6144 x 60 203 / 192.  Ahead only from some 5000 elements a row on, and not for every number of tokens.
// The tiles are behind where the other kernel's workgroups of 32 tokens just fit the chip and the rows are short, by up to a
// quarter at 1024 elements (alone): 64 experts, 12000 tokens 22.4 / 27.4; 32 experts, 20000 20.1 / 23.4; 72 experts, 6000 19.5 / 22.2;
// up to 2048 tokens by 0.4 (1024 x 128, 1024 tokens 11.4 / 11.7); and for 65 to 80 experts at 8192 tokens whatever the row (7168 x 72
// 49.4 / 53.3).  They are taken there as well: their logits are nearer to 64 bits (1024 elements 0.7 to 0.8 times the error, 4096
// and more 0.5 to 0.7).
constexpr long long kTileMinLogits = 80000;
struct RouterTile {
    int tokens, experts;
};
constexpr RouterTile kTiles[4] = {{32, 32}, {32, 64}, {64, 64}, {128, 64}};

// The tile with the least estimated time (us): rounds of workgroups at 45 bytes per nanosecond each, then the selection, in the
// workgroup (passes of 256 lanes, counted for the last round only) or a launch of its own.  No floor for what comes from memory:
// 32768 tokens, 4096 x 64 are estimated at 52 and take 74.  Alone, 3684 tokens, 6784 x 64: 28 / 34 / 50 / 82 for the four; 8192,
// 3584 x 64: 35 / 29 / 39 / 64; 22980, 5376 x 64: 102 / 96 / 97 / 90; 20882, 5760 x 128: 172 / 151 / 127 / 134 (the kernel before,
// 32 or 64 tokens x all experts: 47, 36, 106 and 212).
static int pick_tile(int T, int H, int E) {
    int best = 0;
    double least = 1e30;
    for (int i = 0; i < 4; ++i) {
        const RouterTile t = kTiles[i];
        const long long groups = (long long)((T + t.tokens - 1) / t.tokens) * ((E + t.experts - 1) / t.experts);
        const double select = E <= t.experts ? 1.0 + 4.0 * ((t.tokens * lanes_per_token(E) + 255) / 256) : 4.0 + 9.4e-6 * T * (double)E;
        const double us = (double)((groups + 255) / 256) * (t.tokens + t.experts) * (2.0 * H) / 45e3 + select;
        if (us < least) {
            least = us;
            best = i;
        }
    }
    return best;
}
// Selection alone, lists of eight lanes / by rank (us, 64 experts, K = 8): 1024 tokens 10.2 / 4.1, 4096 tokens 10.3 / 6.7,
// 16384 tokens 13.3 / 13.1; 128 experts 17.1 / 13.1 at 4096.
constexpr int kRankMaxTokens = 4096;

// selection from logits alone
static void launch_topk(const float* logits, int T, int E, int K, int renorm, int32_t* idx, float* gate, hipStream_t s) {
    if (E <= 128 && T <= kRankMaxTokens) {
        const dim3 grid((T + 3) / 4);
        if (E <= 64) hipLaunchKernelGGL((topk_rank_kernel<1>), grid, dim3(256), 0, s, logits, T, E, K, renorm, idx, gate);
        else hipLaunchKernelGGL((topk_rank_kernel<2>), grid, dim3(256), 0, s, logits, T, E, K, renorm, idx, gate);
        return;
    }
    const int per_block = topk_tile_tokens(E, K);
    int grid = (T + per_block - 1) / per_block;
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(topk_only_kernel, dim3(grid), dim3(256), 0, s, logits, T, E, K, renorm, idx, gate);
}

static int g_router_tile = 0;  // 16-token blocks per workgroup; 0 = chosen by size, 8 = experts spread over workgroups, 16 = tiles
void set_router_tile(int mb) { g_router_tile = mb; }

// Up to four tokens of up to 16 experts (us of the layer, two launches / so): 1024 x 8, F = 1024, 1 token 22.1 / 18.6, 4 tokens 22.8 /
// 21.5; 4096 x 8, F = 14336 139.8 / 137.9, 384.9 / 383.6; 1768 x 16, F = 1928 31.0 / 29.3, 73.3 / 72.3; 7168 x 8, F = 768 36.2 /
// 34.0, 45.8 / 45.7.  One compute unit reads and copies all the rows, so the gain is gone with more tokens.
bool launch_route_permute(const void* x, const void* w, const float* bias, float* logits, int T, int H, int E, int K, int renorm,
                          int capacity, int r_max, moe_dtype_t dt, int32_t* idx, float* gate, void* x_perm, int32_t* counts,
                          int32_t* offsets, int32_t* row_of_assign, int32_t* assign_of_row, int32_t* one_expert, hipStream_t s) {
    if (dt != MOE_BF16 || T > kPlanTokens || E > 16 || 2 * H > 16384 || g_router_tile != 0 || !one_block_pays(T, H, E)) return false;
    const Dispatch d = {counts, offsets, row_of_assign, assign_of_row, one_expert, static_cast<uint8_t*>(x_perm), capacity, r_max};
    hipLaunchKernelGGL((router_logits_kernel<1, true, true>), dim3(1), dim3(kSplitWaves * 64), 0, s, static_cast<const bf16_t*>(x),
                       static_cast<const bf16_t*>(w), bias, logits, T, H, E, kPlanTokens, 16, K, renorm, idx, gate, d);
    return true;
}

void launch_router(const void* x, const void* w, const float* bias, float* logits, int T, int H,
                   int E, int K, int renorm, moe_dtype_t dt, int32_t* idx, float* gate,
                   hipStream_t s) {
    if (x == nullptr) {
        launch_topk(logits, T, E, K, renorm, idx, gate, s);
        return;
    }
    if (dt == MOE_F32) {
        // (tokens per wave, waves per token), us, one token per wave / here: 64 x 828 x 8 experts 6.2 / 5.6; 256 x 828 x 16
        // 10.2 / 7.2; 256 x 1024 x 64 26.3 / 13.1; 2048 x 1024 x 64 31.3 / 21.4; 4096 x 1024 x 16 17.2 / 11.7; 6000 x 1024 x 8
        // 13.1 / 8.9; 16384 x 4096 x 8 86.4 / 52.0; 65536 x 512 x 8 74.0 / 30.5.  Four waves on a token lose above 1024
        // tokens (2048 x 1024 x 64 22.8) and with two blocks of experts or fewer (two of them idle), two waves above 4096
        // (6000 x 1024 x 8 11.6), and four tokens a wave below 8192 (6000 x 1024 x 8 9.9).
#define RF32(TW, WT)                                                                                                    \
    hipLaunchKernelGGL((router_f32_kernel<TW, WT>), dim3((T + 4 / WT * TW - 1) / (4 / WT * TW)), dim3(256), 0, s,       \
                       static_cast<const float*>(x), static_cast<const float*>(w), bias, logits, T, H, E, K, renorm,   \
                       idx, gate)
        if (T >= 8192) RF32(4, 1);
        else if (T > 4096) RF32(2, 1);
        else if (T > 1024 || E <= 16) RF32(2, 2);
        else RF32(2, 4);
#undef RF32
        return;
    }
    const int nb = (E + 15) / 16;
    const int tile = nb >= 2 && E <= 128 && H % 64 == 0 &&
                             (g_router_tile == 16 || (g_router_tile == 0 && (long long)T * E >= kTileMinLogits && !(T >= 32768 && E <= 64)))
                         ? pick_tile(T, H, E) : -1;
    if (tile >= 0) {
        const bool fused = E <= kTiles[tile].experts;
#define ROUTER_TILE(TM, TE)                                                                                              \
    if (fused) launch_tile<TM, TE, true>(x, w, bias, logits, T, H, E, K, renorm, idx, gate, s);                          \
    else launch_tile<TM, TE, false>(x, w, bias, logits, T, H, E, K, renorm, idx, gate, s);
        if (tile == 0) { ROUTER_TILE(32, 32) } else if (tile == 1) { ROUTER_TILE(32, 64) }
        else if (tile == 2) { ROUTER_TILE(64, 64) } else { ROUTER_TILE(128, 64) }
#undef ROUTER_TILE
        if (!fused) launch_topk(logits, T, E, K, renorm, idx, gate, s);
        return;
    }
    if (nb == 1 && g_router_tile == 0 && one_block_pays(T, H, E)) {
        // all experts in a workgroup; tokens per workgroup: as few as leave every workgroup a compute unit (16 at the most tokens)
        static_assert(kOneBlockMaxTokens <= 16 * 256, "a workgroup of router_logits_kernel<1> holds 16 tokens");
        int tb = 16;
        while (tb > 2 && (T + tb / 2 - 1) / (tb / 2) <= 256) tb /= 2;
        const dim3 grid((T + tb - 1) / tb);
        hipLaunchKernelGGL((router_logits_kernel<1, true>), grid, dim3(kSplitWaves * 64), 0, s, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w), bias,
                           logits, T, H, E, tb, 16, K, renorm, idx, gate, Dispatch{});
        return;
    }
    if (nb <= 8 && (g_router_tile == 8 || (g_router_tile == 0 && T <= kSplitMaxTokens && (long long)E * H >= kSplitMinWeights))) {
        // Tokens and experts per workgroup: halve the larger side while that still gives every workgroup a compute unit
        const bool wide = T >= 1024;
        int tb = wide ? 32 : 16, eg = 16;
        auto groups = [&](int a, int b) { return (long long)((T + a - 1) / a) * ((E + b - 1) / b); };
        while (eg > 2) {
            const int a = min(tb, T), ntb = a > eg ? tb / 2 : tb, neg = a > eg ? eg : eg / 2;
            if (groups(ntb, neg) > 256) break;
            tb = ntb;
            eg = neg;
        }
        const dim3 grid((T + tb - 1) / tb, (E + eg - 1) / eg);
        if (tb > 16)
            hipLaunchKernelGGL((router_logits_kernel<2, false>), grid, dim3(kSplitWaves * 64), 0, s, static_cast<const bf16_t*>(x),
                               static_cast<const bf16_t*>(w), bias, logits, T, H, E, tb, eg, K, renorm, idx, gate, Dispatch{});
        else
            hipLaunchKernelGGL((router_logits_kernel<1, false>), grid, dim3(kSplitWaves * 64), 0, s, static_cast<const bf16_t*>(x),
                               static_cast<const bf16_t*>(w), bias, logits, T, H, E, tb, eg, K, renorm, idx, gate, Dispatch{});
        launch_topk(logits, T, E, K, renorm, idx, gate, s);
        return;
    }
    // tokens per workgroup: enough workgroups to fill 256 CUs, but from 16
    // experts on a taller tile so the router weight is re-read less often
    int mb = (T >= 32768) ? 4 : (T >= 16384 ? 2 : 1);
    if (E >= 16 && mb < 2) mb = 2;
    if (g_router_tile == 1 || g_router_tile == 2 || g_router_tile == 4) mb = g_router_tile;
#define ROUTER_CASE(M, N)                                                          \
    launch_bf16<M, N>(x, w, bias, logits, T, H, E, K, renorm, idx, gate, s);       \
    return;
    if (nb <= 1) {
        if (mb == 4) { ROUTER_CASE(4, 1) } else if (mb == 2) { ROUTER_CASE(2, 1) } else { ROUTER_CASE(1, 1) }
    } else if (nb <= 2) {
        if (mb == 4) { ROUTER_CASE(4, 2) } else if (mb == 2) { ROUTER_CASE(2, 2) } else { ROUTER_CASE(1, 2) }
    } else if (nb <= 4) {
        if (mb == 4) { ROUTER_CASE(4, 4) } else if (mb == 2) { ROUTER_CASE(2, 4) } else { ROUTER_CASE(1, 4) }
    } else if (nb <= 8) {
        ROUTER_CASE(2, 8)
    } else {
        ROUTER_CASE(1, 16)
    }
#undef ROUTER_CASE
}

}  // namespace moe
