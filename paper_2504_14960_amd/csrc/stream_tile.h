// Pieces shared by the weight-streaming kernels (gemm_stream.hip) and the small tiles (gemm_tiles.hip): the tile of a workgroup,
// where it starts in its contraction, loads of the operands, the epilogue.
//
// MODE of the kernels: 0 one product, 1 the SwiGLU pair, 2 the pair with its pre-activations stored too, 3 as 1 for the shapes
// that the persistent large tiles do not take (see silu_mul)
#pragma once

#include "fp8_convert.h"
#include "gemm_stream.h"
#include "gemm_tile.h"

namespace moe {

struct StreamArgs {
    const uint8_t* A;
    const int32_t* offsets;
    const uint8_t* B0;
    const uint8_t* B1;
    void* C;
    void* GU;
    float* amax;
    unsigned long long* ticks;   // clock sample of workgroup 0, or null
    float s0, s1, s2;
    int E, N, kbytes, ntn;
    int units, S, r_max;   // wide kernel: 32-row units per tile, splits of the contraction; rows of a partial plane
    float* part;           // split partial sums [S][r_max][N, or 2 N with SwiGLU], or null
};

// the small tiles (gemm_tiles.hip)
void launch_tiles(int elt, const StreamArgs& p, int form, int r_max, hipStream_t s);
// bf16 shapes whose silu has the full expf and divide (see silu_mul)
inline bool full_silu(const StreamArgs& p) { return p.N % 64 || p.kbytes % 128 || p.kbytes < 256; }

namespace {

// The tile of a workgroup, as find_tile orders them, worked out by every wave for itself with its lanes (lane l: experts 4 l ..
// 4 l + 3): one read of the offsets, no LDS and no barrier in front of the first load of the operands.  The LDS form reads the
// tile's two offsets from memory once more and meets two barriers; a launch of one round of workgroups shows all of it (us of
// the layer: 256 fp32 tokens, 128 x 256 27.0 / 25.7; one token of Mixtral-8x7B 141.9 / 140.0; FP8, 32 tokens 276.7 / 274.8).
template <int BM>
__device__ __forceinline__ Tile locate_tile(const int32_t* __restrict__ offsets, int E, int ntn, unsigned block) {
    constexpr int MG = 8;
    const int lane = threadIdx.x & 63;
    int lo[5], mt[4], s = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j) lo[j] = offsets[min(4 * lane + j, E)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        mt[j] = max(0, (lo[j + 1] - lo[j] + BM - 1) / BM);
        s += mt[j];
    }
    int incl = s;
    for (int d = 1; 4 * d < E; d <<= 1) {   // lanes past the last expert have nothing to add
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    Tile t;
    t.valid = false;
    t.expert = 0; t.row0 = 0; t.rows = 0; t.row_end = 0; t.ntile = 0;
    const int MT = __builtin_amdgcn_readlane(incl, (E - 1) >> 2);
    const int total = MT * ntn, per = (total + 7) / 8;
    const int j = (int)(block >> 3), L = (int)(block & 7) * per + j;
    if (j >= per || L >= total) return t;
    const int qm = L / ntn;
    int hit = -1, my_p = 0, my_mt = 0, my_lo = 0, my_hi = 0, p = incl - s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (p <= qm && qm < p + mt[q]) {
            hit = q; my_p = p; my_mt = mt[q]; my_lo = lo[q]; my_hi = lo[q + 1];
        }
        p += mt[q];
    }
    // the M-tile ranges of the experts partition [0, MT): exactly one lane (those past the last expert hold empty ones)
    const int src = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)__ballot(hit >= 0)) - 1);
    const int p_e = __builtin_amdgcn_readlane(my_p, src), mt_e = __builtin_amdgcn_readlane(my_mt, src);
    const int row_lo = __builtin_amdgcn_readlane(my_lo, src);
    t.expert = 4 * src + __builtin_amdgcn_readlane(hit, src);
    t.row_end = __builtin_amdgcn_readlane(my_hi, src);
    // the expert's M-tiles in groups of nearly equal size (see find_tile)
    const int Le = L - p_e * ntn;
    const int ng = (mt_e + MG - 1) / MG, gbase = mt_e / ng, grem = mt_e % ng;
    const int big = grem * (gbase + 1) * ntn;
    const bool first = Le < big;
    const int gsz = first ? gbase + 1 : gbase, at = first ? Le : Le - big;
    const int g = at / (gsz * ntn), rem = at - g * gsz * ntn;
    const int n = rem / gsz, m = (first ? 0 : grem * (gbase + 1)) + g * gsz + rem - n * gsz;
    t.row0 = row_lo + m * BM;
    t.rows = min(BM, t.row_end - t.row0);
    t.ntile = n;
    t.valid = true;
    return t;
}

// What a lane holds of a 128-byte k-step of one operand row: lane group j = lane / 16 of row lane % 16 holds the 32 bytes
// from 32 j (two 16-byte loads; the four groups together ask for the row's whole line).  The contraction order inside a step
// is the same for both operands, so any assignment of bytes to contraction slots is right.
struct Piece {
    u32x4 lo, hi;
};

// 16 bytes of global memory (the pointer arithmetic below hides from the compiler where its pointers point)
__device__ __forceinline__ u32x4 ld16(const uint8_t* p) {
    return *(const __attribute__((address_space(1))) u32x4*)p;
}

// Where a workgroup starts in its n steps of the contraction.  Operand rows lie a whole row apart, so workgroups that
// walk the contraction in step ask the same few memory channels at a time.  The order of a row's sum is thus that of its
// weight tile and expert, and beyond that of the form: the number of rows in its tile, and the plan, which follows r_max.  The
// same call gives the same bits; another batch around a row may not.  Measured (us, all from step 0 / so): down 4096 x 14336,
// 2 experts x 8 rows 51.0 / 44.6, 8 experts x 32 rows 187.7 / 175.1; gate/up 1408 x 2048, 16 experts x 8 rows 43.2 / 38.7.
__device__ __forceinline__ int rotation(const Tile& t, int n) {
    return n > 0 ? __builtin_amdgcn_readfirstlane((int)((unsigned)(t.ntile * 3 + t.expert * 5) % (unsigned)n)) : 0;
}

// One lane's piece of a row's last, partial 128-byte block: bytes past the row's end count as zeros (`row`: the row at
// the block's start; rem: bytes left, a multiple of 16).
__device__ __forceinline__ Piece tail_piece(const uint8_t* row, int j, int rem) {
    const bool lo_in = 32 * j < rem, hi_in = 32 * j + 16 < rem;
    Piece v;
    v.lo = ld16(row + (lo_in ? 32 * j : 0));
    v.hi = ld16(row + (hi_in ? 32 * j + 16 : 0));
    if (!lo_in) v.lo = u32x4{0u, 0u, 0u, 0u};
    if (!hi_in) v.hi = u32x4{0u, 0u, 0u, 0u};
    return v;
}

// silu(g) * u as the persistent large tiles form it for the shapes they take, with the fast exponential and reciprocal; for
// the rest (fp32; MODE 3: H or F not a multiple of 64, or H = 64) with the full expf and divide of the plain FMA kernel:
// the fast exponential's error grows with |g|, some 40 units in the last place at g = -60.  (gate/up of 2331 rows on 12
// experts, 1000 x 1416: 50.4 us with the fast form, 51.6 with the full one.)
template <int ELT, int MODE>
__device__ __forceinline__ float silu_mul(float g, float u) {
    if constexpr (ELT == kStreamF32 || MODE == 3) return (g / (1.f + expf(-g))) * u;
    else return g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * u;
}

// Stores four consecutive columns of a row (if `in`) from their sums: v (with SwiGLU the gate's) and up.  Returns the largest |h|
// stored (FP8).
template <int ELT, int MODE>
__device__ __forceinline__ float store_four(const StreamArgs& p, bool in, int row, int col, f32x4 v, f32x4 up) {
    constexpr bool SWIGLU = MODE != 0;
    const size_t at = (size_t)row * p.N + col;
    float amax = 0.f;
    if constexpr (SWIGLU) {
        if constexpr (ELT == kStreamFp8) { v *= p.s0; up *= p.s1; }
        if (MODE == 2 && in) {
            u32x2 g2 = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
            u32x2 u2 = {pack2_bf16(up[0], up[1]), pack2_bf16(up[2], up[3])};
            bf16_t* gu = static_cast<bf16_t*>(p.GU) + (size_t)row * (2 * p.N) + col;
            *reinterpret_cast<u32x2*>(gu) = g2;
            *reinterpret_cast<u32x2*>(gu + p.N) = u2;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = silu_mul<ELT, MODE>(v[q], up[q]);
    } else if constexpr (ELT == kStreamFp8) {
        v *= p.s0;
    }
    if (!in) return amax;
    if constexpr (ELT == kStreamF32) {
        *reinterpret_cast<f32x4*>(static_cast<float*>(p.C) + at) = v;
    } else if constexpr (ELT == kStreamFp8 && SWIGLU) {
#pragma unroll
        for (int q = 0; q < 4; ++q) amax = fmaxf(amax, fabsf(v[q]));
        *reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(p.C) + at) =
            f32x4_to_e4m3(v[0] * p.s2, v[1] * p.s2, v[2] * p.s2, v[3] * p.s2);
    } else {
        u32x2 o = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
        *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.C) + at) = o;
    }
    return amax;
}

// max |h| of the workgroup into *amax: one atomic per workgroup at most, and none if the value read is already as large
// (*amax only grows; as floats >= 0 compare like their bit patterns).  One per wave put thousands of them on one address
// at the end of the first round: gate/up of 32 tokens, 8 experts, 14336 x 4096, 200 us against 162 with *amax preset.
__device__ __forceinline__ void fold_amax(const StreamArgs& p, float amax, float* scratch) {
    if (!p.amax) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = amax;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (unsigned w = 1; w < blockDim.x / 64; ++w) amax = fmaxf(amax, scratch[w]);
    if (amax > __builtin_nontemporal_load(p.amax)) atomicMax(reinterpret_cast<int*>(p.amax), __float_as_int(amax));
}

}  // namespace

}  // namespace moe
