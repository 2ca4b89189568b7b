// fp32 expert products on the bf16 matrix instruction.
//
// The fp32 matrix instruction runs at 1/16 of the bf16 one's rate.  An fp32 value is the sum of three bf16 values (8 bits of
// significand each: a0 = bf16(a), a1 = bf16(a - a0), a2 = a - a0 - a1, all exact), so a product of two is nine bf16 products, of
// which the three smallest (2^-26 of the largest and less) are left out: six instead of sixteen times the work.  The largest
// product, a0 b0, has an accumulator of its own; the five others, 2^-8 of it and less, share a second one that is added at the
// end, so a sum is rounded once per 16 terms: the results are nearer to 64 bits than those of the fp32 instruction (relative
// 2-norm, fp32 instruction / here: 256 terms 2.1e-7 to 4.2e-7 / 1.4e-7, 800 terms 7.6e-7 / 2.5e-7, 1500 terms 6.9e-7 / 2.5e-7).
//
// Measured (us, the streaming kernel on the fp32 instruction / here):
//   8 experts x 34 rows, H x F = 976 x 1136     gate/up  72 /  31,  down  58 /  18
//   16 experts x 32 rows, 800 x 1500            gate/up 110 /  49,  down  63 /  41
//   16 experts x 1024 rows, 800 x 1500          gate/up 654 / 489,  down 393 / 283
// Over 220 products (4 to 16 experts, 2 to 2000 rows per expert, H to 1024, F to 2044) 1.35 times as fast on average.
#include "stream_tile.h"

namespace moe {

namespace {

struct Split {
    bf16x8 p[3];
};

// Eight values into their three parts.  (Infinities and NaN leave NaN in the second part: see `finite` below.)
__device__ __forceinline__ Split split8(u32x4 lo, u32x4 hi) {
    u32x4 out[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = __uint_as_float(i < 2 ? lo[2 * i] : hi[2 * i - 4]), y = __uint_as_float(i < 2 ? lo[2 * i + 1] : hi[2 * i - 3]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t b = pack2_bf16(x, y);
            out[k][i] = b;
            x -= __uint_as_float(b << 16);
            y -= __uint_as_float(b & 0xffff0000u);
        }
    }
    Split s;
#pragma unroll
    for (int k = 0; k < 3; ++k) s.p[k] = __builtin_bit_cast(bf16x8, out[k]);
    return s;
}

// KG groups of WGM x WGN waves of FM x FN blocks of 32 rows x 32 weight rows (with SwiGLU 16 gate rows and the matching up rows).
// The groups take the 128-byte blocks of the contraction in turn and their sums meet in LDS at the end.  A ring of D stages, one
// block for each group.  What bounds it is the splitting (44 instructions for 8 values, in every wave that wants them): one wave on
// a SIMD issues an ordinary instruction every 7.5 clocks, two every 3.8, four every 2.6, so the small forms leave room for many
// waves.  PIPE, where 256 registers a wave leave room for two: a step of 16 values multiplies what the step before has read and
// split, and reads and splits for the next under its products (128 x 128 tiles, 8192 tokens on 16 experts, 800 x 1500: 498 / 489).
template <int MODE, int KG, int WGM, int WGN, int FM, int FN, int D, bool PIPE>
__global__ __launch_bounds__(KG * WGM * WGN * 64, FM * FN == 1 ? 4 : 2) void gemm_f32_kernel(const StreamArgs p) {
    constexpr int NWV = KG * WGM * WGN, BM = 32 * FM * WGM, BN = 32 * FN * WGN, OUTN = MODE != 0 ? BN / 2 : BN;
    constexpr int BLOCK = (BM + BN) * 128, STAGE = KG * BLOCK, PER = STAGE / (1024 * NWV);   // bytes; direct loads per wave
    static_assert(STAGE % (1024 * NWV) == 0 && (D - 2) * PER < 64, "whole loads; vmcnt holds 6 bits");
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const Tile t = locate_tile<BM>(p.offsets, p.E, p.ntn);
    if (!t.valid) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / (WGM * WGN), wm = wave / WGN % WGM, wn = wave % WGN, r = lane & 31, h = lane >> 5;
    const uint32_t kb = (uint32_t)p.kbytes;
    const int n0 = t.ntile * OUTN;
    const uint8_t* const a0 = p.A + (size_t)t.row0 * kb;
    const size_t w0 = ((size_t)t.expert * p.N + n0) * kb;
    // row i of the tile: rows, then weight rows; past the last one: that one again
    auto row_at = [&](int i) -> const uint8_t* {
        if (i < BM) return a0 + (size_t)((uint32_t)min(i, t.rows - 1) * kb);
        const int w = i - BM, c = MODE != 0 ? 16 * (w / 32) + (w & 15) : w;
        return (MODE != 0 && (w & 16) ? p.B1 : p.B0) + w0 + (size_t)((uint32_t)min(c, p.N - 1 - n0) * kb);
    };
    const uint8_t* src[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int row = 8 * (q * NWV + wave) + (lane >> 3);   // of all groups' blocks, one after the other
        src[q] = row_at(row % (BM + BN)) + 128 * (row / (BM + BN)) + 16 * ((lane & 7) ^ lds_swizzle(row));
    }
    f32x16 big[FM][FN], rest[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) big[i][j][v] = rest[i][j][v] = 0.f;
    const int nst = p.kbytes / (128 * KG), rot = rotation(t, nst);
    auto issue = [&](int slot, int s) {
        // past the last stage: one line again and again, never used (the waits count loads)
        const uint32_t k = s >= nst ? 0u : (uint32_t)(s + rot >= nst ? s + rot - nst : s + rot) * (128u * KG);
#pragma unroll
        for (int q = 0; q < PER; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[q] + k),
                                             (__attribute__((address_space(3))) void*)(smem + slot * STAGE + (q * NWV + wave) * 1024), 16, 0, 0);
    };
    struct Operands {
        Split a[FM], b[FN];
    };
    auto multiply = [&](const Operands& o) {
#pragma unroll
        for (int x = 0; x < 6; ++x)   // the products of each block's second accumulator apart
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    constexpr int pa[6] = {2, 0, 0, 1, 1, 0}, pb[6] = {0, 0, 2, 1, 0, 1};
                    f32x16& c = x == 1 ? big[i][j] : rest[i][j];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.b[j].p[pb[x]], o.a[i].p[pa[x]], c, 0, 0, 0);
                }
    };
    const bool idle = wm * 32 * FM >= t.rows;   // no rows for this wave: only its loads and the barriers
    const int sw = lds_swizzle(r);
    const uint8_t* const arow = smem + kg * BLOCK + (wm * 32 * FM + r) * 128;
    const uint8_t* const brow = smem + kg * BLOCK + (BM + wn * 32 * FN + r) * 128;
    auto fetch = [&](int at, int ks, Operands& o) {
        const int c_lo = at + ((4 * ks + 2 * h) ^ sw) * 16, c_hi = at + ((4 * ks + 2 * h + 1) ^ sw) * 16;
        u32x4 lo[FM + FN], hi[FM + FN];
#pragma unroll
        for (int i = 0; i < FM + FN; ++i) {
            const uint8_t* row = i < FM ? arow + i * 4096 : brow + (i - FM) * 4096;
            lo[i] = *reinterpret_cast<const u32x4*>(row + c_lo);
            hi[i] = *reinterpret_cast<const u32x4*>(row + c_hi);
        }
#pragma unroll
        for (int i = 0; i < FM + FN; ++i) (i < FM ? o.a[i] : o.b[i - FM]) = split8(lo[i], hi[i]);
    };
    if (PIPE && nst > 0) {
        // under every product the splitting that is its share
        auto interleave = [&] {
            constexpr int N = 6 * FM * FN, V = (44 * (FM + FN) + N - 1) / N;
            __builtin_amdgcn_sched_group_barrier(0x100, 2 * (FM + FN), 0);
#pragma unroll
            for (int x = 0; x < N; ++x) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, V, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto landed = [&] {   // this wave's loads of the next stage have landed and its reads of this one are in registers
            constexpr int W = (D - 2) * PER;
            __builtin_amdgcn_s_waitcnt((W & 0xF) | ((W >> 4) << 14) | 0x70);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };
        Operands o0, o1;
#pragma unroll
        for (int d = 0; d < D - 1; ++d) issue(d, d);
        landed();
        issue(D - 1, D - 1);
        if (!idle) fetch(0, 0, o0);
        int slot = 0;
        for (int s = 0; s < nst; ++s) {
            const int next = slot + 1 == D ? 0 : slot + 1;
            if (!idle) {
                __builtin_amdgcn_sched_barrier(0);
                fetch(slot * STAGE, 1, o1);
                multiply(o0);
                interleave();
            }
            landed();
            issue(slot, s + D);   // this stage's slot: everyone has read it
            if (!idle) {
                __builtin_amdgcn_sched_barrier(0);
                fetch(next * STAGE, 0, o0);   // past the last stage: never used
                multiply(o1);
                interleave();
            }
            slot = next;
        }
    } else if (nst > 0) {
#pragma unroll
        for (int d = 0; d < D - 1; ++d) issue(d, d);
        int slot = 0;
        for (int s = 0; s < nst; ++s) {
            // this wave's loads of the stage have landed and its reads of the stage before are in registers
            constexpr int W = (D - 2) * PER;
            __builtin_amdgcn_s_waitcnt((W & 0xF) | ((W >> 4) << 14) | 0x70);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            issue(slot == 0 ? D - 1 : slot - 1, s + D - 1);
            if (!idle)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    Operands o;
                    fetch(slot * STAGE, ks, o);
                    multiply(o);
                }
            slot = slot + 1 == D ? 0 : slot + 1;
        }
    }
    const uint8_t *ga[FM], *gb[FN];   // this lane's rows in memory
#pragma unroll
    for (int i = 0; i < FM; ++i) ga[i] = row_at(wm * 32 * FM + 32 * i + r);
#pragma unroll
    for (int j = 0; j < FN; ++j) gb[j] = row_at(BM + wn * 32 * FN + 32 * j + r);
    // what whole stages leave over, one block for each group, straight from memory; bytes past the end count as zeros
    const int first = (nst * KG + kg) * 128, rem = idle ? 0 : min(p.kbytes - first, 128);
    for (int k = 0; k < rem; k += 64) {
        Operands o;
        auto read = [&](const uint8_t* row) {
            const int at = k + 32 * h;
            const bool lo_in = at < rem, hi_in = at + 16 < rem;
            const u32x4 none = {0u, 0u, 0u, 0u};
            const u32x4 lo = ld16(row + first + (lo_in ? at : 0)), hi = ld16(row + first + (hi_in ? at + 16 : 0));
            return split8(lo_in ? lo : none, hi_in ? hi : none);
        };
#pragma unroll
        for (int i = 0; i < FM; ++i) o.a[i] = read(ga[i]);
#pragma unroll
        for (int j = 0; j < FN; ++j) o.b[j] = read(gb[j]);
        multiply(o);
    }
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): nothing lands in the ring any more
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) big[i][j][v] += rest[i][j][v];
    if constexpr (KG > 1) {
        // [group - 1][wave of the group][block][four values][lane]
        f32x4* const red = reinterpret_cast<f32x4*>(smem) + ((wave % (WGM * WGN)) * FM * FN * 4) * 64 + lane;
        constexpr int GROUP = WGM * WGN * FM * FN * 4 * 64;
        __syncthreads();
        if (kg > 0)
#pragma unroll
            for (int x = 0; x < FM * FN * 4; ++x) {
                const f32x16& c = big[x / 4 / FN][x / 4 % FN];
                red[(kg - 1) * GROUP + x * 64] = f32x4{c[4 * (x % 4)], c[4 * (x % 4) + 1], c[4 * (x % 4) + 2], c[4 * (x % 4) + 3]};
            }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 0; g < KG - 1; ++g)
#pragma unroll
            for (int x = 0; x < FM * FN * 4; ++x) {
                const f32x4 v = red[g * GROUP + x * 64];
#pragma unroll
                for (int u = 0; u < 4; ++u) big[x / 4 / FN][x / 4 % FN][4 * (x % 4) + u] += v[u];
            }
    }
    if (idle) return;
    bool finite = true;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) finite = finite && fabsf(big[i][j][v]) < INFINITY;
    if (!__all(finite)) {
        // An infinity or a NaN among the operands (its parts cannot be told apart), or a sum past the largest number: the
        // fp32 matrix instruction on the same rows says which of the results are infinite.
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                f32x16 c;
#pragma unroll
                for (int v = 0; v < 16; ++v) c[v] = 0.f;
                for (uint32_t k = 0; k < kb; k += 16) {
                    const u32x2 x = *(const __attribute__((address_space(1))) u32x2*)(ga[i] + k + 8 * h);
                    const u32x2 w = *(const __attribute__((address_space(1))) u32x2*)(gb[j] + k + 8 * h);
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(w[e]), __uint_as_float(x[e]), c, 0, 0, 0);
                }
                big[i][j] = c;
            }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = wm * 32 * FM + 32 * i + r;
        if (m >= t.rows) continue;
        float* const out = static_cast<float*>(p.C) + (size_t)(t.row0 + m) * p.N;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < (MODE != 0 ? 2 : 4); ++q) {
                const int col = n0 + (MODE != 0 ? 16 : 32) * (wn * FN + j) + 8 * q + 4 * h;
                f32x4 v;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float g = big[i][j][4 * q + u];
                    if constexpr (MODE != 0) v[u] = (g / (1.f + expf(-g))) * big[i][j][8 + 4 * q + u];
                    else v[u] = g;
                }
                if (col < p.N) *reinterpret_cast<f32x4*>(out + col) = v;   // N is a multiple of 4
            }
    }
}

template <int MODE, int KG, int WGM, int WGN, int FM, int FN, int D, bool PIPE>
void launch(StreamArgs p, int r_max, hipStream_t s) {
    constexpr int BM = 32 * FM * WGM, BN = 32 * FN * WGN, OUTN = MODE != 0 ? BN / 2 : BN, smem = KG * (BM + BN) * 128 * D;
    p.ntn = (p.N + OUTN - 1) / OUTN;
    auto kern = gemm_f32_kernel<MODE, KG, WGM, WGN, FM, FN, D, PIPE>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), smem);
    hipLaunchKernelGGL(kern, dim3(grid_for(r_max, p.E, BM, p.ntn)), dim3(KG * WGM * WGN * 64), smem, s, p);
}

template <int MODE>
void launch_form(int form, const StreamArgs& p, int r_max, hipStream_t s) {
    if (form == 0) launch<MODE, 8, 1, 1, 1, 1, 2, false>(p, r_max, s);
    else if (form == 1) launch<MODE, 4, 1, 2, 1, 1, 3, false>(p, r_max, s);
    else if (form == 2) launch<MODE, 1, 1, 4, 1, 1, 2, false>(p, r_max, s);
    else if (form == 3) launch<MODE, 2, 2, 2, 1, 1, 2, false>(p, r_max, s);
    else launch<MODE, 1, 2, 2, 2, 2, 2, true>(p, r_max, s);
}

}  // namespace

void launch_f32_tiles(const StreamArgs& p, int form, int r_max, hipStream_t s) {
    if (p.B1) launch_form<1>(form, p, r_max, s);
    else launch_form<0>(form, p, r_max, s);
}

}  // namespace moe
