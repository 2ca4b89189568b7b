// Expert products in small tiles of 32 to 128 rows x 32 to 128 weight rows, one per workgroup: for the products in between, whose
// tiles of 128 to 256 rows x 256 weight rows are too few for 256 compute units, and whose rows are too many to only stream the
// weights past them.  There neither memory nor what a compute unit can take in (110 to 135 bytes per ns from the L2) bounds the
// other kernels, but what a few waves do one after the other: 84 k-tiles of 128 x 256 on 66 compute units take 0.7 us each.
// Smaller tiles use more compute units, the waves of a workgroup share the contraction as well as the tile, and a ring of 96 to
// 144 KB keeps enough loads under way (some 1.3 us from memory) that a stage of 24 to 32 KB takes 0.3 to 0.5 us.
//
// Measured (us, the best of the other kernels / here): bf16, 2 experts x 151 rows, 5376 x 1408 gate/up 55 / 37, down 21 / 13; 8 x 34,
// 1152 x 1216 17 / 12, 16 / 9; one x 60, 4416 x 12096 down 57 / 31;  FP8, 2 x 525, 1664 x 3200 down 20 / 13, 8 x 20, 1152 x 13824
// down 64 / 31.  With many experts or rows the large tiles are ahead by up to two times.
//
// Odd bf16 sizes, which the large tiles do not take, have a form for many rows too: 128 x 128 in four waves of 64 x 64, a ring of
// two stages (64 KB), two workgroups to a compute unit.  The form with one to a compute unit is bound by what its eight waves of 64 x
// 32 read from the LDS (96 KB a stage, where four of 64 x 64 read 64) and by the first and last microseconds of every round, which
// nothing else runs under.  us, that form / so: 16 experts x 272 rows, 1496 x 1816 down 57 / 49, 16 x 442, 1288 x 1952 gate/up 163 /
// 134, 12 x 356, 1456 x 1272 79 / 71, 12 x 567, 1696 x 1992 down 100 / 90.  Not kept: stages of 64 bytes of the contraction, five
// of them (134 -> 160: twice the barriers); four waves on 64 x 128, three stages (12 x 194, 1000 x 1416 gate/up 42 -> 38, but mostly
// behind); eight waves on 256 x 128, three stages (134 -> 127, but 49 -> 73 where tiles fall badly).
//
// fp32 layers run here on the bf16 matrix instruction, the fp32 one having 1/16 of its rate.  An fp32 value is the sum of three
// bf16 values (8 bits of significand each: a0 = bf16(a), a1 = bf16(a - a0), a2 = a - a0 - a1; the splitting of Henry, Tang and
// Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", 2019).  The parts are exact
// from 2^-110 on.  Below, they end at the smallest bf16 number, 2^-133, and an operand is up to 2^-134 off (2.6e-6 of it at 1e-35, 2.7e-4 at
// 1e-37; below 2^-134 it counts as zero).  That is less than 2^-24 of any result from 2^-80 on, as long as the magnitudes in its two
// rows add up to less than 2^30; smaller results are taken with the fp32 instruction once more, like those that are infinite or NaN.
// A product of two values is nine bf16 products, of which the three smallest (2^-26 of the largest and less) are left out: six instead of sixteen times the
// work.  The largest product, a0 b0, has an accumulator of its own; the five others, 2^-8 of it and less, share a second one that
// is added at the end, so a sum is rounded once per 16 terms: the results are nearer to 64 bits than those of the fp32 instruction
// (relative 2-norm, fp32 instruction / here: 256 terms 2.1e-7 to 4.2e-7 / 1.4e-7, 800 terms 7.6e-7 / 2.5e-7, 1500 terms 6.9e-7 /
// 2.5e-7).  What bounds it is the splitting (44 instructions for 8 values, in every wave that wants them): one wave on a SIMD
// issues an ordinary instruction every 7.5 clocks, two every 3.8, four every 2.6, so the small forms leave room for many waves.
//
// Measured (us, the streaming kernel on the fp32 instruction / here):
//   8 experts x 34 rows, H x F = 976 x 1136     gate/up  72 /  31,  down  58 /  18
//   16 experts x 32 rows, 800 x 1500            gate/up 110 /  49,  down  63 /  41
//   16 experts x 1024 rows, 800 x 1500          gate/up 654 / 489,  down 393 / 283
// Over 220 products (4 to 16 experts, 2 to 2000 rows per expert, H to 1024, F to 2044) 1.38 times as fast on average.
#include "stream_tile.h"

namespace moe {

namespace {

struct Split {
    bf16x8 p[3];
};

// Whether a sum of products of parts stands: not if it is infinite or NaN, nor below 2^-80, unless it is zero.
constexpr uint32_t kInfinity2 = 0xff000000u, kSmall2 = (127u - 80u) << 24;   // bits without the sign, twice
__device__ __forceinline__ uint32_t above_small(float v) { return (__float_as_uint(v) << 1) - kSmall2; }   // below: wraps, like a zero
__device__ __forceinline__ bool holds(float v) { return above_small(v) < kInfinity2 - kSmall2 || v == 0.f; }

// Eight values into their three parts.  (Infinities and NaN leave NaN in the second part: see `holds`.)
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

// What a wave multiplies at a time: a step, 64 bytes of the contraction (bf16: 32).  Lane (r, h) = (lane % 32, lane / 32) holds half
// of row r's.  The order of the contraction inside a step is the same for both operands, so any assignment is right.
template <int ELT> constexpr int kSteps = ELT == kStreamBf16 ? 4 : 2;   // steps in 128 bytes
typedef __attribute__((ext_vector_type(8))) int i32x8;
template <int ELT> struct Frag;
template <> struct Frag<kStreamF32> {
    Split s;
    __device__ __forceinline__ void set(u32x4 lo, u32x4 hi) { s = split8(lo, hi); }
};
template <> struct Frag<kStreamBf16> {
    bf16x8 v;
    __device__ __forceinline__ void set(u32x4 lo, u32x4) { v = __builtin_bit_cast(bf16x8, lo); }
};
template <> struct Frag<kStreamFp8> {
    i32x8 v;
    __device__ __forceinline__ void set(u32x4 lo, u32x4 hi) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = (int)lo[i];
            v[i + 4] = (int)hi[i];
        }
    }
};

// KB blocks of 128 bytes of the contraction in a stage, each shared by KS groups (a group takes its share of the block's steps);
// KB KS groups of WGM x WGN waves of FM x FN blocks of 32 rows x 32 weight rows (with SwiGLU 16 gate rows and the matching up rows).
// The groups' sums meet in LDS at the end.  A ring of D stages filled by direct loads, one barrier a stage.  PIPE (fp32): a step
// multiplies what the step before has read and split, and reads and splits for the next under its products.
template <int ELT, int MODE, int KB, int KS, int WGM, int WGN, int FM, int FN, int D, bool PIPE>
__global__ __launch_bounds__(KB * KS * WGM * WGN * 64, ELT == kStreamF32 && FM * FN == 1 ? 4 : 2) void gemm_tiles_kernel(const StreamArgs p) {
    constexpr int KG = KB * KS, NWV = KG * WGM * WGN, BM = 32 * FM * WGM, BN = 32 * FN * WGN, OUTN = MODE != 0 ? BN / 2 : BN;
    constexpr int BLOCK = (BM + BN) * 128, STAGE = KB * BLOCK, PER = STAGE / (1024 * NWV);   // bytes; direct loads per wave
    constexpr int STEPS = kSteps<ELT> / KS, STEP = 128 / kSteps<ELT>;   // of a group in a block; bytes
    static_assert(kSteps<ELT> % KS == 0 && STAGE % (1024 * NWV) == 0 && (D - 2) * PER < 64, "whole steps, whole loads; vmcnt holds 6 bits");
    static_assert(!PIPE || (ELT == kStreamF32 && STEPS == 2), "two steps to a stage");
    constexpr bool SWIGLU = MODE != 0;
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const Tile t = locate_tile<BM>(p.offsets, p.E, p.ntn, blockIdx.x);
    if (!t.valid) return;
    const bool sample = ELT == kStreamBf16 && p.ticks != nullptr && blockIdx.x == 0;
    unsigned long long tk_entry = 0, rt_entry = 0;
    if (sample) {
        tk_entry = __builtin_amdgcn_s_memtime();
        rt_entry = __builtin_amdgcn_s_memrealtime();
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = KG > 1 ? wave / (WGM * WGN) : 0, wm = wave / WGN % WGM, wn = wave % WGN, r = lane & 31, h = lane >> 5;
    const int kblock = kg / KS, step0 = kg % KS * STEPS;
    const uint32_t kb = (uint32_t)p.kbytes;
    const int n0 = t.ntile * OUTN;
    const uint8_t* const a0 = p.A + (size_t)t.row0 * kb;
    const size_t w0 = ((size_t)t.expert * p.N + n0) * kb;
    // row i of the tile: rows, then weight rows; past the last one: that one again
    auto row_at = [&](int i) -> const uint8_t* {
        if (i < BM) return a0 + (size_t)((uint32_t)min(i, t.rows - 1) * kb);
        const int w = i - BM, c = SWIGLU ? 16 * (w / 32) + (w & 15) : w;
        return (SWIGLU && (w & 16) ? p.B1 : p.B0) + w0 + (size_t)((uint32_t)min(c, p.N - 1 - n0) * kb);
    };
    const uint8_t* src[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int row = 8 * (q * NWV + wave) + (lane >> 3);   // of all blocks of the stage, one after the other
        src[q] = row_at(row % (BM + BN)) + 128 * (row / (BM + BN)) + 16 * ((lane & 7) ^ lds_swizzle(row));
    }
    f32x16 acc[FM][FN], rest[ELT == kStreamF32 ? FM : 1][ELT == kStreamF32 ? FN : 1];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][j][v] = 0.f;
                if constexpr (ELT == kStreamF32) rest[i][j][v] = 0.f;
            }
    const int nst = p.kbytes / (128 * KB), rot = rotation(t, nst);
    auto issue = [&](int slot, int s) {
        // past the last stage: one line again and again, never used (the waits count loads)
        const uint32_t k = s >= nst ? 0u : (uint32_t)(s + rot >= nst ? s + rot - nst : s + rot) * (128u * KB);
#pragma unroll
        for (int q = 0; q < PER; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[q] + k),
                                             (__attribute__((address_space(3))) void*)(smem + slot * STAGE + (q * NWV + wave) * 1024), 16, 0, 0);
    };
    struct Operands {
        Frag<ELT> a[FM], b[FN];
    };
    auto multiply = [&](const Operands& o) {
        if constexpr (ELT == kStreamF32) {
#pragma unroll
            for (int x = 0; x < 6; ++x)   // the products of each block's second accumulator apart
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        constexpr int pa[6] = {2, 0, 0, 1, 1, 0}, pb[6] = {0, 0, 2, 1, 0, 1};
                        f32x16& c = x == 1 ? acc[i][j] : rest[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.b[j].s.p[pb[x]], o.a[i].s.p[pa[x]], c, 0, 0, 0);
                    }
        } else {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    if constexpr (ELT == kStreamBf16)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.b[j].v, o.a[i].v, acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(o.b[j].v, o.a[i].v, acc[i][j], 0, 0, 0, 0, 0, 0);
                }
        }
    };
    const bool idle = wm * 32 * FM >= t.rows;   // no rows for this wave: only its loads and the barriers
    const int sw = lds_swizzle(r);
    const uint8_t* const arow = smem + kblock * BLOCK + (wm * 32 * FM + r) * 128;
    const uint8_t* const brow = smem + kblock * BLOCK + (BM + wn * 32 * FN + r) * 128;
    auto fetch = [&](int at, int step, Operands& o) {
        constexpr int PIECES = STEP / 32;   // 16-byte pieces of a lane in a step
        const int c0 = (2 * step + h) * PIECES;
        const int c_lo = at + (c0 ^ sw) * 16, c_hi = at + ((c0 + PIECES - 1) ^ sw) * 16;
        u32x4 lo[FM + FN], hi[FM + FN];
#pragma unroll
        for (int i = 0; i < FM + FN; ++i) {
            const uint8_t* row = i < FM ? arow + i * 4096 : brow + (i - FM) * 4096;
            lo[i] = *reinterpret_cast<const u32x4*>(row + c_lo);
            hi[i] = PIECES == 2 ? *reinterpret_cast<const u32x4*>(row + c_hi) : lo[i];
        }
#pragma unroll
        for (int i = 0; i < FM + FN; ++i) (i < FM ? o.a[i] : o.b[i - FM]).set(lo[i], hi[i]);
    };
    auto landed = [&] {   // this wave's loads of the next stage have landed and its reads so far are in registers
        constexpr int W = (D - 2) * PER;
        __builtin_amdgcn_s_waitcnt((W & 0xF) | ((W >> 4) << 14) | 0x70);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    if (nst > 0) {
#pragma unroll
        for (int d = 0; d < D - 1; ++d) issue(d, d);
        int slot = 0;
        if constexpr (PIPE) {
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
            Operands o0, o1;
            landed();
            issue(D - 1, D - 1);
            if (!idle) fetch(0, 0, o0);
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
        } else {
            for (int s = 0; s < nst; ++s) {
                landed();
                issue(slot == 0 ? D - 1 : slot - 1, s + D - 1);   // the slot of the stage before
                if (!idle)
#pragma unroll
                    for (int ks = 0; ks < STEPS; ++ks) {
                        Operands o;
                        fetch(slot * STAGE, step0 + ks, o);
                        multiply(o);
                    }
                slot = slot + 1 == D ? 0 : slot + 1;
            }
        }
    }
    const uint8_t *ga[FM], *gb[FN];   // this lane's rows in memory
#pragma unroll
    for (int i = 0; i < FM; ++i) ga[i] = row_at(wm * 32 * FM + 32 * i + r);
#pragma unroll
    for (int j = 0; j < FN; ++j) gb[j] = row_at(BM + wn * 32 * FN + 32 * j + r);
    // what whole stages leave over, straight from memory; bytes past the end count as zeros
    const int first = (nst * KB + kblock) * 128, rem = idle ? 0 : p.kbytes - first;
#pragma unroll 1
    for (int ks = step0; ks < step0 + STEPS && ks * STEP < rem; ++ks) {
        Operands o;
        auto read = [&](const uint8_t* row, Frag<ELT>& f) {
            constexpr int HALF = STEP / 2;   // bytes of a lane: 16 or 32
            const int at = ks * STEP + HALF * h;
            const bool lo_in = at < rem, hi_in = at + HALF - 16 < rem;
            const u32x4 none = {0u, 0u, 0u, 0u};
            const u32x4 lo = ld16(row + first + (lo_in ? at : 0)), hi = HALF == 32 ? ld16(row + first + (hi_in ? at + 16 : 0)) : lo;
            f.set(lo_in ? lo : none, hi_in ? hi : none);
        };
#pragma unroll
        for (int i = 0; i < FM; ++i) read(ga[i], o.a[i]);
#pragma unroll
        for (int j = 0; j < FN; ++j) read(gb[j], o.b[j]);
        multiply(o);
    }
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): nothing lands in the ring any more
    if constexpr (ELT == kStreamF32)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] += rest[i][j][v];
    if constexpr (KG > 1) {
        // [group - 1][wave of the group][block][four values][lane]
        f32x4* const red = reinterpret_cast<f32x4*>(smem) + ((wave % (WGM * WGN)) * FM * FN * 4) * 64 + lane;
        constexpr int GROUP = WGM * WGN * FM * FN * 4 * 64;
        static_assert((KG - 1) * GROUP * 16 <= D * STAGE, "the groups' sums fit the ring");
        __syncthreads();
        if (kg > 0 && !idle)
#pragma unroll
            for (int x = 0; x < FM * FN * 4; ++x) {
                const f32x16& c = acc[x / 4 / FN][x / 4 % FN];
                red[(kg - 1) * GROUP + x * 64] = f32x4{c[4 * (x % 4)], c[4 * (x % 4) + 1], c[4 * (x % 4) + 2], c[4 * (x % 4) + 3]};
            }
        __syncthreads();
        if (kg == 0 && !idle)
#pragma unroll 1
            for (int g = 0; g < KG - 1; ++g)
#pragma unroll
                for (int x = 0; x < FM * FN * 4; ++x) {
                    const f32x4 v = red[g * GROUP + x * 64];
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc[x / 4 / FN][x / 4 % FN][4 * (x % 4) + u] += v[u];
                }
    }
    float amax = 0.f;
    // (As a condition around the epilogue this has the compiler spill 600 registers of the pipelined form.)
    if constexpr (!(ELT == kStreamFp8 && MODE == 1))
        if (kg > 0 || idle) return;
    if (ELT != kStreamFp8 || MODE != 1 || (kg == 0 && !idle)) {
        if constexpr (ELT == kStreamF32) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    // all at once, without zeros (each value in turn costs a product 2 %: down of 16 experts x 1024 rows, 800 x 1500 261 / 265 us)
                    uint32_t worst = 0;
#pragma unroll
                    for (int v = 0; v < 16; ++v) worst = max(worst, above_small(acc[i][j][v]));
                    if (__all(worst < kInfinity2 - kSmall2)) continue;
                    bool all = true;
#pragma unroll
                    for (int v = 0; v < 16; ++v) all = all && holds(acc[i][j][v]);
                    if (__all(all)) continue;
                    // An infinity or a NaN among the operands (its parts cannot be told apart), a sum past the largest number, or one
                    // so small that its operands may have lost bits: the fp32 matrix instruction on the same rows has the result.  The other
                    // values of the block keep theirs.  The loads follow one another, so a block that is done again takes several times
                    // as long (us, none / a NaN in one row / in one row of 128 / all rows tiny: the product above 262 / 456 / 810 / 1500;
                    // 16 experts x 32 rows 21 / 156 / 159 / 160).
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
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = holds(acc[i][j][v]) ? acc[i][j][v] : c[v];
                }
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int m = wm * 32 * FM + 32 * i + r;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < (SWIGLU ? 2 : 4); ++q) {
                    const int col = n0 + (SWIGLU ? 16 : 32) * (wn * FN + j) + 8 * q + 4 * h;
                    f32x4 v, up;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        v[u] = acc[i][j][4 * q + u];
                        up[u] = acc[i][j][SWIGLU ? 8 + 4 * q + u : 0];
                    }
                    amax = fmaxf(amax, store_four<ELT, MODE>(p, m < t.rows && col < p.N, t.row0 + m, col, v, up));
                }
        }
    }
    if (sample && threadIdx.x == 0) {
        p.ticks[0] = __builtin_amdgcn_s_memtime() - tk_entry;
        p.ticks[1] = __builtin_amdgcn_s_memrealtime() - rt_entry;
    }
    if constexpr (ELT == kStreamFp8 && MODE == 1) {
        // The scratch lies in the ring: the other waves have read the last stage and the groups' sums, and none of their loads, those
        // past the last stage among them, is still to land.
        __syncthreads();
        fold_amax(p, amax, reinterpret_cast<float*>(smem));
    }
}

template <int ELT, int MODE, int KB, int KS, int WGM, int WGN, int FM, int FN, int D, bool PIPE = false>
void launch(StreamArgs p, int r_max, hipStream_t s) {
    constexpr int BM = 32 * FM * WGM, BN = 32 * FN * WGN, OUTN = MODE != 0 ? BN / 2 : BN, smem = KB * (BM + BN) * 128 * D;
    p.ntn = (p.N + OUTN - 1) / OUTN;
    auto kern = gemm_tiles_kernel<ELT, MODE, KB, KS, WGM, WGN, FM, FN, D, PIPE>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), smem);
    hipLaunchKernelGGL(kern, dim3(grid_for(r_max, p.E, BM, p.ntn)), dim3(KB * KS * WGM * WGN * 64), smem, s, p);
}

template <int ELT, int MODE>
void launch_form(int form, const StreamArgs& p, int r_max, hipStream_t s) {
    if constexpr (ELT == kStreamF32) {
        if (form == 0) launch<ELT, MODE, 4, 2, 1, 1, 1, 1, 4>(p, r_max, s);
        else if (form == 1) launch<ELT, MODE, 2, 2, 1, 2, 1, 1, 6>(p, r_max, s);
        else if (form == 2) launch<ELT, MODE, 1, 1, 1, 4, 1, 1, 2>(p, r_max, s);
        else if (form == 3) launch<ELT, MODE, 1, 2, 2, 2, 1, 1, 4>(p, r_max, s);
        else launch<ELT, MODE, 1, 1, 2, 2, 2, 2, 2, true>(p, r_max, s);
    } else {
        constexpr int Q = kSteps<ELT>;   // steps to share
        if (form == 0) launch<ELT, MODE, 2, Q, 1, 1, 1, 2, 6>(p, r_max, s);           // 32 x 64, 24 KB a stage
        else if (form == 1) launch<ELT, MODE, 2, 2, 2, 1, 1, 2, 4>(p, r_max, s);      // 64 x 64, 32 KB
        else if (form == 2) launch<ELT, MODE, 1, 2, 2, 2, 1, 2, 6>(p, r_max, s);      // 64 x 128, 24 KB
        else if (form == 3 || ELT != kStreamBf16 || (MODE != 0 && MODE != 3)) launch<ELT, MODE, 1, 1, 2, 4, 2, 1, 4>(p, r_max, s);   // 128 x 128, 32 KB
        else if constexpr (ELT == kStreamBf16 && (MODE == 0 || MODE == 3)) launch<ELT, MODE, 1, 1, 2, 2, 2, 2, 2>(p, r_max, s);      // the same, two to a compute unit
    }
}

}  // namespace

void launch_tiles(int elt, const StreamArgs& p, int form, int r_max, hipStream_t s) {
    if (elt == kStreamF32) {
        if (p.B1) launch_form<kStreamF32, 1>(form, p, r_max, s);
        else launch_form<kStreamF32, 0>(form, p, r_max, s);
    } else if (elt == kStreamBf16) {
        if (p.GU) launch_form<kStreamBf16, 2>(form, p, r_max, s);
        else if (p.B1 && full_silu(p)) launch_form<kStreamBf16, 3>(form, p, r_max, s);
        else if (p.B1) launch_form<kStreamBf16, 1>(form, p, r_max, s);
        else launch_form<kStreamBf16, 0>(form, p, r_max, s);
    } else {
        if (p.B1) launch_form<kStreamFp8, 1>(form, p, r_max, s);
        else launch_form<kStreamFp8, 0>(form, p, r_max, s);
    }
}

}  // namespace moe
