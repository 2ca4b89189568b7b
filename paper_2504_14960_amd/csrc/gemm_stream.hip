// Grouped expert GEMM (a3) for experts with few rows, and for every shape the large-tile kernels do not take (fp32
// layers, bf16 layers whose H or F is not a multiple of 64).
//
// With few rows per expert the product is a read of the weights: what bounds it is how many bytes of them are on
// their way from HBM at a time.  The large-tile kernel has one workgroup per 256 weight rows, so the down projection of
// two experts (4096 outputs, one decoded token) is 32 workgroups on 256 compute units, and a tile of 128 rows or more is
// multiplied whatever it holds.  Here a workgroup owns 16 to 256 weight rows, the weights go straight from memory into the
// matrix instruction's operand registers (each byte is wanted by one wave only; two 16-byte loads per lane cover
// whole 128-byte lines of 16 rows), and the rows of the tile decide how the other operand travels:
//
//   up to 16 rows    registers as well (direct_tile): no barrier and no LDS in the loop, the waves take the blocks of
//                    the contraction in turn;
//   17 to 128 rows   through LDS, shared by the waves (shared_tile, narrow workgroups of four waves; wide_tile, eight
//                    waves and up to 256 weight rows); with more rows than that per expert the read of the rows
//                    outweighs the weights and the large tiles are mostly the better kernel.
//
// Measured (us, the large tiles / here; weights of several launches, so that no cache holds them):
//   2 experts x 1 row, H x F = 4096 x 14336    gate/up 102 /  89 (5.3 TB/s of weights), down 251 /  46
//   64 experts x 8 rows, 3584 x 2560           gate/up 417 / 400 (5.9 TB/s),            down 236 / 213
//   8 experts x 8 rows, 4096 x 14336           gate/up 458 / 314 (6.0 TB/s),            down 289 / 161
//   the same in FP8                            gate/up 211 / 166 (5.7 TB/s),            down 148 /  88
// and against the plain FMA kernel, which took these shapes before:
//   12 experts, 2331 rows, 1000 x 1416         gate/up 310 /  50,                       down 271 /  30
//   fp32, 8 experts x 64 rows, 128 x 256       gate/up  29 /   8,                       down  36 /   7
// (fp32 with more than some 12 rows per expert, and much of bf16 and FP8 between these rows and the large tiles': gemm_tiles.hip)
#include <type_traits>

#include "stream_tile.h"
#include "tile_cost.h"

namespace moe {

namespace {

constexpr int NW = 4;   // waves per workgroup
constexpr int kScratch = 64;   // bytes of LDS behind the ring: one float per wave (fold_amax)

constexpr int kEltF32 = kStreamF32, kEltBf16 = kStreamBf16, kEltFp8 = kStreamFp8;

template <int ELT>
__device__ __forceinline__ f32x4 mul_step(const Piece& w, const Piece& a, f32x4 acc) {
    if constexpr (ELT == kEltBf16) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w.lo), __builtin_bit_cast(bf16x8, a.lo), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w.hi), __builtin_bit_cast(bf16x8, a.hi), acc, 0, 0, 0);
    } else if constexpr (ELT == kEltFp8) {
        typedef __attribute__((ext_vector_type(8))) int i32x8;
        i32x8 wv, av;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            wv[i] = (int)w.lo[i]; wv[i + 4] = (int)w.hi[i];
            av[i] = (int)a.lo[i]; av[i + 4] = (int)a.hi[i];
        }
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wv, av, acc, 0, 0, 0, 0, 0, 0);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.lo[i]), __uint_as_float(a.lo[i]), acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.hi[i]), __uint_as_float(a.hi[i]), acc, 0, 0, 0);
    }
    return acc;
}

// Where a workgroup's tile lies: FB blocks of 16 weight rows (with SwiGLU half of them gate rows and half the matching
// up rows) against the rows of one expert.
template <int MODE, int FB>
struct TileAt {
    static constexpr int NF = MODE != 0 ? FB / 2 : FB;   // blocks of 16 output columns
    const uint8_t* a;
    const uint8_t* b[2];
    int n0;
    __device__ __forceinline__ TileAt(const StreamArgs& p, const Tile& t) {
        n0 = t.ntile * (16 * NF);
        a = p.A + (size_t)t.row0 * (uint32_t)p.kbytes;
        const size_t wrow = ((size_t)t.expert * p.N + n0) * (uint32_t)p.kbytes;
        b[0] = p.B0 + wrow;
        b[1] = (MODE != 0 ? p.B1 : p.B0) + wrow;
    }
};

// Stores the 16 x 16 output block (row block i, column block f) from its sums: v (with SwiGLU the gate's) and up.  A
// lane holds row 16 i + lane % 16 and four consecutive columns.  Returns the largest |h| stored (FP8).
template <int ELT, int MODE>
__device__ __forceinline__ float store_block(const StreamArgs& p, const Tile& t, int n0, int i, int f, f32x4 v, f32x4 up) {
    const int lane = threadIdx.x & 63;
    const int m = 16 * i + (lane & 15), col = n0 + 16 * f + 4 * (lane >> 4);
    return store_four<ELT, MODE>(p, m < t.rows && col < p.N, t.row0 + m, col, v, up);
}

// Sums the partial products red[slot][row block][weight block][lane] in slot order and stores the outputs.
template <int ELT, int MODE, int FB, int MF, int SLOTS>
__device__ __forceinline__ float finish_tile(const StreamArgs& p, const Tile& t, int n0, const f32x4* red) {
    constexpr int NF = TileAt<MODE, FB>::NF;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float amax = 0.f;
    for (int u = wave; u < MF * NF; u += NW) {
        const int i = u / NF, f = u - i * NF;
        auto total = [&](int ff) {
            f32x4 v = red[(i * FB + ff) * 64 + lane];
#pragma unroll
            for (int w = 1; w < SLOTS; ++w) v += red[((w * MF + i) * FB + ff) * 64 + lane];
            return v;
        };
        const f32x4 v = total(f), up = MODE != 0 ? total(f + NF) : v;
        amax = fmaxf(amax, store_block<ELT, MODE>(p, t, n0, i, f, v, up));
    }
    return amax;
}

// At most 16 rows: both operands go straight from memory to registers, the waves take the 128-byte blocks of the
// contraction in turn and their partial sums meet in LDS.  No barrier in the loop.
template <int ELT, int MODE, int FB>
__device__ __forceinline__ float direct_tile(const StreamArgs& p, const Tile& t, uint8_t* smem) {
    typedef TileAt<MODE, FB> At;
    constexpr int NF = At::NF;
    constexpr int D = 12 / (1 + FB) > 2 ? 12 / (1 + FB) : 2;   // blocks in flight: about 96 registers of operands
    const At at(p, t);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, j = lane >> 4;
    const uint32_t kb = (uint32_t)p.kbytes;
    const uint32_t arow = (uint32_t)min(r, t.rows - 1) * kb;
    uint32_t brow[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) brow[f] = (uint32_t)min(16 * f + r, p.N - 1 - at.n0) * kb;

    f32x4 acc[FB];
#pragma unroll
    for (int f = 0; f < FB; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    Piece fa[D], fb[D][FB];
    const int nfull = p.kbytes / 128;
    const int rot = rotation(t, nfull);
    auto load = [&](int d, int s) {
        const int sr = s + rot >= nfull ? s + rot - nfull : s + rot;
        const uint32_t k = (uint32_t)sr * 128u + 32u * j;
#pragma unroll
        for (int f = 0; f < FB; ++f) {
            const uint8_t* q = at.b[f / NF] + (k + brow[f % NF]);
            fb[d][f].lo = ld16(q);
            fb[d][f].hi = ld16(q + 16);
        }
        const uint8_t* q = at.a + (k + arow);
        fa[d].lo = ld16(q);
        fa[d].hi = ld16(q + 16);
    };
    auto use = [&](int d) {
#pragma unroll
        for (int f = 0; f < FB; ++f) acc[f] = mul_step<ELT>(fb[d][f], fa[d], acc[f]);
    };
    const int cnt = nfull > wave ? (nfull - wave + NW - 1) / NW : 0;   // this wave's whole blocks: wave, wave + NW, ...
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < cnt) load(d, wave + d * NW);
    int i0 = 0;
    for (; i0 + 2 * D <= cnt; i0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            use(d);
            load(d, wave + (i0 + D + d) * NW);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (i0 + d < cnt) use(d);
        if (i0 + D + d < cnt) load(d, wave + (i0 + D + d) * NW);
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (i0 + D + d < cnt) use(d);
    const int rem = p.kbytes & 127;
    if (rem && (nfull % NW) == wave) {
        const uint32_t k = (uint32_t)nfull * 128u;
#pragma unroll
        for (int f = 0; f < FB; ++f) fb[0][f] = tail_piece(at.b[f / NF] + (k + brow[f % NF]), j, rem);
        fa[0] = tail_piece(at.a + (k + arow), j, rem);
        use(0);
    }
    f32x4* const red = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int f = 0; f < FB; ++f) red[(wave * FB + f) * 64 + lane] = acc[f];
    __syncthreads();
    return finish_tile<ELT, MODE, FB, 1, NW>(p, t, at.n0, red);
}

// 17 to 128 rows: wave = (weight block, share of the contraction).  The weights still go straight to registers (no
// other wave wants them); the rows are shared, so they pass through LDS: a ring of stages filled by direct
// global-to-LDS loads, KS 128-byte blocks of the contraction per stage, one barrier per stage.
template <int ELT, int MODE, int FB, int MF, int RING, int NBW>
__device__ __forceinline__ float shared_tile(const StreamArgs& p, const Tile& t, uint8_t* smem) {
    typedef TileAt<MODE, FB> At;
    constexpr int NF = At::NF;
    constexpr int WB = FB / NBW;                     // waves side by side over the weight blocks
    constexpr int KS = NW / WB;
    constexpr int SUB = MF * 16 * 128;               // bytes of one block of the rows
    constexpr int STAGE = SUB * KS;
    constexpr int D = RING / STAGE < 8 ? RING / STAGE : 8;
    static_assert(D >= 2, "the ring holds at least two stages");
    constexpr int PA = STAGE / (NW * 1024);          // direct loads per thread and stage
    constexpr int PER = PA + 2 * NBW;                      // vector loads per thread and stage
    static_assert((D - 2) * PER < 64, "vmcnt holds 6 bits");
    const At at(p, t);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fw = wave % WB, kg = wave / WB;        // this wave: weight blocks fw NBW .. + NBW - 1, share kg
    const int r = lane & 15, j = lane >> 4;
    const uint32_t kb = (uint32_t)p.kbytes;
    // weight block of slot f: with SwiGLU a wave of two slots holds a gate block and the matching up block
    auto block_of = [&](int f) { return MODE != 0 && NBW == 2 ? fw + f * NF : fw * NBW + f; };
    const uint8_t* b_base[NBW];
    uint32_t boff[NBW];
#pragma unroll
    for (int f = 0; f < NBW; ++f) {
        b_base[f] = at.b[MODE != 0 ? block_of(f) / NF : 0] + 128 * kg;
        boff[f] = (uint32_t)min(16 * (block_of(f) % NF) + r, p.N - 1 - at.n0) * kb + 32u * j;
    }
    // direct load q of a stage: unit u = q NW + wave covers rows 8 (u mod 2 MF) .. + 7 of block u / (2 MF)
    uint32_t aoff[PA];
#pragma unroll
    for (int q = 0; q < PA; ++q) {
        const int u = q * NW + wave, row = 8 * (u % (2 * MF)) + (lane >> 3);
        aoff[q] = (uint32_t)min(row, t.rows - 1) * kb + 128u * (u / (2 * MF)) + 16u * ((lane & 7) ^ lds_swizzle(row));
    }
    f32x4 acc[MF][NBW];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int f = 0; f < NBW; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    Piece fb[D][NBW];
    const int nfull = p.kbytes / 128;
    const int nst = nfull / KS;   // whole stages
    const int rot = rotation(t, nst);
    auto issue = [&](int slot, int s) {
        // past the last stage: one line again and again, never used (the waits count loads)
        const bool over = s >= nst;
        const int sr = s + rot >= nst ? s + rot - nst : s + rot;
        const uint32_t k = over ? 0u : (uint32_t)sr * (128u * KS);
        const uint32_t mask = over ? 0u : ~0u;
#pragma unroll
        for (int q = 0; q < PA; ++q)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(at.a + k + (aoff[q] & mask)),
                (__attribute__((address_space(3))) void*)(smem + slot * STAGE + (q * NW + wave) * 1024), 16, 0, 0);
#pragma unroll
        for (int f = 0; f < NBW; ++f) {
            const uint8_t* b = (over ? at.a : b_base[f] + k) + (boff[f] & mask);
            fb[slot][f].lo = ld16(b);
            fb[slot][f].hi = ld16(b + 16);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const int sw = lds_swizzle(r);   // blocks of 16 rows: the swizzle of row 16 i + r
    const uint8_t* const arow = smem + kg * SUB + r * 128;
    const int c_lo = ((2 * j) ^ sw) * 16, c_hi = ((2 * j + 1) ^ sw) * 16;
    auto use = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            Piece a;
            a.lo = *reinterpret_cast<const u32x4*>(arow + slot * STAGE + i * 2048 + c_lo);
            a.hi = *reinterpret_cast<const u32x4*>(arow + slot * STAGE + i * 2048 + c_hi);
#pragma unroll
            for (int f = 0; f < NBW; ++f) acc[i][f] = mul_step<ELT>(fb[slot][f], a, acc[i][f]);
        }
    };
    if (nst > 0) {
#pragma unroll
        for (int d = 0; d < D - 1; ++d) issue(d, d);
        for (int s0 = 0; s0 < nst; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                // this wave's loads of the stage have landed and its reads of the stage before are in registers
                constexpr int W = (D - 2) * PER;
                __builtin_amdgcn_s_waitcnt((W & 0xF) | ((W >> 4) << 14) | 0x70);
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
                issue((d + D - 1) % D, s0 + d + D - 1);
                if (s0 + d < nst) use(d);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // blocks left over after the whole stages, and the partial one: one per share, straight from memory
    const int blk = nst * KS + kg;
    const int rem = p.kbytes - 128 * blk;
    if (rem > 0) {
        const int left = min(rem, 128);
#pragma unroll
        for (int f = 0; f < NBW; ++f) fb[0][f] = tail_piece(b_base[f] - 128 * kg + 128 * blk + (boff[f] - 32u * j), j, left);
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const Piece a = tail_piece(at.a + 128 * blk + (size_t)((uint32_t)min(16 * i + r, t.rows - 1) * kb), j, left);
#pragma unroll
            for (int f = 0; f < NBW; ++f) acc[i][f] = mul_step<ELT>(fb[0][f], a, acc[i][f]);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): nothing lands in the ring any more
    if constexpr (KS == 1 && (MODE == 0 || NBW == 2)) {
        float amax = 0.f;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            if (16 * i >= t.rows) break;
            if constexpr (MODE != 0)
                amax = fmaxf(amax, store_block<ELT, MODE>(p, t, at.n0, i, fw, acc[i][0], acc[i][NBW - 1]));
            else
#pragma unroll
                for (int f = 0; f < NBW; ++f) store_block<ELT, MODE>(p, t, at.n0, i, block_of(f), acc[i][f], acc[i][f]);
        }
        return amax;
    }
    __syncthreads();
    f32x4* const red = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int f = 0; f < NBW; ++f) red[((kg * MF + i) * FB + block_of(f)) * 64 + lane] = acc[i][f];
    __syncthreads();
    return finish_tile<ELT, MODE, FB, MF, KS>(p, t, at.n0, red);
}

// ---- wide tiles: 17 rows per expert and more ----
// A compute unit takes in some 25 bytes per nanosecond of a stream from HBM, and the rows that pass through LDS count
// like the weights (loads return in order), so what a workgroup reads per weight byte is what matters: eight waves and
// up to 256 weight rows on one ring of row stages, one workgroup per compute unit.  The number of weight rows is
// chosen per launch (units x 32) so that the tiles fill whole rounds of the compute units, and where that leaves too
// few of them and there is room (the layer's shared expert) the contraction is split: the splits leave fp32 partial sums
// that stream_reduce_kernel adds in split order.  Measured (us, the better of the narrow kernel
// and large tiles of 256 rows / here):
//   one expert, gate/up 20480 x 3584: 64 rows 84 / 61 (160 weight rows each on 256 workgroups), 125 rows 86 / 74
//   the same, down: 64 rows 70 / 185 whole, 42 in 16 parts; 250 rows 126 / 68 and 500 rows 162 / 110 in parts
//   (500 rows: the large tiles in parts take 87)
//   8 experts, gate/up 14336 x 4096, 125 rows 421 / 404;  16 experts, gate/up 1408 x 2048, 64 rows 51 / 44
constexpr int kWideWaves = 8, kWideRing = 128 * 1024;

template <int ELT, int MODE, int MF>
__device__ __forceinline__ float wide_tile(const StreamArgs& p, const Tile& t, int n, int ks, uint8_t* smem) {
    constexpr int STAGE = MF * 16 * 128;                // bytes of one 128-byte block of the rows
    constexpr int D = kWideRing / STAGE < 8 ? kWideRing / STAGE : 8;
    constexpr int PA = STAGE / (kWideWaves * 1024);     // direct loads per thread and stage
    constexpr int PER = PA + 4;                         // vector loads per thread and stage
    static_assert(PA >= 1 && (D - 2) * PER < 64, "vmcnt holds 6 bits");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, j = lane >> 4;
    const uint32_t kb = (uint32_t)p.kbytes;
    // a unit is 32 weight rows: with SwiGLU 16 gate rows and the matching up rows, else 32 rows; one unit per wave
    const int n0 = n * p.units * (MODE != 0 ? 16 : 32);
    const int col0 = n0 + wave * (MODE != 0 ? 16 : 32);
    const bool idle = wave >= p.units || col0 >= p.N;
    const uint8_t* const a0 = p.A + (size_t)t.row0 * kb;
    const uint8_t* b_base[2];
    uint32_t boff[2];
    {
        const size_t wrow = ((size_t)t.expert * p.N + (idle ? 0 : col0)) * kb;
        b_base[0] = p.B0 + wrow;
        b_base[1] = (MODE != 0 ? p.B1 : p.B0) + wrow;
#pragma unroll
        for (int f = 0; f < 2; ++f)
            boff[f] = idle ? 0u : (uint32_t)min((MODE != 0 ? 0 : 16 * f) + r, p.N - 1 - col0) * kb + 32u * j;
    }
    // direct load q of a stage: unit u = q waves + wave covers rows 8 u .. + 7
    uint32_t aoff[PA];
#pragma unroll
    for (int q = 0; q < PA; ++q) {
        const int row = 8 * (q * kWideWaves + wave) + (lane >> 3);
        aoff[q] = (uint32_t)min(row, t.rows - 1) * kb + 16u * ((lane & 7) ^ lds_swizzle(row));
    }
    f32x4 acc[MF][2];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    Piece fb[D][2];
    const int nfull = p.kbytes / 128;
    const int st0 = (int)((long long)nfull * ks / p.S), nst = (int)((long long)nfull * (ks + 1) / p.S) - st0;
    Tile tn = t;
    tn.ntile = n;
    const int rot = rotation(tn, nst);
    auto issue = [&](int slot, int s) {
        // past the last stage: one line again and again, never used (the waits count loads)
        const bool over = s >= nst;
        const int sr = s + rot >= nst ? s + rot - nst : s + rot;
        const uint32_t k = over ? 0u : (uint32_t)(st0 + sr) * 128u;
        const uint32_t mask = over ? 0u : ~0u;
#pragma unroll
        for (int q = 0; q < PA; ++q)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(a0 + k + (aoff[q] & mask)),
                (__attribute__((address_space(3))) void*)(smem + slot * STAGE + (q * kWideWaves + wave) * 1024), 16, 0, 0);
        const bool none = over || idle;
        const uint32_t bmask = none ? 0u : ~0u;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const uint8_t* b = (none ? a0 : b_base[f] + k) + (boff[f] & bmask);
            fb[slot][f].lo = ld16(b);
            fb[slot][f].hi = ld16(b + 16);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const int sw = lds_swizzle(r);   // blocks of 16 rows: the swizzle of row 16 i + r
    const uint8_t* const arow = smem + r * 128;
    const int c_lo = ((2 * j) ^ sw) * 16, c_hi = ((2 * j + 1) ^ sw) * 16;
    auto use = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            Piece a;
            a.lo = *reinterpret_cast<const u32x4*>(arow + slot * STAGE + i * 2048 + c_lo);
            a.hi = *reinterpret_cast<const u32x4*>(arow + slot * STAGE + i * 2048 + c_hi);
#pragma unroll
            for (int f = 0; f < 2; ++f) acc[i][f] = mul_step<ELT>(fb[slot][f], a, acc[i][f]);
        }
    };
    if (nst > 0) {
#pragma unroll
        for (int d = 0; d < D - 1; ++d) issue(d, d);
        for (int s0 = 0; s0 < nst; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                // this wave's loads of the stage have landed and its reads of the stage before are in registers
                constexpr int W = (D - 2) * PER;
                __builtin_amdgcn_s_waitcnt((W & 0xF) | ((W >> 4) << 14) | 0x70);
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
                issue((d + D - 1) % D, s0 + d + D - 1);
                if (s0 + d < nst && !idle) use(d);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the partial block at the end of the rows: straight from memory, by the last split
    const int rem = p.kbytes & 127;
    if (rem && ks == p.S - 1 && !idle) {
#pragma unroll
        for (int f = 0; f < 2; ++f) fb[0][f] = tail_piece(b_base[f] + 128 * nfull + (boff[f] - 32u * j), j, rem);
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const Piece a = tail_piece(a0 + 128 * nfull + (size_t)((uint32_t)min(16 * i + r, t.rows - 1) * kb), j, rem);
#pragma unroll
            for (int f = 0; f < 2; ++f) acc[i][f] = mul_step<ELT>(fb[0][f], a, acc[i][f]);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0): nothing lands in the ring any more
    if (idle) return 0.f;
    if (p.part) {
        const int cols = MODE != 0 ? 2 * p.N : p.N;
        float* const plane = p.part + (size_t)ks * p.r_max * cols;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int m = 16 * i + r;
            if (m >= t.rows) break;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int c = col0 + (MODE != 0 ? 0 : 16 * f) + 4 * j;
                if (c < p.N) *reinterpret_cast<f32x4*>(plane + (size_t)(t.row0 + m) * cols + (MODE != 0 ? f * p.N : 0) + c) = acc[i][f];
            }
        }
        return 0.f;
    }
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        if (16 * i >= t.rows) break;
        if constexpr (MODE != 0)
            amax = fmaxf(amax, store_block<ELT, MODE>(p, t, col0, i, 0, acc[i][0], acc[i][1]));
        else
#pragma unroll
            for (int f = 0; f < 2; ++f) store_block<ELT, MODE>(p, t, col0, i, f, acc[i][f], acc[i][f]);
    }
    return amax;
}

template <int ELT, int MODE>
__global__ __launch_bounds__(kWideWaves * 64, 2) void gemm_wide_kernel(const StreamArgs p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const Tile t = locate_tile<128>(p.offsets, p.E, p.ntn * p.S, blockIdx.x);
    if (!t.valid) return;
    const int n = t.ntile / p.S, ks = t.ntile - n * p.S;
    const bool sample = ELT == kEltBf16 && p.ticks != nullptr && blockIdx.x == 0;
    unsigned long long tk_entry = 0, rt_entry = 0;
    if (sample) {
        tk_entry = __builtin_amdgcn_s_memtime();
        rt_entry = __builtin_amdgcn_s_memrealtime();
    }
    const float amax = t.rows <= 64 ? wide_tile<ELT, MODE, 4>(p, t, n, ks, smem) : wide_tile<ELT, MODE, 8>(p, t, n, ks, smem);
    if (sample && threadIdx.x == 0) {
        p.ticks[0] = __builtin_amdgcn_s_memtime() - tk_entry;
        p.ticks[1] = __builtin_amdgcn_s_memrealtime() - rt_entry;
    }
    if constexpr (ELT == kEltFp8 && MODE == 1) fold_amax(p, amax, reinterpret_cast<float*>(smem + kWideRing));
}

// The sums of the S partial planes, in split order, through the epilogue.  One thread per four columns of a row.
template <int MODE>
__global__ __launch_bounds__(256) void stream_reduce_kernel(const float* __restrict__ part, const int32_t* __restrict__ offsets,
                                                            int E, int S, int r_max, int N, bf16_t* __restrict__ C) {
    const int q = N / 4, cols = MODE != 0 ? 2 * N : N;
    const long long total = (long long)offsets[E] * q;
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < total; i += gridDim.x * 256ll) {
        const int row = (int)(i / q), c = (int)(i - (long long)row * q) * 4;
        const float* src = part + (size_t)row * cols + c;
        f32x4 v = *reinterpret_cast<const f32x4*>(src);
        f32x4 up = v;
        if (MODE != 0) up = *reinterpret_cast<const f32x4*>(src + N);
#pragma unroll 4
        for (int s = 1; s < S; ++s) {
            src += (size_t)r_max * cols;
            v += *reinterpret_cast<const f32x4*>(src);
            if (MODE != 0) up += *reinterpret_cast<const f32x4*>(src + N);
        }
        if (MODE != 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = silu_mul<kEltBf16, MODE>(v[k], up[k]);
        const u32x2 o = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
        *reinterpret_cast<u32x2*>(C + (size_t)row * N + c) = o;
    }
}

template <int MODE>
void reduce_planes(const float* part, const int32_t* offsets, int E, int S, int r_max, int N, void* C, hipStream_t s) {
    const long long groups = ((long long)r_max * N / 4 + 255) / 256;
    hipLaunchKernelGGL((stream_reduce_kernel<MODE>), dim3((int)(groups < 2048 ? groups : 2048)), dim3(256), 0, s, part, offsets, E, S,
                       r_max, N, static_cast<bf16_t*>(C));
}

template <int FB> constexpr int tile_rows() { return FB == 1 ? 64 : 128; }
template <int FB> constexpr int blocks_per_wave() { return FB == 8 ? 2 : 1; }
// LDS of a workgroup: the ring of shared_tile (two workgroups per compute unit; one where the waves share the
// contraction, which happens when there are too few workgroups for two anyway), or the partial sums of direct_tile
template <int FB, bool DIRECT> constexpr int lds_bytes() {
    return DIRECT ? 4 * FB * 1024 : FB >= 4 ? 64 * 1024 : 128 * 1024;
}

// A narrow workgroup, number `block` of its product.
template <int ELT, int MODE, int FB, bool DIRECT, int RING>
__device__ __forceinline__ void narrow_workgroup(const StreamArgs& p, unsigned block, uint8_t* smem) {
    constexpr int NBW = blocks_per_wave<FB>();
    const Tile t = locate_tile<tile_rows<FB>()>(p.offsets, p.E, p.ntn, block);
    if (!t.valid) return;
    const bool sample = ELT == kEltBf16 && p.ticks != nullptr && blockIdx.x == 0;
    unsigned long long tk_entry = 0, rt_entry = 0;
    if (sample) {
        tk_entry = __builtin_amdgcn_s_memtime();
        rt_entry = __builtin_amdgcn_s_memrealtime();
    }
    float amax = 0.f;
    if (DIRECT || t.rows <= 16) {
        amax = direct_tile<ELT, MODE, FB>(p, t, smem);
    } else if constexpr (!DIRECT) {
        if (t.rows <= 32)
            amax = shared_tile<ELT, MODE, FB, 2, RING, NBW>(p, t, smem);
        else if (t.rows <= 64 || FB == 1)
            amax = shared_tile<ELT, MODE, FB, 4, RING, NBW>(p, t, smem);
        else
            amax = shared_tile<ELT, MODE, FB, FB == 1 ? 4 : 8, RING, NBW>(p, t, smem);
    }
    if (sample && threadIdx.x == 0) {
        p.ticks[0] = __builtin_amdgcn_s_memtime() - tk_entry;
        p.ticks[1] = __builtin_amdgcn_s_memrealtime() - rt_entry;
    }
    if constexpr (ELT == kEltFp8 && MODE == 1) fold_amax(p, amax, reinterpret_cast<float*>(smem + RING));
}

// DIRECT: the launch has at most 16 rows in all, so no tile needs the ring (and more workgroups fit a compute unit).
template <int ELT, int MODE, int FB, bool DIRECT>
__global__ __launch_bounds__(256, 2) void gemm_stream_kernel(const StreamArgs p) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    narrow_workgroup<ELT, MODE, FB, DIRECT, lds_bytes<FB, DIRECT>()>(p, blockIdx.x, smem);
}

// The shared expert's product q and the routed experts' p in one launch (bf16): the first workgroups take q, whose tiles are the
// longer ones where its contraction is.
constexpr int kPairRing = 64 * 1024;   // two workgroups to a compute unit
template <int MODE, int FB, int FBS, bool DIRECT>
__global__ __launch_bounds__(256, 2) void gemm_stream_pair_kernel(const StreamArgs p, const StreamArgs q, unsigned first) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    if (blockIdx.x < first) narrow_workgroup<kEltBf16, MODE, FBS, DIRECT, kPairRing>(q, blockIdx.x, smem);
    else narrow_workgroup<kEltBf16, MODE, FB, DIRECT, kPairRing>(p, blockIdx.x - first, smem);
}

template <int ELT, int MODE, int FB, bool DIRECT>
void launch(StreamArgs p, int r_max, hipStream_t s) {
    constexpr int BN = 16 * TileAt<MODE, FB>::NF;
    constexpr int smem = lds_bytes<FB, DIRECT>() + kScratch;
    p.ntn = (p.N + BN - 1) / BN;
    auto kern = gemm_stream_kernel<ELT, MODE, FB, DIRECT>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), smem);
    hipLaunchKernelGGL(kern, dim3(grid_for(r_max, p.E, tile_rows<FB>(), p.ntn)), dim3(256), smem, s, p);
}

template <int MODE, int FB, int FBS, bool DIRECT>
void launch_pair(StreamArgs p, StreamArgs q, int r_max, hipStream_t s) {
    constexpr int BN = 16 * TileAt<MODE, FB>::NF, BNS = 16 * TileAt<MODE, FBS>::NF;
    constexpr int smem = DIRECT ? 4 * (FB > FBS ? FB : FBS) * 1024 : kPairRing;
    p.ntn = (p.N + BN - 1) / BN;
    q.ntn = (q.N + BNS - 1) / BNS;
    auto kern = gemm_stream_pair_kernel<MODE, FB, FBS, DIRECT>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), smem);
    const int first = grid_for(q.r_max, 1, tile_rows<FBS>(), q.ntn);   // a multiple of eight
    hipLaunchKernelGGL(kern, dim3(first + grid_for(r_max, p.E, tile_rows<FB>(), p.ntn)), dim3(256), smem, s, p, q, first);
}

int g_stream = -1;   // see set_gemm_stream
int forced_blocks() { return g_stream > 10 && g_stream < 20 ? g_stream - 10 : 0; }
bool forced_wide() { return g_stream >= 100 && g_stream < 2000; }
int forced_form() { return g_stream >= 20 && g_stream < 25 ? g_stream - 20 : -1; }
int forced_large_splits() { return g_stream >= 2000 ? g_stream - 2000 : 0; }

// Weight blocks of a narrow workgroup: as many as leave enough workgroups.  A wider workgroup reads the rows less often
// and keeps more weight bytes in flight, but 256 compute units want work.  Measured (us, blocks 8 / 4 / 2 / 1):
//   down 4096 x 14336, 8 experts x 8 rows    182 / 166 / 172 / 209   (256 / 512 / 1024 / 2048 workgroups)
//   the same, 2 experts x 1 row                - /  57 /  36 /  39   ( 64 / 128 /  256 /  512)
//   the same, 8 experts x 64 rows            206 / 242 / 328 / 538
//   down 3584 x 20480, one expert x 64 rows  207 / 116 /  83 /  66   ( 28 /  56 /  112 /  224)
//   the same, 500 rows                       237 / 159 / 230 / 408   (112 / 224 /  448 / 1792)
//   gate/up 2560 x 3584, 64 experts x 8 rows 385 / 392 / 537 /  -
int narrow_blocks(int r_max, int E, int N, bool swiglu) {
    if (const int fb = forced_blocks()) return r_max <= 16 ? (fb >= 4 ? 4 : 2) : swiglu && fb == 1 ? 2 : fb;
    const int experts = E < r_max ? E : r_max;
    const bool few = (long long)r_max <= 16ll * experts;   // up to 16 rows per expert on average
    const long long mt = r_max / 128 + experts;            // M-tiles, at most
    auto groups = [&](int fb) { const int bn = 16 * (swiglu ? fb / 2 : fb); return mt * ((N + bn - 1) / bn); };
    if (r_max <= 16) return groups(4) >= 400 ? 4 : 2;
    const long long want = few ? 400 : 200;
    return groups(8) >= want ? 8 : groups(4) >= want ? 4 : swiglu || groups(2) >= want ? 2 : 1;
}

template <int ELT, int MODE>
void launch_narrow(const StreamArgs& p, int r_max, hipStream_t s) {
    const int fb = narrow_blocks(r_max, p.E, p.N, MODE != 0);
    if (r_max <= 16) {
        if (fb == 4) launch<ELT, MODE, 4, true>(p, r_max, s);
        else launch<ELT, MODE, 2, true>(p, r_max, s);
    } else if (fb == 8) {
        launch<ELT, MODE, 8, false>(p, r_max, s);
    } else if (fb == 4) {
        launch<ELT, MODE, 4, false>(p, r_max, s);
    } else {
        if (MODE != 0 || fb == 2) launch<ELT, MODE, 2, false>(p, r_max, s);
        else launch<ELT, MODE, MODE != 0 ? 2 : 1, false>(p, r_max, s);
    }
}

template <int ELT, int MODE>
void launch_wide(StreamArgs p, int r_max, const StreamPlan& plan, float* part, hipStream_t s) {
    constexpr int smem = kWideRing + kScratch;
    const int bn = plan.units * (MODE != 0 ? 16 : 32);
    p.units = plan.units;
    p.S = plan.splits;
    p.part = plan.splits > 1 ? part : nullptr;
    p.ntn = (p.N + bn - 1) / bn;
    auto kern = gemm_wide_kernel<ELT, MODE>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), smem);
    hipLaunchKernelGGL(kern, dim3(grid_for(r_max, p.E, 128, p.ntn * p.S)), dim3(kWideWaves * 64), smem, s, p);
    if constexpr (ELT == kEltBf16 && MODE != 2)
        if (p.S > 1) reduce_planes<MODE>(part, p.offsets, p.E, p.S, r_max, p.N, p.C, s);
}

template <int ELT, int MODE>
void launch_any(const StreamArgs& p, int r_max, const StreamPlan& plan, float* part, hipStream_t s) {
    if (plan.kind == kPlanTiles) {
        launch_tiles(ELT, p, plan.units, r_max, s);
        return;
    }
    if constexpr (ELT != kEltF32) {
        if (plan.kind == kPlanWide) {
            launch_wide<ELT, MODE>(p, r_max, plan, part, s);
            return;
        }
    }
    launch_narrow<ELT, MODE>(p, r_max, s);
}


// ---- which kernel: estimated times (us) of the three ----
// The large tiles: tile_cost.h.  A round of the streaming workgroups takes (bytes of its weight rows) x 43 us/MB (36 where
// several M-tiles share them), plus its rows at a smaller rate, plus its start and end, which the narrow workgroups, two to a
// compute unit, mostly hide.  Fitted to gate/up and down at (E, H, F) = (1, 3584, 20480), (1, 2 and 8, 4096, 14336), (64, 3584,
// 2560), (16, 2048, 1408) and (8, 2048, 4096) with 1 to 2000 rows per expert.  Over 682
// products each (31 layers of 2 to 128 experts, 40 to 2200 rows per expert, even and skewed experts) the kernel they pick is behind
// the best of all (the large tiles at each height, narrow, wide, small tiles) by 2.9 % (gate/up), 3.3 % (down), 3.6 and 4.3 % (FP8) on
// average, by more than a tenth in 47, 32, 44 and 52 of them: up to 64 rows per expert above all, on 8 to 16 experts or with a skewed
// router, which the host cannot know (us, as picked / best: down, 12 experts x 40 rows, skewed, 3072 x 2048, 62 / 28 on the large
// tiles; 10 x 64, 2560 x 4096, 55 / 38 on the small ones; gate/up, 16 x 40, 2048 x 1408, 40 / 30 on the large; 8 x 64, 5120 x 1536, 76 / 50 on
// the small).
struct Work {
    int experts, rows, N, kbytes, r_max;
    bool swiglu, fp8, odd;   // odd: bf16 sizes that the large tiles do not take
};
constexpr int kUnitsCU = 256;   // compute units the estimates are made for (gfx950, not partitioned)

int blocks_of(int a, int b) { return (a + b - 1) / b; }

// M-tiles of all experts.  With equal experts that would be ceil(rows / height) each; a skewed router makes up to
// r_max / height more.  Half of those are counted where an expert with three times the average rows would need a second
// tile (less down to a third): a plan must not spill into another round for a tile or two (8 experts x 3264 x 1984, 618
// rows of a Zipf-1.2 router: the layer took 148 us with equal experts assumed and takes 125).  A capacity that rules the
// skew out is not known here: r_max is all that is.
double skew_share(const Work& w, int height) {
    const double near = 3.0 * w.rows / height - 1.0;
    return w.experts == 1 || w.rows <= 16 || near < 0.0 ? 0.0 : near > 1.0 ? 1.0 : near;
}
double m_tiles(const Work& w, int height) {
    const double even = (double)w.experts * blocks_of(w.rows, height), most = w.experts + (double)w.r_max / height;
    return most > even ? even + 0.5 * skew_share(w, height) * (most - even) : even;
}
double rounds_of(double tiles) { return (double)(long long)((tiles + kUnitsCU - 1) / kUnitsCU); }

// the partial planes written, read and added
double reduce_us(const Work& w, int S) {
    return S > 1 ? 4.0 + (double)S * w.r_max * w.N * (w.swiglu ? 16.0 : 8.0) / 4.5e6 : 0.0;
}

// The large tiles choose their height on the device, from the rows every expert has.  Here only the average is known: the
// time for equal experts and the time for experts of 0.4 to 1.8 times the average, half of each.
double large_us(const Work& w, int S = 1) {
    constexpr double kSpread[8] = {0.386, 0.552, 0.717, 0.883, 1.048, 1.214, 1.434, 1.766};
    const TileCosts& c = w.fp8 ? kCostFp8 : kCostBf16;
    const int ntn = blocks_of(w.N, w.swiglu ? 128 : 256);
    auto best = [&](bool equal) {
        double t = 1e30;
        for (const int height : {256, 192, 128}) {
            double mt = (double)w.experts * blocks_of(w.rows, height);
            if (!equal) {
                mt = 0.0;
                for (const double f : kSpread) mt += w.experts / 8.0 * (double)(long long)((w.rows * f + height - 1e-6) / height);
            }
            const HeightCost& h = height == 256 ? c.h256 : height == 192 ? c.h192 : c.h128;
            t = fmin(t, tiles_us(h, (float)mt, (float)w.experts, ntn * S, kUnitsCU, w.kbytes / 128 / S));
        }
        return t;
    };
    return 4.0 + (w.experts == 1 ? best(true) : 0.5 * (best(true) + best(false))) + reduce_us(w, S);
}

double narrow_us(const Work& w, int fb) {
    const int tr = fb == 1 ? 64 : 128, mt = blocks_of(w.rows, tr);
    const int nt = blocks_of(w.N, 16 * (w.swiglu ? fb / 2 : fb));
    const double tiles = m_tiles(w, tr) * nt, even_tiles = (double)mt * w.experts * nt;
    // a second workgroup on a compute unit adds less than a round while the weights are what is waited for, a third waits
    // for one of the two
    const double whole = rounds_of(tiles), over = tiles / kUnitsCU - (whole - 1.0);
    const double q = whole <= 1.0 || mt > 1 || over > 0.6 ? whole : whole - (whole <= 2.0 ? 0.6 : 0.3);
    const bool direct = w.rows <= 16;
    const int rows = w.rows < tr ? w.rows : tr;
    const double weight = direct ? 41e-6 : mt > 1 ? 36e-6 : 43e-6;
    const double risk = whole > 1.0 && even_tiles <= kUnitsCU ? 1.1 : 1.0;   // a skewed router would cost a round
    // what the same 730 products took beyond this, by weight blocks and rows per expert
    const int some = w.rows <= 16 ? 0 : w.rows <= 64 ? 1 : 2;
    constexpr double kBeyond[4][3] = {{1.4, 1.1, 1.1}, {1.2, 1.15, 1.0}, {1.05, 1.15, 0.95}, {1.0, 1.06, 1.0}};
    const double beyond = w.r_max <= 16 ? 1.0 : kBeyond[fb == 1 ? 0 : fb == 2 ? 1 : fb == 4 ? 2 : 3][some] * (w.odd && some > 0 ? 1.15 : 1.0);
    return beyond * (risk * q * w.kbytes * (16 * fb * weight + rows * (direct ? 8e-6 : 18e-6)) + (direct ? 2.0 : 3.0) * (long long)((whole + 1) / 2));
}

double wide_us(const Work& w, int units, int S) {
    const int mt = blocks_of(w.rows, 128);
    const double tiles = m_tiles(w, 128) * blocks_of(w.N, units * (w.swiglu ? 16 : 32)) * S;
    const int rows = w.rows < 128 ? w.rows : 128;
    const double round = w.kbytes / (double)S * (32 * units * (mt > 1 ? 36e-6 : 43e-6) + rows * (rows <= 64 ? 5e-6 : 12e-6)) + 10.0;
    // one workgroup to a compute unit: a tile too many costs a round, so a plan for skewed experts keeps some slack
    return rounds_of(tiles * (1.0 + 0.12 * skew_share(w, 128))) * round + reduce_us(w, S);
}

// The small tiles (gemm_tiles.hip): a start and, together with what the weights take from memory, whole rounds of workgroups (one to
// a compute unit, or what that comes to), each a start and its stages of the contraction.  From 85 to 105 % of a round on a
// part of another is counted: the experts are not equal.  Fitted to 380 products in bf16 (2 to 128 experts, 4 to 1500 rows per expert,
// routers without bias, with a normal and a Zipf-1.2 one), 90 of odd sizes, 260 in FP8, 220 in fp32; rms error 15 % where a form is
// within 40 % of the best.
struct TileForm {
    int rows, weights, blocks;   // of a tile, of a stage
    double start, block, round, power, stream, fill, more;   // us; TB/s of the weights; rounds
};
constexpr TileForm kTilesF32[] = {{32, 32, 4, 1.70, 0.584, 3.46, 2.8, 4.7, 1.06, 0.69},
                                  {32, 64, 2, 1.66, 0.528, 3.73, 1.9, 5.2, 1.06, 0.68},
                                  {32, 128, 1, 4.47, 0.523, 0.60, 1.7, 6.3, 0.59, 0.40},
                                  {64, 64, 1, 3.44, 0.507, 1.16, 6.0, 6.2, 0.60, 0.36},
                                  {128, 128, 1, 4.17, 1.215, 3.34, 6.8, 5.0, 1.02, 0.56}};
constexpr TileForm kTilesBf16[] = {{32, 64, 2, 0.77, 0.289, 4.25, 1.9, 5.6, 1.01, 0.59},
                                   {64, 64, 2, 1.16, 0.438, 3.21, 2.2, 5.6, 1.00, 0.47},
                                   {64, 128, 1, 0.70, 0.352, 3.96, 2.3, 5.6, 1.02, 0.58},
                                   {128, 128, 1, 0.78, 0.539, 3.30, 4.1, 5.6, 1.01, 0.70}};
constexpr TileForm kTilesOdd[] = {{32, 64, 2, 0.84, 0.340, 4.49, 8.0, 5.6, 0.45, 0.47},
                                  {64, 64, 2, 0.81, 0.500, 3.68, 2.6, 6.0, 1.03, 0.52},
                                  {64, 128, 1, 0.61, 0.298, 4.91, 2.0, 6.3, 1.02, 1.04},
                                  {128, 128, 1, 3.78, 0.447, 1.08, 6.6, 6.3, 1.04, 2.47},
                                  {128, 128, 1, 1.99, 0.675, 2.00, 1.6, 6.3, 0.71, 0.26}};   // four waves, two workgroups to a compute unit
constexpr TileForm kTilesFp8[] = {{32, 64, 2, 0.87, 0.276, 4.18, 2.1, 5.6, 0.80, 0.73},
                                  {64, 64, 2, 1.07, 0.340, 4.04, 2.4, 5.4, 0.87, 0.54},
                                  {64, 128, 1, 0.81, 0.322, 3.41, 2.0, 5.6, 0.91, 0.55},
                                  {128, 128, 1, 0.33, 0.538, 3.46, 7.3, 5.6, 0.82, 0.51}};
struct TileForms {
    const TileForm* form;
    int count;
};
TileForms tile_forms(int elt, bool odd) {
    if (elt == kStreamF32) return {kTilesF32, 5};
    if (elt == kStreamFp8) return {kTilesFp8, 4};
    if (odd) return {kTilesOdd, 5};
    return {kTilesBf16, 4};
}

double small_tiles_per_cu(const Work& w, const TileForm& f) {
    constexpr double kSpread[8] = {0.386, 0.552, 0.717, 0.883, 1.048, 1.214, 1.434, 1.766};   // as large_us
    double mt = 0.0;
    for (const double x : kSpread) mt += w.experts / 8.0 * (double)(long long)((w.rows * x + f.rows - 1e-6) / f.rows);
    mt = 0.5 * (mt + (double)w.experts * blocks_of(w.rows, f.rows));
    return mt * blocks_of(w.N, w.swiglu ? f.weights / 2 : f.weights) / kUnitsCU;
}

double small_tiles_us(const Work& w, const TileForm& f, double per_cu) {
    const double mul = (per_cu <= f.fill ? 1.0 : per_cu + f.more) * (f.round + f.block * blocks_of(w.kbytes, 128) / f.blocks);
    const double mem = (double)w.experts * w.N * (w.swiglu ? 2 : 1) * w.kbytes / (f.stream * 1e6);
    return f.start + pow(pow(mul, f.power) + pow(mem, f.power), 1.0 / f.power);
}

constexpr size_t kMaxPartBytes = 64u << 20;   // partial planes of one product, at most

}  // namespace

void set_gemm_stream(int v) { g_stream = v; }

void launch_stream_reduce(bool swiglu, const float* part, const int32_t* offsets, int E, int splits, int r_max, int N, void* C,
                          hipStream_t s) {
    if (swiglu) reduce_planes<1>(part, offsets, E, splits, r_max, N, C, s);
    else reduce_planes<0>(part, offsets, E, splits, r_max, N, C, s);
}

bool stream_covers(long long K_bytes) { return K_bytes <= (1 << 24); }

StreamPlan plan_stream(int elt, int r_max, int E, int N, int K, bool swiglu, bool large_ok, size_t part_bytes) {
    StreamPlan plan = {kPlanNarrow, 0, 1, 0.0};
    if (r_max <= 0) return plan;
    Work w;
    w.experts = E < r_max ? E : r_max;
    w.rows = (r_max + w.experts - 1) / w.experts;
    w.N = N;
    const long long kbytes = (long long)K * (elt == kEltF32 ? 4 : elt == kEltBf16 ? 2 : 1);
    if (large_ok && (g_stream == 0 || (g_stream < 0 && persist_grid_overridden()) || !stream_covers(kbytes))) {
        plan.kind = kPlanLarge;
        return plan;
    }
    w.kbytes = (int)kbytes;
    w.r_max = r_max;
    w.swiglu = swiglu;
    w.fp8 = elt == kStreamFp8;
    w.odd = elt == kEltBf16 && !large_ok;
    if (g_stream == 1 || forced_blocks() || !stream_covers(kbytes)) return plan;
    const TileForms small = tile_forms(elt, w.odd);
    if (forced_form() >= 0) {
        plan.kind = kPlanTiles;
        plan.units = forced_form() < small.count ? forced_form() : small.count - 1;
        return plan;
    }
    // A form is taken where it is ahead by more than a part of what the estimates are off by: more for gate/up of odd sizes, whose silu
    // they do not count, less for the fifth form of the odd sizes, whose estimate does.
    // The forms with one workgroup to a compute unit are estimated too low from the second round on, by up to two times (64 experts x 502
    // rows, 816 x 3568 gate/up, 128 x 128: 456 / 908).  In FP8, and in odd sizes, which have a form for many rounds, they are taken where
    // they come to one round (counting 5 % more, for what the experts differ): there one of them is within 2 % of the best kernel for
    // most products, with more rounds for 1 in 20.  Compared with the choice among the other kernels alone, slower by more than 3 % / 10 %
    // (without this line): of 400 odd products, 4 to 16 experts, 256 to 2048 wide, 38 / 12 (39 / 16 of 520 others), 11 % faster on average; of
    // 376, 1 to 64 experts, 256 to 6144 wide, 54 / 14 (95 / 66 of 560 others), 11 %; of 262 in FP8 9 / 2 (16 / 11 of 458), 4 %.  The
    // worst are behind by a third: few experts or a skewed router, whose tiles spill into a second round.  In bf16 the line would
    // change nothing, the large tiles being ahead there by their estimate.
    auto rounds_fit = [&](int f, double per_cu) { return !(w.odd || w.fp8) || f == 4 || per_cu <= 1.05; };
    auto margin = [&](int f) { return elt == kEltF32 ? 1.0 : !w.odd ? 1.1 : f == 4 ? 1.05 : swiglu ? 1.25 : 1.1; };
    int form = 0;
    double form_us = 1e30;
    for (int f = 0; f < small.count; ++f) {
        const double per_cu = small_tiles_per_cu(w, small.form[f]);
        if (!rounds_fit(f, per_cu)) continue;
        const double t = margin(f) * small_tiles_us(w, small.form[f], per_cu);
        if (t < form_us) {
            form_us = t;
            form = f;
        }
    }
    if (elt == kEltF32) {
        // Up to 12 rows per expert most tiles have at most 16 and the narrow kernel's form for those is the better one (us, fp32
        // instruction / tiles: 4 experts x 4 rows, 572 x 632 4.6 / 7.5; 8 x 12, 308 x 456 6.0 / 8.2; 16 x 12, 996 x 460 27 / 18)
        if (2 * r_max <= 25 * w.experts) return plan;
        plan.kind = kPlanTiles;
        plan.units = form;
        return plan;
    }
    // a split leaves at least 16 blocks of the contraction to a workgroup
    auto splits_fit = [&](int S) {
        return S == 1 || (elt == kEltBf16 && kbytes / 128 >= 16 * S && (size_t)S * r_max * N * (swiglu ? 8 : 4) <= part_bytes);
    };
    if (forced_wide()) {
        plan.kind = kPlanWide;
        plan.units = g_stream % 100;
        plan.splits = g_stream / 100;
        while (!splits_fit(plan.splits)) plan.splits /= 2;
        return plan;
    }
    // a split of the large tiles leaves at least eight k-tiles to a tile
    auto large_splits_fit = [&](int S) {
        return large_ok && elt == kEltBf16 && kbytes / 128 >= 8 * S && (size_t)S * r_max * N * (swiglu ? 8 : 4) <= part_bytes;
    };
    if (forced_large_splits()) {
        plan.kind = large_ok ? kPlanLarge : kPlanNarrow;
        if (large_splits_fit(forced_large_splits())) plan.splits = forced_large_splits();
        return plan;
    }
    double best = g_stream == 2 ? 1e30 : narrow_us(w, narrow_blocks(r_max, E, N, swiglu));
    if (g_stream < 0 && large_ok) {
        const double t = large_us(w);
        if (t < best) {
            best = t;
            plan.kind = kPlanLarge;
        }
    }
    // Only the layer's shared expert has room for partial sums, and of one expert the M-tiles are known.  The
    // shared expert's two products, H x Fs = 3584 x 20480 (us, large tiles whole / split wide workgroups / so): 300 tokens 363 / 247
    // / 188, 500 tokens 423 / 334 / 255, 1000 534 / 574 / 422, 2000 771 / 1040 / 749; 1500 tokens, 2048 x 8192 195 / 231 / 161.
    if (g_stream < 0 && w.experts == 1)
        for (int S = 2; S <= 16 && large_splits_fit(S); ++S) {
            const double t = large_us(w, S);
            if (t < best) {
                best = t;
                plan.kind = kPlanLarge;
                plan.splits = S;
            }
        }
    // The small tiles; not with up to 16 rows in all, where the narrow kernel has no ring, nor where most tiles of an odd
    // size have as few.  (us, as chosen without the small tiles / so, a pass: expert-parallel share, 2 experts x 302 rows, 5376 x
    // 1408 104 / 81; FP8, 4 experts x 24 rows, 5632 x 2560 85 / 69; training, 8 x 58 rows, 2432 x 4992 727 / 559.  Over 730 products in all 7 % faster
    // on average, 30 % where the form changes; slower by more than 3 %: 31, mostly few experts with a skewed router.)
    if (g_stream < 0 && r_max > 16 && !(w.odd && w.rows <= 16) && form_us < best) {
        best = form_us;
        plan.kind = kPlanTiles;
        plan.units = form;
        plan.splits = 1;
    }
    for (int units = 8; units >= 3; --units)
        for (int S = 1; S <= 16; S *= 2) {
            if (!splits_fit(S)) break;
            const double t = wide_us(w, units, S);
            if (t < best) {
                best = t;
                plan.kind = kPlanWide;
                plan.units = units;
                plan.splits = S;
            }
        }
    plan.us = best;
    return plan;
}

static StreamArgs stream_args(int elt, const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0, const void* B1,
                              void* C) {
    StreamArgs p;
    p.A = static_cast<const uint8_t*>(A);
    p.offsets = offsets;
    p.B0 = static_cast<const uint8_t*>(B0);
    p.B1 = static_cast<const uint8_t*>(B1);
    p.C = C;
    p.GU = nullptr;
    p.amax = nullptr;
    p.ticks = persist_clock_sample();
    p.s0 = p.s1 = p.s2 = 0.f;
    p.E = E; p.N = N; p.ntn = 0;
    p.units = 0; p.S = 1; p.r_max = r_max; p.part = nullptr;
    p.kbytes = K * (elt == kEltF32 ? 4 : elt == kEltBf16 ? 2 : 1);
    return p;
}

static int g_pair_blocks = -1;
void set_pair_blocks(int v) { g_pair_blocks = v; }

int plan_pair(int elt, const StreamPlan& routed, int r_max, int E, int N, int K, const StreamPlan& shared, int tokens, int sN, int sK,
              bool swiglu) {
    // silu as both products have it alone; a narrow workgroup of one weight block has no pair
    auto plain = [&](int n, int k) { return !swiglu || (n % 64 == 0 && k % 64 == 0 && k >= 128); };
    if (g_pair_blocks == 0 || g_stream >= 0 || elt != kStreamBf16 || routed.kind != kPlanNarrow || tokens > 128 || !plain(N, K) ||
        !plain(sN, sK) || narrow_blocks(r_max, E, N, swiglu) == 1)
        return 0;
    // With a capacity there may be fewer routed rows than tokens.  Workgroups for up to 16 rows in all have no ring, and the shared
    // expert's rows would need one.
    if (r_max <= 16 && tokens > 16) return 0;
    const int forced = g_pair_blocks < 0 ? -1 : swiglu ? g_pair_blocks / 10 : g_pair_blocks % 10;
    if (forced >= 0) return forced;
    // What the second launch costs are its first and last microseconds, an end of the first one in which compute units stand idle, and
    // partial sums (us of the layer, one after the other / so: 3 tokens, 32 experts, 1152 x 1280, shared 2112 48 / 36; one token, 32,
    // 6144 x 768, 17152 183 / 152; 27 tokens, 64, 1024 x 2176, 6144 123 / 99; 42 tokens, 16, 7040 x 4352, 14080 723 / 663).
    // The figures below: 731 layers of 2 to 64 experts, 1024 to 6336 x 512 to 8192, shared 512 to 20288, each product of each width
    // paired alone, per layer against one after the other.
    if (swiglu) {
        // Workgroups of the same length, so the two lists become one; as wide as the tokens ask for (paired always: 1 to 16 tokens 0.940 /
        // 0.953 / 0.957 of the time with 2 / 4 / 8 blocks, 17 to 48 0.996 / 0.985 / 0.991, 65 to 128 1.011 / 0.997 / 0.992).  Where all of
        // them find a place at once in narrower ones, an eight-block one would only last longer: 20 tokens, 4 experts, 3712 x 960, with
        // 2112 65 one after the other, 59 / 64 / 78; 121 tokens, 8, 3968 x 704, 2752 93, 87 / 92 / 107.
        const int fb = narrow_blocks(r_max, E, N, true), slots = 2 * kUnitsCU;
        const int experts = E < r_max ? E : r_max, rows = (r_max + experts - 1) / experts;
        const double own = (double)experts * blocks_of(rows, 128) * blocks_of(N, 8 * fb);
        int fbs = r_max <= 16 ? 2 : tokens <= 16 ? 4 : 8;
        if (tokens > 16)
            while (fbs > 2 && fbs / 2 >= fb && own + blocks_of(sN, 4 * fbs) <= slots) fbs /= 2;
        const double more = blocks_of(sN, 8 * fbs) * (double)fbs / fb;
        const double both = fmax(1.0, (own + more) / slots) / fmax(1.0, own / slots);
        // More tokens take the wide kernel further ahead alone.  64 tokens on 64 experts, 3584 x 2560, with 20480 more take 7 us longer
        // so: 5.0 rounds of routed workgroups become 5.6.  332 layers of 17 to 128 tokens take 2.8 % less on average, 47 of them more than
        // 1 % longer, 27 more than 3 %, the worst 12 %: few experts whose workgroups leave half the chip idle, and a long shared
        // product, whose rows suit the wide kernel.  Factors of 0.9 to 1.04 pair the same layers; from 1.06 on gains are lost before losses.
        return (tokens <= 48 ? 0.98 : tokens <= 64 ? 1.04 : 1.1) * routed.us * both < routed.us + shared.us + 4.0 ? fbs : 0;
    }
    // The shared expert's contraction is the longer one, and one of its workgroups takes so long for it, beside the others (us for 128
    // bytes: 0.1 with both operands straight to registers; else the more the fewer stages of the rows the ring holds).  It should end
    // with the routed experts' and have its own weights to read as well.  (Half of the shared product's time: 1 to 16 tokens 0.972 of
    // the time, 12 of 141 layers slower by more than 1 %, the worst by 7; none of it 0.977, 4, 4; paired always 0.978, 30, 18.  17 to 48
    // tokens 0.981, 7 of 202, 7 / 0.983, 3, 4 / 0.996, 60, 23; more tokens 0.995, 1 of 144, 2 / 0.995, 1, 2 / 1.119, 92, 99.)
    // Four blocks where the output is wide enough for as many workgroups as with two: above 16 tokens, from 5632 columns on, where
    // pairing gains 1.6 % with four and 0.9 % with two, below 0.3 % and 1.4 %.
    const double serial = blocks_of(2 * sK, 128) * (tokens <= 16 ? 0.11 : fmax(0.2, 0.0115 * tokens));
    return serial <= routed.us + 0.5 * shared.us ? (tokens > 16 && sN >= 5632 ? 4 : 2) : 0;
}

void launch_stream_pair(int blocks, const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0, const void* B1,
                        void* C, const void* sA, const int32_t* s_offsets, int tokens, int sN, int sK, const void* sB0, const void* sB1,
                        void* sC, hipStream_t s) {
    const StreamArgs p = stream_args(kStreamBf16, A, offsets, r_max, E, N, K, B0, B1, C);
    const StreamArgs q = stream_args(kStreamBf16, sA, s_offsets, tokens, 1, sN, sK, sB0, sB1, sC);
    const int fb = narrow_blocks(r_max, E, N, B1 != nullptr);
    const bool direct = r_max <= 16 && tokens <= 16;   // both products' rows
    auto go = [&](auto mode, auto own) {
        constexpr int MODE = decltype(mode)::value, FB = decltype(own)::value;
        if constexpr (FB <= 4) {
            if (direct) {
                launch_pair<MODE, FB, 2, true>(p, q, r_max, s);
                return;
            }
        }
        // the widths that plan_pair chooses: gate/up eight, four, or two beside two; down four or two
        if constexpr (MODE == 1) {
            if (blocks == 8) {
                launch_pair<MODE, FB, 8, false>(p, q, r_max, s);
                return;
            }
        }
        if constexpr (MODE == 0 || FB == 2) {
            if (blocks == 2) {
                launch_pair<MODE, FB, 2, false>(p, q, r_max, s);
                return;
            }
        }
        launch_pair<MODE, FB, 4, false>(p, q, r_max, s);
    };
    auto width = [&](auto mode) {
        if (fb == 8) go(mode, std::integral_constant<int, 8>{});
        else if (fb == 4) go(mode, std::integral_constant<int, 4>{});
        else go(mode, std::integral_constant<int, 2>{});
    };
    if (B1) width(std::integral_constant<int, 1>{});
    else width(std::integral_constant<int, 0>{});
}

size_t stream_part_bytes(int elt, int r_max, int E, int N, int K, bool swiglu, bool large_ok) {
    const StreamPlan plan = plan_stream(elt, r_max, E, N, K, swiglu, large_ok, kMaxPartBytes);
    return plan.splits > 1 ? (size_t)plan.splits * r_max * N * (swiglu ? 8 : 4) : 0;
}

void launch_stream(const StreamPlan& plan, int elt, const void* A, const int32_t* offsets, int r_max, int E, int N, int K,
                   const void* B0, const void* B1, void* C, void* GU, float s0, float s1, float s2, float* amax,
                   float* part, hipStream_t s) {
    StreamArgs p = stream_args(elt, A, offsets, r_max, E, N, K, B0, B1, C);
    p.GU = GU;
    p.amax = amax;
    p.s0 = s0; p.s1 = s1; p.s2 = s2;
    if (elt == kEltF32) {
        if (B1) launch_any<kEltF32, 1>(p, r_max, plan, part, s); else launch_any<kEltF32, 0>(p, r_max, plan, part, s);
    } else if (elt == kEltBf16) {
        if (GU) launch_any<kEltBf16, 2>(p, r_max, plan, part, s);
        else if (B1 && full_silu(p)) launch_any<kEltBf16, 3>(p, r_max, plan, part, s);
        else if (B1) launch_any<kEltBf16, 1>(p, r_max, plan, part, s);
        else launch_any<kEltBf16, 0>(p, r_max, plan, part, s);
    } else {
        if (B1) launch_any<kEltFp8, 1>(p, r_max, plan, part, s); else launch_any<kEltFp8, 0>(p, r_max, plan, part, s);
    }
}

}  // namespace moe
