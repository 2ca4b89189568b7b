// Grouped expert GEMM (a3) for experts with few rows, and for every shape the large-tile kernels do not take (fp32
// layers, bf16 layers whose H or F is not a multiple of 64).
//
// With few rows per expert the product is a read of the weights: what bounds it is how many bytes of them are on
// their way from HBM at a time.  The large-tile kernel has one workgroup per 256 weight rows, so the down projection of
// two experts (4096 outputs, one decoded token) is 32 workgroups on 256 compute units, and a 256-row tile is multiplied
// whatever it holds.  Here a workgroup owns 16 to 128 weight rows, the weights go straight from memory into the
// matrix instruction's operand registers (each byte is wanted by one wave only; two 16-byte loads per lane cover
// whole 128-byte lines of 16 rows), and the rows of the tile decide how the other operand travels:
//
//   up to 16 rows    registers as well (direct_tile): no barrier and no LDS in the loop, the waves take the blocks of
//                    the contraction in turn;
//   17 to 128 rows   through LDS, shared by the waves (shared_tile); with more rows than that per expert the read of
//                    the rows outweighs the weights and the large tiles are the better kernel.
//
// Measured (bf16, weights of several launches so that no cache holds them; before: the large-tile kernel):
//   down, 2 experts x 1 row, 4096 x 14336     231 us -> 36 us   (6.6 TB/s of weights)
//   gate/up, 64 experts x 8 rows, 2560 x 3584  420 us -> 385 us  (6.1 TB/s);  down 234 us -> 206 us
//   gate/up, 8 experts x 8 rows, 14336 x 4096  470 us -> 325 us  (5.8 TB/s);  down 292 us -> 166 us
//   the same in FP8                            230 us -> 161 us  (5.8 TB/s);  down 148 us ->  86 us
//   12 experts, 2331 rows, H = 1000, F = 1416  330 us ->  47 us  (plain FMA kernel before);  down 293 us -> 25 us
//   fp32, 8 experts, 512 rows, H = 128, F = 256  27 us ->  9 us;  down 31 us -> 8 us
#include "fp8_convert.h"
#include "gemm_stream.h"
#include "gemm_tile.h"

namespace moe {

namespace {

constexpr int NW = 4;   // waves per workgroup

constexpr int kEltF32 = kStreamF32, kEltBf16 = kStreamBf16, kEltFp8 = kStreamFp8;

// What a lane holds of a 128-byte k-step of one operand row: lane group j = lane / 16 of row lane % 16 holds bytes
// 16 j .. 16 j + 15 of both 64-byte halves (a load instruction then asks for whole 64-byte sectors).  The contraction order inside a step is the same for both operands, so any
// assignment of bytes to contraction slots is right.
struct Piece {
    u32x4 lo, hi;
};

// 16 bytes of global memory (the pointer arithmetic below hides from the compiler where its pointers point)
__device__ __forceinline__ u32x4 ld16(const uint8_t* p) {
    return *(const __attribute__((address_space(1))) u32x4*)p;
}

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
};

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

// Where a workgroup starts in its n steps of the contraction.  Operand rows lie a whole row apart, so workgroups that
// walk the contraction in step ask the same few memory channels at a time.  Depends on the weight tile only, so a row's
// result does not depend on which rows it is computed with.  Measured (us, all from step 0 / so): down 4096 x 14336, 2
// experts x 8 rows 51.0 / 44.6, 8 experts x 32 rows 187.7 / 175.1; gate/up 1408 x 2048, 16 experts x 8 rows 43.2 / 38.7.
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

// Stores the 16 x 16 output block (row block i, column block f) from its sums: v (with SwiGLU the gate's) and up.  A
// lane holds row 16 i + lane % 16 and four consecutive columns.  Returns the largest |h| stored (FP8).
template <int ELT, int MODE>
__device__ __forceinline__ float store_block(const StreamArgs& p, const Tile& t, int n0, int i, int f, f32x4 v, f32x4 up) {
    constexpr bool SWIGLU = MODE != 0;
    const int lane = threadIdx.x & 63;
    const int m = 16 * i + (lane & 15), col = n0 + 16 * f + 4 * (lane >> 4);
    const bool in = m < t.rows && col < p.N;
    const size_t at = (size_t)(t.row0 + m) * p.N + col;
    float amax = 0.f;
    if constexpr (SWIGLU) {
        if constexpr (ELT == kEltFp8) { v *= p.s0; up *= p.s1; }
        if (MODE == 2 && in) {
            u32x2 g2 = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])};
            u32x2 u2 = {pack2_bf16(up[0], up[1]), pack2_bf16(up[2], up[3])};
            bf16_t* gu = static_cast<bf16_t*>(p.GU) + (size_t)(t.row0 + m) * (2 * p.N) + col;
            *reinterpret_cast<u32x2*>(gu) = g2;
            *reinterpret_cast<u32x2*>(gu + p.N) = u2;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (ELT == kEltF32)
                v[q] = (v[q] / (1.f + expf(-v[q]))) * up[q];
            else
                v[q] = v[q] * __builtin_amdgcn_rcpf(1.f + __expf(-v[q])) * up[q];
        }
    } else if constexpr (ELT == kEltFp8) {
        v *= p.s0;
    }
    if (!in) return amax;
    if constexpr (ELT == kEltF32) {
        *reinterpret_cast<f32x4*>(static_cast<float*>(p.C) + at) = v;
    } else if constexpr (ELT == kEltFp8 && SWIGLU) {
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

template <int FB> constexpr int tile_rows() { return FB == 1 ? 64 : 128; }
template <int FB> constexpr int blocks_per_wave() { return FB == 8 ? 2 : 1; }
// LDS of a workgroup: the ring of shared_tile (two workgroups per compute unit; one where the waves share the
// contraction, which happens when there are too few workgroups for two anyway), or the partial sums of direct_tile
template <int FB, bool DIRECT> constexpr int lds_bytes() {
    return DIRECT ? 4 * FB * 1024 : FB >= 4 ? 64 * 1024 : 128 * 1024;
}

// DIRECT: the launch has at most 16 rows in all, so no tile needs the ring (and more workgroups fit a compute unit).
template <int ELT, int MODE, int FB, bool DIRECT>
__global__ __launch_bounds__(256, 2) void gemm_stream_kernel(const StreamArgs p) {
    constexpr int RING = lds_bytes<FB, DIRECT>();
    constexpr int NBW = blocks_per_wave<FB>();
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const Tile t = find_tile<tile_rows<FB>()>(p.offsets, p.E, p.ntn, reinterpret_cast<int*>(smem + RING));
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
    if constexpr (ELT == kEltFp8 && MODE == 1) {
        // one atomic per wave; h >= 0 as a float compares like its bit pattern, and *amax only grows
        if (p.amax) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
            if ((threadIdx.x & 63) == 0 && amax > __builtin_nontemporal_load(p.amax))
                atomicMax(reinterpret_cast<int*>(p.amax), __float_as_int(amax));
        }
    }
}

template <int ELT, int MODE, int FB, bool DIRECT>
void launch(StreamArgs p, int r_max, hipStream_t s) {
    constexpr int BN = 16 * TileAt<MODE, FB>::NF;
    constexpr int smem = lds_bytes<FB, DIRECT>() + (kMaxExperts + 2) * 4;
    p.ntn = (p.N + BN - 1) / BN;
    auto kern = gemm_stream_kernel<ELT, MODE, FB, DIRECT>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(grid_for(r_max, p.E, tile_rows<FB>(), p.ntn)), dim3(256), smem, s, p);
}

// Weight blocks per workgroup: as many as leave enough workgroups.  A wider workgroup reads the rows less often and
// keeps more weight bytes in flight, but 256 compute units want work.  Measured (us, blocks 8 / 4 / 2 / 1):
//   down 4096 x 14336, 8 experts x 8 rows    182 / 166 / 172 / 209   (256 / 512 / 1024 / 2048 workgroups)
//   the same, 2 experts x 1 row                - /  57 /  36 /  39   ( 64 / 128 /  256 /  512)
//   the same, 8 experts x 64 rows            206 / 242 / 328 / 538
//   down 3584 x 20480, one expert x 64 rows  207 / 116 /  83 /  66   ( 28 /  56 /  112 /  224)
//   the same, 500 rows                       237 / 159 / 230 / 408   (112 / 224 /  448 / 1792)
//   gate/up 2560 x 3584, 64 experts x 8 rows 385 / 392 / 537 /  -
template <int ELT, int MODE>
void launch_any(const StreamArgs& p, int r_max, hipStream_t s) {
    const int experts = p.E < r_max ? p.E : r_max;
    const bool few = (long long)r_max <= 16ll * experts;   // up to 16 rows per expert on average
    const long long mt = r_max / 128 + experts;            // M-tiles, at most
    auto groups = [&](int fb) { const int bn = 16 * (MODE != 0 ? fb / 2 : fb); return mt * ((p.N + bn - 1) / bn); };
    if (r_max <= 16) {
        if (groups(4) >= 400)
            launch<ELT, MODE, 4, true>(p, r_max, s);
        else
            launch<ELT, MODE, 2, true>(p, r_max, s);
        return;
    }
    const long long want = few ? 400 : 200;
    if (groups(8) >= want)
        launch<ELT, MODE, 8, false>(p, r_max, s);
    else if (groups(4) >= want)
        launch<ELT, MODE, 4, false>(p, r_max, s);
    else if (MODE != 0 || groups(2) >= want)
        launch<ELT, MODE, 2, false>(p, r_max, s);
    else
        launch<ELT, MODE, MODE != 0 ? 2 : 1, false>(p, r_max, s);
}

int g_stream = -1;   // -1: by size; 0: only where no other kernel takes the shape; 1: always

}  // namespace

void set_gemm_stream(int v) { g_stream = v; }

bool stream_covers(long long K_bytes) { return K_bytes <= (1 << 24); }

// Against the 256-row tiles (us, large tiles / here): gate/up 2560 x 3584 on 64 experts with 8 rows each 420 / 385, with
// 16 rows 438 / 410, with 31 rows 427 / 433, with 62 rows 440 / 490; down there 234 / 206, 238 / 231, 239 / 255, 252 /
// 284: the line lies at 24 rows per expert.  With more rows than that the large tiles lose only where they are too few
// to occupy the compute units (down 3584 x 20480 for one expert's 500 rows, 28 tiles: 356 / 159).
bool stream_preferred(int r_max, int E, int N, bool swiglu) {
    if (g_stream >= 0) return g_stream != 0;
    if (persist_grid_overridden()) return false;
    const int experts = E < r_max ? E : r_max;
    if ((long long)r_max <= 24ll * experts) return true;
    const int outn = swiglu ? 128 : 256;
    return (long long)(r_max / 256 + experts) * ((N + outn - 1) / outn) <= 128;
}

void launch_stream(int elt, const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0,
                   const void* B1, void* C, void* GU, float s0, float s1, float s2, float* amax, hipStream_t s) {
    StreamArgs p;
    p.A = static_cast<const uint8_t*>(A);
    p.offsets = offsets;
    p.B0 = static_cast<const uint8_t*>(B0);
    p.B1 = static_cast<const uint8_t*>(B1);
    p.C = C;
    p.GU = GU;
    p.amax = amax;
    p.ticks = persist_clock_sample();
    p.s0 = s0; p.s1 = s1; p.s2 = s2;
    p.E = E; p.N = N; p.ntn = 0;
    p.kbytes = K * (elt == kEltF32 ? 4 : elt == kEltBf16 ? 2 : 1);
    if (elt == kEltF32) {
        if (B1) launch_any<kEltF32, 1>(p, r_max, s); else launch_any<kEltF32, 0>(p, r_max, s);
    } else if (elt == kEltBf16) {
        if (GU) launch_any<kEltBf16, 2>(p, r_max, s);
        else if (B1) launch_any<kEltBf16, 1>(p, r_max, s);
        else launch_any<kEltBf16, 0>(p, r_max, s);
    } else {
        if (B1) launch_any<kEltFp8, 1>(p, r_max, s); else launch_any<kEltFp8, 0>(p, r_max, s);
    }
}

}  // namespace moe
