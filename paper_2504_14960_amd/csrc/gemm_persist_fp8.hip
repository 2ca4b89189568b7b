// Grouped expert GEMM (a3) on FP8 operands with per-tensor delayed scaling
// (Section 4.5, "FP8 Training Performance").
//
// Same persistent engine as gemm_persist.hip, byte for byte on the memory
// side: output tiles of 256, 192 or 128 rows x 256 columns, LDS rows of 128
// bytes (here 128 E4M3 values, so a k-tile spans 128 of the contraction index),
// three LDS stages for the weight tile and two for the activation tile filled
// by direct global->LDS loads, the k-tiles of successive output tiles as one stream, register-
// resident tile scheduler, epilogue staged through the idle LDS stage.
//
// What differs: the matrix instruction is the 16x16x128 FP8 MFMA (each lane
// feeds 32 bytes of a row: a whole k-tile per instruction, twice the math per
// byte moved), and so the halves of a period are not two steps of the
// contraction but the two halves of a wave's columns: the first multiplies all
// its rows by the first half of its weight rows, the second by the rest.  The
// fragments of one k-tile (128 registers beside the 256 accumulators) are all
// there is room for: each is read again, for the next k-tile, as soon as it has
// been used for the last time.  And the epilogues differ: the gate/up GEMM
// dequantises g and u, applies SwiGLU, records max |h| for the next step's scale
// and writes h as E4M3 with this step's (delayed) scale; the down GEMM
// dequantises into bf16.  Bound by power with many rows (see gemm_persist.hip).
// Measured, gate/up and down, us, 32x32x64 / this: 8 experts of 16384 rows, 6144 x
// 16384, 2550 and 1262 / 2458 and 1191 (2.7 and 2.8 PFLOP/s); 8 x 4096 rows, 6144 x
// 2048, 645 and 372 / 605 and 350; 64 skewed experts of 82000 rows, 4096 x 1408, 822
// and 502 / 783 and 479.
#include <type_traits>

#include "fp8_convert.h"
#include "gemm_persist.h"
#include "gemm_stream.h"

namespace moe {

namespace {

typedef __attribute__((ext_vector_type(8))) int i32x8;

// Epilogue of the gate/up GEMM: h = silu(g) * u from the dequantised
// accumulators, one byte per value.  Staged through a wave-private LDS patch of
// W = 16*FO bytes per row (16-byte granules XOR-swizzled by the row) so that the
// global stores are whole 16-byte pieces along the rows.
template <int FM, int FN, int WM>
__device__ __forceinline__ float store_h_fp8(f32x4 (&acc)[FM][FN], int t_row0, int t_rows, int t_n0, uint8_t* C,
                                             int N, int wm, int wn, int lane, uint8_t* stage, float dq_gate,
                                             float dq_up, float scale_h, float amax) {
    constexpr int FO = FN / 2;
    constexpr int W = FO * 16;        // bytes per staged row
    constexpr int GPR = W / 16;       // granules per row: a fragment's columns are one
    constexpr int RP256 = 256 / W;    // rows per 256 bytes
    constexpr int RPI = 1024 / W;     // rows per 64-lane read
    static_assert(W <= 256 && 256 % W == 0 && 32 % RPI == 0, "staged row must divide the bank window");
    asm volatile("" : "+v"(lane));    // keeps the addresses below from being hoisted out of the tile loop
    const int fr = lane & 15, fk = lane >> 4;
    static_assert((16 / RP256) % GPR == 0, "both row blocks of a patch have the same swizzle");
    const int xw = (fr / RP256) & (GPR - 1);
    uint8_t* wrow = stage + fr * W + 4 * fk;
    const int rl = lane / GPR, gl = lane % GPR;
    const int col = t_n0 + wn * (FO * 16) + gl * 16;
#pragma unroll
    for (int i = 0; i < FM / 2; ++i) {   // 32 rows at a time
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[2 * i + q][j]));   // see gemm_persist.hip
#pragma unroll
            for (int j = 0; j < FO; ++j) {
                float hv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float g = acc[2 * i + q][j][u] * dq_gate;
                    const float up = acc[2 * i + q][j + FO][u] * dq_up;
                    hv[u] = g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * up;   // silu(g) * up
                    amax = fmaxf(amax, fabsf(hv[u]));
                }
                const uint32_t packed = f32x4_to_e4m3(hv[0] * scale_h, hv[1] * scale_h, hv[2] * scale_h,
                                                      hv[3] * scale_h);
                // lane's 4 columns: bytes 16j + 4fk .. +3 of the row
                *reinterpret_cast<uint32_t*>(wrow + q * (16 * W) + ((j ^ xw) << 4)) = packed;
                asm volatile("" : "+v"(amax));   // now, or the values wait for it in scratch memory
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const int first = wm * WM + i * 32;
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int row = it * RPI + rl;
            const int xr = (row / RP256) & (GPR - 1);
            const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * W + ((gl ^ xr) << 4));
            const int grow = first + row;
            if (grow < t_rows && col < N) *reinterpret_cast<u32x4*>(C + (size_t)(t_row0 + grow) * N + col) = v;
        }
    }
    return amax;
}

// Epilogue of the down GEMM: y = acc * dq as bf16, staged like the bf16 kernel's.
template <int FM, int FN, int WM>
__device__ __forceinline__ void store_y_bf16(f32x4 (&acc)[FM][FN], int t_row0, int t_rows, int t_n0, bf16_t* C,
                                             int N, int wm, int wn, int lane, uint8_t* stage, float dq) {
    constexpr int W = FN * 32;
    constexpr int GPR = W / 16;
    constexpr int RP256 = 256 / W;
    constexpr int RPI = 1024 / W;
    static_assert(W <= 256 && 256 % W == 0, "staged row must divide the bank window");
    asm volatile("" : "+v"(lane));
    const int fr = lane & 15, fk = lane >> 4;
    static_assert((16 / RP256) % GPR == 0, "both row blocks of a patch have the same swizzle");
    const int xw = (fr / RP256) & (GPR - 1);
    uint8_t* wrow = stage + fr * W + 8 * (fk & 1);
    const int gw = fk >> 1;           // a fragment is two granules wide
    const int rl = lane / GPR, gl = lane % GPR;
    const int col = t_n0 + wn * (FN * 16) + gl * 8;
#pragma unroll
    for (int i = 0; i < FM / 2; ++i) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[2 * i + q][j]));
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4& a = acc[2 * i + q][j];
                u32x2 o;
                o[0] = pack2_bf16(a[0] * dq, a[1] * dq);
                o[1] = pack2_bf16(a[2] * dq, a[3] * dq);
                *reinterpret_cast<u32x2*>(wrow + q * (16 * W) + (((2 * j + gw) ^ xw) << 4)) = o;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const int first = wm * WM + i * 32;
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int row = it * RPI + rl;
            const int xr = (row / RP256) & (GPR - 1);
            const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * W + ((gl ^ xr) << 4));
            const int grow = first + row;
            if (grow < t_rows && col < N) *reinterpret_cast<u32x4*>(C + (size_t)(t_row0 + grow) * N + col) = v;
        }
    }
}

// A [rows, K] E4M3, B0/B1 [E, N, K] E4M3 (SWIGLU: gate and up), K a multiple of
// 128.  SWIGLU: C is h [rows, N] E4M3, s0/s1 dequantise g/u, s2 scales h, amax
// receives max |h|.  Otherwise C is y [rows, N] bf16 and s0 dequantises it.
// DEEP_B: the weight tile, not the activation tile, gets the three LDS stages (see gemm_persist.hip).
template <int BM, bool SWIGLU, bool IDLE_SKIP, bool DEEP_B>
__device__ __forceinline__ void fp8_body(
    const uint8_t* __restrict__ A, const int32_t* __restrict__ offsets, int E, int N, int K,
    const uint8_t* __restrict__ B0, const uint8_t* __restrict__ B1, void* __restrict__ C, int ntn, float s0,
    float s1, float s2, float* __restrict__ amax_out, uint8_t* smem) {
    constexpr int BN = 256, WGM = 2, WGN = 2;
    constexpr int NW = WGM * WGN;
    constexpr int NT = NW * 64;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / 16, FN = WN / 16;
    constexpr int ROWB = 128;                   // bytes (= E4M3 values) per tile row and k-tile
    constexpr int CPR = ROWB / 16;
    constexpr int RPP = NT / CPR;
    constexpr int PA = BM / RPP, PB = BN / RPP;
    constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB;
    constexpr int B_REGION = (DEEP_B ? 2 : 3) * A_BYTES;
    constexpr int PBD = SWIGLU ? PB / 2 : PB;   // passes of one weight matrix
    // "early" operand: two slots; "late": three, fetched half a period earlier (see gemm_persist.hip)
    constexpr int PE = DEEP_B ? PA : PB, PL = DEEP_B ? PB : PA;
    constexpr int OUTN = SWIGLU ? BN / 2 : BN;
    constexpr int NLOAD = PA + PB;
    constexpr int FH = FN / 2;                  // weight fragments of half a period
    constexpr int NSLOT = FM * FH;              // one MFMA (32 cycles) per slot
    static_assert(PE <= NSLOT && PL <= NSLOT && 4 * FH <= NSLOT, "slots");
    static_assert((DEEP_B ? 2 * A_BYTES + 3 * B_BYTES : 3 * A_BYTES + 2 * B_BYTES) <= 160 * 1024, "tile stages exceed the 160 KiB of LDS");
    static_assert(NW * 32 * (FN * 32) <= (DEEP_B ? B_BYTES : A_BYTES), "epilogue patches must fit into one slot of the late operand");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    const uint8_t* const B1b = SWIGLU ? B1 : B0;
    TileSched<BM> sched;
    sched.init(offsets, E, ntn, lane);
    int ti = 0;
    const uint8_t *c_a, *c_b0, *c_b1, *n_a, *n_b0, *n_b1;
    uint32_t c_alim, c_blim, n_alim, n_blim;
    int c_row0, c_rows, c_n0, n_row0, n_rows, n_n0;
    bool n_valid;
    {
        const PTile t = sched.get(0, A, B0, B1b, N, (size_t)K, OUTN);
        if (!t.valid) return;
        c_a = t.a; c_b0 = t.b0; c_b1 = t.b1; c_alim = t.a_lim; c_blim = t.b_lim;
        c_row0 = t.row0; c_rows = t.rows; c_n0 = t.n0;
    }
    auto fetch_next_tile = [&](int i) {
        const PTile t = sched.get(i, A, B0, B1b, N, (size_t)K, OUTN);
        n_a = t.a; n_b0 = t.b0; n_b1 = t.b1; n_alim = t.a_lim; n_blim = t.b_lim;
        n_row0 = t.row0; n_rows = t.rows; n_n0 = t.n0; n_valid = t.valid;
    };
    fetch_next_tile(1);

    // global side of the direct loads (see gemm_persist.hip)
    const int frow = tid / CPR, fchunk = tid % CPR;
    const uint32_t rowb = (uint32_t)K;
    const uint32_t vrow = (uint32_t)frow * rowb;
    const uint32_t vswz = (uint32_t)((fchunk ^ lds_swizzle(frow)) * 16);
    const uint32_t step = (uint32_t)RPP * rowb;
    const int wbase = (wave * 64 / CPR) * ROWB;
    // the k-tile that a period fetches: see gemm_persist.hip
    const int KT = K / ROWB;
    const uint8_t *f_a, *f_b0, *f_b1;
    uint32_t off_a[PA], off_b[PBD];
    auto fetch_from = [&](const uint8_t* a, const uint8_t* b0, const uint8_t* b1, uint32_t alim, uint32_t blim) {
        f_a = a; f_b0 = b0; f_b1 = b1;
        uint32_t first = vrow;   // hidden, or the rows' sums below are kept across the whole loop, in scratch memory
        asm volatile("" : "+v"(first));
#pragma unroll
        for (int p = 0; p < PA; ++p) off_a[p] = min(first + (uint32_t)p * step, alim) + vswz;  // ragged tail: a valid row again
#pragma unroll
        for (int p = 0; p < PBD; ++p) off_b[p] = min(first + (uint32_t)p * step, blim) + vswz;
    };
    auto fetch_step = [&]() {
        f_a += ROWB;
        f_b0 += ROWB;
        if (SWIGLU) f_b1 += ROWB;
    };
    auto fetch_a = [&](int p, uint8_t* st) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(f_a + off_a[p]),
                                         (__attribute__((address_space(3))) void*)(st + p * RPP * ROWB + wbase), 16, 0, 0);
    };
    auto fetch_b = [&](int p, uint8_t* st) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((p >= PBD ? f_b1 : f_b0) + off_b[p % PBD]),
                                         (__attribute__((address_space(3))) void*)(st + p * RPP * ROWB + wbase), 16, 0, 0);
    };
    // load i of a period: the early operand's passes first, then the late operand's
    auto fetch_one = [&](int i, uint8_t* ld_b, uint8_t* ld_a) {
        if constexpr (DEEP_B) {
            if (i < PA) fetch_a(i, ld_a);
            else fetch_b(i - PA, ld_b);
        } else {
            if (i < PB) fetch_b(i, ld_b);
            else fetch_a(i - PB, ld_a);
        }
    };
    auto advance = [&](int kt) {
        fetch_step();
        if (kt == KT - 2) {
            if (n_valid)
                fetch_from(n_a, n_b0, n_b1, n_alim, n_blim);
            else {   // behind the last tile its last two k-tiles again, never used
                f_a -= 2 * ROWB;
                f_b0 -= 2 * ROWB;
                if (SWIGLU) f_b1 -= 2 * ROWB;
            }
        }
    };

    const int fr = lane & 15, fk = lane >> 4;
    int a_off[FM], b_off[FN];
    const int f_sw = lds_swizzle(fr);
#pragma unroll
    for (int i = 0; i < FM; ++i) a_off[i] = (wm * WM + i * 16 + fr) * ROWB;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        int r;
        if (SWIGLU)
            r = (j < FH) ? (wn * (WN / 2) + j * 16 + fr) : (BN / 2 + wn * (WN / 2) + (j - FH) * 16 + fr);
        else
            r = wn * WN + j * 16 + fr;
        b_off[j] = r * ROWB;
    }

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

    // Fragments as two 16-byte pieces: a lane's 32 bytes are the pieces fk and fk + 4 of its row (activations and weights use
    // the same bytes, which is all the instruction needs; neighbouring pieces in one read have no bank conflicts).
    u32x4 afh[FM][2], bfh[FN][2];
    auto read_a = [&](const uint8_t* sa, int i) {
#pragma unroll
        for (int h = 0; h < 2; ++h) afh[i][h] = *reinterpret_cast<const u32x4*>(sa + a_off[i] + (((4 * h + fk) ^ f_sw) << 4));
    };
    auto read_b = [&](const uint8_t* sb, int j) {
#pragma unroll
        for (int h = 0; h < 2; ++h) bfh[j][h] = *reinterpret_cast<const u32x4*>(sb + b_off[j] + (((4 * h + fk) ^ f_sw) << 4));
    };
    auto frag = [&](const u32x4 (&h)[2]) -> i32x8 {
        i32x8 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            v[t] = (int)h[0][t];
            v[4 + t] = (int)h[1][t];
        }
        return v;
    };
    // Half a period: all rows by the weight fragments of half HALF.  Slots of {one MFMA; the next fragment's reads; at most one
    // direct load}.  Half 0 reads the weight fragments of half 1 (sb: this k-tile); half 1 the activation fragments, each
    // behind its last use, and the weight fragments of half 0 (sa, sb: the next k-tile).
    auto half_period = [&](auto half, const uint8_t* sa, const uint8_t* sb, int ld_begin, int ld_end, uint8_t* ld_b, uint8_t* ld_a) {
        constexpr int HALF = decltype(half)::value;
        int ld = ld_begin;
#pragma unroll
        for (int slot = 0; slot < NSLOT; ++slot) {
            // boustrophedon over the wave's blocks: successive MFMAs share one operand fragment
            const int i = slot / FH, jj = (i & 1) ? FH - 1 - slot % FH : slot % FH, j = HALF * FH + jj;
            // E4M3 x E4M3 (formats 0, 0), no block scales; weight fragment first as in the bf16 kernels
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(frag(bfh[j]), frag(afh[i]), acc[i][j], 0, 0, 0, 0, 0, 0);
            // the first MFMA waits for the reads before this half: keep the new ones behind it
            if (slot == 0) __builtin_amdgcn_sched_barrier(0);
            if (slot % 4 == 1 && slot / 4 < FH) read_b(sb, (1 - HALF) * FH + slot / 4);
            if (HALF == 1 && slot % FH == FH - 1) read_a(sa, i);
            if (ld < ld_end && slot == 1 + (ld - ld_begin) * NSLOT / (ld_end - ld_begin)) {
                fetch_one(ld, ld_b, ld_a);
                ++ld;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using First = std::integral_constant<int, 0>;
    using Second = std::integral_constant<int, 1>;
    auto first_reads = [&](const uint8_t* sa, const uint8_t* sb) {
#pragma unroll
        for (int j = 0; j < FH; ++j) read_b(sb, j);
#pragma unroll
        for (int i = 0; i < FM; ++i) read_a(sa, i);
    };

    uint8_t* const a_region = smem;
    uint8_t* const b_region = smem + B_REGION;
    {
        // late(0), early(0), late(1); the first two must have landed before the first fragment reads
        fetch_from(c_a, c_b0, c_b1, c_alim, c_blim);
#pragma unroll
        for (int i = PE; i < NLOAD; ++i) fetch_one(i, b_region, a_region);
#pragma unroll
        for (int i = 0; i < PE; ++i) fetch_one(i, b_region, a_region);
        fetch_step();
#pragma unroll
        for (int i = PE; i < NLOAD; ++i) fetch_one(i, b_region + (DEEP_B ? B_BYTES : 0), a_region + (DEEP_B ? 0 : A_BYTES));
        __builtin_amdgcn_s_waitcnt(0x0F70 | (PL & 0xF) | ((PL >> 4) << 14));  // vmcnt(PL)
        __builtin_amdgcn_s_barrier();
        first_reads(a_region, b_region);
#pragma unroll
        for (int i = 0; i < PE; ++i) fetch_one(i, b_region + B_BYTES, a_region + A_BYTES);
    }

    float amax = 0.f;
    // slots of k-tiles kt, kt+1 (, kt+2): three for the late operand, two for the early one
    int a0 = 0, a1 = A_BYTES, a2 = DEEP_B ? 0 : 2 * A_BYTES;
    int b0 = 0, b1 = B_BYTES, b2 = DEEP_B ? 2 * B_BYTES : 0;
    auto rotate = [&]() {
        if constexpr (DEEP_B) {
            const int ta = a0; a0 = a1; a1 = ta;
            const int tb = b0; b0 = b1; b1 = b2; b2 = tb;
        } else {
            const int ta = a0; a0 = a1; a1 = a2; a2 = ta;
            const int tb = b0; b0 = b1; b1 = tb;
        }
    };
    for (;;) {
        // IDLE_SKIP (launches with many experts): a wave whose rows of the tile all lie past its last valid row
        // only issues its share of the loads and meets the barriers, up to the last k-tile (see gemm_persist.hip)
        const bool wave_idle = IDLE_SKIP && wm * WM >= c_rows;   // wave-uniform
        int kt = 0;
        if (IDLE_SKIP) {
            for (const int idle = wave_idle ? KT - 1 : 0; kt < idle; ++kt) {
                advance(kt);
#pragma unroll
                for (int i = PE; i < NLOAD; ++i) fetch_one(i, b_region + (DEEP_B ? b2 : b1), a_region + (DEEP_B ? a1 : a2));
                __builtin_amdgcn_s_waitcnt((PL & 0xF) | ((PL >> 4) << 14));
                __builtin_amdgcn_s_barrier();
#pragma unroll
                for (int i = 0; i < PE; ++i) fetch_one(i, b_region + b0, a_region + a0);
                rotate();
            }
        }
        for (; kt < KT; ++kt) {
            advance(kt);
            __builtin_amdgcn_sched_barrier(0);
            // half 0: late(kt+2)
            half_period(First{}, a_region + a0, b_region + b0, PE, NLOAD, b_region + (DEEP_B ? b2 : b1), a_region + (DEEP_B ? a1 : a2));
            // all but the PL youngest loads (those of late(kt+2)) have landed; this
            // wave's fragment reads of k-tile kt are in registers
            __builtin_amdgcn_s_waitcnt((PL & 0xF) | ((PL >> 4) << 14));
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // half 1: first fragments of k-tile kt+1, early(kt+2) into the freed slot
            half_period(Second{}, a_region + a1, b_region + b1, 0, PE, b_region + b0, a_region + a0);
            rotate();
        }
        uint8_t* stage = (DEEP_B ? b_region + b2 : a_region + a2) + wave * (32 * FN * 32);
        if (SWIGLU) {
            const float m = store_h_fp8<FM, FN, WM>(acc, c_row0, c_rows, c_n0, static_cast<uint8_t*>(C), N, wm, wn, lane, stage,
                                                    s0, s1, s2, amax);
            if (!wave_idle) amax = m;
        } else
            store_y_bf16<FM, FN, WM>(acc, c_row0, c_rows, c_n0, static_cast<bf16_t*>(C), N, wm, wn, lane, stage, s0);
        if (!n_valid) break;
        c_a = n_a; c_b0 = n_b0; c_b1 = n_b1; c_alim = n_alim; c_blim = n_blim;
        c_row0 = n_row0; c_rows = n_rows; c_n0 = n_n0;
        ++ti;
        fetch_next_tile(ti + 1);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave is done with its patch
        __builtin_amdgcn_s_barrier();
    }
    wait_vmcnt0();  // loads past the end of the last tile may still be landing in LDS
    if (SWIGLU && amax_out) {
        // max |h| over the wave, then one atomic per wave; h >= 0 as a float compares like its bit pattern.
        // Rows past the tile's valid rows may have contributed garbage: they were computed from re-read valid
        // rows of the same expert, so they are values h takes anyway.
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        if (lane == 0 && amax > __builtin_nontemporal_load(amax_out))   // *amax_out only grows; NaN compares false
            atomicMax(reinterpret_cast<int*>(amax_out), __float_as_int(amax));
    }
}

// Tiles of 256, 192 or 128 rows, chosen on the device from the rows that every expert really has; `rows` != 0: those.
template <bool SWIGLU, bool IDLE_SKIP, bool DEEP_B>
__global__ __launch_bounds__(256) void gemm_fp8_persist_kernel(
    const uint8_t* __restrict__ A, const int32_t* __restrict__ offsets, int E, int N, int K,
    const uint8_t* __restrict__ B0, const uint8_t* __restrict__ B1, void* __restrict__ C, int ntn, float s0,
    float s1, float s2, float* __restrict__ amax_out, int rows) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    if constexpr (!DEEP_B) {
        fp8_body<256, SWIGLU, IDLE_SKIP, DEEP_B>(A, offsets, E, N, K, B0, B1, C, ntn, s0, s1, s2, amax_out, smem);
    } else {
        const int height = rows != 0 ? rows : pick_height(kCostFp8, offsets, E, ntn, K / 128, threadIdx.x & 63);
        if (height == 256)
            fp8_body<256, SWIGLU, IDLE_SKIP, DEEP_B>(A, offsets, E, N, K, B0, B1, C, ntn, s0, s1, s2, amax_out, smem);
        else if (height == 192)
            fp8_body<192, SWIGLU, IDLE_SKIP, DEEP_B>(A, offsets, E, N, K, B0, B1, C, ntn, s0, s1, s2, amax_out, smem);
        else
            fp8_body<128, SWIGLU, IDLE_SKIP, DEEP_B>(A, offsets, E, N, K, B0, B1, C, ntn, s0, s1, s2, amax_out, smem);
    }
}

static int g_fp8_deep_b = 1;   // three LDS stages for the weight tile (0: for the activation tile)

template <bool SWIGLU>
void launch_fp8(const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0, const void* B1,
                void* C, float s0, float s1, float s2, float* amax, hipStream_t s) {
    constexpr int OUTN = SWIGLU ? 128 : 256;
    constexpr size_t smem = (size_t)(3 * 256 + 2 * 256) * 128;
    const int ntn = (N + OUTN - 1) / OUTN;
    const bool idle_skip = persist_idle_skip(E);
    const bool deep = g_fp8_deep_b != 0;
    auto kern = deep ? (idle_skip ? gemm_fp8_persist_kernel<SWIGLU, true, true> : gemm_fp8_persist_kernel<SWIGLU, false, true>)
                     : (idle_skip ? gemm_fp8_persist_kernel<SWIGLU, true, false> : gemm_fp8_persist_kernel<SWIGLU, false, false>);
    static OncePerDevice lds[2][2];
    allow_lds(lds[deep][idle_skip], reinterpret_cast<const void*>(kern), (int)smem);
    const int grid = min(persist_grid(), grid_for(r_max, E, deep ? 128 : 256, ntn));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), smem, s, static_cast<const uint8_t*>(A), offsets, E, N, K,
                       static_cast<const uint8_t*>(B0), static_cast<const uint8_t*>(B1), C, ntn, s0, s1, s2, amax,
                       persist_tile_rows());
}

}  // namespace

void set_fp8_deep_b(int v) { g_fp8_deep_b = v; }

bool fp8_ffn_supported(int H, int F) { return H % 128 == 0 && F % 128 == 0 && H >= 256 && F >= 256; }

void launch_expert_ffn_fp8(const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E,
                           const void* w_gate, const void* w_up, const void* w_down, float dq_gate, float dq_up,
                           float scale_h, float dq_down, void* h, float* amax_h, void* y_perm, int phase,
                           hipStream_t s) {
    if (phase & 1) {
        const StreamPlan plan = plan_stream(kStreamFp8, r_max, E, F, H, true, true, 0);
        if (plan.kind != kPlanLarge)
            launch_stream(plan, kStreamFp8, x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, nullptr, dq_gate, dq_up, scale_h,
                          amax_h, nullptr, s);
        else
            launch_fp8<true>(x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, dq_gate, dq_up, scale_h, amax_h, s);
    }
    if (phase & 2) {
        const StreamPlan plan = plan_stream(kStreamFp8, r_max, E, H, F, false, true, 0);
        if (plan.kind != kPlanLarge)
            launch_stream(plan, kStreamFp8, h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, nullptr, dq_down, 0.f, 0.f,
                          nullptr, nullptr, s);
        else
            launch_fp8<false>(h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, dq_down, 0.f, 0.f, nullptr, s);
    }
}

}  // namespace moe
