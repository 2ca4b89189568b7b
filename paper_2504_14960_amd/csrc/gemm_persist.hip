// Grouped expert GEMM (a3), persistent kernel: one workgroup per compute unit
// walks a static list of output tiles and treats their k-tiles as ONE stream.
//
// Tiles of 256, 192 or 128 rows (pick_height) x 256 columns, k-tiles of 64
// elements through LDS: direct global->LDS loads spread in source order between
// the matrix instructions, one barrier per k-tile, three LDS stages for the
// weight tile and two for the activation tile.
//
// What bounds it with many rows per expert is power: the clock settles at what
// the board allows, and the time is the energy of a tile.  So the matrix
// instruction is the 16x16x32 one, which adds a contraction of 32 to its
// accumulators where 32x32x16 adds one of 16 (half the accumulator traffic; the
// bare loop over workload-like operands in LDS, probe.hip: 1889 TFLOP/s, with the
// other 1777 to 1826), and
// four waves of 128 x 128 share a tile, not eight of 128 x 64 (a third fewer LDS
// bytes per k-tile).  With one wave per SIMD nothing covers what stands between
// two matrix instructions, so the k loop holds little else: 128 of them, 32
// fragment reads, 16 loads and 27 scalar and vector instructions per k-tile, the
// sources of the loads kept from k-tile to k-tile.  Measured, gate/up and down, us,
// eight waves of 32x32x16 / this: 8 experts of 16384 rows, 6144 x 16384, 5200 and
// 2700 / 4850 and 2435 (1.36 PFLOP/s each); 8 x 4096 rows, 6144 x 2048, 1310 and 686 /
// 1168 and 627; 64 skewed experts of 82000 rows, 4096 x 1408, 1663 and 919 / 1480
// and 836.  Few rows and short contractions run on eight waves (launch_persist_chosen);
// with many, eight waves against this, on another card,
// neither with scratch memory: 5122 and 2618 / 4875 and 2434; 1255 and 668 / 1188 and
// 636; 1632 and 896 / 1487 and 834.
//
// What happens at a tile boundary:
//
//  * the loads issued during the last two k-tiles of a tile already fetch the
//    first two k-tiles of the workgroup's NEXT tile, so the pipeline never
//    drains and there is no per-tile prologue;
//  * the tile scheduler (prefix of per-expert M-tile counts) lives in registers
//    of every wave and is evaluated with wave-level operations only: no LDS, no
//    barrier, no memory access per tile (the weight gradients', whose tiles are
//    short: 64 tiles at a time, which reads the offsets and searches them across
//    the lanes once more, behind the stores of the 64th);
//  * the epilogue goes through the one LDS stage that is idle at that moment:
//    every wave transposes its accumulators through a private, XOR-swizzled
//    patch of it and writes whole 16-byte-per-lane row segments, instead of
//    8-byte pieces scattered over 32 rows per store instruction.
//
// The workgroups never wait for one another, so any number of them may be
// resident; the launcher asks for one per compute unit.
#include <type_traits>

#include "gemm_persist.h"
#include "gemm_stream.h"


namespace moe {

static int g_persist_workgroups = 0;  // 0: one per compute unit
static int g_persist_idle_skip = -1;  // -1: chosen from the expert count; 0 / 1: forced
static int g_persist_tile_rows = 0;   // 0: chosen from the rows of the experts; 256, 192 or 128: forced
static unsigned long long* g_persist_ticks = nullptr;  // device cell pair of the clock sample, or none

bool persist_grid_overridden() { return g_persist_workgroups > 0; }

int persist_grid() {
    // every one of the 8 tile shares needs a workgroup with its residue mod 8
    if (g_persist_workgroups > 0) return g_persist_workgroups < 8 ? 8 : g_persist_workgroups;
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            cus = prop.multiProcessorCount;
        if (cus < 8) cus = 256;
    }
    return cus;
}

namespace {

// Epilogue through LDS.  Two fragment row blocks at a time the wave writes its
// 32 x (16*FO) bf16 outputs (8 bytes per lane per store: row l%16 of a block, 4
// consecutive columns) into a private patch of W = 32*FO bytes per row, 16-byte
// granules XOR-swizzled by the row so that neither side has bank conflicts, reads
// them back as whole 16-byte granules along the rows and stores those.
//
// MODE 0: C = acc.  MODE 1: C = silu(gate) * up, the gate in the first half of
// the fragments and the up projection in the second.  MODE 2: as 1, and the
// two pre-activations themselves go to GU [rows, 2N] (gate in columns
// [0, N), up in [N, 2N)) for a backward pass that does not recompute them.
// STREAM_OUT (weight gradients of few rows per expert): the output is as many bytes as the operands' panels that the next tiles
// find in the L2, and nobody reads it soon, so it is streamed past them.
template <int FM, int FN, int WM, int MODE, bool ACC_IN_AGPR, bool STREAM_OUT>
__device__ __forceinline__ void store_tile_staged(f32x4 (&acc)[FM][FN], int t_row0, int t_rows, int t_n0,
                                                  bf16_t* __restrict__ C, bf16_t* __restrict__ GU, int N, int wm,
                                                  int wn, int lane, uint8_t* stage) {
    constexpr bool SWIGLU = MODE == 1 || MODE == 2;
    constexpr int FO = SWIGLU ? FN / 2 : FN;
    constexpr int W = FO * 32;        // bytes per staged row
    constexpr int GPR = W / 16;       // granules per row
    constexpr int RP256 = 256 / W;    // rows per 256 bytes (one pass over all banks)
    constexpr int RPI = 1024 / W;     // rows per 64-lane read
    static_assert(W <= 256 && 256 % W == 0, "staged row must divide the bank window");
    // the lane-dependent addresses below are cheap to recompute per tile; hiding
    // the lane id keeps them from being hoisted out of the tile loop, where they
    // would occupy registers across the whole k loop
    asm volatile("" : "+v"(lane));
    const int fr = lane & 15, fk = lane >> 4;
    static_assert((16 / RP256) % GPR == 0, "both row blocks of a patch have the same swizzle");
    const int xw = (fr / RP256) & (GPR - 1);
    uint8_t* wrow = stage + fr * W + 8 * (fk & 1);
    const int gw = fk >> 1;           // a fragment is two granules wide
    const int rl = lane / GPR, gl = lane % GPR;
    const int col = t_n0 + wn * (FO * 16) + gl * 8;
    const uint32_t pitch = (uint32_t)N * 2u;
    const uint32_t c_off = col < N ? (uint32_t)rl * pitch + (uint32_t)col * 2u : kNoColumn;   // STREAM_OUT
#pragma unroll
    for (int i = 0; i < FM / 2; ++i) {
        // 32 rows at a time.  With 256 accumulators per lane they live in
        // the accumulation registers; naming them there once more per block keeps
        // the copies into ordinary registers from being made all at once, which
        // would push the loop's long-lived values out to scratch memory
        __builtin_amdgcn_sched_barrier(0);
        if (ACC_IN_AGPR) {
#pragma unroll
            for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[2 * i][j]), "+a"(acc[2 * i + 1][j]));
        }
        if (MODE == 2) {
            // the pre-activations first: gate half, then up half, each through the same patch
#pragma unroll
            for (int half = 0; half < 2; ++half) {
#pragma unroll
                for (int j = 0; j < FO; ++j) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const f32x4& a = acc[2 * i + q][j + half * FO];
                        u32x2 o;
                        o[0] = pack2_bf16(a[0], a[1]);
                        o[1] = pack2_bf16(a[2], a[3]);
                        *reinterpret_cast<u32x2*>(wrow + q * (16 * W) + (((2 * j + gw) ^ xw) << 4)) = o;
                    }
                }
#pragma unroll
                for (int it = 0; it < 32 / RPI; ++it) {
                    const int row = it * RPI + rl;
                    const int xr = (row / RP256) & (GPR - 1);
                    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * W + ((gl ^ xr) << 4));
                    const int grow = wm * WM + i * 32 + row;
                    if (grow < t_rows && col < N)
                        *reinterpret_cast<u32x4*>(GU + (size_t)(t_row0 + grow) * (2 * N) + half * N + col) = v;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int j = 0; j < FO; ++j) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (SWIGLU) {
                        const float g = acc[2 * i + q][j][u];
                        const float up = acc[2 * i + q][j + FO][u];
                        v[u] = g * __builtin_amdgcn_rcpf(1.f + __expf(-g)) * up;  // silu(g) * up
                    } else {
                        v[u] = acc[2 * i + q][j][u];
                    }
                }
                u32x2 o;
                o[0] = pack2_bf16(v[0], v[1]);
                o[1] = pack2_bf16(v[2], v[3]);
                *reinterpret_cast<u32x2*>(wrow + q * (16 * W) + (((2 * j + gw) ^ xw) << 4)) = o;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (MODE == 3) {
            // the saved pre-activations of this row block first (their addresses do not depend on the staging)
            u32x4 gv[32 / RPI], uv[32 / RPI];
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int grow = wm * WM + i * 32 + it * RPI + rl;
                gv[it] = u32x4{0u, 0u, 0u, 0u};
                uv[it] = u32x4{0u, 0u, 0u, 0u};
                if (grow < t_rows && col < N) {
                    const bf16_t* src = GU + (size_t)(t_row0 + grow) * (2 * N) + col;
                    gv[it] = *reinterpret_cast<const u32x4*>(src);
                    uv[it] = *reinterpret_cast<const u32x4*>(src + N);
                }
            }
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int row = it * RPI + rl;
                const int xr = (row / RP256) & (GPR - 1);
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * W + ((gl ^ xr) << 4));
                const int grow = wm * WM + i * 32 + row;
                u32x4 og, ou;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float dgv[2], duv[2];
#pragma unroll
                    for (int hlf = 0; hlf < 2; ++hlf) {
                        const float dh = __uint_as_float(hlf ? (v[j] & 0xffff0000u) : (v[j] << 16));
                        const float g = __uint_as_float(hlf ? (gv[it][j] & 0xffff0000u) : (gv[it][j] << 16));
                        const float up = __uint_as_float(hlf ? (uv[it][j] & 0xffff0000u) : (uv[it][j] << 16));
                        const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-g));
                        duv[hlf] = dh * g * sg;
                        dgv[hlf] = dh * up * sg * (1.f + g * (1.f - sg));
                    }
                    og[j] = pack2_bf16(dgv[0], dgv[1]);
                    ou[j] = pack2_bf16(duv[0], duv[1]);
                }
                if (grow < t_rows && col < N) {
                    bf16_t* dst = C + (size_t)(t_row0 + grow) * (2 * N) + col;
                    *reinterpret_cast<u32x4*>(dst) = og;
                    *reinterpret_cast<u32x4*>(dst + N) = ou;
                }
            }
        } else if constexpr (STREAM_OUT) {
            const int first = wm * WM + i * 32;
            const RowBuffer out(C + (size_t)(t_row0 + first) * N, t_rows - first, pitch);
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int row = it * RPI + rl;
                const int xr = (row / RP256) & (GPR - 1);
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * W + ((gl ^ xr) << 4));
                out.store(v, c_off + (uint32_t)(it * RPI) * pitch);
            }
        } else {
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int row = it * RPI + rl;
                const int xr = (row / RP256) & (GPR - 1);
                const u32x4 v = *reinterpret_cast<const u32x4*>(stage + row * W + ((gl ^ xr) << 4));
                const int grow = wm * WM + i * 32 + row;
                if (grow < t_rows && col < N) *reinterpret_cast<u32x4*>(C + (size_t)(t_row0 + grow) * N + col) = v;
            }
        }
    }
}

// Partial sums as they are, [rows, N] or, gate and up, [rows, 2 N] fp32: a lane holds one row and four columns at a time.
template <int FM, int FN, int WM, int WN, bool SWIGLU>
__device__ __forceinline__ void store_partial(f32x4 (&acc)[FM][FN], int t_row0, int t_rows, int t_n0, float* __restrict__ part,
                                              int N, int wm, int wn, int lane) {
    asm volatile("" : "+v"(lane));   // see store_tile_staged
    const int fr = lane & 15, fk = lane >> 4;
    constexpr int FO = SWIGLU ? FN / 2 : FN;
    const int pitch = SWIGLU ? 2 * N : N;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int row = wm * WM + i * 16 + fr;
        if (row >= t_rows) continue;
        float* const prow = part + (size_t)(t_row0 + row) * pitch;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = t_n0 + wn * (FO * 16) + (j % FO) * 16 + 4 * fk;
            if (col < N) *reinterpret_cast<f32x4*>(prow + (j >= FO ? N : 0) + col) = acc[i][j];
        }
    }
}

// GROUPK (MODE 0 only): the weight-gradient form C [E, M, N]; A and B0 are the
// transposed operands [M, K] and [N, K] with K = elements per row, every expert
// contracting over its own zero-padded column segment (see WgradSched); `ntn`
// carries M.  Experts without rows get no tiles here (their gradient is zeroed
// by wgrad_zero_empty_kernel).
//
// KMAJ (with GROUPK): the same product on the activations AS THE LAYER HOLDS THEM, A [rows, lda] and B0 [rows,
// ldb] row-major (K carries lda), no transposed copies.  A k-tile is then 64 rows x 256 features (512-byte LDS
// rows, 16-byte pieces XOR-swizzled by the row), and a fragment's eight contraction values per lane come from two
// transposing LDS loads (ds_read_b64_tr_b16: the 16 lanes of a group address a 4 x 16 block, four consecutive
// features each, and lane i receives feature i of the four rows).  Both operands are read the same way, so they
// agree on the order of the contraction values.  Rows past the expert's last one are fetched from the zero row
// that GU points at (512 bytes of zeros).
//
// DEEP_B: which operand gets the three LDS stages.  false: the activation tile (three stages, fetched two k-tiles
// ahead) and two stages for the weight tile; true: the other way round -- the weights are what streams in from
// HBM (every weight byte is used by one M-group only), the activation panels are re-read from the caches.
template <int BM, int BN, int WGM, int WGN, int MODE, bool GROUPK, bool KMAJ, bool IDLE_SKIP, bool DEEP_B, bool BY_ROUND,
          bool STREAM_OUT, bool SPLIT>
__device__ __forceinline__ void persist_body(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ offsets, int E, int N, int K,
    const bf16_t* __restrict__ B0, const bf16_t* __restrict__ B1, bf16_t* __restrict__ C, bf16_t* __restrict__ GU,
    int ntn, int ldb, int splits, int plane_rows, unsigned long long* __restrict__ ticks, uint8_t* smem) {
    static_assert(!SPLIT || (!GROUPK && MODE <= 1), "the forward's products can be split");
    static_assert(!GROUPK || MODE == 0, "the weight-gradient form has a plain epilogue");
    static_assert(!KMAJ || (GROUPK && BM == 256 && BN == 256 && WGM * WGN == 8), "row-major form: 256 x 256 tiles, 8 waves");
    static_assert(!(KMAJ && DEEP_B), "the row-major form keeps three activation stages");
    constexpr bool SWIGLU = MODE == 1 || MODE == 2;
    constexpr int BK = 64;
    constexpr int NW = WGM * WGN;
    constexpr int NT = NW * 64;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int FM = WM / 16, FN = WN / 16;
    constexpr int CPR = BK / 8;
    constexpr int RPP = NT / CPR;               // tile rows fetched per pass of the workgroup
    constexpr int PA = BM / RPP, PB = BN / RPP;
    constexpr int PBD = SWIGLU ? PB / 2 : PB;   // passes of one weight matrix
    constexpr int ROWB = BK * 2;
    constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB;
    constexpr int B_REGION = (DEEP_B ? 2 : 3) * A_BYTES;   // the activation slots, then the weight slots
    // "early" operand: two slots, a k-tile fetched as soon as the slot is read, behind the barrier of the period before;
    // "late" operand: three slots, fetched half a period earlier
    constexpr int PE = DEEP_B ? PA : PB, PL = DEEP_B ? PB : PA;
    constexpr int OUTN = SWIGLU ? BN / 2 : BN;
    constexpr int NLOAD = PA + PB;              // direct loads per thread per k-tile
    constexpr int NREAD = FM + FN;
    constexpr int NSLOT = FM * FN;
    // Activation fragments with one set of registers, read again as soon as the k-step has used them; the others, and the
    // weight fragments, have two sets.  (Eight waves and 256 rows: 128 accumulators leave no room for two sets of all.)
    constexpr int A_ONE = NW == 8 && FM == 8 ? FM - 2 : 0;
    constexpr int NTWO = NREAD - A_ONE;
    // The early operand's loads are issued behind the barrier, in k-step 1, the late operand's in k-step 0: what a barrier
    // waits for is a whole period old.  (Tiles of 128 rows with the early ones, the activations',
    // one behind the other and not spread over the k-step: us, spread / so, 16 experts x 60 rows, 4096 x 1408, gate/up 77.8 / 75.3, but 24 x
    // 130, 2816 x 768, 39.1 / 41.1 and 12 x 315, 2944 x 512, 33.4 / 34.6; over 96 products of 12 layers level.)
    // STREAM_OUT: stores of a tile's epilogue, per wave (RowBuffer).  Loads and stores are counted together and complete in
    // order, and a wait for the loads behind an epilogue is a wait for its stores.  All that the first period of a tile waits
    // for was asked for in front of the stores of the tile before, so it need not wait for them; the second period, 1.5 us
    // later, does.  (Three gradients of 64 experts x 172 rows, 6144 x 2048: 1738 us waiting at once, 1643 so, 1222 with
    // no stores at all; of 64 x 390, 5248 x 1792: 1780 and 1720.)
    constexpr int NSTORE = STREAM_OUT ? FM / 2 * (32 / (1024 / (FN * 32))) : 0;
    constexpr int FO = SWIGLU ? FN / 2 : FN;
    static_assert(BM % RPP == 0 && BN % RPP == 0 && RPP % 8 == 0, "tile rows must divide into fetch passes");
    static_assert(!SWIGLU || ((BN / 2) % RPP == 0 && FN % 2 == 0), "gate/up halves must be pass- and fragment-aligned");
    static_assert(PL + NSTORE < 64, "vmcnt holds 6 bits");
    static_assert(PE <= NSLOT && PL <= NSLOT && NTWO <= NSLOT, "not enough slots for the loads and reads");
    static_assert((DEEP_B ? 2 * A_BYTES + 3 * B_BYTES : 3 * A_BYTES + 2 * B_BYTES) <= 160 * 1024, "tile stages exceed the 160 KiB of LDS");
    static_assert(NW * 32 * FO * 32 <= (DEEP_B ? B_BYTES : A_BYTES), "epilogue patches must fit into one slot of the late operand");

    // clock sample (ticks != NULL): shader-clock and 100 MHz reference ticks workgroup 0 spends in the kernel
    const bool sample = ticks != nullptr && blockIdx.x == 0;
    unsigned long long tk_entry = 0, rt_entry = 0;
    if (sample) {
        tk_entry = __builtin_amdgcn_s_memtime();
        rt_entry = __builtin_amdgcn_s_memrealtime();
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    const uint8_t* const Ab = reinterpret_cast<const uint8_t*>(A);
    const uint8_t* const B0b = reinterpret_cast<const uint8_t*>(B0);
    const uint8_t* const B1b = SWIGLU ? reinterpret_cast<const uint8_t*>(B1) : B0b;

    typename std::conditional<KMAJ, WgradSchedKM<BM, BN>,
                              typename std::conditional<GROUPK, WgradSched<BM, BN>, TileSched<BM, BY_ROUND>>::type>::type sched;
    if constexpr (GROUPK)
        sched.init(offsets, E, ntn, N, lane);
    else
        sched.init(offsets, E, ntn, lane, SPLIT ? splits : 1);
    auto get_tile = [&](int i) -> PTile {
        if constexpr (KMAJ)
            return sched.get(i, Ab, B0b, ntn, N, K, ldb);
        else if constexpr (GROUPK)
            return sched.get(i, Ab, B0b, ntn, N, K);
        else
            return sched.template get<SPLIT>(i, Ab, B0b, B1b, N, (size_t)K * 2, OUTN, splits);
    };
    // current and next tile of this workgroup, as plain wave-uniform scalars
    int ti = 0;
    const uint8_t *c_a, *c_b0, *c_b1, *n_a, *n_b0, *n_b1;
    uint32_t c_alim, c_blim, n_alim, n_blim;
    int c_row0, c_rows, c_n0, n_row0, n_rows, n_n0;
    int c_kt = K / BK, n_kt = K / BK;   // k-tiles per output tile: per tile in the weight-gradient form
    int c_split = 0, n_split = 0;       // part of the contraction
    int c_krows = 0, n_krows = 0;       // row-major form: rows of the tile's expert
    bool n_valid;
    {
        const PTile t = get_tile(0);
        if (!t.valid) return;
        c_a = t.a; c_b0 = t.b0; c_b1 = t.b1; c_alim = t.a_lim; c_blim = t.b_lim;
        c_row0 = t.row0; c_rows = t.rows; c_n0 = t.n0;
        if (GROUPK || SPLIT) c_kt = t.kt;
        if (SPLIT) c_split = t.split;
        if (KMAJ) c_krows = t.krows;
    }
    auto fetch_next_tile = [&](int i) {
        const PTile t = get_tile(i);
        n_a = t.a; n_b0 = t.b0; n_b1 = t.b1; n_alim = t.a_lim; n_blim = t.b_lim;
        n_row0 = t.row0; n_rows = t.rows; n_n0 = t.n0; n_valid = t.valid;
        if (GROUPK || SPLIT) n_kt = t.kt;
        if (SPLIT) n_split = t.split;
        if (KMAJ) n_krows = t.krows;
    };
    fetch_next_tile(1);

    // global side of the direct loads: thread (frow, fchunk) of a pass fetches
    // 16 bytes of tile row p*RPP + frow; the chunk it asks for is XOR-swizzled
    // so that the LDS side can stay linear (lane * 16 bytes)
    const int frow = tid / CPR, fchunk = tid % CPR;
    const uint32_t k2 = (uint32_t)K * 2u;
    const uint32_t vrow = (uint32_t)frow * k2;
    const uint32_t vswz = (uint32_t)((fchunk ^ lds_swizzle(frow)) * 16);   // every pass starts at a multiple of 16 rows
    const uint32_t step = (uint32_t)RPP * k2;
    const int wbase = (wave * 64 / CPR) * ROWB;

    // row-major form: a pass covers 16 rows of 512 bytes; thread = (row tid / 32, piece tid % 32); the piece it asks
    // for is XOR-swizzled by the row in units of 32 bytes: a 16-lane group of a transposing read touches 32 bytes
    // of four consecutive rows, which then lie in the four different quarters of the 128-byte bank window
    const int km_row = tid >> 5;
    const uint32_t km_piece = (uint32_t)(((tid & 31) ^ (2 * (km_row & 3))) * 16);
    const uint8_t* const zero_row = reinterpret_cast<const uint8_t*>(GU) + (tid & 31) * 16;
    auto fetch_km = [&](int p, const uint8_t* base, uint32_t ld2, uint32_t lim, int rows_left, uint8_t* st) {
        const int krow = 16 * p + km_row;
        const uint8_t* src = base + (uint32_t)krow * ld2 + min(km_piece, lim);
        if (krow >= rows_left) src = zero_row;   // past the expert's last row: contributes nothing
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(st + p * RPP * ROWB + wbase), 16,
                                         0, 0);
    };
    // Where the k-tile that a period fetches (kt + 2: the first two of the next tile in a tile's last two periods) lies: a
    // pointer per operand that moves on by a k-tile each period, and what a thread adds to it in each pass, the same for all
    // k-tiles of a tile: kept with four waves, formed for every load with eight, which have no registers left for it.
    constexpr bool KEEP = !KMAJ && NW == 4;
    const uint8_t *f_a, *f_b0, *f_b1;
    uint32_t off_a[KEEP ? PA : 1], off_b[KEEP ? PBD : 1];
    uint32_t f_alim = 0, f_blim = 0;
    int f_rows = 0;                                            // row-major form: valid rows from the k-tile's first row on
    const size_t kstep_a = KMAJ ? (size_t)64 * K * 2 : BK * 2;   // a k-tile is 64 elements along the rows, or 64 rows
    const size_t kstep_b = KMAJ ? (size_t)64 * ldb * 2 : BK * 2;
    auto pass_offset = [&](int p, uint32_t lim) {   // ragged tail: a valid row again
        uint32_t first = vrow;
        if (!KEEP) asm volatile("" : "+v"(first));   // hidden, or the rows' sums are kept across the whole loop
        return min(first + (uint32_t)p * step, lim) + vswz;
    };
    auto fetch_from = [&](const uint8_t* a, const uint8_t* b0, const uint8_t* b1, uint32_t alim, uint32_t blim, int krows) {
        f_a = a; f_b0 = b0; f_b1 = b1;
        if constexpr (KEEP) {
#pragma unroll
            for (int p = 0; p < PA; ++p) off_a[p] = pass_offset(p, alim);
#pragma unroll
            for (int p = 0; p < PBD; ++p) off_b[p] = pass_offset(p, blim);
        } else {
            f_alim = alim; f_blim = blim; f_rows = krows;
        }
    };
    auto fetch_step = [&]() {
        f_a += kstep_a;
        f_b0 += kstep_b;
        if (SWIGLU) f_b1 += kstep_b;
        if (KMAJ) f_rows -= 64;
    };
    auto fetch_a = [&](int p, uint8_t* st) {
        if constexpr (KMAJ)
            fetch_km(p, f_a, k2, f_alim, f_rows, st);
        else
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(f_a + (KEEP ? off_a[KEEP ? p : 0] : pass_offset(p, f_alim))),
                                             (__attribute__((address_space(3))) void*)(st + p * RPP * ROWB + wbase), 16, 0, 0);
    };
    auto fetch_b = [&](int p, uint8_t* st) {
        if constexpr (KMAJ)
            fetch_km(p, f_b0, (uint32_t)ldb * 2u, f_blim, f_rows, st);
        else
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((p >= PBD ? f_b1 : f_b0) + (KEEP ? off_b[KEEP ? p % PBD : 0] : pass_offset(p % PBD, f_blim))),
                                             (__attribute__((address_space(3))) void*)(st + p * RPP * ROWB + wbase), 16, 0, 0);
    };
    // load i of a period: i < PE -> pass i of the early operand's tile, else pass i - PE of the late operand's;
    // ld_b / ld_a: the weight / activation slot being filled
    auto fetch_one = [&](int i, uint8_t* ld_b, uint8_t* ld_a) {
        if constexpr (DEEP_B) {
            if (i < PA) fetch_a(i, ld_a);
            else fetch_b(i - PA, ld_b);
        } else {
            if (i < PB) fetch_b(i, ld_b);
            else fetch_a(i - PB, ld_a);
        }
    };

    const int fr = lane & 15, fk = lane >> 4;
    int a_off[FM], b_off[FN];   // row-major form: see km_off
    int km_off[4];
    const int f_sw = lds_swizzle(fr);  // fragments start at multiples of 16 rows
    if constexpr (KMAJ) {
        // lane (group g = lane / 16, s = lane % 16) addresses row 8 g + s / 4 (and, second load, the row four further) of a
        // k-step's 32, features 4 (s % 4) .. + 3 of the fragment's 16; its row decides the swizzle of the 64-byte unit.  The
        // swizzle moves a fragment inside its 128 bytes only: four offsets do for all fragments of both operands.
        const int sl = lane & 15;
        const int r8 = 8 * fk + (sl >> 2);
        const int piece_in = (sl & 3) >> 1;   // 16-byte piece inside the fragment's 32 bytes
#pragma unroll
        for (int i = 0; i < 4; ++i) km_off[i] = r8 * 512 + ((2 * i + piece_in) ^ (2 * (r8 & 3))) * 16 + 8 * (sl & 1);
    } else {
#pragma unroll
        for (int i = 0; i < FM; ++i) a_off[i] = (wm * WM + i * 16 + fr) * ROWB;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            int r;
            if (SWIGLU) {
                constexpr int half = FN / 2;
                r = (j < half) ? (wn * (WN / 2) + j * 16 + fr) : (BN / 2 + wn * (WN / 2) + (j - half) * 16 + fr);
            } else {
                r = wn * WN + j * 16 + fr;
            }
            b_off[j] = r * ROWB;
        }
    }

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

    bf16x8 af[2][FM], bfg[2][FN];
    auto set_of = [](int q, int buf) { return q < A_ONE ? 0 : buf; };
    // fragment q (the activations', then the weights') of k-step s (32 elements along the rows) into set buf
    auto read_one = [&](const uint8_t* sa, const uint8_t* sb, int s, int buf, int q) {
        if constexpr (KMAJ) {
            // k-step s = rows 32 s .. 32 s + 31: two transposing loads of four rows for a lane's eight values
            typedef __attribute__((ext_vector_type(4))) short s16x4;
            typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
            const int t = q < FM ? q : q - FM;   // 16 features each, 32 bytes
            const uint8_t* p = (q < FM ? sa + wm * (WM * 2) : sb + wn * (WN * 2)) + (t >> 2) * 128 + s * (32 * 512) + km_off[t & 3];
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * 512));
            typedef __attribute__((ext_vector_type(8))) short s16x8;
            const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            if (q < FM)
                af[set_of(q, buf)][q] = __builtin_bit_cast(bf16x8, v);
            else
                bfg[buf][q - FM] = __builtin_bit_cast(bf16x8, v);
            return;
        }
        const int c = ((4 * s + fk) ^ f_sw) << 4;
        if (q < FM)
            af[set_of(q, buf)][q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sa + a_off[q] + c));
        else
            bfg[buf][q - FM] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sb + b_off[q - FM] + c));
    };
    auto mfma_one = [&](int buf, int m) {
        // boustrophedon over the wave's blocks: successive MFMAs share one operand fragment
        const int i = m / FN, j = (i & 1) ? FN - 1 - m % FN : m % FN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfg[buf][j], af[set_of(i, buf)][i], acc[i][j], 0, 0, 0);
    };
    // the order in which fragments with two sets of registers are read: the first a k-step needs first
    auto two_sets = [](int r) {
        if (A_ONE == 0) return r == 0 ? 0 : r <= FN ? FM + r - 1 : r - FN;
        return r < FN ? FM + r : A_ONE + r - FN;
    };
    // one k-step in issue order: NSLOT slots of {one matrix instruction on set mf_buf; at most a fragment read or two of k-step
    // rd_s into the other set; at most one direct load}
    auto kstep = [&](int mf_buf, const uint8_t* rd_a, const uint8_t* rd_b, int rd_s, int ld_begin, int ld_end, uint8_t* ld_b,
                     uint8_t* ld_a) {
        int ld = ld_begin;
#pragma unroll
        for (int slot = 0; slot < NSLOT; ++slot) {
            mfma_one(mf_buf, slot);
            // the k-step's first MFMA waits (lgkmcnt) for the fragments read during the previous k-step; keep
            // this k-step's reads behind it, or the compiler hoists them and that wait also covers reads issued
            // a moment ago (a full LDS round trip in front of every k-step)
            if (slot == 0) __builtin_amdgcn_sched_barrier(0);
            constexpr int RS = NSLOT * 7 / 8;   // the barrier behind k-step 0 waits for the last of them
#pragma unroll
            for (int r = (slot * NTWO + RS - 1) / RS; r < ((slot + 1) * NTWO + RS - 1) / RS && r < NTWO; ++r)
                read_one(rd_a, rd_b, rd_s, mf_buf ^ 1, two_sets(r));
            if (A_ONE > 0 && slot % FN == FN - 1 && slot / FN < A_ONE) read_one(rd_a, rd_b, rd_s, mf_buf ^ 1, slot / FN);
            if (ld < ld_end && slot == 1 + (ld - ld_begin) * NSLOT / (ld_end - ld_begin)) {
                fetch_one(ld, ld_b, ld_a);
                ++ld;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    uint8_t* const a_region = smem;
    uint8_t* const b_region = smem + B_REGION;

    // prologue (first tile of this workgroup only): late(0), early(0), then late(1); only the first two must have
    // landed before the first fragment reads
    {
        fetch_from(c_a, c_b0, c_b1, c_alim, c_blim, c_krows);
#pragma unroll
        for (int i = PE; i < NLOAD; ++i) fetch_one(i, b_region, a_region);
#pragma unroll
        for (int i = 0; i < PE; ++i) fetch_one(i, b_region, a_region);
        fetch_step();
#pragma unroll
        for (int i = PE; i < NLOAD; ++i) fetch_one(i, b_region + (DEEP_B ? B_BYTES : 0), a_region + (DEEP_B ? 0 : A_BYTES));
        __builtin_amdgcn_s_waitcnt(0x0F70 | (PL & 0xF) | ((PL >> 4) << 14));  // vmcnt(PL)
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int q = 0; q < NREAD; ++q) read_one(a_region, b_region, 0, 0, q);
        // early(1) into the early operand's slot 1
#pragma unroll
        for (int i = 0; i < PE; ++i) fetch_one(i, b_region + B_BYTES, a_region + A_BYTES);
    }

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
    // the source of the loads of period kt: k-tile kt + 2 of the stream that starts at the current tile's first.  Every tile has
    // at least two k-tiles, so that is one of this tile's or of the next one's first two; behind the last tile the last two
    // k-tiles are fetched again, and never used.
    auto advance = [&](int kt) {
        fetch_step();
        if (kt == c_kt - 2) {
            if (n_valid)
                fetch_from(n_a, n_b0, n_b1, n_alim, n_blim, n_krows);
            else {
                f_a -= 2 * kstep_a;
                f_b0 -= 2 * kstep_b;
                if (SWIGLU) f_b1 -= 2 * kstep_b;
                if (KMAJ) f_rows += 128;
            }
        }
    };
    int stored = 0;   // the epilogue of a tile has just been through
    for (;;) {
        // (IDLE_SKIP instantiations, chosen for launches with many experts, i.e. many ragged tails.)  A wave whose rows of the
        // tile all lie past the tile's last valid row (ragged tail of an expert) has nothing to multiply: it keeps issuing its
        // share of the loads and meeting the barriers, and leaves the matrix pipe and the LDS reads alone (under a power cap
        // that is clock for the other workgroups).  The last k-tile it multiplies like the others, whatever its registers
        // hold: that leaves the next tile's first fragments in the registers where the loop expects them, and the sums are
        // not stored.
        int kt = 0;
        if (IDLE_SKIP) {
            for (const int idle = wm * WM >= c_rows ? c_kt - 1 : 0; kt < idle; ++kt) {   // wave-uniform
                advance(kt);
                uint8_t* lb = b_region + (DEEP_B ? b2 : b1);
                uint8_t* la = a_region + (DEEP_B ? a1 : a2);
#pragma unroll
                for (int i = PE; i < NLOAD; ++i) fetch_one(i, lb, la);
                wait_memory<PL, NSTORE>(stored);
                __builtin_amdgcn_s_barrier();
#pragma unroll
                for (int i = 0; i < PE; ++i) fetch_one(i, b_region + b0, a_region + a0);
                rotate();
            }
        }
        for (; kt < c_kt; ++kt) {
            advance(kt);
            const uint8_t* ca = a_region + a0;
            const uint8_t* cb = b_region + b0;
            // this period fills late(kt+2) and, once k-tile kt is read, early(kt+2)
            uint8_t* lb = b_region + (DEEP_B ? b2 : b1);
            uint8_t* la = a_region + (DEEP_B ? a1 : a2);
            __builtin_amdgcn_sched_barrier(0);
            kstep(0, ca, cb, 1, PE, NLOAD, lb, la);  // k-step 0
            // early(kt+1) and late(kt+1) were issued a period ago, late(kt+2) in this one: all but the PL youngest
            // loads must have landed; this wave's fragment reads of k-tile kt are in registers
            wait_memory<PL, NSTORE>(stored);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // k-step 1: first fragments of k-tile kt+1; the early operand's slot of k-tile
            // kt is free, early(kt+2) goes into it
            kstep(1, a_region + a1, b_region + b1, 0, 0, PE, b_region + b0, a_region + a0);
            rotate();
        }
        // Epilogue.  The late operand's slot that held the last k-tile (now its third) is
        // idle: every wave finished reading it before the last barrier, and the
        // next loads into it are issued only after the barrier below.
        if constexpr (SPLIT)
            store_partial<FM, FN, WM, WN, SWIGLU>(acc, c_row0, c_rows, c_n0,
                                                  reinterpret_cast<float*>(C) + (size_t)c_split * plane_rows * (SWIGLU ? 2 * N : N), N, wm,
                                                  wn, lane);
        else
            store_tile_staged<FM, FN, WM, MODE, (FM * FN * 4 > 128), STREAM_OUT>(
                acc, c_row0, c_rows, c_n0, C, GU, N, wm, wn, lane,
                (DEEP_B ? b_region + b2 : a_region + a2) + wave * (32 * FO * 32));
        if (!n_valid) break;
        c_a = n_a; c_b0 = n_b0; c_b1 = n_b1; c_alim = n_alim; c_blim = n_blim;
        c_row0 = n_row0; c_rows = n_rows; c_n0 = n_n0;
        if (GROUPK || SPLIT) c_kt = n_kt;
        if (SPLIT) c_split = n_split;
        if (KMAJ) c_krows = n_krows;
        ++ti;
        stored = 1;
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
    if (sample && tid == 0) {
        ticks[0] = __builtin_amdgcn_s_memtime() - tk_entry;
        ticks[1] = __builtin_amdgcn_s_memrealtime() - rt_entry;
    }
}

// BM = 0: the height of the tiles is chosen on the device, from the rows that every expert really has (pick_height);
// 256, 192 or 128 rows, all of BN = 256 columns (ldb: a height to be taken instead, or 0).  A row's sums are formed in the same order whatever the height.
template <int BM, int BN, int WGM, int WGN, int MODE, bool GROUPK = false, bool KMAJ = false, bool IDLE_SKIP = false,
          bool DEEP_B = false, bool BY_ROUND = true, bool STREAM_OUT = false, bool SPLIT = false>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_bf16_persist_kernel(
    const bf16_t* __restrict__ A, const int32_t* __restrict__ offsets, int E, int N, int K,
    const bf16_t* __restrict__ B0, const bf16_t* __restrict__ B1, bf16_t* __restrict__ C, bf16_t* __restrict__ GU,
    int ntn, int ldb, int splits, int plane_rows, unsigned long long* __restrict__ ticks) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    if constexpr (BM != 0) {
        persist_body<BM, BN, WGM, WGN, MODE, GROUPK, KMAJ, IDLE_SKIP, DEEP_B, BY_ROUND, STREAM_OUT, SPLIT>(
            A, offsets, E, N, K, B0, B1, C, GU, ntn, ldb, splits, plane_rows, ticks, smem);
    } else {
        const int height = ldb != 0 ? ldb : pick_height(kCostBf16, offsets, E, ntn * (SPLIT ? splits : 1), K / 64 / (SPLIT ? splits : 1),
                                                        threadIdx.x & 63);
        auto run = [&](auto rows) {
            persist_body<decltype(rows)::value, BN, WGM, WGN, MODE, false, false, IDLE_SKIP, DEEP_B, BY_ROUND, false, SPLIT>(
                A, offsets, E, N, K, B0, B1, C, GU, ntn, ldb, splits, plane_rows, ticks, smem);
        };
        if (height == 256) run(std::integral_constant<int, 256>{});
        else if (height == 192) run(std::integral_constant<int, 192>{});
        else run(std::integral_constant<int, 128>{});
    }
}

template <int BM, int BN, int WGM, int WGN, int MODE, bool DEEP_B = false>
void launch_persist(const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0,
                    const void* B1, void* C, void* GU, hipStream_t s) {
    constexpr int OUTN = (MODE == 1 || MODE == 2) ? BN / 2 : BN;
    constexpr int HMAX = BM != 0 ? BM : 256, HMIN = BM != 0 ? BM : 128;   // tallest and lowest tile
    constexpr size_t smem = (size_t)(DEEP_B ? 2 * HMAX + 3 * BN : 3 * HMAX + 2 * BN) * 64 * 2;
    if constexpr (BM == 0 && MODE != 3 && WGM * WGN == 4) {
        // Many rows on many experts: 256 rows are mostly the best height, and the kernel that holds it alone has no choice to make.
        // r_max is a bound, not the rows there are, and a launch of a few rounds can be better off lower.  (The height chosen, of the
        // time so, 660 to 3500 rows per expert: 7 layers of 32 to 128 experts, gate/up 1.003 to 1.010, down 0.984 to 1.003; 16 and 24
        // experts 0.978 to 1.017 and 0.970 to 1.006, between 0.86 and 1.09: 16 x 660 rows, 2048 x 1408, gate/up 126 us so and 113 with
        // the height chosen, 16 x 1024, 1024 x 4096, down 154 and 137; 24 x 800, 2048 x 1024, gate/up 132 and 143.)
        if (g_persist_tile_rows == 0 && E >= 16 && r_max >= 640ll * E) {
            launch_persist<256, BN, WGM, WGN, MODE, DEEP_B>(A, offsets, r_max, E, N, K, B0, B1, C, GU, s);
            return;
        }
    }
    const int ntn = (N + OUTN - 1) / OUTN;
    // many experts = many ragged tail tiles: the instantiation whose idle waves skip the multiplication.  (With the skip, of the time
    // without: 11 layers of 16 to 128 experts, 660 to 3500 rows, gate/up 0.978, down 0.989, saved gate/up 0.994; 8 layers of 1 to 12, 150 to
    // 3333 rows, 0.995, 0.990 and 1.000, gate/up slower by 2 to 7 % in a tenth of them.)
    const bool idle_skip = MODE != 3 && persist_idle_skip(E);
    constexpr bool SKIP = MODE != 3;
    // Whole rounds of tiles are dealt to the XCDs round by round, but for many experts of few rows: contiguous shares.  (Both products of a
    // layer by rounds, of the time by shares: 8 layers of 1 to 12 experts, 200 to 2048 rows, 0.996; 11 layers of 16 to 128 experts, 800 and 1280
    // rows, 0.993 and 0.997, with the pre-activations saved 0.984 and 0.991; with 200 rows 0.993, between 0.962 and 1.027; the
    // training step of 64 experts x 172 rows, 6144 x 2048, takes 5882 us by shares and 5922 by rounds, dx 675 and 715 of them.)
    constexpr bool SHARES = BM == 0 && MODE != 3;
    const bool by_round = !SHARES || E < 16;
    auto pick = [&](auto skip, auto round) {
        constexpr bool S = decltype(skip)::value, R = decltype(round)::value;
        return gemm_bf16_persist_kernel<BM, BN, WGM, WGN, MODE, false, false, S, DEEP_B, R>;
    };
    using Yes = std::true_type;
    using No = std::false_type;
    using Skip = std::integral_constant<bool, SKIP>;
    using Shares = std::integral_constant<bool, !SHARES>;
    auto kern = idle_skip ? (by_round ? pick(Skip{}, Yes{}) : pick(Skip{}, Shares{})) : (by_round ? pick(No{}, Yes{}) : pick(No{}, Shares{}));
    static OncePerDevice lds[2][2];
    allow_lds(lds[idle_skip][by_round], reinterpret_cast<const void*>(kern), (int)smem);
    // never more workgroups than the static bound on the tile count
    const int grid = min(persist_grid(), grid_for(r_max, E, HMIN, ntn));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WGM * WGN * 64), smem, s, static_cast<const bf16_t*>(A), offsets, E, N,
                       K, static_cast<const bf16_t*>(B0), static_cast<const bf16_t*>(B1), static_cast<bf16_t*>(C),
                       static_cast<bf16_t*>(GU), ntn, g_persist_tile_rows, 1, 0, g_persist_ticks);
}

// dw[e] = 0 for every expert without rows (the persistent weight-gradient kernel gives them no tiles)
__global__ __launch_bounds__(256) void wgrad_zero_empty_kernel(const int32_t* __restrict__ offsets, size_t per_expert,
                                                               bf16_t* __restrict__ dw0, bf16_t* __restrict__ dw1,
                                                               bf16_t* __restrict__ dw2) {
    const int e = blockIdx.y;
    if (offsets[e + 1] - offsets[e] > 0) return;
    bf16_t* const dw = blockIdx.z == 0 ? dw0 : blockIdx.z == 1 ? dw1 : dw2;
    u32x4* dst = reinterpret_cast<u32x4*>(dw + (size_t)e * per_expert);   // per_expert is a multiple of 8
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < per_expert / 8; i += (size_t)gridDim.x * 256)
        dst[i] = u32x4{0u, 0u, 0u, 0u};
}

template <int BM, int BN, int WGM, int WGN, bool STREAM_OUT, bool DEEP_B = false>
void launch_persist_groupk(const void* A, const void* B, const int32_t* offsets, int E, int M, int N, int ld,
                           void* C, hipStream_t s) {
    constexpr size_t smem = (size_t)(DEEP_B ? 2 * BM + 3 * BN : 3 * BM + 2 * BN) * 64 * 2;
    auto kern = gemm_bf16_persist_kernel<BM, BN, WGM, WGN, 0, true, false, false, DEEP_B, true, STREAM_OUT>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), (int)smem);
    const long long tiles = (long long)E * ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    const int grid = (int)min((long long)persist_grid(), (tiles + 7) / 8 * 8);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WGM * WGN * 64), smem, s, static_cast<const bf16_t*>(A), offsets, E, N,
                       ld, static_cast<const bf16_t*>(B), static_cast<const bf16_t*>(B), static_cast<bf16_t*>(C),
                       static_cast<bf16_t*>(nullptr), M, 0, 1, 0, g_persist_ticks);
}

// weight gradients straight from the row-major activations (no transposed copies): see the kernel's KMAJ form
template <int BM, int BN, int WGM, int WGN>
void launch_persist_groupk_rowmajor(const void* A, int lda, const void* B, int ldb, const int32_t* offsets, int E,
                                    int M, int N, const void* zero_row, void* C, hipStream_t s) {
    constexpr size_t smem = (size_t)(3 * BM + 2 * BN) * 64 * 2;
    auto kern = gemm_bf16_persist_kernel<BM, BN, WGM, WGN, 0, true, true>;
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(kern), (int)smem);
    const long long tiles = (long long)E * ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    const int grid = (int)min((long long)persist_grid(), (tiles + 7) / 8 * 8);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WGM * WGN * 64), smem, s, static_cast<const bf16_t*>(A), offsets, E, N,
                       lda, static_cast<const bf16_t*>(B), static_cast<const bf16_t*>(B), static_cast<bf16_t*>(C),
                       static_cast<bf16_t*>(const_cast<void*>(zero_row)), M, ldb, 1, 0, g_persist_ticks);
}

// Four waves or eight, the tile's height chosen on the device.  Four are ahead where power is what bounds a product.  With few rows
// and a short contraction a tile is a few k-tiles of which memory is waited for, and two waves to a SIMD cover more of that, of the
// epilogue and of the tails that leave waves idle.  The line: rows per expert x contraction.  (Down, us, four / eight: K = 384, 40 experts, N =
// 3968, 140, 300 and 500 rows 39.3, 60.9 and 92.8 / 36.3, 57.0 and 88.5; 640, 32, 2688, 140, 300 and 400 32.6, 44.9 and 51.9 / 30.6, 42.4 and
// 52.7; 896, 32, 1664, 140, 220 and 400 26.3, 30.9 and 45.1 / 25.9, 29.9 and 46.9; 1024, 60, 2688, 140 and 220 86.5 and 111 / 86.9 and
// 114; 1280, 24, 1536, 140 and 260 24.4 and 31.9 / 23.5 and 32.4; 2048, 48, 2048, 40, 110 and 200 106, 109 and 126 / 103, 109 and
// 129.  Gate/up, K = 2048, 48 experts x 40 rows, N = 2048, 187 / 181; 3584, 24 x 200, 896, 88.5 / 93.0.  Longer contractions are level, or
// behind: dx, K = 4096, 64 x 64 rows, N = 6144, 577 / 594.)
// The gate/up product that saves its pre-activations stores three times as much, and eight waves stay ahead for twice the rows (96 x 200
// rows, 1280 x 1792, 292 / 275; 48 x 152 and x 400, 2048 x 2048, 211 and 347 / 204 and 338; 60 x 154, 1664 x 1920, 218 / 208).
template <int MODE>
void launch_persist_chosen(const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0, const void* B1,
                           void* C, void* GU, hipStream_t s) {
    if constexpr (MODE != 3) {
        if (K <= 2048 && (long long)r_max * K <= (MODE == 2 ? 440000ll : 220000ll) * E) {
            launch_persist<0, 256, 2, 4, MODE, true>(A, offsets, r_max, E, N, K, B0, B1, C, GU, s);
            return;
        }
    }
    launch_persist<0, 256, 2, 2, MODE, true>(A, offsets, r_max, E, N, K, B0, B1, C, GU, s);
}

template <int BM, int BN, int WGM, int WGN, bool DEEP_B = false>
void run_persist_pair(const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E,
                      const void* w_gate, const void* w_up, const void* w_down, void* h, void* y_perm, int phase,
                      hipStream_t s) {
    if (phase & 1) launch_persist<BM, BN, WGM, WGN, 1, DEEP_B>(x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, nullptr, s);
    if (phase & 2) launch_persist<BM, BN, WGM, WGN, 0, DEEP_B>(h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, nullptr, s);
}

}  // namespace

void set_persist_workgroups(int n) { g_persist_workgroups = n; }
void set_persist_idle_skip(int v) { g_persist_idle_skip = v; }
void set_persist_tile_rows(int v) { g_persist_tile_rows = v; }
int persist_tile_rows() { return g_persist_tile_rows; }
void set_persist_clock_sample(unsigned long long* ticks) { g_persist_ticks = ticks; }
unsigned long long* persist_clock_sample() { return g_persist_ticks; }
bool persist_idle_skip(int E) { return g_persist_idle_skip < 0 ? E >= 16 : g_persist_idle_skip != 0; }

// C [rows, N] = A [rows, K] . B[e]^T with B [E, N, K], rows grouped by expert (bf16): the
// down-projection form of the persistent kernel, for any operands of that shape
bool launch_grouped_nt(const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B,
                       void* C, hipStream_t s) {
    if (K < 128 || K % 64 || N % 8) return false;
    const StreamPlan plan = plan_stream(kStreamBf16, r_max, E, N, K, false, true, 0);
    if (plan.kind != kPlanLarge) {
        launch_stream(plan, kStreamBf16, A, offsets, r_max, E, N, K, B, nullptr, C, nullptr, 0.f, 0.f, 0.f, nullptr, nullptr, s);
        return true;
    }
    launch_persist_chosen<0>(A, offsets, r_max, E, N, K, B, nullptr, C, nullptr, s);
    return true;
}

// One launch for the three gradients of a layer: a launch that finds nothing to do still takes 4.8 us.
void launch_wgrad_zero_empty(const int32_t* offsets, int E, size_t per_expert, void* dw0, void* dw1, void* dw2,
                             hipStream_t s) {
    hipLaunchKernelGGL(wgrad_zero_empty_kernel, dim3(64, E, 3), dim3(256), 0, s, offsets, per_expert,
                       static_cast<bf16_t*>(dw0), static_cast<bf16_t*>(dw1), static_cast<bf16_t*>(dw2));
}

// dw [E, M, N] = per expert a_t[:, seg_e] . b_t[:, seg_e]^T (see WgradSched); M, N multiples of 8, ld of 64
void launch_persist_wgrad(const void* a_t, const void* b_t, const int32_t* offsets, int E, int M, int N, int ld,
                          void* dw, hipStream_t s) {
    const long long per_expert = (long long)((M + 255) / 256) * ((N + 255) / 256), tiles = E * per_expert;
    // Up to some 97 rows per expert (the padding included, a tile is then two k-tiles and its store): four waves wait between the two,
    // eight of 64 x 64 cover it.  Tiles of 128 rows, the 256 columns in three stages, streamed.  The backward, us, four waves of 256 rows / so:
    // 4 experts x 60 rows, 2048 x 2048, 114 / 100; 24 x 60, 2048 x 512, 139 / 126; 32 x 40, 2048 x 2048, 468 / 426; 60 x 40, 1664 x 1920, 639 / 585;
    // 40 x 60, 3072 x 1792, 670 / 640; 16 x 60, 6144 x 2048, 580 / 576; 64 x 100, 2560 x 1536, level.  On the other side of the lines: 128 experts
    // x 60 rows, 2048 x 768, 698 / 722; 96 x 59, 2048 x 1024, 694 / 717; 64 x 60, 2816 x 2048, 1054 / 1080; 32 x 43, 4096 x 2048, 759 / 797; 4 x 60, 4096 x 4096, 257 / 261; 48 x 122, 4096 x
    // 1024, 710 / 742 (8 to 16 experts gain up to 160 rows, 2 to 9 %).  The tiles' operands, one and a half times as many, are what costs.
    if (ld <= 224ll * E && E <= 64 && per_expert < 256 && (long long)E * M * N < 1ll << 28 && N <= kMaxColumns) {
        launch_persist_groupk<128, 256, 2, 4, true, true>(a_t, b_t, offsets, E, M, N, ld, dw, s);
        return;
    }
    // Tiles of 128 rows where those of 256 are at most one to every second workgroup: a compute unit has one tile then, as long
    // as its k-tiles are one after the other, and with four waves nothing covers what they wait for.  One gradient, us, 256 rows /
    // 128 (streamed too, at any number of rows): 4 experts x 53 rows, 1024 x 1024, 9.8 / 8.4 not streamed; 4 x 60, 4 x 250 and
    // 4 x 600, 1024 x 1792, 15.1, 21.4 and 36.6 / 8.0, 10.3 and 16.1; 8 x 60, 500 and 2000, 1024 x 1024 (128 tiles of 256)
    // 10.4, 18.3 and 53.0 / 8.3, 15.6 and 41.6, not streamed 10.1, 18.9 and 42.1.
    if (2 * tiles <= persist_grid() && N <= kMaxColumns) {
        launch_persist_groupk<128, 256, 2, 2, true, true>(a_t, b_t, offsets, E, M, N, ld, dw, s);
        return;
    }
    // Streamed past the L2 whatever the rows (the expert FFN's backward streamed, of what it takes stored as usual; 19 layers of 1 to 128
    // experts: 200 rows per expert 0.83 to 0.94, 450 rows 0.86 to 1.02, 800 rows 0.93 to 1.02, 1280 rows 0.95 to 1.01, 2048 rows 0.98 to
    // 0.99; the two above 1 are 8 experts, 6144 x 16384, 1.6 and 2.1 % at 450 and 800 rows, which at 2048 take 0.7 % less).
    if (N <= kMaxColumns)
        launch_persist_groupk<256, 256, 2, 2, true>(a_t, b_t, offsets, E, M, N, ld, dw, s);
    else
        launch_persist_groupk<256, 256, 2, 2, false>(a_t, b_t, offsets, E, M, N, ld, dw, s);
}

// dw [E, M, N] = per expert A[rows_e, 0:M]^T . B[rows_e, 0:N], A [rows, lda] and B [rows, ldb] row-major; M, N
// multiples of 8 and lda, ldb multiples of 8; zero_row: 512 bytes of zeros
void launch_persist_wgrad_rowmajor(const void* a, int lda, const void* b, int ldb, const int32_t* offsets, int E,
                                   int M, int N, const void* zero_row, void* dw, hipStream_t s) {
    launch_persist_groupk_rowmajor<256, 256, 2, 4>(a, lda, b, ldb, offsets, E, M, N, zero_row, dw, s);
}

// dg | du [rows, 2N] from dh = A . B[e]^T (never stored) and the saved pre-activations gu [rows, 2N]
bool launch_grouped_nt_swiglu_bwd(const void* A, const int32_t* offsets, int r_max, int E, int N, int K,
                                  const void* B, const void* gu, void* dgdu, hipStream_t s) {
    if (K < 128 || K % 64 || N % 8) return false;
    launch_persist_chosen<3>(A, offsets, r_max, E, N, K, B, nullptr, dgdu, const_cast<void*>(gu), s);
    return true;
}

// h = silu(x W_gate^T) * (x W_up^T) as in the forward, and the two pre-activations to gu [rows, 2F]
bool launch_gate_up_saving(const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E,
                           const void* w_gate, const void* w_up, void* h, void* gu, hipStream_t s) {
    if (H < 128 || H % 64 || F % 8) return false;
    const StreamPlan plan = plan_stream(kStreamBf16, r_max, E, F, H, true, true, 0);   // the same choice as the plain forward's
    if (plan.kind != kPlanLarge) {
        launch_stream(plan, kStreamBf16, x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, gu, 0.f, 0.f, 0.f, nullptr, nullptr, s);
        return true;
    }
    launch_persist_chosen<2>(x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, gu, s);
    return true;
}

// One product with its contraction in `splits` parts, fp32 planes [splits][r_max][N, or 2 N with w_up] in part
bool launch_persist_split(const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0, const void* B1,
                          float* part, int splits, hipStream_t s) {
    if (K % 64 || N % 8 || K / 64 < 2 * splits) return false;
    auto go = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value, OUTN = MODE == 1 ? 128 : 256;
        constexpr size_t smem = (size_t)(2 * 256 + 3 * 256) * 64 * 2;
        auto kern = gemm_bf16_persist_kernel<0, 256, 2, 2, MODE, false, false, false, true, true, false, true>;
        static OncePerDevice lds;
        allow_lds(lds, reinterpret_cast<const void*>(kern), (int)smem);
        const int ntn = (N + OUTN - 1) / OUTN;
        const int grid = min(persist_grid(), grid_for(r_max, E, 128, ntn * splits));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), smem, s, static_cast<const bf16_t*>(A), offsets, E, N, K,
                           static_cast<const bf16_t*>(B0), static_cast<const bf16_t*>(B1), reinterpret_cast<bf16_t*>(part),
                           static_cast<bf16_t*>(nullptr), ntn, g_persist_tile_rows, splits, r_max, g_persist_ticks);
    };
    if (B1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 0>{});
    return true;
}

bool launch_persist_ffn(const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E,
                        const void* w_gate, const void* w_up, const void* w_down, void* h, void* y_perm,
                        int variant, int phase, hipStream_t s) {
    if (H < 128 || F < 128) return false;  // the k stream needs at least two k-tiles per output tile
    switch (variant) {
        case 0:
            if (phase & 1) launch_persist_chosen<1>(x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, nullptr, s);
            if (phase & 2) launch_persist_chosen<0>(h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, nullptr, s);
            return true;
        case 40: run_persist_pair<256, 256, 2, 2>(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, phase, s); return true;
        case 41: run_persist_pair<256, 256, 2, 4>(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, phase, s); return true;
        case 42: run_persist_pair<0, 256, 2, 2, true>(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, phase, s); return true;
        case 43: run_persist_pair<0, 256, 2, 4, true>(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, phase, s); return true;
        default: return false;
    }
}

}  // namespace moe
