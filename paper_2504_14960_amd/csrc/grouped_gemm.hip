// a3. Grouped SwiGLU expert FFN (Section 3.1.2 "Expert Computation"; f_e of
// Eq. 1): for every expert e, over its contiguous rows,
//     h = silu(X_e W_gate,e^T) * (X_e W_up,e^T),   Y_e = h W_down,e^T.
//
// Both products are "NT" GEMMs (activations [rows, K] and weights [N, K] are
// both contiguous along the contraction index), which is exactly the operand
// order the gfx950 bf16 MFMA wants: each lane feeds 8 consecutive-K values.
//
// This file holds the dispatch and a plain FMA kernel.  The MFMA kernels live in
// gemm_persist.hip (one persistent workgroup per compute unit walking a
// device-side tile list), gemm_stream.hip (few rows per expert, fp32 layers, odd
// shapes) and gemm_pipe3.hip (one workgroup per tile; taken when the contraction
// is too shallow for the persistent kernel's k stream).  For the first GEMM a weight
// tile holds 128 gate rows and the 128 matching up rows and every wave owns the
// same feature range of both, so silu(g)*u happens in registers and only h is
// written.
//
// Ragged scheduling: the per-expert row offsets live in device memory; the
// kernels derive the real tile list from them, no host round trip.
#include "gemm_stream.h"
#include "gemm_tile.h"

namespace moe {

namespace {

// ---------------------------------------------------------------------------
// Plain tiled kernel: "gemm_variant" 99, and rows too long for the others' 32-bit offsets.  64x64 outputs per workgroup, 16-wide K
// slices in LDS, 4x4 outputs per thread, fp32 FMA.  Every access is guarded.
template <typename TIn, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_simple_kernel(
    const TIn* __restrict__ A, const int32_t* __restrict__ offsets, int E, int N, int K,
    const TIn* __restrict__ B0, const TIn* __restrict__ B1, TIn* __restrict__ C, int ntn) {
    constexpr int BM = 64, BN = 64, BK = 16;
    __shared__ float As[BK][BM + 4];
    __shared__ float Bs[SWIGLU ? 2 : 1][BK][BN + 4];
    __shared__ int sched[kMaxExperts + 2];
    const Tile tile = find_tile<BM>(offsets, E, ntn, sched);
    if (!tile.valid) return;
    const int tid = threadIdx.x;
    const int tx = tid % 16, ty = tid / 16;
    const int n0 = tile.ntile * BN;
    auto ldv = [](const TIn* p) -> float {
        if constexpr (sizeof(TIn) == 2) return bf16_to_f32(*reinterpret_cast<const bf16_t*>(p));
        else return *reinterpret_cast<const float*>(p);
    };
    float acc[SWIGLU ? 2 : 1][4][4];
#pragma unroll
    for (int z = 0; z < (SWIGLU ? 2 : 1); ++z)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[z][i][j] = 0.f;

    for (int k0 = 0; k0 < K; k0 += BK) {
        for (int i = tid; i < BM * BK; i += 256) {
            const int r = i / BK, k = i % BK;
            float v = 0.f;
            if (r < tile.rows && k0 + k < K) v = ldv(A + (size_t)(tile.row0 + r) * K + k0 + k);
            As[k][r] = v;
        }
        for (int i = tid; i < BN * BK; i += 256) {
            const int r = i / BK, k = i % BK;
            float v0 = 0.f, v1 = 0.f;
            if (n0 + r < N && k0 + k < K) {
                const size_t at = ((size_t)tile.expert * N + n0 + r) * K + k0 + k;
                v0 = ldv(B0 + at);
                if (SWIGLU) v1 = ldv(B1 + at);
            }
            Bs[0][k][r] = v0;
            if (SWIGLU) Bs[SWIGLU ? 1 : 0][k][r] = v1;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < BK; ++k) {
            float a[4], b[SWIGLU ? 2 : 1][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
            for (int z = 0; z < (SWIGLU ? 2 : 1); ++z)
#pragma unroll
                for (int j = 0; j < 4; ++j) b[z][j] = Bs[z][k][tx * 4 + j];
#pragma unroll
            for (int z = 0; z < (SWIGLU ? 2 : 1); ++z)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[z][i][j] = fmaf(a[i], b[z][j], acc[z][i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = ty * 4 + i;
        if (r >= tile.rows) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + tx * 4 + j;
            if (col >= N) continue;
            float v;
            if (SWIGLU) {
                const float g = acc[0][i][j];
                v = (g / (1.f + expf(-g))) * acc[SWIGLU ? 1 : 0][i][j];
            } else {
                v = acc[0][i][j];
            }
            TIn* dst = C + (size_t)(tile.row0 + r) * N + col;
            if constexpr (sizeof(TIn) == 2) *reinterpret_cast<bf16_t*>(dst) = f32_to_bf16(v);
            else *reinterpret_cast<float*>(dst) = v;
        }
    }
}

template <typename TIn, bool SWIGLU>
void launch_simple_gemm(const void* A, const int32_t* offsets, int r_max, int E, int N, int K,
                        const void* B0, const void* B1, void* C, hipStream_t s) {
    const int ntn = (N + 63) / 64;
    const int grid = grid_for(r_max, E, 64, ntn);
    hipLaunchKernelGGL((gemm_simple_kernel<TIn, SWIGLU>), dim3(grid), dim3(256), 0, s,
                       static_cast<const TIn*>(A), offsets, E, N, K, static_cast<const TIn*>(B0),
                       static_cast<const TIn*>(B1), static_cast<TIn*>(C), ntn);
}

}  // namespace

// whether the MFMA kernels with large tiles take the layer
static bool large_covers(moe_dtype_t dt, int H, int F) { return dt == MOE_BF16 && H % 64 == 0 && F % 64 == 0; }

size_t expert_ffn_part_bytes(int r_max, int H, int F, int E, moe_dtype_t dt) {
    if (dt == MOE_F32) return 0;
    const bool large = large_covers(dt, H, F);
    const size_t a = stream_part_bytes(kStreamBf16, r_max, E, F, H, true, large);
    const size_t b = stream_part_bytes(kStreamBf16, r_max, E, H, F, false, large);
    return a > b ? a : b;
}

// One of the two products (ph 1: gate/up, 2: down) by its plan
static bool launch_phase(const StreamPlan& plan, int ph, int elt, const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E,
                         const void* w_gate, const void* w_up, const void* w_down, void* h, void* y_perm, void* part, hipStream_t s) {
    const int N = ph == 1 ? F : H, K = ph == 1 ? H : F;
    const void* const A = ph == 1 ? x_perm : h;
    const void* const B0 = ph == 1 ? w_gate : w_down;
    const void* const B1 = ph == 1 ? w_up : nullptr;
    void* const C = ph == 1 ? h : y_perm;
    if (plan.kind != kPlanLarge) {
        launch_stream(plan, elt, A, offsets, r_max, E, N, K, B0, B1, C, nullptr, 0.f, 0.f, 0.f, nullptr, static_cast<float*>(part), s);
        return true;
    }
    if (plan.splits > 1 && launch_persist_split(A, offsets, r_max, E, N, K, B0, B1, static_cast<float*>(part), plan.splits, s)) {
        launch_stream_reduce(ph == 1, static_cast<float*>(part), offsets, E, plan.splits, r_max, N, C, s);
        return true;
    }
    return launch_persist_ffn(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, 0, ph, s) ||
           launch_pipe3_ffn(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, ph == 1 ? 31 : 30, ph, s);
}

bool launch_expert_ffn(const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E,
                       const void* w_gate, const void* w_up, const void* w_down, moe_dtype_t dt,
                       void* h, void* y_perm, int variant, int phase, void* part, size_t part_bytes, hipStream_t s) {
    const bool f32 = dt == MOE_F32;
    const bool large = large_covers(dt, H, F);
    const int elt = f32 ? kStreamF32 : kStreamBf16;
    if (variant == 99 || (!large && !stream_covers((H > F ? H : F) * (f32 ? 4ll : 2ll)))) {
        if (f32) {
            if (phase & 1) launch_simple_gemm<float, true>(x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, s);
            if (phase & 2) launch_simple_gemm<float, false>(h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, s);
        } else {
            if (phase & 1) launch_simple_gemm<bf16_t, true>(x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, s);
            if (phase & 2) launch_simple_gemm<bf16_t, false>(h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, s);
        }
        return true;
    }
    if (variant == 0 || !large) {
        // Tuned default, phase by phase (the second product reads what the first wrote): few rows per expert, and shapes
        // without a large-tile kernel, go to the streaming kernel, the rest to the persistent kernel with three
        // LDS stages for the weight tile, on four or eight waves, and layers too shallow for its k stream to the one-workgroup-per-tile kernels
        // (8 waves gate/up, 4 waves down).
        bool ok = true;
        for (int ph = 1; ph <= 2; ph <<= 1) {
            if (!(phase & ph)) continue;
            const StreamPlan plan = plan_stream(elt, r_max, E, ph == 1 ? F : H, ph == 1 ? H : F, ph == 1, large, part_bytes);
            ok = launch_phase(plan, ph, elt, x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, part, s) && ok;
        }
        return ok;
    }
    if (variant >= 40 && launch_persist_ffn(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, variant, phase, s))
        return true;
    if (variant >= 30 && launch_pipe3_ffn(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, variant, phase, s))
        return true;
    return false;   // unknown variant
}

bool launch_expert_ffn_shared(const void* x_perm, const int32_t* offsets, int r_max, int H, int F, int E, const void* w_gate,
                              const void* w_up, const void* w_down, moe_dtype_t dt, void* h, void* y_perm, const void* x, int tokens,
                              int Fs, const void* ws_gate, const void* ws_up, const void* ws_down, void* s_h, void* s_y, const int32_t* s_offsets,
                              int variant, void* part, size_t part_bytes, hipStream_t s) {
    const bool large = large_covers(dt, H, F), s_large = large_covers(dt, H, Fs);
    const int elt = dt == MOE_F32 ? kStreamF32 : kStreamBf16;
    const long long longest = (dt == MOE_F32 ? 4ll : 2ll) * (H > F ? (H > Fs ? H : Fs) : (F > Fs ? F : Fs));
    if (variant != 0 || !stream_covers(longest))
        return launch_expert_ffn(x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, dt, h, y_perm, variant, 3, nullptr, 0, s) &&
               launch_expert_ffn(x, s_offsets, tokens, H, Fs, 1, ws_gate, ws_up, ws_down, dt, s_h, s_y, variant, 3, part, part_bytes, s);
    StreamPlan plan[3], s_plan[3];
    int pair[3];   // by phase, 1 and 2
    for (int ph = 1; ph <= 2; ++ph) {
        const int N = ph == 1 ? F : H, K = ph == 1 ? H : F, sN = ph == 1 ? Fs : H, sK = ph == 1 ? H : Fs;
        plan[ph] = plan_stream(elt, r_max, E, N, K, ph == 1, large, 0);
        s_plan[ph] = plan_stream(elt, tokens, 1, sN, sK, ph == 1, s_large, part_bytes);
        pair[ph] = plan_pair(elt, plan[ph], r_max, E, N, K, s_plan[ph], tokens, sN, sK, ph == 1);
    }
    auto routed = [&](int ph) {
        return launch_phase(plan[ph], ph, elt, x_perm, offsets, r_max, H, F, E, w_gate, w_up, w_down, h, y_perm, nullptr, s);
    };
    auto shared = [&](int ph) {
        return launch_phase(s_plan[ph], ph, elt, x, s_offsets, tokens, H, Fs, 1, ws_gate, ws_up, ws_down, s_h, s_y, part, s);
    };
    // A down product finds the rows that its gate/up product left in the memory-side cache if nothing long comes between (500 tokens,
    // 64 experts, 3584 x 2560, with 20480 shared: the layer takes 11 us longer with the shared gate/up in between).
    bool ok = true;
    if (pair[1] > 0) {
        launch_stream_pair(pair[1], x_perm, offsets, r_max, E, F, H, w_gate, w_up, h, x, s_offsets, tokens, Fs, H, ws_gate, ws_up, s_h, s);
    } else {
        if (pair[2] > 0) ok = shared(1);
        ok = routed(1) && ok;
    }
    if (pair[2] > 0) {
        launch_stream_pair(pair[2], h, offsets, r_max, E, H, F, w_down, nullptr, y_perm, s_h, s_offsets, tokens, H, Fs, ws_down, nullptr, s_y, s);
        return ok;
    }
    ok = routed(2) && ok;
    if (pair[1] == 0) ok = shared(1) && ok;
    return shared(2) && ok;
}

}  // namespace moe
