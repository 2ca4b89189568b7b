// Measurement probe, not part of the layer: how fast this GPU issues the bf16
// matrix instruction of the grouped GEMM when nothing else is in the way.
//
// Every workgroup copies a 64 KiB operand image into LDS once (256 rows of 64
// bf16 values for each of the two operands, rows of 128 bytes, 16-byte pieces
// XOR-swizzled by the row as in the GEMM kernels) and then loops over it: four
// waves, each with a 128 x 128 accumulator block, read their fragments from LDS
// and issue 16x16x32 MFMAs, as the GEMM's k loop does, with no global memory
// traffic, no barrier and no epilogue in the loop.  The rate depends on the VALUES in the image: all-zero
// operands run at the published peak, operands distributed like the workload's
// (activations ~N(0,1), weights ~N(0,0.02^2)) draw more power and the clock
// falls; the kernel reports the shader clock it ran at next to the elapsed time
// the caller measures.
#include "common.h"

namespace moe {

namespace {

__global__ __launch_bounds__(256) void probe_mfma_bf16_kernel(const uint32_t* __restrict__ image, int iters,
                                                              float* __restrict__ sink,
                                                              unsigned long long* __restrict__ ticks) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < 65536 / 16; i += 256)
        reinterpret_cast<u32x4*>(lds)[i] = reinterpret_cast<const u32x4*>(image)[i];
    __syncthreads();
    const unsigned long long c0 = __builtin_amdgcn_s_memtime(), r0 = __builtin_amdgcn_s_memrealtime();
    f32x4 acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int fr = lane & 15, fk = lane >> 4;
    const int row_a = (wave >> 1) * 128 + fr, row_b = (wave & 1) * 128 + fr;
    auto frag = [&](const uint8_t* base, int r, int ks) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(base + r * 128 + (((4 * ks + fk) ^ lds_swizzle(r)) << 4)));
    };
    // fragments as the GEMM reads them: the next k-step's under this one's matrix instructions, into the other of two sets
    bf16x8 a[2][8], b[2][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[0][i] = frag(lds, row_a + 16 * i, 0);
#pragma unroll
    for (int j = 0; j < 8; ++j) b[0][j] = frag(lds + 32768, row_b + 16 * j, 0);
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int m = 0; m < 64; ++m) {   // there and back over the columns
                const int i = m / 8, j = (i & 1) ? 7 - m % 8 : m % 8;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[ks][j], a[ks][i], acc[i][j], 0, 0, 0);
                if (m % 4 == 0) {
                    const int q = m / 4;
                    if (q < 8) a[ks ^ 1][q] = frag(lds, row_a + 16 * q, ks ^ 1);
                    else b[ks ^ 1][q - 8] = frag(lds + 32768, row_b + 16 * (q - 8), ks ^ 1);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) s += acc[i][j][v];
    sink[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
    if (ticks && blockIdx.x == 0 && threadIdx.x == 0) {
        ticks[0] = __builtin_amdgcn_s_memtime() - c0;       // shader clocks
        ticks[1] = __builtin_amdgcn_s_memrealtime() - r0;   // 100 MHz reference clocks
    }
}

typedef __attribute__((ext_vector_type(8))) int probe_i32x8;

// The same loop for the FP8 path: rows of 128 E4M3 bytes, every lane feeds 32
// bytes of a row (two 16-byte pieces, half a row apart) to a 16x16x128 MFMA, one
// per pair of fragments and pass over the image.
__global__ __launch_bounds__(256) void probe_mfma_fp8_kernel(const uint32_t* __restrict__ image, int iters,
                                                             float* __restrict__ sink,
                                                             unsigned long long* __restrict__ ticks) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < 65536 / 16; i += 256)
        reinterpret_cast<u32x4*>(lds)[i] = reinterpret_cast<const u32x4*>(image)[i];
    __syncthreads();
    const unsigned long long c0 = __builtin_amdgcn_s_memtime(), r0 = __builtin_amdgcn_s_memrealtime();
    f32x4 acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int fr = lane & 15, fk = lane >> 4;
    const int row_a = (wave >> 1) * 128 + fr, row_b = (wave & 1) * 128 + fr;
    auto frag = [&](const uint8_t* base, int r) -> probe_i32x8 {
        const u32x4 lo = *reinterpret_cast<const u32x4*>(base + r * 128 + ((fk ^ lds_swizzle(r)) << 4));
        const u32x4 hi = *reinterpret_cast<const u32x4*>(base + r * 128 + (((4 + fk) ^ lds_swizzle(r)) << 4));
        probe_i32x8 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            v[t] = (int)lo[t];
            v[4 + t] = (int)hi[t];
        }
        return v;
    };
    // one set of fragments, as the GEMM has it: all rows by half of the columns, then by the rest; each read again behind its last use
    probe_i32x8 a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = frag(lds, row_a + 16 * i);
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = frag(lds + 32768, row_b + 16 * j);
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int m = 0; m < 32; ++m) {
                const int i = m / 4, j = 4 * half + ((i & 1) ? 3 - m % 4 : m % 4);
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a[i], acc[i][j], 0, 0, 0, 0, 0, 0);
                if (m % 4 == 1 && m / 4 < 4) b[4 * (1 - half) + m / 4] = frag(lds + 32768, row_b + 16 * (4 * (1 - half) + m / 4));
                if (half == 1 && m % 4 == 3) a[i] = frag(lds, row_a + 16 * i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) s += acc[i][j][v];
    sink[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
    if (ticks && blockIdx.x == 0 && threadIdx.x == 0) {
        ticks[0] = __builtin_amdgcn_s_memtime() - c0;
        ticks[1] = __builtin_amdgcn_s_memrealtime() - r0;
    }
}

}  // namespace

void launch_probe_mfma_fp8(const void* image, int iters, int workgroups, float* sink, unsigned long long* ticks,
                           hipStream_t s) {
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(probe_mfma_fp8_kernel), 65536);
    hipLaunchKernelGGL(probe_mfma_fp8_kernel, dim3(workgroups), dim3(256), 65536, s,
                       static_cast<const uint32_t*>(image), iters, sink, ticks);
}

void launch_probe_mfma_bf16(const void* image, int iters, int workgroups, float* sink, unsigned long long* ticks,
                            hipStream_t s) {
    static OncePerDevice lds;
    allow_lds(lds, reinterpret_cast<const void*>(probe_mfma_bf16_kernel), 65536);
    hipLaunchKernelGGL(probe_mfma_bf16_kernel, dim3(workgroups), dim3(256), 65536, s,
                       static_cast<const uint32_t*>(image), iters, sink, ticks);
}

}  // namespace moe
