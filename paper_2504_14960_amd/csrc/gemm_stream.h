// The weight-streaming grouped GEMM (gemm_stream.hip): few rows per expert, and the shapes no other kernel takes.
#pragma once

#include "common.h"

namespace moe {

enum { kStreamF32 = 0, kStreamBf16 = 1, kStreamFp8 = 2 };   // operand type of launch_stream

// rows of at most 16 MiB (32-bit offsets inside a tile)
bool stream_covers(long long K_bytes);
// whether this product is better off here than on the 256-row-tile kernels (see the definition)
bool stream_preferred(int r_max, int E, int N, bool swiglu);
// -1 (default): by size; 0: only the shapes no other kernel takes; 1: always
void set_gemm_stream(int v);

// C [rows, N] = A [rows, K] . B0[e]^T; with B1 the SwiGLU pair silu(A B0^T) * (A B1^T), and with GU (bf16) also its two
// pre-activations, [rows, 2N].  FP8: s0, s1 dequantise the two products, s2 is the scale of the stored codes, amax
// (may be null) receives max |h|; without B1 the output is bf16.
void launch_stream(int elt, const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0,
                   const void* B1, void* C, void* GU, float s0, float s1, float s2, float* amax, hipStream_t s);

}  // namespace moe
