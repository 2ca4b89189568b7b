// The weight-streaming grouped GEMM (gemm_stream.hip): few rows per expert, and the shapes no other kernel takes.
#pragma once

#include "common.h"

namespace moe {

enum { kStreamF32 = 0, kStreamBf16 = 1, kStreamFp8 = 2 };   // operand type
// large tiles (another kernel), four waves, eight waves, small tiles (gemm_tiles.hip)
enum { kPlanLarge = 0, kPlanNarrow = 1, kPlanWide = 2, kPlanTiles = 3 };

struct StreamPlan {
    int kind;
    int units;    // wide: blocks of 32 weight rows per workgroup; small tiles: their form
    int splits;   // wide, large: parts of the contraction
    double us;    // what it is estimated to take, where kernels were compared
};

// rows of at most 16 MiB (32-bit offsets inside a tile)
bool stream_covers(long long K_bytes);
// The kernel for one product of r_max rows on E experts, [N, K] weights each; large_ok: the large tiles cover the shape;
// part_bytes: room for partial sums (0: the contraction is not split).  Depends on nothing but its arguments and options.
StreamPlan plan_stream(int elt, int r_max, int E, int N, int K, bool swiglu, bool large_ok, size_t part_bytes);
// room for partial sums that the plan wants, at most 64 MiB
size_t stream_part_bytes(int elt, int r_max, int E, int N, int K, bool swiglu, bool large_ok);
// C [rows, N] in bf16 from the partial planes [splits][r_max][N, or 2 N: gate and up] fp32, added in split order
void launch_stream_reduce(bool swiglu, const float* part, const int32_t* offsets, int E, int splits, int r_max, int N, void* C,
                          hipStream_t s);
// Weight blocks per workgroup (2, 4 or 8, see launch_stream_pair) of the shared expert's product (`tokens` rows) in one narrow launch with the routed
// experts', or 0: one after the other
int plan_pair(int elt, const StreamPlan& routed, int r_max, int E, int N, int K, const StreamPlan& shared, int tokens, int sN, int sK,
              bool swiglu);
// that launch: C [rows, N] as launch_stream, sC [tokens, sN] from the rows sA, all of one expert (s_offsets: 0, tokens)
void launch_stream_pair(int blocks, const void* A, const int32_t* offsets, int r_max, int E, int N, int K, const void* B0, const void* B1,
                        void* C, const void* sA, const int32_t* s_offsets, int tokens, int sN, int sK, const void* sB0, const void* sB1,
                        void* sC, hipStream_t s);
// -1 (default): by size; else 10 G + D: G weight blocks for gate/up and D for down (0: never, 2, 4 or 8, or the nearest that is built)
// where they can be paired
void set_pair_blocks(int v);
// -1 (default): by size; 0: only the shapes no other kernel takes; 1: always the narrow, 2: always the wide form.  10 + FB:
// narrow with FB (1, 2, 4, 8) blocks of 16 weight rows per workgroup (2 for 1 with SwiGLU; 2 or 4 for at most 16 rows in
// all); 20 + form: small tiles of that form; 100 S + U: wide with U (3 .. 8) units and S (1, 2, 4, 8, 16) splits, halved until they fit the contraction and the room; 2000 + S:
// the large tiles, their contraction in S (2 .. 16) parts where that fits the contraction and the room
void set_gemm_stream(int v);

// C [rows, N] = A [rows, K] . B0[e]^T; with B1 the SwiGLU pair silu(A B0^T) * (A B1^T), and with GU (bf16) also its two
// pre-activations, [rows, 2N].  FP8: s0, s1 dequantise the two products, s2 is the scale of the stored codes, amax
// (may be null) receives max |h|; without B1 the output is bf16.  part: the room the plan was made with.
void launch_stream(const StreamPlan& plan, int elt, const void* A, const int32_t* offsets, int r_max, int E, int N, int K,
                   const void* B0, const void* B1, void* C, void* GU, float s0, float s1, float s2, float* amax,
                   float* part, hipStream_t s);

}  // namespace moe
