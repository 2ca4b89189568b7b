// Helpers of the expert FFN's backward (Section 3.3: the backward workflow
// mirrors the forward; f_e of Eq. 1 by the chain rule).  The grouped GEMM
// kernels of this library multiply operands that are both contiguous along the
// contraction index ("NT").  The backward needs the other layouts, so operands
// are re-laid once and the same GEMM engine is reused:
//
//   transpose_batched_kernel   weights [B, R, C] -> [B, C, ld] (at a column
//                              offset, so W_gate^T and W_up^T can sit side by
//                              side for the input-gradient GEMM)
//   ragged_transpose_kernel    activations [rows, C] -> [C, Rp]: the rows of
//                              expert e become columns poff_e .. poff_e + n_e,
//                              every expert's segment padded with zeros to a
//                              multiple of 64 (at least 128) columns, so the
//                              weight-gradient GEMMs contract over whole k-tiles
//   swiglu_backward_kernel     (dh, g, u) -> dg | du side by side
//
// All bf16, tiles through LDS for the transposes.
#include "common.h"

namespace moe {

namespace {

// ---- transposes ----
// Bound by HBM: every byte is read once and written once.  What counts is where the workgroups that run at the same time
// read and write.
// Weights, results of more than 140 MiB (gate, up and down together): tiles of 256 rows x 64 columns, neighbours below one
// another, so that together they write whole rows of the result, 512 bytes each (and read whole 128-byte lines, some rows
// apart), loads and stores streamed past the caches.  64 matrices of 2048 x 6144, into rows of 4096, and of 6144 x 2048, us:
// 128 x 128 tiles, neighbours beside one another, 631 and 601 (5.1 and 5.4 TB/s); below one another and streamed, 593 and
// 576; 256 x 64 so 532 and 535 (6.0 TB/s), not streamed 574 and 576.  A plain copy of 1 GiB runs at 5.5 TB/s, streamed at 6.0
// to 6.2.
// Weights, smaller results: 128 x 128 tiles, neighbours beside one another, not streamed.  The products behind find the results
// in the 256 MB memory-side cache; larger ones they would not, and what is still to be written back holds them up.  The
// three transposes, dh and dx, us, streamed in tiles of 256 x 64 / so: 4 experts x 53 rows, 1024 x 1024 (25 MB) 55 / 47; 8 x
// 60, 1024 x 2048 (101 MB) 97 / 74; 8 x 100 and 8 x 800, 1024 x 2560 (126 MB) 113 / 102 and 216 / 223; 16 x 50 and 16 x 200,
// 1024 x 1408 (138 MB) 114 / 109 and 144 / 147; 8 x 100 and 8 x 600, 1024 x 3072 (151 MB) 127 / 126 and 229 / 236; 8 x 200,
// 2048 x 1536 (151 MB) 139 / 146.
// Activations: 128 x 128 tiles, neighbours beside one another; which of the two forms is ahead depends on the sizes: the four of
// a training step of 2048 tokens, 64 experts, 6144 x 2048, 174 so and 191 in tiles of 256 x 64, of 8192 tokens, 8 experts,
// 6144 x 16384, 787 and 772.
// All eight loads of a thread in flight, and 32-bit LDS traffic: a thread takes the same eight columns of two adjacent
// rows, so that a dword of the transposed tile is one of its element pairs, and the tile [column][row pair] is read back 16
// bytes at a time.  Group g of four dwords of column c lies at g ^ (c / 8) (64 columns: g ^ 2 (c / 8)): the 64 dwords a wave
// writes at a time then fall into 64 different banks.
struct TransposeRows {   // where 64 of the tile's rows come from
    int first, valid;    // first source row; how many of the 64 exist, the rest count as zeros
};

template <int TR, int TC, bool STREAM>   // tile: rows, columns
struct TransposeTile {
    static constexpr int PARTS = TR / 64, TP = TR / 2;                  // row pairs
    static constexpr int VC = TC / 8, RPT = 256 / VC, NP = TP / RPT;    // 16-byte pieces across; row pairs a pass; passes
    static constexpr int VR = TR / 8, CPT = 256 / VR;                   // pieces along a row of the result; columns a pass
    static_assert(RPT <= 32 && 32 % RPT == 0, "a pass lies in one part");
    uint32_t pair[TC][TP];

    static __device__ __forceinline__ int at(int group, int c) { return 4 * (group ^ ((c >> 3) * (128 / TC))); }

    // columns c0 .. c0 + TC - 1 (below `cols`) of PARTS times 64 rows of `src`
    __device__ __forceinline__ void load(const uint16_t* __restrict__ src, size_t ld, int c0, int cols,
                                         const TransposeRows (&part)[PARTS]) {
        const int c = (threadIdx.x % VC) * 8, rp = threadIdx.x / VC;
        u32x4 v[NP][2];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const TransposeRows h = part[p * RPT / 32];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int rr = 2 * (p * RPT % 32 + rp) + k;
                v[p][k] = u32x4{0u, 0u, 0u, 0u};
                if (rr < h.valid && c0 + c < cols) {   // cols is a multiple of 8
                    const u32x4* from = reinterpret_cast<const u32x4*>(src + (size_t)(h.first + rr) * ld + c0 + c);
                    v[p][k] = STREAM ? __builtin_nontemporal_load(from) : *from;
                }
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int q = p * RPT + rp, to = at(q >> 2, c) + (q & 3);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                pair[c + 2 * j][to] = (v[p][0][j] & 0xffffu) | (v[p][1][j] << 16);
                pair[c + 2 * j + 1][to] = (v[p][0][j] >> 16) | (v[p][1][j] & 0xffff0000u);
            }
        }
    }

    // output row c0 + c gets the tile's column c at dst[(c0 + c) * ldo + o0 ..], n_out elements of it (a multiple of 8)
    __device__ __forceinline__ void store(uint16_t* __restrict__ dst, size_t ldo, int c0, int cols, size_t o0, int n_out) const {
        const int g = threadIdx.x % VR;
#pragma unroll
        for (int p = 0; p < TC / CPT; ++p) {
            const int c = CPT * p + threadIdx.x / VR;
            if (c0 + c >= cols || g * 8 >= n_out) continue;
            const u32x4 v = *reinterpret_cast<const u32x4*>(&pair[c][at(g, c)]);
            u32x4* const to = reinterpret_cast<u32x4*>(dst + (size_t)(c0 + c) * ldo + o0 + g * 8);
            if (STREAM) __builtin_nontemporal_store(v, to);
            else *to = v;
        }
    }
};
using ActTile = TransposeTile<128, 128, false>;
constexpr int kActTile = 128;
constexpr size_t kCachedBytes = 140u << 20;   // results up to here are left to the caches

// dst[b][c][col0 + r] = src[b][r][c];  R, C multiples of 8.  DOWN: neighbouring workgroups below one another.
template <int TR, int TC, bool STREAM, bool DOWN>
__global__ __launch_bounds__(256) void transpose_batched_kernel(const uint16_t* __restrict__ src, int R, int C,
                                                                uint16_t* __restrict__ dst, size_t ldo, int col0) {
    using Tile = TransposeTile<TR, TC, STREAM>;
    __shared__ __attribute__((aligned(16))) Tile tile;
    const unsigned across = DOWN ? (R + TR - 1) / TR : (C + TC - 1) / TC;
    const int near = (int)(blockIdx.x % across), far = (int)(blockIdx.x / across);
    const int b = blockIdx.z, r0 = (DOWN ? near : far) * TR, c0 = (DOWN ? far : near) * TC;
    TransposeRows part[Tile::PARTS];
#pragma unroll
    for (int q = 0; q < Tile::PARTS; ++q) part[q] = {r0 + 64 * q, R - r0 - 64 * q};
    tile.load(src + (size_t)b * R * C, (size_t)C, c0, C, part);
    __syncthreads();
    tile.store(dst + (size_t)b * C * ldo, ldo, c0, C, (size_t)col0 + r0, min(TR, R - r0));
}

template <int TR, int TC, bool STREAM, bool DOWN>
void transpose_batched(const void* src, int B, int R, int C, void* dst, size_t ldo, int col0, hipStream_t s) {
    hipLaunchKernelGGL((transpose_batched_kernel<TR, TC, STREAM, DOWN>), dim3((unsigned)((R + TR - 1) / TR) * ((C + TC - 1) / TC), 1, B),
                       dim3(256), 0, s, static_cast<const uint16_t*>(src), R, C, static_cast<uint16_t*>(dst), ldo, col0);
}

// padded length of an expert's column segment in the transposed activations
__device__ __forceinline__ int padded_rows(int n) { return n <= 0 ? 0 : max(128, (n + 63) & ~63); }

// poff[e] = first column of expert e's zero-padded segment (exclusive prefix of the padded row counts), e = 0..E.
// One workgroup of 256 threads; E <= 256.
__global__ __launch_bounds__(256) void ragged_offsets_kernel(const int32_t* __restrict__ offsets, int E,
                                                             int32_t* __restrict__ poff) {
    __shared__ int scan[2][256];
    const int tid = threadIdx.x;
    const int pn = (tid < E) ? padded_rows(offsets[tid + 1] - offsets[tid]) : 0;
    scan[0][tid] = pn;
    __syncthreads();
    int cur = 0;
    for (int d = 1; d < 256; d <<= 1) {
        scan[cur ^ 1][tid] = scan[cur][tid] + ((tid >= d) ? scan[cur][tid - d] : 0);
        cur ^= 1;
        __syncthreads();
    }
    if (tid < E) poff[tid + 1] = scan[cur][tid];
    if (tid == 0) poff[0] = 0;
}

// dst[c][poff_e + (r - lo_e)] = src[r][c] for the rows r of expert e; the pad up to
// padded_rows(n_e) is zero.  One workgroup per (128-column block, 128-row block of the
// padded axis); the expert of a padded position is the one whose segment [poff_e,
// poff_e+1) holds it (segments are multiples of 64, so a half block never straddles two).
__global__ __launch_bounds__(256) void ragged_transpose_kernel(const uint16_t* __restrict__ src,
                                                               const int32_t* __restrict__ offsets,
                                                               const int32_t* __restrict__ poff, int E, int C,
                                                               uint16_t* __restrict__ dst, size_t ldo) {
    __shared__ __attribute__((aligned(16))) ActTile tile;
    __shared__ int seg[2][2];   // of each half: first source row, valid rows from there on (-1: past the last segment)
    const int p0 = blockIdx.y * kActTile, c0 = blockIdx.x * kActTile;
    if (threadIdx.x < 2) seg[threadIdx.x][1] = -1;
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 256) {
        const int lo_p = poff[e], hi_p = poff[e + 1];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = p0 + 64 * h;
            if (lo_p <= p && p < hi_p) {   // at most one expert
                const int lo = offsets[e], n = offsets[e + 1] - lo;
                seg[h][0] = lo + (p - lo_p);
                seg[h][1] = max(0, n - (p - lo_p));   // 0: 64 positions of pure padding
            }
        }
    }
    __syncthreads();
    if (seg[0][1] < 0) return;   // past the last expert's padding: nothing to write
    const TransposeRows half[2] = {{seg[0][0], min(64, seg[0][1])}, {seg[1][0], min(64, seg[1][1])}};
    const int n_out = seg[1][1] < 0 ? 64 : kActTile;
    tile.load(src, (size_t)C, c0, C, half);
    __syncthreads();
    tile.store(dst, ldo, c0, C, (size_t)p0, n_out);
}

// dg | du from dh [rows, F] and g, u (bf16, rows ld_gu elements apart; out [rows, 2F]): with s = 1/(1+e^-g),
//   du = dh * g * s,   dg = dh * u * s * (1 + g * (1 - s)).
// Only rows below *n_rows (device: the kept-row count) are processed.
__global__ __launch_bounds__(256) void swiglu_backward_kernel(const uint16_t* __restrict__ dh,
                                                              const uint16_t* __restrict__ g,
                                                              const uint16_t* __restrict__ u, size_t ld_gu,
                                                              const int32_t* __restrict__ n_rows, int F,
                                                              uint16_t* __restrict__ out) {
    const int rows = *n_rows;
    const int vpr = F / 8;  // 16-byte vectors per row
    const size_t nvec = (size_t)rows * vpr;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (size_t)gridDim.x * 256) {
        const size_t r = i / vpr;
        const int c = (int)(i - r * vpr) * 8;
        const u32x4 a = *reinterpret_cast<const u32x4*>(dh + r * F + c);
        const u32x4 b = *reinterpret_cast<const u32x4*>(g + r * ld_gu + c);
        const u32x4 d = *reinterpret_cast<const u32x4*>(u + r * ld_gu + c);
        u32x4 og, ou;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float dgv[2], duv[2];
#pragma unroll
            for (int hlf = 0; hlf < 2; ++hlf) {
                const float dhv = __uint_as_float(hlf ? (a[j] & 0xffff0000u) : (a[j] << 16));
                const float gv = __uint_as_float(hlf ? (b[j] & 0xffff0000u) : (b[j] << 16));
                const float uv = __uint_as_float(hlf ? (d[j] & 0xffff0000u) : (d[j] << 16));
                const float s = __builtin_amdgcn_rcpf(1.f + __expf(-gv));
                duv[hlf] = dhv * gv * s;
                dgv[hlf] = dhv * uv * s * (1.f + gv * (1.f - s));
            }
            og[j] = pack2_bf16(dgv[0], dgv[1]);
            ou[j] = pack2_bf16(duv[0], duv[1]);
        }
        *reinterpret_cast<u32x4*>(out + r * 2 * F + c) = og;
        *reinterpret_cast<u32x4*>(out + r * 2 * F + F + c) = ou;
    }
}

}  // namespace

void launch_weights_transpose(const void* w_gate, const void* w_up, const void* w_down, int E, int H, int F, void* wgu_t,
                              void* wd_t, hipStream_t s) {
    const auto transpose = (size_t)6 * E * H * F <= kCachedBytes ? transpose_batched<128, 128, false, false>
                                                                 : transpose_batched<256, 64, true, true>;
    transpose(w_gate, E, F, H, wgu_t, (size_t)2 * F, 0, s);   // [E,F,H] -> [E,H,0:F]
    transpose(w_up, E, F, H, wgu_t, (size_t)2 * F, F, s);     //            [E,H,F:2F]
    transpose(w_down, E, H, F, wd_t, (size_t)H, 0, s);        // [E,H,F] -> [E,F,H]
}

void launch_ragged_offsets(const int32_t* offsets, int E, int32_t* poff, hipStream_t s) {
    hipLaunchKernelGGL(ragged_offsets_kernel, dim3(1), dim3(256), 0, s, offsets, E, poff);
}

// rp_max: the static bound on the padded axis (a multiple of 64); blocks past the real padded length exit.
// poff: the E + 1 segment starts written by launch_ragged_offsets
void launch_ragged_transpose(const void* src, const int32_t* offsets, const int32_t* poff, int E, int C, int rp_max,
                             void* dst, hipStream_t s) {
    if (rp_max <= 0 || C <= 0) return;
    hipLaunchKernelGGL(ragged_transpose_kernel, dim3((C + kActTile - 1) / kActTile, (rp_max + kActTile - 1) / kActTile), dim3(256),
                       0, s, static_cast<const uint16_t*>(src), offsets, poff, E, C, static_cast<uint16_t*>(dst),
                       (size_t)rp_max);
}

void launch_swiglu_backward(const void* dh, const void* g, const void* u, size_t ld_gu, const int32_t* n_rows,
                            int r_max, int F, void* out, hipStream_t s) {
    if (r_max <= 0) return;
    size_t blocks = ((size_t)r_max * (F / 8) + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    hipLaunchKernelGGL(swiglu_backward_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                       static_cast<const uint16_t*>(dh), static_cast<const uint16_t*>(g),
                       static_cast<const uint16_t*>(u), ld_gu, n_rows, F, static_cast<uint16_t*>(out));
}

}  // namespace moe
