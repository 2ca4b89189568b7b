// Pieces shared by the persistent grouped-GEMM kernels (bf16 and FP8): the
// register-resident tile scheduler and small helpers.
#pragma once

#include "gemm_tile.h"
#include "tile_cost.h"

namespace moe {

// workgroups a persistent grouped-GEMM kernel is launched with: one per compute
// unit unless overridden (at least 8, one per tile share)
int persist_grid();
// rows of the tiles of every launch that would choose them (256, 192 or 128); 0: chosen (see pick_height)
int persist_tile_rows();
// whether a launch over E experts uses the kernels whose waves without valid rows skip the multiplications
bool persist_idle_skip(int E);

namespace {

// force a wave-uniform value into scalar registers
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ const uint8_t* uni(const uint8_t* p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = uni((uint32_t)u), hi = uni((uint32_t)(u >> 32));
    return reinterpret_cast<const uint8_t*>(((uint64_t)hi << 32) | lo);
}

// sum of v over the lanes that describe E experts, four to a lane (the others hold nothing), in lane 0
__device__ __forceinline__ int expert_sum(int v, int E) {
    for (int d = 1; 4 * d < E; d <<= 1) v += __shfl_xor(v, d, 64);
    return __builtin_amdgcn_readfirstlane(v);
}

// The height of the tiles of a launch: 256, 192 or 128 rows, whichever takes least by the estimate (a lower one only where
// it is ahead by 3 %).  Every wave of every workgroup comes to the same result: it depends on the offsets and on the launch
// alone.  What the lower tiles gain is rows of padding and nearly empty last rounds, what they cost is more reads of the
// weight panels per row: at full size a row of a 192-row tile takes as long as one of a 256-row tile, a row of a 128-row
// tile a fifth longer.
__device__ __forceinline__ int pick_height(const TileCosts& c, const int32_t* __restrict__ offsets, int E, int ntn, int kt, int lane) {
    int m256 = 0, m192 = 0, m128 = 0, some = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int e = lane * 4 + j;
        const int n = e < E ? max(0, offsets[e + 1] - offsets[e]) : 0;
        m256 += (n + 255) / 256;
        m192 += (n + 191) / 192;
        m128 += (n + 127) / 128;
        some += n > 0;
    }
    m256 = expert_sum(m256, E);
    m192 = expert_sum(m192, E);
    m128 = expert_sum(m128, E);
    some = expert_sum(some, E);
    if (some == 0) return 256;
    const int slots = gridDim.x;
    float best = 0.97f * tiles_us(c.h256, m256, some, ntn, slots, kt);
    int h = 256;
    const float t192 = tiles_us(c.h192, m192, some, ntn, slots, kt), t128 = tiles_us(c.h128, m128, some, ntn, slots, kt);
    if (t192 < best) {
        best = t192;
        h = 192;
    }
    if (t128 < best) h = 128;
    return __builtin_amdgcn_readfirstlane(h);
}

// A block of at most 32 output rows as a buffer: `rows` rows of `pitch` bytes from `base` on, and stores past them are dropped by the hardware.  A
// store is thus one instruction whatever lanes have rows or columns to store, so that a wait can count it (see persist_body).
struct RowBuffer {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ RowBuffer(void* base, int rows, uint32_t pitch)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(base, 0, (int)((uint32_t)min(max(rows, 0), 32) * pitch), 0x00027000)) {}
    // streamed past the caches, as __builtin_nontemporal_store
    __device__ __forceinline__ void store(u32x4 v, uint32_t offset) const {
        __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)offset, 0, 2);
    }
};
constexpr uint32_t kNoColumn = 0x80000000u;   // an offset past the end of every row buffer
constexpr int kMaxColumns = 1 << 24;          // 32 rows of so many bf16 columns end below kNoColumn

// All but the LOADS youngest vector memory operations of this wave are complete, or, with stores_too (wave-uniform), all but the
// LOADS + STORES youngest; and its LDS reads are in registers.  stores_too is false afterwards.  The compiler peels the first
// turn of the k loop for the branch; a form that kept one copy was 6 % slower (gradients of 64 experts x 172 rows, 6144 x 2048).
template <int LOADS, int STORES>
__device__ __forceinline__ void wait_memory(int& stores_too) {
    constexpr int ALL = LOADS + STORES;
    __builtin_amdgcn_s_waitcnt((ALL & 0xF) | ((ALL >> 4) << 14));   // vmcnt(ALL), lgkmcnt(0)
    if constexpr (STORES != 0) {
        if (!uni(stores_too)) __builtin_amdgcn_s_waitcnt((LOADS & 0xF) | ((LOADS >> 4) << 14));
        stores_too = 0;
    }
}

// wave-uniform description of one output tile
struct PTile {
    const uint8_t* a;   // first activation row of the tile (k = 0)
    const uint8_t* b0;  // first weight row: gate (SwiGLU) or down projection
    const uint8_t* b1;  // first up-projection row (SwiGLU only)
    uint32_t a_lim;     // byte offset (from a) of the last valid activation row
    uint32_t b_lim;     // byte offset (from b0 / b1) of the last valid weight row
    int row0, rows, n0;
    int kt;             // k-tiles of this output tile (weight-gradient form; 0 = the launch's common count)
    int split;          // contraction in parts: which one
    int krows;          // row-major weight-gradient form: rows of the expert, i.e. valid length of the contraction
    bool valid;
};

// Every wave keeps the whole schedule in registers: lane l describes experts
// 4l .. 4l+3 (first row, row count, exclusive prefix of M-tile counts).
template <int BM, bool BY_ROUND = true>
struct TileSched {
    int lo[4], n[4], pex[4], pend;
    int MT, ntn, per, nwx, wgx, xcd, total;

    // splits: parts of the contraction, each a tile list of its own
    __device__ __forceinline__ void init(const int32_t* __restrict__ offsets, int E, int ntn_, int lane, int splits = 1) {
        int mt[4], s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = lane * 4 + j;
            lo[j] = 0;
            n[j] = 0;
            if (e < E) {
                lo[j] = offsets[e];
                n[j] = offsets[e + 1] - lo[j];
            }
            mt[j] = (n[j] > 0) ? (n[j] + BM - 1) / BM : 0;
            s += mt[j];
        }
        int incl = s;
        for (int d = 1; 4 * d < E; d <<= 1) {   // lanes past the last expert have nothing to add
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        pex[0] = incl - s;
#pragma unroll
        for (int j = 1; j < 4; ++j) pex[j] = pex[j - 1] + mt[j - 1];
        pend = incl;
        MT = __builtin_amdgcn_readlane(incl, (E - 1) >> 2);
        ntn = ntn_;
        total = MT * ntn * splits;
        per = (total + 7) / 8;              // tiles per XCD share
        xcd = blockIdx.x & 7;               // workgroups are dealt round-robin to the 8 XCDs
        wgx = blockIdx.x >> 3;
        nwx = (gridDim.x + 7 - xcd) >> 3;   // workgroups of this launch that share the XCD
    }

    // the i-th tile of this workgroup
    // row_bytes: bytes per operand row (contraction length times element size)
    template <bool SPLIT = false>
    __device__ __forceinline__ PTile get(int i, const uint8_t* A, const uint8_t* B0, const uint8_t* B1, int N,
                                         size_t row_bytes, int outn, int splits = 1) const {
        constexpr int MG = 8;
        PTile t;
        t.a = A; t.b0 = B0; t.b1 = B1; t.a_lim = 0; t.b_lim = 0; t.row0 = 0; t.rows = 0; t.n0 = 0; t.kt = 0; t.split = 0; t.krows = 0;
        // BY_ROUND: whole rounds (one tile per workgroup of the launch) are dealt to the XCDs round by round: in
        // round i XCD x runs the nwx consecutive tiles from (8 i + x) nwx on, so at any time the eight XCDs work on
        // neighbouring stretches of the list and what they have in common (activation panels of one M-group) is
        // fetched from memory once and found in the memory-side cache by the others.  The tiles left over after
        // the last whole round are cut into eight contiguous shares.  Otherwise every XCD takes a contiguous
        // eighth of the list.
        int L;
        if (BY_ROUND && (gridDim.x & 7) == 0) {
            const int round_tiles = 8 * nwx, whole = total / round_tiles;
            if (i < whole) {
                L = (i * 8 + xcd) * nwx + wgx;
                t.valid = true;
            } else {
                const int left = total - whole * round_tiles, share = (left + 7) >> 3;
                const int j = wgx + (i - whole) * nwx;
                L = whole * round_tiles + xcd * share + j;
                t.valid = (j < share) && (L < total);
            }
        } else {
            const int j = wgx + i * nwx;
            L = xcd * per + j;
            t.valid = (j < per) && (L < total);
        }
        if (!t.valid) return t;
        if constexpr (SPLIT) {
            t.split = uni(L / (MT * ntn));
            L -= t.split * (MT * ntn);
        }
        const int qm = L / ntn;
        int hit = -1, my_p = 0, my_end = 0, my_lo = 0, my_n = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int end = (q < 3) ? pex[q + 1] : pend;
            if (pex[q] <= qm && qm < end) {
                hit = q; my_p = pex[q]; my_end = end; my_lo = lo[q]; my_n = n[q];
            }
        }
        const uint64_t bal = __ballot(hit >= 0);  // exactly one lane: the M-tile ranges partition [0, MT)
        const int src = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)bal) - 1);
        const int e = 4 * src + __builtin_amdgcn_readlane(hit, src);
        const int p_e = __builtin_amdgcn_readlane(my_p, src);
        const int mt_e = __builtin_amdgcn_readlane(my_end, src) - p_e;
        const int lo_e = __builtin_amdgcn_readlane(my_lo, src);
        const int n_e = __builtin_amdgcn_readlane(my_n, src);
        // inside an expert: ceil(mt/MG) groups of near-equal size, tiles ordered
        // (M-group, N, M-in-group) so that concurrently running tiles share panels in L2
        const int Le = L - p_e * ntn;
        const int ng = (mt_e + MG - 1) / MG;
        const int gbase = mt_e / ng, grem = mt_e % ng;
        const int big = grem * (gbase + 1) * ntn;
        int g, gsz, m_first, rem;
        if (Le < big) {
            gsz = gbase + 1;
            g = Le / (gsz * ntn);
            rem = Le - g * gsz * ntn;
            m_first = g * gsz;
        } else {
            gsz = gbase;
            g = (Le - big) / (gsz * ntn);
            rem = (Le - big) - g * gsz * ntn;
            m_first = grem * (gbase + 1) + g * gsz;
        }
        const int nt = rem / gsz;
        const int m = m_first + rem - nt * gsz;
        t.row0 = uni(lo_e + m * BM);
        t.rows = uni(min(BM, lo_e + n_e - t.row0));
        t.n0 = uni(nt * outn);
        const size_t k2 = row_bytes;
        t.a = uni(A + (size_t)t.row0 * k2);
        const size_t brow = ((size_t)e * N + t.n0) * k2;
        t.b0 = uni(B0 + brow);
        t.b1 = uni(B1 + brow);
        t.a_lim = uni((uint32_t)(t.rows - 1) * (uint32_t)k2);
        t.b_lim = uni((uint32_t)(min(outn, N - t.n0) - 1) * (uint32_t)k2);
        if constexpr (SPLIT) {
            const int all = (int)(row_bytes / 128), k0 = uni((int)((long long)all * t.split / splits));
            t.kt = uni((int)((long long)all * (t.split + 1) / splits)) - k0;
            t.a += (size_t)k0 * 128;
            t.b0 += (size_t)k0 * 128;
            t.b1 += (size_t)k0 * 128;
        }
        return t;
    }
};

// What lane l of a wave holds of experts 4l .. 4l+3, and the search over it: `first[q]` ascends over the experts.  All lanes of
// the wave take part in both calls: a lane's values can be read while it is active only.
struct ExpertLanes {
    int first[4];   // exclusive prefix of what the experts have

    // The last expert whose prefix is at most v (v differs from lane to lane): its lane, and its place q in that lane's four
    __device__ __forceinline__ void find(int v, int E, int& lane_of, int& q) const {
        lane_of = 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const int c = lane_of + d;
            if (__shfl(first[0], c, 64) <= v && 4 * c < E) lane_of = c;
        }
        q = 0;
#pragma unroll
        for (int j = 1; j < 4; ++j)
            if (__shfl(first[j], lane_of, 64) <= v) q = j;
    }
    // of four values per lane, the one of the expert found
    static __device__ __forceinline__ int at(const int (&v)[4], int lane_of, int q) {
        int r = __shfl(v[0], lane_of, 64);
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            const int o = __shfl(v[j], lane_of, 64);
            if (q == j) r = o;
        }
        return r;
    }
};

// Schedule of the weight-gradient form: C [E, M, N], for expert e the product of
// A_t[:, seg_e] and B_t[:, seg_e]^T over the expert's zero-padded column segment
// (padded length = 0 for an expert without rows, else max(128, n rounded up to
// 64)).  Every non-empty expert has the same mt x nt output tiles; what differs
// from tile to tile is the number of k-tiles, so the XCD shares are cut by work,
// not by tile count: every XCD takes the same eighth of EVERY expert's tiles (a
// contiguous block of the expert's tile order, so the tiles an XCD runs at once
// still share panels in its L2), and its workgroups walk that list round-robin.
// The tiles of a workgroup are worked out 64 at a time: lane l of every wave describes the l-th of them, so that the search for
// its expert and the divisions are made once for 64 tiles, and a tile costs a few readlanes.  A tile of these is a few k-tiles,
// and finding it anew stood between two of them with the matrix pipe empty (three gradients of 64 experts x 172 rows, 6144 x
// 2048: 1660 / 1628 us.  In the forward's schedule it made the down product 0.5 % faster and the gate/up product 1 % slower.)
template <int BM, int BN>
struct WgradSched {
    int t_m, t_n, t_e, t_seg, t_kt;                        // this lane's tile: k-tiles 0 = none
    const int32_t* offsets;
    int E, lane, batch, mt, nt;

    __device__ __forceinline__ void init(const int32_t* __restrict__ offsets_, int E_, int M, int N, int lane_) {
        offsets = offsets_;
        E = E_;
        lane = lane_;
        mt = (M + BM - 1) / BM;
        nt = (N + BN - 1) / BN;
        fill(0);
    }

    // tiles 64 b .. 64 b + 63 of this workgroup
    __device__ __forceinline__ void fill(int b) {
        constexpr int MG = 8;
        batch = b;
        int seg[4], len[4];   // segment start / padded length (elements)
        ExpertLanes x;        // over the experts with rows
        int s_len = 0, s_cnt = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = lane * 4 + j;
            int n = 0;
            if (e < E) n = offsets[e + 1] - offsets[e];
            len[j] = n <= 0 ? 0 : max(128, (n + 63) & ~63);
            s_len += len[j];
            s_cnt += len[j] > 0;
        }
        int incl_len = s_len, incl_cnt = s_cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int ol = __shfl_up(incl_len, d, 64), oc = __shfl_up(incl_cnt, d, 64);
            if (lane >= d) {
                incl_len += ol;
                incl_cnt += oc;
            }
        }
        seg[0] = incl_len - s_len;
        x.first[0] = incl_cnt - s_cnt;
#pragma unroll
        for (int j = 1; j < 4; ++j) {
            seg[j] = seg[j - 1] + len[j - 1];
            x.first[j] = x.first[j - 1] + (len[j - 1] > 0);
        }
        const int xcd = blockIdx.x & 7, tpe = mt * nt;
        const int part0 = (int)((long long)xcd * tpe / 8);           // this XCD's slice of an expert's tiles
        const int part_n = (int)((long long)(xcd + 1) * tpe / 8) - part0;
        const int total = __builtin_amdgcn_readlane(incl_cnt, 63) * part_n;   // tiles of this XCD
        const int nwx = (gridDim.x + 7 - xcd) >> 3;
        const int j = (int)(blockIdx.x >> 3) + (64 * b + lane) * nwx;
        const bool valid = j < total;
        const int qe = valid ? j / part_n : 0;   // index among the experts with rows (part_n > 0 since total > 0)
        int at, q;
        x.find(qe, E, at, q);   // experts without rows behind the qe-th one have the next index, those in front come first
        t_e = 4 * at + q;
        t_seg = ExpertLanes::at(seg, at, q);
        const int len_e = ExpertLanes::at(len, at, q);
        t_kt = valid ? len_e / 64 : 0;
        // inside an expert: groups of MG M-tiles, ordered (M-group, N, M-in-group)
        const int Le = part0 + (valid ? j - qe * part_n : 0);
        const int full = (mt / MG) * MG * nt;
        if (Le < full) {
            const int g = Le / (MG * nt), rem = Le - g * MG * nt;
            t_n = rem / MG;
            t_m = g * MG + rem - t_n * MG;
        } else {
            const int tail = max(mt % MG, 1), rem = Le - full;   // a tile here has tail > 0
            t_n = rem / tail;
            t_m = (mt / MG) * MG + rem - t_n * tail;
        }
    }

    // the i-th tile of this workgroup (asked for in ascending order); ld = elements per row of A_t and B_t
    __device__ __forceinline__ PTile get(int i, const uint8_t* A, const uint8_t* B, int M, int N, int ld) {
        PTile t;
        t.a = A; t.b0 = B; t.b1 = B; t.a_lim = 0; t.b_lim = 0; t.row0 = 0; t.rows = 0; t.n0 = 0; t.kt = 0; t.split = 0; t.krows = 0;
        if (uni(i >> 6) != batch) fill(uni(i >> 6));
        const int l = uni(i & 63);
        t.kt = __builtin_amdgcn_readlane(t_kt, l);
        t.valid = t.kt > 0;
        if (!t.valid) return t;
        const int m = __builtin_amdgcn_readlane(t_m, l), n = __builtin_amdgcn_readlane(t_n, l);
        const int e = __builtin_amdgcn_readlane(t_e, l), seg_e = __builtin_amdgcn_readlane(t_seg, l);
        const size_t k2 = (size_t)ld * 2;
        t.rows = uni(min(BM, M - m * BM));
        t.row0 = uni(e * M + m * BM);
        t.n0 = uni(n * BN);
        t.a = uni(A + (size_t)(m * BM) * k2 + (size_t)seg_e * 2);
        t.b0 = uni(B + (size_t)(n * BN) * k2 + (size_t)seg_e * 2);
        t.b1 = t.b0;
        t.a_lim = uni((uint32_t)(t.rows - 1) * (uint32_t)k2);
        t.b_lim = uni((uint32_t)(min(BN, N - t.n0) - 1) * (uint32_t)k2);
        return t;
    }
};

// Schedule of the weight-gradient form on ROW-MAJOR activations: C [E, M, N], for expert e the product
// A[rows_e, :]^T B[rows_e, :] with A [rows, lda] and B [rows, ldb] as the layer holds them (rows grouped by expert).
// The contraction runs over the expert's rows in k-tiles of 64 rows; rows past the expert's last one are read from a
// zero row by the kernel.  Tile order and XCD shares as in WgradSched.  Every tile gets at least two k-tiles (the
// k stream needs them; the second of a short expert is all zero rows).  Lane l describes experts 4l .. 4l+3.
template <int BM, int BN>
struct WgradSchedKM {
    int lo[4], n[4], pex[4], pend;
    int mt, nt, tpe, nwx, wgx, part0, part_n, total;

    __device__ __forceinline__ void init(const int32_t* __restrict__ offsets, int E, int M, int N, int lane) {
        int s_cnt = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = lane * 4 + j;
            lo[j] = 0;
            n[j] = 0;
            if (e < E) {
                lo[j] = offsets[e];
                n[j] = max(0, offsets[e + 1] - lo[j]);
            }
            s_cnt += n[j] > 0;
        }
        int incl_cnt = s_cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int oc = __shfl_up(incl_cnt, d, 64);
            if (lane >= d) incl_cnt += oc;
        }
        pex[0] = incl_cnt - s_cnt;
#pragma unroll
        for (int j = 1; j < 4; ++j) pex[j] = pex[j - 1] + (n[j - 1] > 0);
        pend = incl_cnt;
        mt = (M + BM - 1) / BM;
        nt = (N + BN - 1) / BN;
        tpe = mt * nt;
        const int xcd = blockIdx.x & 7;
        part0 = (int)((long long)xcd * tpe / 8);
        part_n = (int)((long long)(xcd + 1) * tpe / 8) - part0;
        total = __builtin_amdgcn_readlane(incl_cnt, 63) * part_n;
        wgx = blockIdx.x >> 3;
        nwx = (gridDim.x + 7 - xcd) >> 3;
    }

    // lda, ldb: elements per row of A and B
    __device__ __forceinline__ PTile get(int i, const uint8_t* A, const uint8_t* B, int M, int N, int lda,
                                         int ldb) const {
        constexpr int MG = 8;
        PTile t;
        t.a = A; t.b0 = B; t.b1 = B; t.a_lim = 0; t.b_lim = 0; t.row0 = 0; t.rows = 0; t.n0 = 0; t.kt = 0; t.split = 0; t.krows = 0;
        const int j = wgx + i * nwx;
        t.valid = j < total;
        if (!t.valid) return t;
        const int qe = j / part_n;
        int hit = -1, my_lo = 0, my_n = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (n[q] > 0 && pex[q] == qe) {
                hit = q; my_lo = lo[q]; my_n = n[q];
            }
        const uint64_t bal = __ballot(hit >= 0);
        const int src = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)bal) - 1);
        const int e = 4 * src + __builtin_amdgcn_readlane(hit, src);
        const int lo_e = __builtin_amdgcn_readlane(my_lo, src);
        const int n_e = __builtin_amdgcn_readlane(my_n, src);
        const int Le = part0 + j - qe * part_n;
        const int full = (mt / MG) * MG * nt;
        int m, nn;
        if (Le < full) {
            const int g = Le / (MG * nt), rem = Le - g * MG * nt;
            nn = rem / MG;
            m = g * MG + rem - nn * MG;
        } else {
            const int tail = mt % MG, rem = Le - full;
            nn = rem / tail;
            m = (mt / MG) * MG + rem - nn * tail;
        }
        t.rows = uni(min(BM, M - m * BM));
        t.row0 = uni(e * M + m * BM);
        t.n0 = uni(nn * BN);
        t.krows = uni(n_e);
        t.kt = uni(max(2, (n_e + 63) / 64));
        t.a = uni(A + ((size_t)lo_e * lda + (size_t)m * BM) * 2);
        t.b0 = uni(B + ((size_t)lo_e * ldb + (size_t)t.n0) * 2);
        t.b1 = t.b0;
        // last 16-byte piece of a tile row that still lies inside the matrix row
        t.a_lim = uni((uint32_t)(t.rows * 2 - 16));
        t.b_lim = uni((uint32_t)(min(BN, N - t.n0) * 2 - 16));
        return t;
    }
};

}  // namespace

}  // namespace moe
