// Batched ensemble scoring.  Two kernels, both giving the fp32 sum of the
// reached leaves in tree order from +0.0f (and the leaf indices):
//   k_rows   up to 64 rows a workgroup, a row's trees spread over its lanes
//            and waves (compact forms): any size, row length and alignment
//   k_score  256 rows a workgroup, a lane walks every tree of its row
//            (32-bit node words): large batches, and ensembles with
//            thresholds above six bits, of 28, 44 or 48 feature quads (GEMM
//            and conv2d loop-context rows, relation rows)
#include <algorithm>

#include "at_chain.h"

namespace at {
namespace {

using namespace dev;

constexpr int SWG = 256;

// ==========================================================================
// k_rows.  A workgroup scores R rows (a power of two up to 64).  Their
// features sit in a 64-column byte tile at LDS address 0 (byte (f & 3) of
// dword (f >> 2) * 64 + column holds 4x+3, x clamped to [0, 63]; column l
// holds row l % R), so every lane reads its own bank.  The trees pass through
// two LDS buffers in chunks; while chunk k is walked, its successor is on
// its way (direct-to-LDS loads of every wave) and wave 0 folds the leaf
// values of chunk k - 1, one lane per row.  One barrier a chunk.
//
// A walk lane takes row lane % R and four consecutive trees of the chunk.
// TAIL: only levels 0 .. d-2 are streamed (local_top) and the last level
// with its leaf comes from the tree's 16-byte tail record; else whole trees
// (local_full).
//
// One lane a row (k_score, the only way before) leaves the chip idle below
// some 200 K rows: every row's trees are one lane's chain of dependent LDS
// reads.  Here the chain is a chunk's walk, then the fold's dependent adds.
// Measured, calls one after another (one lane a row -> this): 64 rows x 500
// trees of depth 8 on 176 features 111 -> 8 us; 4099 rows of the same 130 ->
// 14; 20011 rows x 500 trees on 110 features 230 -> 33; 65537 rows x 1000
// trees 236 -> 156 (169 for a launch the card is idle before).
// Small batches are bound by the fold (500 adds at about 9 clocks each) and
// the stream of the tree tops; large ones by the tail gathers (64 lanes take
// 64 clocks of a compute unit's address path per tree) and the LDS reads.
// ==========================================================================
struct RowsArgs {
    const int32_t* feats;
    int64_t n;
    float* scores;
    uint16_t* leaves;         // or null
    int accumulate;
    int F;
    int quads;                // ceil(F / 4)
    int vec;                  // rows are 16-byte aligned
    int R;                    // rows per workgroup
    int T;
    int ct;                   // trees per chunk, a multiple of 4
    int n_chunks;
    const uint32_t* tw;       // local form, a tree every local_stride words
    const uint4* tail;
    uint32_t off_ring, ring_bytes;
    uint32_t off_lv;
    int lv_stride;            // floats per row of leaf values
};

template <int DEPTH, bool TAIL>
__global__ __launch_bounds__(1024) void k_rows(RowsArgs a) {
    constexpr int WALK = TAIL ? DEPTH - 1 : DEPTH;
    constexpr uint32_t TB = (uint32_t)local_stride(DEPTH, TAIL) * 4u;
    constexpr uint32_t NBB = 4u << (DEPTH - 1);   // node block bytes of a whole tree
    extern __shared__ uint4 lds4[];
    uint8_t* lds = reinterpret_cast<uint8_t*>(lds4);
    uint32_t* tile = reinterpret_cast<uint32_t*>(lds);
    // 0: the kernel has no static LDS (checked at the launch)
    const uint32_t lbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)lds;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nthreads = (int)blockDim.x;
    const int R = a.R;
    const int64_t r0 = (int64_t)blockIdx.x * R;
    const int nr = (a.n - r0 < R) ? (int)(a.n - r0) : R;

    auto load_chunk = [&](int k) {
        const int t0 = k * a.ct;
        const int nt = a.T - t0 < a.ct ? a.T - t0 : a.ct;
        const int n16 = (nt * (int)TB + 15) >> 4;   // the forms end in 16 bytes of slack
        const uint4* src = reinterpret_cast<const uint4*>(a.tw + (size_t)t0 * (TB / 4u));
        uint4* d = reinterpret_cast<uint4*>(lds + a.off_ring + (uint32_t)(k & 1) * a.ring_bytes);
        for (int base = wave * 64; base < n16; base += nthreads)
            if (base + lane < n16) __builtin_amdgcn_global_load_lds(src + base + lane, d + base, 16, 0, 0);
    };
    load_chunk(0);
    // the tile: a wave takes min(R, 16) rows x 64 / min(R, 16) quads at a
    // time, so that its loads cover whole lines and its stores spread over
    // the banks; rows past the end repeat the last one
    {
        const int rg = R < 16 ? R : 16, qg = 64 / rg;
        const int groups = R / rg, qgroups = (a.quads + qg - 1) / qg;
        const int nw = nthreads >> 6;
        for (int task = wave; task < groups * qgroups; task += nw) {
            const int j = (task % groups) * rg + lane % rg, q = (task / groups) * qg + lane / rg;
            if (q >= a.quads) continue;
            const int32_t* f = a.feats + (r0 + (j < nr ? j : nr - 1)) * a.F + 4 * q;
            int4 v;
            if (a.vec) {
                v = *reinterpret_cast<const int4*>(f);
            } else {
                const int left = a.F - 4 * q;
                v.x = f[0];
                v.y = left > 1 ? f[1] : 0;
                v.z = left > 2 ? f[2] : 0;
                v.w = left > 3 ? f[3] : 0;
            }
            auto b = [](int x) { return (uint32_t)min(max(x, 0), (int)NODE_THR_MAX); };
            const uint32_t w = ((b(v.x) | (b(v.y) << 8) | (b(v.z) << 16) | (b(v.w) << 24)) << 2) | 0x03030303u;
            for (int c = j; c < 64; c += R) tile[q * 64 + c] = w;
        }
    }
    const uint32_t fb = lbase | (uint32_t)lane * 4u;
    const int jr = lane & (R - 1);
    const int u = (tid - 64) / R;                 // tree slot of a walk lane
    float acc = 0.0f;
    for (int it = 0; it <= a.n_chunks; ++it) {
        // this wave's part of chunk `it` has landed, then everyone's
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        if (it + 1 < a.n_chunks) load_chunk(it + 1);
        if (wave == 0) {
            if (it > 0 && lane < R) {
                const int t0 = (it - 1) * a.ct;
                const float* row = reinterpret_cast<const float*>(lds + a.off_lv) +
                                   (((it - 1) & 1) * R + lane) * a.lv_stride;
                acc = fold_row(acc, row, a.T - t0 < a.ct ? a.T - t0 : a.ct);
            }
        } else if (it < a.n_chunks) {
            const int t0 = it * a.ct;
            const int nt = a.T - t0 < a.ct ? a.T - t0 : a.ct;
            if (4 * u < nt) {
                uint32_t nb[4], q[4], v[4];
                const uint32_t rb = lbase + a.off_ring + (uint32_t)(it & 1) * a.ring_bytes;
                // (a last group's missing trees repeat its first)
#pragma unroll
                for (int g = 0; g < 4; ++g) nb[g] = rb + (uint32_t)(4 * u + (4 * u + g < nt ? g : 0)) * TB;
                walk4_local<(WALK > 0 ? WALK : 1)>(nb, fb, q);
                if constexpr (TAIL) {
                    uint4 rec[4];
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        rec[g] = a.tail[((size_t)(t0 + 4 * u + (4 * u + g < nt ? g : 0)) << WALK) + q[g]];
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const uint32_t node = rec[g].x;
                        const uint32_t x4 = lds[((node & LOCAL_TILE_MASK) | fb) - lbase];
                        const bool right = x4 >= (node & 0xffu);
                        v[g] = right ? rec[g].z : rec[g].y;
                        q[g] = 2u * q[g] + (right ? 1u : 0u);
                    }
                } else {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        v[g] = *reinterpret_cast<const uint32_t*>(lds + (nb[g] - lbase) + NBB + 4u * q[g]);
                }
                float* lv = reinterpret_cast<float*>(lds + a.off_lv) + ((it & 1) * R + jr) * a.lv_stride + 4 * u;
                *reinterpret_cast<float4*>(lv) = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]),
                                                             __uint_as_float(v[2]), __uint_as_float(v[3]));
                if (a.leaves && jr < nr) {
                    uint16_t* o = a.leaves + (r0 + jr) * a.T + t0 + 4 * u;
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        if (4 * u + g < nt) o[g] = (uint16_t)q[g];
                }
            }
        }
    }
    if (wave == 0 && lane < nr) a.scores[r0 + lane] = a.accumulate ? a.scores[r0 + lane] + acc : acc;
}

// ==========================================================================
// k_score: 256 rows a workgroup on the 32-bit node words.
// ==========================================================================

// Four features, on any 4-byte boundary.
struct __attribute__((packed, aligned(4))) Quad {
    int x, y, z, w;
};

template <int DEPTH> struct ScoreShape {
    static constexpr int W = 2 << DEPTH;                       // words per tree
    static constexpr int CW = DEPTH <= 10 ? 2048 : (DEPTH == 11 ? 4096 : 8192);   // words per chunk
    static constexpr int CT = CW / W;                          // trees per chunk
    static constexpr int G = CT < 4 ? CT : 4;                  // trees walked together
    static constexpr int PER = CW / 4 / SWG;                   // 16-byte pieces per thread
};

template <int DEPTH, int GR, bool LEAVES>
__device__ __forceinline__ void walk_add(const uint8_t* L, uint32_t off, uint32_t fb, float& acc, uint16_t* lrow,
                                         int t_global) {
    uint32_t lw[GR], li[GR];
    walk_pair<DEPTH, GR>(L, off, fb, lw, li);
#pragma unroll
    for (int g = 0; g < GR; ++g) {
        acc = acc + __uint_as_float(lw[g]);
        // lanes past the last row have no output row (lrow is null)
        if (LEAVES && lrow) lrow[t_global + g] = (uint16_t)li[g];
    }
}

// walks r (< 2*H) remaining trees of a partial chunk in groups of H, H/2, ..., 1
template <int DEPTH, int H, bool LEAVES>
__device__ __forceinline__ void walk_add_rest(const uint8_t* L, int t, int r, uint32_t fb, float& acc,
                                              uint16_t* lrow, int t0) {
    constexpr uint32_t TB = (2u << DEPTH) * 4u;
    if (r >= H) {
        walk_add<DEPTH, H, LEAVES>(L, (uint32_t)t * TB, fb, acc, lrow, t0 + t);
        t += H;
        r -= H;
    }
    if constexpr (H > 1) walk_add_rest<DEPTH, H / 2, LEAVES>(L, t, r, fb, acc, lrow, t0);
}

// SQ: feature quads of a row (28, 44 or 48); accumulate: add the score to the
// value already in scores (fp32, that value first) instead of storing it.
// Bytes past the last feature are never read.
template <int DEPTH, bool LEAVES, int SQ>
__global__ __launch_bounds__(SWG) void k_score(EnsembleDesc e, const int32_t* __restrict__ feats, int64_t n,
                                               float* __restrict__ scores, uint16_t* __restrict__ leaves,
                                               int accumulate) {
    using S = ScoreShape<DEPTH>;
    constexpr uint32_t TB = (uint32_t)S::W * 4u;
    __shared__ uint32_t lds[S::CW + SQ * SWG];
    const uint8_t* L = reinterpret_cast<const uint8_t*>(lds);
    uint4* chunk4 = reinterpret_cast<uint4*>(lds);
    uint32_t* tile = lds + S::CW;
    const int tid = threadIdx.x;
    const int64_t row = (int64_t)blockIdx.x * SWG + tid;
    const uint4* src = reinterpret_cast<const uint4*>(e.words);

    const int F = e.n_features;
    // (the arguments in one round trip)
    asm volatile("" ::"s"(F), "s"(feats), "s"(n), "s"(src));
    // first chunk in flight while the feature rows are packed into the tile
    uint32_t pre[S::PER * 4];
#pragma unroll
    for (int u = 0; u < S::PER; ++u) {
        const uint4 x = src[tid + u * SWG];
        pre[4 * u] = x.x; pre[4 * u + 1] = x.y; pre[4 * u + 2] = x.z; pre[4 * u + 3] = x.w;
    }
    {
        // A wave packs its 64 rows, 16 at a time: a load takes four quads of
        // each, 64 bytes in one piece (rows are 4-byte aligned), and the next
        // 16 rows are on their way while these are packed.  Rows past the end
        // repeat the last row; their results are not stored.  With a lane on
        // each row a load touched 64 lines, which left the first-level cache
        // before their next piece was asked for, in three forms by the rows'
        // alignment: 2^20 rows of 192 features x 200 trees of depth 6 took
        // 358 us against 317, of 176 x 500 of depth 8 874 against 834, of 110
        // x 100 of depth 4 199 against 92.
        constexpr int QG = SQ / 4;
        const int lane = tid & 63, q0 = lane >> 4;
        auto byte = [](int x) { return (uint32_t)min(max(x, 0), 255); };
        // a row that ends within its last quad gives its last four features
        // there, moved down to their places
        const int last = min(16 * (QG - 1) + 4 * q0, F - 4) - 4 * q0, down = 8 * (16 * (QG - 1) - last);
        Quad v[2][QG];
        auto load = [&](int rg) {
            const int64_t at = (int64_t)blockIdx.x * SWG + (tid & ~63) + rg * 16 + (lane & 15);
            const int32_t* fr = feats + (at < n ? at : n - 1) * F + 4 * q0;
#pragma unroll
            for (int g = 0; g + 1 < QG; ++g) v[rg & 1][g] = *reinterpret_cast<const Quad*>(fr + 16 * g);
            v[rg & 1][QG - 1] = *reinterpret_cast<const Quad*>(fr + last);
        };
        load(0);
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            if (rg + 1 < 4) load(rg + 1);
            asm volatile("" ::: "memory");
            uint32_t* d = tile + q0 * SWG + (tid & ~63) + rg * 16 + (lane & 15);
#pragma unroll
            for (int g = 0; g < QG; ++g) {
                const Quad& x = v[rg & 1][g];
                const uint32_t w = byte(x.x) | (byte(x.y) << 8) | (byte(x.z) << 16) | (byte(x.w) << 24);
                d[4 * g * SWG] = g + 1 < QG ? w : w >> down;
            }
        }
    }
    const uint32_t fb = (uint32_t)S::CW * 4u + (uint32_t)tid * 4u;
    uint16_t* lrow = (LEAVES && row < n) ? leaves + row * e.n_trees : nullptr;
    float acc = 0.0f;
    const int nchunks = (e.n_trees + S::CT - 1) / S::CT;
    for (int k = 0; k < nchunks; ++k) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < S::PER; ++u)
            chunk4[tid + u * SWG] = make_uint4(pre[4 * u], pre[4 * u + 1], pre[4 * u + 2], pre[4 * u + 3]);
        __syncthreads();
        // next chunk (the last one is fetched again on the final pass; the
        // packed ensemble is padded so every fetch stays in bounds)
        const int kn = (k + 1 < nchunks) ? k + 1 : k;
        const uint4* s4 = src + (size_t)kn * (S::CW / 4);
#pragma unroll
        for (int u = 0; u < S::PER; ++u) {
            const uint4 x = s4[tid + u * SWG];
            pre[4 * u] = x.x; pre[4 * u + 1] = x.y; pre[4 * u + 2] = x.z; pre[4 * u + 3] = x.w;
        }
        const int t0 = k * S::CT;
        const int nt = (e.n_trees - t0 < S::CT) ? e.n_trees - t0 : S::CT;
        if (nt == S::CT) {
#pragma unroll 4
            for (int t = 0; t < S::CT; t += S::G)
                walk_add<DEPTH, S::G, LEAVES>(L, (uint32_t)t * TB, fb, acc, lrow, t0 + t);
        } else {
            int t = 0;
            for (; t + S::G <= nt; t += S::G)
                walk_add<DEPTH, S::G, LEAVES>(L, (uint32_t)t * TB, fb, acc, lrow, t0 + t);
            if constexpr (S::G > 1) walk_add_rest<DEPTH, S::G / 2, LEAVES>(L, t, nt - t, fb, acc, lrow, t0);
        }
    }
    if (row < n) scores[row] = accumulate ? scores[row] + acc : acc;
}

template <int DEPTH, int SQ>
hipError_t score_q(const EnsembleDesc& e, const int32_t* feats, int64_t n, float* scores, uint16_t* leaves,
                   bool accumulate, hipStream_t stream) {
    const unsigned grid = (unsigned)((n + SWG - 1) / SWG);
    if (leaves)
        hipLaunchKernelGGL((k_score<DEPTH, true, SQ>), dim3(grid), dim3(SWG), 0, stream, e, feats, n, scores, leaves,
                           accumulate ? 1 : 0);
    else
        hipLaunchKernelGGL((k_score<DEPTH, false, SQ>), dim3(grid), dim3(SWG), 0, stream, e, feats, n, scores, leaves,
                           accumulate ? 1 : 0);
    return hipGetLastError();
}

template <int DEPTH>
hipError_t score_depth(const EnsembleDesc& e, const int32_t* feats, int64_t n, float* scores, uint16_t* leaves,
                       bool accumulate, hipStream_t stream) {
    switch ((e.n_features + 3) / 4) {
        case 28: return score_q<DEPTH, 28>(e, feats, n, scores, leaves, accumulate, stream);
        case 44: return score_q<DEPTH, 44>(e, feats, n, scores, leaves, accumulate, stream);
        case 48: return score_q<DEPTH, 48>(e, feats, n, scores, leaves, accumulate, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_score_wide(const EnsembleDesc& e, const int32_t* feats, int64_t n, float* scores, uint16_t* leaves,
                             bool accumulate, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    switch (e.depth) {
        case 1: return score_depth<1>(e, feats, n, scores, leaves, accumulate, stream);
        case 2: return score_depth<2>(e, feats, n, scores, leaves, accumulate, stream);
        case 3: return score_depth<3>(e, feats, n, scores, leaves, accumulate, stream);
        case 4: return score_depth<4>(e, feats, n, scores, leaves, accumulate, stream);
        case 5: return score_depth<5>(e, feats, n, scores, leaves, accumulate, stream);
        case 6: return score_depth<6>(e, feats, n, scores, leaves, accumulate, stream);
        case 7: return score_depth<7>(e, feats, n, scores, leaves, accumulate, stream);
        case 8: return score_depth<8>(e, feats, n, scores, leaves, accumulate, stream);
        case 9: return score_depth<9>(e, feats, n, scores, leaves, accumulate, stream);
        case 10: return score_depth<10>(e, feats, n, scores, leaves, accumulate, stream);
        case 11: return score_depth<11>(e, feats, n, scores, leaves, accumulate, stream);
        case 12: return score_depth<12>(e, feats, n, scores, leaves, accumulate, stream);
        default: return hipErrorInvalidValue;
    }
}

namespace {

// Dynamic LDS a scoring workgroup may use: the compute unit's 160 KB less 1 KB
// (no static LDS, as the launch checks).
constexpr size_t SCORE_LDS_BYTES = 163840 - 1024;

struct RowsPlan {
    bool tail = false;
    int R = 0, ct = 0, waves = 0;
    size_t lds = 0;
};

// LDS layout of a plan; false when it takes more than `limit` bytes.
bool rows_layout(const EnsembleDesc& e, RowsPlan& pl, RowsArgs& a, size_t limit) {
    const uint32_t tb = (uint32_t)local_stride(e.depth, pl.tail) * 4u;
    a.quads = (e.n_features + 3) / 4;
    a.tw = pl.tail ? e.local_top : e.local_full;
    a.R = pl.R;
    a.ct = pl.ct;
    a.n_chunks = (e.n_trees + pl.ct - 1) / pl.ct;
    a.off_ring = (uint32_t)a.quads * 256u;
    a.ring_bytes = ((uint32_t)pl.ct * tb + 15u) / 16u * 16u;
    a.off_lv = a.off_ring + (a.n_chunks > 1 ? 2u : 1u) * a.ring_bytes;
    // 16-byte rows an odd number of 16-byte units apart (LDS banks)
    a.lv_stride = 4 * (pl.ct / 4 | 1);
    pl.lds = a.off_lv + (size_t)(a.n_chunks > 1 ? 2 : 1) * pl.R * a.lv_stride * 4;
    return pl.lds <= limit;
}

// Plan of k_rows.  The lines lie where a sweep of rows a workgroup, waves,
// chunk and form (n 16 .. 300000, depths 4 .. 10, 100 .. 1500 trees, 110 and
// 176 features) put them; over it the plans are within 5 % of the best in the
// geometric mean, and further off just past a line (below).
//  - Rows a workgroup: 8 up to 2048 rows (a workgroup streams the whole
//    ensemble, so fewer rows a workgroup only repeat that), then doubled, up
//    to 32, until 256 workgroups at most are left; 64 when even so the chip
//    is full several times over (above 24576 rows; above 12288 for deep
//    trees, whose streaming costs more).  Just past a line half the compute
//    units have no workgroup, or each has two of half the LDS (500 trees of
//    depth 8 on 176 features, us, with leaf indices in brackets): 2048 rows
//    9.1 (10.0), 2049 9.8 (12.3); 4096 11.1 (13.9), 4097 14.3 (19.1); 8192
//    14.8 (23.2), 8193 21.1 (25.4); 24576 32.3 (53.6), 24577 37.7 (79.1).
//  - Up to one workgroup a compute unit: 16 waves and all of its LDS; more:
//    12 waves and half of it, 8 waves from 98304 rows (500 trees of depth 8
//    on 176 features, 4099 rows: 14.3 us with 16 waves, 17.4 with 6; 131072
//    rows: 143 us with 8 or 12, 157 with 4).
//  - Tails from depth 5: they stream a sixth of a whole tree's bytes, so more
//    trees and workgroups fit (65537 rows x 1000 trees of depth 8: 158 us
//    against 219); below, the tail gathers cost more than the leaves.
bool plan_rows(const EnsembleDesc& e, int64_t n, RowsPlan& pl, RowsArgs& a) {
    pl.tail = e.depth >= 5;
    pl.R = 8;
    while (pl.R < 32 && n > (int64_t)256 * pl.R) pl.R *= 2;
    if (n > (e.depth >= 9 ? 12288 : 24576)) pl.R = 64;
    const bool one = (n + pl.R - 1) / pl.R <= 256;
    pl.waves = one ? 16 : (n < 98304 ? 12 : 8);
    const size_t limit = one ? SCORE_LDS_BYTES : SCORE_LDS_BYTES / 2;
    const int want = (e.n_trees + 3) / 4 * 4, per_wave = 256 / pl.R;
    const int cap = (pl.waves - 1) * per_wave;
    pl.ct = want < cap ? want : cap;
    while (pl.ct >= 4 && !rows_layout(e, pl, a, limit)) pl.ct -= 4;
    if (pl.ct < 4) return false;
    // chunks of one size; waves that a single chunk leaves without trees go
    const int chunks = a.n_chunks;
    pl.ct = ((e.n_trees + chunks - 1) / chunks + 3) / 4 * 4;
    if (chunks == 1) pl.waves = std::min(pl.waves, std::max(4, 1 + (pl.ct + per_wave - 1) / per_wave));
    return rows_layout(e, pl, a, limit);
}

template <int DEPTH>
hipError_t rows_depth(const RowsPlan& pl, const RowsArgs& a, hipStream_t stream) {
    static std::atomic<uint64_t> done[2];
    constexpr bool TAILS = DEPTH >= 2;
    const bool tail = TAILS && pl.tail;
    const void* fn = tail ? reinterpret_cast<const void*>(&k_rows<DEPTH, TAILS>)
                          : reinterpret_cast<const void*>(&k_rows<DEPTH, false>);
    // the walks address the tile with an and-or, which needs the dynamic LDS
    // block at address 0: no static LDS in the kernel
    hipError_t e = prepare_kernel(fn, 0, SCORE_LDS_BYTES, done[tail]);
    if (e != hipSuccess) return e;
    void* args[] = {const_cast<RowsArgs*>(&a)};
    return hipLaunchKernel(fn, dim3((unsigned)((a.n + pl.R - 1) / pl.R)), dim3(pl.waves * 64), args, pl.lds, stream);
}

// Whether a call that both kernels take goes to k_score.  The lines come from
// both kernels' times at 16385 .. 262144 rows of 110, 176 and 192 features,
// depths 2 .. 9, 20 .. 400 trees (us, k_rows -> k_score, 176 features):
//  - Scores.  k_rows' time grows with the rows, k_score's with the workgroups
//    a compute unit has (a step every 65536 rows), and the fewer and
//    shallower the trees the more of either is the rows' load, which k_score
//    does in fewer passes.  20 trees of depth 5: 40001 rows 10 -> 8, 131072 26
//    -> 17; 60 of depth 6: 49153 rows 15 -> 14; 400 of depth 6: 81921 rows 73
//    -> 77, 98305 79 -> 78; 400 of depth 8: 114689 rows 109 -> 115, 180001
//    152 -> 147.  Deeper trees leave a lane one or two trees in flight (depth
//    10, 131072 rows: 237 -> 307).
//  - With leaf indices: k_rows' lanes store eight bytes of a row at a time,
//    all over the rows of a workgroup, which costs more than the walk from 64
//    rows a workgroup (24577 rows) on; a k_score lane goes along its own row.
//    131072 rows x 100 trees of depth 4 75 -> 34, x 250 of depth 8 171 ->
//    114; 150 of depth 8: 32769 rows 35 -> 41, 49153 47 -> 44; 150 of depth 9:
//    131072 rows 120 -> 94, 180001 160 -> 169.
bool one_lane_a_row(const EnsembleDesc& e, int64_t n, bool leaves) {
    const int quads = (e.n_features + 3) / 4, d = e.depth;
    if ((quads != 28 && quads != 44 && quads != 48) || d > 9) return false;
    const int64_t work = (int64_t)e.n_trees * d * d;
    if (leaves) {
        if (d <= 6) return n >= 24577;
        if (d == 7 || (d == 8 && work <= 4000)) return n >= 32769;
        if (d == 8) return n >= 45057;
        return work <= 2000 ? n >= 65537 : n >= 81921 && n <= 131072;
    }
    if (d == 9) return work <= 4000 && n >= (work <= 2000 ? 65537 : 98305);
    if (work <= 1600) return n >= 32769;
    if (work <= 4000 && d <= 7) return n >= 49153;
    if (d <= 6 || work <= 4000 || (d == 7 && work <= 8000)) return n >= 98305;
    if (d == 7 || work <= 10000) return n >= 114689;
    return n >= 131072;
}

}  // namespace

hipError_t launch_score(const EnsembleDesc& e, const int32_t* feats, int64_t n, float* scores, uint16_t* leaves,
                        bool accumulate, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    // A launch holds at most 2^32 threads, and k_rows takes four to 128 a
    // row: larger calls are cut into pieces (2^28 rows keep a piece's rows as
    // aligned as the call's).
    constexpr int64_t PIECE = (int64_t)1 << 28;
    for (; n > PIECE; n -= PIECE) {
        const hipError_t err = launch_score(e, feats, PIECE, scores, leaves, accumulate, stream);
        if (err != hipSuccess) return err;
        feats += PIECE * e.n_features;
        scores += PIECE;
        if (leaves) leaves += PIECE * e.n_trees;
    }
    const bool vec = e.n_features % 4 == 0 && (reinterpret_cast<uintptr_t>(feats) & 15u) == 0;
    RowsPlan pl;
    RowsArgs a{};
    if (one_lane_a_row(e, n, leaves != nullptr))
        return launch_score_wide(e, feats, n, scores, leaves, accumulate, stream);
    if (!plan_rows(e, n, pl, a)) return hipErrorInvalidConfiguration;
    a.feats = feats;
    a.n = n;
    a.scores = scores;
    a.leaves = leaves;
    a.accumulate = accumulate ? 1 : 0;
    a.F = e.n_features;
    a.vec = vec ? 1 : 0;
    a.T = e.n_trees;
    a.tail = e.tail;
    switch (e.depth) {
        case 1: return rows_depth<1>(pl, a, stream);
        case 2: return rows_depth<2>(pl, a, stream);
        case 3: return rows_depth<3>(pl, a, stream);
        case 4: return rows_depth<4>(pl, a, stream);
        case 5: return rows_depth<5>(pl, a, stream);
        case 6: return rows_depth<6>(pl, a, stream);
        case 7: return rows_depth<7>(pl, a, stream);
        case 8: return rows_depth<8>(pl, a, stream);
        case 9: return rows_depth<9>(pl, a, stream);
        case 10: return rows_depth<10>(pl, a, stream);
        case 11: return rows_depth<11>(pl, a, stream);
        case 12: return rows_depth<12>(pl, a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace at
