// HIP kernels for gfx950 (CDNA4): loop-context features, tree-ensemble
// scoring and parallel simulated annealing.
//
// Nothing here is a dense contraction, so there is no MFMA: the features are
// integer bookkeeping bound by HBM writes, and the tree walk is a chain of
// dependent LDS gathers bound by LDS and VALU issue.
//
// Exactness: features are integers; a score is the fp32 sum of the reached
// leaves added one tree after another in tree order from +0.0f, exactly as
// the model defines it, so every kernel reproduces it bit for bit.  The
// library is compiled with -ffp-contract=off.
#include "at_device.h"

namespace at {
namespace {

using namespace dev;

// ==========================================================================
// Feature extraction.  A workgroup of four waves makes the rows of 64
// configurations, lane r of every wave configuration r: the waves share out
// the knobs when the indices are decoded (split factors and annotation
// knobs go through LDS), then the loops of the nest (a wave's loops are
// known at compile time, and the products over the loops inside them are
// cheap), and the finished rows, signed bytes in LDS, leave as int32 with
// consecutive lanes covering consecutive 16-byte pieces of the block.
//
// Bound by HBM writes at large sizes and by its own latency at small ones.
// One configuration a lane and 256 a workgroup left both a longer serial
// chain and, with up to 99 KB of LDS a workgroup, too few workgroups to keep
// the stores going: 200003 conv2d rows took 33.8 us in the 208-column form
// and 75.7 in the 384-column one against 29.2 and 51.7 (5.7 and 5.9 TB/s),
// one buffer written again and again, part of it still in the cache behind
// the L2s; the two forms in turn, 473 MB, take 34.4 and 58.8.  2^20 rows of
// 176 take 143 us, the rate of sustained writes.  Non-temporal stores
// measured 62 us on the 384-column rows.
// ==========================================================================
constexpr int ROWS = 64;               // configurations per workgroup
constexpr int WAVES = WG / 64;

// PER columns per loop: 11 (loop-context rows), 13 (full Appendix A.2 rows
// with top-down and bottom-up) or 24 (full rows with a one-hot annotation).
// A row in LDS takes RS bytes: an odd number of dwords, so that the lanes'
// stores spread over the banks, or, when its length is no multiple of four,
// just its F bytes, so that the block is one flat byte array.
template <int TMPL, int PER = 11>
struct RowLayout {
    static constexpr int F = Nest<TMPL>::L * PER;
    static constexpr bool FLAT = F % 4 != 0;
    static constexpr int RS = FLAT ? F : (F / 4 | 1) * 4;
};

// The block of 64 rows a workgroup makes.  Workgroups go round the eight XCDs
// in turn; for outputs past the 256 MB cache behind the L2s an XCD takes runs
// of 16 blocks, so that it writes longer pieces of memory: 2^20 conv2d rows of
// 208 columns 171.5 -> 165.7 us, of 176 146.8 -> 141.6, 1500001 of 384 432 ->
// 413 (runs of 4: 167.9, 144.8, 418; of 64: 165.4, 143.1, 411); below, the
// written lines leave the caches in the order of the rows and runs cost
// (200003 rows of 384, 307 MB: 51.3 -> 54.8).
constexpr unsigned RUN = 16;
constexpr int64_t RUN_BYTES = (int64_t)320 << 20;

__device__ __forceinline__ int64_t row_block(int runs) {
    const unsigned b = blockIdx.x, whole = gridDim.x / (8u * RUN) * (8u * RUN);
    if (!runs || b >= whole) return b;
    const unsigned xcd = b % 8u, i = b / 8u;
    return (int64_t)(i / RUN * 8u + xcd) * RUN + i % RUN;
}

// Split factors and annotation knobs of a workgroup's configurations.
struct Decoded {
    uint64_t fac[MAX_AXES][ROWS];
    uint8_t ann[ROWS][4];              // auto_unroll_max_step, unroll_explicit, vectorize, vthread
};

// Decodes configuration base + lane (mixed radix, knob 0 most significant;
// indices and weights fit 32 bits), wave w taking knobs w, w + 4, ....
// Returns whether the lane's index is out of range (decoded as index 0).
template <int TMPL>
__device__ __forceinline__ bool decode_rows(const SpaceDesc& sd, const uint64_t* __restrict__ factors,
                                            const uint64_t* __restrict__ cfgs, int64_t base, int64_t n, int wave,
                                            int lane, Decoded& s) {
    constexpr int A = (TMPL == AT_TMPL_GEMM) ? 3 : 6;
    const int64_t row = base + lane < n ? base + lane : n - 1;
    const uint64_t cfg64 = cfgs[row];
    const bool bad = cfg64 >= sd.n_configs;
    const uint32_t cfg = bad ? 0u : (uint32_t)cfg64;
    for (int j = wave; j < sd.n_knobs; j += WAVES) {
        const uint32_t rad = (uint32_t)sd.radix[j], size = sd.knob_size[j];
        const uint32_t q = cfg / rad;
        const uint32_t kv = q - q / size * size;
        if (j < A) s.fac[j][lane] = factors[sd.split_off[j] + kv];
        else s.ann[lane][j - A] = (uint8_t)kv;
    }
    return bad;
}

// Factors and annotation knobs of row r.
template <int TMPL>
__device__ __forceinline__ AnnKnobs decoded_row(const SpaceDesc& sd, const Decoded& s, int r, uint32_t (&fac)[6][4]) {
    constexpr int A = (TMPL == AT_TMPL_GEMM) ? 3 : 6;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        if (a < A) unpack_split(s.fac[a][r], fac[a]);
        else fac[a][0] = fac[a][1] = fac[a][2] = fac[a][3] = 1u;
    }
    uint32_t kv[MAX_KNOBS];
#pragma unroll
    for (int j = 0; j < MAX_KNOBS; ++j) kv[j] = (j >= A && j < A + 4) ? s.ann[r][j >= A && j < A + 4 ? j - A : 0] : 0u;
    return ann_knobs_of<TMPL>(sd, kv);
}

// Loops LO .. HI-1 of a row into its place in LDS.
template <int TMPL, int PER, int LO, int HI>
__device__ __forceinline__ void emit_loops(const SpaceDesc& sd, const uint32_t (&fac)[6][4], const AnnKnobs& ak,
                                           uint8_t* my) {
    using RL = RowLayout<TMPL, PER>;
    if constexpr (RL::FLAT) {
        nest_features<TMPL, PER, LO, HI>(sd, fac, ak, [&](int f, uint32_t v) { my[f] = (uint8_t)v; });
    } else {
        static_assert(LO * PER % 4 == 0 && HI * PER % 4 == 0, "whole dwords a wave");
        constexpr int F0 = LO * PER, NW = (HI - LO) * PER / 4;
        uint32_t w[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) w[i] = 0u;
        nest_features<TMPL, PER, LO, HI>(sd, fac, ak,
                                         [&](int f, uint32_t v) { w[(f - F0) >> 2] |= v << (8 * ((f - F0) & 3)); });
        uint32_t* d = reinterpret_cast<uint32_t*>(my + F0);
#pragma unroll
        for (int i = 0; i < NW; ++i) d[i] = w[i];
    }
}

__device__ __forceinline__ int4 widen(uint32_t w) {
    return make_int4((int)(int8_t)(w & 0xffu), (int)(int8_t)((w >> 8) & 0xffu), (int)(int8_t)((w >> 16) & 0xffu),
                     (int)(int8_t)(w >> 24));
}

// The block's rows (rows_here of them, F bytes each, RS apart) to out.
template <int F, int RS>
__device__ __forceinline__ void store_rows(const uint8_t* rows, int32_t* __restrict__ out, int rows_here, bool vec,
                                           int tid, int threads) {
    const int total = rows_here * F;
    if (vec) {
        for (int g = tid; g < total / 4; g += threads) {
            int at = 4 * g;
            if constexpr (F != RS) at = g / (F / 4) * RS + g % (F / 4) * 4;
            reinterpret_cast<int4*>(out)[g] = widen(*reinterpret_cast<const uint32_t*>(rows + at));
        }
        if constexpr (F % 4 != 0)
            for (int e = total / 4 * 4 + tid; e < total; e += threads) out[e] = (int32_t)(int8_t)rows[e];
    } else {
        for (int e = tid; e < total; e += threads) out[e] = (int32_t)(int8_t)rows[e / F * RS + e % F];
    }
}

// vec: feats is 16-byte aligned
template <int TMPL, int PER>
__global__ __launch_bounds__(WG) void k_extract(SpaceDesc sd, const uint64_t* __restrict__ factors,
                                                const uint64_t* __restrict__ cfgs, int64_t n,
                                                int32_t* __restrict__ feats,
                                                unsigned long long* __restrict__ n_bad, int vec, int runs) {
    using RL = RowLayout<TMPL, PER>;
    constexpr int F = RL::F, RS = RL::RS, L = Nest<TMPL>::L;
    __shared__ __attribute__((aligned(16))) uint8_t rows[ROWS * RS];
    __shared__ Decoded s;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int64_t base = row_block(runs) * ROWS;
    const int rows_here = n - base < ROWS ? (int)(n - base) : ROWS;
    const bool bad = decode_rows<TMPL>(sd, factors, cfgs, base, n, wave, lane, s);
    __syncthreads();
    {
        uint8_t* my = rows + lane * RS;
        uint32_t fac[6][4];
        const AnnKnobs ak = decoded_row<TMPL>(sd, s, lane, fac);
        switch (wave) {
            case 0: emit_loops<TMPL, PER, 0, L / 4>(sd, fac, ak, my); break;
            case 1: emit_loops<TMPL, PER, L / 4, L / 2>(sd, fac, ak, my); break;
            case 2: emit_loops<TMPL, PER, L / 2, L * 3 / 4>(sd, fac, ak, my); break;
            default: emit_loops<TMPL, PER, L * 3 / 4, L>(sd, fac, ak, my); break;
        }
    }
    __syncthreads();
    // out-of-range rows: -1 throughout, counted once
    const bool mine = bad && lane < rows_here;
    if (__ballot(mine)) {
        if (wave == 0 && mine) atomicAdd(n_bad, 1ull);
        if (mine)
            for (int f = wave; f < F; f += WAVES) rows[lane * RS + f] = 0xff;
        __syncthreads();
    }
    store_rows<F, RS>(rows, feats + base * F, rows_here, vec != 0, tid, WG);
}

// ==========================================================================
// Context relation features (Section 4; Appendix A.2).  Per buffer b and t =
// 1..REL_T, over the loops whose sub-nest touches fewer than 2^t elements of
// b (bitlen(touch) <= t):
//   R[0][b][t-1] = the largest bitlen(reuse ratio),
//   R[1][b][t-1] = the largest bitlen(top-down product of the outer lengths),
// 0 when no loop qualifies.  The workgroup makes 64 rows as k_extract does;
// each wave's loop quantities go through LDS, then wave b < 3 makes the
// maxima of buffer b.
// ==========================================================================
constexpr int REL_F = RELATION_FEATURES;
constexpr int REL_RS = REL_F + 4;           // 49 dwords per LDS row

template <int TMPL>
__global__ __launch_bounds__(WG) void k_relation(SpaceDesc sd, const uint64_t* __restrict__ factors,
                                                 const uint64_t* __restrict__ cfgs, int64_t n,
                                                 int32_t* __restrict__ feats, unsigned long long* __restrict__ n_bad,
                                                 int runs) {
    using N = Nest<TMPL>;
    constexpr int L = N::L;
    __shared__ __attribute__((aligned(16))) uint8_t rows[ROWS * REL_RS];
    __shared__ Decoded s;
    __shared__ uint8_t tc[3][L][ROWS], ru[3][L][ROWS], td[L][ROWS];   // bitlens of touch, reuse, top-down
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int64_t base = row_block(runs) * ROWS;
    const int rows_here = n - base < ROWS ? (int)(n - base) : ROWS;
    const bool bad = decode_rows<TMPL>(sd, factors, cfgs, base, n, wave, lane, s);
    __syncthreads();
    {
        uint32_t fac[6][4];
        const AnnKnobs ak = decoded_row<TMPL>(sd, s, lane, fac);
        auto keep = [&](int f, uint32_t v) {
            const int p = f / 13, c = f - p * 13;
            if (c == 2) td[p][lane] = (uint8_t)v;
            if (c >= 4 && (c - 4) % 3 == 0) tc[(c - 4) / 3][p][lane] = (uint8_t)v;
            if (c >= 4 && (c - 4) % 3 == 1) ru[(c - 4) / 3][p][lane] = (uint8_t)v;
        };
        switch (wave) {
            case 0: nest_features<TMPL, 13, 0, L / 4>(sd, fac, ak, keep); break;
            case 1: nest_features<TMPL, 13, L / 4, L / 2>(sd, fac, ak, keep); break;
            case 2: nest_features<TMPL, 13, L / 2, L * 3 / 4>(sd, fac, ak, keep); break;
            default: nest_features<TMPL, 13, L * 3 / 4, L>(sd, fac, ak, keep); break;
        }
    }
    __syncthreads();
    if (wave < 3) {
        const int b = wave;
        uint32_t w0[REL_NW], w1[REL_NW];
        relation_maxima<L>([&](int p) { return (uint32_t)tc[b][p][lane]; },
                           [&](int p) { return (uint32_t)ru[b][p][lane]; },
                           [&](int p) { return (uint32_t)td[p][lane]; }, w0, w1);
        if (bad) {
#pragma unroll
            for (int w = 0; w < REL_NW; ++w) w0[w] = w1[w] = 0xffffffffu;
            if (b == 0 && lane < rows_here) atomicAdd(n_bad, 1ull);
        }
        // rows are dword aligned (REL_RS = 196 bytes) and so is each 32-byte block
        uint32_t* d0 = reinterpret_cast<uint32_t*>(rows + lane * REL_RS + (0 * 3 + b) * REL_T);
        uint32_t* d1 = reinterpret_cast<uint32_t*>(rows + lane * REL_RS + (1 * 3 + b) * REL_T);
#pragma unroll
        for (int w = 0; w < REL_NW; ++w) {
            d0[w] = w0[w];
            d1[w] = w1[w];
        }
    }
    __syncthreads();
    store_rows<REL_F, REL_RS>(rows, feats + base * REL_F, rows_here, true, tid, WG);
}

// ==========================================================================
// Tree-ensemble traversal shared by scoring and annealing.
// A workgroup holds the features of its 256 rows (chains or candidates) in
// an LDS tile and streams the packed trees through LDS in chunks.  Each lane
// walks every tree for its own row and adds the leaves in tree order.
// ==========================================================================

// Scores the row in this lane's tile column against every tree; all lanes
// of the workgroup must call it together (it stages chunks with barriers).
template <int DEPTH>
__device__ __forceinline__ float score_tile(const EnsembleDesc& e, const uint32_t* __restrict__ tile, uint32_t* __restrict__ chunk,
                            int chunk_trees, uint16_t* __restrict__ leaves_row) {
    constexpr int W = 2 << DEPTH;
    constexpr int G = 4;
    const uint8_t* tile_b = reinterpret_cast<const uint8_t*>(tile);
    const uint32_t fb = threadIdx.x * 4u;
    float acc = 0.0f;
    for (int t0 = 0; t0 < e.n_trees; t0 += chunk_trees) {
        const int nt = (e.n_trees - t0 < chunk_trees) ? (e.n_trees - t0) : chunk_trees;
        __syncthreads();
        stage_words(chunk, e.words + (size_t)t0 * W, nt * W);
        __syncthreads();
        int t = 0;
        for (; t + G <= nt; t += G) {
            uint32_t lw[G], li[G];
            walk<DEPTH, G>(chunk, tile_b, fb, t * W, lw, li);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                acc = acc + __uint_as_float(lw[g]);
                if (leaves_row) leaves_row[t0 + t + g] = (uint16_t)li[g];
            }
        }
        for (; t < nt; ++t) {
            uint32_t lw[1], li[1];
            walk<DEPTH, 1>(chunk, tile_b, fb, t * W, lw, li);
            acc = acc + __uint_as_float(lw[0]);
            if (leaves_row) leaves_row[t0 + t] = (uint16_t)li[0];
        }
    }
    return acc;
}

// Trees per LDS chunk: the largest count whose words fit `bytes`.
__host__ __device__ inline int chunk_trees_for(int depth, int bytes) {
    int w = 2 << depth;
    int t = bytes / (w * 4);
    return t < 1 ? 1 : t;
}

constexpr int CHUNK_BYTES = 32768;

template <int DEPTH>
__global__ __launch_bounds__(WG) void k_predict(EnsembleDesc e, const int32_t* __restrict__ feats, int64_t n,
                                                float* __restrict__ scores, uint16_t* __restrict__ leaves,
                                                int chunk_trees, int accumulate) {
    extern __shared__ uint32_t lds[];
    const int Q = (e.n_features + 3) / 4;
    uint32_t* tile = lds;
    uint32_t* chunk = lds + Q * WG;
    const int tid = threadIdx.x;
    const int64_t row = (int64_t)blockIdx.x * WG + tid;
    const int F = e.n_features;
    // own row -> tile column, 4 features per dword, clamped to [0, 255]
    for (int q = 0; q < Q; ++q) {
        uint32_t w = 0;
        if (row < n) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int f = q * 4 + k;
                if (f < F) {
                    int x = feats[row * F + f];
                    x = x < 0 ? 0 : (x > 255 ? 255 : x);
                    w |= (uint32_t)x << (8 * k);
                }
            }
        }
        tile[q * WG + tid] = w;
    }
    uint16_t* lrow = (leaves && row < n) ? leaves + row * e.n_trees : nullptr;
    const float s = score_tile<DEPTH>(e, tile, chunk, chunk_trees, lrow);
    if (row < n) scores[row] = accumulate ? scores[row] + s : s;
}

__global__ __launch_bounds__(WG) void k_export(const SpaceDesc* descs, const int64_t* offsets, int n_spaces,
                                               const uint16_t* knobs, const float* score, int64_t n,
                                               uint64_t* cur_cfg, float* cur_score) {
    const int64_t c = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (c >= n) return;
    int w = 0;
    while (w + 1 < n_spaces && offsets[w + 1] <= c) ++w;
    const SpaceDesc& sd = descs[w];
    if (cur_cfg) {
        uint64_t x = 0;
        for (int j = 0; j < sd.n_knobs; ++j) x += (uint64_t)knobs[c * MAX_KNOBS + j] * sd.radix[j];
        cur_cfg[c] = x;
    }
    if (cur_score) cur_score[c] = score[c];
}

// ==========================================================================
// Which loop-context features are constant over a space.  Every
// configuration index below n is visited (grid-stride loop, one per lane);
// flags[f] becomes 1 when some configuration's feature f differs from that
// of configuration 0, and workgroup 0 writes configuration 0's row to ref.
// A feature left unflagged therefore takes one value over the whole space.
// ==========================================================================
template <int TMPL>
__global__ __launch_bounds__(WG) void k_feature_scan(SpaceDesc sd, const uint64_t* __restrict__ factors, uint64_t n,
                                                     uint32_t* __restrict__ flags, uint32_t* __restrict__ ref_out) {
    constexpr int F = RowLayout<TMPL>::F;
    __shared__ uint32_t ref[F];
    __shared__ uint32_t diff[F];
    const int tid = threadIdx.x;
    auto row_of = [&](uint64_t cfg, auto&& put) {
        // mixed radix, knob 0 most significant (indices below n fit 32 bits)
        uint32_t rest = (uint32_t)cfg;
        uint32_t kv[MAX_KNOBS];
#pragma unroll
        for (int j = MAX_KNOBS - 1; j >= 0; --j) {
            if (j < sd.n_knobs) {
                const uint32_t sz = sd.knob_size[j];
                const uint32_t q = rest / sz;
                kv[j] = rest - q * sz;
                rest = q;
            } else {
                kv[j] = 0u;
            }
        }
        uint32_t fac[6][4];
        gather_factors<TMPL>(sd, factors, kv, fac);
        nest_features<TMPL, 11>(sd, fac, ann_knobs_of<TMPL>(sd, kv), put);
    };
    for (int f = tid; f < F; f += WG) diff[f] = 0u;
    if (tid == 0) row_of(0, [&](int f, uint32_t v) { ref[f] = v; });
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * WG;
    for (uint64_t cfg = (uint64_t)blockIdx.x * WG + tid; cfg < n; cfg += stride)
        row_of(cfg, [&](int f, uint32_t v) {
            if (v != ref[f]) diff[f] = 1u;
        });
    __syncthreads();
    for (int f = tid; f < F; f += WG) {
        if (diff[f]) flags[f] = 1u;
        if (blockIdx.x == 0) ref_out[f] = ref[f];
    }
}

}  // namespace

namespace {

template <class T>
struct Same {
    using type = T;
};

// A launch without the compiler's launch stub, which pushes and pops the
// launch's shape and copies every argument once more: a call on a few rows is
// bound by the host (two calls on 64 GEMM rows, medians of three processes:
// 16.2 -> 14.4 us).
template <class... A>
hipError_t launch_rows(void (*kern)(A...), unsigned grid, hipStream_t stream, const typename Same<A>::type&... args) {
    void* ptrs[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), dim3(grid), dim3(WG), ptrs, 0, stream);
}

template <int PER>
hipError_t extract_per(const at_space_s& sp, const uint64_t* cfgs, int64_t n, int32_t* feats, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const unsigned grid = (unsigned)((n + ROWS - 1) / ROWS);
    const uint64_t* fac = static_cast<const uint64_t*>(sp.d_factors.p);
    auto* bad = static_cast<unsigned long long*>(sp.d_errors.p);
    const int vec = (reinterpret_cast<uintptr_t>(feats) & 15u) == 0 ? 1 : 0;
    const int runs = n * (sp.descs[0].n_features / 11 * PER) * 4 > RUN_BYTES ? 1 : 0;
    auto kern = sp.tmpl == AT_TMPL_GEMM ? k_extract<AT_TMPL_GEMM, PER> : k_extract<AT_TMPL_CONV2D_NCHW, PER>;
    return launch_rows(kern, grid, stream, sp.descs[0], fac, cfgs, n, feats, bad, vec, runs);
}

}  // namespace

hipError_t launch_extract(const at_space_s& sp, const uint64_t* cfgs, int64_t n, int32_t* feats,
                          hipStream_t stream) {
    return extract_per<11>(sp, cfgs, n, feats, stream);
}

hipError_t launch_extract_full(const at_space_s& sp, const uint64_t* cfgs, int64_t n, int32_t* feats,
                               hipStream_t stream) {
    return extract_per<13>(sp, cfgs, n, feats, stream);
}

hipError_t launch_extract_onehot(const at_space_s& sp, const uint64_t* cfgs, int64_t n, int32_t* feats,
                                 hipStream_t stream) {
    return extract_per<24>(sp, cfgs, n, feats, stream);
}

hipError_t launch_relation(const at_space_s& sp, const uint64_t* cfgs, int64_t n, int32_t* feats,
                           hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const unsigned grid = (unsigned)((n + ROWS - 1) / ROWS);
    const uint64_t* fac = static_cast<const uint64_t*>(sp.d_factors.p);
    auto* bad = static_cast<unsigned long long*>(sp.d_errors.p);
    const int runs = n * REL_F * 4 > RUN_BYTES ? 1 : 0;
    auto kern = sp.tmpl == AT_TMPL_GEMM ? k_relation<AT_TMPL_GEMM> : k_relation<AT_TMPL_CONV2D_NCHW>;
    return launch_rows(kern, grid, stream, sp.descs[0], fac, cfgs, n, feats, bad, runs);
}

namespace {

template <int DEPTH>
hipError_t predict_depth(const EnsembleDesc& e, const int32_t* feats, int64_t n, float* scores, uint16_t* leaves,
                         bool accumulate, hipStream_t stream) {
    const int Q = (e.n_features + 3) / 4;
    const int ct = chunk_trees_for(DEPTH, CHUNK_BYTES);
    const size_t lds = (size_t)Q * WG * 4 + (size_t)ct * (2 << DEPTH) * 4;
    static std::atomic<uint64_t> done;
    const hipError_t err = prepare_kernel(reinterpret_cast<const void*>(&k_predict<DEPTH>), -1,
                                          MAX_TILE_QUADS * WG * 4 + CHUNK_BYTES, done);
    if (err != hipSuccess) return err;
    const unsigned grid = (unsigned)((n + WG - 1) / WG);
    hipLaunchKernelGGL((k_predict<DEPTH>), dim3(grid), dim3(WG), lds, stream, e, feats, n, scores, leaves, ct,
                       accumulate ? 1 : 0);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_predict(const EnsembleDesc& e, const int32_t* feats, int64_t n, float* scores,
                          uint16_t* leaves, bool accumulate, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    // thresholds within six bits: the compact forms, any size and alignment
    if (leaves ? e.leaf6 : e.score6) return launch_score(e, feats, n, scores, leaves, accumulate, stream);
    const int quads = (e.n_features + 3) / 4;
    if (quads == 28 || quads == 44 || quads == 48)
        return launch_score_wide(e, feats, n, scores, leaves, accumulate, stream);
    switch (e.depth) {
        case 1: return predict_depth<1>(e, feats, n, scores, leaves, accumulate, stream);
        case 2: return predict_depth<2>(e, feats, n, scores, leaves, accumulate, stream);
        case 3: return predict_depth<3>(e, feats, n, scores, leaves, accumulate, stream);
        case 4: return predict_depth<4>(e, feats, n, scores, leaves, accumulate, stream);
        case 5: return predict_depth<5>(e, feats, n, scores, leaves, accumulate, stream);
        case 6: return predict_depth<6>(e, feats, n, scores, leaves, accumulate, stream);
        case 7: return predict_depth<7>(e, feats, n, scores, leaves, accumulate, stream);
        case 8: return predict_depth<8>(e, feats, n, scores, leaves, accumulate, stream);
        case 9: return predict_depth<9>(e, feats, n, scores, leaves, accumulate, stream);
        case 10: return predict_depth<10>(e, feats, n, scores, leaves, accumulate, stream);
        case 11: return predict_depth<11>(e, feats, n, scores, leaves, accumulate, stream);
        case 12: return predict_depth<12>(e, feats, n, scores, leaves, accumulate, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_feature_scan(const at_space_s& sp, uint32_t* flags, uint32_t* ref, hipStream_t stream) {
    const SpaceDesc& sd = sp.descs[0];
    const uint64_t n = sd.n_configs;
    if (n == 0) return hipSuccess;
    const uint64_t blocks = (n + WG - 1) / WG;
    const unsigned grid = (unsigned)(blocks < 4096 ? blocks : 4096);
    const uint64_t* fac = static_cast<const uint64_t*>(sp.d_factors.p);
    if (sp.tmpl == AT_TMPL_GEMM)
        hipLaunchKernelGGL(k_feature_scan<AT_TMPL_GEMM>, dim3(grid), dim3(WG), 0, stream, sd, fac, n, flags, ref);
    else
        hipLaunchKernelGGL(k_feature_scan<AT_TMPL_CONV2D_NCHW>, dim3(grid), dim3(WG), 0, stream, sd, fac, n, flags,
                           ref);
    return hipGetLastError();
}

hipError_t launch_export(const at_chains_s& ch, uint64_t* cur_cfg, float* cur_score, hipStream_t stream) {
    if (ch.n_chains == 0) return hipSuccess;
    const unsigned grid = (unsigned)((ch.n_chains + WG - 1) / WG);
    hipLaunchKernelGGL(k_export, dim3(grid), dim3(WG), 0, stream, static_cast<const SpaceDesc*>(ch.d_descs.p),
                       static_cast<const int64_t*>(ch.d_offsets.p), ch.n_spaces,
                       static_cast<const uint16_t*>(ch.d_knobs.p), static_cast<const float*>(ch.d_score.p),
                       ch.n_chains, cur_cfg, cur_score);
    return hipGetLastError();
}

}  // namespace at
