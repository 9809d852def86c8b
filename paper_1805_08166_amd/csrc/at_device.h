// Device helpers shared by the HIP kernels: loop-context feature evaluation
// of the two schedule templates, the tree walk over LDS-resident node words,
// and best-list insertion.
#pragma once

#include "at_internal.h"

namespace at {
namespace dev {

constexpr int WG = 256;   // workgroup size of every kernel (4 wave64s)

// bitlen(x): bits needed to write x (0 for 0).
__device__ __forceinline__ uint32_t bitlen(uint32_t x) { return 32u - (uint32_t)__clz((int)x); }

// bitlen(floor(a / b)) for a >= b >= 1 without a division: with
// k = bitlen(a) - bitlen(b) >= 0 the quotient lies in [2^(k-1), 2^(k+1)),
// and it reaches 2^k exactly when floor(a / 2^k) >= b.
__device__ __forceinline__ uint32_t bitlen_quot(uint32_t a, uint32_t b) {
    uint32_t k = bitlen(a) - bitlen(b);
    return k + ((a >> k) >= b ? 1u : 0u);
}

// Distinct values of S*x + y for x over A consecutive integers and y over B
// consecutive integers: one run of (A-1)*S + B when the windows touch
// (B >= S, or a single x), else A*B isolated windows.
__device__ __forceinline__ uint32_t distinct_affine(uint32_t A, uint32_t B, uint32_t S) {
    return (A == 1u || B >= S) ? (A - 1u) * S + B : A * B;
}

// --------------------------------------------------------------------------
// Loop nests of the two templates, outer to inner.  Axis ids: GEMM i=0 j=1
// k=2; conv oc=0 oh=1 ow=2 rc=3 ry=4 rx=5.  FUSED marks the kernel-window
// loop r_l = (ry_l outer, rx_l inner).  Binding ids follow the annotation
// column: 3/4/5 blockIdx.x/y/z, 6/7/8 threadIdx.x/y/z, 0 serial.  The
// spatial axes (the first SPATIAL) are those whose third tiling level a
// vthread knob binds to virtual threads (id 9); a vectorize knob marks the
// innermost loop vectorized (id 10).
// --------------------------------------------------------------------------
constexpr int FUSED = -1;
constexpr uint32_t ANN_VTHREAD = 9u, ANN_VECTORIZE = 10u;
constexpr int ANN_KINDS = 12;   // one-hot annotation columns (ids 0 .. 11)

template <int TMPL> struct Nest;

template <> struct Nest<AT_TMPL_GEMM> {
    static constexpr int L = 10;
    static constexpr int F = 110;
    static constexpr int axis[L] = {0, 1, 0, 1, 2, 0, 1, 2, 0, 1};
    static constexpr int level[L] = {0, 0, 1, 1, 0, 2, 2, 1, 3, 3};
    static constexpr int bind[L] = {4, 3, 7, 6, 0, 0, 0, 0, 0, 0};
    static constexpr int SPATIAL = 2;
    // touch counts from the per-axis ranges of a sub-nest
    __device__ static void touched(const uint32_t (&r)[6], uint32_t, uint32_t (&t)[3]) {
        t[0] = r[2] * r[0];   // A[k][i]
        t[1] = r[2] * r[1];   // B[k][j]
        t[2] = r[0] * r[1];   // C[i][j]
    }
};

template <> struct Nest<AT_TMPL_CONV2D_NCHW> {
    static constexpr int L = 16;
    static constexpr int F = 176;
    static constexpr int axis[L] = {0, 1, 2, 0, 1, 2, 3, FUSED, 0, 1, 2, 3, FUSED, 0, 1, 2};
    static constexpr int level[L] = {0, 0, 0, 1, 1, 1, 0, 0, 2, 2, 2, 1, 1, 3, 3, 3};
    static constexpr int bind[L] = {5, 4, 3, 8, 7, 6, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    static constexpr int SPATIAL = 3;
    __device__ static void touched(const uint32_t (&r)[6], uint32_t S, uint32_t (&t)[3]) {
        // data_pad[rc][oh*S+ry][ow*S+rx], unclipped padded coordinates
        t[0] = r[3] * distinct_affine(r[1], r[4], S) * distinct_affine(r[2], r[5], S);
        t[1] = r[0] * r[3] * r[4] * r[5];   // kernel[oc][rc][ry][rx]
        t[2] = r[0] * r[1] * r[2];          // output[oc][oh][ow]
    }
};

// Annotation id of loop p: its thread or block binding, else virtual
// threads (vth set, third level of a spatial axis), else vectorized (vec set,
// innermost loop), else unrolled (id unroll_id) when auto_unroll_max_step is
// on and its sub-nest has at most that many iterations, else serial.
template <int TMPL>
__device__ __forceinline__ uint32_t annotation_of(int p, uint32_t bottom_up, uint32_t unroll_max, uint32_t unroll_id,
                                                  uint32_t vec, uint32_t vth) {
    using N = Nest<TMPL>;
    if (N::bind[p]) return (uint32_t)N::bind[p];
    if (vth && N::level[p] == 2 && N::axis[p] >= 0 && N::axis[p] < N::SPATIAL) return ANN_VTHREAD;
    if (vec && p == N::L - 1) return ANN_VECTORIZE;
    return (unroll_max > 0u && bottom_up <= unroll_max) ? unroll_id : 0u;
}

// The annotation knobs of configuration kv: auto_unroll_max_step,
// unroll_explicit (id 1 or 2 for unrolled loops) and, for the annotated
// templates, vectorize and vthread.
struct AnnKnobs {
    uint32_t unroll_max, unroll_id, vec, vth;
};
template <int TMPL>
__device__ __forceinline__ AnnKnobs ann_knobs_of(const SpaceDesc& sd, const uint32_t (&kv)[MAX_KNOBS]) {
    constexpr int A = (TMPL == AT_TMPL_GEMM) ? 3 : 6;
    AnnKnobs k;
    k.unroll_max = kv[A] == 0u ? 0u : (kv[A] == 1u ? 512u : 1500u);
    k.unroll_id = 1u + kv[A + 1];
    k.vec = sd.ann_knobs ? kv[A + 2] : 0u;
    k.vth = sd.ann_knobs ? kv[A + 3] : 0u;
    return k;
}

// Factors of the chosen split of axis a: four 16-bit fields, outer level first.
__device__ __forceinline__ void unpack_split(uint64_t w, uint32_t (&f)[4]) {
    f[0] = (uint32_t)(w & 0xffff);
    f[1] = (uint32_t)((w >> 16) & 0xffff);
    f[2] = (uint32_t)((w >> 32) & 0xffff);
    f[3] = (uint32_t)(w >> 48);
}

// Loop-context features of one schedule.  The nest is walked from the
// innermost loop outwards so that each loop's sub-nest quantities are running
// products: range[a] is the extent of axis a covered by the sub-nest, and a
// loop's stride in buffer b is b's weight of the loop's axis times the range
// of that axis strictly inside the loop.  emit(f, value) receives feature f.
// PER = 13 gives the full rows of Appendix A.2: bitlen(top-down) and
// bitlen(bottom-up) follow the annotation.  Top-down is the nest's iteration
// count (the product of every factor, below 2^31 for any space) divided by
// bottom-up, the quotient's bitlen taken without a division.  PER = 24 gives
// the full rows with the annotation one-hot: ANN_KINDS columns, 1 at the
// loop's annotation id, 0 elsewhere.  Only loops LO .. HI-1 are emitted (the
// loops inside them take part in the products alone).
template <int TMPL, int PER = 11, int LO = 0, int HI = Nest<TMPL>::L, class Emit>
__device__ __forceinline__ void nest_features(const SpaceDesc& sd, const uint32_t (&fac)[6][4], const AnnKnobs& ak,
                                              Emit&& emit) {
    static_assert(PER == 11 || PER == 13 || PER == 24, "loop-context rows, full rows or one-hot rows");
    using N = Nest<TMPL>;
    constexpr int HOT = PER == 24 ? ANN_KINDS : 1;          // annotation columns
    constexpr int B0 = 1 + HOT + (PER == 11 ? 0 : 2);       // first buffer column
    uint32_t range[6] = {1u, 1u, 1u, 1u, 1u, 1u};
    uint32_t bottom_up = 1u;
    const uint32_t S = (uint32_t)sd.stride;
    uint32_t total = 1u;
    if constexpr (PER != 11) {
#pragma unroll
        for (int a = 0; a < 6; ++a)
#pragma unroll
            for (int l = 0; l < 4; ++l) total *= fac[a][l];
    }
#pragma unroll
    for (int p = N::L - 1; p >= LO; --p) {
        uint32_t ext, strd[3];
        if (N::axis[p] == FUSED) {
            const int l = N::level[p];
            const uint32_t fy = fac[4][l], fx = fac[5][l];
            ext = fy * fx;
            // one step of r moves rx when rx has several values, else ry
#pragma unroll
            for (int b = 0; b < 3; ++b)
                strd[b] = (fx > 1u) ? (uint32_t)sd.coef[b][5] * range[5] : (uint32_t)sd.coef[b][4] * range[4];
            range[4] *= fy;
            range[5] *= fx;
        } else {
            const int a = N::axis[p];
            ext = fac[a][N::level[p]];
#pragma unroll
            for (int b = 0; b < 3; ++b) strd[b] = (uint32_t)sd.coef[b][a] * range[a];
            range[a] *= ext;
        }
        bottom_up *= ext;
        if (p >= HI) continue;
        uint32_t t[3];
        N::touched(range, S, t);
        const uint32_t ann = annotation_of<TMPL>(p, bottom_up, ak.unroll_max, ak.unroll_id, ak.vec, ak.vth);
        emit(p * PER + 0, bitlen(ext));
        if constexpr (PER == 24) {
#pragma unroll
            for (int h = 0; h < ANN_KINDS; ++h) emit(p * PER + 1 + h, ann == (uint32_t)h ? 1u : 0u);
        } else {
            emit(p * PER + 1, ann);
        }
        if constexpr (PER != 11) {
            emit(p * PER + 1 + HOT, bitlen_quot(total, bottom_up));
            emit(p * PER + 2 + HOT, bitlen(bottom_up));
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            emit(p * PER + B0 + 3 * b, bitlen(t[b]));
            emit(p * PER + B0 + 1 + 3 * b, bitlen_quot(bottom_up, t[b]));
            emit(p * PER + B0 + 2 + 3 * b, bitlen(strd[b]));
        }
    }
}

// Per-loop tables for loop_features, two or three bits a loop in one word:
// the outermost level of axis a at or inside loop p (levels outside p are
// those whose loop comes before it), and loop p's axis (5 for a fused loop).
template <int TMPL>
__host__ __device__ constexpr int levels_outside(int a, int p) {
    using N = Nest<TMPL>;
    int c = 0;
    for (int q = 0; q < p; ++q) c += (N::axis[q] == a || (N::axis[q] == FUSED && a >= 4)) ? 1 : 0;
    return c;
}
template <int TMPL>
__host__ __device__ constexpr uint32_t level_table(int a) {
    uint32_t t = 0;
    for (int p = 0; p < Nest<TMPL>::L; ++p) {
        const int l = levels_outside<TMPL>(a, p);
        t |= (uint32_t)(l < 3 ? l : 3) << (2 * p);
    }
    return t;
}
// bit p: every level of axis a lies outside loop p
template <int TMPL>
__host__ __device__ constexpr uint32_t outside_table(int a) {
    uint32_t t = 0;
    for (int p = 0; p < Nest<TMPL>::L; ++p) t |= (levels_outside<TMPL>(a, p) == 4 ? 1u : 0u) << p;
    return t;
}
template <int TMPL>
__host__ __device__ constexpr uint64_t axis_table() {
    uint64_t t = 0;
    for (int p = 0; p < Nest<TMPL>::L; ++p) {
        const int a = Nest<TMPL>::axis[p] == FUSED ? 5 : Nest<TMPL>::axis[p];
        t |= (uint64_t)a << (3 * p);
    }
    return t;
}

// The loop-context features of loop p alone (out[0..10]) of the configuration
// with knob values kv, for evaluating one schedule with one lane per loop.
// The same quantities as nest_features, from the split choices' suffix
// products (sfx: field l of a choice is the product of its factors at levels
// l and inside): the range of axis a at or inside loop p is the field of its
// outermost level there, and the range strictly inside p the next field of
// p's own axis, so every quantity is a few reads and a product of ranges
// (below 2^16 each, so pairs multiply in 24 bits).  Walking the nest and
// multiplying the loops up, as before, cost some 80 full 32-bit products a
// loop, at a quarter of the other instructions' rate.  bitlen(length) is the
// bitlen of the exact quotient of the two ranges.  td receives, when asked
// for, bitlen(top-down): the nest's iteration count over bottom-up.
template <int TMPL>
__device__ __forceinline__ void loop_features(const SpaceDesc& sd, const uint64_t* __restrict__ sfx,
                                              const uint32_t (&kv)[MAX_KNOBS], int p, uint32_t (&out)[11],
                                              uint32_t& td, bool want_td) {
    using N = Nest<TMPL>;
    constexpr bool CONV = TMPL == AT_TMPL_CONV2D_NCHW;
    constexpr int A = CONV ? 6 : 3;
    const uint16_t* f16 = reinterpret_cast<const uint16_t*>(sfx);
    // field index of each axis's range, and the ranges
    uint32_t at[A], r[6] = {1u, 1u, 1u, 1u, 1u, 1u};
#pragma unroll
    for (int a = 0; a < A; ++a) {
        at[a] = 4u * ((uint32_t)sd.split_off[a] + kv[a]) + ((level_table<TMPL>(a) >> (2 * p)) & 3u);
        r[a] = f16[at[a]];
        const uint32_t inner = outside_table<TMPL>(a);   // the loops inside every level of axis a: range 1
        if (inner != 0u) r[a] = ((inner >> p) & 1u) ? 1u : r[a];
    }
    // loop p's own axis: its range at and strictly inside p (1 inside the
    // innermost of four levels; both axes for a fused loop)
    const uint32_t ax = (uint32_t)(axis_table<TMPL>() >> (3 * p)) & 7u;
    uint32_t own = at[0], rown = r[0];
#pragma unroll
    for (int a = 1; a < A; ++a) {
        own = ax == (uint32_t)a ? at[a] : own;
        rown = ax == (uint32_t)a ? r[a] : rown;
    }
    uint32_t rin = 1u;
    if ((own & 3u) != 3u) rin = f16[own + 1u];
    uint32_t incl = rown, excl = rin, axs = ax, inside = rin;
    if constexpr (CONV) {
        const bool fused = ax == 5u;
        const uint32_t rin4 = f16[at[4] + (fused ? 1u : 0u)];   // read by every lane, used by fused loops
        incl = fused ? __umul24(r[4], r[5]) : rown;
        excl = fused ? __umul24(rin4, rin) : rin;
        // one step of a fused loop moves rx when rx has several values, else ry
        const bool ry = fused && rown == rin;
        axs = ry ? 4u : ax;
        inside = ry ? rin4 : rin;
    }
    const uint32_t r01 = __umul24(r[0], r[1]);
    uint32_t bottom_up, t[3], total = 1u;
    if constexpr (CONV) {
        const uint32_t r45 = __umul24(r[4], r[5]), r23 = __umul24(r[2], r[3]);
        bottom_up = r01 * r23 * r45;
        const uint32_t S = (uint32_t)sd.stride;
        auto distinct = [&](uint32_t x, uint32_t y) {
            return (x == 1u || y >= S) ? __umul24(x - 1u, S) + y : __umul24(x, y);
        };
        t[0] = r[3] * distinct(r[1], r[4]) * distinct(r[2], r[5]);
        t[1] = __umul24(r[0], r[3]) * r45;
        t[2] = r01 * r[2];
    } else {
        bottom_up = r01 * r[2];
        t[0] = __umul24(r[2], r[0]);
        t[1] = __umul24(r[2], r[1]);
        t[2] = r01;
    }
    td = 0u;
    if (want_td) {
        // field 0 of any choice of an axis is its extent
#pragma unroll
        for (int a = 0; a < A; ++a) total *= (uint32_t)f16[4u * (uint32_t)sd.split_off[a]];
        td = bitlen_quot(total, bottom_up);
    }
    out[0] = bitlen_quot(incl, excl);
    // annotation: binding, virtual threads, vectorized, unrolled, serial
    {
        const AnnKnobs ak = ann_knobs_of<TMPL>(sd, kv);
        uint64_t binds = 0;
        uint32_t vthr = 0;
#pragma unroll
        for (int q = 0; q < N::L; ++q) {
            binds |= (uint64_t)N::bind[q] << (4 * q);
            vthr |= (N::level[q] == 2 && N::axis[q] >= 0 && N::axis[q] < N::SPATIAL ? 1u : 0u) << q;
        }
        const uint32_t bind = (uint32_t)(binds >> (4 * p)) & 15u;
        uint32_t ann = (ak.unroll_max > 0u && bottom_up <= ak.unroll_max) ? ak.unroll_id : 0u;
        if (ak.vec && p == N::L - 1) ann = ANN_VECTORIZE;
        if (ak.vth && ((vthr >> p) & 1u)) ann = ANN_VTHREAD;
        out[1] = bind ? bind : ann;
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        out[2 + 3 * b] = bitlen(t[b]);
        out[3 + 3 * b] = bitlen_quot(bottom_up, t[b]);
        out[4 + 3 * b] = bitlen((uint32_t)sd.coef[b][axs] * inside);
    }
}

// Context relation features of one buffer (thresholds t = 1 .. 32): byte t-1
// of w0 is the largest ru(p), of w1 the largest td(p), over the loops p with
// tc(p) <= t; tc, ru and td give the bitlens of loop p's touch count, reuse
// ratio and top-down product.  A sub-nest touches no fewer elements than any
// sub-nest inside it, so the loops a threshold admits are the innermost ones
// from some loop p* on, and each maximum is a suffix maximum (over p* and
// the loops inside it).  Visiting the loops from the innermost outwards,
// loop p writes its suffix maxima into every threshold it admits; the
// outermost admitted loop, p*, writes last.  Four thresholds share a word:
// byte j of word w is t = 4w + 1 + j, admitted when j >= tc(p) - 1 - 4w.
constexpr int REL_T = 32;
constexpr int REL_NW = REL_T / 4;
template <int L, class Tc, class Ru, class Td>
__device__ __forceinline__ void relation_maxima(Tc&& tc, Ru&& ru, Td&& td, uint32_t (&w0)[REL_NW],
                                                uint32_t (&w1)[REL_NW]) {
#pragma unroll
    for (int w = 0; w < REL_NW; ++w) w0[w] = w1[w] = 0u;
    uint32_t s0 = 0u, s1 = 0u;
#pragma unroll
    for (int p = L - 1; p >= 0; --p) {
        s0 = max(s0, ru(p));
        s1 = max(s1, td(p));
        const int t = (int)tc(p);
        const uint32_t b0 = s0 * 0x01010101u, b1 = s1 * 0x01010101u;
#pragma unroll
        for (int w = 0; w < REL_NW; ++w) {
            const int kb = min(max(t - 1 - 4 * w, 0), 4);
            const uint32_t m = (uint32_t)(0xffffffffull << (8 * kb));
            w0[w] = (b0 & m) | (w0[w] & ~m);
            w1[w] = (b1 & m) | (w1[w] & ~m);
        }
    }
}

// Factors of every axis for knob values kv (split knob a = axis a).
template <int TMPL>
__device__ __forceinline__ void gather_factors(const SpaceDesc& sd, const uint64_t* __restrict__ factors,
                                               const uint32_t (&kv)[MAX_KNOBS], uint32_t (&fac)[6][4]) {
    constexpr int A = (TMPL == AT_TMPL_GEMM) ? 3 : 6;
#pragma unroll
    for (int a = 0; a < 6; ++a) {
        if (a < A) unpack_split(factors[sd.split_off[a] + kv[a]], fac[a]);
        else fac[a][0] = fac[a][1] = fac[a][2] = fac[a][3] = 1u;
    }
}

// Copies `words` packed tree words (a multiple of 4) from global to LDS.
__device__ __forceinline__ void stage_words(uint32_t* __restrict__ dst, const uint32_t* __restrict__ src,
                                            int words) {
    const uint4* s4 = reinterpret_cast<const uint4*>(src);
    uint4* d4 = reinterpret_cast<uint4*>(dst);
    for (int i = threadIdx.x; i < words / 4; i += WG) d4[i] = s4[i];
}

// Walks GROUP trees of depth DEPTH starting at chunk word `cb` (tree stride
// W words) for the lane whose feature column starts at byte `fb` of the
// tile; returns the leaf words and leaf indices.
template <int DEPTH, int GROUP>
__device__ __forceinline__ void walk(const uint32_t* __restrict__ chunk, const uint8_t* __restrict__ tile_b,
                                     uint32_t fb, int cb, uint32_t (&leafw)[GROUP], uint32_t (&leafi)[GROUP]) {
    constexpr int W = 2 << DEPTH;
    uint32_t m[GROUP];
#pragma unroll
    for (int g = 0; g < GROUP; ++g) m[g] = 1u;
#pragma unroll
    for (int l = 0; l < DEPTH; ++l) {
        uint32_t node[GROUP];
#pragma unroll
        for (int g = 0; g < GROUP; ++g) node[g] = chunk[cb + g * W + m[g]];
#pragma unroll
        for (int g = 0; g < GROUP; ++g) {
            const uint32_t x = tile_b[fb + (node[g] & 0xffffu)];
            m[g] = 2u * m[g] + (x >= (node[g] >> 16) ? 1u : 0u);
        }
    }
#pragma unroll
    for (int g = 0; g < GROUP; ++g) {
        leafw[g] = chunk[cb + g * W + m[g]];
        leafi[g] = m[g] - (1u << DEPTH);
    }
}

// Walks GROUP trees whose words start at byte tree_off (tree stride 4*W
// bytes) of the LDS block L, for the row whose feature column starts at byte
// fb of L.  One LDS round trip per level: the current node's feature byte and
// the pair of its children (words 2m, 2m+1, bytes 8m..8m+7) are read
// together and the child is then selected; at the last level the pair holds
// two leaves.  Returns the leaf words and leaf indices.
template <int DEPTH, int GROUP>
__device__ __forceinline__ void walk_pair(const uint8_t* __restrict__ L, uint32_t tree_off, uint32_t fb,
                                          uint32_t (&leafw)[GROUP], uint32_t (&leafi)[GROUP]) {
    constexpr uint32_t TB = (2u << DEPTH) * 4u;
    uint32_t node[GROUP], a[GROUP];
#pragma unroll
    for (int g = 0; g < GROUP; ++g) {
        node[g] = *reinterpret_cast<const uint32_t*>(L + tree_off + g * TB + 4u);
        a[g] = 8u;
    }
#pragma unroll
    for (int l = 0; l < DEPTH; ++l) {
        uint32_t x[GROUP];
        uint2 pr[GROUP];
#pragma unroll
        for (int g = 0; g < GROUP; ++g) {
            x[g] = L[fb + (node[g] & 0xffffu)];
            pr[g] = *reinterpret_cast<const uint2*>(L + tree_off + g * TB + a[g]);
        }
#pragma unroll
        for (int g = 0; g < GROUP; ++g) {
            const bool right = x[g] >= (node[g] >> 16);
            node[g] = right ? pr[g].y : pr[g].x;
            a[g] = 2u * a[g] + (right ? 8u : 0u);
        }
    }
#pragma unroll
    for (int g = 0; g < GROUP; ++g) {
        leafw[g] = node[g];
        leafi[g] = (a[g] >> 3) - (1u << DEPTH);
    }
}

}  // namespace dev
}  // namespace at
