// Parallel simulated annealing (Section 3.3), chain-local, for ensembles that
// stay in one workgroup's LDS and at most four chains per workgroup.
//
// One persistent workgroup owns its chains for the whole run.  Every tree
// (or every tree's top levels, with the last level and its leaves in a
// 16-byte record in global memory) is loaded once, and a scoring round is
// two phases between LDS-only barriers:
//   A  every wave walks: lane (tid % cpb, tid / cpb) takes chain tid % cpb
//      and the trees tid / cpb, + S, ... (S lanes a chain), and writes the
//      reached leaf values to LDS;
//   B  wave 0 folds them, one lane per chain (fp32, from +0.0f, in tree
//      order), and takes the Metropolis decision; beside it waves 1-2 make
//      both candidates that can follow (a move from this round's candidate
//      and one from the configuration the round starts from) with the
//      features of both, wave 3 offers the previous round's candidates to the
//      best lists, wave 4 draws the moves after next and the last wave brings
//      the next thresholds.
// The walk reads a candidate's feature bytes from the row itself (4x+3 per
// byte, feature order), in the row set of the outcome that came true, so
// nothing is copied between the decision and the next walk.
//
// Bound by latency: the fold's dependent adds (about 9 clocks each) and one
// LDS round trip a tree level.  The three-barrier form before, which copied
// the rows into a 64-column tile each round and kept the chains' books in
// wave 0, took 3.76 us a step on the C2 search (1024 chains, 500 trees of
// depth 8) and 2.50 on the GEMM one (64 chains, 100 trees of depth 6); this
// one 3.3 and 1.26.
#include <type_traits>

#include "at_chain.h"

namespace at {
namespace {

using namespace dev;

constexpr int SINGLE_FAC_MAX = 1024;          // split choices staged in LDS
constexpr int SINGLE_CHAINS = 4;              // chains per workgroup at most
constexpr int SINGLE_WIDE_WALKS = 1024;       // tree walks a round above which a workgroup has 1024 threads
// dynamic LDS per workgroup: the compute unit's 160 KB less 1 KB; the launch
// checks that the kernel has no static LDS
constexpr size_t SINGLE_LDS_BYTES = 163840 - 1024;

// One chain's record.  Rounds are numbered from 0 (the initial draw, when
// there is one, is round 0); arrays indexed by round keep the last two or
// four, so that a phase's readers never meet its writers.
struct SingleRec {
    uint64_t cfg;                          // best-list offer in hand (group_offer)
    float score;
    uint32_t count;
    float kth_score;
    uint32_t pad;
    uint64_t kth_cfg;
    uint64_t scfg[4][2];                   // round's two possible candidates: index ...
    uint32_t snx[4][2][MAX_KNOBS / 2];     // ... and knobs in pairs (0: after an accept, 1: after a reject)
    uint32_t ssel[4];                      // which of them is the round's: the outcome of the round before
    uint64_t curcfg[2];                    // the configuration the round starts from
    uint32_t curk[2][MAX_KNOBS / 2];
    uint64_t mvr[2];                       // the round's move: knob weight, knob, value
    int32_t mvj[2];
    uint32_t mvv[2];
    float psc[2];                          // the round's score
    float thr[2];                          // the round's threshold
};

struct SingleArgs {
    const SpaceDesc* descs;
    const int64_t* offsets;
    int n_spaces;
    const uint64_t* suffix;   // split choices as suffix products
    uint16_t* knobs;          // [n][MAX_KNOBS] current configuration
    float* cur_score;         // [n]
    at_entry* top;            // [n][topk] best lists
    ChainMeta* meta;          // [n]
    int topk;
    int cpb;                  // chains per workgroup: 1, 2 or 4
    int64_t n;
    uint64_t chain0;
    uint64_t seed;
    int init;                 // round 0 draws, scores and offers the initial configurations
    int steps;
    uint32_t step0;           // absolute step of local step 0
    const float* thr;         // [n][steps]
    at_entry* trace;          // [n][steps] or null
    at_entry* best;           // [n][topk]
    const uint32_t* tw;       // local form, a tree every local_stride words
    int T;
    const uint4* tail_rec;    // [T][2^(d-1)] records {node, left leaf, right leaf, 0}
    // dynamic LDS layout (byte offsets; the trees are at 0)
    uint32_t off_lv, off_lists, off_rec, off_frow, off_desc;
    int lv_stride;            // floats per chain row of leaf values
    uint32_t frow_stride;     // bytes between row sets: set 2 (r & 1) + o is round r's candidates after outcome o
    int early;                // the evaluating waves do not walk (see k_single)
};

// One level of a tree whose row's features are read from LDS byte rb + f:
// right = (low byte of the node) <= x4, the child's node, the heap index,
// then the next feature address rb + (quad * 4 + byte) and pair address.
// Between a compare and the reads of VCC lie two other instructions (gfx950
// wait states).
#define AT_RL_CMP(i) "v_cmp_le_u32_sdwa vcc, %[n" #i "], %[x" #i "] src0_sel:BYTE_0 src1_sel:DWORD\n\t"
#define AT_RL_SEL(i)                                                                                               \
    "v_cndmask_b32_sdwa %[n" #i "], %[r" #i "], %[r" #i                                                            \
    "], vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_1\n\t"                               \
    "v_addc_co_u32 %[p" #i "], vcc, %[p" #i "], %[p" #i "], vcc\n\t"
#define AT_RL_SH(i)                                                                                                \
    "v_lshrrev_b32 %[f" #i "], 6, %[n" #i "]\n\t"                                                                  \
    "v_lshl_add_u32 %[a" #i "], %[p" #i "], 2, %[b" #i "]\n\t"
#define AT_RL_BF(i) "v_bfi_b32 %[f" #i "], 3, %[n" #i "], %[f" #i "]\n\t"
#define AT_RL_AD(i) "v_add_u32 %[f" #i "], %[f" #i "], %[rb]\n\t"

__device__ __forceinline__ uint32_t row_byte(uint32_t node) { return ((node >> 6) & 0xfcu) | (node & 3u); }

// Node indices at level DEPTH (0 .. 2^DEPTH - 1) of G trees (1, 2 or 4) for
// the row at LDS byte rb; nb: LDS byte addresses of the trees' node blocks.
template <int DEPTH, int G>
__device__ __forceinline__ void walk_row(const uint32_t (&nb)[G], uint32_t rb, uint32_t (&q)[G]) {
    static_assert(G == 1 || G == 2 || G == 4, "trees together");
    uint32_t node[G], p[G], fa[G], pa[G], x[G];
    if constexpr (G == 4)
        asm volatile("ds_read_u16 %0, %4\n\tds_read_u16 %1, %5\n\tds_read_u16 %2, %6\n\tds_read_u16 %3, %7\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(node[0]), "=&v"(node[1]), "=&v"(node[2]), "=&v"(node[3])
                     : "v"(nb[0]), "v"(nb[1]), "v"(nb[2]), "v"(nb[3])
                     : "memory");
    else if constexpr (G == 2)
        asm volatile("ds_read_u16 %0, %2\n\tds_read_u16 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(node[0]), "=&v"(node[1])
                     : "v"(nb[0]), "v"(nb[1])
                     : "memory");
    else
        asm volatile("ds_read_u16 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(node[0]) : "v"(nb[0]) : "memory");
#pragma unroll
    for (int g = 0; g < G; ++g) {
        p[g] = 1u;
        fa[g] = rb + row_byte(node[g]);
        pa[g] = nb[g] + 4u;
    }
#pragma unroll
    for (int l = 0; l + 1 < DEPTH; ++l) {
        uint32_t pr[G];
        if constexpr (G == 4) {
            asm volatile(
                "ds_read_u8 %0, %8\n\tds_read_b32 %4, %12\n\tds_read_u8 %1, %9\n\tds_read_b32 %5, %13\n\t"
                "ds_read_u8 %2, %10\n\tds_read_b32 %6, %14\n\tds_read_u8 %3, %11\n\tds_read_b32 %7, %15\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(pr[0]), "=&v"(pr[1]), "=&v"(pr[2]),
                  "=&v"(pr[3])
                : "v"(fa[0]), "v"(fa[1]), "v"(fa[2]), "v"(fa[3]), "v"(pa[0]), "v"(pa[1]), "v"(pa[2]), "v"(pa[3])
                : "memory");
            asm(AT_RL_CMP(0) "s_nop 1\n\t" AT_RL_SEL(0) AT_RL_CMP(1) AT_RL_SH(0) AT_RL_SEL(1) AT_RL_CMP(2) AT_RL_SH(1)
                    AT_RL_SEL(2) AT_RL_CMP(3) AT_RL_SH(2) AT_RL_SEL(3) AT_RL_BF(0) AT_RL_SH(3) AT_RL_BF(1) AT_RL_AD(0)
                        AT_RL_BF(2) AT_RL_AD(1) AT_RL_BF(3) AT_RL_AD(2) AT_RL_AD(3)
                : [n0] "+v"(node[0]), [n1] "+v"(node[1]), [n2] "+v"(node[2]), [n3] "+v"(node[3]), [p0] "+v"(p[0]),
                  [p1] "+v"(p[1]), [p2] "+v"(p[2]), [p3] "+v"(p[3]), [f0] "=&v"(fa[0]), [f1] "=&v"(fa[1]),
                  [f2] "=&v"(fa[2]), [f3] "=&v"(fa[3]), [a0] "=&v"(pa[0]), [a1] "=&v"(pa[1]), [a2] "=&v"(pa[2]),
                  [a3] "=&v"(pa[3])
                : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [r0] "v"(pr[0]), [r1] "v"(pr[1]),
                  [r2] "v"(pr[2]), [r3] "v"(pr[3]), [rb] "v"(rb), [b0] "v"(nb[0]), [b1] "v"(nb[1]), [b2] "v"(nb[2]),
                  [b3] "v"(nb[3])
                : "vcc");
        } else if constexpr (G == 2) {
            asm volatile("ds_read_u8 %0, %4\n\tds_read_b32 %2, %6\n\tds_read_u8 %1, %5\n\tds_read_b32 %3, %7\n\t"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(x[0]), "=&v"(x[1]), "=&v"(pr[0]), "=&v"(pr[1])
                         : "v"(fa[0]), "v"(fa[1]), "v"(pa[0]), "v"(pa[1])
                         : "memory");
            asm(AT_RL_CMP(0) "s_nop 1\n\t" AT_RL_SEL(0) AT_RL_CMP(1) AT_RL_SH(0) AT_RL_SEL(1) AT_RL_BF(0) AT_RL_SH(1)
                    AT_RL_AD(0) AT_RL_BF(1) AT_RL_AD(1)
                : [n0] "+v"(node[0]), [n1] "+v"(node[1]), [p0] "+v"(p[0]), [p1] "+v"(p[1]), [f0] "=&v"(fa[0]),
                  [f1] "=&v"(fa[1]), [a0] "=&v"(pa[0]), [a1] "=&v"(pa[1])
                : [x0] "v"(x[0]), [x1] "v"(x[1]), [r0] "v"(pr[0]), [r1] "v"(pr[1]), [rb] "v"(rb), [b0] "v"(nb[0]),
                  [b1] "v"(nb[1])
                : "vcc");
        } else {
            asm volatile("ds_read_u8 %0, %2\n\tds_read_b32 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(x[0]), "=&v"(pr[0])
                         : "v"(fa[0]), "v"(pa[0])
                         : "memory");
            asm(AT_RL_CMP(0) "s_nop 1\n\t" AT_RL_SEL(0) AT_RL_SH(0) AT_RL_BF(0) AT_RL_AD(0)
                : [n0] "+v"(node[0]), [p0] "+v"(p[0]), [f0] "=&v"(fa[0]), [a0] "=&v"(pa[0])
                : [x0] "v"(x[0]), [r0] "v"(pr[0]), [rb] "v"(rb), [b0] "v"(nb[0])
                : "vcc");
        }
    }
    if constexpr (G == 4)
        asm volatile("ds_read_u8 %0, %4\n\tds_read_u8 %1, %5\n\tds_read_u8 %2, %6\n\tds_read_u8 %3, %7\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])
                     : "v"(fa[0]), "v"(fa[1]), "v"(fa[2]), "v"(fa[3])
                     : "memory");
    else if constexpr (G == 2)
        asm volatile("ds_read_u8 %0, %2\n\tds_read_u8 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(x[0]), "=&v"(x[1])
                     : "v"(fa[0]), "v"(fa[1])
                     : "memory");
    else
        asm volatile("ds_read_u8 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(x[0]) : "v"(fa[0]) : "memory");
#pragma unroll
    for (int g = 0; g < G; ++g) q[g] = 2u * p[g] + (x[g] >= (node[g] & 0xffu) ? 1u : 0u) - (1u << DEPTH);
}

template <int TMPL, int DEPTH, bool TAIL, int NT>
__global__ __launch_bounds__(NT) void k_single(SingleArgs a) {
    using N = Nest<TMPL>;
    constexpr int RS = (N::F + 3) / 4 * 4 + 4;            // feature row stride: an odd number of dwords
    static_assert(RS / 4 % 2 == 1, "rows spread over the LDS banks");
    constexpr int WALK = TAIL ? DEPTH - 1 : DEPTH;
    constexpr uint32_t TB = (uint32_t)local_stride(DEPTH, TAIL) * 4u;
    constexpr uint32_t NBB = 4u << (DEPTH - 1);           // node block bytes of a whole tree
    extern __shared__ uint4 lds4[];
    uint8_t* lds = reinterpret_cast<uint8_t*>(lds4);
    const uint32_t lbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)lds;
    float* lv = reinterpret_cast<float*>(lds + a.off_lv);
    at_entry* lists = reinterpret_cast<at_entry*>(lds + a.off_lists);
    SingleRec* rec = reinterpret_cast<SingleRec*>(lds + a.off_rec);
    uint8_t* frow = lds + a.off_frow;
    SpaceDesc& s_desc = *reinterpret_cast<SpaceDesc*>(lds + a.off_desc);
    uint64_t* s_fac = reinterpret_cast<uint64_t*>(lds + a.off_desc + sizeof(SpaceDesc));

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    constexpr int nthreads = NT, nwaves = nthreads >> 6;
    // (with 1024 threads every lane walks, and two copies of the evaluation
    // would not fit the registers)
    const bool early = NT == 512 && a.early;
    const int cpb = a.cpb;
    const int64_t c0 = (int64_t)blockIdx.x * cpb;
    const int nc = (a.n - c0 < cpb) ? (int)(a.n - c0) : cpb;
    const int k = a.topk;
    const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);

    // the trees, moved straight into LDS by every wave
    {
        const int n16 = (int)(((uint32_t)a.T * TB + 15u) >> 4);   // the forms end in 16 bytes of slack
        const uint4* src = reinterpret_cast<const uint4*>(a.tw);
        for (int base = wave * 64; base < n16; base += nthreads)
            if (base + lane < n16) __builtin_amdgcn_global_load_lds(src + base + lane, lds4 + base, 16, 0, 0);
    }
    // space tables: staged in LDS when every chain of the workgroup uses one space
    const int w_lo = space_of(a.offsets, a.n_spaces, c0), w_hi = space_of(a.offsets, a.n_spaces, c0 + nc - 1);
    int fac_lo = 0, fac_n = 0;
    if (w_lo == w_hi) {
        const SpaceDesc& g = a.descs[w_lo];
        fac_lo = g.split_off[0];
        for (int ax = 0; ax < g.n_axes; ++ax) fac_n += (int)g.knob_size[ax];
    }
    const bool staged = w_lo == w_hi && fac_n <= SINGLE_FAC_MAX;
    if (staged) {
        constexpr int DW = (int)(sizeof(SpaceDesc) / 4);
        constexpr int SO = (int)(offsetof(SpaceDesc, split_off) / 4);
        const uint32_t* gd = reinterpret_cast<const uint32_t*>(a.descs + w_lo);
        uint32_t* ld = reinterpret_cast<uint32_t*>(&s_desc);
        for (int i = tid; i < DW; i += nthreads)
            ld[i] = (i >= SO && i < SO + MAX_AXES) ? gd[i] - (uint32_t)fac_lo : gd[i];
        for (int i = tid; i < fac_n; i += nthreads) s_fac[i] = a.suffix[fac_lo + i];
    }
    // f(descriptor, split choices) of chain j's space; each branch (uniform
    // in the workgroup) reads one address space directly
    auto with_space = [&](int j, auto&& f) {
        if (staged) f(s_desc, static_cast<const uint64_t*>(s_fac));
        else f(a.descs[space_of(a.offsets, a.n_spaces, c0 + j)], a.suffix);
    };
    for (int e = tid; e < nc * k; e += nthreads) {
        at_entry z;
        z.cfg = 0;
        z.score = 0.0f;
        z.flag = 0u;
        lists[e] = a.init ? z : a.top[c0 * k + e];
    }
    auto unpack = [](const uint32_t* w, uint32_t (&kv)[MAX_KNOBS]) {
#pragma unroll
        for (int j = 0; j < MAX_KNOBS; ++j) kv[j] = (w[j >> 1] >> (16 * (j & 1))) & 0xffffu;
    };
    auto pack = [](const uint32_t (&kv)[MAX_KNOBS], uint32_t* w) {
#pragma unroll
        for (int j = 0; j < MAX_KNOBS / 2; ++j) w[j] = kv[2 * j] | (kv[2 * j + 1] << 16);
    };
    const int first_step = a.init ? -1 : 0;       // step of round 0 (-1: the initial draw)
    const int rounds = a.steps - first_step;
    // the move of round r for chain j into its record
    auto draw_into = [&](int j, int r) {
        const uint32_t gch = (uint32_t)(a.chain0 + (uint64_t)(c0 + j));
        int jm = -1;
        uint32_t v = 0u;
        uint64_t radix = 0;
        with_space(j, [&](const SpaceDesc& sd, const uint64_t*) {
            draw_move(sd, k0, k1, gch, a.step0 + (uint32_t)(first_step + r), jm, v, radix);
        });
        rec[j].mvj[r & 1] = jm;
        rec[j].mvv[r & 1] = v;
        rec[j].mvr[r & 1] = radix;
    };
    // loop l's features (4x+3) of configuration kv of chain j into row dst
    auto eval_loop = [&](const uint32_t (&kv)[MAX_KNOBS], int j, int l, uint8_t* dst) {
        uint32_t f[11], td;
        with_space(j, [&](const SpaceDesc& sd, const uint64_t* sfx) { loop_features<TMPL>(sd, sfx, kv, l, f, td, false); });
#pragma unroll
        for (int i = 0; i < 11; ++i) dst[l * 11 + i] = (uint8_t)(4u * f[i] + 3u);
    };
    // every wave's tables and trees are in place
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    const bool owner = tid < nc;
    float cur_s = 0.0f;
    if (owner) {
        const int64_t c = c0 + tid;
        SingleRec& R = rec[tid];
        ChainMeta m;
        m.count = 0;
        m.kth_score = 0.0f;
        m.kth_cfg = 0;
        if (!a.init) m = a.meta[c];
        R.count = m.count;
        R.kth_score = m.kth_score;
        R.kth_cfg = m.kth_cfg;
        cur_s = a.cur_score[c];
        uint32_t cur[MAX_KNOBS], nx[MAX_KNOBS];
        load_knobs(a.knobs, c, cur);
        uint64_t cur_cfg = 0, cfg = 0;
        // "round -1" left the current configuration as its accepted candidate
        with_space(tid, [&](const SpaceDesc& sd, const uint64_t*) {
#pragma unroll
            for (int j = 0; j < MAX_KNOBS; ++j)
                if (j < sd.n_knobs) cur_cfg += (uint64_t)cur[j] * sd.radix[j];
            if (a.init) {
                const uint32_t gch = (uint32_t)(a.chain0 + (uint64_t)c);
                U4 rr{0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < MAX_KNOBS; ++j) {
                    if ((j & 3) == 0) rr = philox(k0, k1, U4{gch, 0u, 1u, (uint32_t)(j >> 2)});
                    const uint32_t word = (j & 3) == 0 ? rr.x : (j & 3) == 1 ? rr.y : (j & 3) == 2 ? rr.z : rr.w;
                    nx[j] = (j < sd.n_knobs) ? uniform_below(word, sd.knob_size[j]) : 0u;
                    if (j < sd.n_knobs) cfg += (uint64_t)nx[j] * sd.radix[j];
                }
            }
        });
        if (!a.init && rounds > 0) {
            draw_into(tid, 0);
            apply_move(cur, cur_cfg, R.mvj[0], R.mvv[0], R.mvr[0], nx, cfg);
            R.thr[0] = a.thr[c * a.steps];
        } else if (!a.init) {
#pragma unroll
            for (int j = 0; j < MAX_KNOBS; ++j) nx[j] = cur[j];
        }
        pack(cur, R.snx[3][0]);
        R.scfg[3][0] = cur_cfg;
        pack(nx, R.snx[0][0]);
        R.scfg[0][0] = cfg;
        R.ssel[3] = R.ssel[0] = 0u;
        if (rounds > 1) draw_into(tid, 1);
    }
    lds_barrier();
    if ((tid >> 4) < nc && (tid & 15) < N::L) {
        const int j = tid >> 4;
        uint32_t kv[MAX_KNOBS];
        unpack(rec[j].snx[0][0], kv);
        eval_loop(kv, j, tid & 15, frow + j * RS);
    }
    lds_barrier();

    // offers round r's candidates, by the 16-lane groups of one wave (group g
    // takes chain g), and records them in the trace
    auto offer_round = [&](int r) {
        const int g = lane >> 4, gl = lane & 15;
        const bool on = g < nc;
        SingleRec& R = rec[on ? g : 0];
        const uint32_t o = R.ssel[r & 3];
        const uint64_t pc = R.scfg[r & 3][o];
        const float ps = R.psc[r & 1];
        const bool q = on && ((a.init && r == 0) || (int)R.count < k || precedes(ps, pc, R.kth_score, R.kth_cfg));
        if (on) {
            // (the same values from every lane of the group, which reads them back)
            R.cfg = pc;
            R.score = ps;
        }
        if (gl == 0 && on && a.trace && first_step + r >= 0) {
            at_entry t;
            t.cfg = pc;
            t.score = ps;
            t.flag = R.ssel[(r + 1) & 3] == 0u ? 1u : 0u;
            a.trace[(c0 + g) * a.steps + first_step + r] = t;
        }
        group_offer(lists + (on ? g : 0) * k, R, k, gl, 0xffffull << (16 * g), q);
    };

    // Everything beside the fold depends on the round's candidate and on
    // earlier rounds alone, so a wave that does not walk does its share
    // during the walk: the evaluating waves when the others take all trees in
    // as few passes without them (`early`: small ensembles, whose fold is
    // shorter than an evaluation), and any helper wave past the last tree.
    const int ew = early ? (cpb + 1) / 2 : 0;   // evaluating waves kept from walking
    const bool walks = wave == 0 || wave > ew;
    const int wt = tid - (wave == 0 ? 0 : 64 * ew);
    const int S = (nthreads - 64 * ew) / cpb, ja = wt & (cpb - 1), slot = wt / cpb;
    const int jr = ja < nc ? ja : nc - 1;
    const int per = (a.T + S - 1) / S;            // trees a lane
    const bool idle = walks && wave > 0 && (wt & ~63) / cpb >= a.T;   // no tree for any lane of the wave
    // phase A for trees base + slot, + S, ...: H times G of them, G walked
    // together.  With tails the first half's records are on their way while
    // the second half is walked (C2 search: 3.42 us a step against 3.65 with
    // both walked first).
    auto walk_pass = [&](auto gc, auto hc, int base, uint32_t rb) {
        constexpr int G = decltype(gc)::value, H = decltype(hc)::value;
        uint4 rec4[TAIL ? G * H : 1];
        int ti[G * H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            uint32_t nb[G], q[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int t = base + slot + (h * G + g) * S;
                ti[h * G + g] = t < a.T ? t : -1;
                nb[g] = lbase + (uint32_t)(t < a.T ? t : 0) * TB;
            }
            walk_row<(WALK > 0 ? WALK : 1), G>(nb, rb, q);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int t = ti[h * G + g];
                if constexpr (TAIL) {
                    rec4[h * G + g] = a.tail_rec[((size_t)(t >= 0 ? t : 0) << WALK) + q[g]];
                } else {
                    const uint32_t v = *reinterpret_cast<const uint32_t*>(lds + (nb[g] - lbase) + NBB + 4u * q[g]);
                    if (t >= 0 && ja < nc) lv[ja * a.lv_stride + t] = __uint_as_float(v);
                }
            }
        }
        if constexpr (TAIL) {
#pragma unroll
            for (int i = 0; i < G * H; ++i) {
                const uint32_t x4 = lds[rb - lbase + row_byte(rec4[i].x)];
                const uint32_t v = x4 >= (rec4[i].x & 0xffu) ? rec4[i].z : rec4[i].y;
                if (ti[i] >= 0 && ja < nc) lv[ja * a.lv_stride + ti[i]] = __uint_as_float(v);
            }
        }
    };
    using One = std::integral_constant<int, 1>;
    using Each = std::integral_constant<int, TAIL ? 1 : 2>;    // two trees a pass
    using Pair = std::integral_constant<int, TAIL ? 2 : 4>;    // four trees a pass
    using Halves = std::integral_constant<int, TAIL ? 2 : 1>;

    // Both candidates that can follow round r, with the features of both
    // (waves 1 .. ceil(cpb / 2)): item (v * cpb + j) * 16 + l is loop l of
    // chain j's next candidate after outcome v of this round.  A wave that
    // does this during the walk passes the barrier after the walk halfway.
    auto make_next = [&](int r, bool halfway) {
        const int it = tid - 64;
        const int l = it & 15, jv = it >> 4, j = jv & (cpb - 1), v = jv >= cpb ? 1 : 0;
        const bool on = it < 32 * cpb && j < nc && l < N::L;
        uint32_t nx[MAX_KNOBS];
        if (on) {
            SingleRec& R = rec[j];
            const uint32_t o = R.ssel[r & 3], op = R.ssel[(r + 3) & 3];
            // this round's candidate (v = 0; after the initial draw, which is
            // always accepted, also v = 1), or the configuration the round
            // starts from: the previous round's candidate if it was accepted,
            // else what that round started from
            const bool from_cand = v == 0 || (a.init && r == 0);
            const uint32_t* src = from_cand ? R.snx[r & 3][o]
                                : o == 0u   ? R.snx[(r + 3) & 3][op]
                                            : R.curk[(r + 1) & 1];
            const uint64_t bcfg = from_cand ? R.scfg[r & 3][o]
                                : o == 0u   ? R.scfg[(r + 3) & 3][op]
                                            : R.curcfg[(r + 1) & 1];
            uint32_t w[MAX_KNOBS / 2], base[MAX_KNOBS];
#pragma unroll
            for (int i = 0; i < MAX_KNOBS / 2; ++i) w[i] = src[i];
            if (v == 1 && l == 0) {
#pragma unroll
                for (int i = 0; i < MAX_KNOBS / 2; ++i) R.curk[r & 1][i] = w[i];
                R.curcfg[r & 1] = bcfg;
            }
            uint64_t ncfg;
            unpack(w, base);
            const int sl = (r + 1) & 1;
            apply_move(base, bcfg, R.mvj[sl], R.mvv[sl], R.mvr[sl], nx, ncfg);
            if (l == 0 && r + 1 < rounds) {
                pack(nx, R.snx[(r + 1) & 3][v]);
                R.scfg[(r + 1) & 3][v] = ncfg;
            }
        }
        if (halfway) lds_barrier();
        if (on && r + 1 < rounds) eval_loop(nx, j, l, frow + (2 * ((r + 1) & 1) + v) * a.frow_stride + j * RS);
    };
    // The other work beside a fold: waves 3 and 4 and the last one.
    auto side_work = [&](int r) {
        if (wave == 3 && r > 0) offer_round(r - 1);
        if (wave == 4 && lane < nc && r + 2 < rounds) draw_into(lane, r + 2);
        if (wave == nwaves - 1 && lane < nc && r + 1 < rounds)
            rec[lane].thr[(r + 1) & 1] = a.thr[(c0 + lane) * a.steps + first_step + r + 1];
    };

    for (int r = 0; r < rounds; ++r) {
        // ---- A: walk
        if (NT == 512 && !walks) {
            make_next(r, true);      // with this round's barrier after the walk
            lds_barrier();
            continue;
        }
        if (idle) {
            side_work(r);
        } else {
            const uint32_t o = rec[jr].ssel[r & 3];
            const uint32_t rb = lbase + a.off_frow + (2u * (uint32_t)(r & 1) + o) * a.frow_stride + (uint32_t)jr * RS;
            if (per == 1) {
                if (slot < a.T) walk_pass(One{}, One{}, 0, rb);
            } else if (per == 2) {
                walk_pass(Each{}, Halves{}, 0, rb);
            } else {
                for (int base = 0; base < a.T; base += 4 * S) walk_pass(Pair{}, Halves{}, base, rb);
            }
        }
        lds_barrier();
        // ---- B
        if (wave == 0) {
            if (owner) {
                SingleRec& R = rec[lane];
                const float thr_v = R.thr[r & 1];
                // the adds depend on one another: this wave goes first
                // whenever it can issue
                __builtin_amdgcn_s_setprio(3);
                const float sc = fold_row(0.0f, lv + lane * a.lv_stride, a.T);
                __builtin_amdgcn_s_setprio(0);
                const bool acc = (a.init && r == 0) || (sc - cur_s) >= thr_v;
                R.ssel[(r + 1) & 3] = acc ? 0u : 1u;
                R.psc[r & 1] = sc;
                if (acc) cur_s = sc;
            }
        } else {
            if (!early && wave <= (cpb + 1) / 2) make_next(r, false);
            if (!idle) side_work(r);
        }
        lds_barrier();
    }
    if (wave == 3 && rounds > 0) offer_round(rounds - 1);
    // write the chain state and the best lists back
    __syncthreads();
    if (owner) {
        const int64_t c = c0 + tid;
        const SingleRec& R = rec[tid];
        const int r = rounds;
        uint32_t cur[MAX_KNOBS];
        unpack(R.ssel[r & 3] == 0u ? R.snx[(r + 3) & 3][R.ssel[(r + 3) & 3]] : R.curk[(r + 1) & 1], cur);
        store_knobs(a.knobs, c, cur);
        a.cur_score[c] = cur_s;
        ChainMeta m;
        m.count = R.count;
        m.kth_score = R.kth_score;
        m.kth_cfg = R.kth_cfg;
        a.meta[c] = m;
    }
    for (int e = tid; e < nc * k; e += nthreads) {
        const at_entry x = lists[e];
        a.top[c0 * k + e] = x;
        a.best[c0 * k + e] = x;
    }
}

template <int TMPL, int DEPTH, bool TAIL, int NT>
hipError_t launch_single_nt(const SingleArgs& a, const LocalPlan& pl, hipStream_t stream) {
    static std::atomic<uint64_t> done;
    const void* fn = reinterpret_cast<const void*>(&k_single<TMPL, DEPTH, TAIL, NT>);
    const hipError_t e = prepare_kernel(fn, -1, SINGLE_LDS_BYTES, done);
    if (e != hipSuccess) return e;
    void* args[] = {const_cast<SingleArgs*>(&a)};
    return hipLaunchKernel(fn, dim3(pl.grid), dim3(NT), args, pl.lds_bytes, stream);
}

template <int TMPL, int DEPTH, bool TAIL>
hipError_t launch_single_t(const SingleArgs& a, const LocalPlan& pl, hipStream_t stream) {
    // 1024 threads are for more than 1024 walks of at most four chains, and
    // 257 whole trees of depth 7, or tops of depth 10, do not fit the LDS
    if constexpr ((SINGLE_WIDE_WALKS / SINGLE_CHAINS + 1) * local_stride(DEPTH, TAIL) * 4 <= (int)SINGLE_LDS_BYTES) {
        if (pl.threads == 1024) return launch_single_nt<TMPL, DEPTH, TAIL, 1024>(a, pl, stream);
    }
    if (pl.threads != 512) return hipErrorInvalidConfiguration;
    return launch_single_nt<TMPL, DEPTH, TAIL, 512>(a, pl, stream);
}

template <int TMPL, bool TAIL>
hipError_t launch_single_d(const SingleArgs& a, const LocalPlan& pl, int depth, hipStream_t stream) {
    switch (depth) {
        case 1: return launch_single_t<TMPL, 1, false>(a, pl, stream);
        case 2: return launch_single_t<TMPL, 2, TAIL>(a, pl, stream);
        case 3: return launch_single_t<TMPL, 3, TAIL>(a, pl, stream);
        case 4: return launch_single_t<TMPL, 4, TAIL>(a, pl, stream);
        case 5: return launch_single_t<TMPL, 5, TAIL>(a, pl, stream);
        case 6: return launch_single_t<TMPL, 6, TAIL>(a, pl, stream);
        case 7: return launch_single_t<TMPL, 7, TAIL>(a, pl, stream);
        case 8: return launch_single_t<TMPL, 8, TAIL>(a, pl, stream);
        case 9: return launch_single_t<TMPL, 9, TAIL>(a, pl, stream);
        case 10: return launch_single_t<TMPL, 10, TAIL>(a, pl, stream);
        case 11: return launch_single_t<TMPL, 11, TAIL>(a, pl, stream);
        case 12: return launch_single_t<TMPL, 12, TAIL>(a, pl, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Plan of the single-pass kernel for pl.cpb chains per workgroup (at most
// four): whole trees when they all fit beside the chains' state, else the
// tree tops.  False when neither does.  A lane takes one, two or four trees
// a pass: 1024 threads when 512 would give it more than two (the C2 search,
// 2000 tree walks a round: 1685 us a run against 1790).
bool plan_single(const at_space_s& sp, const EnsembleDesc& e, const at_chains_s& ch, LocalPlan& pl) {
    if (pl.cpb > SINGLE_CHAINS) return false;
    const int64_t n = ch.n_chains;
    const int RS = (sp.descs[0].n_features + 3) / 4 * 4 + 4;
    int fac_max = 0;
    for (const SpaceDesc& x : sp.descs) {
        int f = 0;
        for (int ax = 0; ax < x.n_axes; ++ax) f += (int)x.knob_size[ax];
        fac_max = f > fac_max ? f : fac_max;
    }
    if (fac_max > SINGLE_FAC_MAX) fac_max = SINGLE_FAC_MAX;
    auto al16 = [](size_t x) { return (x + 15) & ~(size_t)15; };
    const int T = e.n_trees, T4 = (T + 3) / 4 * 4;
    for (const bool tail : {false, true}) {
        if (tail && e.depth < 2) continue;
        const int ts = local_stride(e.depth, tail);
        size_t off = al16((size_t)T * ts * 4);
        pl.ring_bytes = (uint32_t)off;
        pl.off_lv = (uint32_t)off;
        pl.lv_stride = T4 + 4;
        off += al16((size_t)pl.cpb * pl.lv_stride * 4);
        pl.off_lists = (uint32_t)off;
        off += al16((size_t)pl.cpb * ch.topk * sizeof(at_entry));
        pl.off_rec = (uint32_t)off;
        off += al16((size_t)pl.cpb * sizeof(SingleRec));
        pl.off_frow = (uint32_t)off;
        pl.frow_stride = (uint32_t)al16((size_t)pl.cpb * RS);
        off += 4 * pl.frow_stride;
        pl.off_desc = (uint32_t)off;
        off += al16(sizeof(SpaceDesc) + (size_t)fac_max * 8);
        if (off > SINGLE_LDS_BYTES) continue;
        pl.single = 1;
        pl.resident = tail ? 0 : 1;
        pl.tail = tail ? 1 : 0;
        pl.gather = 0;
        pl.ts = ts;
        pl.ct = T;
        pl.n_chunks = 1;
        pl.threads = T * pl.cpb > SINGLE_WIDE_WALKS ? 1024 : 512;
        // the evaluating waves stay out of the walk when that costs no pass
        const int ew = (pl.cpb + 1) / 2;
        auto passes = [&](int lanes) {
            const int S = lanes / pl.cpb, per = (T + S - 1) / S;
            return per <= 2 ? per : (per + 3) / 4 * 4;
        };
        pl.walk_waves = pl.threads / 64;
        if (pl.threads == 512 && passes(pl.threads - 64 * ew) == passes(pl.threads)) pl.walk_waves -= ew;
        pl.grid = (int)((n + pl.cpb - 1) / pl.cpb);
        pl.lds_bytes = off;
        pl.round_bytes = tail ? (double)pl.cpb * T * 64 : 0.0;
        return true;
    }
    return false;
}

hipError_t launch_sa_single(const at_space_s& sp, const EnsembleDesc& e, at_chains_s& ch, const LocalPlan& pl,
                            int steps, bool init, const float* thr, at_entry* best, at_entry* trace,
                            hipStream_t stream) {
    SingleArgs a{};
    a.descs = static_cast<const SpaceDesc*>(sp.d_descs.p);
    a.offsets = static_cast<const int64_t*>(sp.d_offsets.p);
    a.n_spaces = sp.n_spaces;
    a.suffix = sp.suffix;
    a.knobs = static_cast<uint16_t*>(ch.d_knobs.p);
    a.cur_score = static_cast<float*>(ch.d_score.p);
    a.top = static_cast<at_entry*>(ch.d_top.p);
    a.meta = static_cast<ChainMeta*>(ch.d_meta.p);
    a.topk = ch.topk;
    a.cpb = pl.cpb;
    a.n = ch.n_chains;
    a.chain0 = (uint64_t)ch.chain0;
    a.seed = ch.seed;
    a.init = init ? 1 : 0;
    a.steps = steps;
    a.step0 = (uint32_t)ch.step_abs;
    a.thr = thr;
    a.trace = trace;
    a.best = best;
    a.tw = pl.tail ? e.local_top : e.local_full;
    a.T = e.n_trees;
    a.tail_rec = e.tail;
    a.early = pl.walk_waves < pl.threads / 64 ? 1 : 0;
    a.off_lv = pl.off_lv;
    a.off_lists = pl.off_lists;
    a.off_rec = pl.off_rec;
    a.off_frow = pl.off_frow;
    a.off_desc = pl.off_desc;
    a.lv_stride = pl.lv_stride;
    a.frow_stride = pl.frow_stride;
    if (sp.tmpl == AT_TMPL_GEMM)
        return pl.tail ? launch_single_d<AT_TMPL_GEMM, true>(a, pl, e.depth, stream)
                       : launch_single_d<AT_TMPL_GEMM, false>(a, pl, e.depth, stream);
    return pl.tail ? launch_single_d<AT_TMPL_CONV2D_NCHW, true>(a, pl, e.depth, stream)
                   : launch_single_d<AT_TMPL_CONV2D_NCHW, false>(a, pl, e.depth, stream);
}

}  // namespace at
