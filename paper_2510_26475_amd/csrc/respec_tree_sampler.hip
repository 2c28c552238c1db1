// Rejection sampling over a tree of drafts for gfx950 (Section 4.1: several candidate
// branches per position, branching factor t, validated in one target forward).
//
// The paper gives the chain rule (Section 2.2, Eq. 1 and Eq. 2) and leaves the rule for
// sibling candidates open; this kernel takes the reading that keeps the output distributed
// as the target: the children of a node are candidates drawn independently from the
// drafter's distribution q at that node, tried in row order against a running distribution
// that starts as the target's p at that node.  A candidate x is accepted with probability
// min(1, p_r(x)/q(x)) (Eq. 1 with p_r in the place of p); a rejection replaces p_r by
// p_{r+1} = max(0, p_r - q)/Z_{r+1} (Eq. 2 applied to p_r).  An accepted child becomes the
// node; when no child is left the one final token is drawn from the running distribution.
// A chain is the tree with one child per node and gives exactly the chain sampler's tokens.
//
// One work-group of 512 threads walks one sequence, or, while the batch leaves compute units idle, two or four do,
// a part of the vocabulary each: after every pass they exchange their partial results and take the same decisions
// from the same numbers (respec_sampler_share.hpp).  p_r(x) is a pointwise function of
// p(x), q(x) and the r scalars Z_1..Z_r, so nothing is materialised: every rejection costs
// one streaming pass over the node's row pair that sums max(0, p_r - q) (region totals in
// fp64, which also serve the final draw when the rejected child was the last), and an
// acceptance test needs only the candidate's own two logits.
#include "respec_sampler_share.hpp"
#include "respec_tree_candidate.hpp"

#include <algorithm>
#include <type_traits>

namespace respec {
namespace {

// The two logits of a candidate as they are in memory, requested behind a pass's first batch, so that the test behind
// the pass waits for nothing (its chain of loads, token, logits and uniform, took 1.5 us of every pass).  WORD: through
// the scalar cache, the same for every thread and in scalar registers, so that the pass keeps its vector registers; a
// 16-bit logit then comes with the rest of its aligned word.
struct Candidate {
    uint32_t p, q;
};

__device__ inline uint32_t scalar_word(uint64_t at) {
    const uint64_t uniform = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)at) |
                             (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)) << 32;
    return *(const uint32_t __attribute__((address_space(4))) *)uniform;
}

template <bool BF16, bool WORD>
__device__ inline Candidate fetch_candidate(const char *rowp, const char *rowq, int x) {
    if constexpr (WORD) {
        Candidate c{scalar_word(candidate_word_at(reinterpret_cast<uintptr_t>(rowp), x, BF16)),
                    scalar_word(candidate_word_at(reinterpret_cast<uintptr_t>(rowq), x, BF16))};
        asm volatile("" : "+s"(c.p), "+s"(c.q));  // (here, not where they are used)
        return c;
    } else {
        // (as they come: whatever is done to them here would wait for them here)
        return Candidate{reinterpret_cast<const uint16_t *>(rowp)[x], reinterpret_cast<const uint16_t *>(rowq)[x]};
    }
}

template <bool BF16, bool WORD>
__device__ inline float candidate_logit(uint32_t word, const char *row, int x) {
    static_assert(WORD || BF16, "fp32 logits are words");
    return __uint_as_float(WORD ? candidate_bits(word, reinterpret_cast<uintptr_t>(row), x, BF16) : word << 16);
}

constexpr int kMaxTreeRows = 64;   // rows (nodes) of one sequence: the attention's mask width
constexpr int kRegDepth = 3;       // rejection depths whose normalisers are held in registers

struct TreeParams : RowMath {
    const void *target;
    const void *draft;
    const int32_t *node_tokens;
    const int32_t *parent;
    const int32_t *q_indptr;
    const float *u_accept;
    const float *u_final;
    int32_t *out_tokens;
    int32_t *out_path;
    int32_t *out_num_accepted;
    int32_t *out_flags;
    int32_t B, total_q, max_depth, V;
    int64_t ld_t, ld_d;
    int split;        // work-groups per sequence
    uint32_t claim;   // their call's key in the library's mailboxes, and ...
    int claim_ticks;  // ... how long they wait to meet
};

// The running distribution after `depth` rejections at one node, without its normaliser:
// a_0 = p, a_j = max(0, a_{j-1} / Z_{j-1} - q) with Z_0 = 1, so that p_depth = a_depth / Z_depth.
// inv_z[j] = 1/Z_j lives in LDS; the first few are passed in registers.
struct Depth {
    int depth;
    double z1, z2;          // inv_z[1], inv_z[2] (1.0 while unused)
    const double *inv_z;    // LDS, [kMaxTreeRows]
};

__device__ inline double running_weight(double pe, double qe, const Depth &d) {
    double a = pe;
    if (d.depth >= 1) a = fmax(a - qe, 0.0);
    if (d.depth >= 2) a = fmax(a * d.z1 - qe, 0.0);
    if (d.depth >= 3) a = fmax(a * d.z2 - qe, 0.0);
    for (int j = kRegDepth; j < d.depth; ++j) a = fmax(a * d.inv_z[j] - qe, 0.0);
    return a;
}

// The passes are instantiated by depth: KIND = 0, 1 and 2 rejections (nearly all of them), kAnyDepth
// = the loop over d.depth.  The passes are bound by instruction issue; with the depth tested per
// element they had nine branches and 220 vector instructions per eight logits of both rows, now 88
// (KIND 1) and 112 (KIND 2): B = 128, trees of 3 x 2 candidates, V = 151,936 bf16, T = 0.6 took 139.8
// and takes 98.7 us.
constexpr int kAnyDepth = 3;

// fp64 weights a_depth(x) of the elements of one slot.
template <bool BF16, int KIND>
__device__ inline void tree_slot_weights(const u32x4 &vp, const u32x4 &vq, float Mp, double Cp, float Mq,
                                         double Cq, const Depth &d, const RowMath &p,
                                         double (&w)[Elem<BF16>::EPV]) {
    constexpr int EPV = Elem<BF16>::EPV;
    float zp[EPV], zq[EPV];
    unpack<BF16>(vp, zp);
    if constexpr (KIND > 0) unpack<BF16>(vq, zq);
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
        const double pe = (double)hw_exp2(exp2_arg(zp[j], Mp, p.c_hi, p.c_lo)) * Cp;
        if constexpr (KIND == 0) {
            w[j] = pe;
        } else {
            const double qe = (double)hw_exp2(exp2_arg(zq[j], Mq, p.c_hi, p.c_lo)) * Cq;
            if constexpr (KIND == kAnyDepth) {
                w[j] = running_weight(pe, qe, d);
            } else {
                w[j] = fmax(pe - qe, 0.0);
                if constexpr (KIND == 2) w[j] = fmax(w[j] * d.z1 - qe, 0.0);
            }
        }
    }
}

// The same weights in fp32 (calls whose exponent constant rounds well), times a factor common to
// the row: probabilities as in FastNorm, the weights of a slot summed in fp32 in a fixed pairwise
// order (returned); everything above a slot is carried in fp64.  KIND 1 forms the chain sampler's
// weights, a_1 / (1 + ep).  KIND 2 forms Z_1 a_2 / (1 + ep) = max(0, a_1 / (1 + ep) - q Z_1 / (1 + ep)),
// which scales q instead of dividing the first difference: g = Z_1 (1 + eq) / (1 + ep), a two-term
// binary32 constant so that no systematic error enters.  kAnyDepth forms a_depth itself, with
// every 1/Z_j as such a constant.
struct FastDepth {
    int depth;
    float g_hi, g_lo;           // KIND 2
    float z1h, z1l, z2h, z2l;   // kAnyDepth: 1/Z_1 and 1/Z_2 as hi + lo
    const double *inv_z;
};

// raw_1: the sum of KIND 1's weights over the row.
__device__ inline FastDepth make_fast_depth(const Depth &d, double raw_1, const FastNorm &f) {
    FastDepth r;
    r.depth = d.depth;
    const double g = raw_1 + raw_1 * (double)f.eq;
    r.g_hi = (float)g;
    r.g_lo = (float)(g - (double)r.g_hi);
    r.z1h = (float)d.z1;
    r.z1l = (float)(d.z1 - (double)r.z1h);
    r.z2h = (float)d.z2;
    r.z2l = (float)(d.z2 - (double)r.z2h);
    r.inv_z = d.inv_z;
    return r;
}

__device__ inline float running_weight_f32(float pe, float qe, const FastDepth &d) {
    float a = pe;
    if (d.depth >= 1) a = fmaxf(a - qe, 0.f);
    if (d.depth >= 2) a = fmaxf(fmaf(a, d.z1h, a * d.z1l) - qe, 0.f);
    if (d.depth >= 3) a = fmaxf(fmaf(a, d.z2h, a * d.z2l) - qe, 0.f);
    for (int j = kRegDepth; j < d.depth; ++j) {
        const float zh = (float)d.inv_z[j], zl = (float)(d.inv_z[j] - (double)zh);
        a = fmaxf(fmaf(a, zh, a * zl) - qe, 0.f);
    }
    return a;
}

template <bool BF16, int KIND>
__device__ inline float tree_slot_weights_f32(const u32x4 &vp, const u32x4 &vq, const FastNorm &f,
                                              const FastDepth &d, const RowMath &p,
                                              float (&w)[Elem<BF16>::EPV]) {
    constexpr int EPV = Elem<BF16>::EPV;
    float zp[EPV], zq[EPV];
    unpack<BF16>(vp, zp);
    if constexpr (KIND > 0) unpack<BF16>(vq, zq);
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
        const float pe = hw_exp2(fmaf(zp[j], p.c_f, f.Kp));
        if constexpr (KIND == 0) {
            w[j] = pe;
        } else {
            const float qe = hw_exp2(fmaf(zq[j], p.c_f, f.Kq));
            if constexpr (KIND == kAnyDepth) {
                w[j] = running_weight_f32(fmaf(pe, f.ep, pe), fmaf(qe, f.eq, qe), d);
            } else {
                w[j] = fmaxf(fmaf(-qe, f.e_rel, pe - qe), 0.f);
                if constexpr (KIND == 2) w[j] = fmaxf(fmaf(-qe, d.g_lo, fmaf(-qe, d.g_hi, w[j])), 0.f);
            }
        }
    }
    if constexpr (EPV == 8)
        return ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
    else
        return (w[0] + w[1]) + (w[2] + w[3]);
}

// Region totals of the running distribution: each wave owns a contiguous eighth of the row (or of a part of it)
// and streams it with coalesced loads; lanes keep their own fp64 sums, one reduction per wave
// gives the region total (left in sh.wave_total; of a shared sequence those of all parts, in vocabulary order, in
// sh.xchg).  tree_region_totals returns Z = the ordered sum of the region totals, the same bits in every thread.  At depth 0
// only the target row is read.
// `meanwhile` is called once the first batch has been requested.
template <bool BF16, bool FULL, bool FAST, bool PARTIAL, int KIND, class Meanwhile>
__device__ __forceinline__ void part_region_totals(const void *rowp, const void *rowq, int nslots, int V, float Mp,
                                                   double Sp, float Mq, double Sq, const Depth &d, double raw_1, SharedState &sh,
                                                   const RowMath &p, Meanwhile &&meanwhile) {
    constexpr int EPV = Elem<BF16>::EPV;
    const int lane = opaque_thread_index() & 63, wave = threadIdx.x >> 6;
    constexpr bool two = KIND > 0;
    const double Cp = 1.0 / Sp, Cq = two ? 1.0 / Sq : 0.0;
    const FastNorm fn = make_fast_norm(Mp, Sp, Mq, two ? Sq : Sp, p);
    const FastDepth fd = make_fast_depth(d, raw_1, fn);
    const int span = ((nslots + kWaves - 1) / kWaves + 63) / 64 * 64;
    const int whole = PARTIAL ? whole_slots<BF16>(nslots, V) : nslots;
    const int beg = min(wave * span, nslots), end_all = min(beg + span, nslots), end = min(end_all, whole);
    __syncthreads();  // the totals of an earlier pass have been read by everyone
    double lane_sum = 0.0;
    auto load_batch = [&](int s0, u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kUnroll; ++c) {  // no select behind a load: the loads of a batch go out together
            const int slot = s0 + c * 64 + lane;
            vp[c] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(rowp, slot < end ? slot : beg, V);
            if constexpr (two) vq[c] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(rowq, slot < end ? slot : beg, V);
            else vq[c] = vp[c];
        }
    };
    if (beg < end) {  // wave-uniform
        // two register sets take turns: one is summed while the other's loads are in flight
        u32x4 vp[kUnroll], vq[kUnroll], np[kUnroll], nq[kUnroll];
        // (whole: every slot of the batch lies inside the region, true for all but a region's last)
        auto sum_batch = [&](int s0, const u32x4 (&xp)[kUnroll], const u32x4 (&xq)[kUnroll], auto whole) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < kUnroll; ++c) {
                if (!decltype(whole)::value && s0 + c * 64 >= end) break;  // wave-uniform
                const bool in = decltype(whole)::value || s0 + c * 64 + lane < end;  // slots past the region count as -inf
                const u32x4 a = in ? xp[c] : neg_inf_slot<BF16>(), b = in ? xq[c] : neg_inf_slot<BF16>();
                if constexpr (FAST) {
                    float w[EPV];
                    lane_sum += (double)tree_slot_weights_f32<BF16, KIND>(a, b, fn, fd, p, w);
                } else {
                    double w[EPV];
                    tree_slot_weights<BF16, KIND>(a, b, Mp, Cp, Mq, Cq, d, p, w);
#pragma unroll
                    for (int j = 0; j < EPV; ++j) lane_sum += w[j];
                }
            }
        };
        constexpr int kStep = 64 * kUnroll;
        load_batch(beg, vp, vq);
        meanwhile();
        // (the loads of the steady state are unconditional: behind a condition the wait for the
        // batch in front of a load becomes a wait for everything in flight)
        int s0 = beg;
        for (; s0 + 2 * kStep < end; s0 += 2 * kStep) {
            load_batch(s0 + kStep, np, nq);
            sum_batch(s0, vp, vq, std::true_type{});
            load_batch(s0 + 2 * kStep, vp, vq);
            sum_batch(s0 + kStep, np, nq, std::true_type{});
        }
        if (s0 + kStep < end) {
            load_batch(s0 + kStep, np, nq);
            sum_batch(s0, vp, vq, std::true_type{});
            sum_batch(s0 + kStep, np, nq, std::false_type{});
        } else {
            sum_batch(s0, vp, vq, std::false_type{});
        }
    }
    if (beg >= end) meanwhile();
    if constexpr (PARTIAL) {
        if (beg <= whole && whole < end_all && lane == 0) {  // the row's partial slot
            const u32x4 a = load_partial_slot<BF16>(rowp, whole, V), b = two ? load_partial_slot<BF16>(rowq, whole, V) : a;
            double w[EPV];
            tree_slot_weights<BF16, KIND>(a, b, Mp, Cp, Mq, Cq, d, p, w);
#pragma unroll
            for (int j = 0; j < EPV; ++j) lane_sum += w[j];
        }
    }
    double region_total = wave_sum(lane_sum);
    if (PARTIAL && region_total > kFastMost) region_total = (double)INFINITY;
    if (lane == 0) sh.wave_total[wave] = region_total;
    __syncthreads();
}

// (the rows from their starts; `own`: this block's part)
template <bool BF16, bool FULL, bool FAST, bool PARTIAL, int KIND, bool SHARED, class Meanwhile = Nothing>
__device__ inline double tree_region_totals(const char *rowp, const char *rowq, const PartView &own, int V, float Mp,
                                            double Sp, float Mq, double Sq, const Depth &d, double raw_1, SharedState &sh,
                                            Mailbox &mb, const RowMath &p, Meanwhile &&meanwhile = Nothing{}) {
    double Z = 0.0;
    if constexpr (SHARED) {
        static_assert(kWaves == 8, "a part publishes eight numbers");
        for_parts<BF16, true>(mb, own, V, sh, [&](int, const PartView &v, double(&mine)[8]) __attribute__((always_inline)) {
            part_region_totals<BF16, FULL, FAST, PARTIAL, KIND>(rowp + (size_t)v.lo * 16, rowq + (size_t)v.lo * 16, v.nslots, v.Vrow, Mp, Sp,
                                                                Mq, Sq, d, raw_1, sh, p, meanwhile);
#pragma unroll
            for (int w = 0; w < kWaves; ++w) mine[w] = sh.wave_total[w];
        });
        for (int w = 0; w < mb.split * kWaves; ++w) Z += sh.xchg[w / kWaves][w % kWaves];
    } else {
        part_region_totals<BF16, FULL, FAST, PARTIAL, KIND>(rowp, rowq, own.nslots, V, Mp, Sp, Mq, Sq, d, raw_1, sh, p, meanwhile);
        for (int w = 0; w < kWaves; ++w) Z += sh.wave_total[w];
    }
    return lane_value(Z, 0);  // (every lane's, in scalar registers)
}

// The final draw, given the region totals that tree_region_totals left (Z > 0): first token, in ascending
// id, whose running sum of weights exceeds u*Z.  Every thread finds the region that holds the
// crossing from the ordered prefix over the region totals; the block re-reads that region,
// each thread a short contiguous run of slots: thread totals -> one block scan -> the first
// thread whose running sum passes u*Z walks its run element by element.  The re-read adds
// the same numbers in another order than the region pass, so at the last bit a crossing can
// fall off the end of the region; that draw takes the last token with mass and is flagged.
// SHARED: -1 with mine = false when the region lies in another part of the row.
template <bool BF16, bool FULL, bool FAST, bool PARTIAL, int KIND, bool SHARED>
__device__ inline int tree_draw(const char *row_p, const char *row_q, const PartView &own, int V_row, float Mp, double Sp,
                                float Mq, double Sq, const Depth &d, double raw_1, double u, SharedState &sh,
                                const Mailbox &mb, const RowMath &p, int &near_edge, bool &mine) {
    constexpr int EPV = Elem<BF16>::EPV;
    const int lane = opaque_thread_index() & 63, wave = threadIdx.x >> 6;
    constexpr bool two = KIND > 0;
    const double Cp = 1.0 / Sp, Cq = two ? 1.0 / Sq : 0.0;
    const FastNorm fn = make_fast_norm(Mp, Sp, Mq, two ? Sq : Sp, p);
    const FastDepth fd = make_fast_depth(d, raw_1, fn);
    if (threadIdx.x == 0) {
        sh.token = -1;
        sh.near_edge = 0;
        sh.first_thread = kThreads;
        sh.last_positive = -1;
    }
    const int regions = SHARED ? mb.split * kWaves : kWaves;
    auto total_of = [&](int w) { return SHARED ? sh.xchg[w / kWaves][w % kWaves] : sh.wave_total[w]; };
    double Z = 0.0;
    for (int w = 0; w < regions; ++w) Z += total_of(w);
    const double t = u * Z;
    int rstar = -1, rlast = 0;
    double base = 0.0, prefix = 0.0;
    for (int w = 0; w < regions; ++w) {
        const double tot = total_of(w);
        const double next = prefix + tot;  // same additions, same order as Z above
        if (rstar < 0 && next > t) {
            rstar = w;
            base = prefix;
        }
        if (tot > 0.0) rlast = w;
        prefix = next;
    }
    const bool forced = rstar < 0;  // u*Z rounded up to Z: take the last token with mass
    if (forced) rstar = rlast;
    mine = true;
    PartView v = own;
    if constexpr (SHARED) {
        mine = mb.alone || rstar / kWaves == mb.part;  // block-uniform
        if (!mine) return -1;
        if (mb.alone) v = part_view<BF16>(V_row, __builtin_amdgcn_readfirstlane(rstar / kWaves), mb.split);
        rstar %= kWaves;
    }
    const char *rowp = row_p + (size_t)v.lo * 16, *rowq = row_q + (size_t)v.lo * 16;
    const int nslots = v.nslots, V = v.Vrow, span = ((nslots + kWaves - 1) / kWaves + 63) / 64 * 64;
    __syncthreads();

    const int whole = PARTIAL ? whole_slots<BF16>(nslots, V) : nslots;
    auto any_slot = [&](const void *row, int sidx) {
        if constexpr (FULL && !PARTIAL) return load_slot<BF16, FULL, false, true>(row, sidx, V);
        else if constexpr (FULL) {
            const u32x4 v = load_slot_or_last<BF16>(row, sidx, V);
            return sidx < whole ? v : partial_slot<BF16>(v, whole, V);
        } else return load_slot<BF16>(row, sidx, V);
    };
    const int rb = min(rstar * span, nslots), re = min(rb + span, nslots);
    const int per = (re - rb + kThreads - 1) / kThreads;
    const int my0 = rb + threadIdx.x * per, my1 = min(my0 + per, re);
    double my_total = 0.0;
    int my_last = -1;
    auto load_chunk = [&](int c0, u32x4 (&vp)[kChunk], u32x4 (&vq)[kChunk]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {  // no select behind a load: the loads go out together
            const int slot = c0 + j < my1 ? c0 + j : rb;
            if constexpr (PARTIAL) {
                vp[j] = load_slot_or_last<BF16>(rowp, slot, V);
                if constexpr (two) vq[j] = load_slot_or_last<BF16>(rowq, slot, V);
            } else {
                vp[j] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(rowp, slot, V);
                if constexpr (two) vq[j] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(rowq, slot, V);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {  // slots past the run count as -inf
            const bool in = c0 + j < my1;
            if (PARTIAL && c0 + j == whole) {
                vp[j] = partial_slot<BF16>(vp[j], whole, V);
                if constexpr (two) vq[j] = partial_slot<BF16>(vq[j], whole, V);
            }
            vp[j] = in ? vp[j] : neg_inf_slot<BF16>();
            if constexpr (two) vq[j] = in ? vq[j] : neg_inf_slot<BF16>();
            else vq[j] = vp[j];
        }
    };
    double slot_total[kChunk];
#pragma unroll
    for (int j = 0; j < kChunk; ++j) slot_total[j] = 0.0;
    for (int c0 = my0; c0 < my1; c0 += kChunk) {
        u32x4 vp[kChunk], vq[kChunk];
        load_chunk(c0, vp, vq);
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
            double st = 0.0;
            if constexpr (FAST) {
                float w[EPV];
                st = (double)tree_slot_weights_f32<BF16, KIND>(vp[j], vq[j], fn, fd, p, w);
#pragma unroll
                for (int e = 0; e < EPV; ++e)
                    if (w[e] > 0.f) my_last = (c0 + j) * EPV + e;
            } else {
                double w[EPV];
                tree_slot_weights<BF16, KIND>(vp[j], vq[j], Mp, Cp, Mq, Cq, d, p, w);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    st += w[e];
                    if (w[e] > 0.0) my_last = (c0 + j) * EPV + e;
                }
            }
            my_total += st;
            if (c0 == my0) slot_total[j] = st;
        }
    }
    const double incl_wave = wave_inclusive_scan(my_total, lane);
    if (lane == 63) sh.scan_total[wave] = incl_wave;
    __syncthreads();
    double before_wave = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        if (w < wave) before_wave += sh.scan_total[w];
    const double run_incl = base + (before_wave + incl_wave);
    const double run_excl = base + (before_wave + (incl_wave - my_total));
    note_first_and_last(!forced && run_incl > t && my_total > 0.0, my_last, &sh.first_thread, &sh.last_positive);
    __syncthreads();
    if ((int)threadIdx.x == sh.first_thread) {  // at most one thread
        double c = run_excl;
        int tok = -1, edge = 0;
        double before = c, after = c;
        auto walk_slot = [&](int slot, const u32x4 &vp, const u32x4 &vq) __attribute__((always_inline)) {
            double w[EPV];
            if constexpr (FAST) {
                float wf[EPV];
                (void)tree_slot_weights_f32<BF16, KIND>(vp, vq, fn, fd, p, wf);
#pragma unroll
                for (int e = 0; e < EPV; ++e) w[e] = (double)wf[e];
            } else {
                tree_slot_weights<BF16, KIND>(vp, vq, Mp, Cp, Mq, Cq, d, p, w);
            }
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                if (tok < 0) {
                    const double cn = c + w[e];
                    if (cn > t) {
                        tok = slot * EPV + e;
                        before = c;
                        after = cn;
                    }
                    c = cn;
                }
            }
        };
        // first chunk: skip whole slots by their totals, walk only the slot of the crossing
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
            if (tok < 0 && my0 + j < my1) {
                const double cn = c + slot_total[j];
                if (cn > t) {
                    const u32x4 vp = any_slot(rowp, my0 + j);
                    u32x4 vq = vp;
                    if constexpr (two) vq = any_slot(rowq, my0 + j);
                    walk_slot(my0 + j, vp, vq);
                    // (a crossing lost to rounding inside the slot carries on with the next one)
                } else {
                    c = cn;
                }
            }
        }
        for (int c0 = my0 + kChunk; c0 < my1 && tok < 0; c0 += kChunk) {
            u32x4 vp[kChunk], vq[kChunk];
            load_chunk(c0, vp, vq);
#pragma unroll
            for (int j = 0; j < kChunk; ++j) walk_slot(c0 + j, vp[j], vq[j]);
        }
        if (tok < 0) {  // the thread's own walk rounds differently from the block scan
            tok = my_last;
            edge = 1;
        } else {
            const double lo = fabs(t - before), hi = fabs(after - t);
            if (fmin(lo, hi) <= kBoundaryEps * Z) edge = 1;
        }
        sh.token = tok;
        sh.near_edge = edge;
    }
    __syncthreads();
    int tok = sh.token;
    near_edge = sh.near_edge;
    if (tok < 0) {  // no thread saw the crossing (forced, or it fell off the region's end)
        tok = sh.last_positive;
        near_edge = 1;
    }
    __syncthreads();
    return v.lo * EPV + tok;
}

template <bool BF16, bool ONE_TERM, bool FULL, bool PARTIAL, bool SHARED>
__device__ __forceinline__ void tree_rejection_sample(const TreeParams &p) {
    static_assert(FULL || !SHARED, "the guarded form is not shared");
    constexpr bool kWord = candidate_by_word(BF16, FULL && !PARTIAL);
    __shared__ SharedState sh;
    __shared__ uint32_t sh_epoch;
    __shared__ int sh_parent[kMaxTreeRows];
    __shared__ double sh_inv_z[kMaxTreeRows];
    __shared__ int sh_token[kMaxTreeRows];
    __shared__ float sh_u[kMaxTreeRows];
    constexpr int EPV = Elem<BF16>::EPV;
    const int split = SHARED ? p.split : 1;
    const int b = blockIdx.x / split, part = blockIdx.x % split;
    Mailbox mb{nullptr, nullptr, 0u, part, split, 0, 0u, &sh_epoch, false};
    if constexpr (SHARED) {
        uint32_t epoch;
        const bool alone = !claim_meet(claim_box(p.claim, b), p.claim, part, split, p.claim_ticks, &sh_epoch, sh, epoch);  // block-uniform
        if (alone && part != 0) return;
        mb = claim_mailbox(claim_box(p.claim, b), part, split, epoch, &sh_epoch, alone);
    }
    // bounds come from device data: clamp them by the host-side totals so that no value of
    // q_indptr or parent can push a row outside the logits buffers
    const int row0 = max(0, min(p.q_indptr[b], p.total_q - 1));
    const int R = max(1, min(p.q_indptr[b + 1] - row0, min(kMaxTreeRows, p.total_q - row0)));
    const PartView own = part_view<BF16>(p.V, part, split);  // this block's part of the vocabulary
    const size_t esz = BF16 ? 2 : 4;
    const char *tbase = static_cast<const char *>(p.target);
    const char *dbase = static_cast<const char *>(p.draft);
    // (the output rows are addressed where they are written and the final uniform is loaded where
    // it is used: values that live across the streaming passes cost registers there)
    auto out_row = [&]() { return p.out_tokens + (size_t)b * (p.max_depth + 1); };
    auto path_row = [&]() { return p.out_path + (size_t)b * max(p.max_depth, 1); };
    if (threadIdx.x < kMaxTreeRows) {
        sh_parent[threadIdx.x] = (int)threadIdx.x < R ? p.parent[row0 + threadIdx.x] : -2;
        sh_inv_z[threadIdx.x] = 1.0;
        if (threadIdx.x > 0 && (int)threadIdx.x < R) {  // (the root has neither a token nor a test)
            sh_token[threadIdx.x] = max(0, min(p.node_tokens[row0 + threadIdx.x], p.V - 1));  // memory safety only; ids outside [0,V) are a caller error
            sh_u[threadIdx.x] = p.u_accept[row0 + threadIdx.x];
        }
    }
    __syncthreads();

    int cur = 0, n = 0, flag_accept = 0, flag_cdf = 0, final_token = -1, parity = 0;
    // the walk ends at a node whose running distribution (depth, its normalisers) the final token
    // is drawn from; the passes that the draw needs stand once, behind the walk
    const char *rowp = tbase, *rowq = dbase;
    float Mp = 0.f, Mq = 0.f;
    double Sp = 1.0, Sq = 1.0;
    double raw_1 = 1.0;        // what the pass behind the node's first rejection summed (see FastDepth)
    int depth = 0;
    bool have_totals = false;  // sh.wave_total holds the running distribution's region totals
    bool have_norm = false;    // Mp, Sp belong to the node
    for (int guard = 0; guard < kMaxTreeRows; ++guard) {  // `cur` grows with every turn
        rowp = tbase + (size_t)(row0 + cur) * p.ld_t * esz;
        rowq = dbase + (size_t)(row0 + cur) * p.ld_d * esz;
        depth = 0;
        have_totals = have_norm = false;
        int c = cur + 1;
        while (c < R && sh_parent[c] != cur) ++c;
        if (c >= R || n >= p.max_depth) break;  // a leaf (or the output row is full): draw from the target
        Candidate cand{};
        int x = 0;
        auto fetch = [&]() __attribute__((always_inline)) {  // child c's token and its logits
            x = __builtin_amdgcn_readfirstlane(sh_token[c]);
            cand = fetch_candidate<BF16, kWord>(rowp, rowq, x);
        };
        row_stats_any<BF16, true, ONE_TERM, FULL, SHARED, PARTIAL, kThreads, SHARED>(rowp, rowq, own, p.V, sh, parity, mb, p, Mp, Sp, Mq, Sq, fetch);
        parity ^= 1;
        have_norm = true;
        bool moved = false;
        double Zd = 1.0;  // normaliser of the running distribution (Z_depth)
        while (c < R) {
            const float zpx = candidate_logit<BF16, kWord>(cand.p, rowp, x), zqx = candidate_logit<BF16, kWord>(cand.q, rowq, x);
            const double u = (double)sh_u[c];
            // Eq. 1 in fp64 against the running distribution: rho = p_depth(x)/q(x)
            double rho;
            if (depth == 0) {
                if (zqx == -INFINITY)
                    rho = (zpx == -INFINITY) ? 0.0 : (double)INFINITY;
                else
                    rho = exp((((double)zpx - (double)Mp) - ((double)zqx - (double)Mq)) * p.inv_T) * (Sq / Sp);
            } else {
                const double px = exp(((double)zpx - (double)Mp) * p.inv_T) / Sp;
                const double qx = exp(((double)zqx - (double)Mq) * p.inv_T) / Sq;
                const Depth d{depth, lane_value(sh_inv_z[1], 0), lane_value(sh_inv_z[2], 0), sh_inv_z};
                const double a = running_weight(px, qx, d) / Zd;
                if (qx == 0.0)
                    rho = a > 0.0 ? (double)INFINITY : 0.0;
                else
                    rho = a / qx;
            }
            const double thr = rho < 1.0 ? rho : 1.0;
            if (fabs(u - thr) <= kBoundaryEps) flag_accept = 1;
            if (u < thr) {  // accepted: the child becomes the node
                if (threadIdx.x == 0 && part == 0) {
                    out_row()[n] = x;
                    path_row()[n] = c;
                }
                n += 1;
                cur = c;
                moved = true;
                break;
            }
            // rejected: the running distribution becomes max(0, p_depth - q)/Z (Eq. 2)
            depth += 1;
            ++c;
            while (c < R && sh_parent[c] != cur) ++c;
            auto fetch_next = [&]() __attribute__((always_inline)) {
                if (c < R) fetch();
            };
            {
                const Depth d{depth, lane_value(sh_inv_z[1], 0), lane_value(sh_inv_z[2], 0), sh_inv_z};
                if (depth == 1) {
                    raw_1 = tree_region_totals<BF16, FULL, ONE_TERM, PARTIAL, 1, SHARED>(rowp, rowq, own, p.V, Mp, Sp, Mq, Sq, d, raw_1, sh, mb, p, fetch_next);
                    Zd = raw_1;
                    if constexpr (ONE_TERM) Zd += raw_1 * (double)make_fast_norm(Mp, Sp, Mq, Sq, p).ep;
                } else if (depth == 2) {
                    Zd = tree_region_totals<BF16, FULL, ONE_TERM, PARTIAL, 2, SHARED>(rowp, rowq, own, p.V, Mp, Sp, Mq, Sq, d, raw_1, sh, mb, p, fetch_next);
                    if constexpr (ONE_TERM) Zd /= raw_1;
                } else {
                    Zd = tree_region_totals<BF16, FULL, ONE_TERM, PARTIAL, kAnyDepth, SHARED>(rowp, rowq, own, p.V, Mp, Sp, Mq, Sq, d, raw_1, sh, mb, p, fetch_next);
                }
            }
            if (Zd > 0.0) {
                have_totals = true;
                if (threadIdx.x == 0 && depth < kMaxTreeRows) sh_inv_z[depth] = 1.0 / Zd;
            } else {  // an exact tie, impossible in exact arithmetic: start again from the target
                depth = 0;
                Zd = 1.0;
                have_totals = false;
                flag_cdf = 1;
            }
            __syncthreads();
        }
        if (!moved) break;  // every child was rejected: one draw from the running distribution
    }
    const Depth d{depth, lane_value(sh_inv_z[1], 0), lane_value(sh_inv_z[2], 0), sh_inv_z};
    double Z = 1.0;
    if (!have_totals) {  // a leaf, or an exact tie: the target row itself
        // At a leaf one pass serves instead of two: the draw compares running sums with u times
        // their total, so any reference that keeps the weights in range will do; a total that is
        // not a positive finite number sends the draw the ordinary way (normalisers first).
        bool trial = FULL && !have_norm;
        if (trial) {
            Mp = block_max_of_row_start<BF16, !PARTIAL, kRefSlots<ONE_TERM>>(rowp, p.V / EPV, sh);
            Sp = 1.0;
            trial = Mp > -INFINITY && Mp < INFINITY;  // block-uniform
        }
        for (;;) {
            if (!trial && !have_norm) {
                row_stats_any<BF16, false, ONE_TERM, FULL, SHARED, PARTIAL, kThreads, SHARED>(rowp, rowp, own, p.V, sh, parity, mb, p, Mp, Sp, Mq, Sq);
                have_norm = true;
            }
            Z = tree_region_totals<BF16, FULL, ONE_TERM, PARTIAL, 0, SHARED>(rowp, rowp, own, p.V, Mp, Sp, Mp, Sp, d, raw_1, sh, mb, p);
            if (!trial || (Z > 0.0 && Z < 1.0e300)) break;
            trial = false;
        }
    }
    bool mine = part == 0;
    if (Z > 0.0) {
        const double u = (double)p.u_final[b];
        int edge = 0;
        if (depth == 0)
            final_token = tree_draw<BF16, FULL, ONE_TERM, PARTIAL, 0, SHARED>(rowp, rowp, own, p.V, Mp, Sp, Mp, Sp, d, raw_1, u, sh, mb, p, edge, mine);
        else if (depth == 1)
            final_token = tree_draw<BF16, FULL, ONE_TERM, PARTIAL, 1, SHARED>(rowp, rowq, own, p.V, Mp, Sp, Mq, Sq, d, raw_1, u, sh, mb, p, edge, mine);
        else if (depth == 2)
            final_token = tree_draw<BF16, FULL, ONE_TERM, PARTIAL, 2, SHARED>(rowp, rowq, own, p.V, Mp, Sp, Mq, Sq, d, raw_1, u, sh, mb, p, edge, mine);
        else
            final_token = tree_draw<BF16, FULL, ONE_TERM, PARTIAL, kAnyDepth, SHARED>(rowp, rowq, own, p.V, Mp, Sp, Mq, Sq, d, raw_1, u, sh, mb, p, edge, mine);
        flag_cdf |= edge;
    } else {  // row without any finite logit: report the last token
        final_token = p.V - 1;
        flag_cdf = 1;
    }
    if (threadIdx.x == 0) {
        const bool failed = SHARED && sh.failed != 0;  // a wait for a part that was there ran out
        if (mine) {
            int32_t *out = out_row(), *path = path_row();
            out[n] = final_token;
            for (int j = n + 1; j <= p.max_depth; ++j) out[j] = -1;
            for (int j = n; j < p.max_depth; ++j) path[j] = -1;
            p.out_num_accepted[b] = failed ? -1 : n;
            if (p.out_flags) p.out_flags[b] = (flag_accept ? 1 : 0) | (flag_cdf ? 2 : 0);
        } else if (failed) {
            p.out_num_accepted[b] = -1;
        }
        if constexpr (SHARED) {
            if (!mb.alone && !failed) claim_leave(claim_box(p.claim, b), split, mb.epoch);
        }
    }
}

template <bool BF16, bool ONE_TERM, bool FULL>
__global__ __launch_bounds__(kThreads) void tree_rejection_sample_kernel(TreeParams p) {
    tree_rejection_sample<BF16, ONE_TERM, FULL, false, false>(p);
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void shared_tree_kernel(TreeParams p) {
    tree_rejection_sample<BF16, true, true, false, true>(p);
}

// Rows that are not whole aligned slots (fp64 weights); shared sequences with a two-term constant take it for
// any rows.
template <bool BF16, bool SHARED>
__global__ __launch_bounds__(kThreads) void tree_partial_rows_kernel(TreeParams p) {
    tree_rejection_sample<BF16, false, true, true, SHARED>(p);
}

}  // namespace
}  // namespace respec

extern "C" respec_status_t respec_tree_rejection_sample(
    const void *target_logits, const void *draft_logits, const int32_t *node_tokens, const int32_t *parent,
    const int32_t *q_indptr, const float *u_accept, const float *u_final, int32_t *out_tokens,
    int32_t *out_path, int32_t *out_num_accepted, int32_t *out_flags, int32_t B, int32_t total_q,
    int32_t max_q_per_seq, int32_t max_depth, int32_t V, int64_t ld_t, int64_t ld_d, float temperature,
    respec_dtype_t logits_dt, void *hip_stream) {
    using namespace respec;
    if (B <= 0 || total_q < B || max_depth < 0 || V <= 0)
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: need B > 0, total_q >= B, max_depth >= 0, V > 0 "
                    "(B=%d total_q=%d max_depth=%d V=%d)", B, total_q, max_depth, V);
    if (max_q_per_seq < 1 || (int64_t)max_q_per_seq * B < total_q)
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: max_q_per_seq too small for total_q");
    if (max_q_per_seq > kMaxTreeRows)
        return fail(RESPEC_ERR_UNSUPPORTED, "tree_rejection_sample: at most %d rows per sequence (got %d)",
                    kMaxTreeRows, max_q_per_seq);
    if (!(temperature > 0.f) || !std::isfinite(temperature))
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: temperature must be finite and > 0");
    if (logits_dt != RESPEC_F32 && logits_dt != RESPEC_BF16)
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: unknown logits dtype %d", (int)logits_dt);
    if (!target_logits || !draft_logits || !node_tokens || !parent || !q_indptr || !u_accept || !u_final ||
        !out_tokens || !out_path || !out_num_accepted)
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: null pointer argument");
    if (ld_t < V || ld_d < V)
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: row stride smaller than V");
    const size_t esz = logits_dt == RESPEC_BF16 ? 2 : 4;
    if (!aligned_to(target_logits, esz) || !aligned_to(draft_logits, esz))
        return fail(RESPEC_ERR_INVALID_ARG, "tree_rejection_sample: logits pointer not element aligned");

    TreeParams p{};
    p.target = target_logits;
    p.draft = draft_logits;
    p.node_tokens = node_tokens;
    p.parent = parent;
    p.q_indptr = q_indptr;
    p.u_accept = u_accept;
    p.u_final = u_final;
    p.out_tokens = out_tokens;
    p.out_path = out_path;
    p.out_num_accepted = out_num_accepted;
    p.out_flags = out_flags;
    p.B = B;
    p.total_q = total_q;
    p.max_depth = max_depth;
    p.V = V;
    p.ld_t = ld_t;
    p.ld_d = ld_d;
    set_row_math(p, temperature);

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int epv = logits_dt == RESPEC_BF16 ? 8 : 4;
    const bool full = V >= epv && knobs().get(&Knobs::sampler_guarded, 0) == 0;
    // (rows of whole, aligned slots take fp32 weights, the others keep fp64 ones, as in the chain sampler)
    const bool whole_rows = V % epv == 0 && aligned_to(target_logits, 16) && (ld_t * esz) % 16 == 0 &&
                            aligned_to(draft_logits, 16) && (ld_d * esz) % 16 == 0;
    p.one_term = p.one_term && whole_rows;
    const bool bf = logits_dt == RESPEC_BF16, one = p.one_term != 0;
    // Work-groups per sequence: while compute units are idle and a part keeps 4800 slots (fp32, half as many elements: 9216; two per
    // sequence on the whole device, which memory bounds: 6144, fp32 16,384); below, what a pass gets shorter by is less than meeting and
    // exchanging cost.  One work-group / shared, us per call, T = 0.6: 3 x 2 candidates, bf16, V = 151,936, B = 128 86.8 / 78.3, B = 64
    // 86.2 / 60.0, B = 1 55.7 / 40.2, V = 77,777, B = 100 74.2 / 65.5; V = 32,768, B = 64 36.0 / 41.9; fp32, V = 151,936, B = 64 90.3 / 71.1;
    // 2 x 2 candidates, bf16, V = 66,000, B = 64 and 128 42.8 / 44.1, 44.0 / 46.5, V = 80,000 and 110,000, B = 128 47.5 / 48.3, 57.6 / 57.8; fp32, B = 64, V = 66,000 and 74,000 40.8 / 41.8, 44.3 / 43.7,
    // B = 128, V = 66,000, 77,777, 110,000, 131,072 48.0 / 54.4, 58.8 / 59.8, 72.5 / 73.6, 85.4 / 83.2.
    p.split = 1;
    const Knobs kn = knobs();
    if (full && kn.get(&Knobs::sampler_claim, 1) != 0) {
        int dev = 0, cus = 256;
        if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        cus = std::min(cus, kClaimGroups);
        const long slots_row = ((long)V + epv - 1) / epv, least = (long)B * 4 > cus ? (bf ? 6144 : 16384) : (bf ? 4800 : 9216);
        while (p.split < kClaimSplit && (long)B * p.split * 2 <= cus && slots_row / (p.split * 2) >= least) p.split *= 2;
    }
    if (p.split > 1) {
        p.claim = next_claim_key();
        p.claim_ticks = (int)kn.get(&Knobs::sampler_claim_ticks, kClaimTicks);
    }
#define RESPEC_LAUNCH_TREE(KERNEL) hipLaunchKernelGGL(KERNEL, dim3((unsigned)(B * p.split)), dim3(kThreads), 0, stream, p)
    const bool shared = p.split > 1;
    if (!full) {
        if (bf) RESPEC_LAUNCH_TREE((tree_rejection_sample_kernel<true, false, false>));
        else RESPEC_LAUNCH_TREE((tree_rejection_sample_kernel<false, false, false>));
    } else if (shared && one) {
        if (bf) RESPEC_LAUNCH_TREE((shared_tree_kernel<true>));
        else RESPEC_LAUNCH_TREE((shared_tree_kernel<false>));
    } else if (shared) {
        if (bf) RESPEC_LAUNCH_TREE((tree_partial_rows_kernel<true, true>));
        else RESPEC_LAUNCH_TREE((tree_partial_rows_kernel<false, true>));
    } else if (!whole_rows) {
        if (bf) RESPEC_LAUNCH_TREE((tree_partial_rows_kernel<true, false>));
        else RESPEC_LAUNCH_TREE((tree_partial_rows_kernel<false, false>));
    } else {
        if (bf && one) RESPEC_LAUNCH_TREE((tree_rejection_sample_kernel<true, true, true>));
        else if (bf) RESPEC_LAUNCH_TREE((tree_rejection_sample_kernel<true, false, true>));
        else if (one) RESPEC_LAUNCH_TREE((tree_rejection_sample_kernel<false, true, true>));
        else RESPEC_LAUNCH_TREE((tree_rejection_sample_kernel<false, false, true>));
    }
#undef RESPEC_LAUNCH_TREE
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess)
        return fail(RESPEC_ERR_HIP, "tree_rejection_sample: launch failed: %s", hipGetErrorString(err));
    clear_error();
    return RESPEC_OK;
}
