// Speculative rejection sampling over the vocabulary (Section 2.2, Eq. 1 and Eq. 2) for
// gfx950.  A sequence is walked position by position: for each drafted position the target
// row and the drafter row are streamed once (16-byte loads, fp32 exp2, sums carried in
// fp64), the acceptance test is taken in fp64, and at the first rejection a second pass
// over that one row pair draws from max(0, p-q) by an ordered fp64 prefix scan.  Rows after
// the first rejection are never used (a shared sequence may have read the pair right behind
// the rejected position ahead of the test, see row_stats_two_items; short rows are read eight
// positions at a time).
//
// Parallelisation.  The chain of positions of one sequence is sequential and its length
// differs from sequence to sequence, so one work-group per sequence leaves most of the
// device idle when there are fewer sequences than compute units.  A sequence can therefore
// be shared by SPLIT work-groups (one per compute unit), each owning a
// contiguous part of the vocabulary.  After every streaming pass the parts exchange their
// partial results (a few numbers) through a small mailbox in the workspace and then take
// the same decision from the same numbers.  An exchange costs a few memory round trips, so
// sequences are shared only while that fills otherwise idle compute units (batches of at
// most half as many sequences as the device has compute units).  The mailbox is
// self-synchronising across calls (an epoch counter per sequence), so it only has to be
// zero before its first use.  Without a workspace a sequence of a call with one temperature gets
// one work-group and no mailbox is touched; calls with a temperature per sequence, which have no
// workspace, share their sequences through mailboxes of the library's own (respec_sampler_share.hpp).
//
// Numerics.  Token decisions are discontinuous in the sums, so everything that decides a
// token is carried in fp64; only exp2 of a single element runs in fp32 (hardware exp2,
// 1 ulp, argument formed as (z-ref)*log2(e)/T with a two-term constant so that no
// systematic error enters).  "ref" is a per-thread reference near the row maximum, not
// necessarily the maximum: fp32 keeps full relative precision for any offset, and the
// references are reconciled in fp64 when threads (and parts) are combined.
#include "respec_sampler_share.hpp"

#include <algorithm>
#include <type_traits>

namespace respec {
namespace {

// How a sequence is walked: by a work-group of its own, or by several that take one or two items of its chain per stage.
enum Share { kOwn, kOneAtATime, kTwoAtATime };

// Threads of a work-group.  The stages of two items share short passes that lie between reductions, barriers and
// exchanges, which cost less with half the waves, while four waves, one per SIMD, still reach most of the
// issue rate of eight (256 / 512 threads, us per call: bf16, V = 151,936, k = 4, T = 0.6, B = 64 43.1 / 45.7; V = 32,000
// 24.8 / 28.7; fp32, V = 50,257, B = 32, k = 2 22.9 / 23.8).  Longer passes want the eight (V = 151,936 in two parts, B = 128
// 56.0 / 53.7; whole rows at mixed temperatures, B = 256 110 / 96; trees 112 / 97).
constexpr int share_threads(int share) { return share == kTwoAtATime ? 256 : kThreads; }

struct SamplerParams : RowMath {
    const void *target;
    const void *draft;
    const int32_t *draft_tokens;
    const int32_t *q_indptr;
    const float *u_accept;
    const float *u_final;
    int32_t *out_tokens;
    int32_t *out_num_accepted;
    int32_t *out_flags;
    int32_t B, total_q, max_k, V;
    int64_t ld_t, ld_d;
    int split;         // work-groups per sequence
    char *boxes;       // [B] mailboxes of kBoxBytes in the workspace (split > 1 and claim == 0)
    const float *temps;  // [B] one temperature per sequence (0: greedy), or NULL: the RowMath constants hold
    int tab_slots;       // > 0: the launch carries dynamic LDS for one float per slot of a row
    uint32_t claim;      // > 0: the parts of a sequence meet in the library's own mailboxes, under this key, ...
    int claim_ticks;     // ... and wait for each other that long
};


// The normalisers of one row pair: references and sums of the p row and the q row.
struct DrawNorm {
    float Mp, Mq;
    double Sp, Sq;
};

// Shared sequences: the normalisers of two consecutive items of a chain in one
// stage.  Item A is the row pair of position i, item B the row pair of position i + 1 or, when
// i + 1 is past the last draft, the target row of the bonus token alone (b_pair false).  B is
// streamed before A's acceptance test is known: when A rejects, B's bytes were read for nothing,
// but a shared sequence runs on compute units that would otherwise idle, an exchange costs more
// than a part's pass over a row pair, and this halves the exchanges of a chain.
//
// Numbers that a part cannot vouch for (an overflow, or a sum of next to nothing beside a wave without a reference) are
// taken again by that part with the guarded pass, while the others wait in the exchange.  A part without
// any finite logit (most of the vocabulary masked) is no such case where two batches are all of it: a wave that finds none
// in the first takes kRefInit, against which a finite logit of the second overflows, so that a sum of 0 is one.  (When every
// part repeated such items twice, one by one: k = 4, all but the first sixth masked, bf16, V = 32,000, B = 64 83 us, now 24,
// nothing masked 23.5, by one work-group 28; V = 151,936, B = 64 158, now 84.)
//
// The two items are one stream of batches: B's first batch is requested ahead of A's last, and the
// four sums are reduced together behind one barrier (one pass after the other left the memory pipeline
// empty for 3 us of every stage).
// The rows' share of one part (pointers at its first slot): leaves its own normalisers in A and Bn.
template <bool BF16, bool ONE_TERM, bool PARTIAL, int TH, class Meanwhile>
__device__ __forceinline__ void part_stats_two_items(const char *pa, const char *qa, const char *pb, const char *qb,
                                                     bool b_pair, int nslots_all, int Vrow, SharedState &sh,
                                                     const SamplerParams &p, DrawNorm &A, DrawNorm &Bn, Meanwhile &&meanwhile) {
    constexpr int EPV = Elem<BF16>::EPV, kThreads = TH, kWaves = TH / 64, kBatch = kThreads * kUnroll;
    A.Mp = A.Mq = Bn.Mp = Bn.Mq = kRefInit;
    A.Sp = A.Sq = Bn.Sp = Bn.Sq = 0.0;
    if (nslots_all > 0) {  // (a part without slots has nothing to read and no mass)
        const int nslots = PARTIAL ? whole_slots<BF16>(nslots_all, Vrow) : nslots_all;
        const int tid = opaque_thread_index(), lane = tid & 63, wave = threadIdx.x >> 6;
        const int n = (nslots + kBatch - 1) / kBatch;  // batches of an item; block-uniform, >= 1
        const float no_ref = n <= 2 ? kRefInit : 0.f;
        float ref[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, acc[2][EPV], K[2] = {0.f, 0.f};  // [item][p/q]; acc, K: the current item's
        double sum[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
        u32x4 part_slot[2][2];
        if constexpr (PARTIAL) {
            if (nslots < nslots_all) {  // block-uniform
                part_slot[0][0] = load_slot_or_last<BF16>(pa, nslots, Vrow);
                part_slot[0][1] = load_slot_or_last<BF16>(qa, nslots, Vrow);
                part_slot[1][0] = load_slot_or_last<BF16>(pb, nslots, Vrow);
                part_slot[1][1] = load_slot_or_last<BF16>(qb, nslots, Vrow);
            }
        }
        // batch `it` of the stream, clamped to the rows; unconditional (see row_stats_fast).  Without a
        // drafter row in B its target row is requested twice, the second time from a cache.
        auto load_batch = [&](int it, u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
            it = min(it, 2 * n - 1);
            const void *rowp = it < n ? pa : pb, *rowq = it < n ? qa : qb;
            const int s0 = (it < n ? it : it - n) * kBatch + tid;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int safe = max(0, min(s0 + u * kThreads, nslots - 1));
                vp[u] = load_slot<BF16, true, false, !PARTIAL>(rowp, safe, Vrow);
                vq[u] = load_slot<BF16, true, false, !PARTIAL>(rowq, safe, Vrow);
            }
        };
        // every condition below is block-uniform
        auto sum_batch = [&](int it, u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
            const int item = it < n ? 0 : 1, at = it - item * n;
            const bool two = item == 0 || b_pair;
            if (at == n - 1) {  // an item's last batch: slots past the row are inert
                const int s0 = at * kBatch + tid;
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const bool in = s0 + u * kThreads < nslots;
                    vp[u] = in ? vp[u] : neg_inf_slot<BF16>();
                    vq[u] = in ? vq[u] : neg_inf_slot<BF16>();
                }
            }
            if (at == 0) {  // its first: the references
                float m[2] = {-INFINITY, -INFINITY};
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    m[0] = fmaxf(m[0], slot_max<BF16>(vp[u]));
                    m[1] = fmaxf(m[1], slot_max<BF16>(vq[u]));
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const float w = wave_max(m[r]);
                    const float f = (w > -INFINITY && w < INFINITY) ? w : no_ref;
                    K[r] = -f * p.c_f;
                    if (item == 0) ref[0][r] = f; else ref[1][r] = f;
#pragma unroll
                    for (int j = 0; j < EPV; ++j) acc[r][j] = 0.f;
                }
            }
            const float rp = item == 0 ? ref[0][0] : ref[1][0], rq = item == 0 ? ref[0][1] : ref[1][1];
            if (two && at < n - 1) {
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    fast_absorb<BF16, ONE_TERM>(vp[u], acc[0], rp, K[0], p);
                    fast_absorb<BF16, ONE_TERM>(vq[u], acc[1], rq, K[1], p);
                }
            } else {
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    if (at * kBatch + u * kThreads >= nslots) break;  // (nothing of the row in this group of slots)
                    fast_absorb<BF16, ONE_TERM>(vp[u], acc[0], rp, K[0], p);
                    if (two) fast_absorb<BF16, ONE_TERM>(vq[u], acc[1], rq, K[1], p);
                }
            }
            if (at == n - 1) {
                if (PARTIAL && nslots < nslots_all && tid == 0) {
                    fast_absorb<BF16, ONE_TERM>(partial_slot<BF16>(item == 0 ? part_slot[0][0] : part_slot[1][0], nslots, Vrow), acc[0], rp, K[0], p);
                    if (two) fast_absorb<BF16, ONE_TERM>(partial_slot<BF16>(item == 0 ? part_slot[0][1] : part_slot[1][1], nslots, Vrow), acc[1], rq, K[1], p);
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    double t = 0.0;
#pragma unroll
                    for (int j = 0; j < EPV; ++j) t += (double)acc[r][j];
                    if (PARTIAL && t > kFastMost) t = (double)INFINITY;
                    if (item == 0) sum[0][r] = t; else sum[1][r] = t;
                }
            }
        };
        u32x4 vp[2][kUnroll], vq[2][kUnroll];  // one set is summed while the other's loads are in flight
        load_batch(0, vp[0], vq[0]);
        meanwhile();
        for (int it = 0; it < 2 * n; it += 2) {
            load_batch(it + 1, vp[1], vq[1]);
            sum_batch(it, vp[0], vq[0]);
            load_batch(it + 2, vp[0], vq[0]);
            sum_batch(it + 1, vp[1], vq[1]);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const double s = wave_sum(sum[x >> 1][x & 1]);
            if (lane == 0) {
                sh.m[x >> 1][x & 1][wave] = ref[x >> 1][x & 1];
                sh.s[x >> 1][x & 1][wave] = s;
            }
        }
        __syncthreads();
        // lane group x: (item, p/q) = x; one exp2 per lane (see block_combine_fast)
        const int x = (lane / kWaves) & 3, w = lane & (kWaves - 1);
        const float my_m = sh.m[x >> 1][x & 1][w], mm = group_max<kWaves>(my_m);
        double e = (double)(my_m - mm) * p.c_d;
        if constexpr (ONE_TERM) e -= (double)(-my_m * p.c_f) + (double)my_m * (double)p.c_f;
        const double s_w = sh.s[x >> 1][x & 1][w];
        const double part = group_sum<kWaves>(s_w != 0.0 ? s_w * exp2_f64(e) : 0.0);  // (kRefInit c_f is rounded to 2^76)
        const bool sound = (part > kFastLeast && part < 1.0e300) || (part == 0.0 && mm == kRefInit);
        const unsigned long long doubts = __ballot(!sound && (x < 3 || b_pair)) & ((1ull << (4 * kWaves)) - 1);
        A.Mp = lane_value(mm, 0), A.Mq = lane_value(mm, kWaves), Bn.Mp = lane_value(mm, 2 * kWaves);
        A.Sp = lane_value(part, 0), A.Sq = lane_value(part, kWaves), Bn.Sp = lane_value(part, 2 * kWaves);
        if (b_pair) {
            Bn.Mq = lane_value(mm, 3 * kWaves);
            Bn.Sq = lane_value(part, 3 * kWaves);
        }
#pragma unroll 1
        for (int item = 0; item < 2; ++item) {
            if (__builtin_expect(((doubts >> (item * 2 * kWaves)) & ((1ull << (2 * kWaves)) - 1)) == 0, 1)) continue;  // block-uniform
            // (the guarded pass a slot at a time: as unrolled as row_stats it is 20 KB of instructions in the way of every call)
            const void *rowp = item == 0 ? pa : pb, *rowq = item == 0 ? qa : qb;
            ThreadSum<BF16> t[2];
            t[0].init();
            t[1].init();
            auto load = [&](const void *row, int s) __attribute__((always_inline)) {
                if constexpr (!PARTIAL) return load_slot<BF16, true, false, true>(row, s, Vrow);
                const u32x4 v = load_slot_or_last<BF16>(row, s, Vrow);
                return s < nslots ? v : partial_slot<BF16>(v, nslots, Vrow);
            };
#pragma unroll 1
            for (int s = tid; s < nslots_all; s += kThreads) {
                const u32x4 vp = load(rowp, s), vq = load(rowq, s);
                t[0].absorb(vp, p);
                t[1].absorb(vq, p);
            }
            __syncthreads();  // every thread has read the combine buffers
            DrawNorm d;
            block_combine<TH>(t[0].ref, t[0].total(), sh, item, 0, p, d.Mp, d.Sp);
            block_combine<TH>(t[1].ref, t[1].total(), sh, item, 1, p, d.Mq, d.Sq);
            if (item == 0) A = d; else Bn = d;
        }
    } else {
        meanwhile();
        __syncthreads();  // (as in row_stats_any)
    }
}

// (the rows from their starts)
template <bool BF16, bool ONE_TERM, bool PARTIAL, int TH, bool MEETS, class Meanwhile>
__device__ inline void row_stats_two_items(const char *pa, const char *qa, const char *pb, const char *qb, bool b_pair,
                                           const PartView &own, SharedState &sh, Mailbox &mb, const SamplerParams &p,
                                           DrawNorm &A, DrawNorm &Bn, Meanwhile &&meanwhile) {
    for_parts<BF16, MEETS>(mb, own, p.V, sh, [&](int, const PartView &v, double(&mine)[8]) __attribute__((always_inline)) {
        const size_t at = (size_t)v.lo * 16;
        part_stats_two_items<BF16, ONE_TERM, PARTIAL, TH>(pa + at, qa + at, pb + at, qb + at, b_pair, v.nslots, v.Vrow, sh, p, A, Bn,
                                                          meanwhile);
        // two binary32 references travel as the halves of one 8-byte word (moved, never computed with)
        auto pack = [](float lo, float hi) {
            return __builtin_bit_cast(double, (unsigned long long)__float_as_uint(lo) |
                                                  ((unsigned long long)__float_as_uint(hi) << 32));
        };
        mine[0] = pack(A.Mp, A.Mq), mine[1] = A.Sp, mine[2] = A.Sq;
        mine[3] = pack(Bn.Mp, Bn.Mq), mine[4] = Bn.Sp, mine[5] = Bn.Sq;
        mine[6] = mine[7] = 0.0;
    });
    // in every wave (see row_stats_any): lane 8 (2 item + row) + j: part j; one exp2 per lane
    const int g = (threadIdx.x / kMaxSplit) & 3, j = threadIdx.x & (kMaxSplit - 1);
    const int item = g >> 1, r = g & 1;
    const bool have = j < mb.split;
    float m_j = -INFINITY;
    if (have) {
        const unsigned long long w = __builtin_bit_cast(unsigned long long, sh.xchg[j][3 * item]);
        m_j = __uint_as_float((uint32_t)(r ? w >> 32 : w & 0xffffffffull));
    }
    const float M = group_max<kMaxSplit>(m_j);
    const double S = group_sum<kMaxSplit>(have ? sh.xchg[j][3 * item + 1 + r] * exp2_f64(((double)m_j - (double)M) * p.c_d) : 0.0);
    A.Mp = lane_value(M, 0), A.Mq = lane_value(M, kMaxSplit);
    A.Sp = lane_value(S, 0), A.Sq = lane_value(S, kMaxSplit);
    Bn.Mp = lane_value(M, 2 * kMaxSplit), Bn.Mq = lane_value(M, 3 * kMaxSplit);
    Bn.Sp = lane_value(S, 2 * kMaxSplit), Bn.Sq = lane_value(S, 3 * kMaxSplit);
}

// fp64 weights of one slot, times Sp: p(x) (RESID = false) or max(0, p(x) - q(x)) (Eq. 2), that is
// max(0, pe - qe g) with g = Sp / Sq.  (A draw only compares running sums with u times their total.  Multiplying both
// exponentials by their normalisers' reciprocals took two operations more per element of this pass, which is
// bound by instruction issue, and rounded twice more.)
template <bool BF16, bool RESID>
__device__ inline void slot_weights(const u32x4 &vp, const u32x4 &vq, float Mp, float Mq, double g, const RowMath &p,
                                    double (&w)[Elem<BF16>::EPV]) {
    constexpr int EPV = Elem<BF16>::EPV;
    float zp[EPV], zq[EPV];
    unpack<BF16>(vp, zp);
    if constexpr (RESID) unpack<BF16>(vq, zq);
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
        const double pe = (double)hw_exp2(exp2_arg(zp[j], Mp, p.c_hi, p.c_lo));
        if constexpr (RESID) {
            const double qe = (double)hw_exp2(exp2_arg(zq[j], Mq, p.c_hi, p.c_lo));
            w[j] = fmax(fma(-qe, g, pe), 0.0);
        } else {
            w[j] = pe;
        }
    }
}

// The same weights in fp32, for calls whose exponent constant rounds well (RowMath::one_term):
// p(x) = exp2(z c_f + K) (1 + e) with K + log2(1 + e) = -M c_f - log2(S) split so that the
// rounding of K is put back to first order; the weights of a slot are summed in fp32 in a
// fixed pairwise order, and everything above a slot is carried in fp64.  A draw only compares
// running sums with u times their total, so the weights may carry a common factor: they are
// formed as w / (1 + ep), that is pe - qe (1 + eq - ep) for Eq. 2 and plain pe for a row of p,
// which takes one correction per pair of elements instead of two.  A weight is within a few
// 1e-7 (relative) of its fp64 value (times the common factor), far inside the boundary band of
// 1e-6; the scan is bound by instruction issue, and this form needs about half of the
// instructions.  Returns the slot's total (fp32, pairwise); w[] are its elements' weights.
template <bool BF16, bool RESID>
__device__ inline float slot_weights_f32(const u32x4 &vp, const u32x4 &vq, const FastNorm &f, const RowMath &p,
                                         float (&w)[Elem<BF16>::EPV]) {
    constexpr int EPV = Elem<BF16>::EPV;
    float zp[EPV], zq[EPV];
    unpack<BF16>(vp, zp);
    if constexpr (RESID) unpack<BF16>(vq, zq);
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
        const float pe = hw_exp2(fmaf(zp[j], p.c_f, f.Kp));
        if constexpr (RESID) {
            const float qe = hw_exp2(fmaf(zq[j], p.c_f, f.Kq));
            w[j] = fmaxf(fmaf(-qe, f.e_rel, pe - qe), 0.f);
        } else {
            w[j] = pe;
        }
    }
    if constexpr (EPV == 8)
        return ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
    else
        return (w[0] + w[1]) + (w[2] + w[3]);
}

// The single final draw of a sequence: first token, in ascending id, whose running sum of
// weights exceeds u*Z (all sums in fp64).
//   phase A  (draw_region_totals) each wave owns a contiguous eighth of the part at hand and
//            streams it with coalesced loads; lanes keep their own fp64 sums, one reduction per
//            wave gives the region total;
//   choice   every thread takes the ordered prefix over the region totals of the whole row and
//            finds the region that holds the crossing;
//   phase B  the whole block re-reads that one region, each thread a short contiguous run of
//            slots: thread totals -> one block scan -> the first thread whose running sum
//            passes u*Z walks its run element by element.
// Phase B adds the same numbers in another order than phase A, so at the last bit a crossing
// can fall off the end of the region; that draw then takes the last token with mass and is
// flagged as a boundary draw (it is within rounding of a CDF edge).

// One contiguous part of a row (pair) as a block sees it: pointers at the part's first slot.
struct RowPart {
    const void *rowp;
    const void *rowq;
    int nslots;   // slots of the part
    int Vrow;     // elements from the part's first slot to the end of the row
    int tok_off;  // token id of the part's first element
    float *tab;   // LDS room for one float per slot of the part (fp32 form of the weights), or NULL
};

// Phase A over one part: leaves the waves' region totals in sh.wave_total (no barrier), and with
// a table every slot's total in part.tab.
template <bool BF16, bool RESID, bool FULL, bool FAST, bool PARTIAL, int TH>
__device__ inline void draw_region_totals(const RowPart &part, const DrawNorm &nm, SharedState &sh,
                                          const RowMath &p) {
    constexpr int kWaves = TH / 64;
    constexpr int EPV = Elem<BF16>::EPV;
    const int lane = opaque_thread_index() & 63, wave = threadIdx.x >> 6;
    const void *rowp = part.rowp, *rowq = part.rowq;
    const int nslots = part.nslots, Vrow = part.Vrow;
    float *tab = part.tab;
    const float Mp = nm.Mp, Mq = nm.Mq;
    const double Sp = nm.Sp, Sq = nm.Sq;
    // FAST with a table: phase A leaves every slot's total there, and phase B works from the
    // table instead of reading the region again.
    const bool use_tab = FAST && tab != nullptr;  // block-uniform
    const double g = RESID ? Sp / Sq : 0.0;
    const int span = ((nslots + kWaves - 1) / kWaves + 63) / 64 * 64;
    const int whole = PARTIAL ? whole_slots<BF16>(nslots, Vrow) : nslots;
    const int beg = min(wave * span, nslots), end_all = min(beg + span, nslots), end = min(end_all, whole);

    // phase A: region totals (the next batch of slots is in flight while one is summed; batches
    // twice as long measured the same)
    double lane_sum = 0.0;
    // (no select behind a load: it would make the loads of a batch wait for one another; slots
    // past the region are replaced by -inf when the batch is summed)
    auto load_batch = [&](int s0, u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kUnroll; ++c) {
            const int slot = s0 + c * 64 + lane;
            vp[c] = load_slot<BF16, FULL, true, FULL && !PARTIAL>(rowp, slot < end ? slot : beg, Vrow);
            if constexpr (RESID) vq[c] = load_slot<BF16, FULL, true, FULL && !PARTIAL>(rowq, slot < end ? slot : beg, Vrow);
        }
    };
    if (beg < end) {  // wave-uniform
        // a ring of register sets: all but one are in flight while one is summed
        constexpr int NSETS = FULL ? kSetsDraw : 2;  // (the guarded loads of the general form need the registers)
        u32x4 rp[NSETS][kUnroll], rq[NSETS][kUnroll];
        // (the loads of the steady state are unconditional: behind a condition, the wait for the
        // batch in front of a load becomes a wait for everything in flight; batches past the
        // region read its first slot again and are never summed)
        constexpr int kStep = 64 * kUnroll;
#pragma unroll
        for (int s = 0; s + 1 < NSETS; ++s) load_batch(beg + s * kStep, rp[s], rq[s]);
        const FastNorm fn = make_fast_norm(Mp, Sp, Mq, RESID ? Sq : Sp, p);  // (two logarithms in the loads' shadow)
        // (whole: every slot of the batch lies inside the region, which holds for all batches but
        // a region's last; the selects that a ragged batch needs are a tenth of the loop)
        auto sum_batch = [&](int s0, const u32x4 (&xp)[kUnroll], const u32x4 (&xq)[kUnroll], auto whole) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < kUnroll; ++c) {
                if (!decltype(whole)::value && s0 + c * 64 >= end) break;  // wave-uniform
                const bool in = decltype(whole)::value || s0 + c * 64 + lane < end;
                const u32x4 a = in ? xp[c] : neg_inf_slot<BF16>();
                const u32x4 b = RESID ? (in ? xq[c] : neg_inf_slot<BF16>()) : a;
                if constexpr (FAST) {
                    float w[EPV];
                    const float ts = slot_weights_f32<BF16, RESID>(a, b, fn, p, w);
                    lane_sum += (double)ts;
                    if (use_tab && in) tab[s0 + c * 64 + lane] = ts;
                } else {
                    double w[EPV];
                    slot_weights<BF16, RESID>(a, b, Mp, Mq, g, p, w);
#pragma unroll
                    for (int j = 0; j < EPV; ++j) lane_sum += w[j];
                }
            }
        };
        const int n_b = (end - beg + kStep - 1) / kStep;  // wave-uniform, >= 1
        int ib = 0;  // set s holds batch ib + s for s < NSETS - 1
        for (; ib + NSETS < n_b; ib += NSETS) {
#pragma unroll
            for (int s = 0; s < NSETS; ++s) {
                constexpr int kAhead = NSETS - 1;
                load_batch(beg + (ib + s + kAhead) * kStep, rp[(s + kAhead) % NSETS], rq[(s + kAhead) % NSETS]);
                sum_batch(beg + (ib + s) * kStep, rp[s], rq[s], std::true_type{});
            }
        }
        const int rem = n_b - ib;  // 1..NSETS
        if (rem == NSETS) load_batch(beg + (ib + NSETS - 1) * kStep, rp[NSETS - 1], rq[NSETS - 1]);
#pragma unroll
        for (int s = 0; s < NSETS; ++s)
            if (s < rem) {
                if (beg + (ib + s + 1) * kStep <= end) sum_batch(beg + (ib + s) * kStep, rp[s], rq[s], std::true_type{});
                else sum_batch(beg + (ib + s) * kStep, rp[s], rq[s], std::false_type{});
            }
    }
    if constexpr (PARTIAL) {
        if (beg <= whole && whole < end_all && lane == 0) {  // the row's partial slot
            const u32x4 a = load_partial_slot<BF16>(rowp, whole, Vrow), b = RESID ? load_partial_slot<BF16>(rowq, whole, Vrow) : a;
            double w[EPV];
            slot_weights<BF16, RESID>(a, b, Mp, Mq, g, p, w);
#pragma unroll
            for (int j = 0; j < EPV; ++j) lane_sum += w[j];
        }
    }
    double region_total = wave_sum(lane_sum);
    // (The bound holds for weights against a reference that nothing is known of, those of the one-pass draw, whose
    // normaliser is taken as 1 and whose caller falls back.  A draw that has the normaliser adds up to at most that: it has
    // nothing to fall back to, and a sum of 2^41 may well be what the normaliser's pass found.)
    if (PARTIAL && region_total > kFastMost * Sp) region_total = (double)INFINITY;
    if (lane == 0) sh.wave_total[wave] = region_total;
}

// Choice and phase B.  `tot` are the region totals of the whole row in vocabulary order, a lane each
// (zero in the lanes behind them); the regions [my_reg0, my_reg0 + kWaves) are those of `part`, this block's part of the
// row.  SHARED: the totals are this block's weights times `scale` (and the other blocks' times
// theirs).  Returns the token, or -1 with mine = false when another block holds the crossing, or
// -1 with Z_out <= 0 when the row carries no mass.  Ends with a barrier.
template <bool BF16, bool RESID, bool FULL, bool FAST, bool SHARED, bool PARTIAL, int TH>
__device__ inline int draw_finish(double tot, int my_reg0, const RowPart &part,
                                  const DrawNorm &nm, double u, SharedState &sh, const RowMath &p, int &near_edge,
                                  double &Z_out, bool &mine, double scale) {
    constexpr int EPV = Elem<BF16>::EPV;
    constexpr int kThreads = TH, kWaves = TH / 64;
    static_assert(kMaxSplit * kWaves <= 64, "a wave holds the totals of all regions");
    const int lane = opaque_thread_index() & 63, wave = threadIdx.x >> 6;
    const float Mp = nm.Mp, Mq = nm.Mq;
    const double Sp = nm.Sp, Sq = nm.Sq;
    const double g = RESID ? Sp / Sq : 0.0;
    const FastNorm fn = make_fast_norm(Mp, Sp, Mq, RESID ? Sq : Sp, p);
    if (threadIdx.x == 0) {
        sh.token = -1;
        sh.near_edge = 0;
        sh.first_thread = kThreads;
        sh.last_positive = -1;
    }
    // every wave: ordered prefix over the regions, a lane each, and the region holding the crossing (one
    // thread after the other through 32 totals took 2 us of a shared draw)
    const double incl = wave_inclusive_scan(tot, lane);
    double Z = lane_value(incl, 63);
    Z_out = Z;
    mine = false;
    if (!(Z > 0.0)) {  // caller falls back (residual of an exact tie) or reports the last token
        __syncthreads();
        near_edge = 1;
        return -1;
    }
    double t = u * Z;
    const unsigned long long with_mass = __ballot(tot > 0.0), past = with_mass & __ballot(incl > t);
    const int rlast = with_mass != 0ull ? 63 - __builtin_clzll(with_mass) : 0;
    int rstar = past != 0ull ? __builtin_ctzll(past) : -1;
    double base = rstar > 0 ? lane_value(incl, rstar - 1) : 0.0;
    const bool forced = rstar < 0;  // u*Z rounded up to Z: take the last token with mass
    if (forced) rstar = rlast;
    __syncthreads();  // the totals may be rewritten from here on; sh.token and friends are set
    if (rstar < my_reg0 || rstar >= my_reg0 + kWaves) {  // another block finishes the draw
        near_edge = 0;
        return -1;
    }
    mine = true;
    if constexpr (SHARED) {  // from here on in the units of this block's own weights
        t /= scale;
        base /= scale;
        Z /= scale;
    }
    const void *rowp = part.rowp, *rowq = part.rowq;
    const int nslots = part.nslots, Vrow = part.Vrow, tok_off = part.tok_off;
    float *tab = part.tab;
    const bool use_tab = FAST && tab != nullptr;  // block-uniform
    const int span = ((nslots + kWaves - 1) / kWaves + 63) / 64 * 64;
    const int whole = PARTIAL ? whole_slots<BF16>(nslots, Vrow) : nslots;
    // one slot, the partial one included (a single thread's read)
    auto any_slot = [&](const void *row, int sidx) {
        if constexpr (FULL && !PARTIAL) return load_slot<BF16, FULL, false, true>(row, sidx, Vrow);
        else if constexpr (FULL) {
            const u32x4 v = load_slot_or_last<BF16>(row, sidx, Vrow);
            return sidx < whole ? v : partial_slot<BF16>(v, whole, Vrow);
        } else return load_slot<BF16>(row, sidx, Vrow);
    };
    const int wstar = rstar % kWaves;

    // phase B: the block walks region wstar; thread i owns slots [rb + i*per, rb + (i+1)*per)
    const int rb = min(wstar * span, nslots), re = min(rb + span, nslots);
    const int per = (re - rb + kThreads - 1) / kThreads;  // <= 5 for a 151,936-wide bf16 row
    const int my0 = rb + threadIdx.x * per, my1 = min(my0 + per, re);
    if constexpr (FAST) {
        if (use_tab) {
            // thread totals from the table; my_last_slot: the last slot of the run with mass
            double my_total = 0.0;
            int my_last_slot = -1;
            for (int sidx = my0; sidx < my1; ++sidx) {
                const float ts = tab[sidx];
                my_total += (double)ts;
                if (ts > 0.f) my_last_slot = sidx;
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
            note_first_and_last(!forced && run_incl > t && my_total > 0.0, my_last_slot, &sh.first_thread, &sh.last_positive);
            __syncthreads();
            // one slot's elements, formed again from memory: the last of them with mass, and (if
            // walk) the first whose running sum passes t
            auto open_slot = [&](int sidx, bool walk, double &c, int &tok, double &before, double &after) -> int {
                const u32x4 vp = any_slot(rowp, sidx);
                u32x4 vq = vp;
                if constexpr (RESID) vq = any_slot(rowq, sidx);
                float wf[EPV];
                (void)slot_weights_f32<BF16, RESID>(vp, vq, fn, p, wf);
                int last = -1;
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    if (wf[e] > 0.f) last = tok_off + sidx * EPV + e;
                    if (walk && tok < 0) {
                        const double cn = c + (double)wf[e];
                        if (cn > t) {
                            tok = tok_off + sidx * EPV + e;
                            before = c;
                            after = cn;
                        }
                        c = cn;
                    }
                }
                return last;
            };
            const bool walker = (int)threadIdx.x == sh.first_thread;  // at most one thread
            const bool nobody = sh.first_thread == kThreads;          // forced, or lost to rounding
            if (walker || (nobody && threadIdx.x == 0)) {
                double c = run_excl, before = c, after = c;
                int tok = -1, edge = 0;
                if (walker) {
                    for (int sidx = my0; sidx < my1 && tok < 0; ++sidx) {
                        const double cn = c + (double)tab[sidx];
                        if (cn > t) (void)open_slot(sidx, true, c, tok, before, after);  // (a crossing lost to
                        else c = cn;                                                    // rounding carries on)
                    }
                }
                if (tok < 0) {  // take the last token with mass (of the run, or of the region)
                    const int sidx = walker ? my_last_slot : sh.last_positive;
                    if (sidx >= 0) tok = open_slot(sidx, false, c, tok, before, after);
                    edge = 1;
                } else {
                    const double lo = fabs(t - before), hi = fabs(after - t);
                    if (fmin(lo, hi) <= kBoundaryEps * Z) edge = 1;
                }
                sh.token = tok;
                sh.near_edge = edge;
            }
            __syncthreads();
            const int tok = sh.token;
            near_edge = sh.near_edge;
            __syncthreads();
            return tok;
        }
    }
    // a thread's run is read kChunk slots at a time, all loads of a chunk in flight together
    // (a 151,936-wide bf16 row needs one chunk)
    double my_total = 0.0;
    int my_last = -1;
    // (the loads carry no select, which would make them wait for one another; mask_chunk puts
    // -inf into the slots past the run once all of them are on their way)
    auto load_chunk = [&](int c0, u32x4 (&vp)[kChunk], u32x4 (&vq)[kChunk]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
            const int slot = c0 + j < my1 ? c0 + j : rb;
            if constexpr (PARTIAL) {
                vp[j] = load_slot_or_last<BF16>(rowp, slot, Vrow);
                if constexpr (RESID) vq[j] = load_slot_or_last<BF16>(rowq, slot, Vrow);
            } else {
                vp[j] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(rowp, slot, Vrow);
                if constexpr (RESID) vq[j] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(rowq, slot, Vrow);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
            const bool in = c0 + j < my1;
            if (PARTIAL && c0 + j == whole) {  // (whole == nslots: there is no such slot, and no such j inside the run)
                vp[j] = partial_slot<BF16>(vp[j], whole, Vrow);
                if constexpr (RESID) vq[j] = partial_slot<BF16>(vq[j], whole, Vrow);
            }
            vp[j] = in ? vp[j] : neg_inf_slot<BF16>();
            if constexpr (RESID) vq[j] = in ? vq[j] : neg_inf_slot<BF16>();
            else vq[j] = vp[j];
        }
    };
    // the totals of the slots of the first chunk are kept for the walk, and (when the registers
    // allow: not in the form that several work-groups share) so are the slots themselves
    constexpr bool kKeepSlots = !SHARED;
    double slot_total[kChunk];
    u32x4 keep_p[kKeepSlots ? kChunk : 1], keep_q[kKeepSlots ? kChunk : 1];
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
                st = (double)slot_weights_f32<BF16, RESID>(vp[j], vq[j], fn, p, w);
#pragma unroll
                for (int e = 0; e < EPV; ++e)
                    if (w[e] > 0.f) my_last = tok_off + (c0 + j) * EPV + e;
            } else {
                double w[EPV];
                slot_weights<BF16, RESID>(vp[j], vq[j], Mp, Mq, g, p, w);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    st += w[e];
                    if (w[e] > 0.0) my_last = tok_off + (c0 + j) * EPV + e;
                }
            }
            my_total += st;
            if (c0 == my0) {
                slot_total[j] = st;
                if constexpr (kKeepSlots) {
                    keep_p[j] = vp[j];
                    keep_q[j] = vq[j];
                }
            }
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
        auto walk_slot = [&](int slot, const u32x4 &vp, const u32x4 &vq) {
            double w[EPV];
            if constexpr (FAST) {
                float wf[EPV];
                (void)slot_weights_f32<BF16, RESID>(vp, vq, fn, p, wf);
#pragma unroll
                for (int e = 0; e < EPV; ++e) w[e] = (double)wf[e];
            } else {
                slot_weights<BF16, RESID>(vp, vq, Mp, Mq, g, p, w);
            }
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                if (tok < 0) {
                    const double cn = c + w[e];
                    if (cn > t) {
                        tok = tok_off + slot * EPV + e;
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
                    if constexpr (kKeepSlots) {
                        walk_slot(my0 + j, keep_p[j], keep_q[j]);
                    } else {
                        const u32x4 vp = any_slot(rowp, my0 + j);
                        u32x4 vq = vp;
                        if constexpr (RESID) vq = any_slot(rowq, my0 + j);
                        walk_slot(my0 + j, vp, vq);
                    }
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
    return tok;
}

// What the weights of one part are formed against (a drawing block's own part).  scale: what brings them to the scale that
// the parts of a sequence share (NaN: no usable reference; every block then finds Z_out NaN).
struct PartRef {
    float M;
    double scale;
};

// The draw of a block that sees one part of the row: its own share of a sequence that several
// work-groups walk together (SHARED: the region totals are exchanged, and the block that holds
// the crossing finishes), or the whole row.  `ref_of(view)`: the reference of a part, for draws whose parts
// have references of their own (OwnRefs; the normaliser is then taken as 1); others go by `nm`.
template <bool BF16, bool RESID, bool FULL, bool SHARED, bool FAST, bool PARTIAL, int TH, bool MEETS, bool OwnRefs, class RefOf>
__device__ inline int inverse_cdf_pass(const char *rowp, const char *rowq, const PartView &own, const DrawNorm &nm, double u,
                                       SharedState &sh, Mailbox &mb, const SamplerParams &p, int &near_edge, double &Z_out,
                                       bool &mine, float *tab, RefOf &&ref_of) {
    constexpr int EPV = Elem<BF16>::EPV, kWaves = TH / 64;
    const int lane = threadIdx.x & 63;
    auto row_part = [&](const PartView &v) __attribute__((always_inline)) {
        return RowPart{rowp + (size_t)v.lo * 16, rowq + (size_t)v.lo * 16, v.nslots, v.Vrow, v.lo * EPV, tab};
    };
    auto norm_at = [&](float M) __attribute__((always_inline)) { return OwnRefs ? DrawNorm{M, M, 1.0, 1.0} : nm; };
    if constexpr (!SHARED) {
        const RowPart part = row_part(own);
        draw_region_totals<BF16, RESID, FULL, FAST, PARTIAL, TH>(part, nm, sh, p);
        __syncthreads();
        const double tot = lane < kWaves ? sh.wave_total[lane] : 0.0;
        return draw_finish<BF16, RESID, FULL, FAST, false, PARTIAL, TH>(tot, 0, part, nm, u, sh, p, near_edge, Z_out, mine, 1.0);
    } else {
        PartRef ref{0.f, 1.0};
        for_parts<BF16, MEETS>(mb, own, p.V, sh, [&](int j, const PartView &v, double(&pub)[8]) __attribute__((always_inline)) {
            if constexpr (OwnRefs) {
                ref = ref_of(v);
                if constexpr (MEETS)
                    if (threadIdx.x == 0) {
                        sh.part_ref[j] = ref.M;
                        sh.part_scale[j] = ref.scale;
                    }
            }
            draw_region_totals<BF16, RESID, FULL, FAST, PARTIAL, TH>(row_part(v), norm_at(ref.M), sh, p);
            __syncthreads();
#pragma unroll
            for (int w = 0; w < 8; ++w) pub[w] = w < kWaves ? sh.wave_total[w] * ref.scale : 0.0;
        });
        // the region totals of all parts, in vocabulary order
        const double tot = lane < mb.split * kWaves ? sh.xchg[lane / kWaves][lane % kWaves] : 0.0;
        if constexpr (!MEETS) {
            return draw_finish<BF16, RESID, FULL, FAST, true, PARTIAL, TH>(tot, mb.part * kWaves, row_part(own), norm_at(ref.M), u, sh, p,
                                                                           near_edge, Z_out, mine, ref.scale);
        } else {
            PartView v = own;
            for (int j = mb.part;;) {  // (conditions are block-uniform; a part without the crossing only looks for it)
                if constexpr (OwnRefs) ref = PartRef{sh.part_ref[j], sh.part_scale[j]};
                const int tok = draw_finish<BF16, RESID, FULL, FAST, true, PARTIAL, TH>(tot, j * kWaves, row_part(v), norm_at(ref.M), u, sh,
                                                                                        p, near_edge, Z_out, mine, ref.scale);
                if (__builtin_expect(!mb.alone, 1) || mine || !(Z_out > 0.0) || ++j == mb.split) return tok;
                v = part_view<BF16>(p.V, j, mb.split);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// one temperature per sequence; temperature 0 = greedy verification
// ------------------------------------------------------------------------------------------
// The exponent constants of one sequence, formed on the device as set_row_math forms them on
// the host (IEEE double division and conversions are the same on both).
__device__ inline void device_row_math(RowMath &m, float temperature) {
    const double T = (double)temperature;
    m.c_d = 1.4426950408889634074 / T;
    float c_hi = (float)m.c_d;
    if ((double)c_hi >= m.c_d) c_hi = __uint_as_float(__float_as_uint(c_hi) - 1u);  // next binary32 towards 0
    m.c_hi = c_hi;
    m.c_lo = (float)(m.c_d - (double)c_hi);
    m.c_f = (float)m.c_d;
    m.one_term = 0;
    m.inv_T = 1.0 / T;
    m.gap = (float)(40.0 / m.c_d);
}

// The first argmax of a row: its largest logit, the lowest token id among equal ones (an
// all -inf row gives token 0).  Every thread returns the same value.  Ends with a barrier.
// `value`: that largest logit.
template <bool BF16, bool FULL, bool PARTIAL, int TH>
__device__ inline int row_argmax(const void *row, int nslots_all, int V, SharedState &sh, float &value) {
    constexpr int EPV = Elem<BF16>::EPV, kThreads = TH, kWaves = TH / 64;
    const int nslots = PARTIAL ? whole_slots<BF16>(nslots_all, V) : nslots_all;
    constexpr int kBatch = kThreads * kUnroll;
    const int lane = opaque_thread_index() & 63, wave = threadIdx.x >> 6;
    const int n_iter = (nslots + kBatch - 1) / kBatch;
    // loads are clamped to the row and carry no select (a select right behind a load makes the
    // loads of a batch wait for one another); slots past the row are skipped when compared
    auto load_batch = [&](int it, u32x4 (&v)[kUnroll]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int slot = it * kBatch + u * kThreads + (int)threadIdx.x;
            v[u] = load_slot<BF16, FULL, false, FULL && !PARTIAL>(row, it + 1 < n_iter ? slot : max(0, min(slot, nslots - 1)), V);
        }
    };
    float best = -INFINITY;
    int best_i = 0x7fffffff;
    auto compare_batch = [&](int it, const u32x4 (&x)[kUnroll]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            float z[EPV];
            unpack<BF16>(x[u], z);
            const int slot = it * kBatch + u * kThreads + (int)threadIdx.x;
            const int e0 = slot * EPV;
#pragma unroll
            for (int j = 0; j < EPV; ++j)  // ascending ids within a thread: strict > keeps the first
                if (slot < nslots && z[j] > best) {
                    best = z[j];
                    best_i = e0 + j;
                }
        }
    };
    // two register sets take turns; the loads of the steady state are unconditional (behind a
    // condition the wait for the batch in front of a load becomes a wait for everything in flight)
    u32x4 v[kUnroll], nv[kUnroll];
    load_batch(0, v);
    int it = 0;  // v holds batch `it`; conditions are block-uniform
    for (; it + 2 < n_iter; it += 2) {
        load_batch(it + 1, nv);  // in flight while batch `it` is compared
        compare_batch(it, v);
        load_batch(it + 2, v);
        compare_batch(it + 1, nv);
    }
    if (it + 1 < n_iter) {
        load_batch(it + 1, nv);
        compare_batch(it, v);
        compare_batch(it + 1, nv);
    } else {
        compare_batch(it, v);
    }
    if (PARTIAL && nslots < nslots_all && threadIdx.x == 0) {  // the row's partial slot (the highest ids)
        float z[EPV];
        unpack<BF16>(load_partial_slot<BF16>(row, nslots, V), z);
#pragma unroll
        for (int j = 0; j < EPV; ++j)
            if (z[j] > best) {
                best = z[j];
                best_i = nslots * EPV + j;
            }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const float ob = __shfl_xor(best, o);
        const int oi = __shfl_xor(best_i, o);
        if (ob > best || (ob == best && oi < best_i)) {
            best = ob;
            best_i = oi;
        }
    }
    if (lane == 0) {
        sh.arg_val[wave] = best;
        sh.arg_idx[wave] = best_i;
    }
    __syncthreads();
    best = sh.arg_val[0];
    best_i = sh.arg_idx[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
        const float ob = sh.arg_val[w];
        const int oi = sh.arg_idx[w];
        if (ob > best || (ob == best && oi < best_i)) {
            best = ob;
            best_i = oi;
        }
    }
    __syncthreads();  // everyone has read the wave results before the next row overwrites them
    value = best;
    return best_i == 0x7fffffff ? 0 : best_i;
}

// Greedy verification of one sequence (the T -> 0 limit of Eq. 1 and Eq. 2): a drafted token is
// accepted iff it is the first argmax of its target row; the first one that is not is replaced
// by that argmax; if all are accepted the bonus token is the argmax of row k.  Reads target
// rows 0..n only, no drafter logits and no uniforms.
// A shared sequence's parts look through a part of the row each and exchange what they found.
template <bool BF16, bool FULL, bool PARTIAL, bool SHARED, int TH>
__device__ inline void greedy_sequence(const SamplerParams &p, int b, int row0, int drow0, int k, const PartView &own,
                                       SharedState &sh, Mailbox &mb) {
    constexpr int EPV = Elem<BF16>::EPV;
    const size_t esz = BF16 ? 2 : 4;
    int32_t *out = p.out_tokens + (size_t)b * (p.max_k + 1);
    int n = 0, a;
    for (;;) {
        const char *rowp = static_cast<const char *>(p.target) + (size_t)(row0 + n) * p.ld_t * esz;
        float value;
        if constexpr (!SHARED) {
            a = row_argmax<BF16, FULL, PARTIAL, TH>(rowp, own.nslots, p.V, sh, value);
        } else {
            for_parts<BF16, true>(mb, own, p.V, sh, [&](int, const PartView &v, double(&mine)[8]) __attribute__((always_inline)) {
                if (v.nslots > 0) {  // block-uniform
                    a = v.lo * EPV + row_argmax<BF16, FULL, PARTIAL, TH>(rowp + (size_t)v.lo * 16, v.nslots, v.Vrow, sh, value);
                } else {  // a part without slots (a split forced on a short row): nothing to read
                    __syncthreads();  // (as in row_stats_any)
                    value = -INFINITY;
                    a = 0;
                }
                mine[0] = (double)value, mine[1] = (double)a;
                mine[2] = mine[3] = mine[4] = mine[5] = mine[6] = mine[7] = 0.0;
            });
            double best = sh.xchg[0][0];
            a = (int)sh.xchg[0][1];
            for (int j = 1; j < mb.split; ++j)  // in vocabulary order: strict > keeps the first
                if (sh.xchg[j][0] > best) {
                    best = sh.xchg[j][0];
                    a = (int)sh.xchg[j][1];
                }
        }
        if (n >= k) break;
        const int x = p.draft_tokens[drow0 + n];
        if (x != a) break;
        if (threadIdx.x == 0 && mb.part == 0) out[n] = x;
        ++n;
    }
    if (threadIdx.x == 0 && mb.part == 0) {
        out[n] = a;
        for (int j = n + 1; j <= p.max_k; ++j) out[j] = -1;
        p.out_num_accepted[b] = SHARED && sh.failed != 0 ? -1 : n;
        if (p.out_flags) p.out_flags[b] = 0;
    }
}

// SHORT: the form for rows of at most kShortSlots slots (one work-group per sequence).
// CLAIM: the parts of a shared sequence meet in the library's own mailboxes (one temperature per sequence).
template <bool BF16, bool ONE_TERM, bool FULL, int SHARE, bool SHORT, bool PARTIAL, bool CLAIM = false>
__device__ __forceinline__ void rejection_sample(SamplerParams &p) {
    static_assert(!CLAIM || (SHARE != kOwn && !ONE_TERM), "shared, and two-term constants");
    constexpr bool SHARED = SHARE != kOwn;
    constexpr int kThreads = share_threads(SHARE), kWaves = kThreads / 64, TH = kThreads;
    __shared__ SharedState sh;
    __shared__ uint32_t sh_epoch;
    // the fp32 form of the final draw's weights: calls whose exponent constant rounds well (the
    // parts of a shared sequence form identical constants from the identical normalisers they
    // hold after the exchange); the table holds the totals of the slots of this block's part
    constexpr bool kFastScan = ONE_TERM;
    extern __shared__ __align__(16) char sampler_smem[];
    float *tab = kFastScan && p.tab_slots > 0 ? reinterpret_cast<float *>(sampler_smem) : nullptr;
    const int split = SHARED ? p.split : 1;
    const int b = blockIdx.x / split, part = blockIdx.x % split;
    uint32_t claim_epoch = 0;
    bool alone = false;  // block-uniform
    if constexpr (CLAIM) {
        alone = !claim_meet(claim_box(p.claim, b), p.claim, part, split, p.claim_ticks, &sh_epoch, sh, claim_epoch);
        if (alone && part != 0) return;
    }
    // bounds come from device data: clamp them by the host-side totals so that no value of
    // q_indptr can push a row outside the logits buffers
    const int row0 = max(0, min(p.q_indptr[b], p.total_q - 1));
    int k = p.q_indptr[b + 1] - row0 - 1;
    k = max(0, min(k, min(p.max_k, p.total_q - 1 - row0)));
    const int drow0 = row0 - b;
    if (drow0 < 0 || drow0 + k > p.total_q - p.B) k = 0;
    const PartView own = part_view<BF16>(p.V, part, split);  // this block's part of the vocabulary
    const size_t esz = BF16 ? 2 : 4;
    const char *tbase = static_cast<const char *>(p.target);
    const char *dbase = static_cast<const char *>(p.draft);
    int32_t *out = p.out_tokens + (size_t)b * (p.max_k + 1);
    Mailbox mb{nullptr, nullptr, 0u, part, split, 0, 0u, &sh_epoch, false};
    if (threadIdx.x == 0) sh.failed = 0;
    if constexpr (CLAIM) {
        mb = claim_mailbox(claim_box(p.claim, b), part, split, claim_epoch, &sh_epoch, alone);
    } else if constexpr (SHARED) {
        mb.words = reinterpret_cast<uint32_t *>(p.boxes + (size_t)b * kBoxBytes);
        mb.payload = reinterpret_cast<unsigned long long *>(p.boxes + (size_t)b * kBoxBytes + kBoxHeaderBytes);
        if (threadIdx.x == 0) mb.epoch = load_dev(mb.words);
    }
    auto leave = [&]() __attribute__((always_inline)) {  // one thread of the block, behind its last exchange
        if constexpr (CLAIM) {
            // (a box whose wait ran out stays taken: sequences that come to it are walked alone from then on)
            if (!mb.alone && sh.failed == 0) claim_leave(claim_box(p.claim, b), mb.split, mb.epoch);
        }
    };
    if constexpr ((!SHARED || CLAIM) && !ONE_TERM) {
        if (p.temps != nullptr) {  // block-uniform
            const float T = p.temps[b];
            const bool bad = !(T >= 0.f) || T == INFINITY ||
                             (T > 0.f && k > 0 && (p.draft == nullptr || p.u_accept == nullptr));
            if (bad) {  // a caller error: make it impossible to miss
                if (threadIdx.x == 0 && part == 0) {
                    for (int j = 0; j <= p.max_k; ++j) out[j] = -1;
                    p.out_num_accepted[b] = -1;
                    if (p.out_flags) p.out_flags[b] = 0;
                }
                if (threadIdx.x == 0) leave();
                return;
            }
            if (T == 0.f) {
                greedy_sequence<BF16, FULL, PARTIAL, SHARED, TH>(p, b, row0, drow0, k, own, sh, mb);
                if (threadIdx.x == 0) leave();
                return;
            }
            device_row_math(p, T);
        }
    }
    const double u_fin = (double)p.u_final[b];
    int n = 0, flag_accept = 0, flag_cdf = 0, final_token = -1;
    bool rejected = false, mine = false;
    // shared sequences walk their chain two items per stage (see row_stats_two_items); `ahead`
    // holds the normalisers of item `ahead_of` (a position, or k for the bonus token's row)
    constexpr bool kTwoItems = SHARE == kTwoAtATime;
    static_assert(!kTwoItems || FULL, "the guarded form takes one item at a time");
    DrawNorm ahead{};
    int ahead_of = -1;
    float last_Mp = 0.f;  // reference of the target row of the position tested last
    const char *scan_row = tbase;  // row, reference and sum of the final inverse-CDF walk over p
    float scan_M = 0.f;
    double scan_S = 1.0;
    // Eq. 1 in fp64: rho = p(x)/q(x) = exp(((zp-Mp) - (zq-Mq))/T) * Sq/Sp
    auto ratio = [&](float zpx, float zqx, float Mp, double Sp, float Mq, double Sq) __attribute__((always_inline)) {
        if (zqx == -INFINITY) return (zpx == -INFINITY) ? 0.0 : (double)INFINITY;
        return exp((((double)zpx - (double)Mp) - ((double)zqx - (double)Mq)) * p.inv_T) * (Sq / Sp);
    };
    // A drafted token, its two logits and the uniform of its test: requested while the position's first batch is on its
    // way, so that neither the pass nor the test waits for a chain of dependent loads.
    struct Draft {
        int x;
        float zpx, zqx;
        double u;
    };
    auto draft_at = [&](int i) __attribute__((always_inline)) {
        Draft d;
        d.x = max(0, min(p.draft_tokens[drow0 + i], p.V - 1));  // memory safety only; ids outside [0,V) are a caller error
        d.zpx = logit_at<BF16>(tbase + (size_t)(row0 + i) * p.ld_t * esz, d.x);
        d.zqx = logit_at<BF16>(dbase + (size_t)(drow0 + i) * p.ld_d * esz, d.x);
        d.u = (double)p.u_accept[drow0 + i];
        return d;
    };
    Draft d{}, d_ahead{};
    // Short rows: a position's chain of loads, reductions and barriers takes 3 us whatever the row's
    // length, so eight positions are taken at a time, one per wave, rows behind a rejected position
    // read for nothing (never used).  (An instantiation of its own: tested at run time it cost the
    // long rows 1-2 %.)  Where the line lies stands at the launch.
    static_assert(!SHORT || !SHARED, "short rows are not shared");
    for (int i = 0; i < k; ++i) {
        const char *rowp = tbase + (size_t)(row0 + i) * p.ld_t * esz;
        const char *rowq = dbase + (size_t)(drow0 + i) * p.ld_d * esz;
        if constexpr (SHORT) {
            const int wave = threadIdx.x >> 6;
            if ((i & (kWaves - 1)) == 0) {
                __syncthreads();  // (the numbers of the eight positions before have been read)
                if (i + wave < k) {
                    const char *rp = rowp + (size_t)wave * p.ld_t * esz, *rq = rowq + (size_t)wave * p.ld_d * esz;
                    const int x = max(0, min(p.draft_tokens[drow0 + i + wave], p.V - 1));
                    const float zpx = logit_at<BF16>(rp, x), zqx = logit_at<BF16>(rq, x);
                    const double u = (double)p.u_accept[drow0 + i + wave];
                    float M[2];
                    double S[2];
                    wave_row_pair_stats<BF16>(rp, rq, own.nslots, own.Vrow, p, M, S);
                    const double rho = ratio(zpx, zqx, M[0], S[0], M[1], S[1]);
                    if ((threadIdx.x & 63) == 0) {
                        sh.pos_m[0][wave] = M[0];
                        sh.pos_m[1][wave] = M[1];
                        sh.pos_s[0][wave] = S[0];
                        sh.pos_s[1][wave] = S[1];
                        sh.pos_rho[wave] = rho;
                        sh.pos_u[wave] = u;
                        sh.pos_x[wave] = x;
                    }
                }
                __syncthreads();
            }
        }
        float Mp = 0.f, Mq = 0.f;
        double Sp = 0.0, Sq = 0.0;
        if constexpr (SHORT) {
            const int w = i & (kWaves - 1);
            d.x = sh.pos_x[w];
            d.u = sh.pos_u[w];
            Mp = sh.pos_m[0][w], Sp = sh.pos_s[0][w], Mq = sh.pos_m[1][w], Sq = sh.pos_s[1][w];
        }
        if constexpr (kTwoItems) {
            if (ahead_of == i) {  // this position's numbers came with the previous stage (block-uniform)
                Mp = ahead.Mp, Sp = ahead.Sp, Mq = ahead.Mq, Sq = ahead.Sq;
                d = d_ahead;
            } else {
                // one stage for this position and the next item of the chain: position i + 1, or
                // the bonus token's row when this is the last draft
                const bool b_pair = i + 1 < k;
                const char *rowpb = tbase + (size_t)(row0 + i + 1) * p.ld_t * esz;
                const char *rowqb = b_pair ? dbase + (size_t)(drow0 + i + 1) * p.ld_d * esz : rowpb;
                DrawNorm a;
                row_stats_two_items<BF16, ONE_TERM, PARTIAL, TH, CLAIM>(
                    rowp, rowq, rowpb, rowqb, b_pair, own, sh, mb, p, a, ahead, [&]() __attribute__((always_inline)) {
                        d = draft_at(i);
                        if (b_pair) d_ahead = draft_at(i + 1);
                    });
                ahead_of = i + 1;
                Mp = a.Mp, Sp = a.Sp, Mq = a.Mq, Sq = a.Sq;
            }
        } else if constexpr (!SHORT) {
            row_stats_any<BF16, true, ONE_TERM, FULL, SHARED, PARTIAL, TH, CLAIM>(rowp, rowq, own, p.V, sh, i & 1, mb, p, Mp, Sp, Mq, Sq, [&]() __attribute__((always_inline)) { d = draft_at(i); });
        }
        last_Mp = Mp;
        double rho;
        if constexpr (SHORT) rho = sh.pos_rho[i & (kWaves - 1)];
        else rho = ratio(d.zpx, d.zqx, Mp, Sp, Mq, Sq);
        const double thr = rho < 1.0 ? rho : 1.0;
        if (fabs(d.u - thr) <= kBoundaryEps) flag_accept = 1;
        if (d.u < thr) {
            if (threadIdx.x == 0 && part == 0) out[i] = d.x;
            n = i + 1;
            continue;
        }
        // first rejection: one draw from the residual distribution (Eq. 2)
        double Z;
        int edge = 0;
        final_token = inverse_cdf_pass<BF16, true, FULL, SHARED, kFastScan, PARTIAL, TH, CLAIM, false>(
            rowp, rowq, own, DrawNorm{Mp, Mq, Sp, Sq}, u_fin, sh, mb, p, edge, Z, mine, tab, Nothing{});
        flag_cdf = edge;
        rejected = true;
        scan_row = rowp;
        scan_M = Mp;
        scan_S = Sp;
        // an empty residual (an exact tie, Z = 0 in every part) falls back to the target itself
        if (!(Z > 0.0)) final_token = -2;
        break;
    }
    bool scan_target = false;
    bool drawn = false;
    if constexpr (FULL) {
        // The bonus token's draw needs no normaliser: it compares running sums of weights with u
        // times their total, so exp((z - M0)/T) serves for any reference M0 that keeps the weights in
        // range: one pass over the row instead of two.  M0 is the largest logit among the first slots
        // of the row, or of this block's part of it, so no total is small beside its largest
        // weight.  (A reference of another row may lie far above this one: the small weights are then
        // lost below 2^-126 while the total is still positive.)  The blocks of a shared sequence bring
        // their fp64 totals to one scale, weights against last_Mp, which all of them hold (a sequence
        // without drafts, or whose bonus row came with the last stage, goes the ordinary way); a part that starts
        // without any finite logit looks for one further on, and one that has none has no mass.  A total
        // that is not a positive number in the middle of the fp64 range (an outlier far above M0)
        // leaves the draw to the two passes below; every block sees the same total and decides alike.
        if (!rejected && (!SHARED || (k > 0 && ahead_of != k))) {
            scan_row = tbase + (size_t)(row0 + k) * p.ld_t * esz;
            auto start_max = [&](const PartView &v) __attribute__((always_inline)) {
                const char *part_row = scan_row + (size_t)v.lo * 16;
                const int whole = PARTIAL ? whole_slots<BF16>(v.nslots, v.Vrow) : v.nslots;
                float M0 = block_max_of_row_start<BF16, !PARTIAL, kRefSlots<ONE_TERM>, TH>(part_row, whole, sh);
                if constexpr (SHARED) {  // block-uniform
                    for (int at = kRefSlots<ONE_TERM> * TH; M0 == -INFINITY && at < whole; at += kUnroll * TH)
                        M0 = block_max_of_row_start<BF16, !PARTIAL, kUnroll, TH>(part_row + (size_t)at * 16, whole - at, sh);
                }
                return M0;
            };
            auto ref_of = [&](const PartView &v) __attribute__((always_inline)) {  // (shared sequences)
                PartRef ref{start_max(v), 1.0};
                if (ref.M > -INFINITY && ref.M < INFINITY) {  // block-uniform
                    // what the weights are formed with: exp2(z c_f + K) or exp2((z - M0) c)
                    if constexpr (kFastScan) ref.scale = exp2_f64(-(double)make_fast_norm(ref.M, 1.0, ref.M, 1.0, p).Kp - (double)last_Mp * (double)p.c_f);
                    else ref.scale = exp2_f64(((double)ref.M - (double)last_Mp) * p.c_d);
                } else {  // no mass, unless the partial slot has some
                    const int whole = PARTIAL ? whole_slots<BF16>(v.nslots, v.Vrow) : v.nslots;
                    ref.scale = ref.M == -INFINITY && whole == v.nslots ? 1.0 : (double)NAN;
                    ref.M = 0.f;
                }
                return ref;
            };
            float M0 = 0.f;
            if constexpr (!SHARED) M0 = start_max(own);
            if (SHARED || (M0 > -INFINITY && M0 < INFINITY)) {  // block-uniform
                double Z;
                int edge = 0;
                const int tok = inverse_cdf_pass<BF16, false, FULL, SHARED, kFastScan, PARTIAL, TH, CLAIM, SHARED>(
                    scan_row, scan_row, own, DrawNorm{M0, M0, 1.0, 1.0}, u_fin, sh, mb, p, edge, Z, mine, tab, ref_of);
                if (Z > 1.0e-280 && Z < 1.0e280) {
                    final_token = tok;
                    flag_cdf = edge;
                    drawn = true;
                } else {
                    mine = false;
                }
            }
        }
    }
    if (drawn) {
        // (nothing left to do)
    } else if (!rejected) {  // every draft accepted (or none offered): bonus token from target row k
        scan_row = tbase + (size_t)(row0 + k) * p.ld_t * esz;
        float Mq;
        double Sq;
        if (kTwoItems && ahead_of == k) {
            scan_M = ahead.Mp;
            scan_S = ahead.Sp;
        } else {
            row_stats_any<BF16, false, ONE_TERM, FULL, SHARED, PARTIAL, TH, CLAIM>(scan_row, scan_row, own, p.V, sh, k & 1, mb, p, scan_M,
                                                                                   scan_S, Mq, Sq);
        }
        scan_target = true;
    } else if (final_token == -2) {
        scan_target = true;
    }
    if (scan_target) {
        double Z;
        int edge = 0;
        final_token = inverse_cdf_pass<BF16, false, FULL, SHARED, kFastScan, PARTIAL, TH, CLAIM, false>(
            scan_row, scan_row, own, DrawNorm{scan_M, scan_M, scan_S, scan_S}, u_fin, sh, mb, p, edge, Z, mine, tab, Nothing{});
        flag_cdf = rejected ? 1 : edge;
        if (!(Z > 0.0)) {  // row without any finite logit: part 0 reports the last token
            mine = part == 0;
            final_token = p.V - 1;
        }
    }
    // the part that made the final draw writes the sequence's results
    if (threadIdx.x == 0) {
        const bool failed = sh.failed != 0;
        if (mine) {
            out[n] = final_token;
            for (int j = n + 1; j <= p.max_k; ++j) out[j] = -1;
            p.out_num_accepted[b] = failed ? -1 : n;
            if (p.out_flags) p.out_flags[b] = (flag_accept ? 1 : 0) | (flag_cdf ? 2 : 0);
        } else if (failed) {
            p.out_num_accepted[b] = -1;  // a wait for a partner ran out: make it impossible to miss
        }
        if constexpr (CLAIM) {
            leave();
        } else if constexpr (SHARED) {
            // Part 0 advances the epoch; a part whose wait ran out poisons the box instead (a
            // partner that turns up later must not find an epoch it could publish under, and the
            // next call must not trust what this one left).  Both are atomic maxima, so the
            // poison wins whatever the order.
            if (failed) {
                __hip_atomic_fetch_max(mb.words, kBoxPoison, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else if (part == 0) {
                __hip_atomic_fetch_max(mb.words, mb.epoch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <bool BF16, bool ONE_TERM, bool FULL, bool SHARED>
__global__ __launch_bounds__(kThreads) void rejection_sample_kernel(SamplerParams p) {
    rejection_sample<BF16, ONE_TERM, FULL, SHARED ? kOneAtATime : kOwn, false, false>(p);
}

template <bool BF16, bool ONE_TERM>
__global__ __launch_bounds__(share_threads(kTwoAtATime)) void two_items_sample_kernel(SamplerParams p) {
    rejection_sample<BF16, ONE_TERM, true, kTwoAtATime, false, false>(p);
}

// Rows that are not whole aligned slots (fp64 weights).
template <bool BF16, bool SHARED>
__global__ __launch_bounds__(kThreads) void partial_rows_sample_kernel(SamplerParams p) {
    rejection_sample<BF16, false, true, SHARED ? kOneAtATime : kOwn, false, true>(p);
}

template <bool BF16>
__global__ __launch_bounds__(share_threads(kTwoAtATime)) void partial_rows_two_items_kernel(SamplerParams p) {
    rejection_sample<BF16, false, true, kTwoAtATime, false, true>(p);
}

// One temperature per sequence, shared between work-groups that meet in the library's mailboxes.
template <bool BF16, bool PARTIAL>
__global__ __launch_bounds__(kThreads) void claimed_sample_kernel(SamplerParams p) {
    rejection_sample<BF16, false, true, kOneAtATime, false, PARTIAL, true>(p);
}

template <bool BF16, bool PARTIAL>
__global__ __launch_bounds__(share_threads(kTwoAtATime)) void claimed_two_items_kernel(SamplerParams p) {
    rejection_sample<BF16, false, true, kTwoAtATime, false, PARTIAL, true>(p);
}

template <bool BF16, bool ONE_TERM>
__global__ __launch_bounds__(kThreads) void short_rows_sample_kernel(SamplerParams p) {
    rejection_sample<BF16, ONE_TERM, true, kOwn, true, !ONE_TERM>(p);
}

// Both entry points: `temps` NULL = one temperature for the batch (`temperature`), else one per
// sequence on the device (no workspace then: sequences are shared through the library's own mailboxes).
respec_status_t sample_common(const void *target_logits, const void *draft_logits, const int32_t *draft_tokens,
                              const int32_t *q_indptr, const float *u_accept, const float *u_final,
                              int32_t *out_tokens, int32_t *out_num_accepted, int32_t *out_flags, int32_t B,
                              int32_t total_q, int32_t max_k, int32_t V, int64_t ld_t, int64_t ld_d,
                              float temperature, const float *temps, respec_dtype_t logits_dt, void *workspace,
                              size_t workspace_bytes, void *hip_stream) {
    if (B <= 0 || total_q < B || max_k < 0 || V <= 0)
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: need B > 0, total_q >= B, max_k >= 0, V > 0 "
                    "(B=%d total_q=%d max_k=%d V=%d)", B, total_q, max_k, V);
    if (!temps && (!(temperature > 0.f) || !std::isfinite(temperature)))
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: temperature must be finite and > 0");
    if (logits_dt != RESPEC_F32 && logits_dt != RESPEC_BF16)
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: unknown logits dtype %d", (int)logits_dt);
    if (!target_logits || !q_indptr || !u_final || !out_tokens || !out_num_accepted)
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: null pointer argument");
    const bool has_drafts = total_q > B;
    // with one temperature per sequence a batch may be all greedy: then only the drafted tokens are read
    if (has_drafts && (!draft_tokens || (!temps && (!draft_logits || !u_accept))))
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: drafted tokens present but a draft pointer is null");
    if (has_drafts && !draft_logits) ld_d = ld_t;
    if (ld_t < V || (has_drafts && ld_d < V))
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: row stride smaller than V");
    if ((int64_t)max_k * B < (int64_t)total_q - B)
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: max_k too small for total_q");
    const size_t esz = logits_dt == RESPEC_BF16 ? 2 : 4;
    if (!aligned_to(target_logits, esz) || (has_drafts && draft_logits && !aligned_to(draft_logits, esz)))
        return fail(RESPEC_ERR_INVALID_ARG, "rejection_sample: logits pointer not element aligned");

    SamplerParams p{};
    p.target = target_logits;
    p.draft = has_drafts ? draft_logits : target_logits;
    p.temps = temps;
    p.draft_tokens = draft_tokens;
    p.q_indptr = q_indptr;
    p.u_accept = u_accept;
    p.u_final = u_final;
    p.out_tokens = out_tokens;
    p.out_num_accepted = out_num_accepted;
    p.out_flags = out_flags;
    p.B = B;
    p.total_q = total_q;
    p.max_k = max_k;
    p.V = V;
    p.ld_t = ld_t;
    p.ld_d = has_drafts ? ld_d : ld_t;
    const Knobs kn = knobs();
    set_row_math(p, temps ? 1.0f : temperature, kn.get(&Knobs::sampler_two_term, 0) != 0);
    if (temps) p.one_term = 0;  // the per-sequence constants are formed on the device, two-term

    // work-groups per sequence: as many as there are otherwise idle compute units, as long as a
    // part keeps a useful share of the row; one (and no mailbox) with one temperature and no workspace
    int split = 1, cus = 256;
    bool two_items = false;
    // (per-sequence temperatures have no workspace argument: their parts meet in the library's own mailboxes)
    const bool claim = temps && V >= (logits_dt == RESPEC_BF16 ? 8 : 4) && kn.get(&Knobs::sampler_guarded, 0) == 0 &&
                       kn.get(&Knobs::sampler_claim, 1) != 0;
    if (workspace || claim) {
        if (workspace && (workspace_bytes < (size_t)B * kBoxBytes || !aligned_to(workspace, 16)))
            return fail(RESPEC_ERR_WORKSPACE, "rejection_sample: workspace of %zu bytes (16-byte aligned) needed, got %zu",
                        (size_t)B * kBoxBytes, workspace_bytes);
        int dev = 0;
        if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        // Two chain items per stage read a row pair that the chain may not need.  That pays while
        // the extra bytes are cheaper than the exchange they save: up to a quarter as many sequences
        // as compute units (one item / two, us per call: bf16, V = 151,936, B = 96 63.0 / 60.6, B = 128 56.6 / 64.4;
        // fp32, V = 50,257, B = 100 40.3 / 43.7).
        two_items = kn.get(&Knobs::sampler_two_items, (long)B * 4 <= cus ? 1 : 0) != 0;
        // A stage of two items costs little beside its pass, so parts may be shorter there, for rows whose passes are long enough
        // to begin with (k = 4, us per call by one work-group / two / four: bf16, B = 64, V = 18,432 23.9 / 24.8 / 22.4 but k = 3
        // 20.4 / 24.1 / 21.7, V = 26,624 25.9 / 26.0 / 23.2, k = 3 22.2 / 25.4 / 22.4, V = 32,000 27.0 / 26.9 / 23.5, k = 3 22.8 / 25.4 / 22.4; fp32,
        // whose slots hold half as many elements, V = 12,288 19.1 / 22.1 / 20.6, V = 16,384 20.2 / 23.1 / 21.0); with one item per
        // stage they may not (V = 32,000, B = 100 30.2 / 33.5 in parts of 2000), nor where a chain has one stage (V = 32,000,
        // B = 64, k = 1 15.2 / 16.4 in parts of 1000, k = 0 10.2 / 12.7).
        const int epv0 = logits_dt == RESPEC_BF16 ? 8 : 4;
        const long slots_row = ((long)V + epv0 - 1) / epv0;
        long least = two_items && max_k >= 3 && slots_row >= (logits_dt == RESPEC_BF16 ? 3328 : 4096) ? 768 : 2048;  // slots of a part
        // Parts that have to meet first want longer rows (mixed temperatures, by one work-group / shared, us per call: bf16, one item, B = 100,
        // V = 36,000 and 44,000 32.4 / 36.4, 35.0 / 37.3, V = 50,000, B = 128 40.9 / 39.8; two items, V = 30,000 and more 34.1 / 28.7; fp32, whose
        // slots hold half as many elements: two items, B = 64, k = 3, V = 32,000 in two and four 26.3 / 30.5, 26.0 / 27.2, V = 40,000 in two 28.7 / 33.3,
        // V = 50,000 in four 33.3 / 32.4; one item, B = 128, V = 50,000 35.3 / 39.5, V = 70,000 43.4 / 43.9).
        if (claim) {
            const bool bf16 = logits_dt == RESPEC_BF16, wide_chain = two_items && max_k >= 3;
            if (!bf16) least = !two_items ? 9600 : slots_row >= 4 * 3072 ? 3072 : slots_row;
            else if (!wide_chain) least = two_items ? 4096 : 3072;
            else if (slots_row < 3700) least = slots_row;
        }
        while (split < kMaxSplit && (long)B * split * 2 <= cus && slots_row / (split * 2) >= least) split *= 2;
        const long forced = kn.get(&Knobs::sampler_split, 0);
        if (forced == 1 || forced == 2 || forced == 4 || forced == 8) split = (int)forced;
        // The parts of a sequence wait for one another, so all of them have to be on the device at
        // once: never more work-groups than compute units, whatever the knob asks for.  And a
        // pass's mark has ten bits for the stage (at most one per position, and four): very long draft chains take one work-group.
        while (split > 1 && (long)B * split > cus) split /= 2;
        // the part that holds a row's partial slot also holds whole ones
        if (V % epv0 != 0)
            while (split > 1 && (long)(split - 1) * (((slots_row + split - 1) / split + 63) / 64 * 64) >= V / epv0) split /= 2;
        if (2 * ((long)max_k + 1) + 4 >= 1024) split = 1;
        if (claim) {
            split = std::min(split, kClaimSplit);
            while (split > 1 && (long)B * split > kClaimGroups) split /= 2;
        }
    }
    if (claim && split > 1) {
        p.claim = next_claim_key();
        p.claim_ticks = (int)kn.get(&Knobs::sampler_claim_ticks, kClaimTicks);
    }
    if ((int64_t)B * split > 0x7fffffffLL)
        return fail(RESPEC_ERR_UNSUPPORTED, "rejection_sample: too many work-groups");
    p.split = split;
    p.boxes = static_cast<char *>(workspace);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int epv = logits_dt == RESPEC_BF16 ? 8 : 4;
    const bool full = V >= epv && kn.get(&Knobs::sampler_guarded, 0) == 0;
    const bool whole_rows = V % epv == 0 && aligned_to(target_logits, 16) && (ld_t * esz) % 16 == 0 &&
                            (!has_drafts || !draft_logits || (aligned_to(draft_logits, 16) && (ld_d * esz) % 16 == 0));
    // rows of whole, aligned slots take fp32 weights when the exponent constant rounds well; the
    // others keep the fp64 weights they always had
    p.one_term = p.one_term && whole_rows;
    const bool bf = logits_dt == RESPEC_BF16, one = p.one_term != 0;
    // the final draw's table of slot totals (fp32 form, one work-group per sequence): one float
    // per 16-byte slot of a row in dynamic LDS, when that fits beside the static part
    size_t smem = 0;
    {
        const size_t slots_row = ((size_t)V + epv - 1) / epv;
        // (a part of a shared sequence: the kernel's own rounding of the split)
        const size_t slots_part = split > 1 ? ((slots_row + split - 1) / split + 63) / 64 * 64 : slots_row;
        if (full && one && slots_part * sizeof(float) <= kTableMaxBytes &&
            kn.get(&Knobs::sampler_no_table, 0) == 0) {
            smem = round_up(slots_part * sizeof(float), 16);
            p.tab_slots = (int)slots_part;
        }
    }
// several work-groups per sequence
#define RESPEC_LAUNCH_SAMPLER_SHARED(KERNEL, SHARE)                                                                 \
    do {                                                                                                           \
        if (smem > 48 * 1024) { /* (only whole rows need more than the default limit) */                          \
            smem = 0;                                                                                              \
            p.tab_slots = 0;                                                                                       \
        }                                                                                                          \
        hipLaunchKernelGGL(KERNEL, dim3((unsigned)(B * split)), dim3(share_threads(SHARE)), smem, stream, p);      \
    } while (0)
#define RESPEC_LAUNCH_FORM(BF, ONE)                                                                                 \
    do {                                                                                                           \
        if (split == 1) RESPEC_LAUNCH_SAMPLER_ONE((rejection_sample_kernel<BF, ONE, true, false>));                 \
        else if (two_items) RESPEC_LAUNCH_SAMPLER_SHARED((two_items_sample_kernel<BF, ONE>), kTwoAtATime); \
        else RESPEC_LAUNCH_SAMPLER_SHARED((rejection_sample_kernel<BF, ONE, true, true>), kOneAtATime);     \
    } while (0)
#define RESPEC_LAUNCH_CLAIMED(BF, PARTIAL)                                                                          \
    do {                                                                                                           \
        if (two_items) RESPEC_LAUNCH_SAMPLER_SHARED((claimed_two_items_kernel<BF, PARTIAL>), kTwoAtATime);         \
        else RESPEC_LAUNCH_SAMPLER_SHARED((claimed_sample_kernel<BF, PARTIAL>), kOneAtATime);                      \
    } while (0)
#define RESPEC_LAUNCH_GUARDED(BF)                                                                                   \
    do {                                                                                                           \
        if (split == 1) RESPEC_LAUNCH_SAMPLER_ONE((rejection_sample_kernel<BF, false, false, false>));              \
        else RESPEC_LAUNCH_SAMPLER_SHARED((rejection_sample_kernel<BF, false, false, true>), kOneAtATime);  \
    } while (0)
#define RESPEC_LAUNCH_PARTIAL(BF)                                                                                   \
    do {                                                                                                           \
        if (split == 1) RESPEC_LAUNCH_SAMPLER_ONE((partial_rows_sample_kernel<BF, false>));                         \
        else if (two_items) RESPEC_LAUNCH_SAMPLER_SHARED((partial_rows_two_items_kernel<BF>), kTwoAtATime); \
        else RESPEC_LAUNCH_SAMPLER_SHARED((partial_rows_sample_kernel<BF, true>), kOneAtATime);             \
    } while (0)
// one work-group per sequence
#define RESPEC_LAUNCH_SAMPLER_ONE(KERNEL)                                                                           \
    do {                                                                                                           \
        if (smem > 0 && hipFuncSetAttribute(reinterpret_cast<const void *>(&KERNEL),                               \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess) { \
            smem = 0;                                                                                              \
            p.tab_slots = 0;                                                                                       \
        }                                                                                                          \
        hipLaunchKernelGGL(KERNEL, dim3((unsigned)B), dim3(kThreads), smem, stream, p);                            \
    } while (0)
    // Short rows eight positions at a time (long form / this one, us per call, fp32, k = 4 unless said):
    // V = 1024, B = 4 17.4 / 10.1, B = 512 34.3 / 19.5; V = 2048, B = 4 18.1 / 11.5, B = 512 35.1 / 23.8.
    // It takes the same time however early the chains end, so it loses where every sequence of the
    // batch rejects its first draft (V = 1024, B = 4 8.9 / 9.4, V = 2048 9.6 / 10.8; not at B = 512, where
    // some sequence goes on: 24.2 / 23.2), with a single draft (V = 2048 9.5 / 10.6) and at 1024 slots
    // (V = 4096, B = 2048 128 / 135, drafts rarely accepted 87 / 133).
    const bool short_rows = full && split == 1 && max_k > 1 && ((int64_t)V + epv - 1) / epv <= kShortSlots;
    if (p.claim) {
        if (bf) { if (whole_rows) RESPEC_LAUNCH_CLAIMED(true, false); else RESPEC_LAUNCH_CLAIMED(true, true); }
        else { if (whole_rows) RESPEC_LAUNCH_CLAIMED(false, false); else RESPEC_LAUNCH_CLAIMED(false, true); }
    } else if (short_rows && bf) {
        if (one) RESPEC_LAUNCH_SAMPLER_ONE((short_rows_sample_kernel<true, true>));
        else RESPEC_LAUNCH_SAMPLER_ONE((short_rows_sample_kernel<true, false>));
    } else if (short_rows) {
        if (one) RESPEC_LAUNCH_SAMPLER_ONE((short_rows_sample_kernel<false, true>));
        else RESPEC_LAUNCH_SAMPLER_ONE((short_rows_sample_kernel<false, false>));
    } else if (!full) {
        if (bf) RESPEC_LAUNCH_GUARDED(true); else RESPEC_LAUNCH_GUARDED(false);
    } else if (!whole_rows) {
        if (bf) RESPEC_LAUNCH_PARTIAL(true); else RESPEC_LAUNCH_PARTIAL(false);
    } else if (bf) {
        if (one) RESPEC_LAUNCH_FORM(true, true); else RESPEC_LAUNCH_FORM(true, false);
    } else {
        if (one) RESPEC_LAUNCH_FORM(false, true); else RESPEC_LAUNCH_FORM(false, false);
    }
#undef RESPEC_LAUNCH_FORM
#undef RESPEC_LAUNCH_CLAIMED
#undef RESPEC_LAUNCH_GUARDED
#undef RESPEC_LAUNCH_PARTIAL
#undef RESPEC_LAUNCH_SAMPLER_SHARED
#undef RESPEC_LAUNCH_SAMPLER_ONE
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess)
        return fail(RESPEC_ERR_HIP, "rejection_sample: launch failed: %s", hipGetErrorString(err));
    clear_error();
    return RESPEC_OK;
}

}  // namespace
}  // namespace respec

extern "C" {

size_t respec_rejection_sample_workspace_bytes(int32_t B, int32_t, int32_t, respec_dtype_t) {
    return B > 0 ? (size_t)B * respec::kBoxBytes : 0;
}

respec_status_t respec_rejection_sample(const void *target_logits, const void *draft_logits,
                                        const int32_t *draft_tokens, const int32_t *q_indptr,
                                        const float *u_accept, const float *u_final,
                                        int32_t *out_tokens, int32_t *out_num_accepted,
                                        int32_t *out_flags, int32_t B, int32_t total_q,
                                        int32_t max_k, int32_t V, int64_t ld_t, int64_t ld_d,
                                        float temperature, respec_dtype_t logits_dt,
                                        void *workspace, size_t workspace_bytes,
                                        void *hip_stream) {
    return respec::sample_common(target_logits, draft_logits, draft_tokens, q_indptr, u_accept, u_final, out_tokens,
                                 out_num_accepted, out_flags, B, total_q, max_k, V, ld_t, ld_d, temperature, nullptr,
                                 logits_dt, workspace, workspace_bytes, hip_stream);
}

respec_status_t respec_rejection_sample_per_seq(const void *target_logits, const void *draft_logits,
                                                const int32_t *draft_tokens, const int32_t *q_indptr,
                                                const float *u_accept, const float *u_final,
                                                const float *temperature, int32_t *out_tokens,
                                                int32_t *out_num_accepted, int32_t *out_flags, int32_t B,
                                                int32_t total_q, int32_t max_k, int32_t V, int64_t ld_t,
                                                int64_t ld_d, respec_dtype_t logits_dt, void *hip_stream) {
    if (!temperature)
        return respec::fail(RESPEC_ERR_INVALID_ARG, "rejection_sample_per_seq: null temperature array");
    return respec::sample_common(target_logits, draft_logits, draft_tokens, q_indptr, u_accept, u_final, out_tokens,
                                 out_num_accepted, out_flags, B, total_q, max_k, V, ld_t, ld_d, 1.0f, temperature,
                                 logits_dt, nullptr, 0, hip_stream);
}

}  // extern "C"
