// Sequences that several work-groups walk together: the mailbox their parts exchange results through, the
// normalisers of a row they see a part of each, and the library's own mailboxes for calls without a
// workspace.
#pragma once

#include "respec_sampler_rows.hpp"

#include <atomic>

namespace respec {
namespace {

// ------------------------------------------------------------------------------------------
// mailbox: the few numbers the parts of one sequence exchange after a streaming pass
// ------------------------------------------------------------------------------------------
// Layout of one box (kBoxBytes): word 0 the epoch (calls that have used the box), then
// [part][stage parity][16] tagged words of payload: the eight doubles a part publishes per
// stage, each as two 64-bit words that carry 32 bits of the value below a 32-bit mark,
// mark = epoch*1024 + stage + 1.  A word is written and read with one 8-byte device-scope
// access, so a reader that finds the mark it waits for has the value that belongs to it: no
// separate flag and no fence; a reader fetches a partner's sixteen words together and is done
// after one memory round trip once the partner has published (a flag behind the payload costs
// three: the writer's wait for its stores, the reader's poll, the reader's dependent read).
// A part that has read every partner's stage s may publish stage s+1 into the other parity
// buffer, and nobody can be two stages ahead of the slowest reader, so a word is never
// overwritten while somebody still waits for it.  Part 0 bumps the epoch when it leaves (every
// partner has read it by then: they publish their first stage after reading it, and part 0 has
// read that stage), so nothing needs resetting and the box only has to be zero before its
// first use (a mark is never 0).  All accesses are device-scope atomics: the parts run on
// compute units whose L2 caches are not coherent with each other.
struct Mailbox {
    uint32_t *words;
    unsigned long long *payload;
    uint32_t base;          // valid from the first exchange on
    int part, split, stage;
    uint32_t epoch;         // thread 0: the box's epoch, requested at the start of the kernel
    uint32_t *sh_epoch;     // LDS word it is handed to the block in
    bool alone;             // the parts did not meet (MEETS forms only): this one does the work of all
};

// A part of the vocabulary: its first slot, its slots and the elements from there to the end of the row.  Parts are a
// whole number of 64-slot groups (the last one aside).
struct PartView {
    int lo, nslots, Vrow;
};

template <bool BF16>
__device__ inline PartView part_view(int V, int part, int split) {
    constexpr int EPV = Elem<BF16>::EPV;
    const int slots = (V + EPV - 1) / EPV, span = split > 1 ? ((slots + split - 1) / split + 63) / 64 * 64 : slots;
    const int lo = min(part * span, slots);
    return PartView{lo, min(lo + span, slots) - lo, V - lo * EPV};
}

// One exchange.  Every thread of the block calls it with the same `mine`; afterwards
// sh.xchg[j] holds what part j published.  Ends with a barrier.  A wait that runs out of its
// (very large) spin budget marks the block as failed and goes on, so that every block ends.
__device__ inline void exchange(Mailbox &mb, const double (&mine)[8], SharedState &sh) {
    if (mb.stage == 0) {  // block-uniform; (by now the epoch has arrived: the first pass did not wait for it)
        if (threadIdx.x == 0) {
            *mb.sh_epoch = mb.epoch;
            // a box that an earlier call left poisoned (one of its waits ran out) cannot be trusted
            // until the caller has zeroed it again: every part reports failure without waiting
            if (mb.epoch == kBoxPoison) sh.failed = 1;
        }
        __syncthreads();
        mb.base = *mb.sh_epoch * 1024u;
    }
    const int parity = mb.stage & 1;
    const uint32_t mark = mb.base + (uint32_t)mb.stage + 1u;
    const unsigned long long tag = (unsigned long long)mark << 32;
    if (threadIdx.x == 64) {  // (a thread of the second wave publishes, the first wave collects)
        unsigned long long *dst = mb.payload + (mb.part * 2 + parity) * 16;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned long long bits = __builtin_bit_cast(unsigned long long, mine[i]);
            __hip_atomic_store(dst + 2 * i, tag | (bits & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(dst + 2 * i + 1, tag | (bits >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if ((int)threadIdx.x < mb.split) {
        const int j = threadIdx.x;
        if (j == mb.part) {
#pragma unroll
            for (int i = 0; i < 8; ++i) sh.xchg[j][i] = mine[i];
        } else {
            const unsigned long long *src = mb.payload + (j * 2 + parity) * 16;
            unsigned long long w[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) w[i] = 0;
            if (!sh.failed) {
                int spin = 0;
                for (;;) {
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        w[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    bool all = true;
#pragma unroll
                    for (int i = 0; i < 16; ++i) all = all && (uint32_t)(w[i] >> 32) == mark;
                    if (all) break;
                    if (++spin > kSpinLimit) {
                        sh.failed = 1;
#pragma unroll
                        for (int i = 0; i < 16; ++i) w[i] = 0;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                sh.xchg[j][i] = __builtin_bit_cast(double, (w[2 * i] & 0xffffffffull) | (w[2 * i + 1] << 32));
        }
    }
    ++mb.stage;
    __syncthreads();
}

// One stage of a shared sequence: `work(j, view, mine)` does part j's share and leaves the eight numbers it publishes;
// afterwards sh.xchg holds those of all parts.  Has a barrier behind the work; the work has one of its own
// ahead of which every wave has read what the last stage left in sh.xchg.
// MEETS, and the parts did not: one work-group does their work in turn, on the same parts with the same
// threads, so that a sequence's numbers have the same bits however it was walked.
// (One copy of the work, in a loop that a part that has met runs through once: with a copy of its own for the lone work-group
// the instructions took longer to fetch, mixed temperatures, k = 3, B = 64 47.2 -> 55.2 us.)
template <bool BF16, bool MEETS, class Work>
__device__ __forceinline__ void for_parts(Mailbox &mb, const PartView &own, int V, SharedState &sh, Work &&work) {
    if constexpr (!MEETS) {
        double mine[8];
        work(mb.part, own, mine);
        exchange(mb, mine, sh);
    } else {
        PartView view = own;
#pragma unroll 1
        for (int j = mb.part;;) {  // every condition is block-uniform
            double mine[8];
            work(j, view, mine);
            if (__builtin_expect(!mb.alone, 1)) {
                exchange(mb, mine, sh);
                break;
            }
            if (threadIdx.x == 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) sh.xchg[j][i] = mine[i];
            }
            __syncthreads();
            if (++j == mb.split) break;
            view = part_view<BF16>(V, j, mb.split);
        }
    }
}

// (M, S) of a row (and, if TWO, of the drafter row) over the whole vocabulary.  This block
// streams its own part (`own`; the whole row when the sequence is not shared); with several parts the partial
// results are exchanged and combined in part order, so every part holds the same bits afterwards.  A
// part whose fast pass overflowed or came out empty repeats it by itself, the others wait for it in the exchange.
template <bool BF16, bool TWO, bool ONE_TERM, bool FULL, bool SHARED, bool PARTIAL, int TH, bool MEETS = false, class Meanwhile = Nothing>
__device__ inline void row_stats_any(const char *rowp, const char *rowq, const PartView &own, int V, SharedState &sh,
                                     int parity, Mailbox &mb, const RowMath &p, float &Mp,
                                     double &Sp, float &Mq, double &Sq, Meanwhile &&meanwhile = Nothing{}) {
    if constexpr (!FULL) meanwhile();
    if constexpr (!SHARED) {
        if constexpr (FULL) {
            if (row_stats_fast<BF16, TWO, ONE_TERM, PARTIAL, TH>(rowp, rowq, own.nslots, V, sh, parity, p, Mp, Sp, Mq, Sq, meanwhile))
                return;        // block-uniform
            __syncthreads();   // every thread has read the combine buffers of this parity
        }
        row_stats<BF16, TWO, TH>(rowp, rowq, own.nslots, V, sh, parity, p, Mp, Sp, Mq, Sq);
        return;
    }
    for_parts<BF16, MEETS>(mb, own, V, sh, [&](int, const PartView &v, double(&mine)[8]) __attribute__((always_inline)) {
        const char *vp = rowp + (size_t)v.lo * 16, *vq = rowq + (size_t)v.lo * 16;
        bool ok = false;  // block-uniform
        if (v.nslots <= 0) {  // a part without slots (tiny vocabulary): nothing to read, no mass
            if constexpr (FULL) meanwhile();
            __syncthreads();  // (in place of the pass's own: every wave has read what the last exchange brought)
            Mp = Mq = kRefInit;
            Sp = Sq = 0.0;
            ok = true;
        } else if constexpr (FULL) {
            ok = row_stats_fast<BF16, TWO, ONE_TERM, PARTIAL, TH>(vp, vq, v.nslots, v.Vrow, sh, parity, p, Mp, Sp, Mq, Sq, meanwhile);
            if (!ok) __syncthreads();  // every thread has read the combine buffers of this parity
        }
        if (!ok) row_stats<BF16, TWO, TH>(vp, vq, v.nslots, v.Vrow, sh, parity, p, Mp, Sp, Mq, Sq);
        mine[0] = (double)Mp, mine[1] = Sp, mine[2] = (double)Mq, mine[3] = Sq;
        mine[4] = mine[5] = mine[6] = mine[7] = 0.0;
    });
    // In every wave, so that no barrier is needed (the next exchange has one ahead of it): lane 8 r + j: row r (p, q)
    // of part j; one exp2 per lane.
    const int r = (threadIdx.x / kMaxSplit) & 1, j = threadIdx.x & (kMaxSplit - 1);
    const bool have = j < mb.split;
    const float m_j = have ? (float)sh.xchg[j][2 * r] : -INFINITY;
    const float M = group_max<kMaxSplit>(m_j);
    const double S = group_sum<kMaxSplit>(have ? sh.xchg[j][2 * r + 1] * exp2_f64(((double)m_j - (double)M) * p.c_d) : 0.0);
    Mp = lane_value(M, 0);
    Sp = lane_value(S, 0);
    Mq = lane_value(M, kMaxSplit);
    Sq = lane_value(S, kMaxSplit);
}

// ------------------------------------------------------------------------------------------
// mailboxes of the library's own, for entry points that have no workspace argument
// ------------------------------------------------------------------------------------------
// A call's parts meet before the walk begins: each enters its bit in the state word of its sequence's box, and
// only if all of them turn up in time is the sequence shared (then all of them run, so that every later wait ends).
// Otherwise whoever gives up leaves the box free again, part 0 does the work of all parts (for_parts) and the others
// end.  All of it is one compare-and-swap per step on one word, so the parts agree: a box's word goes from "all
// arrived" to "free" only when every part has left.  A box that belongs to another call in flight (they take
// turns over kClaimRegions sets of boxes, by a number of the call that its replays keep) counts as not
// found, and so does one whose call never ended: such sequences are walked alone.
//
// What that costs, us per call, V = 151,936 bf16, shared / every sequence alone / unshared kernels: mixed temperatures,
// k = 3, B = 32, 64, 128 46, 47, 61 / 126, 128, 93 / 79, 79, 81; trees of 3 x 2 at T = 0.6, B = 64, 128 68, 78 / 101, 108 /
// 88, 89; and up to kClaimTicks ahead of it.  Beside another stream's kernels (shared where they meet / unshared): a copy of
// 1 GB 83, 89, 111 / 149, 152, 156 and 128, 139 / 187, 193; matrix products of 8192, between whose work-groups both wait for
// compute units, 885, 861, 838 / 820, 829, 850 and 866, 869 / 867, 866.
//
// State word: epoch (22 bits: uses of the box, what the marks in its payload are made from), key of the call that
// holds it (30 bits, 0: free), parts that have arrived (4), parts that have left (4).
constexpr int kClaimSplit = 4;      // parts of a sequence
constexpr int kClaimGroups = 256;   // work-groups of a call
constexpr int kClaimRegions = 32;
constexpr size_t kClaimBoxBytes = kBoxHeaderBytes + (size_t)kClaimSplit * 2 * 16 * 8;
constexpr int kClaimBoxes = kClaimGroups / 2;  // per region: at least two parts each
static __device__ __align__(256) unsigned char claim_boxes[kClaimRegions * kClaimBoxes * kClaimBoxBytes];
constexpr unsigned long long kClaimEpoch = (1ull << 22) - 1, kClaimKey = ((1ull << 30) - 1) << 22;
constexpr int kClaimArrived = 52, kClaimLeft = 56;

__device__ inline unsigned long long *claim_box(uint32_t key, int b) {
    return reinterpret_cast<unsigned long long *>(claim_boxes + ((size_t)(key % kClaimRegions) * kClaimBoxes + b) * kClaimBoxBytes);
}

// One thread of each part calls this; true: all parts are here, `epoch` is the box's.  ticks: 10 ns each, how long
// the others are waited for (negative: the box is left alone, and so is every sequence).
__device__ inline bool claim_arrive(unsigned long long *state, uint32_t key, int part, int split, int ticks, uint32_t &epoch) {
    if (ticks < 0) return false;
    const unsigned long long mine = (unsigned long long)key << 22, bit = 1ull << (kClaimArrived + part);
    const unsigned long long all = ((1ull << split) - 1) << kClaimArrived;
    auto swap = [&](unsigned long long &seen, unsigned long long want) {  // on failure `seen` is what the word holds
        return __hip_atomic_compare_exchange_strong(state, &seen, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    unsigned long long s = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int turn = 0;; ++turn) {
        unsigned long long want;
        if ((s & kClaimKey) == 0) want = (s & kClaimEpoch) | mine | bit;
        else if ((s & kClaimKey) == mine && (s >> kClaimLeft) == 0 && !(s & bit)) want = s | bit;
        else return false;
        if (turn == 64) return false;
        if (swap(s, want)) {
            s = want;
            break;
        }
    }
    epoch = (uint32_t)(s & kClaimEpoch);
    const uint64_t start = __builtin_amdgcn_s_memrealtime();
    while ((s & all) != all) {
        if ((int64_t)(__builtin_amdgcn_s_memrealtime() - start) >= ticks) {
            if (swap(s, (s + 1) & kClaimEpoch)) return false;
        } else {
            __builtin_amdgcn_s_sleep(1);
            s = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if ((s & kClaimKey) != mine || (uint32_t)(s & kClaimEpoch) != epoch) return false;  // another part gave up
    }
    return true;
}

// Every thread of a part calls this; true: the sequence is shared, `epoch` (uniform) is the box's.
__device__ inline bool claim_meet(unsigned long long *state, uint32_t key, int part, int split, int ticks, uint32_t *sh_epoch, SharedState &sh,
                                  uint32_t &epoch) {
    if (threadIdx.x == 0) {
        uint32_t e = 0;
        sh.failed = 0;
        sh.token = claim_arrive(state, key, part, split, ticks, e) ? 1 : 0;
        *sh_epoch = e;
    }
    __syncthreads();
    epoch = (uint32_t)__builtin_amdgcn_readfirstlane((int)*sh_epoch);
    return __builtin_amdgcn_readfirstlane(sh.token) != 0;
}

// One thread of each part of a shared sequence, behind its last exchange.
__device__ inline void claim_leave(unsigned long long *state, int split, uint32_t epoch) {
    const unsigned long long before = __hip_atomic_fetch_add(state, 1ull << kClaimLeft, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((int)(before >> kClaimLeft) == split - 1)
        __hip_atomic_store(state, ((unsigned long long)epoch + 1) & kClaimEpoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline Mailbox claim_mailbox(unsigned long long *state, int part, int split, uint32_t epoch, uint32_t *sh_epoch, bool alone) {
    return Mailbox{reinterpret_cast<uint32_t *>(state), state + kBoxHeaderBytes / sizeof(*state), 0u, part, split, 0, epoch, sh_epoch, alone};
}

// The key of a call.
inline uint32_t next_claim_key() {
    static std::atomic<uint32_t> calls{0};
    return calls.fetch_add(1, std::memory_order_relaxed) % ((1u << 30) - 1) + 1;
}

// How long a part waits for the others (10 ns ticks): they are launched together and meet within 2 us; where another stream's kernels
// hold the compute units a part may be missing for as long as those run.
constexpr int kClaimTicks = 2000;

}  // namespace
}  // namespace respec
