// Reward-weighted knowledge distillation of the drafter, per logits row, for gfx950
// (Section 5.3, "Reward-Weighted Knowledge Distillation"; Algorithm 1): for every row
//     loss = w * KL(p || q),  p = softmax(target row),  q = softmax(drafter row),
// and the gradient with respect to the drafter's logits, w * (q - p).  w is the weight w(r) of
// the row's sample, supplied per row.
//
// The gradient of a row needs both normalisers of the row first, so a row pair has to be kept, or
// read twice, between the two passes over it.  kd_team_kernel keeps it: a team of work-groups holds
// a row pair in its LDS, a part each, and exchanges the parts' normalisers through the workspace.
// kd_stream_kernel is the form for rows too long for any team, for rows that a team does not pay for (kd_team), for a gradient
// written over its inputs where a team would have several members, and for workspaces without room for the
// exchange: one work-group per row pair, which it streams twice.
//
// Numerics: exp2 of one element in fp32 (hardware exp2, two-term constant), row sums carried in
// fp64, p and q formed in the log2 domain in fp32 (relative error about 2e-6), the KL terms
// summed per thread in fp32 over one batch of slots (at most 32 terms) and in fp64 from there on.
#include "respec_kd_absent.hpp"
#include "respec_sampler_rows.hpp"

#include <algorithm>
#include <type_traits>
#include <utility>

// v_mul_legacy_f32: zero times anything is zero.  (The intrinsic and not an asm statement: its operand comes
// straight from v_exp_f32, whose result the next vector instruction may not read; the compiler
// puts the wait state between the two only where it knows both instructions.)
extern "C" __device__ float legacy_mul(float, float) __asm("llvm.amdgcn.fmul.legacy");

namespace respec {
namespace {

// Both kernels form an exponent's argument with one multiply-add: the temperature is 1, and log2(e) rounds well
// (RowMath::one_term).
constexpr double kLog2e = 1.4426950408889634074;
static_assert((double)(float)kLog2e / kLog2e - 1.0 <= 2.0e-8 && 1.0 - (double)(float)kLog2e / kLog2e <= 2.0e-8);

struct KdParams : RowMath {
    const void *target;
    const void *draft;
    const float *weight;
    void *grad;
    float *row_loss;
    double *total_loss;
    double *row_kl;      // [rows][team] unweighted KL of every row, by parts
    uint64_t *box;       // [rows][team][kKdBoxWords] tagged words: the parts' normalisers
    int32_t rows, V;
    int64_t ld_t, ld_d, ld_g;
    int32_t team;        // work-groups that share a row pair (1 in kd_stream_kernel)
    int32_t part_slots;  // 16-byte slots of a row that each of them takes
    int32_t spin;        // 10 ns ticks that a part is waited for before it is computed here
};

struct KdShared {
    SharedState rows;                 // reduction buffers of the row primitives
    double loss_wave[kWaves];
};

template <bool BF16>
__device__ inline void store_grad(void *dst, const float (&g)[Elem<BF16>::EPV]) {
    if constexpr (BF16) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float floatx2 __attribute__((ext_vector_type(2)));
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            w[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{g[2 * j], g[2 * j + 1]}, bf16x2));
        // (written once and not read here: the non-temporal hint keeps the stores from
        // displacing the rows that pass 2 is about to read again; 605 -> 570 us on 2048 rows)
        __builtin_nontemporal_store(u32x4{w[0], w[1], w[2], w[3]}, reinterpret_cast<u32x4 *>(dst));
    } else {
        __builtin_nontemporal_store(
            u32x4{__float_as_uint(g[0]), __float_as_uint(g[1]), __float_as_uint(g[2]), __float_as_uint(g[3])},
            reinterpret_cast<u32x4 *>(dst));
    }
}

// Work-group g takes rows g, g + gridDim.x, ...  Pass 2 walks a row back to front: what pass 1
// read last is the most likely to be still in a cache.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void kd_stream_kernel(KdParams p) {
    constexpr int EPV = Elem<BF16>::EPV;
    constexpr int kBatch = kThreads * kUnroll;
    __shared__ KdShared sh;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nslots = p.V / EPV;
    const int n_iter = (nslots + kBatch - 1) / kBatch;
    const size_t esz = BF16 ? 2 : 4;
    int parity = 0;
    for (int r = blockIdx.x; r < p.rows; r += gridDim.x) {
        const float w = p.weight[r];
        char *g = static_cast<char *>(p.grad) + (size_t)r * p.ld_g * esz;
        if (w == 0.f) {  // block-uniform: the row is not read
            for (int s = threadIdx.x; s < nslots; s += kThreads)
                *reinterpret_cast<u32x4 *>(g + (size_t)s * 16) = u32x4{0u, 0u, 0u, 0u};
            if (threadIdx.x == 0) p.row_kl[r] = 0.0;
            continue;
        }
        const char *rp = static_cast<const char *>(p.target) + (size_t)r * p.ld_t * esz;
        const char *rq = static_cast<const char *>(p.draft) + (size_t)r * p.ld_d * esz;
        float Mp, Mq;
        double Sp, Sq;
        if (!row_stats_fast<BF16, true, true>(rp, rq, nslots, p.V, sh.rows, parity, p, Mp, Sp, Mq, Sq)) {
            __syncthreads();  // block-uniform: an overflow or an empty sum, repeat with running references
            row_stats<BF16, true>(rp, rq, nslots, p.V, sh.rows, parity, p, Mp, Sp, Mq, Sq);
        }
        parity ^= 1;
        // The log2 of a probability is one multiply-add, z c_f + K with K = -M c_f - log2(S) rounded to
        // binary32; what the rounding of K leaves out (dKa, dKb, a few 1e-7) shifts every term
        // of the row's KL alike and is put back once per row.
        const double ka = -(double)Mp * (double)p.c_f - log2(Sp), kb = -(double)Mq * (double)p.c_f - log2(Sq);
        const float Ka = (float)ka, Kb = (float)kb;
        const double kl_shift = (ka - (double)Ka) - (kb - (double)Kb);
        auto load_batch = [&](int it, u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int s = it * kBatch + u * kThreads + (int)threadIdx.x;
                const int safe = s < nslots ? s : 0;
                // (the rows' last read: non-temporal, 568 -> 532 us on 2048 rows)
                vp[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(rp + (size_t)safe * 16));
                vq[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(rq + (size_t)safe * 16));
            }
        };
        double kl = 0.0;
        // `whole`: every slot of the batch lies inside the row (all batches but the row's last, which the pass takes first)
        auto work_batch = [&](int it, const u32x4 (&xp)[kUnroll], const u32x4 (&xq)[kUnroll], auto whole) __attribute__((always_inline)) {
            float klb = 0.f;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int s = it * kBatch + u * kThreads + (int)threadIdx.x;
                if (decltype(whole)::value || s < nslots) {
                    float zp[EPV], zq[EPV], gr[EPV];
                    unpack<BF16>(xp[u], zp);
                    unpack<BF16>(xq[u], zq);
#pragma unroll
                    for (int j = 0; j < EPV; ++j) {
                        const float a = fmaf(zp[j], p.c_f, Ka), b = fmaf(zq[j], p.c_f, Kb);
                        const float pe = hw_exp2(a), qe = hw_exp2(b);
                        // (a token without target mass adds nothing, whatever a - b is then, -inf
                        // minus -inf included: the legacy multiply takes 0 times anything as 0)
                        klb += legacy_mul(pe, a - b);
                        gr[j] = w * (qe - pe);
                    }
                    store_grad<BF16>(g + (size_t)s * 16, gr);
                }
                __builtin_amdgcn_sched_barrier(0);  // one slot at a time: interleaving all of them spills
            }
            kl += (double)klb;
        };
        // two register sets take turns: one batch is worked on while the next one's loads are in
        // flight.  (The loads of the steady state are unconditional: behind a condition the wait
        // for the batch in front of a load becomes a wait for everything in flight.)
        auto pass2 = [&]() __attribute__((always_inline)) {
            constexpr std::true_type whole{};
            u32x4 vp[kUnroll], vq[kUnroll], wp[kUnroll], wq[kUnroll];
            load_batch(n_iter - 1, vp, vq);
            if (n_iter == 1) {
                work_batch(0, vp, vq, std::false_type{});
                return;
            }
            load_batch(n_iter - 2, wp, wq);
            work_batch(n_iter - 1, vp, vq, std::false_type{});  // the row's last, ragged batch
            int it = n_iter - 2;  // wp holds batch `it`
            for (; it >= 2; it -= 2) {
                load_batch(it - 1, vp, vq);
                work_batch(it, wp, wq, whole);
                load_batch(it - 2, wp, wq);
                work_batch(it - 1, vp, vq, whole);
            }
            if (it == 1) {
                load_batch(0, vp, vq);
                work_batch(1, wp, wq, whole);
                work_batch(0, vp, vq, whole);
            } else {
                work_batch(0, wp, wq, whole);
            }
        };
        pass2();
        // KL(p || q) of the row in nats, summed in a fixed order
        const double kw = wave_sum(kl);
        if (lane == 0) sh.loss_wave[wave] = kw;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int x = 0; x < kWaves; ++x) t += sh.loss_wave[x];
            // (sum_x p(x) = 1)
            p.row_kl[r] = (t + kl_shift) * 0.69314718055994530942;
        }
        // (the next row's normaliser pass has a barrier before anything writes loss_wave again)
    }
}

// ---------------------------------------------------------------- a row pair kept in a team's LDS
constexpr int kKdThreads = kThreads + 64;  // eight streaming waves and the one that exchanges normalisers
constexpr int kKdChunk = 64;               // slots of a wave's piece: a lane's 16 bytes each
constexpr int kKdMaxChunks = 38;           // pieces of a part: two rows, two buffers, 152 KiB of LDS
constexpr int kKdMaxTeam = 32;
constexpr int kKdFill = 256;               // compute units that few rows are spread over
constexpr int kKdBoxWords = 8;             // a part's sums (two words each) and references; two words spare: 64 bytes
constexpr uint32_t kKdTag = 1u;            // in the upper half of every word (the words are cleared ahead of the kernel)

struct KdTeamShared {
    float m[2][2][kWaves];        // [row parity][p/q][wave]: reference and sum of a wave's pieces
    double s[2][2][kWaves];
    double kl[2][kWaves];
    uint32_t pay[kKdMaxTeam][kKdBoxWords];
    float K[2][2];                // [row parity][p/q]: constants of the gradient pass
    double shift[2];              // [row parity]: what the row's KL gets for their rounding
    int row[2];                   // [row parity]: the row
    uint32_t stats_seq[kWaves];   // rows whose m, s (kl) a wave has left, and whose K is there
    uint32_t kl_seq[kWaves];
    uint32_t const_seq;
};

typedef volatile uint32_t __attribute__((address_space(3))) *KdCounter;

// (a wave's LDS operations execute in order: a counter written after the data needs no fence, only
// the compiler kept from moving it)
__device__ inline void kd_set(uint32_t &word, uint32_t v) {
    asm volatile("" ::: "memory");
    *(KdCounter)&word = v;
}

__device__ inline void kd_wait(uint32_t &word, uint32_t v) {
    while (*(KdCounter)&word < v) __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
}

// 16 bytes per lane, global memory to LDS (lane i to lds + 16 i), counted by vmcnt.  Non-temporal:
// every row is read once.  (No result register, so nothing to keep alive.  The instruction takes the LDS address from m0,
// whose write needs one wait state, and its base from scalar registers, which need five if a vector instruction
// wrote them last, as the reload of a spilled one does.  A scalar move of the base needs none, and is the wait state of m0;
// three more idle states cost 2048 rows of 151,936 logits 0.7 %.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // (m0 is reserved: never allocated, but set by the compiler for its own use)
__device__ inline void kd_load_to_lds(uint32_t lds, const char *base, uint32_t off) {
    const char *from;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0 nt" : "=&s"(from) : "s"(lds), "v"(off), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop

// Waits until at most n vector memory operations of the wave are outstanding (they complete in issue order).
__device__ inline void kd_wait_vm(int n) {
    switch (n) {  // wave-uniform
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
        case 7: asm volatile("s_waitcnt vmcnt(7)" ::: "memory"); break;
        case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
        case 9: asm volatile("s_waitcnt vmcnt(9)" ::: "memory"); break;
        case 10: asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); break;
        case 11: asm volatile("s_waitcnt vmcnt(11)" ::: "memory"); break;
        case 12: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
        case 13: asm volatile("s_waitcnt vmcnt(13)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

// Reference and sum of one wave's pieces of a row pair: S = sum exp(z - M), the same bits wherever
// the pieces are read from.  load(c, vp, vq) gives piece c, -inf past the part's end.  The
// reference is the largest element of the first piece; a wave whose first piece has no finite element, or
// whose sum overflows, takes its pieces again with running references (kRefInit, 0 for none at all).
template <bool BF16, class Load>
__device__ inline void kd_wave_stats(int n_pieces, const RowMath &p, float (&M)[2], double (&S)[2], Load &&load) {
    constexpr int EPV = Elem<BF16>::EPV;
    float acc[2][EPV], K[2] = {0.f, 0.f};
    bool ok = true;
    M[0] = M[1] = kRefInit;
    S[0] = S[1] = 0.0;
    if (n_pieces == 0) return;
#pragma unroll
    for (int j = 0; j < EPV; ++j) acc[0][j] = acc[1][j] = 0.f;
    for (int c = 0; c < n_pieces; ++c) {
        u32x4 v[2];
        load(c, v[0], v[1], true);
        if (c == 0) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                M[r] = wave_max(slot_max<BF16>(v[r]));
                ok = ok && M[r] > -INFINITY && M[r] < INFINITY;
                K[r] = -M[r] * p.c_f;
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) fast_absorb<BF16, true>(v[r], acc[r], M[r], K[r], p);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < EPV; ++j) t += (double)acc[r][j];
        S[r] = wave_sum(t);
        ok = ok && S[r] < 1.0e300;
    }
    if (ok) {  // wave-uniform
        // exp2(z c_f + K) with K rounded: the residue, at most 2^-24 of |K|, is put back to second order
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const double d = 0.69314718055994530942 * ((double)K[r] + (double)M[r] * (double)p.c_f);
            S[r] *= 1.0 - d + 0.5 * d * d;
        }
        return;
    }
    ThreadSum<BF16> t[2];
    t[0].init();
    t[1].init();
    for (int c = 0; c < n_pieces; ++c) {
        u32x4 v[2];
        load(c, v[0], v[1], false);
        t[0].absorb(v[0], p);
        t[1].absorb(v[1], p);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        M[r] = wave_max(t[r].ref);
        S[r] = wave_sum(t[r].total() * exp2_f64((double)(t[r].ref - M[r]) * p.c_d));
    }
}

// (M, S) over groups of LANES neighbouring lanes; every lane of a group gets the same bits.
template <int LANES>
__device__ inline void kd_fold(float &M, double &S, const RowMath &p) {
    static_assert(LANES == 8 || LANES == 32);
    float mm = dpp_max<kDppOtherQuad>(dpp_max<kDppXor2>(dpp_max<kDppXor1>(M)));
    if constexpr (LANES == 32) {
        mm = dpp_max<kDppOtherEight>(mm);
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(mm), __float_as_uint(mm), false, false);
        mm = fmaxf(as_f32(x[0]), as_f32(x[1]));
    }
    double t = S * exp2_f64((double)(M - mm) * p.c_d);
    t = dpp_add<kDppOtherQuad>(dpp_add<kDppXor2>(dpp_add<kDppXor1>(t)));
    if constexpr (LANES == 32) {
        t = dpp_add<kDppOtherEight>(t);
        const uint64_t u = __builtin_bit_cast(uint64_t, t);
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
        t = __builtin_bit_cast(double, (uint64_t)lo[0] | ((uint64_t)hi[0] << 32)) + __builtin_bit_cast(double, (uint64_t)lo[1] | ((uint64_t)hi[1] << 32));
    }
    M = mm;
    S = t;
}

// Team t takes the rows t, t + teams, ... of those whose weight is not zero; member m of it the slots
// [m, m + 1) * part_slots of each.  A streaming wave goes through its pieces of row i + 1 (sums for the
// normalisers), then of row i (gradient, whose constants have had that long to arrive); a piece
// of row i + 2 is requested into the same place as soon as one of row i has been read, so a row is read from
// memory once and the exchange is not waited for.  Nothing but counters in LDS orders the waves.
//
// What bounds it: HBM.  2048 rows of 151,936 bf16 logits 438 us (one work-group per row pair, read twice) -> 370 us; a
// kernel that reads two arrays of that size and writes a third takes 328 us, this one without its wait for the other
// members 352, without its stores as well 237, the arithmetic alone 199.
// Also measured: all requests of a row ahead of its gradients' stores 402 us (their issue blocks), requests from three
// waves of their own, so that no streaming wave waits for its stores' acknowledgements 465 us; plain instead of
// non-temporal stores 404 us, plain loads 387 us.
//
// A member that does not answer within `spin` (its work-group is not running yet: another stream's kernels
// hold the device) is not needed: its part is computed from the rows, with the same operations in the same order, by one wave
// of every other member; on the rows behind that it is waited for a sixteenth as long until it answers again (KdAbsent).
// Beside other streams' kernels the form is no slower than one work-group per row pair that streams it twice (2048 rows of 151,936
// bf16 logits, us per call, streamed / by teams, and ms until both streams were done: beside attention over 256 sequences
// 632 / 587, 9.9 / 8.8; samplers of 64 sequences 464 / 427, 10.3 / 9.2; bf16 products of 8192 818 / 722, 9.8 / 8.7 (9.4 to
// 9.8 when an absent member was waited for in full on every row); scans of 32 long rows 483 / 487, 13.0 / 10.5).
template <bool BF16>
__global__ __launch_bounds__(kKdThreads) void kd_team_kernel(KdParams p) {
    constexpr int EPV = Elem<BF16>::EPV;
    extern __shared__ u32x4 kd_rows_lds[];  // [buffer][piece][p/q][lane]
    __shared__ KdTeamShared sh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int member = (int)(blockIdx.x % (unsigned)p.team), first_row = (int)(blockIdx.x / (unsigned)p.team);
    const int teams = (int)(gridDim.x / (unsigned)p.team);
    const size_t esz = BF16 ? 2 : 4;
    const int nslots = p.V / EPV;
    const int n_pieces = (p.part_slots + kKdChunk - 1) / kKdChunk;
    typedef const float __attribute__((address_space(4))) *ConstWeight;  // scalar loads: they do not count with the pieces'
    const ConstWeight weight = (ConstWeight)(uintptr_t)p.weight;
    if (threadIdx.x < kWaves) sh.stats_seq[threadIdx.x] = sh.kl_seq[threadIdx.x] = 0;
    if (threadIdx.x == 0) sh.const_seq = 0;
    __syncthreads();
    auto row_of = [&](const void *base, int64_t ld, int r) { return static_cast<const char *>(base) + (size_t)r * ld * esz; };

    if (wave < kWaves) {
        const int begin = member * p.part_slots, end = min(begin + p.part_slots, nslots);  // (end <= begin: nothing)
        const int mine = end > begin ? ((end - begin + kKdChunk - 1) / kKdChunk - wave + kWaves - 1) / kWaves : 0;
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)kd_rows_lds;
        auto slot_of = [&](int c) { return begin + (c * kWaves + wave) * kKdChunk + lane; };
        auto place = [&](int buf, int c) { return ((buf * n_pieces + c * kWaves + wave) * 2) * kKdChunk; };  // in slots
        auto request = [&](int r, int buf, int c) __attribute__((always_inline)) {
            const uint32_t off = (uint32_t)min(slot_of(c), end - 1) * 16u;
            const uint32_t at = lds0 + (uint32_t)place(buf, c) * 16u;
            kd_load_to_lds(at, row_of(p.target, p.ld_t, r), off);
            kd_load_to_lds(at + kKdChunk * 16u, row_of(p.draft, p.ld_d, r), off);
        };
        // the next of the team's rows from r on whose weight is not zero; gradients of the others are zero
        auto next_row = [&](int r) __attribute__((always_inline)) {
            while (r < p.rows && weight[r] == 0.f) {
                char *g = static_cast<char *>(p.grad) + (size_t)r * p.ld_g * esz;
                for (int c = 0; c < mine; ++c)
                    if (slot_of(c) < end) *reinterpret_cast<u32x4 *>(g + (size_t)slot_of(c) * 16) = u32x4{0u, 0u, 0u, 0u};
                r += teams;
            }
            return r;
        };
        // the sums over row number i (the i-th with a weight)
        auto stats = [&](int i) __attribute__((always_inline)) {
            float M[2];
            double S[2];
            kd_wave_stats<BF16>(mine, p, M, S, [&](int c, u32x4 &vp, u32x4 &vq, bool first) __attribute__((always_inline)) {
                // (behind piece c's requests: two for each further piece, and where they were made by the
                // gradient pass a store for each and for c)
                if (first) kd_wait_vm((mine - 1 - c) * (i < 2 ? 2 : 3) + (i < 2 ? 0 : 1));
                vp = kd_rows_lds[place(i & 1, c) + lane];
                vq = kd_rows_lds[place(i & 1, c) + kKdChunk + lane];
                if (slot_of(c) - lane + kKdChunk > end) {  // the part's last, ragged piece
                    vp = slot_of(c) < end ? vp : neg_inf_slot<BF16>();
                    vq = slot_of(c) < end ? vq : neg_inf_slot<BF16>();
                }
            });
            if (lane < 2) {
                sh.m[i & 1][lane][wave] = lane ? M[1] : M[0];
                sh.s[i & 1][lane][wave] = lane ? S[1] : S[0];
            }
            kd_set(sh.stats_seq[wave], (uint32_t)i + 1);
        };
        // the gradient of row number i, at r, and its KL terms; requests row r2 into the places that become free
        auto gradient = [&](int i, int r, int r2) __attribute__((always_inline)) {
            kd_wait(sh.const_seq, (uint32_t)i + 1);
            const float Ka = as_f32(__builtin_amdgcn_readfirstlane((int)__float_as_uint(sh.K[i & 1][0])));
            const float Kb = as_f32(__builtin_amdgcn_readfirstlane((int)__float_as_uint(sh.K[i & 1][1])));
            const float w = weight[r];
            char *g = static_cast<char *>(p.grad) + (size_t)r * p.ld_g * esz;
            double kl = 0.0;
            for (int c = 0; c < mine; ++c) {
                const u32x4 vp = kd_rows_lds[place(i & 1, c) + lane];
                const u32x4 vq = kd_rows_lds[place(i & 1, c) + kKdChunk + lane];
                if (r2 < p.rows) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::"v"(vp), "v"(vq) : "memory");  // the piece has left LDS
                    request(r2, i & 1, c);
                }
                float zp[EPV], zq[EPV], gr[EPV], klc = 0.f;
                unpack<BF16>(vp, zp);
                unpack<BF16>(vq, zq);
#pragma unroll
                for (int j = 0; j < EPV; ++j) {
                    const float a = fmaf(zp[j], p.c_f, Ka), b = fmaf(zq[j], p.c_f, Kb);
                    const float pe = hw_exp2(a), qe = hw_exp2(b);
                    // (a token without target mass adds nothing, whatever a - b is then, -inf
                    // minus -inf included: the legacy multiply takes 0 times anything as 0)
                    klc += legacy_mul(pe, a - b);
                    gr[j] = w * (qe - pe);
                }
                if (slot_of(c) < end) {
                    store_grad<BF16>(g + (size_t)slot_of(c) * 16, gr);
                    kl += (double)klc;
                }
            }
            kl = wave_sum(kl);
            if (lane == 0) sh.kl[i & 1][wave] = kl;
            kd_set(sh.kl_seq[wave], (uint32_t)i + 1);
        };
        int r0 = next_row(first_row);
        if (r0 >= p.rows) return;
        for (int c = 0; c < mine; ++c) request(r0, 0, c);
        int r1 = next_row(r0 + teams);
        if (r1 < p.rows)
            for (int c = 0; c < mine; ++c) request(r1, 1, c);
        stats(0);
        for (int i = 0; r0 < p.rows; ++i) {
            const int r2 = r1 < p.rows ? next_row(r1 + teams) : p.rows;
            if (r1 < p.rows) stats(i + 1);
            gradient(i, r0, r2);
            r0 = r1;
            r1 = r2;
        }
        return;
    }

    // the exchanging wave
    auto next_row = [&](int r) {
        while (r < p.rows && weight[r] == 0.f) r += teams;
        return r;
    };
    KdAbsent absent;  // wave-uniform
    auto write_kl = [&](int i) {  // of row number i
        double t = lane < kWaves ? sh.kl[i & 1][lane] : 0.0;
#pragma unroll
        for (int o = kWaves / 2; o >= 1; o >>= 1) t += __shfl_xor(t, o);
        if (lane == 0) p.row_kl[(size_t)sh.row[i & 1] * p.team + member] = (member == 0 ? t + sh.shift[i & 1] : t) * 0.69314718055994530942;
    };
    auto fold_waves = [&](float M, double S) {  // lanes 0..7: the p row's waves, 8..15: the q row's
        kd_fold<kWaves>(M, S, p);
        return std::pair<float, double>(M, S);
    };
    auto set_pay = [&](int m, float M, double S) {
        if (lane == 0 || lane == 8) {
            const int r = lane >> 3;
            const uint64_t u = __builtin_bit_cast(uint64_t, S);
            sh.pay[m][2 * r] = (uint32_t)u;
            sh.pay[m][2 * r + 1] = (uint32_t)(u >> 32);
            sh.pay[m][4 + r] = __float_as_uint(M);
        }
        asm volatile("" ::: "memory");
    };
    int i = 0;
    for (int r = next_row(first_row); r < p.rows; r = next_row(r + teams), ++i) {
        while (__any(*(KdCounter)&sh.stats_seq[lane & 7] < (uint32_t)i + 1)) {}
        asm volatile("" ::: "memory");
        const auto own = fold_waves(sh.m[i & 1][(lane >> 3) & 1][lane & 7], sh.s[i & 1][(lane >> 3) & 1][lane & 7]);
        set_pay(member, own.first, own.second);
        if (p.team == 1) {
            if (i >= 2) write_kl(i);
        } else {
            uint64_t *box = p.box + (size_t)r * p.team * kKdBoxWords;
            if (lane < 6)
                __hip_atomic_store(box + member * kKdBoxWords + lane, (uint64_t)sh.pay[member][lane] | ((uint64_t)kKdTag << 32),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            constexpr int kPer = kKdMaxTeam * kKdBoxWords / 64;
            uint32_t missing = 0;  // bit u: this lane's word u
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int idx = u * 64 + lane, m = idx / kKdBoxWords;
                if (m < p.team && m != member && idx % kKdBoxWords < 6) missing |= 1u << u;
            }
            if (i >= 2) write_kl(i);  // of row number i - 2, which all waves have passed
            const uint64_t t0 = wall_clock64();
            for (;;) {
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    if (u * 64 >= p.team * kKdBoxWords) break;
                    if (missing & (1u << u)) {
                        const int idx = u * 64 + lane;
                        const uint64_t v = __hip_atomic_load(box + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if ((uint32_t)(v >> 32) == kKdTag) {
                            sh.pay[idx / kKdBoxWords][idx % kKdBoxWords] = (uint32_t)v;
                            missing &= ~(1u << u);
                        }
                    }
                }
                if (!__any(missing != 0)) break;
                const uint64_t waited = wall_clock64() - t0;
                uint32_t give_up = 0;
                if (waited >= (uint64_t)p.spin || absent.known != 0) {
                    uint32_t late = 0;  // members with a missing word
#pragma unroll
                    for (int u = 0; u < kPer; ++u) {
                        const unsigned long long b = __ballot((missing & (1u << u)) != 0);
#pragma unroll
                        for (int x = 0; x < 64 / kKdBoxWords; ++x)
                            if ((b >> (x * kKdBoxWords)) & 0xff) late |= 1u << (u * (64 / kKdBoxWords) + x);
                    }
                    give_up = absent.give_up(late, waited, (uint64_t)p.spin);
                }
                while (give_up != 0) {
                    const int m = __builtin_ctz(give_up);
                    give_up &= give_up - 1;
                    const int b0 = m * p.part_slots, e0 = min(b0 + p.part_slots, nslots);
                    const char *rp = row_of(p.target, p.ld_t, r), *rq = row_of(p.draft, p.ld_d, r);
                    float Ml = kRefInit;
                    double Sl = 0.0;
                    for (int w = 0; w < kWaves; ++w) {
                        float M[2];
                        double S[2];
                        const int n = e0 > b0 ? ((e0 - b0 + kKdChunk - 1) / kKdChunk - w + kWaves - 1) / kWaves : 0;
                        kd_wave_stats<BF16>(n, p, M, S, [&](int c, u32x4 &vp, u32x4 &vq, bool) __attribute__((always_inline)) {
                            const int s = b0 + (c * kWaves + w) * kKdChunk + lane;
                            vp = load_slot<BF16, true, false, true>(rp, min(s, e0 - 1), 0);
                            vq = load_slot<BF16, true, false, true>(rq, min(s, e0 - 1), 0);
                            vp = s < e0 ? vp : neg_inf_slot<BF16>();
                            vq = s < e0 ? vq : neg_inf_slot<BF16>();
                        });
                        if ((lane & 7) == w) {
                            Ml = lane & 8 ? M[1] : M[0];
                            Sl = lane & 8 ? S[1] : S[0];
                        }
                    }
                    const auto part = fold_waves(Ml, Sl);
                    set_pay(m, part.first, part.second);
#pragma unroll
                    for (int u = 0; u < kPer; ++u)
                        if ((u * 64 + lane) / kKdBoxWords == m) missing &= ~(1u << u);
                }
                __builtin_amdgcn_s_sleep(1);
            }
            absent.row_done();
        }
        // lanes 0..31: the members' p parts, 32..63: the q parts
        const int m = lane & 31, which = lane >> 5;
        float M = kRefInit;
        double S = 0.0;
        if (m < p.team) {
            M = as_f32(sh.pay[m][4 + which]);
            S = __builtin_bit_cast(double, (uint64_t)sh.pay[m][2 * which] | ((uint64_t)sh.pay[m][2 * which + 1] << 32));
        }
        kd_fold<32>(M, S, p);
        // The log2 of a probability is one multiply-add, z c_f + K with K = -M c_f - log2(S) rounded to
        // binary32; what the rounding leaves out (a few 1e-7) shifts every term of the row's KL alike
        // and is put back once per row, since the probabilities sum to one.
        const double k = -(double)M * (double)p.c_f - log2(S);
        const float K = (float)k;
        const double rest = k - (double)K;
        sh.shift[i & 1] = lane_value(rest, 0) - lane_value(rest, 32);
        sh.row[i & 1] = r;
        if (m == 0) sh.K[i & 1][which] = K;
        kd_set(sh.const_seq, (uint32_t)i + 1);
    }
    for (int x = max(0, i - 2); x < i; ++x) {
        for (int w = 0; w < kWaves; ++w) kd_wait(sh.kl_seq[w], (uint32_t)x + 1);
        write_kl(x);
    }
}

// The words that the members exchange, cleared ahead of the kernel.
__global__ __launch_bounds__(256) void kd_clear_kernel(u32x4 *words, size_t n) {
    for (size_t x = blockIdx.x * 256u + threadIdx.x; x < n; x += (size_t)gridDim.x * 256u) words[x] = u32x4{0u, 0u, 0u, 0u};
}

// row_loss[r] = w[r] * KL of the row; total = sum over rows in a fixed order.  One work-group.
__global__ __launch_bounds__(1024) void kd_finish_kernel(KdParams p) {
    __shared__ double sh[1024];
    double acc = 0.0;
    for (int r = threadIdx.x; r < p.rows; r += 1024) {
        double l = 0.0;
        if (p.weight[r] != 0.f) {
            double kl = 0.0;
#pragma unroll 8
            for (int m = 0; m < p.team; ++m) kl += p.row_kl[(size_t)r * p.team + m];
            l = (double)p.weight[r] * kl;
        }
        p.row_loss[r] = (float)l;
        acc += l;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 512; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0 && p.total_loss) *p.total_loss = sh[0];
}

// Work-groups that share a row pair, 0 for one that streams it twice.  The smallest power of two whose
// members' parts fit their LDS; few rows are shared by more, as long as every streaming wave
// keeps a piece of its own, until the device is full.  Times in us, streamed twice / by a team:
//   - a row pair that one work-group can keep needs no exchange and is always better kept: bf16, V = 8000, 100 rows
//     11.5 / 10.3, 2048 rows 57 / 35; V = 16,000, 2048 rows 70 / 50;
//   - longer ones cost the exchange and one more small kernel (about 4 us).  Few rows: worth it from 48,000 logits on (bf16,
//     V = 32,000, 1 to 64 rows 13.4 / 15.3, 40,000 14.5 / 15.4, 48,000 16 / 15.2, 151,936, 8 rows 35 / 15.3; fp32, 32,000 13.2 / 15.3,
//     40,000 14.2 / 15.4, 48,000 15.6 / 15.3, 56,000 17 / 15.3).
//   - More rows of 12,288 slots and more: the row pairs under way do not fit the L2s, and the second read is one from memory
//     (bf16, V = 112,000, 96 to 2047 rows 0.82 to 0.95 of the time, 256 rows 46.1 / 46.4; V = 151,936, 2048 rows 438 / 374; fp32, 64,000,
//     512 rows 0.81, 2048 rows 360 / 290; at 12,000 slots bf16, 256 rows 40.5 / 42.5).
//   - Shorter ones: over many rows, where a member's LDS is well filled (parts of 1600 slots, or half a row; bf16,
//     2048 rows, V = 20,000 73 / 68, 32,000 98 / 88, 56,000 157 / 147, 64,000 183 / 165, but parts of 1250 and 1500 V = 40,000 110 / 125, 48,000
//     129 / 137, 80,000 219 / 242; 2047 rows are not worth it; fp32, 1500 rows, V = 16,000 0.95, 28,000 0.96, 32,000 0.92, but
//     20,000 75 / 84, 24,000 89 / 93; 1024 rows, 11,200 35.7 / 37.0).
int kd_team(int32_t rows, int32_t V, bool bf16) {
    const int64_t slots = V / (bf16 ? 8 : 4);
    int team = 1;
    while (team <= kKdMaxTeam && (slots + team - 1) / team > kKdMaxChunks * kKdChunk) team *= 2;
    if (team == 1) return 1;
    if (team > kKdMaxTeam) return 0;
    const bool few = rows <= 64 && V >= 48000;
    if (!few && slots < 12288 && (rows < (bf16 ? 2048 : 1500) || (team > 2 && slots < 1600 * team))) return 0;
    while (team < kKdMaxTeam && (int64_t)rows * team * 2 <= kKdFill && slots / (2 * team) >= kThreads) team *= 2;
    return team;
}

// Whether the bytes of two [rows, V] matrices have an address in common, as far as their ends tell.
bool ranges_meet(const void *a, int64_t ld_a, const void *b, int64_t ld_b, int32_t rows, int32_t V, size_t esz) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    const uintptr_t a1 = a0 + ((size_t)(rows - 1) * ld_a + V) * esz, b1 = b0 + ((size_t)(rows - 1) * ld_b + V) * esz;
    return a0 < b1 && b0 < a1;
}

size_t kd_kl_bytes(int32_t rows, int team) { return round_up((size_t)rows * team * sizeof(double), 256); }
size_t kd_box_bytes(int32_t rows, int team) { return team > 1 ? (size_t)rows * team * kKdBoxWords * 8 : 0; }
// What a call takes, the streaming form's share where no team does.
size_t kd_call_bytes(int32_t rows, int32_t V, bool bf16) {
    const int team = kd_team(rows, V, bf16);
    return kd_kl_bytes(rows, std::max(team, 1)) + round_up(kd_box_bytes(rows, team), 256);
}

template <bool BF16>
hipError_t launch_kd_team(KdParams &p, int cus, hipStream_t stream) {
    static bool configured[64] = {false};  // per device; benign race: the attribute is idempotent
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
    if (dev < 0 || !configured[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kd_team_kernel<BF16>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kKdMaxChunks * kKdChunk * 64);
        if (e != hipSuccess) return e;
        if (dev >= 0) configured[dev] = true;
    }
    const int slots = p.V / Elem<BF16>::EPV;
    p.part_slots = ((slots + p.team - 1) / p.team + 7) / 8 * 8;  // (whole 128-byte lines)
    const int pieces = (p.part_slots + kKdChunk - 1) / kKdChunk;
    long teams = knobs().get(&Knobs::kd_wgs, (long)cus) / p.team;
    if (teams > p.rows) teams = p.rows;
    if (teams < 1) teams = 1;
    p.spin = (int32_t)knobs().get(&Knobs::kd_spin, 5000);  // 50 us
    if (p.team > 1) {
        const size_t words = kd_box_bytes(p.rows, p.team) / 16;
        hipLaunchKernelGGL(kd_clear_kernel, dim3((unsigned)std::min<size_t>((words + 255) / 256, (size_t)cus)), dim3(256), 0, stream,
                           reinterpret_cast<u32x4 *>(p.box), words);
    }
    hipLaunchKernelGGL((kd_team_kernel<BF16>), dim3((unsigned)(teams * p.team)), dim3(kKdThreads), (size_t)pieces * kKdChunk * 64, stream, p);
    return hipGetLastError();
}

template <bool BF16>
hipError_t launch_kd(KdParams &p, hipStream_t stream) {
    int cus = 256, dev = 0;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    hipError_t err = hipSuccess;
    if (p.team > 0) {
        err = launch_kd_team<BF16>(p, cus, stream);
    } else {
        p.team = 1;
        long wgs = knobs().get(&Knobs::kd_wgs, (long)cus);  // tests and sweeps
        if (wgs > p.rows) wgs = p.rows;
        if (wgs < 1) wgs = 1;
        hipLaunchKernelGGL((kd_stream_kernel<BF16>), dim3((unsigned)wgs), dim3(kThreads), 0, stream, p);
    }
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kd_finish_kernel, dim3(1), dim3(1024), 0, stream, p);
    return hipGetLastError();
}

}  // namespace
}  // namespace respec

extern "C" {

size_t respec_kd_rows_workspace_bytes(int32_t rows, int32_t V, respec_dtype_t dt) {
    using namespace respec;
    if (rows <= 0 || V <= 0 || (dt != RESPEC_F32 && dt != RESPEC_BF16)) return 0;
    // Fewer rows may be shared by more work-groups and take more room: enough for any number up to these (from kKdFill rows on
    // teams are as small as they get, and the call with the most rows takes the most)
    size_t most = kd_call_bytes(rows, V, dt == RESPEC_BF16);
    for (int32_t r = std::min(rows, (int32_t)kKdFill); r >= 1; --r) most = std::max(most, kd_call_bytes(r, V, dt == RESPEC_BF16));
    return most;
}

respec_status_t respec_kd_rows(const void *target_logits, const void *draft_logits, const float *row_weight,
                               void *grad_draft_logits, float *row_loss, double *total_loss, int32_t rows,
                               int32_t V, int64_t ld_t, int64_t ld_d, int64_t ld_g, respec_dtype_t logits_dt,
                               void *workspace, size_t workspace_bytes, void *hip_stream) {
    using namespace respec;
    if (rows <= 0 || V <= 0)
        return fail(RESPEC_ERR_INVALID_ARG, "kd_rows: need rows > 0 and V > 0 (rows=%d V=%d)", rows, V);
    if (logits_dt != RESPEC_F32 && logits_dt != RESPEC_BF16)
        return fail(RESPEC_ERR_INVALID_ARG, "kd_rows: unknown logits dtype %d", (int)logits_dt);
    if (!target_logits || !draft_logits || !row_weight || !grad_draft_logits || !row_loss)
        return fail(RESPEC_ERR_INVALID_ARG, "kd_rows: null pointer argument");
    if (ld_t < V || ld_d < V || ld_g < V)
        return fail(RESPEC_ERR_INVALID_ARG, "kd_rows: row stride smaller than V");
    const size_t esz = logits_dt == RESPEC_BF16 ? 2 : 4;
    if ((V * esz) % 16 != 0 || (ld_t * esz) % 16 != 0 || (ld_d * esz) % 16 != 0 || (ld_g * esz) % 16 != 0 ||
        !aligned_to(target_logits, 16) || !aligned_to(draft_logits, 16) || !aligned_to(grad_draft_logits, 16))
        return fail(RESPEC_ERR_UNSUPPORTED, "kd_rows: rows must be whole 16-byte pieces (V, strides and base pointers)");
    const size_t need = kd_kl_bytes(rows, 1);  // (less than the size function asks for: one work-group per row pair)
    if (!workspace || workspace_bytes < need || !aligned_to(workspace, 256))
        return fail(RESPEC_ERR_WORKSPACE, "kd_rows: workspace of %zu bytes (256-byte aligned) needed, got %zu", need,
                    workspace ? workspace_bytes : (size_t)0);

    KdParams p{};
    set_row_math(p, 1.0f);
    p.target = target_logits;
    p.draft = draft_logits;
    p.weight = row_weight;
    p.grad = grad_draft_logits;
    p.row_loss = row_loss;
    p.total_loss = total_loss;
    p.row_kl = static_cast<double *>(workspace);
    p.team = kd_team(rows, V, logits_dt == RESPEC_BF16);
    if (knobs().get(&Knobs::kd_team, 1) == 0 || workspace_bytes < kd_call_bytes(rows, V, logits_dt == RESPEC_BF16)) p.team = 0;
    // A gradient written over one of its inputs: a member computes an absent one's part from the rows, which
    // that one may overwrite by then.  (One work-group per row pair reads what it writes over before.)
    if (p.team > 1 && (ranges_meet(grad_draft_logits, ld_g, target_logits, ld_t, rows, V, esz) ||
                       ranges_meet(grad_draft_logits, ld_g, draft_logits, ld_d, rows, V, esz)))
        p.team = 0;
    p.box = reinterpret_cast<uint64_t *>(static_cast<char *>(workspace) + kd_kl_bytes(rows, std::max((int)p.team, 1)));
    p.rows = rows;
    p.V = V;
    p.ld_t = ld_t;
    p.ld_d = ld_d;
    p.ld_g = ld_g;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    hipError_t err;
    err = logits_dt == RESPEC_BF16 ? launch_kd<true>(p, stream) : launch_kd<false>(p, stream);
    if (err != hipSuccess)
        return fail(RESPEC_ERR_HIP, "kd_rows: launch failed: %s", hipGetErrorString(err));
    clear_error();
    return RESPEC_OK;
}

}  // extern "C"
