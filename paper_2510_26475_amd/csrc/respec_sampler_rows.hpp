// Row-streaming primitives shared by the rejection samplers (chain and tree of drafts) for
// gfx950: 16-byte slot loads, the fast and the guarded softmax-normaliser passes over one
// row (or a target/drafter row pair), wave and block reductions.  Everything that decides a
// token is carried in fp64; only exp2 of a single element runs in fp32.
#pragma once

#include "respec_common.hpp"

#include <cmath>
#include <type_traits>

namespace respec {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kUnroll = 4;
// Register sets of the streaming loops (one is summed while the others' loads are in flight).
// Two is the measured optimum: a work-group's pass is bound by the issue of its arithmetic (a
// sequence alone on the device is as fast on rows flushed from the caches as on rows in L2), so
// one batch in flight covers the latency and further sets only cost registers (headline
// workload: 103 us with two sets, 109 us with three, 135 us with four).
constexpr int kSetsTwoRows = 2;  // fast normaliser pass over a row pair
constexpr int kSetsOneRow = 2;   // ... over one row
constexpr int kSetsDraw = 2;     // the final draw's pass over the row pair
constexpr int kChunk = 5;   // slots of a thread's run in the inverse-CDF walk that are loaded together
constexpr float kRefInit = -1.0e30f;
constexpr double kBoundaryEps = 1e-6;
constexpr int kShortSlots = 512;      // rows up to this many slots: a wave takes a row pair, eight positions at a time
constexpr int kMaxSplit = 8;          // work-groups that can share one sequence
constexpr int kBoxHeaderBytes = 128;                      // epoch at word 0
constexpr int kBoxPayload = kMaxSplit * 2 * 16;           // [part][stage parity][8 doubles as 16 tagged words]
constexpr size_t kBoxBytes = kBoxHeaderBytes + (size_t)kBoxPayload * 8;
constexpr int kSpinLimit = 1 << 22;
constexpr uint32_t kBoxPoison = 0xffffffffu;             // epoch word of a box whose call failed
constexpr size_t kTableMaxBytes = 96 * 1024;  // LDS a launch may add for the final draw's slot totals

// The exponent constants of one call: exp((z - ref)/T) is taken as exp2((z - ref) * log2(e)/T).
struct RowMath {
    float c_f;         // log2(e)/T rounded to nearest binary32
    int one_term;      // c_f is close enough to log2(e)/T for the one-fma exponent of the fast pass
    float c_hi, c_lo;  // log2(e)/T = c_hi + c_lo, c_lo > 0
    double c_d;        // log2(e)/T
    double inv_T;
    float gap;         // logit distance above the reference that forces a re-reference
};

inline void set_row_math(RowMath &m, float temperature, bool force_two_term = false) {
    const double T = (double)temperature;
    m.c_d = 1.4426950408889634074 / T;
    float c_hi = (float)m.c_d;
    if ((double)c_hi >= m.c_d) c_hi = std::nextafterf(c_hi, 0.f);  // keep the low term positive
    m.c_hi = c_hi;
    m.c_lo = (float)(m.c_d - (double)c_hi);
    m.c_f = (float)m.c_d;
    m.one_term = std::fabs((double)m.c_f / m.c_d - 1.0) <= 2.0e-8 ? 1 : 0;
    if (force_two_term) m.one_term = 0;
    m.inv_T = 1.0 / T;
    m.gap = (float)(40.0 / m.c_d);
}

template <bool BF16>
struct Elem {
    static constexpr int EPV = BF16 ? 8 : 4;  // elements per 16-byte slot
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline float as_f32(uint32_t u) { return __uint_as_float(u); }

template <bool BF16>
__device__ inline void unpack(const u32x4 &v, float (&z)[Elem<BF16>::EPV]) {
    if constexpr (BF16) {
        z[0] = as_f32(v[0] << 16);
        z[1] = as_f32(v[0] & 0xffff0000u);
        z[2] = as_f32(v[1] << 16);
        z[3] = as_f32(v[1] & 0xffff0000u);
        z[4] = as_f32(v[2] << 16);
        z[5] = as_f32(v[2] & 0xffff0000u);
        z[6] = as_f32(v[3] << 16);
        z[7] = as_f32(v[3] & 0xffff0000u);
    } else {
        z[0] = as_f32(v[0]);
        z[1] = as_f32(v[1]);
        z[2] = as_f32(v[2]);
        z[3] = as_f32(v[3]);
    }
}

// A slot filled with -inf: inert in every sum and never chosen.
template <bool BF16>
__device__ inline u32x4 neg_inf_slot() {
    const uint32_t w = BF16 ? 0xff80ff80u : 0xff800000u;
    return u32x4{w, w, w, w};
}

// 16 bytes of row `row` starting at element slot*EPV; elements at or beyond V read as -inf.
// FULL: the slot lies inside the row (the caller takes a row's last, partial slot separately).
// Rows start wherever their element type may (an odd vocabulary leaves them 2 or 4 bytes aligned):
// the 16-byte loads of this device take any address, a wave's 1 KiB then touches one cache line more.
// (Element loads for such rows took 2 to 8 times the instructions: B = 32, k = 2, fp32, V = 50,257
// 43.5 -> 26.8 us per call.)
// LAST_USE: the pass that reads the row for the last time marks its loads non-temporal, which
// leaves the caches to rows that are still to be read again (3 % of the sampler's time, 6 % of
// the distillation kernel's; the same hint on a row's first read costs 5 %: the second read
// then misses).  ALIGNED: the row is known to start on 16 bytes.
template <bool BF16, bool FULL = false, bool LAST_USE = false, bool ALIGNED = false>
__device__ inline u32x4 load_slot(const void *row, int slot, int V) {
    constexpr int EPV = Elem<BF16>::EPV;
    typedef u32x4 u32x4_elem __attribute__((aligned(2)));
    typedef std::conditional_t<ALIGNED, u32x4, u32x4_elem> Slot;
    // (a 32-bit unsigned byte offset from the row's uniform base: the load then takes a scalar
    // base and one offset register instead of a 64-bit address pair formed per load; rows are
    // shorter than 4 GiB, checked on the host)
    const Slot *whole = reinterpret_cast<const Slot *>(static_cast<const char *>(row) + ((uint32_t)slot * 16u));
    if constexpr (FULL) return LAST_USE ? __builtin_nontemporal_load(whole) : *whole;
    const int e0 = slot * EPV;
    if (e0 + EPV <= V) return LAST_USE ? __builtin_nontemporal_load(whole) : *whole;
    uint32_t w[4];
    if constexpr (BF16) {
        const uint16_t *r = static_cast<const uint16_t *>(row);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t lo = (e0 + 2 * j < V) ? r[e0 + 2 * j] : 0xff80u;
            const uint32_t hi = (e0 + 2 * j + 1 < V) ? r[e0 + 2 * j + 1] : 0xff80u;
            w[j] = lo | (hi << 16);
        }
    } else {
        const uint32_t *r = static_cast<const uint32_t *>(row);
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = (e0 + j < V) ? r[e0 + j] : 0xff800000u;
    }
    return u32x4{w[0], w[1], w[2], w[3]};
}

template <bool BF16>
__device__ inline float logit_at(const char *row, int x) {
    if constexpr (BF16)
        return as_f32((uint32_t) reinterpret_cast<const uint16_t *>(row)[x] << 16);
    else
        return reinterpret_cast<const float *>(row)[x];
}

// The partial slot behind `whole` whole ones from the row's last 16 bytes (what it is loaded as: the
// same kind of load as every other slot's, so that a batch of loads needs no condition): its
// elements moved to the front, -inf behind them.
template <bool BF16>
__device__ inline u32x4 partial_slot(const u32x4 &last, int whole, int Vrow) {
    const uint32_t fill = neg_inf_slot<BF16>()[0];
    const int bytes = (Elem<BF16>::EPV - (Vrow - whole * Elem<BF16>::EPV)) * (BF16 ? 2 : 4);  // to drop
    uint32_t w[5];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        w[j] = fill;
#pragma unroll
        for (int i = j; i < 4; ++i) w[j] = j + bytes / 4 == i ? last[i] : w[j];
    }
    w[4] = fill;
    u32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (bytes & 2) ? (w[j] >> 16) | (w[j + 1] << 16) : w[j];
    return v;
}

// 16 bytes of slot `slot` of a row with Vrow elements (at least one slot's worth), the row's last 16
// bytes for its partial slot.
template <bool BF16>
__device__ inline u32x4 load_slot_or_last(const void *row, int slot, int Vrow) {
    typedef u32x4 u32x4_elem __attribute__((aligned(2)));
    const uint32_t off = min((uint32_t)slot * 16u, (uint32_t)Vrow * (BF16 ? 2u : 4u) - 16u);
    return *reinterpret_cast<const u32x4_elem *>(static_cast<const char *>(row) + off);
}

// The partial slot itself.
template <bool BF16>
__device__ inline u32x4 load_partial_slot(const void *row, int whole, int Vrow) {
    return partial_slot<BF16>(load_slot_or_last<BF16>(row, whole, Vrow), whole, Vrow);
}

// Of nslots slots from the start of a row (or of a part of one) with Vrow elements to the row's end,
// those that lie inside the row; one more, the partial one, follows when this is nslots - 1.
template <bool BF16>
__device__ inline int whole_slots(int nslots, int Vrow) {
    return min(nslots, Vrow / Elem<BF16>::EPV);
}

__device__ inline float hw_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// fp64 exp2 is only needed a few times per row (reconciling references).
__device__ inline double exp2_f64(double x) { return exp2(x); }

// exp2 argument of one element: (z - ref) * (c_hi + c_lo).  c_lo > 0 keeps -inf at -inf.
__device__ inline float exp2_arg(float z, float ref, float c_hi, float c_lo) {
    const float d = z - ref;
    return fmaf(d, c_hi, d * c_lo);
}

// Running sum of exp((z-ref)/T) of one thread: fp32 lanes per slot position, fp64 carry.
template <bool BF16>
struct ThreadSum {
    float ref = kRefInit;
    double carry = 0.0;
    float acc[Elem<BF16>::EPV];

    __device__ inline void init() {
#pragma unroll
        for (int j = 0; j < Elem<BF16>::EPV; ++j) acc[j] = 0.f;
    }

    __device__ inline void absorb(const u32x4 &v, const RowMath &p) {
        constexpr int EPV = Elem<BF16>::EPV;
        float z[EPV];
        unpack<BF16>(v, z);
        float vmax = z[0];
#pragma unroll
        for (int j = 1; j < EPV; ++j) vmax = fmaxf(vmax, z[j]);
        if (vmax - ref > p.gap) {  // first finite slot, or an element far above the reference
            double s = carry;
#pragma unroll
            for (int j = 0; j < EPV; ++j) {
                s += (double)acc[j];
                acc[j] = 0.f;
            }
            carry = s * exp2_f64((double)(ref - vmax) * p.c_d);
            ref = vmax;
        }
#pragma unroll
        for (int j = 0; j < EPV; ++j) acc[j] += hw_exp2(exp2_arg(z[j], ref, p.c_hi, p.c_lo));
    }

    __device__ inline double total() const {
        double s = carry;
#pragma unroll
        for (int j = 0; j < Elem<BF16>::EPV; ++j) s += (double)acc[j];
        return s;
    }
};

// Sums, maxima and prefix sums over a wave by lane-permuting adds (DPP): no LDS round trip per step,
// as the shuffles have (six of them in a row, two words each, took 0.3 us of every pass).  All 64
// lanes have to be active.  Lanes a row shift reads from outside its sixteen count as zero.
template <int CTRL>
__device__ inline double dpp_add(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return x + __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

__device__ inline double lane_value(double x, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane), hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}

__device__ inline float lane_value(float x, int lane) {
    return as_f32((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane));
}

template <int CTRL>
__device__ inline float dpp_max(float x) {
    return fmaxf(x, as_f32(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true)));
}

// (control words of the permutations)
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;              // lane ^ 1, lane ^ 2
constexpr int kDppOtherQuad = 0x141, kDppOtherEight = 0x140; // the other quad of eight lanes, the other eight of sixteen
constexpr int kDppShr1 = 0x111, kDppShr2 = 0x112, kDppShr4 = 0x114, kDppShr8 = 0x118;  // lane - 1, ... of sixteen

__device__ inline float wave_max(float x) {
    x = dpp_max<kDppOtherEight>(dpp_max<kDppOtherQuad>(dpp_max<kDppXor2>(dpp_max<kDppXor1>(x))));
    return fmaxf(fmaxf(lane_value(x, 0), lane_value(x, 16)), fmaxf(lane_value(x, 32), lane_value(x, 48)));
}

__device__ inline double wave_sum(double x) {
    x = dpp_add<kDppOtherEight>(dpp_add<kDppOtherQuad>(dpp_add<kDppXor2>(dpp_add<kDppXor1>(x))));
    return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

__device__ inline double wave_inclusive_scan(double x, int lane) {
    x = dpp_add<kDppShr8>(dpp_add<kDppShr4>(dpp_add<kDppShr2>(dpp_add<kDppShr1>(x))));
    const double s1 = lane_value(x, 15), s2 = s1 + lane_value(x, 31), s3 = s2 + lane_value(x, 47);
    const double before = lane < 32 ? (lane < 16 ? 0.0 : s1) : (lane < 48 ? s2 : s3);
    return before + x;
}

// The block-wide "first thread for which `hit` holds" and "largest `last` (a value that grows
// with the thread index, -1 = none)" of the draw's walk, left in sh_first / sh_last (preset to
// kThreads / -1): one ballot per wave and one LDS atomic per wave.  (An atomic from every thread
// on one LDS word is served one lane at a time: 512 of them took 4 us of every draw.)
__device__ inline void note_first_and_last(bool hit, int last, int *sh_first, int *sh_last) {
    const int lane = threadIdx.x & 63;
    const unsigned long long hits = __ballot(hit), have = __ballot(last >= 0);
    if (hits != 0ull && lane == 0) atomicMin(sh_first, (int)(threadIdx.x & ~63u) + __builtin_ctzll(hits));
    if (have != 0ull) {
        const int top = 63 - __builtin_clzll(have);  // wave-uniform: the values grow with the lane
        const int v = __builtin_amdgcn_readlane(last, top);
        if (lane == 0) atomicMax(sh_last, v);
    }
}

// The thread's index (or lane) as a value the compiler cannot trace back to threadIdx: per-lane
// offsets formed from it are formed in the pass that uses them instead of being kept in
// registers across every pass of a long kernel (which cost the tree sampler and the general
// forms of the chain sampler up to 60 spilled registers).
__device__ inline int opaque_thread_index() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

struct SharedState {
    float m[2][2][kWaves];   // [parity][row p/q][wave]
    double s[2][2][kWaves];
    double wave_total[kWaves];
    double scan_total[kWaves];
    double xchg[kMaxSplit][8];             // what the parts published in the current stage
    int failed;                            // a bounded wait for a partner ran out
    float part_ref[kMaxSplit];             // references and scales of the parts of a draw
    double part_scale[kMaxSplit];
    float arg_val[kWaves];                 // per-wave (largest logit, its first token) of an argmax pass
    int arg_idx[kWaves];
    float pos_m[2][kWaves];                // short rows: [p/q][position] references and sums, ...
    double pos_s[2][kWaves];
    double pos_rho[kWaves], pos_u[kWaves]; // ... acceptance ratios, uniforms and tokens of eight positions
    int pos_x[kWaves];
    int token;
    int near_edge;
    int last_positive;
    int first_thread;
};

// Maximum and sum over groups of N neighbouring lanes (N = waves of a block); every lane of a group gets
// the same bits.
template <int N>
__device__ inline float group_max(float x) {
    static_assert(N == 4 || N == 8);
    x = dpp_max<kDppXor2>(dpp_max<kDppXor1>(x));
    return N == 8 ? dpp_max<kDppOtherQuad>(x) : x;
}

template <int N>
__device__ inline double group_sum(double x) {
    static_assert(N == 4 || N == 8);
    x = dpp_add<kDppXor2>(dpp_add<kDppXor1>(x));
    if constexpr (N == 8) x = dpp_add<kDppOtherQuad>(x);
    return x;
}

// Combine the per-thread (ref, sum) pairs of the block into one (M, S) with
// S = sum_x exp((z_x - M)/T).  Every thread returns the same bits.
template <int TH = kThreads>
__device__ inline void block_combine(float ref, double sum, SharedState &sh, int parity, int which,
                                     const RowMath &p, float &M, double &S) {
    constexpr int kWaves = TH / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float mw = wave_max(ref);
    const double sw = wave_sum(sum * exp2_f64((double)(ref - mw) * p.c_d));
    if (lane == 0) {
        sh.m[parity][which][wave] = mw;
        sh.s[parity][which][wave] = sw;
    }
    __syncthreads();
    const int w = lane & (kWaves - 1);
    const float my_m = sh.m[parity][which][w];
    const float mm = group_max<kWaves>(my_m);
    M = mm;
    S = group_sum<kWaves>(sh.s[parity][which][w] * exp2_f64((double)(my_m - mm) * p.c_d));
}

// The same for the fast pass, both rows at once.  The threads of a wave share one reference
// there (the pass sets it per wave), so a wave's sums add up as they are; sixteen lanes then
// reconcile the eight (reference, sum) pairs of each row behind a single barrier, with one fp64
// exp2 each.  ONE_TERM: the sums were taken as exp2(z c_f + K) with K = -ref c_f rounded; the
// residue K + ref c_f is undone in the same exp2.  Every thread returns the same bits.
template <bool TWO, bool ONE_TERM, int TH = kThreads>
__device__ inline void block_combine_fast(float refp, double sp, float refq, double sq, SharedState &sh, int parity,
                                          const RowMath &p, float &Mp, double &Sp, float &Mq, double &Sq) {
    constexpr int kWaves = TH / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double swp = wave_sum(sp);
    const double swq = TWO ? wave_sum(sq) : 0.0;
    if (lane == 0) {
        sh.m[parity][0][wave] = refp;
        sh.s[parity][0][wave] = swp;
        if constexpr (TWO) {
            sh.m[parity][1][wave] = refq;
            sh.s[parity][1][wave] = swq;
        }
    }
    __syncthreads();
    const int w = lane & (kWaves - 1), r = TWO ? (lane / kWaves) & 1 : 0;  // (the second group of lanes: the q row)
    const float my_m = sh.m[parity][r][w];
    const float mm = group_max<kWaves>(my_m);
    double e = (double)(my_m - mm) * p.c_d;
    if constexpr (ONE_TERM) e -= (double)(-my_m * p.c_f) + (double)my_m * (double)p.c_f;
    const double part = group_sum<kWaves>(sh.s[parity][r][w] * exp2_f64(e));
    Mp = lane_value(mm, 0);
    Sp = lane_value(part, 0);
    if constexpr (TWO) {
        Mq = lane_value(mm, kWaves);
        Sq = lane_value(part, kWaves);
    }
}

// One thread's share of the fast pass: 8 (bf16) or 4 (f32) running sums of
// exp2(z*c + K) = exp((z - ref)/T), no branches.  ONE_TERM: c = c_f, K = -ref*c_f rounded (the
// rounding residue is put back in fp64 when threads are combined).
template <bool BF16, bool ONE_TERM>
__device__ inline void fast_absorb(const u32x4 &v, float (&acc)[Elem<BF16>::EPV], float ref, float K,
                                   const RowMath &p) {
    constexpr int EPV = Elem<BF16>::EPV;
    float z[EPV];
    unpack<BF16>(v, z);
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
        const float t = ONE_TERM ? fmaf(z[j], p.c_f, K) : exp2_arg(z[j], ref, p.c_hi, p.c_lo);
        acc[j] += hw_exp2(t);
    }
}

template <bool BF16>
__device__ inline float slot_max(const u32x4 &v) {
    constexpr int EPV = Elem<BF16>::EPV;
    float z[EPV];
    unpack<BF16>(v, z);
    float m = z[0];
#pragma unroll
    for (int j = 1; j < EPV; ++j) m = fmaxf(m, z[j]);
    return m;
}

// The largest logit among the first kThreads x PER of a row's nslots whole slots; every
// thread returns the same value (-inf when none of them is finite).  Ends with a barrier.
template <bool BF16, bool ALIGNED, int PER, int TH = kThreads>
__device__ inline float block_max_of_row_start(const void *row, int nslots, SharedState &sh) {
    constexpr int kThreads = TH, kWaves = TH / 64;
    const int lane = opaque_thread_index() & 63, wave = threadIdx.x >> 6;
    float m = -INFINITY;
    if ((int)threadIdx.x < nslots) {
        u32x4 v[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u)  // (slots past the row's end: its last one again)
            v[u] = load_slot<BF16, true, false, ALIGNED>(row, min((int)threadIdx.x + u * kThreads, nslots - 1), 0);
#pragma unroll
        for (int u = 0; u < PER; ++u) m = fmaxf(m, slot_max<BF16>(v[u]));
    }
    m = wave_max(m);
    __syncthreads();  // (earlier readers of arg_val are done)
    if (lane == 0) sh.arg_val[wave] = m;
    __syncthreads();
    float r = sh.arg_val[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) r = fmaxf(r, sh.arg_val[w]);
    __syncthreads();
    return r;
}

// The guarded pass moves a reference once an element lies 40 binary orders above it (RowMath::gap). The
// fast passes over rows that are not whole aligned slots leave to it what it would have handled that
// way: a thread's or a region's sum above this counts as an overflow.  (Without the bound elements up
// to 127 orders above their reference were summed, with exponents rounded to 2^-18 instead of 2^-20.)
constexpr double kFastMost = 0x1p40;

// A wave whose first slots hold no finite logit sums against 0: what lies below 2^-126 there is lost, at most 2^-108 of a
// row.  The row's reference is then at least 0, so a sum above this bound cannot miss it; one below is left to
// the guarded pass.  (Sums against references that are logits of the row are 1 and more.)
constexpr double kFastLeast = 0x1p-72;

// Slots per thread that the one-pass draws take their reference from.  A binary32 exponent is exact to
// 2^-24 of its own size, so a weight loses accuracy with its distance from the reference.  The forms
// with fp64 weights look as far into the row as the normaliser pass (whose reference they would
// otherwise have) does; the fp32 forms, whose weights carry a few 1e-7 in any case, at one slot.
template <bool ONE_TERM>
constexpr int kRefSlots = ONE_TERM ? 1 : kUnroll;

// Fast streaming pass over a target row (and, if TWO, the matching drafter row).  The
// reference of a wave is the maximum of the first slots it reads, not the row maximum:
// exp2 keeps full relative precision for any offset, only a logit more than ~88/c above the
// reference would overflow.  Returns false (every thread alike) when a sum came out
// non-finite, empty or next to empty, and the caller then repeats the row with the guarded pass below.
// PARTIAL: the row need not be aligned nor hold whole slots only (it has at least one); an
// instantiation of its own, since what it adds cost whole rows 1-2 %.  `meanwhile` is called once the
// first batch has been requested.
struct Nothing {
    __device__ inline void operator()() const {}
};

template <bool BF16, bool TWO, bool ONE_TERM, bool PARTIAL = false, int TH = kThreads, class Meanwhile = Nothing>
__device__ inline bool row_stats_fast(const void *rowp, const void *rowq, int nslots_all, int Vrow,
                                      SharedState &sh, int parity, const RowMath &p, float &Mp,
                                      double &Sp, float &Mq, double &Sq, Meanwhile &&meanwhile = Nothing{}) {
    constexpr int EPV = Elem<BF16>::EPV;
    const int nslots = PARTIAL ? whole_slots<BF16>(nslots_all, Vrow) : nslots_all;
    constexpr int kThreads = TH;
    constexpr int kBatch = kThreads * kUnroll;  // slots per block iteration
    const int tid = opaque_thread_index();
    float accp[EPV], accq[EPV];
#pragma unroll
    for (int j = 0; j < EPV; ++j) accp[j] = accq[j] = 0.f;
    float refp = 0.f, refq = 0.f, Kp = 0.f, Kq = 0.f;
    const int n_iter = (nslots + kBatch - 1) / kBatch;  // block-uniform, >= 1
    // batch `it` of this thread: slots it*kBatch + tid + u*kThreads; only the last batch can
    // run past the row.  Its loads are clamped to the row and all issued together; the slots
    // past the row are replaced by -inf when the batch is consumed (mask_last), not here: a
    // select right behind each load makes the loads wait for one another.
    auto load_batch = [&](int it, u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
        const int s0 = it * kBatch + tid;
        if (it + 1 < n_iter) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                vp[u] = load_slot<BF16, true, false, !PARTIAL>(rowp, s0 + u * kThreads, Vrow);
                if constexpr (TWO) vq[u] = load_slot<BF16, true, false, !PARTIAL>(rowq, s0 + u * kThreads, Vrow);
            }
        } else {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int safe = max(0, min(s0 + u * kThreads, nslots - 1));
                vp[u] = load_slot<BF16, true, false, !PARTIAL>(rowp, safe, Vrow);
                if constexpr (TWO) vq[u] = load_slot<BF16, true, false, !PARTIAL>(rowq, safe, Vrow);
            }
        }
    };
    auto mask_last = [&](u32x4 (&vp)[kUnroll], u32x4 (&vq)[kUnroll]) __attribute__((always_inline)) {
        const int s0 = (n_iter - 1) * kBatch + tid;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const bool in = s0 + u * kThreads < nslots;
            vp[u] = in ? vp[u] : neg_inf_slot<BF16>();
            if constexpr (TWO) vq[u] = in ? vq[u] : neg_inf_slot<BF16>();
        }
    };
    // A ring of NSETS register sets: NSETS - 1 batches are in flight while one is summed.  The
    // loads of the steady state are unconditional: a load behind a condition makes
    // the compiler's wait for the batch in front of it a wait for everything in flight (it must
    // assume the branch was not taken), and then no load overlaps any sum.  Batches past the
    // row's end read its last slot again and are never summed.
    constexpr int NSETS = TWO ? kSetsTwoRows : kSetsOneRow;
    u32x4 rp[NSETS][kUnroll], rq[NSETS][kUnroll];
#pragma unroll
    for (int s = 0; s + 1 < NSETS; ++s) load_batch(s, rp[s], rq[s]);
    meanwhile();
    if (n_iter == 1) mask_last(rp[0], rq[0]);  // block-uniform
    {   // references from the first batch
        float mp = slot_max<BF16>(rp[0][0]), mq = -INFINITY;
#pragma unroll
        for (int u = 1; u < kUnroll; ++u) mp = fmaxf(mp, slot_max<BF16>(rp[0][u]));
        mp = wave_max(mp);
        refp = (mp > -INFINITY && mp < INFINITY) ? mp : 0.f;
        Kp = -refp * p.c_f;
        if constexpr (TWO) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) mq = fmaxf(mq, slot_max<BF16>(rq[0][u]));
            mq = wave_max(mq);
            refq = (mq > -INFINITY && mq < INFINITY) ? mq : 0.f;
            Kq = -refq * p.c_f;
        }
    }
    // (live: of the batch's kUnroll groups of slots, those with a slot inside the row; block-uniform.  The first two are
    // summed in any case: a branch ahead of each cost rows of few batches more than it saved, bf16, V = 32,000, B = 65, k = 3 22.9 / 24.6 us)
    auto absorb_batch = [&](const u32x4 (&xp)[kUnroll], const u32x4 (&xq)[kUnroll], int live) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (u >= kUnroll / 2 && u >= live) break;
            fast_absorb<BF16, ONE_TERM>(xp[u], accp, refp, Kp, p);
            if constexpr (TWO) fast_absorb<BF16, ONE_TERM>(xq[u], accq, refq, Kq, p);
        }
    };
    int it = 0;  // set s holds batch it + s for s < NSETS - 1; every condition below is block-uniform
    for (; it + NSETS < n_iter; it += NSETS) {
#pragma unroll
        for (int s = 0; s < NSETS; ++s) {
            constexpr int kAhead = NSETS - 1;
            load_batch(it + s + kAhead, rp[(s + kAhead) % NSETS], rq[(s + kAhead) % NSETS]);
            absorb_batch(rp[s], rq[s], kUnroll);
        }
    }
    // the last 1..NSETS batches
    const int rem = n_iter - it;
    if (rem == NSETS) load_batch(it + NSETS - 1, rp[NSETS - 1], rq[NSETS - 1]);
#pragma unroll
    for (int s = 0; s < NSETS; ++s) {
        if (s < rem) {
            if (s == rem - 1) {
                mask_last(rp[s], rq[s]);  // (a second time when the row has one batch: harmless)
                absorb_batch(rp[s], rq[s], (nslots - (n_iter - 1) * kBatch + kThreads - 1) / kThreads);
            } else {
                absorb_batch(rp[s], rq[s], kUnroll);
            }
        }
    }
    if (PARTIAL && nslots < nslots_all && tid == 0) {  // the row's partial slot
        fast_absorb<BF16, ONE_TERM>(load_partial_slot<BF16>(rowp, nslots, Vrow), accp, refp, Kp, p);
        if constexpr (TWO) fast_absorb<BF16, ONE_TERM>(load_partial_slot<BF16>(rowq, nslots, Vrow), accq, refq, Kq, p);
    }
    double sp = 0.0, sq = 0.0;
#pragma unroll
    for (int j = 0; j < EPV; ++j) {
        sp += (double)accp[j];
        sq += (double)accq[j];
    }
    if constexpr (PARTIAL) {
        if (sp > kFastMost) sp = (double)INFINITY;
        if (TWO && sq > kFastMost) sq = (double)INFINITY;
    }
    // (ONE_TERM: exp2(z c + K) = exp2((z - ref) c) * exp2(K + ref c); the combine undoes the residue)
    block_combine_fast<TWO, ONE_TERM, TH>(refp, sp, refq, sq, sh, parity, p, Mp, Sp, Mq, Sq);
    bool ok = Sp > kFastLeast && Sp < 1.0e300;
    if constexpr (TWO) ok = ok && Sq > kFastLeast && Sq < 1.0e300;
    return ok;
}

// Guarded streaming pass (any finite or -inf logits): per-thread references that follow the
// running maximum.  Used when the fast pass reports an overflow or an empty sum.
template <bool BF16, bool TWO, int TH = kThreads>
__device__ inline void row_stats(const void *rowp, const void *rowq, int nslots, int Vrow, SharedState &sh,
                                 int parity, const RowMath &p, float &Mp, double &Sp,
                                 float &Mq, double &Sq) {
    constexpr int kThreads = TH;
    ThreadSum<BF16> tp, tq;
    tp.init();
    tq.init();
    for (int s0 = opaque_thread_index(); s0 < nslots; s0 += kThreads * kUnroll) {
        u32x4 vp[kUnroll], vq[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int slot = s0 + u * kThreads;
            vp[u] = slot < nslots ? load_slot<BF16>(rowp, slot, Vrow) : neg_inf_slot<BF16>();
            if constexpr (TWO)
                vq[u] = slot < nslots ? load_slot<BF16>(rowq, slot, Vrow)
                                      : neg_inf_slot<BF16>();
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            tp.absorb(vp[u], p);
            if constexpr (TWO) tq.absorb(vq[u], p);
        }
    }
    block_combine<TH>(tp.ref, tp.total(), sh, parity, 0, p, Mp, Sp);
    if constexpr (TWO) block_combine<TH>(tq.ref, tq.total(), sh, parity, 1, p, Mq, Sq);
}

// (M, S) of a short row pair in one wave: a reference and S = sum_x exp((z_x - M)/T) for each row; an
// empty row gives (kRefInit, 0), as the guarded pass does.  The rows (at least one whole slot, at most
// kShortSlots) are held in registers, all loads in flight together.  Every lane's reference is the
// largest of its own elements, every element is added in fp64: the sums are no less exact than the
// block's, which has at most two of such a row's elements per binary32 accumulator (rms error at V =
// 512 to 4096, fp32, T = 0.4 to 1.3, exp2 taken as exact: 5e-10 to 2e-9, the block's 3e-9 to 2e-8; with
// one reference and binary32 accumulators per lane up to 5e-8).
template <bool BF16>
__device__ inline void wave_row_pair_stats(const void *rowp, const void *rowq, int nslots, int Vrow, const RowMath &p,
                                           float (&M)[2], double (&S)[2]) {
    constexpr int EPV = Elem<BF16>::EPV;
    constexpr int kPer = kShortSlots / 64;
    const int lane = threadIdx.x & 63, whole = whole_slots<BF16>(nslots, Vrow);
    u32x4 v[2][kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {  // (the conditions on u and nslots are wave-uniform)
        if (u * 64 >= nslots) break;
        v[0][u] = load_slot_or_last<BF16>(rowp, lane + u * 64, Vrow);
        v[1][u] = load_slot_or_last<BF16>(rowq, lane + u * 64, Vrow);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        float m = -INFINITY;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (u * 64 >= nslots) break;
            const int slot = lane + u * 64;
            if (whole - u * 64 < 64) {  // the last slots of the row
                if (whole < nslots && slot == whole) v[r][u] = partial_slot<BF16>(v[r][u], whole, Vrow);
                if (slot >= nslots) v[r][u] = neg_inf_slot<BF16>();
            }
            m = fmaxf(m, slot_max<BF16>(v[r][u]));
        }
        const float ref = m > -INFINITY ? m : kRefInit;
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (u * 64 >= nslots) break;
            float z[EPV];
            unpack<BF16>(v[r][u], z);
#pragma unroll
            for (int j = 0; j < EPV; ++j) t += (double)hw_exp2(exp2_arg(z[j], ref, p.c_hi, p.c_lo));
        }
        M[r] = wave_max(ref);
        S[r] = wave_sum(t * exp2_f64((double)(ref - M[r]) * p.c_d));
    }
}

// fp32 form of a normalised probability, for calls whose exponent constant rounds well
// (RowMath::one_term): p(x) = exp2(z c_f + K) (1 + e), where K + log2(1 + e) = -M c_f - log2(S)
// is split so that the rounding of K is put back to first order through e.
struct FastNorm {
    float Kp, ep, Kq, eq;
    float e_rel;  // eq - ep: the q row's correction relative to the p row's
};

__device__ inline FastNorm make_fast_norm(float Mp, double Sp, float Mq, double Sq, const RowMath &p) {
    FastNorm f;
    const double kp = -(double)Mp * (double)p.c_f - log2(Sp);
    const double kq = -(double)Mq * (double)p.c_f - log2(Sq);
    f.Kp = (float)kp;
    f.Kq = (float)kq;
    f.ep = (float)((kp - (double)f.Kp) * 0.69314718055994530942);
    f.eq = (float)((kq - (double)f.Kq) * 0.69314718055994530942);
    f.e_rel = (float)(((kq - (double)f.Kq) - (kp - (double)f.Kp)) * 0.69314718055994530942);
    return f;
}

// Device-scope accesses for the few words that work-groups on different compute units (whose
// L2 caches are not coherent with each other) exchange.
__device__ inline uint32_t load_dev(const uint32_t *ptr) {
    return __hip_atomic_load(ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void store_dev(uint32_t *ptr, uint32_t v) {
    __hip_atomic_store(ptr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline double load_dev_f64(const double *ptr) {
    return __builtin_bit_cast(double, __hip_atomic_load(reinterpret_cast<const unsigned long long *>(ptr),
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

__device__ inline void store_dev_f64(double *ptr, double v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(ptr), __builtin_bit_cast(unsigned long long, v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace
}  // namespace respec
