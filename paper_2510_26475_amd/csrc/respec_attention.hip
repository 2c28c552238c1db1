// Verify attention for gfx950: the attention of the single target forward that scores the
// k drafted tokens plus one (Section 2.2, "Validation"; Figure 2).  (k_b+1) causal query
// rows per sequence, grouped-query heads, ragged token-major KV cache.
//
// bf16 path.  The G*(k_b+1) query rows that share one KV head are the columns of 16-wide
// MFMA tiles.  Work is cut into 32-key tiles of one (KV head, sequence); the tiles form flat
// lists ordered (head, sequence, tile) that are split evenly over a fixed number of ranges
// (two to four per compute unit), so every range streams the same number of bytes whatever the mix
// of sequence lengths.  One work-group per compute unit holds four producer waves, which walk a
// range ahead of its consumers and only move tiles (global memory -> registers -> a ring in LDS),
// and four or eight consumer waves, which compute.  Scores are computed
// transposed (S^T = K Q^T, v_mfma_f32_16x16x32_bf16) so that a lane's four accumulator rows
// are keys and its column is one query row: the probabilities then feed the second product
// (O^T = V^T P^T) straight from registers, and the softmax statistics of a row live in one
// lane column.  The contraction indices of both products are permuted freely (any order is
// valid as long as both operands agree), which is what lets K be read from LDS in 16-byte
// pieces and V with the transposing LDS reads of gfx950.
// A range is walked as segments (one sequence each).  A segment that covers a whole sequence
// writes the output; a sequence cut by a range border leaves partials (max, sum, unnormalised
// O as 16-bit fixed point), at most two per range, which a second kernel folds in a fixed
// order (deterministic, no float atomics).
//
// fp32 path.  A plain fp32 kernel (no MFMA, no split; the fp32 workload is the small parity
// case), one work-group per (sequence, query head, query row).
#include "respec_common.hpp"

#include <algorithm>
#include <cmath>
#include <mutex>

// Scratch of respec_verify_attention_static (the entry point for callers that cannot allocate):
// one copy per GPU, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the kernels get the device address that call returns.
constexpr size_t kStaticScratchBytes = (size_t)40 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace respec {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kTileKeys = 32;         // keys per wave tile
constexpr int kColTile = 16;          // query rows per MFMA column tile
constexpr int kMaxColsPerBlock = 64;  // 4 column tiles
constexpr float kRescaleSlack = 8.f;  // log2 units
constexpr float kNoMax = -3.402823466e38f;  // reference of a row that has seen no key (finite: -inf minus it is -inf)
constexpr int kProducers = 4;         // waves per work-group that move tiles (one per SIMD), beside four
                                      // or eight computing ones; one work-group per compute unit
constexpr int kSlots = 2;             // tiles in a producer's LDS ring = tiles it keeps in flight
constexpr int kMaxWaves = 2048;       // upper bound of the split width (sizes the workspace)

// Where a wave's range of the flat tile list starts and how many tiles it holds, with the
// bounds of its first sequence already resolved (one look-up instead of a chain of them before
// the first tile can be requested).
struct __align__(16) WaveStart {
    int32_t h, b, t, n;
    int32_t q0, R, L, tiles;
    int64_t kv0;
    int64_t pad;
};

struct AttnParams {
    const void *q;
    const void *k;
    const void *v;
    const int32_t *q_indptr;
    const int64_t *kv_indptr;
    const uint64_t *tree_mask;  // [total_q] or NULL (chain): bit j = the sequence's j-th new token is
                                // visible to the row (its ancestors in the draft tree and itself)
    // paged cache (page_table != NULL): k and v are [num_pages, page_size, Hkv, D], sequence b
    // owns the page ids page_table[page_indptr[b] .. page_indptr[b+1]) and holds kv_len[b] tokens
    const int32_t *page_table;
    const int32_t *page_indptr;
    const int32_t *kv_len;
    int32_t num_pages, table_len, page_size, page_shift;  // page_size = 1 << page_shift, >= 16
    void *out;
    float *lse;
    int16_t *ws_o;         // [2*W, Mpad, D]   unnormalised partial outputs, 16-bit fixed point
                           //                  relative to the row's largest magnitude
    float *ws_ml;          // [2*W, Mpad, 4]   (max in log2 units, sum, largest magnitude, -)
    int32_t *tile_prefix;  // [B+1] prefix sum of ceil(L_b / kTileKeys)
    WaveStart *wave_start; // [W]
    int32_t B, total_q;
    int64_t total_kv;
    int32_t max_q, max_kv_len;
    int32_t Hq, Hkv, G;
    int32_t W;             // waves the tile list is split over
    int32_t HI;            // KV-head interleave: the HI waves u with equal u / HI (waves of one
                           // work-group) walk the same keys of different heads, so that the
                           // pieces of a cache row are requested together (HI divides W, Hkv
                           // and the waves of a work-group; 1 = one head-major list)
    int32_t *error_flag;   // set to 1 by a wave whose bounded wait for its partner ran out
    int32_t *cuts;         // [B][Hkv][4] first and last part that hold tiles of the (sequence,
                           // head), first query row, query rows; error_flag[1]: every part owns tiles
    int32_t Mpad;          // G*max_q rounded up to kColTile
    float scale2;          // sm_scale * log2(e) (fp32 kernel)
    float scale_abs;       // its magnitude, at least 1e-37, and ...
    uint32_t q_sign;       // ... the sign bits that make up for it, two bf16 (bf16 kernel)
    int32_t inline_setup;  // the main kernel builds the split itself (no set-up kernel in front of it)
    uint32_t g_inverse;    // ceil(65536 / G)
};

struct SeqInfo {
    int32_t q0, R;
    int64_t kv0;    // first token of the sequence in the cache; paged: its first entry in page_table
    int32_t L;
    int32_t tiles;  // ceil(L / kTileKeys), 0 for a sequence without rows
};

// The index arrays are read-only for the whole launch.  Reading them through the constant
// address space lets a wave-uniform index become a scalar load, which does not count as a
// vector memory request: a look-up in the middle of the tile stream then waits for itself
// only, not for every tile request in flight.
template <typename T>
using ConstPtr = const T __attribute__((address_space(4))) *;

template <typename T>
__device__ inline ConstPtr<T> as_constant(const T *ptr) {
    return (ConstPtr<T>)ptr;
}

// Per-sequence bounds, clamped by the host-side totals so that no device data can push an
// access outside the buffers.
__device__ inline SeqInfo seq_info(const AttnParams &p, int b) {
    SeqInfo s;
    const ConstPtr<int32_t> q_indptr = as_constant(p.q_indptr);
    const ConstPtr<int64_t> kv_indptr = as_constant(p.kv_indptr);
    s.q0 = q_indptr[b];
    int32_t R = q_indptr[b + 1] - s.q0;
    s.q0 = max(0, min(s.q0, p.total_q));
    R = max(0, min(R, min(p.max_q, p.total_q - s.q0)));
    s.R = R;
    if (p.page_table) {
        const ConstPtr<int32_t> page_indptr = as_constant(p.page_indptr);
        int32_t e0 = page_indptr[b];
        int32_t pages = page_indptr[b + 1] - e0;
        e0 = max(0, min(e0, p.table_len));
        pages = max(0, min(pages, p.table_len - e0));
        int64_t L = as_constant(p.kv_len)[b];
        L = min(L, (int64_t)pages << p.page_shift);
        L = max((int64_t)0, min(L, (int64_t)p.max_kv_len));
        s.kv0 = e0;
        s.L = (int32_t)L;
        s.tiles = R > 0 ? (s.L + kTileKeys - 1) / kTileKeys : 0;
        return s;
    }
    int64_t kv0 = kv_indptr[b];
    int64_t L = kv_indptr[b + 1] - kv0;
    kv0 = kv0 < 0 ? 0 : (kv0 > p.total_kv ? p.total_kv : kv0);
    if (L > p.total_kv - kv0) L = p.total_kv - kv0;
    if (L > p.max_kv_len) L = p.max_kv_len;
    if (L < 0) L = 0;
    s.kv0 = kv0;
    s.L = (int32_t)L;
    s.tiles = R > 0 ? (s.L + kTileKeys - 1) / kTileKeys : 0;
    return s;
}

__device__ inline float hw_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Partner values across the four 16-lane rows of a wave, through the gfx950 lane-swap
// instructions (no LDS round trip).  With both operands equal to x, v_permlane32_swap leaves
// in the two results the lane's own value and the value of lane ^ 32; v_permlane16_swap does
// the same for lane ^ 16.
__device__ inline float max_across_rows(float x) {
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ inline float sum_across_rows(float x) {
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The split.  The KV heads form HI sub-lists of Hkv/HI heads (sub-list s: the heads s, s + HI,
// ...: the heads that the waves of one work-group read at a time are neighbours in a cache row);
// a sub-list is the flat tile list (head, sequence, tile) of its heads, `sub_total` tiles long,
// cut evenly into W/HI parts.
// Wave u takes part u / HI of sub-list u % HI.  Part r owns flat tiles
// [range_begin(r), range_begin(r+1)) of its sub-list.
struct Split {
    int64_t T;           // tiles of one KV head
    int64_t sub_total;   // tiles of one sub-list
    int32_t parts, hps;  // parts per sub-list, heads per sub-list
};

// (Unequal parts were tried twice, to make up for dies that are served less bandwidth under
// saturation: with equal parts the work-groups of two to four of the eight dies end 10-15 us
// after the others', and the launch lasts as long as they do.  Which dies are the slow ones
// changes from launch to launch, so no fixed weighting helps: 200-204 us with the odd-numbered
// dies' parts 2-7 % smaller, 203-204 us with equal parts.)
__device__ inline Split make_split(const AttnParams &p, int64_t T) {
    Split s;
    s.T = T;
    s.hps = p.Hkv / p.HI;
    s.sub_total = T * s.hps;
    s.parts = p.W / p.HI;
    return s;
}

// Quotient of two non-negative 64-bit numbers.  A 64-bit division is a long instruction sequence
// on this hardware; the operands here nearly always fit 32 bits, where it is a short one.  Both
// branches give the same integer.
__device__ inline int64_t div_nonneg(int64_t num, int64_t den) {
    if (((uint64_t)num | (uint64_t)den) <= 0xffffffffull) return (int64_t)((uint32_t)num / (uint32_t)den);
    return num / den;
}

__device__ inline int64_t range_begin(const Split &s, int r) {
    const int64_t num = (int64_t)r * s.sub_total;
    if ((s.parts & (s.parts - 1)) == 0) return num >> (31 - __builtin_clz(s.parts));  // the usual case
    return div_nonneg(num, s.parts);
}

__device__ inline int part_of_tile(const Split &s, int64_t x) {  // x: flat index in the sub-list
    return (int)div_nonneg((x + 1) * s.parts - 1, s.sub_total);
}

__device__ inline bool part_owns_tiles(const Split &s, int r) {
    return range_begin(s, r + 1) > range_begin(s, r);
}

// Where wave w of the split starts: `prefix(i)` is the tile prefix over sequences and `info(b)`
// the bounds of sequence b (from LDS, or from the index arrays in global memory).
template <typename Prefix, typename Info>
__device__ inline WaveStart make_wave_start(const AttnParams &p, const Split &sp, int w, Prefix prefix, Info info) {
    WaveStart st{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t T = sp.T;
    if (T > 0) {
        const int r = w / p.HI, sub = w % p.HI;
        const int64_t a0 = range_begin(sp, r), a1 = range_begin(sp, r + 1);
        st.n = (int32_t)(a1 - a0);
        const int64_t head = a0 < T ? 0 : div_nonneg(a0, T);  // (one head per sub-list: always 0)
        st.h = (int32_t)head * p.HI + sub;
        const int32_t rem = (int32_t)(a0 - head * T);
        int lo = 0, hi = p.B - 1;          // last b with prefix[b] <= rem
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (prefix(mid) <= rem) lo = mid; else hi = mid - 1;
        }
        st.b = lo;
        st.t = rem - prefix(lo);
        const SeqInfo si = info(lo);
        st.q0 = si.q0;
        st.R = si.R;
        st.L = si.L;
        st.tiles = si.tiles;
        st.kv0 = si.kv0;
    }
    return st;
}

// For (sequence, KV head) idx: the first and the last part that hold its tiles, its first query
// row and its query rows (what the combine kernel needs; the 64-bit divisions behind the parts
// are done once here, not by every thread of that kernel).
template <typename Prefix, typename Info>
__device__ inline void write_cut(const AttnParams &p, const Split &sp, int idx, Prefix prefix, Info info) {
    const int b = idx / p.Hkv, kvh = idx % p.Hkv;
    const int tiles = prefix(b + 1) - prefix(b);
    int r_first = 0, r_last = 0;
    if (tiles > 0) {
        const int64_t first_tile = (int64_t)(kvh / p.HI) * sp.T + prefix(b);
        r_first = part_of_tile(sp, first_tile);
        r_last = part_of_tile(sp, first_tile + tiles - 1);
    }
    const SeqInfo si = info(b);
    *reinterpret_cast<int4 *>(p.cuts + 4 * (int64_t)idx) = int4{r_first, r_last, si.q0, si.R};
}

// Set-up kernel (one work-group): builds the tile prefix over sequences, every wave's starting
// point and the cut table.  Only batches too large for the main kernel to do this itself in its
// prologue (kInlineSeqs) take this extra launch.
constexpr int kPrepLdsSeqs = 8192;  // batches up to this size keep the prefix in LDS for the searches
constexpr int kInlineSeqs = 2048;   // batches up to this size: the main kernel's work-groups build the split themselves

__global__ __launch_bounds__(1024) void attn_prep_kernel(AttnParams p) {
    __shared__ int sh_scan[1024];
    __shared__ int sh_prefix[kPrepLdsSeqs + 1];
    __shared__ int sh_base;
    const int tid = threadIdx.x;
    const bool in_lds = p.B <= kPrepLdsSeqs;
    if (tid == 0) {
        sh_base = 0;
        p.tile_prefix[0] = 0;
        sh_prefix[0] = 0;
        *p.error_flag = 0;
    }
    __syncthreads();
    for (int b0 = 0; b0 < p.B; b0 += 1024) {
        const int b = b0 + tid;
        const int nt = b < p.B ? seq_info(p, b).tiles : 0;
        // inclusive scan of the block: lane shuffles inside a wave, wave totals through LDS
        int incl = nt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o);
            if ((tid & 63) >= o) incl += y;
        }
        if ((tid & 63) == 63) sh_scan[tid >> 6] = incl;
        __syncthreads();
        int before = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w)
            if (w < (tid >> 6)) before += sh_scan[w];
        incl += before;
        const int base = sh_base;
        if (b < p.B) {
            p.tile_prefix[b + 1] = base + incl;
            if (in_lds) sh_prefix[b + 1] = base + incl;
        }
        __syncthreads();
        if (tid == 1023) sh_base = base + incl;
        __syncthreads();
    }
    auto prefix = [&](int i) { return in_lds ? sh_prefix[i] : p.tile_prefix[i]; };
    const Split sp = make_split(p, sh_base);
    auto info = [&](int b) { return seq_info(p, b); };
    for (int w = tid; w < p.W; w += 1024) p.wave_start[w] = make_wave_start(p, sp, w, prefix, info);
    for (int idx = tid; idx < p.B * p.Hkv; idx += 1024) write_cut(p, sp, idx, prefix, info);
    if (tid == 0) p.error_flag[1] = sp.sub_total >= sp.parts ? 1 : 0;
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel
// ------------------------------------------------------------------------------------------
template <int D>
struct Bf16Cfg {
    static constexpr int kRowElems = D + 8;                 // padded LDS row (bf16 elements)
    static constexpr int kRowBytes = kRowElems * 2;
    // (V rows are padded by 32 bytes: the four rows that sixteen lanes of a transposing read touch
    // then fall into different banks; K rows by 16: sixteen rows read at one column do)
    static constexpr int kVRowBytes = (D + 16) * 2;
    static constexpr int kTileBytes = kTileKeys * kRowBytes;    // one K tile
    static constexpr int kVTileBytes = kTileKeys * kVRowBytes;  // one V tile
    static constexpr int kWaveBytes = kTileBytes + kVTileBytes; // K + V
    static constexpr int kLanesPerRow = D / 8;                // 16-byte pieces per key row
    static constexpr int kRowsPerLoad = 64 / kLanesPerRow;
    static constexpr int kLoads = kTileKeys / kRowsPerLoad;   // global loads per tile per lane
    static constexpr int kKSteps = D / 32;                    // MFMA k-steps of S^T
    static constexpr int kDTiles = D / 16;                    // 16-row d tiles of O^T
    static constexpr int kMergeStride = D + 4;                // fp32 row of the write-out staging (floats)
};

// One 32-key tile of one KV head: kLoads 16-byte loads per lane, rows row_bytes apart.
// `tile` (the address of the tile's first row) is wave-uniform, so a load is (scalar base) +
// (32-bit per-lane offset).  A tile that lies wholly inside its sequence uses the offsets
// row_off[] computed once per kernel.  In a sequence's last, partial tile the rows past
// `rows_valid` re-read the last valid row (they are masked later): the clamp is on the row
// index relative to the tile, two VALU operations per load.  rows_valid = 0 turns the whole
// request into one 256-byte piece.  Both forms issue the same number of loads.
// With 16-token pages a tile spans two pages: `tile` is then the address of the first page's
// rows and `tile_hi` the address the second page's rows would have if row 16 followed row 15
// (second page's base minus 16 rows), so that the same offsets serve both halves; each load
// lies in one half.  Everywhere else tile_hi == tile.
// K, V, the outputs and the partials pass through once: their loads and stores carry the
// non-temporal hint, so that they do not displace what is read again (query rows, partials on
// their way to the combine kernel).  Measured on B = 256 at the 7B shape: 224 -> 210 us with
// the loads marked, 206 us with the stores as well.
template <typename T>
__device__ inline T stream_load(const T *ptr) {
    return __builtin_nontemporal_load(ptr);
}

template <typename T>
__device__ inline void stream_store(T *ptr, const T &v) {
    __builtin_nontemporal_store(v, ptr);
}

template <int D>
__device__ inline void load_tile(u32x4 (&r)[Bf16Cfg<D>::kLoads], const char *tile, const char *tile_hi,
                                 int32_t row_bytes, const uint32_t (&row_off)[Bf16Cfg<D>::kLoads],
                                 int rows_valid, int lane) {
    using C = Bf16Cfg<D>;
    static_assert(C::kLoads % 2 == 0 && (C::kLoads / 2) * C::kRowsPerLoad == 16, "a load lies in one 16-row half");
    if (rows_valid >= kTileKeys - 1) {  // wave-uniform
#pragma unroll
        for (int j = 0; j < C::kLoads; ++j)
            r[j] = stream_load(reinterpret_cast<const u32x4 *>((j < C::kLoads / 2 ? tile : tile_hi) + row_off[j]));
    } else {
        const uint32_t rl = lane / C::kLanesPerRow, cl16 = (lane % C::kLanesPerRow) * 16;
#pragma unroll
        for (int j = 0; j < C::kLoads; ++j) {
            const uint32_t row = min(rl + (uint32_t)(j * C::kRowsPerLoad), (uint32_t)rows_valid);
            const char *base = row < 16u ? tile : tile_hi;
            r[j] = stream_load(reinterpret_cast<const u32x4 *>(base + (row * (uint32_t)row_bytes + cl16)));
        }
    }
}

// Byte offsets, in the K or V pool, of the two 16-row halves of tile t of a paged sequence
// (head h): lo = rows 0..15, hi = what rows 16..31 are addressed from (see load_tile).  The
// page ids come from device memory and are clamped to the pool.
struct TileOffsets {
    int64_t lo, hi;
};

__device__ inline TileOffsets paged_tile_offsets(const AttnParams &p, const SeqInfo &si, int t, int h, int D2,
                                                 int32_t row_bytes) {
    const ConstPtr<int32_t> table = as_constant(p.page_table);
    const int key0 = t * kTileKeys;
    const int last_entry = max(si.L - 1, 0) >> p.page_shift;  // the sequence's last page that holds tokens
    const int e_lo = min(key0 >> p.page_shift, last_entry);
    const int e_hi = min((key0 + 16) >> p.page_shift, last_entry);
    const int64_t pg_lo = max(0, min(table[si.kv0 + e_lo], p.num_pages - 1));
    const int64_t pg_hi = max(0, min(table[si.kv0 + e_hi], p.num_pages - 1));
    const int in_lo = key0 & (p.page_size - 1), in_hi = (key0 + 16) & (p.page_size - 1);
    TileOffsets o;
    o.lo = ((pg_lo << p.page_shift) + in_lo) * (int64_t)row_bytes + (int64_t)h * D2;
    o.hi = ((pg_hi << p.page_shift) + in_hi - 16) * (int64_t)row_bytes + (int64_t)h * D2;
    return o;
}

template <int D, int RowBytes>
__device__ inline void store_tile(const u32x4 (&r)[Bf16Cfg<D>::kLoads], char *lds, int lane) {
    using C = Bf16Cfg<D>;
    const int rl = lane / C::kLanesPerRow, cl = lane % C::kLanesPerRow;
#pragma unroll
    for (int j = 0; j < C::kLoads; ++j)
        *reinterpret_cast<u32x4 *>(lds + (j * C::kRowsPerLoad + rl) * RowBytes + cl * 16) = r[j];
}

// Position of a wave in the flat tile list.  The bounds of the next sequence that has tiles
// are fetched as soon as a sequence is entered, long before they are needed.
struct Cursor {
    int32_t b, h, t;  // sequence, KV head, tile within the sequence
    SeqInfo si;       // bounds of b
    int32_t nb, nh;   // next (sequence, KV head) with tiles; nh == Hkv: the list ends
    SeqInfo nsi;
};

__device__ inline void cursor_find_next(const AttnParams &p, Cursor &c) {
    c.nb = c.b;
    c.nh = c.h;
    for (;;) {
        if (++c.nb >= p.B) {
            c.nb = 0;
            c.nh += p.HI;  // the next head of this wave's sub-list
        }
        if (c.nh >= p.Hkv) return;
        c.nsi = seq_info(p, c.nb);
        if (c.nsi.tiles > 0) return;
    }
}

__device__ inline void cursor_advance(const AttnParams &p, Cursor &c) {
    if (c.t + 1 < c.si.tiles) {
        ++c.t;
        return;
    }
    c.b = c.nb;
    c.h = c.nh;
    c.si = c.nsi;
    c.t = 0;
    if (c.h < p.Hkv) cursor_find_next(p, c);
}

template <int N>
struct Const {
    static constexpr int value = N;
};

// Waits of the tile hand-over.  `flag` is a counter in LDS that only the partner wave
// advances.  The spin is bounded: when the bound is hit the wave records the failure (the
// combine kernel then poisons the output) and stops waiting for the rest of the launch, so
// that every wave reaches its end whatever happens.
constexpr int kSpinLimit = 1 << 24;

// The counters are addressed as LDS explicitly: through a generic pointer every poll would be
// a flat load, which counts as (and waits for) vector memory traffic.
typedef volatile uint32_t __attribute__((address_space(3))) *LdsCounter;

__device__ inline void wait_at_least(LdsCounter flag, uint32_t need, bool &alive, int32_t *error_flag) {
    if (!alive) return;
    for (int spin = 0; spin < kSpinLimit; ++spin) {
        if (*flag >= need) return;
        __builtin_amdgcn_s_sleep(1);
    }
    alive = false;
    *error_flag = 1;
}

// LDS of one form of the kernel.  Eight consumers beside the four producers leave a wave 168
// registers; two column tiles at D = 128 do not fit with their query rows (32 registers), which
// then live in LDS, in the room of every producer's second slot.  A range of four consumers has two
// producers, whose slots alternate; a range of two has one, whose next tiles wait in its registers
// until the slot is free (k = 9, B = 512 at the 14B shape 826 us per call; 860 with two slots, query
// rows in registers and one consumer per SIMD).
template <int D, int NT, int NC>
struct Bf16Form {
    using C = Bf16Cfg<D>;
    static constexpr bool kQueryInLds = D == 128 && NT == 2 && NC == 8;
    static constexpr int kLdsSlots = kQueryInLds ? 1 : kSlots;
    static constexpr int kQueryBytes = kQueryInLds ? NT * kColTile * C::kRowBytes : 0;  // per consumer
    static constexpr int kQueryOffset = kProducers * kLdsSlots * C::kWaveBytes;
    static constexpr int kCounterOffset = kQueryOffset + NC * kQueryBytes;
    static constexpr int kBytes = kCounterOffset + (kProducers + 2 * NC) * (int)sizeof(uint32_t);
};

// One work-group per compute unit: NC consumer waves (one or two per SIMD) and four producer
// waves.  CW = 1: consumer i owns an equal range of the flat tile list; producer i walks the same
// range ahead of it and does nothing but move tiles: global memory -> registers (two tiles in
// flight) -> the pair's two-slot ring in LDS.  A wave that computes cannot keep the memory
// pipeline of its compute unit full (a request can only be issued between two tiles' worth of
// arithmetic, and the unit accepts only a few tiles' worth of requests at a time), a wave that
// only moves data can.  The pair shares two counters in LDS: `filled` (tiles the producer has
// written) and `consumed` (tiles the consumer has finished reading).  A wave's LDS operations
// execute in order, so a counter written after the data (or after the last read) needs no
// further fence.
//
// CW ("column ways") = 2 and 4: that many consumers share one range, each with NT column tiles of
// its own (the accumulators and query rows of 64 columns do not fit a wave's registers), and the
// producers that the work-group has per range (PW) move its tiles in turn, producer w the tiles
// j = w mod PW.  Each consumer keeps its own `consumed`; a producer reuses a slot once all of them
// have passed it.  Every consumer of a range sees every tile, so these forms are bound by the
// consumers: with one per SIMD (NC = 4) the dependent phases of a tile (scores, softmax, second
// product) leave the SIMD idle between them.  NC = 8 puts two on each SIMD, on different ranges
// (B = 256 at the 7B shape, trees of 91 columns: 409 -> 340 us per call by HIP events, 311 us with
// the shorter loop below as well).
template <int D, int NT, typename OutT, int CW, int NC>
__device__ __forceinline__ void attn_bf16(const AttnParams &p) {
    using C = Bf16Cfg<D>;
    static_assert(CW == 1 || CW == 2 || CW == 4, "one, two or four consumers per range");
    constexpr int kStreams = NC / CW;             // ranges per work-group
    constexpr int PW = kProducers / kStreams;     // producers per range
    static_assert(PW >= 1 && kStreams * PW == kProducers, "the producers are shared out evenly");
    using F = Bf16Form<D, NT, NC>;
    extern __shared__ __align__(16) char smem[];  // [kProducers][F::kLdsSlots][kWaveBytes] | query rows | counters
    const LdsCounter counters = (LdsCounter)(smem + F::kCounterOffset);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform by construction
    const bool producer = wave >= NC;
    const int role = producer ? wave - NC : wave;  // index among the producers / consumers
    const int stream = producer ? role / PW : role / CW, way = producer ? role % PW : role % CW;
    const int c16 = lane & 15, g4 = lane >> 4;
    const int u = blockIdx.x * kStreams + stream;  // index of this range in the split
    // columns of a column block: 64 with one consumer per range, else what the consumers hold
    constexpr int kBlockCols = CW == 1 ? kMaxColsPerBlock : CW * NT * kColTile;
    const int col0 = blockIdx.y * kBlockCols + (producer ? 0 : way * NT * kColTile);

    if (threadIdx.x < kProducers + 2 * NC) counters[threadIdx.x] = 0;
    // The split, built by every work-group for itself when the batch is small enough (one kernel
    // launch and its gap less in front of every call).  The bounds of all sequences and their
    // tile prefix are staged in the LDS that the rings will use afterwards, so the searches below
    // read no global memory.  Each work-group also leaves its own starting points and its share
    // of the cut table in the workspace: the combine kernel reads the table, and a later layer
    // of the same forward reads the starting points.
    __shared__ int32_t sh_wave_sum[NC + kProducers];
    __shared__ WaveStart sh_start[kStreams];
    if (p.inline_setup) {  // uniform over the launch
        constexpr int kBlock = (NC + kProducers) * 64;
        static_assert((size_t)kInlineSeqs * sizeof(SeqInfo) + (kInlineSeqs + 1) * sizeof(int32_t) <=
                          (size_t)F::kCounterOffset, "the staging fits where the rings will be");
        SeqInfo *sh_seq = reinterpret_cast<SeqInfo *>(smem);
        int32_t *sh_prefix = reinterpret_cast<int32_t *>(smem + (size_t)kInlineSeqs * sizeof(SeqInfo));
        int base = 0;
        for (int b0 = 0; b0 < p.B; b0 += kBlock) {
            const int b = b0 + (int)threadIdx.x;
            int incl = 0;
            if (b < p.B) {
                const SeqInfo si = seq_info(p, b);
                sh_seq[b] = si;
                incl = si.tiles;
            }
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            if (lane == 63) sh_wave_sum[threadIdx.x >> 6] = incl;
            __syncthreads();
            int before = 0, all = 0;
#pragma unroll
            for (int w = 0; w < NC + kProducers; ++w) {
                const int x = sh_wave_sum[w];
                if (w < (int)(threadIdx.x >> 6)) before += x;
                all += x;
            }
            if (b < p.B) sh_prefix[b + 1] = base + before + incl;
            base += all;
            __syncthreads();
        }
        if (threadIdx.x == 0) sh_prefix[0] = 0;
        __syncthreads();
        auto prefix = [&](int i) { return sh_prefix[i]; };
        auto info = [&](int b) { return sh_seq[b]; };
        const Split sp = make_split(p, base);
        if ((int)threadIdx.x < kStreams) {  // (first wave: the starting points; the others: the cut table)
            const int w = blockIdx.x * kStreams + (int)threadIdx.x;
            WaveStart st{0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            if (w < p.W) {
                st = make_wave_start(p, sp, w, prefix, info);
                if (blockIdx.y == 0) p.wave_start[w] = st;
            }
            sh_start[threadIdx.x] = st;
        }
        if (blockIdx.y == 0 && threadIdx.x >= 64) {
            const int n_cuts = p.B * p.Hkv, per = (n_cuts + (int)gridDim.x - 1) / (int)gridDim.x;
            for (int j = (int)threadIdx.x - 64; j < per; j += kBlock - 64) {
                const int idx = blockIdx.x * per + j;
                if (idx < n_cuts) write_cut(p, sp, idx, prefix, info);
            }
            if (blockIdx.x == 0) {
                for (int b = (int)threadIdx.x - 64; b <= p.B; b += kBlock - 64) p.tile_prefix[b] = sh_prefix[b];
                if (threadIdx.x == 64) {
                    p.error_flag[0] = 0;
                    p.error_flag[1] = sp.sub_total >= sp.parts ? 1 : 0;
                }
            }
        }
    }
    __syncthreads();  // the last barrier, before any wave can leave
    // filled[r]: tiles producer r has written to its ring; consumed[r]: tiles of the range that
    // consumer r has finished with; read_done[r]: tiles whose K and V consumer r has read (CW > 1)
    const LdsCounter filled = counters;
    const LdsCounter consumed = counters + kProducers;
    const LdsCounter read_done = consumed + NC;

    if (u >= p.W) return;  // wave-uniform, and the same for all waves of a range
    int32_t start[10];  // the fields of this range's WaveStart, wave-uniform
    if (p.inline_setup) {
        const int32_t *src = reinterpret_cast<const int32_t *>(&sh_start[stream]);
#pragma unroll
        for (int j = 0; j < 10; ++j) start[j] = __builtin_amdgcn_readfirstlane(src[j]);
    } else {
        const ConstPtr<int32_t> src = as_constant(reinterpret_cast<const int32_t *>(p.wave_start + u));
#pragma unroll
        for (int j = 0; j < 10; ++j) start[j] = src[j];
    }
    const int n_tiles = start[3];
    if (n_tiles <= 0 || start[0] >= p.Hkv) return;

    const int32_t row_bytes = p.Hkv * D * 2;
    bool alive = true;

    // Position of this wave in its range.  The bounds of the sequence after the first are
    // looked up only after the first requests (tile or query rows) have gone out.
    Cursor cp;
    cp.h = start[0];
    cp.b = start[1];
    cp.t = start[2];
    cp.si.q0 = start[4];
    cp.si.R = start[5];
    cp.si.L = start[6];
    cp.si.tiles = start[7];
    cp.si.kv0 = (int64_t)(uint32_t)start[8] | ((int64_t)start[9] << 32);
    cp.nb = cp.b;
    cp.nh = cp.h;
    cp.nsi = cp.si;

    if (producer) {
        // ------------------------------------------------------------------------------------
        // producer: tile j travels through register buffer j % 2 into ring slot j % 2
        // ------------------------------------------------------------------------------------
        uint32_t row_off[C::kLoads];  // byte offset of this lane's piece of each load, full tiles
#pragma unroll
        for (int j = 0; j < C::kLoads; ++j)
            row_off[j] = (uint32_t)(lane / C::kLanesPerRow + j * C::kRowsPerLoad) * (uint32_t)row_bytes +
                         (uint32_t)(lane % C::kLanesPerRow) * 16u;
        u32x4 kr[kSlots][C::kLoads], vr[kSlots][C::kLoads];
        char *ring = smem + role * (F::kLdsSlots * C::kWaveBytes);
        // this producer moves the range's tiles way, way + PW, ...: `pos` is the tile the cursor
        // points at, n_local the number of tiles that are this producer's
        int pos = way;
        const int n_local = (n_tiles - way + PW - 1) / PW;
        // Every step issues its tile requests, also when the range has no tile left: the count
        // of requests behind a buffer's own is then the same on every path, and the wait for a
        // buffer leaves exactly the younger ones in flight.  An idle request re-reads one
        // 256-byte piece of the last tile, which the caches hold.
        bool next_known = false;  // cp.nb / cp.nh / cp.nsi have been looked up
        if (PW > 1 && way > 0 && way < n_tiles) {  // producer `way` starts `way` tiles in
            cursor_find_next(p, cp);
            next_known = true;
            for (int c = 0; c < way; ++c) cursor_advance(p, cp);
        }
        const bool paged = p.page_table != nullptr;
        TileOffsets next_off{0, 0};
        if (paged) next_off = paged_tile_offsets(p, cp.si, cp.t, cp.h, D * 2, row_bytes);
        auto request = [&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            const bool live = pos < n_tiles;
            TileOffsets off;
            if (paged) {
                off = next_off;  // looked up when the cursor moved here
            } else {
                off.lo = (cp.si.kv0 * p.Hkv + cp.h) * (int64_t)(D * 2) + (int64_t)(cp.t * kTileKeys) * row_bytes;
                off.hi = off.lo;
            }
            const int rows_valid = live ? cp.si.L - 1 - cp.t * kTileKeys : 0;
            load_tile<D>(kr[s], static_cast<const char *>(p.k) + off.lo, static_cast<const char *>(p.k) + off.hi,
                         row_bytes, row_off, rows_valid, lane);
            load_tile<D>(vr[s], static_cast<const char *>(p.v) + off.lo, static_cast<const char *>(p.v) + off.hi,
                         row_bytes, row_off, rows_valid, lane);
            if (!next_known) {  // once, with the first tile already on its way
                cursor_find_next(p, cp);
                next_known = true;
            }
            if (live) {
                if (pos + PW < n_tiles) {
#pragma unroll
                    for (int c = 0; c < PW; ++c) cursor_advance(p, cp);
                    // the page ids of the tile after this one: a scalar look-up that has a whole
                    // step to arrive
                    if (paged) next_off = paged_tile_offsets(p, cp.si, cp.t, cp.h, D * 2, row_bytes);
                }
                pos += PW;
            }
        };
        // j: index among this producer's own tiles (tile PW * j + way of the range)
        auto move = [&](auto S, const int j) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            if (j < n_local) {
                // slot s is free once every consumer of the range has finished with the tile
                // that was in it, this producer's tile j - kLdsSlots
                if (j >= F::kLdsSlots) {
                    const uint32_t need = (uint32_t)(PW * (j - F::kLdsSlots) + way + 1);
#pragma unroll
                    for (int c = 0; c < CW; ++c)
                        wait_at_least(consumed + stream * CW + c, need, alive, p.error_flag);
                }
                asm volatile("" ::: "memory");
                char *slot = ring + (s % F::kLdsSlots) * C::kWaveBytes;
                store_tile<D, C::kRowBytes>(kr[s], slot, lane);
                store_tile<D, C::kVRowBytes>(vr[s], slot + C::kTileBytes, lane);
                asm volatile("" ::: "memory");
                filled[role] = (uint32_t)(j + 1);
            }
            request(S);
        };
        request(Const<0>{});
        request(Const<1>{});
        for (int j = 0; j < n_local; j += kSlots) {
            move(Const<0>{}, j);
            move(Const<1>{}, j + 1);
        }
        return;
    }

    // ----------------------------------------------------------------------------------------
    // consumer
    // ----------------------------------------------------------------------------------------
    if (CW > 1 && col0 >= p.G * p.max_q) {
        // no query row of any sequence has a column here (a block of 91 columns leaves the fourth
        // consumer of 32 without any): never waited for
        read_done[role] = 0x7fffffffu;
        consumed[role] = 0x7fffffffu;
        return;
    }
    // this lane's columns: query row i and head gh within the group, fixed for the kernel
    int col_i[NT], col_gh[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = col0 + nt * kColTile + c16;
        col_i[nt] = n / p.G;
        col_gh[nt] = n % p.G;
    }
    // (where registers are short the pair is packed into one of them)
    constexpr bool kPackColumns = F::kQueryInLds || (D == 128 && NT >= 3);
    int col_packed[NT];
    if constexpr (kPackColumns) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            col_packed[nt] = col_i[nt] << 16 | col_gh[nt];
            asm volatile("" : "+v"(col_packed[nt]));
        }
    }
    auto unpack_columns = [&]() __attribute__((always_inline)) {
        if constexpr (kPackColumns) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                int v = col_packed[nt];
                asm volatile("" : "+v"(v));
                col_i[nt] = v >> 16;
                col_gh[nt] = v & 0xffff;
            }
        }
    };

    // (the rows as they are: their sign is applied where they are first used, for an operation
    // right behind a load waits for it)
    auto load_q = [&](bf16x8(&dst)[NT][C::kKSteps], const SeqInfo &s, int kvh) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const bool valid = col_i[nt] < s.R;
            const char *qrow = static_cast<const char *>(p.q) +
                               ((int64_t)(s.q0 + (valid ? col_i[nt] : 0)) * p.Hq + kvh * p.G + col_gh[nt]) * (D * 2);
#pragma unroll
            for (int t = 0; t < C::kKSteps; ++t) {
                u32x4 raw = {0u, 0u, 0u, 0u};
                if (valid) raw = *reinterpret_cast<const u32x4 *>(qrow + (t * 32 + g4 * 8) * 2);
                dst[nt][t] = __builtin_bit_cast(bf16x8, raw);
            }
        }
    };
    auto signed_q = [&](const bf16x8 &x) __attribute__((always_inline)) {  // (a negative scale: the rows are negated, which is exact)
        return __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, x) ^ p.q_sign);
    };

    bf16x8 qreg[NT][C::kKSteps];  // query rows of the segment at hand (F::kQueryInLds: in LDS instead)
    if constexpr (!F::kQueryInLds) load_q(qreg, cp.si, cp.h);  // of the first segment, requested before anything else
    char *q_lds = smem + F::kQueryOffset + role * F::kQueryBytes;  // F::kQueryInLds: this wave's rows
    cursor_find_next(p, cp);
    // query rows of the next segment, requested when the current one begins (not kept for the
    // widest column blocks at D = 128, where the registers do not allow it: a segment then
    // starts by waiting for its query rows)
    constexpr bool kPrefetchQ = !(D == 128 && NT >= 3) && !F::kQueryInLds;
    bf16x8 qnext[kPrefetchQ ? NT : 1][C::kKSteps];
    bool qnext_valid = false;
    bool q_in_place = false;  // qreg already holds the rows of the segment that begins
    bool q_unsigned = !F::kQueryInLds && p.q_sign != 0;  // ... without their sign

    // per-segment state
    int seg_t_first = 0;
    int first_masked_key = 0;  // keys from here on are hidden from some query row
    int col_limit[NT];         // last visible key of the column's query row (-1: no row)
    uint64_t col_mask[NT];     // draft tree: which of the sequence's new tokens the row sees
    const bool tree = p.tree_mask != nullptr;
    float m_run[NT], l_run[NT];
    floatx4 acc_o[NT][C::kDTiles];

    for (int idx = 0; idx < n_tiles; ++idx) {
        const int key0 = cp.t * kTileKeys;
        const int kvh = cp.h;
        // tile idx of the range is tile idx / PW of producer idx % PW of this range
        const int src = stream * PW + idx % PW;
        char *k_lds = smem + src * (F::kLdsSlots * C::kWaveBytes) + ((idx / PW) % F::kLdsSlots) * C::kWaveBytes;
        char *v_lds = k_lds + C::kTileBytes;
        if (idx == 0 || cp.t == 0) {  // a segment begins
            unpack_columns();
            seg_t_first = cp.t;
            first_masked_key = cp.si.L - cp.si.R + 1;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                col_limit[nt] = col_i[nt] < cp.si.R ? (tree ? cp.si.L - 1 : cp.si.L - cp.si.R + col_i[nt]) : -1;
                col_mask[nt] = tree && col_i[nt] < cp.si.R ? p.tree_mask[cp.si.q0 + col_i[nt]] : 0;
                m_run[nt] = kNoMax;
                l_run[nt] = 0.f;
#pragma unroll
                for (int t = 0; t < C::kDTiles; ++t) acc_o[nt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            if constexpr (F::kQueryInLds) {
                bf16x8 qrow[NT][C::kKSteps];
                load_q(qrow, cp.si, cp.h);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int t = 0; t < C::kKSteps; ++t)
                        *reinterpret_cast<u32x4 *>(q_lds + (nt * kColTile + c16) * C::kRowBytes + (t * 32 + g4 * 8) * 2) =
                            __builtin_bit_cast(u32x4, signed_q(qrow[nt][t]));
            } else if (q_in_place) {
                // (moved over at the end of the previous segment)
            } else if (kPrefetchQ && qnext_valid) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int t = 0; t < C::kKSteps; ++t) qreg[nt][t] = signed_q(qnext[kPrefetchQ ? nt : 0][t]);
            } else if (idx > 0) {
                load_q(qreg, cp.si, cp.h);
                q_unsigned = p.q_sign != 0;
            }
            q_in_place = false;
            if constexpr (kPrefetchQ) {
                qnext_valid = cp.nh < p.Hkv;  // the segment after this one, if the list goes on
                if (qnext_valid) load_q(qnext, cp.nsi, cp.nh);
            }
        }

        wait_at_least(filled + src, (uint32_t)(idx / PW + 1), alive, p.error_flag);
        asm volatile("" ::: "memory");
        if constexpr (!F::kQueryInLds) {
            if (q_unsigned) {  // wave-uniform
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int t = 0; t < C::kKSteps; ++t) qreg[nt][t] = signed_q(qreg[nt][t]);
                q_unsigned = false;
            }
        }

        // S^T[key, col] = sum_d K[key, d] Q[col, d]; two 16-key sub-tiles
        floatx4 s_acc[NT][2];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) s_acc[nt][0] = s_acc[nt][1] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (F::kQueryInLds) {
            // one step = the four (NT = 2) fragments of a 32-wide slice of d: both key sub-tiles and
            // every column tile, read one step ahead of the products that use them
            u32x4 kf[2][2], qf[2][NT];
            auto read_step = [&](const int t) __attribute__((always_inline)) {
#pragma unroll
                for (int js = 0; js < 2; ++js)
                    kf[t & 1][js] = *reinterpret_cast<const u32x4 *>(k_lds + (js * 16 + c16) * C::kRowBytes + (t * 32 + g4 * 8) * 2);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    qf[t & 1][nt] = *reinterpret_cast<const u32x4 *>(q_lds + (nt * kColTile + c16) * C::kRowBytes + (t * 32 + g4 * 8) * 2);
            };
            read_step(0);
#pragma unroll
            for (int t = 0; t < C::kKSteps; ++t) {
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < C::kKSteps) read_step(t + 1);
#pragma unroll
                for (int js = 0; js < 2; ++js)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        s_acc[nt][js] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, kf[t & 1][js]), __builtin_bit_cast(bf16x8, qf[t & 1][nt]), s_acc[nt][js], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
            // The K fragments are read a few steps ahead of the products that use them: with one
            // consumer wave per SIMD nothing else hides the latency of a read, and left to
            // itself the compiler waits for each read right behind its issue.  The scheduling
            // barriers keep the order written here.
            constexpr int kFrags = 2 * C::kKSteps;  // (js, t) pairs, js-major
            constexpr int kAhead = 3;
            u32x4 kf[kFrags];
            auto read_k = [&](const int i) __attribute__((always_inline)) {
                const int js = i / C::kKSteps, t = i % C::kKSteps;
                kf[i] = *reinterpret_cast<const u32x4 *>(k_lds + (js * 16 + c16) * C::kRowBytes + (t * 32 + g4 * 8) * 2);
            };
#pragma unroll
            for (int i = 0; i < kAhead; ++i) read_k(i);
#pragma unroll
            for (int i = 0; i < kFrags; ++i) {
                __builtin_amdgcn_sched_barrier(0);
                if (i + kAhead < kFrags) read_k(i + kAhead);
                const bf16x8 a = __builtin_bit_cast(bf16x8, kf[i]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    s_acc[nt][i / C::kKSteps] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qreg[nt][i % C::kKSteps], s_acc[nt][i / C::kKSteps], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        // Online softmax per column; accumulator element (js, i) is key key0 + 16 js + 4 g4 + i.  The
        // scores stay unscaled: the scale is positive, so it commutes with the maximum, and it is
        // applied in the multiply-add that forms the exponent.
        const bool tail = key0 + kTileKeys > first_masked_key;  // wave-uniform
        if (tail) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int js = 0; js < 2; ++js)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int key = key0 + js * 16 + g4 * 4 + i;
                        bool seen = key <= col_limit[nt];
                        if (tree) {
                            const int j = key - (first_masked_key - 1);  // index among the new tokens
                            seen = seen && (j < 0 || ((col_mask[nt] >> (j & 63)) & 1u));
                        }
                        s_acc[nt][js][i] = seen ? s_acc[nt][js][i] : -INFINITY;
                    }
        }
        // The exponent reference m_run follows the running maximum lazily: it moves only when some
        // key's score exceeds it by more than kRescaleSlack (probabilities then stay below
        // 2^kRescaleSlack, harmless in bf16 and fp32).  Nearly every tile therefore takes one
        // comparison per lane and column; the maximum across lanes, the factor for what has been
        // accumulated and its application belong to the rare tile that moves a reference.  (With
        // the maximum across lanes formed for every tile and the scale applied to every score the
        // loop had about 270 vector instructions per tile and consumer at two column tiles, the byte
        // permutes that the transposing reads of V replace included; it has about 190.)
        float lane_max[NT];
        bool rescale = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const floatx4 x = s_acc[nt][0], y = s_acc[nt][1];
            lane_max[nt] = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])));
            rescale |= fmaf(lane_max[nt], p.scale_abs, -m_run[nt]) > kRescaleSlack;
        }
        if (__any(rescale)) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float mloc = max_across_rows(lane_max[nt]) * p.scale_abs;
                const float mnew = mloc > m_run[nt] + kRescaleSlack ? mloc : m_run[nt];
                const float alpha = hw_exp2(m_run[nt] - mnew);
                m_run[nt] = mnew;
                l_run[nt] *= alpha;
#pragma unroll
                for (int t = 0; t < C::kDTiles; ++t) acc_o[nt][t] *= alpha;
            }
        }
        bf16x8 pfrag[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float psum = 0.f;
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pv[e] = hw_exp2(fmaf(s_acc[nt][e / 4][e % 4], p.scale_abs, -m_run[nt]));
                psum += pv[e];
            }
            l_run[nt] += psum;
            bf16x8 pf;
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const bf16x2 two = __builtin_convertvector(floatx2{pv[e], pv[e + 1]}, bf16x2);
                pf[e] = two[0];
                pf[e + 1] = two[1];
            }
            pfrag[nt] = pf;
        }

        // O^T[d, col] += sum_key V[key, d] P[key, col]; contraction slot e of lane group g4 is
        // key 16 (e/4) + 4 g4 + e%4, matching the score accumulators.  V is read with the
        // transposing LDS read: the sixteen lanes of a group address four keys x sixteen d (lane i:
        // key i/4, the four d from 4 (i%4)) and lane i receives d = i of the four keys, which is
        // the A operand of the product as it stands (8-byte reads along d needed 32 byte permutes
        // per tile to regroup them).
        {
            typedef s16x4 __attribute__((address_space(3))) *LdsV;
            constexpr int kAhead = 3;
            s16x4 vf[C::kDTiles][2];
            const char *v_lane = v_lds + (4 * g4 + c16 / 4) * C::kVRowBytes + (c16 % 4) * 8;
            auto read_v = [&](const int t) __attribute__((always_inline)) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    vf[t][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsV)(v_lane + h * 16 * C::kVRowBytes + t * 32));
            };
#pragma unroll
            for (int t = 0; t < kAhead; ++t) read_v(t);
#pragma unroll
            for (int t = 0; t < C::kDTiles; ++t) {
                __builtin_amdgcn_sched_barrier(0);
                if (t + kAhead < C::kDTiles) read_v(t + kAhead);
                const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vf[t][0], vf[t][1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc_o[nt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pfrag[nt], acc_o[nt][t], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        if (idx == n_tiles - 1 || cp.t == cp.si.tiles - 1) {  // the segment ends
            // A segment that covers its whole sequence writes the output; otherwise it leaves a
            // partial in one of this pair's two slots (0: the sequence began in an earlier
            // range, 1: it starts here and continues in the next one).  Lane (c16, g4) holds,
            // for column c16 of each column tile, d = 16 t + 4 g4 + r in acc_o[nt][t][r]:
            // written out like that, every store would scatter 16-byte pieces over 64 rows.
            // The columns go through the ring slot of the tile just finished (still owned by
            // the consumers of the range) instead, 32 at a time, and leave it as whole rows.
            // Two consumers that share the range take half of the slot each, 16 columns at a
            // time, once both have read the tile.
            unpack_columns();
            const bool whole = seg_t_first == 0 && cp.t == cp.si.tiles - 1;
            const int64_t slot = 2 * (int64_t)u + (seg_t_first > 0 ? 0 : 1);
            // The next segment's query rows (requested when this segment began) move into place
            // now, ahead of the stores below: vector memory operations complete in issue order,
            // so taking them over after the stores would wait for every store's acknowledgement
            // while the ring fills up behind this wave.
            if constexpr (kPrefetchQ) {
                if (qnext_valid && idx + 1 < n_tiles) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int t = 0; t < C::kKSteps; ++t) qreg[nt][t] = signed_q(qnext[nt][t]);
                    q_in_place = true;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // (the staging reuses memory that other code reads and writes as 32-bit integer
            // vectors: keep the compiler from moving either across the borders of this block;
            // the hardware runs a wave's LDS operations in order)
            asm volatile("" ::: "memory");
            if constexpr (CW > 1) {
                read_done[role] = (uint32_t)(idx + 1);
#pragma unroll
                for (int c = 1; c < CW; ++c)  // every consumer of the range has read the tile
                    wait_at_least(read_done + stream * CW + (way + c) % CW, (uint32_t)(idx + 1), alive, p.error_flag);
                asm volatile("" ::: "memory");
            }
            // columns staged together: what fits this consumer's share of the slot
            constexpr int kStageCols = 2 * kColTile / CW;     // 32, 16 or 8
            constexpr int kPasses = (NT * kColTile + kStageCols - 1) / kStageCols;
            float *stage = reinterpret_cast<float *>(k_lds + way * (C::kWaveBytes / CW));  // [kStageCols][kMergeStride]
            float *stat = stage + kStageCols * C::kMergeStride;  // [kStageCols]: max, sum, output row, largest magnitude
            static_assert((kStageCols * C::kMergeStride + kStageCols * 4) * 4 <= C::kWaveBytes / CW, "staging fits its share of a slot");
            static_assert((C::kWaveBytes / CW) % 16 == 0, "shares of a slot stay 16-byte aligned");
            constexpr int kLanesPerOutRow = D / 4;            // lanes that cover a row, 4 floats each
            constexpr int kRowsPerPass = 64 / kLanesPerOutRow;
#pragma unroll
            for (int pp = 0; pp < kPasses; ++pp) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    // column tile nt has columns nt*16 .. nt*16+15 of this consumer; pass pp
                    // stages columns pp*kStageCols .. +kStageCols-1 of them
                    if ((nt * kColTile) / kStageCols <= pp && pp <= (nt * kColTile + kColTile - 1) / kStageCols) {
                        const int local = nt * kColTile + c16 - pp * kStageCols;   // row of the stage, if in this pass
                        const bool mine = local >= 0 && local < kStageCols;       // (lane-dependent only for 8-column passes)
                        const float lt = sum_across_rows(l_run[nt]);
                        float amax = 0.f;  // largest magnitude of the column (scale of a partial)
                        if (!whole) {
#pragma unroll
                            for (int t = 0; t < C::kDTiles; ++t)
#pragma unroll
                                for (int r = 0; r < 4; ++r) amax = fmaxf(amax, fabsf(acc_o[nt][t][r]));
                            amax = max_across_rows(amax);
                        }
                        if (mine) {
                            float *row = stage + local * C::kMergeStride;
#pragma unroll
                            for (int t = 0; t < C::kDTiles; ++t)
                                *reinterpret_cast<floatx4 *>(row + 16 * t + 4 * g4) = acc_o[nt][t];
                            if (g4 == 0) {
                                const int ci = col_i[nt];
                                const int orow = ci < cp.si.R ? (cp.si.q0 + ci) * p.Hq + kvh * p.G + col_gh[nt] : -1;
                                *reinterpret_cast<floatx4 *>(stat + local * 4) =
                                    floatx4{m_run[nt], lt, __int_as_float(orow), amax};
                            }
                        }
                    }
                }
                const int n_cols = min(kStageCols, NT * kColTile - pp * kStageCols);  // columns staged in this pass
#pragma unroll
                for (int it = 0; it < kStageCols / kRowsPerPass; ++it) {
                    if (it * kRowsPerPass >= n_cols) break;
                    const int cl = it * kRowsPerPass + lane / kLanesPerOutRow;
                    const int d4 = (lane % kLanesPerOutRow) * 4;
                    const floatx4 st4 = *reinterpret_cast<const floatx4 *>(stat + cl * 4);
                    const floatx4 x = *reinterpret_cast<const floatx4 *>(stage + cl * C::kMergeStride + d4);
                    const float mt = st4[0], lt = st4[1];
                    const int orow = __float_as_int(st4[2]);
                    if (orow >= 0) {
                        if (whole) {
                            const float inv = lt > 0.f ? 1.f / lt : 0.f;
                            OutT *dst = static_cast<OutT *>(p.out) + (int64_t)orow * D + d4;
                            const bf16x2 a = __builtin_convertvector(floatx2{x[0] * inv, x[1] * inv}, bf16x2);
                            const bf16x2 c2 = __builtin_convertvector(floatx2{x[2] * inv, x[3] * inv}, bf16x2);
                            stream_store(reinterpret_cast<u32x2 *>(dst),
                                      (u32x2{__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, c2)}));
                            if (p.lse && d4 == 0)
                                p.lse[orow] = lt > 0.f ? (mt + log2f(lt)) * 0.6931471805599453f : -INFINITY;
                        } else {
                            // (row = wave-uniform part + this lane's row of the pass: written so
                            // that the address is a scalar base plus one 32-bit lane offset that
                            // all passes share; as one 64-bit per-lane expression the compiler
                            // kept a register pair per pass alive through the whole kernel and
                            // spilled some of them)
                            const int64_t prow_u = slot * p.Mpad + col0 + pp * kStageCols + it * kRowsPerPass;
                            const uint32_t lane_row = (uint32_t)(lane / kLanesPerOutRow);
                            // A partial is written as 16-bit fixed point relative to the row's
                            // largest magnitude (error below 2^-16 of it, far under the bf16
                            // rounding of the output): stores into a stream of reads cost several
                            // times their size in read bandwidth, so bytes count here.  A row
                            // that has overflowed keeps its inf/NaN in the scale.
                            const float amax = st4[3];
                            const float qs = (amax > 0.f && amax < INFINITY) ? 32767.f / amax : 0.f;
                            const int q0 = (int)__builtin_rintf(x[0] * qs), q1 = (int)__builtin_rintf(x[1] * qs);
                            const int q2 = (int)__builtin_rintf(x[2] * qs), q3 = (int)__builtin_rintf(x[3] * qs);
                            stream_store(reinterpret_cast<u32x2 *>(p.ws_o + prow_u * D + (lane_row * (uint32_t)D + (uint32_t)d4)),
                                      (u32x2{((uint32_t)q0 & 0xffffu) | ((uint32_t)q1 << 16),
                                             ((uint32_t)q2 & 0xffffu) | ((uint32_t)q3 << 16)}));
                            if (d4 == 0)
                                *reinterpret_cast<floatx4 *>(p.ws_ml + prow_u * 4 + lane_row * 4u) = floatx4{mt, lt, amax, 0.f};
                        }
                    }
                }
                asm volatile("" ::: "memory");
            }
        }
        // every read of the slot has been issued: hand it back
        asm volatile("" ::: "memory");
        consumed[role] = (uint32_t)(idx + 1);
        if (idx + 1 < n_tiles) cursor_advance(p, cp);
    }
}

// Consumers of a work-group: one per range and SIMD, or two per SIMD where they share ranges.
constexpr int consumers_of(int cw) { return cw == 1 ? 4 : 8; }

template <int D, int NT, typename OutT, int CW>
__global__ __launch_bounds__((consumers_of(CW) + kProducers) * 64, 1) void attn_bf16_kernel(AttnParams p) {
    attn_bf16<D, NT, OutT, CW, consumers_of(CW)>(p);
}

// The form for the smallest batches: one column tile per consumer, four consumers on one range.
template <int D, typename OutT>
__global__ __launch_bounds__((4 + kProducers) * 64, 1) void attn_bf16_small_kernel(AttnParams p) {
    attn_bf16<D, 1, OutT, 4, 4>(p);
}


// ------------------------------------------------------------------------------------------
// bf16 kernel for batches of a few tiles per compute unit (the end of a rollout, short prompts)
// ------------------------------------------------------------------------------------------
// Bound by the chain of latencies, not by bandwidth: launch, index arrays, first tile, write-out.  The
// main kernel's chain is long there (a split searched by binary steps behind three barriers, a tile that
// passes through a producer's registers and a ring, four consumers that each see every tile of a
// range).  Here a work-group takes one part of one sequence's tiles for one KV head, its four waves
// every fourth tile of it with all columns, K from memory straight into the registers that the
// product reads, V through LDS for the transposing reads; the waves' results meet in LDS.  A wave's next
// tile is requested as the registers of the one at hand become free (requested two ahead from two
// sets of registers the code is twice as long, which a kernel that runs through it once pays for in
// instruction fetches: 15.4 against 18.2 us below).  The registers are held at 256: beyond, the compiler
// moves the accumulators between two register files for every tile.  What a call takes (main and
// combine kernel; the main kernel's forms / this one, us): 3B shape, 512 to 4096 tokens, k = 0 and 4, B = 8
// 17.5 / 11.3 and 20.4 / 14.1; k = 3, B = 1, 24, 64 17.4 / 11.1, 25.3 / 18.2, 40.8 / 35.0; 7B shape, k = 3, B = 8
// and 32 22.6 / 16.0 and 38.8 / 32.3; heads of 64, two KV heads, k = 2, B = 8 16.3 / 10.5.  In cycles, B = 8, k = 4:
// split 2.6 thousand, query rows 3.3, first tile 4 (memory, 2.4 of arithmetic), second 2.4, merge and
// write-out 4.4.
constexpr int kFewSeqs = 64;    // sequences: a lane each
constexpr int kFewWaves = 4;    // waves per work-group

template <int D, int NT>
struct FewForm {
    using C = Bf16Cfg<D>;
    static constexpr int kCols = NT * kColTile;
    // a wave's LDS: a V tile while it works, its accumulators once it has finished
    static constexpr int kStageBytes = kCols * C::kMergeStride * 4;
    static constexpr int kWaveBytes = kStageBytes > C::kVTileBytes ? kStageBytes : C::kVTileBytes;
    static constexpr int kStatOffset = kFewWaves * kWaveBytes;  // [kFewWaves][kCols] (max, sum)
    static constexpr int kQueryOffset = kStatOffset + kFewWaves * kCols * 8;
    static constexpr int kBytes = kQueryOffset + kCols * C::kRowBytes;
    // where a row's 16-byte piece c is staged: two pieces that a thread reads together lie half a row
    // apart, so that the threads of a row read neighbouring pieces (in row order: two-way bank conflicts)
    static constexpr int chunk(int c) { return c / 2 + c % 2 * (D / 8); }
    static_assert(kBytes <= 160 * 1024, "fits the LDS of a compute unit");
};

// Inclusive sums over the lanes of a wave, without LDS.
__device__ inline int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// Query row of a column (below 256): col / G without a division.
__device__ inline int column_row(const AttnParams &p, int col) { return (int)(((uint32_t)col * p.g_inverse) >> 16); }

template <int CTRL>
__device__ inline float dpp_mov(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

template <int D, int NT>
__global__ __launch_bounds__(kFewWaves * 64, D == 128 && NT == 4 ? 1 : 2) void attn_bf16_few_kernel(AttnParams p) {
    using C = Bf16Cfg<D>;
    using F = FewForm<D, NT>;
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c16 = lane & 15, g4 = lane >> 4;
    // The split: every sequence is cut into parts, as equal as its tiles allow, so that all (part, KV head)
    // pairs find a work-group: ceil(f t) parts of a sequence of t tiles are less than f total + seqs in all.
    // Of four values of f the largest is taken whose parts fit; the first always does.  (At most a part
    // per four tiles, a tile for each wave: smaller parts only add partials; one sequence of 4096 tokens, 3B
    // shape, k = 4 14.4 -> 12.2 us.)  Every wave works it out for itself, a lane per sequence: one round
    // trip to memory and no barrier.
    const int r = blockIdx.x, kvh = blockIdx.y, u = r * p.Hkv + kvh;
    SeqInfo si{};
    int t0 = 0, n = 0;
    int4 cut = {0, 0, 0, 0}, no_cut = {0, 0, 0, 0};
    int cut_at = -1;           // entry of the cut table that is this work-group's to write
    bool empty_lane = false;   // work-group 0: this lane's sequence has no tiles
    if (p.inline_setup) {      // uniform over the launch
        SeqInfo mine{};
        if (lane < p.B) mine = seq_info(p, lane);
        const int tiles = mine.tiles, rows = gridDim.x;
        const int seqs = __popcll(__ballot(tiles > 0));
        const float t = (float)tiles, per_tile = 1.f / (float)max(__builtin_amdgcn_readlane(wave_scan(tiles), 63), 1);
        int parts = 0, upto = 0;  // of this lane's sequence; up to and with it
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float f = fminf((float)(4 * (rows - seqs) + i * seqs) * 0.2499999f * per_tile, 0.25f);
            const int x = tiles > 0 ? min(max((int)ceilf(t * f), 1), tiles) : 0;
            const int sum = wave_scan(x);
            if (i == 0 || __builtin_amdgcn_readlane(sum, 63) <= rows) {
                parts = x;
                upto = sum;
            }
        }
        const int b = __popcll(__ballot(upto <= r));
        if (b < kFewSeqs) {  // (64: no part is left for this work-group)
            auto of_b = [&](int x) { return __builtin_amdgcn_readlane(x, b); };
            si.q0 = of_b(mine.q0);
            si.R = of_b(mine.R);
            si.L = of_b(mine.L);
            si.tiles = of_b(mine.tiles);
            si.kv0 = (int64_t)(uint32_t)of_b((int)mine.kv0) | ((int64_t)of_b((int)(mine.kv0 >> 32)) << 32);
            const int n_parts = of_b(parts), first = of_b(upto) - n_parts, part = r - first;
            const int least = (int)((uint32_t)si.tiles / (uint32_t)n_parts), more = si.tiles - least * n_parts;
            t0 = part * least + min(part, more);
            n = least + (part < more ? 1 : 0);
            cut = int4{first, first + n_parts - 1, si.q0, si.R};
            cut_at = part == 0 ? b * p.Hkv + kvh : -1;
        }
        empty_lane = u == 0 && lane < p.B && tiles == 0;
        no_cut = int4{0, 0, mine.q0, mine.R};
    } else {
        const ConstPtr<int32_t> src = as_constant(reinterpret_cast<const int32_t *>(p.wave_start + u));
        t0 = src[2];
        n = src[3];
        si.q0 = src[4];
        si.R = src[5];
        si.L = src[6];
        si.tiles = src[7];
        si.kv0 = (int64_t)(uint32_t)src[8] | ((int64_t)src[9] << 32);
    }
    const int count = n > wave ? (n - wave + kFewWaves - 1) / kFewWaves : 0;  // this wave's tiles: t0 + wave, + kFewWaves, ...
    char *own = smem + wave * F::kWaveBytes;
    float *stage = reinterpret_cast<float *>(own);  // [kCols][kMergeStride]
    floatx2 *stat = reinterpret_cast<floatx2 *>(smem + F::kStatOffset);

    // what the combine kernel and the later layers of a forward read (behind the first requests)
    auto leave_plan = [&]() __attribute__((always_inline)) {
        if (p.inline_setup && wave == kFewWaves - 1) {
            if (lane == 0) {
                p.wave_start[u] = WaveStart{kvh, 0, t0, n, si.q0, si.R, si.L, si.tiles, si.kv0, 0};
                if (cut_at >= 0) *reinterpret_cast<int4 *>(p.cuts + 4 * (int64_t)cut_at) = cut;
                if (u == 0) {
                    p.error_flag[0] = 0;
                    p.error_flag[1] = 1;  // every part that the cut table names owns tiles
                }
            }
            if (empty_lane)
                for (int h = 0; h < p.Hkv; ++h) *reinterpret_cast<int4 *>(p.cuts + 4 * ((int64_t)lane * p.Hkv + h)) = no_cut;
        }
    };
    if (n > 0) {  // block-uniform
        const int32_t row_bytes = p.Hkv * D * 2;
        // query rows: loaded by the waves together, for each of them through LDS
        constexpr int kPieces = F::kCols * (D / 8), kQLoads = (kPieces + kFewWaves * 64 - 1) / (kFewWaves * 64);
        char *q_lds = smem + F::kQueryOffset;
        u32x4 qr[kQLoads];
#pragma unroll
        for (int i = 0; i < kQLoads; ++i) {  // (a column without a row reads row 0; nothing reads its result)
            const int piece = min(i * kFewWaves * 64 + (int)threadIdx.x, kPieces - 1);
            const int col = piece / (D / 8), row = column_row(p, col), gh = col - row * p.G;
            qr[i] = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.q) +
                                                     ((int64_t)(si.q0 + (row < si.R ? row : 0)) * p.Hq + kvh * p.G + gh) * (D * 2) +
                                                     (piece % (D / 8)) * 16);
        }
        // K goes from memory to the registers that the product reads (lane: key c16 of a half tile, 16 bytes
        // of every 64), V through LDS for the transposing reads
        u32x4 kr[2][C::kKSteps], vr[C::kLoads];
        TileOffsets off;
        auto locate = [&](const int j) __attribute__((always_inline)) {
            const int t = t0 + min(wave + j * kFewWaves, n - 1);
            if (p.page_table) {
                off = paged_tile_offsets(p, si, t, kvh, D * 2, row_bytes);
            } else {
                off.lo = (si.kv0 * p.Hkv + kvh) * (int64_t)(D * 2) + (int64_t)(t * kTileKeys) * row_bytes;
                off.hi = off.lo;
            }
        };
        // (rows past the sequence's end read its last one: a tile's 16-row halves lie at off.lo and off.hi)
        auto request_k = [&](const int j) __attribute__((always_inline)) {
            const int rows_valid = si.L - 1 - (t0 + min(wave + j * kFewWaves, n - 1)) * kTileKeys;
#pragma unroll
            for (int js = 0; js < 2; ++js) {
                const char *base = static_cast<const char *>(p.k) + (js == 1 && rows_valid >= 16 ? off.hi : off.lo);
                const uint32_t o = __umul24((uint32_t)min(js * 16 + c16, rows_valid), (uint32_t)row_bytes) + (uint32_t)g4 * 16u;
#pragma unroll
                for (int x = 0; x < C::kKSteps; ++x)
                    kr[js][x] = stream_load(reinterpret_cast<const u32x4 *>(base + (o + (uint32_t)x * 64u)));
            }
        };
        auto request_v = [&](const int j) __attribute__((always_inline)) {
            const int rows_valid = si.L - 1 - (t0 + min(wave + j * kFewWaves, n - 1)) * kTileKeys;
#pragma unroll
            for (int x = 0; x < C::kLoads; ++x) {
                const char *base = static_cast<const char *>(p.v) + (x >= C::kLoads / 2 && rows_valid >= 16 ? off.hi : off.lo);
                const uint32_t row = (uint32_t)min(lane / C::kLanesPerRow + x * C::kRowsPerLoad, rows_valid);
                vr[x] = stream_load(reinterpret_cast<const u32x4 *>(base + (__umul24(row, (uint32_t)row_bytes) + (uint32_t)(lane % C::kLanesPerRow) * 16u)));
            }
        };
        // which of the sequence's new tokens a column's row sees (a tree's mask, or those up to its own)
        const int first_new = si.L - si.R;
        uint64_t col_mask[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int row = min(column_row(p, nt * kColTile + c16), si.R - 1);
            col_mask[nt] = p.tree_mask ? p.tree_mask[si.q0 + row] & (~0ull >> (64 - si.R)) : (2ull << row) - 1;
        }
        // (a wave without tiles requests the last one as well: the wait for the query rows then leaves
        // the same requests in flight on every path)
        locate(0);
        request_k(0);
        request_v(0);
        leave_plan();
#pragma unroll
        for (int i = 0; i < kQLoads; ++i) {
            const int piece = min(i * kFewWaves * 64 + (int)threadIdx.x, kPieces - 1);
            // (a negative scale: the rows are negated, which is exact)
            *reinterpret_cast<u32x4 *>(q_lds + piece / (D / 8) * C::kRowBytes + (piece % (D / 8)) * 16) = qr[i] ^ p.q_sign;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");  // (LDS only: the tiles stay in flight)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");

        float m_run[NT], l_run[NT];
        floatx4 acc_o[NT][C::kDTiles];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            m_run[nt] = kNoMax;
            l_run[nt] = 0.f;
#pragma unroll
            for (int t = 0; t < C::kDTiles; ++t) acc_o[nt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
        }

#pragma unroll 1
        for (int j = 0; j < count; ++j) {
            const int key0 = (t0 + wave + j * kFewWaves) * kTileKeys;
            // (the query rows of a step are read one step ahead: all of them at once do not fit the registers)
            bf16x8 qf[2][NT];
            auto read_q = [&](const int x) __attribute__((always_inline)) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    qf[x & 1][nt] = *reinterpret_cast<const bf16x8 *>(q_lds + (nt * kColTile + c16) * C::kRowBytes + (x * 32 + g4 * 8) * 2);
            };
            floatx4 s_acc[NT][2];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s_acc[nt][0] = s_acc[nt][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            read_q(0);
#pragma unroll
            for (int x = 0; x < C::kKSteps; ++x) {
                __builtin_amdgcn_sched_barrier(0);
                if (x + 1 < C::kKSteps) read_q(x + 1);
#pragma unroll
                for (int js = 0; js < 2; ++js)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        s_acc[nt][js] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[js][x]), qf[x & 1][nt],
                                                                                s_acc[nt][js], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // (the next tile's requests go out as its registers become free)
            if (j + 1 < count) {
                locate(j + 1);
                request_k(j + 1);
            }
            asm volatile("" ::: "memory");
            store_tile<D, C::kVRowBytes>(vr, own, lane);
            asm volatile("" ::: "memory");
            if (j + 1 < count) request_v(j + 1);

            // online softmax as in the main kernel: the reference moves only when a score exceeds it by
            // more than kRescaleSlack
            if (key0 + kTileKeys > first_new + 1) {  // wave-uniform: some row does not see some key
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int js = 0; js < 2; ++js) {
                        const int at = key0 + js * 16 + g4 * 4 - first_new;  // first of four keys, among the new tokens
                        const uint64_t after = at > 63 ? 0 : col_mask[nt] >> (at & 63), before = ~(~col_mask[nt] << (-at & 63));
                        const uint32_t seen = (uint32_t)(at >= 0 ? after : at > -4 ? before : ~0ull);
#pragma unroll
                        for (int i = 0; i < 4; ++i) s_acc[nt][js][i] = (seen >> i) & 1u ? s_acc[nt][js][i] : -INFINITY;
                    }
            }
            float lane_max[NT];
            bool rescale = false;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const floatx4 x = s_acc[nt][0], y = s_acc[nt][1];
                lane_max[nt] = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])));
                rescale |= fmaf(lane_max[nt], p.scale_abs, -m_run[nt]) > kRescaleSlack;
            }
            if (__any(rescale)) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const float mloc = max_across_rows(lane_max[nt]) * p.scale_abs;
                    const float mnew = mloc > m_run[nt] + kRescaleSlack ? mloc : m_run[nt];
                    const float alpha = hw_exp2(m_run[nt] - mnew);
                    m_run[nt] = mnew;
                    if (j > 0) {  // wave-uniform
                        l_run[nt] *= alpha;
#pragma unroll
                        for (int t = 0; t < C::kDTiles; ++t) acc_o[nt][t] *= alpha;
                    }
                }
            }
            bf16x8 pfrag[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float psum = 0.f;
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const float a = hw_exp2(fmaf(s_acc[nt][e / 4][e % 4], p.scale_abs, -m_run[nt]));
                    const float c = hw_exp2(fmaf(s_acc[nt][e / 4][e % 4 + 1], p.scale_abs, -m_run[nt]));
                    psum += a;
                    psum += c;
                    const bf16x2 two = __builtin_convertvector(floatx2{a, c}, bf16x2);
                    pfrag[nt][e] = two[0];
                    pfrag[nt][e + 1] = two[1];
                }
                l_run[nt] += psum;
            }

            typedef s16x4 __attribute__((address_space(3))) *LdsV;
            const char *v_lane = own + (4 * g4 + c16 / 4) * C::kVRowBytes + (c16 % 4) * 8;
            s16x4 vf[C::kDTiles][2];
#pragma unroll
            for (int t = 0; t < C::kDTiles; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    vf[t][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsV)(v_lane + h * 16 * C::kVRowBytes + t * 32));
#pragma unroll
            for (int t = 0; t < C::kDTiles; ++t) {
                const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vf[t][0], vf[t][1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc_o[nt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pfrag[nt], acc_o[nt][t], 0, 0, 0);
            }
            asm volatile("" ::: "memory");  // (the reads have been issued: a wave's LDS operations run in order)
        }

        asm volatile("" ::: "memory");
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {  // (of a wave without tiles: zeros)
            const float lt = sum_across_rows(l_run[nt]);
            float *row = stage + (nt * kColTile + c16) * C::kMergeStride;
#pragma unroll
            for (int t = 0; t < C::kDTiles; ++t) *reinterpret_cast<floatx4 *>(row + F::chunk(4 * t + g4) * 4) = acc_o[nt][t];
            if (g4 == 0) stat[wave * F::kCols + nt * kColTile + c16] = floatx2{m_run[nt], lt};
        }
    } else {
        leave_plan();
    }
    __syncthreads();

    // the waves' results are merged in wave order; eight values of a column per thread
    constexpr int kTpc = D / 8;
    constexpr int kColsPerPass = kFewWaves * 64 / kTpc;
    const bool whole = n == si.tiles;
    const int64_t slot = 2 * (int64_t)u + (t0 > 0 ? 0 : 1);
    const int M = n > 0 ? p.G * si.R : 0;
    constexpr int kPasses = (F::kCols + kColsPerPass - 1) / kColsPerPass;
    const int d8 = ((int)threadIdx.x % kTpc) * 8;
    // (all reads ahead of all arithmetic: left alone the compiler keeps two of them in flight)
    floatx2 ml[kPasses][kFewWaves];
    floatx4 part[kPasses][kFewWaves][2];
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
        const int col = min(i * kColsPerPass + (int)threadIdx.x / kTpc, F::kCols - 1);
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) {
            const float *src = reinterpret_cast<const float *>(smem + w * F::kWaveBytes) + col * C::kMergeStride + d8 / 2;
            ml[i][w] = stat[w * F::kCols + col];
            part[i][w][0] = *reinterpret_cast<const floatx4 *>(src);
            part[i][w][1] = *reinterpret_cast<const floatx4 *>(src + D / 2);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    floatx4 o[kPasses][2];
    float mt[kPasses], lt[kPasses], amax[kPasses];
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
        mt[i] = kNoMax;
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) mt[i] = fmaxf(mt[i], ml[i][w][0]);
        lt[i] = 0.f;
        o[i][0] = o[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kFewWaves; ++w) {
            const float wgt = hw_exp2(ml[i][w][0] - mt[i]);
            lt[i] += ml[i][w][1] * wgt;
            o[i][0] = o[i][0] + part[i][w][0] * wgt;
            o[i][1] = o[i][1] + part[i][w][1] * wgt;
        }
        // (16-bit fixed point relative to the row's largest magnitude, as the main kernel writes it)
        float m = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(o[i][e / 4][e % 4]));
        m = fmaxf(m, dpp_mov<0xb1>(m));                     // quad_perm:[1,0,3,2]
        m = fmaxf(m, dpp_mov<0x4e>(m));                     // quad_perm:[2,3,0,1]
        m = fmaxf(m, dpp_mov<0x141>(m));                    // row_half_mirror
        if (kTpc == 16) m = fmaxf(m, dpp_mov<0x140>(m));    // row_mirror
        amax[i] = m;
    }
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
        const int col = i * kColsPerPass + (int)threadIdx.x / kTpc;
        if (col >= M) break;
        const floatx4 a = o[i][0], c = o[i][1];
        if (whole) {
            const float inv = lt[i] > 0.f ? 1.f / lt[i] : 0.f;
            const int row = column_row(p, col), gh = col - row * p.G;
            const int64_t orow = (int64_t)(si.q0 + row) * p.Hq + kvh * p.G + gh;
            auto pack = [&](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{x * inv, y * inv}, bf16x2)); };
            stream_store(reinterpret_cast<u32x4 *>(static_cast<uint16_t *>(p.out) + orow * D + d8),
                         (u32x4{pack(a[0], a[1]), pack(a[2], a[3]), pack(c[0], c[1]), pack(c[2], c[3])}));
            if (p.lse && d8 == 0) p.lse[orow] = lt[i] > 0.f ? (mt[i] + log2f(lt[i])) * 0.6931471805599453f : -INFINITY;
        } else {
            const float qs = (amax[i] > 0.f && amax[i] < INFINITY) ? 32767.f / amax[i] : 0.f;
            auto pack = [&](float x, float y) { return ((uint32_t)(int)__builtin_rintf(x * qs) & 0xffffu) | ((uint32_t)(int)__builtin_rintf(y * qs) << 16); };
            const int64_t row = slot * p.Mpad + col;
            *reinterpret_cast<u32x4 *>(p.ws_o + row * D + d8) = u32x4{pack(a[0], a[1]), pack(a[2], a[3]), pack(c[0], c[1]), pack(c[2], c[3])};
            if (d8 == 0) *reinterpret_cast<floatx4 *>(p.ws_ml + row * 4) = floatx4{mt[i], lt[i], amax[i], 0.f};
        }
    }
}

// ------------------------------------------------------------------------------------------
// fp32 kernel: one work-group per (sequence, query head, query row), no split
// ------------------------------------------------------------------------------------------
// A chunk of 256 keys at a time: each thread forms one key's score, a wave's scores are reduced in
// the wave, and the probabilities of the chunk, relative to their wave's maximum, go through LDS
// (two buffers in turn: one barrier per chunk) to the threads that own four values of d of every
// sixteenth (D = 64) or eighth key.  The workloads that run in fp32 are small, so what bounds the
// kernel is the chain of latencies: index arrays, query row, key rows, barrier, value rows, merge.
// Sixteen loads of a key row and eight value rows are in flight together (with one value per thread,
// one load in flight and six barriers per chunk: B = 4, k = 4, 4 heads of 64, up to 256 keys
// 11.1 us; now 7.4 us).
// A row of at most 64 visible keys is one wave's work: the other three leave at once, and a wave without
// keys reads none (with all four at work on rows of a few keys the loads of keys that nobody has took
// most of the time).  The registers are held at four waves per SIMD, between the loads in flight that
// small grids want and the work-groups that large ones do.  D = 64, k = 3, us per call (one value per
// thread, then, now): B = 128, 16 keys 7.2, 13.8, 6.4; 80 keys 13.7, 16.2, 13.0; 256 keys 40.9, 38.5, 36.5;
// 1000 keys 144, 143, 149; B = 512, 16 keys 18.8, 44.0, 15.6; B = 4, k = 4, 16 keys 5.3, 5.5, 4.6; 256 keys 14.6,
// 7.8, 7.7.
constexpr int kF32Threads = 256;

// One row: query row i and head h of a sequence, by THREADS threads (a whole number of waves).
template <int D, int THREADS>
__device__ __forceinline__ void attn_f32_row(const AttnParams &p, const SeqInfo &si, int h, int i, int k_end) {
    constexpr int kWaves = THREADS / 64;
    constexpr int kLanesPerKey = D / 4;                       // threads that cover a value row, four values each
    constexpr int kGroups = THREADS / kLanesPerKey;           // keys handled at a time in the second product
    constexpr int kDepth = 8;                                 // value rows in flight per thread
    __shared__ floatx4 sh_q[D / 4];
    __shared__ float sh_p[2][THREADS];
    __shared__ float sh_m[2][kWaves], sh_l[2][kWaves];
    __shared__ floatx4 sh_part[kGroups][kLanesPerKey];

    auto sync = [&]() __attribute__((always_inline)) {  // (one wave: its LDS operations run in order)
        if constexpr (THREADS > 64) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };
    const int kvh = h / p.G;
    const bool tree = p.tree_mask != nullptr;
    const uint64_t row_mask = tree ? p.tree_mask[si.q0 + i] : 0;
    const int first_new = si.L - si.R;
    const int64_t qrow = (int64_t)(si.q0 + i) * p.Hq + h;
    const bool paged = p.page_table != nullptr;
    // element offset of key j's row of this KV head in the K or V buffer
    auto key_row = [&](int j) __attribute__((always_inline)) -> int64_t {
        if (!paged) return ((si.kv0 + j) * p.Hkv + kvh) * (int64_t)D;
        const int64_t pg = max(0, min(p.page_table[si.kv0 + (j >> p.page_shift)], p.num_pages - 1));
        return (((pg << p.page_shift) + (j & (p.page_size - 1))) * p.Hkv + kvh) * (int64_t)D;
    };
    const float *kb = static_cast<const float *>(p.k);
    const float *vb = static_cast<const float *>(p.v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < D / 4) sh_q[threadIdx.x] = reinterpret_cast<const floatx4 *>(static_cast<const float *>(p.q) + qrow * D)[threadIdx.x];
    sync();

    const int d4 = threadIdx.x % kLanesPerKey, group = threadIdx.x / kLanesPerKey;
    float m_run = -INFINITY, l_run = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    int turn = 0;
    for (int t0 = 0; t0 < k_end; t0 += THREADS, turn ^= 1) {
        const int key = t0 + threadIdx.x;
        floatx4 dot4 = {0.f, 0.f, 0.f, 0.f};
        if (THREADS == 64 || t0 + wave * 64 < k_end) {  // (a wave without keys reads nothing)
            // (keys past the end read the last visible one; their score is dropped)
            const floatx4 *kr = reinterpret_cast<const floatx4 *>(kb + key_row(min(key, k_end - 1)));
#pragma unroll 16
            for (int c = 0; c < D / 4; ++c) {
                const floatx4 x = kr[c], y = sh_q[c];
#pragma unroll
                for (int e = 0; e < 4; ++e) dot4[e] = fmaf(x[e], y[e], dot4[e]);
            }
        }
        const bool seen = key < k_end && (!tree || key < first_new || ((row_mask >> (key - first_new)) & 1u));
        const float s = seen ? ((dot4[0] + dot4[1]) + (dot4[2] + dot4[3])) * p.scale2 : -INFINITY;
        float m_w = s;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) m_w = fmaxf(m_w, __shfl_xor(m_w, o));
        const float pr = seen ? exp2f(s - m_w) : 0.f;
        float l_w = pr;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) l_w += __shfl_xor(l_w, o);
        sh_p[turn][threadIdx.x] = pr;
        if (lane == 0) {
            sh_m[turn][wave] = m_w;
            sh_l[turn][wave] = l_w;
        }
        sync();  // (a buffer is written again two chunks later, behind the next chunk's barrier)
        float m_new = m_run;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) m_new = fmaxf(m_new, sh_m[turn][w]);
        // (no key of the row seen so far, a tree's mask may hide a whole chunk: nothing to add)
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = exp2f(m_run - m_safe);
        float wgt[kWaves];
        l_run *= alpha;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            wgt[w] = exp2f(sh_m[turn][w] - m_safe);
            l_run += sh_l[turn][w] * wgt[w];
        }
        acc *= alpha;
        m_run = m_new;
        const int nk = min(THREADS, k_end - t0);
        for (int j0 = group; j0 < nk; j0 += kGroups * kDepth) {
            floatx4 v[kDepth];
            float pj[kDepth];
#pragma unroll
            for (int e = 0; e < kDepth; ++e) {
                const int j = j0 + e * kGroups;
                v[e] = *reinterpret_cast<const floatx4 *>(vb + key_row(t0 + min(j, nk - 1)) + d4 * 4);
                const int w = min(j, THREADS - 1) >> 6;
                float f = wgt[0];
#pragma unroll
                for (int x = 1; x < kWaves; ++x) f = w == x ? wgt[x] : f;
                pj[e] = j < nk ? sh_p[turn][j] * f : 0.f;
            }
#pragma unroll
            for (int e = 0; e < kDepth; ++e)
                if (j0 + e * kGroups < nk)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] = fmaf(pj[e], v[e][c], acc[c]);
        }
    }
    sh_part[group][d4] = acc;
    sync();
    for (int d = threadIdx.x; d < D; d += THREADS) {
        float o = 0.f;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) o += sh_part[g][d / 4][d % 4];
        static_cast<float *>(p.out)[qrow * D + d] = l_run > 0.f ? o / l_run : 0.f;
        if (p.lse && d == 0)
            p.lse[qrow] = l_run > 0.f ? (m_run + log2f(l_run)) * 0.6931471805599453f : -INFINITY;
    }
}

template <int D>
__global__ __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(1, 4))) void attn_f32_kernel(AttnParams p) {
    const int h = blockIdx.x % p.Hq;
    const int b = blockIdx.x / p.Hq;
    const int i = blockIdx.y;
    const SeqInfo si = seq_info(p, b);
    if (i >= si.R || si.L <= 0) return;
    const int k_end = p.tree_mask ? si.L : min(si.L, si.L - si.R + i + 1);  // one past the last visible key
    if (k_end <= 64) {  // block-uniform
        if (threadIdx.x < 64) attn_f32_row<D, 64>(p, si, h, i, k_end);
    } else {
        attn_f32_row<D, kF32Threads>(p, si, h, i, k_end);
    }
}

// ------------------------------------------------------------------------------------------
// combine: merge the partials of every (sequence, KV head) that a work-group boundary cut
// ------------------------------------------------------------------------------------------
// A column's row of D values is covered by D/8 lanes, eight values each.  What bounds the kernel
// is memory latency, not bandwidth: the cut table, then the partials, a few in flight at a time.
// PW = 1: a wave folds all parts of its columns, four waves per work-group.  PW > 1: the PW waves
// of a work-group share the columns of one wave and fold a contiguous slice of the parts each;
// the slices are merged through LDS in part order.  A short batch cuts every sequence into many
// parts (one sequence: all of the split), which one wave per column walks four at a time, a round
// trip each.  Measured (3B shape, k = 4; PW = 1 / 4 / 8): 8 sequences of 2304 tokens, 16 parts
// each, 7.5 / 4.3 / 5.2 us; one sequence of 4096 tokens, 64 parts, 21.7 / 5.9 / 5.2 us, of 16,384
// tokens, 128 parts, 41.6 / 9.3 / 7.3 us; 14B shape, 32 sequences of 5 parts each, 4.9 / 9.9 / 14.2 us.
// (With the loads of a batch behind conditions and one fold per part the first took 13 to 20 us.)
template <int D, typename OutT, int PW>
__global__ __launch_bounds__(PW == 1 ? 256 : 64 * PW) void attn_combine_kernel(AttnParams p) {
    constexpr int kTpc = D / 8;                   // lanes per column
    constexpr int kColsPerWave = 64 / kTpc;
    constexpr int kColWaves = PW == 1 ? 4 : 1;    // waves of the work-group with columns of their own
    constexpr int kBatch = PW == 1 ? 4 : 8;       // parts in flight per wave
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kvh = blockIdx.x % p.Hkv;  // blockIdx.x = sequence * Hkv + KV head
    const int4 cut = *reinterpret_cast<const int4 *>(p.cuts + 4 * (int64_t)blockIdx.x);
    const bool dense = p.error_flag[1] != 0;  // every part owns tiles
    const bool poison = blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && p.error_flag[0] != 0;
    const int r_first = cut.x, r_last = cut.y;
    const int R = cut.w, M = p.G * R;
    if (r_first != r_last) {  // block-uniform (equal: one wave saw the whole sequence and wrote it, or no tiles)
        Split sp{};
        if (!dense) sp = make_split(p, p.tile_prefix[p.B]);
        const int sub = kvh % p.HI;
        const int n = (blockIdx.y * kColWaves + (PW == 1 ? wave : 0)) * kColsPerWave + lane / kTpc;
        const int d8 = (lane % kTpc) * 8;
        const int nc = max(0, min(n, M - 1));  // lanes past the last column read it again and write nothing
        // partials in key order: slot 2*u+1 of the first part's wave u, then slot 2*u of the later
        // ones; when there are fewer tiles than parts some own no tile and wrote nothing.  The
        // loads of a batch carry no condition, so that they are in flight together; what a batch
        // reads past the slice, or of a part without tiles, gets weight zero.
        const int per = (r_last - r_first + PW) / PW;  // parts of a slice
        const int r0 = r_first + (PW == 1 ? 0 : wave * per), r1 = min(r0 + per, r_last + 1);
        float mt = -INFINITY, lt = 0.f;
        floatx4 o = {0.f, 0.f, 0.f, 0.f}, o2 = {0.f, 0.f, 0.f, 0.f};
        for (int rb = r0; rb < r1; rb += kBatch) {
            floatx4 stats[kBatch];
            u32x4 q[kBatch];
            bool have[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int r = min(rb + j, r1 - 1);
                const int w = r * p.HI + sub;
                const int64_t row = (int64_t)(r == r_first ? 2 * w + 1 : 2 * w) * p.Mpad + nc;
                stats[j] = *reinterpret_cast<const floatx4 *>(p.ws_ml + row * 4);
                q[j] = *reinterpret_cast<const u32x4 *>(p.ws_o + row * D + d8);
                have[j] = rb + j < r1 && (dense || part_owns_tiles(sp, r));
            }
            float mnew = mt;
#pragma unroll
            for (int j = 0; j < kBatch; ++j) mnew = fmaxf(mnew, have[j] ? stats[j][0] : -INFINITY);
            const float msafe = mnew == -INFINITY ? 0.f : mnew;
            const float keep = exp2f(mt - msafe);
            lt *= keep;
            o *= keep;
            o2 *= keep;
            mt = mnew;
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const float wgt = have[j] ? exp2f(stats[j][0] - msafe) : 0.f;
                const float unit = have[j] ? stats[j][2] * (1.f / 32767.f) * wgt : 0.f;
                const floatx4 x = {(float)(int16_t)(q[j][0] & 0xffffu), (float)(int16_t)(q[j][0] >> 16),
                                   (float)(int16_t)(q[j][1] & 0xffffu), (float)(int16_t)(q[j][1] >> 16)};
                const floatx4 x2 = {(float)(int16_t)(q[j][2] & 0xffffu), (float)(int16_t)(q[j][2] >> 16),
                                    (float)(int16_t)(q[j][3] & 0xffffu), (float)(int16_t)(q[j][3] >> 16)};
                lt += have[j] ? stats[j][1] * wgt : 0.f;
                o = o + x * unit;
                o2 = o2 + x2 * unit;
            }
        }
        if constexpr (PW > 1) {
            __shared__ floatx4 sh_o[PW][2][64];
            __shared__ floatx2 sh_ml[PW][64];
            sh_o[wave][0][lane] = o;
            sh_o[wave][1][lane] = o2;
            sh_ml[wave][lane] = floatx2{mt, lt};
            __syncthreads();
            if (wave == 0) {
                floatx2 ml[PW];
                float mall = -INFINITY;
#pragma unroll
                for (int w = 0; w < PW; ++w) {
                    ml[w] = sh_ml[w][lane];
                    mall = fmaxf(mall, ml[w][0]);
                }
                const float msafe = mall == -INFINITY ? 0.f : mall;
                lt = 0.f;
                o = o2 = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < PW; ++w) {
                    const float wgt = exp2f(ml[w][0] - msafe);
                    lt += ml[w][1] * wgt;
                    o = o + sh_o[w][0][lane] * wgt;
                    o2 = o2 + sh_o[w][1][lane] * wgt;
                }
                mt = mall;
            }
        }
        if (n < M && (PW == 1 || wave == 0)) {
            const int i = n / p.G, gh = n % p.G;
            const float inv = lt > 0.f ? 1.f / lt : 0.f;
            const int64_t orow = (int64_t)(cut.z + i) * p.Hq + kvh * p.G + gh;
            OutT *dst = static_cast<OutT *>(p.out) + orow * D + d8;
            const bf16x2 a = __builtin_convertvector(floatx2{o[0] * inv, o[1] * inv}, bf16x2);
            const bf16x2 c2 = __builtin_convertvector(floatx2{o[2] * inv, o[3] * inv}, bf16x2);
            const bf16x2 a2 = __builtin_convertvector(floatx2{o2[0] * inv, o2[1] * inv}, bf16x2);
            const bf16x2 c4 = __builtin_convertvector(floatx2{o2[2] * inv, o2[3] * inv}, bf16x2);
            *reinterpret_cast<u32x4 *>(dst) =
                u32x4{__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, c2),
                      __builtin_bit_cast(uint32_t, a2), __builtin_bit_cast(uint32_t, c4)};
            if (p.lse && d8 == 0)
                p.lse[orow] = lt > 0.f ? (mt + log2f(lt)) * 0.6931471805599453f : -INFINITY;
        }
    }
    if (poison) {
        // a wave of the main kernel gave up waiting for its partner: the results cannot be
        // trusted, so make that impossible to miss (this thread's own row was written above)
        static_cast<OutT *>(p.out)[0] = (OutT)0x7fc0;
        if (p.lse) p.lse[0] = NAN;
    }
}

// ------------------------------------------------------------------------------------------
// commit of the accepted tokens in a paged cache
// ------------------------------------------------------------------------------------------
struct CommitParams {
    void *k;
    void *v;
    const int32_t *q_indptr;
    const int32_t *page_indptr;
    const int32_t *page_table;
    int32_t *kv_len;
    const int32_t *path;          // [B, path_stride] rows of the accepted nodes, or NULL (chain: 1..n)
    const int32_t *num_accepted;
    int32_t B, total_q, max_q, path_stride;
    int32_t num_pages, table_len, page_size, page_shift;
    int32_t token_bytes;          // Hkv * D * sizeof(element), a multiple of 16
};

// One work-group per sequence.  The new tokens sit at positions first_new + row; the K/V of
// accepted node j (row path[j] >= j + 1) moves to position first_new + 1 + j, in ascending j,
// and the length becomes first_new + 1 + n.  A thread always handles the same 16-byte pieces
// of a token, and a later move never reads what an earlier one wrote over (rows increase along
// the path), so program order within the thread is all the ordering the moves need.
__global__ __launch_bounds__(256) void commit_accepted_kernel(CommitParams p) {
    const int b = blockIdx.x;
    const int q0 = max(0, min(p.q_indptr[b], p.total_q));
    const int R = max(0, min(p.q_indptr[b + 1] - q0, min(p.max_q, p.total_q - q0)));
    int e0 = p.page_indptr[b];
    int pages = p.page_indptr[b + 1] - e0;
    e0 = max(0, min(e0, p.table_len));
    pages = max(0, min(pages, p.table_len - e0));
    const int64_t cap = (int64_t)pages << p.page_shift;
    // The length is read once, by the thread that overwrites it at the end, and handed to the
    // others through LDS: a wave that starts late must not see the new length in its place.
    __shared__ int sh_len;
    if (threadIdx.x == 0) sh_len = p.kv_len[b];
    __syncthreads();
    const int64_t L = max((int64_t)0, min((int64_t)sh_len, cap));
    if (R < 1 || L < R) return;  // nothing that could be committed: the length stays (block-uniform)
    const int first_new = (int)(L - R);
    int n = max(0, min(p.num_accepted[b], R - 1));
    if (p.path) n = min(n, p.path_stride);
    const int pieces = p.token_bytes / 16;
    auto slot = [&](int pos) __attribute__((always_inline)) -> int64_t {  // byte offset of a token's K or V
        const int64_t pg = max(0, min(p.page_table[e0 + (pos >> p.page_shift)], p.num_pages - 1));
        return ((pg << p.page_shift) + (pos & (p.page_size - 1))) * (int64_t)p.token_bytes;
    };
    int done = 0;
    for (int j = 0; j < n; ++j) {
        const int r = p.path ? p.path[(int64_t)b * p.path_stride + j] : j + 1;
        if (r < j + 1 || r >= R) break;  // not a path: keep what has been committed so far
        done = j + 1;
        if (r == j + 1) continue;        // already in place
        const int64_t src = slot(first_new + r), dst = slot(first_new + 1 + j);
        for (int i = threadIdx.x; i < pieces; i += blockDim.x) {
            const u32x4 a = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.k) + src + (int64_t)i * 16);
            const u32x4 c = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.v) + src + (int64_t)i * 16);
            *reinterpret_cast<u32x4 *>(static_cast<char *>(p.k) + dst + (int64_t)i * 16) = a;
            *reinterpret_cast<u32x4 *>(static_cast<char *>(p.v) + dst + (int64_t)i * 16) = c;
        }
    }
    if (threadIdx.x == 0) p.kv_len[b] = first_new + 1 + done;
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
thread_local hipEvent_t g_mark_before_main = nullptr;
thread_local hipEvent_t g_mark_after_main = nullptr;

struct Plan {
    int32_t Mpad;
    size_t ws_o_bytes, ws_ml_bytes, prefix_bytes, start_bytes, flag_bytes, cut_bytes, ws_bytes;
};

bool make_plan(int32_t B, int64_t total_kv, int32_t max_q, int32_t max_kv_len, int32_t Hq,
               int32_t Hkv, int32_t D, respec_dtype_t dt, Plan &pl, int max_waves = kMaxWaves) {
    if (B <= 0 || total_kv <= 0 || max_q <= 0 || max_kv_len <= 0 || Hq <= 0 || Hkv <= 0) return false;
    if (Hq % Hkv != 0 || (D != 64 && D != 128)) return false;
    if (dt != RESPEC_F32 && dt != RESPEC_BF16) return false;
    const int32_t G = Hq / Hkv;
    if ((int64_t)G * max_q > 256) return false;
    pl.Mpad = (G * max_q + kColTile - 1) / kColTile * kColTile;
    // sized for the widest split so that the query needs no device
    pl.ws_o_bytes = round_up((size_t)2 * max_waves * pl.Mpad * D * sizeof(int16_t), 256);
    pl.ws_ml_bytes = round_up((size_t)2 * max_waves * pl.Mpad * 4 * sizeof(float), 256);
    pl.prefix_bytes = round_up((size_t)(B + 1) * sizeof(int32_t), 256);
    pl.start_bytes = round_up((size_t)max_waves * sizeof(WaveStart), 256);
    pl.flag_bytes = 256;
    pl.cut_bytes = round_up((size_t)B * Hkv * 4 * sizeof(int32_t), 256);
    pl.ws_bytes = pl.ws_o_bytes + pl.ws_ml_bytes + pl.prefix_bytes + pl.start_bytes + pl.flag_bytes + pl.cut_bytes;
    return true;
}

// Compute units of the current device (cached per device).
int compute_units() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

// One launch of a form of the main kernel (Form: its LDS).
template <auto kernel, typename Form>
hipError_t launch_bf16(const AttnParams &p, dim3 grid, int waves, hipStream_t stream) {
    static bool configured[64] = {false};  // per kernel and device; benign race: the attribute is idempotent
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
    if (dev < 0 || !configured[dev]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, Form::kBytes);
        if (e != hipSuccess) return e;
        if (dev >= 0) configured[dev] = true;
    }
    hipLaunchKernelGGL(kernel, grid, dim3(waves * 64), Form::kBytes, stream, p);
    return hipGetLastError();
}

// The combine kernel's form (see there), by the parts that the longest sequence's heads have: the
// average, times how much longer than the average the longest can be (at most twice that is
// counted: the bound is the caller's and may be the model's).  Sharing them between waves wins from
// 16 parts on (7.5 -> 4.3 us) and loses at 8 (5.5 -> 6.8 us); eight waves win over four from 64 on
// (5.9 -> 5.2 us).  most: parts that a sequence can have (the form for few tiles gives four tiles to a
// part); forced: 1, 4 or 8 (RESPEC_ATTN_COMBINE), 0 = by this rule.
template <int D>
hipError_t launch_combine(const AttnParams &p, int M, int64_t kv_tokens, double most, long forced, hipStream_t stream) {
    const int cols_per_wave = 64 / (D / 8);
    const int64_t pairs = (int64_t)p.B * p.Hkv;
    const int groups = (M + cols_per_wave - 1) / cols_per_wave;
    const double longest = std::fmin(2.0, std::fmax(1.0, (double)p.max_kv_len * p.B / (double)kv_tokens));
    const double parts = std::fmin((double)p.W / (double)pairs * longest, most);
    const long pw = forced == 1 || forced == 4 || forced == 8 ? forced : parts >= 64.0 ? 8 : parts >= 12.0 ? 4 : 1;
    if (pw == 8)
        hipLaunchKernelGGL((attn_combine_kernel<D, uint16_t, 8>), dim3((unsigned)pairs, (unsigned)groups), dim3(512), 0, stream, p);
    else if (pw == 4)
        hipLaunchKernelGGL((attn_combine_kernel<D, uint16_t, 4>), dim3((unsigned)pairs, (unsigned)groups), dim3(256), 0, stream, p);
    else
        hipLaunchKernelGGL((attn_combine_kernel<D, uint16_t, 1>), dim3((unsigned)pairs, (unsigned)((groups + 3) / 4)), dim3(256), 0, stream, p);
    return hipGetLastError();
}

// nt: column tiles of a column block; cw: consumers that share a range; nc: consumers of a work-group
template <int D>
hipError_t launch_bf16_nt(int nt, int cw, int nc, const AttnParams &p, dim3 grid, hipStream_t stream) {
#define RESPEC_FORM(NT, CW) launch_bf16<&attn_bf16_kernel<D, NT, uint16_t, CW>, Bf16Form<D, NT, consumers_of(CW)>>(p, grid, consumers_of(CW) + kProducers, stream)
    if (cw == 4 && nc == 4) return launch_bf16<&attn_bf16_small_kernel<D, uint16_t>, Bf16Form<D, 1, 4>>(p, grid, 4 + kProducers, stream);
    if (cw == 4) return nt <= 4 ? RESPEC_FORM(1, 4) : RESPEC_FORM(2, 4);
    if (cw == 2) return nt <= 2 ? RESPEC_FORM(1, 2) : RESPEC_FORM(2, 2);
    if constexpr (D == 128)
        if (nt == 3) return RESPEC_FORM(3, 1);
    return RESPEC_FORM(1, 1);
}

template <int D>
hipError_t launch_few(int nt, const AttnParams &p, hipStream_t stream) {
    const dim3 grid((unsigned)(p.W / p.Hkv), (unsigned)p.Hkv);
#define RESPEC_FEW(NT) launch_bf16<&attn_bf16_few_kernel<D, NT>, FewForm<D, NT>>(p, grid, kFewWaves, stream)
    return nt == 1 ? RESPEC_FEW(1) : nt == 2 ? RESPEC_FEW(2) : nt == 3 ? RESPEC_FEW(3) : RESPEC_FEW(4);
}

// Work-groups per compute unit that a batch gets in the form for few tiles (attn_bf16_few_kernel), 0 where
// the main kernel's forms are the better ones.  What counts is how many tiles its largest part has, on
// work-groups in number one or two per compute unit: the longest sequence's, or what the split leaves
// (which gets coarse where there are nearly as many pairs as work-groups).  Lines, from a sweep over
// 1 to 64 sequences of 40 to 250, 512 to 4096 and 2000 to 8192 tokens at the 3B, 7B and 14B shapes and with
// heads of 64, one to four column tiles (us per call: main kernel's forms / one / two per unit, at the
// tiles of the largest part with one): one column tile: 7B shape 11 18.3, 15.1, 14.8; 24 22.9, 23.1, 21.4;
// 41 31.6, 34.2, 30.8; 74 43.6, 75.0, 44.8; two: 3B 19 27.0, 20.1, 22.1; 51 40.8, 36.3, 35.0; 126 77.4, 76.5, 69.8;
// 7B 46 38.8, 35.0, 32.3; 128 64.6, 83.4, 65.8; three and four: 7B 46 42.0, 36.8, 39.3; 82 59.9, 59.2, 60.5; 128
// 69.4, 85.9, 69.5; heads of 64, two tiles: 15 18.1, 13.7, 12.8; 126 42.0, 44.0, 37.7.  With eight KV heads a
// part reads an eighth of every cache row, and the lines lie lower: 14B, one tile 15 19.5, 18.7, 18.0; 24 22.0,
// 22.5, 23.6; two 48 43.3, 40.0, 41.2; 96 60.2, 61.7, 63.7; three 48 46.0, 41.6, 46.1; 59 47.8, 49.7, 46.2.
// The upper line of two per unit (48 tiles) is the 7B shape's; with two KV heads two per unit still win at 126 (the
// 3B and the heads of 64 above), which the line leaves to the main kernel.
int few_tiles_groups(int D, int nt, int32_t B, int32_t Hkv, int64_t kv_tokens, int32_t max_kv_len) {
    const int units = compute_units();
    if (B > kFewSeqs || (int64_t)B * Hkv > units) return 0;
    const double tiles = (double)kv_tokens / kTileKeys + B;  // of one KV head, about
    const double longest = ((double)max_kv_len + kTileKeys - 1) / kTileKeys;
    auto largest_part = [&](int groups) {
        const double seats = (double)(units * groups / Hkv) - 0.6 * B;
        return std::fmin(longest, tiles / std::fmax(seats, 1e-3));
    };
    const bool many_heads = Hkv >= 8;
    if (D == 64 || nt <= 2) {  // two fit a compute unit
        const double two_from = D == 64 ? (nt <= 2 ? 12 : 26) : nt == 1 ? 13 : 34;
        const double most = nt == 1 ? (many_heads ? 8 : D == 64 ? 48 : 20) : many_heads ? 28 : 48;
        if (largest_part(1) < two_from) return 1;
        return largest_part(2) <= most ? 2 : 0;
    }
    return largest_part(1) <= (many_heads ? 56 : 84) ? 1 : 0;
}

}  // namespace
}  // namespace respec

extern "C" {

void respec_profile_mark_main(void *before_main, void *after_main) {
    respec::g_mark_before_main = static_cast<hipEvent_t>(before_main);
    respec::g_mark_after_main = static_cast<hipEvent_t>(after_main);
}

size_t respec_verify_attention_workspace_bytes(int32_t B, int32_t total_q, int64_t total_kv,
                                               int32_t max_q_per_seq, int32_t max_kv_len,
                                               int32_t Hq, int32_t Hkv, int32_t D,
                                               respec_dtype_t dt) {
    respec::Plan pl;
    (void)total_q;
    if (!respec::make_plan(B, total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, dt, pl)) return 0;
    return pl.ws_bytes;
}

}  // extern "C"

namespace respec {
namespace {

// The page table of a paged cache (all NULL / 0 for the contiguous layout).
struct Pages {
    const int32_t *page_indptr;
    const int32_t *page_table;
    const int32_t *kv_len;
    int32_t num_pages, table_len, page_size;
};

int page_shift_of(int32_t page_size) {  // log2 of a supported page size, -1 otherwise
    for (int s = 4; s <= 10; ++s)
        if (page_size == (1 << s)) return s;
    return -1;
}

respec_status_t verify_attention_any(const void *q, const void *k_cache, const void *v_cache,
                                     const int32_t *q_indptr, const int64_t *kv_indptr, const Pages &pg,
                                     const uint64_t *tree_mask, void *out, float *lse, int32_t B,
                                     int32_t total_q, int64_t total_kv, int32_t max_q_per_seq,
                                     int32_t max_kv_len, int32_t Hq, int32_t Hkv, int32_t D, float sm_scale,
                                     respec_dtype_t dt, void *workspace, size_t workspace_bytes,
                                     void *hip_stream, bool reuse_plan = false, int max_waves = kMaxWaves) {
    const bool paged = pg.page_table != nullptr;
    if (tree_mask && max_q_per_seq > 64)
        return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention_tree: at most 64 rows per sequence, got %d",
                    max_q_per_seq);
    if (paged) {
        if (!pg.page_indptr || !pg.kv_len)
            return fail(RESPEC_ERR_INVALID_ARG, "verify_attention_paged: null pointer argument");
        if (pg.num_pages < 1 || pg.table_len < 1)
            return fail(RESPEC_ERR_INVALID_ARG, "verify_attention_paged: need num_pages >= 1 and page_table_len >= 1");
        if (page_shift_of(pg.page_size) < 0)
            return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention_paged: page size %d is not a power of two in [16, 1024]",
                        pg.page_size);
        total_kv = (int64_t)pg.num_pages * pg.page_size;
    } else if (!kv_indptr) {
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: null pointer argument");
    }
    if (B <= 0 || total_q < B || total_kv < (paged ? 1 : total_q) || max_q_per_seq < 1 || max_kv_len < 1)
        return fail(RESPEC_ERR_INVALID_ARG,
                    "verify_attention: need B > 0, total_q >= B, total_kv >= total_q, max_q_per_seq >= 1, "
                    "max_kv_len >= 1 (B=%d total_q=%d total_kv=%lld)", B, total_q, (long long)total_kv);
    if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0)
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: Hq=%d must be a positive multiple of Hkv=%d", Hq, Hkv);
    if (dt != RESPEC_F32 && dt != RESPEC_BF16)
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: unknown dtype %d", (int)dt);
    if (!std::isfinite(sm_scale))
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: sm_scale must be finite");
    if (D != 64 && D != 128)
        return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention: head size %d not in {64,128}", D);
    if ((int64_t)(Hq / Hkv) * max_q_per_seq > 256)
        return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention: G*max_q_per_seq = %lld exceeds 256",
                    (long long)(Hq / Hkv) * max_q_per_seq);
    if ((int64_t)B * max_q_per_seq < total_q)
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: max_q_per_seq too small for total_q");
    if (!q || !k_cache || !v_cache || !q_indptr || !out)
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: null pointer argument");
    if (!aligned_to(q, 16) || !aligned_to(k_cache, 16) || !aligned_to(v_cache, 16) || !aligned_to(out, 16))
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: q, k_cache, v_cache and out must be 16-byte aligned");
    Plan pl;
    if (!make_plan(B, total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, dt, pl, max_waves))
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention: could not plan the launch");
    if (!workspace || workspace_bytes < pl.ws_bytes || !aligned_to(workspace, 256))
        return fail(RESPEC_ERR_WORKSPACE, "verify_attention: workspace of %zu bytes (256-byte aligned) needed, got %zu",
                    pl.ws_bytes, workspace ? workspace_bytes : (size_t)0);
    if ((int64_t)B * Hkv > 0x0fffffffLL)
        return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention: B*Hkv exceeds 2^28-1");
    if ((int64_t)total_q * Hq > 0x7fffffffLL)
        return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention: total_q*Hq exceeds 2^31-1");
    if (dt == RESPEC_F32 && (int64_t)B * Hq > 0x7fffffffLL)
        return fail(RESPEC_ERR_UNSUPPORTED, "verify_attention: B*Hq too large for the fp32 path");

    AttnParams p{};
    p.q = q;
    p.k = k_cache;
    p.v = v_cache;
    p.q_indptr = q_indptr;
    p.kv_indptr = kv_indptr;
    p.tree_mask = tree_mask;
    p.page_table = pg.page_table;
    p.page_indptr = pg.page_indptr;
    p.kv_len = pg.kv_len;
    p.num_pages = pg.num_pages;
    p.table_len = pg.table_len;
    p.page_size = paged ? pg.page_size : 0;
    p.page_shift = paged ? page_shift_of(pg.page_size) : 0;
    p.out = out;
    p.lse = lse;
    char *ws = static_cast<char *>(workspace);
    p.ws_o = reinterpret_cast<int16_t *>(ws);
    p.ws_ml = reinterpret_cast<float *>(ws + pl.ws_o_bytes);
    p.tile_prefix = reinterpret_cast<int32_t *>(ws + pl.ws_o_bytes + pl.ws_ml_bytes);
    p.wave_start = reinterpret_cast<WaveStart *>(ws + pl.ws_o_bytes + pl.ws_ml_bytes + pl.prefix_bytes);
    p.error_flag = reinterpret_cast<int32_t *>(ws + pl.ws_o_bytes + pl.ws_ml_bytes + pl.prefix_bytes + pl.start_bytes);
    p.cuts = p.error_flag + pl.flag_bytes / sizeof(int32_t);
    p.B = B;
    p.total_q = total_q;
    p.total_kv = total_kv;
    p.max_q = max_q_per_seq;
    p.max_kv_len = max_kv_len;
    p.Hq = Hq;
    p.Hkv = Hkv;
    p.G = Hq / Hkv;
    p.g_inverse = (65536u + (uint32_t)p.G - 1) / (uint32_t)p.G;
    p.Mpad = pl.Mpad;
    p.scale2 = (float)((double)sm_scale * 1.4426950408889634074);
    // (a scale of zero becomes 1e-37: every exponent rounds to the one it has at zero, and a hidden
    // key's -inf stays -inf when it is scaled)
    p.scale_abs = std::fmax(std::fabs(p.scale2), 1e-37f);
    p.q_sign = p.scale2 < 0.f ? 0x80008000u : 0u;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    hipError_t err;
    const int M = p.G * max_q_per_seq;
    if (dt == RESPEC_F32) {
        if (g_mark_before_main) {
            (void)hipEventRecord(g_mark_before_main, stream);
            g_mark_before_main = nullptr;
        }
        const dim3 grid((unsigned)(B * Hq), (unsigned)max_q_per_seq);
        if (D == 128)
            hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(kF32Threads), 0, stream, p);
        else
            hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(kF32Threads), 0, stream, p);
        err = hipGetLastError();
        if (err != hipSuccess)
            return fail(RESPEC_ERR_HIP, "verify_attention: launch failed: %s", hipGetErrorString(err));
        if (g_mark_after_main) {
            (void)hipEventRecord(g_mark_after_main, stream);
            g_mark_after_main = nullptr;
        }
        clear_error();
        return RESPEC_OK;
    }

    // The form of the main kernel: consumers that share a range (cw, each with its own column
    // tiles), consumers of a work-group (nc) and, from them, the split.  Times are us per call, main and
    // combine kernel, medians over calls in turn (lengths 512 to 4096; they scatter by 1-2 %); "tiles"
    // are those per consumer of the device.
    // One column tile: a range per consumer; bound by HBM.
    // Two tiles: two consumers per range, eight per work-group (two per SIMD hide each other's dependent
    // phases; one consumer per range with both tiles / two): B = 8, 64, 256, 512 at the 7B shape, k = 3,
    // 31.1 / 25.0, 67.2 / 63.7, 219 / 217, 405 / 405; B = 512 at the 14B shape, k = 4, 785 / 782; B = 768 at the
    // 3B shape, k = 3, 318 / 312, and with heads of 64 167 / 163.  With fewer than two tiles four
    // consumers of one tile each share a range, four per work-group: a quarter of the ranges and of the
    // partials to fold (two consumers / four: 24.8 / 23.4 at B = 6, 21.8 / 18.2 at B = 2, 7B; 19.5 / 18.1 at
    // B = 8, 3B with heads of 64; from two tiles on 28.1 / 28.9 at B = 12, 7B; 29.7 / 32.0 at B = 32, 3B).
    // (Most batches that small take the form for few tiles, few_tiles_groups: what comes here has more than
    // 64 sequences, or more pairs of a sequence and a KV head than compute units.)
    // Three and four tiles: four consumers per range, eight per work-group (one, two and four consumers
    // per range: k = 4, B = 256 and 768 at the 3B shape 135, 133, 124 and 336, 331, 318; k = 5, B = 256 at the
    // 7B shape 239, 237, 233; k = 7, B = 64 at the 14B shape 125, 121, 117).  But that form's two ranges
    // read two neighbouring heads of a cache row at a time where the others read four, which shows with
    // eight KV heads or more and a batch that HBM bounds.  Heads of 64 from 32 tiles on (19 tiles 48.6, 48.1
    // with two and four, 34 tiles 72.0, 73.7, 146 tiles 235, 250; one, two and four, 45 columns, 146 tiles
    // 234, 232, 246; with two KV heads, 109 tiles, 178, 174, 171).  Heads of 128 from 64 on (14B shape; k = 7:
    // 52 tiles 179, 176, 171, 71 tiles 226, 224, 224, 288 tiles 806, 815, 824; k = 10: 34 tiles -, 126, 122,
    // 71 tiles -, 227, 230, 146 tiles -, 437, 443): three tiles then in one consumer, four in two.
    // More than 64 columns: blocks of 128, four consumers of 32 columns per range, K and V read once
    // per block (91 columns, B = 256 at the 7B shape: 272 us against 380 us with four consumers per
    // work-group and the longer loop).
    // (cached tokens: the host-side total, for a paged cache what its page-table entries can hold, in
    // either case no more than the longest length allows: a table with room to grow takes the form of the
    // tokens it may hold, not of its room)
    const Knobs kn = knobs();
    const int64_t kv_tokens = std::min(paged ? (int64_t)pg.table_len * pg.page_size : total_kv, (int64_t)B * max_kv_len);
    const int64_t tiles = (kv_tokens / kTileKeys + B) * (int64_t)Hkv;  // of all (head, sequence) pairs, about
    const int64_t tiles_per_consumer = tiles / ((int64_t)kProducers * compute_units());
    const long quad_env = kn.get(&Knobs::attn_quad, 1);  // 0: never, 2: always four consumers per range
    const long wide = kn.get(&Knobs::attn_wide, -1);     // 0 / 1: one (three tiles, D = 128) / two consumers per range up to 64 columns
    const bool quad = M > kMaxColsPerBlock && quad_env != 0;
    const int block_cols = quad ? 2 * kMaxColsPerBlock : kMaxColsPerBlock;
    const int col_blocks = (M + block_cols - 1) / block_cols;
    const int cols = col_blocks == 1 ? M : kMaxColsPerBlock;
    const int nt = quad ? 8 : (cols + kColTile - 1) / kColTile;  // column tiles of a block
    const bool many_heads = Hkv >= 8 && tiles_per_consumer >= (D == 64 ? 32 : 64);
    const bool one = nt == 1 || (nt == 3 && D == 128 && wide != 1 && (wide == 0 || many_heads));
    int cw;
    if (quad || (quad_env == 2 && nt >= 2 && M <= kMaxColsPerBlock)) cw = 4;
    else if (one) cw = 1;
    else if (wide >= 0 || quad_env == 0 || M > kMaxColsPerBlock) cw = 2;
    else if (nt == 2) cw = tiles_per_consumer < 2 ? 4 : 2;
    else cw = many_heads ? 2 : 4;
    const long nc_env = kn.get(&Knobs::attn_consumers, 0);  // 4 / 8: the narrow four-way form's consumers
    const int nc = cw == 1 ? 4 : cw == 4 && nt <= 4 && (nc_env ? nc_env == 4 : tiles_per_consumer < 2) ? 4 : 8;
    const int streams = nc / cw;  // ranges per work-group
    // the split width: one range per consumer (or group of consumers) of the device
    // (RESPEC_ATTN_WGS overrides it, for tests and sweeps)
    // A tiny batch gets no more ranges than it can have tiles, were all sequences as long as the longest
    // may be (a bound that the contiguous and the paged entry point share): ranges without a tile cost
    // their launch, and every part the combine kernel walks.  us per call at the 3B shape with as many
    // ranges as the device takes (1024 at k = 0, 256 at k = 4), with as many as tiles, and with half as
    // many: 4 sequences of 8 to 64 tokens, k = 0 15.2, 12.1, 14.2, k = 4 14.7, 13.5, 17.1; 48 of 8 to 32
    // tokens, k = 4 11.8, 11.9, 15.6 (a second tile in a range is a second sequence there); one of 60 to
    // 70 tokens, k = 0 20.5, 11.1, 11.5.  Half as many are better where each range is one whole sequence,
    // which no bound tells: 4 of 33 to 64 tokens, k = 0 15.0, 12.2, 10.9, k = 4 14.8, 13.2, 11.8.
    // Where sequences may have more than 16 tiles a range gets two tiles at least: the partials that the combine kernel folds
    // halve with the ranges, a second tile of the same sequence takes 0.5 us, and few ranges cross from
    // one sequence to the next (2 sequences of 2300 tokens: k = 0 at the 3B shape 21.7 us per call with
    // 1024 ranges, 16.3 us with 128; k = 6, 4 query heads of 64, 17.0 us with 256, 14.6 with 128).
    // Between 512 and 2048 tokens the two are even on the whole, by how the ends of the ranges meet those
    // of the sequences (k = 4, 3B shape, one tile / two: 2 of 300 to 512 tokens 15.5 / 19.4; 2 of 512 to 1024
    // 17.7 / 15.7, of 1024 to 2048 19.2 / 15.8; 4 of 520 15.4 / 20.1, of 512 to 1024 17.4 / 18.4)
    long W = kn.get(&Knobs::attn_wgs, 0);
    if (W <= 0) {
        W = (long)streams * compute_units() / col_blocks;
        const int64_t longest = ((int64_t)max_kv_len + kTileKeys - 1) / kTileKeys;  // (a caller without a bound passes the largest int32)
        const int per = longest > 16 ? 2 : 1;
        const int64_t most = ((int64_t)B * longest * Hkv + per - 1) / per;
        if (W > most) W = (long)((most + streams - 1) / streams * streams);
    }
    // (a knob that shapes the main kernel keeps to it)
    const long few_env = kn.get(&Knobs::attn_few, -1);  // 0: never, 1 / 2: that many work-groups per compute unit wherever the form takes the batch
    int few = 0;
    if (M <= kMaxColsPerBlock && B <= kFewSeqs && (int64_t)B * Hkv <= compute_units()) {
        if (few_env >= 0) few = (int)std::min(few_env, 2l);
        else if (kn.get(&Knobs::attn_wgs, 0) <= 0 && quad_env == 1 && wide < 0 && nc_env == 0 && kn.get(&Knobs::attn_head_major, 0) == 0 &&
                 kn.get(&Knobs::attn_inline, 1) != 0)
            few = few_tiles_groups(D, nt, B, Hkv, kv_tokens, max_kv_len);
    }
    if (few) W = (long)compute_units() * few / Hkv * Hkv;
    if (W < 1) W = 1;
    if (W > max_waves) W = max_waves;
    p.W = (int32_t)W;
    int hi = Hkv % 4 == 0 ? 4 : (Hkv % 2 == 0 ? 2 : 1);
    if (hi > streams) hi = streams;
    if (W % hi != 0 || kn.get(&Knobs::attn_head_major, 0) != 0) hi = 1;
    p.HI = few ? Hkv : hi;  // (the few-tiles form: work-group part * Hkv + head)

    // the set-up depends on the index arrays and the sizes only: the layers of one forward share
    // it (reuse_plan: the workspace still holds what the set-up of an earlier call left there)
    // (small batches: the main kernel's work-groups build it in their prologue and leave it in
    // the workspace; large ones take a set-up kernel in front)
    p.inline_setup = !reuse_plan && B <= kInlineSeqs && (few || kn.get(&Knobs::attn_inline, 1) != 0) ? 1 : 0;
    if (!reuse_plan && !p.inline_setup) {
        hipLaunchKernelGGL(attn_prep_kernel, dim3(1), dim3(1024), 0, stream, p);
        err = hipGetLastError();
        if (err != hipSuccess)
            return fail(RESPEC_ERR_HIP, "verify_attention: prep launch failed: %s", hipGetErrorString(err));
    }
    if (g_mark_before_main) {
        (void)hipEventRecord(g_mark_before_main, stream);
        g_mark_before_main = nullptr;
    }
    const dim3 grid((unsigned)((W + streams - 1) / streams), (unsigned)col_blocks);
    if (few)
        err = D == 128 ? launch_few<128>(nt, p, stream) : launch_few<64>(nt, p, stream);
    else
        err = D == 128 ? launch_bf16_nt<128>(nt, cw, nc, p, grid, stream) : launch_bf16_nt<64>(nt, cw, nc, p, grid, stream);
    if (err != hipSuccess)
        return fail(RESPEC_ERR_HIP, "verify_attention: main launch failed: %s", hipGetErrorString(err));
    if (g_mark_after_main) {
        (void)hipEventRecord(g_mark_after_main, stream);
        g_mark_after_main = nullptr;
    }
    {
        const double most = few ? (double)max_kv_len / (4 * kTileKeys) + 1 : (double)kMaxWaves;
        err = D == 128 ? launch_combine<128>(p, M, kv_tokens, most, kn.get(&Knobs::attn_combine, 0), stream)
                       : launch_combine<64>(p, M, kv_tokens, most, kn.get(&Knobs::attn_combine, 0), stream);
        if (err != hipSuccess)
            return fail(RESPEC_ERR_HIP, "verify_attention: combine launch failed: %s", hipGetErrorString(err));
    }
    clear_error();
    return RESPEC_OK;
}

}  // namespace
}  // namespace respec

extern "C" {

respec_status_t respec_verify_attention(const void *q, const void *k_cache, const void *v_cache,
                                        const int32_t *q_indptr, const int64_t *kv_indptr,
                                        void *out, float *lse, int32_t B, int32_t total_q,
                                        int64_t total_kv, int32_t max_q_per_seq,
                                        int32_t max_kv_len, int32_t Hq, int32_t Hkv, int32_t D,
                                        float sm_scale, respec_dtype_t dt, void *workspace,
                                        size_t workspace_bytes, void *hip_stream) {
    return respec::verify_attention_any(q, k_cache, v_cache, q_indptr, kv_indptr, respec::Pages{}, nullptr, out, lse,
                                        B, total_q, total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, sm_scale, dt,
                                        workspace, workspace_bytes, hip_stream);
}

respec_status_t respec_verify_attention_next_layer(const void *q, const void *k_cache, const void *v_cache,
                                                   const int32_t *q_indptr, const int64_t *kv_indptr,
                                                   const uint64_t *tree_mask, void *out, float *lse, int32_t B,
                                                   int32_t total_q, int64_t total_kv, int32_t max_q_per_seq,
                                                   int32_t max_kv_len, int32_t Hq, int32_t Hkv, int32_t D,
                                                   float sm_scale, respec_dtype_t dt, void *workspace,
                                                   size_t workspace_bytes, void *hip_stream) {
    return respec::verify_attention_any(q, k_cache, v_cache, q_indptr, kv_indptr, respec::Pages{}, tree_mask, out,
                                        lse, B, total_q, total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, sm_scale,
                                        dt, workspace, workspace_bytes, hip_stream, true);
}

respec_status_t respec_verify_attention_tree(const void *q, const void *k_cache, const void *v_cache,
                                             const int32_t *q_indptr, const int64_t *kv_indptr,
                                             const uint64_t *tree_mask, void *out, float *lse, int32_t B,
                                             int32_t total_q, int64_t total_kv, int32_t max_q_per_seq,
                                             int32_t max_kv_len, int32_t Hq, int32_t Hkv, int32_t D,
                                             float sm_scale, respec_dtype_t dt, void *workspace,
                                             size_t workspace_bytes, void *hip_stream) {
    if (!tree_mask)
        return respec::fail(RESPEC_ERR_INVALID_ARG, "verify_attention_tree: null tree_mask");
    return respec::verify_attention_any(q, k_cache, v_cache, q_indptr, kv_indptr, respec::Pages{}, tree_mask, out,
                                        lse, B, total_q, total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, sm_scale,
                                        dt, workspace, workspace_bytes, hip_stream);
}

respec_status_t respec_verify_attention_paged(const void *q, const void *k_pages, const void *v_pages,
                                              const int32_t *q_indptr, const int32_t *page_indptr,
                                              const int32_t *page_table, const int32_t *kv_len,
                                              const uint64_t *tree_mask, void *out, float *lse, int32_t B,
                                              int32_t total_q, int32_t num_pages, int32_t page_table_len,
                                              int32_t page_size, int32_t max_q_per_seq, int32_t max_kv_len,
                                              int32_t Hq, int32_t Hkv, int32_t D, float sm_scale,
                                              respec_dtype_t dt, void *workspace, size_t workspace_bytes,
                                              void *hip_stream) {
    if (!page_table)
        return respec::fail(RESPEC_ERR_INVALID_ARG, "verify_attention_paged: null page_table");
    const respec::Pages pg{page_indptr, page_table, kv_len, num_pages, page_table_len, page_size};
    return respec::verify_attention_any(q, k_pages, v_pages, q_indptr, nullptr, pg, tree_mask, out, lse, B, total_q,
                                        0, max_q_per_seq, max_kv_len, Hq, Hkv, D, sm_scale, dt, workspace,
                                        workspace_bytes, hip_stream);
}

respec_status_t respec_verify_attention_paged_next_layer(const void *q, const void *k_pages, const void *v_pages,
                                                         const int32_t *q_indptr, const int32_t *page_indptr,
                                                         const int32_t *page_table, const int32_t *kv_len,
                                                         const uint64_t *tree_mask, void *out, float *lse,
                                                         int32_t B, int32_t total_q, int32_t num_pages,
                                                         int32_t page_table_len, int32_t page_size,
                                                         int32_t max_q_per_seq, int32_t max_kv_len, int32_t Hq,
                                                         int32_t Hkv, int32_t D, float sm_scale, respec_dtype_t dt,
                                                         void *workspace, size_t workspace_bytes,
                                                         void *hip_stream) {
    if (!page_table)
        return respec::fail(RESPEC_ERR_INVALID_ARG, "verify_attention_paged: null page_table");
    const respec::Pages pg{page_indptr, page_table, kv_len, num_pages, page_table_len, page_size};
    return respec::verify_attention_any(q, k_pages, v_pages, q_indptr, nullptr, pg, tree_mask, out, lse, B, total_q,
                                        0, max_q_per_seq, max_kv_len, Hq, Hkv, D, sm_scale, dt, workspace,
                                        workspace_bytes, hip_stream, true);
}

}  // extern "C"

namespace respec {
namespace {

constexpr int kStaticMaxWaves = 1024;  // split width the static scratch is sized for
constexpr int kMaxDevices = 64;

// Device address of `scratch` on the current device, looked up once per device (each GPU holds
// its own copy of the array at its own address).  Returns NULL and sets the error text on failure.
void *static_scratch_address() {
    static std::mutex mu;
    static void *addr[kMaxDevices] = {nullptr};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        fail(RESPEC_ERR_HIP, "static scratch: no usable current device (%s)", hipGetErrorString(e));
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            fail(RESPEC_ERR_HIP, "static scratch: hipGetSymbolAddress failed on device %d: %s", dev,
                 hipGetErrorString(e));
            return nullptr;
        }
        addr[dev] = ptr;
    }
    return addr[dev];
}

}  // namespace
}  // namespace respec

extern "C" {

size_t respec_static_scratch_bytes(void) { return kStaticScratchBytes; }

respec_status_t respec_static_scratch_init(void) {
    if (!respec::static_scratch_address()) return RESPEC_ERR_HIP;
    respec::clear_error();
    return RESPEC_OK;
}

respec_status_t respec_verify_attention_static(const void *q, const void *k_cache, const void *v_cache,
                                               const int32_t *q_indptr, const int64_t *kv_indptr, void *out,
                                               float *lse, int32_t B, int32_t total_q, int64_t total_kv,
                                               int32_t max_q_per_seq, int32_t max_kv_len, int32_t Hq,
                                               int32_t Hkv, int32_t D, float sm_scale, respec_dtype_t dt,
                                               void *hip_stream) {
    using namespace respec;
    Plan pl;
    if (!make_plan(B, total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, dt, pl, kStaticMaxWaves))
        return fail(RESPEC_ERR_INVALID_ARG, "verify_attention_static: sizes out of range (see respec_verify_attention)");
    if (pl.ws_bytes > kStaticScratchBytes)
        return fail(RESPEC_ERR_WORKSPACE,
                    "verify_attention_static: this batch needs %zu bytes of scratch, the built-in buffer holds %zu; "
                    "use respec_verify_attention with a workspace", pl.ws_bytes, kStaticScratchBytes);
    void *ws = static_scratch_address();
    if (!ws) return RESPEC_ERR_HIP;
    return verify_attention_any(q, k_cache, v_cache, q_indptr, kv_indptr, Pages{}, nullptr, out, lse, B, total_q,
                                total_kv, max_q_per_seq, max_kv_len, Hq, Hkv, D, sm_scale, dt, ws,
                                kStaticScratchBytes, hip_stream, false, kStaticMaxWaves);
}

respec_status_t respec_commit_accepted_paged(void *k_pages, void *v_pages, const int32_t *q_indptr,
                                             const int32_t *page_indptr, const int32_t *page_table,
                                             int32_t *kv_len, const int32_t *path, int32_t path_stride,
                                             const int32_t *num_accepted, int32_t B, int32_t total_q,
                                             int32_t max_q_per_seq, int32_t num_pages, int32_t page_table_len,
                                             int32_t page_size, int32_t Hkv, int32_t D, respec_dtype_t dt,
                                             void *hip_stream) {
    using namespace respec;
    if (!k_pages || !v_pages || !q_indptr || !page_indptr || !page_table || !kv_len || !num_accepted)
        return fail(RESPEC_ERR_INVALID_ARG, "commit_accepted_paged: null pointer argument");
    if (B <= 0 || total_q < B || max_q_per_seq < 1 || num_pages < 1 || page_table_len < 1 || Hkv <= 0 || D <= 0)
        return fail(RESPEC_ERR_INVALID_ARG, "commit_accepted_paged: sizes must be positive (B=%d total_q=%d)", B, total_q);
    if (path && path_stride < 1)
        return fail(RESPEC_ERR_INVALID_ARG, "commit_accepted_paged: path_stride must be >= 1 with a path");
    if (dt != RESPEC_F32 && dt != RESPEC_BF16)
        return fail(RESPEC_ERR_INVALID_ARG, "commit_accepted_paged: unknown dtype %d", (int)dt);
    const int shift = page_shift_of(page_size);
    if (shift < 0)
        return fail(RESPEC_ERR_UNSUPPORTED, "commit_accepted_paged: page size %d is not a power of two in [16, 1024]",
                    page_size);
    const int64_t token_bytes = (int64_t)Hkv * D * (dt == RESPEC_BF16 ? 2 : 4);
    if (token_bytes % 16 != 0 || token_bytes > 0x7fffffffLL)
        return fail(RESPEC_ERR_UNSUPPORTED, "commit_accepted_paged: Hkv*D*sizeof(element) must be a multiple of 16");
    if (!aligned_to(k_pages, 16) || !aligned_to(v_pages, 16))
        return fail(RESPEC_ERR_INVALID_ARG, "commit_accepted_paged: k_pages and v_pages must be 16-byte aligned");
    CommitParams p{};
    p.k = k_pages;
    p.v = v_pages;
    p.q_indptr = q_indptr;
    p.page_indptr = page_indptr;
    p.page_table = page_table;
    p.kv_len = kv_len;
    p.path = path;
    p.num_accepted = num_accepted;
    p.B = B;
    p.total_q = total_q;
    p.max_q = max_q_per_seq;
    p.path_stride = path_stride;
    p.num_pages = num_pages;
    p.table_len = page_table_len;
    p.page_size = page_size;
    p.page_shift = shift;
    p.token_bytes = (int32_t)token_bytes;
    hipLaunchKernelGGL(commit_accepted_kernel, dim3((unsigned)B), dim3(256), 0, static_cast<hipStream_t>(hip_stream), p);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess)
        return fail(RESPEC_ERR_HIP, "commit_accepted_paged: launch failed: %s", hipGetErrorString(err));
    clear_error();
    return RESPEC_OK;
}

}  // extern "C"
