// Internal declarations shared by the HIP translation units of libmp.
// Nothing here is part of the public ABI (include/mp.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "mp.h"
#include "mp_probe.h"

namespace mp {

constexpr int kWave = 64;

// ---- radix sort geometry (COO -> CSR) ---------------------------------------
#ifndef MP_SORT_BLOCK
#define MP_SORT_BLOCK 1024
#endif
#ifndef MP_SORT_ITEMS
#define MP_SORT_ITEMS 16
#endif
constexpr int kSortBlock = MP_SORT_BLOCK;          // threads per workgroup
constexpr int kSortItems = MP_SORT_ITEMS;          // keys per thread
constexpr int kSortTile = kSortBlock * kSortItems; // keys per workgroup
constexpr int kSortMaxBits = 9;                    // digit width cap (512 buckets)

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Number of key bits for keys in [0, n): at least 1.
inline int key_bits(int64_t n) {
    int b = 1;
    while (b < 62 && (int64_t(1) << b) < n) ++b;
    return b;
}

// The digits of an LSD sort of `bits`-bit keys: as few passes of at most
// kSortMaxBits as cover the key, the bits split as evenly as possible, with
// the one-bit-wider digits on the last passes.  (The low digits of
// destination ids take all their values evenly, so a narrower digit there
// lengthens every digit run of a tile; the top bits of ids below N often
// take fewer values than their width allows.)
struct DigitPlan {
    int passes;
    int shift[4], width[4];
    int min_width, max_width;
};
inline DigitPlan digit_plan(int bits) {
    DigitPlan d{};
    d.min_width = kSortMaxBits;
    d.passes = (bits + kSortMaxBits - 1) / kSortMaxBits;
    const int base = bits / d.passes, extra = bits % d.passes;
    for (int p = 0, s = 0; p < d.passes; ++p) {
        d.width[p] = base + (p >= d.passes - extra ? 1 : 0);
        d.shift[p] = s;
        s += d.width[p];
        if (d.width[p] > d.max_width) d.max_width = d.width[p];
        if (d.width[p] < d.min_width) d.min_width = d.width[p];
    }
    return d;
}

// ---- wave-level multisplit -------------------------------------------------
// Lanes of the wavefront that hold a valid key with the same digit as this
// lane: one ballot per digit bit; a lane differs from this one where the
// ballot's bit differs from this lane's own bit (sign-extended to a full
// word, so that one XOR per half-mask finds those lanes).  The bits are
// unrolled up to MAXBITS under a wave-uniform test.
template <int MAXBITS>
__device__ inline uint64_t digit_peers(bool ok, uint32_t d, int bits = MAXBITS) {
    uint32_t dlo = 0, dhi = 0;  // lanes whose digit differs in some bit
#pragma unroll
    for (int b = 0; b < MAXBITS; ++b) {
        if (b < bits) {
            const int32_t sb = (int32_t)(d << (31 - b)) >> 31;  // 0 or -1
            const uint64_t bal = __ballot(sb != 0);
            dlo |= (uint32_t)bal ^ (uint32_t)sb;
            dhi |= (uint32_t)(bal >> 32) ^ (uint32_t)sb;
        }
    }
    return __ballot(ok) & ~(((uint64_t)dhi << 32) | dlo);
}

// Set bits of m below this lane.
__device__ inline uint32_t count_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ---- stable LSD radix sort, one sweep per digit (sort.hip) ----------------
//
// radix_sort_begin() computes the global digit histogram of every pass in one
// read of the keys (and clears the scratch); then each radix_sort_pass()
// ranks, offsets and scatters in a single kernel, getting the offsets of
// earlier tiles by decoupled look-back.
constexpr int kMaxPasses = 4;  // keys of at most 31 bits, digits of at most 9 bits

struct RadixScratch {
    uint64_t* desc;     // [tiles * R] look-back descriptors (R = 2^bits <= 512)
    uint32_t* ghist;    // [kMaxPasses * 512] global digit histograms
    uint32_t* counter;  // [kMaxPasses] dynamic tile ids
    uint32_t* err;      // nonzero: a look-back wait gave up (the result is invalid)
    uint32_t* a_or;     // the OR of payload a (where it was asked for)
    // for rowptr: the sorted keys (rowptr_by_keys), or
    uint32_t* keys;     // [n]
    uint32_t* starts;   // [N] first position of every row that has edges
    uint32_t* first;    // [tiles of N + 1 rows] scratch of rowptr
    size_t bytes;
};
// n keys below N; base may be nullptr (sizes only)
size_t radix_scratch_bytes(int64_t n, int64_t N);
RadixScratch radix_scratch(void* base, int64_t n, int64_t N);

struct RadixPass {
    // the first pass reads keys_in and a_in (b is the element's index), the
    // others kv_in (and b_in, where words have no room for b)
    const uint32_t* keys_in;  // [n]
    const int32_t* a_in;      // [n]
    const uint64_t* kv_in;    // [n]
    const int32_t* b_in;      // [n], with b_out
    // the last pass writes a_out (and b_out) and the rows' starts, the others
    // kv_out (and b_out)
    int32_t* a_out;           // [n]
    int32_t* b_out;           // [n], or nullptr: b is not carried
    uint64_t* kv_out;         // [n]
    int64_t n, rows;          // keys lie below rows
    int pass, shift, bits;
    int prev_shift, prev_bits;  // the digit of the pass before
    // with b: bits of a key, of a (0: as many as sc.a_or says) and of b, and
    // the narrowest and widest digit of the passes
    int key_bits, a_bits, b_bits, min_width, max_width;
    RadixScratch sc;
};
// a: nullptr, or the payload whose bits sc.a_or collects
hipError_t radix_sort_begin(const uint32_t* keys, const int32_t* a, int64_t n, int64_t N,
                            const DigitPlan& dp, const RadixScratch& sc, hipStream_t s);
hipError_t radix_sort_pass(const RadixPass& p, hipStream_t s);

// The whole COO -> CSR of at most kSortSmall edges and rows by one workgroup.
// perm, val_in and val_out, status: nullptr where not wanted.
constexpr int kSortSmall = 16384;
struct SmallSort {
    const uint32_t* dst;
    const int32_t* src;
    const float* val_in;
    int32_t* col;
    int32_t* perm;
    float* val_out;
    void* rowptr;
    int32_t* status;
    int n, rows;
    int passes, width;  // digits, and bits of each
};
hipError_t launch_sort_small(SmallSort p, int key_bits, int rp64, hipStream_t s);

// Write MP_OK into the caller's status word (nullptr: nothing).
hipError_t launch_status_ok(int32_t* status, hipStream_t s);
// After the last pass: rowptr (left alone if the sort failed) and the
// caller's status word (nullptr: not wanted).
hipError_t launch_rowptr(const RadixScratch& sc, int key_bits, int64_t E, int64_t N, void* rowptr,
                         int rp64, int32_t* status, hipStream_t s);
// Whether rowptr comes from the sorted keys rather than from the rows' starts.
bool rowptr_by_keys(int64_t E, int64_t N);
// rowptr of keys sorted by the caller, by binary search (bounded work for
// any order of keys)
hipError_t launch_rowptr_by_search(const uint32_t* keys, int64_t E, int64_t N, void* rowptr,
                                   int rp64, hipStream_t s);
hipError_t launch_fill_rowptr_zero(int64_t N, void* rowptr, int rp64, hipStream_t s);
hipError_t launch_gather_f32(const float* in, const int32_t* idx, int64_t n, float* out,
                             hipStream_t s);
hipError_t launch_validate_coo(const int32_t* src, const int32_t* dst, int64_t E, int64_t N_src,
                               int64_t N_dst, int64_t* d_count, hipStream_t s);
hipError_t launch_validate_csr(const void* rowptr, int rp64, const int32_t* col, int64_t N_dst,
                               int64_t N_src, int64_t E, int64_t* d_count, hipStream_t s);
hipError_t launch_copy_i32(const int32_t* in, int64_t n, int32_t* out, hipStream_t s);
// Relations r < n listed one after another: src[r][i] + src_add[r] and dst[r][i]
// + dst_add[r] at off[r] + i, for i < E[r].
constexpr int kConcatMax = 32;
struct ConcatParams {
    int n;
    const int32_t* src[kConcatMax];
    const int32_t* dst[kConcatMax];
    int64_t E[kConcatMax], off[kConcatMax];
    int32_t src_add[kConcatMax], dst_add[kConcatMax];
    int64_t block_off[kConcatMax];  // filled by the launch
    int32_t* src_out;
    int32_t* dst_out;
};
hipError_t launch_concat_relations(ConcatParams p, hipStream_t s);
hipError_t launch_iota(int64_t n, int32_t* out, hipStream_t s);
hipError_t launch_copy_f32(const float* in, int64_t n, float* out, hipStream_t s);
hipError_t launch_validate_sorted(const int32_t* dst, int64_t E, int64_t* d_count, hipStream_t s);

// ---- aggregation (spmm.hip) --------------------------------------------------
enum : int { kSum = MP_SUM, kMean = MP_MEAN, kMax = MP_MAX };

// Feature-row geometry of one launch: a row of F elements is cut into Ltot
// lane-chunks of EPL elements (one vector load each).  A wavefront holds S
// slots of L lanes; when Ltot > 64 the row is split into FT feature tiles of
// 64 lanes, each handled by its own wavefront.
struct Geometry {
    bool wide;       // the wide cut of rows that only narrow loads divide
    int elem_bytes;  // 4 (fp32) or 2 (bf16)
    int epl;         // elements per lane-chunk: vector bytes / elem_bytes
    int64_t ltot;    // lane-chunks per feature row
    int L, S, FT;    // lanes per slot, slots per wave, feature tiles
};
// x_align: the feature pointer value(s) and row strides in bytes, OR-ed
// (only the low bits matter).  wide: rows that only narrow loads divide (an odd
// F, or a table that starts anywhere) are cut into chunks of four elements too,
// whose last may begin inside the one before it (wide_rows); otherwise chunks
// divide the row and are aligned.
Geometry make_geometry(int64_t F, int x_dtype, uintptr_t x_align, bool wide);
// Whether rows that only narrow loads divide are better cut into wide chunks,
// by what is done with them (reduce: of kUseAggregate) and by how long they are.
enum RowUse { kUseAggregate, kUseStats, kUseDot };
struct RowLengths {
    int64_t rows, edges;
    bool planned;        // the plan has counted
    int64_t ge32, ge64;  // the rows of at least 32 and 64 edges (or more than those)
};
bool wide_rows(RowUse use, int reduce, int64_t F, int x_dtype, uintptr_t x_align,
               const RowLengths& r);
constexpr int64_t kWideAlways = 33;  // features from which plans take rows by the wide cut

// Degree classes of the plan (keys of the row sort).
constexpr int kSmallClasses = 16;       // small rows: see plan_row
constexpr int kClassMid = kSmallClasses;
constexpr int kClassHub = kSmallClasses + 1;
constexpr int kPlanClasses = kClassHub + 1;
constexpr int kPlanClassBits = 5;       // of a class
constexpr int kMaxChunksPerHub = 2048;  // hub rows are split into <= this many chunks
constexpr int kTinyDeg = 7;             // rows of at most this many edges: tiny-row kernel
constexpr int kTinyClassEnd = 4;        // classes 0..3 (bit length <= 3) are tiny
constexpr int64_t kTinyWaves = 4096;    // persistent wavefronts of the tiny-row kernel

struct SpmmParams {
    const void* rowptr;
    int rp64;
    const int32_t* col;  // nullptr: col[p] = p (a readout over contiguous segments)
    const float* w;
    int n_tables;
    const char* table_ptr[MP_MAX_TYPES];
    int64_t table_off[MP_MAX_TYPES + 1];
    // byte offset from table_ptr[0] such that global row c of table t starts
    // at table_ptr[0] + voff[t] + c * ldx * elem_bytes
    int64_t voff[MP_MAX_TYPES];
    int64_t F;
    int64_t ldx;  // row stride of the feature tables in elements (>= F)
    int off32;    // one table, all of it within 4 GiB of table_ptr[0]
    int L, S, FT;
    int64_t ltot;
    // work list (waves, in launch order): hub chunks, mid rows, small groups
    const int32_t* rowlist;  // nullptr: rows 0..N-1 all handled as "mid"
    const int32_t* rowbeg;   // [N] rowptr[rowlist[k]] (plan only)
    const int32_t* rowend;   // [N] rowptr[rowlist[k] + 1] (plan only)
    int64_t n_hub_waves, n_mid_waves, n_small_waves;
    int64_t hub_base, mid_base, small_base, n_small, n_hub;
    int64_t n_tiny;          // rowlist[0, n_tiny): rows for the tiny-row kernel
    const uint32_t* chunk_off;  // indexed by rowlist position
    int reduce;
    void* out;
    int out_bf16;
    void* out_max;
    int max_bf16;
    int32_t* argout;
    // masked sum (gradient of max): edge t contributes feature f only where
    // bit f of the win mask of forward position ekey[t] is set (word
    // mbits[ekey[t] * mw + f / 32], bit f % 32); both nullptr otherwise.
    // mbits holds at least mw words even without edges: the kernels load
    // word 0 for invalid edges and discard it.
    const int32_t* ekey;
    const uint32_t* mbits;
    int64_t mw;
    // the same by win records (backward.hip) in place of the masks: nullptr,
    // or kWinWords words per forward position; an edge of more wins than a
    // record holds reads its destination's argmax and gradient rows (g)
    const uint32_t* recs;
    const int32_t* win_arg;
    const void* win_g;
    int win_g_bf16;
    // stats mode (stacked statistics from one gather): each non-null output
    // [N_dst, F] fp32 (arguments int32) is written
    int stats;
    float* o_sum;
    float* o_mean;
    float* o_max;
    int32_t* o_amax;
    float* o_min;
    int32_t* o_amin;
    float* o_var;
    float* o_std;
    float* part_sum;
    float* part_max;
    int32_t* part_arg;
    float* part_dsum;  // stats: hub partial sums of (m - K)
    float* part_sq;    // stats: hub partial sums of (m - K)^2
    float* part_min;
    int32_t* part_amin;
};

// ---- rows of CSR positions ---------------------------------------------------
// Start of row v (0 for row 0, E for row N and beyond), clamped to [0, E].
template <typename IT>
__device__ inline int64_t row_bound(const IT* __restrict__ rowptr, int64_t N, int64_t E, int64_t v) {
    if (v <= 0) return 0;
    if (v >= N) return E;
    const int64_t b = (int64_t)rowptr[v];
    return b < 0 ? 0 : (b > E ? E : b);
}

// The last row v in [0, N) that starts at or before position p (the row of p
// when 0 <= p < E), found by the whole wavefront: every round splits the
// candidates into 64 parts by one load per lane, so 2.4M rows take four
// round trips.  p is the same in all lanes; all of them must be active.  The
// number of rounds depends on N alone, so it ends whatever rowptr holds.
template <typename IT>
__device__ inline int64_t row_of_position(const IT* __restrict__ rowptr, int64_t N, int64_t E,
                                          int64_t p, int lane) {
    int64_t lo = 0, n = N;  // the row is one of lo .. lo + n - 1
    while (n > 1) {
        const int64_t step = (n + kWave - 1) / kWave;
        // candidate starts lo + (lane + 1) * step, while they lie in the range
        const int64_t c = (int64_t)(lane + 1) * step;
        const bool le = c < n && row_bound(rowptr, N, E, lo + c) <= p;
        const int k = __popcll(__ballot(le));
        lo += (int64_t)k * step;
        const int64_t left = n - (int64_t)k * step;
        n = left < step ? left : step;
    }
    return lo;
}

// ---- merged ranges -------------------------------------------------------------
// out[q] = the number of values a(i) <= q, for q in [0, m), of n nondecreasing
// values in [0, m]: the row of every position from the rows' ends, or every
// row's start from sorted keys.  Values and outputs are taken in merged order
// (value i before output q where a(i) <= q; value i is item a(i) + i), and each
// workgroup takes SPAN consecutive ITEMS, so its work is the same where many
// values lie between two outputs, and many outputs between two values.  Two
// wavefronts find the ends of its range by 64-way searches (mostly two round
// trips), its values are staged in LDS and each lane searches them for
// four consecutive outputs, which it stores together.
//
// Whatever the values, every output is written, with a count in [0, n], and the
// work ends: a search has at most one round per six bits of n and one more, and
// neighbouring workgroups search for the same ends.

// The number of values whose item lies before item d (the whole wavefront; all
// lanes active).  A first round looks around the place that evenly spread
// values would give, which mostly leaves one more round.
template <typename A>
__device__ inline int64_t merge_search(const A& a, int64_t n, int64_t items, int64_t d, int lane) {
    int64_t r = 0, c = n;  // the result is in [r, r + c]
    constexpr int64_t kWindow = kWave * kWave;
    if (n > 2 * kWindow) {
        const int64_t guess = (int64_t)((double)d * ((double)n / (double)items)) - kWindow / 2;
        const int64_t w0 = guess < 0 ? 0 : (guess > n - kWindow ? n - kWindow : guess);
        const int64_t i = w0 + (int64_t)(lane + 1) * kWave - 1;
        const int k = __popcll(__ballot(a(i) + i < d));
        if (k == 0) {  // in [0, w0 + kWave - 1]
            c = w0 + kWave - 1;
        } else {
            r = w0 + (int64_t)k * kWave;
            c = k == kWave ? n - r : kWave - 1;
        }
    }
    while (c > 0) {
        const int64_t step = (c + kWave - 1) / kWave;
        const int64_t i = (int64_t)(lane + 1) * step - 1;
        const bool before = i < c && a(r + i) + r + i < d;
        const int64_t k = (int64_t)__popcll(__ballot(before)) * step;
        r += k;
        c = c - k < step ? c - k : step - 1;
    }
    return r;
}

// VEC: out is 16-byte aligned.  For a workgroup of kMergeBlock threads.
constexpr int kMergeBlock = 256;

template <int SPAN, bool VEC, typename OUT, typename A>
__device__ inline void merge_counts(const A& a, int64_t n, int64_t m, OUT* __restrict__ out) {
    __shared__ int32_t s[SPAN];
    __shared__ int64_t s_end[2];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int64_t d0 = (int64_t)blockIdx.x * SPAN;
    const int64_t d1 = d0 + SPAN < n + m ? d0 + SPAN : n + m;
    if (wv < 2) {
        const int64_t r = merge_search(a, n, n + m, wv == 0 ? d0 : d1, lane);
        if (lane == 0) s_end[wv] = r;
    }
    __syncthreads();
    const int64_t r0 = s_end[0], r1 = s_end[1];
    int64_t q0 = d0 - r0, q1 = d1 - r1;
    q0 = q0 < 0 ? 0 : (q0 > m ? m : q0);
    q1 = q1 < 0 ? 0 : (q1 > m ? m : q1);
    const int nr = (int)(r1 - r0 < 0 ? 0 : (r1 - r0 > SPAN ? SPAN : r1 - r0));
    // values relative to q0, cut to the range
    for (int i = threadIdx.x; i < nr; i += kMergeBlock) {
        const int64_t v = a(r0 + i) - q0;
        s[i] = (int32_t)(v < 0 ? 0 : (v > SPAN ? SPAN : v));
    }
    __syncthreads();
    constexpr int V = VEC ? 4 : 1;
    const int top = nr > 0 ? 1 << (31 - __clz(nr)) : 0;  // the largest power of two up to nr
    for (int64_t q = q0 / V * V + (int)threadIdx.x * V; q < q1; q += kMergeBlock * V) {
        // the first value beyond each output
        OUT v[V];
        if (nr > SPAN / 4) {
            // the V searches side by side, their LDS reads in flight together
            int lo[V] = {};
            for (int step = top; step > 0; step >>= 1) {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const int i = lo[e] + step - 1;
                    if (i < nr && s[i] <= q + e - q0) lo[e] += step;
                }
            }
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = (OUT)(r0 + lo[e]);
        } else {
            // few values next to outputs: mostly that of the output before, or
            // one close by
            int lo = 0;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const int64_t x = q + e - q0;
                bool found = false;
                if (e > 0) {
#pragma unroll
                    for (int near = 0; near < 4; ++near) {
                        found = !(lo < nr && s[lo] <= x);
                        if (found) break;
                        ++lo;
                    }
                }
                if (!found) {
                    int hi = nr;
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (s[mid] <= x) lo = mid + 1; else hi = mid;
                    }
                }
                v[e] = (OUT)(r0 + lo);
            }
        }
        if constexpr (VEC) {
            if (q >= q0 && q + V <= q1) {
                struct alignas(16) Block { OUT x[V]; };
                *reinterpret_cast<Block*>(out + q) = *reinterpret_cast<const Block*>(v);
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (q + e >= q0 && q + e < q1) out[q + e] = v[e];
            }
        } else {
            out[q] = v[0];
        }
    }
}

// Items per workgroup: many where the ends' searches would be much of the
// work, few where long ranges would leave most of the card idle.
constexpr int64_t kMergeLong = int64_t(1) << 22;  // items from which ranges are long
constexpr int kMergeSpanLong = 4096, kMergeSpanShort = 1024;

// ---- backward (backward.hip) -----------------------------------------------
struct GradWParams {
    const void* rowptr;
    int rp64;
    const int32_t* col;     // row of x read by position p; nullptr: p itself
    const int32_t* row;     // destination row of every CSR position; nullptr: p
    const void* x;          // [N_src, F]
    const void* g;          // [N_dst, F] gradient of the aggregation output
    const int32_t* argout;  // [N_dst, F] (max only)
    int64_t F, E;
    int L, S, FT;
    int64_t ltot;
    int reduce;             // exactly one of kSum, kMean, kMax
    float* grad_w;          // [E]
    const int32_t* oidx;    // nullptr, or grad_w[oidx[p]] receives position p's dot
};
hipError_t launch_rows_of_edges(const void* rowptr, int rp64, int64_t N, int64_t E, int32_t* row,
                                hipStream_t s);
hipError_t launch_scale_inv_deg(const void* g, int g_bf16, const void* rowptr, int rp64, int64_t N,
                                int64_t F, float* out, hipStream_t s);
hipError_t launch_spmm_grad_w(const GradWParams& p, int x_dtype, int g_dtype, int epl,
                              hipStream_t s);
// Win masks of the max aggregation: for every forward CSR position p, mw =
// ceil(F / 32) words whose bit f says argout[row(p), f] == p.
inline int64_t win_mask_words(int64_t F) { return (F + 31) / 32; }
hipError_t launch_win_masks(const void* rowptr, int rp64, const int32_t* argout, int64_t N,
                            int64_t F, uint32_t* bits, hipStream_t s);
// Win records of the max aggregation: per forward CSR position, the values and
// feature ids of its first kWinValues wins and the number of its wins.
constexpr int kWinWords = 8;
constexpr int kWinValues = 6;
constexpr int64_t kWinMaxF = 256;  // feature ids are bytes
// Whether the gradient of max goes by win records rather than masks.
bool use_win_records(int64_t N_dst, int64_t E, int64_t F);
hipError_t launch_win_records(const void* rowptr, int rp64, const int32_t* argout, const void* g,
                              int g_bf16, int64_t N, int64_t E, int64_t F, uint32_t* recs,
                              hipStream_t s);
// Sum over the rows of P (a transposed CSR) of the wins in P.recs.
hipError_t launch_win_gather(const SpmmParams& p, hipStream_t s);

// ---- segment matmul (gmm.hip) --------------------------------------------------
struct GmmParams {
    const uint16_t* A;  // bf16 rows of the left operand
    const uint16_t* B;  // bf16: per segment Bt[t] = B + t * b_stride (gmm_nt), or G (weight grad)
    void* C;            // output (gmm_nt)
    float* part;        // fp32 partial tiles (weight grad)
    int64_t lda, ldb, ldc, b_stride;
    int64_t M, N, K;    // gmm_nt: N columns, K inner; weight grad: M x N = F x Fo
    int T;
    int64_t seg[MP_MAX_TYPES + 1];       // row offsets of the segments
    int64_t tile_off[MP_MAX_TYPES + 1];  // first tile (gmm_nt) or chunk (weight grad) of each
    int64_t rows_per_chunk;
    int c_bf16;
};
hipError_t launch_gmm_nt(const GmmParams& p, int64_t tiles, hipStream_t s);
hipError_t launch_gmm_weight_grad(const GmmParams& p, int64_t chunks, float* dW, hipStream_t s);
hipError_t launch_transpose_w(const uint16_t* W, int64_t T, int64_t F, int64_t Fo, uint16_t* Wt,
                              hipStream_t s);
int64_t gmm_tile_rows();
int64_t gmm_tile_cols();

hipError_t launch_spmm(const SpmmParams& p, int x_dtype, int epl, hipStream_t s);
hipError_t launch_spmm_tiny(const SpmmParams& p, int x_dtype, int epl, hipStream_t s);
hipError_t launch_spmm_fixup(const SpmmParams& p, hipStream_t s);

// ---- plan (scan.hip) -----------------------------------------------------------
constexpr int64_t kPlanSingleRows = 16384;  // up to here one workgroup builds the plan
struct PlanParams {
    const void* rowptr;
    int rp64;
    int64_t N;
    // a class starts after `split` edges too; rows beyond long_min are counted
    int64_t split, small_max, hub_min, long_min;
    int chunk_min;
    uint32_t* tile_cnt;   // [plan_tile_counts(N)]
    int32_t* rowlist;     // [N] rows by class, then by id
    int32_t* rowbeg;      // [N] their ranges
    int32_t* rowend;      // [N]
    uint32_t* chunk_off;  // [N + 1] first chunk of every hub row's entry; [N]: all chunks
    // first row-list position of every class, N, the number of chunks, and of
    // rows beyond long_min
    uint32_t* header;     // [kPlanClasses + 3]
};
int64_t plan_tile_counts(int64_t N);
hipError_t launch_plan(const PlanParams& p, hipStream_t s);

// ---- edge-materialized messages (messages.hip) ----------------------------------
struct MessageGather {
    const int32_t* idx;  // [E] row of x of every message
    const float* w;      // [E] or nullptr
    const void* x;       // [N_src, F]
    int x_bf16;
    void* msg;           // [E, F]: fp32, or bf16 (unweighted bf16 x, an exact copy)
    int msg_bf16;
    int64_t E, F;
    int epl;             // elements per lane-chunk (message_epl)
};
struct MessageBackward {
    const void* rowptr;
    int rp64;
    const int32_t* argout;  // [N_dst, F] (max only)
    const void* g;          // [N_dst, F] dL/dout
    int g_bf16;
    int64_t N, E, F;
    int reduce;             // exactly one of kSum, kMean, kMax
    int epl;
    float* dmsg;            // [E, F]
};
// Largest lane-chunk width in {max_epl, ..., 2, 1} that divides F, keeps each
// listed element size within 16 bytes per access and divides every pointer.
int message_epl(int64_t F, const uintptr_t* ptrs, const int* elem_bytes, int n, int max_epl);
hipError_t launch_message_gather(const MessageGather& a, hipStream_t s);
hipError_t launch_message_scale(const float* in, float* out, const float* mask,
                                const int32_t* idx, int64_t E, int64_t F, int epl, hipStream_t s);
hipError_t launch_message_backward(const MessageBackward& a, hipStream_t s);

// ---- feature-table layout (layout.hip) -------------------------------------------
// out[r, 0:F] = in[r, 0:F] for r < N, rows ld_in / ld_out elements apart.
hipError_t launch_copy_rows(const void* in, int64_t ld_in, void* out, int64_t ld_out, int64_t N,
                            int64_t F, int elem_bytes, hipStream_t s);

// ---- bandwidth probes (probe.hip) ---------------------------------------------
hipError_t launch_probe_read(const void* p, int64_t n16, uint32_t* sink, hipStream_t s);
hipError_t launch_probe_copy(const void* in, void* out, int64_t n16, hipStream_t s);
hipError_t launch_probe_scatter(const void* in, const int32_t* dest, int64_t n, int elem_bytes,
                                void* out, hipStream_t s);
hipError_t launch_probe_gather(const int32_t* idx, int64_t n, const void* table,
                               int64_t stride_bytes, int L, uint32_t* sink, hipStream_t s);

}  // namespace mp
