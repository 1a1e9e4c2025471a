// C ABI of libmp (declared in include/mp.h): argument validation, workspace
// layout and launch sequencing.  Every compute step runs in the HIP kernels
// of the .hip sources; this file only checks arguments, carves
// caller-provided buffers and enqueues launches.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "mp_internal.hpp"


using namespace mp;

namespace {

inline hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }

inline int hip_status(hipError_t e) { return e == hipSuccess ? MP_OK : MP_ERR_HIP; }

// Sequential carve of a caller buffer into 256-byte aligned pieces.
struct Carver {
    char* base;
    size_t off = 0;
    explicit Carver(void* b) : base(static_cast<char*>(b)) {}
    template <typename T>
    T* take(size_t count) {
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off = align_up(off + count * sizeof(T), 256);
        return p;
    }
};

bool valid_itype(int t) { return t == MP_I32 || t == MP_I64; }
bool valid_dtype(int t) { return t == MP_F32 || t == MP_BF16; }
bool valid_reduce(int r) {
    return r == MP_SUM || r == MP_MEAN || r == MP_MAX || r == (MP_SUM | MP_MAX) ||
           r == (MP_MEAN | MP_MAX);
}

// ---- COO -> CSR workspace layout ---------------------------------------------

// The passes before the last write 8-byte words, ping-ponging between kv[0]
// and kv[1]; the last writes src into col.  The COO-id payload, when asked for,
// travels in the words, or where their bits do not suffice (which the device
// finds out) as a 4-byte array ping-ponging between eid_tmp and the output.
struct CsrLayout {
    DigitPlan dp;
    int key_bits;
    int32_t *eid_tmp, *eid_final;
    uint64_t* kv[2];
    RadixScratch sc;
    size_t bytes;
};

CsrLayout csr_layout(void* ws, int64_t E, int64_t N, int with_payload) {
    CsrLayout L{};
    L.key_bits = key_bits(N);
    L.dp = digit_plan(L.key_bits);
    Carver c(ws);
    const size_t e = (size_t)(E > 0 ? E : 1);
    L.kv[0] = L.dp.passes > 1 ? c.take<uint64_t>(e) : nullptr;
    L.kv[1] = L.dp.passes > 2 ? c.take<uint64_t>(e) : nullptr;
    L.eid_tmp = (with_payload && L.dp.passes > 1) ? c.take<int32_t>(e) : nullptr;
    L.eid_final = with_payload ? c.take<int32_t>(e) : nullptr;
    char* scratch = c.take<char>(radix_scratch_bytes(E, N));
    if (ws) L.sc = radix_scratch(scratch, E, N);
    L.bytes = c.off;
    return L;
}

int check_csr_sizes(int64_t E, int64_t N) {
    if (E < 0 || E > INT32_MAX || N < 1 || N > INT32_MAX) return MP_ERR_SIZE;
    return MP_OK;
}

// a_bits: bits of every src (0: not known).
int coo_to_csr_impl(const int32_t* src, const int32_t* dst, int64_t E, int64_t N, void* rowptr,
                    int itype, int32_t* col, int32_t* perm, const float* val_in, float* val_out,
                    int a_bits, void* ws, size_t ws_bytes, int32_t* status, hipStream_t s) {
    const int rp64 = itype == MP_I64;
    if (E == 0) {
        hipError_t e = launch_fill_rowptr_zero(N, rowptr, rp64, s);
        if (e == hipSuccess) e = launch_status_ok(status, s);
        return hip_status(e);
    }
    const int payload = (perm != nullptr || val_out != nullptr) ? 1 : 0;
    CsrLayout L = csr_layout(ws, E, N, payload);
    if (ws_bytes < L.bytes) return MP_ERR_WORKSPACE;
    if (E <= kSortSmall && N <= kSortSmall)
        return hip_status(launch_sort_small(
            SmallSort{reinterpret_cast<const uint32_t*>(dst), src, val_in, col, perm,
                      val_in ? val_out : nullptr, rowptr, status, (int)E, (int)N, 0, 0},
            L.key_bits, rp64, s));
    int32_t* eid_final = perm ? perm : L.eid_final;
    const int passes = L.dp.passes;

    const uint32_t* keys = reinterpret_cast<const uint32_t*>(dst);
    const int32_t* measure = payload && !a_bits ? src : nullptr;
    if (radix_sort_begin(keys, measure, E, N, L.dp, L.sc, s) != hipSuccess) return MP_ERR_HIP;
    for (int p = 0; p < passes; ++p) {
        const bool last_parity = ((passes - 1 - p) % 2) == 0;  // lands where the final pass writes
        RadixPass rp{};
        if (p == 0) {
            rp.keys_in = keys;
            rp.a_in = src;
        } else {
            rp.kv_in = L.kv[(p - 1) % 2];
            rp.b_in = payload ? (last_parity ? L.eid_tmp : eid_final) : nullptr;
            rp.prev_shift = L.dp.shift[p - 1];
            rp.prev_bits = L.dp.width[p - 1];
        }
        if (p < passes - 1) rp.kv_out = L.kv[p % 2];
        else rp.a_out = col;
        rp.b_out = payload ? (last_parity ? eid_final : L.eid_tmp) : nullptr;
        rp.n = E;
        rp.rows = N;
        rp.pass = p;
        rp.shift = L.dp.shift[p];
        rp.bits = L.dp.width[p];
        rp.key_bits = L.key_bits;
        rp.a_bits = a_bits;
        rp.b_bits = key_bits(E);
        rp.min_width = L.dp.min_width;
        rp.max_width = L.dp.max_width;
        rp.sc = L.sc;
        if (radix_sort_pass(rp, s) != hipSuccess) return MP_ERR_HIP;
    }
    hipError_t e = launch_rowptr(L.sc, L.key_bits, E, N, rowptr, rp64, status, s);
    if (e == hipSuccess && val_in && val_out) e = launch_gather_f32(val_in, eid_final, E, val_out, s);
    return hip_status(e);
}

// ---- plan --------------------------------------------------------------------

struct PlanLayout {
    uint32_t* tile_cnt;
    int32_t* rowlist;
    int32_t* rowbeg;
    int32_t* rowend;
    uint32_t* chunk_off;
    uint32_t* header;
    size_t bytes;
};

PlanLayout plan_layout(void* buf, int64_t N) {
    PlanLayout L{};
    Carver c(buf);
    const size_t n = (size_t)(N > 0 ? N : 1);
    L.rowlist = c.take<int32_t>(n);
    L.rowbeg = c.take<int32_t>(n);
    L.rowend = c.take<int32_t>(n);
    L.chunk_off = c.take<uint32_t>(n + 1);
    L.tile_cnt = c.take<uint32_t>((size_t)plan_tile_counts(N));
    L.header = c.take<uint32_t>(64);
    L.bytes = c.off;
    return L;
}

}  // namespace

struct mp_plan {
    const void* rowptr;
    int itype;
    int64_t N_dst, E, F;
    int x_dtype;
    int64_t small_max, hub_min;
    int chunk_min;
    // rows of the list that are small for narrow chunks of features (the first
    // n_small_narrow) and for wide ones (n_small); then mid rows up to hub_base
    int64_t n_tiny, n_small_narrow, n_small, n_hub, n_chunks;
    int64_t hub_base;
    int64_t ge32, ge64;  // rows of at least 32 and 64 edges (or more)
    int32_t* rowlist;
    int32_t* rowbeg;
    int32_t* rowend;
    uint32_t* chunk_off;
};

namespace {

// A single feature table of `rows` rows, `ld` elements apart, is addressed
// with 32-bit byte offsets from its base: it spans under 4 GiB, and row
// indices and the row stride in bytes fit 24 bits, so that the kernels form
// an offset with one 24-bit multiply-add.
inline int fits_off32(int64_t rows, int64_t ld, int elem_bytes) {
    return rows * ld * elem_bytes <= (int64_t)UINT32_MAX && rows <= ((int64_t)1 << 24) &&
                   ld * elem_bytes < ((int64_t)1 << 24)
               ? 1
               : 0;
}

RowLengths row_lengths(const mp_plan* plan, int64_t N_dst) {
    return plan ? RowLengths{N_dst, plan->E, true, plan->ge32, plan->ge64}
                : RowLengths{N_dst, 0, false, 0, 0};
}

// Fill the work description of SpmmParams from a plan (or the plan-free
// generic layout) and launch the main kernel plus the hub fix-up.
int run_spmm(const mp_plan* plan, SpmmParams& P, const Geometry& g, int x_dtype, int64_t N_dst,
             void* ws, size_t ws_bytes, hipStream_t s) {
    if (P.ldx == 0) P.ldx = P.F;  // contiguous feature rows
    P.L = g.L;
    P.S = g.S;
    P.FT = g.FT;
    P.ltot = g.ltot;
    const bool hx = P.stats != 0;
    const bool hs = hx || (P.reduce & (MP_SUM | MP_MEAN)) != 0;
    const bool hm = hx || (P.reduce & MP_MAX) != 0;
    // tiny rows have a kernel of their own when slots are wide enough and its
    // wavefronts (kTinyWaves at most) have several groups of rows each to
    // pipeline; fewer rows go with the small ones, a launch less (10k rows of 4 edges,
    // F = 64: fp32 sum 15.9 -> 12.9 us, statistics 24.7 -> 21.5; at 8192
    // groups 19.3 -> 15.7; beyond, the tiny kernel is the faster)
    const bool tiny = plan && g.L > kTinyDeg && !P.recs &&
                      ceil_div(plan->n_tiny, g.S) * g.FT > 2 * kTinyWaves;
    // wavefronts per row or chunk, and rows per wavefront of small ones
    const int64_t ft = P.recs ? 1 : g.FT, slots = P.recs ? 8 : g.S;
    if (plan) {
        P.rowlist = plan->rowlist;
        P.rowbeg = plan->rowbeg;
        P.rowend = plan->rowend;
        P.chunk_off = plan->chunk_off;
        P.n_tiny = tiny ? plan->n_tiny : 0;
        P.small_base = P.n_tiny;
        P.mid_base = g.wide || P.recs ? plan->n_small : plan->n_small_narrow;
        P.n_small = P.mid_base - P.n_tiny;
        P.n_hub = plan->n_hub;
        P.hub_base = plan->hub_base;
        P.n_hub_waves = plan->n_chunks * ft;
        P.n_mid_waves = (plan->hub_base - P.mid_base) * ft;
        P.n_small_waves = ceil_div(P.n_small, slots) * ft;
        if (plan->n_chunks > 0) {
            Carver c(ws);
            const size_t cells = (size_t)plan->n_chunks * (size_t)P.F;
            P.part_sum = hs ? c.take<float>(cells) : nullptr;
            P.part_max = hm ? c.take<float>(cells) : nullptr;
            P.part_arg = hm ? c.take<int32_t>(cells) : nullptr;
            P.part_dsum = hx ? c.take<float>(cells) : nullptr;
            P.part_sq = hx ? c.take<float>(cells) : nullptr;
            P.part_min = hx ? c.take<float>(cells) : nullptr;
            P.part_amin = hx ? c.take<int32_t>(cells) : nullptr;
            if (ws_bytes < c.off || !ws) return MP_ERR_WORKSPACE;
        }
    } else {
        P.rowlist = nullptr;
        P.n_mid_waves = N_dst * ft;
    }
    const int64_t waves = P.n_hub_waves + P.n_mid_waves + P.n_small_waves;
    if (ceil_div(waves, 4) > (int64_t)UINT32_MAX) return MP_ERR_SIZE;
    hipError_t e = P.recs ? launch_win_gather(P, s) : launch_spmm_tiny(P, x_dtype, g.epl, s);
    if (e != hipSuccess) return MP_ERR_HIP;
    if (!P.recs) e = launch_spmm(P, x_dtype, g.epl, s);
    if (e != hipSuccess) return MP_ERR_HIP;
    if (plan && plan->n_hub > 0) {
        e = launch_spmm_fixup(P, s);
        if (e != hipSuccess) return MP_ERR_HIP;
    }
    return MP_OK;
}

// The row classes only steer work to kernels (any classification gives the
// same result), so a plan built for one feature dtype serves the other too;
// F must match because hub partials are sized by it.
int check_plan(const mp_plan* plan, const void* rowptr, int itype, int64_t N_dst, int64_t F) {
    if (!plan) return MP_OK;
    if (plan->rowptr != rowptr || plan->itype != itype || plan->N_dst != N_dst || plan->F != F)
        return MP_ERR_PLAN;
    return MP_OK;
}

// ---- stacked aggregations ---------------------------------------------------------

constexpr int kAllAggr = MP_SUM | MP_MEAN | MP_MAX | MP_MIN | MP_VAR | MP_STD;

// Check the output list and fill the stats-mode outputs of P.
int fill_multi_outputs(int n_out, const mp_aggr_out* outs, int64_t rows, SpmmParams& P) {
    if (n_out < 1 || n_out > 6) return MP_ERR_SIZE;
    if (!outs) return MP_ERR_NULL;
    int seen = 0;
    for (int k = 0; k < n_out; ++k) {
        const mp_aggr_out& o = outs[k];
        const int a = o.aggr;
        if ((a & kAllAggr) != a || a == 0 || (a & (a - 1)) != 0 || (seen & a)) return MP_ERR_REDUCE;
        seen |= a;
        const bool has_arg = a == MP_MAX || a == MP_MIN;
        if (rows > 0 && (!o.out || (has_arg && !o.arg))) return MP_ERR_NULL;
        if ((uintptr_t)o.out % 4 || (uintptr_t)o.arg % 4) return MP_ERR_ALIGN;
        switch (a) {
            case MP_SUM: P.o_sum = o.out; break;
            case MP_MEAN: P.o_mean = o.out; break;
            case MP_MAX: P.o_max = o.out; P.o_amax = o.arg; break;
            case MP_MIN: P.o_min = o.out; P.o_amin = o.arg; break;
            case MP_VAR: P.o_var = o.out; break;
            default: P.o_std = o.out; break;
        }
    }
    P.stats = 1;
    P.reduce = MP_SUM | MP_MAX;
    return MP_OK;
}

int multi_impl(const mp_plan* plan, const void* rowptr, int rowptr_itype, const int32_t* col,
               const float* w, const void* x, int x_dtype, int64_t N_src, int64_t N_dst, int64_t F,
               int64_t ldx, int n_out, const mp_aggr_out* outs, void* ws, size_t ws_bytes,
               hipStream_t s) {
    if (!valid_itype(rowptr_itype) || !valid_dtype(x_dtype)) return MP_ERR_DTYPE;
    if (N_src < 0 || N_src > INT32_MAX || N_dst < 0 || N_dst > INT32_MAX || F < 1 || F > 65536 ||
        ldx < F)
        return MP_ERR_SIZE;
    if (!rowptr) return MP_ERR_NULL;
    if (N_dst > 0 && !x) return MP_ERR_NULL;
    SpmmParams P{};
    int st = fill_multi_outputs(n_out, outs, N_dst, P);
    if (st != MP_OK) return st;
    st = check_plan(plan, rowptr, rowptr_itype, N_dst, F);
    if (st != MP_OK) return st;
    const int eb = x_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)x % eb || (uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4) ||
        (uintptr_t)col % 4 || (uintptr_t)w % 4)
        return MP_ERR_ALIGN;
    if (N_dst == 0) return MP_OK;
    const uintptr_t align = (uintptr_t)x | (uintptr_t)(ldx * eb);
    Geometry g = make_geometry(F, x_dtype, align,
                               wide_rows(kUseStats, 0, F, x_dtype, align, row_lengths(plan, N_dst)));
    P.rowptr = rowptr;
    P.rp64 = rowptr_itype == MP_I64;
    P.col = col;
    P.w = w;
    P.n_tables = 1;
    P.table_ptr[0] = static_cast<const char*>(x);
    P.F = F;
    P.ldx = ldx;
    P.off32 = fits_off32(N_src, ldx, eb);
    return run_spmm(plan, P, g, x_dtype, N_dst, ws, ws_bytes, s);
}

// ---- aggregation call (mp_spmm, mp_message_aggregate) ---------------------------

// The arguments of one aggregation; col == nullptr reads position p as
// column p (a table of materialized messages).
struct SpmmCall {
    const mp_plan* plan;
    const void* rowptr;
    int rowptr_itype;
    const int32_t* col;
    const float* w;
    const void* x;
    int x_dtype;
    int64_t N_src, N_dst, F;
    int64_t ldx;  // row stride of x in elements (>= F)
    int reduce;
    void* out;
    int out_dtype;
    void* out_max;
    int max_dtype;
    int32_t* argout;
    void* ws;
    size_t ws_bytes;
};

// Every argument check of an aggregation, before anything is enqueued.
int spmm_check(const SpmmCall& c) {
    if (!valid_reduce(c.reduce)) return MP_ERR_REDUCE;
    if (!valid_itype(c.rowptr_itype) || !valid_dtype(c.x_dtype)) return MP_ERR_DTYPE;
    const bool hs = (c.reduce & (MP_SUM | MP_MEAN)) != 0;
    const bool hm = (c.reduce & MP_MAX) != 0;
    if (hs && !valid_dtype(c.out_dtype)) return MP_ERR_DTYPE;
    if (hm && !valid_dtype(c.max_dtype)) return MP_ERR_DTYPE;
    if (hm && c.max_dtype == MP_BF16 && (c.x_dtype != MP_BF16 || c.w != nullptr))
        return MP_ERR_DTYPE;
    if (c.N_src < 0 || c.N_src > INT32_MAX || c.N_dst < 0 || c.N_dst > INT32_MAX || c.F < 1 ||
        c.F > 65536 || c.ldx < c.F)
        return MP_ERR_SIZE;
    if (!c.rowptr) return MP_ERR_NULL;
    if (c.N_dst > 0) {
        if (!c.x) return MP_ERR_NULL;
        if (hs && !c.out) return MP_ERR_NULL;
        if (hm && (!c.out_max || !c.argout)) return MP_ERR_NULL;
    }
    int st = check_plan(c.plan, c.rowptr, c.rowptr_itype, c.N_dst, c.F);
    if (st != MP_OK) return st;
    const int eb = c.x_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)c.x % eb || (uintptr_t)c.rowptr % (c.rowptr_itype == MP_I64 ? 8 : 4) ||
        (uintptr_t)c.col % 4 || (uintptr_t)c.w % 4 || (uintptr_t)c.argout % 4 ||
        (hs && (uintptr_t)c.out % (c.out_dtype == MP_BF16 ? 2 : 4)) ||
        (hm && (uintptr_t)c.out_max % (c.max_dtype == MP_BF16 ? 2 : 4)))
        return MP_ERR_ALIGN;
    size_t need = 0;
    mp_spmm_workspace(c.plan, c.reduce, &need);
    if (c.N_dst > 0 && need > 0 && (c.ws_bytes < need || !c.ws)) return MP_ERR_WORKSPACE;
    return MP_OK;
}

// Enqueue a checked aggregation.
int spmm_launch(const SpmmCall& c, hipStream_t s) {
    if (c.N_dst == 0) return MP_OK;
    const int eb = c.x_dtype == MP_BF16 ? 2 : 4;
    const uintptr_t align = (uintptr_t)c.x | (uintptr_t)(c.ldx * eb);
    Geometry g = make_geometry(c.F, c.x_dtype, align,
                               wide_rows(kUseAggregate, c.reduce, c.F, c.x_dtype, align,
                                         row_lengths(c.plan, c.N_dst)));
    SpmmParams P{};
    P.rowptr = c.rowptr;
    P.rp64 = c.rowptr_itype == MP_I64;
    P.col = c.col;
    P.w = c.w;
    P.n_tables = 1;
    P.table_ptr[0] = static_cast<const char*>(c.x);
    P.table_off[0] = 0;
    P.F = c.F;
    P.ldx = c.ldx;
    P.off32 = fits_off32(c.N_src, c.ldx, eb);
    P.reduce = c.reduce;
    P.out = c.out;
    P.out_bf16 = c.out_dtype == MP_BF16;
    P.out_max = c.out_max;
    P.max_bf16 = c.max_dtype == MP_BF16;
    P.argout = c.argout;
    return run_spmm(c.plan, P, g, c.x_dtype, c.N_dst, c.ws, c.ws_bytes, s);
}

// ---- edge-materialized messages ---------------------------------------------------

// Check a message gather and describe it.
int gather_check(const int32_t* idx, const float* w, const void* x, int x_dtype, int64_t N_src,
                 int64_t E, int64_t F, void* msg, int msg_dtype, MessageGather* a) {
    if (!valid_dtype(x_dtype) || !valid_dtype(msg_dtype)) return MP_ERR_DTYPE;
    if (msg_dtype == MP_BF16 && (x_dtype != MP_BF16 || w != nullptr)) return MP_ERR_DTYPE;
    if (E < 0 || E > INT32_MAX || N_src < 0 || N_src > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    if (E > 0 && (!idx || !x || !msg)) return MP_ERR_NULL;
    const int bx = x_dtype == MP_BF16 ? 2 : 4, bm = msg_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)idx % 4 || (uintptr_t)w % 4 || (uintptr_t)x % bx || (uintptr_t)msg % bm)
        return MP_ERR_ALIGN;
    const uintptr_t ptrs[2] = {(uintptr_t)x, (uintptr_t)msg};
    const int sizes[2] = {bx, bm};
    *a = MessageGather{idx, w, x, x_dtype == MP_BF16, msg, msg_dtype == MP_BF16, E, F,
                       message_epl(F, ptrs, sizes, 2, 8)};
    return MP_OK;
}

// ---- segment matmul ------------------------------------------------------------

constexpr int64_t kGmmRowsPerChunk = 2048;  // rows per partial of the weight gradient

// Validate the host segment offsets; fill P.seg and return the row count.
int gmm_segments(const int64_t* seg, int T, GmmParams& P, int64_t* N_rows) {
    if (!seg) return MP_ERR_NULL;
    if (T < 1 || T > MP_MAX_TYPES) return MP_ERR_SIZE;
    if (seg[0] != 0) return MP_ERR_SIZE;
    for (int t = 0; t < T; ++t)
        if (seg[t + 1] < seg[t]) return MP_ERR_SIZE;
    if (seg[T] > INT32_MAX) return MP_ERR_SIZE;
    P.T = T;
    for (int t = 0; t <= T; ++t) P.seg[t] = seg[t];
    *N_rows = seg[T];
    return MP_OK;
}

int gmm_dims(int64_t F, int64_t Fo) {
    // 16-byte row chunks of bf16
    if (F < 8 || Fo < 8 || F > 65536 || Fo > 65536 || F % 8 || Fo % 8) return MP_ERR_SIZE;
    return MP_OK;
}

int64_t gmm_chunks(const int64_t* seg, int T, int64_t* off) {
    int64_t c = 0;
    for (int t = 0; t < T; ++t) {
        off[t] = c;
        c += ceil_div(seg[t + 1] - seg[t], kGmmRowsPerChunk);
    }
    off[T] = c;
    return c;
}

}  // namespace

extern "C" {

int mp_version(void) { return MP_VERSION; }

const char* mp_status_str(int status) {
    switch (status) {
        case MP_OK: return "ok";
        case MP_ERR_NULL: return "a required pointer is NULL";
        case MP_ERR_SIZE: return "size out of range";
        case MP_ERR_DTYPE: return "unsupported dtype or index type";
        case MP_ERR_REDUCE: return "unsupported reduction";
        case MP_ERR_WORKSPACE: return "workspace or plan buffer too small";
        case MP_ERR_PLAN: return "plan does not match the arguments";
        case MP_ERR_HIP: return "HIP launch or copy failed";
        case MP_ERR_ALIGN: return "pointer not aligned to its element size";
        case MP_ERR_CALLBACK: return "the message callback failed";
        case MP_ERR_SORT: return "a device sort gave up waiting; its output is invalid";
        default: return "unknown status";
    }
}

int mp_coo_to_csr_workspace(int64_t E, int64_t N, int rowptr_itype, int with_payload,
                            size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    int st = check_csr_sizes(E, N);
    if (st != MP_OK) return st;
    *bytes = E == 0 ? 0 : csr_layout(nullptr, E, N, with_payload ? 1 : 0).bytes;
    return MP_OK;
}

int mp_coo_to_csr(const int32_t* src, const int32_t* dst, int64_t E, int64_t N, void* rowptr,
                  int rowptr_itype, int32_t* col, int32_t* perm, const float* val_in,
                  float* val_out, void* ws, size_t ws_bytes, int32_t* status, void* stream) {
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    int st = check_csr_sizes(E, N);
    if (st != MP_OK) return st;
    if (!rowptr) return MP_ERR_NULL;
    if (E > 0 && (!src || !dst || !col || !ws)) return MP_ERR_NULL;
    if (E > 0 && (val_in == nullptr) != (val_out == nullptr)) return MP_ERR_NULL;
    if ((uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4) || (uintptr_t)status % 4)
        return MP_ERR_ALIGN;
    return coo_to_csr_impl(src, dst, E, N, rowptr, rowptr_itype, col, perm, val_in, val_out, 0, ws,
                           ws_bytes, status, as_stream(stream));
}

int mp_sorted_coo_to_csr(const int32_t* src, const int32_t* dst, int64_t E, int64_t N,
                         void* rowptr, int rowptr_itype, int32_t* col, int32_t* perm,
                         const float* val_in, float* val_out, void* stream) {
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    int st = check_csr_sizes(E, N);
    if (st != MP_OK) return st;
    if (!rowptr) return MP_ERR_NULL;
    if (E > 0 && (!src || !dst || !col)) return MP_ERR_NULL;
    if (E > 0 && (val_in == nullptr) != (val_out == nullptr)) return MP_ERR_NULL;
    if ((uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4)) return MP_ERR_ALIGN;
    hipStream_t s = as_stream(stream);
    const int rp64 = rowptr_itype == MP_I64;
    if (E == 0) return hip_status(launch_fill_rowptr_zero(N, rowptr, rp64, s));
    // the sorted keys are dst itself (non-negative int32 read as uint32);
    // a binary search per row keeps the work bounded if dst is not sorted
    hipError_t e = launch_rowptr_by_search(reinterpret_cast<const uint32_t*>(dst), E, N,
                                           rowptr, rp64, s);
    if (e == hipSuccess) e = launch_copy_i32(src, E, col, s);
    if (e == hipSuccess && perm) e = launch_iota(E, perm, s);
    if (e == hipSuccess && val_in) e = launch_copy_f32(val_in, E, val_out, s);
    return hip_status(e);
}

int mp_spmm_plan_size(int64_t N_dst, int64_t E, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (N_dst < 0 || N_dst > INT32_MAX || E < 0 || E > INT32_MAX) return MP_ERR_SIZE;
    *bytes = plan_layout(nullptr, N_dst).bytes;
    return MP_OK;
}

int mp_spmm_plan_build(const void* rowptr, int rowptr_itype, int64_t N_dst, int64_t E, int64_t F,
                       int x_dtype, void* plan_buf, size_t plan_bytes, void* stream,
                       mp_plan** out) {
    return mp_spmm_plan_build_opts(rowptr, rowptr_itype, N_dst, E, F, x_dtype, plan_buf,
                                   plan_bytes, nullptr, stream, out);
}

int mp_spmm_plan_build_opts(const void* rowptr, int rowptr_itype, int64_t N_dst, int64_t E,
                            int64_t F, int x_dtype, void* plan_buf, size_t plan_bytes,
                            const mp_plan_opts* opts, void* stream, mp_plan** out) {
    if (!out || !rowptr || !plan_buf) return MP_ERR_NULL;
    if (!valid_itype(rowptr_itype) || !valid_dtype(x_dtype)) return MP_ERR_DTYPE;
    if (N_dst < 0 || N_dst > INT32_MAX || E < 0 || E > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    const mp_plan_opts o = opts ? *opts : mp_plan_opts{0, 0, 0};
    if (o.small_max < 0 || o.hub_min < 0 || o.chunk_min < 0 || o.chunk_min > INT32_MAX)
        return MP_ERR_SIZE;
    PlanLayout L = plan_layout(plan_buf, N_dst);
    if (plan_bytes < L.bytes) return MP_ERR_WORKSPACE;
    hipStream_t s = as_stream(stream);
    const int rp64 = rowptr_itype == MP_I64;

    mp_plan* p = new (std::nothrow) mp_plan{};
    if (!p) return MP_ERR_SIZE;
    p->rowptr = rowptr;
    p->itype = rowptr_itype;
    p->N_dst = N_dst;
    p->E = E;
    p->F = F;
    p->x_dtype = x_dtype;
    // rows of up to 16 edges per slot get one slot; longer rows a wavefront.  Where
    // rows may be cut into narrow or wide chunks (wide_rows), each has its
    // limit; of up to 32 features, wide ones are taken only where no or few rows
    // have 64 edges, and all others are small then
    const Geometry nar = make_geometry(F, x_dtype, 16, false);
    const Geometry wid = make_geometry(F, x_dtype, 16, true);
    p->small_max = o.small_max > 0 ? o.small_max : 16 * (int64_t)nar.S;
    if (p->small_max > 16383) p->small_max = 16383;
    const int64_t split = p->small_max;
    if (o.small_max <= 0 && wid.wide) {
        const int64_t most = F < kWideAlways ? 63 : 16 * (int64_t)wid.S;
        if (p->small_max < most) p->small_max = most;
    }
    // a wavefront takes S * U edges per step; rows longer than 32 steps are
    // split into chunks of up to 32 steps (of the wide cut where the edges give
    // 4096 wavefronts that many), so that no wavefront runs a long chain of
    // dependent steps on its own
    auto unroll = [](const Geometry& g) { return (int64_t)(g.S * 8 > 64 ? 64 / g.S : 8); };
    const int64_t step_edges = nar.S * unroll(nar);
    const bool by_wide_cut = F >= kWideAlways && wide_rows(kUseAggregate, MP_SUM, F, x_dtype, 16,
                                                           RowLengths{N_dst, E, true, 0, 0});
    const int64_t wide_steps = by_wide_cut ? 32 * wid.S * unroll(wid) / step_edges : 32;
    const int64_t mean = N_dst > 0 ? E / N_dst : 0;
    const bool few_hubs = 32 * step_edges >= 4 * mean;  // long rows are the exception
    // Where the edges do not give enough wavefronts 32 steps, shorter chunks.
    // With few hubs the longest chain is the call's time: down to half the chain
    // of the small rows, 8 steps at least, and for rows of more than two of these
    // (power-law graph of 120k edges, F = 75: fp32 sum 28 -> 20 us, max 35 -> 25;
    // 325k edges, 61 a row, F = 171: the sum's training pass 62 -> 56; far below the
    // small rows' chain only the combining of the chunks adds, F = 20, 20k edges:
    // max 46 -> 49).  Where most rows are long, each chunk costs more than the filled
    // card gives: a quarter of the wavefronts (1024 segments of 500 rows, F = 100:
    // statistics 51 -> 40 us; of 2392 rows, F = 16, bf16: 91 -> 62)
    // (and of rows that go by the wide cut 8 of its steps, up to 32 narrow ones)
    int64_t least = few_hubs ? 8 * nar.S / unroll(nar) : 8;
    if (few_hubs && least < wide_steps / 4 && by_wide_cut)
        least = wide_steps / 4 < 32 ? wide_steps / 4 : 32;
    int64_t steps = E / ((few_hubs ? 4096 : 1024) * step_edges);
    if (steps < least) steps = least;
    steps = steps < 8 ? 8 : (steps > 32 ? 32 : steps);
    const int64_t by_wide = E / (4096 * step_edges);
    if (by_wide > steps) steps = by_wide < wide_steps ? by_wide : (wide_steps > steps ? wide_steps : steps);
    // -- as far as the partials stay within mp_spmm_noalloc's scratch whatever the
    // reduction (a hub's chunks are under twice its edges / chunk, a partial at
    // most 12 bytes per feature); explicit thresholds go with the most steps
    const int64_t cells = MP_NOALLOC_SCRATCH_BYTES / 12 - 256;
    const int64_t steps_fit = E * F / (cells / 2 * step_edges) + 1;
    if (steps < steps_fit) steps = steps_fit < wide_steps ? steps_fit : wide_steps;
    if (o.hub_min > 0 || o.chunk_min > 0) steps = wide_steps;
    p->chunk_min = (int)(o.chunk_min > 0 ? o.chunk_min : steps * step_edges);
    const bool soon = few_hubs && steps < 16 && 2 * steps * step_edges >= 2 * mean;
    const int64_t long_min = (steps > 32 ? steps : 32) * step_edges;
    p->hub_min = o.hub_min > 0 ? o.hub_min : (soon ? 2 * steps * step_edges : long_min);
    if (p->hub_min < p->small_max) p->hub_min = p->small_max;
    p->rowlist = L.rowlist;
    p->rowbeg = L.rowbeg;
    p->rowend = L.rowend;
    p->chunk_off = L.chunk_off;
    if (N_dst == 0) {
        *out = p;
        return MP_OK;
    }
    hipError_t e = launch_plan(PlanParams{rowptr, rp64, N_dst, split, p->small_max, p->hub_min, long_min,
                                          p->chunk_min, L.tile_cnt, L.rowlist, L.rowbeg, L.rowend,
                                          L.chunk_off, L.header},
                               s);
    uint32_t h[kPlanClasses + 3] = {0};
    if (e == hipSuccess) e = hipMemcpyAsync(h, L.header, sizeof(h), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        delete p;
        return MP_ERR_HIP;
    }
    p->hub_base = h[kClassHub];
    p->n_small = h[kClassMid];
    // the first class beyond `edges` edges (small rows: bit length, plus one beyond split)
    auto class_after = [&](int64_t edges) {
        int bits = 0;
        while (edges >> bits) ++bits;
        const int c = bits + 1;
        return c < kClassMid ? c : kClassMid;
    };
    p->n_small_narrow = h[class_after(split)];
    // (rows of 2^k edges and more have bit length k + 1: class k + 1, or k + 2)
    p->ge32 = N_dst - h[32 > split ? 7 : 6];
    p->ge64 = N_dst - h[64 > split ? 8 : 7];
    // tiny rows: the first classes (the list is sorted by class), if small
    p->n_tiny = h[kTinyClassEnd] < (uint32_t)p->n_small ? h[kTinyClassEnd] : p->n_small;
    p->n_hub = N_dst - p->hub_base;
    p->n_chunks = h[kPlanClasses + 1];
    // rows of more than two short chunks are hubs only where some row has more
    // than 32 steps: the combining is a launch more (160k edges, none such, F = 11:
    // mean and max 21.1 -> 17.9 us)
    if (soon && o.hub_min <= 0 && h[kPlanClasses + 2] == 0) {
        p->hub_base = N_dst;
        p->n_hub = p->n_chunks = 0;
    }
    *out = p;
    return MP_OK;
}

void mp_spmm_plan_free(mp_plan* plan) { delete plan; }

int mp_spmm_workspace(const mp_plan* plan, int reduce, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (!valid_reduce(reduce)) return MP_ERR_REDUCE;
    if (!plan || plan->n_chunks == 0) {
        *bytes = 0;
        return MP_OK;
    }
    const size_t cells = (size_t)plan->n_chunks * (size_t)plan->F;
    size_t b = 0;
    if (reduce & (MP_SUM | MP_MEAN)) b += align_up(cells * 4, 256);
    if (reduce & MP_MAX) b += 2 * align_up(cells * 4, 256);
    *bytes = b;
    return MP_OK;
}

int mp_spmm_multi_workspace(const mp_plan* plan, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (!plan || plan->n_chunks == 0) {
        *bytes = 0;
        return MP_OK;
    }
    // hub partials: sum, shifted sum and sum of squares, max and min values,
    // their positions
    *bytes = 7 * align_up((size_t)plan->n_chunks * (size_t)plan->F * 4, 256);
    return MP_OK;
}

int mp_spmm_multi(const mp_plan* plan, const void* rowptr, int rowptr_itype, const int32_t* col,
                  const float* w, const void* x, int x_dtype, int64_t N_src, int64_t N_dst,
                  int64_t F, int64_t ldx, int n_out, const mp_aggr_out* outs, void* ws,
                  size_t ws_bytes, void* stream) {
    if (N_dst > 0 && !col) return MP_ERR_NULL;
    return multi_impl(plan, rowptr, rowptr_itype, col, w, x, x_dtype, N_src, N_dst, F, ldx, n_out,
                      outs, ws, ws_bytes, as_stream(stream));
}

int mp_readout_multi(const mp_plan* plan, const void* ptr, int ptr_itype, const void* x,
                     int x_dtype, int64_t N_nodes, int64_t N_seg, int64_t F, int64_t ldx,
                     int n_out, const mp_aggr_out* outs, void* ws, size_t ws_bytes,
                     void* stream) {
    // segments of consecutive node rows: the CSR of the sorted batch vector,
    // whose column of position p is p itself
    return multi_impl(plan, ptr, ptr_itype, nullptr, nullptr, x, x_dtype, N_nodes, N_seg, F, ldx,
                      n_out, outs, ws, ws_bytes, as_stream(stream));
}

}  // extern "C"

// ---- mp_spmm_noalloc: hub partials in a static device array --------------------

// The workspace of mp_spmm_noalloc.  In host code its name is only the host
// stand-in of the device symbol: host code uses the address that
// hipGetSymbolAddress returns for the current device (each GPU holds its own
// copy), never the name.
static __device__ __align__(256) unsigned char scratch[MP_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of `scratch`, looked up once per device.
int noalloc_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return MP_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return MP_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return MP_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MP_OK;
}

}  // namespace

extern "C" {

int mp_spmm_noalloc(const mp_plan* plan, const void* rowptr, int rowptr_itype,
                    const int32_t* col, const float* w, const void* x, int x_dtype,
                    int64_t N_src, int64_t N_dst, int64_t F, int64_t ldx, int reduce, void* out,
                    int out_dtype, void* out_max, int max_dtype, int32_t* argout, void* stream) {
    if (N_dst > 0 && !col) return MP_ERR_NULL;
    size_t need = 0;
    int st = mp_spmm_workspace(plan, reduce, &need);
    if (st != MP_OK) return st;
    if (need > MP_NOALLOC_SCRATCH_BYTES) return MP_ERR_WORKSPACE;
    SpmmCall c{plan, rowptr, rowptr_itype, col, w, x, x_dtype, N_src, N_dst, F, ldx, reduce,
               out, out_dtype, out_max, max_dtype, argout, nullptr, 0};
    if (need > 0) {
        // every other argument is checked before the array is looked up; the
        // check only needs to know that a large enough workspace will come
        c.ws = &g_scratch_ptr;
        c.ws_bytes = MP_NOALLOC_SCRATCH_BYTES;
    }
    st = spmm_check(c);
    if (st != MP_OK) return st;
    if (need > 0 && N_dst > 0) {
        st = noalloc_scratch(&c.ws);
        if (st != MP_OK) return st;
    }
    return spmm_launch(c, as_stream(stream));
}

int mp_spmm(const mp_plan* plan, const void* rowptr, int rowptr_itype, const int32_t* col,
            const float* w, const void* x, int x_dtype, int64_t N_src, int64_t N_dst, int64_t F,
            int64_t ldx, int reduce, void* out, int out_dtype, void* out_max, int max_dtype,
            int32_t* argout, void* ws, size_t ws_bytes, void* stream) {
    if (N_dst > 0 && !col) return MP_ERR_NULL;
    SpmmCall c{plan, rowptr, rowptr_itype, col, w, x, x_dtype, N_src, N_dst, F, ldx, reduce,
               out, out_dtype, out_max, max_dtype, argout, ws, ws_bytes};
    const int st = spmm_check(c);
    return st != MP_OK ? st : spmm_launch(c, as_stream(stream));
}

// ---- backward ------------------------------------------------------------------

int mp_csr_transpose_workspace(int64_t E, int64_t N_src, int rowptrT_itype, int with_payload,
                               size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (!valid_itype(rowptrT_itype)) return MP_ERR_DTYPE;
    int st = check_csr_sizes(E, N_src);
    if (st != MP_OK) return st;
    if (E == 0) {
        *bytes = 0;
        return MP_OK;
    }
    *bytes = align_up((size_t)E * 4, 256) + csr_layout(nullptr, E, N_src, with_payload ? 1 : 0).bytes;
    return MP_OK;
}

int mp_csr_transpose(const void* rowptr, int rowptr_itype, const int32_t* col, int64_t N_dst,
                     int64_t N_src, int64_t E, void* rowptrT, int rowptrT_itype, int32_t* colT,
                     int32_t* posT, const float* val_in, float* val_out, void* ws,
                     size_t ws_bytes, int32_t* status, void* stream) {
    if (!valid_itype(rowptr_itype) || !valid_itype(rowptrT_itype)) return MP_ERR_DTYPE;
    int st = check_csr_sizes(E, N_src);
    if (st != MP_OK) return st;
    if (N_dst < 1 || N_dst > INT32_MAX) return MP_ERR_SIZE;
    if (!rowptr || !rowptrT) return MP_ERR_NULL;
    if (E > 0 && (!col || !colT || !ws)) return MP_ERR_NULL;
    if (E > 0 && (val_in == nullptr) != (val_out == nullptr)) return MP_ERR_NULL;
    if ((uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4) ||
        (uintptr_t)rowptrT % (rowptrT_itype == MP_I64 ? 8 : 4) || (uintptr_t)status % 4)
        return MP_ERR_ALIGN;
    hipStream_t s = as_stream(stream);
    if (E == 0) {
        hipError_t e = launch_fill_rowptr_zero(N_src, rowptrT, rowptrT_itype == MP_I64, s);
        if (e == hipSuccess) e = launch_status_ok(status, s);
        return hip_status(e);
    }
    size_t need = 0;
    mp_csr_transpose_workspace(E, N_src, rowptrT_itype, posT || val_out, &need);
    if (ws_bytes < need) return MP_ERR_WORKSPACE;
    // the forward CSR listed as COO (row of every position, col) is already in
    // position order, so a stable sort by col keeps forward order per source
    Carver c(ws);
    int32_t* row = c.take<int32_t>((size_t)E);
    if (launch_rows_of_edges(rowptr, rowptr_itype == MP_I64, N_dst, E, row, s) != hipSuccess)
        return MP_ERR_HIP;
    return coo_to_csr_impl(row, col, E, N_src, rowptrT, rowptrT_itype, colT, posT, val_in,
                           val_out, key_bits(N_dst), static_cast<char*>(ws) + c.off,
                           ws_bytes - c.off, status, s);
}

// Extra workspace of mp_spmm_backward_x beyond the aggregation's own: the
// fp32 grad_out / in-degree table (mean) or the win masks (max).
size_t backward_x_extra(int64_t N_dst, int64_t E, int64_t F, int reduce) {
    if (reduce == MP_MEAN) return align_up((size_t)N_dst * (size_t)F * 4, 256);
    // (at least one position's words: the gather may load word 0 unread)
    if (reduce == MP_MAX)
        return align_up((size_t)(E > 0 ? E : 1) * (size_t)win_mask_words(F) * 4, 256);
    return 0;
}

// The same for win records, never less than for the masks.
size_t win_records_bytes(int64_t E) { return align_up((size_t)E * kWinWords * 4, 256); }

// Records hold fp32 values; the masks' way reads a bf16 gradient as it is, half
// the bytes, which is ahead where few edges share a row's read and records are
// mostly empty (us by masks -> by records, four edges a row: 2M edges F = 7 151 ->
// 165, F = 12 160 -> 177, 8M edges F = 12 654 -> 746; eight edges a row: F = 5 94 ->
// 108, F = 13 126 -> 112).
static bool masks_for_bf16(int g_dtype, int64_t N_dst, int64_t E, int64_t F) {
    return g_dtype == MP_BF16 && (F < 8 || E < 6 * N_dst);
}

int mp_spmm_backward_x_workspace(const mp_plan* planT, int64_t N_dst, int64_t E, int64_t F,
                                 int reduce, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (reduce != MP_SUM && reduce != MP_MEAN && reduce != MP_MAX) return MP_ERR_REDUCE;
    if (N_dst < 0 || N_dst > INT32_MAX || E < 0 || E > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    size_t b = 0;
    int st = mp_spmm_workspace(planT, MP_SUM, &b);
    if (st != MP_OK) return st;
    const size_t extra = reduce == MP_MAX && use_win_records(N_dst, E, F)
                             ? win_records_bytes(E)
                             : backward_x_extra(N_dst, E, F, reduce);
    if (extra) b = align_up(b, 256) + extra;
    *bytes = b;
    return MP_OK;
}

int mp_spmm_backward_x(const mp_plan* planT, const void* rowptrT, int rowptrT_itype,
                       const int32_t* colT, const int32_t* posT, const float* wT,
                       const void* rowptr, int rowptr_itype, const int32_t* argout,
                       const void* grad_out, int g_dtype, int64_t N_dst, int64_t N_src, int64_t E,
                       int64_t F, int reduce, void* grad_x, int out_dtype, void* ws,
                       size_t ws_bytes, void* stream) {
    if (reduce != MP_SUM && reduce != MP_MEAN && reduce != MP_MAX) return MP_ERR_REDUCE;
    const bool need_rp = reduce != MP_SUM;
    if (!valid_itype(rowptrT_itype) || !valid_dtype(g_dtype) || !valid_dtype(out_dtype))
        return MP_ERR_DTYPE;
    if (need_rp && !valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    if (N_src < 0 || N_src > INT32_MAX || N_dst < 0 || N_dst > INT32_MAX || E < 0 ||
        E > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    if (!rowptrT) return MP_ERR_NULL;
    if (N_src > 0) {
        if (!colT || !grad_out || !grad_x) return MP_ERR_NULL;
        if (need_rp && !rowptr) return MP_ERR_NULL;
        if (reduce == MP_MAX && (!argout || !posT)) return MP_ERR_NULL;
    }
    int st = check_plan(planT, rowptrT, rowptrT_itype, N_src, F);
    if (st != MP_OK) return st;
    if (planT && planT->E != E) return MP_ERR_PLAN;
    const int eb = g_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)grad_out % eb || (uintptr_t)rowptrT % (rowptrT_itype == MP_I64 ? 8 : 4) ||
        (uintptr_t)colT % 4 || (uintptr_t)posT % 4 || (uintptr_t)wT % 4 ||
        (uintptr_t)argout % 4 || (uintptr_t)grad_x % (out_dtype == MP_BF16 ? 2 : 4) ||
        (need_rp && (uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4)))
        return MP_ERR_ALIGN;
    // workspace: the aggregation's hub partials, then the reduction's extra
    size_t part = 0;
    mp_spmm_workspace(planT, MP_SUM, &part);
    const size_t extra = backward_x_extra(N_dst, E, F, reduce);
    if (extra) {
        part = align_up(part, 256);
        if (ws_bytes < part + extra || !ws) return MP_ERR_WORKSPACE;
    }
    if (N_src == 0) return MP_OK;
    hipStream_t s = as_stream(stream);
    const void* table = grad_out;
    int t_dtype = g_dtype;
    void* spmm_ws = ws;
    size_t spmm_ws_bytes = extra ? part : ws_bytes;
    char* extra_buf = extra ? static_cast<char*>(ws) + part : nullptr;
    if (reduce == MP_MEAN) {
        // mean: a sum over the transposed CSR of grad_out / in-degree
        float* scaled = reinterpret_cast<float*>(extra_buf);
        if (launch_scale_inv_deg(grad_out, g_dtype == MP_BF16, rowptr, rowptr_itype == MP_I64,
                                 N_dst, F, scaled, s) != hipSuccess)
            return MP_ERR_HIP;
        table = scaled;
        t_dtype = MP_F32;
    }
    uint32_t* mbits = nullptr;
    // (a workspace with room for the masks alone gets the masks)
    const bool records = reduce == MP_MAX && use_win_records(N_dst, E, F) &&
                         !masks_for_bf16(g_dtype, N_dst, E, F) &&
                         ws_bytes >= part + win_records_bytes(E);
    if (reduce == MP_MAX) {
        // max: the wins of every forward position, then a sum over the
        // transposed CSR of the features each edge wins
        mbits = reinterpret_cast<uint32_t*>(extra_buf);
        if (records) {
            if (launch_win_records(rowptr, rowptr_itype == MP_I64, argout, grad_out,
                                   g_dtype == MP_BF16, N_dst, E, F, mbits, s) != hipSuccess)
                return MP_ERR_HIP;
        } else if (E > 0 && launch_win_masks(rowptr, rowptr_itype == MP_I64, argout, N_dst, F, mbits,
                                             s) != hipSuccess) {
            return MP_ERR_HIP;
        }
    }
    // (a lane's win-mask bits must lie in one word)
    const bool masked = reduce == MP_MAX && !records;
    Geometry g = make_geometry(
        F, t_dtype, (uintptr_t)table,
        !masked && wide_rows(kUseAggregate, MP_SUM, F, t_dtype, (uintptr_t)table,
                             row_lengths(planT, N_src)));
    SpmmParams P{};
    P.rowptr = rowptrT;
    P.rp64 = rowptrT_itype == MP_I64;
    P.col = colT;
    P.w = wT;
    P.n_tables = 1;
    P.table_ptr[0] = static_cast<const char*>(table);
    P.F = F;
    P.off32 = fits_off32(N_dst, F, t_dtype == MP_BF16 ? 2 : 4);
    P.reduce = MP_SUM;
    P.out = grad_x;
    P.out_bf16 = out_dtype == MP_BF16;
    if (records) {
        P.ekey = posT;
        P.recs = mbits;
        P.win_arg = argout;
        P.win_g = grad_out;
        P.win_g_bf16 = g_dtype == MP_BF16;
    } else if (reduce == MP_MAX) {
        P.ekey = posT;
        P.mbits = mbits;
        P.mw = win_mask_words(F);
    }
    return run_spmm(planT, P, g, t_dtype, N_src, spmm_ws, spmm_ws_bytes, s);
}

int mp_spmm_backward_w_workspace(int64_t E, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (E < 0 || E > INT32_MAX) return MP_ERR_SIZE;
    *bytes = E == 0 ? 0 : align_up((size_t)E * 4, 256);
    return MP_OK;
}

int mp_spmm_backward_w(const void* rowptr, int rowptr_itype, const int32_t* col, const void* x,
                       int x_dtype, const void* grad_out, int g_dtype, const int32_t* argout,
                       int64_t N_src, int64_t N_dst, int64_t E, int64_t F, int reduce,
                       float* grad_w, void* ws, size_t ws_bytes, void* stream) {
    if (reduce != MP_SUM && reduce != MP_MEAN && reduce != MP_MAX) return MP_ERR_REDUCE;
    if (!valid_itype(rowptr_itype) || !valid_dtype(x_dtype) || !valid_dtype(g_dtype))
        return MP_ERR_DTYPE;
    if (N_src < 0 || N_src > INT32_MAX || N_dst < 1 || N_dst > INT32_MAX || E < 0 ||
        E > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    if (!rowptr) return MP_ERR_NULL;
    if (E == 0) return MP_OK;
    if (!col || !x || !grad_out || !grad_w || !ws) return MP_ERR_NULL;
    if (reduce == MP_MAX && !argout) return MP_ERR_NULL;
    if (ws_bytes < align_up((size_t)E * 4, 256)) return MP_ERR_WORKSPACE;
    const int ex = x_dtype == MP_BF16 ? 2 : 4, eg = g_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4) || (uintptr_t)col % 4 ||
        (uintptr_t)x % ex || (uintptr_t)grad_out % eg || (uintptr_t)argout % 4 ||
        (uintptr_t)grad_w % 4)
        return MP_ERR_ALIGN;
    hipStream_t s = as_stream(stream);
    int32_t* row = static_cast<int32_t*>(ws);
    if (launch_rows_of_edges(rowptr, rowptr_itype == MP_I64, N_dst, E, row, s) != hipSuccess)
        return MP_ERR_HIP;
    // one lane-chunk of EPL elements per table: x's vector width must keep
    // every table's chunk aligned (g and argout scaled to x's element size)
    uintptr_t al = (uintptr_t)x;
    al |= eg == ex ? (uintptr_t)grad_out : (eg > ex ? (uintptr_t)grad_out >> 1 : (uintptr_t)grad_out << 1);
    if (reduce == MP_MAX) al |= ex == 4 ? (uintptr_t)argout : (uintptr_t)argout >> 1;
    Geometry g = make_geometry(F, x_dtype, al, wide_rows(kUseDot, 0, F, x_dtype, al,
                                                        RowLengths{N_dst, E, false, 0, 0}));
    GradWParams P{};
    P.rowptr = rowptr;
    P.rp64 = rowptr_itype == MP_I64;
    P.col = col;
    P.row = row;
    P.x = x;
    P.g = grad_out;
    P.argout = argout;
    P.F = F;
    P.E = E;
    P.L = g.L;
    P.S = g.S;
    P.FT = g.FT;
    P.ltot = g.ltot;
    P.reduce = reduce;
    P.grad_w = grad_w;
    return hip_status(launch_spmm_grad_w(P, x_dtype, g_dtype, g.epl, s));
}

// ---- feature-table layout --------------------------------------------------------

int mp_copy_rows(const void* in, int64_t ld_in, void* out, int64_t ld_out, int64_t N, int64_t F,
                 int dtype, void* stream) {
    if (!valid_dtype(dtype)) return MP_ERR_DTYPE;
    if (N < 0 || F < 1 || ld_in < F || ld_out < F) return MP_ERR_SIZE;
    if (N == 0) return MP_OK;
    if (!in || !out) return MP_ERR_NULL;
    const int eb = dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)in % eb || (uintptr_t)out % eb) return MP_ERR_ALIGN;
    return hip_status(launch_copy_rows(in, ld_in, out, ld_out, N, F, eb, as_stream(stream)));
}

// ---- edge-materialized messages ------------------------------------------------

int mp_csr_rows(const void* rowptr, int rowptr_itype, int64_t N_dst, int64_t E, int32_t* row,
                void* stream) {
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    if (N_dst < 1 || N_dst > INT32_MAX || E < 0 || E > INT32_MAX) return MP_ERR_SIZE;
    if (!rowptr || (E > 0 && !row)) return MP_ERR_NULL;
    if ((uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4) || (uintptr_t)row % 4)
        return MP_ERR_ALIGN;
    return hip_status(launch_rows_of_edges(rowptr, rowptr_itype == MP_I64, N_dst, E, row,
                                           as_stream(stream)));
}

int mp_message_gather(const int32_t* idx, const float* w, const void* x, int x_dtype,
                      int64_t N_src, int64_t E, int64_t F, void* msg, int msg_dtype,
                      void* stream) {
    MessageGather a{};
    const int st = gather_check(idx, w, x, x_dtype, N_src, E, F, msg, msg_dtype, &a);
    return st != MP_OK ? st : hip_status(launch_message_gather(a, as_stream(stream)));
}

int mp_message_scale(const float* in, float* out, int64_t E, int64_t F, const float* mask,
                     const int32_t* idx, int64_t n_mask, void* stream) {
    if (E < 0 || E > INT32_MAX || F < 1 || F > 65536 || n_mask < 0) return MP_ERR_SIZE;
    if (E == 0) return MP_OK;
    if (!in || !out || !mask) return MP_ERR_NULL;
    if (!idx && n_mask < E) return MP_ERR_SIZE;
    if ((uintptr_t)in % 4 || (uintptr_t)out % 4 || (uintptr_t)mask % 4 || (uintptr_t)idx % 4)
        return MP_ERR_ALIGN;
    const uintptr_t ptrs[2] = {(uintptr_t)in, (uintptr_t)out};
    const int sizes[2] = {4, 4};
    const int epl = message_epl(F, ptrs, sizes, 2, 4);
    return hip_status(launch_message_scale(in, out, mask, idx, E, F, epl, as_stream(stream)));
}

int mp_message_aggregate(const mp_plan* plan, const void* rowptr, int rowptr_itype,
                         const void* msg, int msg_dtype, int64_t E, int64_t N_dst, int64_t F,
                         int reduce, void* out, int out_dtype, void* out_max, int max_dtype,
                         int32_t* argout, void* ws, size_t ws_bytes, void* stream) {
    if (E < 0 || E > INT32_MAX) return MP_ERR_SIZE;
    SpmmCall c{plan, rowptr, rowptr_itype, nullptr, nullptr, msg, msg_dtype, E, N_dst, F, F,
               reduce, out, out_dtype, out_max, max_dtype, argout, ws, ws_bytes};
    const int st = spmm_check(c);
    return st != MP_OK ? st : spmm_launch(c, as_stream(stream));
}

int mp_spmm_materialized(const mp_plan* plan, const void* rowptr, int rowptr_itype,
                         const int32_t* col, const float* w, const void* x, int x_dtype,
                         int64_t N_src, int64_t N_dst, int64_t E, int64_t F, void* msg,
                         int msg_dtype, mp_message_fn c, void* user, int reduce, void* out,
                         int out_dtype, void* out_max, int max_dtype, int32_t* argout, void* ws,
                         size_t ws_bytes, void* stream) {
    if (E < 0 || E > INT32_MAX) return MP_ERR_SIZE;
    if (plan && plan->E != E) return MP_ERR_PLAN;
    MessageGather a{};
    int st = gather_check(col, w, x, x_dtype, N_src, E, F, msg, msg_dtype, &a);
    if (st != MP_OK) return st;
    SpmmCall agg{plan, rowptr, rowptr_itype, nullptr, nullptr, msg, msg_dtype, E, N_dst, F, F,
                 reduce, out, out_dtype, out_max, max_dtype, argout, ws, ws_bytes};
    st = spmm_check(agg);
    if (st != MP_OK) return st;
    hipStream_t s = as_stream(stream);
    if (launch_message_gather(a, s) != hipSuccess) return MP_ERR_HIP;
    if (c && c(msg, msg_dtype, E, F, user, stream) != 0) return MP_ERR_CALLBACK;
    return spmm_launch(agg, s);
}

int mp_message_backward_workspace(int64_t E, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (E < 0 || E > INT32_MAX) return MP_ERR_SIZE;
    *bytes = 0;  // the kernels need none
    return MP_OK;
}

int mp_message_backward(const void* rowptr, int rowptr_itype, const int32_t* argout,
                        const void* grad_out, int g_dtype, int64_t N_dst, int64_t E, int64_t F,
                        int reduce, float* dmsg, void* ws, size_t ws_bytes, void* stream) {
    if (reduce != MP_SUM && reduce != MP_MEAN && reduce != MP_MAX) return MP_ERR_REDUCE;
    if (!valid_itype(rowptr_itype) || !valid_dtype(g_dtype)) return MP_ERR_DTYPE;
    if (N_dst < 1 || N_dst > INT32_MAX || E < 0 || E > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    if (!rowptr) return MP_ERR_NULL;
    (void)ws;
    (void)ws_bytes;
    if (E == 0) return MP_OK;
    if (!grad_out || !dmsg) return MP_ERR_NULL;
    if (reduce == MP_MAX && !argout) return MP_ERR_NULL;
    const int eg = g_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4) || (uintptr_t)argout % 4 ||
        (uintptr_t)grad_out % eg || (uintptr_t)dmsg % 4)
        return MP_ERR_ALIGN;
    hipStream_t s = as_stream(stream);
    const uintptr_t ptrs[3] = {(uintptr_t)grad_out, (uintptr_t)dmsg,
                               reduce == MP_MAX ? (uintptr_t)argout : 0};
    const int sizes[3] = {eg, 4, 4};
    MessageBackward b{rowptr, rowptr_itype == MP_I64, argout, grad_out, g_dtype == MP_BF16,
                      N_dst, E, F, reduce, message_epl(F, ptrs, sizes, 3, 4), dmsg};
    return hip_status(launch_message_backward(b, s));
}

int mp_edge_dot(const void* a, int a_dtype, const void* b, int b_dtype, const int32_t* bidx,
                int64_t N_b, const int32_t* oidx, int64_t E, int64_t F, float* out,
                void* stream) {
    if (!valid_dtype(a_dtype) || !valid_dtype(b_dtype)) return MP_ERR_DTYPE;
    if (E < 0 || E > INT32_MAX || N_b < 0 || N_b > INT32_MAX || F < 1 || F > 65536)
        return MP_ERR_SIZE;
    if (!bidx && N_b < E) return MP_ERR_SIZE;
    if (E == 0) return MP_OK;
    if (!a || !b || !out) return MP_ERR_NULL;
    const int ea = a_dtype == MP_BF16 ? 2 : 4, eb = b_dtype == MP_BF16 ? 2 : 4;
    if ((uintptr_t)a % ea || (uintptr_t)b % eb || (uintptr_t)bidx % 4 || (uintptr_t)oidx % 4 ||
        (uintptr_t)out % 4)
        return MP_ERR_ALIGN;
    // one lane-chunk of EPL elements per table: b's vector width must keep a's
    // chunk aligned too (a's address scaled to b's element size)
    uintptr_t al = (uintptr_t)b;
    al |= ea == eb ? (uintptr_t)a : (ea > eb ? (uintptr_t)a >> 1 : (uintptr_t)a << 1);
    // (tables of one row per edge: no row's chunks are shared)
    Geometry g = make_geometry(F, b_dtype, al, wide_rows(kUseDot, 0, F, b_dtype, al,
                                                        RowLengths{0, E, false, 0, 0}));
    GradWParams P{};
    P.col = bidx;
    P.row = nullptr;
    P.x = b;
    P.g = a;
    P.F = F;
    P.E = E;
    P.L = g.L;
    P.S = g.S;
    P.FT = g.FT;
    P.ltot = g.ltot;
    P.reduce = MP_SUM;
    P.grad_w = out;
    P.oidx = oidx;
    return hip_status(launch_spmm_grad_w(P, b_dtype, a_dtype, g.epl, as_stream(stream)));
}

int mp_segment_matmul_workspace(int T, int64_t F, int64_t Fo, size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (T < 1 || T > MP_MAX_TYPES) return MP_ERR_SIZE;
    int st = gmm_dims(F, Fo);
    if (st != MP_OK) return st;
    *bytes = align_up((size_t)T * (size_t)F * (size_t)Fo * 2, 256);  // W transposed
    return MP_OK;
}

int mp_segment_matmul(const int64_t* seg, int T, const void* x, const void* W, int64_t F,
                      int64_t Fo, void* out, int out_dtype, void* ws, size_t ws_bytes,
                      void* stream) {
    if (!valid_dtype(out_dtype)) return MP_ERR_DTYPE;
    GmmParams P{};
    int64_t N = 0;
    int st = gmm_segments(seg, T, P, &N);
    if (st != MP_OK) return st;
    st = gmm_dims(F, Fo);
    if (st != MP_OK) return st;
    if (!W || !ws || (N > 0 && (!x || !out))) return MP_ERR_NULL;
    if ((uintptr_t)x % 16 || (uintptr_t)W % 16 || (uintptr_t)ws % 16 ||
        (uintptr_t)out % (out_dtype == MP_BF16 ? 2 : 4))
        return MP_ERR_ALIGN;
    size_t need = 0;
    mp_segment_matmul_workspace(T, F, Fo, &need);
    if (ws_bytes < need) return MP_ERR_WORKSPACE;
    hipStream_t s = as_stream(stream);
    uint16_t* Wt = static_cast<uint16_t*>(ws);
    if (launch_transpose_w(static_cast<const uint16_t*>(W), T, F, Fo, Wt, s) != hipSuccess)
        return MP_ERR_HIP;
    const int64_t ntn = ceil_div(Fo, gmm_tile_cols());
    int64_t tiles = 0;
    for (int t = 0; t < T; ++t) {
        P.tile_off[t] = tiles;
        tiles += ceil_div(seg[t + 1] - seg[t], gmm_tile_rows()) * ntn;
    }
    P.tile_off[T] = tiles;
    P.A = static_cast<const uint16_t*>(x);
    P.lda = F;
    P.K = F;
    P.B = Wt;
    P.ldb = F;
    P.b_stride = Fo * F;
    P.N = Fo;
    P.C = out;
    P.ldc = Fo;
    P.c_bf16 = out_dtype == MP_BF16;
    return hip_status(launch_gmm_nt(P, tiles, s));
}

int mp_segment_matmul_backward_workspace(const int64_t* seg, int T, int64_t F, int64_t Fo,
                                         size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    GmmParams P{};
    int64_t N = 0;
    int st = gmm_segments(seg, T, P, &N);
    if (st != MP_OK) return st;
    st = gmm_dims(F, Fo);
    if (st != MP_OK) return st;
    int64_t off[MP_MAX_TYPES + 1];
    const int64_t chunks = gmm_chunks(seg, T, off);
    *bytes = align_up((size_t)(chunks > 0 ? chunks : 1) * (size_t)F * (size_t)Fo * 4, 256);
    return MP_OK;
}

int mp_segment_matmul_backward(const int64_t* seg, int T, const void* x, const void* W,
                               const void* dout, int64_t F, int64_t Fo, void* dx, int dx_dtype,
                               float* dW, void* ws, size_t ws_bytes, void* stream) {
    if (!valid_dtype(dx_dtype)) return MP_ERR_DTYPE;
    GmmParams P{};
    int64_t N = 0;
    int st = gmm_segments(seg, T, P, &N);
    if (st != MP_OK) return st;
    st = gmm_dims(F, Fo);
    if (st != MP_OK) return st;
    if (!dx && !dW) return MP_ERR_NULL;
    if (N > 0 && !dout) return MP_ERR_NULL;
    if (dx && !W) return MP_ERR_NULL;
    if (dW && (!ws || (N > 0 && !x))) return MP_ERR_NULL;
    if ((uintptr_t)x % 16 || (uintptr_t)W % 16 || (uintptr_t)dout % 16 || (uintptr_t)ws % 16 ||
        (uintptr_t)dx % (dx_dtype == MP_BF16 ? 2 : 4) || (uintptr_t)dW % 4)
        return MP_ERR_ALIGN;
    hipStream_t s = as_stream(stream);
    if (dx && N > 0) {
        // dX = dOut W^T: W[t] stored [F][Fo] is already the transposed operand
        GmmParams Q = P;
        const int64_t ntn = ceil_div(F, gmm_tile_cols());
        int64_t tiles = 0;
        for (int t = 0; t < T; ++t) {
            Q.tile_off[t] = tiles;
            tiles += ceil_div(seg[t + 1] - seg[t], gmm_tile_rows()) * ntn;
        }
        Q.tile_off[T] = tiles;
        Q.A = static_cast<const uint16_t*>(dout);
        Q.lda = Fo;
        Q.K = Fo;
        Q.B = static_cast<const uint16_t*>(W);
        Q.ldb = Fo;
        Q.b_stride = F * Fo;
        Q.N = F;
        Q.C = dx;
        Q.ldc = F;
        Q.c_bf16 = dx_dtype == MP_BF16;
        if (launch_gmm_nt(Q, tiles, s) != hipSuccess) return MP_ERR_HIP;
    }
    if (dW) {
        size_t need = 0;
        mp_segment_matmul_backward_workspace(seg, T, F, Fo, &need);
        if (ws_bytes < need) return MP_ERR_WORKSPACE;
        const int64_t chunks = gmm_chunks(seg, T, P.tile_off);
        P.A = static_cast<const uint16_t*>(x);
        P.lda = F;
        P.B = static_cast<const uint16_t*>(dout);
        P.ldb = Fo;
        P.M = F;
        P.N = Fo;
        P.part = static_cast<float*>(ws);
        P.rows_per_chunk = kGmmRowsPerChunk;
        if (launch_gmm_weight_grad(P, chunks, dW, s) != hipSuccess) return MP_ERR_HIP;
    }
    return MP_OK;
}

// ---- heterogeneous ----------------------------------------------------------

static int hetero_check(int n_types, const int64_t* N_per_type, int n_rel, const mp_relation* rels,
                        int dst_type, int64_t* E_T, int64_t* offs, int64_t* N_rows) {
    if (!N_per_type || (n_rel > 0 && !rels)) return MP_ERR_NULL;
    const bool all = dst_type == MP_ALL_TYPES;
    if (n_types < 1 || n_types > MP_MAX_TYPES || n_rel < 0 ||
        (!all && (dst_type < 0 || dst_type >= n_types)))
        return MP_ERR_SIZE;
    int64_t tot = 0;
    for (int t = 0; t < n_types; ++t) {
        if (N_per_type[t] < 0) return MP_ERR_SIZE;
        offs[t] = tot;
        tot += N_per_type[t];
    }
    offs[n_types] = tot;
    if (tot > INT32_MAX) return MP_ERR_SIZE;
    int64_t e = 0;
    for (int r = 0; r < n_rel; ++r) {
        const mp_relation& R = rels[r];
        if (R.src_type < 0 || R.src_type >= n_types || R.dst_type < 0 || R.dst_type >= n_types ||
            R.E < 0)
            return MP_ERR_SIZE;
        if (all || R.dst_type == dst_type) {
            if (R.E > 0 && (!R.src || !R.dst)) return MP_ERR_NULL;
            e += R.E;
        }
    }
    if (e > INT32_MAX) return MP_ERR_SIZE;
    const int64_t rows = all ? tot : N_per_type[dst_type];
    if (rows < 1) return MP_ERR_SIZE;
    *E_T = e;
    *N_rows = rows;
    return MP_OK;
}

int mp_hetero_build_workspace(int n_types, const int64_t* N_per_type, int n_rel,
                              const mp_relation* rels, int dst_type, int rowptr_itype,
                              size_t* bytes) {
    if (!bytes) return MP_ERR_NULL;
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    int64_t E_T = 0, N_rows = 0, offs[MP_MAX_TYPES + 1];
    int st = hetero_check(n_types, N_per_type, n_rel, rels, dst_type, &E_T, offs, &N_rows);
    if (st != MP_OK) return st;
    size_t cw = 0;
    st = mp_coo_to_csr_workspace(E_T, N_rows, rowptr_itype, 0, &cw);
    if (st != MP_OK) return st;
    *bytes = 2 * align_up((size_t)(E_T > 0 ? E_T : 1) * 4, 256) + cw;
    return MP_OK;
}

int mp_hetero_build(int n_types, const int64_t* N_per_type, int n_rel, const mp_relation* rels,
                    int dst_type, void* rowptr, int rowptr_itype, int32_t* col, void* ws,
                    size_t ws_bytes, int32_t* status, void* stream) {
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    int64_t E_T = 0, N_rows = 0, offs[MP_MAX_TYPES + 1];
    int st = hetero_check(n_types, N_per_type, n_rel, rels, dst_type, &E_T, offs, &N_rows);
    if (st != MP_OK) return st;
    if (!rowptr || (E_T > 0 && (!col || !ws))) return MP_ERR_NULL;
    if ((uintptr_t)status % 4) return MP_ERR_ALIGN;
    size_t need = 0;
    st = mp_hetero_build_workspace(n_types, N_per_type, n_rel, rels, dst_type, rowptr_itype, &need);
    if (st != MP_OK) return st;
    if (ws_bytes < need) return MP_ERR_WORKSPACE;
    hipStream_t s = as_stream(stream);
    Carver c(ws);
    const size_t e = (size_t)(E_T > 0 ? E_T : 1);
    int32_t* src_g = c.take<int32_t>(e);
    int32_t* dst_c = c.take<int32_t>(e);
    int64_t off = 0;
    const bool all = dst_type == MP_ALL_TYPES;
    ConcatParams q{};
    q.src_out = src_g;
    q.dst_out = dst_c;
    for (int r = 0; r < n_rel; ++r) {
        const mp_relation& R = rels[r];
        if ((!all && R.dst_type != dst_type) || R.E == 0) continue;
        // sources (and, over all types, destinations) as global node ids
        q.src[q.n] = R.src;
        q.dst[q.n] = R.dst;
        q.E[q.n] = R.E;
        q.off[q.n] = off;
        q.src_add[q.n] = (int32_t)offs[R.src_type];
        q.dst_add[q.n] = all ? (int32_t)offs[R.dst_type] : 0;
        off += R.E;
        if (++q.n == kConcatMax) {
            if (launch_concat_relations(q, s) != hipSuccess) return MP_ERR_HIP;
            q.n = 0;
        }
    }
    if (q.n > 0 && launch_concat_relations(q, s) != hipSuccess) return MP_ERR_HIP;
    return coo_to_csr_impl(src_g, dst_c, E_T, N_rows, rowptr, rowptr_itype, col, nullptr,
                           nullptr, nullptr, 0, c.base + c.off, ws_bytes - c.off, status, s);
}

int mp_hetero_spmm(int n_types, const int64_t* N_per_type, const void* const* x_per_type,
                   int x_dtype, int64_t F, int dst_type, const mp_plan* plan, const void* rowptr,
                   int rowptr_itype, const int32_t* col, int reduce, void* out, int out_dtype,
                   void* ws, size_t ws_bytes, void* stream) {
    if (reduce != MP_SUM) return MP_ERR_REDUCE;
    if (!valid_itype(rowptr_itype) || !valid_dtype(x_dtype) || !valid_dtype(out_dtype))
        return MP_ERR_DTYPE;
    int64_t E_T = 0, N_dst = 0, offs[MP_MAX_TYPES + 1];
    int st = hetero_check(n_types, N_per_type, 0, nullptr, dst_type, &E_T, offs, &N_dst);
    if (st != MP_OK) return st;
    if (F < 1 || F > 65536) return MP_ERR_SIZE;
    if (!x_per_type || !rowptr || !out || !col) return MP_ERR_NULL;
    st = check_plan(plan, rowptr, rowptr_itype, N_dst, F);
    if (st != MP_OK) return st;
    const int eb = x_dtype == MP_BF16 ? 2 : 4;
    uintptr_t xa = 0;
    for (int t = 0; t < n_types; ++t) {
        if (N_per_type[t] > 0 && !x_per_type[t]) return MP_ERR_NULL;
        if ((uintptr_t)x_per_type[t] % eb) return MP_ERR_ALIGN;
        xa |= (uintptr_t)x_per_type[t];
    }
    if ((uintptr_t)out % (out_dtype == MP_BF16 ? 2 : 4) || (uintptr_t)col % 4 ||
        (uintptr_t)rowptr % (rowptr_itype == MP_I64 ? 8 : 4))
        return MP_ERR_ALIGN;
    Geometry g = make_geometry(F, x_dtype, xa,
                               wide_rows(kUseAggregate, reduce, F, x_dtype, xa,
                                         row_lengths(plan, N_dst)));
    SpmmParams P{};
    P.rowptr = rowptr;
    P.rp64 = rowptr_itype == MP_I64;
    P.col = col;
    P.w = nullptr;
    // tables laid out back to back in one allocation (one typed feature
    // tensor) are a single table indexed by global id
    bool contiguous = true;
    for (int t = 1; t < n_types; ++t)
        if ((uintptr_t)x_per_type[t] != (uintptr_t)x_per_type[0] + (uintptr_t)(offs[t] * F * eb))
            contiguous = false;
    P.n_tables = contiguous ? 1 : n_types;
    for (int t = 0; t < n_types; ++t) {
        P.table_ptr[t] = static_cast<const char*>(x_per_type[t]);
        P.table_off[t] = offs[t];
        P.voff[t] = ((int64_t)(uintptr_t)x_per_type[t] - (int64_t)(uintptr_t)x_per_type[0]) -
                    offs[t] * F * eb;
    }
    P.table_off[n_types] = offs[n_types];
    P.F = F;
    P.reduce = reduce;
    P.out = out;
    P.out_bf16 = out_dtype == MP_BF16;
    return run_spmm(plan, P, g, x_dtype, N_dst, ws, ws_bytes, as_stream(stream));
}

int mp_probe_read(const void* p, int64_t bytes, uint32_t* sink, void* stream) {
    if (!p || !sink) return MP_ERR_NULL;
    if (bytes < 16 || bytes % 16) return MP_ERR_SIZE;
    if ((uintptr_t)p % 16 || (uintptr_t)sink % 4) return MP_ERR_ALIGN;
    return hip_status(launch_probe_read(p, bytes / 16, sink, as_stream(stream)));
}

int mp_probe_copy(const void* in, void* out, int64_t bytes, void* stream) {
    if (!in || !out) return MP_ERR_NULL;
    if (bytes < 16 || bytes % 16) return MP_ERR_SIZE;
    if ((uintptr_t)in % 16 || (uintptr_t)out % 16) return MP_ERR_ALIGN;
    return hip_status(launch_probe_copy(in, out, bytes / 16, as_stream(stream)));
}

int mp_probe_gather(const int32_t* idx, int64_t n, const void* table, int64_t stride_bytes,
                    int64_t row_bytes, uint32_t* sink, void* stream) {
    if (!sink || (n > 0 && (!idx || !table))) return MP_ERR_NULL;
    if (n < 0 || n > INT32_MAX || row_bytes < 16 || row_bytes > 1024 || row_bytes % 16 ||
        stride_bytes < row_bytes)
        return MP_ERR_SIZE;
    if ((uintptr_t)table % 16 || stride_bytes % 16 || (uintptr_t)idx % 4 || (uintptr_t)sink % 4)
        return MP_ERR_ALIGN;
    if (n == 0) return MP_OK;
    return hip_status(launch_probe_gather(idx, n, table, stride_bytes, (int)(row_bytes / 16), sink,
                                          as_stream(stream)));
}

int mp_probe_scatter(const void* in, const int32_t* dest, int64_t n, int64_t elem_bytes, void* out,
                     void* stream) {
    if (n > 0 && (!in || !dest || !out)) return MP_ERR_NULL;
    if (n < 0 || n > INT32_MAX || (elem_bytes != 4 && elem_bytes != 8)) return MP_ERR_SIZE;
    if ((uintptr_t)in % elem_bytes || (uintptr_t)out % elem_bytes || (uintptr_t)dest % 4)
        return MP_ERR_ALIGN;
    if (n == 0) return MP_OK;
    return hip_status(launch_probe_scatter(in, dest, n, (int)elem_bytes, out, as_stream(stream)));
}

int mp_validate_coo(const int32_t* src, const int32_t* dst, int64_t E, int64_t N_src,
                    int64_t N_dst, int64_t* d_count, void* stream) {
    if (!d_count || (E > 0 && (!src || !dst))) return MP_ERR_NULL;
    if (E < 0 || N_src < 0 || N_dst < 0) return MP_ERR_SIZE;
    return hip_status(launch_validate_coo(src, dst, E, N_src, N_dst, d_count, as_stream(stream)));
}

int mp_validate_sorted(const int32_t* dst, int64_t E, int64_t* d_count, void* stream) {
    if (!d_count || (E > 0 && !dst)) return MP_ERR_NULL;
    if (E < 0) return MP_ERR_SIZE;
    return hip_status(launch_validate_sorted(dst, E, d_count, as_stream(stream)));
}

int mp_validate_csr(const void* rowptr, int rowptr_itype, const int32_t* col, int64_t N_dst,
                    int64_t N_src, int64_t E, int64_t* d_count, void* stream) {
    if (!d_count || !rowptr || (E > 0 && !col)) return MP_ERR_NULL;
    if (!valid_itype(rowptr_itype)) return MP_ERR_DTYPE;
    if (E < 0 || N_src < 0 || N_dst < 0) return MP_ERR_SIZE;
    return hip_status(launch_validate_csr(rowptr, rowptr_itype == MP_I64, col, N_dst, N_src, E,
                                          d_count, as_stream(stream)));
}

}  // extern "C"
