// Backward pass of the aggregation (Sec. 2.2 of PyG 2.0: the gradient of an
// aggregation over A runs over the transposed adjacency, which the library
// builds once as a source-major CSR, the analogue of the cached CSC).
//
//   * rows_of_edges: the destination row of every forward CSR position (the
//     keys the transposed CSR is sorted by carry it as payload), by merged
//     ranges of rows and positions.
//   * scale_inv_deg: grad_out / in-degree per destination row, the input of
//     the gradient of mean.
//   * spmm_grad_w: the gradient with respect to the edge weights, one dot
//     product of grad_out[v] and x[col[p]] per CSR edge p of row v (a
//     sampled dense-dense product).  Edge-parallel: every wavefront takes 64
//     consecutive CSR positions, so hub rows need no special handling; the
//     per-edge dots are reduced over the lanes of a slot by recursive
//     halving, a fixed pattern.  With
//     the row or column array absent (position p reads row p) the same kernel
//     gives the per-edge dot products of the edge-materialized path.
//   * win_masks: for the gradient of max, the features each forward edge
//     wins (one bit per feature), so that the masked sum over the transposed
//     CSR reads one mask word per edge and lane instead of the argmax chunk
//     of the edge's destination row.
//   * win_records + win_gather: the same where edges win few features: the
//     routed gradient values travel with the edge, so that the sum over the
//     transposed CSR makes one scattered read per edge.
//
// The gradient with respect to x reuses the aggregation kernels of spmm.hip
// over the transposed CSR (sum, mean after scale_inv_deg, and a masked sum
// for max).
#include <type_traits>

#include "mp_internal.hpp"

namespace mp {
namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
#ifndef MP_GW_UNROLL
#define MP_GW_UNROLL 4  // edges per slot per step of the weight gradient (sum, mean)
#endif

__device__ inline int64_t rp_at(const void* rp, int rp64, int64_t i) {
    return rp64 ? static_cast<const int64_t*>(rp)[i] : (int64_t) static_cast<const int32_t*>(rp)[i];
}

// row[p] = the v with rowptr[v] <= p < rowptr[v+1]: the number of rows that end
// at or before p.  Bound by the 4-byte stores and the 4 or 8 bytes of every
// row's bound.  By merged ranges, as neither fixed rows nor fixed positions a
// wavefront bound its work (us: 64 rows a wavefront; 256 or 1024 positions;
// merged):
//   124M edges over 2.4M rows      171   183   176
//   power law, 1.2M, a row of 36k  240     8     9
//   1M edges over 1M rows            7    17    10
//   300k edges over 20k rows        10     5     5
//   50k edges over 1M rows           6   489     8
//   300 edges over 16k rows          5   883     8
// Bounds are clamped to [0, E], the last row's is E, so ids lie below N whatever
// the input (an inconsistent rowptr only makes ids wrong).
template <typename IT>
struct RowEnds {
    const IT* rowptr;
    int64_t N, E;
    __device__ inline int64_t operator()(int64_t i) const { return row_bound(rowptr, N, E, i + 1); }
};

template <typename IT, bool VEC, int SPAN>
__global__ __launch_bounds__(kMergeBlock) void rows_of_edges(const IT* __restrict__ rowptr, int64_t N,
                                                             int64_t E, int32_t* __restrict__ row) {
    merge_counts<SPAN, VEC>(RowEnds<IT>{rowptr, N, E}, N - 1, E, row);
}

__device__ inline float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// fp32 -> bf16 bits, round to nearest even (finite values).
__device__ inline uint16_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// out[v, f] = g[v, f] / deg(v) in fp32 (0 for an empty row).  Each thread
// takes V consecutive elements of one row (V divides F); the row index uses
// 32-bit division when the table has under 2^32 elements.
template <bool GB, int V>
__global__ __launch_bounds__(kBlock) void scale_inv_deg(const void* __restrict__ g,
                                                        const void* __restrict__ rowptr, int rp64,
                                                        int64_t N, int64_t F,
                                                        float* __restrict__ out) {
    const int64_t n = N * F;
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * V;
    if (i >= n) return;
    const int64_t v = n <= (int64_t)UINT32_MAX ? (int64_t)((uint32_t)i / (uint32_t)F) : i / F;
    const int64_t deg = rp_at(rowptr, rp64, v + 1) - rp_at(rowptr, rp64, v);
    float gv[V];
    if constexpr (GB) {
        const uint16_t* gb = static_cast<const uint16_t*>(g) + i;
        if constexpr (V == 4) {
            const uint2 u = *reinterpret_cast<const uint2*>(gb);
            gv[0] = bf16_bits_to_f32(u.x & 0xFFFFu); gv[1] = __uint_as_float(u.x & 0xFFFF0000u);
            gv[2] = bf16_bits_to_f32(u.y & 0xFFFFu); gv[3] = __uint_as_float(u.y & 0xFFFF0000u);
        } else {
            gv[0] = bf16_bits_to_f32(gb[0]);
        }
    } else {
        const float* gf = static_cast<const float*>(g) + i;
        if constexpr (V == 4) {
            const float4 a = *reinterpret_cast<const float4*>(gf);
            gv[0] = a.x; gv[1] = a.y; gv[2] = a.z; gv[3] = a.w;
        } else {
            gv[0] = gf[0];
        }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) gv[k] = deg > 0 ? gv[k] / (float)deg : 0.f;
    if constexpr (V == 4)
        *reinterpret_cast<float4*>(out + i) = make_float4(gv[0], gv[1], gv[2], gv[3]);
    else
        out[i] = gv[0];
}

// bits[p * MW + w], bit b: feature f = 32 w + b of row v = row(p) has its
// maximum at CSR position p (argout[v, f] == p).  A wavefront takes
// kMaskRows consecutive rows, whose row ranges and first argout loads are
// issued together (a row's own work is short next to a memory round trip).
// The features go in pairs of 64-feature tiles (two argout values per lane,
// up to four words per position); a row's positions in chunks of 64.  For
// each chunk the wavefront clears 4 LDS words per position, every feature
// whose winner lies in the chunk ORs its bit into its winner's word (an
// integer OR, so the order does not matter), and lane i stores the words of
// position i.  Every word of every position is written exactly once.  The
// LDS region is the wavefront's own; LDS operations of one wavefront execute
// in program order, so no barrier is needed.
constexpr int kMaskRows = 4;

template <typename IT>
__global__ __launch_bounds__(kBlock) void win_masks(const IT* __restrict__ rowptr,
                                                    const int32_t* __restrict__ argout, int64_t N,
                                                    int64_t F, int64_t MW,
                                                    uint32_t* __restrict__ bits) {
    __shared__ __align__(16) uint32_t lds[kWavesPerBlock][kWave * 4];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = threadIdx.x / kWave;
    const int64_t v0 =
        (__builtin_amdgcn_readfirstlane(wid) + (int64_t)blockIdx.x * kWavesPerBlock) * kMaskRows;
    if (v0 >= N) return;
    uint32_t* my = lds[wid];
    int64_t rb[kMaskRows + 1];
#pragma unroll
    for (int i = 0; i <= kMaskRows; ++i) rb[i] = (int64_t)rowptr[v0 + i < N ? v0 + i : N];
    // features f0 + lane and f0 + 64 + lane (clamped to the row, masked below)
    const int64_t la = lane < F ? lane : F - 1;
    const int64_t lb = kWave + lane < F ? kWave + lane : F - 1;
    int32_t a0[kMaskRows], b0[kMaskRows];
#pragma unroll
    for (int i = 0; i < kMaskRows; ++i) {
        const int64_t v = v0 + i < N ? v0 + i : N - 1;
        a0[i] = argout[v * F + la];
        b0[i] = argout[v * F + lb];
    }
    const uint32_t bit = 1u << (lane & 31);
    const int half = lane >> 5;
#pragma unroll
    for (int i = 0; i < kMaskRows; ++i) {
        const int64_t v = v0 + i;
        const int64_t beg = rb[i];
        const int64_t deg = rb[i + 1] - beg;
        if (v >= N || deg <= 0) continue;
        for (int64_t f0 = 0; f0 < F; f0 += 2 * kWave) {
            // winners of features f0 + lane and f0 + 64 + lane, relative to
            // the row start (-1: no such feature)
            const int64_t fa = f0 + lane, fb = f0 + kWave + lane;
            int32_t aa = a0[i], ab = b0[i];
            if (f0 > 0) {
                aa = argout[v * F + (fa < F ? fa : F - 1)];
                ab = argout[v * F + (fb < F ? fb : F - 1)];
            }
            const int64_t ra = fa < F ? (int64_t)aa - beg : -1;
            const int64_t rbv = fb < F ? (int64_t)ab - beg : -1;
            const int64_t w0 = f0 >> 5;  // a multiple of 4
            const int nw = (int)(MW - w0 < 4 ? MW - w0 : 4);
            for (int64_t c0 = 0; c0 < deg; c0 += kWave) {
                const int n = (int)(deg - c0 < kWave ? deg - c0 : kWave);
                const int64_t qa = ra - c0, qb = rbv - c0;
                *reinterpret_cast<uint4*>(my + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
                __builtin_amdgcn_wave_barrier();
                if (qa >= 0 && qa < n) atomicOr(my + 4 * qa + half, bit);
                if (qb >= 0 && qb < n) atomicOr(my + 4 * qb + 2 + half, bit);
                __builtin_amdgcn_wave_barrier();
                if (lane < n) {
                    const uint4 r = *reinterpret_cast<const uint4*>(my + 4 * lane);
                    uint32_t* o = bits + (beg + c0 + lane) * MW + w0;
                    if (nw == 4 && (MW & 3) == 0) {
                        *reinterpret_cast<uint4*>(o) = r;  // 16-byte aligned
                    } else {
                        o[0] = r.x;
                        if (nw > 1) o[1] = r.y;
                        if (nw > 2) o[2] = r.z;
                        if (nw > 3) o[3] = r.w;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

// ---- gradient of max by win records ------------------------------------------
//
// A record of 32 bytes per forward CSR position: words 0..5 the routed values
// G[v, f] (fp32) of the first six features f that the position's edge wins, in
// feature order; bytes 24..29 their feature ids; byte 30 zero; byte 31 the
// number of wins (at most 255).

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4w __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kRecRows = 4;        // consecutive rows of a wavefront
constexpr int kRecPart = 1024;     // positions of a row that its own wavefront writes

__device__ inline float grad_at(const void* g, int g_bf16, int64_t i) {
    return g_bf16 ? bf16_bits_to_f32(static_cast<const uint16_t*>(g)[i])
                  : static_cast<const float*>(g)[i];
}

// Bound by its traffic (argout and g read once, 32 bytes written per edge).
// As in win_masks, a wavefront takes kRecRows consecutive rows with their
// first loads in flight together and walks a row's positions in chunks of 64:
// every feature ORs its bit into its winner's mask (LDS, order-free), and then
// its rank among the winner's features, the bits below its own, is its value's
// place in the record.  The chunk's 64 records leave LDS in 16-byte stores.
// A row's positions beyond the first kRecPart go to further wavefronts, as in
// message_backward.  124M edges, F = 100: 1160 us (masks alone: 740 us).
template <typename IT>
__global__ __launch_bounds__(kBlock) void win_records(const IT* __restrict__ rowptr,
                                                      const int32_t* __restrict__ argout,
                                                      const void* __restrict__ g, int g_bf16,
                                                      int64_t N, int64_t E, int64_t F,
                                                      uint32_t* __restrict__ recs) {
    __shared__ __align__(16) uint32_t s_mask[kWavesPerBlock][kWave * 4];
    __shared__ __align__(16) uint32_t s_rec[kWavesPerBlock][kWave * kWinWords];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int64_t wv = wid + (int64_t)blockIdx.x * kWavesPerBlock;
    const int64_t row_waves = (N + kRecRows - 1) / kRecRows;
    uint32_t* const mask = s_mask[wid];
    uint32_t* const rec = s_rec[wid];
    uint8_t* const rec8 = reinterpret_cast<uint8_t*>(rec);
    const uint32_t bit = 1u << (lane & 31);
    const int half = lane >> 5;

    // positions [c0, c1) of row v, relative to its start beg; a0, b0, ga0,
    // gb0: argout and g of the features lane and 64 + lane
    auto span = [&](int64_t v, int64_t beg, int64_t c0, int64_t c1, int32_t a0, int32_t b0,
                    float ga0, float gb0) {
        for (; c0 < c1; c0 += kWave) {
            const int n = (int)(c1 - c0 < kWave ? c1 - c0 : kWave);
            *reinterpret_cast<uint4*>(rec + 8 * lane) = make_uint4(0u, 0u, 0u, 0u);
            *reinterpret_cast<uint4*>(rec + 8 * lane + 4) = make_uint4(0u, 0u, 0u, 0u);
            for (int64_t f0 = 0; f0 < F; f0 += 2 * kWave) {
                const int64_t fa = f0 + lane, fb = f0 + kWave + lane;
                int32_t aa = a0, ab = b0;
                float ga = ga0, gb = gb0;
                if (f0 > 0) {
                    const int64_t ia = v * F + (fa < F ? fa : F - 1);
                    const int64_t ib = v * F + (fb < F ? fb : F - 1);
                    aa = argout[ia];
                    ab = argout[ib];
                    ga = grad_at(g, g_bf16, ia);
                    gb = grad_at(g, g_bf16, ib);
                }
                // winners relative to the chunk (outside 0..n-1: not here)
                const int64_t qa = fa < F ? (int64_t)aa - beg - c0 : -1;
                const int64_t qb = fb < F ? (int64_t)ab - beg - c0 : -1;
                const bool ina = qa >= 0 && qa < n, inb = qb >= 0 && qb < n;
                *reinterpret_cast<uint4*>(mask + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
                __builtin_amdgcn_wave_barrier();
                if (ina) atomicOr(mask + 4 * qa + half, bit);
                if (inb) atomicOr(mask + 4 * qb + 2 + half, bit);
                __builtin_amdgcn_wave_barrier();
                // a feature's place: the wins of earlier tiles (byte 31), then
                // the bits below its own
                if (ina) {
                    const uint4 m = *reinterpret_cast<const uint4*>(mask + 4 * qa);
                    const int r = rec8[32 * qa + 31] + (half ? __popc(m.x) : 0) +
                                  __popc((half ? m.y : m.x) & (bit - 1u));
                    if (r < kWinValues) {
                        rec[8 * qa + r] = __float_as_uint(ga);
                        rec8[32 * qa + 24 + r] = (uint8_t)fa;
                    }
                }
                if (inb) {
                    const uint4 m = *reinterpret_cast<const uint4*>(mask + 4 * qb);
                    const int r = rec8[32 * qb + 31] + __popc(m.x) + __popc(m.y) +
                                  (half ? __popc(m.z) : 0) +
                                  __popc((half ? m.w : m.z) & (bit - 1u));
                    if (r < kWinValues) {
                        rec[8 * qb + r] = __float_as_uint(gb);
                        rec8[32 * qb + 24 + r] = (uint8_t)fb;
                    }
                }
                __builtin_amdgcn_wave_barrier();
                {
                    const uint4 m = *reinterpret_cast<const uint4*>(mask + 4 * lane);
                    const int t = rec8[32 * lane + 31] + __popc(m.x) + __popc(m.y) + __popc(m.z) +
                                  __popc(m.w);
                    rec8[32 * lane + 31] = (uint8_t)(t < 255 ? t : 255);
                }
                __builtin_amdgcn_wave_barrier();
            }
            // (aligned to a word: wherever the caller's workspace begins)
            u32x4w* const out = reinterpret_cast<u32x4w*>(recs + (beg + c0) * kWinWords);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int i = k * kWave + lane;  // 16-byte half i of the chunk's records
                if (i < 2 * n) out[i] = *reinterpret_cast<const u32x4*>(rec + 4 * i);
            }
            __builtin_amdgcn_wave_barrier();
        }
    };

    const int64_t la = lane < F ? lane : F - 1;
    const int64_t lb = kWave + lane < F ? kWave + lane : F - 1;
    if (wv < row_waves) {
        const int64_t v0 = wv * kRecRows;
        int64_t rb[kRecRows + 1];
#pragma unroll
        for (int i = 0; i <= kRecRows; ++i) rb[i] = (int64_t)rowptr[v0 + i < N ? v0 + i : N];
        int32_t a0[kRecRows], b0[kRecRows];
        float ga[kRecRows], gb[kRecRows];
#pragma unroll
        for (int i = 0; i < kRecRows; ++i) {
            const int64_t v = v0 + i < N ? v0 + i : N - 1;
            a0[i] = argout[v * F + la];
            b0[i] = argout[v * F + lb];
            ga[i] = grad_at(g, g_bf16, v * F + la);
            gb[i] = grad_at(g, g_bf16, v * F + lb);
        }
#pragma unroll
        for (int i = 0; i < kRecRows; ++i) {
            const int64_t deg = rb[i + 1] - rb[i];
            if (v0 + i < N)
                span(v0 + i, rb[i], 0, deg < kRecPart ? deg : kRecPart, a0[i], b0[i], ga[i], gb[i]);
        }
    } else {
        const int64_t p0 = (wv - row_waves + 1) * kRecPart;
        if (p0 >= E) return;
        const int64_t v = row_of_position(rowptr, N, E, p0, lane);
        const int64_t beg = (int64_t)rowptr[v];
        const int64_t deg = (int64_t)rowptr[v + 1] - beg;
        const int64_t c0 = p0 - beg > kRecPart ? p0 - beg : kRecPart;
        const int64_t c1 = p0 + kRecPart - beg < deg ? p0 + kRecPart - beg : deg;
        if (c0 < c1)
            span(v, beg, c0, c1, argout[v * F + la], argout[v * F + lb],
                 grad_at(g, g_bf16, v * F + la), grad_at(g, g_bf16, v * F + lb));
    }
}

// Sum of the wins of every row of the transposed CSR.  Bound by its scattered
// reads: one 128-byte line per edge holds its record (124M edges, F = 100:
// 3855 us at 5.1 TB/s of lines; masks and chunks of G, about three lines per
// edge: 7715 us).  A wavefront is 8 slots of 8 lanes; a slot reads one record per load (lane i
// word i), 8 loads in flight, and adds the record's values into its own F
// sums in LDS: lane i adds value i.  The features of one record differ and
// every slot has sums of its own, so no two lanes ever add to one place, and
// each place's order of additions is fixed.  As in spmm_main, a mid row or hub
// chunk takes a wavefront, its edges dealt to the slots (whose sums are added
// in a fixed tree at the end), and small rows take a slot each.
// NF: 64-feature tiles of a row.
constexpr int kWinSlots = 8;

template <bool W, int NF>
__global__ __launch_bounds__(kBlock) void win_gather(SpmmParams P, int fp) {
    extern __shared__ float s_sum[];  // [kWavesPerBlock][kWinSlots][fp]
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int64_t wv = wid + (int64_t)blockIdx.x * kWavesPerBlock;
    if (wv >= P.n_hub_waves + P.n_mid_waves + P.n_small_waves) return;
    const int slot = lane >> 3, i = lane & 7;
    const int F = (int)P.F;
    float* const wave_sum = s_sum + wid * kWinSlots * fp;
    float* const sum = wave_sum + slot * fp;
    for (int k = 4 * lane; k < kWinSlots * fp; k += 4 * kWave)
        *reinterpret_cast<float4*>(wave_sum + k) = make_float4(0.f, 0.f, 0.f, 0.f);
    __builtin_amdgcn_wave_barrier();

    // this lane's word of the record of forward position key (0 without an edge)
    auto word = [&](int32_t key, bool ok) -> uint32_t {
        return ok ? P.recs[(int64_t)key * kWinWords + i] : 0u;
    };
    // add the record whose word i lane i of the slot holds, weight wt
    auto add = [&](uint32_t w, float wt) {
        // words 6 and 7 of the slot's record
        const uint32_t lo = __builtin_amdgcn_ds_swizzle((int)w, (6 << 5) | 0x18);
        const uint32_t hi = __builtin_amdgcn_ds_swizzle((int)w, (7 << 5) | 0x18);
        if (i < kWinValues && i < (int)(hi >> 24)) {
            const uint32_t id = ((i < 4 ? lo : hi) >> (8 * (i & 3))) & 255u;
            float v = __uint_as_float(w);
            if constexpr (W) v = __fmul_rn(wt, v);
            sum[id] += v;
        }
        __builtin_amdgcn_wave_barrier();
    };
    // Edges of more wins than a record holds: the rest from the destination's
    // argmax and gradient rows, by the whole wavefront, each edge's rows
    // loading while the previous edge's are added.
    int32_t pa[NF];
    float pg[NF];
    int pslot = -1;  // the slot whose edge's rows are loading (-1: none)
    int32_t ppos = 0;
    float pwt = 1.f;
    auto flush = [&]() {
        if (pslot < 0) return;
        float* const to = wave_sum + pslot * fp;
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            const int f = q * kWave + lane;
            if (pa[q] == ppos) {  // -1: not read (ppos is a position)
                float x = pg[q];
                if constexpr (W) x = __fmul_rn(pwt, x);
                to[f] += x;
            }
        }
        __builtin_amdgcn_wave_barrier();
        pslot = -1;
    };
    // w: this lane's word of the slot's record; key, col, wt: of the edge,
    // held by lane src(slot)
    auto rest = [&](uint32_t w, int32_t key, int32_t col, float wt, auto src) {
        uint64_t more = __ballot(i == 7 && (int)(w >> 24) > kWinValues);
        while (more) {
            const int l = __ffsll((unsigned long long)more) - 1;  // lane 7 of a slot
            more &= more - 1;
            const int sl = l >> 3;
            const int64_t v = __builtin_amdgcn_readlane(col, src(sl));
            // the record's features ascend: only those past its last are read
            const int last = (int)((uint32_t)__builtin_amdgcn_readlane((int)w, l) >> 8) & 255;
            int32_t na[NF];
            float ng[NF];
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                const int f = q * kWave + lane;
                na[q] = -1;
                ng[q] = 0.f;
                if (f < F && f > last) {
                    na[q] = P.win_arg[v * F + f];
                    ng[q] = grad_at(P.win_g, P.win_g_bf16, v * F + f);
                }
            }
            flush();
#pragma unroll
            for (int q = 0; q < NF; ++q) {
                pa[q] = na[q];
                pg[q] = ng[q];
            }
            pslot = sl;
            ppos = __builtin_amdgcn_readlane(key, src(sl));
            if constexpr (W)
                pwt = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(wt), src(sl)));
        }
    };
    constexpr int U = 8;

    if (wv < P.n_hub_waves + P.n_mid_waves) {
        const bool hub = wv < P.n_hub_waves;
        int64_t row, e0, e1;
        if (hub) {
            // the chunk's row, by binary search over the hub rows' chunk offsets
            int64_t lo = 0, hi = P.n_hub - 1;
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) >> 1;
                if ((int64_t)P.chunk_off[P.hub_base + mid] <= wv) lo = mid; else hi = mid - 1;
            }
            row = P.rowlist[P.hub_base + lo];
            const int64_t r0 = rp_at(P.rowptr, P.rp64, row), r1 = rp_at(P.rowptr, P.rp64, row + 1);
            const uint32_t first = P.chunk_off[P.hub_base + lo];
            const uint32_t n = P.chunk_off[P.hub_base + lo + 1] - first;
            const int64_t csz = ((uint32_t)(r1 - r0) + n - 1) / n;  // as in spmm_main
            e0 = r0 + (wv - (int64_t)first) * csz;
            e1 = e0 + csz < r1 ? e0 + csz : r1;
        } else {
            const int64_t k = P.mid_base + wv - P.n_hub_waves;
            row = P.rowlist ? (int64_t)P.rowlist[k] : k;
            e0 = P.rowbeg ? (int64_t)P.rowbeg[k] : rp_at(P.rowptr, P.rp64, row);
            e1 = P.rowend ? (int64_t)P.rowend[k] : rp_at(P.rowptr, P.rp64, row + 1);
        }
        // 64 edges at a time: edge u * 8 + slot is the slot's u-th; the next
        // 64 edges' indices load while these are gathered
        auto index = [&](int64_t q, int32_t& key, int32_t& col, float& wt) {
            const bool ok = q + lane < e1;
            key = ok ? __builtin_nontemporal_load(P.ekey + q + lane) : 0;
            col = ok ? __builtin_nontemporal_load(P.col + q + lane) : 0;
            wt = 1.f;
            if constexpr (W) wt = ok ? __builtin_nontemporal_load(P.w + q + lane) : 1.f;
        };
        int32_t key, col;
        float wt;
        index(e0, key, col, wt);
        for (int64_t q = e0; q < e1; q += kWave) {
            uint32_t w[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                w[u] = word(__shfl(key, u * kWinSlots + slot), q + u * kWinSlots + slot < e1);
            int32_t nkey, ncol;
            float nwt;
            index(q + kWave, nkey, ncol, nwt);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float x = 1.f;
                if constexpr (W) x = __shfl(wt, u * kWinSlots + slot);
                add(w[u], x);
                rest(w[u], key, col, wt, [&](int sl) { return u * kWinSlots + sl; });
            }
            key = nkey;
            col = ncol;
            wt = nwt;
        }
        flush();
        for (int f = lane; f < F; f += kWave) {
            float s[kWinSlots];
#pragma unroll
            for (int k = 0; k < kWinSlots; ++k) s[k] = wave_sum[k * fp + f];
            const float r = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
            if (hub) P.part_sum[wv * F + f] = r;
            else if (P.out_bf16) static_cast<uint16_t*>(P.out)[row * F + f] = f32_to_bf16_bits(r);
            else static_cast<float*>(P.out)[row * F + f] = r;
        }
        return;
    }

    // small rows: a slot each
    const int64_t k = (wv - P.n_hub_waves - P.n_mid_waves) * kWinSlots + slot;
    const bool row_ok = k < P.n_small;
    int64_t row = 0, e0 = 0;
    int32_t n = 0;
    if (row_ok) {
        row = P.rowlist[P.small_base + k];
        e0 = P.rowbeg[P.small_base + k];
        n = P.rowend[P.small_base + k] - (int32_t)e0;
    }
    int32_t max_n = n;
#pragma unroll
    for (int off = kWinSlots; off < kWave; off <<= 1) {
        const int32_t o = __shfl_xor(max_n, off);
        max_n = o > max_n ? o : max_n;
    }
    max_n = __builtin_amdgcn_readfirstlane(max_n);
    // lane i of a slot loads the indices of the row's next i-th edge
    auto index = [&](int32_t it, int32_t& key, int32_t& col, float& wt) {
        const bool ok = it + i < n;
        key = ok ? __builtin_nontemporal_load(P.ekey + e0 + it + i) : 0;
        col = ok ? __builtin_nontemporal_load(P.col + e0 + it + i) : 0;
        wt = 1.f;
        if constexpr (W) wt = ok ? __builtin_nontemporal_load(P.w + e0 + it + i) : 1.f;
    };
    int32_t key, col;
    float wt;
    index(0, key, col, wt);
    for (int32_t it = 0; it < max_n; it += U) {
        uint32_t w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = word(__shfl(key, (lane & ~7) + u), it + u < n);
        int32_t nkey, ncol;
        float nwt;
        index(it + U, nkey, ncol, nwt);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float x = 1.f;
            if constexpr (W) x = __shfl(wt, (lane & ~7) + u);
            add(w[u], x);
            rest(w[u], key, col, wt, [&](int sl) { return sl * 8 + u; });
        }
        key = nkey;
        col = ncol;
        wt = nwt;
    }
    flush();
    const int64_t left = P.n_small - (k - slot);
    const int rows = left < kWinSlots ? (int)left : kWinSlots;
    for (int s = 0; s < rows; ++s) {
        const int64_t r = ((int64_t)__shfl((int)(row >> 32), s * 8) << 32) |
                          (uint32_t)__shfl((int)(uint32_t)row, s * 8);
        for (int f = lane; f < F; f += kWave) {
            const float x = wave_sum[s * fp + f];
            if (P.out_bf16) static_cast<uint16_t*>(P.out)[r * F + f] = f32_to_bf16_bits(x);
            else static_cast<float*>(P.out)[r * F + f] = x;
        }
    }
}

typedef float f32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2e __attribute__((ext_vector_type(2), aligned(4)));
typedef int32_t i32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t i32x2e __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u32x4h __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2h __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u32h __attribute__((aligned(2)));

// EPL consecutive values of a fp32 or bf16 row, widened to fp32 (wide loads at
// any element).
template <typename T, int EPL>
__device__ inline void load_vals(const T* p, float (&v)[EPL]) {
    if constexpr (std::is_same<T, float>::value) {
        if constexpr (EPL >= 4) {
#pragma unroll
            for (int q = 0; q < EPL / 4; ++q) {
                const f32x4e a = reinterpret_cast<const f32x4e*>(p)[q];
                v[4 * q + 0] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
            }
        } else if constexpr (EPL == 2) {
            const f32x2e a = *reinterpret_cast<const f32x2e*>(p);
            v[0] = a.x; v[1] = a.y;
        } else {
            v[0] = *p;
        }
    } else {
        uint32_t u[(EPL + 1) / 2];
        if constexpr (EPL == 8) {
            const u32x4h a = *reinterpret_cast<const u32x4h*>(p);
            u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w;
        } else if constexpr (EPL == 4) {
            const u32x2h a = *reinterpret_cast<const u32x2h*>(p);
            u[0] = a.x; u[1] = a.y;
        } else if constexpr (EPL == 2) {
            u[0] = *reinterpret_cast<const u32h*>(p);
        } else {
            u[0] = *reinterpret_cast<const uint16_t*>(p);
        }
#pragma unroll
        for (int k = 0; k < EPL; ++k)
            v[k] = (k & 1) ? __uint_as_float(u[k / 2] & 0xFFFF0000u) : bf16_bits_to_f32(u[k / 2] & 0xFFFFu);
    }
}

template <int EPL>
__device__ inline void load_ints(const int32_t* p, int32_t (&v)[EPL]) {
    if constexpr (EPL >= 4) {
#pragma unroll
        for (int q = 0; q < EPL / 4; ++q) {
            const i32x4e a = reinterpret_cast<const i32x4e*>(p)[q];
            v[4 * q + 0] = a.x; v[4 * q + 1] = a.y; v[4 * q + 2] = a.z; v[4 * q + 3] = a.w;
        }
    } else if constexpr (EPL == 2) {
        const i32x2e a = *reinterpret_cast<const i32x2e*>(p);
        v[0] = a.x; v[1] = a.y;
    } else {
        v[0] = *p;
    }
}

// grad_w[p] = sum_f route(v, f, p) * g[v, f] * x[col[p], f] for the CSR edge
// p of row v = row[p]; route is 1 (sum), 1/deg(v) (mean, applied to the
// finished dot) or [argout[v, f] == p] (max).  A wavefront takes 64
// consecutive positions; slot s of its S slots takes positions base + u*S + s
// (u < U) of each step, its L lanes (a power of two, slots aligned) covering
// the feature row in FT tiles.
template <typename TX, typename TG, int EPL, int MODE>
__global__ __launch_bounds__(kBlock) void spmm_grad_w(GradWParams P) {
    constexpr int U = MODE == kMax ? 4 : MP_GW_UNROLL;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)) +
                       (int64_t)blockIdx.x * kWavesPerBlock;
    const int64_t p0 = wv * kWave;
    if (p0 >= P.E) return;
    const int L = P.L, S = P.S;
    const int slot = lane / L;
    const int j = lane - slot * L;
    const bool slot_ok = slot < S;
    const int64_t rem = P.E - p0;

    // absent index arrays are the identity (per-edge dot products of two
    // edge-space tables, or of one edge-space table and gathered rows)
    int32_t myc = 0, myv = 0;
    if (lane < rem) {
        myc = P.col ? __builtin_nontemporal_load(P.col + p0 + lane) : (int32_t)(p0 + lane);
        myv = P.row ? __builtin_nontemporal_load(P.row + p0 + lane) : (int32_t)(p0 + lane);
    }
    // values per lane left by the slot reduction (L < U), and the lane
    // stride between the holders of consecutive edges (L >= U)
    const bool ragged = P.F % EPL != 0;
    const int nv = U > L ? U / L : 1;
    const int hstride = U > L ? 1 : L / U;

    float result = 0.f;  // lane t ends with the dot of position p0 + t
    const int SU = S * U;
    for (int base = 0; base < kWave && base < rem; base += SU) {
        float dot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) dot[u] = 0.f;
        for (int ft = 0; ft < P.FT; ++ft) {
            const int64_t chunk = (int64_t)ft * kWave + j;
            const bool feat_ok = slot_ok && chunk < P.ltot;
            // a row's last chunk may begin inside the one before it: the
            // elements that both hold count in the earlier chunk
            int64_t fe = chunk * EPL;
            int skip = 0;
            if (EPL == 4 && ragged && fe > P.F - EPL) {
                skip = feat_ok ? (int)(fe - (P.F - EPL)) : 0;
                fe = P.F - EPL;
            }
            float xv[U][EPL], gv[U][EPL];
            int32_t mv[MODE == kMax ? U : 1][EPL];
            bool ok[U], fresh[U];
            int32_t vprev = -1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = base + u * S + slot;
                const int32_t c = __shfl(myc, t & (kWave - 1));
                const int32_t v = __shfl(myv, t & (kWave - 1));
                ok[u] = feat_ok && t < kWave && t < rem;
                // consecutive edges of a slot mostly share their row: its
                // gradient chunk (and argmax chunk) is loaded once and reused
                fresh[u] = u == 0 || v != vprev;
                vprev = v;
                if (ok[u]) {
                    load_vals<TX, EPL>(reinterpret_cast<const TX*>(P.x) + (int64_t)c * P.F + fe, xv[u]);
                    if (fresh[u]) {
                        load_vals<TG, EPL>(reinterpret_cast<const TG*>(P.g) + (int64_t)v * P.F + fe, gv[u]);
                        if constexpr (MODE == kMax) load_ints<EPL>(P.argout + (int64_t)v * P.F + fe, mv[u]);
                    }
                }
            }
#pragma unroll
            for (int u = 1; u < U; ++u) {
                if (fresh[u]) continue;  // a valid edge's predecessor in the slot is valid
#pragma unroll
                for (int k = 0; k < EPL; ++k) {
                    gv[u][k] = gv[u - 1][k];
                    if constexpr (MODE == kMax) mv[u][k] = mv[u - 1][k];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!ok[u]) continue;
                const int32_t pos = (int32_t)(p0 + base + u * S + slot);
                float t[EPL];
#pragma unroll
                for (int k = 0; k < EPL; ++k) {
                    t[k] = gv[u][k] * xv[u][k];
                    if constexpr (MODE == kMax) t[k] = mv[u][k] == pos ? t[k] : 0.f;
                }
                // (the products are left out, not one factor set to 0: an
                // infinite feature times 0 would be NaN)
                if (EPL == 4 && ragged) {
#pragma unroll
                    for (int k = 0; k < EPL; ++k) t[k] = k < skip ? 0.f : t[k];
                }
#pragma unroll
                for (int k = 0; k < EPL; ++k) dot[u] += t[k];
            }
        }
        // reduce the U dots over the slot's L lanes (L a power of two, slots
        // aligned) by recursive halving: at stride m the lanes with bit m set
        // keep the upper half of their values, the others the lower half, and
        // each adds its partner's copy of the half it keeps; once one value
        // is left, plain butterflies finish the sum.  A fixed pattern, so the
        // result is deterministic.  Afterwards lane j holds in dot[i] (i < nv)
        // the total of edge u = (j / hstride) * nv + i.
        int m = L >> 1;
#pragma unroll
        for (int h = U / 2; h >= 1; h >>= 1) {
            if (m >= 1) {
                const bool up = (lane & m) != 0;
#pragma unroll
                for (int i = 0; i < h; ++i) {
                    const float send = up ? dot[i] : dot[i + h];
                    const float keep = up ? dot[i + h] : dot[i];
                    dot[i] = keep + __shfl_xor(send, m);
                }
                m >>= 1;
            }
        }
        for (; m >= 1; m >>= 1) dot[0] += __shfl_xor(dot[0], m);
        // lane t picks the total of position base + u*S + s from its holder
        const int rel = lane - base;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = rel - u * S;
            const bool mine = s >= 0 && s < S;
            const int src = ((mine ? s : 0) * L + (u / nv) * hstride) & (kWave - 1);
            float o = __shfl(dot[0], src);
            if (nv > 1) {
#pragma unroll
                for (int i = 1; i < U; ++i) {
                    if (i < nv) {
                        const float q = __shfl(dot[i], src);
                        if (i == u % nv) o = q;
                    }
                }
            }
            if (mine) result = o;
        }
    }
    if (lane < rem) {
        if constexpr (MODE == kMean) {
            const int64_t deg = rp_at(P.rowptr, P.rp64, (int64_t)myv + 1) - rp_at(P.rowptr, P.rp64, myv);
            result = result / (float)deg;
        }
        P.grad_w[P.oidx ? (int64_t)P.oidx[p0 + lane] : p0 + lane] = result;
    }
}

template <typename TX, typename TG, int EPL>
hipError_t launch_gw_mode(const GradWParams& p, unsigned grid, hipStream_t s) {
    if (p.reduce == kMax)
        hipLaunchKernelGGL((spmm_grad_w<TX, TG, EPL, kMax>), dim3(grid), dim3(kBlock), 0, s, p);
    else if (p.reduce == kMean)
        hipLaunchKernelGGL((spmm_grad_w<TX, TG, EPL, kMean>), dim3(grid), dim3(kBlock), 0, s, p);
    else
        hipLaunchKernelGGL((spmm_grad_w<TX, TG, EPL, kSum>), dim3(grid), dim3(kBlock), 0, s, p);
    return hipGetLastError();
}

template <typename TX, typename TG>
hipError_t launch_gw_epl(const GradWParams& p, int epl, unsigned grid, hipStream_t s) {
    switch (epl) {
        case 8: return launch_gw_mode<TX, TG, 8>(p, grid, s);
        case 4: return launch_gw_mode<TX, TG, 4>(p, grid, s);
        case 2: return launch_gw_mode<TX, TG, 2>(p, grid, s);
        default: return launch_gw_mode<TX, TG, 1>(p, grid, s);
    }
}

template <typename IT, int SPAN>
void rows_vec(const IT* rp, int64_t N, int64_t E, int32_t* row, hipStream_t s) {
    const dim3 g((unsigned)ceil_div(N - 1 + E, SPAN)), b(kMergeBlock);
    if ((uintptr_t)row % 16 == 0)  // four ids per store
        hipLaunchKernelGGL((rows_of_edges<IT, true, SPAN>), g, b, 0, s, rp, N, E, row);
    else
        hipLaunchKernelGGL((rows_of_edges<IT, false, SPAN>), g, b, 0, s, rp, N, E, row);
}

template <typename IT>
hipError_t rows_span(const IT* rp, int64_t N, int64_t E, int32_t* row, hipStream_t s) {
    if (N + E < kMergeLong) rows_vec<IT, kMergeSpanShort>(rp, N, E, row, s);
    else rows_vec<IT, kMergeSpanLong>(rp, N, E, row, s);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rows_of_edges(const void* rowptr, int rp64, int64_t N, int64_t E, int32_t* row,
                                hipStream_t s) {
    if (E <= 0 || N <= 0) return hipSuccess;
    return rp64 ? rows_span(static_cast<const int64_t*>(rowptr), N, E, row, s)
                : rows_span(static_cast<const int32_t*>(rowptr), N, E, row, s);
}

hipError_t launch_win_masks(const void* rowptr, int rp64, const int32_t* argout, int64_t N,
                            int64_t F, uint32_t* bits, hipStream_t s) {
    if (N <= 0) return hipSuccess;
    const unsigned grid = (unsigned)ceil_div(ceil_div(N, kMaskRows), kWavesPerBlock);
    if (rp64)
        hipLaunchKernelGGL(win_masks<int64_t>, dim3(grid), dim3(kBlock), 0, s,
                           static_cast<const int64_t*>(rowptr), argout, N, F, win_mask_words(F),
                           bits);
    else
        hipLaunchKernelGGL(win_masks<int32_t>, dim3(grid), dim3(kBlock), 0, s,
                           static_cast<const int32_t*>(rowptr), argout, N, F, win_mask_words(F),
                           bits);
    return hipGetLastError();
}

// Records or masks, by the number of wins of an average edge, N_dst * F / E
// (us of the whole gradient by masks -> by records, uniform graphs of 60M
// edges unless said):
//   * over kWinMeanMax: records overflow, which costs two row reads per edge
//     (F = 64: 4 wins 2144 -> 1766, 8 wins 1302 -> 1837; F = 16: 4 wins 661 ->
//     722; F = 128: 2 wins 2037 -> 1309, 16 wins 2280 -> 3456);
//   * under 0.6: most edges win nothing, and their masks are shorter than
//     their records (F = 32: 1 win 2489 -> 2235, 0.25 wins 1730 -> 1890;
//     F = 64: 0.5 wins 1810 -> 1862; F = 100: 0.78 wins 2002 -> 1544);
//   * under kWinMinEdges the longer chain of a record's building shows
//     (F = 64, 2 wins: 0.5M edges 28 -> 40, 1M 54 -> 54, 2M 107 -> 84).
// The table of records, up to eight times the masks', stays within
// kWinMaxBytes.
bool use_win_records(int64_t N_dst, int64_t E, int64_t F) {
    constexpr int64_t kWinMinEdges = 3 << 19;
    constexpr int64_t kWinMaxBytes = int64_t(1) << 33;
    constexpr int64_t kWinMeanMax = 3;
    const int64_t wins = N_dst * F;
    return F <= kWinMaxF && E >= kWinMinEdges && E * kWinWords * 4 <= kWinMaxBytes &&
           wins <= kWinMeanMax * E && 5 * wins >= 3 * E;
}

hipError_t launch_win_records(const void* rowptr, int rp64, const int32_t* argout, const void* g,
                              int g_bf16, int64_t N, int64_t E, int64_t F, uint32_t* recs,
                              hipStream_t s) {
    if (N <= 0 || E <= 0) return hipSuccess;
    const int64_t waves = ceil_div(N, kRecRows) + ceil_div(E, kRecPart) - 1;
    const unsigned grid = (unsigned)ceil_div(waves, kWavesPerBlock);
    if (rp64)
        hipLaunchKernelGGL(win_records<int64_t>, dim3(grid), dim3(kBlock), 0, s,
                           static_cast<const int64_t*>(rowptr), argout, g, g_bf16, N, E, F, recs);
    else
        hipLaunchKernelGGL(win_records<int32_t>, dim3(grid), dim3(kBlock), 0, s,
                           static_cast<const int32_t*>(rowptr), argout, g, g_bf16, N, E, F, recs);
    return hipGetLastError();
}

hipError_t launch_win_gather(const SpmmParams& p, hipStream_t s) {
    const int64_t waves = p.n_hub_waves + p.n_mid_waves + p.n_small_waves;
    if (waves <= 0) return hipSuccess;
    const int fp = (int)((p.F + 3) / 4 * 4);  // whole 16-byte groups per slot
    const size_t lds = sizeof(float) * kWavesPerBlock * kWinSlots * fp;
    const dim3 g((unsigned)ceil_div(waves, kWavesPerBlock)), b(kBlock);
    static_assert(kWinMaxF <= 4 * kWave, "at most four feature tiles");
    const int nf = (int)ceil_div(p.F, kWave);
    if (p.w && nf <= 2) hipLaunchKernelGGL((win_gather<true, 2>), g, b, lds, s, p, fp);
    else if (p.w) hipLaunchKernelGGL((win_gather<true, 4>), g, b, lds, s, p, fp);
    else if (nf <= 2) hipLaunchKernelGGL((win_gather<false, 2>), g, b, lds, s, p, fp);
    else hipLaunchKernelGGL((win_gather<false, 4>), g, b, lds, s, p, fp);
    return hipGetLastError();
}

hipError_t launch_scale_inv_deg(const void* g, int g_bf16, const void* rowptr, int rp64, int64_t N,
                                int64_t F, float* out, hipStream_t s) {
    const int64_t n = N * F;
    if (n <= 0) return hipSuccess;
    // four elements per thread when rows hold whole groups of four and the
    // gradient is aligned for it (out is a 256-byte aligned workspace)
    const bool v4 = F % 4 == 0 && (uintptr_t)g % (g_bf16 ? 8 : 16) == 0;
    const unsigned grid = (unsigned)ceil_div(v4 ? n / 4 : n, kBlock);
    if (g_bf16 && v4)
        hipLaunchKernelGGL((scale_inv_deg<true, 4>), dim3(grid), dim3(kBlock), 0, s, g, rowptr, rp64, N, F, out);
    else if (g_bf16)
        hipLaunchKernelGGL((scale_inv_deg<true, 1>), dim3(grid), dim3(kBlock), 0, s, g, rowptr, rp64, N, F, out);
    else if (v4)
        hipLaunchKernelGGL((scale_inv_deg<false, 4>), dim3(grid), dim3(kBlock), 0, s, g, rowptr, rp64, N, F, out);
    else
        hipLaunchKernelGGL((scale_inv_deg<false, 1>), dim3(grid), dim3(kBlock), 0, s, g, rowptr, rp64, N, F, out);
    return hipGetLastError();
}

hipError_t launch_spmm_grad_w(const GradWParams& p0, int x_dtype, int g_dtype, int epl,
                              hipStream_t s) {
    if (p0.E <= 0) return hipSuccess;
    // slots of a power-of-two width at aligned lanes, as the dot reduction
    // needs (lanes past the feature row hold zeros)
    GradWParams p = p0;
    if (p.L < kWave) {
        int lp = 1;
        while (lp < p.L) lp *= 2;
        p.L = lp;
        p.S = kWave / lp;
    }
    const int64_t waves = ceil_div(p.E, kWave);
    const unsigned grid = (unsigned)ceil_div(waves, kWavesPerBlock);
    if (x_dtype == MP_F32)
        return g_dtype == MP_F32 ? launch_gw_epl<float, float>(p, epl, grid, s)
                                 : launch_gw_epl<float, uint16_t>(p, epl, grid, s);
    return g_dtype == MP_F32 ? launch_gw_epl<uint16_t, float>(p, epl, grid, s)
                             : launch_gw_epl<uint16_t, uint16_t>(p, epl, grid, s);
}

}  // namespace mp
