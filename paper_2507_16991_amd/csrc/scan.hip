// The aggregation plan: rows sorted by degree class (stable by row id), each
// entry's row range, and the hub rows' chunk offsets (Sec. 2.2: a
// destination-sorted layout lets the aggregation run in parallel over rows).
//
// A counting sort of at most kPlanClasses classes, in as few launches as the
// number of rows allows, since a plan is built for every new graph and the
// launches are most of its time on small ones:
//   * up to kPlanSingleRows rows: plan_scatter alone, in one workgroup;
//   * beyond: plan_count (class counts of every tile of rows), plan_scan (one
//     workgroup: where each class starts, and each tile inside it), and
//     plan_scatter, which ranks its tile's rows again and writes them.
// rowptr is read by the count and the scatter (8 bytes a row); 12 bytes a row
// are written.  (It took ten launches: the classes as keys of a one-pass radix
// sort, the row ranges and chunk counts through the sorted list, a three-step
// scan over all rows and the header.  mp_spmm_plan_build with its copy to the
// host, us before -> now: 2.7k rows 96 -> 34, 169k 100 -> 50, 2.4M 141 -> 63,
// 20M 375 -> 190.)
#include "mp_internal.hpp"

namespace mp {
namespace {

constexpr int kPlanItems = 16;  // rows per thread of a full tile
// scanned rows: the classes' counts, then the chunks, then the long rows
constexpr int kPlanRows = kPlanClasses + 2;

struct PlanRow {
    int64_t beg, end;
    uint32_t cls;
    uint32_t chunks;  // 0 unless a hub
    bool is_long;     // more than long_min edges
};

// Class of a row: small rows by the bit length of the degree (0 for an empty
// row), one more beyond `split` edges, then mid, then hub.  (Two limits of small rows,
// as rows may be aggregated by a narrow and by a wide cut of their features.)
template <typename IT>
__device__ inline PlanRow plan_row(const IT* __restrict__ rowptr, int64_t i, const PlanParams& P) {
    PlanRow r;
    r.beg = (int64_t)rowptr[i];
    r.end = (int64_t)rowptr[i + 1];
    const int64_t d = r.end - r.beg;
    r.chunks = 0;
    r.is_long = d > P.long_min;
    if (d > P.hub_min) {
        r.cls = kClassHub;
        int64_t csz = (d + kMaxChunksPerHub - 1) / kMaxChunksPerHub;
        if (csz < P.chunk_min) csz = P.chunk_min;
        r.chunks = (uint32_t)((d + csz - 1) / csz);
    } else if (d > P.small_max) {
        r.cls = kClassMid;
    } else {
        r.cls = d <= 0 ? 0u : (uint32_t)(64 - __clzll((unsigned long long)d)) + (d > P.split);
    }
    return r;
}

__device__ inline uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

// Inclusive scan over the wavefront.
__device__ inline uint32_t wave_scan(uint32_t v, int lane) {
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(v, off, kWave);
        if (lane >= off) v += o;
    }
    return v;
}

// tile_cnt[c * tiles + tile] = rows of class c (c < kPlanClasses) in the tile,
// in row kPlanClasses its hub rows' chunks, and in the next its long rows.
template <typename IT, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void plan_count(const IT* __restrict__ rowptr,
                                                            PlanParams P) {
    __shared__ uint32_t s_cnt[WAVES][32];
    __shared__ uint32_t s_chunks[WAVES], s_long[WAVES];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    if (lane < 32) s_cnt[wv][lane] = 0;
    __builtin_amdgcn_wave_barrier();
    const int64_t base = ((int64_t)blockIdx.x * WAVES + wv) * kPlanItems * kWave;
    uint32_t chunks = 0, longs = 0;
#pragma unroll 4
    for (int k = 0; k < kPlanItems; ++k) {
        const int64_t i = base + k * kWave + lane;
        const bool ok = i < P.N;
        PlanRow r{0, 0, 0, 0, false};
        if (ok) r = plan_row(rowptr, i, P);
        chunks += r.chunks;
        longs += (uint32_t)__popcll(__ballot(r.is_long));
        const uint64_t peers = digit_peers<kPlanClassBits>(ok, r.cls);
        if (ok && count_below(peers) == 0) s_cnt[wv][r.cls] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    chunks = wave_sum(chunks);
    if (lane == 0) {
        s_chunks[wv] = chunks;
        s_long[wv] = longs;
    }
    __syncthreads();
    if (threadIdx.x < kPlanRows) {
        const int c = threadIdx.x;
        uint32_t t = 0;
        for (int w = 0; w < WAVES; ++w)
            t += c < kPlanClasses ? s_cnt[w][c] : (c == kPlanClasses ? s_chunks[w] : s_long[w]);
        P.tile_cnt[(int64_t)c * gridDim.x + blockIdx.x] = t;
    }
}

// In place, every row of tile_cnt: exclusive scan over the tiles (a wavefront
// per row); header[c] = first row-list position of class c, then N, the
// number of chunks and of long rows; chunk_off[N] = the number of chunks.
__global__ __launch_bounds__(1024) void plan_scan(PlanParams P, int64_t tiles) {
    __shared__ uint32_t s_total[32];
    const int lane = threadIdx.x & (kWave - 1);
    constexpr int kAhead = 4;
    for (int c = threadIdx.x / kWave; c < kPlanRows; c += 1024 / kWave) {
        uint32_t* const row = P.tile_cnt + (int64_t)c * tiles;
        uint32_t carry = 0;
        for (int64_t t0 = 0; t0 < tiles; t0 += kAhead * kWave) {
            uint32_t v[kAhead];
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const int64_t t = t0 + a * kWave + lane;
                v[a] = t < tiles ? row[t] : 0u;
            }
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const int64_t t = t0 + a * kWave + lane;
                const uint32_t inc = wave_scan(v[a], lane);
                if (t < tiles) row[t] = carry + inc - v[a];
                carry += __shfl(inc, kWave - 1);
            }
        }
        if (lane == 0) s_total[c] = carry;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        const uint32_t t = lane < kPlanClasses ? s_total[lane] : 0u;
        const uint32_t inc = wave_scan(t, lane);
        if (lane < kPlanClasses) P.header[lane] = inc - t;
        if (lane == 0) {
            P.header[kPlanClasses] = (uint32_t)P.N;
            P.header[kPlanClasses + 1] = s_total[kPlanClasses];
            P.header[kPlanClasses + 2] = s_total[kPlanClasses + 1];
            P.chunk_off[P.N] = s_total[kPlanClasses];
        }
    }
}

// Rank the tile's rows stably by class and write them.  Rows go to (wavefront,
// round, lane) in order; `items` rounds (kPlanItems, or with SINGLE as many as
// spread the rows over the workgroup).  SINGLE: the only tile, which also
// makes the header.
template <typename IT, int WAVES, bool SINGLE>
__global__ __launch_bounds__(WAVES * kWave) void plan_scatter(const IT* __restrict__ rowptr,
                                                              PlanParams P, int items) {
    __shared__ uint32_t s_cnt[WAVES][32];  // rows of each class, then where a wave's start
    __shared__ uint32_t s_chunks[WAVES], s_long[WAVES];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    if (lane < 32) s_cnt[wv][lane] = 0;
    __builtin_amdgcn_wave_barrier();
    const int64_t base = ((int64_t)blockIdx.x * WAVES + wv) * items * kWave;
    PlanRow r[kPlanItems];
    uint32_t rank[kPlanItems], before[kPlanItems];  // before: chunks of earlier hub rows
    uint32_t chunks = 0, longs = 0;
#pragma unroll
    for (int k = 0; k < kPlanItems; ++k) {
        r[k] = PlanRow{0, 0, 0, 0, false};
        const int64_t i = base + k * kWave + lane;
        if (k < items && i < P.N) r[k] = plan_row(rowptr, i, P);
        if constexpr (SINGLE) longs += (uint32_t)__popcll(__ballot(r[k].is_long));
    }
#pragma unroll
    for (int k = 0; k < kPlanItems; ++k) {
        if (k < items) {
            const bool ok = base + k * kWave + lane < P.N;
            const uint64_t peers = digit_peers<kPlanClassBits>(ok, r[k].cls);
            const uint32_t below = count_below(peers);
            const uint32_t c = s_cnt[wv][r[k].cls];
            rank[k] = c + below;
            __builtin_amdgcn_wave_barrier();
            if (ok && below == 0) s_cnt[wv][r[k].cls] = c + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
            before[k] = 0;
            if (__ballot(r[k].chunks != 0)) {
                const uint32_t inc = wave_scan(r[k].chunks, lane);
                before[k] = chunks + inc - r[k].chunks;
                chunks += __shfl(inc, kWave - 1);
            }
        }
    }
    if (lane == 0) {
        s_chunks[wv] = chunks;
        s_long[wv] = longs;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        // where each class starts for this tile, then for each of its waves
        const int c = lane;
        uint32_t total = 0;
        if (c < kPlanClasses)
            for (int w = 0; w < WAVES; ++w) total += s_cnt[w][c];
        uint32_t run;
        if constexpr (SINGLE) {
            run = wave_scan(total, lane) - total;
            if (c < kPlanClasses) P.header[c] = run;
            if (c == kPlanClasses) P.header[c] = (uint32_t)P.N;
        } else {
            run = c < kPlanClasses
                      ? P.header[c] + P.tile_cnt[(int64_t)c * gridDim.x + blockIdx.x]
                      : 0u;
        }
        if (c < kPlanClasses) {
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t n = s_cnt[w][c];
                s_cnt[w][c] = run;
                run += n;
            }
        }
        if (c == kPlanClasses) {
            uint32_t at = SINGLE ? 0u : P.tile_cnt[(int64_t)c * gridDim.x + blockIdx.x];
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t n = s_chunks[w];
                s_chunks[w] = at;
                at += n;
            }
            if constexpr (SINGLE) {
                P.header[kPlanClasses + 1] = at;
                P.chunk_off[P.N] = at;
                uint32_t all = 0;
                for (int w = 0; w < WAVES; ++w) all += s_long[w];
                P.header[kPlanClasses + 2] = all;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPlanItems; ++k) {
        const int64_t i = base + k * kWave + lane;
        if (k < items && i < P.N) {
            const uint32_t q = s_cnt[wv][r[k].cls] + rank[k];
            P.rowlist[q] = (int32_t)i;
            P.rowbeg[q] = (int32_t)r[k].beg;
            P.rowend[q] = (int32_t)r[k].end;
            if (r[k].cls == kClassHub) P.chunk_off[q] = s_chunks[wv] + before[k];
        }
    }
}

// Rows per tile: small tiles spread few rows over the CUs; large ones keep
// the scan of the tiles' counts short (its one workgroup reads 19 counts per
// tile).
constexpr int64_t kPlanSmallTiles = int64_t(1) << 22;  // rows up to which tiles are small
inline int plan_waves(int64_t N) { return N <= kPlanSmallTiles ? 4 : 16; }
inline int64_t plan_tiles(int64_t N) { return ceil_div(N, (int64_t)plan_waves(N) * kWave * kPlanItems); }

template <typename IT>
hipError_t plan_launch(const PlanParams& p, hipStream_t s) {
    const IT* rp = static_cast<const IT*>(p.rowptr);
    if (p.N <= kPlanSingleRows) {
        const int items = (int)ceil_div(p.N, 1024);
        hipLaunchKernelGGL((plan_scatter<IT, 16, true>), dim3(1), dim3(1024), 0, s, rp, p, items);
        return hipGetLastError();
    }
    const int64_t tiles = plan_tiles(p.N);
    const dim3 g((unsigned)tiles);
    if (plan_waves(p.N) == 4) {
        hipLaunchKernelGGL((plan_count<IT, 4>), g, dim3(256), 0, s, rp, p);
        hipLaunchKernelGGL(plan_scan, dim3(1), dim3(1024), 0, s, p, tiles);
        hipLaunchKernelGGL((plan_scatter<IT, 4, false>), g, dim3(256), 0, s, rp, p, kPlanItems);
    } else {
        hipLaunchKernelGGL((plan_count<IT, 16>), g, dim3(1024), 0, s, rp, p);
        hipLaunchKernelGGL(plan_scan, dim3(1), dim3(1024), 0, s, p, tiles);
        hipLaunchKernelGGL((plan_scatter<IT, 16, false>), g, dim3(1024), 0, s, rp, p, kPlanItems);
    }
    return hipGetLastError();
}

}  // namespace

int64_t plan_tile_counts(int64_t N) {
    return N <= kPlanSingleRows ? 0 : plan_tiles(N) * kPlanRows;
}

hipError_t launch_plan(const PlanParams& p, hipStream_t s) {
    if (p.N <= 0) return hipSuccess;
    return p.rp64 ? plan_launch<int64_t>(p, s) : plan_launch<int32_t>(p, s);
}

}  // namespace mp
