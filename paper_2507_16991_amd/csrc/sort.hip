// Stable LSD radix sort of COO edges by destination, and the small kernels
// around it (rowptr, payload gather, validation).
//
// The sort is one-sweep: radix_ghist counts the digits of every pass in one
// read of the keys; then each pass is ONE kernel, radix_onesweep, in which a
// tile of kSortTile keys (tile ids taken from an atomic counter in launch
// order) ranks its keys stably (wave-level multisplit: one ballot per digit
// bit, per-wavefront LDS counters), publishes its per-digit counts, obtains
// the running totals of all earlier tiles by decoupled look-back over their
// published descriptors, stages the tile in LDS in digit order and writes
// each digit's run contiguously.  Ranks follow (wave, round, lane) order,
// which is element order, so each pass is stable and the whole LSD sort keeps
// ascending COO id within a destination (the order the CSR of Sec. 2.2 must
// have to be unique).  Only integer arithmetic: the result is bit-exact.
//
// Between passes an element is one 8-byte word, so that a digit run is one
// stretch of memory: (key, src), or with the COO-id payload (key, src, id)
// packed where their bits fit 64.  To make them fit, a word leaves out the
// digit its pass has just sorted by: the element's place says it, and the
// next pass puts it back (124M edges, 2.4M rows: 15 + 22 + 27 bits).  The last
// pass writes src and id alone; rowptr comes from where it sees each row
// start (or from the keys, where rows are many).  (Carrying id as a third array
// and keeping the sorted keys for rowptr
// cost 80 bytes of traffic per edge where this takes 56 to 60: passes of 790,
// 880 and 898 us on 124M edges -> 601, 663 and 800, rowptr 155 -> 27; CSR with
// ids and transpose together 6.05 -> 4.85 ms.)
//
// The look-back only waits on tiles that started earlier (their ids were
// taken first), so it always ends; its wait is nevertheless bounded, and a
// tile that gives up records it in an error word that the caller turns into
// MP_ERR_SORT instead of hanging the device.
#include "mp_internal.hpp"

namespace mp {
namespace {

constexpr int kSortWaves = kSortBlock / kWave;
constexpr int kWaveKeys = kWave * kSortItems;  // keys per wavefront per tile
constexpr int kMaxBuckets = 1 << kSortMaxBits;

constexpr int kGhistBlock = 1024;
constexpr int kGhistItems = 8;
constexpr int kGhistCopies = 4;     // LDS copies of the histogram, four wavefronts each
constexpr int kGhistMaxGrid = 512;  // two workgroups per CU
constexpr uint32_t kSpinLimit = 1u << 20;
constexpr uint32_t kNoStart = 0xFFFFFFFFu;  // a row no edge of which has been seen

// look-back descriptor: flag (bits 63..62: 1 tile count, 2 inclusive prefix),
// pass tag (bits 61..56, pass + 1), value (bits 55..0)
constexpr uint64_t kFlagAgg = 1ull << 62;
constexpr uint64_t kFlagPre = 2ull << 62;
__device__ inline uint64_t desc_make(uint64_t flag, uint32_t tag, uint64_t v) {
    return flag | ((uint64_t)tag << 56) | v;
}

__global__ __launch_bounds__(256) void radix_clear(RadixScratch sc, int64_t ndesc, int64_t nstarts) {
    const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t i = i0; i < ndesc; i += step) sc.desc[i] = 0;
    for (int64_t i = i0; i < nstarts; i += step) sc.starts[i] = kNoStart;
    if (i0 < kMaxPasses * kMaxBuckets) sc.ghist[i0] = 0;
    if (i0 < kMaxPasses) sc.counter[i0] = 0;
    if (i0 == 0) {
        *sc.err = 0;
        *sc.a_or = 0;
    }
}

// Global histogram of every pass's digit.  Counts do not depend on order, so
// the wavefronts add into LDS copies with integer atomics (no ranking
// needed), then one integer atomic per (pass, digit) per workgroup.  Few,
// large workgroups: with 2048 of 256 threads the additions to the same 1536
// words were most of the time of a 20M-edge sort's histogram (52 us).
// shifts and widths: one byte per pass (pass p in bits 8p..8p+7).  With a, the
// bits of that payload are collected too.
__global__ __launch_bounds__(kGhistBlock) void radix_ghist(const uint32_t* __restrict__ keys,
                                                           const int32_t* __restrict__ a,
                                                           int64_t n, int passes, uint32_t shifts,
                                                           uint32_t widths, RadixScratch sc) {
    __shared__ uint32_t h[kGhistCopies][kMaxPasses][kMaxBuckets];
    __shared__ uint32_t s_bits;
    if (threadIdx.x == 0) s_bits = 0;
    for (int i = threadIdx.x; i < kGhistCopies * kMaxPasses * kMaxBuckets; i += kGhistBlock)
        (&h[0][0][0])[i] = 0;
    __syncthreads();
    uint32_t(*const my)[kMaxBuckets] = h[(threadIdx.x / kWave) % kGhistCopies];
    uint32_t bits = 0;
    const int64_t tile = (int64_t)kGhistBlock * kGhistItems;
    for (int64_t base = blockIdx.x * tile; base < n; base += gridDim.x * tile) {
        uint32_t key[kGhistItems];
#pragma unroll
        for (int k = 0; k < kGhistItems; ++k) {
            const int64_t i = base + k * kGhistBlock + threadIdx.x;
            key[k] = i < n ? __builtin_nontemporal_load(keys + i) : 0u;
            if (a) bits |= i < n ? (uint32_t)__builtin_nontemporal_load(a + i) : 0u;
        }
#pragma unroll
        for (int k = 0; k < kGhistItems; ++k) {
            if (base + k * kGhistBlock + threadIdx.x >= n) continue;
            for (int p = 0; p < passes; ++p) {
                const uint32_t sh = (shifts >> (8 * p)) & 255u;
                const uint32_t mask = (1u << ((widths >> (8 * p)) & 255u)) - 1u;
                atomicAdd(&my[p][(key[k] >> sh) & mask], 1u);
            }
        }
    }
    if (a) {
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) bits |= __shfl_xor(bits, off);
        if ((threadIdx.x & (kWave - 1)) == 0) atomicOr(&s_bits, bits);
    }
    __syncthreads();
    // (one access to the word per workgroup: one per wavefront, 8192 to the
    // same word, took 88 us of a 10M-edge sort's histogram)
    if (a && threadIdx.x == 0) atomicOr(sc.a_or, s_bits);
    for (int i = threadIdx.x; i < passes * kMaxBuckets; i += kGhistBlock) {
        uint32_t t = 0;
#pragma unroll
        for (int c = 0; c < kGhistCopies; ++c) t += (&h[c][0][0])[i];
        if (t) atomicAdd(&sc.ghist[i], t);
    }
}

// Exclusive scan over N values of LDS or global memory by one wavefront
// (lane l takes N / 64 consecutive ones), to LDS.
template <int N>
__device__ inline void wave_exclusive(const uint32_t* in, int n, uint32_t* out, int lane) {
    constexpr int PER = N / kWave;
    uint32_t t[PER];
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = lane * PER + k;
        t[k] = d < n ? in[d] : 0u;
        sum += t[k];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += o;
    }
    uint32_t run = inc - sum;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = lane * PER + k;
        if (d < n) out[d] = run;
        run += t[k];
    }
}

// How the passes carry (key, a, b) between them: kWide, a (key << 32 | a) word
// and a 4-byte array of b; kKeep, one word of the key, a and b; kDrop, one
// word of the key without the digit just sorted by, a and b.  Decided on the
// device, from the bits a really has.
constexpr int kWide = 0, kKeep = 1, kDrop = 2;
__device__ inline int word_format(const RadixPass& p, int abits) {
    if (p.key_bits + abits + p.b_bits <= 64) return kKeep;
    // (a staged word without its digit needs the digit map, which has bytes)
    if (p.max_width <= 8 && p.key_bits - p.min_width + abits + p.b_bits <= 64) return kDrop;
    return kWide;
}

// key (at most 31 bits) without the digit at [shift, shift + width), and back
__device__ inline uint32_t drop_digit(uint32_t key, int shift, int width) {
    return ((key >> (shift + width)) << shift) | (key & ((1u << shift) - 1u));
}
__device__ inline uint32_t put_digit(uint32_t rest, uint32_t d, int shift, int width) {
    return ((rest >> shift) << (shift + width)) | (d << shift) | (rest & ((1u << shift) - 1u));
}

// A packed word: b in the low bb bits, a in the next ab, the key above, in
// 32-bit operations on its halves (1 <= ab <= 32, 1 <= bb <= 31).
struct WordBits {
    int ab, bb;
    __device__ inline void pack(uint32_t key, uint32_t a, uint32_t b, uint32_t& hi, uint32_t& lo) const {
        lo = b | (a << bb);
        hi = a >> (32 - bb);
        const int kb = ab + bb;  // the key's place
        if (kb >= 32) {
            hi |= key << (kb - 32);
        } else {
            lo |= key << kb;
            hi |= key >> (32 - kb);
        }
    }
    __device__ inline uint32_t key(uint32_t hi, uint32_t lo) const {
        const int kb = ab + bb;
        return kb >= 32 ? hi >> (kb - 32) : __builtin_amdgcn_alignbit(hi, lo, kb);
    }
    __device__ inline int32_t a(uint32_t hi, uint32_t lo) const {
        return (int32_t)(__builtin_amdgcn_alignbit(hi, lo, bb) & (0xFFFFFFFFu >> (32 - ab)));
    }
    __device__ inline int32_t b(uint32_t lo) const { return (int32_t)(lo & ((1u << bb) - 1u)); }
};

// One LSD pass: rank the tile's keys stably (wave-level multisplit, per-wave
// LDS counters), publish the tile's digit counts, stage the tile in LDS in
// digit order, then look back over earlier tiles for their running totals
// and write every digit run contiguously.  Ranks follow (wave, round, lane)
// order, which is element order, and tiles are numbered in the order they
// start, so the pass is stable.  Staging before the look-back frees the
// registers of the keys while the tile waits on its predecessors, so the
// look-back can keep kLookWindow descriptor loads in flight.  Descriptors of
// a pass over R = 2^bits digits lie R apart per tile.
//   HAS_B: the COO-id payload b is carried (b = the element index on FIRST).
//   WIDE:  digits of up to 9 bits (512 buckets: twice the per-wave counters).
//   FIRST: keys and a are read as given; otherwise as words (word_format).
//   LAST:  a (and b) are written alone, and for rowptr the key too, or where
//          the tile first sees a row, starts[row] takes the place (the least
//          over all tiles: a row's edges lie together, in tile order);
//          otherwise words are written.
// A tile's words are staged in LDS as two halves at once (128 KB); in kWide
// with b, the keys, a and b go through one staging buffer in turn, the keys
// before the look-back and the others after the previous array is written.
// In kDrop, as a staged word has no digit, a byte per slot keeps it.
constexpr int kLookWindow = 4;

template <bool HAS_B, bool WIDE, bool FIRST, bool LAST>
__global__ __launch_bounds__(kSortBlock) void radix_onesweep(RadixPass p) {
    static_assert(kSortTile <= 65536, "16-bit counters and staged slots");
    constexpr int NB = WIDE ? kMaxBuckets : kMaxBuckets / 2;  // buckets this variant handles
    // per-wave digit counts, then each wave's run start inside its digit
    using cnt_t = uint16_t;
    __shared__ uint32_t s_stage[2][kSortTile];
    __shared__ uint8_t s_dig[HAS_B && !WIDE ? kSortTile : 1];  // kDrop: digit of every slot
    __shared__ cnt_t s_cnt[kSortWaves][NB];
    __shared__ uint32_t s_tcnt[NB];   // the tile's count of each digit
    __shared__ uint32_t s_start[NB];  // ... and its exclusive scan
    __shared__ uint32_t s_gbase[NB];  // global start of each digit, then of the tile's run
    __shared__ uint32_t s_prev[HAS_B && !FIRST && !WIDE ? NB : 1];  // kDrop: the last pass's digit starts
    __shared__ uint32_t s_tile;

    const int R = 1 << p.bits;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x / kWave;
    for (int i = threadIdx.x; i < kSortWaves * NB; i += kSortBlock) (&s_cnt[0][0])[i] = 0;
    if (threadIdx.x == 0) s_tile = atomicAdd(&p.sc.counter[p.pass], 1u);
    int abits = 0, fmt = kWide;
    if constexpr (HAS_B) {
        abits = p.a_bits ? p.a_bits : 32 - __clz((int)(*p.sc.a_or | 1u));
        fmt = word_format(p, abits);
    }
    const WordBits word{abits, p.b_bits};
    const bool drop = HAS_B && !WIDE && fmt == kDrop;
    if constexpr (HAS_B && !FIRST && !WIDE) {
        if (wv == 1 && fmt == kDrop)
            wave_exclusive<NB>(p.sc.ghist + (p.pass - 1) * kMaxBuckets, 1 << p.prev_bits, s_prev, lane);
    }
    __syncthreads();
    const int64_t tile = s_tile;
    uint64_t* const desc = p.sc.desc + tile * R;

    const int64_t tbase = tile * kSortTile;
    const int64_t wbase = tbase + (int64_t)wv * kWaveKeys;

    uint32_t key[kSortItems];
    int32_t va[kSortItems], vb[HAS_B ? kSortItems : 1];
    uint32_t rank[kSortItems];
    if constexpr (FIRST) {
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int64_t i = wbase + (int64_t)k * kWave + lane;
            const bool ok = i < p.n;
            key[k] = ok ? __builtin_nontemporal_load(p.keys_in + i) : 0u;
            va[k] = ok ? __builtin_nontemporal_load(p.a_in + i) : 0;
            if constexpr (HAS_B) vb[k] = (int32_t)i;
        }
    } else {
        uint64_t w[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int64_t i = wbase + (int64_t)k * kWave + lane;
            w[k] = i < p.n ? __builtin_nontemporal_load(p.kv_in + i) : 0ull;
        }
        if (!HAS_B || fmt == kWide) {
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) {
                key[k] = (uint32_t)(w[k] >> 32);
                va[k] = (int32_t)(uint32_t)w[k];
                if constexpr (HAS_B) {
                    const int64_t i = wbase + (int64_t)k * kWave + lane;
                    vb[k] = i < p.n ? __builtin_nontemporal_load(p.b_in + i) : 0;
                }
            }
        } else if constexpr (HAS_B) {
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) {
                const uint32_t hi = (uint32_t)(w[k] >> 32), lo = (uint32_t)w[k];
                key[k] = word.key(hi, lo);
                va[k] = word.a(hi, lo);
                vb[k] = word.b(lo);
            }
            if constexpr (!WIDE) {
                if (drop) {
                    // the digit of the last pass, from the place: the last d
                    // whose run starts at or before it.  A wavefront's places
                    // mostly lie in one run.
                    const int PR = 1 << p.prev_bits;
                    auto count_le = [&](int64_t pos) {  // run starts at or before pos
                        int c = 0;
                        for (int d = 0; d < PR; d += kWave)
                            c += __popcll(__ballot(d + lane < PR && (int64_t)s_prev[d + lane] <= pos));
                        return c;
                    };
                    const int64_t last = wbase + kWaveKeys - 1 < p.n ? wbase + kWaveKeys - 1 : p.n - 1;
                    const int dA = count_le(wbase) - 1;
                    const int dB = last > wbase ? count_le(last) - 1 : dA;
#pragma unroll
                    for (int k = 0; k < kSortItems; ++k) {
                        const int64_t i = wbase + (int64_t)k * kWave + lane;
                        int lo = dA, hi = dB;
                        while (lo < hi) {
                            const int mid = (lo + hi + 1) >> 1;
                            if ((int64_t)s_prev[mid] <= i) lo = mid; else hi = mid - 1;
                        }
                        key[k] = put_digit(key[k], (uint32_t)lo, p.prev_shift, p.prev_bits);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        const bool ok = wbase + (int64_t)k * kWave + lane < p.n;
        const uint32_t d = (key[k] >> p.shift) & (uint32_t)(R - 1);
        const uint64_t peers = digit_peers<kSortMaxBits>(ok, d, p.bits);
        const uint32_t below = count_below(peers);
        const uint32_t base = s_cnt[wv][d];
        rank[k] = base + below;
        // the lowest peer advances the counter for all of them; every lane has
        // read the old value above (LDS ops of one wavefront run in order)
        if (ok && below == 0) s_cnt[wv][d] = (cnt_t)(base + (uint32_t)__popcll(peers));
    }
    __syncthreads();

    // per digit: each wave's run start inside the digit, and the tile count,
    // which is published at once (earlier publication shortens the waits of
    // later tiles)
    const uint32_t tag = (uint32_t)p.pass + 1u;
    for (int d = threadIdx.x; d < R; d += kSortBlock) {
        uint32_t run = 0;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            uint32_t c = s_cnt[w][d];
            s_cnt[w][d] = (cnt_t)run;
            run += c;
        }
        s_tcnt[d] = run;
        __hip_atomic_store(desc + d, desc_make(tile == 0 ? kFlagPre : kFlagAgg, tag, run),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    // exclusive scans of the tile's digit counts and of the global ones
    if (wv == 0) wave_exclusive<NB>(s_tcnt, R, s_start, lane);
    if (wv == kSortWaves - 1)
        wave_exclusive<NB>(p.sc.ghist + p.pass * kMaxBuckets, R, s_gbase, lane);
    __syncthreads();

    // stage the tile in LDS in digit order (tile-local positions only)
    uint16_t* const s_lp = reinterpret_cast<uint16_t*>(s_stage[1]);  // kWide with b: slot of every key
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        const int64_t i = wbase + (int64_t)k * kWave + lane;
        const uint32_t d = (key[k] >> p.shift) & (uint32_t)(R - 1);
        const uint32_t lp = s_start[d] + s_cnt[wv][d] + rank[k];
        if (i < p.n) {
            if (!HAS_B) {
                s_stage[0][lp] = key[k];
                s_stage[1][lp] = (uint32_t)va[k];
            } else if (fmt == kWide) {
                s_stage[0][lp] = key[k];
                s_lp[k * kSortBlock + threadIdx.x] = (uint16_t)lp;
            } else if constexpr (HAS_B) {
                uint32_t hi, lo;
                word.pack(drop ? drop_digit(key[k], p.shift, p.bits) : key[k], (uint32_t)va[k],
                          (uint32_t)vb[k], hi, lo);
                s_stage[0][lp] = hi;
                s_stage[1][lp] = lo;
                if constexpr (!WIDE)
                    if (drop) s_dig[lp] = (uint8_t)d;
            }
        }
    }

    // decoupled look-back, one thread per digit: add up earlier tiles'
    // counts until one that carries an inclusive prefix, kLookWindow
    // descriptors per round (a descriptor not yet published ends the round;
    // the wait on it is bounded)
    if (threadIdx.x < R) {
        const int d = threadIdx.x;
        const uint64_t* col = p.sc.desc + d;
        uint64_t excl = 0;
        if (tile > 0) {
            int64_t look = tile - 1;
            uint32_t spins = 0;
            bool done = false;
            while (!done) {
                uint64_t v[kLookWindow];
#pragma unroll
                for (int w = 0; w < kLookWindow; ++w)
                    v[w] = look - w >= 0
                               ? __hip_atomic_load(col + (look - w) * R, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT)
                               : 0ull;
                int used = 0;
#pragma unroll
                for (int w = 0; w < kLookWindow; ++w) {
                    if (done || used < w) continue;  // stopped earlier in this round
                    const bool ready = (uint32_t)((v[w] >> 56) & 63u) == tag && (v[w] >> 62) != 0;
                    if (!ready) continue;
                    excl += v[w] & ((1ull << 56) - 1);
                    used = w + 1;
                    if ((v[w] >> 62) == 2 || look - w == 0) done = true;
                }
                if (done) break;
                look -= used;
                if (used == 0) {
                    if (++spins > kSpinLimit) {  // bounded: never hang; flag it instead
                        atomicOr(p.sc.err, 1u);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __hip_atomic_store(desc + d, desc_make(kFlagPre, tag, excl + s_tcnt[d]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        s_gbase[d] += (uint32_t)excl;
    }
    __syncthreads();

    // write the digit runs: thread t takes staged slots t, t + kSortBlock, ...
    // (a staged row start also gives rowptr: the first slot of a run, whose
    // row an earlier tile may have seen too, or a slot after another row's)
    const int nvalid = (int)(p.n - tbase < kSortTile ? p.n - tbase : kSortTile);
    if (!HAS_B || fmt == kWide) {
        int32_t pos[HAS_B ? kSortItems : 1];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int i = (int)threadIdx.x + k * kSortBlock;
            if constexpr (HAS_B) pos[k] = -1;
            if (i < nvalid) {
                const uint32_t kk = s_stage[0][i];
                const uint32_t d = (kk >> p.shift) & (uint32_t)(R - 1);
                const uint32_t run = s_start[d];
                const int64_t q = (int64_t)s_gbase[d] + (i - (int64_t)run);
                if (q < p.n) {  // cannot fail for consistent counts; never write past n
                    if constexpr (HAS_B) pos[k] = (int32_t)q;
                    if constexpr (LAST) {
                        if (p.sc.keys)
                            p.sc.keys[q] = kk;
                        else if ((i == (int)run || kk != s_stage[0][i > 0 ? i - 1 : 0]) &&
                                 (int64_t)kk < p.rows)
                            atomicMin(p.sc.starts + kk, (uint32_t)q);
                        if constexpr (!HAS_B) p.a_out[q] = (int32_t)s_stage[1][i];
                    } else if constexpr (HAS_B) {
                        // the word's key half now, its payload half with the payload
                        reinterpret_cast<uint32_t*>(p.kv_out)[2 * q + 1] = kk;
                    } else {
                        p.kv_out[q] = ((uint64_t)kk << 32) | s_stage[1][i];
                    }
                }
            }
        }
        if constexpr (HAS_B) {
            // a and b, one at a time through the same buffer
            for (int which = 0; which < 2; ++which) {
                // a of a word: the low halves
                const bool half = !LAST && which == 0;
                int32_t* out = half ? reinterpret_cast<int32_t*>(p.kv_out)
                                    : (which == 0 ? p.a_out : p.b_out);
                __syncthreads();  // every read of the buffer's previous contents is done
#pragma unroll
                for (int k = 0; k < kSortItems; ++k) {
                    const int64_t i = wbase + (int64_t)k * kWave + lane;
                    if (i < p.n)
                        s_stage[0][s_lp[k * kSortBlock + threadIdx.x]] =
                            (uint32_t)(which == 0 ? va[k] : vb[k]);
                }
                __syncthreads();
#pragma unroll
                for (int k = 0; k < kSortItems; ++k)
                    if (pos[k] >= 0)
                        out[half ? 2 * (int64_t)pos[k] : (int64_t)pos[k]] =
                            (int32_t)s_stage[0][threadIdx.x + k * kSortBlock];
            }
        }
    } else if constexpr (HAS_B) {
        const bool key_hi = abits + p.b_bits >= 32;  // the key lies in a word's high half alone
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int i = (int)threadIdx.x + k * kSortBlock;
            if (i < nvalid) {
                const uint32_t hi = s_stage[0][i], lo = s_stage[1][i];
                const uint32_t kk = word.key(hi, lo);
                uint32_t d = (kk >> p.shift) & (uint32_t)(R - 1);
                if constexpr (!WIDE)
                    if (drop) d = s_dig[i];
                const uint32_t run = s_start[d];
                const int64_t q = (int64_t)s_gbase[d] + (i - (int64_t)run);
                if (q < p.n) {  // cannot fail for consistent counts; never write past n
                    if constexpr (LAST) {
                        const uint32_t v = drop ? put_digit(kk, d, p.shift, p.bits) : kk;
                        if (p.sc.keys) {
                            p.sc.keys[q] = v;
                        } else {
                            // within a run the keys differ exactly where the words' do
                            const int j = i > 0 ? i - 1 : 0;
                            const uint32_t kb = word.key(s_stage[0][j], key_hi ? 0u : s_stage[1][j]);
                            if ((i == (int)run || kk != kb) && (int64_t)v < p.rows)
                                atomicMin(p.sc.starts + v, (uint32_t)q);
                        }
                        p.a_out[q] = word.a(hi, lo);
                        p.b_out[q] = word.b(lo);
                    } else {
                        p.kv_out[q] = ((uint64_t)hi << 32) | lo;
                    }
                }
            }
        }
    }
}

// COO -> CSR of at most kSortSmall edges and rows, by one workgroup in one
// launch: the keys are counted into LDS for rowptr, then sorted with their COO
// ids by at most two stable passes between registers and LDS (wave-level
// multisplit, as in radix_onesweep), and the payloads are gathered by the sorted
// ids.  The look-back sort of so few edges is six to eight launches, each shorter
// than the gap to the next: mp_coo_to_csr from Python 57 -> 45 us (1k edges, 300
// rows), 72 -> 57 (10k, 2.7k), 88 -> 76 (16k, 16k), with ids and values 65 -> 50,
// 84 -> 65, 104 -> 88.  What bounds it is the serial chain of one CU, which is
// why it ends where radix_onesweep has more than one tile.
constexpr int kSmallBits = 7;
constexpr int kSmallBuckets = 1 << kSmallBits;
static_assert(kSortSmall <= kSortTile && kSortSmall <= 1 << (2 * kSmallBits), "two digits");

template <typename RP>
__global__ __launch_bounds__(kSortBlock) void sort_small(SmallSort p) {
    __shared__ uint32_t s_key[kSortSmall];  // the rows' counts, then keys in order
    __shared__ uint16_t s_id[kSortSmall];
    __shared__ uint16_t s_cnt[kSortWaves][kSmallBuckets];
    __shared__ uint32_t s_tcnt[kSmallBuckets], s_start[kSmallBuckets];
    __shared__ uint32_t s_wave[kSortWaves];
    constexpr int ITEMS = kSortSmall / kSortBlock;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int rounds = (p.n + kSortBlock - 1) / kSortBlock;
    const int wbase = wv * rounds * kWave;  // a wavefront's keys are consecutive

    for (int v = threadIdx.x; v < p.rows; v += kSortBlock) s_key[v] = 0;
    uint32_t key[ITEMS], id[ITEMS], rank[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = wbase + k * kWave + lane;
        id[k] = (uint32_t)i;
        key[k] = k < rounds && i < p.n ? p.dst[i] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k)
        if (k < rounds && wbase + k * kWave + lane < p.n && key[k] < (uint32_t)p.rows)
            atomicAdd(&s_key[key[k]], 1u);
    __syncthreads();

    // rowptr: exclusive scan of the counts, consecutive rows per thread
    {
        const int per = (p.rows + kSortBlock - 1) / kSortBlock;
        const int v0 = threadIdx.x * per;
        uint32_t c[ITEMS];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            c[k] = k < per && v0 + k < p.rows ? s_key[v0 + k] : 0u;
            sum += c[k];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off, kWave);
            if (lane >= off) inc += o;
        }
        if (lane == kWave - 1) s_wave[wv] = inc;
        __syncthreads();
        uint32_t run = inc - sum;
        for (int w = 0; w < wv; ++w) run += s_wave[w];
        RP* const rowptr = static_cast<RP*>(p.rowptr);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (k < per && v0 + k < p.rows) rowptr[v0 + k] = (RP)run;
            run += c[k];
        }
        if (threadIdx.x == 0) {
            rowptr[p.rows] = (RP)p.n;
            if (p.status) *p.status = (int32_t)MP_OK;
        }
    }

    const int R = 1 << p.width;
    for (int pass = 0; pass < p.passes; ++pass) {
        const int shift = pass * p.width;
        for (int i = threadIdx.x; i < kSortWaves * kSmallBuckets; i += kSortBlock)
            (&s_cnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (k < rounds) {
                const bool ok = wbase + k * kWave + lane < p.n;
                const uint32_t d = (key[k] >> shift) & (uint32_t)(R - 1);
                const uint64_t peers = digit_peers<kSmallBits>(ok, d, p.width);
                const uint32_t below = count_below(peers);
                const uint32_t base = s_cnt[wv][d];
                rank[k] = base + below;
                // (LDS operations of one wavefront run in order)
                if (ok && below == 0) s_cnt[wv][d] = (uint16_t)(base + (uint32_t)__popcll(peers));
            }
        }
        __syncthreads();
        for (int d = threadIdx.x; d < R; d += kSortBlock) {
            uint32_t run = 0;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t c = s_cnt[w][d];
                s_cnt[w][d] = (uint16_t)run;
                run += c;
            }
            s_tcnt[d] = run;
        }
        __syncthreads();
        if (wv == 0) wave_exclusive<kSmallBuckets>(s_tcnt, R, s_start, lane);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (k >= rounds || wbase + k * kWave + lane >= p.n) continue;
            const uint32_t d = (key[k] >> shift) & (uint32_t)(R - 1);
            const uint32_t lp = s_start[d] + s_cnt[wv][d] + rank[k];
            s_key[lp] = key[k];
            s_id[lp] = (uint16_t)id[k];
        }
        __syncthreads();
        if (pass + 1 < p.passes) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int i = wbase + k * kWave + lane;
                if (k >= rounds || i >= p.n) continue;
                key[k] = s_key[i];
                id[k] = s_id[i];
            }
        }
    }

    // every payload is read before any is written
    int32_t a[ITEMS];
    float v[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = k * kSortBlock + threadIdx.x;
        if (i >= p.n) continue;
        id[k] = s_id[i];
        a[k] = p.src[id[k]];
        if (p.val_out) v[k] = p.val_in[id[k]];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = k * kSortBlock + threadIdx.x;
        if (i >= p.n) continue;
        p.col[i] = a[k];
        if (p.perm) p.perm[i] = (int32_t)id[k];
        if (p.val_out) p.val_out[i] = v[k];
    }
}

// The caller's status word: MP_OK where no sort ran.
__global__ void status_ok(int32_t* __restrict__ status) {
    if (threadIdx.x == 0) *status = (int32_t)MP_OK;
}

// rowptr where edges are many next to rows, from the rows' first positions
// (kNoStart: an empty row, whose start is that of the next row that has one, E
// after the last): a suffix minimum, as the starts ascend.  rows_first finds
// the least start of every tile of kFirstTile rows; rows_finish looks for the
// next tile that has one, then scans its own tile from the end.
constexpr int kFirstTile = 8192;
constexpr int kFirstBlock = 1024;

__global__ __launch_bounds__(kFirstBlock) void rows_first(const uint32_t* __restrict__ starts,
                                                          int64_t N, uint32_t* __restrict__ first) {
    __shared__ uint32_t s_min[kFirstBlock / kWave];
    uint32_t m = kNoStart;
#pragma unroll
    for (int k = 0; k < kFirstTile / kFirstBlock; ++k) {
        const int64_t v = (int64_t)blockIdx.x * kFirstTile + k * kFirstBlock + threadIdx.x;
        const uint32_t s = v < N ? starts[v] : kNoStart;
        m = s < m ? s : m;
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_xor(m, off);
        m = o < m ? o : m;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) s_min[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kFirstBlock / kWave; ++w) m = s_min[w] < m ? s_min[w] : m;
        first[blockIdx.x] = m;
    }
}

// In place: first[t] = the least of first[t], first[t + 1], ... by one
// workgroup, each thread taking consecutive tiles.  For the many tiles over
// which rows_finish's own look ahead, 64 tiles a step, would become most of its
// time where all edges end in the first rows (140M edges, 64M rows, the whole
// sort: 3627 -> 3437 us).
constexpr int64_t kLookTiles = 1024;  // tiles up to which rows_finish looks itself

__global__ __launch_bounds__(1024) void rows_suffix(uint32_t* __restrict__ first, int64_t tiles) {
    __shared__ uint32_t s_min[1024 / kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int64_t per = (tiles + 1023) / 1024;
    const int64_t t0 = threadIdx.x * per < tiles ? threadIdx.x * per : tiles;
    const int64_t t1 = t0 + per < tiles ? t0 + per : tiles;
    uint32_t m = kNoStart;
    for (int64_t t = t0; t < t1; ++t) m = first[t] < m ? first[t] : m;
    // least of the threads after this one
    uint32_t inc = m;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_down(inc, off, kWave);
        if (lane + off < kWave && o < inc) inc = o;
    }
    if (lane == 0) s_min[wv] = inc;
    __syncthreads();
    uint32_t run = __shfl_down(inc, 1, kWave);
    if (lane == kWave - 1) run = kNoStart;
    for (int w = wv + 1; w < 1024 / kWave; ++w) run = s_min[w] < run ? s_min[w] : run;
    for (int64_t t = t1 - 1; t >= t0; --t) {
        const uint32_t f = first[t];
        run = f < run ? f : run;
        first[t] = run;
    }
}

// Also the caller's status word (nullptr: not wanted); with the sort's error
// word set, rowptr is left alone.  SUFFIX: rows_suffix has run.
template <typename RP, bool SUFFIX>
__global__ __launch_bounds__(kFirstBlock) void rows_finish(const uint32_t* __restrict__ starts,
                                                           int64_t N, int64_t E,
                                                           const uint32_t* __restrict__ first,
                                                           const uint32_t* __restrict__ err,
                                                           int32_t* __restrict__ status,
                                                           RP* __restrict__ rowptr) {
    constexpr int PER = kFirstTile / kFirstBlock;  // consecutive rows per thread
    __shared__ uint32_t s_min[kFirstBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const bool failed = *err != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && status)
        *status = failed ? (int32_t)MP_ERR_SORT : (int32_t)MP_OK;
    if (failed) return;
    // the least start of the later tiles: that of the next tile that has any
    uint32_t after = (uint32_t)E;
    if constexpr (SUFFIX) {
        if ((int64_t)blockIdx.x + 1 < gridDim.x) {
            const uint32_t f = first[blockIdx.x + 1];
            if (f != kNoStart) after = f;
        }
    } else {
        for (int64_t t = (int64_t)blockIdx.x + 1; t < gridDim.x; t += kWave) {
            const uint32_t f = t + lane < gridDim.x ? first[t + lane] : kNoStart;
            const uint64_t some = __ballot(f != kNoStart);
            if (some) {
                after = __shfl(f, __ffsll((unsigned long long)some) - 1);
                break;
            }
        }
    }
    const int64_t v0 = (int64_t)blockIdx.x * kFirstTile + (int64_t)threadIdx.x * PER;
    uint32_t s[PER];
    uint32_t m = kNoStart;
#pragma unroll
    for (int k = PER - 1; k >= 0; --k) {
        s[k] = v0 + k < N ? starts[v0 + k] : kNoStart;
        m = s[k] < m ? s[k] : m;
    }
    // least start of the threads after this one
    uint32_t inc = m;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_down(inc, off, kWave);
        if (lane + off < kWave && o < inc) inc = o;
    }
    if (lane == 0) s_min[wv] = inc;
    __syncthreads();
    uint32_t run = __shfl_down(inc, 1, kWave);
    if (lane == kWave - 1) run = kNoStart;
    for (int w = wv + 1; w < kFirstBlock / kWave; ++w) run = s_min[w] < run ? s_min[w] : run;
    if (after < run) run = after;
#pragma unroll
    for (int k = PER - 1; k >= 0; --k) {
        run = s[k] < run ? s[k] : run;
        if (v0 + k < N) rowptr[v0 + k] = (RP)run;
        if (v0 + k == N) rowptr[N] = (RP)E;
    }
}

// rowptr from the sorted keys, where the rows are many (rowptr_by_keys): the
// number of keys below v, by merged ranges of keys and rows.  Also the caller's
// status word; with the sort's error word set, rowptr is left alone.
struct KeyRows {
    const uint32_t* keys;
    int64_t N;
    uint32_t mask;  // the bits that were sorted by
    __device__ inline int64_t operator()(int64_t i) const {
        const int64_t k = (int64_t)(keys[i] & mask) + 1;
        return k < N ? k : N;
    }
};

template <typename RP, bool VEC, int SPAN>
__global__ __launch_bounds__(kMergeBlock) void rowptr_from_keys(const uint32_t* __restrict__ keys,
                                                                uint32_t mask, int64_t E, int64_t N,
                                                                const uint32_t* __restrict__ err,
                                                                int32_t* __restrict__ status,
                                                                RP* __restrict__ rowptr) {
    const bool failed = *err != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (status) *status = failed ? (int32_t)MP_ERR_SORT : (int32_t)MP_OK;
        if (!failed) rowptr[N] = (RP)E;
    }
    if (failed) return;  // the same for all threads
    merge_counts<SPAN, VEC>(KeyRows{keys, N, mask}, E, N, rowptr);
}

// rowptr[v] = the first position p with keys[p] >= v (E if none), by binary
// search: the CSR of keys sorted by the caller, with work bounded by
// (N + 1) * log2(E) reads whatever the order of keys.
template <typename RP>
__global__ __launch_bounds__(256) void rowptr_by_search(const uint32_t* __restrict__ keys,
                                                        int64_t E, int64_t N, RP* __restrict__ rowptr) {
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v <= N;
         v += (int64_t)gridDim.x * 256) {
        int64_t lo = 0, hi = E;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)keys[mid] < v) lo = mid + 1; else hi = mid;
        }
        rowptr[v] = (RP)(v == N ? E : lo);
    }
}

template <typename RP>
__global__ __launch_bounds__(256) void fill_zero(int64_t n, RP* __restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        out[i] = 0;
}

__global__ __launch_bounds__(256) void gather_f32(const float* __restrict__ in,
                                                  const int32_t* __restrict__ idx, int64_t n,
                                                  float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = in[idx[i]];
}

__global__ __launch_bounds__(256) void copy_i32(const int32_t* __restrict__ in, int64_t n,
                                                int32_t* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = in[i];
}

// The relations' edges one after another, as global (source) and row
// (destination) ids.  Bound by its 16 bytes of traffic per edge: a block takes
// kConcatItems edges per thread of one relation, all loads before all stores.
// (A launch per relation and array, one edge per thread, took 110 us for the
// typed graph's 20.6M edges; now 54 us.)
constexpr int kConcatItems = 8;

__global__ __launch_bounds__(256) void concat_relations(ConcatParams P) {
    int r = 0;
    while (r + 1 < P.n && (int64_t)blockIdx.x >= P.block_off[r + 1]) ++r;
    const int64_t base = ((int64_t)blockIdx.x - P.block_off[r]) * 256 * kConcatItems + threadIdx.x;
    const int64_t E = P.E[r], to = P.off[r];
    int32_t a[kConcatItems], b[kConcatItems];
#pragma unroll
    for (int k = 0; k < kConcatItems; ++k) {
        const int64_t i = base + k * 256;
        a[k] = i < E ? __builtin_nontemporal_load(P.src[r] + i) : 0;
        b[k] = i < E ? __builtin_nontemporal_load(P.dst[r] + i) : 0;
    }
#pragma unroll
    for (int k = 0; k < kConcatItems; ++k) {
        const int64_t i = base + k * 256;
        if (i < E) {
            P.src_out[to + i] = a[k] + P.src_add[r];
            P.dst_out[to + i] = b[k] + P.dst_add[r];
        }
    }
}

__global__ __launch_bounds__(256) void iota_i32(int64_t n, int32_t* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (int32_t)i;
}

__global__ __launch_bounds__(256) void copy_f32(const float* __restrict__ in, int64_t n,
                                                float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = in[i];
}

__global__ void zero_i64(int64_t* p) { *p = 0; }

__global__ __launch_bounds__(256) void validate_sorted(const int32_t* __restrict__ dst, int64_t E,
                                                       unsigned long long* count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i > 0 && i < E && dst[i] < dst[i - 1]) atomicAdd(count, 1ull);
}

__global__ __launch_bounds__(256) void validate_coo(const int32_t* __restrict__ src,
                                                    const int32_t* __restrict__ dst, int64_t E,
                                                    int64_t N_src, int64_t N_dst,
                                                    unsigned long long* count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned bad = 0;
    if (i < E) {
        bad += (src[i] < 0 || src[i] >= N_src) ? 1u : 0u;
        bad += (dst[i] < 0 || dst[i] >= N_dst) ? 1u : 0u;
    }
    if (bad) atomicAdd(count, (unsigned long long)bad);
}

template <typename RP>
__global__ __launch_bounds__(256) void validate_csr(const RP* __restrict__ rowptr,
                                                    const int32_t* __restrict__ col,
                                                    int64_t N_dst, int64_t N_src, int64_t E,
                                                    unsigned long long* count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned bad = 0;
    if (i < N_dst) bad += (rowptr[i + 1] < rowptr[i]) ? 1u : 0u;
    if (i == 0) {
        bad += (rowptr[0] != 0) ? 1u : 0u;
        bad += ((int64_t)rowptr[N_dst] != E) ? 1u : 0u;
    }
    if (i < E) bad += (col[i] < 0 || col[i] >= N_src) ? 1u : 0u;
    if (bad) atomicAdd(count, (unsigned long long)bad);
}

inline unsigned grid_for(int64_t n, int per_block) {
    return (unsigned)ceil_div(n > 0 ? n : 1, per_block);
}

}  // namespace

size_t radix_scratch_bytes(int64_t n, int64_t N) {
    return radix_scratch(nullptr, n, N).bytes;
}

RadixScratch radix_scratch(void* base, int64_t n, int64_t N) {
    const int64_t tiles = ceil_div(n > 0 ? n : 1, kSortTile);
    char* b = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* q = b ? b + off : nullptr;
        off += align_up(bytes, 256);
        return q;
    };
    RadixScratch sc;
    sc.desc = reinterpret_cast<uint64_t*>(take((size_t)tiles * kMaxBuckets * sizeof(uint64_t)));
    sc.ghist = reinterpret_cast<uint32_t*>(take(kMaxPasses * kMaxBuckets * sizeof(uint32_t)));
    sc.counter = reinterpret_cast<uint32_t*>(take(kMaxPasses * sizeof(uint32_t)));
    sc.err = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t)));
    sc.a_or = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t)));
    if (rowptr_by_keys(n, N)) {
        sc.keys = reinterpret_cast<uint32_t*>(take((size_t)n * sizeof(uint32_t)));
        sc.starts = sc.first = nullptr;
    } else {
        sc.keys = nullptr;
        sc.starts = reinterpret_cast<uint32_t*>(take((size_t)N * sizeof(uint32_t)));
        sc.first = reinterpret_cast<uint32_t*>(take((size_t)ceil_div(N + 1, kFirstTile) * sizeof(uint32_t)));
    }
    sc.bytes = off;
    return sc;
}

hipError_t radix_sort_begin(const uint32_t* keys, const int32_t* a, int64_t n, int64_t N,
                            const DigitPlan& dp, const RadixScratch& sc, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (dp.passes < 1 || dp.passes > kMaxPasses) return hipErrorInvalidValue;
    uint32_t shifts = 0, widths = 0;
    for (int p = 0; p < dp.passes; ++p) {
        if (dp.width[p] < 1 || dp.width[p] > kSortMaxBits || dp.shift[p] < 0 ||
            dp.shift[p] + dp.width[p] > 32)
            return hipErrorInvalidValue;
        shifts |= (uint32_t)dp.shift[p] << (8 * p);
        widths |= (uint32_t)dp.width[p] << (8 * p);
    }
    const int64_t tiles = ceil_div(n, kSortTile);
    // a pass over R = 2^width digits uses R descriptors per tile
    const int64_t ndesc = tiles * ((int64_t)1 << dp.max_width);
    const int64_t nstarts = sc.starts ? N : 0;
    unsigned g = grid_for(ndesc > nstarts ? ndesc : nstarts, 256);
    if (g > 8192) g = 8192;
    // every histogram word needs a thread, however few descriptors there are
    if (g < (unsigned)ceil_div(kMaxPasses * kMaxBuckets, 256)) g = (unsigned)ceil_div(kMaxPasses * kMaxBuckets, 256);
    hipLaunchKernelGGL(radix_clear, dim3(g), dim3(256), 0, s, sc, ndesc, nstarts);
    unsigned gh = grid_for(n, kGhistBlock * kGhistItems);
    if (gh > kGhistMaxGrid) gh = kGhistMaxGrid;
    hipLaunchKernelGGL(radix_ghist, dim3(gh), dim3(kGhistBlock), 0, s, keys, a, n, dp.passes, shifts,
                       widths, sc);
    return hipGetLastError();
}

template <bool HAS_B, bool WIDE>
void launch_onesweep(const RadixPass& p, int64_t tiles, hipStream_t s) {
    const dim3 g((unsigned)tiles), b(kSortBlock);
    const bool first = p.keys_in != nullptr, last = p.a_out != nullptr;
    if (first && last)
        hipLaunchKernelGGL((radix_onesweep<HAS_B, WIDE, true, true>), g, b, 0, s, p);
    else if (first)
        hipLaunchKernelGGL((radix_onesweep<HAS_B, WIDE, true, false>), g, b, 0, s, p);
    else if (last)
        hipLaunchKernelGGL((radix_onesweep<HAS_B, WIDE, false, true>), g, b, 0, s, p);
    else
        hipLaunchKernelGGL((radix_onesweep<HAS_B, WIDE, false, false>), g, b, 0, s, p);
}

hipError_t radix_sort_pass(const RadixPass& p, hipStream_t s) {
    if (p.n <= 0) return hipSuccess;
    const int64_t tiles = ceil_div(p.n, kSortTile);
    const bool wide = p.bits > kSortMaxBits - 1;
    if (p.b_out) {
        if (wide) launch_onesweep<true, true>(p, tiles, s);
        else launch_onesweep<true, false>(p, tiles, s);
    } else {
        if (wide) launch_onesweep<false, true>(p, tiles, s);
        else launch_onesweep<false, false>(p, tiles, s);
    }
    return hipGetLastError();
}

hipError_t launch_sort_small(SmallSort p, int key_bits, int rp64, hipStream_t s) {
    p.passes = key_bits > kSmallBits ? 2 : 1;
    p.width = (key_bits + p.passes - 1) / p.passes;
    if (rp64) hipLaunchKernelGGL(sort_small<int64_t>, dim3(1), dim3(kSortBlock), 0, s, p);
    else hipLaunchKernelGGL(sort_small<int32_t>, dim3(1), dim3(kSortBlock), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_status_ok(int32_t* status, hipStream_t s) {
    if (!status) return hipSuccess;
    hipLaunchKernelGGL(status_ok, dim3(1), dim3(64), 0, s, status);
    return hipGetLastError();
}

namespace {

template <typename RP, int SPAN>
hipError_t rowptr_keys_span(const RadixScratch& sc, uint32_t mask, int64_t E, int64_t N, RP* rowptr,
                            int32_t* status, hipStream_t s) {
    const dim3 g((unsigned)ceil_div(E + N, SPAN)), b(kMergeBlock);
    if ((uintptr_t)rowptr % 16 == 0)  // four entries per store
        hipLaunchKernelGGL((rowptr_from_keys<RP, true, SPAN>), g, b, 0, s, sc.keys, mask, E, N, sc.err,
                           status, rowptr);
    else
        hipLaunchKernelGGL((rowptr_from_keys<RP, false, SPAN>), g, b, 0, s, sc.keys, mask, E, N, sc.err,
                           status, rowptr);
    return hipGetLastError();
}

template <typename RP>
hipError_t rowptr_keys(const RadixScratch& sc, uint32_t mask, int64_t E, int64_t N, RP* rowptr,
                       int32_t* status, hipStream_t s) {
    return E + N < kMergeLong
               ? rowptr_keys_span<RP, kMergeSpanShort>(sc, mask, E, N, rowptr, status, s)
               : rowptr_keys_span<RP, kMergeSpanLong>(sc, mask, E, N, rowptr, status, s);
}

template <typename RP>
hipError_t rowptr_starts(const RadixScratch& sc, int64_t E, int64_t N, RP* rowptr, int32_t* status,
                         hipStream_t s) {
    const int64_t tiles = ceil_div(N + 1, kFirstTile);
    const dim3 g((unsigned)tiles), b(kFirstBlock);
    // (a single tile has no later ones)
    if (tiles > 1) hipLaunchKernelGGL(rows_first, g, b, 0, s, sc.starts, N, sc.first);
    if (tiles > kLookTiles) {
        hipLaunchKernelGGL(rows_suffix, dim3(1), dim3(1024), 0, s, sc.first, tiles);
        hipLaunchKernelGGL((rows_finish<RP, true>), g, b, 0, s, sc.starts, N, E, sc.first, sc.err,
                           status, rowptr);
    } else {
        hipLaunchKernelGGL((rows_finish<RP, false>), g, b, 0, s, sc.starts, N, E, sc.first, sc.err,
                           status, rowptr);
    }
    return hipGetLastError();
}

}  // namespace

// The keys cost 8 bytes of traffic per edge, the starts 20 per row, an atomic
// per row that has edges, and a launch more.  Whole COO -> CSR, us, by starts ->
// by keys: 10M edges over 40M rows 515 -> 308 (with ids 600 -> 402), 20M 368 ->
// 290, 10M 289 -> 269, 5M 257 -> 254, 2.5M 241 -> 244; 1M edges over 10M rows
// 149 -> 96, 250k 71 -> 66; 100k over 50k 56 -> 48.  (Filling the rows between
// two keys by the later key's thread was as fast on even rows, but one thread's
// work where no edge ends in the last rows: 1 s for 40M rows.)
bool rowptr_by_keys(int64_t E, int64_t N) {
    return E <= 2 * N || (E <= 4 * N && E < kMergeLong);
}

hipError_t launch_rowptr(const RadixScratch& sc, int key_bits, int64_t E, int64_t N, void* rowptr,
                         int rp64, int32_t* status, hipStream_t s) {
    if (sc.keys) {
        const uint32_t mask = key_bits < 32 ? (1u << key_bits) - 1u : ~0u;
        return rp64 ? rowptr_keys(sc, mask, E, N, static_cast<int64_t*>(rowptr), status, s)
                    : rowptr_keys(sc, mask, E, N, static_cast<int32_t*>(rowptr), status, s);
    }
    return rp64 ? rowptr_starts(sc, E, N, static_cast<int64_t*>(rowptr), status, s)
                : rowptr_starts(sc, E, N, static_cast<int32_t*>(rowptr), status, s);
}

hipError_t launch_rowptr_by_search(const uint32_t* keys, int64_t E, int64_t N, void* rowptr,
                                   int rp64, hipStream_t s) {
    const unsigned g = grid_for(N + 1, 256);
    if (rp64)
        hipLaunchKernelGGL((rowptr_by_search<int64_t>), dim3(g), dim3(256), 0, s, keys, E, N,
                           static_cast<int64_t*>(rowptr));
    else
        hipLaunchKernelGGL((rowptr_by_search<int32_t>), dim3(g), dim3(256), 0, s, keys, E, N,
                           static_cast<int32_t*>(rowptr));
    return hipGetLastError();
}

hipError_t launch_fill_rowptr_zero(int64_t N, void* rowptr, int rp64, hipStream_t s) {
    const int64_t n = N + 1;
    unsigned g = grid_for(n, 256);
    if (g > 65536) g = 65536;
    if (rp64)
        hipLaunchKernelGGL(fill_zero<int64_t>, dim3(g), dim3(256), 0, s, n,
                           static_cast<int64_t*>(rowptr));
    else
        hipLaunchKernelGGL(fill_zero<int32_t>, dim3(g), dim3(256), 0, s, n,
                           static_cast<int32_t*>(rowptr));
    return hipGetLastError();
}

hipError_t launch_gather_f32(const float* in, const int32_t* idx, int64_t n, float* out,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_f32, dim3(grid_for(n, 256)), dim3(256), 0, s, in, idx, n, out);
    return hipGetLastError();
}

hipError_t launch_copy_i32(const int32_t* in, int64_t n, int32_t* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_i32, dim3(grid_for(n, 256)), dim3(256), 0, s, in, n, out);
    return hipGetLastError();
}

hipError_t launch_concat_relations(ConcatParams p, hipStream_t s) {
    int64_t blocks = 0;
    for (int r = 0; r < p.n; ++r) {
        p.block_off[r] = blocks;
        blocks += ceil_div(p.E[r], 256 * kConcatItems);
    }
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(concat_relations, dim3((unsigned)blocks), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_iota(int64_t n, int32_t* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(iota_i32, dim3(grid_for(n, 256)), dim3(256), 0, s, n, out);
    return hipGetLastError();
}

hipError_t launch_copy_f32(const float* in, int64_t n, float* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_f32, dim3(grid_for(n, 256)), dim3(256), 0, s, in, n, out);
    return hipGetLastError();
}

hipError_t launch_validate_sorted(const int32_t* dst, int64_t E, int64_t* d_count,
                                  hipStream_t s) {
    hipLaunchKernelGGL(zero_i64, dim3(1), dim3(1), 0, s, d_count);
    if (E > 1)
        hipLaunchKernelGGL(validate_sorted, dim3(grid_for(E, 256)), dim3(256), 0, s, dst, E,
                           reinterpret_cast<unsigned long long*>(d_count));
    return hipGetLastError();
}

hipError_t launch_validate_coo(const int32_t* src, const int32_t* dst, int64_t E, int64_t N_src,
                               int64_t N_dst, int64_t* d_count, hipStream_t s) {
    hipLaunchKernelGGL(zero_i64, dim3(1), dim3(1), 0, s, d_count);
    if (E > 0)
        hipLaunchKernelGGL(validate_coo, dim3(grid_for(E, 256)), dim3(256), 0, s, src, dst, E,
                           N_src, N_dst, reinterpret_cast<unsigned long long*>(d_count));
    return hipGetLastError();
}

hipError_t launch_validate_csr(const void* rowptr, int rp64, const int32_t* col, int64_t N_dst,
                               int64_t N_src, int64_t E, int64_t* d_count, hipStream_t s) {
    hipLaunchKernelGGL(zero_i64, dim3(1), dim3(1), 0, s, d_count);
    const int64_t n = (N_dst > E ? N_dst : E) + 1;
    auto* c = reinterpret_cast<unsigned long long*>(d_count);
    if (rp64)
        hipLaunchKernelGGL(validate_csr<int64_t>, dim3(grid_for(n, 256)), dim3(256), 0, s,
                           static_cast<const int64_t*>(rowptr), col, N_dst, N_src, E, c);
    else
        hipLaunchKernelGGL(validate_csr<int32_t>, dim3(grid_for(n, 256)), dim3(256), 0, s,
                           static_cast<const int32_t*>(rowptr), col, N_dst, N_src, E, c);
    return hipGetLastError();
}

}  // namespace mp
