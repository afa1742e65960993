// Vectorised dynamic feature cache (section 4.3 of the paper) on gfx950: C ABI of
// include/tns_cache.h and its kernels.  Everything a fetch does is queued on the caller's stream:
// lookup, row gather, score update, selection of the victims (radix select over the scores),
// insertion of the missed rows.  No host round trip, no allocation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <new>
#include <type_traits>

#include "../../include/tns_cache.h"
#include "tns_chain.h"
#include "tns_internal.h"
#include "tns_lanes.h"
#include "tns_test_hooks.h"

using tns::DeviceGuard;
using tns::fail;
using tns::fail_hip;

namespace {

constexpr int kWave = 64;
constexpr int kScanTile = 1024;           // elements per workgroup in the scans
constexpr int kNoIndex = INT_MAX;
constexpr int kStripes = 64;

// Radix select of the victims' threshold: 32-bit keys in digits of 11, 11 and 10 bits, most significant first.  The
// update is a chain of short launches, so a pass less is worth the larger histograms (batch of 66600 ids, 42 K entries:
// 87.3 us per fetch with four passes of 8 bits, 83.1 with three).
constexpr int kPasses = 3, kBins = 2048, kBinsPerThread = kBins / 256;
__host__ __device__ constexpr int digit_shift(int pass) { return pass == 0 ? 21 : (pass == 1 ? 10 : 0); }
__host__ __device__ constexpr uint32_t digit_mask(int pass) { return pass == 2 ? 1023u : 2047u; }

// Device-side scalars of one fetch.
struct Ctl {
    uint32_t prefix, mask;                // radix select: decided high bits of the threshold key (final, after the last pass)
    int32_t remaining;                    // how many entries are still to be taken among keys equal to the threshold
    int32_t m;                            // entries replaced by this update
    int32_t n_unique;                     // distinct missed ids of the batch
    int32_t now;                          // LRU: number of this update; 0 otherwise
    int64_t ring;                         // FIFO: slot of the first entry replaced by this update
    // state after each pass of the radix select (index p = after p passes; 0 = nothing decided) and the histogram
    // each pass fills: a pass's digit is picked by the kernel that follows it, in every workgroup's prologue
    uint32_t sel_prefix[kPasses + 1], sel_mask[kPasses + 1];
    int32_t sel_rem[kPasses + 1];
    alignas(16) int32_t hist[kPasses][kBins];
};

struct CacheState {
    int32_t* slot_of;    // [num_ids]   slot of a cached id, -1 otherwise
    int32_t* first_idx;  // [num_ids]   scratch: first batch position of a missed id (kNoIndex between fetches)
    int32_t* id_of;      // [capacity]  id held by a slot, -1 if empty
    // [capacity]  LFU: access count.  LRU: the number of the update that last accessed the entry; its recent score is that
    // minus the number of the latest update, so that no update has to decrement every score (all arithmetic modulo 2^32).
    int32_t* score;
    int32_t* updates;    // LRU: number of updates so far; 0 otherwise
    float* rows;         // [capacity * dim]
    unsigned long long* counters;  // [kStripes][3]: hits, misses, replaced (striped: one hot word would serialise the batch)
    int64_t* ring;       // FIFO position
    int64_t capacity;
};

__global__ void __launch_bounds__(256) k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// slot_of from id_of (after a restore)
__global__ void __launch_bounds__(256) k_rebuild_map(const int32_t* __restrict__ id_of, int64_t capacity, int64_t num_ids,
                                                     int32_t* __restrict__ slot_of) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s < capacity) {
        const int32_t id = id_of[s];
        if (id >= 0 && id < num_ids) slot_of[id] = (int32_t)s;
    }
}

// Lookup of the batch against the cache as it is before the update; accesses are recorded.  A thread takes
// kLookupUnroll ids, one grid width apart, and runs each dependent step for all of them before the next.
//
// Feature ids follow a power law, so thousands of lanes record an access of the same entry, and a device-wide atomic
// on one word completes about every 20 ns here whatever the rest of the chip does (batch of 2^20 Zipf(1.05) ids, LFU:
// 60 K accesses of the hottest entry, 1150 us for this kernel alone and as long for the row gather beside it).  The
// accesses are therefore combined per workgroup first, in an LDS hash table twice the size of its ids (linear
// probing: it never fills), and one atomic per distinct entry of the workgroup goes to memory.  The same table holds
// the smallest batch position of every missed id.
constexpr int kLookupUnroll = 4;
constexpr int kLookupTable = 2 * 256 * kLookupUnroll;      // power of two
constexpr int32_t kFreeKey = INT_MIN;                      // hits: slot >= 0; misses: -1 - id > INT_MIN
__global__ void __launch_bounds__(256) k_lookup(const CacheState c, int policy, int64_t num_ids, int64_t B,
                                                const int32_t* __restrict__ ids, int32_t* __restrict__ slots,
                                                uint8_t* __restrict__ hit, Ctl* ctl, tns::ScanWorkspace* chain,
                                                uint32_t first_ticket) {
    __shared__ int32_t s_key[kLookupTable], s_val[kLookupTable];
    __shared__ int32_t s_hits, s_misses;
    const int32_t now = policy == TNS_CACHE_LRU ? (int32_t)((uint32_t)*c.updates + 1u) : 0;
    if (blockIdx.x == 0) {          // scalars of this update
        if (threadIdx.x == 0) { ctl->now = now; ctl->prefix = 0; ctl->mask = 0; ctl->remaining = 0; ctl->m = 0; ctl->n_unique = 0; }
        int4* const all = reinterpret_cast<int4*>(&ctl->hist[0][0]);
#pragma unroll
        for (int i = 0; i < kPasses * kBins / 4 / 256; ++i) all[i * 256 + threadIdx.x] = make_int4(0, 0, 0, 0);
        if (chain && threadIdx.x == 1) chain->ticket = first_ticket;
    }
    if (chain && threadIdx.x == 0) chain->status[blockIdx.x] = 0;      // a workgroup here and a tile of the chain are both 1024 ids
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t b0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int32_t id[kLookupUnroll], s[kLookupUnroll];
#pragma unroll
    for (int u = 0; u < kLookupUnroll; ++u) id[u] = ids[min(b0 + (int64_t)u * stride, B - 1)];
#pragma unroll
    for (int u = 0; u < kLookupUnroll; ++u) {
        const bool in_range = id[u] >= 0 && id[u] < num_ids;
        s[u] = c.slot_of[in_range ? id[u] : 0];
        if (!in_range) s[u] = -2;                         // -2: id out of range
    }
    for (int i = threadIdx.x; i < kLookupTable; i += 256) s_key[i] = kFreeKey;
    if (threadIdx.x == 0) { s_hits = 0; s_misses = 0; }
    __syncthreads();
    // entry of `key` in the table; a value starts at 0 (hits count up) and misses keep INT_MAX - (smallest position)
    // as a maximum, so that both start at the same neutral value
    auto entry_of = [&](int32_t key) -> int {
        uint32_t e = ((uint32_t)key * 2654435761u) >> 16;
        while (true) {
            e &= kLookupTable - 1;
            const int32_t k = atomicCAS(&s_key[e], kFreeKey, key);
            if (k == kFreeKey || k == key) return (int)e;
            ++e;
        }
    };
    for (int i = threadIdx.x; i < kLookupTable; i += 256) s_val[i] = 0;
    __syncthreads();
    int32_t h = 0, m = 0;
#pragma unroll
    for (int u = 0; u < kLookupUnroll; ++u) {
        const int64_t b = b0 + (int64_t)u * stride;
        int is_hit = 0, is_miss = 0;
        if (b < B) {
            if (s[u] >= 0) {
                is_hit = 1;
                if (policy == TNS_CACHE_LRU) c.score[s[u]] = now;
                else if (policy == TNS_CACHE_LFU) atomicAdd(&s_val[entry_of(s[u])], 1);
            } else if (s[u] == -1) {
                is_miss = 1;
                atomicMax(&s_val[entry_of(-1 - id[u])], INT_MAX - (int32_t)b);   // first occurrence of a missed id
            }
            slots[b] = s[u];
            if (hit) hit[b] = (uint8_t)is_hit;
        }
        h += __popcll(__ballot(is_hit));
        m += __popcll(__ballot(is_miss));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&s_hits, h);
        atomicAdd(&s_misses, m);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kLookupTable; i += 256) {
        const int32_t key = s_key[i];
        if (key == kFreeKey) continue;
        if (key >= 0) atomicAdd(&c.score[key], s_val[i]);
        else atomicMin(&c.first_idx[-1 - key], INT_MAX - s_val[i]);
    }
    if (threadIdx.x < 2) {
        const int32_t v = threadIdx.x == 0 ? s_hits : s_misses;
        if (v) atomicAdd(&c.counters[(size_t)(blockIdx.x % kStripes) * 3 + threadIdx.x], (unsigned long long)v);
    }
}

// out[b] = cached row or row of the backing store; VEC floats per thread, rows stay coalesced
// The slot comes from the id map directly, so the gather does not
// wait for the lookup kernel, which records the accesses for the update beside it.  A thread moves kGatherUnroll
// pieces, one workgroup's width apart: the kernel is a copy, and a copy on this machine is bound by how much each compute unit has
// in flight.  The row of a piece is found by a multiplication; with 64-bit divisions eight pieces took 849 vector
// instructions and 90 registers (five waves per SIMD), now 233 and 61 (eight).  2^20 rows of 172 floats: Zipf ids 353 -> 342 us,
// consecutive rows 281 -> 272, any of 2^24 rows 380 -> 370: of what a copy reaches, the rest is rows that begin and end inside
// lines and lie anywhere.
constexpr int kGatherUnroll = 8;
// In the launch with the update a thread moves half as many pieces of 16 bytes: its workgroups have 1024 threads, and with eight pieces
// 66600 rows of 172 floats are 350 workgroups, of which a third of the compute units got two and took twice as long (gather done at
// 22 us, half of it at 10).  us per fetch with 8 / 4 / 3 / 2: 66600 rows 33.5 / 31.4 / 31.5 / 32.8, 200000 71.2 / 67.1 / 67.2 / 71.5, 16000 as
// before; pieces of 4 bytes, 66600 rows of 173 floats, 38.0 / 41.6 / 45.9 / 54.1.
__host__ __device__ constexpr int update_unroll(int vec) { return vec == 4 ? 4 : kGatherUnroll; }

// Row of piece t where a row has `per_row` of them, for t < 2^31: floor(t / per_row) = t * mul >> shift, with mul =
// ceil(2^shift / per_row) and 2^(shift - 31) >= per_row, so that the product's error stays below 1 / per_row.
struct RowOf {
    uint32_t mul, shift, per_row;
    __device__ __forceinline__ uint32_t operator()(uint32_t t) const { return (uint32_t)(((uint64_t)t * mul) >> shift); }
};
RowOf row_of(int32_t per_row) {
    uint32_t s = 0;
    while ((int64_t(1) << s) < per_row) ++s;
    const uint64_t p = uint64_t(1) << (31 + s);
    return RowOf{(uint32_t)((p + (uint64_t)per_row - 1) / (uint64_t)per_row), 31 + s, (uint32_t)per_row};
}
constexpr int64_t kGatherPieces = int64_t(1) << 31;       // of one launch

// The pieces of a thread, THREADS apart from t0 on: from cached row s[u], from the store's row id[u] (s[u] = -1), or zeros (s[u] = -2).
template <int VEC, int THREADS, int UNROLL>
__device__ __forceinline__ void move_pieces(const float* __restrict__ rows, const float* __restrict__ store, int32_t dim, uint32_t total,
                                            uint32_t t0, const uint32_t (&col)[UNROLL], const int32_t (&id)[UNROLL], const int32_t (&s)[UNROLL],
                                            float* __restrict__ out) {
    // the output is touched once (non-temporal); the cached rows are what should stay in the L2
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    vec_t v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const float* const from = s[u] >= 0 ? rows : store;
        const uint32_t r = s[u] >= 0 ? (uint32_t)s[u] : (s[u] == -1 ? (uint32_t)id[u] : 0u);
        v[u] = *reinterpret_cast<const vec_t*>(from + ((uint64_t)r * (uint32_t)dim + col[u]));
    }
    // Every row piece has arrived before the first store is issued (what a copy reaches in the two orders: tns_probe.hip).
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        float x = v[u][0];
        asm volatile("" : "+v"(x));         // (the compiler would otherwise move the first load into the branch of its store)
        v[u][0] = x;
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0) only
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const uint32_t t = t0 + (uint32_t)u * THREADS;
        if (s[u] == -2) v[u] = vec_t(0.f);
        if (t < total) __builtin_nontemporal_store(v[u], reinterpret_cast<vec_t*>(out) + t);
    }
}

// slots of ids: -1: not cached, -2: id out of range
template <int N>
__device__ __forceinline__ void look_up(const int32_t (&id)[N], int32_t (&s)[N], int64_t num_ids, const int32_t* __restrict__ slot_of, int n = N) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (u >= n) break;
        const bool in_range = id[u] >= 0 && id[u] < num_ids;
        s[u] = slot_of[in_range ? id[u] : 0];
        if (!in_range) s[u] = -2;
    }
}

// A workgroup's pieces are consecutive, so that a row is read and written by one compute unit, or two.  In k_gather its rows are
// looked up once each and handed over in LDS.  us per fetch with pieces a grid width apart / consecutive / consecutive and
// handed over: 2^20 rows of 172 floats, LFU 371 / 369 / 363, of 128 224 / 218 / 217, of 32 149 / 145 / 146, of 173 (pieces of 4 bytes) 324 /
// 309 / 295.  In k_update, whose workgroups are four times as large, handing over costs more than it gives: 66600 rows of 172 27.6 /
// 27.9 / 28.2, of 173 29.8 / 29.9 / 31.6, 300000 of 172 95.4 / 94.3 / 96.8.  There a workgroup takes `chunk` pieces, as many as the others: with
// 8192 for every one but the last, two workgroups shared 10^4 rows of one float as four to one (LFU 18.8 -> 21.0 us, FIFO 19.7 -> 23.4).
template <int VEC, int THREADS, int UNROLL>
__device__ __forceinline__ void gather_each(const float* __restrict__ rows, const float* __restrict__ store, int32_t dim,
                                            uint32_t total, const RowOf row, int64_t num_ids, const int32_t* __restrict__ ids,
                                            const int32_t* __restrict__ slot_of, float* __restrict__ out, uint32_t bid, uint32_t chunk) {
    const uint32_t t0 = bid * chunk + threadIdx.x;
    total = min(total, (bid + 1) * chunk);
    uint32_t col[UNROLL];
    int32_t id[UNROLL], s[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const uint32_t t = min(t0 + (uint32_t)u * THREADS, total - 1);      // clamped: no load sits in a branch
        const uint32_t b = row(t);
        col[u] = (t - b * row.per_row) * VEC;
        id[u] = ids[b];
    }
    look_up(id, s, num_ids, slot_of);
    move_pieces<VEC, THREADS, UNROLL>(rows, store, dim, total, t0, col, id, s, out);
}
template <int VEC, int THREADS, int UNROLL>
__device__ __forceinline__ void gather_rows(const float* __restrict__ rows, const float* __restrict__ store, int32_t dim,
                                            uint32_t total, const RowOf row, int64_t num_ids, const int32_t* __restrict__ ids,
                                            const int32_t* __restrict__ slot_of, float* __restrict__ out, uint32_t bid) {
    constexpr uint32_t kPieces = THREADS * UNROLL;
    __shared__ int32_t s_from[kPieces];         // the slot of a row, -1 - id if it is not cached, INT_MIN if the id is out of range
    const uint32_t first = bid * kPieces, t0 = first + threadIdx.x;
    const uint32_t r0 = row(first), n = row(min(first + kPieces, total) - 1) - r0 + 1;     // rows of the workgroup, at most kPieces
    const int rounds = (int)((n + THREADS - 1) / THREADS);
    uint32_t col[UNROLL];
    int32_t id[UNROLL], s[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        if (u >= rounds) break;                                 // uniform
        id[u] = ids[r0 + min((uint32_t)u * THREADS + threadIdx.x, n - 1)];
    }
    look_up(id, s, num_ids, slot_of, rounds);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const uint32_t i = (uint32_t)u * THREADS + threadIdx.x;
        if (i < n) s_from[i] = s[u] >= 0 ? s[u] : (s[u] == -1 ? -1 - id[u] : INT_MIN);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
        const uint32_t t = min(t0 + (uint32_t)u * THREADS, total - 1), b = row(t);
        col[u] = (t - b * row.per_row) * VEC;
        const int32_t from = s_from[b - r0];
        id[u] = -1 - from;
        s[u] = from >= 0 ? from : (from == INT_MIN ? -2 : -1);
    }
    move_pieces<VEC, THREADS, UNROLL>(rows, store, dim, total, t0, col, id, s, out);
}

template <int VEC>
__global__ void __launch_bounds__(256) k_gather(const float* __restrict__ rows, const float* __restrict__ store, int32_t dim,
                                                uint32_t total, const RowOf row, int64_t num_ids, const int32_t* __restrict__ ids,
                                                const int32_t* __restrict__ slot_of, float* __restrict__ out) {
    gather_rows<VEC, 256, kGatherUnroll>(rows, store, dim, total, row, num_ids, ids, slot_of, out, blockIdx.x);
}

// ---- compaction of flagged elements in three launches -------------------------------------------
// A flag functor gives each element a packed 64-bit count (one or two counters); (1) per-tile sums,
// (2) exclusive scan of the tile sums by one workgroup, (3) per tile: the flags again, a local scan,
// and the functor's emit() with the number of flagged elements before each one.  No flag array.

constexpr int kPerThread = kScanTile / 256;

template <class F>
__global__ void __launch_bounds__(256) k_flag_tile_sums(const F f, int64_t n, int64_t* __restrict__ sums) {
    __shared__ int64_t s_w[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPerThread;
    int64_t v = 0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
        if (base + i < n) v += f.count(base + i);
    const int lane = threadIdx.x & 63;
    v = tns::wave_inclusive_scan64(v);
    if (lane == 63) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// one workgroup: exclusive scan of the tile sums in place; the functor receives the total
template <class F>
__global__ void __launch_bounds__(1024) k_flag_scan_sums(const F f, int64_t* __restrict__ sums, int64_t num_tiles) {
    __shared__ int64_t s_w[16];
    __shared__ int64_t s_carry;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < num_tiles; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int64_t v = i < num_tiles ? sums[i] : 0;
        const int64_t inc = tns::wave_inclusive_scan64(v);
        if (lane == 63) s_w[wave] = inc;
        __syncthreads();
        int64_t wave_off = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int64_t t = s_w[w];
            if (w < wave) wave_off += t;
            all += t;
        }
        const int64_t carry = s_carry;
        if (i < num_tiles) sums[i] = carry + wave_off + (inc - v);
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + all;
        __syncthreads();
    }
    if (threadIdx.x == 0) f.total(s_carry);
}

// FOLD: `sums` holds the raw tile sums and every workgroup adds up those of the tiles before it by itself (at most
// kFoldTiles of them, read from the L2); the last one also hands the total to the functor.  This saves the
// one-workgroup scan kernel between the two, which is slow beside a kernel that saturates the memory system.
constexpr int64_t kFoldTiles = 2048;
template <class F, bool FOLD>
__device__ __forceinline__ void flag_collect_body(const F& f, int64_t n, const int64_t* __restrict__ sums, int64_t bid, int64_t nblocks) {
    __shared__ int64_t s_w[4], s_t[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t base = bid * kScanTile + (int64_t)threadIdx.x * kPerThread;
    int64_t tile_off = 0;
    if (FOLD) {
        int64_t part = 0;
        for (int64_t t0 = 0; t0 < bid; t0 += 256 * 4) {
            int64_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t t = t0 + u * 256 + threadIdx.x;
                v[u] = sums[min(t, bid)];          // clamped: no load sits in a branch
                if (t >= bid) v[u] = 0;
            }
            part += v[0] + v[1] + v[2] + v[3];
        }
        part = tns::wave_inclusive_scan64(part);
        if (lane == 63) s_t[wave] = part;
    }
    int64_t c[kPerThread], sum = 0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        c[i] = base + i < n ? f.count(base + i) : 0;
        sum += c[i];
    }
    const int64_t inc = tns::wave_inclusive_scan64(sum);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    if (FOLD) tile_off = s_t[0] + s_t[1] + s_t[2] + s_t[3];
    else tile_off = sums[bid];
    int64_t before = tile_off + inc - sum;
    for (int w = 0; w < wave; ++w) before += s_w[w];
    if (FOLD && bid == nblocks - 1 && threadIdx.x == 0) f.total(tile_off + s_w[0] + s_w[1] + s_w[2] + s_w[3]);
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        if (c[i]) f.emit(base + i, before);
        before += c[i];
    }
}

template <class F, bool FOLD>
__global__ void __launch_bounds__(256) k_flag_collect(const F f, int64_t n, const int64_t* __restrict__ sums) {
    flag_collect_body<F, FOLD>(f, n, sums, blockIdx.x, gridDim.x);
}

// Distinct missed ids in the order of their first occurrence (the flag: a missed row that is the first
// of its id), up to max_replace of them; the total fixes how many entries this update replaces.
struct NewIds {
    const int32_t* first_idx;
    const int32_t* ids;
    const int32_t* slots;
    int32_t max_replace;
    int32_t* new_ids;
    Ctl* ctl;
    __device__ int64_t count(int64_t b) const { return slots[b] == -1 && first_idx[ids[b]] == (int32_t)b ? 1 : 0; }
    __device__ void emit(int64_t b, int64_t before) const {
        if (before < max_replace) new_ids[before] = ids[b];
    }
    __device__ void total(int64_t n_unique) const {
        const int32_t m = (int32_t)(n_unique < max_replace ? n_unique : max_replace);
        ctl->n_unique = (int32_t)n_unique;
        ctl->m = m;
        ctl->remaining = m;
    }
};


// ---- victims: the m entries with the lowest (score, slot) --------------------------------------

// unsigned order = signed order of the scores
__device__ __forceinline__ uint32_t score_key(int32_t stored, int32_t now) { return ((uint32_t)stored - (uint32_t)now) ^ 0x80000000u; }

// Radix select of the m-th smallest key.  A pass is one launch that histograms the digit over the entries whose
// decided high bits match; the digit in which the remaining-th smallest key falls is picked by the NEXT kernel, by
// every workgroup for itself in its prologue (a scan over the bins), so a pass needs no launch of its own for the
// pick.  Workgroup 0 also stores the state for whoever reads it later.  Called by all 256 threads of a workgroup;
// returns the state after `pass` passes.
struct SelState { uint32_t prefix, mask; int32_t rem; };
__device__ __forceinline__ SelState select_pick(Ctl* ctl, int pass /* 1..kPasses */, bool store) {
    __shared__ int32_t s_w[4];
    __shared__ SelState s_out;
    SelState prev;
    if (pass == 1) { prev.prefix = 0; prev.mask = 0; prev.rem = ctl->m; }
    else { prev.prefix = ctl->sel_prefix[pass - 1]; prev.mask = ctl->sel_mask[pass - 1]; prev.rem = ctl->sel_rem[pass - 1]; }
    const int shift = digit_shift(pass - 1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t h[kBinsPerThread], mine = 0;          // this thread's consecutive bins
#pragma unroll
    for (int i = 0; i < kBinsPerThread; i += 4) {
        const int4 v = *reinterpret_cast<const int4*>(&ctl->hist[pass - 1][threadIdx.x * kBinsPerThread + i]);
        h[i] = v.x; h[i + 1] = v.y; h[i + 2] = v.z; h[i + 3] = v.w;
    }
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) mine += h[i];
    int32_t inc = tns::wave_inclusive_scan(mine);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    for (int w = 0; w < wave; ++w) inc += s_w[w];
    // the first bin whose inclusive count reaches rem; the last bin if none does
    int32_t before = inc - mine;
    if ((inc >= prev.rem && before < prev.rem) || (threadIdx.x == 255 && inc < prev.rem)) {
        int bin = 0;
#pragma unroll
        for (int i = 0; i < kBinsPerThread - 1; ++i)
            if (bin == i && before + h[i] < prev.rem) {
                before += h[i];
                bin = i + 1;
            }
        s_out.prefix = prev.prefix | ((uint32_t)(threadIdx.x * kBinsPerThread + bin) << shift);
        s_out.mask = prev.mask | (digit_mask(pass - 1) << shift);
        s_out.rem = prev.rem - before;             // entries to take among keys equal to the threshold so far
    }
    __syncthreads();
    const SelState out = s_out;
    if (store && threadIdx.x == 0) {
        ctl->sel_prefix[pass] = out.prefix; ctl->sel_mask[pass] = out.mask; ctl->sel_rem[pass] = out.rem;
        if (pass == kPasses) { ctl->prefix = out.prefix; ctl->mask = out.mask; ctl->remaining = out.rem; }
    }
    __syncthreads();
    return out;
}

// Histogram of pass `pass` (0-based); pass 0 does not know yet whether anything will be replaced and histograms
// regardless.  `bid` / `nb`: this workgroup's index and the number of workgroups that share the pass (the kernel may hold
// other work in its other workgroups).
__device__ __forceinline__ void select_hist_body(const int32_t* __restrict__ score, int64_t capacity, int pass, Ctl* ctl, int64_t bid, int64_t nb) {
    __shared__ int32_t s_h[kBins];
    uint32_t prefix = 0, mask = 0;
    const int32_t now = ctl->now;              // (read here, beside what the pick reads)
    if (pass > 0) {
        if (ctl->m <= 0) return;
        const SelState st = select_pick(ctl, pass, bid == 0);
        prefix = st.prefix;
        mask = st.mask;
    }
    const int shift = digit_shift(pass);
    const uint32_t dmask = digit_mask(pass);
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) s_h[i * 256 + threadIdx.x] = 0;
    __syncthreads();
    for (int64_t s0 = bid * 256; s0 < capacity; s0 += nb * 256) {       // uniform over the workgroup
        const int64_t s = s0 + threadIdx.x;
        bool take = false;
        uint32_t d = 0;
        if (s < capacity) {
            const uint32_t k = score_key(score[s], now);
            take = (k & mask) == prefix;
            d = (k >> shift) & dmask;
        }
        // scores lie close together: mostly a wave's entries share the digit, and one addition serves them all
        const uint64_t active = __ballot(take);
        if (active) {
            const uint32_t d0 = (uint32_t)__shfl((int)d, __builtin_ctzll(active), kWave);
            if (__ballot(take && d == d0) == active) {
                if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&s_h[d0], __popcll(active));
            } else if (take) {
                atomicAdd(&s_h[d], 1);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) {
        const int32_t c = s_h[i * 256 + threadIdx.x];
        if (c) atomicAdd(&ctl->hist[pass][i * 256 + threadIdx.x], c);
    }
}

__global__ void __launch_bounds__(256) k_select_hist(const int32_t* __restrict__ score, int64_t capacity, int pass, Ctl* ctl) {
    select_hist_body(score, capacity, pass, ctl, blockIdx.x, gridDim.x);
}

// The victims in ascending slot order: every entry below the threshold key and the first `remaining`
// entries equal to it.  Packed count: entries below in the high word, equal entries in the low word.
struct Victims {
    const int32_t* score;
    const Ctl* ctl;
    int32_t* victims;
    __device__ int64_t count_with(int64_t s, uint32_t t) const {
        const uint32_t k = score_key(score[s], ctl->now);
        return k < t ? (int64_t(1) << 32) : (k == t ? 1 : 0);
    }
    __device__ int64_t count(int64_t s) const { return ctl->m <= 0 ? 0 : count_with(s, ctl->prefix); }
    __device__ void emit(int64_t s, int64_t before) const {
        const int64_t below_before = before >> 32, eq_before = before & 0xffffffffll, rem = ctl->remaining;
        const bool below = score_key(score[s], ctl->now) < ctl->prefix;
        if (below || eq_before < rem) victims[below_before + (eq_before < rem ? eq_before : rem)] = (int32_t)s;
    }
    __device__ void total(int64_t) const {}
};

// Tile sums of the victims' compaction; the prologue picks the last digit of the radix select (the threshold is
// final from here on: workgroup 0 stores it for the collect kernel).
__global__ void __launch_bounds__(256) k_victims_tile_sums(const Victims f, Ctl* ctl, int64_t n, int64_t* __restrict__ sums) {
    __shared__ int64_t s_w[4];
    int64_t v = 0;
    if (ctl->m > 0) {
        const SelState st = select_pick(ctl, kPasses, blockIdx.x == 0);
        const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPerThread;
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            if (base + i < n) v += f.count_with(base + i, st.prefix);
    }
    const int lane = threadIdx.x & 63;
    v = tns::wave_inclusive_scan64(v);
    if (lane == 63) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}


// Two independent pieces of the update in one launch (the chain of short launches is what the update costs):
// workgroups [0, tiles) collect the distinct missed ids (which also fixes m), the other `hb` workgroups run pass 0
// of the radix select over the scores, which depends on the lookup only.
__global__ void __launch_bounds__(256) k_newids_collect_hist0(const NewIds f, int64_t n, const int64_t* __restrict__ sums, int64_t tiles,
                                                              const int32_t* __restrict__ score, int64_t capacity, Ctl* ctl, int64_t hb) {
    if ((int64_t)blockIdx.x < tiles) flag_collect_body<NewIds, true>(f, n, sums, blockIdx.x, tiles);
    else select_hist_body(score, capacity, 0, ctl, (int64_t)blockIdx.x - tiles, hb);
}

// ---- the update in one launch: FIFO, and caches of up to kOneGroupEntries entries ------------------
//
// What bounds the fetch of a batch of some ten thousand rows is the number of launches that wait for one another: tile sums
// of the missed ids, their collection, three histogram passes, tile sums of the victims, their collection, and two
// events around them.  Here one launch holds all of it, beside the gather.  A workgroup per 1024 ids of the batch counts its
// first occurrences of missed ids and learns from a chained scan over the workgroups what comes before it; the one with
// the last tile then knows the number of entries to replace and selects the victims by itself, every score in a
// register of one of its 1024 threads.  The scores are requested before its ids and arrive meanwhile.
// The threshold, the m-th lowest score, is found by counting the scores below a bound (1.3 us each for 42 K entries):
// the bound rises from the lowest score in steps that grow fourfold and is then bisected.  Victims are the oldest or
// rarest entries and lie within a few values of the lowest, so that one to six counts are usual; any 32-bit scores take at most
// 16 and 32.  (A histogram in LDS has all its lanes adding to a handful of words.)  One workgroup issues about an
// instruction per SIMD every four cycles, so 44 scores per thread make the instructions per score what counts: the victims are
// stored in 2.5 us where the equal ones are all taken or all left, by one comparison; with both compared for
// every score and counted in a pass of their own they took 9.  Time stamps, batch of 66600 of which 8388 are replaced: new ids
// known at 8 us, threshold at 15, victims stored at 18; since then the lowest score is found, and under LRU the eight lowest
// values are counted (kNear), before the tile waits for the others.
// 42 K entries, rows of 172 floats, us per fetch, LRU / LFU / FIFO, one cache again and again: 66600 ids 71 / 74 / 61 -> 31 / 35 / 28, 16000 ids 67 / 67 / 60
// -> 21 / 18 / 17, 600 ids 69 / 67 / 60 -> 16 / 16 / 16, which is what a call from Python takes.  Three caches in turn, so that their rows come from
// memory: 66600 ids 83 / 84 / 65 -> 34 / 38 / 33.
constexpr int kOneGroup = 1024, kOneGroupWaves = kOneGroup / kWave;
constexpr int kItems = 64, kItemStep = 8;                         // scores per thread, and per uniform branch
// LRU: values from the lowest on that are counted at once while new ids are awaited, if these come from enough tiles for the wait to be
// long.  us per fetch without / with: 52 K entries, 34000 ids of 100 floats 32.1 / 30.5, 50000 34.1 / 32.9; 42 K, 66600 of 172 32.7 / 31.2; 10 K, 150000
// of 32 26.1 / 24.6.  In all batches: 52 K entries, 600 ids 15.0 / 17.5, 10000 16.1 / 19.8.  Under LFU, where the lowest value alone
// often has enough entries, 34000 ids 25.6 / 28.4.
constexpr int kNear = 8, kNearTiles = 32;
// Where the line lies: a large gather saturates the memory, and the chain of dependent reads of the tiles beside it then
// takes longer than the short launches do on a stream of their own.  It was drawn where the two forms met at pieces of 16 bytes, when a
// thread of this one moved eight; with four they meet further up.  42 K entries, us per fetch, LRU / LFU / FIFO, this form and the other:
// rows of 172 floats, 262144 (11 M pieces of 16 bytes) 81 / 106 / 81 and 114 / 127 / 95, 390000 (17 M) 114 / 151 / 116 and 141 / 166 / 124, 524288 (23 M)
// 149 / 198 / 149 and 169 / 206 / 153; 2^20 rows of 32 floats (8 M) 81 / 179 / 86 and 104 / 196 / 88, of 64 (17 M) 128 / 224 / 132 and 150 / 221 / 133; rows of
// 173 floats, 66600 (12 M pieces of 4 bytes) 33 / 37 / 29 and 74 / 76 / 59, 97000 (17 M) 41 / 48 / 37 and 74 / 76 / 61, 180000 (31 M) 72 / 85 / 63 and 92 / 98 /
// 74, 262144 (45 M) 103 / 123 / 89 and 105 / 121 / 88.
constexpr int64_t kGatherWithin = int64_t(1) << 24, kOneLaunchIds = int64_t(1) << 20;
constexpr uint32_t kNoWait = 1u << 31;                            // bit of the tickets of tiles that do not wait for one another (tests)
constexpr int64_t kOneGroupEntries = (int64_t)kOneGroup * kItems;

// set bits of `mask` below this lane
__device__ __forceinline__ int32_t lanes_before(uint64_t mask) {
    return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ int32_t fifo_slot(int64_t ring, int64_t i, int64_t capacity) {
    const int64_t s = ring + i;                // ring < capacity, i < capacity
    return (int32_t)(s >= capacity ? s - capacity : s);
}

// Number of keys below `bound` in the workgroup, and in this wave.  `s_cnt`: two rows, used in turn, so that one barrier serves.
__device__ __forceinline__ int32_t count_below(const uint32_t (&key)[kItems], int items, uint32_t bound, int32_t (*s_cnt)[kOneGroupWaves],
                                               int round, int32_t& of_wave) {
    int32_t n = 0;
#pragma unroll
    for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
        if (i0 < items) {                       // uniform
            uint64_t below[kItemStep];
#pragma unroll
            for (int u = 0; u < kItemStep; ++u) below[u] = __ballot(key[i0 + u] < bound);
            __builtin_amdgcn_sched_barrier(0);   // the comparisons back to back, none waits for the count of the one before
#pragma unroll
            for (int u = 0; u < kItemStep; ++u) n += __popcll(below[u]);
        }
    }
    of_wave = n;
    int32_t* const row = s_cnt[round & 1];
    if ((threadIdx.x & (kWave - 1)) == 0) row[threadIdx.x / kWave] = n;
    __syncthreads();
    n = 0;
#pragma unroll
    for (int w = 0; w < kOneGroupWaves; ++w) n += row[w];
    return __builtin_amdgcn_readfirstlane(n);
}

// Distinct missed ids of tile `tile` in the order of their first occurrence, behind those of the tiles before it.
// Returns their number up to and including this tile.  What a tile learns from the chained scan it could count by itself, and
// does so if the tiles before it have not reported within the bound of its wait (or `wait` is false, in tests): every update
// is made, however late a tile is.
// meanwhile(): what the workgroup does before it waits.
template <class Meanwhile>
__device__ __forceinline__ int64_t new_ids_of_tile(const NewIds& f, int64_t B, tns::ScanWorkspace* chain, int64_t tile, bool wait,
                                                   const Meanwhile& meanwhile) {
    __shared__ int32_t s_w[kOneGroupWaves];
    __shared__ int64_t s_excl;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t b = tile * kOneGroup + threadIdx.x;
    const uint64_t first = __ballot(b < B && f.count(b));
    if (lane == 0) s_w[wave] = __popcll(first);
    __syncthreads();
    int32_t total = 0, before = 0;
#pragma unroll
    for (int w = 0; w < kOneGroupWaves; ++w) {
        const int32_t n = s_w[w];
        before += w < wave ? n : 0;
        total += n;
    }
    auto publish = [&](int64_t before_tile) {
        __hip_atomic_store(&chain->status[tile], tns::kStPrefix | (uint64_t)(before_tile + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (threadIdx.x == 0 && tile > 0)
        __hip_atomic_store(&chain->status[tile], tns::kStTotal | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    meanwhile();
    if (wave == 0) {
        int64_t excl = 0;
        if (tile > 0 && !(wait && tns::lookback(chain, tile, lane, excl, [](int64_t v) { return tns::wave_sum64(v); }))) excl = -1;
        if (lane == 0) {
            s_excl = excl;
            if (excl >= 0) publish(excl);
        }
    }
    __syncthreads();
    int64_t excl = s_excl;
    if (excl < 0) {                            // uniform
        int32_t n = 0;
        for (int64_t i = threadIdx.x; i < tile * kOneGroup; i += kOneGroup) n += (int32_t)f.count(i);
        for (int d = kWave / 2; d >= 1; d >>= 1) n += __shfl_xor(n, d, kWave);
        if (lane == 0) s_w[wave] = n;
        __syncthreads();
        excl = 0;
        for (int w = 0; w < kOneGroupWaves; ++w) excl += s_w[w];
        if (threadIdx.x == 0) publish(excl);
    }
    if ((first >> lane) & 1) f.emit(b, excl + before + lanes_before(first));
    return excl + total;
}

// Entries to replace, once the last tile knows the number of distinct missed ids.
__device__ __forceinline__ int32_t entries_to_replace(const NewIds& f, int64_t n_unique) {
    __shared__ int32_t s_m;
    if (threadIdx.x == 0) {
        f.total(n_unique);
        s_m = f.ctl->m;
    }
    __syncthreads();
    return s_m;
}

__device__ __forceinline__ void last_tile(const CacheState& c, const NewIds& f, int64_t B, tns::ScanWorkspace* chain, int64_t tile,
                                          int32_t* __restrict__ victims, bool wait) {
    __shared__ int32_t s_cnt[2][kOneGroupWaves];
    __shared__ uint32_t s_min[kOneGroupWaves];
    __shared__ int32_t s_near[kNear][kOneGroupWaves];
    __shared__ int32_t s_below[kOneGroupWaves], s_equal[kOneGroupWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // a wave holds `items` times 64 consecutive scores: the lanes of a ballot are in slot order
    const int32_t C = (int32_t)c.capacity;
    const int items = (C + kOneGroup * kItemStep - 1) / (kOneGroup * kItemStep) * kItemStep;
    const int32_t base = wave * items * kWave + lane;
    uint32_t key[kItems];                      // beyond the last entry: the highest, below no bound
#pragma unroll
    for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
        if (i0 >= items) continue;             // uniform
#pragma unroll
        for (int i = i0; i < i0 + kItemStep; ++i) key[i] = (uint32_t)c.score[min(base + i * kWave, C - 1)];
    }
    const int32_t now = f.ctl->now;
#pragma unroll
    for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
        if (i0 >= items) continue;
#pragma unroll
        for (int i = i0; i < i0 + kItemStep; ++i) key[i] = base + i * kWave < C ? score_key((int32_t)key[i], now) : ~0u;
    }
    uint32_t lowest = ~0u;
    const bool near = tile >= kNearTiles && now != 0;
    int32_t near_all[kNear] = {}, near_own[kNear] = {};      // keys below lowest + 1 + j: all of them, this wave's
    auto count_near = [&]() {
#pragma unroll
        for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
            if (i0 >= items) continue;
#pragma unroll
            for (int i = i0; i < i0 + kItemStep; ++i) lowest = min(lowest, key[i]);
        }
        for (int d = kWave / 2; d >= 1; d >>= 1) lowest = min(lowest, (uint32_t)__shfl_xor((int)lowest, d, kWave));
        if (lane == 0) s_min[wave] = lowest;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kOneGroupWaves; ++w) lowest = min(lowest, s_min[w]);
        lowest = (uint32_t)__builtin_amdgcn_readfirstlane((int)lowest);
        if (!near) return;
        // a byte per value and thread (at most kItems), then sixteen bits per wave
        uint32_t low = 0, high = 0;
#pragma unroll
        for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
            if (i0 >= items) continue;
#pragma unroll
            for (int i = i0; i < i0 + kItemStep; ++i) {
                const uint32_t d = key[i] - lowest, one = 1u << ((8 * d) & 31u);
                low += d < 4 ? one : 0u;
                high += d - 4 < 4 ? one : 0u;
            }
        }
        const uint32_t even = 0x00ff00ffu;
        const uint32_t pair[4] = {(uint32_t)tns::wave_sum((int)(low & even)), (uint32_t)tns::wave_sum((int)((low >> 8) & even)),
                                  (uint32_t)tns::wave_sum((int)(high & even)), (uint32_t)tns::wave_sum((int)((high >> 8) & even))};
        int32_t n = 0;
#pragma unroll
        for (int j = 0; j < kNear; ++j) {
            n += (int32_t)((pair[j / 4 * 2 + (j & 1)] >> (j & 2 ? 16 : 0)) & 0xffffu);
            near_own[j] = n;
            if (lane == 0) s_near[j][wave] = n;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kNear; ++j) near_all[j] = tns::sum_of_waves(s_near[j], kOneGroupWaves, lane);
    };
    const int64_t n_unique = new_ids_of_tile(f, B, chain, tile, wait, count_near);
    const int32_t m = __builtin_amdgcn_readfirstlane(entries_to_replace(f, n_unique));
    if (m <= 0) return;
    // the m-th lowest key is in [lo, hi); below lo lie below_lo keys, of_lo of them this wave's, and of_hi of this wave's below hi
    uint64_t lo = lowest, hi = 1ull << 32, step = 1;
    int32_t below_lo = 0, of_lo = 0, of_hi = max(min(C - wave * items * kWave, items * kWave), 0);
    if (near && lowest < ~0u - kNear) {      // (no place beyond the last entry was counted)
#pragma unroll
        for (int j = 0; j < kNear; ++j) {
            if (hi != 1ull << 32) continue;
            if (near_all[j] >= m) { hi = (uint64_t)lowest + 1 + j; of_hi = near_own[j]; }
            else { lo = (uint64_t)lowest + 1 + j; below_lo = near_all[j]; of_lo = near_own[j]; }
        }
        step = 2 * kNear;
    }
    int round = 0;
    while (hi - lo > 1) {
        const bool rising = hi == 1ull << 32 && lo + step < hi;      // (at most sixteen times, then never again)
        const uint64_t at = rising ? lo + step : lo + ((hi - lo) >> 1);
        int32_t of_wave;
        const int32_t n = count_below(key, items, (uint32_t)at, s_cnt, round++, of_wave);
        if (n >= m) { hi = at; of_hi = of_wave; }
        else { lo = at; below_lo = n; of_lo = of_wave; step *= rising ? 4 : 1; }
    }
    const uint32_t threshold = (uint32_t)lo;
    const int32_t rem = m - below_lo;          // to take among keys equal to the threshold, lowest slots first
    if (lane == 0) { s_below[wave] = of_lo; s_equal[wave] = of_hi - of_lo; }
    __syncthreads();
    int32_t below_before = 0, equal_before = 0;
    for (int w = 0; w < wave; ++w) { below_before += s_below[w]; equal_before += s_equal[w]; }
    // victims in slot order: every key below the threshold and the first `rem` equal to it, of which `quota` fall to this wave
    const int32_t quota = __builtin_amdgcn_readfirstlane(min(max(rem - equal_before, 0), of_hi - of_lo));
    int32_t at = __builtin_amdgcn_readfirstlane(below_before + min(equal_before, rem));
    if ((quota == 0 || quota == of_hi - of_lo) && threshold != ~0u) {
        // none or all of its equal ones, as in every wave but one: a single bound
        const uint32_t bound = quota ? threshold + 1u : threshold;
#pragma unroll
        for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
            if (i0 >= items) continue;
#pragma unroll
            for (int i = i0; i < i0 + kItemStep; ++i) {
                const bool take = key[i] < bound;
                const uint64_t mask = __ballot(take);
                if (take) victims[(uint32_t)(at + lanes_before(mask))] = base + i * kWave;
                at += __popcll(mask);
            }
        }
    } else {
        int32_t left = quota;
#pragma unroll
        for (int i0 = 0; i0 < kItems; i0 += kItemStep) {
            if (i0 >= items) continue;
#pragma unroll
            for (int i = i0; i < i0 + kItemStep; ++i) {
                const int32_t s = base + i * kWave;
                const bool equal = key[i] == threshold && s < C;
                const uint64_t equals = __ballot(equal);
                const bool take = key[i] < threshold || (equal && lanes_before(equals) < left);
                const uint64_t mask = __ballot(take);
                if (take) victims[(uint32_t)(at + lanes_before(mask))] = s;
                at += __popcll(mask);
                left = max(left - (int32_t)__popcll(equals), 0);
            }
        }
    }
}

// FIFO: the entries this update replaces start at ctl->ring
__device__ __forceinline__ void fifo_advance(int64_t capacity, int64_t* ring, Ctl* ctl, int32_t m) {
    const int64_t r = *ring;
    ctl->ring = r;
    *ring = (r + m) % capacity;
}
__global__ void k_fifo_advance(int64_t capacity, int64_t* ring, Ctl* ctl) { fifo_advance(capacity, ring, ctl, ctl->m); }

// GATHER: floats per piece of the gathered rows
template <bool SELECT, int GATHER>
__global__ void __launch_bounds__(kOneGroup) k_update(const CacheState c, const NewIds f, int64_t B, int64_t tiles, tns::ScanWorkspace* chain,
                                                      int32_t* __restrict__ victims, const float* __restrict__ store, int32_t dim,
                                                      uint32_t pieces, uint32_t chunk, const RowOf row, int64_t num_ids, float* __restrict__ out) {
    __shared__ uint32_t s_ticket;
    if ((int64_t)blockIdx.x >= tiles) {
        gather_each<GATHER, kOneGroup, update_unroll(GATHER)>(c.rows, store, dim, pieces, row, num_ids, f.ids, c.slot_of, out,
                                                              blockIdx.x - (uint32_t)tiles, chunk);
        return;
    }
    // tiles are numbered in the order workgroups start, so that a tile only waits for tiles that have started
    if (threadIdx.x == 0) s_ticket = atomicAdd(&chain->ticket, 1u);
    __syncthreads();
    const int64_t tile = s_ticket & ~kNoWait;
    const bool wait = !(s_ticket & kNoWait);
    if (SELECT && tile == tiles - 1) {
        last_tile(c, f, B, chain, tile, victims, wait);
        return;
    }
    const int64_t n_unique = new_ids_of_tile(f, B, chain, tile, wait, []() {});
    if (!SELECT && tile == tiles - 1) {
        const int32_t m = entries_to_replace(f, n_unique);
        if (threadIdx.x == 0) fifo_advance(c.capacity, c.ring, f.ctl, m);
    }
}

// One wave per replaced entry: maps, score, row copy from the backing store.  What bounds it is the chain of dependent reads,
// so the entry's slot and id are requested beside the number of entries, and its row, in pieces of VEC floats, before anything
// is stored (a load behind stores is only waited for together with them).  Fetch of 66600 rows of 172 floats 33.1 -> 31.9 us.
template <int VEC>
__device__ __forceinline__ void insert_body(const CacheState& c, int policy, int32_t dim, const float* __restrict__ store,
                                            const int32_t* __restrict__ new_ids, const int32_t* __restrict__ victims, const Ctl* ctl,
                                            int64_t bid, int32_t max_replace) {
    typedef float vec_t __attribute__((ext_vector_type(VEC)));
    constexpr int kAhead = 16 / VEC;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t i = bid * 4 + (threadIdx.x >> 6), at = min(i, (int64_t)max_replace - 1);
    const int32_t m = ctl->m, now = ctl->now, id = new_ids[at];
    const int32_t s = policy == TNS_CACHE_FIFO ? fifo_slot(ctl->ring, at, c.capacity) : victims[at];
    if (i >= m) return;
    const int32_t pieces = dim / VEC;
    const vec_t* __restrict__ src = reinterpret_cast<const vec_t*>(store + (int64_t)id * dim);
    vec_t* __restrict__ dst = reinterpret_cast<vec_t*>(c.rows + (int64_t)s * dim);
    const int32_t old = c.id_of[s];
    for (int32_t k0 = 0; k0 < pieces; k0 += kAhead * kWave) {
        vec_t v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (k0 + u * kWave >= pieces) break;             // uniform
            v[u] = src[min(k0 + u * kWave + lane, pieces - 1)];
        }
        if (k0 == 0 && lane == 0) {
            if (old >= 0) c.slot_of[old] = -1;
            c.id_of[s] = id;
            c.slot_of[id] = s;
            c.score[s] = policy == TNS_CACHE_LFU ? 1 : now;
            if (i == 0) atomicAdd(&c.counters[2], (unsigned long long)m);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (k0 + u * kWave >= pieces) break;
            if (k0 + u * kWave + lane < pieces) dst[k0 + u * kWave + lane] = v[u];
        }
    }
}

// The insertion (workgroups [0, insert_blocks)) and the clearing of the batch's first-occurrence marks (the rest),
// which touch different arrays, in one launch at the end of the fetch.
template <int VEC>
__global__ void __launch_bounds__(256) k_insert_clear(CacheState c, int policy, int32_t dim, const float* __restrict__ store,
                                                      const int32_t* __restrict__ new_ids, const int32_t* __restrict__ victims,
                                                      const Ctl* ctl, int64_t insert_blocks, int32_t max_replace, int64_t B,
                                                      const int32_t* __restrict__ ids, const int32_t* __restrict__ slots) {
    if ((int64_t)blockIdx.x < insert_blocks) {
        insert_body<VEC>(c, policy, dim, store, new_ids, victims, ctl, blockIdx.x, max_replace);
    } else {
        const int64_t b = ((int64_t)blockIdx.x - insert_blocks) * 256 + threadIdx.x, at = min(b, B - 1);
        const int32_t slot = slots[at], id = ids[at];
        if (b == 0) *c.updates = ctl->now;
        if (b < B && slot == -1) c.first_idx[id] = kNoIndex;
    }
}

inline unsigned blocks_for(int64_t n, int per = 256) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// flagged elements of [0, n) through the functor (see above); sums = scratch for ceil(n/1024) + 1 int64
template <class F>
void compact_flagged(const F& f, int64_t n, int64_t* sums, hipStream_t stream) {
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    if (tiles > 0 && tiles <= kFoldTiles) {
        hipLaunchKernelGGL((k_flag_tile_sums<F>), dim3((unsigned)tiles), dim3(256), 0, stream, f, n, sums);
        hipLaunchKernelGGL((k_flag_collect<F, true>), dim3((unsigned)tiles), dim3(256), 0, stream, f, n, sums);
        return;
    }
    if (tiles > 0) hipLaunchKernelGGL((k_flag_tile_sums<F>), dim3((unsigned)tiles), dim3(256), 0, stream, f, n, sums);
    hipLaunchKernelGGL((k_flag_scan_sums<F>), dim3(1), dim3(1024), 0, stream, f, sums, tiles);
    if (tiles > 0) hipLaunchKernelGGL((k_flag_collect<F, false>), dim3((unsigned)tiles), dim3(256), 0, stream, f, n, sums);
}

}  // namespace

struct tns_cache {
    tns_cache_config cfg;
    CacheState st{};
    int32_t max_replace = 0;
    // the update (scores, victims) runs beside the row gather on a stream of the cache's own,
    // forked from and joined back into the caller's stream with these events
    hipStream_t side = nullptr;
    hipEvent_t forked = nullptr, joined = nullptr;
    uint32_t first_ticket = 0;       // of the tiles of an update
};

namespace {
struct Workspace {
    Ctl* ctl;
    int32_t *slots, *new_ids, *victims;
    int64_t* sums;
    tns::ScanWorkspace* chain;
    size_t bytes;
};
Workspace carve(const tns_cache* c, int64_t B, void* base) {
    Workspace w{};
    unsigned char* p = static_cast<unsigned char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) { unsigned char* r = p ? p + off : nullptr; off += align256(bytes); return r; };
    const int64_t cap = c->cfg.capacity;
    w.ctl = reinterpret_cast<Ctl*>(take(sizeof(Ctl)));
    w.slots = reinterpret_cast<int32_t*>(take((size_t)B * 4));
    w.new_ids = reinterpret_cast<int32_t*>(take((size_t)std::max(c->max_replace, 1) * 4));
    w.victims = reinterpret_cast<int32_t*>(take((size_t)std::max(c->max_replace, 1) * 4));
    w.sums = reinterpret_cast<int64_t*>(take((size_t)(std::max(B, cap) / kScanTile + 2) * 8));
    w.chain = reinterpret_cast<tns::ScanWorkspace*>(take(sizeof(tns::ScanWorkspace) + (size_t)(B / kScanTile + 1) * 8));
    w.bytes = off;
    return w;
}
}  // namespace

extern "C" {

int tns_cache_create(const tns_cache_config* cfg, tns_cache** out) {
    tns::clear_error();
    if (!cfg || !out) return fail(TNS_EINVAL, "null config or output pointer");
    if (cfg->num_ids < 1 || cfg->num_ids > (int64_t)INT32_MAX) return fail(TNS_EINVAL, "num_ids must be in [1, 2^31-1]");
    if (cfg->capacity < 1 || cfg->capacity > (int64_t)INT32_MAX / 2) return fail(TNS_EINVAL, "capacity must be in [1, 2^30]");
    if (cfg->dim < 1 || cfg->dim > (1 << 20)) return fail(TNS_EINVAL, "dim must be in [1, 2^20]");
    if (cfg->policy < 0 || cfg->policy > 2) return fail(TNS_EINVAL, "unknown policy");
    if (!(cfg->lambda > 0.0f) || cfg->lambda > 1.0f) return fail(TNS_EINVAL, "lambda must be in (0, 1]");
    if (cfg->device < 0) return fail(TNS_EINVAL, "negative device ordinal");
    DeviceGuard guard(cfg->device);
    if (guard.error() != hipSuccess) return fail_hip(guard.error(), "selecting the cache's device");
    tns_cache* c = new (std::nothrow) tns_cache();
    if (!c) return fail(TNS_ENOMEM, "host allocation failed");
    c->cfg = *cfg;
    c->st.capacity = cfg->capacity;
    // (from 2^24 on a capacity may round up on its way to 32 bits; the victims are distinct entries)
    c->max_replace = (int32_t)std::min(std::floor((double)(cfg->lambda * (float)cfg->capacity)), (double)cfg->capacity);
    const int64_t N = cfg->num_ids, C = cfg->capacity;
    struct Alloc { void** p; size_t bytes; };
    const Alloc allocs[] = {{(void**)&c->st.slot_of, (size_t)N * 4}, {(void**)&c->st.first_idx, (size_t)N * 4},
                            {(void**)&c->st.id_of, (size_t)C * 4},   {(void**)&c->st.score, (size_t)C * 4},
                            {(void**)&c->st.updates, 4},             {(void**)&c->st.rows, (size_t)C * cfg->dim * 4},
                            {(void**)&c->st.counters, kStripes * 3 * 8},        {(void**)&c->st.ring, 8}};
    for (const Alloc& a : allocs) {
        const hipError_t e = tns::device_malloc(a.p, a.bytes);
        if (e != hipSuccess) {
            tns_cache_destroy(c);
            return fail_hip(e, "allocating the cache");
        }
    }
    hipError_t es = hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking);
    if (es == hipSuccess) es = hipEventCreateWithFlags(&c->forked, hipEventDisableTiming);
    if (es == hipSuccess) es = hipEventCreateWithFlags(&c->joined, hipEventDisableTiming);
    if (es != hipSuccess) {
        tns_cache_destroy(c);
        return fail_hip(es, "creating the cache's stream and events");
    }
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(N)), dim3(256), 0, nullptr, c->st.slot_of, N, -1);
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(N)), dim3(256), 0, nullptr, c->st.first_idx, N, kNoIndex);
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(C)), dim3(256), 0, nullptr, c->st.id_of, C, -1);
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(C)), dim3(256), 0, nullptr, c->st.score, C, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, nullptr, c->st.updates, 1, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(kStripes * 6)), dim3(256), 0, nullptr, reinterpret_cast<int32_t*>(c->st.counters), kStripes * 6, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, nullptr, reinterpret_cast<int32_t*>(c->st.ring), 2, 0);
    hipError_t e = hipMemsetAsync(c->st.rows, 0, (size_t)C * cfg->dim * 4, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) {
        tns_cache_destroy(c);
        return fail_hip(e, "initialising the cache");
    }
    *out = c;
    return TNS_OK;
}

int tns_cache_workspace(const tns_cache* cache, int64_t B, size_t* bytes) {
    tns::clear_error();
    if (!cache || !bytes || B < 0) return fail(TNS_EINVAL, "null cache/pointer or negative B");
    *bytes = carve(cache, B, nullptr).bytes;
    return TNS_OK;
}

int tns_cache_fetch(tns_cache* cache, int64_t B, const int32_t* d_ids, const float* store, float* d_out, uint8_t* d_hit,
                    void* d_workspace, size_t workspace_bytes, void* hip_stream) {
    tns::clear_error();
    if (!cache) return fail(TNS_EINVAL, "null cache");
    if (B < 0) return fail(TNS_EINVAL, "negative B");
    if (B == 0) return TNS_OK;
    if (B > (int64_t)INT32_MAX) return fail(TNS_ESIZE, "more than 2^31-1 ids in one batch");
    if (!d_ids || !store || !d_out) return fail(TNS_EINVAL, "null ids, store or output");
    if (!d_workspace) return fail(TNS_EINVAL, "null workspace");
    if (reinterpret_cast<uintptr_t>(d_workspace) & 255) return fail(TNS_EINVAL, "workspace must be 256-byte aligned");
    const Workspace w = carve(cache, B, d_workspace);
    if (workspace_bytes < w.bytes) return fail(TNS_ESIZE, "workspace smaller than tns_cache_workspace()");
    DeviceGuard guard(cache->cfg.device);
    if (guard.error() != hipSuccess) return fail_hip(guard.error(), "selecting the cache's device");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const CacheState& st = cache->st;
    const int policy = cache->cfg.policy;
    const int32_t dim = cache->cfg.dim;
    const int64_t C = cache->cfg.capacity, N = cache->cfg.num_ids;
    const int32_t maxrep = cache->max_replace;

    // The rows are gathered (bound by memory bandwidth; each row's threads look the slot up themselves) beside the update:
    // lookup proper (hit flags, counters, recorded accesses, first occurrence of every missed id), distinct misses, scores,
    // victims.  Both only read the maps and rows; the insertion changes them and waits for both.
    const bool vec4 = dim % 4 == 0 && ((reinterpret_cast<uintptr_t>(store) | reinterpret_cast<uintptr_t>(d_out)) & 15) == 0;
    const int32_t per_row = dim / (vec4 ? 4 : 1);
    const int64_t pieces = B * per_row;
    const RowOf row = row_of(per_row);
    // One launch for all but the lookup and the insertion, on the caller's stream; see kGatherWithin.
    const bool one_launch = (policy == TNS_CACHE_FIFO || C <= kOneGroupEntries) && pieces <= kGatherWithin && B <= kOneLaunchIds;
    const int64_t tiles_b = (B + kScanTile - 1) / kScanTile;
    const NewIds nf{st.first_idx, d_ids, w.slots, maxrep, w.new_ids, w.ctl};
    // Otherwise the caller's stream gathers and the update, a chain of launches, runs on a stream of the cache's own.
    hipStream_t us = one_launch ? stream : cache->side;
    if (!one_launch) {
        hipError_t ef = hipEventRecord(cache->forked, stream);
        if (ef == hipSuccess) ef = hipStreamWaitEvent(us, cache->forked, 0);
        if (ef != hipSuccess) return fail_hip(ef, "forking the cache update");
        // (a launch numbers its pieces with 31 bits, and has a whole number of rows)
        const int64_t step = kGatherPieces / per_row;
        for (int64_t b0 = 0; b0 < B; b0 += step) {
            const int64_t n = std::min(step, B - b0) * per_row;
            const dim3 grid(blocks_for((n + kGatherUnroll - 1) / kGatherUnroll));
            auto gather = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, st.rows, store, dim, (uint32_t)n, row, N, d_ids + b0, st.slot_of,
                                   d_out + b0 * dim);
            };
            vec4 ? gather(k_gather<4>) : gather(k_gather<1>);
        }
    }
    hipLaunchKernelGGL(k_lookup, dim3((unsigned)tiles_b), dim3(256), 0, us, st, policy, N, B, d_ids, w.slots, d_hit, w.ctl,
                       one_launch ? w.chain : nullptr, cache->first_ticket);
    if (one_launch) {
        const int unroll = update_unroll(vec4 ? 4 : 1);
        const int64_t gather_blocks = blocks_for((pieces + unroll - 1) / unroll, kOneGroup);
        const int64_t chunk = (pieces + gather_blocks * kOneGroup - 1) / (gather_blocks * kOneGroup) * kOneGroup;      // at most kOneGroup * unroll
        auto update = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles_b + gather_blocks)), dim3(kOneGroup), 0, us, st, nf, B, tiles_b, w.chain, w.victims,
                               store, dim, (uint32_t)pieces, (uint32_t)chunk, row, N, d_out);
        };
        if (policy == TNS_CACHE_FIFO) vec4 ? update(k_update<false, 4>) : update(k_update<false, 1>);
        else vec4 ? update(k_update<true, 4>) : update(k_update<true, 1>);
    } else if (maxrep > 0 && policy == TNS_CACHE_FIFO) {
        compact_flagged(nf, B, w.sums, us);
        hipLaunchKernelGGL(k_fifo_advance, dim3(1), dim3(1), 0, us, C, st.ring, w.ctl);
    } else if (maxrep > 0) {
        // few workgroups for the histograms: they are added to one global one with atomics
        const unsigned hb = (unsigned)std::min<int64_t>(blocks_for(C), 256);
        if (tiles_b <= kFoldTiles) {
            // distinct missed ids: tile sums, then the collect kernel, which shares its launch with pass 0 of the selection
            hipLaunchKernelGGL((k_flag_tile_sums<NewIds>), dim3((unsigned)tiles_b), dim3(256), 0, us, nf, B, w.sums);
            hipLaunchKernelGGL(k_newids_collect_hist0, dim3((unsigned)tiles_b + hb), dim3(256), 0, us, nf, B, w.sums, tiles_b, st.score, C, w.ctl,
                               (int64_t)hb);
        } else {
            compact_flagged(nf, B, w.sums, us);
            hipLaunchKernelGGL(k_select_hist, dim3(hb), dim3(256), 0, us, st.score, C, 0, w.ctl);
        }
        // the passes after the first: each picks the digit of the pass before it in its prologue
        for (int pass = 1; pass < kPasses; ++pass)
            hipLaunchKernelGGL(k_select_hist, dim3(hb), dim3(256), 0, us, st.score, C, pass, w.ctl);
        // victims in slot order; the tile-sum kernel picks the last digit first
        const Victims vf{st.score, w.ctl, w.victims};
        const int64_t tiles_c = (C + kScanTile - 1) / kScanTile;
        hipLaunchKernelGGL(k_victims_tile_sums, dim3((unsigned)tiles_c), dim3(256), 0, us, vf, w.ctl, C, w.sums);
        if (tiles_c <= kFoldTiles) {
            hipLaunchKernelGGL((k_flag_collect<Victims, true>), dim3((unsigned)tiles_c), dim3(256), 0, us, vf, C, w.sums);
        } else {
            hipLaunchKernelGGL((k_flag_scan_sums<Victims>), dim3(1), dim3(1024), 0, us, vf, w.sums, tiles_c);
            hipLaunchKernelGGL((k_flag_collect<Victims, false>), dim3((unsigned)tiles_c), dim3(256), 0, us, vf, C, w.sums);
        }
    }
    if (!one_launch) {
        hipError_t ej = hipEventRecord(cache->joined, us);
        if (ej == hipSuccess) ej = hipStreamWaitEvent(stream, cache->joined, 0);
        if (ej != hipSuccess) return fail_hip(ej, "joining the cache update");
    }
    // the insertion, and the clearing of this batch's first-occurrence marks for the next one, in one launch
    {
        const int64_t ib = maxrep > 0 ? (int64_t)blocks_for(maxrep, 4) : 0;
        auto insert = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(ib + blocks_for(B))), dim3(256), 0, stream, st, policy, dim, store, w.new_ids, w.victims,
                               w.ctl, ib, maxrep, B, d_ids, w.slots);
        };
        dim % 4 == 0 && (reinterpret_cast<uintptr_t>(store) & 15) == 0 ? insert(k_insert_clear<4>) : insert(k_insert_clear<1>);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "launching the cache kernels");
    return TNS_OK;
}

int tns_cache_stats(tns_cache* cache, void* hip_stream, int64_t* hits, int64_t* misses, int64_t* replaced) {
    tns::clear_error();
    if (!cache) return fail(TNS_EINVAL, "null cache");
    DeviceGuard guard(cache->cfg.device);
    if (guard.error() != hipSuccess) return fail_hip(guard.error(), "selecting the cache's device");
    unsigned long long all[kStripes * 3], h[3] = {0, 0, 0};
    hipError_t e = hipMemcpyAsync(all, cache->st.counters, sizeof(all), hipMemcpyDeviceToHost, static_cast<hipStream_t>(hip_stream));
    if (e == hipSuccess) e = hipStreamSynchronize(static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) return fail_hip(e, "reading the cache counters");
    for (int i = 0; i < kStripes; ++i)
        for (int k = 0; k < 3; ++k) h[k] += all[i * 3 + k];
    if (hits) *hits = (int64_t)h[0];
    if (misses) *misses = (int64_t)h[1];
    if (replaced) *replaced = (int64_t)h[2];
    return TNS_OK;
}

int tns_cache_save(tns_cache* cache, void* hip_stream, int32_t* h_id_of, int32_t* h_score, float* h_rows, int64_t* h_ring) {
    tns::clear_error();
    if (!cache || !h_id_of || !h_score || !h_rows || !h_ring) return fail(TNS_EINVAL, "null cache or buffer");
    DeviceGuard guard(cache->cfg.device);
    if (guard.error() != hipSuccess) return fail_hip(guard.error(), "selecting the cache's device");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int64_t C = cache->cfg.capacity;
    hipError_t e = hipMemcpyAsync(h_id_of, cache->st.id_of, (size_t)C * 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(h_score, cache->st.score, (size_t)C * 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(h_rows, cache->st.rows, (size_t)C * cache->cfg.dim * 4, hipMemcpyDeviceToHost, s);
    int32_t updates = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&updates, cache->st.updates, 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(h_ring, cache->st.ring, 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "saving the cache");
    for (int64_t i = 0; i < C; ++i) h_score[i] = (int32_t)((uint32_t)h_score[i] - (uint32_t)updates);
    return TNS_OK;
}

int tns_cache_restore(tns_cache* cache, void* hip_stream, const int32_t* h_id_of, const int32_t* h_score, const float* h_rows,
                      int64_t ring) {
    tns::clear_error();
    if (!cache || !h_id_of || !h_score || !h_rows) return fail(TNS_EINVAL, "null cache or buffer");
    const int64_t C = cache->cfg.capacity, N = cache->cfg.num_ids;
    if (ring < 0 || ring >= C) return fail(TNS_EINVAL, "ring position outside [0, capacity)");
    for (int64_t s = 0; s < C; ++s)
        if (h_id_of[s] < -1 || h_id_of[s] >= N) return fail(TNS_ERANGE, "saved id outside [-1, num_ids)");
    DeviceGuard guard(cache->cfg.device);
    if (guard.error() != hipSuccess) return fail_hip(guard.error(), "selecting the cache's device");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipMemcpyAsync(cache->st.id_of, h_id_of, (size_t)C * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(cache->st.score, h_score, (size_t)C * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(cache->st.rows, h_rows, (size_t)C * cache->cfg.dim * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(cache->st.ring, &ring, 8, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return fail_hip(e, "restoring the cache");
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(N)), dim3(256), 0, s, cache->st.slot_of, N, -1);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, s, cache->st.updates, 1, 0);
    hipLaunchKernelGGL(k_rebuild_map, dim3(blocks_for(C)), dim3(256), 0, s, cache->st.id_of, C, N, cache->st.slot_of);
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "restoring the cache");
    return TNS_OK;
}

TNS_API void tns_test_cache_no_wait(tns_cache* cache) { cache->first_ticket = kNoWait; }

int tns_cache_destroy(tns_cache* cache) {
    tns::clear_error();
    if (!cache) return TNS_OK;
    {
        DeviceGuard guard(cache->cfg.device);
        void* ptrs[] = {cache->st.slot_of, cache->st.first_idx, cache->st.id_of, cache->st.score,
                        cache->st.updates, cache->st.rows,      cache->st.counters, cache->st.ring};
        for (void* p : ptrs)
            if (p) (void)hipFree(p);
        if (cache->forked) (void)hipEventDestroy(cache->forked);
        if (cache->joined) (void)hipEventDestroy(cache->joined);
        if (cache->side) (void)hipStreamDestroy(cache->side);
    }
    delete cache;
    return TNS_OK;
}

}  // extern "C"
