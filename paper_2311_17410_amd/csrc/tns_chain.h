// Single-pass chained scan over workgroup tiles (decoupled look-back): the piece shared by the sampling
// kernels (padding removal fused into sampling) and the device-side store builder (segment numbering and
// pool offsets in one launch each).  Included by .hip files only; everything has internal linkage.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace tns {
namespace {

constexpr int kChainWave = 64;

// ---- single-pass chained scan over workgroup tiles (padding removal fused into sampling) ----
//
// Workspace layout: word 0 = tile ticket, word 1 = error flag, then one 64-bit status per tile:
// bits 62-63 = state (0 not ready, 1 tile total, 2 inclusive prefix), bits 0-61 = value.
// Tiles take their index from the ticket, so a tile only ever waits for tiles that have
// already started; the wait is bounded (lookback_exclusive sets the error flag if the bound is ever hit).
constexpr uint64_t kStTotal = 1ull << 62, kStPrefix = 2ull << 62, kStMask = 3ull << 62;
constexpr int kSpinLimit = 1 << 22;

struct ScanWorkspace {
    uint32_t ticket;
    uint32_t error;
    uint64_t deferred;    // tagged chain: the tag of a launch in which a tile has left its dense rows to the last one
    uint32_t pad[60];
    uint64_t status[1];   // [number of tiles]
};

__device__ __forceinline__ int64_t shfl64(int64_t v, int src) {
    const int lo = __shfl((int)(uint32_t)(v & 0xffffffffll), src, kChainWave);
    const int hi = __shfl((int)(v >> 32), src, kChainWave);
    return ((int64_t)hi << 32) | (uint32_t)lo;
}

// Sum of the totals of all tiles before `tile` (called by one whole wave).  False if a tile had not reported after
// kSpinLimit polls: `excl` is then too small.
__device__ __forceinline__ bool lookback(ScanWorkspace* ws, int64_t tile, int lane, int64_t& excl) {
    excl = 0;
    int64_t idx = tile - 1;
    int spins = 0;
    bool fresh = true;              // new window: every lane reads its tile's state
    uint64_t st = 0;
    while (true) {
        const int64_t t = idx - lane;
        // a lane re-reads only while its tile is not ready
        if (fresh || (st & kStMask) == 0) {
            st = kStPrefix;         // before the first tile: prefix 0
            if (t >= 0) st = __hip_atomic_load(&ws->status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        fresh = false;
        const uint64_t state = st & kStMask;
        const uint64_t is_prefix = __ballot(state == kStPrefix);
        const uint64_t not_ready = __ballot(state == 0);
        const int first = is_prefix ? __builtin_ctzll(is_prefix) : kChainWave;             // nearest tile with a full prefix
        const uint64_t needed = first >= kChainWave - 1 ? ~0ull : ((2ull << first) - 1);    // lanes 0..first
        if (not_ready & needed) {
            if (++spins > kSpinLimit) return false;
            __builtin_amdgcn_s_sleep(16);      // ~0.4 us between polls: late tiles are late by microseconds
            continue;
        }
        int64_t v = (lane <= first) ? (int64_t)(st & ~kStMask) : 0;
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kChainWave);
        excl += v;
        if (first < kChainWave) return true;
        idx -= kChainWave;
        fresh = true;
    }
}

// The same for a scan that cannot do without the tiles before this one: a wait that runs out is reported in *err_flag,
// before this tile publishes anything, so that whoever builds on its (wrong) prefix can see the flag.
__device__ __forceinline__ int64_t lookback_exclusive(ScanWorkspace* ws, uint32_t* err_flag, int64_t tile, int lane) {
    int64_t excl;
    if (!lookback(ws, tile, lane, excl)) {
        if (lane == 0) atomicExch(err_flag, 1u);
        __threadfence();
    }
    return excl;
}

// ---- the same for a small grid, without a launch that clears the state and without tickets --------------------------
//
// A batch of a few hundred tiles is bound by latency: the clearing launch is 2.5 us of it, and tickets, atomics on one word,
// are taken at 18 ns each (14 us for the 782 tiles of 10^5 queries).  Here a tile's word carries a tag next to the total, and
// a word with another tag has not been written yet, whatever the workspace held before.  The host draws a tag anew for every
// launch.  A captured launch is replayed with the tag it has, over words that the replay before may have left, so that there the
// state is cleared by a launch of its own (may_be_replayed).  Memory that by chance holds the tag of a launch: one word in 2^47.
//
// Every tile reads the totals of all tiles before it, four words per lane at a time; there are no prefixes to wait for.  Tiles
// are numbered as the workgroups are, which every XCD starts in that order.  Alone a launch cannot hold itself up, but XCDs
// start the workgroups of two queues in either order: waiting tiles of two launches could each fill an XCD that the other one's
// earlier tiles need.  So only the last tile waits for as long as it takes.  Any other one that has waited for kDeferSpins (about
// two milliseconds, hundreds of times what a tile takes) leaves its dense rows out and makes room, and the last tile's workgroup
// samples it again when all totals are there.  What waits is then one workgroup per launch.
// us per call, 2^21 edges, fan-out 10, tickets and clearing launch / this, recent policy, uniform ids: 65537 queries 22.6 /
// 13.4, 10^5 27.8 / 15.7, 2 * 10^5 37.0 / 25.3, 2^18 - 1 36.9 / 29.2; power-law ids 26.7 / 17.8, 32.5 / 20.5, 40.8 / 28.7, 38.0 / 30.5; uniform
// policy, power-law ids 38.8 / 32.0, 49.3 / 38.9, 66.8 / 58.0, 77.9 / 66.4; prefix layout, recent 32.4 / 23.5, 37.4 / 25.5, 44.7 /
// 32.6, 41.2 / 35.5 (the second figures without tiles that make room).  Both forms in one kernel, chosen at run time, cost the large batches of the prefix layout 1 to 4 %.
constexpr int kTotalBits = 16;                        // a tile's total is below 2^16
constexpr int kTagShift = kTotalBits + 1;             // between them: the tile has left its dense rows to the last one
constexpr uint64_t kDeferredBit = uint64_t(1) << kTotalBits;

// Tile t's word is status[t].
struct TaggedChain {
    ScanWorkspace* ws;
    uint64_t tag;
    int32_t* s_more;         // LDS: 1 if tiles have left their dense rows to this one, the last
    bool last_wg;            // the workgroup of the last tile
    bool again = false;      // which samples other tiles again
    int64_t last_tile = 0;
    __device__ __forceinline__ void start(bool is_last_tile, int32_t* more) {
        last_wg = is_last_tile;
        s_more = more;
    }
    // for every tile of a workgroup
    __device__ __forceinline__ void use(void* scan_ws, uint64_t launch_tag) {
        ws = static_cast<ScanWorkspace*>(scan_ws);
        tag = launch_tag;
    }
    __device__ __forceinline__ void publish(int64_t tile, int32_t total) const {
        if (again) return;
        __hip_atomic_store(&ws->status[tile], tag << kTagShift | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // what an error word holds after a wait of this launch ran out
    __device__ __forceinline__ uint32_t mark() const { return (uint32_t)tag | 1u; }
    // Sum of the totals of all tiles before `tile` (called by one whole wave): four words per lane in flight.  -1: the tile has
    // waited for long enough and leaves its dense rows to the last one.  It says so before its last look: either that look finds
    // what was missing, or the last tile, which goes on once nothing is missing, finds the note.
    __device__ __forceinline__ int64_t exclusive(uint32_t* err_flag, int64_t tile, int lane, int defer_spins) const {
        int64_t sum = 0;
        int spins = 0;
        bool noted = false;
        for (int64_t t0 = 0; t0 < tile; t0 += 4 * kChainWave) {
            uint64_t w[4];
            while (true) {
                bool ready = true;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t t = t0 + i * kChainWave + lane;
                    w[i] = tag << kTagShift;
                    if (t < tile) w[i] = __hip_atomic_load(&ws->status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) ready = ready && w[i] >> kTagShift == tag;
                if (!__ballot(!ready)) break;
                if (noted) return -1;
                if (++spins > kSpinLimit) {
                    if (lane == 0) atomicExch(err_flag, mark());
                    __threadfence();
                    return 0;
                }
                if (!last_wg && spins > defer_spins) {
                    if (lane == 0) {
                        __hip_atomic_fetch_or(&ws->status[tile], kDeferredBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        __threadfence();
                        __hip_atomic_store(&ws->deferred, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    __threadfence();
                    __builtin_amdgcn_wave_barrier();      // no lane looks before the note is made
                    noted = true;
                    continue;
                }
                if (spins < 16) __builtin_amdgcn_s_sleep(2);
                else __builtin_amdgcn_s_sleep(16);
            }
            int64_t v = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) v += (int64_t)(w[i] & (kDeferredBit - 1ull));
            sum += v;
        }
        for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, kChainWave);
        return sum;
    }
    // The end of the launch, by one lane that knows that every tile has published: true if a wait of this launch ran out.
    // An error word that holds anything else is made 0 (it held whatever the workspace did).
    __device__ __forceinline__ bool close(uint32_t* err_flag) const {
        __threadfence();
        const uint64_t left = __hip_atomic_load(&ws->deferred, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool bad = __hip_atomic_load(err_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mark();
        if (left == tag && !bad) *s_more = 1;
        if (!bad) __hip_atomic_store(err_flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return bad;
    }
    // After a tile, by the whole workgroup: true if there is another one for it to sample, again and now with its dense rows.
    // One wave looks for it: a tile's note may come between two waves' looks (it then writes its rows itself), and the waves
    // of a workgroup must go on with one tile.  s_tile, s_arrived: in LDS, of the tile that is done.
    __device__ __forceinline__ bool next(int64_t& tile, int64_t* s_tile, int32_t* s_arrived, int lane) {
        if (!last_wg) return false;
        __syncthreads();
        const int64_t last = again ? last_tile : tile;
        if (threadIdx.x < kChainWave) {
            uint64_t found = 0;
            int64_t t0 = again ? tile + 1 : 0;
            if (!*s_more) t0 = last;
            for (; t0 < last; t0 += kChainWave) {
                uint64_t w = 0;
                if (t0 + lane < last) w = __hip_atomic_load(&ws->status[t0 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                found = __ballot(w >> kTagShift == tag && (w & kDeferredBit));
                if (found) break;
            }
            if (lane == 0) {
                *s_tile = found ? t0 + __builtin_ctzll(found) : -1;
                *s_arrived = 0;
            }
        }
        __syncthreads();
        const int64_t t = *s_tile;
        if (__builtin_amdgcn_readfirstlane((int)(t < 0))) return false;
        last_tile = last;
        again = true;
        tile = t;
        return true;
    }
};

// At the start of every tile of a workgroup that may have several: nothing that follows from these is worth a register between them.
__device__ __forceinline__ void new_tile(int& lane, int& wave) {
    asm volatile("" : "+v"(lane), "+v"(wave));
    lane &= kChainWave - 1;
    wave &= 15;
}

}  // namespace
}  // namespace tns
