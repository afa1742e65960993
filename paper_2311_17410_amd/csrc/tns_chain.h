// Single-pass chained scan over workgroup tiles (decoupled look-back): the piece shared by the sampling
// kernels (padding removal fused into sampling) and the device-side store builder (segment numbering and
// pool offsets in one launch each).  Included by .hip files only; everything has internal linkage.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

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
    uint64_t sampled_again;   // tagged chain: tiles, counted on from whatever this held (read by tests)
    uint64_t failed;          // tagged chain: the tag of a launch in which a wait ran out
    uint32_t noted;           // tagged chain: half the tag of a launch in which a tile has made room
    uint32_t pad[57];
    uint64_t status[1];   // [number of tiles]
};

__device__ __forceinline__ int64_t shfl64(int64_t v, int src) {
    const int lo = __shfl((int)(uint32_t)(v & 0xffffffffll), src, kChainWave);
    const int hi = __shfl((int)(v >> 32), src, kChainWave);
    return ((int64_t)hi << 32) | (uint32_t)lo;
}

// A sum over the wave by shuffles, in place: through a function object the same sum took two more registers of the kernels with a
// query per lane, and the uniform policy's over the prefix layout, which has 80, kept two values in scratch memory (C5, 2^28 queries:
// 24.25 -> 24.94 ms, 8 bytes a query written on top).
struct Shuffles {};

// Sum of the totals of all tiles before `tile` (called by one whole wave).  False if a tile had not reported after
// kSpinLimit polls: `excl` is then too small.  sum_of(v): the sum over the wave, or Shuffles.
template <class Sum>
__device__ __forceinline__ bool lookback(ScanWorkspace* ws, int64_t tile, int lane, int64_t& excl, const Sum& sum_of) {
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
        if constexpr (std::is_same_v<Sum, Shuffles>) {
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kChainWave);
        } else {
            v = sum_of(v);
        }
        excl += v;
        if (first < kChainWave) return true;
        idx -= kChainWave;
        fresh = true;
    }
}

// The same for a scan that cannot do without the tiles before this one: a wait that runs out is reported in *err_flag,
// before this tile publishes anything, so that whoever builds on its (wrong) prefix can see the flag.
template <class Sum>
__device__ __forceinline__ int64_t lookback_exclusive(ScanWorkspace* ws, uint32_t* err_flag, int64_t tile, int lane, const Sum& sum_of) {
    int64_t excl;
    if (!lookback(ws, tile, lane, excl, sum_of)) {
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
// state is cleared by a launch of its own (may_be_replayed).  Memory that by chance holds the tag of a launch: one word in 2^46.
//
// Every tile reads the totals of all tiles before it, four words per lane at a time; there are no prefixes to wait for.  Tiles
// are numbered as the workgroups are, and a tile may find that one before it has not even started: other work can hold an XCD for
// any time, and waiting tiles of two launches could each fill an XCD that the other one's earlier tiles need.  So a tile waits for
// tiles that have started, which publish without waiting for anything, and no more than about two milliseconds (kDeferSpins,
// hundreds of times what a tile takes) for one that has not.  Then it makes room: it leaves its dense rows out, notes that in its
// word and the launch's mark in the workspace's head.  Every tile says that it has started before it reads the head, so that whoever
// starts after the note sees the mark.  Workgroups that have made room or seen the mark look, when their own tile is done, for
// noted tiles and sample them again, beside one another, up to the first tile that has not started: that one will see the mark.
// The last tile, if it makes room, first leaves the end of the call as it would be if a tile never reported.
// What that can cost: 10^5 queries over power-law ids with 775 of their tiles sampled again, most of them by one workgroup, took
// 6.2 ms (8 us a tile) instead of 25 us.
// us per call, 2^21 edges, fan-out 10, tickets and clearing launch / this, 65537, 10^5, 2 * 10^5 and 2^18 - 1 queries: recent policy,
// uniform ids 22.2 / 15.2, 27.9 / 19.6, 37.4 / 30.4, 37.0 / 35.5, power-law ids 26.9 / 20.9, 32.9 / 24.9, 41.1 / 34.5, 38.2 / 36.9; uniform
// policy, power-law ids 39.3 / 33.2, 49.7 / 39.6, 68.5 / 58.2, 77.9 / 65.2; prefix layout, uniform ids, recent 32.3 / 14.4, 38.1 / 17.1,
// 44.9 / 28.5, 41.8 / 32.8, uniform policy 30.6 / 21.3, 36.3 / 23.5, 44.7 / 31.8, 44.7 / 34.7.  Both forms in one kernel, chosen at run time, cost
// the large batches of the prefix layout 1 to 4 %.
constexpr int kTotalBits = 16;                        // a tile's total is below 2^16
constexpr int kTagShift = kTotalBits + 2;
constexpr uint64_t kNotedBit = uint64_t(1) << kTotalBits;             // made room: its dense rows are to be written
constexpr uint64_t kPublishedBit = kNotedBit << 1;                    // (started, but not published: the tag alone)

// Tile t's word is status[t].
struct TaggedChain {
    struct Call {            // what only a tile that makes room or has others to see to needs
        int64_t queries;
        int64_t *end, *total_out;
        uint32_t* err_flag;
    };
    ScanWorkspace* ws;
    uint64_t tag;
    int32_t* s_todo;         // LDS, 0 before: what is left to do when the tile is done
    bool again = false;      // sampling a noted tile
    enum Todo : int32_t { kSeeToNoted = 1, kMakeRoom = 2 };
    // for every tile of a workgroup
    __device__ __forceinline__ void begin(void* scan_ws, uint64_t launch_tag, int64_t tile) {
        ws = static_cast<ScanWorkspace*>(scan_ws);
        tag = launch_tag;
        if (!again && threadIdx.x == 0) __hip_atomic_store(&ws->status[tile], tag << kTagShift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // before a wave's sums are counted in: the tile's start is known to all before its total is, and before its workgroup reads the head
    __device__ __forceinline__ void begun() const { wait_for_stores(); }
    // by one lane
    __device__ __forceinline__ void publish(int64_t tile, int32_t total) const {
        if (again) return;
        __hip_atomic_store(&ws->status[tile], tag << kTagShift | kPublishedBit | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Sum of the totals of all tiles before `tile` (called by one whole wave): four words per lane in flight.  -1: the tile has
    // waited for long enough, writes no dense rows, and is noted by next().  sum_of(v): the sum over the wave; such a call has less
    // than 2^31 dense entries.
    template <class Sum>
    __device__ __forceinline__ int64_t exclusive(int64_t tile, int lane, int defer_spins, const Sum& sum_of) const {
        const uint32_t noted = __hip_atomic_load(&ws->noted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int32_t sum = 0;
        int spins = 0;
        for (int64_t t0 = 0; t0 < tile; t0 += 4 * kChainWave) {
            uint64_t w[4];
            while (true) {
                bool ready = true, started = true;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t t = t0 + i * kChainWave + lane;
                    w[i] = tag << kTagShift | kPublishedBit;
                    if (t < tile) w[i] = __hip_atomic_load(&ws->status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ready = ready && published(w[i]);
                    started = started && w[i] >> kTagShift == tag;
                }
                if (!__ballot(!ready)) break;
                const bool wait = defer_spins >= 0 && !__ballot(!started);
                if (++spins > (wait ? kSpinLimit : defer_spins)) {
                    if (!wait) {
                        wait_for_stores();      // the total, before another wave notes
                        if (lane == 0) *s_todo = kMakeRoom;
                        return -1;
                    }
                    if (spins > kSpinLimit + 1) return 0;
                    fail(lane);      // and a last look: what publishes after it closes a call that has failed
                } else if (spins < 16) __builtin_amdgcn_s_sleep(2);
                else __builtin_amdgcn_s_sleep(16);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) sum += (int32_t)(w[i] & (kNotedBit - 1ull));
        }
        sum = sum_of(sum);
        if (lane == 0 && noted == (uint32_t)tag) *s_todo = kSeeToNoted;
        return sum;
    }
    // The end of the call, by the lane that writes it, all tiles having published: true if a wait of this launch ran out.
    __device__ __forceinline__ bool close(uint32_t* err_flag) const {
        const bool bad = __hip_atomic_load(&ws->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag;
        __hip_atomic_store(err_flag, bad ? 1u : 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return bad;
    }
    // After a tile, by the whole workgroup: true if there is another one for it to sample, again and now with its dense rows.
    // One wave looks for it: other workgroups take tiles too, and the waves of one must go on with the same.  s_tile, s_arrived: in
    // LDS, of the tile that is done; call(): the Call.
    template <class GetCall>
    __device__ __forceinline__ bool next(int64_t& tile, int32_t per_tile, int64_t* s_tile, int32_t* s_arrived, int lane, const GetCall& call) {
        if (!__builtin_amdgcn_readfirstlane(*s_todo)) return false;
        __syncthreads();
        if (threadIdx.x < kChainWave) {
            const Call c = call();
            if (*s_todo == kMakeRoom) note(tile, per_tile, lane, c);
            const int64_t t = take(again ? tile : 0, per_tile, lane, c);
            if (lane == 0) {
                *s_tile = t;
                *s_arrived = 0;
                *s_todo = kSeeToNoted;
            }
        }
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane((int)*s_tile);      // (a tile's number has 31 bits: grid.x)
        if (t < 0) return false;
        again = true;
        tile = t;
        return true;
    }

   private:
    __device__ __forceinline__ static void wait_for_stores() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0): as a rule nothing is on its way where this is called
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ bool published(uint64_t w) const { return w >> kTagShift == tag && (w & kPublishedBit); }
    // these by one whole wave
    __device__ __forceinline__ void fail(int lane) const {
        if (lane == 0) __hip_atomic_store(&ws->failed, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
    }
    __device__ __forceinline__ void note(int64_t tile, int32_t per_tile, int lane, const Call& c) const {
        if (lane == 0) {
            if ((tile + 1) * per_tile >= c.queries) {
                __hip_atomic_store(c.err_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(c.end, (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (c.total_out) __hip_atomic_store(c.total_out, (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __threadfence();      // (whoever samples the tile again overwrites these)
            __hip_atomic_fetch_or(&ws->status[tile], kNotedBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence();
            __hip_atomic_store(&ws->noted, (uint32_t)tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __threadfence();
        __builtin_amdgcn_wave_barrier();      // no lane looks for missing tiles before the note is made
    }
    // A noted tile from `from` on, to be sampled again; -1: none before the first tile that has not started, or a wait ran out.
    __device__ __forceinline__ int64_t take(int64_t from, int32_t per_tile, int lane, const Call& c) const {
        int spins = 0;
        for (int64_t t0 = from; t0 * per_tile < c.queries;) {
            const int64_t t = t0 + lane;
            uint64_t w = tag << kTagShift | kPublishedBit;
            if (t * per_tile < c.queries) w = __hip_atomic_load(&ws->status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t missing = __ballot(!published(w));
            const uint64_t first = missing & -missing;
            const uint64_t noted = __ballot((w & kNotedBit) != 0) & (first - 1);      // (none missing: all lanes)
            if (noted) {
                const int64_t found = t0 + __builtin_ctzll(noted);
                int taken = 0;
                if (lane == 0) {
                    taken = (__hip_atomic_fetch_and(&ws->status[found], ~kNotedBit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kNotedBit) != 0;
                    if (taken) __hip_atomic_fetch_add(&ws->sampled_again, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (__builtin_amdgcn_readfirstlane(taken)) return found;
            } else if (!missing) {
                t0 += kChainWave;
            } else {
                if (first & __ballot(w >> kTagShift != tag) || ++spins > kSpinLimit + 1) return -1;
                if (spins > kSpinLimit) fail(lane);
                else __builtin_amdgcn_s_sleep(16);
            }
        }
        return -1;
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
