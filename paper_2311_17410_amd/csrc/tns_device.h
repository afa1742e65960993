// Device-side building blocks shared by the sampling kernels (tns_kernels.hip, tns_kernels_prefix.hip):
// the chained scan over workgroup tiles, the per-lane block walk of Algorithm 1, the cooperative
// gather and the coalesced stores.  Included by .hip files only; everything has internal linkage.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "../../include/tns.h"
#include "tns_chain.h"
#include "tns_kernels.h"
#include "tns_lanes.h"

namespace tns {
namespace {

constexpr int kXcds = 8;

// Workgroup -> tile mapping that gives each XCD (own L2) one contiguous range of tiles; the
// hardware hands consecutive workgroup ids to the XCDs round-robin.
__device__ __forceinline__ int64_t xcd_tile(int64_t bid, int64_t nb) {
    const int64_t q = nb / kXcds, r = nb % kXcds;
    const int64_t xcd = bid % kXcds, idx = bid / kXcds;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

__device__ __forceinline__ uint32_t div_by(uint32_t s, uint32_t f, uint32_t magic) {
    // floor(s / f) for s < 2^16 with magic = ceil(2^32 / f) (f >= 2)
    return f == 1 ? s : __umulhi(s, magic);
}

// Query of the wave that flat slot s of its 64 f slots belongs to: floor(s / f) for s < 2^12, f <= 64 (a 24-bit product
// with ceil(2^18 / f): the error s * (f - 1) / 2^18 stays below 1 / f).
__host__ __device__ inline uint32_t slot_multiplier(int32_t f) { return ((1u << 18) + (uint32_t)f - 1u) / (uint32_t)f; }
__device__ __forceinline__ uint32_t query_of_slot(uint32_t s, uint32_t f_mul) { return __umul24(s, f_mul) >> 18; }

// Rank in [0, c) for slot j of query qid: splitmix64 output function on the counter
// seed + G * (qid * f + j + 1), top 32 bits scaled by multiply-shift.
__device__ __forceinline__ uint64_t pick_rank(uint64_t seed, int64_t qid, int32_t f, int32_t j, uint64_t c) {
    uint64_t z = seed + 0x9E3779B97F4A7C15ull * ((uint64_t)qid * (uint64_t)f + (uint64_t)j + 1ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return ((z >> 32) * c) >> 32;
}

// Instance of query q, one of the wave's 64 consecutive queries from q0 on: instance b owns queries rowptr[b] ..
// rowptr[b + 1] - 1.  The wave finds the instance of its first query together, 64 probes a round (two dependent reads
// for 256 instances where a binary search per lane makes eight), and only a wave whose queries lie in several instances
// searches on from there lane by lane.  num_instances for a q beyond the last instance.
__device__ __forceinline__ int32_t instance_of(const int64_t* __restrict__ rowptr, int32_t num_instances, int64_t q0, int64_t q,
                                               int64_t Q, int lane) {
    int32_t first = 0, n = num_instances;
    while (n > 0) {
        const int32_t s = (n - 1) / kWave + 1;
        const bool past = rowptr[1 + first + (int32_t)min((int64_t)(lane + 1) * s - 1, (int64_t)n - 1)] <= q0;
        const int32_t cnt = __popcll(__ballot(past));
        const int32_t step = (int32_t)min((int64_t)cnt * s, (int64_t)n);
        first += step;
        n = max(min(s - 1, n - step), 0);
    }
    if (first >= num_instances || rowptr[first + 1] >= min(q0 + kWave, Q)) return first;
    int32_t lo = first, hi = num_instances;
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (rowptr[mid + 1] <= q) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// A value that is the same in all lanes of the wave, as the compiler cannot know: addresses formed from it are a scalar
// base and a 32-bit offset per lane, where 64-bit additions per lane and access were a third of the output stage's
// instructions.
__device__ __forceinline__ int32_t wave_uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t wave_uniform(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v & 0xffffffffll));
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The value of one lane, the same lane for the whole wave.
__device__ __forceinline__ int32_t wave_read(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ int64_t wave_read(int64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v & 0xffffffffll), lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

constexpr int kCoopGroup = 16;        // lanes per query in the cooperative search (recent policy)
constexpr int kGatherChunk = 10;      // gather iterations whose loads are issued together (8 and 5 measured slower)
// ... of which so many are prepared side by side (recent policy).  The last group of a fan-out that is no multiple prepares up
// to four iterations without a slot and re-reads a line in them.  A test around each load instead: 2^20 queries over power-law
// ids, fan-out 1 101.4 -> 100.3 us, 6 112.1 -> 111.6, 16 158 -> 157, but 10 120.0 -> 121.2 and 2^26 queries 6231 -> 6259; edge data
// on the host, any fan-out, no difference.
constexpr int kGatherGroup = 5;

// Unsigned index type of the same width as the LDS position entries: with a 32-bit index the edge
// load is addressed as base + 32-bit offset, one register per address.
template <typename pos_t> struct index_of { using type = uint64_t; };
template <> struct index_of<int32_t> { using type = uint32_t; };

// slot_word as a position entry: where entries are 32 bits wide every slot index is below 2^30, and the division by
// the slots per line is one 32-bit multiplication instead of a 64-bit one.
template <typename pos_t>
__device__ __forceinline__ pos_t slot_pos(int64_t s) {
    if (sizeof(pos_t) == 8) return (pos_t)slot_word(s);
    const uint32_t u = (uint32_t)s, line = u / (uint32_t)kSlotsPerLine;
    return (pos_t)(line * 32u + (u - line * (uint32_t)kSlotsPerLine) * 3u);
}
template <typename pos_t>
__device__ __forceinline__ float time_at(const uint32_t* __restrict__ edges, int64_t slot) {      // Edge::ts is the first word
    return __uint_as_float(edges[(typename index_of<pos_t>::type)slot_pos<pos_t>(slot)]);
}

// Number of leading items of [lo, lo + n) for which qual holds (they come first), by one lane with three reads in
// flight: half as many dependent round trips as a binary search.  Stops once at most `rest` items are undecided: lo
// is then moved past the decided ones and n is what is left.
template <class Qual>
__device__ __forceinline__ void narrow4(int32_t& lo, int32_t& n, int32_t rest, const Qual& qual) {
    while (n > rest) {
        const int32_t i1 = n >> 2, i2 = n >> 1, i3 = (int32_t)((3 * (int64_t)n) >> 2);
        int32_t b1 = qual(lo + i1), b2 = qual(lo + i2), b3 = qual(lo + i3);
        asm("" : "+v"(b1), "+v"(b2), "+v"(b3));      // (the compiler would read one after the other, each where it is first needed)
        const int32_t skip = b3 ? i3 + 1 : (b2 ? i2 + 1 : (b1 ? i1 + 1 : 0));
        const int32_t end = !b1 ? i1 : (!b2 ? i2 : (!b3 ? i3 : n));
        lo += skip;
        n = end - skip;
    }
}

// The same with one read in flight.
template <class Qual>
__device__ __forceinline__ void narrow2(int32_t& lo, int32_t& n, int32_t rest, const Qual& qual) {
    while (n > rest) {
        const int32_t half = n >> 1;
        const bool up = qual(lo + half);
        lo += up ? half + 1 : 0;
        n = up ? n - half - 1 : half;
    }
}

// State of one lane's walk over the blocks of its target node, newest block first
// (Algorithm 1).  `t` numbers the blocks in visiting order.
// SLOTS (recent policy): an entry of s_pos is not the edge's word index but its slot plus the entry's number, as the
// block tables of tns_kernels_recent.hip hold them.
template <int POLICY, bool INCL, typename pos_t, bool SLOTS = false>
struct Walk {
    float tb, te;                 // window [tb, te) or [tb, te]
    int32_t f;
    pos_t* s_pos;                 // this lane's f slots in LDS: word index of each selected edge
    const uint32_t* __restrict__ edges;   // edge lines as 4-byte words
    int32_t k = 0;                // slots filled so far (newest candidates first)
    int64_t c = 0;                // uniform: candidates seen in all overlapping blocks
    int32_t t_first = -1, t_last = -1, hi_first = 0, lo_last = 0;   // uniform: first/last overlapping block
    int32_t n_blocks = 0, n_probes = 0;                              // counted for the byte model
    // recent: search left to the wave.  When the window end falls inside a block, the lane only
    // narrows the search to at most `group` slots [d_lo, d_lo + d_n) of that block (edges before
    // d_lo are known to qualify); the wave then reads those timestamps side by side and counts,
    // right before it gathers from the same lines.
    int32_t group = 0;            // 0: the lane does every search itself
    int64_t d_off = -1;           // slot index of that block's first edge, -1: nothing left to the wave
    int32_t d_lo = 0, d_n = 0;

    // first index i in [0, n) with ts[i] >= x (STRICT=false) or ts[i] > x (STRICT=true)
    template <bool STRICT>
    __device__ __forceinline__ int32_t first_not_before(int64_t off, int32_t n, float x) {
        int32_t lo = 0, hi = n;
        while (lo < hi) {
            const int32_t mid = lo + ((hi - lo) >> 1);
            const float t = time_at<pos_t>(edges, off + mid);
            ++n_probes;
            const bool ge = STRICT ? (t > x) : (t >= x);
            if (ge) hi = mid; else lo = mid + 1;
        }
        return lo;
    }

    // Examine one block; returns false when no older block can contribute.
    __device__ __forceinline__ bool step(const BlockRec& r, int32_t t) {
        ++n_blocks;
        if (INCL ? (te < r.t_min) : (te <= r.t_min)) return true;   // block lies after the window: next older
        if (tb > r.t_max) return false;                             // block lies before the window: stop
        const int32_t size = rec_size(r);
        const int64_t off = rec_off(r);
        // candidate range [lo, hi) of the block; t_min / t_max settle most cases without a search
        int32_t hi = size;
        const bool all_before_end = INCL ? (te >= r.t_max) : (te > r.t_max);
        const bool tomb = rec_tombstones(r);   // some edges of the block are deleted: they count as absent
        if (POLICY == 0 && group > 0 && !tomb && !all_before_end && !(tb > r.t_min)) {
            // only the newest overlapping block can contain the window end, so nothing is recorded yet
            int32_t lo = 0;
            while (hi - lo > group) {
                const int32_t mid = lo + ((hi - lo) >> 1);
                const float tm = time_at<pos_t>(edges, off + mid);
                ++n_probes;
                const bool ge = INCL ? (tm > te) : (tm >= te);
                if (ge) hi = mid; else lo = mid + 1;
            }
            d_off = off; d_lo = lo; d_n = hi - lo;
            // the byte model counts what a binary search over the window would still read, not the
            // d_n timestamps the cooperating lanes fetch side by side
            n_probes += 32 - __clz(d_n);
            return true;            // older blocks supply the remaining slots
        }
        if (!all_before_end) hi = first_not_before<INCL>(off, size, te);
        int32_t lo = 0;
        if (tb > r.t_min) lo = first_not_before<false>(off, hi, tb);
        return record(off, lo, hi, tomb, t);
    }

    // Candidates [lo, hi) of the block whose edges start at slot `off` (visiting order t): records the
    // newest ones while slots are free and counts all of them for the uniform policy.  Returns false
    // when no older block can contribute.
    __device__ __forceinline__ bool record(int64_t off, int32_t lo, int32_t hi, bool tomb, int32_t t) {
        int32_t cnt = hi - lo;
        if (tomb) {
            // slow path: look at every candidate's validity (the edge id word), newest first
            cnt = 0;
            for (int32_t i = hi - 1; i >= lo; --i) {
                const int32_t id = (int32_t)edges[slot_word(off + i) + 2];
                ++n_probes;
                if (id < 0) continue;
                if (k < f) { s_pos[k] = SLOTS ? (pos_t)(off + i + k) : slot_pos<pos_t>(off + i); ++k; }
                ++cnt;
                if (POLICY == 0 && k >= f) break;
            }
            if (POLICY == 1 && cnt > 0) {
                if (t_first < 0) { t_first = t; hi_first = hi; }
                t_last = t; lo_last = lo;
                c += cnt;
            }
        } else if (cnt > 0) {
            const int32_t take = min(f - k, cnt);
            for (int32_t j = 0; j < take; ++j) s_pos[k + j] = SLOTS ? (pos_t)(off + hi - 1 + k) : slot_pos<pos_t>(off + hi - 1 - j);
            k += take > 0 ? take : 0;
            if (POLICY == 1) {
                if (t_first < 0) { t_first = t; hi_first = hi; }
                t_last = t; lo_last = lo;
                c += cnt;
            }
        }
        if (lo > 0) return false;                  // everything older is before the window
        if (POLICY == 0 && k >= f) return false;   // recent: the newest f are found
        return true;
    }

    // Uniform with more candidates than slots: f independent picks, rank counted from the
    // oldest candidate, stored as the negated distance from the newest one until resolved.
    __device__ __forceinline__ void draw(uint64_t seed, int64_t qid) {
        for (int32_t j = 0; j < f; ++j) {
            const int64_t from_newest = c - 1 - (int64_t)pick_rank(seed, qid, f, j, (uint64_t)c);
            s_pos[j] = (pos_t)(-(from_newest + 1));
        }
    }

    // Second visit of an overlapping block: turn the ranks that fall into it into positions.
    __device__ __forceinline__ void resolve(const BlockRec& r, int32_t t, int64_t& cum) {
        ++n_blocks;
        const int32_t hi = (t == t_first) ? hi_first : rec_size(r);
        const int32_t lo = (t == t_last) ? lo_last : 0;
        int64_t cnt = hi - lo;
        const int64_t off = rec_off(r);
        if (rec_tombstones(r)) {
            // ranks count valid edges only: walk them newest first
            cnt = 0;
            for (int32_t i = hi - 1; i >= lo; --i) {
                if ((int32_t)edges[slot_word(off + i) + 2] < 0) continue;
                for (int32_t j = 0; j < f; ++j) {
                    const int64_t sv = (int64_t)s_pos[j];
                    if (sv < 0 && -(sv + 1) - cum == cnt) s_pos[j] = slot_pos<pos_t>(off + i);
                }
                ++cnt;
            }
        } else {
            for (int32_t j = 0; j < f; ++j) {
                const int64_t sv = (int64_t)s_pos[j];
                if (sv < 0) {
                    const int64_t rr = -(sv + 1) - cum;
                    if (rr < cnt) s_pos[j] = slot_pos<pos_t>(off + hi - 1 - rr);
                }
            }
        }
        cum += cnt;
    }
};

// Around the loads of one of two branches that differ in the non-temporal hint alone: without it the compiler takes the loads of both
// for the same and makes one of them, without the hint.
__device__ __forceinline__ void keep_apart() { asm volatile("" ::: "memory"); }

// Ordering between LDS writes and reads of the SAME wave (rows are wave-private): the hardware
// executes a wave's LDS operations in order, so only the compiler must not reorder them.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier for data exchanged through LDS only: the wave waits for its LDS operations and meets the others, its
// stores stay in flight (a store is only done when the L2 has taken it, microseconds under load).  __syncthreads() is a
// fence for global memory as well.  How much of a wave's traffic it waits for is left to the compiler: nothing that needs
// other waves' stores or atomics performed may rely on either.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}


// The wave's cooperative gather: its 64*f slots in flat order, lane l handles slot it*64 + l, so
// consecutive lanes read consecutive edges of one query (12-byte loads within one or two lines)
// and every store instruction covers 256 consecutive bytes of an output array.  The loads of up to
// kGatherChunk iterations are issued together, into registers, before anything is stored: the
// wave pays the memory latency once per batch instead of once per slot.
struct GatherRegs {
    int32_t nbr[kGatherChunk], eid[kGatherChunk];     // eid < 0: empty slot (edge ids are non-negative)
    float ts[kGatherChunk];
};

// BRANCHY: each load sits in its own branch instead (uniform policy: every slot of a query lies in another
// line and the variant below measured slower there, C5 step 35.4 against 31.2 ms).
template <typename pos_t, bool BRANCHY = false>
__device__ __forceinline__ void gather_load(GatherRegs& g, const SampleArgs& p, uint32_t f_mul, int32_t stride,
                                            const pos_t* __restrict__ w_pos, int lane, int32_t it0, int32_t k) {
    const int32_t f = p.fanout;
    // The loads are unconditional (an empty slot reads the first edge of the array and drops it) and all
    // issued before the first result is looked at: loads inside divergent branches make the compiler lose
    // count of the memory operations in flight, and it then waits for ALL of them, stores included, before
    // every store that follows.
    if (BRANCHY) {
#pragma unroll
        for (int i = 0; i < kGatherChunk; ++i) {
            g.nbr[i] = -1; g.eid[i] = -1; g.ts[i] = 0.0f;
            if (it0 + i < f) {
                const uint32_t s = (uint32_t)((it0 + i) * kWave + lane);
                const uint32_t ql = query_of_slot(s, f_mul);
                const int32_t j = (int32_t)(s - ql * (uint32_t)f);
                const int32_t kq = __shfl(k, (int)ql, kWave);
                if (j < kq) {
                    const auto pos = (typename index_of<pos_t>::type)w_pos[ql * stride + j];
                    const Edge e = *reinterpret_cast<const Edge*>(p.edges + pos);
                    g.nbr[i] = e.nbr; g.eid[i] = e.eid; g.ts[i] = e.ts;
                }
            }
        }
        return;
    }
    bool filled[kGatherChunk];
    Edge raw[kGatherChunk];
#pragma unroll
    for (int i = 0; i < kGatherChunk; ++i) {
        filled[i] = false;
        raw[i].ts = 0.0f; raw[i].nbr = -1; raw[i].eid = -1;
        if (it0 + i < f) {          // uniform over the wave
            const uint32_t s = (uint32_t)((it0 + i) * kWave + lane);
            const uint32_t ql = query_of_slot(s, f_mul);
            const int32_t j = (int32_t)(s - ql * (uint32_t)f);
            const int32_t kq = __shfl(k, (int)ql, kWave);
            filled[i] = j < kq;
            // an empty slot reads what the first filled slot of the instruction reads (one request for both;
            // a fixed address instead would make one memory channel everybody's)
            const uint64_t m = __ballot(filled[i]);
            const pos_t own = filled[i] ? w_pos[ql * stride + j] : (pos_t)0;
            const pos_t other = sizeof(pos_t) == 8 ? (pos_t)shfl64((int64_t)own, m ? __builtin_ctzll(m) : 0)
                                                   : (pos_t)__shfl((int)own, m ? __builtin_ctzll(m) : 0, kWave);
            const auto pos = (typename index_of<pos_t>::type)(filled[i] ? own : other);
            raw[i] = *reinterpret_cast<const Edge*>(p.edges + pos);
        }
    }
    // every load of the batch has returned before the first store is issued: the stores that follow then
    // go out back to back without waiting for one another
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0) only
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kGatherChunk; ++i) {
        g.nbr[i] = filled[i] ? raw[i].nbr : -1;
        g.eid[i] = filled[i] ? raw[i].eid : -1;
        g.ts[i] = filled[i] ? raw[i].ts : 0.0f;
    }
}

// padded rows: slots of queries below Q, empty slots get the sentinels
__device__ __forceinline__ void store_padded(const GatherRegs& g, const SampleArgs& p, int lane, int32_t it0, int64_t q0, int64_t Q) {
    if (!p.out_nbr) return;      // dense-only run: the padded rows are not materialised
    const int32_t f = p.fanout;
    const int64_t out0 = q0 * f + (int64_t)it0 * kWave;
    int32_t* const nbr = p.out_nbr + out0;
    int32_t* const eid = p.out_eid + out0;
    float* const ts = p.out_ts + out0;
    const int32_t limit = (int32_t)min((int64_t)kWave, Q - q0) * f - it0 * kWave;       // slots from out0 on
    // (the test per store is kept although a full tile needs none: all stores in one run were slower under the uniform
    // policy, 2^22 queries 417 -> 460 us)
#pragma unroll
    for (int i = 0; i < kGatherChunk; ++i) {
        const uint32_t s = (uint32_t)(i * kWave + lane);
        if ((int32_t)s < limit) {
            __builtin_nontemporal_store(g.nbr[i], &nbr[s]);
            __builtin_nontemporal_store(g.eid[i], &eid[s]);
            __builtin_nontemporal_store(g.ts[i], &ts[s]);
        }
    }
}

// dense copy: `row0` = where the wave's first query starts, `excl` = where the lane's own query starts from there;
// consecutive lanes write consecutive entries
__device__ __forceinline__ void store_dense(const GatherRegs& g, const SampleArgs& p, uint32_t f_mul, int lane,
                                            int32_t it0, int64_t row0, int32_t excl) {
    const int32_t f = p.fanout;
    int32_t* const nbr = p.cmp_nbr + row0;
    int32_t* const eid = p.cmp_eid + row0;
    float* const ts = p.cmp_ts + row0;
    uint32_t at[kGatherChunk];
#pragma unroll
    for (int i = 0; i < kGatherChunk; ++i) {      // (all shuffles first; beyond the last slot their result is not used)
        const uint32_t s = (uint32_t)((it0 + i) * kWave + lane);
        const uint32_t ql = query_of_slot(s, f_mul);
        at[i] = (uint32_t)__shfl(excl, (int)ql, kWave) + (s - ql * (uint32_t)f);
    }
#pragma unroll
    for (int i = 0; i < kGatherChunk; ++i) {
        if (g.eid[i] >= 0) {
            nbr[at[i]] = g.nbr[i];
            eid[at[i]] = g.eid[i];
            ts[at[i]] = g.ts[i];
        }
    }
}

// ---- a workgroup's tile and the padding removal fused into sampling --------------------------------------

// The kernel's first argument, for a tile of a workgroup that may have several: what is read through this is read anew for every tile.
// (As ordinary arguments the loop's invariants fill the scalar registers: 100 to 700 moves to vector registers and back per kernel.)
__device__ __forceinline__ const SampleArgs& arguments_anew() {
    auto* p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const SampleArgs*)p;
}

__device__ __forceinline__ TaggedChain::Call call_of(const SampleArgs& p) {
    const int64_t Q = p.Q_dev ? min(p.Q, *p.Q_dev) : p.Q;
    return TaggedChain::Call{Q, &p.rowptr[Q], p.total_out, p.err_flag};
}

// How a kernel numbers its tiles and learns the dense entries of the tiles before one.
enum Scan : int {
    kNoScan,      // padded rows only
    kTickets,     // tiles numbered in the order workgroups start: a tile only ever waits for tiles that have started
    kTags,        // small grids (TaggedChain)
};
// Dense entries of the largest call without tickets, whatever its fan-out.
constexpr int64_t most_tagged_entries() {
    int64_t most = 0;
    for (int32_t f = 1; f <= TNS_MAX_FANOUT; ++f) most = std::max(most, tagged_queries(f) * f);
    return most;
}
static_assert(most_tagged_entries() < int64_t(1) << 31, "TaggedChain::exclusive adds up in 32 bits");
template <int SCAN>
struct TileChain {
    static constexpr bool kTagged = SCAN == kTags;
    TaggedChain tags;
    int64_t tile;
    __device__ __forceinline__ TileChain(const SampleArgs& p, int64_t* s_tile_base, int32_t* s_arrived, int32_t* s_todo) {
        if (threadIdx.x == 0) *s_arrived = 0;
        if (kTagged) {
            tile = (int64_t)blockIdx.x + p.first_ticket;
            if (threadIdx.x == 0) *s_todo = 0;
            tags.s_todo = s_todo;
            __syncthreads();
        } else {
            if (threadIdx.x == 0) *s_tile_base = (int64_t)atomicAdd(&static_cast<ScanWorkspace*>(p.scan_ws)->ticket, 1u);
            __syncthreads();
            tile = wave_uniform(*s_tile_base);
            __syncthreads();
        }
    }
    // for every tile of a workgroup
    __device__ __forceinline__ void begin(const SampleArgs& p) {
        if (kTagged) tags.begin(p.scan_ws, p.chain_tag, tile);
    }
    // before the wave's sum is counted in
    __device__ __forceinline__ void begun() const {
        if (kTagged) tags.begun();
    }
    __device__ __forceinline__ ScanWorkspace* ws(const SampleArgs& p) const { return static_cast<ScanWorkspace*>(p.scan_ws); }
    // one wave, at once, so that later tiles can look past this one
    __device__ __forceinline__ void publish_total(const SampleArgs& p, int32_t total, int lane) {
        if (lane != 0) return;
        if (kTagged) tags.publish(tile, total);
        else if (tile > 0) __hip_atomic_store(&ws(p)->status[tile], kStTotal | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // by the whole workgroup, after a tile: true if it has another one to sample
    __device__ __forceinline__ bool next(const SampleArgs& p, int64_t* s_tile_base, int32_t* s_arrived, int lane) {
        if (!kTagged) return false;
        return tags.next(tile, (int32_t)blockDim.x, s_tile_base, s_arrived, lane, [&]() { return call_of(p); });
    }
    // one wave: the dense entries of the tiles before this one; -1 (kTags): the tile writes no dense rows
    __device__ __forceinline__ int64_t look_back(const SampleArgs& p, int32_t total, int lane) const {
        if (kTagged) return tags.exclusive(tile, lane, p.defer_spins, [](int32_t v) { return wave_sum(v); });
        // (with tickets the sums stay shuffles: as vector instructions, us, 10^6 queries over the prefix layout 99.9 -> 100.0, where the
        // kernel before took 99.1 to 99.6, two hops from 2^20 roots 399 -> 402)
        const int64_t excl = tile > 0 ? lookback_exclusive(ws(p), p.err_flag, tile, lane, Shuffles{}) : 0;
        if (lane == 0)
            __hip_atomic_store(&ws(p)->status[tile], kStPrefix | (uint64_t)(excl + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return excl;
    }
    // by the last query's lane, whose tile has looked back over every other one: true if any wait ran into its bound
    __device__ __forceinline__ bool failed(const SampleArgs& p) const {
        if (kTagged) return tags.close(p.err_flag);
        __threadfence();
        return __hip_atomic_load(p.err_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    }
};
// Padded rows only: tiles in the order of the workgroups, or a contiguous range per XCD.
template <>
struct TileChain<kNoScan> {
    int64_t tile;
    __device__ __forceinline__ TileChain(const SampleArgs& p, int64_t*, int32_t*, int32_t*)
        : tile(p.xcd_remap ? xcd_tile(blockIdx.x, gridDim.x) : (int64_t)blockIdx.x) {}
    __device__ __forceinline__ void begin(const SampleArgs&) {}
    __device__ __forceinline__ void begun() const {}
    __device__ __forceinline__ bool next(const SampleArgs&, int64_t*, int32_t*, int) const { return false; }
};

// Output stage of a fused kernel: chained scan over the workgroup tiles for the dense offsets, padded rows, dense rows and
// rowptr.  k: the lane's filled slots; load(g, it0): the wave's slots from it0 * 64 on into registers.
// CHAIN_FIRST (recent policy): the look-back reads come before the wave's padded stores (a load result can only be waited
// for together with every store issued before it, and a store takes microseconds to be taken).  Uniform policy: the other
// order measured faster (C5 step 31.2 against 36.6 ms; its waves reach this point far apart).
// Sums over the wave and over the waves are vector instructions, not shuffles and loops, but where that measured slower.
//   kVectorSums: us with shuffles / with these, tickets, recent policy, prefix layout, 10^6 queries 94.6 / 94.0, windowed 87.9 / 86.7, 2^22
//   343 / 340; two hops from 2^20 roots 402 / 393
//   kShuffledScan, recent policy over blocks with tickets: the scan over the wave.  C5, 2^28 queries, 25.75 with it and 25.83 ms without, runs
//   within 0.01 of one another.  It is not for every size: 256 graphs 1341 with it and 1333 without, 2^22 queries 366 and 363, 2^25 and 2^26 the
//   same; but with both forms in the kernel, chosen by the number of queries, C5 takes 25.89
//   kLargeShuffled, uniform policy over the prefix layout without tickets: all of them with fan-outs that are gathered in batches.
//   Power-law ids, vector / this, fan-out 20, 4000 queries 61.8 / 59.8, 33000 69.7 / 67.5, fan-out 32 86.4 / 82.8, 95.4 / 92.1, fan-out 64 148 / 140, 162 / 155
//   kShuffled, the same with tickets: all of them.  Uniform ids, vector / this, fan-out 64, 180000 queries 87.6 / 80.0, 520000 189 / 165, 2 * 10^6
//   593 / 552, fan-out 32 57.6 / 55.1, 120 / 116, 356 / 337; fan-out 10 the same, C5 24.13 / 24.34 ms; chosen by the fan-out as without tickets
//   they are as slow as vector instructions
enum Sums : int { kVectorSums, kShuffledScan, kLargeShuffled, kShuffled };
template <bool CHAIN_FIRST, Sums SUMS, class Chain, class Load>
__device__ __forceinline__ void fused_output(const SampleArgs& p, int64_t* s_tile_base, int32_t* s_wave_sum, int32_t* s_arrived,
                                             Chain& tc, int wave, int waves_per_wg, int lane, int64_t q0, int64_t Q, int32_t k,
                                             uint32_t f_mul, const Load& load) {
    const int32_t f = p.fanout;
    int32_t inc = k;
    if (SUMS == kShuffledScan || SUMS == kShuffled || (SUMS == kLargeShuffled && f > kGatherChunk)) {
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t u = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += u;
        }
    } else {
        inc = wave_inclusive_scan(k);
    }
    tc.begun();
    auto chain = [&](int32_t wg_total) {
        const int64_t excl = tc.look_back(p, wg_total, lane);
        if (lane == 0) *s_tile_base = excl;
    };
    auto write_rowptr = [&](int64_t row0) {
        if (q0 + lane < Q) {
            __builtin_nontemporal_store(row0 + (inc - k), &p.rowptr[q0 + lane]);
            if (q0 + lane == Q - 1) {
                // If any wait ran into its bound the dense rows are not valid: the total then reads 0, so that a hop
                // chained to this one has no queries.
                const int64_t tot = tc.failed(p) ? 0 : row0 + inc;
                p.rowptr[Q] = tot;
                if (p.total_out) *p.total_out = tot;
            }
        }
    };
    auto row_of_wave = [&](int32_t off) {
        const int64_t base = *s_tile_base;
        return wave_uniform(Chain::kTagged && base < 0 ? base : base + off);
    };
    auto sum_before = [&](auto vector, int n) {      // of the first n waves
        if (decltype(vector)::value) return sum_of_waves(s_wave_sum, n, lane);
        int32_t sum = 0;
        for (int i = 0; i < n; ++i) sum += s_wave_sum[i];
        return sum;
    };
    constexpr std::integral_constant<bool, SUMS != kShuffled> small{};
    constexpr std::integral_constant<bool, SUMS != kShuffled && SUMS != kLargeShuffled> large{};
    GatherRegs g;
    if (f <= kGatherChunk) {
        // No barrier between a wave's searches and its gather (the lines the searches fetched are then still in the L2): the
        // waves count themselves in, and the one that arrives last adds up the tile total and publishes it.  Every wave
        // gathers (one batch of loads) and writes its padded rows, the gathered edges stay in registers; the last wave then
        // looks back for the tile's offset (the earlier tiles have had the time of a gather to publish their totals), and
        // only the dense copy waits for it.
        int is_last = 0;
        if (lane == kWave - 1) {
            s_wave_sum[wave] = inc;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            is_last = __hip_atomic_fetch_add(s_arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == waves_per_wg - 1;
        }
        is_last = __shfl(is_last, kWave - 1, kWave);
        int32_t wg_total = 0;
        if (is_last) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            wg_total = sum_before(small, waves_per_wg);
            tc.publish_total(p, wg_total, lane);
        }
        wave_lds_sync();      // what the load reads from LDS was written by this wave's own lanes
        load(g, 0);
        if (CHAIN_FIRST && is_last) chain(wg_total);
        store_padded(g, p, lane, 0, q0, Q);
        if (!CHAIN_FIRST && is_last) chain(wg_total);
        lds_barrier();
        const int64_t row0 = row_of_wave(sum_before(small, wave));
        if (Chain::kTagged && row0 < 0) return;
        write_rowptr(row0);
        store_dense(g, p, f_mul, lane, 0, row0, inc - k);
    } else {
        // larger fan-outs: offset first, then gather in batches and write both
        if (lane == kWave - 1) s_wave_sum[wave] = inc;
        __syncthreads();
        if (wave == 0) {
            const int32_t wg_total = sum_before(large, waves_per_wg);
            tc.publish_total(p, wg_total, lane);
            chain(wg_total);
        }
        __syncthreads();
        const int64_t row0 = row_of_wave(sum_before(large, wave));
        const bool dense = !Chain::kTagged || row0 >= 0;
        if (dense) write_rowptr(row0);
        for (int32_t it0 = 0; it0 < f; it0 += kGatherChunk) {
            load(g, it0);
            store_padded(g, p, lane, it0, q0, Q);
            if (dense) store_dense(g, p, f_mul, lane, it0, row0, inc - k);
        }
    }
}

// Waves per workgroup of a kernel with a query per lane, `most` or fewer by halves, so that a small batch's queries spread over the compute
// units instead of queueing at the address units of a few.
//   sampling alone, and under the uniform policy over the prefix layout (prefix_uniform) with fan-outs above 12: at least 512 workgroups.
//   33000 queries, fan-out 20 / 32 / 64 over power-law ids, 129 workgroups of four waves 70.5 / 97.0 / 164, 516 of one 67.5 / 92.1 / 155
//   with tickets: at least one per compute unit (fewer, larger tiles: a shorter chain), of the largest a quarter more, with
//   larger fan-outs three quarters, whose last ones would have the chip to themselves.  us with 512 / this: 400000
//   queries 58.7 / 55.5, power-law ids 59.9 / 56.6, prefix layout 54.2 / 49.7 and 59.9 / 55.5; fan-out 20, 200000 queries 43.1 / 36.5, 47.6 / 41.5,
//   42.3 / 36.3, 47.4 / 41.2.  Between one per compute unit and these lines, the largest / half of it: 270000 queries 45.3 / 44.3, 55.1 / 52.1, 44.4 / 43.5,
//   53.7 / 52.2, 315000 48.5 / 48.5, 55.0 / 53.6, 44.3 / 45.2, 53.9 / 53.3; fan-out 20, 330000 81.5 / 77.0, 85.5 / 82.3, 65.3 / 65.4, 75.1 / 73.7, 400000
//   89.6 / 89.5, 100.8 / 100.4, 73.2 / 75.4, 82.3 / 83.4
//   without tickets, one round of workgroups: what counts is how many waves the fullest compute unit has, and the fewest tiles with
//   which that is not a third more than it could be; with sixteen waves a workgroup fills a compute unit, so some are left free.
//   us with 512 / this, recent policy, uniform and power-law ids, prefix layout likewise: 40000 queries 12.9 / 12.5, 17.4 / 17.1, 13.2 / 12.3,
//   17.8 / 16.9; 65536 14.8 / 13.7, 19.4 / 18.3, 14.6 / 13.2, 18.9 / 17.5; 10^5 17.9 / 17.3, 21.8 / 21.1, 16.9 / 16.5, 20.6 / 19.9; 2 * 10^5 28.6 / 27.9,
//   31.8 / 31.5, 24.6 / 23.7, 28.4 / 28.1; 2^17, 150000 and 2^18 the same within 2 %
inline int workgroup_waves(int64_t Q, int32_t f, int most, bool fused, bool prefix_uniform = false) {
    constexpr int64_t kUnits = 256;
    auto tiles = [&](int w) { return (Q + (int64_t)w * kWave - 1) / ((int64_t)w * kWave); };
    int waves = most;
    const bool spread = !fused || (prefix_uniform && f > 12);
    if (spread || Q > tagged_queries(f)) {
        const int64_t of_largest = kUnits + (f > 12 ? 3 * kUnits / 4 : kUnits / 4);
        while (waves > 1 && tiles(waves) < (spread ? 2 * kUnits : (waves == most ? of_largest : kUnits))) waves >>= 1;
        return waves;
    }
    auto fullest = [&](int w) { return w * ((tiles(w) + kUnits - 1) / kUnits); };
    int64_t least = fullest(1);
    for (int w = 2; w <= most; w *= 2) least = std::min(least, fullest(w));
    while (waves > 1 && (3 * fullest(waves) > 4 * least || (waves == 16 && 8 * tiles(waves) > 7 * kUnits))) waves >>= 1;
    return waves;
}

// Launches `grid` workgroups, of `tile` queries each, of a kernel with a query per lane in the form that the batch asks for.
template <bool FUSED, class Launch>
hipError_t launch_tiles(const SampleArgs& a, int64_t grid, int64_t tile, hipStream_t stream, const Launch& launch) {
    SampleArgs b = a;
    if (!FUSED) {
        if (grid > 0) launch(std::integral_constant<int, kNoScan>{}, b);
        return hipGetLastError();
    }
    if constexpr (FUSED) {
        if (!b.err_flag) b.err_flag = &static_cast<ScanWorkspace*>(a.scan_ws)->error;
        if (grid > 0 && a.Q <= tagged_queries(a.fanout)) {
            // (sixteen waves and 64 slots would not fit; the LDS of a wave's rows keeps such workgroups smaller)
            if (tile * a.fanout >= (int64_t(1) << kTotalBits)) return hipErrorInvalidValue;
            const hipError_t e = ready_tags(b, grid, stream);
            if (e != hipSuccess) return e;
            launch(std::integral_constant<int, kTags>{}, b);
            return hipGetLastError();
        }
        if (!a.scan_ready) {
            // one state more than tiles: the workspace has it, and a test that starts the tickets at 1 uses it
            const hipError_t e = launch_scan_init(a, grid + 1, stream);
            if (e != hipSuccess) return e;
        }
        if (grid > 0) launch(std::integral_constant<int, kTickets>{}, b);
    }
    return hipGetLastError();
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ BlockRec as_rec(const uint4& u) {
    BlockRec r;
    r.t_min = __uint_as_float(u.x);
    r.t_max = __uint_as_float(u.y);
    r.off_lo = u.z;
    r.size_hi = u.w;
    return r;
}

}  // namespace
}  // namespace tns
