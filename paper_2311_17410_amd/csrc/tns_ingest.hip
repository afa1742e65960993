// gfx950 kernels of the device-side store builder: edge insertion (section 4.1 of the paper:
// append to the node's tail block while it has room, else link a new block at the tail, sized by
// b_v = min(deg(v), tau)) and tombstone deletion, on batches that already live in device memory.
//
// One batch runs in two phases with one host read-back between them:
//   plan   validate -> stable LSD radix sort of (source, time) keys, arrival order as the tie-break ->
//          segment heads (one segment = the batch's edges of one source node) -> per segment: order
//          check against the stored tail, edges that still fit the tail block, capacity and number
//          of the new blocks, edge lines and directory records they need -> exclusive scans of
//          those needs (every segment gets its own range of the pools: no allocation atomics, the
//          layout is reproducible);
//   apply  per segment: tail record, new block records (inline shift or directory run, runs grow
//          by doubling), node entry; per edge: its slot from the segment's plan, one 12-byte store.
// Nothing is changed before the host has seen the plan's status (errors reject the whole batch)
// and made room in the pools.
#include "tns_ingest.h"
#include "tns_chain.h"
#include "tns_lanes.h"

#include <algorithm>

#include "../../include/tns.h"

namespace tns {
namespace {

constexpr int kThreads = 256;
constexpr int kScanPer = 8;
constexpr int kScanTile = kThreads * kScanPer;

struct SegPlan {
    int64_t tail_slot;   // slot after the tail block's last edge: where the first `take` edges go
    int64_t slab_slot;   // small blocks: slot of the first free position of the node's current line
    int32_t take;        // edges that fit the tail block
    int32_t cap;         // capacity of each new block (0: none)
    int32_t nbn;         // number of new blocks
    int32_t k0;          // small blocks: how many fit the node's current line
};
static_assert(sizeof(SegPlan) == 32, "32 bytes per segment");

__device__ __forceinline__ void report(IngestStatus* st, int status, int64_t pos) {
    atomicMin(&st->err_word, ((unsigned long long)pos << 8) | (unsigned long long)(-status));
}

__global__ void __launch_bounds__(64) k_status_reset(IngestStatus* st) {
    if (threadIdx.x == 0) {
        st->err_word = ~0ull;
        st->unsorted = 0;
        st->num_segments = 0;
        st->total_lines = 0;
        st->total_dir = 0;
        st->new_blocks = 0;
        st->new_slots = 0;
        st->counter = 0;
    }
}

// ---- exclusive scan of an int64 array (three launches) -------------------------------------

__global__ void __launch_bounds__(kThreads) k_scan64_sums(const int64_t* __restrict__ in, int64_t n, int64_t* __restrict__ sums) {
    __shared__ int64_t s_w[kThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i)
        if (base + i < n) s += in[base + i];
    s = wave_sum64(s);
    if ((threadIdx.x & (kWave - 1)) == 0) s_w[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// one workgroup: exclusive scan of the tile sums in place, total to *total_out
__global__ void __launch_bounds__(1024) k_scan64_top(int64_t* __restrict__ sums, int64_t nb, int64_t* __restrict__ total_out) {
    __shared__ int64_t s_w[16];
    __shared__ int64_t s_carry;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < nb; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int64_t v = i < nb ? sums[i] : 0;
        const int64_t inc = wave_inclusive_scan64(v);
        if (lane == kWave - 1) s_w[wave] = inc;
        __syncthreads();
        int64_t off = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int64_t t = s_w[w];
            if (w < wave) off += t;
            all += t;
        }
        const int64_t carry = s_carry;
        if (i < nb) sums[i] = carry + off + (inc - v);
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + all;
        __syncthreads();
    }
    if (threadIdx.x == 0 && total_out) *total_out = s_carry;
}

__global__ void __launch_bounds__(kThreads) k_scan64_apply(const int64_t* in, int64_t* out, int64_t n,
                                                           const int64_t* __restrict__ sums) {
    __shared__ int64_t s_w[kThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int64_t v[kScanPer];
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        v[i] = base + i < n ? in[base + i] : 0;
        s += v[i];
    }
    const int64_t inc = wave_inclusive_scan64(s);
    if (lane == kWave - 1) s_w[wave] = inc;
    __syncthreads();
    int64_t run = sums[blockIdx.x] + (inc - s);
    for (int w = 0; w < wave; ++w) run += s_w[w];
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
}

hipError_t exclusive_scan64(const int64_t* in, int64_t* out, int64_t n, int64_t* sums, int64_t* total_out, hipStream_t stream) {
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb > 0) hipLaunchKernelGGL(k_scan64_sums, dim3((unsigned)nb), dim3(kThreads), 0, stream, in, n, sums);
    hipLaunchKernelGGL(k_scan64_top, dim3(1), dim3(1024), 0, stream, sums, nb, total_out);
    if (nb > 0) hipLaunchKernelGGL(k_scan64_apply, dim3((unsigned)nb), dim3(kThreads), 0, stream, in, out, n, sums);
    return hipGetLastError();
}

// ---- keys, radix sort ----------------------------------------------------------------------

// Key = (source id, order-preserving image of the timestamp); the value is the batch position.
// -0.0 and +0.0 compare equal, so both take the key of +0.0 and keep their arrival order.
__device__ __forceinline__ uint64_t key_of(int32_t v, float t) {
    uint32_t u = t == 0.0f ? 0u : __float_as_uint(t);
    u ^= (u >> 31) ? 0xffffffffu : 0x80000000u;
    return ((uint64_t)(uint32_t)v << 32) | u;
}
constexpr uint32_t kZeroTime = 0x80000000u;              // low word of a key: a time of either sign
__device__ __forceinline__ float time_of_key(uint32_t u) { return __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xffffffffu)); }
__global__ void __launch_bounds__(kThreads) k_keys(const IngestArgs a, uint64_t* __restrict__ key, uint32_t* __restrict__ val) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= a.m) return;
    const int32_t v = a.src[i];
    const float t = a.ts[i];
    if ((uint64_t)(uint32_t)v >= (uint64_t)a.num_nodes) report(a.status, TNS_ERANGE, i);
    else if (t != t) report(a.status, TNS_EORDER, i);
    else if (a.eid && a.eid[i] < 0) report(a.status, TNS_EINVAL, i);
    if (i > 0 && a.ts[i - 1] > t) atomicOr(&a.status->unsorted, 1u);
    key[i] = key_of(v, t);
    val[i] = (uint32_t)i;
}

// The four passes over the timestamp bits are skipped (on the device) when the batch arrived
// in time order, the usual case for a stream.
__global__ void __launch_bounds__(kThreads) k_radix_hist(const uint64_t* __restrict__ key, int64_t m, int shift, int64_t chunk,
                                                         int nblk, uint32_t* __restrict__ hist, const IngestStatus* st, int skippable) {
    if (skippable && !st->unsorted) return;
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = min(m, lo + chunk);
    for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) atomicAdd(&h[(uint32_t)(key[i] >> shift) & 255u], 1u);
    __syncthreads();
    hist[(size_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];   // digit-major
}

__global__ void __launch_bounds__(1024) k_radix_scan(uint32_t* __restrict__ hist, int64_t n, const IngestStatus* st, int skippable) {
    if (skippable && !st->unsorted) return;
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_carry;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < n; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const uint32_t v = i < n ? hist[i] : 0;
        uint32_t inc = v;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t u = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += u;
        }
        if (lane == kWave - 1) s_w[wave] = inc;
        __syncthreads();
        uint32_t off = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t t = s_w[w];
            if (w < wave) off += t;
            all += t;
        }
        const uint32_t carry = s_carry;
        if (i < n) hist[i] = carry + off + (inc - v);
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + all;
        __syncthreads();
    }
}

// Stable scatter: a workgroup walks its chunk in tiles of 256 keys; inside a tile a key's rank among
// the keys with the same digit comes from wave ballots (lanes with equal digits) plus the counts of
// the earlier waves.
__global__ void __launch_bounds__(kThreads) k_radix_scatter(const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                            uint64_t* __restrict__ kout, uint32_t* __restrict__ vout, int64_t m,
                                                            int shift, int64_t chunk, int nblk, const uint32_t* __restrict__ hist,
                                                            const IngestStatus* st, int skippable) {
    if (skippable && !st->unsorted) return;
    __shared__ uint32_t s_off[256];
    __shared__ uint32_t s_cnt[kThreads / kWave][256];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    s_off[t] = hist[(size_t)t * nblk + blockIdx.x];
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) s_cnt[w][t] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = min(m, lo + chunk);
    for (int64_t base = lo; base < hi; base += kThreads) {
        const int64_t i = base + t;
        const bool valid = i < hi;
        const uint64_t k = valid ? kin[i] : 0;
        const uint32_t d = (uint32_t)(k >> shift) & 255u;
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            same &= bit ? bal : ~bal;
        }
        const uint32_t rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        if (valid && rank == 0) s_cnt[wave][d] = (uint32_t)__popcll(same);
        __syncthreads();
        if (valid) {
            uint32_t pos = s_off[d] + rank;
            for (int w = 0; w < wave; ++w) pos += s_cnt[w][d];
            if ((int64_t)pos < m) {
                kout[pos] = k;
                vout[pos] = vin[i];
            }
        }
        __syncthreads();
        uint32_t add = 0;
#pragma unroll
        for (int w = 0; w < kThreads / kWave; ++w) {
            add += s_cnt[w][t];
            s_cnt[w][t] = 0;
        }
        s_off[t] += add;
        __syncthreads();
    }
}

// ---- segments ------------------------------------------------------------------------------

__device__ __forceinline__ bool is_head(const uint64_t* key, int64_t p) {
    return p == 0 || (uint32_t)(key[p] >> 32) != (uint32_t)(key[p - 1] >> 32);
}

__global__ void __launch_bounds__(kThreads) k_heads(const uint64_t* __restrict__ key, int64_t m, int64_t* __restrict__ head) {
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p < m) head[p] = is_head(key, p) ? 1 : 0;
}

__global__ void __launch_bounds__(kThreads) k_seg_start(const uint64_t* __restrict__ key, int64_t m,
                                                        const int64_t* __restrict__ head_excl, int32_t* __restrict__ seg_start) {
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= m) return;
    const bool h = is_head(key, p);
    if (h) seg_start[head_excl[p]] = (int32_t)p;
    if (p == m - 1) seg_start[head_excl[p] + (h ? 1 : 0)] = (int32_t)m;
}

__device__ __forceinline__ int64_t dir_run_for(int64_t blocks, int64_t have) {
    int64_t n = have > 2 * kDirAlign ? have : 2 * kDirAlign;
    while (n < blocks) n *= 2;
    return n;
}

__device__ __forceinline__ int64_t lines_of_blocks(int32_t cap, int32_t nbn, int32_t k0) {
    if (nbn == 0) return 0;
    if (cap >= kSlotsPerLine) return (int64_t)nbn * ((cap + kSlotsPerLine - 1) / kSlotsPerLine);
    const int32_t per_line = kSlotsPerLine / cap;
    return (nbn - k0 + per_line - 1) / per_line;
}

// slot of the first edge of the segment's j-th new block; `line0` = first edge line of the segment's range
__device__ __forceinline__ int64_t block_slot(const SegPlan& P, int64_t line0, int32_t j) {
    if (P.cap >= kSlotsPerLine) return (line0 + (int64_t)j * ((P.cap + kSlotsPerLine - 1) / kSlotsPerLine)) * kSlotsPerLine;
    if (j < P.k0) return P.slab_slot + (int64_t)j * P.cap;
    const int32_t per_line = kSlotsPerLine / P.cap, jj = j - P.k0;
    return (line0 + jj / per_line) * kSlotsPerLine + (int64_t)(jj % per_line) * P.cap;
}

__device__ __forceinline__ const BlockRec* tail_of(const IngestArgs& a, const NodeLine& nd, int64_t nidx) {
    if (nd.nblocks <= kInlineBlocks) return &a.nodes[nidx].rec[0];
    return &a.dir[(int64_t)nd.dir_line * kDirAlign + nd.nblocks - 1];
}

// What planning a segment reads of its node: the entry's header and its newest inline record, which lie side by side, the builder
// state, and the time of the segment's first edge.  All of it is requested at once, so that the plan is two dependent round trips,
// not four, and k_fast_plan requests it before the segment's length is known.
struct SegNode {
    uint4 h, r0;
    NodeAux ax;
    float t_first;
};
__device__ __forceinline__ void load_node(const IngestArgs& a, uint32_t v, SegNode& n) {
    if ((uint64_t)v >= (uint64_t)a.num_nodes) return;      // out-of-range ids were reported with the keys
    const int64_t nidx = a.node_base + v;
    n.h = *reinterpret_cast<const uint4*>(&a.nodes[nidx]);
    n.r0 = *(reinterpret_cast<const uint4*>(&a.nodes[nidx]) + 1);
    n.ax = a.aux[nidx];
}
__device__ __forceinline__ void load_segment_node(const IngestArgs& a, uint32_t v, uint32_t first, SegNode& n) {
    load_node(a, v, n);
    if ((uint64_t)v < (uint64_t)a.num_nodes) n.t_first = a.ts[first];
}

// What one segment (the batch's edges p0..p1 of one source node, sorted) needs: how many edges the tail block
// still takes, the new blocks' capacity and number, the edge lines and directory records to reserve.
// v: the node, mm: the number of edges, too_old(): called where the node has a later edge than the segment's first.
template <class TooOld>
__device__ __forceinline__ void plan_segment(const IngestArgs& a, uint32_t v, const SegNode& n, int64_t mm, SegPlan& P, int64_t& lines,
                                             int64_t& dirs, int64_t& blocks, int64_t& slots, const TooOld& too_old) {
    if ((uint64_t)v >= (uint64_t)a.num_nodes) return;
    const int64_t nidx = a.node_base + v;
    const uint4 h = n.h, r0 = n.r0;
    const NodeAux ax = n.ax;
    const float t_first = n.t_first;
    NodeLine nd;
    nd.nblocks = (int32_t)h.x; nd.degree = (int32_t)h.y; nd.dir_line = h.z;
    int64_t room = 0;
    if (nd.nblocks > 0) {
        BlockRec tr;
        if (nd.nblocks <= kInlineBlocks) {
            tr.t_min = __uint_as_float(r0.x); tr.t_max = __uint_as_float(r0.y); tr.off_lo = r0.z; tr.size_hi = r0.w;
        } else {
            tr = *tail_of(a, nd, nidx);
        }
        if (t_first < tr.t_max) too_old();
        room = ax.tail_cap - rec_size(tr);
        P.tail_slot = rec_off(tr) + rec_size(tr);
    }
    const int64_t take = room < mm ? (room > 0 ? room : 0) : mm;
    const int64_t rest = mm - take;
    P.take = (int32_t)take;
    if (rest > 0) {
        int64_t cap;
        if (a.sizing == TNS_SIZING_STRAWMAN) cap = rest;
        else if (a.sizing == TNS_SIZING_FIXED) cap = a.tau;
        else cap = max(rest, min((int64_t)nd.degree + take, (int64_t)a.tau));   // b_v = min(deg(v), tau)
        cap = min(cap, kMaxBlockEdges);
        P.cap = (int32_t)cap;
        P.nbn = (int32_t)(((uint32_t)rest + (uint32_t)cap - 1u) / (uint32_t)cap);       // both below 2^24
        if (cap < kSlotsPerLine && ax.slab_line) {
            P.k0 = min(P.nbn, (kSlotsPerLine - ax.slab_used) / (int32_t)cap);
            P.slab_slot = (int64_t)(ax.slab_line - 1) * kSlotsPerLine + ax.slab_used;
        }
        lines = lines_of_blocks(P.cap, P.nbn, P.k0);
        const int64_t after = (int64_t)nd.nblocks + P.nbn;
        if (after > kInlineBlocks && after > ax.dir_cap) dirs = dir_run_for(after, ax.dir_cap);
        blocks = P.nbn;
        slots = (int64_t)P.nbn * cap;
    }
}

// totals of the new blocks and their capacities: one pair of atomics per workgroup (atomics on one word serialise)
template <int WAVES = kThreads / kWave>
__device__ __forceinline__ void add_block_totals(IngestStatus* st, int64_t blocks, int64_t slots) {
    __shared__ int64_t s_blocks[WAVES], s_slots[WAVES];
    blocks = wave_sum64(blocks);
    slots = wave_sum64(slots);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_blocks[threadIdx.x / kWave] = blocks;
        s_slots[threadIdx.x / kWave] = slots;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        blocks = slots = 0;
        for (int w = 0; w < WAVES; ++w) {
            blocks += s_blocks[w];
            slots += s_slots[w];
        }
        if (blocks) {
            atomicAdd(&st->new_blocks, (unsigned long long)blocks);
            atomicAdd(&st->new_slots, (unsigned long long)slots);
        }
    }
}

__global__ void __launch_bounds__(kThreads) k_plan(const IngestArgs a, const uint64_t* __restrict__ key, const uint32_t* __restrict__ val,
                                                   const int32_t* __restrict__ seg_start, uint32_t* __restrict__ seg_src, SegPlan* __restrict__ plan,
                                                   int64_t* __restrict__ need_lines, int64_t* __restrict__ need_dir) {
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    int64_t blocks = 0, slots = 0;
    if (s < a.m) {
        int64_t lines = 0, dirs = 0;
        if (s < a.status->num_segments) {
            SegPlan P{};
            const int32_t p0 = seg_start[s];
            SegNode n{};
            load_segment_node(a, (uint32_t)(key[p0] >> 32), val[p0], n);
            plan_segment(a, (uint32_t)(key[p0] >> 32), n, seg_start[s + 1] - p0, P, lines, dirs, blocks, slots,
                         [&]() { report(a.status, TNS_EORDER, a.m + (int64_t)(key[p0] >> 32)); });
            seg_src[s] = (uint32_t)(key[p0] >> 32);
            plan[s] = P;
        }
        need_lines[s] = lines;
        need_dir[s] = dirs;
    }
    add_block_totals(a.status, blocks, slots);
}

// Loads of these values are requested together: the compiler would otherwise request one, wait for it, and use its register for the next.
__device__ __forceinline__ void side_by_side(int32_t& a, int32_t& b, int32_t& c) { asm volatile("" : "+v"(a), "+v"(b), "+v"(c)); }

struct SegTimes { float tail, first, last; };      // of the last edge for the tail block; of the first new block's first and last

// A planned batch as the apply phase reads it, left in memory by the planning kernels.
struct PlannedBatch {
    static constexpr bool kAhead = true;
    const uint64_t* __restrict__ key;         // sorted: source in the high word
    const uint32_t* __restrict__ val;         // batch position
    const int64_t* __restrict__ head_excl;    // segment heads before a position
    const int32_t* __restrict__ seg_start;
    const uint32_t* __restrict__ seg_src;     // source of a segment
    const SegPlan* __restrict__ plan;
    const int64_t* __restrict__ lines_base;
    const int64_t* __restrict__ dir_base;
    __device__ __forceinline__ uint32_t source(int64_t p) const { return (uint32_t)(key[p] >> 32); }
    __device__ __forceinline__ uint32_t position(int64_t p) const { return val[p]; }
    // a time lies in its key, but for the sign of a zero
    __device__ __forceinline__ float time_in(const IngestArgs& a, uint32_t u, int64_t p) const { return u == kZeroTime ? a.ts[val[p]] : time_of_key(u); }
    __device__ __forceinline__ float time(const IngestArgs& a, int64_t p) const { return time_in(a, (uint32_t)key[p], p); }
    __device__ __forceinline__ SegTimes times(const IngestArgs& a, const int32_t (&p)[3]) const {
        int32_t u[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) u[i] = (int32_t)(uint32_t)key[p[i]];
        side_by_side(u[0], u[1], u[2]);
        return SegTimes{time_in(a, (uint32_t)u[0], p[0]), time_in(a, (uint32_t)u[1], p[1]), time_in(a, (uint32_t)u[2], p[2])};
    }
};

// One thread per segment: tail record, new block records, node entry, builder state.  n: the node as it was when the segment was planned.
// Everything is read before the first store: a load behind stores is only waited for together with them.
template <class Batch>
__device__ __forceinline__ SegTimes segment_times(const IngestArgs& a, const Batch& b, const SegPlan& P, int32_t p0, int32_t p1) {
    const int32_t fresh = min(p0 + P.take, p1 - 1);
    const int32_t at[3] = {p0 + max(P.take, 1) - 1, fresh, P.cap < p1 - fresh ? max(fresh + P.cap - 1, p0) : p1 - 1};
    return b.times(a, at);
}
// The records of a node's inline list behind its newest, read with the entry (Batch::kAhead): moving them one by one is a round trip
// each, and so is copying a directory run.  It takes k_apply from 60 registers to 85, edges' threads too, eight waves per SIMD to five: us a batch
// without / with, 3 * 10^5 edges over 2^20 nodes 131.9 / 129.3, the others the same within what runs differ by: 10^4 over 2^16 37.8 / 37.6, 10^5
// over 2^18 51.3 / 51.5, over 2^20 power-law ids 74.9 / 73.1, 2^20 over 2^20 365 / 362, 2^21 over 2^20 666 / 672, over 2^22 938 / 944, 2^22 over 2^22
// 1960 / 1970, 2^24 - 1 over 2^22 4616 / 4660.  Not in k_small_batch, whose program would get longer than the round trips cost (2000 edges
// 33.7 -> 36).
typedef uint32_t rec_words __attribute__((ext_vector_type(4)));
struct OlderRecs { rec_words r[kInlineBlocks - 1]; };
__device__ __forceinline__ OlderRecs load_older(const NodeLine* N) {
    OlderRecs o;
#pragma unroll
    for (int j = 0; j < kInlineBlocks - 1; ++j) o.r[j] = *(reinterpret_cast<const rec_words*>(N) + 2 + j);
    return o;
}
static_assert(sizeof(NodeLine) == 16 + kInlineBlocks * 16, "a header and the inline records, 16 bytes each");
constexpr int kCopyAhead = 8;          // directory records in flight per thread
template <class Batch>
__device__ __forceinline__ void apply_node(const IngestArgs& a, const Batch& b, int64_t s, const SegPlan& P, int32_t p0, int32_t p1, int64_t nidx,
                                           const SegNode& n, const OlderRecs& older, const SegTimes& times) {
    const int64_t mm = p1 - p0;
    NodeLine* N = &a.nodes[nidx];
    const int32_t nb = (int32_t)n.h.x;
    const int64_t degree_before = (int32_t)n.h.y, after = (int64_t)nb + P.nbn;
    uint32_t dir_line = n.h.z;
    BlockRec tail;                         // inline list: its newest block
    tail.t_min = __uint_as_float(n.r0.x); tail.t_max = __uint_as_float(n.r0.y); tail.off_lo = n.r0.z; tail.size_hi = n.r0.w;
    if (P.take > 0) {
        BlockRec* tr = nb <= kInlineBlocks ? &N->rec[0] : &a.dir[(int64_t)dir_line * kDirAlign + nb - 1];
        BlockRec o = tail;
        if (nb > kInlineBlocks) o = *tr;
        o = make_rec(o.t_min, times.tail, rec_off(o), rec_size(o) + P.take, rec_tombstones(o));
        tail = o;
        *tr = o;
    }
    if (P.nbn > 0) {
        NodeAux ax = n.ax;
        const int64_t lines = lines_of_blocks(P.cap, P.nbn, P.k0);
        const int64_t line0 = a.used_lines + b.lines_base[s];
        if (line0 + lines > a.cap_lines) { atomicOr(&a.status->internal, 1u); return; }
        const int64_t rest = mm - P.take;
        BlockRec* run = nullptr;
        if (after > kInlineBlocks) {
            if (after > ax.dir_cap) {
                const int64_t room = dir_run_for(after, ax.dir_cap);
                const int64_t start = a.used_dir + b.dir_base[s];
                if (start + room > a.cap_dir) { atomicOr(&a.status->internal, 2u); return; }
                BlockRec* dst = a.dir + start;
                uint32_t* dcum = a.dir_cum + start;
                const BlockRec* old = a.dir + (int64_t)dir_line * kDirAlign;
                const uint32_t* ocum = a.dir_cum + (int64_t)dir_line * kDirAlign;
                uint32_t before = 0;
                if (nb <= kInlineBlocks && Batch::kAhead) {
#pragma unroll
                    for (int j = kInlineBlocks - 1; j >= 0; --j) {                       // oldest first
                        const rec_words newest = {__float_as_uint(tail.t_min), __float_as_uint(tail.t_max), tail.off_lo, tail.size_hi};
                        const rec_words o = j > 0 ? older.r[j > 0 ? j - 1 : 0] : newest;
                        if (j < nb) {
                            *reinterpret_cast<rec_words*>(&dst[nb - 1 - j]) = o;
                            dcum[nb - 1 - j] = before;
                            before += o.w & 0xffffffu;       // rec_size()
                        }
                    }
                } else if (nb <= kInlineBlocks) {
                    for (int j = nb - 1; j >= 0; --j) {
                        BlockRec o = tail;
                        if (j > 0) o = N->rec[j];      // (a choice of one of the two would be one of addresses, with `tail` in memory)
                        dst[nb - 1 - j] = o;
                        dcum[nb - 1 - j] = before;
                        before += (uint32_t)rec_size(o);
                    }
                } else if (Batch::kAhead) {
#pragma unroll 1
                    for (int32_t j0 = 0; j0 < nb; j0 += kCopyAhead) {
                        rec_words o[kCopyAhead];
                        uint32_t c[kCopyAhead];
#pragma unroll
                        for (int u = 0; u < kCopyAhead; ++u) {
                            o[u] = *reinterpret_cast<const rec_words*>(&old[min(j0 + u, nb - 1)]);
                            c[u] = ocum[min(j0 + u, nb - 1)];
                        }
#pragma unroll
                        for (int u = 0; u < kCopyAhead; ++u) {
                            if (j0 + u < nb) {
                                *reinterpret_cast<rec_words*>(&dst[j0 + u]) = o[u];
                                dcum[j0 + u] = c[u];
                            }
                        }
                    }
                } else {
                    for (int32_t j = 0; j < nb; ++j) {
                        dst[j] = old[j];
                        dcum[j] = ocum[j];
                    }
                }
                dir_line = (uint32_t)(start / kDirAlign);
                ax.dir_cap = (int32_t)room;
            }
            run = a.dir + (int64_t)dir_line * kDirAlign;
        } else {
            // newest first: room in front
            if (Batch::kAhead) {
#pragma unroll
                for (int j = 1; j < kInlineBlocks; ++j)
                    if (j < nb) *reinterpret_cast<rec_words*>(&N->rec[j + P.nbn]) = older.r[j - 1];
            } else {
                for (int j = nb - 1; j > 0; --j) N->rec[j + P.nbn] = N->rec[j];
            }
            if (nb > 0) N->rec[P.nbn] = tail;
        }
        uint32_t* run_cum = run ? a.dir_cum + (int64_t)dir_line * kDirAlign : nullptr;
        for (int32_t j = 0; j < P.nbn; ++j) {
            const int64_t first = (int64_t)p0 + P.take + (int64_t)j * P.cap;
            const int64_t size = min((int64_t)P.cap, rest - (int64_t)j * P.cap);
            float t_min = times.first, t_max = times.last;
            if (j > 0) { t_min = b.time(a, first); t_max = b.time(a, first + size - 1); }
            const BlockRec r = make_rec(t_min, t_max, block_slot(P, line0, j), (int32_t)size);
            if (run) {
                run[nb + j] = r;
                run_cum[nb + j] = (uint32_t)(degree_before + P.take + (int64_t)j * P.cap);   // edges in the older blocks
            } else {
                N->rec[P.nbn - 1 - j] = r;
            }
        }
        ax.tail_cap = P.cap;
        if (P.cap < kSlotsPerLine) {
            const int32_t per_line = kSlotsPerLine / P.cap, rem = P.nbn - P.k0;
            if (rem > 0) {
                ax.slab_line = (uint32_t)(line0 + lines - 1 + 1);
                ax.slab_used = ((rem - 1) % per_line + 1) * P.cap;
            } else {
                ax.slab_used += P.nbn * P.cap;
            }
        }
        a.aux[nidx] = ax;
    }
    N->nblocks = (int32_t)after;
    N->degree = (int32_t)(degree_before + mm);
    N->dir_line = dir_line;
}

// The record made ready for the next batch (`internal` stays: it is reported by the next read-back).
__device__ __forceinline__ void ready_status(IngestStatus* st) {
    st->err_word = ~0ull;
    st->unsorted = 0;
    st->num_segments = 0;
    st->total_lines = 0;
    st->total_dir = 0;
    st->new_blocks = 0;
    st->new_slots = 0;
    st->counter = 0;
}

// One thread per edge (sorted position): what is stored, and its slot from the segment's plan.
struct EdgeWords { uint32_t ts, nbr, eid; };
__device__ __forceinline__ EdgeWords load_edge(const IngestArgs& a, uint32_t e) {
    const int32_t* const ids = a.eid ? a.eid : a.dst;      // (no load sits in a branch)
    const uint32_t id = (uint32_t)ids[e];
    return EdgeWords{__float_as_uint(a.ts[e]), (uint32_t)a.dst[e], a.eid ? id : (uint32_t)(int32_t)(a.eid_base + (int64_t)e)};
}
// r: the edge's number in its segment; lines_base: the segment's
__device__ __forceinline__ void apply_edge(const IngestArgs& a, const SegPlan& P, int64_t r, int64_t lines_base, const EdgeWords& edge) {
    int64_t slot;
    if (r < P.take) {
        slot = P.tail_slot + r;
    } else {
        const int64_t rr = r - P.take;
        const int32_t j = (int32_t)((uint32_t)rr / (uint32_t)P.cap);      // both below 2^24
        slot = block_slot(P, a.used_lines + lines_base, j) + (rr - (int64_t)j * P.cap);
    }
    if (slot / kSlotsPerLine >= a.cap_lines) { atomicOr(&a.status->internal, 4u); return; }
    const int64_t w = slot_word(slot);
    a.lines[w] = edge.ts;
    a.lines[w + 1] = edge.nbr;
    a.lines[w + 2] = edge.eid;
}

// Both in one launch: an edge's slot follows from the plan alone, so the two parts do not depend on each other.
// (100 K edges: 14.4 us against 7.8 + 10.2 and the gap between the two launches.)
// What bounds it is the chain of dependent reads: the plan's word to go ahead, the segment, its node and times.  The first two are
// requested together, a segment's source has an array of its own, and a time is read from its key; likewise in k_fast_plan, and
// the keys are made by the first sorting pass, not written for it.  us a batch with the sampling of its events: 10^4 edges over 2^16 nodes
// 45.5 -> 43.3, 10^5 over 2^18 71.5 -> 69.9, over 2^20 power-law ids 120 -> 115, 3 * 10^5 over 2^20 201 -> 198.
__global__ void __launch_bounds__(kThreads) k_apply(const IngestArgs a, const PlannedBatch b, int64_t num_segments, unsigned node_blocks,
                                                    const int64_t* __restrict__ go) {
    // (clamped and requested beside the number of segments, which a launch queued before the host has seen the plan reads)
    int64_t limit = go ? *go : num_segments;
    // the node part first: it is the longer chain of dependent reads
    if (blockIdx.x < node_blocks) {
        const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x, at = min(s, a.m - 1);
        SegPlan P = b.plan[at];
        int32_t p0 = b.seg_start[at], p1 = b.seg_start[at + 1];
        uint32_t source = b.seg_src[at];
        asm volatile("" : "+v"(limit), "+v"(P.tail_slot), "+v"(P.take), "+v"(p0), "+v"(p1), "+v"(source));
        if (s < limit) {
            const int64_t nidx = a.node_base + source;
            SegNode n;
            n.h = *reinterpret_cast<const uint4*>(&a.nodes[nidx]);
            n.r0 = *(reinterpret_cast<const uint4*>(&a.nodes[nidx]) + 1);
            n.ax = a.aux[nidx];
            apply_node(a, b, s, P, p0, p1, nidx, n, load_older(&a.nodes[nidx]), segment_times(a, b, P, p0, p1));
        }
    } else {
        const int64_t p = (int64_t)(blockIdx.x - node_blocks) * kThreads + threadIdx.x, at = min(p, a.m - 1);
        uint32_t e = b.position(at), own = b.source(at), before = b.source(at > 0 ? at - 1 : 0);
        int64_t seg = b.head_excl[at];
        asm volatile("" : "+v"(limit), "+v"(e), "+v"(own), "+v"(before), "+v"(seg));
        if (limit <= 0) return;
        // (the host has read the record or has a copy of it: the next plan needs no launch of its own for it)
        if (p == 0) ready_status(a.status);
        if (p < a.m) {
            if (p > 0 && own == before) --seg;
            const SegPlan P = b.plan[seg];
            const int64_t r = p - b.seg_start[seg], lines_base = b.lines_base[seg];
            apply_edge(a, P, r, lines_base, load_edge(a, e));
        }
    }
}

// ---- short pipeline for stream-sized batches -------------------------------------------------
//
// A batch of the size streams are ingested in (the paper's 100 K edges) spends its time in launches,
// not in memory traffic, so the planning phase above (about 40 dependent launches) is cut to four
// for batches that fit kFastMaxBatch and arrive in time order, the usual case for a stream:
//   k_fast_keys      validation, and every tile's histogram of the first digit;
//   k_fast_scatter   x 2: stable radix pass over one half of the source id's bits.  Every tile adds
//                    up the histograms of the tiles before it by itself (at most kFastMaxTiles rows, read
//                    from the L2), so a pass needs no separate scan launch and no tile waits for another;
//                    the first pass also counts the second digit per destination tile for the second pass;
//   k_fast_plan      segment heads and numbers, the per-segment plan and the pool offsets (chained scans) in one launch.
// Time order is assumed, not known: k_fast_keys sets `unsorted` as the general pipeline does, and
// the host, which reads the status before anything is changed, then runs the general pipeline instead.
// keys per sort tile: small batches take smaller tiles so that they still spread over the compute units, large ones
// larger tiles so that the table of tile histograms every tile reads stays short (us per batch with the sampling of its
// events, 1024 / 2048 / 4096 keys per tile: 10^5 edges 91 / 93 / -, 2 * 10^5 power-law ids 167 / 174 / 190, 2^18 167 / 168 /
// 173, 3 * 10^5 233 / 237 / 238, 2^19 392 / 402 / 389)
constexpr int kFastTileMax = 4096;
inline int fast_tile_keys(int64_t m) { return m <= (int64_t(1) << 17) ? 1024 : (m <= (int64_t(1) << 18) ? 2048 : kFastTileMax); }
constexpr int kScatThreads = 512;                       // the radix passes: 8 waves x 8 keys per lane on the same tiles
constexpr int kScatRows = 13;                            // rows of the table that a thread has in flight
constexpr int kScatGroups = 4;                          // parts of the table of tile histograms that are added up side by side
__host__ __device__ constexpr int scatter_groups(int bins) { return kScatThreads / (bins / 4) < 1 ? 1 : (kScatThreads / (bins / 4) < kScatGroups ? kScatThreads / (bins / 4) : kScatGroups); }
constexpr int kFastMaxTiles = 512;
constexpr int64_t kFastMaxBatch = (int64_t)kFastTileMax * kFastMaxTiles;   // 2^21 edges
constexpr int kFastMaxBits = 12;                        // bits per digit: two digits cover 2^24 nodes
constexpr int kPlanThreads = 512;                       // k_fast_plan: one sorted position per thread, 512 per tile
// Batches planned and applied by one workgroup (k_small_batch).  us per batch with the sampling of its events, with it / with
// the same in two launches and a bitonic sort, which above this size was slower than the five kernels (3000 edges over
// 2^18 nodes 73.2 / 51.9 us without the sampling): 600 edges over 2^18 nodes 46 / 56, 2000 over 2^18 57 / 68, 2000 over 2^16
// power-law ids 48 / 59, 2048 over two nodes 43 / 58.  Twice the size does not fit the LDS.
constexpr int64_t kSmallBatch = 2048;
constexpr uint32_t kInternalScan = 8u;                  // IngestStatus::internal: a chained scan's bounded wait ran out

// Tile index in launch order, and the sum of the totals of the tiles before it: one chained-scan step of a
// workgroup.  `total` is the tile's own sum; the inclusive prefix is published for the tiles after it.
// Called by one whole wave; lane 0 holds the result.  A bounded wait that runs out marks the scan's own error
// word (later tiles and kernels look at it) and the status record the host reads.
__device__ __forceinline__ int64_t chain_wave(ScanWorkspace* ws, IngestStatus* st, int64_t tile, int64_t total, int lane) {
    if (lane == 0 && tile > 0)
        __hip_atomic_store(&ws->status[tile], kStTotal | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t excl = tile > 0 ? lookback_exclusive(ws, &ws->error, tile, lane, [](int64_t v) { return wave_sum64(v); }) : 0;
    if (lane == 0) {
        __hip_atomic_store(&ws->status[tile], kStPrefix | (uint64_t)(excl + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__hip_atomic_load(&ws->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(&st->internal, kInternalScan);
    }
    return excl;
}

// Waits until the wave's memory operations have been performed.  __syncthreads() does not: a wave's atomics may stay in
// flight across a barrier.  Enough where what follows the barrier concerns atomics only; a __threadfence() by every thread
// would write the L2 back as well (batches of 100 K edges 82 -> 103 us).
__device__ __forceinline__ void wait_for_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ IngestStatus load_status(const IngestStatus* st) {      // past the caches of this compute unit
    IngestStatus r;
    const unsigned long long* src = reinterpret_cast<const unsigned long long*>(st);
    unsigned long long* copy = reinterpret_cast<unsigned long long*>(&r);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(IngestStatus) / 8); ++i) copy[i] = __hip_atomic_load(&src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return r;
}

// The finished record goes to the host: the record first, then the batch's sequence number.
__device__ __forceinline__ void send_to_host(const IngestArgs& a, const IngestStatus& r) {
    const unsigned long long* copy = reinterpret_cast<const unsigned long long*>(&r);
    unsigned long long* dst = reinterpret_cast<unsigned long long*>(a.host_status);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(IngestStatus) / 8); ++i) dst[i] = copy[i];
    __threadfence_system();
    __hip_atomic_store(a.host_seq, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The record goes to the host, and the apply kernel queued behind the plan learns whether it may run: the
// batch is sound and in time order and the pools have room.  The host comes to the same conclusion from the record and
// otherwise (an error, the general pipeline, larger pools) goes on by itself.  One thread, after the last update of *status.
__device__ __forceinline__ void hand_over(const IngestArgs& a, const IngestStatus& r) {
    *a.go = ingest_may_apply(r, a) ? r.num_segments : 0;
    send_to_host(a, r);
}

constexpr int kPlanScans = 4;
struct PlanScans { ScanWorkspace* ws[kPlanScans]; };      // of k_fast_plan

template <int TILE>
__global__ void __launch_bounds__(kThreads) k_fast_keys(const IngestArgs a, uint32_t* __restrict__ hist1,
                                                        uint32_t* __restrict__ hist2, int bits, const PlanScans scans, int plan_tiles) {
    extern __shared__ uint32_t s_hist[];     // [bins]
    const int bins = 1 << bits;
    for (int b = threadIdx.x; b < bins; b += kThreads) s_hist[b] = 0;
    __syncthreads();
    constexpr int kFastItems = TILE / kThreads;
    const int64_t base = (int64_t)blockIdx.x * TILE;
    int32_t v_[kFastItems], e_[kFastItems];
    float t_[kFastItems], tp_[kFastItems];
#pragma unroll
    for (int j = 0; j < kFastItems; ++j) {       // all loads first, clamped to the batch
        const int64_t i = min(base + (int64_t)j * kThreads + threadIdx.x, a.m - 1);
        v_[j] = a.src[i];
        t_[j] = a.ts[i];
        tp_[j] = a.ts[i > 0 ? i - 1 : 0];
        e_[j] = a.eid ? a.eid[i] : 0;
    }
#pragma unroll
    for (int j = 0; j < kFastItems; ++j) {
        const int64_t i = base + (int64_t)j * kThreads + threadIdx.x;
        if (i >= a.m) continue;
        const int32_t v = v_[j];
        const float t = t_[j];
        if ((uint64_t)(uint32_t)v >= (uint64_t)a.num_nodes) report(a.status, TNS_ERANGE, i);
        else if (t != t) report(a.status, TNS_EORDER, i);
        else if (e_[j] < 0) report(a.status, TNS_EINVAL, i);
        if (i > 0 && tp_[j] > t) atomicOr(&a.status->unsorted, 1u);
        atomicAdd(&s_hist[(uint32_t)v & (uint32_t)(bins - 1)], 1u);
    }
    __syncthreads();
    uint32_t* row1 = hist1 + (size_t)blockIdx.x * bins;
    uint32_t* row2 = hist2 + (size_t)blockIdx.x * bins;
    for (int b = threadIdx.x; b < bins; b += kThreads) {
        row1[b] = s_hist[b];
        row2[b] = 0;                      // filled by the first scatter pass
    }
    if (blockIdx.x == 0) {
        // tickets, error words and tile states of the plan's chained scans
        for (int i = threadIdx.x; i < plan_tiles + 1; i += kThreads) {
            for (ScanWorkspace* w : scans.ws) w->status[i] = 0;
        }
        if (threadIdx.x == 0) {
            for (ScanWorkspace* w : scans.ws) {
                w->ticket = 0;
                w->error = 0;
            }
        }
    }
}

// One stable radix pass over `bits` bits of the key starting at `shift`.  A wave owns TILE / 8
// consecutive keys of the tile and takes them 64 at a time in order, so "earlier in the tile" is
// (wave, item, lane) order; a key's rank among equal digits is the count of its wave so far plus its rank
// among the lanes of the current item (ballots over the digit's bits).
// The first pass makes its keys from the batch.
template <int TILE, bool FIRST>
__global__ void __launch_bounds__(kScatThreads) k_fast_scatter(const IngestArgs a, const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                           uint64_t* __restrict__ kout, uint32_t* __restrict__ vout, int64_t m,
                                                           int shift, int bits, int tiles, const uint32_t* __restrict__ hist,
                                                           uint32_t* __restrict__ hist_next, int shift_next) {
    extern __shared__ uint32_t smem[];
    const int bins = 1 << bits;
    uint32_t* s_off = smem;                     // [bins]  position of the tile's first key of each digit
    uint32_t* s_cnt = smem + bins;              // [waves][bins]
    // [2][groups][bins]  parts of the table's sums; with the most bins in the waves' rows, for which there is no more LDS
    const bool apart = bins < 1 << kFastMaxBits;
    uint32_t* s_part = apart ? s_cnt + (size_t)(kScatThreads / kWave) * bins : s_cnt;
    __shared__ int32_t s_wave[16];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    const int tile = blockIdx.x;
    const uint32_t mask = (uint32_t)(bins - 1);

    // the tile's keys are requested first: nothing before the ranking needs them, and they arrive while the table is read
    constexpr int kScatItems = TILE / kScatThreads;
    const int64_t wbase = (int64_t)tile * TILE + (int64_t)wave * (kScatItems * kWave);
    uint64_t k_[kScatItems];
    uint32_t v_[kScatItems], r_[kScatItems];
#pragma unroll
    for (int j = 0; j < kScatItems; ++j) {
        const int64_t i = min(wbase + (int64_t)j * kWave + lane, m - 1);   // clamped: no load sits in a branch
        if (FIRST) {
            k_[j] = ((uint64_t)(uint32_t)a.src[i] << 32) | __float_as_uint(a.ts[i]);
            v_[j] = (uint32_t)i;
        } else {
            k_[j] = kin[i];
            v_[j] = vin[i];
        }
    }
    // keys with this digit in earlier tiles, and in all tiles.  A thread adds up four digits (16-byte loads) of every
    // group-th tile, thirteen rows in flight: the rows come from the L2, and with all 98 rows of a batch of 100 K to itself a
    // thread would spend eight round trips here.  The counts' rows are cleared meanwhile.  (A pass of 10^5 edges, mean of both:
    // 11.8 -> 10.7 us with these, of which the table 3, its sums 1, ranks 1.3, and the keys' places 4 in the first pass, whose counts for
    // the second are atomics, and 1.4 in the second.)
    const int quads = bins / 4, groups = scatter_groups(bins);
    uint32_t* const part_before = s_part;                      // [groups][bins] each
    uint32_t* const part_all = s_part + (size_t)groups * bins;
    auto clear_counts = [&]() {
        for (int i = t; i < bins * (kScatThreads / kWave) / 4; i += kScatThreads) reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0, 0, 0, 0);
    };
    if (apart) clear_counts();
    for (int x = t; x < quads * groups; x += kScatThreads) {
        const int q = x % quads, grp = x / quads;
        uint4 before = make_uint4(0, 0, 0, 0), all = make_uint4(0, 0, 0, 0);
        for (int r0 = grp; r0 < tiles; r0 += kScatRows * groups) {
            uint4 c[kScatRows];
#pragma unroll
            for (int u = 0; u < kScatRows; ++u) c[u] = *reinterpret_cast<const uint4*>(hist + (size_t)min(r0 + u * groups, tiles - 1) * bins + 4 * q);
#pragma unroll
            for (int u = 0; u < kScatRows; ++u) {
                const int r = r0 + u * groups;
                if (r < tiles) { all.x += c[u].x; all.y += c[u].y; all.z += c[u].z; all.w += c[u].w; }
                if (r < tile) { before.x += c[u].x; before.y += c[u].y; before.z += c[u].z; before.w += c[u].w; }
            }
        }
        *reinterpret_cast<uint4*>(part_before + (size_t)grp * bins + 4 * q) = before;
        *reinterpret_cast<uint4*>(part_all + (size_t)grp * bins + 4 * q) = all;
    }
    __syncthreads();
    // thread t owns `per` consecutive digits
    const int per = bins >= kScatThreads ? bins / kScatThreads : 1;
    int32_t mine = 0;
    for (int i = 0; i < per; ++i) {
        const int b = t * per + i;
        if (b >= bins) break;
        uint32_t before = 0, all = 0;
        for (int g = 0; g < groups; ++g) {
            before += part_before[(size_t)g * bins + b];
            all += part_all[(size_t)g * bins + b];
        }
        s_off[b] = before;
        part_all[b] = all;             // the first group's: this thread's alone from here on
        mine += (int32_t)all;
    }
    static_assert(kFastMaxBatch < int64_t(1) << 31, "numbers of keys are 32-bit");
    const int32_t inc = wave_inclusive_scan(mine);
    if (lane == kWave - 1) s_wave[wave] = inc;
    __syncthreads();
    uint32_t run = (uint32_t)(sum_of_waves(s_wave, wave, lane) + inc - mine);       // keys with a smaller digit than this thread's first
    for (int k = 0; k < per; ++k) {
        const int b = t * per + k;
        if (b >= bins) break;
        const uint32_t all = part_all[b];
        s_off[b] += run;
        run += all;
    }
    if (!apart) {
        __syncthreads();
        clear_counts();
        __syncthreads();
    }
    uint32_t* my_cnt = s_cnt + (size_t)wave * bins;
#pragma unroll
    for (int j = 0; j < kScatItems; ++j) {
        const int64_t i = wbase + (int64_t)j * kWave + lane;
        const bool valid = i < m;
        const uint32_t d = (uint32_t)(k_[j] >> shift) & mask;
        uint64_t same = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            same &= bit ? bal : ~bal;
        }
        const int leader = same ? __builtin_ctzll(same) : 0;
        uint32_t prev = 0;
        if (valid && lane == leader) {
            prev = my_cnt[d];
            my_cnt[d] = prev + (uint32_t)__popcll(same);
        }
        prev = (uint32_t)__shfl((int)prev, leader, kWave);
        r_[j] = prev + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    }
    __syncthreads();
    // a wave's keys of a digit follow those of the earlier waves
    for (int b = t; b < bins; b += kScatThreads) {
        uint32_t acc = 0;
#pragma unroll
        for (int w = 0; w < kScatThreads / kWave; ++w) {
            const uint32_t c = s_cnt[(size_t)w * bins + b];
            s_cnt[(size_t)w * bins + b] = acc;
            acc += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kScatItems; ++j) {
        const int64_t i = wbase + (int64_t)j * kWave + lane;
        if (i >= m) continue;
        const uint32_t d = (uint32_t)(k_[j] >> shift) & mask;
        const uint32_t pos = s_off[d] + my_cnt[d] + r_[j];
        if ((int64_t)pos < m) {                 // always true for consistent histograms; keeps a bad one in bounds
            kout[pos] = FIRST ? key_of((int32_t)(k_[j] >> 32), __uint_as_float((uint32_t)k_[j])) : k_[j];
            vout[pos] = v_[j];
            if (FIRST) atomicAdd(&hist_next[(size_t)(pos / TILE) * bins + ((uint32_t)(k_[j] >> shift_next) & mask)], 1u);
        }
    }
}

// Segments, the per-segment plan, and every segment's number and offset into the edge-line and directory pools, in one launch.
// A thread per sorted position; those at a segment's first edge plan it.  Four chained scans run side by side in the first
// four waves: segments and new blocks (at most 2^21 of each in a batch, one in the upper half of the value), edge lines,
// directory records, new slots.  The last tile's sums are the batch's, and it hands the record over without anybody being
// counted in.  What it costs is its chain of dependent reads (position, node, tail of a long list, look-back, record): 10^5
// edges 6.5 us for the segments and 21 for their plan as two launches with atomics for the totals.  512 positions a tile: 256
// and 1024 were both slower somewhere (10^4 edges over 2^16 nodes 54 / 56 / 59 us a batch with 256 / 512 / 1024, 2 * 10^5
// power-law ids 194 / 185 / 184).  32 batches of 10^5 edges, each sampled, into a new store: 3380 -> 2930 us together with
// the table of tile histograms read four rows side by side (k_fast_scatter); with the nodes requested before the segments' lengths
// are known and the apply kernel's edges requested beside their segments, 2860 -> 2570 together with the sampling's smaller launches.
__global__ void __launch_bounds__(kPlanThreads) k_fast_plan(const IngestArgs a, const uint64_t* __restrict__ key,
                                                            int64_t* __restrict__ head_excl, int32_t* __restrict__ seg_start,
                                                            uint32_t* __restrict__ seg_src, SegPlan* __restrict__ plan,
                                                            int64_t* __restrict__ lines_base, int64_t* __restrict__ dir_base,
                                                            const PlanScans scans, int plan_tiles) {
    constexpr int kWaves = kPlanThreads / kWave;
    __shared__ int64_t s_tile, s_excl[kPlanScans], s_sum[kPlanScans][kWaves];
    __shared__ int32_t s_heads[kWaves], s_end;
    __shared__ int32_t s_start[kPlanThreads + 1];
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
    // tiles are numbered in the order workgroups start: other work can hold an XCD for any time, and a tile must not wait for one
    // that has not started (a ticket is an atomic on one word, 18 ns each)
    if (t == 0) s_tile = (int64_t)atomicAdd(&scans.ws[0]->ticket, 1u);
    __syncthreads();
    const int64_t tile = s_tile, p0 = tile * kPlanThreads, p = p0 + t;
    const uint64_t k = p < a.m ? key[p] : 0, before = p > 0 && p < a.m ? key[p - 1] : 0;
    const bool head = p < a.m && (p == 0 || (uint32_t)(k >> 32) != (uint32_t)(before >> 32));
    SegNode node{};
    if (head) {
        load_node(a, (uint32_t)(k >> 32), node);
        node.t_first = time_of_key((uint32_t)k);       // (only compared: a zero's sign does not matter)
    }
    if (wave == kWaves - 1) {
        // where the tile's last segment ends: beyond the tile by at most a batch, found 64 positions at a time
        int64_t lo = min(p0 + kPlanThreads, a.m), n = a.m - lo;
        const uint32_t last = (uint32_t)(key[lo - 1] >> 32);
        while (n > 0) {
            // the first 64 positions in the first round (most segments are short), then 64-way
            const int64_t s = lo == p0 + kPlanThreads && n > kWave ? 1 : (n + kWave - 1) / kWave;
            const int64_t at = lo + min((int64_t)(lane + 1) * s - 1, n - 1);
            const int cnt = __popcll(__ballot((uint32_t)(key[at] >> 32) == last));
            const int64_t step = min((int64_t)cnt * s, n);
            lo += step;
            n = cnt == kWave ? n - step : max(min(s - 1, n - step), (int64_t)0);
        }
        if (lane == 0) s_end = (int32_t)lo;
    }
    const uint64_t heads = __ballot(head);
    if (lane == 0) s_heads[wave] = __popcll(heads);
    __syncthreads();
    int32_t local = __popcll(heads & ((1ull << lane) - 1ull)), num_heads = 0;       // heads of the tile before this position
    for (int w = 0; w < kWaves; ++w) {
        const int32_t c = s_heads[w];
        if (w < wave) local += c;
        num_heads += c;
    }
    if (head) s_start[local] = (int32_t)p;
    if (t == 0) s_start[num_heads] = s_end;
    __syncthreads();
    SegPlan P{};
    int64_t lines = 0, dirs = 0, blocks = 0, slots = 0;
    if (head) plan_segment(a, (uint32_t)(k >> 32), node, s_start[local + 1] - p, P, lines, dirs, blocks, slots,
                           [&]() { report(a.status, TNS_EORDER, a.m + (int64_t)(k >> 32)); });
    // exclusive sums of the scans' values over the workgroup
    int64_t v[kPlanScans] = {((int64_t)(head ? 1 : 0) << 32) | blocks, lines, dirs, slots}, total[kPlanScans];
#pragma unroll
    for (int i = 0; i < kPlanScans; ++i) {
        const int64_t own = v[i];
        v[i] = wave_inclusive_scan64(own);
        if (lane == kWave - 1) s_sum[i][wave] = v[i];
        v[i] -= own;
    }
    wait_for_memory();               // this thread's reports have been performed before its tile's totals are published
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPlanScans; ++i) {
        total[i] = 0;
        for (int w = 0; w < kWaves; ++w) {
            const int64_t x = s_sum[i][w];
            if (w < wave) v[i] += x;
            total[i] += x;
        }
    }
    if (wave < kPlanScans) {
        const int64_t excl = chain_wave(scans.ws[wave], a.status, tile,
                                        wave == 0 ? total[0] : (wave == 1 ? total[1] : (wave == 2 ? total[2] : total[3])), lane);
        if (lane == 0) s_excl[wave] = excl;
        wait_for_memory();           // a time-out's report likewise
    }
    __syncthreads();
    const int64_t seg = (v[0] + s_excl[0]) >> 32;
    if (p < a.m) head_excl[p] = seg;
    // (after a chained scan's time-out the sums are short and nothing is applied: the stores stay within the batch)
    if (head && seg < a.m) {
        seg_start[seg] = (int32_t)p;
        seg_src[seg] = (uint32_t)(k >> 32);
        plan[seg] = P;
        lines_base[seg] = v[1] + s_excl[1];
        dir_base[seg] = v[2] + s_excl[2];
    }
    if (tile == plan_tiles - 1 && t == 0) {
        // every earlier tile has published, and reported what it had to before that: the record is complete
        const int64_t nseg = (s_excl[0] + total[0]) >> 32;
        if (nseg <= a.m) seg_start[nseg] = (int32_t)a.m;
        IngestStatus rec = load_status(a.status);
        rec.num_segments = nseg;
        rec.total_lines = s_excl[1] + total[1];
        rec.total_dir = s_excl[2] + total[2];
        rec.new_blocks = (unsigned long long)((s_excl[0] + total[0]) & 0xffffffffll);
        rec.new_slots = (unsigned long long)(s_excl[3] + total[3]);
        IngestStatus* st = a.status;
        st->num_segments = rec.num_segments;
        st->total_lines = rec.total_lines;
        st->total_dir = rec.total_dir;
        st->new_blocks = rec.new_blocks;
        st->new_slots = rec.new_slots;
        if (a.host_status) hand_over(a, rec);
    }
}

// A batch of at most kSmallBatch edges (a mini-batch of a stream), planned and applied by one workgroup: such a batch
// spends its time in dependent launches otherwise.  Everything between the batch and the store stays in LDS, the batch's times and
// errors among it; the record goes to the host while the store is being changed.  Sorted by (source, arrival) with a stable radix
// sort, up to nine bits a pass: a wave ranks 128 keys with ballots, and the counts of a pass are scanned by all threads.
// What bounds it is one workgroup's chain of steps: keys, passes, segments, plans, record, nodes, edges.  So a thread's two edges and
// two segments have their reads requested together and what the plan has read of a node is kept for its change; sums over lanes are
// vector instructions and not shuffles.  Batch of 2000 power-law edges over 2^16 nodes, us from the start: sorted 8.0 -> 7.6, planned 14.4 ->
// 13.9, record on its way 17.1 -> 15.2, done 26.4 -> 22.4, in a stream of batches 25.9 -> 21.1; before that, as a bitonic network of 66 steps, the sort alone took 13.5.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / kWave, kSmallItems = (int)kSmallBatch / kSmallThreads;
constexpr int kSender = kSmallThreads - kWave;                             // whose wave has fewest segments: hands the record over
constexpr int kSmallDigitLeast = 6, kSmallDigitMost = 9;                 // bits a pass (six: a count per thread)
struct SmallShared {
    uint64_t key[kSmallBatch];           // sorted: source in the high word, batch position in the low one
    float ts[kSmallBatch];               // by batch position
    union {
        SegPlan plan[kSmallBatch];
        int32_t count[(1 << kSmallDigitMost) * (kSmallWaves + 1)];      // of a sorting pass: [digit][wave], a word of padding per digit
    };
    int64_t lines_base[kSmallBatch], dir_base[kSmallBatch];
    int32_t seg_start[kSmallBatch + 1];
    int32_t seg_of[kSmallBatch];
    int64_t wave[4][kSmallWaves];        // edge lines, directory records, blocks, slots
    int32_t wave32[kSmallWaves];
    unsigned long long err_word;         // as in IngestStatus
    uint32_t unsorted;
    int32_t go;
};
static_assert(sizeof(SmallShared) <= 160 << 10, "one workgroup's LDS");
struct SmallBatch {                      // as PlannedBatch, in LDS
    static constexpr bool kAhead = false;
    const SmallShared& sh;
    const SegPlan* plan;
    const int32_t* seg_start;
    const int64_t *lines_base, *dir_base;
    __device__ __forceinline__ explicit SmallBatch(const SmallShared& x)
        : sh(x), plan(x.plan), seg_start(x.seg_start), lines_base(x.lines_base), dir_base(x.dir_base) {}
    __device__ __forceinline__ uint32_t source(int64_t p) const { return (uint32_t)(sh.key[p] >> 32); }
    __device__ __forceinline__ uint32_t position(int64_t p) const { return (uint32_t)sh.key[p]; }
    __device__ __forceinline__ float time(const IngestArgs&, int64_t p) const { return sh.ts[position(p)]; }
    __device__ __forceinline__ SegTimes times(const IngestArgs& a, const int32_t (&p)[3]) const {
        return SegTimes{time(a, p[0]), time(a, p[1]), time(a, p[2])};
    }
};

// digit: bits a pass
__global__ void __launch_bounds__(kSmallThreads) k_small_batch(const IngestArgs a, int bits, int digit, uint64_t* __restrict__ key,
                                                               uint32_t* __restrict__ val, int64_t* __restrict__ head_excl,
                                                               int32_t* __restrict__ seg_start, uint32_t* __restrict__ seg_src,
                                                               SegPlan* __restrict__ plan, int64_t* __restrict__ lines_base,
                                                               int64_t* __restrict__ dir_base) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    SmallShared& sh = *reinterpret_cast<SmallShared*>(s_raw);
    const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave, m = (int)a.m;
    // a wave owns kSmallItems * 64 consecutive keys, item by item; the items' reads are requested together
    uint64_t k[kSmallItems];
    int32_t v[kSmallItems], e[kSmallItems], touched[2 * kSmallItems];
    float ts[kSmallItems], before[kSmallItems];
    IngestStatus rec{};
    if (t == kSender) {
        sh.err_word = ~0ull;
        sh.unsorted = 0;
        rec.internal = a.status->internal;         // (what earlier launches have left; this batch's own errors are in LDS)
    }
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
        const int i = min((wave * kSmallItems + j) * kWave + lane, m - 1);
        v[j] = a.src[i];
        ts[j] = a.ts[i];
        before[j] = a.ts[i > 0 ? i - 1 : 0];
        e[j] = a.eid ? a.eid[i] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
        // brings the node's entry and builder state into the L2 while the keys are sorted
        const int64_t nidx = a.node_base + ((uint64_t)(uint32_t)v[j] < (uint64_t)a.num_nodes ? v[j] : 0);
        touched[2 * j] = a.nodes[nidx].nblocks;
        touched[2 * j + 1] = a.aux[nidx].tail_cap;
    }
    auto report_here = [&](int status, int64_t pos) { atomicMin(&sh.err_word, ((unsigned long long)pos << 8) | (unsigned long long)(-status)); };
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
        const int i = (wave * kSmallItems + j) * kWave + lane;
        k[j] = ~0ull;                    // beyond the batch: last in every pass
        if (i < m) {
            if ((uint64_t)(uint32_t)v[j] >= (uint64_t)a.num_nodes) report_here(TNS_ERANGE, i);
            else if (ts[j] != ts[j]) report_here(TNS_EORDER, i);
            else if (e[j] < 0) report_here(TNS_EINVAL, i);
            if (i > 0 && before[j] > ts[j]) sh.unsorted = 1;
            k[j] = ((uint64_t)(uint32_t)v[j] << 32) | (uint32_t)i;
            sh.ts[i] = ts[j];
        }
    }
    const int bins = 1 << digit, per = bins * kSmallWaves / kSmallThreads;      // counts per thread
    uint32_t to[kSmallItems];
#pragma unroll 1
    for (int shift = 0; shift < bits; shift += digit) {
        // rank among the wave's equal digits: those of earlier items, then those of lower lanes
        for (int i = lane; i < bins; i += kWave) sh.count[i * (kSmallWaves + 1) + wave] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t d[kSmallItems], rank[kSmallItems];
        uint64_t same[kSmallItems];
#pragma unroll
        for (int j = 0; j < kSmallItems; ++j) {
            d[j] = (uint32_t)(k[j] >> (32 + shift)) & (uint32_t)(bins - 1);
            same[j] = ~0ull;
        }
        for (int b = 0; b < digit; ++b) {
#pragma unroll
            for (int j = 0; j < kSmallItems; ++j) {
                const bool bit = (d[j] >> b) & 1u;
                const uint64_t bal = __ballot(bit);
                same[j] &= bit ? bal : ~bal;
            }
        }
#pragma unroll
        for (int j = 0; j < kSmallItems; ++j) {
            int32_t* const c = &sh.count[d[j] * (kSmallWaves + 1) + wave];
            const uint32_t earlier = (uint32_t)*c, lower = (uint32_t)__popcll(same[j] & ((1ull << lane) - 1ull));
            rank[j] = earlier + lower;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (lower == 0) *c = (int32_t)(earlier + (uint32_t)__popcll(same[j]));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // exclusive scan of the counts, digit by digit and wave by wave: `per` consecutive ones per thread
        int32_t own = 0;
        for (int i = 0; i < per; ++i) {
            const int c = t * per + i;
            own += sh.count[c / kSmallWaves * (kSmallWaves + 1) + c % kSmallWaves];
        }
        const int32_t inc = wave_inclusive_scan(own);
        if (lane == kWave - 1) sh.wave32[wave] = inc;
        __syncthreads();
        int32_t run = sum_of_waves(sh.wave32, wave, lane) + inc - own;
        for (int i = 0; i < per; ++i) {
            const int c = t * per + i;
            int32_t* const at = &sh.count[c / kSmallWaves * (kSmallWaves + 1) + c % kSmallWaves];
            const int32_t n = *at;
            *at = run;
            run += n;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSmallItems; ++j) to[j] = (uint32_t)sh.count[d[j] * (kSmallWaves + 1) + wave] + rank[j];
#pragma unroll
        for (int j = 0; j < kSmallItems; ++j) sh.key[to[j]] = k[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSmallItems; ++j) k[j] = sh.key[(wave * kSmallItems + j) * kWave + lane];
    }
#pragma unroll
    for (int j = 0; j < 2 * kSmallItems; ++j) asm volatile("" ::"v"(touched[j]));          // the loads' only use
    // segments; every item of a wave is 64 consecutive sorted positions
    int h[kSmallItems];
    uint64_t heads[kSmallItems];
    int32_t in_wave = 0;
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
        const int p = (wave * kSmallItems + j) * kWave + lane;
        h[j] = p < m && (p == 0 || (uint32_t)(sh.key[max(p - 1, 0)] >> 32) != (uint32_t)(k[j] >> 32)) ? 1 : 0;
        heads[j] = __ballot(h[j]);
        in_wave += __popcll(heads[j]);
    }
    if (lane == 0) sh.wave32[wave] = in_wave;
    __syncthreads();
    int32_t run = sum_of_waves(sh.wave32, wave, lane);
    const int32_t nseg = sum_of_waves(sh.wave32, kSmallWaves, lane);
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
        const int p = (wave * kSmallItems + j) * kWave + lane;
        const int32_t s = run + __popcll(heads[j] & ((1ull << lane) - 1ull));       // heads before this position
        if (p < m) {
            sh.seg_of[p] = s + h[j] - 1;
            if (h[j]) sh.seg_start[s] = p;
            if (p == m - 1) sh.seg_start[nseg] = m;
        }
        run += __popcll(heads[j]);
    }
    __syncthreads();
    // plans, 1024 segments at a time (a loop, not unrolled: the program is fetched once from a cold instruction cache,
    // and its length is part of what this kernel costs); what is read of all the nodes is requested first
    SegNode node[kSmallItems] = {};
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
        const int sgm = t + j * kSmallThreads;
        if (sgm < nseg) {
            const uint64_t k0 = sh.key[sh.seg_start[sgm]];
            load_node(a, (uint32_t)(k0 >> 32), node[j]);
            node[j].t_first = sh.ts[(uint32_t)k0];
        }
    }
    static_assert(kSmallItems == 2, "the loops take one node or the other");
    EdgeWords edge[kSmallItems] = {};      // on their way while the nodes are planned
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j)
        if (t + j * kSmallThreads < m) edge[j] = load_edge(a, (uint32_t)sh.key[t + j * kSmallThreads]);
    int64_t all[4] = {0, 0, 0, 0};
#pragma unroll 1
    for (int sgm = t; sgm - t < nseg; sgm += kSmallThreads) {
        int64_t need[4] = {0, 0, 0, 0};
        if (sgm < nseg) {
            const SegNode n = sgm == t ? node[0] : node[1];
            const int p0 = sh.seg_start[sgm];
            const uint32_t source = (uint32_t)(sh.key[p0] >> 32);
            SegPlan P{};
            plan_segment(a, source, n, sh.seg_start[sgm + 1] - p0, P, need[0], need[1], need[2], need[3],
                         [&]() { report_here(TNS_EORDER, a.m + (int64_t)source); });
            sh.plan[sgm] = P;
        }
        const bool some = __ballot(sgm < nseg) != 0;        // (waves without a segment leave the sums out)
        int64_t inc[4] = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (some) inc[i] = wave_inclusive_scan64(need[i]);
            if (lane == kWave - 1) sh.wave[i][wave] = inc[i];
        }
        __syncthreads();
        if (some) {
            const int64_t lines_before = sum_of_waves64(sh.wave[0], wave, lane), dir_before = sum_of_waves64(sh.wave[1], wave, lane);
            if (sgm < nseg) {
                sh.lines_base[sgm] = all[0] + lines_before + inc[0] - need[0];
                sh.dir_base[sgm] = all[1] + dir_before + inc[1] - need[1];
            }
        }
        if (wave == kSmallWaves - 1 || sgm - t + kSmallThreads < nseg) {
#pragma unroll
            for (int i = 0; i < 4; ++i) all[i] += sum_of_waves64(sh.wave[i], kSmallWaves, lane);      // (for the next segments, and the record)
        }
        __syncthreads();
    }
    if (t == kSender) {
        rec.err_word = sh.err_word;
        rec.unsorted = sh.unsorted;
        rec.num_segments = nseg;
        rec.total_lines = all[0];
        rec.total_dir = all[1];
        rec.new_blocks = (unsigned long long)all[2];
        rec.new_slots = (unsigned long long)all[3];
        sh.go = a.host_status && ingest_may_apply(rec, a) ? 1 : 0;
    }
    __syncthreads();
    const bool go = sh.go != 0;
    if (t == kSender) {
        IngestStatus* st = a.status;
        if (go) {
            ready_status(st);
        } else {
            *st = rec;
            __threadfence();
        }
        if (a.host_status) send_to_host(a, rec);
    }
    const SmallBatch batch(sh);
    if (go) {
#pragma unroll 1
        for (int s = t; s < nseg; s += kSmallThreads) {
            const SegNode n = s == t ? node[0] : node[1];
            const SegPlan P = sh.plan[s];
            const int32_t p0 = sh.seg_start[s], p1 = sh.seg_start[s + 1];
            const int64_t nidx = a.node_base + batch.source(p0);
            apply_node(a, batch, s, P, p0, p1, nidx, n, OlderRecs{}, segment_times(a, batch, P, p0, p1));
        }
#pragma unroll 1
        for (int p = t; p < m; p += kSmallThreads) {
            const int32_t sgm = sh.seg_of[p];
            apply_edge(a, sh.plan[sgm], p - sh.seg_start[sgm], sh.lines_base[sgm], edge[0]);
            edge[0] = edge[1];
        }
    } else {
        // an error, a batch out of order, pools without room: the host decides, and a later launch finds the plan in memory
#pragma unroll 1
        for (int p = t; p < m; p += kSmallThreads) {
            key[p] = key_of((int32_t)batch.source(p), batch.time(a, p));
            val[p] = batch.position(p);
            head_excl[p] = sh.seg_of[p] + ((p == sh.seg_start[sh.seg_of[p]]) ? 0 : 1);
        }
#pragma unroll 1
        for (int s = t; s < nseg; s += kSmallThreads) {
            plan[s] = sh.plan[s];
            seg_start[s] = sh.seg_start[s];
            seg_src[s] = batch.source(sh.seg_start[s]);
            lines_base[s] = sh.lines_base[s];
            dir_base[s] = sh.dir_base[s];
            if (s == nseg - 1) seg_start[nseg] = m;
        }
    }
}

// ---- deletion, statistics ------------------------------------------------------------------

__global__ void __launch_bounds__(kThreads) k_delete_edges(NodeLine* nodes, BlockRec* dir, uint32_t* lines, int64_t node_base,
                                                           const int32_t* __restrict__ src, const int32_t* __restrict__ eid, int64_t n,
                                                           IngestStatus* st) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    NodeLine* N = &nodes[node_base + src[i]];
    const int32_t e = eid[i];
    const int32_t nb = N->nblocks;
    unsigned long long hits = 0;
    for (int32_t b = 0; b < nb; ++b) {
        BlockRec* r = nb <= kInlineBlocks ? &N->rec[b] : &dir[(int64_t)N->dir_line * kDirAlign + b];
        const int64_t off = rec_off(*r);
        const int32_t size = rec_size(*r);
        bool here = false;
        for (int32_t k = 0; k < size; ++k) {
            uint32_t* w = &lines[slot_word(off + k) + 2];
            // only one of several requests for the same edge gets the hit
            if (*w == (uint32_t)e && atomicCAS(w, (uint32_t)e, ~(uint32_t)e) == (uint32_t)e) {
                here = true;
                ++hits;
            }
        }
        if (here) atomicOr(&r->size_hi, 0x80000000u);
    }
    if (hits) {
        atomicOr(reinterpret_cast<unsigned int*>(&N->flags), 2u);
        atomicAdd(&st->counter, hits);
    }
}

__global__ void __launch_bounds__(kThreads) k_delete_nodes(NodeLine* nodes, int64_t node_base, const int32_t* __restrict__ ids, int64_t n,
                                                           int32_t deleted) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    unsigned int* f = reinterpret_cast<unsigned int*>(&nodes[node_base + ids[i]].flags);
    if (deleted) atomicOr(f, 1u); else atomicAnd(f, ~1u);
}

__global__ void __launch_bounds__(kThreads) k_max_list_len(const NodeLine* __restrict__ nodes, int64_t first, int64_t count,
                                                           IngestStatus* st) {
    int64_t mx = 0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < count; i += (int64_t)gridDim.x * kThreads)
        mx = max(mx, (int64_t)nodes[first + i].nblocks);
    for (int d = 32; d >= 1; d >>= 1) mx = max(mx, (int64_t)__shfl_xor((long long)mx, d, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0 && mx > 0) atomicMax(&st->counter, (unsigned long long)mx);
}

// ---- workspace -----------------------------------------------------------------------------

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

struct Carve {
    uint64_t *keyA, *keyB;
    uint32_t *valA, *valB, *hist;
    int64_t *head_excl, *lines_base, *dir_base, *sums;
    int32_t* seg_start;
    uint32_t* seg_src;
    SegPlan* plan;
    int64_t chunk;
    int nblk;
    // short pipeline (batches of at most kFastMaxBatch edges)
    uint32_t* tile_hist[2];        // [tiles][bins] per radix pass
    PlanScans scans;
    int fast_tiles, plan_tiles;
    size_t bytes;
};

Carve carve(void* ws, int64_t m) {
    Carve c{};
    // sort chunks: at least 2048 keys and at most 1024 chunks
    c.chunk = std::max<int64_t>(2048, ((m + 1023) / 1024 + kThreads - 1) / kThreads * kThreads);
    c.nblk = (int)std::max<int64_t>(1, (m + c.chunk - 1) / c.chunk);
    unsigned char* p = static_cast<unsigned char*>(ws);
    size_t o = 0;
    auto take = [&](size_t bytes) { unsigned char* r = p ? p + o : nullptr; o += align256(bytes); return r; };
    const size_t mm = (size_t)std::max<int64_t>(m, 1);
    c.keyA = reinterpret_cast<uint64_t*>(take(mm * 8));
    c.keyB = reinterpret_cast<uint64_t*>(take(mm * 8));
    c.valA = reinterpret_cast<uint32_t*>(take(mm * 4));
    c.valB = reinterpret_cast<uint32_t*>(take(mm * 4));
    c.hist = reinterpret_cast<uint32_t*>(take((size_t)256 * c.nblk * 4));
    c.head_excl = reinterpret_cast<int64_t*>(take(mm * 8));
    c.lines_base = reinterpret_cast<int64_t*>(take(mm * 8));
    c.dir_base = reinterpret_cast<int64_t*>(take(mm * 8));
    c.sums = reinterpret_cast<int64_t*>(take(((mm + kScanTile - 1) / kScanTile + 1) * 8));
    c.seg_start = reinterpret_cast<int32_t*>(take((mm + 1) * 4));
    c.seg_src = reinterpret_cast<uint32_t*>(take(mm * 4));
    c.plan = reinterpret_cast<SegPlan*>(take(mm * sizeof(SegPlan)));
    if (m <= kFastMaxBatch) {
        c.fast_tiles = (int)((mm + fast_tile_keys(m) - 1) / fast_tile_keys(m));
        c.plan_tiles = (int)((mm + kPlanThreads - 1) / kPlanThreads);
        for (int p2 = 0; p2 < 2; ++p2)
            c.tile_hist[p2] = reinterpret_cast<uint32_t*>(take((size_t)c.fast_tiles * (size_t(1) << kFastMaxBits) * 4));
        for (ScanWorkspace*& w : c.scans.ws)
            w = reinterpret_cast<ScanWorkspace*>(take(sizeof(ScanWorkspace) + (size_t)(c.plan_tiles + 1) * 8));
    }
    c.bytes = o;
    return c;
}

int src_passes(int64_t num_nodes) {
    int bits = 0;
    while (bits < 32 && (int64_t(1) << bits) < num_nodes) ++bits;
    return (bits + 7) / 8;
}

unsigned grid_for(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + kThreads - 1) / kThreads); }

}  // namespace

size_t ingest_workspace_bytes(int64_t m) { return carve(nullptr, m).bytes; }

hipError_t ingest_status_reset(IngestStatus* status, hipStream_t stream) {
    hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(64), 0, stream, status);
    return hipGetLastError();
}

hipError_t ingest_plan(const IngestArgs& a, hipStream_t stream) {
    if (a.m <= 0 || a.m > kMaxDeviceBatch) return hipErrorInvalidValue;
    const Carve c = carve(a.workspace, a.m);
    const int64_t m = a.m;
    hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(64), 0, stream, a.status);
    hipLaunchKernelGGL(k_keys, dim3(grid_for(m)), dim3(kThreads), 0, stream, a, c.keyA, c.valA);
    // least significant digit first: 4 passes over the time bits (an even number, so a skipped
    // group leaves the data where it is), then the passes over the source id
    uint64_t *kin = c.keyA, *kout = c.keyB;
    uint32_t *vin = c.valA, *vout = c.valB;
    const int passes = 4 + src_passes(a.num_nodes);
    for (int p = 0; p < passes; ++p) {
        const int skippable = p < 4 ? 1 : 0;
        hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)c.nblk), dim3(kThreads), 0, stream, kin, m, 8 * p, c.chunk, c.nblk, c.hist,
                           a.status, skippable);
        hipLaunchKernelGGL(k_radix_scan, dim3(1), dim3(1024), 0, stream, c.hist, (int64_t)256 * c.nblk, a.status, skippable);
        hipLaunchKernelGGL(k_radix_scatter, dim3((unsigned)c.nblk), dim3(kThreads), 0, stream, kin, vin, kout, vout, m, 8 * p,
                           c.chunk, c.nblk, c.hist, a.status, skippable);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    // kin / vin now name the sorted arrays
    hipLaunchKernelGGL(k_heads, dim3(grid_for(m)), dim3(kThreads), 0, stream, kin, m, c.head_excl);
    hipError_t e = exclusive_scan64(c.head_excl, c.head_excl, m, c.sums, &a.status->num_segments, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_seg_start, dim3(grid_for(m)), dim3(kThreads), 0, stream, kin, m, c.head_excl, c.seg_start);
    hipLaunchKernelGGL(k_plan, dim3(grid_for(m)), dim3(kThreads), 0, stream, a, kin, vin, c.seg_start, c.seg_src, c.plan, c.lines_base,
                       c.dir_base);
    e = exclusive_scan64(c.lines_base, c.lines_base, m, c.sums, &a.status->total_lines, stream);
    if (e != hipSuccess) return e;
    return exclusive_scan64(c.dir_base, c.dir_base, m, c.sums, &a.status->total_dir, stream);
}

// Bits per digit of the short pipeline's two radix passes, or 0 if the batch does not qualify.
int fast_digit_bits(int64_t m, int64_t num_nodes) {
    if (m > kFastMaxBatch) return 0;
    int bits = 0;
    while (bits < 32 && (int64_t(1) << bits) < num_nodes) ++bits;
    if (bits > 2 * kFastMaxBits) return 0;
    return std::max(2, (bits + 1) / 2);            // (at least four bins: a table row is read 16 bytes at a time)
}

bool ingest_fast_ok(int64_t m, int64_t num_nodes) { return fast_digit_bits(m, num_nodes) > 0; }

hipError_t ingest_plan_fast(const IngestArgs& args, hipStream_t stream) {
    const int bits = fast_digit_bits(args.m, args.num_nodes);
    if (args.m <= 0 || bits <= 0) return hipErrorInvalidValue;
    const Carve c = carve(args.workspace, args.m);
    IngestArgs a = args;
    a.go = c.sums;
    if (a.m <= kSmallBatch) {
        const int passes = (2 * bits + kSmallDigitMost - 1) / kSmallDigitMost, digit = std::max(kSmallDigitLeast, (2 * bits + passes - 1) / passes);
        hipLaunchKernelGGL(k_small_batch, dim3(1), dim3(kSmallThreads), sizeof(SmallShared), stream, a, 2 * bits, digit, c.keyA, c.valA, c.head_excl,
                           c.seg_start, c.seg_src, c.plan, c.lines_base, c.dir_base);
        return hipGetLastError();
    }
    const int bins = 1 << bits;
    const size_t lds = (size_t)bins * 4 * (1 + kScatThreads / kWave + (bins < 1 << kFastMaxBits ? 2 * scatter_groups(bins) : 0));
#define TNS_FAST_SORT(TILE)                                                                                                          \
    do {                                                                                                                             \
        hipLaunchKernelGGL((k_fast_keys<TILE>), dim3((unsigned)c.fast_tiles), dim3(kThreads), (size_t)bins * 4, stream, a,          \
                           c.tile_hist[0], c.tile_hist[1], bits, c.scans, c.plan_tiles);                                             \
        hipLaunchKernelGGL((k_fast_scatter<TILE, true>), dim3((unsigned)c.fast_tiles), dim3(kScatThreads), lds, stream, a,           \
                           (const uint64_t*)nullptr, (const uint32_t*)nullptr, c.keyB, c.valB, a.m, 32, bits, c.fast_tiles, c.tile_hist[0], c.tile_hist[1], 32 + bits);                  \
        hipLaunchKernelGGL((k_fast_scatter<TILE, false>), dim3((unsigned)c.fast_tiles), dim3(kScatThreads), lds, stream, a, c.keyB,   \
                           c.valB, c.keyA, c.valA, a.m, 32 + bits, bits, c.fast_tiles, c.tile_hist[1], (uint32_t*)nullptr, 0);               \
    } while (0)
    switch (fast_tile_keys(a.m)) {
        case 1024: TNS_FAST_SORT(1024); break;
        case 2048: TNS_FAST_SORT(2048); break;
        default: TNS_FAST_SORT(kFastTileMax); break;
    }
#undef TNS_FAST_SORT
    hipLaunchKernelGGL(k_fast_plan, dim3((unsigned)c.plan_tiles), dim3(kPlanThreads), 0, stream, a, c.keyA, c.head_excl, c.seg_start,
                       c.seg_src, c.plan, c.lines_base, c.dir_base, c.scans, c.plan_tiles);
    return hipGetLastError();
}

hipError_t ingest_apply(const IngestArgs& a, int64_t num_segments, bool fast, hipStream_t stream) {
    if (a.m <= 0 || num_segments > a.m) return hipErrorInvalidValue;
    const Carve c = carve(a.workspace, a.m);
    const bool in_b = !fast && (src_passes(a.num_nodes) & 1) != 0;
    const uint64_t* key = in_b ? c.keyB : c.keyA;
    const uint32_t* val = in_b ? c.valB : c.valA;
    if (num_segments <= 0 && a.m <= kSmallBatch) return hipSuccess;          // k_small_batch has applied the batch, or may not
    const unsigned node_blocks = grid_for(num_segments > 0 ? num_segments : a.m);
    const PlannedBatch b{key, val, c.head_excl, c.seg_start, c.seg_src, c.plan, c.lines_base, c.dir_base};
    hipLaunchKernelGGL(k_apply, dim3(node_blocks + grid_for(a.m)), dim3(kThreads), 0, stream, a, b, num_segments, node_blocks,
                       num_segments > 0 ? nullptr : c.sums);
    return hipGetLastError();
}

hipError_t ingest_delete_edges(NodeLine* nodes, BlockRec* dir, uint32_t* lines, int64_t node_base, const int32_t* src,
                               const int32_t* eid, int64_t n, IngestStatus* status, hipStream_t stream) {
    hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(64), 0, stream, status);
    if (n > 0)
        hipLaunchKernelGGL(k_delete_edges, dim3(grid_for(n)), dim3(kThreads), 0, stream, nodes, dir, lines, node_base, src, eid, n,
                           status);
    return hipGetLastError();
}

hipError_t ingest_delete_nodes(NodeLine* nodes, int64_t node_base, const int32_t* ids, int64_t n, int32_t deleted,
                               hipStream_t stream) {
    if (n > 0) hipLaunchKernelGGL(k_delete_nodes, dim3(grid_for(n)), dim3(kThreads), 0, stream, nodes, node_base, ids, n, deleted);
    return hipGetLastError();
}

hipError_t ingest_max_list_len(const NodeLine* nodes, int64_t first, int64_t count, IngestStatus* status, hipStream_t stream) {
    hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(64), 0, stream, status);
    if (count > 0) {
        const unsigned grid = (unsigned)std::min<int64_t>(4096, (count + kThreads - 1) / kThreads);
        hipLaunchKernelGGL(k_max_list_len, dim3(grid), dim3(kThreads), 0, stream, nodes, first, count, status);
    }
    return hipGetLastError();
}

}  // namespace tns
