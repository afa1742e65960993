// gfx950 sampling kernel for the recent policy, batches that fill the chip, over the default layout, and batches of any size over
// the prefix layout: Algorithm 1 of the paper (section 4.2), the padded write, and the padding removal of section 5 fused in
// when the dense outputs are wanted.
//
// One query per lane, as in tns_kernels.hip (64 independent chains of dependent reads per wave).  What paces the kernel is
// the length of a wave's program, not the memory: time stamps in the kernel before this one, for 2^16 queries over each of 256
// graphs with a window, gave 3.4 us for the node lines and 9.9 for the searches, the positions and the waits between them, and
// 7 of every 27 us a wave spent waiting for the slowest one of its tile.  So the steps are arranged to be short and free of
// waits on one another:
//   node      the wave fetches the 128-byte node lines together, eight lanes per line, and hands them over through LDS
//   blocks    each lane finds, among its up to seven records in registers, the blocks that count as a whole, the one with
//             the window's end and the one with its start
//   search    the lanes that have such a block ask for its timestamps; requests of both kinds are numbered over the wave
//             and served together, sixteen lanes per request and 32 requests in flight, so that steps nobody needs cost
//             nothing and a window costs no second round trip
//   table     each lane leaves in LDS, per block, where its newest candidate lies, and the number of candidates before each
//             block packed into bytes: nothing per slot and no loop over slots
//   gather    lane l takes flat slot it * 64 + l of the wave's 64 f slots, finds the slot's block by comparing all bytes
//             at once, and loads the edge; five such loads are prepared side by side
// (Only loads that have a request are issued, and the queries are requested before their instance is searched for: 2^23 queries
// 688 -> 668 us windowed, 728 -> 713 without, 2^26 6235 -> 6200.)
// Against the kernel in which every lane wrote its slots' positions itself, after two rounds of searches for all 64 queries:
// 256 graphs of 2^16 queries, windowed, 1737 -> 1502 us; 2^22 queries over uniform ids 426 -> 372; 2^26 6624 -> 6236.
// Prefix layout: the lines of a node's prefix are blocks like any other (the node's own line, whose times the lane has, and up to
// three extension lines indexed by the fences), and up to three blocks outside the prefix are read from the directory beside
// them.  The kernel before, in which the lines' requests were served by ten lanes each and every edge was written to a result row
// in LDS, issued 1900 vector instructions per wave and sent every node with a block outside the prefix on the walk, which held up
// its whole tile: two hops from 2^20 roots, windowed, dense rows only 533 -> 402 us, 10^6 queries 122 -> 96, 2^22 412 -> 340, 2^26 5990
// -> 5530, 10^5 25.5 -> 15.  Node lines are read without the non-temporal hint, as the gather comes back for their edges (with it
// 419, 110 and 6070 us).
// Nodes with long lists (directory runs) or with deleted edges take the walk of Algorithm 1 lane by lane instead; their
// row of the table holds one entry per slot.
#include <algorithm>
#include <type_traits>

#include "tns_device.h"
#include "tns_kernels.h"

namespace tns {
namespace {

constexpr int kPrefixBigBlocks = kInlineBlocks - 1 - kPrefixExtLines;      // blocks outside the prefix that a lane holds like inline ones
constexpr int kRequestBatch = 8;                                   // search loads in flight: 32 requests
constexpr int kGroups = kWave / kCoopGroup;                        // requests per search load
constexpr uint32_t kFlagBytes = 0x00404040u;                       // the bytes of the packed counts, and their compare bit

// What the gathering lanes need to know about a query.  Byte i - 1 of `lo` (i = 1..3) and i - 4 of `hi` (i = 4..6): 64
// minus the candidates before block i (at most 64): added to a slot number of 0..63 it reaches 64 where the slot lies in
// block i or an older one.  Top byte of `lo`: filled slots; of `hi`: 1 if the row holds an entry per slot.
struct SlotHead { uint32_t lo, hi; };

// Registers: small grids 127 or 128 and 32 to 72 bytes of scratch, because a workgroup may sample others' tiles again (a loop around
// the kernel; they have one or two waves per SIMD, four at most).  Otherwise nothing is spilled but 44 bytes in the prefix layout's
// form with 64-bit positions and without the scan.  With tickets 82 to 86 (64-bit positions 89 to 100), so that a compute unit holds
// one tile of sixteen waves; without the scan 68 with 32-bit positions, seven waves per SIMD (prefix layout 76, six), and 80 with
// 64-bit ones, six.  The kernel before this one kept seven there too, and was slower
// all the same: 2^20 queries over power-law ids, edge data on the host, unbounded windows 1.40 -> 1.34 ms, windowed 2.15 -> 1.40.
template <bool PREFIX, bool INCL, typename pos_t, int SCAN>
__global__ void __launch_bounds__(SCAN ? 1024 : 256, SCAN ? 4 : 6)
tns_sample_recent_kernel(const SampleArgs args, const int32_t stride, const uint32_t f_mul, const uint32_t chunk) {
    constexpr bool FUSED = SCAN != kNoScan;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int64_t s_tile_base;
    __shared__ int32_t s_wave_sum[16];
    __shared__ int32_t s_arrived;      // fused: waves of the tile that have finished their searches
    __shared__ int32_t s_todo;
    int lane = threadIdx.x & (kWave - 1), wave = wave_uniform((int32_t)(threadIdx.x >> 6));
    const int waves_per_wg = blockDim.x >> 6;

    // number of queries: the host's bound, or fewer when the count lives on the device (later hops); workgroups that
    // have none leave before they take a ticket
    const int64_t Q = args.Q_dev ? min(args.Q, *args.Q_dev) : args.Q;
    if (FUSED && (int64_t)blockIdx.x * blockDim.x >= Q) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {      // no query will write the end of rowptr
            args.rowptr[0] = 0;
            if (args.total_out) *args.total_out = 0;
        }
        return;
    }
    TileChain<SCAN> tc(args, &s_tile_base, &s_arrived, &s_todo);
    if (FUSED && tc.tile * blockDim.x >= Q) return;      // (tests whose tiles start at 1)
sample_tile:
    if (SCAN == kTags) {
        new_tile(lane, wave);
        wave = wave_uniform(wave);
    }
    const SampleArgs& p = [&]() -> const SampleArgs& {
        if constexpr (SCAN == kTags) return arguments_anew();
        else return args;
    }();
    const int64_t tile = SCAN == kTags ? wave_uniform(tc.tile) : tc.tile;
    const int64_t q0 = (tile * waves_per_wg + wave) * kWave;
    const int64_t q = q0 + lane;
    const int32_t f = p.fanout;
    // LDS of the wave: the staging area of the node lines (4 KiB); later, in the same bytes, the rows of the table and
    // behind them the search requests and their results, whose place the slot heads take
    unsigned char* const my_lds = smem + (size_t)wave * chunk;
    pos_t* const rows = reinterpret_cast<pos_t*>(my_lds);
    SearchRequest* const requests = reinterpret_cast<SearchRequest*>(my_lds + (size_t)kWave * stride * sizeof(pos_t));
    SlotHead* const heads = reinterpret_cast<SlotHead*>(requests);
    unsigned char* const found = reinterpret_cast<unsigned char*>(requests + 2 * kWave);

    Walk<0, INCL, pos_t, true> w;
    w.f = f;
    w.s_pos = rows + (size_t)lane * stride;
    w.edges = p.edges;
    w.group = kCoopGroup;
    w.te = 0.0f;
    w.tb = 0.0f;
    // (the queries are requested before the reads that find their instance: two or three dependent ones)
    const bool have = q < Q;
    int32_t v = -1;
    if (have) {
        v = __builtin_nontemporal_load(&p.targets[q0 + lane]);
        w.te = __builtin_nontemporal_load(&p.t_end[q0 + lane]);
        if (p.t_start) w.tb = p.t_start[q0 + lane];
    }
    const int32_t inst = p.inst_rowptr ? instance_of(p.inst_rowptr, p.num_instances, q0, q, Q, lane) : 0;
    if (!p.t_start) w.tb = p.delta == INFINITY ? -INFINITY : w.te - p.delta;
    bool ok = have && (uint32_t)v < (uint64_t)p.num_nodes && !(w.te != w.te) && !(w.tb != w.tb);
    if (p.inst_rowptr) ok = ok && inst < p.num_instances;
    const uint32_t node = ok ? (uint32_t)(inst * p.num_nodes + v) : ~0u;      // the target's entry in the node table (a table of 2^32 lines does not exist)
    tc.begin(p);
    // ---- the node's line: entry and the records of up to seven blocks, newest first -------------------
    u32x4 P[8];
    {
        // Eight lanes fetch one query's line with one instruction (16 bytes each), eight queries per instruction; the
        // pieces reach their owner through LDS.  (In the prefix layout the gather comes back to the line.)
        const int piece = lane & 7, sub = lane >> 3;
        const unsigned char* const table = (PREFIX ? reinterpret_cast<const unsigned char*>(p.edges) : reinterpret_cast<const unsigned char*>(p.nodes)) + piece * 16;
        uint32_t src[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) src[i] = (uint32_t)__shfl((int)node, i * 8 + sub, kWave);
        u32x4 R[8];
        // (a query without a node reads the first line and drops it: no load sits in a branch)
        auto line_of = [&](int i) { return reinterpret_cast<const u32x4*>(table + (uint64_t)(src[i] == ~0u ? 0u : src[i]) * 128u); };
        // (small grids without the hint, which costs their form scratch: 2^18 nodes, 10^5 queries 20.6 / 20.4 us, 250000 39.4 / 37.5, 2^20
        // nodes 21.0 / 21.0 and 39.9 / 38.9)
        if (PREFIX || SCAN == kTags || p.keep_nodes) {
#pragma unroll
            for (int i = 0; i < 8; ++i) R[i] = *line_of(i);
        } else {
            keep_apart();
#pragma unroll
            for (int i = 0; i < 8; ++i) R[i] = __builtin_nontemporal_load(line_of(i));
            keep_apart();
        }
        // in two rounds of 32 queries; 16-byte pieces are swizzled by the query number so that neither the writes nor
        // the reads collide on banks
#pragma unroll
        for (int r = 0; r < 2; ++r) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ql = i * 8 + sub;
                *reinterpret_cast<u32x4*>(my_lds + ql * 128 + ((piece ^ (ql & 7)) << 4)) = R[r * 4 + i];
            }
            wave_lds_sync();
            if ((lane >> 5) == r) {
                const int ql = lane & 31;
#pragma unroll
                for (int j = 0; j < 8; ++j) P[j] = *reinterpret_cast<const u32x4*>(my_lds + ql * 128 + ((j ^ (ql & 7)) << 4));
            }
            wave_lds_sync();
        }
    }
    auto before_end = [&](float t) { return INCL ? t <= w.te : t < w.te; };
    // ---- blocks: short lists without deleted edges ------------------------------------------------------
    // At most one block contains the window's end and at most one its start; the others count as a whole or not at all.
    // Of those two the slots on whose side something is known already are not searched.
    int32_t cnt[kInlineBlocks];        // candidates, newest block first
    pos_t end_slot[kInlineBlocks];     // slot behind the newest one
    int32_t end_block = -1, start_block = -1, b_lo = 0, b_n = 0;
    int32_t newer = 0, whole = 0;      // edges of the blocks newer than the one with the start that count as a whole
    int64_t b_off = 0;
    // block j; t_max: a time that no edge of it is after; undecided: slots to search where a time lies inside
    // the block (its first edge is known to be on the near side)
    auto block = [&](int j, bool there, float t_min, float t_max, int64_t off, int32_t size, int32_t undecided) {
        const bool in = there && before_end(t_min) && !(w.tb > t_max);
        cnt[j] = in ? size : 0;
        end_slot[j] = (pos_t)(off + size);
        if (in && !before_end(t_max)) { w.d_off = off; w.d_lo = 1; w.d_n = undecided; end_block = j; }
        if (in && w.tb > t_min) { b_off = off; b_lo = 1; b_n = undecided; start_block = j; newer = whole; }
        whole += in && before_end(t_max) ? size : 0;
    };
    bool flat;
    int32_t nb = 0;                    // list length (default layout); blocks outside the prefix
    uint32_t dir_line;
    if constexpr (!PREFIX) {
        uint4 hd = make_uint4(0u, 0u, 0u, 0u);
        uint4 L[kInlineBlocks];
#pragma unroll
        for (int j = 0; j < kInlineBlocks; ++j) L[j] = make_uint4(P[1 + j].x, P[1 + j].y, P[1 + j].z, P[1 + j].w);
        if (node != ~0u) hd = make_uint4(P[0].x, P[0].y, P[0].z, P[0].w);
        nb = (hd.w & 1) ? 0 : (int32_t)hd.x;                           // deleted node: no blocks
        dir_line = hd.z;
        flat = nb <= kInlineBlocks && !(hd.w & 2);
#pragma unroll
        for (int j = 0; j < kInlineBlocks; ++j) {
            const BlockRec r = as_rec(L[j]);
            const bool in = flat && j < nb && before_end(r.t_min) && !(w.tb > r.t_max);
            const int32_t size = rec_size(r);
            cnt[j] = in ? size : 0;
            end_slot[j] = (pos_t)(rec_off(r) + size);
            // What block() does, written out: called here it takes 76 registers instead of 68 without the scan, a wave per SIMD, and 97
            // instead of 89 with tickets and 64-bit positions.  (Of a block's slots, the first and the last one lie on different
            // sides of a time inside it.)
            if (in && !before_end(r.t_max)) { w.d_off = rec_off(r); w.d_lo = 1; w.d_n = size - 2; end_block = j; }
            if (in && w.tb > r.t_min) { b_off = rec_off(r); b_lo = 1; b_n = size - 2; start_block = j; newer = whole; }
            whole += in && before_end(r.t_max) ? size : 0;
        }
    } else {
        // Up to three blocks outside the prefix, newest first, then the extension lines and the node's own line as blocks: their
        // time index is the fences, so that a line's latest time is only known not to be after the next fence.
        const int32_t degree = (int32_t)P[6].x;
        const uint32_t meta = P[6].y;
        const bool alive = node != ~0u && !(meta & 1u) && degree > 0;
        nb = alive ? pmeta_big_blocks(meta) : 0;
        dir_line = P[7].w;
        flat = nb <= kPrefixBigBlocks && !(alive && (meta & 2u));
        const int32_t fill = alive && flat ? min(degree, pmeta_prefix_slots(meta)) : 0;       // edges stored in the prefix
        const float fence[kPrefixExtLines + 1] = {__uint_as_float(P[7].x), __uint_as_float(P[7].y), __uint_as_float(P[7].z), INFINITY};
        float after = INFINITY;        // the oldest block outside the prefix
        if (__ballot(nb > 0)) {
            const bool read = flat && nb > 0 && (int64_t)dir_line * kDirAlign + nb <= p.num_dir;
            BlockRec big[kPrefixBigBlocks];
#pragma unroll
            for (int j = 0; j < kPrefixBigBlocks; ++j) {
                big[j] = BlockRec{};
                if (read && j < nb) big[j] = p.dir[(int64_t)dir_line * kDirAlign + (nb - 1 - j)];
            }
#pragma unroll
            for (int j = 0; j < kPrefixBigBlocks; ++j) {
                const bool there = read && j < nb;
                if (there) after = big[j].t_min;
                block(j, there, big[j].t_min, big[j].t_max, rec_off(big[j]), rec_size(big[j]), rec_size(big[j]) - 2);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPrefixBigBlocks; ++j) { cnt[j] = 0; end_slot[j] = 0; }
        }
#pragma unroll
        for (int x = kPrefixExtLines - 1; x >= 0; --x) {
            const int32_t size = min(fill - kInlineSlots - kSlotsPerLine * x, kSlotsPerLine);
            const float next = x + 1 < kPrefixExtLines && size == kSlotsPerLine && fill > kInlineSlots + kSlotsPerLine * (x + 1) ? fence[x + 1] : after;
            const uint32_t line = x == 0 ? P[6].z : P[6].w + (uint32_t)(x - 1);
            block(kInlineBlocks - 2 - x, size > 0, fence[x], next, (int64_t)line * kSlotsPerLine, size, size - 1);
        }
        // the node's own line: its times are here
        const float own[kInlineSlots] = {__uint_as_float(P[0].x), __uint_as_float(P[0].w), __uint_as_float(P[1].z), __uint_as_float(P[2].y),
                                         __uint_as_float(P[3].x), __uint_as_float(P[3].w), __uint_as_float(P[4].z), __uint_as_float(P[5].y)};
        int32_t before = 0, early = 0;
#pragma unroll
        for (int i = 0; i < kInlineSlots; ++i) {
            before += i < fill && before_end(own[i]) ? 1 : 0;
            early += i < fill && own[i] < w.tb ? 1 : 0;
        }
        cnt[kInlineBlocks - 1] = max(before - early, 0);
        end_slot[kInlineBlocks - 1] = (pos_t)((int64_t)node * kSlotsPerLine + before);
    }
    // Where the newer blocks fill the slots, the one with the start is not searched; the walk of Algorithm 1 does not come to it
    // either.  (2^20 queries over power-law ids, window of a quarter of the time span, fan-out 20, padded rows only: edge data on the
    // host 2.51 -> 1.77 ms, in HBM 153 -> 139 us.)
    auto start_matters = [&]() {
        if (newer + (end_block != start_block ? w.d_lo : 0) >= f) b_n = 0;
    };
    if (!flat) {
        // ---- long lists, nodes with deleted edges: Algorithm 1 block by block --------------------------
        if (PREFIX) {
            // the blocks outside the prefix, then the prefix line by line
            const uint32_t* __restrict__ own = p.edges + (uint64_t)node * 32u;
            const uint32_t meta = own[kNodeHdrWord + 1];
            const int32_t fill = min((int32_t)own[kNodeHdrWord], pmeta_prefix_slots(meta));
            const int64_t d0 = (int64_t)dir_line * kDirAlign;
            const BlockRec* __restrict__ d = p.dir + d0;
            const bool dir_ok = nb > 0 && d0 + nb <= p.num_dir;
            int32_t lo = 0, n = dir_ok ? nb : 0, t = 0;
            narrow2(lo, n, 0, [&](int32_t i) { return before_end(d[i].t_min); });
            bool go = true;
#pragma unroll 1
            for (int32_t j = lo - 1; j >= 0 && go; --j, ++t) go = w.step(d[j], t);
            float after = dir_ok ? d[0].t_min : INFINITY;
#pragma unroll 1
            for (int32_t x = kPrefixExtLines - 1; x >= -1 && go; --x) {
                // extension line x, or the node's own line
                const int32_t first = x < 0 ? 0 : kInlineSlots + kSlotsPerLine * x, size = min(fill - first, x < 0 ? kInlineSlots : kSlotsPerLine);
                if (size <= 0) continue;
                const float t_min = __uint_as_float(x < 0 ? own[0] : own[kNodeHdrWord + 4 + x]);
                const uint32_t line = x < 0 ? node : (x == 0 ? own[kNodeHdrWord + 2] : own[kNodeHdrWord + 3] + (uint32_t)(x - 1));
                go = w.step(make_rec(t_min, after, (int64_t)line * kSlotsPerLine, size, (meta & 2u) != 0), t++);
                after = t_min;
            }
        } else if (nb <= kInlineBlocks) {
            bool go = true;
#pragma unroll 1
            for (int32_t j = 0; j < nb && go; ++j) go = w.step(p.nodes[node].rec[j], j);
        } else {
            // all records of the node, oldest first, in one run of the directory; the newest block that starts before the
            // window end is searched for instead of stepping through the newer ones one by one
            const int64_t d0 = (int64_t)dir_line * kDirAlign;
            if (d0 + nb <= p.num_dir) {
                const BlockRec* __restrict__ d = p.dir + d0;
                int32_t lo = 0, n = nb;
                if (FUSED) narrow4(lo, n, 0, [&](int32_t i) { return before_end(d[i].t_min); });
                else narrow2(lo, n, 0, [&](int32_t i) { return before_end(d[i].t_min); });
                bool go = true;
                for (int32_t j = lo - 1; j >= 0 && go; --j) go = w.step(d[j], lo - 1 - j);
            }
        }
    } else if (FUSED) {
        narrow4(w.d_lo, w.d_n, kCoopGroup, [&](int32_t i) { return before_end(time_at<pos_t>(p.edges, w.d_off + i)); });
        start_matters();
        narrow4(b_lo, b_n, kCoopGroup, [&](int32_t i) { return time_at<pos_t>(p.edges, b_off + i) < w.tb; });
    } else {
        // (without the scan one read at a time: of three in flight two are more traffic, 32.0 -> 31.5 ms across the host link)
        narrow2(w.d_lo, w.d_n, kCoopGroup, [&](int32_t i) { return before_end(time_at<pos_t>(p.edges, w.d_off + i)); });
        start_matters();
        narrow2(b_lo, b_n, kCoopGroup, [&](int32_t i) { return time_at<pos_t>(p.edges, b_off + i) < w.tb; });
    }
    // ---- search ------------------------------------------------------------------------------------------
    // Sixteen lanes read the timestamps of one request side by side and a ballot counts those before its time.
    const uint64_t ask_end = __ballot(w.d_n > 0), ask_start = __ballot(b_n > 0);
    const int num_end = __popcll(ask_end), num_requests = num_end + __popcll(ask_start);
    const uint64_t below = (1ull << lane) - 1ull;
    const int my_end = __popcll(ask_end & below), my_start = num_end + __popcll(ask_start & below);
    if (num_requests > 0) {
        if (w.d_n > 0) requests[my_end] = make_request<pos_t>(w.d_off + w.d_lo, w.d_n, w.te, INCL);
        if (b_n > 0) requests[my_start] = make_request<pos_t>(b_off + b_lo, b_n, w.tb, false);
        wave_lds_sync();
        const int g = lane / kCoopGroup, j = lane % kCoopGroup;
#pragma unroll 1
        for (int r0 = 0; r0 < num_requests; r0 += kRequestBatch * kGroups) {
            SearchRequest d[kRequestBatch];
            float t[kRequestBatch];
#pragma unroll
            for (int i = 0; i < kRequestBatch; ++i) {
                if (r0 + i * kGroups >= num_requests) break;       // uniform: a load without a request costs its address cycles
                // (beyond the last request: the last one again, its lines are on their way anyway)
                d[i] = requests[min(r0 + i * kGroups + g, num_requests - 1)];
                t[i] = __uint_as_float(p.edges[request_word<pos_t>(d[i], j)]);
            }
#pragma unroll
            for (int i = 0; i < kRequestBatch; ++i) {
                if (r0 + i * kGroups >= num_requests) break;
                const bool first = j < request_slots(d[i]) && (t[i] < d[i].t || (INCL && request_closed(d[i]) && t[i] == d[i].t));
                const uint32_t c = (uint32_t)__popc((uint32_t)(__ballot(first) >> (g * kCoopGroup)) & 0xffffu);
                found[min(r0 + i * kGroups + g, num_requests - 1)] = (unsigned char)c;
            }
        }
        wave_lds_sync();
    }
    int32_t h = w.d_lo;                // edges of the block with the window's end that lie before it
    if (w.d_n > 0) h += found[my_end];
    if (b_n > 0) b_lo += found[my_start];
    wave_lds_sync();                   // the heads take the place of the requests
    // ---- table -------------------------------------------------------------------------------------------
    int32_t k;
    SlotHead head{kFlagBytes, kFlagBytes};
    if (flat) {
        pos_t* const row = rows + (size_t)lane * stride;
        int32_t cum = 0;
        uint32_t before[kInlineBlocks];
#pragma unroll
        for (int j = 0; j < kInlineBlocks; ++j) {
            pos_t e = end_slot[j];
            int32_t c = cnt[j];
            if (j == end_block) { e += (pos_t)(h - c); c = h; }
            if (j == start_block) c = max(c - b_lo, 0);
            before[j] = (uint32_t)min(cum, kWave);
            row[j] = e - 1 + (pos_t)cum;               // minus the slot's number: where its edge lies
            cum += c;
        }
        k = min(cum, f);
        head.lo -= before[1] | before[2] << 8 | before[3] << 16;
        head.hi -= before[4] | before[5] << 8 | before[6] << 16;
    } else {
        // the first hh slots come from the block whose search the wave finished (newest first); the entries recorded
        // from older blocks move up behind them
        const int32_t hh = w.d_off >= 0 ? min(h, f) : 0;
        k = min(f, hh + w.k);
        for (int32_t j = k - 1; j >= hh; --j) w.s_pos[j] = w.s_pos[j - hh] + (pos_t)hh;
        for (int32_t j = 0; j < hh; ++j) w.s_pos[j] = (pos_t)(w.d_off + h - 1);
        head.hi |= 1u << 24;
    }
    head.lo |= (uint32_t)k << 24;
    heads[lane] = head;
    wave_lds_sync();
    // ---- gather and outputs --------------------------------------------------------------------------------
    // Slots [it0 * 64, (it0 + kGatherChunk) * 64) of the wave, prepared in groups of kGatherGroup.  An empty slot reads what
    // the first filled one of its instruction reads (one request for both; a fixed address instead would make one memory
    // channel everybody's).
    auto load = [&](GatherRegs& g, int32_t it0) {
        bool filled[kGatherChunk];
        Edge raw[kGatherChunk];
#pragma unroll
        for (int i0 = 0; i0 < kGatherChunk; i0 += kGatherGroup) {
            if (it0 + i0 >= f) {                       // uniform over the wave
#pragma unroll
                for (int i = i0; i < i0 + kGatherGroup; ++i) { filled[i] = false; raw[i] = Edge{0.0f, -1, -1}; }
                continue;
            }
            SlotHead sh[kGatherGroup];
            uint32_t ql[kGatherGroup], no[kGatherGroup];
            pos_t e[kGatherGroup];
#pragma unroll
            for (int u = 0; u < kGatherGroup; ++u) {
                const uint32_t s = (uint32_t)((it0 + i0 + u) * kWave + lane);
                ql[u] = min(query_of_slot(s, f_mul), (uint32_t)kWave - 1u);      // (the last group may reach beyond the last slot)
                no[u] = s - ql[u] * (uint32_t)f;
                sh[u] = heads[ql[u]];
            }
#pragma unroll
            for (int u = 0; u < kGatherGroup; ++u) {
                const uint32_t each = no[u] * 0x010101u;
                uint32_t b = (uint32_t)(__popc((each + sh[u].lo) & kFlagBytes) + __popc((each + sh[u].hi) & kFlagBytes));
                if (sh[u].hi >> 24) b = no[u];
                filled[i0 + u] = no[u] < (sh[u].lo >> 24);
                e[u] = rows[ql[u] * (uint32_t)stride + (filled[i0 + u] ? b : 0u)];
            }
#pragma unroll
            for (int u = 0; u < kGatherGroup; ++u) {
                const uint64_t m = __ballot(filled[i0 + u]);
                const pos_t own = e[u] - (pos_t)no[u];
                const pos_t other = m ? wave_read(own, __builtin_ctzll(m)) : (pos_t)0;
                const auto pos = (typename index_of<pos_t>::type)slot_pos<pos_t>(filled[i0 + u] ? own : other);
                raw[i0 + u] = *reinterpret_cast<const Edge*>(p.edges + pos);
            }
        }
        // every load of the batch has returned before the first store is issued: the stores that follow then go out back
        // to back without waiting for one another
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0) only
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kGatherChunk; ++i) {
            g.nbr[i] = filled[i] ? raw[i].nbr : -1;
            g.eid[i] = filled[i] ? raw[i].eid : -1;
            g.ts[i] = filled[i] ? raw[i].ts : 0.0f;
        }
    };
    if constexpr (FUSED) {
        fused_output<true, !PREFIX && SCAN == kTickets ? kShuffledScan : kVectorSums>(p, &s_tile_base, s_wave_sum, &s_arrived, tc, wave, waves_per_wg, lane, q0, Q, k, f_mul, load);
    } else {
        GatherRegs g;
        for (int32_t it0 = 0; it0 < f; it0 += kGatherChunk) {
            load(g, it0);
            store_padded(g, p, lane, it0, q0, Q);
        }
    }
    if (q < Q && p.out_count) __builtin_nontemporal_store(k, &p.out_count[q]);
    if (tc.next(p, &s_tile_base, &s_arrived, lane)) goto sample_tile;
}

template <bool PREFIX, bool INCL, typename pos_t, bool FUSED>
hipError_t launch_recent_t(const SampleArgs& a, hipStream_t stream) {
    const int32_t stride = std::max(a.fanout, kInlineBlocks) | 1;                // odd: conflict-free per-lane rows
    // per wave: the table, the requests and their results; at least the 4 KiB in which the node lines are staged first
    const size_t chunk = std::max<size_t>((((size_t)kWave * stride * sizeof(pos_t) + 15) & ~size_t(15)) + 2 * kWave * (sizeof(SearchRequest) + 1), 4096);
    // The fused variant uses large workgroups: one chained-scan step per 1024 queries keeps the rate at which tiles publish
    // their totals low enough for the look-back to keep up.  The registers would let ten waves each of two workgroups share a compute unit, so
    // that one tile's searches fill the other's waits: with tickets, us with 16 / 10 / 8 waves, prefix layout, 10^6 queries 94.8 / 101.5 /
    // 103.1, windowed 86.7 / 93.5 / 104.3, 2^22 339 / 350 / 357; two hops from 2^20 roots 393 / 395 / 478; 256 graphs 1327 / 1428 / 1535; blocks, 10^6
    // 116 / 120 / 124, power-law ids 120 / 131 / 164, 2^24 1413 / 1601 / 1609.
    constexpr size_t kLds = 159u << 10;
    int waves = FUSED ? 16 : 4;
    while (waves > 1 && (size_t)waves * chunk > kLds) --waves;
    if (!FUSED) {
        // Larger fan-outs: smaller workgroups where a quarter more waves then fit a compute unit's LDS.  (2^20 queries, padded rows
        // only, power-law ids, windowed: fan-out 32, 12 waves as 3 x 4 197 us, 15 as 5 x 3 189; fan-out 20, where 7 x 3 would be 21
        // instead of 20, 139 and 147.)
        const int four = waves;
        auto resident = [&](int n) { return (int)(kLds / (n * chunk)) * n; };
        for (int n = four - 1; n >= 1; --n)
            if (resident(n) * 4 >= resident(four) * 5 && resident(n) > resident(waves)) waves = n;
    }
    waves = workgroup_waves(a.Q, a.fanout, waves, FUSED);
    const int64_t per_wg = (int64_t)waves * kWave;
    const int64_t grid = (a.Q + per_wg - 1) / per_wg;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = chunk * waves;
    auto launch = [&](auto scan, const SampleArgs& b) {
        hipLaunchKernelGGL((tns_sample_recent_kernel<PREFIX, INCL, pos_t, decltype(scan)::value>), dim3((unsigned)grid), dim3(waves * kWave), lds, stream, b,
                           stride, slot_multiplier(a.fanout), (uint32_t)chunk);
    };
    // Padded rows only over the prefix layout: tiles in the order of the workgroups.  With a contiguous range of tiles per XCD, us: 2^22
    // queries 267 -> 296, 2^24 1086 -> 1204, 2^26 4297 -> 4798 (the kernel before the one with block tables, with ranges, 316, 1052 and 4308).
    SampleArgs b = a;
    if (PREFIX && !FUSED) b.xcd_remap = 0;
    return launch_tiles<FUSED>(b, grid, per_wg, stream, launch);
}

}  // namespace

hipError_t launch_sample_recent(const SampleArgs& a, hipStream_t stream) {
    const bool fused = a.scan_ws != nullptr;
#define TNS_DISPATCH(PRE, INC)                                                                                                          \
    (a.wide_offsets ? (fused ? launch_recent_t<PRE, INC, int64_t, true>(a, stream) : launch_recent_t<PRE, INC, int64_t, false>(a, stream)) \
                    : (fused ? launch_recent_t<PRE, INC, int32_t, true>(a, stream) : launch_recent_t<PRE, INC, int32_t, false>(a, stream)))
    if (a.prefix_layout) return a.inclusive_end ? TNS_DISPATCH(true, true) : TNS_DISPATCH(true, false);
    return a.inclusive_end ? TNS_DISPATCH(false, true) : TNS_DISPATCH(false, false);
#undef TNS_DISPATCH
}

}  // namespace tns
