// Launch interface between the C ABI (tns_api.hip) and the gfx950 kernels (tns_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "tns_layout.h"

namespace tns {

constexpr int kDeferSpins = 2048;      // about two milliseconds

struct SampleArgs {
    // store (device)
    const NodeLine* nodes;
    const BlockRec* dir;     // directory pool: record runs of nodes with more than kInlineBlocks blocks
    const uint32_t* dir_cum; // same indexing: number of the node's edges stored in the blocks before this one
    const uint32_t* edges;   // edge lines viewed as 4-byte words: slot s starts at word slot_word(s)
    // queries (device)
    const int32_t* targets;
    const float* t_start;        // may be null: -inf
    const float* t_end;
    const int64_t* inst_rowptr;  // may be null: one instance
    // padded outputs (device)
    int32_t* out_nbr;
    int32_t* out_eid;
    float* out_ts;
    int32_t* out_count;
    // non-null: count what the walk reads (node entries, block records, timestamp probes,
    // edges selected) into counters[0..3] instead of producing outputs
    unsigned long long* counters;
    // non-null: also remove the padding in the same pass (chained scan over workgroups);
    // scan_ws is the caller's workspace, rowptr / cmp_* the dense outputs
    void* scan_ws;
    int64_t* rowptr;
    int32_t* cmp_nbr;
    int32_t* cmp_eid;
    float* cmp_ts;
    int64_t Q;               // number of queries, or an upper bound of it when Q_dev is set
    const int64_t* Q_dev;    // may be null; device-resident number of queries (hops after the first)
    int64_t* total_out;      // may be null; fused variant: also receives the dense total (rowptr[Q])
    float delta;             // window length used when t_start is null: t_start = t_end - delta (+inf: unbounded)
    int64_t num_nodes;
    int64_t num_dir;     // records in the directory pool (walks never index past it)
    int64_t qid_base;
    uint64_t seed;
    int32_t num_instances;
    int32_t fanout;
    int32_t policy;
    int32_t inclusive_end;
    int32_t xcd_remap;
    int32_t keep_nodes;    // node lines are likely to be read again soon: no non-temporal hint on them
    int32_t wide_offsets;  // edge array has 2^31 or more entries: 64-bit positions in LDS
    int32_t first_ticket;  // 0; tests of the chained scan's bounded wait pass 1: tile 0 then never exists
    int32_t defer_spins;   // small grids: rounds of waiting for a tile that has not started (kDeferSpins; tests: -1, for any tile)
    int32_t scan_ready;    // scan_ws is as this launch needs it (multi-hop: one clearing launch for all hops that need it)
    int32_t prefix_layout; // the store is in the prefix layout: `edges` is the one array of lines, node v's line is line v
    uint64_t chain_tag;    // small grids: what tells this launch's tile states from older ones (TaggedChain in tns_chain.h)
    uint32_t* err_flag;    // where a chained scan whose bounded wait ran out reports it (null: the error word of scan_ws)
    // Tile states that scan_ws holds: read by the host alone, and last, because where it lies moves what the kernels request together from
    // their arguments.  Between scan_ws and rowptr / behind cmp_ts / here, large batches, data of several calls in turn, us: recent policy,
    // prefix layout, 10^6 queries 104.4 / 102.8 / 102.4, 2^22 357 / 355 / 354; uniform policy, 10^6 queries, fan-out 10, prefix layout 124.1 /
    // 121.5 / 123.8, blocks 152.0 / 151.2 / 153.4.  Behind cmp_ts / here, fan-out 32 over power-law ids, 2 * 10^5 queries 163 / 152, 330000 262 / 234.
    int64_t scan_states;
};

static_assert(offsetof(SampleArgs, scan_states) == sizeof(SampleArgs) - sizeof(int64_t), "what kernels read lies side by side");

struct CompactArgs {
    const int32_t* nbr;
    const int32_t* eid;
    const float* ts;
    const int32_t* count;
    int64_t* rowptr;
    int32_t* cmp_nbr;
    int32_t* cmp_eid;
    float* cmp_ts;
    int64_t Q;
    const int64_t* Q_dev;    // may be null; device-resident number of queries
    int64_t* total_out;      // may be null; also receives the dense total
    int32_t fanout;
    void* workspace;
};

constexpr size_t kScanHeader = 256;         // of a scan workspace, before the tile states
constexpr int64_t kSmallTile = 16, kMostSmallTiles = 256;      // queries of the smallest tiles; most tiles of a call that are made small
constexpr int kCompactTile = 1024;  // queries per compaction tile

// What a call with Q queries needs, and what it is asked to bring: room for the states of smaller tiles where the batch is small
// (tns_kernels_team.hip).
size_t compact_workspace_least(int64_t Q);
size_t compact_workspace_bytes(int64_t Q);
// tile states in a workspace of that size
int64_t tile_states(size_t bytes);

// Both only enqueue kernels on `stream`; they return the first launch error.
hipError_t launch_sample(const SampleArgs& a, hipStream_t stream);
// The same under the recent policy, a query per lane (tns_kernels_recent.hip); launch_sample forwards to it.
hipError_t launch_sample_recent(const SampleArgs& a, hipStream_t stream);
// The same for a store in the prefix layout (tns_kernels_prefix.hip); launch_sample forwards to it.
hipError_t launch_sample_prefix(const SampleArgs& a, hipStream_t stream);
// The same with sixteen lanes per query (tns_kernels_team.hip); launch_sample forwards to it by the batch size.
hipError_t launch_sample_team(const SampleArgs& a, hipStream_t stream);
// Most queries of a call with fan-out f whose tiles need no cleared scan state (TaggedChain in tns_chain.h): as many as the
// chip holds at once, sixteen waves per compute unit or what the LDS of a wave's result rows allows.
constexpr int64_t tagged_queries(int32_t f) { return int64_t(1) << (f <= 12 ? 18 : (f <= 32 ? 17 : 16)); }
// Draws the tag of such a launch, another one every time, and clears the state where may_be_replayed() says so.
hipError_t ready_tags(SampleArgs& a, int64_t tiles, hipStream_t stream);
// What is launched on the stream is being captured: it may run again as it is.
bool may_be_replayed(hipStream_t stream);
// Clears the chained scan's state for `num_tiles` tiles before a fused launch (kernel, capturable).
hipError_t launch_scan_init(const SampleArgs& a, int64_t num_tiles, hipStream_t stream);
hipError_t launch_compact(const CompactArgs& a, hipStream_t stream);
// Clears `bytes` (a multiple of 8) of chained-scan workspace with a kernel (capturable, unlike a memset).
hipError_t launch_scan_clear(void* ws, size_t bytes, hipStream_t stream);
hipError_t launch_hop_inst_rowptr(const int64_t* cur, const int64_t* rowptr, int32_t num_instances, int64_t* next,
                                  hipStream_t stream);

}  // namespace tns
