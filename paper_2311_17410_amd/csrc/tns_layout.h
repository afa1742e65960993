// Record layouts shared by the host-side store builder and the device kernels.
//
// The paper (section 4.1) lists what a node entry and an edge block hold but not their byte
// layout (it only gives the size of a block's metadata) and links a node's blocks into a doubly-linked
// list.  On MI355X every dependent random read costs a 128-byte line from HBM, so a linked
// list of separately allocated records costs one line per block visited.  Here the records of
// one node sit next to each other instead:
//
//   * NodeLine (128 bytes, line-aligned): the node entry (list length, degree, validity) plus
//     the records of up to 7 blocks, newest first.  One line read gives Algorithm 1 everything
//     it needs to skip, stop or search for nodes with short lists.
//   * nodes with longer lists keep all their records, oldest first, in one contiguous run of
//     the directory pool; the walk starts with a binary search over it instead of stepping
//     through the newer blocks one by one.
//   * BlockRec (16 bytes): earliest and latest timestamp, number of edges, offset of the
//     block's edges.  The capacity is not needed by sampling: every block but the newest is
//     full, and the newest block's capacity is kept on the host.
//   * Edge (12 bytes): timestamp, neighbour id, edge id side by side, so the timestamps probed
//     by the in-block search and the ids gathered afterwards share lines; ten edges per
//     128-byte line (EdgeLine).
#pragma once
#include <cstdint>

namespace tns {

constexpr int kInlineBlocks = 7;
constexpr int64_t kMaxBlockEdges = (int64_t(1) << 24) - 1;  // size field is 24 bits
constexpr int64_t kMaxEdgeOffset = (int64_t(1) << 39) - 1;  // offset (slot index) field is 39 bits

// Edge block metadata (section 4.1: fill, where the edge data is, earliest and latest time).
struct BlockRec {
    float t_min, t_max;  // earliest / latest edge time in the block
    uint32_t off_lo;     // low 32 bits of the slot index of the block's first edge
    uint32_t size_hi;    // bits 0-23: edges held; bits 24-30: offset bits 32-38; bit 31: block holds deleted edges
};
static_assert(sizeof(BlockRec) == 16, "block record is 16 bytes");

#if defined(__HIPCC__)
#define TNS_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define TNS_HD inline
#endif
TNS_HD int32_t rec_size(const BlockRec& r) { return (int32_t)(r.size_hi & 0xffffffu); }
TNS_HD int64_t rec_off(const BlockRec& r) { return (int64_t)r.off_lo | ((int64_t)((r.size_hi >> 24) & 0x7fu) << 32); }
TNS_HD bool rec_tombstones(const BlockRec& r) { return (r.size_hi >> 31) != 0; }
TNS_HD BlockRec make_rec(float t_min, float t_max, int64_t off, int32_t size, bool tombstones = false) {
    BlockRec r;
    r.t_min = t_min;
    r.t_max = t_max;
    r.off_lo = (uint32_t)(off & 0xffffffffu);
    r.size_hi = ((uint32_t)size & 0xffffffu) | (((uint32_t)(off >> 32) & 0x7fu) << 24) | (tombstones ? 0x80000000u : 0u);
    return r;
}

// Node table entry (section 4.1: list length, degree, validity, access to the blocks).
struct alignas(128) NodeLine {
    int32_t nblocks;   // list length
    int32_t degree;    // stored edges (out-degree)
    uint32_t dir_line; // nblocks > kInlineBlocks: where the node's records start in the directory
                       // pool, in units of kDirAlign records (oldest record first)
    int32_t flags;     // bit 0: node deleted; bit 1: some block of the node holds deleted edges
    BlockRec rec[kInlineBlocks];  // nblocks <= kInlineBlocks: rec[0] newest ... rec[nblocks-1] oldest
};
static_assert(sizeof(NodeLine) == 128, "node entry is one 128-byte line");

constexpr int kDirAlign = 8;  // directory runs start on a 128-byte line

// One entry of the graph edge data.  Inside a block, entries are in (timestamp, arrival) order.
// Edge ids are non-negative; a deleted edge (section 4.1: validity cleared, layout kept) stores the
// bitwise complement of its id, so validity costs no extra word and the id stays recoverable.
struct Edge {
    float ts;
    int32_t nbr;
    int32_t eid;
};
static_assert(sizeof(Edge) == 12, "edge entry is 12 bytes");

// The edge array is made of 128-byte lines of 10 edge slots (8 bytes unused per line), so that
// a block of up to 10 slots allocated at a line start is read with one line, and blocks are
// addressed by slot index: slot s lives in line s / 10 at position s % 10.
constexpr int kSlotsPerLine = 10;
struct alignas(128) EdgeLine {
    Edge e[kSlotsPerLine];
    uint32_t unused[2];
};
static_assert(sizeof(EdgeLine) == 128, "edge line is 128 bytes");

// 4-byte word index of slot s inside the edge array (line * 32 + position * 3)
TNS_HD int64_t slot_word(int64_t s) {
    const int64_t line = s / kSlotsPerLine;
    return line * 32 + (s - line * kSlotsPerLine) * 3;
}

// words from the begin of a line to a slot that many slots behind it
TNS_HD uint32_t words_behind(uint32_t slots) { return 3u * slots + 2u * (slots / (uint32_t)kSlotsPerLine); }

// The edges of a block, for addresses of many of its slots: slot i lies at word `base` + words_to(i), below 2^32 words behind it.
// One division of the block's 39-bit slot index by the slots per line, as 2^32 = 10 * 429496729 + 6, and one of 32 bits per slot;
// slot_word takes a 64-bit one per slot, about thirty instructions.
struct BlockWords {
    uint64_t base;      // of the line with the block's first slot
    uint32_t at;        // the first slot's position there
    TNS_HD explicit BlockWords(const BlockRec& r) {
        const uint32_t lo = r.off_lo, hi = (r.size_hi >> 24) & 0x7fu, q = lo / (uint32_t)kSlotsPerLine;
        const uint32_t t = lo - q * (uint32_t)kSlotsPerLine + hi * 6u, tq = (t * 205u) >> 11;      // t <= 771; t / kSlotsPerLine
        base = ((uint64_t)hi * 429496729u + q + tq) * 32u;
        at = t - tq * (uint32_t)kSlotsPerLine;
    }
    TNS_HD uint32_t words_to(int32_t i) const { return words_behind(at + (uint32_t)i); }      // i: up to 2^24
};

// Search request of the sampling kernel for the recent policy: up to sixteen consecutive slots whose timestamps are
// compared with one time by as many lanes.
struct alignas(16) SearchRequest {
    uint32_t line;      // edge line of the first slot, low 32 bits
    float t;            // the time searched for
    uint32_t range;     // bits 0-7: position of the first slot in its line; bits 8-15: number of slots; bit 16: slots at the time
                        // count too; bits 17-31: upper bits of the line (2^39 slots are more than 2^32 lines)
    uint32_t unused;
};
// pos_t (32 or 64 bits): a type that holds every word index of the edge array
template <typename pos_t>
TNS_HD SearchRequest make_request(int64_t slot0, int32_t n, float t, bool closed) {
    const uint64_t line = sizeof(pos_t) == 8 ? (uint64_t)slot0 / (uint32_t)kSlotsPerLine : (uint32_t)slot0 / (uint32_t)kSlotsPerLine;
    const uint32_t at = (uint32_t)slot0 - (uint32_t)line * (uint32_t)kSlotsPerLine;
    return SearchRequest{(uint32_t)line, t, at | (uint32_t)n << 8 | (closed ? 1u << 16 : 0u) | (uint32_t)(line >> 32) << 17, 0u};
}
TNS_HD int32_t request_slots(const SearchRequest& r) { return (int32_t)((r.range >> 8) & 0xffu); }
TNS_HD bool request_closed(const SearchRequest& r) { return ((r.range >> 16) & 1u) != 0; }
// word index of the timestamp in slot j of a request (of the last one for a j beyond it)
template <typename pos_t>
TNS_HD uint64_t request_word(const SearchRequest& r, int32_t j) {
    const int32_t last = request_slots(r) - 1;
    const uint32_t s = (r.range & 0xffu) + (uint32_t)(j < last ? j : last);      // below 25
    const uint32_t lines = (s * 205u) >> 11;                                     // s / kSlotsPerLine
    const uint64_t line = sizeof(pos_t) == 8 ? (uint64_t)(r.range >> 17) << 32 | r.line : r.line;
    return line * 32u + (3u * s + 2u * lines);
}

// ---- prefix layout (TNS_FLAG_PREFIX_LAYOUT) ------------------------------------------------------
//
// A second placement of the same logical structure (node table, chronological block lists, block
// capacities by the sizing rule of section 4.1), made to cut the number of 128-byte lines a query
// touches.  Node table and edge data share ONE array of 128-byte lines of 10 slot positions each, so
// that every edge is addressed by one slot index whatever line it lives in:
//
//   * line v (v < number of nodes) is node v's line: slot positions 0..7 hold the node's first eight
//     edge slots, the last 32 bytes (slot positions 8, 9 and the line's spare 8 bytes) the node entry;
//   * a node's first blocks are carved, in order, out of its "prefix": 38 consecutive slots = the 8
//     slots in its own line plus up to three extension lines of 10 (allocated when a block reaches
//     into them, never moved).  A block belongs to the prefix while the capacities so far fit; the
//     first block that does not fit, and every later one, is placed on its own as in the default
//     layout and gets a 16-byte record in the node's run of the directory pool;
//   * inside the prefix, blocks are contiguous and all but the newest are full, so edge i of the node
//     sits in prefix slot i: the time index over the prefix is one fence per extension line (the
//     timestamp of its first slot), kept in the node entry.  Block capacities of prefix blocks are
//     needed by insertion and inspection only and stay on the host.
constexpr int kInlineSlots = 8;                                    // edge slots in the node's own line
constexpr int kPrefixExtLines = 3;                                 // extension lines of the prefix
constexpr int kPrefixSlots = kInlineSlots + kPrefixExtLines * kSlotsPerLine;   // 38

// Node entry = words 24..31 of the node's line.
constexpr int kNodeHdrWord = 24;
struct PrefixNodeHdr {
    int32_t degree;      // stored edges
    uint32_t meta;       // bit 0: node deleted; bit 1: node holds deleted edges; bits 2-3: extension lines that
                         // hold edges; bits 4-9: slots of the prefix given to blocks; bits 10-31: blocks outside the prefix
    uint32_t ext0;       // line index of the first extension line
    uint32_t ext12;      // line index of the second extension line; the third follows it
    float fence[kPrefixExtLines];   // timestamp of the first slot of each extension line
    uint32_t dir_line;   // blocks outside the prefix: start of the node's record run, in units of kDirAlign records
};
static_assert(sizeof(PrefixNodeHdr) == 32, "node entry is 32 bytes");
TNS_HD int32_t pmeta_ext_lines(uint32_t m) { return (int32_t)((m >> 2) & 3u); }
TNS_HD int32_t pmeta_prefix_slots(uint32_t m) { return (int32_t)((m >> 4) & 63u); }
TNS_HD int32_t pmeta_big_blocks(uint32_t m) { return (int32_t)(m >> 10); }
TNS_HD uint32_t make_pmeta(uint32_t flags, int32_t ext_lines, int32_t prefix_slots, int32_t big_blocks) {
    return (flags & 3u) | ((uint32_t)ext_lines << 2) | ((uint32_t)prefix_slots << 4) | ((uint32_t)big_blocks << 10);
}
constexpr int32_t kMaxBigBlocks = (1 << 22) - 1;
// A line of the prefix layout's array, seen as edge data or as a node's line.
struct alignas(128) PrefixNodeLine {
    Edge e[kInlineSlots];
    PrefixNodeHdr hdr;
};
union alignas(128) StoreLine {
    EdgeLine edges;
    PrefixNodeLine node;
};
static_assert(sizeof(StoreLine) == 128, "a line is 128 bytes");

// A node line is read with the non-temporal hint unless other queries will come back to it: it should not push edge lines out of the
// caches.  They do where an instance's table is at most half of the chip's L2, and where degrees are skewed, which a directory of
// at least a sixteenth of the nodes shows if the mean list is one that a node line holds; longer ones fill a directory of any
// degrees.  Hint / none, us, recent policy and uniform policy: 256 graphs of 4096 nodes, windowed 1500 / 1346 and 1680 / 1417; power-law
// ids, 2^18 nodes 568 / 519 and 915 / 855, 2^19 1205 / 1093 and 1944 / 1811, 2^20 2480 / 2320 and 4424 / 4123; uniform ids, 2^17 nodes 189 /
// 183 and 221 / 213, 2^18 362 / 367 and 421 / 403, 2^19 714 / 755 and 843 / 857, 2^20 1431 / 1490 and 1704 / 1743, 2^21 2966 / 2954 and
// 3422 / 3455, 2^22 6215 / 6191 and 6953 / 6993, 2^20 windowed 1341 / 1425 and 1582 / 1639 (a query per edge each).  A hundred
// edges a node, uniform policy, 2^22 queries: power-law ids, 2^18 nodes (4.6 blocks a list) 1225 / 1204, 2^20 (5.5) 1638 / 1612; uniform
// ids, 2^18 (12.1) 1313 / 1322, 2^20 (14.7) 1472 / 1478, 48 edges (8.2) 1013 / 1021.
constexpr int64_t kSmallTable = int64_t(1) << 17;       // nodes
inline bool node_lines_stay(int64_t nodes_per_instance, int64_t nodes, int64_t num_dir, int64_t num_blocks) {
    return nodes_per_instance <= kSmallTable || (num_dir * 16 >= nodes && num_blocks <= nodes * kInlineBlocks);
}

}  // namespace tns
