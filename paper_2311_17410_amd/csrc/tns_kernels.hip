// gfx950 kernels: temporal neighbourhood sampling (Algorithm 1 of the paper, section 4.2) over
// the block store of section 4.1 with a query per lane, uniform policy (the recent policy has a kernel of its own,
// tns_kernels_recent.hip) and the counting pass of both, and removal of the padding (section 5).
//
// Thread mapping.  The paper runs one thread per sampled neighbour with the f threads of a
// target adjacent.  On a 64-wide wavefront with dependent random reads (node entry -> block
// record -> timestamps -> edge data) what limits throughput is the number of independent
// chains in flight and the number of different 128-byte lines a load instruction touches, so:
//   * the walk runs one query per lane (64 independent chains per wave);
//   * the node entries are fetched by the wave together, eight lanes per 128-byte line, and
//     handed to their lanes through LDS;
//   * each lane leaves the edge positions it selected in LDS, as the paper stages candidate
//     positions in shared memory for uniform sampling; picks on long lists are resolved by the
//     wave, one (query, slot) per lane;
//   * the gather of the selected edges is done by the whole wave, all loads of a phase issued
//     before the first result is used: lane l handles flat slot it*64+l of the wave's 64*f slots,
//     so every store instruction covers 256 consecutive bytes of each output array;
//   * with the dense outputs requested, the workgroups pass their dense offsets along a chain
//     (single-pass scan over tiles) and write the dense rows from registers.
#include "tns_kernels.h"
#include "tns_device.h"

#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <type_traits>

namespace tns {
namespace {

// Clears the ticket, the error flag and the tile states before a fused launch (a kernel rather
// than a memset, so that the launch sequence can be captured into a graph).
__global__ void __launch_bounds__(256) tns_scan_init(ScanWorkspace* ws, int64_t num_tiles, int64_t* rowptr0, int64_t Q,
                                                     const int64_t* Q_dev, int64_t* total_out, uint32_t first_ticket) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) {
        ws->ticket = first_ticket;
        ws->error = 0;
        ws->noted = 0;
        ws->failed = 0;
        if (Q_dev && *Q_dev < Q) Q = *Q_dev;
        if (Q <= 0) {          // no query will write the end of rowptr
            rowptr0[0] = 0;
            if (total_out) *total_out = 0;
        }
    }
    if (i < num_tiles) ws->status[i] = 0;
}

__global__ void __launch_bounds__(256) tns_scan_clear(uint64_t* ws, int64_t words) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < words) ws[i] = 0;
}

// FUSED: also removes the padding in the same pass (rowptr and dense arrays), with the tile
// offsets obtained from a chained scan over the workgroups.
template <int POLICY, bool INCL, typename pos_t, bool COUNT, int SCAN>
__global__ void __launch_bounds__(SCAN ? 1024 : 256, SCAN ? 4 : 6)
tns_sample_kernel(const SampleArgs args, const int32_t stride, const uint32_t f_mul, const uint32_t chunk) {
    constexpr bool FUSED = SCAN != kNoScan;
    static_assert(POLICY == 1 || (COUNT && !FUSED), "the recent policy is sampled by tns_sample_recent_kernel");
    // LDS: one chunk per wave.  First the staging area of the node lines (3 KiB), later, in the same bytes,
    // the wave's rows of selected positions.
    constexpr bool COOP_NODE = !COUNT;
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

    Walk<POLICY, INCL, pos_t> w;
    w.f = f;
    unsigned char* const my_lds = smem + (size_t)wave * chunk;
    w.s_pos = reinterpret_cast<pos_t*>(my_lds) + (size_t)lane * stride;
    w.edges = p.edges;
    // the byte model counts a search as narrowed by the lane and finished together for these fan-outs, as made by the lane alone for
    // larger ones
    w.group = POLICY == 0 && f <= kCoopGroup ? kCoopGroup : 0;
    w.te = 0.0f;
    w.tb = 0.0f;
    int32_t n_nodes = 0;
    int64_t nidx = -1;           // index of the target's entry in the node table, -1: no walk
    const int32_t inst = p.inst_rowptr ? instance_of(p.inst_rowptr, p.num_instances, q0, q, Q, lane) : 0;
    if (q < Q) {
        const int32_t v = __builtin_nontemporal_load(&p.targets[q]);
        w.te = __builtin_nontemporal_load(&p.t_end[q]);
        w.tb = p.t_start ? p.t_start[q] : (p.delta == INFINITY ? -INFINITY : w.te - p.delta);
        int64_t nbase = 0;
        bool ok = (uint32_t)v < (uint64_t)p.num_nodes && !(w.te != w.te) && !(w.tb != w.tb);
        if (p.inst_rowptr) {
            ok = ok && inst < p.num_instances;
            nbase = (int64_t)inst * p.num_nodes;
        }
        if (ok) nidx = nbase + v;
    }
    tc.begin(p);
    // the node's 128-byte line: header + the records of up to 7 blocks, newest first
    uint4 hd = make_uint4(0u, 0u, 0u, 0u);
    uint4 L[kInlineBlocks];
    if (COOP_NODE) {
        // Eight lanes fetch one query's line with one instruction (16 bytes each), eight queries per
        // instruction; the pieces reach their owner through LDS.
        unsigned char* stage = my_lds;
        const int piece = lane & 7, sub = lane >> 3;
        int64_t src[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) src[i] = shfl64(nidx, i * 8 + sub);
        u32x4 R[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) R[i] = u32x4{0u, 0u, 0u, 0u};
        // (As compiled the first of the eight loads is the same in both branches, without the hint.  With the branches kept apart 2^24
        // queries over 2^20 nodes took 1604 instead of 1587 us, 2^26 over 2^22 6450 instead of 6370.)
        if (p.keep_nodes) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (src[i] >= 0) R[i] = *(reinterpret_cast<const u32x4*>(p.nodes + src[i]) + piece);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (src[i] >= 0) R[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p.nodes + src[i]) + piece);
        }
        u32x4 P[8];
        // through LDS in three rounds of 24, 24 and 16 queries (3 KiB of staging); 16-byte pieces are
        // swizzled by the query number so that neither the writes nor the reads collide on banks
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (r * 3 + i < 8) {
                    const int ql = i * 8 + sub;             // query within the round
                    *reinterpret_cast<u32x4*>(stage + ql * 128 + ((piece ^ (ql & 7)) << 4)) = R[(r * 3 + i) & 7];
                }
            }
            wave_lds_sync();
            const int ql = lane - r * 24;
            if (ql >= 0 && ql < 24) {
#pragma unroll
                for (int j = 0; j < 8; ++j) P[j] = *reinterpret_cast<const u32x4*>(stage + ql * 128 + ((j ^ (ql & 7)) << 4));
            }
            wave_lds_sync();
        }
        hd = make_uint4(P[0].x, P[0].y, P[0].z, P[0].w);
#pragma unroll
        for (int j = 0; j < kInlineBlocks; ++j) L[j] = make_uint4(P[1 + j].x, P[1 + j].y, P[1 + j].z, P[1 + j].w);
    } else if (nidx >= 0) {
        // all eight 16-byte pieces are requested at once: the records are needed right after the
        // header for all but empty nodes and long lists
        const uint4* __restrict__ line = reinterpret_cast<const uint4*>(p.nodes + nidx);
        hd = line[0];
#pragma unroll
        for (int j = 0; j < kInlineBlocks; ++j) L[j] = line[1 + j];
    }
    auto before_end = [&](float t) { return INCL ? t <= w.te : t < w.te; };
    // inline list without deleted edges: candidates per block (newest block first) and the blocks that contain the window's
    // end and start
    int32_t cnt[kInlineBlocks];
    int32_t end_block = -1, cut_new = 0, start_block = -1, b_lo = 0, b_n = 0;
    int64_t b_off = 0;
    // Candidates of an inline list once b_lo, the edges of start_block before the window's start, and `inside`, the edges
    // of end_block before the window's end, are known.
    auto count_flat = [&](int32_t inside) {
        int32_t c = 0;
#pragma unroll
        for (int j = 0; j < kInlineBlocks; ++j) {
            if (j == end_block) {
                cut_new = cnt[j] - inside;
                cnt[j] = inside;
            }
            if (j == start_block) cnt[j] = max(cnt[j] - b_lo, 0);
            c += cnt[j];
        }
        return c;
    };
    // Slots 0 .. k-1 from the candidates counted, every slot finding its block among the register counts.
    auto fill_flat = [&](int32_t c, int32_t k) {
#pragma unroll 1
        for (int32_t i = 0; i < k; ++i) {
            int32_t rr = i;               // from the newest candidate
            if (c > f) rr = c - 1 - (int32_t)pick_rank(p.seed, p.qid_base + q, f, i, (uint64_t)c);
            BlockRec r = {};
            int32_t back = -1;            // slots between the picked edge and the end of its block
#pragma unroll
            for (int j = 0; j < kInlineBlocks; ++j) {
                if (back < 0 && rr < cnt[j]) {
                    back = rr + (j == end_block ? cut_new : 0);
                    r.off_lo = L[j].z; r.size_hi = L[j].w;
                }
                rr -= cnt[j];
            }
            w.s_pos[i] = slot_pos<pos_t>(rec_off(r) + rec_size(r) - 1 - back);
        }
    };
    // uniform policy, long list without deleted edges: the run and the candidates [L, R) of the node's sequence
    int32_t long_nb = 0, long_L = 0, long_R = 0;
    uint32_t long_dir = 0;
    if (nidx >= 0) {
        {
            ++n_nodes;
            const int32_t nb = (hd.w & 1) ? 0 : (int32_t)hd.x;      // deleted node: no blocks
            if (!COUNT && nb > 0 && nb <= kInlineBlocks && !(hd.w & 2)) {
                // Inline list without deleted edges.  At most one block contains the window end and at most one its
                // start; the others count as a whole or not at all.  One search each instead of one per block of the unrolled
                // walk.
#pragma unroll
                for (int j = 0; j < kInlineBlocks; ++j) {
                    const BlockRec r = as_rec(L[j]);
                    const bool in = j < nb && before_end(r.t_min) && !(w.tb > r.t_max);
                    cnt[j] = in ? rec_size(r) : 0;
                    if (in && !before_end(r.t_max)) { w.d_off = rec_off(r); w.d_n = rec_size(r); end_block = j; }
                    if (in && w.tb > r.t_min) { b_off = rec_off(r); b_n = rec_size(r); start_block = j; }
                }
                narrow4(w.d_lo, w.d_n, 0, [&](int32_t i) { return before_end(time_at<pos_t>(w.edges, w.d_off + i)); });
                narrow4(b_lo, b_n, 0, [&](int32_t i) { return time_at<pos_t>(w.edges, b_off + i) < w.tb; });
                const int32_t c = count_flat(w.d_lo);
                w.k = min(c, f);
                fill_flat(c, w.k);
            } else if (nb > 0 && nb <= kInlineBlocks) {
                bool go = true;
#pragma unroll
                for (int j = 0; j < kInlineBlocks; ++j)
                    if (go && j < nb) go = w.step(as_rec(L[j]), j);
                if (POLICY == 1 && w.c > (int64_t)f) {
                    w.draw(p.seed, p.qid_base + q);
                    int64_t cum = 0;
#pragma unroll
                    for (int j = 0; j < kInlineBlocks; ++j)
                        if (j >= w.t_first && j <= w.t_last) w.resolve(as_rec(L[j]), j, cum);
                }
            } else if (nb > kInlineBlocks) {
                // long list: all records of the node, oldest first, in one run of the directory
                const int64_t d0 = (int64_t)hd.z * kDirAlign;
                if (POLICY == 1 && d0 + nb <= p.num_dir && !(hd.w & 2)) {
                    // Uniform policy on a long list without deleted edges: the node's edges, blocks
                    // concatenated, form one chronological sequence and the candidates are a contiguous
                    // range [L, R) of it.  With the number of edges before each block kept next to the
                    // records, both ends and every pick cost a binary search over the run instead of
                    // two walks over all overlapping blocks.
                    const BlockRec* __restrict__ d = p.dir + d0;
                    const uint32_t* __restrict__ cum = p.dir_cum + d0;
                    // index in the sequence of the first edge with ts >= x (STRICT: ts > x)
                    auto first_at = [&](float x, auto strict) -> int64_t {
                        constexpr bool STRICT = decltype(strict)::value;
                        auto before = [&](float t) { return STRICT ? t <= x : t < x; };
                        int32_t lo = 0;                   // first block whose newest edge is not before x
                        if (!FUSED) {
                            int32_t hi = nb;
                            while (lo < hi) {
                                const int32_t mid = lo + ((hi - lo) >> 1);
                                ++w.n_blocks;
                                if (before(d[mid].t_max)) lo = mid + 1; else hi = mid;
                            }
                        } else {
                            int32_t n = nb;
                            narrow4(lo, n, 0, [&](int32_t i) { return before(d[i].t_max); });
                        }
                        if (lo == nb) return (int64_t)cum[nb - 1] + rec_size(d[nb - 1]);
                        const BlockRec r = d[lo];
                        ++w.n_blocks;
                        int32_t pos = 0;
                        if (before(r.t_min)) {
                            const int64_t off = rec_off(r);
                            if (!FUSED) {
                                pos = w.template first_not_before<STRICT>(off, rec_size(r), x);
                            } else {
                                int32_t n = rec_size(r) - 1;          // the newest edge is not before x
                                narrow4(pos, n, 0, [&](int32_t i) { return before(time_at<pos_t>(w.edges, off + i)); });
                            }
                        }
                        return (int64_t)cum[lo] + pos;
                    };
                    const int64_t R = first_at(w.te, std::integral_constant<bool, INCL>{});
                    const int64_t L = w.tb == -INFINITY ? 0 : first_at(w.tb, std::false_type{});
                    const int64_t c = R > L ? R - L : 0;
                    w.k = (int32_t)min(c, (int64_t)f);
                    long_nb = nb; long_dir = hd.z; long_L = (int32_t)L; long_R = (int32_t)R;      // slots: below, by the wave
                    if (COUNT) {
                        // byte model: what a binary search per pick reads
                        for (int32_t j = 0; j < w.k; ++j) {
                            const int64_t g = c <= (int64_t)f ? R - 1 - j : L + (int64_t)pick_rank(p.seed, p.qid_base + q, f, j, (uint64_t)c);
                            int32_t lo = 0, hi = nb;          // newest block that starts at or before g
                            while (lo < hi) {
                                const int32_t mid = lo + ((hi - lo) >> 1);
                                ++w.n_probes;
                                if ((int64_t)cum[mid] <= g) lo = mid + 1; else hi = mid;
                            }
                            ++w.n_blocks;
                        }
                    }
                } else if (d0 + nb <= p.num_dir) {
                    const BlockRec* __restrict__ d = p.dir + d0;
                    // newest block that starts before the window end (binary search instead of
                    // stepping through the newer blocks one by one)
                    int32_t lo = 0;
                    if (!FUSED) {
                        int32_t hi = nb;
                        while (lo < hi) {
                            const int32_t mid = lo + ((hi - lo) >> 1);
                            ++w.n_blocks;
                            if (before_end(d[mid].t_min)) lo = mid + 1; else hi = mid;
                        }
                    } else {
                        int32_t n = nb;
                        narrow4(lo, n, 0, [&](int32_t i) { return before_end(d[i].t_min); });
                    }
                    const int32_t j0 = lo - 1;
                    bool go = true;
                    for (int32_t j = j0; j >= 0 && go; --j) go = w.step(d[j], j0 - j);
                    if (POLICY == 1 && w.c > (int64_t)f) {
                        w.draw(p.seed, p.qid_base + q);
                        int64_t cum = 0;
                        for (int32_t t = w.t_first; t <= w.t_last; ++t) w.resolve(d[j0 - t], t, cum);
                    }
                }
            }
        }
    }
    // Uniform policy, picks on long lists: one (query, slot) per lane, kResolve of them side by side, each a binary
    // search over the run's prefix counts.  Neighbouring lanes search the same run, so an instruction touches a dozen
    // lines instead of 64, and the dependent reads of a query's picks overlap instead of following one another
    // (2^23 edges with Zipf(1.1) ids, 2^23 queries, fan-out 10: 2.26 -> 1.92 ms per call).  In the fused kernel, where
    // few waves are resident, the searches over directory runs and their blocks keep three reads in flight and make half
    // the round trips (1.92 -> 1.85 ms); without the scan the plain binary searches are faster (1.53 against 1.59).
    if (POLICY == 1 && !COUNT && __ballot(long_nb > 0)) {
        constexpr int kResolve = 5;
        pos_t* const rows = reinterpret_cast<pos_t*>(my_lds);
        for (int32_t it0 = 0; it0 < f; it0 += kResolve) {
            int32_t lo[kResolve], n[kResolve], g[kResolve];
            uint32_t line[kResolve], dst[kResolve];
            bool any = false;
#pragma unroll
            for (int i = 0; i < kResolve; ++i) {
                lo[i] = 0; n[i] = 0; g[i] = 0; line[i] = 0; dst[i] = 0;
                if (it0 + i < f) {
                    const uint32_t s = (uint32_t)((it0 + i) * kWave + lane);
                    const uint32_t ql = query_of_slot(s, f_mul);
                    const int32_t j = (int32_t)(s - ql * (uint32_t)f);
                    const int32_t nbq = __shfl(long_nb, (int)ql, kWave), Lq = __shfl(long_L, (int)ql, kWave), Rq = __shfl(long_R, (int)ql, kWave);
                    line[i] = (uint32_t)__shfl((int)long_dir, (int)ql, kWave);
                    dst[i] = ql * (uint32_t)stride + (uint32_t)j;
                    const int32_t c = Rq - Lq;
                    if (nbq > 0 && j < min(c, f)) {
                        n[i] = nbq;
                        g[i] = c <= f ? Rq - 1 - j : Lq + (int32_t)pick_rank(p.seed, p.qid_base + q0 + (int64_t)ql, f, j, (uint64_t)c);
                    }
                    any = any || n[i] > 1;
                }
            }
            // newest block that starts at or before g: it is among the n blocks from lo on
            while (!FUSED && __ballot(any)) {
                any = false;
                uint32_t v[kResolve];
#pragma unroll
                for (int i = 0; i < kResolve; ++i) {
                    v[i] = 0;
                    if (n[i] > 1) v[i] = p.dir_cum[(int64_t)line[i] * kDirAlign + lo[i] + (n[i] >> 1)];
                }
#pragma unroll
                for (int i = 0; i < kResolve; ++i) {
                    const int32_t half = n[i] >> 1;
                    if (half > 0) {
                        const bool up = (int32_t)v[i] <= g[i];
                        lo[i] += up ? half : 0;
                        n[i] = up ? n[i] - half : half;
                    }
                    any = any || n[i] > 1;
                }
            }
            while (FUSED && __ballot(any)) {      // three reads per search in flight
                any = false;
                uint32_t v1[kResolve], v2[kResolve], v3[kResolve];
#pragma unroll
                for (int i = 0; i < kResolve; ++i) {
                    v1[i] = v2[i] = v3[i] = 0;
                    if (n[i] > 1) {
                        const uint32_t* __restrict__ run = p.dir_cum + ((int64_t)line[i] * kDirAlign + lo[i]);
                        v1[i] = run[(n[i] + 3) >> 2]; v2[i] = run[n[i] >> 1]; v3[i] = run[(3 * (int64_t)n[i]) >> 2];
                    }
                }
#pragma unroll
                for (int i = 0; i < kResolve; ++i) {
                    if (n[i] > 1) {
                        const int32_t i1 = (n[i] + 3) >> 2, i2 = n[i] >> 1, i3 = (int32_t)((3 * (int64_t)n[i]) >> 2);
                        const bool u1 = (int32_t)v1[i] <= g[i], u2 = (int32_t)v2[i] <= g[i], u3 = (int32_t)v3[i] <= g[i];
                        const int32_t from = u3 ? i3 : (u2 ? i2 : (u1 ? i1 : 0));
                        const int32_t to = !u1 ? i1 : (!u2 ? i2 : (!u3 ? i3 : n[i]));
                        lo[i] += from;
                        n[i] = max(to - from, 1);
                    }
                    any = any || n[i] > 1;
                }
            }
            BlockRec r[kResolve];
            uint32_t cb[kResolve];
#pragma unroll
            for (int i = 0; i < kResolve; ++i) {
                r[i] = BlockRec{}; cb[i] = 0;
                if (n[i] > 0) {
                    r[i] = p.dir[(int64_t)line[i] * kDirAlign + lo[i]];
                    cb[i] = p.dir_cum[(int64_t)line[i] * kDirAlign + lo[i]];
                }
            }
#pragma unroll
            for (int i = 0; i < kResolve; ++i)
                if (n[i] > 0) rows[dst[i]] = slot_pos<pos_t>(rec_off(r[i]) + (g[i] - (int32_t)cb[i]));
        }
    }
    int32_t k = w.k;
    if (COUNT && POLICY == 0 && w.d_off >= 0) {
        // the slots of the window's last block that the search left open
        int32_t h = w.d_lo;
        for (int32_t i = 0; i < w.d_n; ++i) h += before_end(time_at<pos_t>(w.edges, w.d_off + w.d_lo + i)) ? 1 : 0;
        k = min(f, h + w.k);
    }
    if (COUNT) {
        // totals of what this launch reads: node entries, block records, timestamp probes, edges
        unsigned long long v4[4] = {(unsigned long long)n_nodes, (unsigned long long)w.n_blocks,
                                    (unsigned long long)w.n_probes, (unsigned long long)k};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned long long v = v4[i];
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
            if (lane == 0 && v) atomicAdd(&p.counters[i], v);
        }
        return;
    }
    const pos_t* __restrict__ w_pos = reinterpret_cast<const pos_t*>(my_lds);

    auto load = [&](GatherRegs& g, int32_t it0) { gather_load<pos_t, POLICY == 1>(g, p, f_mul, stride, w_pos, lane, it0, k); };
    if constexpr (FUSED) {
        fused_output<false, kVectorSums>(p, &s_tile_base, s_wave_sum, &s_arrived, tc, wave, waves_per_wg, lane, q0, Q, k, f_mul, load);
    } else {
        wave_lds_sync();
        GatherRegs g;
        for (int32_t it0 = 0; it0 < f; it0 += kGatherChunk) {
            load(g, it0);
            store_padded(g, p, lane, it0, q0, Q);
        }
    }
    if (q < Q && p.out_count) __builtin_nontemporal_store(k, &p.out_count[q]);
    if (tc.next(p, &s_tile_base, &s_arrived, lane)) goto sample_tile;
}

// ---- padding removal -------------------------------------------------------------------

// sum of counts per tile of kCompactTile queries
__global__ void __launch_bounds__(256) tns_count_tile_sums(const int32_t* __restrict__ count, int64_t Q,
                                                           const int64_t* __restrict__ Q_dev,
                                                           int32_t* __restrict__ tile_sums) {
    __shared__ int32_t s_w[4];
    if (Q_dev) Q = min(Q, *Q_dev);
    const int64_t base = (int64_t)blockIdx.x * kCompactTile;
    int32_t v = 0;
#pragma unroll
    for (int i = 0; i < kCompactTile / 256; ++i) {
        const int64_t q = base + i * 256 + threadIdx.x;
        if (q < Q) v += count[q];
    }
    const int lane = threadIdx.x & 63;
    v = wave_inclusive_scan(v);
    if (lane == 63) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// exclusive scan of the tile sums (int64), one workgroup; also writes rowptr[Q]
__global__ void __launch_bounds__(1024) tns_scan_tile_sums(const int32_t* __restrict__ tile_sums, int64_t num_tiles,
                                                           int64_t* __restrict__ tile_offs, int64_t* __restrict__ rowptr,
                                                           int64_t Q, const int64_t* __restrict__ Q_dev,
                                                           int64_t* __restrict__ total_out, uint32_t* __restrict__ ws_head) {
    __shared__ int32_t s_w[16];
    __shared__ int64_t s_carry;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < num_tiles; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int32_t v = i < num_tiles ? tile_sums[i] : 0;
        const int32_t inc = wave_inclusive_scan(v);
        if (lane == 63) s_w[wave] = inc;
        __syncthreads();
        int32_t wave_off = 0, all = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int32_t t = s_w[w];
            if (w < wave) wave_off += t;
            all += t;
        }
        const int64_t carry = s_carry;
        if (i < num_tiles) tile_offs[i] = carry + wave_off + (inc - v);
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + all;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (Q_dev) Q = min(Q, *Q_dev);
        rowptr[Q < 0 ? 0 : Q] = s_carry;          // end of rowptr for the actual number of queries
        if (total_out) *total_out = s_carry;
        ws_head[0] = 0;                           // the workspace's status word: no chained scan ran, nothing timed out
        ws_head[1] = 0;
    }
}

// rowptr of the tile's queries and scatter of the filled slots to the dense arrays
__global__ void __launch_bounds__(256) tns_compact_scatter(const CompactArgs a, const int64_t* __restrict__ tile_offs,
                                                           const uint32_t f_magic) {
    __shared__ int32_t s_excl[kCompactTile];
    __shared__ int32_t s_cnt[kCompactTile];
    __shared__ int32_t s_w[4];
    constexpr int kPer = kCompactTile / 256;
    const int64_t Q = a.Q_dev ? min(a.Q, *a.Q_dev) : a.Q;
    const int64_t base = (int64_t)blockIdx.x * kCompactTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t c[kPer];
    int32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int64_t q = base + threadIdx.x * kPer + i;
        c[i] = q < Q ? a.count[q] : 0;
        sum += c[i];
    }
    const int32_t inc = wave_inclusive_scan(sum);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    int32_t excl = inc - sum;
    for (int w = 0; w < wave; ++w) excl += s_w[w];
    const int64_t tile_off = tile_offs[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int ql = threadIdx.x * kPer + i;
        s_excl[ql] = excl;
        s_cnt[ql] = c[i];
        if (base + ql < Q) a.rowptr[base + ql] = tile_off + excl;
        excl += c[i];
    }
    __syncthreads();
    if (!a.cmp_nbr) return;
    const uint32_t f = (uint32_t)a.fanout;
    const uint32_t slots = kCompactTile * f;
    const int64_t in0 = base * f;
    const int64_t in_end = Q * (int64_t)f;
    for (uint32_t s = threadIdx.x; s < slots; s += 256) {
        if (in0 + s >= in_end) break;
        const uint32_t ql = div_by(s, f, f_magic);
        const uint32_t j = s - ql * f;
        if ((int32_t)j < s_cnt[ql]) {
            const int64_t d = tile_off + s_excl[ql] + j;
            a.cmp_nbr[d] = a.nbr[in0 + s];
            a.cmp_eid[d] = a.eid[in0 + s];
            a.cmp_ts[d] = a.ts[in0 + s];
        }
    }
}

// Next hop's instance offsets: instance b's queries of the next hop are the dense entries of its
// queries of this hop, so next[b] = rowptr[cur[b]] (cur[I] = number of queries of this hop).
__global__ void __launch_bounds__(256) tns_hop_inst_rowptr(const int64_t* __restrict__ cur, const int64_t* __restrict__ rowptr,
                                                           int32_t num_instances, int64_t* __restrict__ next) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b <= num_instances) next[b] = rowptr[cur[b]];
}

inline uint32_t magic_for(int32_t f) { return f <= 1 ? 0u : (uint32_t)(((uint64_t(1) << 32) + (uint64_t)f - 1) / (uint64_t)f); }

template <int POLICY, bool INCL, typename pos_t, bool COUNT, bool FUSED>
hipError_t launch_sample_t(const SampleArgs& a, hipStream_t stream) {
    const int32_t stride = a.fanout | 1;                                    // odd: conflict-free per-lane rows
    const size_t per_wave = (size_t)kWave * stride * sizeof(pos_t);
    // per wave: the position rows, and at least the 3 KiB in which the node lines are staged first
    const size_t chunk = std::max<size_t>(per_wave, COUNT ? 0 : 3072);
    // With the padding removal fused in, a workgroup is a tile of the chained scan.  Under the uniform policy the waves of a
    // tile finish far apart (searches and picks) and wait for each other before the dense copy, so small tiles win (C5:
    // 36.5 ms with 16 waves, 32.6 with 8, 31.3 with 4, 34.1 with 2).
    int waves = (int)std::min<size_t>(4, std::max<size_t>(1, (62u << 10) / chunk));
    waves = workgroup_waves(a.Q, a.fanout, waves, FUSED);
    const int64_t per_wg = (int64_t)waves * kWave;
    const int64_t grid = (a.Q + per_wg - 1) / per_wg;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = chunk * waves;
    auto launch = [&](auto scan, const SampleArgs& b) {
        hipLaunchKernelGGL((tns_sample_kernel<POLICY, INCL, pos_t, COUNT, decltype(scan)::value>), dim3((unsigned)grid), dim3(waves * kWave), lds,
                           stream, b, stride, slot_multiplier(a.fanout), (uint32_t)chunk);
    };
    return launch_tiles<FUSED>(a, grid, per_wg, stream, launch);
}

}  // namespace

size_t compact_workspace_least(int64_t Q) {
    // enough for either use: tile sums + offsets of the stand-alone compaction, or the ticket
    // and one state per 64-query wave (the smallest workgroup) of the fused chained scan
    const int64_t tiles = (Q + kCompactTile - 1) / kCompactTile;
    const size_t sums = ((size_t)tiles * sizeof(int32_t) + 255) & ~size_t(255);
    const size_t offs = ((size_t)tiles * sizeof(int64_t) + 255) & ~size_t(255);
    const size_t fused = kScanHeader + (size_t)((Q + kWave - 1) / kWave + 1) * sizeof(uint64_t);
    return std::max(sums + offs + 256, (fused + 255) & ~size_t(255));
}

size_t compact_workspace_bytes(int64_t Q) {
    // (also where this batch's tiles are larger: a smaller batch in the same workspace uses them all)
    const int64_t small_tiles = std::min<int64_t>((Q + kSmallTile - 1) / kSmallTile, kMostSmallTiles);
    return std::max(compact_workspace_least(Q), (kScanHeader + (size_t)(small_tiles + 1) * sizeof(uint64_t) + 255) & ~size_t(255));
}

int64_t tile_states(size_t bytes) { return bytes < kScanHeader ? 0 : (int64_t)((bytes - kScanHeader) / sizeof(uint64_t)); }

hipError_t launch_scan_init(const SampleArgs& a, int64_t num_tiles, hipStream_t stream) {
    const unsigned init_grid = (unsigned)std::max<int64_t>(1, (num_tiles + 255) / 256);
    hipLaunchKernelGGL(tns_scan_init, dim3(init_grid), dim3(256), 0, stream, static_cast<ScanWorkspace*>(a.scan_ws), num_tiles,
                       a.rowptr, a.Q, a.Q_dev, a.total_out, (uint32_t)a.first_ticket);
    return hipGetLastError();
}

bool may_be_replayed(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();      // (no answer, for instance the legacy stream during a capture: the launch reports what is wrong)
    return true;
}

hipError_t ready_tags(SampleArgs& a, int64_t tiles, hipStream_t stream) {
    // splitmix64 from a start of its own: another copy of the library may have left tags in memory that this one is given
    auto start = []() { return (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^ (uint64_t)getpid() << 40; };
    static std::atomic<uint64_t> state{start()};
    do {
        uint64_t z = state.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        a.chain_tag = (z ^ (z >> 31)) >> kTagShift;
    } while (a.chain_tag == 0);      // (what a cleared word holds)
    // one state more than tiles: the workspace has it, and a test whose tiles start at 1 uses it
    return !a.scan_ready && may_be_replayed(stream) ? launch_scan_init(a, tiles + 1, stream) : hipSuccess;
}

hipError_t launch_sample(const SampleArgs& a, hipStream_t stream) {
    if (a.prefix_layout) return launch_sample_prefix(a, stream);
    // Small batches go to the kernel with sixteen lanes per query: up to what the chip holds of it at once, or twice that where
    // every lane of a team has a slot to gather.  us of that kernel / of the one with a query per lane, 2^21 edges: recent
    // policy, fan-out 10, uniform ids, 20000 queries 8.6 / 11.6, 32768 9.3 / 12.0, 49152 13.7 / 13.1, 65536 14.2 / 14.3, power-law ids 11.4 / 16.6,
    // 12.0 / 17.1, 16.8 / 17.9, 19.4 / 19.3; fan-out 20, 32768 11.5 / 17.0 and 15.9 / 21.9, 40000 19.4 / 17.9 and 27.9 / 22.9; fan-out 64,
    // 65536 26.6 / 32.7 and 43.3 / 41.7.  Uniform policy, fan-out 10, uniform ids 9.0 / 12.6, 9.9 / 13.2, 14.5 / 14.6, 15.2 / 15.7, power-law ids
    // 12.7 / 24.6, 13.7 / 26.0, 20.8 / 29.4, 24.2 / 32.4; fan-out 5, 32768 9.3 / 10.8 and 12.9 / 19.2, 65536 14.6 / 11.8 and 21.8 / 23.3.
    static_assert(int64_t(1) << 16 <= tagged_queries(TNS_MAX_FANOUT), "its calls are calls without tickets");
    const int64_t team_max_queries = int64_t(1) << ((a.policy == 0 ? a.fanout <= 32 : a.fanout < 8) ? 15 : 16);
    if (a.scan_ws && !a.counters && a.Q <= team_max_queries) return launch_sample_team(a, stream);
    const bool incl = a.inclusive_end != 0;
    const bool wide = a.wide_offsets != 0;
#define TNS_DISPATCH(POL, CNT, FUS)                                                          \
    (incl ? (wide ? launch_sample_t<POL, true, int64_t, CNT, FUS>(a, stream)                 \
                  : launch_sample_t<POL, true, int32_t, CNT, FUS>(a, stream))                \
          : (wide ? launch_sample_t<POL, false, int64_t, CNT, FUS>(a, stream)                \
                  : launch_sample_t<POL, false, int32_t, CNT, FUS>(a, stream)))
    if (a.counters) return a.policy == 0 ? TNS_DISPATCH(0, true, false) : TNS_DISPATCH(1, true, false);
    if (a.policy == 0) return launch_sample_recent(a, stream);
    return a.scan_ws ? TNS_DISPATCH(1, false, true) : TNS_DISPATCH(1, false, false);
#undef TNS_DISPATCH
}

hipError_t launch_scan_clear(void* ws, size_t bytes, hipStream_t stream) {
    const int64_t words = (int64_t)(bytes / 8);
    if (words > 0)
        hipLaunchKernelGGL(tns_scan_clear, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, static_cast<uint64_t*>(ws), words);
    return hipGetLastError();
}

hipError_t launch_hop_inst_rowptr(const int64_t* cur, const int64_t* rowptr, int32_t num_instances, int64_t* next,
                                  hipStream_t stream) {
    hipLaunchKernelGGL(tns_hop_inst_rowptr, dim3((unsigned)(num_instances / 256 + 1)), dim3(256), 0, stream, cur, rowptr,
                       num_instances, next);
    return hipGetLastError();
}

hipError_t launch_compact(const CompactArgs& a, hipStream_t stream) {
    const int64_t tiles = (a.Q + kCompactTile - 1) / kCompactTile;
    // the first 256 bytes of a workspace hold the status word of the step (read by tns_run_status)
    uint32_t* ws_head = static_cast<uint32_t*>(a.workspace);
    unsigned char* ws = static_cast<unsigned char*>(a.workspace) + 256;
    int32_t* sums = reinterpret_cast<int32_t*>(ws);
    const size_t sums_bytes = ((size_t)tiles * sizeof(int32_t) + 255) & ~size_t(255);
    int64_t* offs = reinterpret_cast<int64_t*>(ws + sums_bytes);
    if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    if (tiles > 0) {
        hipLaunchKernelGGL(tns_count_tile_sums, dim3((unsigned)tiles), dim3(256), 0, stream, a.count, a.Q, a.Q_dev, sums);
    }
    hipLaunchKernelGGL(tns_scan_tile_sums, dim3(1), dim3(1024), 0, stream, sums, tiles, offs, a.rowptr, a.Q, a.Q_dev,
                       a.total_out, ws_head);
    if (tiles > 0) {
        hipLaunchKernelGGL(tns_compact_scatter, dim3((unsigned)tiles), dim3(256), 0, stream, a, offs,
                           magic_for(a.fanout));
    }
    return hipGetLastError();
}

}  // namespace tns
