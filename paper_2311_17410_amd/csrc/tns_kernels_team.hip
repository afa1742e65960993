// gfx950 sampling kernel for small batches (default layout): Algorithm 1 of the paper (section 4.2), the padded write and
// the padding removal of section 5 fused in, with sixteen lanes working on one query.
//
// tns_sample_kernel gives every lane a query of its own, which keeps the most independent reads in flight once a
// batch fills the chip.  A batch that does not fill it is bound by the length of one wave's program instead: with 64
// queries per wave the search and the gather are 16 and 10 unrolled loads with their address arithmetic, fetched once
// from a cold instruction cache (1024 queries: 16 us, of which 3.5 us each in the walk, the search and the gather).
// Here a team of sixteen lanes holds one query in registers, every step is one instruction for the whole query, and
// the program is short:
//   node      eight lanes read the node line, lane b then holds the record of the b-th oldest block
//   window    a node's blocks, concatenated, are one chronological sequence; its candidates are a range [L, R) of
//             it.  Each end is the block that contains it (ballot over the records, or sixteen-way search over a
//             directory run) and the position inside (sixteen-way search over the block's timestamps: one round for
//             blocks of up to 16 edges, four for 8192)
//   gather    lane j takes slot j: its rank (newest first, or its own pick), the block that holds it, the edge.
//             Under the uniform policy the f picks of a query are resolved side by side instead of one after the
//             other.
//   deleted   a node whose flags say that edges of it are deleted has its candidates looked at, sixteen side by side.
//             The flag is read here and not on the host: a captured call may be replayed after a deletion.
// What bounds it is the chain of dependent reads (query, node, search, edge, look-back) and, between them, the instructions of the
// waves that share a SIMD.  Its tiles tag what they publish instead of having the scan state cleared by a launch before it and
// tickets taken (TaggedChain).  A team is a row of sixteen lanes, so that what it shares moves within vector instructions (row_read,
// row_up) and not through the LDS unit, the waves' sums are added up side by side, a block's position is divided by the slots per
// line once, and small batches take small workgroups (launch_team_t).  The kernel, us: 1024 queries over 2^10 edges 7.6 -> 5.9, two
// hops from 600 roots 7.0 + 7.5 -> 5.9 + 6.3, from 4000 under the uniform policy 8.2 + 16.0 -> 6.0 + 13.0; per call 14.2 -> 12.1 and
// 23.7 -> 19.7.  Measured beside the kernels with a query per lane: see the rule in launch_sample.
#include <algorithm>
#include <type_traits>

#include "../../include/tns.h"
#include "tns_device.h"
#include "tns_kernels.h"

namespace tns {
namespace {

constexpr int kTeam = 16;
constexpr int kTeamsPerWave = kWave / kTeam;
constexpr int64_t kComputeUnits = 256;
constexpr int kTileWaves = 16, kFewWaves = 4;      // of the largest workgroups (every workspace holds a tile state per 64 queries) and the smallest
constexpr int64_t kFewQueries = 512;               // up to so many the smallest workgroups are not the best

// For each of CH independent ranges: number of leading items of [0, n) for which qual(u, i) holds (the items for which
// it holds come first), found by the team together: sixteen probes a round, the rounds of all ranges side by side.
// n is the same in all lanes of a team; called by the whole wave.
template <int CH, class Qual>
__device__ __forceinline__ void team_partition(int32_t (&n)[CH], int32_t (&lo)[CH], int lane, const Qual& qual) {
    const int j = lane & (kTeam - 1), shift = lane & ~(kTeam - 1);
    bool any = false;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        lo[u] = 0;
        any = any || n[u] > 0;
    }
    while (__ballot(any)) {
        bool ok[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int32_t s = (n[u] + kTeam - 1) / kTeam;
            ok[u] = n[u] > 0 && qual(u, lo[u] + min((j + 1) * s - 1, n[u] - 1));
        }
        any = false;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int32_t s = (n[u] + kTeam - 1) / kTeam;
            const int32_t cnt = __popcll((__ballot(ok[u]) >> shift) & 0xffffull);
            // the first cnt probes qualify, the next one does not: the answer is less than s items further on
            const int32_t step = min(cnt * s, n[u]);
            lo[u] += step;
            n[u] = max(min(s - 1, n[u] - step), 0);
            any = any || n[u] > 0;
        }
    }
}

// CH: queries per team, all steps of which run side by side; ROUNDS: of sixteen slots
template <int POLICY, bool INCL, int CH, int ROUNDS>
__global__ void __launch_bounds__(kTileWaves * kWave, CH * ROUNDS <= 2 ? 8 : 4) tns_sample_team_kernel(const SampleArgs args) {
    const int tile_waves = (int)(blockDim.x >> 6), tile_queries = tile_waves * kTeamsPerWave * CH;
    __shared__ int64_t s_tile_base;
    __shared__ int32_t s_wave_sum[kTileWaves];
    __shared__ int32_t s_arrived, s_todo;
    __shared__ int32_t s_seq[kTileWaves][CH][kTeamsPerWave][ROUNDS * kTeam];      // nodes with deleted edges: the slots' edges
    int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int32_t f = args.fanout;
    const int64_t Q = args.Q_dev ? min(args.Q, *args.Q_dev) : args.Q;
    // later hops are launched for the most queries they can have: workgroups beyond the actual number leave at once
    if ((int64_t)blockIdx.x * tile_queries >= Q) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {      // no query will write the end of rowptr
            args.rowptr[0] = 0;
            if (args.total_out) *args.total_out = 0;
        }
        return;
    }
    int64_t tile = (int64_t)blockIdx.x + args.first_ticket;
    if (tile * tile_queries >= Q) return;      // (tests whose tiles start at 1)
    if (threadIdx.x == 0) s_arrived = s_todo = 0;
    __syncthreads();
    TaggedChain chain;
    chain.s_todo = &s_todo;
sample_tile:
    new_tile(lane, wave);
    const SampleArgs& p = arguments_anew();
    chain.begin(p.scan_ws, p.chain_tag, tile);
    const int j = lane & (kTeam - 1), team0 = lane & ~(kTeam - 1);
    // a wave's queries are consecutive: team t of the wave has q0 + u * 4 + t
    const int64_t q0 = tile * tile_queries + wave * (kTeamsPerWave * CH) + (lane >> 4);

    // ---- the queries and their nodes ---------------------------------------------------------
    float te[CH], tb[CH];
    int32_t v[CH];
    int64_t nidx[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int64_t q = q0 + u * kTeamsPerWave;
        v[u] = -1; te[u] = 0.0f; tb[u] = 0.0f;
        if (q < Q) {
            v[u] = p.targets[q];
            te[u] = p.t_end[q];
            if (p.t_start) tb[u] = p.t_start[q];
        }
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        if (!p.t_start) tb[u] = p.delta == INFINITY ? -INFINITY : te[u] - p.delta;
        nidx[u] = (uint32_t)v[u] < (uint64_t)p.num_nodes && !(te[u] != te[u]) && !(tb[u] != tb[u]) ? v[u] : -1;
        if (q0 + u * kTeamsPerWave >= Q) nidx[u] = -1;
    }
    if (p.inst_rowptr) {
        // instance b owns queries inst_rowptr[b] .. inst_rowptr[b+1]-1
        int32_t n[CH], b[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) n[u] = q0 + u * kTeamsPerWave < Q ? p.num_instances : 0;
        team_partition<CH>(n, b, lane, [&](int u, int32_t i) { return p.inst_rowptr[i + 1] <= q0 + u * kTeamsPerWave; });
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            if (b[u] >= p.num_instances) nidx[u] = -1;
            if (nidx[u] >= 0) nidx[u] += (int64_t)b[u] * p.num_nodes;
        }
    }
    u32x4 piece[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        piece[u] = u32x4{0u, 0u, 0u, 0u};
        if (nidx[u] >= 0 && j < 8) piece[u] = *(reinterpret_cast<const u32x4*>(p.nodes + nidx[u]) + j);
    }
    int32_t nb_in[CH], nb_long[CH];     // blocks in the node line / in the directory run (one of them is 0)
    uint32_t dline[CH];                 // start of the run in units of kDirAlign records
    BlockRec rec[CH];                   // lane b: record of the b-th oldest block
    int32_t cum[CH];                    // lane b: edges in the older blocks; last lane of the team: the node's flags
    int32_t piv[CH];                    // long lists: lane b: edges in the blocks before the (b * piv_step)-th
    bool any_long = false;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        int32_t nb = row_read<0>((int)piece[u].x);
        dline[u] = (uint32_t)row_read<0>((int)piece[u].z);
        const int32_t flags = row_read<0>((int)piece[u].w);
        if (flags & 1) nb = 0;                                                       // deleted node: no blocks
        if (nb > kInlineBlocks && (int64_t)dline[u] * kDirAlign + nb > p.num_dir) nb = 0;
        nb_in[u] = nb > kInlineBlocks ? 0 : nb;
        nb_long[u] = nb - nb_in[u];
        any_long = any_long || nb_long[u] > 0;
        const int src = team0 + max(nb_in[u] - j, 0);          // inline records are stored newest first
        rec[u].t_min = __uint_as_float((uint32_t)__shfl((int)piece[u].x, src, kWave));
        rec[u].t_max = __uint_as_float((uint32_t)__shfl((int)piece[u].y, src, kWave));
        rec[u].off_lo = (uint32_t)__shfl((int)piece[u].z, src, kWave);
        rec[u].size_hi = (uint32_t)__shfl((int)piece[u].w, src, kWave);
        const int32_t size = j < nb_in[u] ? rec_size(rec[u]) : 0;
        cum[u] = size + row_up<1>(size);
        cum[u] += row_up<2>(cum[u]);
        cum[u] += row_up<4>(cum[u]);
        cum[u] = j == kTeam - 1 ? flags : cum[u] - size;
        piv[u] = 0;
        if (nb_long[u] > 0) piv[u] = (int32_t)p.dir_cum[(int64_t)dline[u] * kDirAlign + min(j * ((nb_long[u] + kTeam - 1) / kTeam), nb_long[u] - 1)];
    }
    any_long = __ballot(any_long) != 0;

    // ---- the window [L, R) in a node's sequence of edges --------------------------------------
    // index of the first edge with ts >= x (STRICT: ts > x)
    auto first_at = [&](const float (&x)[CH], int32_t (&at)[CH], auto strict) {
        constexpr bool STRICT = decltype(strict)::value;
        auto before = [&](int u, float t) { return STRICT ? t <= x[u] : t < x[u]; };
        int32_t b[CH], n[CH], base[CH], size[CH], pos[CH];
        const uint32_t* edges[CH];      // of the block that the search goes through
        uint32_t edges_at[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) b[u] = __popcll((__ballot(j < nb_in[u] && before(u, rec[u].t_max)) >> team0) & 0xffffull);
        if (any_long) {
            int32_t bl[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u) n[u] = nb_long[u];
            team_partition<CH>(n, bl, lane, [&](int u, int32_t i) { return before(u, p.dir[(int64_t)dline[u] * kDirAlign + i].t_max); });
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (nb_long[u] > 0) b[u] = bl[u];
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int32_t nb = nb_in[u] + nb_long[u], bb = max(min(b[u], nb - 1), 0);
            const int src = team0 + (nb_in[u] > 0 ? bb : 0);
            BlockRec r;
            r.t_min = __shfl(rec[u].t_min, src, kWave);
            r.off_lo = (uint32_t)__shfl((int)rec[u].off_lo, src, kWave);
            r.size_hi = (uint32_t)__shfl((int)rec[u].size_hi, src, kWave);
            base[u] = __shfl(cum[u], src, kWave);
            if (nb_long[u] > 0) {
                r = p.dir[(int64_t)dline[u] * kDirAlign + bb];
                base[u] = (int32_t)p.dir_cum[(int64_t)dline[u] * kDirAlign + bb];
            }
            size[u] = rec_size(r);
            const BlockWords words(r);
            edges[u] = p.edges + words.base;
            edges_at[u] = words.at;
            // the block's newest edge is not before x: one item less to search
            n[u] = (b[u] < nb && before(u, r.t_min)) ? size[u] - 1 : 0;
        }
        team_partition<CH>(n, pos, lane, [&](int u, int32_t i) { return before(u, __uint_as_float(edges[u][words_behind(edges_at[u] + (uint32_t)i)])); });
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int32_t nb = nb_in[u] + nb_long[u];
            at[u] = nb <= 0 ? 0 : base[u] + (b[u] >= nb ? size[u] : pos[u]);
        }
    };
    int32_t R[CH], L[CH], c[CH], k[CH];
    first_at(te, R, std::integral_constant<bool, INCL>{});
    bool windowed = false;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        L[u] = 0;
        windowed = windowed || tb[u] > -INFINITY;
    }
    if (__ballot(windowed)) first_at(tb, L, std::false_type{});

#pragma unroll
    for (int u = 0; u < CH; ++u) c[u] = max(R[u] - L[u], 0);

    // ---- nodes with deleted edges: which candidates are there ------------------------------------
    // Whether edge g of the node's sequence is there, for the lanes that ask; called by the whole wave.
    auto present = [&](int u, int32_t g, bool ask) {
        int32_t b = -1;
#pragma unroll 1
        for (int t = 0; t < kInlineBlocks; ++t) b += (t < nb_in[u] && __shfl(cum[u], team0 + t, kWave) <= g) ? 1 : 0;
        const int src = team0 + max(b, 0);
        BlockRec r;
        r.off_lo = (uint32_t)__shfl((int)rec[u].off_lo, src, kWave);
        r.size_hi = (uint32_t)__shfl((int)rec[u].size_hi, src, kWave);
        int32_t before = __shfl(cum[u], src, kWave);
        if (!ask) return false;
        if (nb_long[u] > 0) {
            uint32_t run = dline[u];
            asm volatile("" : "+v"(run));      // an address of its own: one shared with the searches would be kept in registers all along
            const int64_t d0 = (int64_t)run * kDirAlign;
            int32_t lo = 0, n = nb_long[u];
            while (n > 1) {
                const int32_t half = n >> 1;
                const bool up = (int32_t)p.dir_cum[d0 + lo + half] <= g;
                lo += up ? half : 0;
                n = up ? n - half : half;
            }
            r = p.dir[d0 + lo];
            before = (int32_t)p.dir_cum[d0 + lo];
        }
        return (int32_t)p.edges[slot_word(rec_off(r) + (g - before)) + 2] >= 0;      // the edge id word
    };
    bool any_holes = false;             // of the wave's nodes
#pragma unroll
    for (int u = 0; u < CH; ++u) any_holes = any_holes || (j == kTeam - 1 && (cum[u] & 2));
    any_holes = __ballot(any_holes) != 0;
    if (any_holes) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const bool holes = __shfl(cum[u], team0 + kTeam - 1, kWave) & 2;
            // how many of the candidates are there; the recent policy needs no more than f of them
            int32_t at = R[u], n = 0;
            bool go = holes && c[u] > 0;
            while (__ballot(go)) {
                n += __popcll((__ballot(present(u, at - 1 - j, go && at - 1 - j >= L[u])) >> team0) & 0xffffull);
                at -= kTeam;
                go = go && at > L[u] && (POLICY == 1 || n < f);
            }
            if (holes) c[u] = n;
            // the slots' edges: each the one with a given number of newer ones that are there
#pragma unroll 1
            for (int32_t slot_no = j; slot_no < ROUNDS * kTeam; slot_no += kTeam) {
                int32_t newer = slot_no, g = R[u] - 1 - slot_no;
                go = holes && slot_no < min(c[u], f);
                if (POLICY == 1 && go && c[u] > f)
                    newer = c[u] - 1 - (int32_t)pick_rank(p.seed, p.qid_base + q0 + u * kTeamsPerWave, f, slot_no, (uint64_t)c[u]);
                at = R[u];
                n = 0;
                while (true) {
                    const uint64_t open = (__ballot(go) >> team0) & 0xffffull;
                    if (!__ballot(open != 0)) break;
                    uint32_t there = (uint32_t)(__ballot(present(u, at - 1 - j, open != 0 && at - 1 - j >= L[u])) >> team0) & 0xffffu;
                    const int32_t cnt = __popc(there);
                    if (go && newer < n + cnt) {
                        for (int32_t s = newer - n; s > 0; --s) there &= there - 1;
                        g = at - __ffs((int)there);
                        go = false;
                    }
                    n += cnt;
                    at -= kTeam;
                    go = go && at > L[u];
                }
                s_seq[wave][u][lane >> 4][slot_no] = g;
            }
        }
        wave_lds_sync();
    }

    // ---- dense offsets inside the workgroup -----------------------------------------------------
    int32_t excl_in_wave[CH], wave_total = 0;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        k[u] = min(c[u], f);
        const int32_t k0 = wave_read(k[u], 0), k1 = wave_read(k[u], 16), k2 = wave_read(k[u], 32), k3 = wave_read(k[u], 48);
        excl_in_wave[u] = wave_total + (lane >= 16 ? k0 : 0) + (lane >= 32 ? k1 : 0) + (lane >= 48 ? k2 : 0);
        wave_total += k0 + k1 + k2 + k3;
    }
    chain.begun();
    int is_last = 0;
    if (lane == 0) {
        s_wave_sum[wave] = wave_total;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        is_last = __hip_atomic_fetch_add(&s_arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == tile_waves - 1;
    }
    is_last = wave_uniform(is_last);
    int32_t wg_total = 0;
    if (is_last) {
        // the wave that arrives last publishes the tile total at once, so that later tiles can look past this one
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        wg_total = sum_of_waves(s_wave_sum, tile_waves, lane);
        if (lane == 0) chain.publish(tile, wg_total);
    }

    // ---- slots: rank -> block -> edge -----------------------------------------------------------
    Edge e[CH][ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        int32_t g[CH], cb[CH], lo[CH], hi[CH];
        BlockRec rb[CH];
        const int32_t slot_no = r * kTeam + j;
        bool any = false;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            e[u][r].ts = 0.0f; e[u][r].nbr = -1; e[u][r].eid = -1;
            any = any || slot_no < k[u];
        }
        if (!__ballot(any)) continue;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            g[u] = R[u] - 1 - slot_no;                // newest first; so too when all candidates are taken
            if (POLICY == 1 && slot_no < k[u] && c[u] > f)
                g[u] = L[u] + (int32_t)pick_rank(p.seed, p.qid_base + q0 + u * kTeamsPerWave, f, slot_no, (uint64_t)c[u]);
            if (any_holes && (row_read<kTeam - 1>(cum[u]) & 2)) g[u] = s_seq[wave][u][lane >> 4][slot_no];
            // newest inline block that starts at or before g
            int32_t b = -1;
            auto from = [&](auto t) { b += t.value < nb_in[u] && row_read<t.value>(cum[u]) <= g[u] ? 1 : 0; };
            from(std::integral_constant<int, 0>{});
            from(std::integral_constant<int, 1>{});
            from(std::integral_constant<int, 2>{});
            from(std::integral_constant<int, 3>{});
            from(std::integral_constant<int, 4>{});
            from(std::integral_constant<int, 5>{});
            from(std::integral_constant<int, 6>{});
            static_assert(kInlineBlocks == 7, "every block of a node line");
            const int src = team0 + max(b, 0);
            rb[u].off_lo = (uint32_t)__shfl((int)rec[u].off_lo, src, kWave);
            rb[u].size_hi = (uint32_t)__shfl((int)rec[u].size_hi, src, kWave);
            cb[u] = __shfl(cum[u], src, kWave);
        }
        if (any_long) {
            bool more = false;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const int32_t piv_step = (nb_long[u] + kTeam - 1) / kTeam;
                int32_t lo16 = 0;
#pragma unroll
                for (int d = kTeam / 2; d >= 1; d >>= 1) {
                    const int32_t t = lo16 + d;
                    const int32_t w = __shfl(piv[u], team0 + t, kWave);
                    if (t * piv_step < nb_long[u] && w <= g[u]) lo16 = t;
                }
                lo[u] = lo16 * piv_step;
                hi[u] = slot_no < k[u] ? min(lo[u] + piv_step, nb_long[u]) : lo[u];
                more = more || hi[u] - lo[u] > 1;
            }
            while (__ballot(more)) {
                more = false;
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    const int32_t mid = lo[u] + ((hi[u] - lo[u]) >> 1);
                    if (hi[u] - lo[u] > 1) {
                        if ((int32_t)p.dir_cum[(int64_t)dline[u] * kDirAlign + mid] <= g[u]) lo[u] = mid; else hi[u] = mid;
                    }
                    more = more || hi[u] - lo[u] > 1;
                }
            }
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (nb_long[u] > 0 && slot_no < k[u]) {
                    rb[u] = p.dir[(int64_t)dline[u] * kDirAlign + lo[u]];
                    cb[u] = (int32_t)p.dir_cum[(int64_t)dline[u] * kDirAlign + lo[u]];
                }
        }
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (slot_no < k[u]) {
                const BlockWords words(rb[u]);
                e[u][r] = *reinterpret_cast<const Edge*>(p.edges + words.base + words.words_to(g[u] - cb[u]));
            }
    }

    // ---- outputs --------------------------------------------------------------------------------
    if (is_last) {
        const int64_t excl = chain.exclusive(tile, lane, p.defer_spins, [](int32_t v) { return wave_sum(v); });
        if (lane == 0) s_tile_base = excl;
    }
    if (p.out_nbr) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int64_t q = q0 + u * kTeamsPerWave;
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                const int32_t slot_no = r * kTeam + j;
                if (q < Q && slot_no < f) {
                    const int64_t o = q * f + slot_no;
                    __builtin_nontemporal_store(e[u][r].nbr, &p.out_nbr[o]);
                    __builtin_nontemporal_store(e[u][r].eid, &p.out_eid[o]);
                    __builtin_nontemporal_store(e[u][r].ts, &p.out_ts[o]);
                }
            }
        }
    }
    lds_barrier();
    const int64_t tile_row = s_tile_base, wave_row = tile_row + sum_of_waves(s_wave_sum, wave, lane);
    const bool dense = tile_row >= 0;      // (or another workgroup writes them)
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int64_t q = q0 + u * kTeamsPerWave;
        const int64_t row = wave_row + excl_in_wave[u];
        if (q >= Q) continue;
        if (j == 0 && p.out_count) p.out_count[q] = k[u];
        if (!dense) continue;
        if (j == 0) {
            p.rowptr[q] = row;
            if (q == Q - 1) {
                // (a call in which a wait ran out: 0, so that a hop chained to this one has no queries)
                const int64_t tot = chain.close(p.err_flag) ? 0 : row + k[u];
                p.rowptr[Q] = tot;
                if (p.total_out) *p.total_out = tot;
            }
        }
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const int32_t slot_no = r * kTeam + j;
            if (slot_no < k[u]) {
                p.cmp_nbr[row + slot_no] = e[u][r].nbr;
                p.cmp_eid[row + slot_no] = e[u][r].eid;
                p.cmp_ts[row + slot_no] = e[u][r].ts;
            }
        }
    }
    if (chain.next(tile, tile_queries, &s_tile_base, &s_arrived, lane, [&]() { return call_of(p); })) goto sample_tile;
}

template <int POLICY, bool INCL, int CH, int ROUNDS>
hipError_t launch_team_t(const SampleArgs& a, hipStream_t stream) {
    static_assert(kTileWaves * kTeamsPerWave * CH * ROUNDS * kTeam < (1 << kTotalBits), "a tile's total lies below the tag");
    // Workgroups as small as leave no more of them than compute units, if the workspace has room for the states of their tiles:
    // sixteen waves of one workgroup issue four to a SIMD in step, and what a step costs is then mostly their turns.  us, 16 / 8 / 4
    // waves, uniform ids and recent policy, the others alike: 600 queries 7.0 / 6.2 / 6.3, 1000 6.6 / 5.9 / 5.8, 4000 6.5 / 6.5 / 6.1, 8000
    // 6.7 / 6.2 / 6.7, 16000 7.1 / 7.4 / 7.1; 100 queries 5.7 / 5.6 / 6.2 and over power-law ids 6.7 / 6.5 / 7.3.
    auto tiles = [&](int waves) { return (a.Q + waves * kTeamsPerWave * CH - 1) / (waves * kTeamsPerWave * CH); };
    static_assert(kFewWaves * kTeamsPerWave == kSmallTile && kMostSmallTiles == kComputeUnits, "the workspace has room for the states of the smallest tiles");
    int waves = a.Q <= kFewQueries ? 2 * kFewWaves : kFewWaves;
    while (waves < kTileWaves && (tiles(waves) > kComputeUnits || tiles(waves) >= a.scan_states)) waves *= 2;
    const int64_t grid = tiles(waves);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    if (grid <= 0) return a.scan_ready ? hipGetLastError() : launch_scan_init(a, 1, stream);
    SampleArgs b = a;
    if (!b.err_flag) b.err_flag = &static_cast<ScanWorkspace*>(a.scan_ws)->error;
    const hipError_t e = ready_tags(b, grid, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((tns_sample_team_kernel<POLICY, INCL, CH, ROUNDS>), dim3((unsigned)grid), dim3(waves * kWave), 0, stream, b);
    return hipGetLastError();
}

template <int POLICY, bool INCL>
hipError_t launch_team_p(const SampleArgs& a, hipStream_t stream) {
    constexpr int kAllRounds = 4;
    static_assert(kAllRounds * kTeam >= TNS_MAX_FANOUT, "rounds cover the largest fan-out");
    // Queries per team: one while that many fit the chip side by side, or one and a half times as many where the slots are one round;
    // two beyond.  us with one / two, 2^21 edges, uniform and power-law ids: recent policy, fan-out 10, 20000 queries 8.6 / 9.4 and 11.4 /
    // 12.5, 32768 9.3 / 10.1 and 12.0 / 13.7, 49152 13.7 / 14.0 and 16.8 / 19.1, 65536 16.5 / 14.2 and 20.8 / 19.4; fan-out 64, 10000 8.1 / 10.7
    // and 12.6 / 19.2, 20000 14.5 / 11.4 and 22.9 / 21.1; uniform policy, fan-out 10, 49152 14.5 / 14.9 and 20.8 / 22.3, 65536 17.3 / 15.2 and
    // 25.0 / 24.2; fan-out 64, 10000 8.4 / 11.4 and 16.9 / 25.1, 20000 14.7 / 11.8 and 32.6 / 29.0.
    const bool one = a.Q <= kComputeUnits * (int64_t)(kTileWaves * kTeamsPerWave) * (a.fanout > kTeam ? 1 : 3);
    if (a.fanout > kTeam) return one ? launch_team_t<POLICY, INCL, 1, kAllRounds>(a, stream) : launch_team_t<POLICY, INCL, 2, kAllRounds>(a, stream);
    return one ? launch_team_t<POLICY, INCL, 1, 1>(a, stream) : launch_team_t<POLICY, INCL, 2, 1>(a, stream);
}

}  // namespace

hipError_t launch_sample_team(const SampleArgs& a, hipStream_t stream) {
    if (a.policy == 0) return a.inclusive_end ? launch_team_p<0, true>(a, stream) : launch_team_p<0, false>(a, stream);
    return a.inclusive_end ? launch_team_p<1, true>(a, stream) : launch_team_p<1, false>(a, stream);
}

}  // namespace tns
