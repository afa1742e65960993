// gfx950 sampling kernel for a store in the prefix layout (tns_layout.h) under the uniform policy, and the counting pass of
// both policies (the recent policy is sampled by tns_sample_recent_kernel): Algorithm 1 of the paper (section 4.2) with the
// padded write of section 4.2's kernel notes and the padding removal of section 5 fused in, as in tns_kernels.hip.
//
// Node lines are read eight lanes per line, 16 bytes each, and handed to the owning lane through LDS; the lane counts the
// qualifying slots of its own line in registers.  Then it walks the blocks: directory records for the blocks outside the prefix,
// newest first, then the prefix line by line as if every line were a block.
#include <algorithm>
#include <type_traits>

#include "tns_device.h"
#include "tns_kernels.h"

namespace tns {
namespace {

constexpr int kMaxFastFanout = kSlotsPerLine;

__device__ __forceinline__ int ceil_log2_outcomes(int n) { return n <= 0 ? 0 : 32 - __clz(n); }   // probes of a binary search over n sorted items

// Uniform policy: workgroups of at most eight waves, three of them per compute unit (80 registers; at 85, with two of
// them, 2^22 queries took 447 us windowed and 478 without a window instead of 405 and 459); small grids have two at most.
template <int POLICY, bool INCL, typename pos_t, bool COUNT, int SCAN>
__global__ void __launch_bounds__(POLICY == 1 ? 512 : 1024, POLICY == 1 && !COUNT && SCAN != kTags ? 6 : 4) tns_sample_prefix_kernel(const SampleArgs args, const int32_t rs, const uint32_t f_mul,
                                                                 const int32_t gshift, const uint32_t chunk) {
    constexpr bool FUSED = SCAN != kNoScan;
    static_assert(POLICY == 1 || (COUNT && !FUSED), "the recent policy is sampled by tns_sample_recent_kernel");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int64_t s_tile_base;
    __shared__ int32_t s_wave_sum[16];
    __shared__ int32_t s_arrived;
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
    unsigned char* const my_lds = smem + (size_t)wave * chunk;
    uint32_t* const rows = reinterpret_cast<uint32_t*>(my_lds);
    const uint32_t* __restrict__ lines = p.edges;

    // ---- the query and its node ------------------------------------------------------------
    float te = 0.0f, tb = 0.0f;
    int64_t nidx = -1;
    const int32_t inst = p.inst_rowptr ? instance_of(p.inst_rowptr, p.num_instances, q0, q, Q, lane) : 0;
    if (q < Q) {
        const int32_t v = __builtin_nontemporal_load(&p.targets[q]);
        te = __builtin_nontemporal_load(&p.t_end[q]);
        tb = p.t_start ? p.t_start[q] : (p.delta == INFINITY ? -INFINITY : te - p.delta);
        int64_t nbase = 0;
        bool ok = (uint32_t)v < (uint64_t)p.num_nodes && !(te != te) && !(tb != tb);
        if (p.inst_rowptr) {
            ok = ok && inst < p.num_instances;
            nbase = (int64_t)inst * p.num_nodes;
        }
        if (ok) nidx = nbase + v;
    }
    tc.begin(p);
    // ---- node lines: eight lanes per line, handed over through LDS ------------------------------------
    uint32_t w[3 * kInlineSlots];     // the eight edge slots of the node's own line
    uint32_t h_degree, h_meta, h_ext0, h_ext12, h_fence0, h_fence1, h_fence2, h_dir;   // the node entry
    {
        const int piece = lane & 7, sub = lane >> 3;
        u32x4 R[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t src = shfl64(nidx, i * 8 + sub);
            R[i] = u32x4{0u, 0u, 0u, 0u};
            if (src >= 0) R[i] = *(reinterpret_cast<const u32x4*>(lines + src * 32) + piece);
        }
        // through LDS in two rounds of 32 queries (4 KiB of staging); 16-byte pieces are swizzled by the query
        // number so that neither the writes nor the reads collide on banks
        u32x4 v6 = u32x4{0u, 0u, 0u, 0u}, v7 = v6;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ql = i * 8 + sub;             // query within the round
                *reinterpret_cast<u32x4*>(my_lds + ql * 128 + ((piece ^ (ql & 7)) << 4)) = R[r * 4 + i];
            }
            wave_lds_sync();
            if ((lane >> 5) == r) {
                const int ql = lane & 31;
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(my_lds + ql * 128 + ((j ^ (ql & 7)) << 4));
                    w[4 * j] = v.x; w[4 * j + 1] = v.y; w[4 * j + 2] = v.z; w[4 * j + 3] = v.w;
                }
                v6 = *reinterpret_cast<const u32x4*>(my_lds + ql * 128 + ((6 ^ (ql & 7)) << 4));
                v7 = *reinterpret_cast<const u32x4*>(my_lds + ql * 128 + ((7 ^ (ql & 7)) << 4));
            }
            wave_lds_sync();
        }
        h_degree = v6.x; h_meta = v6.y; h_ext0 = v6.z; h_ext12 = v6.w;
        h_fence0 = v7.x; h_fence1 = v7.y; h_fence2 = v7.z; h_dir = v7.w;
    }
    static_assert(kNodeHdrWord == 24 && sizeof(PrefixNodeHdr) == 32, "the node entry is the last two 16-byte pieces of the line");
    // ---- per query: where the window end falls ----------------------------------------------------
    const int32_t degree = (int32_t)h_degree;
    const uint32_t meta = h_meta;
    const bool alive = nidx >= 0 && !(meta & 1u) && degree > 0;
    const bool tomb = (meta & 2u) != 0;
    const int32_t nbig = pmeta_big_blocks(meta);
    const int32_t fill = min(degree, pmeta_prefix_slots(meta));       // edges stored in the prefix
    const int32_t n_in = min(fill, kInlineSlots);
    const int32_t n_ext = fill <= kInlineSlots ? 0 : (fill - kInlineSlots + kSlotsPerLine - 1) / kSlotsPerLine;
    // extension line x (0..2) and its fence, selected without indexing registers by a run-time value
    auto ext_line = [&](int32_t x) -> uint32_t { return x == 0 ? h_ext0 : h_ext12 + (uint32_t)(x - 1); };
    auto fence = [&](int32_t x) -> float { return __uint_as_float(x == 0 ? h_fence0 : (x == 1 ? h_fence1 : h_fence2)); };
    const bool fast = POLICY == 0 && f <= kMaxFastFanout && alive && !tomb && nbig == 0;
    const bool walked = alive && !fast;
    uint32_t* const my_row = rows + lane * rs;
    int32_t k = 0;
    int32_t n_blocks = 0, n_probes = 0;       // byte model (COUNT)

    // ---- byte model of the recent policy on nodes of short lists ------------------------------------------
    // The extension line that holds the window end (-1: the node's own line) follows from the fences alone.
    int32_t e = -1;
    if (fast) {
#pragma unroll
        for (int j = 0; j < kPrefixExtLines; ++j)
            if (j < n_ext && (INCL ? (fence(j) <= te) : (fence(j) < te))) e = j;
    }
    // slots of the node's own line before the window end / before the window start
    int32_t hi_in = 0, lo_in = 0;
#pragma unroll
    for (int i = 0; i < kInlineSlots; ++i) {
        const float t = __uint_as_float(w[3 * i]);
        hi_in += (i < n_in && (INCL ? (t <= te) : (t < te))) ? 1 : 0;
        lo_in += (i < n_in && t < tb) ? 1 : 0;
    }
    if (fast && e < 0) {
        k = max(min(f, hi_in - lo_in), 0);
        n_probes += ceil_log2_outcomes(n_in) + (tb > -INFINITY ? ceil_log2_outcomes(hi_in) : 0);
    } else if (fast) {
        // the line with the window end, then the line before it where slots are left
        const int32_t n_e = min(fill - kInlineSlots - kSlotsPerLine * e, kSlotsPerLine);
        const uint32_t* src = lines + (uint64_t)ext_line(e) * 32u;
        int r1 = 0, l1 = 0;
        for (int x = 0; x < n_e; ++x) {
            const float t = __uint_as_float(src[3 * x]);
            r1 += (INCL ? (t <= te) : (t < te)) ? 1 : 0;
            l1 += t < tb ? 1 : 0;
        }
        k = max(r1 - max(l1, r1 - f), 0);
        n_probes += ceil_log2_outcomes(n_e) + (tb > -INFINITY ? ceil_log2_outcomes(r1) : 0);
        if (l1 == 0 && k < f) {
            if (e == 0) {
                k += min(f - k, kInlineSlots - lo_in);
                if (tb > -INFINITY) n_probes += ceil_log2_outcomes(kInlineSlots);
            } else {
                int l2 = 0;
                src = lines + (uint64_t)ext_line(e - 1) * 32u;
                for (int x = 0; x < kSlotsPerLine; ++x) l2 += __uint_as_float(src[3 * x]) < tb ? 1 : 0;
                k += max(kSlotsPerLine - max(l2, kSlotsPerLine - (f - k)), 0);
                if (tb > -INFINITY) n_probes += ceil_log2_outcomes(kSlotsPerLine);
            }
        }
    }
    // ---- queries that walk the blocks (Algorithm 1 per lane) -------------------------------------------
    Walk<POLICY, INCL, pos_t> wk;
    wk.f = f;
    wk.s_pos = reinterpret_cast<pos_t*>(my_row);
    wk.edges = lines;
    wk.group = (POLICY == 0 && gshift >= 0) ? (1 << gshift) : 0;
    wk.te = te;
    wk.tb = tb;
    if (walked) {
        // the node's blocks, newest first: blocks outside the prefix (records in the directory run, oldest
        // first), then the prefix line by line.  A prefix line is presented as a block record whose latest
        // time is an upper bound (the next fence), which the walk's tests allow.
        const int64_t d0 = (int64_t)h_dir * kDirAlign;
        const bool dir_ok = nbig > 0 && d0 + nbig <= p.num_dir;
        const BlockRec* __restrict__ d = p.dir + d0;
        int32_t j0 = -1;                       // newest block outside the prefix that starts before the window end
        if (dir_ok) {
            int32_t lo = 0, hi = nbig;
            while (lo < hi) {
                const int32_t mid = lo + ((hi - lo) >> 1);
                const float tm = d[mid].t_min;
                ++wk.n_blocks;
                if (INCL ? (tm > te) : (tm >= te)) hi = mid; else lo = mid + 1;
            }
            j0 = lo - 1;
        }
        const int32_t n_big_walk = j0 + 1;     // visiting numbers 0 .. n_big_walk-1 are directory blocks
        const float after_prefix = dir_ok ? d[0].t_min : INFINITY;
        auto prefix_rec = [&](int32_t line_no) -> BlockRec {        // line_no: 0 = own line, 1..3 = extension lines
            if (line_no == 0)
                return make_rec(__uint_as_float(w[0]), n_ext > 0 ? fence(0) : after_prefix, nidx * kSlotsPerLine, n_in, tomb);
            const int32_t x = line_no - 1;
            const int32_t n = min(fill - kInlineSlots - kSlotsPerLine * x, kSlotsPerLine);
            return make_rec(fence(x), x + 1 < n_ext ? fence(x + 1) : after_prefix, (int64_t)ext_line(x) * kSlotsPerLine, n, tomb);
        };
        auto rec_at = [&](int32_t t) -> BlockRec {                   // record of visiting number t
            return t < n_big_walk ? d[j0 - t] : prefix_rec(n_ext - (t - n_big_walk));
        };
        bool go = true;
        int32_t t = 0;
        for (; t < n_big_walk && go; ++t) go = wk.step(d[j0 - t], t);
        for (int32_t x = n_ext; x >= 1 && go; --x, ++t) go = wk.step(prefix_rec(x), t);
        if (go && n_in > 0) {
            // the node's own line: both window ends are known from the registers
            ++wk.n_blocks;
            wk.n_probes += ceil_log2_outcomes(n_in) + (tb > -INFINITY ? ceil_log2_outcomes(hi_in) : 0);
            if (hi_in > lo_in) wk.record(nidx * kSlotsPerLine, lo_in, hi_in, tomb, n_big_walk + n_ext);
        }
        if (POLICY == 1 && wk.c > (int64_t)f) {
            wk.draw(p.seed, p.qid_base + q);
            int64_t cum = 0;
            for (int32_t u = wk.t_first; u <= wk.t_last; ++u) wk.resolve(rec_at(u), u, cum);
        }
    }
    if (walked) {
        int32_t h = 0;
        if (POLICY == 0 && wk.d_off >= 0) {
            // the slots of the window's last block that the walk left open
            h = wk.d_lo;
            for (int32_t i = 0; i < wk.d_n; ++i) {
                const float t = time_at<pos_t>(lines, wk.d_off + wk.d_lo + i);
                h += (INCL ? (t <= te) : (t < te)) ? 1 : 0;
            }
        }
        k = POLICY == 0 ? min(f, h + wk.k) : wk.k;
        n_blocks += wk.n_blocks;
        n_probes += wk.n_probes;
    }
    if (COUNT) {
        unsigned long long v4[4] = {(unsigned long long)(nidx >= 0 ? 1 : 0), (unsigned long long)n_blocks,
                                    (unsigned long long)n_probes, (unsigned long long)k};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned long long v = v4[i];
            for (int dd = 32; dd >= 1; dd >>= 1) v += __shfl_xor(v, dd, kWave);
            if (lane == 0 && v) atomicAdd(&p.counters[i], v);
        }
        return;
    }
    const pos_t* __restrict__ w_pos = reinterpret_cast<const pos_t*>(rows);
    wave_lds_sync();      // rows were written by this wave's own lanes

    // ---- outputs --------------------------------------------------------------------------------------
    auto load = [&](GatherRegs& g, int32_t it0) {
        gather_load<pos_t, POLICY == 1>(g, p, f_mul, rs * 4 / (int32_t)sizeof(pos_t), w_pos, lane, it0, k);
    };
    if constexpr (FUSED) {
        fused_output<false, SCAN == kTickets ? kShuffled : kLargeShuffled>(p, &s_tile_base, s_wave_sum, &s_arrived, tc, wave, waves_per_wg, lane, q0, Q, k, f_mul, load);
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

template <int POLICY, bool INCL, typename pos_t, bool COUNT, bool FUSED>
hipError_t launch_prefix_t(const SampleArgs& a, hipStream_t stream) {
    const int32_t f = a.fanout;
    const int32_t rs = (f | 1) * (int32_t)(sizeof(pos_t) / 4);       // row stride in 4-byte words: odd (conflict-free per-lane rows) in positions
    const size_t rows_bytes = ((size_t)kWave * rs * 4 + 15) & ~size_t(15);
    const int32_t gshift = (POLICY == 0 && f <= kCoopGroup) ? 4 : -1;
    // per wave: the position rows; at least the 4 KiB in which the node lines are staged first, 32 at a time
    const size_t chunk = std::max<size_t>(rows_bytes, 4096);
    // Workgroup size.  With the padding removal fused in, a workgroup is a tile of the chained scan (C5 at 2^26 queries 7.10 /
    // 6.91 / 7.83 ms with 4 / 8 / 16 waves).  Without the scan small workgroups come and go more evenly.
    int waves = FUSED ? 8 : 2;
    while (waves > 1 && (size_t)waves * chunk > (size_t)(159u << 10)) --waves;      // LDS of a workgroup: 160 KiB
    waves = workgroup_waves(a.Q, a.fanout, waves, FUSED, true);
    const int64_t per_wg = (int64_t)waves * kWave;
    const int64_t grid = (a.Q + per_wg - 1) / per_wg;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = chunk * waves;
    auto launch = [&](auto scan, const SampleArgs& b) {
        hipLaunchKernelGGL((tns_sample_prefix_kernel<POLICY, INCL, pos_t, COUNT, decltype(scan)::value>), dim3((unsigned)grid), dim3(waves * kWave),
                           lds, stream, b, rs, slot_multiplier(f), gshift, (uint32_t)chunk);
    };
    return launch_tiles<FUSED>(a, grid, per_wg, stream, launch);
}

}  // namespace

hipError_t launch_sample_prefix(const SampleArgs& a, hipStream_t stream) {
    const bool incl = a.inclusive_end != 0;
    const bool wide = a.wide_offsets != 0;
#define TNS_DISPATCH(POL, CNT, FUS)                                                          \
    (incl ? (wide ? launch_prefix_t<POL, true, int64_t, CNT, FUS>(a, stream)                 \
                  : launch_prefix_t<POL, true, int32_t, CNT, FUS>(a, stream))                \
          : (wide ? launch_prefix_t<POL, false, int64_t, CNT, FUS>(a, stream)                \
                  : launch_prefix_t<POL, false, int32_t, CNT, FUS>(a, stream)))
    if (a.counters) return a.policy == 0 ? TNS_DISPATCH(0, true, false) : TNS_DISPATCH(1, true, false);
    if (a.policy == 0) return launch_sample_recent(a, stream);
    return a.scan_ws ? TNS_DISPATCH(1, false, true) : TNS_DISPATCH(1, false, false);
#undef TNS_DISPATCH
}

}  // namespace tns
