// What csrc/tns_chain.h needs of the HIP runtime, for the host: workgroups of two waves run as fibers, one per lane, of one
// thread.  A random scheduler (seeded, so that a run can be repeated) decides at every access to global memory which lane goes
// on; cross-lane operations and barriers wait for the lanes that take part.  What a lane stores reaches the others some time later,
// stores to different places in any order, or when the lane waits for its stores.
#pragma once
#include <setjmp.h>
#include <ucontext.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <random>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0

namespace sim {
constexpr int kLanes = 64, kWaves = 2;
struct Dim { unsigned x; };
struct Meeting {                   // of the lanes of a wave, or of a workgroup
    int live = 0, here = 0;
    unsigned gen = 0;
    uint64_t in[kLanes], out[kLanes];
    void close() {
        if (here != live || here == 0) return;
        for (int i = 0; i < kLanes; ++i) out[i] = in[i];
        here = 0;
        ++gen;
    }
};
struct Group;
struct Fiber {
    ucontext_t ctx;                // where it begins
    jmp_buf at;                    // where it goes on
    bool begun = false;
    std::unique_ptr<char[]> stack;
    Group* group;
    Dim tid;
    bool done = false;
    const unsigned* waits_for = nullptr;
    unsigned waits_past = 0;
    bool ready() const { return !done && (!waits_for || *waits_for != waits_past); }
};
struct Group {
    int id;
    bool started = false;
    Meeting wave[kWaves], all;
    int weight[kWaves];
    std::vector<Fiber> lane;
    int live = 0;
    int64_t base;                  // the program's LDS
    int32_t wave_sum[kWaves], arrived, todo;
};
inline Fiber* me;
struct Stored {                    // and not yet seen by others
    Fiber* by;
    void* at;
    uint64_t value;
    int bytes;
};
inline std::vector<Stored> on_their_way;
inline void arrive(size_t i) {
    const Stored s = on_their_way[i];
    on_their_way.erase(on_their_way.begin() + (long)i);
    std::memcpy(s.at, &s.value, (size_t)s.bytes);
}
inline size_t first_of_place(size_t i) {
    for (size_t j = 0; j < i; ++j)
        if (on_their_way[j].by == on_their_way[i].by && on_their_way[j].at == on_their_way[i].at) return j;
    return i;
}
inline void wait_for_stores(const void* at = nullptr) {        // of this lane (to one place)
    for (size_t i = 0; i < on_their_way.size();)
        if (on_their_way[i].by == me && (!at || on_their_way[i].at == at)) arrive(i);
        else ++i;
}
inline jmp_buf scheduler;
inline void pause() {
    if (!_setjmp(me->at)) _longjmp(scheduler, 1);
}
inline void go_on(Fiber& f) {
    me = &f;
    if (_setjmp(scheduler)) return;
    if (f.begun) _longjmp(f.at, 1);
    f.begun = true;
    setcontext(&f.ctx);
}
inline void meet(Meeting& m) {
    const unsigned gen = m.gen;
    ++m.here;
    m.close();
    while (m.gen == gen) {
        me->waits_for = &m.gen;
        me->waits_past = gen;
        pause();
    }
    me->waits_for = nullptr;
}
inline Meeting& my_wave() { return me->group->wave[me->tid.x / kLanes]; }
inline Meeting& among_lanes(uint64_t v) {
    Meeting& m = my_wave();
    m.in[me->tid.x % kLanes] = v;
    meet(m);
    return m;
}
inline uint64_t ballot(bool p) {
    const Meeting& m = among_lanes(p);
    uint64_t r = 0;
    for (int i = 0; i < kLanes; ++i) r |= (m.out[i] & 1) << i;
    return r;
}
template <class T> T from_lane(T v, int src) { return (T)among_lanes((uint64_t)(int64_t)v).out[src]; }

// Runs `program` in `groups` workgroups, at most `resident` at a time, started in a random order.  False if nothing can go on.
template <class Program>
bool run(int groups, int resident, std::mt19937& rng, const Program& program) {
    static const Program* entry;
    entry = &program;
    auto main_of_lane = +[]() {
        (*entry)(*me->group, (int)me->tid.x);
        Fiber* f = me;
        Group& g = *f->group;
        f->done = true;
        --g.live;
        Meeting& w = g.wave[f->tid.x / kLanes];
        --w.live;
        --g.all.live;
        w.close();
        g.all.close();
        pause();
    };
    std::vector<Group> all(groups);
    std::vector<int> order(groups);
    for (int i = 0; i < groups; ++i) {
        order[i] = i;
        all[i].id = i;
        all[i].lane.resize(kWaves * kLanes);
        all[i].live = all[i].all.live = kWaves * kLanes;
        for (int w = 0; w < kWaves; ++w) {
            all[i].wave[w].live = kLanes;
            all[i].weight[w] = 1 << (rng() % 12);         // waves of very different speeds
        }
        for (int t = 0; t < kWaves * kLanes; ++t) {
            Fiber& f = all[i].lane[t];
            f.group = &all[i];
            f.tid.x = (unsigned)t;
        }
    }
    for (int i = groups - 1; i > 0; --i) std::swap(order[i], order[rng() % (i + 1)]);
    int begun = 0;
    for (long step = 0; step < 40000000; ++step) {
        int running = 0;
        long total = 0;
        for (Group& g : all) running += g.started && g.live > 0;
        if (begun < groups && running < resident && (running == 0 || rng() % 64 == 0)) {
            Group& g = all[order[begun++]];
            g.started = true;
            for (Fiber& f : g.lane) {
                f.stack.reset(new char[16384]);
                getcontext(&f.ctx);
                f.ctx.uc_stack.ss_sp = f.stack.get();
                f.ctx.uc_stack.ss_size = 16384;
                f.ctx.uc_link = nullptr;
                makecontext(&f.ctx, main_of_lane, 0);
            }
            ++running;
        }
        if (running == 0) {
            while (!on_their_way.empty()) arrive(0);
            return true;
        }
        if (!on_their_way.empty() && rng() % 32 == 0) arrive(first_of_place(rng() % on_their_way.size()));
        struct Choice { Group* g; int w; };
        static std::vector<Choice> can;
        can.clear();
        for (Group& g : all) {
            if (!g.started || g.live == 0) continue;
            for (int w = 0; w < kWaves; ++w)
                for (int l = 0; l < kLanes; ++l)
                    if (g.lane[w * kLanes + l].ready()) {
                        can.push_back({&g, w});
                        total += g.weight[w];
                        break;
                    }
        }
        if (can.empty()) {
            if (!on_their_way.empty()) { arrive(0); continue; }
            if (begun < groups && running < resident) continue;
            return false;
        }
        long at = (long)(rng() % (unsigned long)total);
        size_t c = 0;
        while ((at -= can[c].g->weight[can[c].w]) >= 0) ++c;
        const int first = (int)(rng() % kLanes), most = rng() % 8 ? kLanes : 1 + (int)(rng() % kLanes);
        for (int l = 0, ran = 0; l < kLanes && ran < most; ++l) {
            Fiber& f = can[c].g->lane[can[c].w * kLanes + (first + l) % kLanes];
            if (!f.ready()) continue;
            go_on(f);
            ++ran;
        }
    }
    return false;
}
template <class T, class V> void store(T* p, V v) {
    pause();
    Stored s{me, p, 0, (int)sizeof(T)};
    const T value = (T)v;
    std::memcpy(&s.value, &value, sizeof(T));
    on_their_way.push_back(s);
}
template <class T> T load(const T* p) {
    pause();
    T v = *p;
    for (const Stored& s : on_their_way)
        if (s.by == me && s.at == p) std::memcpy(&v, &s.value, sizeof(T));
    return v;
}
template <class T> void before_change(T* p) { pause(); wait_for_stores(p); }
template <class T, class V> T exchange(T* p, V v) { before_change(p); T o = *p; *p = (T)v; return o; }
template <class T, class V> T fetch_or(T* p, V v) { before_change(p); T o = *p; *p |= (T)v; return o; }
template <class T, class V> T fetch_and(T* p, V v) { before_change(p); T o = *p; *p &= (T)v; return o; }
template <class T, class V> T fetch_add(T* p, V v) { before_change(p); T o = *p; *p += (T)v; return o; }
}  // namespace sim

#define threadIdx (sim::me->tid)
#define __hip_atomic_store(p, v, o, s) sim::store(p, v)
#define __hip_atomic_load(p, o, s) sim::load(p)
#define __hip_atomic_exchange(p, v, o, s) sim::exchange(p, v)
#define __hip_atomic_fetch_or(p, v, o, s) sim::fetch_or(p, v)
#define __hip_atomic_fetch_and(p, v, o, s) sim::fetch_and(p, v)
#define __hip_atomic_fetch_add(p, v, o, s) sim::fetch_add(p, v)
inline uint32_t atomicExch(uint32_t* p, uint32_t v) { return sim::exchange(p, v); }
inline void __threadfence() { sim::wait_for_stores(); }
inline void __syncthreads() { sim::meet(sim::me->group->all); }
inline uint64_t __ballot(bool p) { return sim::ballot(p); }
template <class T> T __shfl(T v, int src, int) { return sim::from_lane(v, src); }
template <class T> T __shfl_xor(T v, int d, int) { return sim::from_lane(v, (int)(sim::me->tid.x % sim::kLanes) ^ d); }
#define __builtin_amdgcn_readfirstlane(v) sim::from_lane((int)(v), 0)
#define __builtin_amdgcn_s_sleep(n) sim::pause()
#define __builtin_amdgcn_s_waitcnt(n) sim::wait_for_stores()
#define __builtin_amdgcn_wave_barrier() (void)sim::among_lanes(0)
