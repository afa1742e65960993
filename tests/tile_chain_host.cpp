// Tiles that tag what they publish (csrc/tns_chain.h), on the host: the rows of every tile and the end of the last one, in many
// orders of the lanes' accesses.  Arguments: first seed, number of seeds.
#include <cstring>

#include "tns_chain.h"

using namespace tns;

static int try_once(uint32_t seed) {
    std::mt19937 rng(seed);
    const int tiles = 1 + (int)(rng() % 8), spins = (int)(rng() % 4) - 1, per_tile = 1 + (int)(rng() % 5);
    const int resident = 1 + (int)(rng() % (unsigned)tiles);
    const int lost = rng() % 8 == 0;                      // tile 0 never exists
    const int64_t queries = (int64_t)tiles * per_tile - (int)(rng() % (unsigned)per_tile);
    std::vector<uint64_t> words(64 + tiles);
    for (uint64_t& w : words) w = rng() % 2 ? 0 : (uint64_t)rng() << 32 | rng();
    auto* ws = reinterpret_cast<ScanWorkspace*>(words.data());
    const uint64_t tag = ((uint64_t)rng() << 32 | rng()) >> kTagShift;
    std::vector<int> count(tiles * sim::kWaves);
    for (int& c : count) c = (int)(rng() % 900);
    std::vector<int64_t> row(tiles * sim::kWaves, -3);
    int64_t end = -3, total_out = -3;
    uint32_t err = rng();
    int wrong = 0;
    const bool went = sim::run(tiles - lost, resident, rng, [&](sim::Group& g, int t) {
        const int lane = t % sim::kLanes, wave = t / sim::kLanes;
        int64_t tile = g.id + lost;
        if (t == 0) g.arrived = g.todo = 0;
        __syncthreads();
        TaggedChain chain;
        chain.s_todo = &g.todo;
        do {
            chain.begin(ws, tag, tile);
            chain.begun();
            int last = 0;
            if (lane == 0) {
                g.wave_sum[wave] = count[tile * sim::kWaves + wave];
                last = g.arrived++ == sim::kWaves - 1;
            }
            last = __shfl(last, 0, sim::kLanes);
            int total = 0;
            if (last) {
                for (int w = 0; w < sim::kWaves; ++w) total += g.wave_sum[w];
                if (lane == 0) chain.publish(tile, total);
                const int64_t before = chain.exclusive(tile, lane, spins, [](int32_t v) {
                    for (int d = sim::kLanes / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, sim::kLanes);
                    return v;
                });
                if (lane == 0) g.base = before;
            }
            __syncthreads();
            int64_t at = g.base;
            if (at >= 0) {
                for (int w = 0; w < wave; ++w) at += g.wave_sum[w];
                if (lane == 0) row[tile * sim::kWaves + wave] = at;
                if (lane == 0 && wave == sim::kWaves - 1 && tile == tiles - 1) {
                    end = total_out = chain.close(&err) ? 0 : at + count[tile * sim::kWaves + wave];
                }
            }
        } while (chain.next(tile, per_tile, &g.base, &g.arrived, lane, [&]() { return TaggedChain::Call{queries, &end, &total_out, &err}; }));
    });
    if (!went) { std::printf("seed %u: nothing goes on\n", seed); return 1; }
    if (lost) {
        for (int64_t r : row) wrong += r != -3;
        if (tiles > 1) wrong += end != 0 || total_out != 0 || err == 0;
        if (wrong) std::printf("seed %u: %d tiles, the first one missing: end %lld, error word %u\n", seed, tiles, (long long)end, err);
        return wrong;
    }
    int64_t at = 0;
    for (size_t i = 0; i < row.size(); ++i) {
        if (row[i] != at) { std::printf("seed %u: %d tiles, row of wave %zu is %lld, not %lld\n", seed, tiles, i, (long long)row[i], (long long)at); ++wrong; }
        at += count[i];
    }
    if (end != at || total_out != at || err != 0) { std::printf("seed %u: end %lld, not %lld, error word %u\n", seed, (long long)end, (long long)at, err); ++wrong; }
    return wrong;
}

int main(int, char** argv) {
    const uint32_t first = (uint32_t)std::atoi(argv[1]), n = (uint32_t)std::atoi(argv[2]);
    int wrong = 0;
    for (uint32_t s = first; s < first + n && wrong < 5; ++s) wrong += try_once(s);
    return wrong ? 1 : 0;
}
