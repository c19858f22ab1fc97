// Host-side lockstep harness for the sampling kernel's all-slots-at-once Floyd rule (csrc/zg_floyd.h), compiled
// with g++ by tests/test_floyd_parallel_rule.py.  For every candidate sequence of the given (deg, F) pairs it runs
// floyd_position for all 64 lanes of a wavefront - as many groups of F lanes as fit, one sequence after another, every third
// group a vertex whose neighbors are all taken, and the lanes left over - and compares the positions with the CPU checker's
// sequential zgo_floyd_resolve.
//
// The lanes of a wavefront exchange values in lockstep; here the lanes run one after another, so the harness
// replays the wavefront several times: an exchange returns what the partner lane handed in at the same exchange of
// the previous replay.  The k-th exchange is right from replay k+1 on (it only depends on earlier exchanges), so
// once a replay hands in what the one before did, every lane has seen exactly what a lockstep run would have shown it.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "zg_floyd.h"
#include "zg_oracle.h"

namespace {

constexpr int kLanes = 64;

struct ReplayWave {
    struct Exchange {
        uint32_t value[kLanes];
    };
    std::vector<Exchange> prev, cur; // per exchange, what every lane handed in
    int lane = 0, gbase = 0, at = 0;

    // what the lanes handed in at this exchange of the previous replay, null while there is none
    const Exchange *exchange(uint32_t mine)
    {
        if ((int)cur.size() <= at) cur.push_back(Exchange());
        cur[at].value[lane] = mine;
        const Exchange *e = at < (int)prev.size() ? &prev[at] : nullptr;
        ++at;
        return e;
    }
    uint32_t up(uint32_t x)
    {
        const Exchange *e = exchange(x);
        return e && lane > 0 ? e->value[lane - 1] : 0u;
    }
    bool flag_of(uint32_t j, bool mine)
    {
        const Exchange *e = exchange(mine ? 1u : 0u);
        return e && e->value[gbase + (int)j] != 0;
    }
    bool any(bool b)
    {
        const Exchange *e = exchange(b ? 1u : 0u);
        if (!e) return true; // unknown yet: keep going
        for (int l = 0; l < kLanes; ++l)
            if (e->value[l]) return true;
        return false;
    }
    void begin_lane(int l, int base) { lane = l; gbase = base; at = 0; }
    bool end_replay() // whether nothing changed
    {
        const bool same = prev.size() == cur.size() && (cur.empty() || std::memcmp(prev.data(), cur.data(), cur.size() * sizeof(Exchange)) == 0);
        prev.swap(cur);
        cur.clear();
        return same;
    }
};

// positions of all slots of `rows` (candidate sequences; an empty one: a vertex of F neighbors or less) by the parallel rule
bool parallel_positions(int64_t deg, int F, const std::vector<std::vector<int64_t>> &rows, std::vector<std::vector<int64_t>> &pos)
{
    ReplayWave wave;
    for (int r = 0; r < 3 * F + 8; ++r) {
        for (int l = 0; l < kLanes; ++l) {
            const int group = l / F, slot = l % F;
            const bool active = group < (int)rows.size() && !rows[group].empty();
            wave.begin_lane(l, group * F);
            const uint32_t cand = active ? (uint32_t)rows[group][slot] : (uint32_t)slot;
            const uint32_t p = zg::floyd_position(wave, (uint32_t)group, (uint32_t)slot, (uint32_t)F, active ? (uint32_t)deg : 0u, active, cand);
            if (group < (int)rows.size()) pos[group][slot] = p;
        }
        if (wave.end_replay()) return true;
    }
    return false;
}

} // namespace

int main(int argc, char **argv)
{
    long cases = 0, bad = 0;
    for (int a = 1; a + 1 < argc; a += 2) {
        const int64_t deg = atoll(argv[a]);
        const int F = atoi(argv[a + 1]);
        if (F < 1 || F > kLanes || deg <= F) return 2;
        std::vector<std::vector<int64_t>> rows, pos(kLanes / F, std::vector<int64_t>(F));
        auto run = [&]() {
            std::vector<int64_t> want(F);
            const bool settled = parallel_positions(deg, F, rows, pos);
            for (size_t g = 0; g < rows.size(); ++g) {
                for (int j = 0; j < F; ++j) want[j] = j;
                if (!rows[g].empty()) {
                    zgo_floyd_resolve(deg, F, rows[g].data(), want.data());
                    ++cases;
                }
                if (settled && want == pos[g]) continue;
                if (++bad <= 5) {
                    fprintf(stderr, "deg=%lld F=%d t=", (long long)deg, F);
                    for (int64_t x : rows[g]) fprintf(stderr, "%lld ", (long long)x);
                    fprintf(stderr, "\n");
                }
            }
            rows.clear();
        };
        std::vector<int64_t> t(F, 0);
        for (bool more = true; more;) { // odometer over t_j in [0, deg-F+j]
            if (rows.size() % 3 == 2) rows.push_back({});
            if ((int)rows.size() < kLanes / F) {
                rows.push_back(t);
                int j = F - 1;
                while (j >= 0 && ++t[j] > deg - F + j) t[j--] = 0;
                more = j >= 0;
            }
            if (!more || (int)rows.size() >= kLanes / F) run();
        }
    }
    printf("%ld %ld\n", cases, bad);
    return bad ? 1 : 0;
}
