// Explores every order in which the blocks of a small verification team can
// pass its exchanges, with the library's own numbering of their words.
//   argv[1]: "library", or a numbering that must be found wanting: "one" (one
//   set of words), "level" (sets by the layer alone)
// Prints "ok", or what goes wrong.
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "team_words.h"

using namespace rheo;

static int mode = 0;

static int set_of(uint64_t first, int level) {
    if (mode == 1) return 0;
    if (mode == 2) return level % kTeamSets;
    return team_set(first, level);
}

// An exchange: its epoch and whether it carries sums (one of the sets, 16-bit
// tags) or maxima (a set of their own, 32-bit tags).
struct Exchange {
    uint64_t epoch;
    int words;                           // 0 .. kTeamSets - 1: sums; kTeamSets: maxima
};
static uint64_t tag_of(const Exchange& x) {
    return x.words == kTeamSets ? (uint32_t)x.epoch : team_tag(x.epoch);
}

// A walk: layer l takes its sum exchange (0), that one, the maxima and the sums
// again (1), or the maxima and the sums (2).
static std::vector<Exchange> walk(uint64_t launch, const std::vector<int>& kinds) {
    const uint64_t first = team_first_epoch(launch);
    std::vector<Exchange> w;
    for (int l = 0; l < (int)kinds.size(); ++l) {
        const int s = set_of(first, l);
        if (kinds[l] != 2) w.push_back({first + 3 * l + 1, s});
        if (kinds[l] != 0) {
            w.push_back({first + 3 * l + 2, kTeamSets});
            w.push_back({first + 3 * l + 3, s});
        }
    }
    return w;
}

// Every reachable state of G blocks: 2 i before publishing exchange i, 2 i + 1
// waiting for it.  The words follow from the states: a block's word of a
// set is its last publication there.  Returns false if some state leaves a
// block waiting for good.
static bool never_stuck(int G, const std::vector<Exchange>& w) {
    typedef std::vector<int> State;
    const int end = 2 * (int)w.size();
    std::set<State> seen;
    std::vector<State> todo{State(G, 0)};
    seen.insert(todo[0]);
    auto word = [&](const State& s, int g, int words) -> uint64_t {
        for (int i = (s[g] + 1) / 2 - 1; i >= 0; --i)
            if (w[i].words == words) return tag_of(w[i]);
        return 0;
    };
    while (!todo.empty()) {
        const State s = todo.back();
        todo.pop_back();
        bool moved = false, done = true;
        for (int g = 0; g < G; ++g) {
            if (s[g] == end) continue;
            done = false;
            bool can = true;
            if (s[g] % 2)
                for (int o = 0; o < G; ++o)
                    can &= word(s, o, w[s[g] / 2].words) == tag_of(w[s[g] / 2]);
            if (!can) continue;
            moved = true;
            State n = s;
            ++n[g];
            if (seen.insert(n).second) todo.push_back(n);
        }
        if (!moved && !done) return false;
    }
    return true;
}

int main(int argc, char** argv) {
    if (argc > 1) mode = !strcmp(argv[1], "one") ? 1 : !strcmp(argv[1], "level") ? 2 : 0;
    for (int G = 2; G <= 4; ++G)
        for (int launch = 0; launch < 2; ++launch)
            for (int k = 0; k < 27; ++k)
                if (!never_stuck(G, walk(launch, {k % 3, k / 3 % 3, k / 9}))) {
                    printf("a block of %d waits for good\n", G);
                    return 0;
                }
    // words left by earlier walks, one layer long but for a longer one now and
    // then: none carries the tag of an exchange that has not taken place
    for (int every : {1, 2, 3, 7, 512, 1023, 1024, 1025})
        for (int layers = 1; layers <= 16; ++layers)
            for (int kind = 0; kind < 3; ++kind) {
                uint64_t last[kTeamSets] = {};
                for (int launch = 0; launch < 3000; ++launch)
                    for (const Exchange& x :
                         walk((uint64_t)launch, std::vector<int>(launch % every ? 1 : layers, kind))) {
                        if (x.words == kTeamSets) continue;
                        if (last[x.words] == tag_of(x)) {
                            printf("launch %d: an old word carries a current tag\n", launch);
                            return 0;
                        }
                        last[x.words] = tag_of(x);
                    }
            }
    // a cleared word is no exchange's
    for (uint64_t launch = 0; launch < 70000; ++launch)
        for (int l = 0; l < 16; ++l)
            for (int i = 1; i <= 3; ++i)
                if (team_tag(team_first_epoch(launch) + 3 * l + i) == 0) {
                    printf("launch %d: tag 0\n", (int)launch);
                    return 0;
                }
    printf("ok\n");
    return 0;
}
