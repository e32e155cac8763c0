// How the words of a verification team's sum exchange are numbered (plain
// integer functions, the same on the host, where a test explores every order in which
// a team's blocks can run).
//
// A launch's exchanges use the epochs of a window of 64: three per layer of a
// walk of at most 16 layers.  A sum word carries its epoch's low 16 bits, and
// waiting for it tests them for equality, since the word holds the sum of
// that exchange alone.  A block that has all sums of a layer may publish the
// next layer's before a slower one has looked at this layer's, so consecutive
// layers use two sets of words in turn: publishing into a set again takes the
// sums of the layer between, which the slower block publishes only after it
// has left its wait.  Launches start with the sets in turn as well, so no
// word is left unwritten for more than two launches and an old one never
// carries a current tag.
#pragma once

#include <cstdint>

namespace rheo {

constexpr int kTeamSets = 2;
constexpr uint64_t team_first_epoch(uint64_t launch) { return 64 * (launch + 1); }
constexpr uint64_t team_tag(uint64_t epoch) { return epoch & 0xFFFFu; }
constexpr int team_set(uint64_t first_epoch, int level) {
    return (int)((first_epoch / 64 + (uint64_t)level) % kTeamSets);
}

}  // namespace rheo
