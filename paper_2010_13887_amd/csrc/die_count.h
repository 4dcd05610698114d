// How a launch with a group of rows per die (kernels_stack_die.hip) knows that its workgroups were dealt to the dies as it needs them.
// No device code: tests/host_checks.cpp plays through placements.
#pragma once
#include <stdint.h>

namespace lsq {

constexpr int kDies = 8;
constexpr int kDieGroup = 32;          // workgroups of a group: one per compute unit of a die

// Every workgroup of a launch adds its word to one of 64 bits: the low half counts workgroups, the high half, four bits per die, those whose
// place in their group is the first (blocks 0 to 7, so no field can run over).  A group that lacks a place but has another waits for it and
// gives up; one without any workgroup has nobody who could, and its rows would stay what they were: it lacks the first place too.
constexpr uint64_t die_word(int die, int place) { return 1 + (place == 0 ? uint64_t{1} << (32 + 4 * die) : 0); }
constexpr bool die_launch_ends(uint64_t before) { return (uint32_t)before == kDies * kDieGroup - 1; }   // with this workgroup
constexpr bool die_groups_there(uint64_t after, int groups) {
  for (int g = 0; g < groups; ++g)
    if ((after >> (32 + 4 * g) & 15) == 0) return false;
  return true;
}

// A workgroup of a die to spare that goes on behind its word (it has the vocabulary product): the last workgroup of the launch to add its word moves
// the launch counter on, which says which of the two sets this launch exchanges in.  So only the first thread looks at the counter, draws the
// workgroup's columns and hands both on to the other wavefronts; `leave` adds the word once look and draw are over (both are complete when the
// function that is passed returns).
template <typename Look, typename Draw, typename Hand, typename Leave>
constexpr void die_spare_signs_off(Look look, Draw draw, Hand hand, Leave leave) {
  const int seq = look();
  const int columns = draw();
  hand(seq, columns);
  leave();
}

}  // namespace lsq
