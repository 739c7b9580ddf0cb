// Slots of the counters that the proposal rounds of a one-workgroup solver
// share (rows still looking, whether anyone proposed).
//
// A round of slot s reads its rows' counts in slot s and counts its losers in
// losers_slot(s); after the barrier that ends it, every wave looks there
// whether the phase is over. If it is, the next phase counts its rows in
// phase_slot(s), with no barrier in between: a wave that is late to look must
// not find them, so this is the third slot. Thread 0 clears the two other
// slots between the barriers around a round's scan (cleared_by). Their last
// readers passed a barrier before: of the round before this one, its rows'
// counts (read before that round's last barrier) and its end test (read
// before the barrier that starts a phase, or the slot is this round's own).
// Their next writers, this round's losers and then the next phase's rows,
// come after the barrier that ends the scan.
#pragma once

#ifdef __HIPCC__
#define PROT_SLOT_FN __host__ __device__ constexpr
#else
#define PROT_SLOT_FN constexpr
#endif

namespace prot {

constexpr int kRoundSlots = 3;
PROT_SLOT_FN int losers_slot(int s) { return s == kRoundSlots - 1 ? 0 : s + 1; }
PROT_SLOT_FN int phase_slot(int s) { return losers_slot(losers_slot(s)); }
// whether thread 0 clears slot i at the start of a round of slot s
PROT_SLOT_FN bool cleared_by(int s, int i) { return i != s; }

}  // namespace prot
