// Boundary words of kOutEdges: PBs of D % 8 != 0 bits (D > 8) share the byte at
// each boundary between two of them.  Each brings its bits of the byte to the
// boundary's word with an exchange; the second finds the first's there and
// writes the byte.  A word names the call that left it, so what an earlier call
// left behind (whole, half done or spoilt by another decode that ran at the same
// time) is taken for an empty word.
#pragma once

#include <stdint.h>

namespace pbvd {

// Calls are numbered 1 .. kEdgeCalls - 1; when the numbers start again the words
// are cleared.  A captured call, whose number is that of every replay, is number
// 0 and clears its words first.
constexpr uint32_t kEdgeCalls = 1u << 23;

// The word a PB of call `call` leaves: bits within the byte, flag, call.
constexpr uint32_t edge_word(uint32_t call, uint32_t bits) { return call << 9 | 0x100u | bits; }
// Whether the word found in place of `mine` is the other PB's.
constexpr bool edge_second(uint32_t mine, uint32_t found) { return (mine ^ found) >> 8 == 0; }
// Number of the call after `call`.
constexpr uint32_t edge_next_call(uint32_t call) { return call + 1 < kEdgeCalls ? call + 1 : 1; }

}  // namespace pbvd
