// Reading back what the tag body stores (pbvd_tags.hpp): the decisions that the
// tags of a wave's slot name, for the survivor export.  A row of a slot holds the
// tags of one group of four stages; the tag of a state at the group's end is the
// origin of its survivor at the group's start, which is four decisions.  States
// inside a group have a decision here only where a survivor of the group's end
// passes through them.  Plain functions of numbers, for the host and the device.
#pragma once

#include <stdint.h>

namespace pbvd {
namespace tag_view {

constexpr int kStages = 4;  // stages per group and decisions per tag

constexpr int gcd(int a, int b) { return b == 0 ? a : gcd(b, a % b); }
// Stages per trip: a wave's PBs end with its last trip.
constexpr int trip(int V) { return V / gcd(V, kStages) * kStages; }
// Position of a state after the stage of phase ph - 1.
constexpr uint32_t position(uint32_t state, int ph, int V) {
    return ph % V == 0 ? state : ((state << (ph % V) | state >> (V - ph % V)) & ((1u << V) - 1u));
}

// Tag of the PB in place `slot` of its wave (2^lb lanes per PB) at position u, from
// row `row` of the wave's slot `sp`: registers r, r + 1 and the two with their
// second highest index bit set share a dword, a byte per half and a nibble per
// that bit; a lane's dwords are stored in pairs.
constexpr uint32_t stored_tag(const uint32_t *sp, int64_t row, int slot, uint32_t u, int V, int lb) {
    const int nr = (1 << (V - 1)) >> lb, ndw = nr / kStages;
    const uint32_t half = u >> (V - 1), full = u & ((1u << (V - 1)) - 1u);
    const uint32_t r = full & (uint32_t)(nr - 1);
    const int64_t lane = (int64_t)slot << lb | full >> (V - 1 - lb);
    const uint32_t top = r >> (V - 2 - lb), low = r & ((1u << (V - 2 - lb)) - 1u);
    const uint32_t dw = low >> 1;
    return sp[row * ndw * 64 + (dw >> 1) * 128 + lane * 2 + (dw & 1)] >> (16 * (low & 1) + 8 * half + 4 * top) & 15u;
}

// The decision (0 / 1) that the stored tags name for `state` after the stage
// `back` stages before the end of its wave (0: the last), or -1 where no
// survivor of the group's end passes through it.  rows: rows of the slot, the
// last one at the wave's end.  Where survivors disagree (they cannot, unless a
// tag is wrong) the one that is not `want` wins.
constexpr int stored_decision(const uint32_t *sp, int64_t rows, int slot, int64_t back, uint32_t state, int V, int lb,
                              int want) {
    const int64_t g = back / kStages;          // groups from the end
    const int m = (int)(back % kStages);       // stages of the group after this one
    // the wave ends at phase 0, so the phase at the group's end counts back
    const int ph = (int)((V - kStages * g % V) % V);
    int got = -1;
    for (uint32_t x = 0; x < (1u << m); ++x) {
        const uint32_t end = state >> m | x << (V - m);
        const uint32_t t = stored_tag(sp, rows - 1 - g, slot, position(end, ph, V), V, lb);
        // backwards from `end` the decisions of the last m stages (bits 3, 2, ..)
        // become the low bits of the state, the last one on top
        uint32_t low = 0;
        for (int k = 0; k < m; ++k) low = low << 1 | (t >> (kStages - 1 - k) & 1u);
        if (low != (state & ((1u << m) - 1u))) continue;
        const int d = (int)(t >> (kStages - 1 - m) & 1u);
        if (got < 0 || d != want) got = d;
    }
    return got;
}

}  // namespace tag_view
}  // namespace pbvd
