// The boundary words of pbvd_edges.hpp on the host: for every pair of bit sets,
// whatever an earlier call left in the word, the two PBs of a boundary give the
// byte exactly once, in either order.
#include <stdio.h>

#include "pbvd_edges.hpp"

using namespace pbvd;

static int writes;
static uint8_t byte;

static void put(uint32_t *word, uint32_t bits, uint32_t call) {
    const uint32_t mine = edge_word(call, bits), found = *word;
    *word = mine;
    if (!edge_second(mine, found)) return;
    byte = (uint8_t)(found | mine);
    ++writes;
}

int main() {
    const uint32_t calls[] = {1, 2, 3, 255, 256, kEdgeCalls - 2, kEdgeCalls - 1};
    int bad = 0;
    for (uint32_t call : calls)
        for (uint32_t split = 1; split < 8; ++split)
            for (uint32_t order = 0; order < 2; ++order) {
                const uint32_t lo = 0xa5u & ((1u << split) - 1u), hi = 0xa5u & ~((1u << split) - 1u);
                // left behind: nothing, half of an earlier call, both of it,
                // a replay of a captured call, another call's of the same bits
                const uint32_t left[] = {0u,           edge_word(call - 1, lo), edge_word(call - 1, 0xa5u),
                                         0x100u | hi,  edge_word(0, 0xffu),     edge_word(call == 1 ? 5 : 1, hi)};
                for (uint32_t l : left) {
                    uint32_t word = l;
                    if (call == 1) word = 0;  // cleared when the numbers start
                    writes = 0;
                    put(&word, order ? hi : lo, call);
                    if (writes != 0) ++bad;
                    put(&word, order ? lo : hi, call);
                    if (writes != 1 || byte != 0xa5u) ++bad;
                }
            }
    // the numbers: 1 after none, never 0 (captured calls), below the limit
    if (edge_next_call(0) != 1 || edge_next_call(1) != 2) ++bad;
    if (edge_next_call(kEdgeCalls - 2) != kEdgeCalls - 1 || edge_next_call(kEdgeCalls - 1) != 1) ++bad;
    if (edge_word(kEdgeCalls - 1, 0xffu) >> 9 != kEdgeCalls - 1) ++bad;
    if (bad) printf("%d wrong\n", bad);
    else printf("ok\n");
    return bad != 0;
}
