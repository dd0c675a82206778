// The survivor export of the tag body on the host: a Viterbi decoder of random
// symbols whose survivors are kept as tags in packed 16-bit metrics and stored
// the way the kernel stores them, read back with pbvd_tag_view.hpp and compared
// with the decisions of every state and stage; then every single wrong bit of a
// tag has to show.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "pbvd_tag_view.hpp"

using namespace pbvd;

static unsigned rnd() {
    static uint64_t s = 88172645463325252ull;
    s ^= s << 13, s ^= s >> 7, s ^= s << 17;
    return (unsigned)(s >> 32);
}

static int run(int V, int lb, int trips) {
    const int N = 1 << V, NR = (N / 2) >> lb, NDW = NR / 4, B = V - 2 - lb;
    const int stages = trips * tag_view::trip(V), groups = stages / 4;
    const unsigned gen[2] = {rnd() | 1u << V, rnd() | 1u};
    std::vector<int> pm(N, 0), nx(N);
    std::vector<std::vector<int>> dec(stages, std::vector<int>(N));
    std::vector<std::vector<unsigned>> from(stages, std::vector<unsigned>(N));
    for (int s = 0; s < stages; ++s) {
        const int q[2] = {(int)(rnd() % 15) - 7, (int)(rnd() % 15) - 7};
        for (int d = 0; d < N; ++d) {
            int m[2];
            for (int low = 0; low < 2; ++low) {
                const int p = ((d << 1) & (N - 1)) | low, reg = p | (d >> (V - 1)) << V;
                m[low] = pm[p];
                for (int r = 0; r < 2; ++r) m[low] += __builtin_parity(reg & gen[r]) ? q[r] : 0;
            }
            dec[s][d] = m[1] < m[0];
            nx[d] = m[dec[s][d]];
        }
        pm = nx;
    }
    // tags of a group: the bits of its phases in the origin's position
    std::vector<uint32_t> sp((size_t)groups * NDW * 64, 0xdeadbeefu);
    const int pbs = 64 >> lb, slot = (int)(rnd() % (unsigned)pbs);
    for (int g = 0; g < groups; ++g) {
        std::vector<int> tag(N);  // by position
        for (int e = 0; e < N; ++e) {
            unsigned s = (unsigned)e;
            for (int k = 3; k >= 0; --k) s = ((s << 1) & (unsigned)(N - 1)) | (unsigned)dec[4 * g + k][s];
            const unsigned u = tag_view::position(s, 4 * g % V, V);
            int t = 0;
            for (int k = 0; k < 4; ++k) t |= (int)(u >> ((4 * g + k) % V) & 1u) << k;
            tag[tag_view::position((unsigned)e, (4 * g + 4) % V, V)] = t;
        }
        // registers of a lane: two halves of 16 bits, the tag at the bottom of
        // each below a metric
        for (int ell = 0; ell < 1 << lb; ++ell) {
            std::vector<uint32_t> reg(NR);
            for (int r = 0; r < NR; ++r) {
                const int u = ell << (V - 1 - lb) | r;
                reg[r] = (rnd() & 0xfff0fff0u) | (uint32_t)tag[u] | (uint32_t)tag[u | 1 << (V - 1)] << 16;
            }
            for (int c = 0; c < NDW / 2; ++c)
                for (int i = 0; i < 2; ++i) {
                    const int r = (2 * c + i) * 2;
                    auto bytes = [&](int a) {  // low bytes of the halves of a and a + 1
                        return (reg[a] & 0xffu) | (reg[a] >> 16 & 0xffu) << 8 | (reg[a + 1] & 0xffu) << 16 |
                               (reg[a + 1] >> 16 & 0xffu) << 24;
                    };
                    const uint32_t v = (bytes(r) & 0x0f0f0f0fu) | (bytes(r | 1 << B) << 4 & 0xf0f0f0f0u);
                    sp[(size_t)g * NDW * 64 + c * 128 + (slot << lb | ell) * 2 + i] = v;
                }
        }
    }
    int bad = 0;
    long known = 0;
    auto differ = [&](int g0, int g1) {
        int n = 0;
        for (int s = 4 * g0; s < 4 * g1; ++s)
            for (int d = 0; d < N; ++d) {
                const int got = tag_view::stored_decision(sp.data(), groups, slot, stages - 1 - s, (unsigned)d, V, lb,
                                                          dec[s][d]);
                if (got >= 0 && got != dec[s][d]) ++n;
                if (got < 0 && s % 4 == 3) ++n;  // every state at a group's end has a survivor
                known += got >= 0;
            }
        return n;
    };
    if (differ(0, groups) || known <= (long)groups * N) ++bad;
    for (int i = 0; i < 200; ++i) {
        const int g = (int)(rnd() % (unsigned)groups);
        const unsigned dw = rnd() % (unsigned)NDW;
        uint32_t &w = sp[(size_t)g * NDW * 64 + (dw >> 1) * 128 + (slot << lb | rnd() % (1u << lb)) * 2 + (dw & 1)];
        const uint32_t flip = 1u << rnd() % 32;
        w ^= flip;
        if (!differ(g, g + 1)) ++bad;
        w ^= flip;
    }
    if (bad) printf("V %d lb %d trips %d: %d wrong\n", V, lb, trips, bad);
    return bad;
}

int main() {
    int bad = 0;
    for (int V = 5; V <= 8; ++V)
        for (int lb = 0; lb <= 3; ++lb)
            if ((1 << (V - 1)) >> lb >= 16)
                for (int trips = 1; trips <= 3; ++trips) bad += run(V, lb, trips);
    if (!bad) printf("ok\n");
    return bad != 0;
}
