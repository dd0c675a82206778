// State-parallel decoder kernel: one wave decodes one parallel block (PB) of
// the parallel block-based Viterbi decoder (arXiv 1608.00066, Sec. III-A),
// one lane per trellis state (Sec. IV-A spreads a PB over threads in the
// same spirit: every thread updates a part of the states of each stage).
//
// Unlike the register kernel of pbvd_kernel.hpp (one lane per PB, the code a
// compile-time parameter) this kernel takes the generators as run-time
// arguments, so it decodes any rate-1/R code with 3 <= K <= 9, R <= 4, and a
// PB's D + 2L stages run 64 lanes wide: a short stream or a single frame
// finishes in a few microseconds instead of the hundreds a lane needs.
//
// Position map.  State d of stage t lives at position u = rotl_V^(t mod V)(d)
// (V = K-1 bits).  Then the butterfly of Sec. III-B at stage t pairs the
// positions that differ in bit ph = t mod V: the even one holds the upper
// predecessor S_2j, the odd one S_2j+1, and the new metrics of S_j (input 0)
// and S_j+2^(V-1) (input 1) go back to the even and the odd position.
// Bits 0..5 of a position choose the lane (see position_of_lane), the bits
// above the register slot (K = 8: 2 slots, K = 9: 4).  For K < 7 the lanes
// above 2^V repeat the low ones.
//
// A stage.  Each lane forms the two candidates that leave its position, the
// one that stays (own target) and the one its partner takes, both as one
// v_dot4_i32_i8 of the stage's R symbols (the same register in every lane) with
// the branch's code-word mask, accumulated onto its metric; v_min_i32 then
// takes the partner's candidate through a DPP lane swap.  The partner is
// lane ^ 1, 2, 7 or 8 for position bits 0..3: the swaps
// DPP does in one instruction (quad permutes, half-row mirror, row rotation);
// bits 4 and 5 use the gfx950 permlane16 / permlane32 swaps of the two
// candidates, slot bits need no exchange.  That is 3 vector instructions per
// stage (4 for bits 4 and 5).
//
// Branch metrics.  A branch's code word is c = (c^(1)..c^(R)) of Eq. 2; its
// metric is sum over r of c_r q_r (the Sec. II distance minus a constant
// shared by all branches of the stage, which changes no decision).  Metrics
// are kept times 64 (mask bytes 0 / 64), the low six bits are the tag.
//
// Survivors.  The tag of a position carries the origin of its survivor path:
// before the first stage of a round (position bits 0..5, phases 0..5) it is
// set to the position itself, and the minimum carries it along, so after the
// last phase of the round it is the position where the path was when the
// round began.  Two candidates of equal metric differ first, from the top, in
// the bit of the current phase (the bits above it have not been replaced
// yet), which is 0 for the path from S_2j: the minimum keeps the upper
// branch on ties, as Eq. 1 asks.  For K = 8, 9 the slot phases form a second
// round, whose tag is the slot.  The tags of floor(32 / V) passes over all V
// phases fill one dword, a trip of W = V * floor(32 / V) stages, which goes to
// HBM as [trip][slot][position].
//
// Traceback (Alg. 1, Kernel 2), V stages at a time on the scalar unit.  The
// input bit of a stage is the bit of its phase in the position the path
// reaches, and every bit is replaced once in V stages, so the V input bits of
// a pass are the position P at its end, and the position at its start is the
// tag stored for P.  A debug variant also stores the per-stage decisions of
// every position, the survivor layout of the plain method.
//
// What bounds it: vector issue where several waves share a SIMD (K = 7: 22
// instructions and a few waits for 6 stages), and for a lone wave the dependent
// chain of every stage, dot product -> swap and minimum.  Path words exchanged
// along with the metrics, a dot product after every exchange, and symbol loads
// that each trip waited for (12.6 instructions per stage) took twice as long:
// 2^20 bits of K = 7 in 2,048 blocks 47.1 -> 20.2 us per decode, 2^22 bits of
// K = 8 rate 1/3 205 -> 93 us, 4096 bits of K = 3 18.6 -> 11.3 us, 2,048 blocks
// of 512 bits of K = 9 rate 1/3 118 -> 55 us.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pbvd_kernel.hpp"
#include "pbvd_wave_args.hpp"

namespace pbvd {
namespace wave {

// Position bits 0..5 of a lane: lane = u0 ^ 2 u1 ^ 7 u2 ^ 8 u3 ^ 16 u4 ^ 32 u5,
// which is its own inverse.  Flipping position bit 2 is then lane ^ 7, the DPP
// half-row mirror (no DPP control flips lane bit 2 alone).
__device__ __forceinline__ int position_of_lane(int lane) { return lane ^ (lane & 4 ? 3 : 0); }

// v of the lane whose position differs in bit B (B < 4).
template <int B>
__device__ __forceinline__ int swap_lane(int v) {
    constexpr int kCtrl = B == 0 ? quad_sel(1, 0, 3, 2)    // lane ^ 1
                        : B == 1 ? quad_sel(2, 3, 0, 1)    // lane ^ 2
                        : B == 2 ? 0x141                   // row_half_mirror: lane ^ 7
                                 : 0x128;                  // row_ror:8: lane ^ 8
    return __builtin_amdgcn_mov_dpp(v, kCtrl, 0xf, 0xf, true);
}

// pm plus the branch metric.  The clamp (metrics never reach it) keeps the
// three-operand form of the dot product: without it the compiler takes the
// accumulating form, which needs a copy of pm for every second candidate.
__device__ __forceinline__ int branch(int q, uint32_t mask, int pm) {
    return __builtin_amdgcn_sdot4(q, (int)mask, pm, true);
}

// (acc:v) >> N of the 64-bit pair with v on top: the low N bits of v enter acc
// at the top.
template <int N>
__device__ __forceinline__ uint32_t push_low(uint32_t acc, int v) {
    return __builtin_amdgcn_alignbit((uint32_t)v, acc, N);
}

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v = min(v, __shfl_xor(v, m, kWave));
    return v;
}

// A 64-bit value every lane holds alike, made provably wave-uniform.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <int V>
__device__ __forceinline__ uint32_t rotl_rt32(uint32_t u, int s) {
    s %= V;
    return s == 0 ? u : (((u << s) | (u >> (V - s))) & ((1u << V) - 1u));
}

typedef int int4v __attribute__((ext_vector_type(4)));

// The PB a wave decodes.
struct Job {
    const uint8_t *in;   // symbols of the first forward stage
    int len;             // forward stages
    int store0;          // first traced (decoded) stage
    int dec_end;         // end of the decoded range (stage index)
    bool known;          // starts from encoder state 0
    bool argmin;         // traceback from the least-metric state
    int64_t out_bit0;    // output bit of the first decoded stage
    int edge;            // kOutEdges: the PB, counted from the call's first
    int32_t *pm_out;     // final metrics or null
};

// DEC: also store each stage's decisions (the debug survivor export) at
// dec_wave, in the [trip][slot][position] layout of the tags.
template <int V, bool DEC>
__device__ __forceinline__ void decode_pb(const Args &a, const Job &j, const WaveCode &code, uint32_t *sp_wave,
                                          uint32_t *dec_wave, uint32_t *q_lds) {
    constexpr int N = 1 << V;
    constexpr int SL = slots(V);
    constexpr int NL = N < kWave ? N : kWave;   // distinct positions per slot
    constexpr int LB = V < 6 ? V : 6;            // lane bits of a position
    constexpr int W = trip_stages(V);
    constexpr int NP = W / V;                    // passes over the V phases per trip
    constexpr int kTag = 63;                     // tag bits of a metric

    // the lane number through an empty asm statement: what derives from it
    // (the branch masks above all) is recomputed for each PB instead of
    // being hoisted out of the persistent loop into registers of their own
    int lane = (int)(threadIdx.x & (kWave - 1));
    asm volatile("" : "+v"(lane));
    const int len = j.len;
    const int R = code.R;
    const bool hard = code.kind == kHardU8;
    // Trips are aligned to the end of the forward range: trip i holds
    // stages [i*W - off, (i+1)*W - off), so the first trip starts off
    // stages in and the last one ends at stage len, at phase 0.
    const int n_trips = (len + W - 1) / W;
    const int off = n_trips * W - len;

    // Symbols: the R symbols of stage t are packed in one dword (bytes
    // 0..R-1; the bytes above belong to the next stage and meet zero mask
    // bytes).  Lane l loads those of stage l of two trips (2 W <= 64 stages)
    // two trips ahead, and puts them in the wave's part of the LDS, from
    // where every lane reads four stages at a time (a read that all lanes
    // make of one address; reading a lane's dword into a scalar register
    // instead cost a vector instruction per stage).  They come through a buffer resource
    // that holds the dwords of the PB's own symbols: loads past it return 0
    // without a branch, so they stay in flight until they are used (a branch
    // around the end of the input made every trip wait for its loads).
    static_assert(2 * W <= kWave, "a lane per stage of two trips");
    const uint32_t mis0 = (uint32_t)((uintptr_t)j.in & 3u);
    const uint8_t *const in_dw = j.in - mis0;
    const __amdgpu_buffer_rsrc_t in_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(in_dw), (short)0, (int)(mis0 + (uint32_t)(len * R) + 3u) & ~3, kBufferFlags);
    struct Raw {
        uint32_t lo, hi, at;  // two dwords and the byte offset of the first symbol in them (mod 4)
    };
    auto load_q = [&](int tt0) PBVD_INLINE_LAMBDA {
        int t = tt0 + lane;
        t = t < 0 ? 0 : t;  // stages before the first are never used
        Raw r;
        r.at = (uint32_t)(t * R) + mis0;  // R: the code's rate, wave-uniform
        // dword by dword: each is in bounds or not as a whole
        r.lo = __builtin_amdgcn_raw_buffer_load_b32(in_rsrc, r.at & ~3u, 0, kRowPolicy);
        r.hi = __builtin_amdgcn_raw_buffer_load_b32(in_rsrc, (r.at & ~3u) + 4, 0, kRowPolicy);
        return r;
    };
    auto make_q = [&](const Raw &r) PBVD_INLINE_LAMBDA {
        const uint32_t q = __builtin_amdgcn_alignbyte(r.hi, r.lo, r.at);
        return hard ? 0x01010101u + (q & 0x01010101u) * 0xfeu : q;  // bit -> +1 / -1
    };

    // the second trip's symbols start at a dword quadruple (lanes past them
    // share the buffer's last dword, which W < 32 leaves unused)
    uint32_t *const q_lane = q_lds + (lane < W ? lane : min(lane - W, kWave / 2 - 1) + kWave / 2);

    // the first trip's and the next two trips' symbols are requested before
    // the masks are formed
    const Raw raw_first = load_q(-off);
    Raw raw_next = load_q(W - off);

    // ---- code-word masks (bytes 0 / 64) of the two branches that leave each
    //      position, per phase and slot (Eq. 2 with the run-time generators):
    //      m0 / m1 the one that stays and the one the partner takes (lane
    //      swaps), or the ones with input 0 and 1 (permlane and slot phases).
    //      The register's state part enters as the parity of u and the
    //      generator rotated like the state; the input adds g_{K-1}. ----
    const int upos = position_of_lane(lane);
    uint32_t gk = 0;  // 64 in the bytes of generators that tap the input
#pragma unroll
    for (int r = 0; r < 4; ++r) gk |= ((code.gen[r] >> V) & 1u) << (8 * r + 6);
    uint32_t m0[V][SL], m1[V][SL];
#pragma unroll
    for (int ph = 0; ph < V; ++ph) {
        uint32_t rg[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) rg[r] = rotl_rt32<V>(code.gen[r] & (uint32_t)(N - 1), ph);
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const uint32_t u = (uint32_t)(s * kWave + (upos & (NL - 1)));
            uint32_t c = 0;  // bit counts (at most 8) in bytes; generators past R are 0
#pragma unroll
            for (int r = 0; r < 4; ++r) c |= (uint32_t)__builtin_popcount(u & rg[r]) << (8 * r);
            c = (c & 0x01010101u) << 6;
            if (ph < 4 && ph < LB && ((u >> ph) & 1u)) c ^= gk;  // the branch that stays has input u_ph
            m0[ph][s] = c;
            m1[ph][s] = c ^ gk;
        }
    }

    // ---- initial metrics: with a known start, state 0 (position 0 at any
    //      phase) at 0 and the others at 8192; otherwise all 0; tags set for
    //      the first round ----
    int pm[SL];
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int u = s * kWave + (upos & (NL - 1));
        pm[s] = ((j.known && u != 0) ? 8192 * (kTag + 1) : 0) | (upos & (NL - 1));
    }

    // tags of the trip's passes, the last pushed on top
    uint32_t hist[SL];
#pragma unroll
    for (int s = 0; s < SL; ++s) hist[s] = 0;

    // [trip][slot][position] tags, through a buffer resource: the trip's
    // offset is a scalar
    const __amdgpu_buffer_rsrc_t sp_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        sp_wave, (short)0, (int)(pb_dwords(V, len) * 4), kBufferFlags);

    // one trellis stage, the k-th of its trip (phase k mod V), with symbols q,
    // and the tags at the end of a round.  live: the stage belongs to the PB
    // (the first trip may start in the middle; its skipped rounds only set
    // tags).
    auto stage = [&](auto kc, int q, uint32_t (&acc)[SL], bool live) PBVD_INLINE_LAMBDA {
        constexpr int k = decltype(kc)::value;
        constexpr int PH = k % V;
        if (live) {
            if constexpr (PH < LB) {
#pragma unroll
                for (int s = 0; s < SL; ++s) {
                    const int a = branch(q, m0[PH][s], pm[s]);
                    const int b = branch(q, m1[PH][s], pm[s]);
                    if constexpr (PH < 4) {
                        pm[s] = min(a, swap_lane<PH>(b));
                    } else if constexpr (PH == 4) {
                        // rows 1, 3 of the first operand swap with rows 0, 2
                        // of the second: each lane gets the two candidates of
                        // its own target (input 0 for rows 0, 2)
                        const auto r = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
                        pm[s] = min((int)r[0], (int)r[1]);
                    } else {
                        const auto r = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
                        pm[s] = min((int)r[0], (int)r[1]);
                    }
                }
            } else {
                constexpr int M = 1 << (PH - 6);  // slot bit
#pragma unroll
                for (int s = 0; s < SL; ++s) {
                    if (s & M) continue;
                    const int e = pm[s], o = pm[s | M];
                    pm[s] = min(branch(q, m0[PH][s], e),
                                branch(q, m0[PH][s | M], o));
                    pm[s | M] = min(branch(q, m1[PH][s], e),
                                    branch(q, m1[PH][s | M], o));
                }
            }
            if constexpr (DEC) {
                // the decision of this stage is its phase's bit of the tag
                constexpr int bit = PH < 6 ? PH : PH - 6;
#pragma unroll
                for (int s = 0; s < SL; ++s) acc[s] = (acc[s] << 1) | (((uint32_t)pm[s] >> bit) & 1u);
            }
        }
        if constexpr (PH == LB - 1 || PH == V - 1) {
            constexpr int kBits = PH < 6 ? LB : V - 6;  // of the round that ends
            constexpr bool kSlotsNext = PH < V - 1;
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                hist[s] = push_low<kBits>(hist[s], pm[s]);
                pm[s] = (pm[s] & ~kTag) | (kSlotsNext ? s : (upos & (NL - 1)));
            }
        }
    };

    // The traceback reads the tags of trips trip_bot..n_trips-1
    // through a ring of kRing trips.  With one slot, the tags of the last
    // trip stay in registers and the loads of the trips below it are issued
    // at the start of the last forward trip, so that they have arrived when
    // the traceback starts.
    const int trip_bot = (j.store0 + off) / W;
    constexpr int kRing = SL == 1 ? 8 : SL == 2 ? 6 : 4;
    constexpr bool kEarlyRing = SL == 1;
    uint32_t ring[kRing][SL];
    auto load_trip = [&](uint32_t (&dst)[SL], int trip) PBVD_INLINE_LAMBDA {
        trip = trip < trip_bot ? trip_bot : trip;
#pragma unroll
        for (int s = 0; s < SL; ++s)
            dst[s] = __builtin_amdgcn_raw_buffer_load_b32(sp_rsrc, lane * 4, (trip * SL + s) * (kWave * 4), kRowPolicy);
    };

    // ---- forward procedure (Eq. 1) ----
    auto run_forward = [&](auto first, auto half, int trip) PBVD_INLINE_LAMBDA {
        if constexpr (kEarlyRing) {
            if (trip + 1 == n_trips) {
                // trips below the last one are stored already (a clamped
                // load of the last trip itself is never used)
                static_for<1, kRing - 1>([&](auto dc) PBVD_INLINE_LAMBDA {
                    load_trip(ring[decltype(dc)::value], trip - decltype(dc)::value);
                    return true;
                });
            }
        }
        uint32_t acc[SL];
#pragma unroll
        for (int s = 0; s < SL; ++s) acc[s] = 0;
        const int4v *const q4 = reinterpret_cast<const int4v *>(q_lds) + decltype(half)::value * (kWave / 8);
        static_for<0, (W + 3) / 4>([&](auto ic) PBVD_INLINE_LAMBDA {
            constexpr int i = decltype(ic)::value;
            const int4v q = q4[i];
            static_for<0, W - 4 * i < 4 ? W - 4 * i : 4>([&](auto kc) PBVD_INLINE_LAMBDA {
                constexpr int k = 4 * i + decltype(kc)::value;
                stage(std::integral_constant<int, k>{}, q[decltype(kc)::value], acc, !decltype(first)::value || k >= off);
                return true;
            });
            return true;
        });
        // pass p of the trip at bits 32 - V (NP - p) ..
#pragma unroll
        for (int s = 0; s < SL; ++s)
            __builtin_amdgcn_raw_buffer_store_b32(hist[s], sp_rsrc, upos * 4, (trip * SL + s) * (kWave * 4), kRowPolicy);
        if constexpr (DEC) {
            // step k of the trip at bit W-1-k
#pragma unroll
            for (int s = 0; s < SL; ++s)
                __builtin_nontemporal_store(acc[s], dec_wave + upos + (trip * SL + s) * kWave);
        }
        // exact renormalization: every metric minus one shared value
        const int ref = __builtin_amdgcn_readfirstlane(pm[0]) & ~kTag;
#pragma unroll
        for (int s = 0; s < SL; ++s) pm[s] -= ref;
    };
    constexpr std::integral_constant<int, 0> kLow{};   // half of the LDS buffer that holds a trip's symbols
    constexpr std::integral_constant<int, 1> kHigh{};
    // (one wave's LDS accesses stay in order: no wait between a buffer's last
    // reads and its next contents)
    *q_lane = make_q(raw_first);
    run_forward(std::true_type{}, kLow, 0);  // the first trip starts at step off
    for (int trip = 1; trip < n_trips; trip += 2) {
        *q_lane = make_q(raw_next);
        raw_next = load_q((trip + 2) * W - off);  // (past the input's end: 0)
        run_forward(std::false_type{}, kLow, trip);
        if (trip + 1 == n_trips) break;
        run_forward(std::false_type{}, kHigh, trip + 1);
    }

    // ---- final metrics and traceback start (Sec. III-A; Sec. II at the end
    //      of an unterminated stream).  The forward range ends at phase 0:
    //      position u holds state u. ----
    uint32_t P = 0;
    if (j.argmin || j.pm_out) {
#pragma unroll
        for (int s = 0; s < SL; ++s) pm[s] >>= 6;  // drop the tags
        int m = pm[0];
#pragma unroll
        for (int s = 1; s < SL; ++s) m = min(m, pm[s]);
        m = wave_min(m);
        if (j.argmin) {
            int best = N;
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                const int u = s * kWave + (upos & (NL - 1));
                if (pm[s] == m && u < best) best = u;
            }
            P = (uint32_t)__builtin_amdgcn_readfirstlane(wave_min(best));
        }
        if (j.pm_out && upos < NL) {
#pragma unroll
            for (int s = 0; s < SL; ++s) j.pm_out[s * kWave + upos] = pm[s] - m;
        }
    }

    // ---- traceback (Alg. 1, Kernel 2) ----
    // A trip at a time from its tags; stages below the decoded range at the
    // bottom are harmless.  Only the chain of positions runs trip by trip;
    // the input bits of a trip (bit i = its i-th stage) go to a lane of
    // `bits`, trip base + l to lane l.  Once kChunk trips are there (or the
    // last), every lane makes one output word from the two or three trips
    // it spans and all words are stored at once.  (Merging and storing word
    // by word inside the chain took twice as long: 13.8 k -> 7.6 k cycles
    // for the 20 trips of a K = 7 block of 512 bits.)
    const int n_dec = j.dec_end - j.store0;
    constexpr int kChunk = kWave - 2;  // lanes 62, 63: the two trips above the chunk
    int base = trip_bot + (n_trips - 1 - trip_bot) / kChunk * kChunk;
    uint32_t bits = 0;
    // kOutEdges: bits up to the PB's first whole byte
    const int head = a.out_mode == kOutEdges ? (int)(-j.out_bit0 & 7) : 0;
    auto emit = [&]() PBVD_INLINE_LAMBDA {
        // word m of the PB starts at virtual stage first + 32 m; this
        // chunk's words start in trips base .. base + kChunk - 1.  Word -1
        // is the head, the stages before first.
        const int first = j.store0 + off + head;
        const int lowest = base * W - first;
        const int m = (lowest > 0 ? (lowest + 31) >> 5 : head > 0 ? -1 : 0) + lane;
        const int at = (m < 0 ? -head : 32 * m) - lowest;  // from the chunk's first stage
        const int i = at / W, sh = at - i * W;
        uint32_t v = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * i, (int)bits) >> sh;
        v |= (uint32_t)__builtin_amdgcn_ds_bpermute(4 * i + 4, (int)bits) << 1 << (W - 1 - sh);
        const uint32_t top = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * i + 8, (int)bits);
        if (2 * W - sh < 32) v |= top << (2 * W - sh);
        if (m < 0) {
            v &= (1u << (n_dec < head ? n_dec : head)) - 1u;
            put_edge(a.out_words + j.edge, a.out + (j.out_bit0 >> 3), v << (j.out_bit0 & 7), a.edge_call);
            return;
        }
        const int nb = n_dec - head - 32 * m < 32 ? n_dec - head - 32 * m : 32;
        if (i >= kChunk || nb <= 0) return;
        if (nb < 32) v &= (1u << nb) - 1u;
        const int64_t bitpos = j.out_bit0 + head + 32 * m;
        if (a.out_mode == kOutAtomic) {
            const uint32_t shf = (uint32_t)(bitpos & 31);
            uint32_t *wp = a.out_words + (bitpos >> 5);
            atomicOr(wp, v << shf);
            if (shf && (v >> (32 - shf))) atomicOr(wp + 1, v >> (32 - shf));
            return;
        }
        uint8_t *ob = a.out + (bitpos >> 3);
        if (nb == 32 && ((uintptr_t)ob & 3u) == 0) {
            *reinterpret_cast<uint32_t *>(ob) = v;
        } else {
            const bool shared = a.out_mode == kOutEdges && (nb & 7) != 0 && bitpos + nb != a.out_bits;
            for (int bb = 0; bb < ((nb + (shared ? 0 : 7)) >> 3); ++bb) ob[bb] = (uint8_t)(v >> (8 * bb));
            if (shared) put_edge(a.out_words + j.edge + 1, ob + (nb >> 3), v >> (nb & ~7) & 0xffu, a.edge_call);
        }
    };

    auto run_trip = [&](const uint32_t (&hw)[SL], int trip) PBVD_INLINE_LAMBDA {
        uint32_t word = 0;
        static_for<0, NP>([&](auto pc) PBVD_INLINE_LAMBDA {
            constexpr int p = NP - 1 - decltype(pc)::value;
            constexpr int sh = 32 - V * (NP - p);  // the pass's tags in the trip's word
            word |= P << (V * p);
            const int l = (int)(P & 63u);
            if constexpr (SL == 1) {
                P = ((uint32_t)__builtin_amdgcn_readlane((int)hw[0], l) >> sh) & (uint32_t)(N - 1);
            } else {
                // the slot round's tag (top V - 6 bits of the pass) names the
                // slot whose lane round led here; a pass's tags of all slots,
                // a byte each, are put together before the lane is known
                // (a choice between scalars became a table in scratch memory)
                uint32_t f = 0;
#pragma unroll
                for (int s = 0; s < SL; ++s) f |= (hw[s] >> sh & (uint32_t)(N - 1)) << (8 * s);
                f = (uint32_t)__builtin_amdgcn_readlane((int)f, l);
                const uint32_t slot = (f >> (P >> 6 << 3) & (uint32_t)(N - 1)) >> 6;
                P = slot << 6 | (f >> (slot << 3) & 63u);
            }
            return true;
        });
        bits = lane == trip - base ? word : bits;
        if (trip == base) {
            emit();
            // the chunk below sees this chunk's two lowest trips as its top
            const uint32_t t0 = (uint32_t)__builtin_amdgcn_readlane((int)bits, 0);
            const uint32_t t1 = (uint32_t)__builtin_amdgcn_readlane((int)bits, 1);
            bits = lane == kChunk ? t0 : lane == kChunk + 1 ? t1 : bits;
            base -= kChunk;
        }
    };

    const int trip_top = n_trips - 1;
    if constexpr (kEarlyRing) {
#pragma unroll
        for (int s = 0; s < SL; ++s)  // from lane to position order (lane ^ 3 where lane bit 2 is set)
            ring[0][s] = (uint32_t)__builtin_amdgcn_update_dpp((int)hist[s], (int)hist[s], quad_sel(3, 2, 1, 0), 0xf,
                                                               0xa, false);
    } else {
        static_for<0, kRing - 1>([&](auto dc) PBVD_INLINE_LAMBDA {
            load_trip(ring[decltype(dc)::value], trip_top - decltype(dc)::value);
            return true;
        });
    }
    int trip = trip_top;
    for (;;) {
        const bool more = static_for<0, kRing>([&](auto dc) PBVD_INLINE_LAMBDA {
            constexpr int d = decltype(dc)::value;
            load_trip(ring[(d + kRing - 1) % kRing], trip - (kRing - 1));
            run_trip(ring[d], trip);
            if (trip <= trip_bot) return false;
            --trip;
            return true;
        });
        if (!more) break;
    }
}

// Job of PB `idx` of a stream (Sec. III-A geometry; stream mode).
template <int V>
__device__ __forceinline__ Job stream_job(const Args &a, const uint8_t *syms, int64_t idx) {
    constexpr int N = 1 << V;
    Job j;
    const int64_t b = a.pb_first + idx;
    const int64_t D = a.D, L = a.L;
    const int64_t d0 = b * D;
    const int64_t f0 = d0 - L < 0 ? 0 : d0 - L;
    const int64_t f1 = d0 + D + L > a.T ? a.T : d0 + D + L;
    const int64_t d1 = d0 + D > a.n ? a.n : d0 + D;
    j.in = syms + f0 * a.codes[0].R;
    j.len = (int)(f1 - f0);
    j.store0 = (int)(d0 - f0);
    j.dec_end = (int)(d1 - f0);
    j.known = f0 == 0;
    j.argmin = f1 == a.T && !a.terminated;
    j.out_bit0 = idx * D;
    j.edge = (int)idx;
    j.pm_out = a.final_pm ? a.final_pm + idx * N : nullptr;
    return j;
}

// Job of descriptor idx of a work list (batches); *code_idx receives its code.
__device__ __forceinline__ Job desc_job(const Args &a, const uint8_t *syms, int64_t idx, int *code_idx, bool *active) {
    Job j;
    const LaneDesc &d = a.descs[idx];
    j.in = syms + uniform64(d.sym);
    j.len = __builtin_amdgcn_readfirstlane(d.len);
    j.store0 = __builtin_amdgcn_readfirstlane(d.store0);
    j.dec_end = __builtin_amdgcn_readfirstlane(d.dec_end);
    const int fl = __builtin_amdgcn_readfirstlane(d.flags);
    j.known = (fl & kLaneKnown) != 0;
    j.argmin = (fl & kLaneArgmin) != 0;
    j.out_bit0 = uniform64(d.out_bit);
    j.edge = 0;
    j.pm_out = nullptr;
    *code_idx = (fl >> kDescCodeShift) & 0xff;
    *active = (fl & kLaneActive) != 0;
    return j;
}

// One wave per PB; 4 independent waves per 256-thread workgroup.  Modes:
// kModeList, a stream's PBs (descs == null) or a work list's PBs (descs),
// one per wave; kModePersist, persistent waves that take the work list's
// PBs in list order (longest first) from work counters until it is exhausted --
// one launch for the PBs of every code of this K, whatever their count (a
// kernel of its own: the state it keeps across PBs would cost the other
// modes a wave per SIMD); kModeDecisions, a stream's PBs with every stage's
// decisions stored as well (a.dec_sp, the debug survivor export).
// syms: the symbol buffer (the same pointer as a.syms), a separate parameter
// so that its loads may use the scalar unit (nothing the kernel writes
// aliases it).
template <int V, int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(V <= 7 ? 8 : 4)))
    decode_wave_kernel(const Args a, const uint8_t *__restrict__ syms) {
    // the waves' symbol buffers (decode_pb)
    __shared__ __align__(16) uint32_t q_block[256];
    uint32_t *const q_lds = q_block + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * kWave;
    const int64_t wl = (int64_t)blockIdx.x * (blockDim.x / kWave) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (wl >= a.n_waves) return;
    uint32_t *const sp = a.sp + wl * a.sp_wave_dwords;
    if constexpr (MODE == kModePersist) {
        // The next PB from the counter of this workgroup's XCD (workgroups
        // go to the 8 XCDs in turn): with nc counters (8, fewer for grids
        // of fewer workgroups, so that every counter has waves), counter x
        // hands out PBs x, x + nc, x + 2 nc, ... of the list, so each XCD
        // takes an equal share of every length, longest first, and the
        // counters spread the atomics.
        const int lane = (int)(threadIdx.x & (kWave - 1));
        const int nc = gridDim.x < (unsigned)kCounters ? (int)gridDim.x : kCounters;
        const int x = (int)(blockIdx.x % (unsigned)nc);
        for (;;) {
            uint32_t got = 0;
            if (lane == 0) got = atomicAdd(a.counter + kCounterStride * x, 1u);
            const int64_t idx = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)got) * nc + x;
            if (idx >= a.n_items) return;
            int ci;
            bool active;
            const Job j = desc_job(a, syms, idx, &ci, &active);
            if (active) decode_pb<V, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        }
    } else if constexpr (MODE == kModeDecisions) {
        decode_pb<V, true>(a, stream_job<V>(a, syms, a.wave_begin + wl), a.codes[0], sp,
                           a.dec_sp + wl * a.sp_wave_dwords, q_lds);
    } else {
        const int64_t idx = a.wave_begin + wl;
        int ci = 0;
        bool active = true;
        const Job j = a.descs ? desc_job(a, syms, idx, &ci, &active) : stream_job<V>(a, syms, idx);
        if (active) decode_pb<V, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
    }
}

}  // namespace wave
}  // namespace pbvd
