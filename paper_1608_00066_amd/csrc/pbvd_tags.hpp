// Register kernel body with survivor tags (16-bit metrics, trellises of 32 to
// 256 states): the same mapping as decode_body of pbvd_kernel.hpp (a PB per
// lane or per group of 2^LB lanes, path metrics packed two to a register, the
// butterfly of Sec. III-B in place, code and phases compile-time), with the
// decisions carried inside the metrics.
//
// Tags.  A metric is kept times 16; its low four bits are the tag.  Before the
// first stage of a group of four stages the tag of every state is set to the
// four bits of its position that the group's phases replace, and the minimum
// of the add-compare-select carries it along, so after the group it names the
// position where the state's survivor was when the group began: the group's
// four decisions.  Two candidates of equal metric differ first, from the top,
// in the bit of the current phase, which is 0 for the path from S_2j: the
// minimum keeps the upper branch on ties (Eq. 1).  A stage is two additions
// and a minimum per two states; once per four stages the tags are gathered
// (two byte permutes, a shift and a bit-field insert for 8 states) and set anew
// (one and-or per register).  Decisions taken from the sign of a difference,
// stage by stage, cost 2.57 instructions per add-compare-select; this is 1.9.
//
// Range.  Four tag bits leave 12 bits of metric, so metrics are renormalized
// often, but through the branch metrics: a reference is subtracted from the
// 2^R branch metrics of a stage instead of from every state.  The reference is
// the mean of two (or four) states' metrics chosen at compile time, because
// the distance of a metric from that mean is bounded tightly: the survivors
// of states d and e can share their state K-1 stages back, so their metrics
// differ by at most 128 w(d ^ e), w(x) being the weight of the code words on
// the K-1 stages from state 0 to x, and |m(d) - (m(0) + m(x)) / 2| <= 64 (w(d)
// + w(d ^ x)).  tag_plan() takes the x of the least bound and derives from it
// at which phases the reference has to be renewed.
//
// Start.  All PBs of a wave end at the same stage (a trip boundary, phase 0)
// and start where their length puts them; symbols before a PB's start are
// read as 0, which leaves equal metrics equal.  A PB that starts from the known
// encoder state 0 takes the upper branch in its first K-1 stages whatever the
// metrics: following upper branches K-1 stages back from any state leads to
// state 0, so its metrics are then those of the paths that leave state 0, and
// its tags name them.  Until then only the states that a path from state 0
// reaches count: they are kept in range without a reference (a state of the
// mean may be unreached): at most 128 times the code words' weight from the
// start, or the sum of the half symbol sums.
//
// What bounds it.  A lone wave of K = 7, R = 2, a PB per lane: 560 cycles of
// vector issue per warm-up stage and 620 per traced one (140 instructions, of
// which 96 are the add-compare-selects), then 100 per stage of traceback; with
// a wave on every SIMD the traceback reads its rows all at once, 270 cycles per
// stage or 4.6 TB/s.  2^27 bits move 3.1 GB of rows and symbols in 0.71 ms,
// 4.3 TB/s where a large copy reaches 4.8.  Per decode, with decisions taken
// stage by stage and with tags: 2^27 bits of K = 7 819 -> 707 us, 2^25 bits of
// K = 9 rate 1/3 993 -> 829 us, 12 Mbit of K = 7 in 24,001 PBs 163 -> 128 us (of
// which 12 by the output without staging).
#pragma once

#include "pbvd_kernel.hpp"

namespace pbvd {

constexpr int kTagBits = 4;             // decisions per tag, stages per group
constexpr int kTagMetricMax = 2047;     // 12-bit metrics

// How one code keeps its metrics in range (compile time).
struct TagPlan {
    bool ok;            // the metrics fit
    int n_ref;          // states in the reference mean: 2 or 4
    int ref[4];
    bool center;        // subtract half the symbol sum from every branch metric
    int period;         // stages between references
};

template <class C>
constexpr TagPlan tag_plan() {
    constexpr int V = C::V, N = C::N;
    // w[d]: weight of the code words on the V stages from state 0 to d
    int w[N] = {};
    for (int d = 0; d < N; ++d) {
        int s = 0;
        for (int t = 0; t < V; ++t) {
            const int x = (d >> t) & 1;
            int c = C::out0(s) ^ (x ? C::gcol(C::K - 1) : 0);
            for (; c; c &= c - 1) ++w[d];
            s = (s >> 1) | (x << (V - 1));
        }
    }
    int best2 = 1 << 30, x2 = 0;
    for (int x = 1; x < N; ++x) {
        int m = 0;
        for (int d = 0; d < N && m < best2; ++d) m = w[d] + w[d ^ x] > m ? w[d] + w[d ^ x] : m;
        if (m < best2) best2 = m, x2 = x;
    }
    // stages a reference lasts: a stage moves every metric by at most g
    // (128 R, or 64 R + 1 around half the symbol sum); the reference itself
    // is rounded by less than 2
    auto stages = [](int bound, int g) { return (kTagMetricMax - bound - 2) / g; };
    TagPlan p{false, 2, {0, x2, 0, 0}, false, 0};
    p.period = stages(64 * best2, 128 * C::R);
    if (p.period < 1) {
        p.center = true;
        p.period = stages(64 * best2, 64 * C::R + 1);
    }
    if (p.period < 1) {
        int best4 = 1 << 30;
        for (int x = 1; x < N; ++x)
            for (int y = x + 1; y < N && y < 16; ++y) {
                int m = 0;
                for (int d = 0; d < N && m < best4; ++d) {
                    const int t = w[d] + w[d ^ x] + w[d ^ y] + w[d ^ x ^ y];
                    m = t > m ? t : m;
                }
                if (m < best4) best4 = m, p.ref[1] = x, p.ref[2] = y, p.ref[3] = x ^ y;
            }
        p.n_ref = 4;
        p.period = stages(32 * best4, 64 * C::R + 1);
    }
    int w_max = 0;
    for (int d = 0; d < N; ++d) w_max = w[d] > w_max ? w[d] : w_max;
    p.ok = p.period >= 1 && (p.center ? V * (64 * C::R + 1) : 128 * w_max) <= kTagMetricMax;
    return p;
}

// Layout of the tag body.  Position u = rotl(state, phase): bit V-1 is the
// half of a register, the bits below it the register, its top LB bits the lane
// of the group.  A group's tags: 4 registers per dword, one per byte pair
// and nibble.  Survivor index (idx) of a position: bits 0..4 the shift that
// brings its tag to the bottom of its dword, the bits above the dword (in the
// lane, then the lane).
template <class C, int LB>
struct TagLayout {
    static constexpr int V = C::V;
    static constexpr int NR = C::NR >> LB;        // packed registers per lane
    static constexpr int NDW = NR / 4;            // survivor dwords per lane and group
    static constexpr int gcd(int a, int b) { return b == 0 ? a : gcd(b, a % b); }
    static constexpr int U = V / gcd(V, kTagBits) * kTagBits;  // stages per trip
    static constexpr int CY = U / kTagBits;       // groups per trip
    static constexpr int B = V - 2 - LB;          // position bit that chooses the nibble
    static constexpr int pos(int t) { return t == V - 1 ? 3 : t == 0 ? 4 : t == B ? 2 : t < B ? 4 + t : 3 + t; }
    // phases of group q of a trip: first, then the next three (mod V)
    static constexpr int phase(int q, int k) { return (q * kTagBits + k) % V; }
    // tag of position bits u before group q
    static constexpr uint32_t tag(int q, int u) {
        uint32_t t = 0;
        for (int k = 0; k < kTagBits; ++k) t |= (uint32_t)((u >> phase(q, k)) & 1) << k;
        return t;
    }
    // rows the traceback keeps in flight, in groups (whole trips, so that a
    // slot's phases are static)
    static constexpr int kRing = 2 * CY * NDW <= (NR >= 128 ? 128 : 64) ? 2 * CY : CY;
};

// Path metrics of 16 bits and at least 32 states decode with tags.
template <class C, class P>
__host__ __device__ constexpr bool uses_tags() {
    return std::is_same<P, PM16>::value && C::N >= 32;
}

// Lane groups a code supports (compile-time mirror of lanes_allowed on the host).
template <class C, class P, int LB>
__host__ __device__ constexpr bool lanes_supported() {
    return LB == 0 || (uses_tags<C, P>() && LB <= 3 && (C::NR >> LB) >= 16);
}

// on-lanes of a wave-constant lane pattern take b, the others a: one
// v_cndmask_b32 with the pattern in a scalar register pair
__device__ __forceinline__ int select_lanes(int a, int b, uint64_t pattern) {
    int r;
    asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(pattern));
    return r;
}

// ---------------------------------------------------------------------------
// Lanes per PB.  With 2^LB lanes per PB (LB = 1, 2 or 3) the registers of a PB
// are spread over a group of consecutive lanes: lane l of the group holds the
// states whose register index has l in its top LB bits.  Stages whose
// butterfly pairs registers of different lanes swap candidates with DPP (quad
// permutes, row shifts across quads); every lane keeps its own half of each pair.
// ---------------------------------------------------------------------------
// quad-permute control: flip lane bit 0 / 1
template <int B> __host__ __device__ constexpr int quad_flip() { return B == 0 ? quad_sel(1, 0, 3, 2) : quad_sel(2, 3, 0, 1); }
// Lane bit 2 (groups of 8) crosses quads: DPP row shifts by 4 inside a row of
// 16 lanes, written only to the banks (groups of 4 lanes) that need them.
constexpr int kRowShl4 = 0x104;  // lane l reads lane l + 4 of its row
constexpr int kRowShr4 = 0x114;  // lane l reads lane l - 4 of its row
// v of the lane with bit 2 cleared / set (lanes that are that lane keep v)
__device__ __forceinline__ int bit2_lo(int v) { return __builtin_amdgcn_update_dpp(v, v, kRowShr4, 0xf, 0xa, false); }
__device__ __forceinline__ int bit2_hi(int v) { return __builtin_amdgcn_update_dpp(v, v, kRowShl4, 0xf, 0x5, false); }
// v of the lane whose bit 2 differs
__device__ __forceinline__ int bit2_flip(int v) {
    const int t = __builtin_amdgcn_update_dpp(v, v, kRowShl4, 0xf, 0x5, false);
    return __builtin_amdgcn_update_dpp(t, v, kRowShr4, 0xf, 0xa, false);
}

// (x & keep) | bits as one instruction (a constant in a scalar register; the
// compiler makes an and and an or with literals of it).
__device__ __forceinline__ uint32_t keep_or(uint32_t x, uint32_t keep, uint32_t bits) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(keep), "s"(bits));
    return r;
}
__device__ __forceinline__ uint32_t keep_or_v(uint32_t x, uint32_t keep, uint32_t bits) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(keep), "v"(bits));
    return r;
}
// hi where mask is set, else lo (a select whose condition is a lane mask, not
// a comparison that the compiler would repeat per use).
__device__ __forceinline__ uint32_t bit_select(uint32_t mask, uint32_t hi, uint32_t lo) {
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(mask), "v"(hi), "v"(lo));
    return r;
}

// One stage on the NR registers of a lane at phase PH; pair[c] holds the
// branch metric of code word c in the lower half and of c ^ (the column of the
// position bit that the halves differ in) in the upper one, relabeled for
// the lane.  FORCE: lanes with `force` set take the upper branch.
template <class C, int PH, int LB, bool FORCE>
__device__ __forceinline__ void acs_tags(PM16::T (&pm)[C::NR >> LB], const PM16::T (&pair)[C::NC], bool force, int ell) {
    using T = PM16::T;
    constexpr int V = C::V, NR = C::NR >> LB;
    constexpr int G0 = C::gcol(0), GK = C::gcol(C::K - 1);
    constexpr int kCross = V - 1 - LB;  // first phase whose pair bit is a lane bit
    auto pick = [&](T upper, T lower) PBVD_INLINE_LAMBDA {
        const T m = PM16::vmin(upper, lower);
        if constexpr (FORCE) return __builtin_bit_cast(T, force ? __builtin_bit_cast(int, upper) : __builtin_bit_cast(int, m));
        else return m;
    };
    if constexpr (PH < kCross) {
        static_for<0, NR / 2>([&](auto kc) PBVD_INLINE_LAMBDA {
            constexpr int k = decltype(kc)::value;
            constexpr int X = ((k >> PH) << (PH + 1)) | (k & ((1 << PH) - 1));
            constexpr int Y = X | (1 << PH);
            constexpr int alpha = C::out0(rotr_v<V>(X, PH));  // c(S_2j, 0) of the lower half
            const T x = pm[X], y = pm[Y];
            pm[X] = pick(PM16::add(x, pair[alpha]), PM16::add(y, pair[alpha ^ G0]));
            pm[Y] = pick(PM16::add(x, pair[alpha ^ GK]), PM16::add(y, pair[alpha ^ G0 ^ GK]));
            return true;
        });
    } else if constexpr (PH < V - 1) {
        // the pair bit is lane bit B: a lane forms the candidate that stays
        // and the one its partner takes, and swaps the latter (the lane's own
        // bit enters through its relabeled metrics)
        constexpr int B = PH - kCross;
        const bool odd = (ell >> B) & 1;
        static_for<0, NR>([&](auto xc) PBVD_INLINE_LAMBDA {
            constexpr int X = decltype(xc)::value;
            constexpr int alpha = C::out0(rotr_v<V>(X, PH));
            const T own = PM16::add(pm[X], pair[alpha]);
            const T snd = PM16::add(pm[X], pair[alpha ^ GK]);
            T got;
            if constexpr (B < 2) got = PM16::template dpp<quad_flip<B>()>(snd);
            else got = PM16::each(snd, bit2_flip);
            if constexpr (FORCE) {
                const T m = PM16::vmin(own, got);
                pm[X] = __builtin_bit_cast(T, force ? (odd ? __builtin_bit_cast(int, got) : __builtin_bit_cast(int, own))
                                                    : __builtin_bit_cast(int, m));
            } else {
                pm[X] = PM16::vmin(own, got);
            }
            return true;
        });
    } else {
        // each register holds (S_2j, S_2j+1): broadcast operands
        static_for<0, NR>([&](auto xc) PBVD_INLINE_LAMBDA {
            constexpr int X = decltype(xc)::value;
            constexpr int alpha = C::out0(2 * X);
            const T x = pm[X];
            pm[X] = pick(PM16::add(PM16::bcast_lo(x), pair[alpha]), PM16::add(PM16::bcast_hi(x), pair[alpha ^ G0]));
            return true;
        });
    }
}

// Relabeling of the code words for lane bit j at phase PH.  The code word of a
// branch is linear (over GF(2)) in the state bits, so the lane bits add the
// same mask to every branch of a lane: the lane uses metric[c ^ mask] where
// the stage code above uses metric[c].  In a stage whose pair bit is lane bit
// j, the candidate that stays of a lane with that bit set comes from S_2j+1
// and goes to the input-1 target (Eq. 4, Eq. 6).
template <class C, int LB>
__host__ __device__ constexpr int tag_lane_mask(int PH, int j) {
    constexpr int V = C::V;
    const int kCross = V - 1 - LB;
    if (PH >= kCross && PH < V - 1 && PH - kCross == j) return C::gcol(0) ^ C::gcol(C::K - 1);
    return C::out0(rotr_v<V>(1 << (kCross + j), PH));
}

__device__ __forceinline__ int wave_reduce_max(int v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v = max(v, __shfl_xor(v, m, kWave));
    return __builtin_amdgcn_readfirstlane(v);
}

// Decodes the 64 >> LB PBs of a wave.  VARLEN: lanes may run fewer stages than
// the wave.  sp_wave: the wave's survivor slot of sp_dwords dwords,
// [group][dword pair][lane].
template <class C, int KIND, bool VARLEN, int LB>
__device__ __forceinline__ void tag_body(const WaveJob &j, uint32_t *sp_wave, int64_t sp_dwords) {
    using T = PM16::T;
    using LY = TagLayout<C, LB>;
    constexpr TagPlan kPlan = tag_plan<C>();
    static_assert(kPlan.ok, "the code's metrics fit 12 bits");
    constexpr int V = C::V, NR = LY::NR, R = C::R, NC = C::NC, U = LY::U, CY = LY::CY, NDW = LY::NDW;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int ell = LB ? lane & ((1 << LB) - 1) : 0;

    // ---- virtual stages: the wave runs n_trips trips of U stages, its PBs
    //      end with the last; vs: the lane's first stage, ds: its first decoded
    //      (traced) one ----
    const int n_trips = (j.len + U - 1) / U;
    const int off = n_trips * U - j.len;
    const int vs = off + (VARLEN ? j.len - j.my_len : 0);
    const int ds = vs + j.my_store0;
    const int n_dec = j.my_dec_end - j.my_store0;
    const int start_hi = VARLEN ? wave_reduce_max(vs) : off;
    const int ds_lo = VARLEN ? -wave_reduce_max(-ds) : off + j.store0_min;
    const int force_end = __ballot(j.known) == 0 ? 0 : VARLEN ? wave_reduce_max(j.known ? vs + V : 0) : off + V;
    const int g0 = ds_lo / kTagBits;           // first traced group
    const int n_groups = n_trips * CY;

    // ---- symbols: a trip's NB bytes as NW + 1 dwords, a whole number of
    //      dwords per trip, so the lane's misalignment is constant ----
    constexpr int NB = U * R, NW = NB / 4;
    static_assert(NB % 4 == 0, "a trip spans whole dwords");
    const uint32_t mis = (uint32_t)((uintptr_t)j.in & 3u);
    const uint8_t *const in_dw = j.in - mis;   // keeps the global address space
    const int first_byte = (int)mis - vs * R;  // of virtual stage 0, from in_dw
    const uint32_t sh = (uint32_t)(first_byte & 3) * 8u;
    const int base = first_byte & ~3;
    const int64_t in_left = (int64_t)(j.in_end - in_dw);
    const uint32_t rel_end = (uint32_t)(in_left < 0x7ffffff0 ? in_left + 3 : 0x7ffffff0) & ~3u;
    // every lane's last window lies inside the input
    const bool end_ok = __ballot((int64_t)(base + (n_trips - 1) * NB + 4 * (NW + 1)) > in_left) == 0;
    // and the one after it, which belongs to later symbols
    const bool next_ok = __ballot((int64_t)base + (int64_t)n_trips * NB + 4 * (NW + 1) > in_left) == 0;
    const uint8_t *const win = in_dw + base;
    auto fetch = [&](uint32_t (&raw)[NW + 1], int trip) PBVD_INLINE_LAMBDA {
        const uint32_t *q = reinterpret_cast<const uint32_t *>(win + (int64_t)trip * NB);
        static_for<0, NW + 1>([&](auto jc) PBVD_INLINE_LAMBDA {
            raw[decltype(jc)::value] = q[decltype(jc)::value];
            return true;
        });
    };
    // hard bits as soft symbols: bit b -> 1 - 2 b in every byte
    auto soft = [&](uint32_t x) PBVD_INLINE_LAMBDA {
        if constexpr (KIND != kHardU8) return x;
        const uint32_t s = x & 0x01010101u;
        return 0x01010101u | ((s << 8) - s);
    };
    // symbols (as soft ones) with those before the PB's first read as 0;
    // dwords outside the input are not loaded
    auto fetch_safe = [&](uint32_t (&raw)[NW + 1], int trip) PBVD_INLINE_LAMBDA {
        static_for<0, NW + 1>([&](auto jc) PBVD_INLINE_LAMBDA {
            const int r = base + trip * NB + 4 * decltype(jc)::value;
            const bool ok = (uint32_t)r < rel_end;
            const uint32_t v = *reinterpret_cast<const uint32_t *>(in_dw + (ok ? r : 0));
            raw[decltype(jc)::value] = ok ? (r == 0 ? soft(v) & (0xffffffffu << (8 * mis)) : soft(v)) : 0u;
            return true;
        });
    };
    // (an explicit alignbit: a 64-bit shift of two neighbours is first made a
    // 64-bit load of the array, which then stays in memory, and its indexing
    // by thread made every wave read the launch's packet from host memory at
    // its start: 14 us until the last of 1024 waves had begun)
    auto align_trip = [&](uint32_t (&raw)[NW + 1], uint32_t (&w)[NW], auto convert) PBVD_INLINE_LAMBDA {
        static_for<0, NW>([&](auto jc) PBVD_INLINE_LAMBDA {
            constexpr int jj = decltype(jc)::value;
            constexpr bool kConvert = decltype(convert)::value;
            const uint32_t lo = kConvert ? soft(raw[jj]) : raw[jj], hi = kConvert ? soft(raw[jj + 1]) : raw[jj + 1];
            w[jj] = __builtin_amdgcn_alignbit(hi, lo, sh);
            return true;
        });
    };
    // symbols b0 and b1 (byte numbers of the trip) times 16 in the two halves
    auto pair_of = [&](const uint32_t (&w)[NW], auto b0c, auto b1c) PBVD_INLINE_LAMBDA {
        constexpr int b0 = decltype(b0c)::value, b1 = decltype(b1c)::value;
        constexpr int d0 = b0 / 4, d1 = b1 / 4;
        static_assert(d1 == d0 || d1 == d0 + 1, "neighbours");
        // each symbol to the top byte of its half, 0 below
        constexpr uint32_t sel = 0x0cu | (uint32_t)(b0 % 4) << 8 | 0x0cu << 16 | (uint32_t)(b1 % 4 + 4 * (d1 - d0)) << 24;
        const uint32_t x = __builtin_amdgcn_perm(w[d1], w[d0], sel);
        const T v = __builtin_bit_cast(T, x);
        return (T)(v >> (T)(8 - kTagBits));
    };

    // ---- metrics ----
    T pm[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) pm[r] = PM16::make(0, 0);
    auto bcast_state = [&](int s, auto phc) PBVD_INLINE_LAMBDA -> T {
        // metric of state s (compile-time) at phase PH in both halves
        constexpr int PH = decltype(phc)::value;
        const int u = rotl_v<V>(s, PH);
        const int r = u & (C::NR - 1);
        T m = (u >> (V - 1)) ? PM16::bcast_hi(pm[r & (NR - 1)]) : PM16::bcast_lo(pm[r & (NR - 1)]);
        if constexpr (LB > 0) {
            const int owner = r >> (V - 1 - LB);
            const T q0 = PM16::template dpp<quad_sel(0, 0, LB == 1 ? 2 : 0, LB == 1 ? 2 : 0)>(m);
            const T q1 = PM16::template dpp<quad_sel(1, 1, LB == 1 ? 3 : 1, LB == 1 ? 3 : 1)>(m);
            if constexpr (LB == 1) {
                m = owner ? q1 : q0;
            } else {
                const T q2 = PM16::template dpp<quad_sel(2, 2, 2, 2)>(m);
                const T q3 = PM16::template dpp<quad_sel(3, 3, 3, 3)>(m);
                m = (owner & 3) == 0 ? q0 : (owner & 3) == 1 ? q1 : (owner & 3) == 2 ? q2 : q3;
            }
            if constexpr (LB == 3) m = owner & 4 ? PM16::each(m, bit2_hi) : PM16::each(m, bit2_lo);
        }
        return m;
    };
    uint32_t keep = 0xfff0fff0u;  // metric bits of both halves
    asm("" : "+v"(keep));
    // set the tags for group q (TAGS) or clear them
    auto set_tags = [&](auto qc, auto tagsc) PBVD_INLINE_LAMBDA {
        constexpr int q = decltype(qc)::value % CY;
        constexpr bool kTags = decltype(tagsc)::value;
        uint32_t mine = 0;  // the lane's bits of the position
        if constexpr (LB > 0 && kTags) {
#pragma unroll
            for (int k = 0; k < kTagBits; ++k) {
                constexpr int kLow = V - 1 - LB;
                const int t = LY::phase(q, k);
                if (t >= kLow && t < V - 1) mine |= (uint32_t)((ell >> (t - kLow)) & 1) << k;
            }
            mine |= mine << 16;
        }
        static_for<0, NR>([&](auto rc) PBVD_INLINE_LAMBDA {
            constexpr int r = decltype(rc)::value;
            constexpr uint32_t c = LY::tag(q, r) | LY::tag(q, r | 1 << (V - 1)) << 16;
            const uint32_t v = __builtin_bit_cast(uint32_t, pm[r]);
            uint32_t s;
            if constexpr (!kTags) s = v & 0xfff0fff0u;
            else if constexpr (LB == 0) s = keep_or(v, keep, c);
            else s = keep_or_v(v, keep, mine | c);
            pm[r] = __builtin_bit_cast(T, s);
            return true;
        });
    };

    const __amdgpu_buffer_rsrc_t sp_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(sp_wave, (short)0, (int)(sp_dwords * 4), kBufferFlags);
    constexpr int kGroupBytes = NDW * kWave * 4;
    // gather and store the tags of the group that ends (row >= 0)
    auto store_tags = [&](int row) PBVD_INLINE_LAMBDA {
        static_for<0, NDW / 2>([&](auto cc) PBVD_INLINE_LAMBDA {
            constexpr int c = decltype(cc)::value;
            uint32_t v[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = (2 * c + i) * 2;  // registers r, r+1 and the two with bit B set
                constexpr int kTop = 1 << LY::B;
                const uint32_t lo = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, pm[r + 1]),
                                                          __builtin_bit_cast(uint32_t, pm[r]), 0x06040200u);
                const uint32_t hi = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, pm[(r | kTop) + 1]),
                                                          __builtin_bit_cast(uint32_t, pm[r | kTop]), 0x06040200u);
                v[i] = (lo & 0x0f0f0f0fu) | (hi << 4 & 0xf0f0f0f0u);
            }
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, sp_rsrc, lane * 8 + c % 8 * kWave * 8,
                                                  row * kGroupBytes + c / 8 * 4096, kRowPolicy);
            return true;
        });
    };

    // ---- one trip: kWarm no tags, kStore tags of groups from g0 on, kSlow
    //      the same with forced upper branches (known starts) ----
    enum { kWarm, kStore, kSlow };
    uint32_t w[NW];
    constexpr uint64_t kBit[3] = {0xaaaaaaaaaaaaaaaaull, 0xccccccccccccccccull, 0xf0f0f0f0f0f0f0f0ull};
    auto run_trip = [&](auto modec, int trip) PBVD_INLINE_LAMBDA {
        constexpr int MODE = decltype(modec)::value;
        auto stage = [&](auto kc) PBVD_INLINE_LAMBDA {
            constexpr int k = decltype(kc)::value, PH = k % V;
            // symbols of the stage times 16, two to a register
            T q[R];
            auto sym = [&](auto rc) PBVD_INLINE_LAMBDA {
                constexpr int r = decltype(rc)::value;
                if constexpr (r + 1 < R) {
                    const T x = pair_of(w, std::integral_constant<int, k * R + r>{}, std::integral_constant<int, k * R + r + 1>{});
                    q[r] = PM16::bcast_lo(x);
                    q[r + 1] = PM16::bcast_hi(x);
                } else {
                    q[r] = pair_of(w, std::integral_constant<int, k * R + r>{}, std::integral_constant<int, k * R + r>{});
                }
            };
            sym(std::integral_constant<int, 0>{});
            if constexpr (R > 2) sym(std::integral_constant<int, 2>{});
            // what the stage subtracts from every metric: at the reference
            // phases (slow trips: at every stage, but not while a known start
            // is under way) the reference, with `center` half the symbol sum
            bool force = false;
            if constexpr (MODE == kSlow) force = j.known && trip * U + k - vs < V && trip * U + k >= vs;
            constexpr bool kRef = MODE == kSlow || PH % kPlan.period == 0;
            T shift = PM16::make(0, 0);
            if constexpr (kPlan.center) {
                T sum = q[0];
#pragma unroll
                for (int r = 1; r < R; ++r) sum = PM16::add(sum, q[r]);
                shift = (T)(sum >> (T)1);
            }
            if constexpr (kRef) {
                constexpr std::integral_constant<int, PH> phc{};
                T ref;
                constexpr int kLog = kPlan.n_ref == 2 ? 1 : 2;  // divided before they are added: no overflow
                ref = (T)(bcast_state(kPlan.ref[0], phc) >> (T)kLog);
#pragma unroll
                for (int i = 1; i < kPlan.n_ref; ++i) ref = PM16::add(ref, (T)(bcast_state(kPlan.ref[i], phc) >> (T)kLog));
                if constexpr (MODE == kSlow) ref = force ? PM16::make(0, 0) : ref;
                shift = PM16::add(shift, ref);
            }
            constexpr bool kShift = kPlan.center || kRef;
            if constexpr (kShift)
                shift = __builtin_bit_cast(T, __builtin_bit_cast(uint32_t, shift) & 0xfff0fff0u);  // keep the tags
            // branch metrics: the halves differ in the column of their
            // position bit (at phase V-1 in the input's)
            constexpr int GP = PH < V - 1 ? C::gcol(V - 1 - PH) : C::gcol(C::K - 1);
            T pair[NC];
            {
                T p0 = PM16::sub(PM16::make(0, 0), shift);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if ((GP >> (R - 1 - r)) & 1)
                        p0 = PM16::add(p0, __builtin_bit_cast(T, __builtin_bit_cast(uint32_t, q[r]) & 0xffff0000u));
                pair[0] = p0;
                // code word c from c without its lowest bit
                T step[R];
#pragma unroll
                for (int r = 0; r < R; ++r) step[r] = (GP >> (R - 1 - r)) & 1 ? (T)(q[r] * T{1, -1}) : q[r];
#pragma unroll
                for (int c = 1; c < NC; ++c) {
                    const int low = c & -c;
                    const int r = R - 1 - (low == 1 ? 0 : low == 2 ? 1 : low == 4 ? 2 : 3);
                    pair[c] = PM16::add(pair[c ^ low], step[r]);
                }
            }
            if constexpr (LB > 0) {
                auto relabel = [&](auto mc, auto jc) PBVD_INLINE_LAMBDA {
                    constexpr int M = decltype(mc)::value;
                    if constexpr (M != 0) {
                        T t[NC];
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            t[c] = __builtin_bit_cast(T, select_lanes(__builtin_bit_cast(int, pair[c]),
                                                                      __builtin_bit_cast(int, pair[c ^ M]),
                                                                      kBit[decltype(jc)::value]));
#pragma unroll
                        for (int c = 0; c < NC; ++c) pair[c] = t[c];
                    }
                };
                relabel(std::integral_constant<int, tag_lane_mask<C, LB>(PH, 0)>{}, std::integral_constant<int, 0>{});
                if constexpr (LB >= 2)
                    relabel(std::integral_constant<int, tag_lane_mask<C, LB>(PH, 1)>{}, std::integral_constant<int, 1>{});
                if constexpr (LB >= 3)
                    relabel(std::integral_constant<int, tag_lane_mask<C, LB>(PH, 2)>{}, std::integral_constant<int, 2>{});
            }
            acs_tags<C, PH, LB, MODE == kSlow>(pm, pair, force, ell);
        };
        static_for<0, U>([&](auto kc) PBVD_INLINE_LAMBDA {
            constexpr int k = decltype(kc)::value;
            // (the stages before the wave's first leave the metrics 0)
            if (MODE != kSlow || trip * U + k >= off) stage(kc);
            if constexpr (MODE != kWarm && (k + 1) % kTagBits == 0) {
                constexpr int q = k / kTagBits;
                const int g = trip * CY + q;
                if (g >= g0) store_tags(g - g0);
                set_tags(std::integral_constant<int, q + 1>{}, std::true_type{});
            }
            return true;
        });
    };
    constexpr std::integral_constant<int, 0> kFirstGroup{};
    constexpr std::integral_constant<int, kWarm> kWarmTrip{};
    constexpr std::integral_constant<int, kStore> kStoreTrip{};
    constexpr std::integral_constant<int, kSlow> kSlowTrip{};

    // Trips: slow ones while a later trip still holds a lane's start or a
    // known start is under way (their successors' symbols are fetched
    // safely), then the warm-up trips that lie before the first traced group,
    // then the storing ones.  Where the window after the last trip's runs past
    // the input the last one is a slow one again, the last two where its own
    // does.  A slow trip takes half as long again per stage, but the first trip
    // as a slow one leaves out the stages before the wave's first.  (With
    // a slow last trip in every wave, and without: 48Ki blocks of 64 bits of
    // K = 7 54.3 and 52.3 us, 128Ki of 16 bits of K = 8 136.6 and 129.6.)
    uint32_t raw[NW + 1];
    fetch_safe(raw, 0);
    align_trip(raw, w, std::false_type{});
    const int hot_end = n_trips - (next_ok ? 0 : end_ok ? 1 : 2);
    int n_slow = (start_hi + U - 1) / U - 1;
    if ((force_end + U - 1) / U > n_slow) n_slow = (force_end + U - 1) / U;
    int trip = 0;
    set_tags(kFirstGroup, std::true_type{});
    auto slow_trips = [&](int end) PBVD_INLINE_LAMBDA {
        for (; trip < end; ++trip) {
            if (trip + 1 < n_trips) fetch_safe(raw, trip + 1);
            run_trip(kSlowTrip, trip);
            align_trip(raw, w, std::false_type{});
        }
    };
    const int warm_end = ds_lo / U < hot_end ? ds_lo / U : hot_end;
    int slow_end = n_slow < hot_end ? n_slow : n_trips;
    for (;;) {
        slow_trips(slow_end);
        if (trip >= n_trips) break;
        if (trip < warm_end) {
            set_tags(kFirstGroup, std::false_type{});
            for (; trip < warm_end; ++trip) {
                fetch(raw, trip + 1);
                run_trip(kWarmTrip, trip);
                align_trip(raw, w, std::true_type{});
            }
            set_tags(kFirstGroup, std::true_type{});
        }
        for (; trip < hot_end; ++trip) {
            fetch(raw, trip + 1);
            run_trip(kStoreTrip, trip);
            align_trip(raw, w, std::true_type{});
        }
        slow_end = n_trips;
    }

    // ---- final metrics and traceback start (Sec. III-A; Sec. II at an
    //      unterminated stream end); the wave ends at phase 0: position u
    //      holds state u ----
    uint32_t idx = 0;
    auto state_idx = [&](uint32_t u) PBVD_INLINE_LAMBDA {
        uint32_t v = 0;
#pragma unroll
        for (int t = 0; t < V; ++t) v |= ((u >> t) & 1u) << LY::pos(t);
        return v;
    };
    if (j.need_final) {
        const int ubase = ell << (V - 1 - LB);
        // a start from state 0 fewer than V stages back reaches only states
        // with that many low zero bits
        const int reach = j.known && j.my_len < V ? (1 << (V - j.my_len)) - 1 : 0;
        auto metric = [&](T v, int half, int s) PBVD_INLINE_LAMBDA {
            const int m = (half ? PM16::hi(v) : PM16::lo(v)) >> kTagBits;
            return s & reach ? 0x7fffffff : m;
        };
        int m = 0x7fffffff;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            m = min(m, metric(pm[r], 0, ubase | r));
            m = min(m, metric(pm[r], 1, ubase | r | (1 << (V - 1))));
        }
        if constexpr (LB >= 1) m = min(m, dpp_int<quad_flip<0>()>(m));
        if constexpr (LB >= 2) m = min(m, dpp_int<quad_flip<1>()>(m));
        if constexpr (LB >= 3) m = min(m, bit2_flip(m));
        if (j.argmin) {
            int best = C::N;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int s_lo = ubase | r, s_hi = s_lo | (1 << (V - 1));
                if (metric(pm[r], 0, s_lo) == m && s_lo < best) best = s_lo;
                if (metric(pm[r], 1, s_hi) == m && s_hi < best) best = s_hi;
            }
            if constexpr (LB >= 1) best = min(best, dpp_int<quad_flip<0>()>(best));
            if constexpr (LB >= 2) best = min(best, dpp_int<quad_flip<1>()>(best));
            if constexpr (LB >= 3) best = min(best, bit2_flip(best));
            idx = state_idx((uint32_t)best);
        }
        if (j.pm_out && j.active) {
            // (the host asks for final metrics only where every state is reached)
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                j.pm_out[ubase | r] = (PM16::lo(pm[r]) >> kTagBits) - m;
                j.pm_out[ubase | r | (1 << (V - 1))] = (PM16::hi(pm[r]) >> kTagBits) - m;
            }
        }
    }

    // ---- traceback (Alg. 1), a group at a time: the group's input bits are
    //      the bits of its phases in the position at its end, the tag replaces
    //      them by the decisions.  Rows do not depend on the traced state and
    //      are loaded ahead into a ring; each lane of a group loads what it
    //      stored.  Input bits are collected in words of 32 virtual stages; a
    //      lane's output words start at ds and span two of them. ----
    const bool writer = j.active && ell == 0;
    // kOutEdges: bits up to the PB's first whole byte
    const int head = j.out_mode == kOutEdges ? (int)(-j.out_bit0 & 7) : 0;
    auto put_word = [&](uint32_t v, int rel) PBVD_INLINE_LAMBDA {
        const int nb = n_dec - rel < 32 ? n_dec - rel : 32;
        if (nb < 32) v &= (1u << nb) - 1u;
        const int64_t bitpos = j.out_bit0 + rel;
        if (j.out_mode == kOutAtomic) {
            const uint32_t s = (uint32_t)(bitpos & 31);
            uint32_t *wp = j.out_words + (bitpos >> 5);
            atomicOr(wp, v << s);
            if (s && (v >> (32 - s))) atomicOr(wp + 1, v >> (32 - s));
        } else {
            // the lane owns whole bytes: its first bit is byte aligned
            uint8_t *ob = j.out + (bitpos >> 3);
            if (nb == 32 && (((uintptr_t)ob & 3u) == 0)) {
                *reinterpret_cast<uint32_t *>(ob) = v;
            } else {
                const bool shared = j.out_mode == kOutEdges && (nb & 7) != 0 && bitpos + nb != j.out_bits;
                for (int bb = 0; bb < ((nb + (shared ? 0 : 7)) >> 3); ++bb) ob[bb] = (uint8_t)(v >> (8 * bb));
                if (shared) put_edge(j.out_words + j.edge + 1, ob + (nb >> 3), v >> (nb & ~7) & 0xffu, j.edge_call);
            }
        }
    };
    // the PB's bits before its first whole byte (kOutEdges)
    auto put_head = [&](uint32_t v) PBVD_INLINE_LAMBDA {
        v &= (1u << (n_dec < head ? n_dec : head)) - 1u;
        put_edge(j.out_words + j.edge, j.out + (j.out_bit0 >> 3), v << (j.out_bit0 & 7), j.edge_call);
    };
    uint32_t word = 0, above = 0;
    auto emit = [&](int g) PBVD_INLINE_LAMBDA {
        // word holds the stages from 4 g up; the word of 32 that contains it
        const int v0 = (g & ~7) * kTagBits;
        const uint32_t cur = word << ((g & 7) * kTagBits);
        const int rel = v0 + ((ds + head) & 31) - ds;  // head and a multiple of 32
        const uint32_t v = __builtin_amdgcn_alignbit(above, cur, (uint32_t)(ds + head) & 31u);
        if (writer && rel >= 0 && rel < n_dec) put_word(v, rel);
        if (j.out_mode == kOutEdges && writer && rel < 0 && rel > -32) put_head(v >> -rel);
        above = cur;
        word = 0;
    };
    // byte offset of a group's row; rows before the first are not used and
    // read the first
    auto load_group = [&](uint32_t (&dst)[NDW], int off) PBVD_INLINE_LAMBDA {
        static_for<0, NDW / 2>([&](auto cc) PBVD_INLINE_LAMBDA {
            constexpr int c = decltype(cc)::value;
            const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(sp_rsrc, lane * 8 + c % 8 * kWave * 8, off + c / 8 * 4096,
                                                                 kRowPolicy);
            dst[2 * c] = t.x;
            dst[2 * c + 1] = t.y;
            return true;
        });
    };
    // the tag of idx in the low bits (garbage above)
    auto lookup = [&](const uint32_t (&row)[NDW]) PBVD_INLINE_LAMBDA {
        uint32_t v[NDW];
#pragma unroll
        for (int i = 0; i < NDW; ++i) v[i] = row[i];
        constexpr int kLog = NDW >= 32 ? 5 : NDW >= 16 ? 4 : NDW >= 8 ? 3 : 2;
#pragma unroll
        for (int half = NDW / 2, bit = 4 + kLog; half >= 1; half /= 2, --bit) {
            const uint32_t up = (uint32_t)((int)(idx << (31 - bit)) >> 31);
#pragma unroll
            for (int i = 0; i < half; ++i) v[i] = bit_select(up, v[i + half], v[i]);
        }
        uint32_t s = v[0];
        if constexpr (LB > 0) {
            const uint32_t owner = (idx >> (5 + kLog)) & ((1u << LB) - 1);
            if constexpr (LB == 1) {
                const uint32_t b0 = (uint32_t)dpp_int<quad_sel(0, 0, 2, 2)>((int)s);
                const uint32_t b1 = (uint32_t)dpp_int<quad_sel(1, 1, 3, 3)>((int)s);
                s = owner ? b1 : b0;
            } else {
                const uint32_t b0 = (uint32_t)dpp_int<quad_sel(0, 0, 0, 0)>((int)s);
                const uint32_t b1 = (uint32_t)dpp_int<quad_sel(1, 1, 1, 1)>((int)s);
                const uint32_t b2 = (uint32_t)dpp_int<quad_sel(2, 2, 2, 2)>((int)s);
                const uint32_t b3 = (uint32_t)dpp_int<quad_sel(3, 3, 3, 3)>((int)s);
                s = owner & 2u ? (owner & 1u ? b3 : b2) : (owner & 1u ? b1 : b0);
                if constexpr (LB == 3) {
                    const uint32_t other = (uint32_t)bit2_flip((int)s);
                    s = ((owner >> 2) & 1u) != (uint32_t)((ell >> 2) & 1) ? other : s;
                }
            }
        }
        return s >> (idx & 31u);
    };
    auto step = [&](auto qc, const uint32_t (&row)[NDW]) PBVD_INLINE_LAMBDA {
        constexpr int q = decltype(qc)::value;
        // the phases' bits of idx in runs of consecutive places
        constexpr auto run_of = [](int k) {
            int n = 1;
            while (k + n < kTagBits && LY::pos(LY::phase(q, k + n)) == LY::pos(LY::phase(q, k)) + n) ++n;
            return n;
        };
        const uint32_t t = lookup(row);
        uint32_t nib = 0, next = idx;
        static_for<0, kTagBits>([&](auto kc) PBVD_INLINE_LAMBDA {
            constexpr int k = decltype(kc)::value;
            constexpr int p = LY::pos(LY::phase(q, k));
            if constexpr (k == 0 || LY::pos(LY::phase(q, k == 0 ? 0 : k - 1)) + 1 != p) {
                constexpr uint32_t m = (1u << run_of(k)) - 1u;
                nib |= ((idx >> p) & m) << k;
                next = (next & ~(m << p)) | ((p >= k ? t << (p - k) : t >> (k - p)) & (m << p));
            }
            return true;
        });
        word = word << kTagBits | nib;
        idx = next;
    };
    constexpr int kRing = LY::kRing;
    uint32_t ring[kRing][NDW];
    int row_off = (n_groups - 1 - g0) * kGroupBytes;  // of the row to load next
    auto load_next = [&](uint32_t (&dst)[NDW]) PBVD_INLINE_LAMBDA {
        load_group(dst, row_off);
        row_off -= kGroupBytes;
        asm("" : "+s"(row_off));  // or the two become a saturating vector subtraction
        row_off = row_off > 0 ? row_off : 0;
    };
    static_for<0, kRing - 1>([&](auto dc) PBVD_INLINE_LAMBDA {
        load_next(ring[decltype(dc)::value]);
        return true;
    });
    // a word of 32 stages is complete at every eighth group and at the first
    // one; the groups down to there are counted, so that a step on the way has
    // one scalar subtraction and a branch not taken
    int event = (n_groups - 1) & ~7;
    if (event < g0) event = g0;
    int left = n_groups - event;
    for (;;) {
        const bool more = static_for<0, kRing>([&](auto dc) PBVD_INLINE_LAMBDA {
            constexpr int d = decltype(dc)::value;
            load_next(ring[(d + kRing - 1) % kRing]);
            step(std::integral_constant<int, CY - 1 - d % CY>{}, ring[d]);
            if (__builtin_expect(--left == 0, 0)) {
                emit(event);
                if (event == g0) return false;
                left = event - g0 < 8 ? event - g0 : 8;
                event -= left;
            }
            return true;
        });
        if (!more) break;
    }
    if (j.out_mode == kOutEdges) emit((g0 & ~7) - 8);  // heads in the word below
}

}  // namespace pbvd
