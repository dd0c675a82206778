// Kernels of the register mapping: the stream kernel and the batch (tile)
// kernels, on the tag body (pbvd_tags.hpp: 16-bit metrics, 32 states and more)
// or the row body (decode_body of pbvd_kernel.hpp: 32-bit metrics, and the
// trellises of 4 to 16 states, whose several stages share a survivor dword).
#pragma once

#include "pbvd_tags.hpp"

namespace pbvd {

// Register target for the 256-state trellis (waves per SIMD the compiler
// must leave room for).  Two waves force scratch spills inside the stage
// loop, which measured 2x slower than one wave with accumulator-register
// spills.
#ifndef PBVD_BIG_TRELLIS_WAVES_PER_EU
#define PBVD_BIG_TRELLIS_WAVES_PER_EU 1
#endif
// Register target for 64 metric VGPRs per lane (a 256-state trellis on lane
// pairs or 128 states on one lane, 16-bit metrics).  Three waves spill: K = 9 rate
// 1/3 on pairs 88 registers in the stream kernel and 164 in the tile kernel
// (whose two bodies share it), K = 8 on one lane 84 and 168, mostly outside the
// stage loops; the storing loop of K = 9 moves 43 per trip of 8 stages (some
// 2,250 vector instructions), that of K = 8 3 to 6 per 28 stages, the stream
// kernel's warm-up loops none.  With room for two waves K = 9 rate 1/3 on pairs is
// 4 to 8 % faster at D = 64 (64Ki PBs 228 -> 211 us) and 1 to 3 % slower on long
// streams of D = 512 (256Ki PBs 2962 -> 3057 us).
#ifndef PBVD_MID_TRELLIS_WAVES_PER_EU
#define PBVD_MID_TRELLIS_WAVES_PER_EU 3
#endif
// MW = VGPRs of path metrics per lane
template <int MW>
__host__ __device__ constexpr int waves_per_eu_target() {
    return MW >= 128 ? PBVD_BIG_TRELLIS_WAVES_PER_EU : (MW >= 64 ? PBVD_MID_TRELLIS_WAVES_PER_EU : 1);
}

// The wave's PBs on the body of the code and metric width.
template <class C, class P, int KIND, bool VARLEN, int LB>
__device__ __forceinline__ void wave_body(const WaveJob &j, uint32_t *sp, int64_t sp_dwords) {
    if constexpr (uses_tags<C, P>()) {
        tag_body<C, KIND, VARLEN, LB>(j, sp, sp_dwords);
    } else {
        static_assert(LB == 0, "the row body decodes a PB per lane");
        using LY = Layout<C, P>;
        RowStore<LY::NDW> rows;
        rows.rsrc = __builtin_amdgcn_make_buffer_rsrc(sp, (short)0, (int)(sp_dwords * 4), kBufferFlags);
        rows.lane_off = (uint32_t)(threadIdx.x & (kWave - 1)) * (LY::NDW * 4);
        decode_body<C, P, KIND, VARLEN>(j, rows);
    }
}

// ---------------------------------------------------------------------------
// Stream kernel: the PBs of one stream (Sec. III-A, Fig. 2).  Interior PBs
// (full geometry) go 64 to a wave.  PBs at the stream ends take the free
// slots the interior leaves (moved to the front of wave 0), so that they add
// no wave of their own while there is room; the others get a wave each.
// Waves of one SIMD run nearly one after another (the oldest wave issues
// first), so a single extra wave lengthens the whole launch by its share.
// ---------------------------------------------------------------------------
template <class C, class P, int KIND, int LB>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(waves_per_eu_target<(C::NR >> LB) * (int)(sizeof(typename P::T) / 4)>())))
    decode_kernel(const KernelArgs a) {
    constexpr int R = C::R, N = C::N, PW = kWave >> LB;
    constexpr int ND = (Layout<C, P>::U * R + 3) / 4 + 1;

    const int lane = threadIdx.x & (kWave - 1);
    const int pl = lane >> LB;  // the lane's PB inside the wave
    // wave index made provably uniform so that all geometry stays scalar
    const int64_t wave_local = (int64_t)blockIdx.x * (blockDim.x / kWave) +
                               __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (wave_local >= a.n_waves) return;
    const int64_t wave = a.wave_begin + wave_local;
    const int64_t D = a.D, L = a.L;

    uint32_t *const sp = a.sp + wave_local * a.sp_wave_dwords;
    WaveJob j;
    j.out_mode = a.out_mode;
    j.out = a.out;
    j.out_words = a.out_words;
    j.out_bits = a.out_bits;
    j.edge_call = a.edge_call;
    j.in_end = a.syms + a.T * R;

    if (wave == 0 && a.n_fold > 0) {
        // ---- wave 0 with folded edge PBs: every lane has its own geometry
        //      (Sec. III-A, clipped to the stream), decoded like a batch tile.
        //      In the row body all lanes start together and a lane shorter than
        //      the wave runs on past its own end, so its metrics at the wave's
        //      end are not its final metrics: therefore the host folds no PB
        //      that starts its traceback from the best state and folds nothing
        //      when final metrics are asked for.  (In the tag body all lanes
        //      end together.) ----
        int64_t b;
        bool active = true;
        if (pl < a.n_fold) {
            b = pl < a.n_head ? a.pb_first + pl : a.b_hi + (pl - a.n_head);
        } else {
            b = a.b_lo + (pl - a.n_fold);
            if (b >= a.b_hi) {
                b = a.b_hi - 1;
                active = false;
            }
        }
        const int64_t d0 = b * D;
        const int64_t f0 = d0 - L < 0 ? 0 : d0 - L;
        const int64_t f1 = d0 + D + L > a.T ? a.T : d0 + D + L;
        const int64_t d1 = d0 + D > a.n ? a.n : d0 + D;
        j.len = (int)(D + 2 * L);
        j.store0_min = a.n_head > 0 ? (int)(a.pb_first * D) : (int)L;
        j.i_safe = a.fold_i_safe;
        j.fetch_safe = a.fold_wide != 0;
        j.need_final = false;
        j.in = a.syms + f0 * R;
        j.my_len = (int)(f1 - f0);
        j.my_store0 = (int)(d0 - f0);
        j.my_dec_end = (int)(d1 - f0);
        j.known = f0 == 0;
        j.argmin = false;
        j.active = active;
        j.store0_uniform = false;
        j.out_bit0 = (b - a.pb_first) * D;
        j.edge = (int)(b - a.pb_first);
        j.pm_out = nullptr;
        wave_body<C, P, KIND, true, LB>(j, sp, a.sp_wave_dwords);
        return;
    }

    // ---- block geometry (Sec. III-A with M = L, clipped to the stream) ----
    int64_t b, f0w, f1w, d0w, d1w;   // wave-uniform PB geometry (interior: lane 0's)
    bool active;
    int64_t lane_stage_off;           // this lane's stage offset from f0w
    int64_t far_lane;                 // the wave's last real lane
    if (wave < a.n_int_waves) {
        const int64_t bw = a.b_lo + wave * PW - a.n_fold;
        b = bw + pl;
        active = b < a.b_hi;
        lane_stage_off = (active ? (int64_t)pl : (a.b_hi - 1 - bw)) * D;
        if (!active) b = a.b_hi - 1;
        far_lane = a.b_hi - 1 - bw < PW - 1 ? a.b_hi - 1 - bw : PW - 1;
        d0w = bw * D;
        f0w = d0w - L;
        f1w = d0w + D + L;
        d1w = d0w + D;
    } else {
        const int64_t e = wave - a.n_int_waves + a.n_fold;
        b = e < a.n_head ? a.pb_first + e : a.b_hi + (e - a.n_head);
        active = pl == 0;
        lane_stage_off = 0;
        far_lane = 0;
        d0w = b * D;
        f0w = d0w - L < 0 ? 0 : d0w - L;
        f1w = d0w + D + L > a.T ? a.T : d0w + D + L;
        d1w = d0w + D > a.n ? a.n : d0w + D;
    }
    // stage counts fit in 32 bits (at most D + 2L), which keeps the loop
    // control on the scalar unit
    j.len = (int)(f1w - f0w);
    j.store0_min = (int)(d0w - f0w);
    j.my_len = j.len;
    j.my_store0 = j.store0_min;
    j.my_dec_end = (int)(d1w - f0w);
    j.in = a.syms + (f0w + lane_stage_off) * R;
    // wave-uniform: every wide fetch of every lane stays inside the input;
    // only the last wave(s) of a stream take the byte-load path
    j.fetch_safe = a.syms + (f0w + far_lane * D + (j.len - 1)) * R + 4 * ND <= j.in_end;
    const int64_t safe_bytes = (int64_t)(j.in_end - (a.syms + (f0w + far_lane * D) * R)) - 4 * ND;
    j.i_safe = safe_bytes < 0 ? -1 : (safe_bytes / R > j.len ? j.len : (int)(safe_bytes / R));
    j.known = f0w + lane_stage_off == 0;  // an interior PB can start at 0 when L is a multiple of D
    j.argmin = f1w == a.T && !a.terminated;
    j.need_final = j.argmin || a.final_pm != nullptr;
    j.active = active;
    j.store0_uniform = true;
    j.out_bit0 = (b - a.pb_first) * D;
    j.edge = (int)(b - a.pb_first);
    j.pm_out = a.final_pm ? a.final_pm + (b - a.pb_first) * N : nullptr;
    wave_body<C, P, KIND, false, LB>(j, sp, a.sp_wave_dwords);
}

// ---------------------------------------------------------------------------
// Batch kernel: one wave per tile of up to 64 >> LB PBs of one code taken
// from any frames (lengths may differ inside a tile).  With lane groups the
// descriptor of a PB is repeated for each lane of its group.
// ---------------------------------------------------------------------------
// One tile of a batch (the wave's PBs, their descriptors and survivor slot).
template <class C, class P, int KIND, int LB>
__device__ __forceinline__ void tile_body(const TileArgs &a, int64_t wave_local, int lane, const TileHead &h,
                                          int tflags) {
    const int64_t tile = a.tile_begin + wave_local;
    const LaneDesc d = a.lanes[tile * kWave + lane];

    WaveJob j;
    j.len = __builtin_amdgcn_readfirstlane(h.len);
    j.store0_min = __builtin_amdgcn_readfirstlane(h.store0_min);
    j.fetch_safe = (tflags & kTileWide) != 0;
    j.i_safe = j.fetch_safe ? j.len : __builtin_amdgcn_readfirstlane(h.i_safe);
    j.need_final = (tflags & kTileFinal) != 0;
    j.in_end = a.syms + a.sym_bytes;
    j.in = a.syms + d.sym;
    j.my_len = d.len;
    j.my_store0 = d.store0;
    j.my_dec_end = d.dec_end;
    j.known = (d.flags & kLaneKnown) != 0;
    j.argmin = (d.flags & kLaneArgmin) != 0;
    j.active = (d.flags & kLaneActive) != 0;
    j.store0_uniform = (tflags & kTileStore0) != 0;
    j.out_mode = kOutBytes;
    j.out = a.out;
    j.out_words = nullptr;
    j.out_bits = 0;
    j.edge_call = 0;
    j.edge = 0;
    j.out_bit0 = d.out_bit;
    j.pm_out = nullptr;

    uint32_t *const sp = a.sp + wave_local * a.sp_wave_dwords;
    if (tflags & kTileUniform) {
        j.my_len = j.len;
        j.my_store0 = j.store0_min;
        j.my_dec_end = __builtin_amdgcn_readfirstlane(d.dec_end);
        wave_body<C, P, KIND, false, LB>(j, sp, a.sp_wave_dwords);
    } else {
        wave_body<C, P, KIND, true, LB>(j, sp, a.sp_wave_dwords);
    }
}

template <class C, class P, int KIND, int LB>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(waves_per_eu_target<(C::NR >> LB) * (int)(sizeof(typename P::T) / 4)>())))
    decode_tiles_kernel(const TileArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave_local = (int64_t)blockIdx.x * (blockDim.x / kWave) +
                               __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (wave_local >= a.n_tiles) return;
    const TileHead h = a.heads[a.tile_begin + wave_local];
    tile_body<C, P, KIND, LB>(a, wave_local, lane, h, __builtin_amdgcn_readfirstlane(h.flags));
}

// Batch kernel for a pair of codes of one constraint length: the tiles of
// both in one launch (longest first over both), each tile decoded with the
// code its head names (kTileCode1: the second).  One launch instead of one
// per code: no fork and join of streams, and the waves of both codes share
// the compute units from the first to the last tile.
template <class C0, class C1, class P, int KIND, int LB>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(waves_per_eu_target<(C0::NR >> LB) * (int)(sizeof(typename P::T) / 4)>())))
    decode_tiles_pair_kernel(const TileArgs a) {
    static_assert(C0::K == C1::K, "a pair shares one trellis size");
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t wave_local = (int64_t)blockIdx.x * (blockDim.x / kWave) +
                               __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (wave_local >= a.n_tiles) return;
    const TileHead h = a.heads[a.tile_begin + wave_local];
    const int tflags = __builtin_amdgcn_readfirstlane(h.flags);
    if (tflags & kTileCode1) tile_body<C1, P, KIND, LB>(a, wave_local, lane, h, tflags);
    else tile_body<C0, P, KIND, LB>(a, wave_local, lane, h, tflags);
}

}  // namespace pbvd
