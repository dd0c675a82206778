// State-parallel decoder of a work list whose codes have different constraint
// lengths: one launch, a wave per PB (pbvd_wave.hpp).
//
// What bounds it: a few hundred PBs are less than a wave per SIMD, so a launch
// lasts as long as its longest PB's chain of stages, and a launch for every K
// on forked streams, joined by events, cost more than the decoding: 64 frames
// of K = 3, 7 and 9 (40 to 6144 bits, D = 64) 55 -> 18 us.  The kernel has the
// registers of its largest K, 4 waves per SIMD at least.
#include "pbvd_wave.hpp"
#include "pbvd_registry.hpp"

namespace pbvd {
namespace wave {

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
    decode_wave_mixed_kernel(const Args a, const uint8_t *__restrict__ syms) {
    __shared__ __align__(16) uint32_t q_block[256];
    uint32_t *const q_lds = q_block + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * kWave;
    const int64_t wl = (int64_t)blockIdx.x * (blockDim.x / kWave) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (wl >= a.n_waves) return;
    uint32_t *const sp = a.sp + wl * a.sp_wave_dwords;
    int ci;
    bool active;
    const Job j = desc_job(a, syms, a.wave_begin + wl, &ci, &active);
    if (!active) return;
    switch (a.codes[ci].K) {
        case 3: return decode_pb<2, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        case 4: return decode_pb<3, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        case 5: return decode_pb<4, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        case 6: return decode_pb<5, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        case 7: return decode_pb<6, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        case 8: return decode_pb<7, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        case 9: return decode_pb<8, false>(a, j, a.codes[ci], sp, nullptr, q_lds);
        default: return;
    }
}

}  // namespace wave

hipError_t launch_wave_mixed(const WaveLaunchRequest &req) {
    hipLaunchKernelGGL(wave::decode_wave_mixed_kernel, dim3(req.grid), dim3(kBlockThreads), 0, req.stream, req.args,
                       req.args.syms);
    return hipGetLastError();
}

}  // namespace pbvd
