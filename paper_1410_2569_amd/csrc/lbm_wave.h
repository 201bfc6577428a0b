// lbm_wave.h -- a wave's cross-lane moves for the marching strips (lbm_march.h).
#pragma once
#include <hip/hip_runtime.h>

namespace lbm {

// DPP wavefront shifts by one lane; a lane past the end reads 0.
struct DppLane {
    // hides a value's origin, so that nothing computed from it leaves its place
    static __device__ __forceinline__ void opaque(unsigned& v) { asm volatile("" : "+v"(v)); }
    template <int CTRL>
    static __device__ __forceinline__ double shift(double v) {
        union { double d; int i[2]; } u;
        u.d = v;
        u.i[0] = __builtin_amdgcn_update_dpp(0, u.i[0], CTRL, 0xf, 0xf, true);
        u.i[1] = __builtin_amdgcn_update_dpp(0, u.i[1], CTRL, 0xf, 0xf, true);
        return u.d;
    }
    static __device__ __forceinline__ double left(double v) { return shift<0x138>(v); }   // wave_shr:1
    static __device__ __forceinline__ double right(double v) { return shift<0x130>(v); }  // wave_shl:1
};

// Waves of a marching workgroup: neighbouring strips of one segment, one per SIMD of a compute unit.
constexpr int kMarchWaves = 4;

}  // namespace lbm
