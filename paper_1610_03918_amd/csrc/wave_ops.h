// Wavefront reductions without LDS, and words exchanged between work-groups
// of one launch through device memory (gfx950).
#pragma once

#include "pic_internal.h"

namespace pic {

typedef unsigned long long u64;

__device__ __forceinline__ double dpp_add(double v, const int ctrl_kind)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    int l2, h2;
    switch (ctrl_kind) {
    case 0:                            // row_ror:8
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xF, 0xF, false);
        break;
    case 1:                            // row_ror:4
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0x124, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0x124, 0xF, 0xF, false);
        break;
    case 2:                            // quad_perm [2,3,0,1]
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, false);
        break;
    default:                           // quad_perm [1,0,3,2]
        l2 = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, false);
        h2 = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, false);
        break;
    }
    return v + __hiloint2double(h2, l2);
}

// a: lanes 0..31 of a and of b;  b: lanes 32..63 of a and of b.
__device__ __forceinline__ void swap32(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}

// The same with 16-lane rows: a gets rows 0, 2 of a and of b, b rows 1, 3.
__device__ __forceinline__ void swap16(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The wave_sum tree (partners 32, 16, 8, 4, 2, 1 lanes apart) of four values
// at once, without LDS: the two widest steps fold two values into one register.
// Uniform results.
__device__ __forceinline__ void wave_sum4(double (&v)[4])
{
    swap32(v[0], v[1]);
    double x = v[0] + v[1];            // lanes 0-31: value 0, 32-63: value 1
    swap32(v[2], v[3]);
    double y = v[2] + v[3];
    swap16(x, y);
    x = x + y;                         // rows 0, 2: values 0, 1; rows 1, 3: values 2, 3
    x = dpp_add(x, 0);
    x = dpp_add(x, 1);
    x = dpp_add(x, 2);
    x = dpp_add(x, 3);
    v[0] = lane_value(x, 0);
    v[1] = lane_value(x, 32);
    v[2] = lane_value(x, 16);
    v[3] = lane_value(x, 48);
}

// The same tree of one value.
__device__ __forceinline__ double wave_sum1(double x)
{
    double y = x;
    swap32(x, y);
    x = x + y;
    y = x;
    swap16(x, y);
    x = x + y;
    x = dpp_add(x, 0);
    x = dpp_add(x, 1);
    x = dpp_add(x, 2);
    x = dpp_add(x, 3);
    return lane_value(x, 0);
}

template <int N> struct Int {
    static constexpr int value = N;
};

__device__ __forceinline__ u64 ld_agent(const u64 *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(u64 *p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 tagged(unsigned data, unsigned epoch) { return ((u64)epoch << 32) | data; }

// True while a poll may go on; false once its time is up or another
// work-group gave up.  (A step that is not finite ends the launch too, but
// every word that is polled until then has been published by then.)
struct Patience {
    long long start;
    int spins;
    __device__ __forceinline__ Patience() : start(0), spins(0) {}
    __device__ __forceinline__ bool more(const int *abort_word, long long wait)
    {
        if (wait < 0) return false;
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 1023) != 0) return true;
        const long long now = wall_clock64();
        if (start == 0) start = now;
        if (now - start > wait) return false;
        return __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kAbortGaveUp;
    }
};

} // namespace pic
