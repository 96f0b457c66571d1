// Wave-level building blocks shared by the edge-streaming kernels: DPP
// shifts and the inclusive wave sum, and raw buffer descriptor constants.
#pragma once

#include "common.h"

namespace cagra {

// ---- wave-level scans with DPP (row shifts within 16 lanes, then row broadcasts)
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143, kDppWaveShr1 = 0x138;

template <int CTRL, int ROWMASK>
__device__ __forceinline__ int32_t dpp_i(int32_t old, int32_t x) {
    return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWMASK, 0xf, false);
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_f(float old, float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL, ROWMASK, 0xf,
                                                      false));
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ int32_t dpp_t(int32_t old, int32_t x) { return dpp_i<CTRL, ROWMASK>(old, x); }
template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_t(float old, float x) { return dpp_f<CTRL, ROWMASK>(old, x); }

template <int CTRL, int ROWMASK>
__device__ __forceinline__ void add_step(int32_t &x) { x += dpp_i<CTRL, ROWMASK>(0, x); }

__device__ __forceinline__ int32_t wave_incl_sum(int32_t x) {
    add_step<kDppRowShr1, 0xf>(x);
    add_step<kDppRowShr2, 0xf>(x);
    add_step<kDppRowShr4, 0xf>(x);
    add_step<kDppRowShr8, 0xf>(x);
    add_step<kDppRowBcast15, 0xa>(x);
    add_step<kDppRowBcast31, 0xc>(x);
    return x;
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ void max_step(int32_t &x) {
    x = max(x, dpp_i<CTRL, ROWMASK>(0, x));
}
// Inclusive maximum over the wave of values >= 0.
__device__ __forceinline__ int32_t wave_incl_max(int32_t x) {
    max_step<kDppRowShr1, 0xf>(x);
    max_step<kDppRowShr2, 0xf>(x);
    max_step<kDppRowShr4, 0xf>(x);
    max_step<kDppRowShr8, 0xf>(x);
    max_step<kDppRowBcast15, 0xa>(x);
    max_step<kDppRowBcast31, 0xc>(x);
    return x;
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ void or_step(int32_t &x) {
    x |= dpp_i<CTRL, ROWMASK>(0, x);
}
__device__ __forceinline__ uint32_t wave_or(int32_t x) {
    or_step<kDppRowShr1, 0xf>(x);
    or_step<kDppRowShr2, 0xf>(x);
    or_step<kDppRowShr4, 0xf>(x);
    or_step<kDppRowShr8, 0xf>(x);
    or_step<kDppRowBcast15, 0xa>(x);
    or_step<kDppRowBcast31, 0xc>(x);
    return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}
// The wave's values OR-ed, in scalar registers.
__device__ __forceinline__ uint64_t wave_or64(uint64_t x) {
    return (uint64_t)wave_or((int32_t)(uint32_t)(x >> 32)) << 32 | wave_or((int32_t)(uint32_t)x);
}
// Bits of a uniform mask below the lane's.
__device__ __forceinline__ int32_t lanes_below(uint64_t m) {
    return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// A value that is the same in the whole wave, in scalar registers (the compiler
// loads it per lane where the kernel also writes memory).
__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename P>
__device__ __forceinline__ P *uniform(P *p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(a >> 32));
    return reinterpret_cast<P *>(((uint64_t)hi << 32) | lo);
}

constexpr int32_t kBufFlags = 0x00020000;   // raw buffer descriptor word 3 (gfx9)
constexpr int kNonTemporal = 2;             // cache policy: streaming
constexpr uint32_t kOutOfRange = 0x80000000u;

}  // namespace cagra
