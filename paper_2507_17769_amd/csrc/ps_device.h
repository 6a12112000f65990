// Device-side helpers for the gfx950 kernels: bf16 packing, MFMA operand types, wave shuffles.
#pragma once
#include "ps_common.h"

#include <type_traits>

namespace ps {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));  // 4 bf16 bit patterns (16x16x16 MFMA operand)
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// two floats -> packed bf16 pair, round-to-nearest-even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    bf16x2_t v;
    v.x = (__bf16)lo;
    v.y = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

__device__ __forceinline__ uint4 ldg16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
// the same with the non-temporal hint: for data that is read once (streamed weights, decode KV)
__device__ __forceinline__ uint4 ldg16_stream(const void* p) {
    typedef unsigned u32x4_nt_t __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt_t*>(p)));
}

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }

// Sum over the wavefront: rotations within each row of 16 lanes (DPP, no trip through LDS as a shuffle takes), then the four rows.
__device__ __forceinline__ float wave_sum(float v) {
    const auto ror = [](float x, auto n) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + decltype(n)::value, 0xf, 0xf, true));
    };
    v += ror(v, std::integral_constant<int, 8>{});
    v += ror(v, std::integral_constant<int, 4>{});
    v += ror(v, std::integral_constant<int, 2>{});
    v += ror(v, std::integral_constant<int, 1>{});
    const auto row = [&](int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16 * i)); };
    return (row(0) + row(1)) + (row(2) + row(3));
}


// A word at a wavefront-uniform address that no kernel writes while this one runs, through the scalar cache.
__device__ __forceinline__ int scalar_read(const int32_t* p) {
    return *(const __attribute__((address_space(4))) int32_t*)p;
}

// ---- HBM -> LDS copies without a register hop, and the LDS reads that go with them -------------
// global_load_lds writes lane l's 16 bytes at the (wavefront-uniform) LDS address + 16 l and counts
// in vmcnt.  The compiler cannot tell an ordinary LDS read from the LDS writes of such loads in
// flight and would drain the load queue before each one, so the kernels that use these copies read
// LDS through lds_read16 (inline assembly) and wait with lgkm_tie, which names the registers it
// makes valid so that their consumers cannot move above the wait.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

#define PS_GLOBAL_TO_LDS(gp, lp)                                                                                     \
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gp),                            \
                                     (__attribute__((address_space(3))) void*)(lp), 16, 0, 0)

__device__ __forceinline__ u32x4_t lds_read16(uint32_t addr, int off) {
    u32x4_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(off) : "memory");
    return v;
}
// wait until at most CNT LDS operations are outstanding; the named registers are tied to the wait
template <int CNT>
__device__ __forceinline__ void lgkm_tie(u32x4_t& a) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(CNT));
}
template <int CNT>
__device__ __forceinline__ void lgkm_tie(u32x4_t& a, u32x4_t& b, u32x4_t& c) {
    asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(a), "+v"(b), "+v"(c) : "n"(CNT));
}
template <int CNT>
__device__ __forceinline__ void lgkm_tie(u32x4_t& a, u32x4_t& b, u32x4_t& c, u32x4_t& d, u32x4_t& e) {
    asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e) : "n"(CNT));
}
// the same with a count that is a constant once the caller's loop is unrolled
__device__ __forceinline__ void lgkm_tie_dyn(u32x4_t& a, int cnt) {
    switch (cnt) {
        case 0: lgkm_tie<0>(a); break;
        case 1: lgkm_tie<1>(a); break;
        case 2: lgkm_tie<2>(a); break;
        case 3: lgkm_tie<3>(a); break;
        case 4: lgkm_tie<4>(a); break;
        case 5: lgkm_tie<5>(a); break;
        default: lgkm_tie<6>(a); break;
    }
}
template <int CNT>
__device__ __forceinline__ void vm_wait() {
    // s_waitcnt immediate: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]; others left open
    __builtin_amdgcn_s_waitcnt((CNT & 15) | ((CNT >> 4) << 14) | 0x0F70);
}

}  // namespace ps
