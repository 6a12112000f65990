// Rotation and KV append of four rotation pairs of one token and head, shared by rope_append and by the GEMM that makes a small
// QKV projection in one piece.
#pragma once
#include "ps_device.h"

namespace ps {

// (cos, sin) of pairs j .. j + 3 of a token
struct RopeAngles { float4 c01, c23; };
__device__ __forceinline__ RopeAngles rope_angles(const RopeOut& o, int position, int j) {
    const float4* cp = reinterpret_cast<const float4*>(o.cs + (size_t)position * (o.d >> 1) + j);
    return RopeAngles{cp[0], cp[1]};
}

// Token t's head hh (query heads, then key, then value heads), pairs j .. j + 3 (j a multiple of 4): every value is rounded to bf16
// once, after the rotation; queries go to q, keys and values to the token's cache slot.
__device__ __forceinline__ void rope_store(const RopeOut& o, int t, int slot, int hh, int j, const float (&lo)[4], const float (&hi)[4], const RopeAngles& a) {
    const int half = o.d >> 1;
    uint2 plo, phi;
    if (hh < o.n_q + o.n_kv) {
        const float co[4] = {a.c01.x, a.c01.z, a.c23.x, a.c23.z}, si[4] = {a.c01.y, a.c01.w, a.c23.y, a.c23.w};
        float rlo[4], rhi[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            rlo[e] = lo[e] * co[e] - hi[e] * si[e];
            rhi[e] = hi[e] * co[e] + lo[e] * si[e];
        }
        plo = uint2{pack_bf16(rlo[0], rlo[1]), pack_bf16(rlo[2], rlo[3])};
        phi = uint2{pack_bf16(rhi[0], rhi[1]), pack_bf16(rhi[2], rhi[3])};
    } else {
        plo = uint2{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3])};
        phi = uint2{pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
    }
    if (hh < o.n_q) {
        bf16_t* qr = o.q + ((size_t)t * o.n_q + hh) * o.d;
        *reinterpret_cast<uint2*>(qr + j) = plo;
        *reinterpret_cast<uint2*>(qr + j + half) = phi;
    } else if (hh < o.n_q + o.n_kv) {
        bf16_t* kc = o.pool + (((size_t)(slot >> 4) * o.n_kv + (hh - o.n_q)) * 2 + 0) * (size_t)(16 * o.d);
        // j is a multiple of 4: the four elements sit in one 8-element group of the key chunk
        *reinterpret_cast<uint2*>(kc + k_elem_offset(slot & 15, j)) = plo;
        *reinterpret_cast<uint2*>(kc + k_elem_offset(slot & 15, j + half)) = phi;
    } else {
        bf16_t* vc = o.pool + (((size_t)(slot >> 4) * o.n_kv + (hh - o.n_q - o.n_kv)) * 2 + 1) * (size_t)(16 * o.d);
        const uint32_t wl[2] = {plo.x, plo.y}, wh[2] = {phi.x, phi.y};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            vc[v_elem_offset(slot & 15, j + e)] = (bf16_t)(wl[e >> 1] >> (16 * (e & 1)));
            vc[v_elem_offset(slot & 15, j + half + e)] = (bf16_t)(wh[e >> 1] >> (16 * (e & 1)));
        }
    }
}

}  // namespace ps
