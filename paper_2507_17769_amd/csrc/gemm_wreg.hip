// Weight GEMM for the token counts between pure weight streaming and large matrix products (gemm.hip describes the
// operands and the two other kernels).
//
// What bounds those two here is LDS.  Streaming gives a wavefront 16 columns, so every activation operand read from LDS
// feeds one matrix instruction (8 clocks of LDS for 4 clocks of a compute unit's matrix pipes); the 128x128 tiles pass both
// operands through LDS.  Here a wavefront owns 64 columns and all row tiles of the block: its weights go straight from
// memory into registers, an activation operand read from LDS feeds four matrix instructions, and nothing but activations
// passes through LDS.
//
// A block is eight wavefronts = NC groups of 64 columns x NK = 8 / NC shares of the block's K range, two wavefronts on
// every SIMD, one block per compute unit.  The NC wavefronts of a K share copy its activation k-blocks into their own part
// of an LDS ring; the NK sums are added up through LDS at the end, always in the same order, so that a small output does
// not need one buffer of fp32 partials per K share.
//
// What is left (8B gate/up, 256 tokens, 67 us): the matrix instructions and LDS reads alone take 45 us, which is the rate the
// matrix pipes hold under the power limit on the 224 compute units that have a block; all loads served by the caches 50 us;
// the weights from memory make up the rest.  Measured (8B shape, us, other kernel / this one): gate/up 80 / 67 at 256 tokens,
// 115 / 69 at 271, 187 / 157 at 640; down 45 / 38, 52 / 39, 94 / 66 (1.13 PFLOP/s); QKV 24 / 22 at 97 tokens, 46 / 43 at 640.
#include "ps_device.h"
#include "gemm_wreg.h"

#include <algorithm>
#include <mutex>
#include <type_traits>

namespace ps {

struct WregParams {
    const bf16_t* A;
    const bf16_t* Wp;
    int M, N, K;
    void* out;             // fp32 [split][M][N] row-major, or bf16 [M][N/2] in operand order
    int row_tiles;         // blocks of 16 TM rows
    int splits;
    int stages;            // 32-wide k-blocks per K share: K / 32 = splits * NK * stages
    int units, units_per_xcd;
};

// Raw buffer over `bytes` bytes from p: an access past its end loads nothing (and returns zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}
template <bool STREAM>   // STREAM: the non-temporal hint, for data that one block reads once
__device__ __forceinline__ u32x4_t buffer_read16(__amdgpu_buffer_rsrc_t b, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, STREAM ? 2 : 0);
}
__device__ __forceinline__ void buffer_to_lds16(__amdgpu_buffer_rsrc_t b, uint8_t* dst, uint32_t off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)dst, 16, off, 0, 0, 0);
}

// acc += A . B in place (see mfma16_acc in gemm.hip for why this is assembly)
__device__ __forceinline__ void wreg_mfma(f32x4_t& c, const u32x4_t& a, const u32x4_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <int TM, int NC, int KIND, bool STREAM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_wreg_kernel(WregParams p) {
    constexpr int NK = 8 / NC;
    constexpr int NS = WREG_STAGES, D = NS - 1;    // register sets of weights; stages (one k-block per K share) they are requested ahead
    constexpr int RING = wreg_ring(TM, NC);        // slots of the activation ring: copies are requested RING - 1 stages ahead
    constexpr int DX = RING - 1;
    constexpr int SHARE = TM * 1024;               // bytes of a K share's activations in a stage
    constexpr int SLOT = NK * SHARE;
    constexpr int CPW = (TM + NC - 1) / NC;        // activation copies per wavefront and stage
    constexpr int XW = TM == 10 ? 2 : TM == 8 ? 4 : TM % 3 == 0 ? 3 : TM;   // activation operands in registers or on their way there
    constexpr int LOADS = 4 + CPW;
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / NC, wc = wave % NC;
    const int r = lane & 15, g = lane >> 4;
    // units in the order (column block, split, row tile), the row tile fastest, dealt contiguously to the XCDs: the blocks
    // that read the same weights run side by side on one L2
    const int unit = (blockIdx.x & 7) * p.units_per_xcd + (blockIdx.x >> 3);
    if (unit >= p.units) return;
    const int rt = unit % p.row_tiles, rest = unit / p.row_tiles;
    const int split = rest % p.splits, cb = rest / p.splits;
    const int KB = p.K >> 5, n = p.stages;
    const int kb0 = (split * NK + kg) * n;
    const int m_tiles = (p.M + 15) >> 4;
    const int n_groups = p.N >> 6;
    const int ng_own = cb * NC + wc;
    const bool have_group = ng_own < n_groups;     // a group past the last one streams the last one again and stores nothing
    const int ng = have_group ? ng_own : n_groups - 1;

    // Buffer addressing: requests past the K share's last stage get an offset out of the buffer's range, which fetches
    // nothing, so that every stage issues the same loads and the wait counts are constants.
    const __amdgpu_buffer_rsrc_t w_buf = raw_buffer(p.Wp, (uint32_t)p.N * (uint32_t)p.K * 2u);
    const __amdgpu_buffer_rsrc_t x_buf = raw_buffer(p.A, (uint32_t)m_tiles * (uint32_t)KB * 1024u);
    const uint32_t w_off = ((uint32_t)ng * KB + kb0) * 4096u + lane * 16;
    uint32_t x_off[CPW];
#pragma unroll
    for (int i = 0; i < CPW; i++)   // surplus copies repeat the last block: the same bytes to the same place
        x_off[i] = ((uint32_t)min(rt * TM + min(wc + NC * i, TM - 1), m_tiles - 1) * KB + kb0) * 1024u + lane * 16;
    const uint32_t x_lane = (uint32_t)(uintptr_t)lds + kg * SHARE + lane * 16;

    f32x4_t acc[TM][4];
#pragma unroll
    for (int mt = 0; mt < TM; mt++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[mt][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t w[NS][4];

    // stage s's activation copies into slot byte offset `slot`, and its weights
    auto copy_x = [&](int s, int slot, int i) {
        buffer_to_lds16(x_buf, lds + slot + kg * SHARE + min(wc + NC * i, TM - 1) * 1024, x_off[i] + (uint32_t)s * 1024u + (s < n ? 0u : 0x80000000u));
    };
    auto load_w = [&](u32x4_t (&ws)[4], int s, int i) { ws[i] = buffer_read16<STREAM>(w_buf, w_off + (uint32_t)s * 4096u + (s < n ? 0u : 0x80000000u) + i * 1024); };
    u32x4_t x[XW];
    int slot = 0, last = DX * SLOT;   // byte offsets of this stage's slot and of the one before it, which is refilled
    // Stage s.  One barrier: everybody's copies of stage s + 1 have landed, and everybody has read stage s - 1, whose slot and
    // registers the new requests take.  Vector loads return in order, so the wait for the copies of stage s + 1 must not
    // cover younger weights: with a ring of one slot more than there are weight sets those copies were requested before the
    // weights of stage s.  Each activation operand is read XW operands ahead of its matrix instructions, across the barrier
    // into the next stage, so that a stage begins with its first operands in registers.
    auto stage = [&](auto set_c, int s) {
        constexpr int I = decltype(set_c)::value;
        vm_wait<(DX - 2) * LOADS + 4>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int next = slot + SLOT == RING * SLOT ? 0 : slot + SLOT;
#pragma unroll
        for (int mt = 0; mt < TM; mt++) {
            lgkm_tie_dyn(x[mt % XW], XW - 1);
#pragma unroll
            for (int j = 0; j < 4; j++) wreg_mfma(acc[mt][j], w[I][j], x[mt % XW]);
            __builtin_amdgcn_sched_barrier(0);
            x[mt % XW] = mt + XW < TM ? lds_read16(x_lane + slot, (mt + XW) * 1024) : lds_read16(x_lane + next, (mt + XW - TM) * 1024);
#pragma unroll
            for (int i = 0; i < LOADS; i++)
                if (i * TM / LOADS == mt) {
                    if (i < CPW) copy_x(s + DX, last, i);
                    else load_w(w[(I + D) % NS], s + D, i - CPW);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        last = slot;
        slot = next;
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = -DX; s < 0; s++) {   // the requests of the stages before the first
#pragma unroll
        for (int i = 0; i < CPW; i++) copy_x(s + DX, (s + DX) * SLOT, i);
        __builtin_amdgcn_sched_barrier(0);
        if (s + D >= 0) {
#pragma unroll
            for (int i = 0; i < 4; i++) load_w(w[s + D < 0 ? 0 : s + D], s + D, i);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    vm_wait<(DX - 1) * LOADS + (DX > D ? 0 : 4)>();   // the copies of stage 0
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < XW; i++) x[i] = lds_read16(x_lane, i * 1024);
    for (int s = 0; s < n; s += NS) {   // n is a multiple of NS
        stage(c0, s);
        stage(c1, s + 1);
        stage(c2, s + 2);
        stage(c3, s + 3);
    }
    vm_wait<0>();   // the surplus requests and reads: nothing is on its way into the ring or out of it any more
#pragma unroll
    for (int i = 0; i < XW; i++) lgkm_tie<0>(x[i]);
    // the last matrix instructions have written their accumulators before anything reads them
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // Add up the K shares: share kg keeps the row tiles mt with mt % NK == kg and hands the others over through LDS, half of
    // the columns (column tiles h and h + 2, for the gate/up matrix a gate tile and its up tile) at a time.
    // lane holds C[m = 16 mt + r][n = 64 ng + 16 j + 4 g + 0..3]
    f32x4_t* const xch = reinterpret_cast<f32x4_t*>(lds);
#pragma unroll
    for (int h = 0; h < 2; h++) {
        __syncthreads();   // the ring (h = 0) or the first half's sums (h = 1) have been read by everyone
#pragma unroll
        for (int mt = 0; mt < TM; mt++) {
            const int owner = mt % NK;
            if (owner == kg) continue;
            const int rank = (kg - owner - 1 + NK) % NK;   // 0 .. NK - 2 among the shares that hand this row tile over
#pragma unroll
            for (int q = 0; q < 2; q++) xch[((((wc * TM + mt) * 2 + q) * (NK - 1)) + rank) * 64 + lane] = acc[mt][h + 2 * q];
        }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < TM; mt++) {
            if (mt % NK != kg) continue;
            f32x4_t sum[2];
#pragma unroll
            for (int q = 0; q < 2; q++) {
                sum[q] = acc[mt][h + 2 * q];
#pragma unroll
                for (int o = 0; o < NK - 1; o++) sum[q] += xch[((((wc * TM + mt) * 2 + q) * (NK - 1)) + o) * 64 + lane];
            }
            const int m = (rt * TM + mt) * 16 + r;
            if (m >= p.M || !have_group) continue;
            if constexpr (KIND == GemmOut::SWIGLU_BF16) {
                uint2 o;
                o.x = pack_bf16(silu_f(sum[0][0]) * sum[1][0], silu_f(sum[0][1]) * sum[1][1]);
                o.y = pack_bf16(silu_f(sum[0][2]) * sum[1][2], silu_f(sum[0][3]) * sum[1][3]);
                *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.out) + act_offset(m, ng * 32 + h * 16 + 4 * g, p.N >> 1)) = o;
            } else {
                float* out = static_cast<float*>(p.out) + ((size_t)split * p.M + m) * p.N + ng * 64 + 16 * h + 4 * g;
                *reinterpret_cast<f32x4_t*>(out) = sum[0];
                *reinterpret_cast<f32x4_t*>(out + 32) = sum[1];
            }
        }
    }
}

template <int TM, int NC, int KIND, bool STREAM>
static hipError_t launch_one(const WregParams& p, hipStream_t st) {
    constexpr int NK = 8 / NC;
    constexpr int ring = NK * TM * 1024 * wreg_ring(TM, NC), xch = NC * TM * 2 * (NK - 1) * 1024;
    constexpr int lds_bytes = ring > xch ? ring : xch;
    static_assert(lds_bytes <= 160 * 1024, "LDS of a compute unit");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {   // more dynamic LDS than the default limit: raise it once per kernel
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_wreg_kernel<TM, NC, KIND, STREAM>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL((gemm_wreg_kernel<TM, NC, KIND, STREAM>), dim3(8 * p.units_per_xcd), dim3(512), lds_bytes, st, p);
    return hipGetLastError();
}

template <int TM, int NC, int KIND>
static hipError_t launch_kind(const WregParams& p, hipStream_t st) {
    return p.row_tiles == 1 ? launch_one<TM, NC, KIND, true>(p, st) : launch_one<TM, NC, KIND, false>(p, st);
}
template <int TM>
static hipError_t launch_tm(const WregParams& p, int nc, int kind, hipStream_t st) {
    if (kind == GemmOut::SWIGLU_BF16) return nc == 4 ? launch_kind<TM, 4, GemmOut::SWIGLU_BF16>(p, st) : launch_kind<TM, 2, GemmOut::SWIGLU_BF16>(p, st);
    return nc == 4 ? launch_kind<TM, 4, GemmOut::PARTIAL_F32>(p, st) : launch_kind<TM, 2, GemmOut::PARTIAL_F32>(p, st);
}

hipError_t launch_gemm_wreg(const GemmArgs& a, const WregPlan& g, hipStream_t st) {
    if (!wreg_valid(g, a.M, a.N, a.K, a.kind)) return hipErrorInvalidValue;
    WregParams p;
    p.A = a.A; p.Wp = a.Wp; p.M = a.M; p.N = a.N; p.K = a.K; p.out = a.out;
    p.row_tiles = g.row_tiles;
    p.splits = g.splits;
    p.stages = a.K / 32 / (g.splits * (8 / g.nc));
    p.units = g.row_tiles * g.splits * ((a.N / 64 + g.nc - 1) / g.nc);
    p.units_per_xcd = (p.units + 7) / 8;
    switch (g.tm) {
        case 5: return launch_tm<5>(p, g.nc, a.kind, st);
        case 6: return launch_tm<6>(p, g.nc, a.kind, st);
        case 7: return launch_tm<7>(p, g.nc, a.kind, st);
        case 8: return launch_tm<8>(p, g.nc, a.kind, st);
        case 9: return launch_tm<9>(p, g.nc, a.kind, st);
        case 10: return launch_tm<10>(p, g.nc, a.kind, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace ps
