// Which GEMM kernel serves a projection, with which tiles and K splits, and what that needs in memory: pure functions of the
// shape, the options and the number of compute units, without HIP, so that they can be checked on their own.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <limits>

#include "sk_decomp.h"

namespace ps {

struct GemmOut {
    enum Kind : int { PARTIAL_F32 = 0, SWIGLU_BF16 = 1 };
};

// What a caller may fix about a plan; all zero: automatic.
struct GemmOptions {
    int split_k = 0;   // K splits (partial buffers)
    int tile = 0;      // M > 64: 0 = choose, 128 or 256 = block tile edge of the tiled kernel, which then serves the product
    int sk_mode = 0;   // tiled kernel: 0 = the cost model decides whether the tail's K loops are cut, 1 = never (whole tiles only), 2 = wherever possible
    // weights-in-registers kernel: 0 = the cost model decides, 1 = never, 10 tm + nc = with this block (and split_k K splits, or
    // one) for more than 64 tokens, wherever K is a whole number of rounds of its shares
    int wreg = 0;
    // The weights-in-registers kernel takes no more K splits than the kernel that it replaces would: the partial sums then need
    // no more memory than without it.  Set for every step that a static step's scratch can hold, whichever call runs it.
    bool cap_splits = false;
};

// ------------------------------------------------------------------------- weights in registers (gemm_wreg.hip)
constexpr int WREG_MIN_TM = 5, WREG_MAX_TM = 10;

constexpr int WREG_STAGES = 4;   // register sets of weights; a K share is a whole number of rounds through them
// slots of the activation ring: one more than weight sets where LDS holds it (8 / nc K shares of tm KiB per slot)
constexpr int wreg_ring(int tm, int nc) { return 8 / nc * tm * (WREG_STAGES + 1) <= 160 ? WREG_STAGES + 1 : WREG_STAGES; }

struct WregPlan {
    int tm;         // 16-row tiles per block
    int nc;         // 64-column groups per block: 2 or 4 (8 / nc shares of K inside the block)
    int splits;     // K splits over blocks, each with its own fp32 output (1 for the gate/up matrix)
    int row_tiles;  // blocks over the rows: 16 tm row_tiles >= M
};

// true: the kernel computes this product with this plan
inline bool wreg_valid(const WregPlan& g, int M, int N, int K, int kind) {
    if (g.tm < WREG_MIN_TM || g.tm > WREG_MAX_TM || (g.nc != 2 && g.nc != 4) || g.splits < 1 || g.row_tiles < 1) return false;
    if (M <= 0 || N % 64 || K % 32 || (kind == GemmOut::SWIGLU_BF16 && g.splits != 1)) return false;
    if ((long long)16 * g.tm * g.row_tiles < M) return false;
    // 32-bit buffer offsets, the upper half of which marks a request as one past the end
    if ((long long)N * K * 2 >= (1ll << 31) || (long long)(M + 15) / 16 * 16 * K * 2 >= (1ll << 31)) return false;
    const int shares = g.splits * (8 / g.nc);
    return (K / 32) % (shares * WREG_STAGES) == 0;
}

// ----------------------------------------------------------------------------------------------- the three kernels
struct GemmPlan {
    bool wstream;
    bool wreg;          // weights in registers (gemm_wreg.hip), with the plan below
    WregPlan wreg_plan;
    bool big_tile;      // tiled: 256x256 blocks (else 128x128)
    int splits;         // partial buffers written
    int kb_per_split;   // 32-wide k-blocks per split
    bool cut_tail;      // tiled: cut the K loops of the last, partial wave of tiles over the blocks (one split only)
    int slots_per_xcd;  // tiled: parked pieces an XCD may hold
};

// Estimated time (us) of the tiled kernel for one choice of tile edge, K splits and tail cutting, from the rates measured
// on the layer shapes: a block takes about 1.4 us (0.9 us for a 128x128 tile, two of which share a compute unit) per pair
// of k-blocks plus a fixed prologue and epilogue per unit; blocks take units in waves; every split beyond the first is
// written and read back by the consumer; parked pieces of a cut tail cost about 1.4 us per MB all told (store, count,
// reload by the last block and the clock the extra traffic costs the rest of the step: measured on the gate/up and O
// matrices), less where whole tiles follow to hide them behind.
inline double tiled_estimate(int M, int N, int K, int edge, int splits, bool cut, int cus, int* kp_per_split, int* eff_splits, int* slots_per_xcd) {
    const int B = cus * (edge == 256 ? 1 : 2) / 8;
    const int KPt = K / 64;
    const int kps = (KPt + splits - 1) / splits, s_eff = (KPt + kps - 1) / kps;
    const int tiles = ((M + edge - 1) / edge) * ((N + edge - 1) / edge), units = tiles * s_eff;
    const int upx = (units + 7) / 8;
    const double t_pair = edge == 256 ? 1.4 : 0.9, t_fix = edge == 256 ? 8.0 : 4.0;
    const double unit_us = kps * t_pair + t_fix;
    double waves = 0, waves_uncut = 0;
    int slots = 0, pieces = 0;
    bool any_full = false;
    for (int x = 0; x < 8; x++) {
        const int T = std::min(units, (x + 1) * upx) - x * upx;
        if (T <= 0) break;
        const int full = T / B, R = T % B;
        any_full |= full > 0;
        waves_uncut = std::max(waves_uncut, (double)full + (R > 0));
        if (!cut || R == 0) { waves = std::max(waves, (double)full + (R > 0)); continue; }
        const int Bt = sk_tail_blocks(B, R, kps);
        waves = std::max(waves, full + (double)R / Bt);
        slots = std::max(slots, sk_slots(Bt, R));
        pieces += Bt > R ? sk_slots(Bt, R) : 0;
    }
    *kp_per_split = kps;
    *eff_splits = s_eff;
    *slots_per_xcd = slots;
    // With 256x256 tiles on every compute unit the device runs at its power limit, and compute units left idle by an
    // uncut tail give part of their share back as clock for the busy ones: measured on the 70B-shaped gate/up matrix,
    // cutting the tail of 4.4 waves bought nothing, where the arithmetic says 11 %.  Half the gain is what is counted.
    if (cut && edge == 256) waves = waves_uncut - 0.5 * (waves_uncut - waves);
    double us = waves * unit_us;
    if (s_eff > 1) us += 2.0 * (s_eff - 1) * (double)M * N * 4 / 3e6;
    if (cut) us += pieces * (double)edge * edge * 4 / 0.7e6 * (any_full ? 0.6 : 1.0) + 10.0;
    return us;
}

// Estimated time (us) of the weights-in-registers kernel for one plan: blocks run one per compute unit in waves, a stage
// costs 0.34 + 0.07 per row tile with four column groups (0.22 + 0.096 with two, whose K shares copy twice the activations),
// a block 8 more for its first loads and its epilogue, a wave that is not full three quarters of its time plus a quarter of
// its fill (the blocks that do run have the memory to themselves); the weights stream at 6.2 TB/s, and the shorter of the
// two times hides all but 15 % of itself.  Fitted to 190 runs of the 8B shapes at 80 to 1024 tokens; the plan it picks is within
// 8 % of the best one measured at every one of them.  Partial sums are read back by the consumer.
inline double wreg_estimate(const WregPlan& g, int M, int N, int K, int cus) {
    const int shares = 8 / g.nc, n = K / 32 / (g.splits * shares);
    const int blocks = g.row_tiles * g.splits * ((N / 64 + g.nc - 1) / g.nc);
    const int full = blocks / cus, rem = blocks % cus;
    const double waves = full + (rem ? 0.77 + 0.23 * rem / cus : 0.0);
    const double core = 2.0 + waves * (8.0 + n * (g.nc == 4 ? 0.34 + 0.07 * g.tm : 0.22 + 0.096 * g.tm));
    const double hbm = 2.0 * N * K / 6.2e6;
    return std::max(core, hbm) + 0.15 * std::min(core, hbm) + (g.splits - 1) * (double)M * N * 4 / 5e6;
}

// The best plan of the weights-in-registers kernel, or an estimate of infinity where it does not serve the shape.
// At most max_splits K splits.
inline double wreg_best(int M, int N, int K, int kind, int split_opt, int max_splits, int cus, WregPlan* best) {
    double best_us = std::numeric_limits<double>::infinity();
    const int tiles = (M + 15) / 16;
    const int s_lo = kind == GemmOut::SWIGLU_BF16 ? 1 : (split_opt > 0 ? std::min(split_opt, 8) : 1);
    const int s_hi = std::min(max_splits, kind == GemmOut::SWIGLU_BF16 ? 1 : (split_opt > 0 ? s_lo : 8));
    for (int rt = (tiles + WREG_MAX_TM - 1) / WREG_MAX_TM; rt <= (tiles + WREG_MIN_TM - 1) / WREG_MIN_TM; rt++) {
        const int tm = std::max(WREG_MIN_TM, (tiles + rt - 1) / rt);
        if (rt > 1 && tm * (rt - 1) >= tiles) continue;   // the last row block would be empty
        for (int nc : {4, 2})
            for (int sp = s_lo; sp <= s_hi; sp++) {
                const WregPlan g{tm, nc, sp, rt};
                if (!wreg_valid(g, M, N, K, kind)) continue;
                const double us = wreg_estimate(g, M, N, K, cus);
                if (us < best_us) { best_us = us; *best = g; }
            }
    }
    return best_us;
}

inline GemmPlan plan_gemm(int M, int N, int K, int kind, const GemmOptions& o, int cus) {
    const int split_opt = o.split_k, tile_opt = o.tile, sk_mode = o.sk_mode;
    GemmPlan g;
    g.wreg = false;
    const bool allow_wreg = o.wreg == 0 && M > 64 && tile_opt == 0 && sk_mode == 0;   // the options that name the tiled kernel get it
    // measured: streaming wins up to 96 tokens for every projection, and up to 160 (ten row tiles) for all but the QKV-shaped
    // one (more columns than rows of weights: 48 blocks per split and six splits of partial sums; 129 tokens: 29 vs 24 us),
    // above all for the gate/up matrix (129 tokens: 61 vs 75 us) and the down projection (42 vs 46)
    g.wstream = M <= 64 || (tile_opt == 0 && (M <= 96 || (M <= 160 && (kind == GemmOut::SWIGLU_BF16 || N <= K))));
    g.big_tile = false;
    g.splits = 1;
    g.kb_per_split = K / 32;
    g.cut_tail = false;
    g.slots_per_xcd = 0;
    if (o.wreg > 1 && M > 64) {
        const int tm = o.wreg / 10, splits = kind == GemmOut::SWIGLU_BF16 ? 1 : std::min(std::max(split_opt, 1), 8);
        const WregPlan w{tm, o.wreg % 10, splits, ((M + 15) / 16 + tm - 1) / tm};
        if (wreg_valid(w, M, N, K, kind)) {
            g.wreg = true;
            g.wreg_plan = w;
            g.wstream = false;
            g.splits = splits;
            return g;
        }
    }
    if (g.wstream) {
        const int groups = N / 64, KB = K / 32;
        int s = 1;
        if (kind != GemmOut::SWIGLU_BF16) {
            s = split_opt > 0 ? split_opt : (512 + groups - 1) / groups;  // aim at two blocks per CU
            s = std::min(s, 8);
            s = std::min(s, std::max(1, KB / 8));  // keep at least two k-blocks per wavefront slice
            s = std::max(s, 1);
        }
        int kps = (KB + s - 1) / s;
        kps += kps & 1;  // whole stages of two k-blocks
        g.kb_per_split = kps;
        g.splits = (KB + kps - 1) / kps;
        // Measured against streaming up to 160 tokens (us, streaming / weights in registers): gate/up of the 8B shape 41.9 /
        // 42.6 at 80 tokens, 46.9 / 45.9 at 97, 53.4 / 49.1 at 144, 58.9 / 49.8 at 160; of the 70B shape, where streaming
        // puts two blocks on a compute unit, 157 / 136 at 80 and 217 / 155 at 128; QKV 17.7 / 15.0 at 80; the O and down
        // projections are no faster (11.5 / 12.4, 24.4 / 25.2 at 80, 14.4 / 14.4, 29.6 / 30.9 at 144).
        const bool gate_up = kind == GemmOut::SWIGLU_BF16;
        if (allow_wreg && ((gate_up && (M > 96 || N / 128 > cus)) || (!gate_up && N > K))) {
            const double us = wreg_best(M, N, K, kind, split_opt, o.cap_splits ? g.splits : 8, cus, &g.wreg_plan);
            g.wreg = std::isfinite(us) && g.wreg_plan.row_tiles * g.wreg_plan.splits * (N / 64 / g.wreg_plan.nc) >= cus / 2;
        }
        if (g.wreg) {
            g.wstream = false;
            g.splits = g.wreg_plan.splits;
        }
    } else {
        // every combination of tile edge, K splits (none for the gate/up matrix, whose epilogue is not linear) and, for
        // one split, tail cutting; the smallest estimate wins
        const int s_lo = kind == GemmOut::SWIGLU_BF16 ? 1 : (split_opt > 0 ? std::min(split_opt, 8) : 1);
        const int s_hi = kind == GemmOut::SWIGLU_BF16 ? 1 : (split_opt > 0 ? s_lo : 8);
        double best = 0;
        bool first = true;
        for (int edge : {128, 256}) {
            if ((tile_opt == 128 || tile_opt == 256) && edge != tile_opt) continue;
            for (int sp = s_lo; sp <= s_hi; sp++)
                for (int cut = 0; cut < (sp == 1 && sk_mode != 1 ? 2 : 1); cut++) {
                    int kps, eff, slots;
                    double us = tiled_estimate(M, N, K, edge, sp, cut != 0, cus, &kps, &eff, &slots);
                    if (cut && slots == 0) continue;
                    if (cut && sk_mode == 2) us -= 1e9;   // test knob: a tail that can be cut is cut
                    if (first || us < best) {
                        first = false; best = us;
                        g.big_tile = edge == 256; g.splits = eff; g.kb_per_split = 2 * kps; g.cut_tail = cut != 0; g.slots_per_xcd = slots;
                    }
                }
        }
        // The tiled estimate runs below what is measured: by a sixth with 128x128 tiles (5 to 30 % over 40 shapes), by an eighth
        // with 256x256 ones.  Where the weights-in-registers kernel wins
        // (8B shape, us, tiled / it): gate/up 80.2 / 67.0 at 256 tokens, 115 / 69.2 at 271, 187 / 158 at 640, 434 / 379 at
        // 1600; down 45.3 / 38.1, 52.3 / 39.3, 94.1 / 66.4; 70B shape at 264 tokens: gate/up 443 / 307, down 212 / 146.
        // The tiled kernel keeps what fills its 256x256 tiles: gate/up at 512 tokens 112 / 121, at 2048 444 / 460.
        WregPlan w;
        if (allow_wreg && wreg_best(M, N, K, kind, split_opt, o.cap_splits ? g.splits : 8, cus, &w) < (g.big_tile ? 1.12 : 1.17) * best) {
            g.wreg = true;
            g.wreg_plan = w;
            g.splits = w.splits;
            g.cut_tail = false;
            g.slots_per_xcd = 0;
        }
    }
    return g;
}

// Bytes of the output of launch_gemm for these options.
inline size_t gemm_plan_out_bytes(int M, int N, int K, int kind, const GemmOptions& o, int cus) {
    if (kind == GemmOut::SWIGLU_BF16) {
        // dense [rows][N/2] in operand order.  The tiled kernel stores whole row tiles without a row check
        // (rows past M are never read back), so the buffer holds M rounded up to its largest tile.
        const size_t rows = M <= 64 ? (size_t)((M + 15) / 16 * 16) : (size_t)((M + 255) / 256 * 256);
        return rows * (N / 2) * sizeof(uint16_t);
    }
    return (size_t)plan_gemm(M, N, K, kind, o, cus).splits * M * N * sizeof(float);
}

// What launch_gemm needs beside its output (both 0 unless the tiled kernel serves the product).
inline void gemm_plan_workspace(int M, int N, int K, int kind, const GemmOptions& o, int cus, size_t* frag_bytes, int* n_counters) {
    *frag_bytes = 0;
    *n_counters = 0;
    if (M <= 0) return;
    const GemmPlan g = plan_gemm(M, N, K, kind, o, cus);
    if (g.wstream || g.wreg) return;
    const int b = g.big_tile ? 256 : 128;
    *frag_bytes = (size_t)8 * g.slots_per_xcd * b * b * sizeof(float);
    *n_counters = ((M + b - 1) / b) * ((N + b - 1) / b);
}

}  // namespace ps
