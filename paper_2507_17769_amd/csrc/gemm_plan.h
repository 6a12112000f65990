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
    int cus = 0;       // compute units to plan for: 0 = the current device's (contexts without a device name them)
};

// ------------------------------------------------------------------------- weights in registers (gemm_wreg.hip)
constexpr int WREG_MIN_TM = 5, WREG_MAX_TM = 10;
constexpr int WREG_MAX_M = 6144;   // tokens up to which the choice between the kernels has been measured

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
    int k_shares;       // weight streaming: K shares that a block adds up (1 or 2)
    int splits;         // partial buffers written
    int kb_per_split;   // 32-wide k-blocks per split
    bool cut_tail;      // tiled: cut the K loops of the last, partial wave of tiles over the blocks (one split only)
    int slots_per_xcd;  // tiled: parked pieces an XCD may hold
    double waves;       // tiled: waves of units that the blocks of a compute unit go through, by tiled_estimate
};

// Estimated time (us) of the tiled kernel for one choice of tile edge, K splits and tail cutting, from the rates measured
// on the layer shapes: a block takes about 1.4 us (0.9 us for a 128x128 tile, two of which share a compute unit) per pair
// of k-blocks plus a fixed prologue and epilogue per unit; blocks take units in waves; every split beyond the first is
// written and read back by the consumer; parked pieces of a cut tail cost about 1.4 us per MB all told (store, count,
// reload by the last block and the clock the extra traffic costs the rest of the step: measured on the gate/up and O
// matrices), less where whole tiles follow to hide them behind.
inline double tiled_estimate(int M, int N, int K, int edge, int splits, bool cut, int cus, int* kp_per_split, int* eff_splits, int* slots_per_xcd, double* waves_out) {
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
    *waves_out = waves;
    double us = waves * unit_us;
    if (s_eff > 1) us += 2.0 * (s_eff - 1) * (double)M * N * 4 / 3e6;
    if (cut) us += pieces * (double)edge * edge * 4 / 0.7e6 * (any_full ? 0.6 : 1.0) + 10.0;
    return us;
}

// Time (us) of the consumer's read of `splits` fp32 partial buffers beyond the first: 8 TB/s, half of that for what lies beyond
// the 256 MB of the last-level cache.  Measured behind the QKV and O projections at 97 to 2048 tokens.
inline double partials_us(int splits, int M, int N) {
    const double bytes = (double)M * N * 4;
    return (splits - 1) * bytes / 8e6 + std::max(0.0, splits * bytes - 256e6) / 8e6;
}

// The two times below (us) are of the kernel and of its consumer's read of the partial sums, so that K splits are charged alike.
// Both are fitted to measured times on the projections of the 8B and the 70B shape at 65 to 6144 tokens: 10 680 runs of the
// weights-in-registers kernel over its row tiles, column groups and K splits, and the plans that tiled_estimate picks for the
// tiled one.  In both a quarter of a long run goes by its operations alone, whatever the plan: the power limit.

// Weights in registers: blocks run one per compute unit in waves, the last one as long as any.  A stage costs 0.46 + 0.033
// per row tile with four column groups (0.39 + 0.073 with two, whose K shares copy twice the activations); the weights stream
// at 7.9 TB/s, and of the shorter of the two times about half is hidden; partial sums are written at 2.9 TB/s.  6 % rms from
// the measured kernel times; the plan it picks takes 0.3 % longer than the best one in the mean, 9 % at worst.
inline double wreg_time(const WregPlan& g, int M, int N, int K, int kind, int cus) {
    const int shares = 8 / g.nc, n = K / 32 / (g.splits * shares);
    const int blocks = g.row_tiles * g.splits * ((N / 64 + g.nc - 1) / g.nc), waves = (blocks + cus - 1) / cus;
    double core = 4.0 + waves * (3.0 + n * (g.nc == 4 ? 0.46 + 0.033 * g.tm : 0.39 + 0.073 * g.tm));
    core += 0.24 * std::max(0.0, 2.0 * M * N * K / 0.8e9 - core);
    const double hbm = 2.0 * N * K / 7.9e6, us = std::max(core, hbm) + 0.48 * std::min(core, hbm);
    if (kind == GemmOut::SWIGLU_BF16) return 0.9 * us;   // bf16 of half the columns: a quarter of the output bytes
    return us + (g.splits - 1) * (double)M * N * 4 / 2.9e6 + partials_us(g.splits, M, N);
}

// The tiled kernel with a plan that tiled_estimate has picked (which ranks tiles, splits and cuts against each other, and runs 3
// to 30 % below the measured times).  A pair of k-blocks costs 1.1 us, 1.3 with 256x256 tiles; two blocks of 128x128 tiles share
// a compute unit, and a wave of them takes 0.59 of its time where every unit has one, 0.8 to 1 where some have two.  7 % rms from the
// measured kernel times, 22 % at worst.
inline double tiled_time(const GemmPlan& g, int M, int N, int K, int kind, int cus) {
    const int edge = g.big_tile ? 256 : 128, pairs = g.kb_per_split / 2, per_wave = g.big_tile ? cus : 2 * cus;
    const int units = ((M + edge - 1) / edge) * ((N + edge - 1) / edge) * g.splits, full = units / per_wave;
    const double rem = (double)(units % per_wave) / per_wave;
    double waves = g.waves;
    if (!g.cut_tail) waves = full + (rem == 0 ? 0.0 : g.big_tile ? 1.0 : rem <= 0.5 ? 0.59 : 0.795 + 0.41 * (rem - 0.5));
    double core = waves * (g.big_tile ? 1.3 * pairs + 3.6 : 1.1 * pairs + 5.4);
    core += 0.26 * std::max(0.0, 2.0 * M * N * K / 1.0e9 - core);
    const double hbm = 2.0 * N * K / 6.5e6, us = std::max(core, hbm) + 0.29 * std::min(core, hbm);
    if (kind == GemmOut::SWIGLU_BF16) return 0.92 * us;
    return us + (g.splits - 1) * (double)M * N * 4 / 2.8e6 + partials_us(g.splits, M, N);
}

// The best plan of the weights-in-registers kernel with at most max_splits K splits, and its time, or infinity where the kernel
// does not serve the shape or would leave more than half of the compute units without a block.
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
                if (!wreg_valid(g, M, N, K, kind) || rt * sp * (N / 64 / nc) < cus / 2) continue;
                const double us = wreg_time(g, M, N, K, kind, cus);
                if (us < best_us) { best_us = us; *best = g; }
            }
    }
    return best_us;
}

inline GemmPlan plan_gemm(int M, int N, int K, int kind, const GemmOptions& o, int cus) {
    const int split_opt = o.split_k, tile_opt = o.tile, sk_mode = o.sk_mode;
    GemmPlan g;
    g.wreg = false;
    const bool allow_wreg = o.wreg == 0 && M > 64 && M <= WREG_MAX_M && tile_opt == 0 && sk_mode == 0;   // the options that name the tiled kernel get it
    // measured against the tiled kernel: streaming wins up to 96 tokens for every projection, and up to 160 (ten row tiles) for all but the QKV-shaped
    // one (more columns than rows of weights: 48 blocks per split and six splits of partial sums; 129 tokens: 29 vs 24 us),
    // above all for the gate/up matrix (129 tokens: 61 vs 75 us) and the down projection (42 vs 46)
    g.wstream = M <= 64 || (tile_opt == 0 && (M <= 96 || (M <= 160 && (kind == GemmOut::SWIGLU_BF16 || N <= K))));
    g.big_tile = false;
    g.k_shares = 1;
    g.splits = 1;
    g.kb_per_split = K / 32;
    g.cut_tail = false;
    g.slots_per_xcd = 0;
    g.waves = 0;
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
        const bool wide = N > K && (double)N * K >= 16e6;   // from 65 tokens on a case for the weights in registers, see below
        // A wavefront with a short run of K (up to 24 k-blocks) spends as long on its start and on writing its partial sums as on
        // the weights: two K shares inside a block add up through LDS, and three quarters as many blocks as compute units
        // take the place of two each.  Measured with the kernel behind it (us, one share in 8 splits / two shares in 3): O of the 8B
        // shape 13.5 / 12.5 at 8 tokens, 18.1 / 16.0 at 64, 21.9 / 19.3 at 97, 24.6 / 21.5 at 144; QKV up to 32 tokens 11.4 /
        // 12.6, from there on 16.4 / 16.3 with a third of the partial sums; QKV from 33 tokens on and O of the tiny shape 0.4 to 0.6 less.
        // Longer runs lose: O of the 70B shape 28.0 / 28.9 at 16 tokens, down of the 8B shape 28.4 / 29.9 at 64.  In between it
        // depends on what one share makes of the device: where its splits put exactly two blocks on every unit, 4096 columns, runs of
        // 16 gain 5 to 8 % at 8 to 144 tokens and runs of 17 to 24 lose up to 3.6 % (22: 19.9 / 20.6 at 64 tokens; 28: 22.6 / 24.1);
        // where they leave wavefronts to be had, 1024 to 3072 columns, runs of 20 to 24 gain 0.4 to 11 % from 64 tokens on, 5 % less to
        // 8 % more at 8; where they leave a tail, 5120 columns, 24 gain 13 to 16 % from 64 tokens on.
        const int run = (KB + s - 1) / s, longest = groups * s == 2 * cus ? 16 : 24;
        if (kind != GemmOut::SWIGLU_BF16 && KB % 4 == 0 && run <= longest && (N <= K || (M > 32 && (M <= 64 || !wide)))) {
            g.k_shares = 2;
            if (split_opt == 0) s = std::max(1, std::min(s, (3 * cus / 4 + groups / 2) / groups));
        }
        int kps = (KB + s - 1) / s;
        kps = (kps + 2 * g.k_shares - 1) / (2 * g.k_shares) * (2 * g.k_shares);  // whole stages of two k-blocks for every share
        g.kb_per_split = kps;
        g.splits = (KB + kps - 1) / kps;
        // Measured against streaming (kernel and consumer, us, streaming / weights in registers): gate/up of the 8B shape 45 / 45 at
        // 65 and 80 tokens, 49.6 / 49.1 at 97, 56.5 / 52.9 at 144, 61.5 / 54.0 at 160; of the 70B shape, where streaming puts two
        // blocks on a compute unit, 154 / 140 at 65, 188 / 147 at 128, 212 / 153 at 160.  Matrices wider than deep: QKV of the
        // 8B shape 28.7 / 25.4 at 65, 32.4 / 28.0 at 96, of the 70B shape 51.9 / 47.4 and 58.4 / 50.4; the output projection onto
        // 128256 columns 239 / 204 at 65 and 240 / 210 at 96 (4096 deep), 432 / 356 and 398 / 364 (8192 deep); 4096 columns 2048
        // deep 19 / 21 and 22 / 21, so that small ones stay, as do the O and down projections.
        const bool gate_up = kind == GemmOut::SWIGLU_BF16;
        if (allow_wreg && ((gate_up && (M > 96 || N / 128 > cus)) || (!gate_up && wide)))
            g.wreg = std::isfinite(wreg_best(M, N, K, kind, split_opt, o.cap_splits ? g.splits : 8, cus, &g.wreg_plan));
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
                    double waves;
                    double us = tiled_estimate(M, N, K, edge, sp, cut != 0, cus, &kps, &eff, &slots, &waves);
                    if (cut && slots == 0) continue;
                    if (cut && sk_mode == 2) us -= 1e9;   // test knob: a tail that can be cut is cut
                    if (first || us < best) {
                        first = false; best = us;
                        g.big_tile = edge == 256; g.splits = eff; g.kb_per_split = 2 * kps; g.cut_tail = cut != 0; g.slots_per_xcd = slots; g.waves = waves;
                    }
                }
        }
        // The smaller time decides; the half percent keeps the down projection of the 8B shape at 800 and 832 tokens (113 / 102 us
        // with its consumer in the tiled kernel / in this one).  Checked on stacks deep enough that no weights stay in a cache, on
        // either side of every crossing: no layer is more than 1 % slower than without this kernel.
        WregPlan w;
        if (allow_wreg && wreg_best(M, N, K, kind, split_opt, o.cap_splits ? g.splits : 8, cus, &w) < 1.005 * tiled_time(g, M, N, K, kind, cus)) {
            g.wreg = true;
            g.wreg_plan = w;
            g.splits = w.splits;
            g.cut_tail = false;
            g.slots_per_xcd = 0;
        }
    }
    return g;
}

// Memory of a product with these options, all of one plan: the output of launch_gemm, and what it needs beside it (0 unless the
// tiled kernel serves the product and cuts its tail: only the blocks that share a tile count in on it).
struct GemmSizes {
    size_t out_bytes, frag_bytes;
    int n_counters;
};
inline GemmSizes gemm_plan_sizes(int M, int N, int K, int kind, const GemmOptions& o, int cus) {
    GemmSizes z{0, 0, 0};
    if (M <= 0) return z;
    const GemmPlan g = plan_gemm(M, N, K, kind, o, cus);
    if (kind == GemmOut::SWIGLU_BF16) {
        // dense [rows][N/2] in operand order.  The tiled kernel stores whole row tiles without a row check
        // (rows past M are never read back), so the buffer holds M rounded up to its largest tile.
        const size_t rows = M <= 64 ? (size_t)((M + 15) / 16 * 16) : (size_t)((M + 255) / 256 * 256);
        z.out_bytes = rows * (N / 2) * sizeof(uint16_t);
    } else {
        z.out_bytes = (size_t)g.splits * M * N * sizeof(float);
    }
    if (g.cut_tail) {
        const int b = g.big_tile ? 256 : 128;
        z.frag_bytes = (size_t)8 * g.slots_per_xcd * b * b * sizeof(float);
        z.n_counters = ((M + b - 1) / b) * ((N + b - 1) / b);
    }
    return z;
}

inline size_t gemm_plan_out_bytes(int M, int N, int K, int kind, const GemmOptions& o, int cus) {
    return gemm_plan_sizes(M, N, K, kind, o, cus).out_bytes;
}

inline void gemm_plan_workspace(int M, int N, int K, int kind, const GemmOptions& o, int cus, size_t* frag_bytes, int* n_counters) {
    const GemmSizes z = gemm_plan_sizes(M, N, K, kind, o, cus);
    *frag_bytes = z.frag_bytes;
    *n_counters = z.n_counters;
}

}  // namespace ps
