// Checks of the GEMM planner (gemm_plan.h), compiled for the host by test_host_gemm_plan.py.  Walks the projections of
// several model shapes over token counts and options and checks every plan against what the kernels and their buffers need.
// With arguments (M N K kind wreg cap ...) it prints the plan of each: kernel, row tiles, column groups, K splits, row blocks.
#include <cstdio>
#include <cstdlib>

#include "gemm_plan.h"

using namespace ps;

struct Shape { int N, K, kind; };
constexpr int P = GemmOut::PARTIAL_F32, G = GemmOut::SWIGLU_BF16;
// QKV, O, gate/up, down of the 8B shape, the 70B shape, the tiny one and one whose K loops divide evenly nowhere; some whose
// k-blocks are two more than a multiple of four
const Shape shapes[] = {{6144, 4096, P}, {4096, 4096, P}, {28672, 4096, G}, {4096, 14336, P},
                        {10240, 8192, P}, {8192, 8192, P}, {57344, 8192, G}, {8192, 28672, P},
                        {512, 256, P}, {256, 256, P}, {1408, 256, G}, {256, 704, P},
                        {3456, 1152, P}, {1152, 1152, P}, {6400, 1152, G}, {1152, 3200, P},
                        {1344, 1088, P}, {1088, 1088, P}, {1088, 960, P}, {320, 704, P}};

static int n_checked = 0;
#define REQUIRE(cond)                                                                                                              \
    if (!(cond)) {                                                                                                                 \
        printf("%s: M=%d N=%d K=%d kind=%d split_k=%d cap=%d\n", #cond, M, s.N, s.K, s.kind, o.split_k, (int)o.cap_splits);      \
        exit(1);                                                                                                                   \
    }

static void check(int M, const Shape& s, const GemmOptions& o, int cus) {
    const GemmPlan g = plan_gemm(M, s.N, s.K, s.kind, o, cus);
    REQUIRE(g.splits >= 1 && g.splits <= 8 && (s.kind == P || g.splits == 1));
    REQUIRE(!(g.wreg && g.wstream));
    if (g.wreg) {
        const WregPlan& w = g.wreg_plan;
        REQUIRE(M > 64 && wreg_valid(w, M, s.N, s.K, s.kind) && w.splits == g.splits);
        REQUIRE(16 * w.tm * (w.row_tiles - 1) < M);   // no row block without a row
    } else {
        REQUIRE((g.splits - 1) * g.kb_per_split < s.K / 32 && g.splits * g.kb_per_split >= s.K / 32);
    }
    // Whole stages of two k-blocks for every K share of a block, in the last split too: what is over would be left out.
    if (g.wstream) {
        REQUIRE(g.k_shares == 1 || (g.k_shares == 2 && s.kind == P));
        REQUIRE(s.K / 32 % (2 * g.k_shares) == 0 && g.kb_per_split % (2 * g.k_shares) == 0);
    } else {
        REQUIRE(g.k_shares == 1);
    }
    // what the buffers hold is what the plan writes
    if (s.kind == P) REQUIRE(gemm_plan_out_bytes(M, s.N, s.K, s.kind, o, cus) == (size_t)g.splits * M * s.N * 4);
    const WregPlan forced{o.wreg / 10, o.wreg % 10, g.splits, g.wreg_plan.row_tiles};
    REQUIRE(o.wreg != 1 || !g.wreg);
    if (o.wreg > 1 && M > 64 && (s.K / 32) % (8 / forced.nc * WREG_STAGES * std::max(1, s.kind == G ? 1 : std::min(o.split_k, 8))) == 0)
        REQUIRE(g.wreg && g.wreg_plan.tm == forced.tm && g.wreg_plan.nc == forced.nc);
    if (o.cap_splits && o.wreg == 0) {   // and no more than without the weights-in-registers kernel
        GemmOptions without = o;
        without.wreg = 1;
        size_t frag, frag_w;
        int cnt, cnt_w;
        gemm_plan_workspace(M, s.N, s.K, s.kind, o, cus, &frag, &cnt);
        gemm_plan_workspace(M, s.N, s.K, s.kind, without, cus, &frag_w, &cnt_w);
        REQUIRE(gemm_plan_out_bytes(M, s.N, s.K, s.kind, o, cus) <= gemm_plan_out_bytes(M, s.N, s.K, s.kind, without, cus));
        REQUIRE(frag <= frag_w && cnt <= cnt_w);
    }
    n_checked++;
}

int main(int argc, char** argv) {
    for (int i = 1; i + 5 < argc; i += 6) {
        GemmOptions o;
        o.wreg = atoi(argv[i + 4]);
        o.cap_splits = atoi(argv[i + 5]) != 0;
        const GemmPlan g = plan_gemm(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]), o, 256);
        if (g.wreg) printf("wreg %d %d %d %d\n", g.wreg_plan.tm, g.wreg_plan.nc, g.splits, g.wreg_plan.row_tiles);
        else printf("%s 0 0 %d 0\n", g.wstream ? "wstream" : "tiled", g.splits);
    }
    if (argc > 1) return 0;
    for (int cus : {256, 304, 64})
        for (const Shape& s : shapes)
            for (int M = 1; M < 9000; M += M < 720 ? 1 : 41)
                for (int split : {0, 1, 2, 3, 5, 8, 64})
                    for (bool cap : {false, true}) {
                        GemmOptions o;
                        o.split_k = split;
                        o.cap_splits = cap;
                        check(M, s, o, cus);
                        if (M > 700) continue;
                        for (int wreg : {1, 52, 54, 72, 104}) {
                            o.wreg = wreg;
                            check(M, s, o, cus);
                        }
                    }
    printf("OK %d\n", n_checked);
    return 0;
}
