// Checks of the attention plan, compiled for the host by test_host_attn_plan.py:
// every page pair of every (decode or query block, KV head) is given out once, in order, the blocks of either kind fit the
// places of an XCD, and no team has more than its part of what eight teams would share, however the batch is mixed.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <tuple>

#include "planner.h"

using namespace ps;

#define REQUIRE(cond)                                                                                            \
    if (!(cond)) {                                                                                               \
        printf("%s: case %d (group %d, one block %d): %d teams, %d workers\n", #cond, n, cfg.group, (int)cfg.one_block_per_cu, plan.n_team_workers, workers); \
        return 1;                                                                                                \
    }

int main() {
    std::mt19937 rng(7);
    auto log_uniform = [&](double lo, double hi) { return (int)(lo * std::pow(hi / lo, std::uniform_real_distribution<>(0, 1)(rng))); };
    int n = 0, crowded = 0;
    for (; n < 4000; n++) {
        PlanConfig cfg;
        cfg.n_kv_heads = n % 5 == 0 ? 2 : 8;
        cfg.group = n % 3 == 0 ? 8 : 4;
        cfg.prefill_tokens = 12 * (16 / cfg.group);
        cfg.compute_units = 256;
        cfg.one_block_per_cu = n % 7 == 0;
        const int chunks = n % 4 == 0 ? 0 : log_uniform(1, 4), decodes = n % 4 == 1 ? 0 : log_uniform(1, 300);
        std::vector<ps_seq> seqs;
        std::vector<std::vector<int32_t>> tables;
        for (int i = 0; i < chunks + decodes; i++) {
            const int q = i < chunks ? log_uniform(1, 1700) : 1, kv = q + log_uniform(1, 9000) - 1;
            tables.emplace_back((kv + 15) / 16, 0);
            seqs.push_back(ps_seq{i, q, kv, nullptr, (int32_t)tables.back().size()});
        }
        for (size_t i = 0; i < seqs.size(); i++) seqs[i].page_table = tables[i].data();
        StepPlan plan;
        build_indices(seqs.data(), (int)seqs.size(), plan);
        build_attention_plan(cfg, plan);
        const int workers = (int)plan.worker_begin.size() - 1;
        if (seqs.empty()) continue;
        REQUIRE(workers >= 1 && plan.worker_begin[0] == 0 && plan.worker_begin[workers] == (int)plan.items.size());
        for (int w = 0; w < workers; w++) REQUIRE(plan.worker_begin[w] <= plan.worker_begin[w + 1]);
        // places of an XCD: 32 compute units of two blocks each
        const int per_xcd = (plan.n_team_workers + 7) / 8 + ((workers - plan.n_team_workers + 3) / 4 + 7) / 8;
        REQUIRE(per_xcd <= 64);
        REQUIRE(!cfg.one_block_per_cu || per_xcd <= 32);
        crowded += per_xcd > 32;
        // a small chunk is spread over eight teams, or as many as there are four pairs for
        int pairs_team = 0, longest = 0;
        for (int w = 0; w < plan.n_team_workers; w++) {
            int run = 0;
            for (int i = plan.worker_begin[w]; i < plan.worker_begin[w + 1]; i++) run += (plan.items[i].page_end - plan.items[i].page_begin + 1) / 2;
            pairs_team += run;
            longest = std::max(longest, run);
        }
        const int spread = std::max(1, std::min(8, pairs_team / 4));
        REQUIRE(longest <= (pairs_team + spread - 1) / spread + 1);
        std::map<std::tuple<int, int, int>, int> next;   // (sequence, head, query block) -> page its items have reached
        for (const AttnItem& it : plan.items) {
            int& at = next[std::make_tuple(it.seq, it.kv_head, it.q_tok0)];
            REQUIRE(it.page_begin == at && it.page_end > at);
            at = it.page_end;
        }
        size_t want = 0;
        for (const SeqInfo& s : plan.seqs) {
            const int qb = s.n_new <= 16 / cfg.group ? 16 / cfg.group : cfg.prefill_tokens;
            for (int q0 = 0; q0 < s.n_new; q0 += qb, want += cfg.n_kv_heads)
                for (int h = 0; h < cfg.n_kv_heads; h++)
                    REQUIRE(next[std::make_tuple((int)(&s - plan.seqs.data()), h, q0)] == (s.kv_len - s.n_new + q0 + std::min(qb, s.n_new - q0) + 15) / 16);
        }
        REQUIRE(next.size() == want);
    }
    if (crowded < 100 || crowded > n - 1000) return printf("one and two blocks per unit are not both covered: %d\n", crowded), 1;
    printf("OK %d\n", n);
    return 0;
}
