// Checks of the attention plan, compiled for the host by test_host_attn_plan.py:
// every page pair of every (decode or query block, KV head) is given out once, in order, the pieces of a stream that was cut and
// their merge groups agree on slots of their own, the blocks of either kind fit the places of an XCD, and no worker has more
// than its part, of which a chunk's teams are eight at least, however the batch is mixed.
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
        cfg.group = n % 3 == 0 ? 8 : n % 11 == 0 ? 1 << rng() % 5 : 4;
        cfg.prefill_tokens = 12 * (16 / cfg.group);
        if (n % 13 == 0) cfg.compute_units = 32 << rng() % 3, cfg.block_slots = 2 * cfg.compute_units;   // a partition of the device
        cfg.one_block_per_cu = n % 7 == 0;
        if (n % 17 == 0) cfg.n_teams = log_uniform(1, 600);
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
        // every worker of a pool has its part to within a pair; a small chunk is spread over eight teams, or as many as there are four
        // pairs for
        int pairs[2] = {0, 0}, longest[2] = {0, 0};
        for (int w = 0; w < workers; w++) {
            int run = 0;
            for (int i = plan.worker_begin[w]; i < plan.worker_begin[w + 1]; i++) run += (plan.items[i].page_end - plan.items[i].page_begin + 1) / 2;
            const int pool = w < plan.n_team_workers ? 0 : 1;
            pairs[pool] += run;
            longest[pool] = std::max(longest[pool], run);
        }
        for (int pool = 0; pool < 2; pool++) {
            const int n_pool = pool == 0 ? plan.n_team_workers : workers - plan.n_team_workers;
            REQUIRE(n_pool == 0 ? pairs[pool] == 0 : longest[pool] <= (pairs[pool] + n_pool - 1) / n_pool + 1);
        }
        // places of an XCD: 32 compute units of a whole device, of two blocks each
        const int per_xcd = (plan.n_team_workers + 7) / 8 + ((workers - plan.n_team_workers + 3) / 4 + 7) / 8;
        const int units_per_xcd = cfg.compute_units / 8;
        const bool asked = cfg.n_teams > 0 && pairs[0] > 0 && pairs[1] > 0;   // a number of teams that the caller names may not fit in whole eighths
        REQUIRE(per_xcd <= 2 * units_per_xcd + (asked ? 1 : 0));
        REQUIRE(!cfg.one_block_per_cu || asked || per_xcd <= units_per_xcd);
        REQUIRE(asked || plan.two_blocks_per_cu || per_xcd <= units_per_xcd);
        REQUIRE(!plan.two_blocks_per_cu || (!asked && !cfg.one_block_per_cu));
        crowded += per_xcd > units_per_xcd;
        REQUIRE(asked || pairs[0] == 0 || plan.n_team_workers >= std::max(1, std::min(8, pairs[0] / 4)));
        // Items of one (sequence, head, query block) follow each other: one with final output, or pieces whose slots the groups of the
        // block's tiles name, in order.
        const int TQ = 16 / cfg.group;
        int slot = 0, n_pieces = 0;
        size_t group = 0;
        for (size_t i = 0; i < plan.items.size();) {
            const AttnItem& first = plan.items[i];
            size_t end = i + 1;
            while (end < plan.items.size() && plan.items[end].seq == first.seq && plan.items[end].kv_head == first.kv_head && plan.items[end].q_tok0 == first.q_tok0) end++;
            if (end - i == 1) {
                REQUIRE(first.partial < 0);
            } else {
                const int tiles = plan.seqs[first.seq].n_new <= TQ ? 1 : cfg.prefill_tokens / TQ;   // slots of a piece
                for (int t = 0; t < (first.q_ntok + TQ - 1) / TQ; t++, group++) {
                    REQUIRE(group < plan.groups.size());
                    const MergeGroup& g = plan.groups[group];
                    REQUIRE(g.tok0 == first.tok_g0 + t * TQ && g.n_tok == std::min(TQ, first.q_ntok - t * TQ) && g.kv_head == first.kv_head);
                    REQUIRE(g.first_slot == slot + t && g.n_splits == (int)(end - i) && g.stride == tiles && t < tiles);
                }
                for (size_t j = i; j < end; j++, slot += tiles) REQUIRE(plan.items[j].partial == slot);
                n_pieces += (int)(end - i);
            }
            i = end;
        }
        REQUIRE(group == plan.groups.size() && slot == plan.n_partial_slots && n_pieces == plan.n_partial_items);
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
