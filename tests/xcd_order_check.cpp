// Checks of the block orders (xcd_order.h), compiled for the host by test_host_xcd_order.py: every row and every merge group is
// taken by exactly one block, rows that share a line meet on one XCD, and small merges reach as many XCDs as they have groups.
#include <cstdio>
#include <set>
#include <vector>

#include "xcd_order.h"

using namespace ps;

int main() {
    for (int n = 1; n <= 3000; n++) {
        std::vector<int> seen(n, -1), group_xcd(n, -1);
        for (int b = 0; b < row_blocks(n); b++) {
            const int r = row_of_block(b, n);
            if (r < 0 || (r < n && seen[r] >= 0)) { printf("row %d of %d\n", r, n); return 1; }
            if (r < n) seen[r] = b & 7;
        }
        for (int r = 0; r < n; r++) {
            if (seen[r] < 0) { printf("row %d of %d has no block\n", r, n); return 1; }
            if (n >= ROW_ROUND && seen[r] != seen[r & ~7]) { printf("rows of an octet on two XCDs, %d of %d\n", r, n); return 1; }
        }
        for (int b = 0; b < merge_blocks(n); b++) {
            const int g = merge_group_of_block(b, n);
            if (g < 0 || (g < n && group_xcd[g] >= 0)) { printf("group %d of %d\n", g, n); return 1; }
            if (g < n) group_xcd[g] = b & 7;
        }
        int per[8] = {0};
        for (int g = 0; g < n; g++) {
            if (group_xcd[g] < 0) { printf("group %d of %d has no block\n", g, n); return 1; }
            per[group_xcd[g]]++;
        }
        int most = 0;
        for (int x : per) most = x > most ? x : most;
        if (most > (n < MERGE_ROUNDS_FROM ? (n + 7) / 8 : (n + 31) / 32 * 4)) { printf("%d of %d groups on one XCD\n", most, n); return 1; }
    }
    printf("OK\n");
    return 0;
}
