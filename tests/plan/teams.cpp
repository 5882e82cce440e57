// Prints, for each line of standard input (head_dim, workgroups, query heads per workgroup, rows per query tile, tokens, chunk length,
// summaries, window chunks): the longest key list, and whether forward and dQ take eight waves per workgroup.
#include <cstdio>

#include "ksa_internal.h"

int main() {
    long long d, n_wg, stack, q_rows, n, c, m, C;
    while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld", &d, &n_wg, &stack, &q_rows, &n, &c, &m, &C) == 8) {
        const int64_t longest = ksa_longest_list(c, m, C, n, n / c * m, q_rows);
        std::printf("%lld %d %d\n", (long long)longest, (int)ksa_two_teams((int)d, n_wg, (int)stack, longest, false),
                    (int)ksa_two_teams((int)d, n_wg, (int)stack, longest, true));
    }
    return 0;
}
