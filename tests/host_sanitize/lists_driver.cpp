// Sizes of a team's lists (team_list_cap, team_list_size) for degree sequences: room for
// the largest pushes of any share, and lists that a few hubs do not blow up.
#include <algorithm>
#include <cstdio>
#include <functional>
#include <numeric>
#include <random>
#include <vector>

#include "gbp_internal.h"

namespace {
int failures = 0;

// regular: `low` neighbours, and `hubs` vertices of `high`.  limit: entries a vertex.
void check(const char* what, int n_v, int low, int hubs, int high, int blocks, double limit) {
    std::vector<int> d(n_v, low);
    for (int i = 0; i < hubs; ++i) d[(long long)i * n_v / std::max(hubs, 1)] = std::min(high, n_v - 1);
    std::mt19937 r(n_v);
    for (int i = 0; i < n_v; i += 7) d[i] += (int)(r() % 4);
    int most = blocks;
    const TeamListCap cap = team_list_cap(n_v, d.data(), most);
    const size_t size = team_list_size(cap, most);
    std::sort(d.begin(), d.end(), std::greater<int>());
    std::vector<long long> sum(n_v + 1, 0);
    std::partial_sum(d.begin(), d.end(), sum.begin() + 1);
    bool ok = most >= std::min(32, blocks) && most <= blocks && size <= (size_t)(limit * n_v);
    for (int s = 1; s <= most; ++s) {
        const long long pushes = std::min<long long>(n_v, sum[std::min(n_v, n_v / s + 1)]);
        ok = ok && (long long)cap(s) >= pushes && s * cap(s) <= size;
    }
    std::printf("%-44s %3d blocks, %.1f entries a vertex%s\n", what, most, (double)size / n_v, ok ? "" : "  <-- FAIL");
    if (!ok) ++failures;
}
}  // namespace

int main() {
    check("box", 262144, 14, 0, 0, 256, 32);
    check("box and one hub", 262144, 14, 1, 300, 256, 32);
    check("slice", 1000000, 6, 0, 0, 128, 16);
    check("slice and one hub", 1000000, 6, 1, 300, 128, 16);
    check("slice and one hub of every vertex", 1000000, 6, 1, 1000000, 128, 64);
    check("hubs everywhere", 1000000, 6, 10000, 3000, 128, 64);
    check("two hubs of every vertex", 9000, 8, 2, 9000, 64, 64);
    for (int n : {1, 2, 3, 5, 31, 63, 64, 65, 255, 257, 4097}) check("small", n, std::min(n - 1, 5), 0, 0, 256, 256);
    std::printf("%s (%d failures)\n", failures ? "FAILED" : "OK", failures);
    return failures != 0;
}
