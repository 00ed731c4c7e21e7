// The scratch layout that the setup forms dense level maps in (plan_collapse): every part within
// the scratch, no two parts overlapping, 16-byte aligned maps, and few passes.  Host compiler
// only, under the sanitizers; no GPU.  Prints "ALL OK" or the first failure.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2004_09389_amd/csrc/hdg_host.h"

namespace {

void require(bool c, const char *what, const std::vector<int> &n, size_t have) {
    if (c) return;
    std::printf("FAIL %s: have %zu, levels", what, have);
    for (int v : n) std::printf(" %d", v);
    std::printf("\n");
    std::exit(1);
}

// launches of the collapse with two smoothing steps: nine per pass
int launches(const std::vector<int> &n, const hdg::CollapsePlan &P) {
    int passes = 0;
    for (size_t l = 1; l < n.size(); ++l) passes += (n[l] + P.cols[l] - 1) / P.cols[l];
    return 9 * passes;
}

void check(const std::vector<int> &n, size_t have) {
    const hdg::CollapsePlan P = hdg::plan_collapse(n, have);
    const int top = (int)n.size() - 1;
    size_t end = 0;
    for (int l = 0; l < top; ++l) {
        require(P.map[l] >= end && P.map[l] % 2 == 0, "maps apart and aligned", n, have);
        end = P.map[l] + hdg::dense_doubles(n[l]);
    }
    require(P.work >= end && P.work % 2 == 0, "work vectors behind the maps", n, have);
    size_t least = P.work;
    for (int l = 1; l <= top; ++l) {
        require(P.cols[l] >= 1 && P.cols[l] <= n[l], "columns of a pass", n, have);
        require(P.work + (size_t)3 * (n[l] + n[l - 1]) * P.cols[l] <= P.total, "work vectors within the scratch", n, have);
        least = std::max(least, P.work + (size_t)3 * (n[l] + n[l - 1]) * std::min(n[l], 64));
    }
    require(P.total == std::max(have, least), "more scratch asked for only where there is too little", n, have);
}

}  // namespace

int main() {
    const std::vector<std::vector<int>> hierarchies = {
        {1, 4}, {9, 36}, {16, 64}, {9, 36, 144}, {121, 484, 1936}, {12, 42, 162, 642, 2562}, {49, 196, 784},
        {16, 64, 256, 1024}, {8192}, {625, 2500}, {7, 3, 5}, {1, 1, 1}, {1024, 4096}, {333, 1111}};
    for (const auto &n : hierarchies)
        for (size_t have : {(size_t)0, (size_t)1, (size_t)4097, (size_t)100000, (size_t)875000, (size_t)12000000,
                            (size_t)1 << 31})
            check(n, have);
    // level-5 sphere, p = 1, 6 right-hand sides: a basis of 31 vectors; 865 launches with 64 columns through all levels
    const std::vector<int> sphere5 = {12, 42, 162, 642, 2562};
    const int a = launches(sphere5, hdg::plan_collapse(sphere5, (size_t)31 * 30720 * 2 * 6));
    // 56 x 56 torus, p = 2, one: a basis smaller than the largest pass
    const std::vector<int> torus56 = {49, 196, 784};
    const int b = launches(torus56, hdg::plan_collapse(torus56, (size_t)31 * 9408 * 3));
    std::printf("launches %d %d\n", a, b);
    require(a <= 100, "launches, level-5 sphere", sphere5, 0);
    require(b <= 60, "launches, 56 x 56 torus", torus56, 0);
    std::printf("ALL OK\n");
    return 0;
}
