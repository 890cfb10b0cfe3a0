// Deals the tiles of expert groups to work-groups, on the host.  Reads problems, one a line: BM ntn n_sel rows...; prints
// for each "covered" or what is wrong, then the least and the most tiles that one of the eight XCDs gets.
#include <cstdio>
#include <vector>

#include "group_tiles.h"

template <int BM>
static void check(int ntn, const std::vector<int>& rows) {
    const int n = (int)rows.size();
    int total = 0, need = 0;
    for (int r : rows) {
        total += r;
        need += (r + BM - 1) / BM * ntn;
    }
    std::vector<std::vector<int>> seen(n);
    for (int i = 0; i < n; ++i) seen[i].assign((size_t)((rows[i] + BM - 1) / BM) * ntn, 0);
    int xcd[8] = {0}, dealt = 0;
    std::vector<int> xcd_of((size_t)n * ntn, -1);
    for (int b = 0; b < (total / BM + n) * ((ntn + 7) / 8 * 8); ++b) {
        haq::GroupTile t;
        if (!haq::deal_group_tile<BM>([&](int i) { return rows[i]; }, n, ntn, b, t)) continue;
        if (t.i < 0 || t.i >= n || t.u < 0 || t.u >= ntn || t.mi < 0 || t.mi >= t.mt || t.mt != (rows[t.i] + BM - 1) / BM) {
            printf("block %d: tile out of range\n", b);
            return;
        }
        int& home = xcd_of[(size_t)t.i * ntn + t.u];
        if (home < 0) home = b % 8;
        if (home != b % 8 || seen[t.i][(size_t)t.mi * ntn + t.u]++) {
            printf("block %d: tile dealt twice, or its weights to two XCDs\n", b);
            return;
        }
        ++xcd[b % 8];
        ++dealt;
    }
    int lo = xcd[0], hi = xcd[0];
    for (int x : xcd) {
        lo = x < lo ? x : lo;
        hi = x > hi ? x : hi;
    }
    printf("%s %d %d\n", dealt == need ? "covered" : "incomplete", lo, hi);
}

int main() {
    int bm, ntn, n;
    while (scanf("%d %d %d", &bm, &ntn, &n) == 3) {
        std::vector<int> rows(n);
        for (int& r : rows)
            if (scanf("%d", &r) != 1) return 1;
        bm == 128 ? check<128>(ntn, rows) : check<256>(ntn, rows);
    }
    return 0;
}
