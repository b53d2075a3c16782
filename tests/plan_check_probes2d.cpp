// Check of the probe lists of the 2D workgroup tiles (host code only; built
// and run by test_plan_probes2d.py): on random grids of several problems,
// every probe is in the list of the one tile that writes its cell, or of
// every tile that loads it, at its place in the tile; lists are in order of
// the rows, probes of one cell in order of their slots.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "common.hpp"
using namespace gem;

int main() {
    std::mt19937 g(3);
    auto U = [&](int a, int b) { return (int)(a + g() % (unsigned)(b - a + 1)); };
    int bad = 0, runs = 0;
    for (int it = 0; it < 1500; ++it) {
        const int np = U(1, 3), cls = U(0, 1), TB = U(1, 15), rows = it % 2 ? wg2d_shape(cls, 0).none : 0;
        std::vector<TileW> tiles;
        std::vector<WgProbe> pr;
        for (int p = 0; p < np; ++p) {
            const int nx = U(3, 300), ny = U(3, 400);
            const int lo = nx > 30 && ny > 30 ? U(0, 12) : 0, s[2] = {lo, lo};
            wg2d_plan(p, nx, ny, cls, 0, TB, s, s, tiles);
            for (int n = U(0, 200), q = 0; q < n; ++q) pr.push_back(WgProbe{p, U(0, nx - 1), U(0, n > 100 ? 2 : ny - 1), q});
        }
        std::vector<int> start, cell, slot;
        wg2d_probes(tiles, rows, pr, start, cell, slot);
        bool ok = start.size() == tiles.size() + 1 && start[0] == 0 && start.back() == (int)cell.size() && cell.size() == slot.size();
        size_t seen = 0;
        for (size_t t = 0; ok && t < tiles.size(); ++t) {
            const TileW &T = tiles[t];
            std::vector<std::pair<int, int>> want;
            for (const WgProbe &p : pr) {
                const bool in = rows ? p.i >= T.a && p.i < T.a + rows && p.j >= T.c && p.j < T.c + 64
                                     : p.i >= T.i0 && p.i < T.i1 && p.j >= T.j0 && p.j < T.j1;
                if (in && p.prob == T.prob) want.push_back({(p.i - T.a) * 64 + (p.j - T.c), p.slot});
            }
            std::sort(want.begin(), want.end());
            ok = start[t + 1] - start[t] == (int)want.size();
            for (size_t q = 0; ok && q < want.size(); ++q)
                ok = cell[(size_t)start[t] + q] == want[q].first && slot[(size_t)start[t] + q] == want[q].second;
            seen += want.size();
        }
        ok = ok && seen == cell.size() && (rows || seen == pr.size());
        bad += !ok;
        ++runs;
    }
    printf("%d bad of %d\n", bad, runs);
    return bad != 0;
}
