// Check of the 2D workgroup-tile plan (host code only; built and run by
// test_plan_wg2d.py).  On random grids, slab widths, size classes and steps
// per pass: every cell is written by exactly one tile; every tile's loads
// lie in the rows its kind holds, a halo of TB cells on every side that is
// not the grid's edge; x-slab rows only in the kinds that hold their CPML
// values (3, 4), y-slab columns likewise (2, 4); kind 0 holds neither walls
// nor cells outside the grid.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "common.hpp"
using namespace gem;

int main() {
    std::mt19937 g(1);
    auto U = [&](int a, int b) { return (int)(a + g() % (unsigned)(b - a + 1)); };
    int kinds[5] = {0, 0, 0, 0, 0}, bad = 0, runs = 0;
    for (int it = 0; it < 12000; ++it) {
        const int nx = U(3, it % 7 == 0 ? 900 : 200), ny = U(3, it % 5 == 0 ? 900 : 260);
        int xl[2] = {0, 0}, yl[2] = {0, 0};
        if (U(0, 3))
            for (int *v : {&xl[0], &xl[1], &yl[0], &yl[1]}) *v = U(0, 20);
        if (xl[0] + xl[1] >= nx) xl[0] = xl[1] = 0;
        if (yl[0] + yl[1] >= ny) yl[0] = yl[1] = 0;
        const int cls = U(0, kWgClasses - 1), mat = U(0, 3), TB = U(1, 15);
        if (!wg2d_supported(ny, xl[0] + xl[1], yl[0] + yl[1], cls, TB)) continue;
        const WgShape sh = wg2d_shape(cls, mat);
        std::vector<TileW> t;
        wg2d_plan(7, nx, ny, cls, mat, TB, xl, yl, t);
        std::vector<unsigned char> own((size_t)nx * ny, 0);
        bool ok = true;
        for (const TileW &T : t) {
            if (T.kind < 0 || T.kind > 4 || T.prob != 7) { ok = false; break; }
            kinds[T.kind]++;
            const int rows = T.kind == 0 ? sh.none : T.kind < 4 ? sh.one : sh.both;
            ok = ok && T.a >= 0 && T.a < nx && T.c >= 0 && T.c < ny && T.i0 < T.i1 && T.j0 < T.j1;
            ok = ok && T.i0 >= T.a && T.i1 <= T.a + rows && T.i1 <= nx && T.j0 >= T.c && T.j1 <= T.c + 64 && T.j1 <= ny;
            ok = ok && (T.a == 0 || T.i0 - T.a >= TB) && (T.a + rows >= nx || T.a + rows - T.i1 >= TB);
            ok = ok && (T.c == 0 || T.j0 - T.c >= TB) && (T.c + 64 >= ny || T.c + 64 - T.j1 >= TB);
            bool hx = false, hy = false;
            for (int i = T.a; i < T.a + rows && i < nx; ++i) hx = hx || i < xl[0] || i >= nx - xl[1];
            for (int j = T.c; j < T.c + 64 && j < ny; ++j) hy = hy || j < yl[0] || j >= ny - yl[1];
            ok = ok && (!hx || T.kind >= 3) && (!hy || T.kind == 2 || T.kind == 4);
            ok = ok && (T.kind != 0 || (T.a >= 1 && T.c >= 1 && T.a + rows <= nx && T.c + 64 <= ny));
            if (!ok) break;
            for (int i = T.i0; i < T.i1; ++i)
                for (int j = T.j0; j < T.j1; ++j) own[(size_t)i * ny + j]++;
        }
        for (unsigned char o : own) ok = ok && o == 1;
        ++runs;
        if (!ok) {
            ++bad;
            printf("bad: %dx%d slabs %d %d %d %d class %d mat %d TB %d\n", nx, ny, xl[0], xl[1], yl[0], yl[1], cls, mat, TB);
        }
    }
    for (int k = 0; k < 5; ++k) bad += kinds[k] == 0;
    printf("%d bad of %d\n", bad, runs);
    return bad != 0;
}
