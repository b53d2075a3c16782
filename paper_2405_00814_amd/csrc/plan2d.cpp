// Host-side tile plan of the 2D multi-step kernel (pure integer work).
#include <algorithm>
#include <array>
#include <iterator>
#include <vector>

#include "common.hpp"

namespace gem {

bool tb2d_supported(int ny, int V, int TB, int TX) {
    if (!(V == 1 || V == 2 || V == 4) || !(TB == 2 || TB == 4)) return false;
    if (TX < 1 || TX > 65536) return false;
    return ny % V == 0;
}

// The default row chunk.  Measured on 1448^2 - 6400^2 dielectric grids
// (four steps per pass, CPML tiles on a second stream, one column per lane):
// 32-row chunks where the interior workgroups (four strips each) still
// number at least 4 per CU, else 16 where they number 2 per CU, else 8 or
// 4 (4096^2: 373 Gcell/s at 32 rows, 376 at 16; 6400^2: 454 vs 412;
// 3000^2: 334 vs 317; 2048^2: 16 rows, 234 vs 214).  With two columns per
// lane: 32 rows where the interior workgroups number 4-5 per CU, 16 in
// that band, else 8.
int tb2d_default_tx(int nx, int ny, int V, int cus) {
    const int own = tb2d_own(V, 4);
    auto wgs = [&](int tx) { return (int64_t)((nx + tx - 1) / tx) * ((ny + own - 1) / own) / 4; };
    if (V == 2) {
        for (int tx : {32, 16})
            if (wgs(tx) >= 4 * (int64_t)cus && wgs(tx) <= 5 * (int64_t)cus) return tx;
        return 8;
    }
    if (wgs(32) >= 4 * (int64_t)cus) return 32;
    for (int tx : {16, 8})
        if (wgs(tx) >= 2 * (int64_t)cus) return tx;
    return 4;
}

void tb2d_plan(int prob, int nx, int ny, int V, int TB, int TX, int TXo, const int *xlohi, const int *ylohi,
               std::vector<Tile2T> &inner, std::vector<Tile2T> &outer) {
    if (TXo < 1) TXo = TX;
    const int ow = tb2d_own(V, TB), hw = tb2d_halo(V, TB) * V;
    auto clear = [](int n, int lo, int hi, int a, int b) {  // no slab index in [a, b)
        a = std::max(a, 0);
        b = std::min(b, n);
        for (int q = a; q < b; ++q)
            if (q < lo || q >= n - hi) return false;
        return true;
    };
    for (int i0 = 0; i0 < nx; i0 += TX) {
        const int i1 = std::min(i0 + TX, nx);
        const bool xc = clear(nx, xlohi[0], xlohi[1], i0 - TB, i1 + TB);
        for (int ja = 0; ja < ny; ja += ow) {
            const bool yc = clear(ny, ylohi[0], ylohi[1], ja - hw, ja - hw + 64 * V);
            if (xc && yc) {
                inner.push_back(Tile2T{prob, i0, i1, ja});
            } else {
                // tiles with the CPML code in pieces of TXo rows
                for (int a = i0; a < i1; a += TXo) outer.push_back(Tile2T{prob, a, std::min(a + TXo, i1), ja});
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Workgroup tiles (k2dw.hpp)
// ---------------------------------------------------------------------------
bool wg2d_supported(int ny, int sx, int sy, int cls, int TB) {
    // byte offsets of a tile's rows and of the x slabs' rows fit 31 bits; a
    // tile keeps cells to write
    return ny >= 3 && ny <= (1 << 20) && (int64_t)sx * ny < (1 << 29) && sy <= (1 << 20) && cls >= 0 && cls < kWgClasses && TB >= 1 && TB <= 15 &&
           wg2d_shape(cls, 2).both > 2 * TB;
}

bool res2d_supported(int nx, int ny, bool cpml, int np) {
    if (cpml || nx < 1 || ny < 1 || ny > 1024 || np > 64) return false;
    const int bands = 1024 / ((ny + 63) / 64 * 64);
    return (nx + bands - 1) / bands <= 16;
}

// Measured over 64^2 .. 6400^2 on 256 CUs (us per step): tiles of 32 rows
// while there are at most two per CU at 12 steps per pass (250^2 1.18
// against 1.70 with 64 rows, 400^2 1.43 against 1.61), then 64 rows up to
// about two per CU (1024^2 2.42 against 2.46 with 96 rows and 3.0 with 32),
// then 96 (2048^2 4.8 against 6.0).  More steps per pass cost halo and save
// launches: 14 while all tiles run at once, 12, or 10 where 12 would start
// another round (1024^2: 10 steps 2.42, 12 steps 2.79; 4096^2: 12 steps
// 14.3, 8 steps 18.0; with a Db map, 64-row tiles, 10 steps 20.1, 12 20.8).
void wg2d_default(const std::vector<std::pair<int, int>> &grids, int mat, int cus, int &cls, int &TB) {
    auto along = [](int n, int h, int tb) { return n <= h ? 1 : 2 + std::max(0, (n - 2 * (h - tb) + h - 2 * tb - 1) / (h - 2 * tb)); };
    auto count = [&](int h, int tb) {
        int64_t n = 0;
        for (const auto &g : grids) n += (int64_t)along(g.first, h, tb) * along(g.second, 64, tb);
        return n;
    };
    // (a grid of at most 32 rows would leave the rest of taller tiles empty:
    // 8x100000 2.9 us per step in passes of 12, 4.4 in tiles of 56 rows)
    const bool thin = std::all_of(grids.begin(), grids.end(), [](const auto &g) { return g.first <= 32; });
    if (thin || count(32, 12) <= 2 * (int64_t)cus) {
        cls = 0;
        TB = count(32, 14) <= cus ? 14 : 12;
        return;
    }
    if (count(64, 10) * 4 <= 9 * (int64_t)cus) {
        cls = 1;
        for (TB = 14; TB > 10 && count(64, TB) * 10 > 21 * (int64_t)cus;) TB -= 2;
        return;
    }
    cls = 2;
    TB = mat == 2 ? 10 : 12;
}

// A pass moves and computes all 32 rows of its tiles, a single step the
// grid's own.  On grids of few rows with more than two tiles per CU, us
// with r = tiles per CU: a pass of k steps 3 + r (1.5 + 0.16 k), a single
// step 3.1 + 0.058 r nx (3x80000, r = 7.8: calls of 3 steps 1.15 times a
// single step's time in tiles, of 4 0.97; 8x80000: of 2 1.23, of 3 0.96;
// 12x80000: of 2 1.07; 16x80000: of 2 0.87).
int wg2d_least(int nx, int ntiles, int cus) {
    const double r = (double)ntiles / cus;
    if (nx > 32 || r <= 2) return 2;
    for (int k = 2; k <= 15; ++k)
        if (3 + r * (1.5 + 0.16 * k) <= k * (3.1 + 0.058 * r * nx)) return k;
    return 16;
}

int trial_steps_of(const fdtd_kernel_config &k, int ndim, int trial) {
    const int per = k.variant != 3 ? 1 : ndim == 2 ? k.tile[2] : 2;
    return (trial + per - 1) / per * per;
}

void wg2d_plan(int prob, int nx, int ny, int cls, int mat, int TB, const int *xlohi, const int *ylohi,
               std::vector<TileW> &tiles) {
    const WgShape sh = wg2d_shape(cls, mat);
    const int xlo = xlohi[0], xhi = xlohi[1], ylo = ylohi[0], yhi = ylohi[1];
    std::vector<TileW> t;
    for (int j0 = 0; j0 < ny;) {
        const int c = j0 > 0 ? j0 - TB : 0;
        const int j1 = c + 64 >= ny ? ny : c + 64 - TB;
        // the strip's loaded columns: slab cells, walls or ghosts
        const bool py = (ylo > 0 && c < ylo) || (yhi > 0 && c + 64 > ny - yhi);
        const bool ey = c == 0 || c + 64 > ny;
        for (int i0 = 0; i0 < nx;) {
            int a = i0 > 0 ? i0 - TB : 0;
            auto slab = [&](int rows) { return (xlo > 0 && a < xlo) || (xhi > 0 && a + rows > nx - xhi); };
            // the tallest tile that the rows from a allow: clear of the x
            // slabs, and (kind 0) of the walls and the grid's end
            const int tall = py ? sh.one : sh.none;
            const bool edge = ey || a == 0;
            int kind, rows;
            if (!slab(tall) && (py || (!edge && a + tall <= nx))) {
                kind = py ? 2 : 0;
                rows = tall;
            } else {
                // a tile that would reach into the last slab (or past the
                // last row) is moved up to end before it, where that leaves
                // it at least half its rows
                const int a2 = nx - xhi - tall;
                if (a2 < a && a2 >= std::max(xlo, 1) && (py ? xhi > 0 : !ey) &&
                    a2 + tall - (xhi > 0 ? TB : 0) - i0 >= (tall - 2 * TB) / 2) {
                    a = a2;
                    kind = py ? 2 : 0;
                    rows = tall;
                } else if (!slab(sh.one)) {
                    kind = py ? 2 : 1;
                    rows = sh.one;
                } else {
                    kind = py ? 4 : 3;
                    rows = py ? sh.both : sh.one;
                }
            }
            const int i1 = a + rows >= nx ? nx : a + rows - TB;
            t.push_back(TileW{prob, kind, i0, i1, j0, j1, a, c});
            i0 = i1;
        }
        j0 = j1;
    }
    // rows together: neighbouring strips share their halo rows' lines
    std::stable_sort(t.begin(), t.end(), [](const TileW &u, const TileW &v) { return u.i0 < v.i0; });
    tiles.insert(tiles.end(), t.begin(), t.end());
}

void wg2d_probes(const std::vector<TileW> &tiles, int rows, const std::vector<WgProbe> &probes, std::vector<int> &start,
                 std::vector<int> &cell, std::vector<int> &slot) {
    std::vector<std::array<int, 3>> ent;  // {tile, cell, slot}
    auto put = [&](int t, const WgProbe &p) {
        ent.push_back({t, (p.i - tiles[(size_t)t].a) << 6 | (p.j - tiles[(size_t)t].c), p.slot});
    };
    if (rows > 0) {
        for (size_t t = 0; t < tiles.size(); ++t)
            for (const WgProbe &p : probes) {
                const TileW &T = tiles[t];
                if (p.prob == T.prob && p.i >= T.a && p.i < T.a + rows && p.j >= T.c && p.j < T.c + 64) put((int)t, p);
            }
    } else {
        // a problem's tiles are one range; a few probes look through it,
        // many through its tiles sorted by strip and first row
        for (size_t u = 0, v = 0; u < probes.size(); u = v) {
            const int prob = probes[u].prob;
            while (v < probes.size() && probes[v].prob == prob) ++v;
            const size_t b = (size_t)(std::lower_bound(tiles.begin(), tiles.end(), prob,
                                                       [](const TileW &T, int q) { return T.prob < q; }) -
                                      tiles.begin());
            size_t e = b;
            while (e < tiles.size() && tiles[e].prob == prob) ++e;
            std::vector<std::array<int, 3>> at;  // {first column, first row, tile}
            if (v - u >= 16) {
                for (size_t t = b; t < e; ++t) at.push_back({tiles[t].j0, tiles[t].i0, (int)t});
                std::sort(at.begin(), at.end());
            }
            auto last = [&](int j, int i) {  // the last tile not beyond (j, i)
                return *std::prev(std::upper_bound(at.begin(), at.end(), std::array<int, 3>{j, i, INT32_MAX}));
            };
            for (size_t q = u; q < v; ++q) {
                const WgProbe &p = probes[q];
                size_t t = b;
                if (!at.empty()) t = (size_t)last(last(p.j, INT32_MAX)[0], p.i)[2];
                else while (!(p.i >= tiles[t].i0 && p.i < tiles[t].i1 && p.j >= tiles[t].j0 && p.j < tiles[t].j1)) ++t;
                put((int)t, p);
            }
        }
    }
    std::sort(ent.begin(), ent.end());
    start.assign(tiles.size() + 1, 0);
    cell.clear();
    slot.clear();
    for (const auto &e : ent) {
        start[(size_t)e[0] + 1]++;
        cell.push_back(e[1]);
        slot.push_back(e[2]);
    }
    for (size_t t = 0; t < tiles.size(); ++t) start[t + 1] += start[t];
}

}  // namespace gem
