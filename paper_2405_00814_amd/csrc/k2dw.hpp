// 2D TMz: several leapfrog steps per pass, one workgroup per tile, the
// tile's state in registers (device code; instantiated in k2dw*.hip).
//
// A tile is 64 columns (one per lane) by W * R rows: wavefront w holds rows
// a + w R .. of Ez, Hx, Hy and the coefficients, R rows of one column per
// lane, in registers.  The tile advances all the steps of the pass in
// place; each step shrinks its exact part by one row and one column per
// side (the H layer reads Ez at i+1 and j+1, the E layer Hy at i-1 and Hx at
// j-1), so a pass of TB steps needs a halo of TB cells and writes what is
// left.  Tiles start at the grid's edge where they meet it (no halo: the
// walls are exact).  Tiles are independent: no order between workgroups.
//
// Neighbours: j+-1 by the DPP lane shifts (a modifier of the subtraction);
// i+-1 from the thread's own registers; across wavefronts only Ez is
// exchanged, the first and last row of each through LDS, double buffered,
// one barrier per step: a wavefront keeps its own copy of Hy of the row
// above its first one and recomputes it.
//
// What bounds it: on small grids the latency of a dependent launch (3.6 us)
// and of the tile's loads (about 3 us), spread over the steps of the pass,
// then 0.35-0.55 us per step (VALU of one CU and a barrier); on large grids
// the VALU (counters, 4096^2 with a Ca map: busy 0.73 of the launch, its
// wavefronts 0.21 of their time waiting for memory, LDS or barriers, 0.47
// to issue; 4.0 TB/s).  The marching kernel (k2dt.hip) moves the state of
// every row through a pipeline of register copies and executes about 32 VALU
// instructions per cell and step besides its halo; here a cell and step
// costs 9 in the step loop (interior, no Ca map; 11.7 over the whole launch
// with one, loads, stores and layers counted), because nothing moves.  Measured, us per
// step with CPML against the default before (single steps below 1.5 M
// cells, four-step marching passes above): 250^2 1.18 (6.3), 400^2 1.43
// (7.4), 1024^2 2.42 (9.5), 2048^2 4.8 (17.3), 4096^2 14.3 (41.5; with a Ca
// map 15.5 against 44.0), 6400^2 32.5 (80.9).  Tiles of 176 rows in two
// workgroups per CU were as fast at 4096^2 (15.6) and slower below (2048^2
// 5.8); 16 wavefronts of 2 or 4 rows no faster than 8 of 4 or 8.
//
// Arithmetic: explicit fused multiply-adds, the same sequence per cell in
// every instance (a CPML term of a cell outside the slabs adds an exact
// zero), so a cell's value does not depend on which tile computed it nor on
// how the steps are grouped into passes.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "devutil.hpp"

namespace gem {

// Lane shifts that read 0 beyond the wavefront's ends.
__device__ __forceinline__ float lane_next0(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_prev0(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}

// Row tables of the x axis for the CPML tiles, in LDS: per row of the tile
// (and the row above it) {1/(kappa d), b, c} of the H and the E type.
struct RowTab {
    float4 h, e;
};

// A uniform value the compiler must not relate to its other uses: per-row
// conditions and offsets derived from it are formed where they are used
// (scalar instructions) instead of being kept for all rows across the step
// loop, where they would spill.
__device__ __forceinline__ int opaque(int x) {
    x = __builtin_amdgcn_readfirstlane(x);
    asm volatile("" : "+s"(x));
    return x;
}

// A value at a uniform address that nothing writes while the kernel runs, by
// scalar loads.
template <class T>
__device__ __forceinline__ T load_const(const T *p) {
#ifdef __HIP_DEVICE_COMPILE__
    typedef const T __attribute__((address_space(4))) *cptr;
    return *(cptr)(uintptr_t)p;
#else
    return *p;
#endif
}

// f(0) .. f(N - 1) with compile-time indices: the row arrays are indexed by
// constants from the start, so they live in registers (loops unrolled by the
// optimiser left some of them in scratch memory).
template <int N, class F>
__device__ __forceinline__ void rows(F &&f) {
    if constexpr (N > 0) {
        rows<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}
#define GEM_INL __attribute__((always_inline))

// Buffer access to an array from a uniform base: one lane offset serves all
// rows (a row is a scalar offset), where global loads would form and hold a
// 64-bit address per row and array.  In bounds by construction; the record
// count is the array's own end.
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Buf(const float *base, int64_t first, int64_t len)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base) + first, (short)0,
                                              (int)(len - first < 0x3fffffff ? (len - first) * 4 : 0xfffffffcll),
                                              0x00027000)) {}
    __device__ __forceinline__ float ld(int voff, int soff) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    }
    __device__ __forceinline__ void st(float v, int voff, int soff) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, soff, 0);
    }
};

// The entries of a tile's probe list (ordered by row) that lie in its rows
// [r0, r0 + n): the first and their number.
__device__ __forceinline__ void wave_entries(const ProbeTiles &pt, int tile, int r0, int n, int lane, int &first,
                                             int &count) {
    first = count = 0;
    if (pt.start == nullptr) return;
    const int b = load_const(pt.start + tile), e = load_const(pt.start + tile + 1);
    for (int q = b; q < e; q += 64) {
        const int row = q + lane < e ? pt.cell[q + lane] >> 6 : -1;
        const uint64_t m = __ballot(row >= r0 && row < r0 + n);
        if (m == 0) continue;
        if (count == 0) first = q + __builtin_ctzll(m);
        count += __popcll(m);
    }
    first = __builtin_amdgcn_readfirstlane(first);
    count = __builtin_amdgcn_readfirstlane(count);
}

template <int W, int RP>
struct WgShared {
    float e[2][W][2][64];        // Ez of each wavefront's first and last row
    int2 pr[W][64];              // each wavefront's first 64 probes: {row << 6 | column, slot}
    RowTab x[W * RP + 1];        // x-axis tables (CPML tiles); entry 0: row a - 1
};

// MAT: 0 = Cb map; 1 = Ca, 2 = Ca and Db, 3 = Db map besides it.
// EDGE: the tile holds wall cells (row 0, column 0) or cells outside the
// grid; PX, PY: it holds x-slab rows, y-slab columns (imply EDGE).  XT: 0 = none, 1 = the
// design cells' values are kept (adjoint), 2 = monitor samples are kept.
template <int R, int W, int MAT, bool EDGE, bool PX, bool PY, int XT, class SH>
__device__ __forceinline__ void wg_tile(const Prob2D &p, const TileW &T, const WgArgs &A, int64_t step, int tile,
                                        SH &sh) {
#pragma clang fp contract(off)
    constexpr bool CA = MAT == 1 || MAT == 2, DB = MAT >= 2;
    const int lane = (int)(threadIdx.x & 63);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nx = p.nx, ny = p.ny;
    const int ib = T.a + w * R;       // first row of the wavefront
    const int j = T.c + lane;
    const bool colin = !EDGE || j < ny;
    const int jc = EDGE ? min(j, ny - 1) : j;
    const bool colup = !EDGE || (j >= 1 && j < ny);
    const int nsteps = A.nsteps;
    const float db0 = p.db0;

    // y profile of the lane's column, x profile of the interior
    const float kHy = PY ? p.y.kH[jc] : p.y.kH[p.y.lo], kEy = PY ? p.y.kE[jc] : p.y.kE[p.y.lo];
    const float kHx0 = p.x.kH[p.x.lo], kEx0 = p.x.kE[p.x.lo];
    const float wHy = db0 * kHy, wHx0 = db0 * kHx0;  // H-layer weights (uniform Db)
    int jj = -1;
    float bHy = 0.f, cHy = 0.f, bEy = 0.f, cEy = 0.f;
    const int syw = p.y.lo + p.y.hi;
    if constexpr (PY) {
        jj = colin ? slab_index(p.y, jc) : -1;
        if (jj >= 0) {
            bHy = p.y.bH[jc]; cHy = p.y.cH[jc];
            bEy = p.y.bE[jc]; cEy = p.y.cE[jc];
        }
    }
    if constexpr (PX) {
        // x tables of rows a - 1 .. a + W R - 1
        for (int q = (int)threadIdx.x; q <= W * R; q += 64 * W) {
            const int i = T.a - 1 + q;
            RowTab t{make_float4(kHx0, 0.f, 0.f, 0.f), make_float4(kEx0, 0.f, 0.f, 0.f)};
            if (i >= 0 && i < nx) {
                const bool in = slab_index(p.x, i) >= 0;
                t.h = make_float4(p.x.kH[i], in ? p.x.bH[i] : 0.f, in ? p.x.cH[i] : 0.f, 0.f);
                t.e = make_float4(p.x.kE[i], in ? p.x.bE[i] : 0.f, in ? p.x.cE[i] : 0.f, 0.f);
            }
            if (!DB) t.h.x *= db0;
            sh.x[q] = t;
        }
    }

    float ez[R], hx[R], hy[R], cb[R];
    float ca[CA ? R : 1], db[DB ? R : 1];
    float phx[PY ? R : 1], pzy[PY ? R : 1], phy[PX ? R : 1], pzx[PX ? R : 1];
    const int64_t first = (int64_t)T.a * ny, len = (int64_t)nx * ny;
    const int rb = ny * 4, vo = jc * 4;  // bytes per row, the lane's column
    {
        const Buf bez(p.s0.ez, first, len), bhx(p.s0.hx, first, len), bhy(p.s0.hy, first, len), bcb(p.cb, first, len);
        const Buf bca(CA ? p.ca : p.cb, first, len), bdb(DB ? p.db : p.cb, first, len);
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const int i = ib + r;
            const bool rin = !EDGE || i < nx;
            const int so = ((EDGE ? min(i, nx - 1) : i) - T.a) * rb;
            const bool in = rin && colin;
            const float e = bez.ld(vo, so), x = bhx.ld(vo, so), y = bhy.ld(vo, so), b = bcb.ld(vo, so);
            ez[r] = in ? e : 0.f;
            hx[r] = in ? x : 0.f;
            hy[r] = in ? y : 0.f;
            // Cb > 0 in every cell the E layer updates; 0 marks the others
            cb[r] = in && colup && (!EDGE || i >= 1) ? b : 0.f;
            if constexpr (CA) {
                const float c = bca.ld(vo, so);
                ca[r] = in ? c : 1.f;
            }
            if constexpr (DB) db[r] = bdb.ld(vo, so);
        });
    }
    if constexpr (PY) {
        const int vy = max(jj, 0) * 4, sb = syw * 4;
        const int64_t f0 = (int64_t)T.a * syw, l0 = (int64_t)nx * syw;
        const Buf phxb(p.s0.psi_hx, f0, l0), pzyb(p.s0.psi_ezy, f0, l0);
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const int so = (min(ib + r, nx - 1) - T.a) * sb;
            const float x = phxb.ld(vy, so), y = pzyb.ld(vy, so);
            const bool in = jj >= 0 && ib + r < nx;
            phx[r] = in ? x : 0.f;
            pzy[r] = in ? y : 0.f;
        });
    }
    if constexpr (PX) {
        const int64_t lx = (int64_t)(p.x.lo + p.x.hi) * ny;
        const Buf phyb(p.s0.psi_hy, 0, lx), pzxb(p.s0.psi_ezx, 0, lx);
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const int ii = ib + r < nx ? slab_index(p.x, ib + r) : -1;
            phy[r] = pzx[r] = 0.f;
            if (ii >= 0 && colin) {
                phy[r] = phyb.ld(vo, ii * rb);
                pzx[r] = pzxb.ld(vo, ii * rb);
            }
        });
    }
    // Hy (and its x-slab psi, Db) of the row above the wavefront's first:
    // not needed where it is outside the grid or the tile's first row
    float hyp = 0.f, php = 0.f, dbp = db0;
    if (w > 0 && (!EDGE || ib - 1 < nx)) {
        const int64_t row = (int64_t)(ib - 1) * ny;
        const float y = (p.s0.hy + row)[jc];
        hyp = colin ? y : 0.f;
        if constexpr (DB) dbp = (p.db + row)[jc];
        if constexpr (PX) {
            const int ii = slab_index(p.x, ib - 1);
            if (ii >= 0 && colin) php = (p.s0.psi_hy + (int64_t)ii * ny)[jc];
        }
    }

    // source rows of this wavefront
    const bool hs = p.src_idx >= 0;
    const int si0 = hs ? p.src_box[0] : 0, si1 = hs ? p.src_box[1] : 0, sj0 = p.src_box[2], sj1 = p.src_box[3];
    const bool srcw = hs && si0 < ib + R && si1 > ib && sj0 < T.c + 64 && sj1 > T.c;
    const bool srcj = j >= sj0 && j < sj1;
    auto src_at = [&](int64_t n) { return srcw && n < p.src_len ? load_const(p.src_vals + n) : 0.f; };
    float sval = src_at(step);

    // probes in this wavefront's rows, one per lane: the first 64, and the
    // rows that hold them, in registers where the rows leave some (4 rows:
    // 128^2 with four probes 0.79 us per step, 0.87 without), else in LDS;
    // further ones read again at every step.  A lane's value comes from the
    // lane of its column, row by row over the rows that hold probes (looked
    // up one by one, behind scalar loads, 64 probes on a 64^2 grid took 16 us
    // per step, 0.88 so)
    constexpr bool KEEP = R <= 4;
    int2 mine = make_int2(0, 0);
    int pfirst, pcount;
    wave_entries(A.pt, tile, w * R, R, lane, pfirst, pcount);
    if (pcount > 0) {  // (uniform: the wait for these loads is a wait for all before them)
        const int q = pfirst + min(lane, pcount - 1);
        mine = make_int2(A.pt.cell[q] - (w * R << 6), A.pt.slot[q]);
        if (!KEEP) sh.pr[w][lane] = mine;
    }
    // the rows (bits) that hold entries
    auto rows_of = [&](int row) GEM_INL {
        unsigned m = 0;
        rows<R>([&](auto rc) GEM_INL { m |= __any(row == decltype(rc)::value) ? 1u << decltype(rc)::value : 0u; });
        return m;
    };
    const unsigned first_rows = KEEP && pcount > 0 ? rows_of(mine.x >> 6) : 0u;
    auto record = [&](int g, int64_t n) GEM_INL {
        const bool on = g + lane < pcount;
        int2 q = make_int2(0, 0);
        if (g == 0) q = KEEP ? mine : sh.pr[w][lane];
        else if (on) q = make_int2(A.pt.cell[pfirst + g + lane] - (w * R << 6), A.pt.slot[pfirst + g + lane]);
        const int row = on ? q.x >> 6 : -1, col = (q.x & 63) << 2;
        const unsigned in = KEEP ? (unsigned)opaque((int)(g == 0 ? first_rows : rows_of(row))) : 0u;
        float v = 0.f;
        auto take = [&](const float (&f)[R]) GEM_INL {
            rows<R>([&](auto rc) GEM_INL {
                constexpr int r = decltype(rc)::value;
                if (KEEP ? (in >> r & 1) != 0 : (bool)__any(row == r)) {
                    const float x = __int_as_float(__builtin_amdgcn_ds_bpermute(col, __float_as_int(f[r])));
                    v = row == r ? x : v;
                }
            });
        };
        // (the three conditions opaque: known to exclude one another, the
        // arrays were merged into one indexed access, in memory)
        if (opaque(p.probe_comp == FDTD_EZ)) take(ez);
        if (opaque(p.probe_comp == FDTD_HX)) take(hx);
        if (opaque(p.probe_comp == FDTD_HY)) take(hy);
        if (on) p.rec[(int64_t)q.y * p.rec_stride + (n - p.rec_base)] = v;
    };

    // design-cell capture and monitor rows
    const bool ownj = j >= T.j0 && j < T.j1;
    const bool capj = XT == 1 && ownj && j >= A.cap.design.z && j < A.cap.design.w;
    const bool capw = XT == 1 && A.cap.design.x < min(ib + R, T.i1) && A.cap.design.y > max(ib, T.i0);
    const int cw = XT == 1 ? A.cap.design.w - A.cap.design.z : 0;
    const bool tapj = XT == 2 && ownj && j >= A.tap.j0 && j < A.tap.j1;
    const bool tapw = XT == 2 && A.tap.i0 < min(ib + R, T.i1) && A.tap.i1 > max(ib, T.i0);

    sh.e[0][w][0][lane] = ez[0];
    sh.e[0][w][1][lane] = ez[R - 1];
    __syncthreads();

    for (int s = 0; s < nsteps; ++s) {
        const float svn = s + 1 < nsteps ? src_at(step + s + 1) : 0.f;
        const float up = w > 0 ? sh.e[s & 1][w > 0 ? w - 1 : 0][1][lane] : 0.f;
        const float dn = w < W - 1 ? sh.e[s & 1][w < W - 1 ? w + 1 : w][0][lane] : 0.f;
        // ---- H layer ----
        {
            const float d = ez[0] - up;
            float k = DB ? kHx0 : wHx0, b = 0.f, c = 0.f;
            if constexpr (PX) { const float4 t = sh.x[w * R].h; k = t.x; b = t.y; c = t.z; }
            if constexpr (PX) php = __builtin_fmaf(c, d, b * php);
            if constexpr (DB) {
                float t = d * k;
                if constexpr (PX) t += php;
                hyp = __builtin_fmaf(dbp, t, hyp);
            } else {
                hyp = __builtin_fmaf(k, d, hyp);
                if constexpr (PX) hyp = __builtin_fmaf(db0, php, hyp);
            }
        }
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const float e = ez[r];
            const float dy = lane_next0(e) - e;
            const float dx = (r + 1 < R ? ez[r + 1 < R ? r + 1 : r] : dn) - e;
            float k = DB ? kHx0 : wHx0, b = 0.f, c = 0.f;
            if constexpr (PX) { const float4 t = sh.x[w * R + r + 1].h; k = t.x; b = t.y; c = t.z; }
            if constexpr (PY) phx[r] = __builtin_fmaf(cHy, dy, bHy * phx[r]);
            if constexpr (PX) phy[r] = __builtin_fmaf(c, dx, b * phy[r]);
            if constexpr (DB) {
                float ty = dy * kHy, tx = dx * k;
                if constexpr (PY) ty += phx[r];
                if constexpr (PX) tx += phy[r];
                hx[r] = __builtin_fmaf(-db[r], ty, hx[r]);
                hy[r] = __builtin_fmaf(db[r], tx, hy[r]);
            } else {
                hx[r] = __builtin_fmaf(-wHy, dy, hx[r]);
                hy[r] = __builtin_fmaf(k, dx, hy[r]);
                if constexpr (PY) hx[r] = __builtin_fmaf(-db0, phx[r], hx[r]);
                if constexpr (PX) hy[r] = __builtin_fmaf(db0, phy[r], hy[r]);
            }
            if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        });
        // ---- E layer ----
        const int ib1 = XT == 1 ? opaque(ib) : ib;
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const float dy = hy[r] - (r > 0 ? hy[r > 0 ? r - 1 : 0] : hyp);
            const float dx = hx[r] - lane_prev0(hx[r]);
            const bool upd = !EDGE || cb[r] != 0.f;
            float k = kEx0, b = 0.f, c = 0.f;
            if constexpr (PX) { const float4 t = sh.x[w * R + r + 1].e; k = t.x; b = t.y; c = t.z; }
            float t = __builtin_fmaf(k, dy, -(kEy * dx));
            if constexpr (PX) {
                const float q = __builtin_fmaf(c, dy, b * pzx[r]);
                pzx[r] = upd ? q : pzx[r];
                t += q;
            }
            if constexpr (PY) {
                const float q = __builtin_fmaf(cEy, dx, bEy * pzy[r]);
                pzy[r] = upd ? q : pzy[r];
                t -= q;
            }
            if constexpr (XT == 1) {
                const int i = ib1 + r;
                if (capw && i >= T.i0 && i < T.i1 && i >= A.cap.design.x && i < A.cap.design.y && capj && upd) {
                    const int64_t q = (step + s - A.cap.k0) * A.cap.nd + (int64_t)(i - A.cap.design.x) * cw +
                                      (j - A.cap.design.z);
                    A.cap.ez[q] = ez[r];
                    A.cap.br[q] = t;
                }
            }
            float n;
            // (fma(ca, ez, cb t) needed more registers than there are: 4096^2
            // 22 us per step for 16)
            if constexpr (CA) n = __builtin_fmaf(cb[r], t, ca[r] * ez[r]);
            else n = __builtin_fmaf(cb[r], t, ez[r]);
            ez[r] = upd ? n : ez[r];
            if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        });
        if (srcw) {
            const unsigned q0 = (unsigned)opaque(ib - si0), q1 = (unsigned)(si1 - si0);
            const float v = srcj ? sval : 0.f;
            rows<R>([&](auto rc) GEM_INL {
                constexpr int r = decltype(rc)::value;
                if (q0 + (unsigned)r < q1) ez[r] += v;
            });
        }
        sval = svn;
        sh.e[(s + 1) & 1][w][0][lane] = ez[0];
        sh.e[(s + 1) & 1][w][1][lane] = ez[R - 1];
        for (int g = 0; g < pcount; g += 64) record(g, step + s);
        if constexpr (XT == 2) {
            if (tapw) {
                float *row = A.tap.ring + (int64_t)s * A.tap.npts;
                const int ib2 = opaque(ib);
                auto tap = [&](const float (&v)[R]) GEM_INL {
                    rows<R>([&](auto rc) GEM_INL {
                        constexpr int r = decltype(rc)::value;
                        const int i = ib2 + r;
                        if (i < T.i0 || i >= T.i1 || i < A.tap.i0 || i >= A.tap.i1 || !tapj) return;
                        row[(int64_t)(i - A.tap.i0) * (A.tap.j1 - A.tap.j0) + (j - A.tap.j0)] = v[r];
                    });
                };
                if (opaque(A.tap.comp == FDTD_EZ)) tap(ez);
                if (opaque(A.tap.comp == FDTD_HX)) tap(hx);
                if (opaque(A.tap.comp == FDTD_HY)) tap(hy);
            }
        }
        __syncthreads();
    }

    {
        const int i3 = opaque(ib), so3 = opaque(rb), vs = j * 4;
        const Buf bez(p.s1.ez, first, len), bhx(p.s1.hx, first, len), bhy(p.s1.hy, first, len);
        if (ownj)
            rows<R>([&](auto rc) GEM_INL {
                constexpr int r = decltype(rc)::value;
                const int i = i3 + r, so = (i - T.a) * so3;
                if (i < T.i0 || i >= T.i1) return;
                bez.st(ez[r], vs, so);
                bhx.st(hx[r], vs, so);
                bhy.st(hy[r], vs, so);
            });
        if constexpr (PX || PY) {
            const int fi = T.a, vy = max(jj, 0) * 4, sb = opaque(syw * 4);
            const Buf phxb(p.s1.psi_hx, (int64_t)fi * syw, (int64_t)nx * syw),
                pzyb(p.s1.psi_ezy, (int64_t)fi * syw, (int64_t)nx * syw);
            const int64_t lx = (int64_t)(p.x.lo + p.x.hi) * ny;
            const Buf phyb(p.s1.psi_hy, 0, lx), pzxb(p.s1.psi_ezx, 0, lx);
            if (ownj)
                rows<R>([&](auto rc) GEM_INL {
                    constexpr int r = decltype(rc)::value;
                    const int i = i3 + r;
                    if (i < T.i0 || i >= T.i1) return;
                    if (PY && jj >= 0) {
                        phxb.st(phx[PY ? r : 0], vy, (i - fi) * sb);
                        pzyb.st(pzy[PY ? r : 0], vy, (i - fi) * sb);
                    }
                    const int ii = PX ? slab_index(p.x, i) : -1;
                    if (ii >= 0) {
                        phyb.st(phy[PX ? r : 0], vs, ii * so3);
                        pzxb.st(pzx[PX ? r : 0], vs, ii * so3);
                    }
                });
        }
    }
}

// R, RQ, RP: rows per wavefront of the tiles of kind 0, kinds 1 to 3, kind
// 4; W wavefronts; MW: wavefronts per SIMD the
// registers must allow.
template <int R, int RQ, int RP, int W, int MAT, int XT, class SH>
__device__ __forceinline__ void wg_kind(const Prob2D &p, const TileW &T, const WgArgs &A, int64_t step, int tile,
                                        SH &sh) {
    if (T.kind == 0) wg_tile<R, W, MAT, false, false, false, XT>(p, T, A, step, tile, sh);
    else if (T.kind == 1) wg_tile<RQ, W, MAT, true, false, false, XT>(p, T, A, step, tile, sh);
    else if (T.kind == 2) wg_tile<RQ, W, MAT, true, false, true, XT>(p, T, A, step, tile, sh);
    else if (T.kind == 3) wg_tile<RQ, W, MAT, true, true, false, XT>(p, T, A, step, tile, sh);
    else wg_tile<RP, W, MAT, true, true, true, XT>(p, T, A, step, tile, sh);
}

template <int R, int RQ, int RP, int W, int MW, int MAT, bool BATCH, int XT>
__global__ __launch_bounds__(64 * W, MW) void k2d_wg(WgArgs A) {
    __shared__ WgShared<W, (RQ > RP ? RQ : RP)> sh;
    const int tile = xcd_block((int)blockIdx.x, (int)gridDim.x);
    if (tile >= A.ntiles) return;  // whole workgroup
    const TileW T = load_const(A.tiles + tile);
    // the problem by value: its pointers and sizes are scalars for the whole
    // tile (behind a pointer they were read again after every store, into
    // vector registers)
    const Prob2D p = BATCH ? load_const(A.probs + T.prob) : A.p;
    const int64_t step = (BATCH ? load_const(A.step_base) : 0) + A.step;
    // a batch's problem runs the code of its own maps (MAT stands for all the
    // maps that any of them has, and for the tiles' rows)
    constexpr bool CA = MAT == 1 || MAT == 2, DB = MAT >= 2;
    if constexpr (!BATCH || MAT == 0) {
        wg_kind<R, RQ, RP, W, MAT, XT>(p, T, A, step, tile, sh);
    } else {
        const bool ca = CA && p.ca != nullptr, db = DB && p.db != nullptr;
        if (!ca && !db) wg_kind<R, RQ, RP, W, 0, XT>(p, T, A, step, tile, sh);
        if constexpr (CA)
            if (ca && !db) wg_kind<R, RQ, RP, W, 1, XT>(p, T, A, step, tile, sh);
        if constexpr (CA && DB)
            if (ca && db) wg_kind<R, RQ, RP, W, 2, XT>(p, T, A, step, tile, sh);
        if constexpr (DB)
            if (!ca && db) wg_kind<R, RQ, RP, W, 3, XT>(p, T, A, step, tile, sh);
    }
}

template <int R, int RQ, int RP, int W, int MW, int MAT>
static hipError_t wg_go(const WgArgs &a, int xt, hipStream_t st) {
    // the instances that keep design values or samples need more registers
    constexpr int MX = R > 8 ? 3 : MW;
    const dim3 g((unsigned)((a.ntiles + 7) / 8 * 8)), b(64 * W);
    if (a.probs) {
        if (xt != 0) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k2d_wg<R, RQ, RP, W, MW, MAT, true, 0>), g, b, 0, st, a);
    } else if (xt == 0) {
        hipLaunchKernelGGL((k2d_wg<R, RQ, RP, W, MW, MAT, false, 0>), g, b, 0, st, a);
    } else if (xt == 1) {
        hipLaunchKernelGGL((k2d_wg<R, RQ, RP, W, MX, MAT, false, 1>), g, b, 0, st, a);
    } else {
        hipLaunchKernelGGL((k2d_wg<R, RQ, RP, W, MX, MAT, false, 2>), g, b, 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace gem
