// Fused single 3D Yee step, one thread per cell (H layer, E layer, CPML,
// source and probes in one kernel): the step of grids that the caches hold.
//
// Threads take consecutive cells of the linear order, whatever the row
// length, so every lane works and every load is coalesced; a thread writes
// H^{n+1/2} and E^{n+1} of its cell and recomputes the six H values that
// its E layer gathers from the cells at i-1, j-1 and k-1.  Nothing is
// exchanged and nothing is carried from plane to plane: all loads of a
// thread are independent and in flight together.  The marching kernel
// (k3dw.hip) reads each value once from memory but walks its planes in a
// dependent chain: on a grid of 10^5 - 10^7 cells its few workgroups leave
// the chip idle.  Bound by the launch (4 us), then by the latency and rate
// of about 40 cached loads per thread (59 on average on 100x90x84 with
// 10-cell CPML, up to 90 in its corners; counters there: VALU busy 0.42 of
// the launch, 580 instructions per cell, 0.44 of a wavefront's time waiting):
// 19 us per step (118 before), 100^3 without CPML 11 (42).  More wavefronts
// per SIMD at fewer registers spilled and were slower (5: 22 us, 6: 37).
//
// CPML: the values a wavefront needs of an axis' slabs (psi, b, c,
// 1/(kappa d)) are loaded up front, behind one branch per axis that is
// uniform over the wavefront; a cell outside keeps psi = 0 and the interior
// 1/d.
#include <algorithm>

#include "common.hpp"
#include "devutil.hpp"
#include "k3dcell.hpp"

namespace gem {

namespace {

// c / d for 0 <= c < 2^31 and 1 <= d < 2^31: (c * m) >> (32 + s)
struct Div {
    unsigned m, s;
};

Div make_div(unsigned d) {
    if (d == 1) return Div{0, 0};
    unsigned s = 0;
    while (((uint64_t)1 << (s + 1)) < d) ++s;  // 2^s < d <= 2^(s+1)
    // m = ceil(2^(32+s) / d) < 2^32 since d > 2^s; exact for c < 2^31
    // because the error term c (m d - 2^(32+s)) < 2^31 d <= 2^(32+s) d / 2^(s+1)
    const uint64_t m = ((((uint64_t)1 << 32) << s) + d - 1) / d;
    return Div{(unsigned)m, s};
}

}  // namespace

__device__ __forceinline__ int div_by(int c, Div d) {
    return d.m == 0 ? c : (int)(__umulhi((unsigned)c, d.m) >> d.s);
}

// One axis at a cell's index and at the one below: interior or slab values.
struct FlatAx {
    float kH, bH, cH, kE, bE, cE;  // at the index
    float kHm, bHm, cHm;           // at index - 1
    int s, sm;                     // slab indices (-1: outside)
};

template <bool PML>
__device__ __forceinline__ FlatAx flat_axis(const AxisDev &a, int i) {
    FlatAx r;
    r.kH = r.kHm = a.kH[a.lo];
    r.kE = a.kE[a.lo];
    r.bH = r.cH = r.bE = r.cE = r.bHm = r.cHm = 0.f;
    r.s = r.sm = -1;
    if (PML) {
        r.s = slab_index(a, i);
        r.sm = i >= 1 ? slab_index(a, i - 1) : -1;
        if (__any(r.s >= 0 || r.sm >= 0)) {
            const int im = i >= 1 ? i - 1 : 0;
            r.kH = a.kH[i]; r.kE = a.kE[i]; r.kHm = a.kH[im];
            const float bh = a.bH[i], ch = a.cH[i], be = a.bE[i], ce = a.cE[i], bm = a.bH[im], cm = a.cH[im];
            r.bH = r.s >= 0 ? bh : 0.f; r.cH = r.s >= 0 ? ch : 0.f;
            r.bE = r.s >= 0 ? be : 0.f; r.cE = r.s >= 0 ? ce : 0.f;
            r.bHm = r.sm >= 0 ? bm : 0.f; r.cHm = r.sm >= 0 ? cm : 0.f;
        }
    }
    return r;
}

// z slabs: psi' = b psi + c d; 0 outside (x and y slabs round the other
// product, as the marching kernel does).
__device__ __forceinline__ float psi_next(float b, float c, float d, bool in, float psi) {
    return in ? __builtin_fmaf(b, psi, c * d) : 0.f;
}

// part: 0 = every cell; 1, 2 (per-launch profiles) = the cells outside, inside
// the x and y slabs.
template <int MAT, bool PML>
__global__ __launch_bounds__(256) void k3d_flat(Prob3D p, Div dplane, Div drow, ProbeTiles pt, int64_t step, int part) {
#pragma clang fp contract(off)
    const int blk = xcd_block((int)blockIdx.x, (int)gridDim.x);
    const int nz = p.nz, ny = p.ny, nx = p.nx;
    const int sx = ny * nz, n = nx * sx;
    const int c0 = blk * 256, c = c0 + (int)threadIdx.x;
    if (c0 >= n) return;
    const int cc = min(c, n - 1);
    const int i = div_by(cc, dplane), jk = cc - i * sx, j = div_by(jk, drow), k = jk - j * nz;
    const bool xi = i + 1 < nx, yj = j + 1 < ny, zk = k + 1 < nz, im = i >= 1, jm = j >= 1, km = k >= 1;
    const FlatAx X = flat_axis<PML>(p.x, i), Y = flat_axis<PML>(p.y, j), Z = flat_axis<PML>(p.z, k);

    const bool ok = c < n && (part == 0 || (part == 2) == (X.s >= 0 || Y.s >= 0));

    // neighbours' offsets; 0 (the cell itself) where there is none
    const int ox = xi ? sx : 0, oy = yj ? nz : 0, oz = zk ? 1 : 0;
    const int mx = im ? sx : 0, my = jm ? nz : 0, mz = km ? 1 : 0;
    const float *Ex = p.s0.f[FDTD_EX] + cc, *Ey = p.s0.f[FDTD_EY] + cc, *Ez = p.s0.f[FDTD_EZ] + cc;
    const float *Hx = p.s0.f[FDTD_HX] + cc, *Hy = p.s0.f[FDTD_HY] + cc, *Hz = p.s0.f[FDTD_HZ] + cc;
    // old state: own cell, +1 and -1 along each axis (a = x, b = y, c = z)
    const float ex = Ex[0], ey = Ey[0], ez = Ez[0], hx = Hx[0], hy = Hy[0], hz = Hz[0];
    const float eya = Ey[ox], eza = Ez[ox], exb = Ex[oy], ezb = Ez[oy], exc = Ex[oz], eyc = Ey[oz];
    const float exA = Ex[-mx], eyA = Ey[-mx], ezA = Ez[-mx], hyA = Hy[-mx], hzA = Hz[-mx];
    const float exAb = Ex[oy - mx], exAc = Ex[oz - mx];
    const float exB = Ex[-my], eyB = Ey[-my], ezB = Ez[-my], hxB = Hx[-my], hzB = Hz[-my];
    const float eyBa = Ey[ox - my], eyBc = Ey[oz - my];
    const float exC = Ex[-mz], eyC = Ey[-mz], ezC = Ez[-mz], hxC = Hx[-mz], hyC = Hy[-mz];
    const float ezCa = Ez[ox - mz], ezCb = Ez[oy - mz];
    const float cb = p.cb[cc];
    float ca = 1.f, db = p.db0, dbA = db, dbB = db, dbC = db;
    if (MAT == 1 || (MAT == 2 && p.ca)) ca = p.ca[cc];  // (a Db map may come without a Ca map)
    if (MAT == 2) { db = p.db[cc]; dbA = p.db[cc - mx]; dbB = p.db[cc - my]; dbC = p.db[cc - mz]; }

    // psi: H of the own cell (w*), of the cells below (A: i-1, B: j-1, C:
    // k-1), E of the own cell (e*)
    float *const *P0 = p.s0.psi;
    float wxy = 0.f, wxz = 0.f, wyz = 0.f, wyx = 0.f, wzx = 0.f, wzy = 0.f;
    float ayx = 0.f, azx = 0.f, ayz = 0.f, azy = 0.f;  // A
    float bxy = 0.f, bzy = 0.f, bxz = 0.f, bzx = 0.f;  // B
    float cxz = 0.f, cyz = 0.f, cxy = 0.f, cyx = 0.f;  // C
    float qxy = 0.f, qxz = 0.f, qyz = 0.f, qyx = 0.f, qzx = 0.f, qzy = 0.f;
    const int ly = p.y.lo + p.y.hi, lz = p.z.lo + p.z.hi;
    unsigned px = 0, py = 0, pz = 0;
    if (PML) {
        // (loads of lanes outside a slab read its first entry and are
        // dropped: no divergent branch, no wait between the loads)
        if (__any(X.s >= 0 || X.sm >= 0)) {
            const bool a = X.s >= 0, b = X.sm >= 0;
            px = a ? xs3(X.s, j, k, ny, nz) : 0;
            const unsigned pm = b ? xs3(X.sm, j, k, ny, nz) : 0;
            const unsigned pb = a && jm ? px - nz : 0, pc = a && km ? px - 1 : 0;
            const float v0 = P0[PSI_HYX][px], v1 = P0[PSI_HZX][px], v2 = P0[PSI_EYX][px], v3 = P0[PSI_EZX][px];
            const float v4 = P0[PSI_HYX][pm], v5 = P0[PSI_HZX][pm], v6 = P0[PSI_HZX][pb], v7 = P0[PSI_HYX][pc];
            wyx = a ? v0 : 0.f; wzx = a ? v1 : 0.f; qyx = a ? v2 : 0.f; qzx = a ? v3 : 0.f;
            ayx = b ? v4 : 0.f; azx = b ? v5 : 0.f; bzx = a ? v6 : 0.f; cyx = a ? v7 : 0.f;
        }
        if (__any(Y.s >= 0 || Y.sm >= 0)) {
            const bool a = Y.s >= 0, b = Y.sm >= 0;
            py = a ? ys3(i, Y.s, k, ly, nz) : 0;
            const unsigned pm = b ? ys3(i, Y.sm, k, ly, nz) : 0;
            const unsigned pa = a && im ? py - (unsigned)ly * nz : 0, pc = a && km ? py - 1 : 0;
            const float v0 = P0[PSI_HXY][py], v1 = P0[PSI_HZY][py], v2 = P0[PSI_EXY][py], v3 = P0[PSI_EZY][py];
            const float v4 = P0[PSI_HXY][pm], v5 = P0[PSI_HZY][pm], v6 = P0[PSI_HZY][pa], v7 = P0[PSI_HXY][pc];
            wxy = a ? v0 : 0.f; wzy = a ? v1 : 0.f; qxy = a ? v2 : 0.f; qzy = a ? v3 : 0.f;
            bxy = b ? v4 : 0.f; bzy = b ? v5 : 0.f; azy = a ? v6 : 0.f; cxy = a ? v7 : 0.f;
        }
        if (__any(Z.s >= 0 || Z.sm >= 0)) {
            const bool a = Z.s >= 0, b = Z.sm >= 0;
            pz = a ? zs3(i, j, Z.s, ny, lz) : 0;
            const unsigned pm = b ? zs3(i, j, Z.sm, ny, lz) : 0;
            const unsigned pa = a && im ? pz - (unsigned)ny * lz : 0, pb = a && jm ? pz - lz : 0;
            const float v0 = P0[PSI_HXZ][pz], v1 = P0[PSI_HYZ][pz], v2 = P0[PSI_EXZ][pz], v3 = P0[PSI_EYZ][pz];
            const float v4 = P0[PSI_HXZ][pm], v5 = P0[PSI_HYZ][pm], v6 = P0[PSI_HYZ][pa], v7 = P0[PSI_HXZ][pb];
            wxz = a ? v0 : 0.f; wyz = a ? v1 : 0.f; qxz = a ? v2 : 0.f; qyz = a ? v3 : 0.f;
            cxz = b ? v4 : 0.f; cyz = b ? v5 : 0.f; ayz = a ? v6 : 0.f; bxz = a ? v7 : 0.f;
        }
    }

    // The update's roundings are those of the marching kernel: differences
    // along x and y with their psi, the z difference with the interior 1/dz
    // in one fused multiply-add, then the z slab's (1/(kappa dz) - 1/dz) d +
    // psi.
    const float idH = p.z.kH[p.z.lo], idE = p.z.kE[p.z.lo];
    const bool inx = PML && X.s >= 0, iny = PML && Y.s >= 0, inz = PML && Z.s >= 0;
    const bool inxm = PML && X.sm >= 0, inym = PML && Y.sm >= 0, inzm = PML && Z.sm >= 0;
    auto term = [](float k, float b, float c, float d, bool in, float &psi) {
        psi = in ? __builtin_fmaf(c, d, b * psi) : 0.f;
        return __builtin_fmaf(k, d, psi);
    };
    // Hx from its y and z differences, Hy from z and x, Hz from x and y
    auto hxOf = [&](float h, float db1, float ty, float dz, float kz, float bz, float cz, bool in, float &psi) {
        float r = __builtin_fmaf(-db1, __builtin_fmaf(-idH, dz, ty), h);
        psi = psi_next(bz, cz, dz, in, psi);
        return in ? __builtin_fmaf(db1, __builtin_fmaf(kz - idH, dz, psi), r) : r;
    };
    auto hyOf = [&](float h, float db1, float tx, float dz, float kz, float bz, float cz, bool in, float &psi) {
        float r = __builtin_fmaf(-db1, __builtin_fmaf(idH, dz, -tx), h);
        psi = psi_next(bz, cz, dz, in, psi);
        return in ? __builtin_fmaf(-db1, __builtin_fmaf(kz - idH, dz, psi), r) : r;
    };
    // ---- H layer: own cell (E beyond the last plane, row or cell is 0) ----
    const float dEzy = (yj ? ezb : 0.f) - ez, dEyz = (zk ? eyc : 0.f) - ey;
    const float dExz = (zk ? exc : 0.f) - ex, dEzx = (xi ? eza : 0.f) - ez;
    const float dEyx = (xi ? eya : 0.f) - ey, dExy = (yj ? exb : 0.f) - ex;
    const float nhx = hxOf(hx, db, term(Y.kH, Y.bH, Y.cH, dEzy, iny, wxy), dEyz, Z.kH, Z.bH, Z.cH, inz, wxz);
    const float nhy = hyOf(hy, db, term(X.kH, X.bH, X.cH, dEzx, inx, wyx), dExz, Z.kH, Z.bH, Z.cH, inz, wyz);
    const float nhz = __builtin_fmaf(-db, term(X.kH, X.bH, X.cH, dEyx, inx, wzx) -
                                          term(Y.kH, Y.bH, Y.cH, dExy, iny, wzy), hz);
    // ---- and of the cells below that the E layer gathers (0 beyond the
    // grid's first plane, row or cell) ----
    const float vhyA = hyOf(hyA, dbA, term(X.kHm, X.bHm, X.cHm, ez - ezA, inxm, ayx), (zk ? exAc : 0.f) - exA, Z.kH,
                            Z.bH, Z.cH, inz, ayz);
    const float vhzA = __builtin_fmaf(-dbA, term(X.kHm, X.bHm, X.cHm, ey - eyA, inxm, azx) -
                                            term(Y.kH, Y.bH, Y.cH, (yj ? exAb : 0.f) - exA, iny, azy), hzA);
    const float vhxB = hxOf(hxB, dbB, term(Y.kHm, Y.bHm, Y.cHm, ez - ezB, inym, bxy), (zk ? eyBc : 0.f) - eyB, Z.kH,
                            Z.bH, Z.cH, inz, bxz);
    const float vhzB = __builtin_fmaf(-dbB, term(X.kH, X.bH, X.cH, (xi ? eyBa : 0.f) - eyB, inx, bzx) -
                                            term(Y.kHm, Y.bHm, Y.cHm, ex - exB, inym, bzy), hzB);
    // Below a cell at which a wavefront of the marching kernel's default
    // starts, that kernel's roundings of the values it recomputes: in the
    // x and y slabs k d + psi in two; in a tile clear of them (rows in groups
    // of 8) the y difference in the fused multiply-add; psi of z as of x, y.
    // So the bits do not depend on which of the two kernels ran.
    const bool seam = (k & (64 * (nz % 4 == 0 ? 4 : nz % 2 == 0 ? 2 : 1) - 1)) == 0;
    bool clear = true;
    if (PML) {
        const int g = j & ~7;
        clear = (p.x.lo == 0 || i > p.x.lo) && i < nx - p.x.hi && (p.y.lo == 0 || g > p.y.lo) &&
                min(g + 8, ny) <= ny - p.y.hi;
    }
    const float dCy = (yj ? ezCb : 0.f) - ezC, dCx = (xi ? ezCa : 0.f) - ezC, dCyz = ey - eyC, dCxz = ex - exC;
    float tCy = term(Y.kH, Y.bH, Y.cH, dCy, iny, cxy), tCx = term(X.kH, X.bH, X.cH, dCx, inx, cyx);
    if (PML && seam) {
        if (iny) tCy = Y.kH * dCy + cxy;
        if (inx) tCx = X.kH * dCx + cyx;
    }
    float sC = __builtin_fmaf(-idH, dCyz, tCy);
    if (seam && clear) sC = __builtin_fmaf(Y.kH, dCy, -(idH * dCyz));
    float vhxC = __builtin_fmaf(-dbC, sC, hxC), vhyC = __builtin_fmaf(-dbC, __builtin_fmaf(idH, dCxz, -tCx), hyC);
    if (inzm) {
        const float kz = Z.kHm - idH;
        const float vxz = seam ? __builtin_fmaf(Z.cHm, dCyz, Z.bHm * cxz) : psi_next(Z.bHm, Z.cHm, dCyz, true, cxz);
        const float vyz = seam ? __builtin_fmaf(Z.cHm, dCxz, Z.bHm * cyz) : psi_next(Z.bHm, Z.cHm, dCxz, true, cyz);
        vhxC = __builtin_fmaf(dbC, __builtin_fmaf(kz, dCyz, vxz), vhxC);
        vhyC = __builtin_fmaf(-dbC, __builtin_fmaf(kz, dCxz, vyz), vhyC);
    }
    const float nhyA = im ? vhyA : 0.f, nhzA = im ? vhzA : 0.f, nhxB = jm ? vhxB : 0.f, nhzB = jm ? vhzB : 0.f;
    const float nhxC = km ? vhxC : 0.f, nhyC = km ? vhyC : 0.f;

    // ---- E layer (tangential E on the low walls stays; so does its psi) ----
    float nex = ex, ney = ey, nez = ez;
    auto eOf = [&](float e, float t) { return MAT >= 1 ? __builtin_fmaf(ca, e, cb * t) : __builtin_fmaf(cb, t, e); };
    if (jm && km) {
        const float dz = nhy - nhyC, ty = term(Y.kE, Y.bE, Y.cE, nhz - nhzB, iny, qxy);
        nex = eOf(ex, __builtin_fmaf(-idE, dz, ty));
        qxz = psi_next(Z.bE, Z.cE, dz, inz, qxz);
        if (inz) nex = __builtin_fmaf(-cb, __builtin_fmaf(Z.kE - idE, dz, qxz), nex);
    }
    if (im && km) {
        const float dz = nhx - nhxC, tx = term(X.kE, X.bE, X.cE, nhz - nhzA, inx, qyx);
        ney = eOf(ey, __builtin_fmaf(idE, dz, -tx));
        qyz = psi_next(Z.bE, Z.cE, dz, inz, qyz);
        if (inz) ney = __builtin_fmaf(cb, __builtin_fmaf(Z.kE - idE, dz, qyz), ney);
    }
    if (im && jm)
        nez = eOf(ez, term(X.kE, X.bE, X.cE, nhy - nhyA, inx, qzx) - term(Y.kE, Y.bE, Y.cE, nhx - nhxB, iny, qzy));
    if (p.src_idx >= 0 && step < p.src_len && in_src(p.src_box, i, j, k)) {
        const float sval = p.src_vals[step];
        if (p.src_comp == FDTD_EX) nex += sval;
        else if (p.src_comp == FDTD_EY) ney += sval;
        else nez += sval;
    }
    if (ok) {
        p.s1.f[FDTD_EX][c] = nex;
        p.s1.f[FDTD_EY][c] = ney;
        p.s1.f[FDTD_EZ][c] = nez;
        p.s1.f[FDTD_HX][c] = nhx;
        p.s1.f[FDTD_HY][c] = nhy;
        p.s1.f[FDTD_HZ][c] = nhz;
        if (PML) {
            float *const *P1 = p.s1.psi;
            if (X.s >= 0) {
                P1[PSI_HYX][px] = wyx; P1[PSI_HZX][px] = wzx; P1[PSI_EYX][px] = qyx; P1[PSI_EZX][px] = qzx;
            }
            if (Y.s >= 0) {
                P1[PSI_HXY][py] = wxy; P1[PSI_HZY][py] = wzy; P1[PSI_EXY][py] = qxy; P1[PSI_EZY][py] = qzy;
            }
            if (Z.s >= 0) {
                P1[PSI_HXZ][pz] = wxz; P1[PSI_HYZ][pz] = wyz; P1[PSI_EXZ][pz] = qxz; P1[PSI_EYZ][pz] = qyz;
            }
        }
    }
    // probes of the block's cells
    if (pt.start != nullptr)
        for (int q = pt.start[blk]; q < pt.start[blk + 1]; ++q) {
            if (pt.cell[q] != c || !ok) continue;
            float v;
            switch (p.probe_comp) {
                case FDTD_EX: v = nex; break;
                case FDTD_EY: v = ney; break;
                case FDTD_EZ: v = nez; break;
                case FDTD_HX: v = nhx; break;
                case FDTD_HY: v = nhy; break;
                default: v = nhz; break;
            }
            p.rec[(int64_t)pt.slot[q] * p.rec_stride + (step - p.rec_base)] = v;
        }
}

hipError_t launch_3d_flat(const Prob3D &p, const ProbeTiles &pt, int64_t step, int part, hipStream_t st) {
    const int64_t n = (int64_t)p.nx * p.ny * p.nz;
    if (n >= ((int64_t)1 << 31) - 4096) return hipErrorInvalidValue;
    const unsigned nb = (unsigned)(((n + 255) / 256 + 7) / 8 * 8);
    const Div dp = make_div((unsigned)p.ny * p.nz), dr = make_div((unsigned)p.nz);
    const bool pml = p.x.lo + p.x.hi + p.y.lo + p.y.hi + p.z.lo + p.z.hi > 0;
    const int mat = p.db ? 2 : (p.ca ? 1 : 0);
#define GEM_F(MA)                                                                                          \
    do {                                                                                                   \
        if (pml) hipLaunchKernelGGL((k3d_flat<MA, true>), dim3(nb), dim3(256), 0, st, p, dp, dr, pt, step, part); \
        else hipLaunchKernelGGL((k3d_flat<MA, false>), dim3(nb), dim3(256), 0, st, p, dp, dr, pt, step, part);   \
    } while (0)
    if (mat == 0) GEM_F(0);
    else if (mat == 1) GEM_F(1);
    else GEM_F(2);
#undef GEM_F
    return hipGetLastError();
}

}  // namespace gem
