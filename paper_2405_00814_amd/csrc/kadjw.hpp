// Discrete adjoint of the 2D TMz step: several backward steps per pass, one
// workgroup per tile, the adjoint state in registers (device code;
// instantiated in kadjw*.hip).
//
// The tiles, their halo of one cell per step and their exchange are those of
// the forward pass (k2dw.hpp).  A backward step of a cell:
//   A  u = Cb a (a: adjoint Ez); messages gy = u kEx + cEx px, gx = -u kEy +
//      cEy py with px = u + psi_Ex, py = -u + psi_Ey, psi <- b p; the design
//      sums gain a Ez and a bracket; a <- Ca a
//   B  hy += gy(i) - gy(i+1), hx += gx(j) - gx(j+1); wy = Db hy + psi_Hx,
//      wx = -Db hx + psi_Hy, psi <- b w; ex = Db hy kHx + cHx wy, ey = -Db hx
//      kHy + cHy wx
//   C  a += ey(j-1) - ey(j) + ex(i-1) - ex(i), then the probe-loss seed
// in one sweep over a thread's rows, each row's A one row ahead of its B and
// C.  Across wavefronts only a is exchanged: a wavefront recomputes the
// message gy of the row below its last one and, with its own copies of Hy,
// psi and Db, ex of the row above its first.
//
// Bound by latency at few wavefronts: 176 registers leave a CU one workgroup
// of eight wavefronts, and 1024^2 with CPML makes 536 of them, two full
// rounds of the 256 CUs and a third of 24 (counters: VALU busy 0.33 of the
// launch, 4.2 wavefronts resident per CU, 0.39 of their time waiting).
// Measured beside the recompute's launches there, 256^2 design cells: 7.2 us per
// step in passes of 8 (13.2 with one step per launch, k_adj_fused); 16
// wavefronts of 4 rows instead of 8 of 8 were 8 % faster there and 4 %
// slower at 2048^2.
//
// Every sum of a design cell is held in registers for the pass and gains one
// product per step, in the order of the steps: neither the tiles nor the
// grouping of steps into passes change its bits.
#pragma once

#include "k2dw.hpp"

namespace gem {

template <int W, int R>
struct AwShared {
    float e[2][W][2][64];  // adjoint Ez of each wavefront's first and last row
    RowTab x[W * R + 2];   // x-axis tables of rows a - 1 .. a + W R
};

// EDGE, PX, PY as in wg_tile; MU: sums for the mu_r gradient too.
template <int R, int W, int MAT, bool EDGE, bool PX, bool PY, bool MU, class SH>
__device__ __forceinline__ void adj_tile(const Prob2D &p, const TileW &T, const AdjWArgs &A, int tile, SH &sh) {
#pragma clang fp contract(off)
    const int lane = (int)(threadIdx.x & 63);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nx = p.nx, ny = p.ny;
    const int ib = T.a + w * R, j = T.c + lane;
    const bool colin = !EDGE || j < ny;
    const int jc = EDGE ? min(j, ny - 1) : j;
    const bool colup = !EDGE || (j >= 1 && j < ny);
    const float db0 = p.db0;
    const float kHy = PY ? p.y.kH[jc] : p.y.kH[p.y.lo], kEy = PY ? p.y.kE[jc] : p.y.kE[p.y.lo];
    const float kHx0 = p.x.kH[p.x.lo], kEx0 = p.x.kE[p.x.lo];
    const int syw = p.y.lo + p.y.hi;
    int jj = -1;
    float bHy = 0.f, cHy = 0.f, bEy = 0.f, cEy = 0.f;
    if constexpr (PY) {
        jj = colin ? slab_index(p.y, jc) : -1;
        if (jj >= 0) {
            bHy = p.y.bH[jc]; cHy = p.y.cH[jc];
            bEy = p.y.bE[jc]; cEy = p.y.cE[jc];
        }
    }
    if constexpr (PX) {
        for (int q = (int)threadIdx.x; q < W * R + 2; q += 64 * W) {
            const int i = T.a - 1 + q;
            RowTab t{make_float4(kHx0, 0.f, 0.f, 0.f), make_float4(kEx0, 0.f, 0.f, 0.f)};
            if (i >= 0 && i < nx) {
                const bool in = slab_index(p.x, i) >= 0;
                t.h = make_float4(p.x.kH[i], in ? p.x.bH[i] : 0.f, in ? p.x.cH[i] : 0.f, 0.f);
                t.e = make_float4(p.x.kE[i], in ? p.x.bE[i] : 0.f, in ? p.x.cE[i] : 0.f, 0.f);
            }
            sh.x[q] = t;
        }
    }

    float ez[R], hx[R], hy[R], cb[R];
    float ca[MAT >= 1 ? R : 1], db[MAT == 2 ? R : 1];
    float phx[PY ? R : 1], pzy[PY ? R : 1], phy[PX ? R : 1], pzx[PX ? R : 1];
    const int64_t first = (int64_t)T.a * ny, len = (int64_t)nx * ny;
    const int rb = ny * 4, vo = jc * 4;
    const Buf bez(A.l0.ez, first, len), bhx(A.l0.hx, first, len), bhy(A.l0.hy, first, len), bcb(p.cb, first, len);
    const Buf bca(MAT >= 1 && p.ca ? p.ca : p.cb, first, len), bdb(MAT == 2 && p.db ? p.db : p.cb, first, len);
    rows<R>([&](auto rc) GEM_INL {
        constexpr int r = decltype(rc)::value;
        const int i = ib + r;
        const bool in = (!EDGE || i < nx) && colin;
        const int so = ((EDGE ? min(i, nx - 1) : i) - T.a) * rb;
        const float e = bez.ld(vo, so), x = bhx.ld(vo, so), y = bhy.ld(vo, so), b = bcb.ld(vo, so);
        ez[r] = in ? e : 0.f;
        hx[r] = in ? x : 0.f;
        hy[r] = in ? y : 0.f;
        const bool upd = in && colup && (!EDGE || i >= 1);
        cb[r] = upd ? b : 0.f;  // no messages from the walls
        if constexpr (MAT >= 1) {
            ca[r] = 1.f;
            if (p.ca) { const float c = bca.ld(vo, so); ca[r] = upd ? c : 1.f; }
        }
        if constexpr (MAT == 2) {
            db[r] = db0;
            if (p.db) db[r] = bdb.ld(vo, so);
        }
    });
    if constexpr (PY) {
        const int vy = max(jj, 0) * 4, sb = syw * 4;
        const int64_t f0 = (int64_t)T.a * syw, l0 = (int64_t)nx * syw;
        const Buf phxb(A.l0.psi_hx, f0, l0), pzyb(A.l0.psi_ezy, f0, l0);
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const int so = (min(ib + r, nx - 1) - T.a) * sb;
            const float x = phxb.ld(vy, so), y = pzyb.ld(vy, so);
            const bool in = jj >= 0 && ib + r < nx;
            phx[r] = in ? x : 0.f;
            pzy[r] = in ? y : 0.f;
        });
    }
    const int64_t lx = (int64_t)(p.x.lo + p.x.hi) * ny;
    auto xslab = [&](const float *f, int i) GEM_INL {  // x-slab psi of row i
        const int ii = i >= 0 && i < nx ? slab_index(p.x, i) : -1;
        float v = 0.f;
        if (ii >= 0 && colin) v = Buf(f, 0, lx).ld(vo, ii * rb);
        return v;
    };
    if constexpr (PX)
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            phy[r] = xslab(A.l0.psi_hy, ib + r);
            pzx[r] = xslab(A.l0.psi_ezx, ib + r);
        });
    // the row above the wavefront's first (w > 0) and the one below its last
    float hyp = 0.f, cbp = 0.f, php = 0.f, pzp = 0.f, dbp = db0, cbn = 0.f, pzn = 0.f;
    if (w > 0 && (!EDGE || ib - 1 < nx)) {
        const int so = (ib - 1 - T.a) * rb;
        const float y = bhy.ld(vo, so), b = bcb.ld(vo, so);
        hyp = colin ? y : 0.f;
        cbp = colup && (!EDGE || ib - 1 >= 1) ? b : 0.f;
        if constexpr (MAT == 2) {
            if (p.db) dbp = bdb.ld(vo, so);
        }
        if constexpr (PX) {
            php = xslab(A.l0.psi_hy, ib - 1);
            pzp = xslab(A.l0.psi_ezx, ib - 1);
        }
    }
    if (w < W - 1 && (!EDGE || ib + R < nx)) {
        const float b = bcb.ld(vo, (ib + R - T.a) * rb);
        cbn = colup ? b : 0.f;
        if constexpr (PX) pzn = xslab(A.l0.psi_ezx, ib + R);
    }

    // design cells of this wavefront's own rows and columns: their sums, and
    // the captured values of the box around them
    const int4 D = A.design, C = A.cbox;
    const bool ownj = j >= T.j0 && j < T.j1;
    const bool gw = D.x < min(ib + R, T.i1) && D.y > max(ib, T.i0) && D.z < T.j1 && D.w > T.j0;
    const bool gj = gw && ownj && j >= D.z && j < D.w;
    const int dw = D.w - D.z, cw = C.w - C.z;
    double sez[R], sbr[R], shx[MU ? R : 1], shy[MU ? R : 1];
    auto each_design = [&](auto f) GEM_INL {
        const int i0 = opaque(ib);
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            const int i = i0 + r;
            if (gj && i >= T.i0 && i < T.i1 && i >= D.x && i < D.y) f(rc, (int64_t)(i - D.x) * dw + (j - D.z));
        });
    };
    rows<R>([&](auto rc) GEM_INL {
        constexpr int r = decltype(rc)::value;
        sez[r] = sbr[r] = 0.0;
        if constexpr (MU) shx[r] = shy[r] = 0.0;
    });
    if (gw)
        each_design([&](auto rc, int64_t q) GEM_INL {
            constexpr int r = decltype(rc)::value;
            sez[r] = A.sez[q];
            sbr[r] = A.sbr[q];
            if constexpr (MU) { shx[r] = A.shx[q]; shy[r] = A.shy[q]; }
        });

    // seeds of the tile's loaded cells (halo included); the first cached
    const int pbeg = load_const(A.pt.start + tile), pend = load_const(A.pt.start + tile + 1);
    int np = 0, pq = pend;
    for (int q = pbeg; q < pend; ++q) {
        const int pi = load_const(A.pt.cell + q) / ny;
        if (pi < ib || pi >= ib + R) continue;
        if (np == 0) pq = q;
        ++np;
    }

    sh.e[0][w][0][lane] = ez[0];
    sh.e[0][w][1][lane] = ez[R - 1];
    __syncthreads();

    const int nsteps = A.nsteps;
    for (int s = 0; s < nsteps; ++s) {
        const int64_t k = A.k - s;  // the step being transposed
        const float up = w > 0 ? sh.e[s & 1][w > 0 ? w - 1 : 0][1][lane] : 0.f;
        const float dn = w < W - 1 ? sh.e[s & 1][w < W - 1 ? w + 1 : w][0][lane] : 0.f;
        // captured values of this step, in flight while the rows compute
        float ce[R + 1], cr[R];
        if (gw) {
            const int i0 = opaque(ib);
            const float *pe = A.cap_ez + (k - A.k0) * A.nd, *pr = A.cap_br + (k - A.k0) * A.nd;
            const bool cj = j >= C.z && j < C.w;
            rows<R + 1>([&](auto rc) GEM_INL {
                constexpr int r = decltype(rc)::value;
                const int i = i0 + r;
                const bool in = cj && i >= C.x && i < C.y;
                const int64_t q = in ? (int64_t)(i - C.x) * cw + (j - C.z) : 0;
                if constexpr (MU || r < R) {
                    const float e = pe[q];
                    ce[r] = in ? e : 0.f;
                }
                if constexpr (r < R) cr[r] = pr[q];
            });
        }
        // A of one row: messages from a with Cb cbv (psi updated)
        auto phaseA = [&](float a, float cbv, int q, float &px, float &py, float &gx, float &gy) GEM_INL {
            const float u = cbv * a;
            float kE = kEx0, bE = 0.f, cE = 0.f;
            if constexpr (PX) { const float4 t = sh.x[q].e; kE = t.x; bE = t.y; cE = t.z; }
            gy = u * kE;
            gx = -(u * kEy);
            if constexpr (PX) {
                const float v = u + px;
                px = bE * v;
                gy = __builtin_fmaf(cE, v, gy);
            }
            if constexpr (PY) {
                const float v = py - u;
                py = bEy * v;
                gx = __builtin_fmaf(cEy, v, gx);
            }
        };
        // ex of a row from its updated Hy
        auto exOf = [&](float h, float dbv, int q, float &ps) GEM_INL {
            float kH = kHx0, bH = 0.f, cH = 0.f;
            if constexpr (PX) { const float4 t = sh.x[q].h; kH = t.x; bH = t.y; cH = t.z; }
            const float w0 = dbv * h;
            float ex = w0 * kH;
            if constexpr (PX) {
                const float v = w0 + ps;
                ps = bH * v;
                ex = __builtin_fmaf(cH, v, ex);
            }
            return ex;
        };
        float dump = 0.f, gxd, gyp, gxc, gyc, gyn;
        phaseA(up, cbp, w * R, pzp, dump, gxd, gyp);
        dump = 0.f;
        phaseA(dn, cbn, w * R + R + 1, pzn, dump, gxd, gyn);
        const float a0 = ez[0];
        phaseA(a0, cb[0], w * R + 1, pzx[0], pzy[0], gxc, gyc);
        hyp = (hyp + gyp) - gyc;
        float exp_ = exOf(hyp, MAT == 2 ? dbp : db0, w * R, php);
        float acur = a0;
        rows<R>([&](auto rc) GEM_INL {
            constexpr int r = decltype(rc)::value;
            constexpr int rn = r + 1 < R ? r + 1 : r;
            float gxn = 0.f, gy1 = gyn, anext = 0.f;
            if constexpr (r + 1 < R) {
                anext = ez[rn];
                phaseA(anext, cb[rn], w * R + 1 + rn, pzx[PX ? rn : 0], pzy[PY ? rn : 0], gxn, gy1);
            }
            const float gxr = lane_next0(gxc);
            hx[r] = (hx[r] + gxc) - gxr;
            hy[r] = (hy[r] + gyc) - gy1;
            const float dbv = MAT == 2 ? db[MAT == 2 ? r : 0] : db0;
            const float w0 = -(dbv * hx[r]);
            float ey = w0 * kHy;
            if constexpr (PY) {
                const float v = w0 + phx[r];
                phx[r] = bHy * v;
                ey = __builtin_fmaf(cHy, v, ey);
            }
            const float ex = exOf(hy[r], dbv, w * R + 1 + r, phy[PX ? r : 0]);
            const float eyl = lane_prev0(ey);
            const float e = MAT >= 1 ? acur * ca[MAT >= 1 ? r : 0] : acur;
            ez[r] = ((e - ey) - ex + eyl) + exp_;
            if (gw) {
                sez[r] += (double)acur * (double)ce[r];
                sbr[r] += (double)acur * (double)cr[r];
                if constexpr (MU) {
                    const float ey1 = lane_next0(ce[r]);
                    shx[r] += (double)hx[r] * (double)((ey1 - ce[r]) * kHy);
                    shy[r] += (double)hy[r] * (double)((ce[r + 1] - ce[r]) * kHx0);
                }
            }
            exp_ = ex;
            gxc = gxn;
            gyc = gy1;
            acur = anext;
        });
        // probe-loss seed of step k - 1
        if (np > 0 && k > A.n0 && k <= A.n1) {
            int left = np;
            for (int q = pq; left > 0; ++q) {
                const int cell = load_const(A.pt.cell + q), pi = cell / ny, pj = cell - pi * ny;
                if (pi < ib || pi >= ib + R) continue;
                --left;
                const float add = 2.f * load_const(A.rec + (int64_t)load_const(A.pt.slot + q) * A.rec_stride + (k - 1));
                const int rr = opaque(pi - ib);
                const bool mine = lane == pj - T.c;
                rows<R>([&](auto rc) GEM_INL {
                    constexpr int r = decltype(rc)::value;
                    if (r == rr && mine) ez[r] += add;
                });
            }
        }
        sh.e[(s + 1) & 1][w][0][lane] = ez[0];
        sh.e[(s + 1) & 1][w][1][lane] = ez[R - 1];
        __syncthreads();
    }

    {
        const int i3 = opaque(ib), so3 = opaque(rb), vs = j * 4;
        const Buf oez(A.l1.ez, first, len), ohx(A.l1.hx, first, len), ohy(A.l1.hy, first, len);
        if (ownj)
            rows<R>([&](auto rc) GEM_INL {
                constexpr int r = decltype(rc)::value;
                const int i = i3 + r, so = (i - T.a) * so3;
                if (i < T.i0 || i >= T.i1) return;
                oez.st(ez[r], vs, so);
                ohx.st(hx[r], vs, so);
                ohy.st(hy[r], vs, so);
            });
        if constexpr (PX || PY) {
            const int vy = max(jj, 0) * 4, sb = opaque(syw * 4);
            const int64_t f0 = (int64_t)T.a * syw, l0 = (int64_t)nx * syw;
            const Buf phxb(A.l1.psi_hx, f0, l0), pzyb(A.l1.psi_ezy, f0, l0);
            const Buf phyb(A.l1.psi_hy, 0, lx), pzxb(A.l1.psi_ezx, 0, lx);
            if (ownj)
                rows<R>([&](auto rc) GEM_INL {
                    constexpr int r = decltype(rc)::value;
                    const int i = i3 + r;
                    if (i < T.i0 || i >= T.i1) return;
                    if (PY && jj >= 0) {
                        phxb.st(phx[PY ? r : 0], vy, (i - T.a) * sb);
                        pzyb.st(pzy[PY ? r : 0], vy, (i - T.a) * sb);
                    }
                    const int ii = PX ? slab_index(p.x, i) : -1;
                    if (ii >= 0) {
                        phyb.st(phy[PX ? r : 0], vs, ii * so3);
                        pzxb.st(pzx[PX ? r : 0], vs, ii * so3);
                    }
                });
        }
    }
    if (gw)
        each_design([&](auto rc, int64_t q) GEM_INL {
            constexpr int r = decltype(rc)::value;
            A.sez[q] = sez[r];
            A.sbr[q] = sbr[r];
            if constexpr (MU) { A.shx[q] = shx[r]; A.shy[q] = shy[r]; }
        });
}

template <int R, int W, int MW, int MAT, bool MU>
__global__ __launch_bounds__(64 * W, MW) void k_adj_wg(AdjWArgs A) {
    __shared__ AwShared<W, R> sh;
    const int tile = xcd_block((int)blockIdx.x, (int)gridDim.x);
    if (tile >= A.ntiles) return;  // whole workgroup
    const TileW T = load_const(A.tiles + tile);
    const Prob2D p = A.p;
    if (T.kind == 0) adj_tile<R, W, MAT, false, false, false, MU>(p, T, A, tile, sh);
    else if (T.kind == 1) adj_tile<R, W, MAT, true, false, false, MU>(p, T, A, tile, sh);
    else if (T.kind == 2) adj_tile<R, W, MAT, true, false, true, MU>(p, T, A, tile, sh);
    else if (T.kind == 3) adj_tile<R, W, MAT, true, true, false, MU>(p, T, A, tile, sh);
    else adj_tile<R, W, MAT, true, true, true, MU>(p, T, A, tile, sh);
}

// MW, MWU: wavefronts per SIMD the registers must allow, without and with
// the mu_r sums.
template <int R, int W, int MW, int MWU>
static hipError_t adj_go(const AdjWArgs &a, int mat, hipStream_t st) {
    const dim3 g((unsigned)((a.ntiles + 7) / 8 * 8)), b(64 * W);
#define GEM_A(MA)                                                                      \
    do {                                                                               \
        if (a.shx) hipLaunchKernelGGL((k_adj_wg<R, W, MWU, MA, true>), g, b, 0, st, a); \
        else hipLaunchKernelGGL((k_adj_wg<R, W, MW, MA, false>), g, b, 0, st, a);      \
    } while (0)
    if (mat == 0) GEM_A(0);
    else if (mat == 1) GEM_A(1);
    else GEM_A(2);
#undef GEM_A
    return hipGetLastError();
}

}  // namespace gem
