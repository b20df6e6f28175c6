// 3D fused phi + mu step: xy tiles that walk z, neighbours exchanged through LDS.
//
// A block owns a BX (x) by BY (y) tile, one thread per column, and walks a
// segment of z planes.  Each staged cell also stores its scaled mobility M~ so
// that faces never recompute h of a neighbour.  The z face between planes m and
// m+1 stays in registers (its W, J) and becomes the lower face of plane m+1;
// in-plane faces are evaluated by both of their cells with identical code and
// inputs.  Blocks are dealt XCD-aware so that a band of tiles shares one XCD's
// L2.  What the planes keep in LDS sets how many blocks a CU holds, and both
// forms below need all they can get: the kernel is bound by the latency of the
// march (a barrier per plane), not by one unit.
//
// Isotropic faces see only the two cells they separate, so a plane's neighbours
// are read in that plane alone: two slots alternate (the plane being computed,
// the next one being filled), and the cell above, the z face's other side, is
// the thread's own and stays in registers.
//
// Anisotropic faces also see the tangential differences of phi on the planes
// above and below: phi keeps a ring of four planes (m-1, m, m+1 and the one
// being filled), mu and M~ a ring of three (m, m+1 and the one being filled).
#pragma once

#include "diag_cell.hpp"
#include "gp_device.hpp"

namespace mp {

// Tile of a block and what its threads stage: position 0 is the thread's own
// cell, the others lie on the halo ring (CORNERS: with its corners, which only
// tangential differences read).
template <int BX, int BY, bool CORNERS>
struct Tile3d {
    static constexpr int PW = BX + 2;
    static constexpr int PP = PW * (BY + 2);
    static constexpr int NT = BX * BY;
    static constexpr int ROW = CORNERS ? PW : BX;  // cells of the rows above and below
    static constexpr int NHALO = 2 * ROW + 2 * BY;
    static constexpr int NPOS = 1 + (NHALO + NT - 1) / NT;

    int x0, y0, m0, m1;
    int64_t off[NPOS];  // in-plane element offset of each staged cell
    int pos[NPOS];      // its LDS position
    int tid;

    __device__ __forceinline__ bool has(int k) const { return k == 0 || tid + (k - 1) * NT < NHALO; }

    __device__ __forceinline__ void init(const Geom& g, int seg, int ntx, int nty) {
        const int nb = gridDim.x;
        const int q8 = nb / 8;
        const int b = blockIdx.x;
        const int tile = (b < 8 * q8) ? (b % 8) * q8 + b / 8 : b;
        const int rest = tile / ntx;
        x0 = (tile % ntx) * BX;
        y0 = (rest % nty) * BY;
        m0 = (rest / nty) * seg;
        m1 = min(m0 + seg, g.nz);
        tid = threadIdx.x;
        const bool perx = g.bcx == MP_BC_PERIODIC;
        const bool pery = g.bcy == MP_BC_PERIODIC;
#pragma unroll
        for (int k = 0; k < NPOS; ++k) {
            int ix = 1 + tid % BX, iy = 1 + tid / BX;
            if (k > 0) {
                const int q = tid + (k - 1) * NT;
                if (q < 2 * ROW) {
                    iy = q < ROW ? 0 : BY + 1;
                    ix = (q < ROW ? q : q - ROW) + (CORNERS ? 0 : 1);
                } else {
                    const int w = min(q - 2 * ROW, 2 * BY - 1);
                    iy = 1 + (w >> 1);
                    ix = (w & 1) * (PW - 1);
                }
            }
            pos[k] = iy * PW + ix;
            off[k] = gmap(x0 - 1 + ix, g.nx, perx) + gmap(y0 - 1 + iy, g.ny, pery) * (int64_t)g.nx;
        }
    }
};

// New values of a column's cell written at out + o (and added to the diagnostics).
template <typename R, int NP, int NM, bool GEN, bool DIAG, bool NT>
__device__ __forceinline__ void store3d(R* __restrict__ out, const Geom& g, int64_t o, const R (&phin)[NP],
                                        const R (&mun)[NM], int gy, DiagAcc* da, const DiagCoef* dc) {
    store_cell<R, NP, NM, NT>(out, g.fstride, o, phin, mun);
    if constexpr (DIAG) {
        double p[NP], u[NM];
#pragma unroll
        for (int a = 0; a < NP; ++a) p[a] = (double)phin[a];
#pragma unroll
        for (int k = 0; k < NM; ++k) u[k] = (double)mun[k];
        diag_cell<NP, NM, GEN>(p, u, dc->tt0 + dc->tslope * (double)gy, *dc, *da);
    }
}

// The isotropic step of one block (GEN: the extended model's arithmetic, x its terms).
template <typename R, int NP, int NM, bool OBST, int BX, int BY, bool GEN, bool DIAG, bool NT>
__device__ __forceinline__ void step3d_iso(const R* __restrict__ in, R* __restrict__ out, const Geom& g,
                                           const Coef<R>& c, const int64_t* __restrict__ stepctr, int kstep,
                                           double tb0, double tdn, double tslope, int seg, int ntx, int nty,
                                           const CoefX<R>* x, DiagAcc* da, const DiagCoef* dc) {
    constexpr int NF = NP + NM;
    constexpr int NMM = mob_n<NM, GEN>();
    typedef Tile3d<BX, BY, false> Tile;
    constexpr int PW = Tile::PW, PP = Tile::PP, NPOS = Tile::NPOS;
    __shared__ R sv[2][NF][PP];
    __shared__ R sm[2][NMM][PP];
    Tile t;
    t.init(g, seg, ntx, nty);
    const bool perz = g.bcz == MP_BC_PERIODIC;
    const int64_t sz = (int64_t)g.nx * g.ny;
    const int64_t fs = g.fstride;

    // the thread's own cell of one plane
    struct Cell {
        R phi[NP], mu[NM], h[NP], Mt[NMM];
    };
    R reg[NPOS][NF];
    auto fetch = [&](int m) {
        const R* p = in + (int64_t)gmap(m, g.nz, perz) * sz;
#pragma unroll
        for (int k = 0; k < NPOS; ++k)
            if (t.has(k)) {
#pragma unroll
                for (int f = 0; f < NF; ++f) reg[k][f] = p[f * fs + t.off[k]];
            }
    };
    auto own = [&](Cell& C) {
#pragma unroll
        for (int a = 0; a < NP; ++a) C.phi[a] = moved(reg[0][a]);
#pragma unroll
        for (int k = 0; k < NM; ++k) C.mu[k] = moved(reg[0][NP + k]);
        interp_h<R, NP>(C.phi, C.h);
        mobility_any<R, NP, NM, GEN>(C.h, c, x, C.Mt);
    };
    auto stage = [&](int m, const Cell& C) {
        const int sl = m & 1;
#pragma unroll
        for (int k = 0; k < NPOS; ++k)
            if (t.has(k)) {
                R Mt[NMM];
                if (k == 0) {
#pragma unroll
                    for (int kk = 0; kk < NMM; ++kk) Mt[kk] = C.Mt[kk];
                } else {
                    R ph[NP], hh[NP];
#pragma unroll
                    for (int a = 0; a < NP; ++a) ph[a] = reg[k][a];
                    interp_h<R, NP>(ph, hh);
                    mobility_any<R, NP, NM, GEN>(hh, c, x, Mt);
                }
#pragma unroll
                for (int f = 0; f < NF; ++f) sv[sl][f][t.pos[k]] = reg[k][f];
#pragma unroll
                for (int kk = 0; kk < NMM; ++kk) sm[sl][kk][t.pos[k]] = Mt[kk];
            }
    };
    const R tau[1][NP] = {};
    // face between the cell C and its in-plane neighbour at LDS position p
    auto face = [&](int sl, const Cell& C, int p, bool below, R(&U)[NP], R(&W)[NP], R(&J)[NM]) {
        R pn[NP], un[NM], mn[NMM];
#pragma unroll
        for (int a = 0; a < NP; ++a) pn[a] = sv[sl][a][p];
#pragma unroll
        for (int k = 0; k < NM; ++k) un[k] = sv[sl][NP + k][p];
#pragma unroll
        for (int k = 0; k < NMM; ++k) mn[k] = sm[sl][k][p];
        if (below)
            face_core<R, NP, NM, false, 0, GEN>(pn, C.phi, tau, mn, C.Mt, un, C.mu, c, U, W, J);
        else
            face_core<R, NP, NM, false, 0, GEN>(C.phi, pn, tau, C.Mt, mn, C.mu, un, c, U, W, J);
    };

    const int gx = t.x0 + t.tid % BX;
    const int gy = t.y0 + t.tid / BX;
    const bool valid = gx < g.nx && gy < g.ny;
    const int64_t o0 = (int64_t)gx + (int64_t)gy * g.nx;
    const int pc = t.pos[0];
    const double tbase = tb0 + tdn * (double)(*stepctr + kstep);
    R Cs[NP];  // T - Te depends on y only
    const R tt = (R)(tbase + tslope * (double)gy);
    psi_const_any<R, NP, GEN>(tt, c, x, Cs);

    Cell A, B;
    R Wlo[NP], Jlo[NM];  // z face between planes m-1 and m
    fetch(t.m0 - 1);
    own(B);
    fetch(t.m0);
    own(A);
    stage(t.m0, A);
    fetch(t.m0 + 1);
    {
        R Ud[NP];
        face_core<R, NP, NM, false, 0, GEN>(B.phi, A.phi, tau, B.Mt, A.Mt, B.mu, A.mu, c, Ud, Wlo, Jlo);
    }
    own(B);
    __syncthreads();

    // Plane m with its own cells in C and plane m+1's in N; leaves plane m+2's
    // in C.  A wait for loads waits for the stores before them as well (they are
    // jumped over in a wave outside the grid, so no count of them can be left
    // out): the plane's loads are issued at its start and waited for before its
    // stores, so that either has a plane's arithmetic to complete in.
    auto plane = [&](int m, Cell& C, Cell& N) {
        if (m + 1 < t.m1) stage(m + 1, N);
        if (m + 2 <= t.m1) fetch(m + 2);
        const int sl = m & 1;
        R Gs[NP], Js[NM];
        {
            R Ul[NP], Wl[NP], Jl[NM], Uh[NP], Wh[NP], Jh[NM];
            face(sl, C, pc - 1, true, Ul, Wl, Jl);
            face(sl, C, pc + 1, false, Uh, Wh, Jh);
#pragma unroll
            for (int a = 0; a < NP; ++a) Gs[a] = Uh[a] - Wl[a];
#pragma unroll
            for (int k = 0; k < NM; ++k) Js[k] = Jh[k] - Jl[k];
        }
        {
            R Ul[NP], Wl[NP], Jl[NM], Uh[NP], Wh[NP], Jh[NM];
            face(sl, C, pc - PW, true, Ul, Wl, Jl);
            face(sl, C, pc + PW, false, Uh, Wh, Jh);
#pragma unroll
            for (int a = 0; a < NP; ++a) Gs[a] = Gs[a] + (Uh[a] - Wl[a]);
#pragma unroll
            for (int k = 0; k < NM; ++k) Js[k] = Js[k] + (Jh[k] - Jl[k]);
        }
        {
            R Uh[NP], Wh[NP], Jh[NM];
            face_core<R, NP, NM, false, 0, GEN>(C.phi, N.phi, tau, C.Mt, N.Mt, C.mu, N.mu, c, Uh, Wh, Jh);
#pragma unroll
            for (int a = 0; a < NP; ++a) {
                Gs[a] = Gs[a] + (Uh[a] - Wlo[a]);
                Wlo[a] = Wh[a];
            }
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                Js[k] = Js[k] + (Jh[k] - Jlo[k]);
                Jlo[k] = Jh[k];
            }
        }
        R phin[NP], mun[NM], h1[NP];
        cell_update_any<R, NP, NM, OBST, GEN>(C.phi, C.mu, C.h, Gs, Js, Cs, tt, CoefSrc<R, false>{c, x}, phin, mun, h1);
        pin(phin);
        pin(mun);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        own(C);
        if (valid) store3d<R, NP, NM, GEN, DIAG, NT>(out, g, o0 + (int64_t)m * sz, phin, mun, gy, da, dc);
        __syncthreads();
    };
    for (int m = t.m0; m < t.m1;) {
        plane(m, A, B);
        if (++m >= t.m1) break;
        plane(m, B, A);
        ++m;
    }
}

// The anisotropic step of one block.
template <typename R, int NP, int NM, bool OBST, int BX, int BY, bool GEN, bool DIAG, bool NT>
__device__ __forceinline__ void step3d_aniso(const R* __restrict__ in, R* __restrict__ out, const Geom& g,
                                             const Coef<R>& c, const int64_t* __restrict__ stepctr, int kstep,
                                             double tb0, double tdn, double tslope, int seg, int ntx, int nty,
                                             const CoefX<R>* x, DiagAcc* da, const DiagCoef* dc) {
    constexpr int NF = NP + NM;
    constexpr int NMM = mob_n<NM, GEN>();
    typedef Tile3d<BX, BY, true> Tile;
    constexpr int PW = Tile::PW, PP = Tile::PP, NPOS = Tile::NPOS;
    __shared__ R sp[4][NP][PP];
    __shared__ R su[3][NM][PP];
    __shared__ R sm[3][NMM][PP];
    Tile t;
    t.init(g, seg, ntx, nty);
    const bool perz = g.bcz == MP_BC_PERIODIC;
    const int64_t sz = (int64_t)g.nx * g.ny;
    const int64_t fs = g.fstride;

    R reg[NPOS][NF];
    auto fetch = [&](int m) {
        const R* p = in + (int64_t)gmap(m, g.nz, perz) * sz;
#pragma unroll
        for (int k = 0; k < NPOS; ++k)
            if (t.has(k)) {
#pragma unroll
                for (int f = 0; f < NF; ++f) reg[k][f] = p[f * fs + t.off[k]];
            }
    };
    // phi of plane m into slot m & 3, its mu and M~ into slot su_
    auto stage = [&](int m, int su_) {
        const int sl = m & 3;
#pragma unroll
        for (int k = 0; k < NPOS; ++k)
            if (t.has(k)) {
                R ph[NP], hh[NP], Mt[NMM];
#pragma unroll
                for (int a = 0; a < NP; ++a) {
                    ph[a] = reg[k][a];
                    sp[sl][a][t.pos[k]] = ph[a];
                }
                interp_h<R, NP>(ph, hh);
                mobility_any<R, NP, NM, GEN>(hh, c, x, Mt);
#pragma unroll
                for (int kk = 0; kk < NM; ++kk) su[su_][kk][t.pos[k]] = reg[k][NP + kk];
#pragma unroll
                for (int kk = 0; kk < NMM; ++kk) sm[su_][kk][t.pos[k]] = Mt[kk];
            }
    };

    // Face between positions (sL, pL) and (sR, pR) of the phi ring (uL, uR:
    // slots of mu and M~); tangential axes given as (slot, offset) steps: tS[t]
    // is the plane step, tP[t] the in-plane position step.
    auto face = [&](int sL, int uL_, int pL, int sR, int uR_, int pR, const int (&tS)[2], const int (&tP)[2],
                    R(&U)[NP], R(&Wf)[NP], R(&J)[NM]) {
        R phL[NP], phR[NP], uL[NM], uR[NM], mL[NMM], mR[NMM];
#pragma unroll
        for (int a = 0; a < NP; ++a) {
            phL[a] = sp[sL][a][pL];
            phR[a] = sp[sR][a][pR];
        }
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            uL[k] = su[uL_][k][pL];
            uR[k] = su[uR_][k][pR];
        }
#pragma unroll
        for (int k = 0; k < NMM; ++k) {
            mL[k] = sm[uL_][k][pL];
            mR[k] = sm[uR_][k][pR];
        }
        R tau[2][NP];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int sLp = (sL + tS[i]) & 3, sLm = (sL - tS[i]) & 3;
            const int sRp = (sR + tS[i]) & 3, sRm = (sR - tS[i]) & 3;
#pragma unroll
            for (int a = 0; a < NP; ++a)
                tau[i][a] = (sp[sLp][a][pL + tP[i]] - sp[sLm][a][pL - tP[i]]) +
                            (sp[sRp][a][pR + tP[i]] - sp[sRm][a][pR - tP[i]]);
        }
        face_core<R, NP, NM, true, 2, GEN>(phL, phR, tau, mL, mR, uL, uR, c, U, Wf, J);
    };

    // slots of mu and M~: of the plane being computed, the next one, and the
    // one being filled (the prologue puts plane m0 - 1 there; its z face reads
    // only the thread's own cell of that slot)
    int ua = 0, ub = 1, uc = 2;
    fetch(t.m0 - 1);
    stage(t.m0 - 1, uc);
    fetch(t.m0);
    stage(t.m0, ua);
    fetch(t.m0 + 1);
    stage(t.m0 + 1, ub);
    __syncthreads();

    const int pc = t.pos[0];
    const int gx = t.x0 + t.tid % BX;
    const int gy = t.y0 + t.tid / BX;
    const bool valid = gx < g.nx && gy < g.ny;
    const int64_t o0 = (int64_t)gx + (int64_t)gy * g.nx;
    const double tbase = tb0 + tdn * (double)(*stepctr + kstep);
    R Cs[NP];  // T - Te depends on y only
    const R tt = (R)(tbase + tslope * (double)gy);
    psi_const_any<R, NP, GEN>(tt, c, x, Cs);

    // tangential steps: x faces see (y, z), y faces see (x, z), z faces see (x, y)
    const int tSx[2] = {0, 1}, tPx[2] = {PW, 0};
    const int tSy[2] = {0, 1}, tPy[2] = {1, 0};
    const int tSz[2] = {0, 0}, tPz[2] = {1, PW};

    R Wlo[NP], Jlo[NM];  // z face between planes m-1 and m
    {
        R Ud[NP];
        face((t.m0 - 1) & 3, uc, pc, t.m0 & 3, ua, pc, tSz, tPz, Ud, Wlo, Jlo);
    }

    for (int m = t.m0; m < t.m1; ++m) {
        if (m + 2 <= t.m1) fetch(m + 2);
        const int s0 = m & 3;
        const int sp1 = (m + 1) & 3;

        R Gs[NP], Js[NM];
        {
            R Ul[NP], Wl[NP], Jl[NM], Uh[NP], Wh[NP], Jh[NM];
            face(s0, ua, pc - 1, s0, ua, pc, tSx, tPx, Ul, Wl, Jl);
            face(s0, ua, pc, s0, ua, pc + 1, tSx, tPx, Uh, Wh, Jh);
#pragma unroll
            for (int a = 0; a < NP; ++a) Gs[a] = Uh[a] - Wl[a];
#pragma unroll
            for (int k = 0; k < NM; ++k) Js[k] = Jh[k] - Jl[k];
        }
        {
            R Ul[NP], Wl[NP], Jl[NM], Uh[NP], Wh[NP], Jh[NM];
            face(s0, ua, pc - PW, s0, ua, pc, tSy, tPy, Ul, Wl, Jl);
            face(s0, ua, pc, s0, ua, pc + PW, tSy, tPy, Uh, Wh, Jh);
#pragma unroll
            for (int a = 0; a < NP; ++a) Gs[a] = Gs[a] + (Uh[a] - Wl[a]);
#pragma unroll
            for (int k = 0; k < NM; ++k) Js[k] = Js[k] + (Jh[k] - Jl[k]);
        }
        {
            R Uh[NP], Wh[NP], Jh[NM];
            face(s0, ua, pc, sp1, ub, pc, tSz, tPz, Uh, Wh, Jh);
#pragma unroll
            for (int a = 0; a < NP; ++a) {
                Gs[a] = Gs[a] + (Uh[a] - Wlo[a]);
                Wlo[a] = Wh[a];
            }
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                Js[k] = Js[k] + (Jh[k] - Jlo[k]);
                Jlo[k] = Jh[k];
            }
        }

        R phi[NP], mu[NM], h0[NP];
#pragma unroll
        for (int a = 0; a < NP; ++a) phi[a] = sp[s0][a][pc];
#pragma unroll
        for (int k = 0; k < NM; ++k) mu[k] = su[ua][k][pc];
        interp_h<R, NP>(phi, h0);
        R phin[NP], mun[NM];
        R h1[NP];
        cell_update_any<R, NP, NM, OBST, GEN>(phi, mu, h0, Gs, Js, Cs, tt, CoefSrc<R, false>{c, x}, phin, mun, h1);
        // staged before the stores: the wait for the loads would wait for them as well
        pin(phin);
        pin(mun);
        if (m + 2 <= t.m1) stage(m + 2, uc);
        if (valid) store3d<R, NP, NM, GEN, DIAG, NT>(out, g, o0 + (int64_t)m * sz, phin, mun, gy, da, dc);
        const int u = ua;
        ua = ub;
        ub = uc;
        uc = u;
        __syncthreads();
    }
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, int BX, int BY, bool GEN, bool DIAG = false,
          bool NT = false>
__device__ __forceinline__ void step3d_block(const R* __restrict__ in, R* __restrict__ out, const Geom& g,
                                             const Coef<R>& c, const int64_t* __restrict__ stepctr, int kstep,
                                             double tb0, double tdn, double tslope, int seg, int ntx, int nty,
                                             const CoefX<R>* x, DiagAcc* da = nullptr,
                                             const DiagCoef* dc = nullptr) {
    if constexpr (ANISO)
        step3d_aniso<R, NP, NM, OBST, BX, BY, GEN, DIAG, NT>(in, out, g, c, stepctr, kstep, tb0, tdn, tslope, seg, ntx,
                                                         nty, x, da, dc);
    else
        step3d_iso<R, NP, NM, OBST, BX, BY, GEN, DIAG, NT>(in, out, g, c, stepctr, kstep, tb0, tdn, tslope, seg, ntx,
                                                       nty, x, da, dc);
}

// FP64 at three waves per SIMD where the kernel fits their 168 registers: the
// isotropic plain ones (three phases and two mu fields take 182 otherwise) and
// the isotropic general ones of up to four fields without an obstacle.  The
// others are left to their registers: bound to three waves they spilled up to
// 91 of them.  Measured, us per step of 256^3, bound / free: three phases and
// one mu field, anisotropic, 1107 / 655, general with the active-set obstacle
// 1404 / 629; general isotropic of five fields 784 / 370, of four with the
// obstacle 292 / 259 and 286 / 275, of four without 249 / 267 and 253 / 254.
#define MP3_WAVES(R, FITS) (sizeof(R) == 4 ? 2 : (FITS) ? 3 : 1)

template <typename R, int NP, int NM, bool ANISO, bool OBST, int BX, int BY, bool NT>
__global__ void __launch_bounds__(BX * BY) __attribute__((amdgpu_waves_per_eu(MP3_WAVES(R, !ANISO))))
k_step3d(const R* __restrict__ in, R* __restrict__ out, Geom g, Coef<R> c,
         const int64_t* __restrict__ stepctr, int kstep, double tb0, double tdn, double tslope,
         int seg, int ntx, int nty) {
    step3d_block<R, NP, NM, ANISO, OBST, BX, BY, false, false, NT>(in, out, g, c, stepctr, kstep, tb0, tdn, tslope,
                                                                   seg, ntx, nty, nullptr);
}

// The extended model's 3D kernel (32 x 8 tiles).
template <typename R, int NP, int NM, bool ANISO, bool OBST>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MP3_WAVES(R, !ANISO && !OBST && NP + NM < 5))))
k_step3d_gen(const R* __restrict__ in, R* __restrict__ out, Geom g, Coef<R> c,
             const int64_t* __restrict__ stepctr, int kstep, double tb0, double tdn, double tslope,
             int seg, int ntx, int nty, CoefX<R> x) {
    step3d_block<R, NP, NM, ANISO, OBST, 32, 8, true>(in, out, g, c, stepctr, kstep, tb0, tdn, tslope, seg, ntx,
                                                      nty, &x);
}

// The same tiles writing, beside the state, one partial diagnostics record
// per block (block b's at d.part + b * DIAG_VALS): the diagnostics of the
// state they store.
template <typename R, int NP, int NM, bool ANISO, bool OBST, int BX, int BY, bool GEN>
__global__ void __launch_bounds__(BX * BY)
k_step3d_diag(const R* __restrict__ in, R* __restrict__ out, Geom g, Coef<R> c,
              const int64_t* __restrict__ stepctr, int kstep, double tb0, double tdn, double tslope,
              int seg, int ntx, int nty, CoefX<R> x, DiagOut d) {
    constexpr int NW = BX * BY / 64;
    __shared__ double drec[NW][DIAG_VALS];
    DiagAcc A;
    acc_init(A);
    step3d_block<R, NP, NM, ANISO, OBST, BX, BY, GEN, true>(in, out, g, c, stepctr, kstep, tb0, tdn, tslope, seg,
                                                            ntx, nty, GEN ? &x : nullptr, &A, &d.dc);
    diag_wave_store(A, drec[threadIdx.x >> 6]);
    __syncthreads();
    if (threadIdx.x == 0) {
        DiagRec T;
        rec_load(T, drec[0]);
        for (int w = 1; w < NW; ++w) {
            DiagRec B;
            rec_load(B, drec[w]);
            rec_merge(T, B);
        }
        rec_store(d.part + (int64_t)blockIdx.x * DIAG_VALS, T);
    }
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, int BY, bool GEN>
int call_3d_diag(const StepLaunch& L, const Coef<R>& c, const CoefX<R>& x, KernelCall& k) {
    constexpr int BX = 64;
    const int ntx = (L.g.nx + BX - 1) / BX;
    const int nty = (L.g.ny + BY - 1) / BY;
    const int nseg = (L.g.nz + L.seg - 1) / L.seg;
    const long long nblocks = (long long)ntx * nty * nseg;
    if (nblocks <= 0 || nblocks > 0x7fffffffLL || !L.diag) return MP_E_PARAM;
    k.func = (const void*)&k_step3d_diag<R, NP, NM, ANISO, OBST, BX, BY, GEN>;
    k.grid = dim3((unsigned)nblocks);
    k.block = dim3(BX * BY);
    k.nrec = nblocks;
    k.arg((const R*)L.in);
    k.arg((R*)L.out);
    k.arg(L.g);
    k.arg(c);
    k.arg(L.stepctr);
    k.arg(L.kstep);
    k.arg(L.tb0);
    k.arg(L.tdn);
    k.arg(L.tslope);
    k.arg(L.seg);
    k.arg(ntx);
    k.arg(nty);
    k.arg(x);
    k.arg(*L.diag);
    return MP_OK;
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, bool DIAG = false>
int call_3d_gen(const StepLaunch& L, const Coef<R>& c, const CoefX<R>& x, KernelCall& k) {
    if constexpr (DIAG) return call_3d_diag<R, NP, NM, ANISO, OBST, 4, true>(L, c, x, k);
    const int ntx = (L.g.nx + 31) / 32;
    const int nty = (L.g.ny + 7) / 8;
    const int nseg = (L.g.nz + L.seg - 1) / L.seg;
    const long long nblocks = (long long)ntx * nty * nseg;
    if (nblocks <= 0 || nblocks > 0x7fffffffLL) return MP_E_PARAM;
    k.func = (const void*)&k_step3d_gen<R, NP, NM, ANISO, OBST>;
    k.grid = dim3((unsigned)nblocks);
    k.block = dim3(256);
    k.arg((const R*)L.in);
    k.arg((R*)L.out);
    k.arg(L.g);
    k.arg(c);
    k.arg(L.stepctr);
    k.arg(L.kstep);
    k.arg(L.tb0);
    k.arg(L.tdn);
    k.arg(L.tslope);
    k.arg(L.seg);
    k.arg(ntx);
    k.arg(nty);
    k.arg(x);
    return MP_OK;
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, int BX, int BY>
int call_3d_by(const StepLaunch& L, const Coef<R>& c, KernelCall& k) {
    const int ntx = (L.g.nx + BX - 1) / BX;
    const int nty = (L.g.ny + BY - 1) / BY;
    const int nseg = (L.g.nz + L.seg - 1) / L.seg;
    const long long nblocks = (long long)ntx * nty * nseg;
    if (nblocks <= 0 || nblocks > 0x7fffffffLL) return MP_E_PARAM;
    k.func = L.nt ? (const void*)&k_step3d<R, NP, NM, ANISO, OBST, BX, BY, true>
                  : (const void*)&k_step3d<R, NP, NM, ANISO, OBST, BX, BY, false>;
    k.grid = dim3((unsigned)nblocks);
    k.block = dim3(BX * BY);
    k.arg((const R*)L.in);
    k.arg((R*)L.out);
    k.arg(L.g);
    k.arg(c);
    k.arg(L.stepctr);
    k.arg(L.kstep);
    k.arg(L.tb0);
    k.arg(L.tdn);
    k.arg(L.tslope);
    k.arg(L.seg);
    k.arg(ntx);
    k.arg(nty);
    return MP_OK;
}

// bx = threads per block: 256 (32 x 8 tiles: a row is one 128-byte line in
// FP32, and the halo, 1.33 staged cells per cell, is the smallest for the size)
// or 512 (64 x 8), accepted where four planes of phi, mu and M~ of such a tile
// fit in 64 KiB: FP32 with N + 2 (K - 1) <= 6 (the kernels keep fewer planes than
// that; the rule is what mp_set_tile has always taken).
// FP32 512^3 anisotropic: 897 us with 32 x 8 tiles, 913 with 64 x 4, 904 with
// 64 x 8; FP64 256^3 with three phases 318 / 336 us (32 x 8, 64 x 4). The
// diagnostics instances take 64 x 4 and 64 x 8.
template <typename R, int NP, int NM, int BY>
constexpr int lds3d_bytes() {
    return 4 * (NP + 2 * NM) * 66 * (BY + 2) * (int)sizeof(R);
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, bool DIAG = false>
int call_3d(const StepLaunch& L, const Coef<R>& c, KernelCall& k) {
    if constexpr (DIAG) {
        const CoefX<R> none{};
        if (L.bx == 512) {
            if constexpr (lds3d_bytes<R, NP, NM, 8>() <= 64 * 1024)
                return call_3d_diag<R, NP, NM, ANISO, OBST, 8, false>(L, c, none, k);
            return MP_E_PARAM;
        }
        return call_3d_diag<R, NP, NM, ANISO, OBST, 4, false>(L, c, none, k);
    } else {
        if (L.bx == 512) {
            if constexpr (lds3d_bytes<R, NP, NM, 8>() <= 64 * 1024)
                return call_3d_by<R, NP, NM, ANISO, OBST, 64, 8>(L, c, k);
            return MP_E_PARAM;
        }
        return call_3d_by<R, NP, NM, ANISO, OBST, 32, 8>(L, c, k);
    }
}

}  // namespace mp
