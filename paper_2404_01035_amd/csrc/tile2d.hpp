// Several 2D steps in one launch for grids that cannot fill the GPU: a block
// keeps a TW x TW region of the grid in LDS and steps it T times.
//
// On such grids a strip launch lasts as long as the launch itself and one
// wave's chain of rows take (4.3 us for any number of cells up to some ten
// thousand), so what counts is steps per launch.  The block's region covers
// its (TW - 2T)^2 output cells and T cells around them; step s is computed for
// the cells at least s away from the region's rim, so after T steps the output
// cells are right and nothing has been exchanged between blocks.  The rim is
// computed again by the neighbouring blocks, lanes that would idle otherwise.
// One thread per cell: it keeps its cell (phi, mu, h, M~) in registers, reads
// the four neighbours (anisotropy: eight) from LDS and evaluates its four
// faces, the same code on the same operands in the same order as the strips
// do, so the results are their bits.  Two LDS copies alternate, one barrier a
// step.  A ghost beyond a no-flux edge is the edge cell itself (the neighbour
// index stops there); a cell beyond a periodic edge is stepped as the image it
// is.
#pragma once

#include <type_traits>

#include "gp_device.hpp"

namespace mp {

template <typename R, int NP, int NM, bool ANISO, bool OBST, bool GEN, int TW>
__device__ __forceinline__ void tile2d_block(const R* __restrict__ in, R* __restrict__ out, const Geom& g,
                                             const Coef<R>& c, double tb0, double tdn, double tslope, double n,
                                             int T, int ntx, const CoefX<R>* x) {
    constexpr int NF = NP + NM;
    constexpr int NMM = mob_n<NM, GEN>();
    constexpr int NC = TW * TW;
    __shared__ R sv[2][NF][NC];
    __shared__ R sm[2][NMM][NC];

    const int ow = TW - 2 * T;  // output cells per side
    const int tid = threadIdx.x;
    const int lx = tid % TW, ly = tid / TW;
    const int gx = (int)(blockIdx.x % ntx) * ow - T + lx;
    const int gy = (int)(blockIdx.x / ntx) * ow - T + ly;
    const bool perx = g.bcx == MP_BC_PERIODIC, pery = g.bcy == MP_BC_PERIODIC;
    // cells beyond a no-flux edge are never stepped; their loads are clamped
    const bool live = (perx || (gx >= 0 && gx < g.nx)) && (pery || (gy >= 0 && gy < g.ny));
    const int cx = perx ? wrap(gx, g.nx) : min(max(gx, 0), g.nx - 1);
    const int cy = pery ? wrap(gy, g.ny) : min(max(gy, 0), g.ny - 1);
    const int64_t o = (int64_t)cy * g.nx + cx;
    // neighbour steps in the tile
    const int dl = !perx && gx == 0 ? 0 : -1, dr = !perx && gx == g.nx - 1 ? 0 : 1;
    const int dd = !pery && gy == 0 ? 0 : -TW, du = !pery && gy == g.ny - 1 ? 0 : TW;
    // distance from the rim, and whether the cell is one of the block's outputs
    const int rim = min(min(lx, TW - 1 - lx), min(ly, TW - 1 - ly));
    const bool mine = live && rim >= T && gx < g.nx && gy < g.ny;

    R phi[NP], mu[NM], h[NP], Mt[NMM];
#pragma unroll
    for (int a = 0; a < NP; ++a) phi[a] = in[a * g.fstride + o];
#pragma unroll
    for (int k = 0; k < NM; ++k) mu[k] = in[(NP + k) * g.fstride + o];
    interp_h<R, NP>(phi, h);
    mobility_any<R, NP, NM, GEN>(h, c, x, Mt);

    for (int s = 1; s <= T; ++s) {
        R(&v)[NF][NC] = sv[s & 1];
        R(&m)[NMM][NC] = sm[s & 1];
#pragma unroll
        for (int a = 0; a < NP; ++a) v[a][tid] = phi[a];
#pragma unroll
        for (int k = 0; k < NM; ++k) v[NP + k][tid] = mu[k];
#pragma unroll
        for (int k = 0; k < NMM; ++k) m[k][tid] = Mt[k];
        __syncthreads();
        if (live && rim >= s) {
            // one face between this cell and its neighbour at step d: the
            // neighbour is the left/lower cell (LO) or the right/upper one;
            // t1 is the step to the tangential neighbours above, t0 below
            auto face = [&](auto lo, int d, int t0, int t1, R(&U)[NP], R(&W)[NP], R(&J)[NM]) {
                constexpr bool LO = decltype(lo)::value;
                R pn[NP], un[NM], mn[NMM], tau[1][NP];
#pragma unroll
                for (int a = 0; a < NP; ++a) pn[a] = v[a][tid + d];
#pragma unroll
                for (int k = 0; k < NM; ++k) un[k] = v[NP + k][tid + d];
#pragma unroll
                for (int k = 0; k < NMM; ++k) mn[k] = m[k][tid + d];
                if constexpr (ANISO) {
#pragma unroll
                    for (int a = 0; a < NP; ++a) {
                        const R own = v[a][tid + t1] - v[a][tid + t0];
                        const R nbr = v[a][tid + d + t1] - v[a][tid + d + t0];
                        tau[0][a] = LO ? nbr + own : own + nbr;
                    }
                }
                if constexpr (LO)
                    face_core<R, NP, NM, ANISO, 1, GEN>(pn, phi, tau, mn, Mt, un, mu, c, U, W, J);
                else
                    face_core<R, NP, NM, ANISO, 1, GEN>(phi, pn, tau, Mt, mn, mu, un, c, U, W, J);
            };
            R Gs[NP], Js[NM];
            {
                R Ul[NP], Wl[NP], Jl[NM], Uh[NP], Wh[NP], Jh[NM];
                face(std::true_type(), dl, dd, du, Ul, Wl, Jl);
                face(std::false_type(), dr, dd, du, Uh, Wh, Jh);
#pragma unroll
                for (int a = 0; a < NP; ++a) Gs[a] = Uh[a] - Wl[a];
#pragma unroll
                for (int k = 0; k < NM; ++k) Js[k] = Jh[k] - Jl[k];
            }
            {
                R Ul[NP], Wl[NP], Jl[NM], Uh[NP], Wh[NP], Jh[NM];
                face(std::true_type(), dd, dl, dr, Ul, Wl, Jl);
                face(std::false_type(), du, dl, dr, Uh, Wh, Jh);
#pragma unroll
                for (int a = 0; a < NP; ++a) Gs[a] = Gs[a] + (Uh[a] - Wl[a]);
#pragma unroll
                for (int k = 0; k < NM; ++k) Js[k] = Js[k] + (Jh[k] - Jl[k]);
            }
            R Cs[NP];
            const R tt = (R)((tb0 + tdn * (n + (double)(s - 1))) + tslope * (double)cy);
            psi_const_any<R, NP, GEN>(tt, c, x, Cs);
            R pn[NP], un[NM], h1[NP];
            cell_update_any<R, NP, NM, OBST, GEN>(phi, mu, h, Gs, Js, Cs, tt, CoefSrc<R, false>{c, x}, pn, un, h1);
#pragma unroll
            for (int a = 0; a < NP; ++a) {
                phi[a] = pn[a];
                h[a] = h1[a];
            }
#pragma unroll
            for (int k = 0; k < NM; ++k) mu[k] = un[k];
            mobility_any<R, NP, NM, GEN>(h, c, x, Mt);
        }
    }
    if (mine) {
#pragma unroll
        for (int a = 0; a < NP; ++a) out[a * g.fstride + o] = phi[a];
#pragma unroll
        for (int k = 0; k < NM; ++k) out[(NP + k) * g.fstride + o] = mu[k];
    }
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, int TW>
__global__ void __launch_bounds__(TW * TW)
k_tile2d(const R* __restrict__ in, R* __restrict__ out, Geom g, Coef<R> c, const int64_t* __restrict__ stepctr,
         int kstep, double tb0, double tdn, double tslope, int T, int ntx) {
    tile2d_block<R, NP, NM, ANISO, OBST, false, TW>(in, out, g, c, tb0, tdn, tslope, (double)(*stepctr + kstep), T,
                                                    ntx, nullptr);
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, int TW>
__global__ void __launch_bounds__(TW * TW)
k_tile2d_gen(const R* __restrict__ in, R* __restrict__ out, Geom g, Coef<R> c, const int64_t* __restrict__ stepctr,
             int kstep, double tb0, double tdn, double tslope, int T, int ntx, CoefX<R> x) {
    tile2d_block<R, NP, NM, ANISO, OBST, true, TW>(in, out, g, c, tb0, tdn, tslope, (double)(*stepctr + kstep), T,
                                                   ntx, &x);
}

// One launch of L.fuse steps on regions of TW x TW cells.
template <typename R, int NP, int NM, bool ANISO, bool OBST, bool GEN, int TW>
int call_tile_w(const StepLaunch& L, const Coef<R>& c, const CoefX<R>* x, KernelCall& k) {
    const int ow = TW - 2 * L.fuse;
    if (L.fuse < 1 || ow < 1 || L.g.nz != 1) return MP_E_PARAM;
    const int ntx = (L.g.nx + ow - 1) / ow;
    const long long nblocks = (long long)ntx * ((L.g.ny + ow - 1) / ow);
    if (nblocks <= 0 || nblocks > 0x7fffffffLL) return MP_E_PARAM;
    if constexpr (GEN)
        k.func = (const void*)&k_tile2d_gen<R, NP, NM, ANISO, OBST, TW>;
    else
        k.func = (const void*)&k_tile2d<R, NP, NM, ANISO, OBST, TW>;
    k.grid = dim3((unsigned)nblocks);
    k.block = dim3(TW * TW);
    k.arg((const R*)L.in);
    k.arg((R*)L.out);
    k.arg(L.g);
    k.arg(c);
    k.arg(L.stepctr);
    k.arg(L.kstep);
    k.arg(L.tb0);
    k.arg(L.tdn);
    k.arg(L.tslope);
    k.arg(L.fuse);
    k.arg(ntx);
    if constexpr (GEN) k.arg(*x);
    return MP_OK;
}

template <typename R, int NP, int NM, bool ANISO, bool OBST, bool GEN>
int call_tile_v(const StepLaunch& L, const Coef<R>& c, const CoefX<R>* x, KernelCall& k) {
    if (L.tw == 16) return call_tile_w<R, NP, NM, ANISO, OBST, GEN, 16>(L, c, x, k);
    if (L.tw == 24) return call_tile_w<R, NP, NM, ANISO, OBST, GEN, 24>(L, c, x, k);
    if (L.tw == 32) return call_tile_w<R, NP, NM, ANISO, OBST, GEN, 32>(L, c, x, k);
    return MP_E_PARAM;
}

// (the general kernels' obstacle projections share one instance: the choice is CoefX::proj)
template <typename R, int NP, int NM, bool GEN>
int call_tile_flags(const StepLaunch& L, const Coef<R>& c, const CoefX<R>* x, KernelCall& k) {
    const bool obst = GEN ? L.potential != MP_WELL : L.potential == MP_OBSTACLE;
    if (L.aniso)
        return obst ? call_tile_v<R, NP, NM, true, true, GEN>(L, c, x, k)
                    : call_tile_v<R, NP, NM, true, false, GEN>(L, c, x, k);
    return obst ? call_tile_v<R, NP, NM, false, true, GEN>(L, c, x, k)
                : call_tile_v<R, NP, NM, false, false, GEN>(L, c, x, k);
}

template <typename R, bool GEN>
int call_tile(const StepLaunch& L, const Coef<R>& c, const CoefX<R>* x, KernelCall& k) {
    if (L.nphases == 2 && L.nmu == 1) return call_tile_flags<R, 2, 1, GEN>(L, c, x, k);
    if (L.nphases == 2 && L.nmu == 2) return call_tile_flags<R, 2, 2, GEN>(L, c, x, k);
    if (L.nphases == 3 && L.nmu == 1) return call_tile_flags<R, 3, 1, GEN>(L, c, x, k);
    if (L.nphases == 3 && L.nmu == 2) return call_tile_flags<R, 3, 2, GEN>(L, c, x, k);
    return MP_E_PARAM;
}

}  // namespace mp
