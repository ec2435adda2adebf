// One time step in one launch: forces, collision, streaming and the RK4
// temperature step of lbb_device.hpp on one tile, for the coupled model.
//
// A tile of TXF interior columns has a halo of HF = 5 nodes: four for the RK4
// stages, whose coefficients need rho and v of this step on their halo, and
// one more for the psi stencil behind that v.  The halo's densities, psi,
// forces and velocities are formed again by each tile that needs them; rho
// and v never leave the block.  Every value is formed by the expressions of
// the two-launch step (k_lb, k_thermal) on the same operands, and the mass
// sums are exact, so both paths reach the same state bit for bit.
//
// With one launch per step nothing in a launch may wait for another block of
// it, so the bookkeeping runs one launch behind: a launch of state t
//   - sums the mass partials that the launch before it left (rho_ave of t),
//   - lets its block 0 form the heat-flux sample of state t,
//   - leaves mass partials of state t+1 in the other half of I.mpart.
// I.rel counts the launches since the state index I.sc->tA (two slots, each
// launch reads one and writes the other); k_flush_step ends a sequence: it
// brings rho_ave, the heat flux and tA up to the last state and clears I.rel.
#pragma once

#include "lbb_device.hpp"

namespace lbb {

constexpr int HF = 5;             // halo of the one-launch step
constexpr int TXF = 64 - 2 * HF;  // its tile width: tile + halo is one wave wide

// Sum of this launch's input mass partials by one wave (all lanes take part),
// valid in every lane.
__device__ __forceinline__ double wave_rho_ave(const Inst &I, const MassSum *__restrict__ part_)
{
    const gmem<MassSum> *__restrict__ part = (const gmem<MassSum> *)part_;
    MassSum s{0, 0};
    for (int k = threadIdx.x & 63; k < I.npF; k += 4 * 64) {
        long long hi[4], lo[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = k + 64 * j < I.npF;
            hi[j] = in ? part[k + 64 * j].hi : 0;
            lo[j] = in ? part[k + 64 * j].lo : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s.hi += hi[j];
            s.lo += lo[j];
        }
    }
    s.hi = wave_sum_to_last(s.hi);
    s.lo = wave_sum_to_last(s.lo);
    MassSum u;
    u.hi = ((long long)__builtin_amdgcn_readlane((int)(s.hi >> 32), 63) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)s.hi, 63);
    u.lo = ((long long)__builtin_amdgcn_readlane((int)(s.lo >> 32), 63) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)s.lo, 63);
    return u.value(I.P.mass_q) / ((double)I.P.nx * (double)I.P.ny);
}

// The tile form: a block of NW waves owns I.tyF interior rows; region row r
// belongs to wave r mod NW (RPW rows a wave), lane = column.  psi, rho, v and
// the stage inputs pass between rows through LDS, between columns by lane
// shifts.
template <typename S, int NW, int RPW>
__global__ __launch_bounds__(64 * NW, 4) void k_step(const Inst *__restrict__ insts, const int *__restrict__ blk2inst,
                                                     int cf, int cT, int par, int aux)
{
    using C = typename ThermalCfg<S>::C;
    constexpr int HM = NW * RPW;  // region rows the block has room for
    __shared__ double buf[HM][64];  // psi, then the stage inputs
    __shared__ C X[3][HM][64];      // rho, vx, vy
    __shared__ C T0[HM][64];
    __shared__ MassSum red[NW];
    __shared__ double s_rho_ave;
    const Inst &I = insts[blk2inst[blockIdx.x]];
    const DevParams &P = I.P;
    Scalars *__restrict__ sc = I.sc;
    const S *__restrict__ fin = static_cast<const S *>(I.f[cf]);
    const S *__restrict__ Tin = static_cast<const S *>(I.T[cT]);
    const int blk = (int)blockIdx.x - I.blkF0;
    const long long since = I.rel[par], t = sc->tA + since;
    if (blk == 0) {
        sample_heat_flux<S, NW>(I, fin, Tin, t);
        if (threadIdx.x == 0) I.rel[par ^ 1] = since + 1;
        return;
    }
    S *__restrict__ fout = static_cast<S *>(I.f[cf ^ 1]);
    S *__restrict__ Tout = static_cast<S *>(I.T[cT ^ 1]);
    const int tile = xcd_tile(blk - 1, I.nbxF * I.nbyF);
    const int bx = tile % I.nbxF, by = tile / I.nbxF;
    const int TY = I.tyF, H = TY + 2 * HF;
    const int x0 = bx * TXF, y0 = by * TY;
    const size_t N = (size_t)P.nx * P.ny;
    const bool walls = !P.periodic_y;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gx = wrapi(x0 + lane - HF, P.nx);
    const unsigned gxu = (unsigned)gx;

    // lattice row of region row r (wrapped when periodic); false beyond a wall
    auto row_of = [&](int r, int &gy) -> bool {
        gy = y0 + r - HF;
        if (P.periodic_y) {
            gy = wrapi(gy, P.ny);
            return r < H;
        }
        return r < H && gy >= 0 && gy < P.ny;
    };

    // phase 1: populations and T of the wave's rows; rho and psi
    S fs[RPW][9], Tv[RPW];
    double rho[RPW];
    int gys[RPW];
    bool inl[RPW];
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        inl[m] = row_of(wv + NW * m, gys[m]);
        if (!inl[m]) continue;
        const unsigned o = ((unsigned)gys[m] * (unsigned)P.nx + gxu) * (unsigned)sizeof(S);
#pragma unroll
        for (int a = 0; a < 9; ++a) fs[m][a] = ld_at(fin + (size_t)a * N, o);
        Tv[m] = ld_at(Tin, o);
    }
    if (wv == 0) {  // wave 0 owns a halo row: it has the least to do
        const double ra = since ? wave_rho_ave(I, I.mpart + (size_t)par * I.npF) : sc->rho_ave;
        if (lane == 0) s_rho_ave = ra;
    }
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        rho[m] = 1.0;
        if (!inl[m]) continue;
        const int r = wv + NW * m;
        double fl[9];
        complete_node(P, fs[m], gys[m], fl);
        rho[m] = node_density(fl);
        buf[r][lane] = checked_psi(P, rho[m], P.T_ref + (double)Tv[m], sc, t);
        X[0][r][lane] = (C)(S)rho[m];
        T0[r][lane] = (C)Tv[m];
    }
    __syncthreads();
    const double rho_ave = s_rho_ave;

    // phase 2: force and velocity on the region shrunk by one node; collision
    // and streaming of the interior nodes
    MassSum mass{0, 0};
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        const int r = wv + NW * m, gy = gys[m];
        if (!inl[m] || r < 1 || r >= H - 1) continue;
        const bool wall_row = walls && (gy == 0 || gy == P.ny - 1);
        const bool live = r >= HF && r < HF + TY && y0 + r - HF < P.ny;
        long long units = 0;
        if (lane >= 1 && lane < 63) {
            double f[9];
            const double rh = rho[m];
            double Fx, Fy, Q;
            node_force<64>(P, &buf[0][0], lane - 1, r - 1, gy, rh, rho_ave, Fx, Fy, Q);
            complete_node(P, fs[m], gy, f);
            const Moments mo = node_moments(f);
            const double tau = P.tau_0 + rh * P.tau_slope, i2 = rcp_nr(rh * tau);
            const double inv_rho = tau * i2, s_nu = rh * i2;
            const double hx = mo.jx + 0.5 * Fx, hy = mo.jy + 0.5 * Fy;
            const double vx = hx * inv_rho, vy = hy * inv_rho;
            const S vxs = wall_row ? S(0) : S(vx), vys = wall_row ? S(0) : S(vy);
            X[1][r][lane] = (C)vxs;
            X[2][r][lane] = (C)vys;
            if (live && lane >= HF && lane < HF + TXF && x0 + lane - HF < P.nx) {
                if (aux) {
                    const unsigned oc = ((unsigned)gy * (unsigned)P.nx + gxu) * (unsigned)sizeof(S);
                    st_at(static_cast<S *>(I.rho), oc, S(rh));
                    st_at(static_cast<S *>(I.vx), oc, vxs);
                    st_at(static_cast<S *>(I.vy), oc, vys);
                }
                collide(P, mo, rh, hx, hy, vx, vy, Fx, Fy, Q, s_nu, f);
                units = push_node<S>(P, fout, N, gx, gy, f);
            }
        }
        if (live) mass.add(wave_sum_to_last(units));
    }
    if (lane == 63) red[wv] = mass;
    __syncthreads();
    if (threadIdx.x == 0) {
        MassSum s{0, 0};
        for (int k = 0; k < NW; ++k) s.add(red[k]);
        I.mpart[(size_t)(par ^ 1) * I.npF + tile] = s;
    }

    // phase 3: coefficients of the temperature equation
    const C chi6 = (C)(P.chi * (1.0 / 6.0));
    bool act[RPW];
    SlopeCoef<C> cfr[RPW];
    C acc[RPW];
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        const int r = wv + NW * m;
        acc[m] = C(0);
        cfr[m] = SlopeCoef<C>{};
        act[m] = inl[m] && !(walls && (gys[m] == 0 || gys[m] == P.ny - 1));
        if (!act[m] || r < 2 || r >= H - 2) continue;
        cfr[m] = slope_coef<C>(P, chi6, X[0][r][lane], X[0][r + 1][lane], X[0][r - 1][lane], X[1][r][lane], X[1][r + 1][lane],
                               X[1][r - 1][lane], X[2][r][lane], X[2][r + 1][lane], X[2][r - 1][lane]);
    }

    // phase 4: the RK4 stages; stage st reads T0 (st = 0) or the other of two
    // planes and writes one.  The planes take the place of psi (and, in FP64,
    // of rho), which no later phase reads.
    C(*Ts[2])[64];
    Ts[0] = reinterpret_cast<C(*)[64]>(&buf[0][0]);
    Ts[1] = sizeof(C) == 4 ? Ts[0] + HM : X[0];
    const C Tref = (C)P.T_ref;
    const C cst[3] = {C(0.5), C(0.5), C(1.0)};
    const C wst[4] = {C(1), C(2), C(2), C(1)};
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int rad = 3 - st;
        const C(*in)[64] = st == 0 ? T0 : Ts[(st - 1) & 1];
#pragma unroll
        for (int m = 0; m < RPW; ++m) {
            const int r = wv + NW * m;
            if (r >= H || r < HF - rad || r >= HF + TY + rad) continue;
            C h = C(0);
            if (act[m]) {
                h = stage_slope<C>(in[r][lane], in[r + 1][lane], in[r - 1][lane], cfr[m], Tref, chi6);
                acc[m] = st == 0 ? h : fma(wst[st], h, acc[m]);
            }
            if (st < 3) Ts[st & 1][r][lane] = fma(cst[st], h, T0[r][lane]);
        }
        if (st < 3) __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        const int r = wv + NW * m;
        if (r < HF || r >= HF + TY || lane < HF || lane >= HF + TXF) continue;
        if (x0 + lane - HF >= P.nx || y0 + r - HF >= P.ny || !act[m]) continue;
        const S Tn = (S)(T0[r][lane] + acc[m] * C(1.0 / 6.0));
        const double Tabs = P.T_ref + (double)Tn;
        if (!(Tabs > 0.0) || !(Tabs < 1e300)) flag_error(sc, t, ERR_T);
        st_at(Tout, ((unsigned)gys[m] * (unsigned)P.nx + gxu) * (unsigned)sizeof(S), Tn);
    }
}

// End of a sequence of one-launch steps: rho_ave, the heat-flux sample and
// the state index of the last state, whose buffers are cf, cT; without a
// launch since the last flush, the sample of the current state.  One block of
// NT threads.
template <typename S>
__device__ __forceinline__ void flush_step(const Inst &I, int cf, int cT)
{
    __shared__ MassSum red[NT / 64];
    const long long r0 = I.rel[0], r1 = I.rel[1], t0 = I.sc->tA;
    const int par = r1 > r0;
    const long long since = par ? r1 : r0;
    if (since == 0) {
        reduce_heat_flux(I.hf_part, I.nbxB, I.P.nx, I.sc, t0);
        return;
    }
    MassSum s{0, 0};
    if (I.P.mode == MODE_ISOTHERMAL) {  // the partials of k_lb
        const size_t np = (size_t)I.nbxA * I.P.ny;
        const gmem<long long> *part = (const gmem<long long> *)I.mass_part + par * np;
        for (size_t k = threadIdx.x; k < np; k += NT) s.add(part[k]);
    } else {
        const gmem<MassSum> *part = (const gmem<MassSum> *)I.mpart + (size_t)par * I.npF;
        for (int k = threadIdx.x; k < I.npF; k += NT) {
            s.hi += part[k].hi;
            s.lo += part[k].lo;
        }
    }
    s.hi = wave_sum_to_last(s.hi);
    s.lo = wave_sum_to_last(s.lo);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = s;
    // the barrier inside also covers red and the reads of rel and tA above
    sample_heat_flux<S, NT / 64>(I, static_cast<const S *>(I.f[cf]), static_cast<const S *>(I.T[cT]), t0 + since);
    if (threadIdx.x == 0) {
        MassSum u{0, 0};
        for (int k = 0; k < NT / 64; ++k) u.add(red[k]);
        I.sc->rho_ave = u.value(I.P.mass_q) / ((double)I.P.nx * (double)I.P.ny);
        I.sc->tA = t0 + since;
        I.sc->tB = t0 + since - 1;  // as the two-launch step leaves it
        I.rel[0] = I.rel[1] = 0;
    }
}

template <typename S>
__global__ __launch_bounds__(NT) void k_flush_step(const Inst *__restrict__ insts, int cf, int cT)
{
    flush_step<S>(insts[blockIdx.x], cf, cT);
}

}  // namespace lbb
