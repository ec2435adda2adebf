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
__device__ __forceinline__ double wave_rho_ave(const Inst &I, const MassSum *__restrict__ part_, int npF)
{
    const gmem<MassSum> *__restrict__ part = (const gmem<MassSum> *)part_;
    MassSum s{0, 0};
    for (int k = threadIdx.x & 63; k < npF; k += 4 * 64) {
        long long hi[4], lo[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = k + 64 * j < npF;
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
// Index of the state a launch starts from, read where it is used.
struct StepIndex {
    const gmem<long long> *rel;
    const gmem<Scalars> *sc;
    __device__ __forceinline__ operator long long() const { return sc->tA + *rel; }
};

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
    // All that the first loads of populations need is read from the table
    // together, and the step index not waited for before they are issued: as
    // the uses came, four scalar loads and that one followed each other (128x64
    // FP64 6.83 us per step, 7.03 before; 600x151 FP32 8.12, 8.49 before).
    Scalars *__restrict__ sc = I.sc;
    const S *__restrict__ fin = static_cast<const S *>(I.f[cf]);
    const S *__restrict__ Tin = static_cast<const S *>(I.T[cT]);
    const gmem<long long> *rel = (const gmem<long long> *)I.rel;
    const int blkF0 = I.blkF0, nbx = I.nbxF, nby = I.nbyF, TY = I.tyF, nx_ = P.nx, ny_ = P.ny, per = P.periodic_y;
    const unsigned divF = I.divF;
    const int npF = I.npF;
    MassSum *mpart = I.mpart;
    asm volatile("" : : "s"(divF), "s"(npF), "s"(mpart), "s"(sc), "s"(fin), "s"(Tin), "s"(rel), "s"(blkF0), "s"(nbx), "s"(nby), "s"(TY), "s"(nx_),
                 "s"(ny_), "s"(per));
    const int blk = (int)blockIdx.x - blkF0;
    const StepIndex t{rel + par, (const gmem<Scalars> *)sc};
    const long long since = *t.rel;
    if (blk == 0) {
        sample_heat_flux<S, NW, 2>(I, fin, Tin, t, &buf[0][0]);
        if (threadIdx.x == 0) I.rel[par ^ 1] = since + 1;
        return;
    }
    S *__restrict__ fout = static_cast<S *>(I.f[cf ^ 1]);
    S *__restrict__ Tout = static_cast<S *>(I.T[cT ^ 1]);
    const int tile = xcd_tile(blk - 1, nbx * nby);
    const int by = divF ? (int)__umulhi((unsigned)tile, divF) : tile, bx = tile - by * nbx;
    const int H = TY + 2 * HF;
    const int x0 = bx * TXF, y0 = by * TY;
    const size_t N = (size_t)P.nx * P.ny;
    const bool walls = !P.periodic_y;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gx = wrap_col(x0 + lane - HF, nx_);
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
        const double ra = since ? wave_rho_ave(I, mpart + (size_t)par * npF, npF) : ((const gmem<Scalars> *)sc)->rho_ave;
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
    NodeMass units{0, 0};  // of the wave's rows
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        const int r = wv + NW * m, gy = gys[m];
        if (!inl[m] || r < 1 || r >= H - 1) continue;
        const bool wall_row = walls && (gy == 0 || gy == P.ny - 1);
        const bool live = r >= HF && r < HF + TY && y0 + r - HF < P.ny;
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
                units.add(push_node<S>(P, fout, N, gx, gy, f));
            }
        }
    }
    const MassSum mass = wave_mass(units);
    if (lane == 63) red[wv] = mass;
    __syncthreads();
    if (threadIdx.x == 0) {
        MassSum s{0, 0};
        for (int k = 0; k < NW; ++k) s.add(red[k]);
        mpart[(size_t)(par ^ 1) * npF + tile] = s;
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
        cfr[m] = slope_coef<C>(P, X[0][r][lane], X[0][r + 1][lane], X[0][r - 1][lane], X[1][r][lane], X[1][r + 1][lane],
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

// Density and moments of a wall node, its populations completed on a copy.
__device__ __forceinline__ double wall_density(const double f[9], int bottom)
{
    double g[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) g[a] = f[a];
    zou_he(g, bottom);
    return node_density(g);
}

__device__ __forceinline__ Moments wall_moments(const double f[9], int bottom)
{
    double g[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) g[a] = f[a];
    zou_he(g, bottom);
    return node_moments(g);
}

// The marching form, for lattices that fill the chip many times over.  A wave
// owns a strip of TXF columns (with its halo one wave wide, lane = column) and
// marches up I.tyF rows; everything a row needs from the rows around it stays
// in the wave's registers and everything from the columns around it comes by
// lane shifts, so there is no LDS traffic and no barrier: the loads of row
// j + 1, the density and psi of row j, force, velocity, collision and streaming
// of row j - 1, the coefficients and the first RK4 stage of row j - 2 and the
// stages 2 to 4 of rows j - 3 to j - 5 run side by side in one iteration.  Five
// rows below and above the wave's own are formed again (their collision not).
// Blocks are WB waves on neighbouring strips; they only meet at the end, to
// add up their mass.
template <typename S, int WB>
__global__ __launch_bounds__(64 * WB, sizeof(S) == 4 ? 3 : 2) void k_march(const Inst *__restrict__ insts,
                                                                           const int *__restrict__ blk2inst, int cf,
                                                                           int cT, int par)
{
    using C = typename ThermalCfg<S>::C;
    __shared__ MassSum red[WB];
    __shared__ double part[NSAMPLE];
    const Inst &I = insts[blk2inst[blockIdx.x]];
    const DevParams &P = I.P;
    Scalars *__restrict__ sc = I.sc;
    const S *__restrict__ fin = static_cast<const S *>(I.f[cf]);
    const S *__restrict__ Tin = static_cast<const S *>(I.T[cT]);
    const int blk = (int)blockIdx.x - I.blkF0;
    // (global loads: a flat one still pending would turn waits in the loop into
    // waits for everything)
    const gmem<Scalars> *scg = (const gmem<Scalars> *)sc;
    const long long since = ((const gmem<long long> *)I.rel)[par], t = scg->tA + since;
    if (blk == 0) {
        sample_heat_flux<S, WB, 4>(I, fin, Tin, t, part);
        if (threadIdx.x == 0) I.rel[par ^ 1] = since + 1;
        return;
    }
    S *__restrict__ fout = static_cast<S *>(I.f[cf ^ 1]);
    S *__restrict__ Tout = static_cast<S *>(I.T[cT ^ 1]);
    const int nx = P.nx, ny = P.ny;
    const size_t N = (size_t)nx * ny;
    const int tile = xcd_tile(blk - 1, I.npF);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int id = tile * WB + wv;  // strips row by row; the last block may have waves to spare
    const int by = id / I.nbxF, strip = id - by * I.nbxF;
    const int x0 = strip * TXF;
    const int gx = wrap_col(x0 + lane - HF, nx);
    const int y0 = by * I.tyF, y1 = by < I.nbyF ? min(y0 + I.tyF, ny) : y0;
    const bool walls = !P.periodic_y;
    const bool mine = lane >= HF && lane < HF + TXF && x0 + lane - HF < nx;
    double rho_ave = scg->rho_ave;
    if (since) rho_ave = wave_rho_ave(I, I.mpart + (size_t)par * I.npF, I.npF);
    asm volatile("" : "+v"(rho_ave));  // here, before the loop

    // lattice row of row r (at most ny beyond the lattice when periodic), and
    // whether there is one
    auto inside = [&](int r) { return !walls || (r >= 0 && r < ny); };
    auto row = [&](int r) { return walls ? r : (r < 0 ? r + ny : (r >= ny ? r - ny : r)); };
    // A row's place in a plane is uniform over the wave and goes into the
    // scalar base; a lane adds its column and the columns its populations
    // stream to.
    constexpr unsigned sz = (unsigned)sizeof(S);
    const unsigned og = (unsigned)gx * sz;
    const unsigned oe = (unsigned)(gx + 1 == nx ? 0 : gx + 1) * sz, ow = (unsigned)(gx == 0 ? nx - 1 : gx - 1) * sz;

    // rows by their number mod 3: populations and T as loaded, psi, rho, vx,
    // vy, inputs of the stages 2 to 4
    S fr[3][9], Tr[3];
    Moments mp = {};  // of row j - 1
    double ps[3] = {};
    C xr[3] = {}, xu[3] = {}, xv[3] = {}, T1[3] = {}, T2[3] = {}, T3[3] = {};
    // T of rows j - 5 .. j; coefficients and slope sums of rows j - 5 .. j - 2
    C t0[6] = {}, acc[4] = {};
    SlopeCoef<C> kf[4] = {};
    double rc = 1.0;  // density of row j - 1
    NodeMass units{0, 0};
    const C Tref = (C)P.T_ref;
    const C chi6 = (C)(P.chi * (1.0 / 6.0));

    auto load = [&](int r, S f[9], S &T) {
        // always ten loads, of the nearest row where there is none, so that the
        // wait for the row before needs not wait for these
        const size_t o = (size_t)(walls ? min(max(r, 0), ny - 1) : row(r)) * nx;
        // opaque copies: scalar plane bases formed on the way, one 32-bit lane
        // offset, instead of a 64-bit address per plane and lane
        size_t n = N;
        unsigned v = og;
        asm volatile("" : "+s"(n), "+v"(v));
        T = ld_at(Tin + o, v);
        const S *p = fin + o;
#pragma unroll
        for (int a = 0; a < 9; ++a, p += n) f[a] = ld_at(p, v);
    };

    // Iteration j; K = j - (y0 - HF) mod 3.  The rows of the first iterations
    // that lie below the wave's halo are computed like any other, from whatever
    // the registers hold, and never used.
    auto body = [&](auto Kc, int j) {
        constexpr int K = decltype(Kc)::value, K1 = (K + 1) % 3, K2 = (K + 2) % 3;  // rows j, j - 2 (and j + 1), j - 1
        load(j + 1, fr[K1], Tr[K1]);
        // row j: density and psi
        double rj = 1.0;
        Moments mj = mp;
#pragma unroll
        for (int q = 0; q < 5; ++q) t0[q] = t0[q + 1];
        if (inside(j)) {
            double fl[9];
#pragma unroll
            for (int a = 0; a < 9; ++a) fl[a] = (double)fr[K][a];
            rj = node_density(fl);
            mj = node_moments(fl);
            if (walls && (j == 0 || j == ny - 1)) {
                rj = j == 0 ? wall_density(fl, 1) : wall_density(fl, 0);
                mj = j == 0 ? wall_moments(fl, 1) : wall_moments(fl, 0);
            }
            ps[K] = checked_psi(P, rj, P.T_ref + (double)Tr[K], sc, t);
            t0[5] = (C)Tr[K];
        }
        // row c = j - 1: force, velocity; collision and streaming
        {
            const int c = j - 1, gy = row(c);
            const bool bot = walls && gy == 0, top = walls && gy == ny - 1;
            double pN = ps[K], pS = ps[K1];
            if (bot) pS = pN;  // a ghost layer mirrors the first fluid row
            if (top) pN = pS;
            const double u = 4.0 * ps[K2] + (pN + pS), d = pN - pS;
            double Fx, Fy, Q;
            force_of(P, ps[K2], lane_from_right(u) - lane_from_left(u),
                     4.0 * d + (lane_from_right(d) + lane_from_left(d)), bot || top, gy, rc, rho_ave, Fx, Fy, Q);
            if ((bot || top) && !P.ghost) Fx = Fy = Q = 0.0;
            double f[9];
            const Moments mo = mp;
            const double tau = P.tau_0 + rc * P.tau_slope, i2 = rcp_nr(rc * tau);
            const double inv_rho = tau * i2, s_nu = rc * i2;
            const double hx = mo.jx + 0.5 * Fx, hy = mo.jy + 0.5 * Fy;
            const double vx = hx * inv_rho, vy = hy * inv_rho;
            xr[K2] = (C)(S)rc;
            xu[K2] = (C)(S)vx;
            xv[K2] = (C)(S)vy;
            if (bot || top) xu[K2] = xv[K2] = C(0);
            if (c >= y0 && c < y1) {
                collide(P, mo, rc, hx, hy, vx, vy, Fx, Fy, Q, s_nu, f);
                const NodeMass m = pushed_mass(P, gy, f);
                if (mine) {
                    // push streaming as push_node
                    units.add(m);
                    size_t n = N;
                    unsigned vg = og, ve = oe, vw = ow;
                    asm volatile("" : "+s"(n), "+v"(vg), "+v"(ve), "+v"(vw));
                    S *p = fout + (size_t)gy * nx;
                    st_at(p, vg, S(f[0]));
                    st_at(p + n, ve, S(f[1]));
                    st_at(p + 3 * n, vw, S(f[3]));
                    if (!walls || gy + 1 < ny) {
                        S *q = fout + 2 * n + (size_t)(gy + 1 == ny ? 0 : gy + 1) * nx;
                        st_at(q, vg, S(f[2]));
                        st_at(q + 3 * n, ve, S(f[5]));
                        st_at(q + 4 * n, vw, S(f[6]));
                    }
                    if (!walls || gy > 0) {
                        S *q = fout + 4 * n + (size_t)(gy == 0 ? ny - 1 : gy - 1) * nx;
                        st_at(q, vg, S(f[4]));
                        st_at(q + 3 * n, vw, S(f[7]));
                        st_at(q + 4 * n, ve, S(f[8]));
                    }
                }
            }
        }
        rc = rj;
        mp = mj;
        // rows j - 2 .. j - 5: coefficients and the four stages (no slope on
        // the wall rows)
        auto at_wall = [&](int r) { return walls && (r <= 0 || r >= ny - 1); };
#pragma unroll
        for (int q = 3; q > 0; --q) {
            kf[q] = kf[q - 1];
            acc[q] = acc[q - 1];
        }
        kf[0] = slope_coef<C>(P, xr[K1], xr[K2], xr[K], xu[K1], xu[K2], xu[K], xv[K1], xv[K2], xv[K]);
        C h = stage_slope<C>(t0[3], t0[4], t0[2], kf[0], Tref, chi6);
        if (at_wall(j - 2)) h = C(0);
        acc[0] = h;
        T1[K1] = fma(C(0.5), h, t0[3]);
        h = stage_slope<C>(T1[K], T1[K1], T1[K2], kf[1], Tref, chi6);
        if (at_wall(j - 3)) h = C(0);
        acc[1] = fma(C(2), h, acc[1]);
        T2[K] = fma(C(0.5), h, t0[2]);
        h = stage_slope<C>(T2[K2], T2[K], T2[K1], kf[2], Tref, chi6);
        if (at_wall(j - 4)) h = C(0);
        acc[2] = fma(C(2), h, acc[2]);
        T3[K2] = fma(C(1), h, t0[1]);
        h = stage_slope<C>(T3[K1], T3[K2], T3[K], kf[3], Tref, chi6);
        const int r = j - 5;
        if (r >= y0 && r < y1 && !at_wall(r)) {
            const C a = fma(C(1), h, acc[3]);
            const S Tn = (S)(t0[0] + a * C(1.0 / 6.0));
            if (mine) {
                const double Tabs = P.T_ref + (double)Tn;
                if (!(Tabs > 0.0) || !(Tabs < 1e300)) flag_error(sc, t, ERR_T);
                unsigned v = og;
                asm volatile("" : "+v"(v));
                st_at(Tout + (size_t)row(r) * nx, v, Tn);
            }
        }
    };

    if (y0 < y1) {
        load(y0 - HF, fr[0], Tr[0]);
        // whole turns of the three register names.  Heights are 2 modulo 3, so
        // full strips end with row y1 + HF - 1; a ragged last strip may run two
        // rows past it and load one more, which are never used, and wrap once
        // into a periodic lattice of at least 8 rows (the host asks for 32).
        for (int j = y0 - HF; j < y1 + HF; j += 3) {
            body(std::integral_constant<int, 0>{}, j);
            body(std::integral_constant<int, 1>{}, j + 1);
            body(std::integral_constant<int, 2>{}, j + 2);
        }
    }
    MassSum m{0, 0};
    m.add(units.hi, units.lo);
    m.hi = wave_sum_to_last(m.hi);
    m.lo = wave_sum_to_last(m.lo);
    if (lane == 63) red[wv] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        MassSum u{0, 0};
#pragma unroll
        for (int k = 0; k < WB; ++k) u.add(red[k]);
        I.mpart[(size_t)(par ^ 1) * I.npF + tile] = u;
    }
}

// Launches since the last flush: the larger of the two counts.
__device__ __forceinline__ long long steps_since(const Inst &I, int &par)
{
    const long long r0 = I.rel[0], r1 = I.rel[1];
    par = r1 > r0;
    return par ? r1 : r0;
}

// The heat-flux partials of the last state of a sequence of one-launch steps,
// a wave a chunk: before the flush of wide lattices (block y: the lattice).
template <typename S>
__global__ __launch_bounds__(64) void k_flush_chunks(const Inst *__restrict__ insts, int cf, int cT)
{
    const Inst &I = insts[blockIdx.y];
    int par;
    if ((int)blockIdx.x >= I.nbxB || steps_since(I, par) == 0) return;
    const double q = chunk_flux<S>(I.P, static_cast<const S *>(I.f[cf]), static_cast<const S *>(I.T[cT]), (int)blockIdx.x);
    if (threadIdx.x == 0) I.hf_part[blockIdx.x] = q;
}

// End of a sequence of one-launch steps: rho_ave, the heat-flux sample and
// the state index of the last state, whose buffers are cf, cT (its partials
// there already if `ready`); without a launch since the last flush, the sample
// of the current state.  One block of NTH threads.
template <typename S, int NTH>
__device__ __forceinline__ void flush_step(const Inst &I, int cf, int cT, bool ready)
{
    __shared__ MassSum red[NTH / 64];
    __shared__ double part[NSAMPLE];
    int par;
    const long long t0 = I.sc->tA, since = steps_since(I, par);
    if (since == 0) {
        reduce_heat_flux(I.hf_part, I.nbxB, I.P.nx, I.sc, t0);
        return;
    }
    MassSum s{0, 0};
    const gmem<MassSum> *mp = (const gmem<MassSum> *)I.mpart + (size_t)par * I.npF;
    for (int k = threadIdx.x; k < I.npF; k += NTH) {
        s.hi += mp[k].hi;
        s.lo += mp[k].lo;
    }
    s.hi = wave_sum_to_last(s.hi);
    s.lo = wave_sum_to_last(s.lo);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = s;
    // the barrier of either branch also covers red and the reads of rel and tA above
    if (ready) {
        __syncthreads();
        reduce_heat_flux(I.hf_part, I.nbxB, I.P.nx, I.sc, t0 + since);
    } else {
        sample_heat_flux<S, NTH / 64, 4>(I, static_cast<const S *>(I.f[cf]), static_cast<const S *>(I.T[cT]), t0 + since,
                                         part);
    }
    if (threadIdx.x == 0) {
        MassSum u{0, 0};
        for (int k = 0; k < NTH / 64; ++k) u.add(red[k]);
        I.sc->rho_ave = u.value(I.P.mass_q) / ((double)I.P.nx * (double)I.P.ny);
        I.sc->tA = t0 + since;
        I.sc->tB = t0 + since - 1;  // as the two-launch step leaves it
        I.rel[0] = I.rel[1] = 0;
    }
}

template <typename S, int NTH>
__global__ __launch_bounds__(NTH) void k_flush_step(const Inst *__restrict__ insts, int cf, int cT, int ready)
{
    const Inst &I = insts[blockIdx.x];
    flush_step<S, NTH>(I, cf, cT, ready != 0);
    if (threadIdx.x == 0 && I.host) *I.host = *I.sc;  // the thread that wrote the scalars
}

}  // namespace lbb
