// Device code of the discrete adjoint: gradient of the time-averaged bottom
// wall heat flux J = (1/N) sum_{n=1..N} q^n (Sec. 3.2) with respect to the
// bottom-wall temperatures T_b(x) (Sec. 3.1) and the wall strength G_w
// (Eq. (22)).  One reverse step transposes the forward step of
// lbb_device.hpp stage by stage, in reverse order, over whole-lattice work
// arrays.  A launch covers any number of lattices through a lattice table (one
// lattice, or every member of a batch).  A wave is 64 columns of a row, with
// the halo columns its stencils need; every stencil and every transposed one
// is a column sum combined over the neighbouring lanes by lane shifts.  The
// blocks of an XCD take a contiguous run of tiles, so the rows and cache lines
// that tiles share are fetched once per XCD.  Per reverse step of state
// t -> t+1:
//   a_theradj  forces (Eqs. (7), (9), (22)) and velocity (Eq. (6)) of the
//              state on the tile and its halo (rho_ave from the mass
//              partials of the state); then the RK4 temperature step
//              (Eqs. (18)-(20)) transposed: div v and the coefficients of
//              Eq. (18), stage inputs recomputed and the four stages
//              transposed in one tile
//   a_lb       stencil transposes of grad rho and div v, push streaming
//              transposed (gather), MRT collision transposed in moment space,
//              velocity transposed, per-node force parts; then
//   a_final    interaction-force stencil transposed, EOS transposed,
//              rho = sum f, Zou-He completion transposed, the heat-flux sample
//              of state t transposed, and rho, j, psi of state t-1 for the
//              next reverse step: the second half of a_lb's launch on small
//              lattices, a launch of its own on large ones
// a_macro forms rho, j, psi of a state where no reverse step precedes it, and
// a_hf the heat-flux source of the last state.  The state of a node is its
// stored populations: wall-row populations that arrive from outside are
// completions of the stored ones (Zou-He), so their adjoint is folded into
// the stored ones.  The adjoint covers lattices with walls (periodic x).
#pragma once

#include "lbb_device.hpp"

namespace lbb {

// The LB adjoint's blocks: each wave a row, lane = column, 60 columns of a tile
// with two halo columns either side.  In one launch (ONE) the first and last
// row of a block are halo, in two launches none is.
constexpr int lb_waves(bool one) { return one ? 8 : 4; }
constexpr int lb_rows(bool one) { return one ? 6 : 4; }
constexpr int LBX = 60;
// Threads that sum partials in a temperature adjoint block: fewer than any
// block has, so the order of the sum does not depend on the tile shape.
constexpr int NSUM = 512;

// Work arrays of one lattice.  The per-node arrays are in the lattice's
// storage precision S (the forward values they hold are formed in FP64 from
// the stored state and rounded once; the adjoint parts are rounded once per
// reverse step), the partial sums and accumulators in FP64.  The host fills
// AdjW, whose per-node pointers are untyped; the kernels read the same
// pointers as AdjWG<S>.  A plane of S is below 2^32 bytes, so its accesses are
// a scalar base and a 32-bit byte offset (ld_at, st_at).
template <typename D, typename R>
struct AdjWT {
    // rho and psi of the state being reversed ([cur]) and of the state before
    // it, which a_lb leaves in the other; j of the state to be reversed next
    D *rho[2], *psi[2], *jx, *jy;
    D *gdiv, *grho, *gvx, *gvy;  // the temperature step's parts (grho: then with those of the LB step)
    D *gpsi, *gsx, *gsy;         // force parts between the two launches of the LB adjoint
    MassSum *mpart;  // block mass partials of the state being reversed (exact sums)
    // partials by lattice row and tile column, so that no sum depends on the
    // blocks: the rho_ave adjoint of the last reverse step; row 1's dJ/dG_w,
    // accumulated over the steps, by tile column
    R *fpart, *gpart;
    R *scal;    // [0] rho_ave of the state being reversed, [1] the rho_ave
                // adjoint of the last reverse step per node, [2] dJ/dG_w
};
using AdjW = AdjWT<void, double>;
template <typename S>
using AdjWG = AdjWT<S, double>;

// a device array as a global-address-space pointer
template <typename T>
__device__ __forceinline__ gmem<T> *gp(T *p)
{
    return (gmem<T> *)p;
}

// One lattice of an adjoint launch: its parameters, work arrays, stored
// states and adjoint buffers, and its place in the launch grid.  A launch
// covers any number of lattices; a block finds its lattice through a block ->
// lattice table and its tile from its index within the lattice.
struct AdjInst {
    DevParams P;
    AdjW w;
    const void *seg;          // stored states of the segment: slot k at 10 k nx ny elements
    const void *T0;           // T of the state the lattice starts from
    void *lf[2];              // adjoint of f in the storage precision: [cur] the later state, [cur ^ 1] the earlier
    double *lT[2];            // adjoint of T (FP64), same parity
    double *gr[2];            // density adjoint of interior nodes not yet added to lf (same parity)
    int gx;                   // LB adjoint tiles per lattice row
    int blk0;                 // first block of this lattice in the grid
    int nb;                   // blocks of this lattice
    int tgx, tblk0;           // temperature-adjoint tiles per row, first tile in its grid
};

#define A_INST                                            \
    const int blk = xcd_tile((int)blockIdx.x, (int)gridDim.x); \
    const AdjInst &I = ai[amap[blk]];                     \
    const DevParams &P = I.P;                             \
    const AdjWG<S> &w = reinterpret_cast<const AdjWG<S> &>(I.w); \
    const int q = blk - I.blk0;                           \
    (void)w;

// This wave's row gj and its lane's column gx of the block's tile: node c
// (clamped to the lattice) is the tile's own when `own` (row: own_row).
#define A_TILE(ONE)                                                                         \
    constexpr int LBY = lb_rows(ONE), HC = (64 - LBX) / 2, LBW = lb_waves(ONE);             \
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); \
    const int x = (q % I.gx) * LBX + lane - HC;                                             \
    const int gj = (q / I.gx) * LBY + wv - (ONE ? 1 : 0);                                   \
    const int gx = wrap_col(x, P.nx);                                                       \
    const size_t N = (size_t)P.nx * P.ny;                                                   \
    const bool inside = gj >= 0 && gj < P.ny;                                               \
    const bool own_row = inside && (!ONE || (wv >= 1 && wv < LBW - 1));                     \
    const bool own = own_row && lane >= HC && lane < HC + LBX && x < P.nx;                  \
    auto at = [&](int m) { /* node of row gj + m, clamped to the lattice */                 \
        const int gy = gj + m;                                                              \
        return (unsigned)(gy < 0 ? 0 : (gy >= P.ny ? P.ny - 1 : gy)) * (unsigned)P.nx + (unsigned)gx; \
    };                                                                                      \
    const unsigned c = at(0);                                                               \
    constexpr unsigned B = sizeof(S);                                                       \
    (void)B;                                                                                \
    (void)N;                                                                                \
    (void)own;

// stored state k of lattice I (populations; T follows at 9 nx ny)
template <typename S>
__device__ __forceinline__ const S *a_slot(const AdjInst &I, int k)
{
    return static_cast<const S *>(I.seg) + (size_t)k * 10 * (size_t)I.P.nx * I.P.ny;
}

#define A_ARGS const AdjInst *__restrict__ ai, const int *__restrict__ amap

__device__ __forceinline__ bool a_int(const DevParams &P, int j) { return j > 0 && j < P.ny - 1; }

// Mass of an LB adjoint block's nodes (0 where a lane has none) as an exact
// sum, valid in thread 0; all threads call it.
template <int LBW>
__device__ __forceinline__ MassSum a_block_mass(const DevParams &P, double rho, MassSum *red /* [LBW] */)
{
    MassSum s = wave_mass(mass_units(P.mass_c, P.mass_r, rho));
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = s;
    __syncthreads();
    s = {0, 0};
    if (threadIdx.x == 0)
        for (int k = 0; k < LBW; ++k) s.add(red[k]);
    return s;
}

// sum of one double per lane in a fixed order, in every lane
__device__ __forceinline__ double a_wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// 12 d_x T, 12 d_y T and 6 lap T from a column's rows r + 1, r, r - 1
struct ColGrad {
    double x, y, lap;
};
__device__ __forceinline__ ColGrad col_grad(double tN, double tc, double tS)
{
    const double v = (tN + tS) + 4.0 * tc, d = tN - tS;
    const double vW = lane_from_left(v), vE = lane_from_right(v);
    return {vE - vW, (lane_from_left(d) + lane_from_right(d)) + 4.0 * d, (vW + vE) + 4.0 * v - 36.0 * tc};
}

// 12 times the isotropic gradient transposed: what the vectors (x, y) of the
// neighbours (rows N, c, S of a column) send to a node
__device__ __forceinline__ double col_grad_T(double xN, double xc, double xS, double yN, double yS)
{
    const double U = 4.0 * xc + (xN + xS), V = yS - yN;
    return (lane_from_left(V + U) + lane_from_right(V - U)) + 4.0 * V;
}

// Force (Eqs. (7), (22), (9)) and velocity (Eq. (6)) of a node, zero force on
// the wall rows, from the column sums of psi: the stencil sums sx, sy of psi.
struct NodeForce {
    double sx, sy, Fx, Fy, vx, vy;
};
__device__ __forceinline__ NodeForce node_force(const DevParams &P, bool in, int gj, double pN, double pc, double pS,
                                                double r, double ir, double jx, double jy, double rho_ave)
{
    const ColGrad g = col_grad(pN, pc, pS);
    NodeForce o;
    o.sx = in ? g.x * (1.0 / 12.0) : 0.0;
    o.sy = in ? g.y * (1.0 / 12.0) : 0.0;
    o.Fx = -P.G * pc * o.sx;
    o.Fy = -P.G * pc * o.sy;
    if (in) {
        if (gj == 1) o.Fy += P.Gw_bottom * (1.0 / 6.0) * pc * pc;
        if (gj == P.ny - 2) o.Fy -= P.Gw_top * (1.0 / 6.0) * pc * pc;
        o.Fy -= (r - rho_ave) * P.g;
    }
    o.vx = (jx + 0.5 * o.Fx) * ir;
    o.vy = (jy + 0.5 * o.Fy) * ir;
    return o;
}

// phi'(T) and phi''(T) of the Peng-Robinson alpha function (Eq. (21)), and
// u = sqrt(T / T_c).  One reciprocal square root y = 1/sqrt(T / T_c) gives
// u = (T / T_c) y and 1/(T_c u) = y / T_c.
__device__ __forceinline__ void phi_derivs(const DevParams &P, double T, double &d1, double &d2, double &u)
{
    const double x = T * P.inv_Tc;
    const double y = rsq_nr(x);
    u = x * y;
    const double iu = y * P.inv_Tc;
    d1 = -P.kappa * (1.0 + P.kappa * (1.0 - u)) * iu;
    d2 = 0.5 * P.kappa * (1.0 + P.kappa) * iu * iu * iu * P.Tc;
}

// (dp/drho)_T and (dp/dT)_rho of Eq. (21); 1/D1 and 1/D2 from one reciprocal
__device__ __forceinline__ void eos_derivs(const DevParams &P, double r, double T, double &dpdr, double &dpdT)
{
    double d1, d2, u;
    phi_derivs(P, T, d1, d2, u);
    const double s = 1.0 + P.kappa * (1.0 - u);
    const double phi = s * s;
    const double D1 = 1.0 - P.b * r, D2 = 1.0 + 2.0 * P.b * r - P.b * P.b * r * r;
    const double i12 = rcp_nr(D1 * D2), i1 = D2 * i12, i2 = D1 * i12;
    dpdr = P.R * T * i1 * i1 - P.a * phi * 2.0 * r * (1.0 + P.b * r) * i2 * i2;
    dpdT = r * P.R * i1 - P.a * r * r * d1 * i2;
}

// Zou-He completion transposed: the adjoint of the completed populations of
// a wall node folded onto the stored (known) ones; the others are zeroed.
__device__ __forceinline__ void zou_he_T(double g[9], int bottom)
{
    if (bottom) {
        g[4] += g[2];
        g[7] += g[5];
        g[8] += g[6];
        g[1] += -0.5 * g[5] + 0.5 * g[6];
        g[3] += 0.5 * g[5] - 0.5 * g[6];
        g[2] = g[5] = g[6] = 0.0;
    } else {
        g[2] += g[4];
        g[5] += g[7];
        g[6] += g[8];
        g[1] += 0.5 * g[7] - 0.5 * g[8];
        g[3] += -0.5 * g[7] + 0.5 * g[8];
        g[4] = g[7] = g[8] = 0.0;
    }
}

// rho, j and psi of a stored state at node c into set b; returns rho
template <typename S>
__device__ __forceinline__ double a_macro_node(const DevParams &P, const S *__restrict__ f, const S *__restrict__ T,
                                               size_t N, unsigned c, int gj, const AdjWG<S> &w, int b)
{
    constexpr unsigned B = sizeof(S);
    S fs[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) fs[a] = ld_at(f + a * N, c * B);
    const double Tv = P.T_ref + (double)ld_at(T, c * B);
    double fl[9];
    complete_node(P, fs, gj, fl);
    double r = 0.0;
    for (int a = 0; a < 9; ++a) r += fl[a];
    st_at(w.rho[b], c * B, S(r));
    st_at(w.jx, c * B, S(fl[1] - fl[3] + fl[5] - fl[6] - fl[7] + fl[8]));
    st_at(w.jy, c * B, S(fl[2] - fl[4] + fl[5] + fl[6] - fl[7] - fl[8]));
    st_at(w.psi[b], c * B, S(pseudopotential(P, r, Tv)));
    return r;
}

template <typename S, bool ONE>
__global__ __launch_bounds__(64 * lb_waves(ONE)) void a_macro(A_ARGS, int k, int cur)
{
    __shared__ MassSum red[lb_waves(ONE)];
    A_INST
    A_TILE(ONE)
    const S *f = a_slot<S>(I, k);
    const double m = own ? a_macro_node<S>(P, f, f + 9 * N, N, c, gj, w, cur) : 0.0;
    const MassSum s = a_block_mass<LBW>(P, m, red);
    if (threadIdx.x == 0) w.mpart[q] = s;
}

// ---------------------------------------------------------------------------
// The temperature step transposed in one launch: the RK4 stage inputs
// T_2..T_4 recomputed (Eqs. (19)-(20)) and the four stages transposed, last
// first, on one tile with a halo of 7 (three forward stencil stages, four
// reverse ones).  Lane = column (tile TAX = 50 wide, one wave64 with the
// halo); each of the TAW waves owns RPW consecutive region rows in registers,
// so a tile is RPW TAW - 14 rows high.  Every stencil is a column sum (own
// column, rows r - 1 .. r + 1) combined over the neighbouring lanes by lane
// shifts; only the first and last row of each wave pass through LDS, one
// exchange and one barrier a stage.  Stage k's slope adjoint is
// g_k = w_k lT^{t+1}/6 + c_{k+1} gT_{k+1} (RK4 weights w = (1, 2, 2, 1),
// g_3 = lT^{t+1}/6), gT_k being the adjoint of the stage input T_k: the
// transposed slope of the slope adjoints of the node and its neighbours,
// which are zero outside the interior.  Outputs on the tile: the adjoint of
// T^t (lT^{t+1} plus the four gT_k) and the rho, grad rho, v and div v parts
// of the four stages.  The registers between stages hold the storage
// precision (the forward stages of an FP32 lattice run in FP32 too), the
// arithmetic is FP64.
//
// Bound by vector issue, about 650 instructions a region row at 128 registers
// (one block, 16 waves, a compute unit), with the loads before and the stores
// after the stages exposed.  Gathers of all eight neighbours from LDS planes,
// 24 reads a node and reverse stage, took about 1400.  Sixteen 384x192 FP32:
// 92.7 us a launch with them, 67.9 with column sums, 55.4 with the coefficient
// planes and six node fields neither written nor read, 32-bit addresses and
// neighbouring tiles on one XCD; 256x128 FP64: 14.6 -> 9.8.
constexpr int TAH = 7;
constexpr int TAX = 64 - 2 * TAH;

template <typename S, int RPW, int TAW>
__global__ __launch_bounds__(64 * TAW) void a_theradj(const AdjInst *__restrict__ ai, const int *__restrict__ tmap,
                                                      int k0, int cur)
{
    constexpr int H = RPW * TAW;       // region rows
    constexpr int TAY = H - 2 * TAH;   // tile rows
    // first ([0]) and last ([1]) row of each wave: the stage inputs T_1..T_4
    // (the advection coefficients pass through planes 2 and 3 before T_3 and
    // T_4 do) and the slope adjoints, alternating (the velocity before them)
    __shared__ S eT[4][TAW][2][64];
    __shared__ S eG[2][TAW][2][64];
    __shared__ MassSum s_mass[TAW];
    __shared__ double s_sum[NSUM / 64];
    const int blk = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const AdjInst &I = ai[tmap[blk]];
    const DevParams &P = I.P;
    const AdjWG<S> &w = reinterpret_cast<const AdjWG<S> &>(I.w);
    const int q = blk - I.tblk0;
    const int x0 = (q % I.tgx) * TAX, y0 = (q / I.tgx) * TAY;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wN = wv + 1 < TAW ? wv + 1 : wv, wS = wv > 0 ? wv - 1 : 0;  // waves of the rows beyond this wave's
    const int gx = wrap_col(x0 + lane - TAH, P.nx);
    const gmem<double> *__restrict__ lT1 = gp(I.lT[cur]);
    gmem<double> *__restrict__ lT0 = gp(I.lT[cur ^ 1]);
    const S *__restrict__ T = a_slot<S>(I, k0) + 9 * (size_t)P.nx * P.ny;
    const S *__restrict__ psi = w.psi[cur], *__restrict__ den = w.rho[cur];
    constexpr unsigned B = sizeof(S);
    const double chi = P.chi;
    const int r0 = wv * RPW, gy0 = y0 + r0 - TAH;  // first region row and lattice row of this wave
    // phi' = pk2 - pk1 y with y = sqrt(T_c / T); T phi'' + phi' = pk2 - pk1 y / 2
    const double pk1 = P.kappa * (1.0 + P.kappa) * P.inv_Tc, pk2 = P.kappa * P.kappa * P.inv_Tc;
    auto inside = [&](int m) { return gy0 + m >= 0 && gy0 + m < P.ny; };
    auto interior = [&](int m) { return a_int(P, gy0 + m); };
    auto at = [&](int m) {  // node of row m, clamped to the lattice
        const int gy = gy0 + m;
        return (unsigned)(gy < 0 ? 0 : (gy >= P.ny ? P.ny - 1 : gy)) * (unsigned)P.nx + (unsigned)gx;
    };
    auto share = [&](S(*e)[2][64], const S (&v)[RPW]) {
        e[wv][0][lane] = v[0];
        e[wv][1][lane] = v[RPW - 1];
    };
    // rows m + 1 and m - 1 of a quantity held in v and shared in e
    auto north = [&](const S(*e)[2][64], const S (&v)[RPW], int m) -> double {
        return m + 1 < RPW ? v[m + 1 < RPW ? m + 1 : 0] : e[wN][0][lane];
    };
    auto south = [&](const S(*e)[2][64], const S (&v)[RPW], int m) -> double {
        return m > 0 ? v[m > 0 ? m - 1 : 0] : e[wS][1][lane];
    };

    // force and velocity of the stored state (rho_ave of Eq. (9): every block
    // sums the lattice's mass partials in the same fixed order)
    S vx[RPW], vy[RPW], t[4][RPW], g3[RPW];
    double ax0[RPW], ay0[RPW];  // chi d rho / rho
    {
        S ps[RPW + 2], rh[RPW + 2], jx[RPW], jy[RPW];
        double l1[RPW];
#pragma unroll
        for (int m = 0; m < RPW + 2; ++m) {
            ps[m] = ld_at(psi, at(m - 1) * B);
            rh[m] = ld_at(den, at(m - 1) * B);
        }
#pragma unroll
        for (int m = 0; m < RPW; ++m) {
            jx[m] = ld_at(w.jx, at(m) * B);
            jy[m] = ld_at(w.jy, at(m) * B);
            t[0][m] = S(P.T_ref + (double)ld_at(T, at(m) * B));
            l1[m] = lT1[at(m)];
        }
        // sums over the lattice: mass, and in one block a lattice the rho_ave
        // adjoint of the last step, for a_lb
        MassSum sm{0, 0};
        const gmem<long long> *mp = (const gmem<long long> *)w.mpart;
        for (int k = threadIdx.x; k < I.nb; k += 64 * TAW) sm.add(MassSum{mp[2 * k], mp[2 * k + 1]});
        sm.hi = wave_sum_to_last(sm.hi);
        sm.lo = wave_sum_to_last(sm.lo);
        if (lane == 63) s_mass[wv] = sm;
        if (q == 0 && wv < NSUM / 64) {
            double sf = 0.0;
            for (int k = threadIdx.x; k < I.gx * P.ny; k += NSUM) sf += gp(w.fpart)[k];
            sf = a_wave_sum(sf);
            if (lane == 0) s_sum[wv] = sf;
        }
        __syncthreads();
        sm = {0, 0};
#pragma unroll
        for (int k = 0; k < TAW; ++k) sm.add(s_mass[k]);
        const double nodes = (double)P.nx * (double)P.ny, rho_ave = sm.value(P.mass_q) / nodes;
        if (q == 0 && threadIdx.x == 0) {
            double sf = 0.0;
            for (int k = 0; k < NSUM / 64; ++k) sf += s_sum[k];
            w.scal[0] = rho_ave;
            w.scal[1] = sf / nodes;
        }
#pragma unroll
        for (int m = 0; m < RPW; ++m) {
            g3[m] = interior(m) ? S(l1[m] * (1.0 / 6.0)) : S(0);
            const double r = rh[m + 1];
            const double ir = rcp_nr(r);
            const NodeForce o = node_force(P, interior(m), gy0 + m, ps[m + 2], ps[m + 1], ps[m], r, ir, jx[m], jy[m], rho_ave);
            const ColGrad d = col_grad(rh[m + 2], r, rh[m]);
            ax0[m] = chi * (1.0 / 12.0) * d.x * ir;
            ay0[m] = chi * (1.0 / 12.0) * d.y * ir;
            // the velocity the temperature equation sees is zero on the wall rows
            vx[m] = interior(m) ? S(o.vx) : S(0);
            vy[m] = interior(m) ? S(o.vy) : S(0);
        }
    }
    share(eG[0], vx);
    share(eG[1], vy);
    __syncthreads();

    // div v and the coefficients of Eq. (18) (wall rows carry none):
    // K(T) = ax d_x T + ay d_y T + chi lap T - cA T + cB T phi'(T) with
    // ax = -vx + chi d_x rho / rho, cA = div v R / ((1 - b rho) c_v),
    // cB = div v a rho / ((1 + 2 b rho - b^2 rho^2) c_v)
    S ax[RPW], ay[RPW];
    double cA[RPW], cB[RPW];
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        ax[m] = ay[m] = S(0);
        cA[m] = cB[m] = 0.0;
        if (interior(m)) {
            const double sv = 4.0 * vx[m] + (north(eG[0], vx, m) + south(eG[0], vx, m));
            const double dy = north(eG[1], vy, m) - south(eG[1], vy, m);
            const double dv = ((lane_from_right(sv) - lane_from_left(sv)) + (4.0 * dy + (lane_from_left(dy) + lane_from_right(dy)))) *
                    (1.0 / 12.0);
            const double r = ld_at(den, at(m) * B);
            const double D1 = 1.0 - P.b * r, D2 = 1.0 + 2.0 * P.b * r - P.b * P.b * r * r;
            const double i12 = rcp_nr(D1 * D2);
            ax[m] = S((ax0[m] - vx[m]) * (1.0 / 12.0));
            ay[m] = S((ay0[m] - vy[m]) * (1.0 / 12.0));
            cA[m] = P.R_cv * (D2 * i12) * dv;
            cB[m] = P.a_cv * r * (D1 * i12) * dv;
        }
    }
    share(eT[0], t[0]);
    share(eT[2], ax);
    share(eT[3], ay);
    __syncthreads();
    const double axN = eT[2][wN][0][lane], axS = eT[2][wS][1][lane];
    const double ayN = eT[3][wN][0][lane], ayS = eT[3][wS][1][lane];
    share(eG[0], g3);

    // The stages are straight-line over a wave's rows (shared terms are formed
    // once and the rows' chains overlap); rows outside the lattice or the
    // shrunk region hold values that nothing on the tile reads, and a wave
    // with no row in the region leaves a stage out.

    // forward stages: T_{s+1} = T_1 + c_s K(T_s) on the region shrunk by s + 1
    const double c2 = chi * (1.0 / 6.0);
#pragma unroll
    for (int s = 1; s <= 3; ++s) {
        const double cs = s == 3 ? 1.0 : 0.5;
        if (r0 + RPW - 1 > s && r0 < H - 1 - s) {
#pragma unroll
            for (int m = 0; m < RPW; ++m) {
                const double tc = t[s - 1][m];
                const ColGrad d = col_grad(north(eT[s - 1], t[s - 1], m), tc, south(eT[s - 1], t[s - 1], m));
                const double y = rsq_nr(tc * P.inv_Tc);
                const double h = ax[m] * d.x + ay[m] * d.y + c2 * d.lap + (cB[m] * (pk2 - pk1 * y) - cA[m]) * tc;
                const S v = S((double)t[0][m] + cs * h);
                t[s][m] = interior(m) ? v : t[0][m];
            }
            share(eT[s], t[s]);
        } else {
#pragma unroll
            for (int m = 0; m < RPW; ++m) t[s][m] = t[0][m];
        }
        __syncthreads();
    }

    // reverse stages k = 3..0 on the region shrunk by 7 - k: gT gathers what
    // the slope adjoint G sends over the transposed stencils.  With P = G ax/12
    // and Q = G ay/12 a column sends V + U to its right, V - U to its left and
    // 4 V - 16 c2 G_c to itself, U = 4 P_c + P_N + P_S, V = Q_S - Q_N +
    // c2 (4 G_c + G_N + G_S), c2 = chi/6; the Laplacian's centre weight adds
    // -20 c2 G_c.
    double lt[RPW], acc[RPW][4];
    S g[RPW];
#pragma unroll
    for (int m = 0; m < RPW; ++m) {
        lt[m] = 0.0;
        g[m] = g3[m];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][j] = 0.0;
    }
#pragma unroll
    for (int k = 3; k >= 0; --k) {
        const int R = 7 - k;
        const S(*e)[2][64] = eG[k & 1 ? 0 : 1];
        const double ck = k == 3 ? 1.0 : 0.5;
        const double wk = (k == 1) ? 1.0 : 2.0;        // RK4 weight of slope k-1
        if (r0 + RPW - 1 >= R && r0 < H - R) {
            // G, P and Q of rows -1 .. RPW
            double G[RPW + 2], Pg[RPW + 2], Qg[RPW + 2];
#pragma unroll
            for (int m = 0; m < RPW; ++m) {
                G[m + 1] = g[m];
                Pg[m + 1] = G[m + 1] * ax[m];
                Qg[m + 1] = G[m + 1] * ay[m];
            }
            G[0] = e[wS][1][lane];
            Pg[0] = G[0] * axS;
            Qg[0] = G[0] * ayS;
            G[RPW + 1] = e[wN][0][lane];
            Pg[RPW + 1] = G[RPW + 1] * axN;
            Qg[RPW + 1] = G[RPW + 1] * ayN;
            const bool tile_rows = r0 + RPW - 1 >= TAH && r0 < TAH + TAY;
#pragma unroll
            for (int m = 0; m < RPW; ++m) {
                const double gc = G[m + 1];
                const double U = 4.0 * Pg[m + 1] + (Pg[m + 2] + Pg[m]);
                const double V = (Qg[m] - Qg[m + 2]) + c2 * (4.0 * gc + (G[m + 2] + G[m]));
                const double Tv = t[k][m];
                const double y = rsq_nr(Tv * P.inv_Tc);
                const double ctr = cB[m] * (pk2 - (0.5 * pk1) * y) - cA[m] - 36.0 * c2;
                const double gT = (lane_from_left(V + U) + lane_from_right(V - U)) + (4.0 * V + gc * ctr);
                lt[m] += gT;
                if (k > 0) g[m] = interior(m) ? S(wk * (double)g3[m] + ck * gT) : S(0);
                if (tile_rows) {
                    // this stage's part of the rho, grad rho, v, div v adjoints at the node
                    const ColGrad d = col_grad(north(eT[k], t[k], m), Tv, south(eT[k], t[k], m));
                    const double gt = gc * Tv;
                    acc[m][0] += gc * d.x;
                    acc[m][1] += gc * d.y;
                    acc[m][2] += gt;
                    acc[m][3] += gt * (pk2 - pk1 * y);
                }
            }
        }
        if (k == 0) break;
        // the plane written here was last read before the previous barrier
        share(eG[k & 1], g);
        __syncthreads();
    }

    // outputs on the tile; what only they need of the state is formed again
    // here rather than held through the stages
    if (r0 + RPW - 1 < TAH || r0 >= TAH + TAY) return;
    const double pcv = 1.0 / P.R_cv;
    {
        double rh[RPW + 2];
#pragma unroll
        for (int m = 0; m < RPW + 2; ++m) rh[m] = ld_at(den, at(m - 1) * B);
#pragma unroll
        for (int m = 0; m < RPW; ++m) {
            const int r = r0 + m;
            const ColGrad gr = col_grad(rh[m + 2], rh[m + 1], rh[m]);
            if (r < TAH || r >= TAH + TAY || !inside(m) || lane < TAH || lane >= TAH + TAX || x0 + lane - TAH >= P.nx)
                continue;
            const unsigned c = at(m);
            lT0[c] = lT1[c] + lt[m];
            double avx = 0.0, avy = 0.0, adiv = 0.0, arho = 0.0;
            if (interior(m)) {
                // the rho derivatives E1 = R b / (D1^2 c_v), E2 = a (1 + b^2
                // rho^2) / (D2^2 c_v) of the pressure-work coefficients;
                // div v = cA D1 c_v / R
                const double ro = rh[m + 1];
                const double D1 = 1.0 - P.b * ro, D2 = 1.0 + 2.0 * P.b * ro - P.b * P.b * ro * ro;
                const double inv = rcp_nr(ro * D1 * D2);
                const double ri = D1 * D2 * inv, i1 = ro * D2 * inv, i2 = ro * D1 * inv;
                const double gx_ = acc[m][0] * (1.0 / 12.0), gy_ = acc[m][1] * (1.0 / 12.0);
                const double kr = chi * ri;
                avx = -gx_;
                avy = -gy_;
                adiv = P.a_cv * ro * i2 * acc[m][3] - P.R_cv * i1 * acc[m][2];
                // grad rho is constant over the stages: its part of the rho
                // adjoint is grad rho . (sum of g grad T)
                arho = -kr * ri * (1.0 / 12.0) * (gr.x * gx_ + gr.y * gy_) - P.b * cA[m] * i1 * acc[m][2] +
                       P.a_cv * (1.0 + P.b * P.b * ro * ro) * (i2 * i2) * cA[m] * D1 * pcv * acc[m][3];
            }
            st_at(w.gvx, c * B, S(avx));
            st_at(w.gvy, c * B, S(avy));
            st_at(w.gdiv, c * B, S(adiv));
            st_at(w.grho, c * B, S(arho));
        }
    }
}

// Heat-flux sample q = -(c_v chi / nx) sum_i rho(i,0) (-3 T0 + 4 T1 - T2)/2
// of a stored state, transposed with weight wq, at node (gi, gj) of rows
// 0..2: the population part (row 0, Zou-He folded) and the temperature part.
template <typename S>
__device__ __forceinline__ void hf_source(const DevParams &P, const S *__restrict__ f_, const S *__restrict__ T_,
                                          double wq, size_t N, int gi, int gj,
                                          double gpop[9], double &gtem)
{
    const gmem<S> *__restrict__ f = gp(f_), *__restrict__ T = gp(T_);
    const double k = -P.cv_chi / P.nx * wq;
    for (int a = 0; a < 9; ++a) gpop[a] = 0.0;
    gtem = 0.0;
    if (gj > 2) return;
    double fl[9];
    load_node(P, f, N, (size_t)gi, 0, fl);
    double r0 = 0.0;
    for (int a = 0; a < 9; ++a) r0 += fl[a];
    if (gj == 0) {
        const double t0 = (double)T[gi], t1 = (double)T[P.nx + gi], t2 = (double)T[2 * P.nx + gi];
        for (int a = 0; a < 9; ++a) gpop[a] = k * (-3.0 * t0 + 4.0 * t1 - t2) / 2.0;
        zou_he_T(gpop, 1);
    }
    gtem = k * r0 * (gj == 0 ? -1.5 : (gj == 1 ? 2.0 : -0.5));
}

// Force parts of a node's adjoint: of rho (with the other parts of the step),
// of psi (the node's own) and of the stencil sums of psi.
struct ForcePart {
    double grho, gpsi, gsx, gsy;
};

// The rest of a node's reverse step once its neighbours' force parts are
// known (rows N and S of its column given; all lanes of a row call it): the
// interaction-force stencil transposed, EOS transposed, rho = sum f, Zou-He
// completion transposed, the heat-flux source of the state (when it is a
// sample, wq > 0), and rho, j, psi of the state before (`prev`), whose rho is
// returned.
template <typename S>
__device__ __forceinline__ double a_node_end(const AdjInst &I, const AdjWG<S> &w, size_t N, unsigned c, int gx, int gj,
                                             bool own, const ForcePart &fo, double xN, double xS, double yN,
                                             double yS, int k, int cur, double wq, int prev)
{
    const DevParams &P = I.P;
    const S *__restrict__ f = a_slot<S>(I, k);
    const S *__restrict__ T = f + 9 * N;
    S *lf0 = static_cast<S *>(I.lf[cur ^ 1]);
    constexpr unsigned B = sizeof(S);
    const double gp_ = fo.gpsi + col_grad_T(xN, fo.gsx, xS, yN, yS) * (1.0 / 12.0);
    if (!own) return 0.0;
    double gr = fo.grho, gT = 0.0;
    if (gp_ != 0.0) {
        const double r = ld_at(w.rho[cur], c * B), Tv = P.T_ref + (double)ld_at(T, c * B);
        double dpdr, dpdT;
        eos_derivs(P, r, Tv, dpdr, dpdT);
        const double gq = gp_ * 0.5 * rcp_nr(ld_at(w.psi[cur], c * B)) * P.two_over_G;
        gr += gq * (dpdr - 1.0 / 3.0);
        gT = gq * dpdT;
    }
    double gpop[9], gtem = 0.0;
    if (wq != 0.0 && gj <= 2) hf_source<S>(P, f, T, wq, N, gx, gj, gpop, gtem);
    if (a_int(P, gj)) {
        // rho = sum f: the density adjoint joins every population of the
        // node; kept apart and added where the next step gathers lf
        gp(I.gr[cur ^ 1])[c] = gr;
    } else {
        double g[9];
        for (int a = 0; a < 9; ++a) g[a] = (double)ld_at(lf0 + a * N, c * B) + gr;
        zou_he_T(g, gj == 0);
        if (wq != 0.0 && gj == 0)
            for (int a = 0; a < 9; ++a) g[a] += gpop[a];
        for (int a = 0; a < 9; ++a) st_at(lf0 + a * N, c * B, S(g[a]));
    }
    gp(I.lT[cur ^ 1])[c] += gT + gtem;
    if (!prev) return 0.0;
    const S *__restrict__ fp = a_slot<S>(I, k - 1);
    return a_macro_node<S>(P, fp, fp + 9 * N, N, c, gj, w, cur ^ 1);
}

// The LB step transposed on one tile: the stencil transposes of grad rho and
// div v, push streaming transposed (gather), MRT collision transposed in
// moment space, velocity and force transposed per node; then, the force
// adjoints of neighbouring nodes exchanged (lane shifts within a row, LDS
// between waves), the interaction-force stencil transposed, EOS transposed,
// rho = sum f, Zou-He completion transposed and the heat-flux source of the
// state (when it is a sample, wq > 0); last rho, j, psi of the state before
// (`prev`) with its mass partials.  The state's F and v are formed again from
// psi, rho and f.  The rho_ave adjoint needs the sum over the lattice of a
// part formed here: it is one number a lattice, so the next reverse step adds
// it where it gathers (interior nodes take it whole, wall nodes through the
// completion).
// Near 27 us of vector issue and 30 us of memory traffic for sixteen 384x192
// FP32 in the two-launch form, four waves a SIMD to overlap them: 47.9 us plus
// 25.3 us for a_final (47.8 and 31.3 with aligned 64-column patches, every
// neighbour gathered from memory and the state's F and v read; 57.2 and 29.6
// before neighbouring tiles shared an XCD).  The one-launch form computes the
// two halo rows again (8/6) but neither writes nor reads the force parts and
// saves a launch: 256x128 FP64 9.7 us against 6.3 + 7.0.
template <typename S, bool ONE>
__global__ __launch_bounds__(64 * lb_waves(ONE), 4) void a_lb(A_ARGS, int k, int cur, double wq, int prev)
{
    __shared__ double eS[2][ONE ? lb_waves(ONE) : 1][64];  // (s_x, s_y) adjoints of the rows
    __shared__ MassSum red[ONE ? lb_waves(ONE) : 1];
    A_INST
    A_TILE(ONE)
    const S *__restrict__ f = a_slot<S>(I, k);
    const S *__restrict__ lf1 = static_cast<const S *>(I.lf[cur]);
    const gmem<double> *__restrict__ gr1 = gp(I.gr[cur]);
    S *lf0 = static_cast<S *>(I.lf[cur ^ 1]);
    const S *__restrict__ psi = w.psi[cur], *__restrict__ den = w.rho[cur];
    const int dW = gx > 0 ? -1 : P.nx - 1, dE = gx < P.nx - 1 ? 1 : 1 - P.nx;  // to the columns either side
    const double rho_ave = w.scal[0], srn = w.scal[1];
    ForcePart fo{0.0, 0.0, 0.0, 0.0};
    double pr = 0.0, pg = 0.0;
    if (inside) {
        const bool in = a_int(P, gj);
        const unsigned cN = at(1), cS = at(-1);
        // push streaming transposed: f'(c + e_a, a) = f*(c, a).  Interior
        // nodes keep their density adjoint apart (added here); wall nodes
        // hold the complete adjoint (Zou-He transposed) but for srn.
        double gfs[9];
        {
            double l[9];
            l[0] = ld_at(lf1, (c) * B);
            l[1] = ld_at(lf1 + N, (c + dE) * B);
            l[2] = ld_at(lf1 + 2 * N, (cN) * B);
            l[3] = ld_at(lf1 + 3 * N, (c + dW) * B);
            l[4] = ld_at(lf1 + 4 * N, (cS) * B);
            l[5] = ld_at(lf1 + 5 * N, (cN + dE) * B);
            l[6] = ld_at(lf1 + 6 * N, (cN + dW) * B);
            l[7] = ld_at(lf1 + 7 * N, (cS + dW) * B);
            l[8] = ld_at(lf1 + 8 * N, (cS + dE) * B);
            double g[3];  // rows S, c, N
#pragma unroll
            for (int e = -1; e <= 1; ++e) {
                const double v = gr1[at(e)];
                g[e + 1] = a_int(P, gj + e) ? v + srn : 0.0;
            }
            const double gE[3] = {lane_from_right(g[0]), lane_from_right(g[1]), lane_from_right(g[2])};
            const double gW[3] = {lane_from_left(g[0]), lane_from_left(g[1]), lane_from_left(g[2])};
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const int jj = gj + kEY[a];
                const double *row = kEX[a] == 0 ? g : (kEX[a] > 0 ? gE : gW);
                // share of srn that a wall node's completion passes to
                // population a: twice for those leaving through the wall, none
                // for those entering from it
                const double z = jj == 0 ? 1.0 - kEY[a] : (jj == P.ny - 1 ? 1.0 + kEY[a] : 0.0);
                const bool ok = jj >= 0 && jj < P.ny;
                gfs[a] = ok ? l[a] + row[kEY[a] + 1] + z * srn : 0.0;
            }
        }
        // f* = M^T diag(1/n) m*  ->  gm* = diag(1/n) M gf*
        double gms[9];
        {
            const double g14 = gfs[1] + gfs[2] + gfs[3] + gfs[4], g58 = gfs[5] + gfs[6] + gfs[7] + gfs[8];
            double a0 = 0.0;
            for (int a = 0; a < 9; ++a) a0 += gfs[a];
            gms[0] = a0 * (1.0 / 9.0);
            gms[1] = (-4.0 * gfs[0] - g14 + 2.0 * g58) * (1.0 / 36.0);
            gms[2] = (4.0 * gfs[0] - 2.0 * g14 + g58) * (1.0 / 36.0);
            gms[3] = (gfs[1] - gfs[3] + gfs[5] - gfs[6] - gfs[7] + gfs[8]) * (1.0 / 6.0);
            gms[4] = (-2.0 * gfs[1] + 2.0 * gfs[3] + gfs[5] - gfs[6] - gfs[7] + gfs[8]) * (1.0 / 12.0);
            gms[5] = (gfs[2] - gfs[4] + gfs[5] + gfs[6] - gfs[7] - gfs[8]) * (1.0 / 6.0);
            gms[6] = (-2.0 * gfs[2] + 2.0 * gfs[4] + gfs[5] + gfs[6] - gfs[7] - gfs[8]) * (1.0 / 12.0);
            gms[7] = (gfs[1] - gfs[2] + gfs[3] - gfs[4]) * 0.25;
            gms[8] = (gfs[5] - gfs[6] + gfs[7] - gfs[8]) * 0.25;
        }
        S fs[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) fs[a] = ld_at(f + a * N, c * B);
        double fl[9];
        complete_node(P, fs, gj, fl);
        // grad rho and div v of the temperature equation transposed (only
        // interior nodes carry them: both are zero on the walls)
        const double rN = (double)ld_at(den, cN * B), r = (double)ld_at(den, c * B), rS = (double)ld_at(den, cS * B), ir = rcp_nr(r);
        double gr = (double)ld_at(w.grho, c * B), gvx = 0.0, gvy = 0.0;
        {
            const double kN = P.chi * rcp_nr(rN), kc = P.chi * ir, kS = P.chi * rcp_nr(rS);
            const double xN = (double)ld_at(w.gvx, cN * B), xc = (double)ld_at(w.gvx, c * B), xS = (double)ld_at(w.gvx, cS * B);
            const double yN = (double)ld_at(w.gvy, cN * B), yc = (double)ld_at(w.gvy, c * B), yS = (double)ld_at(w.gvy, cS * B);
            // the grad rho adjoint is -(chi / rho) times the v adjoint
            gr -= col_grad_T(kN * xN, kc * xc, kS * xS, kN * yN, kS * yS) * (1.0 / 12.0);
            const double dN = (double)ld_at(w.gdiv, cN * B), dS = (double)ld_at(w.gdiv, cS * B);
            const double C = 4.0 * (double)ld_at(w.gdiv, c * B) + (dN + dS), e = dS - dN;
            if (in) {
                gvx = xc + (lane_from_left(C) - lane_from_right(C)) * (1.0 / 12.0);
                gvy = yc + ((lane_from_left(e) + lane_from_right(e)) + 4.0 * e) * (1.0 / 12.0);
            }
        }
        const double ps = (double)ld_at(psi, c * B);
        // moments of f and the equilibrium (Eq. (5)), forcing (Eq. (8))
        const double jx = fl[1] - fl[3] + fl[5] - fl[6] - fl[7] + fl[8];
        const double jy = fl[2] - fl[4] + fl[5] + fl[6] - fl[7] - fl[8];
        const double m7 = fl[1] - fl[2] + fl[3] - fl[4], m8 = fl[5] - fl[6] + fl[7] - fl[8];
        const NodeForce o = node_force(P, in, gj, (double)ld_at(psi, cN * B), ps, (double)ld_at(psi, cS * B), r, ir, jx, jy, rho_ave);
        const double vx = o.vx, vy = o.vy, Fx = o.Fx, Fy = o.Fy;
        const double v2 = vx * vx + vy * vy;
        const double meq7 = r * (vx * vx - vy * vy), meq8 = r * vx * vy;
        const double S7 = 2.0 * (vx * Fx - vy * Fy), S8 = vx * Fy + vy * Fx;
        const double tau = P.tau_V + (r - P.rho_V) * P.tau_slope, s_nu = rcp_nr(tau);
        const double L[9] = {P.s_rho, P.s_e, P.s_zeta, P.s_j, P.s_q, P.s_j, P.s_q, s_nu, s_nu};
        // m* = m - L (m - m_eq) + (1 - L/2) S
        double gq[9], gS[9];
        for (int k = 0; k < 9; ++k) {
            gq[k] = L[k] * gms[k];
            gS[k] = (1.0 - 0.5 * L[k]) * gms[k];
        }
        const double gsnu = gms[7] * (-(m7 - meq7) - 0.5 * S7) + gms[8] * (-(m8 - meq8) - 0.5 * S8);
        // m_eq(rho, v) of Eq. (5)
        gr += gq[0] + gq[1] * (-2.0 + 3.0 * v2) + gq[2] * (1.0 - 3.0 * v2) + gq[3] * vx - gq[4] * vx +
              gq[5] * vy - gq[6] * vy + gq[7] * (vx * vx - vy * vy) + gq[8] * vx * vy;
        gvx += r * (6.0 * vx * (gq[1] - gq[2]) + gq[3] - gq[4] + 2.0 * vx * gq[7] + vy * gq[8]);
        gvy += r * (6.0 * vy * (gq[1] - gq[2]) + gq[5] - gq[6] - 2.0 * vy * gq[7] + vx * gq[8]);
        // S(v, F, Q) of Eq. (8)
        const double a6 = gS[1] - gS[2];
        double gFx = 6.0 * a6 * vx + gS[3] - gS[4] + 2.0 * vx * gS[7] + vy * gS[8];
        double gFy = 6.0 * a6 * vy + gS[5] - gS[6] - 2.0 * vy * gS[7] + vx * gS[8];
        gvx += 6.0 * a6 * Fx + 2.0 * Fx * gS[7] + Fy * gS[8];
        gvy += 6.0 * a6 * Fy - 2.0 * Fy * gS[7] + Fx * gS[8];
        const double gQ = P.sig_e * gS[1] - P.sig_z * gS[2];
        // s_nu = 1 / tau(rho)
        gr += gsnu * (-P.tau_slope * s_nu * s_nu);
        // v = (j + F/2)/rho
        const double gjx = gvx * ir, gjy = gvy * ir;
        gFx += 0.5 * gvx * ir;
        gFy += 0.5 * gvy * ir;
        gr += -(gvx * vx + gvy * vy) * ir;
        __builtin_amdgcn_sched_barrier(0);
        double gm[9];
        for (int k = 0; k < 9; ++k) gm[k] = (1.0 - L[k]) * gms[k];
        // m = M f  ->  gf += M^T gm
        double gf[9];
        gf[0] = gm[0] - 4.0 * gm[1] + 4.0 * gm[2];
        gf[1] = gm[0] - gm[1] - 2.0 * gm[2] + gm[3] - 2.0 * gm[4] + gm[7];
        gf[2] = gm[0] - gm[1] - 2.0 * gm[2] + gm[5] - 2.0 * gm[6] - gm[7];
        gf[3] = gm[0] - gm[1] - 2.0 * gm[2] - gm[3] + 2.0 * gm[4] + gm[7];
        gf[4] = gm[0] - gm[1] - 2.0 * gm[2] - gm[5] + 2.0 * gm[6] - gm[7];
        gf[5] = gm[0] + 2.0 * gm[1] + gm[2] + gm[3] + gm[4] + gm[5] + gm[6] + gm[8];
        gf[6] = gm[0] + 2.0 * gm[1] + gm[2] - gm[3] - gm[4] + gm[5] + gm[6] - gm[8];
        gf[7] = gm[0] + 2.0 * gm[1] + gm[2] - gm[3] - gm[4] - gm[5] - gm[6] + gm[8];
        gf[8] = gm[0] + 2.0 * gm[1] + gm[2] + gm[3] + gm[4] - gm[5] - gm[6] - gm[8];
        if (own)
            for (int a = 0; a < 9; ++a) st_at(lf0 + a * N, c * B, S(gf[a] + kEX[a] * gjx + kEY[a] * gjy));
        // per-node force parts (no force on the wall rows)
        if (in) {
            gr += -P.g * gFy;
            if (own) pr += P.g * gFy;
            if (gj == 1) {
                fo.gpsi += gFy * P.Gw_bottom * ps / 3.0;
                if (own) pg += gFy * ps * ps / 6.0;
            }
            if (gj == P.ny - 2) fo.gpsi += -gFy * P.Gw_top * ps / 3.0;
            fo.gpsi += -P.G * (o.sx * gFx + o.sy * gFy);
            fo.gsx = -P.G * ps * gFx + 2.0 * P.G * P.G * o.sx * gQ;
            fo.gsy = -P.G * ps * gFy + 2.0 * P.G * P.G * o.sy * gQ;
        }
        // in the storage precision in either form
        fo.grho = S(gr);
        fo.gpsi = S(fo.gpsi);
        fo.gsx = S(fo.gsx);
        fo.gsy = S(fo.gsy);
    }
    if (own_row) {
        pr = a_wave_sum(pr);
        if (lane == 0) w.fpart[gj * I.gx + q % I.gx] = pr;
        if (gj == 1) {
            pg = a_wave_sum(pg);
            if (lane == 0) w.gpart[q % I.gx] += pg;
        }
    }
    if constexpr (ONE) {
        eS[0][wv][lane] = fo.gsx;
        eS[1][wv][lane] = fo.gsy;
        __syncthreads();
        double mass = 0.0;
        if (own_row)
            mass = a_node_end<S>(I, w, N, c, gx, gj, own, fo, eS[0][wv + 1][lane], eS[0][wv - 1][lane],
                                 eS[1][wv + 1][lane], eS[1][wv - 1][lane], k, cur, wq, prev);
        if (prev) {
            const MassSum s = a_block_mass<LBW>(P, mass, red);
            if (threadIdx.x == 0) w.mpart[q] = s;
        }
    } else if (own) {
        st_at(w.grho, c * B, S(fo.grho));
        st_at(w.gpsi, c * B, S(fo.gpsi));
        st_at(w.gsx, c * B, S(fo.gsx));
        st_at(w.gsy, c * B, S(fo.gsy));
    }
}

// The second launch of the two-launch form.
template <typename S>
__global__ __launch_bounds__(64 * lb_waves(false)) void a_final(A_ARGS, int k, int cur, double wq, int prev)
{
    __shared__ MassSum red[lb_waves(false)];
    A_INST
    A_TILE(false)
    double mass = 0.0;
    if (own_row) {
        const unsigned cN = at(1), cS = at(-1);
        const ForcePart fo{(double)ld_at(w.grho, c * B), (double)ld_at(w.gpsi, c * B), (double)ld_at(w.gsx, c * B), (double)ld_at(w.gsy, c * B)};
        mass = a_node_end<S>(I, w, N, c, gx, gj, own, fo, (double)ld_at(w.gsx, cN * B), (double)ld_at(w.gsx, cS * B), (double)ld_at(w.gsy, cN * B), (double)ld_at(w.gsy, cS * B), k, cur, wq, prev);
    }
    if (prev) {
        const MassSum s = a_block_mass<LBW>(P, mass, red);
        if (threadIdx.x == 0) w.mpart[q] = s;
    }
}

// The Dirichlet wall rows of T of the states the lattices start from, copied
// into each of `slots` stored states, whose steps do not rewrite them.  One
// block per table entry and slot.
template <typename S>
__global__ __launch_bounds__(256) void a_walls_T(const AdjInst *__restrict__ ai, int slots)
{
    const AdjInst &I = ai[blockIdx.x / slots];
    const int nx = I.P.nx;
    const size_t N = (size_t)nx * I.P.ny;
    const gmem<S> *T = gp(static_cast<const S *>(I.T0));
    gmem<S> *to = gp(const_cast<S *>(a_slot<S>(I, (int)(blockIdx.x % slots)))) + 9 * N;
    for (int x = threadIdx.x; x < nx; x += 256) {
        to[x] = T[x];
        to[N - nx + x] = T[N - nx + x];
    }
}

// The heat-flux sample of stored state k transposed, weight wq, added to the
// adjoint [cur] of that state (nodes of rows 0..2 act).
template <typename S, bool ONE>
__global__ __launch_bounds__(64 * lb_waves(ONE)) void a_hf(A_ARGS, int k, double wq, int cur)
{
    A_INST
    A_TILE(ONE)
    if (!own || gj > 2) return;
    const S *f = a_slot<S>(I, k);
    double gpop[9], gtem;
    hf_source<S>(P, f, f + 9 * N, wq, N, gx, gj, gpop, gtem);
    if (gj == 0) {
        gmem<S> *lf = gp(static_cast<S *>(I.lf[cur]));
        for (int a = 0; a < 9; ++a) lf[(size_t)a * N + c] = S((double)lf[(size_t)a * N + c] + gpop[a]);
    }
    gp(I.lT[cur])[c] += gtem;
}

// dJ/dG_w of each lattice from its tile columns' sums, one wave a lattice
__global__ __launch_bounds__(64) void a_wall(const AdjInst *__restrict__ ai)
{
    const AdjInst &I = ai[blockIdx.x];
    double s = 0.0;
    for (int b = threadIdx.x; b < I.gx; b += 64) s += I.w.gpart[b];
    s = a_wave_sum(s);
    if (threadIdx.x == 0) I.w.scal[2] = s;
}

}  // namespace lbb
