// lbm_adjoint.hpp -- gfx950 kernels of the hand-written adjoint of one step.
//
// Forward step n (arXiv:1703.04594 section 3; order of section 5):
//   g = bc(propagate(f_n)),   f_{n+1} = g + (f^eq(M(g)) - g) / tau,
// M(g) = (rho, j, E) the raw moments of eq. (2).  Given lambda = dL/df_{n+1}:
//
//  collide^T (site-local, rank-4 update):
//    mu_l = (1 - 1/tau) lambda_l + q_rho + q_jx xi_x,l + q_jy xi_y,l + q_E |xi_l|^2
//    with q = J_M^T J_eq^T (lambda / tau): the 4 dot products of lambda with
//    d f^eq / d(rho, u*, T*) pulled back through u = j / rho,
//    T = (E / rho - |u|^2) / 2 and the gravity shift.
//  d step / d tau:  -(1/tau^2) <lambda, f^eq - g> + <lambda / tau, d f^eq / d tau>
//    (the last term through u* = u + tau g, T* = T + tau (1 - tau) g^2 / 2).
//  propagate^T and bc^T, evaluated as a pull by the step that needs lambda_n
//  (the next reverse step, or the readers of lambda): the buffer holds mu at
//  each site, and
//    lambda_n,l(s) = [s + e_l inside the lattice] mu_l(s + e_l) + beta(s),
//  since the pull g_l(s') = f_l(s' - e_l) reads f_l(s) only from s' = s + e_l,
//  and a slot s' whose source s is inside is never a wall slot.  beta (rows
//  0-2 and ly-3..ly-1 only) is bc^T: a wall slot (l, w) carries
//  E^w_l rho(m) with rho(m) = sum_k f_k(m) at the mirror site m of its
//  source, so every population of m receives E^w_l mu_l(w).  For a site s
//  in row r from a wall, the wall slots mirroring onto it are
//  w = (x + e_x,l, e_n - 1 - r) counted from that wall, for each l whose
//  component e_n into the lattice exceeds r.
//  Storing mu at its own site keeps every store aligned (a push would write
//  e_y-shifted partial lines) and folds bc^T into the gather.
#pragma once

#include "lbm_kernels.hpp"

namespace lbm {

struct AdjArgs { double tau, omega, gy; };

// Per-site scalars of collide^T that depend only on the gathered moments.
struct AdjSite {
    double rho, inv, ux, uy, uys, E, th, u2, cux, cuy;
};

__host__ __device__ __forceinline__ AdjSite adj_site_scalars(double m0, double sx, double sy, double s2, const AdjArgs& a)
{
    AdjSite q;
    q.rho = m0;
    q.inv = 1.0 / m0;
    q.ux = C * sx * q.inv;
    q.uy = C * sy * q.inv;
    q.E = C2 * s2;
    const double T = 0.5 * (q.E * q.inv - (q.ux * q.ux + q.uy * q.uy));
    q.uys = q.uy + a.tau * a.gy;
    q.th = T - 1.0 + a.tau * (1.0 - a.tau) * a.gy * a.gy * 0.5;
    q.u2 = q.ux * q.ux + q.uys * q.uys;
    q.cux = C * q.ux;
    q.cuy = C * q.uys;
    return q;
}

// OPP.v[l]: index of the hop opposite to l (e_l' = -e_l; same shell),
// tabulated at compile time so that indexing with an unrolled l folds.
struct OppTable { int v[NPOP]; };
constexpr OppTable make_opp()
{
    OppTable t{};
    for (int l = 0; l < NPOP; ++l)
        for (int k = 0; k < NPOP; ++k)
            if (EX[k] == -EX[l] && EY[k] == -EY[l]) t.v[l] = k;
    return t;
}
constexpr OppTable OPP = make_opp();
static_assert(OPP.v[0] == 0 && OPP.v[1] == 3 && OPP.v[2] == 4 && OPP.v[36] == 32, "opposite hops");

// mu <- collide^T lambda at one site, in place, given the gathered moments
// (m0, sx, sy, s2) and Lg = sum_l lambda_l g_l; returns the site's d/dtau term.
//
// The equilibrium factor of population l is a polynomial in a_l = xi_l . u*,
//   P(a) = 1 + A0m1 + A1 a + A2 a^2 + a^3/6 + a^4/24,
// with shell coefficients A0m1, A1, A2 (functions of |u*|^2 and theta).
// collide^T needs, per shell, sum lambda P, sum e lambda dP/da, and
// sum lambda dP/d|u|^2, sum lambda dP/dtheta.  Opposite hops l, l' share the
// shell and have a_l' = -a_l, so each polynomial splits into an even part
// (shared) and an odd part (sign flipped): a pair contributes through
// lambda_l + lambda_l' and lambda_l - lambda_l' only, and every polynomial is
// evaluated once per pair.  Shell coefficients are formed shell by shell
// (populations are ordered by shell), so only one shell's worth is live.
__host__ __device__ __forceinline__ double adjoint_site(double m0, double sx, double sy, double s2, double Lg,
                                                        double (&lam)[NPOP], const AdjArgs& a)
{
    using K = ShellK<double>;
    const AdjSite q = adj_site_scalars(m0, sx, sy, s2, a);
    double SP = 0.0, Sax = 0.0, Say = 0.0, Su2 = 0.0, Sth = 0.0;
#pragma unroll
    for (int s = 0; s < NSHELL; ++s) {
        const double A0m1 = q.u2 * (-0.5 + 0.125 * q.u2) + q.th * (K::k1(s) + q.u2 * K::k2(s) + q.th * K::k3(s));
        const double A1 = 1.0 - 0.5 * q.u2 + q.th * K::k4(s);
        const double A2 = 0.5 - 0.25 * q.u2 + q.th * K::k5(s);
        const double dA0du2 = -0.5 + 0.25 * q.u2 + q.th * K::k2(s);
        const double dA0dth = K::k1(s) + q.u2 * K::k2(s) + 2.0 * q.th * K::k3(s);
        double sP = 0.0, sax = 0.0, say = 0.0, su2 = 0.0, sth = 0.0;
#pragma unroll
        for (int l = 0; l < NPOP; ++l) {
            if (SHELL[l] != s) continue;
            if (l == 0) {
                sP += lam[0] * (1.0 + A0m1);
                su2 += lam[0] * dA0du2;
                sth += lam[0] * dA0dth;
                continue;
            }
            const int m = OPP.v[l];
            if (m < l) continue;                 // each pair once, from its first hop
            const double av = hop_dot<double>(l, q.cux, q.cuy);
            const double a2 = av * av;
            const double sg = lam[l] + lam[m], dl = lam[l] - lam[m];
            // even and odd parts of P, dP/da, dP/d|u|^2, dP/dtheta
            const double PE = (1.0 + A0m1) + a2 * (A2 + a2 * (1.0 / 24.0));
            const double PO = av * (A1 + a2 * (1.0 / 6.0));
            const double DE = A1 + 0.5 * a2;
            const double DO = av * (2.0 * A2 + a2 * (1.0 / 6.0));
            sP += sg * PE + dl * PO;
            const double Z = dl * DE + sg * DO;   // sum over the pair of sign(e) lambda dP/da
            if (EX[l] != 0) sax += (double)EX[l] * Z;
            if (EY[l] != 0) say += (double)EY[l] * Z;
            su2 += sg * (dA0du2 - 0.25 * a2) - 0.5 * (dl * av);
            sth += sg * (dA0dth + K::k5(s) * a2) + K::k4(s) * (dl * av);
        }
        const double ws = W_SHELL[s];
        SP += ws * sP;
        Sax += ws * sax;
        Say += ws * say;
        Su2 += ws * su2;
        Sth += ws * sth;
    }
    const double om = a.omega;
    const double bux = om * q.rho * (C * Sax + 2.0 * q.ux * Su2);
    const double buy = om * q.rho * (C * Say + 2.0 * q.uys * Su2);
    const double bth = om * q.rho * Sth;
    const double bP = om * SP;
    // sum_l lambda_l (f^eq_l - g_l) = rho SP - Lg
    const double D = q.rho * SP - Lg;
    const double dtau = -om * om * D + buy * a.gy + bth * (1.0 - 2.0 * a.tau) * a.gy * a.gy * 0.5;
    const double buxt = bux - bth * q.ux, buyt = buy - bth * q.uy;
    const double bE = 0.5 * bth * q.inv;
    const double bjx = buxt * q.inv, bjy = buyt * q.inv;
    const double brho = bP - (buxt * q.ux + buyt * q.uy) * q.inv - 0.5 * bth * q.E * q.inv * q.inv;
    const double cjx = C * bjx, cjy = C * bjy, c2E = C2 * bE;
    // mu_l = (1 - 1/tau) lambda_l + brho + xi_l . bj + |xi_l|^2 bE: the |e|^2
    // part is shared by a pair, the e part flips sign
    lam[0] = (1.0 - om) * lam[0] + brho;
#pragma unroll
    for (int l = 1; l < NPOP; ++l) {
        const int m = OPP.v[l];
        if (m < l) continue;
        const double even = brho + (double)R2_OF(l) * c2E;
        double odd = 0.0;
        if (EX[l] != 0) odd += (double)EX[l] * cjx;
        if (EY[l] != 0) odd += (double)EY[l] * cjy;
        const double ll = lam[l], lm = lam[m];
        lam[l] = (1.0 - om) * ll + (even + odd);
        lam[m] = (1.0 - om) * lm + (even - odd);
    }
    return dtau;
}

// One block sum of a double into partials[blockIdx linear].
template <int T = SITE_THREADS>
__device__ __forceinline__ void block_sum1(double v, double* __restrict__ partials, bool add = false)
{
    double a[1] = {v};
    block_sum_store<1, T>(a, partials + (size_t)blockIdx.y * gridDim.x + blockIdx.x, add);
}

// Threads per block of the reverse step: 256 with FP64 lambda, 64 with FP32
// lambda, where the smaller blocks ran 2.4% (2048x4096), 6% (1024x2048) and
// 8% (512x512) faster over FP32 states; with FP64 lambda they ran 1% slower.
template <typename L>
constexpr int adj_threads() { return sizeof(L) == 4 ? 64 : SITE_THREADS; }
// With FP64 lambda too, small blocks on lattices that few_rows_fill names (us
// per reverse step, FP64 / FP32 states: 211x333 17.6 / 15.6 with 256 threads,
// 14.5 / 13.1 with 64; 301x1030 51.5 / 43.8 and 50.7 / 43.8; with nothing to
// fill, 256x256 13.0 / 11.7 and 14.8 / 13.5).

// WALL_HOP.of[l]: the hop of WH that population l (e_y != 0) is at its wall
struct WallHopOf { int of[NPOP]; };
constexpr WallHopOf make_wall_hop_of()
{
    WallHopOf t{};
    for (int j = 0; j < NWS; ++j) t.of[WH.bot[j]] = t.of[WH.top[j]] = j;
    return t;
}
constexpr WallHopOf WALL_HOP = make_wall_hop_of();

// lambda_{n+1} at site (x, y) (see the header): from a buffer that holds mu
// of the later step (GATHER), or lambda itself at each site (after a seed or
// an explicit set).  Loads are unconditional: in the three rows next to a
// wall the e_y-shifted ones reach into the ghost rows, and those values are
// replaced by 0 in mend_lambda, with the mu of the wall slots that mirror onto
// the site, which are read here: 15 loads in flight behind the others.
template <typename L> struct WallMu { L mu[NWS]; };
template <typename L, bool WALLS, bool GATHER>
__device__ __forceinline__ void load_lambda(const L* __restrict__ buf, const Geo& lg, int x, int y, double (&lam)[NPOP],
                                            WallMu<L>& wm)
{
    const unsigned yd = (unsigned)y * (unsigned)sizeof(L);
    const L* col[7];   // columns x - 3 .. x + 3, at the running population
#pragma unroll
    for (int k = 0; k < 7; ++k) col[k] = buf + lg.origin + (long long)(GATHER ? wrap_x(x + k - 3, lg.lx) : x) * lg.cs;
    unsigned yp[7];    // byte offsets of rows y - 3 .. y + 3 of a lattice without walls
#pragma unroll
    for (int k = 0; k < 7; ++k) yp[k] = (unsigned)wrap_x(y + k - 3, lg.ly) * (unsigned)sizeof(L);
    const int r = y < 3 ? y : lg.ly - 1 - y;   // rows from the wall
    const bool near = WALLS && GATHER && r < 3;
    long long lo = 0;
#pragma unroll
    for (int l = 0; l < NPOP; ++l) {
        const L* p = col[GATHER ? 3 + EX[l] : 3] + lo;
        if (!GATHER) lam[l] = (double)ld_at(p, yd);
        else lam[l] = (double)(WALLS ? ld_at(p + EY[l], yd) : ld_at(p, yp[3 + EY[l]]));
        lo += lg.ps;
        asm volatile("" : "+s"(lo));   // one running offset, not 37 column addresses
    }
    if (near) {
        // the slot's row mirrors onto this one: en - 1 - r rows from the wall
        if (y < 3) {
#pragma unroll
            for (int j = 0; j < NWS; ++j)
                wm.mu[j] = ld_at(col[3 + WH.ex[j]] + WH.bot[j] * lg.ps, (unsigned)max(WH.en[j] - 1 - r, 0) * (unsigned)sizeof(L));
        } else {
#pragma unroll
            for (int j = 0; j < NWS; ++j)
                wm.mu[j] = ld_at(col[3 + WH.ex[j]] + WH.top[j] * lg.ps,
                                 (unsigned)(lg.ly - 1 - max(WH.en[j] - 1 - r, 0)) * (unsigned)sizeof(L));
        }
    }
}
// the wall W's part, r rows from it: populations from beyond the wall are 0,
// and the wall slots that mirror onto the site act on its density
template <typename L, int W>
__device__ __forceinline__ void mend_lambda(double (&lam)[NPOP], int r, const WallTable& wt, const WallMu<L>& wm)
{
    double beta = 0.0;
#pragma unroll
    for (int l = 0; l < NPOP; ++l) {
        if (EY[l] == 0) continue;
        const int en = W == 0 ? EY[l] : -EY[l];      // hop component into the lattice
        if (en < 0) {
            lam[l] = -en > r ? 0.0 : lam[l];         // from beyond the wall
        } else {
            L mu = wm.mu[WALL_HOP.of[l]];
            asm volatile("" : "+v"(mu));             // waited for and converted here
            const double b = fma_(wt.ew[W][l], (double)mu, beta);
            beta = en > r ? b : beta;
        }
    }
#pragma unroll
    for (int l = 0; l < NPOP; ++l) lam[l] += beta;
}
template <typename L, bool WALLS, bool GATHER>
__device__ __forceinline__ void mend_lambda(double (&lam)[NPOP], int y, int ly, const WallTable& wt, const WallMu<L>& wm)
{
    if (!(WALLS && GATHER)) return;
    if (y < 3) mend_lambda<L, 0>(lam, y, wt, wm);
    else if (y >= ly - 3) mend_lambda<L, 1>(lam, ly - 1 - y, wt, wm);
}

// One reverse step at site (x, y): lambda_{n+1} (load_lambda), the gather
// g = bc(propagate(f_n)) of the snapshot f_n, collide^T, and mu stored at the
// site (aligned streaming stores); the block's d/dtau term goes to its slot of
// partials (add: added to the slot, which then sums the terms of many steps).
//
// HBM bounds it on large lattices (2048 x 4096, FP32 states: 5.9 TB/s with
// FP64 lambda); below, the latency of its loads, of which 168 registers (three
// waves per SIMD) hold both gathers.  The waves at a wall read the wall rule's
// densities and mirrored mu together: as each was used, one latency each, they
// held up the whole launch (us per step, before and after, with the column
// addresses as one running offset: FP32 states and FP64 lambda 256x256 16.5 ->
// 11.6, 512x512 44.3 -> 35.9, 1024x1024 184 -> 145; both FP64 512x512 48.5 -> 43.6,
// 1024x2048 341 -> 334; both FP32 512x512 32.3 -> 26.5, 1024x2048 179 -> 170).
template <typename S, typename L, bool WALLS, bool GATHER, int T = adj_threads<L>(), StoreKind ST = STORE_DEV>
__global__ __launch_bounds__(T, 3) void k_adj_collide(
    const S* __restrict__ fn, Geo g, const L* __restrict__ lam_in, L* __restrict__ mu_out, Geo lg,
    AdjArgs a, const double* __restrict__ wall_rho, WallTable wt, double* __restrict__ partials, int add)
{
    const SiteBlock sb = site_block<true, T>(g);
    const int x = sb.x, y = sb.y;
    double dtau = 0.0;
    if (y < g.ly) {
        using Cc = typename Store<S>::C;
        const unsigned yb = (unsigned)y * (unsigned)sizeof(S);
        const unsigned yd = (unsigned)y * (unsigned)sizeof(L);
        double lam[NPOP];
        WallMu<L> wm;
        load_lambda<L, WALLS, GATHER>(lam_in, lg, x, y, lam, wm);
        // FP64 states leave no registers for the wall's part beside both gathers
        constexpr bool EARLY = sizeof(S) == 8;
        if (EARLY) mend_lambda<L, WALLS, GATHER>(lam, y, g.ly, wt, wm);
        // the raw gather of f_n (storage precision; unconditional -- wall
        // slots read ghost rows and are replaced below)
        const int r = y < 3 ? y : g.ly - 1 - y;   // rows from the wall
        const bool near = WALLS && r < 3;
        Cc gl[NPOP];
        {
            const S* col[7];   // columns x - 3 .. x + 3, at the running population
#pragma unroll
            for (int k = 0; k < 7; ++k) col[k] = fn + g.origin + (long long)wrap_x(x + k - 3, g.lx) * g.cs;
            unsigned yp[7];    // byte offsets of rows y - 3 .. y + 3 of a lattice without walls
#pragma unroll
            for (int k = 0; k < 7; ++k) yp[k] = (unsigned)wrap_x(y + k - 3, g.ly) * (unsigned)sizeof(S);
            long long lo = 0;
#pragma unroll
            for (int l = 0; l < NPOP; ++l) {
                const S* p = col[3 - EX[l]] + lo;
                gl[l] = (Cc)(WALLS ? ld_at(p - EY[l], yb) : ld_at(p, yp[3 - EY[l]]));
                lo += g.ps;
                asm volatile("" : "+s"(lo));
            }
        }
        // raw moments of g and Lg = sum_l lambda_l g_l, in FP64
        double m0 = 0.0, sx = 0.0, sy = 0.0, s2 = 0.0, Lg = 0.0;
        auto add = [&](int l, double v) {
            m0 += v;
            if (EX[l] != 0) sx += (double)EX[l] * v;
            if (EY[l] != 0) sy += (double)EY[l] * v;
            if (R2_OF(l) != 0) s2 += (double)R2_OF(l) * v;
            Lg += lam[l] * v;
        };
        auto raw = [&](int l) {
            asm volatile("" : "+v"(gl[l]));   // converted where it is used, not for both branches ahead
            return Store<S>::shifted ? (double)gl[l] + W_SHELL[SHELL[l]] : (double)gl[l];
        };
        if (near) {
            if (!EARLY) mend_lambda<L, WALLS, GATHER>(lam, y, g.ly, wt, wm);
            const int W = y < 3 ? 0 : 1;
            const double* w0 = wall_rho + W * 3 * g.lx;
            constexpr int CH = EARLY ? 13 : NPOP;   // populations whose densities are in flight together
#pragma unroll
            for (int c = 0; c < NPOP; c += CH) {
                __builtin_amdgcn_sched_barrier(0);
                double d[CH];
#pragma unroll
                for (int l = c; l < c + CH && l < NPOP; ++l)
                    if (EY[l] != 0) {
                        const int en = EY[l] > 0 ? EY[l] : -EY[l];
                        d[l - c] = w0[max(en - 1 - r, 0) * g.lx + wrap_x(x - EX[l], g.lx)];
                    }
#pragma unroll
                for (int l = c; l < c + CH && l < NPOP; ++l) {
                    double v = raw(l);
                    if (EY[l] != 0) {
                        const int w = EY[l] > 0 ? 0 : 1, en = w == 0 ? EY[l] : -EY[l];
                        v = W == w && en > r ? wt.ew[w][l] * d[l - c] : v;
                    }
                    add(l, v);
                }
            }
        } else {
#pragma unroll
            for (int l = 0; l < NPOP; ++l) add(l, raw(l));
        }
        dtau = adjoint_site(m0, sx, sy, s2, Lg, lam, a);
        L* mcol = mu_out + lg.origin + (long long)x * lg.cs;
#pragma unroll
        for (int l = 0; l < NPOP; ++l) st_stream<ST>(mcol + (size_t)l * lg.ps, yd, (L)lam[l]);
    }
    block_sum1<T>(dtau, partials, add != 0);
}

// lambda_l = d(x,y) dT/df_l = d (|xi_l - u|^2 - 2T) / (2 rho), with
// d = dT(x,y) (SEED) or d = T - T_target (LOSS, plus 1/2 d^2 into partials).
template <typename S, typename L, bool LOSS>
__global__ __launch_bounds__(SITE_THREADS) void k_adj_seed_T(const S* __restrict__ fbuf, Geo g, L* __restrict__ lam, Geo lg,
                                                          const double* __restrict__ d_in, double* __restrict__ partials)
{
    const SiteBlock sb = site_block(g);
    const int x = sb.x, y = sb.y;
    double loss = 0.0;
    if (y < g.ly) {
        double rho, ux, uy, T;
        site_macros<S>(fbuf + g.origin + (long long)x * g.cs, (unsigned)y * (unsigned)sizeof(S), g.ps, rho, ux, uy, T);
        double d = d_in[(long long)x * g.ly + y];
        if (LOSS) { d = T - d; loss = 0.5 * d * d; }
        const double k = d / (2.0 * rho);
        L* lp = lam + lg.origin + (long long)x * lg.cs + y;
#pragma unroll
        for (int l = 0; l < NPOP; ++l) {
            const double dx = C * EX[l] - ux, dy = C * EY[l] - uy;
            lp[(size_t)l * lg.ps] = (L)(k * (dx * dx + dy * dy - 2.0 * T));
        }
    }
    if (LOSS) block_sum1(loss, partials);
}

// dL/dP from lambda_0 for f_0 = f^eq(rho0(P), 0, T0(P)):
//   T0 = t_mid - t_amp tanh(z), z = (y - y_mid - P) / width, rho0 = p0 / T0,
//   f^eq_l(rho, 0, T) = w_l rho (1 + th K1 + th^2 K3), th = T - 1.
template <typename L, bool WALLS, bool GATHER>
__global__ __launch_bounds__(SITE_THREADS) void k_adj_init_rt(const L* __restrict__ lam_buf, Geo lg, WallTable wt,
                                                           const double* __restrict__ P, RtProfile pr, double* __restrict__ dP)
{
    using K = ShellK<double>;
    const SiteBlock sb = site_block(lg);
    const int x = sb.x, y = sb.y;
    if (y >= lg.ly) return;
    const long long s = (long long)x * lg.ly + y;
    const double th_z = tanh((y - pr.y_mid - P[s]) / pr.width);
    const double T0 = pr.t_mid - pr.t_amp * th_z;
    const double r0 = pr.p0 / T0;
    const double dT = pr.t_amp * (1.0 - th_z * th_z) / pr.width;
    const double dr = -pr.p0 / (T0 * T0) * dT;
    const double th = T0 - 1.0;
    double lam[NPOP];
    WallMu<L> wm;
    load_lambda<L, WALLS, GATHER>(lam_buf, lg, x, y, lam, wm);
    mend_lambda<L, WALLS, GATHER>(lam, y, lg.ly, wt, wm);
    double acc = 0.0;
#pragma unroll
    for (int l = 0; l < NPOP; ++l) {
        const int sh = SHELL[l];
        const double Pl = 1.0 + th * (K::k1(sh) + th * K::k3(sh));
        const double dPl = K::k1(sh) + 2.0 * th * K::k3(sh);
        acc += lam[l] * W_SHELL[sh] * (Pl * dr + r0 * dPl * dT);
    }
    dP[s] = acc;
}

// the canonical array of a lambda that was never seeded
__global__ __launch_bounds__(256) void k_zero(double* __restrict__ p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0.0;
}

// lambda (load_lambda) -> canonical FP64 [37][lx][ly], one thread per site
template <typename L, bool WALLS, bool GATHER>
__global__ __launch_bounds__(SITE_THREADS) void k_lambda_to_canon(const L* __restrict__ buf, Geo lg, WallTable wt,
                                                               double* __restrict__ canon)
{
    const SiteBlock sb = site_block(lg);
    const int x = sb.x, y = sb.y;
    if (y >= lg.ly) return;
    double lam[NPOP];
    WallMu<L> wm;
    load_lambda<L, WALLS, GATHER>(buf, lg, x, y, lam, wm);
    mend_lambda<L, WALLS, GATHER>(lam, y, lg.ly, wt, wm);
#pragma unroll
    for (int l = 0; l < NPOP; ++l) canon[((size_t)l * lg.lx + x) * lg.ly + y] = lam[l];
}

// canonical FP64 [37][lx][ly] -> lambda at each site of a padded buffer of type L
template <typename L>
__global__ __launch_bounds__(256) void k_lambda_from_canon(L* __restrict__ buf, const double* __restrict__ canon, Geo g)
{
    const int nyb = (g.ly + 255) / 256;
    const int l = blockIdx.y, x = (int)(blockIdx.x / (unsigned)nyb);
    const int y = (int)(blockIdx.x % (unsigned)nyb) * 256 + threadIdx.x;
    if (y >= g.ly) return;
    buf[(size_t)l * g.ps + g.origin + (long long)x * g.cs + y] = (L)canon[((size_t)l * g.lx + x) * g.ly + y];
}

}  // namespace lbm
