// lbm_api.hip -- host side of liblbm.so: the C ABI declared in include/lbm.h.
//
// The context keeps only host metadata; every byte of device memory the
// library uses is carved out of the caller's workspace (see plan()).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>

#include "lbm.h"
#include "lbm_rollout.h"
#include "lbm_adjoint.hpp"
#include "lbm_kernels.hpp"
#include "lbm_twostep.hpp"

using namespace lbm;

namespace {

constexpr size_t ALIGN = 256;
constexpr size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Plan {
    Geo geo;          // population buffers, storage precision
    Geo lgeo;         // adjoint lambda buffers, FP64
    size_t elem;      // bytes per stored population value
    size_t buf_bytes; // one population buffer
    size_t wall_bytes;// one wall-density table (6 * lx doubles)
    size_t state_bytes; // snapshot: population buffer + its wall densities
    size_t off_buf[2];
    size_t off_wall;  // 3 x 6 * lx doubles (double-buffered wall densities, and those of the state in between), and a word
    size_t off_part;  // RED_BLOCKS * 4 doubles, then 2 doubles of loss/dtau scratch
    size_t off_lam[2];
    size_t off_apart; // adjoint: one double per collide block
    size_t off_adacc; // adjoint: per-block sums of deferred d/dtau terms
    size_t total;
};

Geo make_geo(int lx, int ly, size_t elem, int layout) { return padded_geo(lx, ly, elem, layout == LBM_LAYOUT_PLANES); }

bool valid(const lbm_params* p)
{
    if (!p) return false;
    if (p->lx < 7 || p->ly < 7) return false;
    if (!(p->tau > 0.5) || !std::isfinite(p->tau) || !std::isfinite(p->g_y)) return false;
    if (p->precision != LBM_FP64 && p->precision != LBM_FP32_SHIFTED && p->precision != LBM_FP32_SHIFTED_F32SUMS)
        return false;
    if (p->ybc != LBM_Y_WALLS && p->ybc != LBM_Y_PERIODIC) return false;
    if (p->xmode != LBM_X_WRAP && p->xmode != LBM_X_HALO) return false;
    if (p->step_kind != LBM_STEP_SPLIT && p->step_kind != LBM_STEP_FUSED) return false;
    if (p->layout != LBM_LAYOUT_PLANES && p->layout != LBM_LAYOUT_COLUMNS) return false;
    if (p->adjoint < 0 || p->adjoint > 2) return false;
    if ((long long)p->lx * p->ly > (1LL << 31)) return false;
    return true;
}

Plan plan(const lbm_params* p)
{
    Plan pl{};
    pl.elem = p->precision == LBM_FP64 ? 8 : 4;
    pl.geo = make_geo(p->lx, p->ly, pl.elem, p->layout);
    pl.lgeo = make_geo(p->lx, p->ly, p->adjoint == 2 ? 4 : 8, p->layout);
    pl.buf_bytes = align_up((size_t)pl.geo.total * pl.elem, ALIGN);
    pl.wall_bytes = align_up(6 * (size_t)p->lx * 8, ALIGN);
    pl.state_bytes = pl.buf_bytes + pl.wall_bytes;
    size_t off = 0;
    pl.off_buf[0] = off; off += pl.buf_bytes;
    pl.off_buf[1] = off; off += pl.buf_bytes;
    pl.off_wall = off; off += 3 * pl.wall_bytes + ALIGN;
    pl.off_part = off; off += align_up(((size_t)RED_BLOCKS * 4 + 2) * 8, ALIGN);
    if (p->adjoint) {
        const size_t lb = align_up((size_t)pl.lgeo.total * (p->adjoint == 2 ? 4 : 8), ALIGN);
        pl.off_lam[0] = off; off += lb;
        pl.off_lam[1] = off; off += lb;
        // one partial per block of the reverse step (its blocks are the
        // smallest of the adjoint launches)
        const int at = p->adjoint == 2 ? adj_threads<float>()
                                       : (few_rows_fill(p->ly) ? SMALL_THREADS : adj_threads<double>());
        const size_t nb = (size_t)((p->ly + at - 1) / at) * p->lx;
        pl.off_apart = off; off += align_up(nb * 8, ALIGN);
        pl.off_adacc = off; off += align_up(nb * 8, ALIGN);
    }
    pl.total = off;
    return pl;
}

thread_local std::string g_create_error;

}  // namespace

struct lbm_ctx {
    lbm_params p;
    Plan pl;
    char* ws;
    hipStream_t stream;
    int cur;           // current population buffer
    // the other buffer holds the state before the last propagate, except after a
    // pass of two steps: that state's wall densities are in table WALL_MID then
    // (set_mid_word)
    bool have_prev;
    int lam_cur;
    bool have_lambda;
    // lambda buffer lam_cur holds mu of the last reverse step (lambda is its
    // propagate^T + bc^T gather) rather than lambda itself
    bool lam_is_mu;
    // wall densities (rows 0..2 and ly-3..ly-1) of population buffer wr_buf
    // (-1: none) live in wall table wr_cur; the other table receives the
    // densities the next collide or fused step writes
    int wr_cur;
    int wr_buf;
    WallTable wt;
    CollideArgs cargs;
    unsigned fused_lds;  // dynamic LDS of the fused step's launch (occupancy cap; 0: none)
    int fused_threads;   // threads per block of the FP64 fused step (64, 256 or 512)
    unsigned collide_lds;// the same for the split step's collide
    bool dev_stores;     // fused and reverse steps with device-scope stores (dev_stores_for)
    StoreKind adj_stores; // kind of the reverse step's stores
    bool adj_small;      // reverse step with FP64 lambda in 64-thread blocks
    TwoStep two;         // how lbm_step takes two steps in one pass (fused step, wrapped index)
    std::string err;

    void* buf(int i) { return ws + pl.off_buf[i]; }
    double* wall_rho(int i) { return reinterpret_cast<double*>(ws + pl.off_wall + i * pl.wall_bytes); }
    static constexpr int WALL_MID = 2;
    // the table of the states in between, and the word behind it; NULL where no
    // pass takes two steps or there are no walls
    double* wall_mid() { return two.kind != TWO_STEP_NONE && p.ybc == LBM_Y_WALLS ? wall_rho(WALL_MID) : nullptr; }
    bool mid_may_be_set;  // the word may be 1: a pass of two steps has run since it was last cleared ...
    bool two_captured;    // ... or may run at any time
    double* mid_word() { return wall_mid() ? wall_mid() + 6 * (size_t)p.lx : nullptr; }
    double* partials() { return reinterpret_cast<double*>(ws + pl.off_part); }
    double* scratch2() { return partials() + (size_t)RED_BLOCKS * 4; }
    template <typename L> L* lam(int i) { return reinterpret_cast<L*>(ws + pl.off_lam[i]); }
    bool fp64() const { return p.precision == LBM_FP64; }
    bool f32_sums() const { return p.precision == LBM_FP32_SHIFTED_F32SUMS; }
    bool lam32() const { return p.adjoint == 2; }
};

namespace {

lbm_status fail(lbm_ctx* c, lbm_status s, const char* what)
{
    c->err = what;
    return s;
}

lbm_status check_launch(lbm_ctx* c, const char* what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        c->err = std::string(what) + ": " + hipGetErrorString(e);
        return LBM_ERR_HIP;
    }
    return LBM_OK;
}

void set_collide_args(lbm_ctx* c)
{
    const double tau = c->p.tau, g = c->p.g_y;
    c->cargs.omega = 1.0 / tau;
    c->cargs.tau_g = tau * g;
    c->cargs.grav_th = tau * (1.0 - tau) * g * g / 2.0;
    c->cargs.g = g;
    c->cargs.g_over_c = g / C;
    c->cargs.g_f = (float)g;
    c->cargs.omega_f = (float)c->cargs.omega;
    c->cargs.tau_g_f = (float)c->cargs.tau_g;
    c->cargs.grav_th_f = (float)c->cargs.grav_th;
}

// 1-D grid of site blocks, renumbered per XCD inside the kernels (site_block)
dim3 site_grid(const Geo& g) { return dim3((unsigned)((g.ly + SITE_THREADS - 1) / SITE_THREADS) * (unsigned)g.lx); }

template <typename S, bool CACHED>
lbm_status launch_propagate_kind(lbm_ctx* c, const S* src, S* dst)
{
    const Geo& g = c->pl.geo;
    constexpr int VEC = sizeof(S) == 8 ? 2 : 4;
    constexpr int UNROLL = PROP_UNROLL;
    constexpr int CH = PROP_THREADS * VEC * UNROLL;
    const size_t nch = (size_t)((g.ly + CH - 1) / CH);
    const size_t nblk = nch * NPOP * (size_t)g.lx;
    if (nblk > 0xffffffffull) return fail(c, LBM_ERR_SIZE, "propagate: lattice too large for one grid");
    const unsigned gx = nblk < PROP_GRID_X ? (unsigned)nblk : PROP_GRID_X;
    const dim3 grid(gx, (unsigned)((nblk + gx - 1) / gx));
    const bool cols = c->p.layout == LBM_LAYOUT_COLUMNS;
    const bool wrap = c->p.xmode == LBM_X_WRAP;
    const unsigned nb = (unsigned)nblk;
    if (wrap && cols)
        hipLaunchKernelGGL((k_propagate<S, VEC, UNROLL, true, true, CACHED>), grid, dim3(PROP_THREADS), 0, c->stream, src, dst, g,
                           nb);
    else if (wrap)
        hipLaunchKernelGGL((k_propagate<S, VEC, UNROLL, true, false, CACHED>), grid, dim3(PROP_THREADS), 0, c->stream, src, dst, g,
                           nb);
    else if (cols)
        hipLaunchKernelGGL((k_propagate<S, VEC, UNROLL, false, true, CACHED>), grid, dim3(PROP_THREADS), 0, c->stream, src, dst, g,
                           nb);
    else
        hipLaunchKernelGGL((k_propagate<S, VEC, UNROLL, false, false, CACHED>), grid, dim3(PROP_THREADS), 0, c->stream, src, dst, g,
                           nb);
    return check_launch(c, "propagate");
}
// the split step's kernels with cached loads and stores
bool split_cached(const lbm_ctx* c)
{
    const size_t both = 2 * c->pl.buf_bytes;
    return both >= SPLIT_CACHED_MIN_BYTES && both <= CACHED_STORES_MAX_BYTES;
}
template <typename S>
lbm_status launch_propagate(lbm_ctx* c, const S* src, S* dst)
{
    return split_cached(c) ? launch_propagate_kind<S, true>(c, src, dst) : launch_propagate_kind<S, false>(c, src, dst);
}

template <typename S>
lbm_status launch_pre_stream(lbm_ctx* c, S* src, bool ghosts)
{
    // halos the pull of the current buffer needs: y ghost rows if periodic
    // and asked for, then x halo columns (whole padded columns, so corners
    // follow).
    const Geo& g = c->pl.geo;
    if (ghosts && c->p.ybc == LBM_Y_PERIODIC) {
        dim3 grid((g.lx * 3 + 255) / 256, NPOP);
        hipLaunchKernelGGL((k_fill_y_ghosts<S>), grid, dim3(256), 0, c->stream, src, g);
        lbm_status s = check_launch(c, "fill_y_ghosts");
        if (s) return s;
    }
    if (c->p.xmode == LBM_X_HALO) {
        dim3 grid((g.lyp + 255) / 256, 3, NPOP);
        hipLaunchKernelGGL((k_fill_x_halo<S>), grid, dim3(256), 0, c->stream, src, g);
        lbm_status s = check_launch(c, "fill_x_halo");
        if (s) return s;
    }
    return LBM_OK;
}

template <typename S>
lbm_status launch_wall_density(lbm_ctx* c, const S* src, double* out)
{
    const Geo& g = c->pl.geo;
    hipLaunchKernelGGL((k_wall_density<S>), dim3((6 * g.lx + WALL_DENSITY_THREADS - 1) / WALL_DENSITY_THREADS),
                       dim3(WALL_DENSITY_THREADS), 0, c->stream, src, g, out);
    return check_launch(c, "wall_density");
}

// Makes wall table wr_cur hold the wall densities of population buffer b.
template <typename S>
lbm_status ensure_wall_density(lbm_ctx* c, int b)
{
    if (c->wr_buf == b) return LBM_OK;
    lbm_status s = launch_wall_density<S>(c, (const S*)c->buf(b), c->wall_rho(c->wr_cur));
    if (s) return s;
    c->wr_buf = b;
    return LBM_OK;
}

bool capturing(lbm_ctx* c)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) (void)hipGetLastError();
    return st != hipStreamCaptureStatusNone;
}

template <typename S>
lbm_status do_propagate(lbm_ctx* c)
{
    S* src = (S*)c->buf(c->cur);
    S* dst = (S*)c->buf(1 - c->cur);
    lbm_status s = launch_pre_stream<S>(c, src, true);
    if (s) return s;
    if (c->mid_word()) {
        const bool cap = capturing(c);   // passes of two steps may run before a replay
        if (cap || c->mid_may_be_set) {
            hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, c->stream, c->mid_word(), (size_t)1);
            s = check_launch(c, "propagate");
            if (s) return s;
        }
        if (!cap) c->mid_may_be_set = c->two_captured;
    }
    s = launch_propagate<S>(c, src, dst);
    if (s) return s;
    if (c->wr_buf == 1 - c->cur) c->wr_buf = -1;   // destination overwritten
    c->cur = 1 - c->cur;
    c->have_prev = true;
    return LBM_OK;
}

template <typename S>
lbm_status do_bc(lbm_ctx* c)
{
    if (c->p.ybc == LBM_Y_PERIODIC) return LBM_OK;
    if (!c->have_prev) return fail(c, LBM_ERR_STATE, "bc: no propagate since the state was set");
    const Geo& g = c->pl.geo;
    lbm_status s = ensure_wall_density<S>(c, 1 - c->cur);
    if (s) return s;
    hipLaunchKernelGGL((k_bc_apply<S>), dim3((NSLOT * g.lx + 255) / 256), dim3(256), 0, c->stream,
                       (S*)c->buf(c->cur), g, (const double*)c->wall_rho(c->wr_cur), (const double*)c->wall_mid(), c->wt);
    return check_launch(c, "bc_apply");
}

// In-place collide of the current buffer; wo receives the wall densities
// (WALLS) -- FP32 storage with FP32 sums takes the WIDE = false kernels.
template <typename S, bool WALLS, bool WIDE>
void launch_collide_wide(lbm_ctx* c, double* wo)
{
    const Geo& g = c->pl.geo;
    if (split_cached(c))
        hipLaunchKernelGGL((k_collide<S, WALLS, WIDE, true>), site_grid(g), dim3(SITE_THREADS), 0, c->stream,
                           (S*)c->buf(c->cur), g, c->cargs, wo);
    else
        hipLaunchKernelGGL((k_collide<S, WALLS, WIDE, false>), site_grid(g), dim3(SITE_THREADS), c->collide_lds, c->stream,
                           (S*)c->buf(c->cur), g, c->cargs, wo);
}
template <typename S, bool WALLS>
void launch_collide(lbm_ctx* c, double* wo)
{
    if constexpr (std::is_same<S, float>::value) {
        if (c->f32_sums()) {
            launch_collide_wide<S, WALLS, false>(c, wo);
            return;
        }
    }
    launch_collide_wide<S, WALLS, true>(c, wo);
}

template <typename S>
lbm_status do_collide(lbm_ctx* c)
{
    if (c->p.ybc == LBM_Y_WALLS) {
        launch_collide<S, true>(c, c->wall_rho(1 - c->wr_cur));
        lbm_status s = check_launch(c, "collide");
        if (s) return s;
        c->wr_cur = 1 - c->wr_cur;
        c->wr_buf = c->cur;
        return LBM_OK;
    }
    launch_collide<S, false>(c, (double*)nullptr);
    return check_launch(c, "collide");
}

// One fused step src -> dst (wall densities read from wr, written to wo),
// T threads per block, stores of kind ST.
template <typename S, bool WIDE, int T, StoreKind ST>
void launch_fused_kernel(lbm_ctx* c, const S* src, S* dst, const double* wr, double* wo, double* mid_word)
{
    const Geo& g = c->pl.geo;
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    const bool wrap = c->p.xmode == LBM_X_WRAP;
    const unsigned lds = sizeof(S) == 8 ? c->fused_lds : 0u;
    const dim3 grid((unsigned)((g.ly + T - 1) / T) * (unsigned)g.lx);
    if (wrap && walls)
        hipLaunchKernelGGL((k_step_fused<S, true, true, WIDE, T, ST>), grid, dim3(T), lds, c->stream, src, dst, g,
                           c->cargs, wr, c->wt, wo, mid_word);
    else if (wrap)
        hipLaunchKernelGGL((k_step_fused<S, true, false, WIDE, T, ST>), grid, dim3(T), lds, c->stream, src, dst, g,
                           c->cargs, wr, c->wt, wo, mid_word);
    else if (walls)
        hipLaunchKernelGGL((k_step_fused<S, false, true, WIDE, T, ST>), grid, dim3(T), lds, c->stream, src, dst, g,
                           c->cargs, wr, c->wt, wo, mid_word);
    else
        hipLaunchKernelGGL((k_step_fused<S, false, false, WIDE, T, ST>), grid, dim3(T), lds, c->stream, src, dst, g,
                           c->cargs, wr, c->wt, wo, mid_word);
}

// buffers: population buffers that a run of such steps goes through; mid_word:
// NULL for a step between snapshots
template <typename S>
void launch_fused(lbm_ctx* c, const S* src, S* dst, const double* wr, double* wo, int buffers, double* mid_word)
{
    const StoreKind st = store_kind_for(c->dev_stores, (size_t)buffers * c->pl.buf_bytes, STEP_CACHED_MIN_BYTES);
#define FUSED(WIDE, T)                                                                              \
    (st == STORE_CACHED ? launch_fused_kernel<S, WIDE, T, STORE_CACHED>(c, src, dst, wr, wo, mid_word) \
     : st == STORE_NT   ? launch_fused_kernel<S, WIDE, T, STORE_NT>(c, src, dst, wr, wo, mid_word)   \
                        : launch_fused_kernel<S, WIDE, T, STORE_DEV>(c, src, dst, wr, wo, mid_word))
    if constexpr (std::is_same<S, float>::value) {
        if (c->f32_sums()) FUSED(false, SITE_THREADS);
        else FUSED(true, SITE_THREADS);
    } else if (c->fused_threads == FUSED_FP64_WIDE_THREADS) {   // beyond the caches
        if (st == STORE_DEV) launch_fused_kernel<S, true, FUSED_FP64_WIDE_THREADS, STORE_DEV>(c, src, dst, wr, wo, mid_word);
        else launch_fused_kernel<S, true, FUSED_FP64_WIDE_THREADS, STORE_NT>(c, src, dst, wr, wo, mid_word);
    } else if (c->fused_threads == SMALL_THREADS) {             // below device-scope stores
        if (st == STORE_CACHED) launch_fused_kernel<S, true, SMALL_THREADS, STORE_CACHED>(c, src, dst, wr, wo, mid_word);
        else launch_fused_kernel<S, true, SMALL_THREADS, STORE_NT>(c, src, dst, wr, wo, mid_word);
    } else {
        FUSED(true, SITE_THREADS);
    }
#undef FUSED
}

template <typename S>
lbm_status do_step_fused(lbm_ctx* c)
{
    S* src = (S*)c->buf(c->cur);
    S* dst = (S*)c->buf(1 - c->cur);
    lbm_status s = launch_pre_stream<S>(c, src, false);
    if (s) return s;
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    if (walls) {
        s = ensure_wall_density<S>(c, c->cur);
        if (s) return s;
    }
    launch_fused<S>(c, src, dst, c->wall_rho(c->wr_cur), c->wall_rho(1 - c->wr_cur), 2, c->mid_word());
    s = check_launch(c, "step_fused");
    if (s) return s;
    c->cur = 1 - c->cur;
    c->have_prev = true;
    if (walls) {
        c->wr_cur = 1 - c->wr_cur;
        c->wr_buf = c->cur;
    }
    return LBM_OK;
}

// Two fused steps in one pass, current buffer -> the other (lbm_twostep.hpp).
template <typename S, bool WALLS, bool WIDE>
void launch_two_step(lbm_ctx* c, const S* src, S* dst, const double* wr, double* mid, double* wo)
{
    const Geo& g = c->pl.geo;
    auto tiles = [&](int tx, int ty) { return dim3((unsigned)(((g.lx + tx - 1) / tx) * ((g.ly + ty - 1) / ty))); };
    switch (c->two.kind) {
    case TWO_STEP_TILE_8X8:
        hipLaunchKernelGGL((k_twostep_tile<S, WALLS, WIDE, 8, 8>), tiles(8, 8), dim3(tile_threads<8, 8>()), 0, c->stream,
                           src, dst, g, c->cargs, wr, c->wt, mid, wo);
        break;
    case TWO_STEP_TILE_8X16:
        hipLaunchKernelGGL((k_twostep_tile<S, WALLS, WIDE, 8, 16>), tiles(8, 16), dim3(tile_threads<8, 16>()), 0,
                           c->stream, src, dst, g, c->cargs, wr, c->wt, mid, wo);
        break;
    case TWO_STEP_TILE_16X16:
        hipLaunchKernelGGL((k_twostep_tile<S, WALLS, WIDE, 16, 16>), tiles(16, 16), dim3(tile_threads<16, 16>()), 0,
                           c->stream, src, dst, g, c->cargs, wr, c->wt, mid, wo);
        break;
    default:
        hipLaunchKernelGGL((k_twostep_march<S, WALLS, WIDE>), dim3((unsigned)c->two.march.nblk),
                           dim3(2 * MarchShape<S>::waves * 64), 0, c->stream, src, dst, g, c->cargs, wr, c->wt, mid, wo,
                           c->two.march);
    }
}

template <typename S>
lbm_status launch_two_steps(lbm_ctx* c, const S* src, S* dst, const double* wr, double* wo)
{
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    double* mid = c->wall_rho(lbm_ctx::WALL_MID);
    c->mid_may_be_set = true;
    if constexpr (std::is_same<S, float>::value) {
        if (c->f32_sums()) {
            if (walls) launch_two_step<S, true, false>(c, src, dst, wr, mid, wo);
            else launch_two_step<S, false, false>(c, src, dst, wr, mid, wo);
        } else {
            if (walls) launch_two_step<S, true, true>(c, src, dst, wr, mid, wo);
            else launch_two_step<S, false, true>(c, src, dst, wr, mid, wo);
        }
    } else {
        if (walls) launch_two_step<S, true, true>(c, src, dst, wr, mid, wo);
        else launch_two_step<S, false, true>(c, src, dst, wr, mid, wo);
    }
    return check_launch(c, "two_steps");
}

template <typename S>
lbm_status do_two_steps(lbm_ctx* c)
{
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    if (walls) {
        lbm_status s = ensure_wall_density<S>(c, c->cur);
        if (s) return s;
    }
    const lbm_status s = launch_two_steps<S>(c, (const S*)c->buf(c->cur), (S*)c->buf(1 - c->cur), c->wall_rho(c->wr_cur),
                                             c->wall_rho(1 - c->wr_cur));
    if (s) return s;
    c->cur = 1 - c->cur;
    c->have_prev = true;
    if (walls) {
        c->wr_cur = 1 - c->wr_cur;
        c->wr_buf = c->cur;
    }
    return LBM_OK;
}

template <typename S>
lbm_status do_step(lbm_ctx* c, int64_t n)
{
    // Passes of two steps go in pairs, so that every four steps end on the
    // buffers they began with, as four single steps do (a graph of an even
    // number of steps can then be replayed).
    if (c->p.step_kind == LBM_STEP_FUSED && c->two.kind != TWO_STEP_NONE && n >= 4) {
        c->two_captured = c->two_captured || capturing(c);
        for (; n >= 4; n -= 4) {
            lbm_status s = do_two_steps<S>(c);
            if (!s) s = do_two_steps<S>(c);
            if (s) return s;
        }
    }
    for (int64_t i = 0; i < n; ++i) {
        lbm_status s;
        if (c->p.step_kind == LBM_STEP_FUSED) {
            s = do_step_fused<S>(c);
        } else {
            s = do_propagate<S>(c);
            if (!s) s = do_bc<S>(c);
            if (!s) s = do_collide<S>(c);
        }
        if (s) return s;
    }
    return LBM_OK;
}

#define DISPATCH(c, fn, ...) ((c)->fp64() ? fn<double>(c, ##__VA_ARGS__) : fn<float>(c, ##__VA_ARGS__))
// storage type S and adjoint-state type L
#define ADJ_DISPATCH(c, fn, ...)                                                                \
    ((c)->fp64() ? ((c)->lam32() ? fn<double, float>(c, ##__VA_ARGS__) : fn<double, double>(c, ##__VA_ARGS__)) \
                 : ((c)->lam32() ? fn<float, float>(c, ##__VA_ARGS__) : fn<float, double>(c, ##__VA_ARGS__)))
#define LAM_DISPATCH(c, fn, ...) ((c)->lam32() ? fn<float>(c, ##__VA_ARGS__) : fn<double>(c, ##__VA_ARGS__))

// Copies take non-temporal accesses from this many bytes on: source and
// destination then exceed the 256 MB Infinity Cache.  301 x 1030 FP64 (99 MB)
// took 29 us without and 32 us with them, 1000 x 1501 FP32 (233 MB) 90 and 72.
constexpr size_t COPY_NT_MIN_BYTES = 128u << 20;

// Kernels that only read or only write a population buffer take non-temporal
// accesses where the 64-byte pieces of its sites are well beyond the Infinity
// Cache.  us without and with them, sites' pieces in MB (10^6 bytes): init FP64
// 20000x33 (237) 55 / 69, 950x950 (270) 46 / 54, 17x60000 (302) 49 / 56, 1050x1000
// (311) 57 / 56, 1100x1000 (326) 67 / 58, 1024x2048 (621) 170 / 127; FP32, whose
// short rows leave most of a line unwritten, 100000x7 (237) 97 / 153, 60000x17
// (284) 80 / 140, 200000x7 (474) 338 / 306; macros FP64 950x950 45 / 52, 1050x1000 62
// / 58.
constexpr size_t STREAM_NT_MIN_BYTES = 300u << 20;
bool streamed(const Geo& g, size_t elem)
{
    return NPOP * (size_t)g.lx * align_up((size_t)g.ly * elem, 64) >= STREAM_NT_MIN_BYTES;
}

// the state was set, with its wall densities where there are walls
void state_initialised(lbm_ctx* c)
{
    c->have_prev = false;
    c->wr_buf = c->p.ybc == LBM_Y_WALLS ? c->cur : -1;
}
template <typename S>
lbm_status do_init(lbm_ctx* c, const double* rho, const double* ux, const double* uy, const double* T)
{
    double* wr = c->p.ybc == LBM_Y_WALLS ? c->wall_rho(c->wr_cur) : nullptr;
    if (streamed(c->pl.geo, sizeof(S)))
        hipLaunchKernelGGL((k_init_fields<S, true>), site_grid(c->pl.geo), dim3(SITE_THREADS), 0, c->stream,
                           (S*)c->buf(c->cur), c->pl.geo, rho, ux, uy, T, wr);
    else
        hipLaunchKernelGGL((k_init_fields<S, false>), site_grid(c->pl.geo), dim3(SITE_THREADS), 0, c->stream,
                           (S*)c->buf(c->cur), c->pl.geo, rho, ux, uy, T, wr);
    state_initialised(c);
    return check_launch(c, "init");
}
template <typename S>
lbm_status do_init_rt(lbm_ctx* c, const double* P, RtProfile pr)
{
    double* wr = c->p.ybc == LBM_Y_WALLS ? c->wall_rho(c->wr_cur) : nullptr;
    if (streamed(c->pl.geo, sizeof(S)))
        hipLaunchKernelGGL((k_init_rt<S, true>), site_grid(c->pl.geo), dim3(SITE_THREADS), 0, c->stream,
                           (S*)c->buf(c->cur), c->pl.geo, P, pr, wr);
    else
        hipLaunchKernelGGL((k_init_rt<S, false>), site_grid(c->pl.geo), dim3(SITE_THREADS), 0, c->stream,
                           (S*)c->buf(c->cur), c->pl.geo, P, pr, wr);
    state_initialised(c);
    return check_launch(c, "init_rt");
}
template <typename S>
lbm_status do_macros(lbm_ctx* c, double* rho, double* ux, double* uy, double* T)
{
    if (streamed(c->pl.geo, sizeof(S)))
        hipLaunchKernelGGL((k_macros<S, true>), site_grid(c->pl.geo), dim3(SITE_THREADS), 0, c->stream,
                           (const S*)c->buf(c->cur), c->pl.geo, rho, ux, uy, T);
    else
        hipLaunchKernelGGL((k_macros<S, false>), site_grid(c->pl.geo), dim3(SITE_THREADS), 0, c->stream,
                           (const S*)c->buf(c->cur), c->pl.geo, rho, ux, uy, T);
    return check_launch(c, "macros");
}
template <typename S, bool TO_CANON, bool NT>
void launch_canon(lbm_ctx* c, S* canon)
{
    const Geo& g = c->pl.geo;
    constexpr int VEC = 16 / (int)sizeof(S);
    const int nv = (g.ly + VEC - 1) / VEC;
    int lts = 0;
    while (lts < 8 && (1 << lts) < nv) ++lts;
    const int waves = (nv + 63) / 64;
    const unsigned nch = (unsigned)((waves + CANON_THREADS / 64 - 1) / (CANON_THREADS / 64));
    // chunks of a long segment in as few waves as its vectors fill
    const int threads = nch == 1 ? CANON_THREADS : (waves + (int)nch - 1) / (int)nch * 64;
    const size_t spb = nch == 1 ? (size_t)CANON_THREADS >> lts : 1;
    const size_t nblk = (((size_t)NPOP * g.lx + spb - 1) / spb) * nch;
    const unsigned gx = nblk < PROP_GRID_X ? (unsigned)nblk : PROP_GRID_X;
    const dim3 grid(gx, (unsigned)((nblk + gx - 1) / gx));
    // segments in the order of the array that is written
    if (!TO_CANON && c->p.layout == LBM_LAYOUT_COLUMNS)
        hipLaunchKernelGGL((k_canon_copy<S, TO_CANON, true, NT>), grid, dim3(threads), 0, c->stream,
                           (S*)c->buf(c->cur), canon, g, lts, nch, (unsigned)nblk);
    else
        hipLaunchKernelGGL((k_canon_copy<S, TO_CANON, false, NT>), grid, dim3(threads), 0, c->stream,
                           (S*)c->buf(c->cur), canon, g, lts, nch, (unsigned)nblk);
}
template <typename S>
lbm_status do_canon(lbm_ctx* c, void* canon, bool to_canon)
{
    const bool nt = c->pl.buf_bytes >= COPY_NT_MIN_BYTES;
    if (to_canon && nt) launch_canon<S, true, true>(c, (S*)canon);
    else if (to_canon) launch_canon<S, true, false>(c, (S*)canon);
    else if (nt) launch_canon<S, false, true>(c, (S*)canon);
    else launch_canon<S, false, false>(c, (S*)canon);
    if (!to_canon) {
        c->have_prev = false;
        c->wr_buf = -1;
    }
    return check_launch(c, "canonical copy");
}
// Copies a population buffer and (walls) its wall densities, nw bytes.
lbm_status copy_state(lbm_ctx* c, const void* buf, void* to_buf, const void* wall, void* to_wall, size_t nw, const char* what)
{
    const size_t na = c->pl.buf_bytes;
    // the runtime's copy for a snapshot at an odd address (buf_bytes is a multiple of
    // 256), and where it is one copy within the caches (us, it and the kernel: FP64
    // without walls 64x64 3.8 and 4.2, 513x513 24.1 and 24.6, 700x700 63.5 and 48.6;
    // with walls, two copies, 64x64 6.2 and 4.1)
    if (((uintptr_t)buf | (uintptr_t)to_buf) % 16 || (!nw && na < COPY_NT_MIN_BYTES)) {
        if (hipMemcpyAsync(to_buf, buf, na, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
            (nw && hipMemcpyAsync(to_wall, wall, nw, hipMemcpyDeviceToDevice, c->stream) != hipSuccess))
            return check_launch(c, what);
        return LBM_OK;
    }
    const size_t nblk = ((na + nw) / 16 + STATE_THREADS - 1) / STATE_THREADS;
    const unsigned gx = nblk < PROP_GRID_X ? (unsigned)nblk : PROP_GRID_X;
    const dim3 grid(gx, (unsigned)((nblk + gx - 1) / gx));
    if (na >= COPY_NT_MIN_BYTES)
        hipLaunchKernelGGL((k_state_copy<true>), grid, dim3(STATE_THREADS), 0, c->stream, (const v16_t*)buf, (v16_t*)to_buf,
                           na / 16, (const v16_t*)wall, (v16_t*)to_wall, nw / 16);
    else
        hipLaunchKernelGGL((k_state_copy<false>), grid, dim3(STATE_THREADS), 0, c->stream, (const v16_t*)buf,
                           (v16_t*)to_buf, na / 16, (const v16_t*)wall, (v16_t*)to_wall, nw / 16);
    return check_launch(c, what);
}
// snapshot = current population buffer + its wall densities (walls only)
template <typename S>
lbm_status do_get_state(lbm_ctx* c, char* dst)
{
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    if (walls) {
        lbm_status s = ensure_wall_density<S>(c, c->cur);
        if (s) return s;
    }
    return copy_state(c, c->buf(c->cur), dst, c->wall_rho(c->wr_cur), dst + c->pl.buf_bytes, walls ? c->pl.wall_bytes : 0,
                      "get_state");
}

// A chain of steps through snapshots goes through more buffers than two: counted
// as four for the kind of its stores (us per step of a chain through four,
// non-temporal / cached: FP32 512x512 15.8 / 14.2, 768x768 33.1 / 35.2, FP64 512x512
// 26.2 / 27.9).
constexpr int CHAIN_BUFFERS = 4;

// One fused step from snapshot src into snapshot dst (both buffer + wall
// densities); the context's own buffers and wall tables are not touched.
template <typename S>
lbm_status do_step_state(lbm_ctx* c, char* src, char* dst)
{
    S* sb = (S*)src;
    S* db = (S*)dst;
    lbm_status s = launch_pre_stream<S>(c, sb, false);   // padding of the source only
    if (s) return s;
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    const double* wr = walls ? (const double*)(src + c->pl.buf_bytes) : nullptr;
    double* wo = walls ? (double*)(dst + c->pl.buf_bytes) : nullptr;
    launch_fused<S>(c, sb, db, wr, wo, CHAIN_BUFFERS, nullptr);
    return check_launch(c, "step_state");
}

// n fused steps (n >= 1) from snapshot src, or the current state if NULL, into
// snapshot dst, or the current state if NULL: the first pass reads src and the
// last writes dst, so a snapshot at either end costs no copy (1024 x 2048 FP32:
// 110 us each).  The passes between use the context's buffers, and passes of two
// steps its table WALL_MID, so lbm_bc is refused until a state precedes the
// current one again.
template <typename S>
lbm_status do_advance_state(lbm_ctx* c, char* src, char* dst, int64_t n)
{
    c->have_prev = false;
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    S* sb = src ? (S*)src : (S*)c->buf(c->cur);
    const double* wr = src ? (const double*)(src + c->pl.buf_bytes) : c->wall_rho(c->wr_cur);
    if (!src && walls) {
        lbm_status s = ensure_wall_density<S>(c, c->cur);
        if (s) return s;
        wr = c->wall_rho(c->wr_cur);
    }
    while (n > 0) {
        const int k = n >= 2 && c->two.kind != TWO_STEP_NONE ? 2 : 1;
        const bool out = dst && n == k;
        const int b = 1 - c->cur, w = 1 - c->wr_cur;
        S* db = out ? (S*)dst : (S*)c->buf(b);
        double* wo = out ? (double*)(dst + c->pl.buf_bytes) : c->wall_rho(w);
        lbm_status s = LBM_OK;
        if (k == 2) {
            s = launch_two_steps<S>(c, sb, db, wr, wo);
        } else {
            s = launch_pre_stream<S>(c, sb, false);
            if (s) return s;
            launch_fused<S>(c, sb, db, wr, wo, src || dst ? CHAIN_BUFFERS : 2, nullptr);
            s = check_launch(c, "advance_state");
        }
        if (s) return s;
        n -= k;
        if (out) break;
        c->cur = b;
        c->wr_cur = w;
        c->wr_buf = walls ? b : -1;
        sb = db;
        wr = wo;
    }
    return LBM_OK;
}

template <typename S>
void launch_conservation_partial(const Geo& g, const S* buf, double* part, hipStream_t st)
{
    if (g.ly % 64 == 0 && streamed(g, sizeof(S)))
        hipLaunchKernelGGL((k_conservation_partial<S, true>), dim3(RED_BLOCKS), dim3(256), 0, st, buf, g, part);
    else
        hipLaunchKernelGGL((k_conservation_partial<S, false>), dim3(RED_BLOCKS), dim3(256), 0, st, buf, g, part);
}

template <typename S>
lbm_status do_conservation(lbm_ctx* c, double* out4)
{
    launch_conservation_partial<S>(c->pl.geo, (const S*)c->buf(c->cur), c->partials(), c->stream);
    lbm_status s = check_launch(c, "conservation");
    if (s) return s;
    hipLaunchKernelGGL((k_reduce_partials<4, false>), dim3(1), dim3(REDUCE_THREADS), 0, c->stream,
                       c->partials(), RED_BLOCKS, out4);
    return check_launch(c, "conservation reduce");
}
}  // namespace

// ----------------------------------------------------------------------------
// Scratch of lbm_conservation_noalloc: the reduction's block partials
// (RED_BLOCKS x 4 doubles, 32 KiB) in a fixed device array instead of a
// workspace.  In host code `scratch` names a host-side stand-in, not device
// memory: its device address is looked up once per device with
// hipGetSymbolAddress (that device current) and only that address reaches
// kernels.  Every call on one device shares the array.
// ----------------------------------------------------------------------------
static __device__ __align__(256) double scratch[RED_BLOCKS * 4];

namespace {

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[NOALLOC_MAX_DEVICES];   // device address of `scratch`, per device

// Device address of `scratch` on the current device (looked up on the first
// call there).
lbm_status scratch_on_current_device(double** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= NOALLOC_MAX_DEVICES) {
        g_create_error = "conservation_noalloc: no usable current device";
        return LBM_ERR_HIP;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            g_create_error = std::string("conservation_noalloc: hipGetSymbolAddress: ") + hipGetErrorString(e);
            return LBM_ERR_HIP;
        }
        g_scratch_dev[dev] = static_cast<double*>(p);
    }
    *out = g_scratch_dev[dev];
    return LBM_OK;
}

// Geometry of a canonical [37][lx][ly] array: no padding, no halos.
Geo canonical_geo(int lx, int ly)
{
    Geo g{};
    g.lx = lx;
    g.ly = ly;
    g.lyp = ly;
    g.g = 0;
    g.cs = ly;
    g.ps = (long long)lx * ly;
    g.origin = 0;
    g.total = NPOP * g.ps;
    return g;
}

template <typename S>
lbm_status launch_conservation_noalloc(const Geo& g, const void* pops, double* part, double* out4, hipStream_t st)
{
    launch_conservation_partial<S>(g, (const S*)pops, part, st);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL((k_reduce_partials<4, false>), dim3(1), dim3(REDUCE_THREADS), 0, st,
                           part, RED_BLOCKS, out4);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        g_create_error = std::string("conservation_noalloc: ") + hipGetErrorString(e);
        return LBM_ERR_HIP;
    }
    return LBM_OK;
}

}  // namespace

// ============================================================================
// C ABI
// ============================================================================
extern "C" {

size_t lbm_workspace_bytes(const lbm_params* p) { return valid(p) ? plan(p).total : 0; }

size_t lbm_state_bytes(const lbm_params* p) { return valid(p) ? plan(p).state_bytes : 0; }

lbm_status lbm_create(const lbm_params* p, void* dev_workspace, size_t bytes, void* hip_stream, lbm_ctx** out)
{
    if (!out) { g_create_error = "out is NULL"; return LBM_ERR_INVALID; }
    *out = nullptr;
    if (!valid(p)) { g_create_error = "invalid parameters"; return LBM_ERR_INVALID; }
    Plan pl = plan(p);
    if (!dev_workspace) { g_create_error = "workspace is NULL"; return LBM_ERR_INVALID; }
    if ((uintptr_t)dev_workspace % ALIGN) { g_create_error = "workspace not 256-byte aligned"; return LBM_ERR_INVALID; }
    if (bytes < pl.total) { g_create_error = "workspace too small"; return LBM_ERR_SIZE; }
    lbm_ctx* c = new lbm_ctx();
    c->p = *p;
    c->pl = pl;
    c->ws = (char*)dev_workspace;
    c->stream = (hipStream_t)hip_stream;
    c->cur = 0;
    c->have_prev = false;
    c->lam_cur = 0;
    c->have_lambda = false;
    c->lam_is_mu = false;
    c->wr_cur = 0;
    c->wr_buf = -1;
    for (int l = 0; l < NPOP; ++l) {
        c->wt.ew[0][l] = feq_pop<false>(l, 1.0, 0.0, 0.0, p->t_bottom);
        c->wt.ew[1][l] = feq_pop<false>(l, 1.0, 0.0, 0.0, p->t_top);
        c->wt.w[l] = W_SHELL[SHELL[l]];
    }
    set_collide_args(c);
    // occupancy caps of the FP64 fused step and of the collide on large
    // lattices (lbm_kernels.hpp)
    c->fused_lds = 0;
    c->fused_threads = SITE_THREADS;
    c->collide_lds = 0;
    c->dev_stores = false;
    c->two = TwoStep{TWO_STEP_NONE, MarchLaunch{}};
    c->mid_may_be_set = false;
    c->two_captured = false;
    int dev = 0, ncu = 0, max_lds = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && ncu > 0) {
        const FusedLaunch fl = fused_fp64_launch(site_grid(pl.geo).x, ncu, max_lds);
        c->fused_threads = fl.threads;
        c->fused_lds = fl.lds;
        c->dev_stores = dev_stores_for(site_grid(pl.geo).x, ncu);
        if (fl.lds == 0 && !c->dev_stores && few_rows_fill(p->ly)) c->fused_threads = SMALL_THREADS;
        if (p->step_kind == LBM_STEP_FUSED)
            c->two = p->precision == LBM_FP64
                         ? choose_two_step<double>(pl.geo, ncu, max_lds, p->ybc == LBM_Y_WALLS, false)
                         : choose_two_step<float>(pl.geo, ncu, max_lds, p->ybc == LBM_Y_WALLS, c->f32_sums());
        if ((size_t)site_grid(pl.geo).x >= (size_t)FUSED_FP64_CAP_MIN_BLOCKS_PER_CU * (size_t)ncu) {
            const unsigned coll = p->precision == LBM_FP64 ? COLLIDE_FP64_LDS_RESERVE : COLLIDE_FP32_LDS_RESERVE;
            if ((size_t)max_lds >= coll && (p->precision != LBM_FP64 || p->layout == LBM_LAYOUT_COLUMNS))
                c->collide_lds = coll;
        }
    }
    c->adj_stores = store_kind_for(c->dev_stores, pl.buf_bytes + 2 * (pl.off_lam[1] - pl.off_lam[0]), ADJ_CACHED_MIN_BYTES);
    c->adj_small = p->adjoint == 1 && !c->dev_stores && few_rows_fill(p->ly);
    // Everything but the adjoint state, whose sites a seed or a set writes first
    // and whose padding no result depends on (512 x 512 with FP64 lambda: 78 of
    // 234 MB, 16 us of 48).  In stream order; a context cannot be created in a
    // capture.
    const size_t lam0 = p->adjoint ? pl.off_lam[0] : pl.total, lam1 = p->adjoint ? pl.off_apart : pl.total;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone ||
        hipMemsetAsync(c->ws, 0, lam0, c->stream) != hipSuccess ||
        (lam1 < pl.total && hipMemsetAsync(c->ws + lam1, 0, pl.total - lam1, c->stream) != hipSuccess)) {
        g_create_error = "workspace initialisation failed";
        delete c;
        return LBM_ERR_HIP;
    }
    *out = c;
    return LBM_OK;
}

void lbm_destroy(lbm_ctx* ctx) { delete ctx; }

lbm_status lbm_set_tau(lbm_ctx* c, double tau)
{
    if (!c) return LBM_ERR_INVALID;
    if (!(tau > 0.5) || !std::isfinite(tau)) return fail(c, LBM_ERR_INVALID, "tau must be > 0.5");
    c->p.tau = tau;
    set_collide_args(c);
    return LBM_OK;
}


lbm_status lbm_init(lbm_ctx* c, const double* rho, const double* ux, const double* uy, const double* T)
{
    if (!c) return LBM_ERR_INVALID;
    if (!rho || !ux || !uy || !T) return fail(c, LBM_ERR_INVALID, "init: NULL field");
    return DISPATCH(c, do_init, rho, ux, uy, T);
}

lbm_status lbm_init_rt(lbm_ctx* c, const double* P, const lbm_rt_profile* prof)
{
    if (!c) return LBM_ERR_INVALID;
    if (!P || !prof) return fail(c, LBM_ERR_INVALID, "init_rt: NULL argument");
    if (!(prof->width > 0.0) || !(prof->p0 > 0.0)) return fail(c, LBM_ERR_INVALID, "init_rt: width and p0 must be > 0");
    RtProfile pr{prof->t_mid, prof->t_amp, prof->p0, prof->width, prof->y_mid};
    return DISPATCH(c, do_init_rt, P, pr);
}

lbm_status lbm_propagate(lbm_ctx* c)
{
    if (!c) return LBM_ERR_INVALID;
    return DISPATCH(c, do_propagate);
}

lbm_status lbm_bc(lbm_ctx* c)
{
    if (!c) return LBM_ERR_INVALID;
    return DISPATCH(c, do_bc);
}

lbm_status lbm_collide(lbm_ctx* c)
{
    if (!c) return LBM_ERR_INVALID;
    return DISPATCH(c, do_collide);
}

lbm_status lbm_step(lbm_ctx* c, int64_t n)
{
    if (!c) return LBM_ERR_INVALID;
    if (n < 0) return fail(c, LBM_ERR_INVALID, "step: n < 0");
    return DISPATCH(c, do_step, n);
}

lbm_status lbm_get_macros(lbm_ctx* c, double* rho, double* ux, double* uy, double* T)
{
    if (!c) return LBM_ERR_INVALID;
    if (!rho || !ux || !uy || !T) return fail(c, LBM_ERR_INVALID, "get_macros: NULL field");
    return DISPATCH(c, do_macros, rho, ux, uy, T);
}

lbm_status lbm_get_pops(lbm_ctx* c, void* dst)
{
    if (!c) return LBM_ERR_INVALID;
    if (!dst) return fail(c, LBM_ERR_INVALID, "get_pops: NULL");
    return DISPATCH(c, do_canon, dst, true);
}

lbm_status lbm_set_pops(lbm_ctx* c, const void* src)
{
    if (!c) return LBM_ERR_INVALID;
    if (!src) return fail(c, LBM_ERR_INVALID, "set_pops: NULL");
    return DISPATCH(c, do_canon, const_cast<void*>(src), false);
}

lbm_status lbm_get_state(lbm_ctx* c, void* dst)
{
    if (!c) return LBM_ERR_INVALID;
    if (!dst) return fail(c, LBM_ERR_INVALID, "get_state: NULL");
    return DISPATCH(c, do_get_state, (char*)dst);
}

lbm_status lbm_set_state(lbm_ctx* c, const void* src)
{
    if (!c) return LBM_ERR_INVALID;
    if (!src) return fail(c, LBM_ERR_INVALID, "set_state: NULL");
    const char* s = (const char*)src;
    const bool walls = c->p.ybc == LBM_Y_WALLS;
    lbm_status st = copy_state(c, s, c->buf(c->cur), s + c->pl.buf_bytes, c->wall_rho(c->wr_cur),
                               walls ? c->pl.wall_bytes : 0, "set_state");
    if (st) return st;
    c->have_prev = false;
    c->wr_buf = walls ? c->cur : -1;
    return LBM_OK;
}

lbm_status lbm_step_state(lbm_ctx* c, void* src_state, void* dst_state)
{
    if (!c) return LBM_ERR_INVALID;
    if (!src_state || !dst_state) return fail(c, LBM_ERR_INVALID, "step_state: NULL");
    if (((uintptr_t)src_state | (uintptr_t)dst_state) % ALIGN != 0)
        return fail(c, LBM_ERR_INVALID, "step_state: snapshots must be 256-byte aligned");
    const char* a = (const char*)src_state;
    const char* b = (const char*)dst_state;
    const size_t n = c->pl.state_bytes;
    if (a < b + n && b < a + n) return fail(c, LBM_ERR_INVALID, "step_state: snapshots overlap");
    return DISPATCH(c, do_step_state, (char*)src_state, (char*)dst_state);
}

lbm_status lbm_advance_state(lbm_ctx* c, void* src_state, void* dst_state, int64_t n)
{
    if (!c) return LBM_ERR_INVALID;
    if (n < 1) return fail(c, LBM_ERR_INVALID, "advance_state: n < 1");
    if (((uintptr_t)src_state | (uintptr_t)dst_state) % ALIGN != 0)
        return fail(c, LBM_ERR_INVALID, "advance_state: snapshots must be 256-byte aligned");
    const char* a = (const char*)src_state;
    const char* b = (const char*)dst_state;
    const size_t sz = c->pl.state_bytes;
    if (a && b && a < b + sz && b < a + sz) return fail(c, LBM_ERR_INVALID, "advance_state: snapshots overlap");
    return DISPATCH(c, do_advance_state, (char*)src_state, (char*)dst_state, n);
}

lbm_two_step lbm_two_step_form(const lbm_ctx* c)
{
    switch (c ? c->two.kind : TWO_STEP_NONE) {
    case TWO_STEP_TILE_8X8: return LBM_TWO_STEP_TILE_8X8;
    case TWO_STEP_TILE_8X16: return LBM_TWO_STEP_TILE_8X16;
    case TWO_STEP_TILE_16X16: return LBM_TWO_STEP_TILE_16X16;
    case TWO_STEP_MARCH: return LBM_TWO_STEP_MARCH;
    default: return LBM_TWO_STEP_NONE;
    }
}

lbm_status lbm_conservation(lbm_ctx* c, double* dev_out4)
{
    if (!c) return LBM_ERR_INVALID;
    if (!dev_out4) return fail(c, LBM_ERR_INVALID, "conservation: NULL");
    return DISPATCH(c, do_conservation, dev_out4);
}

lbm_status lbm_conservation_noalloc(int precision, int lx, int ly, const void* pops, double* dev_out4,
                                    void* hip_stream)
{
    if (precision != LBM_FP64 && precision != LBM_FP32_SHIFTED && precision != LBM_FP32_SHIFTED_F32SUMS) {
        g_create_error = "conservation_noalloc: unknown precision";
        return LBM_ERR_INVALID;
    }
    if (lx < 1 || ly < 1) {
        g_create_error = "conservation_noalloc: lx and ly must be >= 1";
        return LBM_ERR_INVALID;
    }
    if ((long long)lx * ly > LBM_NOALLOC_MAX_SITES) {
        g_create_error = "conservation_noalloc: lattice exceeds LBM_NOALLOC_MAX_SITES (2^31) sites";
        return LBM_ERR_SIZE;
    }
    if (!pops || !dev_out4) {
        g_create_error = "conservation_noalloc: NULL pointer";
        return LBM_ERR_INVALID;
    }
    double* part = nullptr;
    lbm_status s = scratch_on_current_device(&part);
    if (s) return s;
    const Geo g = canonical_geo(lx, ly);
    const hipStream_t st = (hipStream_t)hip_stream;
    return precision == LBM_FP64 ? launch_conservation_noalloc<double>(g, pops, part, dev_out4, st)
                                 : launch_conservation_noalloc<float>(g, pops, part, dev_out4, st);
}

lbm_status lbm_sync(lbm_ctx* c)
{
    if (!c) return LBM_ERR_INVALID;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        c->err = std::string("sync: ") + hipGetErrorString(e);
        return LBM_ERR_HIP;
    }
    return LBM_OK;
}

const char* lbm_last_error(const lbm_ctx* c) { return c ? c->err.c_str() : g_create_error.c_str(); }

void lbm_velocity_table(int8_t ex[LBM_NPOP], int8_t ey[LBM_NPOP])
{
    for (int l = 0; l < NPOP; ++l) { ex[l] = (int8_t)EX[l]; ey[l] = (int8_t)EY[l]; }
}

void lbm_weights(double w[LBM_NPOP])
{
    for (int l = 0; l < NPOP; ++l) w[l] = W_SHELL[SHELL[l]];
}

double lbm_scale_c(void) { return C; }

}  // extern "C"

#include "lbm_adjoint_api.inc"
#include "lbm_layouts_api.inc"
#include "lbm_hetero_api.inc"
