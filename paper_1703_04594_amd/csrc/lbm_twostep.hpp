// lbm_twostep.hpp -- two time steps per pass over memory (gfx950).
//
// A single fused step reads and writes every population once (592 B per site
// in FP64) and runs at the speed of that traffic.  A pass here takes a state
// two steps on for the same traffic: the first step of a block's sites, and of
// the three rows and columns around them that the second step's hops reach, is
// collided into LDS; the second step gathers from there.  The populations in
// between never leave the CU.  What LDS holds is stored by destination: for
// every population the value of each site that will pull it, so no value is
// kept that the block does not use.
//
// Two forms (choose_two_step picks one for a lattice):
//  - tiles: a block per tile of the lattice.  All sites of the first step run
//    at once, then all of the second.  The ring around a tile is stepped twice
//    by neighbouring blocks (1.9x the first step's work for a 16 x 16 tile),
//    but a pass is one short launch: the form of small lattices.
//  - march: a block per segment of a strip of rows; it walks along x, a column
//    at a time, and keeps only the last columns of the step in between (four
//    per population on average, as hop e_x needs e_x + 4).  Half of its waves
//    run the first step, half the second, three columns behind.  Only the
//    strip's six outer rows and six columns per segment are stepped twice: the
//    form of large lattices.
//
// Both evaluate the expressions of the single step in its order, wall rule
// included, so n steps are bitwise those of n single steps.
#pragma once

#include <type_traits>

#include "lbm_kernels.hpp"

namespace lbm {

// Populations grouped by hop: number of populations with hop component ex,
// and the index of population l among those of its group.
constexpr int ex_count(int ex)
{
    int n = 0;
    for (int l = 0; l < NPOP; ++l) n += EX[l] == ex;
    return n;
}
constexpr int ex_rank(int l)
{
    int n = 0;
    for (int k = 0; k < l; ++k) n += EX[k] == EX[l];
    return n;
}

// Buffer accesses: block-uniform base, per-lane and uniform 32-bit byte offsets.
template <typename S>
__device__ __forceinline__ S buf_load(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    if constexpr (sizeof(S) == 4) return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    else return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <typename S, int POL>
__device__ __forceinline__ void buf_store(S v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    if constexpr (sizeof(S) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, POL);
    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, voff, soff, POL);
}
template <typename S>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(S* base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, RAW_BUFFER_ALL_BYTES, RAW_BUFFER_WORD3);
}

// ---------------------------------------------------------------------------
// Tiles.  One thread per site of the first step (the tile and three rows and
// columns around it); the tile's own sites, as many threads, run the second.
// Without walls the gather wraps the row as it does the column, so a pass needs
// no ghost rows.
// What bounds a pass: on the smallest lattices the chain of one load, two
// collisions and an LDS exchange (256 x 128 FP64: 10.3 us per two steps against
// 12.1 in single steps); above, the first step's work on the rings (512 x 512 FP64:
// 33 us against 47, FP32 27.4 against 28.2).
// The buffer accesses keep one SGPR offset running over the populations (with
// 64-bit column addresses 512 x 512 FP64 took 40 us).  The wall densities are read
// ahead of the populations.  Stores are plain: the next pass reads them from the
// caches.  With FP32 sums 80 registers are enough for six waves per SIMD; with
// walls they spill 12 bytes a lane (us per step, five waves without spills / six:
// with walls 128x128 4.43 / 4.61, 384x384 9.55 / 8.79, 640x640 17.1 / 16.8; without
// walls 384x384 9.49 / 8.17).  The FP64 sums would spill 95 registers.
// ---------------------------------------------------------------------------
template <int TX, int TY>
constexpr int tile_threads() { return ((TX + 6) * (TY + 6) + 63) / 64 * 64; }

// The tile kernel's wall table, read from its argument segment where it is
// used: as a plain argument the compiler loads it on entry, in several rounds of
// scalar loads ahead of the gather, and spills it (us per step, as an argument and
// so: FP64 128x128 4.8 and 4.4, 256x256 7.3 and 6.6, FP32 384x384 10.9 and 10.1; the
// single step and the reverse step, which have fewer rounds, gain nothing).  Where
// it lies in the segment follows from the kernel's signature: arguments in order,
// each aligned as its type.
template <typename T, typename... P>
constexpr size_t kernarg_offset(void (*)(P...))
{
    size_t off = 0, at = 0;
    ((off = (off + alignof(P) - 1) / alignof(P) * alignof(P), at = std::is_same<T, P>::value ? off : at, off += sizeof(P)),
     ...);
    return at;
}
typedef const __attribute__((address_space(4))) char* kernarg_t;
typedef const __attribute__((address_space(4))) WallTable wall_table_arg_t;
template <size_t OFFSET>
__device__ __forceinline__ wall_table_arg_t& wall_table_arg()
{
    kernarg_t p = (kernarg_t)__builtin_amdgcn_kernarg_segment_ptr() + OFFSET;
    asm volatile("" : "+s"(p));   // not loaded ahead of this point
    return *(wall_table_arg_t*)p;
}

template <typename S, bool WALLS, bool WIDE, int TX, int TY>
__global__ __launch_bounds__((tile_threads<TX, TY>()), WIDE ? 4 : 6) void k_twostep_tile(
    const S* __restrict__ src, S* __restrict__ dst, Geo g, CollideArgs args, const double* __restrict__ wall_rho,
    WallTable wt, double* __restrict__ wall_mid, double* __restrict__ wall_rho_out)
{
    using Cc = typename Store<S>::C;
    constexpr size_t WT_AT = kernarg_offset<WallTable>((decltype(&k_twostep_tile<S, WALLS, WIDE, TX, TY>))nullptr);
    static_assert(WT_AT != 0, "wt is an argument, and not the first");
    __shared__ S post[NPOP][TX * TY];                // the first step, by the second step's sites
    __shared__ double wr[WALLS ? 6 : 1][TX + 6];     // its wall densities
    const int nty = (g.ly + TY - 1) / TY, ntx = (g.lx + TX - 1) / TX;
    const int L = xcd_block(blockIdx.x, nty * ntx);
    const int x0 = L / nty * TX, y0 = L % nty * TY;
    const int x1 = min(x0 + TX, g.lx), y1 = min(y0 + TY, g.ly);
    const int t = (int)threadIdx.x;
    const int stride = (int)(g.ps * (long long)sizeof(S));   // between populations (the whole buffer is below 2 GB)
    {
        const int ax = t / (TY + 6), ay = t % (TY + 6);
        const int X = x0 - 3 + ax;
        int y = y0 - 3 + ay;
        bool on = ax < TX + 6 && X < x1 + 3;
        if (WALLS) on = on && y >= 0 && y < g.ly;
        else {
            on = on && y < y1 + 3;
            y = y < 0 ? y + g.ly : (y >= g.ly ? y - g.ly : y);
        }
        if (on) {
            Cc f[NPOP];
            int xs[7];   // columns X - 3 .. X + 3
#pragma unroll
            for (int k = 0; k < 7; ++k) xs[k] = wrap_x(X + k - 3, g.lx);
            int ys[7];   // rows y - 3 .. y + 3 of a lattice without walls, as offsets from the base below
#pragma unroll
            for (int k = 0; k < 7; ++k) ys[k] = 3 + wrap_x(y + k - 3, g.ly);
            const __amdgpu_buffer_rsrc_t rs = buf_of(src + g.origin - 3);
            const int r = y < 3 ? y : g.ly - 1 - y;   // rows from the wall
            const bool near = WALLS && r < 3;
            double d[NWS];
            if (near) {   // read ahead of the populations, not behind them
                const double* w0 = wall_rho + (y < 3 ? 0 : 3 * g.lx);
#pragma unroll
                for (int j = 0; j < NWS; ++j) d[j] = w0[max(WH.en[j] - 1 - r, 0) * g.lx + xs[3 - WH.ex[j]]];
            }
            int soff = 0;
#pragma unroll
            for (int l = 0; l < NPOP; ++l) {
                const int row = WALLS ? y + 3 - EY[l] : ys[3 - EY[l]];
                f[l] = (Cc)buf_load<S>(rs, (xs[3 - EX[l]] * (int)g.cs + row) * (int)sizeof(S), soff);
                soff += stride;
            }
            if (near) {
                auto& w = wall_table_arg<WT_AT>();
                if (y < 3) put_wall_slots<S, 0>(f, r, w, d);
                else put_wall_slots<S, 1>(f, r, w, d);
            }
            collide_site<Cc, Store<S>::shifted, WIDE>(f, args);
            const int ox = ax - 3, oy = ay - 3;
            const int p = ox * TY + oy;
#pragma unroll
            for (int l = 0; l < NPOP; ++l)
                if ((unsigned)(ox + EX[l]) < (unsigned)TX && (unsigned)(oy + EY[l]) < (unsigned)TY)
                    post[l][p + EX[l] * TY + EY[l]] = (S)f[l];
            if (near) {
                const double d = stored_density<S>(f);
                const int wk = y < 3 ? r : 3 + r;
                wr[wk][ax] = d;
                if (X >= x0 && X < x1) wall_mid[wk * g.lx + X] = d;
            }
        }
    }
    __syncthreads();
    if (t < TX * TY) {
        const int ox = t / TY, oy = t % TY;
        const int X = x0 + ox, y = y0 + oy;
        if (X < x1 && y < y1) {
            Cc f[NPOP];
#pragma unroll
            for (int l = 0; l < NPOP; ++l) f[l] = (Cc)post[l][t];
            const int r = y < 3 ? y : g.ly - 1 - y;
            const bool near = WALLS && r < 3;
            if (near) {
                const int w0 = WALLS && y >= 3 ? 3 : 0;
                double d[NWS];
#pragma unroll
                for (int j = 0; j < NWS; ++j) d[j] = wr[WALLS ? w0 + max(WH.en[j] - 1 - r, 0) : 0][ox + 3 - WH.ex[j]];
                auto& w = wall_table_arg<WT_AT>();
                if (y < 3) put_wall_slots<S, 0>(f, r, w, d);
                else put_wall_slots<S, 1>(f, r, w, d);
            }
            const __amdgpu_buffer_rsrc_t rs = buf_of(dst + g.origin);
            const int off = (X * (int)g.cs + y) * (int)sizeof(S);
            collide_site<Cc, Store<S>::shifted, WIDE>(f, args);
            int soff = 0;
#pragma unroll
            for (int l = 0; l < NPOP; ++l) {
                buf_store<S, 0>((S)f[l], rs, off, soff);
                soff += stride;
            }
            if (near) wall_rho_out[(y < 3 ? r : 3 + r) * g.lx + X] = stored_density<S>(f);
        }
    }
    if (WALLS) set_mid_word(wall_mid + 6 * g.lx, 1.0);
}

// ---------------------------------------------------------------------------
// March.  Waves 0 .. NW-1 run the first step, one column per iteration, rows
// y0-3 .. y0+ny+2, a lane each; waves NW .. 2 NW - 1 the second step of the
// column three behind.  Population l of the step in between goes into a ring
// of e_x + 4 column segments of LDS (148 segments in all), at the row and
// column that will pull it.  Per iteration there are two barriers: the first
// step stores into the rings only after the second step has read its column
// (barrier 1, right after both have taken their moments), and the second step
// reads only after that (barrier 2).  Behind barrier 1 both waves' relaxation
// loops run side by side; they store each population as it is relaxed.
//
// One wave per SIMD issues an instruction about every 5 cycles, so the column
// after next has to be on its way early and cheaply: the loads of column i + 1
// go out one by one between the collision's instructions of column i (a burst
// of 37 stalled the wave for 2,000 cycles), through a second set of registers.
// MARCH_LOADS_EARLY of them go out before barrier 1: 24-28 of 37 in FP64 (all
// after it 1,020 us per two steps at 2048 x 4096, half 936, 28 of them 891, all
// before it 982), few in FP32, whose two waves per SIMD cover them.
// What bounds it: in FP64 HBM (2048 x 4096: 0.435 ms per step against 0.81 in
// single steps; 5.6 TB/s, reads and writes within 1-4% of one each per population
// and pass); in FP32 the vector units (0.26 ms against 0.43).
// ---------------------------------------------------------------------------
// LDS barrier that leaves global loads and stores in flight
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// first segment of the ring of hop group ex
constexpr int ring_base(int ex)
{
    int n = 0;
    for (int k = -3; k < ex; ++k) n += (k + 4) * ex_count(k);
    return n;
}
static_assert(ring_base(4) == 4 * NPOP, "rings hold four columns per population on average");

// Launch of the march over an lx x ly lattice: strips of ny rows, cut along x
// into segments, one block each, all blocks on the GPU at once.
constexpr int MARCH_WALL_COST_PCT = 130;   // a column of a wall strip over one of the others
struct MarchLaunch {
    int ny, nstrip;           // rows of a strip, strips
    int seglen, wall_seglen;  // columns of a segment, away from the walls and at them
    int nin, nblk;            // blocks of the strips away from the walls, and all
    int cost;                 // columns the slowest block steps, wall columns weighted; 0: no launch fits
};
inline MarchLaunch march_launch(int lx, int ly, int rows_max, int align, int slots, bool walls)
{
    MarchLaunch best{};
    int last_ny = 0;
    for (int s = (ly + rows_max - 1) / rows_max; s <= slots && s < (ly + rows_max - 1) / rows_max + 8; ++s) {
        const int ny = ((ly + s - 1) / s + align - 1) / align * align;
        if (ny == last_ny || ny > rows_max) continue;
        last_ny = ny;
        const int nstrip = (ly + ny - 1) / ny;
        const int nw = walls ? (nstrip > 1 ? 2 : 1) : 0, ni = nstrip - nw;
        for (int nsi = 1; nsi <= lx && (ni > 0 ? ni * nsi + nw <= slots : nsi == 1); ++nsi) {
            MarchLaunch m{};
            m.ny = ny;
            m.nstrip = nstrip;
            m.seglen = (lx + nsi - 1) / nsi;
            m.nin = ni * ((lx + m.seglen - 1) / m.seglen);
            m.wall_seglen = lx;
            m.nblk = m.nin;
            if (nw) {
                const int nsw = (slots - m.nin) / nw < lx ? (slots - m.nin) / nw : lx;
                // no more wall segments than keep up with the others
                const int fit = ni > 0 ? (m.seglen + 6) * 100 / MARCH_WALL_COST_PCT - 6 : 1;
                m.wall_seglen = (lx + nsw - 1) / nsw > fit ? (lx + nsw - 1) / nsw : fit;
                m.nblk += nw * ((lx + m.wall_seglen - 1) / m.wall_seglen);
            }
            const int ci = ni > 0 ? m.seglen + 6 : 0;
            const int cw = nw ? (m.wall_seglen + 6) * MARCH_WALL_COST_PCT / 100 : 0;
            m.cost = ci > cw ? ci : cw;
            if (best.cost == 0 || m.cost < best.cost) best = m;
        }
    }
    return best;
}

// Wall slots of one wall by source row: slot value of hop j of WH from mirror
// row k (k < en): 26 (j, k) pairs.
constexpr int NWK = 26;
struct WallPairs { int j[NWK], k[NWK], at[NWS][3]; };
constexpr WallPairs make_wall_pairs()
{
    WallPairs t{};
    int n = 0;
    for (int j = 0; j < NWS; ++j)
        for (int k = 0; k < WH.en[j]; ++k) { t.j[n] = j; t.k[n] = k; t.at[j][k] = n; ++n; }
    return t;
}
constexpr WallPairs WP = make_wall_pairs();
__constant__ WallPairs c_wall_pairs = make_wall_pairs();

template <typename S> struct MarchShape;   // most rows of a strip, waves per step, loads before barrier 1
template <> struct MarchShape<double> { static constexpr int rows = 112, waves = 2, early = 26; };
template <> struct MarchShape<float> { static constexpr int rows = 240, waves = 4, early = 4; };

template <typename S, bool WALLS, bool WIDE>
__global__ __launch_bounds__(2 * MarchShape<S>::waves * 64) void k_twostep_march(
    const S* __restrict__ src, S* __restrict__ dst, Geo g, CollideArgs args, const double* __restrict__ wall_rho,
    WallTable wt, double* __restrict__ wall_mid, double* __restrict__ wall_rho_out, MarchLaunch ml)
{
    using Cc = typename Store<S>::C;
    constexpr int NY = MarchShape<S>::rows, NW = MarchShape<S>::waves, LD1 = MarchShape<S>::early;
    const int ny = ml.ny;
    static_assert(NY + 6 <= NW * 64, "rows of the first step fit its waves");
    __shared__ S wsv[WALLS ? 2 * NWK : 1][16];   // the source's wall slots by (wall, pair) and column
    __shared__ double wew[2][NWS];
    // ring segments of NY rows with 6 rows of padding on either side, so that
    // the first step's lanes store without a test of their rows
    constexpr int RS = NY + 12;
    __shared__ S ring[4 * NPOP * RS + 12];
    const int L = xcd_block(blockIdx.x, ml.nblk);
    // blocks 0 .. nin-1: the strips away from the walls, segment by segment;
    // the others: the strips at the walls, strip by strip, in segments of their own
    const int ni = WALLS ? ml.nstrip - (ml.nstrip > 1 ? 2 : 1) : ml.nstrip;
    const int nws = (g.lx + ml.wall_seglen - 1) / ml.wall_seglen;
    const int m = L - ml.nin;
    const int strip = m < 0 ? (WALLS ? 1 : 0) + L % ni : (m < nws ? 0 : ml.nstrip - 1);
    const int len = m < 0 ? ml.seglen : ml.wall_seglen;
    const int xa = (m < 0 ? L / ni : m % nws) * len, xb = min(xa + len, g.lx);
    const int y0 = strip * ny;
    const int y1 = min(y0 + ny, g.ly);
    const int ncol = xb - xa + 6;
    const int t = (int)threadIdx.x;
    const bool wall_strip = WALLS && (y0 < 6 || y1 > g.ly - 6);
    const int stride8 = (int)(g.ps * (long long)sizeof(S));
    int w[8];   // first row of the ring slot written now, by group (R = ex + 4 slots)
#pragma unroll
    for (int R = 1; R < 8; ++R) w[R] = ring_base(R - 4) * RS;
    auto advance = [&]() {
#pragma unroll
        for (int R = 2; R < 8; ++R) {
            w[R] += ex_count(R - 4) * RS;
            if (w[R] == ring_base(R - 3) * RS) w[R] = ring_base(R - 4) * RS;
        }
    };
    // lanes 0..51 make the wall slots of one source column: pair t of both walls
    const int wp = t < 2 * NWK ? t % NWK : 0, ww = t < NWK ? 0 : 1;
    double wfac = 0.0, wsub = 0.0;
    const double* wrow = wall_rho;
    if (wall_strip) {
        if (t < NWS) {
#pragma unroll
            for (int j = 0; j < NWS; ++j)
                if (t == j) { wew[0][j] = wt.ew[0][WH.bot[j]]; wew[1][j] = wt.ew[1][WH.top[j]]; }
        }
        lds_barrier();
        if (t < 2 * NWK) {
            const int j = c_wall_pairs.j[wp];
            wfac = wew[ww][j];
            if (Store<S>::shifted) {
#pragma unroll
                for (int k = 0; k < NWS; ++k)
                    if (k == j) wsub = W_SHELL[SHELL[WH.bot[k]]];
            }
            wrow = wall_rho + (ww * 3 + c_wall_pairs.k[wp]) * g.lx;
            for (int k = 0; k < 7; ++k) {   // columns xa-6 .. xa
                const int X = xa - 6 + k;
                wsv[t][X & 15] = (S)(wfac * wrow[wrap_x(X, g.lx)] - wsub);
            }
        }
        lds_barrier();
    }
    if (__builtin_amdgcn_readfirstlane(t) < NW * 64) {
        // ---- first step
        const int r = min(t, NY + 5) - 3;
        int y = y0 + r;
        const bool on = t < NY + 6 && (!WALLS || (y >= 0 && y < g.ly));
        if (WALLS) y = min(max(y, 0), g.ly - 1);
        else {
            y = min(y, y1 + 2);
            y = y < 0 ? y + g.ly : (y >= g.ly ? y - g.ly : y);
        }
        const int wall = y < 3 ? 0 : 1, wr = wall ? g.ly - 1 - y : y;   // rows from the wall
        const bool near = WALLS && on && wr < 3;
        int vo = y * (int)sizeof(S);
        int vp[7];   // byte offsets of rows y - 3 .. y + 3 of a lattice without walls
#pragma unroll
        for (int k = 0; k < 7; ++k) vp[k] = (3 + wrap_x(y + k - 3, g.ly)) * (int)sizeof(S);
        // ring row of this lane; lanes without a site store to the padding
        const int rw = 6 + (on ? r : NY + 5);
        const S* cp[7];   // source columns X - 3 .. X + 3 of the first-step column X, three rows down
        int cnew = 0;
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            cnew = wrap_x(xa - 6 + k, g.lx);
            cp[k] = src + g.origin - 3 + (long long)cnew * g.cs;
        }
        double wnew = 0.0;
        int soff = 0;
        __amdgpu_buffer_rsrc_t rs[7];
        // loads of populations lo .. hi-1
        auto load_column = [&](Cc(&f)[NPOP], int lo, int hi) {
            if (lo == 0) soff = 0;
            asm volatile("" : "+s"(soff), "+v"(vo));   // keeps the offsets in the loads' immediates, and one SGPR
            if (lo == 0)
#pragma unroll
                for (int k = 0; k < 7; ++k) rs[k] = buf_of(cp[k]);
#pragma unroll
            for (int l = 0; l < NPOP; ++l) {
                if (l < lo || l >= hi) continue;
                f[l] = (Cc)buf_load<S>(rs[3 - EX[l]], WALLS ? vo + (3 - EY[l]) * (int)sizeof(S) : vp[3 - EY[l]], soff);
                soff += stride8;
            }
        };
        auto next_column = [&](int i) {   // the last column is loaded again
            if (i + 1 < ncol) {
#pragma unroll
                for (int k = 0; k < 6; ++k) cp[k] = cp[k + 1];
                cnew = cnew + 1 == g.lx ? 0 : cnew + 1;
                cp[6] = src + g.origin - 3 + (long long)cnew * g.cs;
            }
        };
        auto body = [&](Cc(&f)[NPOP], Cc(&nxt)[NPOP], int i) {
            const int X = xa - 3 + i;
            next_column(i);
            if (wall_strip) {
                if (t < 2 * NWK) wnew = wrow[wrap_x(X + 4, g.lx)];
                if (near) {
                    S v[NWS];
#pragma unroll
                    for (int j = 0; j < NWS; ++j)
                        v[j] = wsv[wall * NWK + WP.at[j][0] + max(WH.en[j] - 1 - wr, 0)][(X - WH.ex[j]) & 15];
#pragma unroll
                    for (int j = 0; j < NWS; ++j) {
                        const Cc b = f[WH.bot[j]], u = f[WH.top[j]];
                        f[WH.bot[j]] = wall == 0 && wr < WH.en[j] ? (Cc)v[j] : b;
                        f[WH.top[j]] = wall == 1 && wr < WH.en[j] ? (Cc)v[j] : u;
                    }
                }
            }
            S* p[8];
#pragma unroll
            for (int R = 1; R < 8; ++R) p[R] = ring + w[R] + rw;
            if constexpr (LD1 > 0) load_column(nxt, 0, LD1);
            collide_site<Cc, Store<S>::shifted, WIDE>(
                f, args,
                [&]() {
                    if constexpr (LD1 > 0) {
#pragma unroll
                        for (int l = 0; l < LD1; ++l) {
                            __builtin_amdgcn_sched_group_barrier(0x2, (sizeof(S) == 8 ? 130 : 170) / LD1, 0);
                            __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    lds_barrier();       // the second step has read what is overwritten now
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (LD1 < NPOP) load_column(nxt, LD1, NPOP);
                },
                [&](int l) { p[EX[l] + 4][ex_rank(l) * RS + EY[l]] = (S)f[l]; });
            if constexpr (sizeof(S) == 8) {
#pragma unroll
                for (int l = 0; l < NPOP; ++l) {
                    __builtin_amdgcn_sched_group_barrier(0x2, 9, 0);
                    if (l >= LD1) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                }
            } else {
#pragma unroll
                for (int l = 0; l < NPOP; ++l) {
                    __builtin_amdgcn_sched_group_barrier(0x2, 14, 0);
                    if (l >= LD1) __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                }
#pragma unroll
                for (int l = 0; l < NPOP; ++l) {
                    __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (wall_strip) {
                if (near) {
                    double e[NWS];
#pragma unroll
                    for (int j = 0; j < NWS; ++j) e[j] = wew[wall][j];
                    const double d = stored_density<S>(f);
                    // the wall slots of the second step that mirror this row
#pragma unroll
                    for (int j = 0; j < NWS; ++j) {
                        const int up = WH.en[j] - 1 - 2 * wr;   // rows from here into the lattice
                        const int to = wall == 0 ? ex_rank(WH.bot[j]) * RS + up : ex_rank(WH.top[j]) * RS - up;
                        const double sub = Store<S>::shifted ? W_SHELL[SHELL[WH.bot[j]]] : 0.0;
                        if (wr < WH.en[j] && (unsigned)(r + (wall == 0 ? up : -up)) < (unsigned)ny)
                            p[WH.ex[j] + 4][to] = (S)(e[j] * d - sub);
                    }
                    if (X >= xa && X < xb && r >= 0 && r < ny) wall_mid[(wall * 3 + wr) * g.lx + X] = d;
                }
                if (t < 2 * NWK) wsv[t][(X + 4) & 15] = (S)(wfac * wnew - wsub);
            }
            lds_barrier();
            advance();
        };
        Cc fa[NPOP], fb[NPOP];
        load_column(fa, 0, NPOP);
        for (int i = 0;;) {
            body(fa, fb, i);
            if (++i == ncol) break;
            body(fb, fa, i);
            if (++i == ncol) break;
        }
        if (WALLS) set_mid_word(wall_mid + 6 * g.lx, 1.0);
    } else {
        // ---- second step
        const int r = min(t - NW * 64, NY - 1);
        const int y = y0 + r;
        const bool in = t - NW * 64 < ny && y < y1;
        const bool near = WALLS && in && (y < 3 || y >= g.ly - 3);
        const int ob = in ? y * (int)sizeof(S) : (int)0x80000000;   // beyond the stores' bounds
        for (int i = 0; i < 6; ++i) {
            lds_barrier();
            lds_barrier();
            advance();
        }
        lds_barrier();
        lds_barrier();
        advance();   // w[R] is now the slot that the next column will take: the one read for this output
        for (int i = 6; i < ncol; ++i) {   // output column xa - 6 + i, after column i of the first step is in
            const int X = xa - 6 + i;
            Cc q[NPOP];
            const S* p[8];
#pragma unroll
            for (int R = 1; R < 8; ++R) p[R] = ring + w[R] + r + 6;
#pragma unroll
            for (int l = 0; l < NPOP; ++l) q[l] = (Cc)p[EX[l] + 4][ex_rank(l) * RS];
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(dst + g.origin + (long long)X * g.cs), 0, 0x7fffffff, RAW_BUFFER_WORD3);
            collide_site<Cc, Store<S>::shifted, WIDE>(
                q, args,
                [&]() {
                    __builtin_amdgcn_sched_barrier(0);
                    if (i + 1 < ncol) lds_barrier();   // the ring may be overwritten
                    __builtin_amdgcn_sched_barrier(0);
                },
                [&](int l) { buf_store<S, STORE_CPOL_NT_SC1>((S)q[l], rs, ob, l * stride8); });
#pragma unroll
            for (int l = 0; l < NPOP; ++l) {
                __builtin_amdgcn_sched_group_barrier(0x2, sizeof(S) == 8 ? 9 : 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x40, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (wall_strip && near) wall_rho_out[(y < 3 ? y : 3 + (g.ly - 1 - y)) * g.lx + X] = stored_density<S>(q);
            if (i + 1 < ncol) {
                lds_barrier();
                advance();
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Which form a lattice takes.
// ---------------------------------------------------------------------------
enum TwoStepKind { TWO_STEP_NONE = 0, TWO_STEP_TILE_8X8, TWO_STEP_TILE_8X16, TWO_STEP_TILE_16X16, TWO_STEP_MARCH };
struct TwoStep { TwoStepKind kind; MarchLaunch march; };

// Tiles where both buffers stay in the 256 MB Infinity Cache, which covers what
// they read twice; beyond it the march, where its blocks' lanes and columns are
// mostly used: sites over (columns the slowest block steps x rows x CUs) of at
// least 0.55.  us per step, tiles / march with walls, and without (padded buffers
// in MB): FP64 640x640 (239) 26 / 32 and 27 / 30, 680x680 (266) 36 / 38 and 37 / 34,
// 720x720 (296) 41 / 40 and 41 / 38, 1024x1024 (592) 78 / 67 and 77 / 65; FP32 900x900
// (237) 33 / 38 and 34 / 34, 930x930 (254) 41 / 42 and 40 / 37, 1024x1024 (306) 56 / 49
// and 51 / 43; with FP32 sums 900x900 31 / 37 and 29 / 33, 1024x1024 52 / 47 and 49 / 42.
// Beyond the cache and below that share tiles still gain on single steps in FP64
// (20000x33: 80 us per step against 300, the march 129; 1024x1024 78 against 111);
// in FP32, whose collisions are the larger part of a step, up to 16 x 256 sites per
// CU (1024x1024 56 against 56, with FP32 sums 52 against 56; 2048x4096 433 against
// 432).
// The smallest tiles are taken while they leave no CU with more than one (us per
// step with walls, 8x8 / 8x16 / 16x16: FP64 128x128 4.4 / 4.9 / 5.7, 256x128 5.8 / 5.2 /
// 5.9, 256x256 8.0 / 7.3 / 6.6; FP32 4.6 / 5.0 / 5.1, 5.5 / 5.1 / 5.3, 7.7 / 6.6 / 5.6).
// FP32 with FP64 sums, whose collisions bound it, takes 16 x 16 tiles only where
// their rings' columns, 6 to a tile, are less than half of the lattice's (0.6 of
// them up to four tiles per CU, any share up to the two that run at once).  us
// per four steps, single / in pairs: 7x100000 158 / 193, 17x20000 73 / 99, 17x6000
// 30 / 40, 33x10000 70 / 80, 24x40000 208 / 227; 33x5000 48 / 47, 12x12000 46 / 37,
// 7x6000 24 / 23; 37x30000 234 / 169.
inline bool few_columns(int lx, long long tiles, int ncu)
{
    const int ring = (lx + 15) / 16 * 6;
    return ring * 2 >= lx && tiles > (ring * 10 >= lx * 6 ? 2 : 4) * ncu;
}
constexpr int MARCH_MIN_USE_PCT = 55;
constexpr int TILE_FP32_MAX_SITES_PER_CU = 16 * 256;
constexpr long long TILE_CACHE_BYTES = 256LL << 20;
template <typename S>
inline TwoStep choose_two_step(const Geo& g, int ncu, int max_lds, bool walls, bool f32_sums)
{
    TwoStep t{TWO_STEP_NONE, MarchLaunch{}};
    if (ncu <= 0) return t;
    const long long sites = (long long)g.lx * g.ly;
    // LDS of either form: at most 154 KB; offsets of a site's populations in 32 bits
    constexpr int LDS = 157 * 1024;
    if (max_lds < LDS) return t;
    const bool cached = 2 * g.total * (long long)sizeof(S) <= TILE_CACHE_BYTES;
    t.march = march_launch(g.lx, g.ly, MarchShape<S>::rows, 16, ncu, walls);
    if (!cached && t.march.cost > 0 && (long long)NPOP * g.ps * (long long)sizeof(S) < (1LL << 31) &&
        sites * 100 >= (long long)MARCH_MIN_USE_PCT * t.march.cost * MarchShape<S>::rows * ncu) {
        t.kind = TWO_STEP_MARCH;
        return t;
    }
    if (g.total * (long long)sizeof(S) >= (1LL << 31)) return t;
    if (sizeof(S) == 4 && !cached && sites > (long long)TILE_FP32_MAX_SITES_PER_CU * ncu) return t;
    auto tiles = [&](int tx, int ty) { return (long long)((g.lx + tx - 1) / tx) * ((g.ly + ty - 1) / ty); };
    if (tiles(8, 8) <= ncu) t.kind = TWO_STEP_TILE_8X8;
    else if (tiles(8, 16) <= ncu) t.kind = TWO_STEP_TILE_8X16;
    else if (sizeof(S) == 8 || f32_sums || !few_columns(g.lx, tiles(16, 16), ncu)) t.kind = TWO_STEP_TILE_16X16;
    return t;
}

}  // namespace lbm
