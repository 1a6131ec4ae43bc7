// fh_window.hpp -- rules whose nodes reach a few fine-grid cells.
//
// A large occulter seen on a fine pupil grid (a 24 m starshade, h = 2.3 mm)
// puts a million nodes into a window of some 26 x 26 cells of the fine grid.
// Two things change then.  Binning the nodes into tiles, spreading every few
// of them into a tile of their own and merging those tiles moves far more
// than the window holds; and transforming whole rows and columns of the grid
// computes mostly with zeros.  Three kernels take the whole path instead:
//   k_win_spread  every wavefront spreads consecutive nodes, in the order the
//                 rule has them, into a window in LDS, and each workgroup
//                 writes one window;
//   k_win_sum     adds the workgroups' windows in a fixed order;
//   k_win_dft     the window's Fourier sums at the n1 x n2 outputs as two
//                 matrix products (columns, then rows), with the epilogue.
// Type 3 seen from a small pupil has as small a grid, and takes the first two.
#pragma once
#include "fh_kernels.hpp"

namespace fh {
namespace {

// The window: SX x SY cells from cell (sh1, sh2) of the instance's own shift
// on, both at least 16 (the matrix-core tile) and less than the period.
struct WinGeom {
    int nf1, nf2;
    int SX, SY;
    int nblk;  // workgroups of all instances
    int run;   // nodes per wavefront, a multiple of 64
};

constexpr int kWinWaves = 4;  // wavefronts per workgroup

// One window per workgroup in FP64, to which its wavefronts add by LDS
// atomics (sums equal to rounding from call to call, as everywhere by
// default), and one per wavefront in FP32, whose LDS atomics are slow.  Four
// private FP64 windows of 27 x 27 cells leave LDS for two wavefronts per SIMD
// only, and the staging's latency then shows: 998,400 nodes on 2048 x 2048
// outputs 99.6 us, with the shared window 93.4, and 549 against 522 us for
// the gradient over three wavelengths.
template <class R> constexpr int win_tiles() { return sizeof(R) == 8 ? 1 : kWinWaves; }

__host__ __device__ inline size_t win_lds(int SX, int SY, int W, size_t rsize)
{
    return (rsize == 8 ? 1 : kWinWaves) * ((size_t)SX * SY * 2 * rsize) +
           kWinWaves * mfma_wave_lds(1, 17 - W, W, 16, rsize);
}

// Minimum and maximum over each row of 16 lanes.
__device__ __forceinline__ int row_min16(int v)
{
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, false));  // row_ror:8
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, false));
    return min(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, false));
}
__device__ __forceinline__ int row_max16(int v) { return -row_min16(-v); }

// An instance in scalar registers: the compiler keeps one that it reads from a
// table at an index from memory in vector registers (57 spilled instead of 14
// in k_win_spread at W = 11, and batches 15% slower).
__device__ __forceinline__ InstParams uniform(const InstParams& p)
{
    union {
        InstParams ip;
        int w[sizeof(InstParams) / sizeof(int)];
    } v{p};
#pragma unroll
    for (int k = 0; k < (int)(sizeof(InstParams) / sizeof(int)); ++k) v.w[k] = __builtin_amdgcn_readfirstlane(v.w[k]);
    return v.ip;
}

// Spread without binning.  A wavefront walks a run of consecutive nodes, 64
// at a time: a lane computes its node's cell, offsets and strength (as
// k_bin_place does), then sixteen nodes at a time are staged and multiplied
// as in k_spread_mfma, whose 16 x 16 accumulators sit at the window cells
// (ox, oy) on.  A rule's nodes come along a ray or an arc, so sixteen in a
// row nearly always start within the 17 - W cells that one position of the
// accumulators serves, and hundreds do before it has to move: then the
// accumulators are added to the wavefront's window in LDS and start again at
// zero.  Sixteen nodes that lie further apart are taken one by one, moving
// as needed, so any order gives the same sums.
// Bound by the operand staging (VALU and LDS), as k_spread_mfma; held to the
// registers of four wavefronts per SIMD (14 spill in FP64; against three and
// none, 86 and 88 us for 998,400 nodes on 2048 x 2048 outputs).
// table, of_block: the instances and each workgroup's instance (null: p0's).
template <class R, int W>
__global__ void __launch_bounds__(64 * kWinWaves) __attribute__((amdgpu_waves_per_eu(4))) k_win_spread(
    InstParams p0, const InstParams* __restrict__ table, const int* __restrict__ of_block, WinGeom wg,
    typename V2<R>::T* __restrict__ part, const R* __restrict__ poly)
{
    using C = typename V2<R>::T;
    using M = MfmaAcc<R>;
    using V = typename M::V;
    constexpr int MS = 16, T = 17 - W;
    constexpr int NP = poly_np(W), NPAIR = poly_npair(W), NE = poly_ne(W), NO = poly_no(W);
    constexpr int P = mfma_period(1, W), RL = mfma_rows(1, T, W, MS);
    static_assert(T >= 1, "the kernel must fit the matrix-core tile");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, i16 = lane & 15, k4 = lane >> 4;
    const int SX = wg.SX, SY = wg.SY, cells = SX * SY;
    constexpr int NTILE = win_tiles<R>();
    C* tile = reinterpret_cast<C*>(smem_raw) + (NTILE > 1 ? wv : 0) * cells;
    unsigned char* pts = smem_raw + NTILE * cells * sizeof(C) + wv * mfma_wave_lds(1, T, W, MS, sizeof(R));
    R* ttab = reinterpret_cast<R*>(pts + 4 * MfmaPoint<R>::words * MS);
    R* rows = ttab + 2 * MS;
    const int pp = lane % NPAIR, pg = lane / NPAIR;
    R ce[NE], co[NO];
#pragma unroll
    for (int j = 0; j < NE; ++j) ce[j] = poly[NP * W + j * NPAIR + pp];
#pragma unroll
    for (int j = 0; j < NO; ++j) co[j] = poly[NP * W + (NE + j) * NPAIR + pp];
    for (int e = threadIdx.x; e < NTILE * cells; e += 64 * kWinWaves)
        reinterpret_cast<C*>(smem_raw)[e] = C{R(0), R(0)};
    for (int e = lane; e < RL; e += 64) rows[e] = R(0);
    __syncthreads();
    InstParams ip = p0;
    if (table) ip = uniform(table[of_block[blockIdx.x]]);
    const int64_t n0 = min(ip.N, (int64_t)wg.run * (((int)blockIdx.x - ip.tile_off) * kWinWaves + wv));
    const int64_t n1 = min(ip.N, n0 + wg.run);
    int ox = 0, oy = 0;  // the accumulators' first cell, wavefront-uniform
    V are = V{R(0), R(0), R(0), R(0)}, aim = are;
    const uint32_t lane_off = (uint32_t)(i16 * sizeof(R));
    auto move_to = [&](int nx, int ny) {
        wave_lds_order();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            C* t = tile + (oy + M::row(lane, v)) * SX + ox + i16;
            if constexpr (NTILE == 1) {
                atomicAdd(&t->x, are[v]);
                atomicAdd(&t->y, aim[v]);
            } else {
                *t = C{t->x + are[v], t->y + aim[v]};
            }
            are[v] = aim[v] = R(0);
        }
        wave_lds_order();
        ox = nx;
        oy = ny;
    };
    // accumulator position for first cells [mn, mx], mx - mn < T, of S - W + 1
    // possible ones: as much room on both sides as there is
    auto place = [&](int mn, int mx, int S) { return max(0, min(mn - (T - 1 - (mx - mn)) / 2, S - 16)); };
    double x = 0.0, y = 0.0, w = 0.0;
    if (n0 + lane < n1) {
        x = ip.x[n0 + lane];
        y = ip.y[n0 + lane];
        w = ip.w[n0 + lane];
    }
    for (int64_t base = n0; base < n1; base += 64) {
        const int64_t j = base + lane;
        const bool live = j < n1;
        int l1 = 0, l2 = 0;
        double d1 = 0.0, d2 = 0.0, cr = 0.0, ci = 0.0;
        if (live) {
            // the window starts below every stencil: no wrap
            const double g1 = (x - ip.cx) * ip.s1 - (double)ip.sh1, g2 = (y - ip.cy) * ip.s2 - (double)ip.sh2;
            const double f1 = ceil(g1 - 0.5 * W), f2 = ceil(g2 - 0.5 * W);
            if (f1 >= 0.0 && f1 <= (double)(SX - W) && f2 >= 0.0 && f2 <= (double)(SY - W)) {
                l1 = (int)f1;
                l2 = (int)f2;
                d1 = f1 - g1;
                d2 = f2 - g2;
            } else {
                w = 0.0;  // not in the window that its rule's box spans: adds nothing
            }
            const double t = ((x * x + y * y) * ip.pa + (x * ip.px + y * ip.py)) + ip.pc;
            const double f = t - rint(t);
            double sn, cs;
            sincospi(2.0 * f, &sn, &cs);
            cr = w * cs;
            ci = w * sn;
            if (ip.src) {
                const double sr = ip.src[2 * j], si = ip.src[2 * j + 1];
                const double tr = cr * sr - ci * si;
                ci = cr * si + ci * sr;
                cr = tr;
            }
        }
        // the next nodes' loads are in flight while these are spread
        if (j + 64 < n1) {
            x = ip.x[j + 64];
            y = ip.y[j + 64];
            w = ip.w[j + 64];
        }
        // the range of first cells of each sixteen nodes
        const int rnx = row_min16(live ? l1 : 0x7fff), rxx = row_max16(live ? l1 : -1);
        const int rny = row_min16(live ? l2 : 0x7fff), rxy = row_max16(live ? l2 : -1);
        const int np64 = (int)min<int64_t>(64, n1 - base);
        for (int s = 0; s < 4; ++s) {
            const int np = min(MS, np64 - MS * s);
            if (np <= 0) break;  // wavefront-uniform
            const bool mine = k4 == s;
            const int mnx = lane_val(rnx, MS * s), mxx = lane_val(rxx, MS * s);
            const int mny = lane_val(rny, MS * s), mxy = lane_val(rxy, MS * s);
            const bool together = mxx - mnx < T && mxy - mny < T;
            if (together && (mnx < ox || mxx >= ox + T || mny < oy || mxy >= oy + T))
                move_to(place(mnx, mxx, SX), place(mny, mxy, SY));
            if (mine) {
                // nodes past the run's end carry zero strength anywhere; nodes
                // taken one by one find their rows' first value here
                const int rx = live && together ? l1 - ox : 0, ry = live && together ? l2 - oy : 0;
                MfmaPoint<R>::put(pts, MS, i16, C{(R)cr, (R)ci}, (int)(sizeof(R) * (2 * i16 * P + T - 1 - rx)),
                                  (int)(sizeof(R) * ((2 * i16 + 1) * P + T - 1 - ry)));
                reinterpret_cast<C*>(ttab)[i16] = C{R(2) * (R)d1 + R(W - 1), R(2) * (R)d2 + R(W - 1)};
            }
            wave_lds_order();
            mfma_stage_values<R, W, MS>(rows, ttab, ce, co, pg, pp, P, T);
            wave_lds_order();
            if (together) {
                R ky[4], kr[4], ki[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const MfmaPoint<R> pt = MfmaPoint<R>::get(pts, MS, 4 * g + k4);
                    const R kx = *reinterpret_cast<const R*>(reinterpret_cast<const unsigned char*>(rows) + pt.o.x + lane_off);
                    ky[g] = *reinterpret_cast<const R*>(reinterpret_cast<const unsigned char*>(rows) + pt.o.y + lane_off);
                    kr[g] = pt.c.x * kx;
                    ki[g] = pt.c.y * kx;
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    are = M::mma(ky[g], kr[g], are);
                    aim = M::mma(ky[g], ki[g], aim);
                }
            } else {
                for (int q = 0; q < np; ++q) {
                    const int cx = lane_val(l1, MS * s + q), cy = lane_val(l2, MS * s + q);
                    if (cx < ox || cx >= ox + T || cy < oy || cy >= oy + T)
                        move_to(place(cx, cx, SX), place(cy, cy, SY));
                    // the node alone: the other three of the product are zero
                    const MfmaPoint<R> pt = MfmaPoint<R>::get(pts, MS, q);
                    const R kx = rows[2 * q * P + T - 1 - (cx - ox) + i16];
                    const R ky = k4 == 0 ? rows[(2 * q + 1) * P + T - 1 - (cy - oy) + i16] : R(0);
                    are = M::mma(ky, pt.c.x * kx, are);
                    aim = M::mma(ky, pt.c.y * kx, aim);
                }
            }
            // the next sixteen rewrite the staging
            wave_lds_order();
        }
    }
    move_to(0, 0);
    __syncthreads();
    C* out = part + (size_t)blockIdx.x * cells;
    for (int e = threadIdx.x; e < cells; e += 64 * kWinWaves) {
        C v{R(0), R(0)};
#pragma unroll
        for (int k = 0; k < NTILE; ++k) {
            const C t = reinterpret_cast<const C*>(smem_raw)[k * cells + e];
            v.x += t.x;
            v.y += t.y;
        }
        out[e] = v;
    }
}

// G[b] = the sum of instance b's windows (all of them without a table): 16
// cells per workgroup, 16 threads a cell, each over every 16th window, then in
// thread order, in double (an FP32 rule of 5e7 nodes has 24,000 windows).
// WRAP: the window is a whole periodic grid from its cell (-nf1/2, -nf2/2) on
// (type 3), and each sum goes to its place in the period.
template <class R, bool WRAP>
__global__ void __launch_bounds__(256) k_win_sum(const typename V2<R>::T* __restrict__ part,
                                                 const InstParams* __restrict__ table, WinGeom wg,
                                                 typename V2<R>::T* __restrict__ G)
{
    const int cells = wg.SX * wg.SY;
    int nblk = wg.nblk, blk0 = 0;
    if (table) {
        nblk = table[blockIdx.y].nblk;
        blk0 = table[blockIdx.y].tile_off;
    }
    using C = typename V2<R>::T;
    __shared__ double2 s[16][17];
    const int e = blockIdx.x * 16 + (threadIdx.x & 15), k = threadIdx.x >> 4, b = blockIdx.y;
    double2 a = make_double2(0.0, 0.0);
    if (e < cells) {
        const C* p = part + (size_t)blk0 * cells + e;
        // eight loads in flight, also where the count leaves a remainder (past
        // the last window it is read again and adds nothing)
        for (int i = k; i < nblk; i += 128) {
            C v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = p[(size_t)min(i + 16 * q, nblk - 1) * cells];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const bool in = i + 16 * q < nblk;
                a.x += in ? v[q].x : R(0);
                a.y += in ? v[q].y : R(0);
            }
        }
    }
    s[k][threadIdx.x & 15] = a;
    __syncthreads();
    if (k > 0 || e >= cells) return;
#pragma unroll
    for (int i = 1; i < 16; ++i) {
        a.x += s[i][threadIdx.x].x;
        a.y += s[i][threadIdx.x].y;
    }
    if constexpr (WRAP) {
        const int r = e / wg.SX, c = e - r * wg.SX;
        const int y = r - wg.nf2 / 2, x = c - wg.nf1 / 2;
        G[(size_t)(y < 0 ? y + wg.nf2 : y) * wg.nf1 + (x < 0 ? x + wg.nf1 : x)] = C{(R)a.x, (R)a.y};
    } else {
        G[(size_t)b * cells + e] = C{(R)a.x, (R)a.y};
    }
}

// LDS of k_win_dft: the window with its columns padded to a multiple of 4
// and its rows to 16 MT, two tiles of row roots, and the row factors.
inline size_t win_dft_lds(int SX, int MT, int KC, size_t rsize)
{
    return 2 * rsize * (size_t)(16 * MT) * ((SX + 3) / 4 * 4 + 32) + sizeof(double2) * (size_t)KC;
}

// u[k2][k1] = epilogue of sum_r e2(k2 (r + sh2)) sum_c e1(k1 (c + sh1)) G[r][c],
// e(m) = exp(-2 pi i m/nf), read from a table of the nf roots at m mod nf.
// Workgroup (column group, chunk of KC rows, instance); wavefront v takes 16
// columns.  It first sums over c: H = G e1, 16 MT rows x 16 columns, in
// accumulators; their layout is the operand layout of the second product (in
// FP32 with the rows of a group of 16 in another order, which the row roots
// follow), so H never leaves the registers.  Then, 16 output rows at a time,
// u = e2 H, with the row roots staged in LDS for the four wavefronts, the
// next tile's loaded while this one is multiplied.  A complex product takes
// four real ones.
// Bound by the matrix cores: 8 rows flops per output (the columns' sum adds
// SX/KC of that).  2048 x 2048 outputs from 27 x 27 cells in FP64: 35 us,
// where two passes of full transforms, a transposition and the epilogue took
// 101 and the reduce of whole rows before them 21.
template <class R, int MT>
__global__ void __launch_bounds__(256) k_win_dft(const typename V2<R>::T* __restrict__ G, WinGeom wg,
                                                 R* __restrict__ u, EpiParams ep, EpiInst e0,
                                                 const EpiInst* __restrict__ table,
                                                 const double2* __restrict__ roots1,
                                                 const double2* __restrict__ roots2, int KC)
{
    using C = typename V2<R>::T;
    using M = MfmaAcc<R>;
    using V = typename M::V;
    constexpr int RM = 16 * MT;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int SX = wg.SX, SY = wg.SY, SXp = (SX + 3) / 4 * 4;
    C* Gs = reinterpret_cast<C*>(lds_raw);              // [SXp][RM]
    C* Ey = Gs + SXp * RM;                              // 2 x [RM][16]
    double2* E2 = reinterpret_cast<double2*>(Ey + 2 * 16 * RM);
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, i16 = lane & 15, g = lane >> 4;
    const int b = blockIdx.z, k20 = blockIdx.y * KC;
    const EpiInst ei = table ? table[b] : e0;
    const int nf1 = wg.nf1, nf2 = wg.nf2;
    const int sh1 = ((ei.sh1 % nf1) + nf1) % nf1, sh2 = ((ei.sh2 % nf2) + nf2) % nf2;
    const int kc = min(KC, ep.n2 - k20), ntile = (kc + 15) / 16;
    // this thread's row roots: rows r = tid / 16 + 16 i, output row tid % 16
    // of each tile; the index moves by 16 (r + sh2) from tile to tile
    unsigned ri[MT], rs[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const unsigned r = (unsigned)((tid >> 4) + 16 * i + sh2) % (unsigned)nf2;
        const int k2 = k20 + i16 - ep.n2 / 2;
        const unsigned km = (unsigned)((k2 % nf2 + nf2) % nf2);
        ri[i] = (km * r) % (unsigned)nf2;
        rs[i] = (16u * r) % (unsigned)nf2;
    }
    auto fetch = [&](C* v) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const double2 e = roots2[ri[i]];
            v[i] = C{(R)e.x, (R)e.y};
            ri[i] += rs[i];
            if (ri[i] >= (unsigned)nf2) ri[i] -= (unsigned)nf2;
        }
    };
    auto put = [&](int buf, const C* v) {
#pragma unroll
        for (int i = 0; i < MT; ++i) Ey[buf * 16 * RM + ((tid >> 4) + 16 * i) * 16 + i16] = v[i];
    };
    C nx[MT];
    fetch(nx);
    for (int e = tid; e < SXp * RM; e += 256) {
        const int c = e / RM, r = e - c * RM;
        Gs[e] = c < SX && r < SY ? G[((size_t)b * SY + r) * SX + c] : C{R(0), R(0)};
    }
    // row factors exp(i pi eta^2/(lambda z))/Phi2 (the window's shift is in
    // the roots), and this lane's column factor
    for (int k = tid; k < kc; k += 256) {
        const double y = ep.yc + ep.h2 * (k20 + k - ep.n2 / 2);
        double tt = y * y * ei.inv2lz;
        tt -= rint(tt);
        double sn, cs;
        sincospi(2.0 * tt, &sn, &cs);
        const double sc = ep.iphi2[k20 + k];
        E2[k] = make_double2(cs * sc, sn * sc);
    }
    put(0, nx);
    const int ki = blockIdx.x * 64 + wv * 16 + i16, kcl = min(ki, ep.n1 - 1);
    const int k1 = kcl - ep.n1 / 2;
    double2 a;
    {
        const double xx = ep.xc + ep.h1 * k1;
        double tt = xx * xx * ei.inv2lz;
        tt -= rint(tt);
        double sn, cs;
        sincospi(2.0 * tt, &sn, &cs);
        const double sc = ep.iphi1[kcl];
        a = make_double2(cs * sc, sn * sc);
    }
    __syncthreads();
    V Hr[MT], Hi[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) Hr[m] = Hi[m] = V{R(0), R(0), R(0), R(0)};
    {
        const unsigned km = (unsigned)((k1 % nf1 + nf1) % nf1);
        unsigned ci = (km * ((unsigned)(g + sh1) % (unsigned)nf1)) % (unsigned)nf1;
        const unsigned cs = (4u * km) % (unsigned)nf1;
        for (int s = 0; s < SXp; s += 4) {
            const double2 e = roots1[ci];
            ci += cs;
            if (ci >= (unsigned)nf1) ci -= (unsigned)nf1;
            const R er = (R)e.x, em = (R)e.y;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const C v = Gs[(s + g) * RM + 16 * m + i16];
                Hr[m] = M::mma(v.x, er, Hr[m]);
                Hi[m] = M::mma(v.x, em, Hi[m]);
                Hr[m] = M::mma(-v.y, em, Hr[m]);
                Hi[m] = M::mma(v.y, er, Hi[m]);
            }
        }
    }
    C* uv = reinterpret_cast<C*>(u) + (size_t)b * ep.n2 * ep.n1;
    for (int t = 0; t < ntile; ++t) {
        if (t + 1 < ntile) fetch(nx);
        const C* ey = Ey + (t & 1) * 16 * RM + i16;
        V ur = V{R(0), R(0), R(0), R(0)}, ui = ur, vr = ur, vi = ur;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const C e = ey[(16 * m + M::row(lane, v)) * 16];
                ur = M::mma(e.x, Hr[m][v], ur);
                ui = M::mma(e.x, Hi[m][v], ui);
                vr = M::mma(e.y, Hi[m][v], vr);
                vi = M::mma(e.y, Hr[m][v], vi);
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = 16 * t + M::row(lane, v);
            if (k >= kc || ki >= ep.n1) continue;
            const double2 er = E2[k];
            const double ar = a.x * er.x - a.y * er.y, ai = a.x * er.y + a.y * er.x;
            const double fx = (double)(ur[v] - vr[v]), fy = (double)(ui[v] + vi[v]);
            // times 1/(i lambda z)
            double re = (fx * ai + fy * ar) * ei.invlz;
            double im = -(fx * ar - fy * ai) * ei.invlz;
            if (ei.occ) {
                re = 1.0 - re;
                im = -im;
            }
            uv[(size_t)(k20 + k) * ep.n1 + ki] = C{(R)re, (R)im};
        }
        if (t + 1 < ntile) put((t + 1) & 1, nx);
        __syncthreads();
    }
}

}  // namespace
}  // namespace fh
