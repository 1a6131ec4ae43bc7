// fh_direct.hip -- the quadrature sum of a small grid call as it stands.
//
// The Fresnel kernel of eq. faq is a product over the axes,
//   exp(i pi |xi - x|^2/(lambda z)) = Ex(xi_1, x_1) Ey(xi_2, x_2),
// so a grid's field is a product of two matrices,
//   u[k2][k1] = 1/(i lambda z) sum_j (c_j Ey[k2][j]) Ex[k1][j],
// 8 N n1 n2 flops on the matrix cores.  A call of few nodes on a small grid
// spends its time on the latencies of the ten dependent kernels that bin,
// spread, reduce and transform; this takes two, and no kernel truncation.
#include "fh_kernels.hpp"

namespace fh {
namespace {

constexpr int kDirTile = 64;   // outputs per workgroup and axis
constexpr int kDirNodes = 16;  // nodes staged at a time

struct DirectParams {
    const double* x;
    const double* y;
    const double* w;
    const double* src;  // source terms, or null
    int64_t N;
    double inv2lz, inv2lD;  // 1/(2 lambda z); 1/(2 lambda D), 0 for a plane wave
    double h1, h2, xc, yc;
    int n1, n2;
    int per;  // nodes per split (a multiple of 4)
};

// Workgroup (64 columns, 64 rows, split of the nodes): sixteen nodes at a
// time, wavefronts 0 and 2 stage c Ey and wavefronts 1 and 3 Ex, a lane per
// output coordinate (a node's coordinates are uniform across a wavefront),
// with the phase in turns and FP64 as everywhere; then each wavefront
// multiplies its 32 x 32 outputs, four real products per complex one.
// Sixteen-cell blocks past the grid's edge are skipped.
// Bound by the chain staging, barrier, products (64 of 64 cycles in FP64),
// barrier: a small call has two wavefronts per SIMD to overlap and two or
// three stages each.  4800 nodes on 100 x 100 outputs, one call among others:
// 49 us through the tiled path, 28 here (traced apart, 27 this kernel and 5 the
// sum of the splits).
template <class R>
__global__ void __launch_bounds__(256) k_direct(DirectParams p, typename V2<R>::T* __restrict__ part)
{
    using C = typename V2<R>::T;
    using M = MfmaAcc<R>;
    using V = typename M::V;
    __shared__ C st[kDirNodes][2 * kDirTile];
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, g = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = blockIdx.x * kDirTile, r0 = blockIdx.y * kDirTile;
    const int64_t j0 = (int64_t)blockIdx.z * p.per, j1 = min(p.N, j0 + p.per);
    // staging: this wavefront's axis and nodes, this lane's coordinate
    const bool xaxis = wv & 1;
    const double tc = xaxis ? p.xc + p.h1 * (c0 + lane - p.n1 / 2) : p.yc + p.h2 * (r0 + lane - p.n2 / 2);
    const double* __restrict__ crd = xaxis ? p.x : p.y;
    // products: this wavefront's rows and columns, in blocks of 16
    const int rw = r0 + 32 * (wv >> 1), cw = c0 + 32 * (wv & 1);
    const int nbr = min(2, (p.n2 - rw + 15) >> 4), nbc = min(2, (p.n1 - cw + 15) >> 4);
    V are[2][2], aim[2][2];
#pragma unroll
    for (int br = 0; br < 2; ++br)
#pragma unroll
        for (int bc = 0; bc < 2; ++bc) are[br][bc] = aim[br][bc] = V{R(0), R(0), R(0), R(0)};
    // lane i < 8 loads this wavefront's i-th node of a stage, a stage ahead;
    // the staging broadcasts it
    double nc = 0.0, nw = 0.0;
    auto load = [&](int64_t base) {
        const int64_t j = base + 2 * lane + (wv >> 1);
        if (lane < kDirNodes / 2 && j < j1) {
            nc = crd[j];
            nw = p.w[j];
        }
    };
    load(j0);
    for (int64_t base = j0; base < j1; base += kDirNodes) {
        const double pc = nc, pw = nw;
        load(base + kDirNodes);
#pragma unroll 2
        for (int i = 0; i < kDirNodes / 2; ++i) {
            const int q = 2 * i + (wv >> 1);
            const int64_t j = base + q;
            C v{R(0), R(0)};
            if (j < j1) {
                const double d = tc - lane_val(pc, i);
                const double t = d * d * p.inv2lz;
                double sn, cs;
                sincospi(2.0 * (t - rint(t)), &sn, &cs);
                if (!xaxis) {
                    double cr = lane_val(pw, i), ci = 0.0;
                    if (p.inv2lD > 0.0) {
                        const double xj = p.x[j], yj = p.y[j];
                        const double tt = (xj * xj + yj * yj) * p.inv2lD;
                        double s2, c2;
                        sincospi(2.0 * (tt - rint(tt)), &s2, &c2);
                        ci = cr * s2;
                        cr *= c2;
                    }
                    if (p.src) {
                        const double sr = p.src[2 * j], si = p.src[2 * j + 1];
                        const double tr = cr * sr - ci * si;
                        ci = cr * si + ci * sr;
                        cr = tr;
                    }
                    const double tr = cr * cs - ci * sn;
                    sn = cr * sn + ci * cs;
                    cs = tr;
                }
                v = C{(R)cs, (R)sn};
            }
            st[q][(xaxis ? kDirTile : 0) + lane] = v;
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kDirNodes / 4; ++s) {
            if (base + 4 * s >= j1) break;  // wavefront-uniform
            C a[2], b[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                a[k] = st[4 * s + g][32 * (wv >> 1) + 16 * k + i16];
                b[k] = st[4 * s + g][kDirTile + 32 * (wv & 1) + 16 * k + i16];
            }
#pragma unroll
            for (int br = 0; br < 2; ++br)
#pragma unroll
                for (int bc = 0; bc < 2; ++bc) {
                    if (br >= nbr || bc >= nbc) continue;  // wavefront-uniform
                    are[br][bc] = M::mma(a[br].x, b[bc].x, are[br][bc]);
                    aim[br][bc] = M::mma(a[br].x, b[bc].y, aim[br][bc]);
                    are[br][bc] = M::mma(-a[br].y, b[bc].y, are[br][bc]);
                    aim[br][bc] = M::mma(a[br].y, b[bc].x, aim[br][bc]);
                }
        }
        __syncthreads();
    }
    C* out = part + (size_t)blockIdx.z * p.n1 * p.n2;
#pragma unroll
    for (int br = 0; br < 2; ++br)
#pragma unroll
        for (int bc = 0; bc < 2; ++bc)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = rw + 16 * br + M::row(lane, v), c = cw + 16 * bc + i16;
                if (r < p.n2 && c < p.n1) out[(size_t)r * p.n1 + c] = C{are[br][bc][v], aim[br][bc][v]};
            }
}

// u = (sum of the splits' fields)/(i lambda z), 1 - u for an occulter: 16
// outputs per workgroup, 16 threads each, every 16th split, then in thread
// order, in double (the splits' sums of FP32 products cancel).
template <class R>
__global__ void __launch_bounds__(256) k_direct_sum(const typename V2<R>::T* __restrict__ part, int64_t n,
                                                    int splits, double invlz, int occ,
                                                    typename V2<R>::T* __restrict__ u)
{
    using C = typename V2<R>::T;
    __shared__ double2 s[16][17];
    const int64_t e = (int64_t)blockIdx.x * 16 + (threadIdx.x & 15);
    const int k = threadIdx.x >> 4;
    double2 a = make_double2(0.0, 0.0);
    if (e < n) {
#pragma unroll 8
        for (int i = k; i < splits; i += 16) {
            const C v = part[(size_t)i * n + e];
            a.x += v.x;
            a.y += v.y;
        }
    }
    s[k][threadIdx.x & 15] = a;
    __syncthreads();
    if (k > 0 || e >= n) return;
#pragma unroll
    for (int i = 1; i < 16; ++i) {
        a.x += s[i][threadIdx.x].x;
        a.y += s[i][threadIdx.x].y;
    }
    // times 1/(i lambda z)
    double re = a.y * invlz, im = -a.x * invlz;
    if (occ) {
        re = 1.0 - re;
        im = -im;
    }
    u[e] = C{(R)re, (R)im};
}

}  // namespace

// Up to where the sum itself takes less time than the tiled path, whose
// smallest call costs 45 us in FP64 and 42 in mixed precision, all latency, and
// grows slowly.  Two limits, since the sum's time has two parts.  The products:
// nodes times outputs, padded to blocks of 16; in us, FP64 14 at 1.0e7, 24 at
// 3.0e7, 33 at 6.2e7, 37 at 8.2e7, 48 at 1.25e8, 55 at 1.3e8; mixed 11 at
// 1.0e7, 18 at 3.0e7, 28 at 8.2e7, 40 at 1.6e8, 59 to 76 at 2.5e8.  And the
// staging, a sincos per node and coordinate of every 64 x 64 tile however few
// outputs it holds, another per node where there are source terms or a point
// source: nodes times outputs padded to 64, in us against the tiled path's,
// FP64 45 : 50 at 2.6e8 and 58 : 76 to 89 at 4.1e8 (56 : 50 and 77 : 76 with
// source terms), 190 : 134 at 1.6e9; mixed 39 : 45 at 2.0e8, 37 : 45 at
// 2.6e8, 50 : 47 at 4.1e8 (31 : 47 at 1.4e8, 50 : 46 at 1.8e8), 175 : 76 at
// 1.6e9.
constexpr double kDirectWork[2] = {1.0e8, 1.5e8};   // FP64, mixed
constexpr double kDirectStage[2] = {4.2e8, 2.8e8};
constexpr double kDirectLit = 1.65;  // staging with source terms

bool direct_serves(const fh_ctx* c, const fh_quad* q, int n1, int n2)
{
    // Options that set anything about the transform keep it.  So does a
    // tolerance looser than the precision's default: its kernel is narrower
    // and its results are that kernel's.
    const fh_options& o = c->opt;
    if (o.sigma != 0 || o.kernel_width != 0 || o.beta != 0 || o.tile != 0 || o.max_subproblem != 0 ||
        o.spread_method != 0 || o.deterministic != 0)
        return false;
    const bool d = c->prec == FH_FP64;
    if (c->tol > (d ? 1.0001e-9 : 1.0001e-5)) return false;
    auto outputs = [&](int m) { return (double)((n1 + m - 1) / m * m) * ((n2 + m - 1) / m * m); };
    const double stage = (q->src || q->D > 0.0 ? kDirectLit : 1.0) * (double)q->N * outputs(kDirTile);
    return q->N > 0 && (double)q->N * outputs(16) <= kDirectWork[d ? 0 : 1] && stage <= kDirectStage[d ? 0 : 1];
}

template <class R>
static fh_status direct_run(fh_ctx* c, const fh_quad* q, double lambda, double z, int n1, int n2, double h1, double h2,
                     double xc, double yc, int occ, R* u, size_t extra_bytes, void** extra)
{
    using C2 = typename V2<R>::T;
    const int64_t n = (int64_t)n1 * n2;
    const int tx = (n1 + kDirTile - 1) / kDirTile, ty = (n2 + kDirTile - 1) / kDirTile;
    // two workgroups per CU, a stage of nodes each at least
    const int64_t want = std::max<int64_t>(1, (2 * (int64_t)c->cu_count) / (tx * ty));
    const int64_t per = std::max<int64_t>(kDirNodes, ((q->N + want - 1) / want + 3) / 4 * 4);
    const int splits = (int)((q->N + per - 1) / per);
    FH_TRY(arena_reserve(c, aligned_bytes(sizeof(C2) * (size_t)n * splits) + aligned_bytes(extra_bytes)));
    C2* part = c->arena.take<C2>((size_t)n * splits);
    if (extra) *extra = c->arena.take<char>(extra_bytes);
    if (!u) u = static_cast<R*>(*extra);
    const double lz = lambda * z;
    const DirectParams p{q->x,
                         q->y,
                         q->w,
                         q->src,
                         q->N,
                         0.5 / lz,
                         q->D > 0.0 ? 0.5 / (lambda * q->D) : 0.0,
                         h1,
                         h2,
                         xc,
                         yc,
                         n1,
                         n2,
                         (int)per};
    timing_mark(c, 0);
    timing_mark(c, 1);
    hipLaunchKernelGGL((k_direct<R>), dim3(tx, ty, splits), dim3(256), 0, c->stream, p, part);
    timing_mark(c, 2);
    timing_mark(c, 3);
    hipLaunchKernelGGL((k_direct_sum<R>), dim3(nblocks(n, 16)), dim3(256), 0, c->stream, (const C2*)part, n, splits,
                       1.0 / lz, occ, reinterpret_cast<C2*>(u));
    FH_HIP(hipGetLastError());
    timing_mark(c, 4);
    timing_mark(c, 5);
    return FH_OK;
}

fh_status t1_direct(fh_ctx* c, const fh_quad* q, double lambda, double z, int n1, int n2, double h1, double h2,
                    double xc, double yc, int occ, void* u, size_t extra_bytes, void** extra)
{
    if (c->prec == FH_FP64)
        return direct_run<double>(c, q, lambda, z, n1, n2, h1, h2, xc, yc, occ, static_cast<double*>(u), extra_bytes,
                                  extra);
    return direct_run<float>(c, q, lambda, z, n1, n2, h1, h2, xc, yc, occ, static_cast<float*>(u), extra_bytes, extra);
}

}  // namespace fh
