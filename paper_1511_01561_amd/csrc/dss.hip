// Direct stiffness summation, mass-matrix inverse, no-flux projection and the
// SSP-RK3 stage update (the pointwise part of each stage in Code example 1:
// "DSS and multiply with inverse mass matrix", "update q").
//
// The summation is a gather: each unique node sums its element-local copies in
// ascending order.  No atomics, no colouring and no barriers are needed, and the
// result does not depend on scheduling (the paper avoids atomics by re-ordering
// elements and adding barriers; a gather removes the race altogether).
#include "kernels.h"

namespace numa {
namespace {

using namespace dev;

// Where the copies of a unique node are: the box's follow from its lattice
// position (I = gi + ni (gj + nj gk): two elements per direction on an element
// face, wrapped where periodic), the shell's are its horizontal copies in the
// bottom layer (hoff/hidx) in each radial layer that holds its level.  Nothing
// but the copies themselves is read (the shell: its short horizontal list), where
// the inverse map costs 4 bytes per copy and puts a load in front of every copy.
struct DssGeo {
    FastDiv fi, fj;            // box: division by ni and nj; shell: fi by n_horiz
    int nx, ny, nz, walls;     // elements; shell: nz layers
    const int32_t *hoff, *hidx;
    int layer;                 // shell: element-local nodes of one layer
};

// the copies of node I (e (N+1)^3 + l): eight slots, the used ones ascending, the
// others -1
template <int N, bool SHELL>
__device__ __forceinline__ void node_copies(const DssGeo &g, uint32_t I, int *cc)
{
    constexpr int P = N + 1, PP = P * P, NP = PP * P;
    // the two elements (and local indices) of lattice index c of n elements, in
    // ascending element order, the second -1 where there is none
    auto pair = [](int c, int n, bool wrap, int *e, int *l) {
        e[0] = c / N;
        l[0] = c - e[0] * N;
        e[1] = -1;
        l[1] = 0;
        if (e[0] == n) {  // the top level
            e[0] = n - 1;
            l[0] = N;
        } else if (l[0] == 0 && e[0] > 0) {
            e[1] = e[0];
            e[0] -= 1;
            l[0] = N;
        } else if (l[0] == 0 && wrap) {
            e[1] = n - 1;
            l[1] = N;
        }
    };
    int ez[2], lz[2];
    const uint32_t t = fdiv(I, g.fi);
    const int gi = (int)(I - t * g.fi.d);
    if constexpr (SHELL) {
        pair((int)t, g.nz, false, ez, lz);
        const int hb = g.hoff[gi], hn = g.hoff[gi + 1] - hb;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int c = h < hn ? g.hidx[hb + h] : -1;
#pragma unroll
            for (int z = 0; z < 2; ++z) cc[4 * z + h] = h < hn && ez[z] >= 0 ? ez[z] * g.layer + PP * lz[z] + c : -1;
        }
    } else {
        const uint32_t gk = fdiv(t, g.fj);
        int ex[2], lx[2], ey[2], ly[2];
        pair((int)gk, g.nz, !g.walls, ez, lz);
        pair((int)(t - gk * g.fj.d), g.ny, true, ey, ly);
        pair(gi, g.nx, true, ex, lx);
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    cc[4 * z + 2 * y + x] = ez[z] >= 0 && ey[y] >= 0 && ex[x] >= 0
                                                ? (ex[x] + g.nx * (ey[y] + g.ny * ez[z])) * NP + lx[x] +
                                                      P * (ly[y] + P * lz[z])
                                                : -1;
    }
}

// A lane per node and NV variables; the blocks (fb per group of variables, the
// first variable `first`) run through the nodes of one group after the other.
// Bound by memory latency: what counts is waves with loads in flight.  NV = 1 takes
// 46 registers (five variables and all their copies in a lane took 174, two waves
// per SIMD: one variable at N = 7, 1.2 M element-local nodes, 18.6 us).  Shells from
// 300,000 element-local nodes on share a lane's list and addresses among up to five
// variables, four copies of each in flight (62 registers).  us, by the inverse map with
// its copies one after another / NV = 1 / up to 5, for 1 and 5 variables: box
// 64x64x16 N = 4 56 / 32 / 32, 327 / 209 / 253; box 17x13x7 N = 5 4.8 / 4.0 / 4.0,
// 12.0 / 8.5 / 7.2; shell 6x14x14x5 N = 5 9.4 / 7.7 / 7.7, 34.6 / 31.8 / 25.7; shell
// 6x4x4x4 N = 4 4.5 / 3.5 / 3.5, 10.1 / 4.3 / 5.0.
template <int N, bool SHELL, int NV>
__global__ __launch_bounds__(256) void k_dss(PointArgs p, DssGeo g, FastDiv fb, int first, int nvar, const double *cin,
                                             double *out, int flags)
{
    const uint32_t group = fdiv(blockIdx.x, fb), b = (uint32_t)xcd_remap(blockIdx.x - group * fb.d, fb.d);
    const int64_t I = (int64_t)b * 256 + threadIdx.x;
    if (I >= p.nu) return;
    const int v0 = first + (int)group * NV, nv = nvar - v0 < NV ? nvar - v0 : NV;
    const bool wall = (flags & NUMA_DSS_NOFLUX) && p.walls && (I < p.nh || I >= p.nu - p.nh);
    // the projection needs three components: one lane of NV = 1 forms them all
    if (NV == 1 && wall && (v0 == 2 || v0 == 3)) return;
    int cc[8];
    node_copies<N, SHELL>(g, (uint32_t)I, cc);
    const double mi = flags & NUMA_DSS_MASS ? p.Minv[I] : 1.0;
    double r[NV];
    // absent copies are not loaded; the present ones are added in ascending order
    auto sum = [&](const double *src, double *r) {
        constexpr int Z = NV == 1 ? 8 : 4;  // copies in flight
#pragma unroll
        for (int v = 0; v < NV; ++v) r[v] = 0.0;
#pragma unroll
        for (int k0 = 0; k0 < 8; k0 += Z) {
            if (k0 > 0 && cc[k0] < 0) break;  // a second layer has a first copy
            double c[Z][NV];
#pragma unroll
            for (int k = 0; k < Z; ++k)
#pragma unroll
                for (int v = 0; v < NV; ++v) c[k][v] = cc[k0 + k] >= 0 && v < nv ? src[v * p.nl + cc[k0 + k]] : 0.0;
#pragma unroll
            for (int k = 0; k < Z; ++k)
                if (cc[k0 + k] >= 0)
#pragma unroll
                    for (int v = 0; v < NV; ++v) r[v] += c[k][v];
        }
        if (flags & NUMA_DSS_MASS)
#pragma unroll
            for (int v = 0; v < NV; ++v) r[v] *= mi;
    };
    const double *src = cin + v0 * p.nl;
    double *dst = out + v0 * p.nu + I;
    sum(src, r);
    if constexpr (NV == 1) {
        if (wall && v0 == 1) {
            double r2, r3;
            sum(src + p.nl, &r2);
            sum(src + 2 * p.nl, &r3);
            noflux(p, I, r[0], r2, r3);
            dst[p.nu] = r2;
            dst[2 * p.nu] = r3;
        }
    } else if constexpr (NV == 5) {
        if (wall) noflux(p, I, r[1], r[2], r[3]);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if (v < nv) dst[v * p.nu] = r[v];
}

__global__ void k_rk_stage(int64_t n, StageCoef c, const double *qn, const double *qs, const double *r,
                           double *qout)
{
    int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n) return;
    qout[a] = rk_update(c, c.a == 0.0 ? 0.0 : qn[a], qs[a], r[a]);
}

// Finish of a fused stage on the shell: one lane per unique node in unique
// order I = h + n_h gk, so state reads and writes run along the horizontal
// numbering.  The copies of a node factor: its horizontal copies in the
// bottom layer (hoff/hidx, 1 to 4, ascending) times its radial copies (local
// k = 0 of layer gk/N and k = N of the layer below on a layer boundary, else
// one).  The contributions are node-major [n_local][5]; the up to four
// horizontal copies of one radial copy are loaded together (absent ones are
// not loaded).  PLAIN: the
// output is the summed, mass-weighted, projected value (the filter's DSS).
struct ShellFin {
    const int32_t *hoff, *hidx;
    FastDiv fnh;      // division by n_horiz
    int nz;           // element layers
    int64_t layer;    // elements of one layer times (N+1)^3
};

// fold: the contributions away from the bottom and top layers are
// J w (q_s + cdt R) (k_rhs), so M^-1 times their sum is y = q_s + cdt R and
// q_s is not read there (as in box_finish_node)
template <int N, typename T, bool PLAIN = false>
__global__ void k_shell_finish(PointArgs p, ShellFin sf, const T *ev, StageCoef c, int fold, const double *qn,
                               const double *qs, double *qout)
{
    constexpr int P = N + 1, PP = P * P;
    const int64_t t = xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (t >= p.nu) return;
    const int32_t I = (int32_t)t;
    const uint32_t gk = fdiv((uint32_t)I, sf.fnh);
    const int32_t h = I - (int32_t)(gk * sf.fnh.d);
    const double *qsi = qs + I, *qni = qn + I;
    const double mi = p.Minv[I];
    const int top = sf.nz * N;
    const bool folded = !PLAIN && fold && gk != 0 && gk != (uint32_t)top;
    double qsv[5] = {0, 0, 0, 0, 0}, qnv[5] = {0, 0, 0, 0, 0};
    if (!PLAIN)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            qsv[v] = folded ? 0.0 : qsi[v * p.nu];
            qnv[v] = c.a == 0.0 ? 0.0 : qni[v * p.nu];
        }
    // radial copies: (layer, local k)
    int ez[2], kz[2], nzc = 1;
    if (gk == (uint32_t)top) {
        ez[0] = sf.nz - 1;
        kz[0] = N;
    } else {
        ez[0] = (int)(gk / N);
        kz[0] = (int)(gk - (uint32_t)ez[0] * N);
        if (kz[0] == 0 && ez[0] > 0) {
            ez[1] = ez[0] - 1;
            kz[1] = N;
            nzc = 2;
        }
    }
    const int32_t hb = sf.hoff[h], hn = sf.hoff[h + 1] - hb;
    int32_t hc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) hc[q] = sf.hidx[hb + (q < hn ? q : hn - 1)];
    double r[5] = {0, 0, 0, 0, 0};
    for (int z = 0; z < nzc; ++z) {
        const int64_t base = ez[z] * sf.layer + PP * kz[z];
        T c[4][5];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T *src = ev + (base + hc[q]) * 5;
            if (q < hn) {  // absent copies are not loaded
#pragma unroll
                for (int v = 0; v < 5; ++v) c[q][v] = src[v];
            } else {
#pragma unroll
                for (int v = 0; v < 5; ++v) c[q][v] = (T)0;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int v = 0; v < 5; ++v) r[v] += q < hn ? (double)c[q][v] : 0.0;
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v] *= mi;
    double *qoi = qout + I;
    if (folded) {
#pragma unroll
        for (int v = 0; v < 5; ++v) qoi[v * p.nu] = rk_update_folded(c, qnv[v], r[v]);
        return;
    }
    noflux(p, I, r[1], r[2], r[3]);
#pragma unroll
    for (int v = 0; v < 5; ++v) qoi[v * p.nu] = PLAIN ? r[v] : rk_update(c, qnv[v], qsv[v], r[v]);
}

inline unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

template <typename T, bool PLAIN = false>
void launch_shell_finish_t(Mesh &m, const T *ev, const StageCoef &c, const double *qn, const double *qs,
                           double *qout, hipStream_t s, int fold = 0)
{
    PointArgs p = point_args(m);
    if (!PLAIN) p.Minv = stage_minv(m);  // the shell filter takes the stored J w
    ShellFin sf;
    sf.hoff = m.dv.hoff;
    sf.hidx = m.dv.hidx;
    sf.fnh = fast_div((uint32_t)m.nh);
    sf.nz = m.d.ne[2];
    sf.layer = 6 * (int64_t)m.d.ne[0] * m.d.ne[0] * m.np;
    const dim3 grid(nblocks(m.nu, 256)), block(256);
    switch (m.N) {
    case 1: hipLaunchKernelGGL((k_shell_finish<1, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    case 2: hipLaunchKernelGGL((k_shell_finish<2, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    case 3: hipLaunchKernelGGL((k_shell_finish<3, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    case 4: hipLaunchKernelGGL((k_shell_finish<4, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    case 5: hipLaunchKernelGGL((k_shell_finish<5, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    case 6: hipLaunchKernelGGL((k_shell_finish<6, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    case 7: hipLaunchKernelGGL((k_shell_finish<7, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    default: hipLaunchKernelGGL((k_shell_finish<8, T, PLAIN>), grid, block, 0, s, p, sf, ev, c, fold, qn, qs, qout); break;
    }
}

}  // namespace

int32_t launch_dss(Mesh &m, int32_t nvar, const double *cin, double *out, int32_t flags, hipStream_t s)
{
    const bool shell = m.d.kind == NUMA_MESH_SHELL;
    const PointArgs p = point_args(m);
    DssGeo g{};
    g.fi = fast_div((uint32_t)(shell ? m.nh : m.ni));
    g.fj = fast_div((uint32_t)(shell ? 1 : m.nj));
    g.nx = m.d.ne[0];
    g.ny = m.d.ne[1];
    g.nz = m.d.ne[2];
    g.walls = m.walls ? 1 : 0;
    g.hoff = m.dv.hoff;
    g.hidx = m.dv.hidx;
    g.layer = shell ? 6 * m.d.ne[0] * m.d.ne[0] * m.np : 0;
    const uint32_t nb = nblocks(m.nu, 256);
    const FastDiv fb = fast_div(nb);
    const int nv = shell && m.nl >= 300000 ? (nvar < 5 ? nvar : 5) : 1;
    const int groups = (nvar + nv - 1) / nv, most = (int)(((1u << 24) - 1) / nb);  // fewer than 2^32 lanes a launch
    auto launch_nv = [&](auto order, auto vars) {
        constexpr int N = decltype(order)::value, NV = decltype(vars)::value;
        for (int g0 = 0; g0 < groups; g0 += most) {
            const dim3 grid(nb * (unsigned)(groups - g0 < most ? groups - g0 : most));
            if (shell)
                hipLaunchKernelGGL((k_dss<N, true, NV>), grid, dim3(256), 0, s, p, g, fb, g0 * NV, nvar, cin, out, flags);
            else if constexpr (NV == 1)
                hipLaunchKernelGGL((k_dss<N, false, 1>), grid, dim3(256), 0, s, p, g, fb, g0, nvar, cin, out, flags);
        }
    };
    auto launch = [&](auto order) {
        switch (nv) {
        case 1: launch_nv(order, std::integral_constant<int, 1>{}); break;
        case 2: launch_nv(order, std::integral_constant<int, 2>{}); break;
        case 3: launch_nv(order, std::integral_constant<int, 3>{}); break;
        case 4: launch_nv(order, std::integral_constant<int, 4>{}); break;
        default: launch_nv(order, std::integral_constant<int, 5>{}); break;
        }
    };
    switch (m.N) {
    case 1: launch(std::integral_constant<int, 1>{}); break;
    case 2: launch(std::integral_constant<int, 2>{}); break;
    case 3: launch(std::integral_constant<int, 3>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 5: launch(std::integral_constant<int, 5>{}); break;
    case 6: launch(std::integral_constant<int, 6>{}); break;
    case 7: launch(std::integral_constant<int, 7>{}); break;
    default: launch(std::integral_constant<int, 8>{}); break;
    }
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

StageCoef ssp33_stage(int stage, double dt)
{
    if (stage == 0) return StageCoef{0.0, 1.0, dt};
    if (stage == 1) return StageCoef{0.75, 0.25, dt};
    return StageCoef{1.0 / 3.0, 2.0 / 3.0, dt};
}

int32_t launch_rk_stage(Mesh &m, int32_t stage, double dt, const double *qn, const double *qs, const double *r,
                        double *qout, hipStream_t s)
{
    int64_t n = 5 * m.nu;
    hipLaunchKernelGGL(k_rk_stage, dim3(nblocks(n, 256)), dim3(256), 0, s, n, ssp33_stage(stage, dt), qn, qs, r,
                       qout);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

int32_t launch_shell_plain_finish(Mesh &m, const double *ev, double *q, hipStream_t s)
{
    launch_shell_finish_t<double, true>(m, ev, StageCoef{0.0, 1.0, 0.0}, nullptr, nullptr, q, s);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

int32_t launch_stage_finish(Mesh &m, int32_t prec, const StageCoef &c, const double *qn, const double *qs,
                            double *qout, hipStream_t s)
{
    if (prec == NUMA_PREC_MIXED)
        launch_shell_finish_t<float>(m, m.dv.ev32, c, qn, qs, qout, s);
    else
        launch_shell_finish_t<double>(m, m.dv.ev64, c, qn, qs, qout, s, shell_folds(m, prec, c) ? 1 : 0);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

}  // namespace numa
