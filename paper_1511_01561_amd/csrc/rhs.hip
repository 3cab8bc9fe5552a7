// Element-wise right-hand side (the paper's create_rhs): Eq. (discstrongform)
// with the derivatives of Eq. (derivatives) (chain rule through the metric).
//
// One workgroup per element, one lane per element-local node.  The unique
// state is gathered through the element -> unique map, the equation of state
// is evaluated in FP64, and the eight differentiated fields
//   rho u, rho v, rho w, u, v, w, theta', p'   (+ theta_bar on the shell)
// are staged once in LDS so that all fields are differentiated from one tile
// (the paper's "all derivatives of an element in one matrix per direction").
// Each lane keeps its three rows of the derivative matrix in registers.
//
// The kernel writes the element-local contributions J w R (the E-vector),
// element-major so that every element writes whole cache lines: in FP64 for
// numa_rhs, and in the contraction precision for the element half of a fused
// stage (the finish kernel sums them).
#include <cmath>

#include "kernels.h"

namespace numa {
namespace {

using namespace dev;

// NM: node-major output [n_local][5] (the element's 5 (N+1)^3 values staged
// through the tile and written as one contiguous run), for the shell's fused
// stage; otherwise element-major [5][n_local].
template <int N, typename T, typename TO, bool SHELL, int GEO, bool NM = false>
__global__ __launch_bounds__(block_threads<N>()) void k_rhs(RhsArgs<T> a, TO *out)
{
    constexpr int NP = (N + 1) * (N + 1) * (N + 1), NF = SHELL ? 9 : 8, BT = block_threads<N>();
    __shared__ T s[NF][NP];
    const int64_t e = xcd_remap(blockIdx.x, gridDim.x);
    const int l = threadIdx.x;
    NodeOut<T> o;
    if constexpr (NM) {
        static_assert(sizeof(TO) == sizeof(T), "node-major output is staged in the tile");
        // element_rhs, with the node's state kept for the fold
        NodeIn<T> in;
        node_gather<N, T, SHELL, GEO>(a, e, l, in);
        node_stage<N, T, SHELL, GEO>(a, e, l, in, s);
        __syncthreads();
        const bool act = l < NP;
        if (act) {
            T Di[N + 1], Dj[N + 1], Dk[N + 1];
            d_rows<N, T>(a.D, l, Di, Dj, Dk);
            node_derive<N, T, SHELL, GEO>(a, l, in, Di, Dj, Dk, s, o);
        }
        __syncthreads();  // every lane has finished reading the tile
        TO *st = (TO *)&s[0][0];
        if (act) {
            // J w R, or J w (q_s + cdt R) away from the bottom and top layers
            const int ez = (int)fdiv((uint32_t)e, a.feh), k = l / ((N + 1) * (N + 1));
            const bool wall = (ez == 0 && k == 0) || (ez == a.nz - 1 && k == N);
            if (sizeof(T) == 8 && a.fold && !wall) {
                const double qv[5] = {in.rp, in.u, in.v, in.w, in.tp};
#pragma unroll
                for (int v = 0; v < 5; ++v) st[l * 5 + v] = (TO)(o.Jw * fma((T)a.cdt, o.R[v], (T)qv[v]));
            } else {
#pragma unroll
                for (int v = 0; v < 5; ++v) st[l * 5 + v] = (TO)(o.Jw * o.R[v]);
            }
        }
        __syncthreads();
        TO *dst = out + e * (NP * 5);
#pragma unroll
        for (int r = 0; r < (NP * 5 + BT - 1) / BT; ++r) {
            const int t = l + r * BT;
            if (t < NP * 5) dst[t] = st[t];
        }
    } else {
        const bool act = element_rhs<N, T, SHELL, GEO>(a, e, l, s, o);
        if (!act) return;
        TO *p = out + e * NP + l;
#pragma unroll
        for (int v = 0; v < 5; ++v) p[v * a.nl] = (TO)(o.Jw * o.R[v]);
    }
}

// The element kernel of a shell stage with the recomputed metric, a lane per
// (i, j) column: the two-pass tile of the box's k_elem_col2.  One node per lane
// (k_rhs above) reads 15 tile values per field and node at N = 4 (27 contractions
// of 5), forms every node's metric, gravity and reference loads for itself, and
// waits for one gather at three waves per SIMD.  Here the tile holds p', u, v,
// w, theta' (momentum and theta' rows), then rho u, rho v, rho w (mass row; in
// mixed precision they are formed at the gather, from the FP64 velocity as in
// k_rhs, and have the FP32 tile's room beside the others); the zeta derivatives
// come from the lane's own column, which it reads once, the column factors of the
// metric are loaded once per column, and the reference and the layer factors, the
// same for all nodes of a level, once per level from one address.  theta_bar varies
// along zeta only.
//
// Waves per SIMD the registers are held to, and elements per workgroup: as many as
// four wavefronts and the workgroup's share of the LDS at that occupancy hold.
template <int N, typename T> constexpr int shell_waves() { return sizeof(T) == 8 ? 2 : N <= 4 ? 4 : N <= 6 ? 3 : 2; }
// Fluxes in the slots of the fields before them: FP64, and mixed N = 6, where eight
// fields leave room for four elements in place of five (step at 6x12x12x8 274 against
// 271 us; there the fluxes wait in registers, 32 bytes of spill a lane).
template <int N, typename T> constexpr bool shell_two_pass() { return sizeof(T) == 8 || N == 6; }
template <int N, typename T> constexpr int shell_fields() { return shell_two_pass<N, T>() ? 5 : 8; }  // of the tile
// Values after an element's tile that spread the elements of a wavefront over the LDS
// banks.  Mixed: one element's columns follow the other's in the 64 banks (at N = 1
// every element starts at the same bank otherwise: step at 6x60x60x10 201 against
// 150 us); at N = 4 that takes a workgroup off the CU.
template <int N, typename T> constexpr int shell_pad()
{
    constexpr int PP = (N + 1) * (N + 1), over = (shell_fields<N, T>() * PP * (N + 1) - PP) % 64;
    return sizeof(T) == 8 ? (N == 4 ? 8 : 0) : N == 4 ? 0 : (64 - over) % 64;
}
template <int N, typename T> constexpr int shell_eb()
{
    constexpr int PP = (N + 1) * (N + 1), lanes = 256 / PP;
    constexpr int tile = (shell_fields<N, T>() * PP * (N + 1) + shell_pad<N, T>()) * (int)sizeof(T);
    constexpr int lds = 163840 / shell_waves<N, T>() / tile;
    return lanes < lds ? lanes : lds;
}
template <int N, typename T> constexpr int shell_threads()
{
    return (shell_eb<N, T>() * (N + 1) * (N + 1) + 63) / 64 * 64;
}
// The column kernel from this many element-local nodes on: below, too few
// workgroups with too long a chain each (one node per lane / columns, us per step,
// at sizes about the line).  FP64: N = 1 14 k 36 / 38, 28 k 43 / 39; 2: 78 k 39 / 41,
// 159 k 55 / 47; 3: 555 k 87 / 91, 677 k 100 / 97; 4: 432 k 84 / 89, 588 k 102 / 93; 5: 187 k
// 60 / 67, 332 k 82 / 79; 6: 154 k 56 / 83, 296 k 102 / 94; 7: 442 k 113 / 126, 786 k 167 /
// 160; 8: 2.6 M 652 / 709 (spills: not taken).  Mixed: 1: 14 k 34 / 35, 28 k 38 / 35; 2: 41 k
// 34 / 38, 78 k 39 / 39; 3: 276 k 56 / 57, 376 k 64 / 63; 4: 432 k 71 / 78, 588 k 86 / 83; 5:
// 332 k 66 / 68, 648 k 97 / 94; 6: 154 k 48 / 67, 296 k 83 / 77; 7: 786 k 125 / 122; 8: 280 k
// 81 / 94, 437 k 108 / 101.
template <int N, typename T> constexpr int64_t shell_col_from()
{
    constexpr int64_t f64[9] = {0, 20000, 90000, 600000, 560000, 300000, 250000, 700000, INT64_MAX};
    constexpr int64_t f32[9] = {0, 20000, 90000, 350000, 560000, 600000, 250000, 700000, 400000};
    return sizeof(T) == 8 ? f64[N] : f32[N];
}
// Element kernel, one node per lane -> columns: 32x32x10 at N = 4 (61,440
// elements) FP64 304 -> 234 us, mixed 217 -> 142; N = 2 83 -> 37, mixed 61 -> 27; 20x20x8
// at N = 5 215 -> 137, mixed 131 -> 89; 16x16x8 at N = 6 273 -> 170, mixed 188 -> 101;
// 14x14x8 at N = 7 299 -> 205, mixed 169 -> 123; mixed 12x12x8 at N = 8 251 -> 145.
// Waves per SIMD: FP64 at N = 4 three spill 128 bytes (282 against 234 us); N = 7
// spills 32 at two.
template <int N, typename T>
__global__ __launch_bounds__((shell_threads<N, T>()), (shell_waves<N, T>())) void k_shell_col(RhsArgs<T> a, int ne, T *out)
{
    constexpr int P = N + 1, PP = P * P, NP = PP * P, EB = shell_eb<N, T>(), BT = shell_threads<N, T>();
    constexpr bool F64 = sizeof(T) == 8;
    constexpr bool EARLY = F64 || N < 4 || N == 8;
    constexpr bool TWO = shell_two_pass<N, T>();
    constexpr int FL = TWO ? 0 : 5;  // tile slot of the mass fluxes
    __shared__ __align__(16) T s[EB][shell_fields<N, T>() * NP + shell_pad<N, T>()];
    const int e0 = (int)xcd_remap(blockIdx.x, gridDim.x) * EB;
    const int t = threadIdx.x, q = t / PP, c = t % PP, i = c % P, j = c / P;
    const bool act = q < EB && e0 + q < ne;
    T *S = &s[act ? q : 0][0];
    T Di[P], Dj[P];
#pragma unroll
    for (int m = 0; m < P; ++m) {
        Di[m] = a.D[i * P + m];
        Dj[m] = a.D[j * P + m];
    }
    // of the column: metric factors (xi, eta, zeta rows), J w, direction; of its
    // nodes: rho, 1/rho, rho' (FP64) or rho'/rho
    double F[9], jwc = 0.0, dn[3], rho[P];
    T ir[P], bq[P], tb[P], fl[P][3];
    int ez = 0;
    const double *lay = a.slay;
    if (act) {
        ez = (int)fdiv((uint32_t)(e0 + q), a.feh);
        const int eh = e0 + q - ez * (int)a.feh.d;
        lay = a.slay + 4 * ez * P;
        const double *cp = a.scol + (int64_t)eh * (13 * PP) + c;
        auto factors = [&]() {
#pragma unroll
            for (int d = 0; d < 9; ++d) F[d] = cp[d * PP];
            jwc = cp[9 * PP];
#pragma unroll
            for (int d = 0; d < 3; ++d) dn[d] = cp[(10 + d) * PP];
        };
        // before the gather, or behind it where their 26 registers beside its
        // values cost more than the wait (mixed N = 4 spills 48 bytes with them,
        // N = 6 loses a wave: step at 6x12x12x8 271 against 324 us)
        if constexpr (EARLY) factors();
        const int64_t level = a.nh * ((int64_t)ez * N);
        const double *qp = a.q + (level + a.shid[eh * PP + c]), *rf = a.ref + level;
        double qv[P][5], rb[P], tbk[P], pb[P], x[P], pp[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
#pragma unroll
            for (int v = 0; v < 5; ++v) qv[k][v] = qp[v * a.nu + a.nh * k];
            rb[k] = rf[a.nh * k];
            tbk[k] = rf[a.nu + a.nh * k];
            pb[k] = rf[2 * a.nu + a.nh * k];
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            x[k] = box_eos_x(qv[k][0], qv[k][4], rb[k], tbk[k]);
            rho[k] = rb[k] + qv[k][0];
            const double ird = 1.0 / rho[k];
            ir[k] = (T)ird;
            bq[k] = F64 ? (T)qv[k][0] : (T)(qv[k][0] * ird);
            tb[k] = (T)(tbk[k] - tbk[0]);
#pragma unroll
            for (int v = 1; v < 5; ++v) S[v * NP + c + PP * k] = (T)qv[k][v];
            if (!F64)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    const T f = (T)(rho[k] * qv[k][1 + b]);
                    if (TWO) fl[k][b] = f;
                    else S[(FL + b) * NP + c + PP * k] = f;
                }
        }
        eos_nodes<P>(P, x, pb, a.gamma, a.eos, pp);
#pragma unroll
        for (int k = 0; k < P; ++k) S[c + PP * k] = (T)pp[k];
        if constexpr (!EARLY) {
            __builtin_amdgcn_sched_barrier(0);
            factors();
        }
    }
    auto metric = [&](int k, T *mx) {
        const double r = lay[4 * k], z = lay[4 * k + 1];
#pragma unroll
        for (int d = 0; d < 9; ++d) mx[d] = (T)(F[d] * (d < 6 ? r : z));
        mx[9] = (T)(jwc * lay[4 * k + 2]);
    };
    auto folds = [&](int k) { return a.fold && !((ez == 0 && k == 0) || (ez == a.nz - 1 && k == N)); };
    auto derive = [&](int f, int k, T *d) {
        d[0] = dot<P>(Di, [&](int m) { return S[f * NP + m + P * (j + P * k)]; });
        d[1] = dot<P>(Dj, [&](int m) { return S[f * NP + i + P * (m + P * k)]; });
        d[2] = dot<P>(a.D + k * P, [&](int m) { return S[f * NP + c + PP * m]; });
    };
    const T cdt = (T)a.cdt;
    T res[P][5];
    __syncthreads();  // first tile complete
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            T mx[10], d[3], U[3], R[5];
            metric(k, mx);
            T qv[5];
#pragma unroll
            for (int v = 1; v < 5; ++v) qv[v] = S[v * NP + c + PP * k];
#pragma unroll
            for (int b = 0; b < 3; ++b) U[b] = qv[1] * mx[3 * b] + qv[2] * mx[3 * b + 1] + qv[3] * mx[3 * b + 2];
#pragma unroll
            for (int v = 1; v < 5; ++v) {
                derive(v, k, d);
                R[v] = -(U[0] * d[0] + U[1] * d[1] + U[2] * d[2]);
            }
            R[4] -= U[2] * dot<P>(a.D + k * P, [&](int m) { return tb[m]; });
            derive(0, k, d);
            const T bk = F64 ? bq[k] * ir[k] : bq[k];
            const double ga = -lay[4 * k + 3];
#pragma unroll
            for (int b = 0; b < 3; ++b)
                R[1 + b] += bk * (T)(ga * dn[b]) - (d[0] * mx[b] + d[1] * mx[3 + b] + d[2] * mx[6 + b]) * ir[k];
            const bool fold = F64 && folds(k);
#pragma unroll
            for (int v = 1; v < 5; ++v) res[k][v] = mx[9] * (fold ? fma(cdt, R[v], qv[v]) : R[v]);
            __builtin_amdgcn_sched_barrier(0);  // a node's lines at a time: registers
        }
    }
    // the mass fluxes (FP64: formed from the first tile)
    if (act && (F64 || !TWO)) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int b = 0; b < 3; ++b)
                fl[k][b] = F64 ? (T)(rho[k] * (double)S[(1 + b) * NP + c + PP * k]) : S[(FL + b) * NP + c + PP * k];
    }
    if constexpr (TWO) {
        __syncthreads();  // first tile read
        if (act) {
#pragma unroll
            for (int k = 0; k < P; ++k)
#pragma unroll
                for (int b = 0; b < 3; ++b) S[(FL + b) * NP + c + PP * k] = fl[k][b];
        }
        __syncthreads();  // second tile complete
    }
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            T mx[10], dv = 0;
            metric(k, mx);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                T d[3];
                d[0] = dot<P>(Di, [&](int m) { return S[(FL + b) * NP + m + P * (j + P * k)]; });
                d[1] = dot<P>(Dj, [&](int m) { return S[(FL + b) * NP + i + P * (m + P * k)]; });
                d[2] = dot<P>(a.D + k * P, [&](int m) { return fl[m][b]; });
                dv += d[0] * mx[b] + d[1] * mx[3 + b] + d[2] * mx[6 + b];
            }
            const bool fold = F64 && folds(k);
            res[k][0] = mx[9] * (fold ? fma(cdt, -dv, bq[k]) : -dv);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();  // fluxes read
    T *st = &s[0][0];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) st[(q * NP + c + PP * k) * 5 + v] = res[k][v];
    }
    __syncthreads();
    // the workgroup's elements are consecutive: one contiguous run
    const int nel = ne - e0 < EB ? ne - e0 : EB;
    store_run<T>(out + (int64_t)e0 * (NP * 5), st, nel * NP * 5, t, BT);
}

template <int N, typename T, typename TO>
void launch_n(Mesh &m, const RhsArgs<T> &a, TO *out, bool node_major, hipStream_t s)
{
    dim3 grid((unsigned)m.ne), block(block_threads<N>());
    if constexpr (sizeof(TO) == sizeof(T)) {
        if (node_major && m.d.kind == NUMA_MESH_SHELL) {
            if (m.metric_mode == NUMA_METRIC_RECOMPUTE) {
                if (m.nl < shell_col_from<N, T>()) {
                    hipLaunchKernelGGL((k_rhs<N, T, TO, true, kMetricShell, true>), grid, block, 0, s, a, out);
                    return;
                }
                if constexpr (shell_col_from<N, T>() < INT64_MAX) {
                    constexpr int EB = shell_eb<N, T>();
                    hipLaunchKernelGGL((k_shell_col<N, T>), dim3((unsigned)((m.ne + EB - 1) / EB)),
                                       dim3(shell_threads<N, T>()), 0, s, a, (int)m.ne, out);
                }
            } else
                hipLaunchKernelGGL((k_rhs<N, T, TO, true, kMetricStored, true>), grid, block, 0, s, a, out);
            return;
        }
    }
    if (m.d.kind == NUMA_MESH_SHELL && m.metric_mode == NUMA_METRIC_RECOMPUTE)
        hipLaunchKernelGGL((k_rhs<N, T, TO, true, kMetricShell>), grid, block, 0, s, a, out);
    else if (m.d.kind == NUMA_MESH_SHELL)
        hipLaunchKernelGGL((k_rhs<N, T, TO, true, kMetricStored>), grid, block, 0, s, a, out);
    else if (m.metric_mode == NUMA_METRIC_RECOMPUTE)
        hipLaunchKernelGGL((k_rhs<N, T, TO, false, kMetricBox>), grid, block, 0, s, a, out);
    else
        hipLaunchKernelGGL((k_rhs<N, T, TO, false, kMetricStored>), grid, block, 0, s, a, out);
}

template <typename T, typename TO>
void launch_t(Mesh &m, const T *met, const T *D, const double *q, TO *out, bool node_major, hipStream_t s,
              double cdt = 0.0, int fold = 0)
{
    RhsArgs<T> a;
    a.cdt = cdt;
    a.fold = fold;
    a.G = m.dv.G;
    a.q = q;
    a.ref = m.dv.ref;
    a.grav = m.dv.grav;
    a.met = met;
    a.D = D;
    a.nl = m.nl;
    a.nu = m.nu;
    a.gamma = m.gamma;
    a.g0 = m.ph.g0;
    a.hcol = m.dv.hcol;
    a.nx = m.d.ne[0];
    a.ny = m.d.ne[1];
    a.nz = m.d.ne[2];
    a.fx = fast_div((uint32_t)m.d.ne[0]);
    a.fy = fast_div((uint32_t)m.d.ne[1]);
    a.scol = m.dv.scol;
    a.slay = m.dv.slay;
    a.shid = m.dv.shid;
    a.nh = m.nh;
    a.feh = fast_div((uint32_t)(m.d.kind == NUMA_MESH_SHELL ? 6 * m.d.ne[0] * m.d.ne[0] : 1));
    if (m.d.kind == NUMA_MESH_BOX) a.bm = box_metric(m);
    eos_coeffs(m.gamma, a.eos);
    a.xi = m.dv.xi64;
    a.w = m.dv.w64;
    a.ni = (int)m.ni;
    a.nj = (int)m.nj;
    a.nk = m.d.periodic[2] ? (int)m.nk : -1;  // only a periodic z wraps
    switch (m.N) {
    case 1: launch_n<1, T, TO>(m, a, out, node_major, s); break;
    case 2: launch_n<2, T, TO>(m, a, out, node_major, s); break;
    case 3: launch_n<3, T, TO>(m, a, out, node_major, s); break;
    case 4: launch_n<4, T, TO>(m, a, out, node_major, s); break;
    case 5: launch_n<5, T, TO>(m, a, out, node_major, s); break;
    case 6: launch_n<6, T, TO>(m, a, out, node_major, s); break;
    case 7: launch_n<7, T, TO>(m, a, out, node_major, s); break;
    default: launch_n<8, T, TO>(m, a, out, node_major, s); break;
    }
}

}  // namespace

int32_t launch_rhs(Mesh &m, int32_t prec, const double *q, double *evec, hipStream_t s)
{
    if (prec == NUMA_PREC_MIXED)
        launch_t<float, double>(m, m.dv.met32, m.dv.D32, q, evec, false, s);
    else
        launch_t<double, double>(m, m.dv.met, m.dv.D64, q, evec, false, s);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

// element half of a fused stage of the shell: node-major contributions into
// the workspace E-vector (FP32 on the mixed path)
int32_t launch_stage_elements(Mesh &m, int32_t prec, const StageCoef &c, const double *qs, hipStream_t s)
{
    if (prec == NUMA_PREC_MIXED)
        launch_t<float, float>(m, m.dv.met32, m.dv.D32, qs, m.dv.ev32, true, s);
    else
        launch_t<double, double>(m, m.dv.met, m.dv.D64, qs, m.dv.ev64, true, s, c.cdt, shell_folds(m, prec, c) ? 1 : 0);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

}  // namespace numa
