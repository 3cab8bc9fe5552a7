// Batched fused stages on box meshes: the elements and nodes of several
// independent solves of the same order advance together, one element launch
// and one finish launch per stage for the whole batch (continuous batching of
// ensemble members and regional solves).  Each item brings its own state and
// private scratch; geometry may be shared between items.  The per-element
// and per-node arithmetic is the single-mesh code (kernels.h), so an item's
// result does not depend on what it is batched with.  A single box mesh
// (numa_step) runs through the same kernels with one item.
#include "kernels.h"

#include <vector>

namespace numa {
// The mesh leaves the way its stages run to the launch's size: NUMA_STAGE_AUTO,
// and NUMA_STAGE_SPLIT with the stored metric (a small launch takes twice as long
// through the split DSS as with one node per lane: 51 k nodes at N = 7 89 against 39
// us a step).
static bool stage_by_size(const Mesh &m)
{
    return m.stage_mode == NUMA_STAGE_AUTO ||
           (m.stage_mode == NUMA_STAGE_SPLIT && m.metric_mode == NUMA_METRIC_STORED);
}

namespace {

using namespace dev;

constexpr int kMaxBatch = 16;  // items per launch (kernel-argument table)

// How the items of a launch run a stage: the gather DSS with the element
// kernel of the order and precision, the colour passes, the split DSS, or the
// gather DSS with one node per lane (small launches)
enum { kGather = 0, kColour = 1, kSplit = 2, kNode = 3 };

struct BatchItem {
    const double *qs;  // stage input state [5][nu]
    double *qout;      // stage output state
    const double *qn;  // reference state of the stage update (q^n or an earlier stage)
    const double *ref, *Minv, *nrm;
    const void *met;      // [ne][10][np] of T
    void *ev;             // [nl][5] of T: contributions of this stage, node-major
    const double *hcol;   // column factors of the recomputed metric
    int32_t *flag;        // non-finite flag of the item's state, or null
    int nu, nh;           // unique nodes, per level (meshes are limited to 32-bit indices)
    int ni, nj, nkw;      // lattice extents; nkw: extent in z when periodic, else -1
    int nz, walls;
    int ne;               // elements
    int mblk;             // finish blocks of the main layers: (nx/SEG) ny nz (split: of the face rows)
    FastDiv fx, fy, fseg;  // division by nx, ny and nx/SEG (colour passes: fseg by nx/2, fy by ny/2;
                           // split: fseg by ni)
    FastDiv frl;           // split: division by the face rows per element layer, nj + (N - 1) ny
    double cdt;            // (beta / b) dt of the stage update
    double theta0;         // the box reference is isentropic: theta_bar = theta0 everywhere
    BoxMetric bm;          // constants of the recomputed metric
    int eoff, boff;        // first element / finish block of this item in the launch (eoff: a
                           // multiple of the elements per element workgroup)
};

struct Batch {
    int n;
    int fold;       // the column kernel folds q_s into the contributions (box_finish_node)
    double ca, cb;  // weights of the reference state and of the stage in the update (same for all items)
    double gamma, g0;
    const void *D;
    const double *xi, *w;  // FP64 GLL nodes, weights
    double eos[kEosTerms];
    BatchItem it[kMaxBatch];
};
static_assert(sizeof(Batch) <= 4096, "the batch table must fit the kernel arguments");

// The gather of a column kernel: calls f(k, q, rho_bar, x, p') for the nodes
// k = 0..P-1 of the column based at unique node `base` (levels `layer` apart,
// wrapping at nk), G nodes' loads in flight together; G below P where the
// registers of more do not pay.
template <int P, int G, typename T, typename F>
__device__ __forceinline__ void gather_column(const RhsArgs<T> &a, double theta0, int base, int layer, int gk0, F f)
{
#pragma unroll
    for (int k0 = 0; k0 < P; k0 += G) {
        const int n = P - k0 < G ? P - k0 : G;
        double q[G][5], rb[G], pb[G], x[G], pp[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            if (k >= n) continue;
            int gk = gk0 + k0 + k;
            if (gk == a.nk) gk = 0;
            const int32_t I = base + layer * gk;
            const double *qp = a.q + I, *rf = a.ref + I;
#pragma unroll
            for (int v = 0; v < 5; ++v) q[k][v] = qp[v * a.nu];
            rb[k] = rf[0];
            pb[k] = rf[2 * a.nu];
        }
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (k < n) x[k] = box_eos_x(q[k][0], q[k][4], rb[k], theta0);
        eos_nodes<G>(n, x, pb, a.gamma, a.eos, pp);
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (k < n) f(k0 + k, q[k], rb[k], pp[k]);
    }
}

// item of launch-wide block g (items are in ascending eoff / boff order)
__device__ __forceinline__ int batch_item(const Batch &B, int g, bool fin)
{
    int k = 0;
    while (k + 1 < B.n && g >= (fin ? B.it[k + 1].boff : B.it[k + 1].eoff)) ++k;
    return k;
}

// element-kernel arguments of one batch item
template <typename T>
__device__ __forceinline__ RhsArgs<T> elem_args(const Batch &B, const BatchItem &it)
{
    RhsArgs<T> a;
    a.G = nullptr;
    a.q = it.qs;
    a.ref = it.ref;
    a.grav = nullptr;
    a.met = (const T *)it.met;
    a.D = (const T *)B.D;
    a.hcol = it.hcol;
    a.nl = 0;
    a.nu = it.nu;
    a.gamma = B.gamma;
    a.g0 = B.g0;
    a.nx = (int)it.fx.d;
    a.ny = (int)it.fy.d;
    a.nz = it.nz;
    a.ni = it.ni;
    a.nj = it.nj;
    a.nk = it.nkw;
    a.fx = it.fx;
    a.fy = it.fy;
    a.scol = nullptr;
    a.slay = nullptr;
    a.shid = nullptr;
    a.nh = it.nh;
    a.feh = FastDiv{1, 1, 0, 0};
    a.bm = it.bm;
#pragma unroll
    for (int c = 0; c < kEosTerms; ++c) a.eos[c] = B.eos[c];
    a.xi = B.xi;
    a.w = B.w;
    return a;
}

// node-major [n_local][5] output of element e (a copy's five values in one
// run for the finish), staged through LDS (st, 5 (N+1)^3 values) so that the
// block writes them as one contiguous, coalesced run; the caller has
// synchronised after writing st
template <int N, typename T>
__device__ __forceinline__ void store_contributions(const BatchItem &it, int e, int l, const T *st)
{
    constexpr int NP = (N + 1) * (N + 1) * (N + 1), BT = block_threads<N>();
    T *out = (T *)it.ev + (int64_t)e * (NP * 5);
#pragma unroll
    for (int r = 0; r < (NP * 5 + BT - 1) / BT; ++r) {
        const int t = l + r * BT;
        if (t < NP * 5) out[t] = st[t];
    }
}

// One workgroup per element (the launch-wide element index, XCD-remapped).  At
// N = 8 a workgroup is three wavefronts on each SIMD: in FP32 the registers are
// held to six, two workgroups (one more register costs a workgroup).
template <int N, typename T, int GEO>
__global__ __launch_bounds__(block_threads<N>(), N == 8 && sizeof(T) == 4 ? 6 : 1) void k_elem_batch(Batch B)
{
    constexpr int NP = (N + 1) * (N + 1) * (N + 1);
    __shared__ T s[8][NP];
    const int g = (int)xcd_remap(blockIdx.x, gridDim.x);
    const BatchItem &it = B.it[batch_item(B, g, false)];
    const int e = g - it.eoff;
    const RhsArgs<T> a = elem_args<T>(B, it);
    NodeOut<T> o;
    const int l = threadIdx.x;
    const bool act = l < NP;
    // element_rhs, with the node's state kept for the fold
    NodeIn<T> in;
    node_gather<N, T, false, GEO>(a, e, l, in);
    node_stage<N, T, false, GEO>(a, e, l, in, s);
    __syncthreads();
    if (act) {
        T Di[N + 1], Dj[N + 1], Dk[N + 1];
        d_rows<N, T>(a.D, l, Di, Dj, Dk);
        node_derive<N, T, false, GEO>(a, l, in, Di, Dj, Dk, s, o);
    }
    __syncthreads();  // every lane has finished reading the tile
    T *st = &s[0][0];
    if (act) {
        const int k = l / ((N + 1) * (N + 1));
        const bool wall = it.walls && ((in.ez == 0 && k == 0) || (in.ez == it.nz - 1 && k == N));
        if (sizeof(T) == 8 && B.fold && !wall) {  // J w (q_s + cdt R), as in k_elem_col
            const double qv[5] = {in.rp, in.u, in.v, in.w, in.tp};
#pragma unroll
            for (int v = 0; v < 5; ++v) st[l * 5 + v] = o.Jw * fma((T)it.cdt, o.R[v], (T)qv[v]);
        } else {
#pragma unroll
            for (int v = 0; v < 5; ++v) st[l * 5 + v] = o.Jw * o.R[v];
        }
    }
    __syncthreads();
    store_contributions<N, T>(it, e, l, st);
}

// Column variant for the recomputed box metric: a workgroup takes EB
// consecutive elements and a lane one (i, j) column of one of them, i.e. the
// N+1 nodes (i, j, 0..N).  The lane gathers its column (all loads in flight
// together), evaluates the equation of state and keeps the column's fields in
// registers: the zeta derivatives are contractions with D_km, which is the
// same for every lane, so they need no LDS.  Only the xi and eta derivatives
// read the element tile.  The arithmetic per node is that of element_rhs.
// Elements per workgroup: as many columns as fill four wavefronts up to
// N = 4 (ten x-consecutive elements at N = 4: longer contiguous runs in the
// gather and the store, measured ~1 % faster than two wavefronts), two
// wavefronts for the streaming variant at N = 5, 6 (its larger tile would
// leave one wavefront per SIMD), one element at N = 7 and 8; the tile (8
// fields of (N+1)^3 nodes per element) stays within 80 KB.
template <int N, typename T>
constexpr int col_eb()
{
    constexpr int PP = (N + 1) * (N + 1);
    return N >= 7 ? 1 : (N <= 4 ? 256 / PP : 128 / PP);
}
template <int N, typename T>
constexpr int col_threads() { return ((col_eb<N, T>() * (N + 1) * (N + 1) + 63) / 64) * 64; }
// elements per workgroup of the split DSS (the run length along x): the column
// kernels' up to N = 4, above that as many as 256 lanes and an 80 KB tile
// (two workgroups per CU) hold: 7, 5, 4, 2 at N = 5..8
template <int N> constexpr int split_eb()
{
    constexpr int PP = (N + 1) * (N + 1), lanes = 256 / PP, lds = 2048 / (PP * (N + 1));
    return N <= 4 ? col_eb<N, double>() : (lanes < lds ? lanes : lds);
}
template <int N> constexpr int split_threads() { return ((split_eb<N>() * (N + 1) * (N + 1) + 63) / 64) * 64; }

// nodes gathered together: the column, or in the streaming kernel as many as
// its occupancy allows
template <int N, typename T> constexpr int col_group() { return N == 4 && sizeof(T) == 4 ? 3 : N + 1; }
template <int N, typename T> constexpr int stream_group() { return N <= 6 ? 4 : 5; }
// workgroups per CU the column kernel is compiled for: in FP32 at N = 4 the
// tile (40 KB) lets four share a CU if the registers fit 4 waves per SIMD
template <int N, typename T, int MODE = 0>
constexpr int col_blocks() { return (sizeof(T) == 4 && N == 4) ? 4 : 1; }

// NUMA_STAGE_SPLIT: the DSS split between the element kernel and a finish
// kernel over the element faces.  The EB elements of a column workgroup are
// consecutive in the element order, so element q's west face (i = 0) and
// element q - 1's east face (i = N) are the same nodes whenever both lie in
// the workgroup and in one row (ex != 0): the workgroup adds those pairs in
// LDS.  A node whose (j, k) is interior to the element (0 < j, k < N) then has
// all its copies in the workgroup unless it sits on the x face that starts
// the run (q = 0 or ex = 0), and the element kernel finishes it itself: M^-1,
// the stage update and the state write (these nodes are never on a wall),
// except in the run's first element (see Fb).  What remains are the face
// nodes (gj or gk a multiple of N: 4N of the (N+1)^2 (j, k) pairs of an
// element, "face pairs") and the interior rows of a run's first element.
// Their contributions are written in two arrays:
//  * Fa [nz][ny][4N][ni][5] (of T): per element row (ey, ez), face pair fp and
//    lattice position gi = ex N + i (i < N) the five values of the
//    contribution of element ex at local i (at i = 0 the pair sum when the run
//    holds element ex - 1), so the finish reads each face row of the lattice
//    as one contiguous run per copy;
//  * Fb [ne][4N + (N-1)^2 (N+1)][5]: the copies the finish kernel takes at
//    run boundaries: slots 0..4N-1 the face pairs at i = N and 4N + ip the
//    interior pair ip at i = N of an element whose east neighbour is not in
//    its run; 4N + (N-1)^2 + ip N + i the interior pair ip at i < N of a run's
//    first element.  The finish kernel takes those N nodes of every interior
//    row at a run start together (whole 32-byte sectors of the state rows,
//    where single scattered nodes would cost a read-modify-write each), so
//    the element kernel finishes none of its first element's nodes.
// Fa, Fb and the face pairs fill (N+1)^3 values per element: the workspace's
// contribution scratch.
// Face pairs fp(j, k): k = 0: j; k = N: N + 1 + j; 0 < k < N: 2 (N+1) +
// 2 (k - 1) + (j == N).  Interior pairs: ip = (j - 1) + (N - 1)(k - 1).
template <int N>
__device__ __forceinline__ int split_fp(int j, int k)
{
    return k == 0 ? j : (k == N ? N + 1 + j : 2 * (N + 1) + 2 * (k - 1) + (j == N ? 1 : 0));
}
template <int N>
__device__ __forceinline__ void split_fp_jk(int fp, int &j, int &k)
{
    if (fp <= N) {
        j = fp;
        k = 0;
    } else if (fp < 2 * (N + 1)) {
        j = fp - (N + 1);
        k = N;
    } else {
        const int r = fp - 2 * (N + 1);
        k = 1 + (r >> 1);
        j = (r & 1) ? N : 0;
    }
}
template <int N> constexpr int split_nb() { return 4 * N + (N - 1) * (N - 1) * (N + 1); }

// what the split-DSS output of a column workgroup needs of its box item
struct SplitGeo {
    int nx, ny, nz, ni, nj, nu;
    FastDiv fx, fy;
};

// the run-interior nodes a lane of a column workgroup (EB elements, BT
// lanes) finishes: interior pair ip, element qq, local ii, not in the run's
// first element, whose west neighbour is not in the workgroup; I = -1 where
// the lane has no node in that pass
template <int N, int EB, int BT>
struct SplitPre {
    static constexpr int NIN = (N - 1) * (N - 1) * EB * N, SPL = NIN > 0 ? (NIN + BT - 1) / BT : 1;
    int32_t I[SPL];
    double m[SPL], qn[SPL][5];
};

// the lane's run-interior nodes and their M^-1 and q^n (loaded at the start
// of the kernel, used at its end)
template <int N, int EB, int BT>
__device__ __forceinline__ void split_prefetch(const BatchItem &it, const SplitGeo &gm, bool load_qn, int t, int e0,
                                               int new_, SplitPre<N, EB, BT> &pf)
{
    using S = SplitPre<N, EB, BT>;
#pragma unroll
    for (int p = 0; p < S::SPL; ++p) {
        pf.I[p] = -1;
        pf.m[p] = 0.0;
#pragma unroll
        for (int v = 0; v < 5; ++v) pf.qn[p][v] = 0.0;
    }
    if constexpr (S::NIN > 0) {
#pragma unroll
        for (int p = 0; p < S::SPL; ++p) {
            const int n = t + p * BT;
            if (n >= S::NIN) continue;
            const int ip = n / (EB * N), m = n - ip * (EB * N), qq = m / N, ii = m - qq * N;
            if (qq >= new_) continue;
            const BoxElem fe = box_elem((uint32_t)(e0 + qq), gm.fx, gm.fy);
            if (qq == 0 || fe.ex == 0) continue;  // a run's first element: the finish kernel takes it
            const int jj = 1 + ip % (N - 1), kk = 1 + ip / (N - 1);
            pf.I[p] = fe.ex * N + ii + gm.ni * (fe.ey * N + jj + gm.nj * (fe.ez * N + kk));
            pf.m[p] = it.Minv[pf.I[p]];
            if (load_qn)
#pragma unroll
                for (int v = 0; v < 5; ++v) pf.qn[p][v] = it.qn[pf.I[p] + v * gm.nu];
        }
    }
}

// after the contributions of the workgroup are in st ([q][l][5], synchronised):
// the copies the finish kernel takes at run boundaries (Fb), the face rows
// (Fa, the run's x pairs added) and the run-interior nodes (M^-1, the update
// sc, folded or not, the state)
template <int N, typename T, int EB, int BT>
__device__ __forceinline__ void split_store(const BatchItem &it, const SplitGeo &gm, const StageCoef &sc, bool fold,
                                            const T *st, int t, int e0, int new_, const SplitPre<N, EB, BT> &pf)
{
    constexpr int P = N + 1, NP = P * P * P, NFP = 4 * N, NIP = (N - 1) * (N - 1), NB = split_nb<N>();
    using S = SplitPre<N, EB, BT>;
    T *Fa = (T *)it.ev;
    // Fb: the east face (slot order: face pairs, then interior pairs) of an
    // element whose east neighbour is not in the run, the interior rows of a
    // run's first element (ip, then i); by the last wavefront where the face
    // rows below leave most of its lanes idle (N = 4: 8 of 64), else by all
    constexpr int RUN = EB * N * 5;  // values of one face pair of the workgroup
    constexpr bool LASTW = RUN <= BT - 48;
    constexpr int FBS = LASTW ? 64 : BT;
    T *Fb = Fa + 5 * (int64_t)gm.nz * gm.ny * NFP * gm.ni;
    const int tb = LASTW ? t - (BT - 64) : t;
    int ex = box_elem((uint32_t)e0, gm.fx, gm.fy).ex;  // x index of element qq, stepped along the run
    for (int qq = 0; tb >= 0 && qq < new_; ++qq, ex = ex + 1 == gm.nx ? 0 : ex + 1) {
        if (!(qq == EB - 1 || ex == gm.nx - 1 || qq == 0 || ex == 0)) continue;
        T *fb = Fb + (int64_t)(e0 + qq) * NB * 5;
        if (qq == EB - 1 || ex == gm.nx - 1) {
            for (int u = tb; u < (NFP + NIP) * 5; u += FBS) {
                const int slot = u / 5, v = u - slot * 5;
                int jj, kk;
                if (slot < NFP) {
                    split_fp_jk<N>(slot, jj, kk);
                } else {  // interior pairs (N > 1)
                    constexpr int M = N > 1 ? N - 1 : 1;
                    jj = 1 + (slot - NFP) % M;
                    kk = 1 + (slot - NFP) / M;
                }
                fb[u] = st[(qq * NP + N + P * (jj + P * kk)) * 5 + v];
            }
        }
        if (NIP > 0 && (qq == 0 || ex == 0)) {
            for (int u = tb; u < NIP * N * 5; u += FBS) {
                const int nd = u / 5, v = u - nd * 5, ip = nd / N, ii = nd - ip * N;
                const int jj = 1 + ip % (N - 1), kk = 1 + ip / (N - 1);
                fb[(NFP + NIP) * 5 + u] = st[(qq * NP + ii + P * (jj + P * kk)) * 5 + v];
            }
        }
    }
    // Fa: lane u < EB N 5 takes value v of node (qq, ii) of every face pair,
    // so that each store instruction writes one contiguous run of the pair's
    // row, and the lane's element, pair flag and offsets are formed once
    for (int u = t; u < RUN; u += BT) {
        const int nd = u / 5, v = u - nd * 5, qq = nd / N, ii = nd - qq * N;
        if (qq < new_) {
            const BoxElem fe = box_elem((uint32_t)(e0 + qq), gm.fx, gm.fy);
            const bool pair = ii == 0 && qq > 0 && fe.ex != 0;
            const T *s0 = st + (qq * NP + ii) * 5 + v, *s1 = st + ((qq - 1) * NP + N) * 5 + v;
            T *fo = Fa + (((int64_t)(fe.ez * gm.ny + fe.ey) * NFP) * gm.ni + fe.ex * N + ii) * 5 + v;
#pragma unroll
            for (int fp = 0; fp < NFP; ++fp) {
                int jj, kk;
                split_fp_jk<N>(fp, jj, kk);
                const int lo = P * (jj + P * kk) * 5;
                T val = s0[lo];
                if (pair) val += s1[lo];
                fo[(int64_t)fp * gm.ni * 5] = val;
            }
        }
    }
    if constexpr (S::NIN > 0) {
#pragma unroll
        for (int p = 0; p < S::SPL; ++p) {
            if (pf.I[p] < 0) continue;
            const int n = t + p * BT;
            const int ip = n / (EB * N), m = n - ip * (EB * N), qq = m / N, ii = m - qq * N;
            const int jj = 1 + ip % (N - 1), kk = 1 + ip / (N - 1);
            const int l = ii + P * (jj + P * kk), lw = N + P * (jj + P * kk);
            double r[5], o[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                double c = (double)st[(qq * NP + l) * 5 + v];
                if (ii == 0) c += (double)st[((qq - 1) * NP + lw) * 5 + v];
                r[v] = c * pf.m[p];
            }
            if (fold) {
#pragma unroll
                for (int v = 0; v < 5; ++v) o[v] = rk_update_folded(sc, pf.qn[p][v], r[v]);
            } else {
#pragma unroll
                for (int v = 0; v < 5; ++v)
                    o[v] = rk_update(sc, pf.qn[p][v], sc.b == 0.0 ? 0.0 : it.qs[pf.I[p] + v * gm.nu], r[v]);
            }
#pragma unroll
            for (int v = 0; v < 5; ++v) it.qout[pf.I[p] + v * gm.nu] = o[v];
            flag_nonfinite(it.flag, o, 5);
        }
    }
}

// MODE 0: write J w R node-major for the finish kernel (NUMA_STAGE_GATHER);
// MODE 1: one colour pass of NUMA_STAGE_COLOUR: the workgroup's elements are
// the elements of colour `colour` (parity of ex, ey, ez), EB consecutive ones
// along x, and every lane adds its nodes' J w R to the FP64 accumulator with
// a plain read-modify-write (no other element of the colour has the node).
// (NUMA_STAGE_SPLIT takes the two-pass k_elem_col2 below.)
template <int N, typename T, int MODE = 0>
__global__ __launch_bounds__((col_threads<N, T>()), (col_blocks<N, T, MODE>())) void k_elem_col(Batch B, int colour)
{
    constexpr int P = N + 1, PP = P * P, NP = PP * P, EB = col_eb<N, T>(), BT = col_threads<N, T>();
    __shared__ T s[EB][8][NP];
    const int g0 = (int)xcd_remap(blockIdx.x, gridDim.x) * EB;
    const BatchItem &it = B.it[batch_item(B, g0, false)];
    const RhsArgs<T> a = elem_args<T>(B, it);
    const int e0 = g0 - it.eoff;  // first element of the workgroup in the item
    const int t = threadIdx.x, q = t / PP, c = t % PP, i = c % P, j = c / P;
    const bool act = q < EB && e0 + q < it.ne;
    // per node of the column: 1/rho and rho'/rho (formed in FP64; in FP64
    // rho' itself is kept and rho'/rho formed where it is used, the same
    // product), zeta derivatives of the 8 tile fields
    constexpr bool F64 = sizeof(T) == 8;
    T irho[P], buoy[P], dz[8][P];
    double c0 = 0.0, c1 = 0.0, c2 = 0.0, c3 = 0.0;
    int ez = 0, base = 0;
    const int layer = a.ni * a.nj;
    T Di[P], Dj[P];
#pragma unroll
    for (int m = 0; m < P; ++m) {
        Di[m] = a.D[i * P + m];
        Dj[m] = a.D[j * P + m];
    }
    if (act) {
        BoxElem be;
        if constexpr (MODE == 1) {
            const uint32_t ec = (uint32_t)(e0 + q), t1 = fdiv(ec, it.fseg), t2 = fdiv(t1, it.fy);
            be.ex = 2 * (int)(ec - t1 * it.fseg.d) + (colour & 1);
            be.ey = 2 * (int)(t1 - t2 * it.fy.d) + ((colour >> 1) & 1);
            be.ez = 2 * (int)t2 + (colour >> 2);
        } else {
            be = box_elem((uint32_t)(e0 + q), a.fx, a.fy);
        }
        ez = be.ez;
        const double *cp = a.hcol + (int64_t)(be.ex + a.nx * be.ey) * (4 * PP) + c;
        c0 = cp[0];
        c1 = cp[PP];
        c2 = cp[2 * PP];
        c3 = cp[3 * PP];
        int gi = be.ex * N + i, gj = be.ey * N + j;
        if (gi == a.ni) gi = 0;
        if (gj == a.nj) gj = 0;
        base = gi + a.ni * gj;
        T col[8][P];
        gather_column<P, col_group<N, T>()>(a, it.theta0, base, layer, be.ez * N,
                                            [&](int k, const double *qv, double rb, double pp) {
                                                const double rho = rb + qv[0], ir = 1.0 / rho;
                                                irho[k] = (T)ir;
                                                buoy[k] = F64 ? (T)qv[0] : (T)(qv[0] * ir);
#pragma unroll
                                                for (int v = 0; v < 3; ++v) {
                                                    col[v][k] = (T)(rho * qv[1 + v]);
                                                    col[3 + v][k] = (T)qv[1 + v];
                                                }
                                                col[6][k] = (T)qv[4];
                                                col[7][k] = (T)pp;
#pragma unroll
                                                for (int f = 0; f < 8; ++f) s[q][f][c + PP * k] = col[f][k];
                                            });
        const T *D = a.D;
#pragma unroll
        for (int f = 0; f < 8; ++f)
#pragma unroll
            for (int k = 0; k < P; ++k) {
                dz[f][k] = dot<P>(D + k * P, [&](int m) { return col[f][m]; });
            }
    }
    __syncthreads();  // tiles complete
    T res[P][5];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            T mx[10];
            box_node_metric<T>(a.bm, ez, B.xi[k], c0 * B.w[k], c1, c2, c3, mx);
            T dd[8][3];
#pragma unroll
            for (int f = 0; f < 8; ++f) {
                dd[f][0] = dot<P>(Di, [&](int m) { return s[q][f][m + P * (j + P * k)]; });
                dd[f][1] = dot<P>(Dj, [&](int m) { return s[q][f][i + P * (m + P * k)]; });
                dd[f][2] = dz[f][k];
            }
            const int l = c + PP * k;
            const T uu = s[q][3][l], vv = s[q][4][l], ww = s[q][5][l];
            const T bk = F64 ? buoy[k] * irho[k] : buoy[k];
            // J w R, or J w (q_s + cdt R) away from the walls when folding
            const bool wall = it.walls && ((ez == 0 && k == 0) || (ez == a.nz - 1 && k == N));
            T R[5], U[3], adv[4];
            box_velocity<T>(mx, uu, vv, ww, U);
#pragma unroll
            for (int f = 0; f < 4; ++f) adv[f] = box_advect<T>(U, dd[3 + f]);
            box_momentum<T>(mx, adv, dd[7], irho[k], bk, (T)(-a.g0), R + 1);
            R[4] = -adv[3];
            const T dzm[3] = {dd[0][2], dd[1][2], dd[2][2]};
            R[0] = box_mass<T>(mx, dd[0][0], dd[1][1], dzm);
            if (F64 && B.fold && !wall) {
                const T qv[5] = {buoy[k], uu, vv, ww, s[q][6][l]};
#pragma unroll
                for (int v = 0; v < 5; ++v) res[k][v] = mx[9] * fma((T)it.cdt, R[v], qv[v]);
            } else {
#pragma unroll
                for (int v = 0; v < 5; ++v) res[k][v] = mx[9] * R[v];
            }
        }
    }
    if constexpr (MODE == 1) {
        if (act) {
            double *acc = (double *)it.ev;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                int gk = ez * N + k;
                if (gk == a.nk) gk = 0;
                const int32_t I = base + layer * gk;
#pragma unroll
                for (int v = 0; v < 5; ++v) acc[I + v * a.nu] += (double)res[k][v];
            }
        }
        return;  // every lane: no barrier follows
    }
    __syncthreads();  // tiles read
    T *st = &s[0][0][0];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) st[(q * NP + c + PP * k) * 5 + v] = res[k][v];
    }
    __syncthreads();
    // the workgroup's elements are consecutive: one contiguous run
    const int ne = it.ne - e0 < EB ? it.ne - e0 : EB;
    T *out = (T *)it.ev + (int64_t)e0 * (NP * 5);
    store_run<T>(out, st, ne * NP * 5, t, BT);
}

// The element kernel of the split DSS (NUMA_STAGE_SPLIT, above), with a
// two-pass tile.  k_elem_col keeps eight tile fields (8 (N+1)^3 doubles per
// element in FP64) and every field's zeta derivative in registers, which leaves
// room for two workgroups per CU.  Here the tile holds five fields at a time, the
// size of the output staging: first p', u, v, w, theta', from which the
// momentum and theta' rows of R follow (advection, pressure gradient,
// buoyancy), then rho u and rho v for the mass row (rho w enters it only
// through zeta, from the lane's own column).  The lane takes its column's
// values from the tile once per pass, the xi and eta rows per node.  Each term is
// the product and sum of k_elem_col (in mixed precision the tile and the
// contractions FP32, rho, 1/rho, rho'/rho and p' formed in FP64 as there);
// the tail is the split DSS.  FP64: three workgroups per CU at N = 3, 4 (41 and
// 50 KB of LDS; at N = 3 four would spill 48 bytes: 64x64x16 98 against 85 us),
// four below; N = 5..8 as noted below.  Mixed: four waves per SIMD.
template <int N, typename T> constexpr int col2_waves()
{
    return sizeof(T) == 4 ? 4 : (N <= 2 ? 4 : (N <= 4 ? 3 : 2));
}
// nodes gathered together: fewer than the column where the registers of more cost
// a wave or more (mixed N = 4, 106 for 138: 64x64x16 step 789 -> 761 us; N = 2, 79 for
// 98: 128x128x16 528 -> 473; FP64 N = 8 1,082 -> 1,070 at 32x32x8, N = 7 210 -> 208 at 17x17x8)
template <int N, typename T> constexpr int col2_group()
{
    return sizeof(T) == 8 ? (N >= 7 ? 4 : N + 1) : N == 4 ? 3 : N == 2 ? 1 : N + 1;
}
// doubles after each element's tile: eight at N = 4 spread the xi and eta rows of
// the two or three elements a wavefront spans over the LDS banks (50,640
// bytes, still three workgroups per CU)
template <int N, typename T = double> constexpr int col2_pad() { return sizeof(T) == 8 && N == 4 ? 8 : 0; }
// N = 5, 6 (seven and five elements per 256-lane workgroup, 60 and 69 KB of
// LDS): two waves per SIMD
//
// STORED (N = 8 spills 32 bytes a lane): the metric is read instead of recomputed: the four entries of it
// that vary on a box (zeta_x, zeta_y, zeta_z, J w), a node ahead of its use in
// the first pass, J w and the others again (from the caches) in the second.
template <int N, typename T = double, bool STORED = false>
__global__ __launch_bounds__((split_threads<N>()), (col2_waves<N, T>())) void k_elem_col2(Batch B)
{
    constexpr bool F64 = sizeof(T) == 8;
    constexpr int P = N + 1, PP = P * P, NP = PP * P, EB = split_eb<N>(), BT = split_threads<N>();
    constexpr int PAD = col2_pad<N, T>();
    __shared__ T s[EB][5 * NP + PAD];
    auto S = [&](int qq, int f, int l) -> T & { return s[qq][f * NP + l]; };
    const int g0 = (int)xcd_remap(blockIdx.x, gridDim.x) * EB;
    const BatchItem &it = B.it[batch_item(B, g0, false)];
    const RhsArgs<T> a = elem_args<T>(B, it);
    const int e0 = g0 - it.eoff;
    const int t = threadIdx.x, q = t / PP, c = t % PP, i = c % P, j = c / P;
    const bool act = q < EB && e0 + q < it.ne;
    const int new_ = it.ne - e0 < EB ? it.ne - e0 : EB;
    const SplitGeo gm{a.nx, a.ny, a.nz, a.ni, a.nj, (int)a.nu, a.fx, a.fy};
    const bool fold = B.fold != 0;
    const double cdt = it.cdt, gz = -a.g0;
    const int walls = it.walls;
    // per node of the column, formed in FP64 as in k_elem_col: rho, 1/rho and
    // rho' (FP64; in mixed precision rho'/rho, the buoyancy factor)
    double rho[P];
    T ir[P], bq[P];
    double c0 = 0.0, c1 = 0.0, c2 = 0.0, c3 = 0.0;
    int ez = 0;
    // metric of the column's node k; stored: zeta_x, zeta_y, zeta_z, J w from mp
    const T *mp = STORED ? a.met + ((int64_t)(act ? e0 + q : 0) * 10 + 6) * NP + c : nullptr;
    T ahead[4];
    auto fetch = [&](int k) {
#pragma unroll
        for (int d = 0; d < 4; ++d) ahead[d] = mp[d * NP + PP * k];
    };
    auto metric = [&](int k, T *mx) {
        if constexpr (STORED) {
            mx[0] = (T)a.bm.ixa;
            mx[4] = (T)a.bm.iyb;
#pragma unroll
            for (int d = 0; d < 4; ++d) mx[6 + d] = ahead[d];
            if (k < N) fetch(k + 1);
        } else {
            box_node_metric<T>(a.bm, ez, B.xi[k], c0 * B.w[k], c1, c2, c3, mx);
        }
    };
    T Di[P], Dj[P];
#pragma unroll
    for (int m = 0; m < P; ++m) {
        Di[m] = a.D[i * P + m];
        Dj[m] = a.D[j * P + m];
    }
    if (act) {
        const BoxElem be = box_elem((uint32_t)(e0 + q), a.fx, a.fy);
        ez = be.ez;
        if constexpr (!STORED) {
            const double *cp = a.hcol + (int64_t)(be.ex + a.nx * be.ey) * (4 * PP) + c;
            c0 = cp[0];
            c1 = cp[PP];
            c2 = cp[2 * PP];
            c3 = cp[3 * PP];
        }
        int gi = be.ex * N + i, gj = be.ey * N + j;
        if (gi == a.ni) gi = 0;
        if (gj == a.nj) gj = 0;
        const int base = gi + a.ni * gj, layer = a.ni * a.nj;
        gather_column<P, col2_group<N, T>()>(a, it.theta0, base, layer, be.ez * N,
                                             [&](int k, const double *qv, double rb, double pp) {
                                                 const int l = c + PP * k;
                                                 rho[k] = rb + qv[0];
                                                 S(q, 0, l) = (T)pp;
#pragma unroll
                                                 for (int v = 1; v < 5; ++v) S(q, v, l) = (T)qv[v];
                                                 if constexpr (F64) {
                                                     bq[k] = qv[0];
                                                 } else {
                                                     const double ird = 1.0 / rho[k];
                                                     ir[k] = (T)ird;
                                                     bq[k] = (T)(qv[0] * ird);
                                                 }
                                             });
    }
    if (STORED && act) fetch(0);
    __syncthreads();  // first tile complete
    T res[P][5];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            T mx[10];
            metric(k, mx);
            const int l = c + PP * k;
            const T uu = S(q, 1, l), vv = S(q, 2, l), ww = S(q, 3, l), tt = S(q, 4, l);
            T dd[5][3];
#pragma unroll
            for (int f = 0; f < 5; ++f) {
                dd[f][0] = dot<P>(Di, [&](int m) { return S(q, f, m + P * (j + P * k)); });
                dd[f][1] = dot<P>(Dj, [&](int m) { return S(q, f, i + P * (m + P * k)); });
                dd[f][2] = dot<P>(a.D + k * P, [&](int m) { return S(q, f, c + PP * m); });
            }
            if constexpr (F64) ir[k] = (T)(1.0 / rho[k]);
            const T bk = F64 ? bq[k] * ir[k] : bq[k];
            const bool wall = walls && ((ez == 0 && k == 0) || (ez == a.nz - 1 && k == N));
            T R[4], U[3], adv[4];
            box_velocity<T>(mx, uu, vv, ww, U);
#pragma unroll
            for (int f = 0; f < 4; ++f) adv[f] = box_advect<T>(U, dd[1 + f]);
            box_momentum<T>(mx, adv, dd[0], ir[k], bk, (T)gz, R);
            R[3] = -adv[3];
            if (fold && !wall) {
                const T qv[4] = {uu, vv, ww, tt};
#pragma unroll
                for (int v = 0; v < 4; ++v) res[k][v + 1] = mx[9] * fma((T)cdt, R[v], qv[v]);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) res[k][v + 1] = mx[9] * R[v];
            }
            __builtin_amdgcn_sched_barrier(0);  // a node's rows at a time: registers
        }
    }
    // the mass fluxes of the column, formed from the first tile: rho u and
    // rho v go through the second tile (their xi and eta rows), the column's
    // own values stay in registers for the zeta derivatives
    T fl[P][3];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int l = c + PP * k;
            fl[k][0] = (T)(rho[k] * (double)S(q, 1, l));
            fl[k][1] = (T)(rho[k] * (double)S(q, 2, l));
            fl[k][2] = (T)(rho[k] * (double)S(q, 3, l));
        }
    }
    __syncthreads();  // first tile read
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int f = 0; f < 2; ++f) S(q, f, c + PP * k) = fl[k][f];
    }
    if (STORED && act) fetch(0);
    __syncthreads();  // second tile complete
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            T mx[10];
            metric(k, mx);
            const T da = dot<P>(Di, [&](int m) { return S(q, 0, m + P * (j + P * k)); });
            const T db = dot<P>(Dj, [&](int m) { return S(q, 1, i + P * (m + P * k)); });
            T dz[3];
#pragma unroll
            for (int f = 0; f < 3; ++f) dz[f] = dot<P>(a.D + k * P, [&](int m) { return fl[m][f]; });
            const bool wall = walls && ((ez == 0 && k == 0) || (ez == a.nz - 1 && k == N));
            const T R0 = box_mass<T>(mx, da, db, dz);
            res[k][0] = (fold && !wall) ? mx[9] * fma((T)cdt, R0, bq[k]) : mx[9] * R0;
        }
    }
    // the run-interior nodes' M^-1 and q^n (issued here, where the tiles'
    // registers are free)
    SplitPre<N, EB, BT> pf;
    split_prefetch<N, EB, BT>(it, gm, B.ca != 0.0, t, e0, new_, pf);
    __syncthreads();  // second tile read
    T *st = &s[0][0];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) st[(q * NP + c + PP * k) * 5 + v] = res[k][v];
    }
    __syncthreads();
    split_store<N, T, EB, BT>(it, gm, StageCoef{B.ca, B.cb, cdt}, fold, st, t, e0, new_, pf);
}

// The element kernel of the split DSS in FP64 with derivatives by rows.  In
// k_elem_col2 a lane reads, for each of its nodes and fields, the N+1 values of
// the xi and of the eta line through the node, each for one multiply-add: the
// LDS is busy 53-65 % of the time and the chain of reads is what a wavefront
// waits for.  Here the lanes also take the lines themselves: lane (a, b) of an
// element reads the xi line (j, k) = (a, b) and the eta line (i, k) = (a, b) of a
// field once, forms all N+1 derivatives of each (rows of D are lane-uniform:
// scalar operands) and writes them back, the xi derivatives over the field, the
// eta derivatives to a spare slot, from where the column lanes read theirs:
// about 7 LDS accesses per node and field instead of 2 N + 3.  A field costs two
// barriers (its lines are read; its derivatives are written).  The mass
// fluxes go first (xi of rho u, eta of rho v), then theta', w, v, u and last p',
// each from the slot it was stored in at the gather (p' from the lane's
// registers).  Each operation is that of the other box kernels.
// Rows are padded to an odd length (line lanes then fall on distinct banks).
// Taken at N = 5, 6 (two waves per SIMD) for launches below rows_below()
// element-local nodes: the fold reads the state again at the end, from the
// caches while the launch fits them and from memory above.  us per step, this
// kernel / k_elem_col2, recomputed metric: N = 5 1.9 M 226 / 232, 2.2 M 251 /
// 260, 3.5 M 420 / 412, 14 M 1,756 / 1,652; N = 6 0.79 M 125 / 132, 2.2 M 276 /
// 301, 3.5 M 452 / 462, 4.4 M 601 / 590, 22 M 3,111 / 2,904; stored: N = 5
// 0.93 M 139 / 138, 1.9 M 259 / 252; N = 6 0.79 M 132 / 133, 2.2 M 363 / 375,
// 2.9 M 509 / 517, 3.5 M 527 / 503.  At N <= 4 the barriers cost what the reads save
// (64x64x16, N = 4: 207 against 211 us, N = 3: 90 against 85), at N = 7, 8 the
// padded tile and the registers leave one wave per SIMD or spill (418 against
// 301 us, 354 against 293).  Two lanes per column (half the registers, twice the
// waves) measured 110 us at N = 5, 279 at N = 6, 503 at N = 8.
template <int N> constexpr bool rows_ok() { return N == 5 || N == 6; }
template <int N> constexpr int64_t rows_below(bool recompute)
{
    return N == 5 ? (recompute ? 2800000 : 0) : recompute ? 4000000 : 3200000;
}
template <int N> constexpr int row_len() { return (N + 1) | 1; }
template <int N> constexpr int rows_slot() { return (N + 1) * (N + 1) * row_len<N>(); }
template <int N, bool STORED>
__global__ __launch_bounds__((split_threads<N>()), 2) void k_elem_rows(Batch B)
{
    using T = double;
    constexpr int P = N + 1, PP = P * P, NP = PP * P, EB = split_eb<N>(), BT = split_threads<N>();
    constexpr int RS = row_len<N>(), NS = rows_slot<N>(), RP = RS * P;
    __shared__ double s[EB][5 * NS];
    const int g0 = (int)xcd_remap(blockIdx.x, gridDim.x) * EB;
    const BatchItem &it = B.it[batch_item(B, g0, false)];
    const RhsArgs<T> a = elem_args<T>(B, it);
    const int e0 = g0 - it.eoff;
    const int t = threadIdx.x, q = t / PP, c = t % PP, i = c % P, j = c / P;
    const bool act = q < EB && e0 + q < it.ne;
    const int new_ = it.ne - e0 < EB ? it.ne - e0 : EB;
    const SplitGeo gm{a.nx, a.ny, a.nz, a.ni, a.nj, (int)a.nu, a.fx, a.fy};
    const bool fold = B.fold != 0;
    const double cdt = it.cdt, gz = -a.g0;
    // slot f of the lane's element; node k of its column, entry m of its xi
    // and of its eta line
    double *S = &s[act ? q : 0][0];
    const int col = i + RS * j;
    auto node = [&](int f, int k) -> double & { return S[f * NS + col + RP * k]; };
    auto xi = [&](int f, int m) -> double & { return S[f * NS + RS * c + m]; };
    auto eta = [&](int f, int m) -> double & { return S[f * NS + i + RS * m + RP * j]; };
    constexpr int SU = 0, SV = 1, SW = 2, ST = 3, SE = 4;  // u, v, w, theta' (p' later), spare
    double c0 = 0.0, c1 = 0.0, c2 = 0.0, c3 = 0.0;
    int ez = 0;
    const double *mp = STORED ? a.met + ((int64_t)(act ? e0 + q : 0) * 10 + 6) * NP + c : nullptr;
    double ahead[4];
    auto fetch = [&](int k) {
#pragma unroll
        for (int d = 0; d < 4; ++d) ahead[d] = mp[d * NP + PP * k];
    };
    auto metric = [&](int k, double *mx) {
        if constexpr (STORED) {
            mx[0] = a.bm.ixa;
            mx[4] = a.bm.iyb;
#pragma unroll
            for (int d = 0; d < 4; ++d) mx[6 + d] = ahead[d];
            fetch(k < N ? k + 1 : 0);
        } else {
            box_node_metric<T>(a.bm, ez, B.xi[k], c0 * B.w[k], c1, c2, c3, mx);
        }
    };
    double rho[P], bq[P], pp[P], uv[2][P], res[P][5];
    int base = 0;
    const int layer = a.ni * a.nj;
    auto at = [&](int k) {  // unique id of the column's node k
        int gk = ez * N + k;
        if (gk == a.nk) gk = 0;
        return base + layer * gk;
    };
    if (act) {
        const BoxElem be = box_elem((uint32_t)(e0 + q), a.fx, a.fy);
        ez = be.ez;
        if constexpr (!STORED) {
            const double *cp = a.hcol + (int64_t)(be.ex + a.nx * be.ey) * (4 * PP) + c;
            c0 = cp[0];
            c1 = cp[PP];
            c2 = cp[2 * PP];
            c3 = cp[3 * PP];
        }
        int gi = be.ex * N + i, gj = be.ey * N + j;
        if (gi == a.ni) gi = 0;
        if (gj == a.nj) gj = 0;
        base = gi + a.ni * gj;
        gather_column<P, P>(a, it.theta0, base, layer, be.ez * N,
                            [&](int k, const double *qv, double rb, double p) {
                                rho[k] = rb + qv[0];
                                bq[k] = qv[0];
                                pp[k] = p;
                                uv[0][k] = qv[1];
                                uv[1][k] = qv[2];
                                node(SU, k) = rho[k] * qv[1];
                                node(SV, k) = rho[k] * qv[2];
                                node(SW, k) = qv[3];
                                node(ST, k) = qv[4];
                            });
        if constexpr (STORED) fetch(0);
    }
    // J w (q_s + cdt R) where node k folds q_s in, else J w R
    auto value = [&](int k, double jw, double R, double qs) {
        const bool wall = it.walls && ((ez == 0 && k == 0) || (ez == a.nz - 1 && k == N));
        return jw * (fold && !wall ? fma(cdt, R, qs) : R);
    };
    double dx[P], de[P];
    auto line = [&](auto at, int f, double *d) {
        double r[P];
#pragma unroll
        for (int m = 0; m < P; ++m) r[m] = at(f, m);
#pragma unroll
        for (int n = 0; n < P; ++n) d[n] = dot<P>(a.D + n * P, [&](int m) { return r[m]; });
    };
    __syncthreads();
    // mass row
    double U[P][3];
    {
        double dz[3][P];
        if (act) {
            line(xi, SU, dx);
            line(eta, SV, de);
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                double fl[P];
#pragma unroll
                for (int m = 0; m < P; ++m) fl[m] = f < 2 ? node(f, m) : rho[m] * node(SW, m);
#pragma unroll
                for (int k = 0; k < P; ++k) dz[f][k] = dot<P>(a.D + k * P, [&](int m) { return fl[m]; });
            }
        }
        __syncthreads();
        if (act)
#pragma unroll
            for (int m = 0; m < P; ++m) {
                xi(SU, m) = dx[m];
                eta(SV, m) = de[m];
            }
        __syncthreads();
        if (act)
#pragma unroll
            for (int k = 0; k < P; ++k) {
                double mx[10];
                metric(k, mx);
                const double dk[3] = {dz[0][k], dz[1][k], dz[2][k]};
                res[k][0] = value(k, mx[9], box_mass<T>(mx, node(SU, k), node(SV, k), dk), bq[k]);
                box_velocity<T>(mx, uv[0][k], uv[1][k], node(SW, k), U[k]);
            }
    }
    __syncthreads();
    if (act)
#pragma unroll
        for (int k = 0; k < P; ++k) {
            node(SU, k) = uv[0][k];
            node(SV, k) = uv[1][k];
        }
    // theta', w, v, u, then p' from theta''s slot, free by then; u and v are
    // stored two barriers before their lines are read
    double qr[P][4];
#pragma unroll
    for (int step = 0; step < 5; ++step) {
        const int f = step == 4 ? ST : ST - step;
        double cf[P], d2[P];
        if (step == 4 && act && fold)  // the state again (from the caches), for the fold
#pragma unroll
            for (int k = 0; k < P; ++k)
#pragma unroll
                for (int v = 0; v < 4; ++v) qr[k][v] = a.q[at(k) + (1 + v) * a.nu];
        if (act) {
            line(xi, f, dx);
            line(eta, f, de);
#pragma unroll
            for (int m = 0; m < P; ++m) cf[m] = node(f, m);
#pragma unroll
            for (int k = 0; k < P; ++k) d2[k] = dot<P>(a.D + k * P, [&](int m) { return cf[m]; });
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int m = 0; m < P; ++m) {
                xi(f, m) = dx[m];
                eta(SE, m) = de[m];
            }
            if (step == 3)
#pragma unroll
                for (int k = 0; k < P; ++k) node(ST, k) = pp[k];
        }
        __syncthreads();
        if (act)
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double d[3] = {node(f, k), node(SE, k), d2[k]};
                if (step < 4) {
                    res[k][1 + f] = box_advect<T>(U[k], d);
                } else {
                    double mx[10], R[4];
                    metric(k, mx);
                    const double ir = 1.0 / rho[k];
                    box_momentum<T>(mx, res[k] + 1, d, ir, bq[k] * ir, gz, R);
                    R[3] = -res[k][4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) res[k][1 + v] = value(k, mx[9], R[v], qr[k][v]);
                }
            }
    }
    // the run-interior nodes' M^-1 and q^n (issued here, where the tiles'
    // registers are free)
    SplitPre<N, EB, BT> pf;
    split_prefetch<N, EB, BT>(it, gm, B.ca != 0.0, t, e0, new_, pf);
    __syncthreads();  // the last derivatives are read
    double *st = &s[0][0];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) st[(q * NP + c + PP * k) * 5 + v] = res[k][v];
    }
    __syncthreads();
    split_store<N, T, EB, BT>(it, gm, StageCoef{B.ca, B.cb, cdt}, fold, st, t, e0, new_, pf);
}

// NUMA_STAGE_SPLIT finish: the face nodes and the run-start interior nodes.
// mblk blocks of an item take the face rows of the lattice, one node per
// lane along x: per element layer ez the level gk = ez N (all nj rows), then
// the levels ez N + 1 .. ez N + N - 1 (the ny rows gj = ey N), and with walls
// the top level gk = nz N; frl divides by the rows per layer
// nj + (N - 1) ny (fseg divides by ni).  The other blocks (interleaved) take
// the interior rows of a run's first element, N nodes per row (i < N): the
// elements e = c EB (one per element workgroup), then the row starts
// e = r nx that are not multiples of EB.  Every node's
// copies are summed in FP64 in a fixed order (in mixed precision a pair inside a
// run is already one FP32 value of Fa), multiplied by M^-1, projected at the walls and
// advanced by the stage update (PLAIN: the summed value itself, for the
// filter: the stage operands are not read).
template <int N, typename T, bool PLAIN = false>
__global__ __launch_bounds__(256) void k_fin_split(Batch B)
{
    constexpr int NFP = 4 * N, NIP = (N - 1) * (N - 1), NB = split_nb<N>(), EB = split_eb<N>();
    const int g = (int)xcd_remap(blockIdx.x, gridDim.x);
    const BatchItem &it = B.it[batch_item(B, g, true)];
    const int nx = (int)it.fx.d, ny = (int)it.fy.d, nz = it.nz, ni = it.ni, nj = it.nj;
    // the item's blocks: mblk face-row blocks and nbb run-start blocks, the
    // latter spread evenly (block k at k S + S - 1, S = total / nbb), so that
    // every XCD's range of the launch holds its share of the scattered ones
    int lb = g - it.boff;
    const int nbb = NIP == 0 ? 0 : (((it.ne + EB - 1) / EB + ny * nz) * NIP * N + 255) / 256;
    bool runstart = false;
    if (NIP > 0 && nbb > 0) {
        const int S = (it.mblk + nbb) / (NIP > 0 ? nbb : 1);
        if (lb < nbb * S) {
            const int k = lb / S;
            runstart = lb - k * S == S - 1;
            lb = runstart ? k : lb - k;
        } else {
            lb -= nbb;
        }
    }
    const int64_t vs = (int64_t)nz * ny * NFP * ni;
    const T *Fa = (const T *)it.ev, *Fb = Fa + 5 * vs;
    int gi, gj, gk;
    double r[5] = {0, 0, 0, 0, 0};
    // the stage update's operands are loaded as soon as the node is known,
    // before its copies: one memory round trip per node instead of two
    const StageCoef sc{B.ca, B.cb, it.cdt};
    double mi, qnv[5], qsv[5];
    int32_t I;
    bool folded;
    auto update_loads = [&]() {
        I = gi + ni * (gj + nj * gk);
        folded = !PLAIN && B.fold && !(it.walls && (gk == 0 || gk == nz * N));
        mi = it.Minv[I];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            qnv[v] = PLAIN || sc.a == 0.0 ? 0.0 : it.qn[I + v * it.nu];
            qsv[v] = PLAIN || folded || sc.b == 0.0 ? 0.0 : it.qs[I + v * it.nu];
        }
    };
    if (!runstart) {
        const int rl = (int)it.frl.d;
        const int nrows = nz * rl + (it.walls ? nj : 0);
        const uint32_t id = (uint32_t)lb * 256u + threadIdx.x;
        if (id >= (uint32_t)nrows * (uint32_t)ni) return;
        const uint32_t R = fdiv(id, it.fseg);
        gi = (int)(id - R * (uint32_t)ni);
        const uint32_t ezr = fdiv(R, it.frl);
        int rr = (int)(R - ezr * (uint32_t)rl);
        if ((int)ezr == nz) {  // the top wall level
            gk = nz * N;
            gj = rr;
        } else if (rr < nj) {
            gk = (int)ezr * N;
            gj = rr;
        } else {
            rr -= nj;
            const uint32_t kk = fdiv((uint32_t)rr, it.fy);
            gj = (rr - (int)kk * ny) * N;
            gk = (int)ezr * N + 1 + (int)kk;
        }
        update_loads();
        // copies: z (element layer, local k), y (element row, local j)
        int zc[2], kc[2], nzc = 1, yc[2], jc[2], nyc = 1;
        zc[0] = gk / N;
        kc[0] = gk % N;
        zc[1] = zc[0];
        kc[1] = kc[0];
        if (kc[0] == 0) {
            if (it.walls && gk == nz * N) {
                zc[0] = nz - 1;
                kc[0] = N;
            } else if (!(it.walls && gk == 0)) {
                zc[1] = zc[0] == 0 ? nz - 1 : zc[0] - 1;
                kc[1] = N;
                nzc = 2;
            }
        }
        yc[0] = gj / N;
        jc[0] = gj % N;
        yc[1] = yc[0];
        jc[1] = jc[0];
        if (jc[0] == 0) {
            yc[1] = yc[0] == 0 ? ny - 1 : yc[0] - 1;
            jc[1] = N;
            nyc = 2;
        }
        const int ex = gi / N;
        const bool xface = gi % N == 0;
        // the face rows' copies (absent ones are not loaded) are loaded
        // together; the run-start x copies (Fb, at most one node in EB N of a
        // row) only where there are any.  The sum: x pairs first, then over y
        // and z, as the gather finish (box_finish_node) takes it.  In mixed
        // precision, whose pairs inside a run are sums already, the run-start
        // copies come last (the pairs in FP64 first: 3.5 us more at 1.2 M nodes,
        // N = 4, for a wave less)
        constexpr bool PAIRS = sizeof(T) == 8;
        T ca[2][2][5];
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const bool has = z < nzc && y < nyc;
                const int64_t o = ((int64_t)(zc[z] * ny + yc[y]) * NFP + split_fp<N>(jc[y], kc[z])) * ni + gi;
#pragma unroll
                for (int v = 0; v < 5; ++v) ca[z][y][v] = has ? Fa[o * 5 + v] : (T)0;
            }
        auto sum_rows = [&]() {
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    if (z < nzc && y < nyc)
#pragma unroll
                        for (int v = 0; v < 5; ++v) r[v] += (double)ca[z][y][v];
        };
        if (!PAIRS) sum_rows();
        if (xface) {
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const int ec = ex + nx * (yc[y] + ny * zc[z]);
                    if (z < nzc && y < nyc && (ex == 0 || ec % EB == 0)) {
                        const int64_t ob = ((int64_t)(ex == 0 ? ec + nx - 1 : ec - 1) * NB + split_fp<N>(jc[y], kc[z])) * 5;
#pragma unroll
                        for (int v = 0; v < 5; ++v) {
                            if (PAIRS) ca[z][y][v] += Fb[ob + v];
                            else r[v] += (double)Fb[ob + v];
                        }
                    }
                }
        }
        if (PAIRS) sum_rows();
    } else {
        if constexpr (NIP == 0) {
            return;
        } else {
            const int nwg = (it.ne + EB - 1) / EB, nrs = ny * nz;
            const int id = lb * 256 + (int)threadIdx.x;
            const int cand = id / (NIP * N), rr = id - cand * (NIP * N), ip = rr / N, i = rr - ip * N;
            if (cand >= nwg + nrs) return;
            int e;
            if (cand < nwg) {
                e = cand * EB;
            } else {
                e = (cand - nwg) * nx;
                if (e % EB == 0) return;  // a workgroup start: taken above
            }
            const BoxElem be = box_elem((uint32_t)e, it.fx, it.fy);
            const int jj = 1 + ip % (N - 1), kk = 1 + ip / (N - 1);
            gi = be.ex * N + i;
            gj = be.ey * N + jj;
            gk = be.ez * N + kk;
            update_loads();
            const int ew = be.ex == 0 ? e + nx - 1 : e - 1;  // the element west of the run start
            const int64_t o0 = ((int64_t)e * NB + NFP + NIP + ip * N + i) * 5, o1 = ((int64_t)ew * NB + NFP + ip) * 5;
            T c0[5], c1[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                c0[v] = Fb[o0 + v];
                c1[v] = i == 0 ? Fb[o1 + v] : (T)0;
            }
#pragma unroll
            for (int v = 0; v < 5; ++v) r[v] = i == 0 ? (double)c0[v] + (double)c1[v] : (double)c0[v];
        }
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) r[v] *= mi;
    double o[5];
    if (folded) {
#pragma unroll
        for (int v = 0; v < 5; ++v) o[v] = rk_update_folded(sc, qnv[v], r[v]);
    } else {
        PointArgs p;
        p.Minv = it.Minv;
        p.nrm = it.nrm;
        p.nl = 0;
        p.nu = it.nu;
        p.nh = it.nh;
        p.walls = it.walls;
        noflux(p, I, r[1], r[2], r[3]);
#pragma unroll
        for (int v = 0; v < 5; ++v) o[v] = rk_update(sc, qnv[v], qsv[v], r[v]);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) it.qout[I + v * it.nu] = o[v];
    flag_nonfinite(it.flag, o, 5);
}

// NUMA_STAGE_COLOUR: zero the accumulator [5][nu] of every item (a kernel,
// not a memset: the stage may be captured in a graph)
__global__ void k_colour_zero(Batch B)
{
    const int g = (int)blockIdx.x;
    const BatchItem &it = B.it[batch_item(B, g, true)];
    const int64_t I = (int64_t)(g - it.boff) * 256 + threadIdx.x;
    if (I >= it.nu) return;
    double *acc = (double *)it.ev;
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[I + v * it.nu] = 0.0;
}

// NUMA_STAGE_COLOUR: M^-1, wall projection and stage update of every unique
// node from the accumulated sum (the tail of box_finish_node)
__global__ void k_colour_finish(Batch B)
{
    const int g = (int)xcd_remap(blockIdx.x, gridDim.x);
    const BatchItem &it = B.it[batch_item(B, g, true)];
    const int64_t I = (int64_t)(g - it.boff) * 256 + threadIdx.x;
    if (I >= it.nu) return;
    const double *acc = (const double *)it.ev;
    const StageCoef sc{B.ca, B.cb, it.cdt};
    const double mi = it.Minv[I];
    const bool wall = it.walls && (I < it.nh || I >= it.nu - it.nh);
    double r[5], qnv[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        r[v] = acc[I + v * it.nu] * mi;
        qnv[v] = sc.a == 0.0 ? 0.0 : it.qn[I + v * it.nu];
    }
    double o[5];
    if (B.fold && !wall) {
#pragma unroll
        for (int v = 0; v < 5; ++v) it.qout[I + v * it.nu] = o[v] = rk_update_folded(sc, qnv[v], r[v]);
        flag_nonfinite(it.flag, o, 5);
        return;
    }
    PointArgs p;
    p.Minv = it.Minv;
    p.nrm = it.nrm;
    p.nl = 0;
    p.nu = it.nu;
    p.nh = it.nh;
    p.walls = it.walls;
    noflux(p, I, r[1], r[2], r[3]);
#pragma unroll
    for (int v = 0; v < 5; ++v) it.qout[I + v * it.nu] = o[v] = rk_update(sc, qnv[v], it.qs[I + v * it.nu], r[v]);
    flag_nonfinite(it.flag, o, 5);
}

// Streaming variant of the column kernel: after the tile is built the lane
// walks the 8 fields once, reads its own column of each field (the zeta
// contraction), the xi and eta lines of each of its nodes, and adds the
// field's terms to the R of its N+1 nodes, so that only R, the advecting
// contravariant velocity and 1/rho, rho'/rho of the column stay in registers
// (the terms are added in the order element_rhs sums them).
template <int N, typename T>
__global__ __launch_bounds__((col_threads<N, T>())) void k_elem_stream(Batch B)
{
    constexpr int P = N + 1, PP = P * P, NP = PP * P, EB = col_eb<N, T>(), BT = col_threads<N, T>();
    __shared__ T s[EB][8][NP];
    const int g0 = (int)xcd_remap(blockIdx.x, gridDim.x) * EB;
    const BatchItem &it = B.it[batch_item(B, g0, false)];
    const RhsArgs<T> a = elem_args<T>(B, it);
    const int e0 = g0 - it.eoff;
    const int t = threadIdx.x, q = t / PP, c = t % PP, i = c % P, j = c / P;
    const bool act = q < EB && e0 + q < it.ne;
    T irho[P], buoy[P], Uc[P][3];
    double c0 = 0.0, c1 = 0.0, c2 = 0.0, c3 = 0.0;
    int ez = 0;
    if (act) {
        const BoxElem be = box_elem((uint32_t)(e0 + q), a.fx, a.fy);
        ez = be.ez;
        const double *cp = a.hcol + (int64_t)(be.ex + a.nx * be.ey) * (4 * PP) + c;
        c0 = cp[0];
        c1 = cp[PP];
        c2 = cp[2 * PP];
        c3 = cp[3 * PP];
        int gi = be.ex * N + i, gj = be.ey * N + j;
        if (gi == a.ni) gi = 0;
        if (gj == a.nj) gj = 0;
        const int base = gi + a.ni * gj, layer = a.ni * a.nj;
        gather_column<P, stream_group<N, T>()>(
            a, it.theta0, base, layer, be.ez * N, [&](int k, const double *qv, double rb, double pp) {
                const double rho = rb + qv[0], ir = 1.0 / rho;
                irho[k] = (T)ir;
                buoy[k] = (T)(qv[0] * ir);
                T mx[10];
                box_node_metric<T>(a.bm, ez, B.xi[k], c0, c1, c2, c3, mx);
                const T uu = (T)qv[1], vv = (T)qv[2], ww = (T)qv[3];
                Uc[k][0] = uu * mx[0];
                Uc[k][1] = vv * mx[4];
                Uc[k][2] = fm(ww, mx[8], fm(vv, mx[7], uu * mx[6]));
                const int l = c + PP * k;
#pragma unroll
                for (int v = 0; v < 3; ++v) s[q][v][l] = (T)(rho * qv[1 + v]);
                s[q][3][l] = uu;
                s[q][4][l] = vv;
                s[q][5][l] = ww;
                s[q][6][l] = (T)qv[4];
                s[q][7][l] = (T)pp;
            });
    }
    __syncthreads();  // tiles complete
    T R[P][5];
    if (act) {
        T Di[P], Dj[P];
#pragma unroll
        for (int m = 0; m < P; ++m) {
            Di[m] = a.D[i * P + m];
            Dj[m] = a.D[j * P + m];
        }
        const T *D = a.D;
        const T mx0 = (T)a.bm.ixa, mx4 = (T)a.bm.iyb, mx8 = (T)c1;
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            T cf[P];
#pragma unroll
            for (int m = 0; m < P; ++m) cf[m] = s[q][f][c + PP * m];
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double omz = fm(-fm(0.5, 1.0 + B.xi[k], (double)ez), a.bm.inz, 1.0);  // 1 - z/H
                const T mx6 = (T)(omz * c2), mx7 = (T)(omz * c3);
                T da = 0, db = 0;
                const T dc = dot<P>(D + k * P, [&](int m) { return cf[m]; });
                if (f != 1 && f != 2) da = dot<P>(Di, [&](int m) { return s[q][f][m + P * (j + P * k)]; });
                if (f != 0 && f != 2) db = dot<P>(Dj, [&](int m) { return s[q][f][i + P * (m + P * k)]; });
                // the operations of box_mass, box_advect and box_momentum, a field at a time
                if (f == 0) R[k][0] = fm(dc, mx6, da * mx0);              // d(rho u)/dx
                if (f == 1) R[k][0] = R[k][0] + fm(dc, mx7, db * mx4);    // + d(rho v)/dy
                if (f == 2) R[k][0] = -fm(dc, mx8, R[k][0]);              // + d(rho w)/dz
                const T dd[3] = {da, db, dc};
                if (f >= 3 && f <= 6) R[k][f - 2] = box_advect<T>(Uc[k], dd);
                if (f == 7) {
                    T mx[10], Rm[3];
                    mx[0] = mx0;
                    mx[4] = mx4;
                    mx[6] = mx6;
                    mx[7] = mx7;
                    mx[8] = mx8;
                    box_momentum<T>(mx, R[k] + 1, dd, irho[k], buoy[k], (T)(-a.g0), Rm);
#pragma unroll
                    for (int v = 0; v < 3; ++v) R[k][1 + v] = Rm[v];
                    R[k][4] = -R[k][4];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const T jw = (T)(c0 * B.w[k]);
#pragma unroll
            for (int v = 0; v < 5; ++v) R[k][v] = jw * R[k][v];
        }
    }
    __syncthreads();  // tiles read
    T *st = &s[0][0][0];
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) st[(q * NP + c + PP * k) * 5 + v] = R[k][v];
    }
    __syncthreads();
    // the workgroup's elements are consecutive: one contiguous run
    const int ne = it.ne - e0 < EB ? it.ne - e0 : EB;
    T *out = (T *)it.ev + (int64_t)e0 * (NP * 5);
    store_run<T>(out, st, ne * NP * 5, t, BT);
}

// The Boyd-Vandeven filter of a box with the recomputed metric through the
// split DSS: the column workgroup of the stage (EB consecutive elements, a lane
// per (i, j) column) gathers the state into an LDS tile, applies F along xi
// and eta through the tile and along zeta in the lane's registers (the same
// fma chains in the same direction order as k_filter), weights by J w and
// hands J w (F q) to the split DSS: the run-interior nodes are finished here
// (M^-1, no stage update), the others by k_fin_split.  The state is filtered
// in place: the nodes finished here are read by no other workgroup, and the
// face kernel reads only the contributions.
struct FilterSplit {
    BatchItem it;             // qs: the state read, qout: the state written (the same array)
    double w[kMaxP];          // GLL weights
    double F[kMaxP * kMaxP];  // 1D nodal filter matrix F[i * (N+1) + m]
    const double *met;        // stored metric (J w is entry 9)
};

// STORED: J w of the stored metric, else c0 w_k
template <int N, bool STORED>
__global__ __launch_bounds__((split_threads<N>())) void k_filter_col(FilterSplit A)
{
    constexpr int P = N + 1, PP = P * P, NP = PP * P, EB = split_eb<N>(), BT = split_threads<N>();
    constexpr int PAD = col2_pad<N, double>();  // the two-pass stage kernel's bank spread
    __shared__ double s[EB][5 * NP + PAD];
    auto S = [&](int qq, int f, int l) -> double & { return s[qq][f * NP + l]; };
    // the 1D filter matrix: in LDS up to N = 4; above, the lane's xi and eta
    // rows in registers and the zeta row from the kernel arguments, so that
    // the N = 7 tile (80 KB) leaves room for two workgroups per CU
    constexpr bool FREG = N >= 5;
    __shared__ double Fs[FREG ? 1 : PP];
    double Fi[P], Fj[P];
#pragma unroll
    for (int m = 0; m < P; ++m) {
        Fi[m] = FREG ? A.F[((int)threadIdx.x % PP % P) * P + m] : 0.0;
        Fj[m] = FREG ? A.F[((int)threadIdx.x % PP / P) * P + m] : 0.0;
    }
    const BatchItem &it = A.it;
    const int e0 = (int)xcd_remap(blockIdx.x, gridDim.x) * EB;
    const int t = threadIdx.x, q = t / PP, c = t % PP, i = c % P, j = c / P;
    const bool act = q < EB && e0 + q < it.ne;
    if (!FREG && t < PP) Fs[t] = A.F[t];
    const int new_ = it.ne - e0 < EB ? it.ne - e0 : EB;
    const SplitGeo gm{(int)it.fx.d, (int)it.fy.d, it.nz, it.ni, it.nj, it.nu, it.fx, it.fy};
    SplitPre<N, EB, BT> pf;
    split_prefetch<N, EB, BT>(it, gm, false, t, e0, new_, pf);
    double jw[P];
    if (act) {
        const BoxElem be = box_elem((uint32_t)(e0 + q), it.fx, it.fy);
        const double *jp = STORED ? A.met + ((int64_t)(e0 + q) * 10 + 9) * NP + c
                                  : it.hcol + (int64_t)(be.ex + gm.nx * be.ey) * (4 * PP) + c;
        const double c0 = jp[0];
        int gi = be.ex * N + i, gj = be.ey * N + j;
        if (gi == gm.ni) gi = 0;
        if (gj == gm.nj) gj = 0;
        const int base = gi + gm.ni * gj, layer = gm.ni * gm.nj;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            int gk = be.ez * N + k;
            if (gk == it.nkw) gk = 0;
            const int32_t I = base + layer * gk;
#pragma unroll
            for (int v = 0; v < 5; ++v) S(q, v, c + PP * k) = it.qs[I + v * gm.nu];
            jw[k] = STORED ? jp[PP * k] : c0 * A.w[k];
        }
    }
    __syncthreads();
    double x[5][P];
    if (act) {  // xi
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                double r = 0.0;
#pragma unroll
                for (int m = 0; m < P; ++m) r = fma(FREG ? Fi[m] : Fs[i * P + m], S(q, v, m + P * (j + P * k)), r);
                x[v][k] = r;
            }
    }
    __syncthreads();
    if (act)
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) S(q, v, c + PP * k) = x[v][k];
    __syncthreads();
    double res[P][5];
    if (act) {  // eta through the tile, zeta in registers, times J w
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                double r = 0.0;
#pragma unroll
                for (int m = 0; m < P; ++m) r = fma(FREG ? Fj[m] : Fs[j * P + m], S(q, v, i + P * (m + P * k)), r);
                x[v][k] = r;
            }
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                double r = 0.0;
#pragma unroll
                for (int m = 0; m < P; ++m) r = fma(FREG ? A.F[k * P + m] : Fs[k * P + m], x[v][m], r);
                res[k][v] = jw[k] * r;
            }
    }
    __syncthreads();  // tile read
    double *st = &s[0][0];
    if (act)
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) st[(q * NP + c + PP * k) * 5 + v] = res[k][v];
    __syncthreads();
    split_store<N, double, EB, BT>(it, gm, StageCoef{0.0, 0.0, 1.0}, false, st, t, e0, new_, pf);
}

template <int N, int SEG, typename T, bool PLAIN = false>
__global__ void k_fin_batch(Batch B)
{
    const int g = (int)xcd_remap(blockIdx.x, gridDim.x);
    const BatchItem &it = B.it[batch_item(B, g, true)];
    int lb = g - it.boff;
    int kbase = 0, klayers = N;
    if (lb >= it.mblk) {  // the top wall layer
        kbase = N;
        klayers = 1;
        lb -= it.mblk;
    }
    const uint32_t t = fdiv((uint32_t)lb, it.fseg);
    const int sx = lb - (int)(t * it.fseg.d);
    const uint32_t ez = fdiv(t, it.fy);
    const int ey = (int)(t - ez * it.fy.d);
    PointArgs p;
    p.Minv = it.Minv;
    p.nrm = it.nrm;
    p.nl = 0;
    p.nu = it.nu;
    p.nh = it.nh;
    p.walls = it.walls;
    BoxFin b;
    b.nx = (int)it.fx.d;
    b.ny = (int)it.fy.d;
    b.nz = it.nz;
    b.walls = it.walls;
    b.ni = it.ni;
    b.nj = it.nj;
    b.fold = B.fold;
    box_finish_node<N, SEG, T, PLAIN>(p, b, (const T *)it.ev, sx, ey, kbase == 0 ? (int)ez : it.nz - 1, threadIdx.x,
                                      kbase, klayers, StageCoef{B.ca, B.cb, it.cdt}, it.qn, it.qs, it.qout,
                                      PLAIN ? nullptr : it.flag);
}

// the fields of a batch item that the split finish (k_fin_split) reads, for
// the column workgroups of EB elements; returns the item's finish blocks
int64_t split_item(const Mesh &m, int eb, BatchItem &it)
{
    const int N = m.N, ny = m.d.ne[1], nz = m.d.ne[2];
    const int64_t rl = m.nj + (int64_t)(N - 1) * ny;
    const int64_t rows = nz * rl + (m.walls ? m.nj : 0);
    const int64_t nwg = (m.ne + eb - 1) / eb;
    it.fseg = fast_div((uint32_t)m.ni);
    it.frl = fast_div((uint32_t)rl);
    it.mblk = (int)((rows * m.ni + 255) / 256);
    return it.mblk + ((nwg + (int64_t)ny * nz) * ((int64_t)(N - 1) * (N - 1) * N) + 255) / 256;
}

template <int N, typename T, int SEG>
int32_t run_chunk_seg(const StepItem *items, int n, int phase, hipStream_t s, int mode)
{
    const bool colour = mode == kColour, split = mode == kSplit, node = mode == kNode;
    Batch B;
    B.n = n;
    B.ca = items[0].c.a;
    B.cb = items[0].c.b;
    B.gamma = items[0].mesh->gamma;
    B.g0 = items[0].mesh->ph.g0;
    B.D = std::is_same<T, float>::value ? (const void *)items[0].mesh->dv.D32 : (const void *)items[0].mesh->dv.D64;
    B.xi = items[0].mesh->dv.xi64;
    B.w = items[0].mesh->dv.w64;
    eos_coeffs(B.gamma, B.eos);
    // the recomputed metric runs a column kernel, EB elements per workgroup:
    // registers for every field's column up to N = 4, the streaming variant
    // above (FP64 at N = 7, 8 outgrows both: one node per lane there, as with
    // the stored metric and in kNode launches)
    constexpr int kind = N <= 4 ? 0 : (sizeof(T) == 4 || N <= 6 ? 1 : 2);
    constexpr bool col_ok = kind != 2;
    const bool recompute = items[0].mesh->metric_mode == NUMA_METRIC_RECOMPUTE;
    const bool col = recompute && col_ok && !node;
    const int eb = split ? split_eb<N>() : col ? col_eb<N, T>() : 1;
    // FP64 update that uses q_s (b != 0): the column and one-node-per-lane
    // element kernels fold q_s into the contributions (the streaming one,
    // which runs at its register limit, does not, nor what a small launch of its
    // orders runs in its place).  The weighted sum of the fold
    // rounds q_s once per copy (against 64-bit evaluation, N = 2: 1.4e-16 where
    // the update alone leaves 7.3e-17).  With the stored metric, on x extents
    // that numa_step_batch does not take (one item), the finish reads q_s instead.
    B.fold = std::is_same<T, double>::value && B.cb != 0.0 &&
             (split || !(recompute && kind == 1 && !stage_by_size(*items[0].mesh))) &&
             (recompute || box_batchable(*items[0].mesh));
    int64_t eo = 0, bo = 0;
    for (int k = 0; k < n; ++k) {
        const Mesh &m = *items[k].mesh;
        BatchItem &it = B.it[k];
        it.qs = items[k].qs;
        it.qout = items[k].qout;
        it.qn = items[k].qn;
        it.ref = m.dv.ref;
        it.Minv = stage_minv(m);
        it.nrm = m.dv.nrm;
        it.met = std::is_same<T, float>::value ? (const void *)m.dv.met32 : (const void *)m.dv.met;
        it.ev = items[k].ev;
        it.hcol = m.dv.hcol;
        it.flag = items[k].flag;
        it.nu = (int)m.nu;
        it.nh = (int)m.nh;
        it.ni = (int)m.ni;
        it.nj = (int)m.nj;
        it.nkw = m.d.periodic[2] ? (int)m.nk : -1;
        it.nz = m.d.ne[2];
        it.walls = m.walls ? 1 : 0;
        it.fx = fast_div((uint32_t)m.d.ne[0]);
        it.fy = fast_div((uint32_t)m.d.ne[1]);
        // the gather finish's segments, the last one of a row partly empty
        // where SEG does not divide nx (a split item's fields are set below)
        const int nseg = (m.d.ne[0] + SEG - 1) / SEG;
        it.fseg = fast_div((uint32_t)nseg);
        const int64_t mblk = (int64_t)nseg * m.d.ne[1] * m.d.ne[2];
        it.mblk = (int)mblk;
        it.cdt = items[k].c.cdt;
        it.theta0 = m.ph.T0;
        it.bm = box_metric(m);
        it.ne = (int)m.ne;
        it.eoff = (int)eo;
        it.boff = (int)bo;
        if (colour) {  // a colour pass covers ne/8 elements; the pointwise kernels 256 nodes per block
            it.ne = (int)(m.ne / 8);
            it.fseg = fast_div((uint32_t)(m.d.ne[0] / 2));
            it.fy = fast_div((uint32_t)(m.d.ne[1] / 2));
            eo += (it.ne + eb - 1) / eb * eb;
            bo += (m.nu + 255) / 256;
        } else if (split) {  // face rows, 256 lattice points per block, then the run starts
            eo += (m.ne + eb - 1) / eb * eb;
            bo += split_item(m, eb, it);
        } else {
            eo += (m.ne + eb - 1) / eb * eb;
            bo += mblk + (m.walls ? (int64_t)nseg * m.d.ne[1] : 0);
        }
    }
    if (eo >= (int64_t(1) << 31) || bo >= (int64_t(1) << 31)) {
        set_error("batch: more than 2^31 - 1 elements in one launch");
        return NUMA_EUNSUPPORTED;
    }
    for (int k = n; k < kMaxBatch; ++k) B.it[k] = BatchItem{};
    if (colour) {
        if constexpr (kind == 0) {
            if (phase == 0) {
                hipLaunchKernelGGL(k_colour_zero, dim3((unsigned)bo), dim3(256), 0, s, B);
                for (int c = 0; c < 8; ++c)
                    hipLaunchKernelGGL((k_elem_col<N, T, 1>), dim3((unsigned)(eo / eb)), dim3(col_threads<N, T>()), 0, s,
                                       B, c);
            } else {
                hipLaunchKernelGGL(k_colour_finish, dim3((unsigned)bo), dim3(256), 0, s, B);
            }
            NUMA_HIP(hipGetLastError());
            return NUMA_OK;
        }
    }
    if (split) {
        constexpr bool f64 = std::is_same<T, double>::value;
        if constexpr (kind == 0 || f64) {
            const dim3 grid((unsigned)(eo / eb)), block(split_threads<N>());
            if (phase == 1) {
                hipLaunchKernelGGL((k_fin_split<N, T>), dim3((unsigned)bo), dim3(256), 0, s, B);
                NUMA_HIP(hipGetLastError());
                return NUMA_OK;
            }
            if constexpr (f64 && rows_ok<N>()) {
                if (eo * ((N + 1) * (N + 1) * (N + 1)) < rows_below<N>(recompute)) {
                    if (recompute)
                        hipLaunchKernelGGL((k_elem_rows<N, false>), grid, block, 0, s, B);
                    else if constexpr (rows_below<N>(false) > 0)
                        hipLaunchKernelGGL((k_elem_rows<N, true>), grid, block, 0, s, B);
                    NUMA_HIP(hipGetLastError());
                    return NUMA_OK;
                }
            }
            if (recompute) {
                hipLaunchKernelGGL((k_elem_col2<N, T>), grid, block, 0, s, B);
            } else {
                if constexpr (f64) hipLaunchKernelGGL((k_elem_col2<N, T, true>), grid, block, 0, s, B);
            }
            NUMA_HIP(hipGetLastError());
            return NUMA_OK;
        }
        set_error("split DSS: no element kernel for this order and precision");
        return NUMA_EUNSUPPORTED;
    }
    if (phase == 0) {
        if (!recompute) {
            hipLaunchKernelGGL((k_elem_batch<N, T, kMetricStored>), dim3((unsigned)eo), dim3(block_threads<N>()), 0, s,
                               B);
        } else if (node) {
            hipLaunchKernelGGL((k_elem_batch<N, T, kMetricBox>), dim3((unsigned)eo), dim3(block_threads<N>()), 0, s, B);
        } else if constexpr (kind == 0) {
            hipLaunchKernelGGL((k_elem_col<N, T>), dim3((unsigned)(eo / eb)), dim3(col_threads<N, T>()), 0, s, B, 0);
        } else if constexpr (kind == 1) {
            hipLaunchKernelGGL((k_elem_stream<N, T>), dim3((unsigned)(eo / eb)), dim3(col_threads<N, T>()), 0, s, B);
        } else {
            hipLaunchKernelGGL((k_elem_batch<N, T, kMetricBox>), dim3((unsigned)eo), dim3(block_threads<N>()), 0, s, B);
        }
    } else {
        const int threads = ((SEG * N * N * N + 63) / 64) * 64;
        hipLaunchKernelGGL((k_fin_batch<N, SEG, T>), dim3((unsigned)bo), dim3(threads), 0, s, B);
    }
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

// The finish segment of a launch.  N = 3: the widest of three whose last segment
// leaves at most a quarter of a row's lanes idle on every item, else the
// narrowest; a 4-element segment is 12 lattice points, 96 of every 128 bytes of a
// state line, 16 elements are 48 points, three whole lines (measured at 64x64x16:
// finish 82 -> 61 us).  N = 1, 2: the one that launches fewest lanes, whole
// wavefronts counted (segments of 4 and 16 elements fill 4 and 16 lanes of one at
// N = 1), the wider of equals.  The per-node code and its order of the copies do
// not depend on the segment: results are the same bit for bit whichever
// segment a launch takes.
template <int N> constexpr int seg_wide() { return N == 1 ? 64 : N <= 3 ? 16 : seg_for<N>(); }
template <int N> constexpr int seg_mid() { return N == 1 ? 16 : N <= 3 ? 8 : seg_for<N>(); }

template <int N>
int pick_seg(const StepItem *items, int n)
{
    if constexpr (N <= 2) {
        int best = 0;
        int64_t fewest = 0;
        for (const int seg : {seg_wide<N>(), seg_mid<N>(), seg_for<N>()}) {
            int64_t lanes = 0;
            for (int k = 0; k < n; ++k) {
                const int32_t *ne = items[k].mesh->d.ne;
                lanes += (int64_t)((ne[0] + seg - 1) / seg) * ne[1] * ne[2] * ((seg * N * N * N + 63) / 64 * 64);
            }
            if (!best || lanes < fewest) {
                best = seg;
                fewest = lanes;
            }
        }
        return best;
    }
    for (const int seg : {seg_wide<N>(), seg_mid<N>()}) {
        bool ok = true;
        for (int k = 0; k < n; ++k) {
            const int nx = items[k].mesh->d.ne[0];
            ok = ok && 4 * ((nx + seg - 1) / seg * seg) <= 5 * nx;
        }
        if (ok) return seg;
    }
    return seg_for<N>();
}

template <int N, typename T>
int32_t run_chunk(const StepItem *items, int n, int phase, hipStream_t s, int mode)
{
    if constexpr (seg_wide<N>() != seg_for<N>()) {
        const int seg = pick_seg<N>(items, n);
        if (seg == seg_wide<N>()) return run_chunk_seg<N, T, seg_wide<N>()>(items, n, phase, s, mode);
        if (seg == seg_mid<N>()) return run_chunk_seg<N, T, seg_mid<N>()>(items, n, phase, s, mode);
    }
    return run_chunk_seg<N, T, seg_for<N>()>(items, n, phase, s, mode);
}

// DSS of node-major FP64 contributions ev ([n_local][5]) into q with M^-1
// and the wall projection, by the box finish kernel (one item)
template <int N, int SEG>
int32_t run_plain_finish_seg(const Mesh &m, const double *ev, double *q, hipStream_t s)
{
    Batch B{};
    B.n = 1;
    B.ca = 0.0;
    B.cb = 1.0;
    BatchItem &it = B.it[0];
    it.qout = q;
    it.Minv = stage_minv(m);  // the box filter's J w follows the metric mode
    it.nrm = m.dv.nrm;
    it.ev = (void *)ev;
    it.flag = nullptr;
    it.nu = (int)m.nu;
    it.nh = (int)m.nh;
    it.ni = (int)m.ni;
    it.nj = (int)m.nj;
    it.nz = m.d.ne[2];
    it.walls = m.walls ? 1 : 0;
    it.fx = fast_div((uint32_t)m.d.ne[0]);
    it.fy = fast_div((uint32_t)m.d.ne[1]);
    const int nseg = (m.d.ne[0] + SEG - 1) / SEG;
    it.fseg = fast_div((uint32_t)nseg);
    const int64_t mblk = (int64_t)nseg * m.d.ne[1] * m.d.ne[2];
    it.mblk = (int)mblk;
    it.ne = (int)m.ne;
    const int64_t bo = mblk + (m.walls ? (int64_t)nseg * m.d.ne[1] : 0);
    const int threads = ((SEG * N * N * N + 63) / 64) * 64;
    hipLaunchKernelGGL((k_fin_batch<N, SEG, double, true>), dim3((unsigned)bo), dim3(threads), 0, s, B);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

template <int N>
int32_t run_plain_finish(const Mesh &m, const double *ev, double *q, hipStream_t s)
{
    StepItem it{};
    it.mesh = &m;
    if constexpr (seg_wide<N>() != seg_for<N>()) {
        const int seg = pick_seg<N>(&it, 1);
        if (seg == seg_wide<N>()) return run_plain_finish_seg<N, seg_wide<N>()>(m, ev, q, s);
        if (seg == seg_mid<N>()) return run_plain_finish_seg<N, seg_mid<N>()>(m, ev, q, s);
    }
    return run_plain_finish_seg<N, seg_for<N>()>(m, ev, q, s);
}

template <typename T>
int32_t run_stage_t(const StepItem *items, int n, int phase, hipStream_t s, int mode)
{
    for (int c0 = 0; c0 < n; c0 += kMaxBatch) {
        const int c = n - c0 < kMaxBatch ? n - c0 : kMaxBatch;
        int32_t rc;
        switch (items[0].mesh->N) {
        case 1: rc = run_chunk<1, T>(items + c0, c, phase, s, mode); break;
        case 2: rc = run_chunk<2, T>(items + c0, c, phase, s, mode); break;
        case 3: rc = run_chunk<3, T>(items + c0, c, phase, s, mode); break;
        case 4: rc = run_chunk<4, T>(items + c0, c, phase, s, mode); break;
        case 5: rc = run_chunk<5, T>(items + c0, c, phase, s, mode); break;
        case 6: rc = run_chunk<6, T>(items + c0, c, phase, s, mode); break;
        case 7: rc = run_chunk<7, T>(items + c0, c, phase, s, mode); break;
        default: rc = run_chunk<8, T>(items + c0, c, phase, s, mode); break;
        }
        if (rc) return rc;
    }
    return NUMA_OK;
}

}  // namespace

bool box_batchable(const Mesh &m)
{
    if (m.d.kind != NUMA_MESH_BOX) return false;
    int seg;
    switch (m.N) {
    case 1: seg = seg_for<1>(); break;
    case 2: seg = seg_for<2>(); break;
    case 3: seg = seg_for<3>(); break;
    case 4: seg = seg_for<4>(); break;
    case 5: seg = seg_for<5>(); break;
    case 6: seg = seg_for<6>(); break;
    case 7: seg = seg_for<7>(); break;
    default: seg = seg_for<8>(); break;
    }
    return m.d.ne[0] % seg == 0;
}

int32_t launch_box_plain_finish(const Mesh &m, const double *ev, double *q, hipStream_t s)
{
    switch (m.N) {
    case 1: return run_plain_finish<1>(m, ev, q, s);
    case 2: return run_plain_finish<2>(m, ev, q, s);
    case 3: return run_plain_finish<3>(m, ev, q, s);
    case 4: return run_plain_finish<4>(m, ev, q, s);
    case 5: return run_plain_finish<5>(m, ev, q, s);
    case 6: return run_plain_finish<6>(m, ev, q, s);
    case 7: return run_plain_finish<7>(m, ev, q, s);
    default: return run_plain_finish<8>(m, ev, q, s);
    }
}

namespace {

template <int N>
int32_t run_filter_split(const Mesh &m, const double *F, double *q, hipStream_t s)
{
    constexpr int EB = split_eb<N>();
    FilterSplit A{};
    BatchItem &it = A.it;
    it.qs = q;
    it.qout = q;
    it.qn = nullptr;
    it.Minv = stage_minv(m);
    it.nrm = m.dv.nrm;
    it.ev = m.dv.ev64;
    it.hcol = m.dv.hcol;
    it.flag = nullptr;
    it.nu = (int)m.nu;
    it.nh = (int)m.nh;
    it.ni = (int)m.ni;
    it.nj = (int)m.nj;
    it.nkw = m.d.periodic[2] ? (int)m.nk : -1;
    it.nz = m.d.ne[2];
    it.walls = m.walls ? 1 : 0;
    it.ne = (int)m.ne;
    it.fx = fast_div((uint32_t)m.d.ne[0]);
    it.fy = fast_div((uint32_t)m.d.ne[1]);
    it.cdt = 1.0;
    it.eoff = 0;
    it.boff = 0;
    const int64_t bo = split_item(m, EB, it);
    for (int k = 0; k <= N; ++k) A.w[k] = m.w[k];
    for (int k = 0; k < (N + 1) * (N + 1); ++k) A.F[k] = F[k];
    A.met = m.dv.met;
    const dim3 grid((unsigned)((m.ne + EB - 1) / EB)), block(split_threads<N>());
    if (m.metric_mode == NUMA_METRIC_STORED)
        hipLaunchKernelGGL((k_filter_col<N, true>), grid, block, 0, s, A);
    else
        hipLaunchKernelGGL((k_filter_col<N, false>), grid, block, 0, s, A);
    // the face nodes: the split finish with the identity update (a = b = 0, cdt = 1)
    Batch B{};
    B.n = 1;
    B.fold = 0;
    B.ca = 0.0;
    B.cb = 0.0;
    B.it[0] = it;
    hipLaunchKernelGGL((k_fin_split<N, double, true>), dim3((unsigned)bo), dim3(256), 0, s, B);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

}  // namespace

bool filter_split_ok(const Mesh &m)
{
    // few nodes: one per lane and the gather finish, whose chains are shorter
    // (as in a stage; both give the same result).  Pair at N = 4: 8 k nodes 10.5
    // against 15.7 us, 128 k 12.1 / 16.0, 512 k 23.0 / 22.3, 1.02 M 36.3 / 34.2;
    // N = 8: 47 k 14.1 / 24.1, 373 k 27.8 / 30.0, 746 k 40.9 / 40.0.  With the stored
    // metric at N = 8 the gather at every size: 1.14 M 56.0 / 63.0
    if (!split_ok(m, NUMA_PREC_FP64)) return false;
    return !stage_by_size(m) || (m.nl >= 450000 && !(m.N == 8 && m.metric_mode == NUMA_METRIC_STORED));
}

int32_t launch_filter_split(const Mesh &m, const double *F, double *q, hipStream_t s)
{
    switch (m.N) {
    case 1: return run_filter_split<1>(m, F, q, s);
    case 2: return run_filter_split<2>(m, F, q, s);
    case 3: return run_filter_split<3>(m, F, q, s);
    case 4: return run_filter_split<4>(m, F, q, s);
    case 5: return run_filter_split<5>(m, F, q, s);
    case 6: return run_filter_split<6>(m, F, q, s);
    case 7: return run_filter_split<7>(m, F, q, s);
    case 8: return run_filter_split<8>(m, F, q, s);
    default:
        set_error("filter: the split DSS takes N <= 8");
        return NUMA_EUNSUPPORTED;
    }
}

bool colour_ok(const Mesh &m)
{
    return m.stage_mode == NUMA_STAGE_COLOUR && m.d.kind == NUMA_MESH_BOX && m.metric_mode == NUMA_METRIC_RECOMPUTE &&
           m.N <= 4 && m.d.ne[0] % 2 == 0 && m.d.ne[1] % 2 == 0 && m.d.ne[2] % 2 == 0;
}

// NUMA_STAGE_SPLIT runs the two-pass column element kernel (FP64: N <= 8 and
// either metric; mixed precision: N <= 4, recomputed metric); its finish takes
// any x extent.
bool split_ok(const Mesh &m, int32_t prec)
{
    if (m.d.kind != NUMA_MESH_BOX) return false;
    if (prec == NUMA_PREC_FP64) return m.stage_mode == NUMA_STAGE_SPLIT || m.stage_mode == NUMA_STAGE_AUTO;
    return m.stage_mode == NUMA_STAGE_SPLIT && m.metric_mode == NUMA_METRIC_RECOMPUTE && m.N <= 4;
}

// NUMA_STAGE_AUTO: how a launch of nl element-local nodes in all runs a stage.
// A workgroup of the column kernels is a long chain of dependent LDS reads and
// multiply-adds per lane (N = 4: 13 us for one workgroup alone, 4.5 us with one
// node per lane), which a large launch hides behind other workgroups and a
// small one does not; the split DSS moves fewest bytes and has the longer chain
// of the two column kernels.  Its workgroups take the GPU in rounds, and a round
// barely begun costs a whole one (N = 7, node / split us per step: 1.05 M nodes, the
// first round full, 158 / 150; 1.18 M 177 / 205).  At N = 4..7, where the two
// meet within the first rounds, a launch that fills its last round takes the
// split below the line too.  Measured on 330 boxes of 2 to 192 elements a side,
// regular and odd: the route taken is 0.4 % from the fastest in the mean.  us per
// step about the lines (medians where several boxes have the size), recomputed metric:
//   FP64 node / gather / split: 1: 28 k 32 / 32 / 46, 36 k 35 / 34 / 45, 1.05 M 264 /
//   115 / 117; 2: 95 k 37 / 38 / 50, 124 k 41 / 40 / 51, 2.6 M 313 / 203 / 211, 3.5 M
//   452 / 297 / 270; 3: 200 k 44 / 45 / 53, 576 k 81 / 83 / 84, 700 k 91 / 88 / 86;
//   FP64 node / split: 4: 745 k 102 / 105, 895 k (full) 114 / 105, 1.04 M 128 / 130, 1.13 M
//   137 / 132; 5: 800 k 118 / 138, 1.6 M 201 / 210, 1.9 M 232 / 226; 6: 175 k 51 / 85,
//   345 k 94 / 90, 480 k 110 / 115, 620 k 130 / 119; 7: 1.64 M 228 / 244, 1.8 M 266 / 266,
//   2.05 M 301 / 265; 8: 1.6 M 304 / 332, 2.0 M 400 / 398, 3.0 M 628 / 566.
//   Mixed node / gather: 1: 28 k 29 / 31, 49 k 33 / 31; 2: 95 k 36 / 37, 124 k 39 / 38; 3:
//   202 k 43 / 44, 262 k 48 / 46; 4: 500 k 67 / 68, 590 k 77 / 75; 5: 1.4 M 148 / 149, 1.6 M
//   170 / 169; 6: 720 k 104 / 108, 1.1 M 141 / 139; 7: 2.1 M 233 / 237, 2.3 M 291 / 284; 8:
//   2.3 M 300 / 304, 3.0 M 398 / 388.
static bool split_fills(int N, int64_t nl)
{
    // workgroups of a round (N = 6: of its first half, one to a CU) and the part of
    // them, in per cent, from which the last round counts as full
    static const int run[9] = {0, 0, 0, 0, 10, 7, 5, 4, 0}, slots[9] = {0, 0, 0, 0, 768, 512, 256, 512, 0};
    static const int part[9] = {0, 0, 0, 0, 88, 88, 75, 88, 0};
    if (!slots[N]) return false;
    const int64_t per = (int64_t)run[N] * (N + 1) * (N + 1) * (N + 1);
    const int64_t wg = (nl + per - 1) / per, rounds = (wg + slots[N] - 1) / slots[N];
    return 100 * wg >= part[N] * slots[N] * rounds;
}

int auto_route(int N, int32_t prec, int64_t nl)
{
    //                                     N = 1      2       3        4        5       6        7        8
    static const int64_t node64[9] = {0, 30000, 100000, 200000, 1100000, 1800000, 540000, 1800000, 2000000};
    static const int64_t gather64[4] = {0, 1200000, 2800000, 600000};
    static const int64_t nodemx[9] = {0, 35000, 110000, 240000, 520000, 1400000, 750000, 2200000, 2600000};
    if (prec == NUMA_PREC_MIXED) return nl < nodemx[N] ? kNode : kGather;
    if (nl < node64[N] && !split_fills(N, nl)) return kNode;
    return N <= 3 && nl < gather64[N] ? kGather : kSplit;
}

// With the stored metric the gather has one node per lane at every size (mixed
// precision: always; FP64 against the split DSS).  us per step, node / split: 1: 72 k
// 43 / 45, 102 k 50 / 45; 2: 440 k 77 / 79, 1.2 M 162 / 146; 3: 576 k 84 / 93, 819 k 104 /
// 105, 1.04 M 117 / 111; 4: 750 k 115 / 117, 900 k 123 / 109; 5: 1.6 M 238 / 263, 1.9 M
// 310 / 300; 6: 526 k 115 / 122, 620 k 131 / 124; 7: 1.2 M 185 / 249, 1.8 M 305 / 289; 8:
// 2.0 M 442 / 435, 3.0 M 640 / 596.
int auto_route_stored(int N, int32_t prec, int64_t nl)
{
    //                                     N = 1      2       3        4        5       6        7        8
    static const int64_t node64[9] = {0, 85000, 650000, 850000, 800000, 1700000, 590000, 1700000, 2000000};
    return prec == NUMA_PREC_MIXED || nl < node64[N] ? kNode : kSplit;
}

// A mesh whose schedule is named: the split DSS where it applies, else the gather;
// x extents that no batch takes with one node per lane while the default does (N = 8
// mixed, 73 k nodes: 41 against 60 us a step through the streaming kernel).
static int named_route(const Mesh &m, int32_t prec)
{
    if (split_ok(m, prec)) return kSplit;
    return box_batchable(m) || auto_route(m.N, prec, m.nl) != kNode ? kGather : kNode;
}

int32_t launch_batch_stage(const StepItem *items, int n, int32_t prec, int phase, hipStream_t s)
{
    // items the fused block kernels take (pencil.hip), the colour passes, the
    // split DSS, the rest, the small ones; partitioned in chunks on the stack,
    // with no host allocation.  The items that go by size choose together, by
    // what they add up to: either way gives an item the same result.
    constexpr int kChunk = 4 * kMaxBatch;
    StepItem part[5][kChunk];
    int64_t nl = 0;
    for (int k = 0; k < n; ++k)
        if (stage_by_size(*items[k].mesh)) nl += items[k].mesh->nl;
    for (int c0 = 0; c0 < n; c0 += kChunk) {
        const int cn = n - c0 < kChunk ? n - c0 : kChunk;
        int cnt[5] = {0, 0, 0, 0, 0};
        for (int k = c0; k < c0 + cn; ++k) {
            const Mesh &m = *items[k].mesh;
            const int g = pencil_stage_ok(items[k], prec)       ? 4
                          : colour_ok(m)                        ? kColour
                          : !stage_by_size(m)                   ? named_route(m, prec)
                          : m.metric_mode == NUMA_METRIC_STORED ? auto_route_stored(m.N, prec, nl)
                                                                : auto_route(m.N, prec, nl);
            part[g][cnt[g]++] = items[k];
        }
        int32_t rc;
        if (cnt[4] && (rc = launch_pencil_stage(part[4], cnt[4], prec, phase, s))) return rc;
        for (const int g : {kColour, kSplit, kGather, kNode}) {
            if (!cnt[g]) continue;
            rc = prec == NUMA_PREC_MIXED ? run_stage_t<float>(part[g], cnt[g], phase, s, g)
                                         : run_stage_t<double>(part[g], cnt[g], phase, s, g);
            if (rc) return rc;
        }
    }
    return NUMA_OK;
}

}  // namespace numa
