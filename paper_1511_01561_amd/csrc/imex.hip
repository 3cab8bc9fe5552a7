// 1D-IMEX vertical correction (Sec. "Time Discretization": implicit
// corrections along the vertical columns after an explicit leap-frog step;
// Code example 1: "compute IMEX corrections for each vertical column").
//
// After the explicit leap-frog step q* = q^{n-1} + 2 dt L(q^n) (a fused stage
// with the update a q_ref + cdt R), the linearised vertical terms V are taken
// as the trapezoidal mean of the new and the old level:
//   (I - dt V) q^{n+1} = q* - dt V(2 q^n - q^{n-1}),
// then the Robert-Asselin filter q^n <- q^n + ra (q^{n-1} - 2 q^n + q^{n+1}).
// With n the unit vertical (z on the box, radial on the shell), w = u.n and
// s = 1 (box) or r^2 (shell), V linearised about the hydrostatic reference is
//   V_rho' = -(1/s) G(s rho_bar w),
//   V_w    = -(1/rho_bar) G(c2 rho' + kap theta') + g_n rho'/rho_bar   (along n),
//   V_theta' = -beta w,  beta = G(theta_bar),
// with c2 = gamma p_bar / rho_bar, kap = c2 rho_bar / theta_bar, g_n = g.n, and
// zero momentum rows at the walls.  d/dn acts along zeta only in both maps, and
// the DSS of an element-local zeta derivative reduces on a vertical lattice
// line to the 1D operator
//   (G f)_g = sum_{e ∋ g} w_k(g) (D f_e)_k(g) / sum_{e ∋ g} h_e(g) w_k(g),
// h_e = dn/dzeta of element e at the node (z_zeta, or the shell's radial
// h_zeta): the horizontal copies of a node contribute identical terms, and
// on the shell r^2 cancels between J w and the mass.  So each line is an
// independent system in (rho', w, theta'); eliminating
// rho' = r_rho - (dt/s) G(s rho_bar w) and theta' = r_theta - dt beta w leaves
//   A w = r_w - dt (1/rho_bar) G(c2 r_rho + kap r_theta) + dt (g_n/rho_bar) r_rho,
//   A = I - dt^2 (1/rho_bar) G c2 s^-1 G s rho_bar - dt^2 (1/rho_bar) G kap beta
//         + dt^2 (g_n / rho_bar) s^-1 G s rho_bar
// (wall rows: w = r_w), a band matrix of half-width 2N that depends on dt and
// the reference state only.  It is factored once per dt (LU without pivoting:
// I plus dt^2 times a vertical acoustic operator) into the workspace; every
// step then solves each line bottom to top and back; neighbouring lanes hold
// neighbouring lattice lines (coalesced).  The
// new velocity is the explicit one with its n component replaced.
#include "kernels.h"

#include <type_traits>

namespace numa {
namespace {

struct ImexArgs {
    const double *qs;      // q*: the explicit leap-frog step, [5][n_unique]
    double *qcur, *qprev;  // in: q^n, q^{n-1}; out: q^{n+1}, the filtered q^n
    const double *ref;     // [3][n_unique]: rho_bar, theta_bar, p_bar
    const double *hcol;    // box column factors, 1/z_zeta in factor 1
    const double *slay;    // shell layer factors [nz (N+1)][4]: 1/r, 1/h_zeta, ., g0 (a/r)^2
    const double *xu;      // [3][n_unique] coordinates (the shell's radial direction)
    double *lu;            // [n_levels][4N+1][n_lines]: L below, 1/U_gg on, U above the diagonal
    double *sr, *sx, *st, *sb;  // [n_levels][n_lines] line vectors: r_rho; r_w, y, w; r_theta; beta
    int64_t nu, nh;        // unique nodes, lines (horizontal unique nodes)
    int ni, nk, nx, shell; // box: lattice extent along x, elements along x; levels
    double dt, ra, gamma, gz, theta0;
    double D[kMaxP * kMaxP], w[kMaxP];
};

// Per-line geometry: the box's z_zeta is the same for the whole line; the
// shell's radial factors come per (layer, local k).
struct LineGeo {
    double izz;     // box: 1/z_zeta
    double n[3];    // unit vertical
};

template <int N>
__device__ __forceinline__ LineGeo line_geo(const ImexArgs &a, int64_t L)
{
    constexpr int P = N + 1, PP = P * P;
    LineGeo lg;
    if (a.shell) {
        const double x = a.xu[L], y = a.xu[a.nu + L], z = a.xu[2 * a.nu + L];
        const double ir = 1.0 / sqrt(x * x + y * y + z * z);
        lg.n[0] = x * ir;
        lg.n[1] = y * ir;
        lg.n[2] = z * ir;
        lg.izz = 0.0;
    } else {
        const int gi = (int)(L % a.ni), gj = (int)(L / a.ni);
        const int ex = gi / N, ey = gj / N;
        lg.izz = a.hcol[(int64_t)(ex + a.nx * ey) * (4 * PP) + PP + (gi - ex * N) + P * (gj - ey * N)];
        lg.n[0] = 0.0;
        lg.n[1] = 0.0;
        lg.n[2] = 1.0;
    }
    return lg;
}

// dn/dzeta of element e at its local node k
template <int N>
__device__ __forceinline__ double h_of(const ImexArgs &a, const LineGeo &lg, int e, int k)
{
    return a.shell ? 1.0 / a.slay[4 * (e * (N + 1) + k) + 1] : 1.0 / lg.izz;
}

// s (r^2 on the shell) and g.n at level g of the line
template <int N>
__device__ __forceinline__ void level_factors(const ImexArgs &a, int g, double &s, double &gn)
{
    if (a.shell) {
        int e = g / N, k = g - e * N;
        if (e >= (a.nk - 1) / N) {  // the top node: element below, local N
            e -= 1;
            k = N;
        }
        const double ir = a.slay[4 * (e * (N + 1) + k)];
        s = 1.0 / (ir * ir);
        gn = -a.slay[4 * (e * (N + 1) + k) + 3];
    } else {
        s = 1.0;
        gn = a.gz;
    }
}

// G on a line of nk = nz N + 1 levels: (G)_{g m} = g_num / g_den.  Level g
// takes element g / N and, on an element boundary, the one below.  D and w in
// LDS (a lane's own indices: from the kernel arguments each would be a global
// load).
template <int N, typename F>
__device__ __forceinline__ void g_elements(int nk, int g, F f)
{
    const int eg = g / N, kg = g - eg * N;
    if (g != nk - 1) f(eg, kg);  // the top wall node: element below only
    if (kg == 0 && eg != 0) f(eg - 1, N);
}

template <int N>
__device__ __forceinline__ double g_den(const ImexArgs &a, const LineGeo &lg, const double *w, int g)
{
    double den = 0.0;
    g_elements<N>(a.nk, g, [&](int e, int k) { den += h_of<N>(a, lg, e, k) * w[k]; });
    return den;
}

template <int N>
__device__ __forceinline__ double g_num(const double *D, const double *w, int nk, int g, int m)
{
    constexpr int P = N + 1;
    double num = 0.0;
    g_elements<N>(nk, g, [&](int e, int k) {
        const int km = m - e * N;
        if (km >= 0 && km <= N) num += w[k] * D[k * P + km];
    });
    return num;
}

// The factors of A for every line: one 64-lane workgroup per line builds the
// band of G and of A in LDS, factors it and writes the band out.  Bound by the
// chain of LDS round trips and FP64 divisions of a line (the elimination's are
// 118 us of 325 at 32x32x16, N = 4; 145 MB of factors take 30).  The quotients
// that depend on the level alone are formed once per level instead of in the
// entries' inner loop, D and w come from LDS, and an entry's sum over the
// levels between is unrolled: 433 -> 325 us.
template <int N>
__global__ __launch_bounds__(64) void k_imex_factor(ImexArgs a)
{
    constexpr int B = 2 * N, W = 2 * B + 1, GW = 2 * N + 1;
    constexpr int P = N + 1;
    extern __shared__ double sm[];
    const int nk = a.nk, lane = threadIdx.x;
    double *Ab = sm;               // [nk][W]: A_{g m} at g W + m - g + B
    double *Gb = Ab + nk * W;      // [nk][GW]: G_{g m} at g GW + m - g + N
    // per level: rho_bar, c2 then c2 / s, s, g_n then dt^2 g_n / (rho_bar s), the
    // denominator of G then kap beta, theta_bar then dt^2 / rho_bar
    double *rb = Gb + nk * GW, *c2 = rb + nk, *sv = c2 + nk, *gn = sv + nk, *kb = gn + nk, *tb = kb + nk;
    double *D = Ab, *w = Ab + P * P;  // until A is formed: (N+1)(N+2) <= nk W values
    for (int t = lane; t < P * P; t += 64) D[t] = a.D[t];
    if (lane < P) w[lane] = a.w[lane];
    __syncthreads();
    const int64_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t nh = a.nh;
    const LineGeo lg = line_geo<N>(a, L);
    for (int g = lane; g < nk; g += 64) {
        const int64_t I = L + nh * g;
        rb[g] = a.ref[I];
        c2[g] = a.gamma * a.ref[2 * a.nu + I] / a.ref[I];
        tb[g] = a.shell ? a.ref[a.nu + I] : a.theta0;
        level_factors<N>(a, g, sv[g], gn[g]);
        kb[g] = g_den<N>(a, lg, w, g);
    }
    __syncthreads();
    for (int t = lane; t < nk * GW; t += 64) {
        const int g = t / GW, m = g + t % GW - N;
        Gb[t] = (m >= 0 && m < nk) ? g_num<N>(D, w, nk, g, m) / kb[g] : 0.0;
    }
    __syncthreads();
    // kap beta at every level, beta = G(theta_bar); theta_bar is constant on the box
    for (int g = lane; g < nk; g += 64) {
        double beta = 0.0;
        for (int d = 0; d < GW && a.shell; ++d) {
            const int m = g + d - N;
            if (m >= 0 && m < nk) beta += Gb[g * GW + d] * tb[m];
        }
        kb[g] = a.shell ? c2[g] * rb[g] / tb[g] * beta : 0.0;
    }
    __syncthreads();
    // the quotients that only depend on the level
    const double dt2 = a.dt * a.dt;
    for (int g = lane; g < nk; g += 64) {
        c2[g] = c2[g] / sv[g];
        tb[g] = dt2 / rb[g];
        gn[g] = dt2 * gn[g] / (rb[g] * sv[g]);
    }
    __syncthreads();
    for (int t = lane; t < nk * W; t += 64) {
        const int g = t / W, m = g + t % W - B;
        double v = 0.0;
        if (m >= 0 && m < nk) {
            if (g == 0 || g == nk - 1) {
                v = m == g ? 1.0 : 0.0;
            } else {
                double acc = 0.0;  // (G c2 s^-1 G)_{g m}
                const int p0 = (g > m ? g : m) - N, p1 = (g < m ? g : m) + N;
#pragma unroll
                for (int d = -N; d <= N; ++d) {  // one round of LDS reads, not one per term
                    const int p = g + d;
                    const bool in = p >= 0 && p >= p0 && p <= p1 && p < nk;
                    const int pc = in ? p : g;
                    const double term = Gb[g * GW + pc - g + N] * c2[pc] * Gb[pc * GW + (in ? m - p : 0) + N];
                    acc = in ? acc + term : acc;
                }
                const double gm = (m - g >= -N && m - g <= N) ? Gb[g * GW + m - g + N] : 0.0;
                v = (m == g ? 1.0 : 0.0) - tb[g] * acc * sv[m] * rb[m] - tb[g] * gm * kb[m] +
                    gn[g] * gm * sv[m] * rb[m];
            }
        }
        Ab[t] = v;
    }
    __syncthreads();
    // band LU without pivoting; multipliers below the diagonal
    for (int k = 0; k < nk - 1; ++k) {
        const int rmax = k + B < nk - 1 ? k + B : nk - 1;
        if (lane < B && k + 1 + lane <= rmax) {
            const int r = k + 1 + lane;
            Ab[r * W + k - r + B] /= Ab[k * W + B];
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < (B * B + 63) / 64; ++s) {
            const int t = lane + 64 * s, r = k + 1 + t / B, c = k + 1 + t % B;
            if (t < B * B && r <= rmax && c <= rmax)
                Ab[r * W + c - r + B] -= Ab[r * W + k - r + B] * Ab[k * W + c - k + B];
        }
        __syncthreads();
    }
    // out, [g][d][line]; entries outside the line are zero, the diagonal is
    // stored as its reciprocal
    for (int g = lane; g < nk; g += 64) Ab[g * W + B] = 1.0 / Ab[g * W + B];
    __syncthreads();
    for (int t = lane; t < nk * W; t += 64) a.lu[(int64_t)t * nh + L] = Ab[t];
}

// D f on one element's nodes (the zeta derivative); D from LDS (uniform
// addresses: one broadcast read per entry)
template <int N>
__device__ __forceinline__ void dloc(const double *D, const double (&f)[N + 1], double (&df)[N + 1])
{
    constexpr int P = N + 1;
    // read D where it is used: kept live across the element loop it would
    // take (N+1)^2 register pairs
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < P; ++k) {
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < P; ++m) s = fma(D[k * P + m], f[m], s);
        df[k] = s;
    }
}

// G f at local node k of element e: k = 0 above the bottom combines the
// element below through its top derivative dprev and dn/dzeta hprev (the DSS
// of the two copies)
__device__ __forceinline__ double gat(double w0, double wN, int e, int k, double dk, double hk, double dprev,
                                      double hprev)
{
    if (k == 0 && e > 0) return (wN * dprev + w0 * dk) / (wN * hprev + w0 * hk);
    return dk / hk;
}

// One step's vertical correction of the lines that k_imex_lines (below) does not
// take: one lane per line, four passes along it;
// an element's N+1 nodes at a time, node e N + N finishing with element e + 1
// (or as the top wall node).
template <int N, bool SHELL>
__global__ __launch_bounds__(256) void k_imex_solve(ImexArgs a)
{
    constexpr int P = N + 1, B = 2 * N, W = 2 * B + 1;
    __shared__ double D[P * P];
    if (threadIdx.x < P * P) D[threadIdx.x] = a.D[threadIdx.x];
    __syncthreads();
    const int64_t nh = a.nh, nu = a.nu;
    const int64_t L = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (L >= nh) return;
    const int nk = a.nk, nz = (nk - 1) / N;
    const LineGeo lg = line_geo<N>(a, L);
    // the box's vertical is z, its theta_bar constant (beta = 0)
    const double n0 = SHELL ? lg.n[0] : 0.0, n1 = SHELL ? lg.n[1] : 0.0, n2 = SHELL ? lg.n[2] : 1.0;
    const double dt = a.dt, w0 = a.w[0], wN = a.w[N];
    // pass 1: sigma = 2 q^n - q^{n-1};
    //   r_rho = q*_rho + (dt/s) G(s rho_bar sigma_w), beta = G(theta_bar),
    //   r_w = q*_w + dt (G(c2 sigma_rho + kap sigma_theta) - g_n sigma_rho)/rho_bar (q*_w at walls),
    //   r_theta = q*_theta + dt beta sigma_w
    double cf = 0.0, ch = 0.0, ct = 0.0, hp = 0.0;
    for (int e = 0; e < nz; ++e) {
        double f[P], h[P], tb[P], s0v[P], swv[P], rbv[P], df[P], dh[P], dtb[P], hv[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int64_t I = L + nh * (e * N + k);
            double s, gn;
            level_factors<N>(a, e * N + k, s, gn);
            const double rbar = a.ref[I], cc = a.gamma * a.ref[2 * nu + I] / rbar;
            const double tbar = a.shell ? a.ref[nu + I] : a.theta0;
            const double s0 = 2.0 * a.qcur[I] - a.qprev[I];
            const double sw = SHELL ? n0 * (2.0 * a.qcur[nu + I] - a.qprev[nu + I]) +
                                          n1 * (2.0 * a.qcur[2 * nu + I] - a.qprev[2 * nu + I]) +
                                          n2 * (2.0 * a.qcur[3 * nu + I] - a.qprev[3 * nu + I])
                                    : 2.0 * a.qcur[3 * nu + I] - a.qprev[3 * nu + I];
            const double s4 = 2.0 * a.qcur[4 * nu + I] - a.qprev[4 * nu + I];
            f[k] = s * rbar * sw;
            h[k] = cc * s0 + cc * rbar / tbar * s4;
            tb[k] = tbar;
            s0v[k] = s0;
            swv[k] = sw;
            rbv[k] = rbar;
            hv[k] = h_of<N>(a, lg, e, k);
        }
        dloc<N>(D, f, df);
        dloc<N>(D, h, dh);
        if (SHELL) dloc<N>(D, tb, dtb);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k == N && e != nz - 1) continue;
            const int g = e * N + k;
            const int64_t I = L + nh * g;
            double s, gn;
            level_factors<N>(a, g, s, gn);
            const double gf = gat(w0, wN, e, k, df[k], hv[k], cf, hp);
            const double gh = gat(w0, wN, e, k, dh[k], hv[k], ch, hp);
            const bool wall = g == 0 || g == nk - 1;
            const double qw = SHELL ? n0 * a.qs[nu + I] + n1 * a.qs[2 * nu + I] + n2 * a.qs[3 * nu + I]
                                    : a.qs[3 * nu + I];
            a.sr[g * nh + L] = a.qs[I] + dt * gf / s;
            a.sx[g * nh + L] = wall ? qw : qw + dt * (gh - gn * s0v[k]) / rbv[k];
            if (SHELL) {
                const double beta = gat(w0, wN, e, k, dtb[k], hv[k], ct, hp);
                a.st[g * nh + L] = a.qs[4 * nu + I] + dt * beta * swv[k];
                a.sb[g * nh + L] = beta;
            }
        }
        cf = df[N];
        ch = dh[N];
        ct = SHELL ? dtb[N] : 0.0;
        hp = hv[N];
    }
    // pass 2: right side of the w system, and the forward elimination with L
    double yh[B];  // the last B values, newest first
#pragma unroll
    for (int s = 0; s < B; ++s) yh[s] = 0.0;
    ch = 0.0;
    hp = 0.0;
    for (int e = 0; e < nz; ++e) {
        double h[P], rr[P], rbv[P], dh[P], hv[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int g = e * N + k;
            const int64_t I = L + nh * g;
            const double rbar = a.ref[I], cc = a.gamma * a.ref[2 * nu + I] / rbar;
            const double tbar = a.shell ? a.ref[nu + I] : a.theta0;
            rr[k] = a.sr[g * nh + L];
            h[k] = cc * rr[k] + cc * rbar / tbar * (SHELL ? a.st[g * nh + L] : a.qs[4 * nu + I]);
            rbv[k] = rbar;
            hv[k] = h_of<N>(a, lg, e, k);
        }
        dloc<N>(D, h, dh);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k == N && e != nz - 1) continue;
            const int g = e * N + k;
            double s, gn;
            level_factors<N>(a, g, s, gn);
            const double gh = gat(w0, wN, e, k, dh[k], hv[k], ch, hp);
            const bool wall = g == 0 || g == nk - 1;
            const double rw = a.sx[g * nh + L];
            double y = wall ? rw : rw - dt * gh / rbv[k] + dt * gn * rr[k] / rbv[k];
            const double *lgp = a.lu + (int64_t)g * W * nh + L;
#pragma unroll
            for (int s = 1; s <= B; ++s) y -= lgp[(B - s) * nh] * yh[s - 1];
#pragma unroll
            for (int s = B - 1; s > 0; --s) yh[s] = yh[s - 1];
            yh[0] = y;
            a.sx[g * nh + L] = y;
        }
        ch = dh[N];
        hp = hv[N];
    }
    // pass 3: back substitution with U, top to bottom
#pragma unroll
    for (int s = 0; s < B; ++s) yh[s] = 0.0;
    for (int g = nk - 1; g >= 0; --g) {
        const double *ug = a.lu + (int64_t)g * W * nh + L;
        double w = a.sx[g * nh + L];
#pragma unroll
        for (int s = 1; s <= B; ++s) w -= ug[(B + s) * nh] * yh[s - 1];
        w *= ug[B * nh];
#pragma unroll
        for (int s = B - 1; s > 0; --s) yh[s] = yh[s - 1];
        yh[0] = w;
        a.sx[g * nh + L] = w;
    }
    // pass 4: rho' = r_rho - (dt/s) G(s rho_bar w), theta' = r_theta - dt beta w,
    // the velocity's n component replaced by w; the Robert-Asselin filter of q^n
    cf = 0.0;
    hp = 0.0;
    for (int e = 0; e < nz; ++e) {
        double f[P], wv[P], df[P], hv[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int g = e * N + k;
            const int64_t I = L + nh * g;
            double s, gn;
            level_factors<N>(a, g, s, gn);
            wv[k] = a.sx[g * nh + L];
            f[k] = s * a.ref[I] * wv[k];
            hv[k] = h_of<N>(a, lg, e, k);
        }
        dloc<N>(D, f, df);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k == N && e != nz - 1) continue;
            const int g = e * N + k;
            const int64_t I = L + nh * g;
            double s, gn;
            level_factors<N>(a, g, s, gn);
            const double gf = gat(w0, wN, e, k, df[k], hv[k], cf, hp);
            const double u0 = a.qs[nu + I], u1 = a.qs[2 * nu + I], u2 = a.qs[3 * nu + I], w = wv[k];
            double nv[5];
            nv[0] = a.sr[g * nh + L] - dt * gf / s;
            if (SHELL) {
                const double qw = n0 * u0 + n1 * u1 + n2 * u2;
                nv[1] = u0 - qw * n0 + w * n0;
                nv[2] = u1 - qw * n1 + w * n1;
                nv[3] = u2 - qw * n2 + w * n2;
                nv[4] = a.st[g * nh + L] - dt * a.sb[g * nh + L] * w;
            } else {
                nv[1] = u0;
                nv[2] = u1;
                nv[3] = w;
                nv[4] = a.qs[4 * nu + I];
            }
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                const double vc = a.qcur[v * nu + I], vp = a.qprev[v * nu + I];
                a.qprev[v * nu + I] = vc + a.ra * (vp - 2.0 * vc + nv[v]);
                a.qcur[v * nu + I] = nv[v];
            }
        }
        cf = df[N];
        hp = hv[N];
    }
}

// One step's vertical correction with the work of a line spread over lanes: a
// workgroup takes kLines lines and one lane per (line, element layer), so the
// explicit parts of the correction (everything but the band solve, which is
// a recurrence along the line) run for all layers at once.  kLines = 16 lines
// of 8 bytes fill a 128-byte cache line.  Element derivatives meet at the
// layer interfaces through LDS; the right side of the band system and its
// solution stay in LDS (X), the line's other values in the lanes' registers, so
// that values are read once but for theta' of both levels (and where imex_keeps
// says so rho' and w) on the box, and q* on the shell, which come from the caches
// again.  Per unique node (box) 34 doubles are read and 10 written, so the kernel
// is bound by memory: 32x32x16, N = 4 (1.06 M nodes, 16,384 lines, 375 MB) 372 -> 84 us,
// 4.5 TB/s, against one lane per line over the whole kernel (k_imex_solve:
// 64 workgroups there, each value's loads behind the level before it).
constexpr int kLines = 16;
constexpr int kChunk = 8;  // levels of factors staged in LDS at a time

template <int N>
constexpr int solve_stage() { return kChunk * (2 * N + 1) * kLines; }

__host__ __device__ inline int imex_pad_levels(int nk) { return (nk + kChunk - 1) / kChunk * kChunk; }

// LDS of k_imex_lines: X, three interface exchanges, the staged factors
template <int N>
size_t imex_lines_lds(int nk)
{
    const int nz = (nk - 1) / N;
    return 8 * ((size_t)kLines * (imex_pad_levels(nk) + 3 * nz) + solve_stage<N>());
}

// L y = x, then U w = y, on the workgroup's lines by its first wavefront: the
// four 16-lane groups load two levels of factors each (kChunk levels in all, a
// chunk ahead of the recurrence, through registers into F) and run the
// recurrence alike.  The newest value enters last, so a level waits for
// one multiply-add of the level before it.
template <int N>
__device__ __forceinline__ void band_solve(const double *lu, int64_t nh, int64_t L, int nk, double *X, double *F,
                                           int line, int grp)
{
    constexpr int B = 2 * N, W = 2 * B + 1, H = kChunk / 4;
    const int nch = (nk + kChunk - 1) / kChunk;
    double pf[H * (B + 1)], h[B];
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    };
    // factors of chunk c: d = 0..B-1 (L) or B..2B (1/U_gg, U)
    auto load = [&](int c, auto upper) {
        constexpr int D0 = decltype(upper)::value ? B : 0, M = decltype(upper)::value ? B + 1 : B;
#pragma unroll
        for (int r = 0; r < H; ++r) {
            const int g = c * kChunk + grp + 4 * r;
            const double *p = lu + ((int64_t)g * W + D0) * nh + L;
#pragma unroll
            for (int d = 0; d < M; ++d) pf[r * M + d] = g < nk ? p[d * nh] : 0.0;
        }
    };
    auto stage = [&](auto upper) {
        constexpr int M = decltype(upper)::value ? B + 1 : B;
        wave_sync();  // the chunk before has been read
#pragma unroll
        for (int r = 0; r < H; ++r)
#pragma unroll
            for (int d = 0; d < M; ++d) F[((grp + 4 * r) * M + d) * kLines + line] = pf[r * M + d];
        wave_sync();
    };
    using Lo = std::integral_constant<bool, false>;
    using Up = std::integral_constant<bool, true>;
#pragma unroll
    for (int s = 0; s < B; ++s) h[s] = 0.0;
    load(0, Lo{});
    for (int c = 0; c < nch; ++c) {
        stage(Lo{});
        if (c + 1 < nch) load(c + 1, Lo{});
        else load(c, Up{});
#pragma unroll
        for (int l = 0; l < kChunk; ++l) {
            double y = X[(c * kChunk + l) * kLines + line];
#pragma unroll
            for (int s = B; s >= 1; --s) y = fma(-F[(l * B + B - s) * kLines + line], h[s - 1], y);
#pragma unroll
            for (int s = B - 1; s > 0; --s) h[s] = h[s - 1];
            h[0] = y;
            X[(c * kChunk + l) * kLines + line] = y;
        }
    }
#pragma unroll
    for (int s = 0; s < B; ++s) h[s] = 0.0;
    for (int c = nch - 1; c >= 0; --c) {
        stage(Up{});
        if (c > 0) load(c - 1, Up{});
#pragma unroll
        for (int l = kChunk - 1; l >= 0; --l) {
            double w = X[(c * kChunk + l) * kLines + line];
#pragma unroll
            for (int s = B; s >= 1; --s) w = fma(-F[(l * (B + 1) + s) * kLines + line], h[s - 1], w);
            w *= F[l * (B + 1) * kLines + line];  // beyond the line: zero
#pragma unroll
            for (int s = B - 1; s > 0; --s) h[s] = h[s - 1];
            h[0] = w;
            X[(c * kChunk + l) * kLines + line] = w;
        }
    }
}

// D f on one element's nodes (the zeta derivative), once per phase: D from the
// kernel arguments (dloc's callers loop over elements)
template <int N>
__device__ __forceinline__ void derive(const ImexArgs &a, const double (&f)[N + 1], double (&df)[N + 1])
{
    constexpr int P = N + 1;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < P; ++m) s = fma(a.D[k * P + m], f[m], s);
        df[k] = s;
    }
}

// The Robert-Asselin value of the box's rho' and w at the end takes q^n and q^{n-1}
// from registers, or reads them again where those registers cost more than the
// reads (kept / read again, us per step): N = 5, 32x32x16 464 / 379 (two waves per
// SIMD or one), 16x16x17 133 / 132; N = 7, 16x16x17 535 / 469, but 32x32x8 595 / 612;
// N = 8, 16x16x8 257 / 251, but 16x16x17 930 / 1,116; N <= 4 mostly 1 to 3 %
// slower read again, N = 6 equal.
template <int N, int MAXT> constexpr bool imex_keeps()
{
    return !(N == 5 || (N == 7 && MAXT == 512) || (N == 8 && MAXT == 256));
}
template <int N, bool SHELL, int MAXT>
__global__ __launch_bounds__(MAXT) void k_imex_lines(ImexArgs a)
{
    constexpr int P = N + 1;
    extern __shared__ double sm[];
    const int nk = a.nk, nz = (nk - 1) / N, nkp = imex_pad_levels(nk);
    double *X = sm, *E0 = X + nkp * kLines, *E1 = E0 + nz * kLines, *E2 = E1 + nz * kLines, *F = E2 + nz * kLines;
    const int t = threadIdx.x, line = t % kLines, e = t / kLines;
    const int64_t nh = a.nh, nu = a.nu;
    int64_t L = (int64_t)blockIdx.x * kLines + line;
    const bool mine = L < nh;  // lanes past the last line repeat it and write nothing
    if (!mine) L = nh - 1;
    const bool act = e < nz;
    const LineGeo lg = line_geo<N>(a, L);
    const double n0 = SHELL ? lg.n[0] : 0.0, n1 = SHELL ? lg.n[1] : 0.0, n2 = SHELL ? lg.n[2] : 1.0;
    const double dt = a.dt, ra = a.ra, w0 = a.w[0], wN = a.w[N];
    const int top = e == nz - 1 ? P : N;  // nodes the lane owns: k < top
    const int64_t I0 = L + nh * ((int64_t)e * N);
    const int x0 = e * N * kLines + line;
    for (int g = nk + e; g < nkp; g += (int)(blockDim.x / kLines)) X[g * kLines + line] = 0.0;
    // shared by the phases: rho_bar, c2, kap at the nodes; G at an owned node
    // k is (d_k + the derivative of the layer below at k = 0) times gi[k], times
    // w_0 at an interface
    double rb[P], cc[P], kp[P], sv[P], gn[P], gi[P];
    auto gat = [&](int k, double dk, const double *Ex) {
        if (k == 0 && e > 0) return (wN * Ex[(e - 1) * kLines + line] + w0 * dk) * gi[0];
        return dk * gi[k];
    };
    double rr[P], rt[P], be[P], sd0[P], swv[P], rw[P], qr[P], qw3[P];
    double df[P], dh[P], dtb[P];
    if (act) {
        double f[P], h[P], tb[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int64_t I = I0 + nh * k;
            rb[k] = a.ref[I];
            tb[k] = SHELL ? a.ref[nu + I] : a.theta0;
            cc[k] = a.gamma * a.ref[2 * nu + I] / rb[k];
            kp[k] = cc[k] * rb[k] / tb[k];
            const double c0 = a.qcur[I], p0 = a.qprev[I], c4 = a.qcur[4 * nu + I], p4 = a.qprev[4 * nu + I];
            const double c3 = a.qcur[3 * nu + I], p3 = a.qprev[3 * nu + I];
            sd0[k] = 2.0 * c0 - p0;
            if (SHELL) {
                swv[k] = n0 * (2.0 * a.qcur[nu + I] - a.qprev[nu + I]) +
                         n1 * (2.0 * a.qcur[2 * nu + I] - a.qprev[2 * nu + I]) + n2 * (2.0 * c3 - p3);
                const double *sl = a.slay + 4 * (e * P + k);
                sv[k] = 1.0 / (sl[0] * sl[0]);
                gn[k] = -sl[3];
                gi[k] = sl[1];
            } else {
                swv[k] = 2.0 * c3 - p3;
                sv[k] = 1.0;
                gn[k] = a.gz;
                gi[k] = lg.izz;
                qr[k] = c0;  // for the Robert-Asselin values at the end
                qw3[k] = c3;
            }
            f[k] = sv[k] * rb[k] * swv[k];
            h[k] = cc[k] * sd0[k] + kp[k] * (2.0 * c4 - p4);
        }
        if (e > 0)  // the mean of two layers
            gi[0] = SHELL ? 1.0 / (wN / a.slay[4 * ((e - 1) * P + N) + 1] + w0 / gi[0]) : lg.izz / (wN + w0);
        derive<N>(a, f, df);
        derive<N>(a, h, dh);
        E0[t] = df[N];
        E1[t] = dh[N];
        if (SHELL) {
            derive<N>(a, tb, dtb);
            E2[t] = dtb[N];
        }
    }
    __syncthreads();
    double rho_a = 0.0, rt_a = 0.0;  // r_rho and r_theta of the layer's top node
    if (act) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k >= top) continue;
            const int64_t I = I0 + nh * k;
            const int g = e * N + k;
            const double gf = gat(k, df[k], E0), gh = gat(k, dh[k], E1);
            rr[k] = a.qs[I] + dt * gf / sv[k];
            const double qw = SHELL ? n0 * a.qs[nu + I] + n1 * a.qs[2 * nu + I] + n2 * a.qs[3 * nu + I]
                                    : a.qs[3 * nu + I];
            rw[k] = g == 0 || g == nk - 1 ? qw : qw + dt * (gh - gn[k] * sd0[k]) / rb[k];
            rt[k] = a.qs[4 * nu + I];
            if (SHELL) {
                be[k] = gat(k, dtb[k], E2);
                rt[k] += dt * be[k] * swv[k];
            }
        }
    }
    __syncthreads();  // the exchanges are read: E0, E1 carry the interface values downwards
    if (act) {
        E0[t] = rr[0];
        E1[t] = rt[0];
        if (!SHELL && mine) {  // u, v and theta of the box are the explicit step's
#pragma unroll
            for (int k = 0; k < P; ++k) {
                if (k >= top) continue;
#pragma unroll
                for (int v = 1; v < 5; v += v == 2 ? 2 : 1) {
                    const int64_t J = v * nu + I0 + nh * k;
                    const double vc = a.qcur[J], vp = a.qprev[J], nv = v == 4 ? rt[k] : a.qs[J];
                    a.qprev[J] = vc + ra * (vp - 2.0 * vc + nv);
                    a.qcur[J] = nv;
                }
            }
        }
    }
    __syncthreads();
    if (act) {
        double h[P];
        if (top == N) {
            rho_a = E0[t + kLines];
            rt_a = E1[t + kLines];
        }
#pragma unroll
        for (int k = 0; k < P; ++k)
            h[k] = k < N || top == P ? cc[k] * rr[k] + kp[k] * rt[k] : cc[k] * rho_a + kp[k] * rt_a;
        derive<N>(a, h, dh);
        E2[t] = dh[N];
    }
    __syncthreads();
    if (act)
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k >= top) continue;
            const int g = e * N + k;
            const double gh = gat(k, dh[k], E2);
            X[x0 + k * kLines] = g == 0 || g == nk - 1 ? rw[k] : rw[k] - dt * (gh - gn[k] * rr[k]) / rb[k];
        }
    __syncthreads();
    if (t < 64) band_solve<N>(a.lu, nh, L, nk, X, F, line, t / kLines);
    __syncthreads();
    // rho' = r_rho - (dt/s) G(s rho_bar w), theta' = r_theta - dt beta w, the
    // velocity's n component replaced by w; the filtered q^n
    double wv[P];
    if (act) {
        double f[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            wv[k] = X[x0 + k * kLines];
            f[k] = sv[k] * rb[k] * wv[k];
        }
        derive<N>(a, f, df);
        E0[t] = df[N];
    }
    __syncthreads();
    if (act && mine)
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k >= top) continue;
            const int64_t I = I0 + nh * k;
            const double gf = gat(k, df[k], E0), w = wv[k];
            const double nr = rr[k] - dt * gf / sv[k];
            if (SHELL) {
                const double u0 = a.qs[nu + I], u1 = a.qs[2 * nu + I], u2 = a.qs[3 * nu + I];
                const double qw = n0 * u0 + n1 * u1 + n2 * u2;
                const double nv[5] = {nr, u0 - qw * n0 + w * n0, u1 - qw * n1 + w * n1, u2 - qw * n2 + w * n2,
                                      rt[k] - dt * be[k] * w};
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    const double vc = a.qcur[v * nu + I], vp = a.qprev[v * nu + I];
                    a.qprev[v * nu + I] = vc + ra * (vp - 2.0 * vc + nv[v]);
                    a.qcur[v * nu + I] = nv[v];
                }
            } else {
                constexpr bool KEEP = imex_keeps<N, MAXT>();
                const int64_t J = 3 * nu + I;
                const double c0 = KEEP ? qr[k] : a.qcur[I], c3 = KEEP ? qw3[k] : a.qcur[J];
                const double d0 = KEEP ? sd0[k] : 2.0 * c0 - a.qprev[I], d3 = KEEP ? swv[k] : 2.0 * c3 - a.qprev[J];
                a.qprev[I] = c0 + ra * (nr - d0);
                a.qcur[I] = nr;
                a.qprev[J] = c3 + ra * (w - d3);
                a.qcur[J] = w;
            }
        }
}

ImexArgs imex_args(Mesh &m, double dt, double ra, double *qprev, double *qcur)
{
    ImexArgs a{};
    a.qs = m.dv.qs;
    a.qcur = qcur;
    a.qprev = qprev;
    a.ref = m.dv.ref;
    a.hcol = m.dv.hcol;
    a.slay = m.dv.slay;
    a.xu = m.dv.xu;
    a.lu = m.dv.imexLU;
    a.sr = m.dv.qs2;
    a.sx = m.dv.qs2 + m.nu;
    a.st = m.dv.qs2 + 2 * m.nu;
    a.sb = m.dv.qs2 + 3 * m.nu;
    a.nu = m.nu;
    a.nh = m.nh;
    a.ni = (int)m.ni;
    a.nk = (int)m.nk;
    a.nx = m.d.ne[0];
    a.shell = m.d.kind == NUMA_MESH_SHELL ? 1 : 0;
    a.dt = dt;
    a.ra = ra;
    a.gamma = m.gamma;
    a.gz = -m.ph.g0;
    a.theta0 = m.ph.T0;
    for (int k = 0; k < m.P * m.P; ++k) a.D[k] = m.D[k];
    for (int k = 0; k < m.P; ++k) a.w[k] = m.w[k];
    return a;
}

// A lane per (line, element layer) up to 32 layers, 512 lanes, the most that
// leaves a lane 256 registers.  Above 16 layers N >= 6 spills (box 372, 292, 772
// bytes a lane at N = 6, 7, 8, shell N = 5..8 156, 384, 608, 820) and still gains
// (step, one lane per line / per line and layer, us): box N = 5 16x16x24 662 / 179,
// N = 6 1,046 / 340, N = 7 16x16x17 1,154 / 468, N = 8 1,747 / 926; shell N = 5 6x8x8x24
// 1,275 / 347, N = 6 2,102 / 662, N = 7 6x8x8x17 1,671 / 968, N = 8 2,497 / 2,055.  Taller
// lines keep one lane per line, and so do many lines of a single layer, where a
// quarter of the wavefront's lanes have one (nz = 1: box N = 5 57,600 lines 68 / 77, N = 7
// 50,176 99 / 120, shell N = 4 55,296 68 / 78; N = 3 31,104 43 / 41, N = 7 28,224 89 / 75).
template <int N>
bool imex_lines_ok(int nk, int64_t nh)
{
    const int nz = (nk - 1) / N;
    if (nz == 1 && N >= 4 && nh >= 33000) return false;
    return nz * kLines <= 512 && imex_lines_lds<N>(nk) <= 65536;
}

template <int N>
int32_t launch_imex_n(const ImexArgs &a, bool factor, size_t lds, hipStream_t s)
{
    if (factor)
        hipLaunchKernelGGL((k_imex_factor<N>), dim3((unsigned)a.nh), dim3(64), lds, s, a);
    else if (imex_lines_ok<N>(a.nk, a.nh)) {
        const int nz = (a.nk - 1) / N, bt = nz < 4 ? 64 : (nz * kLines + 63) / 64 * 64;
        const dim3 grid((unsigned)((a.nh + kLines - 1) / kLines)), block(bt);
        const size_t ldsl = imex_lines_lds<N>(a.nk);
        if (a.shell && bt <= 256)
            hipLaunchKernelGGL((k_imex_lines<N, true, 256>), grid, block, ldsl, s, a);
        else if (a.shell)
            hipLaunchKernelGGL((k_imex_lines<N, true, 512>), grid, block, ldsl, s, a);
        else if (bt <= 256)
            hipLaunchKernelGGL((k_imex_lines<N, false, 256>), grid, block, ldsl, s, a);
        else
            hipLaunchKernelGGL((k_imex_lines<N, false, 512>), grid, block, ldsl, s, a);
    } else if (a.shell)
        hipLaunchKernelGGL((k_imex_solve<N, true>), dim3((unsigned)((a.nh + 255) / 256)), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((k_imex_solve<N, false>), dim3((unsigned)((a.nh + 255) / 256)), dim3(256), 0, s, a);
    NUMA_HIP(hipGetLastError());
    return NUMA_OK;
}

int32_t launch_imex(Mesh &m, bool factor, double dt, double ra, double *qprev, double *qcur, hipStream_t s)
{
    const ImexArgs a = imex_args(m, dt, ra, qprev, qcur);
    const size_t lds = (size_t)imex_lds_bytes(m);
    switch (m.N) {
    case 1: return launch_imex_n<1>(a, factor, lds, s);
    case 2: return launch_imex_n<2>(a, factor, lds, s);
    case 3: return launch_imex_n<3>(a, factor, lds, s);
    case 4: return launch_imex_n<4>(a, factor, lds, s);
    case 5: return launch_imex_n<5>(a, factor, lds, s);
    case 6: return launch_imex_n<6>(a, factor, lds, s);
    case 7: return launch_imex_n<7>(a, factor, lds, s);
    default: return launch_imex_n<8>(a, factor, lds, s);
    }
}

}  // namespace

uint64_t imex_lds_bytes(const Mesh &m)
{
    return 8ull * (uint64_t)m.nk * ((4 * m.N + 1) + (2 * m.N + 1) + 6);
}

uint64_t imex_factor_bytes(const Mesh &m)
{
    return 8ull * (uint64_t)m.nk * (4 * m.N + 1) * (uint64_t)m.nh;
}

int32_t launch_imex_factor(Mesh &m, double dt, hipStream_t s)
{
    return launch_imex(m, true, dt, 0.0, nullptr, nullptr, s);
}

int32_t launch_imex_correction(Mesh &m, double dt, double ra, double *qprev, double *qcur, hipStream_t s)
{
    return launch_imex(m, false, dt, ra, qprev, qcur, s);
}

}  // namespace numa
