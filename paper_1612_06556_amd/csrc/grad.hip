// grad.hip -- gradient of L = Re<eta, D^-1 b> with respect to the links and
// kappa, given x = D^-1 b and y = D^-dag eta (FP64).
//
// With dL = -Re<y, dD x> and D = T - kappa H, T = 1 - c_sw kappa C,
// C = sum_{mu<nu} sigma_{mu nu} F_{mu nu}:
//   link gradient G = kappa (W + V) (dL = Re sum conj(G_ab) dU_ab, PyTorch's
//   convention), for the link U_mu(x):
//     hopping:  W = s sum_spin [ ((1 - g_mu) y(x)) x(x+mu)^dag + x(x) ((1 + g_mu) y(x+mu))^dag ];
//               a projected spinor's lower half repeats its upper half up to
//               units, so each spin sum is a sum over two half spinors;
//     clover:   every closed loop E0 E1 E2 E3 from E0 = U_mu(x) round a plaquette
//               (corners c0 = x, c1 = x + mu, c2, c3 at the start of each edge)
//               enters Q at each corner, so dL = kappa Re[-i t tr(dU X)],
//               t = +-c_sw / 8 (+ for the orientation mu nu, mu < nu),
//               X = (K1 E1 + E1 K2) E2 E3 + E1 E2 (K3 E3 + E3 K0)
//               with K = M' + M'^dag, M' the traceless part of
//               M_ab = sum_{s,t} sigma_st x_t,a conj(y_s,b), and V += i t X^dag.
//   kappa:  dL/dkappa = Re<y, H x> + c_sw Re<y, C x>.  H is linear and C
//           homogeneous of degree 4 in the links, so it is the sum over links
//           of Re tr(W^dag U) + Re tr(V^dag U) / 4: no further operator pass.
// A thread gathers, for one link, the 6 plaquettes that contain it.
#include "wcl_launch.h"

namespace wcl {

// --- 3x3 helpers (FP64) -------------------------------------------------------
struct Mat {
    cplx<double> a[9];
};
struct Herm {   // d: diagonal; o: entries (0,1), (0,2), (1,2)
    double d[3];
    cplx<double> o[3];
};

WCL_D cplx<double> mentry(const Mat &A, const Mat &B, int i, int j)   // (A B)_ij
{
    cplx<double> s = A.a[i * 3] * B.a[j];
    s = cfma(A.a[i * 3 + 1], B.a[3 + j], s);
    return cfma(A.a[i * 3 + 2], B.a[6 + j], s);
}

WCL_D Mat mmul(const Mat &A, const Mat &B)
{
    Mat C;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) C.a[i * 3 + j] = mentry(A, B, i, j);
    return C;
}

WCL_D Mat mdag(const Mat &A)
{
    Mat C;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) C.a[i * 3 + j] = {A.a[j * 3 + i].re, -A.a[j * 3 + i].im};
    return C;
}

// P E + E Q
WCL_D Mat edge_insert(const Herm &P, const Mat &E, const Herm &Q)
{
    Mat C;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const double d = P.d[i] + Q.d[j];
            cplx<double> s = {d * E.a[i * 3 + j].re, d * E.a[i * 3 + j].im};
#pragma unroll
            for (int k = 0; k < 3; k++) {
                if (k > i) s = cfma(P.o[i + k - 1], E.a[k * 3 + j], s);
                if (k < i) s = cjfma(P.o[i + k - 1], E.a[k * 3 + j], s);
                if (k < j) s = cfma(Q.o[j + k - 1], E.a[i * 3 + k], s);
                if (k > j) s = cjfma(Q.o[j + k - 1], E.a[i * 3 + k], s);
            }
            C.a[i * 3 + j] = s;
        }
    return C;
}

// K field: double [2 p][6 planes][9][Vh], the 3 diagonal entries and Re, Im of
// (0,1), (0,2), (1,2)
WCL_D Herm K_at(const double *K, int p, uint32_t h, uint32_t Vh, int plane)
{
    const uint32_t base = ((uint32_t)(p * 6 + plane) * 9 * Vh + h) * 8u;
    Herm m;
#pragma unroll
    for (uint32_t k = 0; k < 3; k++) {
        m.d[k] = ldf<double>(K, base + k * Vh * 8u);
        m.o[k] = {ldf<double>(K, base + (3 + 2 * k) * Vh * 8u), ldf<double>(K, base + (4 + 2 * k) * Vh * 8u)};
    }
    return m;
}

WCL_D Mat link64(const void *u64, int mu, int p, uint32_t h, uint32_t Vh)
{
    Mat m;
    load_link<double, double>(u64, mu, p, h, Vh, m.a);
    return m;
}

// sigma_{mu nu} in the chiral basis is diag(e_up s_m, e_lo s_m) (2x2 blocks):
//   xy: -s3, xz: +s2, yz: -s1 (both blocks);  xt: s1, yt: s2, zt: s3 (upper), minus them (lower).
// plane order: (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
__host__ __device__ constexpr int plane_pauli(int p) { return p == 0 ? 3 : p == 1 ? 2 : p == 2 ? 1 : p == 3 ? 1 : p == 4 ? 2 : 3; }
__host__ __device__ constexpr double plane_up(int p) { return (p == 0 || p == 3) ? -1.0 : 1.0; }
__host__ __device__ constexpr double plane_lo(int p) { return p == 1 ? 1.0 : -1.0; }

// M_ab for one plane: sum over chirality blocks and s, t of
// e sigma_st x_t,a conj(y_s,b), sigma a Pauli matrix.
template <int PL>
WCL_D cplx<double> plane_m(const cplx<double> x[12], const cplx<double> y[12], int a, int b)
{
    constexpr int m = plane_pauli(PL);
    cplx<double> r = {0.0, 0.0};
#pragma unroll
    for (int blk = 0; blk < 2; blk++) {
        const double e = blk == 0 ? plane_up(PL) : plane_lo(PL);
        const cplx<double> x0 = x[6 * blk + a], x1 = x[6 * blk + 3 + a], y0 = y[6 * blk + b], y1 = y[6 * blk + 3 + b];
        cplx<double> q;
        if constexpr (m == 1) {
            q = cjfma(y0, x1, conjm(y1, x0));                    // s=0,t=1 and s=1,t=0
        } else if constexpr (m == 2) {
            const cplx<double> d = cjfma(y0, x1, -conjm(y1, x0));  // -i (01) + i (10)
            q = {d.im, -d.re};
        } else {
            q = cjfma(y0, x0, -conjm(y1, x1));
        }
        r = {fma(e, q.re, r.re), fma(e, q.im, r.im)};
    }
    return r;
}

template <int PL>
WCL_D void plane_K(const cplx<double> x[12], const cplx<double> y[12], double *K, uint32_t Vh)
{
    double d[3];
#pragma unroll
    for (int a = 0; a < 3; a++) d[a] = 2.0 * plane_m<PL>(x, y, a, a).re;
    const double tr = (d[0] + d[1] + d[2]) / 3.0;
#pragma unroll
    for (int a = 0; a < 3; a++) K[(size_t)(PL * 9 + a) * Vh] = d[a] - tr;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
        const cplx<double> u = plane_m<PL>(x, y, a, b), v = plane_m<PL>(x, y, b, a);
        K[(size_t)(PL * 9 + 3 + 2 * k) * Vh] = u.re + v.re;
        K[(size_t)(PL * 9 + 4 + 2 * k) * Vh] = u.im - v.im;
    }
}

// K of all 6 planes at one site (streaming: two spinors in, 432 bytes out).
__global__ void __launch_bounds__(128) k_grad_K(Geom g, const double2 *X, const double2 *Y, double *K)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= 2 * g.Vh) return;
    const int p = idx / g.Vh;
    const int h = idx - p * g.Vh;
    cplx<double> xs[12], ys[12];
    load_spinor<double, double>(X + (size_t)p * 12 * g.Vh, h, g.Vh, xs);
    load_spinor<double, double>(Y + (size_t)p * 12 * g.Vh, h, g.Vh, ys);
    double *k = K + (size_t)p * 54 * g.Vh + h;
    plane_K<0>(xs, ys, k, g.Vh);
    plane_K<1>(xs, ys, k, g.Vh);
    plane_K<2>(xs, ys, k, g.Vh);
    plane_K<3>(xs, ys, k, g.Vh);
    plane_K<4>(xs, ys, k, g.Vh);
    plane_K<5>(xs, ys, k, g.Vh);
}

// V += i t X^dag for one plaquette.  LOWER: the one on the -nu side, whose
// edges run U_nu(x+mu-nu)^dag, U_mu(x-nu)^dag, U_nu(x-nu).
template <bool LOWER>
WCL_D void clover_plaquette(const Geom &g, const void *u64, const double *K, const Site &s, int p, uint32_t h, int mu,
                            int nu, int plane, Step sm, double t, const Herm &K0, const Herm &K1, Mat &V)
{
    const uint32_t Vh = g.Vh;
    const Step sn = step_of(g, s, nu, LOWER ? -1 : 1);
    const uint32_t hm = at(g, s, sm), hn = at(g, s, sn), hmn = at(g, s, sm, sn);
    const int q = 1 - p;
    Mat E1 = LOWER ? link64(u64, nu, p, hmn, Vh) : link64(u64, nu, q, hm, Vh);
    const Mat E2 = mdag(link64(u64, mu, q, hn, Vh));
    Mat E3 = LOWER ? link64(u64, nu, q, hn, Vh) : link64(u64, nu, p, h, Vh);
    if (LOWER) E1 = mdag(E1);
    else E3 = mdag(E3);
    {
        const Mat A = edge_insert(K1, E1, K_at(K, p, hmn, Vh, plane));
        const Mat B = mmul(E2, E3);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const cplx<double> x = mentry(A, B, i, j);
                V.a[j * 3 + i] = {fma(t, x.im, V.a[j * 3 + i].re), fma(t, x.re, V.a[j * 3 + i].im)};
            }
    }
    {
        const Mat A = mmul(E1, E2);
        const Mat B = edge_insert(K_at(K, q, hn, Vh, plane), E3, K0);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const cplx<double> x = mentry(A, B, i, j);
                V.a[j * 3 + i] = {fma(t, x.im, V.a[j * 3 + i].re), fma(t, x.re, V.a[j * 3 + i].im)};
            }
    }
}

// W_ab of direction MU from the half spinors of y(x), x(x+mu) and x(x), y(x+mu).
template <int MU>
WCL_D void hop_outer(const cplx<double> xn[12], const cplx<double> yn[12], const cplx<double> xf[12],
                     const cplx<double> yf[12], double sgn, Mat &W)
{
    cplx<double> a[6], b[6], c[6], d[6];
    project<MU, -1, double>(yn, a);
    project<MU, -1, double>(xf, b);
    project<MU, 1, double>(xn, c);
    project<MU, 1, double>(yf, d);
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            cplx<double> w = conjm(b[j], a[i]);
            w = cjfma(b[3 + j], a[3 + i], w);
            w = cjfma(d[j], c[i], w);
            w = cjfma(d[3 + j], c[3 + i], w);
            W.a[i * 3 + j] = {sgn * w.re, sgn * w.im};
        }
}

WCL_D double re_trace_dag(const Mat &A, const Mat &U)   // Re tr(A^dag U)
{
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 9; k++) t = fma(A.a[k].re, U.a[k].re, fma(A.a[k].im, U.a[k].im, t));
    return t;
}

// A workgroup takes 32 pairs of x-neighbours (64 sites, both parities), each
// wave one direction, so the four links of a site meet in LDS and the gradient
// leaves in the caller's canonical order (1152-byte runs).  One plaquette is
// one straight piece of code run six times with run-time directions: the
// matrices stay in registers (an earlier form indexed them at run time: 1.2 KB
// of scratch a thread) and the code in the instruction cache.
// Bound by the neighbour matrices' way through L2 (4.8 KB a link) at one wave
// per SIMD: 222 us at 16^3x32 (11.3 TB/s of those reads; 1559 us, then 50 for
// the canonical copy, 261 for C x and 43 for H x, before).  Holding one row of
// a product at a time, or fencing the plaquettes apart, measured 4 to 8% slower.
__global__ void __launch_bounds__(256) k_grad_link(Geom g, const void *u64, const double2 *X, const double2 *Y,
                                                   const double *K, double kappa, double csw, double2 *gU,
                                                   double *partial)
{
    constexpr int ROW = 64 * 9 + 1;   // 16-byte units of one direction
    __shared__ double2 lds[4 * ROW];
    __shared__ uint32_t base[32];     // canonical index of the x-even site | its parity << 31
    __shared__ double red[4];
    const int lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = lane >> 5;
    const uint32_t Vh = g.Vh, h0 = (uint32_t)xcd_block(blockIdx.x, gridDim.x) * 32u;
    const uint32_t np = min(32u, Vh - h0), h = h0 + (lane & 31);
    double gk = 0.0;
    if ((uint32_t)(lane & 31) < np) {
        const Site s = decompose(g, (int)h, p);
        if (mu == 0 && p == 0) base[lane] = pair_base(g, s);
        const Step sm = step_of(g, s, mu, 1);
        const uint32_t hm = at(g, s, sm);
        const Mat U = link64(u64, mu, p, h, Vh);
        Mat G;
#pragma unroll
        for (int k = 0; k < 9; k++) G.a[k] = {0.0, 0.0};
        for (int k = 1; k < 4; k++) {
            const int nu = (mu + k) & 3;
            const int a = min(mu, nu), b = max(mu, nu);
            const int plane = a == 0 ? b - 1 : a + b;
            const double t = (mu < nu ? 0.125 : -0.125) * csw;
            const Herm K0 = K_at(K, p, h, Vh, plane), K1 = K_at(K, 1 - p, hm, Vh, plane);
            clover_plaquette<false>(g, u64, K, s, p, h, mu, nu, plane, sm, t, K0, K1, G);
            clover_plaquette<true>(g, u64, K, s, p, h, mu, nu, plane, sm, -t, K0, K1, G);
        }
        gk = 0.25 * re_trace_dag(G, U);
        Mat W;
        {
            cplx<double> xn[12], yn[12], xf[12], yf[12];
            const double2 *X1 = X + (size_t)p * 12 * Vh, *Y1 = Y + (size_t)p * 12 * Vh;
            const double2 *X2 = X + (size_t)(1 - p) * 12 * Vh, *Y2 = Y + (size_t)(1 - p) * 12 * Vh;
            load_spinor<double, double>(X1, h, Vh, xn);
            load_spinor<double, double>(Y1, h, Vh, yn);
            load_spinor<double, double>(X2, hm, Vh, xf);
            load_spinor<double, double>(Y2, hm, Vh, yf);
            const double sgn = (mu == 3 && g.tbc < 0 && s.x[3] == g.L[3] - 1) ? -1.0 : 1.0;
            if (mu == 0) hop_outer<0>(xn, yn, xf, yf, sgn, W);
            else if (mu == 1) hop_outer<1>(xn, yn, xf, yf, sgn, W);
            else if (mu == 2) hop_outer<2>(xn, yn, xf, yf, sgn, W);
            else hop_outer<3>(xn, yn, xf, yf, sgn, W);
        }
        gk += re_trace_dag(W, U);
#pragma unroll
        for (int k = 0; k < 9; k++)
            lds[mu * ROW + lane * 9 + k] = make_double2(kappa * (G.a[k].re + W.a[k].re), kappa * (G.a[k].im + W.a[k].im));
    }
    gk = wave_sum(gk);
    if (lane == 0) red[mu] = gk;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    for (uint32_t i = threadIdx.x; i < np * 72u; i += 256u) {
        const uint32_t pr = i / 72u, r = i - pr * 72u, xo = r / 36u, e = r - xo * 36u;
        const uint32_t b = base[pr], q = (xo + (b >> 31)) & 1u;
        gU[(size_t)(b & 0x7fffffffu) * 36 + r] = lds[(e / 9u) * ROW + (q * 32u + pr) * 9u + e % 9u];
    }
}

// gamma5 on FP64 e/o fields (nsec sections of Vh sites): negate spins 2, 3.
__global__ void k_gamma5(size_t nsec, size_t Vh, double2 *f)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nsec * Vh) return;
    const size_t sec = i / Vh, h = i - sec * Vh;
    double2 *b = f + sec * 12 * Vh;
#pragma unroll
    for (int c = 6; c < 12; c++) {
        const double2 v = b[c * Vh + h];
        b[c * Vh + h] = make_double2(-v.x, -v.y);
    }
}

int grad_parts(const Geom &g) { return (g.Vh + 31) / 32; }

hipError_t launch_grad(const Geom &g, const void *u64, const void *X, const void *Y, double *K, double kappa,
                       double csw, double *gU, double *partial, hipStream_t st)
{
    const int n2 = 2 * g.Vh;
    k_grad_K<<<(n2 + 127) / 128, 128, 0, st>>>(g, (const double2 *)X, (const double2 *)Y, K);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_grad_link<<<grad_parts(g), 256, 0, st>>>(g, u64, (const double2 *)X, (const double2 *)Y, K, kappa, csw,
                                               (double2 *)gU, partial);
    return hipGetLastError();
}

hipError_t launch_gamma5(size_t nsec, size_t Vh, void *f, hipStream_t st)
{
    const size_t n = nsec * Vh;
    k_gamma5<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(nsec, Vh, (double2 *)f);
    return hipGetLastError();
}

}  // namespace wcl
