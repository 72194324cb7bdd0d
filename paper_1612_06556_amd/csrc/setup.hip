// setup.hip -- gauge ingest (canonical links to the internal copies, SU(3)
// check) and the clover term: field strength, the packed 6x6 blocks T and
// their inverses, in every storage.
#include "wcl_launch.h"

namespace wcl {

// Two-row (12-real) FP32 and FP16 copies of the FP64 links.
__global__ void k_compress_links(Geom g, const void *u64, void *u32c, void *u16c)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 8 * g.Vh) return;
    const int mp = i / g.Vh, h = i - mp * g.Vh;
    cplx<double> u[9];
    load_link<double, double>(u64, mp >> 1, mp & 1, h, g.Vh, u);
    store_link<R12f, double>(u32c, mp >> 1, mp & 1, h, g.Vh, u);
    store_link<R12h, double>(u16c, mp >> 1, mp & 1, h, g.Vh, u);
}

hipError_t launch_compress_links(const Geom &g, const void *u64, void *u32c, void *u16c, hipStream_t st)
{
    k_compress_links<<<(8 * g.Vh + 255) / 256, 256, 0, st>>>(g, u64, u32c, u16c);
    return hipGetLastError();
}

// Largest |row2 - conj(row0 x row1)| over the FP64 links (per-workgroup maxima).
// max that keeps a NaN (fmax would drop it)
WCL_D double nanmax(double m, double d) { return (d > m || d != d) ? d : m; }

// Largest of |row2 - conj(row0 x row1)|, |row norm - 1|, |<row0, row1>| of one link.
WCL_D double su3_defect(const cplx<double> u[9])
{
    cplx<double> r[9];
    double m = 0.0;
#pragma unroll
    for (int k = 0; k < 9; k++) r[k] = u[k];
    su3_third_row(r);
#pragma unroll
    for (int k = 6; k < 9; k++) m = nanmax(m, fmax(fabs(r[k].re - u[k].re), fabs(r[k].im - u[k].im)));
    cplx<double> ip = {0.0, 0.0};
    double n0 = 0.0, n1 = 0.0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const cplx<double> a = u[c], b = u[3 + c];
        n0 += a.re * a.re + a.im * a.im;
        n1 += b.re * b.re + b.im * b.im;
        ip.re += a.re * b.re + a.im * b.im;
        ip.im += a.re * b.im - a.im * b.re;
    }
    m = nanmax(m, fabs(n0 - 1.0));
    m = nanmax(m, fabs(n1 - 1.0));
    return nanmax(m, sqrt(ip.re * ip.re + ip.im * ip.im));
}

__global__ void __launch_bounds__(256) k_su3_check(Geom g, const void *u64, double *partial)
{
    __shared__ double red[256];
    double m = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 8 * g.Vh; i += gridDim.x * blockDim.x) {
        const int mp = i / g.Vh, h = i - mp * g.Vh;
        cplx<double> u[9];
        load_link<double, double>(u64, mp >> 1, mp & 1, h, g.Vh, u);
        m = nanmax(m, su3_defect(u));
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] = nanmax(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

hipError_t launch_su3_check(const Geom &g, const void *u64, double *partial, int nblocks, hipStream_t st)
{
    k_su3_check<<<nblocks, 256, 0, st>>>(g, u64, partial);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gauge ingest: canonical U[V][4][3][3] complex128 to every internal copy in
// one pass.  A workgroup takes 32 pairs of x-neighbours (1152 contiguous bytes
// a pair) through LDS, each wave one direction.  Two-row copies (c32, c16;
// may be null) come with the SU(3) check: *defect (0 before) receives the
// bits of the largest defect above `tol` (non-negative doubles, NaN above all,
// order as their bits).  Bound by HBM: U once in, the copies out: 165 us at
// 24^3x32 with two-row copies (913 MB, 5.5 TB/s; 362 us as three passes, the first
// with 576-byte strides).
__global__ void __launch_bounds__(256) k_ingest_gauge(Geom g, const double2 *__restrict__ canon, void *u64, void *u32,
                                                      void *u16, void *c32, void *c16, double tol,
                                                      unsigned long long *defect)
{
    constexpr int ROW = 64 * 9 + 1;   // 16-byte units of one direction
    __shared__ double2 lds[4 * ROW];
    __shared__ uint32_t base[32];     // canonical index of the x-even site | its parity << 31
    const uint32_t Vh = g.Vh, h0 = blockIdx.x * 32u, np = min(32u, Vh - h0);
    const uint32_t tid = threadIdx.x;
    if (tid < np) base[tid] = pair_base(g, (int)(h0 + tid));
    __syncthreads();
    double2 v[9];
#pragma unroll
    for (int j = 0; j < 9; j++) {
        const uint32_t i = (uint32_t)j * 256u + tid, pr = min(i / 72u, np - 1);
        v[j] = canon[(size_t)(base[pr] & 0x7fffffffu) * 36 + i % 72u];
    }
#pragma unroll
    for (int j = 0; j < 9; j++) {
        const uint32_t i = (uint32_t)j * 256u + tid, pr = i / 72u, r = i % 72u, xo = r / 36u, e = r - xo * 36u;
        if (pr < np) lds[(e / 9u) * ROW + (((xo + (base[pr] >> 31)) & 1u) * 32u + pr) * 9u + e % 9u] = v[j];
    }
    __syncthreads();
    const uint32_t lane = tid & 63u, mu = tid >> 6, p = lane >> 5, h = h0 + (lane & 31u);
    double m = 0.0;
    if ((lane & 31u) < np) {
        cplx<double> u[9];
#pragma unroll
        for (uint32_t k = 0; k < 9; k++) {
            const double2 d = lds[mu * ROW + lane * 9u + k];
            u[k] = {d.x, d.y};
        }
        store_link<double, double>(u64, mu, p, h, Vh, u);
        store_link<float, double>(u32, mu, p, h, Vh, u);
        store_link<__half, double>(u16, mu, p, h, Vh, u);
        if (c32) {
            m = su3_defect(u);
            store_link<R12f, double>(c32, mu, p, h, Vh, u);
            store_link<R12h, double>(c16, mu, p, h, Vh, u);
        }
    }
    if (!(m <= tol)) atomicMax(defect, (unsigned long long)__double_as_longlong(m));
}

hipError_t launch_ingest_gauge(const Geom &g, const double *canon, void *u64, void *u32, void *u16, void *c32, void *c16,
                               double tol, unsigned long long *defect, hipStream_t st)
{
    k_ingest_gauge<<<(g.Vh + 31) / 32, 256, 0, st>>>(g, (const double2 *)canon, u64, u32, u16, c32, c16, tol, defect);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Clover term.  For each site, F_{mu nu} = (Q - Q^dag)/(8i) made traceless,
// Q the sum of the four plaquette leaves in the mu-nu plane.  In the chiral
// basis sum_{mu<nu} sigma_{mu nu} F_{mu nu} is block diagonal:
//   chirality +: sum_k s_k (x) (E_k - B_k),   chirality -: sum_k s_k (x) (-E_k - B_k)
// with E_k = F_{k t} and B = (F_yz, F_zx, F_xy), and s_k (x) G written out as
// [[G_3, G_1 - i G_2], [G_1 + i G_2, -G_3]].
struct M3 {
    cplx<double> a[9];
};

WCL_D M3 m3_mul(const M3 &A, const M3 &B)
{
    M3 C;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            cplx<double> s = A.a[i * 3] * B.a[j];
            s = cfma(A.a[i * 3 + 1], B.a[3 + j], s);
            s = cfma(A.a[i * 3 + 2], B.a[6 + j], s);
            C.a[i * 3 + j] = s;
        }
    return C;
}

WCL_D M3 m3_dag(const M3 &A)
{
    M3 C;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) C.a[i * 3 + j] = {A.a[j * 3 + i].re, -A.a[j * 3 + i].im};
    return C;
}

// Inverse of a Hermitian positive definite 6x6 by Cholesky: A = L L^dag,
// A^-1 = W^dag W with W = L^-1.  Returns false on a non-positive pivot.
WCL_D bool hpd_inverse6(const cplx<double> A[36], cplx<double> Ai[36])
{
    cplx<double> L[36];
#pragma unroll
    for (int k = 0; k < 36; k++) L[k] = {0.0, 0.0};
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; j++) {
        double d = A[j * 6 + j].re;
#pragma unroll
        for (int k = 0; k < j; k++) d -= L[j * 6 + k].re * L[j * 6 + k].re + L[j * 6 + k].im * L[j * 6 + k].im;
        if (!(d > 0.0)) { ok = false; d = 1.0; }
        const double ljj = sqrt(d);
        L[j * 6 + j] = {ljj, 0.0};
        const double inv = 1.0 / ljj;
#pragma unroll
        for (int i = j + 1; i < 6; i++) {
            cplx<double> s = A[i * 6 + j];
#pragma unroll
            for (int k = 0; k < j; k++) s = s - L[i * 6 + k] * cplx<double>{L[j * 6 + k].re, -L[j * 6 + k].im};
            L[i * 6 + j] = inv * s;
        }
    }
    // W = L^-1 (lower triangular), forward substitution column by column
    cplx<double> W[36];
#pragma unroll
    for (int k = 0; k < 36; k++) W[k] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 6; j++) {
        W[j * 6 + j] = {1.0 / L[j * 6 + j].re, 0.0};
#pragma unroll
        for (int i = j + 1; i < 6; i++) {
            cplx<double> s = {0.0, 0.0};
#pragma unroll
            for (int k = j; k < i; k++) s = cfma(L[i * 6 + k], W[k * 6 + j], s);
            W[i * 6 + j] = (-1.0 / L[i * 6 + i].re) * s;
        }
    }
    // Ai = W^dag W
#pragma unroll
    for (int i = 0; i < 6; i++)
#pragma unroll
        for (int j = 0; j < 6; j++) {
            cplx<double> s = {0.0, 0.0};
            const int k0 = i > j ? i : j;
#pragma unroll
            for (int k = k0; k < 6; k++) s = cjfma(W[k * 6 + i], W[k * 6 + j], s);
            Ai[i * 6 + j] = s;
        }
    return ok;
}

WCL_D void pack_block(const cplx<double> A[36], double *out36)
{
#pragma unroll
    for (int i = 0; i < 6; i++) out36[i] = A[i * 6 + i].re;
    int k = 0;
#pragma unroll
    for (int i = 0; i < 6; i++)
#pragma unroll
        for (int j = i + 1; j < 6; j++) {
            out36[6 + 2 * k] = A[i * 6 + j].re;
            out36[7 + 2 * k] = A[i * 6 + j].im;
            k++;
        }
}

// Leaf w into the leaf sum of site i.
template <bool FIRST>
WCL_D void put_leaf(double q[18][128], int i, const M3 &w)
{
#pragma unroll
    for (int k = 0; k < 9; k++) {
        q[2 * k][i] = FIRST ? w.a[k].re : q[2 * k][i] + w.a[k].re;
        q[2 * k + 1][i] = FIRST ? w.a[k].im : q[2 * k + 1][i] + w.a[k].im;
    }
}

// Clover setup in two passes.  Pass 1, one plane mu nu at a time: the plaquette
// with lowest corner c gives four leaves.  With A = U_mu(c) U_nu(c+mu),
// B = U_mu(c+nu)^dag U_nu(c)^dag, C = U_nu(c+mu) U_mu(c+nu)^dag,
// D = U_nu(c)^dag U_mu(c) they are A B at c, C D at c+mu, B A at c+mu+nu and D C at
// c+nu.  A workgroup takes 4 x 8 x 4 sites (mu, nu and the first other
// direction; ragged where the extents are) and, a thread each, the 180
// plaquettes with c in them or one step below; the leaves are added up in LDS,
// one kind after the other (each site gets one of each), and the sites form
// the traceless Hermitian F_{mu nu} = (Q - Q^dag)/(8i) - tr, stored as its upper
// triangle (F00, F11, F22, Re/Im F01, F02, F12: 9 reals) in F[plane][9][2 Vh].
// Planes: E_k = F_{k t} (0..2), B_x = F_yz, -B_y = F_xz, B_z = F_xy (3..5).
// A plaquette's 4 links and 8 products serve its four leaves, which made one
// by one at their own sites read 16 links and take 12 products; the 32 regions
// and 6 planes of an 8^4 block (2.4 MB of links) run side by side on one XCD, so
// its links come from memory once.  Bound by the texture units' 16-byte loads
// and the FP64 products: 420 us at 24^3x32 (739 with one thread a leaf; two
// threads a plaquette measured 756, reading the links twice instead of holding
// them 600, one thread a plaquette of a 4^4 region with its parities mixed in
// the lanes 576).
constexpr int FS_T = 192;
__global__ void __launch_bounds__(FS_T, 2) k_clover_fs(Geom g, const void *u64, double *F)
{
    __shared__ double q[18][128];
    const int lin = xcd_block(blockIdx.x, gridDim.x);
    const int region = lin & 31, plane = (lin >> 5) % 6;   // of an 8^4 block
    // (mu, nu) of the planes: (0,3) (1,3) (2,3) (1,2) (0,2) (0,1); rho < tau the others
    const int mu = plane < 3 ? plane : (plane == 3 ? 1 : 0);
    const int nu = plane < 3 ? 3 : (plane == 5 ? 1 : 2);
    const int rho = mu > 0 ? 0 : (nu > 1 ? 1 : 2), tau = 6 - mu - nu - rho;
    const int id = threadIdx.x;     // plaquette of the region
    const bool here = id < 128;     // c is one of its sites
    int lm, ln, lr;
    if (here) {
        // half a wave holds one parity: consecutive lanes read consecutive
        // half-sites (x is mu or rho, and the region starts at a multiple of 4
        // in every direction but tau)
        const int o = (id >> 1) & 3;
        ln = ((id >> 3) & 3) + 4 * (id >> 6);
        const int x = 2 * (id & 1) + (((id >> 5) + o + ln + (region >> 2)) & 1);
        lm = mu == 0 ? x : o;
        lr = mu == 0 ? o : x;
    } else {
        const int w = (id - 128) >> 2;           // 0..8: a step below in mu; 9..12: in nu
        lr = id & 3;
        lm = w < 9 ? -1 : w - 9;
        ln = w < 9 ? w - 1 : -1;
    }
    int r = lin / 192;
    Site s;
    s.blk = 0;
    s.lin = 0;
    int par = 0;
    bool on = id < 180, in_mu = false, in_nu = false;       // c + mu, c + nu is a site of the region
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int n = (g.L[k] + 7) >> 3;
        const int x = 8 * (r % n) + (k == mu ? 4 * (region & 1) + lm : k == nu ? ln : k == rho ? 2 * (region & 2) + lr : region >> 2);
        r /= n;
        on = on && x < g.L[k];
        if (k == mu) in_mu = lm < 3 && x + 1 < g.L[k];
        if (k == nu) in_nu = ln < 7 && x + 1 < g.L[k];
        const int y = x < 0 ? g.L[k] - 1 : x < g.L[k] ? x : 0;
        s.x[k] = y;
        s.b[k] = y / g.B[k];
        s.l[k] = y - s.b[k] * g.B[k];
        s.blk += s.b[k] * g.sb[k];
        s.lin += s.l[k] * g.sl[k];
        par += y;
    }
    const int p = par & 1;
    const int li = lm + 4 * lr + 16 * ln;
    const uint32_t h = at(g, s, Step{0, 0});
    M3 P, Q, R, S, w;   // U_mu(c), U_nu(c+mu), U_mu(c+nu)^dag, U_nu(c)^dag
    if (on) {
        load_link<double, double>(u64, mu, p, h, g.Vh, P.a);
        load_link<double, double>(u64, nu, 1 - p, at(g, s, step_of(g, s, mu, 1)), g.Vh, Q.a);
        load_link<double, double>(u64, mu, 1 - p, at(g, s, step_of(g, s, nu, 1)), g.Vh, R.a);
        load_link<double, double>(u64, nu, p, h, g.Vh, S.a);
        R = m3_dag(R);
        S = m3_dag(S);
        const M3 A = m3_mul(P, Q), B = m3_mul(R, S);
        w = m3_mul(A, B);
        if (here) put_leaf<true>(q, li, w);
        w = m3_mul(B, A);
        const M3 C = m3_mul(Q, R), D = m3_mul(S, P);
        P = m3_mul(C, D);
        Q = m3_mul(D, C);
    }
    __syncthreads();
    if (on && in_mu && ln >= 0) put_leaf<false>(q, li + 1, P);
    __syncthreads();
    if (on && in_mu && in_nu) put_leaf<false>(q, li + 17, w);
    __syncthreads();
    if (on && in_nu && lm >= 0) put_leaf<false>(q, li + 16, Q);
    __syncthreads();
    if (!on || !here) return;
#pragma unroll
    for (int k = 0; k < 9; k++) Q.a[k] = {q[2 * k][li], q[2 * k + 1][li]};
    M3 f;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const double wr = Q.a[i * 3 + j].re - Q.a[j * 3 + i].re;
            const double wi = Q.a[i * 3 + j].im + Q.a[j * 3 + i].im;
            f.a[i * 3 + j] = {wi * 0.125, -wr * 0.125};
        }
    const double tr = (f.a[0].re + f.a[4].re + f.a[8].re) / 3.0;
    const size_t n = 2 * (size_t)g.Vh;
    double *o = F + (size_t)plane * 9 * n + (size_t)p * g.Vh + h;
    o[0] = f.a[0].re - tr;
    o[n] = f.a[4].re - tr;
    o[2 * n] = f.a[8].re - tr;
    o[3 * n] = f.a[1].re;
    o[4 * n] = f.a[1].im;
    o[5 * n] = f.a[2].re;
    o[6 * n] = f.a[2].im;
    o[7 * n] = f.a[5].re;
    o[8 * n] = f.a[5].im;
}

// Entry (a, b) of plane `plane` of the stored F (the lower triangle by
// Hermiticity).
WCL_D cplx<double> f_entry(const double *F, size_t n, int idx, int plane, int a, int b)
{
    const double *q = F + (size_t)plane * 9 * n + idx;
    if (a == b) return {q[(size_t)a * n], 0.0};
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    const int k = lo == 0 ? (hi == 1 ? 3 : 5) : 7;
    const double re = q[(size_t)k * n], im = q[(size_t)(k + 1) * n];
    return a < b ? cplx<double>{re, im} : cplx<double>{re, -im};
}

// Half (chirality block chi) of a packed clover site in storage S: FP64 and
// FP32 blocks fill whole 16-byte words; FP16 block 0 ends and block 1 starts
// in word 4, whose other half is carried in `keep`.
template <typename S>
WCL_D void store_clover_block(void *base, int p, uint32_t h, uint32_t Vh, int chi, const double c[36], uint2 &keep)
{
    if constexpr (sizeof(S) == 8) {
#pragma unroll
        for (uint32_t k = 0; k < 18; k++)
            stf(base, (((uint32_t)p * 36 + 18 * chi + k) * Vh + h) * 16u, make_double2(c[2 * k], c[2 * k + 1]));
    } else if constexpr (sizeof(S) == 4) {
#pragma unroll
        for (uint32_t k = 0; k < 9; k++)
            stf(base, (((uint32_t)p * 18 + 9 * chi + k) * Vh + h) * 16u,
                make_float4((float)c[4 * k], (float)c[4 * k + 1], (float)c[4 * k + 2], (float)c[4 * k + 3]));
    } else {
        uint32_t w[18];
#pragma unroll
        for (int k = 0; k < 18; k++) w[k] = f22h((float)c[2 * k], (float)c[2 * k + 1]);
        if (chi == 0) {
#pragma unroll
            for (uint32_t k = 0; k < 4; k++)
                stf(base, (((uint32_t)p * 9 + k) * Vh + h) * 16u, make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]));
            keep = make_uint2(w[16], w[17]);
        } else {
            stf(base, (((uint32_t)p * 9 + 4) * Vh + h) * 16u, make_uint4(keep.x, keep.y, w[0], w[1]));
#pragma unroll
            for (uint32_t k = 0; k < 4; k++)
                stf(base, (((uint32_t)p * 9 + 5 + k) * Vh + h) * 16u,
                    make_uint4(w[2 + 4 * k], w[3 + 4 * k], w[4 + 4 * k], w[5 + 4 * k]));
        }
    }
}

// Pass 2: one thread per site builds T = 1 - c_sw kappa sigma.F one
// chirality block at a time from the stored F, inverts it (FP64 Cholesky)
// and writes both into every requested storage.
__global__ void __launch_bounds__(64) k_clover_inv(Geom g, const double *F, double ck, void *t64, void *ti64,
                                                   void *t32, void *ti32, void *t16, void *ti16, int *info)
{
    const size_t n = 2 * (size_t)g.Vh;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int)n) return;
    const int p = idx / g.Vh;
    const int h = idx - p * g.Vh;
    bool ok = true;
    uint2 keepT = make_uint2(0u, 0u), keepTi = make_uint2(0u, 0u);
    for (int chi = 0; chi < 2; chi++) {
        const double se = chi == 0 ? 1.0 : -1.0;
        // G_k = se * E_k - B_k
        cplx<double> A[36];
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                const cplx<double> G1 = se * f_entry(F, n, idx, 0, a, b) - f_entry(F, n, idx, 3, a, b);
                const cplx<double> G2 = se * f_entry(F, n, idx, 1, a, b) + f_entry(F, n, idx, 4, a, b);
                const cplx<double> G3 = se * f_entry(F, n, idx, 2, a, b) - f_entry(F, n, idx, 5, a, b);
                const cplx<double> iG2 = {-G2.im, G2.re};
                const double id = (a == b) ? 1.0 : 0.0;
                A[a * 6 + b] = cplx<double>{id, 0.0} - ck * G3;
                A[(3 + a) * 6 + 3 + b] = cplx<double>{id, 0.0} + ck * G3;
                A[a * 6 + 3 + b] = -ck * (G1 - iG2);
                A[(3 + a) * 6 + b] = -ck * (G1 + iG2);
            }
        double packed[36];
        pack_block(A, packed);
        if (t64) store_clover_block<double>(t64, p, h, g.Vh, chi, packed, keepT);
        if (t32) store_clover_block<float>(t32, p, h, g.Vh, chi, packed, keepT);
        if (t16) store_clover_block<__half>(t16, p, h, g.Vh, chi, packed, keepT);
        cplx<double> Ai[36];
        ok = hpd_inverse6(A, Ai) && ok;
        pack_block(Ai, packed);
        if (ti64) store_clover_block<double>(ti64, p, h, g.Vh, chi, packed, keepTi);
        if (ti32) store_clover_block<float>(ti32, p, h, g.Vh, chi, packed, keepTi);
        if (ti16) store_clover_block<__half>(ti16, p, h, g.Vh, chi, packed, keepTi);
    }
    if (!ok) atomicAdd(info, 1);
}

hipError_t launch_clover_build(const Geom &g, const void *u64, double ck, void *t64, void *ti64, void *t32,
                               void *ti32, void *t16, void *ti16, int *info, double *fbuf, hipStream_t st)
{
    const int n = 2 * g.Vh;
    int blocks = 1;
    for (int k = 0; k < 4; k++) blocks *= (g.L[k] + 7) / 8;
    k_clover_fs<<<192 * blocks, FS_T, 0, st>>>(g, u64, fbuf);
    k_clover_inv<<<(n + 63) / 64, 64, 0, st>>>(g, fbuf, ck, t64, ti64, t32, ti32, t16, ti16, info);
    return hipGetLastError();
}

}  // namespace wcl
