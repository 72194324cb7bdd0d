// kernels.hip -- the even/odd hopping kernel with its fused epilogues, the
// clover apply and the BLAS-1 / reduction kernels of the solvers.
//
// The operator (Wilson-Clover, paper Sec. 1 and Sec. 2):
//   D = T - kappa H,  (H psi)(x) = sum_mu (1 - g_mu) U_mu(x) psi(x+mu)
//                                     + (1 + g_mu) U_mu(x-mu)^dag psi(x-mu),
//   T = 1 - c_sw kappa sum_{mu<nu} sigma_{mu nu} F_{mu nu}  (clover leaves),
// in the chiral basis; H maps one parity onto the other ("hopping matrix
// multiplication", the paper's measured kernel, Sec. 3).
#include <algorithm>

#include "hop_dev.h"

namespace wcl {

// NT: links and clover loaded non-temporally (a single right-hand side reads
// them once per launch).  Off by default: repeated applications in a solver
// find the links in the Infinity Cache only when they were loaded normally.
template <typename SL, typename SS, int MODE, int DEPTH, bool NT, int NS>
__global__ void __launch_bounds__(256) k_hop(HopArgs a)
{
    // workgroup id = site block * nrhs + rhs: the nrhs workgroups of one site
    // block are neighbours in dispatch order (and on one XCD), so each link
    // is fetched from HBM once and served to the other right-hand sides by L2
    // A workgroup takes tpw consecutive site blocks (one contiguous range of
    // every field), one after another.
    const int lin = a.xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int rhs = lin % a.nrhs;
    const int grp = lin / a.nrhs;
    if (a.sc && a.sc[rhs].done) return;
    constexpr int NWORDS = (int)sizeof(SS) * 24 / 16;
    __shared__ uint4 sin[NS > 0 ? NWORDS * NS : 1];
    const int nb = (a.g.Vh + blockDim.x - 1) / blockDim.x;
    for (int k = 0; k < a.tpw; k++) {
        const int bid = grp * a.tpw + k;
        if (bid >= nb) break;                 // uniform in the workgroup
        if (NS > 0 && k) __syncthreads();     // the previous block's staged input is read
        hop_block<SL, SS, MODE, DEPTH, NT, NS>(a, bid, rhs, sin);
    }
}

// ---------------------------------------------------------------------------
// Several right-hand sides per thread (batched inner solves): each link and
// clover block is loaded once into registers and applied to the NR
// right-hand sides of a group, whose neighbour spinors are loaded together.
// FP32 spinors; modes HOP, CLOV_H, XPAY.  A right-hand side whose
// scalars say done is neither computed nor stored.
template <typename SL, int K, int NR>
WCL_D void hop_mr_hop(const HopArgs &a, const Site &s, uint32_t h0, const bool act[NR], const char *const in[NR],
                      cplx<float> acc[NR][12])
{
    constexpr int MU = K >> 1;
    constexpr bool FWD = (K & 1) == 0;
    constexpr int S = FWD ? -1 : 1;
    const Geom &g = a.g;
    const uint32_t Vh = g.Vh;
    uint32_t hn = (uint32_t)neighbour(g, s, MU, FWD ? +1 : -1);
    uint32_t h = h0;
    // this hop's loads wait for the previous hop's work on the first group member
    pipeline_fence(acc[0], hn, h);
    LinkRaw<SL> lr;
    if (FWD) load_link_raw<SL>(a.links, MU, a.p, h, Vh, lr);
    else load_link_raw<SL>(a.links, MU, 1 - a.p, hn, Vh, lr);
    cplx<float> psi[NR][12];
#pragma unroll
    for (int r = 0; r < NR; r++)
        if (act[r]) load_spinor<float, float>(in[r], hn, Vh, psi[r]);
    float sign = 1.f;
    if (MU == 3 && g.tbc < 0 && s.x[3] == (FWD ? g.L[3] - 1 : 0)) sign = -1.f;
    cplx<float> u[9];
    expand_link<SL, float>(lr, u);
#pragma unroll
    for (int r = 0; r < NR; r++) {
        if (!act[r]) continue;
        cplx<float> hh[6], uh[6];
        project<MU, S, float>(psi[r], hh);
        if (MU == 3) {
#pragma unroll
            for (int k = 0; k < 6; k++) hh[k] = sign * hh[k];
        }
        if (FWD) su3_mul(u, hh, uh);
        else su3_dag_mul(u, hh, uh);
        accumulate<MU, S, float>(acc[r], uh);
    }
}

template <typename SL, int K, int NR>
WCL_D void hop_mr_all(const HopArgs &a, const Site &s, uint32_t h, const bool act[NR], const char *const in[NR],
                      cplx<float> acc[NR][12])
{
    if constexpr (K < 8) {
        hop_mr_hop<SL, K, NR>(a, s, h, act, in, acc);
        hop_mr_all<SL, K + 1, NR>(a, s, h, act, in, acc);
    }
}

template <typename SL, int MODE, int NR>
__global__ void __launch_bounds__(256) k_hop_mr(HopArgs a)
{
    // workgroup id = site block * groups + group (the groups of one site block
    // run back to back on one XCD, so L2 serves the links to all of them)
    const int ngr = (a.nrhs + NR - 1) / NR;
    const int lin = a.xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int grp = lin % ngr;
    const int bid = lin / ngr;
    const int r0 = grp * NR;
    bool act[NR];
    bool any = false;
#pragma unroll
    for (int r = 0; r < NR; r++) {
        act[r] = (r0 + r < a.nrhs) && !(a.sc && a.sc[r0 + r].done);
        any = any || act[r];
    }
    if (!any) return;
    const int h = bid * blockDim.x + threadIdx.x;
    if (h >= a.g.Vh) return;
    const uint32_t Vh = a.g.Vh;
    const char *in[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) in[r] = (const char *)a.in + (act[r] ? r0 + r : 0) * a.in_stride;
    const Site s = decompose(a.g, h, a.p);
    cplx<float> acc[NR][12];
#pragma unroll
    for (int r = 0; r < NR; r++)
#pragma unroll
        for (int i = 0; i < 12; i++) acc[r][i] = {0.f, 0.f};
    hop_mr_all<SL, 0, NR>(a, s, h, act, in, acc);

    if constexpr (MODE == HOP) {
#pragma unroll
        for (int r = 0; r < NR; r++)
            if (act[r]) store_spinor<float, float>((char *)a.out + (r0 + r) * a.out_stride, h, Vh, acc[r]);
    } else {
        // one clover chirality block at a time, shared by the group
#pragma unroll
        for (int half = 0; half < 2; half++) {
            float c[36];
            load_clover_half<typename ClovS<SL>::T, float>(a.clov, a.p, h, Vh, half, c);
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (!act[r]) continue;
                cplx<float> o[6];
                clover_mul_half(c, acc[r] + 6 * half, o);
                char *out = (char *)a.out + (r0 + r) * a.out_stride;
                if constexpr (MODE == XPAY) {
                    const char *x = (const char *)a.x + (r0 + r) * a.x_stride;
                    const float cf = (float)a.coef;
#pragma unroll
                    for (int k = 0; k < 3; k++) {
                        const float4 xv = ldf<float4>(x, ((3 * half + k) * Vh + h) * 16u);
                        o[2 * k] = {fmaf(cf, o[2 * k].re, xv.x), fmaf(cf, o[2 * k].im, xv.y)};
                        o[2 * k + 1] = {fmaf(cf, o[2 * k + 1].re, xv.z), fmaf(cf, o[2 * k + 1].im, xv.w)};
                    }
                }
#pragma unroll
                for (int k = 0; k < 3; k++)
                    stf(out, ((3 * half + k) * Vh + h) * 16u,
                        make_float4(o[2 * k].re, o[2 * k].im, o[2 * k + 1].re, o[2 * k + 1].im));
            }
        }
    }
}

template <typename SL, int NR>
static hipError_t hop_mr_dispatch(const HopLaunch &L, const HopArgs &a, dim3 block, hipStream_t st)
{
    const int ngr = (a.nrhs + NR - 1) / NR;
    dim3 grid(((a.g.Vh + block.x - 1) / block.x) * ngr);
    switch (L.mode) {
    case HOP: ext_launch(k_hop_mr<SL, HOP, NR>, grid, block, 0, st, L.ev, a); break;
    case CLOV_H: ext_launch(k_hop_mr<SL, CLOV_H, NR>, grid, block, 0, st, L.ev, a); break;
    case XPAY: ext_launch(k_hop_mr<SL, XPAY, NR>, grid, block, 0, st, L.ev, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename SL>
static hipError_t hop_mr_nr(const HopLaunch &L, const HopArgs &a, dim3 block, hipStream_t st)
{
    if (L.rhs_per_thread == 4) return hop_mr_dispatch<SL, 4>(L, a, block, st);
    return hop_mr_dispatch<SL, 2>(L, a, block, st);
}

// Pipeline-depth variants (hops whose operands are in flight: 2, 3) times
// temporal / non-temporal operator loads.
template <typename SL, typename SS, int MODE>
static hipError_t hop_dispatch_shape(const HopLaunch &L, const HopArgs &a, dim3 grid, dim3 block, hipStream_t st)
{
    const bool nt = L.nontemporal && a.nrhs == 1;
    // staged input spinors (depth 2): one LDS slot per thread; with non-temporal
    // operator loads for single-use (cold) calls
    const bool staged = L.lds_stage && L.depth == 2;
    if (staged && nt && block.x == 64) ext_launch(k_hop<SL, SS, MODE, 2, true, 64>, grid, block, 0, st, L.ev, a);
    else if (staged && nt && block.x == 128) ext_launch(k_hop<SL, SS, MODE, 2, true, 128>, grid, block, 0, st, L.ev, a);
    else if (staged && nt && block.x == 256) ext_launch(k_hop<SL, SS, MODE, 2, true, 256>, grid, block, 0, st, L.ev, a);
    else if (staged && !nt && block.x == 64) ext_launch(k_hop<SL, SS, MODE, 2, false, 64>, grid, block, 0, st, L.ev, a);
    else if (staged && !nt && block.x == 128) ext_launch(k_hop<SL, SS, MODE, 2, false, 128>, grid, block, 0, st, L.ev, a);
    else if (staged && !nt && block.x == 256) ext_launch(k_hop<SL, SS, MODE, 2, false, 256>, grid, block, 0, st, L.ev, a);
    else if (L.depth == 3 && nt) ext_launch(k_hop<SL, SS, MODE, 3, true, 0>, grid, block, 0, st, L.ev, a);
    else if (L.depth == 3) ext_launch(k_hop<SL, SS, MODE, 3, false, 0>, grid, block, 0, st, L.ev, a);
    else if (nt) ext_launch(k_hop<SL, SS, MODE, 2, true, 0>, grid, block, 0, st, L.ev, a);
    else ext_launch(k_hop<SL, SS, MODE, 2, false, 0>, grid, block, 0, st, L.ev, a);
    return hipGetLastError();
}

// The Schur operator's halves in every storage; H alone on FP32 vectors
// (wcl_bench_hop) and the full operator in FP64 (residuals, the solver on the
// full system): applications on the caller's vectors have kernels of their own
// (canon.hip).
template <typename SL, typename SS>
static hipError_t hop_dispatch_mode(const HopLaunch &L, const HopArgs &a, dim3 grid, dim3 block, hipStream_t st)
{
    if (L.mode == CLOV_H) return hop_dispatch_shape<SL, SS, CLOV_H>(L, a, grid, block, st);
    if (L.mode == XPAY) return hop_dispatch_shape<SL, SS, XPAY>(L, a, grid, block, st);
    if constexpr (std::is_same<SS, float>::value)
        if (L.mode == HOP) return hop_dispatch_shape<SL, SS, HOP>(L, a, grid, block, st);
    if constexpr (std::is_same<SS, double>::value)
        if (L.mode == CLOVX) return hop_dispatch_shape<SL, SS, CLOVX>(L, a, grid, block, st);
    return hipErrorInvalidValue;
}

int hop_parts(const HopLaunch &L)
{
    const int bs = L.block > 0 ? L.block : 256;
    return (L.g->Vh + bs - 1) / bs;
}

hipError_t launch_hop(const HopLaunch &L, hipStream_t st)
{
    if (L.nrhs < 1 || L.nrhs > 4096) return hipErrorInvalidValue;
    if (L.nrhs > 1) {
        const size_t sb = spinor_bytes(L.spin_prec == P64 ? 8 : L.spin_prec == P32 ? 4 : 2, (size_t)L.g->Vh);
        if (L.in_stride < sb || L.out_stride < sb || (L.mode >= XPAY && L.x_stride < sb)) return hipErrorInvalidValue;
    }
    HopArgs a;
    a.g = *L.g;
    a.in = L.in;
    a.out = L.out;
    a.links = L.links;
    a.clov = L.clov;
    a.x = L.x;
    a.coef = L.coef;
    a.in_stride = L.in_stride;
    a.out_stride = L.out_stride;
    a.x_stride = L.x_stride;
    a.p = L.p;
    a.xcd = L.xcd;
    a.sc = L.sc;
    a.nrhs = L.nrhs;
    a.tpw = 1;
    const int bs = L.block > 0 ? L.block : 256;
    if (bs > 256 || bs % 64) return hipErrorInvalidValue;
    const int nb = (a.g.Vh + bs - 1) / bs;
    dim3 grid(nb * a.nrhs);
    dim3 block(bs);
    if (L.ndot) return launch_hop_dot(L, a, grid, block, st);
    if (L.tpw > 1) {
        if (L.tpw > 64) return hipErrorInvalidValue;
        a.tpw = L.tpw;
        grid = dim3(((nb + L.tpw - 1) / L.tpw) * a.nrhs);
    }
    if ((L.rhs_per_thread == 2 || L.rhs_per_thread == 4) && a.nrhs >= 2 && L.spin_prec == P32 && L.mode != CLOVX) {
        switch (L.link_prec) {
        case P32: return hop_mr_nr<float>(L, a, block, st);
        case P16: return hop_mr_nr<__half>(L, a, block, st);
        case P32C: return hop_mr_nr<R12f>(L, a, block, st);
        case P16C: return hop_mr_nr<R12h>(L, a, block, st);
        default: break;
        }
    }
    if (L.link_prec == P64 && L.spin_prec == P64) return hop_dispatch_mode<double, double>(L, a, grid, block, st);
    if (L.link_prec == P32 && L.spin_prec == P32) return hop_dispatch_mode<float, float>(L, a, grid, block, st);
    if (L.link_prec == P16 && L.spin_prec == P32) return hop_dispatch_mode<__half, float>(L, a, grid, block, st);
    if (L.link_prec == P16 && L.spin_prec == P16) return hop_dispatch_mode<__half, __half>(L, a, grid, block, st);
    if (L.link_prec == P32C && L.spin_prec == P32) return hop_dispatch_mode<R12f, float>(L, a, grid, block, st);
    if (L.link_prec == P16C && L.spin_prec == P32) return hop_dispatch_mode<R12h, float>(L, a, grid, block, st);
    if (L.link_prec == P16C && L.spin_prec == P16) return hop_dispatch_mode<R12h, __half>(L, a, grid, block, st);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Clover apply: out = A in on one parity (504 flop per site).
template <typename SL, typename SS>
__global__ void __launch_bounds__(256) k_clover(Geom g, int p, const void *clov, const char *in, char *out,
                                               size_t in_stride, size_t out_stride)
{
    using R = typename Real<SL>::T;
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= g.Vh) return;
    in += blockIdx.y * in_stride;
    out += blockIdx.y * out_stride;
    R c[72];
    cplx<R> v[12], o[12];
    load_clover<SL, R>(clov, p, h, g.Vh, c);
    load_spinor<SS, R>(in, h, g.Vh, v);
    clover_mul(c, v, o);
    store_spinor<SS, R>(out, h, g.Vh, o);
}

hipError_t launch_clover(const Geom &g, int lp, int sp, int p, const void *clov, const void *in, void *out,
                         hipStream_t st, int nrhs, size_t in_stride, size_t out_stride, LaunchEvents ev)
{
    dim3 grid((g.Vh + 255) / 256, nrhs), block(256);
    const char *i = (const char *)in;
    char *o = (char *)out;
    if (lp == P32C) lp = P32;
    if (lp == P16C) lp = P16;
    if (lp == P64 && sp == P64) ext_launch(k_clover<double, double>, grid, block, 0, st, ev, g, p, clov, i, o, in_stride, out_stride);
    else if (lp == P32 && sp == P32) ext_launch(k_clover<float, float>, grid, block, 0, st, ev, g, p, clov, i, o, in_stride, out_stride);
    else if (lp == P16 && sp == P32) ext_launch(k_clover<__half, float>, grid, block, 0, st, ev, g, p, clov, i, o, in_stride, out_stride);
    else if (lp == P16 && sp == P16) ext_launch(k_clover<__half, __half>, grid, block, 0, st, ev, g, p, clov, i, o, in_stride, out_stride);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Reductions: wave sums, then one value per wave through LDS.
template <int NV>
WCL_D void block_sum(double v[NV], double *lds /* [NV][16] */)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; k++) {
        v[k] = wave_sum(v[k]);
        if (lane == 0) lds[k * 16 + wid] = v[k];
    }
    __syncthreads();
    if (wid == 0) {
#pragma unroll
        for (int k = 0; k < NV; k++) {
            double t = lane < nw ? lds[k * 16 + lane] : 0.0;
            v[k] = wave_sum(t);
        }
    }
}

// Storage of one complex number (V) and the arithmetic type (C) of the
// flat-vector kernels: FP16 vectors are stored as half2 and computed in FP32.
template <typename T>
struct CT;
template <> struct CT<double> { using V = double2; using C = double; };
template <> struct CT<float> { using V = float2; using C = float; };
template <> struct CT<__half> { using V = __half2; using C = float; };

WCL_D double2 ldv(const double2 &v) { return v; }
WCL_D float2 ldv(const float2 &v) { return v; }
WCL_D float2 ldv(const __half2 &v) { return __half22float2(v); }
WCL_D void stv(double2 &d, double x, double y) { d = make_double2(x, y); }
WCL_D void stv(float2 &d, float x, float y) { d = make_float2(x, y); }
WCL_D void stv(__half2 &d, float x, float y)
{
    fp32_as_computed(x, y);
    d = __floats2half2_rn(x, y);
}

// partials[rhs][(2*k + {0,1}) * RED_BLOCKS + block] = (Re, Im) of sum conj(a_k) b_k
// over the rhs-th slice (stride elements apart); blockIdx.y = rhs.
template <typename T, int NP>
__global__ void __launch_bounds__(RED_THREADS) k_dots(size_t n, size_t stride, const typename CT<T>::V *a0,
                                                      const typename CT<T>::V *b0, const typename CT<T>::V *a1,
                                                      const typename CT<T>::V *b1, const typename CT<T>::V *a2,
                                                      const typename CT<T>::V *b2, double *partials, const Scalars *sc,
                                                      int pstride)
{
    const int rhs = blockIdx.y;
    if (sc && sc[rhs].done) return;
    __shared__ double lds[2 * NP * 16];
    double v[2 * NP];
#pragma unroll
    for (int k = 0; k < 2 * NP; k++) v[k] = 0.0;
    const size_t off = rhs * stride;
    const typename CT<T>::V *A[3] = {a0 + off, a1 + off, a2 + off}, *B[3] = {b0 + off, b1 + off, b2 + off};
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int k = 0; k < NP; k++) {
            const auto x = ldv(A[k][i]), y = ldv(B[k][i]);
            v[2 * k] += (double)x.x * (double)y.x + (double)x.y * (double)y.y;
            v[2 * k + 1] += (double)x.x * (double)y.y - (double)x.y * (double)y.x;
        }
    }
    block_sum<2 * NP>(v, lds);
    if (threadIdx.x == 0) {
        double *pr = partials + (size_t)rhs * 6 * pstride;
#pragma unroll
        for (int k = 0; k < 2 * NP; k++) pr[k * pstride + blockIdx.x] = v[k];
    }
}

hipError_t launch_dots(int prec, size_t n, int np, const void *const *a, const void *const *b, double *partials,
                       const Scalars *sc, hipStream_t st, int nrhs, size_t stride, int pstride)
{
    if (pstride < RED_BLOCKS) return hipErrorInvalidValue;
    const void *A[3] = {a[0], np > 1 ? a[1] : a[0], np > 2 ? a[2] : a[0]};
    const void *B[3] = {b[0], np > 1 ? b[1] : b[0], np > 2 ? b[2] : b[0]};
    dim3 grid(RED_BLOCKS, nrhs), block(RED_THREADS);
#define WCL_DOTS(T, NP)                                                                                   \
    k_dots<T, NP><<<grid, block, 0, st>>>(n, stride, (const CT<T>::V *)A[0], (const CT<T>::V *)B[0],      \
                                          (const CT<T>::V *)A[1], (const CT<T>::V *)B[1],                 \
                                          (const CT<T>::V *)A[2], (const CT<T>::V *)B[2], partials, sc, pstride)
    if (prec == P64) {
        if (np == 1) WCL_DOTS(double, 1);
        else if (np == 2) WCL_DOTS(double, 2);
        else WCL_DOTS(double, 3);
    } else if (prec == P32) {
        if (np == 1) WCL_DOTS(float, 1);
        else if (np == 2) WCL_DOTS(float, 2);
        else WCL_DOTS(float, 3);
    } else if (prec == P16) {
        if (np == 1) WCL_DOTS(__half, 1);
        else if (np == 2) WCL_DOTS(__half, 2);
        else WCL_DOTS(__half, 3);
    } else {
        return hipErrorInvalidValue;
    }
#undef WCL_DOTS
    return hipGetLastError();
}

// The partials of |x - y|^2 per right-hand side (FP64), as k_dots makes them of a
// stored difference: the residual's norm without writing and reading it.
__global__ void __launch_bounds__(RED_THREADS) k_diff_norm(size_t n, size_t stride, const double2 *x, const double2 *y,
                                                           double *partials, int pstride)
{
    __shared__ double lds[16];
    double v[1] = {0.0};
    x += blockIdx.y * stride;
    y += blockIdx.y * stride;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const double2 a = x[i], b = y[i];
        const double dr = a.x - b.x, di = a.y - b.y;
        v[0] += dr * dr + di * di;
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) {
        double *pr = partials + (size_t)blockIdx.y * 6 * pstride + blockIdx.x;
        pr[0] = v[0];
        pr[pstride] = 0.0;
    }
}

hipError_t launch_diff_norm(size_t n, size_t stride, const void *x, const void *y, double *partials, int pstride, int nrhs,
                            hipStream_t st)
{
    if (pstride < RED_BLOCKS) return hipErrorInvalidValue;
    k_diff_norm<<<dim3(RED_BLOCKS, nrhs), RED_THREADS, 0, st>>>(n, stride, (const double2 *)x, (const double2 *)y, partials,
                                                              pstride);
    return hipGetLastError();
}

WCL_D void cdiv(const double a[2], const double b[2], double o[2])
{
    const double d = b[0] * b[0] + b[1] * b[1];
    o[0] = (a[0] * b[0] + a[1] * b[1]) / d;
    o[1] = (a[1] * b[0] - a[0] * b[1]) / d;
}

// omega = <t, s> / <t, t> from the sums (Re, Im <t, s>, <t, t>).
WCL_D void bicg_omega(const double v[3], double omega[2])
{
    const double tt = v[2];
    if (tt == 0.0) { omega[0] = 0.0; omega[1] = 0.0; }
    else { omega[0] = v[0] / tt; omega[1] = v[1] / tt; }
}

// State of the recurrence after <rt, r> and |r|^2: 0 go on, 1 converged, 2 breakdown or NaN.
WCL_D int bicg_stop(const double v[3], const Scalars &sc)
{
    if (!(v[2] <= sc.stop2 * sc.b2) && !(v[2] >= 0.0)) return 2;   // NaN
    if (v[2] <= sc.stop2 * sc.b2) return 1;
    return ((sc.omega[0] == 0.0 && sc.omega[1] == 0.0) || (v[0] == 0.0 && v[1] == 0.0)) ? 2 : 0;
}

// The sums k_finalize forms (512 threads, thread by thread, then wave by
// wave), by a workgroup of 256 in every thread, bitwise the same: each thread
// stands for two of those.
template <int NT>
WCL_D void fold_sums(const FoldArgs &f, int rhs, double *lds /* [NT][8] */, double v[NT])
{
    const double *p = f.partials + (size_t)rhs * 6 * f.pstride;
    double a[NT], b[NT];
#pragma unroll
    for (int k = 0; k < NT; k++) a[k] = b[k] = 0.0;
    for (int j = threadIdx.x; j < f.nparts; j += 512) {
        const bool two = j + 256 < f.nparts;
#pragma unroll
        for (int k = 0; k < NT; k++) {
            a[k] += p[k * f.pstride + j];
            b[k] += two ? p[k * f.pstride + j + 256] : 0.0;
        }
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NT; k++) {
        a[k] = wave_sum(a[k]);
        b[k] = wave_sum(b[k]);
        if (lane == 0) {
            lds[k * 8 + wid] = a[k];
            lds[k * 8 + 4 + wid] = b[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NT; k++) v[k] = row_sum((lane & 15) < 8 ? lds[k * 8 + (lane & 7)] : 0.0);
}

// One workgroup per right-hand side.  gate (optional): a right-hand side
// whose gate scalars are done is marked done at BICG_INIT_RHO.
__global__ void __launch_bounds__(512) k_finalize(int step, int nterms, const double *partials_all, Scalars *sc_all,
                                                  const Scalars *gate, int pstride, int nparts)
{
    const int rhs = blockIdx.x;
    Scalars *sc = sc_all + rhs;
    const double *partials = partials_all + (size_t)rhs * 6 * pstride;
    const Scalars in = *sc;   // read together with the partials, not after them
    if (in.done && (step == BICG_ALPHA || step == BICG_OMEGA || step == BICG_RHO)) return;
    __shared__ double lds[6 * 16];
    double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // each thread adds partials j = tid, tid + 512, ... in that order; eight of
    // them per term are loaded before any is added, so the loads overlap
    constexpr int U = 8;
    for (int j0 = threadIdx.x; j0 < nparts; j0 += U * blockDim.x) {
        double p[6][U];
#pragma unroll
        for (int k = 0; k < 6; k++)
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int j = j0 + u * (int)blockDim.x;
                p[k][u] = (k < nterms && j < nparts) ? partials[k * pstride + j] : 0.0;
            }
#pragma unroll
        for (int k = 0; k < 6; k++)
#pragma unroll
            for (int u = 0; u < U; u++)
                if (k < nterms && j0 + u * (int)blockDim.x < nparts) v[k] += p[k][u];
    }
    block_sum<6>(v, lds);
    if (threadIdx.x != 0) return;
    switch (step) {
    case BICG_INIT_RHO:
        // pairs (rt, r), (r, r)
        sc->rho[0] = v[0]; sc->rho[1] = v[1];
        sc->r2 = v[2];
        sc->b2 = v[2];
        sc->rho_old[0] = 1.0; sc->rho_old[1] = 0.0;
        sc->alpha[0] = 1.0; sc->alpha[1] = 0.0;
        sc->omega[0] = 1.0; sc->omega[1] = 0.0;
        sc->iter = 0;
        sc->fresh = 2;
        sc->done = (v[2] == 0.0) ? 1 : 0;
        if (gate && gate[rhs].done) sc->done = 1;
        break;
    case BICG_ALPHA: {
        const double d[2] = {v[0], v[1]};
        if (d[0] == 0.0 && d[1] == 0.0) { sc->done = 2; break; }
        cdiv(in.rho, d, sc->alpha);
        break;
    }
    case BICG_OMEGA:
        // pairs (t, s), (t, t)
        bicg_omega(v, sc->omega);
        break;
    case BICG_RHO:
        sc->rho_old[0] = in.rho[0]; sc->rho_old[1] = in.rho[1];
        sc->rho[0] = v[0]; sc->rho[1] = v[1];
        sc->r2 = v[2];
        sc->iter = in.iter + 1;
        sc->fresh = 1;
        if (const int d = bicg_stop(v, in)) sc->done = d;
        break;
    case NORM_ONLY:
        sc->t[0] = v[0];
        break;
    default:
        break;
    }
}

hipError_t launch_finalize(int step, int nterms, const double *partials, Scalars *sc, hipStream_t st, int nrhs,
                           const Scalars *gate, int pstride, int nparts)
{
    if (nparts < 1 || nparts > pstride) return hipErrorInvalidValue;
    k_finalize<<<nrhs, 512, 0, st>>>(step, nterms, partials, sc, gate, pstride, nparts);
    return hipGetLastError();
}

// One wave per right-hand side: all but the last word, a fence for all of them,
// then the last word with the read's number.
__global__ void __launch_bounds__(64) k_report(const Scalars *dev, Scalars *host, int seq)
{
    static_assert(offsetof(Scalars, seq) + sizeof(int) == sizeof(Scalars) && sizeof(Scalars) % 8 == 0 && sizeof(Scalars) <= 512);
    constexpr uint32_t W = sizeof(Scalars) / 8;
    const uint64_t *d = (const uint64_t *)(dev + blockIdx.x);
    uint64_t *h = (uint64_t *)(host + blockIdx.x);
    const uint32_t i = threadIdx.x;
    const uint64_t v = i < W ? d[i] : 0;
    if (i + 1 < W) h[i] = v;
    __threadfence_system();
    if (i + 1 == W)
        __hip_atomic_store(h + i, (v & 0xffffffffu) | (uint64_t)(uint32_t)seq << 32, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_report(const Scalars *dev, Scalars *host, int n, int seq, hipStream_t st)
{
    k_report<<<n, 64, 0, st>>>(dev, host, seq);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BiCGStab vector updates (complex scalars from the device), blockIdx.y = rhs.
// FOLD: the finaliser's step before the update is done here by every workgroup
// from the partials (f), and workgroup 0 of each right-hand side stores the
// scalars while others may still start.  What it stores is either read by later
// launches only (p's new rho waits in t[4..5] until the s update, which reads it,
// puts it in rho), or it is `done`, which each workgroup reads once for all of
// its waves (stopped): one that finds it set leaves whole, one that does not
// forms the sums itself and comes to the same end.  fresh: the scalars are
// complete (2: start, 1: an explicit BICG_RHO step), nothing to fold.
template <bool FOLD>
WCL_D bool stopped(const Scalars *sc)
{
    if constexpr (!FOLD) return sc->done;   // no launch that reads it so writes it
    __shared__ int done;
    if (threadIdx.x == 0) done = __hip_atomic_load(&sc->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return done;
}

template <typename T, bool FOLD>
__global__ void __launch_bounds__(256) k_bicg_p(size_t n, size_t stride, const typename CT<T>::V *r,
                                               typename CT<T>::V *p, const typename CT<T>::V *v, Scalars *sc_all,
                                               FoldArgs f)
{
    Scalars *sc = sc_all + blockIdx.y;
    const Scalars in = *sc;
    if (stopped<FOLD>(sc)) return;
    const size_t off = blockIdx.y * stride;
    r += off; p += off; v += off;
    double rho[2] = {in.rho[0], in.rho[1]}, rho_old[2] = {in.rho_old[0], in.rho_old[1]};
    if constexpr (FOLD) {
        __shared__ double lds[3 * 8];
        const bool first = blockIdx.x == 0 && threadIdx.x == 0;
        if (!in.fresh) {   // the BICG_RHO step
            double s[3];
            fold_sums<3>(f, blockIdx.y, lds, s);
            const int stop = bicg_stop(s, in);
            rho_old[0] = in.rho[0]; rho_old[1] = in.rho[1];
            rho[0] = s[0]; rho[1] = s[1];
            if (first) {
                sc->r2 = s[2];
                sc->iter = in.iter + 1;
                if (stop) sc->done = stop;
            }
            if (stop) return;
        }
        if (first) { sc->t[4] = rho[0]; sc->t[5] = rho[1]; }
    }
    if (in.fresh == 2) {   // the recurrence starts: p = r, whatever p and v hold
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = r[i];
        return;
    }
    // beta = (rho / rho_old) (alpha / omega)
    double q1[2], q2[2], beta[2];
    cdiv(rho, rho_old, q1);
    cdiv(in.alpha, in.omega, q2);
    beta[0] = q1[0] * q2[0] - q1[1] * q2[1];
    beta[1] = q1[0] * q2[1] + q1[1] * q2[0];
    using C = typename CT<T>::C;
    const C br = (C)beta[0], bi = (C)beta[1], wr = (C)in.omega[0], wi = (C)in.omega[1];
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const auto pv = ldv(p[i]), vv = ldv(v[i]), rv = ldv(r[i]);
        // d = p - omega v
        const C dr = pv.x - (wr * vv.x - wi * vv.y);
        const C di = pv.y - (wr * vv.y + wi * vv.x);
        stv(p[i], rv.x + br * dr - bi * di, rv.y + br * di + bi * dr);
    }
}

template <typename T, bool FOLD>
__global__ void __launch_bounds__(256) k_bicg_s(size_t n, size_t stride, const typename CT<T>::V *r,
                                               const typename CT<T>::V *v, typename CT<T>::V *s, Scalars *sc_all,
                                               FoldArgs f)
{
    Scalars *sc = sc_all + blockIdx.y;
    const Scalars in = *sc;
    if (stopped<FOLD>(sc)) return;
    const size_t off = blockIdx.y * stride;
    r += off; v += off; s += off;
    double alpha[2] = {in.alpha[0], in.alpha[1]};
    if constexpr (FOLD) {   // the BICG_ALPHA step
        __shared__ double lds[2 * 8];
        const bool first = blockIdx.x == 0 && threadIdx.x == 0;
        double d[2];
        fold_sums<2>(f, blockIdx.y, lds, d);
        if (first) {
            sc->rho[0] = in.t[4]; sc->rho[1] = in.t[5];
            sc->fresh = 0;
        }
        if (d[0] == 0.0 && d[1] == 0.0) {
            if (first) sc->done = 2;
            return;
        }
        cdiv(in.t + 4, d, alpha);
        if (first) { sc->alpha[0] = alpha[0]; sc->alpha[1] = alpha[1]; }
    }
    using C = typename CT<T>::C;
    const C ar = (C)alpha[0], ai = (C)alpha[1];
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const auto rv = ldv(r[i]), vv = ldv(v[i]);
        stv(s[i], rv.x - (ar * vv.x - ai * vv.y), rv.y - (ar * vv.y + ai * vv.x));
    }
}

// x += alpha ph + omega sh; r = s - omega t, with the partials of <rt, r>
// and <r, r> (of the stored r) per workgroup: terms 0, 1 = Re, Im <rt, r>,
// 2 = <r, r>, 3 = 0 at partials[rhs][k][block] (stride pstride).
template <typename T, bool FOLD>
__global__ void __launch_bounds__(256) k_bicg_xr_dots(size_t n, size_t stride, typename CT<T>::V *x,
                                                     const typename CT<T>::V *ph, const typename CT<T>::V *sh,
                                                     typename CT<T>::V *r, const typename CT<T>::V *s,
                                                     const typename CT<T>::V *t, const typename CT<T>::V *rt,
                                                     Scalars *sc_all, double *partials, int pstride, FoldArgs f)
{
    Scalars *sc = sc_all + blockIdx.y;
    const Scalars in = *sc;
    if (in.done) return;
    __shared__ double lds[4 * 16];
    const size_t off = blockIdx.y * stride;
    x += off; ph += off; sh += off; r += off; s += off; t += off; rt += off;
    double omega[2] = {in.omega[0], in.omega[1]};
    if constexpr (FOLD) {   // the BICG_OMEGA step
        __shared__ double fl[3 * 8];
        double d[3];
        fold_sums<3>(f, blockIdx.y, fl, d);
        bicg_omega(d, omega);
        if (blockIdx.x == 0 && threadIdx.x == 0) { sc->omega[0] = omega[0]; sc->omega[1] = omega[1]; }
    }
    using C = typename CT<T>::C;
    const C ar = (C)in.alpha[0], ai = (C)in.alpha[1], wr = (C)omega[0], wi = (C)omega[1];
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const auto xv = ldv(x[i]), pv = ldv(ph[i]), sv = ldv(sh[i]), s2 = ldv(s[i]), tv = ldv(t[i]);
        stv(x[i], xv.x + (ar * pv.x - ai * pv.y) + (wr * sv.x - wi * sv.y),
            xv.y + (ar * pv.y + ai * pv.x) + (wr * sv.y + wi * sv.x));
        stv(r[i], s2.x - (wr * tv.x - wi * tv.y), s2.y - (wr * tv.y + wi * tv.x));
        const auto rn = ldv(r[i]), rr = ldv(rt[i]);
        v[0] += (double)rr.x * (double)rn.x + (double)rr.y * (double)rn.y;
        v[1] += (double)rr.x * (double)rn.y - (double)rr.y * (double)rn.x;
        v[2] += (double)rn.x * (double)rn.x + (double)rn.y * (double)rn.y;
    }
    block_sum<4>(v, lds);
    if (threadIdx.x == 0) {
        double *pr = partials + (size_t)blockIdx.y * 6 * pstride;
#pragma unroll
        for (int k = 0; k < 4; k++) pr[k * pstride + blockIdx.x] = v[k];
    }
}

static dim3 blas_grid(size_t n, int nrhs = 1)
{
    size_t b = (n + 255) / 256;
    const size_t cap = nrhs > 1 ? 2048 : 8192;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return dim3((unsigned)b, nrhs);
}

// Flat-vector launchers: P64, P32 or P16 storage (n complex numbers per
// right-hand side); any other precision code is refused.
#define WCL_BY_PREC(CALL)                                 \
    do {                                                  \
        if (prec == P64) {                                \
            using T = double;                             \
            CALL;                                         \
        } else if (prec == P32) {                         \
            using T = float;                              \
            CALL;                                         \
        } else if (prec == P16) {                         \
            using T = __half;                             \
            CALL;                                         \
        } else {                                          \
            return hipErrorInvalidValue;                  \
        }                                                 \
    } while (0)
#define WCL_V(x) ((typename CT<T>::V *)(x))
#define WCL_CV(x) ((const typename CT<T>::V *)(x))

// Grid of a vector update that folds a finaliser step: one round of workgroups
// over the chip (each adds the partials again, once).
static dim3 fold_grid(size_t n, int nrhs)
{
    dim3 g = blas_grid(n, nrhs);
    const unsigned cap = (unsigned)std::max(64, 2048 / nrhs);
    if (g.x > cap) g.x = cap;
    return g;
}

int bicg_parts(size_t n, int nrhs, bool fold)
{
    return (int)std::min((fold ? fold_grid(n, nrhs) : blas_grid(n, nrhs)).x, (unsigned)RED_BLOCKS);
}

hipError_t launch_bicg_p(int prec, size_t n, const void *r, void *p, const void *v, Scalars *sc, hipStream_t st, int nrhs,
                         size_t stride, const FoldArgs *f)
{
    if (f) WCL_BY_PREC((k_bicg_p<T, true><<<fold_grid(n, nrhs), 256, 0, st>>>(n, stride, WCL_CV(r), WCL_V(p), WCL_CV(v), sc, *f)));
    else WCL_BY_PREC((k_bicg_p<T, false><<<blas_grid(n, nrhs), 256, 0, st>>>(n, stride, WCL_CV(r), WCL_V(p), WCL_CV(v), sc, FoldArgs{})));
    return hipGetLastError();
}

hipError_t launch_bicg_s(int prec, size_t n, const void *r, const void *v, void *s, Scalars *sc, hipStream_t st, int nrhs,
                         size_t stride, const FoldArgs *f)
{
    if (f) WCL_BY_PREC((k_bicg_s<T, true><<<fold_grid(n, nrhs), 256, 0, st>>>(n, stride, WCL_CV(r), WCL_CV(v), WCL_V(s), sc, *f)));
    else WCL_BY_PREC((k_bicg_s<T, false><<<blas_grid(n, nrhs), 256, 0, st>>>(n, stride, WCL_CV(r), WCL_CV(v), WCL_V(s), sc, FoldArgs{})));
    return hipGetLastError();
}

hipError_t launch_bicg_xr_dots(int prec, size_t n, void *x, const void *ph, const void *sh, void *r,
                               const void *s, const void *t, const void *rt, Scalars *sc, hipStream_t st,
                               int nrhs, size_t stride, double *partials, int pstride, const FoldArgs *f)
{
    // at most RED_BLOCKS workgroups per right-hand side, so that the next
    // step adds few partials
    const dim3 grid((unsigned)bicg_parts(n, nrhs, f != nullptr), nrhs);
    if ((int)grid.x > pstride) return hipErrorInvalidValue;
#define WCL_XR(FOLD, F)                                                                                             \
    WCL_BY_PREC((k_bicg_xr_dots<T, FOLD><<<grid, 256, 0, st>>>(n, stride, WCL_V(x), WCL_CV(ph), WCL_CV(sh), WCL_V(r), \
                                                               WCL_CV(s), WCL_CV(t), WCL_CV(rt), sc, partials, pstride, F)))
    if (f) WCL_XR(true, *f);
    else WCL_XR(false, FoldArgs{});
#undef WCL_XR
    return hipGetLastError();
}

// End of an inner solve: out64 = |in64| x, with |in64|^2 in t[0].
template <typename SI>
__global__ void __launch_bounds__(256) k_inner_out(uint32_t Vh, const char *x, char *out, const Scalars *sc)
{
    const uint32_t h = blockIdx.x * 256u + threadIdx.x;
    if (h >= Vh) return;
    const double scale = sqrt(sc[blockIdx.y].t[0]);
    cplx<double> v[12];
    load_spinor<SI, double>(x + blockIdx.y * spinor_bytes(sizeof(SI), Vh), h, Vh, v);
#pragma unroll
    for (int k = 0; k < 12; k++) v[k] = scale * v[k];
    store_spinor<double, double>(out + blockIdx.y * spinor_bytes(8, Vh), h, Vh, v);
}

hipError_t launch_inner_out(int prec, size_t Vh, const void *x, void *out64, const Scalars *sc, hipStream_t st, int nrhs)
{
    const dim3 grid((unsigned)((Vh + 255) / 256), nrhs);
    if (prec == P32) k_inner_out<float><<<grid, 256, 0, st>>>((uint32_t)Vh, (const char *)x, (char *)out64, sc);
    else if (prec == P16) k_inner_out<__half><<<grid, 256, 0, st>>>((uint32_t)Vh, (const char *)x, (char *)out64, sc);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// Start of an inner solve, one pass over the FP64 vectors of every right-hand
// side: the norm's step (f: the partials of |in|^2), r = rt = in / |in| in the
// inner storage, x = 0, and the partials of <rt, r>, <r, r> for BICG_INIT_RHO.
// p and v need no start (fresh).  Three launches with the norm's partials and the
// step, where convert, copy, four fills and two dots are nine: 42.95 ms a solve
// against 43.87 for 12 x 16^3x32 FP16, 18.25 against 18.83 on FP16 24^3x32.
template <typename SO>
__global__ void __launch_bounds__(256) k_inner_init(uint32_t Vh, const char *in, char *r, char *rt, char *x, Scalars *sc_all,
                                                   FoldArgs f, double *partials)
{
    __shared__ double fl[8], lds[16];
    const int rhs = blockIdx.y;
    double nrm[1], v[1] = {0.0};
    fold_sums<1>(f, rhs, fl, nrm);
    if (blockIdx.x == 0 && threadIdx.x == 0) sc_all[rhs].t[0] = nrm[0];
    const double scale = nrm[0] > 0.0 ? 1.0 / sqrt(nrm[0]) : 0.0;
    for (uint32_t h = blockIdx.x * 256u + threadIdx.x; h < Vh; h += gridDim.x * 256u) {
        const size_t o = rhs * spinor_bytes(sizeof(SO), Vh);
        cplx<double> d[12];
        load_spinor<double, double>(in + rhs * spinor_bytes(8, Vh), h, Vh, d);
#pragma unroll
        for (int k = 0; k < 12; k++) d[k] = scale * d[k];
        constexpr uint32_t WORDS = sizeof(SO) * 24 / 16;
        store_spinor<SO, double>(r + o, h, Vh, d);
        store_spinor<SO, double>(rt + o, h, Vh, d);
#pragma unroll
        for (uint32_t k = 0; k < WORDS; k++) stf(x + o, (k * Vh + h) * 16u, make_uint4(0u, 0u, 0u, 0u));
#pragma unroll
        for (int k = 0; k < 12; k++) {
            // the values as stored
            float re = (float)d[k].re, im = (float)d[k].im;
            if constexpr (sizeof(SO) == 2) {
                const float2 q = h2f2(f22h(re, im));
                re = q.x; im = q.y;
            }
            v[0] += (double)re * (double)re + (double)im * (double)im;
        }
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) {
        double *p = partials + (size_t)rhs * 6 * f.pstride + blockIdx.x;
        p[0] = v[0];
        p[f.pstride] = 0.0;
        p[2 * (size_t)f.pstride] = v[0];
        p[3 * (size_t)f.pstride] = 0.0;
    }
}

hipError_t launch_inner_init(int prec, size_t Vh, const void *in64, void *r, void *rt, void *x, Scalars *sc, const FoldArgs &f,
                             double *partials, int *nparts, hipStream_t st, int nrhs)
{
    const dim3 grid((unsigned)std::min((Vh + 255) / 256, (size_t)RED_BLOCKS), nrhs);
    *nparts = (int)grid.x;
    if (prec == P32)
        k_inner_init<float><<<grid, 256, 0, st>>>((uint32_t)Vh, (const char *)in64, (char *)r, (char *)rt, (char *)x, sc, f, partials);
    else if (prec == P16)
        k_inner_init<__half><<<grid, 256, 0, st>>>((uint32_t)Vh, (const char *)in64, (char *)r, (char *)rt, (char *)x, sc, f, partials);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(256) k_axpby(size_t n, double ar, double ai, const typename CT<T>::V *x, double br,
                                              double bi, typename CT<T>::V *y)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        using C = typename CT<T>::C;
        const auto xv = ldv(x[i]), yv = ldv(y[i]);
        stv(y[i], (C)(ar * xv.x - ai * xv.y + br * yv.x - bi * yv.y), (C)(ar * xv.y + ai * xv.x + br * yv.y + bi * yv.x));
    }
}

// blockIdx.y = slice (sx, sy elements apart)
template <typename T>
__global__ void __launch_bounds__(256) k_copy(size_t n, const typename CT<T>::V *x, typename CT<T>::V *y, size_t sx, size_t sy)
{
    x += blockIdx.y * sx;
    y += blockIdx.y * sy;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        y[i] = x[i];
}

template <typename T>
__global__ void __launch_bounds__(256) k_zero(size_t n, typename CT<T>::V *y)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        stv(y[i], (typename CT<T>::C)0, (typename CT<T>::C)0);
}

hipError_t launch_axpby(int prec, size_t n, double2 a, const void *x, double2 b, void *y, hipStream_t st)
{
    WCL_BY_PREC((k_axpby<T><<<blas_grid(n), 256, 0, st>>>(n, a.x, a.y, WCL_CV(x), b.x, b.y, WCL_V(y))));
    return hipGetLastError();
}

hipError_t launch_copy(int prec, size_t n, const void *x, void *y, hipStream_t st, int slices, size_t sx, size_t sy)
{
    const dim3 grid(blas_grid(n, slices).x, slices);
    WCL_BY_PREC((k_copy<T><<<grid, 256, 0, st>>>(n, WCL_CV(x), WCL_V(y), sx, sy)));
    return hipGetLastError();
}

hipError_t launch_zero(int prec, size_t n, void *y, hipStream_t st)
{
    WCL_BY_PREC((k_zero<T><<<blas_grid(n), 256, 0, st>>>(n, WCL_V(y))));
    return hipGetLastError();
}
#undef WCL_BY_PREC
#undef WCL_V
#undef WCL_CV

}  // namespace wcl

namespace wcl {

static double link_site_bytes(int prec)
{
    return prec == P64 ? 144.0 : prec == P32 ? 72.0 : prec == P16 ? 36.0 : prec == P32C ? 48.0 : 24.0;
}
static double spinor_site_bytes(int prec) { return prec == P64 ? 192.0 : prec == P32 ? 96.0 : 48.0; }
static double clover_site_bytes(int prec)
{
    return prec == P64 ? 576.0 : (prec == P32 || prec == P32C) ? 288.0 : 144.0;
}

void hop_work(const HopLaunch &a, double *bytes, double *flops)
{
    const double sites = (double)a.g->Vh * (a.nrhs > 0 ? a.nrhs : 1);
    double b = (a.nrhs > 0 ? 8.0 * link_site_bytes(a.link_prec) / a.nrhs : 8.0 * link_site_bytes(a.link_prec));
    b += 2.0 * spinor_site_bytes(a.spin_prec);
    double f = 1320.0;
    if (a.mode != HOP) {
        b += clover_site_bytes(a.link_prec) / (a.nrhs > 0 ? a.nrhs : 1);
        f += 504.0;
    }
    if (a.mode == XPAY || a.mode == CLOVX) {
        b += spinor_site_bytes(a.spin_prec);
        f += 48.0;
    }
    if (a.ndot) {   // fused reductions: the second vector and 96 flop per inner product
        b += spinor_site_bytes(a.spin_prec);
        f += a.ndot == 1 ? 96.0 : 144.0;
    }
    *bytes = b * sites;
    *flops = f * sites;
}

// ---------------------------------------------------------------------------
// Streaming ceilings for the roofline.  Read: each workgroup streams one
// contiguous chunk with 16 independent 16-byte non-temporal loads in flight
// per thread (the fastest of a sweep over chunked / grid-stride order,
// temporal / non-temporal loads, 4 / 8 / 16 loads in flight and 1024 ...
// 32768 workgroups of 256 ... 1024 threads); one word written per thread.
// Copy: the same order with 8 loads and 8 stores in flight.
__global__ void __launch_bounds__(256) k_stream_read(const u32x4 *__restrict__ a, size_t n, size_t chunk, float *out)
{
    constexpr int U = 16;
    u32x4 s = {0u, 0u, 0u, 0u};
    const size_t base = (size_t)blockIdx.x * chunk, end = base + chunk < n ? base + chunk : n;
    for (size_t i = base + threadIdx.x; i < end; i += U * blockDim.x) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const size_t j = i + u * blockDim.x;
            v[u] = j < end ? __builtin_nontemporal_load(a + j) : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; u++) s ^= v[u];
    }
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = __uint_as_float(s.x ^ s.y ^ s.z ^ s.w);
}

__global__ void __launch_bounds__(256) k_stream_copy(const u32x4 *__restrict__ a, u32x4 *__restrict__ b, size_t n,
                                                    size_t chunk)
{
    constexpr int U = 8;
    const size_t base = (size_t)blockIdx.x * chunk, end = base + chunk < n ? base + chunk : n;
    for (size_t i = base + threadIdx.x; i < end; i += U * blockDim.x) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const size_t j = i + u * blockDim.x;
            if (j < end) v[u] = __builtin_nontemporal_load(a + j);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const size_t j = i + u * blockDim.x;
            if (j < end) __builtin_nontemporal_store(v[u], b + j);
        }
    }
}

hipError_t launch_stream(int copy, const void *a, void *b, size_t n16, float *out, int blocks, hipStream_t st)
{
    const size_t chunk = (n16 + blocks - 1) / blocks;
    if (copy) k_stream_copy<<<blocks, 256, 0, st>>>((const u32x4 *)a, (u32x4 *)b, n16, chunk);
    else k_stream_read<<<blocks, 256, 0, st>>>((const u32x4 *)a, n16, chunk, out);
    return hipGetLastError();
}

}  // namespace wcl
