// hop_dev.h -- device code of the even/odd hopping kernel, shared by the
// per-launch kernel (k_hop) and the persistent inner solver.
#pragma once

#include "wcl_launch.h"

namespace wcl {

// ---------------------------------------------------------------------------
// The hopping kernel.  One thread per output site of parity p; per direction
// the neighbour spinor is projected to a half spinor (12 flop), rotated by
// the link or its adjoint (132 flop) and accumulated with the sign pattern of
// the projector (24 flop): 1320 flop per site over the 8 directions.
struct HopArgs {
    Geom g;
    const void *in;
    void *out;
    const void *links;
    const void *clov;
    const void *x;
    double coef;
    size_t in_stride, out_stride, x_stride;  // bytes between right-hand sides
    int p;
    int xcd;
    int nrhs;
    const Scalars *sc;   // per right-hand side
    int tpw;             // consecutive site blocks per workgroup (k_hop)
};

// The 8 hops of a site run as a two-stage pipeline: the neighbour spinor and
// link of hop k+1 are in flight while hop k is computed; a scheduling barrier
// after each hop keeps the compiler from hoisting further loads (which would
// raise the register count and lower the occupancy).
// The neighbour spinor stays as loaded too where it is FP16: 12 registers, and
// the projection reads the halves directly (project_raw): 16% fewer vector
// instructions, 12 sources at 16^3x32 in the FP16 tier 45.7 -> 44.0 ms a solve.
template <typename SS, typename R>
struct SpinRaw {
    cplx<R> psi[12];
};
template <typename R>
struct SpinRaw<__half, R> {
    uint32_t w[12];   // complex i: re in the low half, im in the high one
};
template <typename SL, typename SS, typename R>
struct HopStage {
    SpinRaw<SS, R> psi;
    LinkRaw<SL> u;   // as loaded; decoded when the hop is computed
    R sign;
};

template <typename SS, typename R>
WCL_D void load_spinor_raw(const void *base, uint32_t h, uint32_t Vh, SpinRaw<SS, R> &r)
{
    if constexpr (sizeof(SS) == 2) {
#pragma unroll
        for (uint32_t k = 0; k < 3; k++) {
            const uint4 u = ldf<uint4>(base, (k * Vh + h) * 16u);
            r.w[4 * k] = u.x; r.w[4 * k + 1] = u.y; r.w[4 * k + 2] = u.z; r.w[4 * k + 3] = u.w;
        }
    } else {
        load_spinor<SS, R>(base, h, Vh, r.psi);
    }
}

// Spins 2 half, 2 half + 1 of an FP64 or FP32 spinor.
template <typename SS, typename R>
WCL_D void load_spinor_half(const void *base, uint32_t h, uint32_t Vh, int half, cplx<R> v[6])
{
    if constexpr (sizeof(SS) == 8) {
#pragma unroll
        for (uint32_t i = 0; i < 6; i++) {
            const double2 d = ldf<double2>(base, ((6 * half + i) * Vh + h) * 16u);
            v[i] = {(R)d.x, (R)d.y};
        }
    } else {
#pragma unroll
        for (uint32_t k = 0; k < 3; k++) {
            const float4 f = ldf<float4>(base, ((3 * half + k) * Vh + h) * 16u);
            v[2 * k] = {(R)f.x, (R)f.y};
            v[2 * k + 1] = {(R)f.z, (R)f.w};
        }
    }
}

// up + lo of two FP16 numbers in FP32 (UH, LH: the high half; NEG: up - lo):
// the conversions of both and the addition in one instruction, rounded once as
// the FP32 addition is (the product with 1 is exact).
template <int UH, int LH, bool NEG>
WCL_D float half_add(uint32_t up, uint32_t lo)
{
    float d;
    if constexpr (UH == 0 && LH == 0 && !NEG) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else if constexpr (UH == 0 && LH == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else if constexpr (UH == 0 && !NEG) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else if constexpr (UH == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else if constexpr (LH == 0 && !NEG) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else if constexpr (LH == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else if constexpr (!NEG) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(up), "v"(lo));
    return d;
}

// up + i^CODE lo
template <int CODE>
WCL_D cplx<float> half_add_unit(uint32_t up, uint32_t lo)
{
    if constexpr ((CODE & 3) == 0) return {half_add<0, 0, false>(up, lo), half_add<1, 1, false>(up, lo)};
    else if constexpr ((CODE & 3) == 1) return {half_add<0, 1, true>(up, lo), half_add<1, 0, false>(up, lo)};
    else if constexpr ((CODE & 3) == 2) return {half_add<0, 0, true>(up, lo), half_add<1, 1, true>(up, lo)};
    else return {half_add<0, 1, false>(up, lo), half_add<1, 0, true>(up, lo)};
}

// project of a spinor as loaded
template <int MU, int S, typename SS, typename R>
WCL_D void project_raw(const SpinRaw<SS, R> &r, cplx<R> h[6])
{
    if constexpr (sizeof(SS) == 2) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            h[c] = half_add_unit<gcode(MU, 0) + (S < 0 ? 2 : 0)>(r.w[c], r.w[(2 + gcol(MU, 0)) * 3 + c]);
            h[3 + c] = half_add_unit<gcode(MU, 1) + (S < 0 ? 2 : 0)>(r.w[3 + c], r.w[(2 + gcol(MU, 1)) * 3 + c]);
        }
    } else {
        project<MU, S, R>(r.psi, h);
    }
}

// hop K: direction MU = K/2, forward (K even) or backward (K odd)
// The load offsets of hop K pass through an empty asm that also "rewrites"
// the accumulator: the loads of hop K then wait for the complete compute of
// hop K-2, so at most two hops' operands are live at a time (no instruction
// is emitted for the fence itself).
template <typename R>
WCL_D void pipeline_fence(cplx<R> acc[12], uint32_t &hn, uint32_t &h)
{
    asm volatile(""
                 : "+v"(acc[0].re), "+v"(acc[0].im), "+v"(acc[1].re), "+v"(acc[1].im), "+v"(acc[2].re),
                   "+v"(acc[2].im), "+v"(acc[3].re), "+v"(acc[3].im), "+v"(acc[4].re), "+v"(acc[4].im),
                   "+v"(acc[5].re), "+v"(acc[5].im), "+v"(acc[6].re), "+v"(acc[6].im), "+v"(acc[7].re),
                   "+v"(acc[7].im), "+v"(acc[8].re), "+v"(acc[8].im), "+v"(acc[9].re), "+v"(acc[9].im),
                   "+v"(acc[10].re), "+v"(acc[10].im), "+v"(acc[11].re), "+v"(acc[11].im), "+v"(hn), "+v"(h));
}

// Staged input: a workgroup first copies the input spinors of its own NS
// consecutive half-sites (its tile, or a part or pair of tiles) into LDS; a
// neighbour inside that range is then read from LDS, one outside it from
// global memory.  In the blocked layout most neighbours of a tile lie in it.
typedef const __attribute__((address_space(3))) u32x4 *lds_u4p;
struct LdsIn {
    lds_u4p s;       // uint4 [words][NS]
    uint32_t base;   // first half index of the tile
};

// A spinor from the LDS copy of the tile (same word layout as the field).
template <typename SS, int NS, typename R>
WCL_D void lds_spinor(lds_u4p s, uint32_t l, SpinRaw<SS, R> &r)
{
    if constexpr (sizeof(SS) == 8) {
#pragma unroll
        for (uint32_t i = 0; i < 12; i++) {
            const u32x4 u = s[i * NS + l];
            r.psi[i] = {(R)__hiloint2double(u.y, u.x), (R)__hiloint2double(u.w, u.z)};
        }
    } else if constexpr (sizeof(SS) == 4) {
#pragma unroll
        for (uint32_t k = 0; k < 6; k++) {
            const u32x4 u = s[k * NS + l];
            r.psi[2 * k] = {(R)__uint_as_float(u.x), (R)__uint_as_float(u.y)};
            r.psi[2 * k + 1] = {(R)__uint_as_float(u.z), (R)__uint_as_float(u.w)};
        }
    } else {
#pragma unroll
        for (uint32_t k = 0; k < 3; k++) {
            const u32x4 u = s[k * NS + l];
            r.w[4 * k] = u.x; r.w[4 * k + 1] = u.y; r.w[4 * k + 2] = u.z; r.w[4 * k + 3] = u.w;
        }
    }
}

template <typename SL, typename SS, int K, bool NT, int NS, typename R>
WCL_D void hop_load(const HopArgs &a, const Site &s, uint32_t h0, const char *in, const LdsIn &li,
                    HopStage<SL, SS, R> &st, cplx<R> acc[12])
{
    constexpr int MU = K >> 1;
    constexpr bool FWD = (K & 1) == 0;
    const Geom &g = a.g;
    const uint32_t Vh = g.Vh;
    uint32_t hn = (uint32_t)neighbour(g, s, MU, FWD ? +1 : -1);
    uint32_t h = h0;
    pipeline_fence(acc, hn, h);
    if constexpr (NS > 0) {
        const uint32_t l = hn - li.base;
        if (l < (uint32_t)NS) lds_spinor<SS, NS, R>(li.s, l, st.psi);
        else load_spinor_raw<SS, R>(in, hn, Vh, st.psi);
    } else {
        load_spinor_raw<SS, R>(in, hn, Vh, st.psi);
    }
    if (FWD) load_link_raw<SL, NT>(a.links, MU, a.p, h, Vh, st.u);
    else load_link_raw<SL, NT>(a.links, MU, 1 - a.p, hn, Vh, st.u);
    st.sign = R(1);
    if (MU == 3 && g.tbc < 0 && s.x[3] == (FWD ? g.L[3] - 1 : 0)) st.sign = R(-1);
}

// forward: (1 - SG g_mu) U_mu(x) psi(x+mu);  backward: (1 + SG g_mu) U_mu(x-mu)^dag psi(x-mu)
template <int K, int SG, typename SL, typename SS, typename R>
WCL_D void hop_compute(const HopStage<SL, SS, R> &st, cplx<R> acc[12])
{
    constexpr int MU = K >> 1;
    constexpr bool FWD = (K & 1) == 0;
    constexpr int S = FWD ? -SG : SG;
    cplx<R> hh[6], uh[6], u[9];
    project_raw<MU, S, SS, R>(st.psi, hh);
#pragma unroll
    for (int k = 0; k < 6; k++) hh[k] = st.sign * hh[k];
    expand_link<SL, R>(st.u, u);
    if (FWD) su3_mul(u, hh, uh);
    else su3_dag_mul(u, hh, uh);
    accumulate<MU, S, R>(acc, uh);
}

template <typename SL, typename SS, int D, int K, bool NT, int NS, typename R>
WCL_D void hop_prologue(const HopArgs &a, const Site &s, uint32_t h, const char *in, const LdsIn &li,
                        HopStage<SL, SS, R> st[D], cplx<R> acc[12])
{
    if constexpr (K < D - 1) {
        hop_load<SL, SS, K, NT, NS, R>(a, s, h, in, li, st[K], acc);
        hop_prologue<SL, SS, D, K + 1, NT, NS, R>(a, s, h, in, li, st, acc);
    }
}

// hop K is computed while the operands of hop K + D - 1 are in flight
template <typename SL, typename SS, int D, int K, bool NT, int NS, typename R>
WCL_D void hop_pipeline(const HopArgs &a, const Site &s, uint32_t h, const char *in, const LdsIn &li,
                        HopStage<SL, SS, R> st[D], cplx<R> acc[12])
{
    if constexpr (K < 8) {
        if constexpr (K + D - 1 < 8)
            hop_load<SL, SS, K + D - 1, NT, NS, R>(a, s, h, in, li, st[(K + D - 1) % D], acc);
        hop_compute<K, 1, SL, SS, R>(st[K % D], acc);
        hop_pipeline<SL, SS, D, K + 1, NT, NS, R>(a, s, h, in, li, st, acc);
    }
}

// The hop with MODE's epilogue on the half-sites [bid * blockDim.x, +
// blockDim.x) of one right-hand side.  Every thread of the workgroup must
// call it (the staged variant, NS == blockDim.x, fills `sin` and waits on a
// workgroup barrier).  NDOT > 0: the thread's output o at its site enters
// dot[0..1] += <w, o> (w a field of the output parity, same storage), and
// with NDOT == 2 dot[2] += |o|^2, accumulated in FP64 (zero for sites past
// the lattice).
template <typename SL, typename SS, int MODE, int DEPTH, bool NT, int NS, int NDOT = 0>
WCL_D void hop_block(const HopArgs &a, int bid, int rhs, uint4 *sin, const void *dotw = nullptr,
                     double *dot = nullptr)
{
    using R = typename Real<SL>::T;
    const unsigned tid = tid_here();
    const int h = bid * blockDim.x + tid;
    const char *in = (const char *)a.in + rhs * a.in_stride;
    constexpr int NWORDS = (int)sizeof(SS) * 24 / 16;   // 16-byte words per input spinor
    LdsIn li{(lds_u4p)sin, 0u};
    if constexpr (NS > 0) {
        // blockDim.x == NS: thread t stages half-site base + t
        li.base = (uint32_t)(bid * NS);
        if (h < a.g.Vh) {
#pragma unroll
            for (int k = 0; k < NWORDS; k++)
                sin[k * NS + tid] = ldf<uint4>(in, ((uint32_t)k * (uint32_t)a.g.Vh + (uint32_t)h) * 16u);
        }
        __syncthreads();
    }
    if (h >= a.g.Vh) return;
    const size_t Vh = a.g.Vh;
    char *out = (char *)a.out + rhs * a.out_stride;
    const Site s = decompose(a.g, h, a.p);
    cplx<R> acc[12];
#pragma unroll
    for (int i = 0; i < 12; i++) acc[i] = {R(0), R(0)};
    HopStage<SL, SS, R> st[DEPTH];
    hop_prologue<SL, SS, DEPTH, 0, NT, NS, R>(a, s, h, in, li, st, acc);
    hop_pipeline<SL, SS, DEPTH, 0, NT, NS, R>(a, s, h, in, li, st, acc);

    cplx<R> o[12];
    if constexpr (MODE == HOP) {
#pragma unroll
        for (int i = 0; i < 12; i++) o[i] = acc[i];
    } else {
        // one chirality block at a time: 36 clover reals live, not 72 (FP64 kernels
        // then fit 256 registers, two waves per SIMD, FP32 ones mostly 128)
        cplx<R> xv[12];
        const char *x = (const char *)a.x + rhs * a.x_stride;
        const R cf = (R)a.coef;
#pragma unroll
        for (int half = 0; half < 2; half++) {
            const uint32_t hc = (uint32_t)h;
            R c[36];
            load_clover_half<typename ClovS<SL>::T, R, NT>(a.clov, a.p, hc, (uint32_t)Vh, half, c);
            if constexpr (MODE != CLOV_H) {
                if constexpr (sizeof(SS) != 2) load_spinor_half<SS, R>(x, hc, (uint32_t)Vh, half, xv + 6 * half);
                else if (half == 0) load_spinor<SS, R>(x, hc, (uint32_t)Vh, xv);   // 1.5 words a half
            }
            cplx<R> *oh = o + 6 * half;
            const cplx<R> *ah = acc + 6 * half, *xh = xv + 6 * half;
            if constexpr (MODE == CLOV_H) {
                clover_mul_half(c, ah, oh);
            } else if constexpr (MODE == XPAY) {
                cplx<R> t[6];
                clover_mul_half(c, ah, t);
#pragma unroll
                for (int i = 0; i < 6; i++) oh[i] = {fmar(cf, t[i].re, xh[i].re), fmar(cf, t[i].im, xh[i].im)};
            } else {
                clover_mul_half(c, xh, oh);
#pragma unroll
                for (int i = 0; i < 6; i++) oh[i] = {fmar(cf, ah[i].re, oh[i].re), fmar(cf, ah[i].im, oh[i].im)};
            }
        }
    }
    store_spinor<SS, R>(out, h, Vh, o);
    if constexpr (NDOT > 0) {
        // the dot products see the stored values (FP16 storage rounds them)
        cplx<R> ov[12], wv[12];
        if constexpr (sizeof(SS) == 2) load_spinor<SS, R>(out, h, Vh, ov);
        else {
#pragma unroll
            for (int i = 0; i < 12; i++) ov[i] = o[i];
        }
        load_spinor<SS, R>((const char *)dotw + rhs * a.out_stride, h, Vh, wv);
#pragma unroll
        for (int i = 0; i < 12; i++) {
            const double wr = wv[i].re, wi = wv[i].im, xr = ov[i].re, xi = ov[i].im;
            dot[0] += wr * xr + wi * xi;
            dot[1] += wr * xi - wi * xr;
            if constexpr (NDOT == 2) dot[2] += xr * xr + xi * xi;
        }
    }
}

struct HopLaunch;
// The XPAY hop with fused reductions (HopLaunch::ndot), grid and block as for
// k_hop with one right-hand side per workgroup.
hipError_t launch_hop_dot(const HopLaunch &L, const HopArgs &a, dim3 grid, dim3 block, hipStream_t st);

}  // namespace wcl
