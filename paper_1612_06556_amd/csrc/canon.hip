// canon.hip -- operators and layout conversions on the caller's canonical
// complex128 spinors.
//
// The half index h of the blocked layout enumerates pairs of x-neighbours:
// the even and the odd site with one h are x = 2j and 2j + 1 of one row, 384
// contiguous bytes of a canonical spinor.  A workgroup here takes NP
// consecutive pairs (both parities), so that its canonical reads and writes
// are runs of 384 bytes or more (768 with 4-wide tiles) and its link and
// clover reads are runs of NP sites; the transposition between the two orders
// goes through LDS.
#include "hop_dev.h"

namespace wcl {

namespace {

constexpr uint32_t CUT = 0x80000000u;   // no LDS slot; beyond every buffer resource

// NP pairs of canonical sites in the storage SS of a tier: component-major
// 16-byte words, slot = parity * NP + pair.  The stride is odd in 16-byte
// units, so neither order of access stays on one set of banks.
template <typename SS, int NP>
struct PairLds {
    static constexpr int WORDS = (int)sizeof(SS) * 24 / 16;
    static constexpr int STRIDE = 2 * NP + 1;
    uint4 w[WORDS * STRIDE];
    uint32_t base[NP];   // canonical index of the pair's x-even site | its parity << 31
};

// One complex number in the storage of a tier: rounded as the tier's fields
// are (FP16 from the FP32 value).
template <typename SS>
WCL_D void put_component(uint4 *w, int stride, int slot, int c, double2 v)
{
    if constexpr (sizeof(SS) == 8) {
        reinterpret_cast<double2 *>(w)[c * stride + slot] = v;
    } else if constexpr (sizeof(SS) == 4) {
        reinterpret_cast<float2 *>(w)[((c >> 1) * stride + slot) * 2 + (c & 1)] = make_float2((float)v.x, (float)v.y);
    } else {
        reinterpret_cast<uint32_t *>(w)[((c >> 2) * stride + slot) * 4 + (c & 3)] = f22h((float)v.x, (float)v.y);
    }
}

template <typename SS>
WCL_D double2 get_component(const uint4 *w, int stride, int slot, int c)
{
    if constexpr (sizeof(SS) == 8) {
        return reinterpret_cast<const double2 *>(w)[c * stride + slot];
    } else if constexpr (sizeof(SS) == 4) {
        const float2 f = reinterpret_cast<const float2 *>(w)[((c >> 1) * stride + slot) * 2 + (c & 1)];
        return make_double2((double)f.x, (double)f.y);
    } else {
        const float2 f = h2f2(reinterpret_cast<const uint32_t *>(w)[((c >> 2) * stride + slot) * 4 + (c & 3)]);
        return make_double2((double)f.x, (double)f.y);
    }
}

// The spinor in one slot.
template <typename SS, typename R>
WCL_D void get_spinor(const uint4 *w, int stride, int slot, cplx<R> v[12])
{
    if constexpr (sizeof(SS) == 8) {
#pragma unroll
        for (int i = 0; i < 12; i++) {
            const double2 d = reinterpret_cast<const double2 *>(w)[i * stride + slot];
            v[i] = {(R)d.x, (R)d.y};
        }
    } else if constexpr (sizeof(SS) == 4) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const uint4 u = w[k * stride + slot];
            v[2 * k] = {(R)__uint_as_float(u.x), (R)__uint_as_float(u.y)};
            v[2 * k + 1] = {(R)__uint_as_float(u.z), (R)__uint_as_float(u.w)};
        }
    } else {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const uint4 u = w[k * stride + slot];
            const float2 a = h2f2(u.x), b = h2f2(u.y), c = h2f2(u.z), d = h2f2(u.w);
            v[4 * k + 0] = {(R)a.x, (R)a.y};
            v[4 * k + 1] = {(R)b.x, (R)b.y};
            v[4 * k + 2] = {(R)c.x, (R)c.y};
            v[4 * k + 3] = {(R)d.x, (R)d.y};
        }
    }
}

template <typename SS, typename R>
WCL_D void put_spinor(uint4 *w, int stride, int slot, const cplx<R> v[12])
{
    if constexpr (sizeof(SS) == 8) {
#pragma unroll
        for (int i = 0; i < 12; i++) reinterpret_cast<double2 *>(w)[i * stride + slot] = make_double2(v[i].re, v[i].im);
    } else if constexpr (sizeof(SS) == 4) {
#pragma unroll
        for (int k = 0; k < 6; k++)
            reinterpret_cast<float4 *>(w)[k * stride + slot] =
                make_float4((float)v[2 * k].re, (float)v[2 * k].im, (float)v[2 * k + 1].re, (float)v[2 * k + 1].im);
    } else {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            uint4 u;
            u.x = f22h((float)v[4 * k].re, (float)v[4 * k].im);
            u.y = f22h((float)v[4 * k + 1].re, (float)v[4 * k + 1].im);
            u.z = f22h((float)v[4 * k + 2].re, (float)v[4 * k + 2].im);
            u.w = f22h((float)v[4 * k + 3].re, (float)v[4 * k + 3].im);
            w[k * stride + slot] = u;
        }
    }
}

// Canonical pairs [h0, h0 + np) into LDS (all threads; the caller's barrier
// follows).  PAR: 2 both parities, 0 the even sites only.
template <typename SS, int NP, int PAR>
WCL_D void stage_pairs(PairLds<SS, NP> &L, const Geom &g, uint32_t h0, uint32_t np, const double2 *canon)
{
    const uint32_t tid = threadIdx.x;
    if (tid < np) L.base[tid] = pair_base(g, (int)(h0 + tid));
    __syncthreads();
    constexpr uint32_t W = PAR == 2 ? 24 : 12;   // complex numbers of a pair
    constexpr int ITER = NP * (int)W / (2 * NP);
    double2 v[ITER];
    // every load in flight before the first is used
#pragma unroll
    for (int j = 0; j < ITER; j++) {
        const uint32_t i = (uint32_t)j * (2u * NP) + tid, pr = i / W, c = i - pr * W;
        if (pr < np) {
            const uint32_t b = L.base[pr];
            const uint32_t xo = PAR == 2 ? 0u : (b >> 31);   // x offset of the even site
            v[j] = canon[(size_t)((b & 0x7fffffffu) + xo) * 12 + c];
        }
    }
#pragma unroll
    for (int j = 0; j < ITER; j++) {
        const uint32_t i = (uint32_t)j * (2u * NP) + tid, pr = i / W, c = i - pr * W;
        if (pr < np) {
            const uint32_t xo = c >= 12u ? 1u : 0u;
            const uint32_t p = PAR == 2 ? ((xo + (L.base[pr] >> 31)) & 1u) : 0u;
            put_component<SS>(L.w, PairLds<SS, NP>::STRIDE, (int)(p * NP + pr), (int)(c - 12u * xo), v[j]);
        }
    }
}

// LDS slots to the canonical pairs by T threads; ODD0: the odd sites are
// written as zero.
template <typename SS, int NP, bool ODD0, int T = 2 * NP>
WCL_D void write_pairs(const PairLds<SS, NP> &L, uint32_t np, double2 *canon)
{
    const uint32_t tid = threadIdx.x;
#pragma unroll 4
    for (uint32_t i = tid; i < 24u * NP; i += (uint32_t)T) {
        const uint32_t pr = i / 24u, c = i - pr * 24u;
        if (pr >= np) break;
        const uint32_t b = L.base[pr];
        const uint32_t xo = c >= 12u ? 1u : 0u, p = (xo + (b >> 31)) & 1u;
        double2 v = make_double2(0.0, 0.0);
        if (!ODD0 || p == 0) v = get_component<SS>(L.w, PairLds<SS, NP>::STRIDE, (int)(p * NP + pr), (int)(c - 12u * xo));
        // written once and not read here again: kept out of the caches' way
        u32x4 w;
        __builtin_memcpy(&w, &v, 16);
        __builtin_nontemporal_store(w, reinterpret_cast<u32x4 *>(canon + (size_t)(b & 0x7fffffffu) * 12 + c));
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Canonical spinors to the e/o fields of a tier and back, nrhs at a time
// (workgroup id = pair group * nrhs + rhs).  Bound by HBM: one pass over the
// canonical vector and one over the field.
template <typename SO, int PAR>
__global__ void __launch_bounds__(256) k_pack(Geom g, const double2 *canon, char *eo, size_t eo_stride, int nrhs)
{
    constexpr int NP = 128;
    __shared__ PairLds<SO, NP> L;
    const uint32_t rhs = blockIdx.x % nrhs, h0 = blockIdx.x / nrhs * NP;
    const uint32_t Vh = g.Vh, np = min((uint32_t)NP, Vh - h0);
    stage_pairs<SO, NP, PAR>(L, g, h0, np, canon + (size_t)rhs * 24 * Vh);
    __syncthreads();
    eo += rhs * eo_stride;
    constexpr int WORDS = PairLds<SO, NP>::WORDS;
    if constexpr (PAR == 2) {
        const uint32_t p = threadIdx.x / NP, i = threadIdx.x % NP;
        if (i >= np) return;
        char *dst = eo + p * spinor_bytes(sizeof(SO), Vh);
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)WORDS; k++)
            stf(dst, (k * Vh + h0 + i) * 16u, L.w[k * PairLds<SO, NP>::STRIDE + threadIdx.x]);
    } else {
        const uint32_t half = threadIdx.x / NP, i = threadIdx.x % NP;
        if (i >= np) return;
        for (uint32_t k = half; k < (uint32_t)WORDS; k += 2)
            stf(eo, (k * Vh + h0 + i) * 16u, L.w[k * PairLds<SO, NP>::STRIDE + i]);
    }
}

template <typename SI, bool ODD0>
__global__ void __launch_bounds__(256) k_unpack(Geom g, const char *eo, size_t eo_stride, double2 *canon, int nrhs)
{
    constexpr int NP = 128;
    __shared__ PairLds<SI, NP> L;
    const uint32_t rhs = blockIdx.x % nrhs, h0 = blockIdx.x / nrhs * NP;
    const uint32_t Vh = g.Vh, np = min((uint32_t)NP, Vh - h0);
    eo += rhs * eo_stride;
    constexpr uint32_t WORDS = PairLds<SI, NP>::WORDS;
    const uint32_t p = threadIdx.x / NP, i = threadIdx.x % NP;
    if (threadIdx.x < np) L.base[threadIdx.x] = pair_base(g, (int)(h0 + threadIdx.x));
    if (i < np) {
        if constexpr (ODD0) {
            uint4 v[(WORDS + 1) / 2];
#pragma unroll
            for (uint32_t k = 0; k < (WORDS + 1) / 2; k++)
                if (2 * k + p < WORDS) v[k] = ldf<uint4>(eo, ((2 * k + p) * Vh + h0 + i) * 16u);
#pragma unroll
            for (uint32_t k = 0; k < (WORDS + 1) / 2; k++)
                if (2 * k + p < WORDS) L.w[(2 * k + p) * PairLds<SI, NP>::STRIDE + i] = v[k];
        } else {
            const char *src = eo + p * spinor_bytes(sizeof(SI), Vh);
            uint4 v[WORDS];
#pragma unroll
            for (uint32_t k = 0; k < WORDS; k++) v[k] = ldf<uint4>(src, (k * Vh + h0 + i) * 16u);
#pragma unroll
            for (uint32_t k = 0; k < WORDS; k++) L.w[k * PairLds<SI, NP>::STRIDE + threadIdx.x] = v[k];
        }
    }
    __syncthreads();
    write_pairs<SI, NP, ODD0>(L, np, canon + (size_t)rhs * 24 * Vh);
}

hipError_t launch_pack(const Geom &g, int prec, bool even_only, const double *canon, void *eo, size_t eo_stride, int nrhs,
                       hipStream_t st)
{
    dim3 grid(((g.Vh + 127) / 128) * nrhs), block(256);
    const double2 *c = (const double2 *)canon;
    char *e = (char *)eo;
#define WCL_PACK(T)                                                                     \
    do {                                                                                \
        if (even_only) k_pack<T, 0><<<grid, block, 0, st>>>(g, c, e, eo_stride, nrhs);  \
        else k_pack<T, 2><<<grid, block, 0, st>>>(g, c, e, eo_stride, nrhs);            \
    } while (0)
    if (prec == P64) WCL_PACK(double);
    else if (prec == P32) WCL_PACK(float);
    else if (prec == P16) WCL_PACK(__half);
    else return hipErrorInvalidValue;
#undef WCL_PACK
    return hipGetLastError();
}

hipError_t launch_unpack(const Geom &g, int prec, bool odd_zero, const void *eo, size_t eo_stride, double *canon, int nrhs,
                         hipStream_t st)
{
    dim3 grid(((g.Vh + 127) / 128) * nrhs), block(256);
    double2 *c = (double2 *)canon;
    const char *e = (const char *)eo;
#define WCL_UNPACK(T)                                                                       \
    do {                                                                                    \
        if (odd_zero) k_unpack<T, true><<<grid, block, 0, st>>>(g, e, eo_stride, c, nrhs);  \
        else k_unpack<T, false><<<grid, block, 0, st>>>(g, e, eo_stride, c, nrhs);          \
    } while (0)
    if (prec == P64) WCL_UNPACK(double);
    else if (prec == P32) WCL_UNPACK(float);
    else if (prec == P16) WCL_UNPACK(__half);
    else return hipErrorInvalidValue;
#undef WCL_UNPACK
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// D, D^dag, H, T or T^-1 from canonical spinor to canonical spinor in one
// launch: the workgroup's own pairs come from LDS (rounded to the tier's
// storage), a neighbour outside them straight from the canonical vector, by
// the lanes that have one there (unconditional loads, reading zero in the
// others, kept the texture units busy 95% of the time on large lattices).  Per site the
// arithmetic and its order are those of the even/odd hop.  Both
// parities in one workgroup read each of its links from memory once.  Output
// and clover go past the caches (non-temporal: 8 to 10% of the time), which
// leaves L2 to the faces that regions share.  Bound by the memory fabric on
// large lattices: D^dag in FP64 on 24^3x32 takes 143 us (844 MB moved for the
// call's 679 MB, 5.9 TB/s; 325 us as pack, one launch per parity and unpack),
// D in FP32 on 32^3x64 485 us (2.8 GB for 2.0, 5.8 TB/s; 1158); by latency on
// 8^4, FP64: 9.7 us a call (31.8).  Grouping right-hand sides by regions whose
// operator fits L2 measured the same.
struct CanonArgs {
    Geom g;
    const double2 *in;
    double2 *out;
    const void *links, *clov;
    double coef;
    int nrhs, xcd;
};

template <typename SL>
struct CanonStage {
    LinkRaw<SL> u;
    double2 far[12];   // the neighbour as read from the canonical vector
    uint32_t slot;     // its LDS slot, or CUT
};

template <typename SL, int K, int NP, typename R>
WCL_D void canon_load(const CanonArgs &a, const double2 *in, const Site &s, uint32_t p, uint32_t h0, uint32_t h,
                      uint32_t n, CanonStage<SL> &st, cplx<R> acc[12])
{
    constexpr int MU = K >> 1;
    constexpr bool FWD = (K & 1) == 0;
    const Geom &g = a.g;
    uint32_t hn = (uint32_t)neighbour(g, s, MU, FWD ? +1 : -1);
    const uint32_t sm = MU == 0 ? 1 : MU == 1 ? g.L[0] : MU == 2 ? g.L[0] * g.L[1] : g.L[0] * g.L[1] * g.L[2];
    uint32_t nn = FWD ? (s.x[MU] == g.L[MU] - 1 ? n - (g.L[MU] - 1) * sm : n + sm)
                      : (s.x[MU] == 0 ? n + (g.L[MU] - 1) * sm : n - sm);
    pipeline_fence(acc, hn, nn);
    const uint32_t l = hn - h0;
    const bool near = l < (uint32_t)NP;
    st.slot = near ? (1u - p) * NP + l : CUT;
    if constexpr (NP == 0) {   // no region: every neighbour
#pragma unroll
        for (uint32_t i = 0; i < 12; i++) st.far[i] = ldf<double2>(in, nn * 192u + i * 16u);
    } else if constexpr (NP == 32) {
        // few waves, each waiting for its own chain of loads: unconditional loads
        // keep the wait counts exact (out of range, so zero, where the LDS serves)
        const uint32_t off = near ? CUT : nn * 192u;
#pragma unroll
        for (uint32_t i = 0; i < 12; i++) st.far[i] = ldb<double2>(field_rsrc(in), off + i * 16u);
    } else if (!near) {
#pragma unroll
        for (uint32_t i = 0; i < 12; i++) st.far[i] = ldf<double2>(in, nn * 192u + i * 16u);
    }
    if (FWD) load_link_raw<SL>(a.links, MU, (int)p, h, g.Vh, st.u);
    else load_link_raw<SL>(a.links, MU, 1 - (int)p, hn, g.Vh, st.u);
}

// A component of the canonical vector as the tier's fields hold it.
template <typename SS, typename R>
WCL_D cplx<R> tier_value(double2 v)
{
    if constexpr (sizeof(SS) == 2) {
        const float2 f = h2f2(f22h((float)v.x, (float)v.y));
        return {f.x, f.y};
    } else {
        return {(R)v.x, (R)v.y};
    }
}

template <typename SL, typename SS, int K, int SG, int NP, typename R>
WCL_D void canon_compute(const CanonArgs &a, const PairLds<SS, NP> &L, const Site &s, const CanonStage<SL> &st,
                         cplx<R> acc[12])
{
    constexpr int MU = K >> 1;
    constexpr bool FWD = (K & 1) == 0;
    constexpr int S = FWD ? -SG : SG;
    const bool near = st.slot != CUT;
    cplx<R> psi[12], hh[6], uh[6], u[9];
    get_spinor<SS, R>(L.w, PairLds<SS, NP>::STRIDE, near ? (int)st.slot : 0, psi);
#pragma unroll
    for (int i = 0; i < 12; i++) {
        const cplx<R> f = tier_value<SS, R>(st.far[i]);
        psi[i] = {near ? psi[i].re : f.re, near ? psi[i].im : f.im};
    }
    project<MU, S, R>(psi, hh);
    if constexpr (MU == 3) {
        const R sign = (a.g.tbc < 0 && s.x[3] == (FWD ? a.g.L[3] - 1 : 0)) ? R(-1) : R(1);
#pragma unroll
        for (int k = 0; k < 6; k++) hh[k] = sign * hh[k];
    }
    expand_link<SL, R>(st.u, u);
    if (FWD) su3_mul(u, hh, uh);
    else su3_dag_mul(u, hh, uh);
    accumulate<MU, S, R>(acc, uh);
}

template <typename SL, typename SS, int K, int SG, int NP, typename R>
WCL_D void canon_hops(const CanonArgs &a, const double2 *in, const PairLds<SS, NP> &L, const Site &s, uint32_t p,
                      uint32_t h0, uint32_t h, uint32_t n, CanonStage<SL> st[2], cplx<R> acc[12])
{
    if constexpr (K < 8) {
        if constexpr (K + 1 < 8) canon_load<SL, K + 1, NP, R>(a, in, s, p, h0, h, n, st[(K + 1) & 1], acc);
        canon_compute<SL, SS, K, SG, NP, R>(a, L, s, st[K & 1], acc);
        canon_hops<SL, SS, K + 1, SG, NP, R>(a, in, L, s, p, h0, h, n, st, acc);
    }
}

// The hops of an odd site with every neighbour from the canonical vector.
template <typename SL, typename SS, int K, typename R>
WCL_D void canon_hops_direct(const CanonArgs &a, const double2 *in, const Site &s, uint32_t h, uint32_t n,
                             CanonStage<SL> st[2], cplx<R> acc[12])
{
    if constexpr (K < 8) {
        constexpr int MU = K >> 1;
        constexpr bool FWD = (K & 1) == 0;
        constexpr int S = FWD ? -1 : 1;
        if constexpr (K + 1 < 8) canon_load<SL, K + 1, 0, R>(a, in, s, 1u, 0u, h, n, st[(K + 1) & 1], acc);
        cplx<R> psi[12], hh[6], uh[6], u[9];
#pragma unroll
        for (int i = 0; i < 12; i++) psi[i] = tier_value<SS, R>(st[K & 1].far[i]);
        project<MU, S, R>(psi, hh);
        if constexpr (MU == 3) {
            const R sign = (a.g.tbc < 0 && s.x[3] == (FWD ? a.g.L[3] - 1 : 0)) ? R(-1) : R(1);
#pragma unroll
            for (int k = 0; k < 6; k++) hh[k] = sign * hh[k];
        }
        expand_link<SL, R>(st[K & 1].u, u);
        if (FWD) su3_mul(u, hh, uh);
        else su3_dag_mul(u, hh, uh);
        accumulate<MU, S, R>(acc, uh);
        canon_hops_direct<SL, SS, K + 1, R>(a, in, s, h, n, st, acc);
    }
}

// MODE: HOP out = H in; CLOVX out = A in + coef H in; CLOV_H out = A in (no hop)
template <typename SL, typename SS, int MODE, bool DAG, int NP>
__global__ void __launch_bounds__(2 * NP) k_canon(CanonArgs a)
{
    using R = typename Real<SL>::T;
    __shared__ PairLds<SS, NP> L;
    const Geom &g = a.g;
    const int lin = a.xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const uint32_t rhs = lin % a.nrhs, h0 = lin / a.nrhs * NP;
    const uint32_t Vh = g.Vh, np = min((uint32_t)NP, Vh - h0);
    const double2 *in = a.in + (size_t)rhs * 24 * Vh;
    stage_pairs<SS, NP, 2>(L, g, h0, np, in);
    __syncthreads();
    const uint32_t p = threadIdx.x / NP, i = threadIdx.x % NP, h = h0 + i;
    cplx<R> o[12];
    if (i < np) {
        cplx<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = {R(0), R(0)};
        if constexpr (MODE != CLOV_H) {
            const Site s = decompose(g, (int)h, (int)p);
            const uint32_t n = (uint32_t)(s.x[0] + g.L[0] * (s.x[1] + g.L[1] * (s.x[2] + g.L[2] * s.x[3])));
            CanonStage<SL> st[2];
            canon_load<SL, 0, NP, R>(a, in, s, p, h0, h, n, st[0], acc);
            canon_hops<SL, SS, 0, DAG ? -1 : 1, NP, R>(a, in, L, s, p, h0, h, n, st, acc);
        }
        if constexpr (MODE == HOP) {
#pragma unroll
            for (int k = 0; k < 12; k++) o[k] = acc[k];
        } else {
            cplx<R> xv[12];
            get_spinor<SS, R>(L.w, PairLds<SS, NP>::STRIDE, (int)threadIdx.x, xv);
            const R cf = (R)a.coef;
#pragma unroll
            for (int half = 0; half < 2; half++) {
                // one chirality block at a time: 36 clover reals live, not 72
                uint32_t hc = h, dummy = 0;
                pipeline_fence(acc, hc, dummy);
                R c[36];
                // non-temporal: L2 keeps what neighbouring workgroups share (FP16: 2% slower
                // for 12 right-hand sides, which share it themselves)
                load_clover_half<typename ClovS<SL>::T, R, sizeof(SS) != 2>(a.clov, (int)p, hc, Vh, half, c);
                clover_mul_half(c, xv + 6 * half, o + 6 * half);
            }
            if constexpr (MODE == CLOVX) {
#pragma unroll
                for (int k = 0; k < 12; k++) o[k] = {fmar(cf, acc[k].re, o[k].re), fmar(cf, acc[k].im, o[k].im)};
            }
        }
    }
    __syncthreads();   // every neighbour has been read
    if (i < np) put_spinor<SS, R>(L.w, PairLds<SS, NP>::STRIDE, (int)threadIdx.x, o);
    __syncthreads();
    write_pairs<SS, NP, false>(L, np, a.out + (size_t)rhs * 24 * Vh);
}

// The same from e/o fields in the tier's storage (parity-major, in_stride bytes
// between right-hand sides) to canonical spinors: neighbours at 16-byte words
// a lane instead of 192 bytes of the canonical vector.
template <typename SL, int K, int SG, typename R, typename SS>
WCL_D void eo_hops(const CanonArgs &a, const char *in, const Site &s, uint32_t p, uint32_t h, HopStage<SL, SS, R> st[2],
                   cplx<R> acc[12])
{
    // hop_load and hop_compute of the even/odd kernel, unstaged
    if constexpr (K < 8) {
        HopArgs q;
        q.g = a.g;
        q.links = a.links;
        q.p = (int)p;
        const LdsIn none{};
        if constexpr (K + 1 < 8) hop_load<SL, SS, K + 1, false, 0, R>(q, s, h, in, none, st[(K + 1) & 1], acc);
        hop_compute<K, SG, SL, SS, R>(st[K & 1], acc);
        eo_hops<SL, K + 1, SG, R, SS>(a, in, s, p, h, st, acc);
    }
}

template <typename SL, typename SS, int MODE, bool DAG>
__global__ void __launch_bounds__(256) k_eo_canon(CanonArgs a, const char *eo, size_t eo_stride)
{
    using R = typename Real<SL>::T;
    constexpr int NP = 128;
    __shared__ PairLds<SS, NP> L;
    const Geom &g = a.g;
    const int lin = a.xcd ? xcd_block(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const uint32_t rhs = lin % a.nrhs, h0 = lin / a.nrhs * NP;
    const uint32_t Vh = g.Vh, np = min((uint32_t)NP, Vh - h0);
    const uint32_t p = threadIdx.x / NP, i = threadIdx.x % NP, h = h0 + i;
    if (threadIdx.x < np) L.base[threadIdx.x] = pair_base(g, (int)(h0 + threadIdx.x));
    eo += rhs * eo_stride;
    if (i < np) {
        const size_t hb = spinor_bytes(sizeof(SS), Vh);
        const char *other = eo + (1 - p) * hb;
        cplx<R> acc[12], o[12];
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = {R(0), R(0)};
        const Site s = decompose(g, (int)h, (int)p);
        HopArgs q;
        q.g = a.g;
        q.links = a.links;
        q.p = (int)p;
        HopStage<SL, SS, R> st[2];
        hop_load<SL, SS, 0, false, 0, R>(q, s, h, other, LdsIn{}, st[0], acc);
        eo_hops<SL, 0, DAG ? -1 : 1, R, SS>(a, other, s, p, h, st, acc);
        if constexpr (MODE == HOP) {
#pragma unroll
            for (int k = 0; k < 12; k++) o[k] = acc[k];
        } else {
            cplx<R> xv[12];
            uint32_t hx = h, dummy = 0;
            pipeline_fence(acc, hx, dummy);
            load_spinor<SS, R>(eo + p * hb, hx, Vh, xv);
            const R cf = (R)a.coef;
#pragma unroll
            for (int half = 0; half < 2; half++) {
                uint32_t hc = h, none = 0;
                pipeline_fence(acc, hc, none);
                R c[36];
                load_clover_half<typename ClovS<SL>::T, R>(a.clov, (int)p, hc, Vh, half, c);
                clover_mul_half(c, xv + 6 * half, o + 6 * half);
            }
#pragma unroll
            for (int k = 0; k < 12; k++) o[k] = {fmar(cf, acc[k].re, o[k].re), fmar(cf, acc[k].im, o[k].im)};
        }
        put_spinor<SS, R>(L.w, PairLds<SS, NP>::STRIDE, (int)threadIdx.x, o);
    }
    __syncthreads();
    write_pairs<SS, NP, false>(L, np, a.out + (size_t)rhs * 24 * Vh);
}

template <typename SL, typename SS>
static hipError_t eo_canon_dispatch(const CanonLaunch &L, const CanonArgs &a, hipStream_t st)
{
    dim3 grid(((a.g.Vh + 127) / 128) * a.nrhs), block(256);
    const char *eo = (const char *)L.eo;
    if (L.mode == HOP && !L.dagger) ext_launch(k_eo_canon<SL, SS, HOP, false>, grid, block, 0, st, L.ev, a, eo, L.eo_stride);
    else if (L.mode == CLOVX && !L.dagger) ext_launch(k_eo_canon<SL, SS, CLOVX, false>, grid, block, 0, st, L.ev, a, eo, L.eo_stride);
    else if (L.mode == CLOVX) ext_launch(k_eo_canon<SL, SS, CLOVX, true>, grid, block, 0, st, L.ev, a, eo, L.eo_stride);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The even/odd operator on small lattices in two launches, canonical to
// canonical: odd = A_oo^-1 H_oe in_e (an e/o field of the tier), then
// out_e = in_e + coef A_ee^-1 H_eo odd, out_o = 0.  NP pairs and NP threads a
// workgroup, one output site each; what pack and unpack launches would do
// rides along (Schur FP32 on 2 x 12x6x10x14: 16.7 us a call, 27.2 with them).
// The neighbours of the first come from the canonical vector, 192 bytes each,
// which large lattices pay for (24^3x32 FP32: 148 against 114 us; even at 16^3x32).
template <typename SL, typename SS, int NP>
__global__ void __launch_bounds__(NP) k_schur_odd(CanonArgs a, char *odd, size_t odd_stride)
{
    using R = typename Real<SL>::T;
    const Geom &g = a.g;
    const uint32_t rhs = blockIdx.x % a.nrhs, h = blockIdx.x / a.nrhs * NP + threadIdx.x;
    const uint32_t Vh = g.Vh;
    if (h >= Vh) return;
    const double2 *in = a.in + (size_t)rhs * 24 * Vh;
    cplx<R> acc[12], o[12];
#pragma unroll
    for (int k = 0; k < 12; k++) acc[k] = {R(0), R(0)};
    const Site s = decompose(g, (int)h, 1);
    const uint32_t n = (uint32_t)(s.x[0] + g.L[0] * (s.x[1] + g.L[1] * (s.x[2] + g.L[2] * s.x[3])));
    CanonStage<SL> st[2];
    canon_load<SL, 0, 0, R>(a, in, s, 1u, 0u, h, n, st[0], acc);
    canon_hops_direct<SL, SS, 0, R>(a, in, s, h, n, st, acc);
#pragma unroll
    for (int half = 0; half < 2; half++) {
        R c[36];
        load_clover_half<typename ClovS<SL>::T, R>(a.clov, 1, h, Vh, half, c);
        clover_mul_half(c, acc + 6 * half, o + 6 * half);
    }
    store_spinor<SS, R>(odd + rhs * odd_stride, h, Vh, o);
}

template <typename SL, typename SS, int NP>
__global__ void __launch_bounds__(NP) k_schur_even(CanonArgs a, const char *odd, size_t odd_stride)
{
    using R = typename Real<SL>::T;
    __shared__ PairLds<SS, NP> L;
    const Geom &g = a.g;
    const uint32_t rhs = blockIdx.x % a.nrhs, h0 = blockIdx.x / a.nrhs * NP, i = threadIdx.x, h = h0 + i;
    const uint32_t Vh = g.Vh, np = min((uint32_t)NP, Vh - h0);
    if (i < np) {
        const uint32_t b = pair_base(g, (int)h);
        L.base[i] = b;
        odd += rhs * odd_stride;
        cplx<R> acc[12], xv[12], o[12];
#pragma unroll
        for (int k = 0; k < 12; k++) acc[k] = {R(0), R(0)};
        // the even site's own spinor, rounded to the tier
        const double2 *x = a.in + (size_t)rhs * 24 * Vh + (size_t)((b & 0x7fffffffu) + (b >> 31)) * 12;
        double2 xr[12];
#pragma unroll
        for (int k = 0; k < 12; k++) xr[k] = x[k];
        const Site s = decompose(g, (int)h, 0);
        HopArgs q;
        q.g = a.g;
        q.links = a.links;
        q.p = 0;
        HopStage<SL, SS, R> st[2];
        hop_load<SL, SS, 0, false, 0, R>(q, s, h, odd, LdsIn{}, st[0], acc);
        eo_hops<SL, 0, 1, R, SS>(a, odd, s, 0u, h, st, acc);
        const R cf = (R)a.coef;
#pragma unroll
        for (int k = 0; k < 12; k++) xv[k] = tier_value<SS, R>(xr[k]);
#pragma unroll
        for (int half = 0; half < 2; half++) {
            R c[36];
            cplx<R> t[6];
            load_clover_half<typename ClovS<SL>::T, R>(a.clov, 0, h, Vh, half, c);
            clover_mul_half(c, acc + 6 * half, t);
#pragma unroll
            for (int k = 0; k < 6; k++)
                o[6 * half + k] = {fmar(cf, t[k].re, xv[6 * half + k].re), fmar(cf, t[k].im, xv[6 * half + k].im)};
        }
        put_spinor<SS, R>(L.w, PairLds<SS, NP>::STRIDE, (int)i, o);
    }
    __syncthreads();
    write_pairs<SS, NP, true, NP>(L, np, a.out + (size_t)rhs * 24 * Vh);
}

template <typename SL, typename SS>
static hipError_t schur_canon_dispatch(const CanonLaunch &L, const CanonArgs &a, hipStream_t st)
{
    constexpr int NP = 64;
    dim3 grid(((a.g.Vh + NP - 1) / NP) * a.nrhs), block(NP);
    if (L.mode == CLOV_H) ext_launch(k_schur_odd<SL, SS, NP>, grid, block, 0, st, L.ev, a, (char *)L.eo, L.eo_stride);
    else ext_launch(k_schur_even<SL, SS, NP>, grid, block, 0, st, L.ev, a, (const char *)L.eo, L.eo_stride);
    return hipGetLastError();
}

hipError_t launch_schur_canon(const CanonLaunch &L, hipStream_t st)
{
    CanonArgs a;
    a.g = *L.g;
    a.in = (const double2 *)L.in;
    a.out = (double2 *)L.out;
    a.links = L.links;
    a.clov = L.clov;
    a.coef = L.coef;
    a.nrhs = L.nrhs;
    a.xcd = 0;
    if (L.nrhs < 1 || !L.eo || (L.mode != CLOV_H && L.mode != XPAY)) return hipErrorInvalidValue;
    switch (L.link_prec) {
    case P64: return schur_canon_dispatch<double, double>(L, a, st);
    case P32: return schur_canon_dispatch<float, float>(L, a, st);
    case P16: return schur_canon_dispatch<__half, __half>(L, a, st);
    case P32C: return schur_canon_dispatch<R12f, float>(L, a, st);
    case P16C: return schur_canon_dispatch<R12h, __half>(L, a, st);
    default: return hipErrorInvalidValue;
    }
}

template <typename SL, typename SS>
static hipError_t canon_dispatch(const CanonLaunch &L, const CanonArgs &a, hipStream_t st)
{
    // 32 pairs a workgroup (one wave) where 128 would leave CUs without one
    const bool small = (long long)a.g.Vh * a.nrhs < 32 * 256 * 4;
    const int np = small ? 32 : 128;
    dim3 grid(((a.g.Vh + np - 1) / np) * a.nrhs), block(2 * np);
#define WCL_CANON(MODE, DAG)                                                                       \
    do {                                                                                           \
        if (small) ext_launch(k_canon<SL, SS, MODE, DAG, 32>, grid, block, 0, st, L.ev, a);        \
        else ext_launch(k_canon<SL, SS, MODE, DAG, 128>, grid, block, 0, st, L.ev, a);             \
    } while (0)
    if (L.mode == HOP && !L.dagger) WCL_CANON(HOP, false);
    else if (L.mode == CLOV_H && !L.dagger) WCL_CANON(CLOV_H, false);
    else if (L.mode == CLOVX && !L.dagger) WCL_CANON(CLOVX, false);
    else if (L.mode == CLOVX) WCL_CANON(CLOVX, true);
    else return hipErrorInvalidValue;
#undef WCL_CANON
    return hipGetLastError();
}

hipError_t launch_canon(const CanonLaunch &L, hipStream_t st)
{
    CanonArgs a;
    a.g = *L.g;
    a.in = (const double2 *)L.in;
    a.out = (double2 *)L.out;
    a.links = L.links;
    a.clov = L.clov;
    a.coef = L.coef;
    a.nrhs = L.nrhs;
    a.xcd = L.xcd;
    if (L.nrhs < 1) return hipErrorInvalidValue;
    if (L.eo) {
        switch (L.link_prec) {
        case P64: return eo_canon_dispatch<double, double>(L, a, st);
        case P32: return eo_canon_dispatch<float, float>(L, a, st);
        case P16: return eo_canon_dispatch<__half, __half>(L, a, st);
        case P32C: return eo_canon_dispatch<R12f, float>(L, a, st);
        case P16C: return eo_canon_dispatch<R12h, __half>(L, a, st);
        default: return hipErrorInvalidValue;
        }
    }
    switch (L.link_prec) {
    case P64: return canon_dispatch<double, double>(L, a, st);
    case P32: return canon_dispatch<float, float>(L, a, st);
    case P16: return canon_dispatch<__half, __half>(L, a, st);
    case P32C: return canon_dispatch<R12f, float>(L, a, st);
    case P16C: return canon_dispatch<R12h, __half>(L, a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace wcl
