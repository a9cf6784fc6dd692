// CG stencils for launches that leave most of the chip idle (gfx950): small
// lattices and few right-hand sides.
//
// In k_cg_mp / k_cg_upd and the half-hops k_eo_* a lane does the eight hops of
// a site one direction after the other; with fewer waves than SIMDs that chain
// of loads and products is the launch's duration.  Here a block takes 64 sites
// of one right-hand side and each of its four waves one direction: the
// projected and transported half spinors meet in LDS, and each wave then
// finishes a part of the twelve components.  The products, the order of the
// sums over hops and over components and the partials per 64 sites are those
// of the one-lane-per-site kernels, so results are bit for bit the same and
// the choice (use_quad) may depend on the size of a launch.
//
// A launch of this size is a chain of latencies, so the stop flag of a source
// is looked at after the hops (its load does not delay theirs).

#include <algorithm>

#include "tm_device.h"
#include "tm_eo.h"
#include "tm_kernels.h"
#include "tm_stencil.h"

namespace tmq {

// the transported half spinor g of one hop: the link at s (forward) or at the
// neighbour y (backward), the spinor at y
template <int MU, bool FWD, bool DAG, typename R, class S, class G>
__device__ __forceinline__ void one_hop(const Geom& geo, const void* links, const void* in, uint32_t s, uint32_t y,
                                        bool flip, cx<R> g[6]) {
    constexpr int SF = DAG == FWD ? -1 : 1;
    const long Vs = geo.Vs;
    if constexpr (std::is_same<G, GH16>::value) {
        uint32_t U[9], A[9], B[9], hu[6];
        h2v p[12], hh[6];
        load_link16(links, Vs, MU, FWD ? s : y, U);
        load_spinor_h2(in, Vs, y, p);
        link_forms<!FWD>(U, A, B);
        proj_h2<MU, SF>(p, hh);
        const uint32_t sgn = flip ? 0x80008000u : 0u;
#pragma unroll
        for (int k = 0; k < 6; k++) hu[k] = MU == 3 ? (as_u32(hh[k]) ^ sgn) : as_u32(hh[k]);
        su3_h2(A, B, hu, g);
    } else {
        cx<R> U[3][3], p[12], h[6];
        load_link<G, R>(links, Vs, MU, FWD ? s : y, U);
        load_spinor<S, R>(in, Vs, y, p);
        proj<MU, SF>(p, h);
        if (MU == 3 && flip) negate6(h);
        if (FWD)
            su3_mul(U, h, g);
        else
            su3_dag_mul(U, h, g);
    }
}

// The hops of direction MU into site s, as two half spinors in LDS
// ([hop][component][site]); EO: s is a half site, c its coordinates
template <int MU, bool EO, bool DAG, typename R, class S, class G>
__device__ __forceinline__ void dir_hops(const Geom& geo, const void* gout, const void* gin, const void* in,
                                         uint32_t s, int par, cx<R>* sh) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t yf, yb;
    int t;
    if constexpr (EO) {
        const EoSite c = eo_coords(geo, s, par);
        yf = eo_nb(geo, s, c, MU, true);
        yb = eo_nb(geo, s, c, MU, false);
        t = c.t;
    } else {
        const Site c = site_coords(geo, s);
        yf = nb_fwd(geo, s, c, MU);
        yb = nb_bwd(geo, s, c, MU);
        t = c.t;
    }
    cx<R> f[6], b[6];
    one_hop<MU, true, DAG, R, S, G>(geo, gout, in, s, yf, t + 1 == geo.L[3] && geo.t_bc < 0, f);
    one_hop<MU, false, DAG, R, S, G>(geo, gin, in, s, yb, t == 0 && geo.t_bc < 0, b);
#pragma unroll
    for (int k = 0; k < 6; k++) {
        sh[((2 * MU) * 6 + k) * 64 + lane] = f[k];
        sh[((2 * MU + 1) * 6 + k) * 64 + lane] = b[k];
    }
}

template <bool EO, bool DAG, typename R, class S, class G>
__device__ __forceinline__ void quad_hops(const Geom& geo, const void* gout, const void* gin, const void* in,
                                          uint32_t s, int par, int w, cx<R>* sh) {
    switch (w) {
    case 0: dir_hops<0, EO, DAG, R, S, G>(geo, gout, gin, in, s, par, sh); break;
    case 1: dir_hops<1, EO, DAG, R, S, G>(geo, gout, gin, in, s, par, sh); break;
    case 2: dir_hops<2, EO, DAG, R, S, G>(geo, gout, gin, in, s, par, sh); break;
    default: dir_hops<3, EO, DAG, R, S, G>(geo, gout, gin, in, s, par, sh); break;
    }
}

// component K of the sum over hops, in the order of hop_all and recon
template <int K, int MU, int SG, typename R>
__device__ __forceinline__ void add_comp(const cx<R>* sh, int hop, cx<R>& acc) {
    const uint32_t lane = threadIdx.x & 63u;
    auto g = [&](int k) { return sh[(hop * 6 + k) * 64 + lane]; };
    if constexpr (K < 6) {
        acc = acc + g(K);
    } else {
        constexpr int a = (K - 6) / 3, c = (K - 6) % 3;
        cx<R> e;
        if (MU == 0)
            e = times_i(g(a == 0 ? 3 + c : c));
        else if (MU == 1) {
            e = g(a == 0 ? 3 + c : c);
            if (a == 1) e = {-e.re, -e.im};
        } else if (MU == 2)
            e = a == 0 ? times_i(g(c)) : times_mi(g(3 + c));
        else
            e = g(a == 0 ? c : 3 + c);
        if (SG > 0)
            acc = acc - e;
        else
            acc = acc + e;
    }
}
template <int K, bool DAG, typename R>
__device__ __forceinline__ cx<R> hop_comp(const cx<R>* sh) {
    constexpr int SF = DAG ? -1 : 1;
    cx<R> acc = {(R)0, (R)0};
    add_comp<K, 0, SF>(sh, 0, acc);
    add_comp<K, 0, -SF>(sh, 1, acc);
    add_comp<K, 1, SF>(sh, 2, acc);
    add_comp<K, 1, -SF>(sh, 3, acc);
    add_comp<K, 2, SF>(sh, 4, acc);
    add_comp<K, 2, -SF>(sh, 5, acc);
    add_comp<K, 3, SF>(sh, 6, acc);
    add_comp<K, 3, -SF>(sh, 7, acc);
    return acc;
}

// Components of a wave's part of a spinor: whole 16-byte vectors, 3 components
// (four waves) in FP64 and 4 (three waves) otherwise.
template <class S>
constexpr int part_comps() {
    return S::NV == 12 ? 3 : 4;
}
template <class S>
constexpr int part_waves() {
    return 12 / part_comps<S>();
}
// part w of the spinor at site s (N components from 16-byte vectors of S)
template <class S, typename R, int N>
__device__ __forceinline__ void load_part(const void* base, long Vs, uint32_t s, int w, cx<R> p[N]) {
    if constexpr (S::NV == 12) {
#pragma unroll
        for (int c = 0; c < N; c++) {
            const double2 v = ld_plane<double2>(base, Vs, w * N + c, s);
            p[c] = {(R)v.x, (R)v.y};
        }
    } else if constexpr (S::NV == 6) {
        static_assert(N == 4, "two vectors");
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const float4 v = ld_plane<float4>(base, Vs, 2 * w + k, s);
            p[2 * k] = {(R)v.x, (R)v.y};
            p[2 * k + 1] = {(R)v.z, (R)v.w};
        }
    } else {
        static_assert(N == 4, "one vector");
        constexpr bool BF = std::is_same<S, SBF16>::value;
        const uint4 v = ld_plane<uint4>(base, Vs, w, s);
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; j++)
            p[j] = {(R)(BF ? bf16_to_f32(u[j] & 0xFFFFu) : f16_to_f32(u[j] & 0xFFFFu)),
                    (R)(BF ? bf16_to_f32(u[j] >> 16) : f16_to_f32(u[j] >> 16))};
    }
}
template <class S, typename R, int N>
__device__ __forceinline__ void store_part(void* base, long Vs, uint32_t s, int w, const cx<R> p[N]) {
    if constexpr (S::NV == 12) {
#pragma unroll
        for (int c = 0; c < N; c++) st_plane(base, Vs, w * N + c, s, make_double2((double)p[c].re, (double)p[c].im));
    } else if constexpr (S::NV == 6) {
#pragma unroll
        for (int k = 0; k < 2; k++)
            st_plane(base, Vs, 2 * w + k, s,
                     make_float4((float)p[2 * k].re, (float)p[2 * k].im, (float)p[2 * k + 1].re, (float)p[2 * k + 1].im));
    } else {
        constexpr bool BF = std::is_same<S, SBF16>::value;
        uint32_t u[4];
#pragma unroll
        for (int j = 0; j < 4; j++)
            u[j] = BF ? pack2_bf16((float)p[j].re, (float)p[j].im) : pack2_f16((float)p[j].re, (float)p[j].im);
        st_plane<uint4>(base, Vs, w, s, make_uint4(u[0], u[1], u[2], u[3]));
    }
}
// values as the storage holds them (round_storage for a part)
template <class S, typename R, int N>
__device__ __forceinline__ void round_part(cx<R> p[N]) {
    if constexpr (S::NV == 3) {
        constexpr bool BF = std::is_same<S, SBF16>::value;
#pragma unroll
        for (int c = 0; c < N; c++)
            p[c] = BF ? cx<R>{bf16_to_f32(f32_to_bf16(p[c].re)), bf16_to_f32(f32_to_bf16(p[c].im))}
                      : cx<R>{f16_to_f32(f32_to_f16(p[c].re)), f16_to_f32(f32_to_f16(p[c].im))};
    }
}

// f<W>(): the body of part W, W a compile-time constant
template <class S, class F>
__device__ __forceinline__ void for_part(int w, F&& f) {
    if (w == 0) f(std::integral_constant<int, 0>{});
    if (w == 1) f(std::integral_constant<int, 1>{});
    if (w == 2) f(std::integral_constant<int, 2>{});
    if constexpr (part_waves<S>() == 4)
        if (w == 3) f(std::integral_constant<int, 3>{});
}

// |v|^2 per site of the components the waves left in LDS ([component][site]),
// summed over the 64 sites by wave 0: a partial of the group
template <typename R>
__device__ __forceinline__ void norm_partial(const cx<R>* sh, bool on, double* out) {
    if (threadIdx.x >= 64) return;
    cx<R> v[12];
#pragma unroll
    for (int k = 0; k < 12; k++) v[k] = sh[k * 64 + threadIdx.x];
    const double n = wave_sum(on ? spinor_norm2(v) : 0.0);
    if (threadIdx.x == 0) *out = n;
}

struct QuadSite {
    uint32_t s, ws, nws;
    int r, w;
};
// block: group of 64 sites (in the order of the one-lane kernels) x right-hand side
template <bool EO>
__device__ __forceinline__ QuadSite quad_site(const Geom& geo, int nrhs) {
    const uint32_t L = xcd_block(blockIdx.x, gridDim.x);
    QuadSite q;
    q.nws = (uint32_t)((geo.V + 63) / 64);
    q.ws = L / (uint32_t)nrhs;
    q.r = (int)(L - q.ws * (uint32_t)nrhs);
    q.w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    q.s = EO ? eo_site(geo, q.ws >> 2, (q.ws & 3u) * 64u + lane) : slab_order(geo, q.ws * 64u + lane);
    return q;
}

// y = D^{-1} H_eo p (DAG: of the adjoint), k_eo_lin of the CG iteration
template <bool DAG, typename R, class S, class G>
__global__ __launch_bounds__(256) void k_quad_lin(EoArgs a) {
    __shared__ cx<R> sh[8 * 6 * 64];
    const Geom& hg = a.hg;
    const QuadSite q = quad_site<true>(hg, a.nrhs);
    const bool act = a.act == nullptr || a.act[q.r].active;
    const long Vs = hg.Vs;
    const bool on = q.s < (uint32_t)hg.V;
    if (on) quad_hops<true, DAG, R, S, G>(hg, a.gout, a.gin, field_rhs<S>(a.in, Vs, q.r), q.s, a.pout, q.w, sh);
    __syncthreads();
    if (!on || !act) return;
    const R tw = (R)(DAG ? -a.twist : a.twist);
    const R inv = (R)(1.0 / (1.0 + a.twist * a.twist));
    const R cf = (R)a.c;
    for_part<S>(q.w, [&](auto W) {
        constexpr int N = part_comps<S>(), K0 = W.value * N;
        cx<R> o[N];
        auto comp = [&](auto C) {
            constexpr int c = C.value, K = K0 + c;
            cx<R> v = cf * hop_comp<K, DAG, R>(sh);
            const R sg = K < 6 ? -tw : tw;  // (mul_diag_inv)
            o[c] = {inv * (v.re - sg * v.im), inv * (v.im + sg * v.re)};
        };
        comp(std::integral_constant<int, 0>{});
        comp(std::integral_constant<int, 1>{});
        comp(std::integral_constant<int, 2>{});
        if constexpr (N == 4) comp(std::integral_constant<int, 3>{});
        store_part<S, R, N>(field_rhs<S>(a.out, Vs, q.r), Vs, q.s, W.value, o);
    });
}

// part W of the operator: EO D v + k2 hops (k2 = -kappa^2), else v - kappa hops
// + i tw g5 v (the expressions of mul_diag and diag_combine; K1 of the whole
// lattice towards its storage, ST = S)
template <bool EO, bool DAG, int K, class ST, typename R>
__device__ __forceinline__ cx<R> op_comp(cx<R> v, const cx<R>* sh, R kap, R tw) {
    const cx<R> h = hop_comp<K, DAG, R>(sh);
    if constexpr (EO) {
        const R sg = K < 6 ? tw : -tw;
        const cx<R> d = {v.re - sg * v.im, v.im + sg * v.re};
        return d + kap * h;
    } else {
        return diag_towards<ST, K, R>(v, h, kap, tw);
    }
}

// K1: t = M p (EO: D p - kappa^2 H_oe y), |t|^2
template <bool EO, typename R, class S, class G>
__global__ __launch_bounds__(256) void k_quad_mp(CgArgs a, EoCg e) {
    __shared__ cx<R> sh[8 * 6 * 64];
    const Geom& geo = a.geo;
    const QuadSite q = quad_site<EO>(geo, a.nrhs);
    const bool act = a.scal[q.r].active != 0;
    const long Vs = geo.Vs;
    const bool on = q.s < (uint32_t)geo.V;
    const void* gout = EO ? e.godd : a.gauge;
    const void* gin = EO ? e.geven : a.gauge;
    if (on) quad_hops<EO, false, R, S, G>(geo, gout, gin, field_rhs<S>(EO ? e.y : a.p, Vs, q.r), q.s, 1, q.w, sh);
    const R tw = (R)a.twist, kap = EO ? (R)(-a.kappa * a.kappa) : (R)a.kappa;
    constexpr int N = part_comps<S>();
    cx<R> o[N];
    if (on && q.w < part_waves<S>()) load_part<S, R, N>(field_rhs<S>(a.p, Vs, q.r), Vs, q.s, q.w, o);
    __syncthreads();
    if (!act) return;  // uniform over the block
    if (on)
        for_part<S>(q.w, [&](auto W) {
            constexpr int K0 = W.value * N;
            o[0] = op_comp<EO, false, K0, S>(o[0], sh, kap, tw);
            o[1] = op_comp<EO, false, K0 + 1, S>(o[1], sh, kap, tw);
            o[2] = op_comp<EO, false, K0 + 2, S>(o[2], sh, kap, tw);
            if constexpr (N == 4) o[3] = op_comp<EO, false, K0 + 3, S>(o[3], sh, kap, tw);
            round_part<S, R, N>(o);
            store_part<S, R, N>(field_rhs<S>(a.t, Vs, q.r), Vs, q.s, W.value, o);
        });
    __syncthreads();  // (every wave has read the hops)
    if (q.w < part_waves<S>())
#pragma unroll
        for (int c = 0; c < N; c++) sh[(q.w * N + c) * 64 + (threadIdx.x & 63u)] = o[c];
    __syncthreads();
    norm_partial<R>(sh, on, a.partials + (size_t)q.r * q.nws + q.ws);
}

// K1 with the step before finished in it (whole lattice, FP64 and FP32):
// p' = r + beta p is formed where the hops and the operator read it and written
// to the other direction buffer pn, so k_cg_p and its launch go: each wave sums
// |r|^2 from the partials of the last K2 (scal_next not null), forms beta and
// the stop test and the first thread hands the state on; the fields and links
// are loaded meanwhile.  The launch is a chain of latencies.  4^4, FP64: an
// iteration of three launches (5.9 + 6.9 + 4.8 us) -> two (7.0 + 6.1 us); a
// solve of 12 sources 390 -> 359 us.
template <int MU, typename R, class S, class G, class B>
__device__ __forceinline__ void dir_hops_fold(const Geom& geo, const void* links, const void* pin, const void* rin,
                                              uint32_t s, cx<R>* sh, B&& beta) {
    const uint32_t lane = threadIdx.x & 63u;
    const long Vs = geo.Vs;
    const Site c = site_coords(geo, s);
    const uint32_t yf = nb_fwd(geo, s, c, MU), yb = nb_bwd(geo, s, c, MU);
    cx<R> pf[12], rf[12], pb[12], rb[12], U[3][3], Ub[3][3], f[6], b[6], h[6];
    load_spinor<S, R>(pin, Vs, yf, pf);
    load_spinor<S, R>(rin, Vs, yf, rf);
    load_spinor<S, R>(pin, Vs, yb, pb);
    load_spinor<S, R>(rin, Vs, yb, rb);
    load_link<G, R>(links, Vs, MU, s, U);
    load_link<G, R>(links, Vs, MU, yb, Ub);
    const R be = beta();
#pragma unroll
    for (int k = 0; k < 12; k++) {
        pf[k] = rf[k] + be * pf[k];
        pb[k] = rb[k] + be * pb[k];
    }
    proj<MU, 1>(pf, h);
    if (MU == 3 && c.t + 1 == geo.L[3] && geo.t_bc < 0) negate6(h);
    su3_mul(U, h, f);
    proj<MU, -1>(pb, h);
    if (MU == 3 && c.t == 0 && geo.t_bc < 0) negate6(h);
    su3_dag_mul(Ub, h, b);
#pragma unroll
    for (int k = 0; k < 6; k++) {
        sh[((2 * MU) * 6 + k) * 64 + lane] = f[k];
        sh[((2 * MU + 1) * 6 + k) * 64 + lane] = b[k];
    }
}

template <typename R, class S, class G>
__global__ __launch_bounds__(256) void k_quad_mp_fold(CgArgs a) {
    __shared__ cx<R> sh[8 * 6 * 64];
    const Geom& geo = a.geo;
    const QuadSite q = quad_site<false>(geo, a.nrhs);
    const long Vs = geo.Vs;
    const bool on = q.s < (uint32_t)geo.V;
    const uint32_t s = on ? q.s : 0u;  // lanes past the lattice compute site 0 and store nothing
    const void *pin = field_rhs<S>(a.p, Vs, q.r), *rin = field_rhs<S>(a.r, Vs, q.r);
    StepEnd e;
    const double* parts = a.partials2 + (size_t)q.r * a.npart;
    e.begin(a.scal + q.r, parts, a.npart);
    const double bst = a.scal[q.r].beta;
    TM_MEM_FENCE();
    constexpr int N = part_comps<S>();
    cx<R> o[N], rv[N];
    if (q.w < part_waves<S>()) {
        load_part<S, R, N>(pin, Vs, s, q.w, o);
        load_part<S, R, N>(rin, Vs, s, q.w, rv);
    }
    bool act = e.c.active != 0;
    double bd = bst;
    auto beta = [&]() {
        TM_MEM_FENCE();  // (the fields are loaded before the sum is waited for)
        if (a.scal_next) {
            bd = e.end(parts, a.npart);
            act = e.go;
        }
        return (R)bd;
    };
    switch (q.w) {
    case 0: dir_hops_fold<0, R, S, G>(geo, a.gauge, pin, rin, s, sh, beta); break;
    case 1: dir_hops_fold<1, R, S, G>(geo, a.gauge, pin, rin, s, sh, beta); break;
    case 2: dir_hops_fold<2, R, S, G>(geo, a.gauge, pin, rin, s, sh, beta); break;
    default: dir_hops_fold<3, R, S, G>(geo, a.gauge, pin, rin, s, sh, beta); break;
    }
    const R tw = (R)a.twist, kap = (R)a.kappa, be = (R)bd;
    if (a.scal_next && q.ws == 0 && q.w == 3) e.write(a.scal_next + q.r, bd);
    __syncthreads();
    if (!act) return;  // uniform over the block: every wave summed the same partials
    if (on)
        for_part<S>(q.w, [&](auto W) {
            constexpr int K0 = W.value * N;
#pragma unroll
            for (int c = 0; c < N; c++) o[c] = rv[c] + be * o[c];
            store_part<S, R, N>(field_rhs<S>(a.pn, Vs, q.r), Vs, q.s, W.value, o);
            o[0] = op_comp<false, false, K0, S>(o[0], sh, kap, tw);
            o[1] = op_comp<false, false, K0 + 1, S>(o[1], sh, kap, tw);
            o[2] = op_comp<false, false, K0 + 2, S>(o[2], sh, kap, tw);
            if constexpr (N == 4) o[3] = op_comp<false, false, K0 + 3, S>(o[3], sh, kap, tw);
            store_part<S, R, N>(field_rhs<S>(a.t, Vs, q.r), Vs, q.s, W.value, o);
        });
    __syncthreads();  // (every wave has read the hops)
    if (q.w < part_waves<S>())
#pragma unroll
        for (int c = 0; c < N; c++) sh[(q.w * N + c) * 64 + (threadIdx.x & 63u)] = o[c];
    __syncthreads();
    norm_partial<R>(sh, on, a.partials + (size_t)q.r * q.nws + q.ws);
}

// K2: q = M^dag t (EO: D^dag t - kappa^2 H_oe^dag y), r -= alpha q, |r|^2, and
// unless XFREE x += alpha p
template <bool EO, typename R, class S, class G, class X, typename RX, bool XFREE>
__global__ __launch_bounds__(256) void k_quad_upd(CgArgs a, EoCg e) {
    __shared__ cx<R> sh[8 * 6 * 64];
    const Geom& geo = a.geo;
    const QuadSite q = quad_site<EO>(geo, a.nrhs);
    StepAlpha sa;
    sa.begin(a, q.r);
    TM_MEM_FENCE();  // (the fields are loaded while the partials are on the way)
    const bool act = sa.active != 0;
    const long Vs = geo.Vs;
    const bool on = q.s < (uint32_t)geo.V;
    const void* gout = EO ? e.godd : a.gauge;
    const void* gin = EO ? e.geven : a.gauge;
    if (on) quad_hops<EO, true, R, S, G>(geo, gout, gin, field_rhs<S>(EO ? e.y : a.t, Vs, q.r), q.s, 1, q.w, sh);
    const R tw = (R)(-a.twist), kap = EO ? (R)(-a.kappa * a.kappa) : (R)a.kappa;
    constexpr int N = part_comps<S>();
    cx<R> o[N], rv[N], pv[N];
    cx<RX> xv[N];
    void* rp = field_rhs<S>(a.r, Vs, q.r);
    void* xp = XFREE ? nullptr : field_rhs<X>(a.x, Vs, q.r);
    if (on && q.w < part_waves<S>()) {
        load_part<S, R, N>(field_rhs<S>(a.t, Vs, q.r), Vs, q.s, q.w, o);
        load_part<S, R, N>(rp, Vs, q.s, q.w, rv);
        if constexpr (!XFREE) {
            static_assert(part_comps<X>() == N, "x in parts of the same components");
            load_part<S, R, N>(field_rhs<S>(a.p, Vs, q.r), Vs, q.s, q.w, pv);
            load_part<X, RX, N>(xp, Vs, q.s, q.w, xv);
        }
    }
    TM_MEM_FENCE();
    const double alpha = sa.end(a, q.r, q.ws == 0 && threadIdx.x == 0);
    const R al = (R)alpha;
    __syncthreads();
    if (!act) return;  // uniform over the block
    if (on)
        for_part<S>(q.w, [&](auto W) {
            constexpr int K0 = W.value * N;
            o[0] = op_comp<EO, true, K0, SF32>(o[0], sh, kap, tw);
            o[1] = op_comp<EO, true, K0 + 1, SF32>(o[1], sh, kap, tw);
            o[2] = op_comp<EO, true, K0 + 2, SF32>(o[2], sh, kap, tw);
            if constexpr (N == 4) o[3] = op_comp<EO, true, K0 + 3, SF32>(o[3], sh, kap, tw);
#pragma unroll
            for (int c = 0; c < N; c++)
                if constexpr (EO)
                    rv[c] = rv[c] - al * o[c];
                else
                    rv[c] = sub_towards<S, R>(rv[c], al, o[c]);
            round_part<S, R, N>(rv);
            store_part<S, R, N>(rp, Vs, q.s, W.value, rv);
            if constexpr (!XFREE) {
                const RX alx = (RX)alpha;
#pragma unroll
                for (int c = 0; c < N; c++)
                    xv[c] = {xv[c].re + alx * (RX)pv[c].re, xv[c].im + alx * (RX)pv[c].im};
                store_part<X, RX, N>(xp, Vs, q.s, W.value, xv);
            }
        });
    __syncthreads();
    if (q.w < part_waves<S>())
#pragma unroll
        for (int c = 0; c < N; c++) sh[(q.w * N + c) * 64 + (threadIdx.x & 63u)] = rv[c];
    __syncthreads();
    norm_partial<R>(sh, on, (a.scal_next ? a.partials2 : a.partials) + (size_t)q.r * q.nws + q.ws);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
// blocks up to which a direction per wave is faster (LP solves, without / with:
// FP32 even-odd 8^4, 4 sources (128 blocks) 336 / 282 us, 12^3 x 24, 4 (1296)
// 466 / 441; FP32 whole lattice 12^3 x 24, 1 (648) 517 / 482, 16^3 x 32, 1
// (2048) 971 / 989)
bool use_quad(int64_t V, int nrhs) { return (V + 63) / 64 * nrhs <= 1536; }

// launches whose K1 finishes the step before (k_quad_mp_fold): those whose
// blocks are all resident at once, one per CU in FP64 and two in FP32.  LP
// solves without / with: FP64 10x12x8x14, 1 source (210 blocks) 376 / 343 us,
// 9x11x7x13, 2 (282) 451 / 468, 10x12x8x14, 2 (420) 465 / 471, 12^3 x 24, 1
// (648) 639 / 733; FP32 9x11x7x13, 1, 3 and 4 (141, 423, 564) 294 / 269, 368 /
// 353 and 408 / 408, 12^3 x 24, 1 and 2 (648, 1296) 419 / 417 and 575 / 620.
bool use_quad_fold(int64_t V, int nrhs, int prec) {
    return (V + 63) / 64 * nrhs <= (prec == P_F64 ? 256 : prec == P_F32 ? 512 : 0);
}

static dim3 quad_grid(const Geom& g, int nrhs) { return dim3((unsigned)((g.V + 63) / 64 * nrhs)); }

template <typename R, class S, class G>
static void quad_lin_typed(hipStream_t st, const EoArgs& a, bool dag) {
    if (dag)
        hipLaunchKernelGGL((k_quad_lin<true, R, S, G>), quad_grid(a.hg, a.nrhs), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_quad_lin<false, R, S, G>), quad_grid(a.hg, a.nrhs), dim3(256), 0, st, a);
}
void launch_quad_lin(hipStream_t st, const EoArgs& a, int prec, bool dag) {
    switch (prec) {
    case P_F64: quad_lin_typed<double, SF64, GF64>(st, a, dag); break;
    case P_F32: quad_lin_typed<float, SF32, GF32>(st, a, dag); break;
    case P_F16: quad_lin_typed<float, SF16, GH16>(st, a, dag); break;
    default: quad_lin_typed<float, SBF16, GF32>(st, a, dag); break;
    }
}

template <bool EO, typename R, class S, class G>
static void quad_mp_typed(hipStream_t st, const CgArgs& a, const EoCg& e) {
    hipLaunchKernelGGL((k_quad_mp<EO, R, S, G>), quad_grid(a.geo, a.nrhs), dim3(256), 0, st, a, e);
}
template <bool EO, typename R, class S, class G, class X, typename RX>
static void quad_upd_typed(hipStream_t st, const CgArgs& a, const EoCg& e, bool xfree) {
    if constexpr (EO ? sizeof(R) == 4 : S::NV == 3) {
        if (xfree) {
            hipLaunchKernelGGL((k_quad_upd<EO, R, S, G, X, RX, true>), quad_grid(a.geo, a.nrhs), dim3(256), 0, st, a, e);
            return;
        }
    }
    hipLaunchKernelGGL((k_quad_upd<EO, R, S, G, X, RX, false>), quad_grid(a.geo, a.nrhs), dim3(256), 0, st, a, e);
}

// e: null for the whole lattice
void launch_quad_mp(hipStream_t st, const CgArgs& a, const EoCg* e, int prec) {
    const EoCg none = {};
    switch (prec) {
    case P_F64:
        e ? quad_mp_typed<true, double, SF64, GF64>(st, a, *e) : quad_mp_typed<false, double, SF64, GF64>(st, a, none);
        break;
    case P_F32:
        e ? quad_mp_typed<true, float, SF32, GF32>(st, a, *e) : quad_mp_typed<false, float, SF32, GF32>(st, a, none);
        break;
    case P_F16:
        e ? quad_mp_typed<true, float, SF16, GH16>(st, a, *e) : quad_mp_typed<false, float, SF16, GF32>(st, a, none);
        break;
    default:
        e ? quad_mp_typed<true, float, SBF16, GF32>(st, a, *e) : quad_mp_typed<false, float, SBF16, GF32>(st, a, none);
        break;
    }
}
// prec: FP64 or FP32
void launch_quad_mp_fold(hipStream_t st, const CgArgs& a, int prec) {
    const dim3 grid = quad_grid(a.geo, a.nrhs);
    if (prec == P_F64)
        hipLaunchKernelGGL((k_quad_mp_fold<double, SF64, GF64>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_quad_mp_fold<float, SF32, GF32>), grid, dim3(256), 0, st, a);
}
void launch_quad_upd(hipStream_t st, const CgArgs& a, const EoCg* e, int prec, bool xfree) {
    const EoCg none = {};
    switch (prec) {
    case P_F64:
        e ? quad_upd_typed<true, double, SF64, GF64, SF64, double>(st, a, *e, xfree)
          : quad_upd_typed<false, double, SF64, GF64, SF64, double>(st, a, none, xfree);
        break;
    case P_F32:
        e ? quad_upd_typed<true, float, SF32, GF32, SF32, float>(st, a, *e, xfree)
          : quad_upd_typed<false, float, SF32, GF32, SF32, float>(st, a, none, xfree);
        break;
    case P_F16:
        e ? quad_upd_typed<true, float, SF16, GH16, SF32, float>(st, a, *e, xfree)
          : quad_upd_typed<false, float, SF16, GF32, SF32, float>(st, a, none, xfree);
        break;
    default:
        e ? quad_upd_typed<true, float, SBF16, GF32, SF32, float>(st, a, *e, xfree)
          : quad_upd_typed<false, float, SBF16, GF32, SF32, float>(st, a, none, xfree);
        break;
    }
}

}  // namespace tmq
