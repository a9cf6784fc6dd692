// Gauge-covariant parallel-transport layers of the learned preconditioner
// (gfx950): forward/adjoint application and the weight gradient.
//
// A layer maps cin spinor fields phi_b to cout fields
//     psi_a(x) = sum_b sum_p W[p][a][b] (T_p phi_b)(x),
// p over nine paths (identity, U_mu(x) phi(x+mu), U_mu(x-mu)^dag phi(x-mu),
// with the time-boundary sign), W[p][a][b] a complex 4x4 spin matrix,
// identity on colour.  The channel/spin mixing is a real GEMM over
// K = 72 cin (path, channel, spin, re/im; padded to 16) on the matrix cores
// (v_mfma_f32_16x16x16_bf16, FP32 accumulation) with the real form of the
// complex weights:
//   * layer application (k_pt_layer): the sites are the GEMM's N side and the
//     transports are computed in registers straight into its B operand (see
//     the comment at the kernel);
//   * weight gradient (k_pt_wgrad): dW = sum_{x,c} g (T_p phi)^dag as the GEMM
//     G^T (16 x rows) A (rows x K) per block of PT_TS sites, A the transports
//     gathered into an LDS tile with rows (colour, site), FP32 block partials
//     reduced in a fixed order.
// The adjoint layer is the same kernel with weights W'[p*][b][a] = W[p][a][b]^dag
// (p* the reversed path), prepared on the host.

#include "tm_device.h"
#include "tm_kernels.h"

namespace tmq {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// weight gradient: 32 sites per block (a 28 KB bfloat16 A tile)
constexpr int PT_TS = 32;             // sites per block
constexpr int PT_ROWS = 3 * PT_TS;    // (colour, site) rows
constexpr int PT_NT = PT_ROWS / 16;   // 16-row MFMA tiles, dealt to the 4 waves
constexpr int PT_KMAX = 144;          // 72 * cin for cin <= 2
constexpr int PT_KP = PT_KMAX + 4;    // LDS row stride (bf16), padded against bank conflicts
constexpr int PT_GP = 16 + 4;         // LDS row stride of the gradient tile

__device__ __forceinline__ uint16_t to_bf16(float f) { return (uint16_t)f32_to_bf16(f); }

// Transport of channel b of `in` along path p, at site s (12 complex, FP32).
template <class Si>
__device__ __forceinline__ void transport_site(const Geom& geo, const void* gauge, const void* in, int b, int p,
                                               uint32_t s, cx<float> v[12]) {
    const void* f = field_rhs<Si>(in, geo.Vs, b);
    if (p == 0) {
        load_spinor<Si, float>(f, geo.Vs, s, v);
        return;
    }
    const int mu = (p - 1) >> 1;
    const bool fwd = (p & 1) != 0;
    const Site c = site_coords(geo, s);
    uint32_t y;
    bool flip;
    switch (mu) {
    case 0: y = fwd ? nb_fwd(geo, s, c, 0) : nb_bwd(geo, s, c, 0); flip = false; break;
    case 1: y = fwd ? nb_fwd(geo, s, c, 1) : nb_bwd(geo, s, c, 1); flip = false; break;
    case 2: y = fwd ? nb_fwd(geo, s, c, 2) : nb_bwd(geo, s, c, 2); flip = false; break;
    default:
        y = fwd ? nb_fwd(geo, s, c, 3) : nb_bwd(geo, s, c, 3);
        flip = geo.t_bc < 0 && (fwd ? (c.t + 1 == geo.L[3]) : (c.t == 0));
        break;
    }
    cx<float> U[3][3], psi[12];
    load_link<GF32, float>(gauge, geo.Vs, mu, fwd ? s : y, U);
    load_spinor<Si, float>(f, geo.Vs, y, psi);
    const float sg = flip ? -1.f : 1.f;
#pragma unroll
    for (int a = 0; a < 4; a++)
#pragma unroll
        for (int i = 0; i < 3; i++) {
            cx<float> t = {0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 3; k++) t = t + (fwd ? U[i][k] * psi[3 * a + k] : cmulc(U[k][i], psi[3 * a + k]));
            v[3 * a + i] = sg * t;
        }
}

// Fill the gradient's A tile: rows (colour c, site i) = c*PT_TS + i, columns
// k = ((p*cin + b)*4 + spin)*2 + re/im, zero-padded to kpad.
template <class Si>
__device__ __forceinline__ void gather_tile(const PtArgs& a, uint32_t site0, uint16_t* As, int kpad) {
    const Geom& geo = a.geo;
    const int nitems = PT_TS * 9 * a.cin;
    for (int item = threadIdx.x; item < nitems; item += 256) {
        const int i = item % PT_TS;
        const int rest = item / PT_TS;
        const int p = rest % 9;
        const int b = rest / 9;
        const uint32_t s = site0 + i;
        cx<float> v[12];
        if (s < geo.V) {
            transport_site<Si>(geo, a.gauge, a.in, b, p, s, v);
        } else {
#pragma unroll
            for (int k = 0; k < 12; k++) v[k] = {0.f, 0.f};
        }
        const int kb = (p * a.cin + b) * 8;
#pragma unroll
        for (int c = 0; c < 3; c++) {
            uint16_t* row = As + (c * PT_TS + i) * PT_KP + kb;
#pragma unroll
            for (int si = 0; si < 4; si++) {
                row[2 * si] = to_bf16(v[3 * si + c].re);
                row[2 * si + 1] = to_bf16(v[3 * si + c].im);
            }
        }
    }
    const int k0 = 72 * a.cin;
    const int kw = kpad - k0;
    if (kw > 0) {
        for (int item = threadIdx.x; item < PT_ROWS * kw; item += 256) {
            const int r = item / kw, k = k0 + item % kw;
            As[r * PT_KP + k] = 0;
        }
    }
}

// ---------------------------------------------------------------------------
// Layer application.  Every wave is independent: it owns 16 consecutive
// sites and loops over the right-hand sides.  The mixing is computed with the
// sites on the N side of the matrix cores,
//     D[out][site] += Wt[out][k] T[k][site]   (v_mfma_f32_16x16x16_bf16),
// one product per colour, so the transports T go from registers straight into
// the B operand: lane l = 16 g + i holds, for site i, the four k = 4g..4g+3 of
// the current k-step, i.e. one (path, channel) and the spin pair 2(g&1),
// 2(g&1)+1.  Each lane therefore transports a half spinor per k-step (18
// complex multiply-adds as bfloat16 dot2 with FP32 accumulation); the link
// comes from a bfloat16-pair copy of the gauge field, through the wave's part
// of LDS.  The D layout gives lane l the output channel g>>1 and the same spin
// pair, which it writes as its half of the output spinor.  No barriers.
// K-steps: for two input channels step ks is path ks (lane channel g>>1); for
// one channel step ks covers paths 2ks and 2ks+1 (lane path 2ks + (g>>1)),
// the tenth "path" being zero padding.
// ---------------------------------------------------------------------------
constexpr int LY_TS = 64;         // sites per block: four waves of 16
constexpr int LY_THREADS = 256;

__device__ __forceinline__ uint4 ldv128(const void* base, uint32_t voff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_of(base), voff, 0, 0));
}
__device__ __forceinline__ uint2 ldv64(const void* base, uint32_t voff) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rsrc_of(base), voff, 0, 0));
}
__device__ __forceinline__ uint32_t ldv32(const void* base, uint32_t voff) {
    return __builtin_amdgcn_raw_buffer_load_b32(rsrc_of(base), voff, 0, 0);
}
// (see st_plane for the wait states after a 128-bit store)
__device__ __forceinline__ void stv128(void* base, uint32_t voff, uint4 val) {
    using V4 = unsigned int __attribute__((ext_vector_type(4)));
    const V4 v = __builtin_bit_cast(V4, val);
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_of(base), voff, 0, 0);
    asm volatile("s_nop 4" ::"v"(v) : "memory");
}
__device__ __forceinline__ void stv64(void* base, uint32_t voff, uint2 val) {
    using V2 = unsigned int __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V2, val), rsrc_of(base), voff, 0, 0);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// acc + a.lo b.lo + a.hi b.hi, bfloat16 pairs, FP32 accumulation (v_dot2_f32_bf16)
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), acc, false);
}
// a.lo b.lo + a.hi b.hi: the three-operand form with a zero accumulator (the
// builtin would first move a zero into a register for the two-operand form)
__device__ __forceinline__ float dot2_0(uint32_t a, uint32_t b) {
    float d;
    asm("v_dot2_f32_bf16 %0, %1, %2, 0" : "=v"(d) : "v"(a), "v"(b));
    return d;
}

// Hidden activations of the network (internal to the layers): bfloat16 pairs
// in three 16-byte planes arranged so that each half spinor is one plane and
// one half plane: plane 0 = components 0-3, plane 1 = 6-9, plane 2 = 4, 5 |
// 10, 11.
struct SBH {
    using V = uint4;
    static constexpr int NV = 3;
};
__device__ __forceinline__ uint32_t swap16(uint32_t x) { return __builtin_amdgcn_alignbit(x, x, 16); }

// The lane's half spinor (components 6h .. 6h+5, spins 2h and 2h+1) of channel
// b at site y: the loads, and later its bfloat16 (re, im) pairs.
template <class Si>
struct HalfRaw {  // 16-bit: one plane and half of another
    uint4 full;
    uint2 half;
    __device__ __forceinline__ void load(const void* f, uint32_t PB, int b, uint32_t y, int h) {
        const uint32_t base = (y << 4) + (uint32_t)b * 3u * PB;
        if constexpr (std::is_same<Si, SBH>::value) {
            full = ldv128(f, base + (uint32_t)h * PB);
            half = ldv64(f, base + 2u * PB + (uint32_t)h * 8u);
        } else {
            // planes of 4 components: h = 0 -> plane 0 + low half of plane 1; h = 1 -> high half of plane 1 + plane 2
            full = ldv128(f, base + (h ? 2u * PB : 0u));
            half = ldv64(f, base + PB + (h ? 8u : 0u));
        }
    }
    __device__ __forceinline__ void pairs(int h, uint32_t q[6]) const {
        if constexpr (std::is_same<Si, SBH>::value) h = 0;
        q[0] = h ? half.x : full.x;
        q[1] = h ? half.y : full.y;
        q[2] = h ? full.x : full.z;
        q[3] = h ? full.y : full.w;
        q[4] = h ? full.z : half.x;
        q[5] = h ? full.w : half.y;
    }
};
template <>
struct HalfRaw<SF32> {  // planes of 2 components: planes 3h, 3h+1, 3h+2
    uint4 v[3];
    __device__ __forceinline__ void load(const void* f, uint32_t PB, int b, uint32_t y, int h) {
        const uint32_t base = (y << 4) + (uint32_t)b * 6u * PB + (uint32_t)h * 3u * PB;
#pragma unroll
        for (int j = 0; j < 3; j++) v[j] = ldv128(f, base + (uint32_t)j * PB);
    }
    __device__ __forceinline__ void pairs(int, uint32_t q[6]) const {
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const float4 w = __builtin_bit_cast(float4, v[j]);
            q[2 * j] = pack2_bf16(w.x, w.y);
            q[2 * j + 1] = pack2_bf16(w.z, w.w);
        }
    }
};

// Per-lane description of the (path, channel) of one k-step.
struct LyPath {
    uint32_t y;      // neighbour site
    uint32_t link;   // link of the path (0 ... 7: +-x, +-y, +-z, +-t)
    uint32_t flip;   // 0x80008000 where the time-boundary sign applies
    bool ident, pad;
};

template <int P>
__device__ __forceinline__ LyPath ly_path(const uint32_t ys[9], uint32_t flip_f, uint32_t flip_b) {
    LyPath d;
    d.pad = P >= 9;
    d.ident = P == 0;
    d.y = (P >= 1 && P <= 8) ? ys[P] : ys[0];
    d.link = (P >= 1 && P <= 8) ? (uint32_t)(P - 1) : 0u;  // identity and padding read direction 0's link
    d.flip = P == 7 ? flip_f : P == 8 ? flip_b : 0u;
    return d;
}
__device__ __forceinline__ LyPath ly_select(bool hi, const LyPath& a, const LyPath& b) {
    LyPath d;
    d.y = hi ? b.y : a.y;
    d.link = hi ? b.link : a.link;
    d.flip = hi ? b.flip : a.flip;
    d.ident = hi ? b.ident : a.ident;
    d.pad = hi ? b.pad : a.pad;
    return d;
}

// The eight links of a wave's 16 sites in LDS, [link][plane][site], each entry
// V of the oriented link (U_mu(x), or U_mu(x - mu)^dag) as the two bfloat16
// pairs that a product with (re, im) takes: dword e: (Re V, -Im V) for the real
// part, dword 9 + e: (Im V, Re V) for the imaginary part, e = 3 c + k.  Lane
// 16 g + i prepares links g and 4 + g of site i.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
constexpr int LY_LP = 5;  // planes of 16 bytes per link (18 dwords)
__device__ __forceinline__ void ly_stage_links(const PtArgs& a, uint32_t PB, const uint32_t ys[9], int g, int i,
                                               v4u* sl) {
    const bool bwd = (g & 1) != 0;  // (link l: mu = l >> 1, backward if odd)
    const uint32_t mb = bwd ? ~0u : 0u;
    uint4 u0[2], u1[2];
    uint32_t u8[2];
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const int l = 4 * it + g;
        // (selections by mask: the compiler turns selected array elements into addresses in scratch)
        const uint32_t yb = ys[4 + 4 * it] ^ ((ys[2 + 4 * it] ^ ys[4 + 4 * it]) & (g == 1 ? ~0u : 0u));
        const uint32_t off = ((ys[0] ^ ((ys[0] ^ yb) & mb)) << 4) + (uint32_t)((l >> 1) * 3) * PB;
        u0[it] = ldv128(a.gaugebf, off);
        u1[it] = ldv128(a.gaugebf, off + PB);
        u8[it] = ldv32(a.gaugebf, off + 2u * PB);
    }
#pragma unroll
    for (int it = 0; it < 2; it++) {
        const uint32_t u[9] = {u0[it].x, u0[it].y, u0[it].z, u0[it].w, u1[it].x, u1[it].y, u1[it].z, u1[it].w, u8[it]};
        const uint32_t s1 = bwd ? 0u : 0x80000000u, s2 = bwd ? 0x8000u : 0u;
        uint32_t w[4 * LY_LP];
#pragma unroll
        for (int c = 0; c < 3; c++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const uint32_t uf = u[3 * c + k], ub = u[3 * k + c], v = uf ^ ((uf ^ ub) & mb);
                w[3 * c + k] = v ^ s1;
                w[9 + 3 * c + k] = swap16(v) ^ s2;
            }
        w[18] = w[19] = 0u;
#pragma unroll
        for (int q = 0; q < LY_LP; q++)
            sl[((4 * it + g) * LY_LP + q) * 16 + i] = (v4u){w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
    }
    // read by the same wave only: its LDS accesses stay in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The link of a k-step, prepared by ly_stage_links
__device__ __forceinline__ void ly_link(const v4u* sl, int i, const LyPath& d, v4u m[LY_LP]) {
    const v4u* p = sl + d.link * (16u * LY_LP) + (uint32_t)i;
#pragma unroll
    for (int q = 0; q < LY_LP; q++) m[q] = p[16 * q];
}

// B operand of one k-step and one right-hand side for the three colours: the
// lane's two spins of the transported (or, for the identity path, the plain)
// half spinor.
template <class Si>
__device__ __forceinline__ void ly_operand(const HalfRaw<Si>& raw, int h, const LyPath& d, const v4u mv[LY_LP],
                                           uint32_t B[3][2]) {
    uint32_t q[6], m[4 * LY_LP];
#pragma unroll
    for (int e = 0; e < 4 * LY_LP; e++) m[e] = mv[e >> 2][e & 3];
    raw.pairs(h, q);
#pragma unroll
    for (int c = 0; c < 3; c++)
#pragma unroll
        for (int t = 0; t < 2; t++) {
            float tr = dot2_0(q[3 * t], m[3 * c]), ti = dot2_0(q[3 * t], m[9 + 3 * c]);
            tr = dot2(q[3 * t + 1], m[3 * c + 1], tr);
            ti = dot2(q[3 * t + 1], m[9 + 3 * c + 1], ti);
            tr = dot2(q[3 * t + 2], m[3 * c + 2], tr);
            ti = dot2(q[3 * t + 2], m[9 + 3 * c + 2], ti);
            // (the time-boundary sign here, not in the link: a dot2 of negated
            // products is not always the negative of the dot2)
            const uint32_t tv = pack2_bf16(tr, ti) ^ d.flip;
            B[c][t] = d.pad ? 0u : d.ident ? q[3 * t + c] : tv;
        }
}

// Right-hand sides go through the wave two at a time (a link read from LDS
// serves both, the MFMA accumulators of both stay live), and a block of 64
// sites handles up to LY_PER of them.  What bounds the layer is the traffic
// between L2 and the memory side: a lane reads nine half spinors and writes
// one, and when a block handled two right-hand sides and every wave read its
// links for itself, four times over, the links were half of the traffic and
// every k-step waited for its loads.  Hence
//   * the links of the 16 sites are staged in LDS once per block, already
//     oriented, conjugated and signed for the two dot products of a complex
//     multiply (per half spinor 36 dot2 and 6 conversions are left);
//   * the half spinors of a k-step are loaded while the one before is computed;
//   * four right-hand sides per block, sites in slab order.
// 16 right-hand sides on 16^3 x 32: layer 2 -> 2 channels 254 -> 190 us,
// 2 -> 1 240 -> 185 us, 1 -> 2 206 -> 135 us (2 right-hand sides per block:
// 202 us for 2 -> 2; 8 and 16: 195; two k-steps ahead: 203; one right-hand
// side at a time with four waves per SIMD: 195).
constexpr uint32_t LY_PER = 4;

// What one wave knows of its 16 sites
struct LyWave {
    uint32_t ys[9];   // the site and its neighbours
    uint32_t sout;    // site to store (~0: past the lattice)
    uint32_t flip_f, flip_b;  // time-boundary sign of its forward and backward time hop
    int g, i;         // lane = 16 g + i
    const v4u* sl;    // links in LDS
};

template <int CIN, int KS>
__device__ __forceinline__ LyPath ly_step(const LyWave& w) {
    if constexpr (CIN == 2)
        return ly_path<KS>(w.ys, w.flip_f, w.flip_b);
    else
        return ly_select((w.g >> 1) != 0, ly_path<2 * KS>(w.ys, w.flip_f, w.flip_b),
                         ly_path<2 * KS + 1>(w.ys, w.flip_f, w.flip_b));
}

template <class Si, int CIN, int KS, int NKS, int NRC>
__device__ __forceinline__ void ly_loads(const PtArgs& a, const LyWave& w, uint32_t PB, uint32_t r0,
                                         HalfRaw<Si> raw[2][NRC]) {
    if constexpr (KS < NKS) {
        const LyPath d = ly_step<CIN, KS>(w);
#pragma unroll
        for (int j = 0; j < NRC; j++)
            raw[KS & 1][j].load(field_rhs<Si>(a.in, a.geo.Vs, (int)((r0 + j) * CIN)), PB,
                                            CIN == 2 ? w.g >> 1 : 0, d.y, w.g & 1);
        __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink the loads to their use)
    }
}

// k-steps KS ... NKS - 1; raw[KS & 1] and m hold step KS
template <class Si, int CIN, int KS, int NKS, int NRC>
__device__ __forceinline__ void ly_steps(const PtArgs& a, const LyWave& w, uint32_t PB, uint32_t r0,
                                         const v4s wf[NKS], HalfRaw<Si> raw[2][NRC],
                                         const v4u m[LY_LP], v4f D[NRC][3]) {
    v4u mn[LY_LP];
    if constexpr (KS + 1 < NKS) ly_link(w.sl, w.i, ly_step<CIN, KS + 1>(w), mn);
    ly_loads<Si, CIN, KS + 1, NKS, NRC>(a, w, PB, r0, raw);
    const LyPath d = ly_step<CIN, KS>(w);
#pragma unroll
    for (int j = 0; j < NRC; j++) {
        uint32_t B[3][2];
        ly_operand<Si>(raw[KS & 1][j], w.g & 1, d, m, B);
#pragma unroll
        for (int c = 0; c < 3; c++) {
            const v4s bo = __builtin_bit_cast(v4s, make_uint2(B[c][0], B[c][1]));
            D[j][c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wf[KS], bo, D[j][c], 0, 0, 0);
        }
    }
    if constexpr (KS + 1 < NKS) ly_steps<Si, CIN, KS + 1, NKS, NRC>(a, w, PB, r0, wf, raw, mn, D);
}

// NRC right-hand sides from r0 on
template <class Si, class So, int CIN, int COUT, int NKS, int NRC>
__device__ __forceinline__ void ly_chunk(const PtArgs& a, const LyWave& w, uint32_t PB, uint32_t r0,
                                         const v4s wf[NKS]) {
    const long Vs = a.geo.Vs;
    const int g = w.g, h = g & 1;
    const uint32_t s = w.sout;
    v4f D[NRC][3];
#pragma unroll
    for (int j = 0; j < NRC; j++)
#pragma unroll
        for (int c = 0; c < 3; c++) D[j][c] = (v4f){0.f, 0.f, 0.f, 0.f};
    HalfRaw<Si> raw[2][NRC];
    ly_loads<Si, CIN, 0, NKS, NRC>(a, w, PB, r0, raw);
    v4u m[LY_LP];
    ly_link(w.sl, w.i, ly_step<CIN, 0>(w), m);
    ly_steps<Si, CIN, 0, NKS, NRC>(a, w, PB, r0, wf, raw, m, D);
    // lane holds channel g>>1, spins 2h and 2h+1: component 6h + 3t + c is
    // (D[c][2t], D[c][2t + 1])
    const int ch = g >> 1;
    if (s == ~0u || ch >= COUT) return;
#pragma unroll
    for (int j = 0; j < NRC; j++) {
        void* out = field_rhs<So>(a.out, Vs, (int)((r0 + j) * COUT));
        float o[12];
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
            for (int c = 0; c < 3; c++) {
                o[2 * (3 * t + c)] = D[j][c][2 * t];
                o[2 * (3 * t + c) + 1] = D[j][c][2 * t + 1];
            }
        if constexpr (std::is_same<So, SBH>::value) {
            uint32_t w[6];
#pragma unroll
            for (int q = 0; q < 6; q++) w[q] = pack2_bf16(o[2 * q], o[2 * q + 1]);
            const uint32_t base = (s << 4) + (uint32_t)ch * 3u * PB;
            stv128(out, base + (uint32_t)h * PB, make_uint4(w[0], w[1], w[2], w[3]));
            stv64(out, base + 2u * PB + (uint32_t)h * 8u, make_uint2(w[4], w[5]));
        } else if constexpr (std::is_same<So, SF32>::value) {
            const uint32_t base = (s << 4) + (uint32_t)ch * 6u * PB + (uint32_t)h * 3u * PB;
#pragma unroll
            for (int q = 0; q < 3; q++)
                stv128(out, base + (uint32_t)q * PB,
                       make_uint4(__float_as_uint(o[4 * q]), __float_as_uint(o[4 * q + 1]),
                                  __float_as_uint(o[4 * q + 2]), __float_as_uint(o[4 * q + 3])));
        } else {
            static_assert(std::is_same<So, SF32>::value || std::is_same<So, SBH>::value, "FP32 or SBH output");
        }
    }
}

template <class Si, class So, int CIN, int COUT>
__global__ __launch_bounds__(LY_THREADS) __attribute__((amdgpu_waves_per_eu(std::is_same<Si, SF32>::value ? 2 : 3))) void k_pt_layer(PtArgs a, uint32_t nrhs,
                                                                               uint32_t per) {
    constexpr int NKS = (9 * CIN + 1) / 2;  // k-steps of 16
    const Geom& geo = a.geo;
    const uint32_t PB = (uint32_t)geo.Vs * 16u;  // plane bytes
    const int lane = threadIdx.x & 63, g = lane >> 4;
    // blocks: (right-hand-side chunk, site tile), chunk slowest
    const uint32_t ntile = (geo.V + LY_TS - 1) / LY_TS;
    const uint32_t L = xcd_block(blockIdx.x, gridDim.x);
    const uint32_t chunk = L / ntile, tile = L - chunk * ntile;
    const uint32_t r_beg = chunk * per;
    const uint32_t r_end = r_beg + per < nrhs ? r_beg + per : nrhs;
    // flexible CG: nothing to do for converged or fallen-back right-hand sides
    uint32_t live = 0;
    for (uint32_t r = r_beg; r < r_end; r++)
        live |= (!a.gate || (a.gate[r].active != 0 && a.gate[r].fell == 0)) ? 1u << (r - r_beg) : 0u;
    if (!live) return;
    const uint32_t s0 = tile * LY_TS + (threadIdx.x >> 6) * 16 + (lane & 15);
    const bool valid = s0 < geo.V;
    const uint32_t s = valid ? slab_order(geo, s0) : 0u;  // lanes past the lattice compute site 0 and store nothing

    LyWave w;
    w.g = g;
    w.i = lane & 15;
    w.sout = valid ? s : ~0u;
    w.flip_f = w.flip_b = 0;
    uint32_t* ys = w.ys;
    {
        const Site c = site_coords(geo, s);
        ys[0] = s;
#pragma unroll
        for (int mu = 0; mu < 4; mu++) {
            ys[1 + 2 * mu] = nb_fwd(geo, s, c, mu);
            ys[2 + 2 * mu] = nb_bwd(geo, s, c, mu);
        }
        if (geo.t_bc < 0) {
            w.flip_f = (c.t + 1 == geo.L[3]) ? 0x80008000u : 0u;
            w.flip_b = (c.t == 0) ? 0x80008000u : 0u;
        }
    }
    __shared__ v4u links[LY_THREADS / 64][8 * LY_LP * 16];
    v4u* sl = links[threadIdx.x >> 6];
    ly_stage_links(a, PB, ys, g, lane & 15, sl);
    w.sl = sl;
    v4s wf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ks++) wf[ks] = ((const v4s*)a.wfrag)[ks * 64 + lane];

    uint32_t r0 = r_beg;
    for (; r0 + 2 <= r_end; r0 += 2, live >>= 2)
        if (live & 3u) ly_chunk<Si, So, CIN, COUT, NKS, 2>(a, w, PB, r0, wf);
    if (live & 1u) ly_chunk<Si, So, CIN, COUT, NKS, 1>(a, w, PB, r0, wf);
}

// Weight gradient of one layer for one right-hand side: block partials of
// C[m][k] = sum_rows G[row][m] A[row][k], m = (out channel, spin, re/im).
template <class Si, class Sg>
__global__ __launch_bounds__(256) void k_pt_wgrad(PtArgs a) {
    __shared__ __attribute__((aligned(16))) uint16_t As[PT_ROWS * PT_KP];
    __shared__ __attribute__((aligned(16))) uint16_t Gs[PT_ROWS * PT_GP];
    const uint32_t blk = blockIdx.x;
    const uint32_t site0 = blk * PT_TS;
    const int kpad = a.kpad;
    gather_tile<Si>(a, site0, As, kpad);
    for (int item = threadIdx.x; item < PT_TS * 2; item += 256) {
        const int i = item % PT_TS, ch = item / PT_TS;
        const uint32_t s = site0 + i;
        cx<float> g[12];
        if (ch < a.cout && s < a.geo.V) {
            load_spinor<Sg, float>(field_rhs<Sg>(a.g, a.geo.Vs, ch), a.geo.Vs, s, g);
        } else {
#pragma unroll
            for (int k = 0; k < 12; k++) g[k] = {0.f, 0.f};
        }
#pragma unroll
        for (int c = 0; c < 3; c++)
#pragma unroll
            for (int so = 0; so < 4; so++) {
                Gs[(c * PT_TS + i) * PT_GP + (ch * 4 + so) * 2] = to_bf16(g[3 * so + c].re);
                Gs[(c * PT_TS + i) * PT_GP + (ch * 4 + so) * 2 + 1] = to_bf16(g[3 * so + c].im);
            }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int nct = kpad / 16;
    for (int ct = w; ct < nct; ct += 4) {
        v4f acc = (v4f){0.f, 0.f, 0.f, 0.f};
        for (int ks = 0; ks < PT_ROWS / 16; ks++) {
            v4s af, bf;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int row = ks * 16 + 4 * (lane >> 4) + j;
                af[j] = (short)Gs[row * PT_GP + (lane & 15)];
                bf[j] = (short)As[row * PT_KP + ct * 16 + (lane & 15)];
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af, bf, acc, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; j++)
            a.partials[((size_t)blk * 16 + 4 * (lane >> 4) + j) * kpad + ct * 16 + (lane & 15)] = acc[j];
    }
}

// grad[m][k] += scale * sum over blocks of partials, FP64, in two coalesced
// stages with a fixed order: chunk sums of WG_CH block partials, then the sum
// of the chunk sums.
constexpr int WG_CH = 256;
__global__ __launch_bounds__(256) void k_pt_wgrad_sum1(const float* partials, int nblocks, int ne, double* part2) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= ne) return;
    const int b0 = blockIdx.y * WG_CH, b1 = min(b0 + WG_CH, nblocks);
    double s = 0;
    for (int b = b0; b < b1; b++) s += (double)partials[(size_t)b * ne + e];
    part2[(size_t)blockIdx.y * ne + e] = s;
}
__global__ __launch_bounds__(256) void k_pt_wgrad_sum2(const double* part2, int nchunk, int ne, const double* scale,
                                                       double* grad) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= ne) return;
    double s = 0;
    for (int c = 0; c < nchunk; c++) s += part2[(size_t)c * ne + e];
    grad[e] += (*scale) * s;
}

// Output error of a training pair: g = y - e (FP32 field), block partials of
// |y - e|^2 and |e|^2; k_pt_loss_fin turns them into the pair's loss share
// and gradient scale.
template <class Se>
__global__ __launch_bounds__(256) void k_pt_loss(Geom geo, const void* y, const void* e, void* g, double* partials) {
    __shared__ double sh[4];
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    double pd = 0, pe = 0;
    if (s < geo.V) {
        cx<float> yv[12], ev[12], gv[12];
        load_spinor<SF32, float>(y, geo.Vs, s, yv);
        load_spinor<Se, float>(e, geo.Vs, s, ev);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            gv[k] = yv[k] - ev[k];
            pd += (double)gv[k].re * gv[k].re + (double)gv[k].im * gv[k].im;
            pe += (double)ev[k].re * ev[k].re + (double)ev[k].im * ev[k].im;
        }
        store_spinor<SF32, float>(g, geo.Vs, s, gv);
    }
    const uint32_t nb = gridDim.x;
    double v = block_sum256(pd, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = v;
    double u = block_sum256(pe, sh);
    if (threadIdx.x == 0) partials[nb + blockIdx.x] = u;
}

// one block: the pair's gradient scale 1 / (|e|^2 npairs) into scal[0], its
// relative error into scal[1], and its loss share added to scal[2]
__global__ __launch_bounds__(256) void k_pt_loss_fin(const double* partials, uint32_t nb, double* scal, int npairs) {
    __shared__ double sh[4];
    double d = 0, e = 0;
    for (uint32_t i = threadIdx.x; i < nb; i += 256) {
        d += partials[i];
        e += partials[nb + i];
    }
    const double d2 = block_sum256(d, sh);
    const double e2 = block_sum256(e, sh);
    if (threadIdx.x == 0) {
        scal[0] = 1.0 / (e2 * npairs);
        scal[1] = d2 / e2;
        scal[2] += d2 / e2 / npairs;
    }
}

template <class Si, class So>
static void launch_pt_layer_t(hipStream_t st, const PtArgs& a, int nrhs) {
    // small lattices: fewer right-hand sides per block while the launch holds
    // less than three blocks per CU
    const unsigned ntile = (unsigned)((a.geo.V + LY_TS - 1) / LY_TS);
    uint32_t per = LY_PER;
    auto nchunk = [&] { return ((unsigned)nrhs + per - 1) / per; };
    while (per > 1 && ntile * nchunk() < 768u) per >>= 1;
    const dim3 grid(ntile * nchunk()), blk(LY_THREADS);
    const uint32_t n = (uint32_t)nrhs;
    if (a.cin == 1 && a.cout == 1) hipLaunchKernelGGL((k_pt_layer<Si, So, 1, 1>), grid, blk, 0, st, a, n, per);
    else if (a.cin == 1) hipLaunchKernelGGL((k_pt_layer<Si, So, 1, 2>), grid, blk, 0, st, a, n, per);
    else if (a.cout == 1) hipLaunchKernelGGL((k_pt_layer<Si, So, 2, 1>), grid, blk, 0, st, a, n, per);
    else hipLaunchKernelGGL((k_pt_layer<Si, So, 2, 2>), grid, blk, 0, st, a, n, per);
}

void launch_pt_layer(hipStream_t st, const PtArgs& a, int in_prec, int out_prec, int nrhs) {
    const bool ob = out_prec == P_BH;
    if (in_prec == P_BH) {
        if (ob) launch_pt_layer_t<SBH, SBH>(st, a, nrhs);
        else launch_pt_layer_t<SBH, SF32>(st, a, nrhs);
    } else if (in_prec == P_BF16) {
        if (ob) launch_pt_layer_t<SBF16, SBH>(st, a, nrhs);
        else launch_pt_layer_t<SBF16, SF32>(st, a, nrhs);
    } else {
        if (ob) launch_pt_layer_t<SF32, SBH>(st, a, nrhs);
        else launch_pt_layer_t<SF32, SF32>(st, a, nrhs);
    }
}

void launch_pt_wgrad(hipStream_t st, const PtArgs& a, int in_prec, const double* scale, double* grad) {
    const int nb = (int)((a.geo.V + PT_TS - 1) / PT_TS);
    if (in_prec == P_BF16)
        hipLaunchKernelGGL((k_pt_wgrad<SBF16, SF32>), dim3(nb), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_pt_wgrad<SF32, SF32>), dim3(nb), dim3(256), 0, st, a);
    const int ne = 16 * a.kpad, nchunk = (nb + WG_CH - 1) / WG_CH;
    hipLaunchKernelGGL(k_pt_wgrad_sum1, dim3((ne + 255) / 256, nchunk), dim3(256), 0, st, a.partials, nb, ne, a.partials2);
    hipLaunchKernelGGL(k_pt_wgrad_sum2, dim3((ne + 255) / 256), dim3(256), 0, st, a.partials2, nchunk, ne, scale, grad);
}

void launch_pt_loss(hipStream_t st, const Geom& g, const void* y, const void* e, int e_prec, void* gout,
                    double* partials, double* scal, int npairs) {
    const unsigned nb = (unsigned)((g.V + 255) / 256);
    if (e_prec == P_BF16)
        hipLaunchKernelGGL((k_pt_loss<SBF16>), dim3(nb), dim3(256), 0, st, g, y, e, gout, partials);
    else
        hipLaunchKernelGGL((k_pt_loss<SF32>), dim3(nb), dim3(256), 0, st, g, y, e, gout, partials);
    hipLaunchKernelGGL(k_pt_loss_fin, dim3(1), dim3(256), 0, st, partials, nb, scal, npairs);
}

int pt_blocks(const Geom& g) { return (int)((g.V + PT_TS - 1) / PT_TS); }
int pt_chunks(const Geom& g) { return (pt_blocks(g) + WG_CH - 1) / WG_CH; }

// Training pair from an iterate x_k: r = eta - M x_k, e = x* - x_k (FP64
// arithmetic, stored as bfloat16); eta regenerated from the hash.
__global__ __launch_bounds__(256) void k_make_pair(Geom geo, uint64_t seed_mixed, const uint64_t* id, const void* xk,
                                                   const void* xstar, const void* mxk, void* r_out, void* e_out) {
    const uint32_t s = blockIdx.x * 256u + threadIdx.x;
    if (s >= geo.V) return;
    cx<double> x[12], xs[12], mx[12];
    load_spinor<SF64, double>(xk, geo.Vs, s, x);
    load_spinor<SF64, double>(xstar, geo.Vs, s, xs);
    load_spinor<SF64, double>(mxk, geo.Vs, s, mx);
    const uint64_t h = noise_bits(seed_mixed, *id, (uint64_t)geo.V, (uint64_t)s);
    cx<float> r[12], e[12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const cx<double> eta = z4_value<double>((uint32_t)(h >> (2 * k)) & 3u);
        const cx<double> rv = eta - mx[k], ev = xs[k] - x[k];
        r[k] = {(float)rv.re, (float)rv.im};
        e[k] = {(float)ev.re, (float)ev.im};
    }
    store_spinor<SBF16, float>(r_out, geo.Vs, s, r);
    store_spinor<SBF16, float>(e_out, geo.Vs, s, e);
}

void launch_make_pair(hipStream_t st, const Geom& g, uint64_t seed_mixed, const uint64_t* id, const void* xk,
                      const void* xstar, const void* mxk, void* r_out, void* e_out) {
    hipLaunchKernelGGL(k_make_pair, dim3((unsigned)((g.V + 255) / 256)), dim3(256), 0, st, g, seed_mixed, id, xk, xstar,
                       mxk, r_out, e_out);
}

}  // namespace tmq
