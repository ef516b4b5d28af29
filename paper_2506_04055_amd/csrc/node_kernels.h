// The node kernels (node_dims.h says what they do and what bounds them).
#pragma once
#include "node_dims.h"

namespace mlp {

typedef ec_v4f v4f;

// ---------------------------------------------------------------------------
// Device
// ---------------------------------------------------------------------------

// A row-major array seen from a workgroup: element (this lane's row, feature
// 16 t + 4 g + r).  The row offset is relative to the workgroup's first row,
// so that loads take (uniform base, 32-bit offset).
struct NdRow {
    float *p;
    unsigned o;
    __device__ __forceinline__ v4f ld(int t) const { return *reinterpret_cast<const v4f *>(p + (o + 16u * t)); }
    __device__ __forceinline__ void st(int t, v4f x) const { *reinterpret_cast<v4f *>(p + (o + 16u * t)) = x; }
};

struct NdLane {
    int n, row0, rel, g;   // rows, the workgroup's first, this lane's in it (clamped), its lane group
    bool ok;
    __device__ __forceinline__ NdLane(int n_, int rows) {
        n = n_;
        row0 = blockIdx.x * rows;
        g = (threadIdx.x & 63) >> 4;
        const int m = row0 + 16 * (threadIdx.x >> 6) + (threadIdx.x & 15);
        ok = m < n;
        rel = min(m, n - 1) - row0;
    }
    // rows of ld floats
    __device__ __forceinline__ NdRow row(const float *a, int ld) const {
        return {const_cast<float *>(a) + (long)row0 * ld, (unsigned)(rel * ld + 4 * g)};
    }
    // row 3 m + d of a vector array
    __device__ __forceinline__ NdRow vec(const float *a, int F, int d) const {
        return {const_cast<float *>(a) + (3L * row0 + d) * F, (unsigned)(rel * 3 * F + 4 * g)};
    }
    // tile t of a vector staged in LDS
    __device__ __forceinline__ v4f vecl(const float *b, int t) const { return *reinterpret_cast<const v4f *>(b + 16 * t + 4 * g); }
};

// operand of block s from an array of NT tiles
template <int P, int NT, class G>
__device__ __forceinline__ EcOp<P> nd_op(int s, G get) {
    const v4f z = {0.f, 0.f, 0.f, 0.f};
    return ec_op<P>(get(2 * s), 2 * s + 1 < NT ? get(2 * s + 1) : z);
}

// Uv, Vv of one direction, tile by tile: f(t, Uv, Vv)
template <int P, int F, class S, class X, class Fn>
__device__ __forceinline__ void nd_uv(S &st, const X &raw, Fn f) {
    using D = NodeDim<F>;
    EcOp<P> x[D::KS];
#pragma unroll
    for (int s = 0; s < D::KS; s++) x[s] = nd_op<P, D::NT>(s, [&](int t) { return raw[t]; });
    ec_for<D::NT>([&](auto t_) __attribute__((always_inline)) {
        constexpr int T = decltype(t_)::value;
        v4f a[2] = {};
        ec_layer<2 * T * D::KS, 2, D::KS>(st, a, [&](auto s) { return x[s]; });
        f(T, a[0], a[1]);
    });
}

// Computed here: without it a value is formed where it is used, and its
// operands stay in registers up to there instead.
__device__ __forceinline__ void nd_here(v4f &x) {
#pragma unroll
    for (int r = 0; r < 4; r++) asm volatile("" : "+v"(x[r]));
}

// SiLU and its derivative with the divided sigmoid: the reciprocal's error
// would show in a large system's energy.
__device__ __forceinline__ float nd_sigmoid(float x) { return 1.0f / (1.0f + __expf(-x)); }
__device__ __forceinline__ v4f nd_silu(v4f x) {
    v4f o;
#pragma unroll
    for (int r = 0; r < 4; r++) o[r] = x[r] * nd_sigmoid(x[r]);
    return o;
}
__device__ __forceinline__ v4f nd_dsilu(v4f x) {
    v4f o;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        const float s = nd_sigmoid(x[r]);
        o[r] = s * (1.0f + x[r] * (1.0f - s));
    }
    return o;
}

// Biases go to LDS first: read from global memory in the chain, each would
// wait for the stores issued before it (one counter, in order).
__device__ __forceinline__ void nd_stage(float *d, const float *b, int n, int pad) {
    for (int q = threadIdx.x; q < pad; q += blockDim.x) d[q] = q < n ? b[q] : 0.f;
}

// Waves of a workgroup that take 16 atoms each; one more fetches the weights.
// The ring is what two workgroups (NC = 3) leave room for in 160 KB.
constexpr int nd_ring(int P, int NC) { return P == 0 ? (NC == 3 ? 3 : 4) : 4; }
template <int NC>
__device__ __forceinline__ bool nd_fetcher() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == NC; }
// weights read a pair ahead where the registers allow it
constexpr bool nd_pre(int P, int F, bool fwd) { return (F == 64 && P) || (F == 128 && P && !fwd); }
template <int P, int F, int NC, bool FWD>
using NdRing = EcRing<P, nd_ring(P, NC), nd_pre(P, F, FWD)>;
constexpr int ND_EU = 2;
// Rows from which workgroups have seven waves of atoms instead of three (two
// workgroups per compute unit, whose phases overlap): the weights are then
// fetched less than half as often, 3 - 6 % of a launch at 1.2M rows, but few
// rows make few workgroups, whose last round is nearly empty.  The node kernels
// of an evaluation, three against seven waves: split bf16, F = 128: 23,000 rows
// 455 and 493 us, 49,000 896 and 964, 98,000 1,743 and 1,903, 131,000 2,342 and
// 2,394, 256,000 4,455 and 4,418, 389,000 6,864 and 6,818; FP32: 49,000 1,341
// and 1,464, 98,000 2,675 and 2,927, 256,000 6,958 and 7,048.  F = 64, split:
// 49,000 461 and 511, 98,000 881 and 957, 171,000 1,509 and 1,523; FP32:
// 256,000 2,949 and 2,905.  Above the line the two stay within 3 % of each
// other to 400,000 rows.
constexpr int ND_LARGE = 100000;

template <int P, int F, int NC>
__global__ void __launch_bounds__(64 * (NC + 1)) __attribute__((amdgpu_waves_per_eu(ND_EU))) k_node_fwd(NodeArgs A) {
    using D = NodeDim<F>;
    using Ring = NdRing<P, F, NC, true>;
    constexpr int NT = D::NT, KS = D::KS, SB = Ring::SB;
    __shared__ __attribute__((aligned(16))) char lds[nd_ring(P, NC) * SB];
    __shared__ __attribute__((aligned(16))) float b1[F], b2[3 * F], b3[F], b4[3 * F];
    nd_stage(b1, A.b1, F, F);
    nd_stage(b2, A.b2, 3 * F, 3 * F);
    nd_stage(b3, A.b3, F, F);
    nd_stage(b4, A.b4, 3 * F, 3 * F);   // (published by the chain's first barrier)
    if (nd_fetcher<NC>()) {
        Ring::produce(lds, reinterpret_cast<const char *>(A.chain), 3 * D::SA + D::SF, D::SA, D::SA, -1, 0);
        return;
    }
    Ring st;
    st.start(lds);
    const NdLane L(A.n, 16 * NC);
    const NdRow s1 = L.row(A.s1, A.ld1);
    v4f n2[NT], dot[NT], uv[3][NT], h[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) {
        n2[t] = v4f{A.eps, A.eps, A.eps, A.eps};
        dot[t] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    // (the next direction's rows are loaded ahead where the registers allow it)
    v4f nx[F <= 64 ? NT : 1];
    auto ahead = [&](int d) __attribute__((always_inline)) {
        if constexpr (F <= 64)
#pragma unroll
            for (int t = 0; t < NT; t++) nx[t] = L.vec(A.v1, F, d).ld(t);
    };
    ahead(0);
#pragma unroll
    for (int d = 0; d < 3; d++) {
#pragma unroll
        for (int t = 0; t < NT; t++) {
            if constexpr (F <= 64) h[t] = nx[t];
            else h[t] = L.vec(A.v1, F, d).ld(t);
        }
        if (d < 2) ahead(d + 1);
        nd_uv<P, F>(st, h, [&](int t, v4f u, v4f v) __attribute__((always_inline)) {
            uv[d][t] = u;
            n2[t] += v * v;
            dot[t] += u * v;
            nd_here(n2[t]);
            nd_here(dot[t]);
        });
    }
#pragma unroll
    for (int t = 0; t < NT; t++) {
        h[t] = L.vecl(b3, t);
        n2[t] = __builtin_elementwise_sqrt(n2[t]);
    }
    v4f sq[2];   // s1 of the next block
    auto block = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; q++) sq[q] = 2 * s + q < NT ? s1.ld(2 * s + q) : v4f{0.f, 0.f, 0.f, 0.f};
    };
    block(0);
    ec_layer<0, NT, 2 * KS>(st, h, [&](auto s) __attribute__((always_inline)) {
        constexpr int S = decltype(s)::value;
        if constexpr (S < KS) {
            const EcOp<P> o = ec_op<P>(sq[0], sq[1]);
            if constexpr (S + 1 < KS) block(S + 1);
            return o;
        } else {
            return nd_op<P, NT>(S - KS, [&](int t) { return n2[t]; });
        }
    });
    EcOp<P> x[KS];
#pragma unroll
    for (int s = 0; s < KS; s++) x[s] = nd_op<P, NT>(s, [&](int t) { return nd_silu(h[t]); });
    // (s1 and v1 of the next tile are loaded ahead of the stores of this one, which they
    // would otherwise wait for)
    v4f w[3], ws = s1.ld(0);
#pragma unroll
    for (int d = 0; d < 3; d++) w[d] = L.vec(A.v1, F, d).ld(0);
    ec_for<NT>([&](auto t_) __attribute__((always_inline)) {
        constexpr int T = decltype(t_)::value;
        v4f a[3] = {L.vecl(b4, T), L.vecl(b4 + F, T), L.vecl(b4 + 2 * F, T)};
        ec_layer<2 * D::Q + 3 * T * KS, 3, KS>(st, a, [&](auto s) { return x[s]; });
        n2[T] = ws + a[1] * dot[T] + a[2];   // s2
        nd_here(n2[T]);
        if constexpr (T + 1 < NT) ws = s1.ld(T + 1);
#pragma unroll
        for (int d = 0; d < 3; d++) {
            uv[d][T] = w[d] + a[0] * uv[d][T];   // v2
            nd_here(uv[d][T]);
            if constexpr (T + 1 < NT) w[d] = L.vec(A.v1, F, d).ld(T + 1);
        }
        if (L.ok) {
            L.row(A.s2, F).st(T, n2[T]);
#pragma unroll
            for (int d = 0; d < 3; d++) L.vec(A.v2, F, d).st(T, uv[d][T]);
        }
    });
#pragma unroll
    for (int t = 0; t < NT; t++) h[t] = L.vecl(b1, t);
    ec_layer<5 * D::Q, NT, KS>(st, h, [&](auto s) __attribute__((always_inline)) {
        return nd_op<P, NT>(decltype(s)::value, [&](int t) { return n2[t]; });
    });
#pragma unroll
    for (int s = 0; s < KS; s++) x[s] = nd_op<P, NT>(s, [&](int t) { return nd_silu(h[t]); });
    const NdRow ph = L.row(A.phi, 3 * F);
    ec_for<NT>([&](auto t_) __attribute__((always_inline)) {
        constexpr int T = decltype(t_)::value;
        v4f a[3] = {L.vecl(b2, T), L.vecl(b2 + F, T), L.vecl(b2 + 2 * F, T)};
        ec_layer<6 * D::Q + 3 * T * KS, 3, KS>(st, a, [&](auto s) { return x[s]; });
        if (L.ok) {
#pragma unroll
            for (int q = 0; q < 3; q++) {
                ph.st(q * NT + T, a[q]);
                L.vec(A.u, F, q).st(T, uv[q][T] * a[0]);
            }
        }
    });
}

// The adjoint of k_node_fwd, or (LAST) the last update with the readout and
// the adjoint of both.
template <int P, int F, int NC, bool LAST>
__global__ void __launch_bounds__(64 * (NC + 1)) __attribute__((amdgpu_waves_per_eu(ND_EU))) k_node_bwd(NodeArgs A) {
    using D = NodeDim<F>;
    using Ring = NdRing<P, F, NC, false>;
    constexpr int NT = D::NT, KS = D::KS, SB = Ring::SB;
    constexpr bool KEEP = D::KEEP;
    const v4f z = {0.f, 0.f, 0.f, 0.f};
    constexpr int H5 = F / 2, H5P = 16 * D::N5;
    __shared__ __attribute__((aligned(16))) char lds[nd_ring(P, NC) * SB];
    __shared__ __attribute__((aligned(16))) float b3[F], b4[2 * F], bx[LAST ? 2 * H5P : F];
    if (!LAST || A.grad) {
        // rows past the layer's set carry no gradient
        for (int q = threadIdx.x; q < 16 * NC * F / 4; q += 64 * (NC + 1)) {
            const int m = blockIdx.x * 16 * NC + q / (F / 4), f = 4 * (q % (F / 4));
            if (m < A.n || m >= A.nz) continue;
            *reinterpret_cast<v4f *>(A.gs1 + (long)m * F + f) = z;
#pragma unroll
            for (int d = 0; d < 3; d++) *reinterpret_cast<v4f *>(A.gv1 + (3L * m + d) * F + f) = z;
        }
    }
    if ((int)(blockIdx.x * 16 * NC) >= A.n) return;   // the whole workgroup leaves
    nd_stage(b3, A.b3, F, F);
    nd_stage(b4, A.b4 + (LAST ? F : 0), 2 * F, 2 * F);
    if constexpr (LAST) {
        nd_stage(bx, A.b5, H5, H5P);
        nd_stage(bx + H5P, A.w6, H5, H5P);
    } else {
        nd_stage(bx, A.b1, F, F);
    }
    __syncthreads();
    if (nd_fetcher<NC>()) {
        constexpr int S0 = LAST ? 0 : D::SI, S1 = LAST ? D::SL : D::SM;
        Ring::produce(lds, reinterpret_cast<const char *>(A.chain) + (LAST ? 0 : (D::SA + D::SF) * SB),
                      LAST && !A.grad ? 3 * D::SA + D::SE : S0 + 3 * D::SA + S1 + 3 * D::SH, S0 + D::SA, D::SA,
                      S0 + D::SA + S1 + D::SH, D::SH);
        return;
    }
    Ring st;
    st.start(lds);
    const NdLane L(A.n, 16 * NC);
    const NdRow s1 = L.row(A.s1, A.ld1), gs = L.row(A.gs1, F);
    v4f raw[NT];
    EcOp<P> x[KS];
    if constexpr (!LAST) {
        // message MLP of layer t + 1: gs2 = ds1 + W1^T (silu'(h1) o W2^T gphi), parked in gs1
        const NdRow s2 = L.row(A.s2, F), gp = L.row(A.gphi, 3 * F);
        v4f h[NT], g[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            raw[t] = s2.ld(t);
            h[t] = L.vecl(bx, t);
            g[t] = z;
        }
        v4f gq[2][2 * KS];
        auto part = [&](int q, v4f *o) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NT; t++) o[t] = gp.ld(q * NT + t);
        };
        part(0, gq[0]);
        ec_layer<0, NT, KS>(st, h, [&](auto s) __attribute__((always_inline)) {
            return nd_op<P, NT>(decltype(s)::value, [&](int t) { return raw[t]; });
        });
        ec_for<3>([&](auto q_) __attribute__((always_inline)) {
            constexpr int Q = decltype(q_)::value;
            if constexpr (Q < 2) part(Q + 1, gq[(Q + 1) & 1]);
            ec_layer<(1 + Q) * D::Q, NT, KS>(st, g, [&](auto s) __attribute__((always_inline)) {
                return nd_op<P, NT>(decltype(s)::value, [&](int t) { return gq[Q & 1][t]; });
            });
        });
#pragma unroll
        for (int t = 0; t < NT; t++) {
            g[t] *= nd_dsilu(h[t]);
            h[t] = gs.ld(t);
        }
        ec_layer<4 * D::Q, NT, KS>(st, h, [&](auto s) __attribute__((always_inline)) {
            return nd_op<P, NT>(decltype(s)::value, [&](int t) { return g[t]; });
        });
        if (L.ok)
#pragma unroll
            for (int t = 0; t < NT; t++) gs.st(t, h[t]);
    }
    // update: Uv, Vv again; n^2, <Uv, Vv> and dE/da_vv = sum_d gv_d Uv_d
    v4f n2[NT], dot[NT], davv[LAST ? 1 : NT], uk[KEEP ? 3 : 1][KEEP ? NT : 1], vk[KEEP ? 3 : 1][KEEP ? NT : 1];
#pragma unroll
    for (int t = 0; t < NT; t++) {
        n2[t] = v4f{A.eps, A.eps, A.eps, A.eps};
        dot[t] = z;
        if constexpr (!LAST) davv[t] = z;
    }
#pragma unroll(KEEP ? 3 : 1)
    for (int d = 0; d < 3; d++) {
        const NdRow vr = L.vec(A.v1, F, d), gr = L.vec(A.gv, F, d);
        v4f gq[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            raw[t] = vr.ld(t);
            if constexpr (!LAST) gq[t] = gr.ld(t);
        }
        nd_uv<P, F>(st, raw, [&](int t, v4f u, v4f v) __attribute__((always_inline)) {
            if constexpr (KEEP) {
                uk[d][t] = u;
                vk[d][t] = v;
            }
            n2[t] += v * v;
            dot[t] += u * v;
            nd_here(n2[t]);
            nd_here(dot[t]);
            if constexpr (!LAST) {
                davv[t] += gq[t] * u;
                nd_here(davv[t]);
            }
        });
    }
    v4f h[NT], rn[NT];   // h3; dn / n
#pragma unroll
    for (int t = 0; t < NT; t++) {
        raw[t] = s1.ld(t);
        h[t] = L.vecl(b3, t);
        n2[t] = __builtin_elementwise_sqrt(n2[t]);
    }
    ec_layer<0, NT, 2 * KS>(st, h, [&](auto s) __attribute__((always_inline)) {
        constexpr int S = decltype(s)::value;
        if constexpr (S < KS) return nd_op<P, NT>(S, [&](int t) { return raw[t]; });
        else return nd_op<P, NT>(S - KS, [&](int t) { return n2[t]; });
    });
    // (SiLU(h3) and SiLU'(h3) are formed where they are taken: kept, they cost
    // registers through the adjoint of W4)
    auto act = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < KS; s++) x[s] = nd_op<P, NT>(s, [&](int t) { return nd_silu(h[t]); });
    };
    v4f asv[NT], g2[NT];   // a_sv; gs2
    if constexpr (LAST) {
        act();
        ec_for<NT>([&](auto t_) __attribute__((always_inline)) {
            constexpr int T = decltype(t_)::value;
            v4f a[2] = {L.vecl(b4, T), L.vecl(b4 + F, T)};
            ec_layer<2 * D::Q + 2 * T * KS, 2, KS>(st, a, [&](auto s) { return x[s]; });
            asv[T] = a[0];
            raw[T] += a[0] * dot[T] + a[1];   // s2
        });
        // readout: U, and dE/ds2 = W5^T (w6 o silu'(h5)) (zero for ghost rows)
        v4f h5[2 * D::K5];
#pragma unroll
        for (int t = 0; t < 2 * D::K5; t++) h5[t] = t < D::N5 ? L.vecl(bx, t) : z;
        ec_layer<4 * D::Q, D::N5, KS>(st, h5, [&](auto s) __attribute__((always_inline)) {
            return nd_op<P, NT>(decltype(s)::value, [&](int t) { return raw[t]; });
        });
        const bool local = A.perm[L.row0 + L.rel] < A.n_local;
        float u = 0.f;
#pragma unroll
        for (int t = 0; t < D::N5; t++) {
            const v4f w = L.vecl(bx + H5P, t);
            const v4f y = nd_silu(h5[t]);
#pragma unroll
            for (int r = 0; r < 4; r++) u = fmaf(w[r], y[r], u);
            h5[t] = local ? w * nd_dsilu(h5[t]) : z;
        }
        u += __shfl_xor(u, 16, 64);
        u += __shfl_xor(u, 32, 64);
        if (L.ok && L.g == 0) A.U[L.row0 + L.rel] = u + A.b6[0];
        if (!A.grad) return;
#pragma unroll
        for (int t = 0; t < NT; t++) g2[t] = z;
        ec_layer<4 * D::Q + D::N5 * KS, NT, D::K5>(st, g2, [&](auto s) __attribute__((always_inline)) {
            return nd_op<P, D::N5>(decltype(s)::value, [&](int t) { return h5[t]; });
        });
    } else {
#pragma unroll
        for (int t = 0; t < NT; t++) g2[t] = gs.ld(t);
    }
    // dE/dh3 = silu'(h3) o W4^T [dE/da_vv | gs2 <Uv, Vv> | gs2]
    {
        constexpr int U0 = LAST ? 4 * D::Q + D::N5 * KS + NT * D::K5 : 2 * D::Q, Q0 = LAST ? 1 : 0;
        v4f g[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) g[t] = z;
        ec_layer<U0, NT, (3 - Q0) * KS>(st, g, [&](auto s) __attribute__((always_inline)) {
            constexpr int S = decltype(s)::value % KS, Q = Q0 + decltype(s)::value / KS;
            if constexpr (Q == 0) return nd_op<P, NT>(S, [&](int t) { return davv[t]; });
            else if constexpr (Q == 1) return nd_op<P, NT>(S, [&](int t) { return g2[t] * dot[t]; });
            else return nd_op<P, NT>(S, [&](int t) { return g2[t]; });
        });
        EcOp<P> y[KS];
#pragma unroll
        for (int s = 0; s < KS; s++) y[s] = nd_op<P, NT>(s, [&](int t) {
            return g[t] * nd_dsilu(h[t]);
        });
        // [ds1 | dn] = W3^T: gs1 = gs2 + ds1; rn = dn / n
        constexpr int U1 = U0 + (3 - Q0) * D::Q;
#pragma unroll
        for (int t = 0; t < NT; t++) {
            g[t] = g2[t];
            rn[t] = z;
        }
        ec_layer<U1, NT, KS>(st, g, [&](auto s) { return y[s]; });
        if (L.ok)
#pragma unroll
            for (int t = 0; t < NT; t++) gs.st(t, g[t]);
        ec_layer<U1 + D::Q, NT, KS>(st, rn, [&](auto s) { return y[s]; });
#pragma unroll
        for (int t = 0; t < NT; t++) {
#pragma unroll
            for (int r = 0; r < 4; r++) rn[t][r] /= n2[t][r];
            nd_here(rn[t]);
        }
    }
    v4f avv[LAST ? 1 : NT];
    if constexpr (!LAST) {
        // (opaque, so that no sigmoid is kept from above)
#pragma unroll
        for (int t = 0; t < NT; t++) nd_here(h[t]);
        act();
        ec_for<NT>([&](auto t_) __attribute__((always_inline)) {
            constexpr int T = decltype(t_)::value;
            v4f a[2] = {L.vecl(b4, T), L.vecl(b4 + F, T)};
            ec_layer<7 * D::Q + 2 * T * KS, 2, KS>(st, a, [&](auto s) { return x[s]; });
            avv[T] = a[0];
            asv[T] = a[1] * g2[T];   // gs2 a_sv from here on
            nd_here(asv[T]);
        });
    } else {
#pragma unroll
        for (int t = 0; t < NT; t++) asv[t] *= g2[t];
    }
    // gv1 = gv + U^T (gv a_vv + gs2 a_sv Vv) + V^T (gs2 a_sv Uv + (dn / n) Vv), per direction
#pragma unroll(KEEP ? 3 : 1)
    for (int d = 0; d < 3; d++) {
        const NdRow gr = L.vec(A.gv, F, d), vr = L.vec(A.v1, F, d);
        v4f o[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            o[t] = z;
            if constexpr (!LAST) o[t] = gr.ld(t);
        }
        EcOp<P> xv[KEEP ? 1 : KS];
        if constexpr (!KEEP) {
#pragma unroll
            for (int s = 0; s < KS; s++) xv[s] = nd_op<P, NT>(s, [&](int t) { return vr.ld(t); });
        }
        ec_for<KS>([&](auto s_) __attribute__((always_inline)) {
            constexpr int S = decltype(s_)::value, US = KEEP ? 2 * NT * S : (4 * KS + 2 * NT) * S;
            v4f du[2] = {z, z}, dv[2] = {z, z};
            ec_for<2>([&](auto h_) __attribute__((always_inline)) {
                constexpr int HH = decltype(h_)::value, T = 2 * S + HH;
                if constexpr (T < NT) {
                    v4f a[2] = {z, z};
                    if constexpr (KEEP) {
                        a[0] = uk[d][T];
                        a[1] = vk[d][T];
                    } else {
                        ec_layer<US + 2 * KS * HH, 2, KS>(st, a, [&](auto s) { return xv[s]; });
                    }
                    du[HH] = asv[T] * a[1];
                    if constexpr (!LAST) du[HH] += gr.ld(T) * avv[T];
                    dv[HH] = asv[T] * a[0] + rn[T] * a[1];
                }
            });
            constexpr int UT = US + (KEEP ? 0 : 4 * KS);
            const EcOp<P> yu = ec_op<P>(du[0], du[1]), yv = ec_op<P>(dv[0], dv[1]);
            ec_layer<UT, NT, 1>(st, o, [&](auto) { return yu; });
            ec_layer<UT + NT, NT, 1>(st, o, [&](auto) { return yv; });
        });
        if (L.ok)
#pragma unroll
            for (int t = 0; t < NT; t++) L.vec(A.gv1, F, d).st(t, o[t]);
    }
}

// ---------------------------------------------------------------------------
// Launches
// ---------------------------------------------------------------------------
template <int P, int F, int NC>
static void launch(hipStream_t s, int which, int rows, const NodeArgs &a) {
    const unsigned nb = (unsigned)((rows + 16 * NC - 1) / (16 * NC));
    if (which == 0) k_node_fwd<P, F, NC><<<nb, 64 * (NC + 1), 0, s>>>(a);
    else if (which == 1) k_node_bwd<P, F, NC, false><<<nb, 64 * (NC + 1), 0, s>>>(a);
    else k_node_bwd<P, F, NC, true><<<nb, 64 * (NC + 1), 0, s>>>(a);
}
template <int P, int F>
static void launch(hipStream_t s, int which, const NodeArgs &a) {
    const int rows = which == 0 || a.nz < a.n ? a.n : a.nz;
    if (rows <= 0) return;
    if (rows > ND_LARGE) launch<P, F, 7>(s, which, rows, a);
    else launch<P, F, 3>(s, which, rows, a);
}
template <int P>
int node_launch(hipStream_t s, int F, int which, const NodeArgs &a) {
    switch (F) {
    case 16: launch<P, 16>(s, which, a); break;
    case 32: launch<P, 32>(s, which, a); break;
    case 64: launch<P, 64>(s, which, a); break;
    default: launch<P, 128>(s, which, a); break;
    }
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

}  // namespace mlp
