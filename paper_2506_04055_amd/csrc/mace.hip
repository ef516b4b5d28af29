// MACE with two interaction layers: energy and forces on the pruned
// neighbour graph.
//
// The paper deploys MACE (Methods, "Graph Neural Networks" and "Chosen
// Architectures": messages in the atomic-cluster-expansion form, many-body
// features built per atom from a one-particle basis) with two layers,
// correlation order 3, l_max = 3, hidden features of 32 scalars and 32
// vectors, 8 radial functions and a polynomial envelope of order 6
// ("Training Details").  The layer equations are those of the cited MACE
// paper; the reading here, per atom i, channel k, directed edge e = (i <- j)
// with r = |r_j - r_i| < rc and rhat = (r_j - r_i) / r:
//   G(l1, l2, L)[a, b, c] = (1 / 4 pi) int Y_l1a Y_l2b Y_Lc  (only l1 + l2 + L even)
//   hb_j,l2   = W_up[l2] h_j,l2                       (layer 1: h = W_emb onehot(Z))
//   R_e       = MLP_rad(B(r))                          (SiLU, no biases; K per conv path)
//   A_i,p,c   = 1/n_avg sum_e R_e,p sum_ab G(l1, l2, L)[a, b, c] Y_l1a(rhat) hb_j,l2b
//               for the conv paths p = (l1, l2, L), l2 a degree the layer takes
//   A'_i,L    = W_A[L] (the A of every path onto L, channels stacked)
//   B_eta     = the nu-fold products of A' of one channel coupled to degree L_o
//               (nu = 1, 2, 3; the nu = 3 ones through an intermediate lambda)
//   m_i,L_o   = sum_eta W_sym[Z_i][L_o][k, eta] B_eta
//   h_i,L_o   = W_out[L_o] m_i,L_o + W_sc[Z_i][L_o] h_i,L_o  (skip where L_o is an input degree)
//   E_i       = w_r1 . h1_i,0 + w_r2 . silu(W_r2 h2_i,0 + b_r2) + b_r3
// Layer 1 takes degree 0 and gives degrees 0 and 1; layer 2 takes 0 and 1 and
// gives 0.  Y are the component-normalised real harmonics of sh.h; the
// couplings are constant expressions of the same harmonics (gaunt.h), so the
// kernels unroll over the nonzero couplings only.
//
// Layout of the work: the radial MLP and the convolution of a layer are one
// kernel each way (k_mc_edge_fwd, k_mc_edge_bwd), the W_A channel mixes GEMMs
// over (atom, m) rows (gemm.hip), all on the matrix cores.  The symmetric
// contraction and the small per-atom channel mixes (W_out, W_sc, W_up, the
// readouts) run with one half-wave per atom and one lane per channel:
// * the symmetric contraction is factorised: the pair products
//   P(l1, l2 -> lambda) = sum_ab G A'_l1a A'_l2b of a channel are formed once
//   in registers and serve both the two-body paths and, coupled with one
//   more A', the three-body paths.
// Systems of few neighbours per atom (mc_edge_kernels) have the radial MLP in
// one kernel and the convolution in another, radial MLPs of other depths or
// widths a kernel per step: the MLP as GEMMs over edges, then the convolution
// with one half-wave per atom:
// * the l2 = 1 conv paths accumulate per atom the moments
//   M_p[a][b] = sum_e R_e,p Y_l1a hb_j,1b and couple them once per atom
//   (A_p,c = sum_ab G[a][b][c] M_p[a][b]); the adjoint contracts G with the
//   atom's dE/dA once (X_p[a][b] = sum_c G[a][b][c] dE/dA_p,c) and then works
//   per edge on X.
// Forces come from a hand-written adjoint: the same kernels reversed, the
// gradient of each source's hb collected from per-edge partials through the
// reverse-edge index (no atomics), per-edge sums over channels by DPP
// exchanges within the half-wave, and per edge G_e = dE/d(r_i - r_j),
// assembled into forces by launch_forces.
#include "internal.h"
#include "gemm.h"
#include "gaunt.h"
#include "sh.h"
#include "edge_chain.h"

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#define MC_INLINE __attribute__((always_inline))

namespace mlp {

namespace {

constexpr int MK = 32;     // channels: one lane each, a half-wave per atom
constexpr int APB = 8;     // atoms per workgroup (256 threads)

inline int nblk(long n, int t) { return (int)((n + t - 1) / t); }

// Conv paths of the second layer in weight order; the first layer's are the
// first four.  0..3: (l1, 0, l1); 4: (0,1,1) 5: (1,1,0) 6: (1,1,2) 7: (2,1,1)
// 8: (2,1,3) 9: (3,1,2).
__host__ __device__ constexpr int cp_l1(int p) {
    return p < 4 ? p : (p == 4 ? 0 : (p <= 6 ? 1 : (p <= 8 ? 2 : 3)));
}
__host__ __device__ constexpr int cp_L(int p) {
    return p < 4 ? p : (p == 4 ? 1 : (p == 5 ? 0 : (p == 6 ? 2 : (p == 7 ? 1 : (p == 8 ? 3 : 2)))));
}
// first accumulator of path p (its 2L + 1 outputs follow)
__host__ __device__ constexpr int cp_off(int p) {
    int o = 0;
    for (int q = 0; q < p; q++) o += 2 * cp_L(q) + 1;
    return o;
}
// position of path p among the paths onto its L (the W_A column block)
__host__ __device__ constexpr int cp_loc(int p) {
    int c = 0;
    for (int q = 0; q < p; q++) c += cp_L(q) == cp_L(p);
    return c;
}
// number of paths onto L among the first np
__host__ __device__ constexpr int cp_nL(int L, int np) {
    int c = 0;
    for (int q = 0; q < np; q++) c += cp_L(q) == L;
    return c;
}
// first moment M_p[a][b] of an l2 = 1 path ((2 l1 + 1) x 3 per path)
__host__ __device__ constexpr int cp_moff(int p) {
    int o = 0;
    for (int q = 4; q < p; q++) o += 3 * (2 * cp_l1(q) + 1);
    return o;
}
constexpr int NMOM = cp_moff(10);
static_assert(cp_off(4) == 16 && cp_off(10) == 40 && NMOM == 72, "accumulator layout");

// ---- compile-time couplings of the conv paths with l2 = 1 ----
struct CEnt {
    int a, b, c;
    float v;
};
struct ConvTab {
    CEnt e[320] = {};
    int beg[11] = {};   // entries of path p: [beg[p], beg[p + 1]), p = 4..9
};
constexpr ConvTab make_conv() {
    ConvTab t{};
    int n = 0;
    for (int p = 4; p < 10; p++) {
        t.beg[p] = n;
        const int l1 = cp_l1(p), L = cp_L(p);
        for (int a = 0; a < 2 * l1 + 1; a++)
            for (int b = 0; b < 3; b++)
                for (int c = 0; c < 2 * L + 1; c++) {
                    const double v = cg::coupling(l1, a, 1, b, L, c);
                    if (v != 0.0) t.e[n++] = CEnt{a, b, c, (float)v};
                }
    }
    t.beg[10] = n;
    return t;
}
inline constexpr ConvTab kConv = make_conv();

// ---- compile-time structure of the symmetric contraction (l_max 3, correlation 3) ----
// Pair products P(l1 <= l2 -> lambda)[mu] = sum_ab G(l1, l2, lambda)[a][b][mu] A_l1a A_l2b.
struct PEnt {
    int i, j, q;   // A slots l1^2 + a, l2^2 + b; P index
    float v;
};
struct PairTab {
    int nc = 0, l1[16] = {}, l2[16] = {}, lam[16] = {}, off[17] = {};
    PEnt e[400] = {};
    int n = 0;
};
constexpr PairTab make_pairs() {
    PairTab t{};
    int q = 0;
    for (int l1 = 0; l1 <= 3; l1++)
        for (int l2 = l1; l2 <= 3; l2++)
            for (int lam = 0; lam <= 3; lam++) {
                if (!cg::couples(l1, l2, lam)) continue;
                const int c = t.nc++;
                t.l1[c] = l1;
                t.l2[c] = l2;
                t.lam[c] = lam;
                t.off[c] = q;
                for (int a = 0; a < 2 * l1 + 1; a++)
                    for (int b = 0; b < 2 * l2 + 1; b++)
                        for (int mu = 0; mu < 2 * lam + 1; mu++) {
                            const double v = cg::coupling(l1, a, l2, b, lam, mu);
                            if (v != 0.0) t.e[t.n++] = PEnt{l1 * l1 + a, l2 * l2 + b, q + mu, (float)v};
                        }
                q += 2 * lam + 1;
            }
    t.off[t.nc] = q;
    return t;
}
inline constexpr PairTab kPair = make_pairs();
constexpr int NPP = kPair.off[kPair.nc];

constexpr int pair_off(int l1, int l2, int lam) {
    for (int c = 0; c < kPair.nc; c++)
        if (kPair.l1[c] == l1 && kPair.l2[c] == l2 && kPair.lam[c] == lam) return kPair.off[c];
    return -1;
}

// Contraction paths onto degree Lo in weight order: kind 1 (A'_Lo), kind 2
// (a pair product onto Lo, P index q0), kind 3 (a pair product onto lambda
// coupled with A'_l3 to Lo: entries (P index, A slot, output component)).
struct SEnt {
    int q, s, d;
    float v;
};
struct SymTab {
    int np = 0, kind[32] = {}, q0[32] = {}, beg[33] = {};
    SEnt e[400] = {};
    int n = 0;
};
constexpr SymTab make_sym(int Lo) {
    SymTab t{};
    t.kind[t.np] = 1;
    t.beg[t.np] = t.n;
    t.np++;
    for (int l1 = 0; l1 <= 3; l1++)
        for (int l2 = l1; l2 <= 3; l2++)
            if (cg::couples(l1, l2, Lo)) {
                t.kind[t.np] = 2;
                t.q0[t.np] = pair_off(l1, l2, Lo);
                t.beg[t.np] = t.n;
                t.np++;
            }
    for (int l1 = 0; l1 <= 3; l1++)
        for (int l2 = l1; l2 <= 3; l2++)
            for (int lam = 0; lam <= 3; lam++) {
                if (!cg::couples(l1, l2, lam)) continue;
                for (int l3 = 0; l3 <= 3; l3++) {
                    if (!cg::couples(lam, l3, Lo)) continue;
                    const int q0 = pair_off(l1, l2, lam);
                    t.kind[t.np] = 3;
                    t.q0[t.np] = q0;
                    t.beg[t.np] = t.n;
                    for (int mu = 0; mu < 2 * lam + 1; mu++)
                        for (int c = 0; c < 2 * l3 + 1; c++)
                            for (int d = 0; d < 2 * Lo + 1; d++) {
                                const double v = cg::coupling(lam, mu, l3, c, Lo, d);
                                if (v != 0.0) t.e[t.n++] = SEnt{q0 + mu, l3 * l3 + c, d, (float)v};
                            }
                    t.np++;
                }
            }
    t.beg[t.np] = t.n;
    return t;
}
inline constexpr SymTab kSym0 = make_sym(0), kSym1 = make_sym(1);
template <int LO>
constexpr const SymTab &sym_tab() {
    if constexpr (LO == 0) return kSym0;
    else return kSym1;
}
static_assert(kSym0.np == 20 && kSym1.np == 27 && NPP == 59, "contraction paths");

__device__ __forceinline__ float mc_sigmoid(float x) { return 1.0f / (1.0f + __expf(-x)); }
__device__ __forceinline__ float mc_silu(float x) { return x * mc_sigmoid(x); }
__device__ __forceinline__ float mc_dsilu(float x) {
    const float s = mc_sigmoid(x);
    return s * (1.0f + x * (1.0f - s));
}

__device__ __forceinline__ void load16(const float *p, float *v) {
    const float4 *p4 = reinterpret_cast<const float4 *>(p);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const float4 x = p4[q];
        v[4 * q] = x.x;
        v[4 * q + 1] = x.y;
        v[4 * q + 2] = x.z;
        v[4 * q + 3] = x.w;
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
// One exchange of a reduce-scatter: the lane whose bit is set keeps the
// upper W values and hands its lower W to the partner, which keeps the lower.
template <int W, int CTRL>
__device__ __forceinline__ void rs_stage(float *v, bool up) {
#pragma unroll
    for (int q = 0; q < W; q++) {
        const float send = up ? v[q] : v[q + W], keep = up ? v[q + W] : v[q];
        v[q] = keep + dpp_mov<CTRL>(send);
    }
}
// Sum of 16 values over the 32 lanes of a half-wave; lane k returns the total
// of value k & 15.  Partners within a row of 16 lanes: lane i and 15 - i
// (row mirror, bit 3 differs), i and 7 - i (half-row mirror, bit 2), i ^ 2 and
// i ^ 1 (quad permutations); then the two rows.
__device__ __forceinline__ float halfwave_sum16(float *v, int k) {
    rs_stage<8, 0x140>(v, (k & 8) != 0);
    rs_stage<4, 0x141>(v, (k & 4) != 0);
    rs_stage<2, 0x4E>(v, (k & 2) != 0);
    rs_stage<1, 0xB1>(v, (k & 1) != 0);
    return v[0] + __shfl_xor(v[0], 16, 64);
}

__device__ __forceinline__ float halfwave_sum(float v) {
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---- symmetric contraction of one channel (A: 16 slots l^2 + m) ----
__device__ __forceinline__ void pair_fwd(const float *A, float *P) {
#pragma unroll
    for (int q = 0; q < NPP; q++) P[q] = 0.f;
    cg::sfor<kPair.n>([&](auto t) MC_INLINE {
        constexpr PEnt E = kPair.e[decltype(t)::value];
        P[E.q] = fmaf(E.v, A[E.i] * A[E.j], P[E.q]);
    });
}

__device__ __forceinline__ void pair_bwd(const float *A, const float *gP, float *gA) {
    cg::sfor<kPair.n>([&](auto t) MC_INLINE {
        constexpr PEnt E = kPair.e[decltype(t)::value];
        const float g = E.v * gP[E.q];
        gA[E.i] = fmaf(g, A[E.j], gA[E.i]);
        gA[E.j] = fmaf(g, A[E.i], gA[E.j]);
    });
}

// m[d] += sum_eta W[eta] B_eta,d for output degree LO; W: this species' and
// channel's weights, path eta at W[eta * MK]
template <int LO>
__device__ __forceinline__ void sym_fwd(const float *A, const float *P, const float *__restrict__ W, float *m) {
    constexpr int NO = 2 * LO + 1;
    cg::sfor<sym_tab<LO>().np>([&](auto eta) MC_INLINE {
        constexpr int h = decltype(eta)::value;
        constexpr int kind = sym_tab<LO>().kind[h];
        const float w = W[h * MK];
        if constexpr (kind == 1) {
#pragma unroll
            for (int d = 0; d < NO; d++) m[d] = fmaf(w, A[LO * LO + d], m[d]);
        } else if constexpr (kind == 2) {
            constexpr int q0 = sym_tab<LO>().q0[h];
#pragma unroll
            for (int d = 0; d < NO; d++) m[d] = fmaf(w, P[q0 + d], m[d]);
        } else {
            constexpr int e0 = sym_tab<LO>().beg[h], ne = sym_tab<LO>().beg[h + 1] - e0;
            float b[NO];
#pragma unroll
            for (int d = 0; d < NO; d++) b[d] = 0.f;
            cg::sfor<ne>([&](auto t) MC_INLINE {
                constexpr SEnt E = sym_tab<LO>().e[e0 + decltype(t)::value];
                b[E.d] = fmaf(E.v, P[E.q] * A[E.s], b[E.d]);
            });
#pragma unroll
            for (int d = 0; d < NO; d++) m[d] = fmaf(w, b[d], m[d]);
        }
    });
}

// adjoint of sym_fwd: gm = dE/dm; adds dE/dA (direct) into gA and dE/dP into gP
template <int LO>
__device__ __forceinline__ void sym_bwd(const float *A, const float *P, const float *__restrict__ W, const float *gm,
                                        float *gA, float *gP) {
    constexpr int NO = 2 * LO + 1;
    cg::sfor<sym_tab<LO>().np>([&](auto eta) MC_INLINE {
        constexpr int h = decltype(eta)::value;
        constexpr int kind = sym_tab<LO>().kind[h];
        const float w = W[h * MK];
        float gb[NO];
#pragma unroll
        for (int d = 0; d < NO; d++) gb[d] = w * gm[d];
        if constexpr (kind == 1) {
#pragma unroll
            for (int d = 0; d < NO; d++) gA[LO * LO + d] += gb[d];
        } else if constexpr (kind == 2) {
            constexpr int q0 = sym_tab<LO>().q0[h];
#pragma unroll
            for (int d = 0; d < NO; d++) gP[q0 + d] += gb[d];
        } else {
            constexpr int e0 = sym_tab<LO>().beg[h], ne = sym_tab<LO>().beg[h + 1] - e0;
            cg::sfor<ne>([&](auto t) MC_INLINE {
                constexpr SEnt E = sym_tab<LO>().e[e0 + decltype(t)::value];
                const float g = E.v * gb[E.d];
                gP[E.q] = fmaf(g, A[E.s], gP[E.q]);
                gA[E.s] = fmaf(g, P[E.q], gA[E.s]);
            });
        }
    });
}

}  // namespace

// Per-L blocks of an atom array (A before and after the W_A mix, and their gradients).
struct McBlk {
    float *p[4];
};

// ---------------------------------------------------------------------------
// Model
// ---------------------------------------------------------------------------
struct McModel {
    int S = 0, NB = 0, NBP = 0, pe = 0, nrad = 0, rh[4] = {0, 0, 0, 0}, RH = 0;
    float rc = 0.f, navg = 1.f, b_r3 = 0.f;
    float *dev = nullptr;     // weights, transposed copies, tables (device)
    void *pk_dev = nullptr;   // packed GEMM operands
    PackedW radF[2][5], radA[2][5], waF[2][4], waA[2][4];
    EdgeMlp rmlp[2];          // the radial MLPs as kernels of their own
    bool fused = false;       // the radial MLP and the convolution in one kernel each way
    char *chain = nullptr;    // its weights in the order of use
    size_t chF[2] = {}, chB[2] = {};
    const float *zero = nullptr, *hb0tab = nullptr, *skip0tab = nullptr;
    const float *w_r1 = nullptr, *W_r2 = nullptr, *b_r2 = nullptr, *w_r2 = nullptr;
    const float *WoutT[2][2] = {}, *Wout[2][2] = {};   // [layer][output degree index]
    const float *WupT1[2] = {}, *Wup1[2] = {};         // second layer's W_up for l2 = 0, 1
    const float *WscT1 = nullptr, *Wsc1 = nullptr;     // second layer's skip (degree 0), [S][K][K]
    const float *Wsym[2][2] = {};                      // [layer][output degree index]: [S][paths][K]
};

// ---------------------------------------------------------------------------
// Forward, per edge: radial functions with the envelope, and the harmonics.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_mc_edge(const int *__restrict__ rowc, int n, const float4 *__restrict__ geom,
                                                 int NB, int NBP, int pe, float rc, float *__restrict__ X0,
                                                 float *__restrict__ Y) {
    const long ne = rowc[n];
    const float c0 = sqrtf(2.0f / rc), th = 3.14159265358979f / rc;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += (long)gridDim.x * blockDim.x) {
        const float4 gm = geom[e];
        const float r = gm.w, ir = 1.0f / r;
        float u, du;
        envelope(r / rc, pe, u, du);
        float sn, cs;
        sincosf(th * r, &sn, &cs);
        float *x = X0 + e * NBP;
        float sk = sn, skm = 0.f;
        for (int k = 0; k < NB; k++) {
            x[k] = c0 * sk * ir * u;
            const float nx = 2.f * cs * sk - skm;
            skm = sk;
            sk = nx;
        }
        for (int k = NB; k < NBP; k++) x[k] = 0.f;
        float y[16];
        sh16(gm.x * ir, gm.y * ir, gm.z * ir, y);
        float4 *y4 = reinterpret_cast<float4 *>(Y + e * 16);
#pragma unroll
        for (int q = 0; q < 4; q++) y4[q] = make_float4(y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]);
    }
}

// ---------------------------------------------------------------------------
// Convolution, one half-wave per destination atom, lane = channel: the A of
// every conv path summed over the atom's edges, scaled by 1 / n_avg, written
// as the rows (i, c) of its L block with the path's position among the paths
// onto L selecting the column block (the W_A GEMM's operand layout).
// ---------------------------------------------------------------------------
template <int LAY>
__global__ void __launch_bounds__(256) k_mc_conv(const int *__restrict__ rowc, const int *__restrict__ colc, int nd,
                                                 const float *__restrict__ Y, const float *__restrict__ R,
                                                 const float *__restrict__ HB, const int *__restrict__ zsp,
                                                 const float *__restrict__ hb0, float scale, McBlk AR) {
    constexpr int NP = LAY == 0 ? 4 : 10, NM = LAY == 0 ? 1 : NMOM;
    const int k = threadIdx.x & 31;
    const int i = blockIdx.x * APB + (threadIdx.x >> 5);
    if (i >= nd) return;
    float acc[16], mom[NM];
#pragma unroll
    for (int q = 0; q < 16; q++) acc[q] = 0.f;
#pragma unroll
    for (int q = 0; q < NM; q++) mom[q] = 0.f;
    const int eend = rowc[i + 1];
    for (int e = rowc[i]; e < eend; e++) {
        const int j = colc[e];
        float h0, h1[3] = {0.f, 0.f, 0.f};
        if constexpr (LAY == 0) {
            h0 = hb0[zsp[j] * MK + k];
        } else {
            const float *hb = HB + (long)j * 4 * MK + k;
            h0 = hb[0];
            h1[0] = hb[MK];
            h1[1] = hb[2 * MK];
            h1[2] = hb[3 * MK];
        }
        float y[16], r[NP];
        load16(Y + (long)e * 16, y);
        const float *rr = R + (long)e * NP * MK + k;
#pragma unroll
        for (int p = 0; p < NP; p++) r[p] = rr[p * MK];
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const float s = r[p] * h0;
#pragma unroll
            for (int c = 0; c < 2 * p + 1; c++) acc[p * p + c] = fmaf(s, y[p * p + c], acc[p * p + c]);
        }
        if constexpr (LAY == 1) {
#pragma unroll
            for (int p = 4; p < NP; p++) {
                const int l1 = cp_l1(p), mo = cp_moff(p);
                const float rb[3] = {r[p] * h1[0], r[p] * h1[1], r[p] * h1[2]};
#pragma unroll
                for (int a = 0; a < 2 * l1 + 1; a++)
#pragma unroll
                    for (int b = 0; b < 3; b++) mom[mo + a * 3 + b] = fmaf(y[l1 * l1 + a], rb[b], mom[mo + a * 3 + b]);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < 4; p++) {
        const int L = p, nc = 2 * L + 1, ld = cp_nL(L, NP) * MK;
        float *o = AR.p[L] + (long)i * nc * ld + cp_loc(p) * MK + k;
#pragma unroll
        for (int c = 0; c < nc; c++) o[(long)c * ld] = acc[p * p + c] * scale;
    }
    if constexpr (LAY == 1) {
        cg::sfor<6>([&](auto pi) MC_INLINE {
            constexpr int p = 4 + decltype(pi)::value, L = cp_L(p), nc = 2 * L + 1, ld = cp_nL(L, 10) * MK,
                          mo = cp_moff(p), e0 = kConv.beg[p];
            float v[nc];
#pragma unroll
            for (int c = 0; c < nc; c++) v[c] = 0.f;
            cg::sfor<kConv.beg[p + 1] - e0>([&](auto t) MC_INLINE {
                constexpr CEnt E = kConv.e[e0 + decltype(t)::value];
                v[E.c] = fmaf(E.v, mom[mo + E.a * 3 + E.b], v[E.c]);
            });
            float *o = AR.p[L] + (long)i * nc * ld + cp_loc(p) * MK + k;
#pragma unroll
            for (int c = 0; c < nc; c++) o[(long)c * ld] = v[c] * scale;
        });
    }
}

// ---------------------------------------------------------------------------
// The radial MLP and the convolution of a layer in one kernel each way (the
// layers chained in registers, edge_chain.h): R [edge][P K] and its gradient
// never reach HBM (128 + 320 floats per edge each, written and read twice per
// evaluation by separate kernels), nor do the radial functions, the harmonics
// and their gradients, which every kernel forms again from the geometry.
//
// Per edge and l2 = 1 path the coupling is applied to the harmonics,
// W_p[b][c] = sum_a G(l1, 1, L)[a][b][c] Y_l1a (channel-independent), so
// A_p,c = sum_e sum_b (R_p hb_b) W_p[b][c].
//   forward: the sums over an atom's edges are products [channel][edge] x
//     [edge][m or c] on the FP32 matrix instruction;
//   adjoint: no sum over edges is needed: with the atom's dE/dA in LDS,
//     V_p,b = sum_c dE/dA_p,c W_p[b][c] gives dE/dR_p = sum_b V_p,b hb_b,
//     dE/dhb_b += R_p V_p,b and dE/dW_p[b][c] = sum_k dE/dA_p,c R_p hb_b; dE/dR_p
//     is at once the operand of the transposed output layer.
// What bounds both: vector and matrix work that depend on each other at two
// waves per SIMD, which the accumulators and one edge's products of a path
// need.  Busy, split bf16 at 143,748 atoms, layer 1 / layer 0: forward vector
// issue 29 / 42 %, matrix cores 44 / 33 %, LDS 19 / 21 %; adjoint 43 / 43, 17 /
// 21 and 23 / 29 %, with the data return of the vector loads at 46 / 41 %.  (In
// FP32 the adjoint's matrix cores are at 25 / 31 %.)  SiLU and its derivative
// are a third of the vector work.  143,748 atoms of fcc
// aluminium, split bf16: 2.75 + 1.18 ms forward (layers 1 and 0), 4.35 + 2.07 ms
// adjoint, the evaluation 20.8 ms with a kernel per step and 13.4 so; 648 atoms
// of water, FP32, 0.050 + 0.026 and 0.083 + 0.041 ms, 0.70 and 0.31; an
// 11k-atom FP32 domain 3.16 and 2.50 ms.  A forward by runs of atoms with the
// sums in LDS, as the adjoint has it, took 4.3 + 1.4 ms on the first and 0.065
// + 0.026 on the second.
// ---------------------------------------------------------------------------
constexpr int MC_SLOTS = 6;   // atoms of a run (their dE/dA, 5 KB each, fill LDS)
struct McEdgeArgs {
    const int *rowc, *colc, *zsp;
    const float4 *geom;
    int nd, per_wg, pe;
    float rc, irc, c0, th, thl, scale;   // 1 / rc, sqrt(2 / rc), pi / rc in two parts, 1 / n_avg
    const char *W;                  // the chain's units
    const float *hb;                // first layer: hb0 [S][K]; second: HB [atom][4][K]
    McBlk A;                        // forward: A (written); adjoint: dE/dA
    float *MSG;                     // adjoint of the second layer
    float4 *G;                      // adjoint
    int n, nd1;                     // first layer's adjoint: all atoms, those of the second layer
};

// first float of degree L's block per atom in dE/dA (paths onto degrees < L)
__host__ __device__ constexpr int mc_goff(int L, int np) {
    int o = 0;
    for (int q = 0; q < L; q++) o += (2 * q + 1) * cp_nL(q, np) * MK;
    return o;
}

// W_p[b][c] of an edge from its harmonics (Y of degree l1 at Y + l1^2)
template <int p>
__device__ __forceinline__ void mc_edge_coupling(const float *Y, float (*Wp)[7]) {
#pragma unroll
    for (int b = 0; b < 3; b++)
#pragma unroll
        for (int c = 0; c < 7; c++) Wp[b][c] = 0.f;
    constexpr int l1 = cp_l1(p), e0 = kConv.beg[p];
    cg::sfor<kConv.beg[p + 1] - e0>([&](auto t) MC_INLINE {
        constexpr CEnt E = kConv.e[e0 + decltype(t)::value];
        Wp[E.b][E.c] = fmaf(E.v, Y[l1 * l1 + E.a], Wp[E.b][E.c]);
    });
}

// What a thread per edge (the first waves) loads, and writes to LDS: the
// harmonics (ys), and 1 / r, the envelope and its r-derivative, sin and cos
// of pi r / rc, the index of the source's hb row, its own slot (eg).
struct McEdge {
    float4 gm;
    int j, slot;
    bool valid;
};
template <int LAY>
__device__ __forceinline__ void mc_edge_load(McEdge &E, const McEdgeArgs &A, int base, int off, const EcRun &r, int ch) {
    if (threadIdx.x < EC_ROWS) {
        E.slot = ec_slot(threadIdx.x, r, off);
        E.valid = (int)threadIdx.x < min(EC_ROWS, r.total - ch * EC_ROWS);
        const int e = base + ch * EC_ROWS + (E.valid ? threadIdx.x : 0);
        E.gm = A.geom[e];
        E.j = A.colc[e];
    }
}
template <int P, int LAY>
__device__ __forceinline__ void mc_edge_put(const McEdge &E, const McEdgeArgs &A, float *ys, float *eg) {
    typedef ec_v4f v4f;
    if (threadIdx.x < EC_ROWS) {
        const int q = threadIdx.x, j = LAY == 0 ? A.zsp[E.j] : E.j;
        const float r = E.gm.w, ir = 1.0f / r;
        float u, du, s1, c1, Y[16];
        envelope(r / A.rc, A.pe, u, du);
        ec_sincos_0pi<P>(A.th, A.thl, r, s1, c1);
        sh16(E.gm.x * ir, E.gm.y * ir, E.gm.z * ir, Y);
        // rows past the end carry nothing: u = 0 (no MLP has a bias)
#pragma unroll
        for (int k = 0; k < 4; k++)
            *reinterpret_cast<v4f *>(ys + 16 * q + 4 * k) = v4f{Y[4 * k], Y[4 * k + 1], Y[4 * k + 2], Y[4 * k + 3]};
        *reinterpret_cast<v4f *>(eg + 8 * q) = v4f{ir, E.valid ? u : 0.f, du * A.irc, s1};
        *reinterpret_cast<v4f *>(eg + 8 * q + 4) = v4f{c1, __int_as_float(j), __int_as_float(E.slot), 0.f};
    }
}

// The hidden layers, units U0 .. U0 + 19 of a chain of NS stages, from this
// edge's radial functions: the pre-activations of the last (p3) and SiLU' of
// those of the first two.
template <int U0, int NS, int P>
__device__ __forceinline__ void mc_hidden(EcStream<P> &st, const char *next, const McEdgeArgs &A, const float *er, int g,
                                          ec_v4f *p1, ec_v4f *p2, ec_v4f *p3) {
    typedef ec_v4f v4f;
    const v4f z4 = v4f{0.f, 0.f, 0.f, 0.f};
    v4f x;
    {
        const v4f e0 = *reinterpret_cast<const v4f *>(er);
        const float s1 = e0[3], c1 = er[4], bu = A.c0 * e0[0] * e0[1];
        float sk, ck;
        ec_angle(g, s1, c1, sk, ck);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            x[k] = bu * sk;
            const float ns = fmaf(sk, c1, ck * s1);
            ck = fmaf(ck, c1, -sk * s1);
            sk = ns;
        }
    }
#pragma unroll
    for (int t = 0; t < 4; t++) p1[t] = p2[t] = p3[t] = z4;
    ec_layer<U0, NS, 4, 1>(st, next, p1, [&](auto) { return ec_op<P>(x, z4); });
    ec_layer<U0 + 4, NS, 4, 2>(st, next, p2, [&](auto s) { return ec_op<P>(ec_silu_d<P>(p1[2 * s]), ec_silu_d<P>(p1[2 * s + 1])); });
    ec_layer<U0 + 12, NS, 4, 2>(st, next, p3, [&](auto s) { return ec_op<P>(ec_silu_d<P>(p2[2 * s]), ec_silu_d<P>(p2[2 * s + 1])); });
}

constexpr int mc_fwd_units(int lay) { return 20 + 4 * (lay == 0 ? 4 : 10); }
constexpr int mc_bwd_units(int lay) { return 20 + 8 * (lay == 0 ? 4 : 10) + 18; }

// Forward: a wave takes one atom at a time (from the workgroup's counter) and
// its edges 16 at a time.  The output layer runs with its operands exchanged:
// lane (k, g) then holds R_p of channel 16 t + k for the edges 4 g + r, which
// times hb is at once the first operand of the FP32 matrix instruction whose
// second is the harmonics (or W_p) of the same edges: the sums over an atom's
// edges stay in the accumulators (row = channel, column = m or c) from tile to
// tile.  No value passes between waves; they share the weight stages only.
// Where a workgroup has at most four atoms (SPLIT), two waves take one
// atom's tiles in turn and the second hands its sums to the first at the end:
// the launch lasts as long as one wave's tiles (648 atoms of water, FP32: 81
// and 40 us with a wave per atom, 50 and 24 with two).
constexpr int MC_FWD_ATOMS = 64;   // most atoms per workgroup

template <int P, int LAY, bool SPLIT>
__global__ void __launch_bounds__(EC_THREADS) __attribute__((amdgpu_waves_per_eu(2))) k_mc_edge_fwd(McEdgeArgs A) {
    typedef ec_v4f v4f;
    constexpr int NP = LAY == 0 ? 4 : 10, NS = (mc_fwd_units(LAY) + EC_U - 1) / EC_U, NC = LAY == 0 ? 1 : 4,
                  NR = 16 + (LAY == 0 ? 0 : 72);   // rows of the wave's LDS: Y_m, then W_p[b][c]
    __shared__ __attribute__((aligned(16))) char wst[2 * EcStream<P>::SB];
    // (split: afterwards QR of the second waves' accumulators at a time)
    constexpr int QR = LAY == 0 ? 2 * NP : NP;
    __shared__ __attribute__((aligned(16))) float ywT[SPLIT ? std::max((EC_THREADS / 64) * NR * 16, 4 * QR * 256) : (EC_THREADS / 64) * NR * 16];
    __shared__ int rows[MC_FWD_ATOMS + 1], ticket;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4,
              m = lane & 15;
    const v4f z4 = v4f{0.f, 0.f, 0.f, 0.f};
    const int a0 = blockIdx.x * A.per_wg, na = min(A.nd - a0, A.per_wg);
    if (na <= 0) return;
    for (int q = tid; q <= na; q += EC_THREADS) rows[q] = A.rowc[a0 + q];
    if (tid == 0) ticket = EC_THREADS / 64;
    EcStream<P> st;
    st.start(wst, A.W);
    __syncthreads();
    // A = 0 for an atom without edges
    auto put_zero = [&](int i) MC_INLINE {
#pragma unroll
        for (int L = 0; L < 4; L++) {
            const int cnt = (2 * L + 1) * cp_nL(L, NP) * MK;
            for (int q = 4 * lane; q < cnt; q += 256) *reinterpret_cast<v4f *>(A.A.p[L] + (long)(a0 + i) * cnt + q) = z4;
        }
    };
    // the first atom from i on (by tickets) with edges: its rows e .. e1
    auto settle = [&](int &i, int &e, int &e1) MC_INLINE {
        while (i < na) {
            e = __builtin_amdgcn_readfirstlane(rows[i]);
            e1 = __builtin_amdgcn_readfirstlane(rows[i + 1]);
            if (e < e1) return;
            put_zero(i);
            int t = 0;
            if (lane == 0) t = atomicAdd(&ticket, 1);
            i = __builtin_amdgcn_readfirstlane(t);
        }
        e = e1 = 0;
    };
    float *yw = ywT + w * NR * 16;
    constexpr int step = SPLIT ? 32 : 16;
    int i = SPLIT ? w >> 1 : w, e = 0, e1 = 0;
    const int mine = i;   // split: the one atom of this wave and its neighbour
    if constexpr (!SPLIT) {
        settle(i, e, e1);
    } else if (i < na) {
        e = __builtin_amdgcn_readfirstlane(rows[i]) + 16 * (w & 1);
        e1 = __builtin_amdgcn_readfirstlane(rows[i + 1]);
        if (e >= e1) i = na;
    }
    float4 gm = make_float4(0.f, 0.f, 1.f, 1.f);
    int j = 0;
    if (i < na) {
        const int q = min(e + m, e1 - 1);
        gm = A.geom[q];
        j = A.colc[q];
    }
    v4f acc[2 * NP];
#pragma unroll
    for (int q = 0; q < 2 * NP; q++) acc[q] = z4;
    // lane (m, g): channels 16 t + 4 g + r of column m
    auto put = [&](int i) MC_INLINE {
        cg::sfor<NP>([&](auto pi) MC_INLINE {
            constexpr int p = decltype(pi)::value, L = cp_L(p), nc = 2 * L + 1, c0 = p < 4 ? p * p : 0;
            if (m >= c0 && m < c0 + nc) {
                float *d = A.A.p[L] + (((long)(a0 + i) * nc + m - c0) * cp_nL(L, NP) + cp_loc(p)) * MK + 4 * g;
#pragma unroll
                for (int t = 0; t < 2; t++) *reinterpret_cast<v4f *>(d + 16 * t) = acc[2 * p + t] * A.scale;
            }
            acc[2 * p] = acc[2 * p + 1] = z4;
        });
    };
    while (__syncthreads_or(i < na)) {
        // the tile after this one
        int ni = i, ne = e + step, ne1 = e1;
        const bool last = i < na && ne >= e1;
        if constexpr (SPLIT) {
            if (last) ni = na;
        } else if (last) {
            int t = 0;
            if (lane == 0) t = atomicAdd(&ticket, 1);
            ni = __builtin_amdgcn_readfirstlane(t);
            settle(ni, ne, ne1);
        }
        // this lane's edge: radial functions; its harmonics and couplings to LDS
        v4f x;
        {
            const float r = gm.w, ir = 1.0f / r;
            float u, du, s1, c1, sk, ck;
            envelope(r / A.rc, A.pe, u, du);
            ec_sincos_0pi<P>(A.th, A.thl, r, s1, c1);
            ec_angle(g, s1, c1, sk, ck);
            // lanes past the atom's edges carry nothing (no MLP has a bias)
            const float bu = e + m < e1 ? A.c0 * ir * u : 0.f;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                x[k] = bu * sk;
                const float ns = fmaf(sk, c1, ck * s1);
                ck = fmaf(ck, c1, -sk * s1);
                sk = ns;
            }
            float Y[16];
            sh16(gm.x * ir, gm.y * ir, gm.z * ir, Y);
            if (g == 0) {
#pragma unroll
                for (int q = 0; q < 16; q++) yw[16 * q + m] = Y[q];
            }
            if constexpr (LAY == 1)
                cg::sfor<6>([&](auto pi) MC_INLINE {
                    constexpr int p = 4 + decltype(pi)::value, nc = 2 * cp_L(p) + 1;
                    float Wp[3][7];
                    mc_edge_coupling<p>(Y, Wp);
                    if (g == 1 + (p & 1))
#pragma unroll
                        for (int b = 0; b < 3; b++)
#pragma unroll
                            for (int c = 0; c < nc; c++) yw[16 * (16 + 3 * (cp_off(p) - 16) + nc * b + c) + m] = Wp[b][c];
                });
        }
        // hb of the edges 4 g + r at the channels 16 t + m (zero for a wave
        // without a tile: any other atom's may not be finite)
        v4f h[NC][2];
#pragma unroll
        for (int c = 0; c < NC; c++) h[c][0] = h[c][1] = z4;
        if (i < na) {
            const int jr = LAY == 0 ? A.zsp[j] : j;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float *hp = A.hb + (long)__shfl(jr, 4 * g + r, 64) * (NC * MK) + m;
#pragma unroll
                for (int c = 0; c < NC; c++)
#pragma unroll
                    for (int t = 0; t < 2; t++) h[c][t][r] = hp[c * MK + 16 * t];
            }
        }
        EcOp<P> o0, o1;
        {
            v4f p1[4], p2[4], p3[4];
#pragma unroll
            for (int t = 0; t < 4; t++) p1[t] = p2[t] = p3[t] = z4;
            ec_layer<0, NS, 4, 1>(st, A.W, p1, [&](auto) { return ec_op<P>(x, z4); });
            ec_layer<4, NS, 4, 2>(st, A.W, p2, [&](auto s) { return ec_op<P>(ec_silu<P>(p1[2 * s]), ec_silu<P>(p1[2 * s + 1])); });
            ec_layer<12, NS, 4, 2>(st, A.W, p3, [&](auto s) { return ec_op<P>(ec_silu<P>(p2[2 * s]), ec_silu<P>(p2[2 * s + 1])); });
            o0 = ec_op<P>(ec_silu<P>(p3[0]), ec_silu<P>(p3[1]));
            o1 = ec_op<P>(ec_silu<P>(p3[2]), ec_silu<P>(p3[3]));
        }
        float4 ngm = gm;
        int nj = j;
        if (ni < na) {
            const int q = min(ne + m, ne1 - 1);
            ngm = A.geom[q];
            nj = A.colc[q];
        }
        const v4f yo = *reinterpret_cast<const v4f *>(yw + 16 * m + 4 * g);   // Y_m of the edges 4 g + r
        cg::sfor<NP>([&](auto pi) MC_INLINE {
            constexpr int p = decltype(pi)::value;
            v4f r[2] = {z4, z4};
            ec_layer<20 + 4 * p, NS, 2, 2, true>(st, A.W, r, [&](auto s) {
                if constexpr (decltype(s)::value == 0) return o0;
                else return o1;
            });
            if constexpr (p < 4) {
                const v4f s0 = r[0] * h[0][0], s1 = r[1] * h[0][1];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    acc[2 * p] = __builtin_amdgcn_mfma_f32_16x16x4f32(s0[q], yo[q], acc[2 * p], 0, 0, 0);
                    acc[2 * p + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(s1[q], yo[q], acc[2 * p + 1], 0, 0, 0);
                }
            } else {
                constexpr int nc = 2 * cp_L(p) + 1;
                const float *wp = yw + 16 * (16 + 3 * (cp_off(p) - 16) + min(m, nc - 1)) + 4 * g;
#pragma unroll
                for (int b = 0; b < 3; b++) {
                    const v4f wo = *reinterpret_cast<const v4f *>(wp + 16 * nc * b);
                    const v4f s0 = r[0] * h[1 + b][0], s1 = r[1] * h[1 + b][1];
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        acc[2 * p] = __builtin_amdgcn_mfma_f32_16x16x4f32(s0[q], wo[q], acc[2 * p], 0, 0, 0);
                        acc[2 * p + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(s1[q], wo[q], acc[2 * p + 1], 0, 0, 0);
                    }
                }
            }
        });
        if constexpr (!SPLIT) {
            if (last) put(i);
        }
        i = ni;
        e = ne;
        e1 = ne1;
        gm = ngm;
        j = nj;
    }
    if constexpr (SPLIT) {
        v4f *half = reinterpret_cast<v4f *>(ywT) + (w >> 1) * QR * 64 + lane;
#pragma unroll
        for (int q0 = 0; q0 < 2 * NP; q0 += QR) {
            __syncthreads();
            if (mine < na && (w & 1))
#pragma unroll
                for (int q = 0; q < QR; q++) half[64 * q] = acc[q0 + q];
            __syncthreads();
            if (mine < na && !(w & 1))
#pragma unroll
                for (int q = 0; q < QR; q++) acc[q0 + q] += half[64 * q];
        }
        if (mine < na && !(w & 1)) put(mine);
    }
}

// Adjoint: a workgroup takes runs of whole atoms with up to 128 edges (EcRun),
// 16 per wave; lane (c, g) holds of edge c the channels 16 t + 4 g + r of both
// channel tiles t, so R_p, hb and all products of one path stay in the lane.
template <int P, int LAY>
__global__ void __launch_bounds__(EC_THREADS) __attribute__((amdgpu_waves_per_eu(2))) k_mc_edge_bwd(McEdgeArgs A) {
    typedef ec_v4f v4f;
    constexpr int NP = LAY == 0 ? 4 : 10, NS = (mc_bwd_units(LAY) + EC_U - 1) / EC_U, NF = mc_goff(4, NP);
    __shared__ __attribute__((aligned(16))) char wst[2 * EcStream<P>::SB];
    // SiLU' of the first hidden layers waits in LDS for the way down (the
    // registers hold the last layer's; 16 per layer)
    constexpr int NPK = LAY == 0 ? 1 : 2;
    __shared__ __attribute__((aligned(16))) float ys[EC_ROWS * 16], eg[EC_ROWS * 8], ga[MC_SLOTS * NF];
    __shared__ v4f park[NPK * 4 * EC_THREADS];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4,
              row = 16 * w + (lane & 15);
    const v4f z4 = v4f{0.f, 0.f, 0.f, 0.f};
    if constexpr (LAY == 0) {   // edges that no layer reaches
        const long ne = A.rowc[A.n];
        for (long e = A.rowc[A.nd] + (long)blockIdx.x * EC_THREADS + tid; e < ne; e += (long)gridDim.x * EC_THREADS)
            A.G[e] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const int a1 = min(A.nd, ((int)blockIdx.x + 1) * A.per_wg);
    int a = blockIdx.x * A.per_wg;
    if (a >= a1) return;
    EcStream<P> st;
    st.start(wst, A.W);
    const float *er = eg + 8 * row, *yr = ys + 16 * row;
    int base = A.rowc[a], off = ec_row_off<MC_SLOTS>(A.rowc, lane, a, a1) - base;
    McEdge ed;
    bool have = false;   // the run's first piece is in ed
    while (a < a1) {
        __syncthreads();   // the last reads of the previous run's LDS
        const EcRun run = ec_run<MC_SLOTS>(lane, a, a1, off);
        const int na = run.na, nch = run.nch, total = run.total;
        const int an = min(a + na, a1), nbase = A.rowc[an], noff = ec_row_off<MC_SLOTS>(A.rowc, lane, an, a1);
        if (total > 0)   // dE/dA of the run's atoms, per degree [slot][c][path][k]
#pragma unroll
            for (int L = 0; L < 4; L++) {
                const int cnt = (2 * L + 1) * cp_nL(L, NP) * MK;
                const float *src = A.A.p[L] + (long)a * cnt;
                float *dst = ga + MC_SLOTS * mc_goff(L, NP);
                for (int q = 4 * tid; q < na * cnt; q += 4 * EC_THREADS)
                    *reinterpret_cast<v4f *>(dst + q) = *reinterpret_cast<const v4f *>(src + q) * A.scale;
            }
        for (int ch = 0; ch < nch && total > 0; ch++) {
            if (nch > 1) __syncthreads();   // the last reads of the previous piece's rows
            if (!have) mc_edge_load<LAY>(ed, A, base, off, run, ch);
            have = false;
            mc_edge_put<P, LAY>(ed, A, ys, eg);
            __syncthreads();
            const int slot = __float_as_int(er[6]);
            const long e = base + ch * EC_ROWS + row;
            const bool valid = ch * EC_ROWS + row < total;
            const float *hp = A.hb + (long)__float_as_int(er[5]) * (LAY == 0 ? 1 : 4) * MK + 4 * g;
            v4f h[LAY == 0 ? 1 : 4][2], gh[LAY == 0 ? 1 : 4][2];
#pragma unroll
            for (int c = 0; c < (LAY == 0 ? 1 : 4); c++)
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    h[c][t] = *reinterpret_cast<const v4f *>(hp + c * MK + 16 * t);
                    gh[c][t] = z4;
                }
            EcOp<P> o0, o1;
            v4f p1[4], p2[4], p3[4];
            mc_hidden<0, NS, P>(st, A.W, A, er, g, p1, p2, p3);
#pragma unroll
            for (int t = 0; t < 4; t++) {
                park[t * EC_THREADS + tid] = p1[t];
                if constexpr (NPK > 1) park[(4 + t) * EC_THREADS + tid] = p2[t];
            }
            o0 = ec_op<P>(ec_silu_d<P>(p3[0]), ec_silu_d<P>(p3[1]));
            o1 = ec_op<P>(ec_silu_d<P>(p3[2]), ec_silu_d<P>(p3[3]));
            float Y[16], gy[16];
            load16(yr, Y);
#pragma unroll
            for (int q = 0; q < 16; q++) gy[q] = 0.f;
            v4f acc[4] = {z4, z4, z4, z4};   // dE/dh of the last hidden layer
            cg::sfor<NP>([&](auto pi) MC_INLINE {
                constexpr int p = decltype(pi)::value, L = cp_L(p), nc = 2 * L + 1, ld = cp_nL(L, NP) * MK;
                v4f r[2] = {z4, z4}, gR[2];
                ec_layer<20 + 8 * p, NS, 2, 2>(st, A.W, r, [&](auto s) {
                    if constexpr (decltype(s)::value == 0) return o0;
                    else return o1;
                });
                const float *gp = ga + MC_SLOTS * mc_goff(L, NP) + slot * nc * ld + cp_loc(p) * MK + 4 * g;
                auto dot4 = [](v4f x, v4f y, float s) MC_INLINE {
                    return fmaf(x[3], y[3], fmaf(x[2], y[2], fmaf(x[1], y[1], fmaf(x[0], y[0], s))));
                };
                if constexpr (p < 4) {
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        const v4f s = r[t] * h[0][t];
                        v4f d = z4;
#pragma unroll
                        for (int c = 0; c < nc; c++) {
                            const v4f x = *reinterpret_cast<const v4f *>(gp + c * ld + 16 * t);
                            d += x * Y[p * p + c];
                            gy[p * p + c] = dot4(x, s, gy[p * p + c]);
                        }
                        gR[t] = d * h[0][t];
                        if constexpr (LAY == 1) gh[0][t] += r[t] * d;
                    }
                } else {
                    float Wp[3][7], gw[3][7];
                    mc_edge_coupling<p>(Y, Wp);
#pragma unroll
                    for (int b = 0; b < 3; b++)
#pragma unroll
                        for (int c = 0; c < 7; c++) gw[b][c] = 0.f;
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        v4f s[3], V[3];
#pragma unroll
                        for (int b = 0; b < 3; b++) {
                            s[b] = r[t] * h[1 + b][t];
                            V[b] = z4;
                        }
#pragma unroll
                        for (int c = 0; c < nc; c++) {
                            const v4f x = *reinterpret_cast<const v4f *>(gp + c * ld + 16 * t);
#pragma unroll
                            for (int b = 0; b < 3; b++) {
                                V[b] += x * Wp[b][c];
                                gw[b][c] = dot4(x, s[b], gw[b][c]);
                            }
                        }
                        gR[t] = V[0] * h[1][t] + V[1] * h[2][t] + V[2] * h[3][t];
#pragma unroll
                        for (int b = 0; b < 3; b++) gh[1 + b][t] += r[t] * V[b];
                    }
                    constexpr int l1 = cp_l1(p), e0 = kConv.beg[p];
                    cg::sfor<kConv.beg[p + 1] - e0>([&](auto t) MC_INLINE {
                        constexpr CEnt E = kConv.e[e0 + decltype(t)::value];
                        gy[l1 * l1 + E.a] = fmaf(E.v, gw[E.b][E.c], gy[l1 * l1 + E.a]);
                    });
                }
                ec_layer<24 + 8 * p, NS, 4, 1>(st, A.W, acc, [&](auto) { return ec_op<P>(gR[0], gR[1]); });
                // (opaque here: gh and gy are used behind branches only, and
                // their sums would be moved there with every operand kept)
#pragma unroll
                for (int q = 0; q < 16; q++) asm volatile("" : "+v"(gy[q]));
                if constexpr (LAY == 1)
#pragma unroll
                    for (int c = 0; c < 4; c++) asm volatile("" : "+v"(gh[c][0]), "+v"(gh[c][1]));
            });
            if constexpr (LAY == 1)
                if (valid)
#pragma unroll
                    for (int c = 0; c < 4; c++)
#pragma unroll
                        for (int t = 0; t < 2; t++)
                            *reinterpret_cast<v4f *>(A.MSG + (e * 4 + c) * MK + 16 * t + 4 * g) = gh[c][t];
            if (ch == nch - 1 && an < a1) {   // the next run's first edges
                const int o = noff - nbase;
                const EcRun nx = ec_run<MC_SLOTS>(lane, an, a1, o);
                if (nx.total > 0) {
                    mc_edge_load<LAY>(ed, A, nbase, o, nx, 0);
                    have = true;
                }
            }
            // down the hidden layers
            constexpr int UH = 20 + 8 * NP;
            v4f gb = z4;
            {
                v4f g2[4] = {z4, z4, z4, z4}, g1[4] = {z4, z4, z4, z4};
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    p1[t] = park[t * EC_THREADS + tid];
                    if constexpr (NPK > 1) p2[t] = park[(4 + t) * EC_THREADS + tid];
                }
                ec_layer<UH, NS, 4, 2>(st, A.W, g2, [&](auto s) { return ec_op<P>(acc[2 * s] * p3[2 * s], acc[2 * s + 1] * p3[2 * s + 1]); });
                ec_layer<UH + 8, NS, 4, 2>(st, A.W, g1, [&](auto s) { return ec_op<P>(g2[2 * s] * p2[2 * s], g2[2 * s + 1] * p2[2 * s + 1]); });
                ec_layer<UH + 16, NS, 1, 2>(st, A.W, &gb, [&](auto s) { return ec_op<P>(g1[2 * s] * p1[2 * s], g1[2 * s + 1] * p1[2 * s + 1]); });
            }
            // dE/dr through this lane's radial functions k = 4 g + 1 .. 4 g + 4,
            // dE/drhat through the harmonics
            const v4f e0 = *reinterpret_cast<const v4f *>(er);
            const float ir = e0[0], u = e0[1], du = e0[2], s1 = e0[3], c1 = er[4];
            float dEdr = 0.f;
            {
                float sk, ck, kt = (4 * g + 1) * A.th;
                ec_angle(g, s1, c1, sk, ck);
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const float dB = A.c0 * ir * (fmaf(kt, ck, -sk * ir) * u + sk * du);
                    dEdr = fmaf(gb[k], dB, dEdr);
                    const float ns = fmaf(sk, c1, ck * s1);
                    ck = fmaf(ck, c1, -sk * s1);
                    sk = ns;
                    kt += A.th;
                }
            }
            const float i3 = 0.57735026918962576f, hx = Y[3] * i3, hy = Y[1] * i3, hz = Y[2] * i3;
            float tx, ty, tz;
            sh16_grad(hx, hy, hz, gy, tx, ty, tz);
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                dEdr += __shfl_xor(dEdr, o, 64);
                tx += __shfl_xor(tx, o, 64);
                ty += __shfl_xor(ty, o, 64);
                tz += __shfl_xor(tz, o, 64);
            }
            if (valid && g == 0) {
                if constexpr (LAY == 1) {   // the second layer's part, for the first layer's kernel
                    A.G[e] = make_float4(dEdr, tx, ty, tz);
                } else {
                    if (a + slot < A.nd1) {
                        const float4 q = A.G[e];
                        dEdr += q.x;
                        tx += q.y;
                        ty += q.z;
                        tz += q.w;
                    }
                    // G_e = dE/d(r_i - r_j) = -(dE/dr rhat + (I - rhat rhat^T) dE/drhat / r)
                    const float rd = tx * hx + ty * hy + tz * hz;
                    A.G[e] = make_float4(-(dEdr * hx + (tx - rd * hx) * ir), -(dEdr * hy + (ty - rd * hy) * ir),
                                         -(dEdr * hz + (tz - rd * hz) * ir), 0.f);
                }
            }
        }
        a += na;
        base = nbase;
        off = noff - nbase;
        have = have && total > 0;
    }
}

// ---------------------------------------------------------------------------
// Per-atom kernels: one half-wave per atom, lane = channel; the lane's A'
// (16 values) and pair products in registers, the channel mixes through a
// per-atom LDS row.  Every thread of a workgroup reaches the barriers (rows
// past nd compute on zeros and write nothing).
// ---------------------------------------------------------------------------
struct McNodeArgs {
    McBlk AP;                      // A' [row][2L + 1][K] per L
    const float *Wsym[2];          // per output degree index: [S][paths][K]
    int np[2];
    const float *WoutT[2];         // [k'][k] per output degree index
    const float *skip0tab;         // first layer: W_sc[Z] h0 per species [S][K]
    const float *WupT1[2];
    const float *WscT1;            // second layer's skip [S][k'][k]
    const float *w_r1, *W_r2, *b_r2, *w_r2;
    float b_r3;
    int RH;
    const float *H1;               // first layer's output [row][4][K]
    float *H1o, *HB1o, *H2;        // outputs
    float *U;                      // per-atom energies (rows past nloc: 0)
    int nloc;                      // rows the second layer covers
};

__device__ __forceinline__ void load_ap(const McBlk &AP, bool act, int i, int k, float *A) {
#pragma unroll
    for (int L = 0; L < 4; L++)
#pragma unroll
        for (int m = 0; m < 2 * L + 1; m++) A[L * L + m] = act ? AP.p[L][((long)i * (2 * L + 1) + m) * MK + k] : 0.f;
}

__device__ __forceinline__ void store_gap(const McBlk &GAP, int i, int k, const float *gA) {
#pragma unroll
    for (int L = 0; L < 4; L++)
#pragma unroll
        for (int m = 0; m < 2 * L + 1; m++) GAP.p[L][((long)i * (2 * L + 1) + m) * MK + k] = gA[L * L + m];
}

// x[c] = sum_k' W[c][k' * K + k] xs[c][k'] for c < NC (W per component, [k'][k])
template <int NC>
__device__ __forceinline__ void mix(const float *const *W, const float *xs, int k, float *x) {
#pragma unroll
    for (int c = 0; c < NC; c++) {
        const float *w = W[c] + k;
        const float *v = xs + c * MK;
        float s = 0.f;
#pragma unroll 8
        for (int q = 0; q < MK; q++) s = fmaf(w[q * MK], v[q], s);
        x[c] = s;
    }
}

template <int LAY>
__global__ void __launch_bounds__(256) k_mc_node(int nd, const int *__restrict__ zsp, McNodeArgs a) {
    __shared__ float sx[APB * 4 * MK];
    const int tid = threadIdx.x, k = tid & 31, ai = tid >> 5;
    const int i = blockIdx.x * APB + ai;
    const bool act = i < nd;
    const int z = act ? zsp[i] : 0;
    float A[16], P[NPP];
    load_ap(a.AP, act, i, k, A);
    pair_fwd(A, P);
    float m[4] = {0.f, 0.f, 0.f, 0.f};
    sym_fwd<0>(A, P, a.Wsym[0] + (long)z * a.np[0] * MK + k, m);
    if constexpr (LAY == 0) sym_fwd<1>(A, P, a.Wsym[1] + (long)z * a.np[1] * MK + k, m + 1);
    float *xs = sx + ai * 4 * MK;
    constexpr int NC = LAY == 0 ? 4 : 1;
#pragma unroll
    for (int c = 0; c < NC; c++) xs[c * MK + k] = m[c];
    __syncthreads();
    float h[4];
    {
        const float *W[4] = {a.WoutT[0], a.WoutT[1], a.WoutT[1], a.WoutT[1]};
        mix<NC>(W, xs, k, h);
    }
    __syncthreads();
    if constexpr (LAY == 0) {
        h[0] += a.skip0tab[z * MK + k];
        if (act)
#pragma unroll
            for (int c = 0; c < 4; c++) a.H1o[((long)i * 4 + c) * MK + k] = h[c];
        const float e = halfwave_sum(a.w_r1[k] * h[0]);
        if (act && k == 0) a.U[i] = i < a.nloc ? e : 0.f;
#pragma unroll
        for (int c = 0; c < 4; c++) xs[c * MK + k] = h[c];
        __syncthreads();
        float hb[4];
        const float *W[4] = {a.WupT1[0], a.WupT1[1], a.WupT1[1], a.WupT1[1]};
        mix<4>(W, xs, k, hb);
        if (act)
#pragma unroll
            for (int c = 0; c < 4; c++) a.HB1o[((long)i * 4 + c) * MK + k] = hb[c];
    } else {
        // skip on degree 0 (species-dependent), then the readout MLP
        xs[k] = act ? a.H1[(long)i * 4 * MK + k] : 0.f;
        __syncthreads();
        {
            const float *w = a.WscT1 + (long)z * MK * MK + k;
            float s = 0.f;
#pragma unroll 8
            for (int q = 0; q < MK; q++) s = fmaf(w[q * MK], xs[q], s);
            h[0] += s;
        }
        __syncthreads();
        if (act) a.H2[(long)i * MK + k] = h[0];
        xs[k] = h[0];
        __syncthreads();
        float e = 0.f;
        if (k < a.RH) {
            const float *w = a.W_r2 + k * MK;
            float zz = a.b_r2[k];
            for (int q = 0; q < MK; q++) zz = fmaf(w[q], xs[q], zz);
            e = a.w_r2[k] * mc_silu(zz);
        }
        e = halfwave_sum(e);
        if (act && k == 0) a.U[i] += e + a.b_r3;
    }
}

// ---------------------------------------------------------------------------
// Adjoint of the per-atom kernels.
// ---------------------------------------------------------------------------
struct McNodeBwdArgs {
    McBlk AP, GAP;                 // A' of the layer and dE/dA' (output)
    const float *Wsym[2];
    int np[2];
    const float *Wout[2];          // [k][k'] per output degree index
    const float *Wup1[2];          // second layer's W_up [k][k'] for l2 = 0, 1
    const float *Wsc1;             // [S][K][K]
    const float *w_r1, *W_r2, *b_r2, *w_r2;
    int RH;
    const float *H2;
    float *GH1S;                   // second layer: dE/dh1 (degree 0) through the skip
    // first layer: dE/dhb1 collected from per-edge partials
    const int *rowc, *colc, *revc;
    const float *MSG;
    int nd1;
    const int *perm;
    int n_local;
};

__global__ void __launch_bounds__(256) k_mc_node1_bwd(int nd, const int *__restrict__ zsp, McNodeBwdArgs a) {
    __shared__ float sx[APB * 4 * MK];
    const int tid = threadIdx.x, k = tid & 31, ai = tid >> 5;
    const int i = blockIdx.x * APB + ai;
    const bool act = i < nd;
    const int z = act ? zsp[i] : 0;
    const float gE = (act && a.perm[i] < a.n_local) ? 1.f : 0.f;
    float *xs = sx + ai * 4 * MK;
    xs[k] = act ? a.H2[(long)i * MK + k] : 0.f;
    __syncthreads();
    float gz = 0.f;
    if (k < a.RH) {
        const float *w = a.W_r2 + k * MK;
        float zz = a.b_r2[k];
        for (int q = 0; q < MK; q++) zz = fmaf(w[q], xs[q], zz);
        gz = gE * a.w_r2[k] * mc_dsilu(zz);
    }
    xs[MK + k] = gz;
    __syncthreads();
    float gh = 0.f;
    for (int q = 0; q < a.RH; q++) gh = fmaf(a.W_r2[q * MK + k], xs[MK + q], gh);
    xs[2 * MK + k] = gh;
    __syncthreads();
    float gm[1] = {0.f}, gs = 0.f;
    {
        const float *wo = a.Wout[0] + k, *ws = a.Wsc1 + (long)z * MK * MK + k;
        const float *v = xs + 2 * MK;
#pragma unroll 8
        for (int q = 0; q < MK; q++) {
            gm[0] = fmaf(wo[q * MK], v[q], gm[0]);
            gs = fmaf(ws[q * MK], v[q], gs);
        }
    }
    if (act) a.GH1S[(long)i * MK + k] = gs;
    float A[16], P[NPP], gA[16], gP[NPP];
    load_ap(a.AP, act, i, k, A);
    pair_fwd(A, P);
#pragma unroll
    for (int q = 0; q < 16; q++) gA[q] = 0.f;
#pragma unroll
    for (int q = 0; q < NPP; q++) gP[q] = 0.f;
    sym_bwd<0>(A, P, a.Wsym[0] + (long)z * a.np[0] * MK + k, gm, gA, gP);
    pair_bwd(A, gP, gA);
    if (act) store_gap(a.GAP, i, k, gA);
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_mc_node0_bwd(int nd, const int *__restrict__ zsp,
                                                                                         McNodeBwdArgs a) {
    __shared__ float sx[APB * 4 * MK];
    const int tid = threadIdx.x, k = tid & 31, ai = tid >> 5;
    const int i = blockIdx.x * APB + ai;
    const bool act = i < nd;
    const int z = act ? zsp[i] : 0;
    const float gE = (act && a.perm[i] < a.n_local) ? 1.f : 0.f;
    // dE/dhb1 of this atom: the partials its out-edges left on their reverse edges
    float gh[4] = {0.f, 0.f, 0.f, 0.f};
    if (act) {
        // eight edges at a time, so that their rows are in flight together
        // (one by one, each edge waited for its reverse index and then for
        // its row: the kernel took 2.19 ms on 143,748 atoms, 1.16 ms so)
        const int eend = a.rowc[i + 1];
        for (int e = a.rowc[i]; e < eend; e += 8) {
            int rv[8];
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const int f = min(e + q, eend - 1);
                rv[q] = e + q < eend && a.colc[f] < a.nd1 ? a.revc[f] : -1;
            }
            float x[8][4];
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const float *mp = a.MSG + (long)max(rv[q], 0) * 4 * MK + k;
#pragma unroll
                for (int c = 0; c < 4; c++) x[q][c] = mp[c * MK];
            }
#pragma unroll
            for (int q = 0; q < 8; q++)
#pragma unroll
                for (int c = 0; c < 4; c++) gh[c] += rv[q] < 0 ? 0.f : x[q][c];
        }
    }
    float *xs = sx + ai * 4 * MK;
#pragma unroll
    for (int c = 0; c < 4; c++) xs[c * MK + k] = gh[c];
    __syncthreads();
    float g1[4];
    {
        const float *W[4] = {a.Wup1[0], a.Wup1[1], a.Wup1[1], a.Wup1[1]};
        mix<4>(W, xs, k, g1);
    }
    g1[0] += gE * a.w_r1[k] + ((act && i < a.nd1) ? a.GH1S[(long)i * MK + k] : 0.f);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; c++) xs[c * MK + k] = g1[c];
    __syncthreads();
    float gm[4];
    {
        const float *W[4] = {a.Wout[0], a.Wout[1], a.Wout[1], a.Wout[1]};
        mix<4>(W, xs, k, gm);
    }
    float A[16], P[NPP], gA[16], gP[NPP];
    load_ap(a.AP, act, i, k, A);
    pair_fwd(A, P);
#pragma unroll
    for (int q = 0; q < 16; q++) gA[q] = 0.f;
#pragma unroll
    for (int q = 0; q < NPP; q++) gP[q] = 0.f;
    sym_bwd<0>(A, P, a.Wsym[0] + (long)z * a.np[0] * MK + k, gm, gA, gP);
    sym_bwd<1>(A, P, a.Wsym[1] + (long)z * a.np[1] * MK + k, gm + 1, gA, gP);
    pair_bwd(A, gP, gA);
    if (act) store_gap(a.GAP, i, k, gA);
}

// ---------------------------------------------------------------------------
// Adjoint of the second layer's convolution, by destination: dE/dR per edge
// (written over R), dE/dY per edge (sums over the channels), and per edge the
// gradient its source's hb receives (MSG[e][4][K]), collected later by the
// source through the reverse edge.  The l2 = 1 paths work on
// X_p[a][b] = sum_c G_p[a][b][c] dE/dA_p,c, formed once per atom.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_mc_conv1_bwd(const int *__restrict__ rowc, const int *__restrict__ colc, int nd,
                                                      const float *__restrict__ Y, float *__restrict__ R,
                                                      const float *__restrict__ HB, float scale, McBlk GAR,
                                                      float *__restrict__ GY, float *__restrict__ MSG) {
    constexpr int NP = 10;
    const int k = threadIdx.x & 31;
    const int i = blockIdx.x * APB + (threadIdx.x >> 5);
    if (i >= nd) return;
    float gA0[16], X[NMOM];
#pragma unroll
    for (int p = 0; p < 4; p++) {
        const int L = p, nc = 2 * L + 1, ld = cp_nL(L, NP) * MK;
        const float *o = GAR.p[L] + (long)i * nc * ld + cp_loc(p) * MK + k;
#pragma unroll
        for (int c = 0; c < nc; c++) gA0[p * p + c] = o[(long)c * ld] * scale;
    }
#pragma unroll
    for (int q = 0; q < NMOM; q++) X[q] = 0.f;
    cg::sfor<6>([&](auto pi) MC_INLINE {
        constexpr int p = 4 + decltype(pi)::value, L = cp_L(p), nc = 2 * L + 1, ld = cp_nL(L, NP) * MK,
                      mo = cp_moff(p), e0 = kConv.beg[p];
        const float *o = GAR.p[L] + (long)i * nc * ld + cp_loc(p) * MK + k;
        float g[nc];
#pragma unroll
        for (int c = 0; c < nc; c++) g[c] = o[(long)c * ld] * scale;
        cg::sfor<kConv.beg[p + 1] - e0>([&](auto t) MC_INLINE {
            constexpr CEnt E = kConv.e[e0 + decltype(t)::value];
            X[mo + E.a * 3 + E.b] = fmaf(E.v, g[E.c], X[mo + E.a * 3 + E.b]);
        });
    });
    const int eend = rowc[i + 1];
    for (int e = rowc[i]; e < eend; e++) {
        const int j = colc[e];
        const float *hb = HB + (long)j * 4 * MK + k;
        const float h0 = hb[0], h1[3] = {hb[MK], hb[2 * MK], hb[3 * MK]};
        float y[16], r[NP];
        load16(Y + (long)e * 16, y);
        float *rr = R + (long)e * NP * MK + k;
#pragma unroll
        for (int p = 0; p < NP; p++) r[p] = rr[p * MK];
        float gy[16], gh[4] = {0.f, 0.f, 0.f, 0.f}, gR[NP];
#pragma unroll
        for (int p = 0; p < 4; p++) {
            float d = 0.f;
#pragma unroll
            for (int c = 0; c < 2 * p + 1; c++) {
                d = fmaf(gA0[p * p + c], y[p * p + c], d);
                gy[p * p + c] = gA0[p * p + c] * (r[p] * h0);
            }
            gR[p] = d * h0;
            gh[0] = fmaf(r[p], d, gh[0]);
        }
#pragma unroll
        for (int p = 4; p < NP; p++) {
            const int l1 = cp_l1(p), mo = cp_moff(p);
            float u[3] = {0.f, 0.f, 0.f};
#pragma unroll
            for (int a = 0; a < 2 * l1 + 1; a++) {
                float wa = 0.f;
#pragma unroll
                for (int b = 0; b < 3; b++) {
                    u[b] = fmaf(X[mo + a * 3 + b], y[l1 * l1 + a], u[b]);
                    wa = fmaf(X[mo + a * 3 + b], h1[b], wa);
                }
                gy[l1 * l1 + a] = fmaf(r[p], wa, gy[l1 * l1 + a]);
            }
            gR[p] = u[0] * h1[0] + u[1] * h1[1] + u[2] * h1[2];
#pragma unroll
            for (int b = 0; b < 3; b++) gh[1 + b] = fmaf(r[p], u[b], gh[1 + b]);
        }
#pragma unroll
        for (int p = 0; p < NP; p++) rr[p * MK] = gR[p];
        float *mp = MSG + (long)e * 4 * MK + k;
#pragma unroll
        for (int c = 0; c < 4; c++) mp[c * MK] = gh[c];
        const float s = halfwave_sum16(gy, k);
        if (k < 16) GY[(long)e * 16 + k] = s;
    }
}

// Adjoint of the first layer's convolution (hb depends on the species only,
// so nothing flows to the sources): dE/dR over R, dE/dY added to the second
// layer's for destinations it covers.
__global__ void __launch_bounds__(256) k_mc_conv0_bwd(const int *__restrict__ rowc, const int *__restrict__ colc, int nd,
                                                      int nd1, const float *__restrict__ Y, float *__restrict__ R,
                                                      const int *__restrict__ zsp, const float *__restrict__ hb0,
                                                      float scale, McBlk GAR, float *__restrict__ GY) {
    const int k = threadIdx.x & 31;
    const int i = blockIdx.x * APB + (threadIdx.x >> 5);
    if (i >= nd) return;
    float gA[16];
#pragma unroll
    for (int L = 0; L < 4; L++)
#pragma unroll
        for (int c = 0; c < 2 * L + 1; c++) gA[L * L + c] = GAR.p[L][((long)i * (2 * L + 1) + c) * MK + k] * scale;
    const bool add = i < nd1;
    const int eend = rowc[i + 1];
    for (int e = rowc[i]; e < eend; e++) {
        const float h0 = hb0[zsp[colc[e]] * MK + k];
        float y[16];
        load16(Y + (long)e * 16, y);
        float *rr = R + (long)e * 4 * MK + k;
        float gy[16];
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const float rp = rr[p * MK];
            float d = 0.f;
#pragma unroll
            for (int c = 0; c < 2 * p + 1; c++) {
                d = fmaf(gA[p * p + c], y[p * p + c], d);
                gy[p * p + c] = gA[p * p + c] * (rp * h0);
            }
            rr[p * MK] = d * h0;
        }
        const float s = halfwave_sum16(gy, k);
        if (k < 16) {
            float *g = GY + (long)e * 16 + k;
            *g = add ? *g + s : s;
        }
    }
}

// Per edge: dE/dr through the radial functions and the envelope, dE/drhat
// from the harmonics, G_e = dE/d(r_i - r_j); edges no layer reaches get 0.
__global__ void k_mc_geom(const int *__restrict__ rowc, int n, const int *__restrict__ e0,
                          const float4 *__restrict__ geom, int NB, int NBP, int pe, float rc,
                          const float *__restrict__ GX, const float *__restrict__ GY, float4 *__restrict__ G) {
    const long ne = rowc[n], ne0 = *e0;
    const float c0 = sqrtf(2.0f / rc), th = 3.14159265358979f / rc;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += (long)gridDim.x * blockDim.x) {
        if (e >= ne0) {
            G[e] = make_float4(0.f, 0.f, 0.f, 0.f);
            continue;
        }
        const float4 gm = geom[e];
        const float r = gm.w, ir = 1.0f / r;
        float u, du;
        envelope(r / rc, pe, u, du);
        du *= 1.0f / rc;
        float sn, cs;
        sincosf(th * r, &sn, &cs);
        const float *gb = GX + e * NBP;
        float dEdr = 0.f;
        float sk = sn, skm = 0.f, ck = cs, ckm = 1.f;
        for (int k = 0; k < NB; k++) {
            const float kt = (k + 1) * th;
            const float dB = c0 * ((kt * ck * ir - sk * ir * ir) * u + sk * ir * du);
            dEdr = fmaf(gb[k], dB, dEdr);
            const float ns = 2.f * cs * sk - skm, nc = 2.f * cs * ck - ckm;
            skm = sk;
            sk = ns;
            ckm = ck;
            ck = nc;
        }
        const float x = gm.x * ir, y = gm.y * ir, z = gm.z * ir;
        float gy[16];
        load16(GY + e * 16, gy);
        float hx, hy, hz;
        sh16_grad(x, y, z, gy, hx, hy, hz);
        const float rd = hx * x + hy * y + hz * z;
        const float gx = dEdr * x + (hx - rd * x) * ir, gyy = dEdr * y + (hy - rd * y) * ir,
                    gz = dEdr * z + (hz - rd * z) * ir;
        G[e] = make_float4(-gx, -gyy, -gz, 0.f);
    }
}

__global__ void k_mc_zero(float *__restrict__ p, long n) {
    for (long q = (long)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (long)gridDim.x * blockDim.x) p[q] = 0.f;
}

// Species tables of the first layer, whose input is the embedding alone:
// hb0[z] = W_up0 W_emb[:, z] and skip0[z] = W_sc0[z] W_emb[:, z].
__global__ void k_mc_species(int S, const float *__restrict__ Wemb, const float *__restrict__ Wup0,
                             const float *__restrict__ Wsc0, float *__restrict__ hb0, float *__restrict__ skip0) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= S * MK) return;
    const int z = t / MK, k = t % MK;
    float a = 0.f, b = 0.f;
    for (int q = 0; q < MK; q++) {
        const float h = Wemb[q * S + z];
        a = fmaf(Wup0[k * MK + q], h, a);
        b = fmaf(Wsc0[((long)z * MK + k) * MK + q], h, b);
    }
    hb0[t] = a;
    skip0[t] = b;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
struct McArena {
    long X0, Y, P[2][4], A[2][4], R[2], GY, GX0, MSG, AR[2], AP[2], GAP, H1, HB1, H2, GH1S, U, EP, total;
};

// Whether a system takes the edge kernels.  They cost 57 ns per atom (FP32: 73)
// up to some 15 neighbours, however few there are: one atom fills a wave's 16
// rows, six a run's 128.  With a kernel for the radial MLP and one for the
// convolution an atom costs 18 ns and an edge 3.8 (20 and 4.9), and their ten
// more launches 40 us.  Gases of 200,000 atoms with 1, 4, 8 and 10 neighbours,
// split bf16: 9.2, 11.3, 11.5 and 11.6 ms with the edge kernels, 4.2, 6.3, 9.5
// and 11.1 without; of 3,000 atoms with 4 and 6 neighbours 273 and 276 us
// against 255 and 285.
static bool mc_edge_kernels(const McModel &a, long N, long E, float skin) {
    const double x = a.rc / (a.rc + skin), deg = N > 0 ? E * x * x * x / (double)N : 0.0;
    return a.fused && deg >= 11.0 - 1.5e4 / (double)N;
}

static McArena mc_layout(const McModel &a, long N, long E, bool edge_kernels) {
    McArena L;
    long o = 0;
    auto take = [&](long cnt) {
        const long r = o;
        o += (cnt + 63) / 64 * 64;
        return r;
    };
    // the edge kernels keep MSG alone per edge; between a radial MLP's kernel and
    // the convolution passes more, and its hidden layers where it takes several
    const long Eh = a.fused ? 0 : E, Es = edge_kernels ? 0 : E;
    L.X0 = take(Es * a.NBP);
    L.Y = take(Es * 16);
    for (int t = 0; t < 2; t++) {
        for (int q = 0; q < 4; q++) L.P[t][q] = L.A[t][q] = 0;
        for (int q = 0; q < a.nrad; q++) {
            L.P[t][q] = take(Eh * a.rh[q]);
            L.A[t][q] = take(Eh * a.rh[q]);
        }
        L.R[t] = take(Es * (t == 0 ? 4 : 10) * MK);
    }
    L.GY = take(Es * 16);
    L.GX0 = take(Es * a.NBP);
    L.MSG = take(E * 4 * MK);
    L.AR[0] = take(N * 16 * MK);
    L.AR[1] = take(N * 40 * MK);
    L.AP[0] = take(N * 16 * MK);
    L.AP[1] = take(N * 16 * MK);
    L.GAP = take(N * 16 * MK);
    L.H1 = take(N * 4 * MK);
    L.HB1 = take(N * 4 * MK);
    L.H2 = take(N * MK);
    L.GH1S = take(N * MK);
    L.U = take(N + 64);
    L.EP = take(2 * energy_part_doubles(N));   // the energy sums' chunk partials (doubles)
    L.total = o + 4096;
    return L;
}

size_t mace_arena_bytes(const mlp_model *m, long n_atoms, long n_edges, float skin, bool counted) {
    const McModel &a = *m->mc;
    return (size_t)mc_layout(a, n_atoms, n_edges, !counted && mc_edge_kernels(a, n_atoms, n_edges, skin)).total * sizeof(float);
}

// The weights of the edge kernels, where the radial MLP fits them: three
// hidden layers of at most 64, at most 16 radial functions.  Other shapes
// take the kernel-per-step path.
static int mc_pack_chain(McModel *a, int P, const float *w, const size_t oRad[2][5]) {
    bool ok = a->nrad == 3 && a->NB <= 16;
    for (int q = 0; q < a->nrad; q++) ok = ok && a->rh[q] <= 64;
    if (!ok) return 0;
    const int NPt[2] = {4, 10}, NB = a->NB, *rh = a->rh;
    EcPack k(P, 2 * (20 + 38) + (4 + 8) * 14 + 4 * EC_U);
    for (int t = 0; t < 2; t++) {
        const float *W0 = w + oRad[t][0], *W1 = w + oRad[t][1], *W2 = w + oRad[t][2], *Wo = w + oRad[t][3];
        // element (o, i) of a row-major matrix of R rows and C columns, zero outside
        auto at = [](const float *M, int R, int C) {
            return [=](int o, int i) { return o < R && i < C ? M[(size_t)o * C + i] : 0.f; };
        };
        auto tr = [](const float *M, int R, int C) {
            return [=](int o, int i) { return i < R && o < C ? M[(size_t)i * C + o] : 0.f; };
        };
        auto hidden = [&]() {
            k.layer(4, 1, at(W0, rh[0], NB));
            k.layer(4, 2, at(W1, rh[1], rh[0]));
            k.layer(4, 2, at(W2, rh[2], rh[1]));
        };
        a->chF[t] = k.bytes();
        hidden();
        for (int p = 0; p < NPt[t]; p++) k.layer(2, 2, at(Wo + (size_t)p * MK * rh[2], MK, rh[2]));
        k.align();
        a->chB[t] = k.bytes();
        hidden();
        for (int p = 0; p < NPt[t]; p++) {
            k.layer(2, 2, at(Wo + (size_t)p * MK * rh[2], MK, rh[2]));
            k.layer(4, 1, tr(Wo + (size_t)p * MK * rh[2], MK, rh[2]));
        }
        k.layer(4, 2, tr(W2, rh[2], rh[1]));
        k.layer(4, 2, tr(W1, rh[1], rh[0]));
        k.layer(1, 2, tr(W0, rh[0], NB));
        k.align();
    }
    if (hipMalloc(&a->chain, k.bytes()) != hipSuccess) {
        (void)hipGetLastError();
        return fail(-2, "mace: weight allocation failed");
    }
    if (hipMemcpy(a->chain, k.data(), k.bytes(), hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(a->chain);
        return fail(-5, "mace: weight copy failed");
    }
    a->fused = true;
    return 0;
}

int mace_create(mlp_model *m, const McDims &d, const float *w, size_t n_weights) {
    if (d.S < 1 || d.S > 64) return fail(-1, "mace: n_species out of range");
    if (d.NB < 1 || d.NB > 16) return fail(-1, "mace: n_basis must be 1..16");
    if (d.p < 1 || d.p > 8) return fail(-1, "mace: envelope_p must be 1..8");
    if (d.lmax != 3 || d.K != MK || d.corr != 3)
        return fail(-1, "mace: this build takes l_max 3, 32 channels and correlation order 3");
    if (d.nrad < 1 || d.nrad > 4) return fail(-1, "mace: radial_hidden needs 1..4 widths");
    for (int q = 0; q < d.nrad; q++)
        if (d.rh[q] < 4 || d.rh[q] % 4 || d.rh[q] > 256) return fail(-1, "mace: radial widths must be multiples of 4 up to 256");
    if (d.RH < 1 || d.RH > MK) return fail(-1, "mace: readout_hidden must be 1..32");
    if (!(d.rc > 0.f) || !(d.navg > 0.f)) return fail(-1, "mace: r_c and avg_neighbors must be positive");
    const int S = d.S, K = MK, NB = d.NB;
    // contraction paths per layer and output degree (layer 1: degrees 0 and 1; layer 2: degree 0)
    const int npath[2][2] = {{kSym0.np, kSym1.np}, {kSym0.np, 0}}, nout[2] = {2, 1};
    // storage order (matrices [out][in]): W_emb (K x S); per layer: W_up per
    // input degree, radial matrices, W_A per L, W_sym per output degree,
    // W_out per output degree, W_sc for degree 0 (the one output degree both
    // layers also take); then w_r1, W_r2, b_r2, w_r2, b_r3
    size_t off = 0;
    auto take = [&](size_t cnt) {
        const size_t r = off;
        off += cnt;
        return r;
    };
    const size_t oEmb = take((size_t)K * S);
    size_t oUp[2][2], oRad[2][5], oWA[2][4], oSym[2][2], oOut[2][2], oSc[2];
    const int NPt[2] = {4, 10};
    for (int t = 0; t < 2; t++) {
        for (int l2 = 0; l2 <= t; l2++) oUp[t][l2] = take((size_t)K * K);
        int prev = NB;
        for (int q = 0; q < d.nrad; q++) {
            oRad[t][q] = take((size_t)d.rh[q] * prev);
            prev = d.rh[q];
        }
        oRad[t][d.nrad] = take((size_t)NPt[t] * K * prev);
        for (int L = 0; L < 4; L++) oWA[t][L] = take((size_t)K * cp_nL(L, NPt[t]) * K);
        for (int q = 0; q < nout[t]; q++) oSym[t][q] = take((size_t)S * K * npath[t][q]);
        for (int q = 0; q < nout[t]; q++) oOut[t][q] = take((size_t)K * K);
        oSc[t] = take((size_t)S * K * K);
    }
    const size_t oR1 = take(K), oWR2 = take((size_t)d.RH * K), oBR2 = take(d.RH), oWr2 = take(d.RH), oBR3 = take(1);
    if (off != n_weights)
        return fail(-1, "mace: weight count " + std::to_string(n_weights) + " does not match the header (" +
                            std::to_string(off) + ")");

    McModel *a = new McModel();
    a->S = S;
    a->NB = NB;
    a->NBP = (NB + 3) / 4 * 4;
    a->pe = d.p;
    a->nrad = d.nrad;
    for (int q = 0; q < d.nrad; q++) a->rh[q] = d.rh[q];
    a->RH = d.RH;
    a->rc = d.rc;
    a->navg = d.navg;
    a->b_r3 = w[oBR3];

    // device floats: the weights as given, then transposed copies and tables
    std::vector<float> host(w, w + n_weights);
    auto push = [&](const std::vector<float> &v) {
        while (host.size() % 64) host.push_back(0.f);
        const size_t r = host.size();
        host.insert(host.end(), v.begin(), v.end());
        return r;
    };
    auto transpose = [&](size_t o) {   // K x K, [k][k'] -> [k'][k]
        std::vector<float> t((size_t)K * K);
        for (int r = 0; r < K; r++)
            for (int c = 0; c < K; c++) t[(size_t)c * K + r] = w[o + (size_t)r * K + c];
        return t;
    };
    size_t oWoutT[2][2] = {}, oWupT1[2], oWscT1, oSymT[2][2] = {};
    for (int t = 0; t < 2; t++)
        for (int q = 0; q < nout[t]; q++) oWoutT[t][q] = push(transpose(oOut[t][q]));
    for (int l2 = 0; l2 < 2; l2++) oWupT1[l2] = push(transpose(oUp[1][l2]));
    {
        std::vector<float> t((size_t)S * K * K);
        for (int z = 0; z < S; z++)
            for (int r = 0; r < K; r++)
                for (int c = 0; c < K; c++) t[((size_t)z * K + c) * K + r] = w[oSc[1] + ((size_t)z * K + r) * K + c];
        oWscT1 = push(t);
    }
    for (int t = 0; t < 2; t++)
        for (int q = 0; q < nout[t]; q++) {
            const int np = npath[t][q];
            std::vector<float> v((size_t)S * np * K);
            for (int z = 0; z < S; z++)
                for (int k = 0; k < K; k++)
                    for (int e = 0; e < np; e++) v[((size_t)z * np + e) * K + k] = w[oSym[t][q] + ((size_t)z * K + k) * np + e];
            oSymT[t][q] = push(v);
        }
    const size_t oZero = push(std::vector<float>(512, 0.f));
    const size_t oHb0 = push(std::vector<float>((size_t)S * K, 0.f));
    const size_t oSkip0 = push(std::vector<float>((size_t)S * K, 0.f));
    float *dev = nullptr;
    if (hipMalloc(&dev, sizeof(float) * host.size()) != hipSuccess) {
        (void)hipGetLastError();
        delete a;
        return fail(-2, "mace: weight allocation failed");
    }
    if (hipMemcpy(dev, host.data(), sizeof(float) * host.size(), hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(dev);
        delete a;
        return fail(-5, "mace: weight copy failed");
    }
    a->dev = dev;
    for (int t = 0; t < 2; t++)
        for (int q = 0; q < nout[t]; q++) {
            a->Wsym[t][q] = dev + oSymT[t][q];
            a->WoutT[t][q] = dev + oWoutT[t][q];
            a->Wout[t][q] = dev + oOut[t][q];
        }
    for (int l2 = 0; l2 < 2; l2++) {
        a->WupT1[l2] = dev + oWupT1[l2];
        a->Wup1[l2] = dev + oUp[1][l2];
    }
    a->WscT1 = dev + oWscT1;
    a->Wsc1 = dev + oSc[1];
    a->zero = dev + oZero;
    a->hb0tab = dev + oHb0;
    a->skip0tab = dev + oSkip0;
    a->w_r1 = dev + oR1;
    a->W_r2 = dev + oWR2;
    a->b_r2 = dev + oBR2;
    a->w_r2 = dev + oWr2;
    k_mc_species<<<nblk((long)S * K, 256), 256>>>(S, dev + oEmb, dev + oUp[0][0], dev + oSc[0], dev + oHb0,
                                                   dev + oSkip0);
    // GEMM operands: radial matrices and W_A, forward and adjoint
    struct Item {
        const float *W;
        int R, C;
        bool tr;
        PackedW *dst;
    };
    if (int rc = mc_pack_chain(a, node_operands(m->precision), w, oRad)) {
        hipFree(dev);
        delete a;
        return rc;
    }
    std::vector<Item> items;
    for (int t = 0; t < 2; t++) {
        int prev = NB;
        for (int q = 0; q <= d.nrad; q++) {
            const int rows = q < d.nrad ? d.rh[q] : NPt[t] * K;
            items.push_back({dev + oRad[t][q], rows, prev, false, &a->radF[t][q]});
            items.push_back({dev + oRad[t][q], rows, prev, true, &a->radA[t][q]});
            prev = rows;
        }
        for (int L = 0; L < 4; L++) {
            const int cols = cp_nL(L, NPt[t]) * K;
            items.push_back({dev + oWA[t][L], K, cols, false, &a->waF[t][L]});
            items.push_back({dev + oWA[t][L], K, cols, true, &a->waA[t][L]});
        }
    }
    size_t pk = 0;
    for (const Item &it : items) pk += packed_bytes(it.R, it.C, it.tr);
    int rc = hipMalloc(&a->pk_dev, pk) == hipSuccess ? 0 : -2;
    for (size_t q = 0, o = 0; rc == 0 && q < items.size(); q++) {
        if (pack_weight(nullptr, items[q].W, items[q].R, items[q].C, items[q].tr, (char *)a->pk_dev + o, items[q].dst))
            rc = -5;
        o += packed_bytes(items[q].R, items[q].C, items[q].tr);
    }
    if (rc == 0 && (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess)) rc = -5;
    if (rc) {
        (void)hipGetLastError();
        if (a->pk_dev) hipFree(a->pk_dev);
        if (a->chain) hipFree(a->chain);
        hipFree(dev);
        delete a;
        return fail(rc, "mace: weight packing failed");
    }
    for (int t = 0; t < 2; t++) {
        a->rmlp[t].nh = d.nrad;
        for (int q = 0; q <= d.nrad; q++) {
            a->rmlp[t].f[q] = a->radF[t][q];
            a->rmlp[t].a[q] = a->radA[t][q];
        }
    }
    m->mc = a;
    return 0;
}

void mace_destroy(mlp_model *m) {
    if (!m || !m->mc) return;
    if (m->mc->pk_dev) hipFree(m->mc->pk_dev);
    if (m->mc->chain) hipFree(m->mc->chain);
    if (m->mc->dev) hipFree(m->mc->dev);
    delete m->mc;
    m->mc = nullptr;
}

static int mgm(hipStream_t s, int P, int epi, const float *A, int lda, const PackedW &B, float *C, int ldc, long M,
               const int *Mc, const float *bias = nullptr, float *C2 = nullptr, int ldc2 = 0,
               const float *R = nullptr, int ldr = 0) {
    if (M <= 0) return 0;
    ProfScope ps(PK_GEMM, s);
    return node_gemm(s, P, epi, A, lda, B, C, ldc, (int)M, bias, C2, ldc2, R, ldr, Mc) ? fail(-5, "mace GEMM failed")
                                                                                         : 0;
}

// The W_A channel mixes of nd atoms, one product per degree over (atom, m)
// rows, in one launch: A' = A W_A (fwd) or dE/dA = dE/dA' W_A^T.
static int mix_wa(hipStream_t s, int P, const McBlk &AR, const McBlk &AP, const PackedW *W, int np, int nd, bool fwd) {
    GemmBatch b;
    b.n = 4;
    for (int L = 0; L < 4; L++) {
        const int ld = cp_nL(L, np) * MK;
        b.A[L] = fwd ? AR.p[L] : AP.p[L];
        b.lda[L] = fwd ? ld : MK;
        b.B[L] = W[L];
        b.C[L] = fwd ? AP.p[L] : AR.p[L];
        b.ldc[L] = fwd ? MK : ld;
        b.M[L] = nd * (2 * L + 1);
    }
    ProfScope ps(PK_GEMM, s);
    return node_gemm_batch(s, P, b) ? fail(-5, "mace GEMM failed") : 0;
}

int mace_evaluate(mlp_model *m, mlp_nbr *g, hipStream_t s, double *energy, float *forces_user,
                  float *atom_energy_user, int n_seg, const int *seg_dev) {
    const McModel &a = *m->mc;
    const int n = g->n_atoms, P = node_operands(m->precision), T = 2;
    const long E = g->n_edges_skin;
    int rc;
    if ((rc = g->act.ensure(mace_arena_bytes(m, n, E, g->skin), 1.2, &g->n_grows))) return rc;
    if ((rc = g->G.ensure(sizeof(float4) * (size_t)E + 64, 1.2, &g->n_grows))) return rc;
    const bool fused = mc_edge_kernels(a, n, E, g->skin);
    const McArena L = mc_layout(a, n, E, fused);
    float *base = g->act.as<float>();
    float *X0 = base + L.X0, *Y = base + L.Y, *GY = base + L.GY, *GX0 = base + L.GX0, *MSG = base + L.MSG,
          *H1 = base + L.H1, *HB1 = base + L.HB1, *H2 = base + L.H2, *GH1S = base + L.GH1S, *U = base + L.U;
    const int *rowc = g->rowc.as<int>(), *colc = g->colc.as<int>(), *revc = g->revc.as<int>(),
              *perm = g->perm.as<int>(), *zsp = g->species.as<int>();
    const float4 *geom = g->geom.as<float4>();
    // rows each layer's node work covers: the first layer the atoms within
    // one hop of the locals, the second the locals (all rows without ghosts)
    const bool ho = g->nhop[0] > 0 && g->nhop[T + 1] == n;
    const int nd0 = ho ? g->nhop[1] : n, nd1 = ho ? g->nhop[0] : n;
    // edge rows of each layer: a prefix of the destination-sorted edges,
    // counted on the device
    const int *e0 = rowc + nd0, *e1 = rowc + nd1;
    const float scale = 1.0f / a.navg;
    const int NPt[2] = {4, 10};
    auto blk = [&](long o, int t) {
        McBlk b;
        long q = o;
        for (int Lq = 0; Lq < 4; Lq++) {
            b.p[Lq] = base + q;
            q += (long)n * (2 * Lq + 1) * (t < 0 ? 1 : cp_nL(Lq, NPt[t])) * MK;
        }
        return b;
    };
    const McBlk AR0 = blk(L.AR[0], 0), AR1 = blk(L.AR[1], 1), AP0 = blk(L.AP[0], -1), AP1 = blk(L.AP[1], -1),
                GAP = blk(L.GAP, -1);
    const int eg = (int)std::max<long>(1, std::min<long>(nblk(E, 256), 16384));

    // the edge kernels of the fused path
    McEdgeArgs ka{};
    ka.rowc = rowc;
    ka.colc = colc;
    ka.zsp = zsp;
    ka.geom = geom;
    ka.pe = a.pe;
    ka.rc = a.rc;
    ka.irc = 1.0f / a.rc;
    ka.c0 = std::sqrt(2.0f / a.rc);
    ec_phase(a.rc, ka.th, ka.thl);
    ka.scale = scale;
    ka.MSG = MSG;
    ka.G = g->G.as<float4>();
    ka.n = n;
    ka.nd1 = nd1;
    ka.per_wg = ec_per_wg(n, E, a.rc, g->skin, MC_SLOTS);
    auto edges = [&](int t, bool fwd, int nd, const McBlk &A) {
        McEdgeArgs k = ka;
        k.nd = nd;
        k.A = A;
        k.W = a.chain + (fwd ? a.chF[t] : a.chB[t]);
        k.hb = t ? HB1 : a.hb0tab;
        // the forward hands its atoms out to eight waves: one each as long as
        // every compute unit (256 of an MI355X) has a workgroup, then up to eight each
        if (fwd) k.per_wg = nd <= 2048 ? (nd + 255) / 256 : std::max(8, std::min(MC_FWD_ATOMS, nd / 2048));
        const bool split = fwd && k.per_wg <= 4;
        const int nb = nblk(nd, k.per_wg);
        ProfScope ps(PK_GEMM, s);
#define EK(P_)                                                                          \
    do {                                                                                \
        if (fwd && t == 0 && split) k_mc_edge_fwd<P_, 0, true><<<nb, EC_THREADS, 0, s>>>(k); \
        else if (fwd && t == 0) k_mc_edge_fwd<P_, 0, false><<<nb, EC_THREADS, 0, s>>>(k); \
        else if (fwd && split) k_mc_edge_fwd<P_, 1, true><<<nb, EC_THREADS, 0, s>>>(k);  \
        else if (fwd) k_mc_edge_fwd<P_, 1, false><<<nb, EC_THREADS, 0, s>>>(k);          \
        else if (t == 0) k_mc_edge_bwd<P_, 0><<<nb, EC_THREADS, 0, s>>>(k);              \
        else k_mc_edge_bwd<P_, 1><<<nb, EC_THREADS, 0, s>>>(k);                          \
    } while (0)
        if (P == 0) EK(0);
        else if (P == 1) EK(1);
        else EK(2);
#undef EK
    };

    // forward
    k_mc_zero<<<nblk(n + 64, 256), 256, 0, s>>>(U, n + 64);
    if (!fused) k_mc_edge<<<eg, 256, 0, s>>>(rowc, n, geom, a.NB, a.NBP, a.pe, a.rc, X0, Y);
    for (int t = 0; t < 2 && !fused; t++) {
        if (a.fused) {
            ProfScope ps(PK_GEMM, s);
            if (edge_mlp_forward(s, P, a.rmlp[t], X0, a.NBP, base + L.R[t], NPt[t] * MK, (int)E, t ? e1 : e0))
                return fail(-5, "mace radial MLP failed");
            continue;
        }
        const float *in = X0;
        int ldin = a.NBP;
        for (int q = 0; q < a.nrad; q++) {
            if ((rc = mgm(s, P, GE_BIAS_SILU, in, ldin, a.radF[t][q], base + L.P[t][q], a.rh[q], E, t ? e1 : e0,
                          a.zero, base + L.A[t][q], a.rh[q])))
                return rc;
            in = base + L.A[t][q];
            ldin = a.rh[q];
        }
        if ((rc = mgm(s, P, GE_STORE, in, ldin, a.radF[t][a.nrad], base + L.R[t], NPt[t] * MK, E, t ? e1 : e0)))
            return rc;
    }
    McNodeArgs na{};
    na.skip0tab = a.skip0tab;
    na.WupT1[0] = a.WupT1[0];
    na.WupT1[1] = a.WupT1[1];
    na.WscT1 = a.WscT1;
    na.w_r1 = a.w_r1;
    na.W_r2 = a.W_r2;
    na.b_r2 = a.b_r2;
    na.w_r2 = a.w_r2;
    na.b_r3 = a.b_r3;
    na.RH = a.RH;
    na.H1 = H1;
    na.H1o = H1;
    na.HB1o = HB1;
    na.H2 = H2;
    na.U = U;
    na.nloc = nd1;
    na.np[0] = kSym0.np;
    na.np[1] = kSym1.np;
    for (int t = 0; t < 2; t++) {
        const int nd = t ? nd1 : nd0;
        if (nd <= 0) continue;
        const McBlk &AR = t ? AR1 : AR0, &AP = t ? AP1 : AP0;
        if (fused)
            edges(t, true, nd, AR);
        else if (t == 0)
            k_mc_conv<0><<<nblk(nd, APB), 256, 0, s>>>(rowc, colc, nd, Y, base + L.R[0], nullptr, zsp, a.hb0tab, scale,
                                                       AR);
        else
            k_mc_conv<1><<<nblk(nd, APB), 256, 0, s>>>(rowc, colc, nd, Y, base + L.R[1], HB1, zsp, a.hb0tab, scale, AR);
        if ((rc = mix_wa(s, P, AR, AP, a.waF[t], NPt[t], nd, true))) return rc;
        na.AP = AP;
        na.Wsym[0] = a.Wsym[t][0];
        na.Wsym[1] = a.Wsym[t][1];
        na.WoutT[0] = a.WoutT[t][0];
        na.WoutT[1] = a.WoutT[t][1];
        if (t == 0) k_mc_node<0><<<nblk(nd, APB), 256, 0, s>>>(nd, zsp, na);
        else k_mc_node<1><<<nblk(nd, APB), 256, 0, s>>>(nd, zsp, na);
    }
    HIP_TRY(hipGetLastError());
    if ((rc = launch_energy(s, U, perm, n, g->n_local, energy, atom_energy_user, n_seg, seg_dev,
                            reinterpret_cast<double *>(base + L.EP))))
        return rc;
    if (!forces_user) return 0;

    // adjoint
    McNodeBwdArgs nb{};
    nb.Wsc1 = a.Wsc1;
    nb.Wup1[0] = a.Wup1[0];
    nb.Wup1[1] = a.Wup1[1];
    nb.w_r1 = a.w_r1;
    nb.W_r2 = a.W_r2;
    nb.b_r2 = a.b_r2;
    nb.w_r2 = a.w_r2;
    nb.RH = a.RH;
    nb.H2 = H2;
    nb.GH1S = GH1S;
    nb.rowc = rowc;
    nb.colc = colc;
    nb.revc = revc;
    nb.MSG = MSG;
    nb.nd1 = nd1;
    nb.perm = perm;
    nb.n_local = g->n_local;
    nb.GAP = GAP;
    nb.np[0] = kSym0.np;
    nb.np[1] = kSym1.np;
    if (nd1 > 0) {
        nb.AP = AP1;
        nb.Wsym[0] = a.Wsym[1][0];
        nb.Wsym[1] = nullptr;
        nb.Wout[0] = a.Wout[1][0];
        nb.Wout[1] = a.Wout[1][0];
        k_mc_node1_bwd<<<nblk(nd1, APB), 256, 0, s>>>(nd1, zsp, nb);
        // dE/dA (before the W_A mix) over the A blocks
        if ((rc = mix_wa(s, P, AR1, GAP, a.waA[1], 10, nd1, false))) return rc;
        if (fused) edges(1, false, nd1, AR1);
        else k_mc_conv1_bwd<<<nblk(nd1, APB), 256, 0, s>>>(rowc, colc, nd1, Y, base + L.R[1], HB1, scale, AR1, GY, MSG);
    }
    if (nd0 > 0) {
        nb.AP = AP0;
        nb.Wsym[0] = a.Wsym[0][0];
        nb.Wsym[1] = a.Wsym[0][1];
        nb.Wout[0] = a.Wout[0][0];
        nb.Wout[1] = a.Wout[0][1];
        k_mc_node0_bwd<<<nblk(nd0, APB), 256, 0, s>>>(nd0, zsp, nb);
        if ((rc = mix_wa(s, P, AR0, GAP, a.waA[0], 4, nd0, false))) return rc;
        if (fused) edges(0, false, nd0, AR0);
        else
            k_mc_conv0_bwd<<<nblk(nd0, APB), 256, 0, s>>>(rowc, colc, nd0, nd1, Y, base + L.R[0], zsp, a.hb0tab, scale,
                                                          AR0, GY);
    }
    if (fused) {
        HIP_TRY(hipGetLastError());
        return launch_forces(s, rowc, revc, g->G.as<float4>(), perm, n, forces_user);
    }
    // the radial MLPs in reverse (dE/dR in R), the first layer's over all its
    // edges first (stored), then the second layer's added on its prefix
    for (int t = 0; t < 2; t++) {
        const int *cnt = t ? e1 : e0;
        if (a.fused) {
            ProfScope ps(PK_GEMM, s);
            if (edge_mlp_adjoint(s, P, a.rmlp[t], X0, a.NBP, base + L.R[t], NPt[t] * MK, GX0, a.NBP, t != 0, (int)E, cnt))
                return fail(-5, "mace radial MLP adjoint failed");
            continue;
        }
        const float *gin = base + L.R[t];
        int ldg = NPt[t] * MK;
        for (int q = a.nrad - 1; q >= 0; q--) {
            float *dst = base + L.A[t][q];
            if ((rc = mgm(s, P, GE_DSILU, gin, ldg, a.radA[t][q + 1], dst, a.rh[q], E, cnt, nullptr, nullptr, 0,
                          base + L.P[t][q], a.rh[q])))
                return rc;
            gin = dst;
            ldg = a.rh[q];
        }
        if ((rc = mgm(s, P, t ? GE_ADD : GE_STORE, gin, ldg, a.radA[t][0], GX0, a.NBP, E, cnt, nullptr, nullptr, 0,
                      GX0, a.NBP)))
            return rc;
    }
    k_mc_geom<<<eg, 256, 0, s>>>(rowc, n, e0, geom, a.NB, a.NBP, a.pe, a.rc, GX0, GY, g->G.as<float4>());
    HIP_TRY(hipGetLastError());
    return launch_forces(s, rowc, revc, g->G.as<float4>(), perm, n, forces_user);
}

}  // namespace mlp
