// Allegro with a single tensor-product layer: energy and forces on the
// pruned neighbour graph.
//
// The paper deploys Allegro (Methods, "Chosen Architectures": edge-centric
// and strictly local; messages pass only between directed edges that share
// their central atom) with one tensor-product layer, l_max = 3, 8 radial
// functions and a polynomial envelope of order 2 for water and aluminium
// ("Training Details").  Per directed edge e = (i <- j), r = |r_j - r_i| < rc,
// rhat = (r_j - r_i) / r, with the layer equations of the cited Allegro
// paper in this reading:
//   u(r)  = 1 - (p+1)(p+2)/2 x^p + p(p+2) x^(p+1) - p(p+1)/2 x^(p+2),  x = r / rc
//   B_k   = sqrt(2 / rc) sin(k pi r / rc) / r u(r)
//   x0    = u(r) MLP_2b([onehot(Z_i) | onehot(Z_j) | B])
//   w0 = Wv x0,  we = We x0                     (one weight per channel c)
//   env_i[c, m] = nu sum_(edges i <- k) we_ik[c] Y_(l_c m)(rhat_ik)
//   S_e[c] = w0_e[c] / (2 l_c + 1) sum_m Y_(l_c m)(rhat_e) env_i[c, m]
//                                 (the l x l -> 0 outputs of the tensor
//                                  product of V_e = w0_e Y(rhat_e) with env_i)
//   x1  = (x0 + u(r) MLP_lat([x0 | S_e])) / sqrt(2)
//   E_e = u(r) MLP_out(x1),  U_i = sum_(edges i <- j) E_e,  E = sum_(i local) U_i
// Y are component-normalised real spherical harmonics (sum_m Y_lm^2 = 2l+1)
// in Cartesian form.  The environment is built once per atom and the scalar
// outputs contracted against it per edge, so the per-edge angular work is
// O(l_max^2) instead of a sum over pairs of edges.  One kernel (k_al_atoms)
// takes runs of whole atoms through all of it, forward and adjoint; widths it
// does not take run a kernel per step, the MLPs as GEMMs over edges (gemm.hip).
// Forces come from a hand-written adjoint: the MLPs transposed, the
// tensor-product contraction reversed per atom (a gradient of the environment
// accumulated over the atom's edges, then sent back to each edge), and per edge G_e = dE/d(r_i - r_j), assembled into
// forces by gathering through the reverse-edge index (no atomics).
#include "internal.h"
#include "gemm.h"
#include "sh.h"
#include "edge_chain.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace mlp {

static inline int nblk(long n, int t) { return (int)((n + t - 1) / t); }
static inline int up4(int x) { return (x + 3) / 4 * 4; }

__device__ __forceinline__ float al_sigmoid(float x) { return 1.0f / (1.0f + __expf(-x)); }
__device__ __forceinline__ float al_dsilu(float x) {
    const float s = al_sigmoid(x);
    return s * (1.0f + x * (1.0f - s));
}

struct AlModel {
    AlDims d;
    int KIN = 0;     // columns of the two-body input, internal order [B | onehot_i | onehot_j | 0]
    int NBP = 0;     // radial functions padded to a multiple of 4
    float *vec = nullptr;                       // biases and the output vector on the device
    const float *b2b[6] = {}, *lat_b1 = nullptr, *lat_b2 = nullptr, *out_b1 = nullptr, *out_w2 = nullptr,
                *out_b2 = nullptr;
    float out_b2_host = 0.f;
    // B operands: forward (B = W^T) and adjoint (B = W); a2b[0] is the radial
    // block of the first two-body matrix only
    PackedW f2b[6], fVE, fL1, fL2, fO1;
    PackedW a2b[6], aVE, aL1, aL2, aO1;
    void *pk_dev = nullptr;
    // the whole evaluation in one kernel (k_al_atoms), where the widths fit it
    bool fused = false;
    char *chain = nullptr;                      // its weights in the order of use, then its constants
    const float *chain_vec = nullptr;
};

// ---------------------------------------------------------------------------
// Forward, per edge: envelope, radial functions, harmonics, two-body input.
// One wave per destination atom, lanes over its edges.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_al_edge_in(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                    const float4 *__restrict__ geom, const int *__restrict__ zsp,
                                                    const int *__restrict__ perm, int n, int n_local, int S, int NB,
                                                    int p, int KIN, float rc, float *__restrict__ H0,
                                                    float *__restrict__ U, float *__restrict__ Y,
                                                    float *__restrict__ GL) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int zi = zsp[i];
    const float loc = perm[i] < n_local ? 1.f : 0.f;   // dE/dE_e: the edge's atom is local
    const float c0 = sqrtf(2.0f / rc), th = 3.14159265358979f / rc;
    for (int e = rowc[i] + lane; e < rowc[i + 1]; e += 64) {
        const float4 gm = geom[e];
        const float r = gm.w, ir = 1.0f / r;
        float u, du;
        envelope(r / rc, p, u, du);
        float sn, cs;
        sincosf(th * r, &sn, &cs);
        float *h = H0 + (long)e * KIN;
        float sk = sn, skm = 0.f;
        for (int k = 0; k < NB; k++) {
            h[k] = c0 * sk * ir * u;
            const float nx = 2.f * cs * sk - skm;
            skm = sk;
            sk = nx;
        }
        const int zj = zsp[colc[e]];
        for (int q = NB; q < KIN; q++) h[q] = 0.f;
        h[NB + zi] = 1.f;
        h[NB + S + zj] = 1.f;
        U[e] = u;
        GL[e] = loc;
        float Ye[16];
        sh16(gm.x * ir, gm.y * ir, gm.z * ir, Ye);
        float4 *y4 = reinterpret_cast<float4 *>(Y + (long)e * 16);
#pragma unroll
        for (int q = 0; q < 4; q++) y4[q] = make_float4(Ye[4 * q], Ye[4 * q + 1], Ye[4 * q + 2], Ye[4 * q + 3]);
    }
}

// out[e][0..D) = u[e] * in[e][0..D) (row strides ldo, ldi), four per thread.
__global__ void k_al_scale_rows(const float *__restrict__ in, int ldi, const float *__restrict__ u,
                                const int *__restrict__ cnt, int D, float *__restrict__ out, int ldo) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int D4 = D / 4;
    const long e = t / D4;
    if (e >= *cnt) return;
    const int f = 4 * (int)(t % D4);
    const float s = u[e];
    const float4 x = *reinterpret_cast<const float4 *>(in + e * ldi + f);
    *reinterpret_cast<float4 *>(out + e * ldo + f) = make_float4(s * x.x, s * x.y, s * x.z, s * x.w);
}

// Channel layout of a lane (= channel c): its degree, first harmonic and the
// 1 / (2 l + 1) of the scalar path.
struct AlChan {
    int l, m0, nm;
    float inv;
    __device__ AlChan(int c, const AlDims &d) {
        int off = 0;
        l = 0;
        for (int q = 0; q <= d.lmax; q++) {
            if (c >= off && c < off + d.ch[q]) l = q;
            off += d.ch[q];
        }
        m0 = l * l;
        nm = 2 * l + 1;
        inv = 1.0f / (float)nm;
    }
};

// The edge's 16 harmonics (the same address in every lane of the wave, so
// they come through the scalar cache) and the lane's own components
// ym[m] = Y_(l, m) for m < 2l + 1, zero above.
__device__ __forceinline__ void al_lane_harm(const float *__restrict__ ye, int l, float *ym) {
    float y[16];
#pragma unroll
    for (int q = 0; q < 16; q++) y[q] = ye[q];
#pragma unroll
    for (int m = 0; m < 7; m++) {
        const float a = m < 1 ? y[m] : 0.f, b = m < 3 ? y[1 + m] : 0.f, c = m < 5 ? y[4 + m] : 0.f, dd = y[9 + m];
        ym[m] = l == 0 ? a : (l == 1 ? b : (l == 2 ? c : dd));
    }
}

// The environment of each atom and the scalar outputs of its edges.  One
// wave per atom (its index made wave-uniform, so the edge loop and the
// harmonic loads are scalar), lane = channel: pass 1 sums env[c][m] over the
// atom's edges, pass 2 contracts each edge's harmonics against it.
__global__ void __launch_bounds__(256) k_al_tp(const int *__restrict__ rowc, int n, AlDims d,
                                               const float *__restrict__ Y, const float *__restrict__ WV,
                                               float *__restrict__ ENV, float *__restrict__ LIN) {
    const int lane = threadIdx.x & 63;
    const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (i >= n) return;
    const int NC = d.NC, ldwv = 2 * d.NC, ldl = d.D + d.NC;
    if (lane >= NC) return;
    const AlChan ch(lane, d);
    const int e0 = rowc[i], e1 = rowc[i + 1];
    float env[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // unrolled so that several edges' loads are in flight together
#pragma unroll 4
    for (int e = e0; e < e1; e++) {
        const float we = WV[(long)e * ldwv + NC + lane];
        float ym[7];
        al_lane_harm(Y + (long)e * 16, ch.l, ym);
#pragma unroll
        for (int m = 0; m < 7; m++) env[m] = fmaf(we, ym[m], env[m]);
    }
    float *en = ENV + ((long)i * NC + lane) * 8;
#pragma unroll
    for (int m = 0; m < 7; m++) {
        env[m] *= d.nu;
        en[m] = env[m];
    }
#pragma unroll 4
    for (int e = e0; e < e1; e++) {
        float ym[7];
        al_lane_harm(Y + (long)e * 16, ch.l, ym);
        float dot = 0.f;
#pragma unroll
        for (int m = 0; m < 7; m++) dot = fmaf(ym[m], env[m], dot);
        LIN[(long)e * ldl + d.D + lane] = WV[(long)e * ldwv + lane] * ch.inv * dot;
    }
}

// x1 = (x0 + u m) / sqrt(2), x0 in the first D columns of LIN.
__global__ void k_al_x1(const float *__restrict__ LIN, int ldl, const float *__restrict__ u,
                        const float *__restrict__ M, const int *__restrict__ cnt, int D, float *__restrict__ X1) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int D4 = D / 4;
    const long e = t / D4;
    if (e >= *cnt) return;
    const int f = 4 * (int)(t % D4);
    const float s = u[e], r2 = 0.70710678118654752f;
    const float4 x = *reinterpret_cast<const float4 *>(LIN + e * ldl + f);
    const float4 m = *reinterpret_cast<const float4 *>(M + e * D + f);
    *reinterpret_cast<float4 *>(X1 + e * D + f) =
        make_float4(r2 * fmaf(s, m.x, x.x), r2 * fmaf(s, m.y, x.y), r2 * fmaf(s, m.z, x.z), r2 * fmaf(s, m.w, x.w));
}

// E_e = u (w2 . HO_e + b2) summed over each atom's edges.  One wave per atom:
// eight lane groups take the edges q, q + 8, ..., the eight lanes of a group
// the row's features four at a time (a row is read as whole 16-byte pieces);
// the sums run in a fixed order (group totals, then a butterfly).
__global__ void __launch_bounds__(256) k_al_energy(const int *__restrict__ rowc, int n, int OH,
                                                   const float *__restrict__ HO, const float *__restrict__ u,
                                                   const float *__restrict__ w2, float b2, float *__restrict__ Uat) {
    const int lane = threadIdx.x & 63, q = lane & 7, grp = lane >> 3;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int e1 = rowc[i + 1];
    float acc = 0.f;
    for (int eb = rowc[i]; eb < e1; eb += 8) {
        const int e = eb + grp;
        float dot = 0.f;
        if (e < e1)
            for (int f = 4 * q; f < OH; f += 32) {
                const float4 h = *reinterpret_cast<const float4 *>(HO + (long)e * OH + f);
                dot += h.x * w2[f] + h.y * w2[f + 1] + h.z * w2[f + 2] + h.w * w2[f + 3];
            }
        dot += __shfl_xor(dot, 1, 64);
        dot += __shfl_xor(dot, 2, 64);
        dot += __shfl_xor(dot, 4, 64);
        if (e < e1 && q == 0) acc = fmaf(u[e], dot + b2, acc);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) Uat[i] = acc;
}

// ---------------------------------------------------------------------------
// Adjoint
// ---------------------------------------------------------------------------

// dE/dE_e = GL[e] (1 for edges into a local atom, 0 otherwise).  Through
// E_e = u (w2 . silu(PO) + b2): GU[e] = dE/du (first part) and the gradient of
// the output layer's pre-activation, written over HO.  Eight lanes per edge,
// four features each.
__global__ void k_al_out_bwd(const int *__restrict__ cnt, int OH, const float *__restrict__ PO,
                             float *__restrict__ HO, const float *__restrict__ u, const float *__restrict__ GL,
                             const float *__restrict__ w2, float b2, float *__restrict__ GU) {
    const long ne = *cnt;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long e = t >> 3;
    const int q = (int)(t & 7);
    float dot = 0.f;
    if (e < ne) {
        const float gE = GL[e], s = gE * u[e];
        for (int f = 4 * q; f < OH; f += 32) {
            float4 *hp = reinterpret_cast<float4 *>(HO + e * OH + f);
            const float4 h = *hp, pp = *reinterpret_cast<const float4 *>(PO + e * OH + f);
            dot += h.x * w2[f] + h.y * w2[f + 1] + h.z * w2[f + 2] + h.w * w2[f + 3];
            *hp = make_float4(s * w2[f] * al_dsilu(pp.x), s * w2[f + 1] * al_dsilu(pp.y),
                              s * w2[f + 2] * al_dsilu(pp.z), s * w2[f + 3] * al_dsilu(pp.w));
        }
    }
    dot += __shfl_xor(dot, 1, 8);
    dot += __shfl_xor(dot, 2, 8);
    dot += __shfl_xor(dot, 4, 8);
    if (e < ne && q == 0) GU[e] = GL[e] * (dot + b2);
}

// Through x1 = (x0 + u m) / sqrt(2): with GX = dE/dx1 (in X), GU += GX . m / sqrt(2),
// M <- dE/dm = u GX / sqrt(2), X <- dE/dx0 (this path) = GX / sqrt(2).
// Sixteen lanes per edge, four features per lane per step.
__global__ void k_al_x1_bwd(const int *__restrict__ cnt, int D, const float *__restrict__ u, float *__restrict__ X,
                            float *__restrict__ M, float *__restrict__ GU) {
    const long ne = *cnt;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long e = t >> 4;
    const int q = (int)(t & 15);
    const float r2 = 0.70710678118654752f;
    float part = 0.f;
    if (e < ne) {
        const float s = u[e] * r2;
        for (int f = 4 * q; f < D; f += 64) {
            float4 *xp = reinterpret_cast<float4 *>(X + e * D + f);
            float4 *mp = reinterpret_cast<float4 *>(M + e * D + f);
            const float4 gx = *xp, m = *mp;
            part += gx.x * m.x + gx.y * m.y + gx.z * m.z + gx.w * m.w;
            *mp = make_float4(s * gx.x, s * gx.y, s * gx.z, s * gx.w);
            *xp = make_float4(r2 * gx.x, r2 * gx.y, r2 * gx.z, r2 * gx.w);
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) part += __shfl_xor(part, off, 16);
    if (e < ne && q == 0) GU[e] += r2 * part;
}

template <int CTRL>
__device__ __forceinline__ float al_dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// The sums over the channels of each degree of q[m] (m < 2l + 1), stored as
// GY[slot l^2 + m] (add: accumulate).  STD: the channel layout (32, 16, 8, 8)
// of degrees 0..3 over the 64 lanes, summed by DPP exchanges (8-lane groups
// by quad permutations and the half-row mirror, 16-lane rows by a row
// rotation, the two rows of degree 0 by one cross-row exchange); otherwise
// through the wave's LDS rows.
template <bool STD>
__device__ __forceinline__ void al_channel_sums(const float *q, int lane, int ny, int kc0, int kc1, int km,
                                                float (*red)[8], float *__restrict__ gy, bool add) {
    if constexpr (STD) {
        float v8[7], v16[3], v32 = 0.f;
#pragma unroll
        for (int m = 0; m < 7; m++) {
            float v = q[m];
            v += al_dpp<0xB1>(v);    // quad_perm [1,0,3,2]
            v += al_dpp<0x4E>(v);    // quad_perm [2,3,0,1]
            v += al_dpp<0x141>(v);   // row_half_mirror: the other quad of the 8
            v8[m] = v;
        }
#pragma unroll
        for (int m = 0; m < 3; m++) v16[m] = v8[m] + al_dpp<0x128>(v8[m]);   // row_ror:8
        v32 = v16[0] + __shfl_xor(v16[0], 16, 64);
        if (lane == 0) gy[0] = add ? gy[0] + v32 : v32;
        if (lane == 32)
#pragma unroll
            for (int m = 0; m < 3; m++) gy[1 + m] = add ? gy[1 + m] + v16[m] : v16[m];
        if (lane == 48)
#pragma unroll
            for (int m = 0; m < 5; m++) gy[4 + m] = add ? gy[4 + m] + v8[m] : v8[m];
        if (lane == 56)
#pragma unroll
            for (int m = 0; m < 7; m++) gy[9 + m] = add ? gy[9 + m] + v8[m] : v8[m];
    } else {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int m = 0; m < 7; m++) red[lane][m] = q[m];
        __builtin_amdgcn_wave_barrier();
        if (lane < ny) {
            float s = 0.f;
            for (int c = kc0; c < kc1; c++) s += red[c][km];
            gy[lane] = add ? gy[lane] + s : s;
        }
    }
}

// Adjoint of k_al_tp, one wave per atom, lane = channel.  With t = dE/dS_e:
//   pass 1: dE/dw0_e[c] = t Y_e . env[c],  genv[c] += t w0_e[c] Y_e,
//           dE/dY_e[m] += sum_c t w0_e[c] env[c][m];   also X <- X + GLIN[:, :D]
//   pass 2 (genv scaled by nu): dE/dwe_e[c] = genv[c] . Y_e,
//           dE/dY_e[m] += sum_c genv[c][m] we_e[c]
template <bool STD>
__global__ void __launch_bounds__(256) k_al_tp_bwd(const int *__restrict__ rowc, int n, AlDims d,
                                                   const float *__restrict__ Y, const float *__restrict__ WV,
                                                   const float *__restrict__ ENV, const float *__restrict__ GLIN,
                                                   float *__restrict__ X, float *__restrict__ GWV,
                                                   float *__restrict__ GY) {
    __shared__ float red[4][64][8];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + w);
    if (i >= n) return;
    const int NC = d.NC, ldwv = 2 * d.NC, ldl = d.D + d.NC, D = d.D;
    const bool act = lane < NC;
    const AlChan ch(act ? lane : 0, d);
    // the harmonic a lane sums in the LDS reductions (lanes 0..15): degree,
    // order, and the channel range of that degree
    int kl = 0, kc0 = 0, kc1 = 0;
    {
        int off = 0;
        for (int q = 0; q <= d.lmax; q++) {
            if (lane >= q * q && lane < (q + 1) * (q + 1)) {
                kl = q;
                kc0 = off;
                kc1 = off + d.ch[q];
            }
            off += d.ch[q];
        }
    }
    const int ny = (d.lmax + 1) * (d.lmax + 1);
    const int km = lane - kl * kl;
    float env[7], genv[7];
#pragma unroll
    for (int m = 0; m < 7; m++) {
        env[m] = act ? ENV[((long)i * NC + lane) * 8 + m] : 0.f;
        genv[m] = 0.f;
    }
    const int e0 = rowc[i], e1 = rowc[i + 1];
#pragma unroll 2
    for (int e = e0; e < e1; e++) {
        float q[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float ym[7];
        al_lane_harm(Y + (long)e * 16, ch.l, ym);
        if (act) {
            const float t = GLIN[(long)e * ldl + D + lane] * ch.inv;
            const float w0 = WV[(long)e * ldwv + lane];
            float dot = 0.f;
#pragma unroll
            for (int m = 0; m < 7; m++) {
                dot = fmaf(ym[m], env[m], dot);
                genv[m] = fmaf(t * w0, ym[m], genv[m]);
                q[m] = t * w0 * env[m];
            }
            GWV[(long)e * ldwv + lane] = t * dot;
        }
        for (int f = lane; f < D; f += 64) X[(long)e * D + f] += GLIN[(long)e * ldl + f];
        al_channel_sums<STD>(q, lane, ny, kc0, kc1, km, red[w], GY + (long)e * 16, false);
    }
#pragma unroll
    for (int m = 0; m < 7; m++) genv[m] *= d.nu;
#pragma unroll 2
    for (int e = e0; e < e1; e++) {
        float q[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float ym[7];
        al_lane_harm(Y + (long)e * 16, ch.l, ym);
        if (act) {
            const float we = WV[(long)e * ldwv + NC + lane];
            float dot = 0.f;
#pragma unroll
            for (int m = 0; m < 7; m++) {
                dot = fmaf(genv[m], ym[m], dot);
                q[m] = genv[m] * we;
            }
            GWV[(long)e * ldwv + NC + lane] = dot;
        }
        al_channel_sums<STD>(q, lane, ny, kc0, kc1, km, red[w], GY + (long)e * 16, true);
    }
}

// Through x0 = u y: GU += GX0 . y, and Yo <- dE/dy = u GX0.
__global__ void k_al_x0_bwd(const int *__restrict__ cnt, int D, const float *__restrict__ u,
                            const float *__restrict__ GX0, float *__restrict__ Yo, float *__restrict__ GU) {
    const long ne = *cnt;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long e = t >> 4;
    const int q = (int)(t & 15);
    float part = 0.f;
    if (e < ne) {
        const float s = u[e];
        for (int f = 4 * q; f < D; f += 64) {
            const float4 g = *reinterpret_cast<const float4 *>(GX0 + e * D + f);
            float4 *yp = reinterpret_cast<float4 *>(Yo + e * D + f);
            const float4 y = *yp;
            part += g.x * y.x + g.y * y.y + g.z * y.z + g.w * y.w;
            *yp = make_float4(s * g.x, s * g.y, s * g.z, s * g.w);
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) part += __shfl_xor(part, off, 16);
    if (e < ne && q == 0) GU[e] += part;
}

// Per edge: dE/dr from the radial functions and the envelope, dE/drhat from
// the harmonics, G_e = dE/d(r_i - r_j) = -(dE/dr rhat + (I - rhat rhat^T) dE/drhat / r).
__global__ void k_al_geom_bwd(const int *__restrict__ rowc, int n, const float4 *__restrict__ geom, int NB,
                              int NBP, int p, float rc, const float *__restrict__ GB, const float *__restrict__ GU,
                              const float *__restrict__ GY, float4 *__restrict__ G) {
    const long ne = rowc[n];
    const float c0 = sqrtf(2.0f / rc), th = 3.14159265358979f / rc;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += (long)gridDim.x * blockDim.x) {
        const float4 gm = geom[e];
        const float r = gm.w, ir = 1.0f / r;
        float u, du;
        envelope(r / rc, p, u, du);
        du *= 1.0f / rc;
        float sn, cs;
        sincosf(th * r, &sn, &cs);
        const float *gb = GB + e * NBP;
        float dEdr = GU[e] * du;
        float sk = sn, skm = 0.f, ck = cs, ckm = 1.f;
        for (int k = 0; k < NB; k++) {
            const float kt = (k + 1) * th;
            // d/dr [c0 sin(k th r) / r u] = c0 [(k th cos / r - sin / r^2) u + sin / r u']
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
        const float4 *g4 = reinterpret_cast<const float4 *>(GY + e * 16);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const float4 v = g4[q];
            gy[4 * q] = v.x;
            gy[4 * q + 1] = v.y;
            gy[4 * q + 2] = v.z;
            gy[4 * q + 3] = v.w;
        }
        float hx, hy, hz;
        sh16_grad(x, y, z, gy, hx, hy, hz);
        const float rd = hx * x + hy * y + hz * z;
        const float gx = dEdr * x + (hx - rd * x) * ir, gyy = dEdr * y + (hy - rd * y) * ir,
                    gz = dEdr * z + (hz - rd * z) * ir;
        G[e] = make_float4(-gx, -gyy, -gz, 0.f);
    }
}

// ---------------------------------------------------------------------------
// The whole evaluation of an atom in one kernel: Allegro is strictly local,
// so an atom's energy and the gradients of all its edges need its own edges
// only, and nothing per edge but the geometry and the final G touches HBM
// (32 bytes; the kernels above keep about 870 floats per edge).
//
// A workgroup of eight waves takes a run of whole atoms with up to 128 edges
// in all (16 per wave, a lane quarter g of each edge's features; see
// edge_chain.h) through three phases:
//   1  geometry, two-body MLP, x0, w0, we;        sum we Y   -> env of each atom
//   2  S, latent MLP, output MLP, E and back down to dE/dS;
//                                                 sum t w0 Y -> genv of each atom
//   3  dE/dwe, the two-body MLP again and the rest of the adjoint, G.
// The sums over an atom's edges go through an LDS tile [edge][channel] (and
// the harmonics [edge][16]): one thread per (channel, m) of an atom runs over
// its edges in order.  An atom with more edges than a workgroup's 128 goes
// through the phases in pieces, the earlier phases recomputed instead of kept.
// Channels (32, 16, 8, 8) of degrees 0..3: tiles 0, 1 are degree 0, tile 2
// degree 1, tile 3 degree 2 in the lane groups 0, 1 and degree 3 in 2, 3.
//
// What bounds it: the chain of dependent layers at two waves per SIMD.  Busy,
// split bf16 at 470,596 atoms: vector issue 44 %, LDS 34 %, matrix cores 25 %,
// data return of the vector loads 19 %, some instruction issued in 63 % of the
// cycles; no unit is full.  Of a run of 125 edges the sums over atoms and the
// geometry, whose loads for the next run are issued ahead of phase 3, are a
// quarter of the time.  Four waves per SIMD need 128 registers and spill (12.0
// against 11.5 ms).
// Measured on 470,596 atoms of fcc aluminium (14.7M edges), split bf16: 64.1 ms
// per evaluation with a kernel per step, 11.2 ms with this one, which takes
// 10.8 of them; 1,536 atoms of water in FP32: 0.84 ms and 0.12 ms (the kernel
// 0.106; 0.20 with one atom to a workgroup and SiLU' formed again in the
// adjoint).
// ---------------------------------------------------------------------------
// (atoms of a run: what LDS holds of env.  With six, a gas of one neighbour per
// atom filled six rows of 128: 100,000 atoms, split bf16, 1.39 ms, 0.43 so, and
// 0.53 with a kernel per step; of eight neighbours 1.64, 1.04 and 3.39 ms)
constexpr int AF_TS = 68, AF_ENV = 224, AF_SLOTS = 60;
// constants in LDS: biases and the output vector, zero-padded
constexpr int AF_B1 = 0, AF_B2 = 16, AF_B3 = 32, AF_B4 = 64, AF_L1 = 128, AF_L2 = 192, AF_O1 = 256, AF_W2 = 288,
              AF_VEC = 320;

struct AlAtomsArgs {
    const int *rowc, *colc, *zsp, *perm;
    const float4 *geom;
    int n, n_local, per_wg, S, p, want_G;
    float rc, nu, b2, irc, c0, th, thl;   // 1 / rc, sqrt(2 / rc), pi / rc in two parts
    const char *W;
    const float *vec;
    float *U;
    float4 *G;
};

template <int P>
__global__ void __launch_bounds__(EC_THREADS) __attribute__((amdgpu_waves_per_eu(2))) k_al_atoms(AlAtomsArgs A) {
    typedef ec_v4f v4f;
    constexpr int N1 = 24 / EcStream<P>::U, N2 = 56 / EcStream<P>::U, N3 = 32 / EcStream<P>::U;   // stages
    __shared__ __attribute__((aligned(16))) char wst[2 * EcStream<P>::SB];
    __shared__ __attribute__((aligned(16))) float tile[EC_ROWS * AF_TS], ys[EC_ROWS * 16], eg[EC_ROWS * 8],
        en[AF_SLOTS * AF_ENV], cb[AF_VEC], es[EC_ROWS];
    __shared__ int roff[AF_SLOTS + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4,
              row = 16 * w + (lane & 15);
    const v4f z4 = v4f{0.f, 0.f, 0.f, 0.f};
    for (int q = tid; q < min(AF_SLOTS, A.per_wg + 1) * AF_ENV; q += EC_THREADS) en[q] = 0.f;   // the padding stays zero
    if (tid < AF_VEC) cb[tid] = A.vec[tid];
    const char *W1 = A.W, *W2 = W1 + N1 * EcStream<P>::SB, *W3 = W2 + N2 * EcStream<P>::SB;
    EcStream<P> st;
    st.start(wst, W1);
    const float *cbg = cb + 4 * g, *yr = ys + 16 * row, *er = eg + 8 * row;
    float *tr = tile + row * AF_TS + 4 * g;
    auto cbv = [&](int o, int t) { return *reinterpret_cast<const v4f *>(cbg + o + 16 * t); };
    const float r2 = 0.70710678118654752f, inv1 = 1.0f / 3.0f, inv3 = g < 2 ? 0.2f : 1.0f / 7.0f;

    const int a1 = min(A.n, ((int)blockIdx.x + 1) * A.per_wg);
    int a = blockIdx.x * A.per_wg;
    if (a >= a1) return;
    // What the first waves (a thread per edge) load of a piece.
    struct Edge {
        float4 gm;
        int zi, cj, pm, slot;
        bool valid;
    };
    auto edge_loads = [&](Edge &E, int a_, int base, int off, const EcRun &r, int ch) __attribute__((always_inline)) {
        if (w < EC_ROWS / 64) {
            E.slot = ec_slot(tid, r, off);
            E.valid = tid < min(EC_ROWS, r.total - ch * EC_ROWS);
            const int e = base + ch * EC_ROWS + (E.valid ? tid : 0);
            E.gm = A.geom[e];
            E.cj = A.colc[e];
            E.zi = A.zsp[a_ + E.slot];
            E.pm = A.perm[a_ + E.slot];
        }
    };
    int base = A.rowc[a], off = ec_row_off<AF_SLOTS>(A.rowc, lane, a, a1) - base;
    Edge ed;
    bool have = false;   // the run's first piece is in ed
    while (a < a1) {
        __syncthreads();   // the last reads of the previous run's LDS
        const EcRun run = ec_run<AF_SLOTS>(lane, a, a1, off);
        const int na = run.na, nch = run.nch, total = run.total;
        // the row offsets of the run after this one
        const int an = min(a + na, a1), nbase = A.rowc[an], noff = ec_row_off<AF_SLOTS>(A.rowc, lane, an, a1);
        if (total == 0) {
            if (tid < na) A.U[a + tid] = 0.f;
            a += na;
            base = nbase;
            off = noff - nbase;
            have = false;
            continue;
        }
        const int prev = __shfl_up(off, 1, 64);   // (every lane active)
        if (w == 0 && lane <= na) roff[lane] = lane ? prev : 0;

        // Per edge in LDS: the harmonics, and 1 / r, the envelope and its
        // r-derivative, sin and cos of pi r / rc, dE/dE_e (1 where the atom is
        // local), the species of both atoms, the atom's slot.
        auto geometry = [&](int ch) __attribute__((always_inline)) {
            if (nch > 1) __syncthreads();   // the last reads of the previous piece's rows
            if (!have) edge_loads(ed, a, base, off, run, ch);
            have = false;
            if (w < EC_ROWS / 64) {
                const int q = tid, zj = A.zsp[ed.cj];
                const float r = ed.gm.w, ir = 1.0f / r;
                float u, du;
                envelope(r / A.rc, A.p, u, du);
                float s1, c1, Y[16];
                ec_sincos_0pi<P>(A.th, A.thl, r, s1, c1);
                sh16(ed.gm.x * ir, ed.gm.y * ir, ed.gm.z * ir, Y);
#pragma unroll
                for (int k = 0; k < 4; k++)
                    *reinterpret_cast<v4f *>(ys + 16 * q + 4 * k) = v4f{Y[4 * k], Y[4 * k + 1], Y[4 * k + 2], Y[4 * k + 3]};
                // rows past the end carry nothing: u = 0
                *reinterpret_cast<v4f *>(eg + 8 * q) = v4f{ir, ed.valid ? u : 0.f, du * A.irc, s1};
                *reinterpret_cast<v4f *>(eg + 8 * q + 4) =
                    v4f{c1, ed.valid && ed.pm < A.n_local ? 1.f : 0.f, __int_as_float(ed.zi + 256 * zj),
                        __int_as_float(ed.slot)};
            }
            __syncthreads();
            return min(EC_ROWS, total - ch * EC_ROWS);
        };
        auto put_tile = [&](const v4f *v) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; t++) *reinterpret_cast<v4f *>(tr + 16 * t) = v[t];
        };
        // dst[slot][c, m] (+)= nu sum over the slot's rows of tile[row][c] Y_m[row]:
        // per atom and 16-channel tile a product over the atom's rows on the
        // FP32 matrix instruction (rows past the atom's last enter as that one
        // times zero: another atom's may not be finite), of which the m of the
        // channels' degrees are kept
        auto atom_sums = [&](float *dst, int nr, bool add) __attribute__((always_inline)) {
            const int m = lane & 15;
            for (int task = w; task < 4 * na; task += EC_THREADS / 64) {
                const int s = task >> 2, t = task & 3;
                const int q0 = nch > 1 ? 0 : roff[s], q1 = nch > 1 ? nr : roff[s + 1];
                v4f acc = z4;
                for (int q = q0; q < q1; q += 32) {
                    float x[8], y[8];
#pragma unroll
                    for (int k = 0; k < 8; k++) {
                        const int rr = q + 4 * k + g, rc = min(rr, q1 - 1);
                        x[k] = tile[rc * AF_TS + 16 * t + m];
                        x[k] = rr < q1 ? x[k] : 0.f;
                        y[k] = ys[rc * 16 + m];
                    }
#pragma unroll
                    for (int k = 0; k < 8; k++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[k], y[k], acc, 0, 0, 0);
                }
                acc *= A.nu;
                // lane (m, g): channels 16 t + 4 g + r
                const int lo = t < 2 ? 0 : (t == 2 ? 1 : (g < 2 ? 4 : 9)), hi = t < 2 ? 1 : (t == 2 ? 4 : (g < 2 ? 9 : 16));
                if (m >= lo && m < hi) {
                    const int st_ = t < 2 ? 1 : (t == 2 ? 4 : 8);
                    float *d = dst + s * AF_ENV + (t < 2 ? 16 * t : (t == 2 ? 32 : 96)) + 4 * g * st_ + m - lo;
#pragma unroll
                    for (int k = 0; k < 4; k++) d[k * st_] = add ? d[k * st_] + acc[k] : acc[k];
                }
            }
        };
        // energies of the atoms, their edges' terms added in a fixed order
        auto atom_energies = [&](int nr, bool add) __attribute__((always_inline)) {
            for (int s = w; s < na; s += EC_THREADS / 64) {
                const int q0 = nch > 1 ? 0 : roff[s], q1 = nch > 1 ? nr : roff[s + 1];
                float acc = 0.f;
                for (int k = q0 + lane; k < q1; k += 64) acc += es[k];
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
                if (lane == 0) A.U[a + s] = add ? A.U[a + s] + acc : acc;
            }
        };
        // the lane's channels of an atom's env (or genv) at E + 4 g, and the
        // harmonics of their degrees
        struct Harm {
            float l1[3], l3[7];
        };
        auto harm = [&]() __attribute__((always_inline)) {
            Harm h;
            float Y[16];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const v4f x = *reinterpret_cast<const v4f *>(yr + 4 * k);
#pragma unroll
                for (int m = 0; m < 4; m++) Y[4 * k + m] = x[m];
            }
#pragma unroll
            for (int m = 0; m < 3; m++) h.l1[m] = Y[1 + m];
#pragma unroll
            for (int m = 0; m < 7; m++) h.l3[m] = g < 2 ? (m < 5 ? Y[4 + m] : 0.f) : Y[9 + m];
            return h;
        };
        auto ld4 = [](const float *q) { return *reinterpret_cast<const v4f *>(q); };
        // o[c] = Y . E[c] over the lane's channels
        auto dot_env = [&](const float *E, v4f *o) __attribute__((always_inline)) {
            const Harm h = harm();
            o[0] = ld4(E + 4 * g);
            o[1] = ld4(E + 16 + 4 * g);
            const float *E1 = E + 32 + 16 * g, *E3 = E + 96 + 32 * g;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const v4f x = ld4(E1 + 4 * k), q = ld4(E3 + 8 * k), z = ld4(E3 + 8 * k + 4);
                o[2][k] = h.l1[0] * x[0] + h.l1[1] * x[1] + h.l1[2] * x[2];
                o[3][k] = h.l3[0] * q[0] + h.l3[1] * q[1] + h.l3[2] * q[2] + h.l3[3] * q[3] + h.l3[4] * z[0] +
                          h.l3[5] * z[1] + h.l3[6] * z[2];
            }
        };
        // g1, g3 += sum over the lane's channels of v[c] E[c], v2 and v3 the
        // values of the tiles 2 and 3 (degree 0 has no gradient)
        auto grad_y = [&](const float *E, v4f v2, v4f v3, float *g1, float *g3) __attribute__((always_inline)) {
            const float *E1 = E + 32 + 16 * g, *E3 = E + 96 + 32 * g;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const v4f x = ld4(E1 + 4 * k), q = ld4(E3 + 8 * k), z = ld4(E3 + 8 * k + 4);
#pragma unroll
                for (int m = 0; m < 3; m++) g1[m] = fmaf(v2[k], x[m], g1[m]);
#pragma unroll
                for (int m = 0; m < 4; m++) g3[m] = fmaf(v3[k], q[m], g3[m]);
#pragma unroll
                for (int m = 0; m < 3; m++) g3[4 + m] = fmaf(v3[k], z[m], g3[4 + m]);
            }
        };
        // the two-body MLP, units U0 .. U0 + 7 of a chain of NS stages
        // (D: p1, p2, p3 hold SiLU' of the pre-activations afterwards)
        auto two_body = [&](auto u0, auto ns, auto d_, const char *next, v4f &p1, v4f &p2, v4f *p3, v4f *y)
            __attribute__((always_inline)) {
            constexpr int U0 = decltype(u0)::value, NS = decltype(ns)::value;
            constexpr bool D = decltype(d_)::value;
            // inputs: radial functions 4 g .. 4 g + 3 of 16, one-hots 4 g .. of 16
            v4f xa, xb = z4;
            {
                const v4f e0 = ld4(er), e1 = ld4(er + 4);
                const float s1 = e0[3], c1 = e1[0], bu = A.c0 * e0[0] * e0[1];
                const int zz = __float_as_int(e1[2]), zi = zz & 255, zj = zz >> 8;
                float sk, ck;
                ec_angle(g, s1, c1, sk, ck);
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    xa[k] = bu * sk;
                    const float ns_ = fmaf(sk, c1, ck * s1);
                    ck = fmaf(ck, c1, -sk * s1);
                    sk = ns_;
                    if (4 * g + k == zi || 4 * g + k == A.S + zj) xb[k] = 1.f;
                }
            }
            p1 = cbv(AF_B1, 0);
            ec_layer<U0, NS, 1, 1>(st, next, &p1, [&](auto) { return ec_op<P>(xa, xb); });
            p2 = cbv(AF_B2, 0);
            ec_layer<U0 + 1, NS, 1, 1>(st, next, &p2, [&](auto) { return ec_op<P>(ec_act<P, D>(p1), z4); });
            p3[0] = cbv(AF_B3, 0);
            p3[1] = cbv(AF_B3, 1);
            ec_layer<U0 + 2, NS, 2, 1>(st, next, p3, [&](auto) { return ec_op<P>(ec_act<P, D>(p2), z4); });
#pragma unroll
            for (int t = 0; t < 4; t++) y[t] = cbv(AF_B4, t);
            ec_layer<U0 + 4, NS, 4, 1>(st, next, y, [&](auto) { return ec_op<P>(ec_act<P, D>(p3[0]), ec_act<P, D>(p3[1])); });
        };

        // carried from phase to phase: x0 then dE/dx0, w0 then dE/dw0, we of
        // the tiles 2 and 3, this lane's parts of dE/du and dE/dY
        v4f sA[4] = {z4, z4, z4, z4}, sB[4] = {z4, z4, z4, z4}, we2 = z4, we3 = z4;
        float gu = 0.f, gy1[3] = {0.f, 0.f, 0.f}, gy3[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // one piece: every phase once; several pieces (of one atom, slot 0,
        // genv in the next slot): env over all of them, then genv, then the
        // rest, the earlier phases run again for each piece
        for (int pass = 0; pass < (A.want_G ? 3 : 2); pass++)
            for (int ch = 0; ch < nch; ch++) {
                const int nr = pass == 0 || nch > 1 ? geometry(ch) : 0;
                if (pass == 0 || nch > 1) {   // ---- phase 1
                    const char *next = pass == 0 && nch > 1 ? W1 : W2;
                    v4f p1, p2, p3[2], acc[8];
                    two_body(std::integral_constant<int, 0>{}, std::integral_constant<int, N1>{}, std::false_type{}, next, p1, p2, p3, sA);
                    const float u = er[1];
#pragma unroll
                    for (int t = 0; t < 4; t++) sA[t] *= u;   // x0
#pragma unroll
                    for (int t = 0; t < 8; t++) acc[t] = z4;
                    ec_layer<8, N1, 8, 2>(st, next, acc, [&](auto s) { return ec_op<P>(sA[2 * s], sA[2 * s + 1]); });
#pragma unroll
                    for (int t = 0; t < 4; t++) sB[t] = acc[t];
                    we2 = acc[6];
                    we3 = acc[7];
                    if (pass == 0) {
                        put_tile(acc + 4);
                        __syncthreads();
                        atom_sums(en, nr, ch > 0);
                        __syncthreads();
                    }
                }
                if (pass == 1 || (pass == 2 && nch > 1)) {   // ---- phase 2
                    const char *next = A.want_G && (nch == 1 || pass == 2) ? W3 : W1;
                    const float *E = en + __float_as_int(er[7]) * AF_ENV;
                    v4f PL[4], M[4];
                    {
                        v4f dp[4];
                        dot_env(E, dp);
                        dp[2] *= inv1;
                        dp[3] *= inv3;
#pragma unroll
                        for (int t = 0; t < 4; t++) {
                            PL[t] = cbv(AF_L1, t);
                            dp[t] *= sB[t];   // S
                        }
                        ec_layer<0, N2, 4, 4>(st, next, PL, [&](auto s_) {
                            constexpr int s = decltype(s_)::value;
                            if constexpr (s < 2) return ec_op<P>(sA[2 * s], sA[2 * s + 1]);
                            else return ec_op<P>(dp[2 * s - 4], dp[2 * s - 3]);
                        });
                    }
#pragma unroll
                    for (int t = 0; t < 4; t++) M[t] = cbv(AF_L2, t);
                    ec_layer<16, N2, 4, 2>(st, next, M, [&](auto s) { return ec_op<P>(ec_silu_d<P>(PL[2 * s]), ec_silu_d<P>(PL[2 * s + 1])); });
                    const float u = er[1], gE = er[5];
#pragma unroll
                    for (int t = 0; t < 4; t++) sA[t] = (M[t] * u + sA[t]) * r2;   // x1
                    v4f PO[2] = {cbv(AF_O1, 0), cbv(AF_O1, 1)};
                    ec_layer<24, N2, 2, 2>(st, next, PO, [&](auto s) { return ec_op<P>(sA[2 * s], sA[2 * s + 1]); });
                    float d2 = 0.f;
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        const v4f w2 = cbv(AF_W2, t), h = ec_silu_d<P>(PO[t]);
#pragma unroll
                        for (int k = 0; k < 4; k++) d2 = fmaf(w2[k], h[k], d2);
                        PO[t] *= w2 * (gE * u);
                    }
                    d2 += __shfl_xor(d2, 16, 64);
                    d2 += __shfl_xor(d2, 32, 64);
                    d2 += A.b2;
                    if (g == 0) es[row] = u * d2;
                    gu = g == 0 ? gE * d2 : 0.f;
#pragma unroll
                    for (int t = 0; t < 4; t++) sA[t] = z4;
                    ec_layer<28, N2, 4, 1>(st, next, sA, [&](auto) { return ec_op<P>(PO[0], PO[1]); });
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        sA[t] *= r2;   // dE/dx0 through x1
#pragma unroll
                        for (int k = 0; k < 4; k++) gu = fmaf(sA[t][k], M[t][k], gu);
                        M[t] = z4;
                    }
                    ec_layer<32, N2, 4, 2>(st, next, M, [&](auto s) { return ec_op<P>(sA[2 * s] * u, sA[2 * s + 1] * u); });
#pragma unroll
                    for (int t = 0; t < 4; t++) M[t] *= PL[t];
                    v4f gl[8];   // dE/d[x0 | S]
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        gl[t] = sA[t];
                        gl[4 + t] = z4;
                    }
                    ec_layer<40, N2, 8, 2>(st, next, gl, [&](auto s) { return ec_op<P>(M[2 * s], M[2 * s + 1]); });
                    // dE/dw0 = t Y . env / (2 l + 1); t w0 / (2 l + 1) goes to the tile
                    gl[6] *= inv1;
                    gl[7] *= inv3;
                    v4f dp[4];
                    dot_env(E, dp);
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        sA[t] = gl[t];
                        M[t] = gl[4 + t] * sB[t];
                        sB[t] = gl[4 + t] * dp[t];
                    }
#pragma unroll
                    for (int m = 0; m < 3; m++) gy1[m] = 0.f;
#pragma unroll
                    for (int m = 0; m < 7; m++) gy3[m] = 0.f;
                    grad_y(E, M[2], M[3], gy1, gy3);
                    if (pass == 1) {
                        put_tile(M);
                        __syncthreads();
                        const int nq = nch > 1 ? nr : 0;
                        if (A.want_G) atom_sums(en + (nch > 1 ? AF_ENV : 0), nq, ch > 0);   // genv
                        atom_energies(nq, ch > 0);
                        __syncthreads();
                    }
                }
                if (pass == 2) {   // ---- phase 3
                    if (nch == 1 && an < a1) {   // the next run's first edges, behind this phase
                        const int o = noff - nbase;
                        const EcRun nx = ec_run<AF_SLOTS>(lane, an, a1, o);
                        if (nx.total > 0) {
                            edge_loads(ed, an, nbase, o, nx, 0);
                            have = true;
                        }
                    }
                    const float *E = en + (nch > 1 ? AF_ENV : __float_as_int(er[7]) * AF_ENV);
                    grad_y(E, we2, we3, gy1, gy3);
                    {
                        v4f gwe[4];
                        dot_env(E, gwe);
                        ec_layer<0, N3, 4, 4>(st, W1, sA, [&](auto s_) {
                            constexpr int s = decltype(s_)::value;
                            if constexpr (s < 2) return ec_op<P>(sB[2 * s], sB[2 * s + 1]);
                            else return ec_op<P>(gwe[2 * s - 4], gwe[2 * s - 3]);
                        });
                    }
                    v4f p1, p2, p3[2], y[4];
                    two_body(std::integral_constant<int, 16>{}, std::integral_constant<int, N3>{}, std::true_type{}, W1, p1, p2, p3, y);
                    const v4f e0 = ld4(er);
                    const float ir = e0[0], u = e0[1], du = e0[2], s1 = e0[3], c1 = er[4];
                    // dE/dx0 complete: x0 = u y
#pragma unroll
                    for (int t = 0; t < 4; t++) {
#pragma unroll
                        for (int k = 0; k < 4; k++) gu = fmaf(sA[t][k], y[t][k], gu);
                        sA[t] *= u;
                    }
                    v4f g3[2] = {z4, z4}, g2 = z4, g1 = z4, gb = z4;
                    ec_layer<24, N3, 2, 2>(st, W1, g3, [&](auto s) { return ec_op<P>(sA[2 * s], sA[2 * s + 1]); });
                    ec_layer<28, N3, 1, 1>(st, W1, &g2, [&](auto) { return ec_op<P>(g3[0] * p3[0], g3[1] * p3[1]); });
                    ec_layer<29, N3, 1, 1>(st, W1, &g1, [&](auto) { return ec_op<P>(g2 * p2, z4); });
                    ec_layer<30, N3, 1, 1>(st, W1, &gb, [&](auto) { return ec_op<P>(g1 * p1, z4); });
                    // dE/dr: the envelope, and this lane's radial functions k = 4 g + 1 .. 4 g + 4
                    float dEdr = gu * du;
                    {
                        float sk, ck, kt = (4 * g + 1) * A.th;
                        ec_angle(g, s1, c1, sk, ck);
#pragma unroll
                        for (int k = 0; k < 4; k++) {
                            // d/dr [c0 sin(k th r) / r u] = c0 [(k th cos / r - sin / r^2) u + sin / r u']
                            const float dB = A.c0 * ir * (fmaf(kt, ck, -sk * ir) * u + sk * du);
                            dEdr = fmaf(gb[k], dB, dEdr);
                            const float ns = fmaf(sk, c1, ck * s1);
                            ck = fmaf(ck, c1, -sk * s1);
                            sk = ns;
                            kt += A.th;
                        }
                    }
                    // dE/drhat is linear in dE/dY: each lane takes its own part
                    float gy[16];
                    gy[0] = 0.f;
#pragma unroll
                    for (int m = 0; m < 3; m++) gy[1 + m] = gy1[m];
#pragma unroll
                    for (int m = 0; m < 5; m++) gy[4 + m] = g < 2 ? gy3[m] : 0.f;
#pragma unroll
                    for (int m = 0; m < 7; m++) gy[9 + m] = g < 2 ? 0.f : gy3[m];
                    // rhat from the harmonics of degree 1: sqrt(3) (y, z, x)
                    const float i3 = 0.57735026918962576f, hx = yr[3] * i3, hy = yr[1] * i3, hz = yr[2] * i3;
                    float tx, ty, tz;
                    sh16_grad(hx, hy, hz, gy, tx, ty, tz);
#pragma unroll
                    for (int o = 16; o <= 32; o <<= 1) {
                        dEdr += __shfl_xor(dEdr, o, 64);
                        tx += __shfl_xor(tx, o, 64);
                        ty += __shfl_xor(ty, o, 64);
                        tz += __shfl_xor(tz, o, 64);
                    }
                    // G_e = dE/d(r_i - r_j) = -(dE/dr rhat + (I - rhat rhat^T) dE/drhat / r)
                    const float rd = tx * hx + ty * hy + tz * hz;
                    if (g == 0 && ch * EC_ROWS + row < total)
                        A.G[base + ch * EC_ROWS + row] =
                            make_float4(-(dEdr * hx + (tx - rd * hx) * ir), -(dEdr * hy + (ty - rd * hy) * ir),
                                        -(dEdr * hz + (tz - rd * hz) * ir), 0.f);
                }
            }
        a += na;
        base = nbase;
        off = noff - nbase;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Offsets (floats) of the per-evaluation arrays in the arena.
struct AlArena {
    long H0, u, GL, Y, P[6], A[6], Yo, LIN, WV, PL, M, X1, PO, HO, GU, GWV, GY, GB, ENV, Uat, EP, total;
};

static AlArena al_layout(const AlModel &a, long N, long E) {
    const AlDims &d = a.d;
    AlArena L;
    long o = 0;
    auto take = [&](long cnt) {
        const long r = o;
        o += (cnt + 63) / 64 * 64;
        return r;
    };
    L.H0 = take(E * a.KIN);
    L.u = take(E);
    L.GL = take(E);
    L.Y = take(E * 16);
    for (int q = 0; q < 6; q++) L.P[q] = L.A[q] = 0;
    for (int q = 0; q + 1 < d.n2b; q++) {
        L.P[q] = take(E * d.d2b[q]);
        L.A[q] = take(E * d.d2b[q]);
    }
    L.Yo = take(E * d.D);
    L.LIN = take(E * (d.D + d.NC));
    L.WV = take(E * 2 * d.NC);
    L.PL = take(E * d.LH);
    L.M = take(E * d.D);
    L.X1 = take(E * d.D);
    L.PO = take(E * d.OH);
    L.HO = take(E * d.OH);
    L.GU = take(E);
    L.GWV = take(E * 2 * d.NC);
    L.GY = take(E * 16);
    L.GB = take(E * a.NBP);
    L.ENV = take(N * d.NC * 8);
    L.Uat = take(N + 64);
    L.EP = take(2 * energy_part_doubles(N));   // the energy sums' chunk partials (doubles)
    L.total = o + 4096;
    return L;
}

// the fused path keeps the atoms' energies only
static long al_fused_floats(long N) { return (N + 64 + 63) / 64 * 64 + 2 * energy_part_doubles(N) + 4096; }

size_t allegro_arena_bytes(const mlp_model *m, long n_atoms, long n_edges, bool counted) {
    if (m->al->fused && !counted) return (size_t)al_fused_floats(n_atoms) * sizeof(float);
    return (size_t)al_layout(*m->al, n_atoms, n_edges).total * sizeof(float);
}

static int check_dims(const AlDims &d) {
    if (d.S < 1 || d.S > 64) return fail(-1, "allegro: n_species out of range");
    if (d.NB < 1 || d.NB > 16) return fail(-1, "allegro: n_basis must be 1..16");
    if (d.p < 1 || d.p > 8) return fail(-1, "allegro: envelope_p must be 1..8");
    if (d.n2b < 1 || d.n2b > 6) return fail(-1, "allegro: mlp_2b needs 1..6 widths");
    if (d.lmax < 0 || d.lmax > 3) return fail(-1, "allegro: l_max must be 0..3");
    if (d.NC < 1 || d.NC > 64) return fail(-1, "allegro: the channels must total 1..64");
    for (int q = 0; q < d.n2b; q++)
        if (d.d2b[q] < 4 || d.d2b[q] % 4 || d.d2b[q] > 256) return fail(-1, "allegro: two-body widths must be multiples of 4 up to 256");
    if (d.D > 64) return fail(-1, "allegro: the latent width must be at most 64");
    if (d.LH < 4 || d.LH % 4 || d.LH > 128 || d.OH < 4 || d.OH % 4 || d.OH > 128)
        return fail(-1, "allegro: latent_hidden and out_hidden must be multiples of 4 up to 128");
    if (d.NC % 4) return fail(-1, "allegro: the channel total must be a multiple of 4");
    if (!(d.rc > 0.f) || !(d.nu > 0.f)) return fail(-1, "allegro: r_c and env_scale must be positive");
    return 0;
}

// The weights and constants of k_al_atoms, where the model's widths fit it:
// four two-body layers, the channel layout of the paper's setting (the
// kernel's lanes know their channels' degrees), every width within the
// padded one the chain is built for.  Other models take the kernels above.
static int al_pack_chain(AlModel *a, int P, const float *w, const std::vector<size_t> &oW, size_t oWv, size_t oWe, size_t oL1, size_t oL2, size_t oO1, const std::vector<size_t> &ob,
                         size_t oLb1, size_t oLb2, size_t oOb1, size_t oOw2) {
    const AlDims &d = a->d;
    const int *h = d.d2b, D = d.D, NC = d.NC, LH = d.LH, OH = d.OH, NB = d.NB, K0 = 2 * d.S + NB;   // stored columns: one-hots, then the radial functions
    if (!(d.n2b == 4 && h[0] <= 16 && h[1] <= 16 && h[2] <= 32 && D <= 64 && LH <= 64 && OH <= 32 &&
          NB <= 16 && d.S <= 8 && d.lmax == 3 && d.ch[0] == 32 && d.ch[1] == 16 && d.ch[2] == 8 && d.ch[3] == 8))
        return 0;
    // element (o, i) of a row-major matrix of R rows and C columns, zero outside
    auto at = [](const float *M, int R, int C, int ld) {
        return [=](int o, int i) { return o < R && i < C ? M[(size_t)o * ld + i] : 0.f; };
    };
    auto tr = [](const float *M, int R, int C, int ld) {
        return [=](int o, int i) { return i < R && o < C ? M[(size_t)i * ld + o] : 0.f; };
    };
    const float *Wv = w + oWv, *We = w + oWe, *L1 = w + oL1, *L2 = w + oL2, *O1 = w + oO1;
    EcPack k(P, 24 + 56 + 32);
    // [x0 | S] and [w0 | we] have 64 columns each in the chain
    auto ve = [&](int o, int i) { return i < D ? (o < 64 ? Wv[(size_t)o * D + i] : We[(size_t)(o - 64) * D + i]) : 0.f; };
    auto two_body = [&]() {
        // inputs: 16 radial functions (zero weights past NB), 16 one-hot columns
        k.layer(1, 1, [&](int o, int i) {
            const int c = i < 16 ? (i < NB ? 2 * d.S + i : -1) : (i - 16 < 2 * d.S ? i - 16 : -1);
            return o < h[0] && c >= 0 ? w[oW[0] + (size_t)o * K0 + c] : 0.f;
        });
        k.layer(1, 1, at(w + oW[1], h[1], h[0], h[0]));
        k.layer(2, 1, at(w + oW[2], h[2], h[1], h[1]));
        k.layer(4, 1, at(w + oW[3], D, h[2], h[2]));
    };
    two_body();
    k.layer(8, 2, ve);
    k.align();
    k.layer(4, 4, [&](int o, int i) {
        const int c = i < 64 ? (i < D ? i : -1) : D + i - 64;
        return o < LH && c >= 0 ? L1[(size_t)o * (D + NC) + c] : 0.f;
    });
    k.layer(4, 2, at(L2, D, LH, LH));
    k.layer(2, 2, at(O1, OH, D, D));
    k.layer(4, 1, tr(O1, OH, D, D));
    k.layer(4, 2, tr(L2, D, LH, LH));
    k.layer(8, 2, [&](int o, int i) {
        const int c = o < 64 ? (o < D ? o : -1) : D + o - 64;
        return i < LH && c >= 0 ? L1[(size_t)i * (D + NC) + c] : 0.f;
    });
    k.align();
    k.layer(4, 4, [&](int o, int i) { return ve(i, o); });
    two_body();
    k.layer(2, 2, tr(w + oW[3], D, h[2], h[2]));
    k.layer(1, 1, tr(w + oW[2], h[2], h[1], h[1]));
    k.layer(1, 1, tr(w + oW[1], h[1], h[0], h[0]));
    k.layer(1, 1, tr(w + oW[0] + 2 * d.S, h[0], NB, K0));
    k.align();
    if (k.units() != 24 + 56 + 32) return fail(-5, "allegro: chain packing");
    const size_t nb = k.bytes();
    std::vector<char> host(nb + sizeof(float) * AF_VEC, 0);
    std::memcpy(host.data(), k.data(), nb);
    float *vec = reinterpret_cast<float *>(host.data() + nb);
    auto put = [&](int o, size_t src, int cnt) { std::copy(w + src, w + src + cnt, vec + o); };
    put(AF_B1, ob[0], h[0]);
    put(AF_B2, ob[1], h[1]);
    put(AF_B3, ob[2], h[2]);
    put(AF_B4, ob[3], D);
    put(AF_L1, oLb1, LH);
    put(AF_L2, oLb2, D);
    put(AF_O1, oOb1, OH);
    put(AF_W2, oOw2, OH);
    if (hipMalloc(&a->chain, host.size()) != hipSuccess) {
        (void)hipGetLastError();
        return fail(-2, "allegro: weight allocation failed");
    }
    if (hipMemcpy(a->chain, host.data(), host.size(), hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(a->chain);
        a->chain = nullptr;
        return fail(-5, "allegro: weight copy failed");
    }
    a->chain_vec = reinterpret_cast<const float *>(a->chain + nb);
    a->fused = true;
    return 0;
}

int allegro_create(mlp_model *m, const AlDims &d, const float *w, size_t n_weights) {
    if (int rc = check_dims(d)) return rc;
    const int S = d.S, NB = d.NB, NC = d.NC, D = d.D, LH = d.LH, OH = d.OH;
    // storage order (matrices [out][in]): 2b_W1 b1 .. 2b_Wn bn, Wv, We,
    // lat_W1 lat_b1 lat_W2 lat_b2, out_W1 out_b1 out_w2 out_b2
    size_t off = 0;
    std::vector<size_t> oW(d.n2b), ob(d.n2b);
    int prev = 2 * S + NB;
    for (int q = 0; q < d.n2b; q++) {
        oW[q] = off;
        off += (size_t)d.d2b[q] * prev;
        ob[q] = off;
        off += d.d2b[q];
        prev = d.d2b[q];
    }
    const size_t oWv = off;
    off += (size_t)NC * D;
    const size_t oWe = off;
    off += (size_t)NC * D;
    const size_t oL1 = off;
    off += (size_t)LH * (D + NC);
    const size_t oLb1 = off;
    off += LH;
    const size_t oL2 = off;
    off += (size_t)D * LH;
    const size_t oLb2 = off;
    off += D;
    const size_t oO1 = off;
    off += (size_t)OH * D;
    const size_t oOb1 = off;
    off += OH;
    const size_t oOw2 = off;
    off += OH;
    const size_t oOb2 = off;
    off += 1;
    if (off != n_weights)
        return fail(-1, "allegro: weight count " + std::to_string(n_weights) + " does not match the header (" +
                            std::to_string(off) + ")");
    AlModel *a = new AlModel();
    a->d = d;
    a->KIN = up4(NB + 2 * S);
    a->NBP = up4(NB);
    a->out_b2_host = w[oOb2];
    if (int rc = al_pack_chain(a, node_operands(m->precision), w, oW, oWv, oWe, oL1, oL2, oO1, ob, oLb1, oLb2, oOb1, oOw2)) {
        delete a;
        return rc;
    }
    if (a->fused) {   // nothing else is read
        m->al = a;
        return 0;
    }
    // host-side matrices in the orientations the GEMMs take: the first
    // two-body matrix with its columns in the internal input order
    // [B | onehot_i | onehot_j | 0], its radial block alone, and [Wv; We]
    std::vector<float> W1p((size_t)d.d2b[0] * a->KIN, 0.f), W1B((size_t)d.d2b[0] * NB);
    for (int o = 0; o < d.d2b[0]; o++) {
        const float *row = w + oW[0] + (size_t)o * (2 * S + NB);
        for (int k = 0; k < NB; k++) W1p[(size_t)o * a->KIN + k] = W1B[(size_t)o * NB + k] = row[2 * S + k];
        for (int z = 0; z < 2 * S; z++) W1p[(size_t)o * a->KIN + NB + z] = row[z];
    }
    // device copies: the permuted W1, W1's radial block, and every block of w
    const size_t nW = n_weights;
    std::vector<float> host(nW + W1p.size() + W1B.size());
    std::copy(w, w + nW, host.begin());
    std::copy(W1p.begin(), W1p.end(), host.begin() + nW);
    std::copy(W1B.begin(), W1B.end(), host.begin() + nW + W1p.size());
    float *dev = nullptr;
    if (hipMalloc(&dev, sizeof(float) * host.size()) != hipSuccess) {
        (void)hipGetLastError();
        delete a;
        return fail(-2, "allegro: weight allocation failed");
    }
    if (hipMemcpy(dev, host.data(), sizeof(float) * host.size(), hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(dev);
        delete a;
        return fail(-5, "allegro: weight copy failed");
    }
    a->vec = dev;
    for (int q = 0; q < d.n2b; q++) a->b2b[q] = dev + ob[q];
    a->lat_b1 = dev + oLb1;
    a->lat_b2 = dev + oLb2;
    a->out_b1 = dev + oOb1;
    a->out_w2 = dev + oOw2;
    a->out_b2 = dev + oOb2;
    const float *dW1p = dev + nW, *dW1B = dev + nW + W1p.size();
    struct Item {
        const float *W;
        int R, C;
        bool tr;
        PackedW *dst;
    };
    std::vector<Item> items;
    items.push_back({dW1p, d.d2b[0], a->KIN, false, &a->f2b[0]});
    items.push_back({dW1B, d.d2b[0], NB, true, &a->a2b[0]});
    prev = d.d2b[0];
    for (int q = 1; q < d.n2b; q++) {
        items.push_back({dev + oW[q], d.d2b[q], prev, false, &a->f2b[q]});
        items.push_back({dev + oW[q], d.d2b[q], prev, true, &a->a2b[q]});
        prev = d.d2b[q];
    }
    // Wv and We are adjacent: [Wv; We] is one 2NC x D matrix
    items.push_back({dev + oWv, 2 * NC, D, false, &a->fVE});
    items.push_back({dev + oWv, 2 * NC, D, true, &a->aVE});
    items.push_back({dev + oL1, LH, D + NC, false, &a->fL1});
    items.push_back({dev + oL1, LH, D + NC, true, &a->aL1});
    items.push_back({dev + oL2, D, LH, false, &a->fL2});
    items.push_back({dev + oL2, D, LH, true, &a->aL2});
    items.push_back({dev + oO1, OH, D, false, &a->fO1});
    items.push_back({dev + oO1, OH, D, true, &a->aO1});
    size_t pk = 0;
    for (const Item &it : items) pk += packed_bytes(it.R, it.C, it.tr);
    int rc = hipMalloc(&a->pk_dev, pk) == hipSuccess ? 0 : -2;
    for (size_t q = 0, o = 0; rc == 0 && q < items.size(); q++) {
        if (pack_weight(nullptr, items[q].W, items[q].R, items[q].C, items[q].tr, (char *)a->pk_dev + o, items[q].dst))
            rc = -5;
        o += packed_bytes(items[q].R, items[q].C, items[q].tr);
    }
    if (rc == 0 && hipDeviceSynchronize() != hipSuccess) rc = -5;
    if (rc) {
        (void)hipGetLastError();
        if (a->pk_dev) hipFree(a->pk_dev);
        hipFree(dev);
        delete a;
        return fail(rc, "allegro: weight packing failed");
    }
    m->al = a;
    return 0;
}

void allegro_destroy(mlp_model *m) {
    if (!m || !m->al) return;
    if (m->al->pk_dev) hipFree(m->al->pk_dev);
    if (m->al->vec) hipFree(m->al->vec);
    if (m->al->chain) hipFree(m->al->chain);
    delete m->al;
    m->al = nullptr;
}

// A GEMM over the edge rows: grid sized for the skin graph's edges, rows
// bounded by the pruned count on the device (Mc)
static int gm(hipStream_t s, int P, int epi, const float *A, int lda, const PackedW &B, float *C, int ldc, long M,
              const int *Mc, const float *bias = nullptr, float *C2 = nullptr, int ldc2 = 0, const float *R = nullptr,
              int ldr = 0) {
    if (M <= 0) return 0;
    ProfScope ps(PK_GEMM, s);
    return node_gemm(s, P, epi, A, lda, B, C, ldc, (int)M, bias, C2, ldc2, R, ldr, Mc) ? fail(-5, "allegro GEMM failed")
                                                                                       : 0;
}

int allegro_evaluate(mlp_model *m, mlp_nbr *g, hipStream_t s, double *energy, float *forces_user,
                     float *atom_energy_user, int n_seg, const int *seg_dev) {
    const AlModel &a = *m->al;
    const AlDims &d = a.d;
    const int n = g->n_atoms, P = node_operands(m->precision);
    // rows of every edge array: the skin graph's edge count bounds the pruned one
    const long E = g->n_edges_skin;
    int rc;
    if ((rc = g->act.ensure(allegro_arena_bytes(m, n, E), 1.2, &g->n_grows))) return rc;
    if ((rc = g->G.ensure(sizeof(float4) * (size_t)E + 64, 1.2, &g->n_grows))) return rc;
    float *base = g->act.as<float>();
    if (a.fused) {
        AlAtomsArgs k{};
        k.rowc = g->rowc.as<int>();
        k.colc = g->colc.as<int>();
        k.zsp = g->species.as<int>();
        k.perm = g->perm.as<int>();
        k.geom = g->geom.as<float4>();
        k.n = n;
        k.n_local = g->n_local;
        k.S = d.S;
        k.p = d.p;
        k.irc = 1.0f / d.rc;
        k.c0 = std::sqrt(2.0f / d.rc);
        ec_phase(d.rc, k.th, k.thl);
        k.want_G = forces_user != nullptr;
        k.rc = d.rc;
        k.nu = d.nu;
        k.b2 = a.out_b2_host;
        k.W = a.chain;
        k.vec = a.chain_vec;
        k.U = base;
        k.G = g->G.as<float4>();
        k.per_wg = ec_per_wg(n, E, d.rc, g->skin, AF_SLOTS);
        const int nb = nblk(n, k.per_wg);
        {
            ProfScope ps(PK_GEMM, s);
            if (P == 0) k_al_atoms<0><<<nb, EC_THREADS, 0, s>>>(k);
            else if (P == 1) k_al_atoms<1><<<nb, EC_THREADS, 0, s>>>(k);
            else k_al_atoms<2><<<nb, EC_THREADS, 0, s>>>(k);
        }
        HIP_TRY(hipGetLastError());
        if ((rc = launch_energy(s, k.U, k.perm, n, g->n_local, energy, atom_energy_user, n_seg, seg_dev,
                                reinterpret_cast<double *>(base + (n + 64 + 63) / 64 * 64))))
            return rc;
        return forces_user ? launch_forces(s, k.rowc, g->revc.as<int>(), k.G, k.perm, n, forces_user) : 0;
    }
    const AlArena L = al_layout(a, n, E);
    float *H0 = base + L.H0, *u = base + L.u, *GLc = base + L.GL, *Y = base + L.Y, *Yo = base + L.Yo, *LIN = base + L.LIN,
          *WV = base + L.WV, *PL = base + L.PL, *M = base + L.M, *X1 = base + L.X1, *PO = base + L.PO,
          *HO = base + L.HO, *GU = base + L.GU, *GWV = base + L.GWV, *GY = base + L.GY, *GB = base + L.GB,
          *ENV = base + L.ENV, *Uat = base + L.Uat;
    const int *rowc = g->rowc.as<int>(), *colc = g->colc.as<int>(), *perm = g->perm.as<int>();
    const float4 *geom = g->geom.as<float4>();
    const int ldl = d.D + d.NC, D = d.D;
    // edge kernels and GEMMs are sized for E rows and stop at the pruned
    // count, which lives on the device (rowc[n])
    const long ne = E;
    const int *cnt = rowc + n;

    // forward
    k_al_edge_in<<<nblk(n, 4), 256, 0, s>>>(rowc, colc, geom, g->species.as<int>(), perm, n, g->n_local, d.S, d.NB,
                                            d.p, a.KIN, d.rc, H0, u, Y, GLc);
    const float *in = H0;
    int ldin = a.KIN;
    for (int q = 0; q + 1 < d.n2b; q++) {
        float *Pq = base + L.P[q], *Aq = base + L.A[q];
        if ((rc = gm(s, P, GE_BIAS_SILU, in, ldin, a.f2b[q], Pq, d.d2b[q], ne, cnt, a.b2b[q], Aq, d.d2b[q]))) return rc;
        in = Aq;
        ldin = d.d2b[q];
    }
    if ((rc = gm(s, P, GE_BIAS, in, ldin, a.f2b[d.n2b - 1], Yo, D, ne, cnt, a.b2b[d.n2b - 1]))) return rc;
    k_al_scale_rows<<<nblk(ne * (D / 4), 256), 256, 0, s>>>(Yo, D, u, cnt, D, LIN, ldl);
    if ((rc = gm(s, P, GE_STORE, LIN, ldl, a.fVE, WV, 2 * d.NC, ne, cnt))) return rc;
    k_al_tp<<<nblk(n, 4), 256, 0, s>>>(rowc, n, d, Y, WV, ENV, LIN);
    {
        GemmChain c;
        c.e1 = GE_BIAS_SILU;
        c.e2 = GE_BIAS;
        c.A = LIN;
        c.lda = ldl;
        c.M = (int)ne;
        c.B1 = &a.fL1;
        c.C1 = PL;
        c.ldc1 = d.LH;
        c.bias1 = a.lat_b1;
        c.B2 = &a.fL2;
        c.C2 = M;
        c.ldc2 = D;
        c.bias2 = a.lat_b2;
        c.Mc = cnt;
        ProfScope ps(PK_GEMM, s);
        if (node_gemm_chain(s, P, c)) return fail(-5, "allegro latent GEMM failed");
    }
    k_al_x1<<<nblk(ne * (D / 4), 256), 256, 0, s>>>(LIN, ldl, u, M, cnt, D, X1);
    if ((rc = gm(s, P, GE_BIAS_SILU, X1, D, a.fO1, PO, d.OH, ne, cnt, a.out_b1, HO, d.OH))) return rc;
    k_al_energy<<<nblk(n, 4), 256, 0, s>>>(rowc, n, d.OH, HO, u, a.out_w2, a.out_b2_host, Uat);
    if ((rc = launch_energy(s, Uat, perm, n, g->n_local, energy, atom_energy_user, n_seg, seg_dev,
                            reinterpret_cast<double *>(base + L.EP))))
        return rc;
    if (!forces_user) return 0;

    // adjoint
    k_al_out_bwd<<<nblk(ne * 8, 256), 256, 0, s>>>(cnt, d.OH, PO, HO, u, GLc, a.out_w2, a.out_b2_host, GU);
    if ((rc = gm(s, P, GE_STORE, HO, d.OH, a.aO1, X1, D, ne, cnt))) return rc;
    k_al_x1_bwd<<<nblk(ne * 16, 256), 256, 0, s>>>(cnt, D, u, X1, M, GU);
    {
        GemmChain c;
        c.e1 = GE_DSILU;
        c.e2 = GE_STORE;
        c.A = M;
        c.lda = D;
        c.M = (int)ne;
        c.B1 = &a.aL2;
        c.R1 = PL;
        c.ldr1 = d.LH;
        c.B2 = &a.aL1;
        c.C2 = LIN;
        c.ldc2 = ldl;
        c.Mc = cnt;
        ProfScope ps(PK_GEMM, s);
        if (node_gemm_chain(s, P, c)) return fail(-5, "allegro latent adjoint GEMM failed");
    }
    const bool std_layout = d.lmax == 3 && d.ch[0] == 32 && d.ch[1] == 16 && d.ch[2] == 8 && d.ch[3] == 8;
    if (std_layout) k_al_tp_bwd<true><<<nblk(n, 4), 256, 0, s>>>(rowc, n, d, Y, WV, ENV, LIN, X1, GWV, GY);
    else k_al_tp_bwd<false><<<nblk(n, 4), 256, 0, s>>>(rowc, n, d, Y, WV, ENV, LIN, X1, GWV, GY);
    if ((rc = gm(s, P, GE_ADD, GWV, 2 * d.NC, a.aVE, X1, D, ne, cnt, nullptr, nullptr, 0, X1, D))) return rc;
    k_al_x0_bwd<<<nblk(ne * 16, 256), 256, 0, s>>>(cnt, D, u, X1, Yo, GU);
    // the two-body MLP in reverse: dE/dy in Yo, pre-activation gradients over the activations
    const float *gin = Yo;
    int ldg = D;
    for (int q = d.n2b - 1; q >= 1; q--) {
        float *Aq = base + L.A[q - 1], *Pq = base + L.P[q - 1];
        if ((rc = gm(s, P, GE_DSILU, gin, ldg, a.a2b[q], Aq, d.d2b[q - 1], ne, cnt, nullptr, nullptr, 0, Pq, d.d2b[q - 1])))
            return rc;
        gin = Aq;
        ldg = d.d2b[q - 1];
    }
    if ((rc = gm(s, P, GE_STORE, gin, ldg, a.a2b[0], GB, a.NBP, ne, cnt))) return rc;
    k_al_geom_bwd<<<(int)std::max<long>(1, std::min<long>(nblk(E, 256), 16384)), 256, 0, s>>>(
        rowc, n, geom, d.NB, a.NBP, d.p, d.rc, GB, GU, GY, g->G.as<float4>());
    HIP_TRY(hipGetLastError());
    return launch_forces(s, rowc, g->revc.as<int>(), g->G.as<float4>(), perm, n, forces_user);
}

}  // namespace mlp
