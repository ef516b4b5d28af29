// PaiNN energy and forces on the pruned neighbour graph.
//
// Per layer (Methods, "Graph Neural Networks": messages aggregated from the
// neighbours, then a node update; "Chosen Architectures": PaiNN), with the
// layer equations of the PaiNN paper the method cites:
//   phi_j = W2 silu(W1 s_j + b1) + b2
//   w_ij  = (A e(r_ij) + c) fc(r_ij),  e_k = sin(k pi r / rc) / r,
//           fc = (cos(pi r / rc) + 1) / 2
//   s_i  += sum_j (phi_j o w_ij)_s
//   v_i  += sum_j v_j o (phi_j o w_ij)_vv + rhat_ij (x) (phi_j o w_ij)_vs
//   Uv = U v, Vv = V v, n = sqrt(sum_d Vv_d^2 + eps)
//   a = W4 silu(W3 [s; n] + b3) + b4
//   v += a_vv o Uv,  s += a_sv o <Uv, Vv> + a_ss
// Readout U_i = w6 . silu(W5 s_i + b5) + b6; E = sum over local atoms in
// FP64 (Eq. 1).  Forces (Eq. 2) come from a hand-written adjoint: the node
// kernels' (node.hip), and per edge the geometric gradient
// G_e = dE/d(r_src - r_dst) with radial filters recomputed (never stored);
// F_k = sum_{e into k} G_e - sum_{e out of k} G_e, assembled by gathering
// through the reverse-edge index, so no floating-point atomics are used and
// results are bitwise reproducible.
#include "internal.h"
#include "gemm.h"
#include "msg.h"
#include "node.h"

#include <cmath>

namespace mlp {

static inline int nblk(long n, int t) { return (int)((n + t - 1) / t); }

// ---------------------------------------------------------------------------
// The layers' node work runs in node.hip, the factorised first layer's
// products in gemm.hip.
// ---------------------------------------------------------------------------
static int gemm(hipStream_t s, int prec, const float *A, int lda, const PackedW &B, float *C, int ldc, int M) {
    if (M <= 0) return 0;
    ProfScope ps(PK_GEMM, s);
    return node_gemm(s, prec, GE_STORE, A, lda, B, C, ldc, M);
}
// Two independent products, the second over three times the rows (s and v of
// the first layer), in one launch where they fit (on 192 atoms a launch is the
// product's time).
static int gemm_sv(hipStream_t s, int prec, const float *A0, int lda0, const PackedW &B0, float *C0, int ldc0,
                    const float *A1, int lda1, const PackedW &B1, float *C1, int ldc1, int M) {
    GemmBatch b;
    b.n = 2;
    b.A[0] = A0, b.lda[0] = lda0, b.B[0] = B0, b.C[0] = C0, b.ldc[0] = ldc0, b.M[0] = M;
    b.A[1] = A1, b.lda[1] = lda1, b.B[1] = B1, b.C[1] = C1, b.ldc[1] = ldc1, b.M[1] = 3 * M;
    {
        ProfScope ps(PK_GEMM, s);
        const int rc = node_gemm_batch(s, prec, b);
        if (rc != -1) return rc;
    }
    if (int rc = gemm(s, prec, A0, lda0, B0, C0, ldc0, M)) return rc;
    return gemm(s, prec, A1, lda1, B1, C1, ldc1, 3 * M);
}

// ---------------------------------------------------------------------------
// Energy, forces and small kernels
// ---------------------------------------------------------------------------

// p[0 .. count) = 0.
__global__ void k_fill_zero(float *__restrict__ p, long count) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) p[t] = 0.f;
}

static void fill_zero(hipStream_t s, float *p, long count) {
    if (count > 0) k_fill_zero<<<nblk(count, 256), 256, 0, s>>>(p, count);
}

// Sum over the 16 lanes of a DPP row.
__device__ __forceinline__ float row16_sum(float x) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, false));   // row_ror:8
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, false));   // row_ror:4
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));    // quad [2,3,0,1]
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));    // quad [1,0,3,2]
    return x;
}

constexpr int ERED = 512;      // threads per block of the energy sums
constexpr int ECH = 16384;     // rows per chunk of a segment

// E_b = sum of U_i over the local atoms of segment b (internal rows
// [seg[b], seg[b+1]), or [0, n) without segments), in FP64 with a fixed
// order that depends on the segment alone: the segment is cut into chunks of
// ECH rows from its first row; block (b, c) sums chunk c (strided partial
// sums, a butterfly within each wave, then the wave totals in order) into
// part[o_b + c], o_b = b + seg[b] / ECH (disjoint: segment b has
// ceil(len / ECH) <= 1 + len / ECH chunks); k_energy_total adds the chunk
// sums of each segment in order.  A segment's energy is therefore the same
// whether it is evaluated alone or packed into a batch.
__global__ void __launch_bounds__(ERED) k_energy_chunk(const float *__restrict__ U, const int *__restrict__ perm,
                                                       const int *__restrict__ seg, int n, int n_local,
                                                       double *__restrict__ part) {
    __shared__ double sh[ERED / 64];
    const int b = blockIdx.x, c = blockIdx.y;
    const int a = seg ? seg[b] : 0, e = seg ? seg[b + 1] : n;
    const int ca = a + c * ECH;
    if (ca >= e && !(c == 0 && a == e)) return;   // past the segment (an empty one keeps chunk 0)
    const int ce = min(ca + ECH, e);
    // eight interleaved partial sums per thread; the row's energy and its
    // local flag are loaded together, so eight pairs of loads are in flight
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i0 = ca + threadIdx.x; i0 < ce; i0 += 8 * ERED) {
        float u[8];
        int pm[8];
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int i = i0 + q * ERED;
            u[q] = i < ce ? U[i] : 0.f;
            pm[q] = i < ce ? perm[i] : n_local;
        }
#pragma unroll
        for (int q = 0; q < 8; q++)
            if (pm[q] < n_local) acc[q] += (double)u[q];
    }
    double x = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    // butterfly within each wave, then the waves' totals in wave order
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < ERED / 64; w++) t += sh[w];
        part[b + a / ECH + c] = t;
    }
}
__global__ void k_energy_total(const int *__restrict__ seg, int n, int n_seg, const double *__restrict__ part,
                               double *__restrict__ E) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_seg) return;
    const int a = seg ? seg[b] : 0, e = seg ? seg[b + 1] : n;
    const int nc = e > a ? (e - a + ECH - 1) / ECH : 1;
    const double *p = part + b + a / ECH;
    double t = 0.0;
    for (int c = 0; c < nc; c++) t += p[c];
    E[b] = t;
}

// F_k = sum over in-edges e of (G at rev(e)) - (G at e), scattered to the
// caller's atom order (SoA).
// Sixteen lanes per atom (one DPP row): lane q takes the atom's edges
// q, q + 16, ..., and the row sum gives the force.
__global__ void k_forces(const int *__restrict__ rowc, const int *__restrict__ revc,
                         const float4 *__restrict__ Gout, const int *__restrict__ perm, int n,
                         float *__restrict__ F) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int k = (int)(t >> 4), q = (int)(t & 15);
    float fx = 0.f, fy = 0.f, fz = 0.f;
    if (k < n) {
        for (int e = rowc[k] + q; e < rowc[k + 1]; e += 16) {
            const int re = revc[e];
            if (re < 0) continue;  // cannot happen for a symmetric graph; never index with it
            const float4 a = Gout[re], b = Gout[e];
            fx += a.x - b.x;
            fy += a.y - b.y;
            fz += a.z - b.z;
        }
    }
    // every lane of the wave takes part in the row sums (n need not fill the grid)
    fx = row16_sum(fx);
    fy = row16_sum(fy);
    fz = row16_sum(fz);
    if (k < n && q == 0) {
        const int u = perm[k];
        F[u] = fx;
        F[(long)n + u] = fy;
        F[2 * (long)n + u] = fz;
    }
}

__global__ void k_scatter_energy(const float *__restrict__ U, const int *__restrict__ perm, int n,
                                 float *__restrict__ out) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[perm[k]] = U[k];
}

// ---------------------------------------------------------------------------
// Host orchestration
// ---------------------------------------------------------------------------
struct Act {
    // s, v and phi of a layer's input, s1 (rows of 2F) and v1 after its message pass
    float *s[MLP_MAX_LAYERS], *v[MLP_MAX_LAYERS], *phi[MLP_MAX_LAYERS], *sn[MLP_MAX_LAYERS], *v1[MLP_MAX_LAYERS];
    float *gv, *gs1, *gv1, *gphi, *U;
    float *work;   // forward: v * phi_vv of the current layer; the first layer's sums and their gradients
    double *epart;
    int *queue;   // the message launches' atom counters, MSG_QUEUE_INTS per launch
};
constexpr long QUEUE_INTS = 2L * MLP_MAX_LAYERS * MSG_QUEUE_INTS;

static size_t act_floats(long N, int F, int T) {
    // per layer s 1, v 3, phi 3, s1 2 (rows of 2F), v1 3; adjoint gv 3, gs1 1, gv1 3, gphi 3, work 6
    return (size_t)((long)N * F * (12 * T + 16) + N + 64 * (5 * T + 32) + 4096 + QUEUE_INTS + 2 * energy_part_doubles(N));
}

static void carve(float *base, long N, int F, int T, Act &A) {
    float *p = base;
    auto take = [&](long cnt) {
        float *r = p;
        p += (cnt + 63) & ~63L;
        return r;
    };
    const long NF = N * F;
    for (int t = 0; t < T; t++) {
        A.s[t] = take(NF);
        A.v[t] = take(3 * NF);
        A.phi[t] = take(3 * NF);
        A.sn[t] = take(2 * NF);
        A.v1[t] = take(3 * NF);
    }
    A.gv = take(3 * NF);
    A.gs1 = take(NF);
    A.gv1 = take(3 * NF);
    A.gphi = take(3 * NF);
    A.work = take(6 * NF);
    A.U = take(N + 64);
    A.epart = reinterpret_cast<double *>(take(2 * energy_part_doubles(N)));
    A.queue = reinterpret_cast<int *>(take(QUEUE_INTS));
}

static MsgArgs msg_args(mlp_nbr *g, mlp_model *m, const LayerW &L, int hop_max) {
    MsgArgs a = {};
    a.rowc = g->rowc.as<int>();
    a.colc = g->colc.as<int>();
    a.geom = g->geom.as<float4>();
    a.n = g->n_atoms;
    a.A = L.A;
    a.c = L.c;
    a.rc = m->rc;
    a.hop = g->hop.as<int8_t>();
    a.hop_max = hop_max;
    a.S = g->Gs.as<float4>();
    a.s_stride = g->n_edges_skin;
    a.species = g->species.as<int>();
    return a;
}

struct L0Layout {
    int ldp, ldr, ldq;
};
static L0Layout l0_layout(int F, int K, int S) {
    const int CS = S * l0_block(K);
    L0Layout l;
    l.ldp = (CS + S + 3) / 4 * 4;
    l.ldr = CS;
    l.ldq = CS;
    (void)F;
    return l;
}

static L0Args l0_args(mlp_nbr *g, mlp_model *m, int hop_max) {
    L0Args a = {};
    a.rowc = g->rowc.as<int>();
    a.colc = g->colc.as<int>();
    a.revc = g->revc.as<int>();
    a.geom = g->geom.as<float4>();
    a.n = g->n_atoms;
    a.rc = m->rc;
    a.hop = g->hop.as<int8_t>();
    a.hop_max = hop_max;
    a.species = g->species.as<int>();
    return a;
}

int first_layer_table(mlp_model *m, hipStream_t s, float *tmp) {
    const int F = m->F, S = m->S;
    const int P = node_operands(m->precision);
    const LayerW L = m->layer(0);
    // the same GEMMs as the later layers' node MLPs, on the S embedding rows
    if (int rc = node_gemm(s, P, GE_BIAS_SILU, m->at(m->off_emb), F, m->pk_phi0[0], tmp, F, S, L.b1, tmp + (long)S * F, F))
        return rc;
    return node_gemm(s, P, GE_BIAS, tmp + (long)S * F, F, m->pk_phi0[1], m->phi0_dev, 3 * F, S, L.b2);
}

// Species-scaled first-layer filter weights (CS = S SB columns of basis
// slots, one block of SB = l0_block(K) per species, zero past slot K):
// Wfs[f][z SB + k] = phi_s(z)_f A'_s[f][k] followed by the embedding columns
// Wfs[f][CS + z] = emb[z][f]; Wbs the same without the embedding;
// Wv[f][z SB + k] = phi_vs(z)_f A'_vs[f][k]; A'[.][0] = c.
__global__ void k_l0_weights(const float *__restrict__ A, const float *__restrict__ c,
                             const float *__restrict__ phi0, const float *__restrict__ emb, int F, int K, int S,
                             float *__restrict__ Wfs, float *__restrict__ Wbs, float *__restrict__ Wv) {
    const int SB = l0_block(K), CS = S * SB;
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < (long)F * CS) {
        const int f = (int)(idx / CS), col = (int)(idx % CS), z = col / SB, k = col % SB;
        float ws = 0.f, wv = 0.f;
        if (k <= K) {
            const float as = k == 0 ? c[F + f] : A[(long)(F + f) * K + k - 1];
            const float av = k == 0 ? c[2 * F + f] : A[(long)(2 * F + f) * K + k - 1];
            ws = phi0[(long)z * 3 * F + F + f] * as;
            wv = phi0[(long)z * 3 * F + 2 * F + f] * av;
        }
        Wfs[(long)f * (CS + S) + col] = ws;
        Wbs[(long)f * CS + col] = ws;
        Wv[(long)f * CS + col] = wv;
    } else if (idx < (long)F * CS + (long)F * S) {
        const long r = idx - (long)F * CS;
        const int f = (int)(r / S), z = (int)(r % S);
        Wfs[(long)f * (CS + S) + CS + z] = emb[(long)z * F + f];
    }
}

int first_layer_factor(mlp_model *m) {
    m->l0f = false;
    const int F = m->F, K = m->K, S = m->S, CS = S * l0_block(K);
    if (!l0_factorised(K, S)) return 0;
    // P and R (forward), Q_s and Q_v (adjoint) must fit the 6 F floats per
    // atom of the work array
    const L0Layout l0 = l0_layout(F, K, S);
    if (l0.ldp + 3 * l0.ldr > 6 * F || 4 * l0.ldq > 6 * F) return 0;
    const LayerW L = m->layer(0);
    float *src = nullptr;
    const size_t nfs = (size_t)F * (CS + S), nb = (size_t)F * CS;
    if (hipMalloc(&src, sizeof(float) * (nfs + 2 * nb)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(-2, "first-layer weight allocation failed");
    }
    float *Wfs = src, *Wbs = src + nfs, *Wv = Wbs + nb;
    const long tot = (long)F * CS + (long)F * S;
    k_l0_weights<<<nblk(tot, 256), 256>>>(L.A, L.c, m->phi0_dev, m->at(m->off_emb), F, K, S, Wfs, Wbs, Wv);
    const float *Ws[4] = {Wfs, Wv, Wbs, Wv};
    const int C[4] = {CS + S, CS, CS, CS};
    const bool tr[4] = {false, false, true, true};
    size_t bytes = 0;
    for (int q = 0; q < 4; q++) bytes += packed_bytes(F, C[q], tr[q]);
    int rc = hipMalloc(&m->pk_l0_dev, bytes) == hipSuccess ? 0 : -2;
    for (size_t q = 0, o = 0; rc == 0 && q < 4; q++) {
        if (pack_weight(nullptr, Ws[q], F, C[q], tr[q], (char *)m->pk_l0_dev + o, &m->pk_l0[q])) rc = -5;
        o += packed_bytes(F, C[q], tr[q]);
    }
    if (hipDeviceSynchronize() != hipSuccess && rc == 0) rc = -5;
    hipFree(src);
    if (rc) {
        (void)hipGetLastError();
        if (m->pk_l0_dev) hipFree(m->pk_l0_dev);
        m->pk_l0_dev = nullptr;
        return fail(rc, "first-layer weight packing failed");
    }
    m->l0f = true;
    return 0;
}

void eval_model_needs(const mlp_model *m, const mlp_nbr *g, size_t *act, size_t *G, size_t *Gs) {
    const size_t ne = (size_t)g->n_edges_skin;
    if (m->al || m->mc) {
        *act = m->al ? allegro_arena_bytes(m, g->n_atoms, (long)ne) : mace_arena_bytes(m, g->n_atoms, (long)ne, g->skin);
        *G = sizeof(float4) * ne + 64;
        *Gs = 64;
        return;
    }
    *act = act_floats(g->n_atoms, m->F, m->T) * sizeof(float);
    *G = sizeof(float4) * ne + 64;
    *Gs = sizeof(float4) * ne * (size_t)msg_slots(m->F, m->T, m->l0f) + 64;
}

size_t counted_act_bytes(const mlp_model *m, const mlp_nbr *g) {
    const long N = g->n_atoms, ne = g->n_edges_skin, T = m->T, F = m->F;
    if (m->al) return allegro_arena_bytes(m, N, ne, true);
    if (m->mc) return mace_arena_bytes(m, N, ne, g->skin, true);
    return (size_t)(N * F * (T * counted_layer(F) + 4 + counted_adjoint(F)) + N + 64 * (12 * T + 32) + 4096 + QUEUE_INTS +
                    2 * energy_part_doubles(N)) * sizeof(float);
}

int launch_energy(hipStream_t s, const float *U, const int *perm, int n, int n_local, double *energy,
                  float *atom_energy_user, int n_seg, const int *seg_dev, double *part) {
    const int ns = std::max(1, n_seg);
    const dim3 grid((unsigned)ns, (unsigned)std::max(1, (n + ECH - 1) / ECH));
    k_energy_chunk<<<grid, ERED, 0, s>>>(U, perm, seg_dev, n, n_local, part);
    k_energy_total<<<(unsigned)((ns + 63) / 64), 64, 0, s>>>(seg_dev, n, ns, part, energy);
    if (atom_energy_user) k_scatter_energy<<<nblk(n, 256), 256, 0, s>>>(U, perm, n, atom_energy_user);
    HIP_TRY(hipGetLastError());
    return 0;
}

int launch_forces(hipStream_t s, const int *rowc, const int *revc, const float4 *G, const int *perm, int n,
                  float *forces_user) {
    k_forces<<<nblk(16L * n, 256), 256, 0, s>>>(rowc, revc, G, perm, n, forces_user);
    HIP_TRY(hipGetLastError());
    return 0;
}

int evaluate(mlp_model *m, mlp_nbr *g, hipStream_t s, double *energy, float *forces_user,
             float *atom_energy_user, int n_seg, const int *seg_dev) {
    if (m->al) return allegro_evaluate(m, g, s, energy, forces_user, atom_energy_user, n_seg, seg_dev);
    if (m->mc) return mace_evaluate(m, g, s, energy, forces_user, atom_energy_user, n_seg, seg_dev);
    const int n = g->n_atoms, F = m->F, K = m->K, T = m->T;
    // MFMA operand forms of the mode for the node GEMMs (P) and for the
    // radial filter (PF): 0 FP32, 1 plain bfloat16, 2 split bfloat16 (hi + lo)
    const int P = node_operands(m->precision);
    const int PF = filter_operands(m->precision);
    int *Gr = &g->n_grows;
    int rc;
    size_t need_act, need_G, need_Gs;
    eval_model_needs(m, g, &need_act, &need_G, &need_Gs);
    if ((rc = g->act.ensure(need_act, 1.2, Gr))) return rc;
    const long ne = g->n_edges_skin;
    if ((rc = g->G.ensure(need_G, 1.2, Gr))) return rc;
    if ((rc = g->Gs.ensure(need_Gs, 1.2, Gr))) return rc;
    Act A;
    carve(g->act.as<float>(), n, F, T, A);
    // every message launch takes its own zeroed atom counters
    fill_zero(s, reinterpret_cast<float *>(A.queue), QUEUE_INTS);
    int nq = 0;
    auto next_queue = [&]() { return A.queue + (long)(nq++) * MSG_QUEUE_INTS; };
    const int *perm = g->perm.as<int>();
    // edge-sum slots: layers 1 .. T-1 take one each, from slot 0; the first
    // layer's come last (one when it is factorised, else one per pass)
    const int slot0 = T - 1, nslot = msg_slots(F, T, m->l0f);
    const L0Layout l0 = l0_layout(F, K, m->S);

    // Per-layer active sets (Results, "Distributed potential computation",
    // pruning): layer t's outputs are needed within T - 1 - t hops of the
    // locals and its message MLP within T - t hops.  With ghosts the internal
    // order is hop-major (the neighbour build), so those sets are the row
    // prefixes NH(h) and every node kernel runs on its prefix; the message
    // kernels skip atoms by the exact hop marks of this evaluation, which the
    // prefixes contain.  Rows past a prefix hold values that no needed row
    // reads, except the gradients a message adjoint gathers from its
    // destinations: those rows are zeroed (their gradient is zero).
    const bool ho = g->nhop[0] > 0 && g->nhop[std::min(T + 1, MLP_MAX_LAYERS + 1)] == n;
    auto NH = [&](int h) { return ho ? g->nhop[std::max(0, std::min(h, T + 1))] : n; };

    // the node work of layer t: rows NH(T - 1 - t), which are also those whose
    // message MLP of layer t + 1 is needed
    auto node_args = [&](int t) {
        const LayerW L = m->layer(t);
        NodeArgs k;
        k.n = NH(T - 1 - t);
        k.nz = NH(T - t + 1);
        k.chain = m->nd[t];
        k.s1 = A.sn[t];
        k.ld1 = 2 * F;
        k.v1 = A.v1[t];
        k.b3 = L.b3;
        k.b4 = L.b4;
        k.eps = m->eps;
        k.gs1 = A.gs1;
        k.gv1 = A.gv1;
        if (t + 1 < T) {
            const LayerW N = m->layer(t + 1);
            k.b1 = N.b1;
            k.b2 = N.b2;
            k.s2 = A.s[t + 1];
            k.v2 = A.v[t + 1];
            k.phi = A.phi[t + 1];
            k.u = A.work;
            k.gphi = A.gphi;
            k.gv = A.gv;
        }
        return k;
    };

    // forward
    for (int t = 0; t < T; t++) {
        LayerW L = m->layer(t);
        const int hop_dst = T - 1 - t;
        const int ndst = NH(T - 1 - t);
        if (t == 0 && m->l0f) {
            // factorised first layer: basis sums per atom and species, then
            // s1 = [P | one-hot] Wfs^T (s0 included) and v1 = R Wv^T
            L0Args la = l0_args(g, m, hop_dst);
            la.P = A.work;
            la.R = A.work + (long)n * l0.ldp;
            la.ldp = l0.ldp;
            la.ldr = l0.ldr;
            if ((rc = msg_l0_basis_sums(s, K, m->S, la))) return fail(rc, "first-layer kernel launch failed");
            if ((rc = gemm_sv(s, P, la.P, l0.ldp, m->pk_l0[0], A.sn[0], 2 * F, la.R, l0.ldr, m->pk_l0[1], A.v1[0], F, ndst)))
                return fail(rc, "first-layer product launch failed");
        } else {
            MsgArgs ma = msg_args(g, m, L, hop_dst);
            ma.layer0 = t == 0;
            // the first layer reads phi and s from the per-species tables
            ma.phi = t == 0 ? m->phi0_dev : A.phi[t];
            ma.u = A.work;
            ma.s = t == 0 ? m->at(m->off_emb) : A.s[t];
            ma.v = A.v[t];
            ma.sn = A.sn[t];
            ma.v1 = A.v1[t];
            ma.queue = next_queue();
            ProfScope ps(PK_MSG_FWD, s);
            if ((rc = msg_forward(s, PF, F, K, ma))) return fail(rc, "message kernel launch failed");
        }
        ProfScope ps(PK_GEMM, s);
        NodeArgs k = node_args(t);
        if (t + 1 < T) {
            rc = node_forward(s, F, P, k);
        } else {
            // the last update, the readout and, for forces, the adjoint of both
            // (the locals are the prefix NH(0); U of the other rows, reported to
            // the caller as per-atom energies, is zero)
            k.b5 = m->at(m->off_b5);
            k.w6 = m->at(m->off_w6);
            k.b6 = m->at(m->off_b6);
            k.perm = perm;
            k.n_local = g->n_local;
            k.U = A.U;
            k.grad = forces_user != nullptr;
            rc = node_last(s, F, P, k);
        }
        if (rc) return fail(rc, "node kernel launch failed");
    }
    const int nloc = NH(0);
    fill_zero(s, A.U + nloc, (long)(n - nloc));
    if ((rc = launch_energy(s, A.U, perm, n, g->n_local, energy, nullptr, n_seg, seg_dev, A.epart))) return rc;
    if (atom_energy_user) k_scatter_energy<<<nblk(n, 256), 256, 0, s>>>(A.U, perm, n, atom_energy_user);
    if (!forces_user) return 0;

    // adjoint.  Destinations past a layer's set carry no gradient; the message
    // adjoint gathers them up to one hop beyond its sources, so the node
    // kernels zero gs1 and gv1 there.
    for (int t = T - 1; t >= 0; t--) {
        LayerW L = m->layer(t);
        const int hop_src = T - t;
        const int nfar = NH(T - t + 1);
        if (t + 1 < T) {
            ProfScope ps(PK_GEMM, s);
            if ((rc = node_adjoint(s, F, P, node_args(t)))) return fail(rc, "node kernel launch failed");
        }
        if (t == 0 && m->l0f) {
            // factorised first layer: Q_s = gs1 Wbs, Q_v = gv1 Wv, then the
            // edge sums from Q in one slot.  The edge kernel reads Q of every
            // destination of a live source (one hop past the sources), so Q
            // covers the rows through nfar (zero past ndst, as gs1 and gv1).
            L0Args la = l0_args(g, m, hop_src);
            float *Qs = A.work, *Qv = A.work + (long)n * l0.ldq;
            if ((rc = gemm_sv(s, P, A.gs1, F, m->pk_l0[2], Qs, l0.ldq, A.gv1, F, m->pk_l0[3], Qv, l0.ldq, nfar)))
                return fail(rc, "first-layer product launch failed");
            la.Qs = Qs;
            la.Qv = Qv;
            la.ldq = l0.ldq;
            la.S = g->Gs.as<float4>() + (size_t)slot0 * ne;
            if ((rc = msg_l0_edge_sums(s, K, m->S, la))) return fail(rc, "first-layer adjoint kernel launch failed");
        } else {
            MsgArgs ma = msg_args(g, m, L, hop_src);
            ma.phi = t == 0 ? m->phi0_dev : A.phi[t];
            ma.v = A.v[t];
            ma.gs1 = A.gs1;
            ma.gv1 = A.gv1;
            ma.gv_in = A.gv;
            ma.gphi = A.gphi;
            ma.S = g->Gs.as<float4>() + (size_t)(t == 0 ? slot0 : t - 1) * ne;
            ma.layer0 = t == 0;
            ma.queue = next_queue();
            ProfScope ps(PK_MSG_BWD, s);
            if ((rc = msg_adjoint(s, PF, F, K, ma))) return fail(rc, "adjoint message kernel launch failed");
        }
    }
    if ((rc = msg_assemble_G(s, g->rowc.as<int>(), n, ne, g->geom.as<float4>(), g->Gs.as<float4>(), ne, nslot,
                             g->G.as<float4>())))
        return fail(rc, "edge-gradient kernel launch failed");
    k_forces<<<nblk(16L * n, 256), 256, 0, s>>>(g->rowc.as<int>(), g->revc.as<int>(), g->G.as<float4>(), perm, n,
                                                forces_user);
    HIP_TRY(hipGetLastError());
    return 0;
}

// ---------------------------------------------------------------------------
// Velocity Verlet (SoA, A/fs, amu, eV/A)
// ---------------------------------------------------------------------------
constexpr float ACC = 9.648533212e-3f;  // (eV / A / amu) -> A / fs^2

__global__ void k_kick_drift(float *__restrict__ x, float *__restrict__ v, const float *__restrict__ f,
                             const float *__restrict__ im, int n, float L0, float L1, float L2, float dt) {
    long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= 3L * n) return;
    int d = idx / n;
    long u = idx % n;
    float vv = fmaf(0.5f * dt * ACC * im[u], f[idx], v[idx]);
    v[idx] = vv;
    float L = d == 0 ? L0 : (d == 1 ? L1 : L2);
    float p = fmaf(dt, vv, x[idx]);
    if (L > 0.f) {
        p = p - L * floorf(p / L);
        if (p >= L) p -= L;
        if (p < 0.f) p += L;
    }
    x[idx] = p;
}

__global__ void k_kick(float *__restrict__ v, const float *__restrict__ f, const float *__restrict__ im, int n,
                       float dt) {
    long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= 3L * n) return;
    long u = idx % n;
    v[idx] = fmaf(0.5f * dt * ACC * im[u], f[idx], v[idx]);
}

int verlet_kick_drift(float *pos, float *vel, const float *forces, const float *inv_mass, int n,
                      const double box[3], float dt, hipStream_t s) {
    k_kick_drift<<<nblk(3L * n, 256), 256, 0, s>>>(pos, vel, forces, inv_mass, n, (float)box[0], (float)box[1],
                                                   (float)box[2], dt);
    HIP_TRY(hipGetLastError());
    return 0;
}

int verlet_kick(float *vel, const float *forces, const float *inv_mass, int n, float dt, hipStream_t s) {
    k_kick<<<nblk(3L * n, 256), 256, 0, s>>>(vel, forces, inv_mass, n, dt);
    HIP_TRY(hipGetLastError());
    return 0;
}

}  // namespace mlp
