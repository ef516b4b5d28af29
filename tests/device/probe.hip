// Device functions of the kernels on inputs of a test's own, for what an
// evaluation's result cannot show: rounding of single products, and kernel
// variants that only the largest systems take.  Built next to the library
// (libprobe.so), loaded by tests/test_gpu_device.py.
#include "../../paper_2506_04055_amd/csrc/msg.hip"
#include "../../paper_2506_04055_amd/csrc/edge_chain.h"

using namespace mlp;

namespace {

// D[s] = A[s] B[s]^T, A and B 16 x K, one wave per s: a layer's FP32 products
constexpr int PK = 128;
__global__ void __launch_bounds__(64) k_products(const float *__restrict__ A, const float *__restrict__ B, float *__restrict__ D) {
    const int l = threadIdx.x, c = l & 15, g = l >> 4;
    const float *a = A + ((long)blockIdx.x * 16 + c) * PK, *b = B + ((long)blockIdx.x * 16 + c) * PK;
    ec_v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < PK; k += 32) {
        auto op = [&](const float *p) {
            return ec_op<0>(*reinterpret_cast<const ec_v4f *>(p + k + 8 * g), *reinterpret_cast<const ec_v4f *>(p + k + 8 * g + 4));
        };
        const EcOp<0> w = op(a), x = op(b);
        ec_mul<0, 1>([&](int) { return w.p; }, [&](int) -> const EcOp<0> & { return x; }, [&](int) -> ec_v4f & { return acc; });
    }
    for (int r = 0; r < 4; r++) D[(long)blockIdx.x * 256 + (4 * g + r) * 16 + c] = acc[r];
}

// The radial filter of 16 edges per workgroup: its basis values e~ [edge][32]
// and the tiles of one pass w [edge][96] (F = 128), of the values or (der) the derivatives.
template <int K>
__global__ void __launch_bounds__(256) k_filter(const float *__restrict__ A, const float *__restrict__ c, const float *__restrict__ r, float rc,
                                                int der, float *__restrict__ e_out, float *__restrict__ w_out) {
    using B = Basis<0, K>;
    __shared__ __attribute__((aligned(16))) char lds[WStage<0, 128, K, 32, true>::BYTES];
    stage_pass<0, 128, K, 32, true>(A, c, 0, lds);
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x, e = lane & 15, g = lane >> 4;
    const long edge = 16L * blockIdx.x;
    const float rr = r[edge + e];
    float eb[B::SLOTS], db[B::SLOTS];
    basis_slots<0, K, true>(rr, __builtin_amdgcn_rcpf(rr), 3.14159265358979f / rc, true, g, eb, db);
    const float *v = der ? db : eb;
    for (int q = 0; q < B::KG; q++) e_out[(edge + e) * 32 + B::KG * g + q] = v[q];
    if (B::LEFT && g == 0) e_out[(edge + e) * 32 + K] = v[B::KG];
    BOp<0, K> b;
    b.set(v, g);
    for (int t = 0; t < 6; t++) {
        const v4f x = filter_tile<0, 128, K, 32, true, true>(lds, t, b, lane);
        for (int q = 0; q < 4; q++) w_out[(edge + 4 * g + q) * 96 + 16 * t + e] = x[q];
    }
}

// sigmoid, SiLU and SiLU' of the edge chains, and the sigmoid's denominator
__global__ void k_sigmoid(const float *__restrict__ x, int n, float4 *__restrict__ o) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    ec_v4f v = {x[i], 0.f, 0.f, 0.f};
    const ec_v4f s = ec_silu_d<0>(v);
    o[i] = make_float4(1.0f + __expf(-x[i]), ec_sigmoid<0>(x[i]), s[0], v[0]);
}

// sin and cos of pi r / rc as the edge chains take them
__global__ void k_phase(const float *__restrict__ r, int n, float th, float thl, float2 *__restrict__ o) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) ec_sincos_0pi<0>(th, thl, r[i], o[i].x, o[i].y);
}

// The message pass or its adjoint with either form of the row offsets
template <int P, int F, int K, bool WIDE>
void message(int adjoint, const MsgArgs &a) {
    if (adjoint)
        k_msg_bwd_pw<P, F, K, WIDE><<<8, 64 * BWD_PIW_WAVES>>>(a.rowc, a.colc, a.geom, a.n, a.phi, a.v, a.gs1, a.gv1, a.A, a.c, a.rc, a.hop,
                                                             a.hop_max, a.queue, a.gv_in, a.gphi, a.S);
    else
        k_msg_fwd_pw<P, F, K, WIDE><<<8, 64 * FWD_PIW_WAVES>>>(a.rowc, a.colc, a.geom, a.n, a.phi, a.u, a.s, a.v, a.A, a.c, a.rc, a.hop,
                                                             a.hop_max, a.queue, a.sn, a.v1);
}
// byte offsets of (row, element) pairs in a row-major array, in the 32-bit form
__global__ void k_row_offset(const int *__restrict__ row, const int *__restrict__ f, int n, int ld, unsigned long long *__restrict__ o) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) o[i] = RowAt<false>(row[i], ld, f[i]).o;
}

}  // namespace

namespace mlp {
int fail(int code, const std::string &) { return code; }
}  // namespace mlp

extern "C" {

static int done() { return hipGetLastError() == hipSuccess && hipDeviceSynchronize() == hipSuccess ? 0 : -5; }

int probe_products(const float *A, const float *B, float *D, int samples) {
    k_products<<<samples, 64>>>(A, B, D);
    return done();
}
int probe_filter(int K, const float *A, const float *c, const float *r, float rc, int n16, int der, float *e, float *w) {
    if (K == 20) k_filter<20><<<n16, 256>>>(A, c, r, rc, der, e, w);
    else if (K == 8) k_filter<8><<<n16, 256>>>(A, c, r, rc, der, e, w);
    else if (K == 6) k_filter<6><<<n16, 256>>>(A, c, r, rc, der, e, w);
    else return -1;
    return done();
}
int probe_sigmoid(const float *x, int n, float *o) {
    k_sigmoid<<<(n + 255) / 256, 256>>>(x, n, reinterpret_cast<float4 *>(o));
    return done();
}
int probe_phase(const float *r, int n, float rc, float *o) {
    float th, thl;
    ec_phase(rc, th, thl);
    k_phase<<<(n + 255) / 256, 256>>>(r, n, th, thl, reinterpret_cast<float2 *>(o));
    return done();
}
// atoms per workgroup of the fused edge kernels (host)
int probe_atoms_per_workgroup(long n, long n_edges_skin, float rc, float skin, int slots) {
    return ec_per_wg(n, n_edges_skin, rc, skin, slots);
}
int probe_wide(long n, int F) { return msg_wide(n, F); }
int probe_row_offset(const int *row, const int *f, int n, int ld, unsigned long long *o) {
    k_row_offset<<<(n + 255) / 256, 256>>>(row, f, n, ld, o);
    return done();
}
// in: rowc colc geom phi u s v gs1 gv1 A c hop; out: forward sn v1, adjoint gv gphi S; queue zeroed
int probe_message(int wide, int adjoint, int F, int n, float rc, int hop_max, const void *const *in, void *const *out, int *queue) {
    MsgArgs a = {};
    a.rowc = (const int *)in[0], a.colc = (const int *)in[1], a.geom = (const float4 *)in[2], a.n = n;
    a.phi = (const float *)in[3], a.u = (const float *)in[4], a.s = (const float *)in[5], a.v = (const float *)in[6];
    a.gs1 = (const float *)in[7], a.gv1 = (const float *)in[8], a.A = (const float *)in[9], a.c = (const float *)in[10];
    a.hop = (const int8_t *)in[11], a.hop_max = hop_max, a.rc = rc, a.queue = queue;
    a.sn = (float *)out[0], a.v1 = (float *)out[1];
    a.gv_in = (float *)out[0], a.gphi = (float *)out[1], a.S = (float4 *)out[2];
    if (F == 64) wide ? message<2, 64, 8, true>(adjoint, a) : message<2, 64, 8, false>(adjoint, a);
    else wide ? message<0, 128, 20, true>(adjoint, a) : message<0, 128, 20, false>(adjoint, a);
    return done();
}

}  // extern "C"
