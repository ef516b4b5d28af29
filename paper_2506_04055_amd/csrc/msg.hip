// Message pass and its adjoint with the radial-filter contraction on MFMA.
//
// Per directed edge (i <- j) the filter is w = A' e~(r), a dense K+1 -> 3F
// contraction with A' = [c | A] and e~ = [fc, e_1 fc, ..., e_K fc],
// e_k = sin(k pi r / rc) / r.  A wave owns one atom and takes its edges 16 at
// a time.  The filter of a chunk is computed as 16 x 16 MFMA tiles (16
// features x 16 edges) from two operands: 16 rows of A' (staged in LDS once
// per workgroup) and e~ of the 16 edges (each lane evaluates the basis slots
// it holds; the slots of padding edges are zero, so they contribute nothing).
// The vector phase works in the accumulator layout of the tiles; no LDS round
// trip sits between the matrix cores and the vector ALUs.  Features are
// processed in passes of W = min(F, 32).  Two arrangements:
//
// * One pass per workgroup (k_msg_fwd, k_msg_bwd: the first layer when it is
//   not factorised, and models with a single pass).  blockIdx.y is the pass;
//   A' is the first MFMA operand, so lane l = 16 g + e holds features
//   4g .. 4g+3 of the tile for edge e: it gathers the matching 16-byte pieces
//   of its edge's neighbour rows (quarter-contiguously, then moved through
//   LDS), sums over the features of an edge stay inside the lane (plus one
//   exchange across the four lane rows), sums over the edges of the atom stay
//   inside the lane over the chunks (plus one 16-lane DPP row reduction per
//   atom).  The basis is evaluated per pass.
// * All passes in the wave (k_msg_fwd_pw, k_msg_bwd_pw: the layers after the
//   first with more than one pass).  The weight images of every pass are in
//   LDS; the basis of a chunk, in MFMA operand form, is evaluated in the first
//   pass and kept in the wave's LDS for the later ones.  e~ is the first MFMA
//   operand, so the tile comes out transposed: lane (f, g) holds feature f of
//   the tile for the edges 4g .. 4g+3.  It gathers 16 consecutive features of
//   a row per quarter-wave (no exchange), adds its four edges in registers,
//   and the sums over an atom's edges reduce over the four lane rows once per
//   atom and pass; the adjoint's sums over the features of an edge go through
//   a reduce-scatter over the 16 lanes of a row.
//
// Precision P = 1: bfloat16 operands; P = 2: split bfloat16 operands
// x = hi + lo (hi = bf16(x), lo = bf16(x - hi)) with the three products
// lo*hi + hi*lo + hi*hi; P = 0: FP32 operands as three bfloat16 parts, six
// products (24 bits; what is dropped is below 2^-26); accumulation FP32 in
// all, on v_mfma_f32_16x16x32_bf16.  The products of a slot share an
// instruction (Basis): per 16 x 16 tile two instructions of 16 cycles for
// K = 20 split and four for FP32, where one per product took three, and
// v_mfma_f32_16x16x4_f32 six of 32 cycles.  48k-atom water slab, FP32, F = 128:
// adjoint 1,460 -> 1,120 us and forward 795 -> 590 us per launch by this alone
// (950 and 490 with all that stands below); 24k atoms, split: 476 -> 447 and
// 268 -> 255 us (357 and 206).  Every sum has a fixed order, so results are
// bitwise reproducible.
//
// The adjoint is organised by source atom j over its in-edges (j <- i), the
// reverses of the edges (i <- j) that carried j's messages; it gathers the
// destination gradients and accumulates dE/dphi_j and dE/dv_j.  For every edge
// it also forms S = (dE/dr, dE/drhat) summed over the features (dE/dr through
// dw/dr = A' de~/dr, a second MFMA): one slot per layer (the all-pass kernel
// adds the passes up in the wave) or per layer and pass (one pass per
// workgroup), each written by one lane only.  The edge gradient
// G = dE/d(x_j - x_i) = (dE/dr) rhat + (I - rhat rhat^T) dE/drhat / r is linear
// in S and is assembled once after the last layer.
#include "internal.h"
#include "msg.h"

namespace mlp {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// How the basis meets the weights.  Plain bfloat16: one product over 32 slots,
// lane group g holding the slots k = 8 g .. 8 g + 7.  Split bfloat16 (parts
// hi, lo) takes three products per slot (lo hi, hi lo, hi hi) and FP32 as
// three bfloat16 parts six (those below 2^-26 dropped): the products of a slot
// are further slots of the same instruction, so 3 (K + 1) or 6 (K + 1) of them
// fill its 32 - two instructions for K = 20 split, four for FP32, where one
// per product takes three or six.  (FP32 with K = 8 or 6 takes a third, so that
// the products of the leading parts have the last to themselves: filter_tile.)
// Lane group g holds the KG values
// k = KG g + j; what four groups leave over (k = K) sits in slots they leave
// free.
template <int P, int K>
struct Basis {
    static constexpr int KG = P == 1 ? 8 : (K + 1) / 4 > 1 ? (K + 1) / 4 : 2;   // values per lane group
    static constexpr bool LEFT = P != 1 && K + 1 > 4 * KG;
    static constexpr int SLOTS = KG + LEFT;                                     // values per lane
    static constexpr int PARTS = P == 0 ? 3 : P;
    static constexpr int NM = P == 1 ? 1 : P == 0 ? (KG == 5 ? 4 : 3) : (3 * (K + 1) + 31) / 32;   // instructions
    static_assert(P == 1 || KG == 5 || KG == 2, "layouts of K = 20, 8 and 6");
};

// Slot q of lane group g in instruction m: the value k and the weight part it
// meets (part < 0: none).
struct WSlot {
    int k, part;
};
template <int P, int K>
__device__ __forceinline__ WSlot weight_slot(int m, int g, int q) {
    using B = Basis<P, K>;
    if constexpr (P == 1) return {8 * g + q, 8 * g + q <= K ? 0 : -1};
    const int k0 = B::KG * g;
    int k, part;
    if constexpr (B::KG == 5) {
        if (q < 4) {
            k = k0 + q;
            part = P == 2 ? (m == 0 ? 1 : 0) : (m == 0 ? 2 : m == 1 ? 1 : 0);
        } else if (P == 2 ? m == 0 : m < 2) {
            k = k0 + q - 4;
            part = P == 2 ? 0 : m;
        } else if (P == 2 || m == 2 || q < 6) {
            k = k0 + 4;
            part = P == 2 ? q == 4 : m == 3 ? 0 : q == 4 ? 2 : q == 5 ? 0 : 1;
            if (P == 2 && q == 7) {
                k = K;
                part = g == 3 ? -1 : g == 2;
            }
        } else {
            k = K;
            part = g == 3 ? -1 : q == 6 ? g : g == 1;
        }
    } else {
        const int d = 4 * m + q / 2, odd = q & 1;   // pair of slots
        const bool left = P == 2 ? d == 3 : d > 4 && d != 8;   // the value left over
        k = left ? K : k0 + odd;
        if (!left) part = P == 2 ? d == 0 : d == 0 ? 2 : d == 2 || d == 3 ? 1 : 0;
        else if (!B::LEFT) part = -1;
        else if (P == 2) part = g == 0 ? 0 : g == 1 && !odd ? 1 : -1;
        else if (g > 0 || d > 9) part = -1;
        else part = d == 5 ? (odd ? 0 : 2) : d == 6 ? 1 : odd ? -1 : 0;
    }
    return {k, k <= K ? part : -1};
}

// sin and cos of th in [0, pi] without range reduction: with x = th - pi/2 in
// [-pi/2, pi/2], sin th = cos x and cos th = -sin x, both from their Taylor
// series (through x^13 and x^14; truncation below 1e-9 on this interval).
__device__ __forceinline__ void sincos_0pi(float th, float &s, float &c) {
    const float x = th - 1.57079632679489662f, x2 = x * x;
    float p = 1.0f / 6227020800.0f;
    p = fmaf(p, x2, -1.0f / 39916800.0f);
    p = fmaf(p, x2, 1.0f / 362880.0f);
    p = fmaf(p, x2, -1.0f / 5040.0f);
    p = fmaf(p, x2, 1.0f / 120.0f);
    p = fmaf(p, x2, -1.0f / 6.0f);
    p = fmaf(p, x2, 1.0f);
    float q = -1.0f / 87178291200.0f;
    q = fmaf(q, x2, 1.0f / 479001600.0f);
    q = fmaf(q, x2, -1.0f / 3628800.0f);
    q = fmaf(q, x2, 1.0f / 40320.0f);
    q = fmaf(q, x2, -1.0f / 720.0f);
    q = fmaf(q, x2, 1.0f / 24.0f);
    q = fmaf(q, x2, -0.5f);
    q = fmaf(q, x2, 1.0f);
    s = q;
    c = -x * p;
}

// Basis values (and optionally their r-derivatives) a lane holds: k = KG g + j
// and, after them, k = K where it is left over.  r < rc for every valid edge,
// so th = pi r / rc lies in [0, pi).  The lane's first angle comes from angle
// sums, the rest from the Chebyshev recurrences
// sin((k+1) th) = 2 cos(th) sin(k th) - sin((k-1) th) (and the same for cos).
// Values k > K meet zero weights, so they do not matter as long as they are
// finite.  Padding edges (valid = false, ir = 0) get exact zeros.
template <int P, int K, bool DERIV>
__device__ __forceinline__ void basis_slots(float r, float ir, float pirc, bool valid, int g, float *eb, float *db) {
    using B = Basis<P, K>;
    float s1, c1;
    sincos_0pi(r * pirc, s1, c1);
    const float fc = valid ? 0.5f * (c1 + 1.0f) : 0.f;
    const float dfc = valid ? -0.5f * pirc * s1 : 0.f;
    const float es = ir * fc;                    // e_k = sin(k th) es
    const float da = pirc * es, dbb = ir * (dfc - es);   // de_k = cos(k th) k da + sin(k th) dbb
    const float s2 = 2.0f * s1 * c1, c2 = fmaf(-2.0f * s1, s1, 1.0f);
    const float s4 = 2.0f * s2 * c2, c4 = fmaf(-2.0f * s2, s2, 1.0f);
    // sin and cos of KG g th, and of 4 KG th
    float x1, y1, x2, y2, x3, y3, sl, cl;
    if constexpr (B::KG == 5) {
        x1 = fmaf(s4, c1, c4 * s1), y1 = fmaf(c4, c1, -s4 * s1);
        x2 = 2.0f * x1 * y1, y2 = fmaf(-2.0f * x1, x1, 1.0f);
    } else if constexpr (B::KG == 2) {
        x1 = s2, y1 = c2;
        x2 = s4, y2 = c4;
    } else {
        x1 = 2.0f * s4 * c4, y1 = fmaf(-2.0f * s4, s4, 1.0f);
        x2 = 2.0f * x1 * y1, y2 = fmaf(-2.0f * x1, x1, 1.0f);
    }
    x3 = fmaf(x2, y1, y2 * x1), y3 = fmaf(y2, y1, -x2 * x1);
    sl = 2.0f * x2 * y2, cl = fmaf(-2.0f * x2, x2, 1.0f);
    float sk = g == 0 ? 0.f : (g == 1 ? x1 : (g == 2 ? x2 : x3));
    float ck = g == 0 ? 1.f : (g == 1 ? y1 : (g == 2 ? y2 : y3));
    float sm = fmaf(sk, c1, -ck * s1);   // sin((KG g - 1) th)
    float cm = fmaf(ck, c1, sk * s1);
    const float tc = 2.0f * c1;
#pragma unroll
    for (int q = 0; q < B::KG; q++) {
        float e = sk * es, de = 0.f;
        if (DERIV) de = fmaf(ck, (float)(B::KG * g + q) * da, sk * dbb);
        if (q == 0 && g == 0) {   // k = 0: the envelope itself
            e = fc;
            de = dfc;
        }
        eb[q] = e;
        if (DERIV) db[q] = de;
        const float sn = fmaf(tc, sk, -sm);
        sm = sk;
        sk = sn;
        if (DERIV) {
            const float cn = fmaf(tc, ck, -cm);
            cm = ck;
            ck = cn;
        }
    }
    if constexpr (B::LEFT) {
        eb[B::KG] = sl * es;
        if (DERIV) db[B::KG] = fmaf(cl, (float)K * da, sl * dbb);
    }
}

// The basis of one chunk as the MFMAs take it.  Kept between passes (Store):
// the operand itself, or in FP32 mode the values, which take fewer words.
template <int P, int K>
struct BOp {
    using B = Basis<P, K>;
    v8bf m[B::NM];
    // (g: the lane's group)
    __device__ __forceinline__ void set(const float *eb, int g) {
        if constexpr (P == 1) {
#pragma unroll
            for (int q = 0; q < 8; q++) m[0][q] = (__bf16)eb[q];
        } else {
            // parts of the values in pairs: word p of part t holds values 2 p
            // and 2 p + 1.  The remainder x - hi (exact) comes from the two-term
            // dot product, whose second factor picks one of the pair; as an
            // inline constant -1.0 it would take the pair (0, -1), so the factors
            // are kept in registers
            constexpr int NP = (B::SLOTS + 1) / 2;
            unsigned k0 = 0x0000BF80u, k1 = 0xBF800000u;
            asm("" : "+s"(k0), "+s"(k1));
            unsigned h[B::PARTS][NP];
#pragma unroll
            for (int p = 0; p < NP; p++) {
                float x = eb[2 * p], y = 2 * p + 1 < B::SLOTS ? eb[2 * p + 1] : 0.f;
#pragma unroll
                for (int t = 0; t < B::PARTS; t++) {
                    const v2bf w = __builtin_convertvector((v2f){x, y}, v2bf);
                    h[t][p] = __builtin_bit_cast(unsigned, w);
                    if (t + 1 < B::PARTS) {
                        x = __builtin_amdgcn_fdot2_f32_bf16(w, __builtin_bit_cast(v2bf, k0), x, false);
                        y = __builtin_amdgcn_fdot2_f32_bf16(w, __builtin_bit_cast(v2bf, k1), y, false);
                    }
                }
            }
            auto low = [](unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); };    // (a.lo, b.lo)
            auto lohi = [](unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060100u); };   // (a.lo, b.hi)
            auto high = [](unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };   // (a.hi, b.hi)
            auto put = [&](int i, unsigned a, unsigned b, unsigned c, unsigned d) {
                m[i] = __builtin_bit_cast(v8bf, (v4u){a, b, c, d});
            };
            if constexpr (P == 2 && B::KG == 5) {
                const unsigned left = g == 1 ? h[1][2] : h[0][2];
                put(0, h[0][0], h[0][1], h[1][0], h[1][1]);
                put(1, h[0][0], h[0][1], low(h[0][2], h[1][2]), lohi(h[0][2], left));
            } else if constexpr (P == 2) {
                unsigned left = 0;
                if constexpr (B::LEFT) left = low(h[0][1], h[1][1]);
                put(0, h[0][0], h[1][0], h[0][0], left);
            } else if constexpr (B::KG == 5) {
                const unsigned f01 = low(h[0][2], h[1][2]), left = g == 2 ? h[2][2] : h[1][2];
                put(0, h[0][0], h[0][1], h[2][0], h[2][1]);
                put(1, h[0][0], h[0][1], h[1][0], h[1][1]);
                put(2, h[1][0], h[1][1], low(h[0][2], h[2][2]), f01);
                put(3, h[0][0], h[0][1], f01, high(h[0][2], left));
            } else {
                unsigned l0 = 0, l1 = 0, l2 = 0, l3 = 0;
                if constexpr (B::LEFT) l0 = h[0][1], l1 = h[1][1], l2 = low(l0, h[2][1]), l3 = low(l1, l0);
                put(0, h[0][0], h[2][0], h[1][0], h[0][0]);
                put(1, h[1][0], l2, l3, l1);
                put(2, h[0][0], l0, 0, 0);
            }
        }
    }
};

// Features per pass (at most WM) and the pass count.
template <int F, int WM>
struct Pass {
    static constexpr int W = F < WM ? F : WM;   // features per pass
    static constexpr int N = F / W;             // passes
    static constexpr int TU = W / 16;           // 16-feature tiles per part and pass
};

// LDS image of the pass's rows of A' = [c | A]: local row q W + f holds the
// global row q F + p W + f (part q = 0, 1, 2), in the layout the A operand
// reads (reduction index contiguous).  Rows are padded against bank
// conflicts (8 bf16 or one float), or, with SW (bf16 only), unpadded and
// swizzled: a 64-byte row is four 16-byte pieces of 8 slots, and piece h of
// row r sits at position h ^ wswz(r), which puts the 16 rows that one
// A-operand read touches (same piece, rows 16 t .. 16 t + 15) on distinct
// 16-byte bank groups for 32 or 64 banks, in 20 % less LDS.
template <int P, int F, int K, int WM, bool SW = false>
struct WStage {
    static constexpr int ROWS = 3 * Pass<F, WM>::W;
    static constexpr int LD = SW ? 32 : 40;                       // row stride (elements)
    static constexpr int ELEMS = ROWS * LD * Basis<P, K>::NM;     // a table per instruction
    static constexpr int BYTES = ELEMS * 2;
};
__device__ __forceinline__ int wswz(int r) { return (((r >> 2) & 1) << 1) | (((r >> 1) ^ (r >> 3)) & 1); }

template <int P, int F, int K, int WM, bool SW = false>
__device__ __forceinline__ void stage_pass(const float *__restrict__ A, const float *__restrict__ c, int p,
                                           void *lds) {
    using WS = WStage<P, F, K, WM, SW>;
    constexpr int W = Pass<F, WM>::W;
    // a thread keeps to one slot, so what it holds is worked out once per table
    const int k = threadIdx.x & 31, pos = k & 7;
#pragma unroll
    for (int mm = 0; mm < Basis<P, K>::NM; mm++) {
        const WSlot w = weight_slot<P, K>(mm, k >> 3, pos);
        const float *src = w.k == 0 ? c : A + (w.k - 1);
        const int ld = w.k == 0 ? 1 : K;
#pragma unroll 4
        for (int lr = threadIdx.x >> 5; lr < WS::ROWS; lr += blockDim.x >> 5) {
            const int f = (lr / W) * F + p * W + lr % W;
            float v = 0.f;
            if (w.part >= 0) v = src[(long)f * ld];
            const float r1 = v - (float)(__bf16)v, r2 = r1 - (float)(__bf16)r1;
            v = w.part == 2 ? r2 : w.part == 1 ? r1 : v;
            reinterpret_cast<__bf16 *>(lds)[(mm * WS::ROWS + lr) * WS::LD + (SW ? (((k >> 3) ^ wswz(lr)) << 3) + pos : k)] = (__bf16)v;
        }
    }
    __syncthreads();
}

// Filter values of local tile t (rows 16t .. 16t+15): lane (e, g) receives
// features 4g .. 4g+3 of the tile for its edge e; with TR (the operands
// swapped, the same products) lane (f, g) receives feature f of the tile for
// the edges 4g .. 4g+3.
template <int P, int F, int K, int WM, bool SW = false, bool TR = false>
__device__ __forceinline__ v4f filter_tile(const void *lds, int t, const BOp<P, K> &b, int lane) {
    using WS = WStage<P, F, K, WM, SW>;
    // FP32: what an instruction adds is cut off, not rounded, below the
    // precision of its largest term, so smaller products summed together with
    // those of the leading parts pull the filter down (8e-9 of it on average,
    // which adds up over the atoms of an energy).  The last instruction, which
    // has the leading parts, sums from zero and is added as a whole (below 1e-10
    // where it has nothing else, 1e-9 with what K = 20 leaves over for it).
    v4f acc = {0.f, 0.f, 0.f, 0.f}, hh = acc;
    const int row = 16 * t + (lane & 15), g = lane >> 4;
    // the swizzled piece position depends on the lane only (16 t leaves bits
    // 1-3 of the row alone)
    const int col = 8 * (SW ? g ^ wswz(lane & 15) : g);
    const __bf16 *t0 = reinterpret_cast<const __bf16 *>(lds) + row * WS::LD + col;
#pragma unroll
    for (int i = 0; i < Basis<P, K>::NM; i++) {
        const v8bf a = *reinterpret_cast<const v8bf *>(t0 + i * WS::ROWS * WS::LD);
        v4f &x = P == 0 && i + 1 == Basis<P, K>::NM ? hh : acc;
        x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(TR ? b.m[i] : a, TR ? a : b.m[i], x, 0, 0, 0);
    }
    if constexpr (P == 0) acc += hh;
    return acc;
}

// DPP move inside rows of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// Sum over the 16 lanes of each row (lanes 16g .. 16g+15), by rotations of the
// row and quad permutations; every lane of the row receives the total.
__device__ __forceinline__ float row_sum16(float x) {
    x += dpp<0x128>(x);   // row_ror:8
    x += dpp<0x124>(x);   // row_ror:4
    x += dpp<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp<0xB1>(x);    // quad_perm [1,0,3,2]
    // materialise the total here: otherwise the last add sinks into the
    // lane-0 store branch, where it cannot take the DPP operand and costs a
    // zeroed register, a DPP move and a plain add per value
    asm volatile("" : "+v"(x));
    return x;
}

// The weight image, at an offset the compiler cannot see through, so the A
// operands are re-read from LDS in every chunk instead of being held in 48
// registers across the chunk loop (which would cost occupancy).
__device__ __forceinline__ const char *lds_chunk(const char *lds) {
    int z = 0;
    asm volatile("" : "+s"(z));
    return lds + z;
}

__device__ __forceinline__ v4f ld4(const float *p) { return *reinterpret_cast<const v4f *>(p); }
__device__ __forceinline__ void st4(float *p, v4f x) { *reinterpret_cast<v4f *>(p) = x; }

// Neighbour rows are gathered quarter-contiguously and then moved to the
// accumulator layout through LDS.  In the accumulator layout lane (g, e) =
// 16 g + e needs features 4g .. 4g+3 (of a 16-feature tile) of edge e, so
// the 16 lanes of a quarter-wave would touch 16 different rows, 16 bytes
// each: the L1 then serves one 16-byte piece per access.  Instead lane
// (g, e) loads features 4(e % 4) .. +3 of the row of edge 4g + e/4 (each
// quarter reads four whole 64-byte pieces) and stores them in LDS at the
// slot of the lane that needs them, 16(e % 4) + 4g + e/4, from where every
// lane reads its own slot.  Slot D sits at index swz(D): its bits 2-3 are
// XOR-ed with its quarter, which keeps the writes and the reads of a
// quarter-wave on 16 distinct 16-byte bank groups.
struct Xch {
    int src;   // lane holding the edge whose row this lane gathers
    int fo;    // feature offset of the gathered piece inside a 16-feature tile
    int wr;    // LDS slot this lane writes
    int rd;    // LDS slot this lane reads
    __device__ static int swz(int d) { return (d & 0x33) | ((((d >> 2) & 3) ^ (d >> 4)) << 2); }
    __device__ Xch(int g, int e) {
        src = 4 * g + (e >> 2);
        fo = 4 * (e & 3);
        wr = swz(16 * (e & 3) + 4 * g + (e >> 2));
        rd = swz(16 * g + e);
    }
    // one 64-lane, 16-byte-per-lane exchange through the wave's buffer slot
    __device__ v4f move(v4f *buf, v4f x) const {
        buf[wr] = x;
        __builtin_amdgcn_wave_barrier();   // the read sees the whole wave's writes
        return buf[rd];
    }
};

#ifndef MSG_MW
#define MSG_MW 4
#endif
constexpr int MW = MSG_MW;   // waves per workgroup
// features per pass of the forward and the adjoint (16 or 32)
#ifndef FWD_W
#define FWD_W 32
#endif
#ifndef BWD_W
#define BWD_W 32
#endif
#ifndef FWD_WAVES
#define FWD_WAVES 4
#endif
#ifndef FWD_WAVES0
#define FWD_WAVES0 5
#endif
#ifndef BWD_WAVES0
#define BWD_WAVES0 4
#endif
#ifndef BWD_WAVES
#define BWD_WAVES 2
#endif

// Atoms for each wave, from a work queue per XCD slice.  Workgroups are
// dispatched round-robin over the XCDs, each with its own L2; with gridDim.x
// a multiple of 8, XCD x runs the workgroups with blockIdx.x % 8 == x and
// works on the contiguous slice [x n / 8, (x+1) n / 8) of the cell-sorted
// atoms.  The waves of a slice take its atoms in order, MSG_QB at a time, from
// one counter, so the atoms in flight on an XCD are always a compact window of
// the slice, whose neighbour rows the XCD's L2 holds (with a fixed
// interleaving the waves drift apart over the slice and the rows in use
// outgrow the L2).  Each counter has its own 128-byte line and starts at
// zero.  The slices partition [0, n) whatever the grid size; every wave leaves
// its loop once its slice's counter has passed the end.
#ifndef MSG_QB
#define MSG_QB 1
#endif
struct AtomQueue {
    int lo, hi;
    int *ctr;
    __device__ __forceinline__ AtomQueue(int n, int *queue, int pass) {
        const int nx = gridDim.x < 8 ? (int)gridDim.x : 8;
        const int x = blockIdx.x % nx;
        lo = (int)((long)n * x / nx);
        hi = (int)((long)n * (x + 1) / nx);
        ctr = queue + (pass * 8 + x) * 32;
    }
    // a ticket: the counter's old value in lane 0 (issue), and the first atom
    // of the wave's batch it names (wave-uniform; >= hi once the slice is
    // drained), read only when needed (resolve), so the atomic's latency can
    // pass under other work
    __device__ __forceinline__ int issue() const {
        int t = 0;
        if ((threadIdx.x & 63) == 0)
            t = __hip_atomic_fetch_add(ctr, MSG_QB, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return t;
    }
    __device__ __forceinline__ int resolve(int t) const { return lo + __builtin_amdgcn_readfirstlane(t); }
    __device__ __forceinline__ int take() const { return resolve(issue()); }
};
// for (each atom I of the wave, in queue order)
#if MSG_QB == 1
#define MSG_ATOMS(Q, I) for (int I = (Q).take(); I < (Q).hi; I = (Q).take())
// The same with the next ticket issued when an atom starts and resolved when
// it ends, so the atomic's latency passes under the atom's work (the last
// one is not used).  Each wave then holds two tickets, which doubles the
// window of atoms in flight: worth it in the adjoint (2 waves per SIMD), not
// in the forward, whose L2 then holds its window's rows less well.
#define MSG_ATOMS_AHEAD(Q, I)                                                \
    for (int I = (Q).take(), I##_t = (Q).issue(); I < (Q).hi; I = (Q).resolve(I##_t), I##_t = (Q).issue())
#else
#define MSG_ATOMS(Q, I)                                           \
    for (int I##_b = (Q).take(); I##_b < (Q).hi; I##_b = (Q).take()) \
        for (int I = I##_b; I < I##_b + MSG_QB && I < (Q).hi; I++)
#define MSG_ATOMS_AHEAD(Q, I) MSG_ATOMS(Q, I)
#endif

// A chunk's basis kept in LDS between passes, stored lane-contiguously so that
// the writes and reads are conflict-free: the operand in 16-byte words, in FP32
// mode the values (a third fewer bytes; the parts are formed again).  Each lane
// reads back only what it wrote itself, so no barrier is needed.
template <int P, int K>
struct BOpStore {
    static constexpr int BYTES = 64 * (P == 0 ? 4 * Basis<P, K>::SLOTS : 16 * Basis<P, K>::NM);   // per operand and wave
};
template <int P, int K>
__device__ __forceinline__ void bop_put(char *slot, int lane, const BOp<P, K> &b, const float *eb) {
    if constexpr (P >= 1) {
        v4f *q = reinterpret_cast<v4f *>(slot) + lane;
#pragma unroll
        for (int i = 0; i < Basis<P, K>::NM; i++) q[64 * i] = __builtin_bit_cast(v4f, b.m[i]);
    } else {
        float *q = reinterpret_cast<float *>(slot) + lane;
#pragma unroll
        for (int s = 0; s < Basis<P, K>::SLOTS; s++) q[64 * s] = eb[s];
    }
}
template <int P, int K>
__device__ __forceinline__ void bop_get(const char *slot, int lane, BOp<P, K> &b) {
    if constexpr (P >= 1) {
        const v4f *q = reinterpret_cast<const v4f *>(slot) + lane;
#pragma unroll
        for (int i = 0; i < Basis<P, K>::NM; i++) b.m[i] = __builtin_bit_cast(v8bf, q[64 * i]);
    } else {
        const float *q = reinterpret_cast<const float *>(slot) + lane;
        float eb[Basis<P, K>::SLOTS];
#pragma unroll
        for (int s = 0; s < Basis<P, K>::SLOTS; s++) eb[s] = q[64 * s];
        b.set(eb, lane >> 4);
    }
}

// ---------------------------------------------------------------------------
// Forward message pass, one feature pass (blockIdx.y) per workgroup: the
// first layer, and models with a single pass.
// ---------------------------------------------------------------------------
template <int P, int F, int K, bool V0>
__global__ void __launch_bounds__(64 * MW) __attribute__((amdgpu_waves_per_eu(V0 ? FWD_WAVES0 : FWD_WAVES))) k_msg_fwd(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                     const float4 *__restrict__ geom, int n,
                                                     const float *__restrict__ phi, const float *__restrict__ uvp,
                                                     const float *__restrict__ s, const float *__restrict__ v,
                                                     const float *__restrict__ Aw,
                                                     const float *__restrict__ cw, float rc,
                                                     const int8_t *__restrict__ hop, int hop_max,
                                                     const int *__restrict__ zsp, int *__restrict__ queue,
                                                     float *__restrict__ sn, float *__restrict__ v1) {
    constexpr int WM = FWD_W;
    constexpr int F3 = 3 * F, SL = Basis<P, K>::SLOTS, W = Pass<F, WM>::W, TU = Pass<F, WM>::TU;
    __shared__ __attribute__((aligned(16))) char lds[WStage<P, F, K, WM>::BYTES];
    // first layer: phi and s are per-species tables (rows by zsp), a few rows
    // that every gather hits in L1, read directly in the accumulator layout
    __shared__ v4f xch[MW][V0 ? 1 : 5][64];
    const int p = blockIdx.y;
    stage_pass<P, F, K, WM>(Aw, cw, p, lds);
    const int lane = threadIdx.x & 63, e = lane & 15, g = lane >> 4;
    const int fo = p * W + 4 * g;   // first feature of this lane (tile u adds 16 u)
    const Xch xc(g, e);
    v4f(*xw)[64] = xch[threadIdx.x >> 6];
    const AtomQueue aq(n, queue, p);
    const float pirc = 3.14159265358979f / rc;
    MSG_ATOMS(aq, i) {
        const int e0 = rowc[i], e1 = rowc[i + 1];
        const int deg = hop[i] <= hop_max ? e1 - e0 : 0;
        v4f as[TU], av[3][TU];
#pragma unroll
        for (int u = 0; u < TU; u++) {
            as[u] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int d = 0; d < 3; d++) av[d][u] = v4f{0.f, 0.f, 0.f, 0.f};
        }
        // edge records of the next chunk are loaded one chunk ahead
        float4 gm_n = make_float4(0.f, 0.f, 0.f, rc);
        int j_n = i;
        if (e < deg) {
            gm_n = geom[e0 + e];
            j_n = colc[e0 + e];
        }
        for (int cb = 0; cb < deg; cb += 16) {
            const char *wl = lds_chunk(lds);
            const bool valid = cb + e < deg;
            const float4 gm = gm_n;
            const int j = j_n;
            gm_n = make_float4(0.f, 0.f, 0.f, rc);
            j_n = i;
            if (cb + 16 + e < deg) {
                gm_n = geom[e0 + cb + 16 + e];
                j_n = colc[e0 + cb + 16 + e];
            }
            // gathered: phi_s, phi_vs and (after the first layer) u = v * phi_vv
            // of the source (5 row slices, quarter-contiguously, then moved to
            // the accumulator layout; the first layer's 2 from the table)
            v4f ph[2][TU], uu[3][TU];
            if constexpr (V0) {
                const float *pj = phi + (long)zsp[j] * F3 + fo;
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    ph[0][u] = ld4(pj + F + 16 * u);
                    ph[1][u] = ld4(pj + 2 * F + 16 * u);
                }
            } else {
                const int jq = __shfl(j, xc.src, 64);
                const float *pj = phi + (long)jq * F3 + p * W + xc.fo;
                const float *uj = uvp + (long)jq * F3 + p * W + xc.fo;
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    ph[0][u] = ld4(pj + F + 16 * u);
                    ph[1][u] = ld4(pj + 2 * F + 16 * u);
#pragma unroll
                    for (int d = 0; d < 3; d++) uu[d][u] = ld4(uj + d * F + 16 * u);
                }
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    ph[0][u] = xc.move(xw[0], ph[0][u]);
                    ph[1][u] = xc.move(xw[1], ph[1][u]);
#pragma unroll
                    for (int d = 0; d < 3; d++) uu[d][u] = xc.move(xw[2 + d], uu[d][u]);
                }
            }
            const float ir = valid ? __builtin_amdgcn_rcpf(gm.w) : 0.f;
            float eb[SL];
            basis_slots<P, K, false>(gm.w, ir, pirc, valid, g, eb, nullptr);
            BOp<P, K> bop;
            bop.set(eb, g);
            const float rx = gm.x * ir, ry = gm.y * ir, rz = gm.z * ir;
#pragma unroll
            for (int u = 0; u < TU; u++) {
                v4f wvv;
                if constexpr (!V0) wvv = filter_tile<P, F, K, WM>(wl, u, bop, lane);
                const v4f ws = filter_tile<P, F, K, WM>(wl, TU + u, bop, lane);
                const v4f wvs = filter_tile<P, F, K, WM>(wl, 2 * TU + u, bop, lane);
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const float xvs = ph[1][u][r] * wvs[r];
                    as[u][r] = fmaf(ph[0][u][r], ws[r], as[u][r]);
                    if constexpr (V0) {
                        av[0][u][r] = fmaf(rx, xvs, av[0][u][r]);
                        av[1][u][r] = fmaf(ry, xvs, av[1][u][r]);
                        av[2][u][r] = fmaf(rz, xvs, av[2][u][r]);
                    } else {
                        av[0][u][r] = fmaf(uu[0][u][r], wvv[r], fmaf(rx, xvs, av[0][u][r]));
                        av[1][u][r] = fmaf(uu[1][u][r], wvv[r], fmaf(ry, xvs, av[1][u][r]));
                        av[2][u][r] = fmaf(uu[2][u][r], wvv[r], fmaf(rz, xvs, av[2][u][r]));
                    }
                }
            }
        }
        // sum over the 16 edge lanes of each row
#pragma unroll
        for (int u = 0; u < TU; u++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                as[u][r] = row_sum16(as[u][r]);
#pragma unroll
                for (int d = 0; d < 3; d++) av[d][u][r] = row_sum16(av[d][u][r]);
            }
        if (e == 0) {
#pragma unroll
            for (int u = 0; u < TU; u++) {
                const int f = fo + 16 * u;
                const long si = V0 ? (long)zsp[i] : (long)i;
                st4(sn + (long)i * 2 * F + f, ld4(s + si * F + f) + as[u]);
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    if constexpr (V0) st4(v1 + (long)i * F3 + d * F + f, av[d][u]);
                    else st4(v1 + (long)i * F3 + d * F + f, ld4(v + (long)i * F3 + d * F + f) + av[d][u]);
                }
            }
        }
    }
}

// What a lane needs of the edges 4g .. 4g+3 of a chunk (the layout of the
// transposed tiles), kept in the wave's LDS through the passes: per edge the
// direction and the row of the other atom.  The lanes of group 0 write it once;
// lane shuffles would move four values per edge in every pass.
typedef v4f EdgeRec;
constexpr int EREC_BYTES = 16 * sizeof(EdgeRec);
__device__ __forceinline__ void edge_rec_put(char *slot, int e, int g, float hx, float hy, float hz, int row) {
    if (g == 0) reinterpret_cast<EdgeRec *>(slot)[e] = EdgeRec{hx, hy, hz, __int_as_float(row)};
    __builtin_amdgcn_wave_barrier();   // the reads see the wave's writes
}
__device__ __forceinline__ EdgeRec edge_rec_get(const char *slot, int k) { return reinterpret_cast<const EdgeRec *>(slot)[k]; }

// Element f of row i of an array of ld floats per row: with a 32-bit byte
// offset from the (uniform) base where the array ends below 4 GB (one
// multiply-add per row instead of a 64-bit one per row and array).
template <bool WIDE>
struct RowAt {
    size_t o;
    __device__ __forceinline__ RowAt(int i, int ld, int f) {
        if constexpr (WIDE) o = 4 * ((size_t)i * ld + f);
        else o = (unsigned)__umul24(i, 4 * ld) + 4u * f;
    }
    __device__ __forceinline__ float at(const float *a, int k) const {
        if constexpr (WIDE) return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a) + o + 4 * k);
        else return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(a) + 4 * k + (unsigned)o);
    }
};
inline bool msg_wide(long n, int F) { return n >= (1 << 24) || n * 12 * F > 0xFFFFFFFFL; }

// ---------------------------------------------------------------------------
// Forward message pass of the layers after the first with more than one
// feature pass: every wave runs all passes of its atom, with the weight
// images of every pass in LDS, and the radial basis of a chunk, in MFMA
// operand form, is evaluated in the first pass and kept in the wave's LDS for
// the later ones (the first NC chunks of the atom: FWD_CACHE, or as many as
// FP32's four weight tables of 128 features leave LDS for).  The filter tiles
// come out transposed (filter_tile with TR): lane (f, g) holds feature f of
// the tile for the edges 4g .. 4g+3, so it gathers 16 consecutive features
// of one source row per quarter-wave and register (no exchange), adds its
// four edges in registers, and the sums over the atom's edges need only a
// sum over the four lane rows at the end.  The basis is evaluated in the
// layout the MFMA operand takes (lane (e, g): slots of edge e); the source
// row and direction of the edges 4g + r are read from the wave's edge records
// (EdgeRec), written once per chunk.
// ---------------------------------------------------------------------------
#ifndef FWD_PIW_WAVES
#define FWD_PIW_WAVES 16
#endif
#ifndef FWD_CACHE
#define FWD_CACHE 3
#endif
template <int P, int F, int K, bool WIDE>
__global__ void __launch_bounds__(64 * FWD_PIW_WAVES) __attribute__((amdgpu_waves_per_eu(FWD_WAVES))) k_msg_fwd_pw(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                     const float4 *__restrict__ geom, int n,
                                                     const float *__restrict__ phi, const float *__restrict__ uvp,
                                                     const float *__restrict__ s, const float *__restrict__ v,
                                                     const float *__restrict__ Aw,
                                                     const float *__restrict__ cw, float rc,
                                                     const int8_t *__restrict__ hop, int hop_max,
                                                     int *__restrict__ queue,
                                                     float *__restrict__ sn, float *__restrict__ v1) {
    constexpr int WM = FWD_W;
    constexpr int F3 = 3 * F, SL = Basis<P, K>::SLOTS, W = Pass<F, WM>::W, TU = Pass<F, WM>::TU;
    constexpr int NP = Pass<F, WM>::N, NC = P == 0 && F == 128 ? 2 : FWD_CACHE;
    constexpr int WB = WStage<P, F, K, WM, true>::BYTES;
    constexpr int CB = BOpStore<P, K>::BYTES;
    __shared__ __attribute__((aligned(16))) char lds[NP * WB];
    __shared__ __attribute__((aligned(16))) char bcache[FWD_PIW_WAVES * NC * CB];
    __shared__ __attribute__((aligned(16))) char ecache[FWD_PIW_WAVES * (NC + 1) * EREC_BYTES];
    // all passes, or (gridDim.y = NP) the one of blockIdx.y
    const int p0 = gridDim.y > 1 ? blockIdx.y : 0, p1 = gridDim.y > 1 ? p0 + 1 : NP;
#pragma unroll 1
    for (int q = p0; q < p1; q++) stage_pass<P, F, K, WM, true>(Aw, cw, q, lds + q * WB);
    const int lane = threadIdx.x & 63, e = lane & 15, g = lane >> 4;
    char *bc = bcache + (threadIdx.x >> 6) * NC * CB, *ec = ecache + (threadIdx.x >> 6) * (NC + 1) * EREC_BYTES;
    const AtomQueue aq(n, queue, p0);
    const float pirc = 3.14159265358979f / rc;
    MSG_ATOMS(aq, i) {
        const int e0 = rowc[i], e1 = rowc[i + 1];
        const int deg = hop[i] <= hop_max ? e1 - e0 : 0;
#pragma unroll 1
        for (int p = p0; p < p1; p++) {
            const int fl = p * W + e;   // this lane's feature (tile u adds 16 u)
            float as[TU], av[3][TU];
#pragma unroll
            for (int u = 0; u < TU; u++) {
                as[u] = 0.f;
#pragma unroll
                for (int d = 0; d < 3; d++) av[d][u] = 0.f;
            }
            // edge records (edge e of the chunk) are loaded one chunk ahead,
            // where the chunk is not at hand from the first pass
            float4 gm_n = make_float4(0.f, 0.f, 0.f, rc);
            int j_n = i;
            if (p == p0 && e < deg) {
                gm_n = geom[e0 + e];
                j_n = colc[e0 + e];
            }
            for (int cb = 0; cb < deg; cb += 16) {
                const char *wl = lds_chunk(lds + p * WB);
                const int c = cb >> 4;
                const bool kept = p > p0 && c < NC;
                char *er = ec + min(c, NC) * EREC_BYTES;
                const bool valid = cb + e < deg;
                const float4 gm = gm_n;
                const float ir = valid ? __builtin_amdgcn_rcpf(gm.w) : 0.f;
                // source rows and directions of the chunk's edges (padding edges:
                // the atom's own row and a zero direction; their filter is 0)
                if (!kept) edge_rec_put(er, e, g, gm.x * ir, gm.y * ir, gm.z * ir, j_n);
                if (p == p0 || c + 1 >= NC) {
                    gm_n = make_float4(0.f, 0.f, 0.f, rc);
                    j_n = i;
                    if (cb + 16 + e < deg) {
                        gm_n = geom[e0 + cb + 16 + e];
                        j_n = colc[e0 + cb + 16 + e];
                    }
                }
                float ps[TU][4], pv[TU][4], uu[3][TU][4], hx[4], hy[4], hz[4];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const EdgeRec h = edge_rec_get(er, 4 * g + r);
                    hx[r] = h[0], hy[r] = h[1], hz[r] = h[2];
                    const RowAt<WIDE> row(__float_as_int(h[3]), F3, fl);
#pragma unroll
                    for (int u = 0; u < TU; u++) {
                        ps[u][r] = row.at(phi, F + 16 * u);
                        pv[u][r] = row.at(phi, 2 * F + 16 * u);
#pragma unroll
                        for (int d = 0; d < 3; d++) uu[d][u][r] = row.at(uvp, d * F + 16 * u);
                    }
                }
                BOp<P, K> bop;
                if (kept) {
                    bop_get<P, K>(bc + c * CB, lane, bop);
                } else {
                    float eb[SL];
                    basis_slots<P, K, false>(gm.w, ir, pirc, valid, g, eb, nullptr);
                    bop.set(eb, g);
                    if (p == p0 && c < NC) bop_put<P, K>(bc + c * CB, lane, bop, eb);
                }
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    const v4f wvv = filter_tile<P, F, K, WM, true, true>(wl, u, bop, lane);
                    const v4f ws = filter_tile<P, F, K, WM, true, true>(wl, TU + u, bop, lane);
                    const v4f wvs = filter_tile<P, F, K, WM, true, true>(wl, 2 * TU + u, bop, lane);
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const float xvs = pv[u][r] * wvs[r];
                        as[u] = fmaf(ps[u][r], ws[r], as[u]);
                        av[0][u] = fmaf(uu[0][u][r], wvv[r], fmaf(hx[r], xvs, av[0][u]));
                        av[1][u] = fmaf(uu[1][u][r], wvv[r], fmaf(hy[r], xvs, av[1][u]));
                        av[2][u] = fmaf(uu[2][u][r], wvv[r], fmaf(hz[r], xvs, av[2][u]));
                    }
                }
            }
            // sum over the four lane rows (edges 4g .. 4g+3 of every chunk)
#pragma unroll
            for (int u = 0; u < TU; u++) {
                as[u] += __shfl_xor(as[u], 16, 64);
                as[u] += __shfl_xor(as[u], 32, 64);
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    av[d][u] += __shfl_xor(av[d][u], 16, 64);
                    av[d][u] += __shfl_xor(av[d][u], 32, 64);
                }
            }
            if (g == 0) {
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    const int f = fl + 16 * u;
                    sn[(long)i * 2 * F + f] = s[(long)i * F + f] + as[u];
#pragma unroll
                    for (int d = 0; d < 3; d++)
                        v1[(long)i * F3 + d * F + f] = v[(long)i * F3 + d * F + f] + av[d][u];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Adjoint of the message pass, one feature pass (blockIdx.y) per workgroup:
// the first layer, and models with a single pass.
// Per chunk of 16 in-edges (j <- i) of the source atom j: the filter tiles and
// their radial derivatives on MFMA, the destinations' gradient pieces
// gathered per lane, dE/dphi_j and dE/dv_j accumulated in registers, and the
// edge sums S = (dE/dr, dE/drhat) of the pass stored in the pass's slot.
// ---------------------------------------------------------------------------
template <int P, int F, int K, bool V0>
__global__ void __launch_bounds__(64 * MW) __attribute__((amdgpu_waves_per_eu(V0 ? BWD_WAVES0 : BWD_WAVES))) k_msg_bwd(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                     const float4 *__restrict__ geom, int n,
                                                     const float *__restrict__ phi, const float *__restrict__ v,
                                                     const float *__restrict__ gs1, const float *__restrict__ gv1,
                                                     const float *__restrict__ Aw, const float *__restrict__ cw,
                                                     float rc, const int8_t *__restrict__ hop, int hop_max,
                                                     const int *__restrict__ zsp, int *__restrict__ queue,
                                                     float *__restrict__ gv_in, float *__restrict__ gphi,
                                                     float4 *__restrict__ S, long s_stride) {
    constexpr int WM = BWD_W;
    constexpr int F3 = 3 * F, SL = Basis<P, K>::SLOTS, W = Pass<F, WM>::W, TU = Pass<F, WM>::TU;
    __shared__ __attribute__((aligned(16))) char lds[WStage<P, F, K, WM>::BYTES];
    __shared__ v4f xch[MW][4][64];
    const int p = blockIdx.y;
    stage_pass<P, F, K, WM>(Aw, cw, p, lds);
    float4 *Sp = S + (long)p * s_stride;
    const int lane = threadIdx.x & 63, e = lane & 15, g = lane >> 4;
    const int fo = p * W + 4 * g;
    const Xch xc(g, e);
    v4f(*xw)[64] = xch[threadIdx.x >> 6];
    const AtomQueue aq(n, queue, p);
    const float pirc = 3.14159265358979f / rc;
    MSG_ATOMS(aq, j) {
        const int e0 = rowc[j], e1 = rowc[j + 1];
        const int deg = hop[j] <= hop_max ? e1 - e0 : 0;
        // first layer: v_j = 0 and no node gradient, so phi_vv, v_j, dE/dphi_j
        // and dE/dv_j drop out and only the edge sums remain.
        // Later layers accumulate Y_d = sum_e dE/dv1_d(i) w_vv (from which both
        // dE/dv_j = phi_vv Y_d and dE/dphi_vv = sum_d v_jd Y_d follow once per
        // atom), dE/dphi_s and dE/dphi_vs; the v_j term of dE/dr enters through
        // c_d = v_jd phi_vv.
        v4f ph[3][TU], cv[3][TU], Y[3][TU], ap[2][TU];
#pragma unroll
        for (int u = 0; u < TU; u++) {
#pragma unroll
            for (int q = V0 ? 1 : 0; q < 3; q++) ph[q][u] = ld4(phi + (V0 ? (long)zsp[j] : (long)j) * F3 + q * F + fo + 16 * u);
            if constexpr (!V0) {
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    cv[d][u] = ld4(v + (long)j * F3 + d * F + fo + 16 * u) * ph[0][u];
                    Y[d][u] = v4f{0.f, 0.f, 0.f, 0.f};
                }
                ap[0][u] = v4f{0.f, 0.f, 0.f, 0.f};
                ap[1][u] = v4f{0.f, 0.f, 0.f, 0.f};
            }
        }
        // edges of an atom beyond the hop range carry no gradient in this layer
        if (hop[j] > hop_max)
            for (int q = e0 + lane; q < e1; q += 64) Sp[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 gm_n = make_float4(0.f, 0.f, 0.f, rc);
        int i_n = j;
        if (e < deg) {
            gm_n = geom[e0 + e];
            i_n = colc[e0 + e];
        }
        for (int cb = 0; cb < deg; cb += 16) {
            const char *wl = lds_chunk(lds);
            const bool valid = cb + e < deg;
            const float4 gm = gm_n;
            const int i = i_n;
            gm_n = make_float4(0.f, 0.f, 0.f, rc);
            i_n = j;
            if (cb + 16 + e < deg) {
                gm_n = geom[e0 + cb + 16 + e];
                i_n = colc[e0 + cb + 16 + e];
            }
            // the destinations' gradient rows, gathered quarter-contiguously and
            // moved to the accumulator layout
            const int iq = __shfl(i, xc.src, 64);
            v4f gs[TU], gv[3][TU];
#pragma unroll
            for (int u = 0; u < TU; u++) {
                gs[u] = ld4(gs1 + (long)iq * F + p * W + xc.fo + 16 * u);
#pragma unroll
                for (int d = 0; d < 3; d++) gv[d][u] = ld4(gv1 + (long)iq * F3 + d * F + p * W + xc.fo + 16 * u);
            }
#pragma unroll
            for (int u = 0; u < TU; u++) {
                gs[u] = xc.move(xw[0], gs[u]);
#pragma unroll
                for (int d = 0; d < 3; d++) gv[d][u] = xc.move(xw[1 + d], gv[d][u]);
            }
            const float ir = valid ? __builtin_amdgcn_rcpf(gm.w) : 0.f;
            float eb[SL], db[SL];
            basis_slots<P, K, true>(gm.w, ir, pirc, valid, g, eb, db);
            BOp<P, K> bop, dop;
            bop.set(eb, g);
            dop.set(db, g);
            // direction of the message edge (i <- j) is x_j - x_i = -(x_i - x_j)
            const float rx = -gm.x * ir, ry = -gm.y * ir, rz = -gm.z * ir;
            float sr = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll
            for (int u = 0; u < TU; u++) {
                v4f w0, w1, d0;
                if constexpr (!V0) {
                    w0 = filter_tile<P, F, K, WM>(wl, u, bop, lane);
                    w1 = filter_tile<P, F, K, WM>(wl, TU + u, bop, lane);
                }
                const v4f w2 = filter_tile<P, F, K, WM>(wl, 2 * TU + u, bop, lane);
                if constexpr (!V0) d0 = filter_tile<P, F, K, WM>(wl, u, dop, lane);
                const v4f d1 = filter_tile<P, F, K, WM>(wl, TU + u, dop, lane);
                const v4f d2 = filter_tile<P, F, K, WM>(wl, 2 * TU + u, dop, lane);
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const float ga = gv[0][u][r], gb = gv[1][u][r], gc = gv[2][u][r], gsr = gs[u][r];
                    const float gxvs = fmaf(ga, rx, fmaf(gb, ry, gc * rz));
                    const float xvs = ph[2][u][r] * w2[r];
                    sx = fmaf(ga, xvs, sx);
                    sy = fmaf(gb, xvs, sy);
                    sz = fmaf(gc, xvs, sz);
                    if constexpr (V0) {
                        sr = fmaf(gsr * ph[1][u][r], d1[r], fmaf(gxvs * ph[2][u][r], d2[r], sr));
                        continue;
                    }
                    const float gc0 = fmaf(ga, cv[0][u][r], fmaf(gb, cv[1][u][r], gc * cv[2][u][r]));
                    Y[0][u][r] = fmaf(ga, w0[r], Y[0][u][r]);
                    Y[1][u][r] = fmaf(gb, w0[r], Y[1][u][r]);
                    Y[2][u][r] = fmaf(gc, w0[r], Y[2][u][r]);
                    ap[0][u][r] = fmaf(gsr, w1[r], ap[0][u][r]);
                    ap[1][u][r] = fmaf(gxvs, w2[r], ap[1][u][r]);
                    sr = fmaf(gc0, d0[r], fmaf(gsr * ph[1][u][r], d1[r], fmaf(gxvs * ph[2][u][r], d2[r], sr)));
                }
            }
            // sum over the four lane rows (all features of the pass)
            sr += __shfl_xor(sr, 16, 64);
            sx += __shfl_xor(sx, 16, 64);
            sy += __shfl_xor(sy, 16, 64);
            sz += __shfl_xor(sz, 16, 64);
            sr += __shfl_xor(sr, 32, 64);
            sx += __shfl_xor(sx, 32, 64);
            sy += __shfl_xor(sy, 32, 64);
            sz += __shfl_xor(sz, 32, 64);
            if (g == 0 && valid) Sp[e0 + cb + e] = make_float4(sr, sx, sy, sz);
        }
        if constexpr (V0) continue;
        // sum over the 16 edge lanes of each row
#pragma unroll
        for (int u = 0; u < TU; u++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
#pragma unroll
                for (int d = 0; d < 3; d++) Y[d][u][r] = row_sum16(Y[d][u][r]);
                ap[0][u][r] = row_sum16(ap[0][u][r]);
                ap[1][u][r] = row_sum16(ap[1][u][r]);
            }
        if (e == 0) {
#pragma unroll
            for (int u = 0; u < TU; u++) {
                const long b = (long)j * F3 + fo + 16 * u;
                const v4f pvv = ld4(phi + b);
                v4f gvv = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    gvv += ld4(v + b + d * F) * Y[d][u];
                    st4(gv_in + b + d * F, ld4(gv1 + b + d * F) + pvv * Y[d][u]);
                }
                st4(gphi + b, gvv);
                st4(gphi + b + F, ap[0][u]);
                st4(gphi + b + 2 * F, ap[1][u]);
            }
        }
    }
}

// One stage of a reduce-scatter over the 16 lanes of a row: lane e keeps the
// half of x[0 .. 2H) its bit selects (U) and adds the partner's copy of it,
// which the DPP pattern CTRL brings (the partner's bit is the opposite one).
template <int CTRL, int H>
__device__ __forceinline__ void rs_half(float *x, bool U) {
#pragma unroll
    for (int k = 0; k < H; k++) {
        const float send = U ? x[k] : x[k + H], keep = U ? x[k + H] : x[k];
        x[k] = keep + dpp<CTRL>(send);
    }
}
// Sums of x[0 .. 16) over the 16 lanes of each row; lane e of the row
// receives the sum of x[e].
__device__ __forceinline__ float row_reduce_scatter16(float *x, int e) {
    rs_half<0x140, 8>(x, e & 8);   // row_mirror: e <-> 15 - e
    rs_half<0x141, 4>(x, e & 4);   // row_half_mirror: e <-> 7 - e inside each half
    rs_half<0x1B, 2>(x, e & 2);    // quad_perm [3,2,1,0]: e <-> e ^ 3
    rs_half<0xB1, 1>(x, e & 1);    // quad_perm [1,0,3,2]: e <-> e ^ 1
    return x[0];
}

// ---------------------------------------------------------------------------
// Adjoint of the message pass of the layers after the first with more than
// one feature pass, organised like k_msg_fwd_pw: every wave runs all passes
// of its source atom j with the weight images of every pass in LDS; the
// radial basis and its derivative of a chunk, in MFMA operand form, are
// evaluated in the first pass and kept in the wave's LDS for the later ones
// (the first BWD_CACHE chunks); the filter tiles come out transposed, so
// lane (f, g) works on feature f of the tile for the in-edges 4g .. 4g+3:
// it gathers the destinations' gradient rows 16 consecutive features per
// quarter-wave, accumulates dE/dphi_j and dE/dv_j over its edges in
// registers (summed over the four lane rows once per atom and pass), and
// holds per-edge partial sums over its feature, which a reduce-scatter over
// the 16 lanes of the row turns into the 16 values (4 edges x (dE/dr,
// dE/drhat)) that the row stores as 64 contiguous bytes.  The edge sums of
// the passes are added up in the wave, in pass order (in LDS for the cached
// chunks, in the slot itself for the others: the lane that adds is the lane
// that stored), so the layer has one slot.
// ---------------------------------------------------------------------------
#ifndef BWD_PIW_WAVES
#define BWD_PIW_WAVES 8
#endif
#ifndef BWD_PIW_EU
#define BWD_PIW_EU 2
#endif
#ifndef BWD_CACHE
#define BWD_CACHE 3
#endif
template <int P, int F, int K, bool WIDE>
__global__ void __launch_bounds__(64 * BWD_PIW_WAVES) __attribute__((amdgpu_waves_per_eu(BWD_PIW_EU))) k_msg_bwd_pw(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                     const float4 *__restrict__ geom, int n,
                                                     const float *__restrict__ phi, const float *__restrict__ v,
                                                     const float *__restrict__ gs1, const float *__restrict__ gv1,
                                                     const float *__restrict__ Aw, const float *__restrict__ cw,
                                                     float rc, const int8_t *__restrict__ hop, int hop_max,
                                                     int *__restrict__ queue,
                                                     float *__restrict__ gv_in, float *__restrict__ gphi,
                                                     float4 *__restrict__ S) {
    constexpr int WM = BWD_W;
    constexpr int F3 = 3 * F, SL = Basis<P, K>::SLOTS, W = Pass<F, WM>::W, TU = Pass<F, WM>::TU;
    constexpr int NP = Pass<F, WM>::N, NC = P == 0 && F == 128 ? 2 : BWD_CACHE;
    constexpr int WB = WStage<P, F, K, WM, true>::BYTES;
    constexpr int CB = 2 * BOpStore<P, K>::BYTES;       // basis and derivative of a chunk
    __shared__ __attribute__((aligned(16))) char lds[NP * WB];
    __shared__ __attribute__((aligned(16))) char bcache[BWD_PIW_WAVES * NC * CB];
    __shared__ __attribute__((aligned(16))) char ecache[BWD_PIW_WAVES * (NC + 1) * EREC_BYTES];
    __shared__ float sacc[BWD_PIW_WAVES][NC][64];       // edge sums of the cached chunks
#pragma unroll 1
    for (int q = 0; q < NP; q++) stage_pass<P, F, K, WM, true>(Aw, cw, q, lds + q * WB);
    const int lane = threadIdx.x & 63, e = lane & 15, g = lane >> 4;
    char *bc = bcache + (threadIdx.x >> 6) * NC * CB, *ec = ecache + (threadIdx.x >> 6) * (NC + 1) * EREC_BYTES;
    float *Sf = reinterpret_cast<float *>(S);
    const AtomQueue aq(n, queue, 0);
    const float pirc = 3.14159265358979f / rc;
    MSG_ATOMS_AHEAD(aq, j) {
        const int e0 = rowc[j], e1 = rowc[j + 1];
        const int deg = hop[j] <= hop_max ? e1 - e0 : 0;
        // edges of an atom beyond the hop range carry no gradient in this layer
        if (hop[j] > hop_max)
            for (int t = e0 + lane; t < e1; t += 64) S[t] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
        for (int p = 0; p < NP; p++) {
            const int fl = p * W + e;   // this lane's feature (tile u adds 16 u)
            // Y_d = sum_e dE/dv1_d(i) w_vv (dE/dv_j = phi_vv Y_d and dE/dphi_vv =
            // sum_d v_jd Y_d follow once per atom), dE/dphi_s, dE/dphi_vs; the v_j
            // term of dE/dr enters through c_d = v_jd phi_vv
            float ph[3][TU], cv[3][TU], Y[3][TU], ap[2][TU];
#pragma unroll
            for (int u = 0; u < TU; u++) {
#pragma unroll
                for (int q = 0; q < 3; q++) ph[q][u] = phi[(long)j * F3 + q * F + fl + 16 * u];
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    cv[d][u] = v[(long)j * F3 + d * F + fl + 16 * u] * ph[0][u];
                    Y[d][u] = 0.f;
                }
                ap[0][u] = 0.f;
                ap[1][u] = 0.f;
            }
            float4 gm_n = make_float4(0.f, 0.f, 0.f, rc);
            int i_n = j;
            if (p == 0 && e < deg) {
                gm_n = geom[e0 + e];
                i_n = colc[e0 + e];
            }
            for (int cb = 0; cb < deg; cb += 16) {
                const char *wl = lds_chunk(lds + p * WB);
                const int c = cb >> 4;
                const bool kept = p > 0 && c < NC;
                char *er = ec + min(c, NC) * EREC_BYTES;
                const bool valid = cb + e < deg;
                const float4 gm = gm_n;
                const float ir = valid ? __builtin_amdgcn_rcpf(gm.w) : 0.f;
                // destinations and directions of the chunk's edges (the direction
                // of the message edge (i <- j) is x_j - x_i = -(x_i - x_j); padding
                // edges: the atom itself and a zero direction; their filter is 0)
                if (!kept) edge_rec_put(er, e, g, -gm.x * ir, -gm.y * ir, -gm.z * ir, i_n);
                if (p == 0 || c + 1 >= NC) {
                    gm_n = make_float4(0.f, 0.f, 0.f, rc);
                    i_n = j;
                    if (cb + 16 + e < deg) {
                        gm_n = geom[e0 + cb + 16 + e];
                        i_n = colc[e0 + cb + 16 + e];
                    }
                }
                float gs[TU][4], gv[3][TU][4], hx[4], hy[4], hz[4];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const EdgeRec h = edge_rec_get(er, 4 * g + r);
                    hx[r] = h[0], hy[r] = h[1], hz[r] = h[2];
                    const RowAt<WIDE> rs(__float_as_int(h[3]), F, fl), rv(__float_as_int(h[3]), F3, fl);
#pragma unroll
                    for (int u = 0; u < TU; u++) {
                        gs[u][r] = rs.at(gs1, 16 * u);
#pragma unroll
                        for (int d = 0; d < 3; d++) gv[d][u][r] = rv.at(gv1, d * F + 16 * u);
                    }
                }
                BOp<P, K> bop, dop;
                if (kept) {
                    bop_get<P, K>(bc + c * CB, lane, bop);
                    bop_get<P, K>(bc + c * CB + CB / 2, lane, dop);
                } else {
                    float eb[SL], db[SL];
                    basis_slots<P, K, true>(gm.w, ir, pirc, valid, g, eb, db);
                    bop.set(eb, g);
                    dop.set(db, g);
                    if (p == 0 && c < NC) {
                        bop_put<P, K>(bc + c * CB, lane, bop, eb);
                        bop_put<P, K>(bc + c * CB + CB / 2, lane, dop, db);
                    }
                }
                // per edge r: (dE/dr, dE/drhat_x, _y, _z) of this lane's feature
                float es[16];
#pragma unroll
                for (int k = 0; k < 16; k++) es[k] = 0.f;
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    const v4f w0 = filter_tile<P, F, K, WM, true, true>(wl, u, bop, lane);
                    const v4f w1 = filter_tile<P, F, K, WM, true, true>(wl, TU + u, bop, lane);
                    const v4f w2 = filter_tile<P, F, K, WM, true, true>(wl, 2 * TU + u, bop, lane);
                    const v4f d0 = filter_tile<P, F, K, WM, true, true>(wl, u, dop, lane);
                    const v4f d1 = filter_tile<P, F, K, WM, true, true>(wl, TU + u, dop, lane);
                    const v4f d2 = filter_tile<P, F, K, WM, true, true>(wl, 2 * TU + u, dop, lane);
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const float ga = gv[0][u][r], gb = gv[1][u][r], gc = gv[2][u][r], gsr = gs[u][r];
                        const float gxvs = fmaf(ga, hx[r], fmaf(gb, hy[r], gc * hz[r]));
                        const float xvs = ph[2][u] * w2[r];
                        es[4 * r + 1] = fmaf(ga, xvs, es[4 * r + 1]);
                        es[4 * r + 2] = fmaf(gb, xvs, es[4 * r + 2]);
                        es[4 * r + 3] = fmaf(gc, xvs, es[4 * r + 3]);
                        const float gc0 = fmaf(ga, cv[0][u], fmaf(gb, cv[1][u], gc * cv[2][u]));
                        Y[0][u] = fmaf(ga, w0[r], Y[0][u]);
                        Y[1][u] = fmaf(gb, w0[r], Y[1][u]);
                        Y[2][u] = fmaf(gc, w0[r], Y[2][u]);
                        ap[0][u] = fmaf(gsr, w1[r], ap[0][u]);
                        ap[1][u] = fmaf(gxvs, w2[r], ap[1][u]);
                        es[4 * r] = fmaf(gc0, d0[r], fmaf(gsr * ph[1][u], d1[r], fmaf(gxvs * ph[2][u], d2[r], es[4 * r])));
                    }
                }
                // lane e of row g receives component e & 3 of edge 4g + (e >> 2),
                // summed over the pass's features
                float o = row_reduce_scatter16(es, e);
                const int ke = cb + 4 * g + (e >> 2);   // the edge this lane stores
                if (ke < deg) {
                    float *acc = c < NC ? &sacc[threadIdx.x >> 6][c][lane] : Sf + 4L * (e0 + cb + 4 * g) + e;
                    if (p > 0) o += *acc;
                    if (c < NC && p + 1 < NP) *acc = o;
                    else Sf[4L * (e0 + cb + 4 * g) + e] = o;
                }
            }
            // sum over the four lane rows
#pragma unroll
            for (int u = 0; u < TU; u++) {
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    Y[d][u] += __shfl_xor(Y[d][u], 16, 64);
                    Y[d][u] += __shfl_xor(Y[d][u], 32, 64);
                }
                ap[0][u] += __shfl_xor(ap[0][u], 16, 64);
                ap[0][u] += __shfl_xor(ap[0][u], 32, 64);
                ap[1][u] += __shfl_xor(ap[1][u], 16, 64);
                ap[1][u] += __shfl_xor(ap[1][u], 32, 64);
            }
            if (g == 0) {
#pragma unroll
                for (int u = 0; u < TU; u++) {
                    const long b = (long)j * F3 + fl + 16 * u;
                    float gvv = 0.f;
#pragma unroll
                    for (int d = 0; d < 3; d++) {
                        gvv = fmaf(v[b + d * F], Y[d][u], gvv);
                        gv_in[b + d * F] = fmaf(ph[0][u], Y[d][u], gv1[b + d * F]);
                    }
                    gphi[b] = gvv;
                    gphi[b + F] = ap[0][u];
                    gphi[b + 2 * F] = ap[1][u];
                }
            }
        }
    }
}

// G of each pruned edge from its edge-sum slots: G = dE/dr rhat + (g - (g . rhat) rhat) / r,
// with rhat the direction of the message edge, the reverse of the stored one.
// The pruned edge count is rowc[n], read on the device.
__global__ void k_assemble_G(const int *__restrict__ rowc, int n, const float4 *__restrict__ geom,
                             const float4 *__restrict__ S, long s_stride, int npass, float4 *__restrict__ G) {
    const long ne = rowc[n];
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += (long)gridDim.x * blockDim.x) {
        float4 a = S[e];
        for (int p = 1; p < npass; p++) {
            const float4 b = S[(long)p * s_stride + e];
            a.x += b.x;
            a.y += b.y;
            a.z += b.z;
            a.w += b.w;
        }
        const float4 gm = geom[e];
        const float ir = 1.0f / gm.w;
        const float rx = -gm.x * ir, ry = -gm.y * ir, rz = -gm.z * ir;
        const float rd = a.y * rx + a.z * ry + a.w * rz;
        G[e] = make_float4(a.x * rx + (a.y - rd * rx) * ir, a.x * ry + (a.z - rd * ry) * ir,
                           a.x * rz + (a.w - rd * rz) * ir, 0.f);
    }
}

// ---------------------------------------------------------------------------
// First layer, factorised.  There v = 0 and phi_j = phi(Z_j) depends on the
// species alone, while the messages are linear in the radial basis e~, so the
// sums over neighbours collapse to per-atom, per-species basis sums:
//   s1_i = s0(Z_i) + sum_Z phi_s(Z) o (A'_s P_i^Z),    P_i^Z   = sum_{j: Z_j = Z} e~(r_ij),
//   v1_i = sum_Z phi_vs(Z) o (A'_vs R_i^{Z,d}),        R_i^{Z,d} = sum_{j: Z_j = Z} rhat_ij,d e~(r_ij),
// and the adjoint's edge sums of the message edge (i <- j) need only the
// per-atom vectors Q_s[i][Z] = A'_s^T (gs1_i o phi_s(Z)) and
// Q_d[i][Z] = A'_vs^T (gv1_i,d o phi_vs(Z)):
//   dE/dr = de~ . (Q_s + sum_d rhat_d Q_d),   dE/drhat_d = e~ . Q_d.
// The products with the species-scaled filter weights (phi(Z) o A') are node
// GEMMs; the two kernels below do the O(K) work per edge.  Each species has
// a block of SB = l0_block(K) columns (slot k at Z SB + k; slots past K meet
// zero weights).  Rows of P: the S SB basis sums, then the species one-hot
// (column S SB + Z), which picks s0(Z_i) out of the same GEMM; rows 3 i + d
// of R and of Q_v, rows i of Q_s: the S SB slot columns.  Lane (g, e) = 16 g + e
// holds basis slots k = 8 g .. 8 g + 7 of edge e, as in the kernels above.
// ---------------------------------------------------------------------------
template <int K, int SS>
__global__ void __launch_bounds__(256) k_l0_basis_sums(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                       const float4 *__restrict__ geom, int n, float rc,
                                                       const int8_t *__restrict__ hop, int hop_max,
                                                       const int *__restrict__ zsp, float *__restrict__ P, int ldp,
                                                       float *__restrict__ R, int ldr) {
    constexpr int SB = l0_block(K);
    const int lane = threadIdx.x & 63, e = lane & 15, g = lane >> 4;
    const float pirc = 3.14159265358979f / rc;
    const int nw = (int)(gridDim.x * (blockDim.x >> 6));
    for (int i = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); i < n; i += nw) {
        const int e0 = rowc[i], e1 = rowc[i + 1];
        const int deg = hop[i] <= hop_max ? e1 - e0 : 0;
        float acc[SS][4][8];
#pragma unroll
        for (int z = 0; z < SS; z++)
#pragma unroll
            for (int t = 0; t < 4; t++)
#pragma unroll
                for (int q = 0; q < 8; q++) acc[z][t][q] = 0.f;
        for (int cb = 0; cb < deg; cb += 16) {
            const bool valid = cb + e < deg;
            float4 gm = make_float4(0.f, 0.f, 0.f, rc);
            int z = 0;
            if (valid) {
                gm = geom[e0 + cb + e];
                z = zsp[colc[e0 + cb + e]];
            }
            const float ir = valid ? __builtin_amdgcn_rcpf(gm.w) : 0.f;
            float eb[8];
            basis_slots<1, K, false>(gm.w, ir, pirc, valid, g, eb, nullptr);
            const float wt[4] = {1.f, gm.x * ir, gm.y * ir, gm.z * ir};
#pragma unroll
            for (int zz = 0; zz < SS; zz++) {
                const bool on = z == zz;
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const float w = on ? wt[t] : 0.f;
#pragma unroll
                    for (int q = 0; q < 8; q++) acc[zz][t][q] = fmaf(w, eb[q], acc[zz][t][q]);
                }
            }
        }
#pragma unroll
        for (int zz = 0; zz < SS; zz++)
#pragma unroll
            for (int t = 0; t < 4; t++)
#pragma unroll
                for (int q = 0; q < 8; q++) acc[zz][t][q] = row_sum16(acc[zz][t][q]);
        // lane row g holds the totals of slots 8 g .. 8 g + 7 (rows past the
        // species block are not stored; slots past K meet zero weights)
        if (e == 0 && 8 * g < SB) {
#pragma unroll
            for (int zz = 0; zz < SS; zz++)
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    float *dst = t == 0 ? P + (long)i * ldp : R + (3L * i + t - 1) * ldr;
                    dst += zz * SB + 8 * g;
                    st4(dst, v4f{acc[zz][t][0], acc[zz][t][1], acc[zz][t][2], acc[zz][t][3]});
                    st4(dst + 4, v4f{acc[zz][t][4], acc[zz][t][5], acc[zz][t][6], acc[zz][t][7]});
                }
        }
        if (lane < SS) P[(long)i * ldp + SS * SB + lane] = zsp[i] == lane ? 1.f : 0.f;
    }
}

template <int K, int SS>
__global__ void __launch_bounds__(256) k_l0_edge_sums(const int *__restrict__ rowc, const int *__restrict__ colc,
                                                      const int *__restrict__ revc, const float4 *__restrict__ geom,
                                                      int n, float rc, const int8_t *__restrict__ hop, int hop_max,
                                                      const int *__restrict__ zsp, const float *__restrict__ Qs,
                                                      const float *__restrict__ Qv, int ldq, float4 *__restrict__ S) {
    constexpr int SB = l0_block(K);
    const int lane = threadIdx.x & 63, e = lane & 15, g = lane >> 4;
    const float pirc = 3.14159265358979f / rc;
    const int nw = (int)(gridDim.x * (blockDim.x >> 6));
    const bool inb = 8 * g < SB;   // this lane row's slots lie inside a species block
    for (int i = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)); i < n; i += nw) {
        const int e0 = rowc[i], deg = rowc[i + 1] - e0;
        if (deg == 0) continue;
        // one or two species: this lane's slots of Q_i for every species, held
        // in registers (Q is zero past K); more species: read per edge below
        constexpr bool REG = SS <= 2;
        float qs[REG ? SS : 1][8], qv[REG ? SS : 1][3][8];
#pragma unroll
        for (int zz = 0; zz < (REG ? SS : 0); zz++)
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const float *src = (t == 0 ? Qs + (long)i * ldq : Qv + (3L * i + t - 1) * ldq) + zz * SB + 8 * g;
                v4f lo = v4f{0.f, 0.f, 0.f, 0.f}, hi = lo;
                if (inb) {
                    lo = ld4(src);
                    hi = ld4(src + 4);
                }
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    float *row = t == 0 ? qs[zz] : qv[zz][t > 0 ? t - 1 : 0];
                    row[q] = lo[q];
                    row[q + 4] = hi[q];
                }
            }
        for (int cb = 0; cb < deg; cb += 16) {
            const bool valid = cb + e < deg;
            float4 gm = make_float4(0.f, 0.f, 0.f, rc);
            int j = i;
            if (valid) {
                gm = geom[e0 + cb + e];
                j = colc[e0 + cb + e];
            }
            const int z = zsp[j];
            const bool live = valid && hop[j] <= hop_max;
            const float ir = valid ? __builtin_amdgcn_rcpf(gm.w) : 0.f;
            float eb[8], db[8];
            basis_slots<1, K, true>(gm.w, ir, pirc, valid, g, eb, db);
            // direction of the message edge (i <- j): x_j - x_i
            const float rx = gm.x * ir, ry = gm.y * ir, rz = gm.z * ir;
            float sr = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
            float ql[4][8];   // this edge's species: slots of Q_s, Q_x, Q_y, Q_z
            if constexpr (REG) {
                const bool z1 = SS == 2 && z == 1;   // plain selects: no indexing by z
#pragma unroll
                for (int q = 0; q < 8; q++) {
                    ql[0][q] = z1 ? qs[REG ? SS - 1 : 0][q] : qs[0][q];
#pragma unroll
                    for (int d = 0; d < 3; d++) ql[1 + d][q] = z1 ? qv[REG ? SS - 1 : 0][d][q] : qv[0][d][q];
                }
            } else {
                // the atom's Q rows stay in L1 across its chunks
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const float *src = (t == 0 ? Qs + (long)i * ldq : Qv + (3L * i + t - 1) * ldq) + z * SB + 8 * g;
                    v4f lo = v4f{0.f, 0.f, 0.f, 0.f}, hi = lo;
                    if (inb) {
                        lo = ld4(src);
                        hi = ld4(src + 4);
                    }
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        ql[t][q] = lo[q];
                        ql[t][q + 4] = hi[q];
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 8; q++) {
                const float a = ql[0][q], bx = ql[1][q], by = ql[2][q], bz = ql[3][q];
                sr = fmaf(db[q], fmaf(rx, bx, fmaf(ry, by, fmaf(rz, bz, a))), sr);
                sx = fmaf(eb[q], bx, sx);
                sy = fmaf(eb[q], by, sy);
                sz = fmaf(eb[q], bz, sz);
            }
            // sum over the four lane rows (all basis slots)
            sr += __shfl_xor(sr, 16, 64);
            sx += __shfl_xor(sx, 16, 64);
            sy += __shfl_xor(sy, 16, 64);
            sz += __shfl_xor(sz, 16, 64);
            sr += __shfl_xor(sr, 32, 64);
            sx += __shfl_xor(sx, 32, 64);
            sy += __shfl_xor(sy, 32, 64);
            sz += __shfl_xor(sz, 32, 64);
            // the sums of edge (i <- j) go to the slot of its reverse (j <- i),
            // where the adjoint of the later layers keeps them
            if (g == 0 && valid)
                S[revc[e0 + cb + e]] = live ? make_float4(sr, sx, sy, sz) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
}

static int grid_x(int n) {
    int b = std::min((n + MW - 1) / MW, 2048);
    if (b >= 8) b -= b % 8;   // keeps blockIdx.x % 8 the XCD in every pass row
    return std::max(1, b);
}

// Workgroups of kern (with the given block size) that the current device
// holds at once: compute units times the workgroups per compute unit.
template <class KERN>
static int resident_grid(KERN kern, int block) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, block, 0) != hipSuccess || per <= 0) per = 1;
    return cus * per;
}

template <int P, int F, int K>
static int launch_fwd(hipStream_t st, const MsgArgs &a) {
    constexpr bool piw = Pass<F, FWD_W>::N > 1;
    if constexpr (piw) {
        if (!a.layer0) {
            auto kern = msg_wide(a.n, F) ? k_msg_fwd_pw<P, F, K, true> : k_msg_fwd_pw<P, F, K, false>;
            constexpr int block = 64 * FWD_PIW_WAVES;
            // (per process: one device type; both have the same registers and LDS)
            static const int resident = resident_grid(k_msg_fwd_pw<P, F, K, false>, block);
            // With an atom per wave the launch lasts as long as whole rounds of
            // atoms; a pass of an atom per wave makes the rounds a pass long, at
            // the price of the basis in every pass (about a fifth of a pass)
            constexpr int NP = Pass<F, FWD_W>::N;
            const long W = (long)resident * FWD_PIW_WAVES, rounds = (a.n + W - 1) / W, split = (NP * (long)a.n + W - 1) / W;
            const int np = 6 * split < 5 * NP * rounds ? NP : 1;
            int b = std::min(resident / np, (a.n + FWD_PIW_WAVES - 1) / FWD_PIW_WAVES);
            if (b >= 8) b -= b % 8;
            kern<<<dim3((unsigned)std::max(1, b), (unsigned)np), block, 0, st>>>(a.rowc, a.colc, a.geom, a.n, a.phi, a.u, a.s, a.v,
                                                                   a.A, a.c, a.rc, a.hop, a.hop_max, a.queue, a.sn,
                                                                   a.v1);
            return hipGetLastError() == hipSuccess ? 0 : -5;
        }
    }
    dim3 grid((unsigned)grid_x(a.n), (unsigned)Pass<F, FWD_W>::N);
    auto kern = a.layer0 ? k_msg_fwd<P, F, K, true> : k_msg_fwd<P, F, K, false>;
    kern<<<grid, 64 * MW, 0, st>>>(a.rowc, a.colc, a.geom, a.n, a.phi, a.u, a.s, a.v, a.A, a.c, a.rc, a.hop,
                                   a.hop_max, a.species, a.queue, a.sn, a.v1);
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

template <int P, int F, int K>
static int launch_bwd(hipStream_t st, const MsgArgs &a) {
    constexpr bool piw = Pass<F, BWD_W>::N > 1;
    if constexpr (piw) {
        if (!a.layer0) {
            auto kern = msg_wide(a.n, F) ? k_msg_bwd_pw<P, F, K, true> : k_msg_bwd_pw<P, F, K, false>;
            constexpr int block = 64 * BWD_PIW_WAVES;
            // (per process: one device type; both have the same registers and LDS)
            static const int resident = resident_grid(k_msg_bwd_pw<P, F, K, false>, block);
            int b = std::min(resident, (a.n + BWD_PIW_WAVES - 1) / BWD_PIW_WAVES);
            if (b >= 8) b -= b % 8;
            kern<<<dim3((unsigned)std::max(1, b)), block, 0, st>>>(a.rowc, a.colc, a.geom, a.n, a.phi, a.v, a.gs1,
                                                                   a.gv1, a.A, a.c, a.rc, a.hop, a.hop_max, a.queue,
                                                                   a.gv_in, a.gphi, a.S);
            return hipGetLastError() == hipSuccess ? 0 : -5;
        }
    }
    dim3 grid((unsigned)grid_x(a.n), (unsigned)Pass<F, BWD_W>::N);
    auto kern = a.layer0 ? k_msg_bwd<P, F, K, true> : k_msg_bwd<P, F, K, false>;
    kern<<<grid, 64 * MW, 0, st>>>(a.rowc, a.colc, a.geom, a.n, a.phi, a.v, a.gs1, a.gv1, a.A, a.c, a.rc, a.hop,
                                   a.hop_max, a.species, a.queue, a.gv_in, a.gphi, a.S, a.s_stride);
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

static unsigned l0_blocks(int n) { return (unsigned)std::max(1, std::min((n + 3) / 4, 8192)); }

template <int K, int SS>
static int l0_sums(hipStream_t st, const L0Args &a) {
    k_l0_basis_sums<K, SS><<<l0_blocks(a.n), 256, 0, st>>>(a.rowc, a.colc, a.geom, a.n, a.rc, a.hop, a.hop_max,
                                                           a.species, a.P, a.ldp, a.R, a.ldr);
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

template <int K, int SS>
static int l0_edges(hipStream_t st, const L0Args &a) {
    k_l0_edge_sums<K, SS><<<l0_blocks(a.n), 256, 0, st>>>(a.rowc, a.colc, a.revc, a.geom, a.n, a.rc, a.hop,
                                                          a.hop_max, a.species, a.Qs, a.Qv, a.ldq, a.S);
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

#define L0_DISPATCH_K(FN, K_)                                      \
    do {                                                           \
        if (S == 1) return FN<K_, 1>(st, a);                       \
        if (S == 2) return FN<K_, 2>(st, a);                       \
        if (S == 3) return FN<K_, 3>(st, a);                       \
        if (S == 4) return FN<K_, 4>(st, a);                       \
    } while (0)
#define L0_DISPATCH(FN)                                            \
    do {                                                           \
        if (K == 20) L0_DISPATCH_K(FN, 20);                        \
        if (K == 8) L0_DISPATCH_K(FN, 8);                          \
        if (K == 6) L0_DISPATCH_K(FN, 6);                          \
    } while (0)

bool l0_factorised(int K, int S) { return (K == 20 || K == 8 || K == 6) && S >= 1 && S <= 4; }

int msg_l0_basis_sums(hipStream_t st, int K, int S, const L0Args &a) {
    const int CS = S * l0_block(K);
    if (a.ldp < CS + S || a.ldr < CS || a.ldp % 4 || a.ldr % 4) return -1;
    L0_DISPATCH(l0_sums);
    return -1;
}

int msg_l0_edge_sums(hipStream_t st, int K, int S, const L0Args &a) {
    if (a.ldq < S * l0_block(K) || a.ldq % 4) return -1;
    L0_DISPATCH(l0_edges);
    return -1;
}

int msg_passes(int F) { return F < BWD_W ? 1 : F / BWD_W; }

int msg_slots(int F, int T, bool l0_factorised) { return T - 1 + (l0_factorised ? 1 : msg_passes(F)); }

static unsigned edge_blocks(long ne_max) { return (unsigned)std::max(1L, std::min((ne_max + 255) / 256, 8192L)); }

int msg_assemble_G(hipStream_t st, const int *rowc, int n, long ne_max, const float4 *geom, const float4 *S,
                   long s_stride, int npass, float4 *G) {
    k_assemble_G<<<edge_blocks(ne_max), 256, 0, st>>>(rowc, n, geom, S, s_stride, npass, G);
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

#define MSG_DISPATCH(FN, P_)                                     \
    do {                                                         \
        if (F == 128 && K == 20) return FN<P_, 128, 20>(st, a);  \
        if (F == 128 && K == 8) return FN<P_, 128, 8>(st, a);    \
        if (F == 64 && K == 20) return FN<P_, 64, 20>(st, a);    \
        if (F == 64 && K == 8) return FN<P_, 64, 8>(st, a);      \
        if (F == 32 && K == 20) return FN<P_, 32, 20>(st, a);    \
        if (F == 32 && K == 8) return FN<P_, 32, 8>(st, a);      \
        if (F == 16 && K == 6) return FN<P_, 16, 6>(st, a);      \
    } while (0)

int msg_forward(hipStream_t st, int precision, int F, int K, const MsgArgs &a) {
    if (precision == 0) MSG_DISPATCH(launch_fwd, 0);
    else if (precision == 1) MSG_DISPATCH(launch_fwd, 1);
    else MSG_DISPATCH(launch_fwd, 2);
    return -1;
}

int msg_adjoint(hipStream_t st, int precision, int F, int K, const MsgArgs &a) {
    if (precision == 0) MSG_DISPATCH(launch_bwd, 0);
    else if (precision == 1) MSG_DISPATCH(launch_bwd, 1);
    else MSG_DISPATCH(launch_bwd, 2);
    return -1;
}

}  // namespace mlp
