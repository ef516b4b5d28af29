// The per-atom work of a PaiNN layer, one kernel each way.
//
// Between two message passes an atom's state goes through
//   Uv = U v1, Vv = V v1, n = sqrt(eps + sum_d Vv_d^2)
//   a = W4 silu(W3 [s1 | n] + b3) + b4
//   s2 = s1 + a_sv <Uv, Vv> + a_ss, v2 = v1 + a_vv Uv             (update, layer t)
//   phi = W2 silu(W1 s2 + b1) + b2, u = v2 phi_vv                  (message MLP, layer t + 1)
// and, after the last update, through the readout
//   U = w6 silu(W5 s2 + b5) + b6.
// node_forward takes the first two, node_adjoint their adjoint, node_last the
// last update with the readout and the adjoint of both.  A wave owns 16 atoms
// as columns of D = W X (edge_chain.h): features stay in the lane from layer
// to layer, the weights stream through LDS.  Only what other atoms or a later
// kernel read goes to HBM: the adjoint forms Uv, Vv, n, a and both hidden
// layers again from s1, v1 and s2 (14 + 16 F floats per atom and layer
// against 84 F with the intermediates stored and a kernel per product pair).
//
// What bounds them: of the 38,500 cycles that a 16-atom tile of the adjoint
// takes on a compute unit at F = 128 and 1.2M rows, 12,700 are matrix cores (all
// four SIMDs), 9,000 LDS (the weights), and its bytes are 24,000 at the rate of
// a copy, overlapped by two waves per SIMD only.
// The directions are taken one after another, which reads U's and V's blocks
// three times but holds one direction's operands (32 registers, not 96).
// Busy at 1.2M rows, forward / adjoint / last layer: the data return of the
// vector loads 84 / 79 / 70 %, matrix cores 24 / 33 / 36 %, LDS 17 / 23 / 25 %
// and vector issue 17 / 22 / 23 %, at under two waves per SIMD.
// Per launch, split bf16, forward / adjoint / last layer: 24,000 atoms of 128
// features 66 / 104 / 80 us (the chained products they replace: forward 120
// and the U V product, adjoint 159); 171,500 atoms of 64 features 178 / 237 /
// 157 (433 and the U V product, 497); 1.2M rows of 128 features 3.4 / 5.3 / 3.3
// ms (4.3 and the U V product, 6.0).  FP32, 48,000 atoms of 128 features: 184 /
// 339 / 268 us.
//
// The kernels of one operand form are a translation unit (node_p0.hip ..
// node_p2.hip: compiled side by side); packing and dispatch are in node.hip.
#pragma once
#include "edge_chain.h"
#include "node.h"

namespace mlp {

// which: 0 forward, 1 adjoint, 2 last layer
template <int P>
int node_launch(hipStream_t s, int F, int which, const NodeArgs &a);

template <int F>
struct NodeDim {
    static constexpr int NT = F / 16, KS = (F + 31) / 32;      // 16-feature tiles, 32-feature blocks
    static constexpr int N5 = F >= 32 ? F / 32 : 1, K5 = (N5 + 1) / 2;   // the readout's hidden layer
    static constexpr bool KEEP = F <= 64;   // Uv, Vv stay in registers through the adjoint
    static constexpr int Q = NT * KS;
    static constexpr int stages(int units) { return (units + EC_U - 1) / EC_U; }
    // stages of the chains' segments: U and V; the forward's other layers;
    // the message MLP's adjoint; the update's (last: with the readout, SE
    // of them up to it); the adjoint of U and V, per direction
    static constexpr int SA = stages(2 * Q), SF = stages(9 * Q), SI = stages(5 * Q), SM = stages(9 * Q),
                         SL = stages(8 * Q + N5 * KS + NT * K5), SE = stages(4 * Q + N5 * KS + 2), SH = stages(KEEP ? 2 * Q : 4 * Q);
};

}  // namespace mlp
