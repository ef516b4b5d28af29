// The host side of a PaiNN evaluation with every launch replaced by a stub
// that returns a code of the test's choosing: each code has to come back from
// evaluate(), and nothing may be launched behind a failed step.
#include "../../paper_2506_04055_amd/csrc/painn.hip"

#include <cstdio>
#include <cstdlib>

namespace {
struct Step {
    const char *name;
    int calls = 0, fail_at = -1, code = 0;
    int operator()() { return ++calls == fail_at ? code : 0; }
};
Step batch{"batch"}, product{"product"}, msg{"msg"}, node{"node"};
Step *const steps[] = {&batch, &product, &msg, &node};
int launches = 0;
std::string last;
}  // namespace

// HIP entry points that an evaluation calls
extern "C" {
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { launches++; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace mlp {
bool g_prof_on = false;
unsigned g_prof_mask = 0;
void prof_begin(int, hipStream_t) {}
void prof_end(int, hipStream_t) {}
int fail(int code, const std::string &m) { last = m; return code; }
int DevBuf::ensure(size_t need, double, int *) { if (bytes < need) p = std::realloc(p, need), bytes = need; return 0; }
size_t packed_bytes(int, int, bool) { return 256; }
int pack_weight(hipStream_t, const float *, int, int, bool, void *, PackedW *) { return 0; }
int node_gemm(hipStream_t, int, int, const float *, int, const PackedW &, float *, int, int, const float *, float *, int,
              const float *, int, const int *) { return product(); }
int node_gemm_batch(hipStream_t, int, GemmBatch) { return batch(); }
int msg_forward(hipStream_t, int, int, int, const MsgArgs &) { return msg(); }
int msg_adjoint(hipStream_t, int, int, int, const MsgArgs &) { return msg(); }
int msg_l0_basis_sums(hipStream_t, int, int, const L0Args &) { return msg(); }
int msg_l0_edge_sums(hipStream_t, int, int, const L0Args &) { return msg(); }
int msg_assemble_G(hipStream_t, const int *, int, long, const float4 *, const float4 *, long, int, float4 *) { return msg(); }
int msg_slots(int, int T, bool) { return T; }
bool l0_factorised(int, int) { return true; }
int node_forward(hipStream_t, int, int, const NodeArgs &) { return node(); }
int node_adjoint(hipStream_t, int, int, const NodeArgs &) { return node(); }
int node_last(hipStream_t, int, int, const NodeArgs &) { return node(); }
size_t allegro_arena_bytes(const mlp_model *, long, long, bool) { return 0; }
size_t mace_arena_bytes(const mlp_model *, long, long, float, bool) { return 0; }
int allegro_evaluate(mlp_model *, mlp_nbr *, hipStream_t, double *, float *, float *, int, const int *) { return 0; }
int mace_evaluate(mlp_model *, mlp_nbr *, hipStream_t, double *, float *, float *, int, const int *) { return 0; }
}  // namespace mlp

using namespace mlp;

static float out[3 * 64], weights[1 << 16];
static mlp_model model;
static mlp_nbr graph;

mlp::LayerW mlp_model::layer(int) const { return {}; }

static int run() {
    for (Step *s : steps) s->calls = 0;
    launches = 0;
    double e;
    return evaluate(&model, &graph, nullptr, &e, out, nullptr, 0, nullptr);
}

int main() {
    model = {};
    model.F = 128, model.K = 20, model.T = 3, model.S = 2, model.rc = 5.f, model.l0f = true, model.w_dev = weights;
    graph.n_atoms = graph.n_local = 64;
    graph.n_edges_skin = 640;
    int bad = 0;
    auto expect = [&](const char *what, bool ok) {
        std::printf("%s: %s\n", what, ok ? "ok" : "FAILED");
        bad += !ok;
    };
    expect("a clean evaluation", run() == 0 && batch.calls == 2 && product.calls == 0);
    int total[4];
    for (int q = 0; q < 4; q++) total[q] = steps[q]->calls;
    // a shape that the batch does not take: the products one by one
    batch.fail_at = 1, batch.code = -1;
    expect("a batch that does not fit", run() == 0 && product.calls == 2);
    product.fail_at = 2, product.code = -5;
    expect("its second product fails", run() == -5 && node.calls == 0);
    product.fail_at = -1;
    // every step in turn
    for (int q = 0; q < 4; q++)
        for (int k = 1; k <= total[q]; k++) {
            for (Step *s : steps) s->fail_at = -1;
            steps[q]->fail_at = k, steps[q]->code = -5;
            char label[64];
            std::snprintf(label, sizeof label, "%s %d fails", steps[q]->name, k);
            const int rc = run();
            expect(label, rc == -5 && steps[q]->calls == k);
        }
    // the first layer's table, made when a model is created
    for (Step *s : steps) s->fail_at = -1;
    for (int k = 1; k <= 2; k++) {
        product.calls = 0, product.fail_at = k, product.code = -5;
        expect("a product of the species table fails", first_layer_table(&model, nullptr, out) == -5 && product.calls == k);
    }
    return bad != 0;
}
