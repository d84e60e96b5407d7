// The look-ups of a step, in its order (metric, gradient, forward pass); built
// with AddressSanitizer by test_plan_cache.py, which names one of the checks:
//   use    the plans of 400 distinct circuits, each read after its last look-up
//   round  128 circuits over and over: no plan is built twice
//   oldest one circuit more evicts the plans not looked up for the longest time
//   registers  the forward pass of every register has a plan
// Prints "ok".
#include <cstdio>
#include <cstring>
#include <type_traits>
#include <utility>

#include "circuit.hpp"
#include "sweep.hpp"

using namespace qng;

namespace {

// circuit k: a rotation on each of 8 qubits, a ring, then k in binary as CNOTs and CZs
Circuit circuit(int k) {
    std::vector<qng_gate> g;
    for (int q = 0; q < 8; ++q) g.push_back({QNG_RY, q, -1, q});
    for (int q = 0; q < 8; ++q) g.push_back({QNG_CNOT, q, (q + 1) % 8, -1});
    for (int b = 0; b < 9; ++b) g.push_back({(k >> b) & 1 ? QNG_CZ : QNG_CNOT, b % 8, (b + 1) % 8, -1});
    qng_circuit c{};
    c.n_qubits = 8;
    c.n_gates = (int)g.size();
    c.n_params = 8;
    c.gates = g.data();
    return compile_circuit(&c);
}

// no look-up hands out a plan that the caller does not own
template <typename C>
auto borrows(int) -> decltype(std::declval<C &>().get(std::declval<const Circuit &>(), 0, 16, 1, true, 2), std::true_type{});
template <typename C> std::false_type borrows(...);
static_assert(!decltype(borrows<SweepCache>(0))::value, "a look-up returns a plan that the cache may free");

}  // namespace

namespace {

struct Plans {
    std::shared_ptr<const SweepPlan> metric, gradient, apply;
};

Plans look_up(SweepCache &cache, int k) {
    const Circuit c = circuit(k);
    Plans p;
    p.metric = cache.get_shared(c, 0, 16, 1, true, 2);
    p.gradient = cache.get_gradient(c, 0, 16, true);
    p.apply = cache.get_apply(c, c.rots[c.P - 1].pos, 16);
    return p;
}

bool use() {
    SweepCache cache;
    long ops = 0;
    for (int k = 0; k < 400; ++k) {
        const Plans p = look_up(cache, k);
        for (const auto &plan : {p.metric, p.gradient, p.apply})
            for (const DevOp &op : plan->dev_ops) ops += op.type;
    }
    return ops > 0;
}

bool round() {
    SweepCache cache;
    std::vector<Plans> first;
    for (int k = 0; k < 128; ++k) first.push_back(look_up(cache, k));
    for (int pass = 0; pass < 2; ++pass)
        for (int k = 0; k < 128; ++k) {
            const Plans p = look_up(cache, k);
            if (p.metric != first[k].metric || p.gradient != first[k].gradient || p.apply != first[k].apply) return false;
        }
    return true;
}

bool oldest() {
    SweepCache cache;
    std::vector<Plans> first;
    for (int k = 0; k < 128; ++k) first.push_back(look_up(cache, k));
    look_up(cache, 0);     // now circuit 1 is the one not seen for the longest time
    look_up(cache, 128);
    if (cache.plans.size() > 384) return false;
    for (int k = 0; k < 128; ++k) {
        if (k == 1) continue;
        if (look_up(cache, k).metric != first[k].metric) return false;
    }
    return look_up(cache, 1).metric != first[1].metric;
}

bool registers() {
    for (int n = 2; n <= 33; ++n) {
        std::vector<qng_gate> g;
        for (int q = 0; q < 8; ++q) g.push_back({QNG_CNOT, q % n, (q + 1) % n, -1});
        qng_circuit qc{};
        qc.n_qubits = n;
        qc.n_gates = (int)g.size();
        qc.gates = g.data();
        const Circuit c = compile_circuit(&qc);
        for (int amp : {8, 16}) {
            size_t gates = 0;
            const SweepPlan plan = build_apply_plan(c, 0, amp);
            for (const HostPass &hp : plan.cols.at(0).passes)
                for (const DevOp &op : hp.ops) gates += op.type == OP_CNOT;
            if (gates != g.size()) return false;
        }
    }
    return true;
}

}  // namespace

int main(int argc, char **argv) {
    const char *check = argc > 1 ? argv[1] : "";
    const bool ok = !std::strcmp(check, "use")      ? use()
                    : !std::strcmp(check, "round")  ? round()
                    : !std::strcmp(check, "oldest") ? oldest()
                    : !std::strcmp(check, "registers") ? registers()
                                                    : false;
    std::puts(ok ? "ok" : "failed");
    return ok ? 0 : 1;
}
