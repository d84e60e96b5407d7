// The look-ups of a step, in its order (metric, gradient, forward pass), over
// more distinct circuits than the cache keeps; built with AddressSanitizer by
// test_plan_cache.py.  Prints "ok".
#include <cstdio>
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

int main() {
    SweepCache cache;
    long ops = 0;
    for (int k = 0; k < 400; ++k) {
        const Circuit c = circuit(k);
        const auto plan = cache.get_shared(c, 0, 16, 1, true, 2);
        const auto gradient = cache.get_gradient(c, 0, 16, true);
        const auto apply = cache.get_apply(c, c.rots[c.P - 1].pos, 0, 16);
        for (const auto &p : {plan, gradient, apply})
            for (const DevOp &op : p->dev_ops) ops += op.type;
    }
    if (ops <= 0) return 1;
    std::puts("ok");
    return 0;
}
