// plan_facts.cpp -- facts of a plan's device tables for the host tests (test_plan_facts.py):
// built against the library's internal headers and linked to libqsv.so.
#include "planner.h"
#include "qsv.h"

namespace qsv {
bool read_gate_public(const qsv_gate& g, int n, InGate& out, std::string& err);
}

extern "C" {

// One pass of a plan, as its launch sees it.
struct PassFacts {
    int tile_qubits, low_qubits, ops, matrix_ops, staged, diag_ops, diag_unstaged, a_len, d_len;
    int pool;   // complex pool entries the pass's ops read
    long long tiles, pool_total;
};

// Plans the circuit with the defaults of `dtype` on tiles of 2^tile amplitudes; the facts of
// up to `max` passes.  Returns the number of passes, or -1.
int plan_facts(int n, int dtype, int tile, const qsv_gate* gates, size_t count, PassFacts* out, int max)
{
    using namespace qsv;
    std::vector<InGate> in(count);
    std::string err;
    for (size_t i = 0; i < count; ++i)
        if (!read_gate_public(gates[i], n, in[i], err)) return -1;
    HostPlan P;
    PlanOpts o = default_opts(dtype);
    o.tile_qubits = tile;
    if (!make_plan(n, dtype, in, o, P, err)) return -1;
    for (size_t p = 0; p < P.pargs.size() && (int)p < max; ++p) {
        const PassArgs& a = P.pargs[p];
        PassFacts f{a.m, a.L, a.op_count, 0, a.staged, 0, 0, a.a_len, a.d_len, 0, P.pgrid[p], (long long)P.pool.size()};
        for (int i = a.op_begin; i < a.op_begin + a.op_count; ++i) {
            const DevOp& d = P.ops[(size_t)i];
            f.matrix_ops += d.kind == OP_DENSE && d.goff >= 0;
            f.diag_ops += d.kind == OP_DIAG;
            f.pool += d.kind != OP_DENSE ? 1 << d.k : d.goff < 0 ? 1 << (2 * d.k) : 0;
            f.diag_unstaged += d.kind == OP_DIAG && d.aoff < 0;
        }
        out[p] = f;
    }
    return (int)P.pargs.size();
}

int reserved_slots(size_t forward, size_t undo, size_t plans, int slots, size_t* bytes)
{
    const qsv::TabReserve r = qsv::tab_reserve(forward, undo, plans, slots);
    *bytes = r.bytes;
    return r.slots;
}

// Runs of a per-device step over the calls' devices; call `failing` (if it runs it) fails.
int runs_per_device(const int* devices, int calls, int failing, int* ran)
{
    std::atomic<unsigned long long> done{0};
    int failures = 0;
    for (int c = 0; c < calls; ++c) {
        ran[c] = 0;
        const hipError_t e = qsv::once_per_device(done, devices[c], [&] {
            ran[c] = 1;
            return c == failing ? hipErrorInvalidValue : hipSuccess;
        });
        failures += e != hipSuccess;
    }
    return failures;
}

}  // extern "C"
