// plan_facts.cpp -- facts of a plan's device tables for the host tests (test_plan_facts.py):
// built against the library's internal headers and linked to libqsv.so.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "planner.h"
#include "qsv.h"

namespace qsv {
bool read_gate_public(const qsv_gate& g, int n, InGate& out, std::string& err);
}

namespace {

using namespace qsv;

bool plan(int n, int dtype, int tile, const qsv_gate* gates, size_t count, HostPlan& P)
{
    std::vector<InGate> in(count);
    std::string err;
    for (size_t i = 0; i < count; ++i)
        if (!read_gate_public(gates[i], n, in[i], err)) return false;
    PlanOpts o = default_opts(dtype);
    o.tile_qubits = tile;
    return make_plan(n, dtype, in, o, P, err);
}

// ---- a matrix-core step as the kernels take it from its tables (kernels.hip: op_mfma4,
// op_mfma3), lane by lane

int word16(const unsigned* w, int i) { return (w[i >> 1] >> (16 * (i & 1))) & 0xffff; }

int deposit(int v, const unsigned* w, int bits)
{
    int o = 0;
    for (int i = 0; i < bits; ++i)
        if ((v >> i) & 1) o ^= word16(w, i);
    return o;
}

struct Step {
    const DevOp *op, *op2;   // op2: the second of a pair, else op
    bool pair;
};

// Which wave reads (writes) the tile's slots, by slot number; false where a slot is reached
// twice or not at all.  With tile and apool, applies the step to the tile's slots.
bool run_step(int dtype, int m, const Step& s, std::vector<int>& reads, std::vector<int>& writes, std::vector<cd>* tile,
              const float* apool)
{
    const int T = 1 << m, eb = dtype == 0 ? 8 : 16;
    const DevOp &a = *s.op, &b = *s.op2;
    const bool three = dtype == 1 && a.k == 3;
    const int J = three ? 2 : 4, blocks = T / (64 * J);
    auto drow = [&](int q, int e) { return dtype == 0 ? 4 * q + e : 4 * e + q; };
    auto entry = [&](const DevOp& o, int lane, int j) {   // an operand's complex entry
        const float* w = apool + o.goff;
        if (dtype == 0) return cd(w[((j >> 1) * 64 + lane) * 4 + 2 * (j & 1)], w[((j >> 1) * 64 + lane) * 4 + 2 * (j & 1) + 1]);
        double d[2];
        std::memcpy(d, w + (size_t)(j * 64 + lane) * 4, 16);
        return cd(d[0], d[1]);
    };
    reads.assign(T, -1);
    writes.assign(T, -1);
    for (int blk = 0; blk < blocks; ++blk) {
        const int sb = deposit(blk, a.bbit, kMaxBlockBits);
        auto slot = [&](const unsigned* lin, const unsigned* jb, int lane, int j) {
            return (sb ^ deposit(lane, lin, 6) ^ deposit(j, jb, three ? 1 : 2)) / eb;
        };
        const unsigned wj = three ? a.jbit >> 16 : b.jbit;   // (a 3-qubit op's write bit is the second)
        cd x[64][4], y[64][4];
        for (int l = 0; l < 64; ++l)
            for (int j = 0; j < J; ++j) {
                const int r = slot(a.lin, &a.jbit, l, j), w = slot(three ? a.lout : b.lin, &wj, l, j);
                if (r >= T || w >= T || reads[r] >= 0 || writes[w] >= 0) return false;
                reads[r] = writes[w] = blk & 3;
                if (tile) x[l][j] = (*tile)[r];
            }
        if (!tile) continue;
        for (int l = 0; l < 64; ++l) {
            const int q = l >> 4, c = l & 15;
            if (three) {   // rows 4 e + q of the real embedding's product, e = 0..3
                double d[4];
                for (int e = 0; e < 4; ++e) {
                    d[e] = 0;
                    for (int k = 0; k < 4; ++k)
                        for (int j = 0; j < 2; ++j) {
                            const cd A = entry(a, 16 * k + 4 * e + q, j), v = x[16 * k + c][j];
                            d[e] += A.real() * v.real() + A.imag() * v.imag();
                        }
                }
                y[l][0] = cd(d[0], d[1]);
                y[l][1] = cd(d[2], d[3]);
                continue;
            }
            for (int e = 0; e < 4; ++e) {
                cd v = 0;
                for (int k = 0; k < 4; ++k)
                    for (int j = 0; j < 4; ++j)
                        v += s.pair ? entry(a, 16 * k + c, j) * x[16 * k + drow(q, e)][j]
                                    : entry(a, 16 * k + drow(q, e), j) * x[16 * k + c][j];
                y[l][e] = v;
            }
        }
        if (s.pair) {
            std::memcpy(x, y, sizeof(x));
            for (int l = 0; l < 64; ++l)
                for (int e = 0; e < 4; ++e) {
                    cd v = 0;
                    for (int k = 0; k < 4; ++k)
                        for (int j = 0; j < 4; ++j) v += entry(b, 16 * k + drow(l >> 4, e), j) * x[16 * k + (l & 15)][j];
                    y[l][e] = v;
                }
        }
        for (int l = 0; l < 64; ++l)
            for (int j = 0; j < J; ++j) (*tile)[slot(three ? a.lout : b.lin, &wj, l, j)] = y[l][j];
    }
    return std::find(reads.begin(), reads.end(), -1) == reads.end();
}

// LDS slot of tile element e (kernels.hip: swz).
int slot_of(int dtype, int e)
{
    return dtype == 0 ? e ^ ((e >> 5) & 31) ^ (e >> 10) : e ^ ((e >> 4) & 15) ^ ((e >> 8) & 15);
}

// The gate g of descriptor d on the tile's slots, from its definition.
void apply_gate(int dtype, int m, const DevOp& d, const FGate& g, std::vector<cd>& tile)
{
    const int D = 1 << g.k;
    int mask = 0;
    for (int j = 0; j < g.k; ++j) mask |= 1 << d.lpos[j];
    for (int e = 0; e < (1 << m); ++e) {
        if (e & mask) continue;
        std::vector<cd> v(D);
        std::vector<int> at(D);
        for (int r = 0; r < D; ++r) {
            int x = e;
            for (int j = 0; j < g.k; ++j) x |= ((r >> j) & 1) << d.lpos[j];
            at[r] = slot_of(dtype, x);
            v[r] = tile[at[r]];
        }
        for (int r = 0; r < D; ++r) {
            cd s = 0;
            for (int c = 0; c < D; ++c) s += g.m[(size_t)r * D + c] * v[c];
            tile[at[r]] = s;
        }
    }
}

}  // namespace

extern "C" {

// Walks every matrix-core step of the plan's passes: each slot of the tile read and written
// once, by the same wave; where no barrier follows a step, the next one is a matrix-core step
// whose waves own the same slots; and (apply) the tables' product on a random tile against the
// gates' definition.  Returns the steps walked, or minus the pass number minus 1 of the first
// fault; worst: the largest error; free_steps: steps without a barrier behind them.
int check_steps(int n, int dtype, int tile, const qsv_gate* gates, size_t count, int apply, double* worst, int* free_steps)
{
    HostPlan P;
    if (!plan(n, dtype, tile, gates, count, P)) return -100000;
    int steps = 0;
    *worst = 0;
    *free_steps = 0;
    for (size_t p = 0; p < P.pargs.size(); ++p) {
        const PassArgs& a = P.pargs[p];
        std::vector<int> owner;   // of the slots, after a step without a barrier
        for (int i = 0; i < a.op_count; ++i) {
            const DevOp& d = P.ops[(size_t)(a.op_begin + i)];
            if (d.kind != OP_DENSE || d.goff < 0) {
                if (!owner.empty()) return -(int)p - 1;
                continue;
            }
            const bool pair = d.flags & 1;
            const int second = pair ? i + 1 : i;
            const Step s{&d, &P.ops[(size_t)(a.op_begin + second)], pair};
            std::vector<int> reads, writes;
            std::vector<cd> t((size_t)1 << a.m), want;
            for (size_t e = 0; e < t.size(); ++e) t[e] = cd(std::sin(1.0 + 0.7 * (double)e), std::cos(2.0 + 1.3 * (double)e));
            want = t;
            if (!run_step(dtype, a.m, s, reads, writes, apply ? &t : nullptr, P.apool.data())) return -(int)p - 1;
            if (reads != writes || (!owner.empty() && owner != reads)) return -(int)p - 1;
            if (apply) {
                for (int x = i; x <= second; ++x)
                    apply_gate(dtype, a.m, P.ops[(size_t)(a.op_begin + x)], P.fused[(size_t)P.passes[p].ops[(size_t)x]], want);
                for (size_t e = 0; e < t.size(); ++e) *worst = std::max(*worst, std::abs(t[e] - want[e]));
            }
            owner = d.nosync ? writes : std::vector<int>();
            *free_steps += d.nosync;
            ++steps;
            i = second;
        }
        if (!owner.empty()) return -(int)p - 1;
    }
    return steps;
}

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
    HostPlan P;
    if (!plan(n, dtype, tile, gates, count, P)) return -1;
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
