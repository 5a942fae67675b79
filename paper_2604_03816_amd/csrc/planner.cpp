// planner.cpp -- DAG gate fusion (Section 5.2, Algorithm 2) and HBM pass scheduling.
//
// DAG (Section 5.1): one scan keeps, per qubit, the most recent gate; the edges are
// these immediate per-qubit predecessors, so |E| <= sum |q(v)| (Eq. 8).  Here the DAG
// is stored as a doubly linked list of nodes per qubit ("line"): prev/next of a node
// on each of its qubits.
//
// Fusion (Algorithm 2): repeated sweeps in topological order; for each gate v and each
// predecessor u, merge v into u when
//   (1) u is a predecessor of v,
//   (2) |q(u) U q(v)| <= kmax  (q_max^fuse),
//   (3) u is v's predecessor on every shared qubit,
//   (4) the merge keeps the graph acyclic.  The paper's conditions (1)-(3) alone allow
//       merges that skip an intervening gate (u{0,1}, w{1,2}, v{0,2}: u and v share
//       qubit 0 with nothing between them there, yet w must run between them).  A merge
//       is sound iff no other path u ~> v exists; we accept it when every other
//       predecessor of v precedes u in the sweep's topological order (then none is a
//       descendant of u), or every other successor of u follows v (then no path from u
//       through them reaches v).  Either rule also gives the fused node a valid slot in
//       the order, so one order serves the whole sweep.
//   (5) cost-aware mode only: the fused op costs no more arithmetic than its parts
//       plus the per-op overhead it removes -- the trade-off of Eq. 13, where fused
//       gates have a higher per-gate cost c_2 than unfused ones (c_1).
// The fused matrix is U_v . U_u on the union of the targets (Eq. 9), each factor
// embedded as identity on the qubits it does not act on; products in FP64.
//
// Pass scheduling: the fused gates, in topological order, are grouped greedily into
// HBM passes.  A pass holds a tile of 2^m amplitudes on chip: the L lowest qubits
// (contiguous in memory, so every tile row is a coalesced run) plus up to m - L other
// qubits.  A gate joins the current pass when its targets fit in the tile, none of
// its qubits is blocked by an earlier deferred gate, and the pass's arithmetic budget
// allows.  Diagonal gates need no tile capacity: qubits outside the tile are
// constant within a tile, so their phase is a per-tile constant.
#include "planner.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <queue>
#include <unordered_map>

namespace qsv {

PlanOpts default_opts(int dtype)
{
    PlanOpts o;
    // Budgets: measured on the 30-qubit depth-20 brickwork (the pass count / per-pass
    // arithmetic trade-off that minimises total time).
    if (dtype == 0) {   // complex64: 8-byte amplitudes
        o.tile_qubits = 12;
        o.low_qubits = 4;
        o.whole_state_max = 13;
        o.pass_budget = 224;
        o.sigma = 8;
        o.mfma_min_k = 3;
        o.fp32_mfma = true;
        o.amp_floats = 2;
        o.stage_floats = 2048;  // 8 KiB (four operands) beside a 32 KiB tile: four workgroups per CU
    } else {            // complex128: 16-byte amplitudes
        o.tile_qubits = 12;
        o.low_qubits = 3;   // 8 contiguous amplitudes: 128-byte runs, as complex64's 16
        o.whole_state_max = 12;
        o.pass_budget = 320;
        o.sigma = 8;
        o.amp_floats = 4;
        o.mfma_min_k = 3;       // FP64 matrix cores: no faster than FP64 VALU in peak, but
                                // free of the VALU path's per-row scalar loads
        o.stage_floats = 4096;  // 16 KiB (four operands) beside a 64 KiB tile: two workgroups per CU
    }
    return o;
}

bool plan_opts_from(int dtype, const qsv_plan_opts* pub, PlanOpts& o, std::string& err)
{
    o = default_opts(dtype);
    if (!pub) return true;
    if (pub->fuse < 0 || pub->fuse > 2) { err = "fuse must be 0, 1 or 2"; return false; }
    o.fuse = pub->fuse;
    if (pub->kmax) o.kmax = pub->kmax;
    if (pub->cost_aware) o.cost_aware = pub->cost_aware;
    if (pub->tile_qubits) o.tile_qubits = pub->tile_qubits;
    if (pub->low_qubits) o.low_qubits = pub->low_qubits;
    if (pub->pass_budget != 0) o.pass_budget = pub->pass_budget;
    if (pub->matrix_cores) {
        if (pub->matrix_cores != -1 && (pub->matrix_cores < 3 || pub->matrix_cores > kMaxMfmaK)) {
            err = "matrix_cores must be 0, -1, 3 or 4 (matrix-core ops have 3 or 4 targets)";
            return false;
        }
        o.mfma_min_k = pub->matrix_cores < 0 ? 0 : pub->matrix_cores;
    }
    if (pub->op_cost < 0) { err = "op_cost must be >= 0"; return false; }
    if (pub->op_cost > 0) o.sigma = pub->op_cost;
    if (pub->commute < -1 || pub->commute > 1) { err = "commute must be 0, 1 or -1"; return false; }
    if (pub->commute) o.commute = pub->commute > 0;
    if (o.fuse != 1) o.commute = 0;
    if (o.fuse == 0) o.max_ops_per_pass = 1;
    return true;
}

namespace {

bool zero(const cd& v) { return v.real() == 0 && v.imag() == 0; }

// Kind of a matrix and, as local bits, the targets it is not diagonal on, in one look at its
// nonzero entries.
int structure(const cd* m, int k, int& off)
{
    const int d = 1 << k;
    int flips = 0, perm = 1;
    unsigned cols = 0;
    for (int r = 0; r < d; ++r) {
        int cnt = 0;
        const cd* row = m + (size_t)r * d;
        for (int c = 0; c < d; ++c) {
            if (zero(row[c])) continue;
            flips |= r ^ c;
            ++cnt;
            if ((cols >> c) & 1) perm = 0;
            cols |= 1u << c;
        }
        if (cnt != 1) perm = 0;
        if (!perm && flips == d - 1) break;
    }
    off = flips;
    return flips == 0 ? OP_DIAG : perm ? OP_PERM : OP_DENSE;
}

// Sets g's kind and its diagonal qubits from its matrix.
void inspect(FGate& g)
{
    int off = 0;
    g.kind = structure(g.m.vec().data(), g.k, off);
    g.dq = 0;
    for (int j = 0; j < g.k; ++j)
        if (!((off >> j) & 1)) g.dq |= 1ull << g.q[j];
}

}  // namespace

int classify(const std::vector<cd>& m, int k)
{
    int off = 0;
    return structure(m.data(), k, off);
}

unsigned long long diag_qubit_mask(const FGate& g)
{
    int off = 0;
    structure(g.m.vec().data(), g.k, off);
    unsigned long long dq = 0;
    for (int j = 0; j < g.k; ++j)
        if (!((off >> j) & 1)) dq |= 1ull << g.q[j];
    return dq;
}

bool ops_commute(const FGate& a, const FGate& b)
{
    unsigned long long qa = 0, qb = 0;
    for (int j = 0; j < a.k; ++j) qa |= 1ull << a.q[j];
    for (int j = 0; j < b.k; ++j) qb |= 1ull << b.q[j];
    const unsigned long long shared = qa & qb;
    return (shared & ~(a.dq & b.dq)) == 0;
}

double op_fma(const FGate& g)
{
    const int d = 1 << g.k;
    if (g.kind == OP_DENSE) return 4.0 * d;     // 2^k complex MACs per amplitude
    if (g.kind == OP_DIAG) return 4.0;          // one complex multiply
    for (int r = 0; r < d; ++r) {               // permutation: free unless it has phases
        for (int c = 0; c < d; ++c) {
            const cd v = g.m[(size_t)r * d + c];
            if (v != cd(0, 0) && v != cd(1, 0)) return 4.0;
        }
    }
    return 0.0;
}

double op_cost(const FGate& g, const PlanOpts& o)
{
    const double f = op_fma(g);
    if (mfma_eligible(g, o)) {
        // complex128: the FP64 VALU's rate, a 4-qubit op as three real products where its
        // embedding would take four.  complex64, per 256 amplitudes and SIMD: a 4-qubit op
        // takes 192 matrix-core clocks and about 200 of the VALU beside them (the exact
        // splits, addresses), where 24 FMA per amplitude on the VALU take 384; a 3-qubit op
        // (run as a 4-qubit one) is priced below that, so that fusion is not driven to
        // widen every 3-qubit op.
        return (o.fp32_mfma ? 0.5 : 1.0) * (g.k == 4 ? 0.75 : 1.0) * f;
    }
    return f;
}

bool mfma_eligible(const FGate& g, const PlanOpts& o)
{
    return g.kind == OP_DENSE && o.mfma_min_k > 0 && g.k >= o.mfma_min_k && g.k <= kMaxMfmaK;
}

namespace {

bool is_identity(const FGate& g)   // (its kind is set)
{
    if (g.kind != OP_DIAG) return false;
    const int d = 1 << g.k;
    for (int r = 0; r < d; ++r)
        if (g.m[(size_t)r * d + r] != cd(1, 0)) return false;
    return true;
}

// Embed matrix `a` (local bit j <-> qa[j], ascending, ka bits) into the ascending qubit
// list Q (kq bits): E[r', r] = a[sub(r'), sub(r)] when r' and r agree outside qa, else 0.
std::vector<cd> embed(const std::vector<cd>& a, const int* qa, int ka, const int* Q, int kq)
{
    const int dq = 1 << kq;
    int pos[kMaxK];
    int amask = 0;
    for (int j = 0; j < ka; ++j) {
        int p = 0;
        while (Q[p] != qa[j]) ++p;
        pos[j] = p;
        amask |= 1 << p;
    }
    auto sub = [&](int r) {
        int s = 0;
        for (int j = 0; j < ka; ++j) s |= ((r >> pos[j]) & 1) << j;
        return s;
    };
    const int da = 1 << ka;
    if (ka == kq) return a;   // a spans Q: its targets are Q itself, in the same order
    int sr[1 << kMaxK];
    for (int r = 0; r < dq; ++r) sr[r] = sub(r);
    std::vector<cd> e((size_t)dq * dq, cd(0, 0));
    for (int r = 0; r < dq; ++r)
        for (int c = 0; c < dq; ++c)
            if ((r & ~amask) == (c & ~amask)) e[(size_t)r * dq + c] = a[(size_t)sr[r] * da + sr[c]];
    return e;
}

// a += w b, the plain product (std::complex's checks for NaN: every entry here is finite)
inline void madd(cd& a, const cd& w, const cd& b)
{
    a = cd(a.real() + (w.real() * b.real() - w.imag() * b.imag()),
           a.imag() + (w.real() * b.imag() + w.imag() * b.real()));
}

// out[b] = sum_t w[t] in[t][b] in ascending t from zero, for an even count of columns: madd's
// products and sums, on vectors of V / 2 complex numbers held in registers over t
// ((re, im) * w.re plus (im, re) * (-w.im, w.im)).
template <typename V>
__attribute__((always_inline)) inline void mix_rows_v(double* out, const cd* w, const double* const* in, int terms,
                                                      int count)
{
    constexpr int L = sizeof(V) / sizeof(double), U = 4;
    for (int b = 0; b < 2 * count; b += L * U) {
        const int nu = std::min(U, (2 * count - b) / L);
        V acc[U];
        for (int u = 0; u < U; ++u) acc[u] = V{};
        for (int t = 0; t < terms; ++t) {
            V wr, wi;
            for (int l = 0; l < L; ++l) {
                wr[l] = w[t].real();
                wi[l] = (l & 1) ? w[t].imag() : -w[t].imag();
            }
            for (int u = 0; u < U; ++u) {
                if (u >= nu) break;
                V x;
                std::memcpy(&x, in[t] + b + u * L, sizeof(V));
                V y;
                for (int l = 0; l < L; ++l) y[l] = x[l ^ 1];
                acc[u] += x * wr + y * wi;
            }
        }
        for (int u = 0; u < nu; ++u) std::memcpy(out + b + u * L, &acc[u], sizeof(V));
    }
}

typedef double v2d __attribute__((vector_size(16)));
typedef double v4d __attribute__((vector_size(32)));

__attribute__((target("avx2"))) void mix_rows_avx2(double* out, const cd* w, const double* const* in, int terms,
                                                   int count)
{
    mix_rows_v<v4d>(out, w, in, terms, count);
}

void mix_rows(double* out, const cd* w, const double* const* in, int terms, int count)
{
    static const bool avx2 = __builtin_cpu_supports("avx2");
    if (avx2) mix_rows_avx2(out, w, in, terms, count);
    else mix_rows_v<v2d>(out, w, in, terms, count);
}

// E(v) . E(u) over the ascending qubit list Q without forming either embedding: row r of
// the product mixes the rows of E(u) that differ from r only in v's bits, in ascending
// order, and such a row has 2^ku entries: the sums of the plain product, term for term
// (zero entries of either factor's embedding skipped).
std::vector<cd> embedded_product(const FGate& v, const FGate& u, const int* Q, int kq)
{
    const int dq = 1 << kq, dv = 1 << v.k, du = 1 << u.k;
    int vspread[1 << kMaxK], uspread[1 << kMaxK], vsub[1 << kMaxK], usub[1 << kMaxK];
    auto lay = [&](const FGate& g, int* spread, int* sub) {   // returns g's bits in Q
        int pos[kMaxK], mask = 0;
        for (int j = 0; j < g.k; ++j) {
            int p = 0;
            while (Q[p] != g.q[j]) ++p;
            pos[j] = p;
            mask |= 1 << p;
        }
        for (int a = 0; a < (1 << g.k); ++a) {
            int x = 0;
            for (int j = 0; j < g.k; ++j) x |= ((a >> j) & 1) << pos[j];
            spread[a] = x;
        }
        for (int r = 0; r < dq; ++r) {
            int x = 0;
            for (int j = 0; j < g.k; ++j) x |= ((r >> pos[j]) & 1) << j;
            sub[r] = x;
        }
        return mask;
    };
    const int vmask = lay(v, vspread, vsub), umask = lay(u, uspread, usub);
    std::vector<cd> C((size_t)dq * dq, cd(0, 0));
    if (v.kind == OP_DIAG && u.kind == OP_DIAG) {
        for (int r = 0; r < dq; ++r)
            madd(C[(size_t)r * dq + r], v.m[(size_t)vsub[r] * dv + vsub[r]], u.m[(size_t)usub[r] * du + usub[r]]);
        return C;
    }
    for (int r = 0; r < dq; ++r) {
        const cd* vrow = &v.m[(size_t)vsub[r] * dv];
        cd* out = &C[(size_t)r * dq];
        if (du == dq) {   // u spans Q: whole rows
            cd w[1 << kMaxK];
            const double* in[1 << kMaxK];
            int terms = 0;
            for (int a = 0; a < dv; ++a) {
                if (zero(vrow[a])) continue;
                w[terms] = vrow[a];
                in[terms++] = reinterpret_cast<const double*>(&u.m[(size_t)((r & ~vmask) | vspread[a]) * du]);
            }
            mix_rows(reinterpret_cast<double*>(out), w, in, terms, dq);
            continue;
        }
        for (int a = 0; a < dv; ++a) {
            const cd w = vrow[a];
            if (zero(w)) continue;
            const int ri = (r & ~vmask) | vspread[a], keep = ri & ~umask;
            const cd* urow = &u.m[(size_t)usub[ri] * du];
            for (int b = 0; b < du; ++b) madd(out[keep | uspread[b]], w, urow[b]);
        }
    }
    return C;
}

// Canonical form of an input gate: ascending targets, rows/columns permuted to match.
FGate canonical(const InGate& g, int index)
{
    FGate f;
    f.k = g.k;
    int order[kMaxK];
    for (int j = 0; j < g.k; ++j) order[j] = j;
    std::sort(order, order + g.k, [&](int a, int b) { return g.t[a] < g.t[b]; });
    for (int j = 0; j < g.k; ++j) f.q[j] = g.t[order[j]];
    const int d = 1 << g.k;
    auto remap = [&](int r) {  // new local index -> old local index
        int o = 0;
        for (int j = 0; j < g.k; ++j) o |= ((r >> j) & 1) << order[j];
        return o;
    };
    std::vector<cd> m((size_t)d * d);
    for (int r = 0; r < d; ++r)
        for (int c = 0; c < d; ++c) m[(size_t)r * d + c] = g.m[(size_t)remap(r) * d + remap(c)];
    f.m = std::move(m);
    f.id = index;
    inspect(f);
    f.first = index;
    f.mem.assign(1, index);
    return f;
}

struct Node {
    FGate g;
    bool alive = true;
    int prev[kMaxK];  // per target slot: node index of the predecessor on that qubit, -1 if none
    int next[kMaxK];
};

int slot_of(const Node& nd, int qubit)
{
    for (int j = 0; j < nd.g.k; ++j)
        if (nd.g.q[j] == qubit) return j;
    return -1;
}

// Kahn's algorithm; ties broken by the smallest member circuit index (deterministic).
std::vector<int> topo_order(const std::vector<Node>& nodes)
{
    const int N = (int)nodes.size();
    std::vector<int> indeg(N, 0);
    for (int i = 0; i < N; ++i) {
        if (!nodes[i].alive) continue;
        int seen[kMaxK], ns = 0;
        for (int j = 0; j < nodes[i].g.k; ++j) {
            const int p = nodes[i].prev[j];
            if (p < 0) continue;
            bool dup = false;
            for (int s = 0; s < ns; ++s) dup |= seen[s] == p;
            if (!dup) seen[ns++] = p;
        }
        indeg[i] = ns;
    }
    using Item = std::pair<int, int>;  // (first, node)
    std::priority_queue<Item, std::vector<Item>, std::greater<Item>> ready;
    for (int i = 0; i < N; ++i)
        if (nodes[i].alive && indeg[i] == 0) ready.push({nodes[i].g.first, i});
    std::vector<int> order;
    order.reserve(N);
    while (!ready.empty()) {
        const int u = ready.top().second;
        ready.pop();
        order.push_back(u);
        int seen[kMaxK], ns = 0;
        for (int j = 0; j < nodes[u].g.k; ++j) {
            const int s = nodes[u].next[j];
            if (s < 0) continue;
            bool dup = false;
            for (int t = 0; t < ns; ++t) dup |= seen[t] == s;
            if (dup) continue;
            seen[ns++] = s;
            if (--indeg[s] == 0) ready.push({nodes[s].g.first, s});
        }
    }
    return order;
}

// Products formed while a plan is made, by their factors' ids: the planner fuses a circuit
// twice (on two DAGs) and most merges are the same.  They are kept without their member lists
// (a chain of G gates on few qubits has G products of up to G members) and up to kKeepBytes
// of matrices; beyond that they are dropped and later ones formed again.
struct Products {
    static constexpr size_t kKeepBytes = 64u << 20;
    std::unordered_map<unsigned long long, FGate> made;
    size_t bytes = 0;
    int next = 0;   // id of the next product

    void keep(unsigned long long key, const FGate& f)   // (f.mem still empty)
    {
        const size_t b = sizeof(FGate) + f.m.size() * sizeof(cd);
        if (bytes + b > kKeepBytes) {
            made.clear();
            bytes = 0;
        }
        made.emplace(key, f);
        bytes += b;
    }
};

FGate fuse_pair(const FGate& u, const FGate& v, int kmax, bool& ok, Products& pr)
{
    const unsigned long long key = ((unsigned long long)(unsigned)u.id << 32) | (unsigned)v.id;
    FGate f;
    const auto hit = pr.made.find(key);
    if (hit != pr.made.end()) {
        ok = hit->second.k <= kmax;
        if (!ok) return FGate{};
        f = hit->second;
    } else {
        int Q[2 * kMaxK], kq = 0;
        for (int j = 0; j < u.k; ++j) Q[kq++] = u.q[j];
        for (int j = 0; j < v.k; ++j) {
            bool dup = false;
            for (int i = 0; i < u.k; ++i) dup |= (u.q[i] == v.q[j]);
            if (!dup) Q[kq++] = v.q[j];
        }
        ok = kq <= kmax;
        if (!ok) return FGate{};
        std::sort(Q, Q + kq);
        f.k = kq;
        for (int j = 0; j < kq; ++j) f.q[j] = Q[j];
        // Eq. 9: U_fused = U_v . U_u (u applied first)
        f.m = embedded_product(v, u, Q, kq);
        inspect(f);
        f.id = pr.next++;
        f.first = std::min(u.first, v.first);
        f.members = u.members + v.members;
        pr.keep(key, f);
    }
    f.mem.reserve(u.mem.size() + v.mem.size());
    f.mem.insert(f.mem.end(), u.mem.begin(), u.mem.end());
    f.mem.insert(f.mem.end(), v.mem.begin(), v.mem.end());
    return f;
}

void run_fusion(std::vector<Node>& nodes, const PlanOpts& o, Products& pr)
{
    const int N = (int)nodes.size();
    std::vector<int> pos(N, 0);
    bool changed = true;
    while (changed) {
        changed = false;
        const std::vector<int> order = topo_order(nodes);
        for (int i = 0; i < (int)order.size(); ++i) pos[order[i]] = i;
        for (const int v : order) {
            if (!nodes[v].alive) continue;
            // distinct predecessors of v, nearest (latest in the order) first
            int preds[kMaxK], np = 0;
            for (int j = 0; j < nodes[v].g.k; ++j) {
                const int p = nodes[v].prev[j];
                if (p < 0) continue;
                bool dup = false;
                for (int s = 0; s < np; ++s) dup |= preds[s] == p;
                if (!dup) preds[np++] = p;
            }
            std::sort(preds, preds + np, [&](int a, int b) { return pos[a] > pos[b]; });
            for (int pi = 0; pi < np; ++pi) {
                const int u = preds[pi];
                Node& U = nodes[u];
                Node& V = nodes[v];
                // (3) u is v's predecessor on every shared qubit
                bool sole = true;
                for (int j = 0; j < V.g.k && sole; ++j)
                    if (slot_of(U, V.g.q[j]) >= 0 && V.prev[j] != u) sole = false;
                if (!sole) continue;
                // (4) acyclicity, by rule A (other preds of v precede u) or
                //     rule B (other succs of u follow v)
                bool ruleA = true, ruleB = true;
                for (int j = 0; j < V.g.k; ++j) {
                    const int p = V.prev[j];
                    if (p >= 0 && p != u && pos[p] > pos[u]) ruleA = false;
                }
                for (int j = 0; j < U.g.k; ++j) {
                    const int s = U.next[j];
                    if (s >= 0 && s != v && pos[s] < pos[v]) ruleB = false;
                }
                if (!ruleA && !ruleB) continue;
                // (2) width, checked before any product is formed
                {
                    unsigned long long qm = 0;
                    for (int j = 0; j < U.g.k; ++j) qm |= 1ull << U.g.q[j];
                    for (int j = 0; j < V.g.k; ++j) qm |= 1ull << V.g.q[j];
                    const int kq = __builtin_popcountll(qm);
                    if (kq > o.kmax) continue;
                    // (5), predicted: a product with a dense factor is dense (exact
                    // cancellation to a cheaper kind is rare and only costs a missed merge)
                    if (o.cost_aware > 0 && (U.g.kind == OP_DENSE || V.g.kind == OP_DENSE)) {
                        FGate probe;
                        probe.k = kq;
                        probe.kind = OP_DENSE;
                        if (op_cost(probe, o) > op_cost(U.g, o) + op_cost(V.g, o) + o.sigma) continue;
                    }
                }
                bool ok = false;
                FGate f = fuse_pair(U.g, V.g, o.kmax, ok, pr);
                if (!ok) continue;
                // (5) arithmetic does not grow beyond what the merge saves
                if (o.cost_aware > 0 && op_cost(f, o) > op_cost(U.g, o) + op_cost(V.g, o) + o.sigma) continue;
                // merge v into u: relink the per-qubit lines
                int nprev[kMaxK], nnext[kMaxK];
                for (int j = 0; j < f.k; ++j) {
                    const int x = f.q[j];
                    const int su = slot_of(U, x), sv = slot_of(V, x);
                    if (su >= 0 && sv >= 0) {
                        nprev[j] = U.prev[su];
                        nnext[j] = V.next[sv];
                    } else if (su >= 0) {
                        nprev[j] = U.prev[su];
                        nnext[j] = U.next[su];
                    } else {
                        nprev[j] = V.prev[sv];
                        nnext[j] = V.next[sv];
                    }
                }
                for (int j = 0; j < f.k; ++j) {
                    const int x = f.q[j];
                    if (nprev[j] >= 0) {
                        Node& P = nodes[nprev[j]];
                        P.next[slot_of(P, x)] = u;
                    }
                    if (nnext[j] >= 0) {
                        Node& S = nodes[nnext[j]];
                        S.prev[slot_of(S, x)] = u;
                    }
                }
                U.g = std::move(f);
                for (int j = 0; j < U.g.k; ++j) {
                    U.prev[j] = nprev[j];
                    U.next[j] = nnext[j];
                }
                V.alive = false;
                if (!ruleA) pos[u] = pos[v];  // rule B: the fused node takes v's slot
                changed = true;
                break;
            }
        }
    }
}

// ---- commutation-aware DAG and fusion (option commute)
//
// Two ops commute when they are both diagonal on every qubit they share, so among the
// ops touching a qubit q only the order between a run of ops diagonal on q and the op
// not diagonal on q that ends the run matters.  The DAG below keeps exactly those
// per-qubit edges: an op diagonal on q depends on the last op not diagonal on q; an op
// not diagonal on q depends on every op of the diagonal run before it (or, without
// one, on the previous op not diagonal on q).  Every pair of ops that may not commute
// is then joined by a path, so any topological order applies the circuit's operator.
//
// Fusion follows the sweep of Algorithm 2 on this DAG.  Its candidates for v are v's
// DAG predecessors and, on each qubit of v, the nearest earlier ops that commute with v
// there (they have no edge to v: a diagonal run); a merge needs the width bound, rule
// A or rule B (either one rules out any path u ~> v besides a direct edge, which also
// makes u and v commute when they have no edge, so the product order U_v . U_u is
// right either way) and, in cost-aware mode, the arithmetic condition.
struct CNode {
    FGate g;
    bool alive = true;
    unsigned long long qm = 0;
    std::vector<int> pred, succ;
};

unsigned long long qubit_mask(const FGate& g)
{
    unsigned long long m = 0;
    for (int j = 0; j < g.k; ++j) m |= 1ull << g.q[j];
    return m;
}

void add_edge(std::vector<CNode>& N, int a, int b)
{
    if (a < 0 || a == b) return;
    std::vector<int>& s = N[a].succ;
    if (std::find(s.begin(), s.end(), b) != s.end()) return;
    s.push_back(b);
    N[b].pred.push_back(a);
}

// Kahn's algorithm over the edge lists; ties broken by the smallest member index.
std::vector<int> topo_order_dag(const std::vector<CNode>& N)
{
    const int G = (int)N.size();
    std::vector<int> indeg(G, 0);
    using Item = std::pair<int, int>;
    std::priority_queue<Item, std::vector<Item>, std::greater<Item>> ready;
    for (int i = 0; i < G; ++i) {
        if (!N[i].alive) continue;
        indeg[i] = (int)N[i].pred.size();
        if (indeg[i] == 0) ready.push({N[i].g.first, i});
    }
    std::vector<int> order;
    order.reserve(G);
    while (!ready.empty()) {
        const int u = ready.top().second;
        ready.pop();
        order.push_back(u);
        for (const int s : N[u].succ)
            if (--indeg[s] == 0) ready.push({N[s].g.first, s});
    }
    return order;
}

// In node x's list, replace `from` by `to` (dropping `from` when `to` is already there).
void relink(std::vector<int>& lst, int from, int to)
{
    const bool has_to = std::find(lst.begin(), lst.end(), to) != lst.end();
    for (size_t i = 0; i < lst.size(); ++i) {
        if (lst[i] != from) continue;
        if (has_to) lst.erase(lst.begin() + (long)i);
        else lst[i] = to;
        return;
    }
}

std::vector<FGate> fuse_commuting(std::vector<FGate> gates, int n, const PlanOpts& o, bool diag_only, Products& pr)
{
    const int G = (int)gates.size();
    std::vector<CNode> N(G);
    {
        std::vector<int> last_nd(n, -1);
        std::vector<std::vector<int>> run(n);
        for (int i = 0; i < G; ++i) {
            N[i].g = std::move(gates[i]);
            const FGate& gi = N[i].g;
            N[i].qm = qubit_mask(gi);
            for (int j = 0; j < gi.k; ++j) {
                const int q = gi.q[j];
                if ((gi.dq >> q) & 1) {
                    add_edge(N, last_nd[q], i);
                    run[q].push_back(i);
                } else {
                    if (run[q].empty()) add_edge(N, last_nd[q], i);
                    for (const int r : run[q]) add_edge(N, r, i);
                    run[q].clear();
                    last_nd[q] = i;
                }
            }
        }
    }
    constexpr int kWindow = 8;   // commuting candidates examined per qubit of v
    std::vector<int> pos(G, 0);
    std::vector<std::vector<int>> lines(n);
    std::vector<int> at((size_t)G * kMaxK, -1), atq((size_t)G * kMaxK, -1);
    bool changed = true;
    while (changed) {
        changed = false;
        const std::vector<int> order = topo_order_dag(N);
        for (int i = 0; i < (int)order.size(); ++i) pos[order[i]] = i;
        // per-qubit lists of the live ops in this sweep's order
        for (auto& l : lines) l.clear();
        for (const int v : order)
            for (int j = 0; j < N[v].g.k; ++j) {
                const int q = N[v].g.q[j];
                atq[(size_t)v * kMaxK + j] = q;
                at[(size_t)v * kMaxK + j] = (int)lines[q].size();
                lines[q].push_back(v);
            }
        const std::vector<int> snapshot_k = [&] {
            std::vector<int> k(G, 0);
            for (const int v : order) k[v] = N[v].g.k;
            return k;
        }();
        std::vector<int> cand;
        for (const int v : order) {
            if (!N[v].alive) continue;
            cand.assign(N[v].pred.begin(), N[v].pred.end());
            for (int j = 0; j < snapshot_k[v]; ++j) {
                const int q = atq[(size_t)v * kMaxK + j];
                const std::vector<int>& line = lines[q];
                int seen = 0;
                for (int t = at[(size_t)v * kMaxK + j] - 1; t >= 0 && seen < kWindow; --t) {
                    const int u = line[t];
                    if (!N[u].alive || u == v || !((N[u].qm >> q) & 1)) continue;
                    ++seen;
                    cand.push_back(u);
                    if (!ops_commute(N[u].g, N[v].g)) break;   // ops further back are ordered before u
                }
            }
            std::sort(cand.begin(), cand.end());
            cand.erase(std::unique(cand.begin(), cand.end()), cand.end());
            std::sort(cand.begin(), cand.end(), [&](int a, int b) { return pos[a] > pos[b]; });
            for (const int u : cand) {
                CNode& U = N[u];
                CNode& V = N[v];
                if (!U.alive || u == v || pos[u] >= pos[v] || !(U.qm & V.qm)) continue;
                if (diag_only && (U.g.kind != OP_DIAG || V.g.kind != OP_DIAG)) continue;
                const int kq = __builtin_popcountll(U.qm | V.qm);
                if (kq > o.kmax) continue;
                bool ruleA = true, ruleB = true;
                for (const int p : V.pred)
                    if (p != u && pos[p] > pos[u]) { ruleA = false; break; }
                for (const int sx : U.succ)
                    if (sx != v && pos[sx] < pos[v]) { ruleB = false; break; }
                if (!ruleA && !ruleB) continue;
                if (o.cost_aware > 0 && (U.g.kind == OP_DENSE || V.g.kind == OP_DENSE)) {
                    FGate probe;
                    probe.k = kq;
                    probe.kind = OP_DENSE;
                    if (op_cost(probe, o) > op_cost(U.g, o) + op_cost(V.g, o) + o.sigma) continue;
                }
                bool ok = false;
                FGate f = fuse_pair(U.g, V.g, o.kmax, ok, pr);
                if (!ok) continue;
                if (o.cost_aware > 0 && op_cost(f, o) > op_cost(U.g, o) + op_cost(V.g, o) + o.sigma) continue;
                // merge v into u: u takes v's edges
                for (const int p : V.pred) {
                    if (p == u) continue;
                    relink(N[p].succ, v, u);
                    if (std::find(U.pred.begin(), U.pred.end(), p) == U.pred.end()) U.pred.push_back(p);
                }
                for (const int sx : V.succ) {
                    relink(N[sx].pred, v, u);
                    if (std::find(U.succ.begin(), U.succ.end(), sx) == U.succ.end()) U.succ.push_back(sx);
                }
                U.succ.erase(std::remove(U.succ.begin(), U.succ.end(), v), U.succ.end());
                U.g = std::move(f);
                U.qm = qubit_mask(U.g);
                V.alive = false;
                V.pred.clear();
                V.succ.clear();
                if (!ruleA) pos[u] = pos[v];   // rule B: the fused op takes v's slot
                changed = true;
                break;
            }
        }
    }
    std::vector<FGate> out;
    for (const int v : topo_order_dag(N)) out.push_back(std::move(N[v].g));
    return out;
}

// Floats of a matrix-core op's staged operand (a complex64 3-qubit op is run as a 4-qubit
// one; complex128's real embedding doubles a 3-qubit matrix).
int operand_floats(int dtype, int k)
{
    return dtype == 1 && k == 4 ? 1024 : 512;
}

// What scheduling asks of an op.
struct OpInfo {
    unsigned long long gm, gd;   // its qubits; those it is diagonal on (commutation-aware plans)
    double cost;                 // op_cost plus the per-op overhead
    int floats;                  // operand or diagonal-table floats to stage
    bool matrix, diag;           // on matrix cores; diagonal
};

std::vector<OpInfo> op_infos(const std::vector<FGate>& fused, const PlanOpts& o)
{
    std::vector<OpInfo> v;
    v.reserve(fused.size());
    for (const FGate& g : fused) {
        OpInfo i;
        i.gm = qubit_mask(g);
        i.gd = o.commute ? g.dq : 0;
        i.cost = op_cost(g, o) + o.sigma;
        i.matrix = mfma_eligible(g, o);
        i.diag = g.kind == OP_DIAG;
        i.floats = i.matrix ? operand_floats(o.fp32_mfma ? 0 : 1, g.k) : i.diag ? o.amp_floats << g.k : 0;
        v.push_back(i);
    }
    return v;
}

// One pass built greedily from the ops not yet done (in their order).  grow: the tile
// starts as `A0` and takes the qubits of every op that joins, up to m; otherwise the
// tile is exactly `A0` and only ops inside it (or diagonal ops) join.  An op joins when
// none of its qubits is blocked by an earlier deferred op it may not commute with, the
// tile holds it and the pass's arithmetic budget and staged block allow.
PassPlan build_pass(int n, const std::vector<OpInfo>& ops, const std::vector<int>& todo, const PlanOpts& o,
                    int m, int L, bool whole, unsigned long long A0, bool grow)
{
    const unsigned long long all = (n >= 64) ? ~0ull : ((1ull << n) - 1);
    PassPlan pp;
    int Lp = L;   // low qubits kept in this pass's tile
    unsigned long long A = whole ? all : A0;
    // qubits of deferred ops: where some deferred op is not diagonal (blocked), and
    // where all of them are (blocked_d).  A later op may run ahead of the deferred
    // ones when it touches no blocked qubit and is itself diagonal on every
    // blocked_d qubit it touches: it then commutes with each of them.
    unsigned long long blocked = 0, blocked_d = 0;
    auto defer = [&](unsigned long long gm, unsigned long long gd) {
        blocked |= gm & ~gd;
        blocked_d |= gm & gd;
        blocked_d &= ~blocked;
    };
    double budget = o.pass_budget;
    // Operands need to be in LDS only where a pass loads its next tile during the ops;
    // elsewhere they come through L2 and only the budget ends a pass.  A plan does not say
    // whether its launches cover one state or two (the adjoint's), so the line is where two
    // would load ahead.  Capped and not, 8-layer ansatz: 22 qubits complex128 12 and 6
    // passes, 523 and 405 us, complex64 10 and 8, 242 and 223 us; 18 qubits complex128 136
    // and 123 us; complex64 at 14, 16 and 19 qubits 66 and 55, 79 and 71, 109 and 98 us (12
    // layers of brickwork 58 and 54, 75 and 70, 97 and 100).
    const bool ahead = loads_ahead(m, L, 2ll << (n - m), kPlanCUs);
    const int cap = o.pass_floats > 0 ? o.pass_floats : ahead ? o.stage_floats : kNoPassCap;
    int afl = 0;   // floats of the pass's block so far
    for (const int i : todo) {
        const OpInfo& g = ops[(size_t)i];
        const unsigned long long gm = g.gm, gd = g.gd;
        if ((gm & blocked) || (gm & ~gd & blocked_d)) {
            defer(gm, gd);
            if ((blocked & all) == all) break;
            continue;
        }
        const double c = g.cost;
        const bool limit_ops = o.max_ops_per_pass > 0 && (int)pp.ops.size() >= o.max_ops_per_pass;
        // a matrix-core op whose operand no longer fits the pass's block waits for the next
        // pass: with one operand in global memory the pass could not load ahead.  A diagonal op
        // joins with its table outside the block if need be (build_device_tables)
        const int af = g.floats;
        const bool fits_operands = whole || !g.matrix || ((afl + 3) & ~3) + af <= cap || pp.ops.empty();
        const bool fits_budget = whole || o.pass_budget < 0 || c <= budget || pp.ops.empty();
        unsigned long long nA = g.diag ? A : (A | gm);
        if (grow && pp.ops.empty() && __builtin_popcountll(nA) > m) {
            // a gate wider than the tile's free slots opens a pass with fewer low qubits
            while (Lp > 0 && __builtin_popcountll(gm | ((1ull << Lp) - 1)) > m) --Lp;
            A = (1ull << Lp) - 1;
            nA = A | gm;
        }
        const bool fits_tile = grow ? __builtin_popcountll(nA) <= m : nA == A;
        if (!limit_ops && fits_budget && fits_operands && fits_tile) {
            A = nA;
            pp.ops.push_back(i);
            budget -= c;
            pp.cost += c;
            if (af > 0 && ((afl + 3) & ~3) + af <= cap) afl = ((afl + 3) & ~3) + af;
        } else {
            defer(gm, gd);
            if ((blocked & all) == all) break;
        }
    }
    // fill the tile up to m qubits with the lowest unused qubits (longer runs)
    for (int b = 0; b < n && __builtin_popcountll(A) < m; ++b) A |= 1ull << b;
    for (int b = 0; b < n; ++b)
        if ((A >> b) & 1) pp.active.push_back(b);
    pp.low = Lp;
    return pp;
}

// Diagonal ops on disjoint qubits share no DAG edge, so fusion leaves them apart, yet
// they commute and their product is again diagonal, costing one complex multiply per
// amplitude like each of them (a layer of single-qubit phase rotations would otherwise
// cost one on-chip round trip per qubit).  Walking the fused list in order, a diagonal
// op moves back past every op it commutes with to the nearest earlier diagonal op whose
// union with it stays within the width bound, and the two become one.  Moving it back
// is exact: it commutes with every op it passes.
void merge_diagonals(std::vector<FGate>& ops, int kmax, Products& pr)
{
    constexpr int kWindow = 64;   // earlier ops examined per diagonal op
    std::vector<FGate> out;
    out.reserve(ops.size());
    for (FGate& v : ops) {
        if (v.kind == OP_DIAG) {
            const unsigned long long qv = qubit_mask(v);
            int hit = -1;
            for (int t = (int)out.size() - 1, seen = 0; t >= 0 && seen < kWindow; --t, ++seen) {
                const FGate& u = out[(size_t)t];
                if (u.kind == OP_DIAG && __builtin_popcountll(qubit_mask(u) | qv) <= kmax) {
                    hit = t;
                    break;
                }
                if (!ops_commute(u, v)) break;
            }
            if (hit >= 0) {
                bool ok = false;
                FGate f = fuse_pair(out[(size_t)hit], v, kmax, ok, pr);
                if (ok && f.kind == OP_DIAG) {
                    out[(size_t)hit] = std::move(f);
                    continue;
                }
            }
        }
        out.push_back(std::move(v));
    }
    ops.clear();
    for (FGate& g : out)
        if (!is_identity(g)) ops.push_back(std::move(g));
}

// An op that can be one of a pair (kernels.hip): a 4-qubit matrix-core op, complex64
// 3-qubit ones too (they are run as 4-qubit ops).
bool pairable(const FGate& g, const PlanOpts& o)
{
    return mfma_eligible(g, o) && (g.k == 4 || o.fp32_mfma);
}

// Order a pass's ops so that ops which can run as a pair are neighbours: an op moves up
// behind an earlier one when it shares no qubit with it or with any op in between (then
// it commutes with each of them exactly).
void pair_up(const std::vector<FGate>& fused, const PlanOpts& o, PassPlan& pp)
{
    std::vector<int> rest(pp.ops), out;
    while (!rest.empty()) {
        const FGate& a = fused[(size_t)rest[0]];
        unsigned long long seen = qubit_mask(a);
        size_t hit = 0;
        if (pairable(a, o)) {
            for (size_t i = 1; i < rest.size() && !hit; ++i) {
                const FGate& b = fused[(size_t)rest[i]];
                const unsigned long long qb = qubit_mask(b);
                if (!(qb & seen) && pairable(b, o)) hit = i;
                seen |= qb;
            }
        }
        out.push_back(rest[0]);
        if (hit) {
            out.push_back(rest[hit]);
            rest.erase(rest.begin() + (long)hit);
        }
        rest.erase(rest.begin());
    }
    pp.ops.swap(out);
}

// Pass scheduling.  Each pass is the best of several greedy candidates: the tile that
// grows with the ops in their order, and tiles fixed in advance to the low L qubits
// plus m - L consecutive others (every window position).  The fixed windows follow the
// locality of nearest-neighbour circuits: within a window an op can run several layers
// ahead of the ops outside it, where the growing tile stops at the first op that
// straddles its edge.  "Best" is the most arithmetic (plus per-op overhead) done, the
// growing tile winning ties; it always makes progress.
bool schedule_passes(int n, const std::vector<FGate>& fused, const PlanOpts& o, std::vector<PassPlan>& passes,
                     std::string& err)
{
    passes.clear();
    const int F = (int)fused.size();
    const bool whole = o.fuse && n <= o.whole_state_max;
    const int m = whole ? n : std::min(o.tile_qubits, n);
    const int L = std::min(o.low_qubits, m);
    const unsigned long long low = (L >= 64) ? ~0ull : ((1ull << L) - 1);
    const bool windows = !whole && o.fuse == 1 && n > m && m > L;
    const std::vector<OpInfo> ops = op_infos(fused, o);
    std::vector<int> todo(F);
    for (int i = 0; i < F; ++i) todo[i] = i;
    std::vector<char> done(F, 0);
    while (!todo.empty()) {
        PassPlan best = build_pass(n, ops, todo, o, m, L, whole, low, true);
        if (windows) {
            const int w = m - L;
            for (int a = L; a + w <= n; ++a) {
                const unsigned long long A0 = low | (((1ull << w) - 1) << a);
                PassPlan c = build_pass(n, ops, todo, o, m, L, whole, A0, false);
                if (c.cost > best.cost) best = std::move(c);
            }
        }
        if (best.ops.empty()) { err = "internal: a gate does not fit any tile"; return false; }
        for (const int i : best.ops) done[i] = 1;
        todo.erase(std::remove_if(todo.begin(), todo.end(), [&](int i) { return done[(size_t)i] != 0; }), todo.end());
        pair_up(fused, o, best);
        passes.push_back(std::move(best));
    }
    return true;
}

// ---- operand tables of matrix-core ops (kernels.hip: op_mfma4, op_mfma3)

// LDS position of tile element e (kernels.hip: swz).
int tile_slot(int dtype, int e)
{
    if (dtype == 0) return e ^ ((e >> 5) & 31) ^ (e >> 10);
    return e ^ ((e >> 4) & 15) ^ ((e >> 8) & 15);
}

// Rank over XOR of the bank bits of a set of tile bits: lanes that run over independent
// bits fall in different LDS banks.
int bank_rank(int dtype, const int* bits, int count)
{
    const int mask = dtype == 0 ? 31 : 15;
    int basis[5] = {0, 0, 0, 0, 0}, rank = 0;
    for (int i = 0; i < count; ++i) {
        int v = tile_slot(dtype, 1 << bits[i]) & mask;
        for (int b = 4; b >= 0 && v; --b) {
            if (!((v >> b) & 1)) continue;
            if (!basis[b]) {
                basis[b] = v;
                ++rank;
                v = 0;
            } else {
                v ^= basis[b];
            }
        }
    }
    return rank;
}

// A 4-qubit op's basis state held by lane group q in its j-th register: which of the op's
// local bits run over q and over j.
struct Spread {
    int q0 = 0, q1 = 1, j0 = 2, j1 = 3;
    int state(int q, int j) const
    {
        return ((q & 1) << q0) | ((q >> 1) << q1) | ((j & 1) << j0) | ((j >> 1) << j1);
    }
};

Spread spread_from(int q0)
{
    Spread s;
    int rest[3], k = 0;
    for (int i = 0; i < 4; ++i)
        if (i != q0) rest[k++] = i;
    s.q0 = q0;
    s.q1 = rest[0];
    s.j0 = rest[1];
    s.j1 = rest[2];
    return s;
}

// The local bit of `t` that lane group bit 0 runs over, best for the banks with the four
// tile bits that lane % 16 runs over.
int best_q0(int dtype, const int* t, const int* lane16)
{
    int best = 0, rank = -1;
    for (int i = 0; i < 4; ++i) {
        const int bits[5] = {lane16[0], lane16[1], lane16[2], lane16[3], t[i]};
        const int r = bank_rank(dtype, bits, 5);
        if (r > rank) { rank = r; best = i; }
    }
    return best;
}

// Appends one 4-qubit operand: lane 16 q + m feeds row row(m) of M, columns col(q, j); its
// four complex entries in the state's precision, in 16-byte units a wave's lanes apart.
template <typename Row, typename Col>
void push_operand(std::vector<float>& out, int dtype, const std::vector<cd>& M, Row row, Col col)
{
    const size_t at = out.size();
    out.resize(at + (dtype == 0 ? 512 : 1024));
    int cols[4][4];
    for (int q = 0; q < 4; ++q)
        for (int j = 0; j < 4; ++j) cols[q][j] = col(q, j);
    for (int l = 0; l < 16; ++l) {
        const cd* mrow = &M[(size_t)row(l) * 16];
        for (int q = 0; q < 4; ++q)
            for (int j = 0; j < 4; ++j) {
                const cd& v = mrow[cols[q][j]];
                const int lane = 16 * q + l;
                if (dtype == 0) {
                    float* w = &out[at + (size_t)((j >> 1) * 64 + lane) * 4 + 2 * (j & 1)];
                    w[0] = (float)v.real();
                    w[1] = (float)v.imag();
                } else {
                    const double w[2] = {v.real(), v.imag()};
                    std::memcpy(&out[at + (size_t)(j * 64 + lane) * 4], w, 16);
                }
            }
    }
}

// What a matrix-core op multiplies: its matrix over the tile bits lpos.
struct Operand {
    int k = 0, lpos[4];
    std::vector<cd> own;             // a widened matrix
    const std::vector<cd>* m = nullptr;

    const std::vector<cd>& matrix() const { return m ? *m : own; }
    unsigned bits() const
    {
        unsigned b = 0;
        for (int j = 0; j < k; ++j) b |= 1u << lpos[j];
        return b;
    }
};

// The operand of gate g in pass pp.  A complex64 3-qubit one gains one more tile qubit, not in
// `avoid` (and put there), as identity.
Operand operand_of(int dtype, const FGate& g, const PassPlan& pp, unsigned long long& avoid)
{
    Operand o;
    o.k = g.k;
    int Q[4] = {g.q[0], g.q[1], g.q[2], g.q[3]};
    if (dtype == 0 && g.k == 3) {
        for (const int b : pp.active)
            if (!((avoid >> b) & 1)) { Q[3] = b; break; }
        avoid |= 1ull << Q[3];
        std::sort(Q, Q + 4);
        o.k = 4;
        o.own = embed(g.m.vec(), g.q, 3, Q, 4);
    } else {
        o.m = &g.m.vec();
    }
    for (int j = 0; j < o.k; ++j)
        o.lpos[j] = (int)(std::find(pp.active.begin(), pp.active.end(), Q[j]) - pp.active.begin());
    return o;
}

// Operand and offset tables of the matrix-core op d (operand u), or of the pair (d, d2) of
// operands u and u2, appended to the plan's operand array; m: the tile's bits.
// wave: the two tile bits that tell the waves apart, none of the targets.
void mfma_tables(int dtype, int m, DevOp& d, const Operand& u, DevOp* d2, const Operand* u2, const int (&wave)[2],
                 std::vector<float>& out)
{
    const std::vector<cd>& M = u.matrix();
    const int eb = dtype == 0 ? 8 : 16;
    auto off = [&](int e) { return tile_slot(dtype, e) * eb; };
    // the matrix instruction's result row held by lane group q in register e, and back
    auto drow = [&](int q, int e) { return dtype == 0 ? 4 * q + e : 4 * e + q; };
    auto dq = [&](int r) { return dtype == 0 ? r >> 2 : r & 3; };
    auto de = [&](int r) { return dtype == 0 ? r & 3 : r >> 2; };
    unsigned used = u.bits() | (d2 ? u2->bits() : 0);
    int col[4];   // tile bits that lane % 16 runs over in the reads
    if (d2) {
        for (int i = 0; i < 4; ++i) col[i] = u2->lpos[i];
    } else {
        int nc = 0;   // independent bank bits first, then any; the wave bits only if nothing else is left
        const unsigned keep = (1u << wave[0]) | (1u << wave[1]);
        for (int pass = 0; pass < 3; ++pass)
            for (int b = 0; b < m && nc < 4; ++b) {
                if ((used >> b) & 1 || (pass < 2 && (keep >> b) & 1)) continue;
                col[nc] = b;
                if (pass == 0 && bank_rank(dtype, col, nc + 1) <= nc) continue;
                used |= 1u << b;
                ++nc;
            }
    }
    while (out.size() & 3) out.push_back(0.0f);
    d.goff = (int)out.size();
    auto bit = [&](int b) { return (unsigned)off(1 << b); };
    auto pack = [](unsigned* w, int i, unsigned v) { w[i >> 1] |= v << (16 * (i & 1)); };
    // lane bits 0-3 run over the tile bits c, bits 4-5 and j over the op's local bits in S
    auto lanes = [&](DevOp& o, const int* c, const Spread& S, const int* t) {
        for (int i = 0; i < 4; ++i) pack(o.lin, i, bit(c[i]));
        pack(o.lin, 4, bit(t[S.q0]));
        pack(o.lin, 5, bit(t[S.q1]));
        pack(&o.jbit, 0, bit(t[S.j0]));
        pack(&o.jbit, 1, bit(t[S.j1]));
    };
    if (u.k == 3) {
        // the real embedding: input column 4 ks + q is the real (ks even) or imaginary part
        // of complex input 4 (ks / 2) + q; matrix row i of the FP64 instruction comes back
        // as element i / 4 of lane group i % 4, and stands for complex row 2 (i % 4) + i / 8,
        // real or imaginary by (i / 4) % 2
        const size_t at = out.size();
        out.resize(at + 512);
        for (int lane = 0; lane < 64; ++lane) {
            const int q = lane >> 4, i = lane & 15, r = 2 * (i & 3) + (i >> 3);
            for (int j = 0; j < 2; ++j) {
                const cd u = M[(size_t)r * 8 + 4 * j + q];
                const double w[2] = {(i >> 2) & 1 ? u.imag() : u.real(), (i >> 2) & 1 ? u.real() : -u.imag()};
                std::memcpy(&out[at + (size_t)(j * 64 + lane) * 4], w, 16);
            }
        }
        for (int i = 0; i < 4; ++i) {
            pack(d.lin, i, bit(col[i]));
            pack(d.lout, i, bit(col[i]));
        }
        for (int i = 0; i < 2; ++i) {
            pack(d.lin, 4 + i, bit(u.lpos[i]));        // rows 4 j + q
            pack(d.lout, 4 + i, bit(u.lpos[1 + i]));   // rows 2 q + j
        }
        pack(&d.jbit, 0, bit(u.lpos[2]));
        pack(&d.jbit, 1, bit(u.lpos[0]));
    } else if (!d2) {
        const Spread S = spread_from(best_q0(dtype, u.lpos, col));
        push_operand(out, dtype, M, [&](int r) { return S.state(dq(r), de(r)); },
                     [&](int q, int j) { return S.state(q, j); });
        lanes(d, col, S, u.lpos);
    } else {
        // reads: lane % 16 is the second op's state, (q, j) the first's (S1); after the
        // first product lane % 16 is the first op's new state and (q, e) the second's,
        // drow(q, e); after the second (q, e) is its new state by S2
        const Spread S1 = spread_from(best_q0(dtype, u.lpos, u2->lpos));
        const Spread S2 = spread_from(best_q0(dtype, u2->lpos, u.lpos));
        push_operand(out, dtype, M, [&](int r) { return r; }, [&](int q, int j) { return S1.state(q, j); });
        lanes(d, u2->lpos, S1, u.lpos);
        d2->goff = (int)out.size();
        push_operand(out, dtype, u2->matrix(), [&](int r) { return S2.state(dq(r), de(r)); },
                     [&](int q, int j) { return drow(q, j); });
        lanes(*d2, u.lpos, S2, u2->lpos);
        d.flags = 1;
    }
    // the block number's bits: the tile bits that are left
    int nb = 0;
    for (const int b : wave)
        if (!((used >> b) & 1)) {
            used |= 1u << b;
            pack(d.bbit, nb++, bit(b));
        }
    for (int b = 0; b < m && nb < kMaxBlockBits; ++b)
        if (!((used >> b) & 1)) pack(d.bbit, nb++, bit(b));
}

// Matrix cores need 16 groups per block in a tile of 2^m amplitudes; complex64 3-qubit ops are
// run as 4-qubit ones on one more tile bit.
bool on_matrix_cores(const FGate& g, const PlanOpts& o, int dtype, int m)
{
    return mfma_eligible(g, o) && m >= (dtype == 0 ? 8 : g.k + 4);
}

// Device tables of a planned circuit (op descriptors, matrix pools, staged operand
// blocks, pass arguments) and the arithmetic statistics, from P.fused and P.passes.
void build_device_tables(HostPlan& P)
{
    const int n = P.n, dtype = P.dtype;
    const PlanOpts& o = P.o;
    P.ops.clear();
    P.pargs.clear();
    P.pgrid.clear();
    P.pwide.clear();
    P.pool.clear();
    P.ipool.clear();
    P.apool.clear();
    P.dense_ops = P.diag_ops = P.perm_ops = P.mfma_ops = 0;
    P.fma_per_amp = P.mfma_fma_per_amp = 0;
    for (const PassPlan& pp : P.passes) {
        PassArgs a{};
        a.m = (int)pp.active.size();
        a.L = pp.low;
        for (int i = 0; i < a.m; ++i) a.phys[i] = (unsigned char)pp.active[i];
        a.nruns = 0;
        {
            unsigned long long A = 0;
            for (int b : pp.active) A |= 1ull << b;
            int b = 0;
            while (b < n) {
                if ((A >> b) & 1) { ++b; continue; }
                int s = b;
                while (b < n && !((A >> b) & 1)) ++b;
                a.run_pos[a.nruns] = (unsigned char)s;
                a.run_len[a.nruns] = (unsigned char)(b - s);
                ++a.nruns;
            }
        }
        a.op_begin = (int)P.ops.size();
        a.op_count = (int)pp.ops.size();
        a.a_off = (int)P.apool.size();
        a.a_len = 0;
        std::vector<int> matrix_ops;   // this pass's matrix-core ops (indices into P.ops)
        // The block's floats that diagonal tables may take.  A pass loads ahead only with all
        // its matrix operands in the block, so where one state's tiles suffice for that they come
        // first and the tables take what they leave; a table read from global memory waits once
        // for the next tile's loads (27-qubit complex64 ansatz of 6 layers, five such passes of
        // ten: 6.00 -> 5.77 ms).  Other passes read their operands through L2, and the tables
        // have the whole block.
        int room = o.stage_floats;
        if (o.pass_floats == 0 && loads_ahead(a.m, a.L, 1ll << (n - a.m), kPlanCUs)) {
            int need = 0;
            for (const int fi : pp.ops)
                if (on_matrix_cores(P.fused[fi], o, dtype, a.m)) need += operand_floats(dtype, P.fused[fi].k);
            if (need <= room) room -= need;
        }
        for (const int fi : pp.ops) {
            const FGate& g = P.fused[fi];
            DevOp d{};
            d.kind = g.kind;
            d.k = g.k;
            for (int j = 0; j < kMaxK; ++j) { d.lpos[j] = -1; d.gbit[j] = 0; }
            for (int j = 0; j < g.k; ++j) {
                d.gbit[j] = g.q[j];
                auto it = std::find(pp.active.begin(), pp.active.end(), g.q[j]);
                d.lpos[j] = (it == pp.active.end()) ? -1 : (int)(it - pp.active.begin());
            }
            const int dd = 1 << g.k;
            d.off = (int)P.pool.size();
            d.aoff = d.goff = -1;
            if (g.kind == OP_DENSE) {
                ++P.dense_ops;
                if (on_matrix_cores(g, o, dtype, a.m)) {   // its operand is all it reads
                    matrix_ops.push_back((int)P.ops.size());
                    ++P.mfma_ops;
                    P.mfma_fma_per_amp += op_fma(g);
                } else {
                    P.pool.insert(P.pool.end(), g.m.vec().begin(), g.m.vec().end());
                }
            } else if (g.kind == OP_DIAG) {
                for (int r = 0; r < dd; ++r) P.pool.push_back(g.m[(size_t)r * dd + r]);
                ++P.diag_ops;
                // the table also goes to LDS (per-lane lookups stay on chip): the entries
                // in the state's precision as raw floats, 16-byte aligned
                const int per = dtype == 0 ? 2 : 4;
                const int at = (a.a_len + 3) & ~3;
                if (at + per * dd <= room) {
                    P.apool.resize((size_t)a.a_off + at, 0.0f);
                    for (int r = 0; r < dd; ++r) {
                        const cd v = g.m[(size_t)r * dd + r];
                        if (dtype == 0) {
                            P.apool.push_back((float)v.real());
                            P.apool.push_back((float)v.imag());
                        } else {
                            const double re = v.real(), im = v.imag();
                            float w[4];
                            std::memcpy(w, &re, 8);
                            std::memcpy(w + 2, &im, 8);
                            P.apool.insert(P.apool.end(), w, w + 4);
                        }
                    }
                    d.aoff = at;
                    a.a_len = at + per * dd;
                }
            } else {
                d.ioff = (int)P.ipool.size();
                d.flags = 0;
                for (int r = 0; r < dd; ++r) {
                    int src = 0;
                    for (int c = 0; c < dd; ++c)
                        if (g.m[(size_t)r * dd + c] != cd(0, 0)) src = c;
                    const cd ph = g.m[(size_t)r * dd + src];
                    P.ipool.push_back(src);
                    P.pool.push_back(ph);
                    if (ph != cd(1, 0)) d.flags = 1;
                }
                ++P.perm_ops;
            }
            P.fma_per_amp += op_fma(g);
            P.ops.push_back(d);
        }
        a.d_len = a.a_len;
        // the matrix-core ops' operands, behind the pass's diagonal tables
        auto gate_of = [&](int oi) -> const FGate& { return P.fused[(size_t)pp.ops[(size_t)(oi - a.op_begin)]]; };
        struct Step {   // one op or one pair
            int oi, oj;
            Operand u, u2;
            unsigned bits() const { return u.bits() | u2.bits(); }
        };
        std::vector<Step> steps;
        for (size_t i = 0; i < matrix_ops.size(); ++i) {
            Step st;
            st.oi = matrix_ops[i];
            st.oj = -1;
            const FGate& g = gate_of(st.oi);
            const int oj = i + 1 < matrix_ops.size() ? matrix_ops[i + 1] : -1;
            if (oj == st.oi + 1 && pairable(g, o) && pairable(gate_of(oj), o) && !(qubit_mask(g) & qubit_mask(gate_of(oj))))
                st.oj = oj;
            unsigned long long avoid = qubit_mask(g) | (st.oj >= 0 ? qubit_mask(gate_of(st.oj)) : 0);
            st.u = operand_of(dtype, g, pp, avoid);
            if (st.oj >= 0) {
                st.u2 = operand_of(dtype, gate_of(st.oj), pp, avoid);
                ++i;
            }
            steps.push_back(std::move(st));
        }
        // runs of neighbouring steps whose targets leave two tile bits free: those bits tell
        // the waves apart in all of them, and no barrier is needed inside the run
        for (size_t i = 0; i < steps.size();) {
            unsigned bits = steps[i].bits();
            size_t e = i + 1;
            auto last = [&](const Step& x) { return x.oj >= 0 ? x.oj : x.oi; };
            while (e < steps.size() && steps[e].oi == last(steps[e - 1]) + 1 &&
                   a.m - __builtin_popcount(bits | steps[e].bits()) >= 2)
                bits |= steps[e++].bits();
            int wave[2] = {0, 0}, nw = 0;   // the two highest free bits: the lanes want the low ones
            for (int b = a.m - 1; b >= 0 && nw < 2; --b)
                if (!((bits >> b) & 1)) wave[nw++] = b;
            for (size_t x = i; x < e; ++x) {
                Step& st = steps[x];
                DevOp* d2 = st.oj >= 0 ? &P.ops[(size_t)st.oj] : nullptr;
                mfma_tables(dtype, a.m, P.ops[(size_t)st.oi], st.u, d2, d2 ? &st.u2 : nullptr, wave, P.apool);
                P.ops[(size_t)st.oi].nosync = nw == 2 && a.m >= 10 && x + 1 < e;
            }
            i = e;
        }
        for (const int oi : matrix_ops) {   // those that fit the staged block, in order
            DevOp& d = P.ops[(size_t)oi];
            const int at = d.goff - a.a_off, len = operand_floats(dtype, d.k);
            if (at + len > o.stage_floats) break;
            d.aoff = at;
            a.a_len = at + len;
        }
        a.staged = matrix_ops.empty() || P.ops[(size_t)matrix_ops.back()].aoff >= 0;
        {
            // complex128 passes with operands beyond the LDS block count as wide too: served,
            // these heavier passes then have a launch of their own (closed loop with the
            // precision chosen per request 366 against 350 circuits/s; a plain pass takes the
            // same time in either variant).  complex64 ones are faster in the lighter variant
            // (22-qubit brickwork 358 and 355 us, 70/30 mix 538 and 549 circuits/s).
            bool wide = false;
            for (int i = a.op_begin; i < a.op_begin + a.op_count; ++i) {
                const DevOp& d = P.ops[(size_t)i];
                wide |= (d.kind == OP_DENSE && (dtype == 0 ? d.goff : d.aoff) < 0 && d.k >= 4) || (d.kind == OP_PERM && d.k >= 3);
            }
            P.pwide.push_back(wide ? 1 : 0);
        }
        P.pargs.push_back(a);
        P.pgrid.push_back(1ll << (n - a.m));
    }
}

}  // namespace

bool make_plan(int n, int dtype, const std::vector<InGate>& gates, const PlanOpts& o,
               HostPlan& P, std::string& err)
{
    P = HostPlan();
    P.n = n;
    P.dtype = dtype;
    P.o = o;
    P.gates_in = gates.size();
    for (const InGate& g : gates) {
        P.shape.push_back(g.k);
        P.shape.insert(P.shape.end(), g.t, g.t + g.k);
    }
    if (o.kmax < 1 || o.kmax > kMaxK) { err = "kmax must be in [1, 5]"; return false; }
    if (o.low_qubits < 1 || o.low_qubits > kLogThreads) { err = "low_qubits must be in [1, 8]"; return false; }
    if (o.tile_qubits < o.low_qubits + 1 || o.tile_qubits < kMaxK + 1 || o.tile_qubits > kMaxTileQubits) {
        err = "tile_qubits must be in [max(low_qubits+1, 6), 13]";
        return false;
    }

    // ---- DAG (Section 5.1): immediate predecessor per qubit
    std::vector<Node> nodes(gates.size());
    std::vector<int> last(n, -1);
    Products pr;
    pr.next = (int)gates.size();
    pr.made.reserve(2 * gates.size());
    std::vector<FGate> canon;   // kept for the second fusion (the matrices are shared)
    canon.reserve(gates.size());
    for (size_t i = 0; i < gates.size(); ++i) {
        Node& nd = nodes[i];
        nd.g = canonical(gates[i], (int)i);
        canon.push_back(nd.g);
        for (int j = 0; j < nd.g.k; ++j) {
            const int x = nd.g.q[j];
            nd.prev[j] = last[x];
            nd.next[j] = -1;
            if (last[x] >= 0) {
                Node& p = nodes[last[x]];
                p.next[slot_of(p, x)] = (int)i;
            }
            last[x] = (int)i;
        }
    }

    // ---- Algorithm 2 on the per-qubit DAG; with `commute`, diagonal ops are then also
    // merged across the commutation-aware DAG, and the whole fusion is run a second time
    // on that DAG: the plan with fewer passes (then less arithmetic) is kept
    {
        if (o.fuse == 1) run_fusion(nodes, o, pr);
        std::vector<FGate> in;
        for (const int v : topo_order(nodes)) in.push_back(std::move(nodes[v].g));
        if (o.fuse == 1 && o.commute) in = fuse_commuting(std::move(in), n, o, true, pr);
        for (FGate& g : in)
            if (!is_identity(g)) P.fused.push_back(std::move(g));
        if (o.fuse == 1 && o.commute) merge_diagonals(P.fused, o.kmax, pr);
    }
    if (!schedule_passes(n, P.fused, o, P.passes, err)) return false;
    if (o.fuse == 1 && o.commute) {
        std::vector<FGate> alt;
        for (FGate& g : fuse_commuting(std::move(canon), n, o, false, pr))
            if (!is_identity(g)) alt.push_back(std::move(g));
        merge_diagonals(alt, o.kmax, pr);
        std::vector<PassPlan> alt_passes;
        if (!schedule_passes(n, alt, o, alt_passes, err)) return false;
        auto arith = [&](const std::vector<FGate>& f) {
            double a = 0;
            for (const FGate& g : f) a += op_cost(g, o);
            return a;
        };
        // Complex64 with fewer tiles than CUs: a step (an LDS round trip of every tile) takes
        // about half of what a pass adds, and the second fusion buys passes with diagonal
        // steps (8-layer ansatz, by passes alone and so: 15 qubits 77 and 67 us, 16 qubits 84
        // and 71, 18 qubits 100 and 95).  Elsewhere passes alone (20-qubit complex128 mix 562
        // and 588 us, 22-qubit complex64 mix 757 and 776) and served (many states a launch).
        const bool few = o.fp32_mfma && o.pass_floats == 0 && 1ll << std::max(0, n - o.tile_qubits) < kPlanCUs;
        const size_t now = 2 * P.passes.size() + (few ? P.fused.size() : 0);
        const size_t then = 2 * alt_passes.size() + (few ? alt.size() : 0);
        if (then < now || (then == now && arith(alt) < arith(P.fused))) {
            P.fused.swap(alt);
            P.passes.swap(alt_passes);
        }
    }

    build_device_tables(P);
    return true;
}


namespace {

// M <- E(g) M for a d x d matrix M over the fused op's targets: g's local bit j sits at
// M's local bit pos[j].  Each column of M is transformed like a state vector.
void apply_on_rows(std::vector<cd>& M, int d, const InGate& g, const int* pos)
{
    const int dg = 1 << g.k;
    int mask = 0;
    for (int j = 0; j < g.k; ++j) mask |= 1 << pos[j];
    int rows[1 << kMaxK];
    cd in[1 << kMaxK];
    for (int r0 = 0; r0 < d; ++r0) {
        if (r0 & mask) continue;
        for (int a = 0; a < dg; ++a) {
            int r = r0;
            for (int j = 0; j < g.k; ++j)
                if ((a >> j) & 1) r |= 1 << pos[j];
            rows[a] = r;
        }
        for (int c = 0; c < d; ++c) {
            for (int a = 0; a < dg; ++a) in[a] = M[(size_t)rows[a] * d + c];
            for (int a = 0; a < dg; ++a) {
                double re = 0, im = 0;   // plain products: every value here is finite
                for (int b = 0; b < dg; ++b) {
                    const cd u = g.m[(size_t)a * dg + b];
                    re += u.real() * in[b].real() - u.imag() * in[b].imag();
                    im += u.real() * in[b].imag() + u.imag() * in[b].real();
                }
                M[(size_t)rows[a] * d + c] = cd(re, im);
            }
        }
    }
}

}  // namespace

bool same_shape(const HostPlan& P, const std::vector<InGate>& gates)
{
    if (gates.size() != P.gates_in) return false;
    size_t at = 0;
    for (const InGate& g : gates) {
        if (at + 1 + (size_t)g.k > P.shape.size() || P.shape[at] != g.k) return false;
        for (int j = 0; j < g.k; ++j)
            if (P.shape[at + 1 + (size_t)j] != g.t[j]) return false;
        at += 1 + (size_t)g.k;
    }
    return at == P.shape.size();
}

bool refresh_plan(HostPlan& P, const std::vector<InGate>& gates)
{
    if (!same_shape(P, gates)) return false;
    size_t covered = 0;
    for (const FGate& f : P.fused) covered += f.mem.size();
    if (covered != gates.size()) return false;   // a product was dropped as the identity
    std::vector<Matrix> mats(P.fused.size());
    for (size_t fi = 0; fi < P.fused.size(); ++fi) {
        const FGate& f = P.fused[fi];
        const int d = 1 << f.k;
        std::vector<cd> M((size_t)d * d, cd(0, 0));
        for (int r = 0; r < d; ++r) M[(size_t)r * d + r] = cd(1, 0);
        for (const int i : f.mem) {
            if (i < 0 || (size_t)i >= gates.size()) return false;
            const InGate& g = gates[(size_t)i];
            int pos[kMaxK];
            for (int j = 0; j < g.k; ++j) {
                pos[j] = -1;
                for (int t = 0; t < f.k; ++t)
                    if (f.q[t] == g.t[j]) pos[j] = t;
                if (pos[j] < 0) return false;   // not the circuit the plan was made for
            }
            if ((int)g.m.size() != (1 << (2 * g.k))) return false;
            apply_on_rows(M, d, g, pos);
        }
        // the structure the planner used must still hold
        FGate probe;
        probe.k = f.k;
        for (int j = 0; j < f.k; ++j) probe.q[j] = f.q[j];
        probe.m = std::move(M);
        if ((diag_qubit_mask(probe) & f.dq) != f.dq) return false;
        if (f.kind == OP_DIAG || f.kind == OP_PERM) {
            for (int r = 0; r < d; ++r)
                for (int c = 0; c < d; ++c)
                    if (f.m[(size_t)r * d + c] == cd(0, 0) && probe.m[(size_t)r * d + c] != cd(0, 0)) return false;
        }
        mats[fi] = probe.m;
    }
    for (size_t fi = 0; fi < P.fused.size(); ++fi) P.fused[fi].m = std::move(mats[fi]);
    build_device_tables(P);
    return true;
}

}  // namespace qsv
