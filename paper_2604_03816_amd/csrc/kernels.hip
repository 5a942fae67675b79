// kernels.hip -- HIP kernels of libqsv for gfx950 (MI355X, CDNA4, wave64).
//
// State layout: 2^n interleaved complex numbers (float2 for complex64, double2 for
// complex128), qubit t = bit t of the index (Eq. 2 / Eq. 3).
//
// Apply pass (k_pass): each workgroup takes tiles in turn.  A tile is 2^m amplitudes whose
// indices differ only in the pass's m tile qubits: the L lowest qubits (so each tile
// row is a contiguous run of 2^L amplitudes in HBM) plus m - L higher qubits (rows
// strided by 2^q).  The workgroup streams its tile from HBM into LDS, applies every
// op of the pass in order on the LDS copy (dense k-qubit unitaries, diagonal phase
// tables, generalised permutations), and streams it back: one HBM round trip per
// pass however many fused gates it carries.  When the whole state fits in LDS the
// single tile is the state and one launch runs the whole circuit.
//
// Reductions read the state once, accumulate in FP64 per thread (products of FP32
// operands are exact in FP64), reduce each workgroup in a fixed order, and leave
// one partial per workgroup; the host combines partials in a fixed order with
// Neumaier's compensated sum, so results are run-to-run deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <type_traits>

#include "qsv_internal.h"

namespace qsv {

// Address-space-qualified pointers: the state lives in global memory, plan tables are
// read-only (constant address space, so uniform reads become scalar loads).  Pointers
// that a kernel reads from memory (batched launches) carry no address space of their
// own; typing the helpers' parameters keeps every access global or scalar, never flat.
// (The host compilation pass of this file never runs these helpers and sees plain
// pointers.)
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T> using gptr = __attribute__((address_space(1))) T*;
template <typename T> using cptr = const __attribute__((address_space(4))) T*;
#else
template <typename T> using gptr = T*;
template <typename T> using cptr = const T*;
#endif

template <typename R> struct CT;
template <> struct CT<float> { using T = float2; };
template <> struct CT<double> { using T = double2; };

// 16-byte register types for bulk moves (native vectors, so that arrays of them stay
// in registers): two complex64 or one complex128 amplitude.
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));
template <typename C> struct Lane16;
template <> struct Lane16<float2> { using T = floatx4; };
template <> struct Lane16<double2> { using T = doublex2; };

template <typename C>
__device__ __forceinline__ C cmul(C a, C b)
{
    C r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}

template <typename C>
__device__ __forceinline__ void cmac(C& acc, C a, C b)
{
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(-a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(a.y, b.x, acc.y);
}

// PassArgs' arrays are indexed with compile-time indices only (fully unrolled loops
// with a uniform guard): a runtime index into a kernel argument becomes a vector load
// plus a wait on every outstanding memory operation, stores and prefetches included.
__device__ __forceinline__ long long tile_base(const PassArgs& a, long long t)
{
    long long base = 0;
#pragma unroll
    for (int i = 0; i < kMaxRuns; ++i) {
        if (i < a.nruns) {
            base |= (t & ((1ll << a.run_len[i]) - 1)) << a.run_pos[i];
            t >>= a.run_len[i];
        }
    }
    return base;
}

// Offset (relative to the tile base) of the local bits [lo, hi) of local index e.
__device__ __forceinline__ long long local_off_bits(const PassArgs& a, int e, int lo, int hi)
{
    long long o = 0;
#pragma unroll
    for (int i = 0; i < kMaxTileQubits; ++i) {
        if (i >= lo && i < hi && ((e >> i) & 1)) o += 1ll << a.phys[i];
    }
    return o;
}

// LDS position of tile element e.  The tile is stored XOR-swizzled so that the lanes of an
// access spread over all banks whichever tile bits they run over: a bank's five (complex64,
// 8-byte elements) or four (complex128) address bits are the XOR of element bits five or
// four apart, so any run of consecutive bits, one per bank bit, is free of conflicts.  The
// map is a bijection on every range [0, 2^m) and linear over XOR: for disjoint bit sets
// a | b = a ^ b, so swz(a | b) = swz(a) ^ swz(b), which lets a uniform (scalar) part and a
// per-lane part be swizzled separately and combined with one XOR.  (planner.cpp's
// tile_slot is the same map.)
template <typename C>
__device__ __forceinline__ int swz(int e)
{
    if constexpr (sizeof(C) == 8) return e ^ ((e >> 5) & 31) ^ (e >> 10);
    else return e ^ ((e >> 4) & 15) ^ ((e >> 8) & 15);
}

// Move a tile between HBM and LDS.  Every lane moves 16 bytes at a time: W = 1
// complex128 or W = 2 adjacent complex64 amplitudes (local bit 0 is qubit 0, so such a
// pair is contiguous in HBM).  Local index e = W (256 * slice + tid) + w: the bits from
// the thread id give an offset computed once per thread, the bits above from the slice
// number; with the slice count NS a compile-time constant every slice's offset is a sum
// of uniform strides (scalar ALU) and all NS accesses of a thread are issued back to
// back before the first is consumed.
__device__ __forceinline__ long long local_stride(const PassArgs& a, int i)
{
    return 1ll << a.phys[i];   // i is a compile-time constant at every call site
}

template <typename C, bool LOAD, int NS, int W>
__device__ __forceinline__ void move_tile_n(gptr<C> __restrict__ st, C* __restrict__ lds, const PassArgs& a,
                                            long long toff)
{
    static_assert(W == 1 || (W == 2 && sizeof(C) == 8), "16-byte lanes");
    using V = typename std::conditional<W == 2, floatx4, C>::type;
    // the state streams through once per pass: nontemporal loads and stores (measured
    // 2 % faster passes than plain ones); the builtins want native vector types
    using NV = typename std::conditional<sizeof(V) == 16, floatx4, float __attribute__((ext_vector_type(2)))>::type;
    constexpr int LW = W == 2 ? 1 : 0;
    constexpr int LB = NS >= 32 ? 5 : NS >= 16 ? 4 : NS >= 8 ? 3 : NS >= 4 ? 2 : NS >= 2 ? 1 : 0;
    long long hs[LB > 0 ? LB : 1];
#pragma unroll
    for (int b = 0; b < LB; ++b) hs[b] = local_stride(a, kLogThreads + LW + b);
    const int tid = threadIdx.x;
    // at most CH 16-byte units in registers at a time: wider tiles move in several
    // batches, so the largest tile does not set the kernel's register count
    constexpr int CH = NS < 8 ? NS : 8;
    V v[CH];
    // 16-byte unit u = 256 j + tid holds tile elements W u .. W u + W - 1; the positions of
    // its elements are those of element W tid (+ 1) XOR the compile-time part of j
    int ut = swz<C>(W * tid);
    asm volatile("" : "+v"(ut));   // keeps the positions of all j from being held across the tile loop
    auto put = [&](int j, const V& x) {
        const int at = ut ^ swz<C>(W * (j << kLogThreads));
        if constexpr (W == 2) {
            lds[at] = C{x.x, x.y};
            lds[at ^ 1] = C{x.z, x.w};
        } else {
            lds[at] = x;
        }
    };
    auto get = [&](int j) {
        const int at = ut ^ swz<C>(W * (j << kLogThreads));
        if constexpr (W == 2) {
            const C p = lds[at], r = lds[at ^ 1];
            return V{p.x, p.y, r.x, r.y};
        } else {
            return lds[at];
        }
    };
    auto off = [&](int j) {
        long long so = 0;
#pragma unroll
        for (int b = 0; b < LB; ++b)
            if ((j >> b) & 1) so += hs[b];
        return so;
    };
#pragma unroll
    for (int j0 = 0; j0 < NS; j0 += CH) {
        if (LOAD) {
#pragma unroll
            for (int j = 0; j < CH; ++j)
                v[j] = __builtin_bit_cast(V, __builtin_nontemporal_load((const NV*)(st + toff + off(j0 + j))));
#pragma unroll
            for (int j = 0; j < CH; ++j) put(j0 + j, v[j]);
        } else {
#pragma unroll
            for (int j = 0; j < CH; ++j) v[j] = get(j0 + j);
#pragma unroll
            for (int j = 0; j < CH; ++j)
                __builtin_nontemporal_store(__builtin_bit_cast(NV, v[j]), (NV*)(st + toff + off(j0 + j)));
        }
    }
}

// The two halves of a tile load for a kernel that has other work in between: NS 16-byte
// units per thread from p (the tile's base plus the thread's offset) into registers, and
// from there to their places in LDS.
template <typename C, int NS, int W>
__device__ __forceinline__ void load_tile(gptr<C> p, const PassArgs& a, floatx4 (&v)[NS])
{
    constexpr int LW = W == 2 ? 1 : 0;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        long long o = 0;
#pragma unroll
        for (int b = 0; (1 << b) < NS; ++b)
            if ((j >> b) & 1) o += local_stride(a, kLogThreads + LW + b);
        v[j] = __builtin_nontemporal_load((const floatx4*)(p + o));
    }
}

template <typename C, int NS, int W>
__device__ __forceinline__ void put_tile(C* __restrict__ lds, const floatx4 (&v)[NS])
{
    int ut = swz<C>(W * (int)threadIdx.x);
    asm volatile("" : "+v"(ut));
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int at = ut ^ swz<C>(W * (j << kLogThreads));
        if constexpr (W == 2) {
            lds[at] = C{v[j].x, v[j].y};
            lds[at ^ 1] = C{v[j].z, v[j].w};
        } else {
            lds[at] = __builtin_bit_cast(C, v[j]);
        }
    }
}

template <typename C, int NS, int W>
__device__ __forceinline__ void get_tile(const C* __restrict__ lds, floatx4 (&v)[NS])
{
    int ut = swz<C>(W * (int)threadIdx.x);
    asm volatile("" : "+v"(ut));
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int at = ut ^ swz<C>(W * (j << kLogThreads));
        if constexpr (W == 2) {
            const C p = lds[at], q = lds[at ^ 1];
            v[j] = floatx4{p.x, p.y, q.x, q.y};
        } else {
            v[j] = __builtin_bit_cast(floatx4, lds[at]);
        }
    }
}

template <typename C, int NS, int W>
__device__ __forceinline__ void store_tile(gptr<C> p, const PassArgs& a, const floatx4 (&v)[NS])
{
    constexpr int LW = W == 2 ? 1 : 0;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        long long o = 0;
#pragma unroll
        for (int b = 0; (1 << b) < NS; ++b)
            if ((j >> b) & 1) o += local_stride(a, kLogThreads + LW + b);
        __builtin_nontemporal_store(v[j], (floatx4*)(p + o));
    }
}

template <typename C, bool LOAD>
__device__ __forceinline__ void move_tile(gptr<C> __restrict__ st, C* __restrict__ lds, const PassArgs& a,
                                          long long base)
{
    const int tid = threadIdx.x;
    if constexpr (sizeof(C) == 8) {
        // complex64 pairs whenever qubit 0 is a tile qubit and a slice is full
        if (a.L >= 1 && a.m > kLogThreads) {
            const long long toff = base + local_off_bits(a, tid << 1, 1, kLogThreads + 1);
            switch (a.m - kLogThreads - 1) {
            case 0: move_tile_n<C, LOAD, 1, 2>(st, lds, a, toff); break;
            case 1: move_tile_n<C, LOAD, 2, 2>(st, lds, a, toff); break;
            case 2: move_tile_n<C, LOAD, 4, 2>(st, lds, a, toff); break;
            case 3: move_tile_n<C, LOAD, 8, 2>(st, lds, a, toff); break;
            default: move_tile_n<C, LOAD, 16, 2>(st, lds, a, toff); break;
            }
            return;
        }
    }
    const int lowb = a.m < kLogThreads ? a.m : kLogThreads;
    const long long toff = base + local_off_bits(a, tid, 0, lowb);
    switch (a.m - kLogThreads) {
    case 0: move_tile_n<C, LOAD, 1, 1>(st, lds, a, toff); break;
    case 1: move_tile_n<C, LOAD, 2, 1>(st, lds, a, toff); break;
    case 2: move_tile_n<C, LOAD, 4, 1>(st, lds, a, toff); break;
    case 3: move_tile_n<C, LOAD, 8, 1>(st, lds, a, toff); break;
    case 4: move_tile_n<C, LOAD, 16, 1>(st, lds, a, toff); break;
    case 5: move_tile_n<C, LOAD, 32, 1>(st, lds, a, toff); break;
    default:   // tiles smaller than one slice (whole states below 256 amplitudes)
        if (tid < (1 << a.m)) {
            if (LOAD) lds[swz<C>(tid)] = st[toff];
            else st[toff] = lds[swz<C>(tid)];
        }
        break;
    }
}

// Offset of local basis row r of an op inside the tile: bit j of r sits at lpos[j].
template <int K>
__device__ __forceinline__ int row_off(int r, const DevOp& op)
{
    int o = 0;
#pragma unroll
    for (int j = 0; j < K; ++j)
        if ((r >> j) & 1) o += 1 << op.lpos[j];
    return o;
}

// Group g of an op: insert a zero bit at each target position (ascending).  The map is
// linear over XOR, so group_base(g0 + tid) = group_base(g0) ^ group_base(tid) when g0 is
// a multiple of the workgroup size: a per-thread part computed once per op and a
// uniform part per iteration.
template <int K>
__device__ __forceinline__ int group_base(int g, const DevOp& op)
{
    int b = g;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int p = op.lpos[j];
        b = ((b >> p) << (p + 1)) | (b & ((1 << p) - 1));
    }
    return b;
}

template <typename C, int K>
__device__ void op_dense(C* __restrict__ lds, int T, const DevOp& op, cptr<C> __restrict__ M)
{
    constexpr int D = 1 << K;
    const int G = T >> K;
    // LDS position of row r of group g0 + tid: swz(group_base(g0)) (uniform, scalar work)
    // ^ swz(group_base(tid)) ^ swz(row_off(r)) (per lane and per op)
    const int bt = swz<C>(group_base<K>(threadIdx.x, op));
    for (int g0 = 0; g0 < G; g0 += kThreads) {
        if (g0 + (int)threadIdx.x >= G) break;
        const int b = __builtin_amdgcn_readfirstlane(swz<C>(group_base<K>(g0, op))) ^ bt;
        C v[D];
#pragma unroll
        for (int r = 0; r < D; ++r) v[r] = lds[b ^ swz<C>(row_off<K>(r, op))];
        // rows are not unrolled for wide gates: the row's matrix entries are uniform
        // (scalar) loads, the inputs stay in registers; two at a time for a complex128
        // 5-qubit gate, whose one wave per SIMD waits on them (29 qubits: 5.85 -> 5.54 ms)
        constexpr int RU = K <= 2 ? D : K == 5 && sizeof(C) == 16 ? 2 : 1;
#pragma unroll RU
        for (int r = 0; r < D; ++r) {
            C acc;
            acc.x = acc.y = 0;
#pragma unroll
            for (int c = 0; c < D; ++c) cmac(acc, M[r * D + c], v[c]);
            lds[b ^ swz<C>(row_off<K>(r, op))] = acc;
        }
    }
}

// ---- dense ops on matrix cores
//
// A 4-qubit op multiplies a 16 x 16 complex matrix M into the tile viewed as 16 rows (the
// op's basis states) by columns (the groups).  A wave takes 16 columns at a time, one block
// of 256 amplitudes: lane (q, c) = (lane / 16, lane % 16) holds four amplitudes of column
// c, of the rows the planner gave to (q, j), j < 4, and gets back the same four rows'
// results.  The planner fixes which tile bits the lane, j and the block number run over
// (planner.cpp, mfma_tables) and stores, per op, the LDS byte offset of each of those bits;
// the address of an access is one XOR of a lane's and a block's part.  It also stores the
// matrix in the order the lanes feed it, so an op's set-up is two or four 16-byte loads.
//
// Pairs.  Two ops on disjoint targets, one after the other, take one LDS round trip: the
// matrix instruction contracts the index that lies on (lane / 16, j) and leaves the other
// on lane % 16, and with the amplitudes as its first operand instead of its second the
// result comes out transposed: the first op's rows on lane % 16, and the columns, which
// are the second op's 16 states, on (lane / 16, j), where the second op needs them.

// complex64: the product in bfloat16 matrix instructions (16 x 16 x 32), each FP32 number
// carried as the sum of three bfloat16 numbers (8 + 8 + 8 significant bits).  Of the nine
// products of parts the six of relative size 2^-18 and more are summed, in FP32, smallest
// first; the three left out are each below 2^-25 of the term, at most 2^-24 together.  The
// sum is exact from 2^-110 (below, the third part is under bfloat16's smallest) to 2^128 -
// 2^119 (from there on the first part is infinite); plans with matrix_cores = -1 take such
// values.  A block takes 192 matrix-core clocks (FP32 matrix instructions in the
// three-product form below take 384) and about as many of the VALU for the splits.
// 30-qubit depth-20 brickwork, per pass: FP32 instructions 4.19 ms, this 4.00 ms, at which the
// chip is at its power limit (2.0 GHz against 2.4); error of a 22-qubit brickwork state
// against 64 bits 9.1e-7 and 3.4e-7.  Tiles scaled into the range and done again in FP32
// where a result is NaN cost 0.4 % there and 4 % where diagonal ops and permutations prevail.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

struct Split8 {
    bf16x8 h, m, l;
};

// Two FP32 numbers to bfloat16 (one instruction) and what that leaves of them: one dot
// product with (-1, 0) or (0, -1) per number subtracts the rounded part, exactly.
__device__ __forceinline__ bf16x2 split_step(float& a, float& b)
{
    const bf16x2 h = __builtin_convertvector((floatx2{a, b}), bf16x2);
    // (-1, 0) and (0, -1) in registers: as an inline constant the instruction reads -1.0 as
    // the other pair
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    asm("" : "+s"(lo), "+s"(hi));
    a = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, lo), a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, hi), b, false);
    return h;
}

__device__ __forceinline__ Split8 split8(const float (&x)[8])
{
    Split8 s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
        const bf16x2 h = split_step(a, b), m = split_step(a, b);
        const bf16x2 l = __builtin_convertvector((floatx2{a, b}), bf16x2);
        s.h[2 * i] = h[0]; s.h[2 * i + 1] = h[1];
        s.m[2 * i] = m[0]; s.m[2 * i + 1] = m[1];
        s.l[2 * i] = l[0]; s.l[2 * i + 1] = l[1];
    }
    return s;
}

// The (Re, -Im) operand of an output's real part, turned into (Im, Re) for its
// imaginary part: halves swapped, the new low half's sign flipped.
__device__ __forceinline__ bf16x8 imag_operand(bf16x8 v)
{
    uintx4 u = __builtin_bit_cast(uintx4, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = __builtin_amdgcn_alignbit(u[i], u[i], 16) ^ 0x8000u;
    return __builtin_bit_cast(bf16x8, u);
}

struct Mat64 {
    Split8 re, im;
};

// A lane's four complex entries (32 bytes, two 16-byte loads), from LDS or global memory.
template <typename P>
__device__ __forceinline__ Mat64 load_mat64(P A, int lane)
{
    const floatx4 u = A[lane], v = A[64 + lane];
    const float x[8] = {u.x, -u.y, u.z, -u.w, v.x, -v.y, v.z, -v.w};
    Mat64 r;
    r.re = split8(x);
    r.im.h = imag_operand(r.re.h);
    r.im.m = imag_operand(r.re.m);
    r.im.l = imag_operand(r.re.l);
    return r;
}

// SWAP: the amplitudes as the first operand (the transposed result).
template <bool SWAP>
__device__ __forceinline__ floatx4 product64(const Split8& a, const Split8& x)
{
    auto mm = [](bf16x8 p, bf16x8 v, floatx4 c) {
        return SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, p, c, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_16x16x32_bf16(p, v, c, 0, 0, 0);
    };
    floatx4 c = {0, 0, 0, 0};
    c = mm(a.l, x.h, c);
    c = mm(a.m, x.m, c);
    c = mm(a.h, x.l, c);
    c = mm(a.m, x.h, c);
    c = mm(a.h, x.m, c);
    c = mm(a.h, x.h, c);
    return c;
}

// complex128: FP64 matrix instructions with three real products instead of four (Gauss's
// form of a complex product): with M = Ar + i Ai, x = xr + i xi and t = Ar (xr + xi),
// Re(M x) = t - (Ar + Ai) xi and Im(M x) = t + (Ai - Ar) xr.
struct Mat128 {
    double r[4], n[4], s[4];
};

template <typename P>
__device__ __forceinline__ Mat128 load_mat128(P A, int lane)
{
    Mat128 m;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const doublex2 u = A[64 * j + lane];
        m.r[j] = u.x;
        m.n[j] = -(u.x + u.y);
        m.s[j] = u.y - u.x;
    }
    return m;
}

template <bool SWAP>
__device__ __forceinline__ void product128(const Mat128& a, const double (&xr)[4], const double (&xi)[4],
                                           doublex4& yr, doublex4& yi)
{
    auto mm = [](double p, double v, doublex4 c) {
        return SWAP ? __builtin_amdgcn_mfma_f64_16x16x4f64(v, p, c, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f64_16x16x4f64(p, v, c, 0, 0, 0);
    };
    doublex4 t = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) t = mm(a.r[j], xr[j] + xi[j], t);
    yr = yi = t;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        yr = mm(a.n[j], xi[j], yr);
        yi = mm(a.s[j], xr[j], yi);
    }
}

// XOR of the offsets of a number's bits: a block's (uniform, scalar unit) or a lane's.
__device__ __forceinline__ int packed16(const unsigned* w, int i)
{
    return (w[i >> 1] >> (16 * (i & 1))) & 0xffff;
}

__device__ __forceinline__ int block_off(int blk, const DevOp& op)
{
    int o = 0;
#pragma unroll
    for (int i = 0; i < kMaxBlockBits; ++i)
        if ((blk >> i) & 1) o ^= packed16(op.bbit, i);
    return __builtin_amdgcn_readfirstlane(o);
}

__device__ __forceinline__ int lane_off(int lane, const unsigned (&bit)[3])
{
    int o = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) o ^= __builtin_amdgcn_sbfe(lane, i, 1) & packed16(bit, i);
    return o;
}

// The operand of an op: from the pass's LDS block (LDSOP: launches whose operands are all
// staged), else from the plan's operand array.
template <typename C, bool LDSOP>
__device__ __forceinline__ auto load_mat(const DevOp& op, cptr<float> __restrict__ apool, const float* __restrict__ alds,
                                         int lane)
{
    if constexpr (sizeof(C) == 8) {
        if constexpr (LDSOP) return load_mat64(reinterpret_cast<const floatx4*>(alds + op.aoff), lane);
        else return load_mat64((cptr<floatx4>)(apool + op.goff), lane);
    } else {
        if constexpr (LDSOP) return load_mat128(reinterpret_cast<const doublex2*>(alds + op.aoff), lane);
        else return load_mat128((cptr<doublex2>)(apool + op.goff), lane);
    }
}

// One 4-qubit op, or a pair of them on disjoint targets (op2: the second).
template <typename C, bool PAIR, bool LDSOP>
__device__ __forceinline__ void op_mfma4(C* __restrict__ lds, int T, const DevOp& op, const DevOp& op2,
                                         cptr<float> __restrict__ apool, const float* __restrict__ alds)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    char* __restrict__ base = reinterpret_cast<char*>(lds);
    const int lin = lane_off(lane, op.lin), lout = PAIR ? lane_off(lane, op2.lin) : lin;
    auto joff = [](int j, const DevOp& o) {
        return ((j & 1) ? packed16(&o.jbit, 0) : 0) ^ ((j & 2) ? packed16(&o.jbit, 1) : 0);
    };
    const int nblk = T >> 8;
    constexpr int NW = kThreads / 64;
    const auto m1 = load_mat<C, LDSOP>(op, apool, alds, lane);
    decltype(load_mat<C, LDSOP>(op, apool, alds, lane)) m2;
    if (PAIR) m2 = load_mat<C, LDSOP>(op2, apool, alds, lane);
    for (int blk = wave; blk < nblk; blk += NW) {
        const int sb = block_off(blk, op);
        C v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const C*>(base + ((sb ^ joff(j, op)) ^ lin));
        if constexpr (sizeof(C) == 8) {
            float x[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                x[2 * j] = v[j].x;
                x[2 * j + 1] = v[j].y;
            }
            Split8 s = split8(x);
            floatx4 yr = product64<PAIR>(m1.re, s), yi = product64<PAIR>(m1.im, s);
            if (PAIR) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[2 * j] = yr[j];
                    x[2 * j + 1] = yi[j];
                }
                s = split8(x);
                yr = product64<false>(m2.re, s);
                yi = product64<false>(m2.im, s);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j].x = yr[j];
                v[j].y = yi[j];
            }
        } else {
            double xr[4], xi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                xr[j] = v[j].x;
                xi[j] = v[j].y;
            }
            doublex4 yr, yi;
            product128<PAIR>(m1, xr, xi, yr, yi);
            if (PAIR) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xr[j] = yr[j];
                    xi[j] = yi[j];
                }
                product128<false>(m2, xr, xi, yr, yi);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j].x = yr[j];
                v[j].y = yi[j];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<C*>(base + ((sb ^ joff(j, PAIR ? op2 : op)) ^ lout)) = v[j];
    }
}

// complex128 3-qubit op: its real embedding [[Re, -Im], [Im, Re]], 16 x 16, fills the
// matrix instruction (three 8 x 8 products would not): lane (q, c) feeds two complex rows
// of column c, 4 j + q, as four real steps and gets rows 2 q and 2 q + 1 back.
template <bool LDSOP>
__device__ __forceinline__ void op_mfma3(double2* __restrict__ lds, int T, const DevOp& op,
                                         cptr<float> __restrict__ apool, const float* __restrict__ alds)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    char* __restrict__ base = reinterpret_cast<char*>(lds);
    doublex2 a0, a1;
    if constexpr (LDSOP) {
        const doublex2* A = reinterpret_cast<const doublex2*>(alds + op.aoff);
        a0 = A[lane];
        a1 = A[64 + lane];
    } else {
        cptr<doublex2> A = (cptr<doublex2>)(apool + op.goff);
        a0 = A[lane];
        a1 = A[64 + lane];
    }
    // target bits: jbit holds bit 2's offset (rows 4 j + q) and bit 0's (rows 2 q + j)
    const int r0 = lane_off(lane, op.lin), r1 = r0 ^ packed16(&op.jbit, 0);
    const int w0 = lane_off(lane, op.lout), w1 = w0 ^ packed16(&op.jbit, 1);
    const int nblk = T >> 7;
    constexpr int NW = kThreads / 64;
    for (int blk = wave; blk < nblk; blk += NW) {
        const int sb = block_off(blk, op);
        const double2 v0 = *reinterpret_cast<const double2*>(base + (sb ^ r0));
        const double2 v1 = *reinterpret_cast<const double2*>(base + (sb ^ r1));
        doublex4 y = {0, 0, 0, 0};
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(a0.x, v0.x, y, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(a0.y, v0.y, y, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(a1.x, v1.x, y, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(a1.y, v1.y, y, 0, 0, 0);
        *reinterpret_cast<double2*>(base + (sb ^ w0)) = double2{y[0], y[1]};
        *reinterpret_cast<double2*>(base + (sb ^ w1)) = double2{y[2], y[3]};
    }
}

template <typename C, int K>
__device__ void op_perm(C* __restrict__ lds, int T, const DevOp& op, cptr<C> __restrict__ ph,
                        cptr<int> __restrict__ src)
{
    constexpr int D = 1 << K;
    const int G = T >> K;
    const bool phased = op.flags != 0;
    const int bt = swz<C>(group_base<K>(threadIdx.x, op));
    for (int g0 = 0; g0 < G; g0 += kThreads) {
        if (g0 + (int)threadIdx.x >= G) break;
        const int b = __builtin_amdgcn_readfirstlane(swz<C>(group_base<K>(g0, op))) ^ bt;
        C v[D];
#pragma unroll
        for (int r = 0; r < D; ++r) v[r] = lds[b ^ swz<C>(row_off<K>(src[r], op))];
#pragma unroll
        for (int r = 0; r < D; ++r) lds[b ^ swz<C>(row_off<K>(r, op))] = phased ? cmul(ph[r], v[r]) : v[r];
    }
}

// Diagonal op: the table (2^k phases) is read from LDS when the planner staged it there
// (per-lane indices; a global read here would also wait on every outstanding memory
// operation of the pass), else from the plan pool.
template <typename C, typename P>
__device__ __forceinline__ void op_diag(C* __restrict__ lds, int T, const DevOp& op, P Dg, long long base)
{
    // targets outside the tile contribute a per-tile constant part of the table index
    int gfix = 0, lp[kMaxDiagK];
#pragma unroll
    for (int j = 0; j < kMaxDiagK; ++j) {
        lp[j] = (j < op.k) ? op.lpos[j] : -1;
        if (j < op.k && lp[j] < 0) gfix |= (int)((base >> op.gbit[j]) & 1) << j;
    }
    const int st = swz<C>(threadIdx.x);
    for (int e = threadIdx.x; e < T; e += kThreads) {
        int idx = gfix;
#pragma unroll
        for (int j = 0; j < kMaxDiagK; ++j)
            if (lp[j] >= 0) idx |= ((e >> lp[j]) & 1) << j;
        const int pe = swz<C>(e - (int)threadIdx.x) ^ st;   // e - tid: a multiple of 256
        lds[pe] = cmul(lds[pe], Dg[idx]);
    }
}

// Workgroup barrier for LDS data only: waits for this wave's LDS operations, then for
// every wave of the workgroup.  Unlike __syncthreads it does not wait for outstanding
// global memory operations (between two ops of a pass only LDS data changes hands).
// The memory clobber keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// WIDE = false leaves out the register-heavy paths (VALU dense ops on 4 or 5 targets,
// permutations on 3 or more): the caller launches that variant only for passes without
// such ops, and its lower register count allows more resident workgroups.  Ends with an LDS
// barrier after the last op.
template <typename C, bool WIDE, bool LDSOP>
__device__ __forceinline__ void apply_ops(C* __restrict__ lds, int T, cptr<DevOp> __restrict__ ops, int op_begin,
                          int op_count, cptr<C> __restrict__ pool, cptr<int> __restrict__ ipool,
                          cptr<float> __restrict__ apool, const float* __restrict__ alds, long long base)
{
    for (int oi = 0; oi < op_count; ++oi) {
        const DevOp op = ops[op_begin + oi];
        cptr<C> M = pool + op.off;
        if (op.kind == OP_DENSE && op.goff >= 0) {
            // matrix cores: a pair, one 4-qubit op, or (complex128 only) a 3-qubit op
            if (op.flags) {
                ++oi;
                op_mfma4<C, true, LDSOP>(lds, T, op, ops[op_begin + oi], apool, alds);
            } else if (sizeof(C) == 8 || op.k == 4) {   // (complex64 3-qubit ops: widened operands)
                op_mfma4<C, false, LDSOP>(lds, T, op, op, apool, alds);
            } else {
                if constexpr (sizeof(C) == 16) op_mfma3<LDSOP>(lds, T, op, apool, alds);
            }
            // the next op's waves read only what the same waves wrote: LDS keeps a wave's order
            if (op.nosync) asm volatile("" ::: "memory");
            else lds_sync();
            continue;
        }
        if (op.kind == OP_DENSE) {
            switch (op.k) {
            case 1: op_dense<C, 1>(lds, T, op, M); break;
            case 2: op_dense<C, 2>(lds, T, op, M); break;
            case 3: op_dense<C, 3>(lds, T, op, M); break;
            case 4: if constexpr (WIDE) op_dense<C, 4>(lds, T, op, M); break;
            default: if constexpr (WIDE) op_dense<C, 5>(lds, T, op, M); break;
            }
        } else if (op.kind == OP_PERM) {
            cptr<int> S = ipool + op.ioff;
            switch (op.k) {
            case 1: op_perm<C, 1>(lds, T, op, M, S); break;
            case 2: op_perm<C, 2>(lds, T, op, M, S); break;
            case 3: if constexpr (WIDE) op_perm<C, 3>(lds, T, op, M, S); break;
            case 4: if constexpr (WIDE) op_perm<C, 4>(lds, T, op, M, S); break;
            default: if constexpr (WIDE) op_perm<C, 5>(lds, T, op, M, S); break;
            }
        } else if (op.aoff >= 0) {
            op_diag<C, const C*>(lds, T, op, reinterpret_cast<const C*>(alds + op.aoff), base);
        } else {
            op_diag<C, cptr<C>>(lds, T, op, M, base);
        }
        lds_sync();
    }
}

// The pass's staged block (diagonal tables, then matrix operands), global -> LDS: 16 bytes
// per thread and step; blocks are multiples of 16 bytes.
__device__ __forceinline__ void stage_operands(float* __restrict__ alds, cptr<float> __restrict__ apool, int off, int len)
{
    cptr<floatx4> src = (cptr<floatx4>)(apool + off);
    floatx4* dst = reinterpret_cast<floatx4*>(alds);
    for (int i = threadIdx.x; i < (len >> 2); i += kThreads) dst[i] = src[i];
}

// One tile of one pass: HBM -> LDS, every op of the pass, LDS -> HBM.
template <typename C, bool WIDE, bool LDSOP>
__device__ __forceinline__ void run_tile(gptr<C> __restrict__ st, C* __restrict__ lds, const PassArgs& a,
                                         long long tile, cptr<DevOp> __restrict__ ops, cptr<C> __restrict__ pool,
                                         cptr<int> __restrict__ ipool, cptr<float> __restrict__ apool,
                                         const float* __restrict__ alds, bool from_zero = false)
{
    const long long base = tile_base(a, tile);
    if (from_zero) {
        // the tile of |0...0> (Eq. 1): built on chip instead of read from HBM (element 0
        // keeps position 0 under the swizzle and every other element is zero)
        for (int e = threadIdx.x; e < (1 << a.m); e += kThreads) {
            C z;
            z.x = (base == 0 && e == 0) ? 1 : 0;
            z.y = 0;
            lds[e] = z;
        }
    } else {
        move_tile<C, true>(st, lds, a, base);
    }
    __syncthreads();
    apply_ops<C, WIDE, LDSOP>(lds, 1 << a.m, ops, a.op_begin, a.op_count, pool, ipool, apool, alds, base);
    move_tile<C, false>(st, lds, a, base);
}

// One work-list entry of a pass launch: the state it belongs to and its tile.  Consecutive
// workgroups run on different XCDs; the map gives each XCD runs of neighbouring tiles, whose
// 128-byte rows are neighbours in memory (30-qubit passes without ops 3.48 -> 3.42 ms
// complex64, 28-qubit complex128 1.72 -> 1.65 ms; with ops 25-qubit complex64 0.131 -> 0.127
// ms for runs of 16 against one run per XCD).  It permutes each full stride of the grid
// (a power of two) and leaves other grids alone.
__device__ __forceinline__ long long xcd_tile(long long t, unsigned grid, long long ntiles)
{
    if ((grid & (grid - 1)) || grid < 128 || ntiles < grid) return t;
    const unsigned w = (unsigned)t & (grid - 1);
    const unsigned k = w >> 3;
    return (t - w) + (k & ~15u) * 8 + (w & 7) * 16 + (k & 15);
}

// WIDE = false: the variant without the register-heavy op paths, for passes free of
// them (fewer registers, so more resident workgroups when LDS allows).  PF: tiles of 2^12
// amplitudes, the next one loaded into registers while the ops run on this one (then no op
// may wait for a global load of its own, which would wait for the tile's too: operands come
// from LDS).  Both the moves and the ops of a pass take most of its time alone, and the few
// workgroups a CU holds (four complex64, two complex128) overlap them only in part; with the
// loads ahead each counts twice: 30-qubit complex64 passes 4.28 -> 4.00 ms (moves alone
// 3.46), 28-qubit complex128 2.71 -> 2.43 ms (moves alone 1.72, ops alone 2.03).
template <typename C, bool WIDE, bool PF>
__global__ __launch_bounds__(kThreads, sizeof(C) == 8 ? 4 : 2) void k_pass(C* __restrict__ st, C* __restrict__ st2,
                                                                     const PassArgs a, long long ntiles,
                                                                     int from_zero, const DevOp* __restrict__ ops,
                                                                     const C* __restrict__ pool,
                                                                     const int* __restrict__ ipool,
                                                                     const float* __restrict__ apool)
{
    // st2 != nullptr: the same pass on a second state of the same shape (tiles ntiles ..
    // 2 ntiles - 1 of the work list), e.g. the adjoint's two vectors.  from_zero: the
    // input is |0...0>, whatever the state buffers hold (a circuit's first pass, with the
    // initialisation folded in)
    extern __shared__ __align__(16) unsigned char smem[];
    C* lds = reinterpret_cast<C*>(smem);
    float* alds = reinterpret_cast<float*>(smem + (sizeof(C) << a.m));
    stage_operands(alds, (cptr<float>)apool, a.a_off, PF ? a.a_len : a.d_len);
    __syncthreads();
    const long long total = st2 ? 2 * ntiles : ntiles;
    if constexpr (PF) {
        constexpr int W = sizeof(C) == 8 ? 2 : 1, NS = 4096 / (kThreads * W);
        constexpr int LW = W == 2 ? 1 : 0;
        const long long tl = local_off_bits(a, (int)threadIdx.x << LW, LW, kLogThreads + LW);
        auto at = [&](long long t, gptr<C>& s) {   // the state of entry t and its tile's base
            const bool second = t >= ntiles;
            s = (gptr<C>)(second ? st2 : st);
            return tile_base(a, xcd_tile(second ? t - ntiles : t, gridDim.x, ntiles));
        };
        floatx4 v[NS];
        long long t = blockIdx.x;
        gptr<C> s;
        long long base = at(t, s);
        load_tile<C, NS, W>(s + base + tl, a, v);
        put_tile<C, NS, W>(lds, v);
        lds_sync();
        for (;;) {
            const long long tn = t + gridDim.x;
            gptr<C> sn = s;
            long long bn = 0;
            if (tn < total) {
                bn = at(tn, sn);
                load_tile<C, NS, W>(sn + bn + tl, a, v);
            }
            apply_ops<C, WIDE, true>(lds, 4096, (cptr<DevOp>)ops, a.op_begin, a.op_count, (cptr<C>)pool,
                                         (cptr<int>)ipool, (cptr<float>)apool, alds, base);
            if (tn >= total) {
                move_tile_n<C, false, NS, W>(s, lds, a, base + tl);
                break;
            }
            // the tile to registers, the next one into its place, then the stores: the wait
            // for the next tile's loads then has no stores behind it to wait for
            floatx4 r[NS];
            get_tile<C, NS, W>(lds, r);
            lds_sync();
            put_tile<C, NS, W>(lds, v);
            store_tile<C, NS, W>(s + base + tl, a, r);
            lds_sync();
            t = tn;
            s = sn;
            base = bn;
        }
    } else {
        for (long long t = blockIdx.x; t < total; t += gridDim.x) {
            const bool second = t >= ntiles;
            run_tile<C, WIDE, false>((gptr<C>)(second ? st2 : st), lds, a,
                                        xcd_tile(second ? t - ntiles : t, gridDim.x, ntiles), (cptr<DevOp>)ops,
                                        (cptr<C>)pool, (cptr<int>)ipool, (cptr<float>)apool, alds, from_zero != 0);
            __syncthreads();
        }
    }
}

// Batched pass for continuous batching: one launch advances many independent states,
// each by its own current pass.  Work item w (a tile of one item's pass) is found by
// binary search over the items' tile prefix sums; the grid is persistent (fixed size,
// strided over the work list) so the launch can be captured once and replayed.
template <typename C, bool WIDE>
__global__ __launch_bounds__(kThreads, sizeof(C) == 8 ? 4 : 2) void k_batch_pass(const BatchItem* __restrict__ table,
                                                                                 const BatchList* __restrict__ list)
{
    extern __shared__ __align__(16) unsigned char smem[];
    C* lds = reinterpret_cast<C*>(smem);
    __shared__ long long ends[kMaxBatchItems];
    const int nitems = min(list->count, kMaxBatchItems);
    if (nitems <= 0) return;
    const BatchItem* __restrict__ items = table + list->first;
    for (int i = threadIdx.x; i < nitems; i += kThreads) ends[i] = items[i].tile_end;
    __syncthreads();
    const long long total = ends[nitems - 1];
    int staged = -1;   // item whose operand block LDS holds (consecutive tiles often share one)
    for (long long w = blockIdx.x; w < total; w += gridDim.x) {
        int lo = 0, hi = nitems - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (ends[mid] <= w) lo = mid + 1;
            else hi = mid;
        }
        // the search runs on LDS values, which live in vector registers; the result is
        // the same on every lane, and saying so keeps every later descriptor and op
        // table read a scalar (uniform) load
        lo = __builtin_amdgcn_readfirstlane(lo);
        const BatchItem& it = items[lo];
        const long long tile = w - (it.tile_end - it.ntiles);
        // pointers read from memory carry no address space: state in global memory
        // (global, not flat, loads and stores), plan tables read-only (scalar loads)
        float* alds = reinterpret_cast<float*>(smem + (sizeof(C) << it.a.m));
        if (it.a.d_len > 0 && lo != staged) {   // diagonal tables only: matrix operands stay in global memory
            stage_operands(alds, (cptr<float>)it.apool, it.a.a_off, it.a.d_len);
            __syncthreads();
            staged = lo;
        }
        run_tile<C, WIDE, false>((gptr<C>)it.state, lds, it.a, tile, (cptr<DevOp>)it.ops, (cptr<C>)it.pool,
                          (cptr<int>)it.ipool, (cptr<float>)it.apool, alds, it.from_zero != 0);
        __syncthreads();   // the next work item reuses the LDS tile
    }
}

// Fill with 16-byte stores: every chunk is `rest` except chunk 0, which is `first`
// (|0...0> has amplitude 1 at index 0).  The state's byte size is a multiple of 16.
__global__ __launch_bounds__(kThreads) void k_fill16(uint4* __restrict__ st, long long nchunks, uint4 first,
                                                     uint4 rest)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nchunks; i += stride)
        st[i] = (i == 0) ? first : rest;
}

// ------------------------------------------------------------------ reductions

struct NSum {
    double s, c;
};

__device__ __forceinline__ void nadd(NSum& a, double x)
{
    const double t = a.s + x;
    a.c += (fabs(a.s) >= fabs(x)) ? ((a.s - t) + x) : ((x - t) + a.s);
    a.s = t;
}

__device__ __forceinline__ NSum ncombine(NSum a, NSum b)
{
    NSum r = a;
    nadd(r, b.s);
    r.c += b.c;
    return r;
}

// Butterfly over a wave's lanes in a fixed order; every lane returns the sum.
__device__ __forceinline__ NSum wave_reduce(NSum v)
{
    for (int d = 32; d >= 1; d >>= 1) {
        NSum o;
        o.s = __shfl_xor(v.s, d);
        o.c = __shfl_xor(v.c, d);
        v = ((threadIdx.x & d) == 0) ? ncombine(v, o) : ncombine(o, v);
    }
    return v;
}

// Fixed-order workgroup reduction of Neumaier pairs: butterfly within each wave,
// then wave results combined in wave order by thread 0.  Returns the result in
// thread 0.
__device__ NSum block_reduce(NSum v, NSum* scratch)
{
    v = wave_reduce(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) scratch[w] = v;
    __syncthreads();
    NSum r = {0.0, 0.0};
    if (threadIdx.x == 0) {
        r = scratch[0];
        for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = ncombine(r, scratch[i]);
    }
    __syncthreads();
    return r;
}

// Squared norm: 16-byte loads (two complex64 or one complex128 amplitude per chunk),
// eight independent loads in flight per thread; each group of eight |a|^2 (FP64,
// exact for FP32 inputs) is summed pairwise and added to a Neumaier pair.
template <typename R>
__global__ __launch_bounds__(kThreads) void k_norm(const float4* __restrict__ st, long long nchunks,
                                                   double* __restrict__ partial)
{
    __shared__ NSum scratch[kThreads / 64];
    constexpr int U = 8;
    NSum a = {0.0, 0.0};
    const long long stride = (long long)gridDim.x * blockDim.x;
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    auto sq = [](float4 v) -> double {
        if constexpr (sizeof(R) == 4) {
            return ((double)v.x * v.x + (double)v.y * v.y) + ((double)v.z * v.z + (double)v.w * v.w);
        } else {
            const double2 d = *reinterpret_cast<const double2*>(&v);
            return d.x * d.x + d.y * d.y;
        }
    };
    for (; i + (U - 1) * stride < nchunks; i += U * stride) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = st[i + u * stride];
        double p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = sq(v[u]);
#pragma unroll
        for (int h = 1; h < U; h <<= 1)
#pragma unroll
            for (int u = 0; u < U; u += 2 * h) p[u] += p[u + h];
        nadd(a, p[0]);
    }
    for (; i < nchunks; i += stride) nadd(a, sq(st[i]));
    const NSum r = block_reduce(a, scratch);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = r.s;
        partial[2 * blockIdx.x + 1] = r.c;
    }
}

// The threads' sums of a launch's terms to one partial each, eight terms at a time through LDS
// (w: 8 x 256 doubles, free to overwrite); wave w finishes terms w and w + 4 of the eight in a
// fixed order.  (A workgroup reduction per term cost two barriers and six shuffles of every
// wave each: two 12-qubit complex128 states 19 -> 9 us.)
__device__ __forceinline__ void finish_terms(const double (&acc)[kMaxTermsPerLaunch], int nterms, double* w,
                                             double* __restrict__ partial)
{
#pragma unroll
    for (int i0 = 0; i0 < kMaxTermsPerLaunch; i0 += 8) {
        if (i0 >= nterms) break;
        __syncthreads();
#pragma unroll
        for (int i = i0; i < i0 + 8; ++i) w[((i - i0) << kLogThreads) + threadIdx.x] = acc[i];
        __syncthreads();
        for (int i = i0 + (threadIdx.x >> 6); i < i0 + 8 && i < nterms; i += kThreads / 64) {
            const double* v = w + ((i - i0) << kLogThreads) + (threadIdx.x & 63);
            NSum r = {v[0], 0.0};
            nadd(r, v[64]);
            nadd(r, v[128]);
            nadd(r, v[192]);
            r = wave_reduce(r);
            if ((threadIdx.x & 63) == 0) {
                partial[((long long)blockIdx.x * nterms + i) * 2] = r.s;
                partial[((long long)blockIdx.x * nterms + i) * 2 + 1] = r.c;
            }
        }
    }
}

// Pauli matrix elements over tiles: value_t = sum_k Re( i^ny conj(a[k xor x]) b[k] ) *
// (-1)^popcount(k & zy), i.e. Re <a|P_t|b> (ny may carry an extra 3 to give Im instead),
// for terms with X/Y factors (Z-only terms go to k_expval_z; here they take the generic
// per-element path).  Each term's X/Y support lies inside the tile.  A thread owns the
// local elements e = 256 j + tid (j < NS) of every tile and keeps them in registers; the
// partner amplitudes a[e xor x] come from an LDS copy of the tile of a.  FP64 per thread;
// the workgroup partials are combined in a fixed order.
struct TermRow {
    int x, z, q, pad;
    long long g;
    double k[4];   // two-state weights (see TermArgs::kw)
};

template <typename C, int NS, bool TWO>
__device__ __forceinline__ void expval_tiles(gptr<C> __restrict__ sa, gptr<C> __restrict__ sb,
                                             C* __restrict__ tla, const TermRow* __restrict__ rows,
                                             const PassArgs& a, int nterms, long long ntiles,
                                             double (&acc)[kMaxTermsPerLaunch])
{
    constexpr int LB = NS >= 32 ? 5 : NS >= 16 ? 4 : NS >= 8 ? 3 : NS >= 4 ? 2 : NS >= 2 ? 1 : 0;
    long long hs[LB > 0 ? LB : 1];
#pragma unroll
    for (int b = 0; b < LB; ++b) hs[b] = local_stride(a, kLogThreads + b);
    const int tid = threadIdx.x;
    const long long tl = local_off_bits(a, tid, 0, kLogThreads);
    auto soff = [&](int j) {
        long long so = 0;
#pragma unroll
        for (int b = 0; b < LB; ++b)
            if ((j >> b) & 1) so += hs[b];
        return so;
    };
    // real part of i^q w for w = conj(p) e
    auto phase_re = [](const C& p, const C& e, int q) {
        const double pr = (double)p.x * (double)e.x + (double)p.y * (double)e.y;
        const double pi = (double)p.x * (double)e.y - (double)p.y * (double)e.x;
        return (q == 0) ? pr : (q == 1) ? -pi : (q == 2) ? -pr : pi;
    };
    for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const long long base = tile_base(a, tile);
        C av[NS], bv[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) av[j] = sa[base + tl + soff(j)];
        if (TWO) {
#pragma unroll
            for (int j = 0; j < NS; ++j) bv[j] = sb[base + tl + soff(j)];
        }
#pragma unroll
        for (int j = 0; j < NS; ++j) tla[(j << kLogThreads) + tid] = av[j];
        __syncthreads();
        // the term index stays a compile-time constant so that acc lives in registers;
        // term rows come from LDS so that nothing per term is hoisted out of the tile loop
#pragma unroll
        for (int i = 0; i < kMaxTermsPerLaunch; ++i) {
            if (i < nterms) {
                const int x = __builtin_amdgcn_readfirstlane(rows[i].x);
                const int z = __builtin_amdgcn_readfirstlane(rows[i].z);
                const int q = __builtin_amdgcn_readfirstlane(rows[i].q);
                const long long g = rows[i].g;
                const bool gneg = __popcll(base & g) & 1;   // Z bits outside the tile
                double val = 0.0;
                if (!TWO && x != 0) {
                    // <a|P|a> over pairs (e, e ^ x), e with x's lowest bit clear: with
                    // w = conj(a[e ^ x]) a[e] the pair adds s(e) i^q (w + (-1)^{|x & z|}
                    // conj(w)), whose real part is 2 Re(i^q w) when |x & z| is even and
                    // 2 Re(i^(q+1) Im(w)) when it is odd: half the elements, one product
                    const int lb = __ffs(x) - 1;
                    const bool odd = __popc(x & z) & 1;
                    // T / 2 pairs, NP per thread (a 2^8 tile has fewer pairs than threads);
                    // the unrolled loop issues every partner read before the arithmetic
                    constexpr int NP = NS >= 2 ? NS / 2 : 1;
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const int pr = p * kThreads + tid;
                        if (NS == 1 && pr >= (kThreads >> 1)) break;
                        const int e = ((pr >> lb) << (lb + 1)) | (pr & ((1 << lb) - 1));
                        const C ap = tla[e ^ x];
                        const C ae = tla[e];
                        double v;
                        if (!odd) {
                            const double re = (double)ap.x * (double)ae.x + (double)ap.y * (double)ae.y;
                            v = (q == 0) ? re : (q == 2) ? -re : 0.0;
                        } else {
                            const double im = (double)ap.x * (double)ae.y - (double)ap.y * (double)ae.x;
                            v = (q == 1) ? -im : (q == 3) ? im : 0.0;
                        }
                        val += (__popc(e & z) & 1) ? -v : v;
                    }
                    val *= 2.0;
                } else if (!TWO) {
                    // x == 0 (Z-only terms normally go to k_expval_z): per element from LDS
#pragma unroll 1
                    for (int j = 0; j < NS; ++j) {
                        const int e = (j << kLogThreads) | tid;
                        const C ae = tla[e];
                        const double v = phase_re(ae, ae, q);
                        val += (__popc(e & z) & 1) ? -v : v;
                    }
                } else if (TWO) {
                    // per element: the partner from LDS, b[e] from this thread's registers,
                    // the weight by the parity of e's Z/Y bits (the bits outside the tile
                    // swap the two weights for the whole tile)
                    const double k0r = gneg ? rows[i].k[2] : rows[i].k[0], k0i = gneg ? rows[i].k[3] : rows[i].k[1];
                    const double k1r = gneg ? rows[i].k[0] : rows[i].k[2], k1i = gneg ? rows[i].k[1] : rows[i].k[3];
#pragma unroll
                    for (int j = 0; j < NS; ++j) {
                        const int e = (j << kLogThreads) | tid;
                        const C ap = tla[e ^ x];
                        const double wr = (double)ap.x * (double)bv[j].x + (double)ap.y * (double)bv[j].y;
                        const double wi = (double)ap.x * (double)bv[j].y - (double)ap.y * (double)bv[j].x;
                        const bool odd = __popc(e & z) & 1;
                        val += (odd ? k1r : k0r) * wr - (odd ? k1i : k0i) * wi;
                    }
                }
                acc[i] += (!TWO && gneg) ? -val : val;
            }
        }
        __syncthreads();   // the next tile overwrites LDS
    }
}

// LDS bytes of one k_expval workgroup for a tile of 2^m amplitudes: the tile of a, and at the
// end eight terms' sums.
__host__ __device__ constexpr size_t expval_lds_bytes(size_t elem, int m)
{
    return (elem << m) > sizeof(double) * 8 * kThreads ? elem << m : sizeof(double) * 8 * kThreads;
}

template <typename C, bool TWO>
__global__ __launch_bounds__(kThreads) void k_expval(const C* __restrict__ sa, const C* __restrict__ sb,
                                                     const PassArgs a, const TermArgs t, long long ntiles,
                                                     double* __restrict__ partial)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TermRow rows[kMaxTermsPerLaunch];
    if (threadIdx.x < t.nterms) {
        const int i = threadIdx.x;
        rows[i] = TermRow{t.xloc[i], t.zloc[i], t.ny[i] & 3, 0, t.zglob[i], {t.kw[i][0], t.kw[i][1], t.kw[i][2], t.kw[i][3]}};
    }
    __syncthreads();
    double acc[kMaxTermsPerLaunch];
#pragma unroll
    for (int i = 0; i < kMaxTermsPerLaunch; ++i) acc[i] = 0.0;
    gptr<C> ga = (gptr<C>)const_cast<C*>(sa), gb = (gptr<C>)const_cast<C*>(sb);
    C* tla = reinterpret_cast<C*>(smem);
    switch (a.m - kLogThreads) {   // tiles of 2^8 .. 2^11 amplitudes
    case 0: expval_tiles<C, 1, TWO>(ga, gb, tla, rows, a, t.nterms, ntiles, acc); break;
    case 1: expval_tiles<C, 2, TWO>(ga, gb, tla, rows, a, t.nterms, ntiles, acc); break;
    case 2: expval_tiles<C, 4, TWO>(ga, gb, tla, rows, a, t.nterms, ntiles, acc); break;
    default: expval_tiles<C, 8, TWO>(ga, gb, tla, rows, a, t.nterms, ntiles, acc); break;
    }
    finish_terms(acc, t.nterms, reinterpret_cast<double*>(smem), partial);
}

// Terms with X/Y factors on few qubits (one state: at most RB = 4; two states: one qubit, its
// Z factor the term's only one, as generators have): the tile goes to LDS once, and in each
// round every thread reads the 2^RB elements that differ in the round's kept bits (RB = 3 for
// two states), so a term pairs registers of one thread: per pair one product and one signed
// addition instead of two LDS reads, index arithmetic and four conversions.  A round serves
// every term inside its bits (a field of single X or Y factors on 12 tile qubits takes three
// rounds).  The next tile's loads fly during the rounds.  What bounds it on large states is
// the read of the state, on ones that the last-level cache holds the FP64 arithmetic and the
// chain of LDS accesses of each term: 30 X terms at 30 qubits complex64 (4 launches) 16.0 ->
// 9.1 ms; 22 Y terms of two 22-qubit complex64 states (3 launches) 155 -> 90 us, of which
// the parity of a pair being known at compile time and the loads ahead gave the last 25.
constexpr int kRowBits = 8;   // 256 threads

// Sum over one thread's pairs (p, p ^ X) of Re (odd: Im) conj(a[p ^ X]) a[p] with the sign of
// p's kept Z bits.
template <int X, int EL>
__device__ __forceinline__ double pair_sum(const double (&re)[EL], const double (&im)[EL], int zr, bool odd)
{
    constexpr int low = X & -X;
    double s = 0.0;
    if (!odd) {
#pragma unroll
        for (int p = 0; p < EL; ++p)
            if (!(p & low)) s = fma(re[p ^ X] * re[p] + im[p ^ X] * im[p], (__popc(p & zr) & 1) ? -1.0 : 1.0, s);
    } else {
#pragma unroll
        for (int p = 0; p < EL; ++p)
            if (!(p & low)) s = fma(re[p ^ X] * im[p] - im[p ^ X] * re[p], (__popc(p & zr) & 1) ? -1.0 : 1.0, s);
    }
    return s;
}

// Two states: w[0] + i w[1] = the sum of conj(a[p ^ X]) b[p] over the p whose kept Z bits have
// even parity, w[2] + i w[3] over the odd ones.
template <int X, int Z, int EL>
__device__ __forceinline__ void pair_sums2(const double (&ar)[EL], const double (&ai)[EL], const double (&br)[EL],
                                           const double (&bi)[EL], double (&w)[4])
{
#pragma unroll
    for (int p = 0; p < EL; ++p) {
        const int o = (__builtin_popcount(p & Z) & 1) * 2;
        w[o] = fma(ar[p ^ X], br[p], w[o]);
        w[o + 1] = fma(ar[p ^ X], bi[p], w[o + 1]);
        w[o] = fma(ai[p ^ X], bi[p], w[o]);
        w[o + 1] = fma(-ai[p ^ X], br[p], w[o + 1]);
    }
}

// The value of another lane of the same group of four (CTRL: a quad permutation).
template <int CTRL>
__device__ __forceinline__ double quad_swap(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <typename C, bool TWO>
__global__ __launch_bounds__(kThreads) void k_expval_r(const C* __restrict__ sa, const C* __restrict__ sb,
                                                       const PassArgs a, const TermArgs t, const RoundArgs rd,
                                                       long long ntiles, double* __restrict__ partial)
{
    constexpr int RB = TWO ? kRoundBitsTwo : kRoundBits, EL = 1 << RB, M = kRowBits + RB;
    constexpr int W = sizeof(C) == 8 ? 2 : 1, LW = W == 2 ? 1 : 0, NS = EL / W;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TermRow rows[kMaxTermsPerLaunch];
    __shared__ int rbits[kMaxRounds], rend[kMaxRounds], qn[kMaxTermsPerLaunch];
    const int tid = threadIdx.x;
    if (tid < t.nterms) {
        // x: kept X bits, z: kept Z bits, q: Z bits of the thread's part
        rows[tid] = TermRow{rd.xr[tid], rd.zr[tid], rd.zl[tid], 0, t.zglob[tid],
                            {t.kw[tid][0], t.kw[tid][1], t.kw[tid][2], t.kw[tid][3]}};
        qn[tid] = t.ny[tid] & 3;
    }
    if (tid < rd.nrounds) {
        rbits[tid] = rd.bits[tid];
        rend[tid] = rd.end[tid];
    }
    C* la = reinterpret_cast<C*>(smem);
    C* lb = la + (1 << M);
    double* sums = reinterpret_cast<double*>(la + ((TWO ? 2 : 1) << M));   // 64 per term
    for (int i = tid; i < t.nterms << 6; i += kThreads) sums[i] = 0.0;
    gptr<C> ga = (gptr<C>)const_cast<C*>(sa), gb = (gptr<C>)const_cast<C*>(sb);
    const long long tl = local_off_bits(a, tid << LW, LW, kRowBits + LW);
    floatx4 va[NS], vb[TWO ? NS : 1];
    auto load = [&](long long tile) {
        const long long o = tile_base(a, tile) + tl;
        load_tile<C, NS, W>(ga + o, a, va);
        if constexpr (TWO) load_tile<C, NS, W>(gb + o, a, vb);
    };
    load(blockIdx.x);
    __syncthreads();
    for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const long long base = tile_base(a, tile);
        put_tile<C, NS, W>(la, va);
        if constexpr (TWO) put_tile<C, NS, W>(lb, vb);
        lds_sync();
        if (tile + gridDim.x < ntiles) load(tile + gridDim.x);
        int i = 0;
        for (int r = 0; r < rd.nrounds; ++r) {
            const int bits = __builtin_amdgcn_readfirstlane(rbits[r]);
            const int end = __builtin_amdgcn_readfirstlane(rend[r]);
            int tb = tid;   // the thread's element with every kept bit clear
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int p = (bits >> (4 * b)) & 15;
                tb = ((tb >> p) << (p + 1)) | (tb & ((1 << p) - 1));
            }
            const int ut = swz<C>(tb);
            double ar[EL], ai[EL], br[TWO ? EL : 1], bi[TWO ? EL : 1];
#pragma unroll
            for (int p = 0; p < EL; ++p) {
                int o = 0;
#pragma unroll
                for (int b = 0; b < RB; ++b)
                    if ((p >> b) & 1) o |= 1 << ((bits >> (4 * b)) & 15);
                const int at = ut ^ swz<C>(o);
                const C v = la[at];
                ar[p] = v.x;
                ai[p] = v.y;
                if constexpr (TWO) {
                    const C u = lb[at];
                    br[p] = u.x;
                    bi[p] = u.y;
                }
            }
            for (; i < end; ++i) {
                const int x = __builtin_amdgcn_readfirstlane(rows[i].x);
                const int z = __builtin_amdgcn_readfirstlane(rows[i].z);
                const int zl = __builtin_amdgcn_readfirstlane(rows[i].q);
                const bool par = (__popc(tb & zl) + __popcll(base & rows[i].g)) & 1;
                // (keeps the products of all supports from being formed ahead of the loop)
#pragma unroll
                for (int p = 0; p < EL; ++p) asm volatile("" : "+v"(ar[p]), "+v"(ai[p]));
                double val;
                if constexpr (!TWO) {
                    const bool odd = x & 16;
                    switch (x & 15) {
                    case 1: val = pair_sum<1>(ar, ai, z, odd); break;
                    case 2: val = pair_sum<2>(ar, ai, z, odd); break;
                    case 3: val = pair_sum<3>(ar, ai, z, odd); break;
                    case 4: val = pair_sum<4>(ar, ai, z, odd); break;
                    case 5: val = pair_sum<5>(ar, ai, z, odd); break;
                    case 6: val = pair_sum<6>(ar, ai, z, odd); break;
                    case 7: val = pair_sum<7>(ar, ai, z, odd); break;
                    case 8: val = pair_sum<8>(ar, ai, z, odd); break;
                    case 9: val = pair_sum<9>(ar, ai, z, odd); break;
                    case 10: val = pair_sum<10>(ar, ai, z, odd); break;
                    case 11: val = pair_sum<11>(ar, ai, z, odd); break;
                    case 12: val = pair_sum<12>(ar, ai, z, odd); break;
                    case 13: val = pair_sum<13>(ar, ai, z, odd); break;
                    case 14: val = pair_sum<14>(ar, ai, z, odd); break;
                    default: val = pair_sum<15>(ar, ai, z, odd); break;
                    }
                    if (par) val = -val;
                } else {
                    double w[4] = {0.0, 0.0, 0.0, 0.0};
                    switch (x & 7) {   // one kept bit (plan_elements), its Z factor present or not
                    case 1: z ? pair_sums2<1, 1>(ar, ai, br, bi, w) : pair_sums2<1, 0>(ar, ai, br, bi, w); break;
                    case 2: z ? pair_sums2<2, 2>(ar, ai, br, bi, w) : pair_sums2<2, 0>(ar, ai, br, bi, w); break;
                    default: z ? pair_sums2<4, 4>(ar, ai, br, bi, w) : pair_sums2<4, 0>(ar, ai, br, bi, w); break;
                    }
                    const double er = par ? w[2] : w[0], ei = par ? w[3] : w[1];
                    const double orr = par ? w[0] : w[2], oi = par ? w[1] : w[3];
                    val = rows[i].k[0] * er - rows[i].k[1] * ei + rows[i].k[2] * orr - rows[i].k[3] * oi;
                }
                // four lanes share a sum in LDS: a run-time term number cannot index registers
                val += quad_swap<0xb1>(val);
                val += quad_swap<0x4e>(val);
                if ((tid & 3) == 0) sums[(i << 6) + (tid >> 2)] += val;
            }
        }
        lds_sync();   // the next tile overwrites LDS
    }
    // wave w finishes terms w, w + 4, ...: its lanes' 64 sums in a fixed order
    for (int i = tid >> 6; i < t.nterms; i += kThreads / 64) {
        const NSum v = wave_reduce(NSum{sums[(i << 6) + (tid & 63)], 0.0});
        if ((tid & 63) == 0) {
            double f = 1.0;
            if (!TWO) {
                // <a|P|a>: a pair adds 2 Re(i^q w) when |x & z| is even and 2 Re(i^(q+1) Im w)
                // when it is odd
                const int q = qn[i];
                f = (rows[i].x & 16) ? (q == 1 ? -2.0 : q == 3 ? 2.0 : 0.0) : (q == 0 ? 2.0 : q == 2 ? -2.0 : 0.0);
            }
            partial[((long long)blockIdx.x * t.nterms + i) * 2] = f * v.s;
            partial[((long long)blockIdx.x * t.nterms + i) * 2 + 1] = f * v.c;
        }
    }
}

// Z-only terms: <a|P|b> with P = i^q Z^z sums s(k) i^q conj(a_k) b_k.  A thread's NS elements
// of a tile (the next tile's are loaded, 16 bytes at a time, while this one's are summed) are
// Walsh-transformed over the tile bits they differ in, after which a term is one lookup of
// its transform slot times signs that are fixed per thread (thread-id bits of z, the phase)
// or per tile (Z bits outside the tile, a uniform mask built from the tile number's bits).
// Each thread reads back only the transform values it wrote, so its LDS slots are private:
// no barrier, no tile copy.  Slot bits of complex64: local bit 0 (a 16-byte unit's two
// elements), then bits 9 and up; of complex128: bits 8 and up.
template <typename C, int NS, bool TWO>
__device__ __forceinline__ void expval_z_tiles(gptr<C> __restrict__ sa, gptr<C> __restrict__ sb,
                                               double* __restrict__ w, const PassArgs& a, const ZTermArgs& t,
                                               long long ntiles, double (&acc)[kMaxTermsPerLaunch])
{
    constexpr int W = sizeof(C) == 8 && NS >= 2 ? 2 : 1, LW = W == 2 ? 1 : 0, NU = NS / W;   // units per thread
    using V = typename std::conditional<sizeof(C) * W == 16, floatx4, float __attribute__((ext_vector_type(2)))>::type;
    const int tid = threadIdx.x;
    const long long tl = local_off_bits(a, tid << LW, LW, kLogThreads + LW);
    auto load = [&](gptr<C> s, long long tile, V (&v)[NU]) {
        const gptr<C> p = s + tile_base(a, tile) + tl;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            long long o = 0;
#pragma unroll
            for (int b = 0; (1 << b) < NU; ++b)
                if ((u >> b) & 1) o += local_stride(a, kLogThreads + LW + b);
            v[u] = *(gptr<const V>)(p + o);
        }
    };
    unsigned tmask = t.neg;   // per-thread signs: the phase and the thread-id bits of z
#pragma unroll
    for (int i = 0; i < kMaxTermsPerLaunch; ++i)
        if (i < t.nterms) tmask ^= (unsigned)(__popc(tid & t.zlo[i]) & 1) << i;
    double* wt = w + tid;     // this thread's slots: wt[j << 8], j < NS (real), NS + j (imaginary)
    V va[NU], vb[TWO ? NU : 1];
    load(sa, blockIdx.x, va);
    if constexpr (TWO) load(sb, blockIdx.x, vb);
    for (long long tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        unsigned gm = 0;      // per-tile signs: Z bits outside the tile
#pragma unroll
        for (int b = 0; b < kMaxTileIndexBits; ++b)
            if ((tile >> b) & 1) gm ^= t.gcol[b];
        struct E { C c[W]; };
        double re[NS], im[NS];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const E ea = __builtin_bit_cast(E, va[u]);
            E eb = ea;
            if constexpr (TWO) eb = __builtin_bit_cast(E, vb[u]);
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int j = W * u + k;
                const C av = ea.c[k], bv = eb.c[k];
                re[j] = (double)av.x * (double)bv.x + (double)av.y * (double)bv.y;
                im[j] = TWO ? (double)av.x * (double)bv.y - (double)av.y * (double)bv.x : 0.0;
            }
        }
        if (tile + gridDim.x < ntiles) {
            load(sa, tile + gridDim.x, va);
            if constexpr (TWO) load(sb, tile + gridDim.x, vb);
        }
#pragma unroll
        for (int h = 1; h < NS; h <<= 1) {
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                if (j & h) continue;
                const double u = re[j], v = re[j | h];
                re[j] = u + v;
                re[j | h] = u - v;
                if (TWO) {
                    const double ui = im[j], vi = im[j | h];
                    im[j] = ui + vi;
                    im[j | h] = ui - vi;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            wt[j << kLogThreads] = re[j];
            if (TWO) wt[(NS + j) << kLogThreads] = im[j];
        }
        const unsigned sg = gm ^ tmask;
#pragma unroll
        for (int i = 0; i < kMaxTermsPerLaunch; ++i) {
            if (i < t.nterms && (TWO || !((t.zero >> i) & 1))) {
                const double v = wt[t.zoff[i] << kLogThreads];
                acc[i] += ((sg >> i) & 1) ? -v : v;
            }
        }
    }
}

template <typename C, bool TWO>
__global__ __launch_bounds__(kThreads) void k_expval_z(const C* __restrict__ sa, const C* __restrict__ sb,
                                                       const PassArgs a, const ZTermArgs t, long long ntiles,
                                                       double* __restrict__ partial)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double* w = reinterpret_cast<double*>(smem);
    double acc[kMaxTermsPerLaunch];
#pragma unroll
    for (int i = 0; i < kMaxTermsPerLaunch; ++i) acc[i] = 0.0;
    gptr<C> ga = (gptr<C>)const_cast<C*>(sa), gb = (gptr<C>)const_cast<C*>(sb);
    switch (a.m - kLogThreads) {   // tiles of 2^8 .. 2^11 amplitudes
    case 0: expval_z_tiles<C, 1, TWO>(ga, gb, w, a, t, ntiles, acc); break;
    case 1: expval_z_tiles<C, 2, TWO>(ga, gb, w, a, t, ntiles, acc); break;
    case 2: expval_z_tiles<C, 4, TWO>(ga, gb, w, a, t, ntiles, acc); break;
    default: expval_z_tiles<C, 8, TWO>(ga, gb, w, a, t, ntiles, acc); break;
    }
    finish_terms(acc, t.nterms, w, partial);
}

// Whole states below 256 amplitudes: one workgroup, a wave per term, straight from the
// definition (the tile is the state).
template <typename C, bool TWO>
__global__ __launch_bounds__(kThreads) void k_expval_small(const C* __restrict__ sa, const C* __restrict__ sb,
                                                           int n, const TermArgs t, double* __restrict__ partial)
{
    const int N = 1 << n, lane = threadIdx.x & 63;
    for (int i = threadIdx.x >> 6; i < t.nterms; i += kThreads / 64) {
        NSum v = {0.0, 0.0};
        for (int e = lane; e < N; e += 64) {
            const C ap = sa[e ^ t.xloc[i]];
            const C be = TWO ? sb[e] : sa[e];
            const double re = (double)ap.x * (double)be.x + (double)ap.y * (double)be.y;
            const double im = (double)ap.x * (double)be.y - (double)ap.y * (double)be.x;
            const bool odd = __popc(e & t.zloc[i]) & 1;
            double val;
            if (TWO) {   // the two-state weights (TermArgs::kw)
                val = (odd ? t.kw[i][2] : t.kw[i][0]) * re - (odd ? t.kw[i][3] : t.kw[i][1]) * im;
            } else {
                const int q = t.ny[i] & 3;
                val = (q == 0) ? re : (q == 1) ? -im : (q == 2) ? -re : im;
                if (odd) val = -val;
            }
            nadd(v, val);
        }
        v = wave_reduce(v);
        if (lane == 0) {
            partial[(long long)i * 2] = v.s;
            partial[(long long)i * 2 + 1] = v.c;
        }
    }
}

// out = sum_t coeff_t P_t in (accumulate != 0: out += ...), with
// (P in)[k] = i^ny (-1)^popcount((k xor x) & zy) in[k xor x].  Each thread gathers its
// amplitude's partners straight from HBM / L2.
template <typename C>
__global__ __launch_bounds__(kThreads) void k_pauli_apply(const C* __restrict__ in, C* __restrict__ out,
                                                          long long N, const PauliSumArgs p, int accumulate)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += stride) {
        double re = 0.0, im = 0.0;
        if (accumulate) {
            const C o = out[k];
            re = o.x;
            im = o.y;
        }
        for (int i = 0; i < p.nterms; ++i) {
            const long long j = k ^ p.x[i];
            const C v = in[j];
            double vr = v.x, vi = v.y;
            const int q = p.ny[i] & 3;   // multiply by i^q
            double tr = (q == 0) ? vr : (q == 1) ? -vi : (q == 2) ? -vr : vi;
            double ti = (q == 0) ? vi : (q == 1) ? vr : (q == 2) ? -vi : -vr;
            const double c = (__popcll(j & p.z[i]) & 1) ? -p.coeff[i] : p.coeff[i];
            re = fma(c, tr, re);
            im = fma(c, ti, im);
        }
        C o;
        o.x = re;
        o.y = im;
        out[k] = o;
    }
}

// ------------------------------------------------------------------ sampling

// Probability of entry i: |alpha_i|^2 in FP64 (state sources) or a table entry.
__device__ __forceinline__ double prob_of(float2 v) { return (double)v.x * v.x + (double)v.y * v.y; }
__device__ __forceinline__ double prob_of(double2 v) { return v.x * v.x + v.y * v.y; }

template <int SRC>
__device__ __forceinline__ double prob_at(const void* src, long long i)
{
    if constexpr (SRC == 0) {
        return prob_of(reinterpret_cast<const float2*>(src)[i]);
    } else if constexpr (SRC == 1) {
        return prob_of(reinterpret_cast<const double2*>(src)[i]);
    } else {
        return reinterpret_cast<const double*>(src)[i];
    }
}

// Place of a chunk's entry i in LDS: one double of padding per 16, so that the 16 entries a
// thread sums in order lie 17 doubles from its neighbours' (no bank conflicts).
__device__ __host__ constexpr int scan_at(int i) { return i + (i >> 4); }

// Inclusive prefix sums of one chunk (2^cb entries, cb <= 12) into scan[scan_at(i)] in LDS, in
// a fixed order: each thread sums its run of E consecutive entries sequentially, the
// thread totals are scanned within each wave (shuffles) and across the four waves.
// Every chunk, in both sampling kernels, goes through this one function, so a chunk's
// total and its last prefix sum are the same number.  Full chunks of a state come in by
// 16-byte loads of neighbouring lanes and go to the threads' runs through LDS (each thread
// reading its own run from memory touched a cache line per lane: 2^16 chunks of a 28-qubit
// complex64 state 1.38 -> 0.55 ms).
template <int SRC>
__device__ void chunk_scan(const void* src, long long chunk, int cb, double* scan, double* wsum)
{
    const int size = 1 << cb;
    const int E = size > kThreads ? size / kThreads : 1;
    const int tid = threadIdx.x;
    const long long base = chunk << cb;
    if (SRC != 2 && size >= 2 * kThreads) {
        constexpr int W = SRC == 0 ? 2 : 1;   // entries per 16 bytes
        using V = typename std::conditional<SRC == 0, floatx4, doublex2>::type;
        const V* p = reinterpret_cast<const V*>(src) + base / W;
        for (int u0 = tid; u0 < size / W; u0 += 8 * kThreads) {
            V v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (u0 + k * kThreads < size / W) v[k] = p[u0 + k * kThreads];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int u = u0 + k * kThreads;
                if (u >= size / W) break;
                if constexpr (SRC == 0) {
                    scan[scan_at(2 * u)] = prob_of(float2{v[k].x, v[k].y});
                    scan[scan_at(2 * u + 1)] = prob_of(float2{v[k].z, v[k].w});
                } else if constexpr (SRC == 1) {
                    scan[scan_at(u)] = prob_of(double2{v[k].x, v[k].y});
                }
            }
        }
    } else {
        for (int i = tid; i < size; i += kThreads) scan[scan_at(i)] = prob_at<SRC>(src, base + i);
    }
    __syncthreads();
    double run = 0.0;
    const bool mine = tid * E < size;
    if (mine) {
        for (int i = 0; i < E; ++i) {
            run += scan[scan_at(tid * E + i)];
            scan[scan_at(tid * E + i)] = run;   // prefix within the thread's run
        }
    }
    // inclusive scan of the thread totals: within the wave, then across waves
    double x = mine ? run : 0.0;
    const int lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    double woff = 0.0;
    for (int i = 0; i < w; ++i) woff += wsum[i];
    const double off = woff + x - (mine ? run : 0.0);   // exclusive offset of this thread
    if (mine) {
        for (int i = 0; i < E; ++i) scan[scan_at(tid * E + i)] += off;
    }
    __syncthreads();
}

template <int SRC>
__global__ __launch_bounds__(kThreads) void k_chunk_totals(const void* __restrict__ src, int cb,
                                                           double* __restrict__ totals)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double* scan = reinterpret_cast<double*>(smem);
    __shared__ double wsum[kThreads / 64];
    chunk_scan<SRC>(src, blockIdx.x, cb, scan, wsum);
    if (threadIdx.x == 0) totals[blockIdx.x] = scan[scan_at((1 << cb) - 1)];
}

// One workgroup per listed chunk: rebuild the chunk's prefix sums, then every shot of
// the chunk finds the smallest k with residual < scan[k] (binary search).  Residuals
// are clamped into [0, total) first: below zero (rounding) picks the first entry of
// nonzero probability, at or above the total picks the last one.
template <int SRC>
__global__ __launch_bounds__(kThreads) void k_sample_chunks(const void* __restrict__ src, int cb,
                                                            const SampleChunk* __restrict__ list,
                                                            const double* __restrict__ residual,
                                                            long long* __restrict__ outcome)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double* scan = reinterpret_cast<double*>(smem);
    __shared__ double wsum[kThreads / 64];
    const SampleChunk c = list[blockIdx.x];
    chunk_scan<SRC>(src, c.chunk, cb, scan, wsum);
    const int size = 1 << cb;
    const double total = scan[scan_at(size - 1)];
    const double below = nextafter(total, 0.0);
    for (long long i = c.lo + threadIdx.x; i < c.hi; i += kThreads) {
        double r = residual[i];
        r = r < 0.0 ? 0.0 : (r >= total ? below : r);
        int lo = 0, hi = size - 1;   // smallest k with r < scan[k]; scan[size - 1] > r
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (r < scan[scan_at(mid)]) hi = mid;
            else lo = mid + 1;
        }
        outcome[i] = (c.chunk << cb) + lo;
    }
}

template <typename C, typename R>
__global__ __launch_bounds__(kThreads) void k_probs_full(const C* __restrict__ st, long long N,
                                                         R* __restrict__ out)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        const C v = st[i];
        out[i] = v.x * v.x + v.y * v.y;
    }
}

// Marginal distribution of a state.  A workgroup sums the blocks of 2^cb consecutive
// amplitudes that share one value of the measured qubits above the block (H values, G
// workgroups each, `per` blocks a workgroup): every thread keeps a Neumaier pair for each of
// its places in the block (16-byte loads, the next block's loads ahead of this one's sums),
// and at the end the block's places that agree on the measured qubits inside it are added
// in a fixed order.  The state is read once, in order; 5 measured qubits of 27, complex64:
// 14.3 -> 0.3 ms with the final sum (a thread per output and chunk gathered single
// amplitudes, and one thread added an output's 32768 chunks).
template <typename C>
__global__ __launch_bounds__(kThreads) void k_marg_blocks(const C* __restrict__ st, const MargBlocks a,
                                                          double* __restrict__ partial, double* __restrict__ out)
{
    constexpr int W = 16 / sizeof(C), NU = 16 / W;   // 16-byte units per thread of a full block
    using V = typename Lane16<C>::T;
    __shared__ double val[1 << kMargBlockBits];
    __shared__ NSum part[kThreads];
    const int tid = threadIdx.x, size = 1 << a.cb;
    const long long h = blockIdx.x / a.G, g = blockIdx.x % a.G;
    auto deposit = [](long long v, const int* pos, int k) {
        long long o = 0;
        for (int j = 0; j < k; ++j) o |= ((v >> j) & 1) << pos[j];
        return o;
    };
    const long long hbase = deposit(h, a.hq, a.nh);
    if (size == 1 << kMargBlockBits) {
        NSum acc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = NSum{0.0, 0.0};
        V v[NU];
        auto load = [&](long long r) {
            const V* p = reinterpret_cast<const V*>(st + (hbase | deposit(r, a.rest, a.nr))) + tid;
#pragma unroll
            for (int u = 0; u < NU; ++u) v[u] = p[u << kLogThreads];
        };
        load(g * a.per);
        for (long long r = g * a.per; r < (g + 1) * a.per; ++r) {
            double p[16];
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if constexpr (W == 2) {
                    p[2 * u] = (double)v[u].x * v[u].x + (double)v[u].y * v[u].y;
                    p[2 * u + 1] = (double)v[u].z * v[u].z + (double)v[u].w * v[u].w;
                } else {
                    p[u] = v[u].x * v[u].x + v[u].y * v[u].y;
                }
            }
            if (r + 1 < (g + 1) * a.per) load(r + 1);
#pragma unroll
            for (int i = 0; i < 16; ++i) nadd(acc[i], p[i]);
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int w = 0; w < W; ++w)
                val[W * ((u << kLogThreads) + tid) + w] = acc[W * u + w].s + acc[W * u + w].c;
    } else {   // smaller blocks: a place per thread and step
        for (int e = tid; e < size; e += kThreads) {
            NSum s = {0.0, 0.0};
            for (long long r = g * a.per; r < (g + 1) * a.per; ++r) {
                const C v = st[hbase | deposit(r, a.rest, a.nr) | e];
                const double x = v.x, y = v.y;
                nadd(s, x * x + y * y);
            }
            val[e] = s.s + s.c;
        }
    }
    __syncthreads();
    // output ol of the block: tp threads each add a share of its 2^(cb - nl) places.  The outputs
    // (places) of a thread's steps differ in at most four high bits: a thread's own bits are
    // laid out once, those of a step are sums of uniform strides (a loop over the bits per
    // step, with its reads of the argument arrays, took longer than the sums: a call for the 12
    // lowest of 15 qubits 49 -> 37 us, for 2 of 24 qubits complex128 124 -> 98).
    constexpr int SB = kMargBlockBits - kLogThreads;
    const int nout = 1 << a.nl, places = size >> a.nl, ltp = a.nl >= kLogThreads ? 0 : min(kLogThreads - a.nl, a.cb - a.nl);
    const int tp = 1 << ltp;
    const long long hout = deposit(h, a.ho, a.nh);
    const long long M = 1ll << a.m;
    const int ot = tid >> ltp, k0 = tid & (tp - 1);
    const int lt = (int)(deposit(ot, a.lq, min(a.nl, kLogThreads)) | deposit(k0, a.lr, ltp));
    const long long ht = hout | deposit(ot, a.lo, min(a.nl, kLogThreads));
    int ls[SB], ks[SB];
    long long hs[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
        const int o = kLogThreads + b, k = ltp + b;
        ls[b] = o < a.nl ? 1 << a.lq[o] : 0;
        hs[b] = o < a.nl ? 1ll << a.lo[o] : 0;
        ks[b] = k < a.cb - a.nl ? 1 << a.lr[k] : 0;
    }
    for (int i = 0; i << kLogThreads < nout; ++i) {   // (one step unless tp is 1)
        const bool mine = ot < nout;
        int at = lt;
        long long o = ht;
#pragma unroll
        for (int b = 0; b < SB; ++b)
            if ((i >> b) & 1) {
                at |= ls[b];
                o |= hs[b];
            }
        NSum s = {0.0, 0.0};
        if (mine)
            for (int c = 0; c << ltp < places; ++c) {
                int pl = at;
#pragma unroll
                for (int b = 0; b < SB; ++b)
                    if ((c >> b) & 1) pl |= ks[b];
                nadd(s, val[pl]);
            }
        if (tp > 1) {
            part[tid] = s;
            __syncthreads();
            if (k0 == 0 && mine)
                for (int k = 1; k < tp; ++k) s = ncombine(s, part[tid + k]);
        }
        if (k0 == 0 && mine) {
            if (a.G == 1) {
                out[o] = s.s + s.c;
            } else {
                partial[2 * (g * M + o)] = s.s;
                partial[2 * (g * M + o) + 1] = s.c;
            }
        }
    }
}

// Marginal of a density matrix's diagonal: the buffer holds vec(rho) of an a.n-qubit density
// matrix (index row + 2^n col) and the probability of basis state k is Re rho[k, k].
template <typename C>
__global__ __launch_bounds__(kThreads) void k_dm_marg(const C* __restrict__ st, const MargArgs a,
                                                      double* __restrict__ partial)
{
    const long long M = 1ll << a.m;
    const long long total = M * a.nchunks;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= total) return;
    const long long o = gid % M;
    const long long ch = gid / M;
    long long ob = 0;
    for (int j = 0; j < a.m; ++j) ob |= ((o >> j) & 1) << a.q[j];
    const int nr = a.n - a.m;
    NSum s = {0.0, 0.0};
    for (long long r = ch * a.chunk; r < (ch + 1) * a.chunk; ++r) {
        long long idx = ob;
        for (int j = 0; j < nr; ++j) idx |= ((r >> j) & 1) << a.rest[j];
        nadd(s, (double)st[idx + (idx << a.n)].x);
    }
    partial[2 * (ch * M + o)] = s.s;
    partial[2 * (ch * M + o) + 1] = s.c;
}

// out[o] = Neumaier sum over chunks of partial[(chunk*M + o)] (pairs), fixed order.  PER: a
// workgroup per output (many chunks); else a thread per output.
template <bool PER>
__global__ __launch_bounds__(kThreads) void k_sum_chunks(const double* __restrict__ partial, long long M,
                                                         long long nchunks, double* __restrict__ out)
{
    __shared__ NSum scratch[kThreads / 64];
    const long long o = PER ? (long long)blockIdx.x : (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= M) return;
    NSum s = {0.0, 0.0};
    for (long long c = PER ? threadIdx.x : 0; c < nchunks; c += PER ? kThreads : 1) {
        nadd(s, partial[2 * (c * M + o)]);
        s.c += partial[2 * (c * M + o) + 1];
    }
    if (PER) s = block_reduce(s, scratch);
    if (!PER || threadIdx.x == 0) out[o] = s.s + s.c;
}

// Per-qubit <Z_i> and norm of finished served states, batched: work item = one chunk of
// 2^14 consecutive amplitudes of one state.  Each workgroup writes, for its chunk, the
// chunk's sum of |alpha|^2 and, for the qubits inside the chunk (bits < 14), the sum
// over amplitudes with that bit set; qubits >= 14 are constant over a chunk and are
// resolved on the host from the chunk sum.  Fixed partition and reduction order.
// A thread's amplitudes e = 256 i + tid share the bits of tid, so it keeps one total and a
// sum per bit of i (pairwise sums of 16); the bits of tid are sums over threads, taken with
// the others from one copy of the threads' sums in LDS (a workgroup reduction per qubit of
// 2^12-amplitude chunks cost 26 barriers and more time than the read, and the host's
// additions over chunks four times as many).
template <typename C>
__global__ __launch_bounds__(kThreads) void k_zsum_batch(const ZItem* __restrict__ table, const BatchList* __restrict__ list,
                                                         double* __restrict__ partial)
{
    constexpr int HB = kZChunkQubits - kLogThreads;   // bits of i
    __shared__ double val[1 + HB][kThreads];
    const int nitems = list->count;
    if (nitems <= 0) return;
    const ZItem* __restrict__ items = table + list->first;
    const long long total = items[nitems - 1].chunk_end;
    const int tid = threadIdx.x;
    for (long long w = blockIdx.x; w < total; w += gridDim.x) {
        int lo = 0, hi = nitems - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (items[mid].chunk_end <= w) lo = mid + 1;
            else hi = mid;
        }
        const ZItem& it = items[lo];
        const long long chunk = w - (it.chunk_end - it.nchunks);
        const int cq = it.n < kZChunkQubits ? it.n : kZChunkQubits;
        const int len = 1 << cq;
        const C* st = (const C*)it.state + (chunk << cq);
        auto prob = [&](int e) {
            const C v = st[e];
            return (double)v.x * v.x + (double)v.y * v.y;
        };
        double tot = 0.0, bits[HB];
#pragma unroll
        for (int b = 0; b < HB; ++b) bits[b] = 0.0;
        if (len >= 16 * kThreads) {
            for (int s = 0; s < len / (16 * kThreads); ++s) {
                double p[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) p[i] = prob(((16 * s + i) << kLogThreads) + tid);
#pragma unroll
                for (int b = 0; b < 4; ++b) {   // p[i] for i < 16 >> b: sums over the bits below b
                    double odd = 0.0;
#pragma unroll
                    for (int i = 0; i < (16 >> b); i += 2) {
                        odd += p[i + 1];
                        p[i / 2] = p[i] + p[i + 1];
                    }
                    bits[b] += odd;
                }
                tot += p[0];
#pragma unroll
                for (int b = 4; b < HB; ++b)
                    if ((s >> (b - 4)) & 1) bits[b] += p[0];
            }
        } else {
            for (int i = 0; (i << kLogThreads) + tid < len; ++i) {
                const double p = prob((i << kLogThreads) + tid);
                tot += p;
#pragma unroll
                for (int b = 0; b < HB; ++b)
                    if ((i >> b) & 1) bits[b] += p;
            }
        }
        val[0][tid] = tot;
#pragma unroll
        for (int b = 0; b < HB; ++b) val[1 + b][tid] = bits[b];
        __syncthreads();
        double* out = partial + (it.partial_off + chunk * (kZChunkQubits + 1));
        // output o (0: the total, 1 + b: bit b), a wave each: bits of tid from the totals of the
        // threads that have them set, the others from their own sums of all threads
        const int lane = tid & 63;
        for (int o = tid >> 6; o <= kZChunkQubits; o += kThreads / 64) {
            const int b = o - 1;
            NSum v = {0.0, 0.0};
            if (b >= 0 && b < kLogThreads) {
                for (int t = lane; t < kThreads / 2; t += 64) {
                    const int j = ((t >> b) << (b + 1)) | (1 << b) | (t & ((1 << b) - 1));
                    nadd(v, val[0][j]);
                }
            } else {
                const double* src = val[b < 0 ? 0 : 1 + b - kLogThreads];
                for (int t = lane; t < kThreads; t += 64) nadd(v, src[t]);
            }
            v = wave_reduce(v);
            if (lane == 0) out[o] = v.s + v.c;
        }
        __syncthreads();   // the next chunk overwrites val
    }
}

// Tr(rho P_t) for an n-qubit density matrix held as vec(rho) (index row + 2^n col):
// P|k> = i^ny (-1)^popcount(k & z) |k xor x>, so Tr(rho P) = sum_k rho[k, k xor x] *
// i^ny (-1)^popcount(k & z).  Only 2^n entries per term are read.  One FP64 Neumaier
// pair per workgroup and term (blockIdx.y; one term after another cost a workgroup reduction
// each: 22 terms of 11 qubits 37 -> 6 us), combined on the host in a fixed order.
template <typename C>
__global__ __launch_bounds__(kThreads) void k_dm_pauli(const C* __restrict__ st, int n, const PauliSumArgs p,
                                                       double* __restrict__ partial)
{
    __shared__ NSum scratch[kThreads / 64];
    const long long N = 1ll << n;
    const long long stride = (long long)gridDim.x * blockDim.x;
    const int t = blockIdx.y;
    const long long x = p.x[t], z = p.z[t];
    const int q = p.ny[t] & 3;
    NSum acc = {0.0, 0.0};
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += stride) {
        const C v = st[k + ((k ^ x) << n)];
        double val = (q == 0) ? v.x : (q == 1) ? -v.y : (q == 2) ? -v.x : v.y;   // Re(i^q v)
        if (__popcll(k & z) & 1) val = -val;
        nadd(acc, val);
    }
    const NSum r = block_reduce(acc, scratch);
    if (threadIdx.x == 0) {
        partial[((long long)blockIdx.x * p.nterms + t) * 2] = r.s;
        partial[((long long)blockIdx.x * p.nterms + t) * 2 + 1] = r.c;
    }
}

// ------------------------------------------------------------------ launchers

hipError_t launch_zsum_batch(int dtype, const ZItem* table, const BatchList* list, double* partial, int grid,
                             hipStream_t s)
{
    if (dtype == 0)
        hipLaunchKernelGGL(k_zsum_batch<float2>, dim3(grid), dim3(kThreads), 0, s, table, list, partial);
    else
        hipLaunchKernelGGL(k_zsum_batch<double2>, dim3(grid), dim3(kThreads), 0, s, table, list, partial);
    return hipGetLastError();
}

// Compute units of the current device (cached per device).
static int device_cus()
{
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) c = 256;
        cus[dev] = c;
    }
    return cus[dev];
}

// Raises the dynamic LDS limit of kernels on the current device (a function's attributes are
// each device's own), once per device and `done`.
template <typename... K>
static hipError_t raise_lds_limit(std::atomic<unsigned long long>& done, int bytes, K... kernels)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    return once_per_device(done, dev, [&] {
        for (const void* k : {(const void*)kernels...}) {
            e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
}

// Workgroups stride over the tiles (the hardware keeps as many resident as registers and
// LDS allow; a finished workgroup's slot is refilled at once).
template <typename C, bool WIDE, bool PF>
hipError_t launch_pass_t(void* st, void* st2, const PassArgs& a, long long ntiles, const DevOp* ops,
                         const void* pool, const int* ipool, const float* apool, hipStream_t s, bool from_zero)
{
    const long long total = st2 ? 2 * ntiles : ntiles;
    // a 64 KiB complex128 tile plus its operand block exceeds the 64 KiB default
    static std::atomic<unsigned long long> raised{0};
    const hipError_t e = raise_lds_limit(raised, 163840, k_pass<C, WIDE, PF>);
    if (e != hipSuccess) return e;
    const size_t lds = (sizeof(C) << a.m) + sizeof(float) * (size_t)(PF ? a.a_len : a.d_len);
    // at most 64 workgroups per CU, each striding over tiles: the operand block is staged
    // once per workgroup rather than once per tile (measured on 2^18-tile passes: 6 %
    // faster for complex64, 10 % for complex128 than one workgroup per tile)
    const long long grid = std::min<long long>(PF ? total / 2 : total, 64ll * device_cus());
    hipLaunchKernelGGL((k_pass<C, WIDE, PF>), dim3((unsigned)grid), dim3(kThreads), lds, s, (C*)st, (C*)st2, a,
                       ntiles, from_zero ? 1 : 0, ops, (const C*)pool, ipool, apool);
    return hipGetLastError();
}

template <typename C, bool WIDE>
static hipError_t launch_batch_pass_t(const BatchItem* table, const BatchList* list, int grid, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL((k_batch_pass<C, WIDE>), dim3(grid), dim3(kThreads), lds, s, table, list);
    return hipGetLastError();
}

// The batched pass kernels may take more than the default 64 KiB of dynamic LDS; the
// limit is raised once, outside any stream capture (the server's step is captured).
hipError_t prepare_batch_pass()
{
    static std::atomic<unsigned long long> raised{0};
    return raise_lds_limit(raised, 98304, k_batch_pass<float2, true>, k_batch_pass<float2, false>,
                           k_batch_pass<double2, true>, k_batch_pass<double2, false>);
}

hipError_t launch_batch_pass(int dtype, const BatchItem* table, const BatchList* list, int grid, int tile_qubits,
                             hipStream_t s, bool wide)
{
    // tile and the pass's diagonal tables of either dtype (matrix operands come through L2)
    const size_t lds = ((dtype == 0 ? sizeof(float2) : sizeof(double2)) << tile_qubits) +
                       sizeof(float) * kServeOperandFloats;
    if (dtype == 0)
        return wide ? launch_batch_pass_t<float2, true>(table, list, grid, lds, s)
                    : launch_batch_pass_t<float2, false>(table, list, grid, lds, s);
    return wide ? launch_batch_pass_t<double2, true>(table, list, grid, lds, s)
                : launch_batch_pass_t<double2, false>(table, list, grid, lds, s);
}

hipError_t launch_pass(int dtype, void* st, const PassArgs& a, long long ntiles, const DevOp* ops,
                       const void* pool, const int* ipool, const float* apool, hipStream_t s, void* st2,
                       bool from_zero, bool wide)
{
    const bool pf = a.staged && !from_zero && loads_ahead(a.m, a.L, (st2 ? 2 : 1) * ntiles, device_cus());
    auto go = [&](auto c, auto w, auto p) {
        return launch_pass_t<decltype(c), decltype(w)::value, decltype(p)::value>(st, st2, a, ntiles, ops, pool, ipool,
                                                                                   apool, s, from_zero);
    };
    auto pick = [&](auto c) {
        if (wide) return pf ? go(c, std::true_type{}, std::true_type{}) : go(c, std::true_type{}, std::false_type{});
        return pf ? go(c, std::false_type{}, std::true_type{}) : go(c, std::false_type{}, std::false_type{});
    };
    return dtype == 0 ? pick(float2{}) : pick(double2{});
}

static hipError_t launch_fill16(void* st, long long bytes, uint4 first, uint4 rest, hipStream_t s)
{
    const long long nchunks = bytes / 16;
    const long long blocks = std::min<long long>((nchunks + kThreads - 1) / kThreads, 8192);
    hipLaunchKernelGGL(k_fill16, dim3((unsigned)blocks), dim3(kThreads), 0, s, (uint4*)st, nchunks, first, rest);
    return hipGetLastError();
}

hipError_t launch_init_zero(int dtype, void* st, long long N, hipStream_t s)
{
    const uint4 zero = make_uint4(0, 0, 0, 0);
    uint4 one = zero;
    if (dtype == 0) {
        const float f = 1.0f;
        memcpy(&one.x, &f, 4);
    } else {
        const double d = 1.0;
        memcpy(&one.x, &d, 8);
    }
    return launch_fill16(st, N * (dtype == 0 ? 8 : 16), one, zero, s);
}

hipError_t launch_zero(int dtype, void* st, long long N, hipStream_t s)
{
    const uint4 zero = make_uint4(0, 0, 0, 0);
    return launch_fill16(st, N * (dtype == 0 ? 8 : 16), zero, zero, s);
}

int norm_grid(long long N)
{
    // eight loads per thread at least: below 2^21 amplitudes more workgroups only add
    // reductions (18-qubit complex128: 1024 workgroups 18.7 us, 128 11.7 us)
    return (int)std::min<long long>(1024, std::max<long long>(1, N / (8 * kThreads)));
}

hipError_t launch_norm(int dtype, const void* st, long long N, double* partial, int grid, hipStream_t s)
{
    const long long nchunks = N * (dtype == 0 ? 8 : 16) / 16;
    if (dtype == 0)
        hipLaunchKernelGGL(k_norm<float>, dim3(grid), dim3(kThreads), 0, s, (const float4*)st, nchunks, partial);
    else
        hipLaunchKernelGGL(k_norm<double>, dim3(grid), dim3(kThreads), 0, s, (const float4*)st, nchunks, partial);
    return hipGetLastError();
}

hipError_t launch_expval(int dtype, const void* sa, const void* sb, const PassArgs& a, const TermArgs& t,
                         long long ntiles, int grid, double* partial, hipStream_t s)
{
    const bool two = sb != nullptr && sb != sa;
    if (a.m < kLogThreads) {   // the whole state is one small tile (grid must be 1)
        if (dtype == 0) {
            auto k = two ? k_expval_small<float2, true> : k_expval_small<float2, false>;
            hipLaunchKernelGGL(k, dim3(1), dim3(kThreads), 0, s, (const float2*)sa, (const float2*)sb, a.m, t, partial);
        } else {
            auto k = two ? k_expval_small<double2, true> : k_expval_small<double2, false>;
            hipLaunchKernelGGL(k, dim3(1), dim3(kThreads), 0, s, (const double2*)sa, (const double2*)sb, a.m, t,
                               partial);
        }
        return hipGetLastError();
    }
    if (a.m > kExpvalMaxTileQubits) return hipErrorInvalidValue;
    if (dtype == 0) {
        auto k = two ? k_expval<float2, true> : k_expval<float2, false>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), expval_lds_bytes(sizeof(float2), a.m), s,
                           (const float2*)sa, (const float2*)sb, a, t, ntiles, partial);
    } else {
        auto k = two ? k_expval<double2, true> : k_expval<double2, false>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), expval_lds_bytes(sizeof(double2), a.m), s,
                           (const double2*)sa, (const double2*)sb, a, t, ntiles, partial);
    }
    return hipGetLastError();
}

hipError_t launch_expval_z(int dtype, const void* sa, const void* sb, const PassArgs& a, const ZTermArgs& t,
                           long long ntiles, int grid, double* partial, hipStream_t s)
{
    const bool two = sb != nullptr && sb != sa;
    if (a.m < kLogThreads || a.m > kExpvalMaxTileQubits) return hipErrorInvalidValue;
    // the threads' transform slots, and at the end eight terms' sums
    const size_t lds = std::max<size_t>(((two ? 2 : 1) * sizeof(double)) << a.m, sizeof(double) * 8 * kThreads);
    if (dtype == 0) {
        auto k = two ? k_expval_z<float2, true> : k_expval_z<float2, false>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), lds, s, (const float2*)sa, (const float2*)sb, a, t, ntiles,
                           partial);
    } else {
        auto k = two ? k_expval_z<double2, true> : k_expval_z<double2, false>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), lds, s, (const double2*)sa, (const double2*)sb, a, t,
                           ntiles, partial);
    }
    return hipGetLastError();
}

hipError_t launch_expval_r(int dtype, const void* sa, const void* sb, const PassArgs& a, const TermArgs& t,
                           const RoundArgs& r, long long ntiles, int grid, double* partial, hipStream_t s)
{
    const bool two = sb != nullptr && sb != sa;
    if (a.m != kRowBits + (two ? kRoundBitsTwo : kRoundBits) || a.L < 1 || r.nrounds > kMaxRounds)
        return hipErrorInvalidValue;
    const size_t lds = (two ? 2 : 1) * ((dtype == 0 ? sizeof(float2) : sizeof(double2)) << a.m) +
                       sizeof(double) * 64 * (size_t)t.nterms;
    if (dtype == 0) {
        auto k = two ? k_expval_r<float2, true> : k_expval_r<float2, false>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), lds, s, (const float2*)sa, (const float2*)sb, a, t, r, ntiles,
                           partial);
    } else {
        auto k = two ? k_expval_r<double2, true> : k_expval_r<double2, false>;
        // 64 KiB tiles beside the terms' sums exceed the default limit
        static std::atomic<unsigned long long> raised{0};
        const hipError_t e = raise_lds_limit(raised, 98304, k_expval_r<double2, true>, k_expval_r<double2, false>);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kThreads), lds, s, (const double2*)sa, (const double2*)sb, a, t, r,
                           ntiles, partial);
    }
    return hipGetLastError();
}

hipError_t launch_pauli_apply(int dtype, const void* in, void* out, long long N, const PauliSumArgs& p,
                              int accumulate, hipStream_t s)
{
    const long long blocks = std::min<long long>((N + kThreads - 1) / kThreads, 16384);
    if (dtype == 0)
        hipLaunchKernelGGL(k_pauli_apply<float2>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const float2*)in,
                           (float2*)out, N, p, accumulate);
    else
        hipLaunchKernelGGL(k_pauli_apply<double2>, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           (const double2*)in, (double2*)out, N, p, accumulate);
    return hipGetLastError();
}

hipError_t launch_probs_full(int dtype, const void* st, long long N, void* out, hipStream_t s)
{
    const long long blocks = std::min<long long>((N + kThreads - 1) / kThreads, 8192);
    if (dtype == 0)
        hipLaunchKernelGGL((k_probs_full<float2, float>), dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           (const float2*)st, N, (float*)out);
    else
        hipLaunchKernelGGL((k_probs_full<double2, double>), dim3((unsigned)blocks), dim3(kThreads), 0, s,
                           (const double2*)st, N, (double*)out);
    return hipGetLastError();
}

static hipError_t launch_sum_chunks(const double* partial, long long M, long long nchunks, double* out, hipStream_t s)
{
    if (nchunks > 32)
        hipLaunchKernelGGL(k_sum_chunks<true>, dim3((unsigned)M), dim3(kThreads), 0, s, partial, M, nchunks, out);
    else
        hipLaunchKernelGGL(k_sum_chunks<false>, dim3((unsigned)((M + kThreads - 1) / kThreads)), dim3(kThreads), 0, s,
                           partial, M, nchunks, out);
    return hipGetLastError();
}

hipError_t launch_marg_blocks(int dtype, const void* st, const MargBlocks& a, double* partial, double* out,
                              hipStream_t s)
{
    const long long blocks = a.G << a.nh;
    if (a.cb > kMargBlockBits || blocks > 0x7fffffffll) return hipErrorInvalidValue;
    if (dtype == 0)
        hipLaunchKernelGGL(k_marg_blocks<float2>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const float2*)st, a,
                           partial, out);
    else
        hipLaunchKernelGGL(k_marg_blocks<double2>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const double2*)st, a,
                           partial, out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.G == 1) return e;
    return launch_sum_chunks(partial, 1ll << a.m, a.G, out, s);
}

hipError_t launch_dm_marg(int dtype, const void* st, const MargArgs& a, double* partial, double* out, hipStream_t s)
{
    const long long M = 1ll << a.m;
    const long long blocks = (M * a.nchunks + kThreads - 1) / kThreads;
    if (dtype == 0)
        hipLaunchKernelGGL(k_dm_marg<float2>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const float2*)st, a, partial);
    else
        hipLaunchKernelGGL(k_dm_marg<double2>, dim3((unsigned)blocks), dim3(kThreads), 0, s, (const double2*)st, a,
                           partial);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_sum_chunks(partial, M, a.nchunks, out, s);
}

hipError_t launch_chunk_totals(int src_dtype, const void* src, int chunk_bits, long long nchunks, double* totals,
                               hipStream_t s)
{
    if (chunk_bits > kSampleChunkBits || nchunks <= 0) return hipErrorInvalidValue;
    const size_t lds = sizeof(double) * scan_at(1 << chunk_bits);
    auto k = src_dtype == 0 ? k_chunk_totals<0> : src_dtype == 1 ? k_chunk_totals<1> : k_chunk_totals<2>;
    hipLaunchKernelGGL(k, dim3((unsigned)nchunks), dim3(kThreads), lds, s, src, chunk_bits, totals);
    return hipGetLastError();
}

hipError_t launch_sample_chunks(int src_dtype, const void* src, int chunk_bits, const SampleChunk* list,
                                long long nlist, const double* residual, long long* outcome, hipStream_t s)
{
    if (chunk_bits > kSampleChunkBits) return hipErrorInvalidValue;
    if (nlist <= 0) return hipSuccess;
    const size_t lds = sizeof(double) * scan_at(1 << chunk_bits);
    auto k = src_dtype == 0 ? k_sample_chunks<0> : src_dtype == 1 ? k_sample_chunks<1> : k_sample_chunks<2>;
    hipLaunchKernelGGL(k, dim3((unsigned)nlist), dim3(kThreads), lds, s, src, chunk_bits, list, residual, outcome);
    return hipGetLastError();
}

hipError_t launch_dm_pauli(int dtype, const void* st, int n, const PauliSumArgs& p, int grid, double* partial,
                           hipStream_t s)
{
    if (dtype == 0)
        hipLaunchKernelGGL(k_dm_pauli<float2>, dim3(grid, p.nterms), dim3(kThreads), 0, s, (const float2*)st, n, p, partial);
    else
        hipLaunchKernelGGL(k_dm_pauli<double2>, dim3(grid, p.nterms), dim3(kThreads), 0, s, (const double2*)st, n, p, partial);
    return hipGetLastError();
}

}  // namespace qsv
