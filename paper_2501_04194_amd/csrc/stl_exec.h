// The generic executor: HIP device code of the STL robustness traces on gfx950
// (MI355X).  Included by the files that compile its kernels (stl_exec_fwd.hip,
// stl_exec_bwd.hip, stl_exec_bwd_ws.hip: apart, since each takes a minute) and
// by stl_kernels.hip for the mask arithmetic the other kernels share.
//
// One work-group owns one trajectory at a time (a persistent grid pulls
// trajectory indices from a counter).  Every node trace of the formula lives
// in an on-chip slot (LDS, or a per-work-group region of the workspace when
// the trajectory is too long for LDS) and the plan's instructions run in
// topological order, each one a work-group-cooperative parallel pass over the
// timesteps.  Only x is read and only the root trace (forward) or dx and the
// mask-bound partial sums (backward) are written to HBM.
//
// Operators (arXiv 2501.04194):
//   windows over [a,b] (Sec. IV-B) are evaluated by van Herk / Gil-Werman
//   block decomposition: blocks of K = b-a+1 positions, block-prefix and
//   block-suffix reductions, and every window is suffix(start) (+) prefix(end)
//   of two adjacent blocks.  The masked (T+K) x T array of the paper is never
//   formed.  Unbounded windows are suffix scans.
//   Smooth windows (Sec. III-C) use the same decomposition on "scaled pairs"
//   (s, r) = s * 2^r, so sums of exp(beta u) never overflow whatever the
//   signal range; beta is folded into base-2 exponents.
//   The smooth time mask (Sec. VI) splits into a constant-weight core (a van
//   Herk window) plus two sigmoid bands summed term by term.
//   Until (Sec. IV-C) runs the running min over the inner index once per
//   output (no 3-D array): hard with compare-selects, smooth with running
//   scaled sums; its adjoint uses checkpointed recomputation.
//   Hard min/max carry the element index so ties resolve to the lowest time
//   index, matching the gradient routing rule.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <algorithm>
#include <type_traits>
#include <stddef.h>
#include "stl_plan.h"

namespace stlmi {

#define DEV static __device__ __forceinline__

constexpr float LOG2E = 1.4426950408889634f;
constexpr int MAX_NT = 512;
constexpr int PAD_NEUTRAL = 0, PAD_LAST = 1, PAD_CONST = 2;

// ------------------------------------------------------------------ types

// scaled pair: value = s * 2^r
struct SP {
    float s;
    int r;
};
constexpr int SP_NEG = -(1 << 29);

DEV SP sp_zero() { return SP{0.f, SP_NEG}; }

DEV SP sp_leaf(float z)  // 2^z
{
    float c = ceilf(fminf(fmaxf(z, -1e9f), 1e9f));
    return SP{__builtin_amdgcn_exp2f(z - c), (int)c};      // z - c in (-1, 0]: no denormal
}

DEV SP sp_add(SP a, SP b)
{
    int m = max(a.r, b.r);
    return SP{ldexpf(a.s, a.r - m) + ldexpf(b.s, b.r - m), m};
}

DEV float sp_log2(SP a) { return (float)a.r + log2f(a.s); }

DEV int clampe(long long e) { return (int)(e < -100000 ? -100000 : (e > 100000 ? 100000 : e)); }

// value of a * 2^z as a float (exact exponent bookkeeping, no intermediate overflow)
DEV float sp_times_exp2(SP a, float z)
{
    float c = ceilf(fminf(fmaxf(z, -1e9f), 1e9f));
    return ldexpf(a.s * exp2f(z - c), clampe((long long)a.r + (long long)c));
}

// scaled pair with a double mantissa: signed sums of many terms (adjoints)
struct SPD {
    double s;
    int r;
};

DEV SPD spd_add(SPD a, SP b)
{
    int m = max(a.r, b.r);
    return SPD{ldexp(a.s, a.r - m) + ldexp((double)b.s, b.r - m), m};
}

// renormalised float scaled pair of a double-mantissa pair
DEV SP spd_to_sp(SPD a)
{
    int e;
    const double mant = frexp(a.s, &e);
    return SP{(float)mant, clampe((long long)a.r + e)};
}

// value with index: hard max with ties to the lowest index
struct VI {
    float v;
    int i;
};

// a's elements come before b's
DEV VI vi_best(VI a, VI b) { return b.v > a.v ? b : a; }

struct OpSP {
    __device__ __forceinline__ SP operator()(SP a, SP b) const { return sp_add(a, b); }
};
struct OpVI {
    __device__ __forceinline__ VI operator()(VI a, VI b) const { return vi_best(a, b); }
};
struct OpD {
    __device__ __forceinline__ double operator()(double a, double b) const { return a + b; }
};

// ------------------------------------------------------------------ scans

struct Shared {
    double scan[2 * MAX_NT / 64];    // totals of the waves (two scans at a time)
    int flag[2 * MAX_NT / 64];
    int ints[8];
    int scan_pos, scan_min;      // flag-scan fix-up: next row index of this work-group, first set flag
};

// the thread index as a value the compiler knows nothing more about
DEV int exec_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    __builtin_assume(t >= 0 && t < MAX_NT);
    return t;
}

struct Env {
    const DevPlan* P;
    const float* x;    // this trajectory, [L, D]
    const float* params;
    int L, Lc, D;
    float* arena;      // slots
    float* scr;        // op scratch
    float* lds;        // LDS beside the slots (smooth Until): export buffers, with slots in the workspace
                       // also the term tile and the checkpoints
    int tile;          // positions of the smooth Until's term tile in lds (0: terms in the scratch)
    Shared* sh;
    int tid;           // threadIdx.x, opaque per instruction: what is derived from it is not kept in registers
                       // across the program (hoisted, it spilled)
    int nt;            // work-group size (blockDim.x is a 16-bit field of the argument segment in host
                       // memory: a vector load of 1 to 2 us wherever the compiler reads it again)
};

// value of another lane by a DPP move (0x110 + k: row_shr:k within rows of 16
// lanes, 0x142: lane 15 of the row below, 0x143: lane 31, 0x138: wave_shr:1;
// 0xB1, 0x4E: lanes 1 and 2 apart in a quad, 0x141, 0x140: mirrored halves of a
// row and rows; lanes without a source read 0), for types of 4 or 8 bytes
template <int CTRL, class T>
DEV T dpp8(T v)
{
    constexpr int N = sizeof(T) / 4;
    static_assert(sizeof(T) == 4 * N && N <= 2, "one or two words");
    int w[N];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = __builtin_amdgcn_update_dpp(0, w[i], CTRL, 0xF, 0xF, true);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// n / K for 0 <= n <= 2^24, inv = 1 / K: the float quotient is below 2^21 for
// K >= 8, so it is off by at most one
DEV int div_k(int n, int K, float inv)
{
    if (K < 8) return n / K;
    int q = (int)((float)n * inv);
    const int r = n - q * K;
    return r < 0 ? q - 1 : (r >= K ? q + 1 : q);
}

// segment heads of the van Herk blocks: p % K == 0 upwards, p % K == K-1 (and
// the last position) downwards; K <= 0: one segment
struct BlockHead {
    int K, n, rem;
    float inv;
    __device__ __forceinline__ BlockHead(int K_, int n_) : K(K_), n(n_), rem(-1), inv(K_ > 0 ? 1.f / (float)K_ : 0.f) {}
};
struct HeadUp : BlockHead {
    using BlockHead::BlockHead;
    __device__ __forceinline__ bool operator()(int p)
    {
        if (K <= 0) return p == 0;
        rem = rem < 0 ? p - div_k(p, K, inv) * K : (rem + 1 == K ? 0 : rem + 1);
        return rem == 0;
    }
};
struct HeadDown : BlockHead {
    using BlockHead::BlockHead;
    __device__ __forceinline__ bool operator()(int p)
    {
        if (K > 0) rem = rem < 0 ? p - div_k(p, K, inv) * K : (rem == 0 ? K - 1 : rem - 1);
        return p == n - 1 || (K > 0 && rem == K - 1);
    }
};

// Segmented inclusive scan of leaf(p), p in [0, n), into x, in two parts with
// a work-group barrier between them (the caller's, so that scans which do not
// depend on each other share it) and one after.  REV scans from n-1 down.
// head(p) starts a segment (asked in scan order by each lane).  Each wave takes
// a contiguous range of the elements and scans it a tile at a time: up to
// SCAN_E consecutive elements per lane, DPP steps over the lanes, a running
// carry between tiles; the totals of the waves before are then joined to what
// precedes a wave's first head.  The scans are bound by latency in short
// trajectories (a Hillis-Steele pass over the work-group cost two barriers and
// two LDS trips per step: a 100-sample hard formula took 17.1 us forward and
// 37.7 us backward) and, with slots in the workspace, by the lines a wave's
// accesses touch (contiguous chunks per thread took 1.4M cycles for a window of
// an 8,192-sample trajectory).  The order of the additions depends on n and
// the work-group size only, not on where the slots lie.
// Every thread must call both parts.
constexpr int SCAN_E = 4;

struct ScanPos {
    int c0, c1;        // the wave's elements
    int free;          // how many of them, in scan order, precede its first segment head
};

template <bool REV, class T, class Op>
DEV T scan_join(T before, T v, Op op)
{
    return REV ? op(v, before) : op(before, v);
}

template <class T>
DEV T readlane8(T v, int l)
{
    int w[2];
    __builtin_memcpy(w, &v, 8);
    w[0] = __builtin_amdgcn_readlane(w[0], l);
    w[1] = __builtin_amdgcn_readlane(w[1], l);
    __builtin_memcpy(&v, w, 8);
    return v;
}

// inclusive scan over the lanes of a wave within the segments that begin at
// the lanes of hm; d: lanes since the last head at or before this one
template <bool REV, class T, class Op>
DEV T scan_wave(T acc, unsigned long long hm, int lane, Op op)
{
    const unsigned long long upto = hm & (~0ull >> (63 - lane));
    const int d = upto ? lane - (63 - __builtin_clzll(upto)) : lane;
#define STLMI_SCAN_STEP(CTRL, COND)                    \
    {                                                  \
        const T b = dpp8<CTRL>(acc);                   \
        if (COND) acc = scan_join<REV>(b, acc, op);    \
    }
    const int dr = min(lane & 15, d);
    STLMI_SCAN_STEP(0x111, dr >= 1)
    STLMI_SCAN_STEP(0x112, dr >= 2)
    STLMI_SCAN_STEP(0x114, dr >= 4)
    STLMI_SCAN_STEP(0x118, dr >= 8)
    STLMI_SCAN_STEP(0x142, (lane & 16) && d >= (lane & 15) + 1)
    STLMI_SCAN_STEP(0x143, lane >= 32 && d >= lane - 31)
#undef STLMI_SCAN_STEP
    return acc;
}

template <bool REV, int E, class T, class Op, class Leaf, class Head>
DEV void scan_local_e(T* x, int n, T ident, Op op, Leaf leaf, Head head, const Env& e, int which, ScanPos& s)
{
    // (E = 1: one tile per wave; the work-group size is a power of two)
    const int nw = e.nt >> 6, w = e.tid >> 6, lane = e.tid & 63;
    const int seg = E == 1 ? 64 : ((n + E * e.nt - 1) >> __builtin_ctz(E * e.nt)) * (64 * E);
    const int cw = REV ? nw - 1 - w : w;
    s.c0 = min(n, cw * seg);
    s.c1 = min(n, s.c0 + seg);
    const int m = s.c1 - s.c0;
    auto pos = [&](int i) { return REV ? s.c1 - 1 - i : s.c0 + i; };
    s.free = m;
    T run = ident, v[E];
    bool seen = false;
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = lane * E + j < m ? leaf(pos(lane * E + j)) : ident;
#pragma unroll 1
    for (int i0 = 0; i0 < (E == 1 ? 1 : m); i0 += 64 * E) {
        const int i = i0 + lane * E;
        T vn[E];                                   // the next tile's leaves, read ahead
        if (E > 1) {
#pragma unroll
            for (int j = 0; j < E; ++j) vn[j] = i + 64 * E + j < m ? leaf(pos(i + 64 * E + j)) : ident;
        }
        int first = E;                             // this lane's first head
        Head h = head;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const bool hj = i + j < m && h(pos(i + j));
            if (j > 0 && !hj) v[j] = scan_join<REV>(v[j - 1], v[j], op);
            if (hj) first = min(first, j);
        }
        const unsigned long long hm = __ballot(first < E);
        const T acc = scan_wave<REV>(v[E - 1], hm, lane, op);
        T carry = dpp8<0x138>(acc);
        const bool open = (hm & ((1ull << lane) - 1)) == 0;      // no head in the lanes before
        if (open && i0 > 0) carry = lane == 0 ? run : scan_join<REV>(run, carry, op);
        const int nf = i0 + lane > 0 ? first : 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            if (j < nf) v[j] = scan_join<REV>(carry, v[j], op);
            if (i + j < m) x[pos(i + j)] = v[j];
        }
        if (!seen && hm) {
            const int fl = __builtin_ctzll(hm);
            s.free = i0 + fl * E + __builtin_amdgcn_readlane(first, fl);
            seen = true;
        }
        run = readlane8(v[E - 1], 63);
        if (E > 1) {
#pragma unroll
            for (int j = 0; j < E; ++j) v[j] = vn[j];
        }
    }
    if (lane == 0) {
        reinterpret_cast<T*>(e.sh->scan)[which * 8 + w] = run;
        e.sh->flag[which * 8 + w] = seen;
    }
}

template <bool REV, class T, class Op, class Leaf, class Head>
DEV void scan_local(T* x, int n, T ident, Op op, Leaf leaf, Head head, const Env& e, int which, ScanPos& s)
{
    if (n <= e.nt) scan_local_e<REV, 1>(x, n, ident, op, leaf, head, e, which, s);
    else scan_local_e<REV, SCAN_E>(x, n, ident, op, leaf, head, e, which, s);
}

template <bool REV, class T, class Op>
DEV void scan_carry(T* x, Op op, const Env& e, int which, const ScanPos& s)
{
    const int w = e.tid >> 6, lane = e.tid & 63;
    if (w == 0) return;                            // nothing comes before
    // lane q % 8 scans the totals of waves 0 .. q (wave w needs those of 0 .. w-1)
    const int q = lane & 7;
    T c = reinterpret_cast<const T*>(e.sh->scan)[which * 8 + q];
    const unsigned hm = (unsigned)__ballot(e.sh->flag[which * 8 + q] != 0) & 0xffu & ((2u << q) - 1u);
    const int d = hm ? q - (31 - __builtin_clz(hm)) : q;
#define STLMI_CARRY_STEP(CTRL, K)                           \
    {                                                       \
        const T b = dpp8<CTRL>(c);                          \
        if (q >= K && d >= K) c = scan_join<REV>(b, c, op); \
    }
    STLMI_CARRY_STEP(0x111, 1)
    STLMI_CARRY_STEP(0x112, 2)
    STLMI_CARRY_STEP(0x114, 4)
#undef STLMI_CARRY_STEP
    c = readlane8(c, __builtin_amdgcn_readfirstlane(w - 1));
    for (int i = lane; i < s.free; i += 64) {
        const int p = REV ? s.c1 - 1 - i : s.c0 + i;
        x[p] = scan_join<REV>(c, x[p], op);
    }
}

// block prefixes and suffixes of the same leaves (K <= 0: suffixes of the
// whole range only)
template <class T, class Op, class Leaf>
DEV void scan_blocks(T* pre, T* suf, int n, int K, T ident, Op op, Leaf leaf, const Env& e)
{
    ScanPos sp, ss;
    scan_local<true>(suf, n, ident, op, leaf, HeadDown(K, n), e, 0, ss);
    if (K > 0) scan_local<false>(pre, n, ident, op, leaf, HeadUp(K, n), e, 1, sp);
    __syncthreads();
    scan_carry<true>(suf, op, e, 0, ss);
    if (K > 0) scan_carry<false>(pre, op, e, 1, sp);
    __syncthreads();
}

// one scan of the whole work-group
template <bool REV, class T, class Op, class Leaf, class Head>
DEV void scan_one(T* x, int n, T ident, Op op, Leaf leaf, Head head, const Env& e)
{
    ScanPos s;
    scan_local<REV>(x, n, ident, op, leaf, head, e, 0, s);
    __syncthreads();
    scan_carry<REV>(x, op, e, 0, s);
    __syncthreads();
}

// does the window of K positions at t (ending at e2, clipped to n-1) lie in one block?
DEV bool one_block(int t, int e2, int K, float inv, bool& at_start)
{
    const int q = div_k(t, K, inv) * K;
    at_start = q == t;
    return e2 < q + K;
}

// deterministic work-group sum of one value per thread (a fixed shuffle tree,
// then the waves in order)
template <class T>
DEV T wg_sum(T v, const Env& e)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
    T* tot = reinterpret_cast<T*>(e.sh->scan);
    if ((e.tid & 63) == 0) tot[e.tid >> 6] = v;
    __syncthreads();
    T r = tot[0];
    for (int w = 1; w < e.nt >> 6; ++w) r += tot[w];
    __syncthreads();
    return r;
}

// ------------------------------------------------------------------ context

// scratch layout (floats): what an operator needs, in units of Lc (at most
// 16; the plan compiler finds each plan's need)
DEV float* S(const Env& e, int unit) { return e.scr + (size_t)unit * e.Lc; }

DEV float* slot(const Env& e, int s) { return e.arena + (size_t)s * e.Lc; }

DEV float pbeta(const Env& e, const Instr& I) { return I.beta >= 0 ? e.params[I.beta] : 1.f; }

// ------------------------------------------------------------------ pointwise ops

// a plan entry read as 32-bit words (scalar loads; single bytes of the
// argument segment would be vector loads)
template <class T>
DEV T load_words(const T* p)
{
    int w[sizeof(T) / 4];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = ((const int*)p)[i];
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// The predicates are evaluated for the whole formula at once: a row of x is
// read once (per predicate it cost 0.5 to 1 us of latency in a short
// trajectory) and feeds every predicate.
constexpr int PRED_TB = 4;    // timesteps per thread and pass of the pointwise loops where a thread has
                              // several: their reads are in flight together (the compiler cannot move
                              // them past the stores)

template <int D>
DEV void load_row(const float* p, bool vec, float (&r)[D])
{
    if (vec && D == 4) {
        const float4 v = *(const float4*)p;
        r[0] = v.x; r[1 % D] = v.y; r[2 % D] = v.z; r[3 % D] = v.w;
    } else if (vec && D == 2) {
        const float2 v = *(const float2*)p;
        r[0] = v.x; r[1 % D] = v.y;
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d) r[d] = p[d];
    }
}

template <int D>
DEV void store_row(float* p, bool vec, const float (&r)[D])
{
    if (vec && D == 4) *(float4*)p = float4{r[0], r[1 % D], r[2 % D], r[3 % D]};
    else if (vec && D == 2) *(float2*)p = float2{r[0], r[1 % D]};
    else {
#pragma unroll
        for (int d = 0; d < D; ++d) p[d] = r[d];
    }
}

// rows of 2 or 4 floats are moved whole where they are aligned
template <int D>
DEV bool vec_rows(const float* p) { return (D == 2 || D == 4) && ((uintptr_t)p & (4 * D - 1)) == 0; }

// A x - p of a norm predicate (rows i < m, others 0) and its squared length
template <class Row>
DEV float norm_rows(const float* cf, int m, int D, Row x, float (&z)[4])
{
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        z[i] = 0.f;
        if (i < m) {
            z[i] = -cf[3 + i];
            for (int d = 0; d < D; ++d) z[i] = fmaf(cf[7 + i * D + d], x[d], z[i]);
            q = fmaf(z[i], z[i], q);
        }
    }
    return q;
}

template <class Row>
DEV float pred_value(int kind, const float* cf, int D, Row x)
{
    if (kind == K_LIN) {
        float s = 0.f;
        for (int d = 0; d < D; ++d) s = fmaf(cf[1 + d], x[d], s);
        return s - cf[0];
    }
    float z[4];
    return cf[2] * (sqrtf(norm_rows(cf, (int)cf[0], D, x, z)) - cf[1]);
}

template <int D, int TB>
DEV void preds_fwd(const Env& e, bool bwdmap)
{
    const DevPlan& P = *e.P;
    const int nt = e.nt;
    const bool vec = vec_rows<D>(e.x);
    for (int t0 = e.tid; t0 < e.L; t0 += TB * nt) {
        float x[TB][D];
#pragma unroll
        for (int j = 0; j < TB; ++j)
            if (t0 + j * nt < e.L) load_row<D>(e.x + (size_t)(t0 + j * nt) * D, vec, x[j]);
#pragma unroll 2
        for (int p = 0; p < P.n_pred; ++p) {
            const PredRef I = load_words(&P.pred[p]);
            float* out = slot(e, bwdmap ? I.b_out : I.f_out);
#pragma unroll
            for (int j = 0; j < TB; ++j)
                if (t0 + j * nt < e.L) out[t0 + j * nt] = pred_value(I.kind, P.coef + I.coef, D, x[j]);
        }
    }
}

DEV void op_preds(const Env& e, bool bwdmap)
{
    const bool one = e.L <= e.nt;
    switch (e.D) {
    case 1: one ? preds_fwd<1, 1>(e, bwdmap) : preds_fwd<1, PRED_TB>(e, bwdmap); return;
    case 2: one ? preds_fwd<2, 1>(e, bwdmap) : preds_fwd<2, PRED_TB>(e, bwdmap); return;
    case 3: one ? preds_fwd<3, 1>(e, bwdmap) : preds_fwd<3, PRED_TB>(e, bwdmap); return;
    case 4: one ? preds_fwd<4, 1>(e, bwdmap) : preds_fwd<4, PRED_TB>(e, bwdmap); return;
    }
    const DevPlan& P = *e.P;
    for (int p = 0; p < P.n_pred; ++p) {
        const PredRef I = load_words(&P.pred[p]);
        float* out = slot(e, bwdmap ? I.b_out : I.f_out);
        for (int t = e.tid; t < e.L; t += e.nt)
            out[t] = pred_value(I.kind, P.coef + I.coef, e.D, e.x + (size_t)t * e.D);
    }
}

// one predicate where the formula names it (plans whose predicates are not
// evaluated together: their traces would take more slots than they may)
template <int D>
DEV void pred_one(const Env& e, const Instr& I, float* out)
{
    const float* cf = e.P->coef + I.coef;
    const bool vec = vec_rows<D>(e.x);
    for (int t0 = e.tid; t0 < e.L; t0 += PRED_TB * e.nt) {
        float x[PRED_TB][D];
#pragma unroll
        for (int j = 0; j < PRED_TB; ++j)
            if (t0 + j * e.nt < e.L) load_row<D>(e.x + (size_t)(t0 + j * e.nt) * D, vec, x[j]);
#pragma unroll
        for (int j = 0; j < PRED_TB; ++j)
            if (t0 + j * e.nt < e.L) out[t0 + j * e.nt] = pred_value(I.kind, cf, D, x[j]);
    }
}

DEV void op_pred(const Env& e, const Instr& I, float* out)
{
    switch (e.D) {
    case 1: pred_one<1>(e, I, out); return;
    case 2: pred_one<2>(e, I, out); return;
    case 3: pred_one<3>(e, I, out); return;
    case 4: pred_one<4>(e, I, out); return;
    }
    const float* cf = e.P->coef + I.coef;
    for (int t = e.tid; t < e.L; t += e.nt) out[t] = pred_value(I.kind, cf, e.D, e.x + (size_t)t * e.D);
}

// d/dx of the predicates: dx[t, d] = sum_p dmu_p/dx_d * g_p[t]; one predicate's part
template <class Row, class Acc>
DEV void pred_dx(int kind, const float* cf, int D, float g, Row x, Acc& acc)
{
    if (kind == K_LIN) {
        for (int d = 0; d < D; ++d) acc[d] = fmaf(cf[1 + d], g, acc[d]);
        return;
    }
    const int m = (int)cf[0];
    float z[4];
    const float q = norm_rows(cf, m, D, x, z);
    if (q > 0.f) {
        const float k = cf[2] * g / sqrtf(q);
        for (int d = 0; d < D; ++d) {
            float v = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i < m) v = fmaf(cf[7 + i * D + d], z[i], v);
            acc[d] = fmaf(k, v, acc[d]);
        }
    }
}

template <int D, int TB>
DEV void preds_dx(const Env& e, float* dx)
{
    const DevPlan& P = *e.P;
    const bool vx = vec_rows<D>(e.x), vd = vec_rows<D>(dx);
    for (int t0 = e.tid; t0 < e.L; t0 += TB * e.nt) {
        float x[TB][D], acc[TB][D];
#pragma unroll
        for (int j = 0; j < TB; ++j) {
#pragma unroll
            for (int d = 0; d < D; ++d) acc[j][d] = 0.f;
            if (t0 + j * e.nt < e.L) load_row<D>(e.x + (size_t)(t0 + j * e.nt) * D, vx, x[j]);
        }
        for (int p = 0; p < P.n_pred; ++p) {
            const PredRef I = load_words(&P.pred[p]);
            const float* gs = slot(e, I.g_out);
            float g[TB];
#pragma unroll
            for (int j = 0; j < TB; ++j) g[j] = t0 + j * e.nt < e.L ? gs[t0 + j * e.nt] : 0.f;
#pragma unroll
            for (int j = 0; j < TB; ++j)
                if (t0 + j * e.nt < e.L) pred_dx(I.kind, P.coef + I.coef, D, g[j], x[j], acc[j]);
        }
#pragma unroll
        for (int j = 0; j < TB; ++j)
            if (t0 + j * e.nt < e.L) store_row<D>(dx + (size_t)(t0 + j * e.nt) * D, vd, acc[j]);
    }
}

DEV void op_dx(const Env& e, float* dx)
{
    const bool one = e.L <= e.nt;
    switch (e.D) {
    case 1: one ? preds_dx<1, 1>(e, dx) : preds_dx<1, PRED_TB>(e, dx); return;
    case 2: one ? preds_dx<2, 1>(e, dx) : preds_dx<2, PRED_TB>(e, dx); return;
    case 3: one ? preds_dx<3, 1>(e, dx) : preds_dx<3, PRED_TB>(e, dx); return;
    case 4: one ? preds_dx<4, 1>(e, dx) : preds_dx<4, PRED_TB>(e, dx); return;
    }
    for (int t = e.tid; t < e.L; t += e.nt) {
        float acc[MAX_D];
#pragma unroll
        for (int d = 0; d < MAX_D; ++d) acc[d] = 0.f;
        for (int p = 0; p < e.P->n_pred; ++p) {
            const PredRef I = load_words(&e.P->pred[p]);
            pred_dx(I.kind, e.P->coef + I.coef, e.D, slot(e, I.g_out)[t], e.x + (size_t)t * e.D, acc);
        }
        for (int d = 0; d < e.D; ++d) dx[(size_t)t * e.D + d] = acc[d];
    }
}

template <int N, int TB>
DEV void nary_fwd(const Env& e, const Instr& I, const int8_t* ch, float* out)
{
    const float sg = (I.flags & F_MIN) ? -1.f : 1.f;
    const bool smooth = I.flags & F_SMOOTH, soft = I.flags & F_SOFT;
    const float bl = smooth ? pbeta(e, I) * LOG2E : 1.f;
    const float* c[N];
#pragma unroll
    for (int k = 0; k < N; ++k) c[k] = slot(e, ch[k]);
    for (int tb = e.tid; tb < e.L; tb += TB * e.nt) {
        float vv[TB][N];
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int k = 0; k < N; ++k) vv[j][k] = tb + j * e.nt < e.L ? sg * c[k][tb + j * e.nt] : 0.f;
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            const int t = tb + j * e.nt;
            if (t >= e.L) break;
            const float(&v)[N] = vv[j];
            float m = v[0];
            if (!smooth) {
#pragma unroll
                for (int k = 1; k < N; ++k)
                    if (v[k] > m) m = v[k];
                out[t] = sg * m;
                continue;
            }
#pragma unroll
            for (int k = 1; k < N; ++k) m = fmaxf(m, v[k]);
            float s0 = 0.f, s1 = 0.f;
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const float q = exp2f((v[k] - m) * bl);
                s0 += q;
                s1 = fmaf(q, v[k], s1);
            }
            // softmax-weighted mean of the oriented values, or logsumexp (Sec. III-C)
            out[t] = sg * (soft ? s1 / s0 : m + log2f(s0) / bl);
        }
    }
}

DEV void op_nary_fwd(const Env& e, const Instr& I, const int8_t* ch, float* out)
{
    const bool one = e.L <= e.nt;
    switch (I.nch) {
    case 1: one ? nary_fwd<1, 1>(e, I, ch, out) : nary_fwd<1, PRED_TB>(e, I, ch, out); break;
    case 2: one ? nary_fwd<2, 1>(e, I, ch, out) : nary_fwd<2, PRED_TB>(e, I, ch, out); break;
    case 3: one ? nary_fwd<3, 1>(e, I, ch, out) : nary_fwd<3, PRED_TB>(e, I, ch, out); break;
    default: one ? nary_fwd<4, 1>(e, I, ch, out) : nary_fwd<4, PRED_TB>(e, I, ch, out); break;
    }
}

template <int N, int TB>
DEV void nary_bwd(const Env& e, const Instr& I)
{
    const float sg = (I.flags & F_MIN) ? -1.f : 1.f;
    const bool smooth = I.flags & F_SMOOTH, soft = I.flags & F_SOFT;
    const float bl = smooth ? pbeta(e, I) * LOG2E : 1.f;
    const float* g = slot(e, I.g_out);
    const float* out = slot(e, I.b_out);
    const float* c[N];
    float* gc[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        c[k] = slot(e, I.b_ch[k]);
        gc[k] = slot(e, I.g_ch[k]);
    }
    for (int tb = e.tid; tb < e.L; tb += TB * e.nt) {
        float vv[TB][N], gg[TB], oo[TB];
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            const int t = tb + j * e.nt;
            const bool in = t < e.L;
            gg[j] = in ? g[t] : 0.f;
            oo[j] = in && smooth ? sg * out[t] : 0.f;
#pragma unroll
            for (int k = 0; k < N; ++k) vv[j][k] = in ? sg * c[k][t] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            const int t = tb + j * e.nt;
            if (t >= e.L) break;
            const float(&v)[N] = vv[j];
            const float gt = gg[j], o = oo[j];
            if (!smooth) {
                int kb = 0;
                float best = v[0];
#pragma unroll
                for (int k = 1; k < N; ++k)
                    if (v[k] > best) { best = v[k]; kb = k; }
#pragma unroll
                for (int k = 0; k < N; ++k) gc[k][t] = (k == kb) ? gt : 0.f;
            } else if (soft) {
                // d r / d v_k = p_k (1 + beta (v_k - r)), r = sg out
                const float beta = bl / LOG2E;
                float m = v[0], s0 = 0.f;
#pragma unroll
                for (int k = 1; k < N; ++k) m = fmaxf(m, v[k]);
#pragma unroll
                for (int k = 0; k < N; ++k) s0 += exp2f((v[k] - m) * bl);
#pragma unroll
                for (int k = 0; k < N; ++k)
                    gc[k][t] = gt * (exp2f((v[k] - m) * bl) / s0) * (1.f + beta * (v[k] - o));
            } else {
#pragma unroll
                for (int k = 0; k < N; ++k) gc[k][t] = gt * exp2f((v[k] - o) * bl);
            }
        }
    }
}

DEV void op_nary_bwd(const Env& e, const Instr& I)
{
    const bool one = e.L <= e.nt;
    switch (I.nch) {
    case 1: one ? nary_bwd<1, 1>(e, I) : nary_bwd<1, PRED_TB>(e, I); break;
    case 2: one ? nary_bwd<2, 1>(e, I) : nary_bwd<2, PRED_TB>(e, I); break;
    case 3: one ? nary_bwd<3, 1>(e, I) : nary_bwd<3, PRED_TB>(e, I); break;
    default: one ? nary_bwd<4, 1>(e, I) : nary_bwd<4, PRED_TB>(e, I); break;
    }
}

// ------------------------------------------------------------------ hard windows

// Hard max (sg=+1) / min (sg=-1) of u over [t+klo, t+khi] (khi<0: to the end)
// with the pad policy.  Writes out[t]; if jstar != NULL also the index of the
// selected element (L when none / a constant pad).
DEV void win_hard(const Env& e, const float* u, float* out, int* jstar, float sg, int klo, int khi,
                  int pad, float padv, VI* Pre, VI* Suf)
{
    const int L = e.L;
    const bool unb = khi < 0;
    const int n = L - klo;
    const int K = unb ? n : khi - klo + 1;
    const float inv = 1.f / (float)K;
    if (n > 0)
        scan_blocks(Pre, Suf, n, unb ? 0 : K, VI{-INFINITY, 0x7fffffff}, OpVI(),
                    [&](int i) { return VI{sg * u[klo + i], klo + i}; }, e);
    const float rho_pad = e.P->rho_pad;
    for (int t = e.tid; t < L; t += e.nt) {
        VI r{-INFINITY, L};
        bool any = false;
        if (t < n) {
            const int e2 = min(t + K - 1, n - 1);
            bool st;
            r = (unb || one_block(t, e2, K, inv, st)) ? Suf[t] : vi_best(Suf[t], Pre[e2]);
            any = true;
        }
        if (!unb && pad != PAD_NEUTRAL && t + khi > L - 1) {
            if (pad == PAD_LAST) {
                if (!any) r = VI{sg * u[L - 1], L - 1};
            } else {
                VI pv{sg * padv, L};
                r = any ? vi_best(r, pv) : pv;
            }
            any = true;
        }
        out[t] = any ? sg * r.v : -sg * rho_pad;
        if (jstar) jstar[t] = any ? r.i : L;
    }
    __syncthreads();
}

// adjoint of a hard window: gu[j] = sum of g[t] over the t whose selected
// index is j.  The selected index is non-decreasing in t, so each j owns a
// contiguous run of t: an fp64 segmented sum of g leaves the run's total (exact
// to fp32 rounding, deterministic) at the run's last t.
DEV void win_hard_adj(const Env& e, const float* g, float* gu, const int* jstar, double* P)
{
    const int L = e.L;
    for (int j = e.tid; j < L; j += e.nt) gu[j] = 0.f;
    scan_one<false>(P, L, 0.0, OpD(), [&](int t) { return (double)g[t]; },
                    [&](int t) { return t == 0 || jstar[t] != jstar[t - 1]; }, e);
    for (int t = e.tid; t < L; t += e.nt) {
        const int j = jstar[t];
        if (j < L && (t == L - 1 || jstar[t + 1] != j)) gu[j] = (float)P[t];
    }
    __syncthreads();
}

// ------------------------------------------------------------------ smooth windows

// Smooth max (sg=+1) / min of u over the integer window [t+klo, t+khi]
// (khi<0: to the end), scaled by a constant weight 2^lw, as scaled pairs:
// acc[t] = sum_j w 2^{z_j}, z = sg*beta*log2(e)*u.  Pads add their copies.
// any[t] (byte flag) tells whether the window is non-empty.
DEV void win_smooth_sum(const Env& e, const float* u, SP* acc, float sgz, int klo, int khi, int pad,
                        float padv, SP* Pre, SP* Suf)
{
    const int L = e.L;
    const bool unb = khi < 0;
    const int n = L - klo;
    const int K = unb ? n : khi - klo + 1;
    const float inv = 1.f / (float)K;
    if (n > 0)
        scan_blocks(Pre, Suf, n, unb ? 0 : K, sp_zero(), OpSP(), [&](int i) { return sp_leaf(sgz * u[klo + i]); },
                    e);
    for (int t = e.tid; t < L; t += e.nt) {
        SP a = sp_zero();
        if (t < n) {
            const int e2 = min(t + K - 1, n - 1);
            bool st;
            a = (unb || one_block(t, e2, K, inv, st)) ? Suf[t] : sp_add(Suf[t], Pre[e2]);
        }
        if (!unb && pad != PAD_NEUTRAL && t + khi > L - 1) {
            int np = min(K, t + khi - (L - 1));
            SP pv = sp_leaf(pad == PAD_LAST ? sgz * u[L - 1] : sgz * padv);
            pv.s *= (float)np;
            a = sp_add(a, pv);
        }
        acc[t] = a;
    }
    __syncthreads();
}

// Window sums of u_j 2^{sgz u_j} (signed scaled pairs) over [t+klo, t+khi]
// (khi < 0: to the end), NEUTRAL pad: the numerator of the softmax-weighted
// mean whose denominator win_smooth_sum gives.
DEV void win_smooth_sum_w(const Env& e, const float* u, SP* acc, float sgz, int klo, int khi, SP* Pre, SP* Suf)
{
    const int L = e.L;
    const bool unb = khi < 0;
    const int n = L - klo;
    const int K = unb ? n : khi - klo + 1;
    const float inv = 1.f / (float)K;
    if (n > 0)
        scan_blocks(Pre, Suf, n, unb ? 0 : K, sp_zero(), OpSP(),
                    [&](int i) {
                        SP v = sp_leaf(sgz * u[klo + i]);
                        v.s *= u[klo + i];
                        return v;
                    },
                    e);
    for (int t = e.tid; t < L; t += e.nt) {
        SP a = sp_zero();
        if (t < n) {
            const int e2 = min(t + K - 1, n - 1);
            bool st;
            a = (unb || one_block(t, e2, K, inv, st)) ? Suf[t] : sp_add(Suf[t], Pre[e2]);
        }
        acc[t] = a;
    }
    __syncthreads();
}

// ratio of two scaled pairs as a float (den > 0)
DEV float sp_ratio(SP num, SP den)
{
    return ldexpf(num.s / den.s, clampe((long long)num.r - den.r));
}

// Transposed window sum for adjoints: for each position j, res[j] = sum over
// t in [j-khi, j-klo] (clipped to [0, n_valid)) of h(t).
template <class Leaf>
DEV void win_smooth_adj_sum(const Env& e, Leaf h, SP* hSuf, SP* hPre, SP* res, int klo, int khi, int n_valid)
{
    const int L = e.L;
    const bool unb = khi < 0;
    const int K = unb ? L : khi - klo + 1;
    const float inv = 1.f / (float)K;
    if (unb) scan_one<false>(hPre, L, sp_zero(), OpSP(), h, HeadUp(0, L), e);
    else scan_blocks(hPre, hSuf, L, K, sp_zero(), OpSP(), h, e);
    for (int j = e.tid; j < L; j += e.nt) {
        SP a = sp_zero();
        const int en = min(j - klo, n_valid - 1);
        const int st = unb ? 0 : max(0, j - khi);
        if (st <= en) {
            bool at_start;
            if (unb) a = hPre[en];
            else if (one_block(st, en, K, inv, at_start)) a = at_start ? hPre[en] : hSuf[st];
            else a = sp_add(hSuf[st], hPre[en]);
        }
        res[j] = a;
    }
    __syncthreads();
}

// ------------------------------------------------------------------ masks

struct MaskInfo {
    int klo, khi;      // support {w > 0}; khi = L-1 .. for unbounded
    int clo, chi;      // constant core (clo > chi: none)
    float wc;          // core weight
    bool any;
};

// Smooth-mask weight of offset k (Sec. VI):
//   w_k = max(sig(c(k-a)) - sig(c(k-b)) - eps, 0)
// using sig(x) - sig(y) = sig(x) sig(-y) (1 - exp(-(x-y))), which has no
// cancellation, and its derivatives d w/da = -c sig'(c(k-a)),
// d w/db = c sig'(c(k-b)) (zero where the clamp is active).
struct MaskP {
    float a, b, c, eps, band;
    bool unb;
};

DEV MaskP mask_params(const float* pm, bool unb)
{
    MaskP m;
    m.a = pm[0];
    m.b = pm[1];
    m.c = pm[2];
    m.eps = pm[3];
    m.unb = unb;
    m.band = unb ? 1.f : 1.f - expf(-m.c * (m.b - m.a));
    return m;
}

DEV float mask_wk(const MaskP& m, int k, float* dwa = nullptr, float* dwb = nullptr)
{
    const float x1 = m.c * ((float)k - m.a);
    const float s1 = 1.f / (1.f + expf(-x1));
    float wk;
    if (m.unb) {
        wk = s1 - m.eps;
    } else {
        const float y1 = m.c * ((float)k - m.b);
        const float sny = 1.f / (1.f + expf(y1));
        wk = s1 * sny * m.band - m.eps;
    }
    wk = wk > 0.f ? wk : 0.f;
    if (dwa) {
        // sig'(x) = e^{-|x|} / (1 + e^{-|x|})^2: accurate in both tails (the
        // form s (1 - s) loses all digits where s rounds to 1)
        const float t1 = expf(-fabsf(x1));
        *dwa = wk > 0.f ? -m.c * (t1 / ((1.f + t1) * (1.f + t1))) : 0.f;
        if (wk > 0.f && !m.unb) {
            const float t2 = expf(-fabsf(m.c * ((float)k - m.b)));
            *dwb = m.c * (t2 / ((1.f + t2) * (1.f + t2)));
        } else {
            *dwb = 0.f;
        }
    }
    return wk;
}

// Offsets that can hold the support {w > 0}: it lies inside [a - 89/c,
// b + 89/c], beyond which a sigmoid's exponential overflows in fp32 (e^x is
// inf for x > 88.73), the factor is exactly 0 and w_k = max(-eps, 0).
DEV void mask_window(const MaskP& mp, int L, int& k0, int& k1)
{
    k0 = 0;
    k1 = L - 1;
    const double a = mp.a, b = mp.b, c = mp.c;
    if (c > 0.0 && isfinite(a) && isfinite(c) && (mp.unb || isfinite(b))) {
        k0 = (int)fmax(0.0, fmin((double)L, floor(a - 89.0 / c) - 2.0));
        if (!mp.unb) k1 = (int)fmin((double)(L - 1), fmax(-1.0, ceil(b + 89.0 / c) + 2.0));
    }
}

// the core where both sigmoid derivatives are below 2^-24 (|c(k-a)|,
// |c(k-b)| > 17), over which w is constant to fp32 rounding, given the
// support [klo, khi]
DEV MaskInfo mask_core(const MaskP& mp, int klo, int khi, int mid_known = INT_MIN, float w_known = 0.f)
{
    MaskInfo mi;
    mi.klo = klo;
    mi.khi = khi;
    mi.any = mi.klo <= mi.khi;
    const float a = mp.a, b = mp.b, c = mp.c;
    if (c > 0.f && mi.any) {
        mi.clo = max(mi.klo, (int)fminf(ceilf(a + 17.f / c), 2e9f));
        mi.chi = mp.unb ? mi.khi : min(mi.khi, (int)fmaxf(floorf(b - 17.f / c), -2e9f));
    } else {
        mi.clo = 1;
        mi.chi = 0;
    }
    // (w at the midpoint, unless the caller has it already)
    if (mi.clo > mi.chi) { mi.clo = 1; mi.chi = 0; mi.wc = 0.f; }
    else mi.wc = (mi.clo + mi.chi) / 2 == mid_known ? w_known : mask_wk(mp, (mi.clo + mi.chi) / 2);
    return mi;
}

// min / max over the wave (an atomic with a value per lane becomes a scalar
// loop over the lanes, which the work-group's waves share: reduce first)
DEV int wave_imin(int v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = min(v, __shfl_xor(v, o));
    return v;
}
DEV int wave_imax(int v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = max(v, __shfl_xor(v, o));
    return v;
}

// Weights for k in [0, L) (stored when w != NULL), the support {w > 0} and
// the core.  Without stored weights only the support's window is searched.
template <class SH>
DEV MaskInfo mask_info(const float* params, const Instr& I, int L, SH& sh, int nt, int tid, float* w, float* dwa, float* dwb)
{
    const MaskP mp = mask_params(params + I.mask, I.flags & F_MASK_UNB);
    int* si = sh.ints;
    if (tid == 0) { si[0] = L; si[1] = -1; }
    __syncthreads();
    int lo = L, hi = -1;
    int k0 = 0, k1 = L - 1;
    if (!w && !dwa) mask_window(mp, L, k0, k1);
    for (int k = k0 + tid; k <= k1; k += nt) {
        float da, db;
        const float wk = mask_wk(mp, k, dwa ? &da : nullptr, &db);
        if (w) w[k] = wk;
        if (dwa) { dwa[k] = da; dwb[k] = db; }
        if (wk > 0.f) { lo = min(lo, k); hi = max(hi, k); }
    }
    lo = wave_imin(lo);
    hi = wave_imax(hi);
    if ((tid & 63) == 0) {
        atomicMin(&si[0], lo);
        atomicMax(&si[1], hi);
    }
    __syncthreads();
    const MaskInfo mi = mask_core(mp, si[0], si[1]);
    __syncthreads();
    return mi;
}

// pad value of a smooth-mask node (carried in the instruction: kernels read
// it without indexing the plan's coefficient table)
DEV float mask_padv(const Instr& I) { return __int_as_float(I.a); }

DEV MaskInfo mask_weights(const Env& e, const Instr& I, float* w, float* dwa, float* dwb)
{
    return mask_info(e.params, I, e.L, *e.sh, e.nt, e.tid, w, dwa, dwb);
}

// Offsets past the signal end, for the LAST / CONST pads of a bounded smooth
// mask: each offset k >= L of the support contributes one pad copy with
// weight w_k.  Past b, w_k <= sig(-c(k - b)) < e^{-c(k - b)}, which is below
// eps (and w_k clamps to 0) from k = b + ln(1/eps)/c on; in fp32 the sigmoid
// itself is 0 once c(k - b) > 89.  The walk stops there, and never runs more
// than MASK_TAIL_MAX offsets past the end.
constexpr int MASK_TAIL_MAX = 65536;

struct MaskTail {
    int lo, hi;          // support offsets >= L (lo > hi: none)
    double s, sa, sb;    // sums of w_k, d w_k/da, d w_k/db over them
};

DEV MaskTail mask_tail(const Env& e, const Instr& I, bool grads)
{
    const int L = e.L;
    const MaskP mp = mask_params(e.params + I.mask, false);
    int kend = -1;
    if (mp.c > 0.f && mp.b == mp.b) {
        const float span = fminf(logf(1.f / fmaxf(mp.eps, 1e-38f)), 89.f) / mp.c + 2.f;
        const float ke = fminf(mp.b + span, (float)L + (float)MASK_TAIL_MAX);
        kend = ke >= (float)L ? (int)ke : -1;
    }
    int* si = e.sh->ints;
    if (e.tid == 0) { si[5] = INT_MAX; si[6] = -1; }
    __syncthreads();
    int lo = INT_MAX, hi = -1;
    double s = 0.0, sa = 0.0, sb = 0.0;
    for (int k = L + e.tid; k <= kend; k += e.nt) {
        float da = 0.f, db = 0.f;
        const float wk = mask_wk(mp, k, grads ? &da : nullptr, &db);
        if (wk > 0.f) {
            lo = min(lo, k);
            hi = max(hi, k);
            s += wk;
            sa += da;
            sb += db;
        }
    }
    atomicMin(&si[5], lo);
    atomicMax(&si[6], hi);
    __syncthreads();
    MaskTail mt;
    mt.lo = si[5];
    mt.hi = si[6];
    mt.s = wg_sum(s, e);
    mt.sa = grads ? wg_sum(sa, e) : 0.0;
    mt.sb = grads ? wg_sum(sb, e) : 0.0;
    return mt;
}

// out[t] = tail + sum_{k=L-t}^{L-1} v[k] for t in [0, L): the part of an
// offset table v (zero outside the mask support) that lies past the signal
// end for the output at t, plus the tail beyond the table.  fp64 sums: one
// contiguous chunk per thread, an exclusive suffix scan over the lanes and
// the totals of the later waves.
DEV void tail_weights(const float* v, float* out, int L, double tail, const Env& e)
{
    Shared& sh = *e.sh;
    const int nt = e.nt, tid = e.tid, lane = tid & 63, wv = tid >> 6;
    const int nw = (nt + 63) >> 6;
    const int ch = (L + nt - 1) / nt;
    const int k0 = min(L, tid * ch), k1 = min(L, k0 + ch);
    double c = 0.0;
    for (int k = k0; k < k1; ++k) c += (double)v[k];
    double r = c;                               // inclusive suffix over the lanes
    for (int d = 1; d < 64; d <<= 1) {
        const double o = __shfl_down(r, d);
        if (lane + d < 64) r += o;
    }
    double ex = __shfl_down(r, 1);              // lanes after this one
    if (lane == 63) ex = 0.0;
    if (lane == 0) sh.scan[wv] = r;
    __syncthreads();
    double acc = tail + ex;
    for (int q = wv + 1; q < nw; ++q) acc += sh.scan[q];
    for (int k = k1 - 1; k >= k0; --k) {
        acc += (double)v[k];
        if (k >= 1) out[L - k] = (float)acc;
    }
    if (tid == 0) out[0] = (float)tail;
    __syncthreads();
}

// ------------------------------------------------------------------ until

// Hard Until, one thread per output t: running min of phi over [t, t+i],
// max over i in [a, b] of min(running min, psi_{t+i}); phi wins ties.
// Adjoint (g != null): every output sends g_t to the one phi or psi sample
// that decides it.  The target of each t goes to `code` (phi index k as k,
// psi index k as -k-1, none as INT_MIN); then each position sums the g_t
// that target it in increasing t, so the result does not depend on the
// order in which threads finish.
DEV void until_hard(const Env& e, int a, int b, const float* phi, const float* psi, float* out,
                    const float* g, float* gphi, float* gpsi, int* code)
{
    const int L = e.L;
    const float rho_pad = e.P->rho_pad;
    for (int t = e.tid; t < L; t += e.nt) {
        const int imax = b < 0 ? L - 1 - t : min(b, L - 1 - t);
        if (a > imax) {
            if (out) out[t] = -rho_pad;
            if (g) code[t] = INT_MIN;
            continue;
        }
        float R = phi[t], best = -INFINITY;
        int kR = t, tgt = -1;
        bool tphi = false;
        for (int i = 0; i <= imax; ++i) {
            const float f = phi[t + i];
            if (f < R) { R = f; kR = t + i; }
            if (i >= a) {
                const float p = psi[t + i];
                const bool pw = R <= p;
                const float v = pw ? R : p;
                if (tgt < 0 || v > best) { best = v; tphi = pw; tgt = pw ? kR : t + i; }
            }
        }
        if (out) out[t] = best;
        if (g) code[t] = tphi ? tgt : -tgt - 1;
    }
    if (!g) return;
    __syncthreads();
    for (int j = e.tid; j < L; j += e.nt) {
        float sp = 0.f, sq = 0.f;
        for (int t = b < 0 ? 0 : max(0, j - b); t <= j; ++t) {
            const int c = code[t];
            if (c == j) sp += g[t];
            else if (c == -j - 1) sq += g[t];
        }
        gphi[j] += sp;
        gpsi[j] += sq;
    }
}

// Hard Until with an unbounded interval [a, inf), O(L) per trajectory.
// With m_a(t) = min of phi over [t, t+a-1] (a > 0) and the a = 0 form
//   U(s) = max_{j >= 0} min(min_{k <= j} phi_{s+k}, psi_{s+j}),
// out(t) = min(m_a(t), U(t+a)).  U satisfies U(s) = f_s(U(s+1)), U(L) = -inf,
// for the clamp map f_s(u) = min(phi_s, max(psi_s, u)) = clamp of u to
// [min(psi_s, phi_s), phi_s]; clamp maps compose into clamp maps, so U is a
// suffix scan of compositions.  The adjoint follows the same ties as the
// walk of until_hard (lowest index, phi wins): output s decides at phi_s
// (phi_s <= psi_s, or psi_s < phi_s <= U(s+1)), at psi_s (U(s+1) <= psi_s
// < phi_s), or passes its adjoint to output s+1 (psi_s < U(s+1) < phi_s); an
// output t goes to the window argmin of m_a when m_a(t) <= U(t+a).  The
// passed-on sums F(s) = h(s) + [s-1 passes] F(s-1) are a scan of affine
// maps; the window part is the hard window's adjoint.  Scratch units 0..15.
struct ClampMap {
    float lo, hi;   // u -> min(hi, max(lo, u)), lo <= hi
};
struct OpClamp {    // a after b
    __device__ __forceinline__ ClampMap operator()(ClampMap a, ClampMap b) const
    {
        auto f = [&](float x) { return x < a.lo ? a.lo : (x > a.hi ? a.hi : x); };
        return ClampMap{f(b.lo), f(b.hi)};
    }
};
struct Affine {
    float h;        // x -> h + c x, c in {0, 1}
    int c;
};
struct OpAffine {   // l then r
    __device__ __forceinline__ Affine operator()(Affine l, Affine r) const
    {
        return Affine{r.c ? r.h + l.h : r.h, l.c & r.c};
    }
};
enum { UH_PHI = 0, UH_PSI = 1, UH_PASS = 2 };

DEV void until_hard_unb(const Env& e, int a, const float* phi, const float* psi, float* out, const float* g,
                        float* gphi, float* gpsi)
{
    const int L = e.L;
    const float rho_pad = e.P->rho_pad;
    float* mA = S(e, 4);
    int* jA = (int*)S(e, 5);
    ClampMap* cm = (ClampMap*)S(e, 6);      // units 6, 7
    if (a > 0) win_hard(e, phi, mA, jA, -1.f, 0, a - 1, PAD_NEUTRAL, 0.f, (VI*)S(e, 0), (VI*)S(e, 2));
    scan_one<true>(cm, L, ClampMap{-INFINITY, INFINITY}, OpClamp(),
                   [&](int s) { return ClampMap{phi[s] <= psi[s] ? phi[s] : psi[s], phi[s]}; }, HeadDown(0, L),
                   e);                                                         // cm[s].lo = U(s)
    if (!g) {
        for (int t = e.tid; t < L; t += e.nt) {
            float v = -rho_pad;
            if (t + a <= L - 1) {
                const float u = cm[t + a].lo;
                v = (a > 0 && mA[t] <= u) ? mA[t] : u;
            }
            out[t] = v;
        }
        __syncthreads();
        return;
    }
    int* code = (int*)S(e, 8);
    Affine* fa = (Affine*)S(e, 9);          // units 9, 10
    float* gw = S(e, 11);                   // adjoint sent to the window argmin of m_a
    for (int s = e.tid; s < L; s += e.nt) {
        const float un = s + 1 < L ? cm[s + 1].lo : -INFINITY;
        int c = UH_PHI;
        if (!(phi[s] <= psi[s])) {
            const float w = phi[s] <= un ? phi[s] : un;
            c = w > psi[s] ? (phi[s] <= un ? UH_PHI : UH_PASS) : UH_PSI;
        }
        code[s] = c;
        // output t = s: to the window argmin, or to U(s + a)
        float gt = 0.f;
        bool win = false;
        if (s + a <= L - 1) {
            gt = g[s];
            win = a > 0 && mA[s] <= cm[s + a].lo;
        }
        gw[s] = win ? gt : 0.f;
    }
    __syncthreads();
    scan_one<false>(fa, L, Affine{0.f, 1}, OpAffine(),
                    [&](int s) {
                        const int t = s - a;
                        const float h = (t >= 0 && !(a > 0 && mA[t] <= cm[s].lo)) ? g[t] : 0.f;
                        return Affine{h, s > 0 && code[s - 1] == UH_PASS ? 1 : 0};
                    },
                    HeadUp(0, L), e);                                         // fa[s].h = F(s)
    for (int s = e.tid; s < L; s += e.nt) {
        if (code[s] == UH_PHI) gphi[s] += fa[s].h;
        else if (code[s] == UH_PSI) gpsi[s] += fa[s].h;
    }
    __syncthreads();
    if (a > 0) {
        float* gu = S(e, 15);
        win_hard_adj(e, gw, gu, jA, (double*)S(e, 12));                          // units 12..14
        for (int j = e.tid; j < L; j += e.nt) gphi[j] += gu[j];
        __syncthreads();
    }
}

// Smooth Until forward, one thread per output t:
//   P_i = sum_{k<=i} 2^{-z_phi(t+k)}   (running scaled sum: smooth min of phi)
//   Y_i = 1 / (P_i + 2^{-z_psi(t+i)})  (= exp(beta * smin(R_i, psi_{t+i})))
//   out = log2(sum_{i in [a,b]} w_i Y_i) / (beta log2 e)
// Ephi / Epsi hold the leaves 2^{-z}; w (smooth mask weights by offset i,
// Sec. VI) is null for the 0/1 interval.
DEV void until_smooth_fwd(const Env& e, int a, int b, const float* w, const SP* Ephi, const SP* Epsi,
                          float* out, float bl)
{
    const int L = e.L;
    const float rho_pad = e.P->rho_pad;
    for (int t = e.tid; t < L; t += e.nt) {
        const int imax = b < 0 ? L - 1 - t : min(b, L - 1 - t);
        if (a > imax) { out[t] = -rho_pad; continue; }
        SP P = sp_zero(), Z = sp_zero();
        for (int i = 0; i <= imax; ++i) {
            P = sp_add(P, Ephi[t + i]);
            if (i >= a) {
                SP Dn = sp_add(P, Epsi[t + i]);
                Z = sp_add(Z, SP{(w ? w[i] : 1.f) / Dn.s, -Dn.r});
            }
        }
        out[t] = sp_log2(Z) / bl;
    }
}

constexpr int UCK = 16;       // steps per block of the fp64 smooth Until adjoints
constexpr int UCK_SP = 32;    // of the scaled-pair adjoint (a checkpoint per block)
constexpr int UCK_CS = 32;    // checkpoint spacing of until_adj_r (two blocks)
constexpr int UCK_UNIT = 4, UCK_UNIT_MASK = 7;    // scratch unit where the checkpoints start (mask tables: units 4-6)
constexpr int UT_RMAX = 4;                        // outputs per lane at most
constexpr int UT_EX = 32;                         // positions of a wave's export buffer
constexpr int UT_TILE_B = 1024;                   // longest interval whose terms are staged in LDS

// checkpoints per lane, one per `per` steps, for the interval's end b (< 0: unbounded)
static __host__ __device__ __forceinline__ int until_cks(int b, int L, int per)
{
    return (b < 0 || b > L - 1 ? L - 1 : (b + UT_RMAX - 1 > L - 1 ? L - 1 : b + UT_RMAX - 1)) / per + 1;
}

// Smooth Until adjoint (checkpointed reverse sweep per output t):
//   d out / d psi_{t+i} = w_i Y_i^2 Q_i / Z,  Q_i = 2^{-z_psi(t+i)}
//   d out / d phi_{t+k} = e_k / Z * sum_{i >= max(k,a)} w_i Y_i^2,  e_k = 2^{-z_phi(t+k)}
//   d out / d w_i = Y_i / (beta Z)   (summed against d w/da, d w/db into pa, pb)
// Pass 1 recomputes Z and stores P every UCK_SP steps; pass 2 walks the
// checkpoint blocks backward, recomputing P inside each block.  The float
// contributions go through the lane-shifted accumulators of lane_stage
// (defined below), in the same fixed order as the fp64 adjoint.
DEV void lane_stage(int i, int tb, int lane, int L, float& accp, float& accq, float& stp, float& stq,
                    float* gphi, float* gpsi);

DEV void until_smooth_adj(const Env& e, int a, int b, const float* w, const float* dwa, const float* dwb,
                          const SP* Ephi, const SP* Epsi, const float* g, float* gphi, float* gpsi, SP* ck,
                          int ncks, float& pa, float& pb)
{
    const int L = e.L;
    const int lane = e.tid & 63;
    for (int base = 0; base < L; base += e.nt) {
        const int tb = base + e.tid - lane;
        const int t = tb + lane;
        const int imax = t >= L ? -1 : (b < 0 ? L - 1 - t : min(b, L - 1 - t));
        const float gt = t < L ? g[t] : 0.f;
        const bool act = a <= imax && gt != 0.f;
        SP* myck = ck + (size_t)e.tid * ncks;
        SP Z = sp_zero();
        if (act) {
            SP P = sp_zero();
            for (int i = 0; i <= imax; ++i) {
                if (i % UCK_SP == 0) myck[i / UCK_SP] = P;
                P = sp_add(P, Ephi[t + i]);
                if (i >= a) {
                    SP Dn = sp_add(P, Epsi[t + i]);
                    Z = sp_add(Z, SP{(w ? w[i] : 1.f) / Dn.s, -Dn.r});
                }
            }
        }
        const float gz = act ? gt / Z.s : 0.f;      // G / Z = gz * 2^{-Z.r}
        const int imax0 = b < 0 ? L - 1 - base : min(b, L - 1 - base);     // t = base: the longest chain
        const int wblk = a <= imax0 ? imax0 / UCK_SP + 1 : 0;
        float accp = 0.f, accq = 0.f, stp = 0.f, stq = 0.f;
        SP A = sp_zero();                   // suffix sum of w_i Y_i^2
        for (int blk = wblk - 1; blk >= 0; --blk) {
            const int i0 = blk * UCK_SP;
            const int i1 = act ? min(imax, i0 + UCK_SP - 1) : i0 - 1;      // this lane's last step in the block
            SP Ps[UCK_SP];
            SP Pc = i0 <= i1 ? myck[blk] : sp_zero();
#pragma unroll
            for (int q = 0; q < UCK_SP; ++q) {
                if (i0 + q <= i1) Pc = sp_add(Pc, Ephi[t + i0 + q]);
                Ps[q] = Pc;
            }
#pragma unroll
            for (int q = UCK_SP - 1; q >= 0; --q) {
                const int i = i0 + q;
                if (i <= i1) {
                    if (i >= a) {
                        const SP Q = Epsi[t + i];
                        const SP Dn = sp_add(Ps[q], Q);
                        const float y = 1.f / Dn.s;       // Y = y * 2^{-Dn.r}
                        const SP Y2{(w ? w[i] : 1.f) * y * y, -2 * Dn.r};
                        A = sp_add(A, Y2);
                        // psi: gz * w Y^2 * Q  (exponent -Z.r - 2 Dn.r + Q.r)
                        accq += ldexpf(gz * Y2.s * Q.s, clampe((long long)Y2.r + Q.r - Z.r));
                        if (w) {
                            const int ex = clampe(-(long long)Dn.r - Z.r);
                            pa += ldexpf(gz * dwa[i] * y, ex);
                            pb += ldexpf(gz * dwb[i] * y, ex);
                        }
                    }
                    const SP E = Ephi[t + i];
                    accp += ldexpf(gz * A.s * E.s, clampe((long long)A.r + E.r - Z.r));
                }
                if (i > 0) lane_stage(i, tb, lane, L, accp, accq, stp, stq, gphi, gpsi);
            }
        }
        if (wblk > 0 && t < L) {
            gphi[t] += accp;
            gpsi[t] += accq;
        }
        __syncthreads();
    }
}

// Smooth Until in fp64 against one reference exponent per trajectory.  The
// leaf terms 2^u, u = -beta log2(e) (phi or psi), are kept as the doubles
// 2^{u - M}, M = ceil(max u) - UF_TOP over both inputs.  While the exponent
// range max u - min u is at most UF_RANGE, they lie in [2^-600, 2^400], a sum of
// 2^25 of them below 2^425, the reciprocals and their sums in 2^-425 .. 2^624,
// and the adjoint's sums over outputs, at most 2^24 |G| / D with |G| < 2^128,
// below 2^752: nothing leaves the fp64 range.  (With M = ceil(max u) a sum
// over the outputs that share a position reached 2^1024 at |G| = 2^24.)  Beyond
// UF_RANGE (or with a non-finite value) the scaled-pair routines above take over.
constexpr int UF_RANGE = 1000, UF_TOP = 400;

// 2^{u - M} with exact exponent bookkeeping (u - ceil(u) is exact)
DEV double uterm(float u, int M)
{
    const float c = ceilf(u);
    return ldexp((double)__builtin_amdgcn_exp2f(u - c), (int)c - M);
}

// 1/d for a positive normal d: the hardware estimate alone.  Its relative
// error is at the float32 level (measured on gfx950: at most 4.6e-8 over 4M
// samples spanning 2^-1010 .. 2^31), which is all the float32 outputs need:
// the fp64 form is there for its exponent range, and every sum it feeds
// (Z, the suffix sums of Y^2) adds positive terms, so relative errors do not
// grow.  A Newton step would cost two more fp64 FMAs per term.
DEV double rcpd(double d)
{
    return __builtin_amdgcn_rcp(d);
}

// log2 of a positive double, as the double (exponent - M) + log2(mantissa)
DEV double log2_minus(double z, int M)
{
    int ez;
    const double mz = frexp(z, &ez);
    return (double)(ez - M) + (double)__builtin_amdgcn_logf((float)mz);
}

// Reference exponent M of the two leaf traces; false when the fp64 form
// cannot hold them.
DEV bool until_ref(const float* phi, const float* psi, int L, float bl, const Env& e, int& M)
{
    Shared& sh = *e.sh;
    int hi = INT_MIN, lo = INT_MAX, bad = 0;
    for (int j = e.tid; j < L; j += e.nt) {
        const float u1 = -bl * phi[j], u2 = -bl * psi[j];
        if (!(fabsf(u1) < 1e9f) || !(fabsf(u2) < 1e9f)) {
            bad = 1;                                 // also catches NaN
        } else {
            hi = max(hi, (int)ceilf(fmaxf(u1, u2)));
            lo = min(lo, (int)floorf(fminf(u1, u2)));
        }
    }
    if (e.tid == 0) {
        sh.ints[2] = INT_MIN;
        sh.ints[3] = INT_MAX;
        sh.ints[4] = 0;
    }
    __syncthreads();
    atomicMax(&sh.ints[2], hi);
    atomicMin(&sh.ints[3], lo);
    if (bad) atomicOr(&sh.ints[4], 1);
    __syncthreads();
    M = sh.ints[2] - UF_TOP;
    const bool ok = sh.ints[4] == 0 && (long long)sh.ints[2] - (long long)sh.ints[3] <= UF_RANGE;
    __syncthreads();
    return ok;
}

// leaf terms of both inputs as doubles 2^{u - M} (Ep, Eq)
DEV void until_terms(const float* phi, const float* psi, int L, float bl, int M, double* Ep, double* Eq, int nt, int tid)
{
    for (int j = tid; j < L; j += nt) {
        Ep[j] = uterm(-bl * phi[j], M);
        Eq[j] = uterm(-bl * psi[j], M);
    }
    __syncthreads();
}

// The fp64 forms: terms p_j = 2^{u_phi - M}, q_j = 2^{u_psi - M}; output t sums
// Y = 1 / D, D_{t,j} = P_{t,j} + q_j, P_{t,j} = p_t + .. + p_j, over j = t+a ..
// t+b: Z_t = sum_j Y (the same sums as until_smooth_fwd, with Y scaled by 2^{-M}).
//
// A lane owns R consecutive outputs t_0 .. t_0+R-1 and walks j = t_0 + s over
// s = 0, 1, ..: since P_{t_0+r,j} = C_r + P_{t_0+R-1,j} with the constant
// C_r = p_{t_0+r} + .. + p_{t_0+R-2}, the outputs share the two term reads
// and the running sum of a step, and every D is one more addition of positive
// terms (nothing cancels, whatever the range).  The walk is bound by vector
// issue: per term an add, a reciprocal (4 issue slots) and the sum, against
// two 8-byte LDS reads per term and a chain of dependent adds with one output
// per thread.  R = 1 or 2 while one pass over the work-group, and a second for at
// most an eighth of it, takes the trajectory (a lane is worth more than the
// shared reads: 300 trajectories of 513 samples, interval [20, 200], 256 threads,
// forward / backward 21.8 / 66.0 us with R = 2 in two passes, 30.4 / 89.2 with
// R = 4 in one), else R = 4.
// n consecutive terms from p: 16-byte reads where the lanes are 2 or 4 outputs
// apart (p is then 16-byte aligned; the 8-byte reads of lanes 32 bytes apart
// fall on each LDS bank four times, and bound the walk)
template <int R, int N>
DEV void load_terms(const double* p, double (&v)[N])
{
    if (R == 1) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = p[k];
    } else {
#pragma unroll
        for (int k = 0; k < N; k += 2) {
            const double2 t = *(const double2*)(p + k);
            v[k] = t.x;
            v[k + 1] = t.y;
        }
    }
}

DEV int until_outputs(int L, int nt)
{
    const int pass = nt + (nt >> 3);
    return L <= pass ? 1 : (L <= 2 * pass ? 2 : 4);
}

// One pass: the outputs base .. base + nt R - 1; Ep, Eq hold the terms from
// position j0 on.
template <int R>
DEV void until_fwd_r(const Env& e, int a, int b, const double* Ep, const double* Eq, int j0, int base, float* out,
                     double* zs, float bl, int M)
{
    const int L = e.L;
    const float rho_pad = e.P->rho_pad;
    const int t0 = base + e.tid * R;
    if (t0 < L) {
        const double* p = Ep + (t0 - j0);
        const double* q = Eq + (t0 - j0);
        const int last = L - 1 - t0;                                 // steps 0 .. last stay inside
        const int smax = b < 0 ? last : min(b + R - 1, last);
        double Z[R], C[R];
#pragma unroll
        for (int r = 0; r < R; ++r) Z[r] = 0.0;
        if (R > 1 && a < R - 1) {
            // steps before output t_0+R-1 begins
            double Pr[R];
#pragma unroll
            for (int r = 0; r < R; ++r) Pr[r] = 0.0;
#pragma unroll
            for (int s = 0; s < R - 1; ++s)
                if (s <= smax) {
                    const double ps = p[s], qs = q[s];
#pragma unroll
                    for (int r = 0; r <= s; ++r) {
                        Pr[r] += ps;
                        if (s - r >= a && (b < 0 || s - r <= b)) Z[r] += rcpd(Pr[r] + qs);
                    }
                }
        }
        C[R - 1] = 0.0;
#pragma unroll
        for (int r = R - 2; r >= 0; --r) C[r] = C[r + 1] + (t0 + r < L ? p[r] : 0.0);
        double P = 0.0;
        int s = R - 1;
        for (; s + 8 <= min(a, smax + 1); s += 8) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = p[s + k];
#pragma unroll
            for (int k = 0; k < 8; ++k) P += v[k];
        }
        for (; s < min(a, smax + 1); ++s) P += p[s];
        // the window's two ends, where only some of the outputs take the term
        auto edge = [&](int hi) {
            for (; s <= hi; ++s) {
                P += p[s];
                const double d = P + q[s];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double y = rcpd(d + C[r]);
                    if (s - r >= a && (b < 0 || s - r <= b)) Z[r] += y;
                }
            }
        };
        const int full = b < 0 ? smax : min(b, smax);                // last step every output takes
        edge(min((a + 2 * R - 2) / R * R - 1, smax));                // (to a multiple of R)
        constexpr int U = 8;
        for (; s + U - 1 <= full; s += U) {
            double v[U], w[U];
            load_terms<R>(p + s, v);
            load_terms<R>(q + s, w);
#pragma unroll
            for (int k = 0; k < U; ++k) {
                P += v[k];
                const double d = P + w[k];
#pragma unroll
                for (int r = 0; r < R; ++r) Z[r] += rcpd(r == R - 1 ? d : d + C[r]);
            }
        }
        edge(smax);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int t = t0 + r;
            if (t >= L) continue;
            if (a > (b < 0 ? L - 1 - t : min(b, L - 1 - t))) {
                out[t] = -rho_pad;
                continue;
            }
            out[t] = (float)(log2_minus(Z[r], M) / (double)bl);
            if (zs) zs[t] = Z[r];
        }
    }
}

// The masked form (weights w_i by offset i): one output per thread, the terms
// read eight at a time (independent loads ahead of the dependent sums).
DEV void until_fwd_w(const Env& e, int a, int b, const float* w, const double* Ep, const double* Eq, float* out,
                     double* zs, float bl, int M)
{
    const int L = e.L;
    const float rho_pad = e.P->rho_pad;
    for (int t = e.tid; t < L; t += e.nt) {
        const int imax = min(b, L - 1 - t);
        if (a > imax) { out[t] = -rho_pad; continue; }
        const double* p = Ep + t;
        const double* q = Eq + t;
        double P = 0.0, Z = 0.0;
        int i = 0;
        for (; i < a; ++i) P += p[i];
        for (; i + 8 <= imax + 1; i += 8) {
            double v[8], x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                v[k] = p[i + k];
                x[k] = q[i + k];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                P += v[k];
                Z += (double)w[i + k] * rcpd(P + x[k]);
            }
        }
        for (; i <= imax; ++i) {
            P += p[i];
            Z += (double)w[i] * rcpd(P + q[i]);
        }
        out[t] = (float)(log2_minus(Z, M) / (double)bl);
        if (zs) zs[t] = Z;
    }
}

// value of the lane below (lane 0 receives 0): one DPP wave shift
DEV float lane_shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}

// One step of the lane-shifted adjoint accumulators of the Until adjoints
// (step i > 0, walked downwards, the same i in every wave of the
// work-group): lane 63 holds the finished sum of position tb + 64 + s,
// s = i - 1; it is parked in lane s % 64 of the staging pair, and a full
// stage (s a multiple of 64: positions tb + 64 + s + lane) is added to the
// adjoint slots, followed by a barrier.  Then the accumulators move up a lane.
DEV void lane_stage(int i, int tb, int lane, int L, float& accp, float& accq, float& stp, float& stq, float* gphi,
                    float* gpsi)
{
    const int s_ = i - 1, j = s_ & 63;
    const float dp = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(accp), 63));
    const float dq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(accq), 63));
    if (lane == j) {
        stp = dp;
        stq = dq;
    }
    if (j == 0) {
        const int pos = tb + 64 + s_ + lane;
        if (pos < L) {
            gphi[pos] += stp;
            gpsi[pos] += stq;
        }
        stp = 0.f;
        stq = 0.f;
        __syncthreads();
    }
    accp = lane_shr1(accp);
    accq = lane_shr1(accq);
}

// Adjoint on the fp64 terms (the derivatives are ratios of terms, so the
// reference cancels).  Z_t comes from the forward recompute (zs).  With
// m_{t,j} = (G_t / Z_t) Y_{t,j}^2,
//   d out / d psi_j = q_j sum_t m_{t,j},  d out / d phi_k = p_k sum_{t <= k <= j} m_{t,j}.
// A lane owns the R outputs of until_fwd_r and walks j = t_0 + s downwards.  A
// forward sweep of additions keeps P_{t_0+R-1,j} every UCK_CS steps; the reverse
// walk rebuilds each block's sums from its checkpoint.  Step s adds
// S = sum_r m_{t_0+r,j} to the psi sum of position j, and the running sum A of
// S over the steps so far (all terms at or past j) to its phi sum.  Below
// step R-1 position t_0+s lies before the last outputs, so the sums B_r over
// the first r+1 outputs are carried as well.
// The lanes of a wave walk the same steps, so the position of lane l, sum c
// (s = R m + c) is that of lane l-1 one macro-step m earlier: the 2 R fp64
// sums move up one lane per R steps (a DPP shift), and the positions leaving
// lane 63 are finished for this wave.  They go to a buffer of the wave, which
// is added to the adjoint slots every UT_EX positions and scaled by p_j, q_j
// there.  All waves of the work-group walk the same steps (those of the
// longest chain of the pass), so the buffers are added at the same points in
// every wave, where they cover disjoint positions, and a barrier separates the
// points: the order of every addition is fixed (bitwise reproducible).
// Against one output per lane (three multiplies, two conversions, two float
// adds, two lane reads and two shifts per term) a term takes an add, the
// reciprocal, two multiplies and about 2.5 adds.
// One pass: the outputs base .. base + nt R - 1; Ep, Eq hold the terms of the
// positions j0 .. jl - 1.
template <int R>
DEV void until_adj_r(const Env& e, int a, int b, const double* Ep, const double* Eq, int j0, int jl, int base,
                     const double* zs, const float* g, float* gphi, float* gpsi, double* ck, double* exb)
{
    const int L = e.L, nt = e.nt;
    const int lane = e.tid & 63;
    double* ex = exb + (e.tid >> 6) * (2 * UT_EX);             // psi sums, then phi sums
    {
        const int tb = base + (e.tid - lane) * R;
        const int t0 = tb + lane * R;
        const double* p = Ep + (t0 - j0);
        const double* q = Eq + (t0 - j0);
        const int last = L - 1 - t0;
        double wz[R], C[R];
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int t = t0 + r;
            const float gt = t < L ? g[t] : 0.f;
            const bool act = gt != 0.f && a <= (b < 0 ? L - 1 - t : min(b, L - 1 - t));
            wz[r] = act ? (double)gt / zs[t] : 0.0;
            any |= act;
        }
        C[R - 1] = 0.0;
#pragma unroll
        for (int r = R - 2; r >= 0; --r) C[r] = C[r + 1] + (t0 + r < L ? p[r] : 0.0);
        // own steps (none where no output has an adjoint), steps of the pass
        const int smax = any ? (b < 0 ? last : min(b + R - 1, last)) : -1;
        const int sw = b < 0 ? L - 1 - base : min(b + R - 1, L - 1 - base);
        const int wblk = a <= sw ? sw / UCK + 1 : 0;
        {
            double P = 0.0;
            for (int blk = 0; blk <= smax / UCK && smax >= 0; ++blk) {
                if (blk % 2 == 0) ck[blk / 2 * nt + e.tid] = P;
                if ((blk + 1) * UCK <= smax) {                       // a next block: this one is whole
                    double v[UCK];
                    load_terms<R>(p + blk * UCK, v);
#pragma unroll
                    for (int k = 0; k < UCK; ++k)
                        if (k >= R - 1 || blk > 0) P += v[k];
                }
            }
        }
        double A = 0.0, B[R], sq[R], sp[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            B[r] = sq[r] = sp[r] = 0.0;
        }
        ex[lane] = 0.0;                                        // (2 UT_EX = 64 sums)
        for (int blk = wblk - 1; blk >= 0; --blk) {
            const int s0 = blk * UCK;
            const int n = min(UCK, smax - s0 + 1);                   // own steps of the block (<= 0: none)
            double v[UCK], d[UCK];
            if (__all(n >= UCK)) {
                load_terms<R>(p + s0, v);
                load_terms<R>(q + s0, d);
            } else {
#pragma unroll
                for (int k = 0; k < UCK; ++k) {
                    v[k] = k < n ? p[s0 + k] : 0.0;
                    d[k] = k < n ? q[s0 + k] : 1e300;                // Y^2 = 0 past the own steps
                }
            }
            double P = n > 0 ? ck[blk / 2 * nt + e.tid] : 0.0;
            if (blk % 2 == 1 && n > 0) {                             // the block before, from its checkpoint
                double u[UCK];
                load_terms<R>(p + (s0 - UCK), u);
#pragma unroll
                for (int k = 0; k < UCK; ++k)
                    if (k >= R - 1 || blk > 1) P += u[k];
            }
#pragma unroll
            for (int k = 0; k < UCK; ++k) {
                if (k >= R - 1 || blk > 0) P += v[k];
                d[k] += P;
            }
            auto steps = [&](auto inner) {
#pragma unroll
                for (int k = UCK - 1; k >= 0; --k) {
                    const int s = s0 + k, c = k % R;
                    double S = 0.0;
                    if (decltype(inner)::value || s >= a) {
                        double Dn[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) Dn[r] = r == R - 1 ? d[k] : d[k] + C[r];
                        if (R > 1 && !decltype(inner)::value && k < R - 1 && blk == 0) {
                            // before output t_0+R-1 begins: P of output r is p_{t_0+r} + .. + p_j
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                double Pr = 0.0;
#pragma unroll
                                for (int i = r; i <= k; ++i) Pr += v[i];
                                Dn[r] = Pr + d[k];
                            }
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const double y = rcpd(Dn[r]);
                            double m = (wz[r] * y) * y;
                            if (!decltype(inner)::value && !(s - r >= a && (b < 0 || s - r <= b))) m = 0.0;
                            S += m;
                            B[r] += S;
                        }
                        A = B[R - 1];
                    }
                    sq[c] += S;
                    sp[c] += (R > 1 && !decltype(inner)::value && k < R - 1 && blk == 0) ? B[k % R] : A;
                    if (c == 0 && s > 0) {
                        // macro-step m = s / R is done: lane 63's positions leave the wave
                        const int i = (s / R - 1) * R & (UT_EX - 1);
                        if (lane == 63) {
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                ex[i + r] = sq[r];
                                ex[UT_EX + i + r] = sp[r];
                            }
                        }
                        if (i == 0) {
                            __threadfence_block();                   // lane 63's values, for the other lanes
                            const int at = lane & (UT_EX - 1), j = tb + 64 * R + s - R + at;
                            const double sum = ex[lane];
                            if (j < jl) {
                                if (lane < UT_EX) gpsi[j] += (float)(sum * Eq[j - j0]);
                                else gphi[j] += (float)(sum * Ep[j - j0]);
                            }
                            ex[lane] = 0.0;
                            __syncthreads();
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            sq[r] = dpp8<0x138>(sq[r]);
                            sp[r] = dpp8<0x138>(sp[r]);
                        }
                    }
                    // (interleaving more steps than this spills)
                    if (k % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                }
            };
            if (s0 >= a + R - 1 && s0 > 0 && (b < 0 || s0 + UCK - 1 <= b)) steps(std::true_type());
            else steps(std::false_type());
        }
        if (wblk > 0)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int j = t0 + r;
                if (j < L) {
                    gpsi[j] += (float)(sq[r] * Eq[j - j0]);
                    gphi[j] += (float)(sp[r] * Ep[j - j0]);
                }
            }
        __syncthreads();
    }
}

// The masked form (weights w_i by offset i, one output per lane): Z = sum w_i Y_i,
// A sums w_i Y_i^2, and d out / d w_i = Y_i / (beta Z) is summed against
// d w/da, d w/db into pa, pb (per thread, before the division by beta).  The
// lane-shifted sums are floats, parked in a staging register pair.
DEV void until_adj_w(const Env& e, int a, int b, const float* w, const float* dwa, const float* dwb,
                     const double* Ep, const double* Eq, const double* zs, const float* g, float* gphi, float* gpsi,
                     double* ck, int ncks, float& pa, float& pb)
{
    const int L = e.L;
    const int lane = e.tid & 63;
    for (int base = 0; base < L; base += e.nt) {
        const int tb = base + e.tid - lane;
        const int t = tb + lane;
        const int imax = t >= L ? -1 : (b < 0 ? L - 1 - t : min(b, L - 1 - t));
        const float gt = t < L ? g[t] : 0.f;
        const bool act = a <= imax && gt != 0.f;
        const int nblk = act ? imax / UCK + 1 : 0;
        const double* ep = Ep + t;
        const double* eq = Eq + t;
        double* myck = ck + (size_t)e.tid * ncks;
        double Z = 1.0;
        if (act) {
            // Z comes from the forward recompute: only the block-start prefixes of P
            Z = zs[t];
            double P = 0.0;
            for (int blk = 0; blk < nblk; ++blk) {
                myck[blk] = P;
                if (blk + 1 < nblk) {                  // blocks before the last are full
                    const int i0 = blk * UCK;
                    double v[UCK];
#pragma unroll
                    for (int k = 0; k < UCK; ++k) v[k] = ep[i0 + k];
#pragma unroll
                    for (int k = 0; k < UCK; ++k) P += v[k];
                }
            }
        }
        const double wz = act ? (double)gt / Z : 0.0;
        const int imax0 = b < 0 ? L - 1 - base : min(b, L - 1 - base);     // t = base: the longest chain
        const int wblk = a <= imax0 ? imax0 / UCK + 1 : 0;
        float accp = 0.f, accq = 0.f;
        float stp = 0.f, stq = 0.f;         // staged finished sums (see the shift below)
        double A = 0.0;                     // G/Z times the suffix sum of w_i Y_i^2
        double da = 0.0, db = 0.0;          // sum of dw_i Y_i
        for (int blk = wblk - 1; blk >= 0; --blk) {
            const int i0 = blk * UCK;
            const int n = blk < nblk ? min(UCK, imax - i0 + 1) : 0;
            double v[UCK], q[UCK], Ps[UCK];
            double Pc = n > 0 ? myck[blk] : 0.0;
#pragma unroll
            for (int k = 0; k < UCK; ++k) {
                v[k] = k < n ? ep[i0 + k] : 0.0;
                q[k] = k < n ? eq[i0 + k] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < UCK; ++k) {
                Pc += v[k];
                Ps[k] = Pc;
            }
#pragma unroll
            for (int k = UCK - 1; k >= 0; --k) {
                const int i = i0 + k;
                if (k < n) {
                    if (i >= a) {
                        const double y = rcpd(Ps[k] + q[k]);
                        const double y2 = wz * (double)w[i] * y * y;       // G/Z w_i Y_i^2
                        A += y2;
                        accq += (float)(y2 * q[k]);
                        da += (double)dwa[i] * y;
                        db += (double)dwb[i] * y;
                    }
                    accp += (float)(A * v[k]);
                }
                if (i > 0) lane_stage(i, tb, lane, L, accp, accq, stp, stq, gphi, gpsi);
            }
        }
        if (wblk > 0 && t < L) {
            gphi[t] += accp;
            gpsi[t] += accq;
        }
        __syncthreads();
        pa += (float)(wz * da);
        pb += (float)(wz * db);
    }
}

// Terms of both inputs for the outputs of the pass at `base` (their windows end
// at b + R - 1 steps) into the LDS tile; returns the first position past it.
// With slots in the workspace the Until's reads (two terms per step and lane,
// 32 bytes apart) would otherwise go through the vector cache.
DEV int until_tile(const Env& e, const float* phi, const float* psi, int base, int n, float bl, int M, double* Ep,
                   double* Eq)
{
    const int jl = min(e.L, base + n);
    __syncthreads();                        // the previous pass has read its tile
#pragma unroll 4
    for (int j = base + e.tid; j < jl; j += e.nt) {
        Ep[j - base] = uterm(-bl * phi[j], M);
        Eq[j - base] = uterm(-bl * psi[j], M);
    }
    __syncthreads();
    return jl;
}

template <int R>
DEV void until_fwd_passes(const Env& e, int a, int b, const float* phi, const float* psi, double* Ep, double* Eq,
                          float* out, double* zs, float bl, int M)
{
    for (int base = 0; base < e.L; base += e.nt * R) {
        if (e.tile) until_tile(e, phi, psi, base, e.nt * R + (b < 0 ? e.L - 1 : b) + R, bl, M, Ep, Eq);
        until_fwd_r<R>(e, a, b, Ep, Eq, e.tile ? base : 0, base, out, zs, bl, M);
    }
}

template <int R>
DEV void until_adj_passes(const Env& e, int a, int b, const float* phi, const float* psi, double* Ep, double* Eq,
                          const double* zs, const float* g, float* gphi, float* gpsi, double* ck, double* exb, float bl,
                          int M)
{
    for (int base = 0; base < e.L; base += e.nt * R) {
        int j0 = 0, jl = e.L;
        if (e.tile) {
            jl = until_tile(e, phi, psi, base, e.nt * R + (b < 0 ? e.L - 1 : b) + R, bl, M, Ep, Eq);
            j0 = base;
        }
        until_adj_r<R>(e, a, b, Ep, Eq, j0, jl, base, zs, g, gphi, gpsi, ck, exb);
    }
}

// The smooth Until without a mask, fp64 form.  The terms lie in the scratch
// (all of them) or pass by pass in the LDS tile (e.tile > 0: its positions).
DEV void until_smooth_fwd_d(const Env& e, int a, int b, const float* phi, const float* psi, float* out, double* zs,
                            float bl, int M)
{
    double* Ep = e.tile ? (double*)e.lds : (double*)S(e, 0);
    double* Eq = e.tile ? Ep + e.tile : (double*)S(e, 2);
    if (!e.tile) until_terms(phi, psi, e.L, bl, M, Ep, Eq, e.nt, e.tid);
    switch (until_outputs(e.L, e.nt)) {
    case 1: until_fwd_passes<1>(e, a, b, phi, psi, Ep, Eq, out, zs, bl, M); break;
    case 2: until_fwd_passes<2>(e, a, b, phi, psi, Ep, Eq, out, zs, bl, M); break;
    default: until_fwd_passes<4>(e, a, b, phi, psi, Ep, Eq, out, zs, bl, M); break;
    }
}

DEV void until_smooth_adj_d(const Env& e, int a, int b, const float* phi, const float* psi, const double* zs,
                            const float* g, float* gphi, float* gpsi, float bl, int M)
{
    double* exb = (double*)e.lds;                       // nt of them: 2 UT_EX per wave
    double* Ep = e.tile ? exb + e.nt : (double*)S(e, 0);
    double* Eq = e.tile ? Ep + e.tile : (double*)S(e, 2);
    double* ck = e.tile ? Eq + e.tile : (double*)S(e, UCK_UNIT);
    if (!e.tile) until_terms(phi, psi, e.L, bl, M, Ep, Eq, e.nt, e.tid);
    switch (until_outputs(e.L, e.nt)) {
    case 1: until_adj_passes<1>(e, a, b, phi, psi, Ep, Eq, zs, g, gphi, gpsi, ck, exb, bl, M); break;
    case 2: until_adj_passes<2>(e, a, b, phi, psi, Ep, Eq, zs, g, gphi, gpsi, ck, exb, bl, M); break;
    default: until_adj_passes<4>(e, a, b, phi, psi, Ep, Eq, zs, g, gphi, gpsi, ck, exb, bl, M); break;
    }
}

// ------------------------------------------------------------------ instructions

DEV bool is_smooth(const Instr& I) { return I.flags & F_SMOOTH; }

// Run one instruction forward with the given slot map (fwd or bwd).  FULL =
// false leaves out the operators of plan_is_plain's complement.
template <bool FULL>
DEV void exec_fwd(const Env& e, const Instr& I, bool bwdmap)
{
    const int o = bwdmap ? I.b_out : I.f_out;
    const int i0 = bwdmap ? I.b_in0 : I.f_in0;
    const int i1 = bwdmap ? I.b_in1 : I.f_in1;
    float* out = slot(e, o);
    const int L = e.L;
    const float sg = (I.flags & F_MIN) ? -1.f : 1.f;
    switch (I.kind) {
    case K_TRUE:
        for (int t = e.tid; t < L; t += e.nt) out[t] = e.P->rho_max;
        break;
    case K_LIN:
    case K_NORM:        // (evaluated by op_preds, before the first instruction, unless the plan has n_pred = 0)
        if (!bwdmap) op_pred(e, I, out);
        break;
    case K_NOT: {
        const float* u = slot(e, i0);
        for (int t = e.tid; t < L; t += e.nt) out[t] = -u[t];
        break;
    }
    case K_NARY:
        op_nary_fwd(e, I, bwdmap ? I.b_ch : I.f_ch, out);
        break;
    case K_WIN: {
        const float* u = slot(e, i0);
        const int khi = (I.flags & F_UNB) ? -1 : I.b;
        const float padv = e.P->coef[I.coef];
        if (!is_smooth(I)) {
            win_hard(e, u, out, nullptr, sg, I.a, khi, I.pad, padv, (VI*)S(e, 0), (VI*)S(e, 2));
        } else if (FULL && (I.flags & F_SOFT)) {
            // softmax-weighted mean over the window: out = sum u 2^{z} / sum 2^{z};
            // LAST / CONST add np copies of the pad value v to both sums
            const float bl = pbeta(e, I) * LOG2E;
            SP* den = (SP*)S(e, 4);
            SP* num = (SP*)S(e, 6);
            win_smooth_sum(e, u, den, sg * bl, I.a, khi, I.pad, padv, (SP*)S(e, 0), (SP*)S(e, 2));
            win_smooth_sum_w(e, u, num, sg * bl, I.a, khi, (SP*)S(e, 0), (SP*)S(e, 2));
            const float v = I.pad == PAD_LAST ? u[L - 1] : padv;
            for (int t = e.tid; t < L; t += e.nt) {
                SP nm = num[t];
                const bool padded = khi >= 0 && I.pad != PAD_NEUTRAL && t + khi > L - 1;
                if (padded) {
                    const int np = min(khi - I.a + 1, t + khi - (L - 1));
                    SP pv = sp_leaf(sg * bl * v);
                    pv.s *= (float)np * v;
                    nm = sp_add(nm, pv);
                }
                out[t] = (t + I.a <= L - 1 || padded) ? sp_ratio(nm, den[t]) : -sg * e.P->rho_pad;
            }
        } else {
            const float bl = pbeta(e, I) * LOG2E;
            SP* acc = (SP*)S(e, 4);
            win_smooth_sum(e, u, acc, sg * bl, I.a, khi, I.pad, padv, (SP*)S(e, 0), (SP*)S(e, 2));
            const bool unb = khi < 0;
            for (int t = e.tid; t < L; t += e.nt) {
                const bool any = (t + I.a <= L - 1) || (!unb && I.pad != PAD_NEUTRAL && t + khi > L - 1);
                out[t] = any ? sg * sp_log2(acc[t]) / bl : -sg * e.P->rho_pad;
            }
        }
        break;
    }
    case K_MASK: {
        if constexpr (FULL) {
        const float* u = slot(e, i0);
        float* w = S(e, 6);
        MaskInfo mi = mask_weights(e, I, w, nullptr, nullptr);
        // LAST / CONST pads of a bounded mask: support offsets past the end
        const bool padm = I.pad != PAD_NEUTRAL && !(I.flags & F_MASK_UNB);
        MaskTail mt{INT_MAX, -1, 0.0, 0.0, 0.0};
        if (padm) mt = mask_tail(e, I, false);
        const int klo = mi.any ? mi.klo : mt.lo;             // whole support
        const int khi = mt.hi >= 0 ? mt.hi : mi.khi;
        const bool anyk = mi.any || mt.hi >= 0;
        const float padv = mask_padv(I);
        if (!is_smooth(I)) {
            if (!anyk) {
                for (int t = e.tid; t < L; t += e.nt) out[t] = -sg * e.P->rho_pad;
            } else {
                const int kh = ((I.flags & F_MASK_UNB) && khi == L - 1) ? -1 : khi;
                win_hard(e, u, out, nullptr, sg, klo, kh, padm ? I.pad : PAD_NEUTRAL, padv, (VI*)S(e, 0),
                         (VI*)S(e, 2));
            }
            break;
        }
        const float bl = pbeta(e, I) * LOG2E;
        SP* acc = (SP*)S(e, 4);
        SP* E = (SP*)S(e, 8);
        float* TW = S(e, 7);
        const bool core = mi.clo <= mi.chi;
        if (core) {
            const int kh = ((I.flags & F_MASK_UNB) && mi.chi == L - 1) ? -1 : mi.chi;
            win_smooth_sum(e, u, acc, sg * bl, mi.clo, kh, PAD_NEUTRAL, 0.f, (SP*)S(e, 0), (SP*)S(e, 2));
        }
        for (int j = e.tid; j < L; j += e.nt) E[j] = sp_leaf(sg * bl * u[j]);
        if (padm) tail_weights(w, TW, L, mt.s, e);
        __syncthreads();
        const SP Ev = sp_leaf(sg * bl * (I.pad == PAD_LAST ? u[L - 1] : padv));
        for (int t = e.tid; t < L; t += e.nt) {
            // band terms are summed one by one (up to a few hundred of them):
            // accumulate with a double mantissa so the error does not grow with the count
            SPD a{0.0, SP_NEG};
            if (core) a = spd_add(a, SP{acc[t].s * mi.wc, acc[t].r});
            const int b0 = mi.klo, b1 = core ? mi.clo - 1 : mi.khi;
            for (int k = b0; k <= b1 && t + k < L; ++k) a = spd_add(a, SP{w[k] * E[t + k].s, E[t + k].r});
            if (core)
                for (int k = mi.chi + 1; k <= mi.khi && t + k < L; ++k)
                    a = spd_add(a, SP{w[k] * E[t + k].s, E[t + k].r});
            const bool pt = padm && anyk && t + khi > L - 1;   // pad copies for this output
            if (pt) a = spd_add(a, SP{TW[t] * Ev.s, Ev.r});
            const bool any = (mi.any && t + mi.klo <= L - 1) || pt;
            out[t] = any ? sg * sp_log2(spd_to_sp(a)) / bl : -sg * e.P->rho_pad;
        }
        }
        break;
    }
    case K_UNTIL: {
        const float* phi = slot(e, i0);
        const float* psi = slot(e, i1);
        // outer index range [ua, ub]; a smooth mask (Sec. VI) replaces it by
        // its support {w > 0} and weights the terms
        int ua = I.a, ub = I.b;
        const float* w = nullptr;
        if constexpr (FULL) if (I.mask >= 0) {
            float* wt = S(e, 4);
            const MaskInfo mi = mask_weights(e, I, wt, nullptr, nullptr);
            if (!mi.any) {
                for (int t = e.tid; t < L; t += e.nt) out[t] = -e.P->rho_pad;
                break;
            }
            ua = mi.klo;
            ub = mi.khi;
            w = wt;
        }
        if (!is_smooth(I)) {
            if (ub < 0 && I.mask < 0) until_hard_unb(e, ua, phi, psi, out, nullptr, nullptr, nullptr);
            else until_hard(e, ua, ub, phi, psi, out, nullptr, nullptr, nullptr, nullptr);
        } else if constexpr (FULL) {
            const float bl = pbeta(e, I) * LOG2E;
            int M;
            if (until_ref(phi, psi, L, bl, e, M)) {
                // the backward's recompute keeps Z in the instruction's slot pair for the adjoint
                double* zs = bwdmap ? (double*)slot(e, I.coef) : nullptr;
                if (!w) {
                    until_smooth_fwd_d(e, ua, ub, phi, psi, out, zs, bl, M);
                    break;
                }
                double* Ep = (double*)S(e, 0);
                double* Eq = (double*)S(e, 2);
                until_terms(phi, psi, L, bl, M, Ep, Eq, e.nt, e.tid);
                until_fwd_w(e, ua, ub, w, Ep, Eq, out, zs, bl, M);
                break;
            }
            SP* Ephi = (SP*)S(e, 0);
            SP* Epsi = (SP*)S(e, 2);
            for (int j = e.tid; j < L; j += e.nt) {
                Ephi[j] = sp_leaf(-bl * phi[j]);
                Epsi[j] = sp_leaf(-bl * psi[j]);
            }
            __syncthreads();
            until_smooth_fwd(e, ua, ub, w, Ephi, Epsi, out, bl);
        }
        break;
    }
    default:
        break;
    }
}

// Adjoint of one instruction (backward slot map).  Children adjoints are
// written (not accumulated): every node has exactly one parent.
template <bool FULL>
DEV void exec_adj(const Env& e, const Instr& I, float* mask_part)
{
    const int L = e.L;
    const float sg = (I.flags & F_MIN) ? -1.f : 1.f;
    const float* g = slot(e, I.g_out);
    switch (I.kind) {
    case K_TRUE:
    case K_LIN:
    case K_NORM:
        break;
    case K_NOT: {
        float* gu = slot(e, I.g_in0);
        for (int t = e.tid; t < L; t += e.nt) gu[t] = -g[t];
        break;
    }
    case K_NARY:
        op_nary_bwd(e, I);
        break;
    case K_WIN: {
        const float* u = slot(e, I.b_in0);
        float* gu = slot(e, I.g_in0);
        const int khi = (I.flags & F_UNB) ? -1 : I.b;
        const float padv = e.P->coef[I.coef];
        if (!is_smooth(I)) {
            int* js = (int*)S(e, 4);
            win_hard(e, u, S(e, 5), js, sg, I.a, khi, I.pad, padv, (VI*)S(e, 0), (VI*)S(e, 2));
            win_hard_adj(e, g, gu, js, (double*)S(e, 6));
            break;
        }
        if constexpr (FULL) if (I.flags & F_SOFT) {
            // d out_t / d u_j = p_j(t) (1 + k (u_j - out_t)), p_j(t) = 2^{z_j} / S0(t), k = sg beta:
            // gu_j = 2^{z_j} [(1 + k u_j) sum_t G_t / S0(t) - k sum_t G_t out_t / S0(t)]
            // over the t whose window holds j (transposed window sums)
            // A LAST pad adds, per output, np copies of u_{L-1}: p_v(t) np (1 + k (u_{L-1} - out_t)).
            const float bl = pbeta(e, I) * LOG2E, kap = sg * bl / LOG2E;
            const float* out = slot(e, I.b_out);
            const int n = L - I.a;
            SP* den = (SP*)S(e, 6);
            win_smooth_sum(e, u, den, sg * bl, I.a, khi, I.pad, padv, (SP*)S(e, 0), (SP*)S(e, 2));
            float lastpad = 0.f;
            const SP zv = sp_leaf(sg * bl * u[L - 1]);
            for (int t = e.tid; t < L; t += e.nt) {
                if (khi >= 0 && I.pad == PAD_LAST && t + khi > L - 1) {
                    const int np = min(khi - I.a + 1, t + khi - (L - 1));
                    const float pv = sp_ratio(zv, den[t]);
                    lastpad += g[t] * (float)np * pv * (1.f + kap * (u[L - 1] - out[t]));
                }
            }
            if (I.pad == PAD_LAST) lastpad = wg_sum(lastpad, e);
            SP* res = (SP*)S(e, 4);
            SP* res2 = (SP*)S(e, 10);
            win_smooth_adj_sum(
                e,
                [&](int t) {
                    const SP d = den[t];
                    return t < n ? SP{g[t] / d.s, -d.r} : sp_zero();
                },
                (SP*)S(e, 0), (SP*)S(e, 2), res, I.a, khi, n);
            win_smooth_adj_sum(
                e,
                [&](int t) {
                    const SP d = den[t];
                    return t < n ? SP{g[t] * out[t] / d.s, -d.r} : sp_zero();
                },
                (SP*)S(e, 0), (SP*)S(e, 2), res2, I.a, khi, n);
            for (int j = e.tid; j < L; j += e.nt) {
                const SP r1 = res[j], r2 = res2[j];
                const SP c = sp_add(SP{r1.s * (1.f + kap * u[j]), r1.r}, SP{-kap * r2.s, r2.r});
                float vj = sp_times_exp2(c, sg * bl * u[j]);
                if (j == L - 1) vj += lastpad;
                gu[j] = vj;
            }
            break;
        }
        const float bl = pbeta(e, I) * LOG2E;
        const float* out = slot(e, I.b_out);
        const bool unb = khi < 0;
        const int n = L - I.a;
        float lastpad = 0.f;
        if (!unb && I.pad == PAD_LAST) {
            for (int t = e.tid; t < L; t += e.nt)
                if (t + khi > L - 1) {
                    const int np = min(khi - I.a + 1, t + khi - (L - 1));
                    const SP q = sp_leaf(-sg * bl * out[t]);
                    lastpad += (float)np * sp_times_exp2(SP{g[t] * q.s, q.r}, sg * bl * u[L - 1]);
                }
            lastpad = wg_sum(lastpad, e);
        }
        SP* res = (SP*)S(e, 4);
        win_smooth_adj_sum(
            e,
            [&](int t) {
                const SP q = sp_leaf(-sg * bl * out[t]);
                return t < n ? SP{g[t] * q.s, q.r} : sp_zero();
            },
            (SP*)S(e, 0), (SP*)S(e, 2), res, I.a, khi, n);
        for (int j = e.tid; j < L; j += e.nt) {
            float v = sp_times_exp2(res[j], sg * bl * u[j]);
            if (j == L - 1) v += lastpad;
            gu[j] = v;
        }
        break;
    }
    case K_MASK: {
        if constexpr (FULL) {
        const float* u = slot(e, I.b_in0);
        float* gu = slot(e, I.g_in0);
        float* w = S(e, 6);
        float* dwa = S(e, 7);
        float* dwb = S(e, 8);
        MaskInfo mi = mask_weights(e, I, w, dwa, dwb);
        const bool padm = I.pad != PAD_NEUTRAL && !(I.flags & F_MASK_UNB);
        MaskTail mt{INT_MAX, -1, 0.0, 0.0, 0.0};
        if (padm) mt = mask_tail(e, I, true);
        const int kall = mi.any ? mi.klo : mt.lo;            // whole support
        const int khi_all = mt.hi >= 0 ? mt.hi : mi.khi;
        const bool anyk = mi.any || mt.hi >= 0;
        if (!is_smooth(I) || !anyk) {
            if (!anyk) {
                for (int j = e.tid; j < L; j += e.nt) gu[j] = 0.f;
            } else {
                const int khi = ((I.flags & F_MASK_UNB) && khi_all == L - 1) ? -1 : khi_all;
                int* js = (int*)S(e, 4);
                win_hard(e, u, S(e, 5), js, sg, kall, khi, padm ? I.pad : PAD_NEUTRAL, mask_padv(I),
                         (VI*)S(e, 0), (VI*)S(e, 2));
                win_hard_adj(e, g, gu, js, (double*)S(e, 10));
            }
            if (I.mslot >= 0 && e.tid == 0) { mask_part[2 * I.mslot] = 0.f; mask_part[2 * I.mslot + 1] = 0.f; }
            break;
        }
        const float bl = pbeta(e, I) * LOG2E;
        const float* out = slot(e, I.b_out);
        const bool core = mi.clo <= mi.chi;
        SP* hb = (SP*)S(e, 9);      // adjoint terms
        SP* E = (SP*)S(e, 11);
        const int nvalid = mi.any ? L - mi.klo : 0;
        float pa = 0.f, pb = 0.f;
        float lastpad = 0.f;
        if (padm) {
            // pad copies: out_t gains TW_t 2^{z_v}; its share of the sum is
            // f_t = TW_t 2^{z_v - O_t}, giving d/du_{L-1} (LAST) = f_t and
            // d/da = TWa_t / TW_t * f_t / beta (d/db alike)
            float* TW = S(e, 13);
            float* TWa = S(e, 14);
            float* TWb = S(e, 15);
            tail_weights(w, TW, L, mt.s, e);
            tail_weights(dwa, TWa, L, mt.sa, e);
            tail_weights(dwb, TWb, L, mt.sb, e);
            const float zv = sg * bl * (I.pad == PAD_LAST ? u[L - 1] : mask_padv(I));
            const float ib0 = sg / pbeta(e, I);
            for (int t = e.tid; t < L; t += e.nt) {
                if (t + khi_all <= L - 1 || !(TW[t] > 0.f)) continue;
                const float f = exp2f(zv - sg * bl * out[t] + log2f(TW[t]));
                const float gf = g[t] * f;
                pa += ib0 * gf * (TWa[t] / TW[t]);
                pb += ib0 * gf * (TWb[t] / TW[t]);
                lastpad += gf;
            }
            if (I.pad == PAD_LAST) lastpad = wg_sum(lastpad, e);
        }
        for (int t = e.tid; t < L; t += e.nt) {
            E[t] = sp_leaf(sg * bl * u[t]);
            SP hv = sp_zero();
            if (t < nvalid) {
                SP q = sp_leaf(-sg * bl * out[t]);
                hv = SP{g[t] * q.s, q.r};
            }
            hb[t] = hv;
        }
        __syncthreads();
        // d/da, d/db: per t, sum over the support bands of dw_k 2^{z_{t+k} - O_t}
        for (int t = e.tid; t < nvalid; t += e.nt) {
            SPD aa{0.0, SP_NEG}, ab{0.0, SP_NEG};
            const int b0 = mi.klo, b1 = core ? mi.clo - 1 : mi.khi;
            for (int k = b0; k <= b1 && t + k < L; ++k) {
                aa = spd_add(aa, SP{dwa[k] * E[t + k].s, E[t + k].r});
                ab = spd_add(ab, SP{dwb[k] * E[t + k].s, E[t + k].r});
            }
            if (core)
                for (int k = mi.chi + 1; k <= mi.khi && t + k < L; ++k) {
                    aa = spd_add(aa, SP{dwa[k] * E[t + k].s, E[t + k].r});
                    ab = spd_add(ab, SP{dwb[k] * E[t + k].s, E[t + k].r});
                }
            const float O = sg * bl * out[t];
            const float ib = sg * g[t] / pbeta(e, I);
            pa += ib * sp_times_exp2(spd_to_sp(aa), -O);
            pb += ib * sp_times_exp2(spd_to_sp(ab), -O);
        }
        pa = wg_sum(pa, e);
        pb = wg_sum(pb, e);
        if (I.mslot >= 0 && e.tid == 0) { mask_part[2 * I.mslot] = pa; mask_part[2 * I.mslot + 1] = pb; }
        // dx: core via the transposed van Herk sum, bands term by term
        SP* res = (SP*)S(e, 4);
        if (core) {
            const int khi = ((I.flags & F_MASK_UNB) && mi.chi == L - 1) ? -1 : mi.chi;
            win_smooth_adj_sum(e, [&](int t) { return hb[t]; }, (SP*)S(e, 0), (SP*)S(e, 2), res, mi.clo, khi, nvalid);
        }
        for (int j = e.tid; j < L; j += e.nt) {
            // signed adjoint terms: accumulate with a double mantissa
            SPD a{0.0, SP_NEG};
            if (core) a = spd_add(a, SP{res[j].s * mi.wc, res[j].r});
            const int b0 = mi.klo, b1 = core ? mi.clo - 1 : mi.khi;
            for (int k = b0; k <= b1 && j - k >= 0; ++k) a = spd_add(a, SP{w[k] * hb[j - k].s, hb[j - k].r});
            if (core)
                for (int k = mi.chi + 1; k <= mi.khi && j - k >= 0; ++k)
                    a = spd_add(a, SP{w[k] * hb[j - k].s, hb[j - k].r});
            float v = sp_times_exp2(spd_to_sp(a), sg * bl * u[j]);
            if (padm && I.pad == PAD_LAST && j == L - 1) v += lastpad;
            gu[j] = v;
        }
        }
        break;
    }
    case K_UNTIL: {
        const float* phi = slot(e, I.b_in0);
        const float* psi = slot(e, I.b_in1);
        float* gphi = slot(e, I.g_in0);
        float* gpsi = slot(e, I.g_in1);
        for (int t = e.tid; t < L; t += e.nt) { gphi[t] = 0.f; gpsi[t] = 0.f; }
        __syncthreads();
        int ua = I.a, ub = I.b;
        const float *w = nullptr, *dwa = nullptr, *dwb = nullptr;
        bool none = false;
        if constexpr (FULL) if (I.mask >= 0) {
            float* wt = S(e, 4);
            float* wa = S(e, 5);
            float* wb = S(e, 6);
            const MaskInfo mi = mask_weights(e, I, wt, wa, wb);
            none = !mi.any;
            ua = mi.klo;
            ub = mi.khi;
            w = wt;
            dwa = wa;
            dwb = wb;
        }
        float pa = 0.f, pb = 0.f;
        if (none) {
            // empty support: constant output
        } else if (!is_smooth(I)) {
            if (ub < 0 && I.mask < 0) until_hard_unb(e, ua, phi, psi, nullptr, g, gphi, gpsi);
            else until_hard(e, ua, ub, phi, psi, nullptr, g, gphi, gpsi, (int*)S(e, 0));
        } else if constexpr (FULL) {
            const float bl = pbeta(e, I) * LOG2E;
            const int cku = I.mask >= 0 ? UCK_UNIT_MASK : UCK_UNIT;
            int M;
            if (until_ref(phi, psi, L, bl, e, M)) {
                const double* zs = (const double*)slot(e, I.coef);
                if (!w) {
                    until_smooth_adj_d(e, ua, ub, phi, psi, zs, g, gphi, gpsi, bl, M);
                } else {
                    double* Ep = (double*)S(e, 0);
                    double* Eq = (double*)S(e, 2);
                    until_terms(phi, psi, L, bl, M, Ep, Eq, e.nt, e.tid);
                    until_adj_w(e, ua, ub, w, dwa, dwb, Ep, Eq, zs, g, gphi, gpsi, (double*)S(e, cku),
                                until_cks(ub, L, UCK), pa, pb);
                }
            } else {
                SP* Ephi = (SP*)S(e, 0);
                SP* Epsi = (SP*)S(e, 2);
                for (int j = e.tid; j < L; j += e.nt) {
                    Ephi[j] = sp_leaf(-bl * phi[j]);
                    Epsi[j] = sp_leaf(-bl * psi[j]);
                }
                __syncthreads();
                until_smooth_adj(e, ua, ub, w, dwa, dwb, Ephi, Epsi, g, gphi, gpsi, (SP*)S(e, cku),
                                 until_cks(ub, L, UCK_SP), pa, pb);
            }
        }
        if (I.mslot >= 0) {
            // d out / d w_i = Y_i / (beta Z); zero for the hard form
            const float ib = is_smooth(I) ? 1.f / pbeta(e, I) : 0.f;
            const float sa = wg_sum(pa * ib, e);
            const float sb = wg_sum(pb * ib, e);
            if (e.tid == 0) { mask_part[2 * I.mslot] = sa; mask_part[2 * I.mslot + 1] = sb; }
        }
        break;
    }
    default:
        break;
    }
}

// Instructions whose thread for timestep t reads only what that thread wrote
// (every pointwise loop maps t to thread t mod blockDim) need no barrier
// between them; the others read and write across threads.
DEV bool crosses_threads(const Instr& I) { return I.kind == K_WIN || I.kind == K_MASK || I.kind == K_UNTIL; }

// ------------------------------------------------------------------ kernels

struct MaskTab;

DEV bool next_item(const KArgs& ka, Shared& sh, int64_t& item, bool first, int64_t B)
{
    if (ka.scan) {
        // the rows blockIdx.x + i gridDim.x whose flag is set, in order of i
        // (the flags of up to ka.nt rows are read at once)
        __syncthreads();
        const int64_t nrow = B > (int64_t)blockIdx.x ? (B - 1 - (int64_t)blockIdx.x) / gridDim.x + 1 : 0;
        for (int64_t i0 = first ? 0 : (int64_t)sh.scan_pos; i0 < nrow; i0 += ka.nt) {
            if (threadIdx.x == 0) sh.scan_min = INT_MAX;
            __syncthreads();
            const int64_t i = i0 + threadIdx.x;
            if (i < nrow && ka.scan[blockIdx.x + i * gridDim.x] != 0) atomicMin(&sh.scan_min, (int)i);
            __syncthreads();
            const int f = sh.scan_min;
            __syncthreads();
            if (f != INT_MAX) {
                item = (int64_t)blockIdx.x + (int64_t)f * gridDim.x;
                if (threadIdx.x == 0) sh.scan_pos = f + 1;
                return true;
            }
        }
        return false;
    }
    if (!ka.persistent) {
        item = blockIdx.x;
        return first;
    }
    __syncthreads();
    if (threadIdx.x == 0) sh.ints[7] = atomicAdd(ka.counter, 1);
    __syncthreads();
    item = sh.ints[7];
    return true;
}

// the only trajectory's mask partials (written by this thread) are the
// parameter gradients: no reduction launch
DEV void gp_from_partials(const DevPlan& P, const float* mp, float* gp)
{
    for (int p = 0; p < P.n_params; ++p) {
        float s = 0.f;
        for (int q = 0; q < 2 * P.n_masks; ++q)
            if (P.mask_param[q >> 1] + (q & 1) == p) s += mp[q];
        gp[p] = s;
    }
}

// One word of every line of the plan that the program uses, requested at
// once: the argument segment lies in host memory, and a line fetched when an
// instruction is reached costs the program 0.5 to 1 us each time.
DEV void plan_touch(const DevPlan* P)
{
    const int* w = (const int*)P;
    constexpr int PR = offsetof(DevPlan, pred) / 4, I0 = offsetof(DevPlan, ins) / 4, C0 = offsetof(DevPlan, coef) / 4;
    int a = 0;
#pragma unroll
    for (int i = 0; i < PR + 32; i += 16) a |= w[i];          // header, the first 16 predicates
#pragma unroll
    for (int i = 0; i < 176; i += 16) a |= w[I0 + i];         // the first 16 instructions
#pragma unroll
    for (int i = 0; i < 64; i += 16) a |= w[C0 + i];
    const int n = P->n_ins * (int)sizeof(Instr) / 4;
    for (int i = 176; i < n; i += 16) a |= w[I0 + i];
    asm volatile("" ::"s"(a));
}

// GLOBAL: the slots lie in the workspace instead of LDS (two kernels, so that
// every slot access of the LDS one is an LDS instruction, not a flat one).
// FULL = false: for plans of predicates, n-ary nodes, integer windows and hard
// Untils only (plan_is_plain).  The smooth Until and the masks set the full
// kernels' registers (256 in the backward: two waves per SIMD), which 1,000
// short trajectories of such a plan would wait for.
template <bool BWD, bool GLOBAL, bool FULL>
__global__ void __launch_bounds__(MAX_NT) stl_exec_kernel(DevPlan plan, Batch bt, KArgs ka)
{
    extern __shared__ __align__(16) float smem[];
    __shared__ Shared sh;
    // The plan is the first kernel argument, at offset 0 of the kernarg
    // segment: read it there.  (Taking the address of the by-value parameter
    // lets the compiler copy all of it into per-lane private memory, which it
    // does once the kernel body grows past some size.)
    const DevPlan* P = (const DevPlan*)__builtin_amdgcn_kernarg_segment_ptr();
    (void)plan;
    // A fix-up launch usually finds no flag set: every wave reads this
    // work-group's flags by itself and leaves without a barrier (no thread of
    // the launch writes them).  Up to 256 rows of a work-group, whose loads are
    // in flight together; beyond, next_item's reads of ka.nt rows at a time
    // take fewer turns.
    if (ka.scan) {
        const int64_t nrow = bt.B > (int64_t)blockIdx.x ? (bt.B - 1 - (int64_t)blockIdx.x) / gridDim.x + 1 : 0;
        if (nrow <= 256 && !(BWD && ka.gp_zero)) {
            int f = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = (int)(threadIdx.x & 63) + 64 * q;
                if (i < nrow) f |= ka.scan[blockIdx.x + (int64_t)i * gridDim.x];
            }
            if (__ballot(f != 0) == 0) return;
            plan_touch(P);
        }
    } else plan_touch(P);
    float* arena = GLOBAL ? ka.garena + (size_t)blockIdx.x * ka.arena_floats : smem;
    const int nslots = BWD ? P->n_slots_bwd : P->n_slots_fwd;
    const int Lc = bt.Lcap;
    int64_t item = 0;
    bool first = true;
    // no mask bound to differentiate: the parameter gradients are 0
    if (BWD && ka.gp_zero && blockIdx.x == 0)
        for (int q = threadIdx.x; q < P->n_params; q += ka.nt) ka.gp_zero[q] = 0.f;
    // an empty fix-up list: nothing to do and no counter to clear
    if (ka.list_mode && *ka.list_count <= 0) return;
    while (next_item(ka, sh, item, first, bt.B)) {
        first = false;
        const int64_t nitems = ka.list_mode ? min(max((int64_t)*ka.list_count, (int64_t)0), bt.B) : bt.B;
        if (item >= nitems) break;
        const int64_t b = ka.list_mode ? (int64_t)ka.list[item] : (bt.order ? (int64_t)bt.order[item] : item);
        const int64_t off = bt.offsets ? bt.offsets[b] : b * bt.T;
        const int64_t len = bt.offsets ? bt.offsets[b + 1] - off : bt.T;
        if (!BWD && ka.saved_none && threadIdx.x == 0) ka.saved_none[b] = 0;
        if (len <= 0) {
            // an empty trajectory adds nothing to d/da, d/db: its partials
            // are still read by the reduction
            if (BWD)
                for (int q = threadIdx.x; q < ka.part_stride * P->n_masks * 2; q += ka.nt)
                    ka.mask_part[b * ka.part_stride * P->n_masks * 2 + q] = 0.f;
            continue;
        }
        if (len > Lc) {
            // trajectory longer than the launch's capacity: report NaN
            for (int64_t t = threadIdx.x; t < len; t += ka.nt) {
                if (!BWD) ka.root[off + t] = NAN;
                else for (int d = 0; d < bt.D; ++d) ka.dx[(off + t) * bt.D + d] = NAN;
            }
            if (BWD)
                for (int q = threadIdx.x; q < ka.part_stride * P->n_masks * 2; q += ka.nt)
                    ka.mask_part[b * ka.part_stride * P->n_masks * 2 + q] = NAN;
            continue;
        }
        Env e;
        e.P = P;
        e.x = bt.x + off * bt.D;
        e.params = ka.params;
        e.L = (int)len;
        e.Lc = Lc;
        e.D = bt.D;
        e.arena = arena;
        e.scr = arena + (size_t)nslots * Lc;
        e.tile = GLOBAL ? ka.tile : 0;
        e.lds = GLOBAL ? smem : smem + ka.arena_floats;
        e.sh = &sh;
        e.nt = ka.nt;
        e.tid = exec_tid();
        op_preds(e, BWD);
        for (int k = P->n_pred; k < P->n_ins; ++k) {
            const Instr I = load_words(&P->ins[k]);
            const bool x = crosses_threads(I);
            if (x) __syncthreads();
            e.tid = exec_tid();
            exec_fwd<FULL>(e, I, BWD);
            if (x) __syncthreads();
        }
        if (!BWD) {
            const float* r = slot(e, P->ins[P->root].f_out);
            for (int t = threadIdx.x; t < e.L; t += ka.nt) ka.root[off + t] = r[t];
            if (ka.nodes) {
                // every node trace (debug): rerun with all slots kept is not
                // needed because the forward map keeps node outputs until
                // overwritten; the host gives every node its own slot when
                // traces are requested.
                // [n_nodes][N_total]: a ragged batch's N_total is offsets[B], read
                // here on the device so the host never waits for it
                const int64_t ntot = bt.offsets ? bt.offsets[bt.B] : ka.n_total;
                for (int k = 0; k < P->n_ins; ++k) {
                    const Instr& I = P->ins[k];
                    if (I.node < 0) continue;
                    const float* s = slot(e, I.f_out);
                    for (int t = threadIdx.x; t < e.L; t += ka.nt)
                        ka.nodes[(int64_t)I.node * ntot + off + t] = s[t];
                }
            }
            __syncthreads();
        } else {
            float* gr = slot(e, P->ins[P->root].g_out);
            for (int t = threadIdx.x; t < e.L; t += ka.nt) gr[t] = ka.G[off + t];
            // one partial row per trajectory; with part_stride > 1 (rows per
            // chunk of the matrix-core path) the trajectory's other rows are cleared
            float* mp = ka.mask_part + b * ka.part_stride * P->n_masks * 2;
            for (int q = threadIdx.x; q < (ka.part_stride - 1) * P->n_masks * 2; q += ka.nt)
                mp[P->n_masks * 2 + q] = 0.f;
            for (int k = P->n_ins - 1; k >= P->n_pred; --k) {
                const Instr I = load_words(&P->ins[k]);
                const bool x = crosses_threads(I);
                if (x) __syncthreads();
                e.tid = exec_tid();
                exec_adj<FULL>(e, I, mp);
                if (x) __syncthreads();
            }
            e.tid = exec_tid();
            op_dx(e, ka.dx + off * bt.D);
            if (FULL && ka.gp_one && e.tid == 0) gp_from_partials(*P, mp, ka.gp_one);
            __syncthreads();
        }
    }
    if (ka.list_mode) {
        // the last work-group out clears the item counter, the list count and
        // this ticket, so that the next call through the same counters starts
        // from zero without a clearing kernel
        __syncthreads();
        if (threadIdx.x == 0 && atomicAdd(ka.counter + 2, 1) == (int)gridDim.x - 1) {
            ka.counter[0] = 0;
            ka.counter[1] = 0;
            ka.counter[2] = 0;
        }
    }
}

}  // namespace stlmi
