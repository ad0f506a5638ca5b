// Interval-vectorised evaluation (Sec. VI, after the smooth-mask equation):
// the robustness at t = 0 of one masked Always / Eventually for many
// (a, b) interval values at once, and its derivatives in a and b.
//
// One work-group takes 256 intervals (one per thread) and a group of up to
// IV_TB trajectories.  With the masking form each interval is an independent
// weighted reduction over a trajectory; the weights depend on the interval
// only, so a thread evaluates w_k, dw_k/da, dw_k/db once per offset and
// applies them to every trajectory of the group, whose terms
// E_j = 2^{z_j - R} (FP64, R the trajectory's largest exponent, as in the
// fused kernels) sit in LDS.
#pragma once
#include <float.h>

namespace stlmi {

constexpr int IV_NT = 256;
constexpr int IV_MAXT = 4096;
constexpr int IV_TB = 8;          // trajectories per work-group (IV_TB * T <= IV_MAXT)

struct IntervalArgs {
    const float* x;
    const float* a;
    const float* b;
    float* rho;
    float* ga;
    float* gb;
    int64_t B, N;
    int T, D, tb;       // tb: trajectories per work-group
    int op_sg;          // +1 Eventually (max), -1 Always (min)
    int smooth;
    float beta, mc, meps, c, rho_pad;
    float w[16];
};

// offsets outside [lo, hi] have w_k <= 0 for eps > 0: sig(c(k-a)) < eps below
// a + ln(eps)/c, and sig(c(k-b)) > 1 - eps above b - ln(eps)/c (one step of
// margin for rounding); eps = 0 leaves every offset
DEV void iv_range(float a, float b, float c, float eps, int T, int& lo, int& hi)
{
    lo = 0;
    hi = T - 1;
    if (eps > 0.f) {
        const float r = logf(eps) / c;                 // < 0
        const float fl = floorf(a + r) - 1.f, fh = ceilf(b - r) + 1.f;
        lo = fl > 0.f ? (fl < (float)T ? (int)fl : T) : 0;
        hi = fh < (float)(T - 1) ? (fh > -1.f ? (int)fh : -1) : T - 1;
    }
}

// smooth value and derivatives of one interval on one trajectory, summed
// against the interval's own largest exponent (when every support term
// underflows against the trajectory's)
DEV void iv_own_ref(const MaskP& mp, const float* U, int lo, int hi, float sg, float bl, float beta, float& rho,
                    float& ga, float& gb)
{
    int zm = INT_MIN;
    bool any = false;
    for (int k = lo; k <= hi; ++k)
        if (mask_wk(mp, k) > 0.f) {
            zm = max(zm, (int)ceilf(fminf(fmaxf(sg * bl * U[k], -1e9f), 1e9f)));
            any = true;
        }
    if (!any) return;
    double S = 0.0, Sa = 0.0, Sb = 0.0;
    for (int k = lo; k <= hi; ++k) {
        float da, db;
        const float w = mask_wk(mp, k, &da, &db);
        if (!(w > 0.f)) continue;
        const double e = exp2d_neg(sg * bl * U[k] - (float)zm);
        S = fma((double)w, e, S);
        Sa = fma((double)da, e, Sa);
        Sb = fma((double)db, e, Sb);
    }
    rho = sg * ((float)zm + log2d(S)) / bl;
    ga = (float)((double)(sg / beta) * (Sa / S));
    gb = (float)((double)(sg / beta) * (Sb / S));
}

template <int TB>
__global__ void __launch_bounds__(IV_NT) stl_interval_kernel(IntervalArgs A)
{
    __shared__ double E[IV_MAXT];     // [tb][T] terms
    __shared__ float U[IV_MAXT];      // [tb][T] predicate trace
    __shared__ int red[TB][IV_NT / 64];
    const int T = A.T, D = A.D, tb = A.tb;
    const float bl = A.beta * LOG2E, sg = (float)A.op_sg;
    const int64_t n = (int64_t)blockIdx.x * IV_NT + threadIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int64_t b0 = (int64_t)blockIdx.y * tb; b0 < A.B; b0 += (int64_t)gridDim.y * tb) {
        const int nb = (int)min<int64_t>(tb, A.B - b0);
        __syncthreads();                   // the previous group's terms are no longer read
        // predicate traces and each trajectory's reference exponent
        for (int t = 0; t < nb; ++t) {
            const float* xb = A.x + (b0 + t) * (int64_t)T * D;
            int zmax = INT_MIN;
            for (int j = threadIdx.x; j < T; j += IV_NT) {
                float u = 0.f;
                for (int d = 0; d < D; ++d) u = fmaf(A.w[d], xb[(int64_t)j * D + d], u);
                u -= A.c;
                U[t * T + j] = u;
                zmax = max(zmax, (int)ceilf(fminf(fmaxf(sg * bl * u, -1e9f), 1e9f)));
            }
            for (int d = 32; d > 0; d >>= 1) zmax = max(zmax, __shfl_xor(zmax, d));
            if (lane == 0) red[t][wv] = zmax;
        }
        __syncthreads();
        int R[TB];
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            int r = INT_MIN;
            if (t < nb)
                for (int k = 0; k < IV_NT / 64; ++k) r = max(r, red[t][k]);
            R[t] = r;
        }
        if (A.smooth)
            for (int i = threadIdx.x; i < nb * T; i += IV_NT) {
                int r = R[0];
#pragma unroll
                for (int t = 1; t < TB; ++t) r = i / T == t ? R[t] : r;
                E[i] = exp2d_neg(sg * bl * U[i] - (float)r);
            }
        __syncthreads();
        if (n >= A.N) continue;
        MaskP mp;
        mp.a = A.a[n];
        mp.b = A.b[n];
        mp.c = A.mc;
        mp.eps = A.meps;
        mp.unb = false;
        mp.band = 1.f - expf(-mp.c * (mp.b - mp.a));
        int lo, hi;
        iv_range(mp.a, mp.b, mp.c, mp.eps, T, lo, hi);
        float rho[TB], ga[TB], gb[TB];
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            rho[t] = -sg * A.rho_pad;
            ga[t] = 0.f;
            gb[t] = 0.f;
        }
        if (!A.smooth) {
            // max (Eventually) / min (Always) over the support
            bool any = false;
            float best[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t) best[t] = 0.f;
            for (int k = lo; k <= hi; ++k) {
                if (!(mask_wk(mp, k) > 0.f)) continue;
#pragma unroll
                for (int t = 0; t < TB; ++t) {
                    const float v = t < nb ? sg * U[t * T + k] : 0.f;
                    best[t] = (!any || v > best[t]) ? v : best[t];
                }
                any = true;
            }
            if (any)
#pragma unroll
                for (int t = 0; t < TB; ++t) rho[t] = sg * best[t];
        } else {
            double S[TB], Sa[TB], Sb[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t) S[t] = Sa[t] = Sb[t] = 0.0;
            bool pos = false;                 // some offset has a positive weight
            for (int k = lo; k <= hi; ++k) {
                float da, db;
                const float w = mask_wk(mp, k, &da, &db);
                if (!(w > 0.f)) continue;
                pos = true;
#pragma unroll
                for (int t = 0; t < TB; ++t) {
                    const double e = t < nb ? E[t * T + k] : 0.0;
                    S[t] = fma((double)w, e, S[t]);
                    Sa[t] = fma((double)da, e, Sa[t]);
                    Sb[t] = fma((double)db, e, Sb[t]);
                }
            }
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                if (t >= nb) continue;
                if (S[t] > 0.0) {
                    rho[t] = sg * ((float)R[t] + log2d(S[t])) / bl;
                    const double iS = (double)(sg / A.beta) / S[t];   // one division for both ratios
                    ga[t] = (float)(iS * Sa[t]);
                    gb[t] = (float)(iS * Sb[t]);
                } else if (pos) {
                    iv_own_ref(mp, U + t * T, lo, hi, sg, bl, A.beta, rho[t], ga[t], gb[t]);
                }
            }
        }
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            if (t >= nb) continue;
            const int64_t o = (b0 + t) * A.N + n;
            A.rho[o] = rho[t];
            if (A.ga) {
                A.ga[o] = ga[t];
                A.gb[o] = gb[t];
            }
        }
    }
}

// Smooth sweep of one or two trajectories: with one thread per interval the
// launch holds too few waves to cover the latency of each thread's serial
// walk over its offsets, so IVS_LPI consecutive lanes share an interval (lane
// r takes offsets lo + r, lo + r + IVS_LPI, ...) and add their partial sums
// with lane exchanges; the first lane of the group writes the outputs.
constexpr int IVS_LPI = 4;

__global__ void __launch_bounds__(IV_NT) stl_interval_split_kernel(IntervalArgs A)
{
    __shared__ double E[IV_MAXT];
    __shared__ float U[IV_MAXT];
    __shared__ int red[IV_NT / 64];
    const int T = A.T, D = A.D;
    const float bl = A.beta * LOG2E, sg = (float)A.op_sg;
    const int64_t gi = (int64_t)blockIdx.x * IV_NT + threadIdx.x;
    const int64_t n = gi / IVS_LPI;
    const int r = (int)(gi % IVS_LPI);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool nok = n < A.N;
    MaskP mp;
    mp.a = nok ? A.a[n] : 0.f;
    mp.b = nok ? A.b[n] : 1.f;
    mp.c = A.mc;
    mp.eps = A.meps;
    mp.unb = false;
    mp.band = 1.f - expf(-mp.c * (mp.b - mp.a));
    int lo, hi;
    iv_range(mp.a, mp.b, mp.c, mp.eps, T, lo, hi);
    for (int64_t b = blockIdx.y; b < A.B; b += gridDim.y) {
        __syncthreads();                   // the previous trajectory's terms are no longer read
        const float* xb = A.x + b * (int64_t)T * D;
        int zmax = INT_MIN;
        for (int j = threadIdx.x; j < T; j += IV_NT) {
            float u = 0.f;
            for (int d = 0; d < D; ++d) u = fmaf(A.w[d], xb[(int64_t)j * D + d], u);
            u -= A.c;
            U[j] = u;
            zmax = max(zmax, (int)ceilf(fminf(fmaxf(sg * bl * u, -1e9f), 1e9f)));
        }
        for (int d = 32; d > 0; d >>= 1) zmax = max(zmax, __shfl_xor(zmax, d));
        if (lane == 0) red[wv] = zmax;
        __syncthreads();
        int R = INT_MIN;
        for (int k = 0; k < IV_NT / 64; ++k) R = max(R, red[k]);
        for (int j = threadIdx.x; j < T; j += IV_NT) E[j] = exp2d_neg(sg * bl * U[j] - (float)R);
        __syncthreads();
        double S = 0.0, Sa = 0.0, Sb = 0.0;
        int pos = 0;
        if (nok)
            for (int k = lo + r; k <= hi; k += IVS_LPI) {
                float da, db;
                const float w = mask_wk(mp, k, &da, &db);
                if (!(w > 0.f)) continue;
                pos = 1;
                const double e = E[k];
                S = fma((double)w, e, S);
                Sa = fma((double)da, e, Sa);
                Sb = fma((double)db, e, Sb);
            }
#pragma unroll
        for (int d = 1; d < IVS_LPI; d <<= 1) {
            S += __shfl_xor(S, d);
            Sa += __shfl_xor(Sa, d);
            Sb += __shfl_xor(Sb, d);
            pos |= __shfl_xor(pos, d);
        }
        if (!nok || r != 0) continue;
        float rho = -sg * A.rho_pad, ga = 0.f, gb = 0.f;
        if (S > 0.0) {
            rho = sg * ((float)R + log2d(S)) / bl;
            const double iS = (double)(sg / A.beta) / S;
            ga = (float)(iS * Sa);
            gb = (float)(iS * Sb);
        } else if (pos) {
            iv_own_ref(mp, U, lo, hi, sg, bl, A.beta, rho, ga, gb);
        }
        const int64_t o = b * A.N + n;
        A.rho[o] = rho;
        if (A.ga) {
            A.ga[o] = ga;
            A.gb[o] = gb;
        }
    }
}

// ------------------------------------------------------------------ batched sweep on the matrix cores

// For many trajectories the smooth sweep is a dense contraction: with
// E_bk = 2^{z_bk - R_b} (z = +-beta log2(e) u, R_b the trajectory's largest
// exponent), S_bn = sum_k w_nk E_bk and the same sums with dw/da, dw/db are
// three products of the [B, T] term matrix with the [T, N] weight matrices,
// which v_mfma_f32_16x16x4f32 computes 16 x 16 outputs at a time (K = 4 per
// instruction).  A wave owns NT tiles of 16 intervals: it evaluates their
// weights once, as A operands (lane l: interval n0 + 16j + l%16, offsets
// 4s + l/16), then walks tiles of 16 trajectories, whose terms are the B
// operands (lane l: trajectory b0 + l%16, offsets 4s + l/16) shared by all its
// interval tiles.  Result lane l, register q of tile j holds interval
// n0 + 16j + 4(l/16) + q, trajectory b0 + l%16: four consecutive outputs, one
// 16-byte store (with the operands the other way round they were four stores;
// rows gathered through LDS into 256-byte pieces took longer).  The terms are fp32 in (0, 1]; an output whose
// sum falls below 2^-100 (its support only reaches terms near or under the fp32
// range) is redone by iv_own_ref from the predicate trace kept in LDS.
// Bound by the 12 B written per output and the vector issue of the epilogue
// beside it: one log, one reciprocal with a correction step and two
// multiplications per output (through the library's general routines the
// epilogue took as long as the writes), without branches.  4,096 signals x
// 90,000 intervals of 20 samples without gradients: 982 -> 443 us.
// SW: the operands the other way round (register q: trajectory b0 + 4(l/16) + q,
// interval n0 + 16j + l%16): four 4-byte stores that cover 4 rows of 64 bytes
// each, instead of one that covers 16.  With three outputs of 1.5 GB each the
// rows in flight count for more than the stores.  With gradients, one set of
// outputs written again and again: 1,137 us before, 1,131 with SW, 1,170
// without; two sets in turn: 1,262, 1,197 and 1,160.  With two interval tiles
// (below about 3,000 signals) SW loses 2 to 6%.
constexpr int IVM_MAXT = 64;

typedef float iv_f4 __attribute__((ext_vector_type(4)));
typedef float iv_f4u __attribute__((ext_vector_type(4), aligned(4)));

// orders the LDS accesses of a wave's lanes on either side of it (a wave's LDS
// instructions execute in order: the compiler has to keep theirs)
DEV void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int KS, int NT, bool GRAD, bool SW>
__global__ void __launch_bounds__(IV_NT, 2) stl_interval_mfma_kernel(IntervalArgs A)
{
    __shared__ float Ush[IV_NT / 64][16 * 4 * KS];     // per wave: 16 predicate traces
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 15, row4 = lane >> 4;
    const int T = A.T, D = A.D;
    const float bl = A.beta * LOG2E, sg = (float)A.op_sg;
    const float sbl = sg * bl, ibl = 1.f / sbl, empty = -sg * A.rho_pad;      // (the sign goes with the quotient)
    const int64_t n0 = ((int64_t)blockIdx.x * (IV_NT / 64) + wv) * (16 * NT);
    auto params = [&](int64_t n) {
        MaskP mp;
        mp.a = n < A.N ? A.a[n] : 0.f;
        mp.b = n < A.N ? A.b[n] : 1.f;
        mp.c = A.mc;
        mp.eps = A.meps;
        mp.unb = false;
        mp.band = 1.f - expf(-mp.c * (mp.b - mp.a));
        return mp;
    };
    int pos[NT];                       // bit i: interval i of the tile has a positive weight
    float W[NT][KS], Wa[NT][GRAD ? KS : 1], Wb[NT][GRAD ? KS : 1];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int64_t n = n0 + 16 * j + col;
        const MaskP mp = params(n);
        int p = 0;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + row4;
            float da = 0.f, db = 0.f, w = 0.f;
            if (n < A.N && k < T) w = mask_wk(mp, k, GRAD ? &da : nullptr, &db);
            W[j][s] = w;
            if (GRAD) {
                Wa[j][s] = da;
                Wb[j][s] = db;
            }
            p |= w > 0.f;
        }
        // an interval whose support misses [0, T) has the empty-window value on
        // every trajectory: no sum and no fallback for it
        const unsigned long long m = __ballot(p != 0);
        pos[j] = (int)((m | m >> 16 | m >> 32 | m >> 48) & 0xffff) >> (SW ? col : 4 * row4);
    }
    float* Uw = Ush[wv];
    const float ib = sg / A.beta;
    for (int64_t b0 = (int64_t)blockIdx.y * 16; b0 < A.B; b0 += (int64_t)gridDim.y * 16) {
        const int64_t b = b0 + col;                   // this lane's trajectory
        const bool bok = b < A.B;
        const float* xb = A.x + (bok ? b : 0) * (int64_t)T * D;
        float z[KS];
        int zm = INT_MIN;
        wave_sync();                                  // the previous tile's traces are no longer read
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + row4;
            float u = 0.f;
            if (bok && k < T) {
                for (int d = 0; d < D; ++d) u = fmaf(A.w[d], xb[(int64_t)k * D + d], u);
                u -= A.c;
                zm = max(zm, (int)ceilf(fminf(fmaxf(sg * bl * u, -1e9f), 1e9f)));
            }
            z[s] = sg * bl * u;
            Uw[col * (4 * KS) + k] = u;               // read by this wave only
        }
        zm = max(zm, __shfl_xor(zm, 16));
        zm = max(zm, __shfl_xor(zm, 32));
        iv_f4 s0[NT], sa[NT], sb[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) s0[j] = sa[j] = sb[j] = iv_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = 4 * s + row4;
            const float e = (bok && k < T) ? exp2f(z[s] - (float)zm) : 0.f;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                s0[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(SW ? e : W[j][s], SW ? W[j][s] : e, s0[j], 0, 0, 0);
                if (GRAD) {
                    sa[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(SW ? e : Wa[j][s], SW ? Wa[j][s] : e, sa[j], 0, 0, 0);
                    sb[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(SW ? e : Wb[j][s], SW ? Wb[j][s] : e, sb[j], 0, 0, 0);
                }
            }
        }
        unsigned redo = 0;                 // outputs 4 j + q that need their own reference
        float fz[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) fz[q] = SW ? (float)__shfl(zm, 4 * row4 + q) : (float)zm;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int64_t n = n0 + 16 * j + (SW ? col : 4 * row4), o = (SW ? b0 + 4 * row4 : b) * A.N + n;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // (branch-free: a wave holds outputs with and without a support)
                const float S = s0[j][q];
                const bool ok = S >= 0x1p-100f;
                redo |= !ok && (pos[j] >> (SW ? 0 : q) & 1) ? 1u << (4 * j + q) : 0u;
                // quotients as estimate and one correction step (S and bl are normal): the value is the
                // correctly rounded quotient, the reciprocal differs from a division's in 3 of a million; the
                // estimate is kept finite, since S is infinite where a sample is and inf - inf would be the
                // correction
                const float v = fz[q] + lg2(S), r = __builtin_amdgcn_fmed3f(v * ibl, -FLT_MAX, FLT_MAX);
                s0[j][q] = ok ? fmaf(fmaf(-r, sbl, v), ibl, r) : empty;
                if (GRAD) {
                    float iS = __builtin_amdgcn_rcpf(S);
                    iS = fmaf(fmaf(-S, iS, 1.f), iS, iS) * ib;
                    sa[j][q] = ok ? sa[j][q] * iS : 0.f;
                    sb[j][q] = ok ? sb[j][q] * iS : 0.f;
                }
            }
            if (SW) {
                if (n < A.N) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (b0 + 4 * row4 + q < A.B) {
                            A.rho[o + q * A.N] = s0[j][q];
                            if (GRAD) {
                                A.ga[o + q * A.N] = sa[j][q];
                                A.gb[o + q * A.N] = sb[j][q];
                            }
                        }
                }
                continue;
            }
            if (!bok) continue;
            if (n + 4 <= A.N) {
                // (16-byte stores need the alignment of a float only: odd N, any buffers)
                *(iv_f4u*)(A.rho + o) = s0[j];
                if (GRAD) {
                    *(iv_f4u*)(A.ga + o) = sa[j];
                    *(iv_f4u*)(A.gb + o) = sb[j];
                }
            } else {
                for (int q = 0; q < 4; ++q)
                    if (n + q < A.N) {
                        A.rho[o + q] = s0[j][q];
                        if (GRAD) {
                            A.ga[o + q] = sa[j][q];
                            A.gb[o + q] = sb[j][q];
                        }
                    }
            }
        }
        if (!SW && !bok) redo = 0;
        wave_sync();                                  // traces visible to every lane of the wave
#pragma unroll 1
        while (redo) {
            const int i = __builtin_ctz(redo);
            redo &= redo - 1;
            const int64_t n = n0 + 16 * (i >> 2) + (SW ? col : 4 * row4 + (i & 3));
            const int bi = SW ? 4 * row4 + (i & 3) : col;
            if (n >= A.N || b0 + bi >= A.B) continue;
            const MaskP mp = params(n);
            int lo, hi;
            iv_range(mp.a, mp.b, mp.c, mp.eps, T, lo, hi);
            float rho = -sg * A.rho_pad, ga = 0.f, gb = 0.f;
            iv_own_ref(mp, Uw + bi * (4 * KS), lo, hi, sg, bl, A.beta, rho, ga, gb);
            A.rho[(b0 + bi) * A.N + n] = rho;
            if (GRAD) {
                A.ga[(b0 + bi) * A.N + n] = ga;
                A.gb[(b0 + bi) * A.N + n] = gb;
            }
        }
    }
}

template <int KS, int NT, bool SW = false>
static void launch_interval_mfma(const IntervalArgs& A, hipStream_t s)
{
    // 64 NT intervals per work-group; enough trajectory-tile groups for about 8192
    // work-groups, of the same number of tiles, and four tiles each while two work-groups
    // per compute unit remain: the weights are evaluated once per work-group, which
    // one or two tiles do not pay for (90,000 intervals x 250 signals, T = 20:
    // 145 us with one tile each, 80 now)
    const int64_t nx = (A.N + 64 * NT - 1) / (64 * NT), tiles = (A.B + 15) / 16;
    int64_t ny = std::max<int64_t>(1, std::min<int64_t>(tiles, std::min<int64_t>(65535, (8192 + nx - 1) / nx)));
    const int64_t per = std::max<int64_t>((tiles + ny - 1) / ny, std::min<int64_t>(4, nx * tiles / 512));
    ny = (tiles + per - 1) / per;
    const dim3 g((unsigned)nx, (unsigned)ny), blk(IV_NT);
    if (A.ga) hipLaunchKernelGGL((stl_interval_mfma_kernel<KS, NT, true, SW>), g, blk, 0, s, A);
    else hipLaunchKernelGGL((stl_interval_mfma_kernel<KS, NT, false, false>), g, blk, 0, s, A);
}

// ------------------------------------------------------------------ pSTL descent

// Gradient descent on the parametric-STL mining loss (Sec. VII-B)
//   L(a, b) = mean_i max(-rho_i, 0) + gamma (a - b),
//   rho_i = robustness at t = 0 of op_[aT, bT](w . x_i - c) with a smooth mask,
// over a = sig(p_a), b = sig(p_b) (fractions of the horizon), the mask
// steepness and beta annealed from (c0, beta0) to (c1, beta1) along a sigmoid
// schedule.  The whole loop runs in one work-group of 16 waves (a step is too
// short to be worth a grid-wide exchange): `lps` lanes share a signal and hold
// its predicate trace in registers, NR values each, through the descent; a step
// evaluates the mask weights once (fp64 in LDS), every signal's rho, d rho/da,
// d rho/db, and reduces the hinge gradient in a fixed order (DPP adds, then the
// waves' sums).  Wave 0 alone adds the sums, updates (p_a, p_b) and evaluates
// the weights: done by every wave they cost more issue slots than the terms.
// Two barriers per step.  The step is bound by this serial chain beside the
// terms' issue.  256 threads walking a signal each, with an fp64 exponent split
// per term and the update on one thread, took 8.75 us per step at 500 signals of
// 20 samples; now 2.6 us.
// REG = false: more signals than threads, the traces stay in LDS.
constexpr int PD_MAXBT = 12288;

struct DescentArgs {
    const float* x;
    float* p;            // [2] logits of (a, b), read and written
    float* loss;         // [steps] or NULL
    int B, T, D, steps, op_sg;
    float eps, c0, c1, beta0, beta1, lr, gamma, c;
    float w[16];
};

DEV float sched(int k, int steps, float lo, float hi)
{
    const float u = (float)k / (float)max(1, steps - 1) - 0.5f;
    return lo + (hi - lo) / (1.f + expf(-12.f * u));
}

constexpr int PD_NT = 1024;

// sum over the wave, in lane 63 (DPP adds in a fixed order)
DEV double wave_add63(double v)
{
    v += dpp8<0x111>(v);
    v += dpp8<0x112>(v);
    v += dpp8<0x114>(v);
    v += dpp8<0x118>(v);
    double o = dpp8<0x142>(v);
    if (threadIdx.x & 16) v += o;
    o = dpp8<0x143>(v);
    if (threadIdx.x & 32) v += o;
    return v;
}

// reduction over the lps lanes of a signal (every lane gets the result)
template <class T, class Op>
DEV T lps_reduce(T v, int lps, Op op)
{
    if (lps > 1) v = op(v, dpp8<0xB1>(v));          // lanes 1 apart
    if (lps > 2) v = op(v, dpp8<0x4E>(v));          // 2 apart
    if (lps > 4) v = op(v, dpp8<0x141>(v));         // the other quad of eight
    if (lps > 8) v = op(v, dpp8<0x140>(v));         // the other eight of the row
    if (lps > 16) v = op(v, __shfl_xor(v, 16));
    if (lps > 32) v = op(v, __shfl_xor(v, 32));
    return v;
}

struct OpMax {
    __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};

// A step takes a signal's terms in FP32 where none of them can leave the normal
// range: beta log2(e) times the trace's extent (and 2^-22 of its magnitude, so
// that every exponent is below 1e9) is at most PD_SPAN.  A wave with any other
// signal, non-finite samples included, takes FP64 terms with an exponent split.
constexpr float PD_SPAN = 120.f;

DEV void spread(float u, float& lo, float& hi, float& far)
{
    lo = fminf(lo, u);
    hi = fmaxf(hi, u);
    far = fmaxf(far, fabsf(u) < INFINITY ? fabsf(u) * 0x1p-22f : INFINITY);
}

template <int NR, bool REG>
__global__ void __launch_bounds__(PD_NT) stl_pstl_descent_kernel(DescentArgs A, int lps)
{
    __shared__ float U[REG ? 1 : PD_MAXBT];
    // offset j = r + lps q is entry [q][r]: the reads of a lane are a constant stride apart
    __shared__ double Wt[3][NR][REG ? 64 : 1];         // w_j, dw_j/da, dw_j/db for the current step
    __shared__ float Wm[NR][REG ? 64 : 1];             // 0 in the support {w > 0}, -inf outside
    __shared__ double red[3][PD_NT / 64];
    __shared__ float cb[2][2];                         // steepness and beta of the current and the next step
    const int B = A.B, T = A.T, D = A.D;
    const float sg = (float)A.op_sg;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = threadIdx.x & (lps - 1), sig0 = threadIdx.x / lps, nsig = PD_NT / lps;
    auto trace = [&](int i, int j) {
        const float* x = A.x + ((int64_t)i * T + j) * D;
        float u = 0.f;
        for (int d = 0; d < D; ++d) u = fmaf(A.w[d], x[d], u);
        return u - A.c;
    };
    float ur[NR], far = 0.f;
#pragma unroll
    for (int k = 0; k < NR; ++k) ur[k] = 0.f;
    if (REG) {
        float lo = INFINITY, hi = -INFINITY;
#pragma unroll
        for (int k = 0; k < NR; ++k)
            if (sig0 < B && r + lps * k < T) {
                ur[k] = sg * trace(sig0, r + lps * k);
                spread(ur[k], lo, hi, far);
            }
        far = lps_reduce(far, lps, OpMax());
        far = fmaxf(far, lps_reduce(hi, lps, OpMax()) + lps_reduce(-lo, lps, OpMax()));
    } else {
        for (int i = threadIdx.x; i < B * T; i += PD_NT) U[i] = sg * trace(i / T, i % T);
    }
    const double ToB = (double)T / B;
    float pa = A.p[0], pb = A.p[1];                    // (wave 0)
    auto schedule = [&](int k) {
        if (lane < 2) cb[k & 1][lane] = lane ? sched(k, A.steps, A.beta0, A.beta1) : sched(k, A.steps, A.c0, A.c1);
    };
    if (wv == PD_NT / 64 - 1) schedule(0);
    __syncthreads();
    if (!REG)
        for (int i = sig0; i < B; i += nsig) {             // (the farthest of this thread's signals)
            float lo = INFINITY, hi = -INFINITY;
            for (int j = 0; j < T; ++j) spread(U[i * T + j], lo, hi, far);
            far = fmaxf(far, hi - lo);
        }
    for (int k = 0; k < A.steps; ++k) {
        float af = 0.f, bf = 0.f;
        if (wv == 0) {
            af = 1.f / (1.f + expf(-pa));
            bf = 1.f / (1.f + expf(-pb));
            MaskP mp;
            mp.a = af * (float)T;
            mp.b = bf * (float)T;
            mp.c = cb[k & 1][0];
            mp.eps = A.eps;
            mp.unb = false;
            mp.band = 1.f - expf(-mp.c * (mp.b - mp.a));
            for (int j = lane; j < lps * NR; j += 64) {
                float da = 0.f, db = 0.f, w = 0.f;
                if (j < T) w = mask_wk(mp, j, &da, &db);
                const int q = j >> __builtin_ctz(lps), s = j & (lps - 1);
                Wt[0][q][s] = w;
                Wt[1][q][s] = da;
                Wt[2][q][s] = db;
                Wm[q][s] = w > 0.f ? 0.f : -INFINITY;
            }
        }
        __syncthreads();
        const float beta = cb[k & 1][1], bl = beta * LOG2E;
        if (wv == PD_NT / 64 - 1) schedule(k + 1);     // (a wave with few signals)
        double ha = 0.0, hb = 0.0, hl = 0.0;      // this thread's hinge sums
        auto signals = [&](auto wide) {
            constexpr bool WIDE = decltype(wide)::value;
            for (int i = sig0; i < B; i += nsig) {
                float u[NR], zm = -INFINITY;
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    u[q] = REG ? ur[q] : (q < T ? U[i * T + q] : 0.f);
                    if (!WIDE) zm = fmaxf(zm, fmaf(bl, u[q], Wm[q][r]));
                    else if (Wm[q][r] == 0.f) zm = fmaxf(zm, fminf(fmaxf(bl * u[q], -1e9f), 1e9f));
                }
                zm = lps_reduce(zm, lps, OpMax());
                const bool any = zm > -INFINITY;
                // reference: the largest exponent of the support; terms are 2^{z - R} (FP32: their exponents
                // outside the support do not matter, their weights are 0)
                const float R = ceilf(fmaxf(zm, -1e9f));
                float e[NR];
                double S = 0.0, Sa = 0.0, Sb = 0.0;
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    if (!WIDE) {
                        e[q] = ex2(fminf(fmaf(bl, u[q], -R), 0.f));
                        S = fma(Wt[0][q][r], (double)e[q], S);
                    } else if (Wm[q][r] == 0.f) {
                        const double t = exp2d_neg(bl * u[q] - R);
                        S = fma(Wt[0][q][r], t, S);
                        Sa = fma(Wt[1][q][r], t, Sa);
                        Sb = fma(Wt[2][q][r], t, Sb);
                    }
                }
                S = lps_reduce(S, lps, OpD());
                const float rho = any ? sg * (R + log2d(S)) / bl : -sg * 1e6f;
                const bool hinge = rho < 0.f;
                if (__ballot(hinge) == 0) continue;  // the gradients are those of the violated signals only
                if (!WIDE) {
#pragma unroll
                    for (int q = 0; q < NR; ++q) {
                        Sa = fma(Wt[1][q][r], (double)e[q], Sa);
                        Sb = fma(Wt[2][q][r], (double)e[q], Sb);
                    }
                }
                Sa = lps_reduce(Sa, lps, OpD());
                Sb = lps_reduce(Sb, lps, OpD());
                if (hinge && r == 0) {
                    if (any) {
                        const double iS = (double)(sg / beta) / S;   // one division for both ratios
                        ha -= (float)(iS * Sa);
                        hb -= (float)(iS * Sb);
                    }
                    hl -= rho;
                }
            }
        };
        if (__ballot(!(bl * far <= PD_SPAN)) == 0) signals(std::false_type());
        else signals(std::true_type());
        if (__ballot(hl != 0.0) != 0) {
            ha = wave_add63(ha);
            hb = wave_add63(hb);
            hl = wave_add63(hl);
        }
        if (lane == 63) {
            red[0][wv] = ha;
            red[1][wv] = hb;
            red[2][wv] = hl;
        }
        __syncthreads();
        if (wv == 0) {
            // (the rows of 16 lanes hold the same 16 values)
            auto total = [&](int q) {
                double v = red[q][lane & 15];
                v += dpp8<0x111>(v);
                v += dpp8<0x112>(v);
                v += dpp8<0x114>(v);
                v += dpp8<0x118>(v);
                return readlane8(v, 15);
            };
            const double sa = total(0), sb = total(1);
            // d L / d a_frac = T mean(-[rho < 0] d rho / d a_steps) + gamma (b: - gamma)
            const float dla = (float)(sa * ToB) + A.gamma, dlb = (float)(sb * ToB) - A.gamma;
            if (A.loss) {
                const double sl = total(2);
                if (lane == 0) A.loss[k] = (float)(sl / B) + A.gamma * (af - bf);
            }
            pa -= A.lr * dla * af * (1.f - af);
            pb -= A.lr * dlb * bf * (1.f - bf);
        }
    }
    if (threadIdx.x == 0) {
        A.p[0] = pa;
        A.p[1] = pb;
    }
}

int pstl_max_BT() { return PD_MAXBT; }

hipError_t launch_pstl_descent(const float* x, int B, int T, int D, const float* w, float c, int op_sg, float eps,
                               float c0, float c1, float beta0, float beta1, int steps, float lr, float gamma,
                               float* p, float* loss, hipStream_t s)
{
    DescentArgs A;
    A.x = x;
    A.p = p;
    A.loss = loss;
    A.B = B;
    A.T = T;
    A.D = D;
    A.steps = steps;
    A.op_sg = op_sg;
    A.eps = eps;
    A.c0 = c0;
    A.c1 = c1;
    A.beta0 = beta0;
    A.beta1 = beta1;
    A.lr = lr;
    A.gamma = gamma;
    A.c = c;
    for (int d = 0; d < 16; ++d) A.w[d] = d < D ? w[d] : 0.f;
    // as many lanes per signal (a power of two) as the work-group has for all of
    // them; then each lane holds at most 24 of B T <= 12288 values, and a step
    // takes all of the kernel's NR (500 signals of 20 samples, 10 values each, 200
    // steps: 590 us with NR = 10, 656 with 12)
    int lps = 1;
    while (lps < 64 && 2 * lps * B <= PD_NT && lps < T) lps *= 2;
    const int nr = (T + lps - 1) / lps;
    const dim3 g(1), blk(PD_NT);
    if (B > PD_NT) hipLaunchKernelGGL((stl_pstl_descent_kernel<12, false>), g, blk, 0, s, A, 1);
    else if (nr <= 4) hipLaunchKernelGGL((stl_pstl_descent_kernel<4, true>), g, blk, 0, s, A, lps);
    else if (nr <= 8) hipLaunchKernelGGL((stl_pstl_descent_kernel<8, true>), g, blk, 0, s, A, lps);
    else if (nr <= 10) hipLaunchKernelGGL((stl_pstl_descent_kernel<10, true>), g, blk, 0, s, A, lps);
    else if (nr <= 12) hipLaunchKernelGGL((stl_pstl_descent_kernel<12, true>), g, blk, 0, s, A, lps);
    else if (nr <= 16) hipLaunchKernelGGL((stl_pstl_descent_kernel<16, true>), g, blk, 0, s, A, lps);
    else if (nr <= 24) hipLaunchKernelGGL((stl_pstl_descent_kernel<24, true>), g, blk, 0, s, A, lps);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

int interval_max_T() { return IV_MAXT; }

hipError_t launch_interval_sweep(int op_sg, int smooth, float beta, float mc, float meps, int D, const float* w,
                                 float c, float rho_pad, const float* x, int64_t B, int T, const float* a,
                                 const float* b, int64_t N, float* rho, float* ga, float* gb, hipStream_t s)
{
    IntervalArgs A;
    A.x = x;
    A.a = a;
    A.b = b;
    A.rho = rho;
    A.ga = ga;
    A.gb = gb;
    A.B = B;
    A.N = N;
    A.T = T;
    A.D = D;
    const bool group = B > 2;             // one trajectory per work-group for tiny batches
    A.tb = group ? std::max(1, std::min(IV_TB, IV_MAXT / T)) : 1;
    A.op_sg = op_sg;
    A.smooth = smooth;
    A.beta = smooth ? beta : 1.f;
    A.mc = mc;
    A.meps = meps;
    A.c = c;
    A.rho_pad = rho_pad;
    for (int d = 0; d < 16; ++d) A.w[d] = d < D ? w[d] : 0.f;
    if (smooth && T <= IVM_MAXT && B >= 16) {
        // batched smooth sweep: matrix cores
        // (interval tiles per wave: as many as 256 registers hold)
        // four tiles of intervals per wave, and with gradients SW, once their
        // weights serve about eight tiles of signals (T = 20, 90,000 intervals: 4,096
        // signals 1,150 us against 1,233 with two; 1,000 signals 312 against 275)
        if (T <= 20 && (N + 255) / 256 * ((B + 15) / 16) >= 65536) launch_interval_mfma<5, 4, true>(A, s);
        else if (T <= 20) launch_interval_mfma<5, 2>(A, s);
        else if (T <= 32) launch_interval_mfma<8, 2>(A, s);
        else launch_interval_mfma<16, 2>(A, s);
        return hipGetLastError();
    }
    if (smooth && !group) {
        const dim3 g((unsigned)((N * IVS_LPI + IV_NT - 1) / IV_NT), (unsigned)std::min<int64_t>(B, 65535)),
            blk(IV_NT);
        hipLaunchKernelGGL(stl_interval_split_kernel, g, blk, 0, s, A);
        return hipGetLastError();
    }
    const int64_t groups = (B + A.tb - 1) / A.tb;
    const dim3 grid((unsigned)((N + IV_NT - 1) / IV_NT), (unsigned)std::min<int64_t>(groups, 65535)), block(IV_NT);
    if (group)
        hipLaunchKernelGGL(stl_interval_kernel<IV_TB>, grid, block, 0, s, A);
    else
        hipLaunchKernelGGL(stl_interval_kernel<1>, grid, block, 0, s, A);
    return hipGetLastError();
}

}  // namespace stlmi
