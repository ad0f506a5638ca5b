// Learned warm-start kernels for gfx950: BF16 matrix product on the matrix
// cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation) with a fused
// bias/ReLU epilogue, BF16 rounding, ReLU derivative mask, column sums, MSE
// gradient, Adam and the trajectory gradient-ascent step.  C ABI in
// include/stlmi_mlp.h and mlp_step.h.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>

#include <cstdarg>
#include <cstdio>
#include <string>

#include "mlp_step.h"

namespace stlmi_mlp {

#define DEV static __device__ __forceinline__

typedef float float4_t __attribute__((ext_vector_type(4)));

// float -> bf16, round to nearest even on the 16 dropped mantissa bits
DEV uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

DEV float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// 8 elements p[0], p[s], .., p[7 s] of which the first nvalid exist (zeros
// after them); one 16-byte load when vec (s = 1, nvalid = 8, aligned)
DEV void load8(const uint16_t* p, int64_t s, int nvalid, bool vec, uint16_t* v)
{
    if (vec) {
        const uint4 u = *(const uint4*)p;
        __builtin_memcpy(v, &u, 16);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = i < nvalid ? p[i * s] : (uint16_t)0;
    }
}

DEV bool al16(const void* p) { return (((uintptr_t)p) & 15) == 0; }

// 8 elements of one operand: rows r (of n_r), k-values kk .. along whichever of
// the two is contiguous (k_cont), zeros outside
DEV void stage_load(const uint16_t* P, int64_t sr, int64_t sk, bool k_cont, int r, int n_r, int k, int K, uint16_t* v)
{
    const int nv = k_cont ? (r < n_r ? max(0, min(8, K - k)) : 0) : (k < K ? max(0, min(8, n_r - r)) : 0);
    const uint16_t* p = P + (int64_t)(k_cont ? min(r, n_r - 1) : r) * sr + (int64_t)(k_cont ? k : min(k, K - 1)) * sk;
    const int64_t st = k_cont ? sk : sr;
    load8(p, st, nv, st == 1 && nv == 8 && al16(p), v);
}

// C[M,N] = act(A[M,K] B[K,N] + bias) on v_mfma_f32_16x16x32_bf16.  Work-group
// tile T x T, four waves of (T/2) x (T/2), K in stages of 2048 / T values: each
// of the 256 threads stages 8 consecutive elements of A and of B along the
// dimension that is contiguous in memory (one 16-byte load when aligned and in
// range); any strides work, transposed operands included.  LDS holds A as
// [m][k] and B as [n][k] (k contiguous), so each lane's MFMA operand (row or
// column l % 16, k = 8 (l / 16) .. + 7) is one 16-byte read.
// The network's products are small (1,024 x 256 x 256): with 64 x 64 tiles they
// fill a quarter of the chip, and a stage that loads, waits and multiplies is
// bound by the loads' latency.  So PD stages are in flight in registers, LDS is
// double-buffered (one barrier per stage), and the tiles are 32 x 32 where 64 x
// 64 ones would leave compute units with less than two work-groups (measured at
// 1,024 x 256 x 256: 18 us before; the accumulation order, K ascending in steps
// of 32, is the same for both).
template <int T>
__global__ void __launch_bounds__(256) gemm_bf16_kernel(const uint16_t* A, int64_t sam, int64_t sak,
                                                        const uint16_t* B, int64_t sbk, int64_t sbn, int M, int N,
                                                        int K, const float* bias, int relu, const uint16_t* pos,
                                                        int64_t ldpos, float* c32, int64_t ldc32, int beta32,
                                                        uint16_t* c16, int64_t ldc16)
{
    constexpr int TK = 2048 / T, LDK = TK + 8;   // (8 of pad: rows fall on distinct banks)
    constexpr int PD = 3, W = T / 32;
    __shared__ __align__(16) uint16_t As[2][T][LDK];
    __shared__ __align__(16) uint16_t Bs[2][T][LDK];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
    const int wm = (w >> 1) * (T / 2), wn = (w & 1) * (T / 2);
    const bool a_k = sak == 1;      // A rows contiguous in k (else chunks run along m)
    const bool b_k = sbk == 1;      // B columns contiguous in k (else chunks run along n)
    // this thread's chunk: (row, k) of the operand's tile
    const int kr = tid / (TK / 8), kk = tid % (TK / 8) * 8;          // contiguous in k
    const int tk = tid / (T / 8), tr = tid % (T / 8) * 8;            // contiguous in m or n
    const int ar = a_k ? kr : tr, ak = a_k ? kk : tk, br = b_k ? kr : tr, bk = b_k ? kk : tk;
    const int S = (K + TK - 1) / TK;
    float4_t acc[W][W];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    __align__(16) uint16_t va[PD][8], vb[PD][8];
#pragma unroll
    for (int d = 0; d < PD; ++d)
        if (d < S) {
            stage_load(A, sam, sak, a_k, m0 + ar, M, d * TK + ak, K, va[d]);
            stage_load(B, sbn, sbk, b_k, n0 + br, N, d * TK + bk, K, vb[d]);
        }
    for (int s0 = 0; s0 < S; s0 += PD) {
#pragma unroll
        for (int d = 0; d < PD; ++d) {
            const int st = s0 + d;
            if (st >= S) break;
            const int buf = st & 1;
            if (a_k) *(uint4*)&As[buf][ar][ak] = *(const uint4*)va[d];
            else
#pragma unroll
                for (int i = 0; i < 8; ++i) As[buf][ar + i][ak] = va[d][i];
            if (b_k) *(uint4*)&Bs[buf][br][bk] = *(const uint4*)vb[d];
            else
#pragma unroll
                for (int i = 0; i < 8; ++i) Bs[buf][br + i][bk] = vb[d][i];
            if (st + PD < S) {
                stage_load(A, sam, sak, a_k, m0 + ar, M, (st + PD) * TK + ak, K, va[d]);
                stage_load(B, sbn, sbk, b_k, n0 + br, N, (st + PD) * TK + bk, K, vb[d]);
            }
            // (a wave writes this buffer again two stages on, behind the next
            // barrier, which every wave reaches after its reads of it)
            __syncthreads();
#pragma unroll
            for (int k = 0; k < TK; k += 32) {
                const int kq = k + 8 * (lane >> 4);
                bf16x8_t a[W], b[W];
#pragma unroll
                for (int i = 0; i < W; ++i) a[i] = *(const bf16x8_t*)&As[buf][wm + 16 * i + (lane & 15)][kq];
#pragma unroll
                for (int j = 0; j < W; ++j) b[j] = *(const bf16x8_t*)&Bs[buf][wn + 16 * j + (lane & 15)][kq];
#pragma unroll
                for (int i = 0; i < W; ++i)
#pragma unroll
                    for (int j = 0; j < W; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = m0 + wm + 16 * i + 4 * (lane >> 4) + q;
                const int col = n0 + wn + 16 * j + (lane & 15);
                if (row >= M || col >= N) continue;
                float v = acc[i][j][q];
                if (bias) v += bias[col];
                if (relu) v = v > 0.f ? v : 0.f;
                if (pos && !(bf2f(pos[(int64_t)row * ldpos + col]) > 0.f)) v = 0.f;
                if (c32) {
                    float* p = c32 + (int64_t)row * ldc32 + col;
                    *p = beta32 ? *p + v : v;
                }
                if (c16) c16[(int64_t)row * ldc16 + col] = f2bf(v);
            }
}

__global__ void cast_bf16_kernel(const float* x, uint16_t* y, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i]);
}

__global__ void relu_grad_kernel(const float* g, const uint16_t* h, uint16_t* g16, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        float v = g[i];
        if (h && !(bf2f(h[i]) > 0.f)) v = 0.f;
        g16[i] = f2bf(v);
    }
}

DEV float as_float(float v) { return v; }
DEV float as_float(uint16_t v) { return bf2f(v); }

// Column sums in a fixed order: a work-group takes 16 columns, 64 groups of
// rows (group r the rows r, r + 64, ..), whose sums a tree adds in LDS.  One
// thread per column walked 1,024 rows one load at a time (236 us).
template <class T>
__global__ void __launch_bounds__(1024) colsum_kernel(const T* x, int rows, int cols, int64_t ld, float* out)
{
    __shared__ float red[64][17];
    const int c = threadIdx.x & 15, r = threadIdx.x >> 4;
    const int j = blockIdx.x * 16 + c;
    float s = 0.f;
    if (j < cols) {
#pragma unroll 8
        for (int i = r; i < rows; i += 64) s += as_float(x[(int64_t)i * ld + j]);
    }
    red[r][c] = s;
    __syncthreads();
    for (int k = 32; k > 0; k >>= 1) {
        if (r < k) red[r][c] += red[r + k][c];
        __syncthreads();
    }
    if (r == 0 && j < cols) out[j] = red[0][c];
}

// work-group sum of one float per thread (256 threads), in thread 0
DEV float wg_sum256(float s)
{
    __shared__ float red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    return red[0];
}

// g = 2 (y - t) / n; with more than one work-group the partial sums of
// (y - t)^2 stand in for g[0 .. grid) until mse_finish_kernel has read them
// (no scratch buffer is passed, and one work-group took 463 us for 409,600
// elements); one work-group writes its sum to loss
__global__ void __launch_bounds__(256) mse_grad_kernel(const float* y, const float* t, float* g, float* loss, int64_t n)
{
    const float sc = 2.f / (float)n;
    const int64_t held = loss && gridDim.x > 1 ? gridDim.x : 0;
    float s = 0.f;
    const int64_t step = (int64_t)gridDim.x * 256;
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    auto one = [&](int64_t at) {
        const float d = y[at] - t[at];
        if (at >= held) g[at] = sc * d;
        s += d * d;
    };
    if (i < n) one(i);                                       // (what is held lies in the first round)
    for (i += step; i + 3 * step < n; i += 4 * step) {
        // read before the stores, which may be to y or t: four reads in flight
        float d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = y[i + k * step] - t[i + k * step];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            g[i + k * step] = sc * d[k];
            s += d[k] * d[k];
        }
    }
    for (; i < n; i += step) one(i);
    if (!loss) return;
    s = wg_sum256(s);
    if (threadIdx.x != 0) return;
    if (held) g[blockIdx.x] = s;
    else loss[0] = s / (float)n;
}

__global__ void __launch_bounds__(256) mse_finish_kernel(const float* y, const float* t, float* g, float* loss, int nb,
                                                         int64_t n)
{
    const int i = threadIdx.x;
    const float s = wg_sum256(i < nb ? g[i] : 0.f);      // (every partial is read before the first is overwritten)
    if (i == 0) loss[0] = s / (float)n;
    if (i < nb) g[i] = 2.f / (float)n * (y[i] - t[i]);
}

// Adam on up to ADAM_MAX tensors in one launch (a launch per tensor of a small
// network costs more than its work); tensor k takes the work-groups
// first[k] .. first[k+1]-1
constexpr int ADAM_MAX = 16;
struct AdamArgs {
    stl_adam_tensor t[ADAM_MAX];
    int first[ADAM_MAX + 1];
    int n;
    float lr, b1, b2, eps, c1, c2;
};

__global__ void __launch_bounds__(256) adam_kernel(AdamArgs A)
{
    int k = 0;
    while (k + 1 < A.n && (int)blockIdx.x >= A.first[k + 1]) ++k;
    const stl_adam_tensor t = A.t[k];
    const int64_t nb = A.first[k + 1] - A.first[k];
    for (int64_t i = (int64_t)(blockIdx.x - A.first[k]) * 256 + threadIdx.x; i < t.n; i += nb * 256) {
        const float gi = t.g[i];
        const float mi = A.b1 * t.m[i] + (1.f - A.b1) * gi;
        const float vi = A.b2 * t.v[i] + (1.f - A.b2) * gi * gi;
        t.m[i] = mi;
        t.v[i] = vi;
        const float wi = t.w[i] - A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
        t.w[i] = wi;
        if (t.w16) t.w16[i] = f2bf(wi);
    }
}

__global__ void ascent_kernel(float* x, const float* dx, const int32_t* active, int64_t N, int T, int D, int t0,
                              int dupd, float lr)
{
    const int64_t total = N * (int64_t)T * D;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int d = (int)(i % D);
        const int64_t r = i / D;
        const int t = (int)(r % T);
        const int64_t nn = r / T;
        if (t < t0 || d >= dupd) continue;
        if (active && !active[nn]) continue;
        x[i] += lr * dx[i];
    }
}

}  // namespace stlmi_mlp

// ------------------------------------------------------------------ C ABI

using namespace stlmi_mlp;

// sets the library's thread-local message returned by stl_last_error()
void stlmi_set_error(const char* msg);

namespace {
stl_status mfail(stl_status s, const char* msg)
{
    stlmi_set_error(msg);
    return s;
}

int grid_for(int64_t n)
{
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    return (int)(g < 1 ? 1 : g);
}

stl_status launched(const char* what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        char buf[256];
        snprintf(buf, sizeof buf, "%s: launch failed: %s", what, hipGetErrorString(e));
        return mfail(STL_E_HIP, buf);
    }
    return STL_OK;
}
}  // namespace

static stl_status gemm(const char* what, const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B, int64_t sbk,
                       int64_t sbn, int32_t M, int32_t N, int32_t K, const float* bias, int32_t relu,
                       const uint16_t* pos, int64_t ldpos, float* c32, int64_t ldc32, int32_t beta32, uint16_t* c16,
                       int64_t ldc16, void* stream)
{
    const int64_t g64 = ((int64_t)M + 63) / 64 * (((int64_t)N + 63) / 64);
    // 32 x 32 tiles below two 64 x 64 work-groups per compute unit (256 of them)
    const int T = g64 < 512 ? 32 : 64;
    const dim3 grid((N + T - 1) / T, (M + T - 1) / T);
    if (grid.y > 65535) return mfail(STL_E_UNSUPPORTED, "stl_bf16_gemm: M too large");
    if (T == 32)
        hipLaunchKernelGGL(gemm_bf16_kernel<32>, grid, dim3(256), 0, (hipStream_t)stream, A, sam, sak, B, sbk, sbn, M, N,
                           K, bias, relu, pos, ldpos, c32, ldc32, beta32, c16, ldc16);
    else
        hipLaunchKernelGGL(gemm_bf16_kernel<64>, grid, dim3(256), 0, (hipStream_t)stream, A, sam, sak, B, sbk, sbn, M, N,
                           K, bias, relu, pos, ldpos, c32, ldc32, beta32, c16, ldc16);
    return launched(what);
}

extern "C" stl_status stl_bf16_gemm(const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B, int64_t sbk,
                                    int64_t sbn, int32_t M, int32_t N, int32_t K, const float* bias, int32_t relu,
                                    float* c32, int64_t ldc32, int32_t beta32, uint16_t* c16, int64_t ldc16,
                                    void* stream)
{
    if (M < 0 || N < 0 || K < 0) return mfail(STL_E_ARG, "stl_bf16_gemm: negative size");
    if (M == 0 || N == 0) return STL_OK;
    if ((K > 0 && (!A || !B)) || (!c32 && !c16)) return mfail(STL_E_ARG, "stl_bf16_gemm: null pointer");
    return gemm("stl_bf16_gemm", A, sam, sak, B, sbk, sbn, M, N, K, bias, relu, nullptr, 0, c32, ldc32, beta32, c16,
                ldc16, stream);
}

extern "C" stl_status stl_bf16_gemm_relu_grad(const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B,
                                              int64_t sbk, int64_t sbn, int32_t M, int32_t N, int32_t K,
                                              const uint16_t* h, int64_t ldh, uint16_t* g16, int64_t ldg, void* stream)
{
    if (M < 0 || N < 0 || K < 0) return mfail(STL_E_ARG, "stl_bf16_gemm_relu_grad: negative size");
    if (M == 0 || N == 0) return STL_OK;
    if ((K > 0 && (!A || !B)) || !h || !g16) return mfail(STL_E_ARG, "stl_bf16_gemm_relu_grad: null pointer");
    return gemm("stl_bf16_gemm_relu_grad", A, sam, sak, B, sbk, sbn, M, N, K, nullptr, 0, h, ldh, nullptr, 0, 0, g16, ldg,
                stream);
}

extern "C" stl_status stl_cast_bf16(const float* x, uint16_t* y, int64_t n, void* stream)
{
    if (n < 0 || (n > 0 && (!x || !y))) return mfail(STL_E_ARG, "stl_cast_bf16: bad arguments");
    if (n == 0) return STL_OK;
    hipLaunchKernelGGL(cast_bf16_kernel, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, x, y, n);
    return launched("stl_cast_bf16");
}

extern "C" stl_status stl_relu_grad_bf16(const float* g, const uint16_t* h, uint16_t* g16, int64_t n, void* stream)
{
    if (n < 0 || (n > 0 && (!g || !g16))) return mfail(STL_E_ARG, "stl_relu_grad_bf16: bad arguments");
    if (n == 0) return STL_OK;
    hipLaunchKernelGGL(relu_grad_kernel, dim3(grid_for(n)), dim3(256), 0, (hipStream_t)stream, g, h, g16, n);
    return launched("stl_relu_grad_bf16");
}

extern "C" stl_status stl_colsum(const float* x, int32_t rows, int32_t cols, int64_t ld, float* out, void* stream)
{
    if (rows < 0 || cols < 0 || (cols > 0 && (!x || !out))) return mfail(STL_E_ARG, "stl_colsum: bad arguments");
    if (cols == 0) return STL_OK;
    hipLaunchKernelGGL(colsum_kernel<float>, dim3((cols + 15) / 16), dim3(1024), 0, (hipStream_t)stream, x, rows, cols, ld,
                       out);
    return launched("stl_colsum");
}

extern "C" stl_status stl_colsum_bf16(const uint16_t* x, int32_t rows, int32_t cols, int64_t ld, float* out, void* stream)
{
    if (rows < 0 || cols < 0 || (cols > 0 && (!x || !out))) return mfail(STL_E_ARG, "stl_colsum_bf16: bad arguments");
    if (cols == 0) return STL_OK;
    hipLaunchKernelGGL(colsum_kernel<uint16_t>, dim3((cols + 15) / 16), dim3(1024), 0, (hipStream_t)stream, x, rows, cols,
                       ld, out);
    return launched("stl_colsum_bf16");
}

extern "C" stl_status stl_mse_grad(const float* y, const float* t, float* g, float* loss, int64_t n, void* stream)
{
    if (n <= 0 || !y || !t || !g) return mfail(STL_E_ARG, "stl_mse_grad: bad arguments");
    // g holds the partial sums between the two launches, so an in-place g keeps
    // to one work-group, as n below 16,384 does (16,383 elements 5.8 us in one
    // work-group, 5.6 in two launches); without a loss there are no sums
    auto apart = [&](const float* a) { return a + n <= g || g + n <= a; };
    const int64_t per = loss ? 4096 : 1024, least = loss ? 16384 : 2048;
    const int nb = n >= least && (!loss || (apart(y) && apart(t))) ? (int)(n / per < 256 ? n / per : 256) : 1;
    hipLaunchKernelGGL(mse_grad_kernel, dim3(nb), dim3(256), 0, (hipStream_t)stream, y, t, g, loss, n);
    stl_status s = launched("stl_mse_grad");
    if (s != STL_OK || !loss || nb == 1) return s;
    hipLaunchKernelGGL(mse_finish_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, y, t, g, loss, nb, n);
    return launched("stl_mse_grad");
}

extern "C" stl_status stl_adam_step_multi(const stl_adam_tensor* tensors, int32_t n_tensors, float lr, float b1, float b2,
                                          float eps, int32_t step, void* stream)
{
    if (n_tensors < 0 || step < 1 || (n_tensors > 0 && !tensors))
        return mfail(STL_E_ARG, "stl_adam_step_multi: bad arguments");
    for (int k = 0; k < n_tensors; ++k) {
        const stl_adam_tensor& t = tensors[k];
        if (t.n < 0 || (t.n > 0 && (!t.w || !t.g || !t.m || !t.v)))
            return mfail(STL_E_ARG, "stl_adam_step_multi: bad tensor");
    }
    for (int k0 = 0; k0 < n_tensors; k0 += ADAM_MAX) {
        AdamArgs A;
        A.n = 0;
        A.first[0] = 0;
        for (int k = k0; k < n_tensors && k < k0 + ADAM_MAX; ++k) {
            if (tensors[k].n == 0) continue;
            A.t[A.n] = tensors[k];
            A.first[A.n + 1] = A.first[A.n] + grid_for(tensors[k].n);
            ++A.n;
        }
        if (A.n == 0) continue;
        A.lr = lr;
        A.b1 = b1;
        A.b2 = b2;
        A.eps = eps;
        A.c1 = 1.f - powf(b1, (float)step);
        A.c2 = 1.f - powf(b2, (float)step);
        hipLaunchKernelGGL(adam_kernel, dim3(A.first[A.n]), dim3(256), 0, (hipStream_t)stream, A);
        const stl_status s = launched("stl_adam_step_multi");
        if (s != STL_OK) return s;
    }
    return STL_OK;
}

extern "C" stl_status stl_adam_step(float* w, const float* g, float* m, float* v, uint16_t* w16, int64_t n, float lr,
                                    float b1, float b2, float eps, int32_t step, void* stream)
{
    if (n < 0 || step < 1 || (n > 0 && (!w || !g || !m || !v))) return mfail(STL_E_ARG, "stl_adam_step: bad arguments");
    const stl_adam_tensor t = {w, g, m, v, w16, n};
    return stl_adam_step_multi(&t, 1, lr, b1, b2, eps, step, stream);
}

extern "C" stl_status stl_ascent_update(float* x, const float* dx, const int32_t* active, int64_t N, int32_t T,
                                        int32_t D, int32_t t0, int32_t d_upd, float lr, void* stream)
{
    if (N < 0 || T < 0 || D < 1 || (N > 0 && (!x || !dx))) return mfail(STL_E_ARG, "stl_ascent_update: bad arguments");
    const int64_t total = N * (int64_t)T * D;
    if (total == 0) return STL_OK;
    hipLaunchKernelGGL(ascent_kernel, dim3(grid_for(total)), dim3(256), 0, (hipStream_t)stream, x, dx, active, N, T,
                       D, t0, d_upd, lr);
    return launched("stl_ascent_update");
}
