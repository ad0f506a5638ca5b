// Parameter reduction, the fused, interval and matrix-core kernels, and the
// launch helpers of the STL robustness library (gfx950).
#include "stl_exec.h"

namespace stlmi {

// One work-group per parameter p: d/dp is the sum, over the per-trajectory
// rows and in a fixed order, of every (mask, bound) column of the partials
// whose parameter index is p (two mask nodes may share a, b); parameters no
// mask bound names get 0.  The kernels overwrite gp, they never accumulate.
struct ReduceArgs {              // (not the whole plan: the argument segment is copied for every launch)
    const float* part;
    float* gp;
    int64_t rows;
    int n_masks;
    int mask_param[MAX_MASKS];
};

__global__ void __launch_bounds__(1024) stl_reduce_params(ReduceArgs A)
{
    const float* part = A.part;
    float* gp = A.gp;
    const int64_t rows = A.rows;
    const int n_masks = A.n_masks;
    __shared__ float red[1024];
    const int tid = threadIdx.x;
    const int p = blockIdx.x;
    int cols[2 * MAX_MASKS];
    int nc = 0;
    for (int q = 0; q < 2 * n_masks; ++q)
        if (A.mask_param[q >> 1] + (q & 1) == p) cols[nc++] = q;
    if (nc == 0) {
        if (tid == 0) gp[p] = 0.f;
        return;
    }
    // each thread: rows tid, tid + 1024, ... (four independent sums, added in a fixed order)
    float s4[4] = {0.f, 0.f, 0.f, 0.f};
    const int64_t stride = (int64_t)blockDim.x;
    for (int64_t r0 = tid; r0 < rows; r0 += 4 * stride) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t r = r0 + u * stride;
            if (r < rows)
                for (int k = 0; k < nc; ++k) s4[u] += part[r * 2 * n_masks + cols[k]];
        }
    }
    red[tid] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    __syncthreads();
    for (int k = blockDim.x >> 1; k > 0; k >>= 1) {
        if (tid < k) red[tid] += red[tid + k];
        __syncthreads();
    }
    if (tid == 0) gp[p] = red[0];
}

__global__ void stl_zero_counter(int* c) { if (threadIdx.x < 3) c[threadIdx.x] = 0; }

__global__ void stl_fill_int(int* p, int64_t n, int v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

}  // namespace stlmi

#include "stl_fused.h"
#include "stl_interval.h"
#include "stl_mx.h"

// ------------------------------------------------------------------ launch helpers (host)

namespace stlmi {

size_t scratch_floats(int Lc, int nt, int units, int until_b, bool until_masked)
{
    size_t s = (size_t)units * Lc;
    // smooth Until adjoint: nt checkpoints per UCK steps
    if (until_b >= 0) {
        const size_t ck = (size_t)nt * until_cks(until_b, Lc, until_masked ? UCK : UCK_CS) * 2;
        s = std::max(s, (size_t)(until_masked ? UCK_UNIT_MASK : UCK_UNIT) * Lc + ck);
    }
    return s + 64;
}

// positions of the smooth Until's LDS tile for slots in the workspace (0: none)
int until_tile_len(int nt, int until_b, bool until_masked)
{
    return until_b < 0 || until_masked || until_b > UT_TILE_B ? 0 : (nt * UT_RMAX + until_b + UT_RMAX + 1) & ~1;
}

// LDS beside the slots for a plan with smooth Untils: the waves' export
// buffers, and the tile with the backward's checkpoints
size_t until_lds_bytes(int nt, int until_b, bool bwd, int tile, int Lc)
{
    if (until_b < 0) return 0;
    size_t s = (size_t)tile * 16;
    if (bwd) s += (size_t)nt * 8 + (tile ? (size_t)nt * until_cks(until_b, Lc, UCK_CS) * 8 : 0);
    return s;
}

// one kernel per direction, slot placement and operator set (stl_exec_*.hip)
hipError_t launch_exec_fwd(bool full, const DevPlan& plan, const Batch& bt, const KArgs& ka, int grid, int nt,
                           size_t lds_bytes, hipStream_t s);
hipError_t launch_exec_bwd(bool full, const DevPlan& plan, const Batch& bt, const KArgs& ka, int grid, int nt,
                           size_t lds_bytes, hipStream_t s);
hipError_t launch_exec_bwd_ws(bool full, const DevPlan& plan, const Batch& bt, const KArgs& ka, int grid, int nt,
                              size_t lds_bytes, hipStream_t s);
hipError_t set_max_lds_exec_fwd(int bytes);
hipError_t set_max_lds_exec_bwd(int bytes);
hipError_t set_max_lds_exec_bwd_ws(int bytes);

// no smooth mask, no smooth Until, no softmax-weighted window: the small kernels
bool plan_is_plain(const DevPlan& plan)
{
    for (int k = plan.n_pred; k < plan.n_ins; ++k) {
        const Instr& I = plan.ins[k];
        if (I.kind == K_MASK || (I.kind == K_UNTIL && (I.mask >= 0 || (I.flags & F_SMOOTH))) ||
            (I.kind == K_WIN && (I.flags & F_SOFT)))
            return false;
    }
    return true;
}

hipError_t launch_exec(bool bwd, const DevPlan& plan, const Batch& bt, const KArgs& ka, int grid, int nt,
                       size_t lds_bytes, hipStream_t s)
{
    const bool full = !plan_is_plain(plan);
    if (!bwd) return launch_exec_fwd(full, plan, bt, ka, grid, nt, lds_bytes, s);
    if (ka.garena) return launch_exec_bwd_ws(full, plan, bt, ka, grid, nt, lds_bytes, s);
    return launch_exec_bwd(full, plan, bt, ka, grid, nt, lds_bytes, s);
}

hipError_t set_max_lds(size_t bytes)
{
    hipError_t e = set_max_lds_exec_fwd((int)bytes);
    if (e == hipSuccess) e = set_max_lds_exec_bwd((int)bytes);
    return e == hipSuccess ? set_max_lds_exec_bwd_ws((int)bytes) : e;
}

size_t fused_lds(int Lc, int n, int D, bool bwd)
{
    (void)n;
    (void)D;
    (void)bwd;
    return fused_lds_bytes(Lc);
}

int fused_max_T() { return FNT * FNO; }

size_t mask_tab_bytes() { return sizeof(MaskTab); }

hipError_t launch_fused(bool bwd, const DevPlan& plan, const Batch& bt, const KArgs& ka, size_t lds, hipStream_t s)
{
    hipLaunchKernelGGL(stl_mask_tables, dim3(plan.fused.n), dim3(256), 0, s, plan, ka.params, (int)bt.T,
                       (MaskTab*)ka.tabs, ka.counter);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)bt.B), block(FNT);
    const bool full = bt.T == FNT * FNO && bt.Lcap == FNT * FNO;
#define STLMI_FUSED_CASE(NN)                                                                            \
    case NN:                                                                                            \
        if (bwd && full)                                                                                \
            hipLaunchKernelGGL((stl_fused_bwd<NN, true>), grid, block, lds, s, plan, bt, ka);           \
        else if (bwd)                                                                                   \
            hipLaunchKernelGGL((stl_fused_bwd<NN, false>), grid, block, lds, s, plan, bt, ka);          \
        else if (full)                                                                                  \
            hipLaunchKernelGGL((stl_fused_fwd<NN, true>), grid, block, lds, s, plan, bt, ka);           \
        else                                                                                            \
            hipLaunchKernelGGL((stl_fused_fwd<NN, false>), grid, block, lds, s, plan, bt, ka);          \
        break;
    switch (plan.fused.n) {
        STLMI_FUSED_CASE(1)
        STLMI_FUSED_CASE(2)
        STLMI_FUSED_CASE(3)
        STLMI_FUSED_CASE(4)
    default:
        return hipErrorInvalidValue;
    }
#undef STLMI_FUSED_CASE
    return hipGetLastError();
}

hipError_t set_max_lds_fused(size_t bytes)
{
    const void* fns[] = {
        (const void*)stl_fused_fwd<1, false>, (const void*)stl_fused_fwd<2, false>, (const void*)stl_fused_fwd<3, false>,
        (const void*)stl_fused_fwd<4, false>, (const void*)stl_fused_bwd<1, false>, (const void*)stl_fused_bwd<2, false>,
        (const void*)stl_fused_bwd<3, false>, (const void*)stl_fused_bwd<4, false>, (const void*)stl_fused_fwd<1, true>,
        (const void*)stl_fused_fwd<2, true>, (const void*)stl_fused_fwd<3, true>, (const void*)stl_fused_fwd<4, true>,
        (const void*)stl_fused_bwd<1, true>, (const void*)stl_fused_bwd<2, true>, (const void*)stl_fused_bwd<3, true>,
        (const void*)stl_fused_bwd<4, true>};
    for (const void* f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_zero_counter(int* c, hipStream_t s)
{
    hipLaunchKernelGGL(stl_zero_counter, dim3(1), dim3(64), 0, s, c);
    return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int64_t n, int v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(stl_fill_int, dim3(grid), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_reduce_params(const float* part, int64_t B, const DevPlan& plan, float* gp, hipStream_t s)
{
    if (plan.n_params < 1) return hipSuccess;
    ReduceArgs A;
    A.part = part;
    A.gp = gp;
    A.rows = B;
    A.n_masks = plan.n_masks;
    for (int m = 0; m < MAX_MASKS; ++m) A.mask_param[m] = plan.mask_param[m];
    hipLaunchKernelGGL(stl_reduce_params, dim3(plan.n_params), dim3(1024), 0, s, A);
    return hipGetLastError();
}

// ------------------------------------------------------------------ matrix-core path

// dynamic LDS of the matrix-core kernels: the rings (n masks x 16 rows), the
// result buffers, and the backward's derivative tiles
size_t mx_lds_bytes(int n, int D, bool bwd)
{
    return (size_t)n * MXG * MXRS + mx_xch_bytes(n, D, bwd) + (bwd ? (size_t)n * NDMAX * 2 * 64 * 16 : 0);
}
size_t mx_static_lds() { return sizeof(MxShared); }

hipError_t set_max_lds_mx(size_t bytes)
{
    hipError_t e = hipSuccess;
#define STLMI_MX_ATTR(KK)                                                                                   \
    {                                                                                                     \
        const hipError_t e2 = hipFuncSetAttribute((const void*)KK, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                                  (int)bytes);                                            \
        if (e2 != hipSuccess) e = e2;                                                                     \
    }
#define STLMI_MX_ATTR2(NN, DD)                                                                            \
    STLMI_MX_ATTR((stl_mx_fwd<NN, DD, false>)) STLMI_MX_ATTR((stl_mx_fwd<NN, DD, true>))                  \
    STLMI_MX_ATTR((stl_mx_bwd<NN, DD, false>)) STLMI_MX_ATTR((stl_mx_bwd<NN, DD, true>))
    STLMI_MX_ATTR2(1, 1) STLMI_MX_ATTR2(1, 2) STLMI_MX_ATTR2(2, 1) STLMI_MX_ATTR2(2, 2)
#undef STLMI_MX_ATTR2
#undef STLMI_MX_ATTR
    return e;
}

static bool al16(const void* p) { return (((uintptr_t)p) & 15) == 0; }

// the forward or backward kernel over groups of 16 trajectories.  The
// 16-byte load / store variants need T a multiple of 4 and 16-byte aligned
// arrays (x; forward: root and saved values; backward: G, saved values, dx).
hipError_t launch_mx(bool bwd, const DevPlan& plan, const Batch& bt, const KArgs& ka, const MxArgs& mx, size_t lds,
                     hipStream_t s)
{
    // (forward: 2n matrix and 4n staging waves; backward: 2n of each)
    const dim3 grid((unsigned)((bt.B + MXG - 1) / MXG)), block((bwd ? 256 : 384) * plan.fused.n);
    const bool d2 = bt.D == 2;
    const bool vec = bt.T % 4 == 0 && bt.T >= 4 && al16(bt.x) &&
                     (bwd ? al16(ka.G) && al16(ka.saved_in) && al16(ka.dx) : al16(ka.root) && al16(ka.saved));
#define STLMI_MX_K(NN, DD, VV)                                                                            \
    if (bwd) hipLaunchKernelGGL((stl_mx_bwd<NN, DD, VV>), grid, block, lds, s, plan, bt, ka, mx);          \
    else hipLaunchKernelGGL((stl_mx_fwd<NN, DD, VV>), grid, block, lds, s, plan, bt, ka, mx);
#define STLMI_MX_CASE(NN)                                                                                 \
    case NN:                                                                                              \
        if (d2 && vec) { STLMI_MX_K(NN, 2, true) }                                                        \
        else if (d2) { STLMI_MX_K(NN, 2, false) }                                                         \
        else if (vec) { STLMI_MX_K(NN, 1, true) }                                                         \
        else { STLMI_MX_K(NN, 1, false) }                                                                 \
        break;
    switch (plan.fused.n) {
        STLMI_MX_CASE(1)
        STLMI_MX_CASE(2)
    default:
        return hipErrorInvalidValue;
    }
#undef STLMI_MX_CASE
#undef STLMI_MX_K
    return hipGetLastError();
}

}  // namespace stlmi
