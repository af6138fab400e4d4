// Sparse (CSR) SBQA step for gfx950: the coupling sum of Eq. 7 over the
// neighbours of spin i, fused with the update of Eqs. 6-7 (pump, Trotter ring,
// kick, drift, wall) and the emission of the next operand f(X) (Eq. 8).
//
// State is spin-major ([N][Cs], Cs = C rounded up to 4): one wavefront owns
// one spin row i and 256 consecutive replica columns (4 per lane), so every
// neighbour gather is one contiguous 256-byte (int8 operand) or 1 KiB (fp32
// ballistic operand) read. Blocks are numbered so that block b handles column
// chunk b % nchunk: with the round-robin block-to-XCD dispatch, the chunks of
// one XCD stay in its L2 and the gathers hit there.
#include "csr_step.h"

namespace sbqa {
namespace {

using namespace csr;

template <bool BALLISTIC, bool RING_SHFL, bool NT>
__global__ __launch_bounds__(256) void k_csr_step(int N, int Cs, int C, int R, int nchunk,
                                                  const int32_t *__restrict__ row_ptr,
                                                  const int32_t *__restrict__ col,
                                                  const float *__restrict__ val, const Tri3 t3,
                                                  const float *__restrict__ h,
                                                  const float *__restrict__ x_in, float *__restrict__ x_out,
                                                  float *__restrict__ y, const int8_t *__restrict__ g_in,
                                                  int8_t *__restrict__ g_out, const float *__restrict__ jp,
                                                  int64_t jp_stride, StepCoef k, int fmode) {
    csr_step_body<BALLISTIC, RING_SHFL, NT>(blockIdx.x, N, Cs, C, R, nchunk, row_ptr, col, val, t3, h, x_in, x_out,
                                            y, g_in, g_out, jp, jp_stride, k, fmode);
}

// Grouped step of every CSR instance of one serving group.
template <bool BALLISTIC, bool RING_SHFL>
__global__ __launch_bounds__(256) void k_group_csr(const GroupHeader *__restrict__ hdr,
                                                   const GroupTask *__restrict__ tasks, int offset) {
    csr_group_blocks<BALLISTIC, RING_SHFL>(hdr, tasks, offset, blockIdx.x, gridDim.x);
}

// Holds a stream for ticks of the 100 MHz clock (a fixed number of looks at it
// at most).
__global__ __launch_bounds__(64) void k_hold(int ticks) {
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    for (int q = 0; q < ticks && (int64_t)(__builtin_amdgcn_s_memrealtime() - t0) < ticks; ++q)
        __builtin_amdgcn_s_sleep(1);
}

__global__ __launch_bounds__(256) void k_csr_operand(int N, int Cs, int C, const float *__restrict__ x,
                                                     int8_t *__restrict__ g, float delta, int fmode) {
    const int64_t e4 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (e4 >= (int64_t)N * Cs) return;
    const int c = (int)(e4 % Cs);
    const float4 v = *reinterpret_cast<const float4 *>(x + e4);
    float f[4] = {f_value(fmode, v.x, delta), f_value(fmode, v.y, delta), f_value(fmode, v.z, delta),
                  f_value(fmode, v.w, delta)};
    for (int e = 0; e < 4; ++e)
        if (c + e >= C) f[e] = 0.f;
    *reinterpret_cast<uint32_t *>(g + e4) = pack_ternary(f[0], f[1], f[2], f[3]);
}

template <bool BALLISTIC>
__global__ __launch_bounds__(256) void k_csr_fields(int N, int Cs, int C, int nchunk,
                                                    const int32_t *__restrict__ row_ptr,
                                                    const int32_t *__restrict__ col,
                                                    const float *__restrict__ val, const Tri3 t3,
                                                    const float *__restrict__ x, const int8_t *__restrict__ g,
                                                    float *__restrict__ phi) {
    const CsrPos pos = csr_pos(blockIdx.x, C, nchunk);
    const int i = pos.i, c = pos.c;
    if (i >= N || c >= C) return;
    float4 v = gather_fields<BALLISTIC, false>(i, c, Cs, row_ptr, col, val, x, g);
    if (t3.ptr) v = gather_fields3<BALLISTIC, false>(i, c, Cs, t3, x, g, v);
    *reinterpret_cast<float4 *>(phi + (int64_t)i * Cs + c) = v;
}


}  // namespace

hipError_t launch_csr_step(int fmode, int N, int Cs, int R, int runs, const int32_t *row_ptr,
                           const int32_t *col, const float *val, const Tri3 &t3, const float *h, const float *x_in,
                           float *x_out, float *y, const int8_t *g_in, int8_t *g_out, const float *jp,
                           int64_t jp_stride, StepCoef k, hipStream_t st) {
    const int C = R * runs;
    if (Cs % 4 || Cs < C) return hipErrorInvalidValue;
    const int nchunk = csr_step_chunks(C);
    dim3 grid(csr_step_blocks(N, C)), block(WAVES * 64);
    const bool shfl = csr_ring_shfl(R);
    // x in, x out and y stream through once per step; when they are larger
    // than the last-level cache (256 MiB on MI355X; 192 MiB leaves room for
    // the operand and the CSR), non-temporal accesses keep them from evicting
    // the gathered operand rows. Smaller states are better served cached.
    const bool nt = 3.0 * 4.0 * (double)N * (double)Cs > 192.0 * 1024 * 1024;
#define SBQA_CSR_LAUNCH(B, S, T)                                                                               \
    hipLaunchKernelGGL((k_csr_step<B, S, T>), grid, block, 0, st, N, Cs, C, R, nchunk, row_ptr, col, val, t3, h,    \
                       x_in, x_out, y, g_in, g_out, jp, jp_stride, k, fmode)
    if (fmode == 2) {
        if (shfl) SBQA_CSR_LAUNCH(true, true, false);
        else SBQA_CSR_LAUNCH(true, false, false);
    } else if (nt) {
        if (shfl) SBQA_CSR_LAUNCH(false, true, true);
        else SBQA_CSR_LAUNCH(false, false, true);
    } else {
        if (shfl) SBQA_CSR_LAUNCH(false, true, false);
        else SBQA_CSR_LAUNCH(false, false, false);
    }
#undef SBQA_CSR_LAUNCH
    return hipGetLastError();
}

int csr_step_blocks(int N, int C) {
    const int rows = WAVES << csr_rpw_shift(C);
    return csr_step_chunks(C) * ((N + rows - 1) / rows);
}

int csr_step_chunks(int C) { return (C + COLS_PER_WAVE - 1) / COLS_PER_WAVE; }

bool csr_ring_shfl(int R) { return (R % 4 == 0) && (COLS_PER_WAVE % R == 0); }

hipError_t launch_group_csr(bool ballistic, bool shfl, const GroupHeader *hdr, const GroupTask *tasks, int grid,
                            int offset, hipStream_t st) {
    if (grid < 1) return hipErrorInvalidValue;
#define SBQA_GCSR(B, S) hipLaunchKernelGGL((k_group_csr<B, S>), dim3(grid), dim3(WAVES * 64), 0, st, hdr, tasks, offset)
    if (ballistic) {
        if (shfl) SBQA_GCSR(true, true);
        else SBQA_GCSR(true, false);
    } else {
        if (shfl) SBQA_GCSR(false, true);
        else SBQA_GCSR(false, false);
    }
#undef SBQA_GCSR
    return hipGetLastError();
}

hipError_t launch_hold(int us, hipStream_t st) {
    hipLaunchKernelGGL(k_hold, dim3(1), dim3(64), 0, st, us * 100);
    return hipGetLastError();
}

hipError_t launch_csr_operand(int fmode, int N, int Cs, int C, const float *x, int8_t *g, float delta,
                              hipStream_t st) {
    const int64_t n4 = (int64_t)N * Cs / 4;
    dim3 grid((unsigned)((n4 + 255) / 256)), block(256);
    hipLaunchKernelGGL(k_csr_operand, grid, block, 0, st, N, Cs, C, x, g, delta, fmode);
    return hipGetLastError();
}

hipError_t launch_csr_fields(int fmode, int N, int Cs, int C, const int32_t *row_ptr, const int32_t *col,
                             const float *val, const Tri3 &t3, const float *x, const int8_t *g, float *phi,
                             hipStream_t st) {
    const int nchunk = csr_step_chunks(C);
    dim3 grid(csr_step_blocks(N, C)), block(WAVES * 64);
    if (fmode == 2)
        hipLaunchKernelGGL(k_csr_fields<true>, grid, block, 0, st, N, Cs, C, nchunk, row_ptr, col, val, t3, x, g, phi);
    else
        hipLaunchKernelGGL(k_csr_fields<false>, grid, block, 0, st, N, Cs, C, nchunk, row_ptr, col, val, t3, x, g, phi);
    return hipGetLastError();
}


}  // namespace sbqa
