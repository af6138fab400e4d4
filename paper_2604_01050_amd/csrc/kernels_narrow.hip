// Register-resident CSR loop of Eqs. 6-7 for few replica columns (gfx950):
// the loop of kernels_resident.hip with W = 2 or 4 columns per workgroup
// instead of 8 and the ring edges exchanged as tagged words.
//
// With 8 columns per workgroup an instance of C columns runs on C / 8 CUs: 16
// of 256 at C = 128. A step's arithmetic takes N * W * 23 VALU instructions on
// the 4 SIMDs of one CU (4.9 us at N = 4096, W = 8), so fewer columns per
// workgroup on more CUs shorten it in proportion, and what is left is the
// ring exchange. Counters (store the edges, wait for the stores, barrier,
// raise the counter, poll it, barrier, load the edges) cost 1.8 us of a step:
// here an edge value travels with its step number in one 64-bit word, stored
// and loaded coherently for the whole device, so that the neighbour polls the
// data itself and a step has one barrier (the operand is double-buffered in
// LDS). The coupling sums, which do not need the edges, are formed before the
// first poll, so that the words are usually there when they are first read.
//
// Measured per step (8 columns per workgroup and counters / 2 columns and
// words): N = 1000, degree 3, C = 128 2.48 / 1.12 us; N = 4096, degree 6, C =
// 128 6.20 / 2.94 us. What is left at N = 1000 is the round trip of the words
// (0.8 us) and the barrier. With 4 columns at N above 2048 a thread's rows are
// taken one at a time (the first polls wait, the later rows' words have
// arrived meanwhile), which needs half the registers: 4.41 us at N = 4096, C =
// 256 against 9.85 with all rows together (60 spilled registers).
//
// A word of step n + 1 goes to the slot of parity n + 1, which holds the word
// of step n - 1. The thread that overwrites it has read the neighbour's word
// of step n for the same row, and the neighbour's thread of that row (rows
// belong to the same thread index in every workgroup) stored that word after
// it had read this slot's step n - 1, so no unread word is overwritten.
#include "csr_common.h"
#include "ring_tags.h"

#include <type_traits>

namespace sbqa {
namespace {

using namespace csr;

template <int W> struct HalfVec;
template <> struct HalfVec<2> { typedef _Float16 type __attribute__((ext_vector_type(2))); };
template <> struct HalfVec<4> { typedef _Float16 type __attribute__((ext_vector_type(4))); };
template <int W> struct FloatVec;
template <> struct FloatVec<2> { typedef float2 type; };
template <> struct FloatVec<4> { typedef float4 type; };

// Weights in LDS (one conflict-free read a term) where a thread's rows and
// columns leave no registers for them (128 at four waves per SIMD); in
// registers otherwise, which keeps the LDS pipe for the operand gathers.
constexpr bool weights_in_lds(int RPT, int D, int W) { return W == 4 && RPT * D >= 16; }

// RPT rows per thread, degree padded to D, NT threads, W columns. Thread t
// owns rows t + q * NT, q < RPT; RPT * NT >= N. Its neighbours' LDS offsets
// stay in registers, two to a register.
template <int RPT, int D, int NT, int W>
__global__ __launch_bounds__(NT) void k_csr_narrow(const ResidentArgs a, uint64_t *__restrict__ words,
                                                 uint32_t *__restrict__ rings) {
    using HV = typename HalfVec<W>::type;
    using FV = typename FloatVec<W>::type;
    constexpr int ROWS = RPT * NT;
    constexpr bool WL = weights_in_lds(RPT, D, W);
    constexpr int G = WL ? 1 : RPT;   // rows whose sums, edges and updates go together
    __shared__ __align__(16) HV op[2][ROWS];   // operand f(X) of the workgroup's columns, by step parity
    __shared__ float wl_lds[WL ? RPT * D * NT : 1];
    const int t = threadIdx.x, w = blockIdx.x, NR = a.nr;
    const int P = a.R / W, c0 = w * W;
    const int run = c0 / a.R, part = (c0 - run * a.R) / W;
    const int wl = run * P + (part + P - 1) % P, wr = run * P + (part + 1) % P;
    // element (row r, column c0 + j) of the column-block state
    const int64_t sbase = (int64_t)(c0 >> 3) * NR * 8 + (c0 & 7);
    // words of parity b, workgroup v, edge e (0: first column, 1: last)
    auto slot = [&](int b, int v, int e) { return words + (((int64_t)b * a.nwg + v) * 2 + e) * ROWS; };

    const uint32_t tag0 = ring_base(rings + 2 * run);   // step s of the launch: tag0 + s + 1
    float xs[RPT][W], ys[RPT][W], wt[WL ? 1 : RPT][WL ? 1 : D], hv[RPT];
    uint32_t off[RPT][D / 2];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = t + q * NT;
        const FV x = *reinterpret_cast<const FV *>(a.x + sbase + (int64_t)r * 8);
        const FV y = *reinterpret_cast<const FV *>(a.y + sbase + (int64_t)r * 8);
        __builtin_memcpy(xs[q], &x, sizeof x);
        __builtin_memcpy(ys[q], &y, sizeof y);
        hv[q] = a.h[r];
#pragma unroll
        for (int p = 0; p < D; ++p) {
            const float v = a.valpad[(int64_t)p * NR + r];
            if constexpr (WL) wl_lds[(q * D + p) * NT + t] = v;   // read back by this thread only
            else wt[q][p] = v;
        }
#pragma unroll
        for (int p = 0; p < D; p += 2)
            off[q][p / 2] = (uint32_t)a.colpad[(int64_t)r * D + p] * (uint32_t)sizeof(HV) |
                            ((uint32_t)a.colpad[(int64_t)r * D + p + 1] * (uint32_t)sizeof(HV)) << 16;
    }
    {
        const float d0 = a.delta[a.n0];   // the operand of step n0 is f(x) at Delta_n0
        uint64_t *pf = slot(a.n0 & 1, w, 0), *pl = slot(a.n0 & 1, w, 1);
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = t + q * NT;
            HV f;
#pragma unroll
            for (int c = 0; c < W; ++c) f[c] = (_Float16)f_value(a.fmode, xs[q][c], d0);
            op[a.n0 & 1][r] = f;
            put_word(pf + r, tagged(__float_as_uint(xs[q][0]), tag0 + 1u));
            put_word(pl + r, tagged(__float_as_uint(xs[q][W - 1]), tag0 + 1u));
        }
    }
    float kA = a.coefA[a.n0], dn = a.delta[a.n0 + 1], jpr = a.jp[(int64_t)run * a.S + a.n0];
    __syncthreads();

    auto step = [&](int s, auto last_c) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(last_c)::value;
        // keeps the neighbour offsets packed (unpacked once per step) and the
        // weights in LDS
        if constexpr (WL) asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < RPT; ++q)
#pragma unroll
            for (int i = 0; i < D / 2; ++i) asm volatile("" : "+v"(off[q][i]));
        const int n = a.n0 + s, b = n & 1;
        const float d = (a.fmode == 1) ? 0.0f : dn;
        const float kA_n = kA, jp_n = jpr;
        if (!LAST) {   // the next step's scalars load while this step runs
            kA = a.coefA[n + 1];
            dn = a.delta[n + 2];
            jpr = a.jp[(int64_t)run * a.S + n + 1];
        }
        const uint8_t *opb = reinterpret_cast<const uint8_t *>(op[b]);
        const uint32_t tag = tag0 + (uint32_t)s + 1u;
        // (uniform base, 32-bit lane offset: no address registers per row)
        const uint64_t *el = slot(b, wl, 1), *er = slot(b, wr, 0);
        uint64_t *pf = slot(1 - b, w, 0), *pl = slot(1 - b, w, 1);
#pragma unroll
        for (int q0 = 0; q0 < RPT; q0 += G) {
            float acc[G][W];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int q = q0 + g;
#pragma unroll
                for (int c = 0; c < W; ++c) acc[g][c] = 0.f;
                if (q >= RPT) continue;
#pragma unroll
                for (int p = 0; p < D; ++p) {
                    const uint32_t jo = (off[q][p / 2] >> (16 * (p & 1))) & 0xFFFFu;
                    const HV f = *reinterpret_cast<const HV *>(opb + jo);
                    float wgt;
                    if constexpr (WL) wgt = wl_lds[(q * D + p) * NT + t];
                    else wgt = wt[q][p];
#pragma unroll
                    for (int c = 0; c < W; ++c) acc[g][c] = __builtin_fmaf(wgt, (float)f[c], acc[g][c]);
                }
            }
            // the neighbours' edges of step n: polled until every word of the
            // wave carries the step's tag
            uint64_t vl[G], vr[G];
            for (int polls = 0;; ++polls) {
                bool ok = true;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int q = q0 + g < RPT ? q0 + g : RPT - 1;
                    vl[g] = get_word(el + q * NT + (uint32_t)t);
                    vr[g] = get_word(er + q * NT + (uint32_t)t);
                }
#pragma unroll
                for (int g = 0; g < G; ++g) ok = ok && (uint32_t)(vl[g] >> 32) == tag && (uint32_t)(vr[g] >> 32) == tag;
                if (__all(ok) || stop_waiting(polls, a.err)) break;
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int q = q0 + g;
                if (q >= RPT) continue;
                const float xl0 = __uint_as_float((uint32_t)vl[g]), xr0 = __uint_as_float((uint32_t)vr[g]);
                float xo[W], yo[W];
                HV f;
#pragma unroll
                for (int c = 0; c < W; ++c) {
                    float sg;
                    update_elem(xs[q][c], ys[q][c], acc[g][c], hv[q], c == 0 ? xl0 : xs[q][c - 1],
                                c == W - 1 ? xr0 : xs[q][c + 1], jp_n, kA_n, a.kB, a.dt, a.kD, xo[c], yo[c], sg);
                    f[c] = (_Float16)(fabsf(xo[c]) > d ? sg : 0.0f);   // f of Eq. 8 (d = 0 for sign)
                }
                if constexpr (!LAST) {
                    put_word(pf + q * NT + (uint32_t)t, tagged(__float_as_uint(xo[0]), tag + 1u));
                    put_word(pl + q * NT + (uint32_t)t, tagged(__float_as_uint(xo[W - 1]), tag + 1u));
                    op[1 - b][t + q * NT] = f;
                }
#pragma unroll
                for (int c = 0; c < W; ++c) {
                    xs[q][c] = xo[c];
                    ys[q][c] = yo[c];
                }
            }
            // groups kept apart in the schedule where registers are short
            if constexpr (G < RPT) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!LAST) __syncthreads();   // step n + 1 reads what step n wrote; step n's reads are done
    };
    for (int s = 0; s + 1 < a.K; ++s) step(s, std::false_type{});
    step(a.K - 1, std::true_type{});
    __syncthreads();   // the last words are read
    if (t == 0) ring_done(rings + 2 * run, P, tag0, a.K);
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = t + q * NT;
        FV x, y;
        __builtin_memcpy(&x, xs[q], sizeof x);
        __builtin_memcpy(&y, ys[q], sizeof y);
        *reinterpret_cast<FV *>(a.x + sbase + (int64_t)r * 8) = x;
        *reinterpret_cast<FV *>(a.y + sbase + (int64_t)r * 8) = y;
    }
}

template <class F>
hipError_t with_narrow(int rows, int D, int W, F &&f) {
    auto by_w = [&](auto rpt, auto nt, auto d) -> hipError_t {
        constexpr int R_ = decltype(rpt)::value, T_ = decltype(nt)::value, D_ = decltype(d)::value;
        if (W == 2) return f(&k_csr_narrow<R_, D_, T_, 2>, T_);
        if (W == 4) return f(&k_csr_narrow<R_, D_, T_, 4>, T_);
        return hipErrorInvalidValue;
    };
    auto by_d = [&](auto rpt, auto nt) -> hipError_t {
        constexpr int R_ = decltype(rpt)::value;
        switch (D) {
            case 4: return by_w(rpt, nt, std::integral_constant<int, 4>{});
            case 6: return by_w(rpt, nt, std::integral_constant<int, 6>{});
            case 8: if constexpr (R_ <= 2) return by_w(rpt, nt, std::integral_constant<int, 8>{}); break;
            case 12: if constexpr (R_ <= 2) return by_w(rpt, nt, std::integral_constant<int, 12>{}); break;
            case 16: if constexpr (R_ <= 2) return by_w(rpt, nt, std::integral_constant<int, 16>{}); break;
            default: break;
        }
        return hipErrorInvalidValue;
    };
    using T5 = std::integral_constant<int, 512>;
    using T10 = std::integral_constant<int, 1024>;
    switch (rows) {
        case 512: return by_d(std::integral_constant<int, 1>{}, T5{});
        case 1024: return by_d(std::integral_constant<int, 1>{}, T10{});
        case 2048: return by_d(std::integral_constant<int, 2>{}, T10{});
        case 3072: return by_d(std::integral_constant<int, 3>{}, T10{});
        case 4096: return by_d(std::integral_constant<int, 4>{}, T10{});
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// rows that the narrow loop computes: N rounded up to whole workgroups of
// threads (at most the padded rows of the state)
int narrow_rows(int N) { return N <= 512 ? 512 : (N + 1023) / 1024 * 1024; }

hipError_t launch_csr_narrow(const ResidentArgs &a, int D, int W, uint64_t *words, uint32_t *rings, hipStream_t st) {
    const int rows = narrow_rows(a.N);
    if ((W != 2 && W != 4) || a.R % W || 8 % W || a.nwg < 1 || a.nwg * W % a.R || rows > a.nr || a.N > rows || a.K < 1)
        return hipErrorInvalidValue;
    return with_narrow(rows, D, W, [&](auto kern, int threads) -> hipError_t {
        hipLaunchKernelGGL(kern, dim3(a.nwg), dim3(threads), 0, st, a, words, rings);
        return hipGetLastError();
    });
}

hipError_t narrow_max_blocks(int D, int W, int N, int *blocks_per_cu) {
    return with_narrow(narrow_rows(N), D, W, [&](auto kern, int threads) -> hipError_t {
        return max_blocks_per_cu(reinterpret_cast<const void *>(kern), threads, 0, blocks_per_cu);
    });
}

}  // namespace sbqa
