// Many-step loop for dense +-1 instances of up to MID_MAX_N spins (gfx950).
//
// One launch per step leaves such an instance to launch and load latency: at N
// = 601, C = 128 the step kernel ran 7.5 us on 32 of the 256 CUs. Here the
// couplings, one bit each, and the state stay in registers for many steps. A
// group of 16 (MB = 2: 32) replica columns, whole runs, is worked on by G
// workgroups, each owning a range of spins: per step a wave forms the coupling
// sums of 16 spins x 16 columns with fp4 MFMAs (+-1 and 0 are exact, the sums
// are exact integers: the same bits as every other dense path), with its rows
// of J expanded in registers and the operand f(X) of all spins in LDS, then
// updates its 4 spins x 1 column per lane (Eqs. 6-7; the ring neighbours are
// lanes of the same row of 16) and emits the new operand, 4 bits per spin.
// Workgroups of a group exchange the operand as 64-bit words of 8 spins and
// the step's tag, stored and loaded coherently for the whole device and polled by
// the readers themselves; nothing else crosses workgroups.
//
// A word of step n + 1 overwrites the one of step n - 1. Its writer has then
// received every other workgroup's words of step n, which were sent after the
// barrier behind that workgroup's reads of step n - 1.
//
// Bound by latency: at N = 601, C = 128 (5 workgroups of 8 waves per group) a
// step takes 1.9 us (7.2 us with one launch per step), 0.9 us of it the words'
// way to the other workgroups; N = 1024 2.15 (7.2), N = 2048 2.95 (8.6). One
// workgroup per group needs no exchange and takes N / 256 times as long for
// its updates: 0.97 us up to 256 spins, 3.8 us at N = 601.
#include "ring_tags.h"

#include <type_traits>

namespace sbqa {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef int i8v __attribute__((ext_vector_type(8)));

constexpr int E8M0_ONE = 127;               // block scale 1

__device__ __forceinline__ float f_mid(int fmode, float x, float delta) {
    const float d = (fmode == 1) ? 0.0f : delta;    // dSB: sign(0) = 0
    return fabsf(x) > d ? __builtin_copysignf(1.0f, x) : 0.0f;
}

// 4 consecutive spins as e2m1 nibbles
__device__ __forceinline__ uint32_t pack_fp4(const float (&f)[4]) {
    uint32_t v = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, f[0], f[1], 1.0f, 0);
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(v, f[2], f[3], 1.0f, 1);
}

// Row rotation within 16 lanes: lane i of a row receives lane i - 1 (LEFT) or
// i + 1, modulo 16.
template <bool LEFT>
__device__ __forceinline__ float row_rotate(float v) {
    constexpr int ctrl = LEFT ? 0x121 : 0x12F;
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, true));
}

// NT threads, RBW row blocks of 16 spins per wave, NS superchunks of 512 spins
// (K), MB column blocks of 16, ROT: R == 16 * MB (the ring is a row rotation).
template <int NT, int RBW, int NS, int MB, bool ROT>
__global__ __launch_bounds__(NT) void k_dense_mid(const MidArgs a) {
    constexpr int NWAVE = NT / 64;
    constexpr int CHUNKS = 4 * NS;               // K chunks of 128 spins
    // operand of the group's columns by step parity: MB column blocks of nch
    // K chunks, 1 KiB each; the exchanged words have the same order, one word
    // per dword
    __shared__ __align__(16) uint8_t op[2][MB * CHUNKS * 1024];
    constexpr int U = MB * CHUNKS * 256 >= NT ? MB * CHUNKS * 256 / NT : 1;   // words per thread
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int grp = blockIdx.x / a.G, part = blockIdx.x - grp * a.G;
    const int nrb = (a.N + 15) / 16, nch = (a.N + 127) / 128;
    const int rb0 = part * (NWAVE * RBW);        // this workgroup's row blocks

    // this lane's columns and the lanes of their ring neighbours
    int col[MB], lsrc[MB], rsrc[MB];
    bool live[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const int j = 16 * b + m;                // column of the group
        const int per = a.cols;                  // columns of a group in use: whole runs
        const int jj = j < per ? j : j % a.R;    // lanes past them repeat the first run
        const int base = jj / a.R * a.R, k = jj - base;
        const int c = grp * per + jj;
        live[b] = j < per && c < a.C;
        col[b] = c < a.C ? c : a.C - 1;
        lsrc[b] = base + (k == 0 ? a.R - 1 : k - 1);
        rsrc[b] = base + (k == a.R - 1 ? 0 : k + 1);
    }

    for (int e = tid; e < 2 * MB * CHUNKS * 64; e += NT)
        reinterpret_cast<uint4 *>(op)[e] = make_uint4(0u, 0u, 0u, 0u);

    const uint32_t tag0 = a.G > 1 ? ring_base(a.rings + 2 * grp) : 0u;   // step s of the launch: tag0 + s + 1
    uint4 J[RBW][NS];
    f4 x[RBW][MB], y[RBW][MB], hv[RBW];
    uint32_t pmask[RBW];                         // operand nibbles of spins below N
#pragma unroll
    for (int q = 0; q < RBW; ++q) {
        const int rb = rb0 + q * NWAVE + wave;
        pmask[q] = 0u;
        if (rb >= nrb) continue;
        const int i4 = 16 * rb + 4 * g;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            J[q][s] = s * 4 < nch ? a.J[((int64_t)rb * a.ns + s) * 64 + lane] : make_uint4(0u, 0u, 0u, 0u);
        hv[q] = *reinterpret_cast<const f4 *>(a.h + i4);
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            x[q][b] = *reinterpret_cast<const f4 *>(a.x + (int64_t)col[b] * a.Np + i4);
            y[q][b] = *reinterpret_cast<const f4 *>(a.y + (int64_t)col[b] * a.Np + i4);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (i4 + e < a.N) pmask[q] |= 0xFu << (4 * e);   // used by lanes of even g: 8 spins
    }
    // the dwords of the operand that other workgroups own (bit u: dword u * NT + tid)
    uint32_t need = 0u;
    if (a.G > 1) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = u * NT + tid, o = e % (nch * 256);
            const int rb = (o >> 8) * 8 + ((o >> 6) & 3) * 2 + ((o >> 1) & 1);   // row block of its 8 spins
            if (e < MB * nch * 256 && rb < nrb && (rb < rb0 || rb >= rb0 + NWAVE * RBW)) need |= 1u << u;
        }
    }
    auto words = [&](int par) { return a.words + ((int64_t)par * a.groups + grp) * (MB * nch * 256); };
    // operand of step n for row block q from f values; published unless alone
    auto emit = [&](int n, int q, int b, const float (&f)[4]) __attribute__((always_inline)) {
        const int rb = rb0 + q * NWAVE + wave, i0 = 16 * rb;
        uint32_t v = pack_fp4(f);
        v |= (uint32_t)__shfl_xor((int)v, 16) << 16;
        if ((g & 1) == 0) {
            v &= pmask[q];
            const uint32_t o = (uint32_t)(b * nch + (i0 >> 7)) * 1024u +
                               (uint32_t)(m + 16 * ((i0 & 127) >> 5)) * 16u + (uint32_t)((i0 & 16) + 4 * g) / 2u;
            *reinterpret_cast<uint32_t *>(&op[n & 1][o]) = v;
            if (a.G > 1)
                put_word(words(n & 1) + o / 4u, tagged(v, tag0 + (uint32_t)(n - a.n0) + 1u));
        }
    };
    __syncthreads();
    {
        const float d0 = a.delta[a.n0];
#pragma unroll
        for (int q = 0; q < RBW; ++q) {
            if (rb0 + q * NWAVE + wave >= nrb) continue;
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = f_mid(a.fmode, x[q][b][e], d0);
                emit(a.n0, q, b, f);
            }
        }
    }
    float jpn[MB];
    float kA = a.coefA[a.n0], dcur = a.delta[a.n0], dn = a.delta[a.n0 + 1];
#pragma unroll
    for (int b = 0; b < MB; ++b) jpn[b] = a.jp[(int64_t)(col[b] / a.R) * a.S + a.n0];

    for (int n = a.n0; n < a.n0 + a.K; ++n) {
        const bool last = n + 1 == a.n0 + a.K;
        // the bits of J are expanded anew every step (the expanded rows would
        // not fit in registers)
#pragma unroll
        for (int q = 0; q < RBW; ++q)
#pragma unroll
            for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(J[q][s].x), "+v"(J[q][s].y), "+v"(J[q][s].z), "+v"(J[q][s].w));
        const float kA_n = kA, d_n = dcur, d_next = dn;
        float jp_n[MB];
#pragma unroll
        for (int b = 0; b < MB; ++b) jp_n[b] = jpn[b];
        if (!last) {   // the next step's scalars load while this step runs
            kA = a.coefA[n + 1];
            dcur = dn;
            dn = a.delta[n + 2];
#pragma unroll
            for (int b = 0; b < MB; ++b) jpn[b] = a.jp[(int64_t)(col[b] / a.R) * a.S + n + 1];
        }
        // the other workgroups' part of the operand
        if (a.G > 1) {
            const uint64_t *src = words(n & 1);
            const uint32_t tag = tag0 + (uint32_t)(n - a.n0) + 1u;
            uint64_t v[U];
            for (int polls = 0;; ++polls) {
                bool ok = true;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if ((need >> u) & 1u) v[u] = get_word(src + u * NT + (uint32_t)tid);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    ok = ok && (((need >> u) & 1u) == 0u || (uint32_t)(v[u] >> 32) == tag);
                if (__all(ok) || stop_waiting(polls, a.err)) break;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if ((need >> u) & 1u) reinterpret_cast<uint32_t *>(op[n & 1])[u * NT + tid] = (uint32_t)v[u];
        }
        __syncthreads();   // step n's operand is whole; step n - 1's reads are done

        f4 acc[RBW][MB];
#pragma unroll
        for (int q = 0; q < RBW; ++q)
#pragma unroll
            for (int b = 0; b < MB; ++b) acc[q][b] = f4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int kc = 4 * s + k;
                if (kc >= nch) continue;
                i8v bv[MB];
#pragma unroll
                for (int b = 0; b < MB; ++b) {
                    const uint4 t = *reinterpret_cast<const uint4 *>(&op[n & 1][(b * nch + kc) * 1024 + lane * 16]);
                    bv[b] = i8v{(int)t.x, (int)t.y, (int)t.z, (int)t.w, 0, 0, 0, 0};
                }
#pragma unroll
                for (int q = 0; q < RBW; ++q) {
                    // bit 4 e + k of dword d: spin 512 s + 128 k + 32 g + 8 d + e, set for -1
                    auto u = [&](uint32_t w) { return (int)(((w << (3 - k)) & 0x88888888u) | 0x22222222u); };
                    const uint4 jw = J[q][s];
                    const i8v av = {u(jw.x), u(jw.y), u(jw.z), u(jw.w), 0, 0, 0, 0};
#pragma unroll
                    for (int b = 0; b < MB; ++b)
                        acc[q][b] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv[b], acc[q][b], 4, 4, 0,
                                                                                     E8M0_ONE, 0, E8M0_ONE);
                }
            }
#pragma unroll
        for (int q = 0; q < RBW; ++q) {
            if (rb0 + q * NWAVE + wave >= nrb) continue;
            f4 xn[MB], yn[MB];
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma clang fp contract(off)
                    float xl, xr;
                    const float xc = x[q][b][e];
                    if constexpr (ROT && MB == 1) {
                        xl = row_rotate<true>(xc);
                        xr = row_rotate<false>(xc);
                    } else if constexpr (ROT) {
                        // two column blocks: the end lanes take the other block's
                        const float l0 = row_rotate<true>(x[q][0][e]), l1 = row_rotate<true>(x[q][1][e]);
                        const float r0 = row_rotate<false>(x[q][0][e]), r1 = row_rotate<false>(x[q][1][e]);
                        xl = (m == 0) ? (b == 0 ? l1 : l0) : (b == 0 ? l0 : l1);
                        xr = (m == 15) ? (b == 0 ? r1 : r0) : (b == 0 ? r0 : r1);
                    } else {
                        const int row = lane & 48;
                        xl = __shfl(x[q][0][e], row | (lsrc[b] & 15));
                        xr = __shfl(x[q][0][e], row | (rsrc[b] & 15));
                        if constexpr (MB == 2) {
                            const float l1 = __shfl(x[q][1][e], row | (lsrc[b] & 15));
                            const float r1 = __shfl(x[q][1][e], row | (rsrc[b] & 15));
                            xl = lsrc[b] >= 16 ? l1 : xl;
                            xr = rsrc[b] >= 16 ? r1 : xr;
                        }
                    }
                    // the diagonal bit reads +1: take f_i back out
                    const float phi = acc[q][b][e] - f_mid(a.fmode, xc, d_n);
                    const float force = (-kA_n * xc + a.kB * (phi + hv[q][e])) + jp_n[b] * (xl + xr);
                    float yv = y[q][b][e] + a.dt * force;
                    float xv = xc + a.kD * yv;
                    if (fabsf(xv) > 1.0f) {
                        xv = xv > 0.0f ? 1.0f : -1.0f;
                        yv = 0.0f;
                    }
                    xn[b][e] = xv;
                    yn[b][e] = yv;
                    f[e] = f_mid(a.fmode, xv, d_next);
                }
                if (!last) emit(n + 1, q, b, f);
            }
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                x[q][b] = xn[b];
                y[q][b] = yn[b];
            }
        }
    }
    // (the barrier of the last step is behind every read of the words)
    if (a.G > 1 && tid == 0) ring_done(a.rings + 2 * grp, a.G, tag0, a.K);
#pragma unroll
    for (int q = 0; q < RBW; ++q) {
        const int rb = rb0 + q * NWAVE + wave;
        if (rb >= nrb) continue;
        const int i4 = 16 * rb + 4 * g;
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            if (!live[b]) continue;
            f4 xv = x[q][b], yv = y[q][b];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i4 + e >= a.N) { xv[e] = 0.0f; yv[e] = 0.0f; }   // padding stays zero
            *reinterpret_cast<f4 *>(a.x + (int64_t)col[b] * a.Np + i4) = xv;
            *reinterpret_cast<f4 *>(a.y + (int64_t)col[b] * a.Np + i4) = yv;
        }
    }
}

// J's bits for the loop from the zero-padded row-major float64 copy: lane l of
// (row block rb, superchunk s) owns the 16 bytes at ((rb * ns + s) * 64 + l);
// bit 4 e + k of its dword d is set where J < 0 at row 16 rb + l % 16, column
// 512 s + 128 k + 32 (l / 16) + 8 d + e.
__global__ __launch_bounds__(256) void k_mid_bits(const double *__restrict__ J64, int N, int Np, int nrb, int ns,
                                                 uint32_t *__restrict__ out) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= nrb * ns * 256) return;
    const int d = q & 3, l = (q >> 2) & 63, s = (q >> 8) % ns, rb = (q >> 8) / ns;
    const int i = 16 * rb + (l & 15);
    uint32_t bits = 0u;
    for (int k = 0; k < 4; ++k)
        for (int e = 0; e < 8; ++e) {
            const int j = 512 * s + 128 * k + 32 * (l >> 4) + 8 * d + e;
            if (i < N && j < N && J64[(int64_t)i * Np + j] < 0.0) bits |= 1u << (4 * e + k);
        }
    out[q] = bits;
}

// The instances that are built: one or two row blocks per wave; four only for
// up to 1024 spins and 16 columns (their registers).
template <class F>
hipError_t with_mid(const MidPlan &p, F &&f) {
    auto by_ring = [&](auto nt, auto rbw, auto ns, auto mb) -> hipError_t {
        constexpr int T = decltype(nt)::value, B = decltype(rbw)::value, S = decltype(ns)::value, M = decltype(mb)::value;
        if (p.rot) return f(&k_dense_mid<T, B, S, M, true>, T);
        return f(&k_dense_mid<T, B, S, M, false>, T);
    };
    auto by_mb = [&](auto nt, auto rbw, auto ns) -> hipError_t {
        constexpr int B = decltype(rbw)::value;
        if (p.MB == 1) return by_ring(nt, rbw, ns, std::integral_constant<int, 1>{});
        if constexpr (B == 1) return by_ring(nt, rbw, ns, std::integral_constant<int, 2>{});
        return hipErrorInvalidValue;
    };
    auto by_ns = [&](auto nt, auto rbw) -> hipError_t {
        switch (p.NS) {
            case 1: return by_mb(nt, rbw, std::integral_constant<int, 1>{});
            case 2: return by_mb(nt, rbw, std::integral_constant<int, 2>{});
            case 4: if constexpr (decltype(rbw)::value <= 2) return by_mb(nt, rbw, std::integral_constant<int, 4>{}); break;
            default: break;
        }
        return hipErrorInvalidValue;
    };
    using I = std::integral_constant<int, 1>;
    using T5 = std::integral_constant<int, 512>;
    using T10 = std::integral_constant<int, 1024>;
    if (p.NT == 512 && p.RBW == 1) return by_ns(T5{}, I{});
    if (p.NT == 1024 && p.RBW == 1) return by_ns(T10{}, I{});
    if (p.NT == 1024 && p.RBW == 2) return by_ns(T10{}, std::integral_constant<int, 2>{});
    if (p.NT == 1024 && p.RBW == 4) return by_ns(T10{}, std::integral_constant<int, 4>{});
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_mid_bits(const double *J64, int N, int Np, int ns, uint4 *out, hipStream_t st) {
    const int nrb = (N + 15) / 16;
    if (N < 1 || N > Np || ns < (N + 511) / 512) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mid_bits, dim3(nrb * ns), dim3(256), 0, st, J64, N, Np, nrb, ns,
                       reinterpret_cast<uint32_t *>(out));
    return hipGetLastError();
}

hipError_t mid_max_blocks(const MidPlan &p, int *blocks_per_cu) {
    return with_mid(p, [&](auto kern, int threads) -> hipError_t {
        return max_blocks_per_cu(reinterpret_cast<const void *>(kern), threads, 0, blocks_per_cu);
    });
}

hipError_t launch_dense_mid(const MidPlan &p, const MidArgs &a, hipStream_t st) {
    const int nrb = (a.N + 15) / 16;
    // every row block has a wave, every column a lane, whole float4 rows
    if (a.N < 1 || a.N > MID_MAX_N || a.N > 512 * p.NS || a.ns < (a.N + 511) / 512 || a.Np % 16 || a.Np < nrb * 16 ||
        p.G < 1 || p.G * (p.NT / 64) * p.RBW < nrb || a.G != p.G || a.groups < 1 || a.R < 1 || a.cols % a.R ||
        a.cols > 16 * p.MB || (int64_t)a.groups * a.cols < a.C || a.K < 1 || a.n0 < 0 || a.n0 + a.K > a.S ||
        (p.rot && (a.R != 16 * p.MB || a.cols != a.R)) || (p.G > 1 && (!a.words || !a.rings)))
        return hipErrorInvalidValue;
    return with_mid(p, [&](auto kern, int threads) -> hipError_t {
        hipLaunchKernelGGL(kern, dim3(a.groups * p.G), dim3(threads), 0, st, a);
        return hipGetLastError();
    });
}

}  // namespace sbqa
