// Dense SBQA kernels for gfx950 (CDNA4, wave64):
//   * one step of the dense path: the coupling sum of Eq. 7 over all runs and
//     replicas, Phi^T[c][i] = sum_j f(X)^T[c][j] J[i][j] (J symmetric, zero
//     diagonal), on MFMA in fp32, e4m3 fp8 or e2m1 fp4 (J as bytes / nibbles
//     or, for J = +-1, one bit per coupling), int8 (integer J) or bf16 hi+lo
//     (three products),
//     with the update of Eqs. 6-7 (pump, Trotter ring, kick, drift, wall) and
//     the next operand f(X) (Eq. 8) fused into its epilogue;
//   * the fp64 energies of spin rows (Eq. 2 at the corners).
// State is replica-major ([C][Np]); the contraction operands are
// fragment-tiled (see sbqa_internal.h).
#include "csr_step.h"

#include <type_traits>
#include <utility>

namespace sbqa {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef int i8v __attribute__((ext_vector_type(8)));
typedef int i4v __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef int i16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

// e4m3 encodings of J = +-1, and e2m1 (fp4) nibbles (sign bit 3, exponent 01,
// mantissa 0).
constexpr uint8_t FP8_P1 = 0x38, FP8_M1 = 0xB8;
constexpr uint32_t FP4_P1 = 0x2, FP4_M1 = 0xA;
// E8M0 block scales 2^(127-127) = 1 and 1/2 of the scaled fp8 and fp4 MFMA.
constexpr int E8M0_ONE = 127, E8M0_HALF = 126;

struct Frag32 { uint4 lo, hi; };  // the 32 K bytes of one lane for a 16x16 block

__device__ __forceinline__ uint4 ld16(const uint8_t *p) { return *reinterpret_cast<const uint4 *>(p); }

template <int PATH> constexpr bool is_fp8 = PATH == PATH_FP8 || PATH == PATH_FP8PK;
template <int PATH> constexpr bool is_fp4 = PATH == PATH_FP4 || PATH == PATH_FP4PK;

// Bit-packed +-1 J: lane l of a fragment owns the dword at 4*l; its bit
// 8*i + k encodes byte i of dword k (k = 0..7) of the lane's 32 fp8 K bytes,
// set for -1. Dword k is then ((w << (7 - k)) & 0x80808080) | e4m3(+1) x 4.
// (in_vgpr: with both constants literal an and-or would be two instructions.)
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v) {
    asm("" : "+v"(v));
    return v;
}
__device__ __forceinline__ Frag32 unpack_pm1(uint32_t w) {
    const uint32_t one = in_vgpr(0x38383838u);
    auto d = [w, one](int k) { return ((w << (7 - k)) & 0x80808080u) | one; };
    return Frag32{make_uint4(d(0), d(1), d(2), d(3)), make_uint4(d(4), d(5), d(6), d(7))};
}

// The same for fp4: a lane owns two dwords (one per 16-byte half of its 32
// bytes = 64 nibbles); bit 4*i + k of a half's dword encodes nibble i of dword
// k (k = 0..3) of that half, set for -1, so dword k is
// ((w << (3 - k)) & 0x88888888) | e2m1(+1) x 8.
__device__ __forceinline__ Frag32 unpack_pm1_fp4(uint2 w) {
    const uint32_t one = in_vgpr(0x22222222u);
    auto d = [one](uint32_t v, int k) { return ((v << (3 - k)) & 0x88888888u) | one; };
    return Frag32{make_uint4(d(w.x, 0), d(w.x, 1), d(w.x, 2), d(w.x, 3)),
                  make_uint4(d(w.y, 0), d(w.y, 1), d(w.y, 2), d(w.y, 3))};
}

// ---------------------------------------------------------------------------
// fp64 energies of spin rows (Eq. 2 at the corners).
// ---------------------------------------------------------------------------
constexpr int ENERGY_SMALL_T = 8;         // spin blocks up to which the latency of K tiles counts
constexpr int LDS_STRIDE = GEMM_KB + 16;  // padded LDS row (bytes): spreads rows over banks
constexpr int TILE_BYTES = GEMM_BM * LDS_STRIDE;
static_assert(GEMM_BM == GEMM_BN, "square block tile assumed by the loaders");

__device__ __forceinline__ Frag32 lds_frag(const uint8_t *tile, int row, int g) {
    const uint8_t *p = tile + row * LDS_STRIDE + g * 32;
    Frag32 f;
    f.lo = *reinterpret_cast<const uint4 *>(p);
    f.hi = *reinterpret_cast<const uint4 *>(p + 16);
    return f;
}

// -1/2 s^T J s of GEMM_BM spin rows at a time, from the lower triangle of the
// symmetric J alone: part[u][c] = -sum over work unit u of s_n (L_n + D_n / 2),
// L_n the sum over the 128-spin blocks below n's and D_n the one over its own.
// A unit is a pair of spin blocks (p, T - 1 - p), so that all units are equally
// long, and one of Z ranges of their K tiles; the sums over n happen here, so that
// no field is written. 8 waves in 2 (rows) x 4 (spins) tiles of 64 x 32,
// K tiles of 16 spins double-buffered in LDS with one barrier each. Bound by
// the fp64 matrix rate: N = 8192, 512 rows 3.5e10 flop in 0.64 ms, 54 of the 70
// TFLOP/s of a large library product (the full product by 4 waves took 1.79 ms:
// twice the flops, and its prefetched operands lived in scratch memory).
// Two workgroups per CU (128 registers); one (185 registers) took 0.75 ms.
// Error (relative 2-norm against 80-bit sums, three seeds of 60 rows): N = 130 1.6e-16, N =
// 1000 3.0e-16, N = 3000 4.1 to 5.0e-16; the full product 2.4, 3.1 and 5.1 to 5.4e-16. Lane group g = lane/16 holds the same 32-byte K slice for
// A and B, so the products pair correctly whatever K order the instruction
// uses in a slice.
__global__ __launch_bounds__(GEMM_THREADS, 4) void k_energy_gemm(const int8_t *__restrict__ S,
                                                              const double *__restrict__ J, int Np, int Cp, int T,
                                                              int Z, double *__restrict__ part) {
    __shared__ __align__(16) uint8_t lds[2][2 * TILE_BYTES];
    __shared__ double red[4 * GEMM_BM];   // per wave along the spins and row
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1, g = lane >> 4, r16 = lane & 15;
    const int p = blockIdx.x / Z, z = blockIdx.x - p * Z, m0 = blockIdx.y * GEMM_BM;
    constexpr int KE = GEMM_KB / 8, KPB = GEMM_BN / KE;   // spins per K tile, K tiles per spin block
    // loader: 4 spins of one row of S, two 16-byte pieces of J's rows
    const int8_t *srow = S + (int64_t)(m0 + (tid >> 2)) * Np + 4 * (tid & 3);
    const int so = (tid >> 2) * LDS_STRIDE + (tid & 3) * 32;
    const int jr = tid >> 3, jc = tid & 7, jo = TILE_BYTES + jr * LDS_STRIDE + jc * 16;
    red[tid] = 0.0;
    // this unit's K tiles: of up to ENERGY_SMALL_T blocks a range of the pair's, the
    // longer block's first; else one of either block's. (Z is a power of two: with 64-bit
    // divisions for the ranges 200 rows of N = 3000 took 192 us, 187 so.)
    const int lz = __builtin_ctz(Z), all = KPB * (T - p) + (2 * p == T - 1 ? 0 : KPB * (p + 1));
    const int r0 = (all * z) >> lz, r1 = (all * (z + 1)) >> lz;
    for (int half = 0; half < 2; ++half) {
        const int t = half == 0 ? T - 1 - p : p;     // the longer block first
        if (half == 1 && t == T - 1 - p) break;      // the middle block of an odd count is alone
        const int nk = KPB * (t + 1), before = half == 0 ? 0 : KPB * (T - p);
        const int k0 = T > ENERGY_SMALL_T ? (nk * z) >> lz : min(max(r0 - before, 0), nk);
        const int k1 = T > ENERGY_SMALL_T ? (nk * (z + 1)) >> lz : min(max(r1 - before, 0), nk);
        if (k0 == k1) continue;
        const int n0 = t * GEMM_BN, kd = KPB * t;    // from K tile kd on: the block's own spins
        const double *jrow = J + (int64_t)(n0 + jr) * Np + 2 * jc;
        d4 acc[4][2];
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = d4{0, 0, 0, 0};
        uint32_t sv = *reinterpret_cast<const uint32_t *>(srow + (int64_t)k0 * KE);
        uint4 j0 = *reinterpret_cast<const uint4 *>(jrow + (int64_t)k0 * KE);
        uint4 j1 = *reinterpret_cast<const uint4 *>(jrow + (int64_t)64 * Np + (int64_t)k0 * KE);
        for (int k = k0; k < k1; ++k) {
            uint8_t *buf = lds[k & 1];
            // (this buffer was last read two K tiles ago, before the last barrier)
            double *sd = reinterpret_cast<double *>(buf + so);
            sd[0] = (double)(int8_t)sv;
            sd[1] = (double)(int8_t)(sv >> 8);
            sd[2] = (double)(int8_t)(sv >> 16);
            sd[3] = (double)(int8_t)(sv >> 24);
            *reinterpret_cast<uint4 *>(buf + jo) = j0;
            *reinterpret_cast<uint4 *>(buf + jo + 64 * LDS_STRIDE) = j1;
            __syncthreads();
            const int kn = k + 1 < k1 ? k + 1 : k;
            sv = *reinterpret_cast<const uint32_t *>(srow + (int64_t)kn * KE);
            j0 = *reinterpret_cast<const uint4 *>(jrow + (int64_t)kn * KE);
            j1 = *reinterpret_cast<const uint4 *>(jrow + (int64_t)64 * Np + (int64_t)kn * KE);
            if (k == kd && k > k0) {   // twice the fields below the block: halved at the end
#pragma unroll
                for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) acc[mb][nb] = acc[mb][nb] + acc[mb][nb];
            }
            Frag32 bf[2];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) bf[nb] = lds_frag(buf + TILE_BYTES, wn * 32 + nb * 16 + r16, g);
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) {
                const Frag32 af = lds_frag(buf, wm * 64 + mb * 16 + r16, g);
                const double *ad = reinterpret_cast<const double *>(&af);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            ad[e], reinterpret_cast<const double *>(&bf[nb])[e], acc[mb][nb], 0, 0, 0);
                // one row block's operand in registers at a time
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // s_n times the fields, over the wave's 32 spins (D[m][n]: column
        // lane%16 of each 16x16 block; register r is row 4*r + lane/16)
        const double w = k1 > kd ? 0.5 : 1.0;
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ml = wm * 64 + mb * 16 + 4 * r + g;
                const int8_t *sn = S + (int64_t)(m0 + ml) * Np + n0 + wn * 32 + r16;
                double v = w * ((double)sn[0] * acc[mb][0][r] + (double)sn[16] * acc[mb][1][r]);
#pragma unroll
                for (int x = 8; x >= 1; x >>= 1) v += __shfl_xor(v, x);
                if (r16 == 0) red[wn * GEMM_BM + ml] += v;
            }
        __syncthreads();   // the last K tiles are read before the next block's are written
    }
    __syncthreads();
    if (tid < GEMM_BM)
        part[(int64_t)blockIdx.x * Cp + m0 + tid] =
            -(((red[tid] + red[GEMM_BM + tid]) + red[2 * GEMM_BM + tid]) + red[3 * GEMM_BM + tid]);
}

// ---------------------------------------------------------------------------
// Operand formats and the fragment-tiled layout.
// ---------------------------------------------------------------------------

// Byte offset of element (row, k) in a fragment-tiled matrix with nkc K chunks
// and groups of G row blocks.
__device__ __forceinline__ int64_t tf_offset(int row, int k, int nkc, int eb, int G) {
    const int kbyte = k * eb;
    const int kc = kbyte >> 7, kb = kbyte & 127, rb = row >> 4;
    const int l = ((kb >> 5) << 4) | (row & 15);
    return (((int64_t)(rb / G) * nkc + kc) * G + rb % G) * FRAG_BYTES + ((kb >> 4) & 1) * 1024 + l * 16 + (kb & 15);
}

// Byte offset of element (row, k) of an operand or J in the path's format
// (fp4: of the byte that holds elements k and k + 1, k even).
template <int PATH>
__device__ __forceinline__ int64_t op_offset(int row, int k, int nkc, int G) {
    if constexpr (is_fp4<PATH>) return tf_offset(row, k >> 1, nkc, 1, G);
    else return tf_offset(row, k, nkc, path_ebytes(Path(PATH)), G);
}

__device__ __forceinline__ float f_value(int fmode, float x, float delta) {
    if (fmode == 2) return x;                       // bSB
    const float d = (fmode == 1) ? 0.0f : delta;    // dSB: sign(0) = 0
    if (fabsf(x) <= d) return 0.0f;
    return x > 0.0f ? 1.0f : -1.0f;
}

__device__ __forceinline__ uint16_t bf16_rne(float v) {
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Operand of the exact paths (ternary f): 2 bits per value, 0 / 01 / 11 for
// 0 / +1 / -1, 16 consecutive K elements to a dword. A lane's 32 K bytes are then
// 8 (fp8, int8) or 16 bytes (fp4), and one shift and mask per dword expands them
// to +-2 (fp8, fp4: the MFMA's block scale halves it) or +-64 (int8: the sum is
// shifted back), which are exact. The reads of a step are mostly operand reads
// and 2 bits are 4 (fp4: 2) times fewer; the split-K step has no other way to
// feed its waves.
// Bit of element 4q + e of a dword's 16: byte e, bits 2q.. for bytes; nibble
// 4 (q % 2) + e, its upper two bits for q < 2, for fp4.
template <int PATH>
__device__ __forceinline__ int op2_bit(int q, int e) {
    if constexpr (is_fp4<PATH>) return 16 * (q & 1) + 4 * e + (q < 2 ? 2 : 0);
    else return 8 * e + 2 * q;
}

// A lane's 32 K bytes of the operand as they lie in memory, and expanded.
template <int PATH> struct OpRaw {
    typedef std::conditional_t<is_fp4<PATH>, uint4, uint2> type;
};
template <> struct OpRaw<PATH_F32> { typedef Frag32 type; };
template <> struct OpRaw<PATH_BF16X3> { typedef Frag32 type; };
template <int PATH> constexpr int OP_LANE = path_op2(Path(PATH)) ? op_frag_bytes(Path(PATH)) / 64 : 16;

template <int PATH>
__device__ __forceinline__ typename OpRaw<PATH>::type load_op(const uint8_t *p) {
    if constexpr (path_op2(Path(PATH))) return *reinterpret_cast<const typename OpRaw<PATH>::type *>(p);
    else return Frag32{ld16(p), ld16(p + 1024)};
}

__device__ __forceinline__ uint4 op2_bytes(uint32_t w) {
    constexpr uint32_t M = 0xC0C0C0C0u;
    return make_uint4((w << 6) & M, (w << 4) & M, (w << 2) & M, w & M);
}
__device__ __forceinline__ uint4 op2_nibbles(uint32_t a, uint32_t b) {
    constexpr uint32_t M = 0xCCCCCCCCu;
    return make_uint4(a & M, (a << 2) & M, b & M, (b << 2) & M);
}
template <int PATH>
__device__ __forceinline__ Frag32 expand_op(const typename OpRaw<PATH>::type &r) {
    if constexpr (is_fp4<PATH>) return Frag32{op2_nibbles(r.x, r.y), op2_nibbles(r.z, r.w)};
    else if constexpr (path_op2(Path(PATH))) return Frag32{op2_bytes(r.x), op2_bytes(r.y)};
    else return r;
}

// Byte offset of the operand's elements (row, k..k+3), k a multiple of 4
// (exact paths: of the dword that holds them).
template <int PATH>
__device__ __forceinline__ int64_t x_offset(int row, int k, int nkc, int G) {
    if constexpr (path_op2(Path(PATH))) {
        constexpr int KPC = path_kpc(Path(PATH)), SL = KPC / 4;   // spins of a chunk, of a lane
        const int kc = k / KPC, kb = k % KPC, rb = row >> 4, l = (kb / SL) * 16 + (row & 15);
        return (((int64_t)(rb / G) * nkc + kc) * G + rb % G) * op_frag_bytes(Path(PATH)) + l * OP_LANE<PATH> +
               (kb % SL) / 16 * 4;
    } else {
        return op_offset<PATH>(row, k, nkc, G);
    }
}

// Four consecutive operand values (same row, K positions k..k+3) at byte
// offset o (from x_offset); the exact paths call it with the lanes 4j..4j+3 of a
// wave holding 16 aligned consecutive values.
template <int PATH>
__device__ __forceinline__ void store_operand(void *g, void *g_lo, int64_t o, float4 f, int fmode) {
    uint8_t *gb = reinterpret_cast<uint8_t *>(g);
    if constexpr (PATH == PATH_F32) {
        *reinterpret_cast<float4 *>(gb + o) = f;
    } else if constexpr (path_op2(Path(PATH))) {
        // the four lanes of 16 consecutive spins add their codes together
        const float v[4] = {f.x, f.y, f.z, f.w};
        const int q = threadIdx.x & 3;
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) w |= (v[e] > 0.0f ? 1u : (v[e] < 0.0f ? 3u : 0u)) << op2_bit<PATH>(q, e);
        w |= (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);   // lanes 1 0 3 2
        w |= (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, true);   // lanes 2 3 0 1
        if (q == 0) *reinterpret_cast<uint32_t *>(gb + o) = w;
    } else {  // BF16X3
        const float v[4] = {f.x, f.y, f.z, f.w};
        uint16_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            hi[e] = bf16_rne(v[e]);
            lo[e] = (fmode == 2) ? bf16_rne(v[e] - bf16_to_f32(hi[e])) : (uint16_t)0;
        }
        uint2 H, L;
        H.x = hi[0] | ((uint32_t)hi[1] << 16);
        H.y = hi[2] | ((uint32_t)hi[3] << 16);
        L.x = lo[0] | ((uint32_t)lo[1] << 16);
        L.y = lo[2] | ((uint32_t)lo[3] << 16);
        *reinterpret_cast<uint2 *>(gb + o) = H;
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint8_t *>(g_lo) + o) = L;
    }
}

// ---------------------------------------------------------------------------
// MFMA terms of one 16x16 block with the 32 K bytes a (operand) and b (J) of
// this lane (a2, b2: bf16 low parts). Term t of T<PATH>::terms; every block
// accumulates its terms in the same order.
// ---------------------------------------------------------------------------
template <int PATH> struct Terms;
template <> struct Terms<PATH_F32> { static constexpr int n = 8; };     // 8 x 16x16x4 f32
template <> struct Terms<PATH_FP8> { static constexpr int n = 1; };     // 1 x 16x16x128 f8f6f4
template <> struct Terms<PATH_FP8PK> { static constexpr int n = 1; };
template <> struct Terms<PATH_BF16X3> { static constexpr int n = 6; };  // lo*hi, hi*lo, hi*hi x 2 halves
template <> struct Terms<PATH_I8> { static constexpr int n = 2; };      // 2 x 16x16x64 i8 (K halves)
template <> struct Terms<PATH_FP4> { static constexpr int n = 2; };     // 2 x 16x16x128 fp4 (K halves)
template <> struct Terms<PATH_FP4PK> { static constexpr int n = 2; };

template <int PATH, int T>
__device__ __forceinline__ void mma_term(f4 &acc, const Frag32 &a, const Frag32 &b, const Frag32 &a2,
                                         const Frag32 &b2) {
    if constexpr (PATH == PATH_F32) {
        const float *af = reinterpret_cast<const float *>(&a);
        const float *bf = reinterpret_cast<const float *>(&b);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af[T], bf[T], acc, 0, 0, 0);
    } else if constexpr (is_fp8<PATH>) {
        i8v av, bv;
        __builtin_memcpy(&av, &a, 32);
        __builtin_memcpy(&bv, &b, 32);
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, acc, 0, 0, 0, E8M0_HALF, 0, E8M0_ONE);
    } else if constexpr (PATH == PATH_I8) {
        // int32 accumulation, carried in the float accumulator's bits; term T
        // takes the lane's K bytes of half T (each 16x16x64 product pairs the
        // same lane bytes of both operands, so the two halves cover the
        // chunk's 128 K exactly once)
        const uint4 &xs = T ? a.hi : a.lo;
        const uint4 &ys = T ? b.hi : b.lo;
        i4v xv, yv;
        __builtin_memcpy(&xv, &xs, 16);
        __builtin_memcpy(&yv, &ys, 16);
        acc = __builtin_bit_cast(f4, __builtin_amdgcn_mfma_i32_16x16x64_i8(xv, yv, __builtin_bit_cast(i4v, acc), 0, 0, 0));
    } else if constexpr (is_fp4<PATH>) {
        // e2m1 operands (format 4 for A and B): term T takes the lane's 16
        // bytes of half T (64 lanes x 32 nibbles = one 16x128 K block each)
        const uint4 &xs = T ? a.hi : a.lo;
        const uint4 &ys = T ? b.hi : b.lo;
        const i8v xv = {(int)xs.x, (int)xs.y, (int)xs.z, (int)xs.w, 0, 0, 0, 0};
        const i8v yv = {(int)ys.x, (int)ys.y, (int)ys.z, (int)ys.w, 0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(xv, yv, acc, 4, 4, 0, E8M0_HALF, 0, E8M0_ONE);
    } else {
        // small products first: lo*hi, hi*lo, then hi*hi; each over both halves
        const Frag32 &x = (T < 2) ? a2 : a;
        const Frag32 &y = (T >= 2 && T < 4) ? b2 : b;
        const uint4 &xs = (T & 1) ? x.hi : x.lo;
        const uint4 &ys = (T & 1) ? y.hi : y.lo;
        bf8v xv, yv;
        __builtin_memcpy(&xv, &xs, 16);
        __builtin_memcpy(&yv, &ys, 16);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, yv, acc, 0, 0, 0);
    }
}

// The 32 x 32 products of the exact paths, rows from a (J), columns from b (the
// operand), with the 32 K bytes of this lane.
template <int PATH>
__device__ __forceinline__ void mma32(f16v &acc, const Frag32 &a, const Frag32 &b) {
    i8v av, bv;
    __builtin_memcpy(&av, &a, 32);
    __builtin_memcpy(&bv, &b, 32);
    const i4v al = {av[0], av[1], av[2], av[3]}, ah = {av[4], av[5], av[6], av[7]};
    const i4v bl = {bv[0], bv[1], bv[2], bv[3]}, bh = {bv[4], bv[5], bv[6], bv[7]};
    if constexpr (is_fp8<PATH>) {
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc, 0, 0, 0, E8M0_ONE, 0, E8M0_HALF);
    } else if constexpr (is_fp4<PATH>) {
        auto wide = [](const i4v &v) { return i8v{v[0], v[1], v[2], v[3], 0, 0, 0, 0}; };
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wide(al), wide(bl), acc, 4, 4, 0, E8M0_ONE, 0, E8M0_HALF);
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wide(ah), wide(bh), acc, 4, 4, 0, E8M0_ONE, 0, E8M0_HALF);
    } else {
        i16v c = __builtin_bit_cast(i16v, acc);
        c = __builtin_amdgcn_mfma_i32_32x32x32_i8(al, bl, c, 0, 0, 0);
        acc = __builtin_bit_cast(f16v, __builtin_amdgcn_mfma_i32_32x32x32_i8(ah, bh, c, 0, 0, 0));
    }
}

template <int PATH> struct Pipe {
    static constexpr int planes = (PATH == PATH_BF16X3) ? 2 : 1;  // bf16: hi and lo
    static constexpr int depth = dense_depth(Path(PATH));          // K chunks in flight
};

// Field value of one accumulator element (int8 path: the exact int32 sum of 64
// times the products, at most 64 * 127 * 65536 < 2^31, shifted back and rounded
// once to float32).
template <int PATH>
__device__ __forceinline__ float acc_field(float v) {
    if constexpr (PATH == PATH_I8) return (float)(__builtin_bit_cast(int, v) >> 6);
    else return v;
}

// f(integral_constant<int, I>) for I = B..E-1, unrolled at compile time.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// ---------------------------------------------------------------------------
// Fused update (Eqs. 6-7 + wall) and operand emission (Eq. 8) for four
// consecutive spins i4..i4+3 of replica column c, with their fields ph. The
// inputs are gathered first (UpdIn) so that a lane can have the loads of all
// its items in flight before the first store.
// The ring neighbours are columns r*R + (k -+ 1 mod R) of the same run.
// ---------------------------------------------------------------------------
struct UpdIn {
    float4 x, xl, xr, y, h;
    float jp;
};

__device__ __forceinline__ void update_load_own(const DenseStepArgs &a, int c, int i4, UpdIn &u) {
    u.x = *reinterpret_cast<const float4 *>(a.x_in + (int64_t)c * a.Np + i4);
    u.y = *reinterpret_cast<const float4 *>(a.y + (int64_t)c * a.Np + i4);
}

__device__ __forceinline__ void update_load_rest(const DenseStepArgs &a, int c, int i4, UpdIn &u) {
    const int Np = a.Np, R = a.R;
    const int r = c / R, kk = c - r * R;
    const int cl = r * R + (kk == 0 ? R - 1 : kk - 1);
    const int cr = r * R + (kk == R - 1 ? 0 : kk + 1);
    u.xl = *reinterpret_cast<const float4 *>(a.x_in + (int64_t)cl * Np + i4);
    u.xr = *reinterpret_cast<const float4 *>(a.x_in + (int64_t)cr * Np + i4);
    u.h = *reinterpret_cast<const float4 *>(a.h + i4);
    u.jp = a.jp[(int64_t)r * a.jp_stride];
}

__device__ __forceinline__ UpdIn update_load(const DenseStepArgs &a, int c, int i4) {
    UpdIn u;
    update_load_own(a, c, i4, u);
    update_load_rest(a, c, i4, u);
    return u;
}

#pragma clang fp contract(off)
template <int PATH, int GM>
__device__ __forceinline__ void update_store(const DenseStepArgs &a, int c, int i4, const UpdIn &u, float4 ph) {
    const StepCoef k = a.k;
    const float xs[4] = {u.x.x, u.x.y, u.x.z, u.x.w}, ls[4] = {u.xl.x, u.xl.y, u.xl.z, u.xl.w};
    const float rs[4] = {u.xr.x, u.xr.y, u.xr.z, u.xr.w}, ys[4] = {u.y.x, u.y.y, u.y.z, u.y.w};
    const float hs[4] = {u.h.x, u.h.y, u.h.z, u.h.w}, ps[4] = {ph.x, ph.y, ph.z, ph.w};
    float xo[4], yo[4], fo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float force = (-k.kA * xs[e] + k.kB * (ps[e] + hs[e])) + u.jp * (ls[e] + rs[e]);
        float yn = ys[e] + k.dt * force;
        float xn = xs[e] + k.kD * yn;
        if (fabsf(xn) > 1.0f) {
            xn = xn > 0.0f ? 1.0f : -1.0f;
            yn = 0.0f;
        }
        if (i4 + e >= a.N) { xn = 0.0f; yn = 0.0f; }  // padding stays zero
        xo[e] = xn;
        yo[e] = yn;
        fo[e] = f_value(a.fmode, xn, k.delta_next);
    }
    const int64_t o = (int64_t)c * a.Np + i4;
    *reinterpret_cast<float4 *>(a.x_out + o) = make_float4(xo[0], xo[1], xo[2], xo[3]);
    *reinterpret_cast<float4 *>(a.y + o) = make_float4(yo[0], yo[1], yo[2], yo[3]);
    store_operand<PATH>(a.g_next, a.g_next_lo, x_offset<PATH>(c, i4, a.nkc, GM ? GM : a.mbw),
                        make_float4(fo[0], fo[1], fo[2], fo[3]), a.fmode);
}
#pragma clang fp contract(on)

// Bit-packed J holds +1 on the diagonal and in the padding: takes the diagonal
// term J'_ii f_i = f_i out of the fields of spins i4.. (fw: the dword of the
// operand this step read) and zeroes those of padded spins, so that their x and
// f stay 0.
template <int PATH>
__device__ __forceinline__ float4 less_diagonal(const DenseStepArgs &a, int i4, uint32_t fw, float4 ph) {
    float v[4] = {ph.x, ph.y, ph.z, ph.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float f = (float)((int)(fw << (30 - op2_bit<PATH>(threadIdx.x & 3, e))) >> 30);
        v[e] = (i4 + e < a.N) ? v[e] - f : 0.0f;
    }
    return make_float4(v[0], v[1], v[2], v[3]);
}

// Epilogue of one wave's tile, row blocks (replica columns) mb0 .. mb0 + MBW
// - 1 by TN spins from n0: transpose each 16 x TN block of Phi through LDS
// (lds: at least 16 x (TN + 4) floats for every wave of the workgroup) so that
// a lane holds 4 consecutive spins of one replica column (f32 MFMA results:
// register r of a lane is row 4*(lane/16) + r, column lane%16); then load
// every input of the lane's items before the first store. GM: row blocks per
// operand group (0: a.mbw).
template <int PATH, int MBW, int EPI, int TN = DENSE_TN, int GM = MBW>
__device__ __forceinline__ void dense_epilogue(const DenseStepArgs &a, f4 (&acc)[MBW][TN / 16], int n0, int mb0,
                                               uint8_t *lds) {
    constexpr int RBT = TN / 16;
    constexpr int TS = TN + 4;
    constexpr bool JPK = path_packed(Path(PATH));
    const int lane = threadIdx.x & 63, wt = threadIdx.x >> 6;
    const int nkc = a.nkc;
    __syncthreads();
    float *T = reinterpret_cast<float *>(lds) + wt * 16 * TS;
    const int g = lane >> 4, r16 = lane & 15;
    constexpr int QPR = TN / 4;               // spin quads per row
    constexpr int ITEMS = 16 * QPR / 64;      // (row, quad) items per lane and m-block
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
#pragma unroll
        for (int p = 0; p < RBT; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r) T[(4 * g + r) * TS + 16 * p + r16] = acc_field<PATH>(acc[mb][p][r]);
        __syncthreads();
        float4 ph[ITEMS];
        int cc[ITEMS], ii[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int flat = it * 64 + lane, row = flat / QPR, q = flat % QPR;
            ph[it] = *reinterpret_cast<const float4 *>(T + row * TS + 4 * q);
            cc[it] = 16 * (mb0 + mb) + row;
            ii[it] = n0 + 4 * q;
        }
        if constexpr (JPK) {
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                if (cc[it] >= a.C) continue;
                const uint32_t fw = *reinterpret_cast<const uint32_t *>(
                    a.g + x_offset<PATH>(cc[it], ii[it], nkc, GM ? GM : a.mbw));
                ph[it] = less_diagonal<PATH>(a, ii[it], fw, ph[it]);
            }
        }
        if constexpr (EPI == EPI_UPDATE) {
            UpdIn u[ITEMS];
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (cc[it] < a.C) u[it] = update_load(a, cc[it], ii[it]);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (cc[it] < a.C) update_store<PATH, GM>(a, cc[it], ii[it], u[it], ph[it]);
        } else {
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
                if (cc[it] < a.C) *reinterpret_cast<float4 *>(a.phi + (int64_t)cc[it] * a.Np + ii[it]) = ph[it];
        }
        __syncthreads();
    }
}


// ---------------------------------------------------------------------------
// One dense step. Workgroup tile: DENSE_TN = 64 spins (4 row blocks of J) x
// 64*MBW replica columns. Wave w owns m-blocks [w*MBW, (w+1)*MBW) of the
// column chunk and all 4 J row blocks: every J fragment is read once per step
// and column chunk, shared by the 4 waves through a double-buffered LDS slot
// (wave w stages row block w), while each wave streams its own operand
// fragments straight into registers, Pipe::depth K chunks ahead. reverse = 1
// walks K backwards: alternating the direction every step starts each step on
// the J chunks the previous one touched last.
// ---------------------------------------------------------------------------
// CG column groups of 4 waves share the tile's J staging (CG = 2: a
// 64-spin x 128*MBW-column workgroup of 8 waves reads every J fragment once
// for twice the columns; with two J planes, group cg stages plane cg).
template <int PATH, int MBW, int EPI, int CG = 1>
__device__ __forceinline__ void dense_step_body(const DenseStepArgs &a, int nt, int mchunk_wg) {
    constexpr int PL = Pipe<PATH>::planes;
    constexpr int PD = Pipe<PATH>::depth;
    constexpr int NT = Terms<PATH>::n;
    constexpr int RBT = DENSE_TN / 16;          // J row blocks per tile
    constexpr int SLOT = PL * RBT * FRAG_BYTES;  // J fragments of one K chunk
    constexpr int TS = DENSE_TN + 4;             // epilogue transpose row stride (floats)
    constexpr int TBYTES = 4 * CG * 16 * TS * 4;
    constexpr int LDS_BYTES = (2 * SLOT > TBYTES) ? 2 * SLOT : TBYTES;
    static_assert(CG == 1 || (CG == 2 && PL == 2), "two column groups split the two J planes");
    __shared__ __align__(16) uint8_t lds[LDS_BYTES];

    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, w = wv & 3, cg = wv >> 2;
    const int mchunk = mchunk_wg * CG + cg;       // this wave's 64*MBW-column chunk
    const int n0 = nt * DENSE_TN;
    const int mb0 = (mchunk * 4 + w) * MBW;       // first m-block of this wave
    const int nkc = a.nkc;
    const int l16 = lane * 16;
    constexpr bool JPK = path_packed(Path(PATH));   // J as one bit per coupling
    constexpr int JFRAG = JPK ? pk_frag_bytes(Path(PATH)) : FRAG_BYTES;
    using JWord = std::conditional_t<is_fp4<PATH>, uint2, uint32_t>;   // a lane's packed J of one chunk
    constexpr int JCH = RBT * JFRAG;        // J bytes of one tile and K chunk
    constexpr int XF = op_frag_bytes(Path(PATH));
    constexpr int XCH = MBW * XF;           // operand bytes of one wave and K chunk

    // this wave stages J row block w of tile nt (both planes); its operand
    // group is m-blocks mb0..mb0+MBW-1
    const int64_t jgrp = (int64_t)nt * nkc * JCH + w * JFRAG + (JPK ? lane * (int)sizeof(JWord) : l16);
    const int64_t xgrp = (int64_t)(mchunk * 4 + w) * nkc * XCH + lane * OP_LANE<PATH>;
    const uint8_t *jsrc = a.J + jgrp;
    const uint8_t *jsrc_lo = (PL == 2) ? a.J_lo + jgrp : jsrc;
    const uint8_t *xsrc = a.g + xgrp;
    const uint8_t *xsrc_lo = (PL == 2) ? a.g_lo + xgrp : xsrc;

    uint4 jr[JPK ? 1 : PD][PL][2];
    JWord jw[JPK ? PD : 1];
    typename OpRaw<PATH>::type xr[PD][MBW][PL];
    f4 acc[MBW][RBT];
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < RBT; ++j) acc[i][j] = f4{0, 0, 0, 0};

    const int rev = a.reverse;
    auto chunk_at = [&](int kc) -> int64_t { return rev ? nkc - 1 - kc : kc; };
    auto load_j = [&](int s, int kc) {
        const int64_t o = chunk_at(kc) * JCH;
        if constexpr (JPK) {
            jw[s] = *reinterpret_cast<const JWord *>(jsrc + o);
        } else if constexpr (CG == 2) {
            const uint8_t *src = cg ? jsrc_lo : jsrc;
            jr[s][0][0] = ld16(src + o);
            jr[s][0][1] = ld16(src + o + 1024);
        } else {
            jr[s][0][0] = ld16(jsrc + o);
            jr[s][0][1] = ld16(jsrc + o + 1024);
            if constexpr (PL == 2) {
                jr[s][PL - 1][0] = ld16(jsrc_lo + o);
                jr[s][PL - 1][1] = ld16(jsrc_lo + o + 1024);
            }
        }
    };
    auto load_x = [&](typename OpRaw<PATH>::type (&d)[MBW][PL], int kc) {
        const int64_t o = chunk_at(kc) * XCH;
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
            d[mb][0] = load_op<PATH>(xsrc + o + mb * XF);
            if constexpr (PL == 2) d[mb][PL - 1] = load_op<PATH>(xsrc_lo + o + mb * XF);
        }
    };

    // nkc is a multiple of PD (the host pads N accordingly). Every chunk
    // issues the same loads (the last PD chunks re-read their own chunk
    // instead of prefetching past the end), so the memory counters the
    // compiler waits on are exact and the loop body has no branches; the
    // prologue issues its loads in the loop's order, J then operand per chunk.
#pragma unroll
    for (int s = 0; s < PD; ++s) {
        load_j(s, s);
        __builtin_amdgcn_sched_barrier(0);
        load_x(xr[s], s);
        __builtin_amdgcn_sched_barrier(0);
    }

#pragma unroll 1
    for (int kc0 = 0; kc0 < nkc; kc0 += PD) {
#pragma unroll
        for (int s = 0; s < PD; ++s) {
            const int kc = kc0 + s;
            const int kn = (kc + PD < nkc) ? kc + PD : kc;
            uint8_t *slot = lds + (kc & 1) * SLOT;
            // publish this wave's J fragment of chunk kc (bit-packed J is
            // expanded to e4m3 bytes here); slot (kc & 1) was last read in
            // chunk kc - 2, which every wave finished before the barrier of
            // chunk kc - 1
            if constexpr (JPK) {
                Frag32 f;
                if constexpr (is_fp4<PATH>) f = unpack_pm1_fp4(jw[s]);
                else f = unpack_pm1(jw[s]);
                uint8_t *dst = slot + w * FRAG_BYTES + l16;
                *reinterpret_cast<uint4 *>(dst) = f.lo;
                *reinterpret_cast<uint4 *>(dst + 1024) = f.hi;
            } else if constexpr (CG == 2) {
                uint8_t *dst = slot + (cg * RBT + w) * FRAG_BYTES + l16;
                *reinterpret_cast<uint4 *>(dst) = jr[s][0][0];
                *reinterpret_cast<uint4 *>(dst + 1024) = jr[s][0][1];
            } else {
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) {
                    uint8_t *dst = slot + (pl * RBT + w) * FRAG_BYTES + l16;
                    *reinterpret_cast<uint4 *>(dst) = jr[s][pl][0];
                    *reinterpret_cast<uint4 *>(dst + 1024) = jr[s][pl][1];
                }
            }
            load_j(s, kn);
            __syncthreads();
            // J fragments of the 4 row blocks, two in registers at a time
            Frag32 bjb[2][PL];
            auto read_j = [&](Frag32 (&d)[PL], int p) {
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) {
                    d[pl].lo = *reinterpret_cast<const uint4 *>(slot + (pl * RBT + p) * FRAG_BYTES + l16);
                    d[pl].hi = *reinterpret_cast<const uint4 *>(slot + (pl * RBT + p) * FRAG_BYTES + 1024 + l16);
                }
            };
            read_j(bjb[0], 0);
            Frag32 ax[MBW], ax2[MBW];
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb) {
                ax[mb] = expand_op<PATH>(xr[s][mb][0]);
                ax2[mb] = expand_op<PATH>(xr[s][mb][PL - 1]);
            }
#pragma unroll
            for (int p = 0; p < RBT; ++p) {
                if (p + 1 < RBT) read_j(bjb[(p + 1) & 1], p + 1);
                const Frag32 &bj = bjb[p & 1][0], &bj2 = bjb[p & 1][PL - 1];
                // term-major order: consecutive MFMAs go to different blocks
                static_for<0, NT>([&](auto tc) {
                    constexpr int T = decltype(tc)::value;
#pragma unroll
                    for (int mb = 0; mb < MBW; ++mb) mma_term<PATH, T>(acc[mb][p], ax[mb], bj, ax2[mb], bj2);
                });
                // keeps the fragment reads two row blocks deep (register pressure)
                __builtin_amdgcn_sched_barrier(0);
            }
            load_x(xr[s], kn);
        }
    }

    dense_epilogue<PATH, MBW, EPI>(a, acc, n0, mb0, lds);
}

template <int PATH, int MBW, int EPI>
__global__ __launch_bounds__(DENSE_THREADS) void k_dense_step(const DenseStepArgs a) {
    dense_step_body<PATH, MBW, EPI>(a, blockIdx.x, blockIdx.y);
}

// The same step with two column groups per workgroup (two J planes, each
// staged by one group): grid (Np / DENSE_TN, Cg / (128 * MBW)).
template <int PATH, int MBW, int EPI>
__global__ __launch_bounds__(2 * DENSE_THREADS) void k_dense_step_cg2(const DenseStepArgs a) {
    dense_step_body<PATH, MBW, EPI, 2>(a, blockIdx.x, blockIdx.y);
}

// The same step for small grids: a wave owns 16 replica columns x 16*NB spins
// and streams both operands straight into registers, PD K chunks ahead, with
// no LDS and no barrier in the K loop; the 4 waves of a workgroup take 4
// column blocks of the same spins, so that J is fetched into the CU's L1 once.
// Every field sums the same terms in the same order as in k_dense_step. Bound
// by the chain of MFMAs into one accumulator (fp32, N = 1500: 384 of 32 cycles,
// 5.1 us of the 10.3 us a step takes; four such chains, LDS and barriers in the
// 64-spin tile 32.2), then by the L1 fill.
template <int PATH, int NB, int PD, int EPI>
__device__ __forceinline__ void dense_fine_body(const DenseStepArgs &a, int bx, int by) {
    constexpr int PL = Pipe<PATH>::planes;
    constexpr int NT = Terms<PATH>::n;
    constexpr int RBG = DENSE_TN / 16;            // row blocks per J group
    constexpr bool JPK = path_packed(Path(PATH));
    constexpr int JFRAG = JPK ? pk_frag_bytes(Path(PATH)) : FRAG_BYTES;
    using JWord = std::conditional_t<is_fp4<PATH>, uint2, uint32_t>;
    __shared__ __align__(16) uint8_t lds[4 * 16 * (16 * NB + 4) * 4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int mb = by * 4 + w, rb0 = bx * NB, nkc = a.nkc, l16 = lane * 16;
    const int xstep = a.mbw * op_frag_bytes(Path(PATH));
    const int64_t xo = (int64_t)(mb / a.mbw) * nkc * xstep + (mb % a.mbw) * op_frag_bytes(Path(PATH)) +
                       lane * OP_LANE<PATH>;
    const uint8_t *xsrc = a.g + xo, *xsrc_lo = (PL == 2) ? a.g_lo + xo : xsrc;
    const uint8_t *jsrc[NB], *jsrc_lo[NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) {
        const int rb = rb0 + p;
        const int64_t jo = (int64_t)(rb / RBG) * nkc * (RBG * JFRAG) + (rb % RBG) * JFRAG +
                           (JPK ? lane * (int)sizeof(JWord) : l16);
        jsrc[p] = a.J + jo;
        jsrc_lo[p] = (PL == 2) ? a.J_lo + jo : jsrc[p];
    }
    const int rev = a.reverse;
    auto chunk_at = [&](int kc) -> int64_t { return rev ? nkc - 1 - kc : kc; };
    typename OpRaw<PATH>::type xr[PD][PL];
    uint4 jr[JPK ? 1 : PD][NB][PL][2];
    JWord jw[JPK ? PD : 1][NB];
    auto load = [&](int s, int kc) {
        const int64_t k = chunk_at(kc);
#pragma unroll
        for (int p = 0; p < NB; ++p) {
            if constexpr (JPK) {
                jw[s][p] = *reinterpret_cast<const JWord *>(jsrc[p] + k * (RBG * JFRAG));
            } else {
                jr[s][p][0][0] = ld16(jsrc[p] + k * (RBG * JFRAG));
                jr[s][p][0][1] = ld16(jsrc[p] + k * (RBG * JFRAG) + 1024);
                if constexpr (PL == 2) {
                    jr[s][p][PL - 1][0] = ld16(jsrc_lo[p] + k * (RBG * JFRAG));
                    jr[s][p][PL - 1][1] = ld16(jsrc_lo[p] + k * (RBG * JFRAG) + 1024);
                }
            }
        }
        xr[s][0] = load_op<PATH>(xsrc + k * xstep);
        if constexpr (PL == 2) xr[s][PL - 1] = load_op<PATH>(xsrc_lo + k * xstep);
    };
    f4 acc[1][NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) acc[0][p] = f4{0, 0, 0, 0};
    // nkc is a multiple of PD; the last PD chunks load their own chunk again
    // instead of the next, so that every chunk issues the same loads. A wave
    // whose 16 columns are all padding has no chunks.
    const int nk = 16 * mb < a.C ? nkc : 0;
#pragma unroll
    for (int s = 0; s < PD; ++s) {
        load(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll 1
    for (int kc0 = 0; kc0 < nk; kc0 += PD) {
#pragma unroll
        for (int s = 0; s < PD; ++s) {
            const int kc = kc0 + s;
            const Frag32 ax = expand_op<PATH>(xr[s][0]), ax2 = expand_op<PATH>(xr[s][PL - 1]);
            Frag32 bj[NB], bj2[NB];
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                if constexpr (JPK) {
                    if constexpr (is_fp4<PATH>) bj[p] = unpack_pm1_fp4(jw[s][p]);
                    else bj[p] = unpack_pm1(jw[s][p]);
                    bj2[p] = bj[p];
                } else {
                    bj[p] = Frag32{jr[s][p][0][0], jr[s][p][0][1]};
                    bj2[p] = Frag32{jr[s][p][PL - 1][0], jr[s][p][PL - 1][1]};
                }
            }
            static_for<0, NT>([&](auto tc) {
                constexpr int T = decltype(tc)::value;
#pragma unroll
                for (int p = 0; p < NB; ++p) mma_term<PATH, T>(acc[0][p], ax, bj[p], ax2, bj2[p]);
            });
            __builtin_amdgcn_sched_barrier(0);
            load(s, kc + PD < nkc ? kc + PD : kc);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    dense_epilogue<PATH, 1, EPI, 16 * NB, 0>(a, acc, rb0 * 16, mb, lds);
}

template <int PATH, int NB, int PD, int EPI>
__global__ __launch_bounds__(DENSE_THREADS) void k_dense_step_fine(const DenseStepArgs a) {
    dense_fine_body<PATH, NB, PD, EPI>(a, blockIdx.x, blockIdx.y);
}

// One step with K split over the waves, for the exact contractions
// (integer-valued sums: the order does not change the result). A wave owns 64
// spins x 64 replica columns and one of KS ranges of K, and streams both operands
// straight into registers: no LDS and no barrier in the K loop. A workgroup of 8
// waves is SG spin groups x CG column groups x KS ranges; the ranges' sums are
// added through LDS, and each wave then updates 1/KS of its tile's columns.
// Workgroups are numbered so that the column tiles of one J tile run on one XCD
// and read J from its L2.
// Expanding J and the operand takes about as many vector instructions as the
// products leave room for, and the two overlap only beside 32 x 32 products: on
// one SIMD, 32 16x16x128 fp4 products with 4 vector instructions each take 981 x 2
// clocks, 16 32x32x64 products of the same work with 7 each 682 x 2. Then the
// epilogue's state traffic at the end of a launch. us per step, the better of the
// 64-spin and the fine tile / split-K, N x C (launches back to back):
//                16384 x 256  16384 x 128  8192 x 256   8192 x 128   4096 x 256
//   fp4, 1 bit   51.0 / 41.4  33.3 / 25.3  20.6 / 17.7  13.9 / 11.4  10.3 /  8.8
//   fp8, 1 bit   72.7 / 58.5  53.7 / 33.4  31.8 / 22.1  21.3 / 13.0  13.9 / 10.2
//   int8         88.1 / 89.0  58.6 / 50.7  28.2 / 25.8  21.6 / 16.7  14.2 / 11.1
// (default_dense_form has the sizes where the tiles are faster)
template <int PATH, int SG, int CG, int EPI>
__global__ __launch_bounds__(2 * DENSE_THREADS) void k_dense_step_sk(const DenseStepArgs a, int nx, int ny) {
    constexpr int KS = 8 / (SG * CG), MB = 4, RB = DENSE_TN / 16;
    constexpr bool JPK = path_packed(Path(PATH));
    constexpr int PD = JPK && KS > 2 ? 4 : 2;   // K chunks in flight
    constexpr int JFRAG = JPK ? pk_frag_bytes(Path(PATH)) : FRAG_BYTES, JCH = RB * JFRAG;
    constexpr int XF = op_frag_bytes(Path(PATH));
    using JRaw = std::conditional_t<JPK, std::conditional_t<is_fp4<PATH>, uint2, uint32_t>, Frag32>;
    __shared__ __align__(16) f4 red[8 * MB * RB * 64];

    const int slot = blockIdx.x >> 3, bx = (slot / ny) * 8 + (blockIdx.x & 7), by = slot % ny;
    if (bx >= nx) return;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kp = wv / (SG * CG), t = wv % (SG * CG), jt = bx * SG + t % SG, mb0 = (by * CG + t / SG) * MB;
    const int nkc = a.nkc, rev = a.reverse, xstep = a.mbw * XF;
    // A lane's operand of a 32 x 32 product is the share of lane sl(T) of a
    // 16-row fragment, T = 0, 1: rows 16q.. of a fragment pair (q = lane / 16 %
    // 2), K slice 2T + lane / 32. Scalar bases and chunk offsets, the lane's part
    // 32 bits.
    const uint32_t sl = (lane & 15) + 16 * (lane >> 5), q = (lane >> 4) & 1;
    constexpr int JL = JPK ? (int)sizeof(JRaw) : 16, XL = OP_LANE<PATH>;
    const uint8_t *jsrc = a.J + (int64_t)jt * nkc * JCH;
    const uint32_t jl = q * JFRAG + sl * JL;
    // row blocks 2m and 2m + 1 of the operand: one group's, or (mbw 1) two
    const uint8_t *xsrc[2];
    const uint32_t xl = (a.mbw == 1 ? q * (uint32_t)nkc * XF : q * XF) + sl * XL;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int mb = mb0 + 2 * m;
        xsrc[m] = a.g + (int64_t)(mb / a.mbw) * nkc * xstep + (mb % a.mbw) * XF;
    }
    // this wave's chunks; none where its 64 columns are all padding
    const int k0 = kp * nkc / KS, k1 = 16 * mb0 < a.C ? (kp + 1) * nkc / KS : k0;
    JRaw jr[PD][2][2];
    typename OpRaw<PATH>::type xr[PD][2][2];
    auto load = [&](int s, int kc) {
        const int k = rev ? nkc - 1 - kc : kc;
        const uint8_t *src = jsrc + (int64_t)k * JCH;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                const uint8_t *at = src + (2 * p * JFRAG + 32 * T * JL) + jl;
                if constexpr (JPK) jr[s][p][T] = *reinterpret_cast<const JRaw *>(at);
                else jr[s][p][T] = Frag32{ld16(at), ld16(at + 1024)};
            }
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int T = 0; T < 2; ++T) xr[s][m][T] = load_op<PATH>(xsrc[m] + (int64_t)k * xstep + 32 * T * XL + xl);
    };
    // This wave's items after the sum over the KS ranges: 64 / KS columns, a lane
    // four spins of every fourth. Their x and y are on the way during the K loop
    // where registers allow (8 items would spill).
    constexpr int IT = 16 / KS;
    constexpr bool EARLY = KS > 2;
    const int cw = (64 / KS) * kp + (lane >> 4), i4 = jt * DENSE_TN + 4 * (lane & 15);
    auto item_c = [&](int it) { return 16 * mb0 + cw + 4 * it; };
    UpdIn u[IT];
    f16v acc[2][2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][p][e] = 0.0f;
    auto compute = [&](int s) {
#pragma unroll
        for (int T = 0; T < 2; ++T) {
            Frag32 ax[2], bj[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) ax[m] = expand_op<PATH>(xr[s][m][T]);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if constexpr (!JPK) bj[p] = jr[s][p][T];
                else if constexpr (is_fp4<PATH>) bj[p] = unpack_pm1_fp4(jr[s][p][T]);
                else bj[p] = unpack_pm1(jr[s][p][T]);
            }
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int m = 0; m < 2; ++m) mma32<PATH>(acc[m][p], bj[p], ax[m]);
        }
    };
    if (k0 < k1) {
#pragma unroll
        for (int s = 0; s < PD; ++s) {
            load(s, min(k0 + s, k1 - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (EPI == EPI_UPDATE && EARLY) {
#pragma unroll
            for (int it = 0; it < IT; ++it)
                if (item_c(it) < a.C) update_load_own(a, item_c(it), i4, u[it]);
        }
        __builtin_amdgcn_sched_barrier(0);
        int kc = k0;
#pragma unroll 1
        for (; kc + PD <= k1; kc += PD) {
#pragma unroll
            for (int s = 0; s < PD; ++s) {
                compute(s);
                __builtin_amdgcn_sched_barrier(0);
                load(s, min(kc + s + PD, k1 - 1));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < PD - 1; ++s)
            if (kc + s < k1) compute(s);
    }
    // Add the KS ranges through LDS. Registers 4e.. of a lane of product (p, m) are
    // spins 32p + 8e + 4 (lane / 32).. of column 32m + lane % 32: four consecutive
    // spins go to row `column`, place (spin / 4) ^ (column % 16) of the wave's share,
    // so that neither writes nor reads meet on a bank.
    // The rest of the items' inputs arrives meanwhile (of 8 items, half before and
    // half after the sums have left their registers).
    uint32_t fw[IT];
    auto fetch = [&](int it) {
        if (item_c(it) >= a.C) return;
        if constexpr (EPI == EPI_UPDATE) {
            if (!EARLY || k0 == k1) update_load_own(a, item_c(it), i4, u[it]);
            update_load_rest(a, item_c(it), i4, u[it]);
        }
        if constexpr (JPK) fw[it] = *reinterpret_cast<const uint32_t *>(a.g + x_offset<PATH>(item_c(it), i4, nkc, a.mbw));
    };
    constexpr int BEFORE = IT < 4 ? IT : 4;
#pragma unroll
    for (int it = 0; it < BEFORE; ++it) fetch(it);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f16v &v = acc[m][p];
                const int col = 32 * m + (lane & 31), quad = 8 * p + 2 * e + (lane >> 5);
                red[((kp * SG * CG + t) * 64 + col) * 16 + (quad ^ (col & 15))] =
                    f4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
            }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = BEFORE; it < IT; ++it) fetch(it);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int c = item_c(it), col = cw + 4 * it;
        if (c >= a.C) continue;
        const f4 *src = red + (t * 64 + col) * 16 + ((lane & 15) ^ (col & 15));
        f4 v = src[0];
#pragma unroll
        for (int r = 1; r < KS; ++r) {
            const f4 o = src[r * SG * CG * 1024];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (PATH == PATH_I8) v[e] = __int_as_float(__float_as_int(v[e]) + __float_as_int(o[e]));
                else v[e] += o[e];
            }
        }
        float4 ph = make_float4(acc_field<PATH>(v[0]), acc_field<PATH>(v[1]), acc_field<PATH>(v[2]), acc_field<PATH>(v[3]));
        if constexpr (JPK) ph = less_diagonal<PATH>(a, i4, fw[it], ph);
        if constexpr (EPI == EPI_UPDATE) update_store<PATH, 0>(a, c, i4, u[it], ph);
        else *reinterpret_cast<float4 *>(a.phi + (int64_t)c * a.Np + i4) = ph;
    }
}

// J in the contraction precision, fragment-tiled (groups of DENSE_TN/16 row
// blocks), from the zero-padded row-major float64 copy: one thread per 4
// consecutive K elements of a row. e4m3 for ternary J, int8 for integer J
// with |J| <= 127 (both validated on the host), float32 round-to-nearest, or
// bf16 hi = rne(J), lo = rne(J - hi) in float64.
template <int PATH>
__global__ __launch_bounds__(256) void k_convert_j(const double *__restrict__ J64, int Np, int nkc,
                                                   uint8_t *__restrict__ Jd, uint8_t *__restrict__ Jd_lo) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nq = (int64_t)Np * (Np / 4);
    if (q >= nq) return;
    const int row = (int)(q / (Np / 4)), k4 = (int)(q % (Np / 4)) * 4;
    const double *src = J64 + (int64_t)row * Np + k4;
    const int64_t o = op_offset<PATH>(row, k4, nkc, DENSE_TN / 16);
    if constexpr (PATH == PATH_F32) {
        *reinterpret_cast<float4 *>(Jd + o) = make_float4((float)src[0], (float)src[1], (float)src[2], (float)src[3]);
    } else if constexpr (PATH == PATH_FP8) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t b = src[e] > 0.0 ? FP8_P1 : (src[e] < 0.0 ? FP8_M1 : 0u);
            w |= b << (8 * e);
        }
        *reinterpret_cast<uint32_t *>(Jd + o) = w;
    } else if constexpr (PATH == PATH_I8) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) w |= ((uint32_t)(int32_t)src[e] & 0xFFu) << (8 * e);
        *reinterpret_cast<uint32_t *>(Jd + o) = w;
    } else if constexpr (PATH == PATH_FP4) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) w |= (src[e] > 0.0 ? FP4_P1 : (src[e] < 0.0 ? FP4_M1 : 0u)) << (4 * e);
        *reinterpret_cast<uint16_t *>(Jd + o) = (uint16_t)w;
    } else {
        uint16_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            hi[e] = bf16_rne((float)src[e]);
            lo[e] = bf16_rne((float)(src[e] - (double)bf16_to_f32(hi[e])));
        }
        *reinterpret_cast<uint2 *>(Jd + o) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
        *reinterpret_cast<uint2 *>(Jd_lo + o) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
    }
}

// Bit-packed +-1 J (layouts of unpack_pm1 / unpack_pm1_fp4), fragment-tiled
// like the byte copy (groups of DENSE_TN/16 row blocks): one thread per
// (fragment, lane, dword), consecutive threads write consecutive dwords. A bit
// is set where J_ij < 0; the diagonal and the padding read 0 and so hold +1
// (the step's epilogue removes both). `neg(i, j)` tells whether J_ij < 0 for
// i, j < Np: from the zero-padded float64 copy, or from row-major sign bits.
template <bool FP4, class Neg>
__device__ __forceinline__ void convert_j_pk(int Np, int nkc, uint32_t *__restrict__ Jd, Neg neg) {
    constexpr int RBT = DENSE_TN / 16, DW = FP4 ? 2 : 1;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (int64_t)(Np / 16) * nkc * 64 * DW) return;
    const int d = (int)(q % DW), lane = (int)((q / DW) & 63);
    const int64_t frag = q / DW / 64;
    const int w = (int)(frag % RBT);
    const int64_t t = frag / RBT;
    const int kc = (int)(t % nkc), rb = (int)(t / nkc) * RBT + w;
    const int g = lane >> 4;
    const int i = 16 * rb + (lane & 15);
    uint32_t bits = 0;
    if constexpr (FP4) {
        // half d: K = 256 kc + 64 g + 32 d + 8 k + i for nibble i of dword k
        const int j0 = 256 * kc + 64 * g + 32 * d;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (neg(i, j0 + 8 * k + e)) bits |= 1u << (4 * e + k);
    } else {
        // byte b = 4 k + e of the lane's 32: K = 128 kc + 32 g + 16 (b / 16) + b % 16
        const int j0 = 128 * kc + 32 * g;
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int bb = 4 * k + e;
                if (neg(i, j0 + 16 * (bb >> 4) + (bb & 15))) bits |= 1u << (8 * e + k);
            }
    }
    Jd[q] = bits;
}

template <bool FP4>
__global__ __launch_bounds__(256) void k_convert_j_pk(const double *__restrict__ J64, int Np, int nkc,
                                                     uint32_t *__restrict__ Jd) {
    convert_j_pk<FP4>(Np, nkc, Jd, [&](int i, int j) { return J64[(int64_t)i * Np + j] < 0.0; });
}

// From row-major sign bits of an N x N matrix (bit j % 32 of word
// i * words + j / 32 set where J_ij < 0); rows and columns past N read +1.
template <bool FP4>
__global__ __launch_bounds__(256) void k_convert_j_pk_bits(const uint32_t *__restrict__ sb, int N, int words, int Np,
                                                          int nkc, uint32_t *__restrict__ Jd) {
    convert_j_pk<FP4>(Np, nkc, Jd, [&](int i, int j) {
        return i < N && j < N && ((sb[(int64_t)i * words + (j >> 5)] >> (j & 31)) & 1u) != 0u;
    });
}

// Calls step(args, block of the task) for the virtual blocks blockIdx.x,
// blockIdx.x + stride, ...
template <class F>
__device__ __forceinline__ void group_blocks(const GroupHeader *hdr, const GroupTask *tasks, int offset, int stride,
                                             F &&step) {
    const int ntask = hdr->ntask, total = hdr->total_blocks;
    for (int vb = blockIdx.x; vb < total; vb += stride) {
        int q = 0;
        while (q + 1 < ntask && tasks[q + 1].first_block <= vb) ++q;
        const GroupTask &t = tasks[q];
        const int n = t.n_base + offset;
        if (n >= t.n_end) continue;
        const int in = n & 1;
        DenseStepArgs a;
        a.N = t.N;
        a.Np = t.ld;
        a.R = t.R;
        a.C = t.C;
        a.nkc = t.nkc;
        a.mbw = t.mbw;
        a.reverse = in;
        a.J = static_cast<const uint8_t *>(t.J);
        a.J_lo = static_cast<const uint8_t *>(t.J_lo);
        a.g = static_cast<const uint8_t *>(t.g[in]);
        a.g_lo = static_cast<const uint8_t *>(t.g_lo[in]);
        a.g_next = static_cast<uint8_t *>(t.g[1 - in]);
        a.g_next_lo = static_cast<uint8_t *>(t.g_lo[1 - in]);
        a.h = t.h;
        a.x_in = t.x[in];
        a.x_out = t.x[1 - in];
        a.y = t.y;
        a.phi = nullptr;
        a.jp = t.jp + n;
        a.jp_stride = t.S;
        a.k.kA = t.coefA[n];
        a.k.kB = t.kB;
        a.k.dt = t.dt;
        a.k.kD = t.kD;
        a.k.delta_next = t.delta[n + 1];
        a.fmode = t.fmode;
        const int lt = vb - t.first_block;
        step(a, lt % t.nchunk, lt / t.nchunk);
    }
}

// Grouped step of every dense instance of one serving group (same path and
// m-blocks per wave): a grid-stride loop over the tiles of all tasks (task q
// owns virtual blocks [first, first + nblocks), nchunk spin tiles per column
// chunk), each running exactly the workgroup of the standalone kernel for the
// task's step n = n_base + offset; tasks past their last step skip.
template <int PATH, int MBW>
__global__ __launch_bounds__(DENSE_THREADS) void k_group_dense(const GroupHeader *__restrict__ hdr,
                                                               const GroupTask *__restrict__ tasks, int offset) {
    group_blocks(hdr, tasks, offset, gridDim.x,
                 [](const DenseStepArgs &a, int bx, int by) { dense_step_body<PATH, MBW, EPI_UPDATE>(a, bx, by); });
}

// The same with the fine tiles (tasks whose nchunk counts tiles of 16 * NB
// spins) in the first ndense workgroups; those behind step the sparse tasks
// (ternary f, ring by lane reads) of chdr/ctasks.
template <int PATH, int NB>
__global__ __launch_bounds__(DENSE_THREADS) void k_group_dense_fine(const GroupHeader *__restrict__ hdr,
                                                                    const GroupTask *__restrict__ tasks, int ndense,
                                                                    const GroupHeader *__restrict__ chdr,
                                                                    const GroupTask *__restrict__ ctasks,
                                                                    int offset) {
    if ((int)blockIdx.x >= ndense) {
        csr::csr_group_blocks<false, true>(chdr, ctasks, offset, blockIdx.x - ndense, gridDim.x - ndense);
        return;
    }
    // the chunk count of every instance is a multiple of it (dense_pad)
    constexpr int PD = dense_pad(Path(PATH)) / path_kpc(Path(PATH)) % 4 == 0 ? 4 : 2;
    group_blocks(hdr, tasks, offset, ndense, [](const DenseStepArgs &a, int bx, int by) {
        dense_fine_body<PATH, NB, PD, EPI_UPDATE>(a, bx, by);
    });
}
static_assert(DENSE_THREADS == csr::WAVES * 64, "sparse tasks ride in the dense launch");

// Operand f(X) from the state: one thread per 4 consecutive spins of column c.
template <int PATH>
__global__ __launch_bounds__(256) void k_dense_operand(int Np, int nkc, int mbw, const float *__restrict__ x, void *g,
                                                       void *g_lo, float delta, int fmode) {
    const int c = blockIdx.y;
    const int i4 = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i4 >= Np) return;
    const float4 v = *reinterpret_cast<const float4 *>(x + (int64_t)c * Np + i4);
    const float4 f = make_float4(f_value(fmode, v.x, delta), f_value(fmode, v.y, delta),
                                 f_value(fmode, v.z, delta), f_value(fmode, v.w, delta));
    store_operand<PATH>(g, g_lo, x_offset<PATH>(c, i4, nkc, mbw), f, fmode);
}

// Readout operand s = sign(x) with sign(0) = +1 (the energy convention of
// Eq. 2 at the corners), 0 for padded spins i >= N: the dense contraction of
// it gives J s exactly (integer J in fp8 / int8, |J s| < 2^24).
template <int PATH>
__global__ __launch_bounds__(256) void k_readout_operand(int N, int Np, int nkc, int mbw, const float *__restrict__ x,
                                                         void *g) {
    const int c = blockIdx.y;
    const int i4 = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i4 >= Np) return;
    const float4 v = *reinterpret_cast<const float4 *>(x + (int64_t)c * Np + i4);
    auto s = [N](float xv, int i) { return i < N ? (xv >= 0.0f ? 1.0f : -1.0f) : 0.0f; };
    const float4 f = make_float4(s(v.x, i4), s(v.y, i4 + 1), s(v.z, i4 + 2), s(v.w, i4 + 3));
    store_operand<PATH>(g, nullptr, x_offset<PATH>(c, i4, nkc, mbw), f, 0);
}

constexpr int MI355X_CUS = 256;

template <int PATH, int NB, int EPI>
hipError_t launch_step_fine(int Cg, const DenseStepArgs &a, hipStream_t st) {
    const dim3 grid(a.Np / (16 * NB), Cg / 64), block(DENSE_THREADS);
    if (a.nkc % 4 == 0) hipLaunchKernelGGL((k_dense_step_fine<PATH, NB, 4, EPI>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_dense_step_fine<PATH, NB, 2, EPI>), grid, block, 0, st, a);
    return hipGetLastError();
}

template <int PATH, int SG, int CG, int EPI>
hipError_t launch_step_sk(int Cg, const DenseStepArgs &a, hipStream_t st) {
    const int nx = a.Np / (DENSE_TN * SG), ny = Cg / (64 * CG);
    hipLaunchKernelGGL((k_dense_step_sk<PATH, SG, CG, EPI>), dim3((nx + 7) / 8 * 8 * ny), dim3(2 * DENSE_THREADS), 0, st,
                       a, nx, ny);
    return hipGetLastError();
}

template <int PATH, int EPI>
hipError_t launch_step_form(DenseForm form, int mbw, dim3 grid, const DenseStepArgs &a, hipStream_t st) {
    const int Cg = (int)grid.y * 64 * mbw;
    switch (form) {
        case FORM_FINE16: return launch_step_fine<PATH, 1, EPI>(Cg, a, st);
        case FORM_FINE32: return launch_step_fine<PATH, 2, EPI>(Cg, a, st);
        case FORM_TILE: break;
        default:
            if constexpr (path_op2(Path(PATH))) {
                if (form == FORM_SK11) return launch_step_sk<PATH, 1, 1, EPI>(Cg, a, st);
                if (form == FORM_SK21) return launch_step_sk<PATH, 2, 1, EPI>(Cg, a, st);
                if (form == FORM_SK12 && Cg % 128 == 0) return launch_step_sk<PATH, 1, 2, EPI>(Cg, a, st);
                if (form == FORM_SK22 && Cg % 128 == 0) return launch_step_sk<PATH, 2, 2, EPI>(Cg, a, st);
            }
            return hipErrorInvalidValue;
    }
    // two J planes: two column groups per workgroup read each J fragment once
    // for 256 columns (half the J traffic of two 128-column workgroups)
    if constexpr (Pipe<PATH>::planes == 2) {
        if (mbw == 2 && grid.y % 2 == 0) {
            hipLaunchKernelGGL((k_dense_step_cg2<PATH, 2, EPI>), dim3(grid.x, grid.y / 2), dim3(2 * DENSE_THREADS), 0, st,
                               a);
            return hipGetLastError();
        }
    }
    switch (mbw) {
        case 1: hipLaunchKernelGGL((k_dense_step<PATH, 1, EPI>), grid, dim3(DENSE_THREADS), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_dense_step<PATH, 2, EPI>), grid, dim3(DENSE_THREADS), 0, st, a); break;
        case 4: hipLaunchKernelGGL((k_dense_step<PATH, 4, EPI>), grid, dim3(DENSE_THREADS), 0, st, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int PATH>
hipError_t launch_step_path(DenseEpilogue epi, DenseForm form, int mbw, dim3 grid, const DenseStepArgs &a,
                            hipStream_t st) {
    return epi == EPI_UPDATE ? launch_step_form<PATH, EPI_UPDATE>(form, mbw, grid, a, st)
                             : launch_step_form<PATH, EPI_FIELDS>(form, mbw, grid, a, st);
}

}  // namespace

EnergyPlan energy_plan(int N, int count) {
    EnergyPlan e;
    e.T = (N + GEMM_BN - 1) / GEMM_BN;
    e.cp = (count + GEMM_BM - 1) / GEMM_BM * GEMM_BM;
    // two workgroups per CU where the K tiles allow it (at least 8 each, at most
    // 16 ranges); up to 8 blocks down to one or two tiles each while that makes no more than 5
    // workgroups per 2 CUs, since a K tile is 2 to 3 us of latency there. us of a readout
    // with 8, 1 at least: N = 130 68 and 46, N = 700 74 and 51, N = 1000 65 and 51
    const int64_t pairs = (e.T + 1) / 2, tiles = pairs * (e.cp / GEMM_BM);
    const int64_t ktiles = (int64_t)(e.T + 1) * (GEMM_BN / (GEMM_KB / 8));   // of a pair
    while (e.Z < 16 && ((ktiles >= 16 * e.Z && tiles * e.Z < 512) ||
                        (e.T <= ENERGY_SMALL_T && ktiles > 2 * e.Z && tiles * e.Z <= 320)))
        e.Z *= 2;
    e.units = (int)pairs * e.Z;
    return e;
}

hipError_t launch_energy_gemm(const EnergyPlan &e, const int8_t *S, const double *J, int Np, double *part,
                              hipStream_t st) {
    if (Np % 16 || e.T < 1 || e.T * GEMM_BN > Np || e.cp % GEMM_BM || e.Z < 1 || (e.Z & (e.Z - 1)) ||
        e.units != (e.T + 1) / 2 * e.Z)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_energy_gemm, dim3(e.units, e.cp / GEMM_BM), dim3(GEMM_THREADS), 0, st, S, J, Np, e.cp, e.T, e.Z,
                       part);
    return hipGetLastError();
}

// us per step of the forms, measured (update form, N a multiple of 512):
//   fine / split-K at 96, 128, 192 and 256 tiles of 64 x 64: fp4 6.9 / 8.2, 8.0 / 8.7,
//     9.0 / 9.8, 11.1 / 9.5; fp8 8.6 / 8.6, 11.2 / 9.7, 11.7 / 9.0, 15.8 / 10.6; int8
//     8.4 / 9.2, 10.0 / 10.4 (64-spin tile at the next two) 11.9 / 10.2, 14.3 / 11.8;
//   64-spin tile / split-K, +-1 J in fp4 at N = 4096 and C = 512 .. 3072 (tiles per CU):
//     2: 14.6 / 14.1, 2.25: 17.3 / 21.3, 3: 18.5 / 19.5, 3.5: 21.6 / 19.9, 4: 23.1 / 23.3,
//     5: 28.3 / 34.2, 6: 31.3 / 35.1, 8: 39.7 / 40.6, 12: 55.1 / 68.0; N = 8192 at 4 and 8:
//     31.4 / 27.0, 56.5 / 49.9; N = 16384 at 4: 51.0 / 41.4;
//   the same with J in bytes (int8): N = 16384, C = 1024 265 / 326, N = 5120, C = 512 26.8 / 28.3.
// A split-K workgroup has a CU to itself, so its rounds have to be full; several
// 64-spin workgroups share one and take any count.
//   Real J: fp32, 64-spin tile / 16 / 32 spins: N = 1500, C = 60 32.2 / 10.3 / 16.2; N =
//     2000, C = 128 41.8 / 13.7 / 21.4; N = 4096, C = 128 (512 and 256 fine workgroups) 78.9 /
//     49.1 / 39.8; N = 5000, C = 128 97 / 89 / 127; bf16 hi+lo N = 4096, C = 128 34.2 / 40.7 / 30.6.
// The 64-spin tile of 256 columns has one wave per SIMD: with up to 4 tiles of 64 x 64
// per CU it takes 1.2 to 1.7 times as long as split-K in one round.
DenseForm default_dense_form(Path path, int Np, int mbw, int Cg) {
    const int64_t n16 = (int64_t)Np / 16 * (Cg / 64), n = n16 / 4;   // fine workgroups; 64 x 64 tiles
    if (!path_op2(path)) return n16 <= MI355X_CUS ? FORM_FINE16 : n16 / 2 <= MI355X_CUS ? FORM_FINE32 : FORM_TILE;
    if (n < (path == PATH_FP4PK ? MI355X_CUS : MI355X_CUS / 2)) return n16 <= MI355X_CUS ? FORM_FINE16 : FORM_FINE32;
    if (n <= MI355X_CUS) return FORM_SK11;
    if (n <= 2 * MI355X_CUS) return Cg % 128 == 0 ? FORM_SK12 : FORM_SK21;
    const int64_t round = 4 * MI355X_CUS, rounds = (n + round - 1) / round;
    if (mbw == 4 && rounds == 1) return FORM_SK22;
    return path_packed(path) && Cg % 128 == 0 && 20 * n >= 17 * rounds * round ? FORM_SK22 : FORM_TILE;
}

hipError_t launch_dense_step(Path path, DenseEpilogue epi, DenseForm form, int mbw, int Cg, const DenseStepArgs &a,
                             hipStream_t st) {
    const int tm = 64 * mbw;
    if (a.Np % DENSE_TN || Cg % tm || a.C > Cg || a.Np % path_kpc(path) || a.nkc != dense_nkc(path, a.Np) ||
        a.nkc % dense_depth(path))
        return hipErrorInvalidValue;
    const dim3 grid(a.Np / DENSE_TN, Cg / tm);
    DenseStepArgs b = a;
    b.mbw = mbw;
    switch (path) {
        case PATH_F32: return launch_step_path<PATH_F32>(epi, form, mbw, grid, b, st);
        case PATH_FP8: return launch_step_path<PATH_FP8>(epi, form, mbw, grid, b, st);
        case PATH_BF16X3: return launch_step_path<PATH_BF16X3>(epi, form, mbw, grid, b, st);
        case PATH_I8: return launch_step_path<PATH_I8>(epi, form, mbw, grid, b, st);
        case PATH_FP8PK: return launch_step_path<PATH_FP8PK>(epi, form, mbw, grid, b, st);
        case PATH_FP4: return launch_step_path<PATH_FP4>(epi, form, mbw, grid, b, st);
        case PATH_FP4PK: return launch_step_path<PATH_FP4PK>(epi, form, mbw, grid, b, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_convert_j_bits(Path path, const uint32_t *sign_bits, int N, int Np, int nkc, void *Jd,
                                 hipStream_t st) {
    if (!path_packed(path) || Np % 128 || Np % path_kpc(path) || nkc != dense_nkc(path, Np) || N > Np)
        return hipErrorInvalidValue;
    const bool fp4 = path_fp4(path);
    const int words = (N + 31) / 32;
    const int64_t nq = (int64_t)(Np / 16) * nkc * 64 * (fp4 ? 2 : 1);
    const dim3 grid((unsigned)((nq + 255) / 256));
    if (fp4)
        hipLaunchKernelGGL(k_convert_j_pk_bits<true>, grid, dim3(256), 0, st, sign_bits, N, words, Np, nkc,
                           static_cast<uint32_t *>(Jd));
    else
        hipLaunchKernelGGL(k_convert_j_pk_bits<false>, grid, dim3(256), 0, st, sign_bits, N, words, Np, nkc,
                           static_cast<uint32_t *>(Jd));
    return hipGetLastError();
}

hipError_t launch_convert_j(Path path, const double *J64, int Np, int nkc, void *Jd, void *Jd_lo, hipStream_t st) {
    if (Np % 128 || Np % path_kpc(path) || nkc != dense_nkc(path, Np)) return hipErrorInvalidValue;
    if (path_packed(path)) {
        const bool fp4 = path_fp4(path);
        const int64_t nq = (int64_t)(Np / 16) * nkc * 64 * (fp4 ? 2 : 1);
        const dim3 grid((unsigned)((nq + 255) / 256));
        if (fp4) hipLaunchKernelGGL(k_convert_j_pk<true>, grid, dim3(256), 0, st, J64, Np, nkc, static_cast<uint32_t *>(Jd));
        else hipLaunchKernelGGL(k_convert_j_pk<false>, grid, dim3(256), 0, st, J64, Np, nkc, static_cast<uint32_t *>(Jd));
        return hipGetLastError();
    }
    const int64_t nq = (int64_t)Np * (Np / 4);
    const dim3 grid((unsigned)((nq + 255) / 256)), block(256);
    uint8_t *d = static_cast<uint8_t *>(Jd), *dl = static_cast<uint8_t *>(Jd_lo);
    switch (path) {
        case PATH_F32: hipLaunchKernelGGL(k_convert_j<PATH_F32>, grid, block, 0, st, J64, Np, nkc, d, dl); break;
        case PATH_FP8: hipLaunchKernelGGL(k_convert_j<PATH_FP8>, grid, block, 0, st, J64, Np, nkc, d, dl); break;
        case PATH_BF16X3: hipLaunchKernelGGL(k_convert_j<PATH_BF16X3>, grid, block, 0, st, J64, Np, nkc, d, dl); break;
        case PATH_I8: hipLaunchKernelGGL(k_convert_j<PATH_I8>, grid, block, 0, st, J64, Np, nkc, d, dl); break;
        case PATH_FP4: hipLaunchKernelGGL(k_convert_j<PATH_FP4>, grid, block, 0, st, J64, Np, nkc, d, dl); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_group_dense(Path path, int mbw, const GroupHeader *hdr, const GroupTask *tasks, int grid, int offset,
                              hipStream_t st) {
    if (grid < 1) return hipErrorInvalidValue;
#define SBQA_GD(P, M) hipLaunchKernelGGL((k_group_dense<P, M>), dim3(grid), dim3(DENSE_THREADS), 0, st, hdr, tasks, offset)
#define SBQA_GD_PATH(P)                 \
    switch (mbw) {                      \
        case 1: SBQA_GD(P, 1); break;   \
        case 2: SBQA_GD(P, 2); break;   \
        case 4: SBQA_GD(P, 4); break;   \
        default: return hipErrorInvalidValue; \
    }
    switch (path) {
        case PATH_F32: SBQA_GD_PATH(PATH_F32); break;
        case PATH_FP8: SBQA_GD_PATH(PATH_FP8); break;
        case PATH_BF16X3: SBQA_GD_PATH(PATH_BF16X3); break;
        case PATH_I8: SBQA_GD_PATH(PATH_I8); break;
        case PATH_FP8PK: SBQA_GD_PATH(PATH_FP8PK); break;
        case PATH_FP4: SBQA_GD_PATH(PATH_FP4); break;
        case PATH_FP4PK: SBQA_GD_PATH(PATH_FP4PK); break;
        default: return hipErrorInvalidValue;
    }
#undef SBQA_GD_PATH
#undef SBQA_GD
    return hipGetLastError();
}

hipError_t launch_group_fine(Path path, int spins, const GroupHeader *hdr, const GroupTask *tasks, int grid,
                             const GroupHeader *chdr, const GroupTask *ctasks, int cgrid, int offset, hipStream_t st) {
    if (grid < 1 || cgrid < 0 || (spins != 16 && spins != 32)) return hipErrorInvalidValue;
#define SBQA_GFN(P, NB)                                                                                            \
    hipLaunchKernelGGL((k_group_dense_fine<P, NB>), dim3(grid + cgrid), dim3(DENSE_THREADS), 0, st, hdr, tasks, grid, \
                       chdr, ctasks, offset)
#define SBQA_GF(P)                      \
    case P:                             \
        if (spins == 16) SBQA_GFN(P, 1); \
        else SBQA_GFN(P, 2);            \
        break;
    switch (path) {
        SBQA_GF(PATH_F32) SBQA_GF(PATH_FP8) SBQA_GF(PATH_BF16X3) SBQA_GF(PATH_I8) SBQA_GF(PATH_FP8PK)
        SBQA_GF(PATH_FP4) SBQA_GF(PATH_FP4PK)
        default: return hipErrorInvalidValue;
    }
#undef SBQA_GF
#undef SBQA_GFN
    return hipGetLastError();
}

hipError_t launch_dense_operand(Path path, int fmode, int N, int Np, int C, int nkc, int mbw, const float *x, void *g,
                                void *g_lo, float delta, hipStream_t st) {
    (void)N;
    dim3 grid((Np / 4 + 255) / 256, C), block(256);
    switch (path) {
        case PATH_F32: hipLaunchKernelGGL(k_dense_operand<PATH_F32>, grid, block, 0, st, Np, nkc, mbw, x, g, g_lo, delta, fmode); break;
        case PATH_FP8: hipLaunchKernelGGL(k_dense_operand<PATH_FP8>, grid, block, 0, st, Np, nkc, mbw, x, g, g_lo, delta, fmode); break;
        case PATH_BF16X3: hipLaunchKernelGGL(k_dense_operand<PATH_BF16X3>, grid, block, 0, st, Np, nkc, mbw, x, g, g_lo, delta, fmode); break;
        case PATH_I8: hipLaunchKernelGGL(k_dense_operand<PATH_I8>, grid, block, 0, st, Np, nkc, mbw, x, g, g_lo, delta, fmode); break;
        case PATH_FP8PK: hipLaunchKernelGGL(k_dense_operand<PATH_FP8>, grid, block, 0, st, Np, nkc, mbw, x, g, g_lo, delta, fmode); break;
        case PATH_FP4:
        case PATH_FP4PK: hipLaunchKernelGGL(k_dense_operand<PATH_FP4>, grid, block, 0, st, Np, nkc, mbw, x, g, g_lo, delta, fmode); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sbqa

namespace sbqa {

hipError_t launch_readout_operand(Path path, int N, int Np, int C, int nkc, int mbw, const float *x, void *g,
                                  hipStream_t st) {
    dim3 grid((Np / 4 + 255) / 256, C), block(256);
    switch (path) {
        case PATH_FP8:
        case PATH_FP8PK: hipLaunchKernelGGL(k_readout_operand<PATH_FP8>, grid, block, 0, st, N, Np, nkc, mbw, x, g); break;
        case PATH_I8: hipLaunchKernelGGL(k_readout_operand<PATH_I8>, grid, block, 0, st, N, Np, nkc, mbw, x, g); break;
        case PATH_FP4:
        case PATH_FP4PK: hipLaunchKernelGGL(k_readout_operand<PATH_FP4>, grid, block, 0, st, N, Np, nkc, mbw, x, g); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sbqa
