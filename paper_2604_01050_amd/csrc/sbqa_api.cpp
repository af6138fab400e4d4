// Host runtime of the SBQA library: validation, schedules (Eq. 5, Eq. 8 and
// the pump of Sec. II.A), the per-run (beta, alpha) auto-tuning draw of
// Sec. II.B, device buffers, and the step / readout / energy dispatch.
#include "sbqa_ctx.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <limits>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <set>
#include <system_error>
#include <tuple>
#include <string>

#include <fcntl.h>
#include <sys/stat.h>
#include <unistd.h>
#include <thread>
#include <vector>

namespace sbqa {

static thread_local std::string g_err;

sbqa_status fail(sbqa_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

void clear_error() { g_err.clear(); }
const char *last_error() { return g_err.c_str(); }

#define HIP_TRY(expr)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return fail(e_ == hipErrorOutOfMemory ? SBQA_ENOMEM : SBQA_EDEVICE, "%s: %s (%s:%d)", \
                        #expr, hipGetErrorString(e_), __FILE__, __LINE__);                     \
    } while (0)

static int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// splitmix64 (Steele, Lea, Flood 2014): host stream for the (beta, alpha) draws.
static uint64_t splitmix64(uint64_t &s) {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static double unit_double(uint64_t &s) { return (double)(splitmix64(s) >> 11) * (1.0 / 9007199254740992.0); }

// ---------------------------------------------------------------- validation
// One pass over a dense J: diagonal, finiteness, symmetry (64 x 64 tiles of
// the upper triangle against their transposes, so both stay in cache), the
// integral / ternary flags and the sum of squares of the entries. Row blocks
// are scanned in parallel; their sums of squares are added in block order, so
// the result does not depend on the number of threads.
struct DenseScan {
    int bad = 0;              // 1 diagonal, 2 not finite, 3 not symmetric
    int64_t i = 0, j = 0;
    bool integral = true, ternary = true, pm1 = true;
    double ss = 0.0, maxabs = 0.0;
};

// f(0), ..., f(nb - 1), on several threads when the work (matrix elements)
// pays for starting them. Where the system refuses a thread the others do its share.
template <class F>
static void over_blocks(int64_t nb, int64_t work, F &&f) {
    const int64_t nt = std::min<int64_t>({nb, work / (1 << 16), 16, (int64_t)std::thread::hardware_concurrency()});
    if (nt <= 1) {
        for (int64_t b = 0; b < nb; ++b) f(b);
        return;
    }
    std::atomic<int64_t> next{0};
    auto run = [&] {
        for (int64_t b; (b = next.fetch_add(1)) < nb;) f(b);
    };
    std::vector<std::thread> pool;
    pool.reserve((size_t)nt);
    try {
        for (int64_t t = 1; t < nt; ++t) pool.emplace_back(run);
    } catch (const std::system_error &) {
    }
    run();
    for (std::thread &t : pool) t.join();
}

// Transpose of a 64 x 64 bit matrix, row r in a[r] (bit c: column c): the
// off-diagonal quadrants swapped at block sizes 32, 16, ..., 1 (the recursive
// bit-matrix transpose of H. S. Warren, Hacker's Delight, chapter 7).
static void transpose64(uint64_t (&a)[64]) {
    uint64_t m = 0x00000000FFFFFFFFull;
    for (int w = 32; w; w >>= 1, m ^= m << w)
        for (int k = 0; k < 64; k = ((k | w) + 1) & ~w) {
            const uint64_t t = ((a[k] >> w) ^ a[k | w]) & m;
            a[k] ^= t << w;
            a[k | w] ^= t;
        }
}

// Whether J is +-1 off the diagonal, zero on it and symmetric, from one pass
// over its bits (80 MB, N = 3158: 1.6 ms on 16 threads, against 12.6 ms for
// the general scan below, which a J that fails goes through for its message).
// bits: row-major sign bits, words64 per row, bit j % 64 of word j / 64 set
// where J_ij < 0. Its entries count half: with a thread per 65536 of them creating
// N = 1024 took 0.65 ms, 0.52 with one per 131072 (N = 3158 3.8 either way).
static bool scan_pm1(const double *A, int64_t N, std::vector<uint64_t> *bits) {
    constexpr uint64_t SIGN = (uint64_t)1 << 63, ONE = 0x3FF0000000000000ull;
    const int64_t words = (N + 63) / 64, nb = words;
    if (N < 2 || std::fabs(A[1]) != 1.0) return false;   // (most others end here, before N^2 / 8 bytes are taken)
    bits->assign((size_t)(N * words), 0);
    std::atomic<bool> good{true};
    auto raw = [](const double *p) {
        uint64_t u;
        std::memcpy(&u, p, sizeof u);
        return u;
    };
    over_blocks(nb, N * N / 2, [&](int64_t b) {
        for (int64_t i = 64 * b; i < std::min(N, 64 * b + 64) && good.load(std::memory_order_relaxed); ++i) {
            const double *row = A + i * N;
            uint64_t *out = bits->data() + i * words, bad = raw(row + i) & ~SIGN;   // the diagonal: +-0
            auto span = [&](int64_t j0, int64_t j1) {   // inside one word
                uint64_t w = 0;
                for (int64_t j = j0; j < j1; ++j) {
                    const uint64_t u = raw(row + j);
                    bad |= (u & ~SIGN) ^ ONE;
                    w |= (u >> 63) << (j & 63);
                }
                return w;
            };
            for (int64_t q = 0; q < words; ++q) {
                const int64_t j0 = 64 * q, j1 = std::min(N, j0 + 64);
                out[q] = i >= j0 && i < j1 ? span(j0, i) | span(i + 1, j1) : span(j0, j1);
            }
            if (bad) good.store(false, std::memory_order_relaxed);
        }
    });
    if (!good.load()) return false;
    over_blocks(nb, N * N / 32, [&](int64_t b) {
        for (int64_t q = b; q < nb && good.load(std::memory_order_relaxed); ++q) {
            uint64_t t[64];
            for (int k = 0; k < 64; ++k) t[k] = 64 * q + k < N ? (*bits)[(size_t)((64 * q + k) * words + b)] : 0;
            transpose64(t);
            uint64_t diff = 0;
            for (int64_t k = 0; k < 64 && 64 * b + k < N; ++k) diff |= t[k] ^ (*bits)[(size_t)((64 * b + k) * words + q)];
            if (diff) good.store(false, std::memory_order_relaxed);
        }
    });
    return good.load();
}

static DenseScan scan_dense(const double *A, int64_t N) {
    constexpr int64_t TB = 64;
    const int64_t nb = (N + TB - 1) / TB;
    std::vector<DenseScan> part((size_t)nb);
    auto scan_block = [&](int64_t bi) {
        DenseScan &r = part[(size_t)bi];
        const int64_t i0 = bi * TB, i1 = std::min(N, i0 + TB);
        for (int64_t i = i0; i < i1; ++i) {
            if (A[i * N + i] != 0.0 && !r.bad) { r.bad = 1; r.i = i; r.j = i; }
            double srow = 0.0;
            for (int64_t j = 0; j < N; ++j) {
                const double v = A[i * N + j];
                if (!std::isfinite(v)) {
                    if (!r.bad) { r.bad = 2; r.i = i; r.j = j; }
                    continue;
                }
                if (r.integral) {   // (a real J leaves these at its first couplings)
                    if (!(std::fabs(v) <= 2147483647.0) || (double)(int32_t)v != v) r.integral = false;
                    if (!(v == 0.0 || v == 1.0 || v == -1.0)) r.ternary = false;
                    if (j != i && !(v == 1.0 || v == -1.0)) r.pm1 = false;
                }
                r.maxabs = std::max(r.maxabs, std::fabs(v));
                srow += v * v;
            }
            r.ss += srow;
            if (!r.integral) r.ternary = r.pm1 = false;
        }
        for (int64_t bj = bi; bj < nb; ++bj) {
            const int64_t j0 = bj * TB, j1 = std::min(N, j0 + TB);
            for (int64_t i = i0; i < i1; ++i)
                for (int64_t j = std::max(j0, i + 1); j < j1; ++j)
                    if (A[i * N + j] != A[j * N + i] && !(std::isnan(A[i * N + j]) && std::isnan(A[j * N + i])) && !r.bad) {
                        r.bad = 3; r.i = i; r.j = j;
                    }
        }
    };
    over_blocks(nb, N * N, scan_block);
    DenseScan out;
    for (const DenseScan &r : part) {
        if (r.bad && !out.bad) { out.bad = r.bad; out.i = r.i; out.j = r.j; }
        out.integral = out.integral && r.integral;
        out.ternary = out.ternary && r.ternary;
        out.pm1 = out.pm1 && r.pm1;
        out.maxabs = std::max(out.maxabs, r.maxabs);
        out.ss += r.ss;
    }
    return out;
}

sbqa_status validate_instance(const sbqa_coupling *J, const double *h, int32_t N, int32_t R, int32_t runs,
                              const sbqa_schedule *s, InstanceFacts *facts, std::vector<uint32_t> *sign_bits) {
    if (!J || !s) return fail(SBQA_EINVAL, "J and schedule must be non-NULL");
    if (N < 1 || R < 1 || runs < 1) return fail(SBQA_EINVAL, "N, R and runs must be >= 1 (got %d, %d, %d)", N, R, runs);
    if ((int64_t)R * runs > (1 << 24)) return fail(SBQA_EINVAL, "runs*R too large");
    if (s->steps < 1) return fail(SBQA_EINVAL, "steps must be >= 1");
    if (!(s->dt > 0) || !std::isfinite(s->dt)) return fail(SBQA_EINVAL, "dt must be finite and > 0");
    if (!(s->a0 > 0) || !std::isfinite(s->a0)) return fail(SBQA_EINVAL, "a0 must be finite and > 0");
    if (!std::isfinite(s->c0)) return fail(SBQA_EINVAL, "c0 must be finite");
    if (s->fmode < 0 || s->fmode > 2) return fail(SBQA_EINVAL, "unknown fmode %d", s->fmode);
    if (!std::isfinite(s->delta_max) || s->delta_max < 0) return fail(SBQA_EINVAL, "delta_max must be finite and >= 0");
    if (s->precision < SBQA_PREC_AUTO || s->precision > SBQA_PREC_FP4) return fail(SBQA_EINVAL, "unknown precision %d", s->precision);
    if (s->loop_kernel < 0 || s->loop_kernel > 2) return fail(SBQA_EINVAL, "unknown loop_kernel %d", s->loop_kernel);
    if (s->j_packing < SBQA_JPACK_AUTO || s->j_packing > SBQA_JPACK_BYTES) return fail(SBQA_EINVAL, "unknown j_packing %d", s->j_packing);
    if (s->reorder < SBQA_REORDER_AUTO || s->reorder > SBQA_REORDER_ON) return fail(SBQA_EINVAL, "unknown reorder %d", s->reorder);
    if (s->dense_tile != 0 && s->dense_tile != 64 && s->dense_tile != 128 && s->dense_tile != 256)
        return fail(SBQA_EINVAL, "dense_tile must be 0 (autotuned), 64, 128 or 256 (got %d)", s->dense_tile);
    if (!(s->init_amp >= 0) || !std::isfinite(s->init_amp)) return fail(SBQA_EINVAL, "init_amp must be finite and >= 0");
    switch (s->jp_kind) {
        case SBQA_JP_LINEAR:
            if (!std::isfinite(s->jp_start) || !std::isfinite(s->jp_end)) return fail(SBQA_EINVAL, "jp_start/jp_end must be finite");
            break;
        case SBQA_JP_PAPER:
            if (!(s->gamma0_over_R > 0) || !std::isfinite(s->gamma0_over_R)) return fail(SBQA_EINVAL, "gamma0_over_R must be > 0");
            if (!s->beta && !(s->beta_lo > 0 && s->beta_hi >= s->beta_lo && std::isfinite(s->beta_hi)))
                return fail(SBQA_EINVAL, "need 0 < beta_lo <= beta_hi");
            if (!s->alpha && !(s->alpha_lo > 0 && s->alpha_hi >= s->alpha_lo && std::isfinite(s->alpha_hi)))
                return fail(SBQA_EINVAL, "need 0 < alpha_lo <= alpha_hi");
            if (s->beta)
                for (int r = 0; r < runs; ++r)
                    if (!(s->beta[r] > 0) || !std::isfinite(s->beta[r])) return fail(SBQA_EINVAL, "beta[%d] must be > 0", r);
            if (s->alpha)
                for (int r = 0; r < runs; ++r)
                    if (!(s->alpha[r] > 0) || !std::isfinite(s->alpha[r])) return fail(SBQA_EINVAL, "alpha[%d] must be > 0", r);
            break;
        case SBQA_JP_TABLE:
            if (!s->jp_table) return fail(SBQA_EINVAL, "JP_TABLE needs jp_table");
            for (int64_t q = 0; q < (int64_t)runs * s->steps; ++q)
                if (!std::isfinite(s->jp_table[q])) return fail(SBQA_EINVAL, "jp_table[%lld] not finite", (long long)q);
            break;
        default: return fail(SBQA_EINVAL, "unknown jp_kind %d", s->jp_kind);
    }

    const bool dense = J->dense != nullptr;
    const bool csr = J->row_ptr || J->col || J->val;
    if (dense == csr) return fail(SBQA_EINVAL, "exactly one of J.dense or the CSR arrays must be given");
    bool integral = true, ternary = true;
    double ss = 0.0, maxabs = 0.0;
    auto note = [&](double v) {
        if (v != std::floor(v) || std::fabs(v) > 2147483647.0) integral = false;
        if (!(v == 0.0 || v == 1.0 || v == -1.0)) ternary = false;
        maxabs = std::max(maxabs, std::fabs(v));
    };
    if (dense) {
        if ((int64_t)N * N > (int64_t)1 << 32) return fail(SBQA_EINVAL, "dense N too large");
        DenseScan d;
        std::vector<uint64_t> bits;
        if (scan_pm1(J->dense, N, &bits)) {
            d.maxabs = 1.0;
            d.ss = (double)N * (double)(N - 1);
            if (sign_bits) {   // 32-bit words, ceil(N / 32) per row
                const int64_t w32 = (N + 31) / 32, w64 = (N + 63) / 64;
                sign_bits->resize((size_t)(N * w32));
                for (int64_t i = 0; i < N; ++i)
                    for (int64_t q = 0; q < w32; ++q)
                        (*sign_bits)[(size_t)(i * w32 + q)] = (uint32_t)(bits[(size_t)(i * w64 + q / 2)] >> (32 * (q & 1)));
            }
        } else {
            d = scan_dense(J->dense, N);
        }
        if (d.bad) {
            switch (d.bad) {
                case 1: return fail(SBQA_EINVAL, "J has a non-zero diagonal at %lld", (long long)d.i);
                case 2: return fail(SBQA_EINVAL, "J[%lld][%lld] is not finite", (long long)d.i, (long long)d.j);
                default: return fail(SBQA_EINVAL, "J is not symmetric at (%lld,%lld)", (long long)d.i, (long long)d.j);
            }
        }
        integral = d.integral;
        ternary = d.ternary;
        facts->pm1 = d.pm1 && N > 1;
        maxabs = d.maxabs;
        ss = d.ss;
        facts->nnz = 0;
    } else {
        if (!J->row_ptr || (J->nnz != 0 && (!J->col || !J->val)))
            return fail(SBQA_EINVAL, "CSR needs row_ptr, and col and val unless nnz is 0");
        const int32_t *rp = J->row_ptr, *cl = J->col;
        const double *vl = J->val;
        if (J->nnz < 0 || rp[0] != 0 || (int64_t)rp[N] != J->nnz) return fail(SBQA_EINVAL, "row_ptr[0] must be 0 and row_ptr[N] == nnz");
        // pass 0: every row's range lies inside [0, nnz] before col or val is read
        for (int32_t i = 0; i < N; ++i)
            if (rp[i + 1] < rp[i] || (int64_t)rp[i + 1] > J->nnz)
                return fail(SBQA_EINVAL, "row_ptr must be non-decreasing within [0, nnz] (row %d)", i);
        // pass 1: structure of every row (so pass 2 may search any row)
        for (int32_t i = 0; i < N; ++i) {
            for (int32_t p = rp[i]; p < rp[i + 1]; ++p) {
                if (cl[p] < 0 || cl[p] >= N) return fail(SBQA_EINVAL, "col[%d] = %d out of range", p, cl[p]);
                if (p > rp[i] && cl[p] <= cl[p - 1]) return fail(SBQA_EINVAL, "columns of row %d not strictly ascending", i);
                if (!std::isfinite(vl[p])) return fail(SBQA_EINVAL, "val[%d] not finite", p);
                if (cl[p] == i && vl[p] != 0.0) return fail(SBQA_EINVAL, "J has a non-zero diagonal at %d", i);
            }
        }
        // pass 2: symmetry J_ij == J_ji
        for (int32_t i = 0; i < N; ++i) {
            for (int32_t p = rp[i]; p < rp[i + 1]; ++p) {
                const int32_t j = cl[p];
                const int32_t *b = cl + rp[j], *e = cl + rp[j + 1];
                const int32_t *f = std::lower_bound(b, e, i);
                if (f == e || *f != i || vl[rp[j] + (f - b)] != vl[p])
                    return fail(SBQA_EINVAL, "CSR J is not symmetric at (%d,%d)", i, j);
                note(vl[p]);
                if (j != i) ss += vl[p] * vl[p];
            }
        }
        facts->nnz = J->nnz;
    }
    facts->int8 = integral && maxabs <= 127.0;   // J only: h enters in fp32
    if (J->n3 < 0) return fail(SBQA_EINVAL, "n3 must be >= 0");
    if (J->n3 > 0) {
        if (dense) return fail(SBQA_EINVAL, "three-body terms need CSR two-body couplings (nnz may be 0)");
        if (!J->tri || !J->K) return fail(SBQA_EINVAL, "three-body terms need tri and K");
        if (J->n3 > (int64_t)1 << 28) return fail(SBQA_EINVAL, "too many three-body terms");
        for (int64_t t = 0; t < J->n3; ++t) {
            const int32_t a = J->tri[3 * t], b = J->tri[3 * t + 1], d = J->tri[3 * t + 2];
            if (a < 0 || a >= N || b < 0 || b >= N || d < 0 || d >= N)
                return fail(SBQA_EINVAL, "triple %lld has a spin index out of range", (long long)t);
            if (a == b || a == d || b == d) return fail(SBQA_EINVAL, "triple %lld repeats a spin", (long long)t);
            if (!std::isfinite(J->K[t])) return fail(SBQA_EINVAL, "K[%lld] not finite", (long long)t);
            if (J->K[t] != std::floor(J->K[t])) integral = false;
            ss += 3.0 * J->K[t] * J->K[t];   // field variance of random spins (c0)
        }
    }
    facts->n3 = J->n3 > 0 ? J->n3 : 0;
    if (h)
        for (int32_t i = 0; i < N; ++i) {
            if (!std::isfinite(h[i])) return fail(SBQA_EINVAL, "h[%d] not finite", i);
            if (h[i] != std::floor(h[i])) integral = false;
        }
    facts->dense = dense;
    facts->integral = integral;
    facts->ternary = ternary;
    facts->rms = (N > 1 && ss > 0) ? std::sqrt(ss / ((double)N * (double)(N - 1))) : 0.0;

    // contraction path
    int prec = s->precision;
    if (!dense) {
        if (prec != SBQA_PREC_AUTO && prec != SBQA_PREC_FP32)
            return fail(SBQA_EINVAL, "CSR couplings support only fp32 precision");
        facts->path = PATH_CSR;
    } else {
        if (prec == SBQA_PREC_AUTO)
            prec = s->fmode == SBQA_F_BALLISTIC ? SBQA_PREC_FP32
                   : ternary                    ? SBQA_PREC_FP4
                   : facts->int8                ? SBQA_PREC_INT8
                                                : SBQA_PREC_FP32;
        if (prec == SBQA_PREC_FP8 || prec == SBQA_PREC_FP4) {
            const char *nm = prec == SBQA_PREC_FP8 ? "FP8" : "FP4";
            if (s->fmode == SBQA_F_BALLISTIC) return fail(SBQA_EINVAL, "%s precision needs ternary or sign f (ballistic operands are not exact)", nm);
            if (!ternary) return fail(SBQA_EINVAL, "%s precision needs J in {-1,0,+1}", nm);
        }
        if (prec == SBQA_PREC_INT8) {
            if (s->fmode == SBQA_F_BALLISTIC) return fail(SBQA_EINVAL, "INT8 precision needs ternary or sign f (ballistic operands are not integers)");
            if (!facts->int8) return fail(SBQA_EINVAL, "INT8 precision needs integer J with |J| <= 127");
        }
        const bool pack = facts->pm1 && s->j_packing == SBQA_JPACK_AUTO;
        facts->path = prec == SBQA_PREC_FP8      ? (pack ? PATH_FP8PK : PATH_FP8)
                      : prec == SBQA_PREC_FP4    ? (pack ? PATH_FP4PK : PATH_FP4)
                      : prec == SBQA_PREC_INT8   ? PATH_I8
                      : prec == SBQA_PREC_BF16X3 ? PATH_BF16X3
                                                 : PATH_F32;
    }
    return SBQA_OK;
}

// The planes of [count rounded up to GEMM_BM][Np] doubles that callers and the
// server's admission allow for the partial sums of float64 energies (an upper
// bound of what energy_plan takes).
int energy_scratch_planes(int Np, int cp) {
    const int64_t tiles = (int64_t)(Np / GEMM_BN) * (cp / GEMM_BM), nke = (int64_t)Np * 8 / GEMM_KB;
    int es = 1;
    while (tiles * es < 512 && es < 8 && nke % (2 * es) == 0 && nke / (2 * es) >= 4) es *= 2;
    return es;
}

// Geometry and byte count of a context (also used by the server's admission).
void plan_layout(int32_t N, int32_t R, int32_t runs, const InstanceFacts &f, Layout *L) {
    const int64_t C = (int64_t)R * runs;
    L->C = (int)C;
    L->Cp = (int)round_up(C, GEMM_BM);
    // the operand is sized for the widest tile the autotuner may pick
    L->mbw = 4;
    L->Cg = (int)round_up(C, 64 * L->mbw);
    L->Np = (int)round_up(N, f.path == PATH_CSR ? GEMM_BN : dense_pad(f.path));
    L->Cs = (int)round_up(C, 4);
    int64_t b = 0;
    if (f.path == PATH_CSR) {
        b += 2 * (int64_t)N * L->Cs * 4 + (int64_t)N * L->Cs * 4;        // x ping-pong, y
        b += 2 * (int64_t)N * L->Cs;                                      // int8 operand ping-pong
        b += (int64_t)(N + 1) * 4 + f.nnz * (4 + 4 + 8);                 // CSR
        b += (int64_t)N * 12;                                             // h32, h64
        // energy row blocks: at least one per reduction slot (ENERGY_SLOTS),
        // about 2048 blocks over the column chunks, >= 4 rows each
        const int64_t ncb = (C + 255) / 256;
        L->csr_nrb = (int)std::max<int64_t>(
            1, std::min<int64_t>((N + 3) / 4, std::max<int64_t>(ENERGY_SLOTS, (2048 + ncb - 1) / ncb)));
        // large instances: shorter row blocks (the first stage walks a
        // block's rows one after another, a chain of dependent loads per row),
        // at least 32 rows each, the partials within 64 MiB
        if (N > 65536)
            L->csr_nrb = (int)std::max<int64_t>(
                L->csr_nrb, std::min<int64_t>((N + 31) / 32, ((int64_t)64 << 20) / ((int64_t)C * 24)));
        b += (int64_t)L->csr_nrb * C * 24;
        if (f.n3) b += (int64_t)(N + 1) * 4 + 3 * f.n3 * (8 + 4 + 8);    // three-body lists
        b += (int64_t)N * L->Cs * 4;                                      // phi (fields hook)
    } else {
        const int planes = f.path == PATH_BF16X3 ? 2 : 1;
        L->nkc = dense_nkc(f.path, L->Np);
        const int es = energy_scratch_planes(L->Np, L->Cp);
        b += 3 * C * (int64_t)L->Np * 4;                                  // x ping-pong, y
        b += 2 * dense_plane_bytes(f.path, L->Cg, L->Np) * planes;        // operand ping-pong
        b += dense_j_bytes(f.path, L->Np) * planes;                       // J
        if (f.jbits) b += (int64_t)N * ((N + 31) / 32) * 4;               // sign bits the J copy is built from
        else b += (int64_t)L->Np * L->Np * 8;                             // J fp64 (energies, source of J)
        b += (int64_t)L->Np * 12;                                         // h
        if (!path_energy_mfma(f.path)) b += (int64_t)L->Cp * L->Np * 8 * (1 + es);   // fp64 readout + energy partials
        L->csr_nrb = 0;
    }
    b += (int64_t)runs * (int64_t)0;  // schedule tables counted by the caller (steps known there)
    b += C * 8 + (int64_t)runs * (16 + N);                                // E, best
    L->bytes = (size_t)b;
}

// ------------------------------------------------------------ tile autotuner
// Kernel form of a context's dense step (DenseForm) and row blocks per operand
// group, mbw (64 * mbw columns of the 64-spin tile). Candidates that pad C by at
// most 2x, or the forms of the tile that the caller gave, are timed once per
// (device, path, C, Np, given tile) on scratch buffers of the instance's shape; the
// fastest is kept. Contexts of the serving loop are stepped by the grouped launches,
// whose 64-spin tiles have 64 * mbw columns: their mbw alone is timed, per power
// of two that holds Np. Every form gives the same bits, so a choice never changes
// results. Choices persist across processes in a tile file (below), so a new
// process (a server restart) does not time them again.
struct DenseChoice {
    int mbw = 0;
    int form = 0;   // DenseForm; 0: served
};

// The device a choice was timed on: architecture and compute-unit count.
static std::string tile_device_tag() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return "";
    static std::mutex mu;
    static std::map<int, std::string> tags;
    std::lock_guard<std::mutex> lk(mu);
    auto it = tags.find(dev);
    if (it != tags.end()) return it->second;
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) != hipSuccess) return "";
    std::string arch(p.gcnArchName);
    for (char &ch : arch)
        if (ch == ' ') ch = '_';
    return tags[dev] = arch + " " + std::to_string(p.multiProcessorCount);
}

// The tile file: SBQA_TUNE_CACHE names it ("" or "off": choices stay in the
// process), else $XDG_CACHE_HOME/sbqa/dense_tiles.txt, else
// $HOME/.cache/sbqa/dense_tiles.txt. One line per choice,
//   sbqa-tile-v1 <arch> <CUs> <path + 16 form (+ 256: a given tile)> <C> <padded N> <mbw>
// (form 0: served) appended with one write; unreadable files and malformed lines are ignored
// (a choice is used only when it is one of the key's candidates).
static std::string tile_file(bool make_dir) {
    const char *env = std::getenv("SBQA_TUNE_CACHE");
    if (env) return (std::strcmp(env, "off") == 0) ? std::string() : std::string(env);
    std::string dir;
    if (const char *x = std::getenv("XDG_CACHE_HOME"); x && *x) dir = std::string(x) + "/sbqa";
    else if (const char *h = std::getenv("HOME"); h && *h) dir = std::string(h) + "/.cache/sbqa";
    else return std::string();
    if (make_dir) {
        const size_t cut = dir.rfind('/');
        if (cut != std::string::npos && cut > 0) (void)::mkdir(dir.substr(0, cut).c_str(), 0755);
        (void)::mkdir(dir.c_str(), 0755);
    }
    return dir + "/dense_tiles.txt";
}

// (device, path, C, padded N, served, mbw of a given tile or 0)
typedef std::tuple<std::string, int, int, int, bool, int> ChoiceKey;
constexpr int GIVEN_TILE = 256;

static void load_tile_file(const std::string &dev, std::map<ChoiceKey, DenseChoice> *cache) {
    const std::string f = tile_file(false);
    if (f.empty()) return;
    FILE *fp = std::fopen(f.c_str(), "r");
    if (!fp) return;
    char line[512];
    while (std::fgets(line, sizeof line, fp)) {
        char tag[32], arch[256];
        int cus = 0, path = 0, C = 0, npb = 0, mbw = 0;
        if (std::sscanf(line, "%31s %255s %d %d %d %d %d", tag, arch, &cus, &path, &C, &npb, &mbw) != 7) continue;
        if (std::strcmp(tag, "sbqa-tile-v1") != 0 || std::string(arch) + " " + std::to_string(cus) != dev) continue;
        const bool given = path >= GIVEN_TILE;
        const int form = (given ? path - GIVEN_TILE : path) >> 4;
        if (path < 0 || form > FORM_SK22 || (given && !form)) continue;
        if (mbw == 1 || mbw == 2 || mbw == 4)
            (*cache)[ChoiceKey(dev, path & 15, C, npb, form == 0, given ? mbw : 0)] = DenseChoice{mbw, form};
    }
    std::fclose(fp);
}

static void append_tile_file(const std::string &dev, int path, int C, int npb, int mbw) {
    const std::string f = tile_file(true);
    if (f.empty()) return;
    char line[512];
    const int n = std::snprintf(line, sizeof line, "sbqa-tile-v1 %s %d %d %d %d\n", dev.c_str(), path, C, npb, mbw);
    if (n <= 0 || n >= (int)sizeof line) return;
    const int fd = ::open(f.c_str(), O_WRONLY | O_APPEND | O_CREAT, 0644);
    if (fd < 0) return;
    (void)!::write(fd, line, (size_t)n);   // one append: whole lines, also from concurrent processes
    ::close(fd);
}

// The candidates of a shape, of the tile given (its mbw) if there is one. The operand
// grouping hardly matters outside the 64-spin tile: there the largest that adds no
// padding. Forms that were nowhere near the fastest at a grid's size are left out.
static std::vector<DenseChoice> dense_candidates(Path path, int C, int Np, bool served, int given) {
    std::vector<int> ms;
    for (int m : {1, 2, 4})
        if (given ? m == given : m == dense_mbw(C) || round_up(C, 64 * m) <= 2 * round_up(C, 64)) ms.push_back(m);
    std::vector<DenseChoice> out;
    if (!served) {
        const int64_t C64 = round_up(C, given ? 64 * given : 64);
        const int m0 = given ? given : C64 % 256 == 0 ? 4 : C64 % 128 == 0 ? 2 : 1;
        const int64_t n = (int64_t)Np / 64 * (C64 / 64);
        if (n <= 1024)
            for (int f : {FORM_FINE16, FORM_FINE32}) out.push_back({m0, f});
        if (path_op2(path) && n >= 64)
            for (int f : {FORM_SK11, FORM_SK21, FORM_SK12, FORM_SK22})
                if (C64 % 128 == 0 || f <= FORM_SK21) out.push_back({m0, f});
        if (n < 96) return out;
    }
    for (int m : ms) out.push_back({m, served ? 0 : (int)FORM_TILE});
    return out;
}

static DenseChoice tune_dense(Path path, int C, int Np, bool served, int given, hipStream_t st) {
    static std::mutex mu;
    static std::map<ChoiceKey, DenseChoice> cache;
    static std::set<std::string> loaded;
    int npk = Np;
    if (served)
        for (npk = 128; npk < Np;) npk *= 2;
    const std::vector<DenseChoice> cand = dense_candidates(path, C, Np, served, given);
    const std::string dev = tile_device_tag();
    const ChoiceKey key(dev, (int)path, C, npk, served, given);
    {
        std::lock_guard<std::mutex> lk(mu);
        if (!dev.empty() && !loaded.count(dev)) {
            load_tile_file(dev, &cache);
            loaded.insert(dev);
        }
        auto it = cache.find(key);
        if (it != cache.end()) {
            const DenseChoice k = it->second;
            const int64_t Cg = round_up(C, 64 * k.mbw);
            if ((given || Cg <= std::max<int64_t>(2 * round_up(C, 64), round_up(C, 64 * dense_mbw(C)))) &&
                (k.form < FORM_SK11 || path_op2(path)) && (k.form < FORM_SK12 || Cg % 128 == 0))
                return k;
        }
    }
    DenseChoice best;
    best.mbw = given ? given : dense_mbw(C);
    best.form = served ? 0 : (int)default_dense_form(path, Np, best.mbw, (int)round_up(C, 64 * best.mbw));
    bool timed = false;
    if (cand.size() > 1) {
        const int planes = path == PATH_BF16X3 ? 2 : 1;
        const int Cgm = (int)round_up(C, 256), nkc = dense_nkc(path, Np);
        std::vector<Block> bufs;
        int device = 0;
        const bool known = hipGetDevice(&device) == hipSuccess;
        auto grab = [&](size_t bytes) -> void * {
            Block b;
            if (!known || pool_get(device, false, bytes, &b) != hipSuccess) return nullptr;
            bufs.push_back(b);
            (void)hipMemsetAsync(b.p, 0, b.bytes, st);
            return b.p;
        };
        const size_t jb = (size_t)dense_j_bytes(path, Np), gb = (size_t)dense_plane_bytes(path, Cgm, Np),
                     sb = (size_t)C * Np * 4;
        DenseStepArgs a{};
        a.N = Np;
        a.Np = Np;
        a.R = 1;
        a.C = C;
        a.nkc = nkc;
        a.J = (const uint8_t *)grab(jb);
        a.J_lo = planes == 2 ? (const uint8_t *)grab(jb) : nullptr;
        a.g = (const uint8_t *)grab(gb);
        a.g_lo = planes == 2 ? (const uint8_t *)grab(gb) : nullptr;
        a.g_next = (uint8_t *)grab(gb);
        a.g_next_lo = planes == 2 ? (uint8_t *)grab(gb) : nullptr;
        a.h = (const float *)grab((size_t)Np * 4);
        a.x_in = (const float *)grab(sb);
        a.x_out = (float *)grab(sb);
        a.y = (float *)grab(sb);
        a.jp = (const float *)grab((size_t)C * 4);
        a.jp_stride = 1;
        a.fmode = 0;
        hipEvent_t e0 = nullptr, e1 = nullptr;
        bool ok = a.J && a.g && a.g_next && a.h && a.x_in && a.x_out && a.y && a.jp && (planes == 1 || (a.J_lo && a.g_lo && a.g_next_lo)) &&
                  hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess;
        auto launch = [&](const DenseChoice &k) {
            return launch_dense_step(path, EPI_UPDATE, served ? FORM_TILE : (DenseForm)k.form, k.mbw,
                                     (int)round_up(C, 64 * k.mbw), a, st) == hipSuccess;
        };
        // (each once for the clocks and the caches, then twice three launches)
        std::vector<float> us(cand.size(), INFINITY);
        for (size_t q = 0; q < cand.size() && ok; ++q) ok = launch(cand[q]);
        for (int round = 0; round < 2; ++round)
            for (size_t q = 0; q < cand.size() && ok; ++q) {
                ok = launch(cand[q]) && hipEventRecord(e0, st) == hipSuccess;
                for (int r = 0; r < 3 && ok; ++r) ok = launch(cand[q]);
                ok = ok && hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
                float ms = 0.0f;
                ok = ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
                if (ok) us[q] = std::min(us[q], ms * 1000.0f / 3.0f);
            }
        if (ok) best = cand[(size_t)(std::min_element(us.begin(), us.end()) - us.begin())];
        const bool done = hipStreamSynchronize(st) == hipSuccess;
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        for (const Block &b : bufs) {
            if (done) pool_put(device, false, b);
            else (void)hipFree(b.p);
        }
        timed = ok;
        (void)hipGetLastError();
    }
    std::lock_guard<std::mutex> lk(mu);
    cache[key] = best;
    if (timed && !dev.empty()) append_tile_file(dev, (int)path + 16 * best.form + (given ? GIVEN_TILE : 0), C, npk, best.mbw);
    return best;
}

// Tile and form of a context (dense_tile: the caller's columns, 0: none given).
static void set_tile(Layout *L, Path path, int dense_tile, bool served, hipStream_t st) {
    DenseChoice k;
    if (served && dense_tile) k.mbw = dense_tile / 64;
    else k = tune_dense(path, L->C, L->Np, served, dense_tile / 64, st);
    L->mbw = k.mbw;
    L->Cg = (int)round_up(L->C, 64 * L->mbw);
    L->form = k.form ? (DenseForm)k.form : default_dense_form(path, L->Np, L->mbw, L->Cg);
}

size_t instance_bytes(int32_t N, int32_t R, int32_t runs, const InstanceFacts &f, uint32_t steps) {
    Layout L;
    plan_layout(N, R, runs, f, &L);
    return L.bytes + ((size_t)runs + 2) * steps * 4 + 4;   // + J_perp table, per-step a_n and Delta_n tables
}

// ----------------------------------------------------------------- schedules
void build_schedule_host(const sbqa_schedule *s, int32_t runs, std::vector<double> &beta, std::vector<double> &alpha,
                         std::vector<float> &jp) {
    const uint32_t S = s->steps;
    beta.assign(runs, 0.0);
    alpha.assign(runs, 0.0);
    uint64_t st = s->seed ^ 0xA5A5F00DBAADC0DEull;
    for (int r = 0; r < runs; ++r) {
        const double u1 = unit_double(st), u2 = unit_double(st);
        beta[r] = s->beta ? s->beta[r] : s->beta_lo + (s->beta_hi - s->beta_lo) * u1;
        alpha[r] = s->alpha ? s->alpha[r] : s->alpha_lo + (s->alpha_hi - s->alpha_lo) * u2;
    }
    jp.assign((size_t)runs * S, 0.0f);
    auto fill = [&](int64_t q0, int64_t q1) {   // entries [q0, q1), run-major
        while (q0 < q1) {
            const int r = (int)(q0 / S);
            const uint32_t n0 = (uint32_t)(q0 - (int64_t)r * S), n1 = (uint32_t)std::min<int64_t>(S, n0 + (q1 - q0));
            float *out = jp.data() + (size_t)r * S;
            for (uint32_t n = n0; n < n1; ++n) {
                const double sn = (double)n / (double)S;   // t/T at the start of step n
                double v;
                if (s->jp_kind == SBQA_JP_LINEAR) v = s->jp_start + (s->jp_end - s->jp_start) * sn;
                else if (s->jp_kind == SBQA_JP_PAPER) {
                    const double gx = s->gamma0_over_R * (std::pow(1.0 - sn, alpha[r]) + 1e-5);  // Eq. 5
                    v = -std::log(std::tanh(beta[r] * gx)) / (2.0 * beta[r]);
                } else v = s->jp_table[(size_t)r * S + n];
                out[n] = (float)v;
            }
            q0 += n1 - n0;
        }
    };
    // Eq. 5 takes about 0.1 us an entry (0.8 ms for 8 runs of 1000 steps, more
    // than the rest of a small context's creation): in parallel from 2048
    // entries on, where it saves more than the threads cost to start (20 us each)
    const int64_t total = (int64_t)runs * S, per = 1024;
    const int64_t nb = s->jp_kind == SBQA_JP_PAPER ? (total + per - 1) / per : 1;
    over_blocks(nb, total / per << 16, [&](int64_t b) { fill(nb == 1 ? 0 : b * per, nb == 1 ? total : std::min(total, (b + 1) * per)); });
}

StepCoef step_coef(const sbqa_schedule *s, double c0, int R, uint32_t n) {
    const double S = (double)s->steps;
    StepCoef k;
    k.kA = (float)((s->a0 - (double)n / S) / (double)R);
    k.kB = (float)(c0 / (double)R);
    k.dt = (float)s->dt;
    k.kD = (float)(s->dt * s->a0 / (double)R);
    k.delta_next = (float)((s->delta_max * (double)(n + 1)) / S);
    return k;
}

float delta_at(const sbqa_schedule *s, uint32_t n) {
    return (float)((s->delta_max * (double)n) / (double)s->steps);
}

}  // namespace sbqa

using namespace sbqa;

// =========================================================================== //
//                                 context                                     //
// =========================================================================== //

namespace sbqa {

// Launches whose workgroups wait for each other, per device (launch_order.h).
struct DeviceOrder {
    std::mutex mu;
    LaunchOrder<hipStream_t> order;
    hipEvent_t passed = nullptr;   // recorded and waited for under mu
};
static DeviceOrder &device_order(int device) {
    static std::mutex mu;
    static auto *all = new std::map<int, std::unique_ptr<DeviceOrder>>();   // (outlives the contexts)
    std::lock_guard<std::mutex> lk(mu);
    auto &d = (*all)[device];
    if (!d) d.reset(new DeviceOrder());
    return *d;
}

static void forget_launches(const sbqa_ctx *c) {
    if (!c->exchanging.workgroups) return;
    DeviceOrder &d = device_order(c->device);
    std::lock_guard<std::mutex> lk(d.mu);
    d.order.forget(c);
}

static bool capturing(hipStream_t st) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &s) != hipSuccess) (void)hipGetLastError();
    return s != hipStreamCaptureStatusNone;
}

// launch() on the context's stream, behind what it must not meet on the device.
// (Recorded launches are ordered by whoever replays them.)
template <class F>
static hipError_t launch_in_order(sbqa_ctx *c, const Exchanging &need, F &&launch) {
    if (!need.workgroups) return launch();
    DeviceOrder &d = device_order(c->device);
    std::lock_guard<std::mutex> lk(d.mu);
    hipError_t e = hipSuccess;
    d.order.before(c, c->stream, need, c->cus, [&](hipStream_t other) {
        if (e != hipSuccess || capturing(c->stream) || capturing(other)) return;
        if (!d.passed) e = hipEventCreateWithFlags(&d.passed, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventRecord(d.passed, other);
        if (e == hipSuccess) e = hipStreamWaitEvent(c->stream, d.passed, 0);
    });
    return e == hipSuccess ? launch() : e;
}

// Steps of one such launch at most: none lasts long (11 us a step or less), so that
// another one's wait for a place on the device stays far below its bound.
constexpr uint32_t MAX_EXCHANGE_STEPS = 4096;

}  // namespace sbqa

sbqa_ctx::~sbqa_ctx() {
    // the pool hands the blocks to other contexts, on other streams: the work
    // on them ends first (blocks of a stream that reports an error are left
    // to the runtime, which waits for the device); recorded work may be
    // replaying on any of the device's streams
    bool done = idle || !stream || hipStreamSynchronize(stream) == hipSuccess;
    if (recorded) {
        int cur = device;
        done = done && hipGetDevice(&cur) == hipSuccess && (cur == device || hipSetDevice(device) == hipSuccess) &&
               hipDeviceSynchronize() == hipSuccess;
        if (cur != device) (void)hipSetDevice(cur);
    }
    forget_launches(this);
    auto back = [&](bool host, Block b) {
        if (done) pool_put(device, host, b);
        else if (host) (void)hipHostFree(b.p);
        else (void)hipFree(b.p);
    };
    for (const Block &b : blocks) back(false, b);
    for (const Chunk &k : chunks) {
        back(false, k.dev);
        back(true, k.host);
    }
    if (rhost_block.p) back(true, rhost_block);
}

// Zeroed device buffer of the context. During creation, buffers up to
// SMALL_BYTES are packed into chunks and become valid with the next flush. A chunk
// holds CHUNK_BYTES, for a small instance what its buffers come to (its estimate,
// a quarter more and 16 KiB for their alignment).
constexpr size_t SMALL_BYTES = (size_t)256 << 10, CHUNK_BYTES = (size_t)1 << 20;
static size_t chunk_bytes(const sbqa_ctx *c) {
    const size_t est = instance_bytes(c->N, c->R, c->runs, c->facts, c->s.steps);
    return std::min(CHUNK_BYTES, (est + est / 4 + ((size_t)16 << 10) + 65535) / 65536 * 65536);
}
// Largest copy that a call takes through pinned memory.
constexpr size_t STAGE_BYTES = (size_t)8 << 20;
// Device buffer of a larger state on its way in (of those that the pool keeps).
constexpr size_t BULK_BYTES = (size_t)64 << 20;

template <class T>
static hipError_t dalloc(sbqa_ctx *c, T **p, size_t n) {
    const size_t bytes = std::max<size_t>(n * sizeof(T), 256), room = (bytes + 255) / 256 * 256;
    hipError_t e;
    if (c->creating && room <= SMALL_BYTES) {
        if (c->chunks.empty() || c->chunks.back().used + room > c->chunks.back().dev.bytes) {
            sbqa_ctx::Chunk k;
            const size_t bytes = std::max(chunk_bytes(c), room);
            if ((e = pool_get(c->device, false, bytes, &k.dev)) != hipSuccess) return e;
            if ((e = pool_get(c->device, true, bytes, &k.host)) != hipSuccess) {
                pool_put(c->device, false, k.dev);
                return e;
            }
            c->chunks.push_back(k);
        }
        sbqa_ctx::Chunk &k = c->chunks.back();
        std::memset(static_cast<uint8_t *>(k.host.p) + k.used, 0, room);
        *p = reinterpret_cast<T *>(static_cast<uint8_t *>(k.dev.p) + k.used);
        k.used += room;
        c->bytes += bytes;
        return hipSuccess;
    }
    Block b;
    if ((e = pool_get(c->device, false, bytes, &b)) != hipSuccess) return e;
    c->blocks.push_back(b);
    c->bytes += bytes;
    *p = static_cast<T *>(b.p);
    return hipMemsetAsync(b.p, 0, bytes, c->stream);
}

// Host values into a device buffer of the context: through the mirror when
// the buffer lies in the part of a chunk that is still to be sent, else
// straight from src, which has to live until settle().
static hipError_t upload(sbqa_ctx *c, void *dst, const void *src, size_t bytes) {
    if (bytes == 0) return hipSuccess;
    const uint8_t *d = static_cast<uint8_t *>(dst);
    for (sbqa_ctx::Chunk &k : c->chunks) {
        uint8_t *base = static_cast<uint8_t *>(k.dev.p);
        if (d >= base + k.sent && d + bytes <= base + k.used) {
            std::memcpy(static_cast<uint8_t *>(k.host.p) + (d - base), src, bytes);
            return hipSuccess;
        }
    }
    c->direct = true;
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, c->stream);
}

// Sends what the mirrors have collected (before a kernel reads or writes the
// small buffers; the mirrors live as long as the context).
static hipError_t flush(sbqa_ctx *c) {
    for (sbqa_ctx::Chunk &k : c->chunks) {
        if (k.sent == k.used) continue;
        const hipError_t e = hipMemcpyAsync(static_cast<uint8_t *>(k.dev.p) + k.sent,
                                            static_cast<uint8_t *>(k.host.p) + k.sent, k.used - k.sent,
                                            hipMemcpyHostToDevice, c->stream);
        if (e != hipSuccess) return e;
        k.sent = k.used;
    }
    return hipSuccess;
}

// Waits for copies straight from host memory (which may be freed afterwards).
static hipError_t settle(sbqa_ctx *c) {
    if (!c->direct) return hipSuccess;
    c->direct = false;
    return hipStreamSynchronize(c->stream);
}

static sbqa_status check_device(int *dev) {
    HIP_TRY(hipGetDevice(dev));
    static std::mutex mu;
    static std::set<int> good;   // devices found to be gfx950
    std::lock_guard<std::mutex> lk(mu);
    if (good.count(*dev)) return SBQA_OK;
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, *dev));
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(SBQA_EDEVICE, "device %d is %s; this library is built for gfx950 (MI355X) only", *dev,
                    prop.gcnArchName);
    good.insert(*dev);
    return SBQA_OK;
}

namespace sbqa {

void note_recording(sbqa_ctx *c) { c->recorded = c->recorded || capturing(c->stream); }

// Build operand f(X) of the current step from the current state.
sbqa_status rebuild_operand(sbqa_ctx *c) {
    const float d = delta_at(&c->s, c->step);
    c->g_stale = false;
    if (c->facts.path == PATH_CSR) {
        // elementwise over the whole buffer: column-block order has C == Cs
        // and zero padded rows, whose operand is 0
        // (the resident loop builds its operand from x at each launch)
        if (c->s.fmode != SBQA_F_BALLISTIC && !c->resident)
            HIP_TRY(launch_csr_operand(c->s.fmode, c->N, c->L.Cs, c->L.C, c->x[c->cur], (int8_t *)c->g[c->cur], d,
                                       c->stream));
    } else {
        HIP_TRY(launch_dense_operand(c->facts.path, c->s.fmode, c->N, c->L.Np, c->L.C, c->L.nkc, c->L.mbw, c->x[c->cur],
                                     c->g[c->cur], c->g_lo[c->cur], d, c->stream));
    }
    return SBQA_OK;
}

// Buffers of the 8-column loop: its published edges, counters and sign bytes.
static hipError_t alloc_wide(sbqa_ctx *c) {
    const size_t nwg = (size_t)c->L.C / resident_cols(), NR = (size_t)c->res_rows;
    hipError_t e = dalloc(c, &c->xpub, 2 * nwg * 2 * NR);
    if (e == hipSuccess) e = dalloc(c, &c->flags, nwg);
    if (e == hipSuccess) e = dalloc(c, &c->epoch_cnt, nwg);
    if (e == hipSuccess) e = dalloc(c, &c->sbits, nwg * NR);
    return e;
}

sbqa_status ctx_upload(sbqa_ctx *c, const sbqa_coupling *J, const double *h, const uint32_t *jbits) {
    const int N = c->N, Np = c->L.Np, Cs = c->L.Cs, C = c->L.C, Cp = c->L.Cp;
    const Path path = c->facts.path;
    const int runs = c->runs;
    const uint32_t S = c->s.steps;
    HIP_TRY(dalloc(c, &c->jp, (size_t)runs * S));
    HIP_TRY(upload(c, c->jp, c->jp_host.data(), sizeof(float) * runs * S));
    {
        // per-step pump and threshold tables (a_n term and Delta_n of Eq. 8),
        // read on the device by the resident loops and the grouped steps
        std::vector<float> ca(S), dtab((size_t)S + 1);
        for (uint32_t n = 0; n < S; ++n) ca[n] = step_coef(&c->s, c->c0, c->R, n).kA;
        for (uint32_t n = 0; n <= S; ++n) dtab[n] = delta_at(&c->s, n);
        HIP_TRY(dalloc(c, &c->coefA, ca.size()));
        HIP_TRY(dalloc(c, &c->delta_tab, dtab.size()));
        HIP_TRY(upload(c, c->coefA, ca.data(), sizeof(float) * ca.size()));
        HIP_TRY(upload(c, c->delta_tab, dtab.data(), sizeof(float) * dtab.size()));
        HIP_TRY(settle(c));   // host staging buffers die here
    }
    HIP_TRY(dalloc(c, &c->E, (size_t)std::max(C, Cp)));
    HIP_TRY(dalloc(c, &c->bestStep, (size_t)runs));
    if (N > BEST_SCRATCH_N) HIP_TRY(dalloc(c, &c->bsel, (size_t)runs));
    c->rbytes = (size_t)8 * runs + 8 + (size_t)runs * N;
    HIP_TRY(dalloc(c, &c->rdev, c->rbytes));
    HIP_TRY(pool_get(c->device, true, c->rbytes, &c->rhost_block));
    c->rhost = static_cast<uint8_t *>(c->rhost_block.p);
    std::memset(c->rhost, 0, c->rbytes);
    {
        void *dp = nullptr;
        if (hipHostGetDevicePointer(&dp, c->rhost, 0) == hipSuccess) c->rhost_dev = static_cast<uint8_t *>(dp);
        else (void)hipGetLastError();   // keep the copy engine path
    }
    c->bestE = reinterpret_cast<double *>(c->rdev);
    c->err = reinterpret_cast<int *>(c->rdev + (size_t)8 * runs);
    c->bestSpins = reinterpret_cast<int8_t *>(c->rdev + (size_t)8 * runs + 8);

    const int hrows = std::max(Np, c->resident ? c->res_rows : 0);
    std::vector<float> h32((size_t)hrows, 0.0f);
    std::vector<double> h64((size_t)N, 0.0);
    if (h)
        for (int i = 0; i < N; ++i) {
            h32[i] = (float)h[i];
            h64[i] = h[i];
        }
    HIP_TRY(dalloc(c, &c->h32, (size_t)hrows));
    HIP_TRY(dalloc(c, &c->h64, (size_t)N));
    HIP_TRY(upload(c, c->h32, h32.data(), sizeof(float) * hrows));
    HIP_TRY(upload(c, c->h64, h64.data(), sizeof(double) * N));
    c->has_h = h != nullptr;

    if (path == PATH_CSR) {
        const int64_t nnz = J->nnz;
        const int rows = c->resident ? c->res_rows : N;   // resident rows are padded with zero rows
        HIP_TRY(dalloc(c, &c->x[0], (size_t)rows * Cs));
        HIP_TRY(dalloc(c, &c->y, (size_t)rows * Cs));
        // the resident loop steps x in place and builds its operand on chip:
        // the second state half, the operand buffers and the fields buffer
        // are only the fields hook's scratch there, allocated at its first call
        if (!c->resident) {
            HIP_TRY(dalloc(c, &c->x[1], (size_t)rows * Cs));
            int8_t *g0, *g1;
            HIP_TRY(dalloc(c, &g0, (size_t)rows * Cs));
            HIP_TRY(dalloc(c, &g1, (size_t)rows * Cs));
            c->g[0] = g0;
            c->g[1] = g1;
        }
        HIP_TRY(dalloc(c, &c->rp, (size_t)N + 1));
        // +8: the CSR step reads neighbour indices in batches of up to 8
        HIP_TRY(dalloc(c, &c->col, (size_t)nnz + 8));
        HIP_TRY(dalloc(c, &c->val, (size_t)nnz + 8));
        HIP_TRY(dalloc(c, &c->val64, (size_t)nnz));
        // row-block partials of the spin-major energies (the column-block
        // readout of a resident context reduces on chip)
        if (c->order != ORDER_COLBLOCK8 || J->n3 > 0)
            HIP_TRY(dalloc(c, &c->csr_partial, (size_t)c->L.csr_nrb * C * 3));
        if (J->n3 > 0) {
            // three-body terms listed per member spin, triples in the given
            // order; +4 entries: the step reads them in batches of up to 4
            std::vector<int32_t> tp((size_t)N + 1, 0);
            for (int64_t t = 0; t < J->n3; ++t)
                for (int e = 0; e < 3; ++e) ++tp[(size_t)J->tri[3 * t + e] + 1];
            for (int32_t i = 0; i < N; ++i) tp[(size_t)i + 1] += tp[(size_t)i];
            const int64_t ne = 3 * J->n3;
            std::vector<int32_t> ab((size_t)2 * (ne + 4), 0), fill(tp.begin(), tp.end() - 1);
            std::vector<float> k32((size_t)ne + 4, 0.0f);
            std::vector<double> k64((size_t)ne, 0.0);
            for (int64_t t = 0; t < J->n3; ++t)
                for (int e = 0; e < 3; ++e) {
                    const int32_t *v = J->tri + 3 * t;
                    const int64_t q = fill[(size_t)v[e]]++;
                    ab[(size_t)2 * q] = v[(e + 1) % 3];
                    ab[(size_t)2 * q + 1] = v[(e + 2) % 3];
                    k32[(size_t)q] = (float)J->K[t];
                    k64[(size_t)q] = J->K[t];
                }
            HIP_TRY(dalloc(c, &c->t3ptr, tp.size()));
            HIP_TRY(dalloc(c, &c->t3ab, ab.size()));
            HIP_TRY(dalloc(c, &c->t3k, k32.size()));
            HIP_TRY(dalloc(c, &c->t3k64, k64.size()));
            HIP_TRY(upload(c, c->t3ptr, tp.data(), sizeof(int32_t) * tp.size()));
            HIP_TRY(upload(c, c->t3ab, ab.data(), sizeof(int32_t) * ab.size()));
            HIP_TRY(upload(c, c->t3k, k32.data(), sizeof(float) * k32.size()));
            HIP_TRY(upload(c, c->t3k64, k64.data(), sizeof(double) * k64.size()));
            HIP_TRY(settle(c));   // host staging buffers die here
        }
        if (!c->resident) HIP_TRY(dalloc(c, &c->phi, (size_t)N * Cs));
        std::vector<float> v32((size_t)nnz);
        for (int64_t p = 0; p < nnz; ++p) v32[p] = (float)J->val[p];
        HIP_TRY(upload(c, c->rp, J->row_ptr, sizeof(int32_t) * (N + 1)));
        HIP_TRY(upload(c, c->col, J->col, sizeof(int32_t) * nnz));
        HIP_TRY(upload(c, c->val, v32.data(), sizeof(float) * nnz));
        HIP_TRY(upload(c, c->val64, J->val, sizeof(double) * nnz));
        std::vector<int32_t> cp, rc;
        std::vector<float> vp;
        std::vector<double> rv, rhv;
        if (c->resident) {
            // padded neighbour lists (CSR order, then index 0 with weight 0),
            // ring exchange buffers
            const int D = c->res_D, NR = c->res_rows;
            cp.assign((size_t)NR * D, 0);
            vp.assign((size_t)D * NR, 0.0f);
            for (int i = 0; i < N; ++i)
                for (int q = 0; q < J->row_ptr[i + 1] - J->row_ptr[i]; ++q) {
                    cp[(size_t)i * D + q] = J->col[J->row_ptr[i] + q];
                    vp[(size_t)q * NR + i] = (float)J->val[J->row_ptr[i] + q];
                }
            // the readout energies' copy, grouped by the energy row blocks:
            // [row in block][neighbour][row block]
            const int nrb = c->L.csr_nrb, rpb = (N + nrb - 1) / nrb, RS = energy_colblock_rows(rpb);
            rc.assign((size_t)nrb * RS * D, 0);
            rv.assign((size_t)nrb * RS * D, 0.0);
            rhv.assign((size_t)nrb * RS, 0.0);
            for (int i = 0; i < N; ++i) {
                const size_t rb = (size_t)(i / rpb), r = (size_t)(i % rpb);
                for (int q = 0; q < J->row_ptr[i + 1] - J->row_ptr[i]; ++q) {
                    rc[(r * D + q) * nrb + rb] = J->col[J->row_ptr[i] + q];
                    rv[(r * D + q) * nrb + rb] = J->val[J->row_ptr[i] + q];
                }
                if (h) rhv[r * nrb + rb] = h[i];
            }
            HIP_TRY(dalloc(c, &c->colpad, cp.size()));
            HIP_TRY(dalloc(c, &c->valpad, vp.size()));
            HIP_TRY(dalloc(c, &c->rcol, rc.size()));
            HIP_TRY(dalloc(c, &c->rval, rv.size()));
            HIP_TRY(dalloc(c, &c->rh, rhv.size()));
            HIP_TRY(upload(c, c->rcol, rc.data(), sizeof(int32_t) * rc.size()));
            HIP_TRY(upload(c, c->rval, rv.data(), sizeof(double) * rv.size()));
            HIP_TRY(upload(c, c->rh, rhv.data(), sizeof(double) * rhv.size()));
            if (c->res_W < resident_cols()) {
                HIP_TRY(dalloc(c, &c->words, (size_t)2 * c->res_nwg * 2 * narrow_rows(N)));
                HIP_TRY(dalloc(c, &c->rings, (size_t)2 * runs));
            } else {
                HIP_TRY(alloc_wide(c));
            }
            HIP_TRY(dalloc(c, &c->rd_cnt, (size_t)runs));
            HIP_TRY(upload(c, c->colpad, cp.data(), sizeof(int32_t) * cp.size()));
            HIP_TRY(upload(c, c->valpad, vp.data(), sizeof(float) * vp.size()));
        }
        HIP_TRY(settle(c));   // host staging buffers die here
        return SBQA_OK;
    }

    const int nkc = c->L.nkc, Cg = c->L.Cg;
    const size_t gbytes = (size_t)dense_plane_bytes(path, Cg, Np);
    HIP_TRY(dalloc(c, &c->x[0], (size_t)C * Np));
    HIP_TRY(dalloc(c, &c->x[1], (size_t)C * Np));
    HIP_TRY(dalloc(c, &c->y, (size_t)C * Np));
    for (int q = 0; q < 2; ++q) {
        uint8_t *gb, *glo = nullptr;
        HIP_TRY(dalloc(c, &gb, gbytes));
        if (path == PATH_BF16X3) HIP_TRY(dalloc(c, &glo, gbytes));
        c->g[q] = gb;
        c->g_lo[q] = glo;
    }
    if (!path_energy_mfma(path)) {   // readout spins and energy partials
        HIP_TRY(dalloc(c, &c->rspins, (size_t)Cp * Np));
        HIP_TRY(dalloc(c, &c->epart, (size_t)energy_plan(N, C).units * Cp));
    }
    if (c->resident) {
        // small dense loop: J float32 [N][N]
        std::vector<float> jsm((size_t)N * N);
        for (size_t q = 0; q < jsm.size(); ++q) jsm[q] = (float)J->dense[q];
        HIP_TRY(dalloc(c, &c->Jsm, jsm.size()));
        HIP_TRY(upload(c, c->Jsm, jsm.data(), sizeof(float) * jsm.size()));
        HIP_TRY(settle(c));   // host staging buffers die here
    }

    if (c->facts.jbits) {
        // +-1 J as sign bits: the bit-packed contraction copy is built from
        // them; no float64 copy (the readout energies run on MFMA)
        if (!jbits || !path_packed(path)) return fail(SBQA_EINVAL, "sign bits need a bit-packed +-1 path");
        uint8_t *jd;
        uint32_t *sb;
        const size_t words = (size_t)(N + 31) / 32;
        HIP_TRY(dalloc(c, &jd, (size_t)dense_j_bytes(path, Np)));
        HIP_TRY(dalloc(c, &sb, (size_t)N * words));
        c->Jd = jd;
        HIP_TRY(upload(c, sb, jbits, sizeof(uint32_t) * N * words));
        HIP_TRY(flush(c));
        HIP_TRY(launch_convert_j_bits(path, sb, N, Np, nkc, jd, c->stream));
        HIP_TRY(settle(c));   // the caller may free the bits on return
        return SBQA_OK;
    }
    // J in the contraction precision (fragment-tiled) and in float64
    // (row-major, energies), zero padded.
    const double *A = J->dense;
    uint8_t *jd, *jlo = nullptr;
    double *j64;
    HIP_TRY(dalloc(c, &jd, (size_t)dense_j_bytes(path, Np)));
    if (path == PATH_BF16X3) HIP_TRY(dalloc(c, &jlo, (size_t)dense_j_bytes(path, Np)));
    HIP_TRY(dalloc(c, &j64, (size_t)Np * Np));
    c->Jd = jd;
    c->Jd_lo = jlo;
    c->J64 = j64;
    // float64 J into the zero-padded row-major copy (energies), then the
    // contraction copy is derived from it on the device. The host array goes
    // up in one contiguous copy (a pitched copy from pageable memory is split
    // into one transfer per row); when rows need padding it lands in a
    // temporary buffer first and is spread into the padded rows on the GPU.
    PoolBlock tmp(c->device, false);
    struct Wait { sbqa_ctx *c; ~Wait() { (void)settle(c); } } wait{c};   // before tmp goes back, on every path
    if (N == Np) {
        HIP_TRY(upload(c, j64, A, sizeof(double) * N * N));
    } else {
        HIP_TRY(tmp.get(sizeof(double) * (size_t)N * N));
        c->direct = true;
        HIP_TRY(hipMemcpyAsync(tmp.as<double>(), A, sizeof(double) * N * N, hipMemcpyHostToDevice, c->stream));
        HIP_TRY(flush(c));
        HIP_TRY(launch_pad_rows(tmp.as<double>(), N, Np, j64, c->stream));
    }
    HIP_TRY(flush(c));
    HIP_TRY(launch_convert_j(path, j64, Np, nkc, jd, jlo, c->stream));
    if (c->mid.NT) {
        HIP_TRY(dalloc(c, &c->Jmid, (size_t)((N + 15) / 16) * c->mid_ns * 64));
        HIP_TRY(flush(c));
        HIP_TRY(launch_mid_bits(j64, N, Np, c->mid_ns, c->Jmid, c->stream));
        if (c->mid.G > 1) {
            HIP_TRY(dalloc(c, &c->words, (size_t)2 * c->mid_groups * c->mid.MB * ((N + 127) / 128) * 256));
            HIP_TRY(dalloc(c, &c->rings, (size_t)2 * c->mid_groups));
        }
    }
    HIP_TRY(settle(c));   // the caller may free J on return
    return SBQA_OK;
}

// Arguments of the dense step kernel at step n from operand/state buffer `in`.
static DenseStepArgs dense_args(sbqa_ctx *c, uint32_t n, int in) {
    DenseStepArgs a{};
    a.N = c->N;
    a.Np = c->L.Np;
    a.R = c->R;
    a.C = c->L.C;
    a.nkc = c->L.nkc;
    a.reverse = (int)(n & 1u);
    a.J = static_cast<const uint8_t *>(c->Jd);
    a.J_lo = static_cast<const uint8_t *>(c->Jd_lo);
    a.g = static_cast<const uint8_t *>(c->g[in]);
    a.g_lo = static_cast<const uint8_t *>(c->g_lo[in]);
    a.g_next = static_cast<uint8_t *>(c->g[1 - in]);
    a.g_next_lo = static_cast<uint8_t *>(c->g_lo[1 - in]);
    a.h = c->h32;
    a.x_in = c->x[in];
    a.x_out = c->x[1 - in];
    a.y = c->y;
    a.phi = nullptr;
    a.jp = c->jp + (n < c->s.steps ? n : 0);
    a.jp_stride = c->s.steps;
    a.k = step_coef(&c->s, c->c0, c->R, n);
    a.fmode = c->s.fmode;
    return a;
}

// One step of Eqs. 6-7 on the device (asynchronous).
sbqa_status ctx_step_once(sbqa_ctx *c) {
    const uint32_t n = c->step;
    const StepCoef k = step_coef(&c->s, c->c0, c->R, n);
    const float *jp = c->jp + n;
    const int64_t jp_stride = c->s.steps;
    const int in = c->cur, out = 1 - c->cur;
    if (c->facts.path == PATH_CSR) {
        HIP_TRY(launch_csr_step(c->s.fmode, c->N, c->L.Cs, c->R, c->runs, c->rp, c->col, c->val, c->tri3(), c->h32, c->x[in],
                                c->x[out], c->y, (const int8_t *)c->g[in], (int8_t *)c->g[out], jp, jp_stride, k,
                                c->stream));
    } else {
        const DenseStepArgs a = dense_args(c, n, in);
        HIP_TRY(launch_dense_step(c->facts.path, EPI_UPDATE, c->L.form, c->L.mbw, c->L.Cg, a, c->stream));
    }
    c->cur = out;
    c->step = n + 1;
    return SBQA_OK;
}

// The sign bytes the resident loop wrote for the current state, or nullptr
// when the state has been replaced since.
static const uint8_t *colblock_signs(const sbqa_ctx *c) {
    return c->sbits_step == (int64_t)c->step ? c->sbits : nullptr;
}

// Energies of the readout of the current state into c->E[0..C).
sbqa_status ctx_state_energies(sbqa_ctx *c) {
    const bool sm = c->facts.path == PATH_CSR;
    const double *h64 = c->has_h ? c->h64 : nullptr;
    if (sm && c->order == ORDER_COLBLOCK8 && !c->facts.n3) {
        const int nrb = c->L.csr_nrb, rpb = (c->N + nrb - 1) / nrb;
        HIP_TRY(launch_csr_energy_colblock(c->N, c->ld, c->L.C, c->res_D, nrb, rpb, c->rcol, c->rval, c->rh,
                                           c->x[c->cur], colblock_signs(c), c->E, c->stream));
    } else if (sm) {
        HIP_TRY(launch_csr_energy_state(c->N, c->order, c->ld, c->L.C, c->rp, c->col, c->val64, c->tri3(), h64, c->x[c->cur],
                                        c->csr_partial, c->L.csr_nrb, c->E, c->stream));
    } else if (c->facts.path == PATH_FP8 || c->facts.path == PATH_FP8PK || c->facts.path == PATH_I8 ||
               path_fp4(c->facts.path)) {
        // integer J: J s on MFMA is exact, so the energies equal the float64
        // ones bit for bit; the free halves of the ping-pong buffers (written
        // in full by the next step before they are read) hold the readout
        // operand and its fields
        const int in = c->cur, sc = 1 - c->cur;
        HIP_TRY(launch_readout_operand(c->facts.path, c->N, c->L.Np, c->L.C, c->L.nkc, c->L.mbw, c->x[in], c->g[sc],
                                       c->stream));
        DenseStepArgs a = dense_args(c, c->step, in);
        a.g = static_cast<const uint8_t *>(c->g[sc]);
        a.phi = c->x[sc];
        HIP_TRY(launch_dense_step(c->facts.path, EPI_FIELDS, c->L.form, c->L.mbw, c->L.Cg, a, c->stream));
        HIP_TRY(launch_energy_fields(c->N, c->L.Np, c->L.C, c->x[in], c->x[sc], h64, c->E, c->stream));
    } else {
        const EnergyPlan e = energy_plan(c->N, c->L.C);
        HIP_TRY(launch_readout_spins(c->N, c->L.Np, c->L.C, e.cp, c->x[c->cur], c->rspins, c->stream));
        HIP_TRY(launch_energy_gemm(e, c->rspins, c->J64, c->L.Np, c->epart, c->stream));
        HIP_TRY(launch_energy_sum(e, c->N, c->L.Np, c->L.C, c->epart, c->rspins, h64, c->E, c->stream));
    }
    return SBQA_OK;
}

sbqa_status ctx_energies_dev(sbqa_ctx *c, const int8_t *ds, int32_t count, double *E, int8_t *S, double *P) {
    const int N = c->N;
    if (c->facts.path != PATH_CSR && !c->J64)
        return fail(SBQA_EINVAL, "this context keeps no float64 copy of J (built from sign bits)");
    const double *h64 = c->has_h ? c->h64 : nullptr;
    if (c->facts.path == PATH_CSR) {
        HIP_TRY(launch_csr_energy_spins(N, count, c->rp, c->col, c->val64, c->tri3(), h64, ds, E, c->stream));
    } else {
        const EnergyPlan e = energy_plan(N, count);
        HIP_TRY(launch_pad_spins(N, c->L.Np, count, e.cp, ds, S, c->stream));
        HIP_TRY(launch_energy_gemm(e, S, c->J64, c->L.Np, P, c->stream));
        HIP_TRY(launch_energy_sum(e, N, c->L.Np, count, P, S, h64, E, c->stream));
    }
    return SBQA_OK;
}

sbqa_status ctx_evaluate(sbqa_ctx *c, bool reset) {
    sbqa_status st = ctx_state_energies(c);
    if (st != SBQA_OK) return st;
    // (the partials of the energies just summed are free again)
    int *sel = c->bsel ? c->bsel : reinterpret_cast<int *>(c->csr_partial);
    HIP_TRY(launch_best_update(c->N, c->R, c->runs, c->order, c->ld, c->x[c->cur], c->E, c->bestE, c->bestStep,
                               c->bestSpins, (int64_t)c->step, reset, sel, c->stream));
    c->last_eval_step = c->step;
    return SBQA_OK;
}

// No best solution yet. The values go up from the pinned readout block, which
// the host writes nowhere else.
sbqa_status ctx_reset_best(sbqa_ctx *c) {
    double *inf = reinterpret_cast<double *>(c->rhost);
    for (int r = 0; r < c->runs; ++r) inf[r] = INFINITY;
    HIP_TRY(hipMemcpyAsync(c->bestE, inf, sizeof(double) * c->runs, hipMemcpyHostToDevice, c->stream));
    c->last_eval_step = -1;
    return SBQA_OK;
}

// Whether the register-resident CSR loop fits this instance on this device.
static bool resident_plan(sbqa_ctx *c, const sbqa_coupling *J, std::string *why) {
    if (c->s.fmode == SBQA_F_BALLISTIC) { *why = "ballistic f needs a float32 operand"; return false; }
    if (c->facts.n3) { *why = "three-body terms run on the streaming kernel"; return false; }
    if (c->R % resident_cols()) { *why = "R is not a multiple of 8"; return false; }
    const int rpt = resident_rpt(c->N);
    if (rpt < 0 || c->N > 65535) { *why = "N above 4096"; return false; }
    int maxdeg = 0;
    for (int i = 0; i < c->N; ++i) maxdeg = std::max(maxdeg, J->row_ptr[i + 1] - J->row_ptr[i]);
    const int D = resident_degree(maxdeg);
    if (D < 0) { *why = "degree above 16"; return false; }
    if (resident_rows(c->N) > 2048 && D > 6) { *why = "N above 2048 with degree above 6 exceeds the register budget"; return false; }
    const size_t lds = resident_lds_bytes(c->N, D);
    if (lds > 160 * 1024) { *why = "LDS demand above 160 KiB"; return false; }
    int bpc = 0, cus = 0;
    if (resident_max_blocks(D, c->N, &bpc) != hipSuccess) { *why = "occupancy query failed"; return false; }
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) { *why = "no CU count"; return false; }
    const int nwg = c->L.C / resident_cols();
    if (nwg > bpc * cus) { *why = "more column blocks than co-resident workgroups"; return false; }
    c->res_D = D;
    c->res_rows = resident_rows(c->N);
    c->res_nwg = nwg;
    c->res_W = resident_cols();
    c->cus = cus;
    c->exchanging = Exchanging{nwg, ((uint64_t)1 << 60) | (uint64_t)c->res_rows << 8 | (uint64_t)D, bpc};
    c->exchanging_wide = c->exchanging;
    // Fewer columns per workgroup (the narrow loop) while the workgroups of
    // four launches still fit on the device together, so that four contexts on
    // streams of their own need not wait for each other (launch_in_order). Two
    // columns up to a quarter of the CUs (128 columns), else four. us per step for W = 8 / 4 / 2: N =
    // 1000, degree 3, C = 128 2.48 / 1.20 / 1.12; N = 4096, degree 6, C = 128
    // 6.20 / 4.35 / 2.94; C = 256 6.33 / 4.41 / 3.81 (two columns do not fit
    // four times there); N = 1000, degree 6, C = 512 2.81 / 1.41 / 1.93 (twice
    // the edge words).
    for (int W : {2, 4}) {
        int nb = 0;
        if (narrow_max_blocks(D, W, c->N, &nb) != hipSuccess || nb < 1) continue;
        if ((int64_t)c->L.C / W * 4 > (int64_t)cus * (W == 2 ? 1 : nb)) continue;
        c->res_W = W;
        c->res_nwg = c->L.C / W;
        c->exchanging = Exchanging{c->res_nwg, ((uint64_t)2 << 60) | (uint64_t)narrow_rows(c->N) << 16 | (uint64_t)D << 8 | (uint64_t)W, nb};
        break;
    }
    return true;
}

// Whether the small dense resident loop fits this instance.
static bool small_plan(sbqa_ctx *c, std::string *why) {
    if (c->facts.path == PATH_BF16X3) { *why = "the small dense loop computes in float32 (every precision but BF16X3)"; return false; }
    if (c->N > SMALL_MAX_N) { *why = "N is above the small dense loop's limit"; return false; }
    if ((int64_t)c->R * c->N > SMALL_MAX_ELEMS) { *why = "R*N is above the small dense loop's limit"; return false; }
    if (small_lds_bytes(c->N, c->R) > 160 * 1024) { *why = "the run state does not fit in LDS"; return false; }
    return true;
}

// The many-step loop of dense +-1 instances (kernels_mid.hip), taken with
// LOOP_AUTO where no small loop fits: groups of 16 or 32 replica columns made
// of whole runs, G workgroups per group. Every path but BF16X3 gives the same
// bits as the loop (exact integer sums). Leaves c->mid.NT 0 when unfit.
static void mid_plan(sbqa_ctx *c) {
    c->mid = MidPlan{};
    if (!c->facts.pm1 || c->facts.jbits || c->facts.path == PATH_BF16X3 || c->s.fmode == SBQA_F_BALLISTIC) return;
    if (c->N > MID_MAX_N || c->R > 32) return;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) return;
    MidPlan p;
    p.MB = c->R > 16 ? 2 : 1;
    p.rot = c->R == 16 * p.MB;
    const int cols = 16 * p.MB / c->R * c->R, groups = (c->L.C + cols - 1) / cols;
    const int nrb = (c->N + 15) / 16;
    const int ns = (c->N + 511) / 512;
    p.NS = ns <= 2 ? ns : 4;
    // Fewest row blocks per workgroup first, so that a step is short, while
    // the workgroups of four launches still fit on the device together (see
    // resident_plan); one workgroup per group waits for nobody. us per
    // step, one launch per step / this loop, at C = 128: N = 300 6.5 / 1.7, N
    // = 601 7.2 / 1.9, N = 1024 7.2 / 2.2, N = 2048 8.6 / 3.0; C = 1600, N =
    // 1000 11.1 / 6.1 (four row blocks per wave, one workgroup per group).
    // Above MID_MAX_N the exchanged operand and the bits of J (registers)
    // grow past what a step saves.
    struct Shape { int NT, RBW; };
    const Shape shapes[] = {{512, 1}, {1024, 1}, {1024, 2}, {1024, 4}};
    auto fits = [&](const Shape &sh, bool alone) {
        const int per = sh.NT / 64 * sh.RBW;
        p.NT = sh.NT;
        p.RBW = sh.RBW;
        p.G = (nrb + per - 1) / per;
        if ((p.G == 1) != alone) return false;
        int nb = 0;
        if (mid_max_blocks(p, &nb) != hipSuccess || nb < 1) return false;
        c->exchanging = alone ? Exchanging{}
                              : Exchanging{groups * p.G,
                                           ((uint64_t)3 << 60) | (uint64_t)p.NT << 20 | (uint64_t)p.RBW << 16 |
                                               (uint64_t)p.NS << 12 | (uint64_t)p.MB << 8 | (uint64_t)p.rot,
                                           nb};
        return alone || (int64_t)groups * p.G * 4 <= (int64_t)cus * nb;
    };
    bool ok = fits({1024, 1}, true);                       // up to 256 spins
    for (int q = 0; q < 3 && !ok; ++q) ok = fits(shapes[q], false);
    for (int q = 2; q < 4 && !ok; ++q) ok = fits(shapes[q], true);
    if (!ok) {
        c->exchanging = Exchanging{};
        return;
    }
    c->cus = cus;
    c->mid = p;
    c->mid_cols = cols;
    c->mid_groups = groups;
    c->mid_ns = ns;
}

// ---------------------------------------------------------------------------
// Internal relabelling of CSR spins for cache locality (sbqa_reorder).
// ---------------------------------------------------------------------------

// Undirected adjacency of the pairs and of the triples' members, as offsets
// and neighbour lists (duplicates allowed).
static void spin_adjacency(const sbqa_coupling *J, int32_t N, std::vector<int64_t> *aptr, std::vector<int32_t> *adj) {
    std::vector<int64_t> deg((size_t)N + 1, 0);
    for (int32_t i = 0; i < N; ++i) deg[(size_t)i + 1] += J->row_ptr[i + 1] - J->row_ptr[i];
    for (int64_t t = 0; t < J->n3; ++t)
        for (int e = 0; e < 3; ++e) deg[(size_t)J->tri[3 * t + e] + 1] += 2;
    for (int32_t i = 0; i < N; ++i) deg[(size_t)i + 1] += deg[(size_t)i];
    adj->assign((size_t)deg[(size_t)N], 0);
    std::vector<int64_t> fill(deg.begin(), deg.end() - 1);
    for (int32_t i = 0; i < N; ++i)
        for (int32_t p = J->row_ptr[i]; p < J->row_ptr[i + 1]; ++p) (*adj)[(size_t)fill[(size_t)i]++] = J->col[p];
    for (int64_t t = 0; t < J->n3; ++t)
        for (int e = 0; e < 3; ++e) {
            const int32_t *v = J->tri + 3 * t;
            (*adj)[(size_t)fill[(size_t)v[e]]++] = v[(e + 1) % 3];
            (*adj)[(size_t)fill[(size_t)v[e]]++] = v[(e + 2) % 3];
        }
    *aptr = std::move(deg);
}

// Mean |label(i) - label(j)| over the adjacency (label = identity when pnew
// is empty).
static double mean_span(const std::vector<int64_t> &aptr, const std::vector<int32_t> &adj, int32_t N,
                        const std::vector<int32_t> &pnew) {
    if (adj.empty()) return 0.0;
    double sum = 0.0;
    for (int32_t i = 0; i < N; ++i)
        for (int64_t p = aptr[(size_t)i]; p < aptr[(size_t)i + 1]; ++p) {
            const int32_t j = adj[(size_t)p];
            sum += pnew.empty() ? std::fabs((double)i - j) : std::fabs((double)pnew[(size_t)i] - pnew[(size_t)j]);
        }
    return sum / (double)adj.size();
}

// Reverse Cuthill-McKee order: breadth-first through every connected
// component, each started at its lowest-degree unvisited spin, neighbours
// taken by increasing degree; the whole order reversed. pnew[i] = new label.
static void rcm_order(const std::vector<int64_t> &aptr, const std::vector<int32_t> &adj, int32_t N,
                      std::vector<int32_t> *pnew) {
    std::vector<int32_t> byDeg((size_t)N), order;
    order.reserve((size_t)N);
    for (int32_t i = 0; i < N; ++i) byDeg[(size_t)i] = i;
    auto deg = [&](int32_t i) { return aptr[(size_t)i + 1] - aptr[(size_t)i]; };
    std::stable_sort(byDeg.begin(), byDeg.end(), [&](int32_t a, int32_t b) { return deg(a) < deg(b); });
    std::vector<char> seen((size_t)N, 0);
    std::vector<int32_t> nb;
    for (int32_t start : byDeg) {
        if (seen[(size_t)start]) continue;
        seen[(size_t)start] = 1;
        size_t head = order.size();
        order.push_back(start);
        while (head < order.size()) {
            const int32_t u = order[head++];
            nb.clear();
            for (int64_t p = aptr[(size_t)u]; p < aptr[(size_t)u + 1]; ++p) {
                const int32_t v = adj[(size_t)p];
                if (!seen[(size_t)v]) { seen[(size_t)v] = 1; nb.push_back(v); }
            }
            std::stable_sort(nb.begin(), nb.end(), [&](int32_t a, int32_t b) { return deg(a) < deg(b); });
            order.insert(order.end(), nb.begin(), nb.end());
        }
    }
    pnew->assign((size_t)N, 0);
    for (int32_t k = 0; k < N; ++k) (*pnew)[(size_t)order[(size_t)(N - 1 - k)]] = k;
}

// Whether (and how) to relabel a CSR instance's spins (sbqa_reorder).
static void plan_reorder(const sbqa_coupling *J, int32_t N, int mode, std::vector<int32_t> *pnew) {
    pnew->clear();
    if (mode == SBQA_REORDER_OFF || (J->nnz == 0 && J->n3 == 0)) return;
    if (mode == SBQA_REORDER_AUTO && N < 16384) return;
    std::vector<int64_t> aptr;
    std::vector<int32_t> adj;
    spin_adjacency(J, N, &aptr, &adj);
    const double before = mean_span(aptr, adj, N, {});
    if (mode == SBQA_REORDER_AUTO && before <= (double)N / 64.0) return;
    std::vector<int32_t> p;
    rcm_order(aptr, adj, N, &p);
    if (mode == SBQA_REORDER_AUTO && mean_span(aptr, adj, N, p) * 4.0 > before) return;
    *pnew = std::move(p);
}

// The coupling with spins relabelled by pnew: row pnew[i] holds spin i's
// couplings in the given order (columns relabelled), triples keep their
// order with relabelled members; h permuted alike. The vectors own the data.
struct Relabelled {
    std::vector<int32_t> rp, col, tri;
    std::vector<double> val, h;
    sbqa_coupling J{};
};
static void relabel(const sbqa_coupling *J, const double *h, int32_t N, const std::vector<int32_t> &pnew,
                    Relabelled *r) {
    std::vector<int32_t> orig((size_t)N);
    for (int32_t i = 0; i < N; ++i) orig[(size_t)pnew[(size_t)i]] = i;
    r->rp.assign((size_t)N + 1, 0);
    for (int32_t k = 0; k < N; ++k) {
        const int32_t i = orig[(size_t)k];
        r->rp[(size_t)k + 1] = r->rp[(size_t)k] + (J->row_ptr[i + 1] - J->row_ptr[i]);
    }
    r->col.resize((size_t)J->nnz);
    r->val.resize((size_t)J->nnz);
    for (int32_t k = 0; k < N; ++k) {
        const int32_t i = orig[(size_t)k];
        int64_t q = r->rp[(size_t)k];
        for (int32_t p = J->row_ptr[i]; p < J->row_ptr[i + 1]; ++p, ++q) {
            r->col[(size_t)q] = pnew[(size_t)J->col[p]];
            r->val[(size_t)q] = J->val[p];
        }
    }
    r->tri.resize((size_t)3 * J->n3);
    for (int64_t q = 0; q < 3 * J->n3; ++q) r->tri[(size_t)q] = pnew[(size_t)J->tri[q]];
    if (h) {
        r->h.resize((size_t)N);
        for (int32_t i = 0; i < N; ++i) r->h[(size_t)pnew[(size_t)i]] = h[i];
    }
    r->J = *J;
    r->J.row_ptr = r->rp.data();
    r->J.col = r->col.data();
    r->J.val = r->val.data();
    r->J.tri = J->n3 ? r->tri.data() : nullptr;
}

// The stream of the contexts created without one: one non-blocking stream per
// device, created at the first such context and kept until the process ends
// (a stream per context cost a hardware queue's creation, 3.5 ms, for each of
// the first few contexts of a process). Their work is ordered on it;
// sbqa_set_stream gives a context a stream of the caller's.
static hipError_t library_stream(int device, hipStream_t *out) {
    static std::mutex mu;
    static std::map<int, hipStream_t> streams;
    std::lock_guard<std::mutex> lk(mu);
    auto it = streams.find(device);
    if (it != streams.end()) {
        *out = it->second;
        return hipSuccess;
    }
    hipStream_t st = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
    streams[device] = st;
    *out = st;
    return hipSuccess;
}

static sbqa_status create(const sbqa_coupling *J, const double *h, int32_t N, int32_t R, int32_t runs,
                          const sbqa_schedule *s, const InstanceFacts &facts, hipStream_t stream, sbqa_ctx **out,
                          bool allow_resident, const uint32_t *jbits) {
    std::unique_ptr<sbqa_ctx> owner(new sbqa_ctx());
    sbqa_ctx *c = owner.get();
    c->N = N;
    c->R = R;
    c->runs = runs;
    c->s = *s;
    c->s.beta = c->s.alpha = nullptr;
    c->s.jp_table = nullptr;
    c->facts = facts;
    c->c0 = s->c0 > 0 ? s->c0 : (facts.rms > 0 ? 0.5 / (std::sqrt((double)N) * facts.rms) : 0.0);
    plan_layout(N, R, runs, facts, &c->L);
    build_schedule_host(s, runs, c->beta, c->alpha, c->jp_host);
    sbqa_status st = check_device(&c->device);
    if (st != SBQA_OK) return st;
    if (stream) c->stream = stream;
    else {
        hipError_t e = library_stream(c->device, &c->default_stream);
        if (e != hipSuccess) return fail(SBQA_EDEVICE, "hipStreamCreate: %s", hipGetErrorString(e));
        c->stream = c->default_stream;
    }
    Relabelled rl;
    if (facts.path == PATH_CSR) {
        plan_reorder(J, N, s->reorder, &c->pnew);
        if (!c->pnew.empty()) {
            relabel(J, h, N, c->pnew, &rl);
            J = &rl.J;
            h = h ? rl.h.data() : nullptr;
        }
    }
    const bool served = !allow_resident;       // stepped by the grouped launches
    if (facts.jbits) allow_resident = false;   // the small dense loop needs J in float32
    {
        std::string why;
        const bool plan = facts.path == PATH_CSR ? resident_plan(c, J, &why) : small_plan(c, &why);
        c->resident = allow_resident && s->loop_kernel != SBQA_LOOP_STREAM && plan;
        if (!c->resident && s->loop_kernel == SBQA_LOOP_RESIDENT) {
            return fail(SBQA_EINVAL, "instance does not fit a resident loop: %s",
                        allow_resident ? why.c_str() : "contexts of the serving loop step one launch at a time");
        }
        if (!c->resident) c->exchanging = Exchanging{};
        if (facts.path != PATH_CSR && !c->resident && allow_resident && s->loop_kernel == SBQA_LOOP_AUTO) mid_plan(c);
    }
    if (facts.path != PATH_CSR)
        set_tile(&c->L, facts.path, s->dense_tile, served, c->stream);
    if (facts.path != PATH_CSR) {
        c->order = ORDER_REPLICA_MAJOR;
        c->ld = c->L.Np;
    } else if (c->resident) {
        c->order = ORDER_COLBLOCK8;   // C is a multiple of 8 (R is), so Cs == C
        c->ld = c->res_rows;
    } else {
        c->order = ORDER_SPIN_MAJOR;
        c->ld = c->L.Cs;
    }
    st = ctx_upload(c, J, h, jbits);
    if (st == SBQA_OK && !c->pnew.empty()) {
        std::vector<int32_t> orig((size_t)N);
        for (int32_t i = 0; i < N; ++i) orig[(size_t)c->pnew[(size_t)i]] = i;
        hipError_t e = dalloc(c, &c->porig, (size_t)N);
        if (e == hipSuccess) e = dalloc(c, &c->pos, (size_t)N);
        if (e == hipSuccess) e = upload(c, c->porig, orig.data(), sizeof(int32_t) * N);
        if (e == hipSuccess) e = upload(c, c->pos, c->pnew.data(), sizeof(int32_t) * N);
        if (e == hipSuccess) e = settle(c);   // the staging vector dies here
        if (e != hipSuccess) st = fail(SBQA_EDEVICE, "relabelling: %s", hipGetErrorString(e));
    }
    c->creating = false;
    if (st == SBQA_OK) {
        hipError_t e = flush(c);
        if (e == hipSuccess)
            e = launch_init_state(N, c->L.C, c->order, c->ld, s->seed, s->init_amp, c->porig, c->x[0], c->y, c->stream);
        if (e != hipSuccess) st = fail(SBQA_EDEVICE, "init: %s", hipGetErrorString(e));
    }
    if (st == SBQA_OK) st = rebuild_operand(c);
    if (st == SBQA_OK) st = ctx_reset_best(c);
    if (st != SBQA_OK) return st;
    *out = owner.release();
    return SBQA_OK;
}

sbqa_status ctx_create(const sbqa_coupling *J, const double *h, int32_t N, int32_t R, int32_t runs,
                       const sbqa_schedule *s, const InstanceFacts &facts, hipStream_t stream, sbqa_ctx **out,
                       bool allow_resident, const uint32_t *jbits) {
    return guarded([&] { return create(J, h, N, R, runs, s, facts, stream, out, allow_resident, jbits); });
}

// K steps of the small dense loop in one launch (one workgroup per run).
static sbqa_status ctx_step_small(sbqa_ctx *c, uint32_t K) {
    SmallArgs a;
    a.N = c->N;
    a.Np = c->L.Np;
    a.R = c->R;
    a.S = (int)c->s.steps;
    a.n0 = (int)c->step;
    a.K = (int)K;
    a.fmode = c->s.fmode;
    a.jbits = c->facts.ternary ? 1 : 0;
    a.J = c->Jsm;
    a.h = c->h32;
    a.x = c->x[c->cur];
    a.y = c->y;
    a.jp = c->jp;
    a.coefA = c->coefA;
    a.delta = c->delta_tab;
    const StepCoef k = step_coef(&c->s, c->c0, c->R, c->step);
    a.kB = k.kB;
    a.dt = k.dt;
    a.kD = k.kD;
    HIP_TRY(launch_dense_small(a, c->runs, c->stream));
    c->step += K;
    c->g_stale = true;
    return SBQA_OK;
}

// The fewest steps for which a launch of the many-step loop is the faster way;
// fewer are taken one launch of the step kernel each, whose operand the state then
// carries. us for 1 / 2 / 4 / 8 / 16 steps, step kernel and loop:
//   one row block per wave: N = 700, C = 128 5 10 20 40 81 and 7 8 12 21 38; N = 130, C = 640
//     5.8 11 23 43 92 and 4.8 5.6 7.4 11 19
//   two column blocks above 1024 spins: N = 2048, R = 32, C = 256 6.6 13 27 52 105 and 12.5 18 30 53 98
//   two row blocks, several workgroups: N = 1500, C = 320 6.6 14 26 53 104 and 11 16 25 44 83
//   four row blocks, one workgroup per group (a * N + b + (c * N + d) K against the
//     step kernel's time): N = 1000, C = 640 7 14 28 55 114 and 22 28 40 64 114;
//     N = 700, C = 640 6.7 14 27 56 107 and 18 22 31 48 82; N = 1000, C = 1600
//     11 22 44 88 177 and 23 29 41 66 114.
static uint32_t mid_min_steps(const sbqa_ctx *c) {
    const double N = c->N, C = c->L.C;
    if (c->N <= 256 && c->mid.MB == 1 && C >= 512) return 1;
    if (c->mid.RBW == 4) {
        const double gain = (4.3 + 0.0042 * C) - (0.1 + 0.006 * N);
        return (uint32_t)std::min(64.0, std::ceil((7.2 + 0.009 * N) / std::max(gain, 0.1)));
    }
    if (c->mid.MB == 2 && c->N > 1024) return 6;
    return c->mid.RBW == 2 && c->mid.G > 1 ? (c->N > 1024 ? 4 : 3) : 2;
}

// K steps of the many-step loop of a dense +-1 instance in one launch.
static sbqa_status ctx_step_mid(sbqa_ctx *c, uint32_t K) {
    MidArgs a;
    a.N = c->N;
    a.Np = c->L.Np;
    a.R = c->R;
    a.C = c->L.C;
    a.S = (int)c->s.steps;
    a.n0 = (int)c->step;
    a.K = (int)K;
    a.fmode = c->s.fmode;
    a.G = c->mid.G;
    a.groups = c->mid_groups;
    a.cols = c->mid_cols;
    a.ns = c->mid_ns;
    a.J = c->Jmid;
    a.h = c->h32;
    a.x = c->x[c->cur];
    a.y = c->y;
    a.jp = c->jp;
    a.coefA = c->coefA;
    a.delta = c->delta_tab;
    const StepCoef k = step_coef(&c->s, c->c0, c->R, c->step);
    a.kB = k.kB;
    a.dt = k.dt;
    a.kD = k.kD;
    a.words = c->words;
    a.rings = c->rings;
    a.err = c->err;
    HIP_TRY(launch_in_order(c, c->exchanging, [&] { return launch_dense_mid(c->mid, a, c->stream); }));
    c->step += K;
    c->g_stale = true;
    return SBQA_OK;
}

// Whether a context of the narrow loop takes K steps with 8 columns per
// workgroup: a launch of the narrow loop reads the couplings by more workgroups
// and ends with the ring's count, which few steps of it do not make up for. us for
// 1 and 4 steps, 8 columns / narrow: N = 200, C = 1024 5.6, 13.1 / 10.0, 14.6; N =
// 1000, C = 512 6.5, 15.4 / 9.6, 15.0; C = 256 6.1, 14.8 / 7.4, 11.7; N = 4096, C = 128
// 13.7, 31.2 / 16.1, 24.5; but N = 1000, C = 64 5.5 / 5.8, C = 32 5.5 / 5.2. Not when recorded:
// the counters of the 8-column loop tell a launch from the one before it, not from
// the same one replayed. Its buffers are taken at the first such call.
static bool wide_step(sbqa_ctx *c, uint32_t K) {
    if (c->L.C < 128 || c->recorded || (int64_t)K > c->L.C / 256 + (c->L.C < 256)) return false;
    if (c->sbits) return true;
    if (alloc_wide(c) == hipSuccess) return true;
    (void)hipGetLastError();   // no room: the narrow loop does it
    c->sbits = nullptr;
    return false;
}

// K steps of the register-resident loop in one launch. A wait that timed out
// sets the error word of the readout block, which every synchronising call
// copies back and reports.
static sbqa_status ctx_step_resident(sbqa_ctx *c, uint32_t K) {
    if (c->mid.NT) {
        if (c->recorded || K >= mid_min_steps(c)) return ctx_step_mid(c, K);
        sbqa_status st = c->g_stale ? rebuild_operand(c) : SBQA_OK;
        for (uint32_t q = 0; q < K && st == SBQA_OK; ++q) st = ctx_step_once(c);
        return st;
    }
    if (c->facts.path != PATH_CSR) return ctx_step_small(c, K);
    const bool narrow = c->res_W < resident_cols() && !wide_step(c, K);
    ResidentArgs a;
    a.N = c->N;
    a.R = c->R;
    a.S = (int)c->s.steps;
    a.n0 = (int)c->step;
    a.K = (int)K;
    a.fmode = c->s.fmode;
    a.nwg = narrow ? c->res_nwg : c->L.C / resident_cols();
    a.colpad = c->colpad;
    a.valpad = c->valpad;
    a.h = c->h32;
    a.x = c->x[c->cur];
    a.y = c->y;
    a.jp = c->jp;
    a.coefA = c->coefA;
    a.delta = c->delta_tab;
    const StepCoef k = step_coef(&c->s, c->c0, c->R, c->step);
    a.kB = k.kB;
    a.dt = k.dt;
    a.kD = k.kD;
    a.xpub = c->xpub;
    a.flags = c->flags;
    a.epoch_cnt = c->epoch_cnt;
    a.epoch = ++c->epoch;
    a.err = c->err;
    a.nr = c->res_rows;
    a.sbits = c->sbits;
    if (narrow) {
        HIP_TRY(launch_in_order(c, c->exchanging, [&] {
            return launch_csr_narrow(a, c->res_D, c->res_W, c->words, c->rings, c->stream);
        }));
        c->step += K;
        return SBQA_OK;
    }
    HIP_TRY(launch_in_order(c, c->exchanging_wide, [&] { return launch_csr_resident(a, c->res_D, c->stream); }));
    c->step += K;
    c->sbits_step = c->step;
    return SBQA_OK;
}

sbqa_status ctx_check_async(sbqa_ctx *c) {
    if (c->rhost && *reinterpret_cast<const int *>(c->rhost + (size_t)8 * c->runs))
        return fail(SBQA_EDEVICE, "many-step loop: a ring-neighbour wait timed out; the state is invalid");
    return SBQA_OK;
}

sbqa_status ctx_sync(sbqa_ctx *c) {
    HIP_TRY(hipMemcpyAsync(c->rhost + (size_t)8 * c->runs, c->err, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return ctx_check_async(c);
}

sbqa_status ctx_step(sbqa_ctx *c, uint32_t n) {
    if ((uint64_t)c->step + n > c->s.steps)
        return fail(SBQA_ESTATE, "step %u + %u exceeds the schedule of %u steps", c->step, n, c->s.steps);
    note_recording(c);
    if (c->resident || c->mid.NT) {
        uint32_t left = n;
        while (left) {
            uint32_t K = left;
            if (c->exchanging.workgroups) K = std::min(K, MAX_EXCHANGE_STEPS);
            if (c->s.energy_every) K = std::min(K, c->s.energy_every - c->step % c->s.energy_every);
            sbqa_status st = ctx_step_resident(c, K);
            if (st != SBQA_OK) return st;
            left -= K;
            if (c->s.energy_every && c->step % c->s.energy_every == 0) {
                st = ctx_evaluate(c);
                if (st != SBQA_OK) return st;
            }
        }
        return SBQA_OK;
    }
    for (uint32_t q = 0; q < n; ++q) {
        sbqa_status st = ctx_step_once(c);
        if (st != SBQA_OK) return st;
        if (c->s.energy_every && c->step % c->s.energy_every == 0) {
            st = ctx_evaluate(c);
            if (st != SBQA_OK) return st;
        }
    }
    return SBQA_OK;
}

// Readout: without energy tracking the best of the current state alone
// (the previous best discarded on the device, no host round trip); then the
// readout block (best energies, error word, best spins) in one copy to the
// pinned host block. Nothing waits: the results are there once the context's
// stream has passed this point.
sbqa_status ctx_readout_async(sbqa_ctx *c) {
    const bool reset = c->s.energy_every == 0;
    const bool eval = reset || c->last_eval_step != (int64_t)c->step;
    if (eval && c->rd_cnt && c->rhost_dev && c->order == ORDER_COLBLOCK8 && !c->facts.n3) {
        // resident context: energies, best update and the host block in one
        // launch (the same values as the three-launch form below)
        const int nrb = c->L.csr_nrb, rpb = (c->N + nrb - 1) / nrb;
        ReadoutFuse f;
        f.R = c->R;
        f.runs = c->runs;
        f.best_E = c->bestE;
        f.best_step = c->bestStep;
        f.best_spins = c->bestSpins;
        f.err = c->err;
        f.cnt = c->rd_cnt;
        f.host = c->rhost_dev;
        f.step = (int64_t)c->step;
        f.reset = reset ? 1 : 0;
        HIP_TRY(launch_csr_readout_colblock(c->N, c->ld, c->L.C, c->res_D, nrb, rpb, c->rcol, c->rval, c->rh,
                                            c->x[c->cur], colblock_signs(c), c->E, f, c->stream));
        c->last_eval_step = c->step;
        return SBQA_OK;
    }
    if (eval) {
        sbqa_status st = ctx_evaluate(c, reset);
        if (st != SBQA_OK) return st;
    }
    // a copy kernel right behind the readout kernels (a runtime copy started
    // 11 us after the last kernel had finished)
    if (c->rhost_dev) HIP_TRY(launch_copy_to_host(c->rdev, c->rhost_dev, c->rbytes, c->stream));
    else HIP_TRY(hipMemcpyAsync(c->rhost, c->rdev, c->rbytes, hipMemcpyDeviceToHost, c->stream));
    return SBQA_OK;
}

// The results of the last ctx_readout_async, once its work has completed.
sbqa_status ctx_readout_collect(sbqa_ctx *c, double *energies, int8_t *spins) {
    const double *bE = reinterpret_cast<const double *>(c->rhost);
    const int8_t *bS = reinterpret_cast<const int8_t *>(c->rhost + (size_t)8 * c->runs + 8);
    if (energies) std::memcpy(energies, bE, sizeof(double) * c->runs);
    if (spins) {
        if (c->pnew.empty()) std::memcpy(spins, bS, (size_t)c->runs * c->N);
        else   // back to the caller's spin order
            for (int r = 0; r < c->runs; ++r)
                for (int i = 0; i < c->N; ++i)
                    spins[(size_t)r * c->N + i] = bS[(size_t)r * c->N + c->pnew[(size_t)i]];
    }
    return ctx_check_async(c);
}

sbqa_status ctx_best(sbqa_ctx *c, double *energies, int8_t *spins) {
    sbqa_status st = ctx_readout_async(c);
    if (st != SBQA_OK) return st;
    HIP_TRY(hipStreamSynchronize(c->stream));
    return ctx_readout_collect(c, energies, spins);
}

// The state from (set) or to the caller's arrays x, y (spin rows of C columns;
// null: skipped), through pinned memory that the device reads or writes itself,
// larger ones to the caller in slabs of rows: no device memory is needed, whatever
// the state's size, and a small state costs two launches and a wait (N * C = 8000:
// get 25 us, set 23; two copies through a device buffer 61). A larger state is set by
// copies into a device buffer where there is room for one (N = 200000, C = 256: 22
// ms, through pinned memory 31). Padding rows and columns hold zero and are not
// written. Returns with the work completed; set rebuilds the operand.
static sbqa_status transfer_state(sbqa_ctx *c, float *x, float *y, bool set) {
    const int N = c->N, C = c->L.C;
    const size_t row = sizeof(float) * C;
    const bool whole = set || 2 * row * N <= STAGE_BYTES;
    const int per = whole ? N : (int)std::max<size_t>(1, STAGE_BYTES / 2 / row);   // rows of a slab
    PoolBlock stage(c->device, true), dev(c->device, false);
    struct Wait { hipStream_t st; ~Wait() { (void)hipStreamSynchronize(st); } } wait{c->stream};
    // n rows from the caller's row r0 on, between buf (rows of C columns) and the state
    auto reorder = [&](float *state, float *buf, int r0, int n, bool host) -> sbqa_status {
        const int32_t *rows = c->pos ? c->pos + r0 : nullptr;
        if (!rows) state += state_off(c->order, c->ld, r0, 0);
        if (set) HIP_TRY(launch_state_reorder(n, C, ORDER_SPIN_MAJOR, C, buf, nullptr, c->order, c->ld, state, rows, host, c->stream));
        else HIP_TRY(launch_state_reorder(n, C, c->order, c->ld, state, rows, ORDER_SPIN_MAJOR, C, buf, nullptr, false, c->stream));
        return SBQA_OK;
    };
    if (set && 2 * row * N > STAGE_BYTES) {
        const int bulk = (int)std::min<size_t>(N, std::max<size_t>(1, BULK_BYTES / row));
        if (dev.get(row * bulk) == hipSuccess) {
            for (int q = 0; q < 2; ++q)
                for (int r0 = 0; r0 < N; r0 += bulk) {
                    const int n = std::min(bulk, N - r0);
                    HIP_TRY(hipMemcpyAsync(dev.as<float>(), (q ? y : x) + (size_t)r0 * C, row * n, hipMemcpyHostToDevice,
                                           c->stream));
                    const sbqa_status st = reorder(q ? c->y : c->x[c->cur], dev.as<float>(), r0, n, false);
                    if (st != SBQA_OK) return st;
                }
            const sbqa_status st = rebuild_operand(c);
            if (st != SBQA_OK) return st;
            HIP_TRY(hipStreamSynchronize(c->stream));
            return SBQA_OK;
        }
        (void)hipGetLastError();   // no room: like a small one
    }
    HIP_TRY(stage.get(2 * row * per));
    void *mapped = nullptr;
    HIP_TRY(hipHostGetDevicePointer(&mapped, stage.as<void>(), 0));
    struct Slab { float *user, *state; int r0, n; };
    std::vector<Slab> slabs;
    for (int q = 0; q < 2; ++q)
        for (int r0 = 0; (q ? y : x) && r0 < N; r0 += per)
            slabs.push_back({q ? y : x, q ? c->y : c->x[c->cur], r0, std::min(per, N - r0)});
    auto half = [&](void *base, size_t k) { return static_cast<float *>(base) + (k & 1) * (size_t)per * C; };
    auto move = [&](size_t k) {   // between the caller's array and the slab's half of the stage
        float *user = slabs[k].user + (size_t)slabs[k].r0 * C, *mine = half(stage.as<void>(), k);
        std::memcpy(set ? mine : user, set ? user : mine, row * slabs[k].n);
    };
    if (!whole) {   // (the error word before anything is handed out)
        const sbqa_status st = ctx_sync(c);
        if (st != SBQA_OK) return st;
    }
    for (size_t k = 0; k < slabs.size(); ++k) {
        if (set) move(k);
        const sbqa_status st = reorder(slabs[k].state, half(mapped, k), slabs[k].r0, slabs[k].n, true);
        if (st != SBQA_OK) return st;
        if (!whole) {   // the host copies one slab while the device works on the next
            if (k) move(k - 1);
            HIP_TRY(hipStreamSynchronize(c->stream));
        }
    }
    if (set) {
        const sbqa_status st = rebuild_operand(c);
        if (st != SBQA_OK) return st;
        HIP_TRY(hipStreamSynchronize(c->stream));
        return SBQA_OK;
    }
    if (whole) {
        const sbqa_status st = ctx_sync(c);
        if (st != SBQA_OK) return st;
    }
    for (size_t k = whole ? 0 : slabs.size() - std::min<size_t>(slabs.size(), 1); k < slabs.size(); ++k) move(k);
    return SBQA_OK;
}

}  // namespace sbqa

// =========================================================================== //
//                                 C ABI                                       //
// =========================================================================== //

extern "C" {

sbqa_schedule sbqa_schedule_default(void) {
    sbqa_schedule s;
    std::memset(&s, 0, sizeof s);
    s.steps = 1000;
    s.dt = 0.5;
    s.a0 = 1.0;
    s.c0 = 0.0;
    s.fmode = SBQA_F_TERNARY;
    s.delta_max = 0.7;
    s.jp_kind = SBQA_JP_PAPER;
    s.jp_start = 0.5;
    s.jp_end = 0.0;
    s.gamma0_over_R = 1.0;
    s.beta_lo = 0.5;
    s.beta_hi = 1.5;
    s.alpha_lo = 0.5;
    s.alpha_hi = 1.0;
    s.seed = 0;
    s.init_amp = 0.1;
    s.precision = SBQA_PREC_AUTO;
    s.energy_every = 0;
    s.loop_kernel = SBQA_LOOP_AUTO;
    s.dense_tile = 0;
    s.j_packing = SBQA_JPACK_AUTO;
    s.reorder = SBQA_REORDER_AUTO;
    return s;
}

const char *sbqa_last_error(void) { return last_error(); }

sbqa_status sbqa_create(const sbqa_coupling *J, const double *h, int32_t N, int32_t R, int32_t runs,
                        const sbqa_schedule *s, sbqa_ctx **out) {
    clear_error();
    if (!out) return fail(SBQA_EINVAL, "out must be non-NULL");
    *out = nullptr;
    InstanceFacts facts;
    sbqa_status st = guarded([&] { return validate_instance(J, h, N, R, runs, s, &facts); });
    if (st != SBQA_OK) return st;
    return ctx_create(J, h, N, R, runs, s, facts, nullptr, out, true);
}

sbqa_status sbqa_step(sbqa_ctx *c, uint32_t n) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    return ctx_step(c, n);
}

sbqa_status sbqa_best(sbqa_ctx *c, double *energies, int8_t *spins) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    return ctx_best(c, energies, spins);
}

sbqa_status sbqa_best_step(sbqa_ctx *c, int64_t *step_of_best) {
    clear_error();
    if (!c || !step_of_best) return fail(SBQA_EINVAL, "NULL argument");
    HIP_TRY(hipMemcpyAsync(step_of_best, c->bestStep, sizeof(int64_t) * c->runs, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return SBQA_OK;
}

static sbqa_status host_energies(sbqa_ctx *c, const int8_t *spins, int32_t count, double *out) {
    if (!c || (!spins && count) || (!out && count)) return fail(SBQA_EINVAL, "NULL argument");
    if (count < 0) return fail(SBQA_EINVAL, "count must be >= 0");
    if (count == 0) return SBQA_OK;
    const int N = c->N;
    const size_t total = (size_t)count * N;
    for (size_t q0 = 0; q0 < total; q0 += 4096) {
        const size_t q1 = std::min(total, q0 + 4096);
        int bad = 0;
        for (size_t q = q0; q < q1; ++q) bad |= (spins[q] != 1) & (spins[q] != -1);
        for (size_t q = q0; bad && q < q1; ++q)
            if (spins[q] != 1 && spins[q] != -1) return fail(SBQA_EINVAL, "spins must be +-1 (index %lld)", (long long)q);
    }
    // pooled buffers; every use of them is behind the synchronisations below
    // or, on a failure, behind the one that Wait makes
    PoolBlock ds(c->device, false), E(c->device, false), S(c->device, false), P(c->device, false);
    PoolBlock stage(c->device, true);
    struct Wait { hipStream_t st; ~Wait() { if (st) (void)hipStreamSynchronize(st); } } wait{c->stream};
    HIP_TRY(ds.get(total));
    HIP_TRY(E.get(sizeof(double) * count));
    // small inputs go up, and the energies come down, through pinned memory
    // (a copy from pageable memory waits for the runtime's own staging)
    const size_t espace = sizeof(double) * count;
    const bool pinned = total <= STAGE_BYTES && espace <= STAGE_BYTES;
    std::vector<int8_t> rows;
    int8_t *host = nullptr;
    if (pinned) {
        HIP_TRY(stage.get(std::max(total, espace)));
        host = stage.as<int8_t>();
    } else if (!c->pnew.empty()) {
        rows.resize(total);
        host = rows.data();
    }
    if (!c->pnew.empty()) {   // the caller's spin order to the internal rows
        for (int32_t m = 0; m < count; ++m)
            for (int i = 0; i < N; ++i) host[(size_t)m * N + c->pnew[(size_t)i]] = spins[(size_t)m * N + i];
    } else if (pinned) {
        std::memcpy(host, spins, total);
    }
    HIP_TRY(hipMemcpyAsync(ds.as<int8_t>(), host ? host : spins, total, hipMemcpyHostToDevice, c->stream));
    if (!pinned) HIP_TRY(hipStreamSynchronize(c->stream));
    if (c->facts.path != PATH_CSR) {
        const EnergyPlan e = energy_plan(N, count);
        HIP_TRY(S.get((size_t)e.cp * c->L.Np));
        HIP_TRY(P.get(sizeof(double) * e.units * e.cp));
    }
    sbqa_status st = ctx_energies_dev(c, ds.as<int8_t>(), count, E.as<double>(), S.as<int8_t>(), P.as<double>());
    if (st != SBQA_OK) return st;
    // (the spins in the stage have been read by then: same stream)
    HIP_TRY(hipMemcpyAsync(pinned ? stage.as<double>() : out, E.as<double>(), espace, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    wait.st = nullptr;
    if (pinned) std::memcpy(out, stage.as<double>(), espace);
    return SBQA_OK;
}

sbqa_status sbqa_energy(sbqa_ctx *c, const int8_t *spins, int32_t count, double *out) {
    clear_error();
    return guarded([&] { return host_energies(c, spins, count, out); });
}

static sbqa_status host_fields(sbqa_ctx *c, float *phi) {
    if (!c || !phi) return fail(SBQA_EINVAL, "NULL argument");
    const int N = c->N, C = c->L.C;
    std::vector<float> buf;
    if (c->facts.path == PATH_CSR) {
        const int Cs = c->L.Cs;
        const float *xs = c->x[c->cur];
        const int8_t *gs = (const int8_t *)c->g[c->cur];
        if (c->order == ORDER_COLBLOCK8) {
            // the fields kernel gathers spin-major rows: a spin-major copy of
            // the state and its operand, and the fields, in buffers allocated
            // at the first call on a resident context
            if (!c->phi) {
                int8_t *gsm0 = nullptr;
                HIP_TRY(dalloc(c, &c->x[1 - c->cur], (size_t)N * Cs));
                HIP_TRY(dalloc(c, &gsm0, (size_t)N * Cs));
                c->g[1 - c->cur] = gsm0;
                HIP_TRY(dalloc(c, &c->phi, (size_t)N * Cs));
            }
            float *xsm = c->x[1 - c->cur];
            int8_t *gsm = (int8_t *)c->g[1 - c->cur];
            HIP_TRY(launch_state_reorder(N, C, c->order, c->ld, xs, nullptr, ORDER_SPIN_MAJOR, Cs, xsm, nullptr, false, c->stream));
            if (c->s.fmode != SBQA_F_BALLISTIC)
                HIP_TRY(launch_csr_operand(c->s.fmode, N, Cs, C, xsm, gsm, delta_at(&c->s, c->step), c->stream));
            xs = xsm;
            gs = gsm;
        }
        HIP_TRY(launch_csr_fields(c->s.fmode, N, Cs, C, c->rp, c->col, c->val, c->tri3(), xs, gs, c->phi, c->stream));
        buf.resize((size_t)N * Cs);
        HIP_TRY(hipMemcpyAsync(buf.data(), c->phi, sizeof(float) * buf.size(), hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        for (int i = 0; i < N; ++i)
            std::memcpy(phi + (size_t)i * C, buf.data() + (size_t)(c->pnew.empty() ? i : c->pnew[(size_t)i]) * Cs,
                        sizeof(float) * C);
        return SBQA_OK;
    }
    const int Np = c->L.Np;
    PoolBlock dev(c->device, false);
    struct Wait { hipStream_t st; ~Wait() { if (st) (void)hipStreamSynchronize(st); } } wait{c->stream};
    HIP_TRY(dev.get(sizeof(float) * (size_t)C * Np));
    float *sum = dev.as<float>();
    if (c->g_stale) {
        const sbqa_status st = rebuild_operand(c);
        if (st != SBQA_OK) return st;
    }
    DenseStepArgs a = dense_args(c, c->step, c->cur);
    a.phi = sum;
    HIP_TRY(launch_dense_step(c->facts.path, EPI_FIELDS, c->L.form, c->L.mbw, c->L.Cg, a, c->stream));
    buf.resize((size_t)C * Np);
    HIP_TRY(hipMemcpyAsync(buf.data(), sum, sizeof(float) * buf.size(), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (int i = 0; i < N; ++i)
        for (int cc = 0; cc < C; ++cc) phi[(size_t)i * C + cc] = buf[(size_t)cc * Np + i];
    return SBQA_OK;
}

sbqa_status sbqa_fields(sbqa_ctx *c, float *phi) {
    clear_error();
    return guarded([&] { return host_fields(c, phi); });
}

sbqa_status sbqa_get_state(sbqa_ctx *c, float *x, float *y) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    return guarded([&] { return transfer_state(c, x, y, false); });
}

sbqa_status sbqa_set_state(sbqa_ctx *c, const float *x, const float *y) {
    clear_error();
    if (!c || !x || !y) return fail(SBQA_EINVAL, "NULL argument");
    const size_t one = (size_t)c->N * c->L.C;
    for (size_t q0 = 0; q0 < one; q0 += 4096) {
        const size_t q1 = std::min(one, q0 + 4096);
        int bad = 0;   // NaN and infinities fail the comparisons
        for (size_t q = q0; q < q1; ++q)
            bad |= !(std::fabs(x[q]) <= 1.0f) | !(std::fabs(y[q]) <= std::numeric_limits<float>::max());
        for (size_t q = q0; bad && q < q1; ++q)
            if (!std::isfinite(x[q]) || !std::isfinite(y[q]) || std::fabs(x[q]) > 1.0f)
                return fail(SBQA_EINVAL, "state must be finite with |x| <= 1 (index %zu)", q);
    }
    c->sbits_step = -1;
    // (transfer_state only reads what it is given in this direction)
    sbqa_status st = guarded([&] { return transfer_state(c, const_cast<float *>(x), const_cast<float *>(y), true); });
    if (st != SBQA_OK) return st;
    c->last_eval_step = -1;
    return SBQA_OK;
}

sbqa_status sbqa_run_params(sbqa_ctx *c, double *beta, double *alpha) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    if (beta) std::memcpy(beta, c->beta.data(), sizeof(double) * c->runs);
    if (alpha) std::memcpy(alpha, c->alpha.data(), sizeof(double) * c->runs);
    return SBQA_OK;
}

sbqa_status sbqa_jperp_table(sbqa_ctx *c, float *jp) {
    clear_error();
    if (!c || !jp) return fail(SBQA_EINVAL, "NULL argument");
    std::memcpy(jp, c->jp_host.data(), sizeof(float) * c->jp_host.size());
    return SBQA_OK;
}

sbqa_status sbqa_set_stream(sbqa_ctx *c, void *hip_stream) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    HIP_TRY(hipStreamSynchronize(c->stream));
    forget_launches(c);
    c->stream = hip_stream ? (hipStream_t)hip_stream : c->default_stream;
    if (!c->stream) return fail(SBQA_ESTATE, "context has no default stream");
    return SBQA_OK;
}

sbqa_status sbqa_info(sbqa_ctx *c, sbqa_info_t *info) {
    clear_error();
    if (!c || !info) return fail(SBQA_EINVAL, "NULL argument");
    info->N = c->N;
    info->R = c->R;
    info->runs = c->runs;
    info->steps = c->s.steps;
    info->step = c->step;
    info->path = c->facts.path;
    info->fmode = c->s.fmode;
    info->c0 = c->c0;
    info->j_integral = c->facts.integral ? 1 : 0;
    info->device_bytes = c->bytes;
    info->resident = c->resident ? 1 : 0;
    info->tile_cols = c->facts.path == PATH_CSR ? 0 : 64 * c->L.mbw;
    info->reordered = c->pnew.empty() ? 0 : 1;
    return SBQA_OK;
}

sbqa_status sbqa_sync(sbqa_ctx *c) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    return ctx_sync(c);
}

sbqa_status sbqa_inject_wait_timeout(sbqa_ctx *c) {
    clear_error();
    if (!c) return fail(SBQA_EINVAL, "NULL context");
    if (!c->exchanging.workgroups || !c->err)
        return fail(SBQA_EINVAL, "the context runs no loop whose workgroups wait for each other");
    static const int timed_out = 1;   // the value a timed-out wait stores
    HIP_TRY(hipMemcpyAsync(c->err, &timed_out, sizeof(int), hipMemcpyHostToDevice, c->stream));
    return SBQA_OK;
}

void sbqa_destroy(sbqa_ctx *c) {
    if (!c) return;
    delete c;   // waits for the context's work
}

void sbqa_release_cached(void) { pool_trim(); }

}  // extern "C"
