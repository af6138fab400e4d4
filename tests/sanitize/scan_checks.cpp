// Host-side checks of the validation of dense couplings and of the schedule
// table, the parts that run on several threads, under host sanitizers (built like
// host_checks.cpp): +-1 matrices and mutated ones in exactly sized buffers, their
// sign bits, and the table of Eq. 5 against its formula. Prints "scan checks passed".
#include "../../paper_2604_01050_amd/csrc/sbqa_api.cpp"

#include <cstdio>
#include <random>

static int g_fail = 0;
#define CHECK(cond)                                                                   \
    do {                                                                              \
        if (!(cond)) {                                                                \
            std::fprintf(stderr, "CHECK failed, line %d: %s\n", __LINE__, #cond);     \
            ++g_fail;                                                                 \
        }                                                                             \
    } while (0)

static void check_scan(std::mt19937_64 &g, int32_t N) {
    std::vector<double> A((size_t)N * N, 0.0);
    for (int32_t i = 0; i < N; ++i)
        for (int32_t j = i + 1; j < N; ++j) A[(size_t)i * N + j] = A[(size_t)j * N + i] = g() & 1 ? 1.0 : -1.0;
    for (int32_t i = 0; i < N; i += 3) A[(size_t)i * N + i] = -0.0;
    sbqa_schedule s = sbqa_schedule_default();
    s.steps = 10;
    sbqa_coupling J{};
    J.dense = A.data();
    InstanceFacts f;
    std::vector<uint32_t> bits;
    CHECK(validate_instance(&J, nullptr, N, 2, 2, &s, &f, &bits) == SBQA_OK);
    CHECK(f.pm1 == (N > 1) && f.ternary && f.int8 && f.integral);
    if (N > 1) {
        const int64_t words = (N + 31) / 32;
        CHECK((int64_t)bits.size() == N * words);
        for (int32_t i = 0; i < N; ++i)
            for (int32_t j = 0; j < 32 * words; ++j) {
                const bool want = j < N && A[(size_t)i * N + j] < 0.0;
                if ((((bits[(size_t)(i * words + j / 32)] >> (j % 32)) & 1u) != 0u) != want) ++g_fail;
            }
    }
    if (N < 3) return;
    for (int q = 0; q < 6; ++q) {
        const size_t i = g() % N, j = (i + 1 + g() % (N - 1)) % N, at = i * N + j;
        const double keep = A[at], bad[6] = {-keep, 0.0, 2.0, 0.5, std::numeric_limits<double>::quiet_NaN(),
                                             std::numeric_limits<double>::infinity()};
        A[at] = bad[q];
        CHECK(validate_instance(&J, nullptr, N, 2, 2, &s, &f, &bits) == SBQA_EINVAL);
        if (q >= 1 && q <= 3) {   // symmetric again: valid, and no +-1 matrix
            A[j * N + i] = bad[q];
            InstanceFacts f2;
            CHECK(validate_instance(&J, nullptr, N, 2, 2, &s, &f2, &bits) == SBQA_OK);
            CHECK(!f2.pm1 && f2.ternary == (q == 1) && f2.int8 == (q != 3));
            A[j * N + i] = keep;
        }
        A[at] = keep;
    }
}

static void check_table(int32_t runs, uint32_t steps) {
    sbqa_schedule s = sbqa_schedule_default();
    s.steps = steps;
    s.seed = 77;
    std::vector<double> beta, alpha;
    std::vector<float> jp;
    build_schedule_host(&s, runs, beta, alpha, jp);
    CHECK(jp.size() == (size_t)runs * steps);
    for (int32_t r = 0; r < runs; ++r)
        for (uint32_t n = 0; n < steps; ++n) {
            const double gx = s.gamma0_over_R * (std::pow(1.0 - (double)n / steps, alpha[r]) + 1e-5);
            if (jp[(size_t)r * steps + n] != (float)(-std::log(std::tanh(beta[r] * gx)) / (2.0 * beta[r]))) ++g_fail;
        }
}

int main() {
    std::mt19937_64 g(5);
    for (int32_t N : {1, 2, 3, 31, 32, 33, 63, 64, 65, 128, 200, 700}) check_scan(g, N);
    for (int32_t runs : {1, 7, 64})
        for (uint32_t steps : {1u, 1023u, 1024u, 1025u, 4000u}) check_table(runs, steps);
    if (g_fail) return std::fprintf(stderr, "%d checks failed\n", g_fail), 1;
    std::printf("scan checks passed\n");
    return 0;
}
