// The order of launches whose workgroups wait for each other (launch_order.h)
// against a model of a device: streams run their launches in order, a launch
// starts once what its stream waits for has ended, running launches end in any
// order. Launches that run together must fit: a CU per workgroup, or as many as fit
// on one where all are of one kind. Prints "order checks passed".
#include "../../paper_2604_01050_amd/csrc/launch_order.h"

#include <cstdio>
#include <random>
#include <vector>

using sbqa::Exchanging;

struct Launch {
    int stream;
    Exchanging need;
    std::vector<int> after;   // launches that end first
    bool started = false, ended = false;
};

static int run(unsigned seed) {
    std::mt19937 g(seed);
    const int cus = 256, streams = 2 + (int)(g() % 5);
    const int per_cu[3] = {1, 2, 4};
    sbqa::LaunchOrder<int> order;
    std::vector<Launch> all;
    std::vector<int> last(streams, -1);
    int waits = 0;
    auto settle = [&](bool everything) {   // lets launches start and end, checks what runs together
        for (int turn = 0;; ++turn) {
            std::vector<int> running;
            for (size_t k = 0; k < all.size(); ++k) {
                Launch &l = all[k];
                bool ready = !l.started;
                for (int a : l.after) ready = ready && all[a].ended;
                if (ready) l.started = true;
                if (l.started && !l.ended) running.push_back((int)k);
            }
            int sum = 0;
            bool same = true;
            for (int k : running) {
                sum += all[k].need.workgroups;
                same = same && all[k].need.kind == all[running[0]].need.kind;
            }
            if (!running.empty() && sum > cus * (same ? all[running[0]].need.per_cu : 1)) {
                std::printf("seed %u: %d workgroups in flight together\n", seed, sum);
                return false;
            }
            if (running.empty()) return true;
            if (!everything && g() % 3 == 0) return true;
            all[running[g() % running.size()]].ended = true;
        }
    };
    for (int n = 0; n < 60; ++n) {
        Launch l;
        l.stream = (int)(g() % streams);
        const int k = (int)(g() % 3);
        l.need.kind = (uint64_t)k + 1;
        l.need.per_cu = per_cu[k];
        l.need.workgroups = 1 + (int)(g() % (cus * per_cu[k]));
        if (g() % 2) l.need.workgroups = 1 + l.need.workgroups / 8;
        if (last[l.stream] >= 0) l.after.push_back(last[l.stream]);
        order.before(&last[l.stream], l.stream, l.need, cus, [&](int t) {
            ++waits;
            if (last[t] >= 0) l.after.push_back(last[t]);
        });
        last[l.stream] = (int)all.size();
        all.push_back(l);
        if (!settle(false)) return 1;
        if (g() % 16 == 0) {   // a context goes: its stream has been waited for
            if (!settle(true)) return 1;
            order.forget(&last[l.stream]);
        }
    }
    return settle(true) ? 0 : 1;
}

int main() {
    for (unsigned seed = 0; seed < 3000; ++seed)
        if (run(seed)) return 1;
    // launches of one shape that fit together, and a lone stream, wait for nobody
    sbqa::LaunchOrder<int> order;
    int waits = 0;
    auto count = [&](int) { ++waits; };
    const Exchanging quarter{128, 1, 2}, whole{256, 2, 1};
    for (int n = 0; n < 20; ++n) order.before(&order, n % 4, quarter, 256, count);
    if (waits) return std::printf("launches that fit waited\n"), 1;
    order.before(&order, 0, whole, 256, count);
    if (waits != 3) return std::printf("%d waits for three streams\n", waits), 1;
    for (int n = 0; n < 20; ++n) order.before(&order, 0, whole, 256, count);
    if (waits != 3) return std::printf("a lone stream waited\n"), 1;
    std::printf("order checks passed\n");
    return 0;
}
