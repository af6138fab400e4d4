// Order of the launches whose workgroups wait for each other (the resident sparse
// loops, the many-step dense loop with several workgroups per group). Such a launch
// ends only if all its workgroups get onto the device: two of them on different
// streams, each holding the CUs that the other's last workgroups need, would
// wait until their bounded polls give up. So launches may be in flight together
// only while every workgroup of theirs has a place whatever the order they are
// handed out in:
//   * a CU each, or
//   * where all are launches of one kernel with one shape, as many as fit on a CU.
// Otherwise the new launch's stream first waits for the other streams. Kernels that
// wait for nobody need no part in this: they end by themselves.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <map>
#include <set>

namespace sbqa {

struct Exchanging {
    int workgroups = 0;
    uint64_t kind = 0;   // the kernel and its launch shape; 0: several
    int per_cu = 1;      // workgroups of it that fit on a CU
};

// The streams of one device that may have such launches in flight. Not
// thread-safe: the caller holds a lock from before() until the launch is issued.
template <class Stream>
class LaunchOrder {
  public:
    // Before a launch on stream s by `owner` (a context): wait(t) is called for each
    // other stream t that s has to wait for, up to its present end.
    template <class Wait>
    void before(const void *owner, Stream s, const Exchanging &launch, int cus, Wait &&wait) {
        Exchanging others;
        bool alone = true;
        for (auto &kv : flight_) {
            if (kv.first == s) continue;
            others = alone ? kv.second.most : both(others, kv.second.most);
            alone = false;
        }
        Entry &mine = flight_[s];
        mine.owners.insert(owner);
        if (!alone && !fits(both(others, launch), cus)) {
            for (auto it = flight_.begin(); it != flight_.end();) {
                if (it->first == s) {
                    ++it;
                    continue;
                }
                wait(it->first);
                it = flight_.erase(it);
            }
            // what s now holds back is still running, beside earlier launches of s
            mine.most = mine.most.workgroups ? both(mine.most, others) : others;
        }
        mine.most = mine.most.workgroups ? larger(mine.most, launch) : launch;
    }

    // The owner's launches have ended, its stream may be gone.
    void forget(const void *owner) {
        for (auto it = flight_.begin(); it != flight_.end();) {
            it->second.owners.erase(owner);
            if (it->second.owners.empty()) it = flight_.erase(it);
            else ++it;
        }
    }

  private:
    struct Entry {
        std::set<const void *> owners;
        Exchanging most;   // an upper bound of what is in flight at a time
    };
    static bool fits(const Exchanging &e, int cus) { return e.workgroups <= cus * (e.kind ? e.per_cu : 1); }
    static Exchanging merged(const Exchanging &a, const Exchanging &b, int workgroups) {
        Exchanging e;
        e.workgroups = workgroups;
        if (a.kind && a.kind == b.kind && a.per_cu == b.per_cu) {
            e.kind = a.kind;
            e.per_cu = a.per_cu;
        }
        return e;
    }
    static Exchanging both(const Exchanging &a, const Exchanging &b) { return merged(a, b, a.workgroups + b.workgroups); }
    static Exchanging larger(const Exchanging &a, const Exchanging &b) {
        return merged(a, b, std::max(a.workgroups, b.workgroups));
    }
    std::map<Stream, Entry> flight_;
};

}  // namespace sbqa
