// The CUs that resident launches of this process hold.  Host code only.
#pragma once

#include <atomic>

// CUs of each device held by resident launches (ch_resident.h) of this
// process.  A call that issues such launches holds a lease on one CU per
// workgroup until its stream has drained, so the workgroups of all leases on a
// device fit it together and no launch waits for workgroups that cannot
// start; a call that gets no lease issues ordinary launches (same results).
// A launch's workgroups go to the eight XCDs in turn from the first on, and each XCD has an
// eighth of the CUs: whole rounds are leased (three launches of 81 would need 33 of the
// 32 CUs of an XCD).
class ResidentLease {
    static constexpr int DEVICES = 64, XCDS = 8;
    static inline std::atomic<int> used[DEVICES];
    std::atomic<int>* u = nullptr;
    int n = 0;

public:
    static constexpr int rounded(int count) { return (count + XCDS - 1) / XCDS * XCDS; }
    ResidentLease() = default;
    ResidentLease(const ResidentLease&) = delete;
    ResidentLease& operator=(const ResidentLease&) = delete;
    ~ResidentLease() { release(); }
    bool take(int device, int cus, int count) {
        release();
        if (device < 0 || device >= DEVICES || count < 1) return false;
        count = rounded(count);
        if (used[device].fetch_add(count) + count > cus) {
            used[device].fetch_sub(count);
            return false;
        }
        u = &used[device];
        n = count;
        return true;
    }
    void release() {
        if (u) u->fetch_sub(n);
        u = nullptr;
    }
};
