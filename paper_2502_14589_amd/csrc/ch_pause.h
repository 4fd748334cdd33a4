// When a context tries resident launches again after a wait of one ran out.
// Host arithmetic only.
#pragma once

#include <algorithm>

// An expired wait costs its bound and says that the launch's workgroups did not fit
// beside what else runs on the device (another process, say), which the next call
// would meet again.  Ordinary launches therefore follow for 32 times that cost, twice as
// long after each further expiry, so that at most about 3% of a context's time goes
// into waits that run out; a call whose resident launches all passed starts over.
struct ResidentPause {
    static constexpr double COST_MIN_S = 0.01, FACTOR = 32.0;
    static constexpr int LEVELS = 10;
    double until = 0.0;
    int level = 0;

    bool over(double now) const { return now >= until; }
    void expired(double now, double wait_s) {
        until = now + FACTOR * std::max(wait_s, COST_MIN_S) * double(1 << level);
        level = std::min(level + 1, LEVELS);
    }
    void passed() { level = 0; }
};
