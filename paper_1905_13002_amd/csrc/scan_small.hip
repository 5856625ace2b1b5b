// scan_small.hip -- dispatch of the small-state (nx <= 4) scans to the
// per-dimension, per-precision kernel instantiations.
#include <algorithm>

#include "pks_internal.h"

namespace pks {

template <int N, typename R>
hipError_t small_run(ScanArgs a, int passes, hipStream_t s);

namespace {

template <typename R>
hipError_t dispatch_n(ScanArgs a, int passes, hipStream_t s) {
    switch (a.nx) {
        case 1: return small_run<1, R>(a, passes, s);
        case 2: return small_run<2, R>(a, passes, s);
        case 3: return small_run<3, R>(a, passes, s);
        case 4: return small_run<4, R>(a, passes, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool small_supported(int nx) { return nx >= 1 && nx <= 4; }

// Defaults measured on MI355X (constant-velocity model, T = 2^20): FP64 is
// fastest with 16 steps per thread, the mixed mode with 8, both with a single
// scan level under the device-wide top level (which folds ceil(waves / 1024)
// aggregates per element).  Beyond 16384 waves (E > 16 sequential folds at the
// top) a second level of one aggregate per thread is inserted.
// pks_autotune overrides these per problem shape.
//
// Short sequences of nx = 3, 4: the folds of a thread are a chain of combines
// (2 to 3 us each), and the threads that would shorten it are idle.  CV model,
// filter + smoother, us, with 4, 2 and 1 steps a thread: T = 1000 FP64 82, 74,
// 68, mixed 74, 68, 59; T = 32768 105, 92, 89 and 92, 80, 78; T = 65536 111,
// 102, 108; time-varying T = 1000 139, 102, 83, T = 65536 197, 156, 151, T =
// 131072 231, 217, 237.  nx = 3: T = 32768 78, 72, 71; T = 65536 82, 78, 88; T
// = 98000 87, 89.  nx <= 2: no gain (37, 36, 35 at T = 1000), 53, 54, 56 at 32000.
constexpr int64_t kOneStep = 1 << 15;                              // up to here one step a thread
int64_t two_steps(int nx) { return nx == 4 ? 1 << 17 : 1 << 16; }  // and two up to here

// Threads that the configurations above and 4 steps a thread need, for `total`
// steps or fewer: it must not fall as the total grows (a workspace sized for one
// length serves every shorter one).
int64_t small_threads(int nx, int64_t total) {
    const int64_t four = (total + 3) / 4;
    if (nx < 3 || nx > 4) return four;
    return std::max(four, std::max(std::min(total, kOneStep), std::min((total + 1) / 2, two_steps(nx) / 2)));
}

TileConfig small_default_config(int nx, int64_t total, bool mixed) {
    TileConfig c;
    // the longest per-thread fold that still gives every SIMD (1024 on the
    // chip) a wave; shorter sequences take the shortest fold (more threads,
    // a shorter dependent chain per thread)
    const int64_t simds = 1024;
    const int emax = mixed ? 8 : 16;
    c.ept = 4;
    for (int e = emax; e > 4; e >>= 1)
        if (total >= (int64_t)64 * e * simds) {
            c.ept = e;
            break;
        }
    if (nx == 3 || nx == 4) c.ept = total <= kOneStep ? 1 : (total <= two_steps(nx) ? 2 : c.ept);
    const int64_t waves = (total + 64 * c.ept - 1) / (64 * c.ept);
    c.ept1 = waves > 16 * 1024 ? 1 : 0;
    return c;
}

hipError_t launch_small(ScanArgs a, bool mixed, int passes, hipStream_t s) {
    return mixed ? dispatch_n<float>(a, passes, s) : dispatch_n<double>(a, passes, s);
}

}  // namespace pks
