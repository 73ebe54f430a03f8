// Host-side internals shared by the solver runtime and the serving loop
// (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <map>
#include <string>
#include <tuple>
#include <utility>
#include <vector>

#include "pdd.h"
#include "pdd_internal.hpp"

namespace pdd {

// Records a thread-local message for pdd_last_error() and returns `code`.
pdd_status fail(pdd_status code, const char *fmt, ...);
extern thread_local std::string g_error;

#define HIP_TRY(expr)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return ::pdd::fail(PDD_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));   \
    } while (0)

constexpr double kGmShift = 0.5826;                    // Alg. 1 boundary shift
constexpr double kBridgeSkip = 24.953298500158186;     // 36 ln 2: p < 2^-36 skipped
constexpr uint64_t kDefaultMaxSteps = 1ull << 26;
constexpr uint64_t kScratchSlots = 1ull << 27;         // record slots per launch
constexpr uint64_t kMaxLaunchSlots = 1ull << 31;
constexpr double kFp64TrigRevolutions = 1 << 25;       // arguments that the FP64 walks reduce themselves (a margin of 8 to 2^31)
constexpr double kHwTrigRevolutions = 256.0;           // input range of the FP32 hardware sine / cosine

struct DeviceBuffer {
    void *ptr = nullptr;
    size_t cap = 0;
};

// One solve (or batch item) after validation.
struct HostItem {
    pdd_problem *prob = nullptr;
    const pdd_grid *u_prev = nullptr, *resid = nullptr;
    const pdd_grid *grad = nullptr;  // dim gradient grids (Ito control variate)
    const double *nodes = nullptr;
    int64_t n_nodes = 0;
    const pdd_solve_opts *o = nullptr;
    pdd_node_stats *out = nullptr;
    int est = kEstPlain;  // kEstPlain, kEstCorrection or kEstIto
    bool score_plain = true, uniform = true, caller_records = false, accumulate = false;
    uint64_t total = 0, max_steps = 0;
    std::vector<uint64_t> starts;  // item-relative prefix (non-uniform counts)
};

// Largest |k_d x_d + phase_d| / (2 pi) of the problem's trig terms over the box
// [lo, hi].
double trig_revolutions(const pdd_problem_desc &d, const double *lo, const double *hi);
// Checks an item's arguments against its problem (nothing is enqueued).
pdd_status validate_item(HostItem &it);
// Key of the launch-shape table: precision, dimension, estimator (kEst*) and
// kernel (specialised box / bridge / Gaussian / analytic, or generic).
inline int tuning_key(int precision, int dim, int est, bool generic)
{
    return precision * 12 + (dim - 2) * 6 + est * 2 + (generic ? 1 : 0);
}
// Whether an item can run in the specialised kernel.
bool specialised(const HostItem &it);
// The launch's refill mask: walk-loop iterations between lane refills, less
// one (the tuning's, else every second iteration in 2D, every fourth in 3D).
template <int D>
inline uint32_t refill_mask(const pdd_tuning &t)
{
    return (uint32_t)((t.refill ? t.refill : (D == 2 ? 2 : 4)) - 1);
}
// Launches of at most this many paths are walked by groups of lanes only: up
// to about one and a half paths per resident lane, one path per lane leaves
// most lanes idle for most of the launch. Measured, group walk against one
// path per lane and a hand-over (18 nodes, h = 1e-3): 180,000 paths 0.44 and
// 0.54 ms in FP32 2D, 0.65 and 0.82 ms in FP64; 360,000: 0.62 and 0.78, 1.06
// and 1.09; 540,000: 0.81 and 0.86, 1.44 and 1.32. A step of FP64 walks with a
// tabulated drift is mostly the gather of it, which the group walk does twice
// (phases 2 and 3): 20 nodes of the paper's example on 513^2 grids 2.4 and 2.5 ms at
// 60,000 paths, 3.3 and 3.0 at 100,000, 9.3 and 5.0 at 399,000; on 129^2 1.9 and
// 2.0, 2.6 and 2.4, 7.3 and 4.2; 3D on 33^3 2.6 and 2.7, 3.5 and 3.1, 9.7 and 4.6.
// Without a buffer for the hand-over (pdd_solve_nodes_noalloc) the lines cross
// later: 513^2 5.7 and 5.1 ms at 220,000, 4.3 and 4.6 at 150,000; 3D 3.5 and 3.3
// at 100,000.
constexpr uint64_t kGroupDirectSlots = 400000;
inline uint64_t group_direct_slots(bool fp64, bool tabulated_drift, bool hand_over, int dim)
{
    if (!fp64 || !tabulated_drift) return kGroupDirectSlots;
    return hand_over ? 65536 : dim == 2 ? 200000 : 100000;
}
// Paths handed over by a launch, at most (their buffer: 33 MB in FP32 3D). The
// items of a batch share it: 64 uneven problems take 140 ms with it and 180 ms
// with half of it, no less with twice of it.
constexpr uint64_t kTailEntries = 1ull << 19;
// Workgroups of a group-walk launch over at most `paths` paths: as many lanes
// per path as two workgroups per CU give (FP32 from 2^17 paths on three: 0.62
// ms for 360,000 paths, 0.69 ms with two; 18,000 paths 0.22 and 0.21 ms).
template <class T>
int group_grid(const pdd_ctx *ctx, uint64_t paths);
// Paths a wave takes from the queue at a time: the tuning's, but not so many
// that waves run dry at very different times (about eight tickets a wave; 18
// nodes x 100,000 correction paths with the tuned 256: 1.94 ms, 1.79 ms), and
// not below 32, where the waves wait for the one counter (2.2 ms with 16).
inline int32_t ticket_size(const pdd_tuning &t, uint64_t paths, uint64_t waves)
{
    const uint64_t even = paths / (waves * 8) / 16 * 16;
    return (int32_t)std::min<uint64_t>((uint64_t)t.grab, std::max<uint64_t>(32, even));
}
// Whether many lanes of a wave are near a face at every step of a walk of
// this problem at step dt (then the dense form of the bridge test is the
// faster one).
bool dense_boundary(const pdd_problem_desc &d, double dt);

// Launch shape for a solve: opts->tuning (fields left 0 take the default),
// else the context's table entry for `key` (tuning_key; < 0: none), else
// {256, occupancy, 64, 0}; checked.
pdd_status read_tuning(const pdd_ctx *ctx, const pdd_solve_opts *o, int key, pdd_tuning &tune);
// Resident workgroups per CU of kernel `fn` at `block` threads, from the
// context's table (filled at pdd_init for the plain kernels; `cache`: add a
// missing entry, which allocates host memory).
int occupancy(pdd_ctx *ctx, const void *fn, int block, bool cache = true);
// The allocation-free solve's device scratch on `device` (made current by the
// caller): looked up once per device; PDD_E_HIP if the lookup fails.
pdd_status noalloc_attach(int device);

// Validates items, then enqueues them on `s`, grouped by (precision,
// dimension, estimator); a group of at most kScratchSlots paths without
// caller records is one launch. one_launch: such a group stays one launch
// whatever the tuning's max_launch_paths says (the serving loop, whose
// results must not depend on the tuning table). The items' problems must
// belong to `owner` (NULL: ctx itself), a context on ctx's device whose
// problems ctx's scratch then serves.
pdd_status run_items(pdd_ctx *ctx, std::vector<HostItem> &items, hipStream_t s, bool one_launch = false,
                     const pdd_ctx *owner = nullptr);

}  // namespace pdd

struct pdd_ctx {
    int device = 0;
    int n_cu = 0;
    hipEvent_t done = nullptr;    // end of the last solve
    hipEvent_t staged = nullptr;  // last copy out of the staging buffer
    bool any_done = false, any_staged = false;
    pdd::DeviceBuffer nodes, starts, acc, rec, partials, gather, cells;
    pdd::DeviceBuffer tail;    // walking paths handed over between path kernels of a launch
    pdd::DeviceBuffer stage2;  // second stage: tables and stencils
    // factors of the last second stage's subdomain matrices, what they factor
    // (the operator, the grid, the interfaces) and how (blocks of the cyclic
    // reduction, or LU), and whether the cyclic reduction is for these matrices:
    // a call with the same ones only solves for its right sides
    pdd::DeviceBuffer stage2_factor;
    std::vector<double> stage2_key;
    bool stage2_blocks = false, stage2_dominant = false;
    bool stage2_refused = false;  // no memory for more than LU factors
    // with LU factors, the subdomains' response columns to their boundary values
    // (and to f), for the key and the problem
    pdd::DeviceBuffer stage2_resp;
    std::vector<double> stage2_resp_key;
    void *stage = nullptr;
    size_t stage_cap = 0;
    void *readback = nullptr;  // pinned host copy of pilot statistics
    size_t readback_cap = 0;
    std::map<std::tuple<const void *, int>, int> occupancy;
    // timing of path-kernel launches (PDD_TIME_KERNEL)
    std::vector<std::pair<hipEvent_t, hipEvent_t>> timed, spare;
    // launch shapes by (precision, dim, estimator), from pdd_autotune / pdd_set_tuning
    std::map<int, pdd_tuning> tuned;
};

namespace pdd {
template <class T>
int group_grid(const pdd_ctx *ctx, uint64_t paths)
{
    constexpr uint64_t waves = kGroupBlock / 64;
    const uint64_t most = (uint64_t)ctx->n_cu * (sizeof(T) == 4 && paths >= (1u << 17) ? 3 : 2);
    uint64_t share = 1;  // paths of a wave
    while (share < 16 && paths > share * most * waves) share *= 2;
    return (int)std::max<uint64_t>(1, std::min(most, (paths + share * waves - 1) / (share * waves)));
}
}  // namespace pdd

struct pdd_problem {
    pdd_ctx *ctx = nullptr;
    pdd_problem_desc desc{};
    // largest |k_d x_d + phase_d| of a trig term over the domain's bounding
    // box, in revolutions: FP32 paths evaluate sines with the hardware
    // instruction, whose argument must stay within +-256 revolutions
    double trig_rev_max = 0.0;
    pdd::DevProblem<float> pf{};
    pdd::DevProblem<double> pd{};
    pdd::DeviceBuffer tab;  // cell layouts of tabulated coefficients (FP32, then FP64)
    uint64_t serial = 0;    // unique per problem created in the process
};
