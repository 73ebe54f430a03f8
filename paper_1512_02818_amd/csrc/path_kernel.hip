// Path kernel of the first-stage PDD nodal solve on gfx950.
//
// One path per lane. A persistent wavefront takes paths from a global queue
// (one atomic per `grab` paths) and refills a lane as soon as its path has
// ended, so waves stay full whatever the spread of exit times. Each path is
// the Euler-Maruyama walk of Alg. 1 (eq. F:E_M, coefficients at the left
// point) with the bridge, shifted-boundary or naive exit test, carrying the
// killing weight Y, the source integral Z and, for the correction estimator,
// the residual integral R (Sec. 2.3; eq. F:Dynkin). Every path writes its
// score and exit step to its own slot; the per-node sums are formed afterwards
// in a fixed order, so results do not depend on scheduling.
#include "path_walk.hpp"

namespace pdd {
namespace {

// Cell layout of grids (see cell_values), values converted from S to T: one
// thread per cell and grid (blockIdx.y).
template <class S>
struct CellGrids {
    const S *data[3];
};
template <class S, class T, int D, class I>
__device__ __forceinline__ void grid_cells(const S *__restrict__ data, I n0, I n1, I n2, T *__restrict__ cells,
                                           uint32_t stride, uint32_t off)
{
    const I m0 = n0 - 1, m1 = n1 - 1, n_cells = m0 * m1 * (D == 3 ? n2 - 1 : 1);
    for (I c = blockIdx.x * (I)blockDim.x + threadIdx.x; c < n_cells; c += (I)gridDim.x * blockDim.x) {
        const I i = c % m0, jk = c / m0, j = D == 3 ? jk % m1 : jk, k = D == 3 ? jk / m1 : 0;
        T *out = cells + (uint64_t)c * stride + off;
#pragma unroll
        for (int dz = 0; dz < (D == 3 ? 2 : 1); ++dz)
#pragma unroll
            for (int dy = 0; dy < 2; ++dy)
#pragma unroll
                for (int dx = 0; dx < 2; ++dx) out[(dz * 2 + dy) * 2 + dx] = (T)data[((k + dz) * n1 + (j + dy)) * n0 + i + dx];
    }
}
template <class S, class T, int D>
__global__ void grid_cells_kernel(const CellGrids<S> g, int n0, int n1, int n2, T *__restrict__ cells,
                                  uint32_t stride, uint32_t off)
{
    const S *data = g.data[blockIdx.y];
    off += blockIdx.y << D;
    // (2^30 points: a thread's next cell still fits in 32 bits)
    if ((uint64_t)n0 * n1 * n2 < (1ull << 30))
        grid_cells<S, T, D, uint32_t>(data, n0, n1, n2, cells, stride, off);
    else
        grid_cells<S, T, D, uint64_t>(data, n0, n1, n2, cells, stride, off);
}

// Point values of a grid converted from S to T into every stride-th slot (a
// field of interleaved records): one thread per point.
template <class S, class T>
__global__ void grid_points_kernel(const S *__restrict__ data, uint64_t n_points, T *__restrict__ out,
                                   uint32_t stride, uint32_t off)
{
    for (uint64_t p = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; p < n_points;
         p += (uint64_t)gridDim.x * blockDim.x)
        out[p * stride + off] = (T)data[p];
}

// Lanes end paths at any step but take new ones only every few iterations of
// the walk loop (two steps per iteration in 2D, one in 3D; the launch's
// refill_mask, by default every second iteration in 2D and every fourth in
// 3D): every path of a wave then starts at a step count that is the same
// modulo 4 across its lanes, so the bridge uniforms of four consecutive steps
// share one Philox block, which the wave then draws at most once per four
// steps, and the scoring and start of new paths run for several lanes at once.

// Queue of the single-item kernel: a wave takes `grab` slots at a time from
// the launch counter, [next, end) launch-relative, and hands them to its idle
// lanes in order.
struct Pool {
    uint32_t next = 0, end = 0;
    bool exhausted = false;

    __device__ __forceinline__ void refill(const LaunchArgs &L, int lane)
    {
        if (next == end && !exhausted) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(L.counter, (uint32_t)L.grab);
            base = __builtin_amdgcn_readfirstlane(base);
            if (base >= L.launch_slots) {
                exhausted = true;
            } else {
                next = base;
                end = min(base + (uint32_t)L.grab, L.launch_slots);
            }
        }
    }
};

// Hands the wave's walking lanes on to the group-walk kernel, once at most
// L.tail_max are left and its item (item_lo + q of the launch) has no more
// slots: their states go to the item's region of L.tail. Returns false once
// that region is full (the lanes that found no room walk on here).
template <class T, int D, class W>
__device__ __forceinline__ bool hand_over_live(const LaunchArgs &L, uint32_t q, int lane, uint64_t below,
                                               uint32_t stream_tag, const W &w, int &st)
{
    const uint64_t live = __ballot(st == 1);
    const uint32_t n = (uint32_t)__popcll(live);
    if (n == 0 || n > L.tail_max) return true;
    const uint32_t off = L.tail_off[q], cap = L.tail_off[q + 1] - off;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(L.tail_n + q, n);
    at = __builtin_amdgcn_readfirstlane(at);
    if (st == 1) {
        const uint32_t i = at + (uint32_t)__popcll(live & below);
        if (i < cap) {
            w.hand_over(static_cast<TailState<T, D> *>(L.tail)[off + i], stream_tag);
            st = 0;
        }
    }
    return at + n <= cap;
}

// The single-item kernel scores ended paths from the wave's ring, as the
// batch kernel does, in its dense bridge form (boundary-dense, short walks)
// and its generic form; in the sparse form, for long walks whose lanes seldom
// end at the same turn, each path is scored as it ends (the ring's
// bookkeeping cost the [0,4]^2 launch 2.7 %).
template <class M>
constexpr bool kRingScoreOne = !std::is_same<M, BoxBridgeGaussT<false>>::value;

// Dynamic LDS of a wave of the single-item kernel: the ring of ended paths,
// and in the generic form (the one that walks tabulated problems) the block
// for gathering pair records.
template <class T, int D, class M>
struct OneWaveLds {
    EndRing<T, D> ring;
    Vec4<T> tr[std::is_same<M, RuntimeMode>::value ? 4 * 64 : 1];
};

// One item, passed by value (FP32 2D plain solves). The source polynomial's
// coefficients are staged through LDS once per workgroup: read from there,
// they stay in vector registers for the whole loop (about 96 registers, five
// waves per SIMD) instead of being reloaded by scalar loads at every step,
// which the scalar register file cannot hold next to the other constants.
template <class M>
constexpr int kOneMinWaves = std::is_same<M, RuntimeMode>::value ? 1 : 5;
template <class T, int D, int EST, class M>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kOneMinWaves<M>, 8)))
    path_kernel_one(const OneItemArgs<T> A)
{
    static_assert(kOneItemKernel<T, D, EST>, "single-item kernel is for FP32 2D plain solves");
    const LaunchArgs &L = A.launch;
    const ItemCore<T> &a = A.item;
    const DevProblem<T> &P = A.prob;
    const int lane = __lane_id();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    __shared__ T s_cf[kMaxDense];
    extern __shared__ __attribute__((aligned(16))) uint64_t s_one[];  // dynamic: OneWaveLds per wave (ring-scoring forms)
    for (uint32_t i = threadIdx.x; i < (uint32_t)kMaxDense; i += blockDim.x) s_cf[i] = P.fdense[i];
    __syncthreads();
    OneWaveLds<T, D, M> *wl = reinterpret_cast<OneWaveLds<T, D, M> *>(s_one) + (threadIdx.x >> 6);
    EndRing<T, D> *ring = &wl->ring;
    Walker<T, D, EST, M, false> w;
    w.cf = s_cf;
    w.mt.init();
    w.tr = std::is_same<M, RuntimeMode>::value ? wl->tr : nullptr;
    w.ks = key_schedule<KeysOf<T>>(P.key0, P.key1);
    int st = 0;  // 0 idle, 1 walking, 2 ended (to be scored)
    Pool pool;
    uint32_t ring_head = 0, ring_count = 0;
    bool tail_open = L.tail_max != 0;

    for (uint32_t iter = 0;; ++iter) {
        if ((iter & L.refill_mask) == 0) {  // refill turn (wave-uniform)
            if constexpr (kRingScoreOne<M>) {
                const uint64_t ended = __ballot(st == 2);
                if (ended) {
                    if (st == 2) {
                        const uint32_t at = (ring_head + ring_count + (uint32_t)__popcll(ended & below)) & (kEndRing - 1);
                        w.stash(ring->e[at], a.rec_base);  // set per launch by the host
                        st = 0;
                    }
                    ring_count += (uint32_t)__popcll(ended);
                }
            } else if (st == 2) {
                w.finish(a, P, a.rec_base);
                st = 0;
            }
            if (tail_open && pool.exhausted && pool.next == pool.end)
                tail_open = hand_over_live<T, D>(L, 0, lane, below, a.stream_tag, w, st);
            const uint64_t idle = __ballot(st == 0);
            if constexpr (kRingScoreOne<M>) {
                const bool leaving = idle == ~0ull && pool.next == pool.end;  // the wave may stop at this turn
                while (ring_count >= 64u || (leaving && ring_count)) {
                    const uint32_t n = min(ring_count, 64u);
                    if ((uint32_t)lane < n) {
                        const EndedPath<T, D> &e = ring->e[(ring_head + (uint32_t)lane) & (kEndRing - 1)];
                        T Xt[D];
#pragma unroll
                        for (int d = 0; d < D; ++d) Xt[d] = e.Xt[d];
                        score_path<T, D, EST, M>(w.mt, a, P, Xt, e.Y, e.Z, e.R, e.word, e.r);
                    }
                    ring_head = (ring_head + n) & (kEndRing - 1);
                    ring_count -= n;
                }
            }
            if (idle) {
                pool.refill(L, lane);
                const uint32_t avail = pool.end - pool.next;
                const uint32_t rank = (uint32_t)__popcll(idle & below);
                if (st == 0 && rank < avail) st = w.start(a, P, L.slot_begin + pool.next + rank, nullptr) ? 1 : 2;  // the one item starts at slot 0
                pool.next += min(avail, (uint32_t)__popcll(idle));
            }
            if (__ballot(st != 0) == 0) {
                if (pool.exhausted) break;
                continue;
            }
        }
        if (st == 1) {
            // One Philox block feeds two steps in 2D (words 0,1 then 2,3), one in 3D.
            if (D == 2) {
                const Block4 q = philox(w.k >> 1, w.j, w.node, w.stream(a), w.ks);
                if (!w.step(a, P, q.w0, q.w1, 0u, 0u))
                    st = 2;
                else if (!w.step(a, P, q.w2, q.w3, 0u, 0u))
                    st = 2;
            } else {
                const Block4 q = philox(w.k, w.j, w.node, w.stream(a), w.ks);
                if (!w.step(a, P, q.w0, q.w1, q.w2, q.w3)) st = 2;
            }
        }
    }
}

// A batch: items and problems in device tables read at wave-uniform indices.
// Each wave keeps the source coefficients of its current problem in its own
// LDS slot (written when it changes item; a wave's LDS accesses complete in
// order, so no barrier is needed).
// FP64 walks are asked to fit three waves per SIMD (168 registers; the few
// spilled values live outside the step loop), which is faster than two, and
// the FP32 2D box / bridge / Gaussian correction walks five (96 registers:
// one 8-byte value is reloaded at refill turns).
template <class T, int D, int EST, class M>
constexpr int kManyMinWaves = sizeof(T) == 8 ? (D == 3 && (EST == kEstIto || std::is_same<M, RuntimeMode>::value) ? 2 : 3)
                              : (D == 2 && EST == kEstCorrection && !std::is_same<M, RuntimeMode>::value) ? 5
                                                                                                          : 1;
template <class T, int D, int EST, class M>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kManyMinWaves<T, D, EST, M>, 8)))
    path_kernel_many(const LaunchArgs L, const ItemDesc<T> *__restrict__ items,
                     const DevProblem<T> *__restrict__ probs)
{
    const int lane = __lane_id();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    __shared__ T s_cf[256 / 64][kMaxDense];
    extern __shared__ uint64_t s_ring[];  // dynamic: one EndRing per wave
    T *my_cf = s_cf[threadIdx.x >> 6];
    EndRing<T, D> *ring = reinterpret_cast<EndRing<T, D> *>(s_ring) + (threadIdx.x >> 6);
    Walker<T, D, EST, M, true> w;
    w.cf = my_cf;
    w.tr = nullptr;
    w.mt.init();
    int st = 0;
    ItemQueue<T> q;
    // Ended paths are scored 64 at a time, one per lane, from the wave's ring
    // (ring_head, ring_count: wave-uniform): scored as each lane ends, the
    // scoring would run for the whole wave at nearly every refill turn of
    // short walks for the two or three lanes that ended. Every ended path of
    // an item is scored before the wave leaves it.
    uint32_t ring_head = 0, ring_count = 0;
    bool tail_open = L.tail_max != 0;

    for (uint32_t iter = 0;; ++iter) {
        if ((iter & L.refill_mask) == 0) {  // refill turn (wave-uniform)
            const uint64_t ended = __ballot(st == 2);
            if (ended) {
                if (st == 2) {
                    const ItemDesc<T> &it = items[q.cur];
                    const uint32_t at = (ring_head + ring_count + (uint32_t)__popcll(ended & below)) & (kEndRing - 1);
                    // scratch records sit at group slot - launch start (modular arithmetic)
                    w.stash(ring->e[at], it.rec_launch ? L.slot_begin - it.slot_begin : it.rec_base);
                    st = 0;
                }
                ring_count += (uint32_t)__popcll(ended);
            }
            if (tail_open && q.cur >= 0 && q.dry && q.next == q.end)
                tail_open = hand_over_live<T, D>(L, (uint32_t)(q.cur - L.item_lo), lane, below, 0u, w, st);
            const uint64_t idle = __ballot(st == 0);
            const bool leaving = idle == ~0ull && q.next == q.end;  // the wave may move or stop at this turn
            while (ring_count >= 64u || (leaving && ring_count)) {
                const uint32_t n = min(ring_count, 64u);
                if ((uint32_t)lane < n) {
                    const ItemDesc<T> &it = items[q.cur];
                    const EndedPath<T, D> &e = ring->e[(ring_head + (uint32_t)lane) & (kEndRing - 1)];
                    T Xt[D];
#pragma unroll
                    for (int d = 0; d < D; ++d) Xt[d] = e.Xt[d];
                    score_path<T, D, EST, M>(w.mt, it, probs[it.prob], Xt, e.Y, e.Z, e.R, e.word, e.r);
                }
                ring_head = (ring_head + n) & (kEndRing - 1);
                ring_count -= n;
            }
            if (idle && q.next == q.end && !q.done) {
                if (!q.dry) q.take(L, lane);
                if (q.dry && idle == ~0ull) {
                    const int prev = q.cur;
                    uint32_t k;
                    if (prev < 0) {  // first item: the one holding this wave's share of the launch
                        const uint32_t waves = gridDim.x * (blockDim.x >> 6);
                        const uint32_t gw = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
                        const uint64_t s0 = L.slot_begin + (uint64_t)gw * L.launch_slots / waves;
                        k = (uint32_t)(find_item(items, L.n_items, s0) - L.item_lo);
                        if (k >= L.n_seg) k = 0;
                    } else {
                        k = (uint32_t)(prev - L.item_lo) + 1;
                        if (k >= L.n_seg) k = 0;
                    }
                    q.move(items, L, lane, k);
                    if (!q.done && q.cur != prev) {
                        const ItemDesc<T> &it = items[q.cur];
                        w.ks = key_schedule<KeysOf<T>>(probs[it.prob].key0, probs[it.prob].key1);
                        if (lane < kMaxDense) my_cf[lane] = probs[it.prob].fdense[lane];
                    }
                    tail_open = L.tail_max != 0;
                }
            }
            if (idle && q.next < q.end) {
                const uint32_t avail = q.end - q.next;
                const uint32_t rank = (uint32_t)__popcll(idle & below);
                if (st == 0 && rank < avail) {
                    const ItemDesc<T> &it = items[q.cur];
                    st = w.start(it, probs[it.prob], L.slot_begin + q.next + rank - it.slot_begin, it.node_rng) ? 1 : 2;
                }
                q.next += min(avail, (uint32_t)__popcll(idle));
            }
            if (__ballot(st != 0) == 0) {
                if (q.done) break;
                continue;
            }
        }
        if (st == 1) {
            const ItemDesc<T> &a = items[q.cur];
            const DevProblem<T> &P = probs[a.prob];
            if (D == 2) {
                const Block4 b4 = philox(w.k >> 1, w.j, w.node, w.stream(a), w.ks);
                if (!w.step(a, P, b4.w0, b4.w1, 0u, 0u))
                    st = 2;
                else if (!w.step(a, P, b4.w2, b4.w3, 0u, 0u))
                    st = 2;
            } else {
                const Block4 b4 = philox(w.k, w.j, w.node, w.stream(a), w.ks);
                if (!w.step(a, P, b4.w0, b4.w1, b4.w2, b4.w3)) st = 2;
            }
        }
    }
}

}  // namespace

template <class T, int D, int EST>
hipError_t launch_path_kernel(const LaunchArgs &l, const ItemDesc<T> *items,
                              const DevProblem<T> *probs, int grid, int block, int kind, hipStream_t s)
{
    const size_t lds = (size_t)(block / 64) * sizeof(EndRing<T, D>);
    if (kind == kKernelDense)
        hipLaunchKernelGGL((path_kernel_many<T, D, EST, BoxBridgeGaussDense>), dim3(grid), dim3(block), lds, s, l,
                           items, probs);
    else if (kind == kKernelSparse)
        hipLaunchKernelGGL((path_kernel_many<T, D, EST, BoxBridgeGauss>), dim3(grid), dim3(block), lds, s, l,
                           items, probs);
    else
        hipLaunchKernelGGL((path_kernel_many<T, D, EST, RuntimeMode>), dim3(grid), dim3(block), lds, s, l, items,
                           probs);
    return hipGetLastError();
}

template <class T, int D, int EST>
hipError_t launch_path_kernel_one(const OneItemArgs<T> &a, int grid, int block, int kind, hipStream_t s)
{
    if constexpr (kOneItemKernel<T, D, EST>) {
        static_assert(sizeof(OneItemArgs<T>) <= 4096, "kernel arguments exceed 4 KiB");
        const size_t waves = (size_t)(block / 64);
        if (kind == kKernelDense)
            hipLaunchKernelGGL((path_kernel_one<T, D, EST, BoxBridgeGaussDense>), dim3(grid), dim3(block),
                               waves * sizeof(OneWaveLds<T, D, BoxBridgeGaussDense>), s, a);
        else if (kind == kKernelSparse)
            hipLaunchKernelGGL((path_kernel_one<T, D, EST, BoxBridgeGauss>), dim3(grid), dim3(block), 0, s, a);
        else
            hipLaunchKernelGGL((path_kernel_one<T, D, EST, RuntimeMode>), dim3(grid), dim3(block),
                               waves * sizeof(OneWaveLds<T, D, RuntimeMode>), s, a);
        return hipGetLastError();
    } else {
        return hipErrorInvalidDeviceFunction;
    }
}

template <class T, int D, int EST>
const void *path_kernel_symbol(bool one, int kind)
{
    if constexpr (kOneItemKernel<T, D, EST>)
        if (one)
            return kind == kKernelDense    ? reinterpret_cast<const void *>(&path_kernel_one<T, D, EST, BoxBridgeGaussDense>)
                   : kind == kKernelSparse ? reinterpret_cast<const void *>(&path_kernel_one<T, D, EST, BoxBridgeGauss>)
                                           : reinterpret_cast<const void *>(&path_kernel_one<T, D, EST, RuntimeMode>);
    return kind == kKernelDense    ? reinterpret_cast<const void *>(&path_kernel_many<T, D, EST, BoxBridgeGaussDense>)
           : kind == kKernelSparse ? reinterpret_cast<const void *>(&path_kernel_many<T, D, EST, BoxBridgeGauss>)
                                   : reinterpret_cast<const void *>(&path_kernel_many<T, D, EST, RuntimeMode>);
}

template <class S, class T, int D>
hipError_t launch_cells(const CellGrids<S> &g, int n_grids, const int32_t *n, T *cells, uint32_t stride, uint32_t off,
                        hipStream_t s)
{
    const uint64_t n_cells = cell_values<T>(n, D) >> D;
    if (n_cells == 0) return hipSuccess;
    const uint64_t blocks = std::min<uint64_t>((n_cells + 255) / 256, 4096);
    hipLaunchKernelGGL((grid_cells_kernel<S, T, D>), dim3((uint32_t)blocks, n_grids), dim3(256), 0, s, g, n[0], n[1],
                       D == 3 ? n[2] : 1, cells, stride, off);
    return hipGetLastError();
}

template <class S, class T, int D>
hipError_t launch_grid_cells_strided(const S *data, const int32_t *n, T *cells, uint32_t stride, uint32_t off,
                                     hipStream_t s)
{
    return launch_cells<S, T, D>(CellGrids<S>{{data, nullptr, nullptr}}, 1, n, cells, stride, off, s);
}

template <class T, int D>
hipError_t launch_grid_cells(const T *const *data, int n_grids, const int32_t *n, T *cells, hipStream_t s)
{
    CellGrids<T> g{};
    for (int c = 0; c < n_grids; ++c) g.data[c] = data[c];
    return launch_cells<T, T, D>(g, n_grids, n, cells, (uint32_t)(n_grids << D), 0u, s);
}

template <class S, class T>
hipError_t launch_grid_points_strided(const S *data, uint64_t n_points, T *out, uint32_t stride, uint32_t off,
                                      hipStream_t s)
{
    if (n_points == 0) return hipSuccess;
    const uint64_t blocks = std::min<uint64_t>((n_points + 255) / 256, 4096);
    hipLaunchKernelGGL((grid_points_kernel<S, T>), dim3((uint32_t)blocks), dim3(256), 0, s, data, n_points, out,
                       stride, off);
    return hipGetLastError();
}
template hipError_t launch_grid_points_strided<float, float>(const float *, uint64_t, float *, uint32_t, uint32_t,
                                                             hipStream_t);
template hipError_t launch_grid_points_strided<float, double>(const float *, uint64_t, double *, uint32_t,
                                                              uint32_t, hipStream_t);
template hipError_t launch_grid_points_strided<double, float>(const double *, uint64_t, float *, uint32_t,
                                                              uint32_t, hipStream_t);
template hipError_t launch_grid_points_strided<double, double>(const double *, uint64_t, double *, uint32_t,
                                                               uint32_t, hipStream_t);

#define PDD_GRID_CELLS(S, T, D) \
    template hipError_t launch_grid_cells_strided<S, T, D>(const S *, const int32_t *, T *, uint32_t, uint32_t, \
                                                            hipStream_t);
template hipError_t launch_grid_cells<float, 2>(const float *const *, int, const int32_t *, float *, hipStream_t);
template hipError_t launch_grid_cells<float, 3>(const float *const *, int, const int32_t *, float *, hipStream_t);
template hipError_t launch_grid_cells<double, 2>(const double *const *, int, const int32_t *, double *, hipStream_t);
template hipError_t launch_grid_cells<double, 3>(const double *const *, int, const int32_t *, double *, hipStream_t);
PDD_GRID_CELLS(float, float, 2)
PDD_GRID_CELLS(float, float, 3)
PDD_GRID_CELLS(double, double, 2)
PDD_GRID_CELLS(double, double, 3)
PDD_GRID_CELLS(float, double, 2)
PDD_GRID_CELLS(float, double, 3)
PDD_GRID_CELLS(double, float, 2)
PDD_GRID_CELLS(double, float, 3)

#define PDD_INSTANTIATE(T, D, EST)                                                              \
    template hipError_t launch_path_kernel<T, D, EST>(const LaunchArgs &, const ItemDesc<T> *, \
                                                     const DevProblem<T> *, int, int, int, hipStream_t); \
    template hipError_t launch_path_kernel_one<T, D, EST>(const OneItemArgs<T> &, int, int, int, hipStream_t); \
    template const void *path_kernel_symbol<T, D, EST>(bool, int);

PDD_INSTANTIATE(float, 2, kEstPlain)
PDD_INSTANTIATE(float, 2, kEstCorrection)
PDD_INSTANTIATE(float, 2, kEstIto)
PDD_INSTANTIATE(float, 3, kEstPlain)
PDD_INSTANTIATE(float, 3, kEstCorrection)
PDD_INSTANTIATE(float, 3, kEstIto)
PDD_INSTANTIATE(double, 2, kEstPlain)
PDD_INSTANTIATE(double, 2, kEstCorrection)
PDD_INSTANTIATE(double, 2, kEstIto)
PDD_INSTANTIATE(double, 3, kEstPlain)
PDD_INSTANTIATE(double, 3, kEstCorrection)
PDD_INSTANTIATE(double, 3, kEstIto)

}  // namespace pdd
