// Group-walk path kernel: several lanes walk one path together.
#include "path_walk.hpp"

namespace pdd {
namespace {

// A walk is a serial chain, and one path per lane makes every step of it cost
// the whole step's instructions: a lone wave takes 0.41 us a step in FP32 2D
// and 1.0 us in FP64. When a launch has fewer paths than lanes, or has only its
// longest paths left, that chain is its time. Here G lanes walk one path
// together, a window of G S steps at a time (S = 2 in 2D, 1 in 3D, the steps of
// one Philox block):
//  1. lane g draws the normals of steps S g .. S g + S - 1 of the window
//     (counter-based, so they need nothing of the walk);
//  2. every lane walks X and Y through the window with all its normals
//     (broadcast by DPP), ignoring exits: b and c only, 17 instructions a step
//     in FP32 2D, and lane g keeps the state before its own steps;
//  3. lane g takes its own S steps from there with the ordinary step code:
//     source, control variate and exit test, for all lanes at once;
//  4. the first lane with an exit, if any, ends the path; the lanes' terms of
//     Z and R up to it are added in step order.
// Every operation on a path and its order are those of the other kernels, so
// the results are bitwise the same. Groups start as quads, 16 paths to a wave
// (more lanes if there are fewer paths), which take new paths as theirs end,
// and grow to 64 lanes as an item's last paths are left: 0.07 us a step then in
// FP32 and 0.09 us in FP64, bound by phase 2's chain. Quads cost 1.5 to 2.5
// times the instructions per path-step of one path per lane (phase 2 runs in
// all four lanes), which decides where the one or the other is used; pairs and
// single lanes in this kernel were slower than quads at every size (18 nodes x
// 10,000 FP64 paths: 0.77 ms from single lanes, 0.66 ms from pairs, 0.64 ms
// from quads, 0.71 ms from groups of eight). Measured, before and with it: 18
// nodes x 1,000 correction paths on the unit square 0.75 and 0.18 ms, x 10,000
// plain FP64 paths 2.0 and 0.64 ms, 64 uneven problems of 4.0e6 paths 295 and
// 141 ms, 1,792 nodes x 8,192 long walks 322 and 293 ms.

// Broadcast within a quad: its lane g's value (quad_perm g, g, g, g).
template <int g>
__device__ __forceinline__ int quad32(int v)
{
    return __builtin_amdgcn_mov_dpp(v, g * 0x55, 0xf, 0xf, false);
}
template <int g>
__device__ __forceinline__ float quad(float v)
{
    return __int_as_float(quad32<g>(__float_as_int(v)));
}
template <int g>
__device__ __forceinline__ double quad(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)quad32<g>((int)(uint32_t)b), hi = (uint32_t)quad32<g>((int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// The value of lane `from` (any lane of the wave, all lanes active).
__device__ __forceinline__ float lane_value(float v, int from)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(from << 2, __float_as_int(v)));
}
__device__ __forceinline__ double lane_value(double v, int from)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from << 2, (int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from << 2, (int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// The path of a group between windows (the same in all its lanes).
template <class T, int D>
struct GroupPath {
    T X[D], Y, m;
    double Z, R;
    uint32_t k;
    bool alive;
};

template <class T, int D, int EST, class M>
struct GroupWalk {
    static constexpr int S = D == 2 ? 2 : 1;
    Walker<T, D, EST, M, true, ScalarKey> w;
    GroupPath<T, D> p;
    ItemQueue<T, true> q;
    EndRing<T, D> *ring;
    T *cf;
    uint32_t ring_head = 0, ring_count = 0;

    // Puts the ended paths of the lanes with `fin` on the ring.
    __device__ __forceinline__ void push(bool fin, const ItemDesc<T> &it, const LaunchArgs &L, uint64_t below)
    {
        const uint64_t m = __ballot(fin);
        if (m == 0) return;
        if (fin) {
            const uint32_t at = (ring_head + ring_count + (uint32_t)__popcll(m & below)) & (kEndRing - 1);
            w.stash(ring->e[at], it.rec_launch ? L.slot_begin - it.slot_begin : it.rec_base);
        }
        ring_count += (uint32_t)__popcll(m);
    }

    __device__ __forceinline__ void score(const ItemDesc<T> *__restrict__ items,
                                          const DevProblem<T> *__restrict__ probs, int lane, bool all)
    {
        while (ring_count >= 64u || (all && ring_count)) {
            const uint32_t n = min(ring_count, 64u);
            if ((uint32_t)lane < n) {
                const ItemDesc<T> &it = items[__builtin_amdgcn_readfirstlane(q.cur)];
                const EndedPath<T, D> &e = ring->e[(ring_head + (uint32_t)lane) & (kEndRing - 1)];
                T Xt[D];
#pragma unroll
                for (int d = 0; d < D; ++d) Xt[d] = e.Xt[d];
                score_path<T, D, EST, M>(w.mt, it, probs[__builtin_amdgcn_readfirstlane(it.prob)], Xt, e.Y, e.Z, e.R, e.word, e.r);
            }
            ring_head = (ring_head + n) & (kEndRing - 1);
            ring_count -= n;
        }
    }

    // One window of every live group of G lanes (4 to 64, a power of two). The
    // lanes' increments and terms are taken four lanes at a time: each quad
    // fetches those of lanes c .. c + 3 of its group (its own, if the group is
    // one quad) and broadcasts them one by one.
    __device__ __forceinline__ void window(int G, const ItemDesc<T> &a, const DevProblem<T> &P, const LaunchArgs &L,
                                           int lane, uint64_t below)
    {
        const int g = lane & (G - 1);
        const int from = (lane & ~(G - 1)) | (lane & 3);
        w.ks = key_schedule<ScalarKey>(P.key0, P.key1);
        // 1. this lane's normals
        T n[S][D];
        w.k = p.k + (uint32_t)(S * g);
        if constexpr (D == 2) {
            const Block4 b4 = philox(w.k >> 1, w.j, w.node, w.stream(a), w.ks);
            w.draw(a, b4.w0, b4.w1, 0u, 0u, n[0]);
            w.draw(a, b4.w2, b4.w3, 0u, 0u, n[S - 1]);
        } else {
            const Block4 b4 = philox(w.k, w.j, w.node, w.stream(a), w.ks);
            w.draw(a, b4.w0, b4.w1, b4.w2, b4.w3, n[0]);
        }
        // 2. the walk without exits; the state before this lane's steps
        T x[D], y = p.Y;
#pragma unroll
        for (int d = 0; d < D; ++d) w.X[d] = x[d] = p.X[d];
        w.Y = y;
        for (int c = 0; c < G; c += 4) {
            T nq[S][D];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int d = 0; d < D; ++d) nq[s][d] = G == 4 ? n[s][d] : lane_value(n[s][d], from + c);
            static_for<0, 4 * S>([&](auto J) {
                constexpr int j = decltype(J)::value;
                if constexpr (j % S == 0) {
                    const bool mine = g == c + j / S;
#pragma unroll
                    for (int d = 0; d < D; ++d) w.X[d] = mine ? x[d] : w.X[d];
                    w.Y = mine ? y : w.Y;
                }
                T b[D], k, f;
                coefficients<T, D, M::kBigTrig>(w.mt, P, x, b, k, f, false, nullptr, M::tab(P));
                y = madd(a.h * y, k, y);
#pragma unroll
                for (int d = 0; d < D; ++d)
                    x[d] = madd(a.sig_sqh, quad<j / S>(nq[j % S][d]), madd(a.h, b[d], x[d]));
            });
        }
        // 3. this lane's steps
        double iz[S], ir[S];
        bool ended = false;
#pragma unroll
        for (int s = 0; s < S; ++s) iz[s] = ir[s] = 0.0;
        if (p.alive) {
            const T dist = point_distance<T, D>(P, M::domain(P), w.X);
            w.m = g == 0 ? p.m : dist;
            w.capped = 0;
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (!ended) {
                    w.Z = w.R = 0.0;
                    ended = !w.advance(a, P, n[s]);
                    iz[s] = w.Z;
                    ir[s] = w.R;
                }
        }
        // 4. the first exit, and the terms up to it in order
        const bool has_z = EST != kEstCorrection || a.score_plain;
        const uint64_t ends = (__ballot(ended) >> (lane & ~(G - 1))) & (~0ull >> (64 - G));
        const int first = ends ? __builtin_ctzll(ends) : G;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            iz[s] = g <= first ? iz[s] : 0.0;
            ir[s] = g <= first ? ir[s] : 0.0;
        }
        for (int c = 0; c < G; c += 4) {
            double zq[S], rq[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                zq[s] = G == 4 || !has_z ? iz[s] : lane_value(iz[s], from + c);
                rq[s] = G == 4 || EST == kEstPlain ? ir[s] : lane_value(ir[s], from + c);
            }
            static_for<0, 4 * S>([&](auto J) {
                constexpr int j = decltype(J)::value;
                if (has_z) p.Z += quad<j / S>(zq[j % S]);
                if (EST != kEstPlain) p.R += quad<j / S>(rq[j % S]);
            });
        }
#pragma unroll
        for (int d = 0; d < D; ++d) p.X[d] = x[d];
        p.Y = y;
        p.m = lane_value(w.m, lane | (G - 1));
        if (first < G) p.alive = false;
        w.Z = p.Z;
        w.R = p.R;
        push(g == first, a, L, below);
        p.k += (uint32_t)(G * S);
    }

    // First lanes of the groups of G.
    __device__ static __forceinline__ uint64_t leaders_of(int G)
    {
        uint64_t m = 1ull;
        for (int s = 32; s >= G; s >>= 1) m |= m << s;
        return m;
    }

    // The wave's first item, or the one to look at after its own: of a launch's
    // slots the one at the wave's share of them, of handed-over paths any.
    __device__ __forceinline__ uint32_t next_item(const LaunchArgs &L, const ItemDesc<T> *__restrict__ items) const
    {
        const uint32_t waves = gridDim.x * (blockDim.x >> 6);
        const uint32_t gw =
            __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
        uint32_t k;
        if (q.cur >= 0)
            k = (uint32_t)(q.cur - L.item_lo) + 1;
        else if (L.tail)
            k = gw % L.n_seg;
        else
            k = (uint32_t)(find_item(items, L.n_items, L.slot_begin + (uint64_t)gw * L.launch_slots / waves) - L.item_lo);
        return k < L.n_seg ? k : 0;
    }

    // Gives the idle groups (`idle`: their first lanes) new paths, after
    // moving a wave with none left to another item.
    __device__ __forceinline__ void refill(const LaunchArgs &L, const ItemDesc<T> *__restrict__ items,
                                           const DevProblem<T> *__restrict__ probs, int lane, uint64_t below,
                                           uint64_t idle, int &G, uint64_t &leaders)
    {
        const bool none = idle == leaders;
        score(items, probs, lane, none && q.next == q.end);
        if (q.next == q.end && !q.done) {
            if (!q.dry) q.take(L, lane);
            if (q.dry && none) {
                const int prev = q.cur;
                q.move(items, L, lane, next_item(L, items));
                G = 64 / (int)q.grab;
                idle = leaders = leaders_of(G);
                if (!q.done && q.cur != prev) {
                    const ItemDesc<T> &it = items[__builtin_amdgcn_readfirstlane(q.cur)];
                    const DevProblem<T> &P = probs[__builtin_amdgcn_readfirstlane(it.prob)];
                    if (lane < kMaxDense) cf[lane] = P.fdense[lane];
                }
            }
        }
        if (q.next == q.end) return;
        const ItemDesc<T> &it = items[__builtin_amdgcn_readfirstlane(q.cur)];
        const uint32_t avail = q.end - q.next;
        const uint32_t rank = (uint32_t)__popcll(idle & ((1ull << (lane & ~(G - 1))) - 1ull));
        bool ended = false;  // before any step
        if (!p.alive && rank < avail) {
            if (L.tail) {
                w.take_over(static_cast<const TailState<T, D> *>(L.tail)[q.next + rank]);
                p.alive = true;
            } else {
                p.alive = w.start(it, probs[__builtin_amdgcn_readfirstlane(it.prob)],
                                  L.slot_begin + q.next + rank - it.slot_begin, it.node_rng);
                ended = !p.alive && (lane & (G - 1)) == 0;
            }
#pragma unroll
            for (int d = 0; d < D; ++d) p.X[d] = w.X[d];
            p.Y = w.Y;
            p.m = w.m;
            p.Z = w.Z;
            p.R = w.R;
            p.k = w.k;
        }
        push(ended, it, L, below);
        q.next += min(avail, (uint32_t)__popcll(idle));
    }

    // Walks paths until there are none left.
    __device__ __forceinline__ void run(const LaunchArgs &L, const ItemDesc<T> *__restrict__ items,
                                        const DevProblem<T> *__restrict__ probs, int lane, uint64_t below)
    {
        int G = 4;
        uint64_t leaders = leaders_of(G);
        for (;;) {
            const uint64_t idle = __ballot(!p.alive) & leaders;
            if (idle) refill(L, items, probs, lane, below, idle, G, leaders);
            const uint64_t live = __ballot(p.alive) & leaders;
            if (live == 0) {
                if (q.done && ring_count == 0) return;
                continue;
            }
            if (q.dry && q.next == q.end) {  // no more for this item: as many lanes as its last paths can take
                const uint32_t n = (uint32_t)__popcll(live);
                const int wider = n <= 1 ? 64 : (int)(64u >> (32 - __builtin_clz(n - 1)));
                if (wider > G) {
                    regroup(lane, live, wider);
                    G = wider;
                    leaders = leaders_of(G);
                }
            }
            const ItemDesc<T> &a = items[__builtin_amdgcn_readfirstlane(q.cur)];
            window(G, a, probs[__builtin_amdgcn_readfirstlane(a.prob)], L, lane, below);
        }
    }

    // Moves the live paths (`live`: the first lanes of their groups) to the
    // first groups of `wider` lanes.
    __device__ __forceinline__ void regroup(int lane, uint64_t live, int wider)
    {
        // lane r learns the r-th live lane, then each group that of its number
        const uint32_t rank = (uint32_t)__popcll(live & (lane ? (~0ull >> (64 - lane)) : 0ull));
        const bool lead = (live >> lane) & 1;
        const int nth = __builtin_amdgcn_ds_permute((lead ? (int)rank : 63) << 2, lane);
        const int group = lane / wider;
        const int n_live = __popcll(live);
        const int src = __shfl(nth, group);
        const bool has = group < n_live;
        const int from = has ? src : lane;
#pragma unroll
        for (int d = 0; d < D; ++d) p.X[d] = __shfl(p.X[d], from);
        p.Y = __shfl(p.Y, from);
        p.m = __shfl(p.m, from);
        p.Z = __shfl(p.Z, from);
        p.R = __shfl(p.R, from);
        p.k = __shfl(p.k, from);
        w.slot = __shfl(w.slot, from);
        w.j = __shfl(w.j, from);
        w.node = __shfl(w.node, from);
        w.tag = __shfl(w.tag, from);
        w.bb_blk = 0xffffffffu;
        p.alive = has;
    }
};

template <class T, int D, int EST, class M>
__global__ void __launch_bounds__(256) path_kernel_group(const LaunchArgs L, const ItemDesc<T> *__restrict__ items,
                                                         const DevProblem<T> *__restrict__ probs)
{
    const int lane = __lane_id();
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    __shared__ T s_cf[256 / 64][kMaxDense];
    extern __shared__ uint64_t s_ring[];  // dynamic: one EndRing per wave
    GroupWalk<T, D, EST, M> G;
    G.cf = s_cf[threadIdx.x >> 6];
    G.ring = reinterpret_cast<EndRing<T, D> *>(s_ring) + (threadIdx.x >> 6);
    G.w.cf = G.cf;
    G.w.tr = nullptr;
    G.w.mt.init();
    G.w.j = G.w.node = G.w.tag = 0;
    G.w.slot = 0;
    G.w.bb_blk = 0xffffffffu;
    G.w.m = (T)0;
#pragma unroll
    for (int d = 0; d < D; ++d) G.p.X[d] = G.w.Xt[d] = (T)0;
    G.p.Y = G.p.m = (T)0;
    G.p.Z = G.p.R = 0.0;
    G.p.k = 0;
    G.p.alive = false;
    G.run(L, items, probs, lane, below);
}

}  // namespace

template <class T, int D, int EST>
hipError_t launch_path_kernel_group(const LaunchArgs &l, const ItemDesc<T> *items, const DevProblem<T> *probs,
                                    int grid, int kind, hipStream_t s)
{
    const size_t lds = (size_t)(kGroupBlock / 64) * sizeof(EndRing<T, D>);
    if (kind == kKernelGeneric)
        hipLaunchKernelGGL((path_kernel_group<T, D, EST, RuntimeMode>), dim3(grid), dim3(kGroupBlock), lds, s, l, items,
                           probs);
    else
        hipLaunchKernelGGL((path_kernel_group<T, D, EST, BoxBridgeGaussDense>), dim3(grid), dim3(kGroupBlock), lds, s, l,
                           items, probs);
    return hipGetLastError();
}

#define PDD_INSTANTIATE_GROUP(T, D, EST)                                                                    \
    template hipError_t launch_path_kernel_group<T, D, EST>(const LaunchArgs &, const ItemDesc<T> *, \
                                                            const DevProblem<T> *, int, int, hipStream_t);

PDD_INSTANTIATE_GROUP(float, 2, kEstPlain)
PDD_INSTANTIATE_GROUP(float, 2, kEstCorrection)
PDD_INSTANTIATE_GROUP(float, 2, kEstIto)
PDD_INSTANTIATE_GROUP(float, 3, kEstPlain)
PDD_INSTANTIATE_GROUP(float, 3, kEstCorrection)
PDD_INSTANTIATE_GROUP(float, 3, kEstIto)
PDD_INSTANTIATE_GROUP(double, 2, kEstPlain)
PDD_INSTANTIATE_GROUP(double, 2, kEstCorrection)
PDD_INSTANTIATE_GROUP(double, 2, kEstIto)
PDD_INSTANTIATE_GROUP(double, 3, kEstPlain)
PDD_INSTANTIATE_GROUP(double, 3, kEstCorrection)
PDD_INSTANTIATE_GROUP(double, 3, kEstIto)

}  // namespace pdd
