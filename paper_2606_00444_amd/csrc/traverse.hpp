// Closest-point / nearest-point traversal pieces shared by the plain query
// kernels and the batched persistent kernel.
//
// Pruning: a child is expanded when its lower bound is <= prune_bound(best):
// the slack keeps a face whose float32 distance ties the best from being
// pruned, whatever order the faces are met in, so every traversal returns the
// lowest original id among the faces at the minimal float32 distance (carried
// in the node record beside each leaf child).  Leaf children hold their
// triangle, so a leaf is tested with the data of the record that referenced it.
#pragma once

#include "mgu_internal.hpp"

#include <climits>

namespace mgu {

constexpr int kLaneBlock = 64;
constexpr int kLdsStack = 32;
constexpr int kMaxStack = 64;
constexpr float kPruneSlack = 1.0f + 1.0f / 1048576.0f;

// The largest lower bound of a node that may still hold a face whose float32
// squared distance ties `best`.  A float32 closest point on a well-shaped
// triangle is off by a few units in the last place of the coordinates'
// magnitude (about |q|_1 + sqrt(best) near q), so its float32 distance may
// fall short of the exact one by delta = 2^-18 (|q|_1 + sqrt(best)) - a wide
// margin - while the box and slab bounds are within a few rounding steps of
// exact: expanding every node with sqrt(bound) <= sqrt(best) + delta (times
// 1 + 2^-20 for the bound's own rounding) keeps such faces.  qm = |q|_1.
__device__ __forceinline__ float prune_bound(float best, float qm) {
    const float d = __builtin_amdgcn_sqrtf(best);
    const float e = fmaf(0x1p-18f, qm + d, d);
    return (e * e) * kPruneSlack;
}

// |q|_1 of a query point (the magnitude of the prune slack and the slab margin).
__device__ __forceinline__ float qnorm1(f3 q) { return (fabsf(q.x) + fabsf(q.y)) + fabsf(q.z); }

constexpr int kBatchWaves = 4;          // waves per workgroup of the batch kernel
// Stack entries before the pop width shrinks, for batches of M queries: room for
// what a triangle tree's seed descents pass by (about 38 entries each).
constexpr int batch_cap(bool tri, int M) { return !tri || M > 16 ? 320 : M > 8 ? 704 : 448; }
constexpr int kPopNodes = 32;           // nodes a triangle round pops: a pair of lanes each
constexpr int batch_alloc(bool tri, int M) { return batch_cap(tri, M) + 64; }
constexpr int kLeafWait = 32;           // waiting leaves that are tested together
constexpr int kLeafNarrow = 8;          // stack entries below which waiting leaves are tested at once

struct QueryArgs {
    const float4 *nodes;                // [n-1][6]
    const float *root;                  // root box: lo at [0..2], hi at [4..6]
    const int32_t *leaf_faces;          // [3][n] (triangles) or nullptr (points)
    const int32_t *prim;                // [n]
    const float *verts;                 // mesh vertices or the points
    int64_t nv, n;
    const float *queries;
    int64_t nq;
    float maxd2;
    int32_t *face;
    float *point, *bary, *dist2, *normal;
    int seed;                           // batch kernel: seed descent first
    const int32_t *order;               // processing order (permutation) or nullptr
    unsigned long long *counters;       // [4] statistics or nullptr
    const int32_t *inv_prim;            // [n] leaf of each original id (id -> position in leaf order)
    const int32_t *leaf_parent;         // [n] record slot of each leaf: 2 x its parent node + the slot
    int32_t *status;                    // error word of the BVH header
    const int32_t *hdr_nv;              // vertex count of the build (header), or nullptr
    uint32_t *queue;                    // batch kernel: dynamic batch counter (zeroed before launch) or nullptr
    const int32_t *hint;                // [nq] original id to start each query from, or nullptr
    int coherent;                       // face ids stored and hints loaded device-coherent (batched form)
    int k;                              // faces kept per query (the k-nearest form; face and dist2 are then [k][nq])
    float eps;                          // its weights are 1 / (distance + eps)
};

// The face id of a result: with `coherent`, a relaxed device-scope store, which the
// other XCDs see without a write-back of the L2 (the batched form reads a scene's
// previous frame as hints while the launch runs).
__device__ __forceinline__ void store_face(const QueryArgs &a, int64_t q, int32_t id) {
    if (a.coherent) __hip_atomic_store(a.face + q, id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else a.face[q] = id;
}

// The first thread of a launch flags a vertex count that differs from the build's.
__device__ __forceinline__ void check_vertex_count(const QueryArgs &a) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.hdr_nv && *a.hdr_nv != a.nv) atomicOr(a.status, 32);
}

// Query processed in position i (order[i], or i); -1 if the order entry is out of range.
__device__ __forceinline__ int64_t query_at(const QueryArgs &a, int64_t i) {
    if (!a.order) return i;
    const int32_t q = a.order[i];
    return (q >= 0 && q < a.nq) ? q : -1;
}

__device__ __forceinline__ void add_counters(const QueryArgs &a, unsigned long long e, unsigned long long lb,
                                             unsigned long long lx, unsigned long long nq) {
    atomicAdd(a.counters + 0, e);
    atomicAdd(a.counters + 1, lb);
    atomicAdd(a.counters + 2, lx);
    atomicAdd(a.counters + 3, nq);
}

__device__ __forceinline__ f3 xyz(float4 v) { return f3{v.x, v.y, v.z}; }

// Exact squared distance to the leaf child stored in a record slot.
template <bool kTri>
__device__ __forceinline__ float leaf_dist2(f3 p, float4 f0, float4 f1, float4 f2) {
    if (kTri) {
        float w1, w2;
        return tri_closest(p, xyz(f0), xyz(f1), xyz(f2), w1, w2);
    }
    const f3 d = p - xyz(f0);
    return fdot(d, d);
}

// Box distance of a leaf child (its triangle's bounds, or the point itself).
template <bool kTri>
__device__ __forceinline__ float leaf_box_dist2(f3 p, float4 f0, float4 f1, float4 f2) {
    if (kTri) {
        const f3 lo = fmin3(fmin3(xyz(f0), xyz(f1)), xyz(f2));
        const f3 hi = fmax3(fmax3(xyz(f0), xyz(f1)), xyz(f2));
        return box_dist2(p, lo, hi);
    }
    const f3 d = p - xyz(f0);
    return fdot(d, d);
}

// Margin of a query's slab distances: 2^-20 of its coordinate magnitudes
// covers the float32 rounding of d.q.
__device__ __forceinline__ float slab_query_margin(f3 q) { return 0x1p-20f * qnorm1(q); }

// Lower bound of the squared distance from q to the faces below an internal
// child slot (c0, c1, c2) = (lo, ref) (hi, a) (d, b): the larger of the box
// distance and, for triangles, of the normal slab and the box's bounding ball
// together.  Along d every point x of the faces is at least the slab distance g
// away; across d, x lies within the ball's radius r of its centre c, so it is at
// least t - r away, t the length of q - c across d; the bound is g^2 + (t - r)^2.
// Either bound alone leaves whole neighbourhoods of a query inside a closed
// surface: the slab is an infinite plate that a neighbour's plane also passes
// near, and an axis-aligned box is as thick as it is wide.  Together they follow
// the surface patch: 1M queries on 500,000 faces expand 97 nodes a query where
// the box and the slab distance alone expanded 352.
//
// Rounding, with w = q - c as computed and u = 2^-24: w is off by at most
// 1.8 u (|q| + 2 |w|) (c rounded, then the difference), |w|^2 by 3 u |w|^2, the
// square of m = d.w by 7 u |w|^2 and, |d| being 1 to 2^-22, by another 8 u |w|^2.
// Taking 32 u |w|^2 = 2^-19 |w|^2 off t^2 = |w|^2 - m^2 covers the last three and
// lowers t by at least 7 u |w|, more than w's own error in |w| and that of the
// square root; dq = 2^-20 |q|_1 added to r covers the error in |q|, and the factor
// 1 + 2^-20 the rounding of r.  The clamp of t^2 keeps an overflow of |w|^2 from
// raising the bound.  dq is also the query's slab margin, and the last factor
// 1 - 2^-19 allows for |d| and the sums.  The box offset is p - median(p, lo, hi):
// one instruction less per axis than two differences and a maximum.
//
// kBall false: the larger of the box and the slab distance alone, a third of the work.
template <bool kTri, bool kBall = true>
__device__ __forceinline__ float child_bound(f3 q, float dq, float4 c0, float4 c1, float4 c2) {
    const float dx = q.x - __builtin_amdgcn_fmed3f(q.x, c0.x, c1.x);
    const float dy = q.y - __builtin_amdgcn_fmed3f(q.y, c0.y, c1.y);
    const float dz = q.z - __builtin_amdgcn_fmed3f(q.z, c0.z, c1.z);
    const float bd = fdot(f3{dx, dy, dz}, f3{dx, dy, dz});
    if (!kTri) return bd;
    const float s = c2.x * q.x + c2.y * q.y + c2.z * q.z;
    const float g = fmaxf(fmaxf(c1.w - s, s - c2.w) - dq, 0.0f);
    if (!kBall) return fmaxf(bd, (g * g) * (1.0f - 0x1p-19f));
    const f3 w = f3{fmaf(-0.5f, c0.x + c1.x, q.x), fmaf(-0.5f, c0.y + c1.y, q.y), fmaf(-0.5f, c0.z + c1.z, q.z)};
    const f3 h = f3{c1.x - c0.x, c1.y - c0.y, c1.z - c0.z};
    const float m = fdot(f3{c2.x, c2.y, c2.z}, w);
    const float t2 = fmaf(fdot(w, w), 1.0f - 0x1p-19f, -(m * m));
    const float t = __builtin_amdgcn_sqrtf(__builtin_amdgcn_fmed3f(t2, 0.0f, 1e37f));
    const float r = fmaf(__builtin_amdgcn_sqrtf(fdot(h, h)), 0.5f * (1.0f + 0x1p-20f), dq);
    const float across = fmaxf(t - r, 0.0f);
    return fmaxf(bd, fmaf(across, across, g * g) * (1.0f - 0x1p-19f));
}

__device__ __forceinline__ unsigned long long pack_best(float d2, int32_t id) {
    return (static_cast<unsigned long long>(__float_as_uint(d2)) << 32) | static_cast<uint32_t>(id);
}

// Final record of query q when no face qualifies.
__device__ __forceinline__ void write_none(const QueryArgs &a, int64_t q, f3 p) {
    store_face(a, q, -1);
    if (a.point) store3(a.point, a.nq, q, p);
    if (a.bary) { a.bary[q] = 0.0f; a.bary[a.nq + q] = 0.0f; }
    if (a.dist2) a.dist2[q] = INFINITY;
    if (a.normal) store3(a.normal, a.nq, q, f3{0.0f, 0.0f, 0.0f});
}

// Final record of query q on face `id`, the triangle ABC.
__device__ __forceinline__ void write_face(const QueryArgs &a, int64_t q, f3 p, int32_t id, f3 A, f3 B, f3 C) {
    float w1, w2;
    const float dd = tri_closest(p, A, B, C, w1, w2);
    store_face(a, q, id);
    if (a.point) store3(a.point, a.nq, q, tri_point(A, B, C, w1, w2));
    if (a.bary) { a.bary[q] = w1; a.bary[a.nq + q] = w2; }
    if (a.dist2) a.dist2[q] = dd;
    if (a.normal) store3(a.normal, a.nq, q, tri_normal(A, B, C));
}

// Final record of query q: recomputed from the winning leaf's face (triangles)
// or point, which the BVH stores bit-identically.
template <bool kTri>
__device__ void write_result(const QueryArgs &a, int64_t q, f3 p, int32_t leaf, int32_t id, float d2) {
    if (!kTri) {
        store_face(a, q, leaf >= 0 ? id : -1);
        if (a.dist2) a.dist2[q] = leaf >= 0 ? d2 : INFINITY;
    } else if (leaf >= 0 && leaf < a.n) {
        write_face(a, q, p, id, vload(a.verts, a.nv, a.leaf_faces[leaf]), vload(a.verts, a.nv, a.leaf_faces[a.n + leaf]),
                   vload(a.verts, a.nv, a.leaf_faces[2 * a.n + leaf]));
    } else {
        write_none(a, q, p);
    }
}

// Final record of query q from the winning original id (-1 / INT_MAX: none).
template <bool kTri>
__device__ void write_result_id(const QueryArgs &a, int64_t q, f3 p, int32_t id, float d2) {
    int32_t leaf = -1;
    if (id >= 0 && id < a.n) {
        leaf = a.inv_prim[id];
        if (leaf < 0 || leaf >= a.n) { atomicOr(a.status, 16); leaf = -1; }
    }
    write_result<kTri>(a, q, p, leaf, id, d2);
}

// Squared distance from p to primitive `id` (original numbering) through its
// leaf; +inf if id or its leaf is out of range.
template <bool kTri>
__device__ __forceinline__ float prim_dist2(const QueryArgs &a, f3 p, int32_t id) {
    if (id < 0 || id >= a.n) return INFINITY;
    const int32_t leaf = a.inv_prim[id];
    if (leaf < 0 || leaf >= a.n) return INFINITY;
    if (kTri) {
        float w1, w2;
        return tri_closest(p, vload(a.verts, a.nv, a.leaf_faces[leaf]), vload(a.verts, a.nv, a.leaf_faces[a.n + leaf]),
                           vload(a.verts, a.nv, a.leaf_faces[2 * a.n + leaf]), w1, w2);
    }
    const f3 d = p - vload(a.verts, a.nv, id);
    return fdot(d, d);
}

// The starting best of query q from its hint: (d^2 bits, id), or `none`.
template <bool kTri>
__device__ __forceinline__ unsigned long long hint_best(const QueryArgs &a, int64_t q, f3 p, unsigned long long none) {
    if (!a.hint) return none;
    const int32_t h = a.coherent ? __hip_atomic_load(a.hint + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                 : a.hint[q];
    const float d2 = prim_dist2<kTri>(a, p, h);
    const unsigned long long c = pack_best(d2, h);
    return d2 < INFINITY && c < none ? c : none;
}

// Test of the single leaf of a one-primitive BVH (no records exist).
template <bool kTri>
__device__ __forceinline__ float single_leaf_dist2(const QueryArgs &a, f3 p) {
    if (kTri) {
        float w1, w2;
        return tri_closest(p, vload(a.verts, a.nv, a.leaf_faces[0]), vload(a.verts, a.nv, a.leaf_faces[a.n]),
                           vload(a.verts, a.nv, a.leaf_faces[2 * a.n]), w1, w2);
    }
    const f3 d = p - vload(a.verts, a.nv, a.prim[0]);
    return fdot(d, d);
}

// --------------------------------------------------------------- batch kernel
// The waves of a workgroup each process batches of M queries with an LDS work
// stack shared by the batch's queries; each round pops up to 32 nodes (a lane per
// child; 64 with a lane per node on points).  A wave whose stack is deep puts its top 64 entries into the
// workgroup's one-chunk mailbox whenever it is empty, and a wave that has
// finished a batch empties the mailbox before it starts another, so a batch
// holding an expensive query (one nearly equidistant from many faces) is
// finished by several waves.  The per-query bests (d^2 bits, original id) stay
// with the owning wave and are lowered by LDS atomics from whichever wave tests
// a face; the owner writes its results once every chunk it gave away is done.

constexpr int kDonateMin = 128;          // a wave keeps at least 64 entries after giving 64
constexpr int kIdleSpinLimit = 1 << 22;  // bounded waits: error word instead of a hang

// A stack entry: high word, the node's lower bound with its low five bits
// replaced by the query's slot in the batch (rounding the bound down, so it
// stays a bound); low word, the node.  A waiting leaf: its parent's high word,
// and 2 x the parent node + the child slot that holds it.  The stack grows from
// the front of e, the waiting leaves from its end.
typedef unsigned long long StackEntry;
constexpr uint32_t kSlotMask = 31u;
__device__ __forceinline__ StackEntry make_entry(float bound, uint32_t slot, uint32_t node) {
    return (static_cast<StackEntry>((__float_as_uint(bound) & ~kSlotMask) | slot) << 32) | node;
}

template <bool kTri, int M, int K>
struct WaveStack {
    static constexpr int kCap = batch_cap(kTri, M), kAlloc = batch_alloc(kTri, M);
    static_assert(M <= kSlotMask + 1, "an entry holds its query's slot in five bits");
    StackEntry e[kAlloc];
    float4 q[M];                        // per query of the batch: the point, and prune_bound of its best
    unsigned long long best[M][K];      // the nearest faces, sorted: (d^2 bits, original id)
    uint32_t code[M];                   // where the best face lies (a record slot); only a guess, see finish_query
};

struct WaveMail {
    StackEntry e[64];
    int32_t count;                      // entries in the chunk
    int32_t owner;                      // wave whose batch the entries belong to
    int32_t state;                      // 0 empty, 1 full, 2 being taken, 3 being filled
    int32_t done;                       // waves that have finished all their batches
    int32_t outstanding[kBatchWaves];   // chunks of each wave's batch held elsewhere
};

template <bool kTri, int M, int K = 1>
struct BatchLds {
    WaveStack<kTri, M, K> st[kBatchWaves];
    WaveMail mail;
};

struct BatchStats {
    unsigned long long exp = 0, lbox = 0, lex = 0, nq = 0;
};

__device__ __forceinline__ int lds_load(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_store(int32_t *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int lds_add(int32_t *p, int v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ bool lds_cas(int32_t *p, int expect, int v) {
    return __hip_atomic_compare_exchange_strong(p, &expect, v, __ATOMIC_ACQ_REL, __ATOMIC_ACQUIRE,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Lane 0's value as a wave-uniform (scalar) one.  The mailbox decisions, the
// chunk's owner and size, the stack depth and the wait conditions are the same
// in every lane; reading them through readfirstlane makes the branches on them
// scalar, so the compiler never treats the regions that use ballots and
// shuffles as divergent (with the decisions taken per lane through a
// shuffle, batches after a wave's first returned faces that were not the
// nearest).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Set bits of a ballot below this lane.
__device__ __forceinline__ int rank_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// The lanes of a wave hand stack entries to each other through LDS (a lane
// pops what another lane pushed, copied or donated).  The hardware keeps a
// wave's LDS operations in order, but the compiler only orders each lane's own
// accesses, and a lane's load of another lane's slot may be moved above the
// store that fills it; this fence keeps every LDS access of the wave on its
// side.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Puts `cand` into a query's k nearest, sorted by (d^2, id): each place keeps the
// smaller of its own and the one coming in and hands the larger on, so lanes and
// waves may insert at once and every element but the dropped ones stays; a face
// tested twice meets itself and stops.
template <int K>
__device__ __forceinline__ void insert_nearest(unsigned long long *best, int k, unsigned long long cand) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (j >= k) break;
        const unsigned long long old = atomicMin(best + j, cand);
        if (old == cand) break;
        if (old > cand) cand = old;
    }
}

// Lowers the prune bounds of wave `O`'s M queries to their k-th nearest.
template <bool kTri, int M, int K>
__device__ __forceinline__ void lower_bounds(WaveStack<kTri, M, K> &O, int k, int lane) {
    wave_sync();                              // the insertions of every lane
    if (lane < M) {
        const float4 q = O.q[lane];
        const float d2 = __uint_as_float(static_cast<uint32_t>(O.best[lane][k - 1] >> 32));
        atomicMin(reinterpret_cast<uint32_t *>(&O.q[lane].w),
                  __float_as_uint(prune_bound(d2, qnorm1(f3{q.x, q.y, q.z}))));
    }
}

// Exact tests of the last `cnt` (<= 64) of wave `self`'s lc waiting leaves, one
// per lane.  A face at most as far as its query's best lowers the best and the
// prune bound (both by LDS atomics: other waves may hold chunks of the batch).
template <bool kTri, int M, int K>
__device__ __forceinline__ int test_leaves(const QueryArgs &a, WaveStack<kTri, M, K> &S, WaveStack<kTri, M, K> &O, int lc, int cnt,
                                           BatchStats &stats) {
    const int lane = threadIdx.x % 64;
    bool act = lane < cnt;
    const StackEntry en = S.e[S.kAlloc - lc + (act ? lane : 0)];
    const uint32_t hi = static_cast<uint32_t>(en >> 32), code = static_cast<uint32_t>(en), slot = hi & kSlotMask;
    const float4 q = O.q[slot];
    act = act && __uint_as_float(hi & ~kSlotMask) <= q.w;   // its parent may have fallen behind by now
    if (a.counters) stats.lex += __popcll(__ballot(act));
    if (act) {
        const float4 *rec = a.nodes + 3 * static_cast<uint64_t>(code);
        const f3 p = f3{q.x, q.y, q.z};
        const float4 f0 = rec[0], f1 = rec[1], f2 = kTri ? rec[2] : f1;
        const float d2 = leaf_dist2<kTri>(p, f0, f1, f2);
        if (d2 <= q.w) {
            const unsigned long long cand = pack_best(d2, __float_as_int(f1.w));
            if (K > 1) {
                insert_nearest<K>(O.best[slot], a.k, cand);
            } else if (cand < atomicMin(&O.best[slot][0], cand)) {
                atomicMin(reinterpret_cast<uint32_t *>(&O.q[slot].w), __float_as_uint(prune_bound(d2, qnorm1(p))));
                O.code[slot] = code;
            }
        }
    }
    if (K > 1) lower_bounds<kTri, M, K>(O, a.k, lane);
    return lc - cnt;
}

// A round over a point BVH: up to 64 nodes, one per lane with both children.  A
// leaf's box is its point, so its bound is its exact squared distance and the
// round settles it; with a box test this cheap, a child per lane only doubles
// the rest of the round (100,000 nearest points of 100,000: 75-87 -> 54-70 us).
template <int M, int K>
__device__ __forceinline__ void point_round(const QueryArgs &a, WaveStack<false, M, K> &S, WaveStack<false, M, K> &O, uint32_t n_nodes,
                                            int take, int &sp, BatchStats &stats) {
    const int lane = threadIdx.x % 64;
    const bool pop = lane < take;
    const StackEntry en = S.e[pop ? sp - 1 - lane : 0];
    sp -= take;
    const uint32_t hi = static_cast<uint32_t>(en >> 32), node = static_cast<uint32_t>(en), slot = hi & kSlotMask;
    const float4 q = O.q[slot];
    const f3 p = f3{q.x, q.y, q.z};
    const bool act = pop && node < n_nodes && __uint_as_float(hi & ~kSlotMask) <= q.w;
    float4 l0{}, l1{}, r0{}, r1{};
    if (act) {
        const float4 *rec = a.nodes + 6 * static_cast<uint64_t>(node);
        l0 = rec[0]; l1 = rec[1]; r0 = rec[3]; r1 = rec[4];
    }
    const int32_t lref = __float_as_int(l0.w), rref = __float_as_int(r0.w);
    const float dl = child_bound<false>(p, 0.0f, l0, l1, l1), dr = child_bound<false>(p, 0.0f, r0, r1, r1);
    const bool il = act && dl <= q.w, ir = act && dr <= q.w;
    const bool pl = il && lref >= 0, pr = ir && rref >= 0;
    unsigned long long cand = ~0ull;
    if (il && lref < 0) cand = pack_best(dl, __float_as_int(l1.w));
    if (ir && rref < 0) {
        const unsigned long long c = pack_best(dr, __float_as_int(r1.w));
        if (c < cand) cand = c;
    }
    if (cand != ~0ull && cand < atomicMin(&O.best[slot][0], cand))
        atomicMin(reinterpret_cast<uint32_t *>(&O.q[slot].w),
                  __float_as_uint(prune_bound(__uint_as_float(static_cast<uint32_t>(cand >> 32)), qnorm1(p))));
    const uint64_t bl = __ballot(pl), br = __ballot(pr);
    if (a.counters) {
        stats.exp += __popcll(__ballot(act));
        stats.lbox += __popcll(__ballot(act && lref < 0)) + __popcll(__ballot(act && rref < 0));
        stats.lex += __popcll(__ballot(il && lref < 0)) + __popcll(__ballot(ir && rref < 0));
    }
    if (pl || pr) {                           // nearer child on top of the stack
        const int off = sp + rank_below(bl) + rank_below(br);
        const bool left_near = dl <= dr, first_left = pl && !(pr && left_near);
        S.e[off] = make_entry(first_left ? dl : dr, slot, static_cast<uint32_t>(first_left ? lref : rref));
        if (pl && pr)
            S.e[off + 1] = make_entry(left_near ? dl : dr, slot, static_cast<uint32_t>(left_near ? lref : rref));
    }
    sp += __popcll(bl) + __popcll(br);
}

// Rounds over wave `self`'s stack (sp entries, and lc waiting leaves) until it is
// empty.  Entries belong to the batch of wave `owner`: its query points and bests.
//
// A round pops up to 32 nodes and gives each child to a lane of its own.  Every
// lane bounds its child without a branch; internal children that survive are
// pushed, the nearer of a pair on top, and leaf children are queued.  Queued
// leaves are tested exactly together, once 32 wait or the stack runs low: tested
// inside the round they left most lanes idle (18 of 64 needed an exact test, in
// two divergent passes, and 26 a bound test of the leaf's box, with two children
// to a lane); with 64 waiting, cold queries' bests came late (299 nodes a query
// instead of 283 on 1,000,000 faces).  Waiting leaves are not tested against
// their box, which costs about what it drops.  A child to a lane halves what a
// lone wave issues in a round, its cost on small launches.
//
// 50,000 hinted queries on 40,000 faces (batches of 16): 117 -> 62 us with the
// joint bound of child_bound, 55% of the time issuing VALU; 1M on 500,000 faces:
// 5,980 -> 1,340 us, 80% issuing and 6.6 TB/s of cache-line misses.
template <bool kTri, int M, int K>
__device__ void run_stack(const QueryArgs &a, BatchLds<kTri, M, K> &L, int self, int owner, int sp, int lc,
                          BatchStats &stats) {
    const int lane = threadIdx.x % 64;
    const uint32_t n_nodes = static_cast<uint32_t>(a.n - 1), odd = lane & 1;
    WaveStack<kTri, M, K> &S = L.st[self];
    WaveStack<kTri, M, K> &O = L.st[owner];
    WaveMail &mail = L.mail;
    // the stack never exceeds kCap + 62: it starts with at most kCap entries (a
    // chunk of 64, or what start_batch leaves), a round of width k pushes at most
    // 2k entries (nodes and leaves together), widths are cut to half the room
    // left, the leaves are tested whenever room runs out, and width-1 rounds are
    // a plain depth-first walk whose growth is bounded by the tree depth; each
    // query expands each internal node at most once, so the round cap only stops
    // a corrupted buffer from looping
    const int64_t max_rounds = 2 * static_cast<int64_t>(M + 1) * a.n + 64;
    for (int64_t round = 0; sp + lc > 0 && round < max_rounds; ++round) {
        wave_sync();                          // the previous round's pushes, or the entries handed in
        if (lc >= kLeafWait || (lc > 0 && (sp < kLeafNarrow || sp + lc > S.kCap - 2 * kPopNodes))) {
            lc = test_leaves<kTri, M, K>(a, S, O, lc, lc < 64 ? lc : 64, stats);
            wave_sync();
            if (sp == 0) continue;
        }
        if (sp >= kDonateMin) {
            int give = 0;
            if (lane == 0 && lds_load(&mail.state) == 0 && lds_cas(&mail.state, 0, 3)) give = 1;
            if (uniform(give)) {
                mail.e[lane] = S.e[sp - 64 + lane];
                wave_sync();
                sp -= 64;
                if (lane == 0) {
                    mail.owner = owner;
                    mail.count = 64;
                    lds_add(&mail.outstanding[owner], 1);
                    lds_store(&mail.state, 1);
                }
            }
        }
        constexpr int kPop = kTri ? kPopNodes : 2 * kPopNodes;
        int take = sp < kPop ? sp : kPop;
        const int room = (S.kCap - sp - lc) / 2;
        if (take > room) take = room > 1 ? room : 1;
        if (sp + lc + take > S.kAlloc) {   // past the bound of a valid tree
            if (lane == 0) atomicOr(a.status, 64);
            break;
        }
        if constexpr (!kTri) {
            point_round<M, K>(a, S, O, n_nodes, take, sp, stats);
            continue;
        }
        const bool pop = lane < 2 * take;
        const StackEntry en = S.e[pop ? sp - 1 - (lane >> 1) : 0];
        sp -= take;
        const uint32_t hi = static_cast<uint32_t>(en >> 32), node = static_cast<uint32_t>(en), slot = hi & kSlotMask;
        const float4 q = O.q[slot];
        const f3 qp = f3{q.x, q.y, q.z};
        const bool act = pop && node < n_nodes && __uint_as_float(hi & ~kSlotMask) <= q.w;
        float4 c0{}, c1{}, c2{};
        if (act) {
            const float4 *rec = a.nodes + 6 * static_cast<uint64_t>(node) + 3 * odd;
            c0 = rec[0]; c1 = rec[1];
            if (kTri) c2 = rec[2];
        }
        const int32_t ref = __float_as_int(c0.w);
        const float d = child_bound<kTri>(qp, 0x1p-20f * qnorm1(qp), c0, c1, c2);
        const bool push = act && ref >= 0 && d <= q.w, leaf = act && ref < 0;
        const uint64_t pm = __ballot(push), lm = __ballot(leaf);
        if (a.counters) {
            stats.exp += __popcll(__ballot(act)) / 2;
            stats.lbox += __popcll(lm);
        }
        // the other child's bound (infinite unless it is pushed too) decides which is on top
        const float mine = push ? d : INFINITY;
        const float other = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(mine), 0xb1, 0xf, 0xf, true));
        const float even = odd ? other : mine, far = odd ? mine : other;
        int pos = sp + rank_below(pm);
        if (even <= far && far < INFINITY) pos += odd ? -1 : 1;      // the even lane's child is the nearer: swap
        if (leaf) pos = S.kAlloc - 1 - lc - rank_below(lm);
        if (push || leaf)
            S.e[pos] = leaf ? (static_cast<StackEntry>(hi) << 32) | (2 * node + odd)
                            : make_entry(d, slot, static_cast<uint32_t>(ref));
        sp += __popcll(pm);
        lc += __popcll(lm);
    }
    wave_sync();                              // the last round's bests, before any lane reads them
}

// Takes the mailbox's chunk, if there is one, onto wave `self`'s (empty) stack:
// its size, and the wave whose batch it belongs to; -1 if there is none.
template <bool kTri, int M, int K>
__device__ __forceinline__ int take_chunk(const QueryArgs &a, BatchLds<kTri, M, K> &L, int self, int &owner) {
    const int lane = threadIdx.x % 64;
    WaveMail &mail = L.mail;
    int got = 0;
    if (lane == 0 && lds_load(&mail.state) == 1 && lds_cas(&mail.state, 1, 2)) got = 1;
    if (!uniform(got)) return -1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    owner = uniform(mail.owner);
    int n = uniform(mail.count);
    if (owner < 0 || owner >= kBatchWaves || n < 0 || n > 64) {
        if (lane == 0) atomicOr(a.status, 16);
        owner = -1;
        n = 0;
    }
    if (lane < n) L.st[self].e[lane] = mail.e[lane];
    wave_sync();
    if (lane == 0) lds_store(&mail.state, 0);
    return n;
}

// The record slot of primitive `id` (original numbering), or -1 if it or its
// leaf is out of range (n > 1).
__device__ __forceinline__ int64_t slot_of(const QueryArgs &a, int32_t id) {
    if (id < 0 || id >= a.n) return -1;
    const int32_t leaf = a.inv_prim[id];
    if (leaf < 0 || leaf >= a.n) return -1;
    const int32_t code = a.leaf_parent[leaf];
    return code >= 0 && (code >> 1) < a.n - 1 ? code : -1;
}

// Squared distance from p to the leaf in record slot `code`, and its id.
template <bool kTri>
__device__ __forceinline__ float slot_dist2(const QueryArgs &a, f3 p, int64_t code, int32_t &id) {
    const float4 *rec = a.nodes + 3 * code;
    const float4 f1 = rec[1];
    id = __float_as_int(f1.w);
    return kTri ? leaf_dist2<kTri>(p, rec[0], f1, rec[2]) : leaf_dist2<kTri>(p, f1, f1, f1);
}

// Another lane's value within each four lanes (mask 1, 2 or 3: the lane's
// number in its four, xor mask).
template <int kMask>
__device__ __forceinline__ uint32_t quad_xor(uint32_t v) {
    constexpr int kPerm = kMask == 1 ? 0xb1 : kMask == 2 ? 0x4e : 0x1b;
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), kPerm, 0xf, 0xf, true));
}
template <int kMask>
__device__ __forceinline__ unsigned long long quad_xor64(unsigned long long v) {
    return (static_cast<unsigned long long>(quad_xor<kMask>(static_cast<uint32_t>(v >> 32))) << 32) |
           quad_xor<kMask>(static_cast<uint32_t>(v));
}

// The seed descent of the batch's queries that `need` one: a walk from the root
// to the leaves that keeps the kLanes / 2 nearest nodes of a level, each query
// in kLanes (2 or 4) lanes, a child to a lane.  Returns, in every lane of the
// query, the nearest of the leaves met on the way (the nearest by its box in
// each lane), and its record slot in `code`.  With one node kept, both children
// in a lane and every leaf on the way tested, 20,002 cold queries on 46,000 faces
// took 58 us; in this form 41 us, and 39 us with kKeep (40 nodes each in all).
//
// kKeep: the children that the walk passes by go to the stack (K.nodes entries)
// and the leaves it meets to the waiting leaves (K.leaves), with their bounds, so
// that the rounds go on from them instead of walking from the root again.
struct Kept {
    StackEntry *e;
    int cap, alloc;                     // entries that may be kept, and the stack's
    int nodes, leaves;
    bool full;                          // they did not fit, or the walk ended early: start from the root
};

template <bool kTri, int kLanes, bool kKeep>
__device__ __forceinline__ unsigned long long seed_descent(const QueryArgs &a, f3 p, bool need, uint32_t &code, Kept &K,
                                                           BatchStats &stats) {
    const uint32_t lane = threadIdx.x % 64, odd = lane & 1, pair = (lane >> 1) & (kLanes / 2 - 1);
    const uint32_t n_nodes = static_cast<uint32_t>(a.n - 1), slot = lane / kLanes;
    const float dq = slab_query_margin(p);
    uint32_t node = need && pair == 0 ? 0u : ~0u;
    float leaf_key = INFINITY;
    uint32_t leaf_code = ~0u;
    for (int lvl = 0; lvl < 64; ++lvl) {
        const bool act = node < n_nodes;
        if (!__ballot(act)) break;
        uint32_t key = ~0u, ref = ~0u;
        float bound = 0.0f;
        bool leaf = false;
        if (act) {
            const float4 *rec = a.nodes + 6 * static_cast<uint64_t>(node) + 3 * odd;
            const float4 c0 = rec[0], c1 = rec[1], c2 = kTri ? rec[2] : c1;
            const uint32_t r = static_cast<uint32_t>(__float_as_int(c0.w));
            if (static_cast<int32_t>(r) < 0) {
                leaf = true;
                bound = leaf_box_dist2<kTri>(p, c0, c1, c2);
                if (bound <= leaf_key) {
                    leaf_key = bound;
                    leaf_code = 2 * node + odd;
                }
            } else {
                bound = child_bound<kTri>(p, dq, c0, c1, c2);
                key = __float_as_uint(bound);
                ref = r;
            }
        }
        const uint32_t here = 2 * node + odd;
        if (a.counters) {
            stats.exp += __popcll(__ballot(act)) / 2;
            stats.lbox += __popcll(__ballot(leaf));
        }
        // unique keys within the query's lanes, absent children last
        key = (key & ~3u) | (lane & 3);
        if (kLanes == 2) {
            static_assert(!kKeep || kLanes == 4, "kept with two nodes a level");
            const uint32_t other = quad_xor<1>(key), other_ref = quad_xor<1>(ref);
            node = other < key ? other_ref : ref;
        } else {
            const uint32_t k1 = quad_xor<1>(key), k2 = quad_xor<2>(key), k3 = quad_xor<3>(key);
            const uint32_t rank = (k1 < key) + (k2 < key) + (k3 < key);
            // the nodes of the two lowest ranks, handed to the two pairs (0: none)
            uint32_t x = rank == 0 ? ref + 1 : 0u, y = rank == 1 ? ref + 1 : 0u;
            x |= quad_xor<1>(x);
            y |= quad_xor<1>(y);
            x |= quad_xor<2>(x);
            y |= quad_xor<2>(y);
            node = (pair ? y : x) - 1;
            if (kKeep) {
                const bool by = ref != ~0u && rank >= 2;
                const uint64_t bm = __ballot(by), lm = __ballot(leaf);
                K.full = K.full || K.nodes + K.leaves + __popcll(bm) + __popcll(lm) > K.cap;
                if (!K.full) {
                    if (by) K.e[K.nodes + rank_below(bm)] = make_entry(bound, slot, ref);
                    if (leaf) K.e[K.alloc - 1 - K.leaves - rank_below(lm)] = make_entry(bound, slot, here);
                    K.nodes += __popcll(bm);
                    K.leaves += __popcll(lm);
                }
            }
        }
    }
    if (kKeep && __ballot(node < n_nodes)) K.full = true;     // deeper than the walk: nothing kept below its last level
    unsigned long long best = ~0ull;
    if (a.counters && !kKeep) stats.lex += __popcll(__ballot(leaf_code != ~0u));   // kept leaves count when the rounds test them
    if (leaf_code != ~0u) {
        int32_t id;
        const float d2 = slot_dist2<kTri>(a, p, leaf_code, id);
        best = pack_best(d2, id);
    }
    code = leaf_code;
    unsigned long long o = quad_xor64<1>(best);
    uint32_t oc = quad_xor<1>(code);
    if (o < best) { best = o; code = oc; }
    if (kLanes == 4) {
        o = quad_xor64<2>(best);
        oc = quad_xor<2>(code);
        if (o < best) { best = o; code = oc; }
    }
    return best;
}

// Starts a wave's batch [qb, qb + nb): points, starting bests (a hint's
// distance, else the seed descent's, else max_dist2) and, on the stack, the root
// or what the descent passed by.  Returns the stack's size, and the number of
// waiting leaves in lc: at most kCap together (run_stack's bound rests on it), so a
// descent leaves room for the roots of the batch's hinted queries.
//
// Going on from the descents' paths took 50,000 cold queries on 40,000 faces from
// 98 to 81 us, 20,002 on 46,000 faces from 43 to 39.
template <bool kTri, int M, int K>
__device__ __forceinline__ int start_batch(const QueryArgs &a, WaveStack<kTri, M, K> &S, int64_t qb, int nb, int &lc,
                                           BatchStats &stats) {
    // Lanes of a query.  On points a second node a level is not worth its lanes: their
    // bounds are exact at the leaves and the walk is not kept (300,000 cold queries on 1M
    // points: 265 us with four lanes, 218 with two; 10,000 on 5,000: 22.3, 21.0).
    constexpr int kLanes = kTri && M <= 16 ? 4 : 2;
    constexpr bool kKeep = kTri && M <= 16;
    Kept kept{S.e, S.kCap, S.kAlloc, 0, 0, false};
    bool walked = false;                          // this lane's query was in the descent
    const int lane = threadIdx.x % 64, i = lane / kLanes;
    const unsigned long long none = pack_best(a.maxd2, INT_MAX);
    const int64_t qid = i < nb ? query_at(a, qb + i) : -1;
    const bool own = qid >= 0, lead = own && lane % kLanes == 0;
    f3 p = f3{0.0f, 0.0f, 0.0f};
    if (own) p = load3(a.queries, a.nq, qid);
    unsigned long long best = none;
    uint32_t code = ~0u;
    float pb = 0.0f;
    bool push = false;
    float rd = 0.0f;
    if (a.n == 1) {
        if (lead) {
            const unsigned long long c = pack_best(single_leaf_dist2<kTri>(a, p), a.prim[0]);
            if (c < none) best = c;
        }
    } else if (K > 1 && a.n > 1) {
        // the seed descent's leaf and its neighbours along the leaf order: k faces,
        // so the farthest bounds the k-th nearest from the start
        if (lead)
#pragma unroll
            for (int j = 0; j < K; ++j) S.best[i][j] = none;
        wave_sync();
        uint32_t at;
        (void)seed_descent<kTri, kLanes, kKeep>(a, p, own, at, kept, stats);
        walked = own;
        if (own && at < 2 * static_cast<uint32_t>(a.n - 1)) {
            const int64_t leaf = ~static_cast<int64_t>(__float_as_int(a.nodes[3 * static_cast<uint64_t>(at)].w));
            int64_t first = leaf - K / 2 < a.n - K ? leaf - K / 2 : a.n - K;
            if (first < 0) first = 0;
#pragma unroll
            for (int u = 0; u < (K + kLanes - 1) / kLanes; ++u) {
                const int64_t l = first + lane % kLanes + u * kLanes;
                if (l >= a.n || lane % kLanes + u * kLanes >= K) continue;
                const int32_t code_l = a.leaf_parent[l];
                if (code_l < 0 || (code_l >> 1) >= a.n - 1) continue;
                int32_t id;
                const float d2 = slot_dist2<kTri>(a, p, code_l, id);
                insert_nearest<K>(S.best[i], a.k, pack_best(d2, id));
            }
        }
        wave_sync();
        rd = box_dist2(p, f3{a.root[0], a.root[1], a.root[2]}, f3{a.root[4], a.root[5], a.root[6]});
        if (own) pb = prune_bound(__uint_as_float(static_cast<uint32_t>(S.best[i][a.k - 1] >> 32)), qnorm1(p));
        push = lead && rd <= pb;
    } else if (a.n > 1) {
        // a hinted primitive's distance starts the query; without one, the seed descent
        bool hinted = false;
        if (a.hint) {
            if (own) {
                const int32_t h = a.coherent ? __hip_atomic_load(a.hint + qid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                             : a.hint[qid];
                const int64_t at = slot_of(a, h);
                if (at >= 0) {
                    int32_t id;
                    const float d2 = slot_dist2<kTri>(a, p, at, id);
                    const unsigned long long c = pack_best(d2, id);
                    if (id == h && d2 < INFINITY && c < none) {
                        best = c;
                        code = static_cast<uint32_t>(at);
                        hinted = true;
                    }
                }
            }
        }
        rd = box_dist2(p, f3{a.root[0], a.root[1], a.root[2]}, f3{a.root[4], a.root[5], a.root[6]});
        // Also without `seed`, unless max_dist2 ends the query at the root: a round's leaves
        // wait, so a query with no face to start from prunes nothing for many rounds (65,536
        // queries on 40,000 faces, batches of 4: 760 us, with the walk 152, leaves tested at
        // once 665; 10,000 on 100,000 points, batches of 8: 595, 25).
        const bool need = own && !hinted && (a.seed || rd <= prune_bound(a.maxd2, qnorm1(p)));
        if (__ballot(need)) {
            uint32_t at;
            kept.cap -= __popcll(__ballot(lead && !need));   // the other queries' roots go on top
            const unsigned long long c = seed_descent<kTri, kLanes, kKeep>(a, p, need, at, kept, stats);
            walked = need;
            if (need && c < best) {
                best = c;
                code = at;
            }
        }
        pb = prune_bound(best < none ? __uint_as_float(static_cast<uint32_t>(best >> 32)) : a.maxd2, qnorm1(p));
        push = lead && rd <= pb;
    }
    if (lead) {
        S.q[i] = make_float4(p.x, p.y, p.z, pb);
        if (K == 1 || a.n <= 1) S.best[i][0] = best;
        if (a.n <= 1)
#pragma unroll
            for (int j = 1; j < K; ++j) S.best[i][j] = none;
        S.code[i] = code;
    }
    int sp = 0;
    lc = 0;
    if (kKeep && !kept.full) {
        // of what the descent passed by, the entries that the starting bests leave
        wave_sync();
        for (int at = 0; at < kept.nodes; at += 64) {
            const StackEntry en = S.e[at + lane < kept.nodes ? at + lane : 0];
            const uint32_t hi = static_cast<uint32_t>(en >> 32);
            const bool keep = at + lane < kept.nodes && __uint_as_float(hi & ~kSlotMask) <= S.q[hi & kSlotMask].w;
            const uint64_t km = __ballot(keep);
            wave_sync();                          // read before any lane writes
            if (keep) S.e[sp + rank_below(km)] = en;
            sp += __popcll(km);
        }
        for (int at = 0; at < kept.leaves; at += 64) {
            const StackEntry en = S.e[S.kAlloc - 1 - (at + lane < kept.leaves ? at + lane : 0)];
            const uint32_t hi = static_cast<uint32_t>(en >> 32);
            const bool keep = at + lane < kept.leaves && __uint_as_float(hi & ~kSlotMask) <= S.q[hi & kSlotMask].w &&
                              (K > 1 || static_cast<uint32_t>(en) != S.code[hi & kSlotMask]);   // not the start itself
            const uint64_t km = __ballot(keep);
            wave_sync();
            if (keep) S.e[S.kAlloc - 1 - lc - rank_below(km)] = en;
            lc += __popcll(km);
        }
        push = push && !walked;
    }
    const uint64_t bm = __ballot(push);
    if (push) S.e[sp + rank_below(bm)] = make_entry(rd, static_cast<uint32_t>(i), 0u);
    return sp + __popcll(bm);
}

// Final record of the query in slot `lane` of the batch, its index qid: the
// face's triangle is read again from its record slot.  The slot noted beside
// the best may be another face's (two waves lowering one best race on it), so
// its id is checked, and the face's slot is looked up where they differ.
template <bool kTri, int M>
__device__ __forceinline__ void finish_query(const QueryArgs &a, const WaveStack<kTri, M, 1> &S, int lane, int64_t qid) {
    const unsigned long long b = S.best[lane][0];
    const float4 q = S.q[lane];
    const f3 p = f3{q.x, q.y, q.z};
    const int32_t id = static_cast<int32_t>(b & 0xffffffffull);
    const float d2 = __uint_as_float(static_cast<uint32_t>(b >> 32));
    if (!kTri || a.n == 1 || id < 0 || id >= a.n) {
        write_result_id<kTri>(a, qid, p, id, d2);
        return;
    }
    int64_t code = S.code[lane];
    if (code >= 2 * (a.n - 1)) code = slot_of(a, id);
    float4 f0{}, f1{}, f2{};
    if (code >= 0) {
        const float4 *rec = a.nodes + 3 * code;
        f0 = rec[0]; f1 = rec[1]; f2 = rec[2];
        if (__float_as_int(f1.w) != id) {
            code = slot_of(a, id);
            if (code >= 0) {
                rec = a.nodes + 3 * code;
                f0 = rec[0]; f1 = rec[1]; f2 = rec[2];
            }
        }
    }
    if (code < 0) {
        atomicOr(a.status, 16);
        write_none(a, qid, p);
        return;
    }
    write_face(a, qid, p, id, xyz(f0), xyz(f1), xyz(f2));
}

// Final records of a batch of the k-nearest form, a lane per query and place:
// the faces and distances, and the closest points combined with
// inverse-distance weights 1 / (d + eps) (the weighted nearest-neighbour
// NearestSurface of Sec. 3.3); a face at distance 0 gives its own point.
template <int M, int K>
__device__ __forceinline__ void finish_nearest(const QueryArgs &a, const WaveStack<true, M, K> &S, int64_t qb, int nb) {
    static_assert(M * K <= 64, "a lane per query and place");
    const int lane = threadIdx.x % 64, i = lane / K < M ? lane / K : 0, j = lane % K;
    const bool own = lane < M * K && i < nb;
    const int64_t qid = own ? query_at(a, qb + i) : -1;
    const float4 q = S.q[i];
    const f3 p = f3{q.x, q.y, q.z};
    const unsigned long long b = S.best[i][j];
    const int32_t id = static_cast<int32_t>(b & 0xffffffffull);
    bool ok = qid >= 0 && j < a.k && id >= 0 && id < a.n;
    f3 c = f3{0.0f, 0.0f, 0.0f};
    float d2 = 0.0f;
    if (ok) {
        f3 A = c, B = c, C = c;
        if (a.n == 1) {
            A = vload(a.verts, a.nv, a.leaf_faces[0]);
            B = vload(a.verts, a.nv, a.leaf_faces[1]);
            C = vload(a.verts, a.nv, a.leaf_faces[2]);
        } else {
            const int64_t code = slot_of(a, id);
            ok = code >= 0;
            if (ok) {
                const float4 *rec = a.nodes + 3 * code;
                A = xyz(rec[0]); B = xyz(rec[1]); C = xyz(rec[2]);
            } else {
                atomicOr(a.status, 16);
            }
        }
        float w1, w2;
        d2 = tri_closest(p, A, B, C, w1, w2);
        c = tri_point(A, B, C, w1, w2);
    }
    if (qid >= 0 && j < a.k) {
        a.face[j * a.nq + qid] = ok ? id : -1;
        if (a.dist2) a.dist2[j * a.nq + qid] = ok ? __uint_as_float(static_cast<uint32_t>(b >> 32)) : INFINITY;
    }
    if (!a.point) return;
    const float w = 1.0f / (sqrtf(d2) + a.eps);
    f3 num = f3{0.0f, 0.0f, 0.0f}, on = p;
    float den = 0.0f;
    bool hit = false;                         // a face at distance 0: its point, unweighted
#pragma unroll
    for (int u = 0; u < K; ++u) {             // in the order of the places, in every lane of the query
        const int from = lane - j + u;
        const f3 cu = f3{__shfl(c.x, from), __shfl(c.y, from), __shfl(c.z, from)};
        const float wu = __shfl(w, from), d2u = __shfl(d2, from);
        if (__shfl(static_cast<int>(ok), from)) {
            if (d2u == 0.0f && !hit) {
                hit = true;
                on = cu;
            }
            num = num + wu * cu;
            den += wu;
        }
    }
    if (qid >= 0 && j == 0) store3(a.point, a.nq, qid, hit ? on : (den > 0.0f ? (1.0f / den) * num : p));
}

// The workgroup's kBatchWaves waves process the query batches [qb, qb + M)
// below q_end (positions in the processing order): wave w takes qb = start +
// w M, then steps by stride or, with a queue, M times the batch numbers it
// takes from the queue.  Every wave of the workgroup calls this.  A wave whose
// batch waits for chunks it gave away, or that has no batch left, empties the
// mailbox; kHelpBetween: also before it starts its next batch.  The batched
// persistent kernel leaves that out: there an earlier form of this loop with it
// returned faces that were not the nearest for queries of later batches, while
// every other form, and the plain kernels with it, matched the all-faces kernel
// exactly.  Each turn of the loop runs one stack, the wave's own or a chunk, so
// the rounds are compiled once.
template <bool kTri, int M, bool kHelpBetween = true, int K = 1>
__device__ void batch_loop(const QueryArgs &a, int64_t start, int64_t stride, int64_t q_end, BatchLds<kTri, M, K> &L) {
    const int lane = threadIdx.x % 64;
    const int self = uniform(static_cast<int>(threadIdx.x / 64));
    WaveStack<kTri, M, K> &S = L.st[self];
    WaveMail &mail = L.mail;
    BatchStats stats;
    if (threadIdx.x == 0) {
        mail.state = 0;
        mail.done = 0;
        for (int w = 0; w < kBatchWaves; ++w) mail.outstanding[w] = 0;
    }
    __syncthreads();

    auto next = [&](int64_t qb) -> int64_t {
        if (!a.queue) return qb + stride;
        uint32_t b = 0;
        if (lane == 0) b = atomicAdd(a.queue, 1u);
        return static_cast<int64_t>(static_cast<uint32_t>(uniform(static_cast<int>(b)))) * M;
    };
    int64_t qb = a.queue ? next(0) : start + static_cast<int64_t>(self) * M;
    bool open = false;                        // batch qb is started and its results not yet written
    bool between = false;                     // a batch was written: chunks go before the next
    bool told = false;                        // this wave's last batch is counted in mail.done
    for (int spin = 0;;) {
        int owner = -1, sp = -1, lc = 0;
        if (open || between || qb >= q_end) sp = take_chunk<kTri, M, K>(a, L, self, owner);
        const int nb = static_cast<int>(q_end - qb < M ? q_end - qb : M);
        if (sp < 0 && !open && qb < q_end) {
            sp = start_batch<kTri, M, K>(a, S, qb, nb, lc, stats);
            owner = self;
            open = true;
            between = false;
        } else if (sp >= 0) {
            owner = owner < 0 ? -1 : owner | kBatchWaves;      // a chunk: counted when done
        }
        if (sp >= 0) {
            spin = 0;
            if (sp + lc > 0) run_stack<kTri, M, K>(a, L, self, owner & (kBatchWaves - 1), sp, lc, stats);
            if (owner >= kBatchWaves && lane == 0) lds_add(&mail.outstanding[owner & (kBatchWaves - 1)], -1);
        }
        // chunks given away must be finished before the results are final
        if (open && uniform(lds_load(&mail.outstanding[self])) == 0) {
            const int64_t qid = lane < nb ? query_at(a, qb + lane) : -1;
            if constexpr (K > 1) finish_nearest<M, K>(a, S, qb, nb);
            else if (qid >= 0) finish_query<kTri, M>(a, S, lane, qid);
            if (a.counters) stats.nq += __popcll(__ballot(qid >= 0));
            open = false;
            between = kHelpBetween;
            qb = next(qb);
            continue;
        }
        if (open || qb < q_end) {
            if (sp >= 0) continue;
        } else {
            if (!told) {
                if (lane == 0) lds_add(&mail.done, 1);
                told = true;
            }
            if (uniform(lds_load(&mail.done)) == kBatchWaves) break;
            if (sp >= 0) continue;
        }
        if (++spin > kIdleSpinLimit) {
            if (lane == 0) atomicOr(a.status, 16);
            break;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    if (a.counters && lane == 0) add_counters(a, stats.exp, stats.lbox, stats.lex, stats.nq);
}

}  // namespace mgu
