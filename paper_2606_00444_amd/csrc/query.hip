// Closest point on a triangle mesh / nearest point of a point set through the
// LBVH, and an all-faces brute force for self-checks (gfx950).
//
// NearestSurface of the paper (Sec. 3.3, Eq. 1-2) projects a point onto a mesh
// with barycentric interpolation; it is read as the single nearest face.  The
// face normal is computed on demand from the three vertices of the winning
// face (Sec. 3.4 step 3), never stored.
//
// Pruning: a child is expanded when its lower bound is <= prune_bound(best)
// (traverse.hpp), a slack that keeps faces whose float32 distance ties the
// best, so ties go to the lowest original id (carried in the node record beside
// each leaf child) in every traversal.  Leaf children hold their triangle, so a
// leaf is tested with the data of the record that referenced it.
//
// Small sets on small trees are scanned (scan_kernel).  Otherwise, two traversals
// (chosen per call, see mg_query_options):
//  * lane:  one query per lane, depth-first, nearer child first; stack in LDS
//           for the first 32 entries and in a private array beyond (Karras trees
//           over 30-bit codes with index tie-break are at most 62 levels deep).
//  * batch: one wave owns M queries and a shared LDS stack of (lower bound,
//           query, node) entries; each round the wave pops up to 32 nodes, bounds
//           each child in a lane of its own, pushes the surviving nodes with
//           ballots and queues the leaves, which are tested exactly together.
//           A query's best is a 64-bit LDS atomic min over (float bits of d^2,
//           original id): non-negative floats order like their bit patterns, so
//           this is the lexicographic (d^2, id) minimum.  A query near the middle
//           of a closed surface has thousands of near-equidistant faces; here they
//           are expanded by the whole wave instead of one lane walking them serially.
#include "traverse.hpp"

#include <atomic>

namespace mgu {
namespace {

// ---------------------------------------------------------------- lane kernel
template <bool kTri, bool kBall>
__global__ __launch_bounds__(kLaneBlock) void traverse_lane_kernel(QueryArgs a) {
    __shared__ int32_t s_stack[kLdsStack][kLaneBlock];
    int32_t deep[kMaxStack - kLdsStack];
    const int lane = threadIdx.x;
    check_vertex_count(a);
    const int64_t pos = static_cast<int64_t>(blockIdx.x) * kLaneBlock + lane;
    if (pos >= a.nq) return;
    const int64_t q = query_at(a, pos);
    if (q < 0) return;
    const f3 p = load3(a.queries, a.nq, q);
    const float dq = slab_query_margin(p);
    float best = a.maxd2;
    int32_t best_id = INT_MAX, best_leaf = -1;
    unsigned long long n_exp = 0, n_lbox = 0, n_lex = 0;
    {
        const unsigned long long h = hint_best<kTri>(a, q, p, pack_best(a.maxd2, INT_MAX));
        if (h != pack_best(a.maxd2, INT_MAX)) {
            best = __uint_as_float(static_cast<uint32_t>(h >> 32));
            best_id = static_cast<int32_t>(h & 0xffffffffull);
            best_leaf = a.inv_prim[best_id];
        }
    }

    auto consider = [&](float d2, int32_t id, int32_t leaf) {
        ++n_lex;
        if (d2 < best || (d2 == best && id < best_id)) {
            best = d2;
            best_id = id;
            best_leaf = leaf;
        }
    };

    if (a.n == 1) {
        consider(single_leaf_dist2<kTri>(a, p), a.prim[0], 0);
    } else if (a.n > 1) {
        const f3 rlo = f3{a.root[0], a.root[1], a.root[2]};
        const f3 rhi = f3{a.root[4], a.root[5], a.root[6]};
        int sp = 0;
        const float qm = qnorm1(p);
        int32_t node = box_dist2(p, rlo, rhi) <= prune_bound(best, qm) ? 0 : -1;
        // each internal node is visited at most once in a valid tree: the step cap
        // and the reference checks keep a corrupted buffer from looping or faulting
        for (int64_t step = 0; node >= 0 && node < a.n - 1 && step < a.n + 64; ++step) {
            const float4 *rec = a.nodes + 6 * static_cast<int64_t>(node);
            const float4 l0 = rec[0], l1 = rec[1], l2 = rec[2], r0 = rec[3], r1 = rec[4], r2 = rec[5];
            const int32_t lref = __float_as_int(l0.w), rref = __float_as_int(r0.w);
            if (lref >= a.n - 1 || rref >= a.n - 1 || ~lref >= a.n || ~rref >= a.n) break;
            ++n_exp;
            n_lbox += (lref < 0) + (rref < 0);
            if (lref < 0 && leaf_box_dist2<kTri>(p, l0, l1, l2) <= prune_bound(best, qm))
                consider(leaf_dist2<kTri>(p, l0, l1, l2), __float_as_int(l1.w), ~lref);
            if (rref < 0 && leaf_box_dist2<kTri>(p, r0, r1, r2) <= prune_bound(best, qm))
                consider(leaf_dist2<kTri>(p, r0, r1, r2), __float_as_int(r1.w), ~rref);
            const float bound = prune_bound(best, qm);
            const float dl = lref >= 0 ? child_bound<kTri, kBall>(p, dq, l0, l1, l2) : INFINITY;
            const float dr = rref >= 0 ? child_bound<kTri, kBall>(p, dq, r0, r1, r2) : INFINITY;
            const bool gl = lref >= 0 && dl <= bound, gr = rref >= 0 && dr <= bound;
            if (gl && gr) {
                const bool left_first = dl <= dr;
                const int32_t far = left_first ? rref : lref;
                node = left_first ? lref : rref;
                if (sp < kLdsStack) s_stack[sp][lane] = far;
                else if (sp < kMaxStack) deep[sp - kLdsStack] = far;
                else atomicOr(a.status, 64);   // past the depth bound of a valid tree
                sp = sp < kMaxStack ? sp + 1 : sp;
            } else if (gl) {
                node = lref;
            } else if (gr) {
                node = rref;
            } else if (sp > 0) {
                --sp;
                node = sp < kLdsStack ? s_stack[sp][lane] : deep[sp - kLdsStack];
            } else {
                node = -1;
            }
        }
    }
    write_result<kTri>(a, q, p, best_leaf, best_id, best);
    if (a.counters) add_counters(a, n_exp, n_lbox, n_lex, 1);
}

// kMinWaves: the fewest waves per SIMD the register allocation must allow.  The
// triangle kernel takes 94 or 95 VGPRs and no scratch with 4 as with 5, so that five
// waves are resident either way and only the compiler's schedule differs.
template <bool kTri, int M, int kMinWaves>
__global__ __launch_bounds__(64 * kBatchWaves) __attribute__((amdgpu_waves_per_eu(kMinWaves))) void traverse_batch_kernel(QueryArgs a) {
    __shared__ BatchLds<kTri, M> lds;
    check_vertex_count(a);
    const int64_t per_block = static_cast<int64_t>(kBatchWaves) * M;
    batch_loop<kTri, M>(a, static_cast<int64_t>(blockIdx.x) * per_block, static_cast<int64_t>(gridDim.x) * per_block,
                        a.nq, lds);
}

// ----------------------------------------------------------------- k nearest
// The batch kernel with the K best per query (k <= K kept), the children pruned
// against the k-th.  20,002 queries, k = 4, on 46,000 faces: 268 -> 51 us
// against one query per lane, depth-first, where a wave waits for its longest walk.
template <int M, int K>
__global__ __launch_bounds__(64 * kBatchWaves) __attribute__((amdgpu_waves_per_eu(4))) void knn_batch_kernel(QueryArgs a) {
    __shared__ BatchLds<true, M, K> lds;
    check_vertex_count(a);
    const int64_t per_block = static_cast<int64_t>(kBatchWaves) * M;
    batch_loop<true, M, true, K>(a, static_cast<int64_t>(blockIdx.x) * per_block,
                                 static_cast<int64_t>(gridDim.x) * per_block, a.nq, lds);
}

// Every face for every query, in original face order (strict < keeps the
// lowest id on exact ties).
__global__ __launch_bounds__(256) void bruteforce_kernel(const float *__restrict__ verts, int64_t nv,
                                                         const int32_t *__restrict__ faces, int64_t nf,
                                                         const float *__restrict__ queries, int64_t nq,
                                                         float maxd2, int32_t *face, float *point,
                                                         float *bary, float *dist2, float *normal) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    const f3 p = load3(queries, nq, q);
    float best = INFINITY;
    int64_t bf = -1;
    for (int64_t f = 0; f < nf; ++f) {
        const f3 A = load3(verts, nv, faces[f]);
        const f3 B = load3(verts, nv, faces[nf + f]);
        const f3 C = load3(verts, nv, faces[2 * nf + f]);
        float w1, w2;
        const float d2 = tri_closest(p, A, B, C, w1, w2);
        if (d2 < best) { best = d2; bf = f; }
    }
    if (bf >= 0 && best <= maxd2) {
        const f3 A = load3(verts, nv, faces[bf]);
        const f3 B = load3(verts, nv, faces[nf + bf]);
        const f3 C = load3(verts, nv, faces[2 * nf + bf]);
        float w1, w2;
        const float d2 = tri_closest(p, A, B, C, w1, w2);
        face[q] = static_cast<int32_t>(bf);
        if (point) store3(point, nq, q, tri_point(A, B, C, w1, w2));
        if (bary) { bary[q] = w1; bary[nq + q] = w2; }
        if (dist2) dist2[q] = d2;
        if (normal) store3(normal, nq, q, tri_normal(A, B, C));
    } else {
        face[q] = -1;
        if (point) store3(point, nq, q, p);
        if (bary) { bary[q] = 0.0f; bary[nq + q] = 0.0f; }
        if (dist2) dist2[q] = INFINITY;
        if (normal) store3(normal, nq, q, f3{0.0f, 0.0f, 0.0f});
    }
}

template <typename T>
inline const T *cat(const void *base, int64_t off) {
    return reinterpret_cast<const T *>(static_cast<const char *>(base) + off);
}

// ---------------------------------------------------------------- scan kernel
// Few queries on a small tree: a wave per query tests every leaf, the lanes 64 of
// them at a time and four such groups' records in flight.  A traversal is bound
// there by its chain, a round of about 1 us for every level of the tree and the
// hint's four dependent reads before it; the scan has no chain beyond a read of
// the leaves' places and one of their records.  Triangles whose box lies beyond
// the best of the groups before are not tested.  Same leaf arithmetic, and the
// least (d^2, id) of all leaves, so the same result; a hint cannot change it and is
// not read.  257 queries on 500 faces: 17.0 us hinted and 19.7 cold, 8.0 so; 2,000
// nearest of 2,080 points 18.0, 11.0.
template <bool kTri>
__global__ __launch_bounds__(64 * kBatchWaves) void scan_kernel(QueryArgs a) {
    constexpr int kGroups = 4;
    check_vertex_count(a);
    const int lane = threadIdx.x % 64;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kBatchWaves + threadIdx.x / 64;
    if (q >= a.nq) return;
    const f3 p = load3(a.queries, a.nq, q);
    const float qm = qnorm1(p);
    const int32_t n = static_cast<int32_t>(a.n), slots = 2 * (n - 1);
    unsigned long long best = pack_best(a.maxd2, INT_MAX);
    const unsigned long long none = best;
    float pb = prune_bound(a.maxd2, qm);
    int32_t at = -1;
    for (int32_t base = 0; base < n; base += 64 * kGroups) {
        int32_t code[kGroups];
        bool ok[kGroups];
#pragma unroll
        for (int u = 0; u < kGroups; ++u) {
            const int32_t leaf = base + 64 * u + lane;
            code[u] = a.leaf_parent[leaf < n ? leaf : 0];
            ok[u] = leaf < n && code[u] >= 0 && code[u] < slots;
            if (leaf < n && !ok[u]) atomicOr(a.status, 16);
        }
        float4 f0[kGroups], f1[kGroups], f2[kGroups];
#pragma unroll
        for (int u = 0; u < kGroups; ++u) {
            const float4 *rec = a.nodes + 3 * (ok[u] ? code[u] : 0);
            f1[u] = rec[1];
            if (kTri) { f0[u] = rec[0]; f2[u] = rec[2]; }
        }
#pragma unroll
        for (int u = 0; u < kGroups; ++u) {
            bool act = ok[u];
            if (kTri) act = act && leaf_box_dist2<kTri>(p, f0[u], f1[u], f2[u]) <= pb;
            if (act) {
                const float d2 = kTri ? leaf_dist2<kTri>(p, f0[u], f1[u], f2[u]) : leaf_dist2<kTri>(p, f1[u], f1[u], f1[u]);
                const unsigned long long cand = pack_best(d2, __float_as_int(f1[u].w));
                if (cand < best) {
                    best = cand;
                    at = code[u];
                }
            }
        }
        if (kTri && base + 64 * kGroups < n) {
            float d2 = __uint_as_float(static_cast<uint32_t>(best >> 32));
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) d2 = fminf(d2, __shfl_xor(d2, o));
            pb = prune_bound(d2, qm);
        }
    }
    unsigned long long m = best;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long x = __shfl_xor(m, o);
        if (x < m) m = x;
    }
    const uint64_t winners = __ballot(m < none && best == m);
    if (winners == 0) {
        if (lane == 0) write_result<kTri>(a, q, p, -1, -1, 0.0f);
        return;
    }
    if ((winners & lanemask_lt()) != 0 || best != m) return;
    const int32_t id = static_cast<int32_t>(m & 0xffffffffull);
    if (id < 0 || id >= n) {
        atomicOr(a.status, 16);
        write_result<kTri>(a, q, p, -1, -1, 0.0f);
    } else if (kTri) {
        const float4 *rec = a.nodes + 3 * at;
        write_face(a, q, p, id, xyz(rec[0]), xyz(rec[1]), xyz(rec[2]));
    } else {
        store_face(a, q, id);
        if (a.dist2) a.dist2[q] = __uint_as_float(static_cast<uint32_t>(m >> 32));
    }
}

// Whether the automatic choice is the scan: it reads every leaf for every query, so
// it pays up to about the size at which that fills the card (us by the batch kernel
// hinted, and by the scan):
//   triangles  1,088 faces: 1,000 queries 18.1 / 13.4, 4,000 23.3 / 18.9, 8,000 23.9 / 31.3;  2,080: 2,000 20.0 / 22.9
//   points     2,080: 4,000 queries 21.5 / 13.3, 8,000 22.0 / 26.3;  4,100: 4,000 22.6 / 24.1
template <bool kTri>
inline bool scans(const mg_query_options *o, int64_t n, int64_t nq) {
    if (o && (o->kernel != MG_QUERY_AUTO || o->batch || o->order || o->counters || o->queue || o->waves)) return false;
    return n >= 2 && n <= (kTri ? 1280 : 3072) && nq <= 4096;
}

// Queries per wave by default: the largest of 16, 8, 4, 2, 1 that leaves at least 512
// workgroups of four waves; on triangles 16 only for more queries than batches of 8 are
// resident at once (five waves on each of 1,024 SIMDs: 40,960), where a second round of
// waves costs more than the fuller batch.  Cold searches of small trees, whose walks are
// most of their work and fill a wave only with 16, differ: 256 workgroups are enough up
// to 2,048 faces, and 16 is not held back up to 16,384.  us in batches of 8 and 16,
// queries near the surface:
//   hinted  4,100 faces: 32,768 queries 27.0 / 27.0, 50,000 42.3 / 32.7;  40,000: 28,000 32.7 / 33.4,
//           40,000 37.2 / 37.3, 50,000 54.0 / 39.6;  500,000: 32,768 55.2 / 60.9, 65,536 94.6 / 74.7
//   cold    500 faces: 32,768 28.3 / 23.9;  4,100: 16,384 29.3 / 30.5, 40,000 42.0 / 35.4;  10,200: 40,000 42.2 / 36.6;
//           40,000: 24,000 36.6 / 38.5, 50,000 69.0 / 46.9;  500,000: 16,384 58.7 / 82.8, 32,768 68.4 / 94.1,
//           50,000 109 / 102
//   k = 4   20,002 queries: 4,100 faces 35.2 / 42.2, 46,460 49.2 / 55.9, 500,000 70.6 / 133
inline int default_batch(bool tri, bool cold, int64_t n, int64_t nq) {
    const int64_t least = tri && cold && n <= 2048 ? 1024 : 2048;
    int batch = 16;
    while (batch > 1 && nq < least * batch) batch >>= 1;
    return tri && !(cold && n <= 16384) && batch == 16 && nq <= 5 * 1024 * 8 ? 8 : batch;
}

// Default traversal when the caller gives no options: the batch kernel with a
// seed descent and the default batch.
inline void resolve(const mg_query_options *o, bool tri, int64_t n, int64_t nq, int &kernel, int &batch, int &seed) {
    kernel = o ? o->kernel : MG_QUERY_AUTO;
    batch = o ? o->batch : 0;
    seed = o ? (o->seed != 0) : 1;
    if (kernel == MG_QUERY_AUTO) kernel = MG_QUERY_BATCH;
    if (batch <= 0) batch = default_batch(tri, !(o && o->hint), n, nq);
}

__global__ void zero_word_kernel(uint32_t *w) { *w = 0u; }

// Without a queue: one workgroup per kBatchWaves batches (at most 4096
// workgroups, striding beyond).  With a queue: as many workgroups as can be
// resident at once, each wave taking batches until none is left.
template <bool kTri, int M, int kMinWaves>
mg_status launch_batch_variant(const QueryArgs &a, hipStream_t s) {
    const int64_t per_block = static_cast<int64_t>(M) * kBatchWaves;
    int64_t grid = std::min<int64_t>((a.nq + per_block - 1) / per_block, 256 * 16);
    if (a.queue) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, traverse_batch_kernel<kTri, M, kMinWaves>,
                                                         64 * kBatchWaves, 0) != hipSuccess)
            return MG_ERR_HIP;
        grid = std::max<int64_t>(1, std::min<int64_t>(grid, static_cast<int64_t>(cus) * std::max(per_cu, 1)));
        hipLaunchKernelGGL(zero_word_kernel, dim3(1), dim3(1), 0, s, a.queue);
    }
    hipLaunchKernelGGL((traverse_batch_kernel<kTri, M, kMinWaves>), dim3(static_cast<unsigned>(grid)),
                       dim3(64 * kBatchWaves), 0, s, a);
    return launch_status();
}

// Compute units of the current device, read once per device (a partitioned
// device has fewer than the full chip's 256).
int device_cus() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int v = cached[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cached[dev].store(v, std::memory_order_relaxed);
    return v;
}

// The five-wave form of the triangle kernel is launched when its batches outnumber
// four waves on every SIMD (CUs x 4 SIMDs x 4 waves; 4,096 on a whole MI355X).  The
// forms differed when four waves took 109 VGPRs (1M queries ran 7% faster with five);
// now both fit five waves and take the same time (1M hinted queries on 500,000 faces
// 1,342 and 1,342 us, 100,000 near it 131 and 131).
// waves: 0 by that rule, 4 or 5 forced.
template <bool kTri, int M>
mg_status launch_batch(const QueryArgs &a, int waves, hipStream_t s) {
    if constexpr (kTri) {
        const int64_t four_wave_slots = static_cast<int64_t>(device_cus()) * 4 * 4;
        if (waves == 5 || (waves == 0 && (a.nq + M - 1) / M > four_wave_slots))
            return launch_batch_variant<kTri, M, 5>(a, s);
    }
    return launch_batch_variant<kTri, M, 4>(a, s);
}

template <bool kTri>
mg_status launch_traverse(QueryArgs a, const mg_query_options *opts, hipStream_t s) {
    int kernel, batch;
    resolve(opts, kTri, a.n, a.nq, kernel, batch, a.seed);
    const int waves = opts ? opts->waves : 0;
    a.order = opts ? opts->order : nullptr;
    a.counters = opts ? reinterpret_cast<unsigned long long *>(opts->counters) : nullptr;
    a.queue = opts ? opts->queue : nullptr;
    a.hint = opts ? opts->hint : nullptr;
    if (scans<kTri>(opts, a.n, a.nq)) {
        hipLaunchKernelGGL(scan_kernel<kTri>, dim3(blocks_for(a.nq, kBatchWaves)), dim3(64 * kBatchWaves), 0, s, a);
        return launch_status();
    }
    if (kernel == MG_QUERY_LANE) {
        // On small trees the ball's part of the bound costs a lane more than what it prunes
        // saves (us without and with it: 65,536 queries near 4,100 faces 96 / 106, uniform ones
        // on 1,088 faces 281 / 323; near 40,000 faces 132 / 137, uniform on 100,800 1,510 / 1,332,
        // 4,097 of them 1,196 / 520).
        const dim3 grid(static_cast<unsigned>(blocks_for(a.nq, kLaneBlock)));
        if constexpr (kTri) {
            if (a.n > 8192) {
                hipLaunchKernelGGL((traverse_lane_kernel<kTri, true>), grid, dim3(kLaneBlock), 0, s, a);
                return launch_status();
            }
        }
        hipLaunchKernelGGL((traverse_lane_kernel<kTri, false>), grid, dim3(kLaneBlock), 0, s, a);
        return launch_status();
    }
    switch (batch) {
        case 1: return launch_batch<kTri, 1>(a, waves, s);
        case 2: return launch_batch<kTri, 2>(a, waves, s);
        case 4: return launch_batch<kTri, 4>(a, waves, s);
        case 8: return launch_batch<kTri, 8>(a, waves, s);
        case 16: return launch_batch<kTri, 16>(a, waves, s);
        case 32: return launch_batch<kTri, 32>(a, waves, s);
        default: return MG_ERR_INVALID_ARGUMENT;
    }
}

template <int M, int K>
mg_status launch_knn(const QueryArgs &a, hipStream_t s) {
    const int64_t per_block = static_cast<int64_t>(M) * kBatchWaves;
    const int64_t grid = std::min<int64_t>((a.nq + per_block - 1) / per_block, 256 * 16);
    hipLaunchKernelGGL((knn_batch_kernel<M, K>), dim3(static_cast<unsigned>(grid)), dim3(64 * kBatchWaves), 0, s, a);
    return launch_status();
}

// Queries per wave as for the single closest point on large trees (lists make small ones
// dearer too: k = 4 of 20,002 queries on 500 faces 30.2 us in batches of 8, 36.3 of 16),
// at most 64 / K.
template <int K>
mg_status launch_knn_k(const QueryArgs &a, hipStream_t s) {
    const int batch = default_batch(true, true, INT32_MAX, a.nq);
    if constexpr (K <= 4)
        if (batch >= 16) return launch_knn<16, K>(a, s);
    if (batch >= 8) return launch_knn<8, K>(a, s);
    if (batch >= 4) return launch_knn<4, K>(a, s);
    if (batch >= 2) return launch_knn<2, K>(a, s);
    return launch_knn<1, K>(a, s);
}

inline bool bad_options(const mg_query_options *o) {
    if (!o) return false;
    if (o->kernel < MG_QUERY_AUTO || o->kernel > MG_QUERY_BATCH) return true;
    if (o->waves != 0 && o->waves != 4 && o->waves != 5) return true;
    return !(o->batch == 0 || o->batch == 1 || o->batch == 2 || o->batch == 4 || o->batch == 8 || o->batch == 16 ||
             o->batch == 32);
}

// ------------------------------------------------------- spreading the queries
// Where the tree is larger than an XCD's L2, queries in no particular order make
// every XCD read all of it.  Spread queries are put in cells of the tree's root
// box (8 a side, in Morton order) and dealt so that an XCD's workgroups take one
// eighth of that sequence, while the queries of one batch come from all over the
// eighth: neighbours are alike in what they cost, and a wave of neighbours that
// are near the middle of everything would end long after the others (250,002 cold
// queries on 1M faces, sorted: 2,840 us; as they come 1,523; spread 1,170).
constexpr int kCells = 512;
constexpr int kSpreadThreads = 1024;
constexpr int kXcds = 8;

__device__ __forceinline__ uint32_t cell_of(const float *__restrict__ root, f3 q) {
    uint32_t c = 0;
    const float x[3] = {q.x, q.y, q.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float lo = root[k], ext = root[4 + k] - lo;
        // outside the box, or not a number: a cell at its end (fmaxf(NaN, 0) is 0)
        const uint32_t u = static_cast<uint32_t>(fminf(fmaxf((x[k] - lo) * (8.0f / ext), 0.0f), 7.0f));
        c |= ((u & 1u) | ((u & 2u) << 2) | ((u & 4u) << 4)) << (2 - k);
    }
    return c;
}

// counts <- queries per cell.  Workgroup b reads queries [b per, (b + 1) per).
__global__ __launch_bounds__(kSpreadThreads) void cell_count_kernel(const float *__restrict__ root,
                                                                    const float *__restrict__ queries, int64_t nq,
                                                                    int64_t per, uint32_t *__restrict__ counts) {
    __shared__ uint32_t s_count[kCells];
    for (int c = threadIdx.x; c < kCells; c += kSpreadThreads) s_count[c] = 0;
    __syncthreads();
    const int64_t q0 = blockIdx.x * per, q1 = q0 + per < nq ? q0 + per : nq;
    for (int64_t i = q0 + threadIdx.x; i < q1; i += kSpreadThreads)
        atomicAdd(&s_count[cell_of(root, load3(queries, nq, i))], 1u);
    __syncthreads();
    for (int c = threadIdx.x; c < kCells; c += kSpreadThreads)
        if (s_count[c]) atomicAdd(counts + c, s_count[c]);
}

// order <- the queries by cell, dealt to the launch's workgroups of 64 queries:
// place p of the sequence belongs to XCD p / (64 T), T workgroups of which take
// its 64 T places; a workgroup's 16 queries of a wave come from 16 parts of them.
// The last nq % 512 places stay at the end.
__global__ __launch_bounds__(kSpreadThreads) void cell_deal_kernel(const float *__restrict__ root,
                                                                   const float *__restrict__ queries, int64_t nq,
                                                                   int64_t per, const uint32_t *__restrict__ counts,
                                                                   uint32_t *__restrict__ taken,
                                                                   int32_t *__restrict__ order) {
    __shared__ uint32_t s_base[kCells], s_count[kCells], s_wave[kCells / 64];
    const int tid = threadIdx.x, lane = tid % 64;
    uint32_t inc = tid < kCells ? counts[tid] : 0u;
    const uint32_t own = inc;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (tid < kCells) {
        s_count[tid] = 0;
        if (lane == 63) s_wave[tid / 64] = inc;
    }
    __syncthreads();
    const int64_t q0 = blockIdx.x * per, q1 = q0 + per < nq ? q0 + per : nq;
    for (int64_t i = q0 + tid; i < q1; i += kSpreadThreads)
        atomicAdd(&s_count[cell_of(root, load3(queries, nq, i))], 1u);
    __syncthreads();
    if (tid < kCells) {
        uint32_t before = inc - own;
        for (int w = 0; w < tid / 64; ++w) before += s_wave[w];
        s_base[tid] = before + (s_count[tid] ? atomicAdd(taken + tid, s_count[tid]) : 0u);
    }
    __syncthreads();
    const uint32_t T = static_cast<uint32_t>(nq / (64 * kXcds)), full = 64u * kXcds * T;
    for (int64_t i = q0 + tid; i < q1; i += kSpreadThreads) {
        const uint32_t p = atomicAdd(&s_base[cell_of(root, load3(queries, nq, i))], 1u);
        uint32_t at = p;
        if (p < full) {
            const uint32_t xcd = p / (64 * T), in = p % (64 * T), part = in / (4 * T), rest = in % (4 * T);
            at = 64 * (kXcds * (rest / 4) + xcd) + 16 * (rest % 4) + part;
        }
        if (at < nq) order[at] = static_cast<int32_t>(i);
    }
}

__global__ __launch_bounds__(2 * kCells) void cell_clear_kernel(uint32_t *__restrict__ counts) { counts[threadIdx.x] = 0; }

}  // namespace
}  // namespace mgu

using namespace mgu;

extern "C" mg_status mg_closest_point_query(const void *bvh, size_t bvh_bytes, int32_t n_prims,
                                            const float *verts, int32_t n_verts, const float *queries,
                                            int32_t n_queries, float max_dist2, int32_t *face,
                                            float *point, float *bary, float *dist2, float *normal,
                                            const mg_query_options *opts, void *stream) {
    if (bad_count(n_prims) || bad_count(n_verts) || bad_count(n_queries) || !bvh || !(max_dist2 >= 0.0f) ||
        bad_options(opts))
        return MG_ERR_INVALID_ARGUMENT;
    mg_lbvh_layout L;
    mg_lbvh_layout_query(n_prims, MG_PRIM_TRIANGLES, &L);
    if (bvh_bytes < static_cast<size_t>(L.total_bytes)) return MG_ERR_WORKSPACE_TOO_SMALL;
    if (n_queries == 0) return MG_OK;
    if (!queries || !face || (n_prims > 0 && (!verts || n_verts == 0))) return MG_ERR_INVALID_ARGUMENT;
    QueryArgs a{};
    a.nodes = cat<float4>(bvh, L.off_nodes);
    a.root = cat<mg_lbvh_header>(bvh, L.off_header)->root_lo;
    a.leaf_faces = cat<int32_t>(bvh, L.off_leaf_faces);
    a.prim = cat<int32_t>(bvh, L.off_prim);
    a.inv_prim = cat<int32_t>(bvh, L.off_inv_prim);
    a.leaf_parent = cat<int32_t>(bvh, L.off_leaf_parent);
    a.status = &const_cast<mg_lbvh_header *>(cat<mg_lbvh_header>(bvh, L.off_header))->status;
    a.hdr_nv = &cat<mg_lbvh_header>(bvh, L.off_header)->n_verts;
    a.verts = verts; a.nv = n_verts; a.n = n_prims;
    a.queries = queries; a.nq = n_queries; a.maxd2 = max_dist2;
    a.face = face; a.point = point; a.bary = bary; a.dist2 = dist2; a.normal = normal;
    return launch_traverse<true>(a, opts, as_stream(stream));
}

extern "C" mg_status mg_query_default_batch(int32_t prim_kind, int32_t n_prims, int32_t n_queries, int32_t hinted,
                                            int32_t *batch) {
    if ((prim_kind != MG_PRIM_TRIANGLES && prim_kind != MG_PRIM_POINTS) || bad_count(n_prims) || bad_count(n_queries) ||
        !batch)
        return MG_ERR_INVALID_ARGUMENT;
    *batch = default_batch(prim_kind == MG_PRIM_TRIANGLES, !hinted, n_prims, n_queries);
    return MG_OK;
}

extern "C" mg_status mg_query_spread(const void *bvh, size_t bvh_bytes, int32_t n_prims, int32_t prim_kind,
                                     const float *queries, int32_t n_queries, int32_t *order, void *ws,
                                     size_t ws_bytes, void *stream) {
    if (bad_count(n_prims) || bad_count(n_queries) || !bvh) return MG_ERR_INVALID_ARGUMENT;
    mg_lbvh_layout L;
    const mg_status st = mg_lbvh_layout_query(n_prims, prim_kind, &L);
    if (st != MG_OK) return st;
    if (bvh_bytes < static_cast<size_t>(L.total_bytes) || ws_bytes < 2 * kCells * sizeof(uint32_t))
        return MG_ERR_WORKSPACE_TOO_SMALL;
    if (n_queries == 0) return MG_OK;
    if (!queries || !order || !ws) return MG_ERR_INVALID_ARGUMENT;
    hipStream_t s = as_stream(stream);
    const float *root = cat<mg_lbvh_header>(bvh, L.off_header)->root_lo;
    uint32_t *counts = static_cast<uint32_t *>(ws);
    const int64_t nq = n_queries;
    const int64_t per = std::max<int64_t>(2 * kSpreadThreads, (nq + 255) / 256);   // at most a workgroup per CU
    const unsigned grid = static_cast<unsigned>((nq + per - 1) / per);
    hipLaunchKernelGGL(cell_clear_kernel, dim3(1), dim3(2 * kCells), 0, s, counts);
    hipLaunchKernelGGL(cell_count_kernel, dim3(grid), dim3(kSpreadThreads), 0, s, root, queries, nq, per, counts);
    hipLaunchKernelGGL(cell_deal_kernel, dim3(grid), dim3(kSpreadThreads), 0, s, root, queries, nq, per, counts,
                       counts + kCells, order);
    return launch_status();
}

extern "C" mg_status mg_nearest_point_query(const void *bvh, size_t bvh_bytes, int32_t n_prims,
                                            const float *points, const float *queries, int32_t n_queries,
                                            float max_dist2, int32_t *index, float *dist2,
                                            const mg_query_options *opts, void *stream) {
    if (bad_count(n_prims) || bad_count(n_queries) || !bvh || !(max_dist2 >= 0.0f) || bad_options(opts))
        return MG_ERR_INVALID_ARGUMENT;
    mg_lbvh_layout L;
    mg_lbvh_layout_query(n_prims, MG_PRIM_POINTS, &L);
    if (bvh_bytes < static_cast<size_t>(L.total_bytes)) return MG_ERR_WORKSPACE_TOO_SMALL;
    if (n_queries == 0) return MG_OK;
    if (!queries || !index || (n_prims > 0 && !points)) return MG_ERR_INVALID_ARGUMENT;
    QueryArgs a{};
    a.nodes = cat<float4>(bvh, L.off_nodes);
    a.root = cat<mg_lbvh_header>(bvh, L.off_header)->root_lo;
    a.leaf_faces = nullptr;
    a.prim = cat<int32_t>(bvh, L.off_prim);
    a.inv_prim = cat<int32_t>(bvh, L.off_inv_prim);
    a.leaf_parent = cat<int32_t>(bvh, L.off_leaf_parent);
    a.status = &const_cast<mg_lbvh_header *>(cat<mg_lbvh_header>(bvh, L.off_header))->status;
    a.hdr_nv = &cat<mg_lbvh_header>(bvh, L.off_header)->n_verts;
    a.verts = points; a.nv = n_prims; a.n = n_prims;
    a.queries = queries; a.nq = n_queries; a.maxd2 = max_dist2;
    a.face = index; a.point = nullptr; a.bary = nullptr; a.dist2 = dist2; a.normal = nullptr;
    return launch_traverse<false>(a, opts, as_stream(stream));
}

extern "C" mg_status mg_closest_point_bruteforce(const float *verts, int32_t n_verts, const int32_t *faces,
                                                 int32_t n_faces, const float *queries, int32_t n_queries,
                                                 float max_dist2, int32_t *face, float *point, float *bary,
                                                 float *dist2, float *normal, void *stream) {
    if (bad_count(n_verts) || bad_count(n_faces) || bad_count(n_queries) || !(max_dist2 >= 0.0f))
        return MG_ERR_INVALID_ARGUMENT;
    if (n_queries == 0) return MG_OK;
    if (!queries || !face || (n_faces > 0 && (!verts || !faces || n_verts == 0)))
        return MG_ERR_INVALID_ARGUMENT;
    hipLaunchKernelGGL(bruteforce_kernel, dim3(blocks_for(n_queries, 256)), dim3(256), 0, as_stream(stream),
                       verts, (int64_t)n_verts, faces, (int64_t)n_faces, queries, (int64_t)n_queries, max_dist2,
                       face, point, bary, dist2, normal);
    return launch_status();
}

extern "C" mg_status mg_knn_surface_query(const void *bvh, size_t bvh_bytes, int32_t n_prims, const float *verts,
                                          int32_t n_verts, const float *queries, int32_t n_queries, int32_t k,
                                          float eps, float max_dist2, int32_t *face_k, float *dist2_k,
                                          float *point, uint64_t *counters, void *stream) {
    if (bad_count(n_prims) || bad_count(n_verts) || bad_count(n_queries) || !bvh || k < 1 || k > 8 ||
        !(eps >= 0.0f) || !(max_dist2 >= 0.0f))
        return MG_ERR_INVALID_ARGUMENT;
    mg_lbvh_layout L;
    mg_lbvh_layout_query(n_prims, MG_PRIM_TRIANGLES, &L);
    if (bvh_bytes < static_cast<size_t>(L.total_bytes)) return MG_ERR_WORKSPACE_TOO_SMALL;
    if (n_queries == 0) return MG_OK;
    if (!queries || !face_k || (n_prims > 0 && (!verts || n_verts == 0))) return MG_ERR_INVALID_ARGUMENT;
    QueryArgs a{};
    a.nodes = cat<float4>(bvh, L.off_nodes);
    a.root = cat<mg_lbvh_header>(bvh, L.off_header)->root_lo;
    a.leaf_faces = cat<int32_t>(bvh, L.off_leaf_faces);
    a.prim = cat<int32_t>(bvh, L.off_prim);
    a.inv_prim = cat<int32_t>(bvh, L.off_inv_prim);
    a.leaf_parent = cat<int32_t>(bvh, L.off_leaf_parent);
    a.status = &const_cast<mg_lbvh_header *>(cat<mg_lbvh_header>(bvh, L.off_header))->status;
    a.hdr_nv = &cat<mg_lbvh_header>(bvh, L.off_header)->n_verts;
    a.verts = verts; a.nv = n_verts; a.n = n_prims;
    a.queries = queries; a.nq = n_queries; a.maxd2 = max_dist2;
    a.point = point;
    a.counters = reinterpret_cast<unsigned long long *>(counters);
    a.face = face_k; a.dist2 = dist2_k;
    a.k = k; a.eps = eps;
    hipStream_t s = as_stream(stream);
    if (k == 1) {                             // the closest point itself, unweighted
        mg_query_options o{};
        o.seed = 1;
        o.counters = counters;
        return launch_traverse<true>(a, &o, s);
    }
    if (k <= 2) return launch_knn_k<2>(a, s);
    if (k <= 4) return launch_knn_k<4>(a, s);
    return launch_knn_k<8>(a, s);
}
