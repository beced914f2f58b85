// Linear BVH over triangles or points: build and refit (gfx950).
//
// The paper builds its collision structures once from the template faces and
// reuses them for every frame (Sec. 3.4, Initialization; O(N_v) per frame);
// the varying-topology baseline destroys and rebuilds them every frame
// (Sec. 4.1).  The BVH kind is not named by the paper; this is a linear BVH
// (Karras 2012) built entirely on the device:
//
//   bounds   per-axis min/max of s = (v0 + v1) + v2 per workgroup, s kept for
//            the next step; clears the build scratch (histograms, look-back
//            words, counters) on the way
//   morton   30-bit codes defined in IEEE binary32 (no contraction), fused
//            with the four 8-bit digit histograms of the radix sort
//            (up to 4,096 primitives: one workgroup makes the codes and sorts them
//            in LDS, instead of this and the next step's launches)
//   sort     4 passes of a stable LSD radix sort of (code, id): one kernel per
//            pass, tiles ranked with wave64 ballots (match masks over the 8
//            digit bits), global digit offsets by decoupled look-back
//   tree     Karras radix tree per internal node + leaf permutation of faces;
//            lists the subtrees of at most C leaves that cut the tree and the
//            "top" nodes above them
//   refit    one kernel: a workgroup per subtree refits it level by level
//            with summary slots in LDS, another lists each top node's two
//            children meanwhile, and the workgroup that finishes the last
//            subtree refits the top nodes from the deposited subtree roots
//            (see refit.hpp)
//
// Node records are child-centric (96 B: both children's boxes, or a leaf
// child's triangle itself) so a traversal step reads one record and a leaf
// test needs no further gathers.
#include <mutex>

#include "refit.hpp"
#include "repose.hpp"

namespace mgu {
namespace {

// Keys of a sort tile: about 256 tiles whatever the size (at least 512 and at
// most 4096 keys), so small sorts still spread over the chip.  Tiles of 512 keys
// take 256 threads, larger ones 4 keys per thread: a tile is alone on its CU, and
// ranking a thread's keys is a chain (1M keys: 23.5 us a pass with 16 keys in
// each of 256 threads, 16.3 us with 4 in 1024 and 16 look-back words).
inline int sort_tile_for(int64_t n) {
    int tile = 512;
    while (tile < 4096 && int64_t(tile) * 256 < n) tile <<= 1;
    return tile;
}
constexpr uint32_t kFlagAgg = 1u << 30;    // look-back word: tile aggregate
constexpr uint32_t kFlagPrefix = 2u << 30; //                 inclusive prefix
constexpr uint32_t kValueMask = (1u << 30) - 1;
constexpr int kSpinLimit = 1 << 24;        // bounded waits: error word instead of a hang
constexpr int kLookback = 16;              // look-back words read at once

constexpr int64_t align256(int64_t x) { return (x + 255) & ~int64_t(255); }

inline mg_lbvh_layout make_layout(int64_t n, int kind) {
    mg_lbvh_layout L{};
    const int64_t m = n > 0 ? n - 1 : 0;
    int64_t o = 0;
    L.off_header = o;      o += align256(sizeof(mg_lbvh_header));
    L.off_codes = o;       o += align256(4 * n);
    L.off_prim = o;        o += align256(4 * n);
    L.off_leaf_faces = o;  o += align256(kind == MG_PRIM_TRIANGLES ? 12 * n : 0);
    L.off_leaf_parent = o; o += align256(4 * n);
    L.off_node_parent = o; o += align256(4 * m);
    L.off_nodes = o;       o += align256(96 * m);
    L.off_node_aux = o;    o += align256(4 * m);
    L.off_child = o;       o += align256(8 * m);
    L.off_top_nodes = o;   o += align256(4 * n);
    L.off_top_child = o;   o += align256(16 * n);
    L.off_subtrees = o;    o += align256(12 * n);
    L.off_deposits = o;    o += align256(48 * n);
    L.off_top_scratch = o; o += align256(52 * n);
    L.off_inv_prim = o;    o += align256(4 * n);
    L.total_bytes = o;
    return L;
}

// Largest subtree C = 2^chunk_log2 leaves: the smallest power of two >= 256
// with n <= 512 C (a few hundred subtrees, so the top tree stays small),
// capped at 2048 (the phase-1 LDS state is 52 B per leaf).  A tree of 257 to 512
// leaves is one subtree: a level more in it is less than a phase for the one
// or two nodes above subtrees of 256 (refits in subtrees of 256 and of 512: 257 faces
// 14.0, 13.0 us; 320 15.7, 13.3; 450 15.7, 13.2; 512 16.6, 14.8; 320 points 9.5, 7.8; but
// 1,120 faces 16.2, 17.7).
inline int chunk_log2_for(int64_t n) {
    int c = n > 256 && n <= 512 ? 9 : 8;
    while ((int64_t(512) << c) < n && c < 11) ++c;
    return c;
}

constexpr int kBoundsBlocks = 1024;        // most workgroups of the bounds kernel
constexpr int64_t kPartialBytes = int64_t(kBoundsBlocks) * 6 * 4;

struct WsLayout {
    int64_t keys_a, vals_a, keys_b, vals_b, hist, partial, lookback, total;
    int64_t tiles;
};

inline WsLayout make_ws(int64_t n) {
    WsLayout W{};
    const int64_t tile = sort_tile_for(n);
    W.tiles = (n + tile - 1) / tile;
    int64_t o = 0;
    W.keys_a = o;   o += align256(4 * n);
    W.vals_a = o;   o += align256(4 * n);
    W.keys_b = o;   o += align256(4 * n);
    W.vals_b = o;   o += align256(4 * n);
    W.hist = o;     o += align256(4 * 4 * 256);
    W.partial = o;  o += kPartialBytes;
    W.lookback = o; o += align256(4 * 4 * 256 * W.tiles);
    W.total = o;
    return W;
}

template <typename T>
inline T *at(void *base, int64_t off) {
    return reinterpret_cast<T *>(static_cast<char *>(base) + off);
}

// ------------------------------------------------------------------ kernels

// s = (v0 + v1) + v2 for face i (three times its centroid), or the point itself.
// Every operation is a separately rounded binary32 add.
__device__ __forceinline__ f3 centroid_sum(const float *__restrict__ v, int64_t nv,
                                           const int32_t *__restrict__ faces, int64_t n, int64_t i) {
    if (faces == nullptr) return load3(v, nv, i);
    const f3 a = load3(v, nv, faces[i]);
    const f3 b = load3(v, nv, faces[n + i]);
    const f3 c = load3(v, nv, faces[2 * n + i]);
    return (a + b) + c;
}

__device__ __forceinline__ float wave_min(float x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fminf(x, __shfl_xor(x, o));
    return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}

// Min and max over a block of kThreads of three values per thread, to every thread.
template <int kThreads>
__device__ __forceinline__ void block_bounds(float mn[3], float mx[3], float (*s_red)[kThreads / kWave], float out[6]) {
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        mn[k] = wave_min(mn[k]);
        mx[k] = wave_max(mx[k]);
    }
    if (lane == 0)
        for (int k = 0; k < 3; ++k) { s_red[k][wave] = mn[k]; s_red[3 + k][wave] = mx[k]; }
    __syncthreads();
    // every wave reduces the waves' values again
    constexpr int kWaves = kThreads / kWave;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        out[k] = s_red[k][lane % kWaves];
        out[3 + k] = s_red[3 + k][lane % kWaves];
#pragma unroll
        for (int o = kWaves / 2; o >= 1; o >>= 1) {
            out[k] = fminf(out[k], __shfl_xor(out[k], o));
            out[3 + k] = fmaxf(out[3 + k], __shfl_xor(out[3 + k], o));
        }
    }
}

// The workgroup's bounds of s into partial[blockIdx.x]; the next kernel reduces
// them, so nothing has to be cleared before this one, which clears the scratch
// of the rest of the build and writes the header instead of a launch of its own.
// A face's s is stored (sx, sy, sz), so that its vertices are gathered once.
__global__ __launch_bounds__(256) void bounds_kernel(const float *__restrict__ v, int64_t nv,
                                                     const int32_t *__restrict__ faces, int64_t n,
                                                     float *__restrict__ sx, float *__restrict__ sy,
                                                     float *__restrict__ sz, float *__restrict__ partial,
                                                     mg_lbvh_header *hdr, uint32_t *__restrict__ hist,
                                                     uint32_t *__restrict__ lookback, int64_t n_lookback, int kind,
                                                     int chunk_log2) {
    __shared__ float s_red[6][4];
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = tid; i < n; i += stride) {
        const f3 s = centroid_sum(v, nv, faces, n, i);
        if (faces) { sx[i] = s.x; sy[i] = s.y; sz[i] = s.z; }
        mn[0] = fminf(mn[0], s.x); mn[1] = fminf(mn[1], s.y); mn[2] = fminf(mn[2], s.z);
        mx[0] = fmaxf(mx[0], s.x); mx[1] = fmaxf(mx[1], s.y); mx[2] = fmaxf(mx[2], s.z);
    }
    if (hist != nullptr)          // no sort scratch when there are no primitives
        for (int64_t i = tid; i < 4 * 256; i += stride) hist[i] = 0;
    if (lookback != nullptr)
        for (int64_t i = tid; i < n_lookback; i += stride) lookback[i] = 0;
    if (tid == 0) {
        hdr->n_prims = static_cast<int32_t>(n);
        hdr->n_verts = static_cast<int32_t>(nv);
        hdr->prim_kind = kind;
        hdr->status = 0;
        for (int k = 0; k < 4; ++k) hdr->tile_counter[k] = 0;
        hdr->refit_arrivals = 0u;
        hdr->chunk_log2 = chunk_log2;
        hdr->n_top = 0;
        hdr->n_sub = 0;
    }
    if (partial == nullptr) return;
    float out[6];
    block_bounds<256>(mn, mx, s_red, out);
    if (threadIdx.x < 6) partial[6 * static_cast<int64_t>(blockIdx.x) + threadIdx.x] = out[threadIdx.x];
}

// Put bit i of a 10-bit value at bit 3 i (magic-number spreading).
__device__ __forceinline__ uint32_t spread10(uint32_t x) {
    x &= 0x3ffu;
    x = (x | (x << 16)) & 0x030000ffu;
    x = (x | (x << 8)) & 0x0300f00fu;
    x = (x | (x << 4)) & 0x030c30c3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

// Quantisation defined in binary32: q = min(1023, trunc((s - lo) * scale)).
__device__ __forceinline__ uint32_t quant10(float s, float lo, float scale) {
#pragma clang fp contract(off)
    const float x = (s - lo) * scale;
    const uint32_t q = static_cast<uint32_t>(x);
    return q < 1023u ? q : 1023u;
}

// The lower corner of the codes' cells and the cells per unit, from the bounds of s.
__device__ __forceinline__ void quantisation(const float bounds[6], float lo[3], float scale[3]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = bounds[k];
        const float hi = bounds[3 + k];
        // 1024 / (hi - lo) correctly rounded to binary32: the binary64 quotient of
        // two binary32 values rounds to the same binary32 as a direct division.
        const float ext = hi - lo[k];
        scale[k] = hi > lo[k] ? static_cast<float>(1024.0 / static_cast<double>(ext)) : 0.0f;
    }
}

__device__ __forceinline__ uint32_t morton_code(f3 s, const float lo[3], const float scale[3]) {
    return (spread10(quant10(s.x, lo[0], scale[0])) << 2) | (spread10(quant10(s.y, lo[1], scale[1])) << 1) |
           spread10(quant10(s.z, lo[2], scale[2]));
}

// The bounds of s from the workgroups' partial ones, to every thread of 1024.
constexpr int kMortonThreads = 1024;
__device__ __forceinline__ void partial_bounds(const float *__restrict__ partial, int n_partial,
                                               float (*s_red)[kMortonThreads / kWave], float bounds[6]) {
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < n_partial; b += kMortonThreads)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            mn[k] = fminf(mn[k], partial[6 * b + k]);
            mx[k] = fmaxf(mx[k], partial[6 * b + 3 + k]);
        }
    block_bounds<kMortonThreads>(mn, mx, s_red, bounds);
}

// s: planes sx, sy, sz of n values (the bounds kernel's, or the points').
__global__ __launch_bounds__(kMortonThreads) __attribute__((amdgpu_waves_per_eu(8))) void morton_kernel(const float *__restrict__ sx, const float *__restrict__ sy,
                                                     const float *__restrict__ sz, int64_t n,
                                                     const float *__restrict__ partial, int n_partial,
                                                     mg_lbvh_header *hdr, uint32_t *__restrict__ keys,
                                                     uint32_t *__restrict__ hist) {
#pragma clang fp contract(off)
    __shared__ uint32_t s_hist[4][256];
    __shared__ float s_red[6][kMortonThreads / kWave];
    for (int i = threadIdx.x; i < 4 * 256; i += blockDim.x) (&s_hist[0][0])[i] = 0;
    float bounds[6];
    partial_bounds(partial, n_partial, s_red, bounds);
    float lo[3], scale[3];
    quantisation(bounds, lo, scale);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) { hdr->quant_lo[k] = lo[k]; hdr->quant_scale[k] = scale[k]; }
        for (int k = 0; k < 6; ++k) hdr->bounds_enc[k] = f2ord(bounds[k]);
    }
    __syncthreads();
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
        const f3 s = f3{sx[i], sy[i], sz[i]};
        const uint32_t code = morton_code(s, lo, scale);
        keys[i] = code;
        // neighbouring faces share their upper digits: the lanes with the first lane's
        // digit add once together instead of queueing on one counter
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t d = (code >> (8 * p)) & 0xffu;
            const uint32_t d0 = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(d)));
            const uint64_t same = __ballot(d == d0);
            if (d != d0) atomicAdd(&s_hist[p][d], 1u);
            else if ((same & lanemask_lt()) == 0) atomicAdd(&s_hist[p][d], static_cast<uint32_t>(__popcll(same)));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 4 * 256; i += blockDim.x) {
        const uint32_t c = (&s_hist[0][0])[i];
        if (c) atomicAdd(hist + i, c);
    }
}

// Exclusive scan of one value per thread over a block of kThreads.
template <int kThreads>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t *s_tmp /*[kThreads / 64]*/) {
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == kWave - 1) s_tmp[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w)               // the digits lie in the first 256 threads
        if (w < wave) before += s_tmp[w];
    __syncthreads();
    return before + inc - x;
}

// Threads of a sort tile of 256 kScale keys (sort_tile_for).
constexpr int sort_threads(int scale) { return scale <= 4 ? 256 : 64 * scale; }

// One stable LSD pass over digit (key >> shift) & 255 for tiles of 256 kScale
// keys.  vals_in == nullptr means the values are the input positions (first
// pass).  The first 256 threads own a digit each.
template <int kScale>
__global__ __launch_bounds__(sort_threads(kScale)) __attribute__((amdgpu_waves_per_eu(8))) void radix_pass_kernel(
    const uint32_t *__restrict__ keys_in, const int32_t *__restrict__ vals_in,
    uint32_t *__restrict__ keys_out, int32_t *__restrict__ vals_out, int64_t n, int shift,
    const uint32_t *__restrict__ hist, uint32_t *lookback, uint32_t *tile_counter, int32_t *status) {
    constexpr int kThreads = sort_threads(kScale), kTile = 256 * kScale, kItems = kTile / kThreads,
                  kWaves = kThreads / kWave;
    __shared__ uint32_t s_tile;
    __shared__ uint32_t s_wave_cnt[kWaves][256];
    __shared__ uint32_t s_digit_start[256];
    __shared__ uint32_t s_global[256];
    __shared__ uint32_t s_tmp[kWaves];
    __shared__ uint32_t s_keys[kTile];
    __shared__ int32_t s_vals[kTile];

    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
    const bool digit = tid < 256;
    const uint32_t hist_d = digit ? hist[tid] : 0u;
    for (int i = tid; i < kWaves * 256; i += kThreads) (&s_wave_cnt[0][0])[i] = 0;
    __syncthreads();
    const int64_t tile = s_tile;
    const int64_t base = tile * kTile;

    uint32_t key[kItems];
    int32_t val[kItems];
    uint32_t rank[kItems];
    const uint64_t lt = lanemask_lt();
    // all of a thread's keys in flight before the first is ranked
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t idx = base + (static_cast<int64_t>(wave) * kItems + j) * kWave + lane;
        const int64_t in = idx < n ? idx : n - 1;
        key[j] = keys_in[in];
        val[j] = vals_in ? vals_in[in] : static_cast<int32_t>(in);
    }
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t idx = base + (static_cast<int64_t>(wave) * kItems + j) * kWave + lane;
        const bool valid = idx < n;
        const uint32_t d = (key[j] >> shift) & 0xffu;
        // lanes of this wave holding the same digit (match mask from 8 ballots)
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint64_t below = m & lt;
        const uint32_t prev = valid ? s_wave_cnt[wave][d] : 0u;
        rank[j] = prev + static_cast<uint32_t>(__popcll(below));
        if (valid && below == 0) s_wave_cnt[wave][d] = prev + static_cast<uint32_t>(__popcll(m));
    }
    __syncthreads();

    // per digit: counts of each wave -> exclusive offsets across waves
    const int d = digit ? tid : 0;
    uint32_t tile_cnt = 0;
    uint32_t *my_word = lookback + tile * 256 + d;
    if (digit) {
        uint32_t c[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) c[w] = s_wave_cnt[w][d];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) tile_cnt += c[w];
        // publish this tile's aggregate as early as possible
        __hip_atomic_store(my_word, (tile == 0 ? kFlagPrefix : kFlagAgg) | tile_cnt, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        uint32_t before = 0;                  // a digit's column is its thread's alone
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            s_wave_cnt[w][d] = before;
            before += c[w];
        }
    }
    const uint32_t dstart = block_excl_scan<kThreads>(tile_cnt, s_tmp);
    if (digit) s_digit_start[d] = dstart;
    const uint32_t dbase = block_excl_scan<kThreads>(hist_d, s_tmp);

    // decoupled look-back: sum the counts of digit d over all earlier tiles, the
    // words of kLookback tiles read at once (a word is a round trip past the XCD's
    // L2, and the tiles in flight together have only their aggregates published)
    uint32_t excl = 0;
    if (tile > 0 && digit) {
        int64_t t = tile - 1;
        int spins = 0;
        for (bool found = false; !found;) {
            uint32_t w[kLookback];
#pragma unroll
            for (int u = 0; u < kLookback; ++u)
                // (32-bit byte offsets: with a 64-bit address each, the loads reused each
                // other's address registers and went one by one)
                w[u] = __hip_atomic_load(
                    reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(lookback) +
                                                       ((t > u ? static_cast<uint32_t>(t) - u : 0u) * 1024u + 4u * d)),
                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int used = 0;
            bool ready = true;
#pragma unroll
            for (int u = 0; u < kLookback; ++u) {
                ready = ready && !found && (w[u] & ~kValueMask) != 0;
                if (ready) {
                    excl += w[u] & kValueMask;
                    ++used;
                    found = (w[u] & kFlagPrefix) != 0;
                }
            }
            t -= used;
            if (used == 0 && ++spins > kSpinLimit) {   // never expected: report instead of hanging
                atomicOr(status, 1);
                break;
            }
        }
        __hip_atomic_store(my_word, kFlagPrefix | (excl + tile_cnt), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (digit) s_global[d] = dbase + excl - dstart;
    __syncthreads();

    // scatter into the tile in digit order (stable), then write out coalesced
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t idx = base + (static_cast<int64_t>(wave) * kItems + j) * kWave + lane;
        if (idx < n) {
            const uint32_t dj = (key[j] >> shift) & 0xffu;
            const uint32_t pos = s_digit_start[dj] + s_wave_cnt[wave][dj] + rank[j];
            s_keys[pos] = key[j];
            s_vals[pos] = val[j];
        }
    }
    __syncthreads();
    const int64_t count = (n - base) < kTile ? (n - base) : kTile;
    for (int i = tid; i < count; i += kThreads) {
        const uint32_t k = s_keys[i];
        const uint32_t out = s_global[(k >> shift) & 0xffu] + i;
        if (out < static_cast<uint64_t>(n)) {
            keys_out[out] = k;
            vals_out[out] = s_vals[i];
        } else {
            atomicOr(status, 2);   // inconsistent histogram: never expected
        }
    }
}

// Codes and the whole sort by one workgroup, keys and ids in LDS, for up to 1024
// kItems primitives.  The tiled sort is five launches there, each a chain of a few
// us over a handful of workgroups; here a pass is its ranking (the ballots of the
// radix passes, kItems keys a thread) and four barriers.  It takes 9 us for up to 1024
// primitives, 13 for 2048, 20 for 4096 and would take 32 for 8192, as the one compute
// unit's ranking grows; builds of (tiled, small) 1,024 faces 54.7, 41.5 us; 2,048 56.5,
// 46.2; 2,160 55.4, 50.5; 4,224 59.3, 66.4.
constexpr int64_t kSmallSort = 4096;
template <int kItems>
__global__ __launch_bounds__(kMortonThreads) void small_sort_kernel(const float *__restrict__ sx,
                                                                    const float *__restrict__ sy,
                                                                    const float *__restrict__ sz, int64_t n,
                                                                    const float *__restrict__ partial, int n_partial,
                                                                    mg_lbvh_header *hdr, uint32_t *__restrict__ codes,
                                                                    int32_t *__restrict__ prim) {
    constexpr int kWaves = kMortonThreads / kWave;
    static_assert(kItems * kMortonThreads <= 65536, "ids in 16 bits");
    __shared__ uint32_t s_keys[kItems * kMortonThreads];
    __shared__ uint16_t s_vals[kItems * kMortonThreads];
    __shared__ uint32_t s_wave_cnt[kWaves][256];
    __shared__ uint32_t s_tmp[kWaves];
    __shared__ float s_red[6][kWaves];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave, ni = static_cast<int>(n);
    const int first = wave * kItems * kWave + lane;          // the thread's keys: first + 64 j
    f3 s[kItems];                                            // in flight while the bounds are reduced
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int i = first + j * kWave < ni ? first + j * kWave : ni - 1;
        s[j] = f3{sx[i], sy[i], sz[i]};
    }
    float bounds[6], lo[3], scale[3];
    partial_bounds(partial, n_partial, s_red, bounds);
    quantisation(bounds, lo, scale);
    if (tid == 0) {
        for (int k = 0; k < 3; ++k) { hdr->quant_lo[k] = lo[k]; hdr->quant_scale[k] = scale[k]; }
        for (int k = 0; k < 6; ++k) hdr->bounds_enc[k] = f2ord(bounds[k]);
    }
    uint32_t key[kItems], val[kItems], rank[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        key[j] = morton_code(s[j], lo, scale);
        val[j] = first + j * kWave;
    }
    const uint64_t lt = lanemask_lt();
    for (int shift = 0; shift < 32; shift += 8) {
        for (int i = tid; i < kWaves * 256; i += kMortonThreads) (&s_wave_cnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const bool valid = first + j * kWave < ni;       // a place holds a key in every pass, or in none
            const uint32_t d = (key[j] >> shift) & 0xffu;
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bb = __ballot(bit);
                m &= bit ? bb : ~bb;
            }
            const uint64_t below = m & lt;
            const uint32_t prev = valid ? s_wave_cnt[wave][d] : 0u;
            rank[j] = prev + static_cast<uint32_t>(__popcll(below));
            if (valid && below == 0) s_wave_cnt[wave][d] = prev + static_cast<uint32_t>(__popcll(m));
        }
        __syncthreads();
        // the first 256 threads own a digit each: its keys before each wave's, from
        // the digit's start
        const int d = tid % 256;
        uint32_t c[kWaves], total = 0;
        if (tid < 256) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) c[w] = s_wave_cnt[w][d];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) total += c[w];
        }
        uint32_t before = block_excl_scan<kMortonThreads>(total, s_tmp);
        if (tid < 256) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                s_wave_cnt[w][d] = before;
                before += c[w];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kItems; ++j)
            if (first + j * kWave < ni) {
                const uint32_t pos = s_wave_cnt[wave][(key[j] >> shift) & 0xffu] + rank[j];
                s_keys[pos] = key[j];
                s_vals[pos] = static_cast<uint16_t>(val[j]);
            }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kItems; ++j)
            if (first + j * kWave < ni) {
                key[j] = s_keys[first + j * kWave];
                val[j] = s_vals[first + j * kWave];
            }
    }
#pragma unroll
    for (int j = 0; j < kItems; ++j)
        if (first + j * kWave < ni) {
            codes[first + j * kWave] = key[j];
            prim[first + j * kWave] = static_cast<int32_t>(val[j]);
        }
}

// Internal node i (i < n - 1) and leaf i (i < n): Karras's range and split
// search; children's parent tags; leaf face permutation; subtree and top lists.
//
// A search step is a dependent read of a code, and there are three searches of
// log2(range) steps, so the few nodes near the root set the time of one search
// per thread (some 48 steps of 0.3 us on 46,000 leaves).  A thread therefore
// searches only ranges that stay within kNear leaves, in a window of codes in
// LDS; the workgroup's other nodes (about six in 256) go to groups of 16 lanes
// that probe 16 places a step.  Hierarchies of 46,000 leaves:
// 17.5 -> 12.3 us, of 1M: 49 -> 29 us (also by leaving the records to the refit).
constexpr int kNear = 64;                  // longest range a thread searches alone
constexpr int kHierThreads = 256;
constexpr int kWindow = kHierThreads + 2 * kNear + 2;

__device__ __forceinline__ int karras_delta(uint32_t ci, uint32_t cj, int i, int j) {
    return ci != cj ? __clz(static_cast<int>(ci ^ cj))
                    : 32 + __clz(static_cast<int>(static_cast<uint32_t>(i) ^ static_cast<uint32_t>(j)));
}

__global__ __launch_bounds__(kHierThreads) void hierarchy_kernel(const uint32_t *__restrict__ codes,
                                                        const int32_t *__restrict__ prim,
                                                        int32_t *__restrict__ inv_prim, int64_t n,
                                                        const int32_t *__restrict__ faces,
                                                        int32_t *__restrict__ leaf_faces,
                                                        int32_t *__restrict__ leaf_parent,
                                                        int32_t *__restrict__ node_parent,
                                                        int32_t *__restrict__ node_aux,
                                                        int32_t *__restrict__ child,
                                                        int32_t *__restrict__ top_nodes,
                                                        int32_t *__restrict__ subtrees,
                                                        mg_lbvh_header *hdr, int chunk_log2) {
    __shared__ uint32_t s_code[kWindow];
    __shared__ int2 s_long[kHierThreads];      // nodes left to the lane groups: local index and sign of d, delta past the near end
    __shared__ int s_nlong;
    const int tid = threadIdx.x;
    const int ni = static_cast<int>(n);
    const int base = static_cast<int>(blockIdx.x) * kHierThreads, w0 = base - kNear - 1;
    const int i = base + tid;
    for (int u = tid; u < kWindow; u += kHierThreads) {
        const int j = w0 + u;
        s_code[u] = j >= 0 && j < ni ? codes[j] : 0u;
    }
    if (tid == 0) s_nlong = 0;
    // the leaf's face is gathered while the searches run
    int32_t f0 = 0, f1 = 0, f2 = 0;
    if (i < ni) {
        const int32_t p = prim[i];
        if (p >= 0 && p < ni) {
            inv_prim[p] = i;
            if (faces) { f0 = faces[p]; f1 = faces[n + p]; f2 = faces[2 * n + p]; }
        } else {
            atomicOr(&hdr->status, 4);
        }
    }
    auto store_leaf = [&]() {
        if (!faces || i >= ni) return;
        leaf_faces[i] = f0;
        leaf_faces[n + i] = f1;
        leaf_faces[2 * n + i] = f2;
    };
    if (n == 1) {
        if (i == 0) {
            leaf_parent[0] = -1;
            subtrees[0] = ~0;         // the one leaf is the one subtree
            subtrees[1] = 0;
            subtrees[2] = 0;
            hdr->n_sub = 1;
        }
        store_leaf();
        return;
    }
    __syncthreads();
    // Writes node x over leaves x and x + l d, split after x + sp d (+ -1 for d < 0).
    auto emit = [&](int x, int d, int l, int sp) {
        const int64_t j = x + l * d;
        const int64_t gamma = x + sp * d + (d < 0 ? -1 : 0);
        const int64_t lo = x < j ? x : j, hi = x < j ? j : x;
        const int32_t tag_l = static_cast<int32_t>(static_cast<uint32_t>(x) << 1), tag_r = tag_l | 1;
        if (lo == gamma) leaf_parent[gamma] = tag_l; else node_parent[gamma] = tag_l;
        if (hi == gamma + 1) leaf_parent[gamma + 1] = tag_r; else node_parent[gamma + 1] = tag_r;
        if (x == 0) node_parent[0] = -1;
        // (the records' own copies of these references are written by the refit)
        child[x] = static_cast<int32_t>(lo == gamma ? ~gamma : gamma);
        child[n - 1 + x] = static_cast<int32_t>(hi == gamma + 1 ? ~(gamma + 1) : gamma + 1);
        // the cut: a node with more than C leaves is a top node, and each of its
        // children with at most C leaves roots a subtree (list order is irrelevant)
        const int64_t C = int64_t(1) << chunk_log2;
        if (hi - lo + 1 > C) {
            const bool s0 = gamma - lo + 1 <= C, s1 = hi - gamma <= C;
            const int32_t t = static_cast<int32_t>(atomicAdd(reinterpret_cast<uint32_t *>(&hdr->n_top), 1u));
            int32_t k = 0;
            if (s0 || s1)
                k = static_cast<int32_t>(atomicAdd(reinterpret_cast<uint32_t *>(&hdr->n_sub), (s0 ? 1u : 0u) + (s1 ? 1u : 0u)));
            top_nodes[t] = x;
            node_aux[x] = t;
            if (s0) {
                subtrees[k] = static_cast<int32_t>(lo == gamma ? ~lo : gamma);
                subtrees[n + k] = static_cast<int32_t>(lo);
                subtrees[2 * n + k] = static_cast<int32_t>(gamma);
                ++k;
            }
            if (s1) {
                subtrees[k] = static_cast<int32_t>(hi == gamma + 1 ? ~hi : gamma + 1);
                subtrees[n + k] = static_cast<int32_t>(gamma + 1);
                subtrees[2 * n + k] = static_cast<int32_t>(hi);
            }
        } else {
            node_aux[x] = -1;
            if (x == 0) {             // the whole tree is one subtree
                atomicAdd(reinterpret_cast<uint32_t *>(&hdr->n_sub), 1u);
                subtrees[0] = 0;
                subtrees[n] = 0;
                subtrees[2 * n] = static_cast<int32_t>(n - 1);
            }
        }
    };
    if (i < ni - 1) {
        const uint32_t ci = s_code[i - w0];
        auto delta = [&](int jx) -> int {      // delta(i, jx) of Karras 2012 in the window; -1 outside [0, n)
            if (static_cast<uint32_t>(jx) >= static_cast<uint32_t>(ni)) return -1;
            return karras_delta(ci, s_code[jx - w0], i, jx);
        };
        const int d = (delta(i + 1) - delta(i - 1)) > 0 ? 1 : -1;
        const int dmin = delta(i - d);
        int lmax = 2;
        while (lmax <= kNear && delta(i + lmax * d) > dmin) lmax <<= 1;
        if (lmax > kNear) {                    // delta(i + kNear d) > dmin: the range is longer
            s_long[atomicAdd(&s_nlong, 1)] = make_int2(2 * tid + (d > 0 ? 1 : 0), dmin);
        } else {
            int l = 0;
            for (int t = lmax >> 1; t >= 1; t >>= 1)
                if (delta(i + (l + t) * d) > dmin) l += t;
            const int dnode = delta(i + l * d);
            int sp = 0;
            for (int k = 1;; ++k) {            // t = ceil(l / 2^k)
                const int t = (l + (1 << k) - 1) >> k;
                if (delta(i + (sp + t) * d) > dnode) sp += t;
                if (t <= 1) break;
            }
            emit(i, d, l, sp);
        }
    }
    __syncthreads();
    // the long ranges: 16 lanes each, all groups of a wave in step
    const int nlong = s_nlong, group = tid / 16, sub = tid % 16, shift = 16 * (group % 4);
    for (int first = 0; first < nlong; first += kHierThreads / 16) {
        const bool on = first + group < nlong;
        const int2 item = s_long[on ? first + group : 0];
        const int x = base + (item.x >> 1), d = (item.x & 1) ? 1 : -1, dmin = item.y;
        const uint32_t cx = s_code[x - w0];
        auto delta = [&](int64_t jx) -> int {
            if (jx < 0 || jx >= ni) return -1;
            return karras_delta(cx, codes[jx], x, static_cast<int>(jx));
        };
        auto votes = [&](bool yes) -> int {    // leading lanes of the group that say yes
            const uint32_t m = static_cast<uint32_t>(__ballot(on && yes) >> shift) & 0xffffu;
            return __builtin_ctz(~m);
        };
        // the largest e in [lo, hi) with ok(e), given ok(lo), not ok(hi), ok falling
        auto search = [&](int64_t lo, int64_t hi, int above) -> int64_t {
            while (__any(on && hi - lo > 1)) {
                const int64_t step = (hi - lo + 16) / 17;
                const int64_t at = lo + (sub + 1) * step;
                const int yes = votes(at < hi && delta(x + at * d) > above);
                if (hi - lo > 1) {
                    const int64_t nlo = lo + yes * step, nhi = nlo + step;
                    hi = nhi < hi ? nhi : hi;
                    lo = nlo;
                }
            }
            return lo;
        };
        int64_t lo = kNear, hi = 0;            // delta(x + kNear d) > dmin
        for (bool more = on; __any(more);) {   // the first power of two past the range
            const int64_t at = lo << (sub + 1);
            const int yes = votes(at <= ni && delta(x + at * d) > dmin);
            if (more) {
                hi = lo << (yes + 1);
                lo <<= yes;
                more = yes == 16;
            }
        }
        const int64_t l = search(lo, hi, dmin);
        const int dnode = delta(x + l * d);
        const int64_t sp = search(0, l, dnode);
        if (on && sub == 0) emit(x, d, static_cast<int>(l), static_cast<int>(sp));
    }
    store_leaf();
}

// Subtrees largest first.  Phase 1 of the refit gives subtree k to workgroup k
// (then k + grid, ...), and workgroups start in index order as compute units free
// up; when more subtrees than resident workgroups exist (LDS allows three per CU at
// 1024-leaf chunks, one at 2048), the late starters should be the small subtrees
// (longest-first list scheduling).  One workgroup deals them by size, a counting
// sort in LDS (the bitonic sort it replaces took 16 us); equal sizes in any order,
// and more than kOrderMax subtrees keep theirs.  The refit's records do not depend
// on the order.
constexpr int kOrderMax = 2048;
__global__ __launch_bounds__(1024) void order_subtrees_kernel(int32_t *__restrict__ subtrees, int64_t n,
                                                              const mg_lbvh_header *__restrict__ hdr) {
    __shared__ uint32_t s_start[2049];         // by 2048 - size: counts, then first places
    __shared__ uint32_t s_wave[16];
    const int ns = hdr->n_sub, tid = threadIdx.x;
    if (ns <= 1 || ns > kOrderMax) return;
    for (int i = tid; i <= 2048; i += 1024) s_start[i] = 0u;
    __syncthreads();
    int32_t r[2], f[2], l[2], bin[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = tid + 1024 * u;
        bin[u] = -1;
        if (i >= ns) continue;
        r[u] = subtrees[i]; f[u] = subtrees[n + i]; l[u] = subtrees[2 * n + i];
        const int size = l[u] - f[u] + 1;
        bin[u] = size < 0 ? 2048 : size > 2048 ? 0 : 2048 - size;
        atomicAdd(&s_start[bin[u]], 1u);
    }
    __syncthreads();
    // exclusive scan of bins 2 tid and 2 tid + 1 (bin 2048, size 0, cannot occur in a valid list)
    const uint32_t c0 = s_start[2 * tid], c1 = s_start[2 * tid + 1], total = c0 + c1;
    uint32_t inc = total;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (tid % kWave >= o) inc += y;
    }
    if (tid % kWave == kWave - 1) s_wave[tid / kWave] = inc;
    __syncthreads();
    uint32_t before = inc - total;
    for (int w = 0; w < tid / kWave; ++w) before += s_wave[w];
    s_start[2 * tid] = before;
    s_start[2 * tid + 1] = before + c0;
    if (tid == 1023) s_start[2048] = before + total;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (bin[u] < 0) continue;
        const uint32_t q = atomicAdd(&s_start[bin[u]], 1u);
        if (q >= static_cast<uint32_t>(ns)) continue;
        subtrees[q] = r[u];
        subtrees[n + q] = f[u];
        subtrees[2 * n + q] = l[u];
    }
}

// The top children: per top node and slot, the child's top index, or ~k when
// the child is the root of subtree k (every top node has two children of
// these kinds), and in planes 2 and 3 a top child's node id (0 for a subtree).
// One workgroup of a build's refit lists them beside the subtrees; device-scope
// stores, since the workgroup that refits the top may be on another XCD.
template <int kThreads>
__device__ void list_top_children(const RefitArgs &a, int T, int NS) {
    const int64_t n = a.n;
    int32_t *top_child = const_cast<int32_t *>(a.top_child);
    // the parent tag of a top node or subtree root names its slot in a top node
    auto put = [&](int32_t tag, int32_t v, int32_t node) {
        if (tag < 0) return;                  // the root
        const int32_t p = tag >> 1;
        if (p >= n - 1) { atomicOr(a.status, 8); return; }
        const int32_t t = a.node_aux[p];
        if (t < 0 || t >= T) { atomicOr(a.status, 8); return; }
        __hip_atomic_store(top_child + (tag & 1) * n + t, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(top_child + (2 + (tag & 1)) * n + t, node, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int t = threadIdx.x; t < T; t += kThreads) {
        const int32_t p = a.top_nodes[t];
        if (p < 0 || p >= n - 1) { atomicOr(a.status, 8); continue; }
        put(a.node_parent[p], t, p);
    }
    for (int k = threadIdx.x; k < NS; k += kThreads) {
        const int32_t r = a.subtrees[k];
        const bool leaf = r < 0;
        const int64_t id = leaf ? ~static_cast<int64_t>(r) : r;
        if (id >= (leaf ? n : n - 1)) { atomicOr(a.status, 8); continue; }
        put(leaf ? a.leaf_parent[id] : a.node_parent[id], ~k, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);            // this wave's stores have completed
    __syncthreads();
}

// The refit over workgroups block, block + nblocks, ...: each takes subtrees
// (kPer nodes per thread) and counts the subtrees it finished into the
// header's arrival word once their deposits are complete; the one that brings
// it to the number of subtrees refits the top nodes (then clears the word for
// the next refit).  smem: refit_lds_bytes(chunk_log2) bytes.
template <bool kTri, int kThreads, int kPer>
__device__ void refit_blocks(const RefitArgs &a, int64_t block, int64_t nblocks, unsigned char *smem) {
    __shared__ int s_last;
    const int32_t ns = *a.n_sub;
    const int T = *a.n_top;
    int mine = 0;
    if (a.list_top) {                         // a build: the first workgroup lists the top children
        if (block == 0) {
            if (ns >= 2 && T >= 1 && T < a.n) list_top_children<kThreads>(a, T, ns);
            ++mine;
        }
        --block;
        --nblocks;
    }
    if (block >= 0)
        for (int64_t k = block; k < ns; k += nblocks) {
            refit_subtree<kTri, kThreads, kPer>(a, k, smem);     // ends with a barrier
            ++mine;
        }
    if (ns < 2 || mine == 0) return;          // one subtree is the whole tree: its root is written
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(a.arrivals, static_cast<uint32_t>(mine), __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT) + mine == static_cast<uint32_t>(ns + a.list_top);
    __syncthreads();
    if (!s_last) return;
    constexpr int kCap = refit_top_cap(kThreads);
    static_assert(kCap % kThreads == 0, "the top nodes kept in LDS are dealt evenly");
    if (T < 1 || T >= a.n) {
        if (threadIdx.x == 0) atomicOr(a.status, 8);
    } else if (T <= kCap) {
        refit_top<kTri, kThreads, false, kCap / kThreads>(a, T, ns, smem);
    } else {
        refit_top<kTri, kThreads, true, 1>(a, T, ns, smem);
    }
    if (threadIdx.x == 0) __hip_atomic_store(a.arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool kTri, int kThreads, int kPer, int kMinWaves>
__global__ __launch_bounds__(kThreads, kMinWaves) void refit_kernel(RefitArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    refit_blocks<kTri, kThreads, kPer>(a, blockIdx.x, gridDim.x, smem);
}

// The frame update in one launch: workgroups [0, sub_blocks) refit (as
// refit_kernel), the next copy_blocks copy the frame into the live buffer,
// and the rest re-pose the Gaussians, gauss_tile each.  Every part reads the
// frame's vertices from the frame store, so none waits for another; the copy
// and re-pose workgroups, dispatched after the refit's, fill the compute units
// the refit leaves idle (its later subtrees and its one-workgroup top phase).
struct FrameWork {
    const float *src;          // frame k, [3][n_verts]
    float *live;               // [3][n_verts]
    int64_t n3;                // 3 n_verts
    int64_t copy_tile;         // floats per copy workgroup
    Inputs in;                 // re-pose inputs (verts = src)
    float *mean, *quat, *cov, *rot;
    int64_t gauss_tile;        // Gaussians per re-pose workgroup
    int64_t sub_blocks, copy_blocks;
};

template <int kThreads, int kPer, int kMinWaves>
__global__ __launch_bounds__(kThreads, kMinWaves) void frame_update_kernel(RefitArgs a, FrameWork w) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t b = blockIdx.x;
    if (b < w.sub_blocks) {
        refit_blocks<true, kThreads, kPer>(a, b, w.sub_blocks, smem);
        return;
    }
    if (b < w.sub_blocks + w.copy_blocks) {
        const int64_t i0 = (b - w.sub_blocks) * w.copy_tile;
        const int64_t i1 = i0 + w.copy_tile < w.n3 ? i0 + w.copy_tile : w.n3;
        for (int64_t i = i0 + threadIdx.x; i < i1; i += kThreads) w.live[i] = w.src[i];
        return;
    }
    const int64_t g0 = (b - w.sub_blocks - w.copy_blocks) * w.gauss_tile;
    const int64_t g1 = g0 + w.gauss_tile < w.in.ng ? g0 + w.gauss_tile : w.in.ng;
    for (int64_t g = g0 + threadIdx.x; g < g1; g += kThreads) repose_store(w.in, g, w.mean, w.quat, w.cov, w.rot);
}

template <bool kTri, int kThreads, int kPer, int kMinWaves>
mg_status launch_refit_t(const RefitArgs &a, int grid, hipStream_t s) {
    const size_t lds = refit_lds_bytes(a.chunk_log2);
    if (lds > 65536)    // beyond the default dynamic LDS limit (gfx950 has 160 KB per workgroup)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&refit_kernel<kTri, kThreads, kPer, kMinWaves>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    hipLaunchKernelGGL((refit_kernel<kTri, kThreads, kPer, kMinWaves>), dim3(grid), dim3(kThreads), lds, s, a);
    return launch_status();
}

// 512-thread workgroups: a thread per internal node of a subtree of up to 256
// or 512 leaves, and 2 nodes per thread for 1024-leaf subtrees.
// Up to 1024 leaves three workgroups fit a CU beside each other (about 50 KB
// of LDS each, six waves per SIMD), so a tree of 500,000 faces has nearly all
// its subtrees resident at once.  256-leaf subtrees leave half the threads
// idle in phase 1, but phase 2 then holds up to 512 top nodes at one node per
// thread (a 40,000-face tree has 276: 24.5 us against 26.4 us with 256-thread
// workgroups, whose phase 2 needs two nodes per thread there).  2048-leaf
// subtrees take a CU's LDS for themselves, so 1024 threads: with 512, 4 nodes each,
// a refit of 540,000 faces took 78 us, now 71, and of 1M 121, now 109.
template <bool kTri>
mg_status launch_refit_k(const RefitArgs &a, int grid, hipStream_t s) {
    if (a.chunk_log2 <= 9) return launch_refit_t<kTri, 512, 1, 6>(a, grid, s);
    if (a.chunk_log2 == 10) return launch_refit_t<kTri, 512, 2, 6>(a, grid, s);
    return launch_refit_t<kTri, 1024, 2, 4>(a, grid, s);
}

mg_status check_kind(int32_t kind) {
    return (kind == MG_PRIM_TRIANGLES || kind == MG_PRIM_POINTS) ? MG_OK : MG_ERR_INVALID_ARGUMENT;
}

RefitArgs refit_args(const float *verts, int64_t nv, void *bvh, int64_t n, int kind) {
    const mg_lbvh_layout L = make_layout(n, kind);
    RefitArgs a;
    a.verts = verts; a.nv = nv;
    a.leaf_faces = kind == MG_PRIM_TRIANGLES ? at<int32_t>(bvh, L.off_leaf_faces) : nullptr;
    a.prim = at<int32_t>(bvh, L.off_prim);
    a.leaf_parent = at<int32_t>(bvh, L.off_leaf_parent);
    a.node_parent = at<int32_t>(bvh, L.off_node_parent);
    a.nodes = at<float4>(bvh, L.off_nodes);
    a.child = at<int32_t>(bvh, L.off_child);
    a.node_aux = at<int32_t>(bvh, L.off_node_aux);
    a.top_nodes = at<int32_t>(bvh, L.off_top_nodes);
    a.top_child = at<int32_t>(bvh, L.off_top_child);
    a.subtrees = at<int32_t>(bvh, L.off_subtrees);
    a.deposit = at<float4>(bvh, L.off_deposits);
    a.top_scratch = at<float4>(bvh, L.off_top_scratch);
    a.tstride = n;
    mg_lbvh_header *hdr = at<mg_lbvh_header>(bvh, L.off_header);
    a.root = hdr->root_lo;
    a.status = &hdr->status;
    a.hdr_nv = &hdr->n_verts;
    a.n_top = &hdr->n_top;
    a.n_sub = &hdr->n_sub;
    a.arrivals = &hdr->refit_arrivals;
    a.n = n;
    a.chunk_log2 = chunk_log2_for(n);
    a.inf = INFINITY;
    a.list_top = 0;
    return a;
}

template <int kThreads, int kPer, int kMinWaves>
mg_status launch_frame_t(const RefitArgs &a, const FrameWork &w, int64_t grid, hipStream_t s) {
    const size_t lds = refit_lds_bytes(a.chunk_log2);
    if (lds > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&frame_update_kernel<kThreads, kPer, kMinWaves>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    hipLaunchKernelGGL((frame_update_kernel<kThreads, kPer, kMinWaves>), dim3(static_cast<unsigned>(grid)),
                       dim3(kThreads), lds, s, a, w);
    return launch_status();
}

// build: the tree is new, so the top children are listed too, by one workgroup more.
mg_status launch_refit(const float *verts, int64_t nv, void *bvh, int64_t n, int kind, bool build, hipStream_t s) {
    RefitArgs a = refit_args(verts, nv, bvh, n, kind);
    a.list_top = build;
    const int64_t C = int64_t(1) << a.chunk_log2;
    const int grid = static_cast<int>(std::min<int64_t>(2 * ((n + C - 1) / C), 65535)) + a.list_top;
    return kind == MG_PRIM_TRIANGLES ? launch_refit_k<true>(a, grid, s) : launch_refit_k<false>(a, grid, s);
}

}  // namespace
}  // namespace mgu

using namespace mgu;

extern "C" mg_status mg_lbvh_layout_query(int32_t n_prims, int32_t prim_kind, mg_lbvh_layout *out) {
    if (!out || bad_count(n_prims) || check_kind(prim_kind) != MG_OK) return MG_ERR_INVALID_ARGUMENT;
    *out = make_layout(n_prims, prim_kind);
    return MG_OK;
}

extern "C" mg_status mg_lbvh_workspace_size(int32_t n_prims, int32_t prim_kind, size_t *ws_bytes) {
    if (!ws_bytes || bad_count(n_prims) || check_kind(prim_kind) != MG_OK) return MG_ERR_INVALID_ARGUMENT;
    *ws_bytes = static_cast<size_t>(make_ws(n_prims).total);
    return MG_OK;
}

namespace mgu {
namespace {

mg_status build_into(const float *verts, int32_t n_verts, const int32_t *faces, int32_t n_prims,
                     int32_t prim_kind, void *bvh, size_t bvh_bytes, void *ws, size_t ws_bytes,
                     void *stream) {
    if (bad_count(n_verts) || bad_count(n_prims) || check_kind(prim_kind) != MG_OK)
        return MG_ERR_INVALID_ARGUMENT;
    if (prim_kind == MG_PRIM_TRIANGLES && n_prims > 0 && (!faces || n_verts == 0))
        return MG_ERR_INVALID_ARGUMENT;
    if (prim_kind == MG_PRIM_POINTS && (faces || n_verts != n_prims)) return MG_ERR_INVALID_ARGUMENT;
    if (!bvh) return MG_ERR_INVALID_ARGUMENT;
    const mg_lbvh_layout L = make_layout(n_prims, prim_kind);
    if (bvh_bytes < static_cast<size_t>(L.total_bytes)) return MG_ERR_WORKSPACE_TOO_SMALL;
    const WsLayout W = make_ws(n_prims);
    if (n_prims > 0 && (!ws || ws_bytes < static_cast<size_t>(W.total))) return MG_ERR_WORKSPACE_TOO_SMALL;
    if (n_prims > 0 && !verts) return MG_ERR_INVALID_ARGUMENT;
    hipStream_t s = as_stream(stream);
    const int64_t n = n_prims;
    mg_lbvh_header *hdr = at<mg_lbvh_header>(bvh, L.off_header);
    uint32_t *hist = n ? at<uint32_t>(ws, W.hist) : nullptr;
    uint32_t *lookback = n ? at<uint32_t>(ws, W.lookback) : nullptr;
    const int64_t n_lookback = 4 * 256 * W.tiles;
    const int32_t *fz = prim_kind == MG_PRIM_TRIANGLES ? faces : nullptr;
    const int grid = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(blocks_for(n, 256), kBoundsBlocks)));
    const bool small = n <= kSmallSort;
    uint32_t *ka = n ? at<uint32_t>(ws, W.keys_a) : nullptr, *kb = n ? at<uint32_t>(ws, W.keys_b) : nullptr;
    int32_t *va = n ? at<int32_t>(ws, W.vals_a) : nullptr, *vb = n ? at<int32_t>(ws, W.vals_b) : nullptr;
    // the sums of faces wait in the sort's planes that no pass has written yet
    float *sx = reinterpret_cast<float *>(kb), *sy = reinterpret_cast<float *>(vb), *sz = reinterpret_cast<float *>(va);
    float *partial = n ? at<float>(ws, W.partial) : nullptr;
    hipLaunchKernelGGL(bounds_kernel, dim3(grid), dim3(256), 0, s, verts, (int64_t)n_verts, fz, n, sx, sy, sz, partial,
                       hdr, small ? nullptr : hist, small ? nullptr : lookback, n_lookback, prim_kind,
                       chunk_log2_for(n_prims));
    if (launch_status() != MG_OK) return MG_ERR_HIP;
    if (n == 0) return MG_OK;
    uint32_t *codes = at<uint32_t>(bvh, L.off_codes);
    int32_t *prim = at<int32_t>(bvh, L.off_prim);
    const float *px = fz ? sx : verts, *py = fz ? sy : verts + n_verts,
                *pz = fz ? sz : verts + 2 * static_cast<int64_t>(n_verts);
    if (small) {
        auto sort = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(kMortonThreads), 0, s, px, py, pz, n, partial, grid, hdr, codes, prim);
        };
        if (n <= 1024) sort(small_sort_kernel<1>);
        else if (n <= 2048) sort(small_sort_kernel<2>);
        else sort(small_sort_kernel<4>);
    } else {
        // at most one workgroup per CU: every one adds its digit counts to the same 1024
        // words (1M faces: 26.8 us with 1024 workgroups of 256 threads, 13.5 us so)
        const int mgrid = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(blocks_for(n, kMortonThreads), 256)));
        hipLaunchKernelGGL(morton_kernel, dim3(mgrid), dim3(kMortonThreads), 0, s, px, py, pz, n, partial, grid, hdr, ka, hist);
        // pass p reads (src) and writes (dst): A->B, B->A, A->B, B->final
        const uint32_t *ksrc[4] = {ka, kb, ka, kb};
        const int32_t *vsrc[4] = {nullptr, vb, va, vb};
        uint32_t *kdst[4] = {kb, ka, kb, codes};
        int32_t *vdst[4] = {vb, va, vb, prim};
        const int tile = sort_tile_for(n);
        for (int p = 0; p < 4; ++p) {
            auto pass = [&](auto kernel, int threads) {
                hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(W.tiles)), dim3(threads), 0, s, ksrc[p],
                                   vsrc[p], kdst[p], vdst[p], n, 8 * p, hist + 256 * p,
                                   lookback + static_cast<int64_t>(p) * 256 * W.tiles, &hdr->tile_counter[p],
                                   &hdr->status);
            };
            if (tile <= 512) pass(radix_pass_kernel<2>, sort_threads(2));
            else if (tile <= 1024) pass(radix_pass_kernel<4>, sort_threads(4));
            else if (tile <= 2048) pass(radix_pass_kernel<8>, sort_threads(8));
            else pass(radix_pass_kernel<16>, sort_threads(16));
        }
    }
    hipLaunchKernelGGL(hierarchy_kernel, dim3(blocks_for(n, kHierThreads)), dim3(kHierThreads), 0, s, codes, prim,
                       at<int32_t>(bvh, L.off_inv_prim), n, fz,
                       fz ? at<int32_t>(bvh, L.off_leaf_faces) : nullptr, at<int32_t>(bvh, L.off_leaf_parent),
                       at<int32_t>(bvh, L.off_node_parent), at<int32_t>(bvh, L.off_node_aux),
                       at<int32_t>(bvh, L.off_child), at<int32_t>(bvh, L.off_top_nodes), at<int32_t>(bvh, L.off_subtrees),
                       hdr, chunk_log2_for(n));
    if (chunk_log2_for(n) >= 10)      // subtrees may outnumber the resident refit workgroups
        hipLaunchKernelGGL(order_subtrees_kernel, dim3(1), dim3(1024), 0, s, at<int32_t>(bvh, L.off_subtrees), n, hdr);
    if (launch_status() != MG_OK) return MG_ERR_HIP;
    return launch_refit(verts, n_verts, bvh, n, prim_kind, true, s);
}

}  // namespace
}  // namespace mgu

extern "C" mg_status mg_lbvh_build(const float *verts, int32_t n_verts, const int32_t *faces,
                                   int32_t n_prims, int32_t prim_kind, void *bvh, size_t bvh_bytes,
                                   void *ws, size_t ws_bytes, void *stream) {
    return build_into(verts, n_verts, faces, n_prims, prim_kind, bvh, bvh_bytes, ws, ws_bytes, stream);
}

// ------------------------------------------------ build without a caller workspace
//
// The sort scratch of mg_lbvh_build_static lives in this array, one copy per
// device for the life of the process.  In host code `scratch` only names the
// symbol: kernels get the device address that hipGetSymbolAddress returns for
// the current device.  Sized for the largest build accepted: four key/value
// planes of 2^20 entries, the four digit histograms, and look-back words for at
// most 256 tiles per pass (sort_tile_for keeps the tile count at or below 256
// up to 2^20 keys).
namespace {
constexpr int64_t kStaticMaxPrims = MG_LBVH_STATIC_MAX_PRIMS;
constexpr int64_t kStaticWsBytes = 4 * (4 * kStaticMaxPrims) + 4 * 4 * 256 + kPartialBytes + 4 * 4 * 256 * 256;
constexpr int kMaxDevices = 64;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticWsBytes];

namespace {
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device, looked up on the first
// call there.
mg_status scratch_address(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return MG_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return MG_ERR_UNSUPPORTED_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MG_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MG_OK;
}
}  // namespace

extern "C" mg_status mg_lbvh_build_static(const float *verts, int32_t n_verts, const int32_t *faces,
                                          int32_t n_prims, int32_t prim_kind, void *bvh, size_t bvh_bytes,
                                          void *stream) {
    if (n_prims < 0 || n_prims > kStaticMaxPrims) return MG_ERR_INVALID_ARGUMENT;
    if (make_ws(n_prims).total > kStaticWsBytes) return MG_ERR_INVALID_ARGUMENT;
    void *ws = nullptr;
    const mg_status st = scratch_address(&ws);
    if (st != MG_OK) return st;
    return build_into(verts, n_verts, faces, n_prims, prim_kind, bvh, bvh_bytes, ws,
                      static_cast<size_t>(kStaticWsBytes), stream);
}

extern "C" mg_status mg_frame_update(const float *frames, int32_t n_frames, int32_t n_verts, int32_t k,
                                     float *live, const int32_t *faces, int32_t n_faces, const int32_t *gface,
                                     const float *bary, const float *q_local, const float *log_scale,
                                     const float *offset, int32_t n_gauss, float *mean, float *quat, float *cov,
                                     float *rot, void *bvh, size_t bvh_bytes, void *stream) {
    if (bad_count(n_verts) || bad_count(n_faces) || bad_count(n_gauss) || n_frames <= 0 || k < 0 ||
        k >= n_frames || n_verts == 0 || n_faces == 0 || !frames || !live || !faces || !bvh)
        return MG_ERR_INVALID_ARGUMENT;
    if (n_gauss > 0 && (!gface || !bary || !q_local || !log_scale || !mean)) return MG_ERR_INVALID_ARGUMENT;
    const mg_lbvh_layout L = make_layout(n_faces, MG_PRIM_TRIANGLES);
    if (bvh_bytes < static_cast<size_t>(L.total_bytes)) return MG_ERR_WORKSPACE_TOO_SMALL;
    const int64_t n3 = 3 * static_cast<int64_t>(n_verts);
    const float *src = frames + static_cast<int64_t>(k) * n3;
    if (src < live + n3 && live < src + n3) return MG_ERR_INVALID_ARGUMENT;   // overlap
    const RefitArgs a = refit_args(src, n_verts, bvh, n_faces, MG_PRIM_TRIANGLES);
    const int64_t C = int64_t(1) << a.chunk_log2;
    FrameWork w;
    w.src = src;
    w.live = live;
    w.n3 = n3;
    w.in = Inputs{src, n_verts, faces, n_faces, gface, bary, q_local, log_scale, offset, n_gauss};
    w.mean = mean; w.quat = quat; w.cov = cov; w.rot = rot;
    w.sub_blocks = 2 * ((n_faces + C - 1) / C);
    const int64_t tile = 512;                // items of a round, whatever the workgroup's size
    w.copy_tile = 16 * tile;
    w.copy_blocks = (n3 + w.copy_tile - 1) / w.copy_tile;
    w.gauss_tile = 2 * tile;
    const int64_t gauss_blocks = (static_cast<int64_t>(n_gauss) + w.gauss_tile - 1) / w.gauss_tile;
    const int64_t grid = w.sub_blocks + w.copy_blocks + gauss_blocks;
    if (grid > 0x7fffffff) return MG_ERR_INVALID_ARGUMENT;
    hipStream_t s = as_stream(stream);
    if (a.chunk_log2 <= 9) return launch_frame_t<512, 1, 6>(a, w, grid, s);
    if (a.chunk_log2 == 10) return launch_frame_t<512, 2, 6>(a, w, grid, s);
    return launch_frame_t<1024, 2, 4>(a, w, grid, s);
}

extern "C" mg_status mg_lbvh_refit(const float *verts, int32_t n_verts, void *bvh, size_t bvh_bytes,
                                   int32_t n_prims, int32_t prim_kind, void *stream) {
    if (bad_count(n_verts) || bad_count(n_prims) || check_kind(prim_kind) != MG_OK || !bvh)
        return MG_ERR_INVALID_ARGUMENT;
    const mg_lbvh_layout L = make_layout(n_prims, prim_kind);
    if (bvh_bytes < static_cast<size_t>(L.total_bytes)) return MG_ERR_WORKSPACE_TOO_SMALL;
    if (prim_kind == MG_PRIM_POINTS && n_verts != n_prims) return MG_ERR_TOPOLOGY_MISMATCH;
    if (n_prims == 0) return MG_OK;
    if (!verts || n_verts == 0) return MG_ERR_INVALID_ARGUMENT;
    return launch_refit(verts, n_verts, bvh, n_prims, prim_kind, false, as_stream(stream));
}
