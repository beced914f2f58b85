// Index signed-distance grid (gfx950): the SDF that the paper builds once from
// the template faces beside the BVH, storing only indices (Sec. 3.4,
// Initialization).  Grid nodes keep the ids of their k nearest template faces
// (found once with mg_knn_surface_query); every frame a node's signed distance
// is recomputed from those faces' current vertices - no search, one pass over
// the grid - and queries interpolate it trilinearly.
//
// Node (i, j, k) of an nx x ny x nz grid sits at lo + h (i, j, k); node index
// i + nx (j + ny k).  A node's value is the minimum point-to-triangle distance
// over its faces (ties to the lowest slot), signed by the winning face's normal
// (positive where the normal points, including the plane itself).
#include "mgu_internal.hpp"

namespace mgu {
namespace {

struct Grid {
    float lo_x, lo_y, lo_z, h;
    int32_t nx, ny, nz;
};

__device__ __forceinline__ f3 node_pos(const Grid &g, int64_t n) {
    const int64_t i = n % g.nx, j = (n / g.nx) % g.ny, k = n / (static_cast<int64_t>(g.nx) * g.ny);
    return f3{g.lo_x + g.h * static_cast<float>(i), g.lo_y + g.h * static_cast<float>(j),
              g.lo_z + g.h * static_cast<float>(k)};
}

__global__ __launch_bounds__(256) void grid_points_kernel(Grid g, int64_t n, float *__restrict__ out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; v < n; v += stride)
        store3(out, n, v, node_pos(g, v));
}

__global__ __launch_bounds__(256) void sdf_update_kernel(const float *__restrict__ verts, int64_t nv,
                                                         const int32_t *__restrict__ faces, int64_t nf,
                                                         const int32_t *__restrict__ face_k, int k, Grid g,
                                                         int64_t n, float *__restrict__ sdf,
                                                         int32_t *__restrict__ face_out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; v < n; v += stride) {
        const f3 p = node_pos(g, v);
        float best = INFINITY;
        int32_t win = -1;
        float side = 1.0f;
        for (int s = 0; s < k; ++s) {
            const int32_t f = face_k[s * n + v];
            if (f < 0 || f >= nf) continue;       // ids outside the mesh are ignored
            const f3 A = load3(verts, nv, faces[f]);
            const f3 B = load3(verts, nv, faces[nf + f]);
            const f3 C = load3(verts, nv, faces[2 * nf + f]);
            float w1, w2;
            const float d2 = tri_closest(p, A, B, C, w1, w2);
            if (d2 < best) {
                best = d2;
                win = f;
                const f3 c = tri_point(A, B, C, w1, w2);
                side = fdot(p - c, tri_normal(A, B, C)) >= 0.0f ? 1.0f : -1.0f;
            }
        }
        sdf[v] = side * sqrtf(best);
        if (face_out) face_out[v] = win;
    }
}

// The faces' current corners as records of three float4 (nine floats, 48 bytes):
// written once per face, they leave a node three wide gathers per face where the
// index and vertex arrays take twelve of four bytes.
constexpr int kRecord = 3;

// At 40,000 faces the pass costs about 4 us, a launch and one chain of loads; at
// 500,000 about 12.
__global__ __launch_bounds__(256) void face_record_kernel(const float *__restrict__ verts, int64_t nv,
                                                          const int32_t *__restrict__ faces, int64_t nf,
                                                          float4 *__restrict__ rec) {
    const int64_t f = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (f >= nf) return;
    f3 c[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int64_t id = faces[j * nf + f];
        c[j] = load3(verts, nv, id >= 0 && id < nv ? id : 0);   // a face no node stores may hold any ids
    }
    rec[kRecord * f] = make_float4(c[0].x, c[0].y, c[0].z, c[1].x);
    rec[kRecord * f + 1] = make_float4(c[1].y, c[1].z, c[2].x, c[2].y);
    rec[kRecord * f + 2] = make_float4(c[2].z, 0.0f, 0.0f, 0.0f);
}

// The values of sdf_update_kernel for a compile-time k: every face id and vertex of
// a node is loaded before any distance is computed (ids outside the mesh read face 0
// and do not count), so the gathers overlap instead of forming one chain per face,
// and the winner's sign is taken once, after the minimum.  Node coordinates use
// 32-bit index arithmetic (grids have fewer than 2^31 nodes).
//
// Bound by the vector cache, which serves a lane's scattered load at a time: 4 faces
// a node are 48 loads from the index and vertex arrays.  kPacked takes them from the
// records of face_record_kernel, 12 loads: 262,144 nodes, k = 4, 40,000 faces
// 17.1 -> 12.1 us with the pass that writes them; 128^3 nodes 84 -> 36 us.  Bricks
// of 4^3, 8 x 8 or 16 x 4 nodes a wave gain the records nothing (12.2, 11.7, ~12 us).
template <int K, bool kPacked>
__global__ __launch_bounds__(256) void sdf_update_k_kernel(const float *__restrict__ verts, int64_t nv,
                                                           const int32_t *__restrict__ faces, int64_t nf,
                                                           const float4 *__restrict__ rec,
                                                           const int32_t *__restrict__ face_k, Grid g, int64_t n,
                                                           float *__restrict__ sdf, int32_t *__restrict__ face_out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
    const uint32_t nx = static_cast<uint32_t>(g.nx), ny = static_cast<uint32_t>(g.ny);
    for (int64_t v = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; v < n; v += stride) {
        const uint32_t u = static_cast<uint32_t>(v), i = u % nx, j = (u / nx) % ny, kk = u / (nx * ny);
        const f3 p = f3{g.lo_x + g.h * static_cast<float>(i), g.lo_y + g.h * static_cast<float>(j),
                        g.lo_z + g.h * static_cast<float>(kk)};
        int32_t fid[K];
        bool ok[K];
#pragma unroll
        for (int s = 0; s < K; ++s) {
            const int32_t f = face_k[s * n + v];
            ok[s] = f >= 0 && f < nf;
            fid[s] = ok[s] ? f : 0;
        }
        f3 A[K], B[K], C[K];
#pragma unroll
        for (int s = 0; s < K; ++s) {
            if (kPacked) {
                const float4 *r = rec + kRecord * static_cast<int64_t>(fid[s]);
                const float4 r0 = r[0], r1 = r[1];
                A[s] = f3{r0.x, r0.y, r0.z};
                B[s] = f3{r0.w, r1.x, r1.y};
                C[s] = f3{r1.z, r1.w, r[2].x};
            } else {
                A[s] = load3(verts, nv, faces[fid[s]]);
                B[s] = load3(verts, nv, faces[nf + fid[s]]);
                C[s] = load3(verts, nv, faces[2 * nf + fid[s]]);
            }
        }
        float best = INFINITY, bw1 = 0.0f, bw2 = 0.0f;
        int32_t win = -1;
        f3 bA = f3{0.0f, 0.0f, 0.0f}, bB = bA, bC = bA;
#pragma unroll
        for (int s = 0; s < K; ++s) {
            float w1, w2;
            const float d2 = tri_closest(p, A[s], B[s], C[s], w1, w2);
            if (ok[s] && d2 < best) {             // ties keep the lowest slot
                best = d2; win = fid[s];
                bA = A[s]; bB = B[s]; bC = C[s]; bw1 = w1; bw2 = w2;
            }
        }
        float side = 1.0f;
        if (win >= 0) {
            const f3 c = tri_point(bA, bB, bC, bw1, bw2);
            side = fdot(p - c, tri_normal(bA, bB, bC)) >= 0.0f ? 1.0f : -1.0f;
        }
        sdf[v] = side * sqrtf(best);
        if (face_out) face_out[v] = win;
    }
}

template <int K>
void launch_update_k(int grid, hipStream_t st, const float *verts, int64_t nv, const int32_t *faces, int64_t nf,
                     const float4 *rec, const int32_t *face_k, const Grid &g, int64_t n, float *sdf, int32_t *face) {
    if (rec)
        hipLaunchKernelGGL((sdf_update_k_kernel<K, true>), dim3(grid), dim3(256), 0, st, verts, nv, faces, nf, rec,
                           face_k, g, n, sdf, face);
    else
        hipLaunchKernelGGL((sdf_update_k_kernel<K, false>), dim3(grid), dim3(256), 0, st, verts, nv, faces, nf, rec,
                           face_k, g, n, sdf, face);
}

__global__ __launch_bounds__(256) void sdf_sample_kernel(const float *__restrict__ sdf, Grid g,
                                                         const float *__restrict__ q, int64_t nq,
                                                         float *__restrict__ out) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t >= nq) return;
    const f3 p = load3(q, nq, t);
    const float r = 1.0f / g.h;
    const float ux = (p.x - g.lo_x) * r, uy = (p.y - g.lo_y) * r, uz = (p.z - g.lo_z) * r;
    if (!(ux >= 0.0f && uy >= 0.0f && uz >= 0.0f && ux <= g.nx - 1 && uy <= g.ny - 1 && uz <= g.nz - 1)) {
        out[t] = INFINITY;
        return;
    }
    const int i = min(static_cast<int>(floorf(ux)), g.nx - 2);
    const int j = min(static_cast<int>(floorf(uy)), g.ny - 2);
    const int k = min(static_cast<int>(floorf(uz)), g.nz - 2);
    const float tx = ux - i, ty = uy - j, tz = uz - k;
    const int64_t sx = 1, sy = g.nx, sz = static_cast<int64_t>(g.nx) * g.ny;
    const int64_t b = i + sy * j + sz * k;
    const float c00 = (1.0f - tx) * sdf[b] + tx * sdf[b + sx];
    const float c10 = (1.0f - tx) * sdf[b + sy] + tx * sdf[b + sy + sx];
    const float c01 = (1.0f - tx) * sdf[b + sz] + tx * sdf[b + sz + sx];
    const float c11 = (1.0f - tx) * sdf[b + sz + sy] + tx * sdf[b + sz + sy + sx];
    const float c0 = (1.0f - ty) * c00 + ty * c10, c1 = (1.0f - ty) * c01 + ty * c11;
    out[t] = (1.0f - tz) * c0 + tz * c1;
}

inline bool bad_grid(float h, int32_t nx, int32_t ny, int32_t nz, int64_t &n) {
    if (!(h > 0.0f) || nx < 2 || ny < 2 || nz < 2) return true;
    n = static_cast<int64_t>(nx) * ny * nz;
    return n > INT32_MAX;
}

}  // namespace
}  // namespace mgu

using namespace mgu;

extern "C" mg_status mg_grid_points(float lo_x, float lo_y, float lo_z, float h, int32_t nx, int32_t ny, int32_t nz,
                                    float *points, void *stream) {
    int64_t n = 0;
    if (bad_grid(h, nx, ny, nz, n) || !points) return MG_ERR_INVALID_ARGUMENT;
    const Grid g{lo_x, lo_y, lo_z, h, nx, ny, nz};
    const int grid = static_cast<int>(std::min<int64_t>(blocks_for(n, 256), 4096));
    hipLaunchKernelGGL(grid_points_kernel, dim3(grid), dim3(256), 0, as_stream(stream), g, n, points);
    return launch_status();
}

// From how many stored ids on the records pay, in units of 2^16, for k = 1, 2, 4, 8 and
// meshes of under 2,048, up to 65,536, up to 262,144 and more faces, if the ids are at
// least as many as the faces: they save a gather-bound update some 4 (k = 4 on 4,100
// faces), 6 (40,000), 7 (100,800) and 10 us (500,000) a million ids, less with fewer faces
// a node (k = 2: 0.7 on 500 faces, 3, 5, 7 and 10; k = 1 on 4,100 faces 1), and the pass
// that writes them takes 1, 2, 6 and 5 us.  us without and with records:
//   k = 1  4,100 faces: 96^3 nodes 10.1 / 10.1, 128^3 19.2 / 17.4;  40,000: 81^3 9.5 / 10.4, 96^3 12.7 / 12.1;
//          100,800: 112^3 19.5 / 19.3;  500,000: 96^3 26.3 / 27.4, 112^3 34.9 / 31.6;  500: 128^3 16.4 / 17.4
//   k = 2  500 faces: 81^3 9.1 / 9.2, 96^3 12.0 / 11.8;  4,100: 64^3 8.1 / 7.0;  40,000: 64^3 10.0 / 9.6;  100,800:
//          81^3 17.5 / 18.2, 96^3 24.3 / 20.2;  500,000: 72^3 24.3 / 25.7, 81^3 39.8 / 29.2
//   k = 4  500 faces: 52^3 7.9 / 7.8;  40,000: 52^3 11.7 / 10.6, 64^3 17.2 / 12.2;  100,800: 52^3 13.1 / 15.0,
//          62^3 18.2 / 18.3, 64^3 19.2 / 16.0;  500,000: 52^3 25.1 / 24.5, 64^3 31.0 / 26.0
//   k = 8  52^3: 500 13.0 / 10.5, 100,800 24.2 / 21.7;  48^3: 40,000 16.9 / 14.2, 500,000 38.5 / 28.2
static size_t record_bytes(int64_t n, int32_t k, int64_t nf) {
    constexpr int64_t kLeast[4][4] = {{INT32_MAX, 13, 24, 16}, {24, 8, 18, 16}, {8, 8, 14, 8}, {8, 8, 8, 8}};
    const int row = k == 1 ? 0 : k == 2 ? 1 : k == 4 ? 2 : k == 8 ? 3 : -1;
    const int mesh = nf < 2048 ? 0 : nf <= 65536 ? 1 : nf <= 262144 ? 2 : 3;
    const bool pays = row >= 0 && nf > 0 && n * k >= kLeast[row][mesh] << 16 && n * k >= nf;
    return pays ? kRecord * sizeof(float4) * static_cast<size_t>(nf) : 0;
}

extern "C" mg_status mg_sdf_records_bytes(int32_t n_faces, int32_t k, int32_t nx, int32_t ny, int32_t nz, size_t *bytes) {
    int64_t n = 0;
    if (bad_grid(1.0f, nx, ny, nz, n) || bad_count(n_faces) || k < 1 || k > 64 || !bytes) return MG_ERR_INVALID_ARGUMENT;
    *bytes = record_bytes(n, k, n_faces);
    return MG_OK;
}

extern "C" mg_status mg_sdf_update_records(const float *verts, int32_t n_verts, const int32_t *faces, int32_t n_faces,
                                           const int32_t *face_k, int32_t k, float lo_x, float lo_y, float lo_z,
                                           float h, int32_t nx, int32_t ny, int32_t nz, float *sdf, int32_t *face,
                                           void *records, size_t records_bytes, void *stream) {
    int64_t n = 0;
    if (bad_grid(h, nx, ny, nz, n) || bad_count(n_verts) || bad_count(n_faces) || k < 1 || k > 64 || !face_k ||
        !sdf || (n_faces > 0 && (!verts || !faces)) || reinterpret_cast<uintptr_t>(records) % sizeof(float4))
        return MG_ERR_INVALID_ARGUMENT;
    const Grid g{lo_x, lo_y, lo_z, h, nx, ny, nz};
    const int grid = static_cast<int>(std::min<int64_t>(blocks_for(n, 256), 8192));
    hipStream_t st = as_stream(stream);
    const int64_t nv = n_verts, nf = n_faces;
    const size_t need = record_bytes(n, k, nf);
    float4 *rec = records && need > 0 && records_bytes >= need ? static_cast<float4 *>(records) : nullptr;
    if (rec)
        hipLaunchKernelGGL(face_record_kernel, dim3(blocks_for(nf, 256)), dim3(256), 0, st, verts, nv, faces, nf, rec);
    if (n_faces > 0 && k == 1)
        launch_update_k<1>(grid, st, verts, nv, faces, nf, rec, face_k, g, n, sdf, face);
    else if (n_faces > 0 && k == 2)
        launch_update_k<2>(grid, st, verts, nv, faces, nf, rec, face_k, g, n, sdf, face);
    else if (n_faces > 0 && k == 4)
        launch_update_k<4>(grid, st, verts, nv, faces, nf, rec, face_k, g, n, sdf, face);
    else if (n_faces > 0 && k == 8)
        launch_update_k<8>(grid, st, verts, nv, faces, nf, rec, face_k, g, n, sdf, face);
    else
        hipLaunchKernelGGL(sdf_update_kernel, dim3(grid), dim3(256), 0, st, verts, nv, faces, nf, face_k, k, g, n,
                           sdf, face);
    return launch_status();
}

extern "C" mg_status mg_sdf_update(const float *verts, int32_t n_verts, const int32_t *faces, int32_t n_faces,
                                   const int32_t *face_k, int32_t k, float lo_x, float lo_y, float lo_z, float h,
                                   int32_t nx, int32_t ny, int32_t nz, float *sdf, int32_t *face, void *stream) {
    return mg_sdf_update_records(verts, n_verts, faces, n_faces, face_k, k, lo_x, lo_y, lo_z, h, nx, ny, nz, sdf,
                                 face, nullptr, 0, stream);
}

extern "C" mg_status mg_sdf_sample(const float *sdf, float lo_x, float lo_y, float lo_z, float h, int32_t nx,
                                   int32_t ny, int32_t nz, const float *queries, int32_t n_queries, float *out,
                                   void *stream) {
    int64_t n = 0;
    if (bad_grid(h, nx, ny, nz, n) || bad_count(n_queries) || !sdf) return MG_ERR_INVALID_ARGUMENT;
    if (n_queries == 0) return MG_OK;
    if (!queries || !out) return MG_ERR_INVALID_ARGUMENT;
    const Grid g{lo_x, lo_y, lo_z, h, nx, ny, nz};
    hipLaunchKernelGGL(sdf_sample_kernel, dim3(blocks_for(n_queries, 256)), dim3(256), 0, as_stream(stream), sdf,
                       g, queries, (int64_t)n_queries, out);
    return launch_status();
}
