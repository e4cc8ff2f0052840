// Fisheye TSDF fusion kernels (Sec. III-C): allocation of voxel blocks along
// the truncation segment of every depth pixel's Eq. (1) ray, the list of
// blocks in view, and the running average of Eq. (2) over their voxels.
//
// The map is a box of nx x ny x nz blocks stored in as many slots; block
// (bx, by, bz) lives in slot ((bz mod nz) ny + (by mod ny)) nx + (bx mod nx).
// Inside the box no two blocks share a slot, so a block is allocated by
// writing its packed coordinates over an empty or a left-behind key, and a
// box that moves only has to empty the slots whose blocks it left.
//
// Three launches an integration, since each costs about 2 us beside its work:
// allocate, blocks (observation counts, left-behind slots, the list of blocks
// in view), integrate.  A new block's voxels are not initialised: its `fresh`
// flag stands for D = 1, w = 0 in all of them until the block is integrated.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tsdf_internal.h"

namespace psw {

namespace {

constexpr unsigned long long kValid = 1ull << 63;
constexpr int kCoordBias = 1 << 20;

__device__ __forceinline__ unsigned long long pack_block(int bx, int by, int bz) {
    return kValid | (unsigned long long)(bx + kCoordBias) | ((unsigned long long)(by + kCoordBias) << 21) |
           ((unsigned long long)(bz + kCoordBias) << 42);
}
__device__ __forceinline__ void unpack_block(unsigned long long k, int *bx, int *by, int *bz) {
    *bx = (int)(k & 0x1fffffull) - kCoordBias;
    *by = (int)((k >> 21) & 0x1fffffull) - kCoordBias;
    *bz = (int)((k >> 42) & 0x1fffffull) - kCoordBias;
}
// place along axis i of the slot grid of the box's block c (0 <= c < nb[i])
__device__ __forceinline__ int place(const TsdfDev &T, int i, int c) {
    const int p = T.w0[i] + c;
    return p >= T.nb[i] ? p - T.nb[i] : p;
}
// camera point of a box-relative world point
__device__ __forceinline__ void to_cam(const TsdfDev &T, float x, float y, float z, float *c) {
    c[0] = fmaf(T.R[0], x, fmaf(T.R[1], y, fmaf(T.R[2], z, T.t[0])));
    c[1] = fmaf(T.R[3], x, fmaf(T.R[4], y, fmaf(T.R[5], z, T.t[1])));
    c[2] = fmaf(T.R[6], x, fmaf(T.R[7], y, fmaf(T.R[8], z, T.t[2])));
}
// unified-model projection; false behind the model's viewpoint
__device__ __forceinline__ bool project(const TsdfDev &T, const float *c, float *u, float *v, float *range) {
    const float m = sqrtf(fmaf(c[0], c[0], fmaf(c[1], c[1], c[2] * c[2])));
    const float den = fmaf(T.xi, m, c[2]);
    *range = m;
    if (!(den > 0.0f)) return false;
    *u = fmaf(T.fx, c[0] / den, T.cx);
    *v = fmaf(T.fy, c[1] / den, T.cy);
    return true;
}

}  // namespace

__global__ void tsdf_reset_kernel(TsdfDev T) {
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < T.nslots; s += gridDim.x * blockDim.x) {
        T.keys[s] = 0ull;
        T.count[s] = 0;
        T.seen[s] = 0;
        T.fresh[s] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) T.counters[0] = 0;
}

// a word that threads of other waves read and write in the same launch, in no
// order that matters: relaxed, and served by the caches like any other (the
// same instructions)
template <typename V> __device__ __forceinline__ V load_shared(const V *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
template <typename V> __device__ __forceinline__ void store_shared(V *p, V v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// One thread per depth pixel: walk the blocks its truncation segment crosses
// (a 3-D digital differential analyser in block units), mark them seen and
// allocate those that are not.  Bound by the latency of its reads of the slots'
// keys and marks.  Every thread that meets a block writes the same words, none
// of which depends on what the others wrote, so the reads are cached loads (a
// thread that misses another's stores only repeats them) and there is no
// compare-and-swap.  The rest is arithmetic: 15 divisions a pixel.  1024x768:
// 18.3 (11 in the best launches) -> 11 us.  Also clears the next kernel's counter.
__global__ __launch_bounds__(256) void tsdf_alloc_kernel(TsdfDev T) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.y == 0 && threadIdx.x == 0) T.counters[0] = 0;
    const int u = blockIdx.x * blockDim.x + threadIdx.x, v = blockIdx.y * blockDim.y + threadIdx.y;
    if (u >= T.w || v >= T.h) return;
    const float d = T.depth[(int64_t)v * T.pitch + u];
    if (!(d > 0.0f) || !(d < 3.0e38f)) return;
    // Eq. (1): unit ray of the pixel
    const float x = ((float)u - T.cx) / T.fx, y = ((float)v - T.cy) / T.fy;
    const float q = fmaf(x, x, y * y);
    const float disc = fmaf(1.0f - T.xi * T.xi, q, 1.0f);
    if (disc < 0.0f) return;
    const float eta = (T.xi + sqrtf(disc)) / (q + 1.0f);
    const float r[3] = {eta * x, eta * y, eta - T.xi};
    const float l0 = fmaxf(d - T.mu, 0.0f), l1 = d + T.mu;
    // segment ends in box-relative world coordinates: R^T (l r - t), in blocks
    const float c0 = l0 * r[0] - T.t[0], c1 = l0 * r[1] - T.t[1], c2 = l0 * r[2] - T.t[2];
    const float d0 = l1 * r[0] - T.t[0], d1 = l1 * r[1] - T.t[1], d2 = l1 * r[2] - T.t[2];
    float a[3], e[3];
    for (int i = 0; i < 3; ++i) {
        a[i] = fmaf(T.R[0 * 3 + i], c0, fmaf(T.R[1 * 3 + i], c1, T.R[2 * 3 + i] * c2)) / T.block;
        e[i] = fmaf(T.R[0 * 3 + i], d0, fmaf(T.R[1 * 3 + i], d1, T.R[2 * 3 + i] * d2)) / T.block;
    }
    int cur[3], step[3];
    float tmax[3], tdel[3];
    for (int i = 0; i < 3; ++i) {
        cur[i] = (int)floorf(a[i]);
        const float dir = e[i] - a[i];
        if (dir > 0.0f) {
            step[i] = 1; tmax[i] = ((float)(cur[i] + 1) - a[i]) / dir; tdel[i] = 1.0f / dir;
        } else if (dir < 0.0f) {
            step[i] = -1; tmax[i] = ((float)cur[i] - a[i]) / dir; tdel[i] = -1.0f / dir;
        } else {
            step[i] = 0; tmax[i] = 3.0e38f; tdel[i] = 3.0e38f;
        }
    }
    // a segment of length L blocks crosses at most L + 3 block faces
    for (int it = 0; it < 64; ++it) {
        if (cur[0] >= 0 && cur[0] < T.nb[0] && cur[1] >= 0 && cur[1] < T.nb[1] && cur[2] >= 0 && cur[2] < T.nb[2]) {
            const int s = (place(T, 2, cur[2]) * T.nb[1] + place(T, 1, cur[1])) * T.nb[0] + place(T, 0, cur[0]);
            const unsigned long long key = pack_block(T.b0[0] + cur[0], T.b0[1] + cur[1], T.b0[2] + cur[2]);
            const unsigned long long had = load_shared(T.keys + s);
            const int marked = load_shared(T.seen + s);
            if (had != key) {
                store_shared(T.count + s, 0);
                store_shared(T.fresh + s, 1);
                store_shared(T.keys + s, key);
            }
            if (!marked) store_shared(T.seen + s, 1);
        }
        const int ax = tmax[0] <= tmax[1] ? (tmax[0] <= tmax[2] ? 0 : 2) : (tmax[1] <= tmax[2] ? 1 : 2);
        if (tmax[ax] > 1.0f) break;
        cur[ax] += step[ax];
        tmax[ax] += tdel[ax];
    }
}

// Eight lanes per slot, one block corner each: empty the slots whose blocks
// lie outside the box, count the observations, and list the allocated blocks
// with a corner in view, with one atomic a wave that has any (an atomic on one
// address costs some 10 ns even so; counting the allocated blocks here as well
// took the kernel from 6.5 to 11 us).
__global__ __launch_bounds__(256) void tsdf_blocks_kernel(TsdfDev T) {
    const int lane = threadIdx.x & 63, c = lane & 7;
    const int s = (blockIdx.x * 256 + threadIdx.x) >> 3;
    const unsigned long long k = s < T.nslots ? T.keys[s] : 0ull;
    int bx = 0, by = 0, bz = 0;
    bool in = false, vis = false;
    if (k) {
        unpack_block(k, &bx, &by, &bz);
        in = bx >= T.b0[0] && bx < T.b0[0] + T.nb[0] && by >= T.b0[1] && by < T.b0[1] + T.nb[1] &&
             bz >= T.b0[2] && bz < T.b0[2] + T.nb[2];
        if (c == 0) {
            if (!in) {
                T.keys[s] = 0ull;
                T.count[s] = 0;
            } else if (T.seen[s]) {
                T.count[s] += 1;
                T.seen[s] = 0;
            }
        }
    }
    if (in) {
        const float ox = (float)(bx - T.b0[0]) * T.block, oy = (float)(by - T.b0[1]) * T.block;
        const float oz = (float)(bz - T.b0[2]) * T.block;
        float cc[3], u, v, rg;
        to_cam(T, ox + ((c & 1) ? T.block : 0.0f), oy + ((c & 2) ? T.block : 0.0f), oz + ((c & 4) ? T.block : 0.0f),
               cc);
        vis = project(T, cc, &u, &v, &rg) && u >= 0.0f && v >= 0.0f && u <= (float)(T.w - 1) && v <= (float)(T.h - 1);
    }
    // bit 0 of each slot's eight lanes: a corner in view
    uint64_t m = __builtin_amdgcn_ballot_w64(vis);
    m |= m >> 4; m |= m >> 2; m |= m >> 1;
    m &= 0x0101010101010101ull;
    if (m == 0) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(T.counters + 0, __popcll(m));
    at = __builtin_amdgcn_readfirstlane(at);
    if ((m >> lane) & 1ull) T.list[at + __popcll(m & ((1ull << lane) - 1))] = s;
}

// Eq. (2) over the listed blocks, one workgroup a block in turn, two
// neighbouring voxels per thread.  A fresh block's voxels are not read: all
// stand for D = 1, w = 0, and all are written.
typedef float F2 __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(256) void tsdf_integrate_kernel(TsdfDev T) {
    const int n = T.counters[0];
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int s = T.list[i];
        const bool fresh = T.fresh[s] != 0;
        int bx, by, bz;
        unpack_block(T.keys[s], &bx, &by, &bz);
        const int rx = (bx - T.b0[0]) * 8, ry = (by - T.b0[1]) * 8, rz = (bz - T.b0[2]) * 8;
        const int e0 = 2 * threadIdx.x;
        F2 *const pd = reinterpret_cast<F2 *>(T.D + (int64_t)s * kBlockVox + e0);
        F2 *const pw = reinterpret_cast<F2 *>(T.W + (int64_t)s * kBlockVox + e0);
        F2 D = {1.0f, 1.0f}, W = {0.0f, 0.0f};
        if (!fresh) {
            D = *pd;
            W = *pw;
        }
        bool changed = fresh;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = e0 + h;
            const float X = ((float)(rx + (e & 7)) + 0.5f) * T.voxel;
            const float Y = ((float)(ry + ((e >> 3) & 7)) + 0.5f) * T.voxel;
            const float Z = ((float)(rz + (e >> 6)) + 0.5f) * T.voxel;
            float c[3], u, v, range;
            to_cam(T, X, Y, Z, c);
            if (!project(T, c, &u, &v, &range)) continue;
            const float fu = floorf(u + 0.5f), fv = floorf(v + 0.5f);   // nearest pixel
            if (!(fu >= 0.0f && fv >= 0.0f && fu <= (float)(T.w - 1) && fv <= (float)(T.h - 1))) continue;
            const float d_obs = T.depth[(int64_t)fv * T.pitch + (int64_t)fu];
            if (!(d_obs > 0.0f) || !(d_obs < 3.0e38f)) continue;
            const float eta = d_obs - range;
            if (eta < -T.mu) continue;
            const float w = W[h];
            D[h] = (w * D[h] + fminf(1.0f, eta / T.mu)) / (w + 1.0f);
            W[h] = fminf(w + 1.0f, T.w_max);
            changed = true;
        }
        if (changed) {
            *pd = D;
            *pw = W;
        }
        if (fresh) {
            __syncthreads();   // every thread has read the flag
            if (threadIdx.x == 0) T.fresh[s] = 0;
        }
    }
}

// Dense copy of the box in world order: a wave per row of voxels along x (or as
// many rows as fill its lanes, in boxes of up to 16 blocks along x), four voxels
// (half a block's row) per lane and step, so that a block's key and its voxels
// are read by 16-byte loads and the copy is written by 16-byte stores.
// Bound by its writes (75 x 4 x 75 blocks, 92 MB: 59.7 -> 18.2 us, 5.1 TB/s; one
// voxel per thread with divisions by the box's sizes before).  A call, one row a
// wave and then shared waves: 1 x 64 x 64 blocks 44.6 -> 10.1 us, 4 x 16 x 128
// 25.3 -> 10.0.
typedef float F4 __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void tsdf_extract_kernel(TsdfDev T, float *out_d, float *out_w, int32_t *out_count) {
    const int ny = T.nb[1] * 8;
    const int64_t rows = (int64_t)ny * T.nb[2] * 8;
    const int quads = T.nb[0] * 2, lane = threadIdx.x & 63;
    const int per = tsdf_extract_rows(T.nb[0]), sub = per > 1 ? lane / quads : 0;
    if (sub >= per) return;
    for (int64_t r = (blockIdx.x * 4ll + (threadIdx.x >> 6)) * per + sub; r < rows; r += gridDim.x * 4ll * per) {
        const int z = (int)(r / ny), y = (int)(r - (int64_t)z * ny);
        const int by = T.b0[1] + (y >> 3), bz = T.b0[2] + (z >> 3);
        const int line = (place(T, 2, z >> 3) * T.nb[1] + place(T, 1, y >> 3)) * T.nb[0];
        for (int q = lane - sub * quads; q < quads; q += 64) {
            const int s = line + place(T, 0, q >> 1);
            const bool here = T.keys[s] == pack_block(T.b0[0] + (q >> 1), by, bz);
            const int seen = here ? T.count[s] : 0;
            F4 D, W = {0.0f, 0.0f, 0.0f, 0.0f};
            const float nan = __builtin_nanf("");
            D[0] = nan; D[1] = nan; D[2] = nan; D[3] = nan;
            if (here && !T.fresh[s]) {
                const int64_t v = (int64_t)s * kBlockVox + ((z & 7) * 8 + (y & 7)) * 8 + (q & 1) * 4;
                W = *reinterpret_cast<const F4 *>(T.W + v);
                if (out_d && seen >= T.min_obs) {
                    const F4 d = *reinterpret_cast<const F4 *>(T.D + v);
#pragma unroll
                    for (int i = 0; i < 4; ++i) D[i] = W[i] > 0.0f ? d[i] : nan;
                }
            }
            const int64_t o = r * (quads * 4ll) + q * 4;
            if (out_w) *reinterpret_cast<F4 *>(out_w + o) = W;
            if (out_d) *reinterpret_cast<F4 *>(out_d + o) = D;
            if (out_count && (q & 1) == 0 && (y & 7) == 0 && (z & 7) == 0)
                out_count[((int64_t)(z >> 3) * T.nb[1] + (y >> 3)) * T.nb[0] + (q >> 1)] = seen;
        }
    }
}

// Allocated blocks (counted now: the integrations keep no count of them, which
// would cost each of those 4.5 us of atomics) and the blocks listed by the last
// integration.  The workgroups' counts are added to a cleared word; one
// workgroup, for maps whose keys it reads in less than that launch takes, writes
// it itself (a call: 22,500 slots 7.4 us, 32,768 8.6; one workgroup and then
// several: 65,536 slots 12.0 and 8.8, 262,144 34.6 and 8.7, 2^22 1,127 and 11.8).
__global__ void tsdf_stats_clear_kernel(TsdfDev T, int32_t *out) {
    if (threadIdx.x == 0) {
        out[0] = 0;
        out[1] = T.counters[0];
    }
}
__global__ __launch_bounds__(1024) void tsdf_stats_kernel(TsdfDev T, int32_t *out) {
    __shared__ int total;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    int n = 0;
    for (int s = blockIdx.x * 1024 + threadIdx.x; s < T.nslots; s += gridDim.x * 1024) n += T.keys[s] != 0ull;
    atomicAdd(&total, n);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (gridDim.x > 1) {
            atomicAdd(out, total);
        } else {
            out[0] = total;
            out[1] = T.counters[0];
        }
    }
}

}  // namespace psw

extern "C" {
const void *psw_tsdf_kernel(int which) {
    switch (which) {
    case 0: return (const void *)&psw::tsdf_reset_kernel;
    case 1: return (const void *)&psw::tsdf_alloc_kernel;
    case 2: return (const void *)&psw::tsdf_blocks_kernel;
    case 3: return (const void *)&psw::tsdf_integrate_kernel;
    case 4: return (const void *)&psw::tsdf_extract_kernel;
    case 5: return (const void *)&psw::tsdf_stats_kernel;
    case 6: return (const void *)&psw::tsdf_stats_clear_kernel;
    }
    return nullptr;
}
}
