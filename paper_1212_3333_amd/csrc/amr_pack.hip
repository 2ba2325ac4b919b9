// Packing on the GPU: ghost layers (Section 5), bricks and value ranges of cell-centred patches.
//
// The host sends the cells as they are; the kernels form the ghost layers in FP64 by the host
// packer's rules (coarser levels before finer ones), lay the bricks out in the pool and reduce the
// value ranges.  The pool has 2.2 floats per cell in the halo-row layout, so sending the cells instead
// of the bricks halves the copy, and no host pass over the data is left.  What bounds it: the
// copy of the cells from pageable memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "amr_pack.h"

namespace amr {

namespace {

// floor division, b > 0
__device__ inline int64_t fdiv_d(int64_t a, int64_t b) {
    const int64_t q = a / b;
    return (a % b != 0 && a < 0) ? q - 1 : q;
}

// Value of padded cell (i, j, k) (-1 and n: the ghost layer, FP64).
__device__ inline double padded(const PackPatch &P, const float *cells, const double *shell, int64_t i, int64_t j, int64_t k) {
    if (i >= 0 && j >= 0 && k >= 0 && i < P.n[0] && j < P.n[1] && k < P.n[2])
        return (double)cells[P.cells + i + P.n[0] * (j + P.n[1] * k)];
    return shell[P.shell + shell_index(P.n, i, j, k)];
}

__device__ inline bool holds(const PackPatch &Q, const int64_t c2[3]) {
    bool in = true;
    for (int a = 0; a < 3; a++) in = in && c2[a] >= 2 * Q.blo[a] && c2[a] < 2 * Q.bhi[a];
    return in;
}

// Trilinear value of coarser patch Q (its ghost layer complete) at c2, twice a finest-level coordinate.
__device__ inline double coarse_interp(const PackPatch &Q, const float *cells, const double *shell, const int64_t c2[3]) {
#pragma clang fp contract(off)
    int64_t i0[3];
    double f[3];
    for (int a = 0; a < 3; a++) {
        const int64_t num = c2[a] - 2 * Q.blo[a] - Q.scale, den = 2 * Q.scale;
        i0[a] = fdiv_d(num, den);
        f[a] = (double)(num - i0[a] * den) / (double)den;
    }
    double v[2][2][2];
    for (int dz = 0; dz < 2; dz++)
        for (int dy = 0; dy < 2; dy++)
            for (int dx = 0; dx < 2; dx++) v[dz][dy][dx] = padded(Q, cells, shell, i0[0] + dx, i0[1] + dy, i0[2] + dz);
    const double x00 = v[0][0][0] + f[0] * (v[0][0][1] - v[0][0][0]);
    const double x10 = v[0][1][0] + f[0] * (v[0][1][1] - v[0][1][0]);
    const double x01 = v[1][0][0] + f[0] * (v[1][0][1] - v[1][0][0]);
    const double x11 = v[1][1][0] + f[0] * (v[1][1][1] - v[1][1][0]);
    const double y0 = x00 + f[1] * (x10 - x00);
    const double y1 = x01 + f[1] * (x11 - x01);
    return y0 + f[2] * (y1 - y0);
}

struct Box2 {
    int64_t lo[3], hi[3];            // the root box
};

// The ghost layers of one level's patches: blockIdx.x the patch, blockIdx.y and the threads its shell.
// g1 a same-level patch holding the ghost's centre (exact copy); g2 a centre outside B is clamped into
// it and g1 asked again; g3 the finest coarser patch holding it; g4 the nearest own cell.
__global__ __launch_bounds__(256) void ghost_kernel(const PackPatch *patches, const int32_t *ids, const int32_t *nbr,
                                                    const float *cells, double *shell, Box2 B) {
    const PackPatch &P = patches[ids[blockIdx.x]];
    const int64_t total = shell_count(P.n);
    const int64_t sx = P.n[0] + 2, sy = P.n[1] + 2;
    for (int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.y * 256) {
        int64_t r = e, idx[3];
        if (r < 2 * sx * sy) {
            const bool up = r >= sx * sy;
            if (up) r -= sx * sy;
            idx[0] = r % sx - 1;
            idx[1] = r / sx - 1;
            idx[2] = up ? P.n[2] : -1;
        } else if ((r -= 2 * sx * sy) < 2 * sx * P.n[2]) {
            const bool up = r >= sx * P.n[2];
            if (up) r -= sx * P.n[2];
            idx[0] = r % sx - 1;
            idx[1] = up ? P.n[1] : -1;
            idx[2] = r / sx;
        } else {
            r -= 2 * sx * P.n[2];
            const bool up = r >= (int64_t)P.n[1] * P.n[2];
            if (up) r -= (int64_t)P.n[1] * P.n[2];
            idx[0] = up ? P.n[0] : -1;
            idx[1] = r % P.n[1];
            idx[2] = r / P.n[1];
        }
        int64_t c2[3];
        for (int a = 0; a < 3; a++) c2[a] = (2 * (P.lo[a] + idx[a]) + 1) * P.scale;
        double val = 0.0;
        bool done = false;
        for (int pass = 0; pass < 2 && !done; pass++) {
            int best = -1, best_level = -1;
            for (int q = P.nbr0; q < P.nbr1; q++) {
                const PackPatch &Q = patches[nbr[q]];
                if (!holds(Q, c2)) continue;
                if (Q.level == P.level) {
                    int64_t m[3];
                    for (int a = 0; a < 3; a++) m[a] = (c2[a] - P.scale) / (2 * P.scale) - Q.lo[a];
                    val = (double)cells[Q.cells + m[0] + Q.n[0] * (m[1] + Q.n[1] * m[2])];
                    done = true;
                    break;
                }
                if (Q.level > best_level) {
                    best = nbr[q];
                    best_level = Q.level;
                }
            }
            if (done) break;
            bool moved = false;
            for (int a = 0; a < 3; a++) {
                const int64_t lo = 2 * B.lo[a] + P.scale, hi = 2 * B.hi[a] - P.scale;
                if (c2[a] < lo) { c2[a] = lo; moved = true; }
                if (c2[a] > hi) { c2[a] = hi; moved = true; }
            }
            if (moved && pass == 0) continue;
            if (best >= 0) {
                val = coarse_interp(patches[best], cells, shell, c2);
                done = true;
            }
            break;
        }
        if (!done) {
            int64_t m[3];
            for (int a = 0; a < 3; a++) m[a] = min(max(idx[a], (int64_t)0), (int64_t)P.n[a] - 1);
            val = (double)cells[P.cells + m[0] + P.n[0] * (m[1] + P.n[1] * m[2])];
        }
        shell[P.shell + e] = val;
    }
}

// One patch's brick in the pool (blockIdx.x the patch), 16 bytes per thread and step; floats outside the
// padded brick are zero.  The pads before the first and after the last brick are cleared too.
__global__ __launch_bounds__(256) void brick_kernel(const PackPatch *patches, int np, int layout, const float *cells,
                                                    const double *shell, float *pool, int64_t pool_floats) {
    const PackPatch &P = patches[blockIdx.x];
    const int64_t pn[3] = {P.n[0] + 2, P.n[1] + 2, P.n[2] + 2};
    float4 *out = reinterpret_cast<float4 *>(pool + P.pool);
    for (int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x; e < P.floats / 4; e += (int64_t)gridDim.y * 256) {
        float v[4];
        int64_t i, j, k;             // padded index of the first of the four, along x
        if (layout == 0) {
            k = -1;
            i = j = 0;               // a row's end may lie among the four: one by one below
        } else {
            const int sh = layout == 2 ? 5 : 4;      // 16-byte groups per block
            const uint32_t blk = (uint32_t)(e >> sh), w = (uint32_t)e & ((1u << sh) - 1u);
            const uint32_t bx = blk % (uint32_t)P.nb[0], t = blk / (uint32_t)P.nb[0];
            const uint32_t by = t % (uint32_t)P.nb[1], bz = t / (uint32_t)P.nb[1];
            const uint32_t row = layout == 2 ? w >> 1 : w;
            i = layout == 2 ? 4 * (int64_t)bx - 1 + 4 * (w & 1u) : 4 * (int64_t)bx;
            j = 4 * (int64_t)by + (row & 3u);
            k = 4 * (int64_t)bz + (row >> 2);
        }
        #pragma unroll
        for (int c = 0; c < 4; c++) {
            int64_t x = i + c, y = j, z = k;
            if (layout == 0) {
                const int64_t f = 4 * e + c;
                x = f % pn[0];
                y = f / pn[0] % pn[1];
                z = f / pn[0] / pn[1];
            }
            const bool in = x >= 0 && x < pn[0] && y < pn[1] && z < pn[2];
            v[c] = in ? (float)padded(P, cells, shell, x - 1, y - 1, z - 1) : 0.f;
        }
        out[e] = make_float4(v[0], v[1], v[2], v[3]);
    }
    if (blockIdx.y == 0 && threadIdx.x < 64) {
        if (blockIdx.x == 0) pool[threadIdx.x] = 0.f;
        if ((int)blockIdx.x == np - 1) pool[pool_floats - 64 + threadIdx.x] = 0.f;
    }
}

// Block-wide range (std::min's and std::max's treatment of NaN: never taken).
__device__ inline void range_reduce(float &mn, float &mx, float *s) {
    for (int o = 32; o > 0; o >>= 1) {
        const float a = __shfl_xor(mn, o, 64), b = __shfl_xor(mx, o, 64);
        mn = a < mn ? a : mn;
        mx = mx < b ? b : mx;
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s[2 * wave] = mn;
        s[2 * wave + 1] = mx;
    }
    __syncthreads();
    for (int w = 0; w < (int)(blockDim.x >> 6); w++) {
        mn = s[2 * w] < mn ? s[2 * w] : mn;
        mx = mx < s[2 * w + 1] ? s[2 * w + 1] : mx;
    }
}

__global__ __launch_bounds__(256) void patch_range_kernel(const PackPatch *patches, const float *cells, const double *shell,
                                                          DPatch *headers, float *ranges) {
    __shared__ float s[8];
    const PackPatch &P = patches[blockIdx.x];
    float mn = INFINITY, mx = -INFINITY;
    const int64_t nc = (int64_t)P.n[0] * P.n[1] * P.n[2], ns = shell_count(P.n);
    for (int64_t e = threadIdx.x; e < nc; e += 256) {
        const float v = cells[P.cells + e];
        mn = v < mn ? v : mn;
        mx = mx < v ? v : mx;
    }
    for (int64_t e = threadIdx.x; e < ns; e += 256) {
        const float v = (float)shell[P.shell + e];
        mn = v < mn ? v : mn;
        mx = mx < v ? v : mx;
    }
    range_reduce(mn, mx, s);
    if (threadIdx.x == 0) {
        headers[blockIdx.x].vmin = mn;
        headers[blockIdx.x].vmax = mx;
        ranges[2 * (int64_t)blockIdx.x] = mn;
        ranges[2 * (int64_t)blockIdx.x + 1] = mx;
    }
}

__global__ __launch_bounds__(256) void leaf_range_kernel(const PackPatch *patches, const PackLeaf *leaves, const float *cells,
                                                         const double *shell, DLeaf *records) {
    __shared__ float s[8];
    const PackLeaf L = leaves[blockIdx.x];
    if (L.patch < 0) return;
    const PackPatch &P = patches[L.patch];
    const int32_t wx = L.hi[0] - L.lo[0] + 1, wy = L.hi[1] - L.lo[1] + 1, wz = L.hi[2] - L.lo[2] + 1;
    float mn = INFINITY, mx = -INFINITY;
    // a wave per row of the box
    for (int64_t r = threadIdx.x >> 6; r < (int64_t)wy * wz; r += 4) {
        const int64_t y = L.lo[1] + (int32_t)(r % wy), z = L.lo[2] + (int32_t)(r / wy);
        for (int32_t x = threadIdx.x & 63; x < wx; x += 64) {
            const float v = (float)padded(P, cells, shell, L.lo[0] + x, y, z);
            mn = v < mn ? v : mn;
            mx = mx < v ? v : mx;
        }
    }
    range_reduce(mn, mx, s);
    if (threadIdx.x == 0) {
        records[blockIdx.x].vmin = mn;
        records[blockIdx.x].vmax = mx;
    }
}

// f(first, count) over 0 .. n in parts of as many blocks of 256 threads as a launch takes (fewer than 2^32
// threads along a grid's x axis).
constexpr int64_t kPart = 1 << 22;
static_assert(kPart * 256 < (int64_t)1 << 32, "threads of one launch");
template <typename F>
void in_parts(int64_t n, F f) {
    for (int64_t k = 0; k < n; k += kPart) f(k, (uint32_t)std::min(kPart, n - k));
}

int64_t up256(int64_t b) { return (b + 255) / 256 * 256; }

int hip_failed(hipError_t e, const char *what) {
    if (e == hipSuccess) return AMR_OK;
    set_error("%s: %s", what, hipGetErrorString(e));
    return AMR_EHIP;
}

// Null where there is no room.
void *stage_take(const PackStage &st, int64_t bytes) {
    void *p = nullptr;
    if (hipMallocFromPoolAsync(&p, (size_t)bytes, (hipMemPool_t)st.pool, (hipStream_t)st.stream) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

}  // namespace

bool pack_stage_alloc(const PackPlan &plan, int64_t nleaves, int device, void *stream, PackStage *st) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = device;
    hipMemPool_t pool = nullptr;
    if (hipStreamIsCapturing((hipStream_t)stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone ||
        hipMemPoolCreate(&pool, &props) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    st->pool = pool;
    const int64_t np = (int64_t)plan.patches.size();
    const int64_t bytes = up256(4 * plan.cell_floats) + up256(8 * plan.shell_doubles) +
                          up256(np * (int64_t)sizeof(PackPatch)) + up256(4 * np) +
                          up256(nleaves * (int64_t)sizeof(PackLeaf)) + up256(8 * np);
    st->stream = stream;
    st->mem = stage_take(*st, bytes);
    if (!st->mem) return false;
    char *p = (char *)st->mem;
    auto take = [&](int64_t b) {
        char *q = p;
        p += up256(b);
        return q;
    };
    st->cells = (float *)take(4 * plan.cell_floats);
    st->shell = (double *)take(8 * plan.shell_doubles);
    st->patches = (PackPatch *)take(np * (int64_t)sizeof(PackPatch));
    st->ids = (int32_t *)take(4 * np);
    st->leaves = (PackLeaf *)take(nleaves * (int64_t)sizeof(PackLeaf));
    st->ranges = (float *)take(8 * np);
    return true;
}

bool pack_stage_neighbours(const PackPlan &plan, PackStage *st) {
    st->nbr = (int32_t *)stage_take(*st, std::max<int64_t>(4 * (int64_t)plan.nbr.size(), 256));
    return st->nbr != nullptr;
}

void pack_stage_free(PackStage *st) {
    if (!st->pool) return;
    hipStream_t s = (hipStream_t)st->stream;
    if (st->nbr) (void)hipFreeAsync(st->nbr, s);
    if (st->mem) (void)hipFreeAsync(st->mem, s);
    (void)hipStreamSynchronize(s);
    (void)hipMemPoolDestroy((hipMemPool_t)st->pool);
    st->mem = st->pool = nullptr;
    st->nbr = nullptr;
}

int pack_upload_cells(const PackPlan &plan, const PackStage &st, int device) {
    hipError_t e = hipSetDevice(device);
    for (size_t p = 0; e == hipSuccess && p < plan.patches.size(); p++) {
        const PackPatch &P = plan.patches[p];
        e = hipMemcpyAsync(st.cells + P.cells, plan.cells[p], 4 * (size_t)P.n[0] * P.n[1] * P.n[2], hipMemcpyHostToDevice,
                           (hipStream_t)st.stream);
    }
    const hipError_t w = hipStreamSynchronize((hipStream_t)st.stream);
    return hip_failed(e != hipSuccess ? e : w, "copy of the cells");
}

int pack_run(const PackPlan &plan, const PackStage &st, void *d_pool, void *d_meta, const void *meta, int64_t meta_bytes,
             int64_t o_leaves, int64_t o_patch, float *vmin, float *vmax, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    const int np = (int)plan.patches.size();
    std::vector<int32_t> ids;
    std::vector<float> r(2 * (size_t)np);
    struct Wait {                      // on every way out: copies read and write the host memory above
        hipStream_t s;
        ~Wait() { (void)hipStreamSynchronize(s); }
    } wait{s};
    for (const auto &l : plan.levels) ids.insert(ids.end(), l.begin(), l.end());
    auto send = [&](void *dst, const void *src, size_t bytes) {
        return bytes ? hip_failed(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s), "copy of the packing tables") : AMR_OK;
    };
    int rc = send(st.patches, plan.patches.data(), plan.patches.size() * sizeof(PackPatch));
    if (!rc) rc = send(st.nbr, plan.nbr.data(), plan.nbr.size() * 4);
    if (!rc) rc = send(st.ids, ids.data(), ids.size() * 4);
    if (!rc) rc = send(st.leaves, plan.leaves.data(), plan.leaves.size() * sizeof(PackLeaf));
    if (!rc) rc = send(d_meta, meta, (size_t)meta_bytes);
    if (rc) return rc;
    Box2 B;
    for (int a = 0; a < 3; a++) {
        B.lo[a] = plan.B_lo[a];
        B.hi[a] = plan.B_hi[a];
    }
    auto chunks = [](int64_t work) { return (uint32_t)std::min<int64_t>(std::max<int64_t>((work + 255) / 256, 1), 1024); };
    size_t first = 0;
    for (const auto &l : plan.levels) {          // coarser ghost layers are complete before finer ones
        if (l.empty()) continue;
        int64_t most = 1;
        for (int32_t p : l) most = std::max(most, shell_count(plan.patches[p].n));
        in_parts((int64_t)l.size(), [&](int64_t k, uint32_t n) {
            hipLaunchKernelGGL(ghost_kernel, dim3(n, chunks(most)), dim3(256), 0, s, st.patches, st.ids + first + k, st.nbr,
                               st.cells, st.shell, B);
        });
        first += l.size();
    }
    int64_t most = 1;
    for (const PackPatch &P : plan.patches) most = std::max(most, P.floats / 4);
    DPatch *headers = (DPatch *)((char *)d_meta + o_patch);
    DLeaf *records = (DLeaf *)((char *)d_meta + o_leaves);
    in_parts(np, [&](int64_t k, uint32_t n) {
        hipLaunchKernelGGL(brick_kernel, dim3(n, chunks(most)), dim3(256), 0, s, st.patches + k, np - (int)k, plan.layout,
                           st.cells, st.shell, (float *)d_pool, plan.pool_floats);
        hipLaunchKernelGGL(patch_range_kernel, dim3(n), dim3(256), 0, s, st.patches + k, st.cells, st.shell, headers + k,
                           st.ranges + 2 * k);
    });
    in_parts((int64_t)plan.leaves.size(), [&](int64_t k, uint32_t n) {
        hipLaunchKernelGGL(leaf_range_kernel, dim3(n), dim3(256), 0, s, st.patches, st.leaves + k, st.cells, st.shell,
                           records + k);
    });
    rc = hip_failed(hipGetLastError(), "packing kernels");
    if (rc) return rc;
    rc = hip_failed(hipMemcpyAsync(r.data(), st.ranges, r.size() * 4, hipMemcpyDeviceToHost, s), "value ranges");
    if (!rc) rc = hip_failed(hipStreamSynchronize(s), "packing kernels");
    if (rc) return rc;
    *vmin = INFINITY;
    *vmax = -INFINITY;
    for (int p = 0; p < np; p++) {
        *vmin = std::min(*vmin, r[2 * (size_t)p]);
        *vmax = std::max(*vmax, r[2 * (size_t)p + 1]);
    }
    return AMR_OK;
}

}  // namespace amr
