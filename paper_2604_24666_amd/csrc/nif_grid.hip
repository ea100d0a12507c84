// Rest-space voxelization and the per-pose deformed acceleration grid.
//
// Methodology: the geometry is voxelized once in rest space; every pose deforms the voxels,
// and rays are traced against the deformed voxels.  Because deformed voxels no longer have
// uniform extents, the voxel under a point cannot be found by index arithmetic ("Voxel
// Traversal under Deformation"); the paper finds the first voxel with a BVH.  Here each pose
// gets a uniform bin grid over its deformed bounding box instead: every occupied voxel is
// listed in the bins its (padded) deformed box overlaps, and a ray walks the bins with a
// 3D-DDA, testing the listed voxels exactly.  The bins only narrow the search; the set of
// voxels a ray crosses, and their order, come from the exact voxel tests.
//
// Build, per pose, all on the device:
//   1 lattice vertices V_ijk = D(i/N, j/N, k/N)              (float4, x fastest)
//   2 occupied voxels compacted once (shared by all poses)
//   3 padded deformed boxes of the occupied voxels, reduced to the pose's bounding box
//   4 bin sizes; per-bin reference counts; exclusive scan; fill.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "nif_internal.hpp"

namespace nif {

// ------------------------------------------------------------------ voxelization

__global__ void k_voxelize(int32_t kind, const float* __restrict__ sp, int32_t N,
                           uint8_t* __restrict__ occ) {
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t n = (int64_t)N * N * N;
    if (c >= n) return;
    int i = (int)(c % N), j = (int)((c / N) % N), k = (int)(c / ((int64_t)N * N));
    float lo = INFINITY, hi = -INFINITY;
    const float inv = 1.f / (float)N;
    for (int cz = 0; cz <= 4; ++cz)
        for (int cy = 0; cy <= 4; ++cy)
            for (int cx = 0; cx <= 4; ++cx) {
                float3 p = make_float3((i + 0.25f * cx) * inv, (j + 0.25f * cy) * inv, (k + 0.25f * cz) * inv);
                float v = scene_f(kind, sp, p);
                lo = fminf(lo, v);
                hi = fmaxf(hi, v);
            }
    occ[c] = (lo <= 0.f && hi >= 0.f) ? 1 : 0;
}

int voxelize_launch(int32_t kind, const float* sp, int32_t N, uint8_t* occ, hipStream_t st) {
    int64_t n = (int64_t)N * N * N;
    hipLaunchKernelGGL(k_voxelize, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, kind, sp, N, occ);
    return check_hip(hipGetLastError(), "voxelize launch");
}

// ------------------------------------------------------------------ build kernels

__global__ void k_vertices(const PoseDev* __restrict__ poses, int32_t N, float4* __restrict__ V) {
    const int p = blockIdx.y;
    const PoseDev P = poses[p];
    int64_t nv = (int64_t)(N + 1) * (N + 1) * (N + 1);
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    int i = (int)(v % (N + 1)), j = (int)((v / (N + 1)) % (N + 1)), k = (int)(v / ((int64_t)(N + 1) * (N + 1)));
    const float inv = 1.f / (float)N;
    float3 q = deform(P, make_float3(i * inv, j * inv, k * inv));
    V[P.vert_off + v] = make_float4(q.x, q.y, q.z, 0.f);
}

__global__ void k_compact(const uint8_t* __restrict__ occ, int64_t n, int32_t* __restrict__ list,
                          int32_t* __restrict__ count) {
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool o = c < n && occ[c];
    uint64_t m = __ballot(o);
    int base = 0;
    if (lane_id() == 0 && m) base = atomicAdd(count, popc64(m));
    base = __shfl(base, 0);
    if (o) list[base + rank_below(m)] = (int32_t)c;
}

// Order-preserving map of floats to signed ints (for atomic min/max of floats).
__device__ inline int32_t f2ord(float f) {
    int32_t i = __float_as_int(f);
    return i >= 0 ? i : (int32_t)(i ^ 0x7fffffff);
}
__host__ inline float ord2f_host(int32_t i) {
    int32_t r = i >= 0 ? i : (int32_t)(i ^ 0x7fffffff);
    float f;
    memcpy(&f, &r, 4);
    return f;
}

__device__ inline void cell_box(const float4* __restrict__ V, int32_t N, int32_t cell, float lo[3], float hi[3]) {
    int i = cell % N, j = (cell / N) % N, k = cell / (N * N);
    lo[0] = lo[1] = lo[2] = INFINITY;
    hi[0] = hi[1] = hi[2] = -INFINITY;
    for (int m = 0; m < 8; ++m) {
        int64_t vi = (int64_t)(i + (m & 1)) + (int64_t)(N + 1) * ((j + ((m >> 1) & 1)) + (int64_t)(N + 1) * (k + (m >> 2)));
        float4 v = V[vi];
        lo[0] = fminf(lo[0], v.x); lo[1] = fminf(lo[1], v.y); lo[2] = fminf(lo[2], v.z);
        hi[0] = fmaxf(hi[0], v.x); hi[1] = fmaxf(hi[1], v.y); hi[2] = fmaxf(hi[2], v.z);
    }
    for (int a = 0; a < 3; ++a) { lo[a] -= kBinPad; hi[a] += kBinPad; }
}

// bbox[p][6] as ordered ints: min x,y,z then max x,y,z.  Few blocks per pose, one set of atomics
// each: the six addresses of a pose take one atomic at a time (one set per wave over 8 poses of the
// 128^3 scene: 214 us).
constexpr int kBoxBlocks = 48;
__global__ void k_pose_bbox(const PoseDev* __restrict__ poses, const float4* __restrict__ V, int32_t N,
                            const int32_t* __restrict__ list, int32_t n_occ, int32_t* __restrict__ bbox) {
    const int p = blockIdx.y;
    const float4* Vp = V + poses[p].vert_off;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_occ; t += (int64_t)gridDim.x * blockDim.x) {
        float a[3], b[3];
        cell_box(Vp, N, list[t], a, b);
        for (int c = 0; c < 3; ++c) { lo[c] = fminf(lo[c], a[c]); hi[c] = fmaxf(hi[c], b[c]); }
    }
    for (int c = 0; c < 3; ++c) {
        for (int off = 32; off > 0; off >>= 1) {
            lo[c] = fminf(lo[c], __shfl_xor(lo[c], off));
            hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], off));
        }
    }
    __shared__ float red[4][6];
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0)
        for (int c = 0; c < 3; ++c) { red[w][c] = lo[c]; red[w][3 + c] = hi[c]; }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int c = (int)threadIdx.x;
        float v = red[0][c];
        for (int k = 1; k < 4; ++k) v = c < 3 ? fminf(v, red[k][c]) : fmaxf(v, red[k][c]);
        if (c < 3) atomicMin(&bbox[6 * p + c], f2ord(v));
        else atomicMax(&bbox[6 * p + c], f2ord(v));
    }
}

__device__ inline void box_bins(const PoseDev& P, const float lo[3], const float hi[3], int b0[3], int b1[3]) {
    for (int a = 0; a < 3; ++a) {
        int x0 = (int)floorf((lo[a] - P.lo[a]) * P.inv_bs[a]);
        int x1 = (int)floorf((hi[a] - P.lo[a]) * P.inv_bs[a]);
        b0[a] = min(max(x0, 0), P.nb[a] - 1);
        b1[a] = min(max(x1, 0), P.nb[a] - 1);
    }
}

__global__ void k_bin_count(const PoseDev* __restrict__ poses, const float4* __restrict__ V, int32_t N,
                            const int32_t* __restrict__ list, int32_t n_occ, int32_t* __restrict__ counts) {
    const int p = blockIdx.y;
    const PoseDev P = poses[p];
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_occ || P.empty) return;
    float lo[3], hi[3];
    cell_box(V + P.vert_off, N, list[t], lo, hi);
    int b0[3], b1[3];
    box_bins(P, lo, hi, b0, b1);
    int32_t* cnt = counts + P.bin_off;
    for (int z = b0[2]; z <= b1[2]; ++z)
        for (int y = b0[1]; y <= b1[1]; ++y)
            for (int x = b0[0]; x <= b1[0]; ++x)
                atomicAdd(&cnt[x + P.nb[0] * (y + P.nb[1] * z)], 1);
}

// Exclusive scan of a pose's counts[0..n) into start[0..n] in chunks of kScanChunk bins: sums of the
// chunks, then every chunk's own scan from the sums before it (one workgroup per pose walked all
// bins alone: 505 us at 64^3 bins).
constexpr int kScanChunk = 4096;

__device__ inline int64_t pose_bins(const PoseDev& P) { return (int64_t)P.nb[0] * P.nb[1] * P.nb[2]; }

// Block (x, p): sum of chunk x of pose p.
__global__ void __launch_bounds__(256) k_chunk_sums(const PoseDev* __restrict__ poses, const int32_t* __restrict__ counts,
                                                    int32_t* __restrict__ sums, int max_chunks) {
    const PoseDev P = poses[blockIdx.y];
    const int64_t n = pose_bins(P), a = (int64_t)blockIdx.x * kScanChunk, b = min(n, a + kScanChunk);
    if (a >= n) return;
    const int32_t* c = counts + P.bin_off;
    int32_t sum = 0;
    for (int64_t i = a + threadIdx.x; i < b; i += 256) sum += c[i];
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    __shared__ int32_t red[4];
    if (lane_id() == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) sums[(int64_t)blockIdx.y * max_chunks + blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Leaves the counts cleared (the fill's cursors).
__global__ void __launch_bounds__(256) k_scan(const PoseDev* __restrict__ poses, int32_t* __restrict__ counts,
                                              const int32_t* __restrict__ sums, int max_chunks, int32_t* __restrict__ start,
                                              int32_t* __restrict__ totals) {
    const int p = blockIdx.y, T = threadIdx.x;
    const PoseDev P = poses[p];
    const int64_t n = pose_bins(P), a = (int64_t)blockIdx.x * kScanChunk;
    if (a >= n) return;
    int32_t* c = counts + P.bin_off;
    int32_t* s = start + P.bin_off;
    __shared__ int32_t part[256], before[256];
    int32_t pre = 0;                                   // the chunks before this one
    for (int k = T; k < (int)blockIdx.x; k += 256) pre += sums[(int64_t)p * max_chunks + k];
    constexpr int PER = kScanChunk / 256;
    const int64_t i0 = a + (int64_t)T * PER;
    int32_t v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        v[k] = i0 + k < n ? c[i0 + k] : 0;
        if (i0 + k < n) c[i0 + k] = 0;
        sum += v[k];
    }
    part[T] = sum;
    before[T] = pre;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int32_t x = T >= off ? part[T - off] : 0, y = T >= off ? before[T - off] : 0;
        __syncthreads();
        part[T] += x;
        before[T] += y;
        __syncthreads();
    }
    int32_t run = before[255] + part[T] - sum;         // exclusive prefix of this thread's bins
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (i0 + k < n) s[i0 + k] = run;
        run += v[k];
    }
    if (a + kScanChunk >= n && T == 255) { s[n] = run; totals[p] = run; }
}

// Per-pose offsets into the shared reference list (one thread).  A pose whose references do
// not fit the allocated capacity is marked empty (its rays then miss) and flagged.
__global__ void k_ref_offsets(PoseDev* __restrict__ poses, int n_poses, const int32_t* __restrict__ totals,
                              int64_t capacity, int32_t* __restrict__ overflow) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int64_t off = 0;
    int32_t ov = 0;
    for (int p = 0; p < n_poses; ++p) {
        poses[p].ref_off = off;
        if (off + totals[p] > capacity) { poses[p].empty = 1; ov = 1; }
        else off += totals[p];
    }
    *overflow = ov;
}

// Bin-grid origin and bin size of every pose from its bounding box (bins per axis fixed).
__global__ void k_pose_bins(PoseDev* __restrict__ poses, int n_poses, const int32_t* __restrict__ bbox, int32_t n_occ) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_poses) return;
    PoseDev& q = poses[p];
    q.empty = n_occ == 0;
    for (int c = 0; c < 3; ++c) {
        const int32_t ilo = bbox[6 * p + c], ihi = bbox[6 * p + 3 + c];
        float lo = __int_as_float(ilo >= 0 ? ilo : (ilo ^ 0x7fffffff));
        float hi = __int_as_float(ihi >= 0 ? ihi : (ihi ^ 0x7fffffff));
        if (q.empty) { lo = 0.f; hi = 1.f; }
        q.lo[c] = lo;
        q.bs[c] = fmaxf((hi - lo) / q.nb[c], 1e-6f);
        q.inv_bs[c] = 1.f / q.bs[c];
    }
}

__global__ void k_fill_i32(int32_t* __restrict__ a, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) a[i] = v;
}

__global__ void k_bbox_init(int32_t* __restrict__ bbox, int n_poses) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 6 * n_poses) return;
    bbox[i] = (i % 6) < 3 ? 0x7f800000 : (int32_t)(0xff800000u ^ 0x7fffffffu);
}

__global__ void k_bin_fill(const PoseDev* __restrict__ poses, const float4* __restrict__ V, int32_t N,
                           const int32_t* __restrict__ list, int32_t n_occ, const int32_t* __restrict__ start,
                           int32_t* __restrict__ cursor, int32_t* __restrict__ cells) {
    const int p = blockIdx.y;
    const PoseDev P = poses[p];
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_occ || P.empty) return;
    const int32_t cell = list[t];
    float lo[3], hi[3];
    cell_box(V + P.vert_off, N, cell, lo, hi);
    int b0[3], b1[3];
    box_bins(P, lo, hi, b0, b1);
    const int32_t* st = start + P.bin_off;
    int32_t* cur = cursor + P.bin_off;
    int32_t* out = cells + P.ref_off;
    const int32_t packed = pack_cell(cell, N);
    for (int z = b0[2]; z <= b1[2]; ++z)
        for (int y = b0[1]; y <= b1[1]; ++y)
            for (int x = b0[0]; x <= b1[0]; ++x) {
                int b = x + P.nb[0] * (y + P.nb[1] * z);
                out[st[b] + atomicAdd(&cur[b], 1)] = packed;
            }
}

// In memory, for lists beyond the LDS (8 poses, 4 bins per axis at 64^3: 22.5 ms a re-pose).
__device__ inline void sort_list(int32_t* __restrict__ c, int32_t first, int32_t end) {
    for (int32_t i = first + 1; i < end; ++i) {
        const int32_t v = c[i];
        int32_t j = i - 1;
        while (j >= first && c[j] > v) { c[j + 1] = c[j]; --j; }
        c[j + 1] = v;
    }
}

// Sort each bin's list by packed voxel, that is by voxel id, so that the build is deterministic
// (insertion sort; lists are short).  A block takes 128 neighbouring bins, whose lists are one range
// of the references: it is sorted in LDS where it fits, so that the chains of a sort are LDS reads.
constexpr int kSortBins = 128, kSortRefs = 3072;
__global__ void __launch_bounds__(kSortBins) k_bin_sort(const PoseDev* __restrict__ poses, const int32_t* __restrict__ start,
                                                        int32_t* __restrict__ cells) {
    __shared__ int32_t s_ref[kSortRefs];
    const int p = blockIdx.y;
    const PoseDev P = poses[p];
    const int64_t nb = pose_bins(P);
    const int64_t b0 = (int64_t)blockIdx.x * kSortBins, b = b0 + threadIdx.x;
    if (b0 >= nb || P.empty) return;
    const int32_t* st = start + P.bin_off;
    int32_t* c = cells + P.ref_off;
    const int32_t r0 = st[b0], r1 = st[min(nb, b0 + kSortBins)];
    const bool staged = r1 - r0 <= kSortRefs;
    if (!staged) {
        if (b < nb) sort_list(c, st[b], st[b + 1]);
        return;
    }
    const int32_t m = r1 - r0;
    for (int32_t i = (int32_t)threadIdx.x; i < m; i += kSortBins) s_ref[i] = c[r0 + i];
    __syncthreads();
    if (b < nb) {
        const int32_t s0 = st[b] - r0, s1 = st[b + 1] - r0;
        for (int32_t i = s0 + 1; i < s1; ++i) {
            const int32_t v = s_ref[i];
            int32_t j = i;
            for (; j > s0 && s_ref[j - 1] > v; --j) s_ref[j] = s_ref[j - 1];
            s_ref[j] = v;
        }
    }
    __syncthreads();
    for (int32_t i = (int32_t)threadIdx.x; i < m; i += kSortBins) c[r0 + i] = s_ref[i];
}

// ------------------------------------------------------------------ host orchestration

void grid_free(nif_grid* g) {
    void* ps[] = {g->poses, g->verts, g->bin_start, g->bin_cells, g->list, g->counts, g->scratch, g->order_pre, g->scan_sums};
    for (void* p : ps)
        if (p) (void)hipFree(p);
    g->poses = nullptr; g->verts = nullptr; g->bin_start = nullptr; g->bin_cells = nullptr;
    g->list = nullptr; g->counts = nullptr; g->scratch = nullptr; g->order_pre = nullptr; g->scan_sums = nullptr;
}

// scratch layout: bbox [6 P] | totals [P] | overflow [1] | n_occ [1]
static int32_t* sc_bbox(nif_grid* g) { return g->scratch; }
static int32_t* sc_totals(nif_grid* g) { return g->scratch + 6 * g->n_poses; }
static int32_t* sc_overflow(nif_grid* g) { return g->scratch + 7 * g->n_poses; }
static int32_t* sc_nocc(nif_grid* g) { return g->scratch + 7 * g->n_poses + 1; }

static int scan_chunks(int64_t max_bins) { return (int)((max_bins + kScanChunk - 1) / kScanChunk); }

// Vertices, boxes, bin sizes, counts, scan and per-pose offsets; fills the reference lists
// when `fill`.  Device work only: no allocation, no synchronisation.
static int grid_rebin(nif_grid* g, bool fill, hipStream_t st) {
    const int P = g->n_poses, N = g->N;
    const int64_t nv = (int64_t)(N + 1) * (N + 1) * (N + 1);
    const int32_t n_occ = (int32_t)g->n_occupied;
    hipLaunchKernelGGL(k_vertices, dim3((unsigned)((nv + 255) / 256), P), dim3(256), 0, st, g->poses, N, g->verts);
    hipLaunchKernelGGL(k_bbox_init, dim3((6 * P + 255) / 256), dim3(256), 0, st, sc_bbox(g), P);
    if (n_occ > 0) {
        unsigned nblk = (unsigned)std::min<int64_t>((n_occ + 255) / 256, kBoxBlocks);
        hipLaunchKernelGGL(k_pose_bbox, dim3(nblk, P), dim3(256), 0, st, g->poses, g->verts, N, g->list, n_occ, sc_bbox(g));
    }
    hipLaunchKernelGGL(k_pose_bins, dim3((P + 63) / 64), dim3(64), 0, st, g->poses, P, sc_bbox(g), n_occ);
    hipLaunchKernelGGL(k_fill_i32, dim3(1024), dim3(256), 0, st, g->counts, g->bin_total, 0);
    const unsigned occ_blk = (unsigned)std::max<int64_t>(1, (n_occ + 255) / 256);
    if (n_occ > 0)
        hipLaunchKernelGGL(k_bin_count, dim3(occ_blk, P), dim3(256), 0, st, g->poses, g->verts, N, g->list, n_occ, g->counts);
    const int chunks = scan_chunks(g->max_bins);
    hipLaunchKernelGGL(k_chunk_sums, dim3(chunks, P), dim3(256), 0, st, g->poses, g->counts, g->scan_sums, chunks);
    hipLaunchKernelGGL(k_scan, dim3(chunks, P), dim3(256), 0, st, g->poses, g->counts, g->scan_sums, chunks, g->bin_start,
                       sc_totals(g));
    hipLaunchKernelGGL(k_ref_offsets, dim3(1), dim3(64), 0, st, g->poses, P, sc_totals(g), fill ? g->ref_capacity : (int64_t)0,
                       sc_overflow(g));
    if (fill && n_occ > 0) {
        hipLaunchKernelGGL(k_bin_fill, dim3(occ_blk, P), dim3(256), 0, st, g->poses, g->verts, N, g->list, n_occ,
                           g->bin_start, g->counts, g->bin_cells);
        hipLaunchKernelGGL(k_bin_sort, dim3((unsigned)((g->max_bins + kSortBins - 1) / kSortBins), P), dim3(kSortBins), 0, st, g->poses,
                           g->bin_start, g->bin_cells);
    }
    return check_hip(hipGetLastError(), "grid rebin launch");
}

static void set_pose_params(std::vector<PoseDev>& P, const nif_pose* poses) {
    for (size_t p = 0; p < P.size(); ++p) {
        P[p].kind = poses[p].kind;
        P[p].s = poses[p].strength;
        pose_constants(P[p].kind, P[p].s, &P[p].k0, &P[p].k1, &P[p].k2);
    }
}

int grid_build(nif_grid* g, const uint8_t* occ, int32_t N, const nif_pose* poses, int32_t n_poses,
               int32_t bins_per_axis, hipStream_t st) {
    g->N = N;
    g->n_poses = n_poses;
    const int64_t nv = (int64_t)(N + 1) * (N + 1) * (N + 1);
    const int64_t ncell = (int64_t)N * N * N;
    const int nbin_axis = bins_per_axis > 0 ? bins_per_axis : (N / 2 > 0 ? N / 2 : 1);
    std::vector<PoseDev> P(n_poses);
    for (int p = 0; p < n_poses; ++p) {
        memset(&P[p], 0, sizeof(PoseDev));
        P[p].vert_off = nv * p;
        P[p].nb[0] = P[p].nb[1] = P[p].nb[2] = 1;
    }
    set_pose_params(P, poses);
    int rc;
#define NIF_TRY(expr, what)                                      \
    do {                                                         \
        if ((rc = check_hip((expr), what)) != NIF_OK) return rc; \
    } while (0)
    NIF_TRY(hipMalloc(&g->poses, sizeof(PoseDev) * n_poses), "hipMalloc poses");
    NIF_TRY(hipMalloc(&g->verts, sizeof(float4) * nv * n_poses), "hipMalloc vertices");
    NIF_TRY(hipMalloc(&g->scratch, sizeof(int32_t) * (7 * n_poses + 8)), "hipMalloc grid scratch");
    NIF_TRY(hipMalloc(&g->order_pre, sizeof(int64_t) * 8 * (n_poses + 1)), "hipMalloc dealing table");
    NIF_TRY(hipMalloc(&g->list, sizeof(int32_t) * (ncell + 1)), "hipMalloc occupied list");
    // occupied voxels, compacted once
    NIF_TRY(hipMemsetAsync(sc_nocc(g), 0, sizeof(int32_t), st), "memset");
    hipLaunchKernelGGL(k_compact, dim3((unsigned)((ncell + 255) / 256)), dim3(256), 0, st, occ, ncell, g->list, sc_nocc(g));
    NIF_TRY(hipGetLastError(), "k_compact");
    int32_t n_occ = 0;
    NIF_TRY(hipMemcpyAsync(&n_occ, sc_nocc(g), sizeof(int32_t), hipMemcpyDeviceToHost, st), "read count");
    NIF_TRY(hipStreamSynchronize(st), "sync");
    g->n_occupied = n_occ;
    // the first poses' bounding boxes fix the bins per axis (by aspect ratio)
    NIF_TRY(hipMemcpyAsync(g->poses, P.data(), sizeof(PoseDev) * n_poses, hipMemcpyHostToDevice, st), "copy poses");
    hipLaunchKernelGGL(k_vertices, dim3((unsigned)((nv + 255) / 256), n_poses), dim3(256), 0, st, g->poses, N, g->verts);
    hipLaunchKernelGGL(k_bbox_init, dim3((6 * n_poses + 255) / 256), dim3(256), 0, st, sc_bbox(g), n_poses);
    if (n_occ > 0) {
        unsigned nblk = (unsigned)std::min<int64_t>((n_occ + 255) / 256, kBoxBlocks);
        hipLaunchKernelGGL(k_pose_bbox, dim3(nblk, n_poses), dim3(256), 0, st, g->poses, g->verts, N, g->list, n_occ, sc_bbox(g));
    }
    NIF_TRY(hipGetLastError(), "bbox");
    std::vector<int32_t> bb(6 * n_poses);
    NIF_TRY(hipMemcpyAsync(bb.data(), sc_bbox(g), sizeof(int32_t) * 6 * n_poses, hipMemcpyDeviceToHost, st), "read bbox");
    NIF_TRY(hipStreamSynchronize(st), "sync");
    int64_t bin_total = 0, max_bins = 1;
    for (int p = 0; p < n_poses; ++p) {
        float e[3], ext = 0.f;
        for (int c = 0; c < 3; ++c) {
            e[c] = n_occ == 0 ? 1.f : ord2f_host(bb[6 * p + 3 + c]) - ord2f_host(bb[6 * p + c]);
            ext = std::max(ext, e[c]);
        }
        for (int c = 0; c < 3; ++c) P[p].nb[c] = std::max(1, std::min((int)std::ceil(nbin_axis * e[c] / ext - 1e-3f), 4096));
        P[p].bin_off = bin_total;
        const int64_t nb = (int64_t)P[p].nb[0] * P[p].nb[1] * P[p].nb[2];
        bin_total += nb + 1;
        max_bins = std::max(max_bins, nb);
    }
    g->bin_total = bin_total;
    g->max_bins = max_bins;
    NIF_TRY(hipMalloc(&g->bin_start, sizeof(int32_t) * bin_total), "hipMalloc bin_start");
    NIF_TRY(hipMalloc(&g->counts, sizeof(int32_t) * bin_total), "hipMalloc bin counts");
    NIF_TRY(hipMalloc(&g->scan_sums, sizeof(int32_t) * (size_t)scan_chunks(max_bins) * n_poses), "hipMalloc scan sums");
    NIF_TRY(hipMemcpyAsync(g->poses, P.data(), sizeof(PoseDev) * n_poses, hipMemcpyHostToDevice, st), "copy poses");
    // count pass, then size the reference lists with headroom for later re-poses
    g->ref_capacity = 0;
    if ((rc = grid_rebin(g, false, st))) return rc;
    std::vector<int32_t> tot(n_poses);
    NIF_TRY(hipMemcpyAsync(tot.data(), sc_totals(g), sizeof(int32_t) * n_poses, hipMemcpyDeviceToHost, st), "read totals");
    NIF_TRY(hipStreamSynchronize(st), "sync");
    int64_t refs = 0;
    for (int p = 0; p < n_poses; ++p) refs += tot[p];
    g->ref_capacity = refs + refs / 2 + 4096;
    NIF_TRY(hipMalloc(&g->bin_cells, sizeof(int32_t) * g->ref_capacity), "hipMalloc bin_cells");
    if ((rc = grid_rebin(g, true, st))) return rc;
    NIF_TRY(hipStreamSynchronize(st), "sync");
    g->poses_host = P;
    g->refs_per_pose.assign(tot.begin(), tot.end());
#undef NIF_TRY
    return NIF_OK;
}

int grid_update(nif_grid* g, const nif_pose* poses, hipStream_t st) {
    set_pose_params(g->poses_host, poses);
    // kind, strength and constants change; boxes, bin sizes and offsets are recomputed on the device
    int rc = check_hip(hipMemcpyAsync(g->poses, g->poses_host.data(), sizeof(PoseDev) * g->n_poses,
                                      hipMemcpyHostToDevice, st), "copy poses");
    if (rc) return rc;
    return grid_rebin(g, true, st);
}

int grid_bounds(const nif_grid* g, int pose, float* lo, float* hi) {
    PoseDev pd;
    int rc = check_hip(hipMemcpy(&pd, g->poses + pose, sizeof(PoseDev), hipMemcpyDeviceToHost), "read pose");
    if (rc) return rc;
    for (int a = 0; a < 3; ++a) {
        lo[a] = pd.empty ? 0.f : pd.lo[a];
        hi[a] = pd.empty ? 0.f : pd.lo[a] + pd.bs[a] * (float)pd.nb[a];
    }
    return NIF_OK;
}

int grid_overflow(nif_grid* g, hipStream_t st, int32_t* overflow) {
    int rc = check_hip(hipMemcpyAsync(overflow, sc_overflow(g), sizeof(int32_t), hipMemcpyDeviceToHost, st), "read overflow");
    if (rc) return rc;
    return check_hip(hipStreamSynchronize(st), "sync");
}

}  // namespace nif
