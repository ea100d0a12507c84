// Query-side host code and the kernels beside the fused query (nif_query.hpp): segment tracing and
// the voxel proxy.
#include "nif_query.hpp"

namespace nif {

__global__ void k_reset(int64_t* counters, int n) {
    if (threadIdx.x < n) counters[threadIdx.x] = 0;
}

// Per-pose timing slots of the stats buffer: [4] start (min over waves), [5, 5+P) completion
// time of each pose, [5+P, 5+2P) rays finished per pose.
__global__ void k_reset_pose_times(int64_t* stats, int n_poses) {
    for (int i = threadIdx.x; i < 1 + 2 * n_poses; i += blockDim.x) stats[4 + i] = i == 0 ? INT64_MAX : 0;
}

// ------------------------------------------------------------------ segments of every ray

// SUB lanes a ray: the time of a launch is that of the longest rays' chains of bins and voxel tests
// (2^17 random rays through 8 poses of the 128^3 blob scene: 5.3 ms with one lane, 1.66 with four,
// 1.60 with eight, 1.78 with sixteen; 3,000 rays: 0.52, 0.38 and 0.27 with four, eight, sixteen; with
// the walk's state in registers, as it is now, 1.33 with eight).
// Four waves per SIMD: the form of 16 lanes takes 129 registers by itself, one above that line (16,300
// rays 433 us, 395 with 128 registers and 12 bytes of scratch).
// points: the rest-space end points are written here; else k_trace_points forms them from t_in, t_out.
template <int SUB>
__global__ void __launch_bounds__(64, 4) k_trace(GridArgs G, RayArgs R, int64_t r0, int32_t max_seg, nif_segments out,
                                               int points) {
    const int64_t r = r0 + (int64_t)blockIdx.x * (64 / SUB) + threadIdx.x / SUB;
    if (r >= R.n) return;
    const bool lead = threadIdx.x % SUB == 0;
    const Ray ray = load_ray(R, r);
    const PoseDev P = G.poses[find_pose(R.off, R.n_poses, r)];
    Trav tv;
    trav_init(P, ray, tv);
    int n = 0;
    const int64_t total = R.n * (int64_t)max_seg;
    all_segments<SUB>(P, G.V, G.bin_start, G.bin_cells, G.N, ray, tv, [&](int32_t cell, float a, float b) {
        if (lead && n < max_seg) {
            const int64_t k = r * max_seg + n;
            if (out.cell) out.cell[k] = cell;
            if (out.t_in) out.t_in[k] = a;
            if (out.t_out) out.t_out[k] = b;
            if (points) {
                const float3 x0 = deform_inv(P, ray_at(ray, a));
                const float3 x1 = deform_inv(P, ray_at(ray, b));
                if (out.x0) { out.x0[k] = x0.x; out.x0[total + k] = x0.y; out.x0[2 * total + k] = x0.z; }
                if (out.x1) { out.x1[k] = x1.x; out.x1[total + k] = x1.y; out.x1[2 * total + k] = x1.z; }
            }
        }
        ++n;
    });
    if (lead && out.count) out.count[r] = n;
}

// Rest-space end points of the stored segments, one lane each: in the walk they would be formed by
// the few lanes that emit at the same time.
__global__ void __launch_bounds__(256) k_trace_points(GridArgs G, RayArgs R, int32_t max_seg, nif_segments out) {
    const int64_t total = R.n * (int64_t)max_seg;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = k / max_seg;
        if (k - r * max_seg >= out.count[r]) continue;
        const Ray ray = load_ray(R, r);
        const PoseDev P = G.poses[find_pose(R.off, R.n_poses, r)];
        if (out.x0) {
            const float3 x = deform_inv(P, ray_at(ray, out.t_in[k]));
            out.x0[k] = x.x; out.x0[total + k] = x.y; out.x0[2 * total + k] = x.z;
        }
        if (out.x1) {
            const float3 x = deform_inv(P, ray_at(ray, out.t_out[k]));
            out.x1[k] = x.x; out.x1[total + k] = x.y; out.x1[2 * total + k] = x.z;
        }
    }
}

// ------------------------------------------------------------------ voxel proxy (no network)
// The first occupied voxel is the hit: D = t_in, rest point D^-1(entry), normal = outward
// rest-space normal of the entered face.

__global__ void __launch_bounds__(256) k_proxy(GridArgs G, RayArgs R, nif_hits out, int64_t* __restrict__ stats) {
    int64_t n_done = 0;
    int bad = 0;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R.n; r += (int64_t)gridDim.x * blockDim.x) {
        const Ray ray = load_ray(R, r);
        const PoseDev P = G.poses[find_pose(R.off, R.n_poses, r)];
        Trav tv;
        trav_init(P, ray, tv);
        Segment sg;
        const float tmax = R.tmax ? R.tmax[r] : INFINITY;
        if (next_segment<1>(P, G.V, G.bin_start, G.bin_cells, G.N, ray, tv, sg, &bad) && sg.a < tmax) {
            const float3 x0 = deform_inv(P, ray_at(ray, sg.a));
            float z[16];
            for (int i = 0; i < 16; ++i) z[i] = 0.f;
            z[0] = 1.f;
            // the face normal enters the outputs as z_n; the distance head is 0 so D = t_in
            if (sg.face >= 0) z[2 + (sg.face >> 1)] = (sg.face & 1) ? 1.f : -1.f;
            write_hit(out, r, sg, x0, x0, z, 1, 1, NIF_DIST_LOG_RELU, tmax, P);
            if (out.ar) out.ar[r] = 0.f;
            if (out.ag) out.ag[r] = 0.f;
            if (out.ab) out.ab[r] = 0.f;
            if (out.material) out.material[r] = 0;
        } else {
            write_miss(out, r, 0, -INFINITY);
        }
        ++n_done;
    }
    if (stats) {
        int64_t a = n_done, c = bad;
        for (int off = 32; off > 0; off >>= 1) { a += __shfl_xor(a, off); c += __shfl_xor(c, off); }
        if (lane_id() == 0) {
            atomicAdd((unsigned long long*)&stats[0], (unsigned long long)a);
            atomicAdd((unsigned long long*)&stats[2], (unsigned long long)c);
        }
    }
}

// ------------------------------------------------------------------ staged query
//
// Launches of many rays evaluate the rays' first segments in stages, each a kernel over all of them:
// search, encoding level by level, MLP, results.  Table lookups then run at the rate of one level's
// table in L2 (nif_panels.hpp) and the matrix cores on full tiles, and the search on all lanes.  The fused kernel takes the rays whose first segment is no hit, from there on,
// and those beyond the list's room (a quarter of the rays; it would otherwise be mostly empty
// launches).  A ray's result depends on neither.

// First segment of every ray, SUB lanes each: rays without one are misses, the others go
// to the list, in order of the blocks.
template <int SUB>
__global__ void __launch_bounds__(256) k_first(GridArgs G, RayArgs R, nif_hits out, int32_t cap, int32_t* __restrict__ list,
                                               int64_t ld, float* __restrict__ x, int32_t* __restrict__ n_list,
                                               int32_t* __restrict__ rest, int32_t* __restrict__ n_rest, int64_t* __restrict__ stats) {
    __shared__ int32_t s_n[4], s_base;
    const int64_t r = (int64_t)blockIdx.x * (256 / SUB) + threadIdx.x / SUB;
    const bool lead = threadIdx.x % SUB == 0;
    const int w = threadIdx.x >> 6, lane = lane_id();
    bool has = false;
    int bad = 0;
    Segment sg;
    float3 x0, x1;
    if (r < R.n) {
        const Ray ray = load_ray(R, r);
        const PoseDev P = G.poses[find_pose(R.off, R.n_poses, r)];
        Trav tv;
        trav_init(P, ray, tv);
        has = next_segment<SUB>(P, G.V, G.bin_start, G.bin_cells, G.N, ray, tv, sg, &bad);
        if (has && R.tmax && sg.a >= R.tmax[r]) has = false;         // occlusion bound reached
        if (has) {
            x0 = deform_inv(P, ray_at(ray, sg.a));
            x1 = deform_inv(P, ray_at(ray, sg.b));
        } else if (lead) {
            write_miss(out, r, 0, -INFINITY);
        }
    }
    has = has && lead;
    const uint64_t mask = ballot(has), below = (1ull << lane) - 1ull;
    if (lane == 0) s_n[w] = popc64(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        const int32_t c = s_n[0] + s_n[1] + s_n[2] + s_n[3];
        s_base = c ? atomicAdd(n_list, c) : 0;
    }
    __syncthreads();
    int32_t k = s_base + popc64(mask & below);
    for (int v = 0; v < w; ++v) k += s_n[v];
    const bool over = has && k >= cap;
    if (has && !over) {
        list[k] = (int32_t)r;
        list[ld + k] = sg.cell;
        list[2 * ld + k] = __float_as_int(sg.a);
        list[3 * ld + k] = __float_as_int(sg.b);
        x[k] = x0.x; x[ld + k] = x0.y; x[2 * ld + k] = x0.z;
        x[3 * ld + k] = x1.x; x[4 * ld + k] = x1.y; x[5 * ld + k] = x1.z;
    }
    const uint64_t om = ballot(over);
    if (om) {
        int32_t base = 0;
        if (lane == 0) base = atomicAdd(n_rest, popc64(om));
        base = __shfl(base, 0);
        if (over) {
            const int32_t at = base + popc64(om & below);
            rest[at] = (int32_t)r;
            rest[kStageRays + at] = -1;
        }
    }
    // every lane counts its own tests; those of a ray beyond the list are counted when it is searched again
    const uint64_t ray_lanes = SUB == 64 ? ~0ull : ((1ull << SUB) - 1ull) << (lane / SUB * SUB);
    if (om & ray_lanes) bad = 0;
    if (stats) wave_add_stat(&stats[2], bad);                        // the misses are counted by k_first_hits
}

// Results of the staged segments: hits are written, the other rays are left for the fused kernel.
// Statistics: one set of atomics per block, and the rays without a segment in one sum (one atomic per
// wave of k_first cost a frame of 2^20 rays 1.6 ms).
__global__ void __launch_bounds__(256) k_first_hits(GridArgs G, RayArgs R, nif_hits out, int H, int dist_head, int32_t cap,
                                                    const int32_t* __restrict__ list, int64_t ld, const float* __restrict__ x,
                                                    const float* __restrict__ heads, const int32_t* __restrict__ n_list,
                                                    int32_t* __restrict__ rest, int32_t* __restrict__ n_rest,
                                                    int64_t* __restrict__ stats) {
    const int32_t n = min(*n_list, cap);
    int64_t n_done = 0, n_eval = 0;
    for (int32_t k0 = (int32_t)blockIdx.x * 256; k0 < n; k0 += (int32_t)gridDim.x * 256) {
        const int32_t k = k0 + (int32_t)threadIdx.x;
        bool left = false;
        if (k < n) {
            const float* z = heads + (int64_t)k * H;
            const int64_t r = list[k];
            ++n_eval;
            if (z[0] > 0.f) {
                Segment sg;
                sg.cell = list[ld + k]; sg.a = __int_as_float(list[2 * ld + k]); sg.b = __int_as_float(list[3 * ld + k]); sg.face = -1;
                write_hit(out, r, sg, make_float3(x[k], x[ld + k], x[2 * ld + k]),
                          make_float3(x[3 * ld + k], x[4 * ld + k], x[5 * ld + k]), z, 1, H - 8, dist_head,
                          R.tmax ? R.tmax[r] : INFINITY, G.poses[find_pose(R.off, R.n_poses, r)]);
                ++n_done;
            } else {
                left = true;
            }
        }
        const uint64_t m = ballot(left);
        if (m) {
            int32_t base = 0;
            if (lane_id() == 0) base = atomicAdd(n_rest, popc64(m));
            base = __shfl(base, 0);
            if (left) {
                const int32_t at = base + popc64(m & ((1ull << lane_id()) - 1ull));
                rest[at] = list[k];
                rest[kStageRays + at] = pack_cell(list[ld + k], G.N);
                rest[2 * kStageRays + at] = list[2 * ld + k];
                rest[3 * kStageRays + at] = __float_as_int(heads[(int64_t)k * H]);
            }
        }
    }
    if (!stats) return;
    __shared__ int64_t s_sum[2];
    if (threadIdx.x < 2) s_sum[threadIdx.x] = 0;
    __syncthreads();
    wave_add_stat(&s_sum[0], n_done);
    wave_add_stat(&s_sum[1], n_eval);
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t done = s_sum[0] + (blockIdx.x == 0 ? R.n - *n_list : 0);
        if (done) atomicAdd((unsigned long long*)&stats[0], (unsigned long long)done);
        if (s_sum[1]) atomicAdd((unsigned long long*)&stats[1], (unsigned long long)s_sum[1]);
    }
}

// ------------------------------------------------------------------ host launchers

int device_cus() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}

static GridArgs grid_args(const nif_grid* g) {
    GridArgs G;
    G.poses = g->poses; G.V = g->verts; G.bin_start = g->bin_start; G.bin_cells = g->bin_cells; G.N = g->N;
    return G;
}

// Pose-ordered dealing: pre[k][p] = rays of poses 0 .. p-1 in range k, whose share of pose q
// is [off[q] + c_q k / 8, off[q] + c_q (k + 1) / 8), c_q the pose's ray count.
__global__ void k_order_prefix(const int64_t* __restrict__ off, int n_poses, int64_t* __restrict__ pre) {
    const int k = threadIdx.x;
    if (k >= 8) return;
    int64_t acc = 0;
    for (int p = 0; p < n_poses; ++p) {
        pre[(int64_t)k * (n_poses + 1) + p] = acc;
        const int64_t c = off[p + 1] - off[p];
        acc += c * (k + 1) / 8 - c * k / 8;
    }
    pre[(int64_t)k * (n_poses + 1) + n_poses] = acc;
}

static RayArgs ray_args(const nif_grid* g, const nif_rays* r, int64_t n) {
    RayArgs R;
    R.ox = r->ox; R.oy = r->oy; R.oz = r->oz; R.dx = r->dx; R.dy = r->dy; R.dz = r->dz;
    R.off = r->pose_offsets; R.tmax = r->tmax; R.n_poses = g->n_poses; R.n = n;
    R.order_pre = nullptr;
    R.rest_n = nullptr;
    R.rest = nullptr;
    R.least = 0;
    R.most = INT64_MAX;
    return R;
}

int trace_launch(const nif_grid* g, const nif_rays* r, int64_t n, int32_t max_seg, const nif_segments* out,
                 hipStream_t st) {
    if (n == 0) return NIF_OK;
    const bool apart = out->t_in && out->t_out && out->t_in != out->t_out && (out->x0 || out->x1);
    const GridArgs G = grid_args(g);
    const RayArgs R = ray_args(g, r, n);
    constexpr int64_t kMaxRays = 1 << 28;              // of one launch: its lanes fit 32 bits
    for (int64_t r0 = 0; r0 < n; r0 += kMaxRays) {
        const int64_t m = std::min(kMaxRays, n - r0);
        if (n < (int64_t)device_cus() * 64)
            hipLaunchKernelGGL(k_trace<16>, dim3((unsigned)((m + 3) / 4)), dim3(64), 0, st, G, R, r0, max_seg, *out, !apart);
        else
            hipLaunchKernelGGL(k_trace<8>, dim3((unsigned)((m + 7) / 8)), dim3(64), 0, st, G, R, r0, max_seg, *out, !apart);
    }
    if (apart && max_seg > 0) {
        const int64_t blocks = std::min<int64_t>((n * (int64_t)max_seg + 255) / 256, (int64_t)device_cus() * 32);
        hipLaunchKernelGGL(k_trace_points, dim3((unsigned)blocks), dim3(256), 0, st, G, R, max_seg, *out);
    }
    return check_hip(hipGetLastError(), "k_trace launch");
}

// Persistent grid size of the fused query: one-wave workgroups per compute unit (tunable).
static int g_query_blocks_per_cu = 12;
// Rays per wave: 0 = by launch size, else 16 or 64.
static int g_query_rays_per_wave = 0;

static int launch_fused(const nif_model* m, const GridArgs& G, const RayArgs& R, const nif_hits* out, int32_t precision,
                        int64_t* stats, int pt, hipStream_t st) {
    const NetParams np = make_net_params(m, precision);
    const int hw = m->desc.hidden_width;
    const QueryShape sh{device_cus(), g_query_blocks_per_cu, g_query_rays_per_wave};
    int rc;
    if (precision == NIF_PREC_FP32) rc = query_fp32(sh, hw, np, G, R, *out, m->counters, stats, pt, st);
    else if (precision == NIF_PREC_BF16) rc = query_bf16(sh, hw, np, G, R, *out, m->counters, stats, pt, st);
    else rc = query_fp16(sh, hw, np, G, R, *out, m->counters, stats, pt, st);
    if (rc) return rc;
    return check_hip(hipGetLastError(), "k_query launch");
}

int64_t stage_cap(const nif_model* m) {
    const int64_t c = stage_chunk(m);
    return (kStageRays / 4 + c - 1) / c * c;
}

static int query_staged(const nif_model* m, const GridArgs& G, RayArgs R, int64_t n, const nif_hits* out, int32_t precision,
                        int64_t* stats, hipStream_t st) {
    int32_t* n_list = reinterpret_cast<int32_t*>(m->counters + 8);
    int32_t* n_rest = reinterpret_cast<int32_t*>(m->counters + 9);
    const int64_t ld = stage_cap(m), chunk = stage_chunk(m);
    const int32_t cap = (int32_t)std::min(std::max<int64_t>(1, (n / 4 + chunk - 1) / chunk) * chunk, n);
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, st, m->counters, 16);
    // with 1, 2, 4, 8 lanes a ray a batch of 1.5 M mixed rays took 4.75, 4.36, 4.79, 5.46 ms (4.11 with two
    // since the walk's state is in registers)
    constexpr int SUB = 2;
    hipLaunchKernelGGL(k_first<SUB>, dim3((unsigned)((n * SUB + 255) / 256)), dim3(256), 0, st, G, R, *out, cap, m->q_list, ld, m->q_x,
                       n_list, m->q_rest, n_rest, stats);
    int rc;
    if ((rc = forward_live_launch(m, m->q_x, ld, n_list, cap, m->q_heads, precision, st))) return rc;
    const unsigned blocks = (unsigned)std::min<int64_t>((cap + 255) / 256, (int64_t)device_cus() * 8);
    hipLaunchKernelGGL(k_first_hits, dim3(blocks), dim3(256), 0, st, G, R, *out, m->H, m->desc.dist_head, cap, m->q_list, ld, m->q_x,
                       m->q_heads, n_list, m->q_rest, n_rest, stats);
    R.rest_n = n_rest;
    R.rest = m->q_rest;
    return launch_fused(m, G, R, out, precision, stats, 0, st);
}

// Launches of so many rays are staged, up to kStageRays.  16,001 rays: 262 us staged, 313 in blocks
// (64^3 spheres), 566 and 627 (128^3 blobs, BF16); 8,001: 529 and 367.  The upper line is the room of
// the model's lists, not where staging stops to pay: at 2^21 rays the staged form is ahead for every
// kind of rays (128^3 blobs, BF16, staged against 64 rays more fused: camera 3.39 and 5.23 ms, half
// secondary 5.63 and 10.06, random 15.3 and 22.2).  Sweeps in stages of 2^21 were measured for coherent
// rays only, and lose there: 25 M camera rays 27.0 ms, 26.2 fused.
constexpr int64_t kStageLeastRays = 1 << 14;

static bool staged(const nif_model* m, int64_t n, uint32_t flags) {
    return uses_panels(m) && n >= kStageLeastRays && n <= kStageRays && !(flags & (NIF_Q_POSE_ORDER | NIF_Q_POSE_TIMES));
}

int query_launch(const nif_model* m, const nif_grid* g, const nif_rays* r, int64_t n, const nif_hits* out,
                 uint32_t flags, int32_t precision, int64_t* stats, hipStream_t st) {
    if (n == 0) return NIF_OK;
    const GridArgs G = grid_args(g);
    RayArgs R = ray_args(g, r, n);
    if (flags & NIF_Q_NO_NETWORK) {
        const int64_t blocks = std::min<int64_t>((n + 255) / 256, (int64_t)device_cus() * 16);
        hipLaunchKernelGGL(k_proxy, dim3((unsigned)blocks), dim3(256), 0, st, G, R, *out, stats);
        return check_hip(hipGetLastError(), "k_proxy launch");
    }
    if (staged(m, n, flags)) return query_staged(m, G, R, n, out, precision, stats, st);
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, st, m->counters, 8);
    if (flags & NIF_Q_POSE_ORDER) {
        hipLaunchKernelGGL(k_order_prefix, dim3(1), dim3(64), 0, st, R.off, R.n_poses, g->order_pre);
        R.order_pre = g->order_pre;
    }
    const int pt = (flags & NIF_Q_POSE_TIMES) && stats ? 1 : 0;
    if (pt) hipLaunchKernelGGL(k_reset_pose_times, dim3(1), dim3(256), 0, st, stats, g->n_poses);
    return launch_fused(m, G, R, out, precision, stats, pt, st);
}

int set_query_blocks_per_cu(int v) {
    g_query_blocks_per_cu = v;
    return NIF_OK;
}

int set_query_rays_per_wave(int v) {
    g_query_rays_per_wave = v;
    return NIF_OK;
}

// Times the fused query on the caller's rays for every launch shape of the search space
// (workgroups per CU x rays per wave), keeps the fastest process-wide and reports it.  The fused kernel
// itself, also where nif_query is staged: there it takes only the rays left over, in 16-ray waves whatever
// the setting, and 16 and 64 would differ by noise alone.  For the same reason a number of workgroups
// that makes the launch of the present one is passed over.
int autotune_query(const nif_model* m, const nif_grid* g, const nif_rays* r, int64_t n, const nif_hits* out,
                   int32_t precision, int32_t reps, int32_t* best, float* best_ms, hipStream_t st) {
    static const int kBpc[] = {4, 6, 8, 10, 12, 14, 16, 20, 24};
    static const int kRpw[] = {16, 64};
    const int save_bpc = g_query_blocks_per_cu, save_rpw = g_query_rays_per_wave;
    const bool listed = std::find(std::begin(kBpc), std::end(kBpc), save_bpc) != std::end(kBpc);
    const GridArgs G = grid_args(g);
    const RayArgs R = ray_args(g, r, n);
    hipEvent_t e0, e1;
    int rc = check_hip(hipEventCreate(&e0), "event");
    if (rc) return rc;
    if ((rc = check_hip(hipEventCreate(&e1), "event"))) { (void)hipEventDestroy(e0); return rc; }
    auto fused = [&]() {
        hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, st, m->counters, 8);
        return launch_fused(m, G, R, out, precision, nullptr, 0, st);
    };
    auto query = [&]() { return query_launch(m, g, r, n, out, 0, precision, nullptr, st); };
    auto timed = [&](auto launch, float* ms) {
        int e = launch();                                              // warm-up
        if (!e) e = check_hip(hipEventRecord(e0, st), "event record");
        for (int i = 0; i < reps && !e; ++i) e = launch();
        if (!e) e = check_hip(hipEventRecord(e1, st), "event record");
        if (!e) e = check_hip(hipEventSynchronize(e1), "event sync");
        if (!e) e = check_hip(hipEventElapsedTime(ms, e0, e1), "elapsed");
        *ms /= (float)reps;
        return e;
    };
    auto workgroups = [&](int bpc, int rpw) { return std::min<int64_t>((n + rpw - 1) / rpw, (int64_t)device_cus() * bpc); };
    float best_t = INFINITY;
    int bb = save_bpc, br = save_rpw;
    for (int rpw : kRpw) {
        for (int bpc : kBpc) {
            if (listed && bpc != save_bpc && workgroups(bpc, rpw) == workgroups(save_bpc, rpw)) continue;
            g_query_blocks_per_cu = bpc;
            g_query_rays_per_wave = rpw;
            float ms = 0.f;
            if ((rc = timed(fused, &ms))) break;
            if (ms < best_t) { best_t = ms; bb = bpc; br = rpw; }
        }
        if (rc) break;
    }
    if (!rc) {
        g_query_blocks_per_cu = bb;
        g_query_rays_per_wave = br;
        if (staged(m, n, 0)) rc = timed(query, &best_t);               // what the caller's launches take
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) {
        g_query_blocks_per_cu = save_bpc;
        g_query_rays_per_wave = save_rpw;
        return rc;
    }
    best[0] = bb;
    best[1] = br;
    if (best_ms) *best_ms = best_t;
    return NIF_OK;
}

}  // namespace nif
