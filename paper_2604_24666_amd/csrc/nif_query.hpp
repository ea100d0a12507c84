// The fused first-hit query kernel and its launch, compiled once per MLP precision
// (nif_query_fp32.hip, nif_query_bf16.hip, nif_query_fp16.hip).
//
// The fused query (Methodology; "Segmented Ray Distance Accumulation") is one persistent
// kernel.  Every lane owns a ray; a wave takes rays from a global counter (one atomic per
// wave, rays of all poses in one index space).  Each round, every lane finds its ray's next
// occupied deformed voxel, maps the voxel's entry/exit points to rest space, and the wave
// evaluates encoding + MLP for all 64 segments together on MFMA.  A lane whose hit logit is
// positive writes the ray's result and takes a new ray; the others continue front to back.
// Lanes whose rays miss everything take new rays before the network round, so the MFMA
// tiles stay full while rays last.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstring>

#include "nif_deal.hpp"
#include "nif_internal.hpp"
#include "nif_net.hpp"
#include "nif_panels.hpp"
#include "nif_trace.hpp"

namespace nif {

struct GridArgs {
    const PoseDev* poses;
    const float4* V;
    const int32_t* bin_start;
    const int32_t* bin_cells;
    int32_t N;
};

struct RayArgs {
    const float *ox, *oy, *oz, *dx, *dy, *dz;
    const int64_t* off;
    const float* tmax;          // nullable: occlusion bound per ray
    int32_t n_poses;
    int64_t n;
    const int64_t* order_pre;   // nullable: pose-ordered dealing, [8][n_poses + 1] (k_order_prefix)
    // nullable: the rays are rest_n[0] entries of a staged query's list [4][kStageRays] instead: ray,
    // packed voxel and entry t of its last segment (-1: none yet), its hit logit
    const int32_t *rest_n, *rest;
    int64_t least, most;        // of a list: the launch does nothing if it is shorter or longer
};

__device__ __forceinline__ Ray load_ray(const RayArgs& R, int64_t r) {
    Ray ray;
    ray.o = make_float3(R.ox[r], R.oy[r], R.oz[r]);
    ray.d = make_float3(R.dx[r], R.dy[r], R.dz[r]);
    return ray;
}

__device__ __forceinline__ float3 ray_at(const Ray& R, float t) {
    return make_float3(fmaf(t, R.d.x, R.o.x), fmaf(t, R.d.y, R.o.y), fmaf(t, R.d.z, R.o.z));
}

// Counts finished rays per pose (one atomic per wave when the finishing lanes share a pose)
// and stamps a pose's completion time when its last ray is done.  Called by the whole wave.
__device__ __forceinline__ void note_finished(int64_t* stats, const int64_t* off, int n_poses, bool fin, int pose) {
    const uint64_t m = ballot(fin);
    if (!m) return;
    const int leader = __ffsll((unsigned long long)m) - 1;
    const int p0 = __shfl(pose, leader);
    const bool uniform = ballot(fin && pose != p0) == 0;
    int64_t* done = stats + 5 + n_poses;
    if (uniform) {
        if (lane_id() == leader) {
            const int64_t total = off[p0 + 1] - off[p0];
            const int64_t c = (int64_t)popc64(m);
            const int64_t old = (int64_t)atomicAdd((unsigned long long*)&done[p0], (unsigned long long)c);
            if (old + c == total) atomicMax((unsigned long long*)&stats[5 + p0], (unsigned long long)wall_clock64());
        }
    } else if (fin) {
        const int64_t total = off[pose + 1] - off[pose];
        const int64_t old = (int64_t)atomicAdd((unsigned long long*)&done[pose], 1ull);
        if (old + 1 == total) atomicMax((unsigned long long*)&stats[5 + pose], (unsigned long long)wall_clock64());
    }
}

// ------------------------------------------------------------------ outputs of one ray

__device__ __forceinline__ void write_miss(const nif_hits& o, int64_t r, int nq, float last_z0) {
    if (o.hit) o.hit[r] = 0;
    if (o.t) o.t[r] = INFINITY;
    if (o.nx) o.nx[r] = 0.f;
    if (o.ny) o.ny[r] = 0.f;
    if (o.nz) o.nz[r] = 0.f;
    if (o.ar) o.ar[r] = 0.f;
    if (o.ag) o.ag[r] = 0.f;
    if (o.ab) o.ab[r] = 0.f;
    if (o.material) o.material[r] = -1;
    if (o.cell) o.cell[r] = -1;
    if (o.hit_logit) o.hit_logit[r] = last_z0;
    if (o.n_queried) o.n_queried[r] = nq;
    if (o.xr) o.xr[r] = 0.f;
    if (o.yr) o.yr[r] = 0.f;
    if (o.zr) o.zr[r] = 0.f;
    if (o.dnx) o.dnx[r] = 0.f;
    if (o.dny) o.dny[r] = 0.f;
    if (o.dnz) o.dnz[r] = 0.f;
}

__device__ __forceinline__ float sigmoidf_(float v) { return 1.f / (1.f + expf(-v)); }

// Writes the hit of segment sg; a hit at or beyond tmax is written as a miss instead.
__device__ __forceinline__ void write_hit(const nif_hits& o, int64_t r, const Segment& sg, float3 x0, float3 x1,
                                          const float* z, int nq, int n_mat, int dist_head, float tmax,
                                          const PoseDev& P) {
    const float ex = x1.x - x0.x, ey = x1.y - x0.y, ez = x1.z - x0.z;
    float f;
    if (dist_head == NIF_DIST_SIGMOID) {
        f = sigmoidf_(z[1]);               // the bounded head: the fraction itself
    } else {
        const float lr = sqrtf(ex * ex + ey * ey + ez * ez);
        const float dh = fmaxf(z[1], 0.f);
        f = lr > 0.f ? fminf(fmaxf(dh / lr, 0.f), 1.f) : 0.f;
    }
    const float D = fmaf(f, sg.b - sg.a, sg.a);
    if (D >= tmax) {
        write_miss(o, r, nq, z[0]);
        return;
    }
    if (o.hit) o.hit[r] = 1;
    if (o.t) o.t[r] = D;
    const float nl = fmaxf(sqrtf(z[2] * z[2] + z[3] * z[3] + z[4] * z[4]), 1e-12f);
    if (o.nx) o.nx[r] = z[2] / nl;
    if (o.ny) o.ny[r] = z[3] / nl;
    if (o.nz) o.nz[r] = z[4] / nl;
    if (o.ar) o.ar[r] = sigmoidf_(z[5]);
    if (o.ag) o.ag[r] = sigmoidf_(z[6]);
    if (o.ab) o.ab[r] = sigmoidf_(z[7]);
    if (o.material) {
        int best = 0;
        if (n_mat == 1) best = z[8] > 0.f ? 1 : 0;
        else
            for (int c = 1; c < n_mat; ++c)
                if (z[8 + c] > z[8 + best]) best = c;
        o.material[r] = best;
    }
    if (o.cell) o.cell[r] = sg.cell;
    if (o.hit_logit) o.hit_logit[r] = z[0];
    if (o.n_queried) o.n_queried[r] = nq;
    if (o.xr) o.xr[r] = fmaf(f, ex, x0.x);
    if (o.yr) o.yr[r] = fmaf(f, ey, x0.y);
    if (o.zr) o.zr[r] = fmaf(f, ez, x0.z);
    if (o.dnx || o.dny || o.dnz) {
        const float3 xh = make_float3(fmaf(f, ex, x0.x), fmaf(f, ey, x0.y), fmaf(f, ez, x0.z));
        const float3 dn = deform_normal(P, xh, make_float3(z[2] / nl, z[3] / nl, z[4] / nl));
        if (o.dnx) o.dnx[r] = dn.x;
        if (o.dny) o.dny[r] = dn.y;
        if (o.dnz) o.dnz[r] = dn.z;
    }
}

// Adds a count of the wave to the statistics, if there is one: the atomics of a launch's waves on one
// address go one after the other (about 18 ns each), so only few waves may add.
__device__ __forceinline__ void wave_add_stat(int64_t* stat, int64_t v) {
    if (!ballot(v != 0)) return;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane_id() == 0) atomicAdd((unsigned long long*)stat, (unsigned long long)v);
}

__device__ __forceinline__ void wave_add_stats(int64_t* stats, int64_t a, int64_t b, int64_t c) {
    wave_add_stat(&stats[0], a);
    wave_add_stat(&stats[1], b);
    wave_add_stat(&stats[2], c);
}

// ------------------------------------------------------------------ fused first-hit query
//
// Register budget.  The traversal state of a lane (ray index, pose, DDA state, current
// segment) is parked in LDS while the wave runs the network, so the encoding + MLP phase
// holds only its own values and the kernel fits more waves per SIMD; the ray and the pose
// constants are re-read (L1/L2 resident) when the lane resumes.  One wave per workgroup.

// Parked words per lane, stored [word][64] (lane-consecutive, no bank conflicts).
enum {
    QW_R_LO, QW_R_HI, QW_POSE, QW_NQ, QW_LASTZ, QW_HAS,
    QW_IX, QW_IY, QW_IZ, QW_TMX, QW_TMY, QW_TMZ, QW_TDX, QW_TDY, QW_TDZ, QW_EX, QW_EY, QW_EZ,
    QW_SX, QW_SY, QW_SZ, QW_TLO, QW_LASTA, QW_LASTC, QW_ACTIVE,
    QW_CELL, QW_A, QW_B,
    QW_WORDS
};

struct Parked {
    int32_t* w;
    int lane;
    __device__ __forceinline__ void put(int k, int32_t v) const { w[k * 64 + lane] = v; }
    __device__ __forceinline__ void putf(int k, float v) const { w[k * 64 + lane] = __float_as_int(v); }
    __device__ __forceinline__ int32_t get(int k) const { return w[k * 64 + lane]; }
    __device__ __forceinline__ float getf(int k) const { return __int_as_float(w[k * 64 + lane]); }
};

__device__ __forceinline__ void park_trav(const Parked& pk, const Trav& T) {
    pk.put(QW_IX, T.ix); pk.put(QW_IY, T.iy); pk.put(QW_IZ, T.iz);
    pk.putf(QW_TMX, T.tmx); pk.putf(QW_TMY, T.tmy); pk.putf(QW_TMZ, T.tmz);
    pk.putf(QW_TDX, T.tdx); pk.putf(QW_TDY, T.tdy); pk.putf(QW_TDZ, T.tdz);
    pk.put(QW_EX, T.ex); pk.put(QW_EY, T.ey); pk.put(QW_EZ, T.ez);
    pk.put(QW_SX, T.sx); pk.put(QW_SY, T.sy); pk.put(QW_SZ, T.sz);
    pk.putf(QW_TLO, T.t_lo); pk.putf(QW_LASTA, T.last_a); pk.put(QW_LASTC, T.last_cell); pk.put(QW_ACTIVE, T.active);
}

__device__ __forceinline__ void unpark_trav(const Parked& pk, Trav& T) {
    T.ix = pk.get(QW_IX); T.iy = pk.get(QW_IY); T.iz = pk.get(QW_IZ);
    T.tmx = pk.getf(QW_TMX); T.tmy = pk.getf(QW_TMY); T.tmz = pk.getf(QW_TMZ);
    T.tdx = pk.getf(QW_TDX); T.tdy = pk.getf(QW_TDY); T.tdz = pk.getf(QW_TDZ);
    T.ex = pk.get(QW_EX); T.ey = pk.get(QW_EY); T.ez = pk.get(QW_EZ);
    T.sx = pk.get(QW_SX); T.sy = pk.get(QW_SY); T.sz = pk.get(QW_SZ);
    T.t_lo = pk.getf(QW_TLO); T.last_a = pk.getf(QW_LASTA); T.last_cell = pk.get(QW_LASTC); T.active = pk.get(QW_ACTIVE);
}

#ifndef NIF_QUERY_MIN_WAVES
#define NIF_QUERY_MIN_WAVES 2
#endif

// RPW rays per wave (64, or 16 for launches too small to hide the latency of a network round:
// then a round is one pass of 16 segments instead of four, four lanes search each ray's voxels, and
// four times as many waves run).
template <int HW, int PREC, int RPW, bool GAMMA = false, int FD = 2>
__global__ void __launch_bounds__(64, NIF_QUERY_MIN_WAVES) k_query(NetParams np, GridArgs G, RayArgs R, nif_hits out,
                                              int64_t* __restrict__ counters, int64_t* __restrict__ stats,
                                              int pose_times) {
    static_assert(RPW == 16 || RPW == 64, "rays per wave");
    constexpr int CB = kQueryCB;
    constexpr int PASSES = RPW / 16 / CB;
    constexpr bool REST = RPW == 16 && !GAMMA && FD == 2;      // takes a staged query's list
    __shared__ int32_t s_park[QW_WORDS * 64];
    __shared__ float s_seg[64 * kSegStride];
    __shared__ float s_z[64 * kZStride];
    // With 16 rays a wave, four lanes share a ray: they hold the same state, search its voxels
    // together (next_segment) and the first of them (lead) writes.  idx: the ray within the wave.
    constexpr int SUB = 64 / RPW;
    const int lane = lane_id();
    const int idx = lane / SUB;
    const bool lead = SUB == 1 || lane % SUB == 0;
    const Parked pk{s_park, lane};
    const int n_mat = np.H - 8;

    // Rays are dealt in 8 contiguous ranges, one per XCD: workgroups are dispatched to the
    // XCDs round-robin, so workgroup b starts on range b mod 8 and the waves sharing an L2
    // walk neighbouring rays (coherent rays touch the same table lines).  A wave whose range
    // runs dry moves on to the next one, so the load still balances across the chip.  With
    // pose-ordered dealing, range k is the concatenation over the poses of the k-th eighth of
    // each pose's rays (positions counted in R.order_pre), so every XCD finishes pose p
    // before it starts pose p + 1.
    const int home = (int)(blockIdx.x & 7);
    const int64_t n_rays = REST && R.rest_n ? *R.rest_n : R.n;
    if (REST && n_rays < R.least) return;
    const int64_t span = (n_rays + 7) / 8;
    const int64_t* opre = R.order_pre;
    auto range_of = [&](int id, int64_t& l, int64_t& h) {
        if (opre) {
            l = 0;
            h = opre[(int64_t)id * (R.n_poses + 1) + R.n_poses];
        } else {
            l = std::min<int64_t>((int64_t)id * span, n_rays);
            h = std::min<int64_t>(l + span, n_rays);
        }
    };
    int cur = 0;                                   // ranges tried (wave-uniform); 8 = none left
    int rid = home;
    int64_t lo, hi;
    range_of(rid, lo, hi);
    int bad = 0;
    int64_t n_done = 0, n_eval = 0;
    if (pose_times && lane == 0) atomicMin((unsigned long long*)&stats[4], (unsigned long long)wall_clock64());
    pk.put(QW_R_LO, -1); pk.put(QW_R_HI, -1); pk.put(QW_HAS, 0); pk.put(QW_POSE, 0);

    for (;;) {
        // ---- resume the lane: ray, pose, and the result of the last network round
        int64_t r = (int64_t)(((uint64_t)(uint32_t)pk.get(QW_R_HI) << 32) | (uint32_t)pk.get(QW_R_LO));
        int pose = pk.get(QW_POSE);
        bool has = pk.get(QW_HAS) != 0;
        int nq = 0;
        float last_z0 = -INFINITY;
        Ray ray;
        ray.o = ray.d = make_float3(0.f, 0.f, 0.f);
        Trav tv;
        tv.active = 0;
        PoseDev P;
        P.kind = 0;
        Segment sg;
        sg.cell = -1; sg.a = sg.b = 0.f; sg.face = -1;
        if (r >= 0) {
            nq = pk.get(QW_NQ);
            last_z0 = pk.getf(QW_LASTZ);
            unpark_trav(pk, tv);
            ray = load_ray(R, r);
            P = G.poses[pose];
        }
        bool hitnow = false;
        if (has) {
            ++nq;
            if (lead) ++n_eval;
            const float* z = s_z + idx * kZStride;
            last_z0 = z[0];
            if (z[0] > 0.f) {
                sg.cell = pk.get(QW_CELL); sg.a = pk.getf(QW_A); sg.b = pk.getf(QW_B);
                const float* my = s_seg + idx * kSegStride;
                if (lead) write_hit(out, r, sg, make_float3(my[0], my[1], my[2]), make_float3(my[4], my[5], my[6]), z, nq, n_mat,
                          np.dist_head, R.tmax ? R.tmax[r] : INFINITY, P);
                r = -1;
                if (lead) ++n_done;
                hitnow = lead;
            }
            has = false;
        }
        if (pose_times) note_finished(stats, R.off, R.n_poses, hitnow, pose);

        // ---- give every lane a segment, taking new rays as old ones finish or miss
        for (;;) {
            const bool need = cur < 8 && r < 0;
            const uint64_t m = ballot(need && lead);
            if (m) {
                // a range that is not the wave's own, or few rays: look first
                const int64_t base = take_tickets(&counters[rid], hi - lo, popc64(m), __ffsll((unsigned long long)m) - 1,
                                                  REST && (cur > 0 || R.rest_n));
                if (need) {
                    // rank of the ray's first lane among those that take one
                    r = lo + base + popc64(m & ((1ull << (lane / SUB * SUB)) - 1ull));
                    if (r >= hi) {
                        r = -1;
                    } else {
                        const int64_t at = r;        // in the staged query's list
                        if (REST && R.rest_n) r = R.rest[at];
                        if (opre) {                  // position r of range rid -> (pose, ray)
                            const int64_t* pre = opre + (int64_t)rid * (R.n_poses + 1);
                            int a = 0, b = R.n_poses - 1;
                            while (a < b) {          // last pose p with pre[p] <= r
                                const int mid = (a + b + 1) >> 1;
                                if (pre[mid] <= r) a = mid; else b = mid - 1;
                            }
                            pose = a;
                            const int64_t cnt = R.off[a + 1] - R.off[a];
                            r = R.off[a] + cnt * rid / 8 + (r - pre[a]);
                        } else {
                            pose = find_pose(R.off, R.n_poses, r);
                        }
                        ray = load_ray(R, r);
                        P = G.poses[pose];
                        trav_init(P, ray, tv);
                        nq = 0;
                        last_z0 = -INFINITY;
                        if (REST && R.rest_n && R.rest[kStageRays + at] >= 0) {
                            tv.last_cell = R.rest[kStageRays + at];
                            tv.last_a = __int_as_float(R.rest[2 * kStageRays + at]);
                            last_z0 = __int_as_float(R.rest[3 * kStageRays + at]);
                            nq = 1;
                        }
                    }
                }
                if (lo + base + popc64(m) >= hi) {       // this range is used up: next one
                    ++cur;
                    rid = (home + cur) & 7;
                    range_of(rid, lo, hi);
                }
            }
            const bool search = r >= 0 && !has;
            if (!ballot(search)) {
                if (cur < 8 && ballot(r < 0)) continue;   // lanes still to fill
                break;
            }
            bool missed = false;
            if (search) {
                has = next_segment<SUB>(P, G.V, G.bin_start, G.bin_cells, G.N, ray, tv, sg, &bad);
                if (has && R.tmax && sg.a >= R.tmax[r]) has = false;     // occlusion bound reached
                if (!has) {
                    if (lead) {
                        write_miss(out, r, nq, last_z0);
                        ++n_done;
                    }
                    r = -1;
                    missed = lead;
                }
            }
            if (pose_times) note_finished(stats, R.off, R.n_poses, missed, pose);
        }
        if (!ballot(has)) break;

        // ---- rest-space entry/exit points (local linearization inside the voxel), park, network
        float3 x0 = make_float3(0.5f, 0.5f, 0.5f), x1 = x0;
        if (has) {
            x0 = deform_inv(P, ray_at(ray, sg.a));
            x1 = deform_inv(P, ray_at(ray, sg.b));
        }
        float* my = s_seg + idx * kSegStride;
        my[0] = x0.x; my[1] = x0.y; my[2] = x0.z;
        my[4] = x1.x; my[5] = x1.y; my[6] = x1.z;
        pk.put(QW_R_LO, (int32_t)(uint32_t)(uint64_t)r); pk.put(QW_R_HI, (int32_t)(uint32_t)((uint64_t)r >> 32));
        pk.put(QW_POSE, pose); pk.put(QW_HAS, has ? 1 : 0);
        if (r >= 0) {
            pk.put(QW_NQ, nq); pk.putf(QW_LASTZ, last_z0);
            park_trav(pk, tv);
            pk.put(QW_CELL, sg.cell); pk.putf(QW_A, sg.a); pk.putf(QW_B, sg.b);
        }
        wave_lds_sync();
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) net_pass<HW, CB, PREC, GAMMA, FD>(np, s_seg, ps * 16 * CB, s_z, nullptr, 0, 0, 0);
        wave_lds_sync();
    }
    if (stats) wave_add_stats(stats, n_done, n_eval, bad);
}

// The fused query for few rays: a block of four waves evaluates 16 rays' segments together.  A launch
// of few rays takes its longest ray's chain of rounds, and a round the latency of its lookups and
// layers: here each wave searches four of the rays with 16 lanes each, looks up every fourth batch of
// levels, and computes a quarter of every layer (block_mlp); a wave of 16 rays does all of it in turn.
// The features meet in LDS, in the operands' form; traversal state stays in registers.  Values and
// results are those of k_query.
template <int PREC>
__host__ __device__ constexpr int feat_bytes() { return (int)sizeof(FeatOp<PREC>) * 64; }   // of one batch

template <int HW, int PREC>
__global__ void __launch_bounds__(256) k_query_block(NetParams np, GridArgs G, RayArgs R, nif_hits out, int64_t* __restrict__ counters,
                                                     int64_t* __restrict__ stats) {
    constexpr int SUB = 16;
    extern __shared__ uint4 s_dyn[];                // features [batch][part][lane], 16 bytes each
    __shared__ float s_h[2][16 * (HW + 4)];
    __shared__ float s_seg[16 * kSegStride];
    __shared__ float s_z[16 * kZStride];
    constexpr int PARTS = feat_bytes<PREC>() / 1024;
    const int w = threadIdx.x >> 6, lane = lane_id(), q = lane >> 4, j = lane & 15;
    const int idx = w * 4 + lane / SUB;
    const bool lead = lane % SUB == 0;
    const int64_t n_rays = R.rest_n ? *R.rest_n : R.n;
    if (n_rays > R.most) return;
    const int home = (int)(blockIdx.x & 7);
    const int64_t span = (n_rays + 7) / 8;
    int cur = 0, rid = home;
    int64_t lo = std::min<int64_t>((int64_t)rid * span, n_rays), hi = std::min<int64_t>(lo + span, n_rays);
    const int L = np.enc.L, S = 1 + 2 * np.enc.F, C = 2 * S, U = (C + 3) >> 2, NLB = L >> 2, T = U * NLB;

    int64_t r = -1, n_done = 0, n_eval = 0;
    int pose = 0, nq = 0, bad = 0;
    float last_z0 = -INFINITY;
    bool has = false;
    Ray ray;
    ray.o = ray.d = make_float3(0.f, 0.f, 0.f);
    PoseDev P;
    P.kind = 0;
    Trav tv;
    tv.active = 0;
    Segment sg;
    sg.cell = -1; sg.a = sg.b = 0.f; sg.face = -1;
    for (;;) {
        // ---- give every ray a segment (as k_query)
        for (;;) {
            const bool need = cur < 8 && r < 0;
            const uint64_t m = ballot(need && lead);
            if (m) {
                const int64_t base = take_tickets(&counters[rid], hi - lo, popc64(m), __ffsll((unsigned long long)m) - 1,
                                                  cur > 0 || R.rest_n);
                if (need) {
                    const int64_t at = lo + base + popc64(m & ((1ull << (lane / SUB * SUB)) - 1ull));
                    if (at < hi) {
                        r = R.rest_n ? R.rest[at] : at;
                        pose = find_pose(R.off, R.n_poses, r);
                        ray = load_ray(R, r);
                        P = G.poses[pose];
                        trav_init(P, ray, tv);
                        nq = 0;
                        last_z0 = -INFINITY;
                        if (R.rest_n && R.rest[kStageRays + at] >= 0) {
                            tv.last_cell = R.rest[kStageRays + at];
                            tv.last_a = __int_as_float(R.rest[2 * kStageRays + at]);
                            last_z0 = __int_as_float(R.rest[3 * kStageRays + at]);
                            nq = 1;
                        }
                    }
                }
                if (lo + base + popc64(m) >= hi) {       // this range is used up: next one
                    ++cur;
                    rid = (home + cur) & 7;
                    lo = std::min<int64_t>((int64_t)rid * span, n_rays);
                    hi = std::min<int64_t>(lo + span, n_rays);
                }
            }
            const bool search = r >= 0 && !has;
            if (!ballot(search)) {
                if (cur < 8 && ballot(r < 0)) continue;
                break;
            }
            if (search) {
                has = next_segment<SUB>(P, G.V, G.bin_start, G.bin_cells, G.N, ray, tv, sg, &bad);
                if (has && R.tmax && sg.a >= R.tmax[r]) has = false;     // occlusion bound reached
                if (!has) {
                    if (lead) {
                        write_miss(out, r, nq, last_z0);
                        ++n_done;
                    }
                    r = -1;
                }
            }
        }
        if (!__syncthreads_or(has)) break;

        // ---- rest-space segments, features, MLP
        if (lead) {
            float3 x0 = make_float3(0.5f, 0.5f, 0.5f), x1 = x0;
            if (has) {
                x0 = deform_inv(P, ray_at(ray, sg.a));
                x1 = deform_inv(P, ray_at(ray, sg.b));
            }
            float* my = s_seg + idx * kSegStride;
            my[0] = x0.x; my[1] = x0.y; my[2] = x0.z;
            my[4] = x1.x; my[5] = x1.y; my[6] = x1.z;
        }
        __syncthreads();
        PEWalk pw;
        pw.p = -1;
        pw.k = -1;
        for (int u = 0; u < U; ++u) {
            const int c_raw = q * U + u;
            const bool live = c_raw < C;
            const int c = live ? c_raw : 0;
            uint32_t smp[3] = {0x80000000u, 0x80000000u, 0x80000000u};
            if (live) {
                double v[3];
                pe_walk(s_seg + j * kSegStride, c, S, pw, v);
#pragma unroll
                for (int a = 0; a < 3; ++a) smp[a] = to_fix32(v[a]);
            }
            for (int lb = 0; lb < NLB; ++lb) {
                const int t = u * NLB + lb;
                if ((t & 3) != w) continue;
                FeatRaw fr;
                float* feat = reinterpret_cast<float*>(fr.f);
                const uint32_t soff = combo_set_offset(np.enc, c, S);
                if (np.enc.f16) {
                    lookup_levels<4, true>(np.enc, 4 * lb, smp, feat, soff);
                } else {
#pragma unroll
                    for (int h = 0; h < 4; h += 2) lookup_levels<2, false>(np.enc, 4 * lb + h, smp, feat + 2 * h, soff);
                }
                if (!live)
#pragma unroll
                    for (int k = 0; k < 4; ++k) fr.f[k] = make_float2(0.f, 0.f);
                const FeatOp<PREC> op = feat_op<PREC>(fr);
                uint4 part[PARTS];
                __builtin_memcpy(part, &op, sizeof(op));
#pragma unroll
                for (int k = 0; k < PARTS; ++k) s_dyn[(t * PARTS + k) * 64 + lane] = part[k];
            }
        }
        __syncthreads();
        block_mlp<HW, PREC, FeatOp<PREC>>(np, T, s_h, s_z, nullptr, 0, 0, [&](int t) {
            uint4 part[PARTS];
#pragma unroll
            for (int k = 0; k < PARTS; ++k) part[k] = s_dyn[(t * PARTS + k) * 64 + lane];
            FeatOp<PREC> op;
            __builtin_memcpy(&op, part, sizeof(op));
            return op;
        });

        // ---- results
        if (has) {
            ++nq;
            if (lead) ++n_eval;
            const float* z = s_z + idx * kZStride;
            last_z0 = z[0];
            if (z[0] > 0.f) {
                const float* my = s_seg + idx * kSegStride;
                if (lead) {
                    write_hit(out, r, sg, make_float3(my[0], my[1], my[2]), make_float3(my[4], my[5], my[6]), z, nq, np.H - 8,
                              np.dist_head, R.tmax ? R.tmax[r] : INFINITY, P);
                    ++n_done;
                }
                r = -1;
            }
            has = false;
        }
    }
    if (stats) wave_add_stats(stats, n_done, n_eval, bad);
}

// ------------------------------------------------------------------ launch

// Below this many rays per compute unit a launch is latency-bound (the serial chain of
// network rounds of its longest rays sets the time), and 16-ray waves finish it sooner.
constexpr int64_t kSmallLaunchRaysPerCU = 8192;
// Up to this many, blocks of four waves per 16 rays.  Against 16-ray waves: 4,096 torus rays 225 and
// 409 us, 8,001 rays through 64^3 spheres 210 and 246, 16,001 313 and 296, through 128^3 blobs 627 and
// 692.
constexpr int64_t kBlockRaysPerCU = 64;
constexpr int kBlockFeatBytes = 112 * 1024;

// Launch shape of the fused query: compute units, one-wave workgroups per unit, rays per wave
// (0 = by launch size, else 16 or 64).
struct QueryShape {
    int cus, blocks_per_cu, rays_per_wave;
};

template <int HW, int PREC>
static void launch_query(const QueryShape& sh, const NetParams& np, const GridArgs& G, RayArgs R, const nif_hits& out, int64_t* ctr,
                         int64_t* stats, int pt, hipStream_t st) {
    int rpw = sh.rays_per_wave;
    if (rpw == 0 || R.rest_n) rpw = R.n < kSmallLaunchRaysPerCU * sh.cus || R.rest_n ? 16 : 64;
    // Blocks of 16 rays: few rays, or the part of a staged query's rest that is few.
    const bool plain = np.gamma_F < 0 && np.enc.Fd == 2 && !R.order_pre && !pt && rpw == 16;
    const int feat = (((2 * (1 + 2 * np.enc.F)) + 3) >> 2) * (np.enc.L >> 2) * feat_bytes<PREC>();
    const int64_t few = (int64_t)sh.cus * kBlockRaysPerCU;
    if (plain && feat <= kBlockFeatBytes && (R.rest_n || R.n <= few)) {
        RayArgs B = R;
        if (R.rest_n) B.most = few;
        const int64_t blocks = std::min<int64_t>((std::min(R.n, few) + 15) / 16, (int64_t)sh.cus * 3);
        hipLaunchKernelGGL((k_query_block<HW, PREC>), dim3((unsigned)blocks), dim3(256), feat, st, np, G, B, out, ctr, stats);
        if (!R.rest_n || R.n <= few) return;
        R.least = few + 1;
    }
    const int64_t waves = (R.n + rpw - 1) / rpw;
    const int64_t blocks = std::max<int64_t>(std::min<int64_t>(waves, (int64_t)sh.cus * sh.blocks_per_cu), 1);
    if (np.gamma_F >= 0 || np.enc.Fd == 3) {     // the method variants: one launch shape
        const int64_t b64 = std::max<int64_t>(std::min<int64_t>((R.n + 63) / 64, (int64_t)sh.cus * sh.blocks_per_cu), 1);
        if (np.enc.Fd == 3)
            hipLaunchKernelGGL((k_query<HW, PREC, 64, false, 3>), dim3((unsigned)b64), dim3(64), 0, st, np, G, R, out, ctr, stats, pt);
        else
            hipLaunchKernelGGL((k_query<HW, PREC, 64, true>), dim3((unsigned)b64), dim3(64), 0, st, np, G, R, out, ctr, stats, pt);
    } else if (rpw == 16) {
        hipLaunchKernelGGL((k_query<HW, PREC, 16>), dim3((unsigned)blocks), dim3(64), 0, st, np, G, R, out, ctr, stats, pt);
    } else {
        hipLaunchKernelGGL((k_query<HW, PREC, 64>), dim3((unsigned)blocks), dim3(64), 0, st, np, G, R, out, ctr, stats, pt);
    }
}

template <int PREC>
static int dispatch_query(const QueryShape& sh, int hw, const NetParams& np, const GridArgs& G, const RayArgs& R, const nif_hits& out,
                          int64_t* ctr, int64_t* stats, int pt, hipStream_t st) {
    switch (hw) {
        case 16: launch_query<16, PREC>(sh, np, G, R, out, ctr, stats, pt, st); break;
        case 32: launch_query<32, PREC>(sh, np, G, R, out, ctr, stats, pt, st); break;
        case 64: launch_query<64, PREC>(sh, np, G, R, out, ctr, stats, pt, st); break;
        case 128: launch_query<128, PREC>(sh, np, G, R, out, ctr, stats, pt, st); break;
        default: return fail(NIF_E_UNSUPPORTED, "hidden_width must be 16, 32, 64 or 128");
    }
    return NIF_OK;
}

// One translation unit per precision.
int query_fp32(const QueryShape& sh, int hw, const NetParams& np, const GridArgs& G, const RayArgs& R, const nif_hits& out,
               int64_t* ctr, int64_t* stats, int pt, hipStream_t st);
int query_bf16(const QueryShape& sh, int hw, const NetParams& np, const GridArgs& G, const RayArgs& R, const nif_hits& out,
               int64_t* ctr, int64_t* stats, int pt, hipStream_t st);
int query_fp16(const QueryShape& sh, int hw, const NetParams& np, const GridArgs& G, const RayArgs& R, const nif_hits& out,
               int64_t* ctr, int64_t* stats, int pt, hipStream_t st);

}  // namespace nif
