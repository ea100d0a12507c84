// The encoding of many point pairs, table level by table level.
//
// The fused kernels walk, per 16 segments, every PE combination and level, so the tables of all
// levels (32 MiB at 16 levels of 2^19 FP16 entries) pass through each XCD's 4 MB L2 together and
// most corner loads miss it: random gathers from 32 MiB run at 65 G/s on this GPU, from up to
// 4 MiB at 264 G/s.  Here all segments of a chunk are encoded at one level before the next, so
// the level's table (2 MiB) stays in every L2, and the features go to memory as panels that the
// MLP kernels read back with full lines.
//
// Panels: enc[g][i][2], g = l C + c: the two features of level l, PE combination c (point-major,
// C = 2 S of them) of segment i; rows of panel_stride(n) segments, so that pairs of segments are
// 16-byte aligned.  Positions: pos[c][axis][i], 32-bit fixed point, the same row length.
// Both hold exactly the values the fused kernels form in registers.  nif_encode uses the same form
// for single points: C = S combinations, FP64 positions.
#pragma once
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "nif_net.hpp"

namespace nif {

__host__ __device__ inline int64_t panel_stride(int64_t n) { return (n + 15) & ~(int64_t)15; }

// Cell and weight of a position on one axis: 32-bit fixed point, or FP64.
__device__ __forceinline__ void axis_at(uint32_t f, uint32_t N, uint32_t& i0, float& w) { fix_axis(f, N, i0, w); }
__device__ __forceinline__ void axis_at(double s, uint32_t N, uint32_t& i0, float& w) { grid_axis(s, (int)N, i0, w); }

// Interpolated features of KC positions at one (wave-uniform) level: the lookup of
// lookup_levels with the roles of levels and positions exchanged, the same arithmetic in the
// same order.
template <int KC, bool F16, class Pos>
__device__ __forceinline__ void lookup_points(const EncParams& ep, int l, const Pos (&f)[KC][3],
                                              const uint32_t (&set_off)[KC], float2 (&out)[KC]) {
    using E = typename TabTypes<F16>::E;
    using Pr = typename TabTypes<F16>::Pr;
    const E* tab = reinterpret_cast<const E*>(ep.tab);
    const uint32_t mask = (1u << ep.log2T) - 1u;
    const uint32_t N = (uint32_t)ep.res[l];
    const bool dense = (ep.dense_mask >> l) & 1u;
    Pr A[KC][4];
    E B[KC][4];
    uint32_t swp[KC], odd[KC];
    float wx[KC], wy[KC], wz[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        uint32_t ix, iy, iz;
        axis_at(f[k][0], N, ix, wx[k]);
        axis_at(f[k][1], N, iy, wy[k]);
        axis_at(f[k][2], N, iz, wz[k]);
        swp[k] = odd[k] = 0u;
        const E* tl = tab + (set_off[k] + ((uint32_t)l << ep.log2T));
        if (dense) {
            const uint32_t n1 = N + 1u;
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                const uint32_t e = ix + n1 * ((iy + (pp & 1)) + n1 * (iz + (pp >> 1)));
                __builtin_memcpy(&A[k][pp], tl + e, sizeof(Pr));
            }
        } else {
            odd[k] = ix & 1u;
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                const uint32_t hyz = ((iy + (pp & 1)) * 2654435761u) ^ ((iz + (pp >> 1)) * 805459861u);
                const uint32_t h0 = (ix ^ hyz) & mask;
                swp[k] |= (h0 & 1u) << pp;
                __builtin_memcpy(&A[k][pp], tl + (h0 & ~1u), sizeof(Pr));
            }
            if (odd[k]) {
#pragma unroll
                for (int pp = 0; pp < 4; ++pp) {
                    const uint32_t hyz = ((iy + (pp & 1)) * 2654435761u) ^ ((iz + (pp >> 1)) * 805459861u);
                    B[k][pp] = tl[((ix + 1u) ^ hyz) & mask];
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        float2 acc = make_float2(0.f, 0.f);
#pragma unroll
        for (int pp = 0; pp < 4; ++pp) {
            E lo, hi;
            pair_split(A[k][pp], lo, hi);
            const bool swap = (swp[k] >> pp) & 1u;
            const E e0 = sel(swap, hi, lo);
            const E e1 = odd[k] ? B[k][pp] : sel(swap, lo, hi);
#pragma unroll
            for (int cx = 0; cx < 2; ++cx) {
                const int c = 2 * pp + cx;
                const float wt = (cx ? wx[k] : 1.f - wx[k]) * (((c >> 1) & 1) ? wy[k] : 1.f - wy[k]) *
                                 (((c >> 2) & 1) ? wz[k] : 1.f - wz[k]);
                const float2 v = entry_f2(cx ? e1 : e0);
                acc.x = fmaf(wt, v.x, acc.x);
                acc.y = fmaf(wt, v.y, acc.y);
            }
        }
        out[k] = acc;
    }
}

// Point pairs have fixed-point positions and two points of S samples, single points S FP64 samples.
template <class Pos>
__host__ __device__ constexpr int combinations(int S) { return std::is_same<Pos, double>::value ? S : 2 * S; }

// Pairs of a launch whose number only the device knows (nif_query's segments): slot `slot` of the
// fewest equal parts of at most `chunk` pairs that min(*count, cap) pairs make.  Without a count the
// launch's own n pairs from 0.
struct Live {
    const int32_t* count;
    int32_t cap, chunk, slot;
};
__device__ __forceinline__ void live_range(const Live& L, int64_t& first, int64_t& n) {
    first = 0;
    if (!L.count) return;
    const int32_t total = min(*L.count, L.cap), k = (total + L.chunk - 1) / L.chunk;
    if (L.slot >= k) { n = 0; return; }
    const int32_t size = ((total + k - 1) / k + 255) & ~255;
    first = (int64_t)L.slot * size;
    n = max((int64_t)0, min((int64_t)size, total - first));
}

// Work of a level-by-level pass: which (level, part) items each XCD goes through, in order.  A part is
// a share of the level's (combination group, segment tile) workgroups.  Workgroup b runs on XCD
// b mod 8 (round-robin dispatch; only the speed depends on it).
constexpr int kEncXcds = 8, kEncMaxItems = 16;
constexpr int kEncKC = 2;           // combinations per thread
struct EncPlan {
    int32_t tiles;                  // segment tiles
    int32_t groups;                 // groups of combinations
    int32_t parts;                  // parts per level
    int32_t per_item;               // workgroups of one part
    int32_t most;                   // items of the fullest XCD
    uint8_t n_items[kEncXcds];
    uint8_t item[kEncXcds][kEncMaxItems];   // level * parts + part
};

// Items of a level-by-level pass.  Two parts per level, dealt to the XCDs longest first: an
// XCD then stays on one level for half of its lookups, and the waves of two levels overlap for a
// small share of the time (2^17 ordered pairs: 0.72 ms; with every level spread over all XCDs,
// where the levels overlap for a third of the time, 0.86; whole levels, unbalanced, 0.84).  A
// hashed level counts twice a dense one (6 against 4 loads, fewer of them in L1).  Tables that
// fit an L2 together need no such care: every level is spread evenly.
inline EncPlan level_plan(const EncParams& ep, int64_t tiles, int groups) {
    EncPlan P;
    memset(&P, 0, sizeof(P));
    P.tiles = (int32_t)tiles;
    P.groups = groups;
    const int64_t table_bytes = ((int64_t)ep.L << ep.log2T) * (ep.f16 ? 4 : 8);
    P.parts = table_bytes <= (4 << 20) ? kEncXcds : 2;
    P.per_item = (int32_t)(((int64_t)P.tiles * P.groups + P.parts - 1) / P.parts);
    int load[kEncXcds] = {};
    for (int pass = 0; pass < 2; ++pass)                // hashed levels first
        for (int l = 0; l < ep.L; ++l) {
            const bool dense = (ep.dense_mask >> l) & 1u;
            if (dense != (pass == 1)) continue;
            for (int k = 0; k < P.parts; ++k) {
                int x = 0;
                for (int y = 1; y < kEncXcds; ++y)
                    if (load[y] < load[x]) x = y;
                P.item[x][P.n_items[x]++] = (uint8_t)(l * P.parts + k);
                load[x] += dense ? 1 : 2;
            }
        }
    P.most = 0;
    for (int x = 0; x < kEncXcds; ++x) P.most = std::max<int32_t>(P.most, P.n_items[x]);
    return P;
}
inline unsigned plan_blocks(const EncPlan& P) { return (unsigned)(kEncXcds * P.most * (int64_t)P.per_item); }

// The (level, combination group, tile) of item v of an XCD's workgroups; false if there is none.
__device__ __forceinline__ bool plan_item(const EncPlan& P, int x, int v, int tiles, int per_item, int& l, int& grp, int& tile) {
    const int item = P.item[x][v / per_item];
    l = item / P.parts;
    const int b = (item % P.parts) * per_item + v % per_item;           // workgroup within the level
    grp = b / tiles;
    tile = b % tiles;
    return grp < P.groups;
}
// The item of this workgroup in a launch of plan_blocks workgroups.
__device__ __forceinline__ bool plan_item(const EncPlan& P, int& l, int& grp, int& tile) {
    const int x = (int)(blockIdx.x % kEncXcds), v = (int)(blockIdx.x / kEncXcds);
    return v < P.n_items[x] * P.per_item && plan_item(P, x, v, P.tiles, P.per_item, l, grp, tile);
}

// Bound: the rate at which L1 and L2 take the lanes' corner requests (about 5 distinct lines per
// lookup on hashed levels).  2^17 spatially ordered pairs at 16 levels of 2^19 FP16 entries:
// 0.72 ms (75 G lookups/s); the fused forward of the same pairs took 1.44 ms, 4,096 pairs 41
// against 277 us.  Two combinations per thread keep 8 to 16 loads in flight; one takes 0.75 ms,
// four (fewer waves) 0.84.
template <int KC, bool F16, class Pos>
__global__ void __launch_bounds__(256) k_encode_levels(EncParams ep, EncPlan plan, const Pos* __restrict__ pos,
                                                       int64_t n, float2* __restrict__ enc, Live lv) {
    const int S = 1 + 2 * ep.F, C = combinations<Pos>(S);
    int64_t first;
    live_range(lv, first, n);
    const int tiles = (int)((n + 255) / 256);
    const int per_item = (int)(((int64_t)tiles * plan.groups + plan.parts - 1) / plan.parts);
    const int64_t pn = panel_stride(n);
    const int x = (int)(blockIdx.x % kEncXcds);
    for (int v = (int)(blockIdx.x / kEncXcds); v < plan.n_items[x] * per_item; v += (int)(gridDim.x / kEncXcds)) {
        int l, grp, tile;
        if (!plan_item(plan, x, v, tiles, per_item, l, grp, tile)) continue;
        const int64_t i = (int64_t)tile * 256 + threadIdx.x;
        if (i >= n) continue;
        Pos f[KC][3];
        uint32_t so[KC];
        float2 o[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int c = min(grp * KC + k, C - 1);
            so[k] = combo_set_offset(ep, c, S);
#pragma unroll
            for (int a = 0; a < 3; ++a) f[k][a] = pos[((int64_t)c * 3 + a) * pn + i];
        }
        lookup_points<KC, F16, Pos>(ep, l, f, so, o);
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int c = grp * KC + k;
            if (c < C) enc[((int64_t)l * C + c) * pn + i] = o[k];
        }
    }
}

// Levels whose entries fit an LDS: encoded from there.  A block of 1024 threads copies the level's
// table (at most kLdsTableBytes) and looks up its share of the (combination, segment) pairs; the
// corners cost LDS reads instead of L2 requests, which bound k_encode_levels (16,212 pairs at 8
// levels of 2^14 FP32 entries: 58 us there).
constexpr int kLdsTableBytes = 152 * 1024;
struct LdsPlan {
    int32_t n;                  // levels
    uint8_t lev[16];
    uint16_t blocks[16];        // blocks of each, by its lookups
    int32_t entries[16];        // entries in use
    int32_t total, bytes;       // blocks in all, largest table
};
inline LdsPlan lds_plan(const EncParams& ep, int64_t lookups, int cus) {
    LdsPlan P;
    memset(&P, 0, sizeof(P));
    if (ep.set_stride) return P;                        // one table set per sample: too many tables
    const int size = ep.f16 ? 4 : 8;
    for (int l = 0; l < ep.L; ++l) {
        const int64_t n1 = ep.res[l] + 1;
        const int64_t e = (ep.dense_mask >> l) & 1u ? n1 * n1 * n1 : (int64_t)1 << ep.log2T;
        if (e * size > kLdsTableBytes) continue;
        P.lev[P.n] = (uint8_t)l;
        P.entries[P.n] = (int32_t)e;
        P.bytes = std::max<int32_t>(P.bytes, (int32_t)((e * size + 15) / 16 * 16));
        ++P.n;
    }
    for (int k = 0; k < P.n; ++k) {
        // one block per compute unit over all levels, each with enough lookups to pay for the copy
        const int64_t least = std::max<int64_t>(4096, P.entries[k] / 2);
        P.blocks[k] = (uint16_t)std::max<int64_t>(1, std::min<int64_t>(lookups / least, cus / P.n));
        P.total += P.blocks[k];
    }
    return P;
}

template <bool F16, class Pos>
__global__ void __launch_bounds__(1024) k_encode_lds(EncParams ep, LdsPlan plan, const Pos* __restrict__ pos, int64_t n_pairs,
                                                     float2* __restrict__ enc, Live lv) {
    using E = typename TabTypes<F16>::E;
    extern __shared__ uint4 s_raw[];
    int64_t first;
    live_range(lv, first, n_pairs);
    const uint32_t n = (uint32_t)n_pairs;
    if (n == 0) return;
    E* s_tab = reinterpret_cast<E*>(s_raw);
    int k = 0, b = (int)blockIdx.x;
    while (b >= plan.blocks[k]) b -= plan.blocks[k++];
    const int l = plan.lev[k], G = plan.blocks[k];
    const E* tab = reinterpret_cast<const E*>(ep.tab) + ((size_t)l << ep.log2T);
    for (int e = threadIdx.x; e < plan.entries[k]; e += 1024) s_tab[e] = tab[e];
    __syncthreads();
    const uint32_t C = combinations<Pos>(1 + 2 * ep.F), all = C * n;
    const int64_t pn = panel_stride(n);
    const uint32_t f0 = (uint32_t)((uint64_t)all * b / G), f1 = (uint32_t)((uint64_t)all * (b + 1) / G);
    const uint32_t N = (uint32_t)ep.res[l], n1 = N + 1u, mask = (1u << ep.log2T) - 1u;
    const bool dense = (ep.dense_mask >> l) & 1u;
    for (uint32_t f = f0 + threadIdx.x; f < f1; f += 1024) {
        const uint32_t c = f / n, i = f - c * n;
        const Pos* p = pos + (int64_t)c * 3 * pn + i;
        uint32_t ix, iy, iz;
        float wx, wy, wz;
        axis_at(p[0], N, ix, wx);
        axis_at(p[pn], N, iy, wy);
        axis_at(p[2 * pn], N, iz, wz);
        E v[4][2];
        if (dense) {
            const uint32_t e = ix + n1 * (iy + n1 * iz);
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                const uint32_t o = e + ((pp & 1) ? n1 : 0u) + ((pp >> 1) ? n1 * n1 : 0u);
                v[pp][0] = s_tab[o];
                v[pp][1] = s_tab[o + 1];
            }
        } else {
            const uint32_t y0 = iy * 2654435761u, z0 = iz * 805459861u;
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                const uint32_t hyz = (y0 + ((pp & 1) ? 2654435761u : 0u)) ^ (z0 + ((pp >> 1) ? 805459861u : 0u));
                v[pp][0] = s_tab[(ix ^ hyz) & mask];
                v[pp][1] = s_tab[((ix + 1u) ^ hyz) & mask];
            }
        }
        float2 acc = make_float2(0.f, 0.f);
#pragma unroll
        for (int pp = 0; pp < 4; ++pp)
#pragma unroll
            for (int cx = 0; cx < 2; ++cx) {
                const float wt = (cx ? wx : 1.f - wx) * ((pp & 1) ? wy : 1.f - wy) * ((pp >> 1) ? wz : 1.f - wz);
                const float2 e = entry_f2(v[pp][cx]);
                acc.x = fmaf(wt, e.x, acc.x);
                acc.y = fmaf(wt, e.y, acc.y);
            }
        enc[((int64_t)l * C + c) * pn + i] = acc;
    }
}

// First layer of segments i0 .. i0 + 16 CB - 1 (of n) from their panels, added to acc: the MFMA
// steps of layer1_levels in the same order on the same values (lane (q, j) supplies combination
// q U + u of segment j, level batches of 4), with the next batch's features and weights in flight
// while this batch multiplies (FP32 at width 128 and CB > 1: features only; a batch's MFMAs take
// 4,096 cycles there and the weights' registers are the accumulators').
template <int HW, int CB, int PREC>
__device__ __forceinline__ void layer1_panels(const NetParams& np, const float2* __restrict__ enc, int64_t n, int64_t i0,
                                              floatx4 (&acc)[HW / 16][CB]) {
    constexpr int OB = HW / 16;
    constexpr bool AHEAD = PREC != P_FP32 || CB == 1 || HW < 128;
    using W = typename std::conditional<PREC == P_FP32, float4, shortx4>::type;     // half a lane's weights of a batch
    const int lane = lane_id(), q = lane >> 4, j = lane & 15;
    const int L = np.enc.L, C = 2 * (1 + 2 * np.enc.F), U = (C + 3) >> 2, NLB = L >> 2;
    const int64_t pn = panel_stride(n);
    const W* w0 = reinterpret_cast<const W*>(np.W0L) + lane;
    int64_t row[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) row[cb] = min(i0 + cb * 16 + j, n - 1);
    auto load = [&](int t, float2 (&f)[CB][4]) {           // batch t = u NLB + lb
        const int u = t / NLB, lb = t - u * NLB;
        const int c = q * U + u;
        const bool live = c < C;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float2* p = enc + ((int64_t)(4 * lb + k) * C + (live ? c : 0)) * pn;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                f[cb][k] = p[row[cb]];
                if (!live) f[cb][k] = make_float2(0.f, 0.f);
            }
        }
    };
    const int T = U * NLB;
    auto weights = [&](int t, W (&w)[OB][2]) {
#pragma unroll
        for (int ob = 0; ob < OB; ++ob) {
            const W* p = w0 + ((size_t)ob * T + t) * 128;
            w[ob][0] = p[0];
            w[ob][1] = p[64];
        }
    };
    float2 nx[CB][4];
    W wn[OB][2];
    load(0, nx);
    if constexpr (AHEAD) weights(0, wn);
    for (int t = 0; t < T; ++t) {
        float2 f[CB][4];
        W w[OB][2];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int k = 0; k < 4; ++k) f[cb][k] = nx[cb][k];
        if constexpr (AHEAD) {
#pragma unroll
            for (int ob = 0; ob < OB; ++ob) { w[ob][0] = wn[ob][0]; w[ob][1] = wn[ob][1]; }
        } else {
            weights(t, w);
        }
        if (t + 1 < T) {
            load(t + 1, nx);
            if constexpr (AHEAD) weights(t + 1, wn);
        }
        if constexpr (PREC == P_FP32) {
#pragma unroll
            for (int ob = 0; ob < OB; ++ob) {
                const float wf[8] = {w[ob][0].x, w[ob][0].y, w[ob][0].z, w[ob][0].w,
                                     w[ob][1].x, w[ob][1].y, w[ob][1].z, w[ob][1].w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) acc[ob][cb] = mfma32(wf[2 * k], f[cb][k].x, acc[ob][cb]);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) acc[ob][cb] = mfma32(wf[2 * k + 1], f[cb][k].y, acc[ob][cb]);
                }
            }
        } else {
            shortx4 pk[CB][2];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    pk[cb][h] = pack4<PREC>(f[cb][2 * h].x, f[cb][2 * h].y, f[cb][2 * h + 1].x, f[cb][2 * h + 1].y);
#pragma unroll
            for (int ob = 0; ob < OB; ++ob)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) acc[ob][cb] = mfma16<PREC>(w[ob][h], pk[cb][h], acc[ob][cb]);
        }
    }
}

// First-layer operands of one batch (four levels of one combination) as a lane holds them: features,
// and packed for the 16-bit MFMAs.
struct FeatRaw {
    float2 f[4];
};
template <int PREC>
struct FeatOp {
    shortx4 v[2];
};
template <>
struct FeatOp<P_FP32> {
    float2 f[4];
};
template <int PREC>
__device__ __forceinline__ FeatOp<PREC> feat_op(const FeatRaw& r) {
    FeatOp<PREC> o;
    if constexpr (PREC == P_FP32) {
#pragma unroll
        for (int k = 0; k < 4; ++k) o.f[k] = r.f[k];
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) o.v[h] = pack4<PREC>(r.f[2 * h].x, r.f[2 * h].y, r.f[2 * h + 1].x, r.f[2 * h + 1].y);
    }
    return o;
}
template <int PREC>
__device__ __forceinline__ const FeatOp<PREC>& feat_op(const FeatOp<PREC>& o) { return o; }

// MLP of 16 pairs by a block of four waves, each computing a quarter of every layer's output blocks:
// the layers' activations meet in LDS (s_h), DEPTH batches of first-layer operands are in flight.  The
// MFMA steps of every output are those of the one-wave forms.  load(t): operands of batch t.
// acts (nullable): activations [layer][act_rows][HW], row seg, if seg < act_rows.  Ends with the heads in
// s_z after a barrier.
template <int HW, int PREC, class Raw, class Load>
__device__ __forceinline__ void block_mlp(const NetParams& np, int T, float (*s_h)[16 * (HW + 4)], float* s_z, float* acts,
                                          int64_t act_rows, int64_t seg, Load load) {
    constexpr int OB = HW / 16, WB = OB >= 4 ? OB / 4 : 1;         // output blocks, of one wave
    constexpr int LDA = HW + 4;
    constexpr int DEPTH = 4;
    using W = typename std::conditional<PREC == P_FP32, float4, shortx4>::type;
    const int w = threadIdx.x >> 6, lane = lane_id(), q = lane >> 4, j = lane & 15;
    const bool live_w = w * WB < OB;
    const W* wl = reinterpret_cast<const W*>(np.W0L) + (size_t)(live_w ? w * WB : 0) * T * 128 + lane;
    floatx4 acc[WB];
    if (live_w) {
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            const float4 bb = *reinterpret_cast<const float4*>(np.b[0] + (w * WB + b) * 16 + 4 * q);
            acc[b] = floatx4{bb.x, bb.y, bb.z, bb.w};
        }
        Raw f[DEPTH];
        W wt[DEPTH][WB][2];
        auto fetch = [&](int t, Raw& ff, W (&ww)[WB][2]) {
            ff = load(t);
#pragma unroll
            for (int b = 0; b < WB; ++b) {
                ww[b][0] = wl[((size_t)b * T + t) * 128];
                ww[b][1] = wl[((size_t)b * T + t) * 128 + 64];
            }
        };
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (d < T) fetch(d, f[d], wt[d]);
        for (int t0 = 0; t0 < T; t0 += DEPTH)
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                if (t0 + d >= T) break;
                const FeatOp<PREC> op = feat_op<PREC>(f[d]);
                if constexpr (PREC == P_FP32) {
#pragma unroll
                    for (int b = 0; b < WB; ++b) {
                        const float wf[8] = {wt[d][b][0].x, wt[d][b][0].y, wt[d][b][0].z, wt[d][b][0].w,
                                             wt[d][b][1].x, wt[d][b][1].y, wt[d][b][1].z, wt[d][b][1].w};
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            acc[b] = mfma32(wf[2 * k], op.f[k].x, acc[b]);
                            acc[b] = mfma32(wf[2 * k + 1], op.f[k].y, acc[b]);
                        }
                    }
                } else {
#pragma unroll
                    for (int b = 0; b < WB; ++b)
#pragma unroll
                        for (int h = 0; h < 2; ++h) acc[b] = mfma16<PREC>(wt[d][b][h], op.v[h], acc[b]);
                }
                if (t0 + d + DEPTH < T) fetch(t0 + d + DEPTH, f[d], wt[d]);
            }
    }
    for (int layer = 1; layer <= np.n_hidden; ++layer) {
        float* h = s_h[layer & 1];
        if (live_w) {
#pragma unroll
            for (int b = 0; b < WB; ++b) {
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[b][r] = fmaxf(acc[b][r], 0.f);
                const float4 v = make_float4(acc[b][0], acc[b][1], acc[b][2], acc[b][3]);
                const int o = (w * WB + b) * 16 + 4 * q;
                *reinterpret_cast<float4*>(h + j * LDA + o) = v;
                if (acts && seg < act_rows)
                    *reinterpret_cast<float4*>(acts + (int64_t)(layer - 1) * act_rows * HW + seg * HW + o) = v;
            }
        }
        __syncthreads();
        const bool is_out = layer == np.n_hidden;
        if (is_out ? w == 0 : live_w) {
            const float* bl = np.b[layer];
#pragma unroll
            for (int b = 0; b < WB; ++b) {
                if (is_out && b > 0) break;
                const int oo = is_out ? 0 : w * WB + b;
                const float4 bb = *reinterpret_cast<const float4*>(bl + oo * 16 + 4 * q);
                floatx4 o = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
                for (int ib = 0; ib < OB; ++ib) {
                    const float4 x = *reinterpret_cast<const float4*>(h + j * LDA + ib * 16 + 4 * q);
                    const size_t at = (size_t)(oo * 16 + j) * HW + ib * 16 + 4 * q;
                    if constexpr (PREC == P_FP32) {
                        const float4 wv = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(np.W[layer]) + at);
                        o = mfma32(wv.x, x.x, o);
                        o = mfma32(wv.y, x.y, o);
                        o = mfma32(wv.z, x.z, o);
                        o = mfma32(wv.w, x.w, o);
                    } else {
                        const shortx4 wa = *reinterpret_cast<const shortx4*>(reinterpret_cast<const uint16_t*>(np.W[layer]) + at);
                        o = mfma16<PREC>(wa, pack4<PREC>(x.x, x.y, x.z, x.w), o);
                    }
                }
                acc[b] = o;
            }
            if (is_out)
#pragma unroll
                for (int r = 0; r < 4; ++r) s_z[j * kZStride + 4 * q + r] = acc[0][r];
        }
    }
    __syncthreads();
}

}  // namespace nif
