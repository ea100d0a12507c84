// The network on given rest-space points: nif_encode, nif_forward and the training forward.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "nif_internal.hpp"
#include "nif_panels.hpp"

namespace nif {

// ------------------------------------------------------------------ network on given points

// Full encoding of n points: out[i][(s L + l) Fd + f], one thread per (point, level).  For three
// features and the concatenated form, which have no panels.
__global__ void __launch_bounds__(256) k_encode(EncParams ep, const float* __restrict__ x, int64_t n,
                                                float* __restrict__ out) {
    const int S = 1 + 2 * ep.F;
    const int W = S * ep.L * ep.Fd;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * ep.L; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / ep.L;
        const int l = (int)(e - i * ep.L);
        PEState pe;
        pe_begin(pe, x[i], x[n + i], x[2 * n + i]);
        for (int s = 0; s < S; ++s) {
            double smp[3];
            pe_sample(pe, s, smp);
            float* o = out + i * W + (s * ep.L + l) * ep.Fd;
            if (ep.f16) grid_lookup_any<true>(ep, l, smp[0], smp[1], smp[2], set_offset(ep, s), o);
            else grid_lookup_any<false>(ep, l, smp[0], smp[1], smp[2], set_offset(ep, s), o);
        }
    }
}

// FP64 PE samples of n points (SoA, stride ld): pos[s][axis][i].
__global__ void __launch_bounds__(64) k_samples(int F, const float* __restrict__ x, int64_t n, int64_t ld,
                                                double* __restrict__ pos) {
    const int S = 1 + 2 * F;
    const int64_t pn = panel_stride(n), i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (i >= n) return;
    PEState pe;
    pe_begin(pe, x[i], x[ld + i], x[2 * ld + i]);
    for (int s = 0; s < S; ++s) {
        double smp[3];
        pe_sample(pe, s, smp);
#pragma unroll
        for (int a = 0; a < 3; ++a) pos[((int64_t)s * 3 + a) * pn + i] = smp[a];
    }
}

// Panels of single points to rows: out[i][s L + l] from enc[l S + s][i], two floats each, by tiles of
// 64 x 64 through LDS, so that both sides move full lines.  Bound: memory (60,001 points at 16 levels
// and 13 samples: 100 MB each way).
__global__ void __launch_bounds__(256) k_panel_rows(int S, int L, const float2* __restrict__ enc, int64_t n,
                                                    float* __restrict__ out) {
    __shared__ float2 s_t[64][65];
    const int64_t pn = panel_stride(n), i0 = (int64_t)blockIdx.x * 64;
    const int G = S * L, g0 = (int)blockIdx.y * 64;
    const int a = threadIdx.x & 63, b = threadIdx.x >> 6;
    for (int k = b; k < 64 && g0 + k < G; k += 4) {
        const int s = (g0 + k) / L, l = (g0 + k) - s * L;
        if (i0 + a < n) s_t[k][a] = enc[((int64_t)l * S + s) * pn + i0 + a];
    }
    __syncthreads();
    if (g0 + a >= G) return;
    for (int p = b; p < 64 && i0 + p < n; p += 4) {
        const float2 v = s_t[a][p];
        __builtin_memcpy(out + ((i0 + p) * G + g0 + a) * 2, &v, sizeof(v));     // any float's alignment
    }
}

// Heads of point pairs for the method variants (concatenated encoding, three features) and for few
// pairs of small networks, gathers and MLP fused.  Each wave evaluates tiles of TILE pairs; acts (nullable) receives the hidden
// activations [layer][B][HW] and enc (nullable) the encoding [B][E], for the training backward.
// x0 / x1 are SoA with row stride ld >= B.
template <int HW, int PREC, bool GAMMA, int TILE, int FD>
__global__ void __launch_bounds__(256, 2) k_forward(NetParams np, const float* __restrict__ x0, const float* __restrict__ x1,
                                                 int64_t B, int64_t ld, float* __restrict__ heads,
                                                 float* __restrict__ acts, float* __restrict__ enc) {
    constexpr int CB = TILE == 16 || HW >= 128 ? 1 : 4;
    constexpr int PASSES = TILE / 16 / CB;
    __shared__ float s_seg_all[4][64 * kSegStride];
    __shared__ float s_z_all[4][64 * kZStride];
    const int w = threadIdx.x >> 6;
    const int lane = lane_id();
    float* s_seg = s_seg_all[w];
    float* s_z = s_z_all[w];
    const int64_t n_tiles = (B + TILE - 1) / TILE;
    const int64_t wave_g = (int64_t)blockIdx.x * 4 + w, n_waves = (int64_t)gridDim.x * 4;
    for (int64_t tile = wave_g; tile < n_tiles; tile += n_waves) {
        const int64_t seg = tile * TILE + lane;
        float* my = s_seg + lane * kSegStride;
        if (lane < TILE && seg < B) {
            my[0] = x0[seg]; my[1] = x0[ld + seg]; my[2] = x0[2 * ld + seg];
            my[4] = x1[seg]; my[5] = x1[ld + seg]; my[6] = x1[2 * ld + seg];
        } else {
            my[0] = my[1] = my[2] = my[4] = my[5] = my[6] = 0.5f;
        }
        wave_lds_sync();
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps)
            net_pass<HW, CB, PREC, GAMMA, FD>(np, s_seg, ps * 16 * CB, s_z, acts, B * HW, tile * TILE + ps * 16 * CB, B, enc);
        wave_lds_sync();
        if (lane < TILE && seg < B)
            for (int h = 0; h < np.H; ++h) heads[seg * np.H + h] = s_z[lane * kZStride + h];
        wave_lds_sync();
    }
}

// Fixed-point PE samples of n point pairs (SoA, stride ld): pos[c][axis][i].  One thread per
// (pair, quarter of the combinations), the runs of layer1_levels, so that the double-angle
// recurrence starts where it does there.
__global__ void __launch_bounds__(256) k_positions(int F, const float* __restrict__ x0, const float* __restrict__ x1,
                                                   int64_t n, int64_t ld, uint32_t* __restrict__ pos, Live lv) {
    const int S = 1 + 2 * F, C = 2 * S, U = (C + 3) >> 2;
    int64_t first;
    live_range(lv, first, n);
    x0 += first;
    x1 += first;
    const int q = blockIdx.y;
    const int64_t pn = panel_stride(n);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float sp[8] = {x0[i], x0[ld + i], x0[2 * ld + i], 0.f, x1[i], x1[ld + i], x1[2 * ld + i], 0.f};
        PEWalk w;
        w.p = -1;
        w.k = -1;
        for (int u = 0; u < U; ++u) {
            const int c = q * U + u;
            if (c >= C) break;
            double v[3];
            pe_walk(sp, c, S, w, v);
#pragma unroll
            for (int a = 0; a < 3; ++a) pos[((int64_t)c * 3 + a) * pn + i] = to_fix32(v[a]);
        }
    }
}

// Heads of n point pairs from their panels: the first layer reads them as MFMA operands, the
// rest of the MLP as in the fused kernels.  acts as in k_forward.  A wave takes 16 CB pairs, so
// its first-layer weights (229 KB at width 64 in FP32, streamed through L1) serve CB columns.
// Bound: at width 128 the FP32 MFMA rate (41 GFLOP per 2^17 pairs), in 16 bits the panels' bytes.
template <int HW, int CB, int PREC>
__global__ void __launch_bounds__(256, 2) k_mlp_panels(NetParams np, const float2* __restrict__ enc, int64_t n,
                                                       float* __restrict__ heads, float* __restrict__ acts, Live lv) {
    int64_t first;
    live_range(lv, first, n);
    heads += first * np.H;
    __shared__ float s_z_all[4][16 * CB * kZStride];
    const int w = threadIdx.x >> 6, lane = lane_id();
    float* s_z = s_z_all[w];
    const int64_t n_tiles = (n + 16 * CB - 1) / (16 * CB);
    const int64_t n_waves = (int64_t)gridDim.x * 4;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + w; tile < n_tiles; tile += n_waves) {
        const int64_t i0 = tile * 16 * CB;
        floatx4 acc[HW / 16][CB];
        layer1_bias<HW, CB>(np, acc);
        layer1_panels<HW, CB, PREC>(np, enc, n, i0, acc);
        mlp_tail<HW, CB, PREC>(np, acc, 0, s_z, acts, n * HW, i0, n);
        wave_lds_sync();
        if (lane < 16 * CB && i0 + lane < n)
            for (int h = 0; h < np.H; ++h) heads[(i0 + lane) * np.H + h] = s_z[lane * kZStride + h];
        wave_lds_sync();
    }
}

// The same for launches too small to fill the chip with waves of 16 pairs: a block of four waves
// shares 16 pairs (block_mlp).  Bound: the latency of the panels and weights, a chain of C L / 16
// batches that a single wave walks with one batch in flight: 2,000 pairs at width 128 in BF16 took
// 45 us.
template <int HW, int PREC>
__global__ void __launch_bounds__(256) k_mlp_panels_block(NetParams np, const float2* __restrict__ enc, int64_t n,
                                                          float* __restrict__ heads, float* __restrict__ acts) {
    __shared__ float s_h[2][16 * (HW + 4)];
    __shared__ float s_z[16 * kZStride];
    const int lane = lane_id(), q = lane >> 4, j = lane & 15;
    const int L = np.enc.L, C = 2 * (1 + 2 * np.enc.F), U = (C + 3) >> 2, NLB = L >> 2;
    const int64_t pn = panel_stride(n);
    for (int64_t tile = blockIdx.x; tile * 16 < n; tile += gridDim.x) {
        const int64_t i0 = tile * 16, row = min(i0 + j, n - 1);
        block_mlp<HW, PREC, FeatRaw>(np, U * NLB, s_h, s_z, acts, n, i0 + j, [&](int t) {
            const int u = t / NLB, lb = t - u * NLB, c = q * U + u;
            const bool live = c < C;
            const float2* p = enc + ((int64_t)(4 * lb) * C + (live ? c : 0)) * pn + row;
            FeatRaw r;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                r.f[k] = p[(int64_t)k * C * pn];
                if (!live) r.f[k] = make_float2(0.f, 0.f);
            }
            return r;
        });
        for (int t = threadIdx.x; t < 16 * np.H; t += 256) {
            const int i = t / np.H, hh = t - i * np.H;
            if (i0 + i < n) heads[(i0 + i) * np.H + hh] = s_z[i * kZStride + hh];
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ host launchers

NetParams make_net_params(const nif_model* m, int32_t precision) {
    NetParams np;
    memset(&np, 0, sizeof(np));
    const nif_model_desc& d = m->desc;
    np.enc.tab = d.table_dtype == NIF_TABLE_F16 ? (const void*)m->tables_h : (const void*)m->tables;
    np.enc.f16 = d.table_dtype == NIF_TABLE_F16;
    np.enc.L = d.levels;
    np.enc.Fd = d.feat_dim;
    np.enc.log2T = d.log2_table;
    np.enc.F = d.concat_encoding ? 0 : d.pe_freqs;      // the grid sees x only in the concatenated form
    np.gamma_F = d.concat_encoding ? d.pe_freqs : -1;
    np.E_phi = 2 * m->S * d.levels * d.feat_dim;
    np.enc.dense_mask = 0;
    np.enc.set_stride = d.per_sample_tables ? ((int64_t)d.levels << d.log2_table) : 0;
    for (int l = 0; l < d.levels; ++l) {
        np.enc.res[l] = d.res[l];
        const uint64_t n1 = (uint64_t)d.res[l] + 1;
        if (n1 * n1 * n1 <= (1ull << d.log2_table)) np.enc.dense_mask |= 1u << l;
    }
    for (int i = 0; i < m->n_layers; ++i) {
        if (precision == NIF_PREC_FP32) np.W[i] = m->mlp_pad_f32 + m->wp_off[i];
        else if (precision == NIF_PREC_BF16) np.W[i] = m->mlp_pad_bf16 + m->wp_off[i];
        else np.W[i] = m->mlp_pad_f16 + m->wp_off[i];
        np.b[i] = m->mlp_pad_f32 + m->bp_off[i];
    }
    np.W0L = precision == NIF_PREC_FP32 ? (const void*)m->w0l_f32
           : precision == NIF_PREC_BF16 ? (const void*)m->w0l_bf16 : (const void*)m->w0l_f16;
    np.n_hidden = d.hidden_layers;
    np.E = m->E;
    np.H = m->H;
    np.dist_head = d.dist_head;
    return np;
}

// Panels of n point pairs or points from their positions.
// (n: the most there can be, with lv).
template <class Pos>
static void launch_lookups(const EncParams& ep, const Pos* pos, int64_t n, float* enc, hipStream_t st, const Live& lv = Live{}) {
    const int C = combinations<Pos>(1 + 2 * ep.F);
    // Small tables are looked up in LDS once the copies pay: 8 levels of 2^14 FP32 entries, 16,212
    // pairs 58 -> 30 us, 60,000 203 -> 60; 500 pairs 9 -> 19 us, hence the least of 2^17 lookups a
    // level.  Only where every level fits: the three coarsest of a 16-level 2^19 grid cost as much
    // from LDS as they save.
    const LdsPlan S = lds_plan(ep, C * n, device_cus());
    if (S.n == ep.L && C * n >= (1 << 17)) {
        if (ep.f16) hipLaunchKernelGGL((k_encode_lds<true, Pos>), dim3(S.total), dim3(1024), S.bytes, st, ep, S, pos, n, (float2*)enc, lv);
        else hipLaunchKernelGGL((k_encode_lds<false, Pos>), dim3(S.total), dim3(1024), S.bytes, st, ep, S, pos, n, (float2*)enc, lv);
        return;
    }
    const EncPlan P = level_plan(ep, (n + 255) / 256, (C + kEncKC - 1) / kEncKC);
    const dim3 g(plan_blocks(P));
    if (ep.f16) hipLaunchKernelGGL((k_encode_levels<kEncKC, true, Pos>), g, dim3(256), 0, st, ep, P, pos, n, (float2*)enc, lv);
    else hipLaunchKernelGGL((k_encode_levels<kEncKC, false, Pos>), g, dim3(256), 0, st, ep, P, pos, n, (float2*)enc, lv);
}

// Positions and panels of n pairs (SoA with stride ld).
static void launch_panels(const NetParams& np, const float* x0, const float* x1, int64_t n, int64_t ld, uint32_t* pos,
                          float* enc, hipStream_t st, const Live& lv) {
    const unsigned pb = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_positions, dim3(pb, 4), dim3(256), 0, st, np.enc.F, x0, x1, n, ld, pos, lv);
    launch_lookups<uint32_t>(np.enc, pos, n, enc, st, lv);
}

// Points go through the forward's panels, by chunks of its size: one lane per point walked its S L
// lookups one after the other (60,001 points at 16 levels of 2^19 FP16 entries: 2.4 ms).
int encode_launch(const nif_model* m, const float* x, int64_t n, float* out, hipStream_t st) {
    if (n == 0) return NIF_OK;
    const EncParams ep = make_net_params(m, NIF_PREC_FP32).enc;
    if (!uses_panels(m)) {
        const int64_t blocks = std::min<int64_t>((n * ep.L + 255) / 256, (int64_t)device_cus() * 32);
        hipLaunchKernelGGL(k_encode, dim3((unsigned)blocks), dim3(256), 0, st, ep, x, n, out);
        return check_hip(hipGetLastError(), "k_encode launch");
    }
    const int G = m->S * ep.L;
    const int64_t most = forward_chunk(m);
    double* pos = reinterpret_cast<double*>(m->fwd_pos);        // S FP64 samples: the bytes of 2 S fixed-point ones
    for (int64_t c0 = 0; c0 < n; c0 += most) {
        const int64_t c = std::min<int64_t>(most, n - c0);
        hipLaunchKernelGGL(k_samples, dim3((unsigned)((c + 63) / 64)), dim3(64), 0, st, ep.F, x + c0, c, n, pos);
        launch_lookups<double>(ep, pos, c, m->fwd_enc, st);
        hipLaunchKernelGGL(k_panel_rows, dim3((unsigned)((c + 63) / 64), (unsigned)((G + 63) / 64)), dim3(256), 0, st, m->S, ep.L,
                           (const float2*)m->fwd_enc, c, out + c0 * G * 2);
    }
    return check_hip(hipGetLastError(), "encode launch");
}

template <int HW, int CB, int PREC>
static void launch_mlp(const NetParams& np, const float* enc, int64_t n, float* heads, float* acts, hipStream_t st, const Live& lv) {
    const int64_t tiles = (n + 16 * CB - 1) / (16 * CB);
    const unsigned blocks = (unsigned)std::min<int64_t>((tiles + 3) / 4, (int64_t)device_cus() * 8);
    hipLaunchKernelGGL((k_mlp_panels<HW, CB, PREC>), dim3(blocks), dim3(256), 0, st, np, (const float2*)enc, n, heads, acts, lv);
}

// 8,001 pairs FP32 / BF16 at width 128: 126 / 116 us with blocks, 171 / 128 with waves; 16,212
// pairs: 234 / 214 against 244 / 199 (forward, all kernels).
constexpr int64_t kBlockMlpPairsPerCU = 40;

// Few pairs of a small network whose first layer is one to four batches of lookups: the fused kernel,
// one launch in place of three.  Fused and in panels, 2^14-entry tables, FP32: 8 levels without PE at
// width 64 13.9 and 18.8 us for one pair, 17 and 24 for 16,384; at width 16 8.3 and 18.4, 9.9 and 19.7;
// four batches at width 16 10.8 and 20.6, 14.1 and 24.2.  Four batches at width 64 have no line
// (16 levels of 2^19 without PE: 18.0 and 19.6 us for one pair, 27.1 and 20.3 for 2,048), and width 128
// is faster in panels (8 levels: 32 and 20.6 us for 256 pairs).  At 40,000 pairs and width 16 two batches
// take 18 and 27 us, three 31 and 33, four 37 and 32.  Heads are the same bits.
static bool forward_fused(const NetParams& np, int hw, int64_t n) {
    const int batches = ((2 * (1 + 2 * np.enc.F) + 3) >> 2) * (np.enc.L >> 2);
    return hw <= 64 && batches <= 4 && batches * hw <= 128 && n <= (batches <= 3 ? 1 << 16 : 1 << 14);
}

// enc: panels of n pairs (panel_stride(n) E floats), or rows [n][E] (nullable) for the variants.
template <int HW, int PREC>
static void launch_forward(const NetParams& np, const float* x0, const float* x1, int64_t n, int64_t ld, float* heads,
                           float* acts, float* enc, uint32_t* pos, hipStream_t st, const Live& lv) {
    if (np.gamma_F < 0 && np.enc.Fd == 2) {
        if constexpr (HW <= 64) {
            if (!acts && !lv.count && forward_fused(np, HW, n)) {
                hipLaunchKernelGGL((k_forward<HW, PREC, false, 16, 2>), dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, np, x0, x1, n, ld,
                                   heads, nullptr, nullptr);
                return;
            }
        }
        launch_panels(np, x0, x1, n, ld, pos, enc, st, lv);
        // a block per 16 pairs while that is what it takes to fill the chip, 16 pairs per wave until two
        // waves per SIMD are busy (one in 16 bits), then as many as the registers hold.  51,000 pairs at
        // width 128 in BF16: 160 us with 16 pairs, 96 with 32; 2^18 pairs in FP32, in parts of 37,449:
        // 3.67 and 3.95 ms.
        constexpr int CB = HW >= 128 ? 2 : 4;
        constexpr int kWavesPerCU = PREC == P_FP32 ? 8 : 4;
        if (!lv.count && n <= (int64_t)device_cus() * kBlockMlpPairsPerCU) {
            const unsigned blocks = (unsigned)((n + 15) / 16);
            hipLaunchKernelGGL((k_mlp_panels_block<HW, PREC>), dim3(blocks), dim3(256), 0, st, np, (const float2*)enc, n, heads, acts);
        } else if (n < (int64_t)device_cus() * kWavesPerCU * 16 * CB) launch_mlp<HW, 1, PREC>(np, enc, n, heads, acts, st, lv);
        else launch_mlp<HW, CB, PREC>(np, enc, n, heads, acts, st, lv);
        return;
    }
    // small launches (up to 2^17 pairs) take 16 pairs per wave so that they still fill the chip
    const bool gamma = np.gamma_F >= 0, small = n <= (1 << 17);
    const int64_t tiles = small || !gamma ? (n + 15) / 16 : (n + 63) / 64;
    const int64_t blocks = std::min<int64_t>((tiles + 3) / 4, (int64_t)device_cus() * 8);
    const dim3 g((unsigned)std::max<int64_t>(blocks, 1)), b(256);
    if (!gamma)                      // three-feature entries: 16 pairs per wave throughout
        hipLaunchKernelGGL((k_forward<HW, PREC, false, 16, 3>), g, b, 0, st, np, x0, x1, n, ld, heads, acts, enc);
    else if (small) hipLaunchKernelGGL((k_forward<HW, PREC, true, 16, 2>), g, b, 0, st, np, x0, x1, n, ld, heads, acts, enc);
    else hipLaunchKernelGGL((k_forward<HW, PREC, true, 64, 2>), g, b, 0, st, np, x0, x1, n, ld, heads, acts, enc);
}

template <int PREC>
static int dispatch_forward(int hw, const NetParams& np, const float* x0, const float* x1, int64_t n, int64_t ld,
                            float* heads, float* acts, float* enc, uint32_t* pos, hipStream_t st, const Live& lv) {
    switch (hw) {
        case 16: launch_forward<16, PREC>(np, x0, x1, n, ld, heads, acts, enc, pos, st, lv); break;
        case 32: launch_forward<32, PREC>(np, x0, x1, n, ld, heads, acts, enc, pos, st, lv); break;
        case 64: launch_forward<64, PREC>(np, x0, x1, n, ld, heads, acts, enc, pos, st, lv); break;
        case 128: launch_forward<128, PREC>(np, x0, x1, n, ld, heads, acts, enc, pos, st, lv); break;
        default: return fail(NIF_E_UNSUPPORTED, "hidden_width must be 16, 32, 64 or 128");
    }
    return NIF_OK;
}

bool uses_panels(const nif_model* m) { return m->desc.feat_dim == 2 && !m->desc.concat_encoding; }

static int forward_any(const nif_model* m, const float* x0, const float* x1, int64_t n, int64_t ld, float* heads,
                       int32_t precision, float* acts, float* enc, uint32_t* pos, hipStream_t st, const Live& lv) {
    if (n == 0) return NIF_OK;
    if (heads == nullptr || ld < n || (uses_panels(m) && (!enc || !pos)))
        return fail(NIF_E_INVALID_ARG, "forward needs a heads buffer, ld >= n and its encoding scratch");
    const NetParams np = make_net_params(m, precision);
    const int hw = m->desc.hidden_width;
    int rc;
    if (precision == NIF_PREC_FP32) rc = dispatch_forward<P_FP32>(hw, np, x0, x1, n, ld, heads, acts, enc, pos, st, lv);
    else if (precision == NIF_PREC_BF16) rc = dispatch_forward<P_BF16>(hw, np, x0, x1, n, ld, heads, acts, enc, pos, st, lv);
    else rc = dispatch_forward<P_FP16>(hw, np, x0, x1, n, ld, heads, acts, enc, pos, st, lv);
    if (rc) return rc;
    return check_hip(hipGetLastError(), "forward launch");
}

int forward_rows_launch(const nif_model* m, const float* x0, const float* x1, int64_t n, int64_t ld, float* heads,
                        int32_t precision, float* acts, float* enc, uint32_t* pos, hipStream_t st) {
    return forward_any(m, x0, x1, n, ld, heads, precision, acts, enc, pos, st, Live{});
}

// Pairs of the panel scratch: 2^16, if that is at most 256 MB.  One part of a staged query takes as
// many (40,192, as nif_forward: its MLP and launches take 5 to 8% longer; 2^17: the same).
int64_t stage_chunk(const nif_model* m) {
    return std::max<int64_t>(4096, std::min<int64_t>(1 << 16, ((int64_t)1 << 28) / ((int64_t)m->E * 4) / 256 * 256));
}

int forward_live_launch(const nif_model* m, const float* x, int64_t ld, const int32_t* count, int32_t cap, float* heads,
                        int32_t precision, hipStream_t st) {
    const int32_t chunk = (int32_t)stage_chunk(m);
    for (int s = 0; s * chunk < cap; ++s) {
        const int rc = forward_any(m, x, x + 3 * ld, std::min(cap, chunk), ld, heads, precision, nullptr, m->fwd_enc, m->fwd_pos, st,
                                   Live{count, cap, chunk, s});
        if (rc) return rc;
    }
    return NIF_OK;
}

// Chunk of nif_forward: its panels stay within 128 MB, half of the Infinity Cache, so the MLP
// reads them from there; 40,192 pairs at E = 832, at most 2^16 (stage_chunk).
int64_t forward_chunk(const nif_model* m) {
    const int64_t per = (int64_t)m->E * 4;
    return std::max<int64_t>(4096, std::min<int64_t>(1 << 16, ((int64_t)1 << 27) / per / 256 * 256));
}

int forward_launch(const nif_model* m, const float* x0, const float* x1, int64_t B, float* heads, int32_t precision,
                   hipStream_t st) {
    if (!uses_panels(m)) return forward_rows_launch(m, x0, x1, B, B, heads, precision, nullptr, nullptr, nullptr, st);
    const int64_t most = forward_chunk(m), parts = (B + most - 1) / most;
    const int64_t chunk = parts > 0 ? ((B + parts - 1) / parts + 255) / 256 * 256 : 0;     // even chunks
    for (int64_t c0 = 0; c0 < B; c0 += chunk) {
        const int64_t n = std::min<int64_t>(chunk, B - c0);
        const int rc = forward_rows_launch(m, x0 + c0, x1 + c0, n, B, heads + c0 * m->H, precision, nullptr,
                                           m->fwd_enc, m->fwd_pos, st);
        if (rc) return rc;
    }
    return NIF_OK;
}

}  // namespace nif
