// CPU emulation of the lanes that share a ray: the library's own traversal (nif_trace.hpp), compiled
// for the host, on a bin grid built here.  Compares the segments of all_segments<SUB> and of repeated
// next_segment<SUB> calls with repeated next_segment<1> calls, ray by ray.  And of the lanes of a wave
// that takes rays from a counter which other waves move meanwhile (nif_deal.hpp).
#include <ucontext.h>

#include <memory>
#include <vector>

#include "nif_deal.hpp"
#include "nif_trace.hpp"

namespace lanes {

constexpr int kMax = 64;
constexpr size_t kStack = 64 * 1024;

struct Lane {
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    int site = -1, from = 0;
    uint64_t value = 0, result = 0;
    bool done = false;
};

static Lane g_lane[kMax];
static ucontext_t g_main;
static int g_cur = 0;
static void (*g_body)(void*) = nullptr;
static void* g_arg = nullptr;

int current() { return g_cur; }

uint64_t exchange(int site, uint64_t v, int from) {
    Lane& l = g_lane[g_cur];
    l.site = site;
    l.value = v;
    l.from = from;
    swapcontext(&l.ctx, &g_main);
    return l.result;
}

static uint64_t g_others = 0, g_taken = 0;

uint64_t counter_read(const unsigned long long* c) {
    const uint64_t v = *c;
    *const_cast<unsigned long long*>(c) += g_others;
    return v;
}
uint64_t counter_add(unsigned long long* c, unsigned long long n) {
    const uint64_t v = *c;
    *c += n + g_others;
    g_taken += n;
    return v;
}

static void enter() {
    g_body(g_arg);
    g_lane[g_cur].done = true;
}

// Runs body in n lanes.  False if they did not keep together.
static bool run(int n, void (*body)(void*), void* arg) {
    g_body = body;
    g_arg = arg;
    for (int i = 0; i < n; ++i) {
        Lane& l = g_lane[i];
        if (!l.stack) l.stack.reset(new char[kStack]);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.get();
        l.ctx.uc_stack.ss_size = kStack;
        l.ctx.uc_link = &g_main;
        l.done = false;
        makecontext(&l.ctx, enter, 0);
    }
    for (;;) {
        for (int i = 0; i < n; ++i) {
            g_cur = i;
            swapcontext(&g_main, &g_lane[i].ctx);
        }
        g_cur = 0;
        for (int i = 1; i < n; ++i)
            if (g_lane[i].done != g_lane[0].done || (!g_lane[0].done && g_lane[i].site != g_lane[0].site)) return false;
        if (g_lane[0].done) return true;
        uint64_t mask = 0;
        for (int i = 0; i < n; ++i) mask |= (g_lane[i].value & 1) << i;
        for (int i = 0; i < n; ++i) g_lane[i].result = g_lane[i].from < 0 ? mask : g_lane[g_lane[i].from].value;
    }
}

struct Seg {
    int32_t cell;
    float a, b;
    bool operator==(const Seg& o) const { return cell == o.cell && a == o.a && b == o.b; }
};

struct Scene {
    int N;
    nif::PoseDev P;
    std::vector<float4> V;
    std::vector<int32_t> start, cells;
};

// One pose, bins per axis as asked for (0: N / 2) by the extent of the occupied voxels.
static Scene build(int N, const uint8_t* occ, int kind, float s, int bins) {
    Scene S;
    S.N = N;
    nif::PoseDev& P = S.P;
    std::memset(&P, 0, sizeof(P));
    P.kind = kind;
    P.s = s;
    nif::pose_constants(kind, s, &P.k0, &P.k1, &P.k2);
    const int n1 = N + 1;
    S.V.resize((size_t)n1 * n1 * n1);
    for (int k = 0; k < n1; ++k)
        for (int j = 0; j < n1; ++j)
            for (int i = 0; i < n1; ++i) {
                const float inv = 1.f / (float)N;
                const float3 q = nif::deform(P, make_float3(i * inv, j * inv, k * inv));
                S.V[i + (size_t)n1 * (j + (size_t)n1 * k)] = {q.x, q.y, q.z, 0.f};
            }
    struct Box { int32_t cell; float lo[3], hi[3]; };
    std::vector<Box> boxes;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int c = 0; c < N * N * N; ++c) {
        if (!occ[c]) continue;
        Box b;
        b.cell = nif::pack_cell(c, N);
        const int i = c % N, j = c / N % N, k = c / (N * N);
        for (int a = 0; a < 3; ++a) { b.lo[a] = INFINITY; b.hi[a] = -INFINITY; }
        for (int m = 0; m < 8; ++m) {
            const float4 v = S.V[(i + (m & 1)) + (size_t)n1 * ((j + ((m >> 1) & 1)) + (size_t)n1 * (k + (m >> 2)))];
            const float x[3] = {v.x, v.y, v.z};
            for (int a = 0; a < 3; ++a) { b.lo[a] = std::fmin(b.lo[a], x[a]); b.hi[a] = std::fmax(b.hi[a], x[a]); }
        }
        for (int a = 0; a < 3; ++a) {
            b.lo[a] -= nif::kBinPad;
            b.hi[a] += nif::kBinPad;
            lo[a] = std::fmin(lo[a], b.lo[a]);
            hi[a] = std::fmax(hi[a], b.hi[a]);
        }
        boxes.push_back(b);
    }
    P.empty = boxes.empty();
    const int per = bins > 0 ? bins : std::max(N / 2, 1);
    const float ext = std::fmax(hi[0] - lo[0], std::fmax(hi[1] - lo[1], hi[2] - lo[2]));
    for (int a = 0; a < 3 && !P.empty; ++a) {
        P.nb[a] = std::max(1, (int)std::ceil(per * (hi[a] - lo[a]) / ext - 1e-3f));
        P.lo[a] = lo[a];
        P.bs[a] = std::fmax((hi[a] - lo[a]) / P.nb[a], 1e-6f);
        P.inv_bs[a] = 1.f / P.bs[a];
    }
    std::vector<std::vector<int32_t>> lists((size_t)P.nb[0] * P.nb[1] * P.nb[2]);
    for (const Box& b : boxes) {                         // ascending voxels: every list is sorted
        int b0[3], b1[3];
        for (int a = 0; a < 3; ++a) {
            b0[a] = std::min(std::max((int)std::floor((b.lo[a] - P.lo[a]) * P.inv_bs[a]), 0), P.nb[a] - 1);
            b1[a] = std::min(std::max((int)std::floor((b.hi[a] - P.lo[a]) * P.inv_bs[a]), 0), P.nb[a] - 1);
        }
        for (int z = b0[2]; z <= b1[2]; ++z)
            for (int y = b0[1]; y <= b1[1]; ++y)
                for (int x = b0[0]; x <= b1[0]; ++x) lists[x + P.nb[0] * (y + (size_t)P.nb[1] * z)].push_back(b.cell);
    }
    S.start.push_back(0);
    for (const auto& l : lists) {
        S.cells.insert(S.cells.end(), l.begin(), l.end());
        S.start.push_back((int32_t)S.cells.size());
    }
    return S;
}

// Bins of the ray's walk in which some lane finds more segments than it has slots for.
static int spills(const Scene& S, const nif::Ray& R, int sub) {
    nif::Trav T;
    nif::trav_init(S.P, R, T);
    if (!T.active) return 0;
    int bins = 0;
    for (;;) {
        nif::BinWalk B;
        nif::open_bin(S.P, S.start.data(), T, B);
        int found[kMax] = {};
        for (int32_t e = B.s0; e < B.s1; ++e) {
            const nif::CellHit h = nif::cell_intervals(S.V.data(), S.N, S.cells[e], R);
            for (int q = 0; q < h.n; ++q) {
                const float a = std::fmax(q == 0 ? h.a0 : h.a1, 0.f), b = q == 0 ? h.b0 : h.b1;
                if (b > a && a >= T.t_lo && a < B.t_hi) ++found[(e - B.s0) % sub];
            }
        }
        bins += *std::max_element(found, found + sub) > nif::kTraceSlots;
        if (B.last) return bins;
        nif::leave_bin(B, T);
    }
}

struct Job {
    const Scene* S;
    nif::Ray R;
    std::vector<Seg> out[kMax];
};

template <int SUB> static void all_body(void* p) {
    Job& j = *static_cast<Job*>(p);
    std::vector<Seg>& out = j.out[current()];
    nif::Trav T;
    nif::trav_init(j.S->P, j.R, T);
    nif::all_segments<SUB>(j.S->P, j.S->V.data(), j.S->start.data(), j.S->cells.data(), j.S->N, j.R, T,
                           [&](int32_t cell, float a, float b) { out.push_back({cell, a, b}); });
}

template <int SUB> static void next_body(void* p) {
    Job& j = *static_cast<Job*>(p);
    std::vector<Seg>& out = j.out[current()];
    nif::Trav T;
    nif::trav_init(j.S->P, j.R, T);
    nif::Segment s;
    int bad = 0;
    while (nif::next_segment<SUB>(j.S->P, j.S->V.data(), j.S->start.data(), j.S->cells.data(), j.S->N, j.R, T, s, &bad))
        out.push_back({s.cell, s.a, s.b});
}

}  // namespace lanes

// Rays o, d (SoA [3][n]) through one pose of an N^3 grid.  result: {rays with a spill, rays whose lanes
// came apart in all_segments, rays with other segments in some lane, the same two for next_segment,
// segments}; spilled (nullable, u8[n]): the rays with a spill.
extern "C" int lanes_check(int N, const uint8_t* occ, int kind, float s, int bins, int sub, int64_t n, const float* o,
                           const float* d, int64_t* result, uint8_t* spilled) {
    using namespace lanes;
    if (sub != 2 && sub != 4 && sub != 8 && sub != 16) return 1;
    const Scene S = build(N, occ, kind, s, bins);
    std::fill(result, result + 6, (int64_t)0);
    for (int64_t r = 0; r < n; ++r) {
        Job j;
        j.S = &S;
        j.R.o = make_float3(o[r], o[n + r], o[2 * n + r]);
        j.R.d = make_float3(d[r], d[n + r], d[2 * n + r]);
        const bool sp = spills(S, j.R, sub) > 0;
        if (spilled) spilled[r] = sp;
        result[0] += sp;
        g_cur = 0;
        next_body<1>(&j);
        const std::vector<Seg> ref = j.out[0];
        result[5] += (int64_t)ref.size();
        for (int form = 0; form < 2; ++form) {
            for (int i = 0; i < sub; ++i) j.out[i].clear();
            void (*body)(void*) = sub == 2 ? (form ? next_body<2> : all_body<2>)
                                : sub == 4 ? (form ? next_body<4> : all_body<4>)
                                : sub == 8 ? (form ? next_body<8> : all_body<8>) : (form ? next_body<16> : all_body<16>);
            const bool together = run(sub, body, &j);
            bool same = true;
            for (int i = 0; i < sub; ++i) same = same && j.out[i] == ref;
            result[1 + 2 * form] += !together;
            result[2 + 2 * form] += !same;
        }
    }
    return 0;
}

namespace lanes {
struct Take {
    int64_t counter, size;
    int n, leader;
    bool look;
    int64_t base[kMax];
};
static void take_body(void* p) {
    Take& t = *static_cast<Take*>(p);
    t.base[current()] = nif::take_tickets(&t.counter, t.size, t.n, t.leader, t.look);
}
}  // namespace lanes

// A wave of 64 lanes takes n tickets of a counter at `at` of a range of `size` rays, while other waves
// take `others` between any two accesses.  Returns the tickets' first one, -1 if the lanes came apart
// or differ, -2 if the counter moved by other than n for this wave (or 0 where nothing was left).
extern "C" int64_t lanes_take(int64_t at, int64_t size, int n, int leader, int look, int64_t others) {
    using namespace lanes;
    Take t{at, size, n, leader, look != 0, {}};
    g_others = (uint64_t)others;
    g_taken = 0;
    if (!run(64, take_body, &t)) return -1;
    for (int i = 1; i < 64; ++i)
        if (t.base[i] != t.base[0]) return -1;
    if (g_taken != (uint64_t)n && !(g_taken == 0 && t.base[0] >= size)) return -2;
    return t.base[0];
}
