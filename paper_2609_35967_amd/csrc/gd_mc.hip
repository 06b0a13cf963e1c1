// gd_mc.hip -- Monte Carlo sampling of collision events against the frozen
// neighbourhood (Sect. 2.5.3).  The post-interval audit is in gd_rates.hip.
//
// A particle draws waiting times dt_w = -ln(U_w)/lambda*_i (Gillespie); an
// event happens iff dt_w fits in the rest of the interval.  Its partner is the first slot whose inclusive prefix of
// lambda*_ij exceeds U_p lambda*_i, its channel the first whose cumulative rate
// exceeds U_c lambda*_ij; the outcome (Sect. 2.5.2) updates only this particle,
// after which every lambda*_ij is recomputed from the new mass against the
// frozen neighbours.  lambda*_i of the start state comes from the rates pass
// (the same function of the same inputs), so particles without events never
// evaluate their pairs here.  Random numbers: Philox4x32-10 keyed by the seed,
// counters (id, interval, event, 0/1); every event uses both calls.
#include "gd_common.hpp"
#include "gd_internal.hpp"
#include "gd_physics.hpp"

#include <algorithm>

namespace gd {

struct McArgs {
    DevProblem P;
    const uint32_t* id;
    const int32_t* nbr;
    const int32_t* cnt;
    const double* dmax;
    const double* m;      // snapshot (frozen) masses
    const double* x;
    const double* y;
    const double* z;
    const double4* snap;  // packed (m, s, N, 1/m) of the frozen neighbourhood
    const double* m_all;  // dimensionless kernels: its masses, in the records' place
    const double* lam_i;
    const gd_interval* iv;
    double* m_out;
    int32_t* n_events;
    int32_t* log;
    int32_t log_cap;
    uint64_t seed;
    uint32_t interval;
    int32_t interval_on_device;  // take the index from iv->n_intervals
    void* ws;
    unsigned long long* ev_counter;
    // the particles with an event, from the screen: entry e < n in list[e],
    // those that expect kEarlyEvents or more in list[n - 1 - e] and those
    // that expect kLongEvents in long_list[e], counted by list_n, early_n and
    // long_n; next is the sampling's next chunk
    int32_t* list;
    int32_t* long_list;
    int32_t* list_n;
    int32_t* early_n;
    int32_t* long_n;
    int32_t* next;
    int32_t screen_rounds;  // particles per thread of the screen
    double long_events;     // expected events of a very long chain
    int64_t n_all;  // length of the snapshot: neighbour indices lie in [0, n_all)
    const int64_t* interval_at;  // when set: the interval index (a spatial group's number in planning order)
    const int32_t* active;       // when set and 0: the run has no interval now (its list is skipped)
};

__device__ inline uint32_t mc_interval(const McArgs& A)
{
    if (A.interval_at) return uint32_t(*A.interval_at);
    return A.interval_on_device ? uint32_t(A.iv->n_intervals) : A.interval;
}

constexpr int kEventCap = 1 << 24;  // safety stop per particle and interval (status-flagged)
constexpr int kSampleBlocks = 1024;  // blocks (4 wavefronts each) of the sampling pass: 4 per SIMD
// Expected events from which a particle is sampled first, and the most
// particles a wavefront takes at a time.  On the warm 1M disk (362K particles
// with events, 2.26M events, the longest chain 1.4K) an interval takes 3.66 ms
// with 64 and 32, 3.50 with 32 and 32, 3.34 with 32 and 8, 3.31 with 16 and 8,
// 3.39 with 8 and 16: later starts and larger chunks leave a longer tail.
constexpr double kEarlyEvents = 16.0;
// Expected events from which a particle has a wavefront to itself: a round of
// 64 local boxes takes 90.4 ms with 1024 and 91.1 with 256, and took 109 with
// none apart (95.7 with a lane, then a wavefront for every particle); the
// warm 1M disk, whose chains are shorter, 3.33 ms with either and 3.28 with
// none (the second loop costs the first a few spilled registers).
constexpr double kLongEvents = 1024.0;

// For a run alone the line lies lower: the longest chain is the end of the
// pass, and beside another particle its events wait for both (sampling of warm
// grains, k = 20, with 1024, 256 and 128: 49,153 of them 1317, 995 and 988 us,
// 160,001 1478, 1110 and 1097, 262,145 2226, 1601 and 1596; a million at k = 32
// 1.92 ms with each).  In a set that gives the launch's 4096 wavefronts only a
// few particles each, all that start first are taken so (5000 at k = 32: 457 us
// with 128, 449 with 16; 20,000 at k = 64: 1.69 and 1.63 ms; but 131,072 at
// k = 64: 1.55 and 1.74).  Above k = 128 that loop is not the shorter one
// (50,021 at k = 256: 4.97 ms with 16, 4.61 with 128).
constexpr double kLongAlone = 128.0;

static double long_events(int64_t n, int32_t k)
{
    const int64_t top = k <= 32 ? 8192 : (k <= 128 ? 32768 : 0);
    return n <= top ? kEarlyEvents : kLongAlone;
}

constexpr int kChunk = 8;

// Sampling runs in two passes.  The screen (one lane per particle, few
// registers) draws each particle's first waiting time against lambda*_i of
// the rates pass: a particle without an event in the interval keeps its mass
// and is done; the others go, compacted, to a list, those that expect many
// events to its far end.  The sampling pass then runs the whole interval of
// each listed particle in half a wavefront (k <= 32) or a whole one, the long
// ones first, and redraws the first event's numbers (the same counters, so
// the same numbers).  One atomic per workgroup and list end.
constexpr int kScreenRounds = 4;

// particles per thread of the screen: each block's add to the list's count
// waits about 12 ns for the ones before it, which is all of the pass at one
// particle a thread and a million particles
static int32_t screen_rounds(int64_t n) { return n > 131072 ? kScreenRounds : 1; }

struct McScreen {
    using Args = McArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B)
    {
        __shared__ int32_t s_w[3][4], s_base[3];
        const int64_t i0 = B.id * int64_t(256 * A.screen_rounds) + threadIdx.x;
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
        const uint64_t below = (uint64_t(1) << lane) - 1;
        const uint32_t interval = mc_interval(A);
        const double dt_exe = A.iv->dt_exe;
        uint64_t b[kScreenRounds][3];  // lanes listed: few, many, very many events
        int32_t cnt[3] = {0, 0, 0};
#pragma unroll
        for (int r = 0; r < kScreenRounds; ++r) {
            const int64_t i = i0 + r * 256;
            int cls = -1;
            if (r < A.screen_rounds && i < A.P.n) {
                const int c = A.cnt[i];
                const double m = A.m[i];
                const double li = A.lam_i[i];
                if (c > 1 && li > 0.0) {
                    double u[4];
                    event_uniforms(A.seed, A.id[i], interval, 0u, u);
                    const double x = li * dt_exe;  // expected events
                    if (!(-log(u[0]) / li > dt_exe)) cls = x >= A.long_events ? 2 : (x >= kEarlyEvents ? 1 : 0);
                }
                if (cls < 0) {
                    A.m_out[i] = m;
                    if (A.n_events) A.n_events[i] = 0;
                }
                if (A.log)
                    for (int f = 0; f < A.log_cap; ++f) A.log[i * A.log_cap + f] = -1;
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                b[r][q] = __ballot(cls == q);
                cnt[q] += int32_t(__popcll(b[r][q]));
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) s_w[q][wv] = cnt[q];
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            const int32_t* w = s_w[threadIdx.x];
            const int32_t tot = w[0] + w[1] + w[2] + w[3];
            int32_t* to = threadIdx.x == 0 ? A.list_n : (threadIdx.x == 1 ? A.early_n : A.long_n);
            s_base[threadIdx.x] = tot ? atomicAdd(to, tot) : 0;
        }
        __syncthreads();
        int32_t at[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            at[q] = s_base[q];
            for (int w = 0; w < wv; ++w) at[q] += s_w[q][w];
        }
#pragma unroll
        for (int r = 0; r < kScreenRounds; ++r) {
            const int32_t i = int32_t(i0 + r * 256);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                if ((b[r][q] >> lane) & 1u) {
                    const int32_t e = at[q] + int32_t(__popcll(b[r][q] & below));
                    if (q == 2) A.long_list[e] = i;
                    else A.list[q == 0 ? e : A.P.n - 1 - e] = i;
                }
                at[q] += int32_t(__popcll(b[r][q]));
            }
        }
    }
};

__global__ __launch_bounds__(256) void k_mc_screen(McArgs A)
{
    McScreen::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

// ---------------------------------------------------------------------------
// The interval of the listed particles.  A particle takes a group of W lanes
// (W = 32, two particles per wavefront, for k <= 32; else the wavefront).
// Lane s < c of the group holds neighbour slot s (and s + 64, ... beyond 64):
// the neighbour's terms that the frozen snapshot fixes for the whole interval
// are computed once, and per event the lane evaluates its pair for the
// particle's current mass and the outcome the event would have with that
// partner.  The prefix over the slots is a scan over the group; the selection
// (first slot whose prefix exceeds the target) is a ballot, and the chosen
// lane's outcome is read across.  The draws do not depend on the mass: lane L
// of the group draws the numbers of event e0 + L, W events at a time, and
// each event reads its own from that lane.  A group whose particle is done
// takes the next of the wavefront's chunk while the other goes on.  The
// pass is bound by the instructions of the pairs: on the warm 1M disk a lane
// per particle for its first events and then a whole wavefront for the rest
// took 2.72 ms an interval, half a wavefront for all of them 1.7 ms, and the
// interval went from 4.39 to 3.31 ms.  128 registers (4 wavefronts per SIMD,
// a few spilled) against 167: 3.70 against 3.83 ms at that step.

// the numbers of events e0 .. e0 + W - 1 (lane L: event e0 + L): -ln U_w, U_p, U_c, U_f
struct Draws {
    double lw, up, uc, uf;
};

__device__ inline void draw_events(const McArgs& A, uint32_t pid, uint32_t interval, uint32_t e0, int s, Draws& d)
{
    double u[4];
    event_uniforms(A.seed, pid, interval, e0 + uint32_t(s), u);
    d.lw = -log(u[0]);
    d.up = u[1];
    d.uc = u[2];
    d.uf = u[3];
}

// x of lane l0 in the first group, of lane W + l1 in the second (l0, l1
// uniform)
template <int G>
__device__ inline double group_read(double x, int l0, int l1, bool second)
{
    const double a = readlane_d(x, l0);
    if (G == 1) return a;
    const double b = readlane_d(x, 32 + l1);
    return second ? b : a;
}

// inclusive prefix sum over each group of 64 / G lanes
template <int G>
__device__ inline double group_scan(double x)
{
    x = x + dpp_take<0x111, 0xf>(x);  // row_shr:1
    x = x + dpp_take<0x112, 0xf>(x);  // row_shr:2
    x = x + dpp_take<0x114, 0xf>(x);  // row_shr:4
    x = x + dpp_take<0x118, 0xf>(x);  // row_shr:8
    x = x + dpp_take<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    if (G == 1) x = x + dpp_take<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
    return x;
}

// the particles of chunk [lo, hi) of the run described by A, entry e of it
// list[n - 1 - e] (`far`) or list[e]; returns their events
template <int KP2, bool F32>
__device__ inline int run_chunk(const McArgs& A, int32_t lo, int32_t hi, bool far, int lane)
{
    constexpr int R = KP2 > kWave ? KP2 / kWave : 1;
    constexpr int G = KP2 <= 32 ? 2 : 1;  // particles side by side
    constexpr int W = kWave / G;
    const bool phys = A.P.kernel == GD_KERNEL_PHYSICAL;
    const double dt_exe = A.iv->dt_exe;
    const uint32_t interval = mc_interval(A);
    const int k = A.P.k;
    const bool second = G == 2 && lane >= W;
    const int sl = lane & (W - 1);
    // uniform per group: live, events done, first event of the draws
    bool live[2] = {false, false};
    int e[2] = {0, 0}, e0[2] = {0, 0}, cg[2] = {0, 0};
    int total = 0;
    // the lanes' own: the group's particle
    int64_t i = 0;
    uint32_t pid = 0;
    int c = 0;
    double t = 0.0, m = 1.0;
    QCtx q{};
    QCtxF qf{};
    Nb nb[R];
    Draws d{};
#pragma unroll
    for (int r = 0; r < R; ++r) nb[r] = Nb{1.0, 0.0, 0.0, 1.0, 0.0, 1.0, 1.0, 1.0};
    for (;;) {
        bool start[2] = {false, false};
        int32_t ent[2] = {0, 0};
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (!live[g] && lo < hi) {
                ent[g] = lo++;
                start[g] = true;
                live[g] = true;
                e[g] = 0;
                e0[g] = 0;
            }
        }
        if (!live[0] && !live[1]) break;
        if (start[0] || start[1]) {
            if (second ? start[1] : start[0]) {
                const int32_t en = second ? ent[1] : ent[0];
                i = A.list[far ? A.P.n - 1 - en : en];
                c = A.cnt[i];
                pid = A.id[i];
                m = A.m[i];
                t = 0.0;
                query_ctx(A.P, A.x[i], A.y[i], A.z[i], A.dmax[i], q);
                if (F32) query_ctx_f32(A.P, q, qf);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int s = r * kWave + sl;
                    int j = s < c ? A.nbr[i * k + s] : 0;
                    if (s < c && (j < 0 || j >= A.n_all)) set_status(A.ws, GD_DEV_INTERNAL);
                    if (j < 0 || j >= A.n_all) j = 0;
                    const double4 sn = A.m_all ? make_double4(A.m_all[j], 0.0, 0.0, 0.0) : A.snap[j];
                    if (F32) {
                        nb[r].mj = sn.x;
                        nb[r].sj = phys ? sn.y : 0.0;
                        nb[r].Nj = phys ? sn.z : 0.0;
                    } else {
                        nb_terms<true>(A.P, q, sn.x, phys ? sn.y : 0.0, phys ? sn.z : 0.0, sn.w, nb[r]);
                    }
                }
                draw_events(A, pid, interval, 0u, sl, d);
            }
            cg[0] = __builtin_amdgcn_readlane(c, 0);
            if (G == 2) cg[1] = __builtin_amdgcn_readlane(c, W);
        }
        bool redraw[2] = {false, false};
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (live[g] && e[g] - e0[g] >= W) {
                e0[g] = e[g];
                redraw[g] = true;
            }
        }
        if (redraw[0] || redraw[1])
            if (second ? redraw[1] : redraw[0]) draw_events(A, pid, interval, uint32_t(second ? e0[1] : e0[0]), sl, d);
        const int L0 = e[0] - e0[0], L1 = (e[1] - e0[1]) & (W - 1);
        const double lw = group_read<G>(d.lw, L0 & (W - 1), L1, second), up = group_read<G>(d.up, L0 & (W - 1), L1, second),
                     uc = group_read<G>(d.uc, L0 & (W - 1), L1, second);
        // the pairs at the current mass, each with its outcome (a fragmentation
        // outcome does not depend on the partner and is made after the selection)
        double si = 0.0;
        Own w{};
        if (phys) si = grain_size(A.P, m);
        if (!F32) own_terms(A.P, q, m, si, false, w);
        const float Stf = F32 && phys ? qf.stfac * float(si) : 0.0f;
        double pre[R], mnew[R];
        int code[R];
        double carry = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int type;
            double r0, lam, Ng;
            if (F32) {
                PairF of;
                pair_eval_f32(A.P, qf, m, 1.0 / m, float(si), Stf, nb[r].mj, float(nb[r].sj), nb[r].Nj, of);
                type = of.type;
                r0 = of.r0;
                lam = double(of.r0) + double(of.r1);  // the channel choice's total
                Ng = of.Ng;
                pre[r] = double(of.lam_star);         // the prefix adds the float rate
            } else {
                Pair o;
                pair_core<true, true>(A.P, q, w, nb[r], o);
                type = o.type;
                r0 = o.r0;
                lam = o.lam_star;
                Ng = o.Ng;
                pre[r] = o.lam_star;
            }
            const int ch = (type == kErosion && !(r0 > uc * lam)) ? 1 : 0;
            const double mj = nb[r].mj;
            mnew[r] = type == kStick ? m + Ng * mj : (ch == 0 ? m - Ng * mj : mj);
            code[r] = (ch << 16) | (type << 24);
            const double x = group_scan<G>(r * kWave + sl < c ? pre[r] : 0.0);
            pre[r] = carry + x;
            carry = carry + group_read<G>(x, W - 1, W - 1, second);
        }
        const double li = carry;
        const double dtw = lw / li;
        const bool cap = (second ? e[1] : e[0]) >= kEventCap;
        const bool go = li > 0.0 && !cap && !(dtw > dt_exe - t);
        const double target = up * li;
        const uint64_t gob = __ballot(go);
        bool on[2];
        on[0] = live[0] && (gob & 1u);
        on[1] = G == 2 && live[1] && ((gob >> (kWave / 2)) & 1u);
        // the first slot below c - 1 whose prefix exceeds the target, else c - 1
        int sel[2] = {cg[0] - 1, cg[1] - 1};
#pragma unroll
        for (int r = R - 1; r >= 0; --r) {
            const uint64_t hit = __ballot(r * kWave + sl < c - 1 && pre[r] > target);
            if (G == 1) {
                if (hit) sel[0] = r * kWave + int(__ffsll((unsigned long long)hit)) - 1;
            } else {
                if (uint32_t(hit)) sel[0] = int(__ffs(uint32_t(hit))) - 1;
                if (uint32_t(hit >> 32)) sel[1] = int(__ffs(uint32_t(hit >> 32))) - 1;
            }
        }
        int cd = 0;
        double mn = 0.0;
        if (G == 2) {
            const int l0 = sel[0] & (W - 1), l1 = sel[1] & (W - 1);
            const int cd0 = __builtin_amdgcn_readlane(code[0], l0), cd1 = __builtin_amdgcn_readlane(code[0], W + l1);
            cd = second ? cd1 : cd0;
            mn = group_read<G>(mnew[0], l0, l1, second);
        } else {
            const int l0 = sel[0] & (kWave - 1), sr = sel[0] / kWave;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r == sr) {  // uniform: sel is the same in every lane
                    cd = __builtin_amdgcn_readlane(code[r], l0);
                    mn = readlane_d(mnew[r], l0);
                }
            }
        }
        if ((cd >> 24) == kFrag) {
            const double uf = group_read<G>(d.uf, L0 & (W - 1), L1, second);
            const double a = sqrt(A.P.s_min);
            const double wf = a + uf * (sqrt(si) - a);
            const double sz = wf * wf;
            mn = div_nr(kPi * A.P.rho_s * sz * sz * sz, 6.0);
        }
        const bool lon = second ? on[1] : on[0];
        const int le = second ? e[1] : e[0];
        if (A.log && lon && sl == 0) {
            if (le < A.log_cap) A.log[i * A.log_cap + le] = (second ? sel[1] : sel[0]) | cd;
            else set_status(A.ws, GD_DEV_LOG_OVERFLOW);
        }
        const bool end = (second ? live[1] : live[0]) && !lon;
        if (end && sl == 0) {
            if (li > 0.0 && cap) set_status(A.ws, GD_DEV_EVENT_CAP);
            A.m_out[i] = m;
            if (A.n_events) A.n_events[i] = le;
        }
        // (an unchanged mass recomputes the same rates: no branch around them)
        t = lon ? t + dtw : t;
        m = lon ? mn : m;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            e[g] += on[g] ? 1 : 0;
            total += on[g] ? 1 : 0;
            live[g] = on[g];
        }
    }
    return total;
}

// The interval of particle i in a whole wavefront, with nothing else in its
// loop: the latency of the longest chain's events sets how long the pass
// takes where one particle has tens of thousands.
template <int KP2, bool F32>
__device__ inline int run_one(const McArgs& A, int32_t i, int lane)
{
    constexpr int R = KP2 > kWave ? KP2 / kWave : 1;
    constexpr int W = KP2 < kWave ? KP2 : kWave;  // lanes holding slots
    const bool phys = A.P.kernel == GD_KERNEL_PHYSICAL;
    const double dt_exe = A.iv->dt_exe;
    const uint32_t interval = mc_interval(A);
    int e = 0;
    double t = 0.0, m = A.m[i];
    const int64_t k = A.P.k;
    const int c = A.cnt[i];
    const uint32_t pid = A.id[i];
    QCtx q{};
    QCtxF qf{};
    query_ctx(A.P, A.x[i], A.y[i], A.z[i], A.dmax[i], q);
    if (F32) query_ctx_f32(A.P, q, qf);
    Nb nb[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = r * kWave + lane;
        const bool mine = s < c && lane < W;
        int j = mine ? A.nbr[i * k + s] : 0;
        if (mine && (j < 0 || j >= A.n_all)) set_status(A.ws, GD_DEV_INTERNAL);
        if (j < 0 || j >= A.n_all) j = 0;
        const double4 sn = A.m_all ? make_double4(A.m_all[j], 0.0, 0.0, 0.0) : A.snap[j];
        if (F32) {
            nb[r].mj = sn.x;
            nb[r].sj = phys ? sn.y : 0.0;
            nb[r].Nj = phys ? sn.z : 0.0;
        } else {
            nb_terms<true>(A.P, q, sn.x, phys ? sn.y : 0.0, phys ? sn.z : 0.0, sn.w, nb[r]);
        }
    }
    uint32_t e0 = 0;
    Draws d;
    draw_events(A, pid, interval, e0, lane, d);
    for (;;) {
        if (uint32_t(e) - e0 >= uint32_t(kWave)) {
            e0 = uint32_t(e);
            draw_events(A, pid, interval, e0, lane, d);
        }
        const int L = int(uint32_t(e) - e0);
        const double lw = readlane_d(d.lw, L), up = readlane_d(d.up, L), uc = readlane_d(d.uc, L);
        // the pairs at the current mass, each with its outcome (a fragmentation
        // outcome does not depend on the partner and is made after the selection)
        double si = 0.0;
        Own w{};
        if (phys) si = grain_size(A.P, m);
        if (!F32) own_terms(A.P, q, m, si, false, w);
        const float Stf = F32 && phys ? qf.stfac * float(si) : 0.0f;
        double pre[R], mnew[R];
        int code[R];
        double carry = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int type;
            double r0, lam, Ng;
            if (F32) {
                PairF of;
                pair_eval_f32(A.P, qf, m, 1.0 / m, float(si), Stf, nb[r].mj, float(nb[r].sj), nb[r].Nj, of);
                type = of.type;
                r0 = of.r0;
                lam = double(of.r0) + double(of.r1);  // the channel choice's total
                Ng = of.Ng;
                pre[r] = double(of.lam_star);         // the prefix adds the float rate
            } else {
                Pair o;
                pair_core<true>(A.P, q, w, nb[r], o);
                type = o.type;
                r0 = o.r0;
                lam = o.lam_star;
                Ng = o.Ng;
                pre[r] = o.lam_star;
            }
            const int ch = (type == kErosion && !(r0 > uc * lam)) ? 1 : 0;
            const double mj = nb[r].mj;
            mnew[r] = type == kStick ? m + Ng * mj : (ch == 0 ? m - Ng * mj : mj);
            code[r] = (ch << 16) | (type << 24);
            const double x = group_scan<1>((r * kWave + lane < c && lane < W) ? pre[r] : 0.0);
            pre[r] = carry + x;
            carry = carry + readlane_d(x, kWave - 1);
        }
        const double li = carry;
        if (!(li > 0.0)) break;
        if (e >= kEventCap) {
            if (lane == 0) set_status(A.ws, GD_DEV_EVENT_CAP);
            break;
        }
        const double dtw = lw / li;
        if (dtw > dt_exe - t) break;
        t = t + dtw;
        const double target = up * li;
        // the first slot below c - 1 whose prefix exceeds the target, else c - 1
        int sel = c - 1;
#pragma unroll
        for (int r = R - 1; r >= 0; --r) {
            const uint64_t hit = __ballot(r * kWave + lane < c - 1 && pre[r] > target);
            if (hit) sel = r * kWave + int(__ffsll((unsigned long long)hit)) - 1;
        }
        const int sl = sel & (kWave - 1), sr = sel / kWave;
        int cd = 0;
        double mn = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r == sr) {  // uniform: sel is the same in every lane
                cd = __builtin_amdgcn_readlane(code[r], sl);
                mn = readlane_d(mnew[r], sl);
            }
        }
        if ((cd >> 24) == kFrag) {
            const double uf = readlane_d(d.uf, L);
            const double a = sqrt(A.P.s_min);
            const double wf = a + uf * (sqrt(si) - a);
            const double sz = wf * wf;
            mn = div_nr(kPi * A.P.rho_s * sz * sz * sz, 6.0);
        }
        if (A.log && lane == 0) {
            if (e < A.log_cap) A.log[i * A.log_cap + e] = sel | cd;
            else set_status(A.ws, GD_DEV_LOG_OVERFLOW);
        }
        ++e;
        // (an unchanged mass recomputes the same rates: no branch around them)
        m = mn;
    }
    if (lane == 0) {
        A.m_out[i] = m;
        if (A.n_events) A.n_events[i] = e;
    }
    return e;
}

// Chunks of a run's lists: first the long chains, one each; then the list's
// far end, a particle per group of lanes (they start at once, spread over the
// wavefronts; two particles one after the other made the sampling of 20,000
// warm grains at k = 256 3.32 ms, 2.93 so), then the rest, up to kChunk a
// chunk while that leaves every wavefront kPer.  A chunk costs an add to the
// counter, 10 ns after the one before it: of a column of 65,536, 43 thousand
// particles with a few events each took 184 us with kPer = 4, 143 with 2 and
// 97 with 1, but 50,021 warm grains, with longer chains, 1.40, 1.41 and 1.43
// ms; over many runs their balance is worth more (64 local boxes 94.5 ms with
// 4, 96.5 with 1).
struct Chunks {
    int32_t nl, n0, n1, c, k0, k;  // particles of each part, chunk size, chunks before the last part, all

    template <int KP2, int kPer>
    __device__ void set(const McArgs& A, int32_t waves)
    {
        constexpr int G = KP2 <= 32 ? 2 : 1;
        nl = *A.long_n;
        n0 = *A.early_n;
        n1 = *A.list_n;
        c = n1 / (kPer * waves);
        c = c < 2 ? 2 : (c > kChunk ? kChunk : c);
        k0 = nl + (n0 + G - 1) / G;
        k = k0 + (n1 + c - 1) / c;
    }
    template <int KP2, bool F32>
    __device__ int run(const McArgs& A, int32_t x, int lane) const
    {
        // the long ones set the pass's length: their wavefronts issue first
        // (3.66 against 3.70 ms per interval of the warm 1M disk)
        if (x < k0) __builtin_amdgcn_s_setprio(3);
        int ev;
        if (x < nl) {
            ev = run_one<KP2, F32>(A, __builtin_amdgcn_readfirstlane(A.long_list[x]), lane);
        } else {
            constexpr int G = KP2 <= 32 ? 2 : 1;
            const bool far = x < k0;
            const int32_t lo = far ? G * (x - nl) : (x - k0) * c, hi = far ? lo + G : lo + c, n = far ? n0 : n1;
            ev = run_chunk<KP2, F32>(A, lo, hi < n ? hi : n, far, lane);
        }
        if (x < k0) __builtin_amdgcn_s_setprio(0);
        return ev;
    }
};

template <int KP2, bool F32>
__global__ __launch_bounds__(256, KP2 <= 32 ? 4 : 1) void k_mc(McArgs A)
{
    const int lane = threadIdx.x & 63;
    const int32_t nw = int32_t(gridDim.x * (blockDim.x / kWave));
    Chunks C;
    C.set<KP2, 2>(A, nw);
    // wavefront w takes chunk w first, then chunks nw, nw + 1, ... from the
    // counter (which is left alone when there are no more than nw); one add of
    // the events per workgroup: adds to one address wait 12 ns each for the
    // ones before them
    __shared__ unsigned long long s_ev[4];
    unsigned long long ev = 0;
    int32_t x = __builtin_amdgcn_readfirstlane(int32_t(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave));
    while (x < C.k) {
        ev += (unsigned long long)C.run<KP2, F32>(A, x, lane);
        if (C.k <= nw) break;
        int32_t next = 0;
        if (lane == 0) next = atomicAdd(A.next, 1);
        x = nw + __builtin_amdgcn_readfirstlane(next);
    }
    if (lane == 0) s_ev[threadIdx.x / kWave] = ev;
    __syncthreads();
    if (threadIdx.x == 0) {
        ev = s_ev[0] + s_ev[1] + s_ev[2] + s_ev[3];
        if (ev) atomicAdd(A.ev_counter, ev);
    }
}

// ---------------------------------------------------------------------------
// Many runs: a table in device memory holds, per slot, the sampling arguments
// of one run (written by its deferred call), after a 256-byte header whose
// first word counts the chunks taken.  One launch runs the lists of every
// slot, all slots' long chains first.
constexpr size_t kTableHeader = 256;
constexpr int kMaxTableSlots = 4096;

__global__ void k_table_put(McArgs* dst, McArgs A)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *dst = A;
}

template <int KP2, bool F32>
__global__ __launch_bounds__(256) void k_mc_batch(char* table, int32_t nbox)
{
    // per slot, the chunks of the slots before it: of long chains and far
    // ends [0], which go first in every slot, and of the rest [1]
    __shared__ int32_t s_pre[2][kMaxTableSlots];
    __shared__ int32_t s_total[2];
    const McArgs* T = reinterpret_cast<const McArgs*>(table + kTableHeader);
    int32_t* counter = reinterpret_cast<int32_t*>(table);
    const int t = threadIdx.x, lane = t & 63;
    const int32_t nw = int32_t(gridDim.x * (blockDim.x / kWave));
    for (int b = t; b < nbox; b += blockDim.x) {
        const bool on = !T[b].active || *T[b].active;
        Chunks C;
        C.set<KP2, 4>(T[b], nw);
        s_pre[0][b] = on ? C.k0 : 0;
        s_pre[1][b] = on ? C.k - C.k0 : 0;
    }
    __syncthreads();
    if (t < 2 * kWave) {  // exclusive prefixes of the slots' counts, 64 at a time, a wavefront each
        int32_t* pre = s_pre[t / kWave];
        int32_t carry = 0;
        for (int c0 = 0; c0 < nbox; c0 += kWave) {
            const int32_t v = c0 + lane < nbox ? pre[c0 + lane] : 0;
            int32_t x = v;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int32_t y = __shfl_up(x, o, kWave);
                if (lane >= o) x += y;
            }
            if (c0 + lane < nbox) pre[c0 + lane] = carry + x - v;
            carry += __shfl(x, kWave - 1, kWave);
        }
        if (lane == 0) s_total[t / kWave] = carry;
    }
    __syncthreads();
    const int32_t total0 = s_total[0], total = total0 + s_total[1];
    int32_t g = __builtin_amdgcn_readfirstlane(int32_t(blockIdx.x * (blockDim.x / kWave) + t / kWave));
    while (g < total) {
        const bool first = g < total0;
        const int32_t* pre = s_pre[first ? 0 : 1];
        const int32_t gg = first ? g : g - total0;
        // the last slot whose prefix is <= gg (slots with no chunks share a prefix)
        int lo = 0, hi = nbox - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pre[mid] <= gg) lo = mid;
            else hi = mid - 1;
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        const McArgs& A = T[lo];
        if (A.P.k > KP2 || (A.P.rates_fp32 != 0) != F32) {
            if (lane == 0) set_status(A.ws, GD_DEV_INTERNAL);
        } else {
            Chunks C;
            C.set<KP2, 4>(A, nw);
            const int ev = C.run<KP2, F32>(A, __builtin_amdgcn_readfirstlane(gg - pre[lo] + (first ? 0 : C.k0)), lane);
            if (lane == 0 && ev) atomicAdd(A.ev_counter, (unsigned long long)ev);
        }
        int32_t next = 0;
        if (lane == 0) next = atomicAdd(counter, 1);
        g = nw + __builtin_amdgcn_readfirstlane(next);
    }
}

// ---------------------------------------------------------------------------
__global__ void k_interval_init(gd_interval* iv, double dt_coll)
{
    if (threadIdx.x != 0) return;
    iv->dt_coll = dt_coll;
    iv->dt_req = 0.0;
    iv->dt_exe = 0.0;
    iv->C = 1.0;
    iv->time = 0.0;
    iv->ticks = 0;
    iv->exe_ticks = 0;
    iv->n_intervals = 0;
    iv->n_events = 0;
    iv->audit_worst = 0.0;
    iv->n_groups = 0;
    iv->pad = 0;
}

void launch_interval_init(gd_interval* iv, double dt_coll, hipStream_t st)
{
    hipLaunchKernelGGL(k_interval_init, dim3(1), dim3(64), 0, st, iv, dt_coll);
}

// the snapshot that the rates pass (or a snapshot launch) left
static void set_snapshot(McArgs& A, const gd_problem* p, const double4* snap)
{
    A.snap = snap;
    A.m_all = p->kernel == GD_KERNEL_PHYSICAL ? nullptr : reinterpret_cast<const double*>(snap);
}

static void set_counts(McArgs& A, McCounts* c)
{
    A.list_n = &c->n;
    A.early_n = &c->early_n;
    A.long_n = &c->long_n;
    A.next = &c->next;
}

static McArgs mc_args(const gd_problem* p, const gd_particles* s, const gd_neighbors* nb, gd_interval* iv,
                      const double* lam_i, uint64_t seed, uint32_t interval, bool interval_on_device,
                      int32_t* n_events, int32_t* log, int32_t log_cap, void* ws, const Layout& L)
{
    WsHeader* h = at<WsHeader>(ws, L.hdr);
    McArgs A{};
    A.P = to_dev(p);
    A.id = s->id;
    A.nbr = nb->nbr;
    A.cnt = nb->cnt;
    A.dmax = nb->dmax;
    A.m = s->m[s->cur];
    A.x = s->x;
    A.y = s->y;
    A.z = s->z;
    set_snapshot(A, p, at<double4>(ws, L.snap));
    A.lam_i = lam_i;
    A.iv = iv;
    A.m_out = s->m[s->cur ^ 1];
    A.n_events = n_events;
    A.log = log_cap > 0 ? log : nullptr;
    A.log_cap = log_cap;
    A.seed = seed;
    A.interval = interval;
    A.interval_on_device = interval_on_device ? 1 : 0;
    A.ws = ws;
    A.ev_counter = reinterpret_cast<unsigned long long*>(&h->scratch[0]);
    A.list = at<int32_t>(ws, L.mclist);
    A.long_list = at<int32_t>(ws, L.mclong);
    set_counts(A, &h->mc);
    A.screen_rounds = screen_rounds(p->n);
    A.long_events = kLongEvents;
    A.n_all = p->n;
    return A;
}

static void launch_screen(const McArgs& A, hipStream_t st)
{
    hipLaunchKernelGGL(k_mc_screen, dim3(unsigned(cdiv(A.P.n, 256 * A.screen_rounds))), dim3(256), 0, st, A);
}

template <bool F32>
static void launch_listed(const McArgs& A, int k, hipStream_t st)
{
    const dim3 g(kSampleBlocks), b(256);
    if (k <= 32) hipLaunchKernelGGL((k_mc<32, F32>), g, b, 0, st, A);
    else if (k <= 64) hipLaunchKernelGGL((k_mc<64, F32>), g, b, 0, st, A);
    else if (k <= 128) hipLaunchKernelGGL((k_mc<128, F32>), g, b, 0, st, A);
    else hipLaunchKernelGGL((k_mc<256, F32>), g, b, 0, st, A);
}

static void launch_listed(const McArgs& A, const gd_problem* p, hipStream_t st)
{
    if (p->rates_fp32) launch_listed<true>(A, p->k, st);
    else launch_listed<false>(A, p->k, st);
}

int launch_sample(const gd_problem* p, const gd_particles* s, const gd_neighbors* nb, gd_interval* iv,
                  const double* lam_i, uint64_t seed, uint32_t interval, bool interval_on_device, int32_t* n_events, int32_t* log,
                  int32_t log_cap, void* ws, const Layout& L, hipStream_t st, void* table, int32_t slot)
{
    McArgs A = mc_args(p, s, nb, iv, lam_i, seed, interval, interval_on_device, n_events, log, log_cap, ws, L);
    prof_mark(GD_PROF_MC, 0, st);
    if (table) {
        McCounts* c = &at<WsHeader>(ws, L.hdr)->mc_table;
        set_counts(A, c);
        launch_fill_i32(&c->n, sizeof(McCounts) / 4, 0, st);
    } else {
        A.long_events = long_events(p->n, p->k);
    }
    if (p->n > 0) launch_screen(A, st);
    if (table) {
        // the list is left to the launch over the whole table
        McArgs* dst = reinterpret_cast<McArgs*>(static_cast<char*>(table) + kTableHeader) + slot;
        hipLaunchKernelGGL(k_table_put, dim3(1), dim3(64), 0, st, dst, A);
        prof_mark(GD_PROF_MC, 1, st);
        return 0;
    }
    launch_listed(A, p, st);
    prof_mark(GD_PROF_MC, 1, st);
    launch_audit(p, s->m[s->cur], s->M, s->m[s->cur ^ 1], p->n, iv, ws, L, st);
    return 0;
}

// Sampling and audit of the slots [lo, hi) only (one spatial group); the
// group's interval state supplies dt_exe and takes the audit.
int launch_sample_group(const gd_problem* p, const gd_particles* s, const gd_neighbors* nb, gd_interval* iv,
                        const double* lam_i, uint64_t seed, uint32_t interval, int64_t lo, int64_t hi,
                        int32_t* n_events, void* ws, const Layout& L, hipStream_t st)
{
    McArgs A = mc_args(p, s, nb, iv, lam_i, seed, interval, false, n_events, nullptr, 0, ws, L);
    const int64_t cnt = hi - lo;
    A.P.n = cnt;
    A.id = s->id + lo;
    A.nbr = nb->nbr + lo * int64_t(p->k);
    A.cnt = nb->cnt + lo;
    A.dmax = nb->dmax + lo;
    A.m = s->m[s->cur] + lo;
    A.x = s->x + lo;
    A.y = s->y + lo;
    A.z = s->z + lo;
    A.lam_i = lam_i + lo;
    A.m_out = s->m[s->cur ^ 1] + lo;
    A.n_events = n_events ? n_events + lo : nullptr;
    prof_mark(GD_PROF_MC, 0, st);
    A.screen_rounds = screen_rounds(cnt);
    A.long_events = long_events(cnt, p->k);
    if (cnt > 0) launch_screen(A, st);
    launch_listed(A, p, st);
    prof_mark(GD_PROF_MC, 1, st);
    launch_audit(p, s->m[s->cur] + lo, s->M + lo, s->m[s->cur ^ 1] + lo, cnt, iv, ws, L, st);
    return 0;
}

size_t sample_table_bytes(int32_t nslot)
{
    return kTableHeader + sizeof(McArgs) * size_t(nslot);
}

int max_table_slots() { return kMaxTableSlots; }

int launch_sample_table(void* table, int32_t nslot, int32_t k, int32_t rates_fp32, hipStream_t st, int32_t nblocks)
{
    launch_fill_i32(static_cast<int32_t*>(table), 1, 0, st);
    char* tb = static_cast<char*>(table);
    const dim3 g(nblocks > 0 ? nblocks : kSampleBlocks), b(256);
    if (rates_fp32) {
        if (k <= 32) hipLaunchKernelGGL((k_mc_batch<32, true>), g, b, 0, st, tb, nslot);
        else if (k <= 64) hipLaunchKernelGGL((k_mc_batch<64, true>), g, b, 0, st, tb, nslot);
        else if (k <= 128) hipLaunchKernelGGL((k_mc_batch<128, true>), g, b, 0, st, tb, nslot);
        else hipLaunchKernelGGL((k_mc_batch<256, true>), g, b, 0, st, tb, nslot);
    } else {
        if (k <= 32) hipLaunchKernelGGL((k_mc_batch<32, false>), g, b, 0, st, tb, nslot);
        else if (k <= 64) hipLaunchKernelGGL((k_mc_batch<64, false>), g, b, 0, st, tb, nslot);
        else if (k <= 128) hipLaunchKernelGGL((k_mc_batch<128, false>), g, b, 0, st, tb, nslot);
        else hipLaunchKernelGGL((k_mc_batch<256, false>), g, b, 0, st, tb, nslot);
    }
    return 0;
}

// Sampling and audit of every run as stages of one interval: the screen, the
// listed particles of every run (one launch through a table of the runs'
// arguments, shaped for the largest k), then the audit.  Draws take the
// interval index from each run's interval state.
static void many_table_step(char* base, const ManyStep& s, hipStream_t st)
{
    launch_sample_table(base + s.tab, int32_t(s.a0), int32_t(s.a1 >> 1), int32_t(s.a1 & 1), st, int32_t(s.nblocks));
}

void many_sample(ManyBuilder& B, const std::vector<ManyRun>& R)
{
    const size_t nr = R.size();
    std::vector<McArgs> ma(nr);
    std::vector<int64_t> nb(nr);
    int kmax = 1, f32 = 0;
    for (size_t r = 0; r < nr; ++r) {
        const ManyRun& x = R[r];
        ma[r] = mc_args(&x.p, &x.out, &x.nb, x.iv, x.lam_i, x.seed, 0u, true, x.n_events, nullptr, 0, x.ws, x.L);
        if (x.snap) set_snapshot(ma[r], &x.p, x.snap);
        if (x.n_all >= 0) ma[r].n_all = x.n_all;
        ma[r].interval_at = x.interval_at;
        ma[r].active = B.active ? B.active + r : nullptr;
        nb[r] = cdiv(x.p.n, 256 * ma[r].screen_rounds);
        kmax = std::max(kmax, int(x.p.k));
        f32 = x.p.rates_fp32 ? 1 : 0;
    }
    B.add<McScreen>(ma, nb);
    // the listed particles of every run: a table (256-byte header, then
    // the runs' arguments) in the arena
    std::vector<char> table(kTableHeader + sizeof(McArgs) * nr, 0);
    memcpy(table.data() + kTableHeader, ma.data(), sizeof(McArgs) * nr);
    const size_t tab = B.put_vec(table);
    ManyStep st{&many_table_step, tab, 0, 0, B.tune.heavy_blocks, int64_t(nr), int64_t(kmax) * 2 + f32};
    B.steps.push_back(st);
    many_audit(B, R);
}

}  // namespace gd
