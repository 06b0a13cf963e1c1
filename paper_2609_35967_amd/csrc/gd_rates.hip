// gd_rates.hip -- rates over the frozen neighbourhood and the interval plan
// (Sect. 2.5.1-2.5.3).
//
//  k_snapshot    snapshot of every particle, the frozen properties neighbours
//                read: mass, diameter s_j, grain count N_j = M_j/m_j, 1/m_j (the
//                dimensionless kernels': the mass, copied by the rates pass)
//  k_rates       one lane per particle: lambda*_ij over its slots in slot order,
//                lambda*_i, controller moments a_i = sum rate <J>, b_i = sum rate <J^2>
//  k_reduce      per-block sums over ilogb(m) bins in double-double, grouped per
//                wavefront with ballots (deterministic order); the block that
//                ends last folds the blocks' sums and runs the plan (merged
//                bins, A_b, B_b, dt_req, dyadic dt_exe into the interval
//                state) or, after sampling, the audit
#include "gd_common.hpp"
#include "gd_internal.hpp"
#include "gd_physics.hpp"

#include <algorithm>

namespace gd {

// The snapshot of every particle.  Physical kernel: a packed record (m_j, s_j,
// N_j = M_j / m_j, 1 / m_j), one 32-byte gather per neighbour.  The
// dimensionless kernels read nothing of a neighbour but its mass, so there the
// snapshot is the masses alone, 8 bytes each, in the records' place.
struct SnapArgs {
    DevProblem P;
    const double* m;
    const double* M;
    int64_t n;
    double4* snap;
};

struct Snapshot {
    using Args = SnapArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B)
    {
        const int64_t i = B.id * int64_t(blockDim.x) + threadIdx.x;
        if (i >= A.n) return;
        const double mi = A.m[i];
        if (A.P.kernel == GD_KERNEL_PHYSICAL)
            A.snap[i] = make_double4(mi, grain_size(A.P, mi), A.M[i] / mi, 1.0 / mi);
        else
            reinterpret_cast<double*>(A.snap)[i] = mi;
    }
};

__global__ __launch_bounds__(256) void k_snapshot(SnapArgs A)
{
    Snapshot::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

struct RatesArgs {
    DevProblem P;
    const int32_t* nbr;
    const int32_t* cnt;
    const double* dmax;
    const double* m;
    const double* x;
    const double* y;
    const double* z;
    const double4* snap;
    const double4* snap_own;  // the particle's own record: snap offset to the first own slot
    double* lam;
    double* lam_pair;
    double* a;
    double* b;
    void* ws;
    int64_t n_all;  // length of the snapshot: neighbour indices lie in [0, n_all)
    // dimensionless kernels: the frozen masses, and (when set) the snapshot
    // that the pass makes of them for the calls that follow
    const double* m_all;
    double* m_copy;
};

__device__ inline double4 neighbour_record(const double4* snap, const double* m_all, int j)
{
    return m_all ? make_double4(m_all[j], 0.0, 0.0, 0.0) : snap[j];
}

constexpr int kGather = 4;  // neighbours whose slot and record loads a lane has in flight together

// A particle's pairs are shared by LANES = 1, 2 or 4 neighbouring lanes: lane
// `sub` takes the slots sub, sub + LANES, ...  The kGather slots of the lane
// from s0 on (those below cmax) and the snapshot records of the valid ones;
// invalid slots are left for the caller to flag.
template <int LANES>
__device__ inline void gather_neighbours(const int32_t* row, int s0, int sub, int cmax, int64_t n, const double4* snap,
                                         const double* m_all, int (&jj)[kGather], double4 (&rec)[kGather])
{
#pragma unroll
    for (int t = 0; t < kGather; ++t) {
        const int s = s0 + t * LANES + sub;
        jj[t] = s < cmax ? row[s] : -1;
    }
#pragma unroll
    for (int t = 0; t < kGather; ++t) 
        rec[t] = (jj[t] >= 0 && jj[t] < n) ? neighbour_record(snap, m_all, jj[t]) : make_double4(0.0, 0.0, 0.0, 0.0);
}

// lane l of every group of LANES lanes read by the whole group (DPP quad
// permutation, no LDS)
template <int LANES, int l>
__device__ inline double group_lane(double x)
{
    constexpr int c = LANES == 4 ? l * 0x55 : (LANES == 2 ? (l | (l << 2) | ((l + 2) << 4) | ((l + 2) << 6)) : 0xE4);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), c, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), c, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// sum + the group's values in lane order, that is in slot order: the same
// additions as one lane's over the slots (a lane without a slot adds +0)
template <int LANES>
__device__ inline double add_in_order(double sum, double v)
{
    if (LANES == 1) return sum + v;
    sum = sum + group_lane<LANES, 0>(v);
    sum = sum + group_lane<LANES, 1>(v);
    if (LANES == 4) {
        sum = sum + group_lane<LANES, LANES == 4 ? 2 : 0>(v);
        sum = sum + group_lane<LANES, LANES == 4 ? 3 : 0>(v);
    }
    return sum;
}

template <int LANES>
struct Rates {
    using Args = RatesArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B);
};

template <int LANES>
__global__ __launch_bounds__(256) void k_rates(RatesArgs A)
{
    Rates<LANES>::body(A, Blk{xcd_block(), int64_t(gridDim.x)});
}

template <int LANES>
__device__ __forceinline__ void Rates<LANES>::body(const Args& A, Blk B)
{
    const int64_t i = (B.id * int64_t(blockDim.x) + threadIdx.x) / LANES;
    const int sub = int(threadIdx.x) % LANES;
    if (i >= A.P.n) return;
    const int k = A.P.k;
    const bool phys = A.P.kernel == GD_KERNEL_PHYSICAL;
    const int c = A.cnt[i];
    double lam = 0.0, sa = 0.0, sb = 0.0;
    if (c > 1) {
        QCtx q;
        query_ctx(A.P, A.x[i], A.y[i], A.z[i], A.dmax[i], q);
        const double mi = A.m[i];
        Own w;
        own_terms(A.P, q, mi, phys ? A.snap_own[i].y : 0.0, true, w);
        if (!(mi > 0.0) || !isfinite(mi)) set_status(A.ws, GD_DEV_NONFINITE);
        const int cmax = c < k ? c : k;
        // neighbours kGather at a time: their slots, then their records, in
        // flight together; the pairs are then taken in slot order
        for (int s0 = 0; s0 < cmax; s0 += kGather * LANES) {
            int jj[kGather];
            double4 rec[kGather];
            gather_neighbours<LANES>(A.nbr + i * k, s0, sub, cmax, A.n_all, A.snap, A.m_all, jj, rec);
#pragma unroll
            for (int t = 0; t < kGather; ++t) {
                if (s0 + t * LANES >= cmax) break;  // the same in the particle's lanes
                const int s = s0 + t * LANES + sub;
                const int j = jj[t];
                double pl = 0.0, pa = 0.0, pb = 0.0;
                if (LANES == 1 || s < cmax) {
                    if (j < 0 || j >= A.n_all) {
                        set_status(A.ws, GD_DEV_INTERNAL);
                        if (LANES == 1) continue;
                    } else {
                        const double4 sn = rec[t];
                        Pair o;
                        pair_eval<true>(A.P, q, w, sn.x, phys ? sn.y : 0.0, phys ? sn.z : 0.0, sn.w, o);
                        pl = o.lam_star;
                        if (A.lam_pair) A.lam_pair[i * k + s] = pl;
                        pair_moments(o, w, sn.x, pa, pb);
                    }
                }
                lam = add_in_order<LANES>(lam, pl);
                sa = add_in_order<LANES>(sa, pa);
                sb = add_in_order<LANES>(sb, pb);
            }
        }
    }
    if (sub != 0) return;
    if (A.m_copy) A.m_copy[i] = A.m[i];
    if (A.lam_pair)
        for (int s = (c > 1 ? c : 0); s < k; ++s) A.lam_pair[i * k + s] = 0.0;
    A.lam[i] = lam;
    A.a[i] = sa;
    A.b[i] = sb;
}

// The same pass with the single-precision pair form (gd_problem.rates_fp32):
// float pair terms, summed in FP64 in slot order.
template <int LANES>
struct RatesF32 {
    using Args = RatesArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B);
};

template <int LANES>
__global__ __launch_bounds__(256) void k_rates_f32(RatesArgs A)
{
    RatesF32<LANES>::body(A, Blk{xcd_block(), int64_t(gridDim.x)});
}

template <int LANES>
__device__ __forceinline__ void RatesF32<LANES>::body(const Args& A, Blk B)
{
    const int64_t i = (B.id * int64_t(blockDim.x) + threadIdx.x) / LANES;
    const int sub = int(threadIdx.x) % LANES;
    if (i >= A.P.n) return;
    const int k = A.P.k;
    const bool phys = A.P.kernel == GD_KERNEL_PHYSICAL;
    const int c = A.cnt[i];
    double lam = 0.0, sa = 0.0, sb = 0.0;
    if (c > 1) {
        QCtx q;
        query_ctx(A.P, A.x[i], A.y[i], A.z[i], A.dmax[i], q);
        QCtxF qf;
        query_ctx_f32(A.P, q, qf);
        const double mi = A.m[i];
        const float si = phys ? float(A.snap_own[i].y) : 0.0f;
        const float Sti = phys ? qf.stfac * si : 0.0f;
        const double rmi = 1.0 / mi;
        float mJf = 0.0f, mJ2f = 0.0f;
        if (phys) {
            double mJ, mJ2;
            frag_moments(A.snap_own[i].y, A.P.s_min, mJ, mJ2);
            mJf = float(mJ);
            mJ2f = float(mJ2);
        }
        if (!(mi > 0.0) || !isfinite(mi)) set_status(A.ws, GD_DEV_NONFINITE);
        const int cmax = c < k ? c : k;
        for (int s0 = 0; s0 < cmax; s0 += kGather * LANES) {
            int jj[kGather];
            double4 rec[kGather];
            gather_neighbours<LANES>(A.nbr + i * k, s0, sub, cmax, A.n_all, A.snap, A.m_all, jj, rec);
#pragma unroll
            for (int t = 0; t < kGather; ++t) {
                if (s0 + t * LANES >= cmax) break;
                const int s = s0 + t * LANES + sub;
                const int j = jj[t];
                double pl = 0.0;
                float pa = 0.0f, pb = 0.0f;
                if (LANES == 1 || s < cmax) {
                    if (j < 0 || j >= A.n_all) {
                        set_status(A.ws, GD_DEV_INTERNAL);
                        if (LANES == 1) continue;
                    } else {
                        const double4 sn = rec[t];
                        PairF o;
                        pair_eval_f32(A.P, qf, mi, rmi, si, Sti, sn.x, phys ? float(sn.y) : 0.0f, phys ? sn.z : 0.0, o);
                        pl = double(o.lam_star);
                        if (A.lam_pair) A.lam_pair[i * k + s] = pl;
                        pair_moments_f32(o, mJf, mJ2f, pa, pb);
                    }
                }
                lam = add_in_order<LANES>(lam, pl);
                sa = add_in_order<LANES>(sa, double(pa));
                sb = add_in_order<LANES>(sb, double(pb));
            }
        }
    }
    if (sub != 0) return;
    if (A.m_copy) A.m_copy[i] = A.m[i];
    if (A.lam_pair)
        for (int s = (c > 1 ? c : 0); s < k; ++s) A.lam_pair[i * k + s] = 0.0;
    A.lam[i] = lam;
    A.a[i] = sa;
    A.b[i] = sb;
}

// Lanes a particle's pairs are shared by: a set that leaves the SIMDs with a
// wavefront or two waits on one lane's chain of pairs.  n counts all particles
// of the launch.  Measured intervals with 1, 2 and 4 lanes: boxes without a
// search 59 / 50 / 44 us at 4096 particles, 65 / 56 / 52 at 32,768, 73 / 66 /
// 66 at 65,536, 98 / 99 / 96 at 131,072; disks 148 / 135 / 127 us at 10,007,
// 179 / 166 / 161 at 32,768, 235 / 226 / 228 at 65,536, 305 / 306 / 305 at
// 100,003, 550 / 553 / 565 at 262,144 (each lane repeats the particle's own
// terms).
constexpr int64_t kRates4 = 49152, kRates2 = 98304;

static int rates_lanes(int64_t n) { return n <= kRates4 ? 4 : (n <= kRates2 ? 2 : 1); }

static void launch_rates_pass(const RatesArgs& A, bool f32, hipStream_t st)
{
    const int lanes = rates_lanes(A.P.n);
    const dim3 g(unsigned(cdiv(A.P.n * lanes, 256))), b(256);
    if (f32) {
        if (lanes == 4) hipLaunchKernelGGL(k_rates_f32<4>, g, b, 0, st, A);
        else if (lanes == 2) hipLaunchKernelGGL(k_rates_f32<2>, g, b, 0, st, A);
        else hipLaunchKernelGGL(k_rates_f32<1>, g, b, 0, st, A);
    } else {
        if (lanes == 4) hipLaunchKernelGGL(k_rates<4>, g, b, 0, st, A);
        else if (lanes == 2) hipLaunchKernelGGL(k_rates<2>, g, b, 0, st, A);
        else hipLaunchKernelGGL(k_rates<1>, g, b, 0, st, A);
    }
}

// ---------------------------------------------------------------------------
// Bin sums of the controller.  Mode 0 (plan): count, M, M a, M b over
// bin(m_snap).  Mode 1 (audit): M |ln(m_new/m_snap)|/3 over bin(m_snap).
// part[(blk * kNBin + bin) * 8 + f]: f = 0 count, (1,2) (3,4) (5,6) dd values,
// written for the bins of the block's mask (mask[2 blk], mask[2 blk + 1]).
// One launch each: the fold over the blocks and the rule were launches of
// their own (4.7 and 10-24 us, the rule one thread's walk over the bins).
constexpr int kRedWaves = 8;  // wavefronts per block

struct ReduceArgs {
    const double* msnap;
    const double* M;
    const double* va;
    const double* vb;
    int64_t n;
    double* part;
    uint64_t* mask;
    gd_interval* iv;
    WsHeader* h;
    double eps, dt_fn_max;
    int32_t nbin_min;
};

// One step of a segmented inclusive double-double scan over the wavefront:
// a lane adds the value the DPP pattern brings it only when the source lane
// belongs to its own run (equal id; ids start at 1, so a lane with no
// source, which reads 0, adds nothing).  Runs must be contiguous in lane
// order; the steps are those of wave_scan_incl.
template <int CTRL, int ROWS>
__device__ inline void seg_step(dd& v, int id)
{
    const int oid = __builtin_amdgcn_update_dpp(0, id, CTRL, ROWS, 0xf, true);
    const dd s = dd_add(v, dd{dpp_take<CTRL, ROWS>(v.hi), dpp_take<CTRL, ROWS>(v.lo)});
    if (oid == id) v = s;
}

template <int NV>
__device__ inline void seg_scan(dd (&v)[NV], int id)
{
#pragma unroll
    for (int u = 0; u < NV; ++u) seg_step<0x111, 0xf>(v[u], id);
#pragma unroll
    for (int u = 0; u < NV; ++u) seg_step<0x112, 0xf>(v[u], id);
#pragma unroll
    for (int u = 0; u < NV; ++u) seg_step<0x114, 0xf>(v[u], id);
#pragma unroll
    for (int u = 0; u < NV; ++u) seg_step<0x118, 0xf>(v[u], id);
#pragma unroll
    for (int u = 0; u < NV; ++u) seg_step<0x142, 0xa>(v[u], id);
#pragma unroll
    for (int u = 0; u < NV; ++u) seg_step<0x143, 0xc>(v[u], id);
}

template <int MODE>
struct Reduce {
    using Args = ReduceArgs;
    static constexpr int kThreads = kRedWaves * kWave;
    static __device__ __forceinline__ void body(const Args& A, Blk B);
};

template <int MODE>
__global__ __launch_bounds__(kRedWaves * kWave) void k_reduce(ReduceArgs A)
{
    Reduce<MODE>::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

// the folded sums of a bin, and the bins that hold particles
using BinRow = double[7];

__device__ inline bool in_mask(uint64_t m0, uint64_t m1, int b) { return ((b < 64 ? m0 : m1) >> (b & 63)) & 1u; }

// Plan (Sect. 2.5.3): bins merged in ascending order until each group holds
// >= nbin_min particles (a short last group joins the previous one);
// A_b = sum M a/sum M, B_b = sum M b/sum M;
// dt_req = min(dt_remain, dt_fn_max, eps C/A_b, (eps C)^2/B_b);
// dt_exe = dt_coll 2^-n, the largest aligned dyadic fraction <= dt_req.
// One wavefront: the merge walks the bins that hold particles, their counts
// in registers; then each lane sums its groups' bins in ascending order.
__device__ inline void plan_rule(const ReduceArgs& A, const BinRow* row, uint64_t m0, uint64_t m1, int lane,
                                 int32_t (&s_first)[kNBin], int32_t (&s_last)[kNBin])
{
    gd_interval* iv = A.iv;
    WsHeader* h = A.h;
    const double dt_coll = iv->dt_coll;
    const double Cf = iv->C;
    const int64_t ticks = iv->ticks;
    const double c0 = row[lane][0], c1 = row[lane + 64][0];
    int ng = 0, last = -1;
    double acc = 0.0;
    bool open = false;
    int g0 = -1, g1 = -1;  // the groups of bins lane and lane + 64
    for (int half = 0; half < 2; ++half) {
        for (uint64_t m = half ? m1 : m0; m; m &= m - 1) {
            const int l = __ffsll((unsigned long long)m) - 1, bb = l + 64 * half;
            const double c = readlane_d(half ? c1 : c0, l);
            if (!open) {
                open = true;
                acc = 0.0;
                if (lane == 0) s_first[ng] = bb;
            }
            last = bb;
            acc = acc + c;
            if (half == 0 && lane == l) g0 = ng;
            if (half == 1 && lane == l) g1 = ng;
            if (acc >= double(A.nbin_min)) {
                if (lane == 0) s_last[ng] = bb;
                ++ng;
                open = false;
            }
        }
    }
    if (open) {  // a short tail joins the previous group, or is the only one
        if (ng > 0) {
            g0 = g0 == ng ? ng - 1 : g0;
            g1 = g1 == ng ? ng - 1 : g1;
        } else {
            ng = 1;
        }
        if (lane == 0) s_last[ng - 1] = last;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const double eC = A.eps * Cf;
    double req = INFINITY;
    for (int g = lane; g < kNBin; g += kWave) {
        double gM = 0.0;
        if (g < ng) {
            dd x[3] = {dd{0.0, 0.0}, dd{0.0, 0.0}, dd{0.0, 0.0}};
            for (int bb = s_first[g]; bb <= s_last[g]; ++bb) {
                if (!in_mask(m0, m1, bb)) continue;
#pragma unroll
                for (int v = 0; v < 3; ++v) x[v] = dd_add(x[v], dd{row[bb][1 + 2 * v], row[bb][2 + 2 * v]});
            }
            gM = x[0].hi;
            const double A_ = gM > 0.0 ? x[1].hi / gM : 0.0;
            const double B_ = gM > 0.0 ? x[2].hi / gM : 0.0;
            if (A_ > 0.0) {
                const double tt = eC / A_;
                if (tt < req) req = tt;
            }
            if (B_ > 0.0) {
                const double tt = (eC * eC) / B_;
                if (tt < req) req = tt;
            }
        }
        h->gM[g] = gM;
    }
    h->group_of[lane] = g0;
    h->group_of[lane + 64] = g1;
    req = wave_min_d(req);
    const double tick = ldexp(dt_coll, -30);
    const double rem = double(kTicks - ticks) * tick;
    // (rem first: a comparison with a NaN on either side keeps the other)
    double r = rem;
    if (A.dt_fn_max < r) r = A.dt_fn_max;
    if (req < r) r = req;
    // lane nh tests the fraction 2^-nh; the first that fits is the largest
    const int64_t mine = kTicks >> (lane <= 30 ? lane : 30);
    const uint64_t fits = __ballot(lane <= 30 && double(mine) * tick <= r && (ticks & (mine - 1)) == 0);
    if (lane != 0) return;
    if (!fits) atomicOr(&h->status, GD_DEV_TICK_FLOOR);
    const int64_t size = fits ? kTicks >> (__ffsll((unsigned long long)fits) - 1) : 1;
    h->n_groups = ng;
    iv->dt_req = r;
    iv->dt_exe = double(size) * tick;
    iv->exe_ticks = size;
    iv->n_groups = ng;
    h->scratch[0] = 0.0;  // event counter of the coming interval
}

// Audit (a reading: the paper names what the audit monitors, not its rule):
// per merged controller bin the mass-weighted mean realised |ln(s'/s)|; if the
// largest exceeds 2 eps C, C halves (floor 0.25), else C grows by 1.25 (cap 1).
// The groups are the plan's, ascending runs of bins.
__device__ inline void audit_rule(const ReduceArgs& A, const BinRow* row, uint64_t m0, uint64_t m1, int lane,
                                  int32_t (&s_first)[kNBin], int32_t (&s_last)[kNBin])
{
    gd_interval* iv = A.iv;
    WsHeader* h = A.h;
    const int32_t g0 = h->group_of[lane], g1 = h->group_of[lane + 64];
    for (int g = lane; g < kNBin; g += kWave) {
        s_first[g] = kNBin;
        s_last[g] = -1;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    if (g0 >= 0) {
        atomicMin(&s_first[g0], lane);
        atomicMax(&s_last[g0], lane);
    }
    if (g1 >= 0) {
        atomicMin(&s_first[g1], lane + 64);
        atomicMax(&s_last[g1], lane + 64);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    double worst = 0.0;
    for (int g = lane; g < kNBin; g += kWave) {
        const double gM = h->gM[g];
        dd x{0.0, 0.0};
        for (int bb = s_first[g]; bb <= s_last[g]; ++bb)
            if (in_mask(m0, m1, bb)) x = dd_add(x, dd{row[bb][1], row[bb][2]});
        if (s_last[g] >= 0 && gM > 0.0) {
            const double r = x.hi / gM;
            if (r > worst) worst = r;
        }
    }
    worst = wave_max_d(worst);
    if (lane != 0) return;
    const double Cf = iv->C;
    const double thr = 2.0 * A.eps * Cf;
    iv->C = (worst > thr) ? fmax(0.25, 0.5 * Cf) : fmin(1.0, 1.25 * Cf);
    iv->audit_worst = worst;
    int64_t tk = iv->ticks + iv->exe_ticks;
    if (tk >= kTicks) tk = 0;
    iv->ticks = tk;
    iv->time = iv->time + iv->dt_exe;
    iv->n_intervals = iv->n_intervals + 1;
    iv->n_events = int64_t(*reinterpret_cast<const unsigned long long*>(&h->scratch[0]));
}

template <int MODE>
__device__ __forceinline__ void Reduce<MODE>::body(const Args& A, Blk B)
{
    constexpr int mode = MODE;
    const double* __restrict__ msnap = A.msnap;
    const double* __restrict__ M = A.M;
    const double* __restrict__ va = A.va;
    const double* __restrict__ vb = A.vb;
    const int64_t n = A.n;
    double* part = A.part;
    WsHeader* h = A.h;
    __shared__ double acc[kRedWaves][kNBin][7];
    // a row of many bins in bin order: bin, run length and the three values
    // of each lane, per wavefront
    __shared__ int32_t sk[kRedWaves][kWave][2];
    __shared__ double sv[kRedWaves][kWave][3];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int e = t; e < kRedWaves * kNBin * 7; e += kRedWaves * kWave) (&acc[0][0][0])[e] = 0.0;
    __syncthreads();
    const int64_t chunk = (n + B.n - 1) / B.n;
    const int64_t beg = B.id * chunk;
    const int64_t end = beg + chunk < n ? beg + chunk : n;
    bool range_bad = false;
    // wavefront w takes the rows of 64 slots w, w + kRedWaves, ... of the
    // block's range; the next row's operands are loaded before the current
    // row is reduced
    struct Row {
        double Mi, ms, a, b;
    };
    auto load = [&](int64_t i, Row& r) {
        const bool in = i < end;
        r.Mi = in ? M[i] : 0.0;
        r.ms = in ? msnap[i] : 1.0;
        r.a = in ? va[i] : 0.0;
        r.b = (in && mode == 0) ? vb[i] : 0.0;
    };
    const int64_t step = int64_t(kRedWaves) * kWave;
    int64_t rb = beg + int64_t(w) * kWave;
    Row cur;
    load(rb + lane, cur);
    for (; rb < end; rb += step) {
        Row nxt;
        load(rb + step + lane, nxt);
        const int64_t i = rb + lane;
        bool valid = i < end && cur.Mi > 0.0;
        double v0 = 0.0, v1 = 0.0, v2 = 0.0;
        int bin = 0;
        if (valid) {
            const double ms = cur.ms;
            bin = bin_of(ms);
            const int lb = ilogb(ms);
            range_bad = range_bad || lb < -kBinOff || lb > kNBin - 1 - kBinOff;
            if (mode == 0) {
                v0 = cur.Mi;
                v1 = cur.Mi * cur.a;
                v2 = cur.Mi * cur.b;
            } else {
                v0 = cur.Mi * (fabs(log(cur.a / ms)) / 3.0);
            }
        }
        // the lanes of the row grouped by bin, from one ballot per bit of the
        // bin: the lanes of my bin, how many of them come before me, and how
        // many lanes hold smaller bins (no lane is lost: invalid lanes take
        // key 255, after every bin)
        const int key = valid ? bin : 255;
        uint64_t same = ~uint64_t(0);
        int less = 0;
#pragma unroll
        for (int bit = 7; bit >= 0; --bit) {
            const uint64_t ones = __ballot((key >> bit) & 1);
            const bool mb = (key >> bit) & 1;
            if (mb) less += int(__popcll(same & ~ones));
            same &= mb ? ones : ~ones;
        }
        const int rank = int(__popcll(same & ((uint64_t(1) << lane) - 1)));
        const int run = int(__popcll(same));
        const uint64_t heads = __ballot(valid && rank == 0);
        if (__popcll(heads) > 1) {
            // several bins: the row in bin order through LDS, then one
            // segmented scan; the last lane of each bin's run adds the run
            const int pos = less + rank;
            sk[w][pos][0] = key;
            sk[w][pos][1] = rank == run - 1 ? run : 0;
            sv[w][pos][0] = v0;
            sv[w][pos][1] = v1;
            sv[w][pos][2] = v2;
            const int kb = sk[w][lane][0], last = sk[w][lane][1];
            dd sd[3] = {dd{sv[w][lane][0], 0.0}, dd{sv[w][lane][1], 0.0}, dd{sv[w][lane][2], 0.0}};
            if (mode == 0) {
                seg_scan<3>(sd, kb + 1);
            } else {
                dd s1[1] = {sd[0]};
                seg_scan<1>(s1, kb + 1);
                sd[0] = s1[0];
            }
            if (last > 0 && kb != 255) {
                double* a = acc[w][kb];
                a[0] += double(last);
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    if (u > 0 && mode != 0) break;
                    const dd x = dd_add(dd{a[1 + 2 * u], a[2 + 2 * u]}, sd[u]);
                    a[1 + 2 * u] = x.hi;
                    a[2 + 2 * u] = x.lo;
                }
            }
        } else {
            uint64_t rem = __ballot(valid);
            while (rem) {
                const int leader = __ffsll((unsigned long long)rem) - 1;
                const int bsel = __builtin_amdgcn_readlane(bin, leader);
                const bool mine = valid && bin == bsel;
                const uint64_t match = __ballot(mine);
                dd s0{mine ? v0 : 0.0, 0.0}, s1{0.0, 0.0}, s2{0.0, 0.0};
                if (mode == 0) {
                    s1 = dd{mine ? v1 : 0.0, 0.0};
                    s2 = dd{mine ? v2 : 0.0, 0.0};
                    wave_sum_dd3(s0, s1, s2);
                } else {
                    s0 = wave_sum_dd(s0);
                }
                if (lane == 0) {
                    double* a = acc[w][bsel];
                    a[0] += double(__popcll(match));
                    dd x = dd_add(dd{a[1], a[2]}, s0);
                    a[1] = x.hi;
                    a[2] = x.lo;
                    x = dd_add(dd{a[3], a[4]}, s1);
                    a[3] = x.hi;
                    a[4] = x.lo;
                    x = dd_add(dd{a[5], a[6]}, s2);
                    a[5] = x.hi;
                    a[6] = x.lo;
                }
                rem &= ~match;
            }
        }
        cur = nxt;
    }
    if (__ballot(range_bad) && lane == 0) atomicOr(&h->status, GD_DEV_MASS_RANGE);
    __syncthreads();
    // the block's sums per bin, in acc[0][bin], and the bins that hold some
    __shared__ uint64_t s_m[2];
    __shared__ int32_t s_last_blk;
    BinRow* row = acc[0];
    if (t < kNBin) {
        double cnt = 0.0;
        dd x0{0.0, 0.0}, x1{0.0, 0.0}, x2{0.0, 0.0};
        for (int ww = 0; ww < kRedWaves; ++ww) {
            const double* a = acc[ww][t];
            cnt += a[0];
            x0 = dd_add(x0, dd{a[1], a[2]});
            if (mode == 0) {
                x1 = dd_add(x1, dd{a[3], a[4]});
                x2 = dd_add(x2, dd{a[5], a[6]});
            }
        }
        const double v[7] = {cnt, x0.hi, x0.lo, x1.hi, x1.lo, x2.hi, x2.lo};
        double* out = part + (B.id * kNBin + t) * 8;
#pragma unroll
        for (int f = 0; f < 7; ++f) {
            row[t][f] = v[f];
            if (B.n > 1 && cnt > 0.0) put_device(out + f, v[f]);
        }
        const uint64_t m = __ballot(cnt > 0.0);
        if (lane == 0) {
            s_m[w] = m;
            if (B.n > 1) put_device(A.mask + 2 * B.id + w, m);
        }
    }
    if (B.n > 1) {
        done_stores();
        __syncthreads();
        if (t == 0) s_last_blk = last_block(&h->red_done, B.n) ? 1 : 0;
        __syncthreads();
        if (!s_last_blk) return;
        // fold: wavefront w takes the bins w, w + kRedWaves, ... of the union
        // of the masks, its lanes the blocks
        constexpr int NR = kRedBlocks / kWave;
        uint64_t b0[NR], b1[NR], u0 = 0, u1 = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int blk = r * kWave + lane;
            b0[r] = blk < B.n ? A.mask[2 * blk] : 0;
            b1[r] = blk < B.n ? A.mask[2 * blk + 1] : 0;
            u0 |= b0[r];
            u1 |= b1[r];
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            u0 |= __shfl_xor((unsigned long long)u0, o, kWave);
            u1 |= __shfl_xor((unsigned long long)u1, o, kWave);
        }
        u0 = readlane_u64(u0, 0);
        u1 = readlane_u64(u1, 0);
        int turn = 0;
        uint64_t left0 = u0, left1 = u1;
        while (left0 | left1) {
            const int bin = left0 ? __ffsll((unsigned long long)left0) - 1 : 63 + __ffsll((unsigned long long)left1);
            if (left0) left0 &= left0 - 1;
            else left1 &= left1 - 1;
            const bool mine = turn == w;
            turn = (turn + 1) & (kRedWaves - 1);
            if (!mine) continue;
            double cnt = 0.0;
            dd x0{0.0, 0.0}, x1{0.0, 0.0}, x2{0.0, 0.0};
            double v[NR][8];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const bool have = in_mask(b0[r], b1[r], bin);
                const double2* a =
                    reinterpret_cast<const double2*>(part + (int64_t(have ? r * kWave + lane : 0) * kNBin + bin) * 8);
#pragma unroll
                for (int f = 0; f < (mode == 0 ? 4 : 2); ++f) {
                    const double2 p = a[f];
                    v[r][2 * f] = have ? p.x : 0.0;
                    v[r][2 * f + 1] = have ? p.y : 0.0;
                }
            }
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                cnt += v[r][0];
                x0 = dd_add(x0, dd{v[r][1], v[r][2]});
                if (mode == 0) {
                    x1 = dd_add(x1, dd{v[r][3], v[r][4]});
                    x2 = dd_add(x2, dd{v[r][5], v[r][6]});
                }
            }
            if (mode == 0) wave_sum_dd3(x0, x1, x2);
            else x0 = wave_sum_dd(x0);
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) cnt += shfl_xor_d(cnt, o);
            if (lane == 0) {
                const double o[7] = {cnt, x0.hi, x0.lo, x1.hi, x1.lo, x2.hi, x2.lo};
#pragma unroll
                for (int f = 0; f < 7; ++f) row[bin][f] = o[f];
            }
        }
        if (t == 0) {
            s_m[0] = u0;
            s_m[1] = u1;
        }
    }
    __syncthreads();
    if (w != 0) return;
    __shared__ int32_t s_first[kNBin], s_last[kNBin];
    if (mode == 0) plan_rule(A, row, s_m[0], s_m[1], lane, s_first, s_last);
    else audit_rule(A, row, s_m[0], s_m[1], lane, s_first, s_last);
    // the coming sampling's list of particles with events starts empty
    if (lane == 0) h->mc = McCounts{0, 0, 0, 0};
}

static ReduceArgs reduce_args(const gd_problem* p, const double* msnap, const double* M, const double* va,
                              const double* vb, int64_t n, gd_interval* iv, void* ws, const Layout& L)
{
    const DevProblem P = to_dev(p);
    ReduceArgs A{};
    A.msnap = msnap;
    A.M = M;
    A.va = va;
    A.vb = vb;
    A.n = n;
    A.part = at<double>(ws, L.part);
    A.mask = at<uint64_t>(ws, L.red);  // (free outside the neighbour build)
    A.iv = iv;
    A.h = at<WsHeader>(ws, L.hdr);
    A.eps = P.eps;
    A.dt_fn_max = P.dt_fn_max;
    A.nbin_min = P.nbin_min;
    return A;
}

// a row of 64 particles per wavefront and block up to kRedBlocks blocks
static int64_t reduce_blocks(int64_t n)
{
    return std::min<int64_t>(kRedBlocks, std::max<int64_t>(1, cdiv(n, kRedWaves * kWave)));
}

void launch_plan(const gd_problem* p, const double* msnap, const double* M, const double* a, const double* b,
                 int64_t n, gd_interval* iv, void* ws, const Layout& L, hipStream_t st)
{
    hipLaunchKernelGGL(k_reduce<0>, dim3(unsigned(reduce_blocks(n))), dim3(kRedWaves * kWave), 0, st,
                       reduce_args(p, msnap, M, a, b, n, iv, ws, L));
}

void launch_audit(const gd_problem* p, const double* msnap, const double* M, const double* mnew, int64_t n,
                  gd_interval* iv, void* ws, const Layout& L, hipStream_t st)
{
    prof_mark(GD_PROF_AUDIT, 0, st);
    hipLaunchKernelGGL(k_reduce<1>, dim3(unsigned(reduce_blocks(n))), dim3(kRedWaves * kWave), 0, st,
                       reduce_args(p, msnap, M, mnew, nullptr, n, iv, ws, L));
    prof_mark(GD_PROF_AUDIT, 1, st);
}

int launch_rates(const gd_problem* p, const gd_particles* s, const gd_neighbors* nb, gd_interval* iv, double* lam_i,
                 double* lam_pair, double* ab, void* ws, const Layout& L, hipStream_t st)
{
    const DevProblem P = to_dev(p);
    const int64_t n = p->n;
    const int g = int((n + 255) / 256);
    const double* m = s->m[s->cur];
    double4* snap = at<double4>(ws, L.snap);
    prof_mark(GD_PROF_RATES, 0, st);
    // (the dimensionless kernels read the masses themselves and copy them as
    // they go: 4096 particles take 40.3 us an interval with a snapshot launch
    // before the rates, 37.8 without)
    const bool records = p->kernel == GD_KERNEL_PHYSICAL;
    if (records) hipLaunchKernelGGL(k_snapshot, dim3(g), dim3(256), 0, st, SnapArgs{P, m, s->M, n, snap});
    RatesArgs A{};
    A.m_all = records ? nullptr : m;
    A.m_copy = records ? nullptr : reinterpret_cast<double*>(snap);
    A.P = P;
    A.nbr = nb->nbr;
    A.cnt = nb->cnt;
    A.dmax = nb->dmax;
    A.m = m;
    A.x = s->x;
    A.y = s->y;
    A.z = s->z;
    A.snap = snap;
    A.lam = lam_i;
    A.lam_pair = lam_pair;
    A.a = ab ? ab : at<double>(ws, L.a);
    A.b = ab ? ab + n : at<double>(ws, L.b);
    A.ws = ws;
    A.n_all = n;
    A.snap_own = snap;
    launch_rates_pass(A, p->rates_fp32 != 0, st);
    launch_plan(p, m, s->M, A.a, A.b, n, iv, ws, L, st);
    prof_mark(GD_PROF_RATES, 1, st);
    return 0;
}

// Rates and plan of the slots [lo, hi) only (one spatial group): the particle's
// own arrays are addressed from lo, the snapshot (refreshed first when asked)
// covers every particle.  The executed interval is then held within 1/16 and
// 16 times the scheduled intervals sched[h] (0: none) of the groups h set in
// the group's interaction row (the lower limit wins a conflict), halved until
// aligned, and recorded in sched[g].
__global__ void k_group_clamp(gd_interval* iv, int g, int G, const unsigned long long* rows, int64_t* sched)
{
    if (threadIdx.x != 0) return;
    const unsigned long long row = rows[g];
    int64_t z_lo = 1, z_hi = kTicks;
    for (int h = 0; h < G; ++h) {
        const int64_t zh = sched[h];
        if (h == g || zh == 0 || !((row >> h) & 1ull)) continue;
        if (zh / 16 > z_lo) z_lo = zh / 16;
        if (16 * zh < z_hi) z_hi = 16 * zh;
    }
    if (z_hi < z_lo) z_hi = z_lo;
    const int64_t ticks = iv->ticks;
    int64_t z = iv->exe_ticks;
    if (z > z_hi) z = z_hi;
    if (z < z_lo) z = z_lo;
    while (z > 1 && ((ticks % z) != 0 || ticks + z > kTicks)) z >>= 1;
    iv->exe_ticks = z;
    iv->dt_exe = double(z) * ldexp(iv->dt_coll, -30);
    sched[g] = z;
}

int launch_rates_group(const gd_problem* p, const gd_particles* s, const gd_neighbors* nb, gd_interval* iv,
                       double* lam_i, int64_t lo, int64_t hi, int32_t group, int32_t n_groups, const uint64_t* rows,
                       int64_t* sched, bool snapshot, void* ws, const Layout& L, hipStream_t st)
{
    DevProblem P = to_dev(p);
    const int64_t n = p->n, cnt = hi - lo;
    const double* m = s->m[s->cur];
    double4* snap = at<double4>(ws, L.snap);
    prof_mark(GD_PROF_RATES, 0, st);
    if (snapshot)
        hipLaunchKernelGGL(k_snapshot, dim3(int((n + 255) / 256)), dim3(256), 0, st, SnapArgs{P, m, s->M, n, snap});
    P.n = cnt;
    RatesArgs A{};
    A.P = P;
    A.nbr = nb->nbr + lo * int64_t(p->k);
    A.cnt = nb->cnt + lo;
    A.dmax = nb->dmax + lo;
    A.m = m + lo;
    A.x = s->x + lo;
    A.y = s->y + lo;
    A.z = s->z + lo;
    A.snap = snap;
    A.snap_own = snap + lo;
    A.m_all = p->kernel == GD_KERNEL_PHYSICAL ? nullptr : reinterpret_cast<const double*>(snap);
    A.lam = lam_i + lo;
    A.lam_pair = nullptr;
    A.a = at<double>(ws, L.a) + lo;
    A.b = at<double>(ws, L.b) + lo;
    A.ws = ws;
    A.n_all = n;
    if (cnt > 0) launch_rates_pass(A, p->rates_fp32 != 0, st);
    launch_plan(p, m + lo, s->M + lo, A.a, A.b, cnt, iv, ws, L, st);
    hipLaunchKernelGGL(k_group_clamp, dim3(1), dim3(64), 0, st, iv, int(group), int(n_groups),
                       reinterpret_cast<const unsigned long long*>(rows), sched);
    prof_mark(GD_PROF_RATES, 1, st);
    return 0;
}

// Rates and plan of every run as stages of one interval: snapshot, rates,
// the bin sums over n / red_div blocks per run (at most kRedBlocks) with the
// plan.
void many_rates(ManyBuilder& B, const std::vector<ManyRun>& R, bool own_snapshot)
{
    const size_t nr = R.size();
    std::vector<SnapArgs> sn(nr);
    std::vector<RatesArgs> ra(nr);
    std::vector<ReduceArgs> pl(nr);
    std::vector<int64_t> nb(nr), nred(nr), f64(nr), f32(nr);
    int64_t total = 0;
    for (size_t r = 0; r < nr; ++r) total += R[r].p.n;
    const int lanes = rates_lanes(total);
    for (size_t r = 0; r < nr; ++r) {
        const ManyRun& x = R[r];
        const gd_problem* p = &x.p;
        const gd_particles* s = &x.out;
        const DevProblem P = to_dev(p);
        const int64_t n = p->n;
        const double* m = s->m[s->cur];
        double4* snap = x.snap ? x.snap : at<double4>(x.ws, x.L.snap);
        sn[r] = SnapArgs{P, m, s->M, n, snap};
        RatesArgs& A = ra[r];
        A = RatesArgs{};
        A.P = P;
        A.nbr = x.nb.nbr;
        A.cnt = x.nb.cnt;
        A.dmax = x.nb.dmax;
        A.m = m;
        A.x = s->x;
        A.y = s->y;
        A.z = s->z;
        A.snap = snap;
        A.snap_own = x.snap ? snap + x.lo : snap;
        A.lam = x.lam_i;
        A.lam_pair = nullptr;
        A.a = at<double>(x.ws, x.L.a);
        A.b = at<double>(x.ws, x.L.b);
        A.ws = x.ws;
        A.n_all = x.n_all >= 0 ? x.n_all : n;
        const bool records = p->kernel == GD_KERNEL_PHYSICAL;
        double* masses = reinterpret_cast<double*>(snap);
        A.m_all = records ? nullptr : (x.snap ? masses : m);
        A.m_copy = records || x.snap ? nullptr : masses;
        nb[r] = records ? cdiv(n, 256) : 0;
        f64[r] = p->rates_fp32 ? 0 : cdiv(n * lanes, 256);
        f32[r] = p->rates_fp32 ? cdiv(n * lanes, 256) : 0;
        nred[r] = std::min<int64_t>(kRedBlocks, std::max<int64_t>(1, cdiv(n, B.tune.red_div)));
        pl[r] = reduce_args(p, m, s->M, A.a, A.b, n, x.iv, x.ws, x.L);
    }
    if (own_snapshot) B.add<Snapshot>(sn, nb);
    if (lanes == 4) {
        B.add<Rates<4>>(ra, f64);
        B.add<RatesF32<4>>(ra, f32);
    } else if (lanes == 2) {
        B.add<Rates<2>>(ra, f64);
        B.add<RatesF32<2>>(ra, f32);
    } else {
        B.add<Rates<1>>(ra, f64);
        B.add<RatesF32<1>>(ra, f32);
    }
    B.add<Reduce<0>>(pl, nred);
}

// the snapshot of a whole particle set as one step (one run; predicated by
// the builder's flags when set)
void many_snapshot(ManyBuilder& B, const gd_problem* p, const gd_particles* s, double4* snap)
{
    std::vector<SnapArgs> sn{SnapArgs{to_dev(p), s->m[s->cur], s->M, p->n, snap}};
    B.add<Snapshot>(sn, std::vector<int64_t>{cdiv(p->n, 256)});
}

// the audit of every run
void many_audit(ManyBuilder& B, const std::vector<ManyRun>& R)
{
    const size_t nr = R.size();
    std::vector<ReduceArgs> au(nr);
    std::vector<int64_t> nred(nr);
    for (size_t r = 0; r < nr; ++r) {
        const ManyRun& x = R[r];
        const gd_particles* s = &x.out;
        const int64_t n = x.p.n;
        nred[r] = std::min<int64_t>(kRedBlocks, std::max<int64_t>(1, cdiv(n, B.tune.red_div)));
        au[r] = reduce_args(&x.p, s->m[s->cur], s->M, s->m[s->cur ^ 1], nullptr, n, x.iv, x.ws, x.L);
    }
    B.add<Reduce<1>>(au, nred);
}

}  // namespace gd
