// gd_knn_wave.hip -- the N_K nearest neighbours of one query per wavefront
// (Sect. 2.5.1), exact, for any k up to kMaxK.  It serves neighbourhoods too
// large for the shared-list searches' registers and LDS lists, and the
// queries those searches hand back.
//
// Per query (one 64-lane wavefront):
//   1. the search radius: the particle's distance from the previous search
//      widened by kHintSlack when that is usable, else the (k-1)-th distance
//      to the others in a window of Morton slots about the query (an upper
//      bound of the one sought), capped by the maximum search scale;
//   2. a depth-first traversal of the box tree in Morton order, kPop nodes at
//      a time: each lane tests child boxes against the query's sphere (the
//      conservative single-precision test of gd_knn.hpp); passing internal
//      children go on an LDS stack, the leftmost on top, passing buckets to a
//      bucket buffer.  Levels grow from the top of the stack down, so the
//      level-1 nodes of a batch lie left of its other nodes and the buckets
//      come out in ascending order;
//   3. the buffered buckets' slots are evaluated kEval per lane: every other
//      at or below the cut (d^2, slot) <= (R2, J) joins an LDS list of
//      (d^2, slot) pairs, compacted across the wavefront in ascending slot
//      order.  When the list would overflow, it is cut in place to its k-1
//      smallest pairs, and the cut moves to the last of them (so equal
//      distances beyond it are decided by slot, and the radius only shrinks,
//      which keeps the pruning of step 2 exact);
//   4. if the previous distance held fewer than k-1 others, the query runs
//      again on the window bound;
//   5. the (k-1)-th smallest pair is selected (select_pair) and the pairs up
//      to it are written as the row: the list is in slot order already, so
//      nothing is sorted.
// d^2 is (dx*dx + dy*dy) + dz*dz with every operation rounded on its own, and
// non-negative doubles order as their bit patterns, so the selection is the
// k-1 smallest (d^2, slot) exactly.
#include "gd_common.hpp"
#include "gd_internal.hpp"
#include "gd_knn.hpp"

namespace gd {

constexpr int kPop = 8;          // nodes expanded at a time, eight lanes each
constexpr int kWBuf = 128;       // buckets waiting for evaluation: flushed from 64 on
constexpr int kEval = 2;         // slots a lane evaluates at a time

// A level's nodes join the stack only when fewer than kPop nodes of lower
// levels were on it (a batch takes them all), so each level has at most
// kPop * kFan nodes waiting.
constexpr int kWStack = (kMaxTreeLevels - 1) * kPop * kFan;

// NL: (d^2, slot) pairs a query keeps
template <int NL>
struct WaveLds {
    static constexpr int kBins = NL > 192 ? 256 : 64;  // of the selection's distance histogram
    uint64_t key[NL];        // d^2 as its bit pattern
    int32_t slot[NL];        // ascending
    int32_t stack[kWStack];  // node: level << 27 | index
    int32_t buf[kWBuf];      // bucket indices, ascending
    uint32_t hist[kBins];
    int32_t bnd[kWave];      // list places of the boundary bin's pairs
};

__device__ inline uint64_t d2_key(double d2) { return uint64_t(__double_as_longlong(d2)); }
__device__ inline uint64_t lanes_below(int lane) { return (uint64_t(1) << lane) - 1; }

// The need-th smallest (key, slot) of the list's n >= need >= 1 pairs, whose
// keys are d^2 <= R2: a histogram of d^2, linear over [0, R2], finds the bin
// that holds it; that bin's pairs (one or two as a rule) are ranked one
// against all.  A bin of more than 64 pairs (many equal distances) is
// resolved by bisection on the key's bits instead, and equal keys by their
// order in the list, which is the slot order.  Sorting
// the list in LDS instead, 45 bitonic stages for 512 pairs and then the slots,
// was most of the search: on a disk of 131,072 particles at k = 256 an
// interval took 4.21 ms with the sorts and takes 1.02 ms without.
template <int NL>
__device__ __forceinline__ void select_pair(WaveLds<NL>& L, int n, int need, double R2, int lane, uint64_t& T, int32_t& J)
{
    constexpr int NP = NL / kWave;
    constexpr int kSelBins = WaveLds<NL>::kBins, NB = kSelBins / kWave;
    uint64_t key[NP];
#pragma unroll
    for (int b = 0; b < NB; ++b) L.hist[b * kWave + lane] = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) key[p] = p * kWave + lane < n ? L.key[p * kWave + lane] : ~uint64_t(0);
    const double sc = R2 > 0.0 ? double(kSelBins) / R2 : 0.0;
    const bool lin = sc > 0.0 && sc < INFINITY;
    auto bin_of_key = [&](uint64_t kk) {
        if (!lin) return 0;
        const double t = __longlong_as_double((long long)kk) * sc;
        return t < double(kSelBins) ? int(t) : kSelBins - 1;
    };
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p)
        if (p * kWave < n && p * kWave + lane < n) atomicAdd(&L.hist[bin_of_key(key[p])], 1u);
    __syncthreads();
    // lane l's bins: NB l .. NB l + NB - 1
    int own[NB], sum = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        own[b] = int(L.hist[lane * NB + b]);
        sum += own[b];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    const uint64_t reach = __ballot(incl >= need);
    const int lsel = __ffsll((unsigned long long)reach) - 1;  // (n >= need: some lane reaches it)
    int bsel = 0, before = incl - sum, inbin = 0;
    bool found = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (!found && before + own[b] >= need) {
            found = true;
            bsel = lane * NB + b;
            inbin = own[b];
        }
        if (!found) before += own[b];
    }
    bsel = __builtin_amdgcn_readlane(bsel, lsel);
    before = __builtin_amdgcn_readlane(before, lsel);
    inbin = __builtin_amdgcn_readlane(inbin, lsel);
    if (inbin <= kWave) {
        const int want = need - before - 1;  // rank of the pair sought within the bin
        int nb = 0;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (p * kWave < n) {
                const bool in = p * kWave + lane < n && bin_of_key(key[p]) == bsel;
                const uint64_t bal = __ballot(in);
                if (in) L.bnd[nb + int(__popcll(bal & lanes_below(lane)))] = p * kWave + lane;
                nb += int(__popcll(bal));
            }
        }
        __syncthreads();
        const bool have = lane < nb;
        const int at = have ? L.bnd[lane] : 0;
        const uint64_t kk = have ? L.key[at] : ~uint64_t(0);
        int rank = 0;  // equal keys: the list order (lane order) decides
        for (int f = 0; f < nb; ++f) {
            const uint64_t kf = readlane_u64(kk, f);
            rank += (kf < kk) | ((kf == kk) & (f < lane));
        }
        const uint64_t hit = __ballot(have && rank == want);
        const int l = __ffsll((unsigned long long)hit) - 1;
        T = readlane_u64(kk, l);
        J = L.slot[__builtin_amdgcn_readlane(at, l)];
        __syncthreads();
        return;
    }
    // the largest T with fewer than `need` keys below it
    uint64_t t = 0;
    int less = 0;
    for (int bit = 62; bit >= 0; --bit) {
        const uint64_t c = t | (uint64_t(1) << bit);
        int cnt = 0;
#pragma unroll
        for (int p = 0; p < NP; ++p) cnt += int(__popcll(__ballot(key[p] < c)));
        if (cnt < need) {
            t = c;
            less = cnt;
        }
    }
    if (t == 0) less = 0;
    T = t;
    int left = need - less;  // the pair sought is the left-th of those with key T, in list order
    J = -1;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint64_t bal = __ballot(p * kWave + lane < n && key[p] == t);
        const int c = int(__popcll(bal));
        if (left > 0 && left <= c) {
            const bool it = ((bal >> lane) & 1u) && int(__popcll(bal & lanes_below(lane))) == left - 1;
            const uint64_t hit = __ballot(it);
            J = L.slot[p * kWave + __ffsll((unsigned long long)hit) - 1];
        }
        left -= c;
    }
    __syncthreads();
}

template <bool PER, int NL>
__device__ __forceinline__ void knn_wave_query(const KnnArgs& A, int q, WaveLds<NL>& L, int lane)
{
    constexpr int NP = NL / kWave;
    const int na = A.h->n_active;
    const int k = A.k;
    const int need = k - 1;
    int32_t* row = A.nbr + int64_t(q) * k;
    if (q >= na || na == 1) {
        const bool act = q < na;
        for (int s = lane; s < k; s += kWave) row[s] = s == 0 ? (act ? q : -1) : -1;
        if (lane == 0) {
            A.cnt[q] = act ? 1 : 0;
            A.dmax[q] = 0.0;
        }
        return;
    }
    const double4 q4 = A.pos[q];
    const double qp[3] = {q4.x, q4.y, q4.z};
    if (!(fabs(qp[0]) < INFINITY && fabs(qp[1]) < INFINITY && fabs(qp[2]) < INFINITY)) {
        if (lane == 0) set_status(A.ws, GD_DEV_NONFINITE);  // non-finite position: self only
        for (int s = lane; s < k; s += kWave) row[s] = s == 0 ? q : -1;
        if (lane == 0) {
            A.cnt[q] = 1;
            A.dmax[q] = 0.0;
        }
        return;
    }
    QF qf;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        qf.c[a] = float(qp[a]);
        qf.p[a] = PER ? float(qp[a] + A.L[a]) : 0.0f;
        qf.m[a] = PER ? float(qp[a] - A.L[a]) : 0.0f;
    }

    // 1. the previous distance as the first radius, when usable: positive,
    //    finite and within the diagonal of the active set's box
    double R2hint = INFINITY;
    {
        const double hv = A.hint[q] * kHintSlack;
        if (hv > 0.0 && hv < INFINITY) {
            if (hv * hv <= diagonal2(A.h)) R2hint = hv * hv;
        }
    }
    // without one, the (k-1)-th distance to the others among the NL slots
    // about the query: an upper bound of the distance sought, some 1.15 times
    // it at the median in a disk or a uniform box
    auto window_bound = [&]() __attribute__((always_inline)) {
        int lo = q - NL / 2;
        lo = lo + NL > na ? na - NL : lo;
        lo = lo < 0 ? 0 : lo;
        int m = 0;
        double far = 0.0;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int j = lo + p * kWave + lane;
            const bool ok = j < na && j != q;
            const double d2 = sep2_slot<PER>(A, qp, ok ? j : q);
            const bool in = ok && d2 < INFINITY;
            const uint64_t bal = __ballot(in);
            if (in) {
                const int at = m + int(__popcll(bal & lanes_below(lane)));
                L.key[at] = d2_key(d2);
                L.slot[at] = j;
                far = fmax(far, d2);
            }
            m += int(__popcll(bal));
        }
        __syncthreads();
        if (m < need) return double(INFINITY);  // (fewer than k slots: every other is a neighbour)
        uint64_t T;
        int32_t J;
        select_pair<NL>(L, m, need, wave_max_d(far), lane, T, J);
        return __longlong_as_double((long long)T);
    };

    bool use_hint = R2hint < INFINITY;
    double R2cap = A.rmax2;
    int n = 0;
    double R2 = 0.0;
    int32_t Jc = INT32_MAX;
    for (;;) {
        if (!use_hint) R2cap = fmin(window_bound(), A.rmax2);
        R2 = use_hint ? fmin(R2hint, R2cap) : R2cap;
        Jc = INT32_MAX;
        n = 0;
        float R2f = r2f(R2);
        int sp = 0, nbuf = 0;
        // cut the list to its k-1 smallest pairs, kept in order; the cut
        // moves to the last of them (n > need here)
        auto cut_list = [&]() __attribute__((always_inline)) {
            uint64_t T;
            int32_t J;
            __syncthreads();
            select_pair<NL>(L, n, need, R2, lane, T, J);
            R2 = __longlong_as_double((long long)T);
            Jc = J;
            R2f = r2f(R2);
            uint64_t key[NP];
            int32_t slot[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const bool in = p * kWave + lane < n;
                key[p] = in ? L.key[p * kWave + lane] : ~uint64_t(0);
                slot[p] = in ? L.slot[p * kWave + lane] : INT32_MAX;
            }
            __syncthreads();
            int kept = 0;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const bool keep = key[p] < T || (key[p] == T && slot[p] <= J);
                const uint64_t bal = __ballot(keep);
                if (keep) {
                    const int at = kept + int(__popcll(bal & lanes_below(lane)));
                    L.key[at] = key[p];
                    L.slot[at] = slot[p];
                }
                kept += int(__popcll(bal));
            }
            n = kept;
            __syncthreads();
        };
        // evaluate the buffered buckets in order, kEval slots per lane at a time
        auto flush = [&]() __attribute__((always_inline)) {
            constexpr int kStep = kWave * kEval / kBucket;  // buckets
            for (int b0 = 0; b0 < nbuf; b0 += kStep) {
                double d2[kEval];
                int32_t jj[kEval];
                bool acc[kEval];
                int total = 0;
#pragma unroll
                for (int t = 0; t < kEval; ++t) {
                    const int p = lane + kWave * t;
                    const int b = b0 + (p >> 2);
                    const int j = b < nbuf ? L.buf[b] * kBucket + (p & 3) : -1;
                    const bool ok = j >= 0 && j < na && j != q;
                    jj[t] = ok ? j : -1;
                }
                // every lane reads a slot (a lane without one its own query)
                // so that the loads are in flight together
#pragma unroll
                for (int t = 0; t < kEval; ++t) d2[t] = sep2_slot<PER>(A, qp, jj[t] >= 0 ? jj[t] : q);
#pragma unroll
                for (int t = 0; t < kEval; ++t) {
                    acc[t] = jj[t] >= 0 && (d2[t] < R2 || (d2[t] == R2 && jj[t] <= Jc));
                    total += int(__popcll(__ballot(acc[t])));
                }
                if (n + total > NL) {
                    cut_list();
#pragma unroll
                    for (int t = 0; t < kEval; ++t)
                        acc[t] = acc[t] && (d2[t] < R2 || (d2[t] == R2 && jj[t] <= Jc));
                }
#pragma unroll
                for (int t = 0; t < kEval; ++t) {
                    const uint64_t bal = __ballot(acc[t]);
                    if (acc[t]) {
                        const int at = n + int(__popcll(bal & lanes_below(lane)));
                        L.key[at] = d2_key(d2[t]);
                        L.slot[at] = jj[t];
                    }
                    n += int(__popcll(bal));
                }
            }
            nbuf = 0;
            __syncthreads();
        };
        // the walk starts on the lowest level of at most 64 nodes, a lane each
        {
            const int lv = A.T.start;
            const bool valid = (int64_t(lane) << (2 + 3 * lv)) < na;  // the node holds active slots
            bool pass = false;
            if (valid) pass = box2f<PER>(A, qf, A.boxes[level_off(A.T, lv) + lane]) <= R2f;
            const uint64_t bal = __ballot(pass);
            const int c = int(__popcll(bal)), at = int(__popcll(bal & lanes_below(lane)));
            if (pass) {
                if (lv == 0) L.buf[at] = lane;
                else L.stack[c - 1 - at] = (lv << 27) | lane;
            }
            if (lv == 0) nbuf = c;
            else sp = c;
            __syncthreads();
        }
        for (;;) {
            if (nbuf >= kWave || sp == 0) flush();
            if (sp == 0) break;
            const int nt = sp < kPop ? sp : kPop;
            const int my = lane >> 3, c = lane & 7;
            const int32_t node = my < nt ? L.stack[sp - 1 - my] : 0;  // the leftmost first
            __syncthreads();
            sp -= nt;
            const int lv = node >> 27, idx = node & ((1 << 27) - 1);
            bool pass = false;
            bool leaf = false;
            const int child = idx * kFan + c;
            if (my < nt && (child << (3 * lv - 1)) < na) {  // the child holds active slots (its first is 4 8^(lv-1) child < 2^31)
                const FBox bx = A.boxes[level_off(A.T, lv - 1) + child];
                pass = box2f<PER>(A, qf, bx) <= R2f;
                leaf = lv == 1;
            }
            const uint64_t bin = __ballot(pass && !leaf), bleaf = __ballot(pass && leaf);
            const int ni = int(__popcll(bin));
            if (pass && !leaf)
                L.stack[sp + ni - 1 - int(__popcll(bin & lanes_below(lane)))] = ((lv - 1) << 27) | child;
            if (pass && leaf) L.buf[nbuf + int(__popcll(bleaf & lanes_below(lane)))] = child;
            sp += ni;
            nbuf += int(__popcll(bleaf));
            __syncthreads();
        }
        if (use_hint && n < need && R2hint < R2cap) {
            use_hint = false;  // the previous distance held too few others: again on the bound
            continue;
        }
        break;
    }
    // 5. the k-1 smallest pairs (all of them when fewer are within the cap),
    //    in slot order
    uint64_t T = ~uint64_t(0);
    int32_t J = INT32_MAX;
    int m = n;
    double maxd2 = 0.0;
    if (n > need) {
        select_pair<NL>(L, n, need, R2, lane, T, J);
        m = need;
    }
    int at = 0;
    if (lane == 0) row[0] = q;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (p * kWave < n) {
            const bool in = p * kWave + lane < n;
            const uint64_t kk = in ? L.key[p * kWave + lane] : ~uint64_t(0);
            const int32_t sl = in ? L.slot[p * kWave + lane] : 0;
            const bool keep = in && (kk < T || (kk == T && sl <= J));
            const uint64_t bal = __ballot(keep);
            if (keep) {
                row[1 + at + int(__popcll(bal & lanes_below(lane)))] = sl;
                maxd2 = fmax(maxd2, __longlong_as_double((long long)kk));
            }
            at += int(__popcll(bal));
        }
    }
    for (int s = 1 + m + lane; s < k; s += kWave) row[s] = -1;
    maxd2 = n > need ? __longlong_as_double((long long)T) : wave_max_d(maxd2);
    if (at != m && lane == 0) set_status(A.ws, GD_DEV_INTERNAL);
    if (lane == 0) {
        A.cnt[q] = 1 + m;
        A.dmax[q] = m > 0 ? sqrt(maxd2) : 0.0;
    }
    __syncthreads();
}

// One query per 64-thread workgroup: every slot [0, n), or the slots of
// `list` [0, *count) when a list is given.
template <bool PER, int NL>
struct KnnWave {
    using Args = WaveArgs;
    static constexpr int kThreads = kWave;
    static __device__ __forceinline__ void body(const Args& W, Blk B)
    {
        __shared__ WaveLds<NL> L;
        const int lane = threadIdx.x;
        if (W.list) {
            // the list, or, with no previous distances, all queries in slot
            // order (handed back by the tiles they came in any order, after 60
            // us: a first search of 300,007 took 806 us, so 728)
            const bool all = !W.A.h->knn_hints;
            const ListShare s = list_share(B.id, B.n, all ? int32_t(W.A.n) : *W.count);
            for (int32_t t = s.first; t < s.end; t += s.step)
                knn_wave_query<PER, NL>(W.A, all ? t : W.list[t], L, lane);
        } else {
            const int64_t q = B.id;
            if (q < W.A.n) knn_wave_query<PER, NL>(W.A, int(q), L, lane);
        }
    }
};

// The search waits on memory and LDS, so the wavefronts in flight set its
// pace: with the short list 4, 5, 6, 7 and 8 of them (8 spills 44 bytes) took
// 608, 577, 543, 538 and 539 us per cadence step at 131,072 particles.
template <bool PER, int NL>
constexpr int kWavesPerSimd<KnnWave<PER, NL>> = NL == 192 ? 7 : 5;

template <bool PER, int NL>
__global__ __launch_bounds__(kWave, (kWavesPerSimd<KnnWave<PER, NL>>)) void k_knn_wave(WaveArgs W)
{
    KnnWave<PER, NL>::body(W, Blk{W.list ? int64_t(blockIdx.x) : xcd_block(), int64_t(gridDim.x)});
}

// the list's length for neighbourhoods of k: the k - 1 pairs a cut keeps and
// an evaluation step of 64 kEval more always fit
constexpr int kListSmall = 192, kListLarge = 384;
constexpr int kSmallK = kListSmall - kEval * kWave + 1;
static_assert(kListLarge >= (kMaxK - 1) + kEval * kWave, "a step after a cut must fit the list");

void launch_knn_wave(const KnnArgs& A, bool per, const int32_t* list, const int32_t* count, int64_t nblocks,
                     hipStream_t st)
{
    const dim3 grid(unsigned(nblocks > 0 ? nblocks : 1));
    const WaveArgs W{A, list, count};
    if (A.k <= kSmallK) {
        if (per) hipLaunchKernelGGL((k_knn_wave<true, kListSmall>), grid, dim3(kWave), 0, st, W);
        else hipLaunchKernelGGL((k_knn_wave<false, kListSmall>), grid, dim3(kWave), 0, st, W);
    } else {
        if (per) hipLaunchKernelGGL((k_knn_wave<true, kListLarge>), grid, dim3(kWave), 0, st, W);
        else hipLaunchKernelGGL((k_knn_wave<false, kListLarge>), grid, dim3(kWave), 0, st, W);
    }
}

void many_add_wave(ManyBuilder& B, const std::vector<WaveArgs>& tab, const std::vector<int64_t>& nb, bool per)
{
    std::vector<int64_t> small(nb), large(nb);
    bool any_s = false, any_l = false;
    for (size_t r = 0; r < nb.size(); ++r) {
        const bool s = tab[r].A.k <= kSmallK;
        (s ? large : small)[r] = 0;
        any_s = any_s || small[r] > 0;
        any_l = any_l || large[r] > 0;
    }
    if (any_s) {
        if (per) B.add<KnnWave<true, kListSmall>>(tab, small);
        else B.add<KnnWave<false, kListSmall>>(tab, small);
    }
    if (any_l) {
        if (per) B.add<KnnWave<true, kListLarge>>(tab, large);
        else B.add<KnnWave<false, kListLarge>>(tab, large);
    }
}

}  // namespace gd
