// gd_sort.hip -- Morton order of the active particles (Sect. 2.5.1: the
// neighbour search runs on an adaptive spatial hierarchy over the Morton
// order).  Bounding box, 30-bit keys with the first digit's counts, stable
// LSD radix sort of (key, slot) pairs with 8-bit digits, and the gather of every state array
// into the sorted order.  All kernels are bandwidth-bound streaming passes:
// coalesced loads of the SoA arrays, one 4-byte key and value per particle.
#include "gd_common.hpp"
#include "gd_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace gd {

// ---------------------------------------------------------------------------
// Bounding box and active count: per-block partials, combined by the block
// that ends last (a launch of its own took 4.6 us).  Clears the sort's
// counts.
struct BboxArgs {
    const double *x, *y, *z, *M;
    int64_t n;
    double* red;
    WsHeader* h;
    int32_t* na_out;  // the caller's copy of the active count, or null
    uint32_t* zero;   // counts cleared for the sort
    int64_t nzero;
};

struct Bbox {
    using Args = BboxArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B);
};

__device__ __forceinline__ void Bbox::body(const Args& A, Blk B)
{
    const double *x = A.x, *y = A.y, *z = A.z, *M = A.M;
    const int64_t n = A.n;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    double cnt = 0.0;
    for (int64_t i = B.id * int64_t(blockDim.x) + threadIdx.x; i < A.nzero; i += B.n * blockDim.x) A.zero[i] = 0u;
    // the four arrays are read for every slot (an inactive one is then left
    // out), so that the unrolled iterations' loads are in flight together
#pragma unroll 4
    for (int64_t i = B.id * int64_t(blockDim.x) + threadIdx.x; i < n; i += B.n * blockDim.x) {
        const bool act = M[i] > 0.0;
        const double c[3] = {x[i], y[i], z[i]};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lo[d] = act ? fmin(lo[d], c[d]) : lo[d];
            hi[d] = act ? fmax(hi[d], c[d]) : hi[d];
        }
        cnt += act ? 1.0 : 0.0;
    }
    __shared__ double s[4][7];
    __shared__ int32_t s_last;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double v[7] = {lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], cnt};
#pragma unroll
    for (int d = 0; d < 3; ++d) v[d] = wave_min_d(v[d]);
#pragma unroll
    for (int d = 3; d < 6; ++d) v[d] = wave_max_d(v[d]);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v[6] += shfl_xor_d(v[6], m);
    if (lane == 0)
        for (int d = 0; d < 7; ++d) s[w][d] = v[d];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int ww = 1; ww < int(blockDim.x >> 6); ++ww) {
            for (int d = 0; d < 3; ++d) s[0][d] = fmin(s[0][d], s[ww][d]);
            for (int d = 3; d < 6; ++d) s[0][d] = fmax(s[0][d], s[ww][d]);
            s[0][6] += s[ww][6];
        }
        for (int d = 0; d < 7; ++d) put_device(A.red + B.id * 8 + d, s[0][d]);
        done_stores();
        s_last = last_block(&A.h->red_done, B.n) ? 1 : 0;
    }
    __syncthreads();
    if (!s_last || threadIdx.x >= kWave) return;
    const double* red = A.red;
    const int nblk = int(B.n);
    WsHeader* h = A.h;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        v[d] = INFINITY;
        v[3 + d] = -INFINITY;
    }
    v[6] = 0.0;
#pragma unroll
    for (int r = 0; r < kRedBlocks / kWave; ++r) {
        const int b = r * kWave + lane;
        const bool have = b < nblk;
        const double* p = red + (have ? b : 0) * 8;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            v[d] = fmin(v[d], p[d]);
            v[3 + d] = fmax(v[3 + d], p[3 + d]);
        }
        v[6] += have ? p[6] : 0.0;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        v[d] = wave_min_d(v[d]);
        v[3 + d] = wave_max_d(v[3 + d]);
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) v[6] += shfl_xor_d(v[6], m);
    if (lane != 0) return;
    double ext = 0.0;
    for (int d = 0; d < 3; ++d) {
        const double e = v[3 + d] - v[d];
        if (e > ext) ext = e;
        h->lo[d] = v[d];
        h->hi[d] = v[3 + d];
    }
    h->inv = ext > 0.0 ? 1024.0 / ext : 0.0;
    h->n_active = int32_t(v[6]);
    h->knn_hints = 0;
    if (A.na_out) *A.na_out = int32_t(v[6]);
}

__global__ __launch_bounds__(256) void k_bbox(BboxArgs A)
{
    Bbox::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

// ---------------------------------------------------------------------------
// Morton key: 10 bits per axis, x in bit 3b, y in 3b+1, z in 3b+2.
__device__ inline uint32_t spread3(uint32_t v)
{
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ inline uint32_t quant(double c, double lo, double inv)
{
    const double t = (c - lo) * inv;
    const uint32_t q = uint32_t(t);
    return q > 1023u ? 1023u : q;
}

// ---------------------------------------------------------------------------
// LSD radix sort, 8-bit digits.  Block b owns the keys [b T, (b + 1) T), T =
// 256 rounds, wavefront w of it the w-th quarter.  A pass is a count (row b
// of hist, and added to the row of b's group of `sup` blocks) and a scatter,
// whose blocks add up the group rows and their own group's block rows
// themselves (a scan kernel between the two took 4.7 us a pass).
struct RadixArgs {
    const uint32_t *kin, *vin;
    uint32_t *kout, *vout;
    int64_t n;
    int shift, rounds;
    uint32_t* hist;
    uint32_t* sums;  // this pass's group rows
    int nblk, sup;
};

// the block's digit counts h (LDS) to its row, and onto its group's
__device__ inline void put_counts(const RadixArgs& A, Blk B, const uint32_t* h)
{
    const int t = threadIdx.x;
    const uint32_t c = h[t];
    A.hist[B.id * 256 + t] = c;
    if (c) atomicAdd(&A.sums[(B.id / A.sup) * 256 + t], c);
}

// the keys (and slots) of every particle, and the first pass's counts
struct MortonArgs {
    const double *x, *y, *z, *M;
    const WsHeader* h;
    uint32_t* keys;
    uint32_t* vals;
    RadixArgs r;
};

struct Morton {
    using Args = MortonArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B)
    {
        __shared__ uint32_t cnt[256];
        cnt[threadIdx.x] = 0;
        __syncthreads();
        const WsHeader* h = A.h;
        const double inv = h->inv;
        const double lo[3] = {h->lo[0], h->lo[1], h->lo[2]};
        const int64_t base = B.id * int64_t(256 * A.r.rounds) + threadIdx.x;
#pragma unroll 4
        for (int r = 0; r < A.r.rounds; ++r) {
            const int64_t i = base + r * 256;
            if (i >= A.r.n) break;
            uint32_t key = 0xFFFFFFFFu;
            if (A.M[i] > 0.0)
                key = spread3(quant(A.x[i], lo[0], inv)) | (spread3(quant(A.y[i], lo[1], inv)) << 1) |
                      (spread3(quant(A.z[i], lo[2], inv)) << 2);
            A.keys[i] = key;
            A.vals[i] = uint32_t(i);
            atomicAdd(&cnt[key & 0xFFu], 1u);
        }
        __syncthreads();
        put_counts(A.r, B, cnt);
    }
};

__global__ __launch_bounds__(256) void k_morton(MortonArgs A)
{
    Morton::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

struct RadixHist {
    using Args = RadixArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B)
    {
        __shared__ uint32_t h[256];
        h[threadIdx.x] = 0;
        __syncthreads();
        const int64_t base = B.id * int64_t(256 * A.rounds) + threadIdx.x;
        const int shift = A.shift;
        // the tile's keys are loaded first, all in flight together
        uint32_t kr[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) kr[r] = r < A.rounds && base + r * 256 < A.n ? A.kin[base + r * 256] : 0u;
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r)
            if (r < A.rounds && base + r * 256 < A.n) atomicAdd(&h[(kr[r] >> shift) & 0xFFu], 1u);
        __syncthreads();
        put_counts(A, B, h);
    }
};

__global__ __launch_bounds__(256) void k_radix_hist(RadixArgs A)
{
    RadixHist::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

// Exclusive scan of 256 values held one per thread of a 256-thread block;
// returns this thread's prefix.
__device__ inline uint32_t block_scan_excl_256(uint32_t v, uint32_t* s_w)
{
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    uint32_t before = 0;
    for (int ww = 0; ww < w; ++ww) before += s_w[ww];
    return before + x - v;
}

// The wavefronts rank their quarters of the tile on their own: each counts
// its digits first, the four counts become places, and then every round of
// 64 keys takes its places from the wavefront's own row, with no barrier
// (four barriers a round, shared rows: 12.7 us a pass on 10,007 keys, 7.3 so;
// 5.1 with the count rows read kRows at a time).
// With kStageRounds keys a thread or more the tile goes to LDS in its new
// order first and from there out, so that the keys of a digit are stored side
// by side: 16.5 -> 13.0 us a pass on 1M keys (16 a thread), 10.0 -> 9.1 on
// 300,007; with fewer a digit has a run of one to three keys, and the barriers
// cost what the stores save.
constexpr int kStageRounds = 4;

struct RadixScatter {
    using Args = RadixArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B);
};

__device__ __forceinline__ void RadixScatter::body(const Args& A, Blk B)
{
    const int64_t n = A.n;
    const int shift = A.shift, rounds = A.rounds;
    __shared__ uint32_t at[4][256];  // per wavefront: counts, then the next place of each digit
    __shared__ uint32_t s_w[4], s_w2[4];
    __shared__ uint32_t s_key[256 * kSortRounds], s_val[256 * kSortRounds], s_delta[256];
    const bool stage = rounds >= kStageRounds;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    // the tile's keys and values are loaded first, all in flight together
    const int64_t base = B.id * int64_t(256 * rounds) + int64_t(w) * (64 * rounds) + lane;
    uint32_t kr[kSortRounds], vr[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const bool in = r < rounds && base + r * 64 < n;
        kr[r] = in ? A.kin[base + r * 64] : 0u;
        vr[r] = in ? A.vin[base + r * 64] : 0u;
    }
    // digit t: the keys of it in all blocks, and in the blocks before this one
    const int grp = int(B.id / A.sup), ngrp = (A.nblk + A.sup - 1) / A.sup;
    // (kRows rows in flight at a time, the missing ones read as row 0 and dropped)
    constexpr int kRows = 16;
    uint32_t total = 0, before = 0;
    for (int g0 = 0; g0 < ngrp; g0 += kRows) {
        uint32_t c[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) c[u] = A.sums[(g0 + u < ngrp ? g0 + u : 0) * 256 + t];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            total += g0 + u < ngrp ? c[u] : 0u;
            before += g0 + u < grp ? c[u] : 0u;
        }
    }
    for (int b0 = grp * A.sup; b0 < int(B.id); b0 += kRows) {
        uint32_t c[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) c[u] = A.hist[(b0 + u < int(B.id) ? b0 + u : 0) * 256 + t];
#pragma unroll
        for (int u = 0; u < kRows; ++u) before += b0 + u < int(B.id) ? c[u] : 0u;
    }
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) at[ww][t] = 0;
    const uint32_t goff = block_scan_excl_256(total, s_w) + before;  // (holds a barrier)
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r)
        if (r < rounds && base + r * 64 < n) atomicAdd(&at[w][(kr[r] >> shift) & 0xFFu], 1u);
    __syncthreads();
    {
        uint32_t p = goff;
        if (stage) {  // places within the tile; digit t's lie s_delta[t] below their global ones
            const uint32_t c = at[0][t] + at[1][t] + at[2][t] + at[3][t];
            p = block_scan_excl_256(c, s_w2);
            s_delta[t] = goff - p;
        }
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
            const uint32_t c = at[ww][t];
            at[ww][t] = p;
            p += c;
        }
    }
    __syncthreads();
    const uint64_t lt = (uint64_t(1) << lane) - 1;
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        if (r >= rounds) break;
        const bool valid = base + r * 64 < n;
        const uint32_t dig = (kr[r] >> shift) & 0xFFu;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool set = (dig >> bit) & 1u;
            const uint64_t bs = __ballot(set);
            peers &= set ? bs : ~bs;
        }
        const uint32_t rank = uint32_t(__popcll(peers & lt));
        if (valid) {
            const uint32_t off = at[w][dig] + rank;
            if (stage) {
                s_key[off] = kr[r];
                s_val[off] = vr[r];
            } else {
                A.kout[off] = kr[r];
                A.vout[off] = vr[r];
            }
            // (the wavefront's LDS operations run in order: every peer has
            // read its place when the last of them moves it on)
            if (rank + 1 == uint32_t(__popcll(peers))) at[w][dig] = off + 1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (!stage) return;
    __syncthreads();
    const int64_t left = n - B.id * int64_t(256 * rounds);
    const int m = left < 256 * rounds ? int(left) : 256 * rounds;
#pragma unroll 4
    for (int e = t; e < m; e += 256) {
        const uint32_t key = s_key[e];
        const uint32_t to = uint32_t(e) + s_delta[(key >> shift) & 0xFFu];
        A.kout[to] = key;
        A.vout[to] = s_val[e];
    }
}

__global__ __launch_bounds__(256) void k_radix_scatter(RadixArgs A)
{
    RadixScatter::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

// ---------------------------------------------------------------------------
// Gather of every state array into Morton order, plus the packed positions.
struct Permute {
    using Args = PermuteArgs;
    static constexpr int kThreads = 256;
    static __device__ __forceinline__ void body(const Args& A, Blk B);
};

__global__ __launch_bounds__(256) void k_permute(PermuteArgs A)
{
    Permute::body(A, Blk{int64_t(blockIdx.x), int64_t(gridDim.x)});
}

__device__ __forceinline__ void Permute::body(const Args& A, Blk B)
{
    const int64_t i = B.id * int64_t(blockDim.x) + threadIdx.x;
    if (i >= A.n) return;
    const uint32_t s = A.perm[i];
    // every gather is issued before any store (the array count is uniform),
    // so a lane keeps all of its loads in flight at once
    double v[16];
#pragma unroll
    for (int a = 0; a < 16; ++a) v[a] = a < A.nd ? A.src[a][s] : 0.0;
    const uint32_t id = A.id_src[s];
    const double hint = A.hint_src ? A.hint_src[s] : 0.0;
#pragma unroll
    for (int a = 0; a < 16; ++a)
        if (a < A.nd) A.dst[a][i] = v[a];
    A.id_dst[i] = id;
    A.pos4[i] = make_double4(v[0], v[1], v[2], 0.0);  // x, y, z are the first three arrays
    A.hint_dst[i] = hint;
    // one block in 16 tells the search whether there are previous distances
    // (it picks the faster of two exact searches, so a sample will do)
    if ((B.id & 15) == 0 && hint > 0.0) *A.hints = 1;
}

__global__ void k_fill_i32(int32_t* __restrict__ a, int64_t n, int32_t v)
{
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i < n) a[i] = v;
}

// ---------------------------------------------------------------------------
// the sort's arguments for one run (state `in` into `out`); the radix passes
// alternate between (keys0, vals0) and (keys1, vals1)
struct SortArgs {
    BboxArgs bbox;
    MortonArgs morton;
    RadixArgs pass[4];
    PermuteArgs perm;
};

static SortArgs sort_args(const gd_problem* p, const gd_particles* in, gd_particles* out, const double* hint,
                          int32_t* na_out, void* ws, const Layout& L)
{
    const int64_t n = p->n;
    WsHeader* h = at<WsHeader>(ws, L.hdr);
    double* red = at<double>(ws, L.red);
    SortArgs S{};
    uint32_t* k0 = at<uint32_t>(ws, L.keys0);
    uint32_t* k1 = at<uint32_t>(ws, L.keys1);
    uint32_t* v0 = at<uint32_t>(ws, L.vals0);
    uint32_t* v1 = at<uint32_t>(ws, L.vals1);
    uint32_t* hist = at<uint32_t>(ws, L.hist);
    const int nsb = L.nsort_blocks;
    uint32_t* sums = hist + int64_t(256) * nsb;  // per pass: the group rows
    const int64_t row = int64_t(256) * L.nsort_sup;
    S.bbox = BboxArgs{in->x, in->y, in->z, in->M, n, red, h, na_out, sums, 4 * row};
    for (int pass = 0; pass < 4; ++pass) {
        const bool odd = pass & 1;
        S.pass[pass] = RadixArgs{odd ? k1 : k0, odd ? v1 : v0, odd ? k0 : k1, odd ? v0 : v1, n, 8 * pass,
                                 L.sort_rounds, hist, sums + pass * row, nsb, L.sort_sup};
    }
    S.morton = MortonArgs{in->x, in->y, in->z, in->M, h, k0, v0, S.pass[0]};
    // sorted (key, slot) pairs are back in (k0, v0)
    PermuteArgs& A = S.perm;
    A.n = n;
    A.perm = v0;
    int nd = 0;
    auto add = [&](const double* s, double* d) {
        if (s) {
            A.src[nd] = s;
            A.dst[nd] = d;
            ++nd;
        }
    };
    add(in->x, out->x);
    add(in->y, out->y);
    add(in->z, out->z);
    add(in->M, out->M);
    add(in->m[in->cur], out->m[in->cur]);
    add(in->r, out->r);
    add(in->th, out->th);
    add(in->ph, out->ph);
    add(in->vr, out->vr);
    add(in->lth, out->lth);
    add(in->lph, out->lph);
    add(in->vz, out->vz);
    add(in->st_mid, out->st_mid);
    A.nd = nd;
    A.id_src = in->id;
    A.id_dst = out->id;
    A.pos4 = at<double4>(ws, L.pos4);
    A.hint_src = hint;
    A.hint_dst = at<double>(ws, L.hint);
    A.hints = &h->knn_hints;
    return S;
}

// blocks of the bounding box: at most kRedBlocks, four slots or more a thread
static int64_t bbox_blocks(int64_t n) { return std::min<int64_t>(kRedBlocks, std::max<int64_t>(1, cdiv(n, 1024))); }

int launch_morton_sort(const gd_problem* p, const gd_particles* in, gd_particles* out, const double* hint,
                       int32_t* na_out, void* ws, const Layout& L, hipStream_t st)
{
    const int64_t n = p->n;
    const SortArgs S = sort_args(p, in, out, hint, na_out, ws, L);
    prof_mark(GD_PROF_SORT, 0, st);
    hipLaunchKernelGGL(k_bbox, dim3(unsigned(bbox_blocks(n))), dim3(256), 0, st, S.bbox);
    const int nb = int((n + 255) / 256);
    const int nsb = L.nsort_blocks;
    hipLaunchKernelGGL(k_morton, dim3(nsb), dim3(256), 0, st, S.morton);
    for (int pass = 0; pass < 4; ++pass) {
        if (pass > 0) hipLaunchKernelGGL(k_radix_hist, dim3(nsb), dim3(256), 0, st, S.pass[pass]);
        hipLaunchKernelGGL(k_radix_scatter, dim3(nsb), dim3(256), 0, st, S.pass[pass]);
    }
    hipLaunchKernelGGL(k_permute, dim3(nb), dim3(256), 0, st, S.perm);
    prof_mark(GD_PROF_SORT, 1, st);
    out->cur = in->cur;
    return 0;
}

void many_sort(ManyBuilder& B, const std::vector<ManyRun>& R)
{
    const size_t nr = R.size();
    std::vector<SortArgs> S(nr);
    std::vector<int64_t> nbb(nr), nb(nr), nsb(nr);
    for (size_t r = 0; r < nr; ++r) {
        const ManyRun& x = R[r];
        const int64_t n = x.p.n;
        nbb[r] = n > 0 ? std::min<int64_t>(kRedBlocks, std::max<int64_t>(1, cdiv(n, B.tune.red_div))) : 0;
        gd_particles out = x.out;
        S[r] = sort_args(&x.p, &x.in, &out, x.nb.dmax, x.nb.n_active, x.ws, x.L);
        nb[r] = cdiv(n, 256);
        nsb[r] = n > 0 ? x.L.nsort_blocks : 0;
    }
    auto pick = [&](auto f) {
        using A = std::remove_reference_t<decltype(f(S[0]))>;
        std::vector<A> v(nr);
        for (size_t r = 0; r < nr; ++r) v[r] = f(S[r]);
        return v;
    };
    B.add<Bbox>(pick([](SortArgs& a) -> BboxArgs& { return a.bbox; }), nbb);
    B.add<Morton>(pick([](SortArgs& a) -> MortonArgs& { return a.morton; }), nsb);
    for (int pass = 0; pass < 4; ++pass) {
        auto tab = pick([pass](SortArgs& a) -> RadixArgs& { return a.pass[pass]; });
        if (pass > 0) B.add<RadixHist>(tab, nsb);
        B.add<RadixScatter>(tab, nsb);
    }
    B.add<Permute>(pick([](SortArgs& a) -> PermuteArgs& { return a.perm; }), nb);
}

void launch_fill_i32(int32_t* a, int64_t n, int32_t v, hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill_i32, dim3(int((n + 255) / 256)), dim3(256), 0, st, a, n, v);
}

}  // namespace gd
