// Index pass: grid cell, in-cell fraction and tile of every sample location,
// a stable counting sort of the samples by tile, and the spread's owner-tile
// lists.
//
// The appendix interpolates each sample from J uniform frequencies at
// offsets k_m + j.  Those taps follow from the cell that contains
// u = omega K / (2 pi) and the fraction of u inside it; the tile order puts
// samples that touch the same region of the oversampled grid next to each
// other, which the gather (cache locality) and the spread (tile ownership)
// rely on.
//
// Arithmetic (bit-exact by construction):
//   u = (double)omega * scale_d   (one FP64 multiply, never contracted)
//   fl = floor(u); frac = (float)(u - fl); cell = fl mod K (integer)
// Non-finite omega or |u| >= 2^40 marks the sample as flagged: cell 0,
// frac 0, tile id ntiles (sorted after every finite sample).
#include "kbn_internal.h"
#include "kbn_window.h"

namespace {

constexpr double kULimit = 1099511627776.0;  // 2^40

// One workgroup per chunk of `chunk` samples: cell, fraction and tile of
// every sample, and the chunk's tile histogram (LDS), stored bin-major
// (counts[bin * nchunks + chunk]) for the scan.
__global__ void __launch_bounds__(256)
k_points_hist(int D, int64_t M, int chunk, int nchunks, int nbins, const float *__restrict__ omega,
              double s0, double s1, double s2, int K0, int K1, int K2, int T0, int T1, int T2, int nt1,
              int nt2, int ntiles, int *__restrict__ cell_tmp, float *__restrict__ frac_tmp,
              int *__restrict__ tile, int *__restrict__ flag, int *__restrict__ counts) {
#pragma clang fp contract(off)
    extern __shared__ int hist[];
    const int ch = blockIdx.x;
    for (int i = threadIdx.x; i < nbins; i += blockDim.x) hist[i] = 0;
    __syncthreads();
    const double sc[3] = {s0, s1, s2};
    const int Kd[3] = {K0, K1, K2};
    const int64_t beg = (int64_t)ch * chunk;
    const int64_t end = beg + chunk < M ? beg + chunk : M;
    for (int64_t m = beg + threadIdx.x; m < end; m += blockDim.x) {
        int c[3] = {0, 0, 0};
        float f[3] = {0.f, 0.f, 0.f};
        bool bad = false;
        for (int d = 0; d < D; ++d) {
            const double u = (double)omega[m * D + d] * sc[d];
            if (!(fabs(u) < kULimit)) {
                bad = true;
                continue;
            }
            const double fl = floor(u);
            f[d] = (float)(u - fl);
            const long long l = (long long)fl;
            long long r = l % (long long)Kd[d];
            if (r < 0) r += Kd[d];
            c[d] = (int)r;
        }
        int t;
        if (bad) {
            for (int d = 0; d < 3; ++d) {
                c[d] = 0;
                f[d] = 0.f;
            }
            t = ntiles;
            atomicOr(flag, 1);
        } else {
            t = c[0] / T0;
            if (D > 1) t = t * nt1 + c[1] / T1;
            if (D > 2) t = t * nt2 + c[2] / T2;
        }
        for (int d = 0; d < D; ++d) {
            cell_tmp[d * M + m] = c[d];
            frac_tmp[d * M + m] = f[d];
        }
        tile[m] = t;
        atomicAdd(&hist[t], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nbins; i += blockDim.x) counts[(int64_t)i * nchunks + ch] = hist[i];
}

__device__ __forceinline__ int block_scan_1024(int x, int *wsum, int &total) {
    // inclusive scan over a 1024-thread block; returns the exclusive prefix
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int inc = x;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) wsum[wid] = inc;
    lds_barrier();
    int wpre = 0, tot = 0;
    for (int w = 0; w < 16; ++w) {
        const int ws = wsum[w];
        if (w < wid) wpre += ws;
        tot += ws;
    }
    lds_barrier();
    total = tot;
    return wpre + inc - x;
}

// Gather subproblems from the tile offsets: bin t with n points contributes
// ceil(n / sub) entries (bin, first sorted position); the last bin holds the
// flagged points.  Run by one 1024-thread workgroup after toff is complete.
__device__ void subproblems_block(int nbins, int sub, const int *__restrict__ toff, int *__restrict__ subs,
                                  int *__restrict__ nsub, int *wsum) {
    const int tid = threadIdx.x;
    const int seg = (nbins + 1023) / 1024;
    const int beg = min(tid * seg, nbins);
    const int end = min(beg + seg, nbins);
    int sum = 0;
    for (int t = beg; t < end; ++t) sum += (toff[t + 1] - toff[t] + sub - 1) / sub;
    int total;
    int run = block_scan_1024(sum, wsum, total);
    for (int t = beg; t < end; ++t) {
        for (int q = toff[t]; q < toff[t + 1]; q += sub) {
            subs[2 * run] = t;
            subs[2 * run + 1] = q;
            ++run;
        }
    }
    if (tid == 0) *nsub = total;
}

// Bins x chunks matrices up to this many counts are scanned by one workgroup
// through LDS (48 KiB); larger ones by the three-phase scan below.
#define KBN_SCAN_SMALL 12288
#define KBN_SCAN_COUNTS ((int64_t)1 << 20)  // a larger matrix only where 4096 samples per chunk need it

// One workgroup: exclusive scan of the S bin-major counts in place
// (counts[b * nchunks + c] becomes the first output position of chunk c's
// samples of bin b), the bin offsets toff[0..nbins] and the gather
// subproblem list.  The counts are loaded and stored coalesced; each thread
// scans a contiguous run of them in LDS.
__global__ void __launch_bounds__(1024)
k_scan_small(int S, int nchunks, int nbins, int sub, int *__restrict__ counts, int *__restrict__ toff,
             int *__restrict__ subs, int *__restrict__ nsub) {
    __shared__ int buf[KBN_SCAN_SMALL];
    __shared__ int wsum[16];
    const int tid = threadIdx.x;
#pragma unroll 4
    for (int i = tid; i < S; i += 1024) buf[i] = counts[i];
    __syncthreads();
    const int per = (S + 1023) / 1024;
    const int beg = min(tid * per, S), end = min(beg + per, S);
    int sum = 0;
    for (int i = beg; i < end; ++i) sum += buf[i];
    int total;
    int run = block_scan_1024(sum, wsum, total);
    for (int i = beg; i < end; ++i) {
        const int v = buf[i];
        buf[i] = run;
        if (i % nchunks == 0) toff[i / nchunks] = run;
        run += v;
    }
    if (S == 0)
        for (int b = tid; b < nbins; b += 1024) toff[b] = 0;
    if (tid == 0) toff[nbins] = total;
    __syncthreads();
#pragma unroll 4
    for (int i = tid; i < S; i += 1024) counts[i] = buf[i];
    subproblems_block(nbins, sub, toff, subs, nsub, wsum);
}

// Three-phase scan of larger count matrices over spans of KBN_SCAN_SPAN
// counts: span sums, an exclusive scan of the span sums (one workgroup),
// then each span rescanned with its offset.  Integer sums, so the order of
// additions does not matter.
#define KBN_SCAN_SPAN 8192

__global__ void __launch_bounds__(1024)
k_scan_sums(int64_t S, const int *__restrict__ counts, int *__restrict__ bsum) {
    __shared__ int wsum[16];
    const int64_t base = (int64_t)blockIdx.x * KBN_SCAN_SPAN;
    int acc = 0;
    for (int k = 0; k < KBN_SCAN_SPAN / 1024; ++k) {
        const int64_t i = base + (int64_t)k * 1024 + threadIdx.x;
        acc += i < S ? counts[i] : 0;
    }
    int tot;
    (void)block_scan_1024(acc, wsum, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// exclusive scan of nb span sums in place; bsum[nb] = total
__global__ void __launch_bounds__(1024) k_scan_top(int nb, int *__restrict__ bsum) {
    __shared__ int wsum[16];
    int run = 0;
    for (int base = 0; base < nb; base += 1024) {
        const int i = base + (int)threadIdx.x;
        const int v = i < nb ? bsum[i] : 0;
        int tot;
        const int ex = block_scan_1024(v, wsum, tot);
        if (i < nb) bsum[i] = run + ex;
        run += tot;
    }
    if (threadIdx.x == 0) bsum[nb] = run;
}

__global__ void __launch_bounds__(1024)
k_scan_apply(int64_t S, int *__restrict__ counts, const int *__restrict__ bsum) {
    __shared__ int wsum[16];
    const int64_t base = (int64_t)blockIdx.x * KBN_SCAN_SPAN;
    int run = bsum[blockIdx.x];
    for (int k = 0; k < KBN_SCAN_SPAN / 1024; ++k) {
        const int64_t i = base + (int64_t)k * 1024 + threadIdx.x;
        const int v = i < S ? counts[i] : 0;
        int tot;
        const int ex = block_scan_1024(v, wsum, tot);
        if (i < S) counts[i] = run + ex;
        run += tot;
    }
}

__global__ void __launch_bounds__(256)
k_scan_offsets(int64_t S, int nchunks, int nbins, const int *__restrict__ counts,
               const int *__restrict__ bsum, int nb, int *__restrict__ toff) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b < nbins) toff[b] = S > 0 ? counts[(int64_t)b * nchunks] : 0;
    if (b == 0) toff[nbins] = S > 0 ? bsum[nb] : 0;
}

__global__ void __launch_bounds__(1024)
k_subproblems(int nbins, int sub, const int *__restrict__ toff, int *__restrict__ subs, int *__restrict__ nsub) {
    __shared__ int wsum[16];
    subproblems_block(nbins, sub, toff, subs, nsub, wsum);
}

__global__ void __launch_bounds__(256) k_zero_ints(int *__restrict__ p, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = 0;
}

// One wavefront per chunk: stable scatter.  Lanes with equal tile ids are
// grouped with ballots; rank = number of equal lanes below, so within a
// chunk the input order is kept, and chunks occupy consecutive ranges.
// The workgroups also clear zero[0..nzero).
template <int D>
__global__ void __launch_bounds__(64)
k_tile_scatter(int64_t M, int chunk, int nchunks, int nbins, int nbits,
               const int *__restrict__ tile, const int *__restrict__ counts,
               const int *__restrict__ cell_tmp, const float *__restrict__ frac_tmp,
               int *__restrict__ order, int *__restrict__ cell, float *__restrict__ frac,
               int *__restrict__ zero, int nzero) {
    extern __shared__ int cursor[];
    const int ch = blockIdx.x;
    const int lane = threadIdx.x;
    // clear the owner-tile counters for the next kernels
    for (int i = ch * 64 + lane; i < nzero; i += nchunks * 64) zero[i] = 0;
#pragma unroll 8
    for (int i = lane; i < nbins; i += 64) cursor[i] = counts[(int64_t)i * nchunks + ch];
    __syncthreads();
    const int64_t beg = (int64_t)ch * chunk;
    const int64_t end = beg + chunk < M ? beg + chunk : M;
    const unsigned long long below = (1ull << lane) - 1ull;
    // steps of 64 samples in batches: every load of a batch is issued before
    // its first ranking step, so only LDS work and stores remain in the steps
    constexpr int NB = 12;
    for (int64_t b0 = beg; b0 < end; b0 += 64 * NB) {
        int tv[NB], cv[NB][D];
        float fv[NB][D];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int64_t m = b0 + 64 * k + lane;
            const bool in = m < end;
            tv[k] = in ? tile[m] : -1;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                cv[k][d] = in ? cell_tmp[d * M + m] : 0;
                fv[k][d] = in ? frac_tmp[d * M + m] : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (b0 + 64 * k >= end) break;
            const int64_t m = b0 + 64 * k + lane;
            const bool valid = m < end;
            const int t = tv[k];
            unsigned long long peers = ~0ull;
            for (int bit = 0; bit <= nbits; ++bit) {
                const bool on = (t >> bit) & 1;
                const unsigned long long bal = __ballot(on);
                peers &= on ? bal : ~bal;
            }
            const int rank = __popcll(peers & below);
            const int cnt = __popcll(peers);
            int pos = 0;
            if (valid) pos = cursor[t] + rank;
            // the workgroup is one wavefront: its LDS accesses complete in
            // program order, so the cursor update needs no workgroup barrier
            // (which would also wait for the global stores)
            __builtin_amdgcn_wave_barrier();
            if (valid && rank == 0) cursor[t] = pos + cnt;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
            if (valid) {
                order[pos] = (int)m;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    cell[d * M + pos] = cv[k][d];
                    frac[d * M + pos] = fv[k][d];
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Owner-tile lists for the spread.  A finite sample whose J taps along axis
// d start at grid cell s_d (modulo K_d) reaches owner tile t when its tap
// interval meets t's cell range on every axis.  Each owner tile collects its
// samples by looking only at the sort tiles whose cells can reach it (the
// samples are already sorted by tile): the cells [lo - HI, hi + LO] around
// its range, taps of a sample in cell c lying in [c - LO, c + HI].  Entries
// of a tile are ordered by candidate sort tile, then by sorted position, so
// the spread's accumulation order is fixed.  Every entry gets its record:
// sorted position, the sample's caller-order index, the tap origin relative
// to the tile's first cell (mod K) and the window fraction per axis.
struct OwnerGeom {
    int D, J, LO, HI;
    int ntiles_sort, ntiles_own;
    int K[3], nto[3], T[3], nt[3];
};

#define KBN_OWN_BLOCK 256
#define KBN_OWN_ILP 4    // candidate positions per thread and step
#define KBN_OWN_MAXC 64  // candidate sort tiles staged per round (one wavefront)
#define KBN_OWN_ALONE 4  // lanes without a partner after which a wavefront's counts are no longer merged
#define KBN_OWN_LDS 12288  // owner tiles that k_owner_finish keeps in LDS (3 ints each, 144 KiB)

// Cell range [lo, hi] of owner tile t and, per axis, the first candidate
// sort tile and their count (walked as (first + i) mod nt).
template <int D>
__device__ __forceinline__ void owner_span(const OwnerGeom &o, int t, int lo[3], int hi[3], int first[3],
                                           int num[3]) {
    int rem = t;
#pragma unroll
    for (int d = D - 1; d >= 0; --d) {
        const int a = rem % o.nto[d];
        rem /= o.nto[d];
        lo[d] = own_lo(a, o.K[d], o.nto[d]);
        hi[d] = own_lo(a + 1, o.K[d], o.nto[d]) - 1;
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int K = o.K[d], T = o.T[d], nt = o.nt[d];
        const int L = hi[d] - lo[d] + 1 + o.LO + o.HI;
        int c0 = lo[d] - o.HI;
        if (c0 < 0) c0 += K;
        first[d] = 0;
        num[d] = nt;
        if (L >= K) continue;
        const int f = c0 / T, c1 = c0 + L - 1;
        if (c1 < K) {
            first[d] = f;
            num[d] = c1 / T - f + 1;
        } else {
            const int e = (c1 - K) / T;  // last tile of the part past the wrap
            if (e < f) {
                first[d] = f;
                num[d] = nt - f + e + 1;
            }
        }
    }
}

template <int D>
__device__ __forceinline__ int owner_candidate(const OwnerGeom &o, const int first[3], const int num[3], int k) {
    int sel[3] = {0, 0, 0};
#pragma unroll
    for (int d = D - 1; d >= 0; --d) {
        sel[d] = k % num[d];
        k /= num[d];
    }
    int st = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        int i = first[d] + sel[d];
        if (i >= o.nt[d]) i -= o.nt[d];
        st = st * o.nt[d] + i;
    }
    return st;
}

// Does the sample at sorted position p reach the owner tile with cell
// ranges [lo, hi]?  On success also the tap origin relative to lo (mod K)
// and the window fraction per axis.
template <int D>
__device__ __forceinline__ bool owner_touch(const OwnerGeom &o, int p, int64_t M, const int *__restrict__ cell,
                                            const float *__restrict__ frac, const int lo[3], const int hi[3],
                                            int rel[3], float fr[3]) {
    bool hit = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        int s;
        float f;
        tap_origin(o.J, cell[d * M + p], frac[d * M + p], s, f);
        const int K = o.K[d];
        const int sw = s < 0 ? s + K : s;
        int a = lo[d] - sw;  // (lo - s) mod K: lo inside the taps when <= J - 1
        if (a < 0) a += K;
        int b = sw - lo[d];  // (s - lo) mod K: s inside the tile when <= hi - lo
        if (b < 0) b += K;
        hit = hit && (a <= o.J - 1 || b <= hi[d] - lo[d]);
        rel[d] = b;
        fr[d] = f;
    }
    return hit;
}

// Threads that walk one owner tile's candidates: a workgroup of four
// wavefronts (W = 4), or one wavefront (W = 1), whose LDS accesses complete in
// program order.
template <int W>
__device__ __forceinline__ void walk_sync() {
    if constexpr (W == 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
    } else {
        lds_barrier();
    }
}

// The first wavefront stages up to KBN_OWN_MAXC candidate sort tiles: their first
// sorted position and the exclusive prefix of their sizes (coff[nk] = total).
template <int D>
__device__ __forceinline__ void owner_stage(const OwnerGeom &o, const int first[3], const int num[3], int k0,
                                            int nk, const int *__restrict__ toff, int *cbeg, int *coff, int k) {
    int b = 0, n = 0;
    if (k < nk) {
        const int st = owner_candidate<D>(o, first, num, k0 + k);
        b = toff[st];
        n = toff[st + 1] - b;
    }
    int inc = n;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(inc, off, 64);
        if (k >= off) inc += y;
    }
    if (k < nk) {
        cbeg[k] = b;
        coff[k] = inc - n;
    }
    if (k == nk - 1) coff[nk] = inc;
}

__device__ __forceinline__ int owner_find(const int *coff, int nk, int i) {  // last k with coff[k] <= i
    int lo = 0, hi = nk - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (coff[mid] <= i) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Exclusive scan over the threads of one walk (total to all).
template <int W>
__device__ __forceinline__ int walk_scan(int x, int *wsum, int &total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int inc = x;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if constexpr (W == 1) {
        total = __shfl(inc, 63, 64);
        return inc - x;
    }
    if (lane == 63) wsum[wid] = inc;
    lds_barrier();
    int wpre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int ws = wsum[w];
        if (w < wid) wpre += ws;
        tot += ws;
    }
    lds_barrier();
    total = tot;
    return wpre + inc - x;
}

// The candidate walk of owner tile t: each step hands a thread KBN_OWN_ILP
// consecutive walk positions (all loads issued before the tests), and the
// caller folds the hits in walk order.
template <int D, int W, class F>
__device__ __forceinline__ void owner_walk(const OwnerGeom &o, int t, int64_t M, const int *__restrict__ cell,
                                           const float *__restrict__ frac, const int *__restrict__ toff,
                                           int *cbeg, int *coff, F &&fold) {
    const int tid = threadIdx.x & (64 * W - 1);
    int lo[3], hi[3], first[3], num[3];
    owner_span<D>(o, t, lo, hi, first, num);
    int ncand = 1;
#pragma unroll
    for (int d = 0; d < D; ++d) ncand *= num[d];
    for (int k0 = 0; k0 < ncand; k0 += KBN_OWN_MAXC) {
        const int nk = min(KBN_OWN_MAXC, ncand - k0);
        walk_sync<W>();
        if (tid < 64) owner_stage<D>(o, first, num, k0, nk, toff, cbeg, coff, tid);
        walk_sync<W>();
        const int tot = coff[nk];
        for (int i0 = 0; i0 < tot; i0 += 64 * W * KBN_OWN_ILP) {
            int p[KBN_OWN_ILP], rel[KBN_OWN_ILP][3];
            float fr[KBN_OWN_ILP][3];
            bool hit[KBN_OWN_ILP];
#pragma unroll
            for (int u = 0; u < KBN_OWN_ILP; ++u) {
                const int i = i0 + tid * KBN_OWN_ILP + u;
                const bool in = i < tot;
                const int k = owner_find(coff, nk, in ? i : 0);
                p[u] = in ? cbeg[k] + i - coff[k] : -1;
            }
#pragma unroll
            for (int u = 0; u < KBN_OWN_ILP; ++u)
                hit[u] = p[u] >= 0 && owner_touch<D>(o, p[u] < 0 ? 0 : p[u], M, cell, frac, lo, hi, rel[u], fr[u]);
            fold(p, hit, rel, fr);
        }
    }
}

// Entry count of every owner tile, pushed from the samples: a finite sample
// reaches, per axis, the owner tile holding its first tap and, when its J
// taps cross into the next tile (modulo K), that one too (owner tiles are at
// least J - 1 wide, so these are exactly the tiles whose cells its taps meet,
// the relation k_owner_write tests).  Lanes of a wavefront that reach the same
// tile add with one atomic, until KBN_OWN_ALONE lanes turned out to be alone;
// the rest then add by themselves (where samples are few, merging took a step per
// lane: 29 x 37 x 29, 156 samples 48 us, now 6; where they are many, more
// atomics cost more: 96^3, 1M samples 78 us, 155 with at most four merged
// tiles).  Integer counts do not depend on the order.
template <int D>
__global__ void __launch_bounds__(KBN_BLOCK)
k_owner_count(OwnerGeom o, int64_t M, const int *__restrict__ cell, const float *__restrict__ frac,
              const int *__restrict__ toff, int *__restrict__ ocount) {
    const int64_t p = (int64_t)blockIdx.x * KBN_BLOCK + threadIdx.x;
    const bool act = p < toff[o.ntiles_sort];
    const int lane = threadIdx.x & 63;
    int first[3] = {0, 0, 0}, second[3] = {0, 0, 0}, num[3] = {1, 1, 1};
    if (act) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            int st;
            float f;
            tap_origin(o.J, cell[d * M + p], frac[d * M + p], st, f);
            const int K = o.K[d];
            const int sw = st < 0 ? st + K : st;
            int se = sw + o.J - 1;
            if (se >= K) se -= K;
            first[d] = own_tile(sw, K, o.nto[d]);
            second[d] = own_tile(se, K, o.nto[d]);
            num[d] = first[d] == second[d] ? 1 : 2;
        }
    }
#pragma unroll
    for (int k = 0; k < (1 << D); ++k) {
        bool on = act;
        int id = 0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int bit = (k >> (D - 1 - d)) & 1;
            on = on && bit < num[d];
            id = id * o.nto[d] + (bit ? second[d] : first[d]);
        }
        unsigned long long todo = __ballot(on);
        int alone = 0;
        while (todo && alone < KBN_OWN_ALONE) {
            const int leader = __ffsll((long long)todo) - 1;
            const int key = __shfl(id, leader, 64);
            const unsigned long long same = __ballot(on && id == key) & todo;
            if (lane == leader) atomicAdd(&ocount[key], __popcll(same));
            todo &= ~same;
            alone += __popcll(same) == 1 ? 1 : 0;
        }
        if ((todo >> lane) & 1ull) atomicAdd(&ocount[id], 1);
    }
}

// The reaching samples of tile t's candidate walk, compacted in walk order from
// entry `run` on, with their records.
template <int D, int W>
__device__ __forceinline__ void owner_write_tile(const OwnerGeom &o, int t, int run, int64_t M,
                                                 const int *__restrict__ cell, const float *__restrict__ frac,
                                                 const int *__restrict__ toff, const int *__restrict__ order,
                                                 int *__restrict__ rec_p, int *__restrict__ rec_q,
                                                 int2 *__restrict__ rec_t, int *cbeg, int *coff, int *wsum) {
    owner_walk<D, W>(o, t, M, cell, frac, toff, cbeg, coff,
                     [&](const int *p, const bool *hit, int (*rel)[3], float (*fr)[3]) {
                         int h = 0;
#pragma unroll
                         for (int u = 0; u < KBN_OWN_ILP; ++u) h += hit[u] ? 1 : 0;
                         int total;
                         int e = run + walk_scan<W>(h, wsum, total);
#pragma unroll
                         for (int u = 0; u < KBN_OWN_ILP; ++u) {
                             if (!hit[u]) continue;
                             rec_p[e] = p[u];
                             rec_q[e] = order[p[u]];
#pragma unroll
                             for (int d = 0; d < D; ++d)
                                 rec_t[(int64_t)e * D + d] = make_int2(rel[u][d], __float_as_int(fr[u][d]));
                             ++e;
                         }
                         run += total;
                     });
}

// Entries and their records of every owner tile, the tiles with most entries
// first: workgroups 0 .. hot - 1 take one tile of more than `few` entries each, the
// others four tiles of fewer, one per wavefront.  Bound by the chain of loads of
// a walk, so by the walks in flight: with a workgroup for each of the 262144 tiles
// of 256^3 50000 samples took 1060 us of an index pass of 1280, which is 450 now,
// and 3M samples 1670 of 2930 (2610).
template <int D>
__global__ void __launch_bounds__(KBN_OWN_BLOCK)
k_owner_write(OwnerGeom o, int hot, int few, int64_t M, const int *__restrict__ cell, const float *__restrict__ frac,
              const int *__restrict__ toff, const int *__restrict__ order, const int *__restrict__ ooff,
              const int *__restrict__ otile_order, int *__restrict__ rec_p, int *__restrict__ rec_q,
              int2 *__restrict__ rec_t) {
    constexpr int W = KBN_OWN_BLOCK / 64;
    __shared__ int cbeg[W][KBN_OWN_MAXC], coff[W][KBN_OWN_MAXC + 1];
    __shared__ int wsum[W];
    if ((int)blockIdx.x < hot) {
        const int t = otile_order[blockIdx.x];
        const int run = ooff[t];
        if (ooff[t + 1] - run <= few) return;
        owner_write_tile<D, W>(o, t, run, M, cell, frac, toff, order, rec_p, rec_q, rec_t, cbeg[0], coff[0], wsum);
    } else {
        const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int k = ((int)blockIdx.x - hot) * W + w;
        if (k >= o.ntiles_own) return;
        const int t = otile_order[k];
        const int run = ooff[t], n = ooff[t + 1] - run;
        if (n == 0 || n > few) return;
        owner_write_tile<D, 1>(o, t, run, M, cell, frac, toff, order, rec_p, rec_q, rec_t, cbeg[w], coff[w], wsum);
    }
}

// Order of the tiles: bins (2^k, 2^(k+1)] of their entry count, larger first, so
// that a bin holds either split tiles or unsplit ones (the entries per work item
// are a power of two).
#define KBN_OWN_KEYS 34
__device__ __forceinline__ int owner_key(int c) { return c == 0 ? 33 : (c == 1 ? 32 : __clz(c - 1)); }

// atomicAdd(&ctr[key], 1) for the active lanes of a wavefront, one LDS
// atomic per distinct key (lanes with equal keys get consecutive values in
// lane order); returns the lane's value.
__device__ __forceinline__ int wave_key_add(int *ctr, int key, bool active) {
    const int lane = threadIdx.x & 63;
    unsigned long long todo = __ballot(active);
    int mine = 0;
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int k = __shfl(key, leader, 64);
        const unsigned long long same = __ballot(active && key == k) & todo;
        int base = 0;
        if (lane == leader) base = atomicAdd(&ctr[k], __popcll(same));
        base = __shfl(base, leader, 64);
        if ((same >> lane) & 1ull) mine = base + __popcll(same & ((1ull << lane) - 1ull));
        todo &= ~same;
    }
    return mine;
}

// Exclusive scans of three values over a 1024-thread workgroup at once.
__device__ __forceinline__ void block_scan3_1024(int x[3], int ex[3], int tot[3], int (*wsum)[16]) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int inc[3] = {x[0], x[1], x[2]};
    for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int y = __shfl_up(inc[j], o, 64);
            if (lane >= o) inc[j] += y;
        }
    }
    if (lane == 63)
        for (int j = 0; j < 3; ++j) wsum[j][wid] = inc[j];
    lds_barrier();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        int wpre = 0, t = 0;
        for (int w = 0; w < 16; ++w) {
            const int ws = wsum[j][w];
            if (w < wid) wpre += ws;
            t += ws;
        }
        ex[j] = wpre + inc[j] - x[j];
        tot[j] = t;
    }
    lds_barrier();
}

// Whether the caller's samples come along a trajectory: of up to 1024 neighbours in
// the sorted order, at least half follow each other in the caller's.  order_step is
// this thread's pair (its loads are in flight until order_vote, which adds +1 or -1 for
// it to *votes in LDS: cleared, and read, behind barriers of the caller).
__device__ __forceinline__ int order_step(const int *__restrict__ order, int64_t M) {
    const int64_t p = (int64_t)threadIdx.x * (M > 1024 ? (M - 1) / 1024 : 1);
    return p + 1 < M ? order[p + 1] - order[p] : 0;
}
__device__ __forceinline__ void order_vote(int step, int *votes) {
    const int yes = __popcll(__ballot(step == 1)), no = __popcll(__ballot(step != 0 && step != 1));
    if ((threadIdx.x & 63) == 0) atomicAdd(votes, yes - no);
}

// Owner offsets (exclusive scan of the counts, ooff[n] = total), the tiles in
// decreasing order of entry count, and the spread work items; up to KBN_OWN_LDS
// tiles in one workgroup, whose counts, offsets and order live in LDS (3 ntiles
// ints) and are written out at the end.
//
// Order: bins of log2 count, so the spread dispatches its longest
// workgroups first.  The order inside a bin is arbitrary; tiles are
// independent and a split tile's partial slots are consecutive and summed in
// item order, so results do not depend on it.
//
// Work items: tile t (hottest first) with n entries becomes ceil(n / seg)
// items of at most seg entries (one item if n == 0, so that every tile is
// written).  Tiles with several items get consecutive partial slots; seg
// doubles until the slots fit in `smax`.  Outputs:
//   work[i] = (tile, first entry, end entry, slot or -1), counts2[0] = items
//   comb[k] = (tile, first slot, number of slots),     counts2[1] = tiles
//   counts2[2] = 1 if the samples (their order sorder) come along a trajectory
__global__ void __launch_bounds__(1024)
k_owner_finish(int ntiles, int seg, int smax, int64_t M, const int *__restrict__ sorder,
               const int *__restrict__ ocount, int *__restrict__ ooff, int *__restrict__ order,
               int *__restrict__ work, int *__restrict__ comb, int *__restrict__ counts2) {
    extern __shared__ int lds[];
    __shared__ int wsum[16];
    __shared__ int wsum3[3][16];
    __shared__ int hist[KBN_OWN_KEYS], start[KBN_OWN_KEYS], votes;
    const int tid = threadIdx.x;
    const int nr = (ntiles + 1023) / 1024;
    int *off = lds + ntiles, *ord = lds + 2 * ntiles;
    const int step = order_step(sorder, M);
#pragma unroll 4
    for (int t = tid; t < ntiles; t += 1024) lds[t] = ocount[t];
    if (tid == 0) votes = 0;
    lds_barrier();
    order_vote(step, &votes);
    const int *cnt = lds;
    // offsets
    int carry = 0;
    for (int r = 0; r < nr; ++r) {
        const int t = r * 1024 + tid;
        int total;
        const int ex = block_scan_1024(t < ntiles ? cnt[t] : 0, wsum, total);
        if (t < ntiles) off[t] = carry + ex;
        carry += total;
    }
    if (tid == 0) ooff[ntiles] = carry;
    // hottest-first order
    if (tid < KBN_OWN_KEYS) hist[tid] = 0;
    lds_barrier();
    for (int t0 = 0; t0 < ntiles; t0 += 1024) {
        const int t = t0 + tid;
        (void)wave_key_add(hist, t < ntiles ? owner_key(cnt[t]) : 0, t < ntiles);
    }
    lds_barrier();
    if (tid == 0) {
        int acc = 0;
        for (int k = 0; k < KBN_OWN_KEYS; ++k) {
            start[k] = acc;
            acc += hist[k];
        }
    }
    lds_barrier();
    for (int t0 = 0; t0 < ntiles; t0 += 1024) {
        const int t = t0 + tid;
        const int q = wave_key_add(start, owner_key(t < ntiles ? cnt[t] : 0), t < ntiles);
        if (t < ntiles) ord[q] = t;
    }
    // entries per work item: double seg until the split tiles' slots fit
    int sg = seg;
    for (int it = 0; it < 31; ++it) {
        int sl = 0;
        for (int t = tid; t < ntiles; t += 1024) {
            const int c = cnt[t];
            if (c > sg) sl += (c + sg - 1) / sg;
        }
        int total;
        (void)block_scan_1024(sl, wsum, total);
        if (total <= smax) break;
        sg *= 2;
    }
    lds_barrier();
    // positions in rounds: prefixes of items, slots and split tiles, and the
    // position's items written at once
    int cw = 0, cs = 0, cc = 0;
    for (int r = 0; r < nr; ++r) {
        const int q = r * 1024 + tid;
        const bool in = q < ntiles;
        const int t = in ? ord[q] : 0;
        const int c = in ? cnt[t] : 0;
        const int ns = in ? (c > sg ? (c + sg - 1) / sg : 1) : 0;
        int x[3] = {ns, ns > 1 ? ns : 0, ns > 1 ? 1 : 0}, ex[3], tot[3];
        block_scan3_1024(x, ex, tot, wsum3);
        if (in) {
            const int e0 = off[t];
            const int wi = cw + ex[0], si = cs + ex[1];
            for (int k = 0; k < ns; ++k) {
                int *w = work + 4 * (wi + k);
                w[0] = t;
                w[1] = e0 + k * sg;
                w[2] = min(e0 + (k + 1) * sg, e0 + c);
                w[3] = ns > 1 ? si + k : -1;
            }
            if (ns > 1) {
                int *cb = comb + 3 * (cc + ex[2]);
                cb[0] = t;
                cb[1] = si;
                cb[2] = ns;
            }
        }
        cw += tot[0];
        cs += tot[1];
        cc += tot[2];
    }
    if (tid == 0) {
        counts2[0] = cw;
        counts2[1] = cc;
        counts2[2] = votes >= 0;
    }
#pragma unroll 4
    for (int t = tid; t < ntiles; t += 1024) {
        ooff[t] = off[t];
        order[t] = ord[t];
    }
}

// The same for more tiles, in spans of KBN_FIN_SPAN tiles: sums per span, one
// workgroup that turns them into starting positions, and the spans again with
// those.  The split tiles come first in the order (owner_key), so an unsplit
// tile's item follows from its position, and the few split ones (at most half of
// the partial slots) take their slots, items and combine entries from counters,
// in any order.  One workgroup over all tiles took a round trip to memory per
// thousand of them and phase: 105 us at 13824 tiles, 490 at 110592, 1130 at 262144.
#define KBN_FIN_SPAN 4096
#define KBN_FIN_LEVELS 24  // entries per work item: seg 2^level, up to 2^30
struct FinScratch {        // [nb] or [keys][nb], [levels][nb]
    int *head;             // log2 of the entries per item, split tiles, their slots, two counters
    int *sum, *hist, *slots;
};
__host__ __device__ inline int fin_spans(int ntiles) { return (ntiles + KBN_FIN_SPAN - 1) / KBN_FIN_SPAN; }
__host__ __device__ inline FinScratch fin_scratch(int *p, int nb) {
    return FinScratch{p, p + 8, p + 8 + nb, p + 8 + nb * (1 + KBN_OWN_KEYS)};
}
inline int64_t fin_ints(int ntiles) {
    return ntiles <= KBN_OWN_LDS ? 0 : 8 + (int64_t)fin_spans(ntiles) * (1 + KBN_OWN_KEYS + KBN_FIN_LEVELS);
}

__global__ void __launch_bounds__(1024)
k_owner_spans(int ntiles, int nb, int seg_log, const int *__restrict__ ocount, int *__restrict__ scratch) {
    __shared__ int wsum[16], hist[KBN_OWN_KEYS], slots[KBN_FIN_LEVELS];
    const int tid = threadIdx.x;
    const FinScratch f = fin_scratch(scratch, nb);
    if (tid < KBN_OWN_KEYS) hist[tid] = 0;
    if (tid < KBN_FIN_LEVELS) slots[tid] = 0;
    int c[KBN_FIN_SPAN / 1024], sum = 0;
#pragma unroll
    for (int u = 0; u < KBN_FIN_SPAN / 1024; ++u) {
        const int t = (int)blockIdx.x * KBN_FIN_SPAN + u * 1024 + tid;
        c[u] = t < ntiles ? ocount[t] : -1;
        sum += max(c[u], 0);
    }
    int total;
    (void)block_scan_1024(sum, wsum, total);  // (its barriers order the cleared LDS too)
#pragma unroll
    for (int u = 0; u < KBN_FIN_SPAN / 1024; ++u) {
        (void)wave_key_add(hist, c[u] >= 0 ? owner_key(c[u]) : 0, c[u] >= 0);
        for (int l = 0; l < KBN_FIN_LEVELS && c[u] > 0 && ((c[u] - 1) >> (seg_log + l)) > 0; ++l)
            atomicAdd(&slots[l], ((c[u] - 1) >> (seg_log + l)) + 1);
    }
    lds_barrier();
    if (tid == 0) f.sum[blockIdx.x] = total;
    if (tid < KBN_OWN_KEYS) f.hist[tid * nb + blockIdx.x] = hist[tid];
    if (tid < KBN_FIN_LEVELS) f.slots[tid * nb + blockIdx.x] = slots[tid];
}

__global__ void __launch_bounds__(1024)
k_owner_top(int ntiles, int nb, int seg_log, int smax, int64_t M, const int *__restrict__ sorder,
            int *__restrict__ scratch, int *__restrict__ ooff, int *__restrict__ counts2) {
    __shared__ int wsum[16], lslots[KBN_FIN_LEVELS], votes;
    const int tid = threadIdx.x;
    const FinScratch f = fin_scratch(scratch, nb);
    const int step = order_step(sorder, M);
    if (tid == 0) votes = 0;
    int run = 0, tot;
    for (int b0 = 0; b0 < nb; b0 += 1024) {
        const int v = b0 + tid < nb ? f.sum[b0 + tid] : 0;
        const int ex = block_scan_1024(v, wsum, tot);
        if (b0 + tid < nb) f.sum[b0 + tid] = run + ex;
        run += tot;
    }
    if (tid == 0) ooff[ntiles] = run;
    order_vote(step, &votes);  // (behind the scan's barriers; read behind the next ones)
    for (int l = tid >> 6; l < KBN_FIN_LEVELS; l += 16) {  // one wavefront per level
        int s = 0;
        for (int b = tid & 63; b < nb; b += 64) s += f.slots[l * nb + b];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
        if ((tid & 63) == 0) lslots[l] = s;
    }
    lds_barrier();
    int level = 0;
    while (level < KBN_FIN_LEVELS - 1 && lslots[level] > smax) ++level;
    const int first = __clz(1 << (seg_log + level)) + 1;  // the first key of unsplit tiles
    run = 0;
    for (int i0 = 0; i0 < KBN_OWN_KEYS * nb; i0 += 1024) {
        const int i = i0 + tid;
        const int v = i < KBN_OWN_KEYS * nb ? f.hist[i] : 0;
        const int ex = block_scan_1024(v, wsum, tot);
        if (i < KBN_OWN_KEYS * nb) f.hist[i] = run + ex;
        if (i == first * nb) {
            const int split = run + ex;
            f.head[0] = seg_log + level;
            f.head[1] = split;
            f.head[2] = lslots[level];
            f.head[3] = 0;
            f.head[4] = 0;
            counts2[0] = lslots[level] + ntiles - split;
            counts2[1] = split;
            counts2[2] = votes >= 0;
        }
        run += tot;
    }
}

__global__ void __launch_bounds__(1024)
k_owner_place(int ntiles, int nb, const int *__restrict__ ocount, int *__restrict__ scratch, int *__restrict__ ooff,
              int *__restrict__ order, int *__restrict__ work, int *__restrict__ comb) {
    __shared__ int wsum[16], start[KBN_OWN_KEYS];
    const int tid = threadIdx.x;
    const FinScratch f = fin_scratch(scratch, nb);
    if (tid < KBN_OWN_KEYS) start[tid] = f.hist[tid * nb + blockIdx.x];
    const int seg_log = f.head[0], split = f.head[1], slots = f.head[2];
    int run = f.sum[blockIdx.x];
#pragma unroll
    for (int u = 0; u < KBN_FIN_SPAN / 1024; ++u) {
        const int t = (int)blockIdx.x * KBN_FIN_SPAN + u * 1024 + tid;
        const bool in = t < ntiles;
        const int c = in ? ocount[t] : 0;
        int tot;
        const int e0 = run + block_scan_1024(c, wsum, tot);
        run += tot;
        const int q = wave_key_add(start, owner_key(c), in);
        if (!in) continue;
        ooff[t] = e0;
        order[q] = t;
        const int ns = c > 0 ? ((c - 1) >> seg_log) + 1 : 1;
        if (ns == 1) {
            int *w = work + 4 * ((int64_t)slots + q - split);
            w[0] = t;
            w[1] = e0;
            w[2] = e0 + c;
            w[3] = -1;
            continue;
        }
        const int si = atomicAdd(&f.head[3], ns), k = atomicAdd(&f.head[4], 1);
        for (int j = 0; j < ns; ++j) {
            int *w = work + 4 * (si + j);
            w[0] = t;
            w[1] = e0 + (j << seg_log);
            w[2] = j + 1 < ns ? e0 + ((j + 1) << seg_log) : e0 + c;
            w[3] = si + j;
        }
        comb[3 * k] = t;
        comb[3 * k + 1] = si;
        comb[3 * k + 2] = ns;
    }
}

}  // namespace

// Histograms of more than 16384 bins need more than the default 64 KiB of
// dynamic LDS per workgroup; gfx950 allows up to 160 KiB once a kernel opts in.
hipError_t allow_large_lds(size_t bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    static const hipError_t once = [] {
        const void *ks[] = {(const void *)k_points_hist, (const void *)k_tile_scatter<1>,
                            (const void *)k_tile_scatter<2>, (const void *)k_tile_scatter<3>,
                            (const void *)k_owner_finish};
        hipError_t r = hipSuccess;
        for (const void *k : ks) {
            // the dynamic part may take what the kernel's static LDS leaves
            hipFuncAttributes fa;
            hipError_t e = hipFuncGetAttributes(&fa, k);
            if (e == hipSuccess)
                e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        160 * 1024 - (int)fa.sharedSizeBytes);
            if (e != hipSuccess) r = e;
        }
        return r;
    }();
    return once;
}

namespace {

// Histogram chunks of M > 0 samples: at most 4096 samples per chunk (one
// wavefront ranks a chunk in steps of 64); otherwise as many chunks as keep the
// count matrix within one workgroup's scan, and at least 256 samples per chunk.
// Where 4096 samples already take the multi-workgroup scan, smaller chunks cost
// it little and fill the GPU, until the strided counts of a million entries cost
// more (index pass of 48^3 with 65536 samples 330 -> 264 us, 75 x 90 x 64 with
// 150001 447 -> 391, of it histogram 35 -> 17 and scatter 72 -> 38; 262144
// entries 279 and 433 us; 96^3 with 1M samples has 13825 bins and stays).
// Never fewer for more samples, which the chunks rounded to 64 samples may be.
int64_t most_chunks(int64_t M, int64_t nbins) {
    const int64_t nmin = (M + 4095) / 4096;
    const int64_t nsmall = std::max<int64_t>(1, KBN_SCAN_SMALL / nbins);
    const int64_t n256 = std::max<int64_t>(1, M / 256);
    return nmin <= nsmall ? std::max(nmin, std::min(nsmall, n256))
                          : std::max(nmin, std::min(n256, KBN_SCAN_COUNTS / nbins));
}

}  // namespace

int kbn_points_chunks(int64_t M, int ntiles, int *chunk) {
    if (M <= 0) {
        *chunk = 64;
        return 0;
    }
    const int64_t want = most_chunks(M, (int64_t)ntiles + 1);
    int64_t c = (M + want - 1) / want;
    c = (c + 63) / 64 * 64;
    *chunk = (int)c;
    return (int)((M + c - 1) / c);
}

// The count matrix and the three-phase scan's span sums.  Sized by most_chunks,
// so that the buffers of M samples hold those of every smaller M too.
int64_t kbn_points_owner_base(int64_t M, int ntiles) {
    const int64_t nbins = (int64_t)ntiles + 1;
    const int64_t S = M > 0 ? most_chunks(M, nbins) * nbins : 0;
    return S + S / KBN_SCAN_SPAN + 2;
}

int64_t kbn_points_counts_size(int64_t M, int ntiles, int ntiles_own) {
    // then the owner tiles' entry counts and the spans of k_owner_spans
    return kbn_points_owner_base(M, ntiles) + (int64_t)ntiles_own + 1 + fin_ints(ntiles_own);
}

hipError_t kbn_launch_points(int D, int64_t M, const float *omega, const double *scale,
                             const int *K, const int *T, const int *nt, int ntiles, int ntiles_own,
                             int sub, const KbnPointsBufs &b, hipStream_t s, hipEvent_t omega_read) {
    const int nbins = ntiles + 1;
    int *ocount = b.counts + kbn_points_owner_base(M, ntiles);
    {
        const hipError_t e = allow_large_lds(sizeof(int) * (size_t)nbins);
        if (e != hipSuccess) return e;
    }
    int chunk;
    const int nchunks = kbn_points_chunks(M, ntiles, &chunk);
    if (M > 0)
        k_points_hist<<<dim3(nchunks), dim3(256), sizeof(int) * nbins, s>>>(
            D, M, chunk, nchunks, nbins, omega, scale[0], D > 1 ? scale[1] : 0.0, D > 2 ? scale[2] : 0.0,
            K[0], D > 1 ? K[1] : 1, D > 2 ? K[2] : 1, T[0], D > 1 ? T[1] : 1, D > 2 ? T[2] : 1,
            D > 1 ? nt[1] : 1, D > 2 ? nt[2] : 1, ntiles, b.cell_tmp, b.frac_tmp, b.tile, b.flag, b.counts);
    if (omega_read) {  // omega is not read after this kernel
        const hipError_t e = hipEventRecord(omega_read, s);
        if (e != hipSuccess) return e;
    }
    const int64_t S = (int64_t)nbins * nchunks;
    if (S <= KBN_SCAN_SMALL) {
        k_scan_small<<<dim3(1), dim3(1024), 0, s>>>((int)S, std::max(nchunks, 1), nbins, sub, b.counts, b.toff,
                                                    b.subs, b.nsub);
    } else {
        int *bsum = b.counts + S;
        const int nb = (int)((S + KBN_SCAN_SPAN - 1) / KBN_SCAN_SPAN);
        k_scan_sums<<<dim3(nb), dim3(1024), 0, s>>>(S, b.counts, bsum);
        k_scan_top<<<dim3(1), dim3(1024), 0, s>>>(nb, bsum);
        k_scan_apply<<<dim3(nb), dim3(1024), 0, s>>>(S, b.counts, bsum);
        k_scan_offsets<<<dim3((nbins + 256) / 256), dim3(256), 0, s>>>(S, nchunks, nbins, b.counts, bsum, nb,
                                                                       b.toff);
        k_subproblems<<<dim3(1), dim3(1024), 0, s>>>(nbins, sub, b.toff, b.subs, b.nsub);
    }
    if (M > 0) {
        int nbits = 0;
        while ((1 << nbits) < nbins) ++nbits;
        auto kern = D == 1 ? k_tile_scatter<1> : (D == 2 ? k_tile_scatter<2> : k_tile_scatter<3>);
        kern<<<dim3(nchunks), dim3(64), sizeof(int) * nbins, s>>>(M, chunk, nchunks, nbins, nbits, b.tile,
                                                                  b.counts, b.cell_tmp, b.frac_tmp, b.order,
                                                                  b.cell, b.frac, ocount, ntiles_own);
    } else {
        k_zero_ints<<<dim3((ntiles_own + 255) / 256), dim3(256), 0, s>>>(ocount, ntiles_own);
    }
    return hipGetLastError();
}

hipError_t kbn_launch_owner_lists(const KbnGeom &g, int64_t M, const int *cell, const float *frac,
                                  const int *toff, const int *order, int *ocount, int *ooff,
                                  int *otile_order, int seg, int smax, int *swork, int *scomb, int *scounts,
                                  int *rec_p, int *rec_q, int2 *rec_t, hipStream_t s) {
    OwnerGeom o;
    o.D = g.D;
    o.J = g.J;
    o.LO = (g.J & 1) ? g.J / 2 : g.J / 2 - 1;
    o.HI = (g.J & 1) ? g.J / 2 + 1 : g.J / 2;
    o.ntiles_sort = g.ntiles;
    o.ntiles_own = g.ntiles_own;
    for (int d = 0; d < 3; ++d) {
        o.K[d] = d < g.D ? g.K[d] : 1;
        o.nto[d] = d < g.D ? g.nto[d] : 1;
        o.T[d] = d < g.D ? g.T[d] : 1;
        o.nt[d] = d < g.D ? g.nt[d] : 1;
    }
    const int n = g.ntiles_own;
    int seg_log = 0;
    while ((1 << seg_log) < seg) ++seg_log;  // seg is a power of two
    {
        const hipError_t e = allow_large_lds(3 * sizeof(int) * (size_t)std::min(n, KBN_OWN_LDS));
        if (e != hipSuccess) return e;
    }
    // Entries up to which one wavefront writes a tile: more in 3D, where a tile has
    // fewer candidates per entry (8-cell sort tiles, 32-cell ones in 2D).  With
    // few tiles a workgroup each leaves room (128^2, 1024 tiles, 9000 samples 74 us
    // against 82; 4096 110 and 115; 6400 126 and 118).  A power of two, so that the
    // tiles above it come first (owner_key); there are at most M 2^D / few of them.
    const int few = n <= 4096 ? 0 : (g.D == 3 ? 64 : 16);
    const int hot = (int)std::min<int64_t>(n, few ? (M << g.D) / few : n);
    const int waves = few ? (n + KBN_OWN_BLOCK / 64 - 1) / (KBN_OWN_BLOCK / 64) : 0;
    const dim3 wgrid((unsigned)(hot + waves));
    switch (g.D) {
#define KBN_OWN(d)                                                                                     \
    case d:                                                                                            \
        if (M > 0)                                                                                     \
            k_owner_count<d><<<dim3((unsigned)((M + KBN_BLOCK - 1) / KBN_BLOCK)), dim3(KBN_BLOCK), 0,  \
                               s>>>(o, M, cell, frac, toff, ocount);                                   \
        if (n <= KBN_OWN_LDS) {                                                                        \
            k_owner_finish<<<dim3(1), dim3(1024), 3 * sizeof(int) * n, s>>>(                           \
                n, seg, smax, M, order, ocount, ooff, otile_order, swork, scomb, scounts);             \
        } else {                                                                                       \
            const int nb = fin_spans(n);                                                               \
            int *scratch = ocount + n + 1;                                                             \
            k_owner_spans<<<dim3(nb), dim3(1024), 0, s>>>(n, nb, seg_log, ocount, scratch);            \
            k_owner_top<<<dim3(1), dim3(1024), 0, s>>>(n, nb, seg_log, smax, M, order, scratch, ooff,  \
                                                       scounts);                                       \
            k_owner_place<<<dim3(nb), dim3(1024), 0, s>>>(n, nb, ocount, scratch, ooff, otile_order,   \
                                                          swork, scomb);                               \
        }                                                                                              \
        if (M > 0)                                                                                     \
            k_owner_write<d><<<wgrid, dim3(KBN_OWN_BLOCK), 0, s>>>(o, hot, few, M, cell, frac, toff,   \
                                                                   order, ooff, otile_order, rec_p,    \
                                                                   rec_q, rec_t);                      \
        break;
        KBN_OWN(1) KBN_OWN(2) KBN_OWN(3)
#undef KBN_OWN
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
