// J-tap Kaiser-Bessel interpolation between the oversampled grid and the
// sample locations (appendix: a~_mn = sum_j u_j*(omega_m) s_n
// exp(-i gamma (k_m + j) n)), and its transpose.
//
// Taps: with u = omega K / (2 pi), k_start = floor(u - J/2) + 1 and taps
// k_start + j, j < J, at distances t_j = u - k_start - j in [-J/2, J/2);
// grid indices wrap modulo K.  The window psi(t) = I0(beta sqrt(1 -
// (2t/J)^2)) / I0(beta) is evaluated per tap by a degree-10 polynomial in
// x = 2 f - 1 (f = fractional position of u - J/2), fitted on the host.
//
// gather (type 2, forward operator): one thread per sorted sample, weights
// computed once and reused over all channels of its group.  Mode 1 fuses
// the omega-Jacobian epilogue of eq. (e,jac,Ax,v): for channel (b, c, d) the
// interpolated value z = [A(s_c x_b r^[d])]_m is folded into
// Im{z conj(v_{b,c,m})} and summed over the channels in registers.
//
// spread (type 1, adjoint operator): each workgroup owns one tile of the
// grid for a group of channels and sums every sample whose taps reach the
// tile (see k_spread_mf2), then writes the tile with plain stores: every grid
// cell is written exactly once, so the grid needs neither zero-initialisation
// nor atomics.
#include "kbn_internal.h"
#include "kbn_window.h"

#include <algorithm>
#include <cstdlib>

namespace {

// index in the k-space array of the sample at sorted position p
__device__ __forceinline__ int sample_index(const int *order, int64_t p) { return order ? order[p] : (int)p; }

// Staged gather: one workgroup per subproblem (<= KBN_SUB sorted points of
// one tile).  Channels are taken CP at a time (CP = 2 or 4): their grid
// regions (tile plus the tap reach) are loaded into LDS interleaved, with
// coalesced reads, and every thread interpolates its point for all CP
// channels from LDS, one 16-byte read per tap and channel pair.  With MAXC > 0
// the region of the next CP channels is loaded into registers while the
// current ones are interpolated (at most MAXC cells per thread, whose grid
// offsets are computed once), so the grid reads overlap the interpolation.  Subproblems
// of the extra tile id ntiles hold the flagged points, whose outputs are NaN.
// Body of one workgroup: subproblem s, channel group gy (the kernel's
// blockIdx.x and blockIdx.y), regions staged in reg4.
template <int D, int J, int MODE, int CP, int MAXC>
__device__ __forceinline__ void gather_staged_wg(const KbnGeom &g, const KbnGatherArgs &a, int cg, int s, int gy,
                                                 float4 *reg4) {
    constexpr int H = CP / 2;  // float4 (channel pairs) per region cell
    if (s >= *a.nsub) return;
    const int tile = a.subs[2 * s];
    const int p0 = a.subs[2 * s + 1];
    const int ch0 = gy * cg;
    const int ch1 = min(ch0 + cg, a.nch);
    const float qnan = __builtin_nanf("");
    if (tile == g.ntiles) {  // flagged points
        const int p = p0 + threadIdx.x;
        if (p < a.M) {
            const int q = sample_index(a.order, p);
            if (MODE == 0) {
                for (int ch = ch0; ch < ch1; ++ch) a.y[(int64_t)ch * a.M + q] = make_float2(qnan, qnan);
            } else {
                float *part = a.part + (int64_t)gy * a.M * D;
                for (int d = 0; d < D; ++d) part[(int64_t)q * D + d] = qnan;
            }
        }
        return;
    }
    const int p1 = min(p0 + KBN_SUB, a.toff[tile + 1]);
    int o[D], E[D];
    {
        int rem = tile;
#pragma unroll
        for (int d = D - 1; d >= 0; --d) {
            const int tc = rem % g.nt[d];
            rem /= g.nt[d];
            const int a0 = tc * g.T[d];
            const int te = min(g.T[d], g.K[d] - a0);
            o[d] = a0 - Reach<J>::LO;
            E[d] = te + Reach<J>::LO + Reach<J>::HI;
        }
    }
    int R = 1;
#pragma unroll
    for (int d = 0; d < D; ++d) R *= E[d];

    const int p = p0 + (int)threadIdx.x;
    const bool act = p < p1;
    int q = 0;
    float w[D][J];
    int base = 0;  // region offset of the point's first tap
    if (act) {
        q = sample_index(a.order, p);
        int stride = 1;
#pragma unroll
        for (int d = D - 1; d >= 0; --d) {
            int start;
            float f;
            tap_origin(J, a.cell[d * a.M + p], a.frac[d * a.M + p], start, f);
            kb_weights<J>(f, g.coef, w[d]);
            base += (start - o[d]) * stride;
            stride *= E[d];
        }
    }
    float jac[KBN_MAX_D] = {0.f, 0.f, 0.f};
    // LA: region cells of this thread and their grid offsets (the same for
    // every channel), and the next channel group's region loaded ahead
    constexpr bool LA = MAXC > 0;
    constexpr int NCELL = LA ? MAXC : 1;
    int goff[NCELL];
    float4 pre[NCELL][H];
    auto fetch = [&](int chb) {
        const int nc = min(CP, ch1 - chb);
#pragma unroll
        for (int k = 0; k < NCELL; ++k) {
            const int i = (int)threadIdx.x + k * KBN_BLOCK;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                float2 v0 = make_float2(0.f, 0.f), v1 = v0;
                if (i < R) {
                    if (2 * h < nc) v0 = a.grid[(int64_t)(chb + 2 * h) * a.gsize + goff[k]];
                    if (2 * h + 1 < nc) v1 = a.grid[(int64_t)(chb + 2 * h + 1) * a.gsize + goff[k]];
                }
                pre[k][h] = make_float4(v0.x, v0.y, v1.x, v1.y);
            }
        }
    };
    if constexpr (LA) {
#pragma unroll
        for (int k = 0; k < NCELL; ++k) {
            const int i = (int)threadIdx.x + k * KBN_BLOCK;
            int rem = i < R ? i : 0;
            int gi = 0, gstride = 1;
#pragma unroll
            for (int d = D - 1; d >= 0; --d) {
                const int e = rem % E[d];
                rem /= E[d];
                gi += wrapk(o[d] + e, g.K[d]) * gstride;
                gstride *= g.K[d];
            }
            goff[k] = gi;
        }
        if (ch0 < ch1) fetch(ch0);
    }
    for (int ch = ch0; ch < ch1; ch += CP) {
        const int nc = min(CP, ch1 - ch);
        if constexpr (LA) {
#pragma unroll
            for (int k = 0; k < NCELL; ++k) {
                const int i = (int)threadIdx.x + k * KBN_BLOCK;
                if (i < R) {
#pragma unroll
                    for (int h = 0; h < H; ++h) reg4[i * H + h] = pre[k][h];
                }
            }
        } else {
            for (int i = threadIdx.x; i < R; i += KBN_BLOCK) {
                int rem = i;
                int64_t gi = 0, gstride = 1;
#pragma unroll
                for (int d = D - 1; d >= 0; --d) {
                    const int e = rem % E[d];
                    rem /= E[d];
                    gi += (int64_t)wrapk(o[d] + e, g.K[d]) * gstride;
                    gstride *= g.K[d];
                }
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const float2 v0 = 2 * h < nc ? a.grid[(int64_t)(ch + 2 * h) * a.gsize + gi] : make_float2(0.f, 0.f);
                    const float2 v1 =
                        2 * h + 1 < nc ? a.grid[(int64_t)(ch + 2 * h + 1) * a.gsize + gi] : make_float2(0.f, 0.f);
                    reg4[i * H + h] = make_float4(v0.x, v0.y, v1.x, v1.y);
                }
            }
        }
        // upstream values of this group (mode 1), read before the next group's loads
        float2 vv[CP];
#pragma unroll
        for (int k = 0; k < CP; ++k)
            vv[k] = (MODE == 1 && act && k < nc) ? a.v[(int64_t)((ch + k) / a.nw) * a.M + q] : make_float2(0.f, 0.f);
        __syncthreads();
        if constexpr (LA) {
            if (ch + CP < ch1) fetch(ch + CP);
        }
        if (act) {
            float4 acc[H];
#pragma unroll
            for (int h = 0; h < H; ++h) acc[h] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (D == 1) {
#pragma unroll
                for (int j0 = 0; j0 < J; ++j0) {
                    const float w0 = w[0][j0];
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        const float4 v = reg4[(base + j0) * H + h];
                        acc[h].x = fmaf(w0, v.x, acc[h].x);
                        acc[h].y = fmaf(w0, v.y, acc[h].y);
                        acc[h].z = fmaf(w0, v.z, acc[h].z);
                        acc[h].w = fmaf(w0, v.w, acc[h].w);
                    }
                }
            } else if (D == 2) {
                // rows one at a time: only one row's taps live in registers
#pragma unroll 1
                for (int j0 = 0; j0 < J; ++j0) {
                    const float4 *row = reg4 + (base + j0 * E[D - 1]) * H;
                    float4 t[H];
#pragma unroll
                    for (int h = 0; h < H; ++h) t[h] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int j1 = 0; j1 < J; ++j1) {
                        const float w1 = w[1][j1];
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            const float4 v = row[j1 * H + h];
                            t[h].x = fmaf(w1, v.x, t[h].x);
                            t[h].y = fmaf(w1, v.y, t[h].y);
                            t[h].z = fmaf(w1, v.z, t[h].z);
                            t[h].w = fmaf(w1, v.w, t[h].w);
                        }
                    }
                    const float w0 = w[0][j0];
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        acc[h].x = fmaf(w0, t[h].x, acc[h].x);
                        acc[h].y = fmaf(w0, t[h].y, acc[h].y);
                        acc[h].z = fmaf(w0, t[h].z, acc[h].z);
                        acc[h].w = fmaf(w0, t[h].w, acc[h].w);
                    }
                }
            } else {
#pragma unroll 1
                for (int j0 = 0; j0 < J; ++j0) {
                    float4 t1[H];
#pragma unroll
                    for (int h = 0; h < H; ++h) t1[h] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int j1 = 0; j1 < J; ++j1) {
                        const float4 *row = reg4 + (base + (j0 * E[1] + j1) * E[2]) * H;
                        float4 t[H];
#pragma unroll
                        for (int h = 0; h < H; ++h) t[h] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                        for (int j2 = 0; j2 < J; ++j2) {
                            const float w2 = w[2][j2];
#pragma unroll
                            for (int h = 0; h < H; ++h) {
                                const float4 v = row[j2 * H + h];
                                t[h].x = fmaf(w2, v.x, t[h].x);
                                t[h].y = fmaf(w2, v.y, t[h].y);
                                t[h].z = fmaf(w2, v.z, t[h].z);
                                t[h].w = fmaf(w2, v.w, t[h].w);
                            }
                        }
                        const float w1 = w[1][j1];
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            t1[h].x = fmaf(w1, t[h].x, t1[h].x);
                            t1[h].y = fmaf(w1, t[h].y, t1[h].y);
                            t1[h].z = fmaf(w1, t[h].z, t1[h].z);
                            t1[h].w = fmaf(w1, t[h].w, t1[h].w);
                        }
                    }
                    const float w0 = w[0][j0];
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        acc[h].x = fmaf(w0, t1[h].x, acc[h].x);
                        acc[h].y = fmaf(w0, t1[h].y, acc[h].y);
                        acc[h].z = fmaf(w0, t1[h].z, acc[h].z);
                        acc[h].w = fmaf(w0, t1[h].w, acc[h].w);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < CP; ++k) {
                if (k >= nc) break;
                const int c = ch + k;
                const float ax = (k & 1) ? acc[k / 2].z : acc[k / 2].x;
                const float ay = (k & 1) ? acc[k / 2].w : acc[k / 2].y;
                if (MODE == 0) {
                    a.y[(int64_t)c * a.M + q] = make_float2(ax, ay);
                } else {
                    const float im = ay * vv[k].x - ax * vv[k].y;  // Im{acc conj(v)}
                    const int wd = c % a.nw;
#pragma unroll
                    for (int d = 0; d < D; ++d)
                        if (wd == d) jac[d] += im;
                }
            }
        }
        __syncthreads();
    }
    if (MODE == 1 && act) {
        float *part = a.part + (int64_t)gy * a.M * D;
#pragma unroll
        for (int d = 0; d < D; ++d) part[(int64_t)q * D + d] = jac[d];
    }
}

template <int D, int J, int MODE, int CP, int MAXC>
__global__ void __launch_bounds__(KBN_BLOCK) k_gather_staged(KbnGeom g, KbnGatherArgs a, int cg) {
    extern __shared__ float4 reg4[];
    gather_staged_wg<D, J, MODE, CP, MAXC>(g, a, cg, kbn_xcd_run_index(blockIdx.x, gridDim.x, blockIdx.y), blockIdx.y,
                                          reg4);
}

// The staged gathers of several plans in one launch: workgroup w belongs to
// the job i with start[i] <= w < start[i + 1] and is that job's workgroup
// (w - start[i]) mod blocks of channel group (w - start[i]) / blocks.
template <int D, int J, int MODE, int CP, int MAXC>
__global__ void __launch_bounds__(KBN_BLOCK)
k_gather_multi(const KbnGatherJob *__restrict__ jobs, const int64_t *__restrict__ start, int njobs) {
    extern __shared__ float4 reg4[];
    const int64_t w = blockIdx.x;
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    const KbnGatherJob &j = jobs[lo];
    const int64_t local = w - start[lo];
    gather_staged_wg<D, J, MODE, CP, MAXC>(j.g, j.a, j.cg, (int)(local % j.blocks), (int)(local / j.blocks), reg4);
}

// Direct gather (no staging): one thread per sorted point reads its taps from
// the grid in global memory; used when a staged region does not fit in LDS.
template <int D, int J, int MODE>
__global__ void __launch_bounds__(KBN_BLOCK) k_gather(KbnGeom g, KbnGatherArgs a, int cg) {
    const int64_t p = (int64_t)blockIdx.x * KBN_BLOCK + threadIdx.x;
    if (p >= a.M) return;
    const int q = sample_index(a.order, p);
    const bool bad = p >= a.toff[g.ntiles];
    float w[D][J];
    int idx[D][J];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        int start;
        float f;
        tap_origin(J, a.cell[d * a.M + p], a.frac[d * a.M + p], start, f);
        kb_weights<J>(f, g.coef, w[d]);
#pragma unroll
        for (int j = 0; j < J; ++j) idx[d][j] = wrapk(start + j, g.K[d]);
    }
    // flatten the leading axes' strides into the index tables
    if (D >= 2) {
#pragma unroll
        for (int j = 0; j < J; ++j) idx[D - 2][j] *= g.K[D - 1];
    }
    if (D == 3) {
#pragma unroll
        for (int j = 0; j < J; ++j) idx[0][j] *= g.K[1] * g.K[2];
    }
    const int ch0 = blockIdx.y * cg;
    const int ch1 = min(ch0 + cg, a.nch);
    float jac[KBN_MAX_D] = {0.f, 0.f, 0.f};
    for (int ch = ch0; ch < ch1; ++ch) {
        const float2 *G = a.grid + (int64_t)ch * a.gsize;
        float2 acc = make_float2(0.f, 0.f);
        if (D == 1) {
#pragma unroll
            for (int j0 = 0; j0 < J; ++j0) {
                const float2 v = G[idx[0][j0]];
                acc.x = fmaf(w[0][j0], v.x, acc.x);
                acc.y = fmaf(w[0][j0], v.y, acc.y);
            }
        } else if (D == 2) {
#pragma unroll
            for (int j0 = 0; j0 < J; ++j0) {
                const float2 *row = G + idx[0][j0];
                float2 s = make_float2(0.f, 0.f);
#pragma unroll
                for (int j1 = 0; j1 < J; ++j1) {
                    const float2 v = row[idx[1][j1]];
                    s.x = fmaf(w[1][j1], v.x, s.x);
                    s.y = fmaf(w[1][j1], v.y, s.y);
                }
                acc.x = fmaf(w[0][j0], s.x, acc.x);
                acc.y = fmaf(w[0][j0], s.y, acc.y);
            }
        } else {
#pragma unroll
            for (int j0 = 0; j0 < J; ++j0) {
                float2 s1 = make_float2(0.f, 0.f);
#pragma unroll
                for (int j1 = 0; j1 < J; ++j1) {
                    const float2 *row = G + idx[0][j0] + idx[1][j1];
                    float2 s = make_float2(0.f, 0.f);
#pragma unroll
                    for (int j2 = 0; j2 < J; ++j2) {
                        const float2 v = row[idx[2][j2]];
                        s.x = fmaf(w[2][j2], v.x, s.x);
                        s.y = fmaf(w[2][j2], v.y, s.y);
                    }
                    s1.x = fmaf(w[1][j1], s.x, s1.x);
                    s1.y = fmaf(w[1][j1], s.y, s1.y);
                }
                acc.x = fmaf(w[0][j0], s1.x, acc.x);
                acc.y = fmaf(w[0][j0], s1.y, acc.y);
            }
        }
        if (MODE == 0) {
            const int64_t bc = ch;  // channel = b_local * C + c
            if (bad) acc = make_float2(__builtin_nanf(""), __builtin_nanf(""));
            a.y[bc * a.M + q] = acc;
        } else {
            const int wd = ch % a.nw;
            const int64_t bc = ch / a.nw;
            const float2 v = a.v[bc * a.M + q];
            const float im = acc.y * v.x - acc.x * v.y;  // Im{acc conj(v)}
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (wd == d) jac[d] += im;
        }
    }
    if (MODE == 1) {
        float *part = a.part + (int64_t)blockIdx.y * a.M * D;
#pragma unroll
        for (int d = 0; d < D; ++d) part[(int64_t)q * D + d] = bad ? __builtin_nanf("") : jac[d];
    }
}

// LDS accumulator pitch of a tile axis: odd for every axis but the first,
// so that lanes stepping along any axis hit distinct LDS banks.
__host__ __device__ inline int acc_pitch(int d, int te) { return d == 0 ? te : (te | 1); }

// Channel plane stride (in float2) of the spread accumulator: padded so that
// consecutive planes start 12 LDS banks apart.
__host__ __device__ inline int spread_plane(int psize) { return psize + ((6 - psize) % 32 + 32) % 32; }

// Owner-computes spread.  Workgroup = (owner tile, channel group); the
// samples reaching the tile come from a precomputed list (index pass).  For a
// batch of list entries the workgroup stages in LDS each sample's local tap
// origin, its window weights and its k-space values; then every lane of a
// wave owns one (trailing tap, channel) pair and, entry after entry, adds its
// product into the tile accumulator with a plain LDS read-modify-write.  For
// one entry all lanes touch distinct cells, and waves own disjoint channels,
// so no two lanes ever update the same cell concurrently: no atomics, and a
// fixed accumulation order.
//   A = 1: lanes = (tap along the last axis) x (64 / J channels)
//   A = 2: lanes = (taps along the last two axes) x (64 / J^2 channels)
template <int D, int J, int A>
__global__ void __launch_bounds__(KBN_BLOCK) k_spread(KbnGeom g, KbnSpreadArgs a, int cw, int nwave, int wk0) {
    constexpr int EB = KBN_SPREAD_EB;
    constexpr int LANES_TAP = A == 1 ? J : J * J;
    constexpr int NEG = -(1 << 28);                // offset of a tap outside the tile
    extern __shared__ float smem[];
    const int wk = wk0 + blockIdx.y;               // work item
    if (wk >= a.scounts[0]) return;
    const int tile = a.swork[4 * wk];
    const int slot = a.swork[4 * wk + 3];
    const int ngroup = nwave * cw;                 // channels per workgroup
    const int ch0 = blockIdx.x * ngroup;
    const int nchg = min(ngroup, a.nch - ch0);
    int a0[KBN_MAX_D], te[KBN_MAX_D], pt[KBN_MAX_D];
    {
        int rem = tile;
        for (int d = D - 1; d >= 0; --d) {
            const int tc = rem % g.nto[d];
            rem /= g.nto[d];
            a0[d] = own_lo(tc, g.K[d], g.nto[d]);
            te[d] = own_lo(tc + 1, g.K[d], g.nto[d]) - a0[d];
            pt[d] = acc_pitch(d, te[d]);
        }
    }
    int psize = 1, tsize = 1;
    int stride[KBN_MAX_D];
    for (int d = D - 1; d >= 0; --d) {
        stride[d] = psize;
        psize *= pt[d];
        tsize *= te[d];
    }
    const int plane = spread_plane(psize);         // float2 per channel plane
    float2 *acc = reinterpret_cast<float2 *>(smem);
    // per staged entry and axis tap: (offset in the tile accumulator or NEG
    // when outside the tile, as int bits; weight)
    float2 *ent_ow = reinterpret_cast<float2 *>(acc + (size_t)ngroup * plane);  // [EB][D][J]
    int *ent_p = reinterpret_cast<int *>(ent_ow + EB * D * J);
    float2 *ent_y = reinterpret_cast<float2 *>(ent_p + EB);  // [ngroup][EB + 1]
    const int nthr = nwave * 64;
    for (int i = threadIdx.x; i < nchg * plane; i += nthr) acc[i] = make_float2(0.f, 0.f);

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int cc = lane / LANES_TAP;
    const int jin = lane - cc * LANES_TAP;
    const int cl = wave * cw + cc;                 // channel of this lane within the group
    const bool lane_on = cc < cw && cl < nchg;
    const int jb = A == 1 ? jin : jin % J;         // tap along the last axis
    const int ja = A == 1 ? 0 : jin / J;           // tap along the axis before it (A == 2)

    const int e0 = a.swork[4 * wk + 1], e1 = a.swork[4 * wk + 2];
    for (int eb = e0; eb < e1; eb += EB) {
        const int n = min(EB, e1 - eb);
        __syncthreads();  // previous batch fully consumed (and acc zeroed)
        if ((int)threadIdx.x < n) {
            // stage entry t: precomputed record -> per-axis tap offsets and weights
            const int t = threadIdx.x;
            const int e = eb + t;
            ent_p[t] = a.rec_p[e];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int2 tr = a.rec_t[(int64_t)e * D + d];
                const int l = tr.x;
                float w[J];
                kb_weights<J>(__int_as_float(tr.y), g.coef, w);
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    int loc = l + j;
                    if (loc >= g.K[d]) loc -= g.K[d];
                    const int off = loc < te[d] ? loc * stride[d] : NEG;
                    ent_ow[(t * D + d) * J + j] = make_float2(__int_as_float(off), w[j]);
                }
            }
        }
        __syncthreads();
        // k-space values of the staged entries: EB entries x channels, with
        // nthr / EB channels per pass (nthr is a multiple of EB)
        {
            const int i = threadIdx.x % EB;
            const int cstep = nthr / EB;
            if (i < n) {
                const int pi = ent_p[i];
                for (int c = threadIdx.x / EB; c < nchg; c += cstep)
                    ent_y[c * (EB + 1) + i] = a.ys[(int64_t)(ch0 + c) * a.M + pi];
            }
        }
        __syncthreads();
        if (lane_on) {
            float2 *accc = acc + (size_t)cl * plane;
            const float2 *yc = ent_y + cl * (EB + 1);
            for (int i = 0; i < n; ++i) {
                const float2 *owi = ent_ow + i * D * J;
                const float2 ib = owi[(D - 1) * J + jb];
                int inner = __float_as_int(ib.x);
                float wv = ib.y;
                if (A == 2) {
                    const float2 ia = owi[(D - 2) * J + ja];
                    inner += __float_as_int(ia.x);
                    wv *= ia.y;
                }
                const float2 yv = yc[i];
                const float2 v = make_float2(wv * yv.x, wv * yv.y);
                constexpr int NO = D - A == 0 ? 1 : (D - A == 1 ? J : J * J);  // outer taps
                float2 o[NO];
                int cidx[NO];
                float wo[NO];
#pragma unroll
                for (int t = 0; t < NO; ++t) {
                    int off = inner;
                    float wt = 1.f;
                    if (D - A >= 1) {
                        const int j0 = D - A == 1 ? t : t / J;
                        const float2 r0 = owi[j0];
                        off += __float_as_int(r0.x);
                        wt = r0.y;
                    }
                    if (D - A == 2) {
                        const int j1 = t % J;
                        const float2 r1 = owi[J + j1];
                        off += __float_as_int(r1.x);
                        wt *= r1.y;
                    }
                    cidx[t] = off;
                    wo[t] = wt;
                    if (off >= 0) o[t] = accc[off];
                }
#pragma unroll
                for (int t = 0; t < NO; ++t)
                    if (cidx[t] >= 0)
                        accc[cidx[t]] = make_float2(fmaf(wo[t], v.x, o[t].x), fmaf(wo[t], v.y, o[t].y));
            }
        }
    }
    __syncthreads();
    // write the owned tile of every channel in the group: to the grid, or
    // (tile split into several work items) to this item's partial slot.
    // Threads cover (channel, row) pairs x last-axis columns; a row is one
    // index tuple of the leading axes.
    int nrows = 1;
    for (int d = 0; d + 1 < D; ++d) nrows *= te[d];
    const int tl = te[D - 1];
    int pstride = 1;
    for (int d = 0; d < D; ++d) pstride *= g.To[d];
    for (int idx = threadIdx.x; idx < nchg * nrows * tl; idx += nthr) {
        const int cr = idx / tl;           // (channel, row) pair
        const int col = idx - cr * tl;
        const int c = cr / nrows;
        const int r = cr - c * nrows;
        int rem = r, lo = col;
        int64_t goff = 0, gstride = g.K[D - 1];
        for (int d = D - 2; d >= 0; --d) {
            const int l = D == 2 ? rem : rem % te[d];
            rem = D == 2 ? 0 : rem / te[d];
            lo += l * stride[d];
            goff += (int64_t)(a0[d] + l) * gstride;
            gstride *= g.K[d];
        }
        const float2 v = acc[(size_t)c * plane + lo];
        if (slot >= 0)
            a.partial[((int64_t)slot * a.nch + ch0 + c) * pstride + r * tl + col] = v;
        else
            a.grid[(int64_t)(ch0 + c) * a.gsize + goff + a0[D - 1] + col] = v;
    }
}

// Output-stationary spread of 2D owner tiles of more than 8 cells per axis (a
// caller's spread_tile).  Workgroup = (work item of one owner tile, group of CPT
// channels); one thread per cell of the tile, which keeps the CPT channel sums
// of its cell in registers.  The work item's list entries are staged in
// batches: per entry the tap origin relative to the tile, the window weights
// of each axis (evaluated once per entry) and the k-space values of the
// channel group.  Then every thread walks the batch: its tap index per axis is
// its cell minus the entry's origin (mod K), its weight the product of the
// axis weights (zero outside the J^2 footprint), and it adds weight * y into
// its sums.  No thread ever writes another thread's cell, so there are no
// atomics and no read-modify-write of shared memory, and the sum order (list
// order) is fixed.  The tile is written once at the end, to the grid or to the
// work item's partial slot.
// Body of one workgroup: channel group gx, work items wy, wy + ny, ...
// (the kernel's blockIdx.x, blockIdx.y and gridDim.y).
template <int J, int CPT, int EB>
__device__ __forceinline__ void spread_os_wg(const KbnGeom &g, const KbnSpreadArgs &a, int gx, int wy, int ny) {
    constexpr int D = 2;
    __shared__ float2 s_y[EB][CPT];
    __shared__ int s_p[EB];
    __shared__ float s_w[EB][D][J];
    __shared__ int s_l[EB][D];
    const int nwork = a.scounts[0];
    const int nthr = blockDim.x;
    int c[D];
    {
        int t = threadIdx.x;
#pragma unroll
        for (int d = D - 1; d >= 0; --d) {
            c[d] = t % g.To[d];
            t /= g.To[d];
        }
    }
    const int ch0 = gx * CPT;
    const int nchg = min(CPT, a.nch - ch0);
    // work items in dispatch order (hottest tiles first); a grid smaller
    // than the work list strides over it
    for (int wk = wy; wk < nwork; wk += ny) {
        const int tile = a.swork[4 * wk];
        const int slot = a.swork[4 * wk + 3];
        int a0[D], te[D];
        {
            int rem = tile;
#pragma unroll
            for (int d = D - 1; d >= 0; --d) {
                const int tc = rem % g.nto[d];
                rem /= g.nto[d];
                a0[d] = own_lo(tc, g.K[d], g.nto[d]);
                te[d] = own_lo(tc + 1, g.K[d], g.nto[d]) - a0[d];
            }
        }
        bool active = true;
#pragma unroll
        for (int d = 0; d < D; ++d) active = active && c[d] < te[d];
        float2 acc[CPT];
#pragma unroll
        for (int k = 0; k < CPT; ++k) acc[k] = make_float2(0.f, 0.f);
        const int e0 = a.swork[4 * wk + 1], e1 = a.swork[4 * wk + 2];
        for (int eb = e0; eb < e1; eb += EB) {
            const int n = min(EB, e1 - eb);
            __syncthreads();  // previous batch (or work item) consumed
            for (int t = threadIdx.x; t < n; t += nthr) {
                s_p[t] = a.rec_q[eb + t];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const int2 tr = a.rec_t[(int64_t)(eb + t) * D + d];
                    s_l[t][d] = tr.x;
                    float w[J];
                    kb_weights<J>(__int_as_float(tr.y), g.coef, w);
#pragma unroll
                    for (int j = 0; j < J; ++j) s_w[t][d][j] = w[j];
                }
            }
            __syncthreads();
            // loads past the batch or the channel group re-read a valid
            // value (never used), so that they are issued without branches
            // and several are in flight at once
#pragma unroll 4
            for (int i = threadIdx.x; i < EB * CPT; i += nthr) {
                const int t = i % EB;
                const int k = i / EB;
                const bool ok = t < n && k < nchg;
                s_y[t][k] = a.y[(int64_t)(ch0 + (ok ? k : 0)) * a.M + (ok ? s_p[t] : 0)];
            }
            __syncthreads();
            for (int i = 0; i < n; ++i) {
                float w = 1.f;
                bool in = true;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    int j = c[d] - s_l[i][d];
                    if (j < 0) j += g.K[d];
                    in = in && j < J;
                    w *= s_w[i][d][j < J ? j : J - 1];
                }
                w = in ? w : 0.f;
#pragma unroll
                for (int k = 0; k < CPT; ++k) {
                    const float2 y = s_y[i][k];
                    acc[k].x = fmaf(w, y.x, acc[k].x);
                    acc[k].y = fmaf(w, y.y, acc[k].y);
                }
            }
        }
        if (active) {
            int pstride = 1, loc = 0, lstride = 1;
            int64_t goff = 0, gstride = 1;
#pragma unroll
            for (int d = D - 1; d >= 0; --d) {
                pstride *= g.To[d];
                loc += c[d] * lstride;
                lstride *= te[d];
                goff += (int64_t)(a0[d] + c[d]) * gstride;
                gstride *= g.K[d];
            }
#pragma unroll
            for (int k = 0; k < CPT; ++k) {
                if (k < nchg) {
                    if (slot >= 0)
                        a.partial[((int64_t)slot * a.nch + ch0 + k) * pstride + loc] = acc[k];
                    else
                        a.grid[(int64_t)(ch0 + k) * a.gsize + goff] = acc[k];
                }
            }
        }
    }
}

template <int J, int CPT>
__global__ void __launch_bounds__(512) k_spread_os(KbnGeom g, KbnSpreadArgs a) {
    spread_os_wg<J, CPT, 32>(g, a, blockIdx.x, blockIdx.y, gridDim.y);
}

// The output-stationary spreads of several plans in one launch (same
// owner-tile shape, so one workgroup size): workgroup row y belongs to the
// job i with ystart[i] <= y < ystart[i + 1], which strides over its work
// items with ny rows; columns past the job's channel groups stop at once.
template <int J, int CPT>
__global__ void __launch_bounds__(512)
k_spread_os_multi(const KbnSpreadJob *__restrict__ jobs, const int *__restrict__ ystart, int njobs) {
    const int y = blockIdx.y;
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ystart[mid] <= y) lo = mid;
        else hi = mid - 1;
    }
    const KbnSpreadJob &j = jobs[lo];
    if ((int)blockIdx.x >= j.ngr) return;
    spread_os_wg<J, CPT, 32>(j.g, j.a, blockIdx.x, y - ystart[lo], j.ny);
}

// Output-stationary spread on the matrix cores, for owner tiles of at most 8
// cells per axis.  The tile's sums are the contraction
//   tile[channel, cell] = sum_entries y[entry, channel] * w[entry, cell],
// and v_mfma_f32_16x16x4_f32 takes four list entries per instruction: A holds
// 16 reals of y (8 channels), B the weights of 16 cells, and the 64 cells of
// an 8 x 8 tile (in 3D: of one x-slice) are four instructions.  One FP32
// matrix instruction adds its four products as a chain of four FMAs in entry
// order, so a cell's sum is the one that an FMA loop over the list would
// form; entries of zero weight and the padding of the last four (value and
// weight zero) leave it unchanged.  Hence the sums do not depend on how the
// channels are grouped.
//
// A batch of entries is staged in LDS, one record per entry: the window
// weights seen by the 8 cell coordinates of each axis (zero outside the
// footprint; every lane evaluates the polynomial of one tap, coefficients in
// registers, and a cross-lane read moves tap to cell) and the channels' values.
// Records past the end are zero.  The next batch's loads are in flight
// while the matrix cores work on the current one (two LDS buffers, one
// barrier per batch).
//
// FP32 matrix instructions share the SIMD's FMA units (measured: their 32
// cycles and the VALU's 4 per instruction add up), so both count: 96^3 x 8
// coils (kooshball, 1M samples) issues 17.5M matrix and 116M vector
// instructions, 1.0M of its 1.35M cycles per SIMD.  Measured against the
// cell-per-lane kernels it replaces: that adjoint's spread 1482 -> 600 us
// (plus 44 us for the copy in tile order), 75 x 90 x 64 x 4 coils 509 -> 73 us,
// 384^2 x 8 coils 60 -> 29 us, 320^2 x 64 channels 118 -> 64 us, 256^2 x 256
// channels (whose 0.54 GB of grid take 0.1 ms to write) 235 -> 194 us.
// Measured and not kept: one autonomous wave per item without staging
// (927 us at 96^3, the weights evaluated per slice), workgroups that stay
// resident and load across items (744 us: static shares; in 2D 29 -> 26 us at
// 384^2 x 8 coils, but 192 -> 201 us at 256 channels), batches sorted by slice
// so that a wave could own all slices (693-920 us).
typedef float mf_f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mf_f4 mfma4(float a, float b, mf_f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// tap polynomial of fraction f with this lane's coefficients
__device__ __forceinline__ float tap_poly(const float (&cf)[KBN_NCOEF], float f) {
    const float x = 2.f * f - 1.f;
    float w = cf[KBN_NCOEF - 1];
#pragma unroll
    for (int k = KBN_NCOEF - 2; k >= 0; --k) w = fmaf(w, x, cf[k]);
    return w;
}

// From the tap values w (tap = lane & 7) of an axis with K cells whose first
// tap sits at cell `rel` of the tile (modulo K): the weight of tile cell c,
// zero outside the footprint or when !ok.
template <int J>
__device__ __forceinline__ float cell_weight(float w, int rel, int c, int K, bool ok) {
    int j = c - rel;
    if (j < 0) j += K;
    const int src = ((int)threadIdx.x & 56) + (j & 7);
    const float v = __int_as_float(__builtin_amdgcn_ds_bpermute(src * 4, __float_as_int(w)));
    return ok && j < J ? v : 0.f;
}

template <int J>
__device__ __forceinline__ void lane_coefs(const float *__restrict__ coef, float (&cf)[KBN_NCOEF]) {
    const int tap = threadIdx.x & 7;
#pragma unroll
    for (int k = 0; k < KBN_NCOEF; ++k) cf[k] = tap < J ? coef[tap * KBN_NCOEF + k] : 0.f;
}

// 2D: a workgroup of four waves per (work item, 32 / CS * NG channels).  CS
// waves share the tile's four 2-row blocks and 4 / CS take different
// channels, 8 * NG each.  The values come from the caller's array, or (grouped,
// samples not along a trajectory) from the copy in tile order with a group's
// channels side by side.
template <int J, int CS, int NG>
__global__ void __launch_bounds__(256, CS * NG > 2 ? 6 : 5)
k_spread_mf2(KbnGeom g, KbnSpreadArgs a, bool may_group) {  // (NG = 2 only)
    constexpr int CHW = 32 / CS * NG;                          // channels per workgroup
    constexpr int BW = 4 / CS;                                 // blocks per wave
    constexpr int EB = CHW <= 8 ? 64 : (CHW <= 32 ? 32 : 16);  // entries per batch
    constexpr int YF = EB * CHW / 256;                         // values per thread and batch
    constexpr int TP = EB / 16;                                // weight passes (16 entries x 2 axes)
    // floats per record: rows (even cells, then odd), columns, values; 16 or
    // 48 modulo 64, so that four consecutive records' values take all banks
    constexpr int STR = CHW == 8 ? 48 : 16 + 2 * CHW;
    __shared__ __align__(16) float rec[2][EB * STR];
    const int tid = threadIdx.x, lane = tid & 63, k = lane >> 4, i = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wch = wv / CS, wcell = wv % CS;  // this wave's channels and blocks
    float cf[KBN_NCOEF];
    lane_coefs<J>(g.coef, cf);
    const int ch0 = blockIdx.x * CHW;
    const int nchg = min(CHW, a.nch - ch0);
    // staging: weights of (entry te + 16 pass, axis ax, cell cc), values of
    // (entry ty, channels kb + 256 / EB r)
    const int te = tid >> 4, ax = (tid >> 3) & 1, cc = tid & 7;
    const bool grouped = NG == 2 && may_group && a.scounts[2] == 0;
    const int ty = grouped ? tid / (256 / EB) : tid % EB, kb = grouped ? tid % (256 / EB) : tid / EB;
    const int Kx = ax ? g.K[1] : g.K[0];
    const int wpos = ax ? 8 + cc : (cc & 1) * 4 + (cc >> 1);
    const float2 *yb[YF];
#pragma unroll
    for (int r = 0; r < YF; ++r) {
        const int c = min(kb + 256 / EB * r, nchg - 1);
        yb[r] = grouped ? a.ys + (int64_t)ch0 * a.M + c : a.y + (int64_t)(ch0 + c) * a.M;
    }
    const int *rec_y = grouped ? a.rec_p : a.rec_q;
    const int ystep = grouped ? nchg : 1;
    const int nwork = a.scounts[0];
    int wk = blockIdx.y;
    int4 item = reinterpret_cast<const int4 *>(a.swork)[wk];  // tile, first entry, end, slot
    int q = 0;
    int2 t[TP];
    float2 yv[YF];
    // loads of the n entries from eb on; lanes past them repeat the last one,
    // so that all loads are issued without branches (stage writes zeros there)
    auto index = [&](int eb, int n) {
        if (n > 0) q = rec_y[eb + min(ty, n - 1)];
    };
    auto fetch = [&](int eb, int n) {
#pragma unroll
        for (int r = 0; r < YF; ++r) yv[r] = yb[r][(int64_t)q * ystep];
        const int2 *tb = a.rec_t + 2 * (int64_t)eb + ax;
#pragma unroll
        for (int p = 0; p < TP; ++p) t[p] = tb[2 * min(te + 16 * p, n - 1)];
    };
    auto stage = [&](float *buf, int n) {
#pragma unroll
        for (int p = 0; p < TP; ++p) {
            if (16 * p >= n) break;  // (no step reads these records)
            buf[(te + 16 * p) * STR + wpos] =
                cell_weight<J>(tap_poly(cf, __int_as_float(t[p].y)), t[p].x, cc, Kx, te + 16 * p < n);
        }
#pragma unroll
        for (int r = 0; r < YF; ++r)
            *reinterpret_cast<float2 *>(buf + ty * STR + 16 + 2 * (kb + 256 / EB * r)) =
                ty < n ? yv[r] : make_float2(0.f, 0.f);
    };
    for (; wk < nwork; wk += gridDim.y) {
        if (wk != (int)blockIdx.y) item = reinterpret_cast<const int4 *>(a.swork)[wk];
        const int e0 = item.y, e1 = item.z;
        mf_f4 acc[NG][BW];
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int b = 0; b < BW; ++b) acc[n][b] = mf_f4{0.f, 0.f, 0.f, 0.f};
        if (e0 < e1) {
            index(e0, e1 - e0);
            fetch(e0, e1 - e0);
            index(e0 + EB, e1 - e0 - EB);
            stage(rec[0], e1 - e0);
        }
        lds_barrier();
        int cur = 0;
        for (int eb = e0; eb < e1; eb += EB, cur ^= 1) {
            const bool more = eb + EB < e1;
            if (more) {
                fetch(eb + EB, e1 - eb - EB);
                index(eb + 2 * EB, e1 - eb - 2 * EB);
            }
            const float *buf = rec[cur] + k * STR;
            const int nst = (min(EB, e1 - eb) + 3) / 4;
            for (int s = 0; s < nst; ++s) {
                const float *rs = buf + 4 * s * STR;
                const float wc = rs[8 + (i & 7)];
                float w[BW], v[NG];
#pragma unroll
                for (int b = 0; b < BW; ++b) w[b] = rs[(i >> 3) * 4 + wcell * BW + b] * wc;
#pragma unroll
                for (int n = 0; n < NG; ++n) v[n] = rs[16 + (wch * NG + n) * 16 + i];
#pragma unroll
                for (int n = 0; n < NG; ++n)
#pragma unroll
                    for (int b = 0; b < BW; ++b) acc[n][b] = mfma4(v[n], w[b], acc[n][b]);
            }
            if (more) stage(rec[cur ^ 1], e1 - eb - EB);
            lds_barrier();
        }
        // lane: cell (row 2 b + i / 8, column i % 8) of channels 8 n + 2 k, + 1
        const int tr = item.x / g.nto[1], tc = item.x - tr * g.nto[1];
        const int a0r = own_lo(tr, g.K[0], g.nto[0]), a0c = own_lo(tc, g.K[1], g.nto[1]);
        const int ter = own_lo(tr + 1, g.K[0], g.nto[0]) - a0r, tec = own_lo(tc + 1, g.K[1], g.nto[1]) - a0c;
        float2 *dst;
        int64_t cs;
        int rs;  // channel and row strides
        if (item.w >= 0) {
            cs = (int64_t)g.To[0] * g.To[1];
            rs = tec;
            dst = a.partial + ((int64_t)item.w * a.nch + ch0) * cs;
        } else {
            cs = a.gsize;
            rs = g.K[1];
            dst = a.grid + (int64_t)ch0 * cs + (int64_t)a0r * rs + a0c;
        }
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = 8 * (wch * NG + n) + 2 * k + h;
#pragma unroll
                for (int b = 0; b < BW; ++b) {
                    const int r = 2 * (wcell * BW + b) + (i >> 3);
                    if (c < nchg && r < ter && (i & 7) < tec)
                        dst[c * cs + r * rs + (i & 7)] = make_float2(acc[n][b][2 * h], acc[n][b][2 * h + 1]);
                }
            }
    }
}

// k-space of each group of `cg` channels in tile order with the group's
// channels side by side, so that one entry's values are one short read:
// ys[group * cg * M + p * width + c] (width = channels of the group).  Nothing to do
// where *along (if given) says that the samples come along a trajectory.
__global__ void __launch_bounds__(KBN_BLOCK)
k_permute_groups(const float2 *__restrict__ y, float2 *__restrict__ ys, const int *__restrict__ order, int64_t M,
                 int nch, int cg, const int *__restrict__ along) {
    if (along && *along) return;
    const int ch0 = blockIdx.y * cg;
    const int w = min(cg, nch - ch0);
    for (int64_t i = (int64_t)blockIdx.x * KBN_BLOCK + threadIdx.x; i < M * w; i += (int64_t)gridDim.x * KBN_BLOCK) {
        const int64_t p = i / w;
        const int c = (int)(i - p * w);
        ys[(int64_t)ch0 * M + i] = y[(int64_t)(ch0 + c) * M + sample_index(order, p)];
    }
}

// 3D: a workgroup of 8 / S * CS waves per (work item, 8 / S channels), each
// wave taking S adjacent x-slices of the tile and, of their four 2-row blocks,
// 4 / CS.  The 16 reals of A are the S slices x 8 / S channels, A = w_x * y,
// and B = w_y * w_z over the 8 x 8 cells of a slice, so that few channels still
// fill the operand.  Of each batch a wave visits only the entries that reach
// its slices (a footprint covers 6 of the 13 positions of its first tap around
// an 8-cell tile), through a list of record offsets padded with the zero
// record.
template <int J, int S, int CS>
__global__ void __launch_bounds__(512 / S * CS, S == 2 ? 5 : 6) k_spread_mf3(KbnGeom g, KbnSpreadArgs a) {
    constexpr int CG = 8 / S;             // channels per group
    constexpr int W = 8 / S * CS;         // waves
    constexpr int BW = 4 / CS;            // blocks per wave
    constexpr int NT = 64 * W;            // threads
    constexpr int EB = 64;                // entries per batch (one per lane)
    constexpr int PE = EB * 8 / NT;       // weight passes per axis (NT / 8 entries each)
    constexpr int YF = EB * CG > NT ? EB * CG / NT : 1;  // values per thread and batch
    static_assert(PE >= 1, "batch shape");
    // floats per record: y (even cells, then odd), z, x, values
    constexpr int STR = 48;
    __shared__ __align__(16) float rec[2][(EB + 1) * STR];
    __shared__ int s_reach[2][EB];        // slices (bits) that each entry reaches
    __shared__ int s_off[W][EB + 4];
    const int tid = threadIdx.x, lane = tid & 63, k = lane >> 4, i = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sx = wv / CS * S;           // this wave's first slice
    const int wcell = wv % CS;            // and its blocks
    const int sub = i / (16 / S);         // slice of this lane's real
    float cf[KBN_NCOEF];
    lane_coefs<J>(g.coef, cf);
    const int ch0 = blockIdx.x * CG;
    const int nchg = min(CG, a.nch - ch0);
    // staging: weights of (entry te + NT / 8 pass, axis, cell cc), values of
    // (entry ty + NT / CG pass, channel yc)
    const int te = tid >> 3, cc = tid & 7;
    const int ty = tid / CG, yc = tid % CG;
    const float2 *yb = a.ys + (int64_t)ch0 * a.M + min(yc, nchg - 1);
    for (int x = tid; x < STR; x += NT) rec[0][EB * STR + x] = rec[1][EB * STR + x] = 0.f;
    const int nwork = a.scounts[0];
    int wk = blockIdx.y;
    int4 item = reinterpret_cast<const int4 *>(a.swork)[wk];  // tile, first entry, end, slot
    int q[YF];
    int2 t[3 * PE];
    float2 yv[YF];
    // loads of the n entries from eb on; lanes past them repeat the last one,
    // so that all loads are issued without branches (stage writes zeros there)
    auto index = [&](int eb, int n) {
        if (n > 0) {
#pragma unroll
            for (int r = 0; r < YF; ++r) q[r] = a.rec_p[eb + min(ty + NT / CG * r, n - 1)];
        }
    };
    auto fetch = [&](int eb, int n) {
#pragma unroll
        for (int r = 0; r < YF; ++r) yv[r] = yb[(int64_t)q[r] * nchg];
        const int2 *tb = a.rec_t + 3 * (int64_t)eb;
#pragma unroll
        for (int p = 0; p < 3 * PE; ++p) t[p] = tb[3 * min(te + NT / 8 * (p % PE), n - 1) + p / PE];
    };
    auto stage = [&](int b, int n) {
        float *buf = rec[b];
#pragma unroll
        for (int p = 0; p < 3 * PE; ++p) {
            const int e = te + NT / 8 * (p % PE);
            const int x = p / PE;
            const int pos = x == 0 ? 16 + cc : (x == 1 ? (cc & 1) * 4 + (cc >> 1) : 8 + cc);
            const float w = cell_weight<J>(tap_poly(cf, __int_as_float(t[p].y)), t[p].x, cc, g.K[x], e < n);
            buf[e * STR + pos] = w;
            if (S < 8 && x == 0) {
                const unsigned long long m = __ballot(w != 0.f);
                if (cc == 0) s_reach[b][e] = (int)(m >> (lane & 56)) & 255;
            }
        }
#pragma unroll
        for (int r = 0; r < YF; ++r)
            if (ty + NT / CG * r < EB)
                *reinterpret_cast<float2 *>(buf + (ty + NT / CG * r) * STR + 24 + 2 * yc) =
                    ty + NT / CG * r < n ? yv[r] : make_float2(0.f, 0.f);
    };
    for (; wk < nwork; wk += gridDim.y) {
        if (wk != (int)blockIdx.y) item = reinterpret_cast<const int4 *>(a.swork)[wk];
        const int e0 = item.y, e1 = item.z;
        mf_f4 acc[BW];
#pragma unroll
        for (int b = 0; b < BW; ++b) acc[b] = mf_f4{0.f, 0.f, 0.f, 0.f};
        if (e0 < e1) {
            index(e0, e1 - e0);
            fetch(e0, e1 - e0);
            index(e0 + EB, e1 - e0 - EB);
            stage(0, e1 - e0);
        }
        lds_barrier();
        int cur = 0;
        for (int eb = e0; eb < e1; eb += EB, cur ^= 1) {
            const bool more = eb + EB < e1;
            if (more) {
                fetch(eb + EB, e1 - eb - EB);
                index(eb + 2 * EB, e1 - eb - 2 * EB);
            }
            const float *buf = rec[cur];
            int n = min(EB, e1 - eb);
            if constexpr (S < 8) {
                // the list is the wave's own: its LDS accesses complete in
                // program order
                const bool hit = ((s_reach[cur][lane] >> sx) & ((1 << S) - 1)) != 0;
                const unsigned long long m = __ballot(hit);
                if (hit) s_off[wv][__popcll(m & ((1ull << lane) - 1ull))] = lane * STR;
                n = __popcll(m);
                if (lane < 3) s_off[wv][n + lane] = EB * STR;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
            }
            const int nst = (n + 3) / 4;
            // operands of one step, read a step ahead for S > 1 (two workgroups
            // of S = 1 need the registers more: six waves per SIMD)
            float wc, wx, v, wr[BW];
            auto operands = [&](int s) {
                const float *rs = buf + (S < 8 ? s_off[wv][4 * s + k] : (4 * s + k) * STR);
                wc = rs[8 + (i & 7)];
                wx = rs[16 + sx + sub];
                v = rs[24 + i % (16 / S)];
#pragma unroll
                for (int b = 0; b < BW; ++b) wr[b] = rs[(i >> 3) * 4 + wcell * BW + b];
            };
            if (S > 1 && nst > 0) operands(0);
            for (int s = 0; s < nst; ++s) {
                if (S == 1) operands(s);
                const float av = wx * v;
                float w[BW];
#pragma unroll
                for (int b = 0; b < BW; ++b) w[b] = wr[b] * wc;
                if (S > 1) operands(min(s + 1, nst - 1));
#pragma unroll
                for (int b = 0; b < BW; ++b) acc[b] = mfma4(av, w[b], acc[b]);
            }
            if (more) stage(cur ^ 1, e1 - eb - EB);
            lds_barrier();
        }
        int a0[3], tn[3];
        {
            int rem = item.x;
#pragma unroll
            for (int x = 2; x >= 0; --x) {
                const int o = rem % g.nto[x];
                rem /= g.nto[x];
                a0[x] = own_lo(o, g.K[x], g.nto[x]);
                tn[x] = own_lo(o + 1, g.K[x], g.nto[x]) - a0[x];
            }
        }
        // lane: cell (row 2 b + i / 8, column i % 8) of the two (slice, channel)
        // pairs of accumulator reals 4 k .. 4 k + 3
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = 4 * k + 2 * h;
            const int x = sx + r / (16 / S), c = (r % (16 / S)) >> 1;
            if (c >= nchg || x >= tn[0] || (i & 7) >= tn[2]) continue;
            float2 *dst;
            int rs;
            if (item.w >= 0) {
                rs = tn[2];
                dst = a.partial + ((int64_t)item.w * a.nch + ch0 + c) * (g.To[0] * g.To[1] * g.To[2]) + x * tn[1] * tn[2];
            } else {
                rs = g.K[2];
                dst = a.grid + (int64_t)(ch0 + c) * a.gsize + ((int64_t)(a0[0] + x) * g.K[1] + a0[1]) * rs + a0[2];
            }
#pragma unroll
            for (int b = 0; b < BW; ++b) {
                const int y = 2 * (wcell * BW + b) + (i >> 3);
                if (y < tn[1]) dst[y * rs + (i & 7)] = make_float2(acc[b][2 * h], acc[b][2 * h + 1]);
            }
        }
    }
}

// Tiles split into several work items: sum their partial tiles in slot
// order (deterministic) and write the grid tile.  Block = (channel, tile).
// Bound by its chain of loads (4 us whatever the grid, with 64 tiles or none):
// the first tile's entry is read beside the count that says whether it exists.
template <int D>
__global__ void __launch_bounds__(KBN_BLOCK) k_spread_combine(KbnGeom g, KbnSpreadArgs a) {
    const int ncomb = a.scounts[1];
    const int ch = blockIdx.x;
    float2 *G = a.grid + (int64_t)ch * a.gsize;
    int k = blockIdx.y;  // < ncomb_max
    int tile = a.scomb[3 * k], slot0 = a.scomb[3 * k + 1], ns = a.scomb[3 * k + 2];
    for (; k < ncomb; k += gridDim.y) {
        if (k != (int)blockIdx.y) tile = a.scomb[3 * k], slot0 = a.scomb[3 * k + 1], ns = a.scomb[3 * k + 2];
        int a0[KBN_MAX_D], te[KBN_MAX_D];
        int rem = tile;
        for (int d = D - 1; d >= 0; --d) {
            const int tc = rem % g.nto[d];
            rem /= g.nto[d];
            a0[d] = own_lo(tc, g.K[d], g.nto[d]);
            te[d] = own_lo(tc + 1, g.K[d], g.nto[d]) - a0[d];
        }
        int tsize = 1, pstride = 1;
        for (int d = 0; d < D; ++d) {
            tsize *= te[d];
            pstride *= g.To[d];
        }
        for (int i = threadIdx.x; i < tsize; i += blockDim.x) {
            float2 sum = make_float2(0.f, 0.f);
            const float2 *part = a.partial + ((int64_t)slot0 * a.nch + ch) * pstride + i;
            const int64_t step = (int64_t)a.nch * pstride;
            for (int s = 0; s < ns; s += 8) {  // eight loads in flight, added in slot order
                float2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = part[min(s + u, ns - 1) * step];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (s + u < ns) {
                        sum.x += v[u].x;
                        sum.y += v[u].y;
                    }
                }
            }
            int r = i;
            int64_t off = 0, stride = 1;
            for (int d = D - 1; d >= 0; --d) {
                const int l = r % te[d];
                r /= te[d];
                off += (int64_t)(a0[d] + l) * stride;
                stride *= g.K[d];
            }
            G[off] = sum;
        }
    }
}

// ys[ch][p] = y[ch][order[p]]: k-space values in tile order, so that the
// spread reads them with coalesced loads.
__global__ void __launch_bounds__(KBN_BLOCK)
k_permute(const float2 *__restrict__ y, float2 *__restrict__ ys, const int *__restrict__ order,
          int64_t M) {
    const int64_t p = (int64_t)blockIdx.x * KBN_BLOCK + threadIdx.x;
    if (p >= M) return;
    const int64_t ch = blockIdx.y;
    ys[ch * M + p] = y[ch * M + sample_index(order, p)];
}

// dst[i] = (accumulate ? dst[i] : 0) + sum_g part[g][i], summed in group order.
// Few samples of many channels make it a chain of loads, so sixteen are in flight
// (one after the other 464 groups of 994 x 2 sums took 109 us, now 13).
__global__ void __launch_bounds__(KBN_BLOCK)
k_reduce_parts(float *__restrict__ dst, const float *__restrict__ part, int64_t n, int groups,
               int accumulate) {
    const int64_t i = (int64_t)blockIdx.x * KBN_BLOCK + threadIdx.x;
    if (i >= n) return;
    float s = accumulate ? dst[i] : 0.f;
    int g = 0;
    for (; g + 16 <= groups; g += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = part[(int64_t)(g + u) * n + i];
#pragma unroll
        for (int u = 0; u < 16; ++u) s += v[u];
    }
    for (; g < groups; ++g) s += part[(int64_t)g * n + i];
    dst[i] = s;
}

}  // namespace

// Channel groups of a gather over `blocks` point blocks and nbc image-coil pairs.
//
// Staged: at least the KBN_GATHER_WG_MIN workgroups that fill the GPU; beyond that
// KBN_GATHER_WG_TARGET of them, whose durations differ with the points they hold,
// so that several rounds even out (five are resident per CU), but only while a
// group keeps KBN_GATHER_PAIRS pairs: every group repeats the points' weights, and
// an omega-Jacobian writes and sums one partial gradient per group.  Forward and
// omega-Jacobian of 256^2 x 256 channels: target 2048 177 and 285 us, 4096 161 and
// 262, 8192 157 and 249, more the same.  Pairs kept, whole calls (us), 1 / 2 / 4: 256^2
// x 2 with M = 2M, omega-Jacobian 153 / 128 / 127; 64^2 x 64 38.4 / 36.0 / 36.0; 239 x
// 137 x 16 forward 55.8 / 55.6 / 58.1; 20^3 x 64 omega-Jacobian 144 / 144 / 151; 48^2 x
// 400 78 / 77 / 81.
//
// Direct: KBN_GATHER_WG_ROUND workgroups are resident at once (four per CU) and each
// evaluates its points' weights and tap indexes first, so either one round of
// them, or so many that a round more or less does not matter.  One round / a
// group per pair (us): 82 x 23 x 25 x 110, J = 8, forward 1115 / 1644, omega-Jacobian
// 3425 / 5005; 105^3 x 4, J = 8, 1026 / 1283; 40^3 x 8, M = 96000 (three rounds), 614 /
// 823.  From four rounds on a group per pair: 50^3 x 8, J = 8, omega-Jacobian 6445
// against 8523 in one round; 40^3 x 12, M = 96000, even.
int64_t kbn_gather_groups(int64_t blocks, int64_t nbc, bool staged) {
    if (!staged) {
        if (blocks * nbc <= KBN_GATHER_WG_ROUND) return std::max<int64_t>(1, nbc);
        if (blocks * nbc < 4 * KBN_GATHER_WG_ROUND && blocks <= KBN_GATHER_WG_ROUND)
            return KBN_GATHER_WG_ROUND / blocks;
        return kbn_gather_groups_most(blocks, nbc, staged);
    }
    const int64_t fill = (KBN_GATHER_WG_MIN + blocks - 1) / blocks;
    const int64_t even = std::min((KBN_GATHER_WG_TARGET + blocks - 1) / blocks, nbc / KBN_GATHER_PAIRS);
    return std::max<int64_t>(1, std::min<int64_t>(nbc, std::max(fill, even)));
}

// The most groups that kbn_gather_groups gives nbc pairs or fewer (its count never
// falls with nbc in the staged form, in the direct one it may).
int64_t kbn_gather_groups_most(int64_t blocks, int64_t nbc, bool staged) {
    if (staged) return kbn_gather_groups(blocks, nbc, staged);
    return std::max<int64_t>(1, std::min<int64_t>(nbc, (KBN_GATHER_WG_TARGET + blocks - 1) / blocks));
}

// Launch shape of the gather: staged (LDS region fits 48 KiB) or direct, and
// the channel grouping (whole weight-channel sets per group).
KbnGatherShape kbn_gather_shape(const KbnGeom &g, int64_t M, int nch, int nw) {
    KbnGatherShape sh;
    const int lo = (g.J & 1) ? g.J / 2 : g.J / 2 - 1;
    const int hi = (g.J & 1) ? g.J / 2 + 1 : g.J / 2;
    int64_t region = 1;
    for (int d = 0; d < g.D; ++d) region *= (int64_t)std::min(g.T[d], g.K[d]) + lo + hi;
    // channels interpolated per pass: pairs (4 at a time measured slower: the
    // larger region allows fewer workgroups per CU)
    sh.cp = 2;
    sh.lds = sh.cp * sizeof(float2) * (size_t)region;
    sh.staged = sh.lds <= 48 * 1024;
    const int64_t nbc = std::max(1, nch / nw);
    int64_t blocks;
    if (sh.staged)
        blocks = (M + KBN_SUB - 1) / KBN_SUB + g.ntiles + 1;
    else
        blocks = std::max<int64_t>(1, (M + KBN_BLOCK - 1) / KBN_BLOCK);
    sh.blocks = blocks;
    const int64_t groups = kbn_gather_groups(blocks, nbc, sh.staged);
    sh.cg = (int)(((nbc + groups - 1) / groups) * nw);
    // the staged gather's whole channel pairs (8 channels one by one 21 us, in
    // pairs 16 us); the direct one takes a channel at a time (40 x 48 x 36 x 2,
    // J = 8: a workgroup row per channel 117 us, one for both 171)
    if (nw == 1 && sh.staged) sh.cg += sh.cg & 1;
    sh.groups = (nch + sh.cg - 1) / sh.cg;
    return sh;
}

namespace {

// the epilogue of the omega-Jacobian gather: the channel groups' partial
// gradients summed in group order
hipError_t reduce_parts(const KbnGeom &g, const KbnGatherArgs &a, int groups, hipStream_t s) {
    const int64_t n = a.M * g.D;
    k_reduce_parts<<<dim3((unsigned)((n + KBN_BLOCK - 1) / KBN_BLOCK)), dim3(KBN_BLOCK), 0, s>>>(
        a.domega, a.part, n, groups, a.accumulate);
    return hipGetLastError();
}

template <int D, int J>
hipError_t gather_dj(const KbnGeom &g, const KbnGatherArgs &a, int mode, hipStream_t s) {
    if (a.M == 0 || a.nch == 0) return hipSuccess;
    const KbnGatherShape sh = kbn_gather_shape(g, a.M, a.nch, a.nw);
    dim3 grid((unsigned)sh.blocks, (unsigned)sh.groups);
    if (sh.staged) {
        grid.x = (unsigned)kbn_xcd_padded(sh.blocks);
        // region cells per thread, loaded ahead in registers: the default
        // tiles' 37^2 (6) and 13^3 (9, or 10 with an edge of 9), in 3D up to
        // the 12 of 48 KiB.  Measured in 2D against loading them between the
        // barriers: 256^2 x 256 channels 184 -> 177 us and 311 -> 284 us
        // (omega-Jacobian), 320^2 x 64 channels 73 -> 58 and 161 -> 126 us
        const int64_t cells = ((int64_t)(sh.lds / (sh.cp * sizeof(float2))) + KBN_BLOCK - 1) / KBN_BLOCK;
#define KBN_GATHER(c)                                                                              \
    do {                                                                                           \
        if (mode == 0)                                                                             \
            k_gather_staged<D, J, 0, 2, c><<<grid, dim3(KBN_BLOCK), sh.lds, s>>>(g, a, sh.cg);     \
        else                                                                                       \
            k_gather_staged<D, J, 1, 2, c><<<grid, dim3(KBN_BLOCK), sh.lds, s>>>(g, a, sh.cg);     \
    } while (0)
        if (D == 2) {
            if (cells <= 6) KBN_GATHER((D == 2 ? 6 : 0));
            else KBN_GATHER(0);
        } else if (D == 3) {
            if (cells <= 10) KBN_GATHER((D == 3 ? 10 : 0));
            else KBN_GATHER((D == 3 ? 12 : 0));
        } else {
            KBN_GATHER(0);
        }
#undef KBN_GATHER
    } else {
        if (mode == 0)
            k_gather<D, J, 0><<<grid, dim3(KBN_BLOCK), 0, s>>>(g, a, sh.cg);
        else
            k_gather<D, J, 1><<<grid, dim3(KBN_BLOCK), 0, s>>>(g, a, sh.cg);
    }
    if (mode == 1) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return reduce_parts(g, a, sh.groups, s);
    }
    return hipGetLastError();
}

template <int D, int J>
hipError_t gather_multi_dj(int mode, const KbnGatherJob *jobs, const int64_t *start, int njobs, int64_t total,
                           size_t lds, hipStream_t s) {
    constexpr int MAXC = D == 3 ? 12 : 0;  // any staged region (48 KiB)
    const dim3 grid((unsigned)total);
    if (mode == 0)
        k_gather_multi<D, J, 0, 2, MAXC><<<grid, dim3(KBN_BLOCK), lds, s>>>(jobs, start, njobs);
    else
        k_gather_multi<D, J, 1, 2, MAXC><<<grid, dim3(KBN_BLOCK), lds, s>>>(jobs, start, njobs);
    return hipGetLastError();
}

// Launch shape of the spread: lanes per tap group (A), channels per wave,
// waves per workgroup, and the LDS bytes.
struct SpreadShape {
    int A, cw, nwave;
    size_t lds;
};

SpreadShape spread_shape(const KbnGeom &g, int nch) {
    SpreadShape sh;
    const int J = g.J, D = g.D;
    sh.A = (D >= 2 && nch < 64 / J) ? 2 : 1;
    sh.cw = sh.A == 1 ? 64 / J : std::max(1, 64 / (J * J));
    int psize = 1;
    for (int d = 0; d < D; ++d) psize *= acc_pitch(d, std::min(g.To[d], g.K[d]));
    const int plane = spread_plane(psize);
    const int EB = KBN_SPREAD_EB;
    auto bytes = [&](int nw) {
        const int ng = nw * sh.cw;
        return sizeof(float2) * (size_t)ng * plane + sizeof(int) * EB * (1 + D * J) +
               sizeof(float) * EB * D * J + sizeof(float2) * (size_t)ng * (EB + 1);
    };
    sh.nwave = 1;
    const int want = (nch + sh.cw - 1) / sh.cw;  // waves that have channels
    while (sh.nwave < 2 && sh.nwave < want && bytes(sh.nwave + 1) <= KBN_SPREAD_LDS) ++sh.nwave;
    sh.lds = bytes(sh.nwave);
    return sh;
}

template <int J>
hipError_t launch_os(const KbnSpreadSel &sel, dim3 grid, const KbnGeom &g, const KbnSpreadArgs &a, hipStream_t s) {
    const dim3 blk((unsigned)sel.tcells);
    switch (sel.cpt) {
        case 1: k_spread_os<J, 1><<<grid, blk, 0, s>>>(g, a); break;
        case 2: k_spread_os<J, 2><<<grid, blk, 0, s>>>(g, a); break;
        case 4: k_spread_os<J, 4><<<grid, blk, 0, s>>>(g, a); break;
        case 8: k_spread_os<J, 8><<<grid, blk, 0, s>>>(g, a); break;
        case 16: k_spread_os<J, 16><<<grid, blk, 0, s>>>(g, a); break;
        default: k_spread_os<J, 32><<<grid, blk, 0, s>>>(g, a); break;
    }
    return hipGetLastError();
}

template <int J>
hipError_t launch_os_multi(const KbnSpreadSel &sel, dim3 grid, const KbnSpreadJob *jobs, const int *ystart,
                           int njobs, hipStream_t s) {
    const dim3 blk((unsigned)sel.tcells);
    switch (sel.cpt) {
        case 1: k_spread_os_multi<J, 1><<<grid, blk, 0, s>>>(jobs, ystart, njobs); break;
        case 2: k_spread_os_multi<J, 2><<<grid, blk, 0, s>>>(jobs, ystart, njobs); break;
        case 4: k_spread_os_multi<J, 4><<<grid, blk, 0, s>>>(jobs, ystart, njobs); break;
        case 8: k_spread_os_multi<J, 8><<<grid, blk, 0, s>>>(jobs, ystart, njobs); break;
        case 16: k_spread_os_multi<J, 16><<<grid, blk, 0, s>>>(jobs, ystart, njobs); break;
        default: k_spread_os_multi<J, 32><<<grid, blk, 0, s>>>(jobs, ystart, njobs); break;
    }
    return hipGetLastError();
}

// the matrix-core spread of one call (channel groups x work items)
template <int D, int J>
hipError_t launch_mf(const KbnSpreadSel &sel, const KbnGeom &g, const KbnSpreadArgs &a, hipStream_t s) {
    const dim3 grid((unsigned)sel.ngr, (unsigned)sel.ny);
    if (sel.grouped) {
        // 2D: a bounded grid, which ends at once where there is nothing to copy
        const int64_t nb = (a.M * sel.cpt + KBN_BLOCK - 1) / KBN_BLOCK;
        const int64_t most = D == 2 ? std::max(1, 8192 / sel.ngr) : nb;
        const dim3 pgrid((unsigned)std::min(nb, most), (unsigned)sel.ngr);
        k_permute_groups<<<pgrid, dim3(KBN_BLOCK), 0, s>>>(a.y, a.ys, a.order, a.M, a.nch, sel.cpt,
                                                           D == 2 ? a.scounts + 2 : nullptr);
    }
    if constexpr (D == 2) {
        switch (sel.cpt) {
            case 8: k_spread_mf2<J, 4, 1><<<grid, dim3(256), 0, s>>>(g, a, sel.grouped); break;
            case 16: k_spread_mf2<J, 2, 1><<<grid, dim3(256), 0, s>>>(g, a, sel.grouped); break;
            case 32: k_spread_mf2<J, 1, 1><<<grid, dim3(256), 0, s>>>(g, a, sel.grouped); break;
            default: k_spread_mf2<J, 1, 2><<<grid, dim3(256), 0, s>>>(g, a, sel.grouped); break;
        }
    } else {
        switch (sel.cpt) {
            case 8: k_spread_mf3<J, 1, 1><<<grid, dim3(512), 0, s>>>(g, a); break;
            case 4: k_spread_mf3<J, 2, 1><<<grid, dim3(256), 0, s>>>(g, a); break;
            case 2: k_spread_mf3<J, 4, 2><<<grid, dim3(256), 0, s>>>(g, a); break;
            default: k_spread_mf3<J, 8, 4><<<grid, dim3(256), 0, s>>>(g, a); break;
        }
    }
    return hipGetLastError();
}

// the partial tiles of owner tiles split over several work items, summed
// in item order
template <int D>
hipError_t spread_combine(const KbnSpreadSel &sel, const KbnGeom &g, const KbnSpreadArgs &a, hipStream_t s) {
    if (a.ncomb_max <= 0) return hipSuccess;
    if (sel.path != KBN_SPREAD_PATH_GENERIC) {
        const int cb = std::min(KBN_BLOCK, (sel.tcells + 63) / 64 * 64);
        const int ny = std::max(1, std::min(a.ncomb_max, 8 * 256 * 4 / a.nch + 1));
        k_spread_combine<D><<<dim3((unsigned)a.nch, (unsigned)ny), dim3(cb), 0, s>>>(g, a);
    } else {
        k_spread_combine<D><<<dim3((unsigned)a.nch, (unsigned)a.ncomb_max), dim3(KBN_BLOCK), 0, s>>>(g, a);
    }
    return hipGetLastError();
}

template <int D, int J>
hipError_t spread_dj(const KbnGeom &g, const KbnSpreadArgs &a, hipStream_t s) {
    if (a.nch == 0) return hipSuccess;
    const KbnSpreadSel sel = kbn_spread_select(g, a);
    hipError_t e = hipSuccess;
    if (sel.path == KBN_SPREAD_PATH_MF) {
        if constexpr (D >= 2) e = launch_mf<D, J>(sel, g, a, s);
    } else if (sel.path == KBN_SPREAD_PATH_OS) {
        if constexpr (D == 2) e = launch_os<J>(sel, dim3((unsigned)sel.ngr, (unsigned)sel.ny), g, a, s);
    } else {
        const SpreadShape sh = spread_shape(g, a.nch);
        const int ngroup = sh.nwave * sh.cw;
        const int ng = (a.nch + ngroup - 1) / ngroup;
        if (a.M > 0) {  // the scatter kernel reads k-space values in tile order
            dim3 pgrid((unsigned)((a.M + KBN_BLOCK - 1) / KBN_BLOCK), (unsigned)a.nch);
            k_permute<<<pgrid, dim3(KBN_BLOCK), 0, s>>>(a.y, a.ys, a.order, a.M);
        }
        // one workgroup row per work item, in several launches beyond the rows of a
        // grid (a loop or a third grid dimension instead: 1D N = 64 21 -> 23 us, 60 x
        // 64 x 70 with 12-cell tiles 532 -> 548)
        for (int wk0 = 0; wk0 < a.nwork_max; wk0 += KBN_GRID_Y_MAX) {
            const dim3 grid((unsigned)ng, (unsigned)std::min(a.nwork_max - wk0, KBN_GRID_Y_MAX));
            if (sh.A == 1 || D == 1)
                k_spread<D, J, 1><<<grid, dim3(64 * sh.nwave), sh.lds, s>>>(g, a, sh.cw, sh.nwave, wk0);
            else
                k_spread<D, J, (D >= 2 ? 2 : 1)><<<grid, dim3(64 * sh.nwave), sh.lds, s>>>(g, a, sh.cw, sh.nwave, wk0);
        }
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    return spread_combine<D>(sel, g, a, s);
}

template <int D>
hipError_t gather_d(const KbnGeom &g, const KbnGatherArgs &a, int mode, hipStream_t s) {
    switch (g.J) {
        case 2: return gather_dj<D, 2>(g, a, mode, s);
        case 3: return gather_dj<D, 3>(g, a, mode, s);
        case 4: return gather_dj<D, 4>(g, a, mode, s);
        case 5: return gather_dj<D, 5>(g, a, mode, s);
        case 6: return gather_dj<D, 6>(g, a, mode, s);
        case 7: return gather_dj<D, 7>(g, a, mode, s);
        default: return gather_dj<D, 8>(g, a, mode, s);
    }
}

template <int D>
hipError_t gather_multi_d(int J, int mode, const KbnGatherJob *jobs, const int64_t *start, int njobs, int64_t total,
                          size_t lds, hipStream_t s) {
    switch (J) {
        case 2: return gather_multi_dj<D, 2>(mode, jobs, start, njobs, total, lds, s);
        case 3: return gather_multi_dj<D, 3>(mode, jobs, start, njobs, total, lds, s);
        case 4: return gather_multi_dj<D, 4>(mode, jobs, start, njobs, total, lds, s);
        case 5: return gather_multi_dj<D, 5>(mode, jobs, start, njobs, total, lds, s);
        case 6: return gather_multi_dj<D, 6>(mode, jobs, start, njobs, total, lds, s);
        case 7: return gather_multi_dj<D, 7>(mode, jobs, start, njobs, total, lds, s);
        default: return gather_multi_dj<D, 8>(mode, jobs, start, njobs, total, lds, s);
    }
}

template <int D>
hipError_t spread_d(const KbnGeom &g, const KbnSpreadArgs &a, hipStream_t s) {
    switch (g.J) {
        case 2: return spread_dj<D, 2>(g, a, s);
        case 3: return spread_dj<D, 3>(g, a, s);
        case 4: return spread_dj<D, 4>(g, a, s);
        case 5: return spread_dj<D, 5>(g, a, s);
        case 6: return spread_dj<D, 6>(g, a, s);
        case 7: return spread_dj<D, 7>(g, a, s);
        default: return spread_dj<D, 8>(g, a, s);
    }
}

}  // namespace

// Which spread kernel a call takes, with its launch shape: the matrix-core
// kernels (2D/3D owner tiles of at most 8 cells per axis: every plan with the
// default owner tile, except J = 8 with a grid edge of 18, 20, 25 or 27, which
// no split into 7- and 8-cell tiles fits), the output-stationary one (2D owner tiles of at
// most 512 cells), else the scatter kernel.
KbnSpreadSel kbn_spread_select(const KbnGeom &g, const KbnSpreadArgs &a) {
    static const bool os_on = [] {
        const char *e = std::getenv("KBN_SPREAD_OS");
        return !(e && e[0] == '0');
    }();
    KbnSpreadSel sel;
    const int D = g.D;
    int tcells = 1, tmax = 1;
    for (int d = 0; d < D; ++d) {
        tcells *= g.To[d];
        tmax = std::max(tmax, g.To[d]);
    }
    sel.tcells = tcells;
    if (D >= 2 && tmax <= 8 && os_on) {
        sel.path = KBN_SPREAD_PATH_MF;
        // channels per workgroup: 2D 8 to 64; 3D the 8 channels of a matrix
        // operand, or fewer with more slices in it
        if (D == 2)
            sel.cpt = a.nch <= 8 ? 8 : (a.nch <= 16 ? 16 : (a.nch <= 32 ? 32 : 64));
        else
            sel.cpt = a.nch <= 1 ? 1 : (a.nch <= 2 ? 2 : (a.nch <= 4 ? 4 : 8));
        sel.ngr = (a.nch + sel.cpt - 1) / sel.cpt;
        sel.ny = std::min(a.nwork_max, KBN_GRID_Y_MAX);
        // The values in tile order first: always in 3D, where eight tiles may read a
        // sample's, and in 2D where it was measured to pay, for samples in no order (whole
        // adjoints, us, straight / grouped): 128^2 x 128, 60000 samples 326 / 229 (J = 4 266
        // / 217; by the cell-per-thread kernel 271); 256^2 x 256, 32768 663 / 607; 256^2 x 64,
        // 131072 460 / 314.  Along a trajectory the values of a tile share their lines
        // (256^2 x 256, 32768 on spokes 483 / 541; 131072 655 / 816), which the index pass
        // finds out on the GPU: the copy's empty launch costs them 4 us, hence only from 3 x
        // 2^20 values on.  Fewer fit the caches (150 x 90 x 48, 5000 samples 40.5 / 43.5), and
        // 2^22 on few tiles (64^2 x 64, 60000, J = 4 87 / 103; 28^2 x 744, 20000 538 / 279; 56^2
        // x 300, 30000 399 / 209).  Not for fewer than four samples a tile (320^2 x 128,
        // 20480, J = 4 414 / 427), up to 32 channels (64^2 x 32, 60000 62 / 68, though 256^2 x
        // 32, 120000 202 / 142) or where y is in tile order already.
        const int64_t vals = a.M * a.nch, tiles = g.ntiles_own;
        const bool many = tiles >= 256 && a.nch * tiles >= 32768 ? vals >= 3 << 20 : tiles >= 25 && vals >= 1 << 22;
        sel.grouped = a.M > 0 && (D == 3 || (a.nch > 32 && a.order && a.M >= 4 * tiles && many));
        return sel;
    }
    if (D == 2 && tcells <= 512 && os_on) {
        sel.path = KBN_SPREAD_PATH_OS;
        const int want = std::min(a.nch, 32);
        int cpt = 1;
        while (cpt < want) cpt *= 2;
        sel.cpt = cpt;
        sel.ngr = (a.nch + cpt - 1) / cpt;
        sel.ny = std::min(a.nwork_max, KBN_GRID_Y_MAX);
        return sel;
    }
    sel.path = KBN_SPREAD_PATH_GENERIC;
    return sel;
}

hipError_t kbn_launch_gather(const KbnGeom &g, const KbnGatherArgs &a, int mode, hipStream_t s) {
    switch (g.D) {
        case 1: return gather_d<1>(g, a, mode, s);
        case 2: return gather_d<2>(g, a, mode, s);
        default: return gather_d<3>(g, a, mode, s);
    }
}

hipError_t kbn_launch_gather_reduce(const KbnGeom &g, const KbnGatherArgs &a, hipStream_t s) {
    if (a.M == 0 || a.nch == 0) return hipSuccess;
    return reduce_parts(g, a, kbn_gather_shape(g, a.M, a.nch, a.nw).groups, s);
}

hipError_t kbn_launch_gather_multi(int D, int J, int mode, const KbnGatherJob *jobs, const int64_t *start, int njobs,
                                   int64_t total, size_t lds, hipStream_t s) {
    if (njobs == 0 || total == 0) return hipSuccess;
    switch (D) {
        case 1: return gather_multi_d<1>(J, mode, jobs, start, njobs, total, lds, s);
        case 2: return gather_multi_d<2>(J, mode, jobs, start, njobs, total, lds, s);
        default: return gather_multi_d<3>(J, mode, jobs, start, njobs, total, lds, s);
    }
}

hipError_t kbn_launch_spread(const KbnGeom &g, const KbnSpreadArgs &a, hipStream_t s) {
    switch (g.D) {
        case 1: return spread_d<1>(g, a, s);
        case 2: return spread_d<2>(g, a, s);
        default: return spread_d<3>(g, a, s);
    }
}

hipError_t kbn_launch_spread_os_multi(const KbnSpreadSel &sel, int J, int maxngr, const KbnSpreadJob *jobs,
                                      const int *ystart, int njobs, int total_y, hipStream_t s) {
    if (njobs == 0 || total_y == 0) return hipSuccess;
    const dim3 grid((unsigned)maxngr, (unsigned)total_y);
    switch (J) {
        case 2: return launch_os_multi<2>(sel, grid, jobs, ystart, njobs, s);
        case 3: return launch_os_multi<3>(sel, grid, jobs, ystart, njobs, s);
        case 4: return launch_os_multi<4>(sel, grid, jobs, ystart, njobs, s);
        case 5: return launch_os_multi<5>(sel, grid, jobs, ystart, njobs, s);
        case 6: return launch_os_multi<6>(sel, grid, jobs, ystart, njobs, s);
        case 7: return launch_os_multi<7>(sel, grid, jobs, ystart, njobs, s);
        default: return launch_os_multi<8>(sel, grid, jobs, ystart, njobs, s);
    }
}

hipError_t kbn_launch_spread_combine(const KbnSpreadSel &sel, const KbnGeom &g, const KbnSpreadArgs &a,
                                     hipStream_t s) {
    switch (g.D) {
        case 1: return spread_combine<1>(sel, g, a, s);
        case 2: return spread_combine<2>(sel, g, a, s);
        default: return spread_combine<3>(sel, g, a, s);
    }
}
