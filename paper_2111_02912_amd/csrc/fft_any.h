// FFT passes along one grid axis for every 7-smooth length up to 1024, with the
// length, the radices and all indices known at compile time.
//
// Same operations as the runtime-length passes in fft.hip.  A length's radices
// (2 .. 10) are chosen for the fewest stages, three for nearly all lengths.  A
// workgroup holds LINES whole lines, and in each stage its threads take the
// LINES * L / R butterflies of radix R in turn, so a radix need not divide a
// fixed number of elements per thread (which lengths such as 490 = 2 5 7^2 would
// exclude); lines and threads are picked per length (split_cost).  The first
// stage reads global memory (zero padding is never read), the last stage
// writes it (cropped rows are never written), and the stages exchange data
// through LDS in place.
//
// What bounds them: the row passes the LDS exchanges (2.3 - 3.8 TB/s of
// algorithmic bytes at 336 points and more), the column passes likewise, at
// 2.4 - 4 TB/s; short lines the launch.  Measured, first + forward column +
// inverse column + last pass of 64 images of (L / 2)^2, us: the runtime-length
// passes against these 150: 90 -> 42, 250: 172 -> 64, 490: 477 -> 188, 630: 883
// -> 290, 1000: 2352 -> 714; register-resident passes with a fixed number of
// elements per thread, which they replace, 300: 115 -> 75, 384: 99 -> 92, 450:
// 224 -> 157, 588: 580 -> 250, 756: 1162 -> 445, 768: 514 -> 468.  The powers of
// two 128, 256 and 512 and the columns of 640 keep those (fft_fast.hip): 512 is
// 135 against 146 us, 640 columns 166 against 175.
//
// This header is compiled once per group of lengths (fft_any_*.hip).
#pragma once

#include <algorithm>

#include "kbn_internal.h"
#include "kbn_window.h"

namespace {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cmulc(float2 a, float2 b) {  // a * conj(b)
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// ---- small DFTs -------------------------------------------------------------
// cos(2 pi m / R) and sin(2 pi m / R) from the Taylor series in FP64 (angles
// folded to at most pi, where 20 terms leave less than 1e-17)
constexpr double trig(int m, int R, bool sine) {
    m %= R;
    const bool neg = 2 * m > R;
    const double x = 2.0 * 3.14159265358979323846 * (neg ? R - m : m) / R;
    double term = sine ? x : 1.0, sum = term;
    for (int k = sine ? 2 : 1; k < 40; k += 2) {
        term *= -x * x / (k * (k + 1.0));
        sum += term;
    }
    return sine && neg ? -sum : sum;
}

template <int R, bool INV>
struct ADft {  // odd prime R: direct, from the symmetric pairs (n, R - n)
    static __device__ __forceinline__ void run(float2 *a) {
        constexpr int H = (R - 1) / 2;
        float2 sp[H], sm[H];
#pragma unroll
        for (int n = 1; n <= H; ++n) {
            sp[n - 1] = make_float2(a[n].x + a[R - n].x, a[n].y + a[R - n].y);
            sm[n - 1] = make_float2(a[n].x - a[R - n].x, a[n].y - a[R - n].y);
        }
        const float2 a0 = a[0];
#pragma unroll
        for (int n = 0; n < H; ++n) a[0] = make_float2(a[0].x + sp[n].x, a[0].y + sp[n].y);
#pragma unroll
        for (int k = 1; k <= H; ++k) {
            float2 A = a0, Bv = make_float2(0.f, 0.f);
#pragma unroll
            for (int n = 1; n <= H; ++n) {
                const float c = (float)trig(n * k, R, false), s = (float)trig(n * k, R, true);
                A.x += sp[n - 1].x * c;
                A.y += sp[n - 1].y * c;
                Bv.x += sm[n - 1].x * s;
                Bv.y += sm[n - 1].y * s;
            }
            // forward: A - i B and A + i B
            const float2 lo = make_float2(A.x + Bv.y, A.y - Bv.x), hi = make_float2(A.x - Bv.y, A.y + Bv.x);
            a[k] = INV ? hi : lo;
            a[R - k] = INV ? lo : hi;
        }
    }
};
template <bool INV>
struct ADft<2, INV> {
    static __device__ __forceinline__ void run(float2 *a) {
        const float2 t = a[0];
        a[0] = make_float2(t.x + a[1].x, t.y + a[1].y);
        a[1] = make_float2(t.x - a[1].x, t.y - a[1].y);
    }
};
template <bool INV>
struct ADft<4, INV> {
    static __device__ __forceinline__ void run(float2 *a) {
        const float2 t0 = make_float2(a[0].x + a[2].x, a[0].y + a[2].y), t1 = make_float2(a[0].x - a[2].x, a[0].y - a[2].y);
        const float2 t2 = make_float2(a[1].x + a[3].x, a[1].y + a[3].y), u = make_float2(a[1].x - a[3].x, a[1].y - a[3].y);
        const float2 t3 = INV ? make_float2(-u.y, u.x) : make_float2(u.y, -u.x);
        a[0] = make_float2(t0.x + t2.x, t0.y + t2.y);
        a[2] = make_float2(t0.x - t2.x, t0.y - t2.y);
        a[1] = make_float2(t1.x + t3.x, t1.y + t3.y);
        a[3] = make_float2(t1.x - t3.x, t1.y - t3.y);
    }
};
// composite R = P Q: Q transforms of length P over the inputs q + Q p, the
// twiddles W^(q k), P transforms of length Q to the outputs k + P m
template <int P, int Q, bool INV>
struct ADft2 {
    static __device__ __forceinline__ void run(float2 *a) {
        constexpr int R = P * Q;
        float2 t[Q][P];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
            for (int p = 0; p < P; ++p) t[q][p] = a[q + Q * p];
            ADft<P, INV>::run(t[q]);
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            float2 u[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float c = (float)trig(q * k, R, false), s = (float)trig(q * k, R, true);
                u[q] = q * k == 0 ? t[q][k] : cmul(t[q][k], make_float2(c, INV ? s : -s));
            }
            ADft<Q, INV>::run(u);
#pragma unroll
            for (int m = 0; m < Q; ++m) a[k + P * m] = u[m];
        }
    }
};
template <bool INV>
struct ADft<6, INV> : ADft2<3, 2, INV> {};
template <bool INV>
struct ADft<8, INV> : ADft2<4, 2, INV> {};
template <bool INV>
struct ADft<9, INV> : ADft2<3, 3, INV> {};
template <bool INV>
struct ADft<10, INV> : ADft2<5, 2, INV> {};

// ---- radices ----------------------------------------------------------------
struct Radices {
    int n = 0;
    int r[6] = {1, 1, 1, 1, 1, 1};
};
// n factors of rem, each at most `most`, in decreasing order; the largest
// first factor kept smallest (balanced stages)
constexpr bool split_radices(int rem, int n, int most, int at, Radices &out) {
    if (n == 0) return rem == 1;
    for (int r = 2; r <= most; ++r) {
        if (rem % r) continue;
        out.r[at] = r;
        if (split_radices(rem / r, n - 1, r, at + 1, out)) return true;
    }
    return false;
}
constexpr Radices radices(int L) {
    Radices out;
    for (int n = 1; n <= 6; ++n) {
        out.n = n;
        if (!split_radices(L, n, 10, 0, out)) continue;
        // a radix divisible by 4 goes first, where it lets the column pass
        // know the zero padding at compile time
        for (int i = 0; i < n; ++i) {
            if (out.r[i] % 4) continue;
            const int r = out.r[i];
            for (int k = i; k > 0; --k) out.r[k] = out.r[k - 1];
            out.r[0] = r;
            break;
        }
        return out;
    }
    out.n = 0;
    return out;
}

// ---- work split ---------------------------------------------------------------
// butterfly rounds of all stages, in elements per thread, and the most that a
// stage keeps in registers
constexpr int stage_rounds(int L, int R, int lines, int nt) { return (lines * (L / R) + nt - 1) / nt; }
constexpr int most_elems(int L, int lines, int nt) {
    const Radices p = radices(L);
    int m = 0;
    for (int s = 0; s < p.n; ++s) m = std::max(m, stage_rounds(L, p.r[s], lines, nt) * p.r[s]);
    return m;
}
constexpr double idle_factor(int L, int lines, int nt) {  // thread slots per element of a stage
    const Radices p = radices(L);
    double f = 0.0;
    for (int s = 0; s < p.n; ++s) f += (double)stage_rounds(L, p.r[s], lines, nt) * p.r[s] * nt / ((double)lines * L);
    return f / p.n;
}
// What a split costs: idle slots, and the elements a thread holds (fewer
// leave room for more waves: 588-point rows 61 us with 18 per thread, 46 with
// 12; 480-point columns 54 us with 18, 45 with 12).
constexpr double split_cost(int L, int lines, int nt) {
    return idle_factor(L, lines, nt) * (1.0 + most_elems(L, lines, nt) / 30.0);
}
// rows: 256 threads and at most 32 KB
constexpr int row_lines(int L) {
    int lines = 1;
    double best = split_cost(L, 1, 256);
    for (int n = 2; n <= 64 && n * L <= 4096; ++n) {
        const double f = split_cost(L, n, 256);
        if (f < 0.99 * best) {
            best = f;
            lines = n;
        }
    }
    return lines;
}
// columns: 16 adjacent ones (128-byte row segments) up to 640 points (80 KB,
// two workgroups per CU), else 8; at most 768 threads (1024 leave 64 registers
// each: 630 points 120 against 88 us)
constexpr int col_lines(int L) { return L <= 640 ? 16 : 8; }
constexpr int col_threads(int L) {
    int nt = 128;
    double best = split_cost(L, col_lines(L), 128);
    for (int n = 192; n <= 768; n += 64) {
        const double f = split_cost(L, col_lines(L), n);
        if (f < 0.99 * best) {
            best = f;
            nt = n;
        }
    }
    return nt;
}

// ---- the stages ----------------------------------------------------------------
// COL: columns side by side in LDS (LINES a power of two); else lines one
// after the other
template <int L_, bool INV_, int NT_, int LINES_, bool COL_>
struct Any {
    static constexpr int L = L_, NT = NT_, LINES = LINES_;
    static constexpr bool INV = INV_, COL = COL_;
    static constexpr Radices P = radices(L_);
    static constexpr int NST = P.n;
    static_assert(NST > 0, "no radix plan for this length");
    static constexpr int VMAX = most_elems(L_, LINES_, NT_);
    template <int S>
    static constexpr int R() { return P.r[S]; }
    template <int S>
    static constexpr int Ns() {
        int n = 1;
        for (int s = 0; s < S; ++s) n *= P.r[s];
        return n;
    }
    template <int S>
    static constexpr int rounds() { return stage_rounds(L, R<S>(), LINES, NT); }
    // line and index of this thread's butterfly b of stage S
    template <int S>
    static __device__ __forceinline__ bool who(int b, int &l, int &j) {
        constexpr int NBF = L / R<S>(), T = LINES * NBF;
        const int w = (int)threadIdx.x + NT * b;
        if (COL) {
            l = w % LINES;
            j = w / LINES;
        } else {
            l = w / NBF;
            j = w - l * NBF;
        }
        return T % NT == 0 || w < T;
    }
    static __device__ __forceinline__ int lds_at(int l, int pos) { return COL ? pos * LINES + l : l * L + pos; }

    // inputs of stage S: f(line, position, input of the butterfly) -> value
    template <int S, class F>
    static __device__ __forceinline__ void load(float2 (&v)[VMAX], F f) {
        constexpr int Rr = R<S>();
#pragma unroll
        for (int b = 0; b < rounds<S>(); ++b) {
            int l, j;
            const bool ok = who<S>(b, l, j);
#pragma unroll
            for (int q = 0; q < Rr; ++q) v[b * Rr + q] = ok ? f(l, j + q * (L / Rr), q) : make_float2(0.f, 0.f);
        }
    }
    // stages S .. NST - 1; sink(slot, line, position, value) takes the outputs
    template <int S, class Sink>
    static __device__ __forceinline__ void run(float2 (&v)[VMAX], const float2 *tw, float2 *lds, Sink sink) {
        constexpr int Rr = R<S>(), N = Ns<S>(), TS = L / (N * Rr);
#pragma unroll
        for (int b = 0; b < rounds<S>(); ++b) {
            int l, j;
            who<S>(b, l, j);
            if (N > 1) {
                const int k = j % N;
#pragma unroll
                for (int q = 1; q < Rr; ++q) {
                    float2 t = tw[q * k * TS];
                    if (INV) t.y = -t.y;
                    v[b * Rr + q] = cmul(v[b * Rr + q], t);
                }
            }
            ADft<Rr, INV>::run(&v[b * Rr]);
        }
        if constexpr (S + 1 < NST && S > 0) lds_barrier();  // stage S's reads are done everywhere
#pragma unroll
        for (int b = 0; b < rounds<S>(); ++b) {
            int l, j;
            if (!who<S>(b, l, j)) continue;
            const int k = j % N, base = (j - k) * Rr + k;
#pragma unroll
            for (int q = 0; q < Rr; ++q) {
                if constexpr (S + 1 < NST)
                    lds[lds_at(l, base + q * N)] = v[b * Rr + q];
                else
                    sink(b * Rr + q, l, base + q * N, v[b * Rr + q]);
            }
        }
        if constexpr (S + 1 < NST) {
            lds_barrier();
            load<S + 1>(v, [&](int l, int pos, int) { return lds[lds_at(l, pos)]; });
            run<S + 1>(v, tw, lds, sink);
        }
    }
};

// image index of line position p for a line of n values centred at r = 0; -1
// for zero-padding positions
template <int L>
__device__ __forceinline__ int any_img(int p, int n) {
    const int h = n / 2;
    if (p < n - h) return p + h;
    if (p >= L - h) return p - L + h;
    return -1;
}

// ---- strided pass along a non-last axis ---------------------------------------
// HALF (forward, input padded to twice its length, K = 2N as on the sigma = 2
// grids, with a first radix divisible by 4): the index of a butterfly's input
// says whether it is an image row, so half of the inputs are zero without an
// address, a test or a load.
template <int L>
constexpr bool half_ok() { return radices(L).r[0] % 4 == 0; }

template <int L, bool INV, bool HALF>
__global__ void __launch_bounds__(col_threads(L)) k_any_cols(KbnMidPassArgs a, const float2 *__restrict__ tw) {
    using F = Any<L, INV, col_threads(L), col_lines(L), true>;
    extern __shared__ float2 lds[];
    const int ntile = (a.inner + F::LINES - 1) / F::LINES;
    const int64_t o = blockIdx.x / ntile;
    const int c0 = (int)(blockIdx.x - o * ntile) * F::LINES;
    // with a derived channel the groups run pair by pair, [unweighted, r^[0],
    // r^[1], ...], so that r^[0] times the unweighted channel re-reads it from
    // cache
    int64_t oi = o, oo = o;
    bool der = false;
    if (!INV && a.dsplit > 0) {
        const int64_t cc = o / (a.dnw + 1);
        const int k = (int)(o - cc * (a.dnw + 1));
        der = k == 1;
        oo = k == 0 ? cc : a.dsplit + cc * a.dnw + (k - 1);
        oi = k <= 1 ? cc : oo;
    }
    const float2 *in = a.in + (oi * a.nin) * (int64_t)a.inner + c0;
    float2 *out = a.out + (oo * a.nout) * (int64_t)a.inner + c0;
    const int cols = a.inner - c0;
    float2 v[F::VMAX];
    F::template load<0>(v, [&](int l, int pos, int q) {
        constexpr int R0 = F::template R<0>();
        if (HALF && q >= R0 / 4 && q < 3 * R0 / 4) return make_float2(0.f, 0.f);
        const int r = HALF ? (q < R0 / 4 ? pos + L / 4 : pos - 3 * L / 4) : a.pad_in ? any_img<L>(pos, a.nin) : pos;
        float2 x = l < cols && (HALF || r >= 0) ? in[(int64_t)r * a.inner + l] : make_float2(0.f, 0.f);
        if (!INV && der) {
            const float f = (float)(r - a.nin / 2);
            x = make_float2(x.x * f, x.y * f);
        }
        return x;
    });
    F::template run<0>(v, tw, lds, [&](int, int l, int pos, float2 val) {
        const int r = a.crop_out ? any_img<L>(pos, a.nout) : pos;
        if (l < cols && r >= 0) out[(int64_t)r * a.inner + l] = val;
    });
}

// ---- rows (last axis) -----------------------------------------------------------
struct AnyLine {  // per line of the workgroup
    int64_t x, s, out;  // image, coil map and output rows
    float f;            // scaling factors of the leading axes (and their coordinate weight)
    int wsel;           // weighted axis (-1: none)
};

template <int L>
__global__ void __launch_bounds__(256) k_any_first(KbnFirstPassArgs a, const float2 *__restrict__ tw) {
    using F = Any<L, false, 256, row_lines(L), false>;
    __shared__ float2 lds[F::LINES * L];
    __shared__ float2 twl[L];
    __shared__ AnyLine info[F::LINES];
    const int64_t line0 = (int64_t)blockIdx.x * F::LINES;
    for (int i = threadIdx.x; i < L; i += 256) twl[i] = tw[i];
    if ((int)threadIdx.x < F::LINES) {
        const int64_t line = line0 + threadIdx.x;
        AnyLine n{-1, 0, 0, 0.f, -1};
        if (line < a.nlines) {
            const int64_t ch = line / a.R0;
            const int row = (int)(line - ch * a.R0);
            int64_t cc, oline = line;
            if (a.nplain > 0) {  // forward plus omega-Jacobian layout (D >= 2)
                if (ch < a.nplain) {
                    cc = ch;
                } else {
                    const int64_t q = ch - a.nplain;
                    cc = q / (a.D - 1);
                    n.wsel = 1 + (int)(q - cc * (a.D - 1));
                    oline = (a.nplain + cc * a.D + n.wsel) * a.R0 + row;
                }
            } else {
                cc = ch / a.nw;
                n.wsel = a.weighted ? (int)(ch - cc * a.nw) : -1;
            }
            const int64_t bl = cc / a.C;
            n.x = (bl * a.R0 + row) * (int64_t)a.Nl;
            n.s = ((cc - bl * a.C) * a.R0 + row) * (int64_t)a.Nl;
            n.out = oline * L;
            float f = 1.f;
            int rem = row;
            for (int d = a.D - 2; d >= 0; --d) {
                const int id = rem % a.N[d];
                rem /= a.N[d];
                f *= a.deap[d][id];
                if (n.wsel == d) f *= (float)(id - a.N[d] / 2);
            }
            n.f = f;
        }
        info[threadIdx.x] = n;
    }
    __syncthreads();
    const float *deap_l = a.deap[a.D - 1];
    float2 v[F::VMAX];
    F::template load<0>(v, [&](int l, int pos, int) {
        const int j = any_img<L>(pos, a.Nl);
        const AnyLine &n = info[l];
        float2 x = make_float2(0.f, 0.f);
        if (j >= 0 && n.x >= 0) {
            x = a.x[n.x + j];
            float f = n.f * deap_l[j];
            if (n.wsel == a.D - 1) f *= (float)(j - a.Nl / 2);
            if (a.smaps) x = cmul(x, a.smaps[n.s + j]);
            x = make_float2(x.x * f, x.y * f);
        }
        return x;
    });
    F::template run<0>(v, twl, lds, [&](int, int l, int pos, float2 val) {
        if (info[l].x >= 0) a.out[info[l].out + pos] = val;
    });
}

// One image or image-coil pair a line, with or without a map: each value is
// weighted and stored as the last stage produces it.
template <int L>
__global__ void __launch_bounds__(256) k_any_last(KbnLastAdjArgs a, const float2 *__restrict__ tw) {
    using F = Any<L, true, 256, row_lines(L), false>;
    __shared__ float2 lds[F::LINES * L];
    __shared__ float2 twl[L];
    __shared__ AnyLine info[F::LINES];
    const int64_t line0 = (int64_t)blockIdx.x * F::LINES;
    for (int i = threadIdx.x; i < L; i += 256) twl[i] = tw[i];
    if ((int)threadIdx.x < F::LINES) {
        const int64_t line = line0 + threadIdx.x;
        AnyLine n{-1, 0, 0, 0.f, -1};
        if (line < a.nlines) {
            const int64_t bl = line / a.R0;
            const int row = (int)(line - bl * a.R0);
            n.x = line * L;
            n.s = ((a.cmod > 0 ? bl % a.cmod : 0) * a.R0 + row) * (int64_t)a.Nl;
            n.out = line * a.Nl;
            float f = 1.f;
            int rem = row;
            for (int d = a.D - 2; d >= 0; --d) {
                const int id = rem % a.N[d];
                rem /= a.N[d];
                f *= a.deap[d][id];
            }
            n.f = f;
        }
        info[threadIdx.x] = n;
    }
    __syncthreads();
    const float *deap_l = a.deap[a.D - 1];
    float2 v[F::VMAX];
    F::template load<0>(v, [&](int l, int pos, int) {
        return info[l].x >= 0 ? a.in[info[l].x + pos] : make_float2(0.f, 0.f);
    });
    F::template run<0>(v, twl, lds, [&](int, int l, int pos, float2 val) {
        const int j = any_img<L>(pos, a.Nl);
        if (j < 0 || info[l].x < 0) return;
        if (a.smaps) val = cmulc(val, a.smaps[info[l].s + j]);
        const float f = info[l].f * deap_l[j];
        val = make_float2(val.x * f, val.y * f);
        float2 *x = a.x + info[l].out + j;
        if (a.accumulate) val = make_float2(x->x + val.x, x->y + val.y);
        *x = val;
    });
}

template <int L>
hipError_t any_first(const KbnFirstPassArgs &a, const float2 *tw, hipStream_t s) {
    constexpr int LINES = row_lines(L);
    k_any_first<L><<<dim3((unsigned)((a.nlines + LINES - 1) / LINES)), dim3(256), 0, s>>>(a, tw);
    return hipGetLastError();
}

template <int L, bool INV, bool HALF>
hipError_t any_cols(const KbnMidPassArgs &a, const float2 *tw, int64_t total, hipStream_t s) {
    constexpr size_t LDS = sizeof(float2) * L * col_lines(L);
    constexpr int NT = col_threads(L);  // (evaluated per launch if it is not a constant here: 2 - 3 us)
    if constexpr (LDS > 64 * 1024) {  // opt in to more than the default (once)
        static const hipError_t ok = hipFuncSetAttribute(
            (const void *)k_any_cols<L, INV, HALF>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS);
        if (ok != hipSuccess) return ok;
    }
    k_any_cols<L, INV, HALF><<<dim3((unsigned)total), dim3(NT), LDS, s>>>(a, tw);
    return hipGetLastError();
}

template <int L>
hipError_t any_mid(const KbnMidPassArgs &a, const float2 *tw, int inverse, hipStream_t s) {
    constexpr int LINES = col_lines(L);
    const int64_t total = a.outer * ((a.inner + LINES - 1) / LINES);
    if (total <= 0) return hipSuccess;
    if (a.dsplit > 0 && (inverse || !a.pad_in || a.dnw < 2 || a.outer != a.dsplit * (a.dnw + 1)))
        return hipErrorInvalidValue;
    if (inverse) return any_cols<L, true, false>(a, tw, total, s);
    if constexpr (half_ok<L>()) {
        if (a.pad_in && 2 * a.nin == L) return any_cols<L, false, true>(a, tw, total, s);
    }
    return any_cols<L, false, false>(a, tw, total, s);
}

template <int L>
hipError_t any_last(const KbnLastAdjArgs &a, const float2 *tw, hipStream_t s) {
    constexpr int LINES = row_lines(L);
    const dim3 grid((unsigned)((a.nlines + LINES - 1) / LINES));
    k_any_last<L><<<grid, dim3(256), 0, s>>>(a, tw);
    return hipGetLastError();
}

}  // namespace

// The passes of one group of lengths (null for a length of another group).
#define KBN_ANY_CASE(n) \
    case n: return KbnAnyPasses{any_first<n>, any_mid<n>, any_last<n>};
#define KBN_ANY_UNIT(name, LENS)             \
    KbnAnyPasses name(int L) {               \
        switch (L) {                         \
            LENS(KBN_ANY_CASE)               \
            default: return KbnAnyPasses{};  \
        }                                    \
    }
