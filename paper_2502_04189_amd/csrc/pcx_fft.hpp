// pcx_fft.hpp -- the x and y transform passes for the lengths with a fixed
// plan: everything about the length (radices, strides, divisions, lines per
// tile) is known at compile time, the first stage takes its points straight
// from memory into registers and, where no corner turn follows, the last one
// stores them straight back, so a tile crosses LDS once per stage boundary
// instead of once more for the copy in, the copy out and every pre- and
// post-step.
//
// A tile is LINES consecutive lines: rows (k, j) with j fastest (x passes)
// or columns (l, k) with k fastest (y passes), counted with the padded
// strides of S1 and S2 so that the corner turns' segments start on 128-byte
// lines (the padding's lines are idle); tiles run over plane and mode
// boundaries, so domains of short planes fill their tiles.  Butterfly b of a
// stage is thread b mod the workgroup's threads.
//
// The passes are bound by memory.  Against the passes that copy each tile
// into LDS and out of it with run-time plans: 512^3 FP64 (2.15 GB a pass)
// the same 0.39-0.44 ms, y of 1024 x 1024 x 512 (8.6 GB) 3.3 -> 2.1 ms forward and 3.8 ->
// 2.0 inverse, x of 256^3 (0.27 GB) 112 -> 54 us, the batch's x and y passes
// (1.1 GB, 192 domains) 837, 803, 695, 680 -> 270, 300, 190, 185 us: there
// the general passes held 216 registers, one workgroup per CU.
#pragma once

#include "pcx_fplan.hpp"
#include "pcx_launch.hpp"
#include "pcx_passes.hpp"

namespace pcx {

// ------------------------------------------------------------ one stage
// exp(-+ 2 pi i e / n), e in [0, n), from the table of the first tw_half(n)
template <bool INV, int N, typename C> __device__ __forceinline__ C troot(const C *tw, int e)
{
    C w;
    if constexpr (N & 1) w = tw[e];
    else w = e < N / 2 ? tw[e] : C{-tw[e - N / 2].x, -tw[e - N / 2].y};
    if (INV) w.y = -w.y;
    return w;
}

// Stage of radix R with NS = product of the radices before it, into LDS:
// rd(line, n) gives input point n of a line, wr(line, n, v) takes output
// point n.  LF: consecutive threads are consecutive lines (else consecutive
// butterflies of a line).  SYNC: a workgroup barrier between the reads and
// the writes (in place in LDS).
template <typename T, bool INV, int N, int R, int NS, int LINES, int NTH, bool LF, bool SYNC, class Rd, class Wr>
__device__ __forceinline__ void fstage(const c2<T> *tw, Rd rd, Wr wr)
{
    using C = c2<T>;
    constexpr int NB = N / R, TOT = LINES * NB, K = (TOT + NTH - 1) / NTH, TS = N / (NS * R);
    C v[K][R];
    auto at = [](int b) { return TOT % NTH ? min(b, TOT - 1) : b; };
    auto where = [](int b, int &line, int &j) {
        if constexpr (LF) {
            line = b % LINES;
            j = b / LINES;
        } else {
            line = b / NB;
            j = b - line * NB;
        }
    };
#pragma unroll
    for (int t = 0; t < K; ++t) {
        int line, j;
        where(at(threadIdx.x + t * NTH), line, j);
#pragma unroll
        for (int r = 0; r < R; ++r) v[t][r] = rd(line, j + r * NB);
    }
    if constexpr (NS > 1) {
#pragma unroll
        for (int t = 0; t < K; ++t) {
            int line, j;
            where(at(threadIdx.x + t * NTH), line, j);
            const int jm = j % NS;
#pragma unroll
            for (int r = 1; r < R; ++r) v[t][r] = cmul(v[t][r], troot<INV, N>(tw, jm * r * TS));
        }
    }
    if constexpr (SYNC) __syncthreads();
#pragma unroll
    for (int t = 0; t < K; ++t) {
        const int b = threadIdx.x + t * NTH;
        if (TOT % NTH == 0 || b < TOT) {
            int line, j;
            where(b, line, j);
            bfly<INV, R, C, T>(v[t]);
            const int o = (j / NS) * NS * R + j % NS;
#pragma unroll
            for (int r = 0; r < R; ++r) wr(line, o + r * NS, v[t][r]);
        }
    }
}

// The last stage of LINES lines (radix R), out of LDS: its rounds do not
// wait for one another, so a thread holds one butterfly at a time.  pre(r,
// line, n) sees the round's output points before its points are read, wr(
// line, n, v, r) takes them.
struct NoPre {
    __device__ __forceinline__ void operator()(int, int, int) const {}
};
template <typename T, bool INV, int N, int R, int LINES, int NTH, class Rd, class Wr, class Pre>
__device__ __forceinline__ void fstage_out(const c2<T> *tw, Rd rd, Wr wr, Pre pre)
{
    using C = c2<T>;
    constexpr int NB = N / R, TOT = LINES * NB, K = (TOT + NTH - 1) / NTH;
#pragma unroll 1
    for (int t = 0; t < K; ++t) {
        const int b = threadIdx.x + t * NTH;
        if (TOT % NTH != 0 && b >= TOT) break;
        const int line = b / NB, j = b - line * NB;
#pragma unroll
        for (int r = 0; r < R; ++r) pre(r, line, j + r * NB);
        C v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = rd(line, j + r * NB);
#pragma unroll
        for (int r = 1; r < R; ++r) v[r] = cmul(v[r], troot<INV, N>(tw, j * r));
        bfly<INV, R, C, T>(v);
#pragma unroll
        for (int r = 0; r < R; ++r) wr(line, j + r * NB, v[r], r);
    }
}

// The stages of LINES lines in the buffer buf (line stride lds_line(N)).
// first: rd feeds the first stage (RD_LDS: from the buffer itself, so a
// barrier goes between), then the middle ones; last: wr takes the last
// stage's points (WR_LDS: into the buffer).  Each ends with a barrier when
// it wrote LDS.
template <typename T, bool INV, int N, int LINES, int NTH> struct LineFft {
    using C = c2<T>;
    static constexpr FPlan P = fplan(N);
    static_assert(P.n >= 2 && P.n <= 4, "a fixed plan");
    static constexpr int LDC = lds_line(N);
    C *buf;
    const C *tw;
    template <bool LF, bool RD_LDS, class Rd> __device__ __forceinline__ void first(Rd rd) const
    {
        C *const b = buf;
        fstage<T, INV, N, P.r[0], 1, LINES, NTH, LF, RD_LDS>(
            tw, rd, [b](int line, int n, C v) { b[line * LDC + pidx(n)] = v; });
        __syncthreads();
    }
    template <int R, int NS> __device__ __forceinline__ void middle() const
    {
        C *const b = buf;
        fstage<T, INV, N, R, NS, LINES, NTH, false, true>(
            tw, [b](int line, int n) { return b[line * LDC + pidx(n)]; },
            [b](int line, int n, C v) { b[line * LDC + pidx(n)] = v; });
        __syncthreads();
    }
    __device__ __forceinline__ void middles() const
    {
        if constexpr (P.n > 2) middle<P.r[1], P.r[0]>();
        if constexpr (P.n > 3) middle<P.r[2], P.r[0] * P.r[1]>();
    }
    template <class Wr, class Pre> __device__ __forceinline__ void last(Wr wr, Pre pre) const
    {
        C *const b = buf;
        fstage_out<T, INV, N, P.r[P.n - 1], LINES, NTH>(
            tw, [b](int line, int n) { return b[line * LDC + pidx(n)]; }, wr, pre);
    }
    // the last stage into the buffer
    __device__ __forceinline__ void last() const { middle<P.r[P.n - 1], N / P.r[P.n - 1]>(); }
};

// Row of an x tile: row j of plane k of line q = k ys + j; on: it exists
// (else a row that does, to read)
struct XLine {
    int k, j;
    bool on;
};
__device__ __forceinline__ XLine xline(const Dom &d, int q)
{
    const int k = q / d.ys, j = q - k * d.ys;
    return XLine{min(k, d.nz - 1), min(j, d.ny - 1), k < d.nz && j < d.ny};
}

// ------------------------------------------------------------- x forward
// Rows of src (f or r) -> half spectra (or cosine modes) -> S1.  M: half
// length.  Same transforms as pass_xfwd; the split into X[l] and the cosine
// step are taken by the thread that stores the mode.
template <typename T, int M> __device__ __forceinline__ void fft_xfwd(const Dom &d, const double *src, int tile, char *smem)
{
    using C = c2<T>;
    constexpr int L = fft_lines(M, sizeof(C)), NTH = fft_threads(M, sizeof(C)), LDC = lds_line(M);
    constexpr int STEP = NTH / L, K = (M / 2 + 1 + STEP - 1) / STEP;
    static_assert(NTH % L == 0, "a thread keeps its row in the corner turn");
    C *buf = (C *)smem, *ltw = buf + L * LDC;
    TwStage<T, NTH> tws;
    tws.fetch(d.fx);
    const int nx = d.nx, q0 = tile * L;
    const bool wx = d.bcx != BC_PER;
    auto row_of = [&](int line) {
        const XLine x = xline(d, q0 + line);
        return src + ((size_t)x.k * d.ny + x.j) * nx;
    };
    tws.put(ltw, d.fx);
    const LineFft<T, false, M, L, NTH> F{buf, ltw};
    if (!wx) {
        F.template first<false, false>([&](int line, int n) {
            const double2 s = ((const double2 *)row_of(line))[n];
            return C{(T)s.x, (T)s.y};
        });
    } else {
        // cosine transform by reordering: real point m of the sequence is
        // s[2m] below the middle, s[2 (nx - 1 - m) + 1] (times -1 for the
        // sine transform) from there on
        const double odd = d.bcx == BC_DIR ? -1.0 : 1.0;
        F.template first<false, false>([&](int line, int n) {
            const double *s = row_of(line);
            auto pt = [&](int m) {
                const bool lo = m < M;
                const double v = s[lo ? 2 * m : 2 * (nx - 1 - m) + 1];
                return (T)(lo ? v : odd * v);
            };
            return C{pt(2 * n), pt(2 * n + 1)};
        });
    }
    F.middles();
    // X[l] = E + W^l O and X[M-l] = conj(E - W^l O) of the half-length
    // spectrum, l in [0, M/2], by one thread: a root and two LDS reads for two
    // modes, the roots from memory ahead of the last stage (in LDS they cost
    // a tile per CU at some lengths)
    const int r = threadIdx.x % L, l0 = threadIdx.x / L;
    const C *twr = (const C *)d.twr;
    C w[K];
#pragma unroll
    for (int t = 0; t < K; ++t) w[t] = twr[min(l0 + t * STEP, M / 2)];
    F.last();
    const XLine x = xline(d, q0 + r);
    const C *z = buf + r * LDC;
    auto pair = [&](int l, C root, C &xl, C &xm) {
        if (l == 0) {
            const C a = z[0];
            xl = C{a.x + a.y, T(0)};
            xm = C{a.x - a.y, T(0)};
            return;
        }
        const C zl = z[pidx(l)], zm = z[pidx(M - l)];
        const C e = {T(0.5) * (zl.x + zm.x), T(0.5) * (zl.y - zm.y)};
        const C o = cmul(root, C{T(0.5) * (zl.y + zm.y), T(-0.5) * (zl.x - zm.x)});
        xl = cadd(e, o);
        xm = C{e.x - o.x, o.y - e.y};
    };
    const int ys = d.ys;
    C *out = (C *)d.s1 + (size_t)x.k * d.nl * ys + x.j;
    const bool on = x.on;
    // A_k = W_{4N}^k X_k: with walls modes Re A_k and, N - k, -Im A_k
    const C *wd = (const C *)d.dctx;
#pragma unroll
    for (int t = 0; t < K; ++t) {
        const int l = l0 + t * STEP, m = M - l;
        if (!on || l > M / 2) continue;
        C xl, xm;
        pair(l, w[t], xl, xm);
        if (!wx) {
            st_stream(out + (size_t)l * ys, xl);
            if (l != m) st_stream(out + (size_t)m * ys, xm);
        } else {
            const C al = cmul(wd[l], xl);
            st_stream(out + (size_t)l * ys, C{al.x, T(0)});
            if (l) st_stream(out + (size_t)(nx - l) * ys, C{-al.y, T(0)});
            if (l == m) continue;
            const C am = cmul(wd[m], xm);
            st_stream(out + (size_t)m * ys, C{am.x, T(0)});
            if (l) st_stream(out + (size_t)(nx - m) * ys, C{-am.y, T(0)});
        }
    }
}

// ------------------------------------------------------------- x inverse
// S1 -> rows of p, stored or accumulated; statistics as pass_xinv, one slot
// per wave.
template <typename T, int MODE, int M> __device__ __forceinline__ void fft_xinv(const Dom &d, int tile, char *smem)
{
    using C = c2<T>;
    constexpr int L = fft_lines(M, sizeof(C)), NTH = fft_threads(M, sizeof(C)), LDC = lds_line(M), STEP = NTH / L;
    static_assert(NTH % L == 0, "a thread keeps its row in the corner turn");
    C *buf = (C *)smem, *ltw = buf + L * LDC;
    TwStage<T, NTH> tws;
    tws.fetch(d.fx);
    const int nx = d.nx, ys = d.ys;
    const int q0 = tile * L, r = threadIdx.x % L, l0 = threadIdx.x / L;
    const bool wx = d.bcx != BC_PER;
    {
        // Z[l] = E + i O, E = X[l] + conj(X[M-l]), O = (X[l] - conj(X[M-l]))
        // conj(W^l); Z[M-l] = conj(E) + i conj(O): the thread that loads both
        // modes forms both points on their way into LDS.  (Formed by the
        // first stage's butterflies, they took 2 LDS reads and a root a
        // point and up to 128 registers, a tile less per CU at many
        // lengths: nx = 576, 34 M cells, 141 us against 102; 972, 167 and 114)
        const XLine x = xline(d, q0 + r);
        const C *in = (const C *)d.s1 + (size_t)x.k * d.nl * ys + x.j, *twr = (const C *)d.twr;
        C *mine = buf + r * LDC;
        constexpr int K = (M / 2 + 1 + STEP - 1) / STEP;
        auto pair = [&](int l, C xl, C xm, C w) {
            if (l == 0) {
                // X[0] and X[M] of a real row are real
                mine[0] = C{xl.x + xm.x, xl.x - xm.x};
                return;
            }
            const C e = {xl.x + xm.x, xl.y - xm.y}, df = {xl.x - xm.x, xl.y + xm.y};
            const C o = cmul(df, cconj(w));
            mine[pidx(l)] = C{e.x - o.y, e.y + o.x};
            if (2 * l != M) mine[pidx(M - l)] = C{e.x + o.y, o.x - e.y};
        };
        C w[K];
#pragma unroll
        for (int t = 0; t < K; ++t) w[t] = twr[min(l0 + t * STEP, M / 2)];
        if (!wx) {
            C a[K], b[K];
#pragma unroll
            for (int t = 0; t < K; ++t) {
                const int l = min(l0 + t * STEP, M / 2);
                a[t] = in[(size_t)l * ys];
                b[t] = in[(size_t)(M - l) * ys];
            }
#pragma unroll
            for (int t = 0; t < K; ++t)
                if (l0 + t * STEP <= M / 2) pair(l0 + t * STEP, a[t], b[t], w[t]);
        } else {
            // real modes X: V_k = conj(W_{4N}^k) (X_k - i X_{N-k}), k in [1, M),
            // V_0 = X_0 and V_M = conj(w_M) (1 - i) X_M, both real
            const C *wd = (const C *)d.dctx;
            T a[K][2], b[K][2]; // X_l, X_{N-l}; X_{M-l}, X_{M+l}
#pragma unroll
            for (int t = 0; t < K; ++t) {
                const int l = min(l0 + t * STEP, M / 2);
                a[t][0] = in[(size_t)l * ys].x;
                a[t][1] = in[(size_t)(nx - max(l, 1)) * ys].x;
                b[t][0] = in[(size_t)(M - l) * ys].x;
                b[t][1] = in[(size_t)(M + l) * ys].x;
            }
#pragma unroll
            for (int t = 0; t < K; ++t) {
                const int l = l0 + t * STEP;
                if (l > M / 2) continue;
                const C vl = l ? cmul(cconj(wd[l]), C{a[t][0], -a[t][1]}) : C{a[t][0], T(0)};
                pair(l, vl, cmul(cconj(wd[M - l]), C{b[t][0], -b[t][1]}), w[t]);
            }
        }
    }
    tws.put(ltw, d.fx);
    __syncthreads();
    const LineFft<T, true, M, L, NTH> F{buf, ltw};
    F.template first<false, true>([&](int line, int n) { return buf[line * LDC + pidx(n)]; });
    F.middles();
    // accumulation also removes the FP64 volume mean of the previous p
    const double shift = MODE == XOUT_ACCUM ? d.pmean[0] : 0.0;
    double emax = 0.0, pmax = 0.0, psum = 0.0;
    double2 *po2 = (double2 *)d.po;
    auto old_p = [&](int line, int h) {
        const XLine x = xline(d, q0 + line);
        return po2[((size_t)x.k * d.ny + x.j) * M + h];
    };
    auto emit = [&](int line, int h, double2 val, double2 old) {
        const XLine x = xline(d, q0 + line);
        if (!x.on) return;
        const double2 pv = MODE == XOUT_ACCUM ? double2{(old.x - shift) + val.x, (old.y - shift) + val.y} : val;
        st_stream(po2 + ((size_t)x.k * d.ny + x.j) * M + h, pv);
        if (d.ppart) psum += (pv.x + pv.y) * d.dzf[x.k];
        emax = amax_nan(amax_nan(emax, val.x), val.y);
        if (MODE == XOUT_ACCUM) pmax = amax_nan(amax_nan(pmax, pv.x), pv.y);
    };
    if (!wx) {
        // accumulate: a round's old p is read ahead of its points
        double2 old[9];
        auto wr = [&](int line, int n, C v, int r) { emit(line, n, double2{(double)v.x, (double)v.y}, old[r]); };
        if constexpr (MODE == XOUT_ACCUM) F.last(wr, [&](int r, int line, int n) { old[r] = old_p(line, n); });
        else F.last(wr, NoPre());
    } else {
        F.last();
        const double odd = d.bcx == BC_DIR ? -1.0 : 1.0;
        constexpr int K = (L * M + NTH - 1) / NTH, G = 4;
#pragma unroll 1
        for (int t0 = 0; t0 < K; t0 += G) {
            double2 old[G];
#pragma unroll
            for (int t = 0; t < G; ++t) {
                const int e = min((int)threadIdx.x + (t0 + t) * NTH, L * M - 1);
                if (MODE == XOUT_ACCUM) old[t] = old_p(e / M, e % M);
            }
#pragma unroll
            for (int t = 0; t < G; ++t) {
                const int e = threadIdx.x + (t0 + t) * NTH, line = e / M, h = e - line * M;
                if (e >= L * M) break;
                const T *z = (const T *)(buf + line * LDC);
                auto real = [&](int m) { return (double)z[2 * pidx(m >> 1) + (m & 1)]; };
                emit(line, h, double2{real(h), odd * real(nx - 1 - h)}, old[t]);
            }
        }
    }
    if (MODE == XOUT_STORE) pmax = emax; // a stored p is the update itself
    const int slot = tile * (NTH / 64) + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (d.ppart) {
        const double ws = wave_sum(psum);
        if (lane == 0) d.ppart[slot] = ws;
    }
    emax = wave_max1(emax);
    pmax = MODE == XOUT_STORE ? emax : wave_max1(pmax);
    if (lane == 0) ((double2 *)d.xpart)[slot] = double2{emax, pmax};
}

// ------------------------------------------------------------- y passes
// Column of a y tile: mode l and plane k of line q = l zs + k; on: as XLine
struct YLine {
    int l, k;
    bool on;
};
__device__ __forceinline__ YLine yline(const Dom &d, int q)
{
    const int l = q / d.zs, k = q - l * d.zs;
    return YLine{min(l, d.nl - 1), min(k, d.nz - 1), l < d.nl && k < d.nz};
}

// S1 -> FFT (cosine transform) in y -> S2
template <typename T, int N> __device__ __forceinline__ void fft_yfwd(const Dom &d, int tile, char *smem)
{
    using C = c2<T>;
    constexpr int L = fft_lines(N, sizeof(C)), NTH = fft_threads(N, sizeof(C)), LDC = lds_line(N), STEP = NTH / L;
    static_assert(NTH % L == 0, "a thread keeps its column in the corner turn");
    C *buf = (C *)smem, *ltw = buf + L * LDC;
    TwStage<T, NTH> tws;
    tws.fetch(d.fy);
    const int nl = d.nl, q0 = tile * L;
    const bool wy = d.bcy != BC_PER, dy = d.bcy == BC_DIR;
    const C *s1 = (const C *)d.s1;
    auto col = [&](int line) {
        const YLine y = yline(d, q0 + line);
        return s1 + ((size_t)y.k * nl + y.l) * d.ys;
    };
    tws.put(ltw, d.fy);
    const LineFft<T, false, N, L, NTH> F{buf, ltw};
    if (!wy) {
        F.template first<false, false>([&](int line, int n) { return ld_stream(col(line) + n); });
    } else {
        // reordered: v[n] = c[2n], v[N-1-n] = c[2n+1] (times -1 for the sine
        // transform), through LDS: read in that order from memory, a wave
        // takes every other point (338 against 250 us for 288 x 250 x 384)
        constexpr int K = (L * N + NTH - 1) / NTH;
        C v[K];
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int e = min((int)threadIdx.x + t * NTH, L * N - 1), line = e / N;
            v[t] = ld_stream(col(line) + (e - line * N));
        }
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int e = threadIdx.x + t * NTH, line = e / N, j = e - line * N;
            if ((L * N) % NTH && e >= L * N) continue;
            buf[line * LDC + pidx((j & 1) ? N - 1 - (j >> 1) : (j >> 1))] = dy && (j & 1) ? C{-v[t].x, -v[t].y} : v[t];
        }
        __syncthreads();
        F.template first<false, true>([&](int line, int n) { return buf[line * LDC + pidx(n)]; });
    }
    F.middles();
    const int c = threadIdx.x % L, m0 = threadIdx.x / L;
    // walls: X_m = (w_m V_m + conj(w_m) V_{N-m}) / 2, X_0 = V_0, and with
    // w_{N-m} = -i conj(w_m) the other point of the pair by the same thread
    const C *wd = (const C *)d.dcty;
    constexpr int KW = (N / 2 + 1 + STEP - 1) / STEP;
    F.last();
    const YLine y = yline(d, q0 + c);
    const int zs = d.zs;
    C *out = (C *)d.s2 + (size_t)y.l * N * zs + y.k;
    const C *z = buf + c * LDC;
    constexpr int K = (N + STEP - 1) / STEP;
    const bool on = y.on;
    if (!wy) {
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int m = m0 + t * STEP;
            if (on && (N % STEP == 0 || m < N)) st_stream(out + (size_t)m * zs, z[pidx(m)]);
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < KW; ++t) {
        const int m = m0 + t * STEP;
        if (!on || m > N / 2) continue;
        if (m == 0) {
            st_stream(out, z[0]);
            continue;
        }
        const C w = wd[m], pv = cmul(w, z[pidx(m)]), g = cmul(cconj(w), z[pidx(N - m)]);
        st_stream(out + (size_t)m * zs, C{T(0.5) * (pv.x + g.x), T(0.5) * (pv.y + g.y)});
        if (2 * m != N) st_stream(out + (size_t)(N - m) * zs, C{T(0.5) * (g.y - pv.y), T(0.5) * (pv.x - g.x)});
    }
}

// S2 -> inverse FFT (cosine transform) in y -> S1
template <typename T, int N> __device__ __forceinline__ void fft_yinv(const Dom &d, int tile, char *smem)
{
    using C = c2<T>;
    constexpr int L = fft_lines(N, sizeof(C)), NTH = fft_threads(N, sizeof(C)), LDC = lds_line(N), STEP = NTH / L;
    static_assert(NTH % L == 0, "a thread keeps its column in the corner turn");
    C *buf = (C *)smem, *ltw = buf + L * LDC;
    TwStage<T, NTH> tws;
    tws.fetch(d.fy);
    const int nl = d.nl, q0 = tile * L;
    const bool wy = d.bcy != BC_PER, dy = d.bcy == BC_DIR;
    C *s1 = (C *)d.s1;
    const int c = threadIdx.x % L;
    const YLine y = yline(d, q0 + c);
    const int zs = d.zs;
    const C *in = (const C *)d.s2 + (size_t)y.l * N * zs + y.k;
    tws.put(ltw, d.fy);
    const LineFft<T, true, N, L, NTH> F{buf, ltw};
    if (!wy) {
        // the first stage's threads take consecutive lines (thread % L is
        // their line in every round), whose points are contiguous in S2
        F.template first<true, false>([&](int, int n) { return ld_stream(in + (size_t)n * zs); });
        F.middles();
        F.last(
            [&](int line, int n, C v, int) {
                const YLine o = yline(d, q0 + line);
                if (o.on) st_stream(s1 + ((size_t)o.k * nl + o.l) * d.ys + n, v);
            },
            NoPre());
        return;
    }
    // V_m = conj(w_m) (X_m - i X_{N-m}), X_N = 0, and with conj(w_{N-m}) = i
    // w_m the other point of the pair, formed by the thread that loads both
    // (as in the x inverse)
    constexpr int K = (N / 2 + 1 + STEP - 1) / STEP;
    {
        const C *wd = (const C *)d.dcty;
        const int m0 = threadIdx.x / L;
        C *mine = buf + c * LDC;
        C xa[K], xb[K], w[K];
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int m = min(m0 + t * STEP, N / 2);
            xa[t] = ld_stream(in + (size_t)m * zs);
            xb[t] = ld_stream(in + (size_t)(N - max(m, 1)) * zs);
            w[t] = wd[m];
        }
#pragma unroll
        for (int t = 0; t < K; ++t) {
            const int m = m0 + t * STEP;
            if (m > N / 2) continue;
            if (m == 0) {
                mine[0] = xa[t];
                continue;
            }
            mine[pidx(m)] = cmul(cconj(w[t]), C{xa[t].x + xb[t].y, xa[t].y - xb[t].x});
            const C g = cmul(w[t], C{xb[t].x + xa[t].y, xb[t].y - xa[t].x});
            if (2 * m != N) mine[pidx(N - m)] = C{-g.y, g.x};
        }
    }
    __syncthreads();
    F.template first<false, true>([&](int line, int n) { return buf[line * LDC + pidx(n)]; });
    F.middles();
    F.last();
    constexpr int KO = (L * N + NTH - 1) / NTH;
#pragma unroll 4
    for (int t = 0; t < KO; ++t) {
        const int e = threadIdx.x + t * NTH, line = e / N, j = e - line * N;
        if (e >= L * N) break;
        const YLine o = yline(d, q0 + line);
        if (!o.on) continue;
        C v = buf[line * LDC + pidx((j & 1) ? N - 1 - (j >> 1) : (j >> 1))];
        if (dy && (j & 1)) v = C{-v.x, -v.y};
        st_stream(s1 + ((size_t)o.k * nl + o.l) * d.ys + j, v);
    }
}

// --------------------------------------------------------------- kernels
enum { FK_XFWD = 0, FK_XINV_STORE, FK_XINV_ACCUM, FK_YFWD, FK_YINV };

template <typename T, int KIND, int N>
__device__ __forceinline__ void fft_pass(const Dom &d, const double *src, int tile, char *smem)
{
    if constexpr (KIND == FK_XFWD) fft_xfwd<T, N>(d, src, tile, smem);
    else if constexpr (KIND == FK_XINV_STORE) fft_xinv<T, XOUT_STORE, N>(d, tile, smem);
    else if constexpr (KIND == FK_XINV_ACCUM) fft_xinv<T, XOUT_ACCUM, N>(d, tile, smem);
    else if constexpr (KIND == FK_YFWD) fft_yfwd<T, N>(d, tile, smem);
    else fft_yinv<T, N>(d, tile, smem);
}

constexpr int fft_kernel_threads(int n, int csz)
{
    return n ? (fft_threads(n, csz) <= 1024 ? fft_threads(n, csz) : throw "more threads than a workgroup has") : FSMALL_TH;
}

constexpr int fft_kernel_waves(int n, int csz) { return n ? fft_waves(n, csz) : 4; }

// One kernel for a lone domain (the descriptor in the kernel arguments, a
// tile per workgroup) and for a batch (an item per workgroup); both read the
// descriptor through the constant address space.  There is no loop over
// items: the compiler keeps every index of the pass that does not change
// between items in registers across such a loop (the general x pass takes
// 216 VGPRs with one and 80 without).  N = 0: every length up to FSMALL, by
// the domain's own.
template <typename T, int KIND, int N>
__global__ __launch_bounds__(fft_kernel_threads(N, 2 * sizeof(T))) __attribute__((amdgpu_waves_per_eu(fft_kernel_waves(N, 2 * sizeof(T))))) void
k_fft(FftArgs unused)
{
    extern __shared__ __align__(16) char smem[];
    typedef const __attribute__((address_space(4))) FftArgs *Arg;
    const Arg A = (Arg)__builtin_amdgcn_kernarg_segment_ptr();
    int tile = blockIdx.x;
    // Column tiles of 64-byte segments: consecutive workgroups go to
    // different XCDs, so workgroups b and b + 8 take the two halves of the
    // same 128-byte lines and meet in one XCD's L2.
    if constexpr ((KIND == FK_YFWD || KIND == FK_YINV) && N > 0) {
        if constexpr (fft_lines(N, 2 * sizeof(T)) * 2 * sizeof(T) < 128) {
            const int full = (int)gridDim.x & ~15;
            if (tile < full) tile = (tile & ~15) + 2 * (tile & 7) + ((tile >> 3) & 1);
        }
    }
    const __attribute__((address_space(4))) Dom *p = &A->d;
    if (A->g.items) {
        p = (const __attribute__((address_space(4))) Dom *)A->g.doms + __builtin_amdgcn_readfirstlane((int)A->g.items[tile].dom);
        tile = __builtin_amdgcn_readfirstlane((int)A->g.items[tile].tile);
    }
    const Dom &d = *(const Dom *)p;
    const double *src = A->resid ? d.r : d.f;
    if constexpr (N > 0) {
        fft_pass<T, KIND, N>(d, src, tile, smem);
    } else {
        switch (KIND == FK_YFWD || KIND == FK_YINV ? d.ny : d.M) {
        case 16: fft_pass<T, KIND, 16>(d, src, tile, smem); break;
        case 18: fft_pass<T, KIND, 18>(d, src, tile, smem); break;
        case 24: fft_pass<T, KIND, 24>(d, src, tile, smem); break;
        case 27: fft_pass<T, KIND, 27>(d, src, tile, smem); break;
        case 32: fft_pass<T, KIND, 32>(d, src, tile, smem); break;
        case 36: fft_pass<T, KIND, 36>(d, src, tile, smem); break;
        case 48: fft_pass<T, KIND, 48>(d, src, tile, smem); break;
        case 54: fft_pass<T, KIND, 54>(d, src, tile, smem); break;
        case 64: fft_pass<T, KIND, 64>(d, src, tile, smem); break;
        case 72: fft_pass<T, KIND, 72>(d, src, tile, smem); break;
        case 81: fft_pass<T, KIND, 81>(d, src, tile, smem); break;
        case 96: fft_pass<T, KIND, 96>(d, src, tile, smem); break;
        case 108: fft_pass<T, KIND, 108>(d, src, tile, smem); break;
        case 128: fft_pass<T, KIND, 128>(d, src, tile, smem); break;
        default: break;
        }
    }
}

// Kernel of a length (NULL: no fixed plan)
template <typename T, int KIND> static const void *fft_kernel(int n)
{
    if (n <= FSMALL) return fplan(n).n ? (const void *)k_fft<T, KIND, 0> : nullptr;
    constexpr bool Y = KIND == FK_YFWD || KIND == FK_YINV;
    switch (n) {
#define PCX_FFT_LEN(N) case N: return (const void *)k_fft<T, KIND, N>;
    PCX_FFT_LEN(144) PCX_FFT_LEN(162) PCX_FFT_LEN(192) PCX_FFT_LEN(216) PCX_FFT_LEN(243) PCX_FFT_LEN(256)
    PCX_FFT_LEN(288) PCX_FFT_LEN(324) PCX_FFT_LEN(384) PCX_FFT_LEN(432) PCX_FFT_LEN(486) PCX_FFT_LEN(512)
#undef PCX_FFT_LEN
    }
    if constexpr (Y) {
        switch (n) {
#define PCX_FFT_LEN(N) case N: return (const void *)k_fft<T, KIND, N>;
        PCX_FFT_LEN(576) PCX_FFT_LEN(648) PCX_FFT_LEN(729) PCX_FFT_LEN(768) PCX_FFT_LEN(864) PCX_FFT_LEN(972)
        PCX_FFT_LEN(1024)
#undef PCX_FFT_LEN
        }
    }
    return nullptr;
}

} // namespace pcx
