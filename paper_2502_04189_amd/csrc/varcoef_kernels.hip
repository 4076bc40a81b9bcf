// varcoef_kernels.hip -- kernels of the variable-coefficient projection
// D((1/rho_f) G p) = (D u*) / dt solved by preconditioned conjugate gradients
// (the preconditioner is the constant-coefficient solve of the plan, run by
// the host between these kernels).  The operator marches in z over tiles of
// its own; the vector kernels take the cells in memory order with at most
// RED_MAX workgroups; the correction runs one thread per cell on the plane
// tiles of flow_tile.hpp.  The inner products are volume-weighted (the dzf factor; dx dy is common to all cells
// and cancels in every ratio the iteration takes) and are reduced in a fixed
// order, so a run is deterministic.  The iteration's scalars stay in device
// memory: no kernel waits for the host.
#include "varcoef_launch.hpp"

namespace pcx {
namespace vc {

using namespace pcx::flow;

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// sums a and b over the workgroup of NTH threads (fixed order); every
// thread gets the sums
template <int NTH> __device__ __forceinline__ void block_sum2(double &a, double &b)
{
    __shared__ double red[2][NTH / 64];
    a = wave_sum(a);
    b = wave_sum(b);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wv] = a;
        red[1][wv] = b;
    }
    __syncthreads();
    a = red[0][0];
    b = red[1][0];
#pragma unroll
    for (int i = 1; i < NTH / 64; ++i) {
        a += red[0][i];
        b += red[1][i];
    }
    __syncthreads(); // red is written again by a second call
}

template <int NTH> __device__ __forceinline__ void put2(const VRed &R, double a, double b)
{
    block_sum2<NTH>(a, b);
    if (threadIdx.x == 0) {
        R.part[blockIdx.x] = a;
        R.part[R.nb + blockIdx.x] = b;
    }
}

// the total of the partials of an earlier kernel, for every thread; the
// second sum only with TWO
template <int NTH, bool TWO> __device__ __forceinline__ void get2(const VRed &R, double &a, double &b)
{
    a = b = 0.0;
    for (int i = threadIdx.x; i < R.nb; i += NTH) {
        a += R.part[i];
        if (TWO) b += R.part[R.nb + i];
    }
    block_sum2<NTH>(a, b);
}

// (1/rho_f) G p on the +D face of the cell s steps along D; 0 on a wall face
template <int D, class X, class R, class P> __device__ __forceinline__ double bflux(const X &x, R rho, P p, int s)
{
    const double f = cgrad<D>(x, p, s) / cface<D>(x, rho, s);
    return x.template wall<D>(s) ? 0.0 : f;
}

// D u at the cell (wall faces carry no flux)
template <class X>
__device__ __forceinline__ double div_cell(const X &x, const double *u, const double *v, const double *w)
{
    return (x.template fv<0>(u, 0, 0, 0) - x.template fv<0>(u, -1, 0, 0)) * x.ih(0) +
           (x.template fv<1>(v, 0, 0, 0) - x.template fv<1>(v, 0, -1, 0)) * x.ih(1) +
           (x.template fv<2>(w, 0, 0, 0) - x.template fv<2>(w, 0, 0, -1)) * x.izf(0);
}

// out = sign D((1/rho_f) G p); with R, partial sums of dzf p out.
// A workgroup marches its tiles' columns upwards with two planes of rho and p
// (tile and one cell of halo) in LDS.  Each face's (1/rho_f) G p is evaluated
// once (plus the tile's west and south edge): the east and north ones of
// plane k + 1 go to LDS while plane k is put together, the top one stays in a
// register; one barrier per plane.  Six divisions per cell, and neighbours
// fetched by every thread, took 25 us at 128^3 (50 MB) on the plane tiles;
// 18 us here.  A wall's face is 0 whatever the halo holds, so all grids run
// this code.
constexpr int ASX = MAI + 2, ASN = ASX * (MAJ + 2);
static_assert(ASN <= 2 * MAT, "two items per thread");
__global__ __launch_bounds__(MAT) void k_vc_apply(FGrid G, ATiles T, const double *rho, const double *p, double *out,
                                                  double sign, VRed R, int want)
{
    __shared__ double sr[2][ASN], sp[2][ASN], sx[2][MAJ * (MAI + 1)], sy[2][(MAJ + 1) * MAI];
    const int nx = G.n[0], ny = G.n[1], nz = G.n[2];
    const size_t sz = (size_t)nx * ny;
    const int tid = threadIdx.x, tx = tid & (MAI - 1), ty = tid / MAI;
    const int me = (ty + 1) * ASX + tx + 1;
    const int q1 = min(tid + MAT, ASN - 1); // second item of a plane
    auto wrapk = [&](int k) { return k < 0 ? (G.per[2] ? nz - 1 : 0) : (k >= nz ? (G.per[2] ? 0 : nz - 1) : k); };
    double acc = 0.0;
    // an XCD's workgroups take a contiguous range of the tiles
    const int per = (T.n + 7) >> 3;
    for (int m = blockIdx.x >> 3; m < per; m += (int)(gridDim.x >> 3)) {
        const int tile = (int)(blockIdx.x & 7) * per + m;
        if (tile >= T.n) break;
        const int ch = tile / (T.nti * T.ntj), rem = tile - ch * (T.nti * T.ntj), jt = rem / T.nti;
        const int i0 = (rem - jt * T.nti) * MAI, j0 = jt * MAJ, i = i0 + tx, j = j0 + ty;
        const int kb = ch * T.ckc, ke = min(kb + T.ckc, nz);
        const bool act = i < nx && j < ny;
        // in-plane offset of cell (i0 + a, j0 + c): wrapped once across a
        // periodic direction; beyond a wall or a partial tile any valid cell
        auto off = [&](int a, int c) {
            int x = i0 + a, y = j0 + c;
            if (G.per[0]) x = x < 0 ? x + nx : (x == nx ? 0 : x);
            if (G.per[1]) y = y < 0 ? y + ny : (y == ny ? 0 : y);
            return (size_t)min(max(y, 0), ny - 1) * nx + min(max(x, 0), nx - 1);
        };
        const size_t o0 = off(tid % ASX - 1, tid / ASX - 1), o1 = off(q1 % ASX - 1, q1 / ASX - 1);
        const bool we = wallf(G, 0, i), wn = wallf(G, 1, j);
        const bool ww = !G.per[0] && i0 == 0, ws = !G.per[1] && j0 == 0;
        // (1/rho_f) G p on the faces of the plane in slot b: own east and
        // north; by the first waves the tile's south edge, then its west
        auto faces = [&](int b) {
            const double *r = sr[b], *q = sp[b];
            const double r0 = r[me], p0 = q[me];
            const double fe = (q[me + 1] - p0) * G.ih[0] / (0.5 * (r0 + r[me + 1]));
            const double fn = (q[me + ASX] - p0) * G.ih[1] / (0.5 * (r0 + r[me + ASX]));
            sx[b][ty * (MAI + 1) + tx + 1] = we ? 0.0 : fe;
            sy[b][(ty + 1) * MAI + tx] = wn ? 0.0 : fn;
            if (tid < MAI + MAJ) {
                const bool south = tid < MAI;
                const int c = south ? tid + 1 : (tid - MAI + 1) * ASX, n = south ? c + ASX : c + 1;
                const double f = (q[n] - q[c]) * (south ? G.ih[1] : G.ih[0]) / (0.5 * (r[c] + r[n]));
                if (south) sy[b][tid] = ws ? 0.0 : f;
                else sx[b][(tid - MAI) * (MAI + 1)] = ww ? 0.0 : f;
            }
        };
        // plane kb into its slot, the next one in flight; the face below kb
        // from the own column
        const size_t own = act ? (size_t)j * nx + i : 0;
        size_t pl = (size_t)kb * sz;
        double r0 = rho[pl + o0], r1 = rho[pl + o1], p0 = p[pl + o0], p1 = p[pl + o1];
        const int kl = wrapk(kb - 1);
        const double rl = rho[(size_t)kl * sz + own], ql = p[(size_t)kl * sz + own];
        const double ro = rho[pl + own], qo = p[pl + own];
        __syncthreads(); // the tile before this one has read its last planes
        sr[kb & 1][tid] = r0;
        sp[kb & 1][tid] = p0;
        if (tid + MAT < ASN) {
            sr[kb & 1][tid + MAT] = r1;
            sp[kb & 1][tid + MAT] = p1;
        }
        pl = (size_t)wrapk(kb + 1) * sz;
        r0 = rho[pl + o0];
        r1 = rho[pl + o1];
        p0 = p[pl + o0];
        p1 = p[pl + o1];
        double dz0 = G.dzf[kb], fb = 0.0;
        if (G.per[2] || kb > 0) {
            const double izc = G.rz[6 * (size_t)kb + 2], dzl = G.dzf[kl];
            fb = (qo - ql) * izc / ((rl * dz0 + ro * dzl) * (0.5 * izc));
        }
        __syncthreads();
        faces(kb & 1);
        for (int k = kb; k < ke; ++k) {
            const int b = k & 1;
            sr[b ^ 1][tid] = r0;
            sp[b ^ 1][tid] = p0;
            if (tid + MAT < ASN) {
                sr[b ^ 1][tid + MAT] = r1;
                sp[b ^ 1][tid + MAT] = p1;
            }
            // the last planes of the chunk are read, not used
            pl = (size_t)wrapk(min(k + 2, ke)) * sz;
            r0 = rho[pl + o0];
            r1 = rho[pl + o1];
            p0 = p[pl + o0];
            p1 = p[pl + o1];
            const double rc = sr[b][me], pc = sp[b][me];
            __syncthreads();
            if (k + 1 < ke) faces(b ^ 1);
            const double dzp = G.dzf[wrapk(k + 1)], izc = G.rz[6 * (size_t)k + 3];
            double ft = (sp[b ^ 1][me] - pc) * izc / ((rc * dzp + sr[b ^ 1][me] * dz0) * (0.5 * izc));
            if (!G.per[2] && k == nz - 1) ft = 0.0;
            const double *fx = sx[b] + ty * (MAI + 1) + tx, *fy = sy[b] + ty * MAI + tx;
            const double q = sign * ((fx[1] - fx[0]) * G.ih[0] + (fy[MAI] - fy[0]) * G.ih[1] +
                                     (ft - fb) * G.rz[6 * (size_t)k]);
            if (act) {
                out[(size_t)k * sz + (size_t)j * nx + i] = q;
                acc += dz0 * pc * q;
            }
            fb = ft;
            dz0 = dzp;
        }
    }
    if (want) put2<MAT>(R, acc, 0.0);
}

// The vector kernels take the cells in memory order, four per thread and
// round, loaded before the first is stored.  With one cell per thread every
// kernel left a partial per 256 cells, and each sum took two more launches (9
// us of the iteration's chain at 128^3, three times); with RED_MAX workgroups
// at most the update takes 18 us (101 MB, 5.7 TB/s) as before, the dot 10
// instead of 12 without r to store.
// Beyond 2^24 cells every workgroup takes 1024 consecutive cells in one round:
// workgroups that come in order keep the launch's reads and writes together
// in memory, and the two folds of their partials cost 10 us.  At 512^3 update
// 1.23 -> 1.15 ms, direction 0.62 -> 0.55, dot 0.40 -> 0.35; an iteration of
// 288 x 256 x 256 843 -> 828 us, of 384^3 2.39 -> 2.31 ms (256^3 alike either way).
struct VCells {
    unsigned n, plane, c, step, next; // step: between the four cells of a round, next: between rounds
    __device__ explicit VCells(const FGrid &G)
        : n((unsigned)G.n[0] * (unsigned)G.n[1] * (unsigned)G.n[2]), plane((unsigned)G.n[0] * (unsigned)G.n[1]),
          next(4 * FT * gridDim.x) // n below 2^31 (grid validation)
    {
        const bool blocks = gridDim.x > RED_MAX; // one round
        c = blockIdx.x * (blocks ? 4 * FT : FT) + threadIdx.x;
        step = blocks ? FT : gridDim.x * FT;
    }
    // f(cells, in[]): every round of the thread, cells past the end clamped
    // to the last one
    template <class F> __device__ __forceinline__ void each(F &&f)
    {
        for (; c < n; c += next) {
            size_t x[4];
            bool in[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                in[u] = c + u * step < n;
                x[u] = in[u] ? c + u * step : n - 1;
            }
            f(x, in);
        }
    }
    __device__ __forceinline__ double weight(const FGrid &G, size_t x) const { return G.dzf[(unsigned)x / plane]; }
};
#define VC4 _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_)

// r = -(D u) / dt; partial sum of dzf r
__global__ __launch_bounds__(FT) void k_vc_rhs(FGrid G, const double *u, const double *v, const double *w, double idt,
                                               double *r, VRed R)
{
    VCells V(G);
    double a = 0.0;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double q[4];
        VC4
        {
            const unsigned k = (unsigned)x[u_] / V.plane, rem = (unsigned)x[u_] - k * V.plane;
            const unsigned j = rem / (unsigned)G.n[0];
            q[u_] = -div_cell(Gen{G, (int)(rem - j * (unsigned)G.n[0]), (int)j, (int)k}, u, v, w) * idt;
        }
        VC4 if (in[u_])
        {
            r[x[u_]] = q[u_];
            a += V.weight(G, x[u_]) * q[u_];
        }
    });
    put2<FT>(R, a, 0.0);
}

// r -= m; partial sum of dzf r^2
__global__ __launch_bounds__(FT) void k_vc_center(FGrid G, double *r, VRed R)
{
    VCells V(G);
    const double m = R.sc[S_M];
    double a = 0.0;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double q[4];
        VC4 q[u_] = r[x[u_]] - m;
        VC4 if (in[u_])
        {
            r[x[u_]] = q[u_];
            a += V.weight(G, x[u_]) * q[u_] * q[u_];
        }
    });
    put2<FT>(R, a, 0.0);
}

// d = -rho0 z (z: the constant-coefficient solve of r); partial dzf r d
__global__ __launch_bounds__(FT) void k_vc_dinit(FGrid G, const double *r, const double *z, double *d, double rho0,
                                                 VRed R)
{
    VCells V(G);
    double a = 0.0;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double q[4], rr[4];
        VC4
        {
            q[u_] = -rho0 * z[x[u_]];
            rr[u_] = r[x[u_]];
        }
        VC4 if (in[u_])
        {
            d[x[u_]] = q[u_];
            a += V.weight(G, x[u_]) * rr[u_] * q[u_];
        }
    });
    put2<FT>(R, a, 0.0);
}

// alpha = rz / (sum of the operator's partials); r -= the mean it drifted by;
// p += alpha d; r -= alpha q; partial sums of dzf r and dzf r^2
__global__ __launch_bounds__(FT) void k_vc_update(FGrid G, double *p, const double *d, double *r, const double *q,
                                                  VRed IN, VRed R)
{
    VCells V(G);
    const double rz = R.sc[S_RZN], m = R.sc[S_DRIFT];
    double dq, a, b;
    get2<FT, false>(IN, dq, a);
    const double al = rz / dq;
    if (blockIdx.x == 0 && threadIdx.x == 0) R.sc[S_RZ] = rz;
    a = b = 0.0;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double pv[4], dv[4], rv[4], qv[4];
        VC4
        {
            pv[u_] = p[x[u_]];
            dv[u_] = d[x[u_]];
            rv[u_] = r[x[u_]];
            qv[u_] = q[x[u_]];
        }
        VC4 if (in[u_])
        {
            p[x[u_]] = pv[u_] + al * dv[u_];
            const double rr = (rv[u_] - m) - al * qv[u_];
            r[x[u_]] = rr;
            const double wz = V.weight(G, x[u_]);
            a += wz * rr;
            b += wz * rr * rr;
        }
    });
    put2<FT>(R, a, b);
}

// partial dzf (r - m) (-rho0 z), m the mean the residual drifted by (the
// update takes it off r)
__global__ __launch_bounds__(FT) void k_vc_dot(FGrid G, const double *r, const double *z, double rho0, VRed R)
{
    VCells V(G);
    const double m = R.sc[S_DRIFT];
    double a = 0.0;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double rv[4], zv[4];
        VC4
        {
            rv[u_] = r[x[u_]];
            zv[u_] = z[x[u_]];
        }
        VC4 if (in[u_]) a += V.weight(G, x[u_]) * (rv[u_] - m) * (-rho0 * zv[u_]);
    });
    put2<FT>(R, a, 0.0);
}

// beta = (sum of the dot's partials) / rz; d = -rho0 z + beta d
__global__ __launch_bounds__(FT) void k_vc_dupd(FGrid G, const double *z, double *d, double rho0, VRed IN)
{
    VCells V(G);
    const double rz = IN.sc[S_RZ];
    double rzn, b;
    get2<FT, false>(IN, rzn, b);
    const double be = rzn / rz;
    if (blockIdx.x == 0 && threadIdx.x == 0) IN.sc[S_RZN] = rzn;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double q[4];
        VC4 q[u_] = -rho0 * z[x[u_]] + be * d[x[u_]];
        VC4 if (in[u_]) d[x[u_]] = q[u_];
    });
}

__global__ __launch_bounds__(FT) void k_vc_pmean(FGrid G, const double *p, VRed R)
{
    VCells V(G);
    double a = 0.0;
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double q[4];
        VC4 q[u_] = p[x[u_]];
        VC4 if (in[u_]) a += V.weight(G, x[u_]) * q[u_];
    });
    put2<FT>(R, a, 0.0);
}

__global__ __launch_bounds__(FT) void k_vc_pshift(FGrid G, double *p, VRed R)
{
    VCells V(G);
    const double m = R.sc[S_PMEAN];
    V.each([&](const size_t(&x)[4], const bool(&in)[4]) {
        double q[4];
        VC4 q[u_] = p[x[u_]] - m;
        VC4 if (in[u_]) p[x[u_]] = q[u_];
    });
}

// u_out = u - dt (1/rho_f) G p on the +face of each direction, 0 on a wall face
__global__ __launch_bounds__(FT) void k_vc_correct(BoxList L, FGrid G, const double *rho, const double *p, const double *u,
                                                   const double *v, const double *w, double dt, double *uo,
                                                   double *vo, double *wo)
{
    const BoxPick pk = box_pick(L);
    const FTile t = btile(G, pk.b, pk.w);
    if (!t.act) return;
    const size_t c = at(G, t.i, t.j, t.k);
    double gx = 0.0, gy = 0.0, gz = 0.0;
    auto flux = [&](const auto &x) {
        gx = bflux<0>(x, rho, p, 0);
        gy = bflux<1>(x, rho, p, 0);
        gz = bflux<2>(x, rho, p, 0);
    };
    if (pk.fast) flux(Fast(G, t.i, t.j, t.k));
    else flux(Gen{G, t.i, t.j, t.k});
    uo[c] = wallf(G, 0, t.i) ? 0.0 : u[c] - dt * gx;
    vo[c] = wallf(G, 1, t.j) ? 0.0 : v[c] - dt * gy;
    wo[c] = wallf(G, 2, t.k) ? 0.0 : w[c] - dt * gz;
}

// the partials R.part in RED_FOLD pairs of sums
__global__ __launch_bounds__(FT) void k_vc_fold(VRed R)
{
    double a = 0.0, b = 0.0;
    for (int i = blockIdx.x * FT + threadIdx.x; i < R.nb; i += RED_FOLD * FT) {
        a += R.part[i];
        b += R.part[R.nb + i];
    }
    block_sum2<FT>(a, b);
    if (threadIdx.x == 0) {
        R.fold[blockIdx.x] = a;
        R.fold[RED_FOLD + blockIdx.x] = b;
    }
}

// the totals and the scalar step of the iteration, one workgroup
__global__ __launch_bounds__(RED_MAX) void k_vc_scal(VRed R, int mode, double *host)
{
    double a, b;
    get2<RED_MAX, true>(R, a, b);
    if (threadIdx.x != 0) return;
    double *sc = R.sc;
    switch (mode) {
    case MODE_MEAN: sc[S_M] = a / sc[S_WTOT]; break;
    case MODE_BNORM:
        sc[S_BNORM] = sqrt(a);
        sc[S_RES] = a > 0.0 && a < INFINITY ? 1.0 : a; // 0, or a norm that is not finite
        sc[S_DRIFT] = 0.0;
        break;
    case MODE_RZ: sc[S_RZN] = a; break;
    case MODE_RES: {
        const double m = a / sc[S_WTOT];
        sc[S_DRIFT] = m;
        // sum dzf (r - m)^2 = sum dzf r^2 - m sum dzf r, below 0 by rounding
        // only; NaN goes through (the host's stop test sees nothing else)
        const double t = b - m * a;
        const double res = sqrt(t < 0.0 ? 0.0 : t) / sc[S_BNORM];
        sc[S_RES] = res;
        if (host) __hip_atomic_store(host, res, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        break;
    }
    case MODE_PMEAN: sc[S_PMEAN] = a / sc[S_WTOT]; break;
    default: break;
    }
}

hipError_t launch_fold(const VRed &R, VRed &out, hipStream_t s)
{
    out = R;
    if (R.nb <= RED_MAX) return hipSuccess;
    if (!R.fold) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_vc_fold, dim3(RED_FOLD), dim3(FT), 0, s, R);
    out.part = R.fold;
    out.nb = RED_FOLD;
    return hipGetLastError();
}
hipError_t launch_apply(const FGrid &G, const ATiles &T, const double *rho, const double *p, double *out, double sign,
                        const VRed *R, hipStream_t s)
{
    if (R && R->nb != T.wgs) return hipErrorInvalidValue;
    const VRed r0{};
    hipLaunchKernelGGL(k_vc_apply, dim3(T.wgs), dim3(MAT), 0, s, G, T, rho, p, out, sign, R ? *R : r0, R ? 1 : 0);
    return hipGetLastError();
}
hipError_t launch_rhs(const FGrid &G, const double *u, const double *v, const double *w, double idt, double *r,
                      const VRed &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_rhs, dim3(R.nb), dim3(FT), 0, s, G, u, v, w, idt, r, R);
    return hipGetLastError();
}
hipError_t launch_center(const FGrid &G, double *r, const VRed &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_center, dim3(R.nb), dim3(FT), 0, s, G, r, R);
    return hipGetLastError();
}
hipError_t launch_dinit(const FGrid &G, const double *r, const double *z, double *d, double rho0, const VRed &R,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_dinit, dim3(R.nb), dim3(FT), 0, s, G, r, z, d, rho0, R);
    return hipGetLastError();
}
hipError_t launch_update(const FGrid &G, double *p, const double *d, double *r, const double *q, const VRed &IN,
                         const VRed &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_update, dim3(R.nb), dim3(FT), 0, s, G, p, d, r, q, IN, R);
    return hipGetLastError();
}
hipError_t launch_dot(const FGrid &G, const double *r, const double *z, double rho0, const VRed &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_dot, dim3(R.nb), dim3(FT), 0, s, G, r, z, rho0, R);
    return hipGetLastError();
}
hipError_t launch_dupd(const FGrid &G, const double *z, double *d, double rho0, const VRed &IN, int nv, hipStream_t s)
{
    VRed t;
    const hipError_t e = launch_fold(IN, t, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_vc_dupd, dim3(nv), dim3(FT), 0, s, G, z, d, rho0, t);
    return hipGetLastError();
}
hipError_t launch_pmean(const FGrid &G, const double *p, const VRed &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_pmean, dim3(R.nb), dim3(FT), 0, s, G, p, R);
    return hipGetLastError();
}
hipError_t launch_correct(const FGrid &G, const TilePlan &tp, const double *rho, const double *p, const double *u,
                          const double *v, const double *w, double dt, double *uo, double *vo, double *wo,
                          hipStream_t s)
{
    return FLOW_LAUNCH_PLAN(tp, k_vc_correct, s, G, rho, p, u, v, w, dt, uo, vo, wo);
}
hipError_t launch_pshift(const FGrid &G, double *p, const VRed &R, hipStream_t s)
{
    hipLaunchKernelGGL(k_vc_pshift, dim3(R.nb), dim3(FT), 0, s, G, p, R);
    return hipGetLastError();
}
hipError_t red_scal(const VRed &R, int mode, hipStream_t s, double *host)
{
    VRed t;
    const hipError_t e = launch_fold(R, t, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_vc_scal, dim3(1), dim3(RED_MAX), 0, s, t, mode, host);
    return hipGetLastError();
}

} // namespace vc
} // namespace pcx
