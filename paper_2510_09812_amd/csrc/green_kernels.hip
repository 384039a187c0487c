// Node and grid passes of the elastic preconditioner B = Q A_g^+ Q^T + omega
// D^-1 (elastic_precond; host setup in green.cpp): the restriction Q^T to the
// auxiliary grid, the mode-by-mode inverse of the grid operator between the
// two FFTs, the prolongation Q back to the nodes with the diagonal term, and
// the CG vector update of the preconditioned iteration.  Node vectors are
// component-major [3][n], grid arrays [3][G] real and [3][Gh] complex, so the
// FFTs run as one batch of three.
#include "device_common.h"
#include "green_fft.h"

namespace gspm {

namespace {

// one thread per item: these passes are bound by the latency of their
// gathers, so every item's loads should be in flight at once
inline int grid_of(int64_t n) {
    const int64_t g = (n + kThreads - 1) / kThreads;
    return static_cast<int>(g < (1 << 30) ? (g > 0 ? g : 1) : (1 << 30));
}

// streaming passes with a per-workgroup reduction: a bounded grid keeps the
// number of atomic adds on the sharded sums small
inline int reduce_grid_of(int64_t n) {
    const int64_t g = (n + kThreads - 1) / kThreads;
    return static_cast<int>(g < 2048 ? (g > 0 ? g : 1) : 2048);
}

// The test of |r_j|^2 <= tol2 |b|^2 (recorded by workgroup 0 as iteration
// j) and the converged state of the set; true when the launch has work.
__device__ __forceinline__ bool pc_live(const CGScalars &cg, int test_k, double tol2) {
    if (cg.done[0] != 0) return false;
    if (test_k < 0) return true;
    const double *const src[2] = {cg.rr_at(0, test_k), cg.bb_at(0)};
    double t[2];
    shard_totals<2>(src, t);
    const int stop = !isfinite(t[0]) ? 2 : (t[0] <= tol2 * t[1] ? 1 : 0);
    if (stop) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            cg.done[0] = stop;
            cg.iters[0] = test_k;
        }
        return false;
    }
    return true;
}

// Trilinear corners of the node at p: the lower grid indices and the weights
// along each axis (FP64), the position wrapped into the periodic cell.
__device__ __forceinline__ void corners(const GreenView &gv, const double p[3], int (&i0)[3], int (&i1)[3],
                                        double (&t)[3]) {
    const int g[3] = {gv.gx, gv.gy, gv.gz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double f = (p[a] - gv.lo[a]) / gv.h[a];
        f -= g[a] * floor(f / g[a]);
        int k = static_cast<int>(floor(f));
        if (k >= g[a]) k = g[a] - 1;
        if (k < 0) k = 0;
        i0[a] = k;
        i1[a] = k + 1 == g[a] ? 0 : k + 1;
        t[a] = f - k;
    }
}

}  // namespace

// Four components of a node's vector, the last unused: one 16-byte (32 in FP64)
// access where a gather of three costs one each.
template <class T>
struct __align__(4 * sizeof(T)) Node4 {
    T v[4];
};

// Q^T r: each row (a grid point, rows in Morton order so that neighbouring
// threads gather nearby nodes) sums w r over its list, after the test of |r_j|.
// NODE4: r as Node4, one access a gathered node.  Bound by the gathers and the
// lists (a thread's own run of entries, so four to a load): at 970k nodes 31 us
// against 52 with scalar accesses to both, 97k 5.8 against 9.3 (FP32).  The
// first entries are on their way while the test's sums are read.
template <class T, bool NODE4>
__global__ void __launch_bounds__(kThreads) k_pc_restrict(GreenView gv, int n, const T *r, CGScalars cg, int test_k,
                                                          double tol2) {
    const Node4<T> *w = static_cast<const Node4<T> *>(gv.rw);
    const int4 *node = reinterpret_cast<const int4 *>(gv.rnode);
    T *grid = static_cast<T *>(gv.grid);
    // entries gathered per batch (their loads, then the nodes'), in fours: a list's length is a multiple of four
    constexpr int kQ = sizeof(T) == 4 ? 3 : 2;
    const int64_t t = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x;
    int e0 = 0, e1 = 0;
    int4 j[kQ];
    int64_t g = 0;
    Node4<T> wj[kQ];
    auto entries = [&](int eb) {
#pragma unroll
        for (int u = 0; u < kQ; ++u)
            if (eb + u < e1) {
                j[u] = node[eb + u];
                wj[u] = w[eb + u];
            }
    };
    if (t < gv.G) {
        e0 = gv.rptr[t];
        e1 = gv.rptr[t + 1];
        g = gv.rgrid[t];
        entries(e0);
    }
    if (!pc_live(cg, test_k, tol2) || t >= gv.G) return;
    auto value = [&](int i) {
        Node4<T> v;
        if (NODE4) {
            v = reinterpret_cast<const Node4<T> *>(r)[i];
        } else {
            v.v[0] = r[i];
            v.v[1] = r[static_cast<size_t>(n) + i];
            v.v[2] = r[2 * static_cast<size_t>(n) + i];
        }
        return v;
    };
    T s0 = T(0), s1 = T(0), s2 = T(0);
    for (int eb = e0; eb < e1; eb += kQ) {
        if (eb > e0) entries(eb);
        Node4<T> v[kQ][4];
#pragma unroll
        for (int u = 0; u < kQ; ++u)
            if (eb + u < e1) {
                v[u][0] = value(j[u].x);
                v[u][1] = value(j[u].y);
                v[u][2] = value(j[u].z);
                v[u][3] = value(j[u].w);
            }
#pragma unroll
        for (int u = 0; u < kQ; ++u)
            if (eb + u < e1)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    s0 += wj[u].v[h] * v[u][h].v[0];
                    s1 += wj[u].v[h] * v[u][h].v[1];
                    s2 += wj[u].v[h] * v[u][h].v[2];
                }
    }
    // packed for the complex transforms: w0 = x0 + i x1, w1 = x2
    grid[2 * g] = s0;
    grid[2 * g + 1] = s1;
    grid[2 * (gv.G + g)] = s2;
    grid[2 * (gv.G + g) + 1] = T(0);
}

// Y(k) = A(k)^-1 X(k) / G on the packed spectra.  The two complex grids hold
// the transforms of w0 = x0 + i x1 and w1 = x2 (x real), so
//   X0(k) = (W0(k) + conj W0(-k)) / 2,  X1(k) = (W0(k) - conj W0(-k)) / 2i,
//   X2(k) = (W1(k) + conj W1(-k)) / 2,
// and the results go back packed the same way with Y(-k) = conj Y(k) (A(-k)
// = conj A(k) for the real stencil), so the inverse transform returns
// y0 + i y1 and y2.  One thread takes a mode k of the half spectrum (kx <=
// gx / 2, the table's index) together with its mirror -k; a pair whose mirror
// is in the half spectrum too is taken once.
template <class T>
__global__ void __launch_bounds__(kThreads) k_pc_modes(GreenView gv, CGScalars cg) {
    if (cg.done[0] != 0) return;
    const T *M = static_cast<const T *>(gv.ainv);
    T *w0 = static_cast<T *>(gv.spec);      // (re, im) pairs, [2][G]
    T *w1 = w0 + 2 * gv.G;
    for (int64_t m = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; m < gv.Gh;
         m += static_cast<int64_t>(gridDim.x) * kThreads) {
        const int kx = static_cast<int>(m % gv.gxh);
        const int ky = static_cast<int>((m / gv.gxh) % gv.gy);
        const int kz = static_cast<int>(m / (static_cast<int64_t>(gv.gxh) * gv.gy));
        const int mx = (gv.gx - kx) % gv.gx, my = (gv.gy - ky) % gv.gy, mz = (gv.gz - kz) % gv.gz;
        const int64_t f = (static_cast<int64_t>(kz) * gv.gy + ky) * gv.gx + kx;
        const int64_t fm = (static_cast<int64_t>(mz) * gv.gy + my) * gv.gx + mx;
        if (mx < gv.gxh && fm < f) continue;
        const T ar = w0[2 * f], ai = w0[2 * f + 1], br = w0[2 * fm], bi = w0[2 * fm + 1];
        const T cr = w1[2 * f], ci = w1[2 * f + 1], dr = w1[2 * fm], di = w1[2 * fm + 1];
        const T h = T(0.5);
        const T xr[3] = {h * (ar + br), h * (ai + bi), h * (cr + dr)};
        const T xi[3] = {h * (ai - bi), h * (br - ar), h * (ci - di)};
        const T *a = M + 9 * m;
        // off-diagonal (a01, a02, a12) and their conjugates below the diagonal
        const T r01 = a[3], i01 = a[4], r02 = a[5], i02 = a[6], r12 = a[7], i12 = a[8];
        const T yr0 = a[0] * xr[0] + (r01 * xr[1] - i01 * xi[1]) + (r02 * xr[2] - i02 * xi[2]);
        const T yi0 = a[0] * xi[0] + (r01 * xi[1] + i01 * xr[1]) + (r02 * xi[2] + i02 * xr[2]);
        const T yr1 = (r01 * xr[0] + i01 * xi[0]) + a[1] * xr[1] + (r12 * xr[2] - i12 * xi[2]);
        const T yi1 = (r01 * xi[0] - i01 * xr[0]) + a[1] * xi[1] + (r12 * xi[2] + i12 * xr[2]);
        const T yr2 = (r02 * xr[0] + i02 * xi[0]) + (r12 * xr[1] + i12 * xi[1]) + a[2] * xr[2];
        const T yi2 = (r02 * xi[0] - i02 * xr[0]) + (r12 * xi[1] - i12 * xr[1]) + a[2] * xi[2];
        if (fm == f) {
            // a self-conjugate mode: X and A^-1 are real there (up to rounding)
            w0[2 * f] = yr0;
            w0[2 * f + 1] = yr1;
            w1[2 * f] = yr2;
            w1[2 * f + 1] = T(0);
            continue;
        }
        // W0(k) = Y0 + i Y1, W0(-k) = conj Y0 + i conj Y1, W1(+-k) = Y2, conj Y2
        w0[2 * f] = yr0 - yi1;
        w0[2 * f + 1] = yi0 + yr1;
        w0[2 * fm] = yr0 + yi1;
        w0[2 * fm + 1] = yr1 - yi0;
        w1[2 * f] = yr2;
        w1[2 * f + 1] = yi2;
        w1[2 * fm] = yr2;
        w1[2 * fm + 1] = -yi2;
    }
}

// z = Q y + omega D^-1 r at every node; rz += r.z.  Several nodes a thread, their
// gathers in flight together: a workgroup's sum ends in an atomic addition, and
// one for every 256 nodes costs a fifth of the pass (970k nodes 30 us, four a
// thread 25).
template <class T, int NN>
__global__ void __launch_bounds__(kThreads) k_pc_prolong(GreenView gv, MeshView mv, const T *r, T *z, double *rz,
                                                         CGScalars cg) {
    if (cg.done[0] != 0) return;
    const int n = mv.n;
    const T *y = static_cast<const T *>(gv.grid);
    const T *dv = static_cast<const T *>(gv.dinv);
    double part = 0.0;
    const int first = blockIdx.x * (kThreads * NN) + threadIdx.x;
    double p[NN][3];
    T rv[NN][3], d[NN][3];
#pragma unroll
    for (int u = 0; u < NN; ++u) {
        const int i = min(first + u * kThreads, n - 1);
        p[u][0] = mv.x[i];
        p[u][1] = mv.y[i];
        p[u][2] = mv.z[i];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            rv[u][a] = r[static_cast<size_t>(a) * n + i];
            d[u][a] = dv[static_cast<size_t>(a) * n + i];
        }
    }
#pragma unroll
    for (int u = 0; u < NN; ++u) {
        const int i = first + u * kThreads;
        int i0[3], i1[3];
        double t[3];
        corners(gv, p[u], i0, i1, t);
        T acc[3] = {T(0), T(0), T(0)};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int ix = (c & 1) ? i1[0] : i0[0], iy = (c & 2) ? i1[1] : i0[1], iz = (c & 4) ? i1[2] : i0[2];
            const double wd = ((c & 1) ? t[0] : 1.0 - t[0]) * ((c & 2) ? t[1] : 1.0 - t[1]) *
                              ((c & 4) ? t[2] : 1.0 - t[2]);
            const T wc = static_cast<T>(wd);
            const int64_t g = (static_cast<int64_t>(iz) * gv.gy + iy) * gv.gx + ix;
            // packed: y0 + i y1 in the first complex grid, y2 in the second
            acc[0] += wc * y[2 * g];
            acc[1] += wc * y[2 * g + 1];
            acc[2] += wc * y[2 * (gv.G + g)];
        }
        if (i >= n) continue;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const T zv = acc[a] + d[u][a] * rv[u][a];
            z[static_cast<size_t>(a) * n + i] = zv;
            part += static_cast<double>(rv[u][a]) * zv;
        }
    }
    block_atomic_add1(part, rz, cg.det);
}

// x += alpha p, r -= alpha q, |r|^2, and r as Node4 (r4) for the restriction's
// gathers.  A thread's first node is on its way while the sums that form alpha
// are read, and a node a thread leaves a third of the atomic additions that a
// value a thread did: 97k nodes FP32 5.4 us against 8.4.
template <class T>
__global__ void __launch_bounds__(kThreads) k_pcg_update(int n, T *x, T *r, Node4<T> *r4, const T *p, const T *q,
                                                         CGScalars cg, int k) {
    const int done = cg.done[0];
    T xv[3], rv[3], pv[3], qv[3];
    auto fetch = [&](int i) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t o = static_cast<size_t>(c) * n + i;
            xv[c] = x[o];
            rv[c] = r[o];
            pv[c] = p[o];
            qv[c] = q[o];
        }
    };
    const int first = blockIdx.x * kThreads + threadIdx.x;
    if (first < n) fetch(first);
    const double *const src[2] = {pcg_rz_at(cg, k), cg.pq_at(0, k)};
    double t[2];
    shard_totals<2>(src, t);
    if (done != 0) return;
    const T alpha = static_cast<T>(t[0] / t[1]);
    double part = 0.0;
    for (int i = first; i < n; i += gridDim.x * kThreads) {
        if (i != first) fetch(i);
        Node4<T> v;
        v.v[3] = T(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const size_t o = static_cast<size_t>(c) * n + i;
            x[o] = xv[c] + alpha * pv[c];
            v.v[c] = rv[c] - alpha * qv[c];
            r[o] = v.v[c];
            part += static_cast<double>(v.v[c]) * v.v[c];
        }
        r4[i] = v;
    }
    block_atomic_add1(part, cg.rr_at(0, k + 1), cg.det);
}

__global__ void __launch_bounds__(kThreads) k_sum3(int n, const double *b, double *aux, DetSums det) {
    double acc[3] = {0.0, 0.0, 0.0};
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads)
#pragma unroll
        for (int a = 0; a < 3; ++a) acc[a] += b[static_cast<size_t>(a) * n + i];
    block_atomic_add<3>(acc, aux, kShards, det);
}

__global__ void __launch_bounds__(kThreads) k_sub_mean3(int n, double *b, const double *aux, double *bb,
                                                        DetSums det) {
    const double *const src[3] = {aux, aux + kShards, aux + 2 * kShards};
    double t[3];
    shard_totals<3>(src, t);
    double part = 0.0;
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const size_t o = static_cast<size_t>(a) * n + i;
            const double v = b[o] - t[a] / n;
            b[o] = v;
            part += v * v;
        }
    block_atomic_add1(part, bb, det);
}

__global__ void k_pin_copy(int n, const double *x, int p0, double *aux) {
    if (threadIdx.x < 3) aux[threadIdx.x] = x[static_cast<size_t>(threadIdx.x) * n + p0];
}

__global__ void __launch_bounds__(kThreads) k_pin_sub(int n, double *x, const double *aux) {
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads)
#pragma unroll
        for (int a = 0; a < 3; ++a) x[static_cast<size_t>(a) * n + i] -= aux[a];
}

// A(k) = sum_o S(o) exp(2 pi i k.o / g) on the half spectrum, inverted by
// cofactors in complex FP64, times factor, stored in its Hermitian form.
struct Stencil27 {
    double s[27 * 9];
};

template <class T>
__global__ void __launch_bounds__(kThreads) k_pc_symbol(GreenView gv, FftPlan fp, Stencil27 st, double factor) {
    T *out = static_cast<T *>(const_cast<void *>(gv.ainv));
    // by mode of the half spectrum, or (fp.pairs) by position along z and column pair
    const int64_t count = fp.pairs ? static_cast<int64_t>(fp.npairs) * gv.gz : gv.Gh;
    for (int64_t m = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; m < count;
         m += static_cast<int64_t>(gridDim.x) * kThreads) {
        const int pair = fp.pairs ? static_cast<int>(m % fp.npairs) : 0;
        const int kx = fp.pairs ? fp.pairs[4 * pair + 2] : static_cast<int>(m % gv.gxh);
        const int ky = fp.pairs ? fp.pairs[4 * pair + 3] : static_cast<int>((m / gv.gxh) % gv.gy);
        const int kz = fp.pairs ? fp.z.freq[m / fp.npairs] : static_cast<int>(m / (static_cast<int64_t>(gv.gxh) * gv.gy));
        T *o = fp.pairs ? out + m : out + 9 * m;
        const int64_t os = fp.pairs ? count : 1;
        if (kx == 0 && ky == 0 && kz == 0) {
#pragma unroll
            for (int q = 0; q < 9; ++q) o[q * os] = T(0);
            continue;
        }
        double ar[3][3] = {}, ai[3][3] = {};
        const double two_pi = 6.283185307179586476925286766559;
        for (int oz = -1; oz <= 1; ++oz)
            for (int oy = -1; oy <= 1; ++oy)
                for (int ox = -1; ox <= 1; ++ox) {
                    const double ph = two_pi * (static_cast<double>(kx) * ox / gv.gx +
                                                static_cast<double>(ky) * oy / gv.gy +
                                                static_cast<double>(kz) * oz / gv.gz);
                    double sn, cs;
                    sincos(ph, &sn, &cs);
                    const double *S = st.s + 9 * ((oz + 1) * 9 + (oy + 1) * 3 + (ox + 1));
#pragma unroll
                    for (int a = 0; a < 3; ++a)
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            ar[a][b] += S[3 * a + b] * cs;
                            ai[a][b] += S[3 * a + b] * sn;
                        }
                }
        // cofactors: C(i, j) = A(i+1, j+1) A(i+2, j+2) - A(i+1, j+2) A(i+2, j+1)
        double cr[3][3], ci[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int r0 = (i + 1) % 3, r1 = (i + 2) % 3, c0 = (j + 1) % 3, c1 = (j + 2) % 3;
                const double pr = ar[r0][c0] * ar[r1][c1] - ai[r0][c0] * ai[r1][c1];
                const double pi = ar[r0][c0] * ai[r1][c1] + ai[r0][c0] * ar[r1][c1];
                const double qr = ar[r0][c1] * ar[r1][c0] - ai[r0][c1] * ai[r1][c0];
                const double qi = ar[r0][c1] * ai[r1][c0] + ai[r0][c1] * ar[r1][c0];
                cr[i][j] = pr - qr;
                ci[i][j] = pi - qi;
            }
        double dr = 0.0, di = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            dr += ar[0][j] * cr[0][j] - ai[0][j] * ci[0][j];
            di += ar[0][j] * ci[0][j] + ai[0][j] * cr[0][j];
        }
        const double den = dr * dr + di * di;
        // inverse(i, j) = C(j, i) / det
        auto inv_re = [&](int i, int j) { return (cr[j][i] * dr + ci[j][i] * di) / den * factor; };
        auto inv_im = [&](int i, int j) { return (ci[j][i] * dr - cr[j][i] * di) / den * factor; };
        o[0 * os] = static_cast<T>(inv_re(0, 0));
        o[1 * os] = static_cast<T>(inv_re(1, 1));
        o[2 * os] = static_cast<T>(inv_re(2, 2));
        o[3 * os] = static_cast<T>(inv_re(0, 1));
        o[4 * os] = static_cast<T>(inv_im(0, 1));
        o[5 * os] = static_cast<T>(inv_re(0, 2));
        o[6 * os] = static_cast<T>(inv_im(0, 2));
        o[7 * os] = static_cast<T>(inv_re(1, 2));
        o[8 * os] = static_cast<T>(inv_im(1, 2));
    }
}

template <class T>
void launch_pc_restrict(const GreenView &gv, int n, const T *r, bool node4, const CGScalars &cg, int test_k, double tol,
                        hipStream_t s) {
    if (node4)
        hipLaunchKernelGGL((k_pc_restrict<T, true>), dim3(grid_of(gv.G)), dim3(kThreads), 0, s, gv, n,
                           static_cast<const T *>(gv.r4), cg, test_k, tol * tol);
    else
        hipLaunchKernelGGL((k_pc_restrict<T, false>), dim3(grid_of(gv.G)), dim3(kThreads), 0, s, gv, n, r, cg, test_k,
                           tol * tol);
}

template <class T>
void launch_pc_modes(const GreenView &gv, const CGScalars &cg, hipStream_t s) {
    hipLaunchKernelGGL(k_pc_modes<T>, dim3(grid_of(gv.Gh)), dim3(kThreads), 0, s, gv, cg);
}

template <class T>
void launch_pc_prolong(const GreenView &gv, const MeshView &mv, const T *r, T *z, double *rz, const CGScalars &cg,
                       hipStream_t s) {
    // (more than one node a thread once every CU has two workgroups)
    if (mv.n >= 4 * kThreads * 512)
        hipLaunchKernelGGL((k_pc_prolong<T, 4>), dim3(grid_of((mv.n + 3) / 4)), dim3(kThreads), 0, s, gv, mv, r, z, rz, cg);
    else
        hipLaunchKernelGGL((k_pc_prolong<T, 1>), dim3(grid_of(mv.n)), dim3(kThreads), 0, s, gv, mv, r, z, rz, cg);
    launch_det_finish(cg.det, s);
}

template <class T>
void launch_pcg_update(const GreenView &gv, int n, T *x, T *r, const T *p, const T *q, const CGScalars &cg, int k,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_pcg_update<T>, dim3(reduce_grid_of(n)), dim3(kThreads), 0, s, n, x, r,
                       static_cast<Node4<T> *>(gv.r4), p, q, cg, k);
    launch_det_finish(cg.det, s);
}

void launch_remove_mean3(int n, double *b, double *aux, double *bb, hipStream_t s, const DetSums &det) {
    launch_fill(aux, 3 * kShards, 0.0, s);
    launch_fill(bb, kShards, 0.0, s);
    hipLaunchKernelGGL(k_sum3, dim3(reduce_grid_of(n)), dim3(kThreads), 0, s, n, b, aux, det);
    launch_det_finish(det, s);
    hipLaunchKernelGGL(k_sub_mean3, dim3(reduce_grid_of(n)), dim3(kThreads), 0, s, n, b, aux, bb, det);
    launch_det_finish(det, s);
}

void launch_pin_shift(int n, double *x, int p0, double *aux, hipStream_t s) {
    hipLaunchKernelGGL(k_pin_copy, dim3(1), dim3(64), 0, s, n, x, p0, aux);
    hipLaunchKernelGGL(k_pin_sub, dim3(grid_of(n)), dim3(kThreads), 0, s, n, x, aux);
}

template <class T>
void launch_pc_symbol(const GreenView &gv, const FftPlan *fp, const double *stencil27, double factor, hipStream_t s) {
    Stencil27 st;
    for (int q = 0; q < 27 * 9; ++q) st.s[q] = stencil27[q];
    hipLaunchKernelGGL(k_pc_symbol<T>, dim3(grid_of(gv.Gh)), dim3(kThreads), 0, s, gv, fp ? *fp : FftPlan{}, st, factor);
}

#define GSPM_PC_INST(T)                                                                                              \
    template void launch_pc_restrict<T>(const GreenView &, int, const T *, bool, const CGScalars &, int, double,   \
                                        hipStream_t);                                                               \
    template void launch_pc_modes<T>(const GreenView &, const CGScalars &, hipStream_t);                            \
    template void launch_pc_prolong<T>(const GreenView &, const MeshView &, const T *, T *, double *,               \
                                       const CGScalars &, hipStream_t);                                             \
    template void launch_pcg_update<T>(const GreenView &, int, T *, T *, const T *, const T *, const CGScalars &,   \
                                       int, hipStream_t);                                                          \
    template void launch_pc_symbol<T>(const GreenView &, const FftPlan *, const double *, double, hipStream_t);
GSPM_PC_INST(double)
GSPM_PC_INST(float)
#undef GSPM_PC_INST

}  // namespace gspm
