// The grid transforms of the elastic preconditioner with its modes between, as
// three launches.
//
// As library transforms they are three passes over memory per direction, for
// lengths the library has no kernel for (46 = 2 x 23) fifteen launches per
// direction; at 97k nodes an application took 165 us, nearly all of it launches
// and passes.  Here
//   1. k_pc_planes_fwd: a workgroup takes one z plane of one packed field into
//      LDS and transforms it along x and y there;
//   2. k_pc_columns: a workgroup takes eight or sixteen pairs of columns (kx,
//      ky), (-kx, -ky) of both fields, transforms along z, applies the symbol inverse to
//      each mode and its mirror, and transforms back;
//   3. k_pc_planes_inv: planes back along y and x.
// Each grid value crosses memory six times instead of fourteen.  (Gathering the
// restriction into the planes as well saved two of them and cost more: 198
// planes at 99^3 are too few to hide a gather, 158 us against 53 + 44.)
// Measured, the three in turn: 11 + 13 + 10 us at 46^3 FP32, 7 + 10 + 8 at
// 30^3 FP64, 21 + 37 + 22 at 99^3 FP32 (87 as library transforms and modes).
//
// A transform of length N = N1 N2 (the factors nearest to each other; N1 = 1
// for a prime) is two stages of direct sums of lengths N1 and N2 with a
// twiddle between, in place: stage A leaves its sum k1 of residue n2 at k1 N2 +
// n2, stage B the frequency k1 + N1 k2 at k1 N2 + k2.  Nothing is put in order:
// the modes look frequencies up by position and the inverse runs the stages
// backwards.  A wave works on 64 sums for the same frequencies, so their
// cosines and sines are the same in every lane and come by scalar loads.  Sums
// of 9 and 11 terms (N = 99) or 2 and 23 (N = 46) take more arithmetic than
// butterflies for each radix would and need none for the factors a mesh
// happens to have.
#include <algorithm>

#include "device_common.h"
#include "green_fft.h"

namespace gspm {

namespace {

constexpr int kPlaneThreads = 1024, kColThreads = 512;
constexpr int kS = kFftSlots;                  // values of k a wave takes at once
// groups of 64 sums x kS pairs of outputs a wave holds between a stage's reads
// and its writes (registers)
template <class T>
constexpr int fft_items() { return sizeof(T) == 4 ? 4 : 3; }

template <class T>
struct Cx {
    T re, im;
};

// One stage in place on LDS: J M sums of length R, sum (j, i) over buf[i si +
// j sj + t es], t < R, its output k back at t = k, times the twiddle tw[j ta +
// k tb] when TW.  With x(t) +- x(R - t) taken together, outputs k and R - k
// come from the same two real-weighted sums:
//   P = sum_t cos(2 pi k t / R) x(t),  Q = sum_t sin(2 pi k t / R) x(t),
//   X(k) = P - i Q, X(R - k) = P + i Q   (the inverse: the other way round),
// a third of the multiply-adds of the plain sums.  A wave takes kS values of k
// for 64 sums at once; cs holds (cos, sin) for t <= R / 2 in rows of
// fft_columns(R) values of k.
template <class T, bool INV, bool TW, int TH>
__device__ __forceinline__ void stage(Cx<T> *buf, int R, int J, int M, int si, int sj, int es, const T *cs,
                                      const T *tw, int ta, int tb) {
    using CT = const __attribute__((address_space(4))) T;
    constexpr int kItems = fft_items<T>();
    CT *C = (CT *)(cs);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NG = J * M, chunks = (NG + 63) >> 6, cols = fft_columns(R), items = chunks * (cols / kS), half = (R - 1) >> 1;
    Cx<T> out[kItems][2 * kS];
    int at[kItems];
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        const int it = wave + m * (TH / 64);
        at[m] = -1;
        if (it >= items) continue;
        const int kb = it / chunks, k0 = kS * kb, g = (it - kb * chunks) * 64 + lane, gg = g < NG ? g : NG - 1;
        const int j = gg / M, i = gg - j * M, base = i * si + j * sj;
        Cx<T> w[2 * kS];
        if constexpr (TW) {                        // loaded ahead of the sums they multiply
#pragma unroll
            for (int q = 0; q < kS; ++q) {
                const int k = k0 + q <= R / 2 ? k0 + q : 0, kr = k > 0 ? R - k : 0;
                w[2 * q] = Cx<T>{tw[2 * (j * ta + k * tb)], tw[2 * (j * ta + k * tb) + 1]};
                w[2 * q + 1] = Cx<T>{tw[2 * (j * ta + kr * tb)], tw[2 * (j * ta + kr * tb) + 1]};
            }
        }
        Cx<T> P[kS], Q[kS];
        const Cx<T> x0 = buf[base];
#pragma unroll
        for (int q = 0; q < kS; ++q) {
            P[q] = x0;
            Q[q] = Cx<T>{T(0), T(0)};
        }
        CT *row = C + 2 * (cols + k0);             // t = 1
#pragma unroll 2
        for (int t = 1; t <= half; ++t, row += 2 * cols) {
            const Cx<T> x = buf[base + t * es], y = buf[base + (R - t) * es];
            const T er = x.re + y.re, ei = x.im + y.im, dr = x.re - y.re, di = x.im - y.im;
#pragma unroll
            for (int q = 0; q < kS; ++q) {
                const T c = row[2 * q], d = row[2 * q + 1];
                P[q].re += c * er;
                P[q].im += c * ei;
                Q[q].re += d * dr;
                Q[q].im += d * di;
            }
        }
        if ((R & 1) == 0) {
            const Cx<T> x = buf[base + (R / 2) * es];
#pragma unroll
            for (int q = 0; q < kS; ++q) {
                const T c = row[2 * q];            // (-1)^k
                P[q].re += c * x.re;
                P[q].im += c * x.im;
            }
        }
#pragma unroll
        for (int q = 0; q < kS; ++q) {
            const T sg = INV ? T(-1) : T(1);
            Cx<T> u{P[q].re + sg * Q[q].im, P[q].im - sg * Q[q].re}, v{P[q].re - sg * Q[q].im, P[q].im + sg * Q[q].re};
            if constexpr (TW) {
                const Cx<T> a = w[2 * q], b = w[2 * q + 1];
                const T ai = INV ? -a.im : a.im, bi = INV ? -b.im : b.im;
                u = Cx<T>{a.re * u.re - ai * u.im, a.re * u.im + ai * u.re};
                v = Cx<T>{b.re * v.re - bi * v.im, b.re * v.im + bi * v.re};
            }
            out[m][2 * q] = u;
            out[m][2 * q + 1] = v;
        }
        if (g < NG) at[m] = base;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        const int it = wave + m * (TH / 64);
        if (it >= items || at[m] < 0) continue;
        const int k0 = kS * (it / chunks);
#pragma unroll
        for (int q = 0; q < kS; ++q) {
            const int k = k0 + q;
            if (k > R / 2) continue;
            buf[at[m] + k * es] = out[m][2 * q];
            if (k > 0 && 2 * k != R) buf[at[m] + (R - k) * es] = out[m][2 * q + 1];
        }
    }
    __syncthreads();
}

// A transform of M lines, line i at i si with element stride es, in place.
template <class T, bool INV, int TH>
__device__ __forceinline__ void transform(Cx<T> *buf, const FftAxis &a, int M, int si, int es) {
    const T *d1 = static_cast<const T *>(a.cs1), *d2 = static_cast<const T *>(a.cs2), *tw = static_cast<const T *>(a.tw);
    if constexpr (!INV) {
        if (a.n1 > 1) stage<T, INV, true, TH>(buf, a.n1, a.n2, M, si, es, a.n2 * es, d1, tw, a.n1, 1);
        stage<T, INV, false, TH>(buf, a.n2, a.n1, M, si, a.n2 * es, es, d2, nullptr, 0, 0);
    } else {
        if (a.n1 == 1) {
            stage<T, INV, false, TH>(buf, a.n2, a.n1, M, si, a.n2 * es, es, d2, nullptr, 0, 0);
        } else {
            stage<T, INV, true, TH>(buf, a.n2, a.n1, M, si, a.n2 * es, es, d2, tw, 1, a.n1);
            stage<T, INV, false, TH>(buf, a.n1, a.n2, M, si, es, a.n2 * es, d1, nullptr, 0, 0);
        }
    }
}

}  // namespace

// One z plane of one field along x and y.
template <class T>
__global__ void __launch_bounds__(kPlaneThreads) k_pc_planes_fwd(GreenView gv, FftPlan fp, CGScalars cg) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (cg.done[0] != 0) return;
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    const int z = blockIdx.x >> 1, f = blockIdx.x & 1, P = gv.gx * gv.gy, rs = gv.gx | 1;
    const Cx<T> *grid = static_cast<const Cx<T> *>(gv.grid) + f * gv.G + static_cast<int64_t>(z) * P;
    for (int t = threadIdx.x; t < P; t += kPlaneThreads) {
        const int y = t / gv.gx;
        buf[y * rs + t - y * gv.gx] = grid[t];
    }
    __syncthreads();
    transform<T, false, kPlaneThreads>(buf, fp.x, gv.gy, rs, 1);
    transform<T, false, kPlaneThreads>(buf, fp.y, gv.gx, 1, rs);
    Cx<T> *spec = static_cast<Cx<T> *>(gv.spec) + f * gv.G + static_cast<int64_t>(z) * P;
    for (int t = threadIdx.x; t < P; t += kPlaneThreads) {
        const int y = t / gv.gx;
        spec[t] = buf[y * rs + t - y * gv.gx];
    }
}

template <class T>
__global__ void __launch_bounds__(kPlaneThreads) k_pc_planes_inv(GreenView gv, FftPlan fp, CGScalars cg) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (cg.done[0] != 0) return;
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    const int z = blockIdx.x >> 1, f = blockIdx.x & 1, P = gv.gx * gv.gy, rs = gv.gx | 1;
    const Cx<T> *spec = static_cast<const Cx<T> *>(gv.spec) + f * gv.G + static_cast<int64_t>(z) * P;
    for (int t = threadIdx.x; t < P; t += kPlaneThreads) {
        const int y = t / gv.gx;
        buf[y * rs + t - y * gv.gx] = spec[t];
    }
    __syncthreads();
    transform<T, true, kPlaneThreads>(buf, fp.y, gv.gx, 1, rs);
    transform<T, true, kPlaneThreads>(buf, fp.x, gv.gy, rs, 1);
    Cx<T> *grid = static_cast<Cx<T> *>(gv.grid) + f * gv.G + static_cast<int64_t>(z) * P;
    for (int t = threadIdx.x; t < P; t += kPlaneThreads) {
        const int y = t / gv.gx;
        grid[t] = buf[y * rs + t - y * gv.gx];
    }
}

// Column pairs: forward along z, Y(k) = A(k)^-1 X(k) / G for each mode and its
// mirror, back along z.  With W0 = X0 + i X1 and W1 = X2 of real fields,
//   X0(k) = (W0(k) + conj W0(-k)) / 2,  X1(k) = (W0(k) - conj W0(-k)) / 2i,
//   X2(k) = (W1(k) + conj W1(-k)) / 2,
// and Y(-k) = conj Y(k) goes back packed the same way.
template <class T, int kColPairs>
__global__ void __launch_bounds__(kColThreads) k_pc_columns(GreenView gv, FftPlan fp, CGScalars cg) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (cg.done[0] != 0) return;
    Cx<T> *buf = reinterpret_cast<Cx<T> *>(smem);
    // LDS: [z][field][pair][this, mirror], rows of 4 kColPairs values and one of padding
    constexpr int W = 4 * kColPairs, rs = W | 1;
    const int64_t P = static_cast<int64_t>(gv.gx) * gv.gy;
    const int gz = gv.gz, p0 = blockIdx.x * kColPairs;
    const int32_t *pairs = fp.pairs;               // [pair]: position of the column, of its mirror; kx, ky of the column
    Cx<T> *spec = static_cast<Cx<T> *>(gv.spec);
    // lanes over [field][this, mirror][pair] of a z: consecutive pairs are consecutive in memory
    for (int t = threadIdx.x; t < gz * W; t += kColThreads) {
        const int z = t / W, c = t - z * W, p = c % kColPairs, s = (c / kColPairs) & 1, f = c / (2 * kColPairs);
        const bool in = p0 + p < fp.npairs;
        const int32_t col = in ? pairs[4 * (p0 + p) + s] : 0;
        buf[z * rs + (f * kColPairs + p) * 2 + s] = in ? spec[f * gv.G + z * P + col] : Cx<T>{T(0), T(0)};
    }
    __syncthreads();
    transform<T, false, kColThreads>(buf, fp.z, W, 1, rs);
    const T *Mt = static_cast<const T *>(gv.ainv);  // [9][position along z][pair]
    for (int t = threadIdx.x; t < gz * kColPairs; t += kColThreads) {
        const int zp = t / kColPairs, p = t - zp * kColPairs;
        if (p0 + p >= fp.npairs) continue;
        const int32_t *pr = pairs + 4 * (p0 + p);
        const bool self = pr[0] == pr[1];          // the column is its own mirror
        const int zm = fp.z.neg[zp], kz = fp.z.freq[zp];
        if (self && fp.z.freq[zm] < kz) continue;  // taken with its mirror
        Cx<T> &A = buf[zp * rs + 2 * p], &B = buf[zm * rs + 2 * p + (self ? 0 : 1)];
        Cx<T> &C = buf[zp * rs + 2 * (kColPairs + p)], &D = buf[zm * rs + 2 * (kColPairs + p) + (self ? 0 : 1)];
        const T ar = A.re, ai = A.im, br = B.re, bi = B.im, cr = C.re, ci = C.im, dr = D.re, di = D.im;
        const T h = T(0.5);
        const T xr[3] = {h * (ar + br), h * (ai + bi), h * (cr + dr)};
        const T xi[3] = {h * (ai - bi), h * (br - ar), h * (ci - di)};
        T a[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) a[q] = Mt[(static_cast<size_t>(q) * gz + zp) * fp.npairs + p0 + p];
        const T r01 = a[3], i01 = a[4], r02 = a[5], i02 = a[6], r12 = a[7], i12 = a[8];
        const T yr0 = a[0] * xr[0] + (r01 * xr[1] - i01 * xi[1]) + (r02 * xr[2] - i02 * xi[2]);
        const T yi0 = a[0] * xi[0] + (r01 * xi[1] + i01 * xr[1]) + (r02 * xi[2] + i02 * xr[2]);
        const T yr1 = (r01 * xr[0] + i01 * xi[0]) + a[1] * xr[1] + (r12 * xr[2] - i12 * xi[2]);
        const T yi1 = (r01 * xi[0] - i01 * xr[0]) + a[1] * xi[1] + (r12 * xi[2] + i12 * xr[2]);
        const T yr2 = (r02 * xr[0] + i02 * xi[0]) + (r12 * xr[1] + i12 * xi[1]) + a[2] * xr[2];
        const T yi2 = (r02 * xi[0] - i02 * xr[0]) + (r12 * xi[1] - i12 * xr[1]) + a[2] * xi[2];
        if (self && zm == zp) {
            // a self-conjugate mode: X and A^-1 are real there (up to rounding)
            A = Cx<T>{yr0, yr1};
            C = Cx<T>{yr2, T(0)};
            continue;
        }
        A = Cx<T>{yr0 - yi1, yi0 + yr1};
        B = Cx<T>{yr0 + yi1, yr1 - yi0};
        C = Cx<T>{yr2, yi2};
        D = Cx<T>{yr2, -yi2};
    }
    __syncthreads();
    transform<T, true, kColThreads>(buf, fp.z, W, 1, rs);
    for (int t = threadIdx.x; t < gz * W; t += kColThreads) {
        const int z = t / W, c = t - z * W, p = c % kColPairs, s = (c / kColPairs) & 1, f = c / (2 * kColPairs);
        if (p0 + p >= fp.npairs || (s && pairs[4 * (p0 + p)] == pairs[4 * (p0 + p) + 1])) continue;
        spec[f * gv.G + z * P + pairs[4 * (p0 + p) + s]] = buf[z * rs + (f * kColPairs + p) * 2 + s];
    }
}

namespace {

size_t plane_lds(const GreenView &gv, size_t cx) { return cx * static_cast<size_t>(gv.gx | 1) * gv.gy; }
size_t column_lds(const GreenView &gv, int pairs, size_t cx) { return cx * (4 * pairs | 1) * static_cast<size_t>(gv.gz); }

// Pairs of a workgroup of the z pass: eight make 64-byte pieces of memory, and
// sixteen whole lines where they still leave every CU a workgroup (at 99^3 42.8
// against 36.6 us; at 46^3 sixteen would leave 66 workgroups).
int column_pairs(const GreenView &gv, int npairs, size_t cx, size_t lds_max) {
    return npairs >= 16 * 256 && column_lds(gv, 16, cx) <= lds_max ? 16 : 8;
}

// items of a stage: 64 sums of length r for kS pairs of outputs
int stage_items(int r, int sums) { return ((sums + 63) / 64) * (fft_columns(r) / kS); }

// whether a wave's registers hold its share of every stage's outputs
bool items_fit(int n1, int n2, int lines, int threads, bool f32) {
    const int most = (f32 ? fft_items<float>() : fft_items<double>()) * (threads / 64);
    return (n1 == 1 || stage_items(n1, n2 * lines) <= most) && stage_items(n2, n1 * lines) <= most;
}

// The chain of a workgroup's transforms of `lines` lines: a wave's items times their terms, a quarter of a microsecond
// each way for every unit.
int chain(int n1, int n2, int lines, int threads) {
    auto stage = [&](int r, int sums) {
        const int waves = threads / 64;
        return r == 1 ? 0 : (stage_items(r, sums) + waves - 1) / waves * (r / 2 + 1);
    };
    return stage(n1, n2 * lines) + stage(n2, n1 * lines);
}

// Whether the three launches beat the library's.  The sums' work grows with the lengths' factors and falls on few
// workgroups where planes (films) or columns (rods) are few; the library's launches cost the same for all lengths of
// small factors and several more for an axis with a prime above 13.  Iterations of the preconditioned solve (own
// against library, us, FP32), over 150 grids:
//   powers of 2, 3 or 5 throughout, where the library is at its best: 32^3 60 against 51, 27^3 57 / 51, 8 x 8 x 256 93 / 59,
//     128 x 128 x 4 129 / 93;
//   other small factors: the own ones up to a chain of 36 (30^3, 22: 60 / 63; 39^3, 30: 69 / 74; 64 x 64 x 24, 34: 83 / 87)
//     or of 16 per 10^5 grid points, whose passes over memory cost the library more (120^3, 184: 425 / 481; 90^3, 115: 219
//     / 240; 99^3, 131: 275 / 269), the library's beyond (72^3, 73: 150 / 139; 100 x 100 x 24, 62: 130 / 114);
//   n axes with a larger prime: the own ones up to 100 n, more on large grids, which the library's extra launches cross
//     each time (46^3, 50: 83 / 160; 97^3, 594: 322 / 443; 101 x 101 x 24, 323: 167 / 170; 24 x 24 x 127, 208: 116 / 93;
//     127 x 127 x 24, 401: 254 / 218; 257 x 8 x 8, 400: 142 / 105).
bool faster_than_library(const GreenView &gv, const int n1[3], const int n2[3], int pairs) {
    const int g[3] = {gv.gx, gv.gy, gv.gz};
    int pure = 0, large = 0;
    for (int n : g) {
        int rest = n, kinds = 0;
        bool high = false;
        for (int f = 2; rest > 1; ++f) {
            if (rest % f) continue;
            ++kinds;
            high |= f > 5;
            while (rest % f == 0) rest /= f;
            large += f > 13 && rest == 1;
        }
        pure += kinds == 1 && !high;
    }
    if (pure == 3) return false;
    constexpr int kCus = 256;
    const int wgs = (gv.gxh * gv.gy + pairs - 1) / pairs;
    const int64_t planes = (2 * gv.gz + kCus - 1) / kCus, columns = (wgs + kCus - 1) / kCus;
    const int64_t work = planes * (chain(n1[0], n2[0], gv.gy, kPlaneThreads) + chain(n1[1], n2[1], gv.gx, kPlaneThreads)) +
                         columns * chain(n1[2], n2[2], 4 * pairs, kColThreads);
    const double points = static_cast<double>(gv.G);
    return large == 0 ? work <= std::max(36.0, 1.6e-4 * points) : work <= 100.0 * large * (1.0 + points / 4e5);
}

}  // namespace

int green_fft_pairs(const GreenView &gv, const int n1[3], const int n2[3], bool f32, size_t lds_max) {
    const size_t cx = f32 ? sizeof(Cx<float>) : sizeof(Cx<double>);
    if (plane_lds(gv, cx) > lds_max || !items_fit(n1[0], n2[0], gv.gy, kPlaneThreads, f32) ||
        !items_fit(n1[1], n2[1], gv.gx, kPlaneThreads, f32))
        return 0;
    for (int pairs = column_pairs(gv, gv.gxh * gv.gy, cx, lds_max); pairs >= 8; pairs /= 2)
        if (column_lds(gv, pairs, cx) <= lds_max && items_fit(n1[2], n2[2], 4 * pairs, kColThreads, f32))
            return faster_than_library(gv, n1, n2, pairs) ? pairs : 0;
    return 0;
}

template <class T>
void launch_pc_fft(const GreenView &gv, const FftPlan &fp, const CGScalars &cg, hipStream_t s) {
    const size_t pl = plane_lds(gv, sizeof(Cx<T>)), cl = column_lds(gv, fp.wg_pairs, sizeof(Cx<T>));
    const dim3 cgrid((fp.npairs + fp.wg_pairs - 1) / fp.wg_pairs);
    hipLaunchKernelGGL(k_pc_planes_fwd<T>, dim3(2 * gv.gz), dim3(kPlaneThreads), pl, s, gv, fp, cg);
    if (fp.wg_pairs == 16)
        hipLaunchKernelGGL((k_pc_columns<T, 16>), cgrid, dim3(kColThreads), cl, s, gv, fp, cg);
    else
        hipLaunchKernelGGL((k_pc_columns<T, 8>), cgrid, dim3(kColThreads), cl, s, gv, fp, cg);
    hipLaunchKernelGGL(k_pc_planes_inv<T>, dim3(2 * gv.gz), dim3(kPlaneThreads), pl, s, gv, fp, cg);
}

template void launch_pc_fft<double>(const GreenView &, const FftPlan &, const CGScalars &, hipStream_t);
template void launch_pc_fft<float>(const GreenView &, const FftPlan &, const CGScalars &, hipStream_t);

}  // namespace gspm
