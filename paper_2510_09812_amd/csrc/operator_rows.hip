// Coefficients of K^mech and K^ms in row form, for the resident solves.
//
// One wave per slice of 64 rows, one lane per row.  For each entry (i, j) the
// lane walks the elements of node i (ascending, so the sums repeat bit for
// bit), and adds the product of the two gradients of those that hold j:
//   G_ab = sum_e V g_i,a g_j,b
// from which K^ms_ij = G_aa and (K^mech_ij)_pq = C_apbq G_ab.  The stiffness is
// one C, so on a periodic cell that the elements fill G (by parts: int d_a phi_i
// d_b phi_j equals int d_b phi_i d_a phi_j) and with it every 3x3 block is
// symmetric and six numbers hold it.  Free surfaces (a cavity, a gap, a body
// that does not reach its box) leave a boundary term in G: a first run looks for
// one, and with it the element kernels keep the elastic solve.  The diagonal is
// minus the sum of the row and not stored; the pinned node's row is zero.  Run
// once per mesh (the look at G, K^ms) or stiffness (K^mech): about 0.3 ms at 97k
// nodes each.
#include "device_common.h"
#include "resident.h"

namespace gspm {

namespace {

constexpr int kVoigt[3][3] = {{0, 5, 4}, {5, 1, 3}, {4, 3, 2}};

// |G_ab - G_ba| over sum_e V |g_i| |g_j| up to which an edge counts as closed.
// Rounding leaves 1e-16 on compact elements, growing with their aspect (1e-14
// at 100); a surface of flat faces leaves a sixth of the length across the edge
// where the sum is a length over the elements' aspect.  Sliver meshes beyond
// this line are solved with the elements, the slower way and right as well.
constexpr double kClosed = 1e-11;

}  // namespace

__global__ void __launch_bounds__(kThreads) k_operator_rows(const OperatorBuild a) {
    const ResLayout &ly = a.ly;
    const int wave = (blockIdx.x * kThreads + threadIdx.x) >> 6, lane = threadIdx.x & 63;
    const int slices = (ly.n + 63) >> 6, sl = wave % slices, part = wave / slices;
    if (part >= a.parts) return;
    const int i = sl * 64 + lane;
    const int32_t beg = ly.off[sl];
    const int w = (ly.off[sl + 1] - beg) >> 6;
    const int g = (sl * 64) / ly.nbr, hb = ly.halo_ptr[g];
    for (int e = part; e < w; e += a.parts) {
        if (i >= ly.n) {
            // lanes past the last row: padding entries of zero
            const size_t o = static_cast<size_t>(beg) + 64 * e;
            if (a.k64)
                for (int t = 0; t < 6; ++t) a.k64[o * 6 + 64 * t + lane] = 0.0;
            if (a.k32)
                for (int t = 0; t < 6; ++t) a.k32[o * 6 + 64 * t + lane] = 0.0f;
            if (a.m64) a.m64[o + lane] = 0.0;
            if (a.m32) a.m32[o + lane] = 0.0f;
            continue;
        }
        const int c = ly.col[beg + 64 * e + lane];
        const int j = c < ly.nbr ? g * ly.nbr + c : ly.halo_ids[hb + c - ly.nbr];
        double G[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, size = 0.0;
        // a padding entry's column is the row itself: zero
        const bool want = i != a.p0 && j != i;
        for (int t = a.inc_ptr[i]; want && t < a.inc_ptr[i + 1]; ++t) {
            const int32_t *v = a.tets + 4 * static_cast<size_t>(a.inc[t]);
            int vi = -1, vj = -1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                vi = v[q] == i ? q : vi;
                vj = v[q] == j ? q : vj;
            }
            if (vj < 0) continue;
            double ed[3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ed[k][0] = near_image(a.x[v[k + 1]] - a.x[v[0]], a.L[0], a.iL[0]);
                ed[k][1] = near_image(a.y[v[k + 1]] - a.y[v[0]], a.L[1], a.iL[1]);
                ed[k][2] = near_image(a.z[v[k + 1]] - a.z[v[0]], a.L[2], a.iL[2]);
            }
            Geo<double> geo;
            tet_geometry_from_edges(ed, geo);
            double gi[3] = {0, 0, 0}, gj[3] = {0, 0, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    gi[b] = q == vi ? geo.g[q][b] : gi[b];
                    gj[b] = q == vj ? geo.g[q][b] : gj[b];
                }
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q) G[p][q] += geo.vol * gi[p] * gj[q];
            size += geo.vol * sqrt((gi[0] * gi[0] + gi[1] * gi[1] + gi[2] * gi[2]) *
                                   (gj[0] * gj[0] + gj[1] * gj[1] + gj[2] * gj[2]));
        }
        if (a.open && !(fmax(fabs(G[0][1] - G[1][0]), fmax(fabs(G[0][2] - G[2][0]), fabs(G[1][2] - G[2][1]))) <=
                        kClosed * size))
            *a.open = 1;
        if (a.m64 || a.m32) {
            const double v = G[0][0] + G[1][1] + G[2][2];
            const size_t o = static_cast<size_t>(beg) + 64 * e + lane;
            if (a.m64) a.m64[o] = v;
            if (a.m32) a.m32[o] = static_cast<float>(a.scale_m * v);
        }
        if (a.k64 || a.k32) {
            double K[3][3];
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    double v = 0.0;
#pragma unroll
                    for (int b = 0; b < 3; ++b)
#pragma unroll
                        for (int d = 0; d < 3; ++d) v += a.C6[6 * kVoigt[b][p] + kVoigt[d][q]] * G[b][d];
                    K[p][q] = v;
                }
            const double s[6] = {K[0][0], K[1][1], K[2][2], 0.5 * (K[1][2] + K[2][1]), 0.5 * (K[0][2] + K[2][0]),
                                 0.5 * (K[0][1] + K[1][0])};
            const size_t o = (static_cast<size_t>(beg) + 64 * e) * 6 + lane;
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                if (a.k64) a.k64[o + 64 * t] = s[t];
                if (a.k32) a.k32[o + 64 * t] = static_cast<float>(a.scale_k * s[t]);
            }
        }
    }
}

void launch_operator_rows(OperatorBuild a, hipStream_t s) {
    a.parts = 4;                           // waves per slice
    const int64_t waves = static_cast<int64_t>(a.parts) * ((a.ly.n + 63) / 64);
    hipLaunchKernelGGL(k_operator_rows, dim3(static_cast<unsigned>((waves * 64 + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, a);
}

}  // namespace gspm
