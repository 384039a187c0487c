// Kernels of the learned elastic warm start (layout and network in mpnn.h).
//
// Node GEMMs run on MFMA (v_mfma_f32_16x16x32_bf16): the output is computed
// transposed, out^T = W x in^T, so the weights are the A operand (held in VGPRs
// for the whole launch) and each lane stores four consecutive channels of one
// node row.  Edge passes give one wave to a node with lane = channel, so every
// neighbour row is one coalesced read and the edge's vector and neighbour index,
// kept per edge, are the same in every lane: they come by scalar loads and cost
// no vector instruction.  A workgroup takes a contiguous run of nodes and an XCD
// a contiguous run of workgroups, so that the rows gathered stay in its caches.
//
// The edge passes are bound by vector instructions (two transcendentals per
// message and channel, 4 x 4 cycles each a wave), the GEMMs by memory.  At 97k
// nodes a layer takes, in us (in brackets as one wave a node with the edge
// vectors recomputed and broadcast, partials by 4-wave workgroups, weight
// gradients through a transposed LDS tile, and a reduction after each):
//   edges forward 56 (74), backward 116 (305); node GEMMs forward 14 + 15 (20 +
//   21), backward 17 + 25 (23 + 29); weight gradients 15 + 16 (74 + 81) with the
//   bias sums (20) among them; the reductions of all layers in one, 10 (1270).

#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "mpnn.h"

namespace gspm {
namespace mpnn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = kThreads / 64, kXcds = 8;
constexpr int kBatch = 8;       // rows loaded before they are used
// Passes that leave a partial gradient per workgroup: one workgroup a CU (the
// partials are then 52 MB) with sixteen waves, four a SIMD, to hide the gathers.
constexpr int kEdgeWgs = 2048, kGemmWgs = 512;    // eight waves a SIMD; two
constexpr int kEncNodes = 16;   // nodes whose inputs a wave forms at once
constexpr int kWideThreads = 1024, kWideWaves = kWideThreads / 64;

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// FP32 -> BF16 bits, round to nearest, ties to even; NaN stays NaN (one instruction for two).
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
    const floatx2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}
__device__ __forceinline__ uint16_t f2bf(float f) { return static_cast<uint16_t>(f2bf2(f, f)); }
__device__ __forceinline__ float round_bf(float f) { return bf2f(f2bf(f)); }

__device__ __forceinline__ float silu(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
    const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-z));
    return fmaf(s, fmaf(-z, s, z), s);      // s (1 + z (1 - s))
}

__device__ __forceinline__ float rdlane(float v, int t) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), t));
}

__device__ __forceinline__ bf16x8 as_bf8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Eight consecutive values of an input row as loaded and, FP32 ones rounded to
// BF16, as an MFMA operand.
struct Raw16 { uint4 v; };
struct Raw32 { float4 a, b; };
__device__ __forceinline__ Raw16 load8(const uint16_t *p) { return {*reinterpret_cast<const uint4 *>(p)}; }
__device__ __forceinline__ Raw32 load8(const float *p) {
    return {reinterpret_cast<const float4 *>(p)[0], reinterpret_cast<const float4 *>(p)[1]};
}
__device__ __forceinline__ bf16x8 operand(const Raw16 &r) { return as_bf8(r.v); }
__device__ __forceinline__ bf16x8 operand(const Raw32 &r) {
    return as_bf8(make_uint4(f2bf2(r.a.x, r.a.y), f2bf2(r.a.z, r.a.w), f2bf2(r.b.x, r.b.y), f2bf2(r.b.z, r.b.w)));
}

int grid_for(int64_t items, int per_block) {
    int64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > 8192) g = 8192;
    return static_cast<int>(g);
}

// The directed edges of node i, in the order of its neighbours: the nearest-image
// vector (x_j - x_i) / hbar and j.
__global__ void __launch_bounds__(kThreads) k_edges(MeshView mv, int n, float ihbar, const int32_t *ptr,
                                                    const int32_t *nbr, float4 *edge) {
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
        const double xi = mv.x[i], yi = mv.y[i], zi = mv.z[i];
        for (int t = ptr[i]; t < ptr[i + 1]; ++t) {
            const int j = nbr[t];
            edge[t] = make_float4(static_cast<float>(near_image(mv.x[j] - xi, mv.Lx, mv.iLx)) * ihbar,
                                  static_cast<float>(near_image(mv.y[j] - yi, mv.Ly, mv.iLy)) * ihbar,
                                  static_cast<float>(near_image(mv.z[j] - zi, mv.Lz, mv.iLz)) * ihbar,
                                  __int_as_float(j));
        }
    }
}

// Nodes of this workgroup: runs of `per` nodes, the runs of the workgroups an
// XCD gets (every eighth) next to each other.
__device__ __forceinline__ void node_run(int n, int &r0, int &r1) {
    const int nwg = gridDim.x, b = blockIdx.x, q = nwg / kXcds, r = nwg % kXcds, x = b % kXcds;
    const int at = x * q + min(x, r) + b / kXcds;
    const int per = (n + nwg - 1) / nwg;
    r0 = static_cast<int>(min(static_cast<int64_t>(n), static_cast<int64_t>(at) * per));
    r1 = min(n, r0 + per);
}

// The wave's number in its workgroup, as a scalar.
__device__ __forceinline__ int wave_of() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

using ScalarInt = const __attribute__((address_space(4))) int32_t;
using ScalarEdge = const __attribute__((address_space(4))) floatx4;

// ------------------------------------------------------------ node GEMMs

enum Epi { EPI_BF16 = 0, EPI_RESID_BF16 = 1, EPI_F32 = 2, EPI_ADD2_F32 = 3 };

struct GemmArgs {
    void *out;
    int ldo;
    const uint16_t *res;        // EPI_RESID_BF16: out = res + acc + bias
    int ldr;
    const float *bias;
    const float *add0, *add1;   // EPI_ADD2_F32: out = acc + add0 + add1
    int lda0, lda1;
    const int32_t *ptr;         // EPI_F32: columns from 64 on are divided by row r's ptr[r + 1] - ptr[r] (0: times 0)
};

// out[r][o] = sum_k in[r][k] W[o][k] for r < n, with in = [src0 | src1]
// (64 columns each when K = 128, src0 alone when K = 64).  W is O x K BF16.
template <int O, int K, class TIn, int EPI>
__global__ void __launch_bounds__(kThreads) k_rowgemm(int n, const TIn *src0, int ld0, const TIn *src1, int ld1,
                                                      const uint16_t *W, GemmArgs ga) {
    constexpr int OT = O / 16, KS = K / 32;
    const int lane = threadIdx.x & 63, grp = lane >> 4, col = lane & 15;
    bf16x8 wa[OT][KS];
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) wa[ot][ks] = operand(load8(W + (ot * 16 + col) * K + ks * 32 + grp * 8));
    const int ntile = (n + 15) >> 4, step = gridDim.x * kWaves;
    decltype(load8(src0)) in[KS];
    // rows beyond the last are the last's, and not stored
    auto fetch = [&](int tile) {
        const size_t row = min(min(tile, ntile - 1) * 16 + col, n - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = ks * 32 + grp * 8;
            in[ks] = K == 64 || ks < 2 ? load8(src0 + row * ld0 + k) : load8(src1 + row * ld1 + (k - 64));
        }
    };
    const int first = blockIdx.x * kWaves + wave_of();
    fetch(first);
    for (int tile = first; tile < ntile; tile += step) {
        const int row = tile * 16 + col;
        const bool live = row < n;
        bf16x8 xb[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) xb[ks] = operand(in[ks]);
        fetch(tile + step);      // the next tile's rows, while this one's are used
        floatx4 acc[OT];
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) {
            acc[ot] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                acc[ot] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[ot][ks], xb[ks], acc[ot], 0, 0, 0);
        }
        if (!live) continue;
        float ideg = 0.0f;
        if (EPI == EPI_F32) {
            const int deg = ga.ptr[row + 1] - ga.ptr[row];
            ideg = deg > 0 ? 1.0f / static_cast<float>(deg) : 0.0f;
        }
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) {
            const int o = ot * 16 + grp * 4;     // this lane holds out[row][o .. o+3]
            float v[4] = {acc[ot][0], acc[ot][1], acc[ot][2], acc[ot][3]};
            if (EPI == EPI_BF16 || EPI == EPI_RESID_BF16) {
                if (EPI == EPI_RESID_BF16) {
                    const uint2 rr = *reinterpret_cast<const uint2 *>(ga.res + static_cast<size_t>(row) * ga.ldr + o);
                    v[0] += bf2f(rr.x & 0xffffu) + ga.bias[o];
                    v[1] += bf2f(rr.x >> 16) + ga.bias[o + 1];
                    v[2] += bf2f(rr.y & 0xffffu) + ga.bias[o + 2];
                    v[3] += bf2f(rr.y >> 16) + ga.bias[o + 3];
                }
                uint2 st;
                st.x = f2bf2(v[0], v[1]);
                st.y = f2bf2(v[2], v[3]);
                *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(ga.out) + static_cast<size_t>(row) * ga.ldo + o) =
                    st;
            } else {
                if (EPI == EPI_ADD2_F32) {
                    const float4 a0 = *reinterpret_cast<const float4 *>(ga.add0 + static_cast<size_t>(row) * ga.lda0 + o);
                    const float4 a1 = *reinterpret_cast<const float4 *>(ga.add1 + static_cast<size_t>(row) * ga.lda1 + o);
                    v[0] += a0.x + a1.x;
                    v[1] += a0.y + a1.y;
                    v[2] += a0.z + a1.z;
                    v[3] += a0.w + a1.w;
                }
                if (EPI == EPI_F32 && ot * 16 >= 64) {
                    v[0] *= ideg;
                    v[1] *= ideg;
                    v[2] *= ideg;
                    v[3] *= ideg;
                }
                *reinterpret_cast<float4 *>(static_cast<float *>(ga.out) + static_cast<size_t>(row) * ga.ldo + o) =
                    make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
}

template <int O, int K, class TIn, int EPI>
void rowgemm(int n, const TIn *src0, int ld0, const TIn *src1, int ld1, const uint16_t *W, const GemmArgs &ga,
             hipStream_t s) {
    hipLaunchKernelGGL((k_rowgemm<O, K, TIn, EPI>), dim3(std::min(kGemmWgs, grid_for((n + 15) / 16, kWaves))), dim3(kThreads), 0,
                       s, n, src0, ld0, src1, ld1, W, ga);
}

// Weight gradients: part[wg][o][k] = sum over the workgroup's rows of
// G[r][o] X[r][k], G FP32 (n x O, row stride ldg), X = [x0 | x1] BF16 (64 columns
// each), and, with COLSUM, part_b[wg][o] = sum of G[r][o] (O = 64).
//
// The contraction runs over rows, and an MFMA sums its k index in any order as
// long as both operands agree: lane (grp, col) holds rows base + 4 i + grp, i <
// 8, and of each row the four channels from 4 col on.  Each operand is then 8
// whole-row loads straight into registers, with no transposition, and operand
// (q, a) is channel 64 q + 4 col + a.  A wave keeps all O x K sums (128
// registers), the four waves' are added through LDS.
template <int O, int K, bool COLSUM>
__global__ void __launch_bounds__(kThreads) k_wgrad(int n, const float *G, int ldg, const uint16_t *x0,
                                                    const uint16_t *x1, float *part, float *part_b) {
    constexpr int OQ = O / 64, KQ = K / 64, R = 8;
    __shared__ __align__(16) float sums[2][O * K];
    const int lane = threadIdx.x & 63, wv = wave_of(), grp = lane >> 4, col = lane & 15;
    int r0, r1;
    node_run(n, r0, r1);
    floatx4 acc[OQ][4][KQ][4];
#pragma unroll
    for (int t = 0; t < O * K / 256; ++t) (&acc[0][0][0][0])[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    float cs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int base = r0 + 32 * wv; base < r1; base += 32 * kWaves) {
        float4 g[OQ][R];
        uint2 x[KQ][R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const size_t row = min(base + 4 * i + grp, r1 - 1);
#pragma unroll
            for (int q = 0; q < OQ; ++q) g[q][i] = *reinterpret_cast<const float4 *>(G + row * ldg + q * 64 + 4 * col);
#pragma unroll
            for (int q = 0; q < KQ; ++q)
                x[q][i] = *reinterpret_cast<const uint2 *>((q == 0 ? x0 : x1) + row * 64 + 4 * col);
        }
        if (base + 32 > r1) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const bool live = base + 4 * i + grp < r1;
#pragma unroll
                for (int q = 0; q < OQ; ++q)
                    g[q][i] = make_float4(live ? g[q][i].x : 0.0f, live ? g[q][i].y : 0.0f, live ? g[q][i].z : 0.0f,
                                          live ? g[q][i].w : 0.0f);
#pragma unroll
                for (int q = 0; q < KQ; ++q) x[q][i] = make_uint2(live ? x[q][i].x : 0u, live ? x[q][i].y : 0u);
            }
        }
        uint4 xb[KQ][4];
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            auto lo = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); };
            auto hi = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };
            xb[q][0] = make_uint4(lo(x[q][0].x, x[q][1].x), lo(x[q][2].x, x[q][3].x), lo(x[q][4].x, x[q][5].x),
                                  lo(x[q][6].x, x[q][7].x));
            xb[q][1] = make_uint4(hi(x[q][0].x, x[q][1].x), hi(x[q][2].x, x[q][3].x), hi(x[q][4].x, x[q][5].x),
                                  hi(x[q][6].x, x[q][7].x));
            xb[q][2] = make_uint4(lo(x[q][0].y, x[q][1].y), lo(x[q][2].y, x[q][3].y), lo(x[q][4].y, x[q][5].y),
                                  lo(x[q][6].y, x[q][7].y));
            xb[q][3] = make_uint4(hi(x[q][0].y, x[q][1].y), hi(x[q][2].y, x[q][3].y), hi(x[q][4].y, x[q][5].y),
                                  hi(x[q][6].y, x[q][7].y));
        }
#pragma unroll
        for (int q = 0; q < OQ; ++q)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                float v[R];
#pragma unroll
                for (int i = 0; i < R; ++i) v[i] = a == 0 ? g[q][i].x : a == 1 ? g[q][i].y : a == 2 ? g[q][i].z : g[q][i].w;
                if (COLSUM) cs[a] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                const bf16x8 ga = as_bf8(
                    make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7])));
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq)
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        acc[q][a][kq][b] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(ga, as_bf8(xb[kq][b]), acc[q][a][kq][b], 0, 0, 0);
            }
    }
    // this lane's sums: o = 64 q + 4 (4 grp + i) + a, k = 64 kq + 4 col + b
    auto each = [&](auto f) {
#pragma unroll
        for (int q = 0; q < OQ; ++q)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        f((q * 64 + 4 * (4 * grp + i) + a) * K + kq * 64 + 4 * col, acc[q][a][kq][0][i],
                          acc[q][a][kq][1][i], acc[q][a][kq][2][i], acc[q][a][kq][3][i]);
    };
    auto put = [&](float *to) {
        each([&](int at, float a, float b, float c, float d) {
            *reinterpret_cast<float4 *>(to + at) = make_float4(a, b, c, d);
        });
    };
    auto add = [&](const float *from) {
#pragma unroll
        for (int q = 0; q < OQ; ++q)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int kq = 0; kq < KQ; ++kq)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float4 t = *reinterpret_cast<const float4 *>(
                            from + (q * 64 + 4 * (4 * grp + i) + a) * K + kq * 64 + 4 * col);
                        acc[q][a][kq][0][i] += t.x;
                        acc[q][a][kq][1][i] += t.y;
                        acc[q][a][kq][2][i] += t.z;
                        acc[q][a][kq][3][i] += t.w;
                    }
    };
    static_assert(kWaves == 4, "the waves' sums are added in two rounds");
    if (wv >= 2) put(sums[wv - 2]);
    __syncthreads();
    if (wv < 2) add(sums[wv]);
    __syncthreads();
    if (wv == 1) put(sums[0]);
    __syncthreads();
    if (wv == 0) {
        add(sums[0]);
        put(part + static_cast<size_t>(blockIdx.x) * kPartStride);
    }
    if (COLSUM) {
        float *c = sums[1];      // read last before the second barrier
#pragma unroll
        for (int a = 0; a < 4; ++a) c[(wv * 4 + grp) * 64 + 4 * col + a] = cs[a];
        __syncthreads();
        if (threadIdx.x < 64) {
            float t = 0.0f;
#pragma unroll
            for (int q = 0; q < 4 * kWaves; ++q) t += c[q * 64 + threadIdx.x];
            part_b[static_cast<size_t>(blockIdx.x) * kPartStride + threadIdx.x] = t;
        }
    }
}

// out[j] = sum_w part[w][j] over all parameters (FP64 accumulation in a fixed
// order: four waves take a quarter of the partials of 64 parameters each).
__global__ void __launch_bounds__(kThreads) k_reduce_part(const float *part, int nwg, int count, float *out) {
    __shared__ double sums[kWaves][64];
    const int lane = threadIdx.x & 63, wv = wave_of(), j = blockIdx.x * 64 + lane;
    const int per = (nwg + kWaves - 1) / kWaves, w0 = wv * per, w1 = min(nwg, w0 + per);
    double s = 0.0;
    if (j < count) {
        int w = w0;
        for (; w + 16 <= w1; w += 16) {
            float v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = part[static_cast<size_t>(w + q) * kPartStride + j];
#pragma unroll
            for (int q = 0; q < 16; ++q) s += v[q];
        }
        for (; w < w1; ++w) s += part[static_cast<size_t>(w) * kPartStride + j];
    }
    sums[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && j < count) out[j] = static_cast<float>((sums[0][lane] + sums[1][lane]) + (sums[2][lane] + sums[3][lane]));
}

// ------------------------------------------------------------ node passes

// Sharded sums of w |m - mprev|^2 and w.
__global__ void __launch_bounds__(kThreads) k_dm_sums(int n, const double *w, const double *m, const double *mp,
                                                      double *red) {
    double a[2] = {0.0, 0.0};
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
        double d2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double d = m[static_cast<size_t>(c) * n + i] - mp[static_cast<size_t>(c) * n + i];
            d2 += d * d;
        }
        a[0] += w[i] * d2;
        a[1] += w[i];
    }
    block_atomic_add<2>(a, red + R_DM2 * kShards, kShards);
}

__device__ __forceinline__ double dm_scale(const double *red) {
    const double *const src[2] = {red + R_DM2 * kShards, red + R_W * kShards};
    double t[2];
    shard_totals<2>(src, t);
    return t[1] > 0.0 ? sqrt(t[0] / t[1]) : 0.0;
}

// The 7 node inputs tag [dm / s_m, m, 1] (zero off the magnetic nodes),
// rounded to BF16 as the network stores them.
__device__ __forceinline__ void node_features(int n, int i, const double *w, const double *m, const double *mp,
                                              double ism, float (&x)[kIn]) {
    const bool mag = w[i] > 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double mc = m[static_cast<size_t>(c) * n + i];
        x[c] = mag ? round_bf(static_cast<float>((mc - mp[static_cast<size_t>(c) * n + i]) * ism)) : 0.0f;
        x[3 + c] = mag ? round_bf(static_cast<float>(mc)) : 0.0f;
    }
    x[6] = mag ? 1.0f : 0.0f;
}

// h0 = SiLU(W0 x + b0), lane = channel; a wave's lanes first form the inputs of
// a node each, which are then broadcast.
__global__ void __launch_bounds__(kThreads) k_encode(int n, const double *w, const double *m, const double *mp,
                                                     const double *red, const float *wr, uint16_t *H0) {
    const double sm = dm_scale(red), ism = sm > 0.0 ? 1.0 / sm : 0.0;
    const int lane = threadIdx.x & 63;
    float w0[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) w0[k] = wr[kOffW0 + lane * kIn + k];
    const float b0 = wr[kOffB0 + lane];
    for (int base = (blockIdx.x * kWaves + wave_of()) * kEncNodes; base < n; base += gridDim.x * kWaves * kEncNodes) {
        const int cnt = min(kEncNodes, n - base);
        float x[kIn];
        node_features(n, base + min(lane, cnt - 1), w, m, mp, ism, x);
        for (int t = 0; t < cnt; ++t) {
            float pre = b0;
#pragma unroll
            for (int k = 0; k < kIn; ++k) pre += w0[k] * rdlane(x[k], t);
            H0[static_cast<size_t>(base + t) * kHid + lane] = f2bf(silu(pre));
        }
    }
}

// a_i = mean_j SiLU(A_i + B_j + We e_ij + c).
__global__ void __launch_bounds__(kThreads) k_edge_fwd(Graph g, const float *wl, const uint16_t *AB, uint16_t *AGG) {
    ScalarInt *ptr = (ScalarInt *)g.ptr;
    ScalarEdge *edge = (ScalarEdge *)g.edge;
    const int lane = threadIdx.x & 63;
    const float we0 = wl[kLWe + lane * 3], we1 = wl[kLWe + lane * 3 + 1], we2 = wl[kLWe + lane * 3 + 2];
    const float cb = wl[kLC + lane];
    int r0, r1;
    node_run(g.n, r0, r1);
    for (int i = r0 + wave_of(); i < r1; i += kWaves) {
        const int beg = ptr[i], end = ptr[i + 1];
        const float ai = bf2f(AB[static_cast<size_t>(i) * 128 + lane]) + cb;
        float acc = 0.0f;
        // eight neighbour rows in flight at a time: the loads are issued back
        // to back (clamped to the last neighbour), then used in pairs
        for (int t0 = beg; t0 < end; t0 += kBatch) {
            floatx4 e[kBatch];
            float bv[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) e[u] = edge[min(t0 + u, end - 1)];
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                bv[u] = bf2f(AB[static_cast<size_t>(__float_as_int(e[u][3])) * 128 + 64 + lane]);
            // (the loads stay here, not with the branches that use them)
#pragma unroll
            for (int u = 0; u < kBatch; ++u) asm volatile("" : "+v"(bv[u]));
            auto message = [&](int u) {
                acc += silu(ai + bv[u] + we0 * e[u][0] + we1 * e[u][1] + we2 * e[u][2]);
            };
#pragma unroll
            for (int u = 0; u < kBatch; u += 2) {
                if (t0 + u + 2 <= end) {
                    message(u);
                    message(u + 1);
                } else if (t0 + u < end) {
                    message(u);
                }
            }
        }
        const int deg = end - beg;
        AGG[static_cast<size_t>(i) * kHid + lane] = f2bf(deg > 0 ? acc / static_cast<float>(deg) : 0.0f);
    }
}

// y = Wd h + bd (FP32, n x 3); optionally d = scale (y - y_p0) as 3 x n FP64.
__global__ void __launch_bounds__(kThreads) k_decode(int n, int p0, const uint16_t *H, const float *wr,
                                                     const double *red, double lambda100, double hbar, float *y,
                                                     double *dvec) {
    const double sm = dm_scale(red), scale = lambda100 * hbar * sm;
    auto dec = [&](int i, float (&o)[3]) {
        o[0] = wr[kOffBd];
        o[1] = wr[kOffBd + 1];
        o[2] = wr[kOffBd + 2];
        const uint4 *row = reinterpret_cast<const uint4 *>(H + static_cast<size_t>(i) * kHid);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const uint4 v = row[q];
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int c = q * 8 + h * 2;
                const float h0 = bf2f(u[h] & 0xffffu), h1 = bf2f(u[h] >> 16);
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    o[a] += wr[kOffWd + a * kHid + c] * h0 + wr[kOffWd + a * kHid + c + 1] * h1;
            }
        }
    };
    float op[3] = {0.0f, 0.0f, 0.0f};
    if (dvec) dec(p0, op);
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
        float o[3];
        dec(i, o);
#pragma unroll
        for (int a = 0; a < 3; ++a) y[static_cast<size_t>(i) * 3 + a] = o[a];
        if (dvec) {
#pragma unroll
            for (int a = 0; a < 3; ++a)
                dvec[static_cast<size_t>(a) * n + i] = i == p0 ? 0.0 : scale * (static_cast<double>(o[a]) - op[a]);
        }
    }
}

// ------------------------------------------------------------ loss

// Sharded sums of y (3) and of the normalised target t = du / (lambda100 hbar s_m) (3).
__global__ void __launch_bounds__(kThreads) k_loss_sums(int n, const float *y, const double *du, double lambda100,
                                                        double hbar, double *red) {
    const double sm = dm_scale(red);
    const double it = sm > 0.0 ? 1.0 / (lambda100 * hbar * sm) : 0.0;
    double a[6] = {0, 0, 0, 0, 0, 0};
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            a[c] += y[static_cast<size_t>(i) * 3 + c];
            a[3 + c] += du[static_cast<size_t>(c) * n + i] * it;
        }
    }
    block_atomic_add<6>(a, red + R_Y * kShards, kShards);
}

// gy = 2 ((y - ybar) - (t - tbar)) / (3n); loss = sum of squares / (3n).
__global__ void __launch_bounds__(kThreads) k_loss_grad(int n, const float *y, const double *du, double lambda100,
                                                        double hbar, double *red, float *gy) {
    const double sm = dm_scale(red);
    const double it = sm > 0.0 ? 1.0 / (lambda100 * hbar * sm) : 0.0;
    const double *const src[6] = {red + R_Y * kShards,       red + (R_Y + 1) * kShards, red + (R_Y + 2) * kShards,
                                  red + R_T * kShards,       red + (R_T + 1) * kShards, red + (R_T + 2) * kShards};
    double mean[6];
    shard_totals<6>(src, mean);
    const double inv3n = 1.0 / (3.0 * n);
    double acc[1] = {0.0};
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double d = (y[static_cast<size_t>(i) * 3 + c] - mean[c] / n) -
                             (du[static_cast<size_t>(c) * n + i] * it - mean[3 + c] / n);
            acc[0] += d * d * inv3n;
            gy[static_cast<size_t>(i) * 3 + c] = static_cast<float>(2.0 * d * inv3n);
        }
    }
    block_atomic_add<1>(acc, red + R_LOSS * kShards, kShards);
}

// ------------------------------------------------------------ backward

// Sum NV per-lane FP32 values over the workgroup's waves; lane c (< lanes)
// writes value k to dst[c * sl + k * sk].
template <int NV>
__device__ __forceinline__ void wave_sum_to_part(const float (&v)[NV], float *dst, int lanes, int sl, int sk) {
    __shared__ float red[kWideWaves][NV][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wv][k][lane] = v[k];
    __syncthreads();
    for (int t = threadIdx.x; t < NV * 64; t += kWideThreads) {
        const int k = t >> 6;
        if (lane >= lanes) continue;
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < kWideWaves; ++q) s += red[q][k][lane];
        dst[lane * sl + k * sk] = s;
    }
    __syncthreads();
}

// gh = gy Wd (n x 64); partials of dWd (3 x 64, [a][c]) and dbd (3).
__global__ void __launch_bounds__(kWideThreads) k_dec_bwd(int n, const uint16_t *H, const float *gy, const float *wr,
                                                      float *gh, float *part) {
    const int lane = threadIdx.x & 63;
    const float wd0 = wr[kOffWd + lane], wd1 = wr[kOffWd + kHid + lane], wd2 = wr[kOffWd + 2 * kHid + lane];
    float sw[3] = {0.0f, 0.0f, 0.0f}, sb[3] = {0.0f, 0.0f, 0.0f};
    int r0, r1;
    node_run(n, r0, r1);
#pragma unroll 4
    for (int i = r0 + wave_of(); i < r1; i += kWideWaves) {
        const float g0 = gy[static_cast<size_t>(i) * 3], g1 = gy[static_cast<size_t>(i) * 3 + 1],
                    g2 = gy[static_cast<size_t>(i) * 3 + 2];
        const float h = bf2f(H[static_cast<size_t>(i) * kHid + lane]);
        gh[static_cast<size_t>(i) * kHid + lane] = g0 * wd0 + g1 * wd1 + g2 * wd2;
        sw[0] += g0 * h;
        sw[1] += g1 * h;
        sw[2] += g2 * h;
        sb[0] += g0;     // every lane sees the same gy; lane 0's sums are the ones kept
        sb[1] += g1;
        sb[2] += g2;
    }
    float *dst = part + static_cast<size_t>(blockIdx.x) * kPartStride;
    wave_sum_to_part<3>(sw, dst, 64, 1, kHid);
    wave_sum_to_part<3>(sb, dst + 3 * kHid, 1, 0, 1);
}

// Edge backward of one layer: given ga = d a / degree (gha[:, 64:]), writes
// gab = [dA | dB] and partials of dWe (64 x 3) and dc (64).  A node's own ga is
// taken out of its sums.
__global__ void __launch_bounds__(kWideThreads) k_edge_bwd(Graph g, const float *wl, const uint16_t *AB,
                                                           const float *gha, float *gab, float *part) {
    ScalarInt *ptr = (ScalarInt *)g.ptr;
    ScalarEdge *edge = (ScalarEdge *)g.edge;
    const int lane = threadIdx.x & 63;
    const float we0 = wl[kLWe + lane * 3], we1 = wl[kLWe + lane * 3 + 1], we2 = wl[kLWe + lane * 3 + 2];
    const float cb = wl[kLC + lane];
    float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int r0, r1;
    node_run(g.n, r0, r1);
    for (int v = r0 + wave_of(); v < r1; v += kWideWaves) {
        const int beg = ptr[v], end = ptr[v + 1];
        const size_t rv = static_cast<size_t>(v) * 128 + lane;
        const float av = bf2f(AB[rv]) + cb, bv = bf2f(AB[rv + 64]) + cb, gav = gha[rv + 64];
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f}, gB = 0.0f;
        for (int t0 = beg; t0 < end; t0 += kBatch) {
            floatx4 e[kBatch];
            float au[kBatch], bu[kBatch], gu[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) e[q] = edge[min(t0 + q, end - 1)];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const size_t ru = static_cast<size_t>(__float_as_int(e[q][3])) * 128;
                au[q] = bf2f(AB[ru + lane]);
                bu[q] = bf2f(AB[ru + 64 + lane]);
                gu[q] = gha[ru + 64 + lane];
            }
            auto message = [&](int q) {
                const float e0 = e[q][0], e1 = e[q][1], e2 = e[q][2];
                const float wde = we0 * e0 + we1 * e1 + we2 * e2;
                // edge v -> u (message into v)
                const float d1 = dsilu(av + bu[q] + wde);
                t[0] += d1 * e0;
                t[1] += d1 * e1;
                t[2] += d1 * e2;
                t[3] += d1;
                // edge u -> v (message into u), edge vector -e
                gB += gu[q] * dsilu(au[q] + bv - wde);
            };
#pragma unroll
            for (int q = 0; q < kBatch; q += 2) {
                if (t0 + q + 2 <= end) {
                    message(q);
                    message(q + 1);
                } else if (t0 + q < end) {
                    message(q);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] += gav * t[k];
        gab[rv] = gav * t[3];
        gab[rv + 64] = gB;
    }
    float *dst = part + static_cast<size_t>(blockIdx.x) * kPartStride;
    const float we[3] = {s[0], s[1], s[2]};
    wave_sum_to_part<3>(we, dst, 64, 3, 1);          // dWe[c][a]
    const float c1[1] = {s[3]};
    wave_sum_to_part<1>(c1, dst + 3 * kHid, 64, 1, 0);   // dc[c]
}

// Encoder backward: partials of dW0 (64 x 7) and db0 (64).
__global__ void __launch_bounds__(kWideThreads) k_enc_bwd(int n, const double *w, const double *m, const double *mp,
                                                      const double *red, const float *wr, const float *gh,
                                                      float *part) {
    const double sm = dm_scale(red), ism = sm > 0.0 ? 1.0 / sm : 0.0;
    const int lane = threadIdx.x & 63;
    float w0[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) w0[k] = wr[kOffW0 + lane * kIn + k];
    const float b0 = wr[kOffB0 + lane];
    float s[kIn + 1] = {0, 0, 0, 0, 0, 0, 0, 0};
    int r0, r1;
    node_run(n, r0, r1);
    for (int base = r0 + wave_of() * kEncNodes; base < r1; base += kWideWaves * kEncNodes) {
        const int cnt = min(kEncNodes, r1 - base);
        float xl[kIn], gl[kEncNodes];
        node_features(n, base + min(lane, cnt - 1), w, m, mp, ism, xl);
#pragma unroll
        for (int t = 0; t < kEncNodes; ++t) gl[t] = gh[static_cast<size_t>(base + min(t, cnt - 1)) * kHid + lane];
#pragma unroll
        for (int t = 0; t < kEncNodes; ++t) {
            if (t >= cnt) continue;
            float x[kIn], pre = b0;
#pragma unroll
            for (int k = 0; k < kIn; ++k) {
                x[k] = rdlane(xl[k], t);
                pre += w0[k] * x[k];
            }
            const float gp = gl[t] * dsilu(pre);
#pragma unroll
            for (int k = 0; k < kIn; ++k) s[k] += gp * x[k];
            s[kIn] += gp;
        }
    }
    float *dst = part + static_cast<size_t>(blockIdx.x) * kPartStride;
    float wv[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) wv[k] = s[k];
    wave_sum_to_part<kIn>(wv, dst, 64, kIn, 1);          // dW0[c][k]
    const float bb[1] = {s[kIn]};
    wave_sum_to_part<1>(bb, dst + kHid * kIn, 64, 1, 0);  // db0[c]
}

// ------------------------------------------------------------ optimiser, weights

__global__ void __launch_bounds__(kThreads) k_adam(float *p, const float *g, float *m1, float *m2, float lr, float c1,
                                                   float c2) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    for (int j = blockIdx.x * kThreads + threadIdx.x; j < kNParam; j += gridDim.x * kThreads) {
        const float gj = g[j];
        const float a = b1 * m1[j] + (1.0f - b1) * gj;
        const float b = b2 * m2[j] + (1.0f - b2) * gj * gj;
        m1[j] = a;
        m2[j] = b;
        p[j] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
    }
}

__global__ void __launch_bounds__(kThreads) k_prepare(const float *p, float *wr, uint16_t *mats) {
    for (int j = blockIdx.x * kThreads + threadIdx.x; j < kNParam; j += gridDim.x * kThreads) wr[j] = round_bf(p[j]);
    for (int j = blockIdx.x * kThreads + threadIdx.x; j < kLayers * kMat; j += gridDim.x * kThreads) {
        const int l = j / kMat, q = j % kMat;
        const float *L = p + kOffL0 + l * kLayerSize;
        uint16_t *M = mats + static_cast<size_t>(l) * 4 * kMat;
        const uint16_t ab = f2bf(L[kLWa + q]);   // [Wa;Wb] row-major 128 x 64: row q / 64, col q % 64
        const uint16_t wu = f2bf(L[kLWu + q]);   // Wu 64 x 128: row q / 128, col q % 128
        M[q] = ab;
        M[kMat + q] = wu;
        M[2 * kMat + (q % 128) * 64 + q / 128] = wu;        // Wu^T 128 x 64
        M[3 * kMat + (q % 64) * 128 + q / 64] = ab;         // [Wa;Wb]^T 64 x 128
    }
}

// Sums of the least-squares system of the start on span{d, e}: (Kd.Kd, Kd.Ke,
// Ke.Ke, Kd.r0, Ke.r0); a null direction contributes 0.
__global__ void __launch_bounds__(kThreads) k_minres_sums(int n3, const double *d, const double *kd, const double *e,
                                                            const double *ke, const double *r0, double *red) {
    double a[kMrSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n3; i += gridDim.x * kThreads) {
        const double r = r0[i];
        const double kdi = d ? kd[i] : 0.0, kei = e ? ke[i] : 0.0;
        a[G_DKD] += kdi * kdi;
        a[G_DKE] += kdi * kei;
        a[G_EKE] += kei * kei;
        a[G_DR] += kdi * r;
        a[G_ER] += kei * r;
    }
    block_atomic_add<kMrSums>(a, red, kShards);
}

__device__ __forceinline__ void minres_coef(const double (&t)[kMrSums], double &ca, double &cc) {
    const double dd = t[G_DKD], de = t[G_DKE], ee = t[G_EKE], dr = t[G_DR], er = t[G_ER];
    const double det = dd * ee - de * de;
    ca = cc = 0.0;
    if (dd > 0.0 && ee > 0.0 && det > 1e-10 * dd * ee) {
        ca = (dr * ee - er * de) / det;
        cc = (er * dd - dr * de) / det;
    } else {
        const double gd = dd > 0.0 ? dr * dr / dd : 0.0, ge = ee > 0.0 ? er * er / ee : 0.0;
        if (gd >= ge) ca = dd > 0.0 ? dr / dd : 0.0;
        else cc = er / ee;
    }
    if (!__builtin_isfinite(ca) || !__builtin_isfinite(cc)) ca = cc = 0.0;
}

__global__ void __launch_bounds__(kThreads) k_minres_apply(int n3, const double *d, const double *e, double *x,
                                                             const double *red, double *coef) {
    const double *const src[kMrSums] = {red, red + kShards, red + 2 * kShards, red + 3 * kShards,
                                         red + 4 * kShards};
    double t[kMrSums];
    shard_totals<kMrSums>(src, t);
    double ca, cc;
    minres_coef(t, ca, cc);
    if (blockIdx.x == 0 && threadIdx.x == 0 && coef) {
        coef[0] = ca;
        coef[1] = cc;
    }
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < n3; i += gridDim.x * kThreads)
        x[i] += (d ? ca * d[i] : 0.0) + (e ? cc * e[i] : 0.0);
}

__global__ void __launch_bounds__(kThreads) k_sub(int64_t n3, const double *a, const double *b, double *out) {
    for (int64_t i = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; i < n3;
         i += static_cast<int64_t>(gridDim.x) * kThreads)
        out[i] = a[i] - b[i];
}

}  // namespace

// ------------------------------------------------------------ launchers

static void layer_gemm_ab(int n, const uint16_t *H, const uint16_t *wab, uint16_t *AB, hipStream_t s) {
    GemmArgs ga{};
    ga.out = AB;
    ga.ldo = 128;
    rowgemm<128, 64, uint16_t, EPI_BF16>(n, H, kHid, nullptr, 0, wab, ga, s);
}

void launch_forward(const Graph &g, const MeshView &mv, const Net &net, const double *m, const double *mprev,
                    double *red, const Acts &a, double lambda100, double *dvec, hipStream_t s) {
    const int n = g.n;
    launch_fill(red, R_COUNT * kShards, 0.0, s);
    hipLaunchKernelGGL(k_dm_sums, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, mv.w, m, mprev, red);
    hipLaunchKernelGGL(k_encode, dim3(grid_for(n, kWaves * kEncNodes)), dim3(kThreads), 0, s, n, mv.w, m, mprev, red, net.wr,
                       a.H[0]);
    for (int l = 0; l < kLayers; ++l) {
        const uint16_t *mats = net.mats + static_cast<size_t>(l) * 4 * kMat;
        const float *wl = net.wr + kOffL0 + l * kLayerSize;
        layer_gemm_ab(n, a.H[l], mats, a.AB[l], s);
        hipLaunchKernelGGL(k_edge_fwd, dim3(std::min(kEdgeWgs, grid_for(n, kWaves))), dim3(kThreads), 0, s, g, wl,
                           a.AB[l], a.AGG[l]);
        GemmArgs ga{};
        ga.out = a.H[l + 1];
        ga.ldo = kHid;
        ga.res = a.H[l];
        ga.ldr = kHid;
        ga.bias = wl + kLBu;
        rowgemm<64, 128, uint16_t, EPI_RESID_BF16>(n, a.H[l], kHid, a.AGG[l], kHid, mats + kMat, ga, s);
    }
    const double hbar = 1.0 / g.ihbar;
    hipLaunchKernelGGL(k_decode, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, mv.p0, a.H[kLayers], net.wr,
                       red, lambda100, hbar, a.y, dvec);
}

void launch_loss_backward(const Graph &g, const MeshView &mv, const Net &net, const double *m, const double *mprev,
                          const double *du, double lambda100, double *red, const Acts &a, const Grads &gr,
                          float *grad, hipStream_t s) {
    const int n = g.n;
    const double hbar = 1.0 / g.ihbar;
    hipLaunchKernelGGL(k_loss_sums, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, a.y, du, lambda100, hbar,
                       red);
    hipLaunchKernelGGL(k_loss_grad, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, s, n, a.y, du, lambda100, hbar,
                       red, gr.gy);
    const int nwg = gr.part_wgs;
    hipLaunchKernelGGL(k_dec_bwd, dim3(nwg), dim3(kWideThreads), 0, s, n, a.H[kLayers], gr.gy, net.wr, gr.gh,
                       gr.part + kOffWd);       // Wd then bd: contiguous
    for (int l = kLayers - 1; l >= 0; --l) {
        const uint16_t *mats = net.mats + static_cast<size_t>(l) * 4 * kMat;
        const float *wl = net.wr + kOffL0 + l * kLayerSize;
        float *pl = gr.part + kOffL0 + l * kLayerSize;
        // d[h ; a] = gh Wu  (n x 128), d a over the degree
        GemmArgs g1{};
        g1.out = gr.gha;
        g1.ldo = 128;
        g1.ptr = g.ptr;
        rowgemm<128, 64, float, EPI_F32>(n, gr.gh, kHid, nullptr, 0, mats + 2 * kMat, g1, s);
        // dWu = gh^T [H | AGG], dbu = sum gh
        hipLaunchKernelGGL((k_wgrad<64, 128, true>), dim3(nwg), dim3(kThreads), 0, s, n, gr.gh, kHid, a.H[l], a.AGG[l],
                           pl + kLWu, pl + kLBu);
        // edge pass: We (64 x 3) then c (64), contiguous in the layout
        hipLaunchKernelGGL(k_edge_bwd, dim3(nwg), dim3(kWideThreads), 0, s, g, wl, a.AB[l], gr.gha, gr.gab, pl + kLWe);
        // dWab = gab^T H
        hipLaunchKernelGGL((k_wgrad<128, 64, false>), dim3(nwg), dim3(kThreads), 0, s, n, gr.gab, 128, a.H[l], nullptr,
                           pl + kLWa, nullptr);
        // gh <- gh + d[h](from gha) + gab [Wa;Wb]
        GemmArgs g2{};
        g2.out = gr.gh;
        g2.ldo = kHid;
        g2.add0 = gr.gh;
        g2.lda0 = kHid;
        g2.add1 = gr.gha;
        g2.lda1 = 128;
        rowgemm<64, 128, float, EPI_ADD2_F32>(n, gr.gab, 128, gr.gab + 64, 128, mats + 3 * kMat, g2, s);
    }
    hipLaunchKernelGGL(k_enc_bwd, dim3(nwg), dim3(kWideThreads), 0, s, n, mv.w, m, mprev, red, net.wr, gr.gh,
                       gr.part + kOffW0);
    hipLaunchKernelGGL(k_reduce_part, dim3((kNParam + 63) / 64), dim3(kThreads), 0, s, gr.part, nwg, kNParam, grad);
}

void launch_edges(const Graph &g, const MeshView &mv, const int32_t *nbr, float *edge, hipStream_t s) {
    hipLaunchKernelGGL(k_edges, dim3(grid_for(g.n, kThreads)), dim3(kThreads), 0, s, mv, g.n, g.ihbar, g.ptr, nbr,
                       reinterpret_cast<float4 *>(edge));
}

void launch_adam(float *master, const float *grad, float *m1, float *m2, float lr, int64_t t, hipStream_t s) {
    const float c1 = static_cast<float>(1.0 - std::pow(0.9, static_cast<double>(t)));
    const float c2 = static_cast<float>(1.0 - std::pow(0.999, static_cast<double>(t)));
    hipLaunchKernelGGL(k_adam, dim3(grid_for(kNParam, kThreads)), dim3(kThreads), 0, s, master, grad, m1, m2, lr, c1,
                       c2);
}

void launch_prepare_weights(const float *master, float *wr, uint16_t *mats, hipStream_t s) {
    hipLaunchKernelGGL(k_prepare, dim3(grid_for(kNParam, kThreads)), dim3(kThreads), 0, s, master, wr, mats);
}

void launch_minres(int n, const double *d, const double *kd, const double *e, const double *ke, const double *r0,
                     double *x, double *red, double *coef, hipStream_t s) {
    const int n3 = 3 * n;
    launch_fill(red, kMrSums * kShards, 0.0, s);
    hipLaunchKernelGGL(k_minres_sums, dim3(grid_for(n3, kThreads)), dim3(kThreads), 0, s, n3, d, kd, e, ke, r0, red);
    hipLaunchKernelGGL(k_minres_apply, dim3(grid_for(n3, kThreads)), dim3(kThreads), 0, s, n3, d, e, x, red, coef);
}

void launch_sub(int64_t n3, const double *a, const double *b, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_sub, dim3(grid_for(n3, kThreads)), dim3(kThreads), 0, s, n3, a, b, out);
}

}  // namespace mpnn
}  // namespace gspm
