// Whole CG solves in one launch, their vectors on the chip.
//
// The CG iterations of the step are small: at 100k nodes a GS iteration moves
// 20 to 40 MB and at 1000 nodes next to nothing, so a launch for each of them
// is bound by the launch and by its chain of dependent phases.  Here one
// cooperative launch of at most one workgroup per CU runs a solve to its end:
// the start's residual, the CG iterations, and in the mixed form every FP64
// refinement around the FP32 inner solves.  Each workgroup owns a contiguous
// range of rows of the assembled operator; r, x and q of its rows stay in
// registers, p of its rows and of their halo columns in LDS, and so do the
// rows' coefficients where a thread has one row (beyond, they stream from L2
// and Infinity Cache).  An iteration by launches (with the gaps between them)
// against one here, us, FP64 / FP32 inner:
//   GS, three components: 729 nodes 13.4 -> 4.1 / -; 97k 19.3 -> 6.6 / 22.1 ->
//   6.1; 358k 42 -> 18 / 30 -> 14; 970k - / 54 -> 29, where the rows' stream of
//   85 MB from Infinity Cache would take 12 at that cache's copy rate;
//   elastic: 729 nodes 20.2 -> 3.4 / 18.0 -> 3.2; 97k 28.7 -> 8.1 / 20.7 -> 5.4;
//   149k 36 -> 20 / 26 -> 13; 250k 49 -> 29 / 32 -> 18;
//   K^ms, three components: 250k 59 -> 12 / 41 -> 9; 970k - / 100 -> 24.
// A mixed solve also loses the host's turn in each refinement.
//
// The halo keeps its own r and p: every workgroup applies the same alpha and
// beta to the halo values it staged, so an iteration exchanges q alone, and q
// only of the nodes that are some other workgroup's halo.  One exchange per
// iteration: q and the workgroup's partial sums go out, the other workgroups'
// come in, and single-reduction CG (the scalars of ElasticCgOp and
// k_gs_rows_cg) needs nothing else.
//
// Exchanged values carry their own arrival mark: every 64-bit word holds 32
// bits of data and a 32-bit tag, written and read by relaxed agent-scope
// atomics, so a reader that sees the tag has the data and no fence, flag or
// cache flush is needed (across the XCDs' separate L2s neither).  Words
// alternate between two buffers: a workgroup writes round t + 2 only after it
// has all of round t + 1, which the others write after reading round t.  Up to
// kGroup workgroups read each other's sums directly; more of them go through
// leaders of kGroup workgroups (all-to-all over 256 workgroups took 6.8 us per
// exchange in a probe, two hops over groups of 16 about 3).  One wave sums
// either hop's slots straight from its loads, and a leader does so before it
// waits for its halo: with the slots polled by all, summed through LDS behind
// two barriers, and the leader's halo first, an elastic iteration of 97k nodes
// took 6.2 us in FP32 and 9.0 in FP64 instead of 5.7 and 8.4.
// All totals are added in a fixed order, the same in every workgroup, so all
// take the same decisions, and results repeat bitwise.
//
// Every wait is bounded (wait_ticks of the 100 MHz clock, 5 s unless the caller
// says otherwise): a workgroup whose wait runs out says so to the host and
// leaves, the others' waits run out in turn, and the host solves again from
// what x holds with a launch per iteration.  Cooperative launches are resident
// as a whole, but the clock runs on while the device serves another process,
// so a wait can run out in one workgroup and not in another: the outcome
// workgroup 0 reports counts only if none gave up.
#pragma once

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "resident.h"

namespace gspm {

namespace {

using u64 = unsigned long long;

constexpr int kTh = kResThreads;
constexpr int kHB = 4;                         // halo nodes per thread polled while the sums are on their way

// Nodes' values travel in 16-byte chunks of two words, each word with its own
// tag (a chunk is one access, but nothing relies on more than its words being
// whole): a double to a chunk, two floats to a chunk.  Chunks are stored
// [parity][chunk][export slot], so consecutive halo nodes of one neighbour are
// consecutive in memory.  (With 8-byte words node by node the exchange of a
// 97k-node FP64 iteration took 7 us instead of 3.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kAgent = 16;                     // cache policy of the accesses: sc1, as agent-scope atomics have

template <class S, int NC>
struct Wire {
    static constexpr int kChunks = sizeof(S) == 8 ? NC : (NC + 1) / 2;
    static __device__ __forceinline__ u32x4 pack(const S (&v)[NC], int j, uint32_t tag) {
        if constexpr (sizeof(S) == 8) {
            const u64 b = static_cast<u64>(__double_as_longlong(v[j]));
            return u32x4{static_cast<uint32_t>(b), tag, static_cast<uint32_t>(b >> 32), tag};
        } else {
            const float a = v[2 * j], c = 2 * j + 1 < NC ? v[2 * j + 1 < NC ? 2 * j + 1 : 0] : 0.0f;
            return u32x4{__float_as_uint(a), tag, __float_as_uint(c), tag};
        }
    }
    static __device__ __forceinline__ void unpack(const u32x4 (&w)[kChunks], S (&v)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (sizeof(S) == 8)
                v[c] = __longlong_as_double(static_cast<long long>(w[c][0] | (static_cast<u64>(w[c][2]) << 32)));
            else
                v[c] = __uint_as_float(w[c / 2][(c & 1) ? 2 : 0]);
        }
    }
};

struct Spin {
    long long t0 = 0;
    int n = 0;
    // true when the wait has run out (the clock is looked at every poll_mask + 1 polls)
    __device__ __forceinline__ bool over(const ResArgs &a) {
        if ((++n & a.poll_mask) != 0) return false;
        const long long t = wall_clock64();
        if (t0 == 0) t0 = t;
        return t - t0 > a.wait_ticks;
    }
};

// an LDS value that is the same in every lane, kept in scalar registers
__device__ __forceinline__ double uniform(double v) {
    const u64 b = static_cast<u64>(__double_as_longlong(v));
    const u64 lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b)));
    const u64 hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32)));
    return __longlong_as_double(static_cast<long long>(lo | (hi << 32)));
}

// the staged vector of a node: NC components, padded to 4 for NC = 3 so wide LDS reads fetch it
template <class T, int NC>
struct Vec {
    static constexpr int kPad = NC == 3 ? 4 : NC;
    T v[kPad];
};
// the FP64 staging of a residual is not padded
template <int NC>
struct VecX {
    double v[NC];
};

// Barrier of the workgroup for data in LDS alone.  __syncthreads() also waits
// for every outstanding global store, here the exchange's write-through
// stores: 4 us of a 13 us iteration.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A value from another lane of the same row of 16, by DPP.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return __uint_as_float(dpp<CTRL>(__float_as_uint(v))); }
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const u64 b = static_cast<u64>(__double_as_longlong(v));
    const u64 lo = dpp<CTRL>(static_cast<uint32_t>(b)), hi = dpp<CTRL>(static_cast<uint32_t>(b >> 32));
    return __longlong_as_double(static_cast<long long>(lo | (hi << 32)));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor7 = 0x141, kXor8 = 0x128;   // partner lane i ^ 1, i ^ 2, i ^ 7, i ^ 8

// Exchange halves of a pair of values between lanes that differ in bit 5 (or
// 4): a gets the lower lanes' a and b side by side, b the upper lanes'.
template <int BIT>
__device__ __forceinline__ void swap_halves(double &a, double &b) {
    const u64 x = static_cast<u64>(__double_as_longlong(a)), y = static_cast<u64>(__double_as_longlong(b));
    uint32_t w[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t p = static_cast<uint32_t>(x >> (32 * j)), q = static_cast<uint32_t>(y >> (32 * j));
        const auto r = BIT == 32 ? __builtin_amdgcn_permlane32_swap(p, q, false, false)
                                 : __builtin_amdgcn_permlane16_swap(p, q, false, false);
        w[0][j] = r[0];
        w[1][j] = r[1];
    }
    a = __longlong_as_double(static_cast<long long>(w[0][0] | (static_cast<u64>(w[0][1]) << 32)));
    b = __longlong_as_double(static_cast<long long>(w[1][0] | (static_cast<u64>(w[1][1]) << 32)));
}

// Sums of NV per-thread values over the wave: values and lanes are halved
// together (a lane bit decides which half of the values a lane goes on with),
// so 16 values take 15 + 2 exchanges instead of 6 each.  out[k] is written by
// the first lane of the group that ends with value k.
template <int NV>
__device__ __forceinline__ void wave_sums(const double (&v)[NV], double *out) {
    constexpr int P = NV > 8 ? 16 : NV > 4 ? 8 : 4;
    const int lane = threadIdx.x & 63;
    double a[P];
#pragma unroll
    for (int k = 0; k < P; ++k) a[k] = k < NV ? v[k] : 0.0;
    // lane bit 5, then bit 4
#pragma unroll
    for (int k = 0; k < P / 2; ++k) {
        swap_halves<32>(a[k], a[P / 2 + k]);
        a[k] += a[P / 2 + k];
    }
#pragma unroll
    for (int k = 0; k < P / 4; ++k) {
        swap_halves<16>(a[k], a[P / 4 + k]);
        a[k] += a[P / 4 + k];
    }
    if constexpr (P >= 8) {
        const bool up = (lane & 8) != 0;
#pragma unroll
        for (int k = 0; k < P / 8; ++k) {
            const double keep = up ? a[P / 8 + k] : a[k], give = up ? a[k] : a[P / 8 + k];
            a[k] = keep + dpp<kXor8>(give);
        }
    }
    if constexpr (P >= 16) {
        const bool up = (lane & 4) != 0;
        const double keep = up ? a[1] : a[0], give = up ? a[0] : a[1];
        a[0] = keep + dpp<kXor7>(give);
    }
    double s = a[0];
    if constexpr (P < 8) s += dpp<kXor8>(s);
    s += dpp<kXor1>(s);
    s += dpp<kXor2>(s);
    if constexpr (P < 16) s += dpp<kXor7>(s);
    constexpr int kLow = 64 / P;
    const int k = lane / kLow;
    if ((lane & (kLow - 1)) == 0 && k < NV) out[k] = s;
}

// Sum over the L lanes of a row, in every lane.
template <int L, class M>
__device__ __forceinline__ M lanes_sum(M v) {
    if constexpr (L >= 2) v += dpp<kXor1>(v);
    if constexpr (L >= 4) v += dpp<kXor2>(v);
    if constexpr (L >= 8) v += dpp<kXor7>(v);
    return v;
}

// A slice's first entry and width: the slice is the same for a whole wave, so
// both come by scalar loads.
struct Slice {
    int32_t beg, w;
};
__device__ __forceinline__ Slice slice_of(const ResLayout &ly, int g) {
    using CI = const __attribute__((address_space(4))) int32_t;
    CI *off = (CI *)(ly.off);
    const int sl = __builtin_amdgcn_readfirstlane(g >> 6);
    const int32_t b = off[sl];
    return Slice{b, (off[sl + 1] - b) >> 6};
}

// E entries of a row (entries l, l + L, ...): local columns and coefficients,
// one for all components or a symmetric 3x3 block (xx yy zz yz xz xy).
template <class M, bool BLK, int E>
struct Entries {
    M k[E][BLK ? 6 : 1];
    uint16_t c[E];
};

// Entries past the row's end take the coefficients of its first (in bounds)
// and the node `none` for a column (see add_entries).  With END_SELECT that choice is
// left to add_entries (made here, it would wait for the column's load), with
// END_BRANCH (whole waves on one slice, one lane per row) they are skipped.
enum RowEnd { END_LOADED, END_SELECT, END_BRANCH };
template <class M, bool BLK, int L, int E, RowEnd END>
__device__ __forceinline__ void load_entries(const M *A, const uint16_t *col, const Slice &sc, int lane, int l, int e0,
                                             int none, Entries<M, BLK, E> &en) {
    if (sc.w <= 0) {
#pragma unroll
        for (int u = 0; u < E; ++u) {
            en.c[u] = static_cast<uint16_t>(none);
#pragma unroll
            for (int t = 0; t < (BLK ? 6 : 1); ++t) en.k[u][t] = M(0);
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < E; ++u) {
        const int e = e0 + u * L + l;
        const int32_t o = sc.beg + 64 * (e < sc.w ? e : 0);
        const uint16_t c = col[o + lane];
        en.c[u] = END != END_LOADED || e < sc.w ? c : static_cast<uint16_t>(none);
#pragma unroll
        for (int t = 0; t < (BLK ? 6 : 1); ++t)
            en.k[u][t] = BLK ? A[static_cast<size_t>(o) * 6 + 64 * t + lane] : A[o + lane];
    }
}

// acc += the entries (e0 as they were loaded) times the staged vectors less
// `base`.  K^mech and K^ms map constants to zero, their diagonals are minus
// the sum of the row, and base is the row's own vector: rounding of the
// coefficients then acts on differences between neighbours, as it does in the
// element form (with a diagonal instead, FP32 rows left ten times the error in
// the smooth modes).  The GS operator has a diagonal and base is zero.  `none`
// is a staged node equal to base.
template <class M, int NC, bool BLK, int L, int E, RowEnd END, class V>
__device__ __forceinline__ void add_entries(const Entries<M, BLK, E> &en, const Slice &sc, int l, int e0, int none,
                                            const V *f, const M (&base)[NC], M (&acc)[NC]) {
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if (END != END_BRANCH || e0 + u < sc.w) {
            const V x = f[END != END_SELECT || e0 + u * L + l < sc.w ? en.c[u] : none];
            M d[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) d[q] = x.v[q] - base[q];
            if constexpr (BLK) {
                acc[0] += en.k[u][0] * d[0] + en.k[u][5] * d[1] + en.k[u][4] * d[2];
                acc[1] += en.k[u][5] * d[0] + en.k[u][1] * d[1] + en.k[u][3] * d[2];
                acc[2] += en.k[u][4] * d[0] + en.k[u][3] * d[1] + en.k[u][2] * d[2];
            } else {
#pragma unroll
                for (int q = 0; q < NC; ++q) acc[q] += en.k[u][0] * d[q];
            }
        }
    }
}

// the row's entries from e0 on, streamed
template <class M, int NC, bool BLK, int L, class V>
__device__ __forceinline__ void add_rest(const M *A, const uint16_t *col, const Slice &sc, int lane, int l, int e0,
                                         int none, const V *f, const M (&base)[NC], M (&acc)[NC]) {
    constexpr int kE = BLK ? (sizeof(M) == 8 ? 5 : 4) : 8;
    for (int e = e0; e < sc.w; e += kE * L) {
        Entries<M, BLK, kE> en;
        load_entries<M, BLK, L, kE, END_SELECT>(A, col, sc, lane, l, e, none, en);
        add_entries<M, NC, BLK, L, kE, END_SELECT>(en, sc, l, e, none, f, base, acc);
    }
}

}  // namespace

// NS scalar sets (one per component, one for all three in block form), each
// with the sums p.q, r.r, r.D^-1 r, r.D^-1 q, q.D^-1 q.
template <class T, int NC, bool BLK, int L, int RPT>
__global__ void __launch_bounds__(kTh) k_resident(const ResArgs a) {
    constexpr bool kMixed = sizeof(T) == 4;
    constexpr int NS = BLK ? 1 : NC;
    constexpr int NV = 5 * NS;
    constexpr int E = resident_entries(sizeof(T) == 4, BLK, L, RPT);
    // further entries of FP64 block rows in LDS, as many as fit (see resident_fits); the rest streams
    constexpr bool kLdsRows = BLK && sizeof(T) == 8 && RPT == 1 && L <= 2;
    // (fetched ahead with one lane a row, five; with two lanes registers and LDS hold a Kuhn mesh's rows, and loading
    // padding took an iteration of 39k nodes from 5.9 to 8.1 us)
    constexpr int kAhead = kLdsRows && L == 1 ? 5 : 0;
    constexpr int kBuf = RPT > 1 ? 2 : 1;
    using V = Vec<T, NC>;
    // components of x staged at once for an FP64 residual: all, but at eight FP32 rows per thread two (LDS)
    constexpr int XC = resident_xc(sizeof(T) == 4, NC, BLK, RPT);
    using X = VecX<XC>;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_part[kTh / 64][NV];
    __shared__ double s_tot[NV];
    __shared__ double s_al[NS], s_be[NS], s_bb[NS];
    // a wait ran out: before the round's last barrier (stable from there to the next exchange), or in the halo beyond
    // kHB nodes a thread, after it (looked at behind the next barrier)
    __shared__ int s_bad, s_late;
    const ResLayout &ly = a.ly;
    const int tid = threadIdx.x, n = ly.n, G = ly.G;
    const int wg = xcd_block(blockIdx.x, G);
    const int n0 = wg * ly.nbr, cnt = min(ly.nbr, n - n0);
    const int hbeg = ly.halo_ptr[wg], nhalo = ly.halo_ptr[wg + 1] - hbeg;
    const int zero = ly.nbr + nhalo;               // a staged node of zeros
    // rows that sum to zero: K^mech, K^ms (the only one-component solve)
    const bool zero_sum = BLK || NC == 1 || (NC == 3 && a.zero_sum != 0);
    const int l = tid & (L - 1), rstep = kTh / L, row00 = tid / L;
    // the row base, hidden from the optimiser in each phase: addresses are formed where they are used instead of
    // being kept in registers (and spilled) for every row over the whole solve
    auto base_row = [&]() {
        int v = row00;
        asm volatile("" : "+v"(v));
        return v;
    };
    // LDS: staging (p in T, or x in FP64) | halo r | halo 1/D | coefficients
    unsigned char *st = smem;
    V *f = reinterpret_cast<V *>(st);
    X *fx = reinterpret_cast<X *>(st);
    T *hr = reinterpret_cast<T *>(st + a.stage_bytes);
    T *hd = hr + static_cast<size_t>(NC) * nhalo;
    T *sk = hd + ((nhalo + 1) & ~1);               // [entry][6][lane] coefficients, then [entry][lane] columns
    uint16_t *sc_col = reinterpret_cast<uint16_t *>(sk + 6 * static_cast<size_t>(a.lds_entries) * a.lds_threads);
    const T *A = static_cast<const T *>(a.a), *D = static_cast<const T *>(a.d);
    if (tid == 0) s_bad = s_late = 0;
    uint32_t xt = a.epoch[0], rt = a.epoch[1];

    // export slots of the first halo nodes of this thread and of its rows, 1 / D of rows and halo
    int hid[kHB];
#pragma unroll
    for (int u = 0; u < kHB; ++u) {
        const int h = tid + u * kTh;
        hid[u] = h < nhalo ? ly.slot[ly.halo_ids[hbeg + h]] : -1;
    }
    auto slot_of = [&](int h) { return ly.slot[ly.halo_ids[hbeg + h]]; };
    auto inv_d = [&](int g) -> T {
        if (BLK || !a.jacobi) return T(1);
        const T d = D[g];
        return d > T(0) ? T(1) / d : T(0);
    };
    for (int h = tid; h < nhalo; h += kTh) hd[h] = inv_d(ly.halo_ids[hbeg + h]);
    T di[RPT];
    {
    const int row0 = base_row();
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
        const int row = row0 + s * rstep;
        di[s] = row < cnt ? inv_d(n0 + row) : T(0);
    }
    }
    int xport[RPT];
    {
    const int row0 = base_row();
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
        const int row = row0 + s * rstep;
        xport[s] = l == 0 && row < cnt ? ly.slot[n0 + row] : -1;
    }
    }
    if (tid < NS) {
        double t = 0.0;
        for (int sh = 0; sh < kShards; ++sh) t += a.bb[tid * kShards + sh];
        s_bb[tid] = t;
    }
    lds_barrier();
    double bb[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) bb[q] = uniform(s_bb[q]);

    int live[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) live[c] = 1;
    auto set = [](int c) { return BLK ? 0 : c; };

    const __amdgpu_buffer_rsrc_t xq = __builtin_amdgcn_make_buffer_rsrc(
        a.xq, 0, static_cast<int>(resident_xq_bytes(ly.nexp)), 0x00027000);
    auto xq_at = [&](int j, int slot) { return (((xt & 1) * kResChunks + j) * ly.nexp + slot) * 16; };
    // one exported row's values of this round
    auto publish = [&](int slot, const auto (&v)[NC]) {
        using W = Wire<std::remove_cv_t<std::remove_reference_t<decltype(v[0])>>, NC>;
#pragma unroll
        for (int j = 0; j < W::kChunks; ++j)
            __builtin_amdgcn_raw_buffer_store_b128(W::pack(v, j, xt), xq, xq_at(j, slot), 0, kAgent);
    };
    // B halo nodes' values of this round, all loads in flight; waits for them (slot < 0: none)
    auto fetch = [&](const auto &slot, auto &v, int &bad) {
        constexpr int B = sizeof(slot) / sizeof(slot[0]);
        using W = Wire<std::remove_cv_t<std::remove_reference_t<decltype(v[0][0])>>, NC>;
        u32x4 w[B][W::kChunks];
        Spin spin;
        for (;;) {
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (slot[u] >= 0)
#pragma unroll
                    for (int j = 0; j < W::kChunks; ++j)
                        w[u][j] = __builtin_amdgcn_raw_buffer_load_b128(xq, xq_at(j, slot[u]), 0, kAgent);
            bool ok = true;
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (slot[u] >= 0)
#pragma unroll
                    for (int j = 0; j < W::kChunks; ++j) ok &= w[u][j][1] == xt && w[u][j][3] == xt;
            if (ok) break;
            if (spin.over(a)) {
                bad = 1;
                break;
            }
            asm volatile("" ::: "memory");         // the next pass reads again
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (slot[u] >= 0) W::unpack(w[u], v[u]);
            else
#pragma unroll
                for (int c = 0; c < NC; ++c) v[u][c] = 0;
        }
    };
    // the workgroups' slots of NV sums, and the leaders'
    const __amdgpu_buffer_rsrc_t sums = __builtin_amdgcn_make_buffer_rsrc(
        a.slots, 0, static_cast<int>(resident_slot_bytes()), 0x00027000);
    auto put_sum = [&](int slot, int v, double t, uint32_t tag) {
        const u64 b = static_cast<u64>(__double_as_longlong(t));
        __builtin_amdgcn_raw_buffer_store_b128(
            u32x4{static_cast<uint32_t>(b), tag, static_cast<uint32_t>(b >> 32), tag}, sums, (slot * kSlotSums + v) * 16, 0, kAgent);
    };
    // The totals of value sl >> 2 (four lanes of one wave a value, in a fixed order) into s_tot,
    // and alpha and beta of the sets, by the lanes of sums 0 to NS - 1 (meaningful after an iteration's sums only).
    // (few workgroups have few halo nodes: the last wave has none and polls while the first wait for theirs; at 729
    // nodes 3.4 us an iteration against 3.7.  Beyond, every wave has some, and the first is 2 % the faster)
    const bool summer = tid >> 6 == (G <= kGroup ? kTh / 64 - 1 : 0);
    const int sl = tid & 63;
    static_assert(4 * NV <= 64, "four lanes per value");
    auto totals = [&](double t) {
        const int v = sl >> 2, part = sl & 3;
        if (part == 0 && v < NV) s_tot[v] = t;
        const double rr2 = __shfl(t, 4 * (2 * NS) + sl, 64), rzq = __shfl(t, 4 * (3 * NS) + sl, 64),
                     qzq = __shfl(t, 4 * (4 * NS) + sl, 64);
        if (part == 0 && v < NS) {
            const double alpha = rr2 / t, est = rr2 - 2.0 * alpha * rzq + alpha * alpha * qzq;
            s_al[v] = alpha;
            s_be[v] = (est > 0.0 ? est : 0.0) / rr2;
        }
    };
    // the sum of up to kGroup slots, by that wave alone and straight from the loads; over: this
    // lane's wait ran out
    auto wave_slots = [&](int first, int count, bool &over) -> double {
        static_assert(kGroup == 16, "four slots a lane");
        const int v = sl >> 2, part = sl & 3;
        u32x4 w[4];
        double t = 0.0;
        over = false;
        if (v < NV) {
            Spin spin;
            for (;;) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (part + 4 * u < count)
                        w[u] = __builtin_amdgcn_raw_buffer_load_b128(
                            sums, ((first + part + 4 * u) * kSlotSums + v) * 16, 0, kAgent);
                bool ok = true;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (part + 4 * u < count) ok &= w[u][1] == rt && w[u][3] == rt;
                if (ok) break;
                if (spin.over(a)) {
                    over = true;
                    s_bad = 1;
                    break;
                }
                asm volatile("" ::: "memory");     // the next pass reads again
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (part + 4 * u < count)
                    t += __longlong_as_double(static_cast<long long>(w[u][0] | (static_cast<u64>(w[u][2]) << 32)));
        }
        t += __shfl_xor(t, 1, 64);
        t += __shfl_xor(t, 2, 64);
        return t;
    };
    // this workgroup's partial sums out (part: per thread); returns after they are stored
    auto send_sums = [&](const double (&part)[NV]) {
        wave_sums<NV>(part, s_part[tid >> 6]);
        lds_barrier();
        if (tid < NV) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < kTh / 64; ++w) t += s_part[w][tid];
            put_sum((rt & 1) * kResMaxGroups + wg, tid, t, rt);
        }
    };
    // A leader's sum of its group out, before anything else is waited for: every other workgroup waits for it.  One that
    // is not whole, as a wait ran out, goes out under the tag of the round before last, which nobody waits for.
    auto lead = [&]() {
        if (G <= kGroup || wg % kGroup != 0 || !summer) return;
        bool over;
        const double t = wave_slots((rt & 1) * kResMaxGroups + wg, min(kGroup, G - wg), over);
        const bool good = !__any(over);
        if ((sl & 3) == 0 && (sl >> 2) < NV)
            put_sum(2 * kResMaxGroups + (rt & 1) * kGroup + wg / kGroup, sl >> 2, t, good ? rt : rt - 2);
    };
    // all workgroups' sums in: the totals for every thread; false when a wait of this round ran out
    auto recv_sums = [&]() -> bool {
        const int own = (rt & 1) * kResMaxGroups, grp = 2 * kResMaxGroups + (rt & 1) * kGroup;
        bool over;
        if (summer) totals(G <= kGroup ? wave_slots(own, G, over) : wave_slots(grp, (G + kGroup - 1) / kGroup, over));
        lds_barrier();
        return s_bad == 0;
    };

    if constexpr (kLdsRows) {
        // each lane's own entries: no other thread reads them
        const int row = base_row();
        if (row < cnt) {
            const int g = n0 + row;
            const Slice sc = slice_of(ly, g);
            for (int u = 0; u < a.lds_entries; ++u) {
                Entries<T, BLK, 1> one;
                load_entries<T, BLK, L, 1, END_LOADED>(A, ly.col, sc, g & 63, l, (E + u) * L, row, one);
#pragma unroll
                for (int t = 0; t < 6; ++t) sk[(6 * u + t) * a.lds_threads + tid] = one.k[0][t];
                sc_col[u * a.lds_threads + tid] = one.c[0];
            }
        }
    }

    int status = RES_OK, total[NS], refinements = 0;
    double relres[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        total[q] = 0;
        relres[q] = 0.0;
    }
    T r[RPT][NC], x[RPT][NC], qv[RPT][NC];

    for (int outer = 0;; ++outer) {
        // --- the true residual r = b - A x in FP64
#pragma unroll
        for (int c = 0; c < NC; ++c) live[c] = 1;
        if (outer > 0) ++xt;                       // x of the exported rows went out under the next tag (below)
        const uint32_t xtag = xt;
        double part[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) part[k] = 0.0;
#pragma unroll
        for (int c0 = 0; c0 < NC; c0 += XC) {      // components per staging of x
            xt = xtag;
            {
            const int row0 = base_row();
#pragma unroll
            for (int s = 0; s < RPT; ++s) {
                const int row = row0 + s * rstep;
                if (c0 == 0)
#pragma unroll
                    for (int c = 0; c < NC; ++c) x[s][c] = T(0);
                if (l != 0 || row >= cnt) continue;
                X v;
#pragma unroll
                for (int c = 0; c < XC; ++c) {
                    v.v[c] = c0 + c < NC ? a.x[static_cast<size_t>(c0 + c) * n + n0 + row] : 0.0;
                    if (!kMixed && c0 + c < NC) x[s][c0 + c] = static_cast<T>(v.v[c]);
                }
                fx[row] = v;
                if constexpr (RPT > 2) __builtin_amdgcn_sched_barrier(0);
            }
            }
            for (int h = tid; h < nhalo; h += kTh) {
                const int g = ly.halo_ids[hbeg + h];
                double v[1][NC];
                if (outer == 0) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) v[0][c] = c >= c0 && c < c0 + XC ? a.x[static_cast<size_t>(c) * n + g] : 0.0;
                } else {
                    const int sl[1] = {ly.slot[g]};
                    fetch(sl, v, s_bad);
                }
                X hv;
#pragma unroll
                for (int c = 0; c < XC; ++c) hv.v[c] = c0 + c < NC ? v[0][c0 + c < NC ? c0 + c : 0] : 0.0;
                fx[ly.nbr + h] = hv;
            }
            if (tid == 0) fx[zero] = X{};
            lds_barrier();
            ++xt;
            {
            const int row0 = base_row();
#pragma unroll
            for (int s = 0; s < RPT; ++s) {
                const int row = row0 + s * rstep;
                if (c0 == 0)
#pragma unroll
                    for (int c = 0; c < NC; ++c) r[s][c] = T(0);
                if (row >= cnt) continue;
                const int g = n0 + row;
                double acc[XC], bv[XC];
#pragma unroll
                for (int c = 0; c < XC; ++c) bv[c] = c0 + c < NC ? a.b[static_cast<size_t>(c0 + c) * n + g] : 0.0;
#pragma unroll
                for (int c = 0; c < XC; ++c) acc[c] = 0.0;
                double base[XC];
                const X own = fx[row];
                const double dg64 = zero_sum ? 0.0 : a.d64[g];
#pragma unroll
                for (int c = 0; c < XC; ++c) {
                    base[c] = zero_sum ? own.v[c] : 0.0;
                    if (l == 0) acc[c] = dg64 * own.v[c];
                }
                add_rest<double, XC, BLK, L>(a.a64, ly.col, slice_of(ly, g), g & 63, l, 0, zero_sum ? row : zero, fx, base, acc);
#pragma unroll
                for (int c = 0; c < XC; ++c) acc[c] = lanes_sum<L>(acc[c]);
#pragma unroll
                for (int c = 0; c < XC; ++c) {
                    if (c0 + c >= NC) continue;
                    const double rv = bv[c] - acc[c];
                    if (l == 0) part[NS + set(c0 + c)] += rv * rv;
                    r[s][c0 + c] = kMixed ? static_cast<T>(a.scale * rv) : static_cast<T>(rv);
                }
                if (c0 + XC >= NC && xport[s] >= 0) publish(xport[s], r[s]);
                if constexpr (RPT > 2) __builtin_amdgcn_sched_barrier(0);   // one row's loads at a time: registers
            }
            }
            if (c0 + XC < NC) lds_barrier();       // the next components take the staging
        }
        ++rt;
        // a workgroup that gave up keeps its sums back here and in the iterations: no round is completed, and so no x
        // stored, that values which never came had a part in
        if (outer > 0 && s_bad != 0) {
            status = RES_TIMEOUT;
            break;
        }
        send_sums(part);
        T hq[kHB][NC];
        lead();
        fetch(hid, hq, s_bad);
        if (!recv_sums()) {
            status = RES_TIMEOUT;
            break;
        }
        // halo r (in T), each by the thread that updates it
#pragma unroll
        for (int u = 0; u < kHB; ++u)
            if (hid[u] >= 0)
#pragma unroll
                for (int c = 0; c < NC; ++c) hr[(tid + u * kTh) * NC + c] = hq[u][c];
        for (int h = tid + kHB * kTh; h < nhalo; h += kTh) {
            T v[1][NC];
            const int sl[1] = {slot_of(h)};
            fetch(sl, v, s_late);
#pragma unroll
            for (int c = 0; c < NC; ++c) hr[h * NC + c] = v[0][c];
        }
        // --- which scalar sets go on, and the inner thresholds
        double rr0[NS], thr[NS];
        bool conv[NS], all = true, broke = false;
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            rr0[q] = uniform(s_tot[NS + q]);
            conv[q] = bb[q] == 0.0 || rr0[q] <= a.tol2 * bb[q];
            if (kMixed) {
                broke |= !isfinite(rr0[q]);
                const double eta = fmax(0.5 * a.tol * sqrt(bb[q] / rr0[q]), kResInnerFloor);
                thr[q] = eta * eta * rr0[q] * a.scale * a.scale;
            } else {
                thr[q] = a.tol2 * bb[q];
            }
            all &= conv[q];
            relres[q] = bb[q] > 0.0 ? sqrt(fmax(rr0[q], 0.0) / bb[q]) : 0.0;
        }
        if (outer == 0) {
            {
            const int row0 = base_row();
#pragma unroll
            for (int s = 0; s < RPT; ++s) {
                const int row = row0 + s * rstep;
                if (l != 0 || row >= cnt) continue;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (bb[set(c)] == 0.0) a.x[static_cast<size_t>(c) * n + n0 + row] = 0.0;
            }
            }
        }
        if (broke) {
            status = RES_NONFINITE;
            break;
        }
        if (all) break;
        int used = 0;
#pragma unroll
        for (int q = 0; q < NS; ++q) used = max(used, total[q]);
        if (kMixed && used >= a.maxit) {
            status = RES_NOCONV;
            break;
        }
        const int budget = kMixed ? a.maxit - used : a.maxit;
#pragma unroll
        for (int c = 0; c < NC; ++c) live[c] = !conv[set(c)];
#pragma unroll
        for (int s = 0; s < RPT; ++s)
#pragma unroll
            for (int c = 0; c < NC; ++c) qv[s][c] = T(0);
        lds_barrier();                            // x staging read by every row: p takes its place

        // --- single-reduction CG
        auto fill = [&](int row, Entries<T, BLK, E> &to) {
            const int g = n0 + (row < cnt ? row : 0);
            load_entries<T, BLK, L, E, (RPT > 1 ? END_BRANCH : END_LOADED)>(A, ly.col, slice_of(ly, g), g & 63, l, 0, zero_sum ? row : zero, to);
        };
        Entries<T, BLK, E> en[kBuf];
        fill(base_row(), en[0]);
        const T dg = zero_sum ? T(0) : D[n0 + min(base_row(), cnt - 1)];
        T al[NC], be[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) al[c] = be[c] = T(0);
        int iters[NS], ended = 0;
#pragma unroll
        for (int q = 0; q < NS; ++q) iters[q] = 0;
        for (int k = 0;; ++k) {
            if (k > 0) {
                // scalars of iteration k - 1: the first wave formed them with the totals
                bool any = false;
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    const double rrp = uniform(s_tot[NS + q]);
                    const int stop = !isfinite(rrp) ? 2 : (rrp <= thr[q] ? 1 : 0);
                    if (live[BLK ? 0 : q] && stop) {
                        iters[q] = k - 1;
                        if (stop == 2) status = RES_NONFINITE;
                        if (!kMixed) relres[q] = sqrt(fmax(rrp, 0.0) / bb[q]);
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            if (set(c) == q) live[c] = 0;
                    }
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    any |= live[c] != 0;
                    al[c] = live[c] ? static_cast<T>(uniform(s_al[set(c)])) : T(0);
                    be[c] = live[c] ? static_cast<T>(uniform(s_be[set(c)])) : T(0);
                }
                if (!any) break;
                ended = k == budget;
            }
            // the first streamed entries are on their way while the vectors are updated
            Entries<T, BLK, (kAhead > 0 ? kAhead : 1)> ahead;
            if constexpr (kAhead > 0) {
                const int row = base_row(), g = n0 + (row < cnt ? row : 0);
                load_entries<T, BLK, L, kAhead, END_SELECT>(A, ly.col, slice_of(ly, g), g & 63, l, (E + a.lds_entries) * L, row, ahead);
                __builtin_amdgcn_sched_barrier(0);
            }
            // r_k, x_k and p_k = D^-1 r_k + beta p_{k-1} of the rows (x takes alpha p_{k-1})
            {
            const int row0 = base_row();
#pragma unroll
            for (int s = 0; s < RPT; ++s) {
                const int row = row0 + s * rstep;
                if (row >= cnt) continue;
                V p;
                if (k > 0) p = f[row];
                V pn;
#pragma unroll
                for (int c = 0; c < V::kPad; ++c) pn.v[c] = T(0);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if (k > 0) {
                        x[s][c] += al[c] * p.v[c];
                        r[s][c] -= al[c] * qv[s][c];
                    }
                    const T z = r[s][c] * di[s];
                    pn.v[c] = !live[c] ? T(0) : (k > 0 ? z + be[c] * p.v[c] : z);
                }
                if (L > 1) __builtin_amdgcn_wave_barrier();
                if (l == 0 && !ended) f[row] = pn;
                if constexpr (RPT > 2) __builtin_amdgcn_sched_barrier(0);
            }
            }
            if (ended) {
#pragma unroll
                for (int q = 0; q < NS; ++q)
                    if (live[BLK ? 0 : q]) iters[q] = budget;
                if (!kMixed) status = status == RES_NONFINITE ? status : RES_NOCONV;
                break;
            }
            // the halo's, from the q that arrived with the sums
            auto halo = [&](int h, const T (&q)[NC]) {
                const T d = hd[h];
                V p;
                if (k > 0) p = f[ly.nbr + h];
                V pn;
#pragma unroll
                for (int c = 0; c < V::kPad; ++c) pn.v[c] = T(0);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    T rv = hr[h * NC + c];
                    if (k > 0) {
                        rv -= al[c] * q[c];
                        hr[h * NC + c] = rv;
                    }
                    const T z = rv * d;
                    pn.v[c] = !live[c] ? T(0) : (k > 0 ? z + be[c] * p.v[c] : z);
                }
                f[ly.nbr + h] = pn;
            };
#pragma unroll
            for (int u = 0; u < kHB; ++u)
                if (hid[u] >= 0) halo(tid + u * kTh, hq[u]);
            for (int h = tid + kHB * kTh; h < nhalo; h += kTh) {
                T q[1][NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) q[0][c] = T(0);
                if (k > 0) {
                    const int sl[1] = {slot_of(h)};
                    fetch(sl, q, s_late);
                }
                halo(h, q[0]);
            }
            if (k == 0 && tid == 0) f[zero] = V{};
            lds_barrier();
            if (nhalo > kHB * kTh && s_late != 0) {
                status = RES_TIMEOUT;
                break;
            }
            // q_k = A p_k and its sums
            ++xt;
            ++rt;
#pragma unroll
            for (int j = 0; j < NV; ++j) part[j] = 0.0;
            {
            const int row0 = base_row();
#pragma unroll
            for (int s = 0; s < RPT; ++s) {
                const int row = row0 + s * rstep;
                // the next row's entries are on their way while this row's are used
                Entries<T, BLK, E> &cur = en[s & (kBuf - 1)];
                if constexpr (kBuf > 1) {
                    if (s + 1 < RPT) fill(row + rstep, en[(s + 1) & (kBuf - 1)]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (row >= cnt) continue;
                const int g = n0 + row;
                T acc[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] = T(0);
                const V p = f[row];
                const T d = RPT > 1 ? (zero_sum ? T(0) : D[g]) : dg;
                const int none = zero_sum ? row : zero;
                T base[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    base[c] = zero_sum ? p.v[c] : T(0);
                    if (l == 0) acc[c] = d * p.v[c];
                }
                const Slice sc = slice_of(ly, g);
                add_entries<T, NC, BLK, L, E, (RPT > 1 ? END_BRANCH : END_LOADED)>(cur, sc, l, 0, none, f, base, acc);
                if constexpr (kLdsRows) {
#pragma unroll 2
                    for (int u = 0; u < a.lds_entries; ++u) {
                        Entries<T, BLK, 1> one;
#pragma unroll
                        for (int t = 0; t < 6; ++t) one.k[0][t] = sk[(6 * u + t) * a.lds_threads + tid];
                        one.c[0] = sc_col[u * a.lds_threads + tid];
                        add_entries<T, NC, BLK, L, 1, END_LOADED>(one, sc, l, 0, none, f, base, acc);
                    }
                    if constexpr (kAhead > 0)
                        add_entries<T, NC, BLK, L, kAhead, END_SELECT>(ahead, sc, l, (E + a.lds_entries) * L, none, f, base, acc);
                }
                const int held = (E + (kLdsRows ? a.lds_entries + kAhead : 0)) * L;
                if (sc.w > held) add_rest<T, NC, BLK, L>(A, ly.col, sc, g & 63, l, held, none, f, base, acc);
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] = lanes_sum<L>(acc[c]);
                if (xport[s] >= 0) publish(xport[s], acc);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    qv[s][c] = acc[c];
                    if (l != 0 || !live[c]) continue;
                    const double rv = r[s][c], qq = acc[c], dd = di[s];
                    part[set(c)] += static_cast<double>(p.v[c]) * qq;
                    part[NS + set(c)] += rv * rv;
                    part[2 * NS + set(c)] += rv * (dd * rv);
                    part[3 * NS + set(c)] += rv * (dd * qq);
                    part[4 * NS + set(c)] += qq * (dd * qq);
                }
                if constexpr (RPT > 2) __builtin_amdgcn_sched_barrier(0);
            }
            }
            if constexpr (kBuf > 1) fill(base_row(), en[0]);
            send_sums(part);
            lead();
            fetch(hid, hq, s_bad);
            if (!recv_sums()) {
                status = RES_TIMEOUT;
                break;
            }
        }
        if (status == RES_TIMEOUT) break;
        int most = 0;
#pragma unroll
        for (int q = 0; q < NS; ++q)
            if (!conv[q]) {
                total[q] += iters[q];
                most = max(most, iters[q]);
            }
        if (kMixed && status == RES_NONFINITE) break;
        // an inner solve without an iteration (the scaled residual is below FP32's range and its norm reads zero) leaves
        // x as it was, and so would every one after it
        if (kMixed && most == 0) {
            status = RES_NOCONV;
            break;
        }
        if (kMixed) ++refinements;
        // x <- x + d (mixed) or the accumulated x; the next residual needs it from the neighbours
        ++xt;
#pragma unroll
        for (int c = 0; c < NC; ++c) live[c] = 1;
        {
        const int row0 = base_row();
#pragma unroll
        for (int s = 0; s < RPT; ++s) {
            const int row = row0 + s * rstep;
            if (l != 0 || row >= cnt) continue;
            double xn[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const size_t o = static_cast<size_t>(c) * n + n0 + row;
                xn[c] = kMixed || conv[set(c)] ? a.x[o] : static_cast<double>(x[s][c]);
                if (conv[set(c)]) continue;
                if (kMixed) xn[c] += static_cast<double>(x[s][c]);
                a.x[o] = xn[c];
            }
            if (kMixed && xport[s] >= 0) publish(xport[s], xn);
            if constexpr (RPT > 2) __builtin_amdgcn_sched_barrier(0);
        }
        }
        if (!kMixed) break;
        --xt;                                       // the loop's head steps to this tag
        lds_barrier();
    }
    if (status == RES_TIMEOUT && tid == 0) a.result->gave_up = 1;
    if (wg == 0 && tid == 0) {
        a.epoch[0] = xt + 2;
        a.epoch[1] = rt + 1;
        ResResult *o = a.result;
        o->status = status;
        o->refinements = refinements;
        o->stale = xt > 0x70000000u || rt > 0x70000000u;
#pragma unroll
        for (int q = 0; q < kMaxComp; ++q) {
            o->iters[q] = q < NS ? total[q < NS ? q : 0] : 0;
            o->relres[q] = q < NS ? relres[q < NS ? q : 0] : 0.0;
        }
    }
}

namespace {

// Lanes per row and rows per thread of a launch over nbr rows: as many lanes
// (up to 8) as the rows leave threads for, then as few rows as hold them.
void shape(int nbr, int &lanes, int &rpt) {
    lanes = 1;
    while (lanes < 8 && nbr * lanes * 2 <= kTh) lanes <<= 1;
    for (rpt = 1; rpt <= 8 && nbr > rpt * (kTh / lanes);) rpt <<= 1;
}

template <class T, int NC, bool BLK, int L, int RPT>
const void *entry() {
    return reinterpret_cast<const void *>(&k_resident<T, NC, BLK, L, RPT>);
}

template <class T, int NC, bool BLK>
const void *entry_for(int lanes, int rpt) {
    if (rpt == 1)
        return lanes == 1 ? entry<T, NC, BLK, 1, 1>() : lanes == 2 ? entry<T, NC, BLK, 2, 1>()
             : lanes == 4 ? entry<T, NC, BLK, 4, 1>() : entry<T, NC, BLK, 8, 1>();
    if (rpt == 2) return entry<T, NC, BLK, 1, 2>();
    if constexpr (!BLK) {              // (blocks of coefficients stop at two rows per thread: kResElasticRows)
        if (rpt == 4) return entry<T, NC, BLK, 1, 4>();
        if constexpr (sizeof(T) == 4)  // FP64 stops at four: its registers
            if (rpt == 8) return entry<T, NC, BLK, 1, 8>();
    }
    return nullptr;
}

template <class T>
const void *entry_of(int nc, bool blk, int nbr) {
    int lanes, rpt;
    shape(nbr, lanes, rpt);
    if (blk) return entry_for<T, 3, true>(lanes, rpt);
    return nc == 1 ? entry_for<T, 1, false>(lanes, rpt) : nc == 2 ? entry_for<T, 2, false>(lanes, rpt)
                                                                  : entry_for<T, 3, false>(lanes, rpt);
}

// dynamic LDS of a launch
template <class T>
size_t lds_bytes(const ResArgs &a, int nc) {
    return a.stage_bytes + sizeof(T) * ((nc + 1) * static_cast<size_t>(a.ly.nhalo_max) + 2) +
           (6 * sizeof(T) + sizeof(uint16_t)) * static_cast<size_t>(a.lds_entries) * a.lds_threads;
}

}  // namespace

template <class T>
bool resident_fits(ResArgs &a, int nc, bool blk, size_t lds_max, int cus) {
    const ResLayout &ly = a.ly;
    if (ly.nbr <= 0 || ly.G <= 0 || ly.G > kResMaxGroups || ly.G > cus) return false;
    const void *k = entry_of<T>(nc, blk, ly.nbr);
    if (!k) return false;
    const size_t pad = nc == 3 ? 4 : nc;
    int lanes, rpt;
    shape(ly.nbr, lanes, rpt);
    const size_t per = std::max(sizeof(T) * pad, sizeof(double) * resident_xc(sizeof(T) == 4, nc, blk, rpt));
    a.stage_bytes = static_cast<uint32_t>((per * (static_cast<size_t>(ly.nbr) + ly.nhalo_max + 1) + 15) / 16 * 16);
    a.lds_entries = 0;
    a.lds_threads = std::min(kTh, (ly.nbr * lanes + 63) / 64 * 64);
    // the kernel's static LDS besides
    constexpr size_t kStatic = 4096;
    if (lds_bytes<T>(a, nc) + kStatic > lds_max) return false;
    if (blk && sizeof(T) == 8 && rpt == 1 && lanes <= 2) {
        // At 97k nodes four of 14 FP64 blocks per row are in registers; streaming the other ten (48 MB an iteration,
        // 6 MB for each XCD's 4 MB of L2) took 14.6 us of a 21 us iteration.  What LDS has left holds five more, and
        // the last five (24 MB) stay in L2.
        const int e = resident_entries(false, true, lanes, rpt);
        const size_t each = (6 * sizeof(T) + sizeof(uint16_t)) * static_cast<size_t>(a.lds_threads);
        const int most = std::max(0, (ly.wmax + lanes - 1) / lanes - e);
        a.lds_entries = std::min<int>(most, static_cast<int>((lds_max - kStatic - lds_bytes<T>(a, nc)) / each));
    }
    int per_cu = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kTh, lds_bytes<T>(a, nc)) == hipSuccess &&
           per_cu >= 1;
}

template <class T>
int launch_resident(const ResArgs &a, int nc, bool blk, hipStream_t s) {
    const void *k = entry_of<T>(nc, blk, a.ly.nbr);
    if (!k) return static_cast<int>(hipErrorInvalidValue);
    ResArgs v = a;
    void *args[] = {&v};
    return static_cast<int>(
        hipLaunchCooperativeKernel(k, dim3(a.ly.G), dim3(kTh), args, static_cast<unsigned>(lds_bytes<T>(a, nc)), s));
}

}  // namespace gspm
