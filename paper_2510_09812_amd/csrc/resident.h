// CG solves that run to their end in one cooperative launch (resident_kernel.h):
// the row layout they work on, their exchange buffers and their launcher.
#pragma once

#include <string>
#include <vector>

#include "common.h"

namespace gspm {

constexpr int kResThreads = 512;
constexpr int kResMaxGroups = 256;     // workgroups of a launch, at most one per CU
constexpr int kGroup = 16;             // workgroups that read each other's sums, and that a leader sums beyond
constexpr int kSlotSums = 16;          // sums per slot, 16 bytes each
constexpr int kResChunks = 3;          // 16-byte chunks per exchanged node: three doubles
constexpr double kResInnerFloor = 1e-6;
constexpr int64_t kResWaitTicks = 500000000;   // 5 s
constexpr int64_t kResWaitShort = 1000;        // waits below look at the clock at every poll, others at every 256th

enum ResStatus { RES_OK = 0, RES_NOCONV = 1, RES_NONFINITE = 2, RES_TIMEOUT = 3 };

// Rows of a launch: workgroup g owns rows [g nbr, (g + 1) nbr).  Slices,
// widths and the entries' order are those of GsRowsHost; col holds the columns
// as local indices of the workgroup (owned: j - g nbr; halo: nbr + position in
// its halo list).
struct ResLayout {
    const int32_t *off;
    const uint16_t *col;
    const int32_t *halo_ptr, *halo_ids;
    const int32_t *slot;               // n: the node's slot in the exchange buffer, -1 if no other workgroup reads it
    int32_t n, nbr, G, nhalo_max, nexp, wmax;   // wmax: entries of the longest row
};

struct ResLayoutHost {
    int32_t nbr = 0, G = 0, nhalo_max = 0, nexp = 0, wmax = 0;
    std::vector<uint16_t> col;
    std::vector<int32_t> halo_ptr, halo_ids;
    std::vector<int32_t> slot;
};

// What the host reads back (pinned host memory, written by the launch's end):
// workgroup 0's outcome, which every workgroup shares unless a wait ran out in
// some of them, and whether one did in any (cleared by the host before).
struct ResResult {
    int32_t status, refinements, stale, gave_up;
    int32_t iters[kMaxComp];
    double relres[kMaxComp];
};

struct ResArgs {
    ResLayout ly;
    const void *a, *d;                 // coefficients and diagonal (GS) in the iterations' type
    const double *a64, *d64;           // and in FP64 (the residuals)
    double *x;                         // [nc][n] start in, solution out
    const double *b;
    const double *bb;                  // |b|^2 per scalar set, sharded
    double scale;                      // FP32 operator = scale * FP64 operator
    double tol, tol2;
    int32_t maxit, jacobi;
    int32_t zero_sum;                  // the rows sum to zero (K^mech, K^ms): no diagonals given
    int64_t wait_ticks;                // of the 100 MHz clock: the longest wait for another workgroup
    int32_t poll_mask;                 // polls between two looks at it, less one
    void *xq, *slots;
    uint32_t *epoch;                   // [2]: last tags of the exchange and of the sums
    ResResult *result;
    uint32_t stage_bytes;
    int32_t lds_entries, lds_threads;  // entries of each lane kept in LDS, and the lanes that have any
};

// The operators over all elements, K^mech (symmetric 3x3 blocks) and K^ms, in
// the row form of a layout (operator_rows.hip); null outputs are left out.
struct OperatorBuild {
    ResLayout ly;
    const double *x, *y, *z;
    double L[3], iL[3];
    const int32_t *inc_ptr, *inc, *tets;   // elements of each node, ascending; their nodes
    int32_t p0, parts;
    double C6[36];                     // stiffness in the sample frame, Voigt
    double scale_k, scale_m;           // of the FP32 copies
    double *k64, *m64;
    float *k32, *m32;
    int32_t *open;                     // set to 1 when a free surface makes blocks of K^mech asymmetric
};
void launch_operator_rows(OperatorBuild a, hipStream_t s);

// The host functions below throw std::bad_alloc when memory is short; callers
// at the C interface go on without the one-launch form then.
// The elements of each node, ascending; false when there are too many to index.
bool node_elements(int32_t n, const std::vector<int32_t> &tets, std::vector<int32_t> &inc_ptr, std::vector<int32_t> &inc);
// The pattern of those operators: each node's neighbours through its elements
// as slices of columns in GsRowsHost's form (blocks of nb rows; no
// coefficients).  False when a node has 256 or more neighbours or the mesh more
// entries than the layout addresses.
bool operator_pattern(int32_t n, const std::vector<int32_t> &tets, const std::vector<int32_t> &inc_ptr,
                      const std::vector<int32_t> &inc, int32_t nb, GsRowsHost &out);

// The columns of `rows` (any row blocks) for workgroups of nbr rows; false
// when a workgroup would stage more than 65535 nodes.
bool resident_layout(const GsRowsHost &rows, int32_t n, int32_t nbr, ResLayoutHost &out);
// Rows per workgroup (a multiple of 64) for n nodes on a device of `cus` compute units with iterations in FP32 or FP64
// (0: the mesh is too large).
int32_t resident_rows(int32_t n, int32_t cus, bool f32);
// Components of x a residual stages at once.
__host__ __device__ constexpr int resident_xc(bool f32, int nc, bool blk, int rpt) {
    return f32 && nc == 3 && !blk && rpt == 8 ? 2 : nc;
}
// Entries of a row each lane keeps in registers: all of a Kuhn mesh's 14 over
// the whole solve with one row per thread, but four of an FP64 block row (48
// bytes each); with more rows per thread the size of a buffer that is refilled.
__host__ __device__ constexpr int resident_entries(bool f32, bool blk, int lanes, int rpt) {
    const int all = lanes == 1 ? 14 : lanes == 2 ? 7 : 16 / lanes;
    return !blk ? all : f32 ? (rpt > 1 ? 4 : all) : (lanes >= 4 ? all : 4);
}
// Sizes of the exchange buffers in bytes.
__host__ __device__ inline size_t resident_xq_bytes(int32_t nexp) {
    return 2 * static_cast<size_t>(kResChunks) * 16 * static_cast<size_t>(nexp > 0 ? nexp : 1);
}
__host__ __device__ inline size_t resident_slot_bytes() {
    return 2 * static_cast<size_t>(kResMaxGroups + kGroup) * kSlotSums * 16;
}

// Whether the launch (type T, nc components, block form) fits the device; fills stage_bytes.
template <class T>
bool resident_fits(ResArgs &a, int nc, bool blk, size_t lds_max, int cus);
template <class T>
int launch_resident(const ResArgs &a, int nc, bool blk, hipStream_t s);

}  // namespace gspm
