// The HIP runtime as the library's host code uses it, on host memory, so that
// the host code runs under the sanitizers without a device: device and pinned
// memory come from malloc (every allocation by itself, so that an access past
// its end is seen), copies are memcpy, streams run at once.  Kernels do nothing
// but for the caller arrays' checks and permutation, the copies of results to
// the host and fills, which are done here in plain loops.
#include <hip/hip_runtime.h>
#include <rocfft/rocfft.h>

#include <cmath>
#include <cstdlib>
#include <cstring>

#include "context.h"

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 163840 : 256;
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
    *p = std::malloc(n);
    if (*p) std::memset(*p, 0, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 0.0f; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }

rocfft_status rocfft_setup() { return rocfft_status_success; }
rocfft_status rocfft_plan_create(rocfft_plan *p, rocfft_result_placement, rocfft_transform_type, rocfft_precision, size_t,
                                 const size_t *, size_t, const rocfft_plan_description) {
    *p = reinterpret_cast<rocfft_plan>(std::malloc(1));
    return rocfft_status_success;
}
rocfft_status rocfft_plan_destroy(rocfft_plan p) { std::free(p); return rocfft_status_success; }
rocfft_status rocfft_plan_get_work_buffer_size(const rocfft_plan, size_t *n) { *n = 1024; return rocfft_status_success; }
rocfft_status rocfft_execution_info_create(rocfft_execution_info *p) {
    *p = reinterpret_cast<rocfft_execution_info>(std::malloc(1));
    return rocfft_status_success;
}
rocfft_status rocfft_execution_info_destroy(rocfft_execution_info p) { std::free(p); return rocfft_status_success; }
rocfft_status rocfft_execution_info_set_stream(rocfft_execution_info, void *) { return rocfft_status_success; }
rocfft_status rocfft_execution_info_set_work_buffer(rocfft_execution_info, void *, const size_t) { return rocfft_status_success; }
rocfft_status rocfft_execute(const rocfft_plan, void *[], void *[], rocfft_execution_info) { return rocfft_status_success; }
}

namespace gspm {

double g_scratch[16];
int noalloc_scratch_address(int, double **p) { *p = g_scratch; return 0; }
size_t rows_lds_bytes(int, int, bool) { return 1 << 16; }
size_t elem_lds_bytes(int, int) { return 1 << 16; }

void launch_fill(double *p, int64_t n, double v, hipStream_t) { for (int64_t i = 0; i < n; ++i) p[i] = v; }
void launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t) { for (int64_t i = 0; i < n; ++i) p[i] = v; }
void launch_i32_to_host(const int32_t *s, int n, int32_t *d, hipStream_t) { std::memcpy(d, s, sizeof(int32_t) * n); }
void launch_totals_to_host(const ShardSources &, int n, double *d, hipStream_t) { for (int i = 0; i < n; ++i) d[i] = 0.0; }

void launch_user_put(const UserMap &u, int nc, int kind, int seq, double *dst, hipStream_t) {
    const uint64_t key0 = static_cast<uint64_t>(seq) << kUserSeqShift;
    for (int64_t i = 0; i < u.n0; ++i)
        for (int a = 0; a < nc; ++a) {
            const double x = u.v[i * nc + a], f = u.v[static_cast<int64_t>(u.rep[u.user2int[i]]) * nc + a];
            u.dev[i * nc + a] = x;
            const unsigned long long key = key0 | static_cast<uint64_t>((i * 3 + a) * 2);
            if (!std::isfinite(x)) *u.err = std::min(*u.err, key);
            else if (std::fabs(f - x) > 1e-12 * std::max(std::fabs(f), std::fabs(x)))
                *u.err = std::min(*u.err, key | static_cast<unsigned long long>(kUserMismatch));
        }
    *u.report = *u.err;
    if (*u.err != kUserFine) return;
    for (int k = 0; k < u.n; ++k)
        for (int a = 0; a < nc; ++a) dst[static_cast<size_t>(a) * u.n + k] = u.dev[static_cast<int64_t>(u.rep[k]) * nc + a];
    (void)kind;
}
void launch_user_get(const UserMap &u, int nc, const double *src, hipStream_t) {
    for (int64_t i = 0; i < u.n0; ++i)
        for (int a = 0; a < nc; ++a) u.v[i * nc + a] = src[static_cast<size_t>(a) * u.n + u.user2int[i]];
}

// the rows' coefficients: every entry of the layout is written, its column and the elements' lists read
void launch_operator_rows(OperatorBuild a, hipStream_t) {
    double sum = 0.0;
    for (int sl = 0; 64 * sl < a.ly.n; ++sl) {
        const int g = 64 * sl / a.ly.nbr;
        for (int64_t e = a.ly.off[sl]; e < a.ly.off[sl + 1]; ++e) {
            const int c = a.ly.col[e];
            const int j = c < a.ly.nbr ? g * a.ly.nbr + c : a.ly.halo_ids[a.ly.halo_ptr[g] + c - a.ly.nbr];
            if (j < a.ly.n) sum += a.x[j] + a.ly.slot[j];
            for (int t = 0; t < 6; ++t) {
                const int64_t o = (e - e % 64) * 6 + 64 * t + e % 64;
                if (a.k64) a.k64[o] = 1.0;
                if (a.k32) a.k32[o] = 1.0f;
            }
            if (a.m64) a.m64[e] = 1.0;
            if (a.m32) a.m32[e] = 1.0f;
        }
    }
    for (int i = 0; i < a.ly.n; ++i)
        for (int t = a.inc_ptr[i]; t < a.inc_ptr[i + 1]; ++t) sum += a.tets[4 * static_cast<size_t>(a.inc[t]) + 3];
    if (a.open) *a.open = sum < -1e300;
}

// both kinds of transforms' tables; convergence where a preconditioned batch tests it
int green_fft_pairs(const GreenView &gv, const int *, const int *, bool, size_t) { return gv.gz % 2 ? 0 : 8; }
void launch_cg_check(int, bool, const CGScalars &cg, int k, double, hipStream_t) {
    cg.done[0] = 1;
    cg.iters[0] = k;
}

// a one-launch solve that converges in one iteration; x moves so that the caller sees it
template <class T>
bool resident_fits(ResArgs &a, int, bool, size_t, int) { return a.ly.nbr > 0; }
template <class T>
int launch_resident(const ResArgs &a, int nc, bool, hipStream_t) {
    for (int64_t i = 0; i < static_cast<int64_t>(nc) * a.ly.n; ++i) a.x[i] += a.b[i];
    const char *xq = static_cast<const char *>(a.xq) + resident_xq_bytes(a.ly.nexp) - 1,
               *sl = static_cast<const char *>(a.slots) + resident_slot_bytes() - 1;
    a.epoch[1] += 1 + (*xq & 0) + (*sl & 0);
    *a.result = ResResult{};
    for (int q = 0; q < kMaxComp; ++q) a.result->iters[q] = 1;
    return 0;
}
template bool resident_fits<double>(ResArgs &, int, bool, size_t, int);
template bool resident_fits<float>(ResArgs &, int, bool, size_t, int);
template int launch_resident<double>(const ResArgs &, int, bool, hipStream_t);
template int launch_resident<float>(const ResArgs &, int, bool, hipStream_t);

}  // namespace gspm
