// The host layouts of the one-launch solves (resident_host.cpp) when memory or
// threads run out: allocation k fails for every k in turn, on whichever thread
// it falls, and thread creation fails from the first or the second thread on.
// Each time the functions must throw std::bad_alloc to their caller or return
// what they return otherwise; nothing may end the process.
// Usage: resident_faults; exit 0 if so.
#include <dlfcn.h>
#include <pthread.h>

#include <atomic>
#include <cerrno>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "resident.h"
using namespace gspm;

namespace {
std::atomic<long> allocs{0}, fail_at{-1};
std::atomic<int> threads{0}, most_threads{1 << 20};
}  // namespace

void *operator new(size_t n) {
    if (allocs++ == fail_at) throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" int pthread_create(pthread_t *t, const pthread_attr_t *a, void *(*f)(void *), void *x) {
    using Fn = int (*)(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *);
    static const Fn real = reinterpret_cast<Fn>(dlsym(RTLD_NEXT, "pthread_create"));
    return threads++ < most_threads ? real(t, a, f, x) : EAGAIN;
}

namespace {

struct Result {
    bool ok = false, threw = false;
    std::vector<uint16_t> col;
    std::vector<int32_t> halo, slot;
};

void run(int n, const std::vector<int32_t> &tets, Result &r) {
    try {
        std::vector<int32_t> inc_ptr, inc;
        GsRowsHost rows;
        ResLayoutHost ly;
        r.ok = node_elements(n, tets, inc_ptr, inc) && operator_pattern(n, tets, inc_ptr, inc, 64, rows) &&
               resident_layout(rows, n, 64, ly);
        r.col.swap(ly.col);
        r.halo.swap(ly.halo_ids);
        r.slot.swap(ly.slot);
    } catch (const std::bad_alloc &) {
        r.threw = true;
    }
}

}  // namespace

int main() {
    // a periodic 17^3 lattice, six tetrahedra a cell: 77 workgroups and slices, several threads
    const int s = 17, n = s * s * s;
    const int order[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    auto at = [&](const int (&c)[3]) { return ((c[2] % s) * s + c[1] % s) * s + c[0] % s; };
    std::vector<int32_t> tets;
    for (int i = 0; i < n; ++i)
        for (auto &o : order) {
            int c[3] = {i % s, i / s % s, i / (s * s)};
            tets.push_back(at(c));
            for (int k = 0; k < 3; ++k) {
                ++c[o[k]];
                tets.push_back(at(c));
            }
        }
    Result want;
    allocs = 0;
    run(n, tets, want);
    const long total = allocs;
    if (!want.ok || threads == 0) {
        printf("no layout or no threads\n");
        return 1;
    }
    long thrown = 0, tried = 0, wrong = 0;
    auto count = [&](const Result &r, bool may_throw) {
        ++tried;
        thrown += r.threw;
        if (r.threw ? !may_throw : !(r.ok && r.col == want.col && r.halo == want.halo && r.slot == want.slot)) ++wrong;
    };
    for (long k = 0; k < total; k += k < 200 ? 1 : 97) {
        Result r;
        allocs = 0;
        fail_at = k;
        run(n, tets, r);
        fail_at = -1;
        count(r, true);
    }
    for (int most = 0; most < 2; ++most) {
        Result r;
        threads = 0;
        most_threads = most;
        run(n, tets, r);
        count(r, false);
    }
    printf("%ld allocations, %ld runs, %ld threw, %ld wrong\n", total, tried, thrown, wrong);
    return wrong || thrown == 0 ? 1 : 0;
}
