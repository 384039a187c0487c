// Host side of the resident CG solves: the rows' columns for workgroups of a
// given size, and that size.
#include <algorithm>
#include <atomic>
#include <climits>
#include <new>
#include <thread>

#include "resident.h"

namespace gspm {

namespace {

// body(k) for every k in [0, n) on the host's threads, as many of them as there
// are to have.  What a body throws (memory) ends the others and is thrown here as
// std::bad_alloc once all have stopped.
template <class Body>
void for_each_part(int32_t n, Body body) {
    std::atomic<int32_t> next{0};
    std::atomic<bool> failed{false};
    auto worker = [&]() noexcept {
        try {
            for (int32_t k; !failed && (k = next.fetch_add(1)) < n;) body(k);
        } catch (...) {
            failed = true;
        }
    };
    // (a thread costs about as much as 16 parts of the smallest meshes)
    const unsigned hw = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    std::vector<std::thread> pool;
    try {
        for (unsigned t = 1; t < hw && 16 * static_cast<int32_t>(t) < n; ++t) pool.emplace_back(worker);
    } catch (...) {
        // no more threads: those there are do the work
    }
    worker();
    for (auto &t : pool) t.join();
    if (failed) throw std::bad_alloc();
}

}  // namespace

// One workgroup per CU at most, as many as have 64 rows: lanes per row count
// for more than the second hop of the sums (FP64 elastic iterations: 9261 nodes
// 4.9 us with 64 rows, eight lanes each, and 7.4 with 192, two each).  kGroup of
// them need one hop, and small meshes stop there as long as that leaves a
// workgroup 128 rows, four lanes each (1728 nodes: 4.2 us against 4.5).
int32_t resident_rows(int32_t n, int32_t cus, bool f32) {
    const int32_t most = std::min(cus, kResMaxGroups);
    if (most <= 0) return 0;
    const int32_t need = (n + most - 1) / most;
    int32_t nbr = std::max(64, (need + 63) / 64 * 64);
    if (n <= kGroup * 128) nbr = std::max(nbr, (((n + kGroup - 1) / kGroup) + 63) / 64 * 64);
    return nbr <= (f32 ? 4096 : 2048) ? nbr : 0;      // eight rows a thread; FP64 has registers for four
}

bool node_elements(int32_t n, const std::vector<int32_t> &tets, std::vector<int32_t> &inc_ptr, std::vector<int32_t> &inc) {
    if (tets.size() > static_cast<size_t>(INT32_MAX)) return false;
    const int32_t ne = static_cast<int32_t>(tets.size() / 4);
    inc_ptr.assign(static_cast<size_t>(n) + 1, 0);
    for (int32_t v : tets) ++inc_ptr[static_cast<size_t>(v) + 1];
    for (int32_t i = 0; i < n; ++i) inc_ptr[i + 1] += inc_ptr[i];
    inc.resize(tets.size());
    std::vector<int32_t> cur(inc_ptr.begin(), inc_ptr.end() - 1);
    for (int32_t e = 0; e < ne; ++e)
        for (int j = 0; j < 4; ++j) inc[cur[tets[4 * static_cast<size_t>(e) + j]]++] = e;
    return true;
}

bool operator_pattern(int32_t n, const std::vector<int32_t> &tets, const std::vector<int32_t> &inc_ptr,
                      const std::vector<int32_t> &inc, int32_t nb, GsRowsHost &out) {
    // row slices: the sorted neighbours of 64 rows, as a thread's chunk
    const int32_t nsl = (n + 63) / 64;
    std::vector<std::vector<int32_t>> cols(static_cast<size_t>(nsl));
    std::vector<int32_t> width(static_cast<size_t>(nsl), 0);
    std::atomic<bool> ok{true};
    for_each_part(nsl, [&](int32_t s) {
        const int32_t i0 = 64 * s, i1 = std::min(n, i0 + 64);
        std::vector<int32_t> nbr[64];
        for (int32_t i = i0; i < i1; ++i) {
            auto &v = nbr[i - i0];
            for (int32_t t = inc_ptr[i]; t < inc_ptr[i + 1]; ++t)
                for (int j = 0; j < 4; ++j) {
                    const int32_t q = tets[4 * static_cast<size_t>(inc[t]) + j];
                    if (q != i && std::find(v.begin(), v.end(), q) == v.end()) v.push_back(q);
                }
            std::sort(v.begin(), v.end());
            width[s] = std::max(width[s], static_cast<int32_t>(v.size()));
        }
        if (width[s] >= 256) ok = false;
        auto &c = cols[s];
        c.assign(64 * static_cast<size_t>(width[s]), -1);
        for (int32_t i = i0; i < i1; ++i)
            for (size_t k = 0; k < nbr[i - i0].size(); ++k) c[64 * k + i - i0] = nbr[i - i0][k];
    });
    if (!ok) return false;
    out.off.assign(static_cast<size_t>(nsl) + 1, 0);
    int64_t total = 0;
    for (int32_t s = 0; s < nsl; ++s) {
        total += 64 * static_cast<int64_t>(width[s]);
        if (total > INT32_MAX) return false;
        out.off[s + 1] = static_cast<int32_t>(total);
    }
    // blocks of nb rows: halo lists and local columns
    out.nb = nb;
    out.nblk = (n + nb - 1) / nb;
    out.col.assign(static_cast<size_t>(total), 0);
    std::vector<std::vector<int32_t>> halos(static_cast<size_t>(out.nblk));
    for_each_part(out.nblk, [&](int32_t b) {
        const int32_t n0 = b * nb, n1 = std::min(n, n0 + nb);
        auto &h = halos[b];
        for (int32_t s = n0 / 64; s < (n1 + 63) / 64; ++s)
            for (int32_t j : cols[s])
                if (j >= 0 && (j < n0 || j >= n1)) h.push_back(j);
        std::sort(h.begin(), h.end());
        h.erase(std::unique(h.begin(), h.end()), h.end());
        if (static_cast<int64_t>(nb) + static_cast<int64_t>(h.size()) > 65535) {
            ok = false;
            return;
        }
        for (int32_t s = n0 / 64; s < (n1 + 63) / 64; ++s)
            for (size_t k = 0; k < cols[s].size(); ++k) {
                const int32_t j = cols[s][k], i = std::min(n1 - 1, 64 * s + static_cast<int32_t>(k % 64));
                out.col[static_cast<size_t>(out.off[s]) + k] = static_cast<uint16_t>(
                    j < 0 ? i - n0
                    : j >= n0 && j < n1
                        ? j - n0
                        : nb + static_cast<int32_t>(std::lower_bound(h.begin(), h.end(), j) - h.begin()));
            }
    });
    if (!ok) return false;
    out.halo_ptr.assign(static_cast<size_t>(out.nblk) + 1, 0);
    out.nloc_max = 0;
    for (int32_t b = 0; b < out.nblk; ++b) {
        const int32_t sz = static_cast<int32_t>(halos[b].size());
        out.nloc_max = std::max(out.nloc_max, nb + sz);
        out.halo_ptr[b + 1] = out.halo_ptr[b] + sz;
    }
    out.halo_ids.resize(static_cast<size_t>(out.halo_ptr[out.nblk]));
    for (int32_t b = 0; b < out.nblk; ++b)
        std::copy(halos[b].begin(), halos[b].end(), out.halo_ids.begin() + out.halo_ptr[b]);
    return true;
}

bool resident_layout(const GsRowsHost &rows, int32_t n, int32_t nbr, ResLayoutHost &out) {
    out = ResLayoutHost{};
    out.nbr = nbr;
    out.G = (n + nbr - 1) / nbr;
    out.col.assign(rows.col.size(), 0);
    for (size_t k = 0; k + 1 < rows.off.size(); ++k) out.wmax = std::max(out.wmax, (rows.off[k + 1] - rows.off[k]) / 64);
    out.slot.assign(n, -1);
    std::vector<std::vector<int32_t>> halos(static_cast<size_t>(out.G));
    // the global column of entry e of row i
    auto global = [&](int32_t i, size_t e) -> int32_t {
        const int32_t b = i / rows.nb, c = rows.col[e];
        return c < rows.nb ? b * rows.nb + c : rows.halo_ids[static_cast<size_t>(rows.halo_ptr[b]) + c - rows.nb];
    };
    auto block = [&](int32_t g) {
        const int32_t n0 = g * nbr, n1 = std::min(n, n0 + nbr);
        auto &h = halos[g];
        auto each = [&](auto body) {
            for (int32_t i = n0; i < n1; ++i) {
                const int32_t s = i / 64, w = (rows.off[s + 1] - rows.off[s]) / 64;
                for (int32_t k = 0; k < w; ++k) {
                    const size_t e = static_cast<size_t>(rows.off[s]) + 64 * static_cast<size_t>(k) + i % 64;
                    body(e, global(i, e));
                }
            }
        };
        each([&](size_t, int32_t j) {
            if (j < n0 || j >= n1) h.push_back(j);
        });
        std::sort(h.begin(), h.end());
        h.erase(std::unique(h.begin(), h.end()), h.end());
        if (static_cast<int64_t>(nbr) + static_cast<int64_t>(h.size()) > 65534) return;
        each([&](size_t e, int32_t j) {
            out.col[e] = static_cast<uint16_t>(
                j >= n0 && j < n1 ? j - n0 : nbr + static_cast<int32_t>(std::lower_bound(h.begin(), h.end(), j) - h.begin()));
        });
    };
    for_each_part(out.G, block);
    out.halo_ptr.assign(static_cast<size_t>(out.G) + 1, 0);
    for (int32_t g = 0; g < out.G; ++g) {
        const int32_t sz = static_cast<int32_t>(halos[g].size());
        if (nbr + sz > 65534) return false;      // and the staging's zero slot
        out.nhalo_max = std::max(out.nhalo_max, sz);
        out.halo_ptr[g + 1] = out.halo_ptr[g] + sz;
    }
    out.halo_ids.resize(static_cast<size_t>(out.halo_ptr[out.G]));
    for (int32_t g = 0; g < out.G; ++g) {
        std::copy(halos[g].begin(), halos[g].end(), out.halo_ids.begin() + out.halo_ptr[g]);
        for (int32_t j : halos[g]) out.slot[j] = 0;
    }
    for (int32_t j = 0; j < n; ++j)
        if (out.slot[j] == 0) out.slot[j] = out.nexp++;
    return true;
}

}  // namespace gspm
