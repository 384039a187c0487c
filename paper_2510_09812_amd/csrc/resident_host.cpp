// Host side of the resident CG solves: the rows' columns for workgroups of a
// given size, and that size.
#include <algorithm>
#include <atomic>
#include <thread>

#include "resident.h"

namespace gspm {

// One workgroup per CU at most; up to kFlatGroups of them exchange their sums
// in one hop (2.3 us an exchange in a probe, 3 us through leaders), so small
// meshes stop there as long as that leaves a workgroup 256 rows at most, two
// lanes for each.
int32_t resident_rows(int32_t n, int32_t cus) {
    const int32_t most = std::min(cus, kResMaxGroups);
    if (most <= 0) return 0;
    const int32_t need = (n + most - 1) / most;
    int32_t nbr = std::max(64, (need + 63) / 64 * 64);
    if (n <= kFlatGroups * 256) nbr = std::max(nbr, (((n + kFlatGroups - 1) / kFlatGroups) + 63) / 64 * 64);
    return nbr <= 4096 ? nbr : 0;
}

bool resident_layout(const GsRowsHost &rows, int32_t n, int32_t nbr, ResLayoutHost &out) {
    out = ResLayoutHost{};
    out.nbr = nbr;
    out.G = (n + nbr - 1) / nbr;
    out.col.assign(rows.col.size(), 0);
    out.slot.assign(n, -1);
    std::vector<std::vector<int32_t>> halos(static_cast<size_t>(out.G));
    std::atomic<int32_t> next{0};
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
        if (static_cast<int64_t>(nbr) + static_cast<int64_t>(h.size()) > 65535) return;
        each([&](size_t e, int32_t j) {
            out.col[e] = static_cast<uint16_t>(
                j >= n0 && j < n1 ? j - n0 : nbr + static_cast<int32_t>(std::lower_bound(h.begin(), h.end(), j) - h.begin()));
        });
    };
    auto worker = [&]() {
        for (int32_t g; (g = next.fetch_add(1)) < out.G;) block(g);
    };
    const unsigned hw = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    std::vector<std::thread> pool;
    for (unsigned t = 1; t < hw && static_cast<int32_t>(t) < out.G; ++t) pool.emplace_back(worker);
    worker();
    for (auto &t : pool) t.join();
    out.halo_ptr.assign(static_cast<size_t>(out.G) + 1, 0);
    for (int32_t g = 0; g < out.G; ++g) {
        const int32_t sz = static_cast<int32_t>(halos[g].size());
        if (nbr + sz > 65535) return false;
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
