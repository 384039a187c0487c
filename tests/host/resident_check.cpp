// Host check of the row layouts of the one-launch solves (resident_host.cpp):
// the GS rows dealt out to workgroups, and the pattern of the operators over
// all elements, each against neighbour sets formed here from the elements.
//   - every column is a staged node of its workgroup (own rows below the mesh's
//     end, or a halo position) and decodes to the row's neighbours, each once;
//     padding points at the row itself;
//   - halo lists are sorted, outside the workgroup's rows and used;
//   - exchange slots: exactly the nodes of some halo have one, each its own,
//     numbered from 0 without a gap;
//   - if a workgroup reads another's nodes, that one reads its (a round of the
//     exchange is overwritten two rounds later on the strength of this);
//   - the elements of each node are complete and ascending.
// Usage: resident_check <mesh.bin> <compute units> <reorder> <GS row block>; exit 0 if valid.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <string>
#include <vector>

#include "resident.h"
using namespace gspm;

namespace {

long bad = 0;

void fail(const char *what, long a = 0, long b = 0) {
    if (++bad <= 20) printf("%s: %ld %ld\n", what, a, b);
}

void check_layout(const char *name, const GsRowsHost &rows, const ResLayoutHost &ly, int n,
                  const std::vector<std::set<int>> &want) {
    const int G = (n + ly.nbr - 1) / ly.nbr;
    if (ly.G != G || static_cast<int>(ly.halo_ptr.size()) != G + 1 || static_cast<int>(ly.slot.size()) != n ||
        ly.col.size() != rows.col.size() || static_cast<size_t>(ly.halo_ptr[G]) != ly.halo_ids.size()) {
        fail("sizes", ly.G, G);
        return;
    }
    std::vector<char> used(ly.halo_ids.size(), 0);
    std::vector<std::set<int>> reads(G);
    int wmax = 0, nhalo = 0;
    for (int g = 0; g < G; ++g) {
        const int n0 = g * ly.nbr, cnt = std::min(ly.nbr, n - n0), h0 = ly.halo_ptr[g], h1 = ly.halo_ptr[g + 1];
        nhalo = std::max(nhalo, h1 - h0);
        for (int t = h0; t < h1; ++t) {
            const int j = ly.halo_ids[t];
            if (j < 0 || j >= n || (j >= n0 && j < n0 + cnt) || (t > h0 && ly.halo_ids[t - 1] >= j)) fail("halo", g, j);
            else reads[g].insert(j / ly.nbr);
        }
        for (int i = n0; i < n0 + cnt; ++i) {
            const int s = i / 64, w = (rows.off[s + 1] - rows.off[s]) / 64;
            wmax = std::max(wmax, w);
            std::set<int> got;
            for (int k = 0; k < w; ++k) {
                const int c = ly.col[static_cast<size_t>(rows.off[s]) + 64 * static_cast<size_t>(k) + i % 64];
                if (c < ly.nbr ? c >= cnt : c - ly.nbr >= h1 - h0) {
                    fail("column outside the staged nodes", i, c);
                    continue;
                }
                if (c >= ly.nbr) used[h0 + c - ly.nbr] = 1;
                const int j = c < ly.nbr ? n0 + c : ly.halo_ids[h0 + c - ly.nbr];
                if (j == i) continue;
                if (!got.insert(j).second) fail("column twice", i, j);
            }
            if (got != want[i]) fail("neighbours", i, static_cast<long>(got.size()));
        }
    }
    if (wmax != ly.wmax || nhalo != ly.nhalo_max) fail("largest row or halo", wmax, nhalo);
    std::vector<char> exported(n, 0), slot(std::max(ly.nexp, 1), 0);
    for (size_t t = 0; t < ly.halo_ids.size(); ++t) {
        exported[ly.halo_ids[t]] = 1;
        if (!used[t]) fail("halo node not used", static_cast<long>(t));
    }
    for (int i = 0; i < n; ++i) {
        if ((ly.slot[i] >= 0) != (exported[i] != 0)) fail("slot of a node", i, ly.slot[i]);
        if (ly.slot[i] < 0) continue;
        if (ly.slot[i] >= ly.nexp || slot[ly.slot[i]]) fail("slot out of range or taken", i, ly.slot[i]);
        else slot[ly.slot[i]] = 1;
    }
    if (std::count(slot.begin(), slot.end(), 1) != ly.nexp) fail("slots with gaps", ly.nexp);
    for (int g = 0; g < G; ++g)
        for (int h : reads[g])
            if (!reads[h].count(g)) fail("one-sided exchange", g, h);
    printf("%s: n %d, %d workgroups of %d rows, largest halo %d, longest row %d, exported %d\n", name, n, G, ly.nbr, nhalo,
           wmax, ly.nexp);
}

}  // namespace

int main(int argc, char **argv) {
    if (argc < 5) return 2;
    FILE *fp = fopen(argv[1], "rb");
    if (!fp) return 2;
    int64_t n0, ne;
    double lo[3], hi[3];
    size_t got = fread(&n0, 8, 1, fp) + fread(&ne, 8, 1, fp) + fread(lo, 8, 3, fp) + fread(hi, 8, 3, fp);
    if (got != 8) return 2;
    std::vector<double> xyz(3 * n0);
    std::vector<int32_t> tets(4 * ne);
    std::vector<uint8_t> tags(ne);
    got = fread(xyz.data(), 8, 3 * n0, fp) + fread(tets.data(), 4, 4 * ne, fp) + fread(tags.data(), 1, ne, fp);
    fclose(fp);
    if (got != static_cast<size_t>(3 * n0 + 4 * ne + ne)) return 2;
    HostMesh M;
    GsRowsHost gs;
    std::string err;
    if (prepare_mesh(n0, xyz.data(), ne, tets.data(), tags.data(), lo, hi, 256, M, err, atoi(argv[3])) ||
        assemble_gs_rows(M, ne, tets.data(), tags.data(), atoi(argv[4]), gs, err)) {
        printf("%s\n", err.c_str());
        return 1;
    }
    const int n = M.n, nbr = resident_rows(n, atoi(argv[2]), true);
    if (nbr <= 0 || nbr % 64) {
        printf("no rows per workgroup\n");
        return 1;
    }
    std::vector<std::set<int>> mag(n), all(n);
    std::vector<std::vector<int>> elems(n);
    std::vector<int32_t> it(tets.size());
    for (int64_t e = 0; e < ne; ++e)
        for (int a = 0; a < 4; ++a) {
            const int i = M.user2int[tets[4 * e + a]];
            it[4 * e + a] = i;
            elems[i].push_back(static_cast<int>(e));
            for (int b = 0; b < 4; ++b) {
                const int j = M.user2int[tets[4 * e + b]];
                if (i == j) continue;
                all[i].insert(j);
                if (tags[e]) mag[i].insert(j);
            }
        }
    ResLayoutHost ly;
    if (!resident_layout(gs, n, nbr, ly)) fail("GS layout");
    else check_layout("GS", gs, ly, n, mag);
    std::vector<int32_t> inc_ptr, inc;
    GsRowsHost pat;
    if (!node_elements(n, it, inc_ptr, inc)) fail("node_elements");
    for (int i = 0; i < n && !bad; ++i) {
        const std::vector<int> mine(inc.begin() + inc_ptr[i], inc.begin() + inc_ptr[i + 1]);
        if (mine != elems[i]) fail("elements of a node", i);
    }
    if (!operator_pattern(n, it, inc_ptr, inc, nbr, pat) || !resident_layout(pat, n, nbr, ly)) fail("pattern");
    else check_layout("all elements", pat, ly, n, all);
    return bad ? 1 : 0;
}
