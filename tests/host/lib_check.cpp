// The library's host code through its C interface, on the host's own memory
// (hip_on_host.cpp): contexts in both precisions, meshes of several sizes one
// after another on one context, every field both ways, refused arrays, solves
// and steps with and without the preconditioner, the network's calls, in arrays
// of exactly the size the interface asks for.  Meant to run under the
// sanitizers; values are checked where the stand-in computes them.
// Usage: lib_check <mesh.bin> <mesh.bin> ...; exit 0 if every call answered as it should.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <limits>
#include <vector>

#include "gspm.h"

namespace {

struct Mesh {
    int64_t n0 = 0, ne = 0;
    double lo[3], hi[3];
    std::vector<double> xyz;
    std::vector<int32_t> tets;
    std::vector<uint8_t> tags;
};

bool read(const char *path, Mesh &m) {
    FILE *fp = fopen(path, "rb");
    if (!fp) return false;
    size_t got = fread(&m.n0, 8, 1, fp) + fread(&m.ne, 8, 1, fp) + fread(m.lo, 8, 3, fp) + fread(m.hi, 8, 3, fp);
    m.xyz.resize(3 * m.n0);
    m.tets.resize(4 * m.ne);
    m.tags.resize(m.ne);
    got += fread(m.xyz.data(), 8, m.xyz.size(), fp) + fread(m.tets.data(), 4, m.tets.size(), fp) +
           fread(m.tags.data(), 1, m.tags.size(), fp);
    fclose(fp);
    return got == 8 + m.xyz.size() + m.tets.size() + m.tags.size();
}

int failures = 0;
void expect(bool ok, const char *what, gspm_ctx *c) {
    if (ok) return;
    ++failures;
    printf("%s: %s\n", what, gspm_last_error(c));
}

gspm_params params(bool green, bool ld) {
    gspm_params p;
    std::memset(&p, 0, sizeof p);
    p.Ms = 1e6; p.A = 1e-11; p.K1 = 1e4; p.lambda100 = 1e-4; p.lambda111 = 1e-5;
    p.c11 = 2e11; p.c12 = 1e11; p.c44 = 1e11; p.alpha = 0.1; p.mu0 = 1.2566e-6; p.gamma0 = 2.2e5;
    for (int a = 0; a < 3; ++a) p.Nd[4 * a] = 1.0 / 3.0;
    p.cg_tol = 1e-8; p.cg_maxit = 20; p.precession = 1; p.local_demag = ld;
    p.elastic_precond = green ? GSPM_PRECOND_GREEN : GSPM_PRECOND_NONE;
    p.gs_precond = green ? GSPM_PRECOND_JACOBI : GSPM_PRECOND_NONE;
    return p;
}

void use(gspm_ctx *c, const Mesh &m) {
    const size_t n3 = 3 * static_cast<size_t>(m.n0);
    expect(gspm_upload_mesh(c, m.n0, m.xyz.data(), m.ne, m.tets.data(), m.tags.data(), m.lo, m.hi, GSPM_PERIODIC) == GSPM_OK,
           "upload", c);
    std::vector<double> v(n3, 0.25), s(m.n0, 0.5), out(n3), so(m.n0);
    for (int round = 0; round < 2; ++round)
        for (int green = 0; green < 2; ++green)
            for (int ld = 0; ld < 2; ++ld) {
                gspm_params p = params(green, ld);
                if (round) p.c44 *= 1.5;                       // rows and symbol rebuilt
                expect(gspm_set_params(c, &p) == GSPM_OK, "set_params", c);
                expect(gspm_set_field(c, GSPM_FIELD_M, v.data(), m.n0) == GSPM_OK, "set M", c);
                expect(gspm_set_field(c, GSPM_FIELD_U, v.data(), m.n0) == GSPM_OK, "set U", c);
                expect(gspm_set_field(c, GSPM_FIELD_UD, s.data(), m.n0) == GSPM_OK, "set UD", c);
                expect(gspm_get_field(c, GSPM_FIELD_U, out.data(), m.n0) == GSPM_OK && out == v, "get U", c);
                expect(gspm_get_field(c, GSPM_FIELD_UD, so.data(), m.n0) == GSPM_OK && so == s, "get UD", c);
                for (size_t at : {size_t(0), n3 - 1}) {
                    std::vector<double> bad = v;
                    bad[at] = std::numeric_limits<double>::quiet_NaN();
                    expect(gspm_set_field(c, GSPM_FIELD_M, bad.data(), m.n0) == GSPM_E_ARG, "refused M", c);
                    std::vector<double> x = v;
                    expect(gspm_solve(c, GSPM_OP_GS, 1e-17, v.data(), bad.data(), m.n0, 1e-8, 10, nullptr) == GSPM_E_ARG,
                           "refused solve", c);
                }
                for (gspm_op op : {GSPM_OP_GS, GSPM_OP_ELASTIC, GSPM_OP_MS}) {
                    int32_t it = -1;
                    std::vector<double> x(n3, 0.0);
                    const gspm_status st = gspm_solve(c, op, 1e-17, v.data(), x.data(), m.n0, 1e-8, 10, &it);
                    expect(st == GSPM_OK || st == GSPM_E_NOCONV, "solve", c);
                    expect(gspm_apply(c, op, 1e-17, v.data(), out.data(), m.n0) == GSPM_OK, "apply", c);
                }
                gspm_step_stats st;
                const gspm_status rc = gspm_step(c, 1e-12, 3, &st);
                expect(rc == GSPM_OK || rc == GSPM_E_NOCONV, "step", c);
                int32_t path = -1;
                expect(gspm_set_solve_path(c, GSPM_PATH_LAUNCHES, 0.0) == GSPM_OK, "path", c);
                const gspm_status rl = gspm_step(c, 1e-12, 1, &st);
                expect(rl == GSPM_OK || rl == GSPM_E_NOCONV, "step by launches", c);
                expect(gspm_set_solve_path(c, GSPM_PATH_AUTO, 0.0) == GSPM_OK &&
                           gspm_get_solve_path(c, &path) == GSPM_OK && path == GSPM_PATH_AUTO, "path back", c);
            }
    std::vector<float> w(GSPM_MPNN_PARAMS, 0.01f), g(GSPM_MPNN_PARAMS);
    expect(gspm_mpnn_set_params(c, w.data(), GSPM_MPNN_PARAMS) == GSPM_OK, "network", c);
    double loss = 0.0, sm = 0.0, coef[2];
    expect(gspm_mpnn_forward(c, v.data(), v.data(), m.n0, out.data(), &sm) == GSPM_OK, "forward", c);
    expect(gspm_mpnn_train_step(c, v.data(), v.data(), v.data(), m.n0, 1e-3f, 1, &loss, g.data()) == GSPM_OK, "train", c);
    expect(gspm_mpnn_get_params(c, g.data(), GSPM_MPNN_PARAMS) == GSPM_OK && g == w, "weights", c);
    expect(gspm_mpnn_warm_start(c, v.data(), v.data(), m.n0, out.data(), coef) == GSPM_OK, "warm start", c);
}

}  // namespace

int main(int argc, char **argv) {
    std::vector<Mesh> meshes(argc - 1);
    for (int k = 1; k < argc; ++k)
        if (!read(argv[k], meshes[k - 1])) return 2;
    for (int det = 0; det < 2; ++det)
        for (int precision : {GSPM_FP64, GSPM_MIXED}) {
            gspm_create_opts o;
            std::memset(&o, 0, sizeof o);
            o.precision = precision;
            o.deterministic = det;
            o.profile = 1;
            gspm_ctx *c = nullptr;
            if (gspm_create(&c, &o) != GSPM_OK) return 1;
            for (const Mesh &m : meshes) use(c, m);
            use(c, meshes[0]);                                 // a smaller mesh again
            gspm_destroy(c);
        }
    printf("%d meshes, %d failures\n", argc - 1, failures);
    return failures ? 1 : 0;
}
