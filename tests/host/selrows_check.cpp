// The host side of a requested-rows call (tde_api.cpp over a HIP runtime on
// host memory, the kernels' launchers replaced by recorders): an allocation, a
// copy or a launch that fails at any point leaves nothing running behind a
// returned call, and an allocation fails before anything was enqueued; and the
// passes' requests are every request once, at the row it asks for.
#include "fake_hip/hip/hip_runtime.h"

#include <cstdio>
#include <cstdlib>
#include <random>
#include <utility>
#include <vector>

#include "../../include/tde.h"
#include "../../paper_2605_26599_amd/csrc/tde_dense.h"
#include "../../paper_2605_26599_amd/csrc/tde_plan.h"

static int g_launches = 0, g_fail_launch = -1;
static int launched() {
    if (fake::countdown(&g_fail_launch)) return 1;
    ++g_launches;
    ++fake::pending;
    return 0;
}

static std::vector<long long> g_xrows;                  // the rows of the last pass enqueued
static std::vector<std::pair<int, long long>> g_given;  // (request, row) of every pass

namespace tde {
int enqueue_solve(const Plan& p, const Work& w, const double*, const double*, double*, void*, const Ckpt*,
                  const Ckpt* xsrc) {
    if (xsrc) g_xrows = std::vector<long long>(w.xrows, w.xrows + 2 * p.B);
    return launched();
}
int enqueue_selrows_copies(const double*, const double*, long long, int, double*, double*, void*) {
    return launched();
}
int enqueue_selrows_out(double*, long long, const int* order, const SelRequests& req, int copies, const double*,
                        const double*, const double*, const double*, void*) {
    for (int u = 0; u < 2 * copies; ++u)
        for (int i = req.first[u]; i < req.first[u + 1]; ++i) g_given.push_back({order[i], g_xrows[u]});
    return launched();
}
int enqueue_split_flags(const double*, const double*, long long, int*, void*) { return 0; }
int enqueue_merge_runs(const MergeRec*, int, const double*, double*, long long, void*) { return 0; }
int enqueue_backward(const Plan&, const Work&, const Grad&, const Ckpt&, const double*, const double*, const double*,
                     double*, double*, void*) {
    return 0;
}
size_t dense_layout(long long, char*, DenseWork*) { return 0; }
int enqueue_dense_reduce(double*, long long, int, const DenseWork&, void*) { return 0; }
void timing_enable(bool) {}
bool timing_enabled() { return false; }
int timing_read(double*, long long*, int) { return 0; }
}  // namespace tde

static int g_bad = 0;
#define CHECK(c)                                                                              \
    do {                                                                                      \
        if (!(c)) {                                                                           \
            std::fprintf(stderr, "CHECK failed line %d (step %d): %s\n", __LINE__, step, #c); \
            g_bad = 1;                                                                        \
        }                                                                                     \
    } while (0)

struct Call {
    int64_t n, m;
    std::vector<int64_t> rows;
    std::vector<double> d, e, lam, Q;
    std::vector<char> ws;
    Call(int64_t n_, int64_t m_) : n(n_), m(m_), rows((size_t)m_), d((size_t)n_), e((size_t)n_), lam((size_t)n_) {
        std::mt19937 g(7);
        for (auto& r : rows) r = (int64_t)(g() % (unsigned)n);
        Q.resize((size_t)(n * m));
        ws.resize(tde_selrows_workspace_bytes(n, m, nullptr));
    }
    int run() {
        return tde_eigvals_selrows(d.data(), e.data(), n, rows.data(), m, lam.data(), Q.data(), ws.data(), ws.size(),
                                   nullptr, nullptr);
    }
    void reset() {
        tde_release_plans();
        fake::fail_malloc = fake::fail_async = g_fail_launch = -1;
        g_launches = fake::pending = fake::syncs = 0;
        g_given.clear();
    }
};

int main() {
    Call c(300, 70);  // passes of 16 rows and a shorter last one
    int step = -1;
    c.reset();
    CHECK(c.run() == TDE_OK && fake::pending == 0 && g_launches > 8);
    for (auto [n, m] : {std::pair<int, int>{1, 1}, {1, 40}, {2, 3}, {16, 16}, {17, 17}, {33, 500}, {300, 16},
                        {300, 33}, {300, 2000}, {9, 0}}) {
        Call x(n, m);
        x.reset();
        CHECK(x.run() == TDE_OK);
        std::vector<int> seen((size_t)m, 0);
        for (auto [i, row] : g_given) {
            CHECK(i >= 0 && i < m && row == x.rows[(size_t)i]);
            if (i >= 0 && i < m) ++seen[(size_t)i];
        }
        for (int k : seen) CHECK(k == 1);
        step = n;
    }
    for (int kind = 0; kind < 3; ++kind) {
        int failed = 0;
        for (step = 0; step < 200; ++step) {
            c.reset();
            (kind == 0 ? fake::fail_malloc : kind == 1 ? fake::fail_async : g_fail_launch) = step;
            const int rc = c.run();
            const bool hit = (kind == 0 ? fake::fail_malloc : kind == 1 ? fake::fail_async : g_fail_launch) < 0;
            if (!hit) break;  // fewer steps than that
            ++failed;
            CHECK(rc == (kind == 0 ? TDE_ENOMEM : TDE_EDEVICE));
            CHECK(fake::pending == 0);
            if (kind == 0) CHECK(g_launches == 0);
        }
        CHECK(failed >= 4);
    }
    c.reset();
    std::puts(g_bad ? "selrows bad" : "selrows ok");
    return g_bad;
}
