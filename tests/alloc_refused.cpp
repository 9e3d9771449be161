// Calls of libsko while the runtime refuses device memory, for test_gpu_alloc_refused.py.
//
// The program defines hipMalloc, so the library's allocations come here: a refused one is passed on
// as a request no device can hold (the runtime fails it and records the error, as it does when
// memory has run out), any other one is allocated.  Prints "name value" lines.
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "context.h"
#include "sko_internal.h"

static size_t g_from = SIZE_MAX;  // requests of this size and above are refused ...
static int g_refuse = 0;          // ... as many times as this
static size_t g_largest = 0;

extern "C" hipError_t hipMalloc(void** p, size_t bytes) {
    if (bytes >= g_from && g_refuse > 0) {
        --g_refuse;
        return hipExtMallocWithFlags(p, size_t(1) << 60, hipDeviceMallocDefault);
    }
    if (bytes > g_largest) g_largest = bytes;
    return hipExtMallocWithFlags(p, bytes, hipDeviceMallocDefault);
}

template <typename T>
static T* upload(const std::vector<T>& v) {
    void* p = nullptr;
    if (hipExtMallocWithFlags(&p, v.size() * sizeof(T), hipDeviceMallocDefault) != hipSuccess) std::exit(3);
    if (hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) std::exit(3);
    return static_cast<T*>(p);
}

// Five-point stencil on N x N with centre 5 (condition number below 9).
static sko_csr stencil(int N) {
    std::vector<int32_t> rp{0}, ci;
    std::vector<double> va;
    for (int y = 0; y < N; ++y)
        for (int x = 0; x < N; ++x) {
            auto put = [&](int xx, int yy, double v) {
                if (xx >= 0 && xx < N && yy >= 0 && yy < N) {
                    ci.push_back(yy * N + xx);
                    va.push_back(v);
                }
            };
            put(x, y - 1, -1.0);
            put(x - 1, y, -1.0);
            put(x, y, 5.0);
            put(x + 1, y, -1.0);
            put(x, y + 1, -1.0);
            rp.push_back((int32_t)ci.size());
        }
    return sko_csr{(int64_t)N * N, (int64_t)ci.size(), upload(rp), upload(ci), upload(va)};
}

static double* vec(int64_t n, bool ramp) {
    std::vector<double> v((size_t)n, 0.0);
    for (int64_t i = 0; ramp && i < n; ++i) v[(size_t)i] = std::sin(0.37 * (double)i) + 0.1;
    return upload(v);
}

static sko_sketch sparse_sign() {
    sko_sketch s{};
    s.kind = SKO_SKETCH_SPARSE_SIGN;
    s.k = 64;
    s.zeta = 8;
    s.seed = 3;
    return s;
}

static sko_gmres_opts gmres_opts(int precond) {
    sko_gmres_opts o{};
    o.s = 4;
    o.m = o.shat = 12;
    o.two_stage = 1;
    o.precond = precond;
    o.intra = SKO_INTRA_RANDCHOLQR;
    o.sketch = sparse_sign();
    o.tol = 1e-10;
    return o;
}

// 1 if the context's profile holds matrix-powers kernels by diagonals, 0 if CSR ones
static int by_diagonals(sko_ctx c) {
    std::vector<sko_kernel_stat> st(64);
    const int n = sko_profile_read(c, st.data(), 64);
    for (int i = 0; i < n; ++i)
        if (!std::strncmp(st[(size_t)i].name, "spmv dia", 8)) return 1;
    return 0;
}

static void report(const char* name, long long v) { std::printf("%s %lld\n", name, v); }

int main(int argc, char** argv) {
    const std::string mode = argc > 1 ? argv[1] : "";
    sko_ctx c = nullptr;
    if (sko_create(0, nullptr, &c) != SKO_OK) return 2;
    if (mode == "gmres") {
        const sko_csr A = stencil(64);
        double *b = vec(A.n, true), *x = vec(A.n, false);
        const sko_gmres_opts o = gmres_opts(argc > 2);
        sko_gmres_info info{};
        g_from = 1 << 20, g_refuse = 1;
        sko_profile_enable(c, 1);
        report("status", sko_gmres(c, &A, b, x, &o, &info));
        report("refused", 1 - g_refuse);
        report("converged", info.converged && info.relres <= o.tol);
        report("diagonals", by_diagonals(c));
    } else if (mode == "batch") {
        const sko_csr A[3] = {stencil(64), stencil(40), stencil(23)};
        double *b[3], *x[3];
        for (int i = 0; i < 3; ++i) b[i] = vec(A[i].n, true), x[i] = vec(A[i].n, false);
        const sko_gmres_opts o = gmres_opts(1);
        sko_gmres_info info[3] = {};
        g_from = 1 << 20, g_refuse = 1;
        sko_profile_enable(c, 1);
        report("status", sko_gmres_batched(c, 3, A, b, x, &o, info));
        report("refused", 1 - g_refuse);
        report("converged", info[0].converged && info[1].converged && info[2].converged);
        report("diagonals", by_diagonals(c));
    } else {
        const int64_t n = 20000, w = 6, nb = 4, N = nb * w;
        std::vector<double> v((size_t)(n * N));
        for (size_t i = 0; i < v.size(); ++i) v[i] = std::sin(1.0 + 0.001 * (double)i * (double)(1 + i % 97));
        const double* V = upload(v);
        double* Q = vec(n * N, false);
        sko_orth_opts o{};
        o.intra = SKO_INTRA_RANDCHOLQR;
        o.panels_per_big = 1;
        o.sketch = sparse_sign();
        std::vector<double> R((size_t)(N * N)), R0 = R;
        int32_t col = 0;
        if (mode == "every") {
            g_from = 1 << 16, g_refuse = 1000;
            report("refused_status", sko_orth_blocks(c, n, nb, w, V, n, Q, n, R.data(), N, &o, &col));
            g_refuse = 0;
        } else if (mode == "autotune") {
            // single block steps' and panels' passes, tuned or not (projections of 18 columns: 4 tiles)
            const int64_t rows = 1 << 19;
            const int bucket = 11, W = (int)w;
            auto tuned = [&](sko::PassKey k) {
                k.tiles = 4;
                return (long long)c->grid_wpc.count({sko::pass_kernel_id(k), bucket});
            };
            auto solo = [&](int red, int kind) {
                sko::PassKey k{W, false, red, false, 0, false};
                k.pair = kind;
                return k;
            };
            report("tune_one_stage", sko_autotune_orth(c, rows, nb, w, &o));
            report("doubles_per_row", (long long)(g_largest / (8 * (size_t)rows)));
            report("block_steps", tuned({W, false, sko::RED_PROJ, false, 0, false}) +
                                      tuned({W, false, sko::RED_SKETCH_SPARSE, true, 0, true}) +
                                      tuned({W, false, sko::RED_GRAM, false, 1, false}) +
                                      tuned(solo(sko::RED_PROJ, sko::SOLO_PROJ)) +
                                      tuned(solo(sko::RED_GRAM, sko::SOLO_UPD)) +
                                      tuned({W, false, sko::RED_NONE, false, 1, true}));
            report("look_ahead", tuned(solo(sko::RED_PROJ, sko::PAIR_PROJ)) + tuned(solo(sko::RED_GRAM, sko::PAIR_UPD)) +
                                     tuned(solo(sko::RED_SKETCH_SPARSE, sko::PAIR_LEAD)));
            c->grid_wpc.clear();
            o.two_stage = 1;
            o.panels_per_big = 2;
            report("tune_two_stage", sko_autotune_orth(c, rows, nb, w, &o));
            report("panels", tuned({W, false, sko::RED_PROJ, false, 0, false}) +
                                 tuned({W, false, sko::RED_SKETCH_SPARSE, true, 0, true}) +
                                 tuned({W, false, sko::RED_SKETCH_SPARSE, false, 0, false}) +
                                 tuned({W, false, sko::RED_NONE, true, 1, true}) +
                                 tuned({W, false, sko::RED_NONE, false, 1, true}));
            sko_destroy(c);
            return 0;
        } else if (mode == "blocks") {
            g_from = 1 << 16, g_refuse = 1;
        } else {
            return 2;
        }
        report("status", sko_orth_blocks(c, n, nb, w, V, n, Q, n, R.data(), N, &o, &col));
        if (mode == "blocks") report("refused", 1 - g_refuse);
        sko_ctx c2 = nullptr;
        if (sko_create(0, nullptr, &c2) != SKO_OK) return 2;
        g_refuse = 0;
        report("status_plain", sko_orth_blocks(c2, n, nb, w, V, n, Q, n, R0.data(), N, &o, &col));
        double d = 0.0, m = 0.0;
        for (size_t i = 0; i < R.size(); ++i) d = std::fmax(d, std::fabs(R[i] - R0[i])), m = std::fmax(m, std::fabs(R0[i]));
        report("same_r", d <= 1e-11 * m);
        sko_destroy(c2);
    }
    report("left_error", hipPeekAtLastError());
    sko_destroy(c);
    return 0;
}
