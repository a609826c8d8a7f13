// A program that runs the library's host code without a GPU: it defines the
// HIP entry points that libhelmdg calls, on host memory, so that the library
// binds to these instead of the runtime's.  Kernels do not run; of a few of
// them the launch writes the values that the host code goes on with.  Built and
// run by test_host_paths.py; the first argument names the scenario.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "../include/helmdg.h"

namespace {

struct Launch {
    std::string name;
    int device;
    unsigned grid;
    void **args;
};

struct State {
    std::map<const void *, std::string> kernels;     // host stub -> name
    std::map<char *, size_t> live;                   // allocations
    int n_dev = 1, dev = 0;
    int allocations_left = -1;                       // then hipMalloc fails once (-1: never)
    double clock = 0.0;                              // ms, advanced by on_launch
    std::function<void(const Launch &)> on_launch;
};
// (the library registers its kernels before this program's own objects exist)
State &st()
{
    static State s;
    return s;
}

template <typename T>
T arg(const Launch &l, int i) { return *(T *)l.args[i]; }

// what the set-up reads back from its kernels
void default_launch(const Launch &l)
{
    auto is = [&](const char *n) { return l.name.find(n) != std::string::npos; };
    if (is("k_cell_geometry")) {
        for (int64_t i = 0; i < arg<int64_t>(l, 3); ++i) arg<double *>(l, 7)[i] = 1.0;
    } else if (is("k_affine_detect")) {
        for (int64_t i = 0; i < arg<int64_t>(l, 3); ++i) arg<uint8_t *>(l, 6)[i] = 1;
    }
}

struct Dim3 {
    uint32_t x, y, z;
};
struct Config {
    Dim3 grid, block;
    size_t shmem;
    void *stream;
} g_config;

int failures = 0;
void check(bool ok, const char *what)
{
    if (!ok) {
        ++failures;
        printf("FAILED: %s\n", what);
    }
}

// a mesh of 2 x 1 x 1 unit cells, set up in c
void small_mesh(hx_ctx *c, int degree)
{
    std::vector<double> nodes;
    for (int cell = 0; cell < 2; ++cell)
        for (int v = 0; v < 8; ++v)
            for (double x : {double(cell + (v & 1)), double(v >> 1 & 1), double(v >> 2)}) nodes.push_back(x);
    const int64_t nbr[12] = {-1, 1, -1, -1, -1, -1, 0, -1, -1, -1, -1, -1};
    check(hx_setup_mesh(c, degree, 2, 1, nodes.data(), nbr) == HX_OK, "setup_mesh");
}

hx_ctx *context(int device, int degree)
{
    hx_ctx *c = nullptr;
    check(hx_create(&c, device, nullptr) == HX_OK, "create");
    small_mesh(c, degree);
    return c;
}

void coefficients(hx_ctx *c)
{
    const std::vector<double> one(hx_num_dofs(c), 1.0);
    check(hx_set_coefficients(c, one.data(), one.data(), 2.0, 0) == HX_OK, "set_coefficients");
}

// Calls that rebuild the general cell and face data launch their kernels on
// the context's device whatever the caller's current device is.
void device_of_expansion()
{
    st().n_dev = 2;
    hx_ctx *c = context(1, 2);
    int launches = 0;
    st().on_launch = [&](const Launch &l) {
        ++launches;
        check(l.device == 1, ("launch on the caller's device: " + l.name).c_str());
    };
    std::vector<double> out(2 * 7 * 27);
    for (int call = 0; call < 3; ++call) {
        check(hx_set_cell_compression(c, 1) == HX_OK, "compression on");
        coefficients(c);
        st().dev = 0;
        launches = 0;
        if (call == 0) check(hx_set_cell_compression(c, 0) == HX_OK, "compression off");
        else
            check(hx_debug_export(c, call == 1 ? HX_EXPORT_CELL_DATA : HX_EXPORT_FACE_DATA, out.data(),
                                  8 * (int64_t)out.size()) == HX_OK, "export");
        check(launches == 2, "the general data are rebuilt");
    }
    st().on_launch = nullptr;
    hx_destroy(c);
}

// The phase times that a solve reports, on a clock that the launches advance:
// the block dots of step j of a cycle cost 1 + j / 4, a launch of the solve's
// first step 20, every other one 1.  The first five steps are exact; the estimate for
// the others is near the sum over all steps, whatever the restart length.
void phase_times()
{
    hx_ctx *c = context(0, 2);
    coefficients(c);
    const int64_t n = hx_num_dofs(c);
    std::vector<double> b(n, 1.0), x(n);
    for (int method = 0; method < 2; ++method)
        for (int restart : {5, 7, 11, 13, 14, 22, 30, 48})
            for (int iters : {1, 2, 5, 7, 9, 16, 140, 300}) {
                bool first = true;
                double op = 0.0, pc = 0.0, orth = 0.0;
                bool started = false;
                st().on_launch = [&](const Launch &l) {
                    auto is = [&](const char *k) { return l.name.find(k) != std::string::npos; };
                    double cost = first ? 20.0 : 1.0;
                    if (is("k_dcgs_dot")) cost += 0.25 * arg<int>(l, 1);
                    st().clock += cost;
                    // what the host reads: |.|^2 of a dot product, the step's scalars
                    if (is("k_red2")) std::fill_n(arg<double *>(l, 3), l.grid, 1.0);
                    if (is("k_dcgs_coef")) {
                        double *h = arg<double *>(l, 4);
                        std::fill_n(h, 128, 0.0);
                        h[366] = h[367] = 1.0;   // rho, the column's diagonal entry
                        h[368] = 0.0;
                    }
                    if (is("k_dcgs_update")) {
                        std::fill_n(arg<double *>(l, 8), l.grid, 0.0);
                        arg<double *>(l, 8)[0] = 1.0;
                    }
                    if (is("k_cg_pt_red")) *arg<double *>(l, 8) = 1.0;
                    if (is("k_dcgs_update") || is("k_cg_pt_red")) first = false;
                    // the phases (the residual form, with a right-hand side, and
                    // the first preconditioner of CG are outside the steps)
                    if (is("k_apply") && !arg<void *>(l, 2)) {
                        op += cost;
                        started = true;
                    } else if (is("k_bj") && (method == 1 || started)) {
                        pc += cost;
                    } else if (is("k_dcgs") || is("k_mdot1")) {
                        orth += cost;
                    }
                };
                hx_solve_params prm;
                hx_default_params(&prm);
                prm.method = method;
                prm.restart = restart;
                prm.max_iter = iters;
                prm.rtol = 1e-300;
                hx_solve_info info{};
                hx_solve(c, &prm, b.data(), x.data(), &info);
                st().on_launch = nullptr;
                char what[200];
                snprintf(what, sizeof what, "method %d restart %d: %d of %d steps, op %.1f (%.1f) pc %.1f (%.1f) orth %.1f (%.1f)",
                         method, restart, info.iters, iters, info.ms_op, op, info.ms_pc, pc, info.ms_orth, orth);
                check(info.iters == iters, what);
                const double tol = iters <= 5 ? 1e-5 : 0.1;
                auto near = [&](double a, double ref) { return std::fabs(a - ref) <= tol * ref; };
                check(near(info.ms_op, op) && near(info.ms_pc, pc), what);
                // (a cycle's last block dot is summed by a launch of its own)
                if (method == 1) check(std::fabs(info.ms_orth - orth) <= tol * orth + 25.0 * (1 + iters / restart), what);
            }
    hx_destroy(c);
}

// A call that runs out of memory at any of its allocations reports that, and
// made again it has every buffer that it has at the first attempt elsewhere,
// and none twice.
void failed_allocations()
{
    const std::vector<int32_t> parent{0, 1}, octant{0, 0};
    const char *names[] = {"pressure system", "consistent", "Chebyshev", "multigrid"};
    for (int call = 0; call < 4; ++call) {
        size_t buffers = 0;
        int n = -1;   // allocations before the one that fails; -1: none fails
        for (bool more = true; more; ++n) {
            hx_ctx *c = context(0, 2), *coarse = context(0, 2);
            coefficients(c);
            const std::vector<double> one(hx_num_dofs(c), 1.0);
            auto run = [&] {
                switch (call) {
                case 0: return hx_set_pressure_system(c, one.data(), one.data(), 1.4, 1.0, 2.0, 0);
                case 1: return hx_set_consistent(c, one.data(), one.data(), 0);
                case 2: return hx_set_chebyshev(c, 3, 0.1, 2.0);
                default: return hx_set_multigrid(c, coarse, parent.data(), octant.data());
                }
            };
            st().allocations_left = n;
            const hx_status s = run();
            more = n < 0 || s != HX_OK;
            st().allocations_left = -1;
            if (n >= 0 && more) {
                check(s == HX_ERR_OOM, names[call]);
                check(run() == HX_OK, names[call]);
            }
            if (n < 0) buffers = st().live.size();
            char what[100];
            snprintf(what, sizeof what, "%s, allocation %d refused: %zu buffers, not %zu", names[call], n,
                     st().live.size(), buffers);
            check(st().live.size() == buffers, what);
            hx_destroy(c);
            hx_destroy(coarse);
        }
        check(n > 2, "allocations were refused");
    }
}

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *,
                           void *, void *, int *)
{
    st().kernels[host] = name;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t shmem, void *stream)
{
    g_config = {grid, block, shmem, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *shmem, void **stream)
{
    *grid = g_config.grid;
    *block = g_config.block;
    *shmem = g_config.shmem;
    *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **args, size_t, void *)
{
    const Launch l{st().kernels[f], st().dev, grid.x, args};
    default_launch(l);
    if (st().on_launch) st().on_launch(l);
    return 0;
}
int hipGetDeviceCount(int *n) { return *n = st().n_dev, 0; }
int hipSetDevice(int d) { return st().dev = d, 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "refused"; }
int hipMalloc(void **p, size_t n)
{
    if (st().allocations_left >= 0 && st().allocations_left-- == 0) return 2;
    *p = calloc(n, 1);
    st().live[(char *)*p] = n;
    return 0;
}
int hipFree(void *p)
{
    check(st().live.erase((char *)p) == 1, "free of an address that is not allocated");
    free(p);
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) { return *p = calloc(n, 1), 0; }
int hipHostFree(void *p) { return free(p), 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned) { return *d = h, 0; }
int hipGetSymbolAddress(void **p, const void *)
{
    static char scratch[1 << 20];
    return *p = scratch, 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { return memmove(d, s, n), 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return memmove(d, s, n), 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { return memset(d, v, n), 0; }
int hipEventCreateWithFlags(double **e, unsigned) { return *e = new double(0.0), 0; }
int hipEventDestroy(double *e) { return delete e, 0; }
int hipEventRecord(double *e, void *) { return *e = st().clock, 0; }
int hipEventSynchronize(double *) { return 0; }
int hipEventElapsedTime(float *t, double *a, double *b) { return *t = (float)(*b - *a), 0; }
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "device") device_of_expansion();
    else if (what == "times") phase_times();
    else if (what == "memory") failed_allocations();
    else check(false, "unknown scenario");
    check(st().live.empty(), "device memory left allocated");
    printf("%s: %d failures\n", what.c_str(), failures);
    return failures ? 1 : 0;
}
