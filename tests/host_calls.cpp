// Calls into libqpat's host code on the CPU: this program defines the HIP
// runtime functions that the library uses, so allocations come from (and fail
// at) a place the case names, launches are recorded and not run, and what the
// host reads back from the device is zero unless the case wrote it there.
// Contexts are filled in by hand. host_calls CASE prints what went wrong and
// exits with 1, or exits with 0.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <string>
#include <utility>
#include <vector>

#include "../paper_1512_02796_amd/csrc/qpat_internal.h"

namespace {
constexpr size_t kHeld = 1 << 16;   // bytes behind every allocation, whatever its size
int g_fail_at = -1;                 // allocations that still succeed (-1: all)
bool g_failed = false;              // one did not, since fail_at
hipError_t g_last = hipSuccess;     // as the runtime keeps it until it is asked for
std::map<const void*, std::string>& kernel_names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::vector<std::string> g_launched;
dim3 g_grid;                        // of the launch at hand
std::function<void(const std::string&, void**)> g_on_launch;
struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
} g_config;

hipError_t alloc(void** p) {
    if (g_fail_at == 0) {
        *p = nullptr;
        g_failed = true;
        return g_last = hipErrorOutOfMemory;
    }
    if (g_fail_at > 0) --g_fail_at;
    *p = std::calloc(1, kHeld);
    return hipSuccess;
}

void fail_at(int n) {
    g_fail_at = n;
    g_failed = false;
}

int launches(const char* part) {
    int n = 0;
    for (const std::string& k : g_launched) n += k.find(part) != std::string::npos;
    return n;
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* h;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, uint3*, uint3*, dim3*, dim3*, int*) {
    kernel_names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) {
    g_config = {g, b, l, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
    *g = g_config.grid;
    *b = g_config.block;
    *l = g_config.lds;
    *s = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
    const std::string& name = kernel_names()[f];
    g_grid = grid;
    g_launched.push_back(name);
    if (g_on_launch) g_on_launch(name, args);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t) { return alloc(p); }
hipError_t hipHostMalloc(void** p, size_t, unsigned) { return alloc(p); }
hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
    if (k != hipMemcpyDeviceToDevice && n <= kHeld) std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    std::memset(d, v, n < kHeld ? n : kHeld);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 2;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(&g_config);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.f;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return std::exchange(g_last, hipSuccess); }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

using namespace qpat;

namespace {
#define EXPECT(cond)                                                  \
    do {                                                              \
        if (!(cond)) {                                                \
            std::printf("line %d: not so: %s\n", __LINE__, #cond);    \
            return 1;                                                 \
        }                                                             \
    } while (0)

// a context on an nx x ny x nz node Kuhn lattice with n_ill illuminations, solves without graphs or autotuning
qpat_ctx* box(int nx, int ny, int nz, int n_ill) {
    qpat_ctx* c = new qpat_ctx();
    qpat_default_opts(&c->opts);
    c->opts.use_graphs = 0;
    c->opts.autotune = 0;
    c->N = (int64_t)nx * ny * nz;
    c->E = (int64_t)6 * (nx - 1) * (ny - 1) * (nz - 1);
    c->n_ill = n_ill;
    c->n_pad = n_ill <= 16 ? 16 : (n_ill + 15) / 16 * 16;
    c->sell.N = c->N;
    c->lat.on = true;
    c->lat.nx = nx;
    c->lat.ny = ny;
    c->lat.nz = nz;
    c->lat.m = 7;
    for (int8_t& k : c->lat.code) k = -1;
    for (int m = 0; m < 8; ++m) c->lat.code[13 + (m & 1) + 3 * ((m >> 1) & 1) + 9 * (m >> 2)] = static_cast<int8_t>(m);
    for (int m = 1; m < 8; ++m) {
        c->lat.dx[m - 1] = m & 1;
        c->lat.dy[m - 1] = (m >> 1) & 1;
        c->lat.dz[m - 1] = static_cast<int8_t>(m >> 2);
    }
    c->vox = 0;
    for (double& h : c->vox_h) h = 1.0;
    for (double** p : {&c->geo, &c->barea, &c->kappa, &c->mu, &c->K64, &c->Kdinv64, &c->KU64, &c->M64, &c->Mdinv64, &c->MU64,
                       &c->f, &c->phi, &c->x64, &c->b64, &c->partials, &c->acc1, &c->acc2, &c->dvec, &c->lu, &c->lq, &c->lw,
                       &c->lv, &c->lwh, &c->red_partials, &c->red_out, &c->red_host})
        (void)dalloc(c, p, 1);
    for (void** p : {&c->xl, &c->rl, &c->pa, &c->pb, &c->ql}) (void)dalloc(c, reinterpret_cast<char**>(p), 1);
    for (int32_t** p : {&c->tets, &c->bfaces, &c->n2t_ptr, &c->n2t, &c->n2f_ptr, &c->n2f, &c->lat_tab, &c->dev_flag})
        (void)dalloc(c, p, 1);
    (void)dalloc(c, &c->scal, 1);
    (void)dalloc(c, &c->shared, 1);
    (void)dalloc(c, &c->scal_host, 1);
    (void)dalloc(c, &c->live, 1);
    c->live_dev = c->live;
    (void)dalloc(c, &c->ls, 1);
    (void)dalloc(c, &c->ls_host, 1);
    return c;
}

const double kSome[4] = {};   // stands for a caller's device array: never read here
double g_out[4];
// A second set-up of the guess network with other sides of the same product works on those sides.
int guess_sides() {
    qpat_ctx* c = box(5, 16, 2, 1);
    int sides[3] = {};
    g_on_launch = [&](const std::string& name, void** args) {
        if (name.find("k_inputs_raw") != std::string::npos) std::memcpy(sides, args[0], sizeof sides);   // Lat: nx, ny, nz first
    };
    float in[4] = {}, out[4] = {};
    const int want[3][3] = {{5, 16, 2}, {16, 5, 2}, {16, 5, 2}};
    for (const auto& w : want) {
        EXPECT(qpat_guess_setup(c, w[0], w[1], w[2]) == QPAT_OK);
        EXPECT(qpat_guess_eval(c, in, out) == QPAT_OK);
        EXPECT(std::memcmp(sides, w, sizeof sides) == 0);
    }
    const size_t held = c->allocs.size();   // set up again with the same sides: nothing is allocated
    EXPECT(qpat_guess_setup(c, 16, 5, 2) == QPAT_OK && c->allocs.size() == held);
    return 0;
}

// A set-up of the guess network that failed at any of its allocations is not taken for a finished one.
int guess_alloc_failures() {
    qpat_ctx* c = box(5, 16, 2, 1);
    float some[4] = {};
    for (int k = 0;; ++k) {
        fail_at(k);
        const qpat_status s = qpat_guess_setup(c, 5, 16, 2);
        const bool reached = g_failed;
        fail_at(-1);
        if (!reached) {
            EXPECT(s == QPAT_OK);
            break;
        }
        EXPECT(s == QPAT_ERR_OOM);
        EXPECT(qpat_guess_eval(c, some, some) == QPAT_ERR_STATE);
    }
    EXPECT(qpat_guess_eval(c, some, some) == QPAT_OK);
    // the same for a change of sides: every buffer is there again after a later, successful call
    for (int k = 0; k < 3; ++k) {
        fail_at(k);
        EXPECT(qpat_guess_setup(c, 2, 16, 5) == QPAT_ERR_OOM);
        fail_at(-1);
        EXPECT(qpat_guess_eval(c, some, some) == QPAT_ERR_STATE);
    }
    EXPECT(qpat_guess_setup(c, 2, 16, 5) == QPAT_OK);
    EXPECT(qpat_guess_eval(c, some, some) == QPAT_OK);
    return 0;
}

// The voxel kernel of J^T t takes 32-bit offsets into phi [N][n_pad]: the limit is looked at for the n_pad of each
// call, however many illuminations the context had when the form was first checked.
int voxel_limit_per_call() {
    qpat_ctx* c = box(205, 205, 203, 16);   // 8.5 million nodes: 16 columns fit, 64 do not, 16 fit again
    for (const int n_ill : {16, 64, 16}) {
        c->n_ill = c->n_pad = n_ill;
        SolveStats st;
        g_launched.clear();
        EXPECT(vjp_core(c, kSome, 0, g_out, &st) == QPAT_OK);
        const bool fits = c->N * n_ill * 8 < (int64_t(1) << 31);
        EXPECT((launches("k_gadj_vgather") > 0) == fits);
        EXPECT(launches("k_gadj_gather") >= (fits ? 0 : 1));
    }
    return 0;
}

// A product taken while the sliced-ELL form was asked for leaves the question of the voxel form open.
int voxel_form_after_format_0() {
    qpat_ctx* c = box(9, 10, 11, 16);
    c->opts.operator_format = 0;
    SolveStats st;
    EXPECT(vjp_core(c, kSome, 0, g_out, &st) == QPAT_OK);
    bool done = true;
    EXPECT(assemble_K_lattice(c, &done) == QPAT_OK && !done);
    c->opts.operator_format = 1;
    EXPECT(assemble_K_lattice(c, &done) == QPAT_OK && done);
    g_launched.clear();
    EXPECT(vjp_core(c, kSome, 0, g_out, &st) == QPAT_OK);
    EXPECT(launches("k_gadj_vgather") > 0);
    return 0;
}

// A forward call that fails once it has written the coefficients leaves no linearisation point (the products and
// LSQR steps would mix the old fluence with the new coefficients); one refused before that leaves the old one.
int failed_forward_state() {
    double k0 = 1.0, m0 = 1.0;
    const std::function<qpat_status(qpat_ctx*)> calls[] = {
        [](qpat_ctx* c) { return qpat_forward(c, kSome, kSome, nullptr, nullptr, nullptr); },
        [](qpat_ctx* c) { return qpat_forward_x0(c, kSome, kSome, kSome, nullptr, nullptr, nullptr); },
        [](qpat_ctx* c) { return qpat_forward_log(c, 1.0, 1.0, kSome, nullptr, nullptr, nullptr); },
        [&](qpat_ctx* c) { return qpat_fit_background(c, kSome, kSome, &k0, &m0, 1, 0.0, nullptr, nullptr); }};
    for (int i = 0; i < 4; ++i) {
        qpat_ctx* c = box(9, 10, 11, 4);
        if (i < 3) {   // the check of the input finds a value that is not positive and finite
            c->have_forward = c->lsqr_ready = true;
            *c->dev_flag = 16;
            EXPECT(calls[i](c) == QPAT_ERR_ARG);
            EXPECT(c->have_forward == (i < 2) && c->lsqr_ready == (i < 2));   // forward_log has written exp(beta)
            *c->dev_flag = 0;
        }
        c->have_forward = c->lsqr_ready = true;
        fail_at(i < 3 ? 0 : 6);   // the assembly's first array (past the fit's own six)
        EXPECT(calls[i](c) == QPAT_ERR_OOM);
        fail_at(-1);
        EXPECT(qpat_jvp(c, kSome, g_out, nullptr) == QPAT_ERR_STATE);
        EXPECT(qpat_vjp(c, kSome, g_out, nullptr) == QPAT_ERR_STATE);
        EXPECT(qpat_lsqr_step(c, nullptr, nullptr) == QPAT_ERR_STATE);
    }
    return 0;
}

// A prior set-up that fails once it has written the matrices leaves no prior.
int failed_prior_state() {
    qpat_ctx* c = box(9, 10, 11, 4);
    c->have_prior = c->lsqr_ready = true;
    EXPECT(qpat_prior_setup(c, kSome, kSome, -1.0, 1.0, 1.0) == QPAT_ERR_ARG && c->have_prior);
    fail_at(0);
    EXPECT(qpat_prior_setup(c, kSome, kSome, 1.0, 1.0, 1.0) == QPAT_ERR_OOM);
    fail_at(-1);
    EXPECT(qpat_prior_solve(c, kSome, g_out, nullptr) == QPAT_ERR_STATE);
    EXPECT(qpat_prior_apply(c, kSome, g_out) == QPAT_ERR_STATE);
    EXPECT(qpat_lsqr_step(c, nullptr, nullptr) == QPAT_ERR_STATE);
    return 0;
}

// A multigrid set-up that fails at any of its allocations leaves no half-built hierarchy and gives back what it made;
// the next one builds it whole.
int hierarchy_alloc_failures() {
    for (const Op op : {Op::K, Op::Prior}) {
        qpat_ctx* c = box(33, 34, 35, 16);
        const size_t held = c->allocs.size();
        for (int k = 0;; ++k) {
            fail_at(k);
            const qpat_status s = mg_setup(c, op);
            const bool failed = g_failed;
            fail_at(-1);
            EXPECT(s == (failed ? QPAT_ERR_OOM : QPAT_OK));
            EXPECT(mg_ready(c, op) == !failed);
            if (!failed) break;
            const MgState* M = op == Op::K ? c->mgk : c->mg;
            EXPECT(M == nullptr ? c->allocs.size() == held : op == Op::Prior);   // M_delta: past its hierarchy, the regions'
        }
        const size_t whole = c->allocs.size();
        EXPECT(mg_setup(c, op) == QPAT_OK && c->allocs.size() == whole);
        qpat_ctx* d = box(33, 34, 35, 16);   // one that never failed holds as many arrays
        EXPECT(mg_setup(d, op) == QPAT_OK && d->allocs.size() == whole);
    }
    return 0;
}

// The same for what a first solve sets up: the direction ring and the tile schedule.
int solve_alloc_failures() {
    const auto ready = [] {
        qpat_ctx* c = box(33, 34, 35, 16);
        c->opts.autotune = 1;
        (void)mg_setup(c, Op::K);
        return c;
    };
    qpat_ctx* d = ready();   // one that never fails
    SolveStats st;
    EXPECT(mg_solve(d, Op::K, 16, &st) == QPAT_OK);
    int32_t want[8], got[8];
    EXPECT(mg_tile_schedule(d, 16, want) == QPAT_OK && want[0] == 1 && want[7] == 1);
    // (the times of the tuned schedule are kept for the process: another lattice of the same size reuses them, so the
    // failures of the tuning itself are met on lattices of other sizes)
    for (int k = 0, failed = 1; failed; ++k) {
        qpat_ctx* c = box(33, 34, 37 + 2 * k, 16);
        c->opts.autotune = 1;
        EXPECT(mg_setup(c, Op::K) == QPAT_OK);
        fail_at(k);
        const qpat_status s = mg_solve(c, Op::K, 16, &st);
        failed = g_failed;
        fail_at(-1);
        EXPECT(failed ? s != QPAT_OK : s == QPAT_OK);
        EXPECT(mg_solve(c, Op::K, 16, &st) == QPAT_OK);
        EXPECT(c->allocs.size() >= d->allocs.size());
        EXPECT(mg_tile_schedule(c, 16, got) == QPAT_OK && got[0] == 1 && got[7] == 1);
    }
    return 0;
}

// The same for the arrays of the Jacobian's products and the check of the voxel form, which settles nothing when it
// could not be made and gives back its own arrays.
int product_alloc_failures() {
    size_t whole = 0;
    for (int k = -1, failed = 1; failed; ++k) {   // -1: never
        qpat_ctx* c = box(9, 10, 11, 16);
        EXPECT(mg_setup(c, Op::K) == QPAT_OK);
        SolveStats st;
        fail_at(k);
        qpat_status s = jvp_core(c, kSome, 0, g_out, &st);
        if (s == QPAT_OK) s = vjp_core(c, kSome, 0, g_out, &st);
        failed = k < 0 || g_failed;
        fail_at(-1);
        EXPECT(k < 0 || !failed ? s == QPAT_OK : s != QPAT_OK);
        EXPECT(jvp_core(c, kSome, 0, g_out, &st) == QPAT_OK && vjp_core(c, kSome, 0, g_out, &st) == QPAT_OK);
        EXPECT(c->vox == 1 && c->vox_rows == 1);
        if (k < 0) whole = c->allocs.size();
        EXPECT(c->allocs.size() == whole);
    }
    return 0;
}

// Sources whose arrays could not be made leave none: forward calls and products are refused until others are set.
int failed_sources_state() {
    for (int k = 0; k < 6; ++k) {
        qpat_ctx* c = box(9, 10, 11, 4);
        c->have_forward = c->lsqr_ready = true;
        fail_at(k);
        EXPECT(qpat_set_sources(c, 20, kSome) == QPAT_ERR_OOM);
        fail_at(-1);
        EXPECT(qpat_forward(c, kSome, kSome, nullptr, nullptr, nullptr) == QPAT_ERR_STATE);
        EXPECT(qpat_jvp(c, kSome, g_out, nullptr) == QPAT_ERR_STATE);
        EXPECT(qpat_lsqr_step(c, nullptr, nullptr) == QPAT_ERR_STATE);
        EXPECT(qpat_set_sources(c, 20, kSome) == QPAT_OK && c->n_ill == 20 && c->n_pad == 32);
        EXPECT(c->f && c->phi && c->dvec && c->lu && c->lq && c->lw);
    }
    return 0;
}

// A solve whose right-hand sides are all zero, or whose start solves them, ends before its iterations (Jacobi-PCG: some
// of them are there to cover the question); one that the device says nothing about does not.
int idle_solves() {
    for (const bool idle : {true, false})
        for (const bool multigrid : {true, false})
            for (const bool x0 : {false, true})
                for (const int B : {4, 16}) {
                    qpat_ctx* c = box(17, 18, 19, B);
                    c->opts.pcg_precond = multigrid ? 1 : 0;
                    EXPECT(mg_setup(c, Op::K) == QPAT_OK && mg_ready(c, Op::K) == multigrid);
                    c->K_sell = true;
                    g_launched.clear();
                    g_on_launch = [&](const std::string& name, void**) {
                        if (idle && (name.find("k_red_true") != std::string::npos ||
                                     name.find(x0 ? "k_mgp_true_fin" : "k_mgp_init") != std::string::npos))
                            for (int i = 0; i < B; ++i) c->live[i] = c->live_tag;
                    };
                    SolveStats st;
                    EXPECT((multigrid ? mg_solve(c, Op::K, B, &st, x0) : pcg_solve(c, Op::K, B, &st, x0)) == QPAT_OK);
                    EXPECT(st.n_solves == B);
                    EXPECT(idle ? launches("k_mgp_scalars") == 0 && launches("k_red_alpha") <= (x0 ? 2 : 8)
                                : launches("k_mgp_scalars") + launches("k_red_alpha") >= 13);
                    EXPECT(!(multigrid && B == 16 && !x0) || launches("k_mgp_ring_flush") >= 1);   // x = 0 is written
                }
    return 0;
}

// The sliced-ELL product runs no more blocks than the device keeps resident (2 on each of 256 units here).
int resident_blocks() {
    for (const int precision : {0, 1})
        for (const int B : {1, 8, 16}) {
            qpat_ctx* c = box(65, 65, 65, B);
            c->opts.pcg_precond = c->opts.operator_format = 0;
            c->opts.precision = precision;
            c->K_sell = true;
            unsigned most = 0;
            g_on_launch = [&](const std::string& name, void**) {
                if (name.find("k_dir_spmv") != std::string::npos) most = std::max(most, g_grid.x);
            };
            SolveStats st;
            EXPECT(pcg_solve(c, Op::K, B, &st) == QPAT_OK);
            EXPECT(most > 256 && most <= 512);
        }
    return 0;
}
}  // namespace

int main(int argc, char** argv) {
    const std::pair<const char*, int (*)()> cases[] = {
        {"guess_sides", guess_sides},
        {"guess_alloc_failures", guess_alloc_failures},
        {"voxel_limit_per_call", voxel_limit_per_call},
        {"voxel_form_after_format_0", voxel_form_after_format_0},
        {"failed_forward_state", failed_forward_state},
        {"failed_prior_state", failed_prior_state},
        {"hierarchy_alloc_failures", hierarchy_alloc_failures},
        {"solve_alloc_failures", solve_alloc_failures},
        {"product_alloc_failures", product_alloc_failures},
        {"failed_sources_state", failed_sources_state},
        {"idle_solves", idle_solves},
        {"resident_blocks", resident_blocks},
    };
    for (const auto& k : cases)
        if (argc == 2 && std::string(argv[1]) == k.first) return k.second();
    std::printf("no such case\n");
    return 2;
}
