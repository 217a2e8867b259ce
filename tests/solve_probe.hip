// The library's host side (csrc/api.hip) on a model of the device, without a
// GPU: a stream is a list of tasks that run, in order, when the host waits for
// it or copies from it, and one at a time when it asks for it, so what a call
// leaves behind in a stream can be seen, and let run as late as a busy device
// would.  A sweep's task
// adds 1 to the first value of V (nothing behind a closed gate), its norms
// halve from sweep to sweep and go to every block's partial maxima.
// Usage: solve_probe SCENARIO; prints one "name value" per line.
#include "api.hip"

#include <cstdlib>
#include <deque>
#include <functional>
#include <map>

namespace fake {

struct Stream {
    std::deque<std::function<void()>> tasks;
    void step() {
        auto t = std::move(tasks.front());
        tasks.pop_front();
        t();
    }
    void run() {
        while (!tasks.empty()) step();
    }
};
std::map<hipStream_t, Stream> streams;
int mallocs = 0, frees = 0;
bool refuse_mallocs = false, poison = false;   // poison: the FP32 sweeps' norms are NaN

hipError_t put(hipStream_t s, std::function<void()> t) {
    streams[s].tasks.push_back(std::move(t));
    return hipSuccess;
}
size_t queued(hipStream_t s) { return streams[s].tasks.size(); }

template <typename T>
hipError_t sweep(const ptk::SweepPtrs<T>& p, int64_t blocks, bool step, hipStream_t s) {
    return put(s, [=] {
        if (p.gate && *p.gate != 0.0) return;
        const T n = p.vx[0] + T(step ? 1 : 0);
        if (step) p.vx_o[0] = n;
        for (int64_t q = 0; q < blocks * ptk::NNORM; ++q) p.partials[q] = poison && sizeof(T) == 4 ? NAN : std::pow(0.5, (double)n);
    });
}

}  // namespace fake

extern "C" {
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
extern const char __hip_fatbin[64] = {};

hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "model error"; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { *p = const_cast<void*>(symbol); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { fake::streams[s].run(); return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t s) {
    if (!fake::queued(s)) return hipSuccess;
    fake::streams[s].step();
    return hipErrorNotReady;
}
hipError_t hipMemcpyAsync(void* d, const void* a, size_t n, hipMemcpyKind, hipStream_t s) {
    fake::streams[s].run();
    std::memcpy(d, a, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t s) {
    return fake::put(s, [=] { std::memset(d, v, n); });
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    ++fake::mallocs;
    if (fake::refuse_mallocs) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {   // waits for the device
    ++fake::frees;
    for (auto& s : fake::streams) s.second.run();
    std::free(p);
    return hipSuccess;
}
}

namespace ptk {
hipError_t launch_fill(double* d, double v, int64_t n, hipStream_t s) {
    return fake::put(s, [=] { std::fill(d, d + std::min<int64_t>(n, 64), v); });
}
hipError_t launch_iteration(const Geom&, const Tiling& t, const Coef&, const SweepPtrs<double>& p, int mode, int norms,
                            hipStream_t s) {
    return fake::sweep(p, mode == MD_RESID ? t.resid : norms ? t.norms64 : 0, mode != MD_RESID, s);
}
hipError_t launch_correction(const Geom&, const Tiling& t, const Coef&, const SweepPtrs<float>& p, int norms, hipStream_t s) {
    return fake::sweep(p, norms ? t.norms32 : 0, true, s);
}
hipError_t launch_correction64(const Geom&, const Tiling& t, const Coef&, const SweepPtrs<double>& p, int norms,
                               hipStream_t s) {
    return fake::sweep(p, norms ? t.norms64 : 0, true, s);
}
hipError_t launch_reduce_max(const double* part, int64_t nb, double* out, hipStream_t s) {
    return fake::put(s, [=] {
        for (int q = 0; q < NNORM; ++q) {
            out[q] = 0.0;
            for (int64_t b = 0; b < nb; ++b)
                if (!(part[b * NNORM + q] <= out[q])) out[q] = part[b * NNORM + q];
        }
    });
}
hipError_t launch_check(const double* part, int64_t nb, double* out, const double* domain, double* gate, const CheckRule& r,
                        double* slot, double number, hipStream_t s) {
    return fake::put(s, [=] {
        if (gate[0] != 0.0) return;
        double n = 0.0;
        for (int64_t b = 0; b < nb; ++b)
            if (!(part[b * NNORM] <= n)) n = part[b * NNORM];
        const bool stop = !std::isfinite(n) || n / r.ref_v <= r.tol || (r.ref_v2 > 0.0 && n / r.ref_v2 <= r.tol2);
        if (stop) gate[0] = 1.0;
        for (int q = 0; q < NNORM; ++q) out[q] = n;
        if (!slot) return;
        for (int q = 0; q < NNORM; ++q) slot[q] = n;
        slot[NNORM] = *domain;
        slot[NNORM + 1] = stop ? 1.0 : 0.0;
        slot[NNORM + 2] = number;
    });
}
hipError_t launch_copy(const double*, double*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_begin_step(const Geom&, const Coef&, const AuxPtrs&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_refresh(const Geom&, const TileShape&, const Coef&, const RefreshCoef&, const AuxPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_fo_tiled(const Geom&, const TileShape&, const Coef&, const RefreshCoef&, const AuxPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_porosity_step(const Geom&, const Coef&, const AuxPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_set_porosity(const Geom&, const double*, double*, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_damped_residual(const Geom&, const Coef&, const double*, const double*, const double*, const double*, const double*, const double*, const double*, double*, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_prepare_mixed(const Geom&, const MixedPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_apply_correction(const Geom&, const MixedPtrs& m, hipStream_t s) { return fake::put(s, [=] { m.vx[0] += m.dvx[0]; }); }
hipError_t launch_gather(const double*, const int64_t*, int, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_scatter(const double*, const int64_t*, int, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_chi64(const Geom&, const double*, const double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_adjoint_gradient(const Geom&, const Coef&, const double*, const double*, const double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_exp_cells(const Geom&, const double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_mg_taps(double*, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_mg_residual_restrict(const Geom&, const Geom&, const float* const[5], double* const[5], const double[4], const double* const[3][2], hipStream_t) { return hipSuccess; }
hipError_t launch_mg_coef_restrict(const Geom&, const Geom&, const double* const[4], double* const[4], const int[4], const double* const[3], hipStream_t) { return hipSuccess; }
hipError_t launch_mg_prolong_add(const Geom&, const Geom&, const double* const[5], double* const[5], hipStream_t) { return hipSuccess; }
bool mg_coarsest_fits(const Geom&) { return false; }
hipError_t launch_mg_coarsest(const Geom&, const Coef&, const SweepPtrs<double>&, double* const[5], int, hipStream_t) { return hipSuccess; }
hipError_t launch_kry_dots(const Geom&, const KryVecs&, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_kry_update(const Geom&, const KryVecs&, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_kry_save(const Geom&, const KryVecs&, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_porosity(const Geom&, const Coef&, const AdjPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_coef(const Geom&, const Coef&, const AdjPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_step(const Geom&, const Coef&, const AdjPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_history(const Geom&, const Coef&, const AdjPtrs&, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_oldvalues(const Geom&, const Coef&, const double*, const double*, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_absmax5(const Geom&, const double* const*, double* part, int64_t nb, hipStream_t s) {
    return fake::put(s, [=] { std::fill(part, part + nb * NNORM, 1.0); });
}
hipError_t launch_cell_max(const Geom&, const double*, double*, int64_t, hipStream_t) { return hipSuccess; }
}  // namespace ptk

namespace {

constexpr int NUP = 15;

// A handle of n^3 cells on a stream of its own, ready to solve.
struct Handle {
    pt_grid* g = nullptr;
    hipStream_t s;
    explicit Handle(int n, uintptr_t stream) : s(reinterpret_cast<hipStream_t>(stream)) {
        pt_params p{};
        p.version = PT_ABI_VERSION;
        p.lx = p.ly = p.lz = 1.0;
        p.phi0 = 0.1;
        p.kmuf0 = p.eta0 = p.mu0 = p.cmu = p.alpha = p.B = p.G = p.R0 = p.dt = p.dtS = p.rho_i = p.c_v = p.c_pf = 1.0;
        p.beta_d = p.tau0 = 1.0;
        p.nup = NUP;
        check(pt_create(n, n, n, (n + 32) / 32 * 32, &p, &g), "create");
        check(pt_set_stream(g, s), "stream");
        size_t bytes = 0;
        for (int f = 0; f < PT_NFIELDS; ++f)
            for (int c = 0; c < (f < PT_NPING ? 2 : 1); ++c) check(pt_bind_field(g, f, c, room(4096)), "field");
        check(pt_workspace_size(g, &bytes), "size");
        check(pt_bind_workspace(g, room(bytes), bytes), "workspace");
        check(pt_mixed_workspace_size(g, &bytes), "size");
        check(pt_bind_mixed_workspace(g, room(bytes), bytes), "workspace");
        hipStreamSynchronize(s);
    }
    double steps() const { return cur(g, PT_VX)[0]; }   // sweeps in the present copy
    static void* room(size_t bytes) {
        bytes = (bytes + 255) / 256 * 256;
        void* p = std::aligned_alloc(256, bytes);
        std::memset(p, 0, bytes);
        return p;
    }
    static void check(pt_status s, const char* what) {
        if (s != PT_OK) {
            std::fprintf(stderr, "%s: %d\n", what, (int)s);
            std::exit(2);
        }
    }
};

void say(const char* name, double v) { std::printf("%s %.17g\n", name, v); }

// A solve that ends at max_iter, between two checks; then another handle
// on another stream, whose partial maxima lie on the first one's gate.
void tail(bool fixed_scratch) {
    Handle a(8, 0x100), b(40, 0x200);
    auto solve = fixed_scratch ? pt_solve_linear_static : pt_solve_linear;
    int64_t it = 0;
    double rho = 0.0;
    say("covers", b.g->tiling.norms64 > a.g->tiling.most + 2);
    say("status_a", solve(a.g, 1e-300, NUP + 3, &it, &rho));
    say("iters_a", it);
    say("queued_a", fake::queued(a.s));
    say("status_b", solve(b.g, 1e-3, 1000, &it, &rho));
    say("iters_b", it);
    say("queued_b", fake::queued(b.s));
    hipStreamSynchronize(a.s);
    say("steps_a", a.steps());
    say("steps_b", b.steps());
}

// The transposed solve of the adjoints, stopped between two checks.
void tail_transposed() {
    Handle a(8, 0x100);
    size_t bytes = 0;
    Handle::check(pt_adjoint_workspace_size(a.g, 1, &bytes), "size");
    Handle::check(pt_bind_adjoint_workspace(a.g, Handle::room(bytes), bytes, 1), "workspace");
    int copy = 0;
    int64_t it = 0;
    double rho = 0.0;
    say("status", transposed_solve(a.g, cur(a.g, PT_KC), cur(a.g, PT_MUS), 1e-300, NUP + 3, &copy, &it, &rho));
    say("queued", fake::queued(a.s));
    say("iters", it);
    say("steps", ad(a.g, copy ? 8 : 0)[0]);
}

// A mixed solve whose first check finds a NaN.
void mixed_nan() {
    Handle a(8, 0x100);
    fake::poison = true;
    int64_t inner = 0;
    int32_t outer = 0;
    double rho = 0.0;
    say("status", pt_solve_mixed(a.g, 1e-8, 1e-2, 1000, 10, &inner, &outer, &rho));
    say("queued", fake::queued(a.s));
}

// Host memory that a handle's first solves ask for; refuse: and do not get.
void memory(bool refuse) {
    fake::refuse_mallocs = refuse;
    Handle a(8, 0x100), b(8, 0x200), c(8, 0x300);
    int64_t it = 0, inner = 0;
    int32_t outer = 0;
    double rho = 0.0;
    say("status_static", pt_solve_linear_static(a.g, 1e-12, 1000, &it, &rho));
    say("iters_static", it);
    say("rho_static", rho);
    say("steps_static", a.steps());
    say("queued_static", fake::queued(a.s));
    say("mallocs_static", fake::mallocs);
    say("status_linear", pt_solve_linear(b.g, 1e-12, 1000, &it, &rho));
    say("iters_linear", it);
    say("rho_linear", rho);
    say("steps_linear", b.steps());
    say("status_mixed", pt_solve_mixed(c.g, 1e-12, 1e-3, 1000, 10, &inner, &outer, &rho));
    say("inner_mixed", inner);
    say("outer_mixed", outer);
    say("mallocs", fake::mallocs);
}

// Handles that come and go while another stream is busy: one after the
// other, then many at once.
void destroy() {
    const hipStream_t busy = reinterpret_cast<hipStream_t>(0x900);
    fake::put(busy, [] {});
    int64_t it = 0;
    double rho = 0.0;
    bool solved = true;
    for (int q = 0; q < 10; ++q) {
        Handle a(8, 0x100);
        solved = solved && pt_solve_linear(a.g, 1e-12, 1000, &it, &rho) == PT_OK && it == 45 && a.steps() == 45;
        pt_destroy(a.g);
    }
    say("solved", solved);
    say("waited", fake::queued(busy) == 0);
    say("mallocs_in_turn", fake::mallocs);
    std::vector<Handle> many;
    for (int q = 0; q < 200; ++q) {
        many.emplace_back(8, 0x100 + 16 * (uintptr_t)q);
        solved = solved && pt_solve_linear(many.back().g, 1e-12, 1000, &it, &rho) == PT_OK && it == 45;
    }
    for (auto& h : many) pt_destroy(h.g);
    say("solved_many", solved);
    say("kept", fake::mallocs - fake::frees);
}

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "tail") tail(false);
    else if (what == "tail_static") tail(true);
    else if (what == "tail_transposed") tail_transposed();
    else if (what == "mixed_nan") mixed_nan();
    else if (what == "memory") memory(false);
    else if (what == "memory_refused") memory(true);
    else if (what == "destroy") destroy();
    else return 2;
    return 0;
}
