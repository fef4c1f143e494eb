// arc_api.hip -- host side of libarc: the C ABI of include/arc.h.
//
// Validation, fixed-point unit selection, buffer ownership and the two tracing
// schedules. Every per-cell and per-ray step runs in the kernels of arc_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "arc.h"
#include "arc_kernels.h"
#include "arc_mlp_host.h"

using namespace arc;

struct arc_ctx {
    int device = 0;
    int cus = 0;
    std::string err;
    // grid-sized buffers
    size_t ncell_cap = 0;
    void* kappa = nullptr;             // float or float4 per cell
    size_t kappa_bytes = 0;
    unsigned long long* J = nullptr;   // [tile][bin][8 cells]
    size_t J_bytes = 0;
    unsigned long long* M = nullptr;   // conserving correction: moved photons, [tile][2][bin][8]
    size_t M_bytes = 0;
    // source table
    SourceRec* src = nullptr;
    double* src_fill = nullptr;        // [5] per source: the thin fill's copy
    uint32_t* r_out = nullptr;         // measured R_tau<0.1 per source (FP32 bits)
    int src_cap = 0;
    double* src_stage = nullptr;       // the call's sources, pinned: SourceUpload
    uint32_t* r_stage = nullptr;       // r_out on the host, pinned
    // HEALPix centres, levels 0..dirs_levels-1
    float4* dirs = nullptr;
    int dirs_levels = 0;
    long long dir_off[kMaxLevels] = {0};
    // ray arrays (per-level schedule) and work queue (batched)
    RayRec* rays[2] = {nullptr, nullptr};
    size_t rcap[2] = {0, 0};   // records each ray buffer holds
    size_t item_bytes = 0;     // bound on the larger ray buffer of the batched schedule [bytes]
    RayRec* spill = nullptr;
    size_t spill_entries = 0;
    // small device scalars
    RunBlock* run = nullptr;
    // a call leaves these two as it wants to find them (zero; +inf), unless it failed on the way
    ChemBlock* chem_run = nullptr;
    unsigned long long* limits = nullptr;     // the time step's two minima
    bool chem_clean = false, limits_clean = false;
    struct Host {                             // pinned: written by the last kernel of a call
        RunResult run;
        ChemResult chem;
        double limits[2];
    };
    Host* host = nullptr;
    double clock_khz = 1e5;                   // of the device's stamps
    unsigned long long* reject = nullptr;     // learned step: cells for the plain solver, a bit each
    size_t reject_cap = 0;                    // words
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};  // request probes
    // last trace
    int last_nb = 0, last_nx = 0, last_ny = 0, last_nbx8 = 0, last_nby8 = 0;
    size_t last_ncell = 0;
    bool last_moved = false;  // the last trace filled M
    bool have_field = false;
    // the replayed launches of the batched schedule; valid while the launch arguments equal
    // graph_key
    hipStream_t cap_stream = nullptr;
    hipGraphExec_t gexec = nullptr;
    std::vector<unsigned char> graph_key;
    // the chemistry step's, same scheme
    hipGraphExec_t cexec = nullptr;
    std::vector<unsigned char> chem_key;
    unsigned long long* sums = nullptr;  // field checksums of the autotuner
    unsigned long long* static_scratch = nullptr;  // this device's copy of `scratch`
    struct Tuned {
        int nx, ny, nz, nb, level0, lmax, precision, corr, thin;  // (kernels differ by the last three)
        arc_tune_result shape;
    };
    std::vector<Tuned> tuned;
};

// A call's sources, n entries in pinned memory that the first kernel reads: positions, photon
// rates, thin radii, and the sources by decreasing photon rate (work-queue order).
struct SourceUpload {
    size_t pos, ndot, rthin, order, bytes;  // offsets [doubles], size
    explicit SourceUpload(size_t n) : pos(0), ndot(3 * n), rthin(4 * n), order(5 * n), bytes(44 * n) {}
};

// Scratch of the allocation-free entry point (arc_rt_timestep_noalloc): a file-scope device
// array, one copy per GPU, held until the process ends. Host code never passes its name to
// a kernel (on the host the name is a stand-in, not a device address): each context
// resolves the device's copy once, at creation, with hipGetSymbolAddress, and uses that.
constexpr int kStaticScratchWords = 32;  // 256 bytes
constexpr int kTimestepScratchWords = 2; // the two grid minima of section 2.9
static __device__ __align__(256) unsigned long long scratch[kStaticScratchWords];

namespace {

arc_status fail(arc_ctx* c, arc_status s, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    return s;
}

// (the runtime keeps a failed call's error until it is asked for: the next launch would report it)
#define HIP_TRY(ctx, expr)                                                                        \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) {                                                                   \
            (void)hipGetLastError();                                                              \
            return fail(ctx, e_ == hipErrorOutOfMemory ? ARC_E_NOMEM : ARC_E_DEVICE, "%s: %s (%s:%d)", \
                        #expr, hipGetErrorString(e_), __FILE__, __LINE__);                        \
        }                                                                                         \
    } while (0)

template <typename T>
hipError_t grow(T** p, size_t* cap_bytes, size_t need_bytes)
{
    if (*p && *cap_bytes >= need_bytes) return hipSuccess;
    if (*p) {
        hipError_t e = hipFree(*p);
        if (e != hipSuccess) return e;
        *p = nullptr;
        *cap_bytes = 0;
    }
    hipError_t e = hipMalloc((void**)p, need_bytes);
    if (e == hipSuccess) *cap_bytes = need_bytes;
    return e;
}

bool on_lattice(double v) { return std::isfinite(v) && std::floor(v * 4096.0) == v * 4096.0; }

// Split radius of each level, rounded once to float (pi r^2 / (3 4^l) = 1 / Phi).
float split_base(double phi) { return (float)std::sqrt(3.0 / (M_PI * phi)); }

int auto_max_level(int nx, int ny, int nz, double phi)
{
    const double diag = std::sqrt((double)nx * nx + (double)ny * ny + (double)nz * nz);
    const float base = split_base(phi);
    int l = 0;
    while ((double)std::ldexp(base, l) < diag && l < 40) ++l;
    return l;
}

arc_status check_grid(arc_ctx* c, const arc_grid* g)
{
    if (!g || !g->n_h || !g->x_hi || !g->x_hei || !g->x_heii) return fail(c, ARC_E_ARG, "null grid pointer");
    if (g->nx <= 0 || g->ny <= 0 || g->nz <= 0) return fail(c, ARC_E_ARG, "grid dimensions must be positive");
    if (g->nx > 2048 || g->ny > 2048 || g->nz > 2048)
        return fail(c, ARC_E_UNSUPPORTED, "grid dimensions above 2048 are not supported");
    const double ncell = (double)g->nx * g->ny * g->nz;
    if (ncell > 2147483647.0) return fail(c, ARC_E_UNSUPPORTED, "more than 2^31-1 cells");
    if (!(g->cell_cm > 0) || !std::isfinite(g->cell_cm)) return fail(c, ARC_E_RANGE, "cell_cm must be finite and > 0");
    if (!(g->y_he >= 0) || !std::isfinite(g->y_he)) return fail(c, ARC_E_RANGE, "y_he must be finite and >= 0");
    return ARC_OK;
}

arc_status check_bins(arc_ctx* c, const arc_freq_bins* b)
{
    if (!b || !b->frac || !b->e_erg || !b->sigma || !b->e_thr) return fail(c, ARC_E_ARG, "null bin pointer");
    if (b->nbins < 1 || b->nbins > kMaxBins) return fail(c, ARC_E_ARG, "nbins must be 1..4");
    double sum = 0;
    for (int k = 0; k < b->nbins; ++k) {
        if (!(b->frac[k] >= 0) || !std::isfinite(b->frac[k])) return fail(c, ARC_E_RANGE, "frac[%d] invalid", k);
        if (!(b->e_erg[k] > 0) || !std::isfinite(b->e_erg[k])) return fail(c, ARC_E_RANGE, "e_erg[%d] invalid", k);
        if (!(b->sigma[3 * k] > 0) || !std::isfinite(b->sigma[3 * k]))
            return fail(c, ARC_E_RANGE, "sigma_HI of bin %d must be > 0", k);
        for (int s = 1; s < 3; ++s)
            if (!(b->sigma[3 * k + s] >= 0) || !std::isfinite(b->sigma[3 * k + s]))
                return fail(c, ARC_E_RANGE, "sigma[%d][%d] invalid", k, s);
        sum += b->frac[k];
    }
    if (std::fabs(sum - 1.0) > 1e-6) return fail(c, ARC_E_RANGE, "bin fractions sum to %.9g, not 1", sum);
    for (int s = 0; s < 3; ++s)
        if (!(b->e_thr[s] > 0) || !std::isfinite(b->e_thr[s])) return fail(c, ARC_E_RANGE, "e_thr[%d] invalid", s);
    return ARC_OK;
}

arc_status check_sources(arc_ctx* c, const arc_sources* s, const arc_grid* g)
{
    if (!s) return fail(c, ARC_E_ARG, "null sources");
    if (s->n < 0) return fail(c, ARC_E_ARG, "negative source count");
    if (s->n > 0 && (!s->pos || !s->ndot)) return fail(c, ARC_E_ARG, "null source arrays");
    const int dims[3] = {g->nx, g->ny, g->nz};
    for (int i = 0; i < s->n; ++i) {
        for (int a = 0; a < 3; ++a) {
            const double v = s->pos[3 * i + a];
            if (!on_lattice(v)) return fail(c, ARC_E_RANGE, "source %d coordinate %d is not on the 2^-12 lattice", i, a);
            if (!(v >= 0.0 && v < (double)dims[a])) return fail(c, ARC_E_RANGE, "source %d lies outside the grid", i);
        }
        if (!(s->ndot[i] > 0) || !std::isfinite(s->ndot[i])) return fail(c, ARC_E_RANGE, "source %d ndot invalid", i);
    }
    return ARC_OK;
}

arc_status ensure_dirs(arc_ctx* c, int levels, hipStream_t st)
{
    if (levels <= c->dirs_levels) return ARC_OK;
    long long off[kMaxLevels];
    long long total = 0;
    for (int l = 0; l < levels; ++l) {
        off[l] = total;
        total += 12ll << (2 * l);
    }
    float4* nd = nullptr;
    HIP_TRY(c, hipMalloc((void**)&nd, (size_t)total * sizeof(float4)));
    for (int l = 0; l < levels; ++l) {
        hipError_t e = launch_healpix(l, nd + off[l], st);
        if (e != hipSuccess) {
            (void)hipFree(nd);
            return fail(c, ARC_E_DEVICE, "healpix launch: %s", hipGetErrorString(e));
        }
    }
    HIP_TRY(c, hipStreamSynchronize(st));
    if (c->dirs) HIP_TRY(c, hipFree(c->dirs));
    c->dirs = nd;
    c->dirs_levels = levels;
    for (int l = 0; l < levels; ++l) c->dir_off[l] = off[l];
    return ARC_OK;
}

}  // namespace

namespace arc {
int ctx_device(const arc_ctx* c) { return c->device; }
arc_status ctx_fail(arc_ctx* c, arc_status s, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    return s;
}
}  // namespace arc

extern "C" {

arc_status arc_create(int32_t device, arc_ctx** out)
{
    if (!out) return ARC_E_ARG;
    *out = nullptr;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return ARC_E_DEVICE;
    if (hipSetDevice(device) != hipSuccess) return ARC_E_DEVICE;
    arc_ctx* c = new (std::nothrow) arc_ctx();
    if (!c) return ARC_E_NOMEM;
    c->device = device;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
        delete c;
        return ARC_E_DEVICE;
    }
    c->cus = prop.multiProcessorCount;
    c->item_bytes = prop.totalGlobalMem / 6;
    // this device's copy of the static scratch (the device is current)
    if (hipGetSymbolAddress((void**)&c->static_scratch, HIP_SYMBOL(scratch)) != hipSuccess || !c->static_scratch) {
        delete c;
        return ARC_E_DEVICE;
    }
    bool ok = hipMalloc((void**)&c->run, sizeof(RunBlock)) == hipSuccess &&
              hipHostMalloc((void**)&c->host, sizeof(arc_ctx::Host), hipHostMallocDefault) == hipSuccess &&
              hipMalloc((void**)&c->limits, 2 * sizeof(unsigned long long)) == hipSuccess &&
              hipMalloc((void**)&c->chem_run, sizeof(ChemBlock)) == hipSuccess &&
              hipMalloc((void**)&c->sums, 2 * sizeof(unsigned long long)) == hipSuccess;
    for (int i = 0; i < 3 && ok; ++i) ok = hipEventCreate(&c->ev[i]) == hipSuccess;
    if (!ok) {
        arc_destroy(c);
        return ARC_E_NOMEM;
    }
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device) == hipSuccess && khz > 0) c->clock_khz = khz;
    *out = c;
    return ARC_OK;
}

void arc_destroy(arc_ctx* c)
{
    if (!c) return;
    (void)hipSetDevice(c->device);
    void* bufs[] = {c->kappa, c->J, c->M, c->src, c->src_fill, c->r_out, c->dirs, c->rays[0], c->rays[1], c->spill,
                    c->run, c->chem_run, c->limits, c->reject};
    for (void* p : bufs)
        if (p) (void)hipFree(p);
    void* pinned[] = {c->src_stage, c->r_stage, c->host};
    for (void* p : pinned)
        if (p) (void)hipHostFree(p);
    for (int i = 0; i < 3; ++i)
        if (c->ev[i]) (void)hipEventDestroy(c->ev[i]);
    if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
    if (c->cexec) (void)hipGraphExecDestroy(c->cexec);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    if (c->sums) (void)hipFree(c->sums);
    delete c;
}

const char* arc_last_error(const arc_ctx* c) { return c ? c->err.c_str() : "null context"; }

}  // extern "C"

namespace {

// Everything one trace launches with. Zero-filled before use so that its bytes (padding
// included) can serve as the key of the recorded graphs.
struct TracePlan {
    int nb, lmax;
    size_t ncell;
    int nbx8, nby8, nbz8;
    double uj[kMaxBins];
    double sum_ndot;
    int nsrc;
    BeginArgs ba;
    OpacityArgs oa;
    TraceArgs A;
    FinalizeArgs fa;
    ThinFillArgs tf;
    int thin;        // optically thin approximation in use (section 2.6)
    int precision;
    // batched schedule
    int waves, blocks, refill, litem;
    int stack;          // split rays per wave's LDS stack
    int spill_cap_req;  // records of each wave's spill area (0: 4096)
    double n_roots;
    size_t cap[2];  // records of rays0 / rays1
    uint32_t spill_cap;
    RayRec* rays0;
    RayRec* rays1;
    RayRec* spill;
    RunBlock* run;
    RunResult* result;
    uint32_t* r_host;   // pinned: where the measured thin radii go, or null
};

// Validation, fixed-point units, buffers and launch arguments shared by both schedules.
arc_status plan_trace(arc_ctx* c, const arc_grid* g, const arc_sources* s, const arc_freq_bins* b, double dt,
                      const arc_trace_params* p, const arc_rates* out, TracePlan& P)
{
    std::memset(&P, 0, sizeof P);
    arc_status rc;
    if ((rc = check_grid(c, g)) != ARC_OK) return rc;
    if ((rc = check_bins(c, b)) != ARC_OK) return rc;
    if ((rc = check_sources(c, s, g)) != ARC_OK) return rc;
    if (!p) return fail(c, ARC_E_ARG, "null params");
    if (!out || !out->gamma || !out->heat) return fail(c, ARC_E_ARG, "null rate outputs");
    if (!(dt > 0) || !std::isfinite(dt)) return fail(c, ARC_E_RANGE, "dt must be finite and > 0");
    if (!(p->rays_per_cell > 0) || !std::isfinite(p->rays_per_cell)) return fail(c, ARC_E_RANGE, "rays_per_cell must be > 0");
    if (!(p->eps_term >= 0 && p->eps_term < 1)) return fail(c, ARC_E_RANGE, "eps_term must be in [0,1)");
    if (p->precision != ARC_PREC_FP32_COMP && p->precision != ARC_PREC_FP32_PLAIN) return fail(c, ARC_E_ARG, "bad precision");
    if (p->schedule != ARC_SCHED_PLAIN && p->schedule != ARC_SCHED_BATCHED && p->schedule != ARC_SCHED_BATCHED_TUNED)
        return fail(c, ARC_E_ARG, "bad schedule");
    const int lmax = p->max_level < 0 ? auto_max_level(g->nx, g->ny, g->nz, p->rays_per_cell) : p->max_level;
    if (p->level0 < 0 || p->level0 > lmax) return fail(c, ARC_E_ARG, "level0 must be in [0, max_level]");
    if (lmax > 12) return fail(c, ARC_E_UNSUPPORTED, "max_level %d > 12 (pixel ids are 28-bit)", lmax);
    if (!(p->u_j_override >= 0)) return fail(c, ARC_E_ARG, "u_j_override must be >= 0");
    if (p->tree_out && p->tree_cap < 0) return fail(c, ARC_E_ARG, "tree_cap < 0");
    if (p->correction < ARC_CORR_NONE || p->correction > ARC_CORR_FC_SQUARED)
        return fail(c, ARC_E_ARG, "bad correction mode %d", p->correction);
    if (p->correction != ARC_CORR_NONE && p->precision != ARC_PREC_FP32_COMP)
        return fail(c, ARC_E_UNSUPPORTED, "the geometric correction needs ARC_PREC_FP32_COMP");
    if (p->spill_cap < 0) return fail(c, ARC_E_ARG, "spill_cap must be >= 0");
    if (p->tune_stack != 0 && p->tune_stack != 64 && p->tune_stack != 128 && p->tune_stack != 256)
        return fail(c, ARC_E_ARG, "tune_stack must be 0, 64, 128 or 256");
    // optically thin approximation (section 2.6): per-source start radii and/or the measured
    // R_tau<0.1
    bool thin = s->r_thin_out != nullptr;
    double max_r = 0.0;
    if (s->r_thin)
        for (int i = 0; i < s->n; ++i) {
            const double r = s->r_thin[i];
            if (!(r >= 0.0) || !(r < 1048576.0))
                return fail(c, ARC_E_RANGE, "r_thin[%d] must be finite, >= 0 and below 2^20 cells", i);
            thin = thin || r > 0.0;
            max_r = std::max(max_r, (double)(float)r);
        }
    if (thin && p->precision != ARC_PREC_FP32_COMP)
        return fail(c, ARC_E_UNSUPPORTED, "the optically thin approximation needs ARC_PREC_FP32_COMP");

    hipStream_t st = (hipStream_t)p->stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const int nb = b->nbins;
    const size_t ncell = (size_t)g->nx * g->ny * g->nz;
    const int nbx8 = (g->nx + 7) / 8, nby8 = (g->ny + 7) / 8, nbz8 = (g->nz + 7) / 8;
    const size_t nblocked = (size_t)nbx8 * nby8 * nbz8 * 512;  // cells of the blocked layout
    if (nblocked > 2147483648ull) return fail(c, ARC_E_UNSUPPORTED, "blocked grid exceeds 2^31 cells");
    P.nb = nb;
    P.lmax = lmax;
    P.ncell = ncell;
    P.nbx8 = nbx8;
    P.nby8 = nby8;
    P.nbz8 = nbz8;
    P.nsrc = s->n;
    P.precision = p->precision;
    P.thin = thin ? 1 : 0;
    P.spill_cap_req = p->spill_cap;

    // Fixed-point unit per bin. One source deposits at most sqrt(3) S_b into a cell
    // (the photon rate through any sphere is at most S_b and a cell is at most sqrt(3)
    // long), plus a remainder below eps_term S_b sqrt(3) / 0.01 on termination, plus with
    // the optically thin fill at most S_b / pi (r >= 1/2). The sum over sources therefore
    // stays below 2^62 units. With the conserving correction a cell also receives into its
    // field at most half of each of its six neighbours' deposits times the opacity ratio
    // kMovedRatioJ: 1 + 6 * 16 / 2 = 49 times the bound (larger ratios move photons into the
    // moved-photon field, counted in the same unit: all of them together are at most the
    // photons emitted).
    for (int k = 0; k < kMaxBins; ++k) P.uj[k] = 1.0;
    for (int i = 0; i < s->n; ++i) P.sum_ndot += s->ndot[i];
    const double corr_factor = p->correction == ARC_CORR_CONSERVING ? 1.0 + 6.0 * (double)kMovedRatioJ / 2.0 : 1.0;
    for (int k = 0; k < nb; ++k) {
        const double bound = (std::sqrt(3.0) + p->eps_term * std::sqrt(3.0) / (double)kDtauTermMin +
                              (thin ? 1.0 / M_PI : 0.0)) *
                             P.sum_ndot * b->frac[k] * (1.0 + 1e-6) * corr_factor;
        const double need = bound / 4611686018427387904.0;  // 2^62
        if (p->u_j_override > 0) {
            if (p->u_j_override < need)
                return fail(c, ARC_E_OVERFLOW, "fixed-point unit %.6g too small for bin %d (needs >= %.6g)",
                            p->u_j_override, k, need);
            P.uj[k] = p->u_j_override;
        } else {
            P.uj[k] = need > 0 ? need : 1.0;
        }
        P.ba.scale[k] = b->frac[k] / (12.0 * P.uj[k]);
    }

    // Buffers.
    {
        const size_t kb = nblocked * (nb == 1 ? sizeof(float) : sizeof(float4));
        HIP_TRY(c, grow(&c->kappa, &c->kappa_bytes, kb));
        const size_t jb = nblocked * nb * sizeof(unsigned long long);
        const size_t mb = p->correction == ARC_CORR_CONSERVING ? 2 * jb : 0;
        if (jb > c->J_bytes || mb > c->M_bytes) c->have_field = false;
        HIP_TRY(c, grow(&c->J, &c->J_bytes, jb));
        if (mb) HIP_TRY(c, grow(&c->M, &c->M_bytes, mb));
        if (s->n > c->src_cap) {
            void* old[] = {c->src, c->src_fill, c->r_out};
            void* old_pinned[] = {c->src_stage, c->r_stage};
            c->src = nullptr;
            c->src_fill = c->src_stage = nullptr;
            c->r_out = c->r_stage = nullptr;
            c->src_cap = 0;
            for (void* q : old)
                if (q) HIP_TRY(c, hipFree(q));
            for (void* q : old_pinned)
                if (q) HIP_TRY(c, hipHostFree(q));
            const SourceUpload up((size_t)s->n);
            HIP_TRY(c, hipMalloc((void**)&c->src, s->n * sizeof(SourceRec)));
            HIP_TRY(c, hipMalloc((void**)&c->src_fill, s->n * 5 * sizeof(double)));
            HIP_TRY(c, hipMalloc((void**)&c->r_out, s->n * sizeof(uint32_t)));
            HIP_TRY(c, hipHostMalloc((void**)&c->src_stage, up.bytes, hipHostMallocDefault));
            HIP_TRY(c, hipHostMalloc((void**)&c->r_stage, s->n * sizeof(uint32_t), hipHostMallocDefault));
            c->src_cap = s->n;
        }
    }
    if ((rc = ensure_dirs(c, lmax + 1, st)) != ARC_OK) return rc;

    P.run = c->run;
    P.result = &c->host->run;
    P.r_host = thin && s->r_thin_out && s->n > 0 ? c->r_stage : nullptr;
    BeginArgs& ba = P.ba;
    const SourceUpload up((size_t)s->n);
    ba.run = c->run;
    ba.nb = nb;
    ba.nsrc = s->n;
    ba.level0 = p->level0;
    if (s->n > 0) {
        ba.pos = c->src_stage + up.pos;
        ba.ndot = c->src_stage + up.ndot;
        ba.r_thin = thin && s->r_thin ? c->src_stage + up.rthin : nullptr;
        ba.fill = thin ? c->src_fill : nullptr;
        ba.order = reinterpret_cast<const uint32_t*>(c->src_stage + up.order);
    }
    ba.src = c->src;
    ba.r_out = thin ? c->r_out : nullptr;

    OpacityArgs& oa = P.oa;
    oa.nb = nb;
    oa.nx = g->nx;
    oa.ny = g->ny;
    oa.nz = g->nz;
    oa.nbx8 = nbx8;
    oa.nby8 = nby8;
    oa.nbz8 = nbz8;
    oa.ncell = (uint32_t)ncell;
    oa.L = g->cell_cm;
    oa.y = g->y_he;
    for (int k = 0; k < nb; ++k)
        for (int sp = 0; sp < 3; ++sp) oa.sigma[k][sp] = b->sigma[3 * k + sp];
    oa.n_h = g->n_h;
    oa.x_hi = g->x_hi;
    oa.x_hei = g->x_hei;
    oa.x_heii = g->x_heii;
    oa.kappa1 = nb == 1 ? (float*)c->kappa : nullptr;
    oa.kappa4 = nb == 1 ? nullptr : (float4*)c->kappa;
    oa.J = c->J;
    oa.M = p->correction == ARC_CORR_CONSERVING ? c->M : nullptr;
    oa.errflag = &c->run->errflag;

    TraceArgs& A = P.A;
    A.nx = g->nx;
    A.ny = g->ny;
    A.nz = g->nz;
    A.nb = nb;
    A.nbx8 = nbx8;
    A.nby8 = nby8;
    A.level0 = p->level0;
    A.lmax = lmax;
    const float base = split_base(p->rays_per_cell);
    for (int l = 0; l < kMaxLevels; ++l) A.tsplit[l] = l < lmax ? std::ldexp(base, l) : INFINITY;
    A.tau_term = p->eps_term > 0 ? (float)(-std::log(p->eps_term)) : INFINITY;
    A.kappa1 = oa.kappa1;
    A.kappa4 = oa.kappa4;
    A.J = c->J;
    A.src = c->src;
    A.dirs = c->dirs;
    for (int l = 0; l < kMaxLevels; ++l) A.dir_off[l] = l < c->dirs_levels ? c->dir_off[l] : 0;
    A.slots = c->run->before;
    A.tree = (unsigned long long*)p->tree_out;
    A.tree_count = &c->run->tree_count;
    A.tree_cap = p->tree_out ? p->tree_cap : 0;
    A.corr = p->correction;
    A.M = oa.M;
    // softest bin: the lowest photon energy (the first of equal ones)
    A.ksoft = 0;
    for (int k = 1; k < nb; ++k)
        if (b->e_erg[k] < b->e_erg[A.ksoft]) A.ksoft = k;
    A.r_out = thin ? c->r_out : nullptr;

    FinalizeArgs& fa = P.fa;
    fa.nb = nb;
    fa.nx = g->nx;
    fa.ny = g->ny;
    fa.nz = g->nz;
    fa.nbx8 = nbx8;
    fa.nby8 = nby8;
    fa.nbz8 = nbz8;
    fa.ncell = (uint32_t)ncell;
    const double L2 = g->cell_cm * g->cell_cm;
    for (int k = 0; k < nb; ++k) {
        fa.uj[k] = P.uj[k];
        for (int sp = 0; sp < 3; ++sp) {
            fa.gam[k][sp] = P.uj[k] * b->sigma[3 * k + sp] / L2;
            const double excess = b->e_erg[k] - b->e_thr[sp];
            fa.hea[k][sp] = excess > 0 ? P.uj[k] * b->sigma[3 * k + sp] * excess / L2 : 0.0;
        }
    }
    fa.J = c->J;
    fa.M = oa.M;
    fa.kappa1 = oa.kappa1;
    fa.kappa4 = oa.kappa4;
    fa.gamma = out->gamma;
    fa.heat = out->heat;
    fa.slots = c->run->before;
    fa.stamp = &c->run->stamp[kStampRates];

    if (thin) {
        ThinFillArgs& tf = P.tf;
        tf.nb = nb;
        tf.nsrc = s->r_thin && max_r > 0.0 ? s->n : 0;
        // blocks per source: about 8192 cells of the largest bounding box each, a power of two
        const double box = std::pow(2.0 * max_r + 2.0, 3.0);
        int parts = 1;
        while (parts < 1024 && (double)parts * 8192.0 < box) parts *= 2;
        tf.parts = parts;
        tf.nx = g->nx;
        tf.ny = g->ny;
        tf.nz = g->nz;
        tf.nbx8 = nbx8;
        tf.nby8 = nby8;
        tf.src = ba.fill;
        for (int k = 0; k < nb; ++k) {
            tf.coef[k] = b->frac[k] / (4.0 * M_PI * P.uj[k]);
            tf.uj[k] = P.uj[k];
        }
        tf.J = c->J;
        tf.kappa1 = oa.kappa1;
        tf.kappa4 = oa.kappa4;
        tf.slots = c->run->before;
    }
    return ARC_OK;
}

// Default work-item level: five levels below the first. The levels above it are traced
// level by level (all rays of a level in one launch, no stacks); below it a subtree is
// small enough for its wave's LDS stack, so rays seldom spill to memory (1024^3 x 16384
// sources: item level 4 -> 6 took the persistent launch from 1440 to 990 ms and the spills
// from 1.4e8 to 4e5). Lowered while the larger ray buffer would exceed item_bytes.
constexpr int kDefaultItemDepth = 5;

// From level 0, level 6 instead of 5 for 4 to 512 sources, in boxes that do not reach level 8 (up
// to 36^3 with four rays per cell) for 4 to 64: it gives more waves items, which few sources lack at
// level 5; with more of them the rays traced level by level cost more than that gives. Level 5 and
// 6 [ms], gas of the density-field test:
//   32^3   1 source 0.153, 0.161; 4: 0.196, 0.194; 32: 0.598, 0.369; 128: 0.838, 0.974; 512: 2.15, 3.16
//   64^3   1: 0.206, 0.211; 4: 0.341, 0.326; 32: 1.13, 0.70; 512: 7.29, 7.20; 2048: 26.2, 27.1
//   192^3  1: 0.411, 0.426; 4: 0.559, 0.573; 32: 1.83, 1.38; 512: 14.7, 14.0
// Thin gas gains more (64^3 x 32 4.22, 1.78; 256^3 x 4 50.8, 51.3, x 32 301, 104); in thick gas, where
// hardly a ray gets that far, the launch costs 1 to 5 us of 90 to 560.
constexpr int kDeeperSources = 4, kDeeperSourcesEnd = 512, kDeeperSourcesEndSmall = 64;

// Default refill threshold of the persistent launch: a wave refills once 48 of its lanes are
// idle, so that many rays, mostly children of the same splits, start together and share the
// tiles of their deposits; one of the thresholds the autotuner tries. Refill at 32, 40, 48 and 56 idle
// lanes: 256^3 x 1024 sources 27.1, 26.1, 26.0 and 26.3 ms, 128^3 x 64 1.58, 1.50, 1.47 and 1.49,
// 203x100x37 x 200 3.44, 3.21, 3.10 and 3.09; where idle lanes cost more the lower ones are level or
// ahead by 1%: 128^3 x 16 0.70, 0.70, 0.72 and 0.72, corrected 192^3 x 128 7.87, 7.95, 8.02 and 8.11.
constexpr int kDefaultRefill = 48;

// Default depth of each wave's LDS stack: 64 split rays (2 KB), a full split round of the
// wave; deeper stacks spill less but hold fewer waves per compute unit.
constexpr int kDefaultStack = 64;

// Default grid of the persistent launch: the workgroups that are resident at once. Their first work
// items are theirs by their place in the grid, so a wave that has to wait for another's end would
// start its items late (128^3 x 16 sources, three waves per SIMD: 768 workgroups of four waves
// 0.53 ms, 1024 0.63 ms; where the LDS holds three workgroups, three per compute unit and four:
// 2048x2048x32 x 16 sources, long tables of index terms, 0.50 and 0.56, 128^3 x 16 with stacks of
// 256 records 0.64 and 0.70).
int default_workgroups_per_cu(const TracePlan& P, int waves, int stack)
{
    return persistent_workgroups_per_cu(P.nb, P.A.nx + P.A.ny + P.A.nz, waves, stack);
}

// Records of a ray buffer, without keeping its contents.
hipError_t grow_rays(arc_ctx* c, int i, size_t n)
{
    size_t bytes = c->rcap[i] * sizeof(RayRec);
    const hipError_t e = grow(&c->rays[i], &bytes, n * sizeof(RayRec));
    c->rcap[i] = bytes / sizeof(RayRec);
    return e;
}

// Work-item level of the default shape, before shape_batched's bounds.
int default_item_level(const TracePlan& P)
{
    const int litem = P.A.level0 + kDefaultItemDepth;
    const bool deeper = P.nsrc >= kDeeperSources && P.nsrc <= (P.lmax >= 8 ? kDeeperSourcesEnd : kDeeperSourcesEndSmall);
    return litem < 6 && deeper ? 6 : litem;
}

// Launch shape of the batched schedule and the buffers it needs. item_level: the HEALPix
// level whose rays are the persistent launch's work items (0: the default depth); it is
// clamped to [level0, lmax] and to the memory bound.
arc_status shape_batched(arc_ctx* c, TracePlan& P, int waves, int blocks, int refill, int item_level, int stack)
{
    if (stack != 64 && stack != 128 && stack != 256) return fail(c, ARC_E_ARG, "LDS stack depth must be 64, 128 or 256");
    if (waves != 1 && waves != 2 && waves != 4 && waves != 8) return fail(c, ARC_E_ARG, "tune_waves must be 1, 2, 4 or 8");
    if (blocks < 1) return fail(c, ARC_E_ARG, "tune_blocks must be >= 1");
    const int level0 = P.A.level0, lmax = P.lmax;
    const uint32_t npix0 = 12u << (2 * level0);
    const double n_roots = (double)P.nsrc * npix0;
    // rays of level l at most (every ray reaches it)
    auto rays_at = [&](int l) { return n_roots * std::ldexp(1.0, 2 * (l - level0)); };
    int litem = item_level > 0 ? item_level : default_item_level(P);
    litem = std::max(level0, std::min(lmax, litem));
    while (litem > level0 &&
           (rays_at(litem) > (double)0xFFFFFFF0u || rays_at(litem) * sizeof(RayRec) > (double)c->item_bytes))
        --litem;
    if (rays_at(litem) > (double)0xFFFFFFF0u) return fail(c, ARC_E_UNSUPPORTED, "too many work items");
    // buffer b holds the levels l with (l - level0) % 2 == b: the count of its deepest one. The
    // items of litem are families, a record per ray of the level before (else the root rays)
    size_t need[2] = {1, 1};
    for (int l = level0; l <= litem; ++l)
        need[(l - level0) & 1] = std::max(need[(l - level0) & 1], (size_t)rays_at(l < litem ? l : std::max(level0, l - 1)));
    for (int i = 0; i < 2; ++i)
        if (need[i] > c->rcap[i]) HIP_TRY(c, grow_rays(c, i, need[i]));
    const uint32_t spill_cap = P.spill_cap_req > 0 ? (uint32_t)P.spill_cap_req : 4096u;
    const size_t spill_need = (size_t)blocks * waves * spill_cap;
    if (spill_need > c->spill_entries) {
        size_t cap_bytes = c->spill_entries * sizeof(RayRec);
        const hipError_t e = grow(&c->spill, &cap_bytes, spill_need * sizeof(RayRec));
        c->spill_entries = cap_bytes / sizeof(RayRec);  // none where the allocation failed
        HIP_TRY(c, e);
    }
    P.waves = waves;
    P.blocks = blocks;
    P.refill = std::max(1, std::min(64, refill));
    P.stack = stack;
    P.litem = litem;
    P.n_roots = n_roots;
    P.cap[0] = c->rcap[0];
    P.cap[1] = c->rcap[1];
    P.spill_cap = spill_cap;
    P.rays0 = c->rays[0];
    P.rays1 = c->rays[1];
    P.spill = c->spill;
    P.ba.n_roots = (uint32_t)n_roots;
    P.ba.roots = P.nsrc > 0 ? c->rays[0] : nullptr;
    return ARC_OK;
}

// Stage 0: counters, source table and root rays, opacity (section 2.2 cross sections times
// densities).
hipError_t enqueue_common(const TracePlan& P, hipStream_t st)
{
    hipError_t e;
    if ((e = launch_begin(P.ba, st)) != hipSuccess) return e;
    if ((e = launch_opacity(P.oa, st)) != hipSuccess) return e;
    return P.thin ? launch_thin_fill(P.tf, st) : hipSuccess;
}

// Stage 1 (batched): the levels traced level by level before the persistent launch.
hipError_t enqueue_levels(const TracePlan& P, hipStream_t st)
{
    if (P.nsrc == 0) return hipSuccess;
    size_t bound = (size_t)P.n_roots;
    int cur = 0;
    RayRec* r[2] = {P.rays0, P.rays1};
    for (int l = P.A.level0; l < P.litem; ++l) {
        const uint32_t out_cap = (uint32_t)std::min<size_t>(P.cap[1 - cur], 0xFFFFFFF0u);
        // the last level leaves family records: the work items of the persistent launch
        const int fam_out = l + 1 == P.litem ? 1 : 0;
        TraceArgs A = P.A;
        A.stamp = l == P.A.level0 ? &P.run->stamp[kStampTrace] : nullptr;
        const hipError_t e = launch_trace_rays(A, P.precision, r[cur], &P.run->level_rays[l].n, (uint32_t)bound,
                                               r[1 - cur], &P.run->level_rays[l + 1].n, out_cap, fam_out, st);
        if (e != hipSuccess) return e;
        bound *= 4;
        cur = 1 - cur;
    }
    return hipSuccess;
}

// Stage 2: the persistent launch over the work items of level litem.
hipError_t enqueue_persistent(const TracePlan& P, hipStream_t st)
{
    if (P.nsrc == 0) return hipSuccess;
    const int cur = (P.litem - P.A.level0) & 1;
    // above the first level the work items are the family records of the level before
    const int fam = P.litem > P.A.level0 ? 1 : 0;
    TraceArgs A = P.A;
    A.slots = P.run->persistent;
    A.stamp = &P.run->stamp[kStampPersistent];
    return launch_trace_persistent(A, P.precision, cur ? P.rays1 : P.rays0, &P.run->level_rays[P.litem].n, &P.run->head.n,
                                   P.spill, P.spill_cap, P.blocks, P.waves, P.refill, fam, P.stack, st);
}

// Stage 3: rates (eq:ion per absorber, section 2.8 heating) and the absorbed ledger; then the
// call's counters to the host.
hipError_t enqueue_rates(const TracePlan& P, hipStream_t st)
{
    const hipError_t e = launch_finalize(P.fa, st);
    return e != hipSuccess ? e : launch_end(P.run, P.result, P.A.r_out, P.r_host, P.nsrc, st);
}

// The whole batched call.
hipError_t enqueue_batched(const TracePlan& P, hipStream_t st)
{
    hipError_t e;
    if ((e = enqueue_common(P, st)) != hipSuccess) return e;
    if ((e = enqueue_levels(P, st)) != hipSuccess) return e;
    if ((e = enqueue_persistent(P, st)) != hipSuccess) return e;
    return enqueue_rates(P, st);
}

// Section 2.1 iii: one source at a time, one HEALPix level per launch; the host reads
// back the number of children before launching the next level.
arc_status run_plain(arc_ctx* c, const TracePlan& P, hipStream_t st)
{
    const uint32_t npix0 = 12u << (2 * P.A.level0);
    uint32_t* n_out = &c->run->level_rays[kMaxLevels - 1].n;
    bool first = true;
    for (int si = 0; si < P.nsrc; ++si) {
        size_t n = npix0;
        for (int i = 0; i < 2; ++i)
            if (4 * n > c->rcap[i]) HIP_TRY(c, grow_rays(c, i, 4 * n));
        HIP_TRY(c, launch_seed_roots((uint32_t)si, P.A.level0, c->rays[0], st));
        int cur = 0;
        while (n > 0) {
            const size_t need = 4 * n;
            if (need > std::min(c->rcap[0], c->rcap[1])) {
                // grow both arrays, keeping the current level's rays
                RayRec* a = nullptr;
                RayRec* bb = nullptr;
                HIP_TRY(c, hipStreamSynchronize(st));
                HIP_TRY(c, hipMalloc((void**)&a, need * sizeof(RayRec)));
                HIP_TRY(c, hipMalloc((void**)&bb, need * sizeof(RayRec)));
                HIP_TRY(c, hipMemcpyAsync(a, c->rays[cur], n * sizeof(RayRec), hipMemcpyDeviceToDevice, st));
                HIP_TRY(c, hipStreamSynchronize(st));
                HIP_TRY(c, hipFree(c->rays[0]));
                HIP_TRY(c, hipFree(c->rays[1]));
                c->rays[0] = a;
                c->rays[1] = bb;
                cur = 0;
                c->rcap[0] = c->rcap[1] = need;
            }
            HIP_TRY(c, launch_set_u32(n_out, 0u, st));
            TraceArgs A = P.A;
            A.stamp = first ? &c->run->stamp[kStampTrace] : nullptr;
            first = false;
            HIP_TRY(c, launch_trace_rays(A, P.precision, c->rays[cur], nullptr, (uint32_t)n, c->rays[1 - cur], n_out,
                                         (uint32_t)std::min<size_t>(c->rcap[1 - cur], 0xFFFFFFF0u), 0, st));
            uint32_t nn = 0;
            HIP_TRY(c, hipMemcpyAsync(&nn, n_out, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
            HIP_TRY(c, hipStreamSynchronize(st));
            n = nn;
            cur = 1 - cur;
        }
    }
    return ARC_OK;
}

// Records what `enqueue` launches as a graph (on the context's own capture stream) into *exec,
// unless the recorded one was made with the same `size` bytes at `args`.
template <class F>
arc_status ensure_graph(arc_ctx* c, hipGraphExec_t* exec, std::vector<unsigned char>& key, const void* args, size_t size,
                        const char* what, F enqueue)
{
    const unsigned char* bytes = static_cast<const unsigned char*>(args);
    if (*exec && key.size() == size && std::memcmp(key.data(), bytes, size) == 0) return ARC_OK;
    if (*exec) {
        HIP_TRY(c, hipGraphExecDestroy(*exec));
        *exec = nullptr;
    }
    key.clear();
    if (!c->cap_stream) HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    HIP_TRY(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
    const hipError_t e = enqueue(c->cap_stream);
    hipGraph_t graph = nullptr;
    const hipError_t e2 = hipStreamEndCapture(c->cap_stream, &graph);
    if (e != hipSuccess || e2 != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        return fail(c, ARC_E_DEVICE, "graph capture of %s: %s", what, hipGetErrorString(e != hipSuccess ? e : e2));
    }
    const hipError_t e3 = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e3 != hipSuccess) {
        *exec = nullptr;
        return fail(c, ARC_E_DEVICE, "graph instantiation of %s: %s", what, hipGetErrorString(e3));
    }
    key.assign(bytes, bytes + size);
    return ARC_OK;
}

// One whole trace with a planned shape: the sources into pinned memory, the stages (eagerly or
// as a graph), and the counters, ledger and error flags that the last kernel leaves there.
arc_status run_trace(arc_ctx* c, const TracePlan& P, const arc_sources* s, double dt, int schedule, bool graph,
                     hipStream_t st, arc_ledger* ledger)
{
    const bool batched = schedule != ARC_SCHED_PLAIN;
    c->have_field = false;  // until this one's is whole
    if (s->n > 0) {
        const size_t n = (size_t)s->n;
        const SourceUpload up(n);
        std::memcpy(c->src_stage + up.pos, s->pos, 3 * n * sizeof(double));
        std::memcpy(c->src_stage + up.ndot, s->ndot, n * sizeof(double));
        if (s->r_thin) std::memcpy(c->src_stage + up.rthin, s->r_thin, n * sizeof(double));
        if (batched) {
            // the work queue starts with the brightest sources, whose rays travel furthest, so
            // that the longest subtrees are not the last ones taken (the field does not depend
            // on the order: integer sums)
            uint32_t* order = reinterpret_cast<uint32_t*>(c->src_stage + up.order);
            for (size_t i = 0; i < n; ++i) order[i] = (uint32_t)i;
            std::stable_sort(order, order + n, [&](uint32_t a, uint32_t b2) { return s->ndot[a] > s->ndot[b2]; });
        }
    }
    if (batched && graph) {
        arc_status rc = ensure_graph(c, &c->gexec, c->graph_key, &P, sizeof P, "the trace",
                                     [&](hipStream_t cs) { return enqueue_batched(P, cs); });
        if (rc != ARC_OK) return rc;
        HIP_TRY(c, hipGraphLaunch(c->gexec, st));
    } else if (batched) {
        HIP_TRY(c, enqueue_batched(P, st));
    } else {
        HIP_TRY(c, enqueue_common(P, st));
        arc_status rc = run_plain(c, P, st);
        if (rc != ARC_OK) {
            (void)hipStreamSynchronize(st);  // nothing reads the pinned buffers any more
            return rc;
        }
        HIP_TRY(c, enqueue_rates(P, st));
    }
    HIP_TRY(c, hipStreamSynchronize(st));
    for (int i = 0; P.r_host && i < s->n; ++i) {
        float r;
        std::memcpy(&r, &c->r_stage[i], sizeof r);
        s->r_thin_out[i] = (double)r;
    }
    const RunResult& run = c->host->run;
    const unsigned long long *cnt = run.n, *per = run.persistent;
    const double* acc = run.photons;
    auto ms_between = [&](int a, int b2) { return (double)(run.stamp[b2] - run.stamp[a]) / c->clock_khz; };

    c->last_nb = P.nb;
    c->last_ncell = P.ncell;
    c->last_nx = P.A.nx;
    c->last_ny = P.A.ny;
    c->last_nbx8 = P.nbx8;
    c->last_nby8 = P.nby8;
    c->last_moved = P.A.M != nullptr;
    c->have_field = true;
    if (run.errflag) return fail(c, ARC_E_RANGE, "grid values out of range (n_h <= 0, fraction outside [0,1] or non-finite)");
    if (cnt[kQueueOverflow]) return fail(c, ARC_E_QUEUE, "ray queue capacity exceeded (%llu rays dropped)", cnt[kQueueOverflow]);
    if (ledger) {
        std::memset(ledger, 0, sizeof *ledger);
        ledger->emitted = P.sum_ndot * dt;
        double esc = 0;
        for (int k = 0; k < P.nb; ++k) esc += acc[kPhotonsEscaped + k] * P.uj[k];
        ledger->escaped = esc * dt;
        ledger->absorbed = acc[kPhotonsAbsorbed] * dt;
        ledger->absorbed_thin = acc[kPhotonsThin] * dt;
        ledger->crossings = cnt[kCrossings];
        ledger->rays = cnt[kRays];
        ledger->splits = cnt[kSplits];
        ledger->terminated = cnt[kTerminated];
        ledger->escaped_rays = cnt[kEscapedRays];
        ledger->spills = cnt[kSpills];
        ledger->deposits = cnt[kDeposits];
        ledger->tree_count = (int64_t)run.tree_count;
        for (int k = 0; k < kMaxBins; ++k) ledger->u_j[k] = k < P.nb ? P.uj[k] : 0.0;
        const bool levels = !batched || P.litem > P.A.level0;
        if (P.nsrc > 0) ledger->ms_trace = ms_between(levels ? kStampTrace : kStampPersistent, kStampRates);
        ledger->ms_total = ms_between(kStampBegin, kStampEnd);
        if (batched && P.nsrc > 0) {
            ledger->kernel_crossings = per[kCrossings];
            ledger->kernel_deposits = per[kDeposits];
            ledger->ms_kernel = ms_between(kStampPersistent, kStampRates);
        }
    }
    return ARC_OK;
}

arc_tune_result* find_tuned(arc_ctx* c, const arc_grid* g, const TracePlan& P)
{
    for (auto& t : c->tuned)
        if (t.nx == g->nx && t.ny == g->ny && t.nz == g->nz && t.nb == P.nb && t.level0 == P.A.level0 &&
            t.lmax == P.lmax && t.precision == P.precision && t.corr == P.A.corr && t.thin == P.thin)
            return &t.shape;
    return nullptr;
}

arc_status autotune_impl(arc_ctx* c, const arc_grid* g, const arc_sources* s, const arc_freq_bins* b, double dt,
                         const arc_trace_params* p, const arc_rates* out, arc_tune_result* res);

}  // namespace

extern "C" {

arc_status arc_trace(arc_ctx* c, const arc_grid* g, const arc_sources* s, const arc_freq_bins* b, double dt,
                     const arc_trace_params* p, arc_rates* out, arc_ledger* ledger)
{
    if (!c) return ARC_E_ARG;
    c->err.clear();
    TracePlan P;
    arc_status rc = plan_trace(c, g, s, b, dt, p, out, P);
    if (rc != ARC_OK) return rc;
    hipStream_t st = (hipStream_t)p->stream;
    if (p->schedule == ARC_SCHED_BATCHED) {
        const int waves = p->tune_waves > 0 ? p->tune_waves : 4;
        const int refill = p->tune_refill > 0 ? p->tune_refill : kDefaultRefill;
        const int stack = p->tune_stack > 0 ? p->tune_stack : kDefaultStack;
        const int blocks = p->tune_blocks > 0 ? p->tune_blocks : c->cus * default_workgroups_per_cu(P, waves, stack);
        if ((rc = shape_batched(c, P, waves, blocks, refill, p->tune_item_level, stack)) != ARC_OK)
            return rc;
    } else if (p->schedule == ARC_SCHED_BATCHED_TUNED) {
        const arc_tune_result* t = find_tuned(c, g, P);
        arc_tune_result fresh;
        if (!t) {
            // tune on an evenly spaced subset of at most 256 sources
            const int step = std::max(1, (s->n + 255) / 256);
            std::vector<double> pos, nd, rt;
            for (int i = 0; i < s->n; i += step) {
                pos.insert(pos.end(), s->pos + 3 * i, s->pos + 3 * i + 3);
                nd.push_back(s->ndot[i]);
                if (s->r_thin) rt.push_back(s->r_thin[i]);
            }
            // (radii out make it a trace with thin spheres, also where the subset has none)
            std::vector<double> rout(P.thin ? nd.size() : 0);
            const arc_sources sub{(int32_t)nd.size(), pos.data(), nd.data(), s->r_thin ? rt.data() : nullptr,
                                  P.thin ? rout.data() : nullptr};
            if ((rc = autotune_impl(c, g, &sub, b, dt, p, out, &fresh)) != ARC_OK) return rc;
            t = &fresh;
            // the tuning runs changed the plan's buffers: plan again for all sources
            if ((rc = plan_trace(c, g, s, b, dt, p, out, P)) != ARC_OK) return rc;
        }
        const int blocks = std::max(1, c->cus * t->waves_per_cu / t->waves);
        if ((rc = shape_batched(c, P, t->waves, blocks, t->refill, P.A.level0 + t->item_delta, t->stack)) != ARC_OK)
            return rc;
    }
    return run_trace(c, P, s, dt, p->schedule, p->graph != 0, st, ledger);
}

arc_status arc_autotune(arc_ctx* c, const arc_grid* g, const arc_sources* s, const arc_freq_bins* b, double dt,
                        const arc_trace_params* p, arc_rates* out, arc_tune_result* res)
{
    if (!c) return ARC_E_ARG;
    c->err.clear();
    arc_tune_result r;
    arc_status rc = autotune_impl(c, g, s, b, dt, p, out, &r);
    if (rc == ARC_OK && res) *res = r;
    return rc;
}

}  // extern "C"

namespace {

arc_status autotune_impl(arc_ctx* c, const arc_grid* g, const arc_sources* s, const arc_freq_bins* b, double dt,
                         const arc_trace_params* p, const arc_rates* out, arc_tune_result* res)
{
    if (!p) return fail(c, ARC_E_ARG, "null params");
    arc_trace_params q = *p;
    q.schedule = ARC_SCHED_BATCHED;
    q.tree_out = nullptr;
    q.tree_cap = 0;
    TracePlan P;
    arc_status rc = plan_trace(c, g, s, b, dt, &q, out, P);
    if (rc != ARC_OK) return rc;
    if (s->n == 0) return fail(c, ARC_E_ARG, "autotuning needs at least one source");
    hipStream_t st = (hipStream_t)q.stream;
    unsigned long long ref[2] = {0, 0};
    bool have_ref = false;
    int ncand = 0;
    // time one shape twice; check its field against the first shape's
    auto time_shape = [&](const arc_tune_result& t, double* ms_out) -> arc_status {
        const int blocks = std::max(1, c->cus * t.waves_per_cu / t.waves);
        arc_status r2 = shape_batched(c, P, t.waves, blocks, t.refill, P.A.level0 + t.item_delta, t.stack);
        if (r2 != ARC_OK) return r2;
        double best = INFINITY;
        for (int rep = 0; rep < 2; ++rep) {
            arc_ledger led;
            if ((r2 = run_trace(c, P, s, dt, ARC_SCHED_BATCHED, false, st, &led)) != ARC_OK) return r2;
            best = std::min(best, led.ms_trace);
        }
        HIP_TRY(c, launch_zero_u64(c->sums, 2, st));
        const size_t words = (size_t)P.nbx8 * P.nby8 * P.nbz8 * 512 * P.nb;
        HIP_TRY(c, launch_field_checksum(c->J, words, c->sums, st));
        if (P.A.M) HIP_TRY(c, launch_field_checksum(P.A.M, 2 * words, c->sums, st));
        unsigned long long h[2];
        HIP_TRY(c, hipMemcpyAsync(h, c->sums, sizeof h, hipMemcpyDeviceToHost, st));
        HIP_TRY(c, hipStreamSynchronize(st));
        if (!have_ref) {
            ref[0] = h[0];
            ref[1] = h[1];
            have_ref = true;
        } else if (h[0] != ref[0] || h[1] != ref[1]) {
            return fail(c, ARC_E_MISMATCH,
                        "launch shape (waves %d, waves/CU %d, refill %d, item delta %d, stack %d) changed the field",
                        t.waves, t.waves_per_cu, t.refill, t.item_delta, t.stack);
        }
        ++ncand;
        *ms_out = best;
        return ARC_OK;
    };
    // the default shape comes first
    arc_tune_result best{};
    best.waves = 4;
    best.waves_per_cu = best.waves * default_workgroups_per_cu(P, best.waves, kDefaultStack);
    best.refill = kDefaultRefill;
    best.stack = kDefaultStack;
    best.item_delta = default_item_level(P) - P.A.level0;
    double ms_best;
    if ((rc = time_shape(best, &ms_best)) != ARC_OK) return rc;
    const double ms_default = ms_best;
    auto consider = [&](arc_tune_result t) -> arc_status {
        double ms;
        arc_status r2 = time_shape(t, &ms);
        if (r2 != ARC_OK) return r2;
        if (ms < ms_best) {
            ms_best = ms;
            best = t;
        }
        return ARC_OK;
    };
    // (1) work-item level (levels below the first; the run clamps it to the memory bound). Five
    // below the first and on: higher ones win on a source sample, whose subtrees are few,
    // but on the full run their subtrees outgrow the LDS stacks (1024^3 x 16384 sources, four
    // levels below the first: 3.8e8 rays spilled and 760 ms against 712 ms at five).
    const arc_tune_result base1 = best;
    for (int d : {kDefaultItemDepth, kDefaultItemDepth + 1, kDefaultItemDepth + 2}) {
        if (d == base1.item_delta) continue;
        arc_tune_result t = base1;
        t.item_delta = d;
        if ((rc = consider(t)) != ARC_OK) return rc;
    }
    // (2) waves per workgroup and resident waves per CU
    const arc_tune_result base2 = best;
    for (int wv : {2, 4, 8})
        for (int wpc : {8, 12, 16}) {
            if (wv == base2.waves && wpc == base2.waves_per_cu) continue;
            arc_tune_result t = base2;
            t.waves = wv;
            t.waves_per_cu = wpc;
            if ((rc = consider(t)) != ARC_OK) return rc;
        }
    // (3) refill threshold
    const arc_tune_result base3 = best;
    for (int rf : {16, 32, 48, 56, 64}) {
        if (rf == base3.refill) continue;
        arc_tune_result t = base3;
        t.refill = rf;
        if ((rc = consider(t)) != ARC_OK) return rc;
    }
    // (4) depth of the waves' LDS stacks
    const arc_tune_result base4 = best;
    for (int sd : {128, 256}) {
        arc_tune_result t = base4;
        t.stack = sd;
        if ((rc = consider(t)) != ARC_OK) return rc;
    }
    best.ms_best = ms_best;
    best.ms_default = ms_default;
    best.candidates = ncand;
    if (arc_tune_result* known = find_tuned(c, g, P))
        *known = best;
    else
        c->tuned.push_back({g->nx, g->ny, g->nz, P.nb, P.A.level0, P.lmax, P.precision, P.A.corr, P.thin, best});
    *res = best;
    return ARC_OK;
}

}  // namespace

extern "C" {

arc_status arc_get_field(arc_ctx* c, int64_t* dst, int64_t count, void* stream)
{
    if (!c || !dst) return ARC_E_ARG;
    if (!c->have_field) return fail(c, ARC_E_ARG, "no field: call arc_trace first");
    const int64_t parts = c->last_moved ? 3 : 1;
    if (count < parts * (int64_t)(c->last_ncell * c->last_nb))
        return fail(c, ARC_E_ARG, "dst too small (needs %lld entries)", (long long)(parts * c->last_ncell * c->last_nb));
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    HIP_TRY(c, launch_get_field(c->J, c->last_moved ? c->M : nullptr, c->last_nb, c->last_nx, c->last_ny,
                                c->last_nbx8, c->last_nby8, (uint32_t)c->last_ncell, (long long*)dst, st));
    HIP_TRY(c, hipStreamSynchronize(st));
    return ARC_OK;
}

arc_status arc_probe_requests(arc_ctx* c, int64_t items, int64_t cells, uint64_t seed, void* stream,
                              double* deposits_per_s, double* gathers_per_s)
{
    if (!c || !deposits_per_s || !gathers_per_s) return ARC_E_ARG;
    if (items <= 0) return fail(c, ARC_E_ARG, "items must be > 0");
    if (c->last_nb < 2 || !c->J || !c->kappa) return fail(c, ARC_E_ARG, "probe needs a previous trace with 2 to 4 bins");
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    const uint64_t nblocked = (uint64_t)c->last_nbx8 * (uint64_t)c->last_nby8 * 512ull *
                              (uint64_t)((c->last_ncell / ((size_t)c->last_nx * c->last_ny) + 7) / 8);
    if (cells < 0) return fail(c, ARC_E_ARG, "cells must be >= 0");
    const uint64_t ncell = cells > 0 ? std::min<uint64_t>((uint64_t)cells, nblocked) : nblocked;
    // whole tiles of the field: eight cells, a line per bin
    const uint64_t nline = std::max<uint64_t>(1, ncell / 8) * (uint64_t)c->last_nb;
    float ms = 0.0f;
    double best_d = 0.0, best_g = 0.0;
    for (int rep = 0; rep < 3; ++rep) {
        HIP_TRY(c, hipEventRecord(c->ev[0], st));
        HIP_TRY(c, launch_probe_deposits(c->J, nline, (uint64_t)items, seed + rep, c->cus, st));
        HIP_TRY(c, hipEventRecord(c->ev[1], st));
        HIP_TRY(c, launch_probe_gathers((const float4*)c->kappa, ncell, (uint64_t)items, seed + rep, (float*)c->run,
                                        c->cus, st));
        HIP_TRY(c, hipEventRecord(c->ev[2], st));
        HIP_TRY(c, hipEventSynchronize(c->ev[2]));
        HIP_TRY(c, hipEventElapsedTime(&ms, c->ev[0], c->ev[1]));
        best_d = std::max(best_d, (double)items / (ms * 1e-3));
        HIP_TRY(c, hipEventElapsedTime(&ms, c->ev[1], c->ev[2]));
        best_g = std::max(best_g, (double)items / (ms * 1e-3));
    }
    c->have_field = false;  // the field now holds the probe's counts
    *deposits_per_s = best_d;
    *gathers_per_s = best_g;
    return ARC_OK;
}

arc_status arc_healpix_dirs(arc_ctx* c, int32_t level, float* dst, void* stream)
{
    if (!c || !dst) return ARC_E_ARG;
    if (level < 0 || level > 12) return fail(c, ARC_E_ARG, "level must be 0..12");
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(c, hipSetDevice(c->device));
    arc_status rc = ensure_dirs(c, level + 1, st);
    if (rc != ARC_OK) return rc;
    const size_t npix = (size_t)12 << (2 * level);
    // float4 table -> x, y, z triples
    std::vector<float4> h(npix);
    HIP_TRY(c, hipMemcpyAsync(h.data(), c->dirs + c->dir_off[level], npix * sizeof(float4), hipMemcpyDeviceToHost, st));
    HIP_TRY(c, hipStreamSynchronize(st));
    std::vector<float> f(3 * npix);
    for (size_t i = 0; i < npix; ++i) {
        f[3 * i] = h[i].x;
        f[3 * i + 1] = h[i].y;
        f[3 * i + 2] = h[i].z;
    }
    HIP_TRY(c, hipMemcpyAsync(dst, f.data(), f.size() * sizeof(float), hipMemcpyHostToDevice, st));
    HIP_TRY(c, hipStreamSynchronize(st));
    return ARC_OK;
}

}  // extern "C"

namespace {

// Everything the chemistry step launches with, zero-filled (its bytes key the graphs).
struct ChemPlan {
    ChemArgs a;
    mlp::InferArgs ia;
    ChemResult* result;
    int mode;
    int cus;
};

// The network and its gate (learned modes), the sub-cycled solver (plain and gated modes), and
// the statistics to the host.
hipError_t enqueue_chem(const ChemPlan& P, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (P.mode != ARC_CHEM_PLAIN && (e = mlp::launch_infer(P.ia, P.cus, st)) != hipSuccess) return e;
    if (P.mode != ARC_CHEM_MLP_ONLY && (e = launch_chem(P.a, P.cus, st)) != hipSuccess) return e;
    return launch_chem_end(P.a.run, P.result, st);
}

}  // namespace

namespace {

// Checks and launch arguments of the section 2.9 time step, shared by both entry points;
// `out` receives the two minima as bit patterns of non-negative doubles.
arc_status plan_timestep(arc_ctx* c, const arc_grid* g, const arc_rates* r, const arc_freq_bins* b,
                         const arc_chem_params* p, double eps, unsigned long long* out, TimestepArgs& a)
{
    arc_status rc;
    if ((rc = check_grid(c, g)) != ARC_OK) return rc;
    if ((rc = check_bins(c, b)) != ARC_OK) return rc;
    if (!g->temp) return fail(c, ARC_E_ARG, "null temperature");
    if (!r || !r->gamma) return fail(c, ARC_E_ARG, "null rates");
    if (!p) return fail(c, ARC_E_ARG, "null params");
    if (!(eps > 0) || !std::isfinite(eps)) return fail(c, ARC_E_RANGE, "eps must be finite and > 0");
    if (p->rates != 0 && p->rates != 1) return fail(c, ARC_E_ARG, "rates must be 0 or 1");
    if (p->rates == 0 && !(p->alpha_hii >= 0)) return fail(c, ARC_E_RANGE, "alpha_hii must be >= 0");
    a = TimestepArgs{};
    a.ncell = (uint32_t)((size_t)g->nx * g->ny * g->nz);
    a.y = g->y_he;
    a.cell_cm = g->cell_cm;
    a.sigma0 = b->sigma[0];
    a.eps = eps;
    a.n_h = g->n_h;
    a.x_hi = g->x_hi;
    a.x_hei = g->x_hei;
    a.x_heii = g->x_heii;
    a.temp = g->temp;
    a.gamma_hi = r->gamma;
    a.rates = p->rates;
    a.collisional = p->collisional;
    a.alpha_hii = p->alpha_hii;
    a.out = out;
    return ARC_OK;
}

}  // namespace

extern "C" {

arc_status arc_rt_timestep(arc_ctx* c, const arc_grid* g, const arc_rates* r, const arc_freq_bins* b,
                           const arc_chem_params* p, double eps, double* dt_n, double* dt_i)
{
    if (!c) return ARC_E_ARG;
    c->err.clear();
    if (!dt_n || !dt_i) return fail(c, ARC_E_ARG, "null outputs");
    TimestepArgs a;
    arc_status rc = plan_timestep(c, g, r, b, p, eps, c->limits, a);
    if (rc != ARC_OK) return rc;
    hipStream_t st = (hipStream_t)p->stream;
    HIP_TRY(c, hipSetDevice(c->device));
    if (!c->limits_clean) HIP_TRY(c, launch_timestep_reset(c->limits, st));
    c->limits_clean = false;
    HIP_TRY(c, launch_timestep(a, c->cus, st));
    HIP_TRY(c, launch_timestep_end(c->limits, c->host->limits, st));
    HIP_TRY(c, hipStreamSynchronize(st));
    c->limits_clean = true;
    *dt_n = c->host->limits[0];
    *dt_i = c->host->limits[1];
    return ARC_OK;
}

arc_status arc_rt_timestep_noalloc(arc_ctx* c, const arc_grid* g, const arc_rates* r, const arc_freq_bins* b,
                                   const arc_chem_params* p, double eps, double* dt_out)
{
    if (!c) return ARC_E_ARG;
    c->err.clear();
    if (!dt_out) return fail(c, ARC_E_ARG, "null output");
    if (!c->static_scratch) return fail(c, ARC_E_DEVICE, "static scratch of device %d not resolved", c->device);
    // the kernels use kTimestepScratchWords words of the device's static scratch, whatever the
    // grid; grids are bounded by the checks every entry point applies (below 2^31 cells)
    static_assert(kTimestepScratchWords <= kStaticScratchWords, "static scratch too small");
    TimestepArgs a;
    arc_status rc = plan_timestep(c, g, r, b, p, eps, c->static_scratch, a);
    if (rc != ARC_OK) return rc;
    hipStream_t st = (hipStream_t)p->stream;
    HIP_TRY(c, hipSetDevice(c->device));
    // the array keeps the last call's minima: reset them (a kernel, not a memset node)
    HIP_TRY(c, launch_timestep_reset(c->static_scratch, st));
    HIP_TRY(c, launch_timestep(a, c->cus, st));
    HIP_TRY(c, launch_timestep_publish(c->static_scratch, dt_out, st));
    return ARC_OK;
}

arc_status arc_chem_step(arc_ctx* c, const arc_grid* g, const arc_rates* r, double dt, const arc_chem_params* p,
                         arc_chem_stats* stats)
{
    if (!c) return ARC_E_ARG;
    c->err.clear();
    arc_status rc;
    if ((rc = check_grid(c, g)) != ARC_OK) return rc;
    if (!g->temp) return fail(c, ARC_E_ARG, "null temperature");
    if (!r || !r->gamma || !r->heat) return fail(c, ARC_E_ARG, "null rates");
    if (!p) return fail(c, ARC_E_ARG, "null params");
    if (!(dt > 0) || !std::isfinite(dt)) return fail(c, ARC_E_RANGE, "dt must be finite and > 0");
    if (!(p->eps > 0) || !std::isfinite(p->eps)) return fail(c, ARC_E_RANGE, "eps must be > 0");
    if (p->max_sub < 1) return fail(c, ARC_E_RANGE, "max_sub must be >= 1");
    if (p->rates != 0 && p->rates != 1) return fail(c, ARC_E_ARG, "rates must be 0 or 1");
    if (p->rates == 0 && !(p->alpha_hii >= 0)) return fail(c, ARC_E_RANGE, "alpha_hii must be >= 0");
    if (!(p->t_floor > 0)) return fail(c, ARC_E_RANGE, "t_floor must be > 0");
    if (p->mode != ARC_CHEM_PLAIN && p->mode != ARC_CHEM_MLP_GATED && p->mode != ARC_CHEM_MLP_ONLY)
        return fail(c, ARC_E_ARG, "bad chemistry mode %d", p->mode);
    if (p->mode != ARC_CHEM_PLAIN && (!p->mlp || !p->mlp->trained))
        return fail(c, ARC_E_ARG, "the learned modes need a trained network");
    if (p->mode == ARC_CHEM_MLP_GATED && !(p->gate_tol >= 0)) return fail(c, ARC_E_RANGE, "gate_tol must be >= 0");
    hipStream_t st = (hipStream_t)p->stream;
    HIP_TRY(c, hipSetDevice(c->device));
    ChemPlan P;
    std::memset(&P, 0, sizeof P);
    P.mode = p->mode;
    P.cus = c->cus;
    ChemArgs& a = P.a;
    a.ncell = (uint32_t)((size_t)g->nx * g->ny * g->nz);
    a.y = g->y_he;
    a.inv_y = g->y_he > 0 ? 1.0 / g->y_he : 0.0;
    a.n_h = g->n_h;
    a.x_hi = g->x_hi;
    a.x_hei = g->x_hei;
    a.x_heii = g->x_heii;
    a.temp = g->temp;
    a.gamma = r->gamma;
    a.heat = r->heat;
    a.dt = dt;
    a.isothermal = p->isothermal;
    a.rates = p->rates;
    a.collisional = p->collisional;
    a.max_sub = p->max_sub;
    a.alpha_hii = p->alpha_hii;
    a.eps = p->eps;
    a.t_floor = p->t_floor;
    a.run = c->chem_run;
    P.result = &c->host->chem;
    a.mask = nullptr;
    if (p->mode != ARC_CHEM_PLAIN) {
        const size_t words = ((size_t)a.ncell + 63) / 64;
        if (words > c->reject_cap) {
            if (c->reject) HIP_TRY(c, hipFree(c->reject));
            c->reject = nullptr;
            c->reject_cap = 0;
            HIP_TRY(c, hipMalloc((void**)&c->reject, words * sizeof(unsigned long long)));
            c->reject_cap = words;
        }
        mlp::InferArgs& ia = P.ia;
        ia.model = p->mlp->model;
        ia.ncell = a.ncell;
        ia.y = a.y;
        ia.n_h = a.n_h;
        ia.x_hi = a.x_hi;
        ia.x_hei = a.x_hei;
        ia.x_heii = a.x_heii;
        ia.temp = a.temp;
        ia.gamma = a.gamma;
        ia.heat = a.heat;
        ia.dt = dt;
        ia.gated = p->mode == ARC_CHEM_MLP_GATED;
        ia.gate_tol = (float)p->gate_tol;
        ia.gate_min_count = (uint32_t)std::max(0, p->gate_min_count);
        ia.t_floor = (float)p->t_floor;
        ia.reject = c->reject;
        ia.collisional = p->rates == 1 ? p->collisional : 0;
        ia.stamp = &c->chem_run->stamp[0];
        if (p->mode == ARC_CHEM_MLP_GATED) a.mask = c->reject;
    }
    if (!c->chem_clean) HIP_TRY(c, launch_zero_u64((unsigned long long*)c->chem_run, sizeof(ChemBlock) / 8, st));
    c->chem_clean = false;
    if (p->graph) {
        if ((rc = ensure_graph(c, &c->cexec, c->chem_key, &P, sizeof P, "the chemistry step",
                               [&](hipStream_t cs) { return enqueue_chem(P, cs); })) != ARC_OK)
            return rc;
        HIP_TRY(c, hipGraphLaunch(c->cexec, st));
    } else {
        HIP_TRY(c, enqueue_chem(P, st));
    }
    HIP_TRY(c, hipStreamSynchronize(st));
    c->chem_clean = true;
    if (stats) {
        const ChemResult& r2 = c->host->chem;
        const bool solver = p->mode != ARC_CHEM_MLP_ONLY, network = p->mode != ARC_CHEM_PLAIN;
        auto ms_between = [&](int i, int j) { return (double)(r2.stamp[j] - r2.stamp[i]) / c->clock_khz; };
        stats->cells = a.ncell;
        stats->sub_total = (int64_t)r2.sub_total;
        stats->capped = (int64_t)r2.capped;
        stats->sub_max = (int32_t)r2.sub_max;
        stats->ms = ms_between(network ? 0 : 1, 2);
        stats->fallback = p->mode == ARC_CHEM_MLP_GATED ? (int64_t)r2.cells : 0;
        stats->ms_mlp = network ? ms_between(0, solver ? 1 : 2) : 0.0;
    }
    return ARC_OK;
}

}  // extern "C"
