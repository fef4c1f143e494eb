// arc_kernels.h -- launch wrappers of libarc's kernels (host-callable).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "arc_device.h"

namespace arc {

struct OpacityArgs {
    int nb;
    int nx, ny, nz, nbx8, nby8, nbz8;
    uint32_t ncell;
    double L, y;
    double sigma[kMaxBins][3];
    const float *n_h, *x_hi, *x_hei, *x_heii;
    float* kappa1;
    float4* kappa4;
    unsigned long long* J;
    unsigned long long* M;     // moved-photon field of the conserving correction, or null
    int* errflag;
};

struct FinalizeArgs {
    int nb;
    int nx, ny, nz, nbx8, nby8, nbz8;
    uint32_t ncell;
    double gam[kMaxBins][3];   // u_J,b sigma_bS / L^2
    double hea[kMaxBins][3];   // u_J,b sigma_bS (E_b - E_S)^+ / L^2
    double uj[kMaxBins];
    const unsigned long long* J;
    const unsigned long long* M;  // moved-photon field (two limbs per bin), or null
    const float* kappa1;
    const float4* kappa4;
    float *gamma, *heat;       // [3][ncell]
    CounterSlot* slots;        // photons absorbed: sum_c sum_b u_J J kappa
    unsigned long long* stamp;
};

// Set-up of a call. Root rays (batched) are those of the sources order[0 .. nsrc), each source's
// contiguous in pixel order; none without `roots`.
struct BeginArgs {
    RunBlock* run;
    int nb, nsrc, level0;
    uint32_t n_roots;
    const double *pos, *ndot, *r_thin;  // pinned; r_thin: null where no source has a thin sphere
    double* fill;              // [nsrc][5] for the thin fill (position, rate, radius), or null
    double scale[kMaxBins];    // frac_b / (12 u_J,b)
    SourceRec* src;
    uint32_t* r_out;           // measured thin radii, or null
    const uint32_t* order;     // pinned
    RayRec* roots;
};

// Section 2.6 fill of the optically thin spheres.
struct ThinFillArgs {
    int nb, nsrc, parts;       // parts: blocks per source
    int nx, ny, nz, nbx8, nby8;
    const double* src;         // [nsrc][5]: position, photon rate, thin radius
    double coef[kMaxBins];     // frac_b / (4 pi u_J,b)
    double uj[kMaxBins];
    unsigned long long* J;
    const float* kappa1;
    const float4* kappa4;
    CounterSlot* slots;        // photons of the fill: its deposits times u_J kappa
};

// The device's side of one chemistry step: statistics in copies (a 128-byte line each), the next
// chunk of cells, when the stages began. Zero before the step: its last kernel clears what it
// has handed to the host.
constexpr int kChemSlots = 16;
struct __align__(128) ChemSlot {
    unsigned long long sub_total, capped, sub_max, cells;
};
struct ChemBlock {
    ChemSlot slot[kChemSlots];
    unsigned long long stamp[2];  // network, solver
    uint32_t chunk;
};
struct ChemResult {
    unsigned long long sub_total, capped, sub_max, cells, stamp[3];  // stamps: network, solver, end
};
hipError_t launch_chem_end(ChemBlock* run, ChemResult* out, hipStream_t s);

struct ChemArgs {
    uint32_t ncell;
    double y;
    const float* n_h;
    float *x_hi, *x_hei, *x_heii, *temp;
    const float *gamma, *heat;
    double dt;
    int isothermal, rates, collisional, max_sub;
    double alpha_hii, eps, t_floor;
    double inv_y;               // 1 / y (0 where y = 0)
    ChemBlock* run;
    // optional: update only the cells whose bit is set, bit (c mod 64) of word c / 64
    const unsigned long long* mask;
};

hipError_t launch_zero_u64(unsigned long long* p, size_t n, hipStream_t s);
hipError_t launch_set_u32(uint32_t* p, uint32_t v, hipStream_t s);
// out[0] = sum J[i], out[1] = sum J[i] (2i + 1), both mod 2^64; out must be zeroed first.
hipError_t launch_field_checksum(const unsigned long long* J, size_t n, unsigned long long* out, hipStream_t s);
hipError_t launch_opacity(const OpacityArgs& a, hipStream_t s);
hipError_t launch_healpix(int level, float4* out, hipStream_t s);
hipError_t launch_begin(const BeginArgs& a, hipStream_t s);
// r_host (pinned, optional): receives r_out[0 .. nsrc).
hipError_t launch_end(const RunBlock* run, RunResult* out, const uint32_t* r_out, uint32_t* r_host, int nsrc,
                      hipStream_t s);
hipError_t launch_thin_fill(const ThinFillArgs& a, hipStream_t s);
hipError_t launch_seed_roots(uint32_t src, int level0, RayRec* out, hipStream_t s);
// n_in_dev (optional) holds the ray count on the device; n_in bounds it and sizes the grid.
// fam_out: a split ray writes one family record (its own id and depth) instead of its four
// children, for the persistent launch.
hipError_t launch_trace_rays(const TraceArgs& A, int prec, const RayRec* in, const uint32_t* n_in_dev, uint32_t n_in,
                             RayRec* out, uint32_t* n_out, uint32_t out_cap, int fam_out, hipStream_t s);
// fam: the work items are family records (four rays each), else single rays. stack_cap:
// split rays each wave's LDS stack holds (64, 128 or 256).
hipError_t launch_trace_persistent(const TraceArgs& A, int prec, const RayRec* items, const uint32_t* n_items,
                                   uint32_t* head, RayRec* spill, uint32_t spill_cap, int blocks, int waves,
                                   int refill, int fam, int stack_cap, hipStream_t s);
// Waves per SIMD that the persistent kernel's registers allow (a compute unit has four SIMDs).
constexpr int persistent_waves_per_simd(int nb) { return nb <= 3 ? 4 : 3; }
// Workgroups of the persistent kernel that a compute unit holds at once, by their registers and by
// their LDS. sides: nx + ny + nz.
int persistent_workgroups_per_cu(int nb, int sides, int waves, int stack_cap);
// The waves per SIMD of a level's kernel: the fourth wave is worth its spills but with the correction
// (256^3 x 1024 sources: levels 2.08 ms with three, 1.84 with four; corrected 192^3 x 128: 0.60
// and 0.73).
constexpr int level_waves_per_simd(int nb, bool corr) { return corr ? 3 : persistent_waves_per_simd(nb); }
hipError_t launch_finalize(const FinalizeArgs& a, hipStream_t s);
hipError_t launch_probe_deposits(unsigned long long* J, uint64_t nline, uint64_t items, uint64_t seed, int cus,
                                 hipStream_t s);
hipError_t launch_probe_gathers(const float4* kappa, uint64_t ncell, uint64_t items, uint64_t seed, float* sink,
                                int cus, hipStream_t s);
hipError_t launch_get_field(const unsigned long long* J, const unsigned long long* M, int nb, int nx, int ny, int nbx8,
                            int nby8, uint32_t ncell, long long* dst, hipStream_t s);
// cus: compute units of the device (the solver launches resident waves only)
hipError_t launch_chem(const ChemArgs& a, int cus, hipStream_t s);

// Section 2.9 time-step limits: out[0] = min dt_n, out[1] = min dt_I as the bit patterns of
// non-negative doubles (+inf when no cell constrains); reset with launch_timestep_reset.
struct TimestepArgs {
    uint32_t ncell;
    double y, cell_cm, sigma0, eps;
    const float *n_h, *x_hi, *x_hei, *x_heii, *temp;
    const float* gamma_hi;
    int rates, collisional;
    double alpha_hii;
    unsigned long long* out;
};
hipError_t launch_timestep_reset(unsigned long long* out, hipStream_t s);
hipError_t launch_timestep(const TimestepArgs& a, int cus, hipStream_t s);
hipError_t launch_timestep_publish(const unsigned long long* bits, double* out, hipStream_t s);
// The same into pinned host memory, then bits back to +inf for the next call.
hipError_t launch_timestep_end(unsigned long long* bits, double* out, hipStream_t s);

}  // namespace arc
