// arc_chem.hip -- the plain chemistry step of libarc (gfx950):
//
//   k_chem             sub-cycled backward-difference chemistry and energy update, one cell
//                      per lane, lanes refilled from a chunked global cell counter
//   k_timestep         the adaptive RT time step's two grid minima (section 2.9)
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "arc_chem.h"
#include "arc_kernels.h"

namespace arc {

// -------------------------------------------------------------------------------------
// Chemistry (eq:diffeq in the backward-difference form of eq:anninos, sub-cycled with
// the step limit of section 2.7; heating and cooling of section 2.8). One cell per
// lane. Rate coefficients and cooling in FP32, species and energy in FP64.
// Coefficients: Hui & Gnedin (1997) fits with lambda = 2 T_i / T.
// -------------------------------------------------------------------------------------


// State of one cell during its sub-cycled update.
struct ChemCell {
    double nh, nhe, nhi, nhii, nhei, nheii, nheiii, ne, E, t;
    float ghi, ghei, gheii, hhi, hhei, hheii;
    float T;
    int n;
    uint32_t c;
};

// Loads cell lo + i; lo is wave-uniform, so that the addresses are a scalar base and a 32-bit
// lane offset.
__device__ __forceinline__ void chem_load(const ChemArgs& a, uint32_t lo, uint32_t i, ChemCell& s)
{
    s.c = lo + i;
    s.nh = (a.n_h + lo)[i];
    s.nhe = a.y * s.nh;
    s.nhi = s.nh * (double)(a.x_hi + lo)[i];
    s.nhii = s.nh - s.nhi;
    s.nhei = s.nhe * (double)(a.x_hei + lo)[i];
    s.nheii = s.nhe * (double)(a.x_heii + lo)[i];
    s.nheiii = s.nhe - s.nhei - s.nheii;
    if (s.nheiii < 0) s.nheiii = 0;
    s.T = (a.temp + lo)[i];
    s.ne = fma(2.0, s.nheiii, s.nhii + s.nheii);
    s.E = 1.5 * chem::kKB * (double)s.T * (s.nh + s.nhe + s.ne);
    const size_t n = a.ncell;
    s.ghi = (a.gamma + lo)[i];
    s.ghei = (a.gamma + n + lo)[i];
    s.gheii = (a.gamma + 2 * n + lo)[i];
    s.hhi = (a.heat + lo)[i];
    s.hhei = (a.heat + n + lo)[i];
    s.hheii = (a.heat + 2 * n + lo)[i];
    s.t = 0.0;
    s.n = 0;
}

// 1 / b for b > 0 from the hardware reciprocal and two Newton steps (within an ulp or two
// of the rounded value; the solver's tolerances are orders of magnitude looser), far fewer
// instructions than an IEEE division.
__device__ __forceinline__ double rcp64(double b)
{
    double r = __builtin_amdgcn_rcp(b);
    r = fma(r, fma(-b, r, 1.0), r);
    return fma(r, fma(-b, r, 1.0), r);
}

// One sub-step (section 2.7: backward difference for the species, sub-step limited to a
// fraction eps of the shortest change time). Returns true once the cell has reached dt.
template <bool RATES, bool THERMAL, bool COLL>
__device__ __forceinline__ bool chem_substep(const ChemArgs& a, ChemCell& s)
{
    chem::Coef k{};
    chem::Lam l{};
    if constexpr (RATES || THERMAL) l = chem::lambdas(s.T);
    if constexpr (RATES) {
        k = chem::coefficients(l);
        if constexpr (!COLL) k.k_hi = k.k_hei = k.k_heii = 0.0f;
    } else {
        k.a_hii = (float)a.alpha_hii;
    }
    const double gain_hi = (double)k.a_hii * s.ne, loss_hi = fma((double)k.k_hi, s.ne, (double)s.ghi);
    const double ndot_hi = fma(gain_hi, s.nhii, -(loss_hi * s.nhi));
    double edot = 0.0;
    if constexpr (THERMAL)
        edot = fma(s.nhi, (double)s.hhi, fma(s.nhei, (double)s.hhei, s.nheii * (double)s.hheii)) -
               chem::cooling<COLL>(s.T, l, k, s.ne, s.nhi, s.nhii, s.nhei, s.nheii, s.nheiii);
    double h = a.dt - s.t;
    bool last = true;
    if (s.n < a.max_sub) {
        // a limit is divided out only where it binds: most cells take one sub-step
        if constexpr (THERMAL) {
            if (a.eps * s.E < h * fabs(edot)) {
                const double le = a.eps * s.E * rcp64(fabs(edot));
                if (le < h) {
                    h = le;
                    last = false;
                }
            }
        }
        const double m = fmin(s.nhi > 0.0 ? s.nhi : INFINITY, s.nhii > 0.0 ? s.nhii : INFINITY);
        if (a.eps * m < h * fabs(ndot_hi)) {
            const double ln = a.eps * m * rcp64(fabs(ndot_hi));
            if (ln < h) {
                h = ln;
                last = false;
            }
        }
    }
    // a reciprocal each: one of the product would be NaN for all three species where one factor is
    // not finite (and saves nothing: 256^3 cells, relaxed gas 243 us, with fronts 2.48 ms, either way)
    const double d1 = fma(loss_hi, h, 1.0), d2 = fma(fma((double)k.k_hei, s.ne, (double)s.ghei), h, 1.0),
                 d3 = fma((double)k.a_heiii * s.ne, h, 1.0);
    // (the clamps are comparisons, which let a NaN through, not fmin and fmax)
    s.nhi = fma(gain_hi * s.nhii, h, s.nhi) * rcp64(d1);
    if (s.nhi > s.nh) s.nhi = s.nh;
    s.nhii = s.nh - s.nhi;
    double nhei_new = fma((double)k.a_heii * s.ne * s.nheii, h, s.nhei) * rcp64(d2);
    if (nhei_new > s.nhe) nhei_new = s.nhe;
    const double up = fma((double)k.k_heii, s.ne, (double)s.gheii) * s.nheii;
    s.nheiii = fma(up, h, s.nheiii) * rcp64(d3);
    if (s.nheiii > s.nhe - nhei_new) s.nheiii = s.nhe - nhei_new;
    s.nhei = nhei_new;
    s.nheii = s.nhe - s.nhei - s.nheiii;
    if (s.nheii < 0.0) s.nheii = 0.0;
    s.ne = fma(2.0, s.nheiii, s.nhii + s.nheii);
    if constexpr (THERMAL) {
        s.E = fma(edot, h, s.E);
        const double heat_cap = 1.5 * chem::kKB * (s.nh + s.nhe + s.ne);
        double Td = s.E * rcp64(heat_cap);
        if (Td < a.t_floor) {
            Td = a.t_floor;
            s.E = Td * heat_cap;
        }
        s.T = (float)Td;
    }
    s.t = last ? a.dt : s.t + h;
    ++s.n;
    return !(s.t < a.dt);
}

template <bool THERMAL>
__device__ __forceinline__ void chem_store(const ChemArgs& a, const ChemCell& s)
{
    const double inh = rcp64(s.nh);
    a.x_hi[s.c] = (float)(s.nhi * inh);
    if (s.nhe > 0.0) {  // (an empty cell keeps its helium fractions)
        const double inhe = inh * a.inv_y;
        a.x_hei[s.c] = (float)(s.nhei * inhe);
        a.x_heii[s.c] = (float)(s.nheii * inhe);
    }
    if constexpr (THERMAL) a.temp[s.c] = s.T;
}

// Per-cell chemistry (section 2.7). Cells need from one to many sub-steps, so a wave does
// not take 64 cells and wait for the slowest: each lane advances its cell one sub-step per
// iteration and takes the next cell of the wave's chunk when done (refilled once kChemRefill
// lanes are idle). A wave's first chunk is its own by its place in the grid, later ones come
// from a global counter. The kernel is instantiated per combination of options, sums with FMAs
// and divides only where it must: about 400 VALU instructions per sub-step instead of 600, which
// brings VALU issue to where the 60 bytes per cell are (256^3 cells of a running model, one
// sub-step in nearly all of them: 575 -> 245 us, of which the bytes take 186 at a copy's rate).
constexpr int kChemRefill = 16;

template <bool RATES, bool THERMAL, bool COLL>
__global__ __launch_bounds__(256) void k_chem(ChemArgs a, uint32_t chunk)
{
    unsigned long long sub_total = 0, capped = 0, cells = 0;  // wave-uniform
    int sub_max = 0;
    stamp_start(&a.run->stamp[1]);
    const int lane = threadIdx.x & 63;
    const uint32_t wave = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t own = (uint64_t)wave * chunk, shared_from = (uint64_t)gridDim.x * 4u * chunk;
    uint32_t lo = (uint32_t)min(own, (uint64_t)a.ncell);  // the wave's remaining chunk [lo, hi), wave-uniform
    uint32_t hi = (uint32_t)min(own + chunk, (uint64_t)a.ncell);
    bool drained = false;     // wave-uniform
    bool have = false;
    ChemCell s;
    for (;;) {
        const uint64_t idle = __builtin_amdgcn_ballot_w64(!have);
        const int nidle = __popcll(idle);
        if (!drained && (nidle >= kChemRefill || nidle == 64)) {
            // hand the next cells to the idle lanes, in lane order
            const int place = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u));
            int given = 0;
            while (given < nidle && !drained) {
                if (lo >= hi) {
                    uint32_t b0 = 0;
                    if (shared_from < a.ncell) {
                        if (lane == 0) b0 = atomicAdd(&a.run->chunk, 1u);
                        b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
                    }
                    const uint64_t from = shared_from + (uint64_t)b0 * chunk;
                    if (from >= a.ncell) {
                        drained = true;
                        break;
                    }
                    lo = (uint32_t)from;
                    hi = (uint32_t)min(from + chunk, (uint64_t)a.ncell);
                }
                const int take = min(nidle - given, (int)(hi - lo));
                const int rank = place - given;
                if (!have && rank >= 0 && rank < take) {
                    const uint32_t c = lo + (uint32_t)rank;
                    if (!a.mask || ((a.mask[c >> 6] >> (c & 63)) & 1ull)) {
                        chem_load(a, lo, (uint32_t)rank, s);
                        have = true;
                    }
                }
                lo += (uint32_t)take;
                given += take;
            }
            cells += __popcll(__builtin_amdgcn_ballot_w64(have) & idle);
        }
        const uint64_t busy = __builtin_amdgcn_ballot_w64(have);
        if (!busy) {
            if (drained) break;
            continue;
        }
        sub_total += __popcll(busy);
        bool done = false;
        if (have) done = chem_substep<RATES, THERMAL, COLL>(a, s);
        if (done) {
            chem_store<THERMAL>(a, s);
            sub_max = max(sub_max, s.n);
            have = false;
        }
        // the sub-step after max_sub others went to the end of the step whatever its limits
        capped += __popcll(__builtin_amdgcn_ballot_w64(done && s.n > a.max_sub));
    }
    for (int off = 32; off > 0; off >>= 1) sub_max = max(sub_max, __shfl_xor(sub_max, off, 64));
    if (lane == 0) {
        // atomics on one line go one after the other: kChemSlots copies
        ChemSlot& st = a.run->slot[blockIdx.x & (kChemSlots - 1)];
        if (sub_total) atomicAdd(&st.sub_total, sub_total);
        if (capped) atomicAdd(&st.capped, capped);
        if (sub_max) atomicMax(&st.sub_max, (unsigned long long)sub_max);
        if (cells) atomicAdd(&st.cells, cells);
    }
}

// The step's last launch: statistics and stamps to the host's pinned memory, and the block
// cleared for the next step (a launch before it and a copy after it cost 20 us each in gaps).
__global__ __launch_bounds__(64) void k_chem_end(ChemBlock* run, ChemResult* out)
{
    const int t = threadIdx.x;
    if (t == 0) {
        out->stamp[2] = wall_clock64();
        ChemResult r = {0, 0, 0, 0, {0, 0, 0}};
        for (int i = 0; i < kChemSlots; ++i) {
            r.sub_total += run->slot[i].sub_total;
            r.capped += run->slot[i].capped;
            r.sub_max = max(r.sub_max, run->slot[i].sub_max);
            r.cells += run->slot[i].cells;
        }
        out->sub_total = r.sub_total;
        out->capped = r.capped;
        out->sub_max = r.sub_max;
        out->cells = r.cells;
        out->stamp[0] = run->stamp[0];
        out->stamp[1] = run->stamp[1];
        run->chunk = 0u;
        __threadfence_system();
    }
    __syncthreads();
    if (t < kChemSlots) run->slot[t].sub_total = run->slot[t].capped = run->slot[t].sub_max = run->slot[t].cells = 0ull;
}

hipError_t launch_chem_end(ChemBlock* run, ChemResult* out, hipStream_t s)
{
    k_chem_end<<<1, 64, 0, s>>>(run, out);
    return hipGetLastError();
}

template <bool RATES, bool THERMAL, bool COLL>
static hipError_t chem_go(const ChemArgs& a, int cus, hipStream_t s)
{
    // every wave loops until the chunks run out. Six waves per SIMD of the eight that the registers
    // allow: 256^3 cells of relaxed gas 242 us, with eight 260; with fronts, 13 sub-steps in the mean,
    // 2.48 ms and 2.42.
    const size_t want = ((size_t)a.ncell + 255) / 256;
    const unsigned blocks = (unsigned)std::max<size_t>(1, std::min<size_t>(want, (size_t)std::max(1, cus) * 6));
    // Two chunks per wave and more on large grids (the second half goes to whoever is free), at
    // most 2048 cells; on small ones at least the 64 cells of one round, so that all waves work
    // (64^3 cells in chunks of 2048 kept 128 waves busy, 157 us).
    const size_t waves = (size_t)blocks * 4;
    const size_t half = ((size_t)a.ncell / (2 * waves) + 63) / 64 * 64;
    const uint32_t chunk = (uint32_t)std::min<size_t>(2048, std::max<size_t>(64, half));
    k_chem<RATES, THERMAL, COLL><<<blocks, 256, 0, s>>>(a, chunk);
    return hipGetLastError();
}

hipError_t launch_chem(const ChemArgs& a, int cus, hipStream_t s)
{
    const bool coll = a.collisional != 0;
    if (a.rates != 0) {
        if (a.isothermal) return coll ? chem_go<true, false, true>(a, cus, s) : chem_go<true, false, false>(a, cus, s);
        return coll ? chem_go<true, true, true>(a, cus, s) : chem_go<true, true, false>(a, cus, s);
    }
    // fixed alpha_HII: collisional terms are zero
    return a.isothermal ? chem_go<false, false, false>(a, cus, s) : chem_go<false, true, false>(a, cus, s);
}

// -------------------------------------------------------------------------------------
// Adaptive RT time step (section 2.9). Per cell, from the current state and rates, the
// source term of the HI equation ndot = alpha_HII n_e n_HII - (Gamma_HI + k_HI n_e) n_HI
// (FP32 coefficients, FP64 densities, as in the solver); then the neutral-fraction limit
// eps n_HI / |ndot| over cells with tau = n_HI sigma0 L > 0.5 and the intensity limit
// eps / (sigma0 L |ndot|) over all cells. The second falls with |ndot|, so a thread keeps the
// largest |ndot| and divides once; for the first it divides only where the product says that
// the quotient may be a new minimum. Minima over the grid: per workgroup, then one atomic min
// each on the bit patterns of the non-negative doubles (the order of the updates cannot change
// the result). Bound by its 24 bytes per cell; with an atomic per wave it waited for those, carried
// out one after the other (64^3 cells 96 us, 320^3 307 us).
// -------------------------------------------------------------------------------------
constexpr int kStepThreads = 256;
constexpr int kStepAhead = 4;  // cells whose loads a thread has in flight

__global__ void k_timestep_reset(unsigned long long* out)
{
    if (threadIdx.x < 2) out[threadIdx.x] = 0x7FF0000000000000ull;  // +inf
}

hipError_t launch_timestep_reset(unsigned long long* out, hipStream_t s)
{
    k_timestep_reset<<<1, 64, 0, s>>>(out);
    return hipGetLastError();
}

__device__ __forceinline__ double wave_min_f64(double v)
{
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
    return v;
}

__global__ __launch_bounds__(kStepThreads) void k_timestep(TimestepArgs a)
{
    double mn = INFINITY, top = 0.0;
    const double sl = a.sigma0 * a.cell_cm;
    const uint32_t span = kStepThreads * kStepAhead;
    for (uint64_t base = blockIdx.x * (uint64_t)span; base < a.ncell; base += gridDim.x * (uint64_t)span) {
        float f_nh[kStepAhead], f_x[kStepAhead], f_x1[kStepAhead], f_x2[kStepAhead], f_T[kStepAhead], f_g[kStepAhead];
#pragma unroll
        for (int j = 0; j < kStepAhead; ++j) {
            // past the end: the last cell again, which changes no minimum
            const uint32_t c = (uint32_t)min((uint64_t)a.ncell - 1u, base + threadIdx.x + (uint64_t)j * kStepThreads);
            f_nh[j] = a.n_h[c];
            f_x[j] = a.x_hi[c];
            f_x1[j] = a.x_hei[c];
            f_x2[j] = a.x_heii[c];
            f_T[j] = a.temp[c];
            f_g[j] = a.gamma_hi[c];
        }
#pragma unroll
        for (int j = 0; j < kStepAhead; ++j) {
            const double nh = f_nh[j], nhe = a.y * nh;
            const double nhi = nh * (double)f_x[j], nhii = nh - nhi;
            const double nhei = nhe * (double)f_x1[j], nheii = nhe * (double)f_x2[j];
            double nheiii = nhe - nhei - nheii;
            if (nheiii < 0) nheiii = 0;
            const double ne = nhii + nheii + 2.0 * nheiii;
            double a_hii, k_hi = 0.0;
            if (a.rates == 0) {
                a_hii = a.alpha_hii;
            } else {
                const chem::Coef k = chem::coefficients(f_T[j]);
                a_hii = (double)k.a_hii;
                if (a.collisional) k_hi = (double)k.k_hi;
            }
            const double ndot = fabs(a_hii * ne * nhii - ((double)f_g[j] + k_hi * ne) * nhi);
            if (!(ndot > 0.0)) continue;
            const double en = a.eps * nhi;
            if (nhi * sl > 0.5 && en <= mn * ndot * (1.0 + 1e-14)) mn = fmin(mn, en / ndot);
            top = fmax(top, ndot);
        }
    }
    const double mi = top > 0.0 ? a.eps / (sl * top) : INFINITY;
    __shared__ double least[2][kStepThreads / 64];
    const double wn = wave_min_f64(mn), wi = wave_min_f64(mi);
    if ((threadIdx.x & 63) == 0) {
        least[0][threadIdx.x >> 6] = wn;
        least[1][threadIdx.x >> 6] = wi;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double v = INFINITY;
        for (int w = 0; w < kStepThreads / 64; ++w) v = fmin(v, least[threadIdx.x][w]);
        if (v < INFINITY) atomicMin(&a.out[threadIdx.x], (unsigned long long)__double_as_longlong(v));
    }
}

// The two minima as doubles into caller memory (device pointer out[2]).
__global__ void k_timestep_publish(const unsigned long long* bits, double* out)
{
    if (threadIdx.x < 2) out[threadIdx.x] = __longlong_as_double((long long)bits[threadIdx.x]);
}

hipError_t launch_timestep_publish(const unsigned long long* bits, double* out, hipStream_t s)
{
    k_timestep_publish<<<1, 64, 0, s>>>(bits, out);
    return hipGetLastError();
}

__global__ void k_timestep_end(unsigned long long* bits, double* out)
{
    if (threadIdx.x < 2) {
        out[threadIdx.x] = __longlong_as_double((long long)bits[threadIdx.x]);
        bits[threadIdx.x] = 0x7FF0000000000000ull;  // +inf
        __threadfence_system();
    }
}

hipError_t launch_timestep_end(unsigned long long* bits, double* out, hipStream_t s)
{
    k_timestep_end<<<1, 64, 0, s>>>(bits, out);
    return hipGetLastError();
}

hipError_t launch_timestep(const TimestepArgs& a, int cus, hipStream_t s)
{
    const size_t span = (size_t)kStepThreads * kStepAhead;
    const size_t want = ((size_t)a.ncell + span - 1) / span;
    const unsigned blocks = (unsigned)std::max<size_t>(1, std::min<size_t>(want, (size_t)std::max(1, cus) * 6));
    k_timestep<<<blocks, kStepThreads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace arc
