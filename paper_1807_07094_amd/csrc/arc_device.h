// arc_device.h -- device-side data layout and per-ray arithmetic shared by every
// tracing schedule of libarc (gfx950).
//
// The plain and the batched schedules call exactly these functions, so a ray deposits
// the same integers whichever schedule traces it; integer sums do not depend on order,
// which makes the fixed-point field bitwise identical across schedules and runs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace arc {

constexpr int kMaxBins = 4;
constexpr int kMaxLevels = 16;       // HEALPix levels 0..15 (pixel ids fit 28 bits to level 12)
constexpr int kLevelShift = 28;      // packed ray id: level << 28 | pixel
constexpr uint32_t kPixMask = (1u << kLevelShift) - 1u;
constexpr float kDtauTermMin = 0.01f;  // a terminating crossing must be this thick in every bin

enum Event : int { kContinue = 0, kSplit = 1, kTerminate = 2, kEscape = 3 };

constexpr uint32_t kNoCell = 0xFFFFFFFFu;
// Pointer qualifier of the LDS address space.
#define kLds __attribute__((address_space(3)))

// Cell layout of the opacity and the field: 8^3 blocks in x-fastest block order, Morton
// order inside a block, so that the 2x2x2 neighbourhood of a cell shares a 128-byte
// line of opacity (and two lines of field) and a block is 8 KB of opacity.
__host__ __device__ __forceinline__ uint32_t spread3(uint32_t v)
{
    // bits 0, 1, 2 -> 0, 3, 6: bit 2 moves by 4 first, then bits 1 and 2 by 2
    const uint32_t x = ((v << 4) | v) & 0x43u;
    return ((x << 2) | x) & 0x49u;
}
__host__ __device__ __forceinline__ uint32_t blocked_index(int x, int y, int z, int nbx8, int nby8)
{
    const uint32_t b = ((uint32_t)(z >> 3) * (uint32_t)nby8 + (uint32_t)(y >> 3)) * (uint32_t)nbx8 + (uint32_t)(x >> 3);
    const uint32_t m = spread3((uint32_t)x & 7u) | (spread3((uint32_t)y & 7u) << 1) | (spread3((uint32_t)z & 7u) << 2);
    return (b << 9) | m;
}

// Place of a cell's bin in a fixed-point field of `lines` 64-byte lines per 2x2x2 tile, line b of
// the tile holding bin b of its eight cells (the low three bits of the blocked index).
__host__ __device__ __forceinline__ size_t field_word(uint32_t cell, int lines, int b)
{
    return ((size_t)(cell >> 3) * (size_t)lines + (size_t)b) * 8u + (cell & 7u);
}

// A crossing's deposit: the cell (blocked index) and the amount of every bin in field units,
// rounded to the field's integers when the wave deposits it.
template <int NB>
struct Dep {
    uint32_t cell;        // always a valid index, also where there is nothing to deposit
    float v[NB];
};

enum Counter : int {
    kCrossings = 0, kRays, kSplits, kTerminated, kEscapedRays, kSpills, kQueueOverflow,
    kDeposits,  // 64-byte field lines added to after the wave-level merge
    kNumCounters
};
enum Photons : int { kPhotonsEscaped = 0, kPhotonsAbsorbed = kMaxBins, kPhotonsThin };  // escaped: one per bin

// Sums that every wave adds to at its end. Atomics on one line are carried out one after the
// other, about 6 ns each, so a workgroup adds to one of kCounterSlots copies and the last kernel
// sums them (256^3 x 1024 sources with one copy: the levels before the persistent launch took 10.2
// ms instead of 3.4, the rates 0.43 instead of 0.21).
constexpr int kCounterSlots = 64;
struct __align__(256) CounterSlot {
    unsigned long long n[16];  // [Counter]
    double photons[8];         // [Photons] in field units (escaped) or photons/s
    unsigned long long pad[8];
};

// A counter with a line of its own: a level's kernel reads how many rays it has while it counts
// the next level's, and such reads and atomics on one line wait for each other.
struct __align__(128) LineCount {
    uint32_t n, pad[31];
};

// When the stages of a call began (device clock): its first kernel, the trace, the persistent
// launch, the rates, and the end of the last grid pass. Kernels stamp their start: an event
// between two launches leaves the device idle for 6 to 18 us.
enum Stamp : int { kStampBegin = 0, kStampTrace, kStampPersistent, kStampRates, kStampEnd, kNumStamps };

// The device's side of one call, in one block, cleared by its first kernel (but for the stamps).
struct RunBlock {
    CounterSlot before[kCounterSlots];      // everything but the persistent launch
    CounterSlot persistent[kCounterSlots];
    LineCount level_rays[kMaxLevels];       // rays (or families) waiting at each level
    LineCount head;                         // work queue: items taken after the waves' first
    int32_t errflag;                        // grid values out of range
    unsigned long long tree_count;
    unsigned long long stamp[kNumStamps];
};

// What the host reads of it, written to pinned memory by the call's last kernel.
struct RunResult {
    unsigned long long n[kNumCounters], persistent[kNumCounters];
    double photons[8];
    unsigned long long stamp[kNumStamps];
    unsigned long long tree_count;
    int32_t errflag;
};

// The kernel's start into *stamp (if given), by its first workgroup.
__device__ __forceinline__ void stamp_start(unsigned long long* stamp)
{
    if (stamp && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *stamp = wall_clock64();
}

// Per-source constants (section 2.1 keeps the source position on chip; here it is a
// 32-byte record read through L2 once per ray).
struct __align__(16) SourceRec {
    float x, y, z;        // position on the 2^-12 lattice (exact in FP32 up to 2048 cells)
    float r_thin;         // optically thin radius (section 2.6): rays start at this radius
    float scale[4];       // ndot * frac_b / (12 * u_J,b): root-ray photon rate in field units
};

// A ray waiting to be traced: its identity and the optical depth it carries. The start
// radius follows from the level (0 for roots, the parent's split radius for children).
struct __align__(16) RayRec {
    uint32_t src;
    uint32_t lp;          // level << 28 | nested pixel
    uint32_t pad0, pad1;
    float tau[4];         // optical depth per bin (high part)
    float taulo[4];       // compensation terms
};

// The same ray in the compact form kept on a wave's stack (32 bytes for three bins).
template <int NB>
struct StackRec {
    uint32_t src;
    uint32_t lp;
    float tau[NB];
    float taulo[NB];
};

struct TraceArgs {
    int nx, ny, nz, nb;
    int nbx8, nby8;            // 8^3 blocks per row and per column of the cell layout
    int level0, lmax;
    float tsplit[kMaxLevels];  // split radius of each level; +inf from lmax on
    float tau_term;            // +inf = never terminate
    const float* kappa1;       // nb == 1: optical depth per cell length, [cell] (blocked order)
    const float4* kappa4;      // nb > 1: [cell] (bins in x, y, z, w) (blocked order)
    unsigned long long* J;     // fixed-point field [tile][nb][8] (blocked order, field_word)
    const SourceRec* src;
    const float4* dirs;        // HEALPix centres of every level, concatenated
    long long dir_off[kMaxLevels];
    CounterSlot* slots;        // [kCounterSlots]
    unsigned long long* stamp; // where the launch notes its start, or null
    unsigned long long* tree;  // optional record of every ray traced
    unsigned long long* tree_count;
    long long tree_cap;
    int corr;                  // geometric correction: 0 none, 1 f_c, 2 f_c + secondary, 3 f_c^2
    // corr == 2: photons moved into a cell by the secondary correction (eq:correction2), in two
    // limbs per bin, [tile][limb][nb][8]: limb 0 in units of 2^20 u_J,b, limb 1 in units of
    // 2^-12 u_J,b
    unsigned long long* M;
    // optically thin approximation (section 2.6): the bin of lowest photon energy, and per
    // source the least path length at which a ray's depth in it reaches kTauThin (FP32 bits)
    int ksoft;
    unsigned int* r_out;
};

constexpr float kTauThin = 0.1f;  // optical depth that bounds the optically thin sphere

// The blocked cell index is the sum of one term per axis. Every workgroup that traces keeps the
// terms of the three axes in LDS, axis after axis, each between two entries that stand for
// "outside the grid" (nx + ny + nz + 6 words), and a ray carries the addresses of its cell's three
// entries: a step moves one address, and the index costs three LDS reads and an add (computing
// a term takes ten VALU instructions, which bound the trace).
typedef const volatile kLds char* TermAddr;
constexpr uint32_t kOutside = 0x80000000u;  // indices are below 2^31

struct Terms {
    TermAddr base[3];      // entry of coordinate 0 along each axis
};

__device__ __forceinline__ uint32_t term_at(TermAddr p) { return *(const volatile kLds uint32_t*)p; }

// Per-lane ray state. Along axis i the ray meets its next cell boundary at
// t_i = a_i / e_i, where e_i = |d_i| and a_i is the (exact, lattice-valued) distance of
// that boundary from the source; crossing the boundary adds 1 to a_i.
template <int NB>
struct Ray {
    float e[3];           // |d_i|
    float ie[3];          // 1 / |d_i| (hardware reciprocal, within 1 ulp), +inf if d_i == 0
    float a[3];           // next-boundary distance along each axis (exact)
    TermAddr o[3];        // index term of the current cell along each axis
    int step[3];          // bytes to the next cell's term: +4, -4 or 0
    float thi, tlo;       // current path length (double-float)
    float tend;           // split radius or +inf
    float tlim;           // just below the split radius and the way out of the grid
    float tau[NB], taulo[NB];
    float w[NB];          // scale_b * 4^-level
    uint32_t src, lp;
};

// Counts of a wave (wave-uniform, from ballots), its lanes' crossings, and the photons they
// carried out of the grid, in LDS (the registers are worth more: they bound the occupancy).
struct WaveStats {
    unsigned long long rays, splits, terminated, escaped;
    uint32_t crossings;    // per lane
    kLds double* esc;      // [kMaxBins]
    __device__ void clear(kLds double* lds)
    {
        rays = splits = terminated = escaped = 0;
        crossings = 0;
        esc = lds;
        if ((threadIdx.x & 63) < kMaxBins) esc[threadIdx.x & 63] = 0.0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __device__ __forceinline__ void lose(int b, double photons)
    {
        __hip_atomic_fetch_add(esc + b, photons, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
};

__device__ __forceinline__ CounterSlot& my_slot(CounterSlot* slots)
{
    return slots[(blockIdx.x + blockIdx.y) & (kCounterSlots - 1)];
}

__device__ __forceinline__ unsigned long long count_lanes(bool p) { return (unsigned long long)__popcll(__builtin_amdgcn_ballot_w64(p)); }

// ---------------------------------------------------------------------------------
// Exact arithmetic helpers. All operands are non-negative FP32 values.
// ---------------------------------------------------------------------------------

// sign(a*b - c*d), exact: products are split into rounded value and FMA remainder.
__device__ __forceinline__ int cmp_prod(float a, float b, float c, float d)
{
    const float p = a * b, q = c * d;
    if (p != q) return p < q ? -1 : 1;
    const float ep = __builtin_fmaf(a, b, -p), eq = __builtin_fmaf(c, d, -q);
    return ep < eq ? -1 : (ep > eq ? 1 : 0);
}

// Cell index along one axis that the ray occupies just after path length t0:
// x = xs + t0*d. Exact: t0*d is split into a rounded part and its FMA remainder, and
// k - xs is exact on the lattice, so (xs + t0 d) vs k is decided without rounding.
// d > 0: a point on a boundary belongs to the upper cell; d < 0: to the lower cell;
// d == 0: to the upper cell.
__device__ __forceinline__ int start_index(float xs, float t0, float d)
{
    if (d == 0.0f) return (int)floorf(xs);
    const float ph = t0 * d;
    const float pl = __builtin_fmaf(t0, d, -ph);
    int k = (int)floorf(xs + ph);
    // sign((xs + t0 d) - k)
    auto side = [&](int kk) -> int {
        const float m = (float)kk - xs;
        if (ph != m) return ph > m ? 1 : -1;
        return pl > 0.0f ? 1 : (pl < 0.0f ? -1 : 0);
    };
    if (d > 0.0f) {
        while (side(k) < 0) --k;
        while (side(k + 1) >= 0) ++k;
    } else {
        while (side(k) <= 0) --k;
        while (side(k + 1) > 0) ++k;
    }
    return k;
}

// Per-axis terms of blocked_index(): index = term(x, 0) + term(y, 1) + term(z, 2).
__device__ __forceinline__ uint32_t axis_term(const TraceArgs& A, int i, int v)
{
    // grids are at most 2048 cells per axis: the block's first cell index along the axis is
    // below 2^17 and the blocks it stands for below 2^17; with those ranges stated the multiply
    // is the full-rate 24-bit one
    const uint32_t blk9 = ((uint32_t)v << 6) & 0x1FE00u;
    const uint32_t m = spread3((uint32_t)v & 7u) << i;
    if (i == 0) return blk9 + m;
    if (i == 1) return blk9 * ((uint32_t)A.nbx8 & 0x1FFFFu) + m;
    return blk9 * (((uint32_t)A.nbx8 * (uint32_t)A.nby8) & 0x1FFFFu) + m;
}

// Fills the workgroup's table of index terms (nx + ny + nz + 6 words at `table`); all threads of
// the workgroup call it, and a barrier follows before the first use.
__device__ __forceinline__ Terms make_terms(const TraceArgs& A, uint32_t* table)
{
    Terms t;
    const int n[3] = {A.nx, A.ny, A.nz};
    int from = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        for (int k = (int)threadIdx.x - 1; k <= n[i]; k += (int)blockDim.x)
            table[from + 1 + k] = k < 0 || k == n[i] ? kOutside : axis_term(A, i, k);
        t.base[i] = (TermAddr)(table + from + 1);
        from += n[i] + 2;
    }
    return t;
}

// Non-negative float to the nearest int64 (v < 2^63): two exact 32-bit halves.
__device__ __forceinline__ long long round_to_i64(float v)
{
    const float r = rintf(v);
    const float hi = floorf(r * 2.3283064365386963e-10f);   // r / 2^32, exact scaling
    const float lo = __builtin_fmaf(-hi, 4294967296.0f, r);  // exact remainder in [0, 2^32)
    return (long long)(((unsigned long long)(uint32_t)hi << 32) | (unsigned long long)(uint32_t)lo);
}

// e^-tau with the hardware exponential (relative error ~1e-6 for tau up to ~80).
__device__ __forceinline__ float transmission(float tau) { return __builtin_amdgcn_exp2f(-tau * 1.4426950408889634f); }

// ---------------------------------------------------------------------------------
// Per-ray operations.
// ---------------------------------------------------------------------------------

template <int NB>
__device__ __forceinline__ void record_tree(const TraceArgs& A, uint32_t src, uint32_t lp)
{
    if (A.tree) {
        const unsigned long long i = atomicAdd(A.tree_count, 1ull);
        if ((long long)i < A.tree_cap) A.tree[i] = ((unsigned long long)src << 32) | lp;
    }
}

// Load a ray: direction, source, start radius and start cell (section 2.1 iii a/c:
// roots at radius 0, children at the parent's radius with their own direction). With the
// optically thin approximation (THIN, section 2.6) a ray starts no closer than its source's
// thin radius; a ray whose split radius does not lie beyond that start splits at once (it is
// returned active with thi >= tend and crosses nothing).
// Returns false (and books the escape's photons; the caller counts it and, with THIN, books the
// bound `reach`) when the start point lies outside the grid.
template <int NB, bool THIN, class Rec>
__device__ __forceinline__ bool ray_init(const TraceArgs& A, const Terms& terms, const Rec& r, Ray<NB>& ray,
                                         WaveStats& st, float& reach)
{
    ray.src = r.src;
    ray.lp = r.lp;
    const int level = (int)(r.lp >> kLevelShift);
    const uint32_t pix = r.lp & kPixMask;
    const float4 dv = A.dirs[A.dir_off[level] + pix];
    const float d[3] = {dv.x, dv.y, dv.z};
    const SourceRec s = A.src[r.src];
    const float xs[3] = {s.x, s.y, s.z};
    float t0 = level == A.level0 ? 0.0f : A.tsplit[level - 1];
    if constexpr (THIN) t0 = fmaxf(t0, s.r_thin);
    ray.thi = t0;
    ray.tlo = 0.0f;
    ray.tend = A.tsplit[level];
    const float lw = __builtin_ldexpf(1.0f, -2 * level);  // 4^-level, exact
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        ray.tau[b] = r.tau[b];
        ray.taulo[b] = r.taulo[b];
        ray.w[b] = s.scale[b] * lw;
    }
    if constexpr (THIN) {
        if (!(t0 < ray.tend)) return true;  // splits at once
    }
    bool inside = true;
    float texit = ray.tend;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int c = start_index(xs[i], t0, d[i]);
        const int n = i == 0 ? A.nx : (i == 1 ? A.ny : A.nz);
        ray.o[i] = terms.base[i] + 4 * c;
        ray.e[i] = fabsf(d[i]);
        ray.ie[i] = d[i] != 0.0f ? __builtin_amdgcn_rcpf(ray.e[i]) : INFINITY;
        ray.step[i] = d[i] > 0.0f ? 4 : (d[i] < 0.0f ? -4 : 0);
        // d_i = 0: the distance to the upper face (no boundary is met along this axis; the
        // geometric correction reads the position from it)
        ray.a[i] = d[i] < 0.0f ? xs[i] - (float)c : (float)(c + 1) - xs[i];
        // the wall of the grid along this axis is met at the float product the traversal will form
        const float wall = d[i] < 0.0f ? xs[i] : (float)n - xs[i];
        texit = fminf(texit, d[i] != 0.0f ? wall * ray.ie[i] : INFINITY);
        inside = inside && c >= 0 && c < n;
    }
    ray.tlim = texit * 0.999998f;
    if (!inside) {
        float ts = 0.0f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float tb = ray.tau[b] + ray.taulo[b];
            st.lose(b, (double)ray.w[b] * (double)transmission(tb));
            if (b == A.ksoft) ts = tb;
        }
        // a ray that starts outside the grid while still thin bounds the thin radius by its start
        if constexpr (THIN)
            if (ts < kTauThin) reach = t0;
    }
    return inside;
}

template <int NB>
__device__ __forceinline__ void kappa_at(const TraceArgs& A, uint32_t cell, float k[NB])
{
    if constexpr (NB == 1) {
        k[0] = A.kappa1[cell];
    } else {
        const float4 v = A.kappa4[cell];
        k[0] = v.x;
        k[1] = v.y;
        if constexpr (NB > 2) k[2] = v.z;
        if constexpr (NB > 3) k[3] = v.w;
    }
}

// A piece of a ray inside one cell: blocked cell index and length.
struct Seg {
    uint32_t cell;
    float ds;
    uint32_t nb;  // geometric correction: neighbour that receives the moved share (kNoCell: none)
    float fc;     // geometric correction: share the cell keeps (1: uncorrected)
    float t1;     // path length at the segment's end (high part)
};

constexpr double kSqrtPiOver3 = 1.0233267079464885;  // width of a level-0 pixel per unit radius
// Face distances within this many cells count as tied: symmetric geometries tie exactly,
// and the last bits of a midpoint depend on how its path length was summed.
constexpr double kFaceTie = 1e-9;

// The correction a kernel is built for: none, the cell's share alone (modes 1 and 3), or with
// the rest moved to a neighbour (mode 2).
enum Corr : int { kCorrNone = 0, kCorrShare, kCorrMove };

// Geometric correction of the segment [t, t_next) in the ray's current cell (section 2.5,
// eq:correction): D_edge is the distance from the segment's midpoint to the nearest face of
// the cell, L_Pix the width of the ray's pixel there (r sqrt(4 pi / N_pix)); the cell keeps
// f_c = 1/2 + D_edge / L_Pix of the crossing's photons when D_edge < L_Pix / 2 (mode 3: f_c
// squared). Mode 2 also names the neighbour across that face, which receives the rest
// (eq:correction2); without one inside the grid the cell keeps everything. Distances in
// FP64 from the exact boundary numerators; faces within kFaceTie count as tied, and ties go
// to the lower axis, then the lower face.
template <int CORR, int NB>
__device__ __forceinline__ void geom_correction(const TraceArgs& A, const Ray<NB>& ray, float nhi, float nlo, Seg& sg)
{
    sg.nb = kNoCell;
    sg.fc = 1.0f;
    const double tm = 0.5 * (((double)ray.thi + (double)ray.tlo) + ((double)nhi + (double)nlo));
    const int level = (int)(ray.lp >> kLevelShift);
    const double lpix = tm * __builtin_ldexp(kSqrtPiOver3, -level);
    double dmin = INFINITY;
    int axis = 0, side = -1;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        // distance to the face the ray heads for (the upper face when d_i = 0)
        const double ahead = (double)ray.a[i] - tm * (double)ray.e[i];
        const bool up = ray.step[i] >= 0;
        const double hi = up ? ahead : 1.0 - ahead;
        const double lo = up ? 1.0 - ahead : ahead;
        const bool upper = hi < lo - kFaceTie;
        const double di = upper ? hi : lo;
        if (di < dmin - kFaceTie) {
            dmin = di;
            axis = i;
            side = upper ? 1 : -1;
        }
    }
    if (!(dmin < 0.5 * lpix)) return;
    // the decisions above are FP64; the share itself needs FP32 only
    float fc = 0.5f + (float)dmin * __builtin_amdgcn_rcpf((float)lpix);
    if (CORR == kCorrShare && A.corr == 3) fc *= fc;
    if constexpr (CORR == kCorrMove) {
        // the neighbour's per-axis term replaces the cell's along `axis`
        const TermAddr o0 = ray.o[0], o1 = ray.o[1], o2 = ray.o[2];
        const TermAddr oc = axis == 0 ? o0 : (axis == 1 ? o1 : o2);
        const uint32_t there = term_at(oc + 4 * side);
        if (there & kOutside) return;  // no neighbour inside: the cell keeps everything
        sg.nb = sg.cell - term_at(oc) + there;
    }
    sg.fc = fc;
}

// Geometry of the next segment (section 2.4: the step to the next x, y or z boundary, or
// to the split radius), advancing the ray's position and cell. Returns what happens at its end
// (kContinue: next cell; kSplit: the split radius; kEscape: the ray leaves the grid).
//
// Geometric decisions are exact: boundary times are compared through the reciprocal
// products a_i / e_i, whose relative error is below 2e-7, and any comparison closer than
// 1e-6 is settled exactly with cmp_prod (a_i e_j vs a_j e_i). The middle of the three times
// says whether any comparison is that close. The split radius and the grid's walls are looked
// at only within 2e-6 of the nearer of them (tlim): a boundary met before that is neither, so
// an ordinary step is about thirty instructions (a bundle's lanes reach their ends together).
// `term` receives the cell's index terms, whose sum the caller forms later (they come from LDS).
template <int NB, int PREC, int CORR = kCorrNone>
__device__ __forceinline__ int geom_next(const TraceArgs& A, Ray<NB>& ray, Seg& sg, uint32_t (&term)[3])
{
    constexpr float kNear = 1.000001f;
    // values of their own: a select between members of the ray is turned into an indexed access
    // to it, which would move it to scratch memory
    const float a0 = ray.a[0], a1 = ray.a[1], a2 = ray.a[2];
    const float e0 = ray.e[0], e1 = ray.e[1], e2 = ray.e[2];
    // a_i > 0 always, and ie_i = +inf where d_i = 0, so those axes give t_i = +inf
    const float t0 = a0 * ray.ie[0];
    const float t1 = a1 * ray.ie[1];
    const float t2 = a2 * ray.ie[2];
    float tw = fminf(fminf(t0, t1), t2);
    // axes whose boundary the step crosses
    bool m0 = t0 <= tw, m1 = t1 <= tw, m2 = t2 <= tw;
    if constexpr (PREC == 0) {
        if (__builtin_amdgcn_fmed3f(t0, t1, t2) <= tw * kNear) {
            // exact argmin and ties: t_i < t_j  <=>  a_i e_j < a_j e_i (an axis with e = 0 has no
            // boundary)
            float ab = a0, eb = e0;
            tw = t0;
            if (e1 > 0.0f && (!(eb > 0.0f) || cmp_prod(a1, eb, ab, e1) < 0)) {
                ab = a1;
                eb = e1;
                tw = t1;
            }
            if (e2 > 0.0f && (!(eb > 0.0f) || cmp_prod(a2, eb, ab, e2) < 0)) {
                ab = a2;
                eb = e2;
                tw = t2;
            }
            m0 = e0 > 0.0f && cmp_prod(a0, eb, ab, e0) == 0;
            m1 = e1 > 0.0f && cmp_prod(a1, eb, ab, e1) == 0;
            m2 = e2 > 0.0f && cmp_prod(a2, eb, ab, e2) == 0;
        }
    }
    const bool lim = tw >= ray.tlim;
    bool at_end = false;
    if (lim) {
        asm volatile("");
        if constexpr (PREC == 0) {
            const float aw = m0 ? a0 : (m1 ? a1 : a2);
            const float ew = m0 ? e0 : (m1 ? e1 : e2);
            at_end = !(ray.tend > tw * kNear) && (ray.tend * kNear < tw || cmp_prod(ray.tend, ew, aw, 1.0f) <= 0);
        } else {
            at_end = ray.tend <= tw;
        }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) term[i] = term_at(ray.o[i]);
    if constexpr (CORR) sg.cell = term[0] + term[1] + term[2];
    // next path length as a double-float: the low part from the lowest crossed axis. With the
    // correction the position must not move before its distances are taken.
    float nhi = tw, nlo = 0.0f;
    auto low = [&](int i) { return __builtin_fmaf(-tw, ray.e[i], ray.a[i]) * ray.ie[i]; };
    if constexpr (CORR) {
        if (m2) nlo = low(2);
        if (m1) nlo = low(1);
        if (m0) nlo = low(0);
        geom_correction<CORR>(A, ray, at_end ? ray.tend : nhi, at_end ? 0.0f : nlo, sg);
    }
    // one axis after the other under its own lanes (branches, not selects: half the instructions)
    if (m2) {
        asm volatile("");
        if constexpr (PREC == 0 && !CORR) nlo = low(2);
        ray.a[2] += 1.0f;
        ray.o[2] += ray.step[2];
    }
    if (m1) {
        asm volatile("");
        if constexpr (PREC == 0 && !CORR) nlo = low(1);
        ray.a[1] += 1.0f;
        ray.o[1] += ray.step[1];
    }
    if (m0) {
        asm volatile("");
        if constexpr (PREC == 0 && !CORR) nlo = low(0);
        ray.a[0] += 1.0f;
        ray.o[0] += ray.step[0];
    }
    int ev = kContinue;
    if (lim) {
        asm volatile("");
        if (at_end) {
            nhi = ray.tend;
            nlo = 0.0f;
            ev = kSplit;
        } else if ((term_at(ray.o[0]) | term_at(ray.o[1]) | term_at(ray.o[2])) & kOutside) {
            ev = kEscape;
        }
    }
    // ds = t_next - t_cur. The difference's rounding error in three operations: exact where
    // nhi >= thi, and where rounding put nhi below thi the difference itself is exact.
    if constexpr (PREC == 0) {
        const float s = nhi - ray.thi;
        const float err = -ray.thi - (s - nhi);
        sg.ds = s + (err + (nlo - ray.tlo));
    } else {
        sg.ds = nhi - ray.thi;
    }
    sg.t1 = nhi;
    ray.thi = nhi;
    ray.tlo = nlo;
    return ev;
}

// Section 2.6: the least path length at which the ray's depth in the softest bin reaches
// kTauThin, within this segment (ts: depth at its start, dts: its increment, ks: its
// opacity), bounds the source's thin radius. FP32 start plus increment can round to kTauThin where
// the compensated sum stays below it, so a ray may reach it twice: the lesser length counts.
__device__ __forceinline__ void thin_reach(const Seg& sg, float ts, float dts, float ks, float& reach)
{
    if (ts < kTauThin && ts + dts >= kTauThin) reach = fminf(reach, (sg.t1 - sg.ds) + (kTauThin - ts) / ks);
}

// Bounds of the wave's lanes (+inf: none) on their sources' thin radii. Called by all 64 lanes.
// Atomics on one word go one after the other, and every ray of a source has one: the lanes of a
// source (mostly all of them) are reduced first, and a bound that the word already holds is
// dropped (a stale read of it is only larger). 128^3 x 32 sources: the levels before the
// persistent launch 870 us with an atomic per ray.
__device__ __forceinline__ void thin_bounds(const TraceArgs& A, uint32_t src, float reach)
{
    uint64_t left;
    while ((left = __builtin_amdgcn_ballot_w64(reach < INFINITY)) != 0) {
        const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)src, __builtin_ctzll(left));
        float m = src == s ? reach : INFINITY;
        for (int off = 32; off > 0; off >>= 1) m = fminf(m, __shfl_xor(m, off, 64));
        if ((threadIdx.x & 63) == 0) {
            const uint32_t bits = __float_as_uint(m);
            if (bits < __hip_atomic_load(A.r_out + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(A.r_out + s, bits);
        }
        if (src == s) reach = INFINITY;
    }
}

// Bins of a pass that can still add to the field (wave-uniform, one bit per bin). A bin whose
// photons are all but gone in every lane is left out: with photons S = w T at the start of the
// pass a crossing adds at most S ds <= sqrt(3) S, or 173 S more where it terminates, which
// rounds to zero field units once S is below kLiveMin, and S only falls. With the geometric
// correction the largest of a crossing's deposits is 2 S 2^12 (the moved photons' low limb) or
// 16 (sqrt(3) + 173) S. Optical depths are kept for every bin (termination, escape and children
// need them). The soft bins go first: 256^3 x 1024 sources 50.3 ms with all three bins to the
// end, 45.7 with the live ones (three waves per SIMD).
constexpr float kLiveMin = 0.0009765625f;             // 2^-10
constexpr float kLiveMinCorr = 0.000030517578125f;    // 2^-15
template <int NB>
__device__ __forceinline__ uint32_t live_bins(const Ray<NB>& ray, bool active, const float (&T)[NB], float least)
{
    uint32_t live = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) live |= __builtin_amdgcn_ballot_w64(active && ray.w[b] * T[b] >= least) ? 1u << b : 0u;
    return live;
}

// The hardware's maximum and minimum, without the canonicalisation that fmaxf and fminf add.
__device__ __forceinline__ float max_raw(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float min_raw(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Photons of one segment (section 2.4, eq:ion per bin): the amount v_b = S ds g(dtau) for the
// cell in field units, attenuation (compensated tau), then the termination test (a
// terminating crossing adds the rest of the photons, S / kappa, to v_b) and, with THIN, the
// thin-radius measurement. T_b carries the transmission e^-tau_b from one segment to the next
// (one exponential per bin and crossing): with S = w T_b the photons entering the cell, the
// cell absorbs S (1 - e^-dtau) = w (T_b - T'_b), so v_b = w (T_b - T'_b) / kappa_b, and below
// dtau = 0.25, where that difference would cancel, S ds g(dtau) with g's Taylor series
// (truncation < 5e-8 relative). v_b and T_b are kept for the live bins only. Returns whether
// the ray terminates here.
template <int NB, int PREC, bool THIN>
__device__ __forceinline__ bool attenuate_seg(const TraceArgs& A, Ray<NB>& ray, const Seg& sg, const float kap[NB],
                                              uint32_t live, float v[NB], float (&T)[NB], float& reach)
{
    float ts = 0.0f, dts = 0.0f, ks = 1.0f;
    float dtau[NB], taup[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        dtau[b] = kap[b] * sg.ds;
        if constexpr (THIN) {
            if (b == A.ksoft) {
                ts = PREC == 0 ? ray.tau[b] + ray.taulo[b] : ray.tau[b];
                dts = dtau[b];
                ks = kap[b];
            }
        }
        if constexpr (PREC == 0) {
            // the sum's rounding error, exact from the larger of the two terms
            const float hi = max_raw(ray.tau[b], dtau[b]), lo = min_raw(ray.tau[b], dtau[b]);
            ray.tau[b] = hi + lo;
            ray.taulo[b] += lo - (ray.tau[b] - hi);
        } else {
            ray.tau[b] += dtau[b];
        }
        taup[b] = PREC == 0 ? ray.tau[b] + ray.taulo[b] : ray.tau[b];
    }
    float least = taup[0], thin = dtau[0];
#pragma unroll
    for (int b = 1; b < NB; ++b) {
        least = fminf(least, taup[b]);
        thin = fminf(thin, dtau[b]);
    }
    // (tau_term is +inf where rays never terminate)
    const bool term = least >= A.tau_term && thin >= kDtauTermMin && A.tau_term < INFINITY;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (!(live & (1u << b))) continue;
        asm volatile("");  // a branch, not selects: the point is to skip the work
        const float Tn = transmission(taup[b]);
        // 1 / kappa (hardware reciprocal): used where dtau >= 0.25 or on termination (dtau >= 0.01)
        const float rk = __builtin_amdgcn_rcpf(kap[b]), x = dtau[b];
        const float g = __builtin_fmaf(
            x, __builtin_fmaf(x, __builtin_fmaf(x, __builtin_fmaf(x, __builtin_fmaf(x, -1.0f / 720.0f, 1.0f / 120.0f), -1.0f / 24.0f), 1.0f / 6.0f), -0.5f),
            1.0f);
        const float series = ((ray.w[b] * T[b]) * sg.ds) * g;
        const float lost = (ray.w[b] * (T[b] - Tn)) * rk;
        v[b] = x < 0.25f ? series : lost;
        T[b] = Tn;
    }
    if (term) {
        asm volatile("");
        // absorb what is left in this cell: field += remaining photons / opacity
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (!(live & (1u << b))) continue;
            v[b] = __builtin_fmaf(ray.w[b] * T[b], __builtin_amdgcn_rcpf(kap[b]), v[b]);
        }
    }
    if constexpr (THIN) thin_reach(sg, ts, dts, ks, reach);
    return term;
}

// Transmission e^-tau of every bin of a ray at its current depth.
template <int NB, int PREC>
__device__ __forceinline__ void ray_transmission(const Ray<NB>& ray, float (&T)[NB])
{
#pragma unroll
    for (int b = 0; b < NB; ++b) T[b] = transmission(PREC == 0 ? ray.tau[b] + ray.taulo[b] : ray.tau[b]);
}

// A lane's event of the pass into the wave's counts; the photons an escaping lane carried out of
// the grid go into the FP64 ledger.
template <int NB, int PREC, bool THIN>
__device__ __forceinline__ void book_events(const TraceArgs& A, int ev, const Ray<NB>& ray, float reach, WaveStats& st)
{
    st.splits += count_lanes(ev == kSplit);
    st.terminated += count_lanes(ev == kTerminate);
    st.escaped += count_lanes(ev == kEscape);
    if (ev == kEscape) {
        float T[NB];
        ray_transmission<NB, PREC>(ray, T);
#pragma unroll
        for (int b = 0; b < NB; ++b) st.lose(b, (double)(ray.w[b] * T[b]));
        // a ray that leaves the grid while still thin bounds the thin radius by its exit
        if constexpr (THIN) {
            float tsp = 0.0f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if (b == A.ksoft) tsp = PREC == 0 ? ray.tau[b] + ray.taulo[b] : ray.tau[b];
            if (tsp < kTauThin) reach = fminf(reach, ray.thi);
        }
    }
    if constexpr (THIN) thin_bounds(A, ray.src, reach);
}

// Limbs of the moved-photon field: mv = hi 2^20 + lo 2^-12 (units of u_J,b). A crossing's lo
// is below 2^32, so the limb holds 2^31 crossings; hi is bounded like the field.
constexpr float kMovedHiUnit = 1048576.0f;      // 2^20
constexpr float kMovedLoScale = 4096.0f;        // 2^12

// Integer deposit of an amount v in field units: the field's own integers (kWhole), or the
// high or low limb of the moved-photon field, hi = floor(v / 2^20) (an integer float) and the
// rest, v - hi 2^20 (exact: the bits of v below 2^20), in units of 2^-12, rounded.
enum Limb : int { kWhole = 0, kMovedHi = 1, kMovedLo = 2 };
template <int LIMB>
__device__ __forceinline__ long long to_fixed(float v)
{
    if constexpr (LIMB == kWhole) {
        return round_to_i64(v);
    } else {
        const float hi = floorf(v * (1.0f / kMovedHiUnit));
        if constexpr (LIMB == kMovedHi) return round_to_i64(hi);
        return (long long)(uint32_t)rintf(__builtin_fmaf(-hi, kMovedHiUnit, v) * kMovedLoScale);
    }
}

// Opacity ratio up to which the conserving correction's moved share enters the neighbour's
// field directly (beyond it, as photons in the two-limb field M).
constexpr float kMovedRatioJ = 16.0f;

// A segment's deposits with the geometric correction (section 2.5), mode 2: the cell keeps fc of the
// crossing's photons (the termination remainder included). The rest goes to the
// neighbour sg.nb, absorbed there at the neighbour's opacity (eq:correction2, the absorber
// ratio per bin as the opacity ratio kappa / kappa_nb), whatever that ratio. Up to a ratio of
// kMovedRatioJ it enters the neighbour's field directly, (1 - fc) v kappa / kappa_nb (dj);
// beyond it the moved photons, (1 - fc) v kappa (bounded by the ray's own), go to the
// two-limb field M (dm) and are divided by kappa_nb when the rates are formed. A neighbour
// with no absorber of the bin (kappa_nb = 0) leaves the share in the cell. dj and dm name the
// neighbour only when some bin uses them.
template <int NB, int PREC, bool THIN>
__device__ __forceinline__ bool deposit_seg_move(const TraceArgs& A, Ray<NB>& ray, const Seg& sg, const float kap[NB],
                                                 const float kapn[NB], uint32_t live, Dep<NB>& dep, Dep<NB>& dj,
                                                 Dep<NB>& dm, bool& use_j, bool& use_m, float (&T)[NB], float& reach)
{
    float v[NB];
    const bool term = attenuate_seg<NB, PREC, THIN>(A, ray, sg, kap, live, v, T, reach);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (!(live & (1u << b))) continue;
        float keep = v[b], mj = 0.0f, mm = 0.0f;
        if (sg.fc < 1.0f) {
            if (sg.nb == kNoCell) {
                // (never: a share is moved only where there is a neighbour. With the branch 192^3 x 128
                // sources take 8.03 ms, without it 8.75, though two registers are spilled and not nine)
                keep = sg.fc * v[b];
            } else if (kapn[b] > 0.0f) {
                keep = sg.fc * v[b];
                const float moved = (1.0f - sg.fc) * v[b];
                if (kap[b] <= kMovedRatioJ * kapn[b]) {
                    mj = moved * (kap[b] / kapn[b]);
                    use_j = true;
                } else {
                    mm = moved * kap[b];
                    use_m = true;
                }
            }
        }
        dep.v[b] = keep;
        dj.v[b] = mj;
        dm.v[b] = mm;
    }
    return term;
}

// Modes 1 and 3: the cell keeps fc of the crossing's photons, the removed share is dropped.
template <int NB, int PREC, bool THIN>
__device__ __forceinline__ bool deposit_seg_share(const TraceArgs& A, Ray<NB>& ray, const Seg& sg, const float kap[NB],
                                                  uint32_t live, Dep<NB>& dep, float (&T)[NB], float& reach)
{
    float v[NB];
    const bool term = attenuate_seg<NB, PREC, THIN>(A, ray, sg, kap, live, v, T, reach);
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (live & (1u << b)) dep.v[b] = sg.fc < 1.0f ? sg.fc * v[b] : v[b];
    return term;
}

// Segments whose geometry is computed ahead of their deposits (opacity loads in flight per
// lane), all deposited in one merge window. The trace is a long mix of VALU, scalar, LDS and
// branch instructions per wave, so what counts beside their number is how many waves a SIMD has
// to fill the gaps: eight ahead fit the 128 registers of four waves. 256^3 x 1024 sources,
// persistent launch: three waves and twelve ahead 28.9 ms; four waves and eight ahead with
// windows of eight 24.3 (0.096 field lines per crossing), of four 24.9 (0.115); six ahead 25.0,
// five 25.9; five waves and four ahead spill registers, 35. With thin spheres and where the
// correction drops the rest six ahead, with the neighbours' opacities three. With three bins those
// kernels spill: 4 registers with thin spheres, 9 with neighbours (16 with both), 31 with thin
// spheres in the modes that drop the rest; with one, two and four bins none.
constexpr int kSegAhead = 8;
constexpr int kSegAheadThin = 6;
constexpr int kSegAheadMove = 3, kSegAheadShare = 6;
template <int CORR, bool THIN>
constexpr int seg_ahead()
{
    return CORR == kCorrMove ? kSegAheadMove : CORR == kCorrShare ? kSegAheadShare : THIN ? kSegAheadThin : kSegAhead;
}

// Up to K crossings of one lane per pass: the geometry of K segments is computed first
// and their opacities are loaded together (K loads in flight per lane), then the
// segments are deposited in order, the wave's together. With THIN, a lane whose ray starts at or beyond its split radius (inside
// the source's thin sphere) splits at once, without a crossing.
// Returns the lane's final event of the pass (kContinue if the ray goes on).
template <int NB, int PREC, int K, bool THIN, class Depositor>
__device__ __forceinline__ int trace_pass(const TraceArgs& A, Ray<NB>& ray, bool active, WaveStats& st,
                                          Depositor& deposit)
{
    Seg sg[K];
    int nseg = 0;  // segments of the lane (a count, not K lane masks: those spill)
    bool go = active;
    int ev = kContinue;
    if constexpr (THIN) {
        if (active && !(ray.thi < ray.tend)) {
            go = false;
            ev = kSplit;
        }
    }
    // the index terms of a segment are summed one segment later, when they have come from LDS; a
    // lane without the segment keeps older ones (or zero): a valid cell to read
    uint32_t term[2][3] = {{0u, 0u, 0u}, {0u, 0u, 0u}};
#pragma unroll
    for (int j = 0; j <= K; ++j) {
        if (j < K) {
            if (go) {
                ev = geom_next<NB, PREC>(A, ray, sg[j], term[j & 1]);
                nseg = j + 1;
                go = ev == kContinue;
            }
        }
        if (j > 0) {
            const uint32_t(&t)[3] = term[(j - 1) & 1];
            sg[j - 1].cell = t[0] + t[1] + t[2];
        }
    }
    // the gathers are issued unconditionally, so that no branch separates them and each deposit waits for its own gather only
    float kap[K][NB];
#pragma unroll
    for (int j = 0; j < K; ++j) kappa_at<NB>(A, sg[j].cell, kap[j]);
    float T[NB];
    ray_transmission<NB, PREC>(ray, T);
    const uint32_t live = live_bins<NB>(ray, active, T, kLiveMin);
    // every gather is consumed before the pass issues its first atomic (a wait for a gather
    // issued before an unknown number of atomics would wait for all of them)
    Dep<NB> dep[K];
    float reach = INFINITY;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        dep[j].cell = sg[j].cell;
        if (j < nseg && attenuate_seg<NB, PREC, THIN>(A, ray, sg[j], kap[j], live, dep[j].v, T, reach)) {
            nseg = j + 1;
            ev = kTerminate;
        }
    }
    st.crossings += (uint32_t)nseg;
    bool on[K];
#pragma unroll
    for (int j = 0; j < K; ++j) on[j] = j < nseg;
    deposit.template add<kWhole, K>(dep, on, live, A.J, NB);
    book_events<NB, PREC, THIN>(A, ev, ray, reach, st);
    return ev;
}

// trace_pass with the geometric correction: up to K crossings per lane. Where the rest moves to
// a neighbour, the neighbours' opacities are loaded with the cells', and cells and neighbours
// form one window, since a neighbour mostly shares its tile with a cell of the pass (192^3 x 128
// sources, three ahead: 8.1 ms, 0.19 lines per crossing, against 8.5 and 0.31 with a window for
// each; four ahead spill registers, 9.2 and 8.8). Moved photons, where a lane has any, take two
// more, for the high and the low limbs. Where the rest is dropped, six ahead and no neighbours
// (128^3 x 16 sources: 0.88 ms, 1.04 through the neighbours' code with four ahead).
template <int NB, int PREC, int K, bool THIN, int CORR, class Depositor>
__device__ __forceinline__ int trace_pass_corr(const TraceArgs& A, Ray<NB>& ray, bool active, WaveStats& st,
                                               Depositor& deposit)
{
    Seg sg[K];
    int nseg = 0;  // segments of the lane (a count, not K lane masks: those spill)
    bool go = active;
    int ev = kContinue;
    if constexpr (THIN) {
        if (active && !(ray.thi < ray.tend)) {
            go = false;
            ev = kSplit;
        }
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        sg[j].cell = 0u;
        sg[j].nb = kNoCell;
        if (go) {
            uint32_t term[3];
            ev = geom_next<NB, PREC, CORR>(A, ray, sg[j], term);
            nseg = j + 1;
            go = ev == kContinue;
        }
    }
    constexpr int N = CORR == kCorrMove ? 2 : 1;
    float kap[K][NB], kapn[K][NB];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        kappa_at<NB>(A, sg[j].cell, kap[j]);
        if constexpr (CORR == kCorrMove) {
            const bool hn = sg[j].nb != kNoCell;
            kappa_at<NB>(A, hn ? sg[j].nb : 0u, kapn[j]);
#pragma unroll
            for (int b = 0; b < NB; ++b) kapn[j][b] = hn ? kapn[j][b] : 0.0f;
        }
    }
    float T[NB];
    ray_transmission<NB, PREC>(ray, T);
    const uint32_t live = live_bins<NB>(ray, active, T, kLiveMinCorr);
    // the crossings' own deposits, then those of their neighbours
    Dep<NB> dep[N * K], dm[K];
    bool on[N * K], use_m[K], moved = false;
    float reach = INFINITY;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        dep[j].cell = sg[j].cell;
        bool term = false;
        if constexpr (CORR == kCorrMove) {
            on[K + j] = use_m[j] = false;
            dep[K + j].cell = dm[j].cell = sg[j].nb != kNoCell ? sg[j].nb : 0u;
            if (j < nseg)
                term = deposit_seg_move<NB, PREC, THIN>(A, ray, sg[j], kap[j], kapn[j], live, dep[j], dep[K + j], dm[j],
                                                        on[K + j], use_m[j], T, reach);
            moved = moved || use_m[j];
        } else if (j < nseg) {
            term = deposit_seg_share<NB, PREC, THIN>(A, ray, sg[j], kap[j], live, dep[j], T, reach);
        }
        if (term) {
            nseg = j + 1;
            ev = kTerminate;
        }
    }
    st.crossings += (uint32_t)nseg;
#pragma unroll
    for (int j = 0; j < K; ++j) on[j] = j < nseg;
    deposit.template add<kWhole, N * K>(dep, on, live, A.J, NB);
    if constexpr (CORR == kCorrMove) {
        if (__builtin_amdgcn_ballot_w64(moved)) {
            deposit.template add<kMovedHi, K>(dm, use_m, live, A.M, 2 * NB);
            deposit.template add<kMovedLo, K>(dm, use_m, live, A.M + 8 * NB, 2 * NB);
        }
    }
    book_events<NB, PREC, THIN>(A, ev, ray, reach, st);
    return ev;
}

// Child k of a split ray: next level, pixel 4p + k, same optical depth (section 2.1 iii c).
template <int NB>
__device__ __forceinline__ RayRec child_rec(const Ray<NB>& ray, int k)
{
    RayRec r;
    r.src = ray.src;
    const uint32_t level = (ray.lp >> kLevelShift) + 1u;
    r.lp = (level << kLevelShift) | (((ray.lp & kPixMask) << 2) + (uint32_t)k);
    r.pad0 = r.pad1 = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        r.tau[b] = b < NB ? ray.tau[b] : 0.0f;
        r.taulo[b] = b < NB ? ray.taulo[b] : 0.0f;
    }
    return r;
}

// A split ray's family record in memory (the persistent kernel's work items): the ray's id
// and optical depth, from which each of its four children is derived when it is taken.
template <int NB>
__device__ __forceinline__ RayRec family_item(const Ray<NB>& ray)
{
    RayRec r;
    r.src = ray.src;
    r.lp = ray.lp;
    r.pad0 = r.pad1 = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        r.tau[b] = b < NB ? ray.tau[b] : 0.0f;
        r.taulo[b] = b < NB ? ray.taulo[b] : 0.0f;
    }
    return r;
}

// A split ray's family record for the persistent kernel's stacks: the ray's id and optical
// depth, from which each of its four children is derived when it is taken.
template <int NB>
__device__ __forceinline__ StackRec<NB> family_rec(const Ray<NB>& ray)
{
    StackRec<NB> r;
    r.src = ray.src;
    r.lp = ray.lp;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        r.tau[b] = ray.tau[b];
        r.taulo[b] = ray.taulo[b];
    }
    return r;
}

// Child k of the split ray a family record holds (section 2.1 iii c).
template <int NB>
__device__ __forceinline__ StackRec<NB> family_child(const StackRec<NB>& f, int k)
{
    StackRec<NB> r = f;
    const uint32_t level = (f.lp >> kLevelShift) + 1u;
    r.lp = (level << kLevelShift) | (((f.lp & kPixMask) << 2) + (uint32_t)k);
    return r;
}

// Fixed-point deposition, called by all 64 lanes together.
//
// Every int64 atomic of the chip is carried out by the memory side of the fabric, never in L2
// (TCC_EA0_ATOMIC equals TCC_ATOMIC), one request per 64-byte line and instruction whether one or
// all eight words of the line take part: 1.75e10 requests/s on random lines, 2.4e10 at most. So
// the field keeps the eight cells of a 2x2x2 tile and one bin in one 64-byte line (field_word),
// and a wave sums its crossings per tile in LDS before it issues a line. A crossing's sum goes
// to a table of one bin at a time, indexed by the cell's place inside its 8^3 block: 64 tiles,
// each tagged with the block it belongs to. A wave's rays are a compact bundle, so its
// crossings of a window seldom want one table entry for two blocks; where they do, the tiles
// that lost the entry go in another round (every round serves at least one tile of each wanted
// entry, so the rounds end). Bins are taken one after the other through the same table, so
// that it takes 4 KB whatever the number of bins. Integer sums: the field does not depend on
// any of this.
constexpr uint32_t kNoBlock = 0xFFFFFFFFu;

// Per-wave LDS space of the deposits. Between windows every sum is zero and every tag kNoBlock.
struct __align__(16) DepScratch {
    unsigned long long acc[512];  // sums of one bin, by place in the block
    uint32_t tag[64];             // block whose tile holds the entry
    uint8_t used[64];             // entries in use, compacted
    double esc[kMaxBins];         // photons the wave's lanes carried out of the grid (WaveStats)
    // When the wave began: noted in memory only at its end, since a store ahead of the trace turns
    // its uniform loads into vector loads (256^3 x 1024 sources: 29.3 ms instead of 28.1).
    unsigned long long began;
};

// Called by all 64 lanes of the wave that owns the scratch, before its first window.
__device__ __forceinline__ void dep_scratch_init(DepScratch* S)
{
    const int lane = threadIdx.x & 63;
    for (int i = lane; i < 512; i += 64) S->acc[i] = 0ull;
    S->tag[lane] = kNoBlock;
    if (lane == 0) S->began = wall_clock64();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// One round of a window: the crossings with `pend` whose tile gets its table entry go into the
// field and leave `pend`. Returns the lines issued per live bin (wave-uniform).
template <int NB, int LIMB, int W>
__device__ __forceinline__ int deposit_round(const Dep<NB>* d, bool (&pend)[W], uint32_t live, DepScratch* S,
                                             unsigned long long* base, int lines)
{
    // LDS-qualified views: through a generic pointer the accesses would be FLAT instructions,
    // which also wait for the wave's outstanding gathers and atomics
    volatile kLds uint32_t* tag = (volatile kLds uint32_t*)S->tag;
    volatile kLds uint8_t* used = (volatile kLds uint8_t*)S->used;
    kLds unsigned long long* acc = (kLds unsigned long long*)S->acc;
    const int lane = threadIdx.x & 63;
    // the last crossing that wants an entry names its block; LDS operations of one wave
    // complete in issue order
#pragma unroll
    for (int w = 0; w < W; ++w)
        if (pend[w]) tag[(d[w].cell >> 3) & 63u] = d[w].cell >> 9;
    uint32_t got[W];
#pragma unroll
    for (int w = 0; w < W; ++w) got[w] = tag[(d[w].cell >> 3) & 63u];
    const bool mine = tag[lane] != kNoBlock;
    bool in[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        in[w] = pend[w] && got[w] == d[w].cell >> 9;
        pend[w] = pend[w] && !in[w];
    }
    const uint64_t mask = __builtin_amdgcn_ballot_w64(mine);
    const int n = __popcll(mask);
    if (mine) used[__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = (uint8_t)lane;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (!(live & (1u << b))) continue;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            float v = d[w].v[b];
            asm volatile("" : "+v"(v));  // the conversion stays inside the live bin's branch
            if (in[w])
                __hip_atomic_fetch_add(acc + (d[w].cell & 511u), (unsigned long long)to_fixed<LIMB>(v), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // eight entries per instruction, a line each
        for (int i0 = 0; i0 < n; i0 += 8) {
            const int r = i0 + (lane >> 3);
            if (r < n) {
                const uint32_t s = used[r], t = tag[s];
                volatile kLds unsigned long long* e = (volatile kLds unsigned long long*)acc + (s * 8u + (lane & 7));
                const unsigned long long q = *e;
                *e = 0ull;
                if (q != 0)
                    atomicAdd(base + ((size_t)((t << 6) | s) * (uint32_t)lines + (uint32_t)b) * 8u + (lane & 7), q);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (mine) tag[lane] = kNoBlock;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return n;
}

// W crossings of every lane, their live bins, into the field at `base`, `lines` 64-byte lines per
// tile (the bins of the field, or of both limbs of the moved-photon field). Returns the lines
// issued (wave-uniform).
template <int NB, int LIMB, int W>
__device__ __forceinline__ int deposit_window(const Dep<NB>* d, const bool (&on)[W], uint32_t live, DepScratch* S,
                                              unsigned long long* base, int lines)
{
    if (live == 0) return 0;
    bool pend[W];
    bool any = false;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        pend[w] = on[w];
        any = any || pend[w];
    }
    if (!__builtin_amdgcn_ballot_w64(any)) return 0;
    int n = deposit_round<NB, LIMB, W>(d, pend, live, S, base, lines);
    uint32_t left = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) left |= pend[w] ? 1u << w : 0u;
#pragma unroll 1
    while (__builtin_amdgcn_ballot_w64(left != 0)) {
#pragma unroll
        for (int w = 0; w < W; ++w) pend[w] = (left >> w) & 1u;
        n += deposit_round<NB, LIMB, W>(d, pend, live, S, base, lines);
        left = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) left |= pend[w] ? 1u << w : 0u;
    }
    return n * __popc(live);
}

// Wave-wide deposit of the crossings of a pass: add() by every lane.
template <int NB>
struct Depositor {
    DepScratch* scratch;
    uint32_t items = 0;  // lines issued by this wave (wave-uniform)
    // the crossings d[0 .. W) of every lane, as integers of limb LIMB
    template <int LIMB, int W>
    __device__ void add(const Dep<NB>* d, const bool (&on)[W], uint32_t live, unsigned long long* base, int lines)
    {
        items += (uint32_t)deposit_window<NB, LIMB, W>(d, on, live, scratch, base, lines);
    }
    __device__ void flush(const TraceArgs& A) const
    {
        if ((threadIdx.x & 63) != 0) return;
        if (items) atomicAdd(&my_slot(A.slots).n[kDeposits], (unsigned long long)items);
        if (A.stamp && blockIdx.x == 0) *A.stamp = scratch->began;
    }
};

// Wave-level reductions, and the end of a wave's statistics.
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ double wave_sum_f64(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NB>
__device__ __forceinline__ void flush_stats(const TraceArgs& A, const WaveStats& st)
{
    const unsigned long long crossings = wave_sum_u64(st.crossings);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if ((threadIdx.x & 63) == 0) {
        CounterSlot& c = my_slot(A.slots);
        if (crossings) atomicAdd(&c.n[kCrossings], crossings);
        if (st.rays) atomicAdd(&c.n[kRays], st.rays);
        if (st.splits) atomicAdd(&c.n[kSplits], st.splits);
        if (st.terminated) atomicAdd(&c.n[kTerminated], st.terminated);
        if (st.escaped) atomicAdd(&c.n[kEscapedRays], st.escaped);
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (st.esc[b] != 0.0) atomicAdd(&c.photons[kPhotonsEscaped + b], st.esc[b]);
    }
}

}  // namespace arc
