// arc_mlp.hip -- learned chemistry step on gfx950 MFMA.
//
// Network: 8 -> 64 -> 64 -> 2, ReLU hidden units, BF16 weights and activations, FP32
// accumulation (v_mfma_f32_16x16x32_bf16). Inputs: log10 n_H, x_HI, log10 T, log10 Gamma_HI,
// log10 dt, log10 h (photoheating per H atom), x_HeII, x_HeI, standardised. Outputs: the
// standardised corrections x_HI' - x_base and log10 (T'/T), where x_base relaxes x_HI
// exponentially towards photoionisation equilibrium with the rates of the start of the step.
// Helium is not an output: the gate accepts a cell only when its helium is close to steady.
//
//   k_infer       per cell: gate, features, forward pass with the activations kept in registers
//                 (each layer's MFMA output is the next layer's operand); accepted cells are
//                 written, rejected cells get a bit in a mask for the plain solver
//   k_predict     the same forward pass without the gate (validation, evaluation)
//   k_train_grad  quantisation-aware forward and backward of a minibatch (MFMA), one gradient
//                 partial per 64 samples (summed in fixed order: deterministic)
//   k_adam        Adam update of the FP32 master parameters and their BF16 images
//   k_publish     all BF16 weight images for the MFMA operands
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "arc_chem.h"
#include "arc_mlp.h"

namespace arc {
namespace mlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------
// MFMA building block. v_mfma_f32_16x16x32_bf16: D[16x16] += A[16x32] B[32x16]; lane l
// supplies A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16] for i = 0..7 and
// receives D[4 (l / 16) + r][l % 16] for r = 0..3.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float act(float x) { return fmaxf(x, 0.0f); }  // ReLU

// Orders one wave's LDS writes before its later reads by other lanes: LDS operations of
// a wave complete in issue order; the fence keeps the compiler from moving accesses.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------------
// Forward pass with the activations in registers.
//
// Each layer computes out^T = W in^T as 16x16 tiles: rows (the MFMA M dimension) are output
// units, columns (N) are 16 cells, the depth (K) runs over the layer's inputs. Lane l = 16q + n
// receives rows 4q..4q+3 of column n, which are exactly 4 of the 8 depth values that lane must
// supply as the B operand of the next layer, provided that layer's depth slots are taken in
// the order perm_k: slot 8q + i of k-step s stands for input unit 32s + 4q + i (i < 4) or
// 32s + 16 + 4q + i - 4 (i >= 4). The A operands (weights) are laid out in LDS in that same
// order, so no activation leaves the registers.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ int perm_k(int s, int q, int i) { return 32 * s + (i < 4 ? 4 * q + i : 12 + 4 * q + i); }

// The weights as the operand fragments each lane supplies, in LDS (shared by the block):
// frag[f][lane] for f = 0..3 layer 1 (M-tile t = f, the eight inputs repeated in the four depth
// groups), 4..11 layer 2 (t = (f - 4) / 2, k-step s = (f - 4) % 2), 12..13 layer 3 (k-step
// s = f - 12, the two outputs repeated in rows 4j and 4j + 1); biases as float4 per four rows.
constexpr int kFrags = 14;
struct LdsWeights {
    bf16x8 frag[kFrags][64];
    float4 b1[kHid / 4], b2[kHid / 4];
    float b3[kOut];
};

// Called by the whole block, followed by a barrier.
__device__ __forceinline__ void load_lds_weights(const Model* M, LdsWeights& L)
{
    for (int idx = threadIdx.x; idx < kFrags * 64; idx += blockDim.x) {
        const int f = idx >> 6, l = idx & 63, m = l & 15, q = l >> 4;
        bf16x8 v;
        if (f < 4) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = M->w1t[16 * f + m][i];
        } else if (f < 12) {
            const int t = (f - 4) >> 1, s2 = (f - 4) & 1;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = M->w2t[16 * t + m][perm_k(s2, q, i)];
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = M->w3t[m & 3][perm_k(f - 12, q, i)];
        }
        L.frag[f][l] = v;
    }
    for (int i = threadIdx.x; i < kHid / 4; i += blockDim.x) {
        L.b1[i] = make_float4(M->b1[4 * i], M->b1[4 * i + 1], M->b1[4 * i + 2], M->b1[4 * i + 3]);
        L.b2[i] = make_float4(M->b2[4 * i], M->b2[4 * i + 1], M->b2[4 * i + 2], M->b2[4 * i + 3]);
    }
    if (threadIdx.x < kOut) L.b3[threadIdx.x] = M->b3[threadIdx.x];
}

// ReLU of a pair after its BF16 rounding (rounding keeps the sign, so this equals rounding
// after the ReLU): as 16-bit integers the negative BF16 values, -0 included, are exactly
// the negative numbers, and one packed integer max clears both halves.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t relu_bf16x2(float a, float b)
{
    const f32x2 p = {a, b};
    const bf16x2 v = __builtin_convertvector(p, bf16x2);  // one packed round-to-nearest-even
    const i16x2 z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, v), z));
}

// Half a hidden layer: ReLU and BF16 rounding of two M-tiles (biases already in the
// accumulators), packed as one k-step of the next layer's B operand (elements 2j and 2j + 1 of
// an operand are the low and high halves of its word j).
__device__ __forceinline__ bf16x8 hidden_to_operand(const f32x4& a, const f32x4& b)
{
    const u32x4 w = {relu_bf16x2(a[0], a[1]), relu_bf16x2(a[2], a[3]), relu_bf16x2(b[0], b[1]),
                     relu_bf16x2(b[2], b[3])};
    return __builtin_bit_cast(bf16x8, w);
}

// Accumulator start of M-tile t: rows 4q..4q+3 of every column carry the biases of hidden
// units 16t + 4q .. 16t + 4q + 3, so the MFMA adds them.
__device__ __forceinline__ f32x4 bias_acc(const float4* bias, int t, int lane)
{
    const float4 b = bias[4 * t + (lane >> 4)];
    const f32x4 v = {b.x, b.y, b.z, b.w};
    return v;
}

// An LDS object's address that the compiler takes for a new one, so that reads of it inside a
// loop stay there instead of being kept in registers over it.
template <class T>
__device__ __forceinline__ const T& read_here(const T& v)
{
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(&v) + zero);
}

// C tiles of 16 cells at once, so that a weight fragment read from LDS serves C MFMAs. x[c] = the
// layer-1 B operand of tile c: the lanes of one depth group hold the 8 standardised features of
// cell n, the others zeros. out[c]: elements 0 and 1 hold the two outputs of cell n (biases
// included) in every lane of column n.
template <int C>
__device__ __forceinline__ void forward_tiles(const LdsWeights& w, int lane, const bf16x8 (&x)[C], f32x4 (&out)[C])
{
    bf16x8 h[C][2], g[C][2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
        f32x4 d[C][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bf16x8 a = w.frag[2 * s2 + j][lane];
            const f32x4 b = bias_acc(w.b1, 2 * s2 + j, lane);
#pragma unroll
            for (int c = 0; c < C; ++c) d[c][j] = mfma(a, x[c], b);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) h[c][s2] = hidden_to_operand(d[c][0], d[c][1]);
    }
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
        f32x4 d[C][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int t = 2 * s2 + j;
            const bf16x8 a0 = w.frag[4 + 2 * t][lane], a1 = w.frag[5 + 2 * t][lane];
            const f32x4 b = bias_acc(w.b2, t, lane);
#pragma unroll
            for (int c = 0; c < C; ++c) d[c][j] = mfma(a0, h[c][0], b);
#pragma unroll
            for (int c = 0; c < C; ++c) d[c][j] = mfma(a1, h[c][1], d[c][j]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) g[c][s2] = hidden_to_operand(d[c][0], d[c][1]);
    }
    const bf16x8 a0 = w.frag[12][lane], a1 = w.frag[13][lane];
    const f32x4 b3 = {w.b3[0], w.b3[1], 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < C; ++c) out[c] = mfma(a0, g[c][0], b3);
#pragma unroll
    for (int c = 0; c < C; ++c) out[c] = mfma(a1, g[c][1], out[c]);
}

// Forward pass of the 64 cells of a wave, one per lane: f = the lane's standardised features;
// returns the lane's two outputs. Lane 16q + n is both the supplier of cell 16q + n and of depth
// group q, column n, so tile c is the same four words in every lane with all groups but c
// cleared, and its outputs are picked by the lanes with q = c: nothing crosses lanes. Groups of
// kTilesAtOnce tiles with no bit in `need` (wave-uniform) are skipped, their outputs zero.
// Two at once: four need registers that cost a wave per SIMD, one reads LDS twice as often (both
// 3% slower).
constexpr int kTilesAtOnce = 2;
__device__ __forceinline__ void forward_wave(const LdsWeights& w, const float f[kIn], float& o0, float& o1,
                                             uint64_t need = ~0ull)
{
    const int lane = threadIdx.x & 63, q = lane >> 4;
    u32x4 pk;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const f32x2 p = {f[2 * j], f[2 * j + 1]};
        pk[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf16x2));
    }
    o0 = o1 = 0.0f;
#pragma unroll
    for (int c0 = 0; c0 < 4; c0 += kTilesAtOnce) {
        if (((need >> (16 * c0)) & (~0ull >> (64 - 16 * kTilesAtOnce))) == 0) continue;
        bf16x8 x[kTilesAtOnce];
        f32x4 o[kTilesAtOnce];
#pragma unroll
        for (int c = 0; c < kTilesAtOnce; ++c) {
            u32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = q == c0 + c ? pk[j] : 0u;
            x[c] = __builtin_bit_cast(bf16x8, v);
        }
        forward_tiles<kTilesAtOnce>(read_here(w), lane, x, o);
#pragma unroll
        for (int c = 0; c < kTilesAtOnce; ++c)
            if (q == c0 + c) {
                o0 = o[c][0];
                o1 = o[c][1];
            }
    }
}

// Decimal logarithm and power from the hardware base-2 functions (the features and the
// targets of training go through the same two functions as inference).
__device__ __forceinline__ float flog10(float v) { return __builtin_amdgcn_logf(v) * 0.30102999566398120f; }
__device__ __forceinline__ float fexp10(float v) { return __builtin_amdgcn_exp2f(v * 3.3219280948873623f); }
__device__ __forceinline__ float safe_log10(float v, float floor_) { return flog10(fmaxf(v, floor_)); }

// Features of a cell: n_H, x_HI, T, Gamma_HI, dt [s], h = photoheating per H atom, x_HeII, x_HeI.
// The first five are those of the gate.
__device__ __forceinline__ void gate_features(float nh, float x, float T, float gam, float ldt, float f[kIn])
{
    static_assert(kIn == 8 && kGateDims == 5, "eight features fill the first MFMA depth group");
    f[0] = flog10(nh);
    f[1] = x;
    f[2] = flog10(T);
    f[3] = safe_log10(gam, kGammaFloor);
    f[4] = ldt;
}
__device__ __forceinline__ void other_features(float h, float xheii, float xhei, float f[kIn])
{
    f[5] = safe_log10(h, kHeatFloor);
    f[6] = xheii;
    f[7] = xhei;
}
__device__ __forceinline__ void cell_features(float nh, float x, float T, float gam, float ldt, float h, float xheii,
                                              float xhei, float f[kIn])
{
    gate_features(nh, x, T, gam, ldt, f);
    other_features(h, xheii, xhei, f);
}

// Baseline of x_HI': dx/dt = a (1 - x) - b x with a = alpha_HII(T) n_e and b = Gamma_HI +
// k_HI(T) n_e held at their start-of-step values (section 2.7 rates), solved exactly:
// x_base = x_eq + (x - x_eq) exp(-(a + b) dt), x_eq = a / (a + b).
__device__ __forceinline__ float x_baseline(const chem::Coef& k, float nh, float x, float gam, float xheii, float xhei,
                                            float dt, float y, int collisional)
{
    const float xheiii = fmaxf(0.0f, 1.0f - xhei - xheii);
    const float ne = nh * ((1.0f - x) + y * (xheii + 2.0f * xheiii));
    const float a = k.a_hii * ne;
    const float b = gam + (collisional ? k.k_hi * ne : 0.0f);
    const float lam = a + b;
    if (!(lam > 0.0f)) return x;
    const float xeq = a / lam;
    return xeq + (x - xeq) * expf(-lam * dt);
}

// The standardisation's means and the reciprocals of its scales, and the same of the gate's
// ranges, in LDS: in registers they would be spilled through the network (correctly rounded, as
// on the host, so that both sides bin and scale identically).
struct Scales {
    float mu[kIn], isd[kIn];
    float lo[kIn], igate[kIn];
};

// Called by the whole block, followed by a barrier.
__device__ __forceinline__ void load_scales(const Model* M, Scales& z)
{
    const int k = threadIdx.x;
    if (k >= kIn) return;
    z.mu[k] = M->in_mu[k];
    z.isd[k] = 1.0f / M->in_sd[k];
    z.lo[k] = M->lo[k];
    z.igate[k] = k < kGateDims ? 1.0f / (M->hi[k] - M->lo[k]) : 0.0f;
}

__device__ __forceinline__ void standardise(const Scales& scales, bool valid, float f[kIn])
{
    const Scales& z = read_here(scales);
#pragma unroll
    for (int k = 0; k < kIn; ++k) f[k] = valid ? (f[k] - z.mu[k]) * z.isd[k] : 0.0f;
}

// ---------------------------------------------------------------------------------
// Inference with the gate.
// ---------------------------------------------------------------------------------
// Per wave: (1) tiles of 64 cells through the gate's bins, which need four of the fields and turn
// most cells away; those that pass wait in LDS until 64 of them fill a wave, then (2) the network,
// its baseline and the screens behind it run on full waves, reading the cells' fields by index (a
// line read a few tiles ago). 256^3 cells of which 34% end accepted, spread over 79% of the tiles:
// 314 us, against 440 with the network on every tile that has a cell past the gate, and 646 with,
// besides, each fragment read from LDS once per 16 cells (704 LDS cycles per tile and compute
// unit), features and results moved across lanes, and the gate's tables read by each of 4096
// workgroups. What bounds it is the vector instructions of the three parts, one after the other in
// a wave (reads alone 100 us). Five waves per SIMD: four 324 us, six (one tile at once) 324; the
// loads of the next tile issued a tile ahead change nothing.
// The cells of a wave that are past the gate's bins and wait for the network: fewer than 64, then
// those of one more tile of 64 cells. They come from at most 64 tiles, whose words of rejected
// cells wait with them.
struct Waiting {
    unsigned long long reject[64];
    uint32_t tile[64];
    uint16_t cell[128];  // tile's place << 6 | cell in the tile
};

__global__ __launch_bounds__(256, kInferWavesPerSimd) void k_infer(InferArgs a)
{
    const Model* M = a.model;
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.stamp = wall_clock64();
    __shared__ LdsWeights w;
    // the gate's verdict per bin (enough samples, small held-out error) as one bit each, so that
    // a cell's gate test reads LDS instead of two scattered loads from the model's tables
    __shared__ uint32_t gate_ok[kGateBins / 32];
    __shared__ Scales z;
    load_lds_weights(M, w);
    load_scales(M, z);
    if (a.gated) {
        for (uint32_t i = threadIdx.x; i < kGateBins / 32; i += blockDim.x) {
            const uint4* count = reinterpret_cast<const uint4*>(M->gate_count + 32 * i);
            const float4* err = reinterpret_cast<const float4*>(M->gate_err + 32 * i);
            uint32_t bits = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint4 n = count[j];
                const float4 e = err[j];
                bits |= (uint32_t)(n.x >= a.gate_min_count && e.x <= a.gate_tol) << (4 * j);
                bits |= (uint32_t)(n.y >= a.gate_min_count && e.y <= a.gate_tol) << (4 * j + 1);
                bits |= (uint32_t)(n.z >= a.gate_min_count && e.z <= a.gate_tol) << (4 * j + 2);
                bits |= (uint32_t)(n.w >= a.gate_min_count && e.w <= a.gate_tol) << (4 * j + 3);
            }
            gate_ok[i] = bits;
        }
    }
    __shared__ Waiting waiting[4];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    Waiting& wt = waiting[threadIdx.x >> 6];
    const float dtf = (float)a.dt, ldt = flog10(dtf);
    const float yf = (float)a.y;
    const uint32_t stride = gridDim.x * blockDim.x;
    uint32_t nwait = 0, ntile = 0;  // cells waiting, and their tiles (wave-uniform)
    for (uint32_t base = blockIdx.x * blockDim.x + (threadIdx.x & ~63u);; base += stride) {
        const bool more = base < a.ncell;
        if (more) {
            // (1) gate bins: inside the training range, in a bin with enough samples and a small
            //     held-out error
            const uint32_t c = base + lane;
            const bool valid = c < a.ncell;
            bool pass = valid;
            if (valid && a.gated) {
                float f[kIn];
                gate_features(a.n_h[c], a.x_hi[c], a.temp[c], a.gamma[c], ldt, f);
                const Scales& zg = read_here(z);
                uint32_t bin = 0;
#pragma unroll
                for (int k = kGateDims - 1; k >= 0; --k) {
                    const float u = (f[k] - zg.lo[k]) * zg.igate[k];
                    pass = pass && u >= 0.0f && u <= 1.0f;
                    const int b = min(kGate - 1, max(0, (int)(u * kGate)));
                    bin = bin * kGate + (uint32_t)b;
                }
                pass = pass && ((gate_ok[bin >> 5] >> (bin & 31u)) & 1u) != 0u;
            }
            const uint64_t through = __ballot(pass), rej = __ballot(valid && !pass);
            if (through) {
                if (lane == 0) {
                    wt.reject[ntile] = (unsigned long long)rej;
                    wt.tile[ntile] = base >> 6;
                }
                if (pass) wt.cell[nwait + (uint32_t)__popcll(through & __lanemask_lt())] = (uint16_t)(ntile << 6 | lane);
                nwait += (uint32_t)__popcll(through);
                ++ntile;
                wave_sync();
            } else if (lane == 0) {
                a.reject[base >> 6] = (unsigned long long)rej;
            }
        }
        if (nwait >= 64u || (!more && nwait > 0u)) {
            const uint32_t n = min(nwait, 64u);
            const bool valid = (uint32_t)lane < n;
            uint32_t entry = 0, c = 0;
            float nh = 1.0f, T = 1.0f, x0 = 0.0f, xhei = 0.0f, xheii = 0.0f, gam = 0.0f, h = 0.0f;
            if (valid) {
                entry = wt.cell[lane];
                c = (wt.tile[entry >> 6] << 6) + (entry & 63u);
                nh = a.n_h[c];
                T = a.temp[c];
                x0 = a.x_hi[c];
                xhei = a.x_hei[c];
                xheii = a.x_heii[c];
                gam = a.gamma[c];
                h = a.heat[c] * x0 + yf * (a.heat[(size_t)a.ncell + c] * xhei + a.heat[2 * (size_t)a.ncell + c] * xheii);
            }
            float f[kIn];
            cell_features(nh, x0, T, gam, ldt, h, xheii, xhei, f);
            standardise(z, valid, f);
            float o0, o1;
            forward_wave(w, f, o0, o1, ~0ull >> (64u - n));
            const chem::Coef k = chem::coefficients(T);
            const float xb = x_baseline(k, nh, x0, gam, xheii, xhei, dtf, M->base_y, M->base_collisional);
            const float xn = fminf(fmaxf(xb + (o0 * M->out_sd[0] + M->out_mu[0]), 0.0f), 1.0f);
            const float Tn = T * fexp10(o1 * M->out_sd[1] + M->out_mu[1]);
            bool accept = valid;
            if (accept && a.gated) {
                // (2) physical output temperature
                accept = Tn >= a.t_floor && Tn < 1e9f;
                // (3) helium close to steady over dt (the network does not predict helium)
                //     (a screening test: FP32 is ample for a 1e-3 threshold)
                if (accept && a.y > 0.0) {
                    const float nhe = yf * nh;
                    const float nhei = nhe * xhei, nheii = nhe * xheii;
                    const float nheiii = fmaxf(0.0f, nhe - nhei - nheii);
                    const float ne = nh * (1.0f - x0) + nheii + 2.0f * nheiii;
                    const float kc = a.collisional ? 1.0f : 0.0f;
                    const float dhei = k.a_heii * ne * nheii - (a.gamma[(size_t)a.ncell + c] + kc * k.k_hei * ne) * nhei;
                    const float dheiii =
                        (a.gamma[2 * (size_t)a.ncell + c] + kc * k.k_heii * ne) * nheii - k.a_heiii * ne * nheiii;
                    accept = fabsf(dhei) * dtf <= 1e-3f * nhe && fabsf(dheiii) * dtf <= 1e-3f * nhe;
                }
            }
            if (accept) {
                a.x_hi[c] = xn;
                a.temp[c] = Tn;
            }
            // the cells for the plain solver: what is left waiting is of the last tile
            if (valid && !accept) atomicOr(&wt.reject[entry >> 6], 1ull << (entry & 63u));
            wave_sync();
            const uint32_t left = nwait - n, done = left ? ntile - 1u : ntile;
            if ((uint32_t)lane < done) a.reject[wt.tile[lane]] = wt.reject[lane];
            if (left) {
                const unsigned long long rej = wt.reject[done];
                const uint32_t tile = wt.tile[done];
                const uint16_t next = wt.cell[64 + lane] & 63u;
                wave_sync();
                if (lane == 0) {
                    wt.reject[0] = rej;
                    wt.tile[0] = tile;
                }
                if ((uint32_t)lane < left) wt.cell[lane] = next;
                wave_sync();
            }
            nwait = left;
            ntile = left ? 1u : 0u;
        }
        if (!more) break;
    }
}

hipError_t launch_infer(const InferArgs& a, int cus, hipStream_t s)
{
    // the waves that are resident at once: each workgroup fills its tables from the model, and
    // more tiles per wave leave fewer of its last batches unfilled (twice as many: 333 us)
    const size_t blocks = std::min(((size_t)a.ncell + 255) / 256, (size_t)std::max(cus, 1) * kInferWavesPerSimd);
    k_infer<<<(unsigned)std::max<size_t>(blocks, 1), 256, 0, s>>>(a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Forward only (validation, gate calibration, evaluation): raw samples to (x_HI', T').
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void raw_features(const float* x, float f[kIn])
{
    cell_features(x[0], x[1], x[2], x[3], flog10(x[4]), x[5], x[6], x[7], f);
}

__device__ __forceinline__ float raw_baseline(const float* x, float y, int collisional)
{
    return x_baseline(chem::coefficients(x[2]), x[0], x[1], x[3], x[6], x[7], x[4], y, collisional);
}

__global__ __launch_bounds__(256) void k_predict(const Model* M, const float* X, const uint32_t* idx, uint32_t m,
                                                 float* P)
{
    __shared__ LdsWeights w;
    __shared__ Scales z;
    load_lds_weights(M, w);
    load_scales(M, z);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (uint32_t base = blockIdx.x * blockDim.x + (threadIdx.x & ~63u); base < m; base += gridDim.x * blockDim.x) {
        const uint32_t i = base + lane;
        const bool valid = i < m;
        const float* x = X + (size_t)(valid ? (idx ? idx[i] : i) : 0u) * kIn;
        float f[kIn] = {1.0f, 0.0f, 1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        float xb = 0.0f;
        if (valid) {
            raw_features(x, f);
            xb = raw_baseline(x, M->base_y, M->base_collisional);
        }
        standardise(z, valid, f);
        float o0, o1;
        forward_wave(w, f, o0, o1);
        if (valid) {
            P[(size_t)i * 2] = fminf(fmaxf(xb + (o0 * M->out_sd[0] + M->out_mu[0]), 0.0f), 1.0f);
            P[(size_t)i * 2 + 1] = x[2] * fexp10(o1 * M->out_sd[1] + M->out_mu[1]);
        }
    }
}

hipError_t launch_predict(const Model* model, const float* X, const uint32_t* idx, uint32_t m, float* P,
                          hipStream_t s)
{
    size_t blocks = (m + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    k_predict<<<(unsigned)blocks, 256, 0, s>>>(model, X, idx, m, P);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Features and targets of raw samples X [m][kIn] and (x_HI', T').
// ---------------------------------------------------------------------------------
__global__ void k_features(const float* X, const float* Y, uint32_t m, float y, int collisional, float* F, float* Yt)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x) {
        const float* x = X + (size_t)i * kIn;
        raw_features(x, F + (size_t)i * kIn);
        Yt[(size_t)i * 2] = Y[(size_t)i * 2] - raw_baseline(x, y, collisional);
        Yt[(size_t)i * 2 + 1] = flog10(Y[(size_t)i * 2 + 1]) - flog10(x[2]);
    }
}

hipError_t launch_features(const float* X, const float* Y, uint32_t m, float y, int collisional, float* F, float* Yt,
                           hipStream_t s)
{
    size_t blocks = (m + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    k_features<<<(unsigned)blocks, 256, 0, s>>>(X, Y, m, y, collisional, F, Yt);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Training: gradient of the minibatch loss
//   L = sum_s (o0 - y0)^2 + (o1 - y1)^2     (standardised targets; divided by the batch
//                                            size in Adam)
// through the same BF16 forward as inference. 64 samples per workgroup of four waves: a wave
// takes 16 samples through the forward pass and back to both hidden layers without waiting for
// the others, then, after one barrier, a quarter of the weight gradients, which sum over all 64
// samples. A minibatch is only a few workgroups, so the step is a chain of latencies: the weights
// come straight from memory as MFMA operands (all loads issued at the start), every activation
// is written to LDS in the orders in which it is read (16 bytes a lane, rows padded against bank
// conflicts), and the ReLU masks stay in registers. Batch of 1024: 44 us with one wave per 64
// samples, weights staged in LDS and operands gathered element by element, 9 us so.
// ---------------------------------------------------------------------------------
constexpr int kRow = 72;  // padded row of 64 BF16 values in LDS (144 bytes)

__device__ __forceinline__ bf16x8 zero8()
{
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (__bf16)0.0f;
    return v;
}
__device__ __forceinline__ bf16x8 from_f32(const float* p)
{
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (__bf16)p[i];
    return v;
}
__device__ __forceinline__ bf16x8 row8(const __bf16* m, int row, int k) { return *(const bf16x8*)(m + row * kRow + k); }

__global__ __launch_bounds__(256) void k_train_grad(TrainArgs a)
{
    // [sample][unit]: operands of the next layer; [unit][sample]: operands of the weight gradients
    __shared__ __align__(16) __bf16 H1[64 * kRow], H2[64 * kRow];       // H2's rows become D2's
    __shared__ __align__(16) __bf16 H1t[64 * kRow], H2t[64 * kRow], D1t[64 * kRow], D2t[64 * kRow];
    __shared__ __align__(16) __bf16 Xt[kIn * kRow], DOt[kOut * kRow], DO[64 * kOut];
    const int lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4, t = threadIdx.x >> 6;
    const Model* M = a.model;
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const f32x4 none = {0.0f, 0.0f, 0.0f, 0.0f};
    // operands: lane (r16, q) supplies row or column r16, depth 8 q .. 8 q + 7 of a k-step
    const uint32_t s0 = blockIdx.x * 64u + 16u * (uint32_t)t;  // the wave's first sample
    bf16x8 x = zero8();
    if (q == 0) {
        const uint32_t sl = s0 + (uint32_t)r16;
        if (sl < a.count) x = from_f32(a.F + (size_t)a.idx[a.first + sl] * kIn);
#pragma unroll
        for (int k = 0; k < kIn; ++k) Xt[k * kRow + 16 * t + r16] = x[k];
    }
    float y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (r16 < kOut)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t sl = s0 + 4u * (uint32_t)q + (uint32_t)r;
            if (sl < a.count) y[r] = a.Y[(size_t)a.idx[a.first + sl] * 2 + r16];
        }
    bf16x8 w1[4], w2[4][2], w3[2], w2b[4][2], w3b[4];
    float b1[4], b2[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int n = 16 * nt + r16;
        w1[nt] = *(const bf16x8*)&M->w1t[n][8 * q];
        b1[nt] = M->b1[n];
        b2[nt] = M->b2[n];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            w2[nt][k] = *(const bf16x8*)&M->w2t[n][32 * k + 8 * q];
            // the same rounding of the master weights, in the order of the way back
            w2b[nt][k] = from_f32(a.params + kW2 + n * kHid + 32 * k + 8 * q);
        }
        w3b[nt] = zero8();
        if (q == 0) {
            w3b[nt][0] = (__bf16)a.params[kW3 + n * kOut];
            w3b[nt][1] = (__bf16)a.params[kW3 + n * kOut + 1];
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) w3[k] = *(const bf16x8*)&M->w3t[r16][32 * k + 8 * q];
    const float b3 = r16 < kOut ? M->b3[r16] : 0.0f;

    // a tile's element r of a lane is (sample 16 t + 4 q + r, unit 16 nt + r16)
    uint32_t pos1 = 0, pos2 = 0;  // which hidden values are positive, bit 4 nt + r
    auto put = [&](__bf16* rows, __bf16* cols, int nt, const bf16x4& v) {
        if (rows)
#pragma unroll
            for (int r = 0; r < 4; ++r) rows[(16 * t + 4 * q + r) * kRow + 16 * nt + r16] = v[r];
        *(bf16x4*)(cols + (16 * nt + r16) * kRow + 16 * t + 4 * q) = v;
    };
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const f32x4 d = mfma(x, w1[nt], none);
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = (__bf16)act(d[r] + b1[nt]);
            pos1 |= (float)v[r] > 0.0f ? 1u << (4 * nt + r) : 0u;
        }
        put(H1, H1t, nt, v);
    }
    wave_sync();
    {
        const bf16x8 h0 = row8(H1, 16 * t + r16, 8 * q), h1 = row8(H1, 16 * t + r16, 32 + 8 * q);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const f32x4 d = mfma(h1, w2[nt][1], mfma(h0, w2[nt][0], none));
            bf16x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = (__bf16)act(d[r] + b2[nt]);
                pos2 |= (float)v[r] > 0.0f ? 1u << (4 * nt + r) : 0u;
            }
            put(H2, H2t, nt, v);
        }
    }
    wave_sync();
    {
        const bf16x8 h0 = row8(H2, 16 * t + r16, 8 * q), h1 = row8(H2, 16 * t + r16, 32 + 8 * q);
        const f32x4 d = mfma(h1, w3[1], mfma(h0, w3[0], none));
        // output gradient
        if (r16 < kOut) {
            bf16x4 g;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int sl = 16 * t + 4 * q + r;
                g[r] = (__bf16)(blockIdx.x * 64u + (uint32_t)sl < a.count ? 2.0f * ((d[r] + b3) - y[r]) : 0.0f);
                DO[sl * kOut + r16] = g[r];
            }
            *(bf16x4*)(DOt + r16 * kRow + 16 * t + 4 * q) = g;
        }
    }
    wave_sync();
    // dz2 = (dO W3^T) * [H2 > 0]
    {
        bf16x8 g = zero8();
        if (q == 0) {
            g[0] = DO[(16 * t + r16) * kOut];
            g[1] = DO[(16 * t + r16) * kOut + 1];
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const f32x4 d = mfma(g, w3b[nt], none);
            bf16x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (__bf16)((pos2 >> (4 * nt + r)) & 1u ? d[r] : 0.0f);
            put(H2, D2t, nt, v);
        }
    }
    wave_sync();
    // dz1 = (dz2 W2^T) * [H1 > 0]
    {
        const bf16x8 h0 = row8(H2, 16 * t + r16, 8 * q), h1 = row8(H2, 16 * t + r16, 32 + 8 * q);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const f32x4 d = mfma(h1, w2b[nt][1], mfma(h0, w2b[nt][0], none));
            bf16x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (__bf16)((pos1 >> (4 * nt + r)) & 1u ? d[r] : 0.0f);
            put(nullptr, D1t, nt, v);
        }
    }
    __syncthreads();
    // weight gradients over the 64 samples, rows 16 t .. 16 t + 15 of each matrix
    float* P = a.partial + (size_t)blockIdx.x * kNParams;
    {
        // dW2[k][n] = sum_s H1[s][k] dz2[s][n]
        const bf16x8 h0 = row8(H1t, 16 * t + r16, 8 * q), h1 = row8(H1t, 16 * t + r16, 32 + 8 * q);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const f32x4 d = mfma(h1, row8(D2t, 16 * nt + r16, 32 + 8 * q), mfma(h0, row8(D2t, 16 * nt + r16, 8 * q), none));
#pragma unroll
            for (int r = 0; r < 4; ++r) P[kW2 + (16 * t + 4 * q + r) * kHid + 16 * nt + r16] = d[r];
        }
    }
    {
        // dW3[k][n] = sum_s H2[s][k] dO[s][n]
        const bool on = r16 < kOut;
        const bf16x8 g0 = on ? row8(DOt, r16, 8 * q) : zero8(), g1 = on ? row8(DOt, r16, 32 + 8 * q) : zero8();
        const f32x4 d = mfma(row8(H2t, 16 * t + r16, 32 + 8 * q), g1, mfma(row8(H2t, 16 * t + r16, 8 * q), g0, none));
        if (on)
#pragma unroll
            for (int r = 0; r < 4; ++r) P[kW3 + (16 * t + 4 * q + r) * kOut + r16] = d[r];
    }
    {
        // dW1[k][n] = sum_s X[s][k] dz1[s][n], columns 16 t .. 16 t + 15
        const bool on = r16 < kIn;
        const bf16x8 x0 = on ? row8(Xt, r16, 8 * q) : zero8(), x1 = on ? row8(Xt, r16, 32 + 8 * q) : zero8();
        const f32x4 d = mfma(x1, row8(D1t, 16 * t + r16, 32 + 8 * q), mfma(x0, row8(D1t, 16 * t + r16, 8 * q), none));
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * q + r < kIn) P[kW1 + (4 * q + r) * kHid + 16 * t + r16] = d[r];
    }
    // bias gradients: sums over the samples, in their order
    if (t < 2 || (t == 2 && lane < kOut)) {
        const __bf16* m = t == 0 ? D1t : (t == 1 ? D2t : DOt);
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < 64; k += 8) {
            const bf16x8 v = row8(m, lane, k);
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += (float)v[i];
        }
        P[(t == 0 ? kB1 : (t == 1 ? kB2 : kB3)) + lane] = sum;
    }
}

hipError_t launch_train_grad(const TrainArgs& a, hipStream_t s)
{
    k_train_grad<<<(a.count + 63) / 64, 256, 0, s>>>(a);
    return hipGetLastError();
}

// BF16 image or bias of parameter p in the model.
__device__ __forceinline__ void publish_param(Model* M, int p, float v)
{
    if (p < kB1) {
        M->w1t[p % kHid][p / kHid] = (__bf16)v;
    } else if (p < kW2) {
        M->b1[p - kB1] = v;
    } else if (p < kB2) {
        M->w2t[(p - kW2) % kHid][(p - kW2) / kHid] = (__bf16)v;
    } else if (p < kW3) {
        M->b2[p - kB2] = v;
    } else if (p < kB3) {
        M->w3t[(p - kW3) % kOut][(p - kW3) / kOut] = (__bf16)v;
    } else {
        M->b3[p - kB3] = v;
    }
}

// Sums the partial gradients in their order, updates, and publishes the parameter's image (a
// launch of its own before). 64 threads a workgroup: 77 of them share the latencies.
__global__ __launch_bounds__(64) void k_adam(AdamArgs a)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kNParams) return;
    const float m0 = a.m[p], v0 = a.v[p], w0 = a.params[p];
    float g = 0.0f;
    int w = 0;
    for (; w + 8 <= a.nwaves; w += 8) {
        float part[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) part[i] = a.partial[(size_t)(w + i) * kNParams + p];
#pragma unroll
        for (int i = 0; i < 8; ++i) g += part[i];
    }
    for (; w < a.nwaves; ++w) g += a.partial[(size_t)w * kNParams + p];
    g *= a.inv_batch;
    const float m = a.beta1 * m0 + (1.0f - a.beta1) * g;
    const float v = a.beta2 * v0 + (1.0f - a.beta2) * g * g;
    a.m[p] = m;
    a.v[p] = v;
    const float mh = m / (1.0f - powf(a.beta1, (float)a.step));
    const float vh = v / (1.0f - powf(a.beta2, (float)a.step));
    const float wn = w0 - a.lr * mh / (sqrtf(vh) + a.eps);
    a.params[p] = wn;
    publish_param(a.model, p, wn);
}

// Every image from the master parameters, the padding's zeros among them (before training).
__global__ void k_publish(const float* P, Model* M)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kHid * kHid; i += gridDim.x * blockDim.x) {
        const int n = i / kHid, k = i % kHid;  // w2t[n][k] = w2[k][n]
        M->w2t[n][k] = (__bf16)P[kW2 + k * kHid + n];
    }
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kHid * kK1; i += gridDim.x * blockDim.x) {
        const int n = i / kK1, k = i % kK1;
        M->w1t[n][k] = (__bf16)(k < kIn ? P[kW1 + k * kHid + n] : 0.0f);
    }
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kOutP * kHid; i += gridDim.x * blockDim.x) {
        const int n = i / kHid, k = i % kHid;
        M->w3t[n][k] = (__bf16)(n < kOut ? P[kW3 + k * kOut + n] : 0.0f);
    }
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kHid; i += gridDim.x * blockDim.x) {
        M->b1[i] = P[kB1 + i];
        M->b2[i] = P[kB2 + i];
    }
    if (blockIdx.x == 0 && threadIdx.x < kOut) M->b3[threadIdx.x] = P[kB3 + threadIdx.x];
}

hipError_t launch_adam(const AdamArgs& a, hipStream_t s)
{
    k_adam<<<(kNParams + 63) / 64, 64, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_publish(const float* params, Model* model, hipStream_t s)
{
    k_publish<<<16, 256, 0, s>>>(params, model);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace arc
