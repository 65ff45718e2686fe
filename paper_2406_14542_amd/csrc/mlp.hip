// Learned per-point quadrature weights that precondition the least-squares inverse.
//
// A small multilayer perceptron maps features of a point's neighbourhood in a coarse
// density map to a positive weight w_i; the weights form the row preconditioner W of the
// CGLS solve (nusht_solve) and its initial iterate S^H W d.  Everything here is FP32 except
// the transform calls.
//
//   density:  64 x 128 equal-angle (theta, phi) histogram, normalised to 1 for uniform points
//   features: [log rho bilinear at the point, log rho of the 3 x 3 cells around the point's
//              cell (phi periodic, theta clamped), cos theta, sin theta]      (12 values)
//   network:  12 -> 128 -> 128 -> 128 (tanh) -> 1, w = softplus(z) * scale
//   training: loss = <r, r>_m / <a*, a*>_m with r = S^H (W d) - a*; its gradient with respect
//             to w_i is 2 d_i (S r)_i / <a*, a*>_m (one synthesis), then back through the net.
//
// Parameter layout (FP32, transposed weights so a layer's outputs for one input are
// contiguous): W1t[12][128] b1[128] W2t[128][128] b2[128] W3t[128][128] b3[128] w4[128] b4[1].
#include <mutex>

#include "internal.h"

namespace nusht {
namespace {

constexpr int kIn = 12;
constexpr int kHid = 128;
constexpr int oW1 = 0;
constexpr int oB1 = oW1 + kIn * kHid;
constexpr int oW2 = oB1 + kHid;
constexpr int oB2 = oW2 + kHid * kHid;
constexpr int oW3 = oB2 + kHid;
constexpr int oB3 = oW3 + kHid * kHid;
constexpr int oW4 = oB3 + kHid;
constexpr int oB4 = oW4 + kHid;
constexpr int kParams = oB4 + 1;

constexpr int kTileP = 64;        // points per tile
constexpr int kLd = kHid + 4;     // LDS row of a point's activations (see Tile)
constexpr int kLdX = 20;          // LDS row of a point's inputs: 12 features, 1, zeros up to 16
constexpr int kUB = kHid / 16;    // blocks of 16 units

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ inline float softplus(float z) { return z > 20.f ? z : log1pf(expf(z)); }
__device__ inline float sigmoid(float z) { return 1.f / (1.f + expf(-z)); }

// The network's layers are matrix products, run on v_mfma_f32_16x16x4_f32 (FP32 inputs and sums:
// 157 TFLOP/s, twice the unpacked FP32 VALU).  Operands, with c = lane % 16 and g = lane / 16:
// A[row c][k g], B[k g][column c], D[row 4 g + r][column c] in register r.
//
// Rows are units, columns are points: a wave owns the 16 units u0 .. u0 + 15 of a layer for some of
// the tile's points, holds its slice of the layer's weights in 32 registers (fetched per tile: the
// 270 KB of parameters stay in L2), and reads the points' activations from LDS.  The k index
// of MFMA (t, i) in lane group g is 16 t + 4 g + i, so that a lane's operands of four consecutive
// MFMAs are 16 consecutive bytes of its point's row; D holds four consecutive units of a point, which
// go back with one 16-byte store.  Rows of 132 floats put the 16 points of such an access on 16
// different groups of four banks.
__device__ inline void load_w_fwd(const float* __restrict__ Wt, int u0, int c, int g, float (&w)[32])
{
#pragma unroll
    for (int t = 0; t < kUB; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) w[4 * t + i] = Wt[(16 * t + 4 * g + i) * kHid + u0 + c];
}

// the transposed product's slice: rows are the layer's inputs, k its outputs
__device__ inline void load_w_bwd(const float* __restrict__ Wt, int u0, int c, int g, float (&w)[32])
{
    // four-byte alignment only: the blocks of the parameter array start at multiples of 4 bytes
    const float* row = Wt + (u0 + c) * kHid + 4 * g;
#pragma unroll
    for (int t = 0; t < kUB; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) w[4 * t + i] = row[16 * t + i];
}

// acc[pb] += (weight slice) x (act rows pbase + 16 pb ..)
template <int NPB>
__device__ inline void mm_units(const float (&w)[32], const float* act, int pbase, int c, int g,
                                f4 (&acc)[NPB])
{
#pragma unroll
    for (int t = 0; t < kUB; ++t) {
        f4 b[NPB];
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb)
            b[pb] = *reinterpret_cast<const f4*>(act + (pbase + 16 * pb + c) * kLd + 16 * t + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int pb = 0; pb < NPB; ++pb)
                acc[pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[4 * t + i], b[pb][i], acc[pb], 0, 0, 0);
    }
}

// D[NK] (rows: 16 units of `a` per block from k0 on, columns: units j0 .. j0 + 15 of `d`), the sum
// over the tile's points of a[p][k] d[p][j].  Lane group g takes point 16 S + 4 g + s, whose row is
// 16 banks from the next group's.
template <int NK, int LDA>
__device__ inline void mm_points(const float* a, int k0, const float* d, int j0, int c, int g,
                                 f4 (&out)[NK])
{
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) out[kb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int q = 0; q < kTileP / 4; ++q) {
        const int p = (q >> 2) * 16 + 4 * g + (q & 3);
        const float b = d[p * kLd + j0 + c];
#pragma unroll
        for (int kb = 0; kb < NK; ++kb)
            out[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[p * LDA + k0 + 16 * kb + c], b, out[kb], 0,
                                                           0, 0);
    }
}

__device__ inline f4 tanh4(f4 v)
{
    f4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = tanhf(v[r]);
    return o;
}

// b[0 .. 3] of an array aligned to 4 bytes
__device__ inline f4 load4(const float* __restrict__ b)
{
    return f4{b[0], b[1], b[2], b[3]};
}

// Forward pass of one tile by the whole block: a1 and a2 into LDS, the wave's own a3 (units
// u0 + 4 g + r of points pbase + 16 pb + c) into a3, its share of the output layer's sum into zp.
// Ends with a barrier.
template <int NPB>
__device__ inline void tile_forward(const float* __restrict__ prm, const float* __restrict__ feat,
                                    int64_t p0, int64_t npts, int ub, int pbase, int c, int g,
                                    float* x0, float* A1, float* A2, float (*zp)[kTileP],
                                    f4 (&a3)[NPB])
{
    const int u0 = 16 * ub;
    float w[32];
    for (int e = threadIdx.x; e < kTileP * 16; e += blockDim.x) {
        const int p = e >> 4, k = e & 15;
        float v = k == kIn ? 1.f : 0.f;  // the row of ones carries db1
        if (k < kIn && p0 + p < npts) v = feat[(p0 + p) * kIn + k];
        x0[p * kLdX + k] = v;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * g + i;
        w[i] = k < kIn ? prm[oW1 + (k < kIn ? k : 0) * kHid + u0 + c] : 0.f;
    }
    f4 acc[NPB], bias = load4(prm + oB1 + u0 + 4 * g);
    __syncthreads();
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
        acc[pb] = bias;
        const f4 b = *reinterpret_cast<const f4*>(x0 + (pbase + 16 * pb + c) * kLdX + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc[pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], b[i], acc[pb], 0, 0, 0);
    }
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb)
        *reinterpret_cast<f4*>(A1 + (pbase + 16 * pb + c) * kLd + u0 + 4 * g) = tanh4(acc[pb]);
    load_w_fwd(prm + oW2, u0, c, g, w);
    bias = load4(prm + oB2 + u0 + 4 * g);
    __syncthreads();
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) acc[pb] = bias;
    mm_units<NPB>(w, A1, pbase, c, g, acc);
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb)
        *reinterpret_cast<f4*>(A2 + (pbase + 16 * pb + c) * kLd + u0 + 4 * g) = tanh4(acc[pb]);
    load_w_fwd(prm + oW3, u0, c, g, w);
    bias = load4(prm + oB3 + u0 + 4 * g);
    __syncthreads();
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) acc[pb] = bias;
    mm_units<NPB>(w, A2, pbase, c, g, acc);
    const f4 w4 = load4(prm + oW4 + u0 + 4 * g);
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
        a3[pb] = tanh4(acc[pb]);
        float z = a3[pb][0] * w4[0] + a3[pb][1] * w4[1] + a3[pb][2] * w4[2] + a3[pb][3] * w4[3];
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        if (g == 0) zp[ub][pbase + 16 * pb + c] = z;
    }
    __syncthreads();
}

// the output unit of point p from the blocks' shares
__device__ inline float out_unit(const float* __restrict__ prm, const float (*zp)[kTileP], int p)
{
    float z = prm[oB4];
#pragma unroll
    for (int u = 0; u < kUB; ++u) z += zp[u][p];
    return z;
}

// Forward: one block of 8 waves per tile, wave u owns units 16 u .. of all 64 points; two blocks
// per CU (75 KB of LDS each), so that one's tanh and barriers run beside the other's MFMAs.  Bound by
// the FP32 MFMAs (70 kflop a point; 0.90 ms at their peak for 2 M points): 1.49 ms, 94 TFLOP/s,
// against 17.96 ms with one lane per point on the VALU (102 KB of LDS, one block of 4 waves per CU).
__global__ __launch_bounds__(512, 4) void k_mlp_forward(const float* __restrict__ prm,
                                                        const float* __restrict__ feat,
                                                        int64_t npts, float scale,
                                                        float* __restrict__ w)
{
    __shared__ __align__(16) float x0[kTileP * kLdX];
    __shared__ __align__(16) float A1[kTileP * kLd];
    __shared__ __align__(16) float A2[kTileP * kLd];
    __shared__ float zp[kUB][kTileP];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t p0 = (int64_t)blockIdx.x * kTileP;
    f4 a3[4];
    tile_forward<4>(prm, feat, p0, npts, wave, 0, lane & 15, lane >> 4, x0, A1, A2, zp, a3);
    if (threadIdx.x < kTileP && p0 + threadIdx.x < npts)
        w[p0 + threadIdx.x] = softplus(out_unit(prm, zp, threadIdx.x)) * scale;
}

// Backward: grid-stride over tiles by blocks of 16 waves (four per SIMD).  Wave (ub, ph) owns units
// 16 ub .. of points 32 ph .. in the products over units, and the gradient blocks of rows 64 ph ..,
// columns 16 ub .. of W2 and W3 (32 registers) in the products over points.  A tile's gradient is
// summed from zero and then added to the block's running sum, so that the sums' rounding grows
// with the number of tiles, not of points.  Every block writes one partial vector, which
// k_mlp_reduce sums in block order.  The FP32 MFMAs (208 kflop a point; 2.65 ms at their peak for 2 M
// points) are busy 44 % of its time; the rest are the barriers between the layers and 96 registers
// per lane that spill at 16 waves per CU (12 GB at 2 TB/s): 5.95 ms against 85.4 ms on the VALU
// (135 KB of LDS, one block of 4 waves per CU; strided scalar weight loads in the delta products).
__global__ __launch_bounds__(1024) void k_mlp_backward(const float* __restrict__ params,
                                                       const float* __restrict__ feat,
                                                       const float* __restrict__ gw, int64_t npts,
                                                       float scale, float* __restrict__ partial)
{
    __shared__ __align__(16) float x0[kTileP * kLdX];
    __shared__ __align__(16) float A1[kTileP * kLd];
    __shared__ __align__(16) float A2[kTileP * kLd];
    __shared__ __align__(16) float dl[kTileP * kLd];  // delta of the current layer
    __shared__ float zp[kUB][kTileP];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ub = wave & (kUB - 1), ph = wave / kUB, u0 = 16 * ub;
    const int c = lane & 15, g = lane >> 4;
    const int pbase = 32 * ph;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 dW2[4], dW3[4], dW1 = zero, db2 = zero, db3 = zero, dw4 = zero;
    float db4 = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) dW2[k] = dW3[k] = zero;

    const int64_t ntiles = (npts + kTileP - 1) / kTileP;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t p0 = tile * kTileP;
        f4 a3[2];
        // the parameters are fetched anew for every tile: held across tiles, they (and the
        // addresses of their loads) spill
        const float* prm = params;
        int ln = lane;
        asm volatile("" : "+s"(prm), "+v"(ln));
        const int c = ln & 15, g = ln >> 4;
        tile_forward<2>(prm, feat, p0, npts, ub, pbase, c, g, x0, A1, A2, zp, a3);
        // output layer: g4 = dL/dz4 = dL/dw scale sigmoid(z4); delta3 = g4 w4 (1 - a3^2)
        {
            const f4 w4 = load4(prm + oW4 + u0 + 4 * g);
            f4 s4 = zero, s3 = zero;
#pragma unroll
            for (int pb = 0; pb < 2; ++pb) {
                const int p = pbase + 16 * pb + c;
                const float g4 =
                    p0 + p < npts ? gw[p0 + p] * scale * sigmoid(out_unit(prm, zp, p)) : 0.f;
                const f4 d = g4 * w4 * (1.f - a3[pb] * a3[pb]);
                s4 += g4 * a3[pb];
                s3 += d;
                db4 += g4;
                *reinterpret_cast<f4*>(dl + p * kLd + u0 + 4 * g) = d;
            }
            dw4 += s4;
            db3 += s3;
        }
        float w[32];
        f4 t[4], acc[2];
        load_w_bwd(prm + oW3, u0, c, g, w);
        __syncthreads();
        // dW3t[k][j] += sum_p a2[p][k] delta3[p][j];  delta2 = (W3t delta3) (1 - a2^2)
        mm_points<4, kLd>(A2, 64 * ph, dl, u0, c, g, t);
#pragma unroll
        for (int k = 0; k < 4; ++k) dW3[k] += t[k];
        acc[0] = acc[1] = zero;
        mm_units<2>(w, dl, pbase, c, g, acc);
        load_w_bwd(prm + oW2, u0, c, g, w);
        __syncthreads();  // delta3 has been read
#pragma unroll
        for (int pb = 0; pb < 2; ++pb) {
            const int o = (pbase + 16 * pb + c) * kLd + u0 + 4 * g;
            const f4 a = *reinterpret_cast<const f4*>(A2 + o);
            acc[pb] *= 1.f - a * a;
            *reinterpret_cast<f4*>(dl + o) = acc[pb];
        }
        db2 += acc[0] + acc[1];
        __syncthreads();
        // the same for layer 2
        mm_points<4, kLd>(A1, 64 * ph, dl, u0, c, g, t);
#pragma unroll
        for (int k = 0; k < 4; ++k) dW2[k] += t[k];
        acc[0] = acc[1] = zero;
        mm_units<2>(w, dl, pbase, c, g, acc);
        __syncthreads();  // delta2 has been read
#pragma unroll
        for (int pb = 0; pb < 2; ++pb) {
            const int o = (pbase + 16 * pb + c) * kLd + u0 + 4 * g;
            const f4 a = *reinterpret_cast<const f4*>(A1 + o);
            *reinterpret_cast<f4*>(dl + o) = acc[pb] * (1.f - a * a);
        }
        __syncthreads();
        // dW1t and db1 (input row 12 is one)
        if (ph == 0) {
            f4 t1[1];
            mm_points<1, kLdX>(x0, 0, dl, u0, c, g, t1);
            dW1 += t1[0];
        }
        __syncthreads();
    }
    // sums over points held by lanes c (and by the two waves of a unit block): first over the lanes
    float* red = A1;  // [ph][3][kHid], then db4 of the two waves
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dw4[r] += __shfl_xor(dw4[r], o);
            db3[r] += __shfl_xor(db3[r], o);
            db2[r] += __shfl_xor(db2[r], o);
        }
        db4 += __shfl_xor(db4, o);
    }
    if (c == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            red[(3 * ph + 0) * kHid + u0 + 4 * g + r] = dw4[r];
            red[(3 * ph + 1) * kHid + u0 + 4 * g + r] = db3[r];
            red[(3 * ph + 2) * kHid + u0 + 4 * g + r] = db2[r];
        }
        if (ub == 0 && g == 0) red[6 * kHid + ph] = db4;
    }
    __syncthreads();
    float* out = partial + (int64_t)blockIdx.x * kParams;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 64 * ph + 16 * k + 4 * g + r;
            out[oW2 + row * kHid + u0 + c] = dW2[k][r];
            out[oW3 + row * kHid + u0 + c] = dW3[k][r];
        }
    if (ph == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * g + r;
            if (row < kIn) out[oW1 + row * kHid + u0 + c] = dW1[r];
            if (row == kIn) out[oB1 + u0 + c] = dW1[r];
        }
    }
    const int e = threadIdx.x;
    if (e < kHid) {
        out[oW4 + e] = red[e] + red[3 * kHid + e];
        out[oB3 + e] = red[kHid + e] + red[4 * kHid + e];
        out[oB2 + e] = red[2 * kHid + e] + red[5 * kHid + e];
        if (e == 0) out[oB4] = red[6 * kHid] + red[6 * kHid + 1];
    }
}

// grad[i] = sum of the partial vectors: 16 threads of a parameter each sum every 16th vector in
// order, then their sums are added in order
constexpr int kRedRows = 16;
__global__ __launch_bounds__(1024) void k_mlp_reduce(const float* __restrict__ partial, int nblocks,
                                                     float* __restrict__ grad)
{
    __shared__ float sh[kRedRows][64];
    const int x = threadIdx.x & 63, yy = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + x;
    float s = 0.f;
    if (i < kParams)
        for (int b = yy; b < nblocks; b += kRedRows) s += partial[(int64_t)b * kParams + i];
    sh[yy][x] = s;
    __syncthreads();
    if (yy == 0 && i < kParams) {
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < kRedRows; ++k) v += sh[k][x];
        grad[i] = v;
    }
}

__global__ void k_adam(float* __restrict__ prm, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    prm[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---- density map and features ----

__global__ void k_density_count(const double* __restrict__ th, const double* __restrict__ ph,
                                int64_t n, int nt, int np, unsigned int* __restrict__ cnt)
{
    // cell decisions are plain products and differences, rounded one at a time
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int a = (int)(th[i] * (nt / M_PI));
    a = min(max(a, 0), nt - 1);
    double pw = ph[i] - 2.0 * M_PI * floor(ph[i] / (2.0 * M_PI));
    int b = (int)(pw * (np / (2.0 * M_PI)));
    b = min(max(b, 0), np - 1);
    atomicAdd(&cnt[a * np + b], 1u);
}

__global__ void k_zero_counts(unsigned int* __restrict__ cnt, int n)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) cnt[e] = 0u;
}

// rho = count / (N * area / 4 pi): 1 for uniform points
__global__ void k_density_norm(const unsigned int* __restrict__ cnt, int nt, int np, int64_t n,
                               float* __restrict__ rho)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nt * np) return;
    const int a = e / np;
    const double area = (cos(M_PI * a / nt) - cos(M_PI * (a + 1) / nt)) * (2.0 * M_PI / np);
    rho[e] = (float)((double)cnt[e] / ((double)n * area / (4.0 * M_PI)));
}

__device__ inline float log_rho(const float* rho, int a, int b, int nt, int np)
{
    a = min(max(a, 0), nt - 1);
    b = ((b % np) + np) % np;
    return logf(fmaxf(rho[a * np + b], 1e-3f));
}

__global__ void k_features(const double* __restrict__ th, const double* __restrict__ ph, int64_t n,
                           const float* __restrict__ rho, int nt, int np, float* __restrict__ f)
{
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double t = th[i];
    const double pw = ph[i] - 2.0 * M_PI * floor(ph[i] / (2.0 * M_PI));
    // cell-centre coordinates for the bilinear interpolation
    const double u = t * (nt / M_PI) - 0.5, v = pw * (np / (2.0 * M_PI)) - 0.5;
    const int a0 = (int)floor(u), b0 = (int)floor(v);
    const float fu = (float)(u - a0), fv = (float)(v - b0);
    const float l00 = log_rho(rho, a0, b0, nt, np), l01 = log_rho(rho, a0, b0 + 1, nt, np);
    const float l10 = log_rho(rho, a0 + 1, b0, nt, np), l11 = log_rho(rho, a0 + 1, b0 + 1, nt, np);
    float* o = f + i * kIn;
    o[0] = (1 - fu) * ((1 - fv) * l00 + fv * l01) + fu * ((1 - fv) * l10 + fv * l11);
    const int ac = min(max((int)(t * (nt / M_PI)), 0), nt - 1);
    const int bc = min(max((int)(pw * (np / (2.0 * M_PI))), 0), np - 1);
    int q = 1;
    for (int da = -1; da <= 1; ++da)
        for (int db = -1; db <= 1; ++db) o[q++] = log_rho(rho, ac + da, bc + db, nt, np);
    o[10] = (float)cos(t);
    o[11] = (float)sin(t);
}

// ---- weight loss ----

__global__ void k_weighted_map(const float* __restrict__ w, const double* __restrict__ d,
                               double* __restrict__ out, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (double)w[i] * d[i];
}

__global__ void k_sub_alm(double2* __restrict__ c, const double2* __restrict__ a, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 v = c[i];
    const double2 b = a[i];
    v.x -= b.x;
    v.y -= b.y;
    c[i] = v;
}

constexpr int kRB = 1024, kRT = 256;

__global__ __launch_bounds__(kRT) void k_mdot(const double2* __restrict__ a, int64_t n, int lmax,
                                              double* __restrict__ partial)
{
    __shared__ double sh[kRT];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double2 x = a[i];
        const double v = x.x * x.x + x.y * x.y;
        acc += (i <= lmax) ? v : 2.0 * v;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kRT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(kRT) void k_sum(const double* __restrict__ partial, int n,
                                             double* __restrict__ out)
{
    __shared__ double sh[kRT];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) acc += partial[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kRT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

__global__ void k_weight_grad(const double* __restrict__ d, const double* __restrict__ q,
                              const double* __restrict__ den, float* __restrict__ g, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) g[i] = (float)(2.0 * d[i] * q[i] / *den);
}

// blocks of the backward pass: one per CU (106 KB of LDS, 16 waves)
constexpr int kBwdBlocks = 256;

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace
}  // namespace nusht

using namespace nusht;

extern "C" {

int64_t nusht_mlp_param_count(void) { return kParams; }

int nusht_density_map(const double* theta, const double* phi, int64_t npts, int ntheta, int nphi,
                      float* density, void* stream)
{
    if (!theta || !phi || !density || npts < 1 || ntheta < 1 || nphi < 1 ||
        (int64_t)ntheta * nphi > (1 << 24)) {
        set_last_error("nusht_density_map", "bad arguments");
        return NUSHT_EINVAL;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    unsigned int* cnt = nullptr;
    const size_t nb = (size_t)ntheta * nphi;
    NUSHT_HIP(hipMallocAsync((void**)&cnt, nb * sizeof(unsigned int), s));
    NUSHT_HIP(hipMemsetAsync(cnt, 0, nb * sizeof(unsigned int), s));
    hipLaunchKernelGGL(k_density_count, dim3(nblk(npts)), dim3(256), 0, s, theta, phi, npts,
                       ntheta, nphi, cnt);
    hipLaunchKernelGGL(k_density_norm, dim3(nblk((int64_t)nb)), dim3(256), 0, s, cnt, ntheta,
                       nphi, npts, density);
    NUSHT_HIP(hipGetLastError());
    NUSHT_HIP(hipFreeAsync(cnt, s));
    return NUSHT_OK;
}

// Fixed device array holding the cell counts of nusht_density_map_noalloc, one copy per GPU
// for the life of the process (kDensityScratchCells counts, 256 KiB).  Host code never passes
// `scratch` itself to a kernel: its device address on each GPU comes from
// hipGetSymbolAddress, looked up once per device on that device's first call.
constexpr int kDensityScratchCells = 1 << 16;
static __device__ __align__(256) unsigned int scratch[kDensityScratchCells];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned int* g_scratch_ptr[kMaxDevices] = {};

int density_scratch(unsigned int** out)
{
    int dev = 0;
    NUSHT_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        set_last_error("nusht_density_map_noalloc", "device index out of range");
        return NUSHT_EDEVICE;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        NUSHT_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        g_scratch_ptr[dev] = reinterpret_cast<unsigned int*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return NUSHT_OK;
}
}  // namespace

int nusht_density_map_noalloc(const double* theta, const double* phi, int64_t npts, int ntheta,
                              int nphi, float* density, void* stream)
{
    if (!theta || !phi || !density || npts < 1 || ntheta < 1 || nphi < 1) {
        set_last_error("nusht_density_map_noalloc", "bad arguments");
        return NUSHT_EINVAL;
    }
    if ((int64_t)ntheta * nphi > kDensityScratchCells) {
        set_last_error("nusht_density_map_noalloc",
                       "ntheta * nphi exceeds the fixed count buffer (65536 cells)");
        return NUSHT_EINVAL;
    }
    unsigned int* cnt = nullptr;
    NUSHT_TRY(density_scratch(&cnt));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int nb = ntheta * nphi;
    // the counts are cleared by a kernel (the previous call's counts are still there)
    hipLaunchKernelGGL(k_zero_counts, dim3(nblk(nb)), dim3(256), 0, s, cnt, nb);
    hipLaunchKernelGGL(k_density_count, dim3(nblk(npts)), dim3(256), 0, s, theta, phi, npts,
                       ntheta, nphi, cnt);
    hipLaunchKernelGGL(k_density_norm, dim3(nblk((int64_t)nb)), dim3(256), 0, s, cnt, ntheta,
                       nphi, npts, density);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

int nusht_point_features(const double* theta, const double* phi, int64_t npts,
                         const float* density, int ntheta, int nphi, float* features,
                         void* stream)
{
    if (!theta || !phi || !density || !features || npts < 1 || ntheta < 1 || nphi < 1) {
        set_last_error("nusht_point_features", "bad arguments");
        return NUSHT_EINVAL;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_features, dim3(nblk(npts)), dim3(256), 0, s, theta, phi, npts, density,
                       ntheta, nphi, features);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

int nusht_mlp_forward(const float* params, const float* features, int64_t npts, float scale,
                      float* weights, void* stream)
{
    if (!params || !features || !weights || npts < 1) return NUSHT_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t tiles = (npts + kTileP - 1) / kTileP;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)tiles), dim3(512), 0, s, params, features,
                       npts, scale, weights);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

int nusht_mlp_backward(const float* params, const float* features, const float* grad_weights,
                       int64_t npts, float scale, float* grad_params, void* stream)
{
    if (!params || !features || !grad_weights || !grad_params || npts < 1) return NUSHT_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t tiles = (npts + kTileP - 1) / kTileP;
    const int blocks = (int)(tiles < kBwdBlocks ? tiles : kBwdBlocks);
    float* partial = nullptr;
    NUSHT_HIP(hipMallocAsync((void**)&partial, (size_t)blocks * kParams * sizeof(float), s));
    hipLaunchKernelGGL(k_mlp_backward, dim3(blocks), dim3(1024), 0, s, params, features,
                       grad_weights, npts, scale, partial);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((kParams + 63) / 64), dim3(1024), 0, s, partial, blocks,
                       grad_params);
    NUSHT_HIP(hipGetLastError());
    NUSHT_HIP(hipFreeAsync(partial, s));
    return NUSHT_OK;
}

int nusht_adam_step(float* params, const float* grad, float* m, float* v, int64_t n, float lr,
                    float beta1, float beta2, float eps, int step, void* stream)
{
    if (!params || !grad || !m || !v || n < 1 || step < 1) return NUSHT_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(nblk(n)), dim3(256), 0, s, params, grad, m, v, n, lr, beta1,
                       beta2, eps, c1, c2);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

int nusht_weighted_adjoint(nusht_plan_t p, const double* d, const float* weights, double* alm,
                           void* stream)
{
    if (!p || !d || !weights || !alm) {
        set_last_error("nusht_weighted_adjoint", "null argument");
        return NUSHT_EINVAL;
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t n = p->g.npts;
    double* wd = nullptr;
    NUSHT_HIP(hipMallocAsync((void**)&wd, n * sizeof(double), s));
    hipLaunchKernelGGL(k_weighted_map, dim3(nblk(n)), dim3(256), 0, s, weights, d, wd, n);
    const int rc = nusht_adjoint(p, wd, alm, 1, stream);
    hipFreeAsync(wd, s);
    NUSHT_HIP(hipGetLastError());
    return rc;
}

int nusht_weight_loss_grad(nusht_plan_t p, const double* d, const double* astar,
                           const float* weights, float* grad_weights, double* loss, void* stream)
{
    if (!p || !d || !astar || !weights || !loss) return NUSHT_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t n = p->g.npts, na = p->g.nalm;
    double *wd = nullptr, *q = nullptr, *part = nullptr, *sc = nullptr;
    double2* c = nullptr;
    NUSHT_HIP(hipMallocAsync((void**)&wd, n * sizeof(double), s));
    NUSHT_HIP(hipMallocAsync((void**)&q, n * sizeof(double), s));
    NUSHT_HIP(hipMallocAsync((void**)&c, na * sizeof(double2), s));
    NUSHT_HIP(hipMallocAsync((void**)&part, (kRB + 4) * sizeof(double), s));
    sc = part + kRB;
    int rc = NUSHT_OK;
    do {
        hipLaunchKernelGGL(k_weighted_map, dim3(nblk(n)), dim3(256), 0, s, weights, d, wd, n);
        if ((rc = nusht_adjoint(p, wd, reinterpret_cast<double*>(c), 1, stream))) break;
        hipLaunchKernelGGL(k_sub_alm, dim3(nblk(na)), dim3(256), 0, s, c,
                           reinterpret_cast<const double2*>(astar), na);
        hipLaunchKernelGGL(k_mdot, dim3(kRB), dim3(kRT), 0, s, c, na, p->g.lmax, part);
        hipLaunchKernelGGL(k_sum, dim3(1), dim3(kRT), 0, s, part, kRB, sc);
        hipLaunchKernelGGL(k_mdot, dim3(kRB), dim3(kRT), 0, s,
                           reinterpret_cast<const double2*>(astar), na, p->g.lmax, part);
        hipLaunchKernelGGL(k_sum, dim3(1), dim3(kRT), 0, s, part, kRB, sc + 1);
        if (grad_weights) {
            if ((rc = nusht_synthesis(p, reinterpret_cast<const double*>(c), q, 1, stream))) break;
            hipLaunchKernelGGL(k_weight_grad, dim3(nblk(n)), dim3(256), 0, s, d, q, sc + 1,
                               grad_weights, n);
        }
        double h[2];
        if (hipMemcpyAsync(h, sc, 2 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) {
            rc = NUSHT_EDEVICE;
            break;
        }
        *loss = h[1] > 0.0 ? h[0] / h[1] : 0.0;
    } while (0);
    hipFreeAsync(wd, s);
    hipFreeAsync(q, s);
    hipFreeAsync(c, s);
    hipFreeAsync(part, s);
    NUSHT_HIP(hipGetLastError());
    return rc;
}

}  // extern "C"
