// Transforms of the fine grid for lengths that are not 2^K or 5 2^K (arXiv:2406.14542 Sec. III):
// any N = 2^a 3^b 5^c 7^d that fits in LDS, one workgroup per window row (phi pass) or band
// column (theta pass).  The radices (2 .. 10 and 12) come with the launch; every pass is a
// Stockham pass through one LDS array: a thread loads the inputs of its butterflies, transforms
// them in registers, the block synchronises, then the outputs are stored.  The first pass reads
// HBM and the last one writes it, so a row or column moves once in and once out.
//
// The theta pass also holds the DFT over the doubled circle (F, length N_t): the column of the
// Legendre step is transformed, deconvolved, padded and transformed back (or the reverse) without
// leaving LDS.
//
// FP64 plans only: in mixed precision another order of FP32 roundings would move results by 1e-7,
// so those plans keep the transforms they had.
//
// What bounds them: latency of the LDS exchanges and of the twiddle loads.  N / 8 threads give
// twice the waves of a radix-16 split (below 128 registers in FP64) and one or two butterflies
// per thread for every radix.  Measured against rocFFT's chains of 3 to 6 kernels (transposes,
// real post-processing, padded copies): lmax 1500 (columns 6048 and 3024, rows 6048), three
// synthesis maps 1960 -> 565 us (0.9 GB moved, 1.6 TB/s); lmax 1000, mmax 900, five adjoint maps
// 980 -> 366 us.
#include <algorithm>

#include "fft_core.h"
#include "internal.h"

namespace nusht {
namespace {

using T = double;
using C = double2;

// One pass of radix R and span ns over N values: butterfly b reads ld(b + r N / R), output r goes
// to st((b - j) R + j + r ns) with j = b mod ns.  tw[m] = e^{2 pi i m / (2 N)}.  V: values per
// thread (N <= V nt).  BAR: loads and stores meet in the same LDS array.
template <int R, int DIR, int V, bool FIRST, bool BAR, typename C, typename LD, typename ST>
__device__ __forceinline__ void mix_pass(int t, int nt, int N, int ns, const C* __restrict__ tw,
                                         LD ld, ST st)
{
    constexpr int Q = (V + R - 1) / R;
    const int nb = N / R;
    const float inv = 1.0f / (float)ns;
    const int step = 2 * (nb / ns);
    C v[Q][R];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = t + q * nt;
        if (b < nb) {
#pragma unroll
            for (int r = 0; r < R; ++r) v[q][r] = ld(b + r * nb);
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = t + q * nt;
        if (b < nb) {
            if (!FIRST) {
                // exact: b < 2^15, so (b + 1/2) / ns is at least 2^-16 away from an integer
                const int j = b - ns * (int)(((float)b + 0.5f) * inv);
                const int s = j * step;
                C w[R];
                // w, w^2, w^4 and w^8 from the table, the others by at most two products
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    if ((r & (r - 1)) == 0) {
                        w[r] = tw[r * s];
                        if (DIR < 0) w[r].y = -w[r].y;
                    }
                }
#pragma unroll
                for (int r = 3; r < R; ++r) {
                    if ((r & (r - 1)) != 0) {
                        const int top = r >= 8 ? 8 : r >= 4 ? 4 : 2;
                        w[r] = cmul(w[top], w[r - top]);
                    }
                }
#pragma unroll
                for (int r = 1; r < R; ++r) v[q][r] = cmul(v[q][r], w[r]);
            }
            dft<R, DIR>(v[q]);
        }
        // one butterfly's twiddles at a time: several at once would spill (128 registers)
        if (Q > 1 && !FIRST) __builtin_amdgcn_sched_barrier(0);
    }
    if (BAR) __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int b = t + q * nt;
        if (b < nb) {
            const int j = FIRST ? 0 : b - ns * (int)(((float)b + 0.5f) * inv);
            const int base = (b - j) * R + j;
#pragma unroll
            for (int r = 0; r < R; ++r) st(base + r * ns, v[q][r]);
        }
    }
}

template <int DIR, int V, bool FIRST, bool BAR, typename C, typename LD, typename ST>
__device__ __forceinline__ void mix_any(int R, int t, int nt, int N, int ns, const C* __restrict__ tw, LD ld,
                               ST st)
{
    switch (R) {
#define NUSHT_MIX_CASE(RR) \
    case RR: mix_pass<RR, DIR, V, FIRST, BAR>(t, nt, N, ns, tw, ld, st); break;
        NUSHT_MIX_CASE(2) NUSHT_MIX_CASE(3) NUSHT_MIX_CASE(4) NUSHT_MIX_CASE(5) NUSHT_MIX_CASE(6)
        NUSHT_MIX_CASE(7) NUSHT_MIX_CASE(8) NUSHT_MIX_CASE(9) NUSHT_MIX_CASE(10) NUSHT_MIX_CASE(12)
#undef NUSHT_MIX_CASE
    }
}

// all passes; ld(i) gives input i, st(k, v) takes output k.  LDSIN / LDSOUT: ld / st touch buf.
// The caller synchronises after it when st writes buf.
template <int DIR, int V, bool LDSIN, bool LDSOUT, typename C, typename LD, typename ST>
__device__ __forceinline__ void mix_fft(const MixLen& m, C* buf, int t, int nt, const C* __restrict__ tw,
                               LD ld, ST st)
{
    const auto from = [buf](int i) { return buf[pad16(i)]; };
    const auto to = [buf](int i, C v) { buf[pad16(i)] = v; };
    mix_any<DIR, V, true, LDSIN>(m.radix(0), t, nt, m.n, 1, tw, ld, to);
    __syncthreads();
    int ns = m.radix(0);
    for (int p = 1; p < m.np - 1; ++p) {
        // opaque to the compiler: it would move the addresses of all ten cases out of the loop
        int n = m.n, tt = t;
        asm volatile("" : "+s"(n), "+v"(tt));
        mix_any<DIR, V, false, true>(m.radix(p), tt, nt, n, ns, tw, from, to);
        __syncthreads();
        ns *= m.radix(p);
    }
    mix_any<DIR, V, false, LDSOUT>(m.radix(m.np - 1), t, nt, m.n, ns, tw, from, st);
}

__device__ inline C* mix_lds()
{
    extern __shared__ char mix_lds_raw[];
    return reinterpret_cast<C*>(mix_lds_raw);
}

// C2R of window rows (the half-length route of rowfft.hip): blockIdx.x = compact window row
template <int V>
__global__ __launch_bounds__(1024) void k_mix_c2r(MixLen m, const C* __restrict__ rows,
                                                 int64_t rw, int ncol, T* __restrict__ fine, int n1,
                                                 int ra, int rb,
                                                 const C* __restrict__ tw)
{
    C* buf = mix_lds();
    const int q = blockIdx.x, N = m.n, M = ncol - 1;
    const int i = q < ra ? q : n1 - rb + (q - ra);
    rows += (int64_t)blockIdx.y * n1 * rw;  // map of the launch
    fine += (int64_t)blockIdx.y * n1 * (2 * N);
    const C* X = rows + (int64_t)i * rw;
    C* z = reinterpret_cast<C*>(fine + (int64_t)i * (2 * N));
    // Z[k] from X[k] and conj X[N - k]; band columns only (clamped loads, so no branch)
    const auto ld = [=](int k) {
        C xk = X[min(k, M)], xm = X[min(N - k, M)];
        const C w = tw[k];
        if (k > M) xk = cmk<C>(0, 0);
        if (k == 0) xk.y = 0;
        if (k == 0 || N - k > M) xm = cmk<C>(0, 0);
        const C xc = cmk<C>(xm.x, -xm.y);
        const C e = cadd(xk, xc), o = cmul(csub(xk, xc), w);
        return cmk<C>(e.x - o.y, e.y + o.x);
    };
    mix_fft<+1, V, false, false>(m, buf, threadIdx.x, blockDim.x, tw, ld,
                                 [z](int k, C v) { z[k] = v; });
}

// R2C of window rows, columns 0 .. ncol-1 of each row's spectrum
template <int V>
__global__ __launch_bounds__(1024) void k_mix_r2c(MixLen m, const T* __restrict__ fine, int n1, int ra,
                                                 int rb, C* __restrict__ rows,
                                                 int64_t rw, int ncol,
                                                 const C* __restrict__ tw)
{
    C* buf = mix_lds();
    const int q = blockIdx.x, N = m.n;
    const int i = q < ra ? q : n1 - rb + (q - ra);
    rows += (int64_t)blockIdx.y * n1 * rw;  // map of the launch
    fine += (int64_t)blockIdx.y * n1 * (2 * N);
    const C* z = reinterpret_cast<const C*>(fine + (int64_t)i * (2 * N));
    mix_fft<-1, V, false, true>(m, buf, threadIdx.x, blockDim.x, tw, [z](int k) { return z[k]; },
                                [buf](int k, C v) { buf[pad16(k)] = v; });
    __syncthreads();
    C* X = rows + (int64_t)i * rw;
    for (int k = threadIdx.x; k < ncol; k += blockDim.x) {
        const C zk = buf[pad16(k)];
        const C zm = buf[pad16(k == 0 ? 0 : N - k)];
        C w = tw[k];
        w.y = -w.y;
        const C e = cmk<C>((zk.x + zm.x) / 2, (zk.y - zm.y) / 2);
        const C d = cmk<C>((zk.x - zm.x) / 2, (zk.y + zm.y) / 2);
        X[k] = cadd(e, cmul(cmk<C>(d.y, -d.x), w));
    }
}

// synthesis: doubled Legendre columns cs[b][mu][t] (t < N_t) -> band[b][mu][i], window rows only:
// DFT over t, entries |k| <= L times the deconvolution factors, zero-padded DFT back over n1
template <int V>
__global__ __launch_bounds__(1024) void k_mix_theta_inv(
    MixLen mt, MixLen mn, const C* __restrict__ cs,
    C* __restrict__ band, int lmax, const T* __restrict__ d1,
    const T* __restrict__ d2, int ra, int rb, const C* __restrict__ twt,
    const C* __restrict__ twn)
{
    C* buf = mix_lds();
    const int t = threadIdx.x, nt = blockDim.x;
    const int64_t col = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const C* src = cs + col * mt.n;
    C* dst = band + col * mn.n;
    const T fm = d2[blockIdx.x];
    mix_fft<-1, V, false, true>(mt, buf, t, nt, twt, [src](int i) { return src[i]; },
                                [buf](int k, C v) { buf[pad16(k)] = v; });
    __syncthreads();
    const int N = mn.n, Nt = mt.n;
    const auto ld = [=](int i) {
        const int k = kappa_of(i, N);
        const int ak = k < 0 ? -k : k;
        C v = cmk<C>(0, 0);
        if (ak <= lmax) {
            const C c = buf[pad16(k < 0 ? k + Nt : k)];
            const T f = d1[ak] * fm;
            v = cmk<C>(c.x * f, c.y * f);
        }
        return v;
    };
    mix_fft<+1, V, true, false>(mn, buf, t, nt, twn, ld, [=](int i, C v) {
        if (i < ra || i >= N - rb) dst[i] = v;
    });
}

// adjoint: band[b][mu][i] (window rows; the others are zero) -> columns cs[b][mu][t]
template <int V>
__global__ __launch_bounds__(1024) void k_mix_theta_fwd(
    MixLen mt, MixLen mn, const C* __restrict__ band,
    C* __restrict__ cs, int lmax, const T* __restrict__ d1,
    const T* __restrict__ d2, int ra, int rb, const C* __restrict__ twt,
    const C* __restrict__ twn)
{
    C* buf = mix_lds();
    const int t = threadIdx.x, nt = blockDim.x;
    const int64_t col = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int N = mn.n, Nt = mt.n;
    const C* src = band + col * N;
    C* dst = cs + col * Nt;
    const T fm = d2[blockIdx.x];
    const auto in = [=](int i) {
        C v = cmk<C>(0, 0);
        if (i < ra || i >= N - rb) v = src[i];
        return v;
    };
    mix_fft<-1, V, false, true>(mn, buf, t, nt, twn, in, [buf](int k, C v) { buf[pad16(k)] = v; });
    __syncthreads();
    const auto ld = [=](int e) {
        const int k = kappa_of(e, Nt);
        const int ak = k < 0 ? -k : k;
        C v = cmk<C>(0, 0);
        if (ak <= lmax) {
            const C c = buf[pad16(k < 0 ? k + N : k)];
            const T f = d1[ak] * fm;
            v = cmk<C>(c.x * f, c.y * f);
        }
        return v;
    };
    mix_fft<+1, V, true, false>(mt, buf, t, nt, twt, ld, [dst](int e, C v) { dst[e] = v; });
}

// at most 8 values per thread up to 8192 (one butterfly of radix 8 to 12, two of 5 to 7), more above
int threads_for(int n) { return std::min(1024, (n + 511) / 512 * 64); }

// the instance of F for this length, as F<V>
#define NUSHT_MIX_LAUNCH(F, N_, grid, ...)                                                      \
    do {                                                                                            \
        const int nt_ = threads_for(N_);                                                            \
        const size_t lds_ = (size_t)((N_) + (N_) / 16 + 1) * sizeof(C);                        \
        if ((N_) <= 8192)                                                                           \
            hipLaunchKernelGGL(F<8>, grid, dim3(nt_), lds_, s, __VA_ARGS__);                  \
        else                                                                                        \
            hipLaunchKernelGGL(F<9>, grid, dim3(nt_), lds_, s, __VA_ARGS__);                   \
    } while (0)

int mix_row(const nusht_plan_s* p, const MixLen& m, const void* in, void* out, int64_t rw,
            int nb, bool c2r, hipStream_t s)
{
    const nusht_geometry& g = p->g;
    const dim3 grid(p->fine_ra + p->fine_rb, nb);
    const C* tw = reinterpret_cast<const C*>(p->rowtw);
    if (c2r)
        NUSHT_MIX_LAUNCH(k_mix_c2r, m.n, grid, m, reinterpret_cast<const C*>(in), rw, g.mmax + 1,
                         reinterpret_cast<T*>(out), g.n1, p->fine_ra, p->fine_rb, tw);
    else
        NUSHT_MIX_LAUNCH(k_mix_r2c, m.n, grid, m, reinterpret_cast<const T*>(in), g.n1, p->fine_ra,
                         p->fine_rb, reinterpret_cast<C*>(out), rw, g.mmax + 1, tw);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

int mix_theta(const nusht_plan_s* p, const MixLen& mt, const MixLen& mn, const void* in, void* out,
              int nmaps, bool inv, hipStream_t s)
{
    const nusht_geometry& g = p->g;
    const dim3 grid(g.mmax + 1, nmaps);
    const T *d1 = p->dec1, *d2 = p->dec2;
    const C* twt = reinterpret_cast<const C*>(p->torustw);
    const C* twn = reinterpret_cast<const C*>(p->thetatw);
    const C* src = reinterpret_cast<const C*>(in);
    C* dst = reinterpret_cast<C*>(out);
    if (inv)
        NUSHT_MIX_LAUNCH(k_mix_theta_inv, mn.n, grid, mt, mn, src, dst, g.lmax, d1, d2, p->fine_ra,
                         p->fine_rb, twt, twn);
    else
        NUSHT_MIX_LAUNCH(k_mix_theta_fwd, mn.n, grid, mt, mn, src, dst, g.lmax, d1, d2, p->fine_ra,
                         p->fine_rb, twt, twn);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

// fewest passes, then the smallest sum of radices; false when n has other factors
bool factor(int n, int maxr, int depth, int* cur, int* best, int& nbest, int& sbest, int sum)
{
    if (n == 1) {
        if (depth < nbest || (depth == nbest && sum < sbest)) {
            nbest = depth;
            sbest = sum;
            for (int i = 0; i < depth; ++i) best[i] = cur[i];
        }
        return true;
    }
    if (depth >= 8 || depth >= nbest) return false;
    bool any = false;
    for (int r : {12, 10, 9, 8, 7, 6, 5, 4, 3, 2}) {
        if (r > maxr || n % r) continue;
        cur[depth] = r;
        any |= factor(n / r, r, depth + 1, cur, best, nbest, sbest, sum + r);
    }
    return any;
}

}  // namespace

// Two passes at least (one reads HBM, one writes it).  Odd radices first: their stores of stride
// R in the first pass fall on distinct banks.
bool mix_len(int n, MixLen* m)
{
    int cur[8], best[8], nb = 9, sb = 0;
    if (n < 16 || !factor(n, 12, 0, cur, best, nb, sb, 0) || nb < 2 || nb > 8) return false;
    m->n = n;
    m->np = 0;
    m->code = 0;
    for (int odd = 1; odd >= 0; --odd)
        for (int i = 0; i < nb; ++i)
            if ((best[i] & 1) == odd) m->code |= (unsigned long long)best[i] << (4 * m->np++);
    return true;
}

// Both are decided on the geometry alone: every length of the geometry is 7-smooth, so the limit
// is the LDS of one workgroup (N <= 9035: lmax about 2200 at sigma 2).
// Longer ones stay with rocFFT: no kernel here holds them.
bool mixrow_supported(const nusht_geometry& g)
{
    MixLen m;
    return g.dtype == NUSHT_F64 && g.n2 % 2 == 0 && lds_fits<double>(g.n2 / 2) &&
           g.mmax + 1 <= g.n2 / 2 && mix_len(g.n2 / 2, &m);
}

bool mixtheta_supported(const nusht_geometry& g)
{
    MixLen m;
    return g.dtype == NUSHT_F64 && g.dfs_mode == NUSHT_DFS_FUSED && lds_fits<double>(g.n1) &&
           g.ntorus <= g.n1 && mix_len(g.n1, &m) && mix_len(g.ntorus, &m);
}

int launch_mix_row(const nusht_plan_s* p, const void* in, void* out, int64_t rw, int nb,
                   bool c2r, hipStream_t s)
{
    return mix_row(p, p->mix_row, in, out, rw, nb, c2r, s);
}

int launch_mix_theta(const nusht_plan_s* p, const void* in, void* out, int nmaps, bool inv,
                     hipStream_t s)
{
    return mix_theta(p, p->mix_torus, p->mix_theta, in, out, nmaps, inv, s);
}

}  // namespace nusht
