// Legendre step of the iso-latitude transform S (arXiv:2406.14542 Sec. III, "critical part"):
//   synthesis  G_m(theta_j) = sum_{l=m}^{L} a_lm lam_lm(cos theta_j)
//   adjoint    c_lm = sum_j lam_lm(cos theta_j) G'_m(theta_j)
// on the Clenshaw-Curtis rings theta_j = j pi / (N_r - 1).  lam_lm is generated on the fly by
// the three-term recurrence in l (only the O(L^2) coefficient table is stored); the work is
// parallel over rings and m and sequential over l, as the paper describes for SHTns.
//
// gfx950 mapping:
//  * one lane = one pair of mirror rings (j, N_r-1-j): lam_lm(-x) = (-1)^(l+m) lam_lm(x), so
//    one recurrence serves both hemispheres through even/odd-l accumulators;
//  * every lane of a block has the same m, so the recurrence coefficients and a_lm of a step
//    are wave-uniform and are read through the scalar cache;
//  * x * v is formed as v - y v with y = 2 sin^2(theta/2): 1 - cos(theta) keeps full relative
//    precision near the poles, where d lam / d x grows like l^2;
//  * exponent range: lam_mm underflows FP64 for m of a few thousand near the poles.  Each
//    lane carries a count k of 2^256 factors; while any lane of the wave has k > 0 the wave
//    runs a rescaling step, afterwards the plain recurrence.  Terms whose true magnitude is
//    below 2^-200 (below 2^-144 where the test is made once per eight steps) are dropped: they
//    cannot reach the FP64 result.
#include "internal.h"
#include "wave_sum.h"

#include <algorithm>
#include <type_traits>

namespace nusht {
namespace {

constexpr double kBig = 0x1p56;       // rescale once the scaled value reaches this
constexpr double kUnit = 0x1p-256;    // one scale unit
constexpr int kAccumExp = -200;       // terms below 2^-200 are not accumulated

// lam_mm(theta_j) = c_m sin^m(theta_j), returned as v * 2^(-256 k) with v normal.
__device__ inline void lambda_mm_scaled(double cm, int ce, double s, int m, double& v, int& k)
{
    double mant;
    int e;
    if (m == 0) {
        mant = cm;
        e = ce;
    } else if (s == 0.0) {
        v = 0.0;
        k = 0;
        return;
    } else {
        int be;
        double base = frexp(s, &be);
        double r = 1.0;
        int re = 0;
        int mm = m;
        while (mm) {
            int t;
            if (mm & 1) {
                r *= base;
                re += be;
                r = frexp(r, &t);
                re += t;
            }
            mm >>= 1;
            if (mm) {
                base *= base;
                be *= 2;
                base = frexp(base, &t);
                be += t;
            }
        }
        int t;
        mant = frexp(cm * r, &t);
        e = ce + re + t;
    }
    if (e >= kAccumExp) {
        v = ldexp(mant, e);
        k = 0;
    } else {
        k = (kAccumExp - e + 255) / 256;
        v = ldexp(mant, e + 256 * k);
    }
}

// geometry of ring j of a grid with nr rings: returns (s = sin theta_j, y = 1 - cos theta_j)
__device__ inline void ring_geom(int j, int nr, double& s, double& y)
{
    const double denom = (double)(nr - 1);
    s = sinpi((double)j / denom);
    if (2 * j == nr - 1) {
        y = 1.0;
    } else {
        double h = sinpi((double)j / (2.0 * denom));
        y = 2.0 * h * h;
    }
}

// one recurrence step: returns lam_l from (lam_{l-1} = vc, lam_{l-2} = vp)
__device__ inline double rec_step(double2 c, double y, double vc, double vp)
{
    double xv = fma(-y, vc, vc);
    return fma(c.x, xv, -(c.y * vp));
}

// The coefficient stream of one m (recurrence table and MB coefficient rows) is read through
// the scalar cache, one l at a time, by every wave of that m; a miss costs a trip to HBM that
// the few resident waves cannot hide.  Every kPfStep values of l the wave therefore touches
// the next kPfStep coefficients of each stream, kPfStep steps ahead, with one load per
// 128-byte line, so that the scalar loads find them in L2.  The touch is an LDS-DMA load
// (global_load_lds_dword) in inline assembly: it has no register destination, so the
// compiler never waits for it, and the statement is declared free of memory effects, so the
// compiler still knows the coefficients are read-only and keeps their loads scalar.  (It
// does write LDS: a per-wave sink that nothing reads; the wave waits for the DMA once,
// before its LDS is released.)  M0, the DMA's LDS base, is restored afterwards.  The
// statement returns the saved M0 so that it stays live; the caller folds it into a value
// consumed at the end.
constexpr int kPfStep = 32;
constexpr int kPfLines = kPfStep * 16 / 128 + 1;  // lines per stream (unaligned start)

__device__ inline unsigned lds_dma_touch(const void* src, unsigned lds_sink)
{
    unsigned saved;
    asm("s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dword %1, off\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(src), "s"(lds_sink));
    return saved;
}

// the lane's line of the MB + 1 streams (rec, then MB rows of alm): first coefficient, null if none
template <int MB>
__device__ inline const double2* touch_line(const double2* __restrict__ rec,
                                            const double2* __restrict__ alm, int64_t nalm,
                                            int64_t moff, int lane, int& off)
{
    const int stream = lane / kPfLines;
    off = 8 * (lane - stream * kPfLines);
    if (stream > MB) return nullptr;
    return (stream == 0 ? rec : alm + (int64_t)(stream - 1) * nalm) + moff;
}

__device__ inline unsigned touch_coeffs(const double2* line, int off, int lp, int lmax,
                                        unsigned lds_sink)
{
    if (!line || lp > lmax) return 0u;
    return lds_dma_touch(line + min(lp + off, lmax), lds_sink);
}

// ------------------------------------------------------------------------------------
// Synthesis.  FUSED: out[b][m][t], t < N_t, the doubled column of Fig. 1 in (theta, m)
// space: out(t) = G(t) for t < N_r and (-1)^m G(N_t - t) for t >= N_r.  PAPER:
// out[b][j][m], rows of length (N_phi/2 + 1), the input of the per-ring phi-FFT.
// ------------------------------------------------------------------------------------
template <typename OutT>
__device__ inline OutT make_out(double re, double im)
{
    OutT o;
    o.x = re;
    o.y = im;
    return o;
}

// XCD-aware placement: workgroups are handed to the 8 XCDs round-robin by linear id, and
// every XCD has its own L2.  Block id b = 8 q + x goes to XCD x; the q-th block of XCD x
// gets (m, ring block) = (8 (q / nbx) + x, q % nbx), so all nbx ring blocks of one m run
// on the same XCD at about the same time and fetch that m's coefficient stream into one
// L2 once.  The grid is (nbx * mpad, groups) with mpad = mmax + 1 rounded up to 8.
__device__ inline void xcd_block(int b, int nbx, int& m, int& rb)
{
    const int x = b & 7, q = b >> 3;
    m = 8 * (q / nbx) + x;
    rb = q % nbx;
}

// Work split, for each m: the live pairs (from jlive[m] on) are cut into sub-blocks of 64 neighbours,
// counted from the equator; the fewest waves that hold them at R per wave take them in turn, so that
// every wave has pairs of all latitudes and the waves of one m are equally long: waves of unlike
// length, or blocks of unlike weight in a fixed order, leave SIMDs and shader engines idle (the one-map
// adjoint in blocks of 4 waves and 1 wave by turns took 1.24 instead of 0.82 ms at lmax 2047).  A lane
// runs the recurrence of its R pairs, one of each sub-block, and reads every coefficient once for all
// of them.
//
// Exponent range: a sub-block runs in the cheapest of three forms: every pair scaled (the
// recurrence only), some scaled (each value times 1 or 0), none.  Sub-blocks come into range in
// order, the equator first; each state (how many are in range, how many have a pair in range) has a
// loop of its own, straight-line code without copies of the sums.  The rescale test is made once
// per chunk of eight steps, which grow a value by less than 2^56: a scaled value stays below 2^112 and is
// dropped below 2^-144.
//
// Bound by the FP64 VALU: (3 + 2 MB) R instructions per l and wave, and by the coefficients' scalar
// loads.  One map at lmax 127 / 1023 / 1535 / 2047 / 4095: 12 / 84 / 225 / 432 / 2573 us against 43 / 149 /
// 522 / 603 / 3132 us of two kernels (scaled and unscaled rings) on forked streams with contiguous rings
// per wave and coefficients loaded when used; four maps at 127 / 1023 / 2047 / 4095 18 / 165 / 857 / 6270
// against 42 / 250 / 1162 / 7035 us.
constexpr int kSynLC = 8;               // l values per chunk of the synthesis

// Most waves per block.  Four maps: blocks of four are faster up to lmax 3700 (8 / 4 waves in us, lmax
// 2047 915 / 864, 3000 3171 / 2754, 4095 6395 / 6339); one map and its adjoint are slower in blocks
// of four above lmax 3100 (1451 / 1525 and 2139 / 2399 at 3200).
constexpr int sub_waves(int mb) { return mb == 4 ? 4 : 8; }

// Blocks of the kernels that split one m's live pairs over waves of R sub-blocks.  For m > 0 the
// pole's pair is never live, so that 2^k + 1 pairs (lmax = 2^k' - 1) leave no sub-block of one pair: the
// launch has waves for npairs - 1 pairs, and m = 0 gets one more block, in front, where it needs it
// (grid: 8 ids, of which one is used, so that the others keep their XCD).  Wave w of block rb is
// the m's wave w nbx + rb: blocks of equal weight.
struct SubGrid {
    int nbx, wpb, extra;
    __host__ __device__ SubGrid(int npairs, int R, int most)
    {
        const int nw = (npairs + 64 * R - 2) / (64 * R), nw0 = (npairs + 64 * R - 1) / (64 * R);
        const int n = nw > 0 ? nw : 1;
        nbx = (n + most - 1) / most;
        wpb = (n + nbx - 1) / nbx;
        extra = nw0 > nbx * wpb ? 8 : 0;
    }
    // column m and wave pc of this wave; m > mmax: none
    __device__ void place(int block, int wave, int mmax, int& m, int& pc) const
    {
        if (block < extra) {
            m = block == 0 ? 0 : mmax + 1;
            pc = nbx * wpb + wave;
            return;
        }
        int rb;
        xcd_block(block - extra, nbx, m, rb);
        pc = wave * nbx + rb;
    }
};

// State of a wave's R sub-blocks: the first np have no scaled pair, those from nm on no unscaled
// one; kept as np * 8 + nm with nm one of np, np + 1 and R, each of which has its own loop.
// Sub-blocks from np0 on are looked at: k their scale counts, v whether a lane has a value at all.
template <int R>
__device__ inline int sub_state(int np0, const int (&k)[R], const bool (&v)[R])
{
    int np = np0, nm = np0;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r >= np0) {
            if (np == r && !__any(k[r] > 0)) np = r + 1;
            if (__any(k[r] == 0 && v[r])) nm = r + 1;
        }
    if (nm < np) nm = np;
    return np * 8 + (nm > np + 1 ? R : nm);
}

// the rescale test at a chunk's end (powers of two: exact)
__device__ inline void rescale(double& vc, double& vp, int& k)
{
    const bool big = (k > 0) && fmax(fabs(vc), fabs(vp)) >= kBig;
    const double sc = big ? kUnit : 1.0;
    vp *= sc;
    vc *= sc;
    k -= big ? 1 : 0;
}

// Runs f(np, nm), the loop of state np * 8 + nm, for each state in ascending order if it is the
// current one: sub-blocks only ever come into range, so states only ever grow.
template <int R, int NP = 0, typename F>
__device__ inline void run_states(int& st, F&& f)
{
    using np = std::integral_constant<int, NP>;
    if (st == NP * 9) f(np(), np());
    if constexpr (NP + 1 < R)
        if (st == NP * 9 + 1) f(np(), std::integral_constant<int, NP + 1>());
    if constexpr (NP < R) {
        if (st == NP * 8 + R) f(np(), std::integral_constant<int, R>());
        run_states<R, NP + 1>(st, f);
    }
}

template <int MB, int R, bool FUSED, typename OutT>
__global__ __launch_bounds__(64 * sub_waves(MB)) void k_legendre_synth(
    const double2* __restrict__ alm, int64_t nalm, int lmax, int mmax,
    const double2* __restrict__ rec, const double* __restrict__ cm_mant,
    const int* __restrict__ cm_exp, const int* __restrict__ jlive, int nr, int nt,
    OutT* __restrict__ out, int64_t out_map_stride, int64_t out_row_stride)
{
    constexpr int LC = kSynLC;
    __shared__ float pf_sink[sub_waves(MB)][64];
    const int npairs = (nr + 1) / 2;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const SubGrid sg(npairs, R, sub_waves(MB));
    int m, pc;
    sg.place(blockIdx.x, wave, mmax, m, pc);
    if (m > mmax) return;
    const int jl = jlive[m];
    const int nsub = (npairs - jl + 63) >> 6, nwm = (nsub + R - 1) / R;
    alm += (int64_t)blockIdx.y * MB * nalm;
    out += (int64_t)blockIdx.y * MB * out_map_stride;
    const int64_t moff = (int64_t)m * (2 * lmax + 1 - m) / 2;  // index(l, m) = moff + l
    const double sgn = (m & 1) ? -1.0 : 1.0;
    // values of pair j: the rings j (n) and N_r - 1 - j (s) of map b
    auto put = [&](int b, int j, double nre, double nim, double sre, double sim) {
        const int js = nr - 1 - j;
        OutT* o = out + b * out_map_stride;
        if (FUSED) {
            OutT* col = o + (int64_t)m * out_row_stride;
            col[j] = make_out<OutT>(nre, nim);
            if (j >= 1 && j <= nr - 2) col[nt - j] = make_out<OutT>(sgn * nre, sgn * nim);
            if (js != j) {
                col[js] = make_out<OutT>(sre, sim);
                if (js >= 1 && js <= nr - 2) col[nt - js] = make_out<OutT>(sgn * sre, sgn * sim);
            }
        } else {
            o[(int64_t)j * out_row_stride + m] = make_out<OutT>(nre, nim);
            if (js != j) o[(int64_t)js * out_row_stride + m] = make_out<OutT>(sre, sim);
        }
    };
    // pairs below the live bound are zero
    for (int j = pc * 64 + lane; j < jl; j += sg.nbx * sg.wpb * 64)
#pragma unroll
        for (int b = 0; b < MB; ++b) put(b, j, 0.0, 0.0, 0.0, 0.0);
    if (pc >= nwm) return;

    // the recurrence starts one step early: the step (0, -1) into l = m gives lam_mm from
    // vp = lam_mm, vc = 0
    double E[R][MB][2], O[R][MB][2], y[R], vc[R], vp[R];
    int k[R];
    bool has[R];
    const double cm = cm_mant[m];
    const int ce = cm_exp[m];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int b = 0; b < MB; ++b) E[r][b][0] = E[r][b][1] = O[r][b][0] = O[r][b][1] = 0.0;
        const int sub = pc + r * nwm;
        const int jraw = npairs - 1 - 64 * sub - lane;
        const bool valid = jraw >= jl;
        double s;
        ring_geom(max(jraw, jl), nr, s, y[r]);
        vc[r] = 0.0;
        lambda_mm_scaled(cm, ce, s, m, vp[r], k[r]);
        if (!valid) {
            vp[r] = 0.0;
            k[r] = 0;
        }
        has[r] = vp[r] != 0.0;
    }
    int st = sub_state<R>(0, k, has);
    auto step = [&](int r, double2 c) {
        const double vn = rec_step(c, y[r], vc[r], vp[r]);
        vp[r] = vc[r];
        vc[r] = vn;
        return vn;
    };
    auto add = [&](double (&A)[MB][2], const double2 (&a)[MB], double v) {
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            A[b][0] = fma(a[b].x, v, A[b][0]);
            A[b][1] = fma(a[b].y, v, A[b][1]);
        }
    };
    // Coefficients through the constant address space: wave-uniform scalar loads.  Those of the next
    // PL values of l are fetched while the current ones are used: as many as fit the scalar
    // registers twice (a load takes several hundred cycles where no other wave has brought the line
    // into the scalar cache).
    using cptr = const __attribute__((address_space(4))) double*;
    cptr crec = (cptr)(rec + moff), calm = (cptr)(alm + moff);
    auto fetch = [&](auto& cn, auto& an, int l) {
        constexpr int PL = sizeof(cn) / sizeof(cn[0]);
#pragma unroll
        for (int i = 0; i < PL; ++i) {
            cn[i] = make_double2(crec[2 * (l + i)], crec[2 * (l + i) + 1]);
#pragma unroll
            for (int b = 0; b < MB; ++b)
                an[i][b] = make_double2(calm[2 * (b * nalm + l + i)], calm[2 * (b * nalm + l + i) + 1]);
        }
    };
    int l0 = m, pf_at = m, pf_off;
    unsigned pf_keep = 0;
    const double2* pf_line = touch_line<MB>(rec, alm, nalm, moff, lane, pf_off);
    const unsigned lds_sink = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)pf_sink[wave]);
    auto loop = [&](auto np, auto nm) {
        constexpr int NP = decltype(np)::value, NM = decltype(nm)::value;
        constexpr int PL = (NP == R ? 8 : 4) / (MB == 1 ? 2 : MB);
        double2 cn[PL], an[PL][MB];
        if (l0 + LC - 1 <= lmax) {
            fetch(cn, an, l0);
            if (l0 == m) cn[0] = make_double2(0.0, -1.0);
        }
        for (; l0 + LC - 1 <= lmax; l0 += LC) {
            if (l0 >= pf_at) {
                pf_keep ^= touch_coeffs(pf_line, pf_off, l0 + kPfStep, lmax, lds_sink);
                pf_at = l0 + kPfStep;
            }
            double f[R];
#pragma unroll
            for (int r = NP; r < NM; ++r) f[r] = k[r] == 0 ? 1.0 : 0.0;
#pragma unroll
            for (int h = 0; h < LC; h += PL) {
                double2 c[PL], a[PL][MB];
#pragma unroll
                for (int i = 0; i < PL; ++i) {
                    c[i] = cn[i];
#pragma unroll
                    for (int b = 0; b < MB; ++b) a[i][b] = an[i][b];
                }
                fetch(cn, an, min(l0 + h + PL, lmax + 1 - PL));
#pragma unroll
                for (int i = 0; i < PL; ++i)
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double v = step(r, c[i]);
                        if (r < NM) add((h + i) & 1 ? O[r] : E[r], a[i], r < NP ? v : v * f[r]);
                    }
            }
            if constexpr (NP < R) {
#pragma unroll
                for (int r = NP; r < R; ++r) {
                    rescale(vc[r], vp[r], k[r]);
                    has[r] = vc[r] != 0.0 || vp[r] != 0.0;
                }
                const int now = sub_state<R>(NP, k, has);
                if (now > NP * 8 + NM) {
                    st = now;
                    l0 += LC;
                    break;
                }
            }
        }
    };
    run_states<R>(st, loop);
    // the last l values, fewer than a chunk (l0 - m is even)
    for (int i = 0; l0 + i <= lmax; ++i) {
        const int l = l0 + i;
        const double2 c = l == m ? make_double2(0.0, -1.0) : make_double2(crec[2 * l], crec[2 * l + 1]);
        double2 a[MB];
#pragma unroll
        for (int b = 0; b < MB; ++b)
            a[b] = make_double2(calm[2 * (b * nalm + l)], calm[2 * (b * nalm + l) + 1]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double v = k[r] == 0 ? step(r, c) : (step(r, c), 0.0);
            add(i & 1 ? O[r] : E[r], a, v);
        }
    }
    // no LDS-DMA write may be in flight when the workgroup's LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(pf_keep) : "memory");

#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = npairs - 1 - 64 * (pc + r * nwm) - lane;
        if (j < jl) continue;
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            double nre = E[r][b][0] + O[r][b][0], nim = E[r][b][1] + O[r][b][1];
            double sre = E[r][b][0] - O[r][b][0], sim = E[r][b][1] - O[r][b][1];
            if (m == 0) nim = sim = 0.0;  // Im a_l0 is ignored
            put(b, j, nre, nim, sre, sim);
        }
    }
}

// ------------------------------------------------------------------------------------
// Adjoint.  c_lm = sum_j lam_lm(x_j) G'_m(theta_j) is, for one m, a product of the
// (L - m + 1) x N_r matrix of lam values (generated by the recurrence) with the N_r x
// (2 B) matrix of ring data, reduced over rings.  gfx950 mapping:
//  * one lane = one ring pair (j, N_r-1-j): lam_lm(-x) = (-1)^(l+m) lam_lm(x), so the pair
//    enters through its even (N + S) and odd (N - S) combinations, chosen by the parity of
//    l - m; the lane runs the recurrence for 16 consecutive l and parks the values in LDS;
//  * the reduction over ring pairs runs on v_mfma_f64_4x4x4_4b: four 4x4x4 products per
//    instruction, one for each (parity, real/imaginary) pair, with rows = the 4 maps,
//    K = 4 ring pairs and columns = 4 values of l of that parity -- every product term is
//    used (the 16x16x4 shape would spend half of its work on the wrong parity) and this
//    shape sustains close to the FP64 peak on gfx950, the 16x16 one about 60 % of it;
//  * the waves of a block (one pair-chunk) are summed without workgroup barriers: each wave
//    adds its D values of a round of kAdjGroup chunks into one of kAdjSlots LDS slots (LDS
//    FP64 atomics) and counts itself in; the last of the block's live waves to arrive adds
//    the slot into the output, clears it and hands it on to the round kAdjSlots later.  The
//    waves therefore run at their own pace (scaled and unscaled lanes, dead waves) instead of
//    meeting at two barriers after every round;
//  * the pair-chunks of one m run on one XCD and add their sums into the zeroed output with
//    FP64 atomics that resolve in that XCD's L2 (the order of the additions is not fixed:
//    results can differ between runs by FP64 rounding).
// Input: FUSED Tp[b][m][t] (t < N_t), folded here:
//   G'_m(j) = Tp(j) + [1 <= j <= N_r - 2] (-1)^m Tp(N_t - j)      (D^H of Eq. 6)
// PAPER G'[b][j][m] rows of length (N_phi/2 + 1) (output of the per-ring R2C).
// ------------------------------------------------------------------------------------
constexpr int kAdjWaves = 4;     // waves per block: one block reduces up to 256 ring pairs
constexpr int kLC = 16;          // l values per chunk = the MFMA N dimension
constexpr int kLS = kLC + 1;     // padded row of the lam staging area
constexpr int kAdjGroup = 2;     // chunks whose sums go through one slot together
constexpr int kAdjSlots = 2;     // slots in flight per block (power of two)
constexpr int kAdjPfAhead = 4;   // chunks between a coefficient line's L2 touch and its use
constexpr int kAdjSpinLimit = 1 << 22;  // sleeps before a slot wait gives up (never reached)


template <typename InT>
__device__ inline double2 load_c(const InT* p)
{
    InT v = *p;
    return make_double2((double)v.x, (double)v.y);
}

template <bool FUSED, typename InT, bool DET>
__global__ __launch_bounds__(kAdjWaves * 64, DET ? 3 : 4) void k_legendre_adj(
    const InT* __restrict__ in, int64_t in_map_stride, int64_t in_row_stride, int nmaps,
    double* __restrict__ alm, int npc, int64_t nalm, int lmax,
    const double2* __restrict__ rec, const double* __restrict__ cm_mant,
    const int* __restrict__ cm_exp, const int* __restrict__ jlive, int nr, int nt,
    int pairs_per_block, int mmax, int* __restrict__ err)
{
    // per wave: the lam values of one chunk (64 pairs x 16 l); per block: the chunk-sum slots
    // (128 D values: 64 lanes x real/imaginary), their arrival counts and hand-on counts
    __shared__ double stage[kAdjWaves][64 * kLS];
    __shared__ float pf_sink[kAdjWaves][64];
    // DET: one region per wave, summed in wave order by the flushing wave (fixed order)
    constexpr int kSlotWaves = DET ? kAdjWaves : 1;
    __shared__ double slot[kAdjSlots][kSlotWaves][kAdjGroup * 128];
    __shared__ unsigned scnt[kAdjSlots], sgen[kAdjSlots];
    static_assert((kAdjSlots & (kAdjSlots - 1)) == 0, "slot count a power of two");
    // all pair-chunks of one m on one XCD, one after the other: they share the m's
    // coefficient stream in that XCD's L2
    int m, pc;
    xcd_block(blockIdx.x, npc, m, pc);
    if (m > mmax) return;
    // DET: alm is the partial-sum array [npc][nmaps][nalm] (complex); this block's part
    if (DET) alm += (int64_t)pc * nmaps * nalm * 2;
    const int grp = blockIdx.y;
    const int nmb = min(4, nmaps - 4 * grp);
    // the wave index read through a scalar register: everything derived from it (dead waves,
    // the slot protocol) is then known to be wave-uniform
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nwaves = blockDim.x >> 6;
    const int npairs = (nr + 1) / 2;
    const int local = wave * 64 + lane;
    const int pair = pc * pairs_per_block + local;
    const bool valid = local < pairs_per_block && pair < npairs;
    const int j = valid ? pair : 0;
    const int js = nr - 1 - j;
    const int64_t moff = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const double msgn = (m & 1) ? -1.0 : 1.0;
    in += (int64_t)(4 * grp) * in_map_stride;
    double* st = stage[wave];
    const int jl = jlive[m];
    // pairs below jl never carry lam above 2^-300 for l <= lmax: a block made only of them
    // writes zero partial sums, a wave made only of them skips its recurrence and MFMAs
    if (pc * pairs_per_block + pairs_per_block <= jl) return;
    // a wave is dead when all its pairs lie below the live-ring bound or beyond the pairs
    const int wfirst = pc * pairs_per_block + wave * 64;
    const bool wave_dead = wfirst + 64 <= jl || wave * 64 >= pairs_per_block || wfirst >= npairs;

    // ring data of this lane's pair: rows 4 b + {N re, N im, S re, S im}.  All loads are
    // issued before any is used (indices clamped into range, unused ones weighted by 0).
    {
        double2 raw[4][4];
        double wgt[4];
        int64_t off[4];
        if (FUSED) {
            // G'(j) = Tp(j) + [1 <= j <= N_r - 2] (-1)^m Tp(N_t - j), likewise for js
            off[0] = j;
            off[1] = (j >= 1 && j <= nr - 2) ? nt - j : j;
            off[2] = js;
            off[3] = (js >= 1 && js <= nr - 2) ? nt - js : js;
            wgt[0] = 1.0;
            wgt[1] = (j >= 1 && j <= nr - 2) ? msgn : 0.0;
            wgt[2] = js != j ? 1.0 : 0.0;
            wgt[3] = (js != j && js >= 1 && js <= nr - 2) ? msgn : 0.0;
            for (int q = 0; q < 4; ++q) off[q] += (int64_t)m * in_row_stride;
        } else {
            off[0] = (int64_t)j * in_row_stride + m;
            off[2] = (int64_t)js * in_row_stride + m;
            off[1] = off[0];
            off[3] = off[2];
            wgt[0] = 1.0;
            wgt[1] = 0.0;
            wgt[2] = js != j ? 1.0 : 0.0;
            wgt[3] = 0.0;
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int bb = b < nmb ? b : 0;
            const InT* im = in + (int64_t)bb * in_map_stride;
#pragma unroll
            for (int q = 0; q < 4; ++q) raw[b][q] = load_c(im + off[q]);
        }
        // hv[(2 h + c) * 4 + map]: h = 0 the even combination N + S, h = 1 the odd one
        // N - S (lam_lm(-x) = (-1)^(l+m) lam_lm(x)); c = 0 real, 1 imaginary part
        double hv[16];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const double use = (valid && b < nmb) ? 1.0 : 0.0;
            const double nre = use * (wgt[0] * raw[b][0].x + wgt[1] * raw[b][1].x);
            const double nim = use * (wgt[0] * raw[b][0].y + wgt[1] * raw[b][1].y);
            const double sre = use * (wgt[2] * raw[b][2].x + wgt[3] * raw[b][3].x);
            const double sim = use * (wgt[2] * raw[b][2].y + wgt[3] * raw[b][3].y);
            hv[0 * 4 + b] = nre + sre;
            hv[1 * 4 + b] = nim + sim;
            hv[2 * 4 + b] = nre - sre;
            hv[3 * 4 + b] = nim - sim;
        }
#pragma unroll
        for (int c = 0; c < 16; ++c) st[lane * kLS + c] = hv[c];
    }
    for (int e = threadIdx.x; e < kAdjSlots * kSlotWaves * kAdjGroup * 128; e += blockDim.x)
        (&slot[0][0][0])[e] = 0.0;
    if (threadIdx.x < kAdjSlots) {
        scnt[threadIdx.x] = 0;
        sgen[threadIdx.x] = 0;
    }
    __syncthreads();
    // D of v_mfma_f64_4x4x4_4b (measured layout: A_b[i][k] in lane i + 4 b + 16 k,
    // B_b[k][j] in lane j + 4 b + 16 k, D_b[i][j] in lane j + 4 b + 16 i).  Here k = ring
    // pair of the group of four, block b = 2 s + h selects l = l0 + 8 s + 2 j + h of the
    // chunk (s: half-chunk, h: parity of l - l0), so that the four blocks of one B operand
    // hold 16 distinct lam values and every lam value is read from LDS once; i = map, and
    // the real and imaginary parts (c) are two MFMAs on the same B.
    const int kk = lane >> 4, bb = (lane >> 2) & 3, jj = lane & 3;
    const int lidx = 8 * (bb >> 1) + 2 * jj + (bb & 1);  // this lane's l - l0 in B
    // A operand of MFMA (q, c): ring data of pair 4 q + k, part c of the combination of
    // parity h, map i
    double aop[2][16];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 16; ++q)
            aop[c][q] = st[(4 * q + kk) * kLS + (2 * (bb & 1) + c) * 4 + jj];
    __syncthreads();

    double s, y;
    ring_geom(j, nr, s, y);
    double vc, vp = 0.0;
    int k;
    lambda_mm_scaled(cm_mant[m], cm_exp[m], s, m, vc, k);
    if (!valid) {
        vc = 0.0;
        k = 0;
    }
    bool scaled = k > 0;
    unsigned pf_keep = 0;
    const unsigned lds_sink = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)pf_sink[wave]);

    // the coefficient lines of chunks 1 .. kAdjPfAhead (later chunks are touched kAdjPfAhead
    // chunks ahead of their use inside the loop)
    if (!wave_dead && lane < 2 * kAdjPfAhead && m + kLC + 8 * lane <= lmax)
        pf_keep ^= lds_dma_touch(rec + moff + m + kLC + 8 * lane, lds_sink);
    const int nchunks = (lmax - m) / kLC + 1;
    // the table is read through the constant address space: it is never written while the
    // kernel runs, so its wave-uniform reads stay scalar loads next to the atomics below
    const __attribute__((address_space(4))) double* crec =
        (const __attribute__((address_space(4))) double*)rec;
    // the block's live waves take part in the chunk sums; the dead ones leave (they issued no
    // LDS-DMA touches)
    int nlive = 0;
    for (int w = 0; w < nwaves; ++w) {
        const int wf = pc * pairs_per_block + w * 64;
        nlive += (wf + 64 <= jl || w * 64 >= pairs_per_block || wf >= npairs) ? 0 : 1;
    }
    if (wave_dead) return;
    // Cross-wave sums: the wave adds its D values of round r (chunks kAdjGroup r ..) into slot
    // r % kAdjSlots and counts itself in; the wave that completes the count adds the slot into
    // the output, clears it and hands it on to round r + kAdjSlots.
    for (int c0 = 0; c0 < nchunks; c0 += kAdjGroup) {
        double dv[kAdjGroup][2];
#pragma unroll
        for (int g = 0; g < kAdjGroup; ++g) {
            double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
            const int l0 = m + (c0 + g) * kLC;
            if (c0 + g < nchunks) {
                // the chunk's recurrence coefficients in one batch of scalar loads (the table
                // is padded past its end), and the lines of the chunk kAdjPfAhead ahead
                // touched into L2
                double2 cc[kLC];
#pragma unroll
                for (int i = 0; i < kLC; ++i)
                    cc[i] = make_double2(crec[2 * (moff + l0 + i)], crec[2 * (moff + l0 + i) + 1]);
                if (lane < 3 && l0 + kAdjPfAhead * kLC <= lmax)
                    pf_keep ^= lds_dma_touch(rec + moff + l0 + kAdjPfAhead * kLC + 8 * lane,
                                             lds_sink);
                double lam[kLC];
                const bool full = l0 > m && l0 + kLC - 1 <= lmax;
                if (full && !__any(scaled)) {
                    // common case: a full chunk past lam_mm with no lane scaled
#pragma unroll
                    for (int i = 0; i < kLC; ++i) {
                        const double vn = rec_step(cc[i], y, vc, vp);
                        vp = vc;
                        vc = vn;
                        lam[i] = vc;
                    }
                } else if (full) {
                    // a full chunk with some lane still scaled: the rescale test once per
                    // pair of steps (a step grows a value by less than 2^7, far from the
                    // FP64 range above kBig); a pair's values count once its lane is in range
#pragma unroll
                    for (int i = 0; i < kLC; i += 2) {
                        const double v0 = rec_step(cc[i], y, vc, vp);
                        const double v1 = rec_step(cc[i + 1], y, v0, vc);
                        const bool big = (k > 0) && fmax(fabs(v0), fabs(v1)) >= kBig;
                        const double sc = big ? kUnit : 1.0;
                        vp = v0 * sc;
                        vc = v1 * sc;
                        k -= big ? 1 : 0;
                        lam[i] = (k == 0) ? vp : 0.0;
                        lam[i + 1] = (k == 0) ? vc : 0.0;
                    }
                    scaled = k > 0;
                } else {
                    // the first chunk (lam_mm) and a partial last one: per-step tests
                    const bool wscaled = __any(scaled);
#pragma unroll
                    for (int i = 0; i < kLC; ++i) {
                        const int l = l0 + i;
                        if (l > lmax) {
                            lam[i] = 0.0;
                            continue;
                        }
                        if (l > m) {
                            const double vn = rec_step(cc[i], y, vc, vp);
                            vp = vc;
                            vc = vn;
                            if (wscaled) {
                                const bool big = (k > 0) && (fabs(vc) >= kBig);
                                const double sc = big ? kUnit : 1.0;
                                vc *= sc;
                                vp *= sc;
                                k -= big ? 1 : 0;
                            }
                        }
                        lam[i] = (k == 0) ? vc : 0.0;
                    }
                    scaled = k > 0;
                }
                // a chunk after which every live lane still carries a scale factor has only
                // zero lam values (k never increases): it adds nothing
                if (!__all(scaled || !valid)) {
#pragma unroll
                    for (int i = 0; i < kLC; ++i) st[lane * kLS + i] = lam[i];
                    // the wave reads back only its own staging rows
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                    for (int q = 0; q < 16; q += 2) {
                        const double b0 = st[(4 * q + kk) * kLS + lidx];
                        const double b1 = st[(4 * (q + 1) + kk) * kLS + lidx];
                        acc0 = __builtin_amdgcn_mfma_f64_4x4x4f64(aop[0][q], b0, acc0, 0, 0, 0);
                        acc2 = __builtin_amdgcn_mfma_f64_4x4x4f64(aop[1][q], b0, acc2, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f64_4x4x4f64(aop[0][q + 1], b1, acc1, 0, 0,
                                                                  0);
                        acc3 = __builtin_amdgcn_mfma_f64_4x4x4f64(aop[1][q + 1], b1, acc3, 0, 0,
                                                                  0);
                    }
                    // the next chunk rewrites the staging rows: all lanes' reads come first
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            }
            dv[g][0] = acc0 + acc1;
            dv[g][1] = acc2 + acc3;
        }
        // this wave's share of the round into slot r % kAdjSlots, once the round kAdjSlots
        // earlier has been taken out of it.  A slot is handed on as soon as the slowest live
        // wave has added into it, so the slowest wave never waits here and every wait ends; the
        // bound only keeps a broken invariant from hanging the device, and a wave that reaches
        // it sets the error word (the host reports NUSHT_EDEVICE: the sums may be wrong).
        const int rnd = c0 / kAdjGroup;
        const int sl = rnd & (kAdjSlots - 1);
        const unsigned use = (unsigned)(rnd / kAdjSlots);
        bool ready = false;
        for (int it = 0; it < kAdjSpinLimit; ++it) {
            if (__hip_atomic_load(&sgen[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ==
                use) {
                ready = true;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (!ready && lane == 0)
            __hip_atomic_fetch_or(err, kErrAdjWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
        for (int g = 0; g < kAdjGroup; ++g) {
            if (DET) {
                slot[sl][DET ? wave : 0][g * 128 + lane] = dv[g][0];
                slot[sl][DET ? wave : 0][g * 128 + 64 + lane] = dv[g][1];
            } else {
                __hip_atomic_fetch_add(&slot[sl][0][g * 128 + lane], dv[g][0], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(&slot[sl][0][g * 128 + 64 + lane], dv[g][1],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        unsigned arrived = 0;
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(&scnt[sl], 1u, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
        arrived = __builtin_amdgcn_readfirstlane(arrived);
        if ((int)arrived == nlive - 1) {
            // last arrival: the slot holds the block's sums of this round
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            double v[kAdjGroup][2];
#pragma unroll
            for (int g = 0; g < kAdjGroup; ++g) {
                if (DET) {
                    // waves in order; a dead wave's region stays zero
                    v[g][0] = v[g][1] = 0.0;
                    for (int w = 0; w < nwaves; ++w) {
                        v[g][0] += slot[sl][DET ? w : 0][g * 128 + lane];
                        v[g][1] += slot[sl][DET ? w : 0][g * 128 + 64 + lane];
                    }
                } else {
                    v[g][0] = slot[sl][0][g * 128 + lane];
                    v[g][1] = slot[sl][0][g * 128 + 64 + lane];
                    slot[sl][0][g * 128 + lane] = 0.0;
                    slot[sl][0][g * 128 + 64 + lane] = 0.0;
                }
            }
            // the lane index re-read here (opaque to the compiler), so that the lane's output
            // offset is formed in this branch instead of being held in registers throughout
            unsigned ln;
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0"
                         : "=v"(ln));
            const int b = ln >> 4;                // map
            const int blk = (ln >> 2) & 3;        // 2 s + h
            const int dl = 8 * (blk >> 1) + 2 * (ln & 3) + (blk & 1);
#pragma unroll
            for (int g = 0; g < kAdjGroup; ++g) {
                const int l = m + (c0 + g) * kLC + dl;
                if (l <= lmax && b < nmb) {
                    // the lane's map offset in 32 bits (b nalm 2 < 2^32), the rest uniform
                    double* o = alm + ((int64_t)(4 * grp) * nalm + moff + m + (c0 + g) * kLC) * 2 +
                                (unsigned)(b * (unsigned)nalm * 2u + (unsigned)dl * 2u);
                    if (DET) {
                        // this pair-chunk's own partial sums (alm points at them), summed
                        // over the pair-chunks in order afterwards
                        o[0] = v[g][0];
                        o[1] = m > 0 ? v[g][1] : 0.0;
                    } else {
                        if (v[g][0] != 0.0) unsafeAtomicAdd(o, v[g][0]);
                        if (m > 0 && v[g][1] != 0.0) unsafeAtomicAdd(o + 1, v[g][1]);  // c_l0 real
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (lane == 0) {
                // the count is reset before the hand-on becomes visible: a wave that sees the
                // new hand-on count also sees the zero count (release store)
                scnt[sl] = 0;
                __hip_atomic_store(&sgen[sl], use + 1, __ATOMIC_RELEASE,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    // no LDS-DMA write may be in flight when the workgroup's LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(pf_keep) : "memory");
}

// ------------------------------------------------------------------------------------
// Adjoint of one map.  The 4x4x4 products above compute four maps whatever the batch, behind an
// LDS round trip of every lam value; for one map the products with the ring data cost less than that
// on the VALU.  So every lane sums lam times its data over its R ring pairs (two FMAs per pair and
// l) and only the sum over the wave's lanes is a matrix
// product: v_mfma_f64_4x4x4_4b with A_b[i][k] = [i = l mod 4] takes the lane values as they lie (B_b[k][j]
// in lane j + 4 b + 16 k) and adds those of the four lanes x, x + 16, x + 32, x + 48 into row i of D
// (lane x + 16 i), so four MFMAs of four consecutive l leave 16 partial sums of each in one
// register; these are summed within the rows of 16 lanes by DPP (wave_rows).  No LDS, no
// barriers, no waits between waves: a wave is on its own and adds its sums into the zeroed output
// with FP64 atomics (or writes them to its partial array, see part_stride).
//
// Work split, exponent range and loops as in the synthesis (a chunk is 8 values of l here too).
//
// Bound by the FP64 VALU: 5 R instructions per l and wave, and about 6 for the sums.  One map at
// lmax 1023 / 2047 / 4095: 0.13 / 0.60 / 3.75 ms against 0.20 / 1.13 / 7.2 ms of the kernel above.  (The
// same for two maps, 7 R instructions and four MFMAs per l, was slower than that kernel.)
// ------------------------------------------------------------------------------------

template <int R, bool FUSED, typename InT>
__global__ __launch_bounds__(64 * sub_waves(1)) void k_legendre_adj_one(
    const InT* __restrict__ in, int64_t in_row_stride, double* __restrict__ alm, int64_t part_stride,
    int lmax, int mmax,
    const double2* __restrict__ rec, const double* __restrict__ cm_mant,
    const int* __restrict__ cm_exp, const int* __restrict__ jlive, int nr, int nt)
{
    constexpr int LC = 8;  // l values between two flushes: 2 LC / 4 = 4 registers of sums
    __shared__ float pf_sink[sub_waves(1)][64];
    const int npairs = (nr + 1) / 2;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const SubGrid sg(npairs, R, sub_waves(1));
    int m, pc;
    sg.place(blockIdx.x, wave, mmax, m, pc);
    if (m > mmax) return;
    const int jl = jlive[m];
    const int nsub = (npairs - jl + 63) >> 6, nwm = (nsub + R - 1) / R;
    if (pc >= nwm) return;
    const int64_t moff = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const double msgn = (m & 1) ? -1.0 : 1.0;
    const double cm = cm_mant[m];
    const int ce = cm_exp[m];

    // per pair: data of the even and odd combinations (N + S, N - S) and the recurrence, which starts
    // one step early: the step (0, -1) into l = m gives lam_mm from vp = lam_mm, vc = 0
    double H[R][2][2], y[R], vc[R], vp[R];
    int k[R];
    bool has[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int sub = pc + r * nwm;
        const int jraw = npairs - 1 - 64 * sub - lane;
        const bool valid = jraw >= jl;
        const int j = max(jraw, jl), js = nr - 1 - j;
        double2 n, s2 = make_double2(0.0, 0.0);
        if (FUSED) {
            // folded: G'(j) = Tp(j) + [1 <= j <= N_r - 2] (-1)^m Tp(N_t - j), likewise for js
            const InT* col = in + (int64_t)m * in_row_stride;
            n = load_c(col + j);
            if (j >= 1 && j <= nr - 2) {
                const double2 w = load_c(col + (nt - j));
                n.x = fma(msgn, w.x, n.x);
                n.y = fma(msgn, w.y, n.y);
            }
            if (js != j) {
                s2 = load_c(col + js);
                if (js >= 1 && js <= nr - 2) {
                    const double2 w = load_c(col + (nt - js));
                    s2.x = fma(msgn, w.x, s2.x);
                    s2.y = fma(msgn, w.y, s2.y);
                }
            }
        } else {
            n = load_c(in + (int64_t)j * in_row_stride + m);
            if (js != j) s2 = load_c(in + (int64_t)js * in_row_stride + m);
        }
        H[r][0][0] = valid ? n.x + s2.x : 0.0;
        H[r][0][1] = valid ? n.y + s2.y : 0.0;
        H[r][1][0] = valid ? n.x - s2.x : 0.0;
        H[r][1][1] = valid ? n.y - s2.y : 0.0;
        double s;
        ring_geom(j, nr, s, y[r]);
        vc[r] = 0.0;
        lambda_mm_scaled(cm, ce, s, m, vp[r], k[r]);
        if (!valid) {
            vp[r] = 0.0;
            k[r] = 0;
        }
        has[r] = vp[r] != 0.0;
    }
    int st = sub_state<R>(0, k, has);
    // selector rows: sel[i] is 1 in the lanes of row i of the A operand
    double sel[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) sel[i] = (lane & 3) == i ? 1.0 : 0.0;
    const int x = lane & 15;
    // lane x < 4 of row i writes component x & 1 of l = chunk + i + 4 (x >> 1)
    const int out_l = (lane >> 4) + 4 * ((x >> 1) & 1);
    const bool out_lane = x < 4 && !(part_stride == 0 && m == 0 && (x & 1));
    double* out = alm + (int64_t)pc * part_stride + (moff + out_l) * 2 + (x & 1);
    const __attribute__((address_space(4))) double* crec =
        (const __attribute__((address_space(4))) double*)rec;
    unsigned pf_keep = 0;
    const unsigned lds_sink = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)pf_sink[wave]);
    int pf_at = m, pf_off;
    const double2* pf_line = touch_line<0>(rec, nullptr, 0, moff, lane, pf_off);

    // a chunk's coefficients are fetched while the chunk before runs; the table is padded past its
    // end, and steps past lmax run on whatever follows (finite coefficients; their sums are not
    // written)
    auto fetch = [&](double2 (&cn)[LC], int l0) {
#pragma unroll
        for (int i = 0; i < LC; ++i)
            cn[i] = make_double2(crec[2 * (moff + l0 + i)], crec[2 * (moff + l0 + i) + 1]);
    };
    int l0 = m;
    auto loop = [&](auto np, auto nm) {
        constexpr int NP = decltype(np)::value, NM = decltype(nm)::value;
        double2 cn[LC];
        fetch(cn, min(l0, lmax));
        if (l0 == m) cn[0] = make_double2(0.0, -1.0);
        for (; l0 <= lmax; l0 += LC) {
            if (l0 >= pf_at) {
                pf_keep ^= touch_coeffs(pf_line, pf_off, l0 + kPfStep, lmax, lds_sink);
                pf_at = l0 + kPfStep;
            }
            double2 cc[LC];
#pragma unroll
            for (int i = 0; i < LC; ++i) cc[i] = cn[i];
            fetch(cn, min(l0 + LC, lmax));
            double t[LC][2], f[R];
#pragma unroll
            for (int r = NP; r < NM; ++r) f[r] = k[r] == 0 ? 1.0 : 0.0;
#pragma unroll
            for (int i = 0; i < LC; ++i) {
                t[i][0] = t[i][1] = 0.0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double vn = rec_step(cc[i], y[r], vc[r], vp[r]);
                    vp[r] = vc[r];
                    vc[r] = vn;
                    if (r >= NM) continue;
                    const double v = r < NP ? vn : vn * f[r];
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        t[i][e] = r == 0 ? v * H[0][i & 1][e] : fma(v, H[r][i & 1][e], t[i][e]);
                }
            }
            if (NM > 0 || part_stride != 0) {
                double q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int i = 0; i < LC; ++i)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        double& d = q[2 * (i >> 2) + e];
                        d = __builtin_amdgcn_mfma_f64_4x4x4f64(sel[i & 3], t[i][e], d, 0, 0, 0);
                    }
                const double v = wave_rows(q, x);
                if (out_lane && l0 + out_l <= lmax) {
                    double* o = out + 2 * (int64_t)l0;
                    if (part_stride != 0)
                        *o = (m == 0 && (x & 1)) ? 0.0 : v;
                    else if (v != 0.0)
                        unsafeAtomicAdd(o, v);
                }
            }
            if constexpr (NP < R) {
#pragma unroll
                for (int r = NP; r < R; ++r) {
                    rescale(vc[r], vp[r], k[r]);
                    has[r] = vc[r] != 0.0 || vp[r] != 0.0;
                }
                const int now = sub_state<R>(NP, k, has);
                if (now > NP * 8 + NM) {
                    st = now;
                    l0 += LC;
                    break;
                }
            }
        }
    };
    run_states<R>(st, loop);
    // no LDS-DMA write may be in flight when the workgroup's LDS is released
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(pf_keep) : "memory");
}

__global__ void k_fill_zero(double* __restrict__ a, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0.0;
}

// Deterministic adjoint: alm[b][i] = sum over the pair-chunks pc of part[pc][b][i], in pc order.
// Pair-chunks that wrote nothing for the element's m are skipped: those whose ring pairs all lie
// below the live-ring bound jlive[m], or past the last pair (packed: chunk 0 starts at jlive[m]).
__global__ void k_adj_reduce(const double2* __restrict__ part, int npc, int nmaps, int64_t nalm,
                             int lmax, int mmax, const int* __restrict__ jlive, int ppb,
                             int npairs, int packed, double2* __restrict__ alm)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nalm) return;
    // m of index i: the largest m <= mmax whose first index first(m) = idx(m, m) =
    // m (2 lmax + 3 - m) / 2 is <= i.  first() grows with m up to lmax, and the discriminant
    // (2 lmax + 3)^2 - 8 i stays positive over the triangle; the estimate is corrected by
    // steps that cannot leave [0, mmax].
    const double bq = 2.0 * lmax + 3.0;
    const double disc = fmax(bq * bq - 8.0 * (double)i, 0.0);
    int m = (int)fmin(fmax(floor(0.5 * (bq - sqrt(disc))), 0.0), (double)mmax);
    while (m > 0 && (int64_t)m * (2 * lmax + 3 - m) / 2 > i) --m;
    while (m < mmax && (int64_t)(m + 1) * (2 * lmax + 2 - m) / 2 <= i) ++m;
    const int pc0 = packed ? 0 : jlive[m] / ppb;
    const int left = packed ? npairs - jlive[m] : npairs;
    for (int b = 0; b < nmaps; ++b) {
        double2 acc = make_double2(0.0, 0.0);
        for (int pc = pc0; pc < npc && pc * ppb < left; ++pc) {
            const double2 v = part[((int64_t)pc * nmaps + b) * nalm + i];
            acc.x += v.x;
            acc.y += v.y;
        }
        alm[(int64_t)b * nalm + i] = acc;
    }
}

}  // namespace

namespace {

// Two sub-blocks per wave share its coefficient loads and loop, one makes twice the waves and leaves
// the scalar registers to longer fetches.  R = 1 / 2 in us: four maps at 65 pairs (lmax 127) 18 / 25, at
// 129 34 / 36, at 257 80 / 67, at 2049 7485 / 6401; one map at 257 31 / 36, at 513 84 / 85, at 1025
// 470 / 432, at 2049 2950 / 2573; two maps at 513 108 / 128, at 1025 555 / 599, at 2049 3875 / 3934.
// (Four maps in blocks of eight waves.  More than two per wave: spilled scalar registers.)
int synth_pairs_per_lane(int npairs, int mb)
{
    if (mb == 2) return 1;
    return npairs <= (mb == 4 ? 160 : 640) ? 1 : 2;
}

template <int MB, int R, bool FUSED, typename OutT>
int launch_synth(const nusht_plan_s* p, const double2* alm, OutT* out, int groups,
                 int64_t map_stride, int64_t row_stride, hipStream_t s)
{
    const nusht_geometry& g = p->g;
    const int npairs = (g.nrings + 1) / 2;
    const SubGrid sg(npairs, R, sub_waves(MB));
    const int mpad = (g.mmax + 1 + 7) / 8 * 8;
    hipLaunchKernelGGL((k_legendre_synth<MB, R, FUSED, OutT>), dim3(sg.extra + sg.nbx * mpad, groups),
                       dim3(64 * sg.wpb), 0, s, alm, g.nalm, g.lmax, g.mmax, p->rec, p->cm_mant,
                       p->cm_exp, p->jlive, g.nrings, g.ntorus, out, map_stride, row_stride);
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

template <int MB, bool FUSED, typename OutT>
int launch_synth_r(const nusht_plan_s* p, const double2* alm, OutT* out, int groups,
                   int64_t map_stride, int64_t row_stride, hipStream_t s)
{
    if constexpr (MB != 2)
        if (synth_pairs_per_lane((p->g.nrings + 1) / 2, MB) == 2)
            return launch_synth<MB, 2, FUSED, OutT>(p, alm, out, groups, map_stride, row_stride, s);
    return launch_synth<MB, 1, FUSED, OutT>(p, alm, out, groups, map_stride, row_stride, s);
}

template <bool FUSED, typename OutT>
int launch_synth_maps(const nusht_plan_s* p, const double2* alm, OutT* out, int nmaps,
                      int64_t map_stride, int64_t row_stride, hipStream_t s)
{
    // groups of four maps, then of two, then one
    for (int b = 0; b < nmaps;) {
        const int left = nmaps - b, mb = left >= 4 ? 4 : (left >= 2 ? 2 : 1), groups = left / mb;
        const double2* a = alm + (int64_t)b * p->g.nalm;
        OutT* o = out + (int64_t)b * map_stride;
        if (mb == 4)
            NUSHT_TRY((launch_synth_r<4, FUSED, OutT>(p, a, o, groups, map_stride, row_stride, s)));
        else if (mb == 2)
            NUSHT_TRY((launch_synth_r<2, FUSED, OutT>(p, a, o, groups, map_stride, row_stride, s)));
        else
            NUSHT_TRY((launch_synth_r<1, FUSED, OutT>(p, a, o, groups, map_stride, row_stride, s)));
        b += groups * mb;
    }
    return NUSHT_OK;
}

}  // namespace

int launch_legendre_synth(const nusht_plan_s* p, const double* alm, void* out, int nmaps,
                          int fused, int out_f32, hipStream_t s)
{
    const nusht_geometry& g = p->g;
    const double2* a = reinterpret_cast<const double2*>(alm);
    if (fused) {
        const int64_t row = g.ntorus, map = (int64_t)(g.mmax + 1) * g.ntorus;
        if (out_f32)
            return launch_synth_maps<true>(p, a, reinterpret_cast<float2*>(out), nmaps, map, row, s);
        return launch_synth_maps<true>(p, a, reinterpret_cast<double2*>(out), nmaps, map, row, s);
    }
    const int64_t row = g.nphi / 2 + 1, map = (int64_t)g.nrings * row;
    return launch_synth_maps<false>(p, a, reinterpret_cast<double2*>(out), nmaps, map, row, s);
}

namespace {

// Ring pairs per lane of the one-map adjoint: more of them share a wave's sums and coefficient
// loads, fewer make more waves.  R = 1 / 2 / 4 / 6 in us: at 257 pairs (lmax 511) 39 / 47 / 54 / 68, at 513
// 169 / 132 / 140 / 174, at 769 478 / 396 / 324 / 305, at 1025 952 / 726 / 598 / 595, at 2049 6432 / 4737 /
// 3748 / 3997.
int one_map_pairs_per_lane(int npairs) { return npairs <= 320 ? 1 : npairs <= 640 ? 2 : 4; }

// room for the partial sums of deterministic plans
int ensure_partials(nusht_plan_s* p, size_t need, hipStream_t s)
{
    if (need <= p->adj_part_bytes) return NUSHT_OK;
    NUSHT_HIP(hipStreamSynchronize(s));
    if (p->adj_part) hipFree(p->adj_part);
    p->adj_part = nullptr;
    p->adj_part_bytes = 0;
    NUSHT_HIP(hipMalloc((void**)&p->adj_part, need));
    p->adj_part_bytes = need;
    return NUSHT_OK;
}

// the adjoint of one map into alm (zeroed, or, deterministic, written)
template <bool FUSED, typename InT>
int launch_adj_one(nusht_plan_s* p, const void* in, double* alm, int64_t row_stride,
                   hipStream_t s)
{
    const nusht_geometry& g = p->g;
    const int npairs = (g.nrings + 1) / 2;
    const int R = one_map_pairs_per_lane(npairs);
    const int nw = (npairs + 64 * R - 1) / (64 * R);  // most waves of one m
    const SubGrid sg(npairs, R, sub_waves(1));
    const int mpad = (g.mmax + 1 + 7) / 8 * 8;
    double* target = alm;
    int64_t part_stride = 0;
    if (p->deterministic) {
        part_stride = g.nalm * 2;
        NUSHT_TRY(ensure_partials(p, (size_t)nw * part_stride * sizeof(double), s));
        target = p->adj_part;
    }
#define ONE(RV)                                                                                  \
    hipLaunchKernelGGL((k_legendre_adj_one<RV, FUSED, InT>), dim3(sg.extra + sg.nbx * mpad),         \
                       dim3(64 * sg.wpb), 0, s, reinterpret_cast<const InT*>(in), row_stride,     \
                       target, part_stride, g.lmax, g.mmax, p->rec, p->cm_mant, p->cm_exp, p->jlive, g.nrings,        \
                       g.ntorus)
    if (R == 1)
        ONE(1);
    else if (R == 2)
        ONE(2);
    else
        ONE(4);
#undef ONE
    NUSHT_HIP(hipGetLastError());
    if (p->deterministic) {
        hipLaunchKernelGGL(k_adj_reduce, dim3((unsigned)((g.nalm + 255) / 256)), dim3(256), 0, s,
                           reinterpret_cast<const double2*>(target), nw, 1, g.nalm, g.lmax, g.mmax,
                           p->jlive, 64 * R, npairs, 1, reinterpret_cast<double2*>(alm));
        NUSHT_HIP(hipGetLastError());
    }
    return NUSHT_OK;
}

}  // namespace

int launch_legendre_adjoint(nusht_plan_s* p, const void* in, double* alm, int nmaps,
                            int fused, int in_f32, hipStream_t s)
{
    const nusht_geometry& g = p->g;
    int64_t map_stride, row_stride;
    if (fused) {
        row_stride = g.ntorus;
        map_stride = (int64_t)(g.mmax + 1) * g.ntorus;
    } else {
        row_stride = g.nphi / 2 + 1;
        map_stride = (int64_t)g.nrings * row_stride;
    }
    if (!p->deterministic) {
        // the workgroups of one m add their sums into the zeroed output with FP64 atomics, which
        // resolve in the L2 of the XCD those workgroups share
        const int64_t nz = (int64_t)nmaps * g.nalm * 2;
        hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, s, alm,
                           nz);
    }
    const int npairs = (g.nrings + 1) / 2;
    // one map left over after the groups of four has its own kernel; two or three fill a group of
    // the other well enough.  Up to 256 pairs the other kernel has one block per m and leaves the chip
    // idle: a group more costs it less than the launch (five maps at lmax 200 / 400: 25 / 50 us
    // against 37 / 65), so only a lone map goes to its own kernel there (23 -> 19 us).  In a
    // deterministic plan a map's bits do not depend on its batch: no map does.
    const bool own = nmaps % 4 == 1 && (npairs > kAdjWaves * 64 || (nmaps == 1 && !p->deterministic));
    const int one = own ? 1 : 0, many = nmaps - one;
    if (one) {
        const int64_t esz = in_f32 ? sizeof(float2) : sizeof(double2);
        const char* lin = reinterpret_cast<const char*>(in) + many * map_stride * esz;
        double* lout = alm + many * g.nalm * 2;
        if (fused && in_f32)
            NUSHT_TRY((launch_adj_one<true, float2>(p, lin, lout, row_stride, s)));
        else if (fused)
            NUSHT_TRY((launch_adj_one<true, double2>(p, lin, lout, row_stride, s)));
        else
            NUSHT_TRY((launch_adj_one<false, double2>(p, lin, lout, row_stride, s)));
    }
    if (!many) return NUSHT_OK;
    const int npc = (npairs + kAdjWaves * 64 - 1) / (kAdjWaves * 64);
    int ppb = (npairs + npc - 1) / npc;
    ppb = ((ppb + 63) / 64) * 64;
    const int threads = ppb < 128 ? 128 : ppb;
    const int groups = (many + 3) / 4;
    const int mpad = (g.mmax + 1 + 7) / 8 * 8;
    dim3 grid(npc * mpad, groups);
#define ADJ(F, IT, D, OUT)                                                                      \
    hipLaunchKernelGGL((k_legendre_adj<F, IT, D>), grid, dim3(threads), 0, s,                    \
                       reinterpret_cast<const IT*>(in), map_stride, row_stride, many, OUT, npc,   \
                       g.nalm, g.lmax, p->rec, p->cm_mant, p->cm_exp, p->jlive, g.nrings,        \
                       g.ntorus, ppb, g.mmax, p->dstatus)
    if (p->deterministic) {
        // every pair-chunk writes its own partial sums; one pass adds them in pair-chunk order
        NUSHT_TRY(ensure_partials(p, (size_t)npc * many * g.nalm * 2 * sizeof(double), s));
        double* part = p->adj_part;
        if (fused && in_f32) {
            ADJ(true, float2, true, part);
        } else if (fused) {
            ADJ(true, double2, true, part);
        } else {
            ADJ(false, double2, true, part);
        }
        NUSHT_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_adj_reduce, dim3((unsigned)((g.nalm + 255) / 256)), dim3(256), 0, s,
                           reinterpret_cast<const double2*>(part), npc, many, g.nalm, g.lmax,
                           g.mmax, p->jlive, ppb, npairs, 0, reinterpret_cast<double2*>(alm));
    } else {
        if (fused && in_f32) {
            ADJ(true, float2, false, alm);
        } else if (fused) {
            ADJ(true, double2, false, alm);
        } else {
            ADJ(false, double2, false, alm);
        }
    }
#undef ADJ
    NUSHT_HIP(hipGetLastError());
    return NUSHT_OK;
}

}  // namespace nusht
