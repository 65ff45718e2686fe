// Small DFTs and helpers shared by the row and column transforms (rowfft.hip, mixfft.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace nusht {
namespace {

template <typename T>
struct Cx;
template <>
struct Cx<float> {
    using type = float2;
};
template <>
struct Cx<double> {
    using type = double2;
};

template <typename C>
__device__ inline C cmk(decltype(C::x) re, decltype(C::x) im)
{
    C r;
    r.x = re;
    r.y = im;
    return r;
}
template <typename C>
__device__ inline C cadd(C a, C b)
{
    return cmk<C>(a.x + b.x, a.y + b.y);
}
template <typename C>
__device__ inline C csub(C a, C b)
{
    return cmk<C>(a.x - b.x, a.y - b.y);
}
template <typename C>
__device__ inline C cmul(C a, C b)
{
    return cmk<C>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * (DIR i)
template <int DIR, typename C>
__device__ inline C cmul_i(C a)
{
    return DIR > 0 ? cmk<C>(-a.y, a.x) : cmk<C>(a.y, -a.x);
}

// cos and sin of 2 pi e / 16
__device__ constexpr double kCos16[16] = {
    1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
    0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
    -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173,
    0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613};
__device__ constexpr double kSin16[16] = {
    0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613,
    1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
    0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
    -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173};

// a * e^{DIR 2 pi i e / 16}; e is a constant once the callers' loops are unrolled, so the
// branches and the table lookups fold away
template <int DIR, typename C>
__device__ __forceinline__ C rot16(C a, int e)
{
    using T = decltype(C::x);
    e &= 15;
    if (e == 0) return a;
    if (e == 4) return cmul_i<DIR>(a);
    if (e == 8) return cmk<C>(-a.x, -a.y);
    if (e == 12) return cmul_i<-DIR>(a);
    return cmul(a, cmk<C>((T)kCos16[e], (T)(DIR * kSin16[e])));
}

// in-place DFT of R = 1 .. 10, 12 or 16 values, natural order in and out:
// V[k] = sum_n v[n] e^{DIR 2 pi i n k / R}
template <int R, int DIR, typename C>
__device__ inline void dft(C (&v)[R])
{
    if constexpr (R == 2) {
        const C a = v[0];
        v[0] = cadd(a, v[1]);
        v[1] = csub(a, v[1]);
    } else if constexpr (R == 4) {
        const C a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
        const C a2 = cadd(v[1], v[3]), a3 = cmul_i<DIR>(csub(v[1], v[3]));
        v[0] = cadd(a0, a2);
        v[2] = csub(a0, a2);
        v[1] = cadd(a1, a3);
        v[3] = csub(a1, a3);
    } else if constexpr (R == 5) {
        // V[k] = sum_n v[n] w^(n k), w = e^{DIR 2 pi i / 5}: pairs (1, 4) and (2, 3) share
        // cos(2 pi / 5), cos(4 pi / 5) and sin(2 pi / 5), sin(4 pi / 5)
        using T = decltype(C::x);
        const T c1 = (T)0.30901699437494742410, c2 = (T)-0.80901699437494742410;
        const T s1 = (T)0.95105651629515357212, s2 = (T)0.58778525229247312917;
        const C t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]);
        const C t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
        const C a1 = cmk<C>(v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y);
        const C a2 = cmk<C>(v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y);
        const C b1 = cmul_i<DIR>(cmk<C>(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y));
        const C b2 = cmul_i<DIR>(cmk<C>(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y));
        v[0] = cadd(v[0], cadd(t1, t2));
        v[1] = cadd(a1, b1);
        v[4] = csub(a1, b1);
        v[2] = cadd(a2, b2);
        v[3] = csub(a2, b2);
    } else if constexpr (R == 3) {
        using T = decltype(C::x);
        const T s1 = (T)0.866025403784438646764;
        const C t1 = cadd(v[1], v[2]), t2 = csub(v[1], v[2]);
        const C a1 = cmk<C>(v[0].x - (T)0.5 * t1.x, v[0].y - (T)0.5 * t1.y);
        const C b1 = cmul_i<DIR>(cmk<C>(s1 * t2.x, s1 * t2.y));
        v[0] = cadd(v[0], t1);
        v[1] = cadd(a1, b1);
        v[2] = csub(a1, b1);
    } else if constexpr (R == 7) {
        // as for 5: pairs (n, 7 - n) share cos and sin of 2 pi n k / 7
        using T = decltype(C::x);
        const T c[4] = {(T)1, (T)0.623489801858733530525, (T)-0.222520933956314404289, (T)-0.900968867902419126236};
        const T s[4] = {(T)0, (T)0.781831482468029808708, (T)0.974927912181823607018, (T)0.433883739117558120476};
        C p[4], m[4];
#pragma unroll
        for (int n = 1; n < 4; ++n) {
            p[n] = cadd(v[n], v[7 - n]);
            m[n] = csub(v[n], v[7 - n]);
        }
        const C x0 = v[0];
        v[0] = cadd(x0, cadd(p[1], cadd(p[2], p[3])));
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            C a = x0, b = cmk<C>(0, 0);
#pragma unroll
            for (int n = 1; n < 4; ++n) {
                const int e = (n * k) % 7, f = e < 4 ? e : 7 - e;
                const T sn = e < 4 ? s[f] : -s[f];
                a = cmk<C>(a.x + c[f] * p[n].x, a.y + c[f] * p[n].y);
                b = cmk<C>(b.x + sn * m[n].x, b.y + sn * m[n].y);
            }
            b = cmul_i<DIR>(b);
            v[k] = cadd(a, b);
            v[7 - k] = csub(a, b);
        }
    } else if constexpr (R == 9) {
        // n = 3 n1 + n2, k = k1 + 3 k2, twiddles e^{DIR 2 pi i n2 k1 / 9}
        using T = decltype(C::x);
        const C w1 = cmk<C>((T)0.766044443118978035202, (T)(DIR * 0.642787609686539326323));
        const C w2 = cmk<C>((T)0.173648177666930348852, (T)(DIR * 0.984807753012208059367));
        const C w4 = cmk<C>((T)-0.939692620785908384054, (T)(DIR * 0.342020143325668733044));
        C u[3][3];
#pragma unroll
        for (int n2 = 0; n2 < 3; ++n2) {
            C w[3] = {v[n2], v[3 + n2], v[6 + n2]};
            dft<3, DIR>(w);
            u[0][n2] = w[0];
            u[1][n2] = n2 == 0 ? w[1] : cmul(w[1], n2 == 1 ? w1 : w2);
            u[2][n2] = n2 == 0 ? w[2] : cmul(w[2], n2 == 1 ? w2 : w4);
        }
#pragma unroll
        for (int k1 = 0; k1 < 3; ++k1) {
            dft<3, DIR>(u[k1]);
#pragma unroll
            for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = u[k1][k2];
        }
    } else if constexpr (R == 6 || R == 10 || R == 12) {
        // R = A B with coprime factors: n = B n1 + A n2, k = B (1/B mod A) k1 + A (1/A mod B) k2
        // (both mod R) leaves no twiddles between the two small transforms
        constexpr int A = R == 12 ? 4 : 2, B = R / A;
        constexpr int EB = B % A == 1 ? B : 3 * B;  // B (1/B mod A): 3 is its own inverse mod 4
        constexpr int EA = B == 3 ? 4 : 6;  // A (1/A mod B): 2 * 2, 4 * 1, 2 * 3
        C u[A][B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) {
            C w[A];
#pragma unroll
            for (int n1 = 0; n1 < A; ++n1) w[n1] = v[(B * n1 + A * n2) % R];
            dft<A, DIR>(w);
#pragma unroll
            for (int k1 = 0; k1 < A; ++k1) u[k1][n2] = w[k1];
        }
#pragma unroll
        for (int k1 = 0; k1 < A; ++k1) {
            dft<B, DIR>(u[k1]);
#pragma unroll
            for (int k2 = 0; k2 < B; ++k2) v[(EB * k1 + EA * k2) % R] = u[k1][k2];
        }
    } else if constexpr (R == 8 || R == 16) {
        // R = 4 Q: n = Q n1 + n2, k = k1 + 4 k2; DFT_4 over n1, twiddle e^{DIR 2 pi i n2 k1 / R},
        // DFT_Q over n2
        constexpr int Q = R / 4;
        C u[4][Q];
#pragma unroll
        for (int n2 = 0; n2 < Q; ++n2) {
            C w[4] = {v[n2], v[Q + n2], v[2 * Q + n2], v[3 * Q + n2]};
            dft<4, DIR>(w);
#pragma unroll
            for (int k1 = 0; k1 < 4; ++k1) u[k1][n2] = rot16<DIR>(w[k1], n2 * k1 * (16 / R));
        }
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            dft<Q, DIR>(u[k1]);
#pragma unroll
            for (int k2 = 0; k2 < Q; ++k2) v[k1 + 4 * k2] = u[k1][k2];
        }
    }
}

// LDS index with one pad slot per 16 entries (stride-16 accesses stay off one bank)
__device__ inline int pad16(int i) { return i + (i >> 4); }

// tw[k] read through the constant address space: for a wave-uniform k this is a scalar load
template <typename T>
__device__ inline typename Cx<T>::type tw_uniform(const typename Cx<T>::type* tw, int k)
{
    const __attribute__((address_space(4))) T* p = (const __attribute__((address_space(4))) T*)tw;
    return cmk<typename Cx<T>::type>(p[2 * k], p[2 * k + 1]);
}

__device__ inline int kappa_of(int i, int n) { return i <= n / 2 ? i : i - n; }

// one transform of N complex values held in LDS (with the pad slots)
template <typename T>
constexpr bool lds_fits(int N)
{
    return (size_t)(N + N / 16) * 2 * sizeof(T) <= 150 * 1024;
}

}  // namespace
}  // namespace nusht
