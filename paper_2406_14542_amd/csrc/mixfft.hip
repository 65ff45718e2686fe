// Which lengths the general transforms (mixfft_impl.h) take, and their radices.
#include "fft_core.h"
#include "internal.h"

namespace nusht {

int mix_row_f32(const nusht_plan_s* p, const MixLen& m, const void* in, void* out, int64_t rw,
                int nb, bool c2r, hipStream_t s);
int mix_theta_f32(const nusht_plan_s* p, const MixLen& mt, const MixLen& mn, const void* in, void* out,
                  int nmaps, bool inv, hipStream_t s);
int mix_row_f64(const nusht_plan_s* p, const MixLen& m, const void* in, void* out, int64_t rw,
                int nb, bool c2r, hipStream_t s);
int mix_theta_f64(const nusht_plan_s* p, const MixLen& mt, const MixLen& mn, const void* in, void* out,
                  int nmaps, bool inv, hipStream_t s);

namespace {

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

bool fits(const nusht_geometry& g, int n)
{
    return g.dtype == NUSHT_MIXED ? lds_fits<float>(n) : lds_fits<double>(n);
}

}  // namespace

// Both are decided on the geometry alone: every length of the geometry is 7-smooth, so the limit
// is the LDS of one workgroup (N <= 9035 FP64, 18070 FP32: lmax about 2200 and 4500 at sigma 2).
// Longer ones stay with rocFFT: no kernel here holds them.
bool mixrow_supported(const nusht_geometry& g)
{
    MixLen m;
    return g.n2 % 2 == 0 && fits(g, g.n2 / 2) && g.mmax + 1 <= g.n2 / 2 && mix_len(g.n2 / 2, &m);
}

bool mixtheta_supported(const nusht_geometry& g)
{
    MixLen m;
    return g.dfs_mode == NUSHT_DFS_FUSED && fits(g, g.n1) && g.ntorus <= g.n1 &&
           mix_len(g.n1, &m) && mix_len(g.ntorus, &m);
}

int launch_mix_row(const nusht_plan_s* p, const void* in, void* out, int64_t rw, int nb,
                   bool c2r, hipStream_t s)
{
    MixLen m;
    if (!mix_len(p->g.n2 / 2, &m)) return NUSHT_EINVAL;
    return p->g.dtype == NUSHT_MIXED ? mix_row_f32(p, m, in, out, rw, nb, c2r, s)
                                     : mix_row_f64(p, m, in, out, rw, nb, c2r, s);
}

int launch_mix_theta(const nusht_plan_s* p, const void* in, void* out, int nmaps, bool inv,
                     hipStream_t s)
{
    MixLen mt, mn;
    if (!mix_len(p->g.ntorus, &mt) || !mix_len(p->g.n1, &mn)) return NUSHT_EINVAL;
    return p->g.dtype == NUSHT_MIXED ? mix_theta_f32(p, mt, mn, in, out, nmaps, inv, s)
                                     : mix_theta_f64(p, mt, mn, in, out, nmaps, inv, s);
}

}  // namespace nusht
