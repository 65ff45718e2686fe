// Row and column transforms of general lengths in FP32.
#include "mixfft_impl.h"

namespace nusht {

int mix_row_f32(const nusht_plan_s* p, const MixLen& m, const void* in, void* out, int64_t rw,
                int nb, bool c2r, hipStream_t s)
{
    return mix_row<float>(p, m, in, out, rw, nb, c2r, s);
}

int mix_theta_f32(const nusht_plan_s* p, const MixLen& mt, const MixLen& mn, const void* in, void* out,
                  int nmaps, bool inv, hipStream_t s)
{
    return mix_theta<float>(p, mt, mn, in, out, nmaps, inv, s);
}

}  // namespace nusht
