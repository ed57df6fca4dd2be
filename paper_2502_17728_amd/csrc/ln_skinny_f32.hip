// ln_skinny_f32.hip -- LayerNorm/RMSNorm products on packed fp32 weights, every size.
#include "ln_skinny.hpp"

namespace dn {

template <int NC, Skinny KIND>
static hipError_t skinny_rf(int rf, const SkinnyArgs& a, hipStream_t s) {
    switch (rf) {
        case 1: return run_skinny_kernel<float, 1, 8, NC, KIND>(a, s);
        case 2: return run_skinny_kernel<float, 2, 4, NC, KIND>(a, s);
        case 4: return run_skinny_kernel<float, 4, 2, NC, KIND>(a, s);
        default: return run_skinny_kernel<float, 8, 1, NC, KIND>(a, s);
    }
}
// The plan by estimated time, as for bf16 (ln_skinny.hip) with fp32's stages: 0.06 rf nc us of
// matrix work per 64 k and 0.14 + 0.035 rf us besides.  Measured (graph replays, us; before:
// 32 x 64 tiles of a two- to four-stage loop whose x copies were half lines): 128 rows
// 768 -> 3072 12.6 / 15.3, 1 row 4096 -> 6144 22 / 54, 1 row 4992 -> 1104 16 / 64, 477 rows
// 4096 -> 12288 410 / 632 (117 TFLOP/s), 1000 rows 768 -> 3072 46 / 78.
static void plan_f32(int64_t M, int64_t K, int64_t nblocks, bool gated, int* rf_out, int* nc_out) {
    static constexpr int kRf[4] = {1, 2, 4, 8};
    double best = 0;
    for (int rf : kRf)
        for (int nc = gated ? 2 : 1; nc <= 6; nc += gated ? 2 : 1) {
            if (nc == 5 || (rf == 1 && nc == 6)) continue;  // one row block x 6 columns: 2-deep rings only
            const int64_t nrb = (M + 16 * rf - 1) / (16 * rf), wgs = nrb * ((nblocks + nc - 1) / nc);
            const double w_us = (double)nblocks * 64.0 * (double)K / 6.2e6, hbm = w_us * (w_us > 38.0 ? (double)nrb : 1.0);
            const double stage = 0.14 + 0.035 * rf + 0.06 * rf * nc;
            const double body = (double)((wgs + 255) / 256) * (4.0 + (double)K / 64.0 * stage);
            const double us = 1.0 + std::max(hbm + 4.0, body) + 0.15 * std::min(hbm, body);
            if (best == 0 || us < best) {
                best = us;
                *rf_out = rf;
                *nc_out = nc;
            }
        }
}
template <Skinny KIND>
static hipError_t skinny_linear(int rf, int nc, const SkinnyArgs& a, hipStream_t s) {
    switch (nc) {
        case 1: return skinny_rf<1, KIND>(rf, a, s);
        case 2: return skinny_rf<2, KIND>(rf, a, s);
        case 3: return skinny_rf<3, KIND>(rf, a, s);
        case 4: return skinny_rf<4, KIND>(rf, a, s);
        default: return skinny_rf<6, KIND>(rf, a, s);
    }
}
hipError_t launch_skinny_f32(const SkinnyArgs& a, bool gated, bool plain, hipStream_t s) {
    int rf = 0, nc = 0;
    plan_f32(a.M, a.K, a.nblocks, gated, &rf, &nc);
    if (gated) switch (nc) {
            case 2: return skinny_rf<2, Skinny::kSwiGlu>(rf, a, s);
            case 4: return skinny_rf<4, Skinny::kSwiGlu>(rf, a, s);
            default: return skinny_rf<6, Skinny::kSwiGlu>(rf, a, s);
        }
    return plain ? skinny_linear<Skinny::kPlain>(rf, nc, a, s) : skinny_linear<Skinny::kLinear>(rf, nc, a, s);
}

}  // namespace dn
