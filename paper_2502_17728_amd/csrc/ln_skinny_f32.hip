// ln_skinny_f32.hip -- LayerNorm/RMSNorm products on packed fp32 weights, every size.
#include "launch_rules.hpp"
#include "ln_skinny.hpp"

namespace dn {

template <int NC, Skinny KIND>
static hipError_t skinny_rf(int rf, const SkinnyArgs& a, hipStream_t s) {
    switch (rf) {
        case 1:
            if constexpr (NC == 6) return hipErrorInvalidValue;  // not planned: two-deep rings only
            else return run_skinny_kernel<float, 1, 8, NC, KIND>(a, s);
        case 2: return run_skinny_kernel<float, 2, 4, NC, KIND>(a, s);
        case 4: return run_skinny_kernel<float, 4, 2, NC, KIND>(a, s);
        default: return run_skinny_kernel<float, 8, 1, NC, KIND>(a, s);
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
