// ln_skinny.hip -- LayerNorm/RMSNorm products of few rows, bf16: the kernel between the decode
// stream (ln_gemm.hip, up to 16 rows) and the large MFMA tiles.
#include "launch_rules.hpp"
#include "ln_skinny.hpp"

namespace dn {

template <int NC, Skinny KIND>
static hipError_t skinny_rf(int rf, const SkinnyArgs& a, hipStream_t s) {
    switch (rf) {
        case 2: return run_skinny_kernel<__bf16, 2, 4, NC, KIND>(a, s);
        case 3: return run_skinny_kernel<__bf16, 3, 2, NC, KIND>(a, s);
        case 4: return run_skinny_kernel<__bf16, 4, 2, NC, KIND>(a, s);
        case 6: return run_skinny_kernel<__bf16, 6, 1, NC <= 8 ? NC : 8, KIND>(a, s);
        default: return run_skinny_kernel<__bf16, 8, 1, NC <= 8 ? NC : 8, KIND>(a, s);
    }
}

template <Skinny KIND>
static hipError_t skinny_linear(const SkinnyPlan& p, const SkinnyArgs& a, hipStream_t s) {
    switch (p.nc) {
        case 1: return skinny_rf<1, KIND>(p.rf, a, s);
        case 2: return skinny_rf<2, KIND>(p.rf, a, s);
        case 3: return skinny_rf<3, KIND>(p.rf, a, s);
        case 4: return skinny_rf<4, KIND>(p.rf, a, s);
        case 6: return skinny_rf<6, KIND>(p.rf, a, s);
        default: return skinny_rf<7, KIND>(p.rf, a, s);
    }
}
hipError_t launch_skinny(const SkinnyArgs& a, bool gated, bool plain, hipStream_t s) {
    const SkinnyPlan p = plan_skinny(a.M, a.K, a.nblocks, gated);
    if (gated) switch (p.nc) {
            case 2: return skinny_rf<2, Skinny::kSwiGlu>(p.rf, a, s);
            case 4: return skinny_rf<4, Skinny::kSwiGlu>(p.rf, a, s);
            case 6: return skinny_rf<6, Skinny::kSwiGlu>(p.rf, a, s);
            case 8: return skinny_rf<8, Skinny::kSwiGlu>(p.rf, a, s);
            default: return skinny_rf<14, Skinny::kSwiGlu>(p.rf, a, s);
        }
    return plain ? skinny_linear<Skinny::kPlain>(p, a, s) : skinny_linear<Skinny::kLinear>(p, a, s);
}

}  // namespace dn
