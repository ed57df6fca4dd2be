// ln_skinny.hip -- LayerNorm/RMSNorm products of few rows, bf16: the kernel between the decode
// stream (ln_gemm.hip, up to 16 rows) and the large MFMA tiles.
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

// Row fragments per block and column blocks per workgroup, by estimated time: rounds of 256
// workgroups, each filling its rings (4 us) and then K / 64 stages of kRow[rf] + 0.03 nc us
// (fitted to graph replays at K 4096; more rows per block cost more per stage, but W' is read
// fewer times), or W' from HBM at 6.2 TB/s if that is longer.  Of two plans bound the same way
// the one with the shorter other part wins.  Measured: 100 rows on 4096 -> 12288, 64-row blocks
// x 6 column blocks 29 us, 128 x 4 32 us, 128 x 1 100 us; 64 rows of the gated MLP on
// 8192 -> 2 x 28672, 64 x 14 143 us, 64 x 4 187 us, 32-row blocks (W' read twice) 262 us.
struct SkinnyPlan {
    int rf, nc;
    double us;
};
static SkinnyPlan plan_skinny(int64_t M, int64_t K, int64_t nblocks, bool gated) {
    static constexpr int kRf[5] = {2, 3, 4, 6, 8};
    static constexpr double kRow[5] = {0.08, 0.19, 0.21, 0.29, 0.34};
    static constexpr int kNc[6] = {1, 2, 3, 4, 6, 7}, kNcGated[5] = {2, 4, 6, 8, 14};
    SkinnyPlan best{0, 0, 0};
    const double w_us = (double)nblocks * 32.0 * (double)K / 6.2e6;  // one pass over W' (bytes / 6.2 TB/s)
    for (int i = 0; i < 5; ++i)
        for (int j = 0; j < (gated ? 5 : 6); ++j) {
            const int rf = kRf[i], nc = gated ? kNcGated[j] : kNc[j];
            if (nc > 8 && rf > 4) continue;  // registers
            const int64_t nrb = (M + 16 * rf - 1) / (16 * rf), wgs = nrb * ((nblocks + nc - 1) / nc);
            // W' past the last-level cache is read once per row block
            const double hbm = w_us * (w_us > 32.0 ? (double)nrb : 1.0);
            const double body = (double)((wgs + 255) / 256) * (4.0 + (double)K / 64.0 * (kRow[i] + 0.03 * nc));
            const double us = 1.0 + std::max(hbm + 4.0, body) + 0.15 * std::min(hbm, body);
            if (best.rf == 0 || us < best.us) best = SkinnyPlan{rf, nc, us};
        }
    return best;
}
double skinny_estimate_us(int64_t M, int64_t K, int64_t nblocks, bool gated) {
    return plan_skinny(M, K, nblocks, gated).us;
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
