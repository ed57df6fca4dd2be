// launch_rules.hpp -- which kernel and which layout takes a call, from its sizes alone.  Host
// code without HIP, so that the rules can be evaluated (and are tested) without a GPU.
#pragma once
#include <algorithm>
#include <stddef.h>
#include <stdint.h>

namespace dn {

// ------------------------------------------------------- LayerNorm/RMSNorm/gated/plain products
// Workgroups for tm x tn tiles.  Deferred LN: each workgroup takes `group` column
// tiles of one row block and reduces the row moments once, on its first tile.
// With one workgroup per CU the run takes about ceil(workgroups / 256) * group
// tile times; take the group that minimises that, and of equal ones the largest
// (fewest moment reductions).  384 tiles: group 2 (192 workgroups, 2 tile times)
// instead of group 1 (384 workgroups, also 2 tile times, twice the moment work).
struct TilePlan {
    int64_t group, ngroups, wgs, times;
};
inline TilePlan plan_tiles(int64_t tm, int64_t tn, bool grouped) {
    int64_t group = 1;
    if (grouped) {
        int64_t best = -1;
        for (int64_t g = 1; g <= tn; ++g) {
            const int64_t span = (tm * ((tn + g - 1) / g) + 255) / 256 * g;
            if (best < 0 || span <= best) {
                best = span;
                group = g;
            }
        }
    }
    const int64_t ngroups = (tn + group - 1) / group, wgs = tm * ngroups;
    return TilePlan{group, ngroups, wgs, (wgs + 255) / 256 * group};
}

// 256 x 192 tiles where they fill the chip in fewer 256 x 256-tile times: a narrow
// tile costs about kNarrowCost of a square one (three quarters of the MACs, a
// little more operand traffic per MAC).  4096 x 4096 -> 6144: 512 narrow tiles in
// two full rounds instead of 384 square ones in 1.5; 1024 x 4096 -> 12288: 256
// instead of 192 on 256 CUs.
constexpr double kNarrowCost = 0.8;
inline TilePlan plan_256_tiles(int64_t M, int64_t N, bool grouped, bool* narrow) {
    const int64_t tm = (M + 255) / 256;
    const TilePlan square = plan_tiles(tm, (N + 255) / 256, grouped), thin = plan_tiles(tm, (N + 191) / 192, grouped);
    *narrow = (double)thin.times * kNarrowCost < (double)square.times;
    return *narrow ? thin : square;
}

// The 256x256 kernel past 128 rows (and K a multiple of its stage), where the
// 128 x 128 tiles do not fit in one round.  Below one 256 x 256 tile per CU it
// still beats the two-stage 128 x 128 loop, which then needs a second round of
// tiles where the 256 x 256 kernel needs none.  Measured on 4096 -> 12288:
// 768 and 1024 rows 89 / 97 us against 178 / 185 us; 8192 -> 28672 at 384 and
// 512 rows 222 / 226 against 376 / 381 us, at 129-256 rows within 5 %.
inline bool use_big_tiles(int64_t M, int64_t N, int64_t K) {
    if (N >= (int64_t(1) << 22)) return false;  // 256 output rows < 2^31 bytes (32-bit store offsets)
    // K < 2^22 keeps the 32-bit copy offsets of a 256-row panel (256 K bf16) and of a
    // 16-chunk-column W' panel (16 x K/32 KiB) below 4 GiB.
    return K % 64 == 0 && K < (int64_t(1) << 22) && M > 128;
}
// The pipelined kernel on 128 x 128 tiles (4 waves, two workgroups per CU) while
// those tiles number at most one per CU: then a tile takes far less than a
// 256 x 256 one and the chip is as full.  Measured on 4096 -> 12288 at 129 / 256
// rows (192 tiles) 56 / 58 us against 86 us on 256 x 256 tiles, on 8192 -> 28672
// at 65 / 100 rows (224 tiles) 132 / 133 us against 174 / 184 us on the 128 x 128
// two-stage loop; at 288 tiles and more it lost (97-448 us against 89-230 us).
inline bool use_mid_tiles(int64_t M, int64_t N, int64_t K) {
    return K % 64 == 0 && K < (int64_t(1) << 22) && N < (int64_t(1) << 22) &&
           ((M + 127) / 128) * ((N + 127) / 128) <= 256;
}

// bf16 rows up to which the decode kernel runs.
constexpr int64_t kDecodeRows = 16;

// ---- the streamed kernel, bf16
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
inline SkinnyPlan plan_skinny(int64_t M, int64_t K, int64_t nblocks, bool gated) {
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
inline double skinny_estimate_us(int64_t M, int64_t K, int64_t nblocks, bool gated) {
    return plan_skinny(M, K, nblocks, gated).us;
}

// ---- the streamed kernel, fp32
// The plan by estimated time, as for bf16 with fp32's stages: 0.06 rf nc us of
// matrix work per 64 k and 0.14 + 0.035 rf us besides.  Measured (graph replays, us; before:
// 32 x 64 tiles of a two- to four-stage loop whose x copies were half lines): 128 rows
// 768 -> 3072 12.6 / 15.3, 1 row 4096 -> 6144 22 / 54, 1 row 4992 -> 1104 16 / 64, 477 rows
// 4096 -> 12288 410 / 632 (117 TFLOP/s), 1000 rows 768 -> 3072 46 / 78.
inline void plan_f32(int64_t M, int64_t K, int64_t nblocks, bool gated, int* rf_out, int* nc_out) {
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

// The streamed few-row kernel against the tiles.  Up to 128 rows it always runs (4096 -> 12288
// at 24 / 50 / 100 rows 21 / 24 / 32 us, where the decode layout with 2 - 8 row fragments per
// wave took 24 / 38 / 55 us on the same card; 8192 -> 28672 at 60 / 100 rows 79 / 95 against
// 125 / 144 us).  Past that it runs where its estimate is below 0.85 of the tiles' (us, same cards):
// 200 rows 4096 -> 12288 43 / 63, 313 and 500 rows 4096 -> 6144 35 / 58 and 40 / 59, 300 rows
// 768 -> 3072 9 / 17; at 1000 rows 4096 -> 12288 it would take 151 against 105.
// The 0.85 covers the error of the two estimates: at 0.95, 5233 rows of 752 -> 1176 came here
// and took 28.9 us instead of 27.2.  The plain product's tiles carry no moments and take about
// 0.7 of their estimate (streamed / tiles, us: 4096 rows 768 -> 768 13.7 / 10.0, 1500 rows
// 768 -> 2304 11.3 / 10.7, 512 rows 768 -> 2304 8.4 / 9.6).
// Past the 4 MiB of an XCD's L2 the row blocks' reads of x cost about 0.7 us per MB more than the
// plan's estimate (streamed / tiles, eager us: 4096 rows 768 -> 768 15.5 / 14.7, 5500 rows
// 752 -> 1176 29.2 / 27.3, gated 3100 rows 752 -> 1176 26.4 / 24.6; 3300 rows 768 -> 768
// 14.5 / 16.8, 3000 rows 1024 -> 1024 16.7 / 19.2).  128 x 128 tiles with a ragged last row block
// take about 5 % more than their estimate, the two-stage loop 5 % more alone and 5 % less two to a CU.
// Tiles, per 64 k: 128 x 128 in one round 0.83 us, 256 x 256 1.3 us (1.6 us with the chip full
// and its clock down), the two-stage 128 x 128 loop 1.6 us alone and 1.9 us two to a CU.
inline double tiles_estimate_us(int64_t M, int64_t N, int64_t K, bool grouped) {
    const double k64 = (double)K / 64.0;
    if (use_mid_tiles(M, N, K)) return 5.0 + k64 * 0.83;
    const int64_t tm = (M + 255) / 256;
    if (use_big_tiles(M, N, K)) {
        const TilePlan sq = plan_tiles(tm, (N + 255) / 256, grouped), na = plan_tiles(tm, (N + 191) / 192, grouped);
        const double full = (sq.wgs >= 192 ? 1.6 : 1.3) * k64;
        return 5.0 + full * std::min((double)sq.times, (double)na.times * kNarrowCost);
    }
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);  // two fit a CU
    return 5.0 + (tiles > 256 ? 1.9 : 1.6) * k64 * (double)((tiles + 511) / 512);
}
inline bool use_skinny(int64_t M, int64_t N, int64_t K, int64_t nblocks, int dtype, bool gated, bool plain) {
    if (K >= (int64_t(1) << 22)) return false;
    if (dtype == 0) return true;
    if (M <= kDecodeRows) return false;
    if (M <= 128) return true;
    const double us = skinny_estimate_us(M, K, nblocks, gated), tiles = tiles_estimate_us(M, N, K, !plain);
    if (us >= (plain ? 0.7 : 0.85) * tiles) return false;
    const double x_mb = 2e-6 * (double)M * (double)K;
    const int64_t tiles128 = ((M + 127) / 128) * ((N + 127) / 128);
    const double fit = use_mid_tiles(M, N, K)   ? (M % 128 ? 1.05 : 1.0)
                       : use_big_tiles(M, N, K) ? 1.0
                                                : (tiles128 > 256 ? 0.95 : 1.05);
    return plain || x_mb < 4.3 || us + 0.7 * x_mb < fit * tiles;
}

// Which kernel takes a product on packed weights (N counts packed columns).
enum class Product { kDecode, kStreamed, kTiles128, kTiles256, kTwoStage };
inline Product product_kernel(int64_t M, int64_t N, int64_t K, int dtype, bool gated, bool plain) {
    if (dtype == 1 && M <= kDecodeRows) return Product::kDecode;
    if (use_skinny(M, N, K, (N + 15) / 16, dtype, gated, plain)) return Product::kStreamed;
    if (use_mid_tiles(M, N, K)) return Product::kTiles128;
    return use_big_tiles(M, N, K) ? Product::kTiles256 : Product::kTwoStage;
}

// ------------------------------------------------------------------------- Softmax -> P.V
// Layouts, by the number of workgroups they give.  8 waves x 2 fragments (256 queries, two V and
// two S slots like the others, 96 KiB of LDS at d = 128; deeper rings measured no faster) read V
// least and are best once they fill the chip; 8 x 1 (128 queries) and 4 x 1 (64 queries) give 2 and
// 4 times the workgroups, two and more to a CU.  Where one step follows another in too few waves,
// 32 queries: with the keys split two ways inside the workgroup, or (causal rows, and those of one
// step, which have nothing to split) unsplit on 4-deep (d = 128: 3-deep) rings.
// Measured (us, 256 / 128 / 64 queries / 32 split; causal the last one 32 unsplit):
//   full    27 x 5536, d128 443 / 431 / 499 / 583    10 x 4200, d128 127 / 128 / 132 / 158
//           16 x 2048, d128  51 /  37 /  41 /  54    32 x 1000, d128  34 / 24.5 / 27 / 37
//           20 x 3000, d64  105 / 103 / 110 / 132    12 x 512, d64    15 / 10.0 / 8.9 / 7.8
//   causal  32 x 8192, d128 454 / 496 / 496          29 x 7104, d128 349 / 425 / 616
//           15 x 6240, d128 185 / 181 / 223          16 x 2048, d128  49 / 34.5 / 34.5
//           8 x 8192, d64   146 / 122 / 120          11 x 728, d128   24 / 15.3 / 13.2
// The split against 64 queries, by its workgroups n32 and the keys (us, d = 64 and d = 128): at
// most 256 workgroups, 8 heads x 32 queries x 8192 keys 37 / 64 and 46 / 74, 16 x 300 x 3000
// 17.9 / 27.5 and 21.9 / 31.6, 200 x 32 x 2048 15.0 / 20.2 and 22.3 / 23.2 (128 queries 22.7 and
// 27.7); more, 8 x 2048 x 2048
// 17.9 / 20.9 and 24.7 / 23.9, 16 x 1024 x 1024 10.7 / 12.1 and 14.5 / 14.4, 5 x 3000 x 3000
// 31.2 / 29.4 and 39.5 / 33.6, 100 x 100 x 3000 31.9 / 29.5 and 40.6 / 33.7.
// 32 queries unsplit against 64, causal (us): d = 64 8 x 2048 18.2 / 19.4, 4 x 1024 10.5 / 11.1,
// 1 x 64 3.50 / 3.60; d = 128 8 x 2048 27.1 / 23.4, 4 x 1024 15.1 / 13.0.
enum class SoftmaxLayout { k256, k128, k64, k32, kSplit };
inline SoftmaxLayout softmax_layout(int64_t BH, int64_t Lq, int64_t Lk, int64_t d, int causal) {
    const int64_t n256 = BH * ((Lq + 255) / 256), n128 = BH * ((Lq + 127) / 128), n32 = BH * ((Lq + 31) / 32);
    if (causal) {
        if (n256 > 160) return n256 > 512 ? SoftmaxLayout::k256 : SoftmaxLayout::k128;
        return d == 64 ? SoftmaxLayout::k32 : SoftmaxLayout::k64;
    }
    if (n32 <= 256 && Lk > 64) return SoftmaxLayout::kSplit;
    if (n128 > 160) return n128 > 256 ? SoftmaxLayout::k256 : SoftmaxLayout::k128;
    if (Lk <= 64) return SoftmaxLayout::k32;
    return Lk <= (d == 64 ? 2048 : 1024) ? SoftmaxLayout::kSplit : SoftmaxLayout::k64;
}

// ------------------------------------------------------------------------- attention, prefill
// Query rows per workgroup of the prefill layouts (every layout's key step covers 128 keys).
constexpr int64_t kMaxPrefillGrid = (int64_t(1) << 31) - 1;
constexpr int kPrefillBQ[4] = {256, 128, 64, 32};

// Which layout.  Fewer queries per workgroup cost more per score (the K and V fragments read
// from LDS serve fewer queries: per 128-key step at d = 128 and a full chip 3.35 us for 256
// queries, 1.9 for 128, 1.3 for 64, 1.0 for 32), but give more workgroups and split each one's
// keys 1, 2, 4 and 4 ways.  The time is about the larger of the longest workgroup's (its steps
// at the lone-workgroup rate, plus a start and an end) and of all the work over 256 CUs; the
// layout with the smallest estimate runs.  Measured, best layout against 256 queries for all
// (graph replays, us): 8 heads x 512, d64 7.2 / 14; 32 x 1000 causal 20.9 / 29; 16 x 512
// against 3000 keys 27 / 67; 32 x 2048 causal 45 / 51; from 32 x 4096 causal on 256 is best
// (122 / 142 with 128).
inline int prefill_layout(int64_t BH, int64_t Lq, int64_t Lk, int64_t d, int causal) {
    struct Cost {
        double full, alone, ends;  // us per step with every CU busy / alone, us per workgroup
    };
    static constexpr Cost kCost[2][4] = {{{2.0, 1.75, 7.0}, {1.2, 1.1, 6.0}, {0.64, 0.7, 3.5}, {0.44, 0.5, 2.8}},
                                         {{3.35, 2.5, 8.0}, {1.9, 1.55, 6.5}, {1.3, 1.1, 6.0}, {1.0, 0.88, 3.5}}};
    int best = 0;
    double best_t = 0;
    for (int v = 0; v < 4; ++v) {
        const Cost& c = kCost[d == 128][v];
        const int64_t n = (Lq + kPrefillBQ[v] - 1) / kPrefillBQ[v], wgs = BH * n;
        if (wgs > kMaxPrefillGrid) continue;
        const int64_t longest = (Lk + 127) / 128;
        const double mean = causal ? 0.5 * (double)(longest + 1) : (double)longest;
        const double t = std::max((double)longest * c.alone + c.ends, (double)wgs * (mean * c.full + c.ends) / 256.0);
        if (v == 0 || t < best_t) {
            best = v;
            best_t = t;
        }
    }
    return best;
}

// 256 queries per workgroup: the two halves of a workgroup one phase apart, or in step.  In step /
// apart (graph replays, us): d = 128 32 heads x 4096 queries x 64 keys 24.5 / 28.0, 1024 65.3 / 66.5,
// 3000 167.2 / 167.4, 4096 210.8 / 209.4, 8192 806 / 793; causal 512 x 200 28.1 / 34.2, 100 x 700
// 30.2 / 35.5, 64 x 2048 68.3 / 71.0, 32 x 8192 429.2 / 429.4; d = 64 32 x 4096 x 64 13.8 / 17.0,
// 2048 70.8 / 71.0, 4096 133.2 / 132.5, 8192 503 / 496.
inline bool prefill_phased(int64_t Lk) { return Lk > 3072; }

// ------------------------------------------------------------------------- attention, decode
// Workgroups of one resident round: 128 KiB of LDS at d = 128 (1 per CU), 64 KiB at d = 64 (2).
inline int64_t decode_resident(int64_t d) { return d == 64 ? 512 : 256; }
// Runs across heads: `per` units each; fewer than 2 x 256 (d = 128) or 2 x 512 (d = 64) partial
// slots, none where every run is whole heads.
struct DecodePlan {
    int64_t units, per, wgs, slots;
    int nsplit;
};
inline DecodePlan decode_plan(int64_t BH, int64_t Lk, int64_t d) {
    DecodePlan p;
    p.units = (Lk + 127) / 128;
    const int64_t total = BH * p.units;
    p.per = (total + decode_resident(d) - 1) / decode_resident(d);
    p.wgs = (total + p.per - 1) / p.per;
    p.nsplit = p.units % p.per == 0 ? (int)(p.units / p.per) : 0;  // runs that end with each head
    p.slots = p.per % p.units == 0 ? 0 : p.nsplit ? BH * p.nsplit : p.per > p.units ? 2 * p.wgs : BH + p.wgs;
    return p;
}
// The same number of runs for every head (the layout smaller workspaces were sized for).
inline int64_t decode_uniform(int64_t BH, int64_t Lk, int64_t d, int64_t* per) {
    const int64_t units = (Lk + 127) / 128, w = decode_resident(d);
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(units, (w + BH - 1) / BH));
    *per = (units + want - 1) / want;
    return (units + *per - 1) / *per;
}
inline size_t slots_bytes(int64_t slots, int64_t Lq, int64_t d) {
    return (size_t)slots * (size_t)Lq * (size_t)(d + 4) * sizeof(float);
}
inline size_t attention_decode_least_bytes(int64_t BH, int64_t Lq, int64_t Lk, int64_t d) {
    int64_t per;
    return slots_bytes(BH * decode_uniform(BH, Lk, d, &per), Lq, d);
}
inline size_t attention_decode_workspace_bytes(int64_t BH, int64_t Lq, int64_t Lk, int64_t d) {
    return std::max(attention_decode_least_bytes(BH, Lq, Lk, d), slots_bytes(decode_plan(BH, Lk, d).slots, Lq, d));
}
// The same without a workspace: partials go to the library's own array, which calls that overlap
// share, so none are left where the heads alone fill the chip (or one unit holds all keys); then
// one workgroup takes each head: 34.2 us against 29.2 for 300 heads x 1000 keys at d = 128, 235
// against 201 with 8000 keys (the deal's partials in the array), 14.5 against 16.0 for 1100 x 200 at d = 64.
inline size_t attention_decode_partials_bytes(int64_t BH, int64_t Lq, int64_t Lk, int64_t d) {
    int64_t per;
    return decode_uniform(BH, Lk, d, &per) == 1 ? 0 : slots_bytes(decode_plan(BH, Lk, d).slots, Lq, d);
}

}  // namespace dn
