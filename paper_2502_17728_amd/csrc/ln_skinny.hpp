// ln_skinny.hpp -- the streamed LayerNorm/RMSNorm/gated/plain product kernel on packed weights
// (instantiated for bf16 in ln_skinny.hip and for fp32 in ln_skinny_f32.hip).
#pragma once
#include <algorithm>
#include <type_traits>

#include "dn_device.hpp"
#include "dn_launch.hpp"

namespace dn {

// =============================================================================
// Skinny products: row blocks of 16 RF rows (RF 1 .. 8).  bf16: batched decode, short
// prompts, and larger calls whose big tiles would leave CUs idle; fp32: every size.  Every workgroup streams
// the whole x block and its NC blocks of 16 W' columns, so per CU the two streams are of one
// size and what counts is that neither ever waits: both go through LDS rings filled by
// global->LDS copies that need no registers, x NXS and W' NWS stages deep (together up to
// 160 KiB in flight per CU), x as whole 128-byte lines (8 rows x 128 B per copy, 16-byte
// pieces XOR-swizzled), W' as its contiguous KiB chunks.  A stage is CH chunks (32 bf16 or 16 fp32 of K); the
// RF x KH waves take one row fragment and every KH-th chunk each, so a wave's accumulators
// are few and the copies, fragment reads and products of the waves overlap.  The products
// are taken transposed (A = W', B = x): a lane owns one token, its statistics and 4
// consecutive features of each column block.  Moments: bf16 on the matrix cores as in the
// decode kernel (sum x with an all-ones operand, sum x^2 as the diagonal of the Gram block);
// fp32, whose matrix instructions are the bound, on the VALU from the same fragments.
// =============================================================================
template <class T, int RF, int KH, int NC, int NXS, int NWS, bool SW, bool PLAIN>
__global__ __launch_bounds__(RF* KH* kWave) void ln_skinny_kernel(
    const T* __restrict__ x, const char* __restrict__ Wp, int64_t kchunks, int64_t nblocks,
    const float* __restrict__ c_col, const float* __restrict__ b_col, int64_t M_all, int64_t K, int64_t N, float eps,
    int rms, int64_t n_out, const float* __restrict__ row_stats, float* __restrict__ stats_out,
    T* __restrict__ out, const T* __restrict__ bias, int nrb) {
    static_assert(!SW || NC % 2 == 0, "gate/up block pairs");
    static_assert(!(SW && PLAIN), "the plain product has no gate");
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int ES = sizeof(T), EPL = elem<T>::per16, KC = elem<T>::kchunk;
    constexpr int NW = RF * KH;
    constexpr int CH = KH < 2 ? 2 : KH;            // chunks per stage
    constexpr int CPW = CH / KH;                   // chunks per wave and stage
    constexpr int XST = RF * CH * kChunkBytes, WST = NC * CH * kChunkBytes;
    // The first half of the waves copies x, the second W': the counter a wave waits on runs in
    // issue order, so behind one wave's W' loads (HBM) its x copies (L2) could not be waited
    // for on their own, nor W' be left in flight longer than the shallower x ring.
    constexpr int HW = NW / 2;
    constexpr int PX = RF * CH / HW, PW = (NC * CH + HW - 1) / HW;  // copies per wave and stage
    constexpr int RED = (KH - 1) * RF * (NC + 2) * kWave * 16;  // partial sums of the KH - 1 other waves
    constexpr int RING = NXS * XST + NWS * WST;
    static_assert(CH % 2 == 0 && CH % KH == 0 && NW % 2 == 0 && RF * CH % HW == 0, "stage split");
    static_assert(NXS >= 2 && NWS >= 2 && PX * NXS < 64 && PW * NWS < 64 && RING <= 160 * 1024, "rings");
    __shared__ __attribute__((aligned(1024))) char smem[RING > RED ? RING : RED];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rf = wave % RF, kh = wave / RF;
    const int G = lane >> 4, i16 = lane & 15;
    // row blocks of one column group next to each other (they read the same W')
    const int t = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t m0 = (int64_t)(t % nrb) * (16 * RF), nb0 = (int64_t)(t / nrb) * NC;
    const int M = (int)min(M_all - m0, (int64_t)(16 * RF));
    const bool stream = nrb == 1;  // W' is read by this workgroup only
    const T* xm = x + m0 * K;

    // x copies: copy c of a stage covers rows 8 (c % 2RF) .. of its (c / 2RF)-th 128-byte column;
    // lane l fetches piece (l & 7) ^ a_swz(row) of row 8 (..) + (l >> 3).  Rows past M re-read
    // the last one (their results are dropped), pieces past K the row's last (zeroed at use).
    const bool xwave = wave < HW;
    const int cw = xwave ? wave : wave - HW;  // this wave's share of the copies
    const int nst = (int)((kchunks + CH - 1) / CH);
    const uint32_t smem_addr = lds_addr32(smem);
    // Stages before the last need no clamp: fixed lane offsets (x: row and piece; W': column
    // block and chunk) from a scalar base that advances by a stage.
    uint32_t off[PX > PW ? PX : PW];
    const uint64_t base0 = xwave ? uniform_u64(xm) : uniform_u64(Wp + packed_chunk(nb0, 0, kchunks, 0));
    const int nb_left = (int)min(nblocks - nb0, (int64_t)NC) - 1;
#pragma unroll
    for (int j = 0; j < (PX > PW ? PX : PW); ++j) {
        const int cx = cw + j * HW, r = 8 * (cx % (2 * RF)) + (lane >> 3);
        const int c = min(cw + j * HW, NC * CH - 1);  // the last W' copies may repeat a chunk
        off[j] = xwave ? (uint32_t)min(r, M - 1) * (uint32_t)(K * ES) +  // 128 rows of K < 2^22: below 2^32
                             (uint32_t)((cx / (2 * RF)) * 128 + ((lane & 7) ^ a_swz(r)) * 16)
                       : (uint32_t)(min(c / CH, nb_left) * kchunks + c % CH) * kChunkBytes + lane * 16;
    }
    auto issue_x = [&](int s, uint32_t slot) __attribute__((always_inline)) {  // slot: byte offset in the ring
        const uint32_t dst = smem_addr + slot + (uint32_t)(cw * kChunkBytes);
        if (s < nst - 1) {
            const uint64_t src = base0 + (uint64_t)((uint32_t)s * (CH * 64u));
#pragma unroll
            for (int j = 0; j < PX; ++j) g2lds16_async_sb(src, off[j], dst + (uint32_t)(j * HW * kChunkBytes));
        } else {  // the last stage (and its repeats past the end): pieces past K clamp onto the row's last
#pragma unroll
            for (int j = 0; j < PX; ++j) {
                const int cx = cw + j * HW, r = 8 * (cx % (2 * RF)) + (lane >> 3);
                const uint32_t k = (uint32_t)((nst - 1) * CH * 64 + (cx / (2 * RF)) * 128 + ((lane & 7) ^ a_swz(r)) * 16);
                g2lds16_async_sb(base0, (uint32_t)min(r, M - 1) * (uint32_t)(K * ES) + min(k, (uint32_t)(K * ES - 16)),
                                 dst + (uint32_t)(j * HW * kChunkBytes));
            }
        }
    };
    auto issue_w = [&](int s, uint32_t slot) __attribute__((always_inline)) {
        const uint32_t dst = smem_addr + (uint32_t)(NXS * XST) + slot;
        auto go = [&](auto nt) __attribute__((always_inline)) {
            const uint64_t src = base0 + (uint64_t)((uint32_t)min(s, nst - 1) * (uint32_t)(CH * kChunkBytes));
#pragma unroll
            for (int j = 0; j < PW; ++j) {
                const uint32_t c = (uint32_t)min(cw + j * HW, NC * CH - 1);
                uint32_t o = off[j];
                if (s >= nst - 1) {  // the last stage: chunks past the last clamp onto it
                    const int over = (nst - 1) * CH + (int)(c % CH) - ((int)kchunks - 1);
                    o -= (uint32_t)(over > 0 ? over : 0) * kChunkBytes;
                }
                if constexpr (decltype(nt)::value)
                    g2lds16_stream_sb(src, o, dst + c * kChunkBytes);
                else
                    g2lds16_async_sb(src, o, dst + c * kChunkBytes);
            }
        };
        if (stream)
            go(std::true_type{});
        else
            go(std::false_type{});
    };

    const u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const u32x4 zero = {0, 0, 0, 0};
    const f32x4 fz = {0.f, 0.f, 0.f, 0.f};
    f32x4 acc[NC], sx = fz, sxx = fz;
    float s1 = 0.f, s2 = 0.f;  // fp32: the lane's share of its token's moments
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[q] = fz;
    const int xr = rf * 16 + i16;  // the lane's token row in the x tile
    using Frags = u32x4[CPW][NC + 1];  // x, then the W' blocks
    auto read = [&](Frags& f, uint32_t xslot, uint32_t wslot) __attribute__((always_inline)) {
        const char* xb = smem + xslot;
        const char* wb = smem + NXS * XST + wslot;
#pragma unroll
        for (int u = 0; u < CPW; ++u) {
            const int ch = kh + u * KH;  // chunk of the stage
            const int piece = (ch & 1) * 4 + G;
            f[u][0] = lds_ld16(lds_ptr((char*)xb + (ch >> 1) * (2 * RF * kChunkBytes) + xr * 128 +
                                       ((piece ^ a_swz(xr)) << 4)));
#pragma unroll
            for (int q = 0; q < NC; ++q)
                f[u][1 + q] = lds_ld16(lds_ptr((char*)wb + (q * CH + ch) * kChunkBytes + lane * 16));
        }
    };
    auto compute = [&](Frags& f, int s, auto tail) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CPW; ++u) {
            if constexpr (decltype(tail)::value) {  // the last stage may reach past K
                const int ch = s * CH + kh + u * KH;
                if (ch >= (int)kchunks) continue;  // a repeated W' chunk: 0 times an infinite weight is NaN
                f[u][0] = (int64_t)ch * KC + G * EPL < K ? f[u][0] : zero;
            }
            if constexpr (F32) {  // a chunk is four dependent products per block: the blocks' chains interleave
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int q = 0; q < NC; ++q)
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(f[u][1 + q][j]),
                                                                      __uint_as_float(f[u][0][j]), acc[q], 0, 0, 0);
                if constexpr (!PLAIN) chunk_moments<float>(f[u][0], s1, s2);
                continue;
            }
#pragma unroll
            for (int q = 0; q < NC; ++q) acc[q] = mfma_chunk<__bf16>(f[u][1 + q], f[u][0], acc[q]);
            if constexpr (!PLAIN) {
                sx = mfma_chunk<__bf16>(ones, f[u][0], sx);
                sxx = mfma_chunk<__bf16>(f[u][0], f[u][0], sxx);
            }
        }
        if constexpr (!decltype(tail)::value) {  // the next stage's reads beside this one's products
#pragma unroll
            for (int i = 0; i < CPW * (NC + 1); ++i) {
                __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 0);
                __builtin_amdgcn_sched_group_barrier(kSgMfma, F32 ? 2 : 1, 0);
            }
        }
    };
    // Copies run a whole ring ahead: iteration s reads the fragments of stage s + 1 into
    // registers while stage s, read an iteration ago, multiplies, so stage s's slots already
    // take x(s + NXS) and W'(s + NWS).  Stage s + 1 has landed once each wave has at most its
    // copies of the stages after it in flight.
    if (xwave) {
#pragma unroll
        for (int j = 0; j < NXS; ++j) issue_x(j, j * XST);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NXS - 1) * PX) : "memory");
    } else {
#pragma unroll
        for (int j = 0; j < NWS; ++j) issue_w(j, j * WST);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NWS - 1) * PW) : "memory");
    }
    block_barrier();
    Frags f0, f1;
    read(f0, 0, 0);
    uint32_t xs = 0, ws = 0;  // ring slots of stage s, byte offsets
    auto stage = [&](int s, Frags& cur, Frags& next, auto tail) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(tail)::value;
        const uint32_t xo = xs, wo = ws;
        if constexpr (!LAST) {
            if (xwave)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NXS - 2) * PX) : "memory");
            else
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NWS - 2) * PW) : "memory");
            wait_lgkm0();     // this wave's reads of stage s are done
            block_barrier();  // ... and every wave's; every wave's copies of stage s + 1 have landed
            xs = xs + XST == NXS * XST ? 0u : xs + XST;
            ws = ws + WST == NWS * WST ? 0u : ws + WST;
            read(next, xs, ws);
        }
        compute(cur, s, tail);
        if constexpr (!LAST) {  // the copies' issue beside the products
            if (xwave)
                issue_x(s + NXS, xo);
            else
                issue_w(s + NWS, wo);
        }
    };
    using no = std::false_type;
    using yes = std::true_type;
    int s = 0;
    for (; s + 2 < nst; s += 2) {
        stage(s, f0, f1, no{});
        stage(s + 1, f1, f0, no{});
    }
    if (s + 1 < nst) {
        stage(s, f0, f1, no{});
        stage(s + 1, f1, f0, yes{});
    } else {
        stage(s, f0, f1, yes{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy into LDS may outlive the ring

    if constexpr (F32 && !PLAIN) {  // the token's sums over the four lane groups, in every lane
        sx[0] = sum_lane_groups(s1);
        sxx[0] = sum_lane_groups(s2);
    }
    if constexpr (KH > 1) {  // the KH waves of a row fragment: their partial sums meet in LDS
        f32x4* red = reinterpret_cast<f32x4*>(smem);
        wait_lgkm0();
        block_barrier();
        if (kh > 0) {
            f32x4* r = red + ((kh - 1) * RF + rf) * (NC + 2) * kWave + lane;
#pragma unroll
            for (int q = 0; q < NC; ++q) r[q * kWave] = acc[q];
            r[NC * kWave] = sx;
            r[(NC + 1) * kWave] = sxx;
        }
        __syncthreads();
        if (kh > 0) return;
#pragma unroll
        for (int g = 1; g < KH; ++g) {
            const f32x4* r = red + ((g - 1) * RF + rf) * (NC + 2) * kWave + lane;
#pragma unroll
            for (int q = 0; q < NC; ++q) acc[q] += r[q * kWave];
            sx += r[NC * kWave];
            sxx += r[(NC + 1) * kWave];
        }
    }

    // Epilogue: the lane's token r, features 4G .. 4G + 3 of each block.  Every row of sx holds
    // the token's sum; the Gram diagonal (r, r) sits in lane r + 16 (r >> 2), element r & 3.
    const int r = rf * 16 + i16;
    if (rf * 16 >= M) return;
    float mean = 0.f, rstd = 1.f;
    if constexpr (!PLAIN) {
        const int src = i16 + 16 * (i16 >> 2);
        const float d0 = __shfl(sxx[0], src), d1 = __shfl(sxx[1], src), d2 = __shfl(sxx[2], src),
                    d3 = __shfl(sxx[3], src);
        const float dd = F32 ? sxx[0] : (i16 & 2) ? ((i16 & 1) ? d3 : d2) : ((i16 & 1) ? d1 : d0);
        mean = rms ? 0.f : sx[0] / (float)K;
        rstd = rstd_from_moments(dd / (float)K, mean, eps);
        const int64_t row = m0 + min(r, M - 1);
        if (row_stats) {  // serial ablation (the moment products above are then unused)
            mean = row_stats[2 * row];
            rstd = row_stats[2 * row + 1];
        }
        if (stats_out && nb0 == 0 && G == 0 && r < M) {  // the first column group exports them
            stats_out[2 * row] = mean;
            stats_out[2 * row + 1] = rstd;
        }
    }
    constexpr int NOUT = SW ? NC / 2 : NC;
#pragma unroll
    for (int j = 0; j < NOUT; ++j) {
        const int64_t nb = nb0 + (SW ? 2 * j : j);  // packed column block (gate)
        if (nb >= nblocks) break;
        const int64_t o = (SW ? nb / 2 : nb) * 16 + 4 * G;  // the lane's first output column
        const int64_t ncol = SW ? n_out : N;
        if (r >= M || o >= ncol) continue;  // ncol % 8 == 0: 4 columns are in or out together
        float v[4];
        if constexpr (PLAIN) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[j][e] + (bias ? to_f32<T>(bias[o + e]) : 0.f);
        } else {
            const int64_t pc = nb * 16 + 4 * G;
            const f32x4 cg = *reinterpret_cast<const f32x4*>(c_col + pc), bg = *reinterpret_cast<const f32x4*>(b_col + pc);
            const int q0 = SW ? 2 * j : j;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = __builtin_fmaf(rstd, __builtin_fmaf(-mean, cg[e], acc[q0][e]), bg[e]);
            if constexpr (SW) {
                const f32x4 cu = *reinterpret_cast<const f32x4*>(c_col + pc + 16),
                            bu = *reinterpret_cast<const f32x4*>(b_col + pc + 16);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] = silu(v[e]) * __builtin_fmaf(rstd, __builtin_fmaf(-mean, cu[e], acc[q0 + 1][e]), bu[e]);
            }
        }
        T* dst = out + (m0 + r) * ncol + o;
        if constexpr (F32) {
            *reinterpret_cast<f32x4*>(dst) = f32x4{v[0], v[1], v[2], v[3]};
        } else {
            uint2 st;
            st.x = pack_bf16(v[0], v[1]);
            st.y = pack_bf16(v[2], v[3]);
            *reinterpret_cast<uint2*>(dst) = st;
        }
    }
}

// Ring depths: both as deep as 156 KiB of LDS allow.  A CU's loads return in the order they
// were issued, so x, which L2 holds, waits behind W' from HBM and needs the same time ahead.
template <int RF, int KH, int NC>
struct SkinnyRings {
    static constexpr int ch = KH < 2 ? 2 : KH;
    static constexpr int depth = 156 / ((RF + NC) * ch);
    static constexpr int nxs = depth > 16 ? 16 : depth, nws = nxs;
};

enum class Skinny { kLinear, kSwiGlu, kPlain };
template <class T, int RF, int KH, int NC, Skinny KIND>
static hipError_t run_skinny_kernel(const SkinnyArgs& a, hipStream_t s) {
    using R = SkinnyRings<RF, KH, NC>;
    const int64_t nrb = (a.M + 16 * RF - 1) / (16 * RF), ncg = (a.nblocks + NC - 1) / NC;
    ln_skinny_kernel<T, RF, KH, NC, R::nxs, R::nws, KIND == Skinny::kSwiGlu, KIND == Skinny::kPlain>
        <<<dim3((unsigned)(nrb * ncg)), RF * KH * kWave, 0, s>>>(
            (const T*)a.x, (const char*)a.W, a.kchunks, a.nblocks, a.c_col, a.b_col, a.M, a.K, a.N, a.eps, a.rms,
            a.n_out, a.row_stats, a.stats_out, (T*)a.out, (const T*)a.bias, (int)nrb);
    return hipGetLastError();
}
}  // namespace dn
