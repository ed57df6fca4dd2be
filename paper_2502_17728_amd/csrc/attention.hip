// attention.hip -- deferred Softmax -> P.V with the scores formed in the
// kernel from Q and K (Eq. (8) carried past the paper's operation boundary):
//
//   out_i = (1 / l_i) * sum_j exp(s_ij - m_i) V_j,   s_ij = scale * q_i . k_j,
//
// the numerators feeding the matrix core un-normalized, the row maximum kept
// online and the row sum reduced alongside, one division in the epilogue.  S
// never exists in memory, so the work is the two products on the MFMA instead
// of a stream of scores from HBM.
//
// Orientation.  Both products are taken transposed so that every lane keeps
// one query: S^T = K . Q^T (A = K fragments from LDS, B = the wave's Q
// fragments, held in registers for the whole kernel) and out^T = V^T . P~^T
// (A = V^T from LDS, B = the numerators).  A 16x16 S^T block leaves lane
// (i, G) (i = lane & 15, G = lane >> 4) the scores of query i against keys
// 4G .. 4G+3 of the block.  Two adjacent blocks therefore give the lane 8
// scores -- keys 4G..4G+3 and 16+4G..16+4G+3 of a 32-key chunk -- which is
// exactly one B-operand fragment of the P~ . V product once the keys of that
// product are taken in the same order; the V^T fragments are read with that
// key order, so no score ever moves between lanes.  The maximum over a
// query's keys needs one exchange across the four lane groups; the row sum is
// one more MFMA per chunk with A = all ones.
//
// Data movement.  K and V tiles ([keys][d], row-major) go through rings in LDS filled by
// global->LDS copies of whole KiB; 16-byte pieces are XOR-swizzled per key row so that the K
// fragment reads (16 rows at one piece) and the transposing V^T reads (ds_read_b64_tr_b16)
// are free of bank conflicts.  Causal: key steps wholly above the workgroup's queries are
// never read; a wave skips the products of steps wholly above its own queries; keys above
// the diagonal inside a step are masked to -inf before the exponentials.
//
// Prefill (attention_prefill_kernel).  Bound by the matrix cores and by the power they and
// the exponentials draw: causal 32 x 8192, d = 128 runs the pipe 68 % busy at 1.92 GHz (54.6 % at
// 2.03 GHz before the two halves of a workgroup ran out of phase), 434 us against 507 us in one
// run; 4096 keys without a mask 215 us against 235 us.
//
// Decode (a few new queries against a long key/value cache): attention_kernel below.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "dn_device.hpp"
#include "dn_launch.hpp"
#include "launch_rules.hpp"

namespace dn {
namespace fa {
constexpr float kLog2e = 1.4426950408889634f;

template <int N>
__device__ __forceinline__ void wait_vmcnt_asm() {
    static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// v_max3_f32 directly; the caller keeps matrix and transcendental results at a distance.
__device__ __forceinline__ float max3f(float a, float b, float c) {
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
// K rows: the A-operand read takes 16 consecutive rows at one 16-byte piece.
// 256-byte rows span all 64 banks, so each of the 16 rows gets its own slot;
// 128-byte rows alternate bank halves, and the 8 rows of a half get 8 slots.
template <int D>
__device__ __forceinline__ int k_swz(int r) {
    if constexpr (D == 128) return r & 15;
    return (r & 7) ^ ((r >> 3) & 1);
}
// V rows: the transposing read is serviced 32 lanes at a time and, in the key
// order above, covers 8 consecutive key rows; the swizzle (an even piece count,
// so 32-byte blocks stay whole) gives each of them its own 32-byte bank window.
template <int D>
__device__ __forceinline__ int v_swz(int r) {
    if constexpr (D == 128) return 2 * (r & 3) + 8 * ((r >> 2) & 1);
    return 4 * ((r >> 1) & 1) + 2 * ((r >> 2) & 1);
}
// Merging partial sums: 2^(m - mn), and w l rounded by itself (not contracted into the addition
// that follows).  Partials whose scores are all -inf (m = -inf) weigh nothing, also while the
// maximum mn of those seen is still -inf.
__device__ __forceinline__ float part_weight(float m, float mn) {
    return m != -__builtin_inff() ? __builtin_amdgcn_exp2f(m - mn) : 0.f;
}
__device__ __forceinline__ float weighted(float w, float l) {
    float t = w * l;
    asm volatile("" : "+v"(t));
    return t;
}
typedef short v4s_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 lds_tr16(const char* p) {
    v4s_t r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DN_LDS v4s_t*)(DN_LDS char*)p);
    return __builtin_bit_cast(uint2, r);
}
}  // namespace fa

// Prefill.  NQW x QW x 16 queries per workgroup; KSP groups of NQW waves walk KSP
// contiguous runs of the key steps, each through its own K and V rings (two slots each),
// and their partial sums are merged in LDS at the end (Eq. (8) over key ranges).
//
// Schedule.  The eight waves sit two to a SIMD.  A step is an exponential phase (mask,
// maximum, numerators, rare rescale: VALU) and a matrix phase (the products of this step
// and the scores of the next: MFMA and LDS reads); the two halves of the workgroup run one
// phase apart, separated by barriers, so that on every SIMD one wave's exponentials run
// beside the other's matrix instructions.  With few key steps (prefill_phased) the phases' start
// and end cost more than they hide, and the halves run in step (PHASED false).
template <int D, int NQW, int QW, int KSP, int BKV, bool PHASED>
__global__ __launch_bounds__(NQW* KSP * 64) void attention_prefill_kernel(
    const __bf16* __restrict__ Q, const __bf16* __restrict__ K, const __bf16* __restrict__ V, int64_t Lq, int64_t Lk,
    int causal, float sl2, int nqb, __bf16* __restrict__ out, int group) {
    using namespace fa;
    constexpr int NW = NQW * KSP;
    constexpr int BQ = NQW * QW * 16;  // queries per workgroup
    constexpr int NKB = BKV / 16;      // 16-key S^T blocks per step
    constexpr int NKC = BKV / 32;      // 32-key chunks of the P.V product per step
    constexpr int ROW = D * 2;         // bytes per K or V row
    constexpr int TILE = BKV * ROW;    // one K (or V) slot
    constexpr int RING = 4 * TILE;     // a key group's rings: K slots 0, 1, V slots 0, 1
    constexpr int CW = NQW < NW / 2 ? NQW : NW / 2;  // late waves that share a tile's copies
    constexpr int NG = KSP * CW / (NW / 2);          // key groups whose tiles a late wave copies
    constexpr int T_INS = TILE / kChunkBytes / CW;   // copies per late wave per tile
    constexpr int PPR = ROW / 16;      // 16-byte pieces per row
    constexpr int RPI = kChunkBytes / ROW;  // rows per copy instruction
    constexpr int DB = D / 16, DC = D / 32;
    static_assert(TILE % (kChunkBytes * CW) == 0 && KSP % NG == 0, "copies split evenly over the late waves");
    static_assert(NW % 2 == 0, "two halves");
    static_assert(PHASED || KSP == 1, "in step: nothing follows the last step's reads");
    constexpr int XCH = (KSP - 1) * NQW * 64 * QW * (DB + 1) * 16;  // merge exchange
    constexpr int SMEM = KSP * RING > XCH ? KSP * RING : XCH;

    __shared__ __attribute__((aligned(1024))) char smem[SMEM];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qg = wave % NQW, kg = wave / NQW;
    const bool late = wave >= NW / 2;  // the half that runs one phase behind
    // causal: all heads' longest query blocks first; else whole heads in a row on each XCD
    int h, qb;
    if (causal) {
        longest_first(blockIdx.x, nqb, gridDim.x / nqb, h, qb);
    } else {
        const int t = xcd_contiguous(blockIdx.x, gridDim.x);
        h = t / nqb;
        qb = t % nqb;
    }
    const int64_t q0 = (int64_t)qb * BQ;
    const int kv_end = (int)(causal ? min(Lk, q0 + BQ) : Lk);
    // every group walks nsteps steps from its first key on; steps past kv_end are masked
    const int nsteps = ((kv_end + BKV - 1) / BKV + KSP - 1) / KSP;
    const int k_lo = kg * nsteps * BKV;

    const __bf16* Qh = Q + (int64_t)h * Lq * D;
    // grouped-query attention: query head h reads key/value head h / group
    const __bf16* Kh = K + (int64_t)(h / group) * Lk * D;
    const __bf16* Vh = V + (int64_t)(h / group) * Lk * D;
    __bf16* Oh = out + (int64_t)h * Lq * D;

    const int qw0 = (int)q0 + qg * QW * 16;  // first query of this wave (positions fit 32 bits)
    const int G = lane >> 4, i = lane & 15;
    int qrow[QW];
#pragma unroll
    for (int f = 0; f < QW; ++f) qrow[f] = qw0 + f * 16 + i;

    // ---- K/V rings.  The late half issues every copy, at the start of its exponential phase,
    // which has issue slots to spare; each of its waves copies T_INS KiB of the K and V tiles
    // of NG key groups.  Copy instruction j covers tile rows RPI * (cw + j * CW) ..; lane l
    // fetches piece (l % PPR) ^ swz(row), so logical piece p of a row lands in slot p ^ swz(row)
    // (the swizzles repeat every 16 rows, PJ instructions).  Keys past Lk clamp onto the last
    // row (their scores are masked); byte offsets from the head's base fit 32 bits
    // (Lk * d * 2 < 2^31).
    constexpr int PJ = CW * RPI >= 16 ? 1 : 16 / (CW * RPI);
    const int cw = wave % CW, cg = kg % (KSP / NG);  // this wave's share of a tile, its first key group
    const int c_row = cw * RPI + lane / PPR;
    uint32_t k_off[PJ], v_off_g[PJ];
#pragma unroll
    for (int j = 0; j < PJ; ++j) {
        const int r = c_row + j * CW * RPI;
        k_off[j] = (uint32_t)(c_row * ROW + ((lane % PPR) ^ k_swz<D>(r)) * 16);
        v_off_g[j] = (uint32_t)(c_row * ROW + ((lane % PPR) ^ v_swz<D>(r)) * 16);
    }
    const uint64_t k_base = uniform_u64(Kh), v_base = uniform_u64(Vh);
    const uint32_t smem_addr = lds_addr32(smem);
    // K (which = 0) or V (which = 1) of `step` of the wave's key groups
    auto issue = [&](int which, int step) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int gg = cg + g * (KSP / NG);
            const uint32_t base = smem_addr + (uint32_t)(gg * RING + (2 * which + (step & 1)) * TILE + cw * kChunkBytes);
            const uint32_t k0 = (uint32_t)((gg * nsteps + step) * BKV);
            if (k0 + BKV <= (uint32_t)Lk) {  // no row to clamp: the step's offset goes into the scalar base
                const uint64_t src = (which ? v_base : k_base) + (uint64_t)k0 * ROW;
#pragma unroll
                for (int j = 0; j < T_INS; ++j)
                    g2lds16_async_sb(src + (uint64_t)(j * CW * kChunkBytes), which ? v_off_g[j % PJ] : k_off[j % PJ],
                                     base + (uint32_t)(j * CW * kChunkBytes));
            } else {
                const uint32_t last = (uint32_t)(Lk - 1);
#pragma unroll
                for (int j = 0; j < T_INS; ++j) {
                    const uint32_t piece = (which ? v_off_g[j % PJ] : k_off[j % PJ]) - (uint32_t)(c_row * ROW);
                    const uint32_t row = k0 + (uint32_t)(c_row + j * CW * RPI);
                    const uint32_t key = row < last ? row : last;  // a select, no branch
                    g2lds16_async_sb(which ? v_base : k_base, key * (uint32_t)ROW + piece,
                                     base + (uint32_t)(j * CW * kChunkBytes));
                }
            }
        }
    };
    if (late) {
        issue(0, 0);
        if (PHASED && nsteps > 1) issue(0, 1);
        issue(1, 0);
    }

    // Q^T fragments (B operand of S^T): lane (i, G) holds query 16f + i, d 32c + 8G .. +8.
    // The empty statements make the compiler place its waits for these loads here and not
    // inside the key loop, where they would also drain the copies in flight.
    u32x4 qf[QW][DC];
#pragma unroll
    for (int f = 0; f < QW; ++f) {
        const int64_t qr = qrow[f] < Lq ? qrow[f] : Lq - 1;
#pragma unroll
        for (int c = 0; c < DC; ++c) qf[f][c] = ld16(Qh + qr * D + 32 * c + 8 * G);
    }
#pragma unroll
    for (int f = 0; f < QW; ++f)
#pragma unroll
        for (int c = 0; c < DC; ++c) asm volatile("" : "+v"(qf[f][c]));

    // Lane-constant LDS offsets.  K: row 16 kb + i, logical piece 4c + G (the swizzle depends on
    // the row only through i).  V^T: two transposing reads per 16-wide d block, the first
    // covering keys 4G .. 4G+3 of the chunk, the second keys 16+4G .. 16+4G+3 (within a 16-lane
    // group, lane j, slot t gets element j & 3 of the 8 bytes lane 4t + (j >> 2) reads, so lane
    // (i, G) reads row 4G + (i >> 2), d 4 (i & 3) .. +3 of the block).
    int k_rd[DC];
#pragma unroll
    for (int c = 0; c < DC; ++c) k_rd[c] = i * ROW + (((4 * c + G) ^ k_swz<D>(i)) << 4);
    const int vr = 4 * G + (i >> 2);
    const int vsw2 = v_swz<D>(vr) >> 1;  // swizzle of the 32-byte d block
    int v_off[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) v_off[b] = vr * ROW + (i & 3) * 8 + 32 * (b ^ vsw2);

    f32x4 acc[QW][DB], accl[QW];
#pragma unroll
    for (int f = 0; f < QW; ++f) {
#pragma unroll
        for (int b = 0; b < DB; ++b) acc[f][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        accl[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    // Reference maximum per query in scaled log2 units, raised only when a step exceeds it
    // by more than 8 (numerators stay below 256; the rescale, an exact identity, is rare).
    float mref[QW];
#pragma unroll
    for (int f = 0; f < QW; ++f) mref[f] = -__builtin_inff();

    // the wave's steps: those not wholly above its queries
    const int qlast = qw0 + QW * 16 - 1;
    const int n_w = causal ? (qlast >= k_lo ? min(nsteps, (qlast - k_lo) / BKV + 1) : 0) : nsteps;
    const char* kring = smem + kg * RING;
    const char* vring = kring + 2 * TILE;

    f32x4 st[QW][NKB];  // scores S^T of one step
    u32x4 pf[QW][NKC];  // numerators of one step, bf16

    // Matrix phase.  The fragments are read from LDS one group ahead of their products --
    // a 32-key chunk of V^T (2 DB transposing reads) beside the products of the chunk before,
    // a pair of K blocks (2 DC reads) beside the pair before -- in an order fixed by scheduling
    // groups: left to itself the compiler reads two MFMAs ahead, less than the LDS latency,
    // and with one wave per SIMD in this phase nothing else covers it.
    auto read_v = [&](const char* vb, int kc, u32x4(&vf)[DB]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            const uint2 lo = lds_tr16(vb + v_off[b] + (kc * 32) * ROW);
            const uint2 hi = lds_tr16(vb + v_off[b] + (kc * 32 + 16) * ROW);
            vf[b] = u32x4{lo.x, lo.y, hi.x, hi.y};
        }
    };
    auto read_k = [&](const char* kb, int j, u32x4(&kf)[2][DC]) __attribute__((always_inline)) {  // key blocks 2j, 2j + 1
#pragma unroll
        for (int c = 0; c < DC; ++c)
#pragma unroll
            for (int b = 0; b < 2; ++b) kf[b][c] = lds_ld16(lds_ptr((char*)kb + (2 * j + b) * 16 * ROW + k_rd[c]));
    };
    // out^T += V^T . P~^T of `step` (if PV), then S^T = K . Q^T of step + 1 (if QK)
    auto matrix = [&](int step, auto do_pv, auto do_qk) __attribute__((always_inline)) {
        constexpr bool PV = decltype(do_pv)::value, QK = decltype(do_qk)::value;
        const char* vb = vring + (step & 1) * TILE;
        const char* kb = kring + ((step + 1) & 1) * TILE;
        u32x4 vf[2][DB], kf[2][2][DC];
        if constexpr (PV) {
            read_v(vb, 0, vf[0]);
            // the row sums need no fragment from LDS: they cover the latency of the first reads
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
                for (int f = 0; f < QW; ++f) accl[f] = mfma_chunk<__bf16>(ones, pf[f][kc], accl[f]);
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc) {
                if (kc + 1 < NKC) read_v(vb, kc + 1, vf[(kc + 1) & 1]);
                if (QK && kc + 1 == NKC) read_k(kb, 0, kf[0]);
#pragma unroll
                for (int b = 0; b < DB; ++b)
#pragma unroll
                    for (int f = 0; f < QW; ++f) acc[f][b] = mfma_chunk<__bf16>(vf[kc & 1][b], pf[f][kc], acc[f][b]);
            }
        } else {
            read_k(kb, 0, kf[0]);
        }
        if constexpr (QK) {
#pragma unroll
            for (int f = 0; f < QW; ++f)
#pragma unroll
                for (int b4 = 0; b4 < NKB; ++b4) st[f][b4] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NKC; ++j) {
                if (j + 1 < NKC) read_k(kb, j + 1, kf[(j + 1) & 1]);
#pragma unroll
                for (int c = 0; c < DC; ++c)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int f = 0; f < QW; ++f)
                            st[f][2 * j + b] = mfma_chunk<__bf16>(kf[j & 1][b][c], qf[f][c], st[f][2 * j + b]);
            }
        }
        // the order of the reads and products above
        if constexpr (PV) {
            __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2 * DB, 0);
            __builtin_amdgcn_sched_group_barrier(kSgMfma, NKC * QW, 0);
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc) {
                constexpr int NM = QW * DB;
                const int nd = kc + 1 < NKC ? 2 * DB : (QK ? 2 * DC : 0);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 0);
                    const int r = nd * (m + 1) / NM - nd * m / NM;
                    if (r == 1) __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 0);
                    if (r == 2) __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2, 0);
                }
            }
        } else {
            __builtin_amdgcn_sched_group_barrier(kSgDsRead, 2 * DC, 0);
        }
        if constexpr (QK) {
#pragma unroll
            for (int j = 0; j < NKC; ++j) {
                constexpr int NM = QW * 2 * DC;
                const int nd = j + 1 < NKC ? 2 * DC : 0;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 0);
                    const int r = nd * (m + 1) / NM - nd * m / NM;
                    if (r == 1) __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 0);
                }
            }
        }
    };
    auto numerators = [&](int step) __attribute__((always_inline)) {
        const int k0 = k_lo + step * BKV;
        if ((causal && k0 + BKV - 1 > qw0) || k0 + BKV > kv_end) {
#pragma unroll
            for (int f = 0; f < QW; ++f) {
                const int lim = causal ? min(qrow[f], kv_end - 1) : kv_end - 1;
#pragma unroll
                for (int b4 = 0; b4 < NKB; ++b4) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (k0 + 16 * b4 + 4 * G + e > lim) st[f][b4][e] = -__builtin_inff();
                    // one block's compare masks at a time: issued all at once they
                    // took 64 SGPRs and pushed loop-long scalars into VGPR lanes
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // The maxima go through v_max3_f32 in inline assembly (fmaxf on matrix results gets an
        // extra canonicalizing max per operand), which the compiler's hazard pass does not
        // guard: 20 wait states cover the longest matrix-result-to-VALU distance.
#pragma unroll
        for (int f = 0; f < QW; ++f)
#pragma unroll
            for (int b4 = 0; b4 < NKB; ++b4) {
                if (f == 0 && b4 == 0)
                    asm volatile("s_nop 15\n\ts_nop 3" : "+v"(st[f][b4]));
                else
                    asm volatile("" : "+v"(st[f][b4]));
            }
        float tmax[QW];
        bool want = false;
#pragma unroll
        for (int f = 0; f < QW; ++f) {
            float m2[NKB];
#pragma unroll
            for (int b4 = 0; b4 < NKB; ++b4)
                m2[b4] = max3f(max3f(st[f][b4][0], st[f][b4][1], st[f][b4][2]), st[f][b4][3],
                               b4 >= NKB / 2 ? m2[b4 - NKB / 2] : st[f][b4][3]);
            tmax[f] = m2[NKB / 2];
#pragma unroll
            for (int b4 = NKB / 2 + 1; b4 + 1 < NKB; b4 += 2) tmax[f] = max3f(tmax[f], m2[b4], m2[b4 + 1]);
            if constexpr (NKB / 2 % 2 == 0) tmax[f] = max3f(tmax[f], m2[NKB - 1], m2[NKB - 1]);
            want |= tmax[f] * sl2 > mref[f] + 8.0f;
        }
        // a query's reference rises exactly when one of its four lanes' own maxima exceeds it
        // by more than 8 (the scale is positive), so the cross-lane maximum is formed, and the
        // partial sums rescaled, only in the rare steps where some lane asks for it
        if (__any(want)) {
#pragma unroll
            for (int f = 0; f < QW; ++f) {
                const float tmax2 = max_lane_groups(tmax[f]) * sl2;
                const bool raise = tmax2 > mref[f] + 8.0f;
                const float mnew = raise ? tmax2 : mref[f];
                const float alpha = __builtin_amdgcn_exp2f(raise ? mref[f] - mnew : 0.f);
                mref[f] = mnew;
#pragma unroll
                for (int b = 0; b < DB; ++b) acc[f][b] *= alpha;
                accl[f] *= alpha;
            }
        }
#pragma unroll
        for (int f = 0; f < QW; ++f) {
            const float nb = mref[f] == -__builtin_inff() ? 0.f : -mref[f];
            float p[NKB][4];
#pragma unroll
            for (int b4 = 0; b4 < NKB; ++b4)
#pragma unroll
                for (int e = 0; e < 4; ++e) p[b4][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[f][b4][e], sl2, nb));
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc)
                pf[f][kc] = u32x4{pack_bf16(p[2 * kc][0], p[2 * kc][1]), pack_bf16(p[2 * kc][2], p[2 * kc][3]),
                                  pack_bf16(p[2 * kc + 1][0], p[2 * kc + 1][1]),
                                  pack_bf16(p[2 * kc + 1][2], p[2 * kc + 1][3])};
        }
    };
    // Phases: the early half runs the exponentials of step s in phase 2s and its matrix work
    // in phase 2s + 1, the late half one phase later.  K(s+1) and V(s) are read in phases
    // 2s + 1 and 2s + 2; their slots take K(s+3) and V(s+2), issued in phase 2s + 3 and
    // waited for (each wave its own copies) before the barrier that ends phase 2s + 4.
    // In step (not PHASED): K(s+1) and V(s+1) land beside step s, in the slots step s - 1 left.
    using yes = std::true_type;
    using no = std::false_type;
    if constexpr (PHASED) {
        wait_vmcnt_asm<0>();
        block_barrier();
        if (late) block_barrier();
        if (n_w > 0) matrix(-1, no{}, yes{});
        wait_lgkm0();
        block_barrier();
        auto step = [&](int s, auto work, auto next) __attribute__((always_inline)) {  // work: the wave's own step; next: not its last
            if (late) {  // nothing past the last step (tested past the loop: inside, K of one step more costs less)
                if (decltype(next)::value || s + 2 < nsteps) issue(0, s + 2);
                if (decltype(next)::value || s + 1 < nsteps) issue(1, s + 1);
            }
            if constexpr (decltype(work)::value) {
                numerators(s);
                // used here, so that the exponentials are not sunk past the barrier
#pragma unroll
                for (int f = 0; f < QW; ++f)
#pragma unroll
                    for (int kc = 0; kc < NKC; ++kc) asm volatile("" : "+v"(pf[f][kc]));
            }
            block_barrier();
            if constexpr (decltype(work)::value) {
                __builtin_amdgcn_s_setprio(1);
                matrix(s, yes{}, next);
                __builtin_amdgcn_s_setprio(0);
            }
            if (late) wait_vmcnt_asm<0>();
            wait_lgkm0();
            block_barrier();
        };
        int s = 0;
        for (; s < n_w - 1; ++s) step(s, yes{}, yes{});
        if (s < n_w) {
            step(s, yes{}, no{});
            ++s;
        }
        for (; s < nsteps; ++s) step(s, no{}, no{});
        if (!late) block_barrier();
    } else {
        for (int s = 0; s < nsteps; ++s) {
            wait_vmcnt_asm<0>();  // this wave's copies of step s have landed
            wait_lgkm0();         // its reads of step s - 1, whose slots the next copies take, are done
            block_barrier();      // ... and every wave's
            if (late && s + 1 < nsteps) {
                issue(0, s + 1);
                issue(1, s + 1);
            }
            if (s < n_w) {
                matrix(s - 1, no{}, yes{});
                numerators(s);
                matrix(s, yes{}, no{});
            }
        }
    }
    wait_vmcnt_asm<0>();  // no copy into LDS may outlive the workgroup

    if constexpr (KSP > 1) {
        // Merge: groups 1 .. leave (acc, l, m) in LDS (the rings are idle now), group 0
        // rescales everything to the largest reference.  A group without any unmasked key
        // has m = -inf and contributes nothing.
        f32x4* xch = reinterpret_cast<f32x4*>(smem);
        block_barrier();  // every wave's copies have landed
        if (kg > 0) {
#pragma unroll
            for (int f = 0; f < QW; ++f) {
                f32x4* x = xch + (((kg - 1) * NQW + qg) * QW + f) * (DB + 1) * 64 + lane;
#pragma unroll
                for (int b = 0; b < DB; ++b) x[b * 64] = acc[f][b];
                x[DB * 64] = f32x4{accl[f][0], mref[f], 0.f, 0.f};
            }
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int f = 0; f < QW; ++f) {
            float m = mref[f];
            float lg[KSP], mg[KSP];
#pragma unroll
            for (int g = 1; g < KSP; ++g) {
                const f32x4 lm = xch[((((g - 1) * NQW + qg) * QW + f) * (DB + 1) + DB) * 64 + lane];
                lg[g] = lm[0];
                mg[g] = lm[1];
                m = mg[g] > m ? mg[g] : m;
            }
            const float a0 = mref[f] == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(mref[f] - m);
#pragma unroll
            for (int b = 0; b < DB; ++b) acc[f][b] *= a0;
            accl[f][0] *= a0;
#pragma unroll
            for (int g = 1; g < KSP; ++g) {
                const float ag = mg[g] == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(mg[g] - m);
                const f32x4* x = xch + (((g - 1) * NQW + qg) * QW + f) * (DB + 1) * 64 + lane;
#pragma unroll
                for (int b = 0; b < DB; ++b) {
                    const f32x4 v = x[b * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[f][b][e] = __builtin_fmaf(v[e], ag, acc[f][b][e]);
                }
                accl[f][0] = __builtin_fmaf(lg[g], ag, accl[f][0]);
            }
        }
    }

    // ---- epilogue: the single deferred division, one rounding to bf16
#pragma unroll
    for (int f = 0; f < QW; ++f) {
        if (qrow[f] >= Lq) continue;
        const float inv = 1.0f / accl[f][0];
        __bf16* orow = Oh + (int64_t)qrow[f] * D + 4 * G;
#pragma unroll
        for (int b = 0; b < DB; ++b) {
            uint2 v;
            v.x = pack_bf16(acc[f][b][0] * inv, acc[f][b][1] * inv);
            v.y = pack_bf16(acc[f][b][2] * inv, acc[f][b][3] * inv);
            *reinterpret_cast<uint2*>(orow + b * 16) = v;
        }
    }
}

template <int D, int NQW, int QW, int KSP, int BKV, bool PHASED = true>
static hipError_t run_attention(const void* Q, const void* K, const void* V, int64_t BH, int64_t Lq, int64_t Lk,
                                int causal, float scale, void* out, hipStream_t s, int group) {
    constexpr int BQ = NQW * QW * 16;
    const int nqb = (int)((Lq + BQ - 1) / BQ);
    attention_prefill_kernel<D, NQW, QW, KSP, BKV, PHASED><<<dim3((unsigned)(BH * nqb)), NQW * KSP * 64, 0, s>>>(
        (const __bf16*)Q, (const __bf16*)K, (const __bf16*)V, Lq, Lk, causal, scale * fa::kLog2e, nqb,
        (__bf16*)out, group);
    return hipGetLastError();
}

// Decode: up to 16 query rows per head against all keys.  The keys of all heads, in units of
// 128, are dealt in order to at most one resident round of W workgroups, ceil(units / W) to each
// and the rest to the last, so a workgroup takes a run of units that may end one head and begin
// the next, and none has more than an even share rounded up.  Where that rounding is coarse,
// places stay empty: 17 heads x 1992 keys, 272 units, are 136 workgroups of 2 on 256 places.
//
// The four waves of a workgroup take 32 keys of each unit and stream them through K/V rings of
// their own (two slots, no barrier; four waves keep up to 128 KiB in flight, one wave's counter
// 63 KiB).  At the end of a head's run the waves' (acc, l, m) meet in LDS.  A head whose keys
// one workgroup read whole is divided and written; otherwise the workgroup leaves its partial
// sums in the workspace and a merge kernel combines the head's partials in key order -- Eq. (8)
// over key ranges, m = max_g m_g, out = sum_g 2^(m_g - m) acc_g / sum_g 2^(m_g - m) l_g.  (The
// last workgroup of a head to arrive combining them instead, with no second launch, measured the
// same or slower: its waits for device-scope stores and loads cost what the launch does, and up
// to 33 against 18 us where 32 workgroups share a head.)
//
// Bound by HBM.  Against one single-wave workgroup per equal range of each head (graph replays,
// us): 177 heads x 11814 keys, d = 128 170 / 212 (that left a second round of 98 workgroups),
// 300 x 1000 31 / 42, 17 x 1992 11.6 / 22.6, 64 x 5001 32 / 34, 37 x 7242, d = 64 19.6 / 23.9;
// 256 x 8192, where every workgroup has one whole head, 156 / 154 (6.9 TB/s).
struct DecodeArgs {
    int64_t BH;
    int Lq, Lk;
    int units;       // per head, of 128 keys
    int per;         // units per workgroup
    int nsplit;      // > 0: every head in nsplit runs of `per` units, one workgroup each (a
                     // workspace of the size that layout needs); 0: runs across heads
    float sl2;

    // The head's partials lie in a row from slot first_slot on: h + wg where a head spans several
    // workgroups, 2 wg + .. where a workgroup spans heads (then a split head has two parts).
    __device__ int first_wg(int h) const { return nsplit ? 0 : (int)((int64_t)h * units / per); }
    __device__ int64_t first_slot(int h, int f) const {
        return nsplit ? (int64_t)h * nsplit : per >= units ? 2 * (int64_t)f : (int64_t)h + f;
    }
    __device__ int parts(int h, int f) const {
        return nsplit ? nsplit : (int)((((int64_t)h + 1) * units - 1) / per) - f + 1;
    }
};
// ONE_PASS: a workgroup per head and no partials in memory -- where the deal cuts a head in two
// (heads enough to fill the chip are cut no further), the workgroup takes both runs and combines
// their sums in registers, in the merge kernel's arithmetic, so the output is the same bit for bit.
template <int D, bool ONE_PASS>
__global__ __launch_bounds__(256) void attention_kernel(const __bf16* __restrict__ Q,
                                                               const __bf16* __restrict__ K,
                                                               const __bf16* __restrict__ V, DecodeArgs p,
                                                               float* __restrict__ part, __bf16* __restrict__ out) {
    using namespace fa;
    constexpr int ROW = D * 2, TILE = 32 * ROW, SLOT = 2 * TILE;  // 32 keys of K, then V
    constexpr int INS = TILE / kChunkBytes;                       // copies per tile
    constexpr int PPR = ROW / 16, RPI = kChunkBytes / ROW;
    constexpr int DB = D / 16, DC = D / 32;
    constexpr int PR = D + 4;  // floats per partial row: acc[d], l, m and 2 pad floats
    __shared__ __attribute__((aligned(1024))) char smem[4 * 2 * SLOT];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = lane >> 4, i = lane & 15;
    const int wg = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t total = p.BH * p.units;
    int64_t pos = ONE_PASS   ? (int64_t)wg * p.units
                  : p.nsplit ? (int64_t)(wg / p.nsplit) * p.units + (int64_t)(wg % p.nsplit) * p.per
                             : (int64_t)wg * p.per;
    const int64_t end = ONE_PASS   ? pos + p.units
                        : p.nsplit ? min((int64_t)(wg / p.nsplit + 1) * p.units, pos + p.per)
                                   : min(total, pos + p.per);

    // copies: instruction j covers rows RPI j .. of the tile, piece (l % PPR) ^ swz(row)
    const int c_row = lane / PPR;
    constexpr int PJ = RPI >= 16 ? 1 : 16 / RPI;  // the swizzles repeat every 16 rows
    uint32_t k_off[PJ], v_offg[PJ];
#pragma unroll
    for (int j = 0; j < PJ; ++j) {
        k_off[j] = (uint32_t)(((lane % PPR) ^ k_swz<D>(c_row + j * RPI)) * 16);
        v_offg[j] = (uint32_t)(((lane % PPR) ^ v_swz<D>(c_row + j * RPI)) * 16);
    }
    char* ring = smem + wave * 2 * SLOT;
    const uint32_t ring_addr = lds_addr32(ring);
    const uint32_t last = (uint32_t)(p.Lk - 1);
    int k_rd[DC], v_off[DB];
#pragma unroll
    for (int c = 0; c < DC; ++c) k_rd[c] = i * ROW + (((4 * c + G) ^ k_swz<D>(i)) << 4);
    const int vr = 4 * G + (i >> 2);
#pragma unroll
    for (int b = 0; b < DB; ++b) v_off[b] = vr * ROW + (i & 3) * 8 + 32 * (b ^ (v_swz<D>(vr) >> 1));
    const u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    f32x4 v1[DB / 4];  // ONE_PASS: the sums of a cut head's first run
    float m1 = 0.f, l1 = 0.f;

    while (pos < end) {
        const int h = (int)(pos / p.units), u0 = (int)(pos - (int64_t)h * p.units);
        int u1 = (int)min((int64_t)p.units, u0 + (end - pos));  // this run's units of head h
        if constexpr (ONE_PASS) u1 = (int)min((int64_t)u1, u0 + (p.per - pos % p.per));
        pos += u1 - u0;
        const uint64_t k_base = uniform_u64(K + (int64_t)h * p.Lk * D), v_base = uniform_u64(V + (int64_t)h * p.Lk * D);
        // the wave's 32 keys of unit u; steps wholly past Lk are none of its work
        const int kw0 = u0 * 128 + wave * 32;
        const int n_w = kw0 < p.Lk ? min(u1 - u0, (p.Lk - 1 - kw0) / 128 + 1) : 0;
        auto issue = [&](int s) __attribute__((always_inline)) {
            const uint32_t dst = ring_addr + (uint32_t)((s & 1) * SLOT);
            const uint32_t k0 = (uint32_t)(kw0 + s * 128 + c_row);
#pragma unroll
            for (int j = 0; j < INS; ++j) {
                const uint32_t key = min(k0 + j * RPI, last) * (uint32_t)ROW;
                g2lds16_stream_sb(k_base, key + k_off[j % PJ], dst + (uint32_t)(j * kChunkBytes));
            }
#pragma unroll
            for (int j = 0; j < INS; ++j) {
                const uint32_t key = min(k0 + j * RPI, last) * (uint32_t)ROW;
                g2lds16_stream_sb(v_base, key + v_offg[j % PJ], dst + (uint32_t)(TILE + j * kChunkBytes));
            }
        };
        // The first step's copies, then Q: the compiler's wait for Q (placed here by the empty
        // statements, not in the key loop) also waits for that step, which is needed first anyway.
        if (n_w > 0) issue(0);
        const __bf16* Qh = Q + (int64_t)h * p.Lq * D;
        u32x4 qf[DC];
#pragma unroll
        for (int c = 0; c < DC; ++c) qf[c] = ld16(Qh + (int64_t)min(i, p.Lq - 1) * D + 32 * c + 8 * G);
#pragma unroll
        for (int c = 0; c < DC; ++c) asm volatile("" : "+v"(qf[c]));

        f32x4 acc[DB], accl = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < DB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        float mref = -__builtin_inff();
        for (int s = 0; s < n_w; ++s) {
            wait_lgkm0();  // the reads of step s - 1, whose slot the next copies take
            asm volatile("" ::: "memory");
            issue(s + 1);  // past the last step: a slot that is not read (rows clamped)
            wait_vmcnt_asm<2 * INS>();
            const char* kb = ring + (s & 1) * SLOT;
            f32x4 st[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int c = 0; c < DC; ++c)
#pragma unroll
                for (int b4 = 0; b4 < 2; ++b4)
                    st[b4] = mfma_chunk<__bf16>(lds_ld16(lds_ptr((char*)kb + b4 * 16 * ROW + k_rd[c])), qf[c], st[b4]);
            const int k0 = kw0 + s * 128;
            if (k0 + 32 > p.Lk) {
#pragma unroll
                for (int b4 = 0; b4 < 2; ++b4)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (k0 + 16 * b4 + 4 * G + e >= p.Lk) st[b4][e] = -__builtin_inff();
            }
            float tmax = st[0][0];
#pragma unroll
            for (int b4 = 0; b4 < 2; ++b4)
#pragma unroll
                for (int e = 0; e < 4; ++e) tmax = __builtin_fmaxf(tmax, st[b4][e]);
            // the reference rises only where some lane's own maximum exceeds it by more than 8
            if (__any(tmax * p.sl2 > mref + 8.0f)) {
                const float tmax2 = max_lane_groups(tmax) * p.sl2;
                const bool raise = tmax2 > mref + 8.0f;
                const float mnew = raise ? tmax2 : mref;
                const float alpha = __builtin_amdgcn_exp2f(raise ? mref - mnew : 0.f);
                mref = mnew;
#pragma unroll
                for (int b = 0; b < DB; ++b) acc[b] *= alpha;
                accl *= alpha;
            }
            const float nb = mref == -__builtin_inff() ? 0.f : -mref;
            float e8[8];
#pragma unroll
            for (int b4 = 0; b4 < 2; ++b4)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    e8[4 * b4 + e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[b4][e], p.sl2, nb));
            const u32x4 pf = {pack_bf16(e8[0], e8[1]), pack_bf16(e8[2], e8[3]), pack_bf16(e8[4], e8[5]),
                              pack_bf16(e8[6], e8[7])};
            const char* vb = kb + TILE;
#pragma unroll
            for (int b = 0; b < DB; ++b) {
                const uint2 lo = lds_tr16(vb + v_off[b]), hi = lds_tr16(vb + v_off[b] + 16 * ROW);
                acc[b] = mfma_chunk<__bf16>(u32x4{lo.x, lo.y, hi.x, hi.y}, pf, acc[b]);
            }
            accl = mfma_chunk<__bf16>(ones, pf, accl);
        }
        wait_vmcnt_asm<0>();  // the rings are reused below

        // ---- the four waves' sums: wave w combines d blocks w, w + 4 (all lanes of a query
        // hold its l and m)
        __syncthreads();
        f32x4* xa = reinterpret_cast<f32x4*>(smem);             // [wave][block][lane]
        float* xl = reinterpret_cast<float*>(smem + 4 * DB * 1024);  // [wave][16] l, then m
#pragma unroll
        for (int b = 0; b < DB; ++b) xa[(wave * DB + b) * 64 + lane] = acc[b];
        if (G == 0) {
            xl[wave * 16 + i] = accl[0];
            xl[64 + wave * 16 + i] = mref;
        }
        __syncthreads();
        float m = -__builtin_inff(), l = 0.f, wt[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) m = xl[64 + w * 16 + i] > m ? xl[64 + w * 16 + i] : m;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = xl[64 + w * 16 + i];
            wt[w] = mw == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(mw - m);
            l = __builtin_fmaf(wt[w], xl[w * 16 + i], l);
        }
        const bool whole = u0 == 0 && u1 == p.units;
        const int f = p.first_wg(h);
        float* prow = part + ((p.first_slot(h, f) + (p.nsplit ? u0 / p.per : wg - f)) * p.Lq + i) * PR;
        float a1 = 0.f, a2 = 0.f;  // ONE_PASS, a cut head's second run: weights of the first and of this one
        if (ONE_PASS && u0 > 0) {
            const float mn = __builtin_fmaxf(m1, m);
            a1 = part_weight(m1, mn);
            a2 = part_weight(m, mn);
            l = weighted(a1, l1) + weighted(a2, l);
        }
#pragma unroll
        for (int bb = 0; bb < DB / 4; ++bb) {
            const int b = wave + 4 * bb;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const f32x4 x = xa[(w * DB + b) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(wt[w], x[e], v[e]);
            }
            if constexpr (ONE_PASS) {
                if (u0 > 0)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(a2, v[e], __builtin_fmaf(a1, v1[bb][e], 0.f));
                else
                    v1[bb] = v;
            }
            if (i < p.Lq) {
                if (whole || (ONE_PASS && u0 > 0)) {  // the single deferred division, one rounding to bf16
                    const float inv = 1.0f / l;
                    uint2 o;
                    o.x = pack_bf16(v[0] * inv, v[1] * inv);
                    o.y = pack_bf16(v[2] * inv, v[3] * inv);
                    *reinterpret_cast<uint2*>(out + ((int64_t)h * p.Lq + i) * D + b * 16 + 4 * G) = o;
                } else if constexpr (!ONE_PASS) {
                    *reinterpret_cast<f32x4*>(prow + b * 16 + 4 * G) = v;
                }
            }
        }
        m1 = m;
        l1 = l;
        if (!ONE_PASS && !whole && wave == 0 && G == 0 && i < p.Lq) {
            prow[D] = l;
            prow[D + 1] = m;
        }
        __syncthreads();  // the exchange area is the rings' again
    }
}

// Merge of the split heads' partials, one wave per query row: 64 partials at a time, lane g
// holding partial g's l and m, then every lane D / 64 columns, 8 partials in flight.
template <int D>
__global__ __launch_bounds__(256) void attention_merge_kernel(const float* __restrict__ part, DecodeArgs p,
                                                              __bf16* __restrict__ out) {
    using namespace fa;
    constexpr int PR = D + 4, PER = D / 64;
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= p.BH * p.Lq) return;
    const int h = (int)(row / p.Lq), f = p.first_wg(h), n = p.parts(h, f);
    if (n == 1) return;  // written by the workgroup that read the whole head
    const int64_t stride = (int64_t)p.Lq * PR;  // between the head's partials
    const float* pr = part + (p.first_slot(h, f) * p.Lq + row % p.Lq) * PR;
    float m = -__builtin_inff(), l = 0.f, acc[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) acc[j] = 0.f;
    for (int g0 = 0; g0 < n; g0 += 64, pr += 64 * stride) {
        const int ng = min(64, n - g0);
        const float* mine = pr + min(lane, ng - 1) * stride + D;
        const float lg = mine[0], mg = mine[1];
        float mn = mg;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mn = __builtin_fmaxf(mn, __shfl_xor(mn, o));
        mn = __builtin_fmaxf(m, mn);
        const float w = lane < ng ? part_weight(mg, mn) : 0.f;
        const float old = part_weight(m, mn);
        l = __builtin_fmaf(l, old, wave_sum(weighted(w, lg)));
        m = mn;
#pragma unroll
        for (int j = 0; j < PER; ++j) acc[j] *= old;
        for (int g = 0; g < ng; g += 8) {
            float x[8][PER];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int j = 0; j < PER; ++j) x[k][j] = pr[min(g + k, ng - 1) * stride + lane + 64 * j];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float wk = __shfl(w, min(g + k, 63));
                if (g + k < ng)
#pragma unroll
                    for (int j = 0; j < PER; ++j) acc[j] = __builtin_fmaf(wk, x[k][j], acc[j]);
            }
        }
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int j = 0; j < PER; ++j) out[row * D + lane + 64 * j] = (__bf16)(acc[j] * inv);
}

template <int D>
static hipError_t run_decode(const void* Q, const void* K, const void* V, const DecodeArgs& a, int64_t wgs, bool split,
                             void* part, void* out, hipStream_t s) {
    if (part)
        attention_kernel<D, false><<<dim3((unsigned)wgs), 256, 0, s>>>((const __bf16*)Q, (const __bf16*)K,
                                                                       (const __bf16*)V, a, (float*)part, (__bf16*)out);
    else
        attention_kernel<D, true><<<dim3((unsigned)a.BH), 256, 0, s>>>((const __bf16*)Q, (const __bf16*)K,
                                                                       (const __bf16*)V, a, nullptr, (__bf16*)out);
    if (part && split)
        attention_merge_kernel<D><<<dim3((unsigned)((a.BH * a.Lq + 3) / 4)), 256, 0, s>>>((const float*)part, a,
                                                                                          (__bf16*)out);
    return hipGetLastError();
}

hipError_t launch_attention_decode(const void* Q, const void* K, const void* V, int64_t BH, int64_t Lq, int64_t Lk,
                                   int64_t d, float scale, void* workspace, size_t workspace_bytes, void* out,
                                   hipStream_t s) {
    const DecodePlan plan = decode_plan(BH, Lk, d);
    DecodeArgs a{};
    a.BH = BH;
    a.Lq = (int)Lq;
    a.Lk = (int)Lk;
    a.units = (int)plan.units;
    a.sl2 = scale * fa::kLog2e;
    int64_t wgs = plan.wgs;
    a.per = (int)plan.per;
    a.nsplit = plan.nsplit;
    bool split = plan.slots > 0;
    if (slots_bytes(plan.slots, Lq, d) > workspace_bytes) {
        int64_t per;
        a.nsplit = (int)decode_uniform(BH, Lk, d, &per);
        a.per = (int)per;
        wgs = BH * a.nsplit;
        split = a.nsplit > 1;
    }
    if (d == 64) return run_decode<64>(Q, K, V, a, wgs, split, workspace, out, s);
    return run_decode<128>(Q, K, V, a, wgs, split, workspace, out, s);
}

// ---------------------------------------------------------------------------
// Allocation-free decode: the partials go to a file-scope device array instead of a caller
// workspace.  Every call fits it: fewer than 2 W partial slots (W resident workgroups, 512 at
// d = 64, 256 at d = 128), 4.25 MiB at d = 64 and 4.125 MiB at d = 128.  In host code `scratch`
// names a host-side stand-in; its device address (one copy per GPU) is looked up once per device with
// hipGetSymbolAddress and only that address is passed to kernels.
static __device__ __align__(256) float scratch[kDecodeScratchBytes / sizeof(float)];

static hipError_t decode_scratch_address(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // on the current device
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

hipError_t launch_attention_decode_noalloc(const void* Q, const void* K, const void* V, int64_t BH, int64_t Lq,
                                           int64_t Lk, int64_t d, float scale, void* out, hipStream_t s) {
    void* part = nullptr;
    if (attention_decode_partials_bytes(BH, Lq, Lk, d) > 0) {
        const hipError_t e = decode_scratch_address(&part);
        if (e != hipSuccess) return e;
    }
    return launch_attention_decode(Q, K, V, BH, Lq, Lk, d, scale, part, kDecodeScratchBytes, out, s);
}

template <int D>
static hipError_t run_prefill(const void* Q, const void* K, const void* V, int64_t BH, int64_t Lq, int64_t Lk,
                              int causal, float scale, void* out, hipStream_t s, int group) {
    switch (prefill_layout(BH, Lq, Lk, D, causal)) {
        case 0:
            if (prefill_phased(Lk)) return run_attention<D, 8, 2, 1, 128>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
            return run_attention<D, 8, 2, 1, 128, false>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
        case 1: return run_attention<D, 4, 2, 2, 64>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
        case 2: return run_attention<D, 2, 2, 4, 32>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
        default: return run_attention<D, 2, 1, 4, 32>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
    }
}

hipError_t launch_attention_deferred(const void* Q, const void* K, const void* V, int64_t BH, int64_t Lq,
                                     int64_t Lk, int64_t d, int causal, float scale, void* out, hipStream_t s,
                                     int group) {  // BH counts query heads
    if (d == 64) return run_prefill<64>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
    return run_prefill<128>(Q, K, V, BH, Lq, Lk, causal, scale, out, s, group);
}

}  // namespace dn
