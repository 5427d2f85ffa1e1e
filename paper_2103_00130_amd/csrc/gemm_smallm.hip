// Streaming checked u8 x s8 -> s32 GEMM for M <= 64 (tall-skinny, batch-of-requests shapes).
//
// Algorithm 1 of arXiv 2103.00130 (product with the encoded B, row sums, comparison) for the
// shapes where the weight matrix is read once and barely reused: the kernel is bound by
// streaming the packed B from HBM, so the design goal is bytes in flight, not MFMA rate.
//
//  * One workgroup owns 16 columns for the whole K range; its four wavefronts take the
//    k-blocks kb = wave, wave+4, ... and issue their loads in batches, two batches in flight,
//    so that the grid as a whole keeps the entire weight matrix in flight.  No LDS staging:
//    a 16x16x64 int8 MFMA B operand is read straight from the packed layout (four 256-byte
//    runs per instruction), the A operand straight from A (it is small and lives in L2).
//  * u8 -> s8 by XOR 0x80 on the A operand, +128 * (column sum of the streamed B bytes) added
//    back; the checksum column S_B rides as four base-256 digit columns on a second MFMA; the
//    column blocks split its K range between them.
//  * The four partial accumulators meet in LDS; wavefront 0 adds them, forms the row sums with
//    DPP row reductions, stores C, and then adds (row sum - checksum) per row into 64-bit
//    workspace words that also count arrivals (returned integer atomics, at most 64 arrivals at a
//    word up to 2048 column blocks, a 32nd of the blocks beyond): whoever completes a word clears it, and a row's word writes its flag.
//    errCount is cleared at the start and added to.  No workgroup waits for another and there is
//    no closing pass.
#include "../../include/abft_gemm.h"
#include "abft_internal.h"

namespace abft {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));  // sixteen bytes at any address
constexpr int kOutC = 1, kOutQ = 2;
constexpr int kFlatN = 4096, kWideN = 8192;   // up to these widths workgroups of 16 and of 32 columns fit the compute units once

// Up to so many column blocks arrive at a row's word directly; beyond, the blocks of a slot meet at a word of their own first (us,
// directly / by slots: 50 blocks, 1x800x3200, 5.0 / 5.1; 63 4.7 / 4.75; 100 5.1 / 4.7; 256 7.1 / 4.8: arrivals at one word follow
// each other at about 10 ns).
constexpr int kFlatBlocks = 64;

// sum over the 16 lanes of a DPP row; every lane of the row ends up with the total
__device__ inline uint32_t row_sum16(uint32_t s) {
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x141, 0xF, 0xF, true);  // row_half_mirror
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x140, 0xF, 0xF, true);  // row_mirror
    return s;
}

// v mod 127 in [0,126] for |v| < 2^59 (2^28 is 1 modulo 127, so the two parts of v = hi * 2^28 + lo may be added)
__device__ inline int32_t floor_mod127(long long v) {
    const int32_t x = (int32_t)(v >> 28) + (int32_t)(v & 0x0FFFFFFF);
    const int32_t r = x % 127;
    return r < 0 ? r + 127 : r;
}

// RB = 16-row blocks of A (M <= 16*RB); NCB = blocks of 16 columns per workgroup.  With NCB = 2 a workgroup owns a
// whole 32-column unit of the packed weight, with NCB = 4 two neighbouring units: every k-block it reads is 2 or
// 4 KiB of contiguous memory instead of every other 256 bytes of it, and one A operand serves two or four matrix
// instructions (wide weights, whose column blocks alone would come to several workgroups per compute unit).
// kAny: A of any alignment, leading dimension and K >= 16.  The same chunks come in with loads from any byte address; the
// one chunk that holds the end of a row, loaded from K - 16, is shifted down to its place before it is used.
template <int RB, int NCB, bool kCheck, int kOut, bool kAny>
__global__ __launch_bounds__(256) void gemm_smallm_kernel(const GemmParams p, const int n_blocks) {
    constexpr int BATCH = (RB == 1 ? 8 : 4) / NCB > 0 ? (RB == 1 ? 8 : 4) / NCB : 1;  // k-blocks per wave per batch of loads
    constexpr bool kWantC = (kOut & kOutC) != 0, kWantQ = (kOut & kOutQ) != 0;
    __shared__ v4i s_acc[3][NCB][RB][64];
    __shared__ v4i s_chk[3][RB][64];
    __shared__ uint32_t s_bsum[3][NCB][64];
    __shared__ uint32_t s_d[64];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cb = blockIdx.x, col0 = cb * 16 * NCB;
    const int KB = p.KB;
    const int lcol = lane & 15, lkg = lane >> 4;

    // B operand of k-block kb: unit of col0, columns 16*half .. +15, k-group lkg
    const int8_t* const b_src = p.packed + packed_unit_offset(col0 / kTileN, 0, (col0 % kTileN) / kUnitN, KB) +
                                (lkg * kUnitN + (col0 % kUnitN) + lcol) * 16;
    constexpr int64_t B_KB_STRIDE = (int64_t)kUnitsPerTile * kUnitBytes;
    // A operand of row block rb: row rb*16 + lcol (clamped), k-group lkg
    const uint8_t* a_row[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) a_row[rb] = p.A + (int64_t)min(rb * 16 + lcol, p.M - 1) * p.lda;
    // this column block's share of the checksum product's K range
    const int lo = share_begin(cb, p.share_q, p.share_r), hi = share_begin(cb + 1, p.share_q, p.share_r);

    // sum_k S_B[k] for the first column block's share of the check, fetched ahead of its use at the very end
    const int32_t total_sb = (kCheck && cb == 0) ? *p.total : 0;

    // errCount is overwritten: the first column block clears it here and whoever finds corrupted rows adds to it.  No row is
    // complete, and so nothing added, before that block has arrived at the row's word, which it does once this store has
    // been acknowledged.
    const bool clears = kCheck && cb == 0 && p.err_count != nullptr && !p.err_accumulate;
    if (clears && tid == 0) __hip_atomic_store(p.err_count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    v4i acc[NCB][RB], cacc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        cacc[rb] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int c = 0; c < NCB; ++c) acc[c][rb] = v4i{0, 0, 0, 0};
    }
    uint32_t bsum[NCB];
#pragma unroll
    for (int c = 0; c < NCB; ++c) bsum[c] = 0;

    const int over = kAny ? (16 - (p.K & 15)) & 15 : 0;   // bytes the end chunk of a row moves down
    v4i fb[2][BATCH][NCB], fa[2][BATCH][RB], fl[2][BATCH];
    auto issue = [&](int kb0, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int kb = kb0 + 4 * u;
            const int kbc = min(kb, KB - 1);
            // a k-block past the end is fetched from the last one and zeroed below
#pragma unroll
            for (int c = 0; c < NCB; ++c)   // the next 16 columns of a unit lie 256 bytes further on, the next unit 2 KiB
                // (The weight passes through without being kept in the caches.  Kept, of one column block per workgroup: 16x4096x2048 4.76 us
                // against 4.81 with one weight again and again and 5.23 / 5.42 with eight in turn, but 5.82 / 5.53 with fresh ones.)
                fb[s][u][c] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(b_src + (int64_t)kbc * B_KB_STRIDE + (c >> 1) * kUnitBytes + (c & 1) * 256));
            const int k = min(kbc * 64 + lkg * 16, p.K - 16);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if constexpr (kAny) fa[s][u][rb] = *reinterpret_cast<const v4i_any*>(a_row[rb] + k);
                else fa[s][u][rb] = *reinterpret_cast<const v4i*>(a_row[rb] + k);
            }
            if (kCheck) {
                fl[s][u] = v4i{0, 0, 0, 0};
                if (kb >= lo && kb < hi && lcol < kLimbs)
                    fl[s][u] = *reinterpret_cast<const v4i*>(p.limbs + ((((int64_t)kb * 4 + lkg) * kLimbs + lcol) << 4));
            }
        }
    };
    auto consume = [&](int kb0, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int kb = kb0 + 4 * u;
            v4i b[NCB];
#pragma unroll
            for (int c = 0; c < NCB; ++c) {
                b[c] = fb[s][u][c];
                if (kb >= KB) b[c] = v4i{0, 0, 0, 0};
                // bytes of B as biased uint8, summed four at a time; the bias comes off at the end
                bsum[c] = __builtin_amdgcn_sad_u8((uint32_t)b[c].x ^ 0x80808080u, 0u, bsum[c]);
                bsum[c] = __builtin_amdgcn_sad_u8((uint32_t)b[c].y ^ 0x80808080u, 0u, bsum[c]);
                bsum[c] = __builtin_amdgcn_sad_u8((uint32_t)b[c].z ^ 0x80808080u, 0u, bsum[c]);
                bsum[c] = __builtin_amdgcn_sad_u8((uint32_t)b[c].w ^ 0x80808080u, 0u, bsum[c]);
            }
            // (chunks past the end of a row, and bytes of its last chunk past it, meet zero rows of B)
            if (kAny && over != 0 && kb == (p.K >> 6)) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const v4i m = shift_down(fa[s][u][rb], over);
                    if (lkg == ((p.K >> 4) & 3)) fa[s][u][rb] = m;
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const v4i a = fa[s][u][rb] ^ (int)0x80808080;
#pragma unroll
                for (int c = 0; c < NCB; ++c) acc[c][rb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b[c], acc[c][rb], 0, 0, 0);
                if (kCheck) cacc[rb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, fl[s][u], cacc[rb], 0, 0, 0);
            }
        }
    };

    // k-blocks of this wave: wave, wave+4, ...; the same number of batches for every wave
    const int per_wave = (KB + 3) / 4;
    const int n_batches = (per_wave + BATCH - 1) / BATCH;
    issue(wave, 0);
    for (int bt = 0; bt < n_batches; bt += 2) {
        if (bt + 1 < n_batches) issue(wave + 4 * BATCH * (bt + 1), 1);
        consume(wave + 4 * BATCH * bt, 0);
        if (bt + 1 < n_batches) {
            if (bt + 2 < n_batches) issue(wave + 4 * BATCH * (bt + 2), 0);
            consume(wave + 4 * BATCH * (bt + 1), 1);
        }
    }

    // ---- the four partial results meet in wavefront 0 --------------------------------
    if (wave > 0) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
            for (int c = 0; c < NCB; ++c) s_acc[wave - 1][c][rb][lane] = acc[c][rb];
            if (kCheck) s_chk[wave - 1][rb][lane] = cacc[rb];
        }
#pragma unroll
        for (int c = 0; c < NCB; ++c) s_bsum[wave - 1][c][lane] = bsum[c];
    }
    __syncthreads();
    if (wave == 0) {
        if (clears) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
#pragma unroll
        for (int w = 0; w < 3; ++w) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int c = 0; c < NCB; ++c) acc[c][rb] += s_acc[w][c][rb][lane];
                if (kCheck) cacc[rb] += s_chk[w][rb][lane];
            }
#pragma unroll
            for (int c = 0; c < NCB; ++c) bsum[c] += s_bsum[w][c][lane];
        }
        // every lane summed 16 biased bytes per k-block slot; 4 waves x n_batches x BATCH slots x 4 k-groups
        const uint32_t bias = 128u * 16u * 4u * 4u * (uint32_t)(n_batches * BATCH);
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
            // column sum of the streamed B for column lcol: the four k-groups sit in lanes lcol + 16*g
            // (row swap and half swap: both return {own, partner} in an order that depends on the lane)
            const auto r16 = __builtin_amdgcn_permlane16_swap(bsum[c], bsum[c], false, false);
            bsum[c] = r16[0] + r16[1];
            const auto r32 = __builtin_amdgcn_permlane32_swap(bsum[c], bsum[c], false, false);
            bsum[c] = r32[0] + r32[1];
            const int32_t cs128 = 128 * (int32_t)(bsum[c] - bias);
            // accumulator layout of the 16x16 MFMA: lane l, element e is row 4*(l/16) + e, column l%16
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][rb][e] += cs128;
        }

        if (p.n_inj > 0) {
            // simulated faults in the 32-bit intermediate (test hook): XOR before the row sums
            const abft_inject_t* inj = reinterpret_cast<const abft_inject_t*>(p.inj);
            for (int n = 0; n < p.n_inj; ++n) {
                const int r = inj[n].row, c = inj[n].col - col0;
                if (r < 0 || r >= p.M || r >= 16 * RB || c < 0 || c >= 16 * NCB || inj[n].col >= p.N) continue;
                const bool mine = (lcol == (c & 15)) && (lkg == ((r & 15) >> 2));
#pragma unroll
                for (int cc = 0; cc < NCB; ++cc)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (mine && cc == (c >> 4) && rb == (r >> 4) && e == (r & 3)) acc[cc][rb][e] ^= (int)inj[n].xor_mask;
            }
        }

        // stores first (they need no answer), then the check, whose atomics wait for theirs;
        // per (rb, e) one store instruction covers 4 rows x 16 columns
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
            const int col = col0 + c * 16 + lcol;
            RequantCol rqc;   // this lane's column, fetched once
            rqc.sub = 0;
            rqc.mult = 0.0f;
            if (kWantQ && col < p.N) rqc = requant_col(p.colsum[col], col, p.rq);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                uint32_t qw = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = rb * 16 + 4 * lkg + e;
                    if (kWantC && row < p.M && col < p.N) p.C[(int64_t)row * p.ldc + col] = acc[c][rb][e];
                    if (kWantQ) qw = requant_into(qw, e, acc[c][rb][e], rqc, p.rq.zC);
                }
                if (kWantQ) {
                    qw = turn_quad(qw, lane);
                    const int row = rb * 16 + 4 * lkg + (lane & 3), first = col & ~3;
                    if (row < p.M && first < p.N) store_quad(p.Cq + (int64_t)row * p.ldcq + first, qw, p.N - first);
                }
            }
        }
        if (kCheck) {
            const bool mod127 = p.mod127 != 0;
            const int slot = cb & (kSmallMSlots - 1);
            const uint32_t total128 = 128u * (uint32_t)total_sb;  // sum_k 128*S_B[k], once per row (first column block)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // (Algorithm 1 as printed, p.mod127: the entries are exact 32-bit values, K <= 65536, and are
                    // summed as residues; the one live digit column holds rowSum, so its product is exact too)
                    uint32_t mine = 0;   // this lane's entries of the row (residues of them under the printed modulus)
#pragma unroll
                    for (int c = 0; c < NCB; ++c)
                        mine += mod127 ? (uint32_t)floor_mod127((long long)acc[c][rb][e]) : (uint32_t)acc[c][rb][e];
                    const uint32_t rs = row_sum16(mine);
                    uint32_t ck = lcol < kLimbs ? ((uint32_t)cacc[rb][e] << (8 * lcol)) : 0u;
                    ck += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ck, 0xB1, 0xF, 0xF, true);
                    ck += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ck, 0x4E, 0xF, 0xF, true);
                    const int row = rb * 16 + 4 * lkg + e;
                    if (lcol == 0)
                        s_d[row] = mod127 ? (uint32_t)floor_mod127((long long)rs - (long long)(int32_t)ck - 128ll * (long long)total_sb)
                                          : rs - ck - total128;
                }
            // One row per lane.  The row's difference climbs workspace words, each a 64-bit
            // (value << 32 | arrivals) taken with one returned atomic.  With more than kFlatBlocks column
            // blocks the first word is that of (slot, row), shared by the blocks of one slot, whose
            // last arrival carries the slot's sum on; the next is the word of the row, where the last
            // arrival has the complete difference and writes the flag.  Every word is cleared by the
            // arrival that completes it.  Nobody waits for anybody.
            bool bad = false;
            if (lane < 16 * RB && lane < p.M) {
                unsigned long long* const w_slot =
                    reinterpret_cast<unsigned long long*>(p.ws + kWsHeaderInts) + slot * kSmallMRows + lane;
                unsigned long long* const w_row =
                    reinterpret_cast<unsigned long long*>(p.ws + kWsHeaderInts) + kSmallMSlots * kSmallMRows + lane;
                uint32_t t = s_d[lane], n_row = (uint32_t)n_blocks;
                bool go = true;
                if (n_blocks > kFlatBlocks) {
                    const uint32_t n_slot = ((uint32_t)n_blocks - (uint32_t)slot + kSmallMSlots - 1) / kSmallMSlots;
                    const unsigned long long old = __hip_atomic_fetch_add(w_slot, ((unsigned long long)t << 32) | 1ull,
                                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    go = (uint32_t)old == n_slot - 1u;
                    if (go) {
                        t += (uint32_t)(old >> 32);
                        __hip_atomic_store(w_slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    n_row = (uint32_t)kSmallMSlots;
                }
                if (n_blocks == 1) {
                    // a single column block holds the whole row: nothing crosses workgroups
                    bad = mod127 ? (t % 127u != 0u) : (t != 0u);
                    p.row_flags[lane] = (int32_t)bad;
                } else if (go) {
                    const unsigned long long old = __hip_atomic_fetch_add(w_row, ((unsigned long long)t << 32) | 1ull,
                                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((uint32_t)old == n_row - 1u) {
                        const uint32_t diff = (uint32_t)(old >> 32) + t;
                        bad = mod127 ? (diff % 127u != 0u) : (diff != 0u);
                        __hip_atomic_store(w_row, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        p.row_flags[lane] = (int32_t)bad;
                    }
                }
            }
            // errCount is added to by the wavefronts that found corrupted rows (no return value, nobody waits)
            const unsigned long long bad_mask = __ballot(bad);
            if (p.err_count != nullptr && bad_mask != 0ull && lane == __builtin_ctzll(bad_mask))
                __hip_atomic_fetch_add(p.err_count, (int32_t)__builtin_popcountll(bad_mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int RB, int NCB, bool kAny>
hipError_t launch_any(bool check, bool want_c, bool want_q, const GemmParams& p_in, hipStream_t s) {
    GemmParams p = p_in;
    const int n_blocks = (p.N + 16 * NCB - 1) / (16 * NCB);
    p.share_q = p.KB / n_blocks;   // k-blocks of the checksum product per column block
    p.share_r = p.KB % n_blocks;
    const dim3 grid((unsigned)n_blocks), block(256);
#define ABFT_LAUNCH(CK, OUT)                                                         \
    do {                                                                             \
        gemm_smallm_kernel<RB, NCB, CK, OUT, kAny><<<grid, block, 0, s>>>(p, n_blocks);    \
        return hipGetLastError();                                                    \
    } while (0)
#define ABFT_OUT(CK)                                          \
    do {                                                      \
        if (want_c && want_q) ABFT_LAUNCH(CK, kOutC | kOutQ); \
        if (want_c) ABFT_LAUNCH(CK, kOutC);                   \
        ABFT_LAUNCH(CK, kOutQ);                               \
    } while (0)
    if (check) ABFT_OUT(true);
    ABFT_OUT(false);
#undef ABFT_OUT
#undef ABFT_LAUNCH
}

template <int RB, int NCB>
hipError_t launch_rb(bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    // rows of any alignment: up to 16, or 64 columns per workgroup (what gemm_tile_wk.h leaves)
    if constexpr (RB == 1 || (RB == 2 && NCB == 4))
        if (!p.a_vec_ok || p.K % 16 != 0) return launch_any<RB, NCB, true>(check, want_c, want_q, p, s);
    return launch_any<RB, NCB, false>(check, want_c, want_q, p, s);
}

}  // namespace

hipError_t launch_gemm_smallm(bool any_a, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s) {
    if (p.M > 64) return hipErrorNotSupported;
    if (!p.a_vec_ok || p.K % 16 != 0)
        if (!any_a || p.mod127 || p.K < 16 || p.M > 32 || (p.M > 16 && p.N <= kWideN)) return hipErrorNotSupported;
    // As few columns per workgroup as still give every compute unit one workgroup at most (us, NCB = 1 / 2 / 4):
    // 16x4096x4096 7.0 / 8.5 / 11.4; 16x6000x4000 10.3 / 8.8 / 12.4; 16x8192x8192 19.1 / 15.1 / 21.1; 16x12000x12000 37.3 /
    // 34.5 / 29.8; 16x16384x16384 62 / 58 / 43.7 (6.1 TB/s); 32x6000x4000 14.8 / 11.8 / 16.5; 32x16384x16384 90 / 65 / 49.4.
    // (A handful of rows, whose A operands are next to nothing, stays with 32 columns up to 16384: 1x12000x12000 26.6 / 27.2.)
    const int ncb = p.N <= kFlatN ? 1 : (p.N <= kWideN || (p.M <= 8 && p.N < 2 * kWideN)) ? 2 : 4;
    if (p.M <= 16)
        return ncb == 1 ? launch_rb<1, 1>(check, want_c, want_q, p, s)
                        : ncb == 2 ? launch_rb<1, 2>(check, want_c, want_q, p, s) : launch_rb<1, 4>(check, want_c, want_q, p, s);
    if (p.M <= 32)
        return ncb == 1 ? launch_rb<2, 1>(check, want_c, want_q, p, s)
                        : ncb == 2 ? launch_rb<2, 2>(check, want_c, want_q, p, s) : launch_rb<2, 4>(check, want_c, want_q, p, s);
    if (p.M <= 48) return launch_rb<3, 1>(check, want_c, want_q, p, s);
    return launch_rb<4, 1>(check, want_c, want_q, p, s);
}

}  // namespace abft
