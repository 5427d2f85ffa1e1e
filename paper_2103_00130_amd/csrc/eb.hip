// ABFT-checked row-wise quantized EmbeddingBag (include/abft_eb.h): Algorithm 2 of
// arXiv 2103.00130 (Section V) on the operator of Section III-C.
//
// The work is a gather: every pooled row is read once from a table far larger than any
// cache, so the kernels are built around bytes in flight, not arithmetic.
//
//  * Codes are 8 bits wide, or 4 bits wide and packed two per byte (Section V: p = 4 or 8); the
//    kernels are templated on the width and differ only in how a code is cut out of its word.
//  * The table is kept as fused records [codes][scale][bias][C_T][unused]: the row sum that
//    Eq. 4 needs arrives in the same memory transaction as the scale and bias the lookup needs
//    anyway, so the check adds no memory traffic at all.
//  * Batch kernel (very many lookups of a few rows): one lane per 16 code bytes of a row.  Every lane owns the columns
//    of its bytes and reads them per pooled row straight into registers, eight rows in flight per
//    lane; the chip is filled by lookups, and the lanes of a lookup walk its index list in order.
//  * Group kernel: one, two or four wavefronts per lookup.  Their threads fetch different 16-byte
//    pieces of the lookup's records into LDS, then, owning columns, walk the staged rows in index order.
//  * The loads of the records are ordinary ones where lookups are many and the table is no larger than a few times the caches: rows that
//    come back, in the same batch or a later one, are then found there (16384 lookups of 100 rows of 80 bytes from a table of 320 MB,
//    ordinary / marked as streaming: the same ones again and again 49.6 us / 56.2, fresh ones at every call 50.5 / 57.0; 65536 of 4 rows
//    16.0 / 18.1).  Lookups of one or two wavefronts from a larger table mark them (eb_passes_by), and so do four wavefronts per lookup,
//    the form for few lookups, whose time is latency (10 lookups of 100 rows never read before: 5.0 us, 5.55 without; read before: 4.5
//    either way).
//  * Every load is unconditional (clamped position, row 0 in place of a bad index): a load under
//    `if (valid)` is followed by a wait, which would put the loads of a lookup one after the other.
//  Both accumulate every output column in the same order (index order, one fused multiply-add
//  per row, biases summed apart), so they give the same bits; RSum and CSum are taken in
//  binary64.  CSum adds one exactly rounded term per pooled row: in index order in the batch
//  kernel, lanes in parallel (a tree) in the group kernel - Eq. 4 fixes the terms, not their order.
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>

#include "../../include/abft_eb.h"
#include "abft_internal.h"
#include "eb_choice.h"

struct abft_eb_table {
    uint8_t* rec;    // rows * stride bytes: [codes][scale f32][bias f32][C_T i32][unused]
    int64_t rows;
    int64_t stride;  // code bytes + 16, or the next power of two when the records are line-aligned
    int d;           // columns
    int bits;        // 8 or 4 bits per code
    int code_bytes;  // d * bits / 8
    int device;
};

namespace abft {
namespace {

typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct EbParams {
    const uint8_t* tab;
    int64_t stride;  // bytes from one record to the next
    int64_t rows;
    const int64_t* indices;
    int64_t n_indices;
    const int64_t* offsets;
    int64_t n_bags;
    const float* weights;
    float* R;
    int64_t ldr;
    int32_t* flags;
    double* rsum;
    double* csum;
    double bound;
};

__device__ inline float as_f32(unsigned int u) { return __builtin_bit_cast(float, u); }
__device__ inline unsigned int as_u32(float f) { return __builtin_bit_cast(unsigned int, f); }

__device__ inline void bag_range(const EbParams& p, int64_t bag, int64_t* beg, int64_t* end) {
    int64_t b = p.offsets[bag], e = p.offsets[bag + 1];
    b = b < 0 ? 0 : (b > p.n_indices ? p.n_indices : b);
    e = e < b ? b : (e > p.n_indices ? p.n_indices : e);
    *beg = b;
    *end = e;
}

// Algorithm 2, the comparison: err unless |RSum - CSum| <= bound * max(|RSum|, |CSum|) and finite
__device__ inline int compare_sums(double rs, double cs, double bound) {
    const double diff = fabs(rs - cs);
    return (!(diff <= bound * fmax(fabs(rs), fabs(cs))) || !(diff < (double)INFINITY)) ? ABFT_EB_ERR : 0;
}

// Value that lane ^ M holds, without a trip through memory: DPP inside a row of 16 lanes, the swizzle
// crossbar for M = 4 and 8, the row and half swaps beyond (both give {own, partner} in an order that
// depends on the lane, hence the XOR).
template <int M>
__device__ inline unsigned int from_lane_xor(unsigned int v) {
    static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "one bit of the lane number");
    if constexpr (M == 1) return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
    else if constexpr (M == 2) return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
    else if constexpr (M == 4) return (unsigned int)__builtin_amdgcn_ds_swizzle((int)v, 0x101F);
    else if constexpr (M == 8) return (unsigned int)__builtin_amdgcn_ds_swizzle((int)v, 0x201F);
    else if constexpr (M == 16) {
        const auto sw = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return sw[0] ^ sw[1] ^ v;
    } else {
        const auto sw = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return sw[0] ^ sw[1] ^ v;
    }
}

template <int M>
__device__ inline double from_lane_xor(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned long long o = (unsigned long long)from_lane_xor<M>((unsigned int)b) |
                                 ((unsigned long long)from_lane_xor<M>((unsigned int)(b >> 32)) << 32);
    return __builtin_bit_cast(double, o);
}

// sum over the 64 lanes, the same value in every lane: a butterfly (lane pairs, then pairs of pairs, ...)
__device__ inline double wave_sum(double v) {
    v += from_lane_xor<1>(v);
    v += from_lane_xor<2>(v);
    v += from_lane_xor<4>(v);
    v += from_lane_xor<8>(v);
    v += from_lane_xor<16>(v);
    v += from_lane_xor<32>(v);
    return v;
}

// Word w of lane l of a quad becomes word l of lane w (every component for itself).
__device__ inline void turn_quad_columns(v4f& a, v4f& b, v4f& c, v4f& d, int lane) {
    const bool odd = lane & 1, upper = lane & 2;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const unsigned int a0 = as_u32(a[k]), b0 = as_u32(b[k]);
        const unsigned int c0 = as_u32(c[k]), d0 = as_u32(d[k]);
        const unsigned int x = from_lane_xor<1>(odd ? a0 : b0), y = from_lane_xor<1>(odd ? c0 : d0);
        const unsigned int a1 = odd ? x : a0, b1 = odd ? b0 : x, c1 = odd ? y : c0, d1 = odd ? d0 : y;
        const unsigned int u = from_lane_xor<2>(upper ? a1 : c1), t = from_lane_xor<2>(upper ? b1 : d1);
        a[k] = as_f32(upper ? u : a1);
        c[k] = as_f32(upper ? c1 : u);
        b[k] = as_f32(upper ? t : b1);
        d[k] = as_f32(upper ? d1 : t);
    }
}

// the columns held by 16 code bytes of one pooled row: acc[k] = a * code[k] + acc[k].
// 8-bit codes: 16 columns; 4-bit codes: 32 columns, the even column in the low half of its byte.
template <int BITS>
__device__ inline void fma_codes(float (&acc)[128 / BITS], float a, v4u q) {
    constexpr int PER_WORD = 32 / BITS;
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int n = 0; n < PER_WORD; ++n)
            acc[PER_WORD * w + n] = __builtin_fmaf(a, (float)((q[w] >> (BITS * n)) & ((1u << BITS) - 1u)), acc[PER_WORD * w + n]);
}

// ---------------------------------------------------------------------------------------------
// Batch kernel: G lanes per lookup, one per 16 code bytes of a row.
template <int G, int BITS, bool kCheck, bool kWeighted, bool kTwoSets>
__global__ __launch_bounds__(256) void eb_batch_kernel(const EbParams p) {
    constexpr int CB = 16 * G;            // code bytes per row
    constexpr int CPP = 128 / BITS;       // columns per 16-byte piece
    constexpr int D = G * CPP, U = 8;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t bag = t / G;
    const int piece = (int)(t % G);
    if (bag >= p.n_bags) return;  // whole lane groups leave together (256 is a multiple of G)
    int64_t beg, end;
    bag_range(p, bag, &beg, &end);

    float acc[CPP];
#pragma unroll
    for (int k = 0; k < CPP; ++k) acc[k] = 0.0f;
    float beta_sum = 0.0f;
    double cs = 0.0;
    int flag = 0;
    const uint8_t* const base = p.tab + piece * 16;

    // Rows are handled in sets of U.  Every load is unconditional inside its set (clamped position,
    // row 0 in place of a bad index): the index loads of a set go out together, then its row loads,
    // and only then anything waits.
    // kTwoSets: two sets in flight - the row loads of a set go out while the set before it is being
    // pooled, and the indices of the set after it are already on their way - so that the latency of
    // the indices, the latency of the rows and the arithmetic overlap instead of adding up.  A launch
    // of a few wavefronts per SIMD has nothing else to hide them behind; with many wavefronts the
    // other wavefronts do that, and the registers of the second set cost more than it gains.
    // A row that is not pooled enters the sums with scale, bias and row sum 0, which leaves every
    // accumulator as it is, bit for bit.
    struct IdxSet {
        int64_t idx[U];
        float wv[U];
    };
    struct RowSet {
        float wv[U];
        v4u q[U], tl[U];
        bool ok[U];
    };
    auto load_indices = [&](IdxSet& r, int64_t pos) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t pp = pos + u < end ? pos + u : end - 1;
            r.idx[u] = p.indices[pp];
            if (kWeighted) r.wv[u] = p.weights[pp];
        }
    };
    auto load_rows = [&](RowSet& r, const IdxSet& ix, int64_t pos) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = pos + u < end;
            r.ok[u] = in && (uint64_t)ix.idx[u] < (uint64_t)p.rows;
            if (in && !r.ok[u]) flag |= ABFT_EB_BAD_INDEX;
            if (kWeighted) r.wv[u] = ix.wv[u];
            const uint8_t* rec = base + (r.ok[u] ? ix.idx[u] : 0) * p.stride;
            r.q[u] = *reinterpret_cast<const v4u*>(rec);
            r.tl[u] = *reinterpret_cast<const v4u*>(rec + (CB - piece * 16));
        }
    };
    auto pool = [&](const RowSet& r) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float a = as_f32(r.tl[u][0]), c = as_f32(r.tl[u][1]);
            if (kWeighted) {
                a = r.wv[u] * a;
                c = r.wv[u] * c;
            }
            a = r.ok[u] ? a : 0.0f;
            c = r.ok[u] ? c : 0.0f;
            fma_codes<BITS>(acc, a, r.q[u]);
            beta_sum = beta_sum + c;
            if (kCheck) {
                // Eq. 4, the term of one pooled row: scale * C_T + d * bias, rounded once (both products
                // are exact in binary64), then added to the running sum
                cs = cs + fma((double)a, (double)(r.ok[u] ? (int32_t)r.tl[u][2] : 0), (double)D * (double)c);
            }
        }
    };
    if (!kTwoSets) {
        for (int64_t pos = beg; pos < end; pos += U) {
            IdxSet ia;
            RowSet ra;
            load_indices(ia, pos);
            load_rows(ra, ia, pos);
            pool(ra);
        }
    } else if (beg < end) {
        IdxSet ia, ib;
        RowSet ra, rb;
        load_indices(ia, beg);
        load_rows(ra, ia, beg);
        load_indices(ib, beg + U);
        for (int64_t pos = beg;; pos += 2 * U) {
            // here the rows of ra and the indices ib are in flight
            if (pos + U < end) {
                load_rows(rb, ib, pos + U);
                load_indices(ia, pos + 2 * U);
            }
            pool(ra);
            if (pos + U >= end) break;
            if (pos + 2 * U < end) {
                load_rows(ra, ia, pos + 2 * U);
                load_indices(ib, pos + 3 * U);
            }
            pool(rb);
            if (pos + 2 * U >= end) break;
        }
    }

    float* const out = p.R + bag * p.ldr;
    double rs = 0.0;
    v4f v[CPP / 4];
#pragma unroll
    for (int w = 0; w < CPP / 4; ++w) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[w][k] = acc[4 * w + k] + beta_sum;
            if (kCheck) rs += (double)v[w][k];
        }
    }
    if constexpr (G >= 4) {
        // The four lanes of a quad turn their 4x4 groups of four columns, so that a store writes runs of 64 bytes instead of
        // sixteen bytes of every 64 or 128 (4-bit codes: 20000 lookups of 4 rows of 512 bytes 40.6 us, 29.4 this way; 65000 of 2 of
        // 256 bytes 60.2 / 46.2, of 2 of 128 bytes 34.8 / 26.8; 8-bit, 65000 of 2 of 256 bytes 30.5 / 24.9).
#pragma unroll
        for (int h = 0; h < CPP / 16; ++h) {
            turn_quad_columns(v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3], piece);
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<v4f*>(out + ((piece & ~3) + j) * CPP + 16 * h + 4 * (piece & 3)) = v[4 * h + j];
        }
    } else {
#pragma unroll
        for (int w = 0; w < CPP / 4; ++w) *reinterpret_cast<v4f*>(out + piece * CPP + 4 * w) = v[w];
    }
    if (kCheck) {
        if constexpr (G > 1) rs += from_lane_xor<1>(rs);
        if constexpr (G > 2) rs += from_lane_xor<2>(rs);
        if constexpr (G > 4) rs += from_lane_xor<4>(rs);
        if constexpr (G > 8) rs += from_lane_xor<8>(rs);
        if constexpr (G > 16) rs += from_lane_xor<16>(rs);
        if (piece == 0) {
            p.flags[bag] = flag | compare_sums(rs, cs, p.bound);
            if (p.rsum) p.rsum[bag] = rs;
            if (p.csum) p.csum[bag] = cs;
        }
    } else if (p.flags && piece == 0) {
        p.flags[bag] = flag;
    }
}

// ---------------------------------------------------------------------------------------------
// Group kernel: W wavefronts per lookup (a workgroup), rows staged through LDS.
//  1. fetch: every thread loads different 16-byte pieces of the chunk's records (as many instructions as the chunk
//     needs) and they are laid out in LDS record after record.  The row's scalars - the weighted scale and bias, each to an
//     array of its own, and the row's term of Eq. 4, which is added up in a thread - are formed by the thread that holds a
//     record's tail piece where a chunk is one or two load instructions, and else by a thread per row from the staged tails:
//     the few lanes that hold tails would go through the same forty instructions once per load instruction (W = 4, 512-byte
//     rows, one lookup of 112: 8.0 us, 7.0 by rows; 100 of 240 rows of 256 bytes 10.4 / 9.3);
//  2. pooling, rows in index order: threads own columns; eight rows at a time, the next eight on their way from LDS while
//     the current ones are pooled, scales read four to an instruction.  The biases are added up in index order by a
//     wavefront of its own (W = 1: by every lane beside its columns).
//  The indices of the next chunk are on their way while a chunk is pooled.
//  Many lookups of the same total: bound by memory, whole 128-byte lines for every record (16384 lookups of 100 rows of 80
//  bytes: 59.0 us with four wavefronts each as it was before, 50.4 with two now; 272 bytes: 146 and 100).  Short lookups: by
//  what a lookup costs beside its rows (9000 of 27 rows: 18.4 -> 12.3 us, 16384 of 10: 32 -> 10.8, 3000 of 5: 6.8 -> 3.5).
template <int G, int BITS, int W, bool kPassBy, bool kCheck, bool kWeighted>
__global__ __launch_bounds__(W * 64) void eb_group_kernel(const EbParams p) {
    constexpr int NT = W * 64;
    constexpr int CB = 16 * G;                 // code bytes per row
    constexpr int D = CB * 8 / BITS, REC = CB + 16;   // REC: a record as staged in LDS (no padding there)
    constexpr int P = G + 1;                   // 16-byte pieces per record
    constexpr int NL = W >= 2 ? (G >= 16 ? 8 : 4) : (G >= 32 ? 16 : (G >= 4 ? 8 : 4));   // load instructions per thread and chunk
    constexpr int PIECES = NL * NT;
    // Whole records per chunk: with one or two wavefronts in eights, as they are pooled; with four, where a lookup's time is
    // that of its chunks one after the other, as many as the loads fetch (512-byte rows, one lookup of 58 rows: 4.9 us in one
    // chunk of 62, 6.6 with chunks of 56; 128 bytes, 113 rows: 4.6 / 5.7).  The rows that fill up its last eight are whatever
    // lies there, pooled with scale 0.
    constexpr int ROWS = W == 4 ? PIECES / P : PIECES / P / 8 * 8, ROWS8 = (ROWS + 7) / 8 * 8;
    static_assert(ROWS >= 8, "a chunk holds eight rows");
    // with four wavefronts, which run few lookups at a time, the rows of the next chunk come in while a chunk is pooled; with
    // one or two, and with rows of 256 bytes and more, whose chunks are eight load instructions, the registers that takes are
    // worth more as further lookups under way (512-byte rows, 4-bit codes, 1024 lookups of 210: 46.2 us, 39.1 without; 500 of
    // 210 28.7 / 25.9; 100 of 210 20.7 / 21.5)
    constexpr bool kPrefetch = W == 4 && G < 16;
    constexpr int kByRowsFrom = W >= 2 || G >= 4 ? 4 : NL + 1;   // (narrow rows in one wavefront have their tails in most lanes)
    static_assert(ROWS8 == ROWS || kByRowsFrom <= NL, "the rows that fill up a full chunk need their zeros");
    constexpr int BPT = CB > NT ? CB / NT : 1; // code bytes per thread in the pooling phase
    constexpr int CPL = BPT * 8 / BITS;        // columns per thread
    __shared__ v4u s_rec[ROWS8 * P > PIECES ? ROWS8 * P : PIECES];
    __shared__ __align__(16) float s_scale[ROWS8], s_bias[ROWS8];
    __shared__ double s_rs[W], s_cs[W];
    __shared__ float s_beta;
    __shared__ int s_bad[W];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t bag = blockIdx.x;
    int64_t beg, end;
    bag_range(p, bag, &beg, &end);

    float acc[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) acc[k] = 0.0f;
    float beta = 0.0f;
    double cs = 0.0;   // this thread's terms of Eq. 4
    bool bad_any = false;
    const bool col_thread = tid * BPT < CB;
    // the chain of the biases runs on a wavefront that owns few or no columns
    const bool beta_wave = W == 1 || wave == W - 1;
    const uint8_t* const s_bytes = reinterpret_cast<const uint8_t*>(s_rec);
    auto meet = []() __attribute__((always_inline)) {
        if constexpr (W > 1) {
            __syncthreads();
        } else {
            // one wavefront: its LDS operations execute in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    };

    struct Indices {
        int64_t idx[NL];
        float w[NL];
    };
    struct Rows {
        v4u v[NL];
        float w[NL];
        bool ok[NL];
    };
    // Piece g = l*NT + tid of a chunk is piece g % P of row g / P.  All loads are unconditional (clamped row, row 0 in
    // place of a bad index) so that they all go out together.
    auto load_indices = [&](Indices& x, int64_t pos, int n, auto l_c) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < decltype(l_c)::value; ++l) {
            const int r = (l * NT + tid) / P;
            const int64_t at = pos + (r < n ? r : n - 1);
            x.idx[l] = p.indices[at];
            if (kWeighted) x.w[l] = p.weights[at];
        }
    };
    auto load_rows = [&](Rows& x, const Indices& ix, auto l_c) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < decltype(l_c)::value; ++l) {
            const int g = l * NT + tid, pc = g % P;
            x.ok[l] = (uint64_t)ix.idx[l] < (uint64_t)p.rows;
            if (kWeighted) x.w[l] = ix.w[l];
            const v4u* rec = reinterpret_cast<const v4u*>(p.tab + (x.ok[l] ? ix.idx[l] : 0) * p.stride + pc * 16);
            x.v[l] = kPassBy ? __builtin_nontemporal_load(rec) : *rec;
        }
    };
    // A row's scalars go to arrays of their own: the weighted scale and bias, and its term of Eq. 4 to a sum.  A row that is not
    // pooled - a bad index, the rows that fill up the last eight - gets scale, bias and row sum 0, which leaves every accumulator
    // as it is, bit for bit.
    auto scalars = [&](int r, int n, bool ok, float a, float c, unsigned int c_t) __attribute__((always_inline)) {
        const bool use = ok && r < n;
        if (!ok && r < n) bad_any = true;
        a = use ? a : 0.0f;
        c = use ? c : 0.0f;
        s_scale[r] = a;
        s_bias[r] = c;
        // Eq. 4, the term of one pooled row: scale * C_T + d * bias, rounded once (both products are exact in
        // binary64).  The terms are exact to their one rounding; only the order of their sum differs from
        // index order, by at most n * 2^-53 * sum |term|, eleven decimal orders below the bound of the comparison.
        if (kCheck) cs = cs + fma((double)a, (double)(use ? (int32_t)c_t : 0), (double)D * (double)c);
    };
    auto stage = [&](const Rows& x, int n, auto l_c, auto chunk_c) __attribute__((always_inline)) {
        const int rows8 = (n + 7) / 8 * 8;
        constexpr bool kByRows = decltype(l_c)::value >= kByRowsFrom;
#pragma unroll
        for (int l = 0; l < decltype(l_c)::value; ++l) {
            if (decltype(chunk_c)::value && l > 0 && l * NT >= rows8 * P) break;   // (what a short last chunk does not need is left where it is)
            const int g = l * NT + tid, r = g / P;
            const bool tail = g - r * P == G;
            v4u v = x.v[l];
            if constexpr (kByRows) {
                if (kWeighted) {
                    v[0] = tail ? __builtin_bit_cast(unsigned int, x.w[l] * as_f32(v[0])) : v[0];
                    v[1] = tail ? __builtin_bit_cast(unsigned int, x.w[l] * as_f32(v[1])) : v[1];
                }
                v[3] = tail ? (unsigned int)x.ok[l] : v[3];   // (unused in memory)
                s_rec[g] = v;
            } else {
                s_rec[g] = v;
                if (tail && r < ROWS) scalars(r, n, x.ok[l], kWeighted ? x.w[l] * as_f32(v[0]) : as_f32(v[0]), kWeighted ? x.w[l] * as_f32(v[1]) : as_f32(v[1]), v[2]);
            }
        }
        if constexpr (kByRows) {
            meet();
#pragma unroll
            for (int k = 0; k < (ROWS8 + NT - 1) / NT; ++k) {
                const int r = k * NT + tid;
                if (r < rows8) {
                    const v4u t = s_rec[r * P + G];
                    scalars(r, n, t[3] != 0u, as_f32(t[0]), as_f32(t[1]), t[2]);
                }
            }
        }
    };
    struct Eight {
        v4f a[2], c[2];
        unsigned int code[8][BPT > 4 ? 2 : 1];
    };
    // (threads without columns, in narrow tables, repeat the last one's)
    const int at = (col_thread ? tid : CB / BPT - 1) * BPT;
    auto read_eight = [&](Eight& x, int r0, auto cols_c, auto beta_c) __attribute__((always_inline)) {
        constexpr bool COLS = decltype(cols_c)::value, BETA = decltype(beta_c)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (COLS) x.a[h] = *reinterpret_cast<const v4f*>(s_scale + r0 + 4 * h);
            if (BETA) x.c[h] = *reinterpret_cast<const v4f*>(s_bias + r0 + 4 * h);
        }
        if (COLS)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint8_t* const codes = s_bytes + (r0 + i) * REC + at;
                if constexpr (BPT == 1) x.code[i][0] = *codes;
                else if constexpr (BPT == 2) x.code[i][0] = *reinterpret_cast<const uint16_t*>(codes);
                else {
#pragma unroll
                    for (int h = 0; h < BPT / 4; ++h) x.code[i][h] = reinterpret_cast<const unsigned int*>(codes)[h];
                }
            }
    };
    auto pool_eight = [&](const Eight& x, auto cols_c, auto beta_c) __attribute__((always_inline)) {
        constexpr bool COLS = decltype(cols_c)::value, BETA = decltype(beta_c)::value;
        constexpr int CPW = 32 / BITS;   // columns per word of codes
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (COLS)
#pragma unroll
                for (int k = 0; k < CPL; ++k)
                    acc[k] = __builtin_fmaf(x.a[i >> 2][i & 3], (float)((x.code[i][k / CPW] >> (BITS * (k % CPW))) & ((1u << BITS) - 1u)), acc[k]);
            if (BETA) beta = beta + x.c[i >> 2][i & 3];
        }
    };
    auto pool_as = [&](int n, auto cols_c, auto beta_c) __attribute__((always_inline)) {
        Eight x, y;
        read_eight(x, 0, cols_c, beta_c);
        for (int r = 0; r < n; r += 16) {
            if (r + 8 < n) read_eight(y, r + 8, cols_c, beta_c);
            pool_eight(x, cols_c, beta_c);
            if (r + 8 >= n) break;
            if (r + 16 < n) read_eight(x, r + 16, cols_c, beta_c);
            pool_eight(y, cols_c, beta_c);
        }
    };
    auto pool = [&](int n) __attribute__((always_inline)) {
        const bool cols = W == 1 || wave * 64 * BPT < CB;
        if (W == 1) pool_as(n, std::true_type{}, std::true_type{});
        else if (cols && beta_wave) pool_as(n, std::true_type{}, std::true_type{});
        else if (cols) pool_as(n, std::true_type{}, std::false_type{});
        else if (beta_wave) pool_as(n, std::false_type{}, std::true_type{});
    };
    auto short_lookup = [&](int n, auto l_c) __attribute__((always_inline)) {
        Indices ix;
        Rows x;
        load_indices(ix, beg, n, l_c);
        load_rows(x, ix, l_c);
        stage(x, n, l_c, std::false_type{});
        meet();
        pool(n);
    };
    using full_c = std::integral_constant<int, NL>;
    const int64_t total = end - beg;
    if (total <= ROWS) {
        // the whole lookup in one chunk, with as many load instructions as it needs
        const int n = (int)total, need = ((n + 7) / 8 * 8 * P + NT - 1) / NT;
        if (n == 0) {
        } else if (need <= 1) short_lookup(n, std::integral_constant<int, 1>{});
        else if (need <= 2) short_lookup(n, std::integral_constant<int, 2>{});
        else if (NL > 4 && need <= 4) short_lookup(n, std::integral_constant<int, 4>{});
        else short_lookup(n, full_c{});
    } else {
        auto rows_at = [&](int64_t pos) { return (int)(end - pos < ROWS ? end - pos : ROWS); };
        Indices ix;
        Rows x;
        load_indices(ix, beg, ROWS, full_c{});
        load_rows(x, ix, full_c{});
        load_indices(ix, beg + ROWS, rows_at(beg + ROWS), full_c{});
        for (int64_t pos = beg;;) {
            // here the rows of this chunk and the indices of the next are in flight
            const int n = rows_at(pos);
            stage(x, n, full_c{}, std::true_type{});
            meet();
            if (kPrefetch && pos + ROWS < end) load_rows(x, ix, full_c{});
            if (kPrefetch && pos + 2 * ROWS < end) load_indices(ix, pos + 2 * ROWS, rows_at(pos + 2 * ROWS), full_c{});
            pool(n);
            pos += ROWS;
            if (pos >= end) break;
            if (!kPrefetch) {
                load_rows(x, ix, full_c{});
                if (pos + ROWS < end) load_indices(ix, pos + ROWS, rows_at(pos + ROWS), full_c{});
            }
            meet();   // this chunk has been pooled
        }
    }

    if (kCheck) cs = wave_sum(cs);
    const bool bad_wave = __ballot(bad_any) != 0ull;
    if constexpr (W > 1) {
        if (beta_wave && lane == 0) s_beta = beta;
        if (lane == 0) {
            if (kCheck) s_cs[wave] = cs;
            s_bad[wave] = bad_wave;
        }
        __syncthreads();
        beta = s_beta;
    }
    double rs = 0.0;
    if (col_thread) {
        float* const out = p.R + bag * p.ldr + tid * CPL;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            const float v = acc[k] + beta;
            out[k] = v;
            if (kCheck) rs += (double)v;
        }
    }
    int flag = bad_wave ? ABFT_EB_BAD_INDEX : 0;
    if (kCheck) {
        rs = wave_sum(rs);
        if constexpr (W > 1) {
            if (lane == 0) s_rs[wave] = rs;
            __syncthreads();
        }
        if (tid == 0) {
            if constexpr (W > 1) {
                rs = s_rs[0];
                cs = s_cs[0];
#pragma unroll
                for (int w = 1; w < W; ++w) {
                    rs += s_rs[w];
                    cs += s_cs[w];
                    if (s_bad[w]) flag = ABFT_EB_BAD_INDEX;
                }
            }
            p.flags[bag] = flag | compare_sums(rs, cs, p.bound);
            if (p.rsum) p.rsum[bag] = rs;
            if (p.csum) p.csum[bag] = cs;
        }
    } else if (p.flags && tid == 0) {
        if constexpr (W > 1)
#pragma unroll
            for (int w = 1; w < W; ++w)
                if (s_bad[w]) flag = ABFT_EB_BAD_INDEX;
        p.flags[bag] = flag;
    }
}

template <int G, int BITS>
hipError_t launch_g(EbKernel kernel, bool check, bool weighted, const EbParams& p, hipStream_t s) {
    // one set of rows per lane only where the rows are wide and the launch has at least four wavefronts
    // per SIMD (measured at 16384 and 65536 lookups of 256 columns: 2 and 4 % faster than two sets;
    // everywhere else two sets are faster, by up to 30 % at 4096 lookups)
    const bool two_sets = G < 16 || p.n_bags * G < (int64_t)4096 * 64;
    const bool pass_by = eb_passes_by(p.stride, p.rows);
#define ABFT_EB_LAUNCH(CK, WT)                                                                                     \
    do {                                                                                                           \
        if (kernel == kEbGroup1 && pass_by) eb_group_kernel<G, BITS, 1, true, CK, WT><<<dim3((unsigned)p.n_bags), dim3(64), 0, s>>>(p);      \
        else if (kernel == kEbGroup1) eb_group_kernel<G, BITS, 1, false, CK, WT><<<dim3((unsigned)p.n_bags), dim3(64), 0, s>>>(p);      \
        else if (kernel == kEbGroup2 && pass_by) eb_group_kernel<G, BITS, 2, true, CK, WT><<<dim3((unsigned)p.n_bags), dim3(128), 0, s>>>(p); \
        else if (kernel == kEbGroup2) eb_group_kernel<G, BITS, 2, false, CK, WT><<<dim3((unsigned)p.n_bags), dim3(128), 0, s>>>(p); \
        else if (kernel == kEbGroup4) eb_group_kernel<G, BITS, 4, true, CK, WT><<<dim3((unsigned)p.n_bags), dim3(256), 0, s>>>(p); \
        else if (two_sets) eb_batch_kernel<G, BITS, CK, WT, true><<<dim3((unsigned)((p.n_bags * G + 255) / 256)), dim3(256), 0, s>>>(p); \
        else eb_batch_kernel<G, BITS, CK, WT, (G < 16)><<<dim3((unsigned)((p.n_bags * G + 255) / 256)), dim3(256), 0, s>>>(p); \
        return hipGetLastError();                                                                                  \
    } while (0)
    if (check && weighted) ABFT_EB_LAUNCH(true, true);
    if (check) ABFT_EB_LAUNCH(true, false);
    if (weighted) ABFT_EB_LAUNCH(false, true);
    ABFT_EB_LAUNCH(false, false);
#undef ABFT_EB_LAUNCH
}

template <int BITS>
hipError_t launch_bits(int code_bytes, EbKernel kernel, bool check, bool weighted, const EbParams& p, hipStream_t s) {
    switch (code_bytes) {
        case 16: return launch_g<1, BITS>(kernel, check, weighted, p, s);
        case 32: return launch_g<2, BITS>(kernel, check, weighted, p, s);
        case 64: return launch_g<4, BITS>(kernel, check, weighted, p, s);
        case 128: return launch_g<8, BITS>(kernel, check, weighted, p, s);
        case 256: return launch_g<16, BITS>(kernel, check, weighted, p, s);
        case 512: return launch_g<32, BITS>(kernel, check, weighted, p, s);
    }
    return hipErrorNotSupported;
}

hipError_t launch_eb(int code_bytes, int bits, EbKernel kernel, bool check, bool weighted, const EbParams& p, hipStream_t s) {
    return bits == 4 ? launch_bits<4>(code_bytes, kernel, check, weighted, p, s)
                     : launch_bits<8>(code_bytes, kernel, check, weighted, p, s);
}

// ---------------------------------------------------------------------------------------------
// Table build (Section V: row sums computed once), and the small helpers.
// One thread per 16-byte piece of a record; the thread of the tail piece sums the row's codes.
__global__ __launch_bounds__(256) void eb_pack_kernel(const uint8_t* T, int64_t ldt, const float* scale, const float* bias,
                                                      int64_t rows, int code_bytes, int bits, uint8_t* rec, int64_t stride) {
    const int P = code_bytes / 16 + 1;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t row = t / P;
    const int pc = (int)(t - row * P);
    if (row >= rows) return;
    const uint8_t* src = T + row * ldt;
    v4u out;
    if (pc < P - 1) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            unsigned int x = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) x |= (unsigned int)src[pc * 16 + 4 * w + b] << (8 * b);
            out[w] = x;
        }
    } else {
        int32_t sum = 0;
        for (int j = 0; j < code_bytes; ++j) sum += bits == 8 ? (int)src[j] : (int)(src[j] & 15) + (int)(src[j] >> 4);
        out[0] = __builtin_bit_cast(unsigned int, scale[row]);
        out[1] = __builtin_bit_cast(unsigned int, bias[row]);
        out[2] = (unsigned int)sum;
        out[3] = 0u;
    }
    *reinterpret_cast<v4u*>(rec + row * stride + pc * 16) = out;
}

__global__ __launch_bounds__(256) void eb_get_rowsums_kernel(const uint8_t* rec, int64_t stride, int64_t rows, int code_bytes, int32_t* C_T) {
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row < rows) C_T[row] = *reinterpret_cast<const int32_t*>(rec + row * stride + code_bytes + 8);
}

__global__ void eb_flip_kernel(uint8_t* rec, int64_t off, int bit) {
    if (threadIdx.x == 0 && blockIdx.x == 0) rec[off] = (uint8_t)(rec[off] ^ (1u << bit));
}

}  // namespace
}  // namespace abft

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) return abft::set_error(ABFT_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

extern "C" {

int abft_eb_pack_rowsum(const uint8_t* T, int64_t ldt, const float* scale, const float* bias, int64_t rows, int d,
                        unsigned flags, void* stream, abft_eb_table** out) {
    if (!T || !scale || !bias || !out) return abft::set_error(ABFT_EINVAL, "abft_eb_pack_rowsum: null pointer");
    if (rows < 1) return abft::set_error(ABFT_EINVAL, "abft_eb_pack_rowsum: rows=%lld must be >= 1", (long long)rows);
    if (flags & ~(ABFT_EB_PACK_LINE_ALIGNED | ABFT_EB_PACK_INT4)) return abft::set_error(ABFT_EINVAL, "abft_eb_pack_rowsum: unknown flag bits %#x", flags);
    const int bits = (flags & ABFT_EB_PACK_INT4) ? 4 : 8;
    const int code_bytes = d > 0 && d <= 4096 && (d * bits) % 8 == 0 ? d * bits / 8 : 0;
    if (code_bytes != 16 && code_bytes != 32 && code_bytes != 64 && code_bytes != 128 && code_bytes != 256 && code_bytes != 512)
        return abft::set_error(ABFT_EUNSUPPORTED, "abft_eb_pack_rowsum: d=%d with %d-bit codes (supported: rows of 16, 32, 64, 128, 256 or 512 bytes)", d, bits);
    if (ldt < code_bytes) return abft::set_error(ABFT_EINVAL, "abft_eb_pack_rowsum: ldt=%lld smaller than a row of %d bytes", (long long)ldt, code_bytes);
    // line-aligned: records of up to 128 bytes get a power-of-two stride, so none of them straddles a 128-byte line
    int64_t stride = code_bytes + 16;
    if ((flags & ABFT_EB_PACK_LINE_ALIGNED) && stride <= 128) stride = stride <= 32 ? 32 : (stride <= 64 ? 64 : 128);
    const int64_t pieces = rows * (code_bytes / 16 + 1);
    if ((pieces + 255) / 256 > 0x7fffffffll) return abft::set_error(ABFT_EUNSUPPORTED, "abft_eb_pack_rowsum: table too large");
    abft_eb_table* h = new (std::nothrow) abft_eb_table();
    if (!h) return abft::set_error(ABFT_EHIP, "abft_eb_pack_rowsum: out of host memory");
    std::memset(h, 0, sizeof *h);
    h->rows = rows;
    h->d = d;
    h->bits = bits;
    h->code_bytes = code_bytes;
    h->stride = stride;
    hipError_t e = hipGetDevice(&h->device);
    if (e == hipSuccess) e = hipMalloc(&h->rec, (size_t)rows * (size_t)stride);
    if (e == hipSuccess) {
        abft::eb_pack_kernel<<<dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>(
            T, ldt, scale, bias, rows, code_bytes, bits, h->rec, stride);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        (void)hipFree(h->rec);
        delete h;
        return abft::set_error(ABFT_EHIP, "abft_eb_pack_rowsum: %s", hipGetErrorString(e));
    }
    *out = h;
    return ABFT_OK;
}

int abft_eb_table_dims(const abft_eb_table* Tp, int64_t* rows, int* d, int* record_bytes, int* bits) {
    if (!Tp) return abft::set_error(ABFT_EINVAL, "abft_eb_table_dims: null handle");
    if (rows) *rows = Tp->rows;
    if (d) *d = Tp->d;
    if (record_bytes) *record_bytes = (int)Tp->stride;
    if (bits) *bits = Tp->bits;
    return ABFT_OK;
}

int abft_eb_table_get_rowsums(const abft_eb_table* Tp, int32_t* C_T, void* stream) {
    if (!Tp || !C_T) return abft::set_error(ABFT_EINVAL, "abft_eb_table_get_rowsums: null pointer");
    abft::eb_get_rowsums_kernel<<<dim3((unsigned)((Tp->rows + 255) / 256)), dim3(256), 0, (hipStream_t)stream>>>(
        Tp->rec, Tp->stride, Tp->rows, Tp->code_bytes, C_T);
    HIP_TRY(hipGetLastError());
    return ABFT_OK;
}

int abft_eb_table_flip_bit(abft_eb_table* Tp, int64_t row, int col, int bit, void* stream) {
    if (!Tp) return abft::set_error(ABFT_EINVAL, "abft_eb_table_flip_bit: null handle");
    if (row < 0 || row >= Tp->rows || col < 0 || col >= Tp->d || bit < 0 || bit >= Tp->bits)
        return abft::set_error(ABFT_EINVAL, "abft_eb_table_flip_bit: row=%lld col=%d bit=%d outside the table", (long long)row, col, bit);
    // a 4-bit code of an odd column sits in the high half of its byte
    const int64_t off = row * Tp->stride + (Tp->bits == 8 ? col : col / 2);
    const int pos = Tp->bits == 8 ? bit : bit + 4 * (col & 1);
    abft::eb_flip_kernel<<<dim3(1), dim3(64), 0, (hipStream_t)stream>>>(Tp->rec, off, pos);
    HIP_TRY(hipGetLastError());
    return ABFT_OK;
}

void abft_eb_table_destroy(abft_eb_table* Tp) {
    if (!Tp) return;
    (void)hipFree(Tp->rec);
    delete Tp;
}

int abft_eb_u8_checked(const abft_eb_table* Tp, const int64_t* indices, int64_t n_indices, const int64_t* offsets,
                       int64_t n_bags, const float* weights, float* R, int64_t ldr, int32_t* bag_flags,
                       double* rsum, double* csum, double rel_bound, unsigned flags, void* stream) {
    const char* fn = "abft_eb_u8_checked";
    if (!Tp || !offsets) return abft::set_error(ABFT_EINVAL, "%s: null pointer", fn);
    if (n_indices < 0 || n_bags < 0) return abft::set_error(ABFT_EINVAL, "%s: negative count", fn);
    if (n_bags == 0) return ABFT_OK;  // nothing to pool, nothing is written
    if (!R) return abft::set_error(ABFT_EINVAL, "%s: null pointer", fn);
    if (n_indices > 0 && !indices) return abft::set_error(ABFT_EINVAL, "%s: null indices", fn);
    if (flags & ~(ABFT_EB_NOCHECK | ABFT_EB_VARIANT_MASK)) return abft::set_error(ABFT_EINVAL, "%s: unknown flag bits %#x", fn, flags);
    const bool check = (flags & ABFT_EB_NOCHECK) == 0;
    if (check && !bag_flags) return abft::set_error(ABFT_EINVAL, "%s: bag_flags is required unless ABFT_EB_NOCHECK", fn);
    if (check && !(rel_bound >= 0.0)) return abft::set_error(ABFT_EINVAL, "%s: rel_bound must be >= 0", fn);
    if (ldr < Tp->d || ldr % 4 != 0 || (reinterpret_cast<uintptr_t>(R) & 15) != 0)
        return abft::set_error(ABFT_EINVAL, "%s: R needs ldr >= d, ldr a multiple of 4 and 16-byte alignment", fn);
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != Tp->device)
        return abft::set_error(ABFT_EINVAL, "%s: the table lives on device %d, the current device is %d", fn, Tp->device, dev);
    const unsigned variant = flags & ABFT_EB_VARIANT_MASK;
    if (variant != 0 && variant != ABFT_EB_VARIANT_BATCH && variant != ABFT_EB_VARIANT_GROUP)
        return abft::set_error(ABFT_EINVAL, "%s: unknown variant %#x", fn, variant);
    const int G = Tp->code_bytes / 16;
    const bool few = n_bags <= 0x7fffffffll;
    const abft::EbKernel kernel = variant == ABFT_EB_VARIANT_GROUP ? abft::kEbGroup4
                                  : variant == ABFT_EB_VARIANT_BATCH || !few ? abft::kEbBatch : abft::eb_pick_kernel(n_bags, n_indices, G);
    if (!few || abft::eb_work_items(kernel, n_bags, G) > abft::kEbMaxWorkItems)
        return abft::set_error(ABFT_EUNSUPPORTED, "%s: n_bags=%lld too large for one launch", fn, (long long)n_bags);
    abft::EbParams p;
    p.tab = Tp->rec;
    p.stride = Tp->stride;
    p.rows = Tp->rows;
    p.indices = indices;
    p.n_indices = n_indices;
    p.offsets = offsets;
    p.n_bags = n_bags;
    p.weights = weights;
    p.R = R;
    p.ldr = ldr;
    p.flags = bag_flags;
    p.rsum = check ? rsum : nullptr;
    p.csum = check ? csum : nullptr;
    p.bound = rel_bound;
    HIP_TRY(abft::launch_eb(Tp->code_bytes, Tp->bits, kernel, check, weights != nullptr, p, (hipStream_t)stream));
    return ABFT_OK;
}

}  // extern "C"
