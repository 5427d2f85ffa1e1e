// Internal declarations shared by the HIP translation units of libabftgemm.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace abft {

// ---- packed weight layout -----------------------------------------------------------
// B is cut into "units" of 64 k-values x 32 columns = 2 KiB, stored as
// [k-group kg 0..3][column c 0..31][16 consecutive k bytes].  A 32x32x32 int8 MFMA
// takes k-groups {2h, 2h+1} of a unit as its B operand with lane l reading the
// 16 bytes at h*1024 + l*16; a 16x16x64 MFMA takes columns 16s..16s+15 of all four
// k-groups with lane l reading (l/16)*512 + (16s + l%16)*16.  Units are ordered
// [n-tile of 256 columns][k-block of 64][unit 0..7] so that a workgroup streaming
// along K for one n-tile reads consecutive memory.  Rows k >= K and columns
// j >= N are zero, which leaves both the product and the checksum unchanged.
constexpr int kUnitK = 64;        // k-values per unit
constexpr int kUnitN = 32;        // columns per unit
constexpr int kUnitBytes = kUnitK * kUnitN;
constexpr int kTileN = 256;       // columns per packed n-tile
constexpr int kUnitsPerTile = kTileN / kUnitN;
constexpr int kLimbs = 4;         // signed base-256 digits of an int32 checksum entry

__host__ __device__ inline int64_t packed_unit_offset(int ntile, int kb, int unit, int KB) {
    return (((int64_t)ntile * KB + kb) * kUnitsPerTile + unit) * kUnitBytes;
}
// byte offset of logical B[k][j]
__host__ __device__ inline int64_t packed_elem_offset(int k, int j, int KB) {
    const int ntile = j / kTileN, unit = (j % kTileN) / kUnitN, c = j % kUnitN;
    const int kb = k / kUnitK, kg = (k % kUnitK) / 16, b = k % 16;
    return packed_unit_offset(ntile, kb, unit, KB) + (kg * kUnitN + c) * 16 + b;
}
// Checksum digits: [k-block][k-group][digit 0..3][16 k bytes]; digit d of S_B[k]
// multiplies 256^d.  Same k order as the units, so a 16x16x64 MFMA reads digit
// column d with lane l = kg*16 + d.
__host__ __device__ inline int64_t limb_offset(int k, int digit) {
    const int kb = k / kUnitK, kg = (k % kUnitK) / 16, b = k % 16;
    return (((int64_t)kb * 4 + kg) * kLimbs + digit) * 16 + b;
}

}  // namespace abft

struct abft_packed_b {
    int K, N;
    int KB;            // k-blocks of 64, rounded up to an even count (zero padded)
    int NT;            // n-tiles of 256
    int device;
    int8_t* packed;    // NT*KB*8 units
    int8_t* limbs;     // KB*64*4 bytes
    int32_t* S_B;      // [KB*64], zero past K
    int32_t* colsum;   // [NT*256], zero past N
    int32_t* total;    // [0] sum of S_B (wrap-around), [1] sum of S_B127
    int8_t* limbs127;  // as limbs, for rowSum = S_B mod 127 (digit 0 only)
    int32_t* S_B127;   // [KB*64] S_B mod 127 in [0,126], zero past K
    size_t block_bytes;   // of the block that holds all of them, which begins at `packed`; 0: not to be kept for another weight
    int32_t* sums;        // accumulators of the packing, [KB*64] for S_B and then [NT*256] for colsum: zero before a weight is packed and after
    bool sums_zero;       // they are, once what is enqueued has run
};

namespace abft {

// What the one block of a packed weight holds, by offsets in bytes.
struct PackedLayout {
    size_t limbs, limbs127, S_B, colsum, total, S_B127, sums, bytes;
};
inline PackedLayout packed_layout(int KB, int NT) {
    const auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const size_t units = (size_t)NT * KB * kUnitsPerTile * kUnitBytes, digits = (size_t)KB * kUnitK * kLimbs;
    const size_t k_ints = (size_t)KB * kUnitK * sizeof(int32_t), n_ints = (size_t)NT * kTileN * sizeof(int32_t);
    PackedLayout l;
    l.limbs = up(units);
    l.limbs127 = l.limbs + up(digits);
    l.S_B = l.limbs127 + up(digits);
    l.colsum = l.S_B + up(k_ints);
    l.total = l.colsum + up(n_ints);
    l.S_B127 = l.total + 256;
    l.sums = l.S_B127 + up(k_ints);
    l.bytes = l.sums + k_ints + n_ints;
    return l;
}

struct RequantDev {
    int32_t zA, zC;
    const float* mult;
    int32_t per_channel;
    const int32_t* bias;
};

#ifdef __HIPCC__
// Requantization of one 32-bit value (Section III-B with the rank-1 correction of Eq. 1 for a
// symmetric B): t = v - zA * colsum (+ bias) in wrap-around int32, one binary32 multiply, round
// to nearest even, + zC, clamp to [0, 255].  The one place this arithmetic is written down.
// What a column contributes, fetched once per column: colsum * zA - bias as one wrap-around term, and the
// multiplier (a kernel that stores between two uses would otherwise have to fetch them again every time).
struct RequantCol {
    uint32_t sub;   // zA * colsum - bias (mod 2^32)
    float mult;
};
__device__ inline RequantCol requant_col(int32_t cs, int col, const RequantDev& rq) {
    RequantCol c;
    c.sub = (uint32_t)rq.zA * (uint32_t)cs;
    if (rq.bias) c.sub -= (uint32_t)rq.bias[col];
    c.mult = rq.mult[rq.per_channel ? col : 0];
    return c;
}
// the rounded and clamped value, a whole number in [0, 255]
__device__ inline float requant_float(int32_t v, const RequantCol& c, int32_t zC) {
    const uint32_t t = (uint32_t)v - c.sub;
    const float p = __fmul_rn((float)(int32_t)t, c.mult);
    const float y = __builtin_rintf(p) + (float)zC;
    return __builtin_amdgcn_fmed3f(y, 0.0f, 255.0f);   // (clamped; a NaN gives 0, as min(max(y, 0), 255) does)
}
__device__ inline uint8_t requant_with(int32_t v, const RequantCol& c, int32_t zC) { return (uint8_t)requant_float(v, c, zC); }
// ... as byte `row` of w
__device__ inline uint32_t requant_into(uint32_t w, int row, int32_t v, const RequantCol& c, int32_t zC) {
    return __builtin_amdgcn_cvt_pk_u8_f32(requant_float(v, c, zC), row, w);
}
// The matrix cores leave four rows of one column in a lane and neighbouring columns in neighbouring lanes, so that bytes would
// go to memory one at a time.  Here the four lanes of a quad turn their 4x4 bytes: byte r of lane c becomes byte c of lane r,
// and one store writes four columns of the row that the lane now holds.
__device__ inline uint32_t turn_quad(uint32_t w, int lane) {
    const uint32_t p1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, true);   // lane ^ 1
    const uint32_t x = __builtin_amdgcn_perm(p1, w, (lane & 1) ? 0x03070105u : 0x06020400u);      // rows 0 and 2 / 1 and 3, two columns
    const uint32_t p2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true);   // lane ^ 2
    return __builtin_amdgcn_perm(p2, x, (lane & 2) ? 0x03020706u : 0x05040100u);
}
typedef uint32_t u32_any __attribute__((aligned(1)));
__device__ inline void store_quad_nt(uint8_t* p, uint32_t w) { __builtin_nontemporal_store(w, reinterpret_cast<u32_any*>(p)); }
// four bytes of a row at any address, of which the first n (at least one, at most four) exist
__device__ inline void store_quad(uint8_t* p, uint32_t w, int n) {
    if (n >= 4) {
        *reinterpret_cast<u32_any*>(p) = w;
    } else {
#pragma unroll
        for (int b = 0; b < 3; ++b)
            if (b < n) p[b] = (uint8_t)(w >> (8 * b));
    }
}
__device__ inline uint8_t requant_one(int32_t v, int32_t cs, int col, const RequantDev& rq) {
    return requant_with(v, requant_col(cs, col, rq), rq.zC);
}
#endif

struct GemmParams {
    const uint8_t* A;
    int64_t lda;
    int M, N, K, KB;           // KB: k-blocks of 64 in the packed weight (even)
    int KB2;                   // stages of 128 k-values = KB / 2
    int a_vec_ok;              // A and lda are multiples of 16 bytes
    int mod127;                // compare modulo 127 (Algorithm 1 as printed) instead of 2^32
    int err_accumulate;        // flagged rows are added to *err_count instead of overwriting it
    int share_q, share_r;      // the checksum product's K range (stages or k-blocks) is dealt out to the tile columns /
                               // column blocks of the grid: block c takes share_q units, the first share_r blocks one more
                               // (set by the launcher: a division by a run-time count costs a kernel hundreds of cycles)
    const int8_t* packed;
    const int8_t* limbs;
    const int32_t* colsum;
    const int32_t* total;
    int32_t* C;
    int64_t ldc;
    int32_t* row_flags;
    int32_t* err_count;
    uint8_t* Cq;
    int64_t ldcq;
    RequantDev rq;
    const void* inj;           // abft_inject_t[n_inj]
    int n_inj;
    int ksplit;                // K slices across workgroups (split-K kernels; 1 elsewhere)
    int split_q, split_r;      // stages of a slice; the first split_r take one more
    int32_t* ws_tickets;       // split-K: one arrival counter per tile (and finishing wavefront)
    int32_t* ws_part;          // split-K: parts, [tile][slice][value][thread] or [tile][finishing wavefront][slice][value][lane]
    int wk_stages;             // K split among wavefronts: stages of the wavefronts with fewest; those with one more deal out
    int wk_stream;             // ... the weight is not kept in the caches
    union {   // (shared places: with the other members anywhere else a kernel's first loads fall apart, 0.1 to 0.2 us of a short call)
        struct {
            int wk_share_q1, wk_share_r1;   // their k-steps of the checksum product by these instead of share_q, share_r
        };
        struct {
            int slots, slot_rows;           // 64x64 tiles: the words between the arrivals of many tile columns and a row's word (RowSlots)
        };
    };
    size_t ws_ints;            // ints the caller's workspace holds
    unsigned long long* clock_trace;  // diagnostic builds (ABFT_CLOCK_TRACE): 6 words per workgroup, else NULL
    int32_t* ws;               // workspace: counting words in the first kWsHeaderInts ints, then the per-row words
};

constexpr int kWsHeaderInts = 64;
constexpr int kWsDoneSlots = 16;    // 64-bit words at the start of the header where many reports of finished rows meet first
constexpr int kWsDoneWord = 48;     // int offset, inside the header, of the 64-bit word that counts finished rows (low half)
                                    // and corrupted ones among them (high half)
// the streaming kernel spreads its per-row sums over kSmallMSlots slots of kSmallMRows rows
constexpr int kSmallMSlots = 32;
constexpr int kSmallMRows = 64;

// ints of workspace the row words and counting words of a problem with M rows take
inline size_t ws_base_ints(int M) {
    const size_t rows = 2 * ((((size_t)M + 63) / 64) * 64);  // one 64-bit word per row
    // streaming kernel: one 64-bit word per (slot, row) and one per row
    const size_t streaming = 2 * ((size_t)kSmallMSlots * kSmallMRows + kSmallMRows);
    return (size_t)kWsHeaderInts + (rows > streaming ? rows : streaming);
}

// Arrivals of tile columns at a row's word follow each other at 10 to 20 ns.  From 49 tile columns on (never fewer than slots), and as long as
// the words that every call has (2112) hold the slots' too, they meet in slots first: 32 of them for up to 64 rows, 8 for up to 192, 4 for up to 384 (us,
// directly / by slots, 32x32 tiles: 41 columns, 60x1300x128 4.5 / 4.7; 63, 20x2000x900 5.0 / 4.7; 125, 20x3985x848 5.7 / 4.7; 32x64 tiles, 284 columns,
// 29x9088x1872 7.9 / 6.1; 64x64 tiles, 150 columns, 147x9536x112 7.8 / 6.1, 125, 200x8000x128 7.6 / 6.1, 234, 93x14960x2640 21.5 / 18.4).
struct RowSlots {
    int slots, rows;   // (0: none) and the words of a slot
};
inline RowSlots row_slots(int M, int tiles_n) {
    if (tiles_n <= 48 || M > 384) return {0, 0};
    const int rows = (M + 63) / 64 * 64;
    int slots = 32;
    while ((slots + 1) * rows > kSmallMSlots * kSmallMRows + kSmallMRows) slots /= 2;
    return {slots, rows};
}

// What some calls need beyond those words - the tile tickets and partial tiles of a K split, a copy of A with padded rows -
// lies behind the words of any call of up to kWsRows rows, so that one workspace can serve calls of different sizes: the
// words (tickets among them) are zero between calls, the scratch behind them holds whatever the last call left (a call of more
// rows, whose words reach into it, zeroes that part first: launch_gemm_tile).
constexpr int kWsRows = 131072;
constexpr size_t kWsTicketsOff = (size_t)kWsHeaderInts + 2 * (size_t)kWsRows;
constexpr size_t kWsTickets = 1024;
constexpr size_t kWsScratchOff = kWsTicketsOff + kWsTickets;

// Split-K across workgroups (32x32 tiles of gemm_tile_wk.h, grids that would leave most compute units idle): how many K slices,
// and where the tickets and the parts lie in the workspace behind the row words.  One place for the rule, so that
// abft_gemm_workspace_bytes and the launcher agree.
constexpr int kWkPartInts = 4 * 64 * 5;   // per workgroup: four finishing wavefronts x 64 lanes x (four sums and a checksum share)
struct SplitKPlan {
    int z;                                  // slices (1 = no split)
    size_t tickets_off, part_off, total_ints;
    size_t room_ints;                       // for any way the rows of A may lie
};
inline SplitKPlan splitk_plan(int M, int N, int stages, bool whole_a) {
    SplitKPlan pl;
    const int64_t tiles = (int64_t)((M + 31) / 32) * ((N + 31) / 32);
    pl.z = 1;
    // The parts meet through memory (the L2s are not coherent with each other): store them, wait for the acknowledgement, take the
    // ticket, fetch the others' - three dependent device-scope round trips, about 2 us.  A workgroup of eight wavefronts takes
    // eight stages in 0.4 us, 0.85 us where rows are no whole chunks, so slices of sixteen stages pay from 64 stages on, or 36 (us,
    // unsplit / split: 46x128x13504 10.6 / 8.1, 64x64x16384 11.9 / 8.2, 96x96x10000 9.0 / 7.8, 100x1000x8192 in two 8.2 / 9.5;
    // rows that are no whole chunks, 32x240x12600 11.2 / 7.7, 45x1000x5001 8.9 / 7.8, 41x1000x3071 in two slower), and where there
    // are eight tiles at most from 24 (65x64x6144 7.0 / 6.8, 128x64x3072 5.6 / 6.4).  Two or three slices pay for weights that are not in the
    // caches: unsplit, too few workgroups fetch (one weight again and again / fresh ones, unsplit and split: 32x3000x12000 13.0 20.1 / 11.2
    // 14.9, 16x4096x16000 13.6 19.3 / 15.1 15.9, 64x1100x12000 10.1 18.0 / 9.0 11.2, 64x1500x9008 9.0 15.0 / 9.8 11.9, 256x500x12000 10.2 15.0 /
    // 10.8 12.2, 1280x80x16176 18.1 19.2 / 15.2 15.0), not where many rows of tiles meet many columns, which are busy enough (100x1000x12000
    // 10.2 13.5 / 13.1 13.3, 128x1000x12000 10.2 16.6 / 13.5 13.7, 33x2000x12000 10.6 14.0 / 13.4 13.5).  How the rows lie is known when the
    // call comes; there is room in the workspace for either.
    const bool room = M <= kWsRows && tiles <= 128 && stages >= (M > 40 ? 24 : 40);
    if (room && (whole_a ? (tiles <= 64 && stages >= 64) || (tiles <= 8 && M > 40) || (stages >= 70 && (M <= 32 || tiles <= 96 || N <= 768))
                         : stages >= 36)) {
        const int64_t most = (stages + 15) / 16, fit = 256 / tiles;
        pl.z = (int)(most < fit ? most : fit);
        if (pl.z > 16) pl.z = 16;
    }
    pl.tickets_off = kWsTicketsOff;   // (at most 128 tiles are split)
    pl.part_off = kWsScratchOff;
    pl.total_ints = pl.z > 1 ? pl.part_off + (size_t)tiles * pl.z * kWkPartInts : ws_base_ints(M);
    pl.room_ints = room ? pl.part_off + (size_t)(tiles * (256 / tiles < 16 ? 256 / tiles : 16)) * kWkPartInts : ws_base_ints(M);
    return pl;
}

// The split of 64x64 tiles (gemm_tile_async.h): 33 to 64 rows, whose weight these tiles read once, or any number where the 32x64 tiles of
// gemm_tile_wk.h would leave near half of the compute units idle (65 to 85 tiles of 64x64, too many of 32x32), and a K so long that the
// slices' meeting is paid for.  Its 256 workgroups keep more of a weight in flight than the fewer ones of gemm_tile_wk.h with 32 or 64
// columns, which counts where the weight is not in the caches; where the line lies depends on how many of those there are (us, one weight
// again and again / fresh ones; gemm_tile_wk.h, then this split): 64x4200x9008 15.4 22.0 / 14.5 17.5, 64x5000x16000 21.0 30.5 / 19.8 22.7,
// 33x5000x9008 14.5 17.8 / 16.7 16.2, 33x4200x12000 17.8 21.0 / 16.3 17.4, 64x3000x12000 14.3 19.3 / 14.6 16.4, 64x2000x16000 15.1 19.4 /
// 14.5 14.5, 64x6500x16000 22.4 32.5 / 24.2 28.3; but 64x5000x6000 11.4 16.6 / 12.7 14.5, 33x3000x12000 13.3 15.4 / 14.3 16.5, 64x2000x9008
// 9.1 16.0 / 11.5 12.8, 64x6500x9008 16.4 22.9 / 17.7 22.6, 64x1000x16000 10.7 12.5 / 12.5 14.5.  More rows: 164x1440x15312 23.0 24.6 /
// 20.7 20.6, 746x339x14848 19.7 21.3 / 18.0 18.2, 1100x250x12000 19.0 20.0 / 16.5 16.8; but 192x1500x9008 15.1 / 15.7, 128x3000x12000 17.9 24.0 /
// 20.0 24.6, and with fewer than 257 tiles of 32x32 130x1400x11600 14.3 14.6 / 17.6 17.5.
constexpr int kSplit64PartInts = 256 * 17 + 64;   // per workgroup: 256 threads x (16 accumulator values + 1 column sum), 64 rows' checksum shares
struct Split64Plan {
    int z;                // slices (1 = no split)
    size_t total_ints;    // tickets from kWsTicketsOff on, parts from kWsScratchOff on
};
inline Split64Plan split64_plan(int M, int N, int stages) {
    Split64Plan pl = {1, ws_base_ints(M)};
    if (M <= 32 || stages < 60) return pl;
    const int64_t tiles = ((int64_t)M + 63) / 64 * (((int64_t)N + 63) / 64);
    const int64_t t32 = ((int64_t)M + 31) / 32 * (((int64_t)N + 31) / 32);
    const bool third = tiles > 64 && tiles <= 85 && t32 > 256;   // (three slices)
    const int line = tiles <= 20 || tiles > 128 ? 1 << 30 : third ? (M > 64 ? 90 : 60) : tiles > 32 && tiles <= 64 && M > 48 ? 90 : 120;
    if ((M <= 64 || third) && stages >= line) {
        const int most = (int)(256 / tiles), z = stages >= 160 ? 16 : 8;
        pl.z = z < most ? z : most;
    }
    if (pl.z > 1) pl.total_ints = kWsScratchOff + (size_t)tiles * pl.z * kSplit64PartInts;
    return pl;
}

// Rows of A that are no whole, aligned 16-byte chunks (K no multiple of 16, or such a base or leading dimension): either the
// 64x64 kernel with loads through registers takes them as they lie, or a copy with padded rows is made first, in the
// workspace, for the direct-to-LDS kernels (grids that gemm_tile_wk.h does not take).  The copy costs
// about 3 us (a launch and a pass over A); the loads through registers cost 0.2-0.3 us more for every stage that a compute
// unit works through, and the large tiles are out of reach, so the copy pays from about twenty stages per unit on
// (measured in us, loads through registers / copy:
// 2000x1000x1001, 16 stages per unit, 11.5 / 11.8; 256x512x2049, 17, 10.8 / 11.4; 1111x3333x777, 28, 16.5 / 14.9;
// 1000x1000x4097, 33, 20.3 / 16.9; 4096x2048x1023, 64, 30.2 / 23.1; 4096x4096x4095, 512, 148 / 74).
// abft_gemm_workspace_bytes includes the room when K is no multiple of 16 and the copy may be made (copies above 512 MiB
// are not): where the choice is the library's own, beyond the grids of gemm_tile_wk.h, ahead of its 64x64 form (copy_first) and of the
// split of 64x64 tiles, none of which up to 40 rows and 4096 columns and k are; elsewhere the room serves calls that ask for a tile.
// A workspace without it runs without the copy.
struct RealignPlan {
    bool copy;
    size_t off, total_ints;    // ints into the workspace; the copy starts on the next 16-byte boundary
    int64_t lda;               // bytes of a padded row
};
inline RealignPlan realign_plan(int M, int N, int K, int stages) {
    RealignPlan pl;
    const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
    pl.lda = ((int64_t)K + 15) / 16 * 16;
    pl.copy = (tiles + 255) / 256 * stages >= 20 && M <= kWsRows && pl.lda * M <= (512ll << 20);
    // (behind the parts of a K split: with 64x64 tiles asked for, the padded rows may be multiplied in slices that store their
    // parts while others still read the copy)
    const SplitKPlan sk = splitk_plan(M, N, stages, true);
    const Split64Plan s64 = split64_plan(M, N, stages);
    pl.off = s64.z > 1 ? s64.total_ints : kWsScratchOff;
    if (sk.z > 1 && sk.total_ints > pl.off) pl.off = sk.total_ints;
    pl.total_ints = pl.off + (size_t)(pl.lda * M / 4) + 4;
    return pl;
}
inline bool room_for_copy(int M, int N, int K) { return K % 16 != 0 && (M > 40 || (M > 32 && (N > 4096 || K > 4096))); }

// first unit of block c's share (see share_q, share_r)
__host__ __device__ inline int share_begin(int c, int q, int r) { return c * q + (c < r ? c : r); }

#ifdef __HIPCC__
// The sixteen bytes of v (four 32-bit words) moved down by n places, zeros coming in; n is 1..15.  For the end
// of a row whose length is no multiple of 16: its last sixteen bytes, loaded as they lie,
// become the last chunk.
typedef int shift_v4i __attribute__((ext_vector_type(4)));
__device__ inline shift_v4i shift_down(shift_v4i v, int n) {
    const uint64_t lo = ((uint64_t)(uint32_t)v.y << 32) | (uint32_t)v.x, hi = ((uint64_t)(uint32_t)v.w << 32) | (uint32_t)v.z;
    uint64_t l, h;
    if (n < 8) {
        l = (lo >> (8 * n)) | (hi << (64 - 8 * n));
        h = hi >> (8 * n);
    } else {
        l = hi >> (8 * n - 64);
        h = 0;
    }
    return shift_v4i{(int)(uint32_t)l, (int)(uint32_t)(l >> 32), (int)(uint32_t)h, (int)(uint32_t)(h >> 32)};
}
#endif

// Up to 16 rows (one block of the streaming kernel) where that kernel is the better one for a weight that the program has not just used.
// It has a batch of 2048 k of its 16 or 32 columns in flight at once; the wavefronts of gemm_tile_wk.h have 512 or 1024 k of 32 or 64
// columns, and wait once per round for what the caches do not hold.  So the lines lie by the stages of 128 k, where the mean of three
// states favours it: one weight again and again, eight in turn, fresh ones (us each, streaming / gemm_tile_wk.h):
//  * whole chunks: 1x800x2048 4.2 4.3 4.2 / 4.4 4.5 5.3, 1x800x3200 5.0 5.1 5.0 / 4.8 5.0 6.1, 1x832x5312 6.0 6.2 6.0 / 5.6 6.1 7.6, 4x774x5280
//    6.0 6.4 6.2 / 5.8 6.4 7.9, 4x4096x4096 5.5 6.7 6.7 / 5.7 6.3 7.7, 8x2048x4096 5.4 6.3 6.2 / 5.6 6.1 7.3, 1x3500x12000 10.3 10.9 11.0 / 11.1
//    12.6 12.6, 8x12000x1024 4.9 5.9 6.0 / 4.9 6.1 6.9, 1x15000x3008 9.9 10.7 10.7 / 10.4 11.8 12.1; but 8x3000x16000 14.1 14.3 14.4 / 10.2 14.3
//    14.1, 1x800x2560 5.0 5.3 5.2 / 4.4 4.7 5.9, 8x3000x6400 8.4 8.9 8.8 / 6.4 7.3 9.4, 8x800x6400 6.9 8.1 7.9 / 6.0 6.8 8.6, 16x4096x4096 6.5
//    7.5 7.6 / 5.7 6.3 8.0, 4x12000x1152 6.2 / 5.1, 8x15000x5008 15.5 / 14.3
//  * 9 to 16 rows, few or middling columns: 10x464x4064 4.9 / 5.4, 1x145x6128 6.0 / 6.4, 16x4096x2048 4.8 / 5.0; but 16x1200x2048 even,
//    13x144x11067 16.6 / 7.8
//  * rows that are no whole chunks, which the streaming kernel loads row by row: one row 1x300x2001 4.4 / 5.0, 1x800x3201 5.6 5.8 5.8 /
//    5.6 6.0 7.9, 1x800x1001 4.5 4.6 4.4 / 4.3 4.3 5.2, 1x6001x9001 13.0 / 13.4 and fresh 13.4 / 15.8; up to 8 rows of one batch 4x300x2001
//    4.7 / 5.0 and fresh 4.7 / 5.5, 8x8192x1001 4.8 5.6 5.5 / 4.7 5.9 6.4; but 4x800x3201 7.2 / 5.7, 8x3000x2049 8.6 / 5.4, 1x800x2561 and
//    1x8192x16383 even, 1x800x500 4.6 / 3.7
inline bool few_rows_stream(int M, int N, int stages, bool whole_a) {
    if (M > 16 || N >= 16384) return false;
    if (M <= 8 && N > 4096 && (stages == 7 || stages == 8)) return true;
    if (!whole_a) {
        if (N <= 4096 && M <= 8 && stages <= 16) return stages >= (M == 1 ? 8 : 13);
        return M == 1 && (N <= 4096 ? stages <= 32 || (N > 2048 && stages >= 70) : stages >= 48 && stages < 96);
    }
    if (N > 4096) return M <= 8 && N > 12288 && stages >= 24 && stages <= (M <= 4 ? 48 : 32);
    if (stages <= 8) return false;
    if (N <= 640) return stages < 64;
    if (N <= (M == 1 ? 2500 : 1000) && M <= 4 && stages > 40 && stages <= 48) return true;
    if (N <= 1500) return M <= 8 && (stages <= 16 || (stages > 24 && stages <= 32));   // (the last batch at least half full)
    return stages <= 20 || (M <= 8 && (stages <= 32 || (stages >= 72 && N > (M <= 4 ? 2816 : 3264))));
}

// Which form of gemm_tile_wk.h (K split among the wavefronts of a workgroup) takes a call, if any: rows x columns of the tile, wavefronts.
enum WkForm { kWkNone = 0, kWk32x32w4, kWk32x32w8, kWk32x64w4, kWk32x64w8, kWk64x64w4 };
// By the number of tiles and of stages of 128 k (us, the 64x64 tiles of gemm_tile_async.h or up to 32 rows the streaming kernel / this form):
//  * as long as no compute unit has two: 32x32 tiles, eight wavefronts from nine stages on (441x479x1255 8.7 / 5.2, with four 5.3;
//    322x306x80 4.8 / 4.3, with four 4.2);
//  * then 32x64 tiles (674x480x2048 7.8 / 5.7; 1246x204x3856 10.5 / 7.4 with eight wavefronts, 7.6 with four);
//  * then 64x64 tiles where the loop is long enough to pay for the sums at the end (1000x1000x3200 10.1 / 9.6, but 2537x352x1200
//    8.4 / 8.9);
//  * up to two 32x64 tiles per compute unit for a short K where 64 rows a tile are partly padding or the rows are no whole chunks
//    (78x6549x96 7.4 / 6.7, 65x9664x688 9.2 / 6.6, 2042x336x146 6.0 / 4.8; but 773x928x240 5.4 / 5.5);
//  * up to two 64x64 tiles for such rows (2000x1000x479 both outputs 10.9 / 9.4, 900x2000x777 11.1 / 9.9, 600x3000x250 8.9 / 8.1;
//    576 tiles, 1500x1500x700 12.2 / 14.3);
//  * not for one stage (two from 2560 rows on) of more than 1024 rows where the tiles of 64x64 are half as many: their rows are reported in one
//    step instead of two, and of up to 64 columns without meeting other columns (3000x64x128 4.6 / 5.0, 2739x80x112 5.0 / 5.4, 3000x128x256
//    5.2 / 5.5, 1056x300x128 4.8 / 5.0; but 1500x128x112 4.8 / 4.8, 2100x100x256 5.3 / 5.3, 1056x64x256 4.8 / 4.7).
inline WkForm wk_form(int M, int N, int stages, bool whole_a) {
    const int64_t t32 = (int64_t)((M + 31) / 32) * ((N + 31) / 32), t3264 = (int64_t)((M + 31) / 32) * ((N + 63) / 64),
                  t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
    if (few_rows_stream(M, N, stages, whole_a)) return kWkNone;
    if (whole_a && M > 1024 && stages <= (M > 2560 ? 2 : 1) && (t32 > 256 || (N > 32 && N <= 64))) return kWkNone;
    if (t32 <= 256) return stages >= 9 ? kWk32x32w8 : kWk32x32w4;
    if (t3264 <= 256) return stages >= 24 ? kWk32x64w8 : kWk32x64w4;
    if (t64 <= 256 && stages >= 12) return kWk64x64w4;
    if (t3264 <= 512 && stages < 12 && (!whole_a || M <= 128)) return kWk32x64w4;
    if (!whole_a && t64 <= 512 && stages <= 10) return kWk64x64w4;
    return kWkNone;
}

// Rows that are no whole chunks, where the form is the one of 64x64 tiles and the loop is long: with room in the workspace the copy with padded
// rows is made first and multiplied (us, through registers / copied first: 100x5000x3001 12.5 / 12.0, 64x12000x5001 20.0 / 17.9,
// 256x3000x5001 17.9 / 16.9, 128x6500x9001 30.4 / 24.6, 200x4096x9001 30.8 / 24.7; but 256x4096x3001 13.1 / 13.5, 100x5000x2001 10.4 / 12.8).
inline bool copy_first(WkForm form, int stages) { return form == kWk64x64w4 && stages >= 32; }

// Grids of more tiles than compute units, beyond those for which wk_form has a rule of its own: what the kernels take there, in us, as fits of
// about 220 products with rows of whole chunks and 110 without (sizes, outputs and ratios of the sides at random, up to 4096 rows and 16384 columns, one
// weight again and again and fresh ones), 7 to 9 % off in the root mean square.  A kernel's time is a fixed part; its stages of 128 k, each at the rate at
// which a compute unit works through the tiles it has, but no less than the wait for one; the end of its tiles by what they store; and a little for every
// row and column (arrivals, reports).  Tiles of 128 and 256 run one to a compute unit in full rounds; the smaller ones several at a time, and hardly in
// rounds, except for the 64x64 form of gemm_tile_wk.h, two of which fill a unit: a few tiles more than that work through a long K alone (us, the fit,
// measured, and the 128x128 tiles: 513 tiles 524x3629x9632 45.0 52.1 43.1, 520 294x6603x13984 63.6 74.6 62.6, 540 190x11472x9376 Cq 46.2 52.0 45.0).
struct FormCost {
    float fixed, stage, wait, end_c, end_q, end_both, per_row, per_col;
};
enum LargeForm { kLarge256 = 0, kLarge128, kLarge64, kLargeWk32x64, kLargeWk64x64 };
constexpr FormCost kWholeCost[5] = {{-5.95f, 1.283f, 0.409f, 21.4f, 21.0f, 29.8f, 0.60e-3f, 0.136e-3f}, {1.57f, 0.549f, 0.537f, 4.69f, 5.17f, 6.88f, 0.35e-3f, 0.239e-3f},
                                    {4.25f, 0.293f, 0.512f, 0.87f, 0.66f, 1.29f, -0.12e-3f, 0.041e-3f}, {3.88f, 0.163f, 0.293f, 0.66f, 0.58f, 0.84f, 0.22e-3f, 0.058e-3f},
                                    {3.73f, 0.249f, 0.401f, 1.48f, 1.37f, 1.87f, 0.25e-3f, 0.061e-3f}};
// rows that are no whole chunks, taken as they lie (gemm_tile_g64.hip and the forms of gemm_tile_wk.h)
constexpr FormCost kAnyCost[3] = {{4.09f, 0.407f, 0.866f, 0.90f, 0.99f, 1.55f, -0.08e-3f, 0.027e-3f}, {4.17f, 0.198f, 0.339f, 0.72f, 0.73f, 0.90f, 0.10e-3f, 0.002e-3f},
                                  {4.42f, 0.353f, 0.355f, 1.55f, 1.53f, 2.11f, 0.21e-3f, -0.008e-3f}};
constexpr float kCopyFixed = 3.8f, kCopyPerByte = 0.25e-6f;   // the copy with padded rows ahead of a kernel
inline float form_us(const FormCost& c, LargeForm f, int M, int N, int stages, bool want_c, bool want_q) {
    const int bm = f == kLarge256 ? 256 : f == kLarge128 ? 128 : f == kLargeWk32x64 ? 32 : 64, bn = f == kLarge256 ? 256 : f == kLarge128 ? 128 : 64;
    const int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    float rounds = f <= kLarge128 ? (float)((tiles + 255) / 256) : (float)tiles / 256;
    if (f == kLargeWk64x64 && tiles > 512 && tiles < 560) rounds += 0.4f;
    const float work = rounds * stages * c.stage, wait = stages * c.wait, end = want_c && want_q ? c.end_both : want_c ? c.end_c : c.end_q;
    return c.fixed + (work > wait ? work : wait) + (rounds > 1 ? rounds : 1) * end + (M < 4096 ? M : 4096) * c.per_row + (N < 16384 ? N : 16384) * c.per_col;
}
struct LargeChoice {
    LargeForm form;
    bool copy;   // rows that are no whole chunks: copied with padded rows first
};
// (calls of more rows than kWsRows, part of whose words has to be zeroed first, are the tiled kernels' alone)
inline bool beyond_wk_form(int M, int N, int stages) {
    const int64_t t32 = (int64_t)((M + 31) / 32) * ((N + 31) / 32), t3264 = (int64_t)((M + 31) / 32) * ((N + 63) / 64), t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
    return M > 32 && M <= kWsRows && t32 > 256 && t3264 > 256 && !(t64 <= 256 && stages >= 12);
}
// The cheapest by that; `pick`, which older thresholds on tiles and K choose, unless another one is cheaper by more than the fits are off: 10 %,
// unchecked 15 % (the fits are of checked calls), and 15 % for rows that are no whole chunks where those lie within a measured line of wk_form
// (of 50 products there for which the fits promise 5 to 15 % six are 6 to 15 % slower, 0.955 in the mean: 209x8035x1218 Cq 11.1 / 12.4, 474x3836x206 C and Cq 8.0
// / 9.0, 151x10871x168 Cq 7.2 / 7.9; 2086x497x66 Cq 7.2 / 5.8).
// Nor where 256x256 tiles store more than the 256 MiB that the memory-side cache holds, or C alone of more than 128 MiB in rows of more than 12288
// columns: there the time is that of memory, which takes the pieces of 1024 bytes of a row that these tiles store at 3.5 to 4.2 TB/s, the smaller
// tiles' 256 at 2.7 to 3 (256x256 / 64x64: 16400x8240x96 130 / 197, 32800x4120x240 181 / 239, 8200x16480x80 C and Cq 186 / 219, 2824x15456x112 50 / 58,
// 2753x20128x256 72 / 84; but 16400x4120x96, 258 MiB, 1.25 times as fast on 64x64 tiles, and 2100x16480x96, 132 MiB, 1.04).
// Of 560 products of random sizes whose kernel the fits alone would change, up to 130000 rows or columns among them, these lines leave 421; they take
// 0.73 of the thresholds' time in the geometric mean, two of them more than 5 % longer (2111x6067x96 Cq 17.5 / 19.9, 328x127312x777 C and Cq
// 151 / 160).  Drawn afterwards, with these lines: 260 changed, 0.76, two (2099x42736x75 Cq 112 / 123, 653x14644x132 Cq 21.2 / 23.9); of 100 unchecked ones
// 0.78 and four (871x9296x2112 34.8 / 40.5, 785x9216x352 11.4 / 12.9, 1316x5440x1504 Cq 27.0 / 29.9, 280x6075x1721 14.3 / 15.5).
// (us, thresholds / now: 214x4369x2434 19.1 / 12.0, 2545x7104x528 C and Cq 87 / 40, 3350x2688x288 C and Cq 31.5 / 19.4, 90x8237x3824 Cq 23.8 /
// 15.8, 1664x13552x112 C and Cq 60.5 / 29.4, 48x95360x192 Cq 44.4 / 10.8, 71348x106x448 Cq 61.6 / 26.5, 11346x85x7186 60.6 / 35.9.)
inline LargeChoice large_choice(LargeChoice pick, bool whole_a, bool can_copy, int M, int N, int K, int stages, bool want_c, bool want_q, bool check = true) {
    const int64_t stored = (int64_t)M * N * ((want_c ? 4 : 0) + (want_q ? 1 : 0));
    if (pick.form == kLarge256 && (stored > (256ll << 20) || (N > 12288 && !want_q && stored > (128ll << 20)))) return pick;
    LargeChoice best = pick;
    float least = 0, own = 0;
    bool any = false;
    auto look = [&](const FormCost& c, LargeForm f, bool copy, float more) {
        const float t = form_us(c, f, M, N, stages, want_c, want_q) + more;
        if (f == pick.form && copy == pick.copy) own = t;
        if (!any || t < least) {
            least = t;
            best = {f, copy};
            any = true;
        }
    };
    if (!whole_a && K >= 16) {
        if (!pick.copy) look(kAnyCost[0], kLarge64, false, 0);   // (where the copy is worth more than that: realign_plan)
        look(kAnyCost[1], kLargeWk32x64, false, 0);
        look(kAnyCost[2], kLargeWk64x64, false, 0);
    }
    if (whole_a || can_copy)
        for (int f = 0; f < 5; ++f) look(kWholeCost[f], (LargeForm)f, !whole_a, whole_a ? 0.0f : kCopyFixed + kCopyPerByte * (float)M * (float)K);
    const float line = !check || (!whole_a && pick.form >= kLargeWk32x64) ? 0.85f : 0.9f;
    return any && least < line * own ? best : pick;
}

enum Variant { kTile256 = 1, kTile128 = 2, kTile64 = 3, kSmallM = 4, kTile256w24 = 5, kTile256w42 = 6, kVariantEnd = 7 };

// launchers (each returns the hipError_t of its launch)
hipError_t launch_pack(const int8_t* B, int64_t ldb, int transposed, abft_packed_b* h, hipStream_t s);
hipError_t launch_flip_bit(abft_packed_b* h, int k, int j, int bit, hipStream_t s);
hipError_t launch_flip_checksum_bit(abft_packed_b* h, int k, int bit, hipStream_t s);
hipError_t launch_flip_checksum127_bit(abft_packed_b* h, int k, int bit, hipStream_t s);
hipError_t launch_fill_zero(int32_t* p, size_t n_ints, hipStream_t s);
// (refuses what it does not take: a form of kWkNone, K below 16 with rows that are no whole chunks, the printed modulus on such rows)
hipError_t launch_gemm_wk(WkForm form, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s);
// (refuses where split64_plan has none, the workspace has no room for it, or A is not in whole, aligned chunks)
hipError_t launch_gemm_split64(bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s);
hipError_t launch_gemm_tile(int variant, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s);
// any_a: A of any alignment and K >= 16 is taken too (else only whole, aligned 16-byte chunks)
hipError_t launch_gemm_smallm(bool any_a, bool check, bool want_c, bool want_q, const GemmParams& p, hipStream_t s);
// A's rows copied to rows of lda2 bytes (a multiple of 16), zeros behind K
hipError_t launch_realign(const uint8_t* A, int64_t lda, int M, int K, uint8_t* A2, int64_t lda2, hipStream_t s);
hipError_t launch_requantize(const int32_t* C, int64_t ldc, int M, int N, const int32_t* colsum,
                             const RequantDev& rq, uint8_t* Cq, int64_t ldcq, hipStream_t s);
hipError_t launch_verify_rows(const int32_t* C, int64_t ldc, int M, int N, const int32_t* row_chk,
                              int32_t* row_flags, int32_t* err_count, hipStream_t s);
hipError_t launch_list_flagged(const int32_t* flags, int M, int32_t* idx, int32_t* count, hipStream_t s);
hipError_t launch_gather_rows(const uint8_t* A, int64_t lda, const int32_t* idx, int n, int K, uint8_t* A2,
                              int64_t lda2, hipStream_t s);
hipError_t launch_scatter_rows(const int32_t* C2, const uint8_t* Cq2, const int32_t* flags2, const int32_t* idx, int n,
                               int N, int32_t* C, int64_t ldc, uint8_t* Cq, int64_t ldcq, int32_t* flags, hipStream_t s);
hipError_t launch_add_int(int32_t* dst, const int32_t* src, hipStream_t s);
hipError_t launch_gather_rows_bounded(const uint8_t* A, int64_t lda, const int32_t* idx, const int32_t* count, int limit, int K,
                                      uint8_t* A2, int64_t lda2, hipStream_t s);
hipError_t launch_scatter_rows_bounded(const int32_t* C2, const uint8_t* Cq2, const int32_t* flags2, const int32_t* idx,
                                       const int32_t* count, int limit, int N, int32_t* C, int64_t ldc, uint8_t* Cq, int64_t ldcq,
                                       int32_t* flags, hipStream_t s);
hipError_t launch_recount(const int32_t* count, const int32_t* cnt2, int limit, int32_t* err_count, int32_t* status,
                          hipStream_t s);
hipError_t launch_locate_correct(const uint8_t* A, int64_t lda, int M, const abft_packed_b* h, int32_t* C, int64_t ldc,
                                 int32_t* row_flags, int32_t* err_count, const RequantDev* rq, uint8_t* Cq, int64_t ldcq,
                                 int32_t* col_flags, int32_t* report, int32_t* scratch, hipStream_t s);
hipError_t launch_calib_copy(const void* src, void* dst, size_t bytes, hipStream_t s);
hipError_t launch_clock_probe(unsigned long long* out, unsigned long long ticks, hipStream_t s);
hipError_t launch_mfma_peak_probe(unsigned long long* out, int iters, hipStream_t s);
hipError_t launch_row_checksum(const uint8_t* A, int64_t lda, int M, int K, const int32_t* S_B,
                               int32_t* row_chk, hipStream_t s);

// Lets `kern` use `bytes` of dynamic LDS on the current device: the attribute belongs to the device, so it
// is set once per device and kernel (`done`: one bit per device ordinal, shared by the threads of the host)
inline hipError_t allow_dynamic_lds(const void* kern, size_t bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

// records `code` and a message for abft_last_error(); returns `code`
int set_error(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

}  // namespace abft
