// Encode and pack the weight matrix (Algorithm 1 of arXiv 2103.00130: the rowSum[]
// loop and pack(B, rowSum[]); Section IV-A-3: the checksum is packed together with B
// so that the product kernel sees one encoded matrix).  Runs once per weight.
#include "abft_internal.h"

namespace abft {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));

// bytes at .. at + 15 of a row of len bytes, zeros past its end; nothing past the row is read
__device__ inline v4i load16(const int8_t* row, int at, int len) {
    if (at + 16 <= len) return *reinterpret_cast<const v4i_any*>(row + at);
    if (at >= len) return v4i{0, 0, 0, 0};
    if (len >= 16) return shift_down(*reinterpret_cast<const v4i_any*>(row + len - 16), at - (len - 16));
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < 16; ++b)
        if (at + b < len) w[b >> 2] |= (uint32_t)(uint8_t)row[at + b] << (8 * (b & 3));
    return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}

__device__ inline int32_t sum_bytes(v4i v, int32_t s) {
#pragma unroll
    for (int d = 0; d < 4; ++d) s = __builtin_amdgcn_sdot4(v[d], 0x01010101, s, false);
    return s;
}

// One pass over B: the packed units, and what the tile adds to the encoded column S_B (sums over the columns) and to the
// column sums of Eq. 1 (sums over k).  A workgroup takes one packed n-tile of 256 columns by 128 k, 32 KiB, eight 16-byte
// chunks per thread in flight at once; both sums are formed from the bytes in hand and leave with one integer atomic per row and per column
// of the tile (integer addition makes the order irrelevant).  They meet in accumulators of the weight's block that are zero before: encode_kernel, which
// takes them over, clears them again, so that a block that an earlier weight of these dimensions has left needs no kernel that does it ahead.
// Bound by memory: 9.4 us at 4096 x 4096 (and 3.6 of encode_kernel; 9.8 and 4.8 with the tiles' sums stored and added up there, which
// took 4.7 % of a weight's memory for as long as it lived), 134 us (4.0 TB/s, a large copy reaches 4.8) at 16384 x 16384, as a torch Linear
// holds it; 13 and 154 us with K along the rows.  Three passes, two of them strided, took 130 and 2900 us.
constexpr int kPackK = 128;
template <bool kTransposed>
__global__ __launch_bounds__(256) void pack_kernel(const int8_t* __restrict__ B, int64_t ldb, int K, int N, int KB,
                                                   v4i* __restrict__ packed, int32_t* __restrict__ row_sums, int32_t* __restrict__ col_sums,
                                                   int32_t* __restrict__ total) {
    __shared__ __align__(16) int8_t s_tile[kTileN * kPackK];
    __shared__ int32_t s_col[kTileN], s_row[kPackK];
    const int tid = threadIdx.x;
    const int ntile = blockIdx.y, k0 = blockIdx.x * kPackK, j0 = ntile * kTileN;
    v4i* const out = packed + ((int64_t)ntile * KB + blockIdx.x * 2) * (kUnitsPerTile * kUnitBytes / 16);   // 2048 chunks in order
    s_col[tid] = 0;
    if (tid < kPackK) s_row[tid] = 0;
    v4i v[8];
    if constexpr (kTransposed) {
        // rows of B are columns of the product: a chunk is sixteen consecutive bytes of one of them.  Chunk i*256 + tid
        // of the packed order: k-block, unit, k-group, column
        auto at = [&](int c, int& j, int& k) { j = ((c >> 7) & 7) * 32 + (c & 31); k = (c >> 10) * 64 + ((c >> 5) & 3) * 16; };
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            int j, k;
            at(i * 256 + tid, j, k);
            v[i] = j0 + j < N ? load16(B + (int64_t)(j0 + j) * ldb, k0 + k, K) : v4i{0, 0, 0, 0};
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            int j, k;
            at(i * 256 + tid, j, k);
            out[i * 256 + tid] = v[i];
            // a column's 128 bytes, its chunks XOR-swizzled so that the writes of 32 columns spread over the banks
            *reinterpret_cast<v4i*>(s_tile + j * kPackK + ((k >> 4) ^ (j & 7)) * 16) = v[i];
            atomicAdd(&s_col[j], sum_bytes(v[i], 0));
        }
        __syncthreads();
        // sums over the columns: four k per thread, 32 columns each
        const int dk = tid & 31, g = tid >> 5;
        int32_t s[4] = {0, 0, 0, 0};
#pragma unroll 8
        for (int j = g * 32; j < g * 32 + 32; ++j) {
            const int w = *reinterpret_cast<const int*>(s_tile + j * kPackK + ((dk >> 2) ^ (j & 7)) * 16 + (dk & 3) * 4);
#pragma unroll
            for (int b = 0; b < 4; ++b) s[b] = __builtin_amdgcn_sdot4(w, 1 << (8 * b), s[b], false);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) atomicAdd(&s_row[dk * 4 + b], s[b]);
    } else {
        // rows of B run along the columns of the product: the tile goes through LDS, and every thread turns blocks of
        // four columns by sixteen k
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = i * 16 + (tid >> 4), c = (tid & 15) * 16;
            v[i] = k0 + r < K ? load16(B + (int64_t)(k0 + r) * ldb, j0 + c, N) : v4i{0, 0, 0, 0};
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = i * 16 + (tid >> 4), c = (tid & 15) * 16;
            *reinterpret_cast<v4i*>(s_tile + r * kTileN + c) = v[i];
            // (the sixteen lanes of a DPP row hold one row of the tile)
            int32_t rs = sum_bytes(v[i], 0);
            rs += __builtin_amdgcn_update_dpp(0, rs, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
            rs += __builtin_amdgcn_update_dpp(0, rs, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
            rs += __builtin_amdgcn_update_dpp(0, rs, 0x141, 0xF, 0xF, true);  // row_half_mirror
            rs += __builtin_amdgcn_update_dpp(0, rs, 0x140, 0xF, 0xF, true);  // row_mirror
            if ((tid & 15) == 0) s_row[r] = rs;
        }
        __syncthreads();
        const int cq = tid & 63;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int kg = i * 4 + (tid >> 6);   // k-group of the tile, 0..7
            v4i q[4];                            // chunks of columns 4*cq .. + 3
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t w[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) w[b] = *reinterpret_cast<const uint32_t*>(s_tile + (kg * 16 + d * 4 + b) * kTileN + cq * 4);
                // 4x4 bytes turned: first pairs of rows, then pairs of pairs
                const uint32_t lo01 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400), hi01 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602);
                const uint32_t lo23 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400), hi23 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602);
                q[0][d] = (int)__builtin_amdgcn_perm(lo23, lo01, 0x05040100);
                q[1][d] = (int)__builtin_amdgcn_perm(lo23, lo01, 0x07060302);
                q[2][d] = (int)__builtin_amdgcn_perm(hi23, hi01, 0x05040100);
                q[3][d] = (int)__builtin_amdgcn_perm(hi23, hi01, 0x07060302);
            }
            v4i* const o = out + (kg >> 2) * 1024 + (cq >> 3) * 128 + (kg & 3) * 32 + (cq & 7) * 4;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                o[c] = q[c];
                atomicAdd(&s_col[cq * 4 + c], sum_bytes(q[c], 0));
            }
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid < 2) total[tid] = 0;   // (encode_kernel adds to it)
    if (j0 + tid < N && s_col[tid] != 0) atomicAdd(&col_sums[j0 + tid], s_col[tid]);
    if (tid < kPackK && k0 + tid < K && s_row[tid] != 0) atomicAdd(&row_sums[k0 + tid], s_row[tid]);
}

// Digit `digit` of s, the four signed base-256 digits: d0 in [-128,127] with s = d0 + 256*s1, and so on; the last digit
// is s3 reduced to 8 bits, which is exact modulo 2^32.
__device__ inline uint32_t digit_of(int32_t s, int digit) {
    uint32_t out = 0;
#pragma unroll
    for (int d = 0; d < kLimbs; ++d) {
        const int32_t dig = (int32_t)(((uint32_t)s + 128u) & 255u) - 128;
        if (d == digit) out = (uint32_t)dig & 255u;
        s = (int32_t)((uint32_t)s - (uint32_t)dig) >> 8;
    }
    return out;
}
__device__ inline void write_digits(int8_t* limbs, int k, int32_t s) {
#pragma unroll
    for (int d = 0; d < kLimbs; ++d) limbs[limb_offset(k, d)] = (int8_t)digit_of(s, d);
}
__device__ inline int32_t floor_mod127(int32_t s) {
    const int32_t r = s % 127;
    return r < 0 ? r + 127 : r;
}

// What follows from the finished encoded column: its digits, and for Algorithm 1 as printed (Section IV-A-2) rowSum[k] =
// S_B[k] mod 127 in [0,126], as an int32 array and, in the digit layout, as a single live digit column; the sums over k
// of both (wrap-around) go to total[0] and total[1].  One thread per digit of sixteen k, the digit layout's 16 bytes.
// Rows k >= K (padding) hold zeros.  The accumulators of pack_kernel are taken over and cleared: 1024 k a workgroup, then, behind the first
// n_row_blocks of the grid, 256 columns.
__global__ __launch_bounds__(256) void encode_kernel(v4i* __restrict__ row_sums, int32_t* __restrict__ col_sums, int n_chunks, int n_row_blocks, v4i* __restrict__ S_B,
                                                     v4i* __restrict__ limbs, v4i* __restrict__ S_B127, v4i* __restrict__ limbs127, int32_t* __restrict__ total,
                                                     int32_t* __restrict__ colsum) {
    if ((int)blockIdx.x >= n_row_blocks) {
        const int64_t j = (int64_t)((int)blockIdx.x - n_row_blocks) * 256 + threadIdx.x;
        colsum[j] = col_sums[j];
        col_sums[j] = 0;
        return;
    }
    __shared__ int32_t part[2];
    if (threadIdx.x < 2) part[threadIdx.x] = 0;
    const int t = blockIdx.x * 256 + threadIdx.x;
    const v4i* const src = row_sums + (t >> 2) * 4;
    const bool mine = t < n_chunks;
    __syncthreads();
    const int digit = t & (kLimbs - 1);
    int32_t s = 0, r = 0;   // sums of this thread's quarter of the sixteen
    if (mine) {
        v4i out, out127 = v4i{0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i v = src[q];
            v4i m;
            uint32_t w = 0, w127 = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                w |= digit_of(v[b], digit) << (8 * b);
                m[b] = floor_mod127(v[b]);
                w127 |= (uint32_t)m[b] << (8 * b);
            }
            out[q] = (int)w;
            if (digit == 0) out127[q] = (int)w127;
            if (digit == q) {
                S_B[t] = v;      // (chunk t of the array: group t / 4, its quarter)
                S_B127[t] = m;
                s = (int32_t)((uint32_t)v[0] + (uint32_t)v[1] + (uint32_t)v[2] + (uint32_t)v[3]);
                r = m[0] + m[1] + m[2] + m[3];
            }
        }
        limbs[t] = out;
        limbs127[t] = out127;
    }
    for (int off = 32; off > 0; off >>= 1) {
        s = (int32_t)((uint32_t)s + (uint32_t)__shfl_xor(s, off));
        r += __shfl_xor(r, off);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&part[0], s);
        atomicAdd(&part[1], r);
    }
    __syncthreads();
    if (mine) row_sums[t] = v4i{0, 0, 0, 0};   // (each chunk is read by four threads, on the other side of the barrier)
    if (threadIdx.x < 2) atomicAdd(&total[threadIdx.x], part[threadIdx.x]);
}

__global__ void flip_bit_kernel(int8_t* packed, int64_t off, int bit) {
    packed[off] = (int8_t)((uint8_t)packed[off] ^ (uint8_t)(1u << bit));
}

__global__ void flip_checksum_bit_kernel(int32_t* S_B, int8_t* limbs, int32_t* total, int k, int bit) {
    const uint32_t old = (uint32_t)S_B[k];
    const uint32_t now = old ^ (1u << bit);
    S_B[k] = (int32_t)now;
    write_digits(limbs, k, (int32_t)now);
    *total = (int32_t)((uint32_t)*total + (now - old));
}

// the same for the 8-bit column of Algorithm 1 as printed: rowSum[k] is one int8 in memory
__global__ void flip_checksum127_bit_kernel(int32_t* S_B127, int8_t* limbs127, int32_t* total127, int k, int bit) {
    const int32_t old = S_B127[k];
    const int32_t now = (int32_t)(int8_t)((uint8_t)old ^ (uint8_t)(1u << bit));
    S_B127[k] = now;
    write_digits(limbs127, k, now);
    *total127 = (int32_t)((uint32_t)*total127 + ((uint32_t)now - (uint32_t)old));
}

__global__ void fill_zero_kernel(int32_t* p, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace

hipError_t launch_pack(const int8_t* B, int64_t ldb, int transposed, abft_packed_b* h, hipStream_t s) {
    const dim3 grid((unsigned)(h->KB / 2), (unsigned)h->NT);
    v4i* const out = reinterpret_cast<v4i*>(h->packed);
    const int n_chunks = h->KB * kUnitK / 16 * kLimbs, n_row_blocks = (n_chunks + 255) / 256;
    int32_t* const col_sums = h->sums + (size_t)h->KB * kUnitK;
    if (!h->sums_zero) {
        const hipError_t e = launch_fill_zero(h->sums, (size_t)h->KB * kUnitK + (size_t)h->NT * kTileN, s);
        if (e != hipSuccess) return e;
    }
    h->sums_zero = false;
    if (transposed) pack_kernel<true><<<grid, dim3(256), 0, s>>>(B, ldb, h->K, h->N, h->KB, out, h->sums, col_sums, h->total);
    else pack_kernel<false><<<grid, dim3(256), 0, s>>>(B, ldb, h->K, h->N, h->KB, out, h->sums, col_sums, h->total);
    encode_kernel<<<dim3((unsigned)(n_row_blocks + h->NT)), dim3(256), 0, s>>>(
        reinterpret_cast<v4i*>(h->sums), col_sums, n_chunks, n_row_blocks, reinterpret_cast<v4i*>(h->S_B), reinterpret_cast<v4i*>(h->limbs),
        reinterpret_cast<v4i*>(h->S_B127), reinterpret_cast<v4i*>(h->limbs127), h->total, h->colsum);
    const hipError_t e = hipGetLastError();
    h->sums_zero = e == hipSuccess;
    return e;
}

hipError_t launch_flip_bit(abft_packed_b* h, int k, int j, int bit, hipStream_t s) {
    flip_bit_kernel<<<dim3(1), dim3(1), 0, s>>>(h->packed, packed_elem_offset(k, j, h->KB), bit);
    return hipGetLastError();
}

hipError_t launch_flip_checksum_bit(abft_packed_b* h, int k, int bit, hipStream_t s) {
    flip_checksum_bit_kernel<<<dim3(1), dim3(1), 0, s>>>(h->S_B, h->limbs, h->total, k, bit);
    return hipGetLastError();
}

hipError_t launch_flip_checksum127_bit(abft_packed_b* h, int k, int bit, hipStream_t s) {
    flip_checksum127_bit_kernel<<<dim3(1), dim3(1), 0, s>>>(h->S_B127, h->limbs127, h->total + 1, k, bit);
    return hipGetLastError();
}

hipError_t launch_fill_zero(int32_t* p, size_t n_ints, hipStream_t s) {
    if (n_ints == 0) return hipSuccess;
    fill_zero_kernel<<<dim3((unsigned)((n_ints + 255) / 256)), dim3(256), 0, s>>>(p, n_ints);
    return hipGetLastError();
}

}  // namespace abft
