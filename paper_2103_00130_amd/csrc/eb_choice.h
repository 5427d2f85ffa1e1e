// Which kernel runs a checked EmbeddingBag call (eb.hip): a rule on the host, by sizes alone.
#pragma once
#include <cstdint>

namespace abft {

// the batch kernel, or the group kernel with 1, 2 or 4 wavefronts per lookup
enum EbKernel { kEbBatch = 0, kEbGroup1 = 1, kEbGroup2 = 2, kEbGroup4 = 4 };

// work-items of the launch (a HIP launch takes fewer than 2^32); pieces: 16-byte pieces of a row's codes
inline int64_t eb_work_items(EbKernel kernel, int64_t n_bags, int pieces) {
    return kernel == kEbBatch ? (n_bags * pieces + 255) / 256 * 256 : n_bags * 64 * (int)kernel;
}
constexpr int64_t kEbMaxWorkItems = 0xffffffffll;

// Whether lookups of one or two wavefronts mark their loads of records as passing the caches by: tables of so many bytes that hardly a row
// that comes back is still in the 256 MiB of the memory-side cache (us, 16384 lookups of 100 rows of 80 bytes, fresh ones at every call, marked /
// not: tables of 320 MB 57.0 / 50.5, 1.3 GB 57.7 / 56.1, 2.6 GB 57.7 / 60.6, 5.1 GB 58.0 / 63.1; 4096 of 100 rows of 272 bytes, 0.5 GB 33.7 / 30.8,
// 2.2 GB 34.0 / 35.0; one wavefront each, 9000 of 27 rows of 80 bytes, 2.6 GB 12.8 / 13.6).  The batch kernel's handful of rows per lookup is
// faster without from any table (65536 of 4, 2.6 GB 18.3 / 17.4).
inline bool eb_passes_by(int64_t stride, int64_t rows) { return (uint64_t)stride * (uint64_t)rows > (3ull << 29); }

// The choice by the number of lookups and of rows per lookup on average (us, all rows 80 bytes unless said otherwise:
// batch / 4 / 2 / 1 wavefronts).  Few lookups: the latency of one counts and four wavefronts fetch more of it at once (300 of
// 30 rows 10.7 / 3.5 / 3.5 / 3.6; 600 of 60: 24.4 / 4.8 / 5.0 / 5.2; 10 of 100: 25.7 / 4.6 / 5.1 / 5.9), except for narrow rows
// of which there are hardly enough for one (300 of 5: 3.8 / 3.1 / 2.9 / 2.7).  Many lookups: what counts is how many are
// under way, and one wavefront each, without barriers and idle threads, takes the short ones (4000 of 16: 10.5 / 10.0 / 6.3 /
// 5.1; 9000 of 27: 18.4 / 22.0 / 12.4 / 12.3), two the long ones (3000 of 60, ragged: 78 / 14.2 / 12.3 / 13.2; records of 272
// bytes, 1500 of 100: 40 / 19.9 / 16.4 / 18.3; 16384 of 100: 66 / 70 / 56.6 / 56.7).  Very many lookups of a handful of rows: a few
// lanes per lookup (8000 of 4: 4.7 / 12.8 / 7.2 / 5.9; 16384 of 10: 10.8 / 32 / 15.8 / 14.1).
// With more lookups yet that holds for longer ones too: kEbBatchLines, by the width of a row (us, batch / 1 / 2 wavefronts,
// lengths between half and one and a half times the mean: 16 bytes of codes, 49152 lookups of 13 25.6 / 27.6 / 40, of 16 30.5 /
// 29.2 / 41, 196608 of 16 101 / 109 / 160, of 20 128 / 119 / 167; 32 bytes, 32768 of 13 18.6 / 20.4 / 29, of 20 25.5 / 25.2 / 32;
// 64 bytes, 65536 of 20 61 / 65 / 68, 98304 of 13 63 / 80 / 89, of 20 91 / 96 / 100, of 25 108 / 108 / 110; 128 bytes, 262144 of 16
// 262 / 270 / 323, of 20 320 / 311 / 361; 512 bytes, 16384 of 13 41.6 / 44.5 / 41.9, 65536 of 20 206 / 213 / 210, of 25 246 / 249 / 244).
// Lengths all alike gain more from it (64 bytes, 98304 of 12: 55 / 80), very different ones lose (128 bytes, 262144 of 14,
// geometric: 289 / 232), and the host does not know which they are.  Rows of 256 bytes have no line: 16384 of 12, 22.0 / 23.3 at
// best, 13 24.6 / 23.2, geometric 34 / 25.
struct EbBatchLine {
    int pieces;        // rows of so many pieces: ...
    int64_t lookups;   // from so many lookups on ...
    int mean;          // ... up to such a mean length
};
constexpr EbBatchLine kEbBatchLines[] = {{1, 49152, 15}, {1, 196608, 17}, {2, 32768, 17}, {4, 65536, 22}, {8, 262144, 17}, {32, 16384, 13}, {32, 65536, 22}};
inline EbKernel eb_pick_kernel(int64_t n_bags, int64_t n_indices, int pieces) {
    const int64_t avg = n_indices / n_bags;
    if (avg <= 5 ? n_bags >= 6000 : (avg <= 10 && n_bags >= 16000)) return kEbBatch;
    for (const EbBatchLine& l : kEbBatchLines)
        if (pieces == l.pieces && n_bags >= l.lookups && avg <= l.mean) return kEbBatch;
    if (n_bags < 1000) return avg <= 16 && pieces <= 4 ? kEbGroup1 : kEbGroup4;
    // Four wavefronts for long lookups of wide rows a little further (us, four / two): rows of 256 bytes while all lookups are
    // under way at once, four to a compute unit (4-bit, 1024 of 210 25.2 / 28.1, 1100 of 110 16.6 / 17.3 but 8-bit 14.7 / 13.8);
    // of 512 bytes longer (4-bit, 1400 of 110 30.1 / 34.2, 2600 of 210 81.8 / 89.8, 7000 of 110 115.6 / 118.0, 16000 of 110 251.8 /
    // 252.6; 8-bit, 1400 of 50 14.7 / 14.7, 2600 of 80 29.8 / 31.8, 4200 of 50 33.3 / 32.5, of 200 105.7 / 110.0); of 128
    // bytes where a lookup is one chunk with four and two with two (1100 of 50 6.8 / 7.4, of 110 10.9 / 10.6)
    const int64_t most4 = pieces == 32 && avg > 45 ? (avg > 80 ? 9999 : 3999) : pieces >= 16 || (pieces == 8 && avg > 80) ? 1024 : pieces == 8 && avg > 45 ? 1279 : 0;
    if (n_bags <= most4) return kEbGroup4;
    // fewer wavefronts where that many lookups make more work-items than a launch takes, a few lanes where one is too many too
    EbKernel kernel = avg <= 45 && pieces <= 16 ? kEbGroup1 : kEbGroup2;
    if (eb_work_items(kernel, n_bags, pieces) > kEbMaxWorkItems) kernel = kEbGroup1;
    return eb_work_items(kernel, n_bags, pieces) > kEbMaxWorkItems ? kEbBatch : kernel;
}

}  // namespace abft
