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

// The choice by the number of lookups and of rows per lookup on average (us, all rows 80 bytes unless said otherwise:
// batch / 4 / 2 / 1 wavefronts).  Few lookups: the latency of one counts and four wavefronts fetch more of it at once (300 of
// 30 rows 10.7 / 3.5 / 3.5 / 3.6; 600 of 60: 24.4 / 4.8 / 5.0 / 5.2; 10 of 100: 25.7 / 4.6 / 5.1 / 5.9), except for narrow rows
// of which there are hardly enough for one (300 of 5: 3.8 / 3.1 / 2.9 / 2.7).  Many lookups: what counts is how many are
// under way, and one wavefront each, without barriers and idle threads, takes the short ones (4000 of 16: 10.5 / 10.0 / 6.3 /
// 5.1; 9000 of 27: 18.4 / 22.0 / 12.4 / 12.3), two the long ones (3000 of 60, ragged: 78 / 14.2 / 12.3 / 13.2; records of 272
// bytes, 1500 of 100: 40 / 19.9 / 16.4 / 18.3; 16384 of 100: 66 / 70 / 56.6 / 56.7).  Very many lookups of a handful of rows: a few
// lanes per lookup (8000 of 4: 4.7 / 12.8 / 7.2 / 5.9; 16384 of 10: 10.8 / 32 / 15.8 / 14.1; 80000 of 20: 74 / 176 / 82 / 78).
inline EbKernel eb_pick_kernel(int64_t n_bags, int64_t n_indices, int pieces) {
    const int64_t avg = n_indices / n_bags;
    if (avg <= 5 ? n_bags >= 6000 : (avg <= 10 && n_bags >= 16000)) return kEbBatch;
    if (n_bags < 1000) return avg <= 16 && pieces <= 4 ? kEbGroup1 : kEbGroup4;
    // fewer wavefronts where that many lookups make more work-items than a launch takes, a few lanes where one is too many too
    EbKernel kernel = avg <= 45 && pieces <= 16 ? kEbGroup1 : kEbGroup2;
    if (eb_work_items(kernel, n_bags, pieces) > kEbMaxWorkItems) kernel = kEbGroup1;
    return eb_work_items(kernel, n_bags, pieces) > kEbMaxWorkItems ? kEbBatch : kernel;
}

}  // namespace abft
