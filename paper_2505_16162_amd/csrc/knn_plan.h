// Which kernel scans the anchor table: host code only, no HIP.
#pragma once
#include <stddef.h>

namespace ks {

// Scores of a workgroup of knn_rank_kernel: as many as its lanes hold in registers; one workgroup takes up to twice that, since a second
// one costs the hand-over (three queries, K = 8, 5000 anchors: 43 us a call in two slices, 37 in one; 8000: 43.5 / 42.8).
constexpr int KNN_SLICE = 4096;
// Routing over at least so many anchors ranks with knn_rank_kernel's slices instead of knn_argmax_kernel's one workgroup, whose time grows with the
// table; below, what the slices' hand-over costs is more. Whole calls in us, one workgroup / slices: rows of 256 elements, 1000 anchors 20.2 / 21.3,
// 8192 22.6 / 24.3, 12 000 24.2 / 24.8, 13 000 24.8 / 24.9, 14 000 25.1 / 25.1, 16 000 26.5 / 25.9, 100 000 75 / 44; 2048 elements, 12 000 34.5 / 35.2,
// 13 000 36.7 / 36.9, 14 000 37.4 / 37.0; 5120 elements, 8192 44.4 / 45.8, 13 000 60.7 / 60.9, 14 000 62.6 / 62.2, 100 000 344 / 313.
constexpr int KNN_RANK_ONE = 13500;
constexpr int KNN_STREAM_ROUND = 16384;      // anchors that knn_scores_stream_kernel's wavefronts take at a time: 256 x 16 wavefronts, four each

// knn_scores_stream_kernel, or knn_scores_multi_kernel? The first has its queries in LDS and keeps the table's loads rolling across
// anchors, so it gains with the queries per pass and with long rows; it loses what its workgroups spend on the queries in front, and what is
// dead of the last round of anchors. Whole K-best calls in us, multi / stream, with 2, 3 and 4 queries:
//   bf16, 2048 elements: 12 000 anchors 47.6 / 49.3, 49.6 / 51.0, 50.4 / 51.1; 32 768 68.1 / 61.1, 70.7 / 62.5, 70.8 / 63.5; 200 000 179 / 165,
//     197 / 175, 212 / 178; 5120 elements: 12 000 58.9 / 60.5, 63.2 / 62.4, 66.2 / 63.3; 32 768 93 / 89, 103 / 92, 111 / 93; 200 000 364 / 349,
//     417 / 365, 471 / 372; 1000 elements: 32 768 49.3 / 50.7, 51.8 / 52.3, 52.5 / 53.6; 200 000 100 / 105, 114 / 114, 124 / 117
//   fp32, 5120 elements: 16 384 92.5 / 90.3, 97.2 / 91.9, 105 / 93; 20 000 (1.2 rounds) -, 110 / 117, 114 / 118; 24 000 (1.5 rounds) 116 / 120,
//     126 / 122, 139 / 123; 4096 elements: 32 768 121 / 122, 139 / 124, 142 / 125; 2048: 32 768 78 / 80, 84 / 82, 88 / 81, 200 000 285 / 295, 290 / 304, 313 / 306; 1000:
//     32 768 58 / 60, 60 / 61, 62 / 62
//   short rows, 256 elements: fp32 32 768 46.6 / 45.5, 46.5 / 47.1, 48.1 / 46.8; 200 000 87 / 72, 80 / 79, 91 / 79; bf16 200 000 68 / 64, 80 / 74, 82 / 76
// One query: 200 000 x 5120 bf16 353 / 355, fp32 640 / 657. Over 492 sizes (64 to 8192 elements, 2000 to 200 000 anchors) the kernel chosen is
// 0.3 % slower than the better one in the mean, always the first 3.1 %.
inline bool knn_streams(int queries, bool bf16, int n, int d) {
    if (queries < 2) return false;
    if (bf16 ? d >= 2048 : (queries >= 4 ? d >= 2048 : queries == 3 ? d >= 4096 : d > 4096)) {
        // with fp32 rows the gain is smaller, and the last round has to be filled
        const long long rounds = bf16 ? 1 : (n + KNN_STREAM_ROUND - 1LL) / KNN_STREAM_ROUND;
        return queries >= 3 ? 10LL * n >= 7 * rounds * KNN_STREAM_ROUND : n >= KNN_STREAM_ROUND && (bf16 || 10 * rounds * KNN_STREAM_ROUND <= 11LL * n);
    }
    if (n >= 8 * KNN_STREAM_ROUND && (queries >= 4 || d <= 256)) return true;
    return !bf16 && d <= 256 && queries != 3 && n >= 2 * KNN_STREAM_ROUND;
}

}  // namespace ks
