// How a prompt on the any-shape kernels is put on the stream: plain code, no HIP.
#pragma once
#include "../../include/knnssd.h"
#include "device_types.h"

namespace ks {

constexpr int PR_CHUNK = 8, PR_ROWS = 256;     // rows of a chunk; of the chunks side by side, at most

// Rows of a prompt of n rows that go side by side (as chunks, in launches of at most so many rows); 0: 16-row passes one after the other.
// Against passes, rows side by side, whole prompts, us:
//   fp32: always. Two blocks of 520 columns, 17 rows 222 / 105, 250 rows 2362 / 348; 4104 columns 1553 / 1214 and 18 627 / 10 474; one block of 8008 columns
//     3299 / 2381 and 42 255 / 24 299. One block of 64 to 192 columns and 17 rows 68-74 / 62-66 (82 on a machine whose launches cost more).
//   bf16, up to 2800 columns: always. 1000 columns 17 rows 246 / 134, 250 rows 2734 / 743; 2504 columns, one block, 305 / 248 and 3377 / 2227.
//   Wider bf16 rows: a 16-row pass streams its weights twice as fast as fp32 ones, and the rows' way through the L1 is what chunks are bound by. A prompt whose
//     last chunk has few rows then loses: one block, 17, 25, 32 and 33 rows: 3000 columns 343 / 309, 432 / 406, 516 / 418, 594 / 481; 3600 438 / 464, 538 / 597,
//     642 / 636, 742 / 712; 4304 593 / 635, 725 / 805, 889 / 862, 1024 / 963; 4808 769 / 915, 1011 / 1173, 1178 / 1272, 1343 / 1424 (40 rows 1528 / 1543, 64 2328 / 2328);
//     5704 and 40 rows 1822 / 1858, 64 2780 / 2836. 6008 columns lose at every length (64 rows 2929 / 3129), 8008 and 6600 are 0.91 to 1.02 of passes from 64 rows on.
//   256 such rows side by side no longer lie in a die's L2 (250 rows in launches of 256 / 128: 3000 columns 3005 / 2771, 4104 7905 / 7100, 5128 10 329 / 8977, passes
//     3903, 8067, 9653); with fp32 weights it makes no difference (5128 columns 18 900 / 18 100), and narrow rows fill the chip better the more of them there are
//     (520 columns 371 / 410).
inline int prompt_rows(const knnssd_model_cfg &g, int n) {
    if (n <= KS_MAX_ROWS) return 0;
    const int d = g.d_model;
    if (g.weight_dtype == KNNSSD_FP32 || d <= 2800) return PR_ROWS;
    if (d > 5600 || n <= (d > 4700 ? 40 : (d > 3200 ? 32 : KS_MAX_ROWS))) return 0;
    const int launches = (n + PR_ROWS / 2 - 1) / (PR_ROWS / 2), rows = (n + launches - 1) / launches;      // as equal as whole passes' rows allow
    return (rows + KS_MAX_ROWS - 1) / KS_MAX_ROWS * KS_MAX_ROWS;
}

}  // namespace ks
