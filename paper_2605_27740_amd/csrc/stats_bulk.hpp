// Which launches of the statistics kernel write their records past the caches. Host arithmetic on the launch's bounds only
// (no HIP), so that it can be checked without a GPU.
#pragma once
#include <stdint.h>

namespace unique {

// What bounds the bulk build is the mixture of a read stream with a few percent of writes: 131072 pages (4.29 GB of keys,
// 285 MB of records) take 635 us without any store; a plain stream of the same reads with the same writes beside it
// takes 874 to 893. A launch that writes more records than the caches hold therefore writes its means through in
// pieces of 1 KiB and its stds, 32 bytes of a line, non-temporally, with 4 items per wave: 896 us in a row with
// launches on other buffers and 835 after a kernel that only read, against 1013 and 855 with plain stores (8 items per wave
// 905 / 842; stds plain 943 / 830; all non-temporal 878 / 890).
// It needs stores that cover whole lines: a lane of bf16 keys has 32 bytes of fp32 means, which are two stores of every
// other 16 bytes (500 MB of records in a row / after a reading kernel: plain 1027 / 895 us, written through 1024 / 986). And it
// needs few of them among the reads. Plain / written through in a row, plain / written through after a reading kernel:
//   tiles (keys of one page and head) of 4 KiB, D = 128, 100 MB 342 / 334, 323 / 339; 140 MB 526 / 469, 449 / 440 (4 heads 500 / 451,
//   423 / 445); 200 MB 749 / 665,
//   637 / 621; 500 MB 1867 / 1657, 1617 / 1555; fp32 keys and means, 200 MB 744 / 635, 646 / 585
//   tiles of 2 KiB, D = 128, 200 MB 427 / 372, 365 / 373; 300 MB 650 / 556, 529 / 523
//   tiles of 2 KiB, D = 64, 300 MB 1091 / 992, 888 / 897; 500 MB 1745 / 1650, 1488 / 1525; of 1 KiB, 200 MB 444 / 475, 437 / 465
constexpr bool stats_bulk(int64_t record_bytes_written, int head_dim, int page_size, int key_bytes, bool bf16_means) {
  constexpr int64_t kMB = 1 << 20;
  const int tile = head_dim * page_size * key_bytes;
  if (key_bytes == 2 && !bf16_means) return false;
  if (tile >= 4096) return record_bytes_written > 144 * kMB;
  return tile >= 2048 && head_dim == 128 && record_bytes_written > 288 * kMB;
}

}  // namespace unique
