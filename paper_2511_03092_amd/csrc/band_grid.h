// band_grid.h -- workgroups per group of band_rescore.  Host code, no HIP header
// needed.
#pragma once

namespace snap {

// A group's work items (blocks of its band keys, passes of score rows) are
// strided over its workgroups; short prompts have items for the first few only,
// and the others repeat the sorting of the members.
// 64- and 128-wide keys take 16 (8 groups: 10.8 us, 12.9 with 64).  576-wide
// ones (four row passes of long rows per key block) take 31, or 23 from 32 groups
// on (compress calls, 16 / 31 a group: 1 prompt of 131072 tokens, 8 heads, 608 /
// 600 us; 16 of them 1295 / 1287; 16 of 2048 tokens, 16 heads, 141 / 145).  From
// 64 groups on 16 fill the chip.
// The counts are odd: consecutive workgroups go round the 8 XCDs and, as measured
// times fit, an XCD's four shader engines, so with 32 or 64 the first workgroup
// of every group is on the same engine, which then does all the work of short
// prompts.  Compress calls with 16 / 64 or 1024 / groups / 31 or 23 a group: 8
// prompts of up to 2048 tokens, 2 latent heads, 141 / 154 / 142 us; 32 of up to
// 600, 1 head, 141 / 156 / 140; 16 of up to 600, 2 heads, 89 / 101 / 88.
inline int band_workgroups(int d_qk, int groups) {
  if (d_qk <= 128 || groups >= 64) return 16;
  return groups >= 32 ? 23 : 31;
}

}  // namespace snap
