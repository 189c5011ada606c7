// Which attention kernel a batch takes (host code without device types, so that
// it can be compiled and checked by itself).
#pragma once

#include <algorithm>
#include <cstdint>

namespace {

// The item kernel keeps two waves per SIMD for these accumulator columns
// (head_dim x 16-row tiles).
constexpr bool two_waves_per_simd(int columns) { return columns <= 384; }

// How a batch runs: the most chunks the item kernel cuts an item into (1: none
// is cut), or 0 for the wave-split kernel.  items = requests x KV heads, b =
// K/V bytes of the longest context the call can hold per item, d: head_dim, mt:
// 16-row tiles, slots: partial slots of the workspace.
//
// The item kernel has no prologue over the batch, no merge launch when nothing
// is cut, and the hardware hands its workgroups to free CUs; but a whole item's
// time is bound by one CU (about 49 bytes per ns), the fused pass loses the
// order that keeps the writes together, and every item pays its start and end.
// The host knows the longest context but not the others, so a whole item is
// taken only where one CU's time for the longest (past one item per CU: for two of
// them that meet on one CU) stays below what the wave split takes for a batch
// whose other contexts are short, and with larger tiles (whose start and end cost
// more) for few items per CU.  Lines measured on MI355X (us, wave-split kernel as
// it was before the item kernel -> item kernel; 32/8 heads, D 128, K = 4 unless
// said; items x longest context, the others uniform from a quarter of it, or after
// "k of" k such contexts among ones of 16-64 tokens):
//   whole items, read only: 192 x 1024 33 -> 18, 256 x 2048 43 -> 35, 1 of 256 x
//     2048 34 -> 25, but 1 of 256 x 4096 38 -> 44 and (16/8 heads, K = 0) 31 -> 41,
//     so nothing past 1 MiB although 256 x 4096 is 62 -> 59; D 64: 16 of 256 x 4096
//     31 -> 26, 1 of 192 x 8192 31 -> 43;
//     past one item per CU 8 of 512 x 1536 45 -> 24, but 8 of 400 x 2048 among
//     256-512 44 -> 50 (although 512 x 2048 is 67 -> 61), with one 16-row tile (16/1
//     heads, K = 0) 64 of 512 x 2048 41 -> 46 and (16/8) 8 of 400 x 1536 among 256-512
//     35 -> 38, 64 of 512 x 1024 36 -> 26; D 64: 32 of 512 x 3072 30 -> 35, 64 of 1024 x
//     2048 34 -> 38, 64 of 1024 x 1536 32 -> 29;
//   items per CU, read only: one tile of D 128 16384 x 128 147 -> 124, 8192 x 512
//     236 -> 230, 1 of 16384 x 128 90 -> 86; two tiles of D 64 16384 x 512 293 ->
//     256; two of D 128 1 of 2048 x 256 33 -> 30, 1 of 8192 x 256 68 -> 83; three of
//     D 128 1 of 2048 x 256 72 -> 43, 4096 x 256 100 -> 105, 1 of 8192 x 256 110 ->
//     149; 64 rows of D 64 1 of 4096 x 256 52 -> 59;
//   cut items, read only: 8 x 32001 39 -> 31, 8 x 4096 21 -> 14, 64 x 4096
//     32 -> 27, 128 x 4096 45 -> 41, 64 x 16000 even (128 x 16000 124 -> 133);
//   whole items, fused, 30 % arriving: 32 x 256 30 -> 9, 256 x 1024 49 -> 31,
//     512 x 1024 66 -> 56 (2048 x 1024 179 -> 186), 2048 x 512 108 -> 97; 8 of 256 x
//     1536 60 -> 37, but D 64: 1 of 192 x 4096 38 -> 41, so nothing past 768 KiB
//     although 256 x 2048 is 61 -> 51; one tile of D 64 16384 x 512 193 -> 173 (8192
//     x 1024 320 -> 352);
//   cut items, fused: 32 x 1024 35 -> 13, 32 x 4096 37 -> 20, 64 x 4096
//     44 -> 33, 128 x 4096 60 -> 57 (128 x 16000 180 -> 214);
//   64 rows at head_dim 128 (one wave per SIMD): 512 x 1024 57 -> 52 (2048 x
//     1024 173 -> 179, 64 x 4096 41 -> 56).
inline int item_split(int64_t items, int64_t b, int d, int mt, bool fuse, int cus,
                      int64_t slots) {
  constexpr int64_t KB = 1024, MB = 1024 * KB;
  const bool two_waves = two_waves_per_simd(d * mt);
  const int64_t total = items * b;
  const int few = two_waves ? cus / 2 : cus / 16;   // so few items leave CUs idle: cut them
  if (items <= few && b > (fuse && two_waves ? 256 : 512) * KB) {
    const bool cut = !two_waves ? total <= 64 * MB
                     : fuse     ? b <= 2 * MB || total <= 150 * MB
                                : total <= 400 * MB;
    if (!cut) return 0;
    // twice the workgroups aimed at: the longest context may take two shares
    return (int)std::max<int64_t>(1, std::min(slots / items, (4 * cus + items - 1) / items));
  }
  if (!two_waves) return b <= 512 * KB && items <= 2 * cus;
  const int64_t many = (d * mt <= 128 ? 64 : 8) * cus;   // (64 per CU: the most measured)
  if (fuse)
    return (b <= 128 * KB && items <= many) || (b <= 256 * KB && items <= 8 * cus) ||
           (b <= 512 * KB && items <= 2 * cus) || (b <= 768 * KB && items <= cus);
  return (b <= (d == 64 ? 384 : 512) * KB && items <= many) ||
         (b <= 768 * KB && items <= 2 * cus && d == 128 && mt > 1) || (b <= MB && items <= cus);
}

}  // namespace
