// What a launch of the small heads' near form takes from the host beside the shape: both are worked out at every launch, in closed form.
#pragma once

namespace blossom {

// The short-term masks of the near form (mfma_f32.hip): bit l of own[r] is whether lane l's element r is seen in the row's (key's) own
// tile, of next[r] in the tile before (after) it.  Lane l = 16g + q holds the elements 4g + r of row q, at a distance of q - (4g + r), or
// 4g + r - q on the key's side, and of 16 more in the next tile; seen are the distances below the window and, under mask block 1, the
// powers of two.  A lane group's 16 bits are a stretch of the word of seen distances, or of that word turned round.  (Element by element
// 0.5 us of the host's time, so 0.02.)
struct NearMasks {
  unsigned long long own[4], next[4];
  NearMasks(int window, bool powers, bool key_side)  // 1 <= window <= 17
  {
    const unsigned seen = ((1u << window) - 1u) | (powers ? 0x10116u : 0u);  // bit d: distance d, 0 <= d < 32
    unsigned turned = 0u;                                                    // bit 31 - d
    for (int d = 0; d <= 16; ++d) turned |= (seen >> d & 1u) << (31 - d);
    for (int r = 0; r < 4; ++r) {
      own[r] = next[r] = 0ull;
      for (int g = 0; g < 4; ++g) {
        const int e = 4 * g + r;
        const unsigned o = key_side ? turned >> (31 - e) : seen << e, n = key_side ? turned >> (15 - e) : seen >> (16 - e);
        own[r] |= (unsigned long long)(o & 0xffffu) << (16 * g);
        next[r] |= (unsigned long long)(n & 0xffffu) << (16 * g);
      }
    }
  }
};

// Workgroups per unit of a launch whose tiles cost about the same: the number whose rounds of the chip (`slots` workgroups at a time)
// times a wavefront's tiles and its start, half a tile, are least, the smallest of several.  For a given number of tiles a wavefront
// the smallest number of workgroups is the one to look at.  (L = 16384: 0.6 us with every number of workgroups, so 0.3.)
// No more than kMostTiles a wavefront: rows of different lengths, which the host does not know, end together only where the workgroups are
// many.  (Backward at H=8, us, without that bound / with it, full rows and lengths U[L/10,L]: B=32 d=32 L=1600 503 / 505 and 372 / 339, d=32
// L=2200 690 / 698 and 390 / 343, d=16 L=2000 187 / 186 and 139 / 133, d=8 L=2000 128 / 130 and 94 / 95.)
constexpr int kMostTiles = 5;
inline int parts_that_end_together(int units, int tiles, int waves, int slots)
{
  int best = 0, parts = 1;
  for (int p = (tiles + waves * kMostTiles - 1) / (waves * kMostTiles);;) {
    const int each = (tiles + waves * p - 1) / (waves * p);
    const int cost = (units * p + slots - 1) / slots * (2 * each + 1);
    if (best == 0 || cost < best) {
      best = cost;
      parts = p;
    }
    if (each <= 1) return parts;
    p = (tiles + waves * (each - 1) - 1) / (waves * (each - 1));
  }
}

}  // namespace blossom
