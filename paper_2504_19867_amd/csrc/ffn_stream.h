// Gated FFN, up to 128 tokens: how many units (16 gate and 16 up rows) a workgroup of the streaming kernel takes.  Host code.
#pragma once

namespace spd {

// `blocks`: of 16 tokens that the kernel's instance takes (1, 2, 4 or 8).  Four to eight units: a wave each.  Two or three: two waves share a unit's slices.
//
// A compute unit runs one workgroup at a time, and one of few waves takes longer per wave (few loads on the way): 64 tokens of hidden
// 4096, inter 7168, all workgroups at once, eight to four waves 53, 50.5, 45.7, 40.4, 35.8 us; 128 tokens 60 and 42.7 with eight and
// four (the x pieces of other counts do not fit their registers: 78 .. 86).  So the number of rounds decides.  64 tokens of
// inter 14336 (896 units), eight waves / the ones taken: 64 CUs 102 / 98 (7), 96 101 / 77 (5), 128 57 / 55.6 (7), 160 57 / 50 (6), 192 57 / 45.5
// (5), 256 57 / 43 (4); with only eight and four to choose from the first five took eight.
// Three or two units, each with two waves that halve the slices: for shares with more compute units than four units leave
// workgroups.  Hidden 8192, inter 7168 (448 units), 64 tokens, four units / the ones taken: 160 and 192 CUs 58 / 51 us (3), 256 58 / 42 (2); 1 token
// 46 / 40, 46 / 37; 128 tokens on 256 CUs 73 / 57 (2).  Where they take more rounds they lose (128 CUs, 64 tokens: 58 / 93, 70).  And where the
// halves are short: adding them up costs as much as what is saved, and a ring of sixteen slices takes hidden 512 at once (inter 512 .. 7168
// on 32 to 256 CUs, time without halves over time with them, on average: hidden 384 0.99 (1 token), 0.91 (17), 0.87 (40, 64, 100); 512 1.15,
// 1.07, 0.91 .. 0.92; 544 1.24, 1.17, 1.06 .. 1.12).
inline int ffn_stream_units(int blocks, int units, int K, int cus) {
  const int cost[] = {blocks <= 4 ? 52 : 57, 60, blocks <= 4 ? 68 : 71, 77, 87, 96, 100};   // of a workgroup of 2 .. 8 units
  const int fewest = K >= (blocks <= 2 ? 512 : 544) ? 2 : 4;
  int per_wg = 8;
  long least = 0;
  for (int n = 8; n >= fewest; --n) {
    if (blocks > 4 && n != 8 && n != 4 && n != 2) continue;
    const long wgs = (units + n - 1) / n, t = ((wgs + cus - 1) / cus) * cost[n - 2];
    if (n == 8 || t < least) {
      least = t;
      per_wg = n;
    }
  }
  return per_wg;
}

}  // namespace spd
