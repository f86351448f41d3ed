// Which stages run as two chains of blocks (see mixaq_stage_forward), and which images a chain takes when.  Host code.
#pragma once
#include <algorithm>

namespace mixaq {

// Two chains pay while the kernels of the stage leave CUs idle for part of their time: up to this many windows in all also for an odd
// batch (one chain -> two: a pair of blocks on 2790 windows at C = 96 181 -> 175 us, on 2888 at 192 452 -> 443, on 1536 at 384
// 640 -> 633).  Beyond, two launches fill the chip either way and only even halves still gain (2 x 2500 at 96 303 -> 296, at 128 407 ->
// 404, at 192 812 -> 797, at 256 1214 -> 1219, at 384 2178 -> 2143; 4 x 1392 at 96 328 -> 322, 4 x 1369 at 128 438 -> 435); where they are
// uneven by more than an eighth the two forms are equal (5 x 1392 at 96 406 both, 3 x 2500 449 and 445).
constexpr int STAGE_SPLIT_MAX_WINDOWS = 4096;
// A chain goes through its half of the images in rounds, whole images, all blocks of a round before the next, so that what a block reads
// was written shortly before.  A round is about this many windows times channels, a map of 53 MB, to the nearest: two chains then
// have about four such maps in use, which is near the 256 MB of the last-level cache (the likely reason; the counters count in front
// of that cache and cannot show it), and a line drawn at windows alone misses the wide maps.  A pair of blocks as halves without
// rounds -> in rounds, us (three sets of handles in turn; the number of rounds in brackets, the rule's own first):
//   C = 96   8 x 1392 windows 682 -> [2] 653, [4] 658      16 x 1392 1390 -> [4] 1313, [3] 1328, [5] 1325
//            16 x 360 331 -> [2] 337       24 x 360 502 -> [2] 503, [3] 515      6 x 1392 493 -> [1], [2] 488, [3] 496
//   C = 128  8 x 1369 938 -> [3, 4] 873, [2] 876      4 x 1369 435 -> [2] 443       16 x 361 451 -> [2] 451, [4] 482
//   C = 192  16 x 360 911 -> [2] 875, [3] 889, [5] 910      32 x 360 1856 -> [4] 1761, [6] 1778      8 x 361 444 -> [2] 450
//   C = 256  16 x 361 1374 -> [3] 1321, [2] 1330, [5] 1340      12 x 361 1012 -> [2] 997, [4] 1019     8 x 361 670 -> [2] 660
//   C = 384  64 x 96 2494 -> [5] 2417, [3] 2441, [2] 2490      32 x 96 1261 -> [2] 1224, [3] 1232      15 x 96 (six blocks) 1665 -> [2] 1701
//            48 x 96 (six blocks) 5453 -> [4] 5198, [2] 5353      28 x 96 (six blocks) 3128 -> [2] 3028, [3] 3081
constexpr long long STAGE_ROUND_WORK = 2800LL * 96;
// Fork and join cost 25 to 30 us, so the stage has to be long enough: the line is drawn at windows times channels over all its
// blocks.  And a chain has to leave the other one something: up to this many windows one chain's launches are at most about one
// workgroup per CU, as long as those of half the images, and two chains lose at every number of blocks.  One chain -> two, us
// (three sets of handles in turn, which share the caller's side stream):
//   two blocks:    C = 96, 396 windows 49 -> 73; 850 77 -> 80; 1200 90 -> 96; 1344 99 -> 99; 1610 117 -> 115
//                  C = 128, 588 68 -> 76; 918 89 -> 92; 1064 105 -> 100      C = 192, 456 87 -> 98; 520 119 -> 111; 588 128 -> 117
//                  C = 256, 300 88 -> 100; 396 118 -> 113; 480 121 -> 125; 560 149 -> 144; 768 186 -> 188; 850 213 -> 205
//                  C = 384, 120 74 -> 91; 234 119 -> 120; 300 159 -> 140; 456 211 -> 202
//   six blocks:    C = 96, 252 119 -> 132; 300 138 -> 136; 396 153 -> 147      C = 128, 234 126 -> 133; 288 143 -> 141; 340 154 -> 148
//                  C = 192, 154 157 -> 165; 182 185 -> 169; 234 186 -> 189; 288 209 -> 194
//                  C = 256, 140 182 -> 196; 154 184 -> 198; 182 223 -> 203; 252 227 -> 227; 340 304 -> 277
//                  C = 384, 72 209 -> 225; 108 212 -> 226; 140 243 -> 239; 154 248 -> 256; 192 340 -> 282
//   twelve:        C = 96, 192 229 -> 235; 288 275 -> 250      C = 128, 154 218 -> 231; 192 244 -> 239      C = 192, 100 269 -> 296; 132 309 -> 304
//                  C = 256, 108 324 -> 358; 140 361 -> 369      C = 384, 72 414 -> 431; 120 424 -> 443; 140 484 -> 452
//   eighteen (24): C = 96 (132 407 -> 435; 192 459 -> 449)      C = 128 (132 424 -> 434; 192 489 -> 460)      C = 192, 100 403 -> 434; 132 463 -> 445
//                  C = 256, 100 482 -> 522; 154 542 -> 548; 182 660 -> 563      C = 384, 72 627 -> 645; 120 657 -> 673; 132 753 -> 694
// Pruned windows count like the others: their share shortens both forms.
constexpr long long STAGE_SPLIT_MIN_WORK = 2200LL * 100;
constexpr int STAGE_SPLIT_MIN_WINDOWS = 128, STAGE_SPLIT_MIN_WINDOWS_256 = 160;     // at C = 256
inline bool stage_split_pays(int B, int nW, int C, int n_blocks)
{
    return B * nW > (C == 256 ? STAGE_SPLIT_MIN_WINDOWS_256 : STAGE_SPLIT_MIN_WINDOWS) && (long long)n_blocks * B * nW * C >= STAGE_SPLIT_MIN_WORK;
}

// whether the map allows two chains
inline bool stage_splits(int B, int nW)
{
    const bool small = B * nW <= STAGE_SPLIT_MAX_WINDOWS, even = B % 2 == 0 || B >= 9;
    return B >= 2 && (small || even);
}

// rounds in which the two chains of such a stage go through their images
inline int stage_rounds(int B, int nW, int C)
{
    const long long work = (long long)B * nW * C / 2;                // of a chain
    return (int)std::max<long long>(1, std::min<long long>(B / 2, (work + STAGE_ROUND_WORK / 2) / STAGE_ROUND_WORK));
}

// images of the first (second) chain, and the most of them that one round takes
inline int chain_images(int B, int chain) { return (B + 1 - chain) / 2; }
inline int round_images(int B, int nW, int C, int chain)
{
    const int rounds = stage_rounds(B, nW, C);
    return (chain_images(B, chain) + rounds - 1) / rounds;
}

// the images of a chain's round
struct StagePart { int first, images; };
inline StagePart stage_part(int B, int nW, int C, int chain, int round)
{
    const int n = chain_images(B, chain), rounds = stage_rounds(B, nW, C);
    const int from = (int)((long long)n * round / rounds), to = (int)((long long)n * (round + 1) / rounds);
    return {(chain ? chain_images(B, 0) : 0) + from, to - from};
}

}  // namespace mixaq
