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
// blocks.  One chain -> two, in us (three sets of handles in turn take the same, as they share the caller's side stream):
//   two blocks:  C = 96, 256 windows 43 -> 77; 392 54 -> 78; 840 79 -> 84; 1352 104 -> 101
//                C = 128, 920 95 -> 94        C = 192, 450 89 -> 100; 924 175 -> 170
//                C = 256, 480 128 -> 128; 1012 245 -> 241      C = 384, 192 114 -> 117; 300 159 -> 140; 450 236 -> 232
//   six blocks:  C = 96, 128 windows 110 -> 142; 392 166 -> 155        C = 128, 512 190 -> 171
//                C = 192, 98 170 -> 176; 200 204 -> 200       C = 256, 220 225 -> 219
//                C = 384, 40 215 -> 231; 70 217 -> 232; 192 335 -> 294
// Pruned windows count like the others: their share shortens both forms.
constexpr long long STAGE_SPLIT_MIN_WORK = 2200LL * 100;
inline bool stage_split_pays(int B, int nW, int C, int n_blocks) { return (long long)n_blocks * B * nW * C >= STAGE_SPLIT_MIN_WORK; }

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
