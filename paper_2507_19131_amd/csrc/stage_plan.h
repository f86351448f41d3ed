// Which stages run as two chains of blocks (see mixaq_stage_forward), and which images a chain takes when.  Host code.
#pragma once
#include <algorithm>

namespace mixaq {

// Two chains pay while the kernels of the stage leave CUs idle for part of their time (one chain -> two: a pair of blocks on 2784
// windows at C = 96 183 -> 174 us, on 1920 at 192 330 -> 314, on 1440 at 384 648 -> 602), up to this many windows in all.
constexpr int STAGE_SPLIT_MAX_WINDOWS = 4096;
// Each chain of a larger batch takes its half of the images in rounds of at most half this many windows, whole images: the tail of
// a kernel still runs beside the other chain's, and what a round reads again is nearer (a pair of blocks on 8 x 1392 windows at
// C = 96 689 -> 660 us, 4 x 1369 at 128 449 -> 442, 16 x 360 at 192 932 -> 897, 16 x 361 at 256 1392 -> 1357, 64 x 96 at 384 2597 -> 2490;
// as two halves without rounds 711 -> 697 and equal for the first two).  Not where the halves are uneven by more than an eighth
// (5 x 1392 at 96 416 -> 419, 3 x 2500 464 -> 467).
constexpr int STAGE_ROUND_WINDOWS = 5600;
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
inline int stage_rounds(int B, int nW)
{
    return (int)std::min<long long>(B / 2, ((long long)B * nW + STAGE_ROUND_WINDOWS - 1) / STAGE_ROUND_WINDOWS);
}

// images of the first (second) chain, and the most of them that one round takes
inline int chain_images(int B, int chain) { return (B + 1 - chain) / 2; }
inline int round_images(int B, int nW, int chain) { return (chain_images(B, chain) + stage_rounds(B, nW) - 1) / stage_rounds(B, nW); }

// the images of a chain's round
struct StagePart { int first, images; };
inline StagePart stage_part(int B, int nW, int chain, int round)
{
    const int n = chain_images(B, chain), rounds = stage_rounds(B, nW);
    const int from = (int)((long long)n * round / rounds), to = (int)((long long)n * (round + 1) / rounds);
    return {(chain ? chain_images(B, 0) : 0) + from, to - from};
}

}  // namespace mixaq
