// Which launches take a whole block in one kernel, a workgroup per window (block_kernel), instead of a window and a token kernel.  Host code.
#pragma once

namespace mixaq {

// By the windows of the launch and those of them that are not pruned; scored: the launch ranks its windows itself.  One kernel saves a
// launch, a round trip of the codes and the staging of the second half, but tiles of 32 and 17 rows instead of 32 and 32 cost a third more
// work, so it is for launches whose computed windows run all at once: one a CU, and at C = 96 and 128, whose registers hold two, a second one
// once most CUs have it (at C = 192 up to 64 workgroups of pruned windows wait behind those and only copy).  Below the first line of
// C = 128 and 192 the window kernel with half the heads a workgroup spreads a window over two CUs.  Two blocks on one map, us, two kernels /
// one:   C = 96   128 windows 33.2 / 31.1   256 37.1 / 32.9 | 264 41.8 / 42.4   320 43.0 / 44.0 | 400 46.5 / 44.7   504 48.9 / 45.9
//        C = 128  128 32.6 / 34.6 | 144 34.8 both   192 39.0 / 35.4   256 40.4 / 36.3 | 264 44.0 / 46.9   320 45.4 / 49.0 |
//                 400 51.6 / 50.3   504 58.0 / 53.5
//        C = 192  128 41.9 / 46.8 | 144 48.4 / 47.0   192 56.5 / 47.8   256 57.9 / 50.3 | 264 65.6 / 84.8   504 93.7 / 90.7
// C = 256 needs sixteen waves a workgroup, which have 128 registers and spill 35 to 44: 64 50.9 / 76.2, 256 75.8 / 88.7.
// Beside other streams' work the line would lie lower, as those fill the CUs that a launch leaves idle, but a call does not know of them.  Two blocks
// on each of so many streams at once, us a pass:   C = 96, 144 windows, two streams 28.7 / 23.0, three 28.8 / 22.5   256 28.2 / 25.0, 28.9 / 22.6   400
// 33.0 / 32.4, 29.2 / 29.3   504 37.6 / 39.1, 34.3 / 36.8      C = 128, 144 28.3 / 23.1, 29.1 / 22.6   256 29.1 / 27.2, 29.6 / 24.4   400 36.5 / 38.8,
// 34.2 / 35.8   504 43.6 / 45.2, 41.4 / 43.7      C = 192, 144 32.3 / 30.7, 28.4 / 26.3   196 38.2 / 36.6, 34.8 / 34.7   256 46.5 / 47.0, 51.3 / 48.1
// A batch that one launch takes this way stays on one chain: six blocks, two chains of two kernels / one chain of one:   C = 96   2 x 96
// windows 104.9 / 90.7   2 x 128 110.1 / 92.9   2 x 192 137.5 / 128.9   2 x 256 146.7 / 134.7      C = 128   2 x 96 115.9 / 100.6   2 x 128
// 121.3 / 104.0   2 x 192 145.1 / 144.2   2 x 256 159.4 / 153.7      C = 192   2 x 72 146.7 / 135.2   2 x 128 177.5 / 143.7.
// Given a list, a pruned window's workgroup copies its window behind the others: 2 x 140 with a fifth pruned 112.4 / 98.7, 126.2 / 110.9 and
// 184.7 / 160.0.  Where few are left the halves are ahead again (2 x 72 at C = 192, 115 computed 129.6 / 134.7).
// Given scores, a pruned window takes a place like any other until its rank is known, and beyond one workgroup a CU windows that are computed
// wait behind it: one block on 320 windows, 256 of them computed, 22.8 / 23.1, 24.7 / 26.2 and 36.3 / 46.5, 160 computed 21.6 / 23.0, 23.2 / 25.8
// and 32.7 / 35.0 (given a list 16.4 / 14.8, 18.5 / 16.7 and 28.7 / 25.1).  Near 512 all have a place (504, 353 computed at C = 96 25.2 / 24.3).
inline bool whole_block(int C, int windows, int computed, bool scored)
{
    constexpr int CUS = 256;
    const int from = C == 96 ? 0 : C == 128 || C == 192 ? 144 : 2 * CUS + 1, second = C == 96 ? 352 : C == 128 ? 400 : 2 * CUS + 1;
    if (computed <= CUS) return computed >= from && windows <= (scored ? CUS : CUS + CUS / 4);
    return computed >= second && windows <= 2 * CUS;
}

// Whether a stage of blocks that are one kernel each stays on one chain where two chains would be taken.  Up to 256 computed windows always.  Near
// 512 only while the stage is short: the fork is paid once, and per block two chains are the faster ones.  Two chains of two kernels / one
// chain of one, us:   C = 96   2 x 176 windows, 8 blocks 172.8 / 170.0   10 210.9 / 211.9   18 363.7 / 378.4      2 x 192, 12 blocks 255.3 / 255.2
//   2 x 224, 12 blocks 261.5 / 260.0   18 384.5 / 388.2      2 x 256, 12 blocks 275.1 / 267.4   24 529.1 / 533.9
//   C = 128  2 x 208, 8 blocks 189.7 / 193.2   18 398.4 / 431.3      2 x 224, 8 blocks 198.8 / 194.8   10 244.5 / 243.3   18 424.4 / 435.4
//   2 x 256, 8 blocks 205.6 / 203.0   10 252.2 / 252.6   18 439.4 / 453.6
inline bool whole_stage(int C, int windows, int computed, int n_blocks)
{
    if (!whole_block(C, windows, computed, false)) return false;
    return computed <= 256 || n_blocks <= (C == 96 ? (computed < 384 ? 8 : 12) : (computed < 448 ? 6 : 8));
}

}  // namespace mixaq
