// Which kernel takes a linear layer of the separate kernels (see kernels.hip), by its sizes.  Host code.
#pragma once

namespace mixaq {

enum { EPI_QKV = 0, EPI_PROJ = 1, EPI_FC1 = 2, EPI_FC2 = 3 };
constexpr int CUS = 256;

// FEW: gemm_few_kernel.  RING64, RING128: gemm_ring_kernel on 64 x 64 or 128 x 128 tiles.  TILE: gemm_tile_kernel.
enum ProductForm { FEW, RING64, RING128, TILE };

// The projection and FC2 with K of the wide blocks at mlp_ratio 4.  Alone, over the number of 32 x 32 tiles, us, ring kernel / few-rows kernel:
//   FC2         C = 512   128 tiles 5.8 / 3.9   256 6.0 / 4.3   512 6.3 / 6.1   640 6.5 / 7.6      C = 768   192 7.4 / 4.5   384 7.8 / 6.7 |
//               576 8.0 / 8.9      C = 1024   256 9.1 / 5.4   512 10.1 / 8.6 | 768 10.7 / 11.9
//   projection  C = 512   128 3.6 / 3.6   256 3.7 / 3.7 | 512 3.9 / 4.5      C = 768   192 4.0 / 3.8 | 384 4.2 / 4.8
//               C = 1024   256 4.6 / 4.0 | 512 4.8 / 5.3
// Within a layer FC2's operands come from beyond the L2 (each XCD reads all rows for N / 256 blocks of channels: the likely reason why the line
// lies lower for small N).  A stage of two blocks, us, ring / few rows:
//   N = 512     K = 2048, 320 tiles 67.2 / 68.8   384 67.0 / 69.6      K = 3072   384 73.3 / 74.4   512 73.6 / 77.0      K = 4096   512 79.3 / 83.0
//   N = 256     K = 2048, 320 74.0 / 78.3   384 74.2 / 78.7
//   N = 768     K = 3072, 288 72.5 / 71.1   384 73.1 / 72.3      N = 1024   K = 2048, 512 76.1 both   K = 3072, 512 81.9 / 80.3   K = 4096, 512 85.9 / 84.9
// FC1 has four times FC2's tiles of a quarter of its K and gains at none of the three widths past the smallest map (C = 512, 512 tiles 4.1 / 3.9;
// C = 768, 768 tiles 4.7 / 5.3; C = 1024, 1024 tiles 5.3 / 6.7): it stays with the ring.
inline bool product_of_few_rows(int epi, int rows, int N, int K)
{
    const int wider = epi == EPI_FC2 ? 4 : 1, tiles = rows / 32 * (N / 32);
    return (epi == EPI_PROJ || epi == EPI_FC2) && N % 256 == 0 && (K == 512 * wider || K == 768 * wider || K == 1024 * wider) &&
           tiles <= (epi == EPI_PROJ || N < 768 ? CUS : 2 * CUS);
}

// Tiles of the ring kernel.  64 x 64: the fewest bytes in front of the first product and the most workgroups; 128 x 128: half the bytes per
// product.  Over the number of 128 x 128 tiles T, us, 64 x 64 / 128 x 128 (gemm_tile_kernel in brackets, which these layers took before):
//   FC1         C = 768    T = 48 4.6 / 9.2 (6.9)   240 8.8 / 10.0 (10.1)   336 11.6 / 10.9 (14.1)   672 19.9 / 15.9 (19.5)   3696 90 / 64 (95)
//               C = 512    32 4.1 / 7.7 (6.1)   320 9.4 / 9.2 (12.0)   608 15.4 / 12.7 (16.6)   1680 35.5 / 25.7 (40.3)
//               C = 1024   64 5.1 / 10.5 (7.5)   320 14.0 / 12.9 (15.5)   1280 45 / 32 (38.5)   3552 117 / 74 (96.8)
//   FC2         C = 768    12 7.4 / 17.0 (8.6)   60 8.4 / 17.8 (9.9)   168 18.4 / 20.6 (27.8)   330 33.3 / 29.7 (44.1)   924 79 / 64 (109)
//               C = 512    8 5.8 / 13.0 (10.3)   152 14.1 / 15.7 (23.5)   420 28.8 / 25.5 (38.3)
//               C = 1024   312 37.1 / 35.6 (53.0)   888 99 / 79 (127)
//   projection  C = 768    12 4.1 / 8.2 (5.2)   168 9.1 / 10.5 (11.1)   330 15.3 / 16.2 (18.7)   924 34.3 / 33.4 (39.4)
//               C = 512    152 7.8 / 8.9 (10.5)   420 15.6 / 15.6 (18.5)      C = 1024   312 15.4 / 18.2 (20.7)   888 37.8 / 37.4 (40.5)
// 64 x 128, 128 x 256 and 256 x 128 tiles lie between the two or behind them everywhere but at T = 330 (14.6 and 29.4).
// N = 128 (FC2 at C = 128): between one and five and a third 64 x 64 tiles a CU gemm_tile_kernel, whose four waves take a row tile's channels at
// once, where the ring's tiles pass the rows twice.  A stage of two blocks, us, tile / ring, K = 640, 768, 896 and 1024:
//   121 windows 66.3 / 63.5   69.1 / 66.4   73.3 / 69.5   74.0 / 70.7      156 69.4 / 68.4   72.5 / 72.1   73.3 both   73.6 / 74.2 |
//   182 74.2 / 75.7   74.1 / 77.1   76.2 / 78.5   79.1 / 81.9      324 85.2 / 85.1   89.6 / 92.0   93.0 / 96.3   95.0 / 96.7
//   506 113.3 / 112.2   120.3 / 125.0   127.0 / 130.6   133.3 / 137.7      650 129.5 / 131.6   134.0 / 140.1   142.5 / 146.8   148.8 / 149.5
//   870 164.9 / 165.1   172.4 / 174.6   182.7 / 183.8   189.3 / 191.2 |    960 176.3 / 172.0   182.8 / 179.9   187.6 / 187.2   195.0 / 196.0
//   1122 205.7 / 202.7   217.1 / 209.7   230.7 / 220.5   242.0 / 228.9
// Other widths have no such range (N = 192 650 windows 241 / 206, N = 256 309 / 267).
inline ProductForm product_form(int epi, int rows, int N, int K)
{
    if (K < 512 || K % 128 || N % 64) return TILE;                   // the ring takes whole stages and tiles, at least as many stages as it holds
    if (product_of_few_rows(epi, rows, N, K)) return FEW;
    const int tiles128 = N % 128 == 0 ? rows / 128 * (N / 128) : 0;
    if (N == 128 && 4 * tiles128 > CUS && 3 * tiles128 <= 4 * CUS && K <= 1024) return TILE;
    return tiles128 <= (epi == EPI_FC1 || K > 1024 ? CUS : 3 * CUS / 2) ? RING64 : RING128;
}

// FC1 on 64 x 64 tiles: a ring of three stages of two slabs, whose 39 KB let four workgroups on a CU, instead of four stages of four slabs, two
// workgroups.  Where the latter would run in rounds the former takes all tiles at once and a stage of fewer bytes starts sooner; with at most a
// workgroup or so a CU it waits for its operands more often.  A stage of two blocks over the number of 64 x 64 tiles, us, four slabs / two:
//   C = 512   128 tiles 58.1 / 59.1   256 62.0 / 62.2   512 67.8 / 68.0 | 640 72.3 / 70.2   896 74.7 / 73.1
//   C = 768   192 63.2 / 65.0   384 72.4 / 72.5 | 576 78.3 / 75.5   768 79.5 / 76.9   960 84.5 / 82.5
//   C = 1024  256 71.1 / 72.1   512 85.2 / 84.1 | 768 92.0 / 88.0   1024 98.2 / 94.0
// (Two slabs in four stages, three workgroups: between the two.  The projection and FC2, which have a quarter of the tiles, lose up to 8 %.)
inline bool fc1_ring_of_four(int rows, int N) { return rows / 64 * (N / 64) > 2 * CUS; }

}  // namespace mixaq
